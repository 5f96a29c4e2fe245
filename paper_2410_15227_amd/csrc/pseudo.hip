// Tree-node pseudo-particles (Sec. 2.4).
//
// The gravity tree here is an octree of the unit cube built from 63-bit
// Morton keys: a node at level l is a run of particles sharing the top 3l key
// bits, a node with more than leaf_max particles (and below max_depth) splits
// into the runs of its next 3-bit digit (child order = octant order x = 1,
// y = 2, z = 4).  Node position is the centre of mass and node size the
// distance from it to the furthest member (Sec. 2.2.1).  So that a host
// reference reproduces the accepted set bit for bit, node sums are formed in a
// fixed order without contraction: a leaf adds its members in ascending
// particle index, an internal node adds its children's sums in octant order.
//
// Walk (Sec. 2.2.2, Sec. 2.4.1): a node is emitted when it is accepted and no
// ancestor is; a leaf that is not accepted and has no accepted ancestor is
// opened and its particles are emitted as themselves (they keep their h).
// Acceptance: for every source, r - s > r_part and not (theta^2 r^2 < s^2)
// (eq. opening_angle).  Each emitted node or opened leaf is one "unit"; the
// units tile the particle order, so depth-first emission order is the order
// of their first particle.
//
// Node smoothing lengths (Sec. 2.4.2, eqs. h_node, n_node, hnode_func,
// hnode_func_deriv, hnode_newton_raphson, hnode_estval): n(h) sums
// W(|r_a - r_b|, h) over all units b (opened leaves stand in for their
// particles; self term included).  Newton from h0 = h_fact 2 s to
// |h_new - h| / h0 < eps_h; Newton fails after 30 steps, when an iterate
// leaves [1e-2 h0, 1e2 h0] or when |f'| < 1e-12; then bisection on
// [1e-2 h0, 1e2 h0] when f changes sign there, else h0.  Newton's sums over
// units are those of unit order: one wavefront per pseudo-particle, or a
// workgroup where the node meets many units (the same sums, bit for bit).
// The nodes Newton leaves go to a third kernel, 16 wavefronts per node, whose
// bracket and bisection steps decide from bounds of 64-unit boxes, then from
// fixed-order tree sums in binary32, then from the unit-order sums, each
// where the one before leaves the sign within its rounding margin, so every
// decision is that of the unit-order sums.
#include "common.hpp"

namespace sphmap {
namespace {

constexpr int kMaxLevels = 22;

struct NodeArrays {
  int32_t *first, *count, *parent, *child_first, *nchild, *level;
};

__global__ void k_check_unit_cube(int64_t n, const double *xyz, int *bad) {
  int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= n) return;
  for (int k = 0; k < 3; ++k) {
    double x = xyz[3 * i + k];
    if (!(x >= 0.0 && x < 1.0)) {
      atomicAdd(bad, 1);
      return;
    }
  }
}

__global__ void k_root(NodeArrays N, int64_t n, int64_t *lv) {
  lv[0] = 0;  // nodes a level lacked room for
  lv[1] = 0;  // the levels' first nodes
  lv[2] = 1;
  N.first[0] = 0;
  N.count[0] = (int32_t)n;
  N.parent[0] = -1;
  N.level[0] = 0;
  N.child_first[0] = -1;
  N.nchild[0] = 0;
}

__device__ inline int digit_of(uint64_t key, int level) {
  // digit selecting the child at `level` (1 = first split below the root)
  return (int)((key >> (3 * (21 - level))) & 7ull);
}

// A level's nodes are [lv[0], lv[1]), at most nb; eight lanes a node, one for
// each octant d, lane t & 7 of node t >> 3.  The launches step through the
// level (strided_blocks): nb is a bound of up to n, and eight lanes each of
// 2^29 nodes are more than one launch takes.
struct Octant {
  int32_t first, count;  // the octant's run of the node's particles
  uint32_t some;         // bit per octant: not empty
  int64_t node;          // -1: no node
};
__device__ __forceinline__ Octant octant_of(const NodeArrays &N, const int64_t *lv, int64_t nb, int64_t t, int level,
                                            const uint64_t *keys, int leaf_max, int max_depth) {
  const int64_t j = t >> 3;
  const int d = (int)t & 7, lane = threadIdx.x & 63;
  Octant o{0, 0, 0u, j < nb && lv[0] + j < lv[1] ? lv[0] + j : -1};
  int32_t f = 0, a = 0;
  if (o.node >= 0) {
    f = N.first[o.node];
    const int32_t c = N.count[o.node];
    a = f;
    if (c > leaf_max && level < max_depth) {
      int32_t z = f + c;  // first position whose digit exceeds d
      if (d == 7) a = z;
      while (a < z) {
        const int32_t mid = a + (z - a) / 2;
        if (digit_of(keys[mid], level + 1) <= d) a = mid + 1;
        else z = mid;
      }
    }
  }
  const int32_t prev = __shfl_up(a, 1, 8);
  o.first = d ? prev : f;
  o.count = a - o.first;
  o.some = (uint32_t)(__ballot(o.count > 0) >> (lane & 56)) & 0xffu;
  return o;
}

// children per node of the level
__global__ void k_split(NodeArrays N, const int64_t *lv, int64_t nb, int level, const uint64_t *keys, int leaf_max,
                        int max_depth, int64_t *nch) {
  for (int64_t t0 = (int64_t)blockIdx.x * 256; t0 < 8 * nb; t0 += (int64_t)gridDim.x * 256) {
    const int64_t t = t0 + threadIdx.x;
    const Octant o = octant_of(N, lv, nb, t, level, keys, leaf_max, max_depth);
    if ((t & 7) == 0 && (t >> 3) < nb) nch[t >> 3] = __popc(o.some);
  }
}

// The children and the next level's range; where they do not fit in cap nodes
// nothing but the number that was lacking room (the next level is then empty,
// and so are those after it).
__global__ void k_children(NodeArrays N, int64_t *lv, int64_t *lacking, int64_t nb, int64_t cap, int level,
                           const uint64_t *keys, int leaf_max, int max_depth, const int64_t *choff) {
  const int64_t next = lv[1], total = choff[nb];
  const bool fits = next + total <= cap;
  if (blockIdx.x == 0 && threadIdx.x == 0) {
    lv[2] = fits ? next + total : next;
    if (!fits) *lacking = total;
  }
  if (!fits) return;
  for (int64_t t0 = (int64_t)blockIdx.x * 256; t0 < 8 * (next - lv[0]); t0 += (int64_t)gridDim.x * 256) {
    const int64_t t = t0 + threadIdx.x;
    const Octant o = octant_of(N, lv, nb, t, level, keys, leaf_max, max_depth);
    if (o.node < 0) continue;
    const int d = (int)t & 7;
    const int64_t first = next + choff[t >> 3];
    if (d == 0) {
      N.nchild[o.node] = __popc(o.some);
      N.child_first[o.node] = o.some ? (int32_t)first : -1;
    }
    if ((o.some >> d) & 1u) {
      const int64_t cid = first + __popc(o.some & ((1u << d) - 1u));
      N.first[cid] = o.first;
      N.count[cid] = o.count;
      N.parent[cid] = (int32_t)o.node;
      N.level[cid] = level + 1;
      N.child_first[cid] = -1;
      N.nchild[cid] = 0;
    }
  }
}

// Leaves: sums over members in ascending particle index.  A leaf whose
// members already lie in ascending index (every leaf at the depth limit:
// its members share the whole key, and the key sort is stable) is summed in
// one pass and marked in asc; any other (at most leaf_max members) takes
// them in order by selection.
__global__ void k_leaf_moments(NodeArrays N, int64_t nn, const int32_t *sidx, const double *xyz, const double *m,
                               double *M, double4 *S, int8_t *asc) {
#pragma clang fp contract(off)
  int64_t node = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (node >= nn || N.nchild[node] != 0) return;
  const int32_t f = N.first[node], c = N.count[node];
  bool up = true;
  for (int32_t u = f + 1; u < f + c && up; ++u) up = sidx[u] > sidx[u - 1];
  asc[node] = up ? 1 : 0;
  double sm = 0.0, sx = 0.0, sy = 0.0, sz = 0.0;
  int32_t prev = -1;
  for (int32_t t = 0; t < c; ++t) {
    int32_t best = INT32_MAX;
    if (up) {
      best = sidx[f + t];
    } else {
      for (int32_t u = f; u < f + c; ++u) {
        int32_t j = sidx[u];
        if (j > prev && j < best) best = j;
      }
    }
    prev = best;
    const double mj = m[best];
    sm += mj;
    sx += mj * xyz[3 * (int64_t)best];
    sy += mj * xyz[3 * (int64_t)best + 1];
    sz += mj * xyz[3 * (int64_t)best + 2];
  }
  M[node] = sm;
  S[node] = make_double4(sx, sy, sz, 0.0);
}

// Internal nodes of one level: children's sums in octant order.
__global__ void k_internal_moments(NodeArrays N, int64_t b, int64_t e, double *M, double4 *S) {
#pragma clang fp contract(off)
  int64_t node = b + (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (node >= e) return;
  const int k = N.nchild[node];
  if (k == 0) return;
  const int32_t c0 = N.child_first[node];
  double sm = 0.0, sx = 0.0, sy = 0.0, sz = 0.0;
  for (int q = 0; q < k; ++q) {
    sm += M[c0 + q];
    double4 s = S[c0 + q];
    sx += s.x;
    sy += s.y;
    sz += s.z;
  }
  M[node] = sm;
  S[node] = make_double4(sx, sy, sz, 0.0);
}

__global__ void k_com(int64_t nn, const double *M, const double4 *S, double4 *com) {
#pragma clang fp contract(off)
  int64_t node = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (node >= nn) return;
  const double mm = M[node];
  const double4 s = S[node];
  com[node] = make_double4(s.x / mm, s.y / mm, s.z / mm, 0.0);
}

constexpr int kBigNode = 4096;  // members above which a node's size takes a whole workgroup

// One wave per node of at most kBigNode members: max squared member
// distance from the centre of mass and the lowest member particle index.
// positions in the sorted order of sidx, so that the node-size kernels read
// each node's particles contiguously instead of gathering them
__global__ void k_sorted_xyz(int64_t n, const int32_t *sidx, const double *xyz, double4 *sx) {
  const int64_t t = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (t >= n) return;
  const int64_t j = sidx[t];
  sx[t] = make_double4(xyz[3 * j], xyz[3 * j + 1], xyz[3 * j + 2], 0.0);
}

__global__ void __launch_bounds__(256) k_node_size(NodeArrays N, int64_t nn, const int32_t *sidx, const double4 *sx,
                                                  const double4 *com, double *s2, int32_t *minidx) {
#pragma clang fp contract(off)
  const int64_t node = ((int64_t)blockIdx.x * blockDim.x + threadIdx.x) >> 6;
  const int lane = threadIdx.x & 63;
  if (node >= nn) return;
  const int32_t f = N.first[node], c = N.count[node];
  if (c > kBigNode) {  // k_node_size_big combines its chunks into these
    if (lane == 0) {
      s2[node] = 0.0;
      minidx[node] = INT32_MAX;
    }
    return;
  }
  const double4 g = com[node];
  double mx = 0.0;
  int32_t mi = INT32_MAX;
  for (int32_t t = f + lane; t < f + c; t += 64) {
    const int32_t j = sidx[t];
    const double4 p = sx[t];
    const double dx = p.x - g.x, dy = p.y - g.y, dz = p.z - g.z;
    const double s = (dx * dx + dy * dy) + dz * dz;
    mx = fmax(mx, s);
    mi = min(mi, j);
  }
  for (int o = 32; o > 0; o >>= 1) {
    mx = fmax(mx, __shfl_xor(mx, o, 64));
    mi = min(mi, __shfl_xor(mi, o, 64));
  }
  if (lane == 0) {
    s2[node] = mx;
    minidx[node] = mi;
  }
}

// Chunks of kBigNode members: none for a node handled by k_node_size.
__global__ void k_flag_big(NodeArrays N, int64_t nn, int64_t *flag) {
  const int64_t node = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (node < nn) {
    const int32_t c = N.count[node];
    flag[node] = c > kBigNode ? (c + kBigNode - 1) / kBigNode : 0;
  }
}

// The node of every chunk (off: each node's first chunk).
__global__ void k_list_big(NodeArrays N, int64_t nn, const int64_t *off, int32_t *list) {
  const int64_t node = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (node < nn && N.count[node] > kBigNode)
    for (int64_t q = off[node]; q < off[node + 1]; ++q) list[q] = (int32_t)node;
}

// The same for the nodes above kBigNode members, one workgroup per chunk of
// kBigNode members (grid-stride over the device-side chunk list); the
// chunks combine by atomic maximum (non-negative binary64 values order as
// their bit patterns) and minimum, which do not depend on the order in
// which they finish.
__global__ void __launch_bounds__(1024) k_node_size_big(NodeArrays N, const int32_t *list, const int64_t *off,
                                                       const int64_t *n_list, const int32_t *sidx, const double4 *sx,
                                                       const double4 *com, double *s2, int32_t *minidx) {
#pragma clang fp contract(off)
  __shared__ double smx[16];
  __shared__ int32_t smi[16];
  const int64_t nb = *n_list;
  const int lane = threadIdx.x & 63, wid = threadIdx.x >> 6;
  for (int64_t b = blockIdx.x; b < nb; b += gridDim.x) {
    const int32_t node = list[b];
    const int32_t k = (int32_t)(b - off[node]);  // the chunk within the node
    const int32_t f0 = N.first[node], c = N.count[node];
    const int32_t f = f0 + k * kBigNode, fe = min(f0 + c, f + kBigNode);
    const double4 g = com[node];
    double mx = 0.0;
    int32_t mi = INT32_MAX;
    for (int32_t t = f + (int32_t)threadIdx.x; t < fe; t += (int32_t)blockDim.x) {
      const int32_t j = sidx[t];
      const double4 p = sx[t];
      const double dx = p.x - g.x, dy = p.y - g.y, dz = p.z - g.z;
      const double s = (dx * dx + dy * dy) + dz * dz;
      mx = fmax(mx, s);
      mi = min(mi, j);
    }
    for (int o = 32; o > 0; o >>= 1) {
      mx = fmax(mx, __shfl_xor(mx, o, 64));
      mi = min(mi, __shfl_xor(mi, o, 64));
    }
    if (lane == 0) {
      smx[wid] = mx;
      smi[wid] = mi;
    }
    __syncthreads();
    if (threadIdx.x == 0) {
      for (int w = 1; w < (int)(blockDim.x >> 6); ++w) {
        mx = fmax(mx, smx[w]);
        mi = min(mi, smi[w]);
      }
      atomicMax((unsigned long long *)&s2[node], (unsigned long long)__double_as_longlong(mx));
      atomicMin(&minidx[node], mi);
    }
    __syncthreads();
  }
}

// Node label: a 1 followed by the octant digits from the root down (3 bits
// per level), read off the Morton key of the node's first member.
__global__ void k_label(NodeArrays N, int64_t nn, const uint64_t *keys, uint64_t *label) {
  const int64_t node = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (node >= nn) return;
  const int l = N.level[node];
  const uint64_t key = keys[N.first[node]];
  label[node] = (1ull << (3 * l)) | (l == 0 ? 0ull : key >> (3 * (21 - l)));
}

// Nodes whose labels are in the sorted list are opened (Sec. 2.4.1: the
// nodes that failed the resolution check).
__global__ void k_force_open(int64_t nn, const uint64_t *label, int64_t n_open, const uint64_t *open, int8_t *acc) {
  const int64_t node = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (node >= nn || !acc[node]) return;
  const uint64_t l = label[node];
  int64_t lo = 0, hi = n_open;
  while (lo < hi) {
    const int64_t mid = (lo + hi) >> 1;
    if (open[mid] < l) lo = mid + 1;
    else hi = mid;
  }
  if (lo < n_open && open[lo] == l) acc[node] = 0;
}

__global__ void k_accept(int64_t nn, const double4 *com, const double *s2, int n_src, const double *src, double r_part,
                         double theta, int8_t *acc) {
#pragma clang fp contract(off)
  int64_t node = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (node >= nn) return;
  const double4 g = com[node];
  const double ss = s2[node];
  const double s = sqrt(ss);
  int8_t ok = 1;
  for (int k = 0; k < n_src && ok; ++k) {
    const double dx = g.x - src[3 * k], dy = g.y - src[3 * k + 1], dz = g.z - src[3 * k + 2];
    const double r2 = (dx * dx + dy * dy) + dz * dz;
    const double r = sqrt(r2);
    if (!(r - s > r_part)) ok = 0;
    else if ((theta * theta) * r2 < ss) ok = 0;
  }
  acc[node] = ok;
}

__global__ void k_fill_i32(int32_t *p, int32_t v, int64_t n) {
  int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i < n) p[i] = v;
}

// Emitted units: accepted without an accepted ancestor, or an opened leaf.
__global__ void k_units(NodeArrays N, int64_t nn, const int8_t *acc, int32_t *unit_at) {
  int64_t node = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (node >= nn) return;
  for (int32_t p = N.parent[node]; p >= 0; p = N.parent[p])
    if (acc[p]) return;
  if (acc[node] || N.nchild[node] == 0) unit_at[N.first[node]] = (int32_t)node;
}

__global__ void k_flag(int64_t n, const int32_t *unit_at, int64_t *flag) {
  int64_t t = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (t < n) flag[t] = unit_at[t] >= 0 ? 1 : 0;
}

__global__ void k_unit_list(int64_t n, const int32_t *unit_at, const int64_t *uoff, int32_t *units) {
  int64_t t = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (t < n && unit_at[t] >= 0) units[uoff[t]] = unit_at[t];
}

__global__ void k_unit_counts(int64_t nu, const int32_t *units, NodeArrays N, const int8_t *acc, int64_t *ecnt,
                              int64_t *pcnt) {
  int64_t u = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (u >= nu) return;
  const int32_t node = units[u];
  const bool a = acc[node] != 0;
  ecnt[u] = a ? 1 : N.count[node];
  pcnt[u] = (a && N.count[node] > 1) ? 1 : 0;
}

__global__ void k_entries(int64_t nu, const int32_t *units, NodeArrays N, const int8_t *acc, const int64_t *eoff,
                          const int64_t *poff, const int32_t *sidx, const double *xyz, const double *hh,
                          const double *m, const double *M, const double4 *com, const double *s2,
                          const int32_t *minidx, double *o_xyz, double *o_h, double *o_m, double *o_s,
                          int32_t *o_kind, int64_t *o_first, int64_t *o_count, int32_t *o_branch, double4 *upos,
                          int32_t *plist, const uint64_t *label, uint64_t *o_label, const int8_t *asc) {
  int64_t u = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (u >= nu) return;
  const int32_t node = units[u];
  const int32_t f = N.first[node], c = N.count[node];
  const double4 g = com[node];
  upos[u] = g;
  int64_t e = eoff[u];
  auto emit_real = [&](int32_t j) {
    o_xyz[3 * e] = xyz[3 * (int64_t)j];
    o_xyz[3 * e + 1] = xyz[3 * (int64_t)j + 1];
    o_xyz[3 * e + 2] = xyz[3 * (int64_t)j + 2];
    o_h[e] = hh[j];
    o_m[e] = m[j];
    if (o_s) o_s[e] = 0.0;
    if (o_kind) o_kind[e] = 0;
    if (o_first) o_first[e] = j;
    if (o_count) o_count[e] = 1;
    if (o_branch) o_branch[e] = -1;
    if (o_label) o_label[e] = label[node];
    ++e;
  };
  if (acc[node]) {
    if (c == 1) {
      emit_real(sidx[f]);
    } else {
      o_xyz[3 * e] = g.x;
      o_xyz[3 * e + 1] = g.y;
      o_xyz[3 * e + 2] = g.z;
      o_h[e] = 0.0;
      o_m[e] = M[node];
      if (o_s) o_s[e] = sqrt(s2[node]);
      if (o_kind) o_kind[e] = 1;
      if (o_first) o_first[e] = minidx[node];
      if (o_count) o_count[e] = c;
      if (o_branch) o_branch[e] = 0;
      if (o_label) o_label[e] = label[node];
      plist[poff[u]] = (int32_t)e;
    }
  } else {
    // opened leaf: its particles in ascending index
    int32_t prev = -1;
    for (int32_t t = 0; t < c; ++t) {
      int32_t best = INT32_MAX;
      if (asc[node]) {
        best = sidx[f + t];
      } else {
        for (int32_t q = f; q < f + c; ++q) {
          int32_t j = sidx[q];
          if (j > prev && j < best) best = j;
        }
      }
      prev = best;
      emit_real(best);
    }
  }
}

// Entry that holds each particle: the sorted position's unit is the last unit
// starting at or before it; an opened leaf's particles are its entries in
// ascending index, so a particle's entry is offset by its rank among them.
__global__ void k_owner(int64_t n, const int64_t *flag, const int64_t *uoff, const int32_t *units, NodeArrays N,
                        const int8_t *acc, const int64_t *eoff, const int32_t *sidx, const int8_t *asc,
                        int64_t *owner) {
  const int64_t q = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (q >= n) return;
  const int64_t u = uoff[q] + flag[q] - 1;
  const int32_t node = units[u];
  const int32_t j = sidx[q];
  int64_t e = eoff[u];
  if (!acc[node]) {
    const int32_t f = N.first[node], c = N.count[node];
    if (asc[node]) e += q - f;  // members in ascending index: the rank is the position
    else
      for (int32_t t = f; t < f + c; ++t) e += sidx[t] < j;
  }
  owner[j] = e;
}

constexpr double kInvPi = 0.31830988618379067154;

__device__ inline double m4w(double q) {
#pragma clang fp contract(off)
  if (q < 1.0) return 1.0 - 1.5 * q * q + 0.75 * q * q * q;
  if (q < 2.0) return 0.25 * (2.0 - q) * (2.0 - q) * (2.0 - q);
  return 0.0;
}
__device__ inline double m4dw(double q) {
#pragma clang fp contract(off)
  if (q < 1.0) return -3.0 * q + 2.25 * q * q;
  if (q < 2.0) return -0.75 * (2.0 - q) * (2.0 - q);
  return 0.0;
}

__device__ inline double readlane_d(double v, int j) {
  const unsigned long long b = (unsigned long long)__double_as_longlong(v);
  const unsigned lo = (unsigned)__builtin_amdgcn_readlane((int)(unsigned)b, j);
  const unsigned hi = (unsigned)__builtin_amdgcn_readlane((int)(unsigned)(b >> 32), j);
  return __longlong_as_double((long long)(((unsigned long long)hi << 32) | lo));
}

// What the node h-solve sums over: the units (their positions and the
// boxes of their tiles of 64 and of their blocks of 64 tiles) and, with
// n_mid > 0, the trial-neighbour ranges.
struct HUnits {
  int64_t nu;
  const double4 *upos;
  const double4 *tlo, *thi;  // tile t: units [64 t, 64 t + 64)
  const double4 *blo, *bhi;  // block b: tiles [64 b, 64 b + 64)
  int64_t n_mid;
  const double4 *mid_com;
  const int32_t *mid_u0, *mid_u1;
  const double *rcut;
};

// The sums of one h-solve step at node position (ax, ay, az) and length he,
// over every unit within 2 he, by one wavefront.
//
// Unit order (fast == false): the 64 lanes evaluate 64 consecutive units at
// a time, the tile's non-zero terms go to LDS (hb, 64 entries) in lane order
// and lanes 0 and 1 add them one after the other (lane 0 the w terms, lane 1
// the dt terms), so sw and sd, returned to every lane, are the sums of a
// plain sequential loop over the units.
//
// Tree order (fast == true): sw only, and only this wave's share, the tiles
// t with t % step == first: each tile's terms are added by a butterfly and
// the tiles in order; every lane holds the share, and nhit counts its
// non-zero terms.
//
// A block or tile whose bounding box lies beyond 2 he holds only zero terms
// and is skipped.  A block's box holds its tiles' boxes and the distance test
// is monotone in the box bounds, so no tile that passes the test is skipped
// with its block.  Blocks and tiles are visited in ascending order.  With
// n_mid > 0 the sums run over trial neighbours only: the units of the ranges
// [mid_u0, mid_u1) of the nodes whose centres of mass lie within rcut[e] of
// the target; the ranges follow unit order, so unit-order terms are still
// added in unit order.
// kBatch: LDS reads in flight in the unit-order adds.
template <int kBatch>
__device__ __forceinline__ void hsums(const HUnits &U, int32_t e, double ax, double ay, double az, double he,
                                      bool fast, int first, int step, double2 *hb, double &sw, double &sd,
                                      int64_t &nhit) {
#pragma clang fp contract(off)
  const int lane = threadIdx.x & 63;
  const uint64_t below = lane == 0 ? 0ull : (~0ull >> (64 - lane));
  const double ih = 1.0 / he;
  double acc = 0.0;  // unit order: lane 0's sw, lane 1's sd
  sw = sd = 0.0;
  nhit = 0;
  // the terms of one tile's units (one per lane, `live` lanes hold one)
  auto tile_terms = [&](const double4 &p, bool live) __attribute__((always_inline)) {
    double w = 0.0, dt = 0.0;
    bool hit = false;
    if (live) {
      const double dx = ax - p.x, dy = ay - p.y, dz = az - p.z;
      const double qq = sqrt((dx * dx + dy * dy) + dz * dz) * ih;
      if (qq < 2.0) {
        hit = true;
        w = m4w(qq);
        if (!fast) dt = -(3.0 * w + qq * m4dw(qq));
      }
    }
    const uint64_t mask = __ballot(hit);
    if (fast) {
      nhit += __popcll(mask);
      if (mask) {
        double v = hit ? w : 0.0;
#pragma unroll
        for (int o = 32; o > 0; o >>= 1) v += __shfl_xor(v, o, 64);
        sw += readlane_d(v, 0);
      }
      return;
    }
    if (mask) {
      if (hit) hb[__popcll(mask & below)] = make_double2(w, dt);
      __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
      __builtin_amdgcn_wave_barrier();
      __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
      if (lane < 2) {  // lane 0 adds the w terms, lane 1 the dt terms
        const double *src = reinterpret_cast<const double *>(hb) + lane;
        const int cnt = __popcll(mask);
        int k = 0;
        for (; k + kBatch <= cnt; k += kBatch) {  // kBatch reads in flight, added in order
          double v[kBatch];
#pragma unroll
          for (int u = 0; u < kBatch; ++u) v[u] = src[2 * (k + u)];
#pragma unroll
          for (int u = 0; u < kBatch; ++u) acc += v[u];
        }
        for (; k < cnt; ++k) acc += src[2 * k];
      }
      __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
      __builtin_amdgcn_wave_barrier();
      __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
    }
  };
  auto beyond = [&](const double4 &lo, const double4 &hi) __attribute__((always_inline)) {
    const double bx = fmax(fmax(lo.x - ax, ax - hi.x), 0.0);
    const double by = fmax(fmax(lo.y - ay, ay - hi.y), 0.0);
    const double bz = fmax(fmax(lo.z - az, az - hi.z), 0.0);
    return !(((bx * bx + by * by) + bz * bz) * ih * ih < 4.0 * (1.0 + 1e-9));
  };
  // units [u0, u1), tiles t with t % step == first
  auto tile_sums = [&](int64_t u0, int64_t u1) __attribute__((always_inline)) {
    const int64_t t0 = u0 >> 6, t1 = (u1 + 63) >> 6;
    const int64_t b0 = t0 >> 6, b1 = (t1 + 63) >> 6;
    for (int64_t bb = b0; bb < b1; bb += 64) {
      const int64_t bi = bb + lane;
      bool bnear = false;
      if (bi < b1) bnear = !beyond(U.blo[bi], U.bhi[bi]);
      uint64_t bm = __ballot(bnear);
      while (bm) {
        const int64_t tb = 64 * (bb + __builtin_ctzll(bm));
        bm &= bm - 1;
        const int64_t ti = tb + lane;
        bool near = false;
        if (ti >= t0 && ti < t1 && ti % step == first) near = !beyond(U.tlo[ti], U.thi[ti]);
        uint64_t nm = __ballot(near);
        while (nm) {
          // up to four near tiles at once: their loads are in flight together,
          // and their terms are added tile after tile
          int64_t ua0, ub0, ua1, ub1, ua2, ub2, ua3, ub3;
          double4 p0, p1, p2, p3;
          auto take = [&](int64_t &ua, int64_t &ub, double4 &pv) __attribute__((always_inline)) {
            ua = ub = 0;
            if (nm) {
              const int64_t t = tb + __builtin_ctzll(nm);
              nm &= nm - 1;
              ua = max(u0, 64 * t);
              ub = min(u1, 64 * t + 64);
            }
            if (ua + lane < ub) pv = U.upos[ua + lane];
          };
          take(ua0, ub0, p0);
          take(ua1, ub1, p1);
          take(ua2, ub2, p2);
          take(ua3, ub3, p3);
          if (ub0 > ua0) tile_terms(p0, ua0 + lane < ub0);
          if (ub1 > ua1) tile_terms(p1, ua1 + lane < ub1);
          if (ub2 > ua2) tile_terms(p2, ua2 + lane < ub2);
          if (ub3 > ua3) tile_terms(p3, ua3 + lane < ub3);
        }
      }
    }
  };
  if (U.n_mid == 0) {
    tile_sums(0, U.nu);
  } else {
    const double rc = U.rcut[e];
    for (int64_t m0 = 0; m0 < U.n_mid; m0 += 64) {
      const int64_t mi = m0 + lane;
      bool flag = false;
      if (mi < U.n_mid) {
        const double4 c = U.mid_com[mi];
        const double dx = ax - c.x, dy = ay - c.y, dz = az - c.z;
        flag = sqrt((dx * dx + dy * dy) + dz * dz) < rc;
      }
      uint64_t fm = __ballot(flag);
      while (fm) {
        const int j = __builtin_ctzll(fm);
        fm &= fm - 1;
        tile_sums(U.mid_u0[m0 + j], U.mid_u1[m0 + j]);
      }
    }
  }
  if (!fast) {
    sw = readlane_d(acc, 0);
    sd = readlane_d(acc, 1);
  }
}

// f(he) = hfact n(he)^(-1/3) - he from sw, the sum of the M4 terms at he
__device__ __forceinline__ double h_residual(double sw, double he, double hfact) {
#pragma clang fp contract(off)
  const double ih = 1.0 / he;
  const double n = sw * ih * ih * ih * kInvPi;
  return hfact * pow(n, -1.0 / 3.0) - he;
}

// The M4 terms of one unit at distance (dx, dy, dz): whether it lies within
// 2 he, w and dt (as hsums forms them).
__device__ __forceinline__ bool unit_terms(double dx, double dy, double dz, double ih, double &w, double &dt) {
#pragma clang fp contract(off)
  const double qq = sqrt((dx * dx + dy * dy) + dz * dz) * ih;
  w = dt = 0.0;
  if (!(qq < 2.0)) return false;
  w = m4w(qq);
  dt = -(3.0 * w + qq * m4dw(qq));
  return true;
}

// Whether a box lies wholly beyond 2 he (the test of hsums).
__device__ __forceinline__ bool box_beyond(const double4 &lo, const double4 &hi, double ax, double ay, double az,
                                           double ih) {
#pragma clang fp contract(off)
  const double bx = fmax(fmax(lo.x - ax, ax - hi.x), 0.0);
  const double by = fmax(fmax(lo.y - ay, ay - hi.y), 0.0);
  const double bz = fmax(fmax(lo.z - az, az - hi.z), 0.0);
  return !(((bx * bx + by * by) + bz * bz) * ih * ih < 4.0 * (1.0 + 1e-9));
}

// One Newton step from h given the unit-order sums.  0: go on with hn;
// 1: converged at hn; -1: failed.
__device__ __forceinline__ int newton_step(double sw, double sd, double h, double h0, double hfact, double eps,
                                           double &hn) {
#pragma clang fp contract(off)
  const double ih = 1.0 / h;
  const double n = sw * ih * ih * ih * kInvPi;
  const double dn = sd * ih * ih * ih * ih * kInvPi;
  const double f = hfact * pow(n, -1.0 / 3.0) - h;
  const double fp = -(1.0 / 3.0) * hfact * dn * pow(n, -4.0 / 3.0) - 1.0;
  if (!(fabs(fp) >= 1e-12)) return -1;
  hn = h - f / fp;
  if (!(hn >= 1e-2 * h0 && hn <= 1e2 * h0)) return -1;
  return fabs(hn - h) / h0 < eps ? 1 : 0;
}

// Near tiles beyond which a node goes to the wide Newton kernel.  Below, its
// two passes and 16-wave barriers cost more than one wave's chain: builds of
// 1,048,576 (octree) and 262,139 (k-d) particles in ms at a line of 48 tiles
// 3.19 and 2.58, 96: 3.09 and 2.65, 160: 3.17 and 2.71, 256: 3.30 and 2.84;
// all on one wave 5.9 and 2.9.
constexpr int kNearTiles = 96;
constexpr int kWideTiles = 2048; // near tiles a workgroup of that kernel can hold
constexpr int kWideWaves = 16;
constexpr int kWideKept = 48;    // tiles whose terms it keeps
constexpr int kNewtonSteps = 30;
// Nodes up to which they take a workgroup each.  A chip holds 256 of those and
// 4,096 and more single wavefronts: sets whose nodes all meet many units (h_fact
// of 5 to 8) have 4,400 to 20,600 such nodes, and took 3.8 and 15.0 ms a build on
// workgroups, 2.3 and 5.1 on wavefronts (k_hsolve_rest); the clouds of a million particles around
// one source have 200 to 900, of which a few take 30 steps.
constexpr int kWideNodes = 2048;

// A node handed from the one-wave to the wide Newton kernel.
struct WideNode {
  int32_t e, it;  // entry, Newton steps taken
  double h;       // the next step's length
};

// Lengths from which the bracket takes binary32 sums: squares of distances
// below 2e-19 underflow there, which moves x by 2e-8 at most for these (and
// 1 / he is finite).  Shorter ones, of nodes at the corner of the box, take
// the binary64 sums.
constexpr double kLeast32 = 1e-11;

// One wavefront's Newton steps it, it + 1, ... from h with unit-order sums (hb:
// 64 entries of LDS).  0: converged at h; -1: failed; 2: left, where `leave(h)`
// says so, before step it from h.
template <class Leave>
__device__ __forceinline__ int newton_wave(const HUnits &U, int32_t e, double ax, double ay, double az, double h0,
                                           double hfact, double eps, double2 *hb, Leave leave, int &it, double &h) {
  for (; it < kNewtonSteps; ++it) {
    if (leave(h)) return 2;
    double sw, sd, hn = h;
    int64_t nhit;
    hsums<16>(U, e, ax, ay, az, h, false, 0, 1, hb, sw, sd, nhit);
    const int v = newton_step(sw, sd, h, h0, hfact, eps, hn);
    if (v < 0) return -1;
    h = hn;
    if (v > 0) return 0;
  }
  return -1;
}
// What becomes of entry e (one lane a node): h, or the bracket's list.
__device__ __forceinline__ void newton_done(int32_t e, int branch, double h, double *o_h, int32_t *o_branch,
                                            unsigned long long *bcount, int32_t *fails, int32_t *n_fails) {
  if ((threadIdx.x & 63) != 0) return;
  if (branch < 0) {
    fails[atomicAdd(n_fails, 1)] = e;
  } else {
    o_h[e] = h;
    if (o_branch) o_branch[e] = branch;
    atomicAdd(&bcount[branch], 1ull);
  }
}

constexpr int kHWaves = 4;    // pseudo-particles per workgroup in the Newton kernel
constexpr int kBWaves = 16;   // wavefronts per pseudo-particle in the bracket kernel

// Node h-solve, first part: up to 30 Newton steps from h0 = 2 hfact s, one
// wavefront per pseudo-particle, with unit-order sums.  A converged node
// writes its h (branch 0); a node whose step fails (a vanishing derivative,
// a step out of [h0/100, 100 h0], or 30 steps) is appended to `fails` for
// the bracket kernel, in whatever order the atomics give (each node's result
// depends on that node alone).  Above `bypass` pseudo-particles every node
// takes h0 (branch 3).  A step that meets more than kNearTiles tiles hands
// its node to the wide kernel: one wave adds a unit-order sum at 13 cycles a
// term, 350 us a step over 62,751 units.
__global__ void __launch_bounds__(64 * kHWaves) k_hsolve_newton(int64_t np, const int32_t *plist, HUnits U,
                                                               const double *o_xyz, const double *o_s, double hfact,
                                                               double eps, int64_t bypass, double *o_h,
                                                               int32_t *o_branch, unsigned long long *bcount,
                                                               int32_t *fails, int32_t *n_fails, WideNode *wide,
                                                               int32_t *n_wide) {
#pragma clang fp contract(off)
  __shared__ double2 hbuf[kHWaves][64];
  const int64_t pid = (int64_t)blockIdx.x * kHWaves + (threadIdx.x >> 6);
  const int lane = threadIdx.x & 63;
  if (pid >= np) return;  // the whole wavefront
  const int32_t e = plist[pid];
  const double ax = o_xyz[3 * (int64_t)e], ay = o_xyz[3 * (int64_t)e + 1], az = o_xyz[3 * (int64_t)e + 2];
  const double h0 = hfact * 2.0 * o_s[e];
  double hres = h0;
  int branch = 3;
  if (np <= bypass) {
    const int64_t nt = (U.nu + 63) >> 6;
    int it = 0;
    const auto near_many = [&](double h) {
      if (!wide || U.n_mid != 0 || nt <= kNearTiles) return false;
      const double ih = 1.0 / h;
      int near = 0;
      for (int64_t b = 0; b < nt && near <= kNearTiles; b += 64) {
        if (box_beyond(U.blo[b >> 6], U.bhi[b >> 6], ax, ay, az, ih)) continue;  // the same in every lane
        const int64_t t = min(b + lane, nt - 1);
        near += __popcll(__ballot(b + lane < nt && !box_beyond(U.tlo[t], U.thi[t], ax, ay, az, ih)));
      }
      return near > kNearTiles;
    };
    branch = newton_wave(U, e, ax, ay, az, h0, hfact, eps, hbuf[threadIdx.x >> 6], near_many, it, hres);
    if (branch == 2) {
      if (lane == 0) wide[atomicAdd(n_wide, 1)] = WideNode{e, it, hres};
      return;
    }
  }
  newton_done(e, branch, hres, o_h, o_branch, bcount, fails, n_fails);
}

// v of the lane a DPP control names, 0 where it names none; row_shr 1, 2, 4, 8
// and row_bcast 15, 31 in turn leave the sum over the wavefront in lane 63.
template <int kCtrl>
__device__ __forceinline__ int dpp0(int v) {
  return __builtin_amdgcn_update_dpp(0, v, kCtrl, 0xf, 0xf, false);
}
template <int kCtrl>
__device__ __forceinline__ float dpp_add(float v) {
  return v + __int_as_float(dpp0<kCtrl>(__float_as_int(v)));
}
template <int kCtrl>
__device__ __forceinline__ double dpp_add(double v) {
  const int lo = dpp0<kCtrl>(__double2loint(v)), hi = dpp0<kCtrl>(__double2hiint(v));
  return v + __hiloint2double(hi, lo);
}
template <typename T>
__device__ __forceinline__ T sum_to_63(T v) {
  v = dpp_add<0x111>(v);
  v = dpp_add<0x112>(v);
  v = dpp_add<0x114>(v);
  v = dpp_add<0x118>(v);
  v = dpp_add<0x142>(v);
  return dpp_add<0x143>(v);
}
// inclusive sums over the wavefront's lanes of values whose sums are exact
template <int kCtrl, int kRows>
__device__ __forceinline__ double dpp_scan(double v) {
  const int lo = __builtin_amdgcn_update_dpp(0, __double2loint(v), kCtrl, kRows, 0xf, false);
  const int hi = __builtin_amdgcn_update_dpp(0, __double2hiint(v), kCtrl, kRows, 0xf, false);
  return v + __hiloint2double(hi, lo);
}
__device__ __forceinline__ double wave_incl(double v) {
  v = dpp_scan<0x111, 0xf>(v);
  v = dpp_scan<0x112, 0xf>(v);
  v = dpp_scan<0x114, 0xf>(v);
  v = dpp_scan<0x118, 0xf>(v);
  v = dpp_scan<0x142, 0xa>(v);     // into rows 1 and 3
  return dpp_scan<0x143, 0xc>(v);  // into rows 2 and 3
}

// Newton for nodes that meet many units, one workgroup a node, its sums bit
// for bit those of a plain loop over the units in order.  While a running sum
// S stays in one binade (spacing u), fl(S + t) = S + u rint(t / u) unless t
// lies half way between two multiples of u: the rounded additions are integer
// additions, which any order gives alike.  So, a step:
//   - the near tiles are listed in order, and their sums taken in any order
//     to foresee the binade each tile starts in;
//   - every tile adds its terms' integers for that binade (and a bound of the
//     sum of their sizes: dt has both signs, and the sums inside the tile have
//     to stay in the binade too), or is marked where a term lies half way;
//   - one wavefront goes through the tiles 64 at a time, adding the integers
//     up to the first tile that starts in another binade, could leave it, or
//     is marked; that tile's terms it adds one by one.
// About 20 to 40 of a step's 980 tiles are added one by one where the sums
// pass their first binades; the terms of the marked tiles and of those foreseen
// to end in another binade are kept in LDS for that.  A step over 62,751 units
// takes 55 us (350 us on one wave; 70 with the walk's scans by shuffles, two
// sums a tile for its bounds and no terms kept); what bounds the kernel is the
// node with the most steps, 30 that wait for each other: 1.6 ms of a
// 1,048,576-particle build, whose Newton part was 4.3 ms and is 1.8 (MI355X).
__global__ void __launch_bounds__(64 * kWideWaves) k_hsolve_wide(const WideNode *wide, const int32_t *n_wide, HUnits U,
                                                                const double *o_xyz, const double *o_s, double hfact,
                                                                double eps, double *o_h, int32_t *o_branch,
                                                                unsigned long long *bcount, int32_t *fails,
                                                                int32_t *n_fails) {
#pragma clang fp contract(off)
  __shared__ int32_t tl[kWideTiles];                      // the near tiles
  // their sums, then where they start (x: w, y: dt); then the integers of w
  __shared__ union {
    float2 f;
    double v;
  } tw[kWideTiles];
  __shared__ double vd[kWideTiles];                       // integers of dt
  __shared__ float va[kWideTiles];                        // bound of the sum of their sizes
  __shared__ int16_t ew[kWideTiles], ed[kWideTiles];      // binades they are in
  __shared__ int wcnt[kWideWaves];
  __shared__ float wsum[2][kWideWaves];
  __shared__ double2 hb[64];
  __shared__ double2 kept[kWideKept][64];                 // terms of tiles expected to be added one by one
  __shared__ int8_t slot[kWideTiles];                     // where, -1: nowhere
  __shared__ int n_kept;
  __shared__ double next_h;
  __shared__ int verdict;
  const int tid = threadIdx.x, lane = tid & 63, wid = __builtin_amdgcn_readfirstlane(tid >> 6);
  const uint64_t below = lane == 0 ? 0ull : (~0ull >> (64 - lane));
  constexpr int16_t kMarked = -32768;
  const int64_t nt = (U.nu + 63) >> 6;
  if (*n_wide > kWideNodes) return;  // k_hsolve_rest takes them
  for (int b = blockIdx.x; b < *n_wide; b += gridDim.x) {
    const WideNode nd = wide[b];
    const double ax = o_xyz[3 * (int64_t)nd.e], ay = o_xyz[3 * (int64_t)nd.e + 1], az = o_xyz[3 * (int64_t)nd.e + 2];
    const double h0 = hfact * 2.0 * o_s[nd.e];
    double h = nd.h;
    int v = -1;
    for (int it = nd.it; it < kNewtonSteps; ++it) {
      const double ih = 1.0 / h;
      // the near tiles, in order
      int T = 0;
      for (int64_t t0 = 0; t0 < nt; t0 += 64 * kWideWaves) {
        const int64_t t = t0 + tid;
        const bool near = t < nt && !box_beyond(U.tlo[t], U.thi[t], ax, ay, az, ih);
        const uint64_t m = __ballot(near);
        if (lane == 0) wcnt[wid] = __popcll(m);
        __syncthreads();
        int at = T + __popcll(m & below);
        for (int w = 0; w < kWideWaves; ++w) {
          if (w < wid) at += wcnt[w];
          T += wcnt[w];
        }
        if (near && at < kWideTiles) tl[at] = (int32_t)t;
        __syncthreads();
      }
      double sw, sd;
      if (T > kWideTiles) {  // more than fit: one wave's plain sums
        if (wid == 0) {
          int64_t nhit;
          hsums<16>(U, nd.e, ax, ay, az, h, false, 0, 1, hb, sw, sd, nhit);
        }
      } else {
        // this lane's terms of tile j
        auto terms = [&](int j, double &w, double &dt) {
          const int64_t u = 64 * (int64_t)tl[j] + lane;
          w = dt = 0.0;
          if (u >= U.nu) return false;
          const double4 p = U.upos[u];
          return unit_terms(ax - p.x, ay - p.y, az - p.z, ih, w, dt);
        };
        // (in binary32: they only foresee the binades)
        const float ihf = (float)ih;
        for (int j = wid; j < T; j += 2 * kWideWaves) {
          float sa[2], sc[2];
#pragma unroll
          for (int q = 0; q < 2; ++q) {
            const int jq = j + q * kWideWaves;
            const int64_t u = 64 * (int64_t)tl[jq < T ? jq : j] + lane;
            const double4 p = U.upos[u < U.nu ? u : 0];
            const float dx = (float)(ax - p.x), dy = (float)(ay - p.y), dz = (float)(az - p.z);
            const float x = __builtin_amdgcn_sqrtf(dx * dx + dy * dy + dz * dz) * ihf, y = 2.0f - x;
            const bool in = jq < T && u < U.nu && x < 2.0f;
            const float w = x < 1.0f ? 1.0f + x * x * (0.75f * x - 1.5f) : 0.25f * y * y * y;
            const float g = x < 1.0f ? x * (2.25f * x - 3.0f) : -0.75f * y * y;
            sa[q] = in ? w : 0.0f;
            sc[q] = in ? -(3.0f * w + x * g) : 0.0f;
          }
#pragma unroll
          for (int q = 0; q < 2; ++q) {
            sa[q] = sum_to_63(sa[q]);
            sc[q] = sum_to_63(sc[q]);
            if (lane == 63 && j + q * kWideWaves < T) tw[j + q * kWideWaves].f = make_float2(sa[q], sc[q]);
          }
        }
        __syncthreads();
        // where each tile starts: two tiles a thread
        {
          static_assert(kWideTiles == 2 * 64 * kWideWaves, "two tiles a thread");
          const int j = 2 * tid;
          const float2 f0 = j < T ? tw[j].f : float2{}, f1 = j + 1 < T ? tw[j + 1].f : float2{};
          float a = f0.x + f1.x, c = f0.y + f1.y;
#pragma unroll
          for (int d = 1; d < 64; d <<= 1) {
            const float ya = __shfl_up(a, d, 64), yc = __shfl_up(c, d, 64);
            if (lane >= d) {
              a += ya;
              c += yc;
            }
          }
          if (lane == 63) {
            wsum[0][wid] = a;
            wsum[1][wid] = c;
          }
          __syncthreads();
          for (int w = 0; w < wid; ++w) {
            a += wsum[0][w];
            c += wsum[1][w];
          }
          const float2 s0 = make_float2(a - f0.x - f1.x, c - f0.y - f1.y), s1 = make_float2(a - f1.x, c - f1.y);
          tw[j].f = s0;
          tw[j + 1].f = s1;
          // a tile that ends in another binade than it starts in is not added as integers
          const auto leaves = [](float2 u, float ex, float ey) {
            return __builtin_amdgcn_frexp_expf(u.x) != __builtin_amdgcn_frexp_expf(ex) ||
                   __builtin_amdgcn_frexp_expf(u.y) != __builtin_amdgcn_frexp_expf(ey);
          };
          slot[j] = leaves(s0, s1.x, s1.y) ? 1 : 0;
          slot[j + 1] = leaves(s1, a, c) ? 1 : 0;
          if (tid == 0) n_kept = 0;
        }
        __syncthreads();
        for (int j = wid; j < T; j += 2 * kWideWaves) {
          double iw[2], id[2];
          float sz[2];
          int kw[2], kd[2];
          bool mark[2];
          int8_t at[2];
#pragma unroll
          for (int q = 0; q < 2; ++q) {
            const int jq = min(j + q * kWideWaves, T - 1);
            double w, dt;
            (void)terms(jq, w, dt);
            const float2 from = tw[jq].f;
            kw[q] = __builtin_amdgcn_frexp_expf(from.x);
            kd[q] = __builtin_amdgcn_frexp_expf(from.y);
            // in units of the spacing of doubles in [2^(k - 1), 2^k)
            const double rw = ldexp(w, 53 - kw[q]), rd = ldexp(dt, 53 - kd[q]);
            iw[q] = rint(rw);
            id[q] = rint(rd);
            mark[q] = __ballot(fabs(rw - iw[q]) == 0.5 || fabs(rd - id[q]) == 0.5) != 0ull;
            sz[q] = (float)fabs(id[q]);
            at[q] = -1;
            if (j + q * kWideWaves < T && (mark[q] || slot[jq])) {  // uniform
              int k = 0;
              if (lane == 0) k = atomicAdd(&n_kept, 1);
              k = __builtin_amdgcn_readfirstlane(k);
              if (k < kWideKept) {
                kept[k][lane] = make_double2(w, dt);
                at[q] = (int8_t)k;
              }
            }
          }
#pragma unroll
          for (int q = 0; q < 2; ++q) {
            iw[q] = sum_to_63(iw[q]);
            id[q] = sum_to_63(id[q]);
            sz[q] = sum_to_63(sz[q]) * (1.0f + 1e-4f);  // above the exact sum
          }
#pragma unroll
          for (int q = 0; q < 2; ++q) {
            const int jq = j + q * kWideWaves;
            if (lane == 63 && jq < T) {
              tw[jq].v = iw[q];
              vd[jq] = id[q];
              va[jq] = sz[q];
              ew[jq] = mark[q] ? kMarked : (int16_t)kw[q];
              ed[jq] = (int16_t)kd[q];
              slot[jq] = at[q];
            }
          }
        }
        __syncthreads();
        if (wid == 0) {
          sw = sd = 0.0;
          int j0 = 0;
          while (j0 < T) {
            const int j = j0 + lane;
            const int kw = __builtin_amdgcn_frexp_exp(sw), kd = __builtin_amdgcn_frexp_exp(sd);
            const bool in = j < T;
            const double xw = in ? tw[j].v : 0.0, xd = in ? vd[j] : 0.0, xa = in ? (double)va[j] : 0.0;
            const double xp = 0.5 * (xa + xd), xn = 0.5 * (xd - xa);  // bounds of the sums of dt > 0 and of dt < 0
            const double cw = wave_incl(xw), cd = wave_incl(xd);
            // the sums at the tile's start and the bounds inside it, in units
            const double bw = ldexp(sw, 53 - kw) + (cw - xw), bd = ldexp(sd, 53 - kd) + (cd - xd);
            constexpr double kOne = 4503599627370496.0, kTwo = 2.0 * kOne;  // the binade is [kOne, kTwo)
            const bool okw = in && sw > 0.0 && ew[in ? j : 0] == kw && bw >= kOne && bw + xw <= kTwo - 1.0;
            const bool okd = sd > 0.0 ? bd + xn >= kOne + 1.0 && bd + xp <= kTwo - 1.0
                                      : bd + xp <= -kOne - 1.0 && bd + xn >= -kTwo + 1.0;
            const uint64_t good = __ballot(okw && sd != 0.0 && ed[in ? j : 0] == kd && okd);
            const int n = good == ~0ull ? 64 : __builtin_ctzll(~good);  // tiles up to the first that is not
            if (n > 0) {
              sw = ldexp(readlane_d(bw + xw, n - 1), kw - 53);
              sd = ldexp(readlane_d(bd + xd, n - 1), kd - 53);
              j0 += n;
            }
            if (n < 64 && j0 < T) {  // that tile term by term (terms of 0 change nothing)
              const int k = __builtin_amdgcn_readfirstlane((int)slot[j0]);
              const double2 *row = k >= 0 ? kept[k] : hb;
              if (k < 0) {
                double w, dt;
                (void)terms(j0, w, dt);
                hb[lane] = make_double2(w, dt);
                __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
                __builtin_amdgcn_wave_barrier();
                __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
              }
              double acc = lane == 0 ? sw : sd;
              if (lane < 2) {
                const double *src = reinterpret_cast<const double *>(row) + lane;
#pragma unroll
                for (int t = 0; t < 64; t += 16) {
                  double x[16];
#pragma unroll
                  for (int u = 0; u < 16; ++u) x[u] = src[2 * (t + u)];
#pragma unroll
                  for (int u = 0; u < 16; ++u) acc += x[u];
                }
              }
              sw = readlane_d(acc, 0);
              sd = readlane_d(acc, 1);
              __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
              __builtin_amdgcn_wave_barrier();
              __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
              ++j0;
            }
          }
        }
      }
      if (wid == 0) {
        double hn = h;
        const int r = newton_step(sw, sd, h, h0, hfact, eps, hn);
        if (lane == 0) {
          next_h = hn;
          verdict = r;
        }
      }
      __syncthreads();
      v = verdict;
      h = next_h;
      __syncthreads();
      if (v != 0) break;
      v = -1;  // unless another step converges
    }
    if (tid == 0) {
      if (v > 0) {
        o_h[nd.e] = h;
        if (o_branch) o_branch[nd.e] = 0;
        atomicAdd(&bcount[0], 1ull);
      } else {
        fails[atomicAdd(n_fails, 1)] = nd.e;
      }
    }
  }
}

// The nodes handed over, more of them than kWideNodes: a wavefront each, from
// where the Newton kernel left them.
__global__ void __launch_bounds__(64 * kHWaves) k_hsolve_rest(const WideNode *wide, const int32_t *n_wide, HUnits U,
                                                             const double *o_xyz, const double *o_s, double hfact,
                                                             double eps, double *o_h, int32_t *o_branch,
                                                             unsigned long long *bcount, int32_t *fails,
                                                             int32_t *n_fails) {
  __shared__ double2 hbuf[kHWaves][64];
  const int wid = threadIdx.x >> 6, n = *n_wide;
  if (n <= kWideNodes) return;
  for (int b = (int)blockIdx.x * kHWaves + wid; b < n; b += (int)gridDim.x * kHWaves) {
    const WideNode nd = wide[b];
    const double *x = o_xyz + 3 * (int64_t)nd.e;
    double h = nd.h;
    int it = nd.it;
    const int branch = newton_wave(U, nd.e, x[0], x[1], x[2], hfact * 2.0 * o_s[nd.e], hfact, eps, hbuf[wid],
                                   [](double) { return false; }, it, h);
    newton_done(nd.e, branch, h, o_h, o_branch, bcount, fails, n_fails);
  }
}

// Node h-solve, second part: the bracket [h0/100, 100 h0] and bisection to
// a width below eps h0, one workgroup of kBWaves wavefronts per node that
// Newton did not solve.  These steps use only the sign of f (and f == 0), so
// they first take sw in tree order, each wave summing its share and the
// shares added in wave order.  The terms are non-negative, so that sum is
// within 2 nhit 2^-53 sw of the unit-order one, which moves f by less than
// nhit 2^-53 he; only when |f| is within that margin are the sums taken again
// in unit order (by the first wave).  Every decision, and so every result,
// is that of the unit-order sums.  Most steps lie far from the root: there
// the tiles' boxes decide, w falling with distance (sw lies between the sums
// of each tile's count times w at its farthest and at its nearest point), for
// a 64th of the work; and nearly all the others binary32 sums within their
// error (he above kLeast32).  The last part of a 1,048,576-particle build took 1.83 ms with
// binary64 sums at every step, 0.68 ms with the boxes, 0.41 ms now (MI355X).
__global__ void __launch_bounds__(64 * kBWaves) k_hsolve_bracket(const int32_t *fails, const int32_t *n_fails,
                                                                HUnits U, const double *o_xyz, const double *o_s,
                                                                double hfact, double eps, double *o_h,
                                                                int32_t *o_branch, unsigned long long *bcount) {
#pragma clang fp contract(off)
  __shared__ double2 hb[64];
  __shared__ double part_sw[kBWaves], part_least[kBWaves];
  __shared__ long long part_hit[kBWaves];
  __shared__ double uo_sw;
  if ((int)blockIdx.x >= *n_fails) return;  // the whole workgroup
  const int wid = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int32_t e = fails[blockIdx.x];
  const double ax = o_xyz[3 * (int64_t)e], ay = o_xyz[3 * (int64_t)e + 1], az = o_xyz[3 * (int64_t)e + 2];
  const double h0 = hfact * 2.0 * o_s[e];
  double lo = 1e-2 * h0, hi = 1e2 * h0;
  double flo = 0.0, hres = h0;
  int phase = 1;  // 1 eval lo, 2 eval hi, 3 bisect, 9 done
  int branch = 1;
  while (phase != 9) {
    double he = lo;
    if (phase == 2) he = hi;
    else if (phase == 3) he = 0.5 * (lo + hi);
    double sw, sd, f;
    int64_t nhit;
    bool known = false;  // the same in every wave
    if (U.n_mid == 0 && he > 1e-90 && he < 1e90) {
      // f < 0 where sw > hfact^3 pi, f > 0 where it is less; 1e-8 covers the
      // rounding of the sums, of f and of this bound
      const double even = hfact * hfact * hfact / kInvPi;
      const auto decide = [&](double least, double most) {
        // over the waves, in wave order
        if ((threadIdx.x & 63) == 0) {
          part_sw[wid] = most;
          part_least[wid] = least;
        }
        __syncthreads();
        most = least = 0.0;
        for (int k = 0; k < kBWaves; ++k) {
          most += part_sw[k];
          least += part_least[k];
        }
        __syncthreads();
        if (least > even + 1e-8 * fabs(even)) {
          known = true;
          f = -1.0;
        } else if (most < even - 1e-8 * fabs(even)) {
          known = true;
          f = 1.0;
        }
      };
      const double ih = 1.0 / he;
      const int64_t nt = (U.nu + 63) >> 6;
      double most = 0.0, least = 0.0;
      for (int64_t t = threadIdx.x; t < nt; t += 64 * kBWaves) {
        const double4 l = U.tlo[t], u = U.thi[t];
        const double cnt = (double)min((int64_t)64, U.nu - 64 * t);
        const double nx = fmax(fmax(l.x - ax, ax - u.x), 0.0), ny = fmax(fmax(l.y - ay, ay - u.y), 0.0),
                     nz = fmax(fmax(l.z - az, az - u.z), 0.0);
        const double mx = fmax(ax - l.x, u.x - ax), my = fmax(ay - l.y, u.y - ay), mz = fmax(az - l.z, u.z - az);
        most += cnt * m4w(sqrt((nx * nx + ny * ny) + nz * nz) * ih * (1.0 - 1e-9));
        least += cnt * m4w(sqrt((mx * mx + my * my) + mz * mz) * ih * (1.0 + 1e-9));
      }
#pragma unroll
      for (int o = 32; o > 0; o >>= 1) {
        most += __shfl_xor(most, o, 64);
        least += __shfl_xor(least, o, 64);
      }
      decide(least * (1.0 - 1e-9), most * (1.0 + 1e-9));
      if (!known && he > kLeast32) {
        // binary32 terms of the near tiles, t = wid mod kBWaves: x within 8e-7,
        // |w'| <= 1, so w within 4e-6; a lane's sum of its tiles within 1e-5
        const int lane = threadIdx.x & 63;
        const float ihf = (float)ih;
        float sum = 0.0f;
        int terms = 0;
        double sum64 = 0.0;
        for (int64_t b = 0; b * kBWaves < nt; b += 64) {
          const int64_t t = (b + lane) * kBWaves + wid;
          uint64_t near = __ballot(t < nt && !box_beyond(U.tlo[t < nt ? t : 0], U.thi[t < nt ? t : 0], ax, ay, az, ih));
          for (; near; near &= near - 1ull) {
            const int64_t u = 64 * ((b + __builtin_ctzll(near)) * kBWaves + wid) + lane;
            const double4 p = U.upos[u < U.nu ? u : 0];
            const float dx = (float)(ax - p.x), dy = (float)(ay - p.y), dz = (float)(az - p.z);
            const float x = __builtin_amdgcn_sqrtf(dx * dx + dy * dy + dz * dz) * ihf, y = 2.0f - x;
            const float w = x < 1.0f ? 1.0f + x * x * (0.75f * x - 1.5f) : 0.25f * y * y * y;
            const bool in = u < U.nu && x < 2.0f;
            sum += in ? w : 0.0f;
            terms += in;
          }
          sum64 += (double)sum;  // at most 64 tiles a lane in binary32
          sum = 0.0f;
        }
        double err = 4e-6 * (double)terms + 1e-5 * sum64 + 1e-9;
#pragma unroll
        for (int o = 32; o > 0; o >>= 1) {
          sum64 += __shfl_xor(sum64, o, 64);
          err += __shfl_xor(err, o, 64);
        }
        decide(sum64 - err, sum64 + err);
      }
    }
    if (!known) {
      hsums<8>(U, e, ax, ay, az, he, true, wid, kBWaves, hb, sw, sd, nhit);
      if ((threadIdx.x & 63) == 0) {
        part_sw[wid] = sw;
        part_hit[wid] = nhit;
      }
      __syncthreads();
      sw = 0.0;
      nhit = 0;
      for (int k = 0; k < kBWaves; ++k) {  // in wave order
        sw += part_sw[k];
        nhit += part_hit[k];
      }
      f = h_residual(sw, he, hfact);
      if (!(fabs(f) > he * (1e-12 + 4.0 * (double)nhit * 0x1p-53))) {  // the same in every wave
        if (wid == 0) {
          hsums<8>(U, e, ax, ay, az, he, false, 0, 1, hb, sw, sd, nhit);
          if ((threadIdx.x & 63) == 0) uo_sw = sw;
        }
        __syncthreads();
        f = h_residual(uo_sw, he, hfact);
      }
      __syncthreads();  // every wave has read the shared sums before they are written again
    }
    if (phase == 1) {
      flo = f;
      if (f == 0.0) {
        hres = lo;
        phase = 9;
      } else {
        phase = 2;
      }
    } else if (phase == 2) {
      if (f == 0.0) {
        hres = hi;
        phase = 9;
      } else if ((flo < 0.0) == (f < 0.0)) {
        hres = h0;
        branch = 2;
        phase = 9;
      } else if (!(hi - lo >= eps * h0)) {
        hres = 0.5 * (lo + hi);
        phase = 9;
      } else {
        phase = 3;
      }
    } else {  // bisection step at mid = he
      if (f == 0.0) {
        hres = he;
        phase = 9;
      } else {
        if ((f < 0.0) == (flo < 0.0)) {
          lo = he;
          flo = f;
        } else {
          hi = he;
        }
        if (!(hi - lo >= eps * h0)) {
          hres = 0.5 * (lo + hi);
          phase = 9;
        }
      }
    }
  }
  if (threadIdx.x == 0) {
    o_h[e] = hres;
    if (o_branch) o_branch[e] = branch;
    atomicAdd(&bcount[branch], 1ull);
  }
}

struct Grow {
  Arena &ar;
  int64_t cap = 0;
  NodeArrays N{};
  explicit Grow(Arena &a) : ar(a) {}
  void ensure(int64_t need, int64_t used, hipStream_t s) {
    if (need <= cap) return;
    int64_t nc = std::max<int64_t>(need, cap * 2);
    NodeArrays M;
    const char *names[6] = {"ps_first", "ps_count", "ps_parent", "ps_cfirst", "ps_nchild", "ps_level"};
    int32_t **dst[6] = {&M.first, &M.count, &M.parent, &M.child_first, &M.nchild, &M.level};
    int32_t *src[6] = {N.first, N.count, N.parent, N.child_first, N.nchild, N.level};
    for (int k = 0; k < 6; ++k) {
      std::string nm = std::string(names[k]) + (cap ? "_b" : "_a") + std::to_string(nc);
      *dst[k] = ar.get<int32_t>(nm, nc);
      if (used > 0) SPH_HIP(hipMemcpyAsync(*dst[k], src[k], used * sizeof(int32_t), hipMemcpyDeviceToDevice, s));
    }
    N = M;
    cap = nc;
  }
};

}  // namespace

namespace {
__global__ void k_unit_tiles(int64_t nu, const double4 *upos, double4 *tlo, double4 *thi) {
  const int64_t t = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (t * 64 >= nu) return;
  double4 lo = make_double4(INFINITY, INFINITY, INFINITY, 0.0), hi = make_double4(-INFINITY, -INFINITY, -INFINITY, 0.0);
  for (int64_t u = 64 * t; u < min(nu, 64 * t + 64); ++u) {
    const double4 p = upos[u];
    lo.x = fmin(lo.x, p.x);
    lo.y = fmin(lo.y, p.y);
    lo.z = fmin(lo.z, p.z);
    hi.x = fmax(hi.x, p.x);
    hi.y = fmax(hi.y, p.y);
    hi.z = fmax(hi.z, p.z);
  }
  tlo[t] = lo;
  thi[t] = hi;
}

// the boxes of blocks of 64 tiles, from the tiles' boxes
__global__ void k_unit_blocks(int64_t nt, const double4 *tlo, const double4 *thi, double4 *blo, double4 *bhi) {
  const int64_t b = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (b * 64 >= nt) return;
  double4 lo = tlo[64 * b], hi = thi[64 * b];
  for (int64_t t = 64 * b + 1; t < min(nt, 64 * b + 64); ++t) {
    const double4 l = tlo[t], u = thi[t];
    lo.x = fmin(lo.x, l.x);
    lo.y = fmin(lo.y, l.y);
    lo.z = fmin(lo.z, l.z);
    hi.x = fmax(hi.x, u.x);
    hi.y = fmax(hi.y, u.y);
    hi.z = fmax(hi.z, u.z);
  }
  blo[b] = lo;
  bhi[b] = hi;
}
}  // namespace

void node_hsolve(Ctx &ctx, int64_t np, const int32_t *plist, int64_t nu, const double4 *upos, const double *o_xyz,
                 const double *o_s, double hfact, double eps, int64_t bypass, double *o_h, int32_t *o_branch,
                 unsigned long long *bcount, int64_t n_mid, const double4 *mid_com, const int32_t *mid_u0,
                 const int32_t *mid_u1, const double *rcut, hipStream_t s) {
  if (np <= 0) return;
  const int64_t nt = div_up(nu, 64);
  double4 *tlo = ctx.arena.get<double4>("hs_tlo", std::max<int64_t>(nt, 1));
  double4 *thi = ctx.arena.get<double4>("hs_thi", std::max<int64_t>(nt, 1));
  const int64_t nb = div_up(nt, 64);
  double4 *blo = ctx.arena.get<double4>("hs_blo", std::max<int64_t>(nb, 1));
  double4 *bhi = ctx.arena.get<double4>("hs_bhi", std::max<int64_t>(nb, 1));
  if (nt > 0) {
    k_unit_tiles<<<(unsigned)div_up(nt, 256), 256, 0, s>>>(nu, upos, tlo, thi);
    SPH_LAUNCH_CHECK();
    k_unit_blocks<<<(unsigned)div_up(nb, 256), 256, 0, s>>>(nt, tlo, thi, blo, bhi);
    SPH_LAUNCH_CHECK();
  }
  int32_t *fails = ctx.arena.get<int32_t>("hs_fails", np);
  int32_t *n_fails = ctx.arena.get<int32_t>("hs_nfails", 2);
  int32_t *n_wide = n_fails + 1;
  // (under a workspace cap, and where memory is short, every node stays with its
  // wave: no new scratch)
  WideNode *wide = ctx.ws.limit ? nullptr : ctx.arena.get_if<WideNode>("hs_wide", np);
  k_fill_i32<<<1, 64, 0, s>>>(n_fails, 0, 2);
  SPH_LAUNCH_CHECK();
  const HUnits U{nu, upos, tlo, thi, blo, bhi, n_mid, mid_com, mid_u0, mid_u1, rcut};
  KernelTimer kt(&ctx, "node_hsolve", s);
  KernelTimer kt1(&ctx, "node_hsolve_newton", s);
  k_hsolve_newton<<<(unsigned)div_up(np, kHWaves), 64 * kHWaves, 0, s>>>(np, plist, U, o_xyz, o_s, hfact, eps, bypass,
                                                                        o_h, o_branch, bcount, fails, n_fails, wide,
                                                                        n_wide);
  SPH_LAUNCH_CHECK();
  if (wide && np <= bypass && n_mid == 0 && nt > kNearTiles) {
    k_hsolve_wide<<<(unsigned)std::min<int64_t>(np, 1024), 64 * kWideWaves, 0, s>>>(
        wide, n_wide, U, o_xyz, o_s, hfact, eps, o_h, o_branch, bcount, fails, n_fails);
    SPH_LAUNCH_CHECK();
    if (np > kWideNodes) {
      k_hsolve_rest<<<(unsigned)div_up(np, kHWaves), 64 * kHWaves, 0, s>>>(wide, n_wide, U, o_xyz, o_s, hfact, eps,
                                                                          o_h, o_branch, bcount, fails, n_fails);
      SPH_LAUNCH_CHECK();
    }
  }
  kt1.done();
  // one workgroup per node that Newton did not solve (the rest exit at
  // once); above the bypass every node took h0 and none is left
  if (np <= bypass) {
    KernelTimer kt2(&ctx, "node_hsolve_bracket", s);
    k_hsolve_bracket<<<(unsigned)np, 64 * kBWaves, 0, s>>>(fails, n_fails, U, o_xyz, o_s, hfact, eps, o_h, o_branch,
                                                           bcount);
    SPH_LAUNCH_CHECK();
    kt2.done();
  }
  kt.done();
}

void pseudo_build(Ctx &ctx, PseudoArgs &a, hipStream_t s) {
  Arena &ar = ctx.arena;
  const int64_t n = a.n;
  const auto &o = a.opts;
  int *bad = ar.get<int>("ps_bad", 1);
  SPH_HIP(hipMemsetAsync(bad, 0, sizeof(int), s));
  k_check_unit_cube<<<(unsigned)div_up(n, 256), 256, 0, s>>>(n, a.xyz, bad);
  SPH_LAUNCH_CHECK();
  int bad_h = 0;
  SPH_HIP(hipMemcpyAsync(&bad_h, bad, sizeof(int), hipMemcpyDeviceToHost, s));
  SPH_HIP(hipStreamSynchronize(s));
  SPH_REQUIRE(bad_h == 0, SPHMAP_EINVAL, std::to_string(bad_h) + " particle(s) outside [0,1)^3");

  // Morton order in the unit cube
  uint64_t *keys = ar.get<uint64_t>("ps_keys", n);
  int32_t *sidx = ar.get<int32_t>("ps_sidx", n);
  morton_keys(a.xyz, 3, n, 0.0, 0.0, 0.0, 1.0, keys, sidx, s);
  radix_sort_u64(ar, keys, sidx, n, 63, s);

  // level-synchronous octree build
  Grow G(ar);
  G.ensure(std::max<int64_t>(2 * n / std::max(o.leaf_max, 1) + 64, 1024), 0, s);
  // The levels' sizes stay on the device: a run of levels is launched on an
  // upper bound of its nodes (eight times as many a level) and read back at
  // its end.  The first run is as deep as the tree has to be for leaves of
  // leaf_max particles, the others two levels; a level past the last is empty
  // and changes nothing, and one without room is run again.  A run of one
  // level, as under a workspace cap, knows its exact size.
  // A level of 1,048,576 particles took 45 us of waiting for its size and 25 us
  // of split by one lane a node; the build 2.96 ms, now 2.76, and of 100,000
  // and 8,000 particles 1.78 and 1.11, now 1.66 and 1.06 (MI355X).
  int64_t *lv = ar.get<int64_t>("ps_lv", kMaxLevels + 4);
  k_root<<<1, 1, 0, s>>>(G.N, n, lv);
  SPH_LAUNCH_CHECK();
  std::vector<int64_t> loff = {0, 1};  // level offsets
  int run = 1;
  if (!ctx.ws.limit)
    while (run < 21 && ((int64_t)std::max(o.leaf_max, 1) << (3 * run)) < n) ++run;
  for (bool done = false; !done;) {
    const int d0 = (int)loff.size() - 2, d1 = std::min(d0 + run, o.max_depth + 1);
    int64_t nb = loff[d0 + 1] - loff[d0];
    for (int d = d0; d < d1; ++d, nb = std::min(8 * nb, n)) {
      // (in buffers that are filled after the build: no scratch of their own)
      const int64_t room = ctx.ws.limit ? nb : n;  // no growth between the launches of a run
      int64_t *nch = ar.get<int64_t>("ps_flag", room + 1);
      int64_t *choff = ar.get<int64_t>("ps_uoff", room + 1);
      k_split<<<strided_blocks(8 * nb), 256, 0, s>>>(G.N, lv + 1 + d, nb, d, keys, o.leaf_max, o.max_depth, nch);
      SPH_LAUNCH_CHECK();
      scan_exclusive_i64(ar, nch, choff, nb, true, s);
      k_children<<<strided_blocks(8 * nb), 256, 0, s>>>(G.N, lv + 1 + d, lv, nb, G.cap, d, keys, o.leaf_max,
                                                              o.max_depth, choff);
      SPH_LAUNCH_CHECK();
    }
    int64_t got[kMaxLevels + 4];
    SPH_HIP(hipMemcpyAsync(got, lv, (d1 + 3) * sizeof(int64_t), hipMemcpyDeviceToHost, s));
    SPH_HIP(hipStreamSynchronize(s));
    run = ctx.ws.limit ? 1 : 2;
    for (int d = d0; d < d1 && !done; ++d) {
      const int64_t e = loff.back(), next = got[d + 3];
      if (next == e && got[0] > 0) {  // this level's children lacked room
        G.ensure(e + got[0], e, s);
        SPH_HIP(hipMemsetAsync(lv, 0, sizeof(int64_t), s));
        break;
      }
      loff.push_back(next);
      done = next == e;
    }
  }
  const int64_t nn = loff.back();
  const NodeArrays &N = G.N;

  // moments
  double *M = ar.get<double>("ps_M", nn);
  double4 *S = ar.get<double4>("ps_S", nn);
  double4 *com = ar.get<double4>("ps_com", nn);
  double *s2 = ar.get<double>("ps_s2", nn);
  int32_t *minidx = ar.get<int32_t>("ps_minidx", nn);
  int8_t *acc = ar.get<int8_t>("ps_acc", nn);
  int8_t *asc = ar.get<int8_t>("ps_asc", nn);
  k_leaf_moments<<<(unsigned)div_up(nn, 256), 256, 0, s>>>(N, nn, sidx, a.xyz, a.m, M, S, asc);
  SPH_LAUNCH_CHECK();
  for (int level = (int)loff.size() - 2; level >= 0; --level) {
    const int64_t b = loff[level], e = loff[level + 1];
    if (e > b) {
      k_internal_moments<<<(unsigned)div_up(e - b, 256), 256, 0, s>>>(N, b, e, M, S);
      SPH_LAUNCH_CHECK();
    }
  }
  k_com<<<(unsigned)div_up(nn, 256), 256, 0, s>>>(nn, M, S, com);
  SPH_LAUNCH_CHECK();
  double4 *sx = ar.get<double4>("ps_sx", n);
  k_sorted_xyz<<<(unsigned)div_up(n, 256), 256, 0, s>>>(n, sidx, a.xyz, sx);
  SPH_LAUNCH_CHECK();
  k_node_size<<<(unsigned)div_up(nn * 64, 256), 256, 0, s>>>(N, nn, sidx, sx, com, s2, minidx);
  SPH_LAUNCH_CHECK();
  {
    int64_t *bflag = ar.get<int64_t>("ps_bflag", nn + 1);
    int64_t *boff = ar.get<int64_t>("ps_boff", nn + 1);
    // the nodes of a level are disjoint, so its big nodes hold at most
    // n / kBigNode + (their number, itself at most n / kBigNode) chunks
    const int64_t bound = std::max<int64_t>(1, (int64_t)(loff.size() - 1) * (2 * (n / kBigNode) + 1));
    int32_t *blist = ar.get<int32_t>("ps_blist", bound);
    k_flag_big<<<(unsigned)div_up(nn, 256), 256, 0, s>>>(N, nn, bflag);
    SPH_LAUNCH_CHECK();
    scan_exclusive_i64(ar, bflag, boff, nn, true, s);
    k_list_big<<<(unsigned)div_up(nn, 256), 256, 0, s>>>(N, nn, boff, blist);
    SPH_LAUNCH_CHECK();
    k_node_size_big<<<(unsigned)std::min<int64_t>(bound, 2048), 1024, 0, s>>>(N, blist, boff, boff + nn, sidx, sx,
                                                                              com, s2, minidx);
    SPH_LAUNCH_CHECK();
  }
  double *src = ar.get<double>("ps_src", 3 * a.n_src);
  SPH_HIP(hipMemcpyAsync(src, a.src, 3 * a.n_src * sizeof(double), hipMemcpyHostToDevice, s));
  k_accept<<<(unsigned)div_up(nn, 256), 256, 0, s>>>(nn, com, s2, a.n_src, src, o.r_part, o.theta, acc);
  SPH_LAUNCH_CHECK();
  uint64_t *label = ar.get<uint64_t>("ps_label", nn);
  k_label<<<(unsigned)div_up(nn, 256), 256, 0, s>>>(N, nn, keys, label);
  SPH_LAUNCH_CHECK();
  if (a.n_open > 0) {
    uint64_t *op = ar.get<uint64_t>("ps_open", a.n_open);
    int32_t *dummy = ar.get<int32_t>("ps_open_idx", a.n_open);
    SPH_HIP(hipMemcpyAsync(op, a.open_labels, a.n_open * sizeof(uint64_t), hipMemcpyDeviceToDevice, s));
    iota_i32(dummy, a.n_open, s);
    radix_sort_u64(ar, op, dummy, a.n_open, 64, s);
    k_force_open<<<(unsigned)div_up(nn, 256), 256, 0, s>>>(nn, label, a.n_open, op, acc);
    SPH_LAUNCH_CHECK();
  }

  // units in depth-first order
  int32_t *unit_at = ar.get<int32_t>("ps_unit_at", n);
  k_fill_i32<<<(unsigned)div_up(n, 256), 256, 0, s>>>(unit_at, -1, n);
  SPH_LAUNCH_CHECK();
  k_units<<<(unsigned)div_up(nn, 256), 256, 0, s>>>(N, nn, acc, unit_at);
  SPH_LAUNCH_CHECK();
  int64_t *flag = ar.get<int64_t>("ps_flag", n + 1);
  int64_t *uoff = ar.get<int64_t>("ps_uoff", n + 1);
  k_flag<<<(unsigned)div_up(n, 256), 256, 0, s>>>(n, unit_at, flag);
  SPH_LAUNCH_CHECK();
  scan_exclusive_i64(ar, flag, uoff, n, true, s);
  int64_t nu = 0;
  SPH_HIP(hipMemcpyAsync(&nu, uoff + n, sizeof(int64_t), hipMemcpyDeviceToHost, s));
  SPH_HIP(hipStreamSynchronize(s));
  int32_t *units = ar.get<int32_t>("ps_units", nu);
  k_unit_list<<<(unsigned)div_up(n, 256), 256, 0, s>>>(n, unit_at, uoff, units);
  SPH_LAUNCH_CHECK();
  int64_t *ecnt = ar.get<int64_t>("ps_ecnt", nu + 1);
  int64_t *eoff = ar.get<int64_t>("ps_eoff", nu + 1);
  int64_t *pcnt = ar.get<int64_t>("ps_pcnt", nu + 1);
  int64_t *poff = ar.get<int64_t>("ps_poff", nu + 1);
  k_unit_counts<<<(unsigned)div_up(nu, 256), 256, 0, s>>>(nu, units, N, acc, ecnt, pcnt);
  SPH_LAUNCH_CHECK();
  scan_exclusive_i64(ar, ecnt, eoff, nu, true, s);
  scan_exclusive_i64(ar, pcnt, poff, nu, true, s);
  int64_t tot[2] = {0, 0};
  SPH_HIP(hipMemcpyAsync(&tot[0], eoff + nu, sizeof(int64_t), hipMemcpyDeviceToHost, s));
  SPH_HIP(hipMemcpyAsync(&tot[1], poff + nu, sizeof(int64_t), hipMemcpyDeviceToHost, s));
  SPH_HIP(hipStreamSynchronize(s));
  const int64_t n_out = tot[0], np = tot[1];
  SPH_REQUIRE(n_out <= a.capacity, SPHMAP_ERANGE,
              "pseudo-particle output needs " + std::to_string(n_out) + " entries, capacity " +
                  std::to_string(a.capacity));
  double4 *upos = ar.get<double4>("ps_upos", nu);
  int32_t *plist = ar.get<int32_t>("ps_plist", np + 1);
  // the solve reads the node sizes back: keep them in scratch when the
  // caller does not ask for them
  double *o_s = a.o_s ? a.o_s : ar.get<double>("ps_os", n_out);
  k_entries<<<(unsigned)div_up(nu, 256), 256, 0, s>>>(nu, units, N, acc, eoff, poff, sidx, a.xyz, a.h, a.m, M, com,
                                                      s2, minidx, a.o_xyz, a.o_h, a.o_m, o_s, a.o_kind, a.o_first,
                                                      a.o_count, a.o_branch, upos, plist, label, a.o_label, asc);
  SPH_LAUNCH_CHECK();
  if (a.o_owner && n > 0) {
    k_owner<<<(unsigned)div_up(n, 256), 256, 0, s>>>(n, flag, uoff, units, N, acc, eoff, sidx, asc, a.o_owner);
    SPH_LAUNCH_CHECK();
  }

  // node smoothing lengths
  unsigned long long *bcount = ar.get<unsigned long long>("ps_bcount", 4);
  SPH_HIP(hipMemsetAsync(bcount, 0, 4 * sizeof(unsigned long long), s));
  node_hsolve(ctx, np, plist, nu, upos, a.o_xyz, o_s, o.h_fact, o.eps_h, o.bypass_threshold, a.o_h, a.o_branch,
              bcount, 0, nullptr, nullptr, nullptr, nullptr, s);
  unsigned long long bc[4] = {0, 0, 0, 0};
  SPH_HIP(hipMemcpyAsync(bc, bcount, sizeof bc, hipMemcpyDeviceToHost, s));
  SPH_HIP(hipStreamSynchronize(s));
  a.n_out = n_out;
  a.stats.n_nodes = nn;
  a.stats.n_units = nu;
  a.stats.n_pseudo = np;
  a.stats.n_real = n_out - np;
  {
    double r2 = 0.0;
    SPH_HIP(hipMemcpyAsync(&r2, s2, sizeof(double), hipMemcpyDeviceToHost, s));
    SPH_HIP(hipStreamSynchronize(s));
    a.stats.s_root = sqrt(r2);
  }
  for (int k = 0; k < 4; ++k) a.stats.branch_count[k] = (int64_t)bc[k];
}

__global__ void k_underresolved_flag(int64_t n, const int32_t *kind, const double *s_node, const double *fneu,
                                     double s_root, double K, int64_t *flag) {
  const int64_t e = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (e >= n) return;
  // eq. resol_param: f_neu,limit = (1/K) (K - 1 / (s_node / s_root))
  flag[e] = (kind[e] == 1 && fneu[e] < (K - 1.0 / (s_node[e] / s_root)) / K) ? 1 : 0;
}

__global__ void k_underresolved_list(int64_t n, const int64_t *flag, const int64_t *off, const uint64_t *label,
                                     uint64_t *out) {
  const int64_t e = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (e < n && flag[e]) out[off[e]] = label[e];
}

int64_t select_underresolved(Ctx &ctx, int64_t n, const int32_t *kind, const uint64_t *label, const double *s_node,
                             const double *fneu, double s_root, double K, uint64_t *out, hipStream_t s) {
  if (n <= 0) return 0;
  int64_t *flag = ctx.arena.get<int64_t>("ur_flag", n + 1);
  int64_t *off = ctx.arena.get<int64_t>("ur_off", n + 1);
  k_underresolved_flag<<<(unsigned)div_up(n, 256), 256, 0, s>>>(n, kind, s_node, fneu, s_root, K, flag);
  SPH_LAUNCH_CHECK();
  scan_exclusive_i64(ctx.arena, flag, off, n, true, s);
  k_underresolved_list<<<(unsigned)div_up(n, 256), 256, 0, s>>>(n, flag, off, label, out);
  SPH_LAUNCH_CHECK();
  int64_t cnt = 0;
  SPH_HIP(hipMemcpyAsync(&cnt, off + n, sizeof(int64_t), hipMemcpyDeviceToHost, s));
  SPH_HIP(hipStreamSynchronize(s));
  return cnt;
}

}  // namespace sphmap
