// The Voronoi grid on the device (Sec. 2.3: the grid code builds the Voronoi
// grid of the generation sites and regularises it with Lloyd iterations
// before the forward mapping).
//
// Cell of generator g: the box cut by the bisector half-space of every
// generator that can reach it.  One wavefront builds one cell.  The convex
// cell is held as the triangulation dual to its faces: each vertex of the
// cell is a triangle (a, b, c) of the three planes that meet there, in an
// orientation shared by all triangles, and a table T[a][b] names the
// triangle holding the directed edge a -> b.  A cut by plane p removes the
// vertices beyond it; every edge a -> b of a removed triangle whose twin
// b -> a belongs to a kept triangle is a cell edge crossing p, and becomes
// the new vertex (a, b, p) at the crossing point.
//
// Building a cell is a chain of about 25 cuts, each a chain of dependent
// steps, so what counts is the latency of one cut (and the waves beside it).
// Vertex t lives in the registers of lane t mod 64 and never moves: a new
// vertex takes a free slot, so only the new triangles' entries of T are
// written.  Whether a vertex is cut is a bit of a scalar mask, counts and
// ranks are population counts of such masks, and the largest vertex distance
// comes from a lane-shift (DPP) reduction; LDS is left for T, for the
// positions of twin vertices and for handing new vertices to their slots.
// (With the vertices compacted and T rebuilt after each cut, shuffles for
// the scans and sums, and a uniform site grid, 131,071 turbulent sites took
// 5.95 ms a construction; now 2.2 ms at first and 1.4 ms once regularised,
// about 26,000 cycles of a SIMD a cell, most of them vector issue, of 64
// lanes for about 25 vertices; the final grid's fixed order 2.7 ms,
// once, against 5.1 ms twice.)
//
// Lloyd iterations find neighbours through nested grids of cubic cells: the
// sites are sorted by the Morton order of the finest level's cells, so that a
// cell of any level is one run of the sorted sites.  A site's search starts
// at the finest level whose own cell holds at least three sites, takes the
// sites within a radius of that cell's size nearest first, and goes on in
// growing radii, each at the level of its size.  A generator at distance D
// can cut only when D/2 does not exceed the largest vertex distance R of the
// current cell, so the search stops once its radius reaches 2R (the security
// radius).  A single grid made for the mean density lists hundreds of sites
// around each site of a dense clump.
//
// The final grid's faces and vertices are numbered by the order of the cuts,
// which callers see (sphmap_tess_export) and which the mixed path's rounding
// follows, so its construction keeps one fixed order: a uniform grid of
// about two generators a cell, searched in rings of growing Chebyshev
// radius; the 64 nearest sites of rings 0 and 1 first, then every site 64
// at a time as the grid lists them, each batch nearest first.  Vertices
// carry their age (the cut that made them, and their place in it), so that
// slots reused in any order still give the numbering of a list that only
// closes up and grows.
//
// Outputs: volume and centroid (Lloyd iterations); face, face vertex and
// vertex counts; the faces themselves (each face's vertex cycle walked
// through T) with the neighbour each one faces.
#include "common.hpp"

namespace sphmap {
namespace {

constexpr int kVP = 64;     // planes per cell: 6 box planes + neighbours
constexpr int kVT = 128;    // vertices per cell
constexpr int kVWaves = 4;  // cells per workgroup
// A cell under construction can have more faces than the finished one (a
// lone site facing a clump); the few that outgrow kVP planes are built again
// with twice the room, and only a finished cell beyond kVP is refused.
constexpr int kVWide = 2;
constexpr int kVLevels = 11;
constexpr int kVStack = 200;
constexpr int kVMany = 256;  // sites in reach beyond which grid cells are tested before sites
constexpr int kVRing = 128;  // the same in the fixed order, whose grid cells are only passed over
constexpr int kVLeaf = 16;   // a grid cell of more sites is then split further

// error bits
constexpr int kErrCoincident = 1;
constexpr int kErrPlanes = 2;
constexpr int kErrVertices = 4;
constexpr int kErrCycle = 8;
constexpr int kErrOutside = 16;

template <int kW>  // kW times the planes and vertices
struct VorLds {    // kW = 1: 9.9 KB, 4 workgroups a CU
  static constexpr int kP = kW * kVP, kT = kW * kVT;
  uint8_t T[kP][kP];              // vertex holding directed edge a -> b
  double vx[kT], vy[kT], vz[kT];  // vertex positions about the generator
  int32_t pid[kP];                // sorted position of the neighbouring generator, or -1..-6 for box planes
  uint32_t stack[kVStack];        // grid cells still to look into: a 1, then the octant digits from the top
  int64_t off[kVLevels];          // the grid levels' first entries (indexed by lane)
  union {
    double foot[kP][3];  // at the end: each plane's offset times its normal
    int32_t list[64];    // positions in the sorted order of the sites of one batch
    uint2 fresh[kP];   // the vertices a cut makes: planes; removed and kept end of the edge they lie on
    struct {             // at the end: the planes of each vertex, its number, a vertex on each plane
      uint32_t tri[kT];
      uint32_t first[kP];
      uint8_t rank[kT], slot[kT];
    } out;
  };
  uint8_t map[kP];
};

struct VorGrid {
  double lo[3], hi[3];
  double cs, ics;       // cell size of the finest level, and its inverse
  int L;                // finest level; level l has cells of cs 2^(L - l)
  int G[3];             // cells of the finest level
  int64_t off[kVLevels];           // each level's first entry in start and end
  const int32_t *start, *end;      // per level and cell (x fastest), into the sorted order
  const double *x;      // [n][3] sites in the sorted order
  const int32_t *id;    // their indices
};

// One cell, spread over a wavefront: vertex lane + 64 h in x[h], y[h], z[h],
// tri[h] (planes a, b, c in bytes 0-2; a free slot has position 0, which no
// bisector cuts); uniform: the live vertex slots, the plane count, and the
// largest vertex distance (rounded up).
// kOrder: with each vertex's age, and R not rounded.
template <int kW, bool kOrder>
struct VorCell {
  static constexpr int kH = 2 * kW;
  double x[kH], y[kH], z[kH];
  uint32_t tri[kH];
  uint32_t age[kOrder ? kH : 1];  // cuts made before it, and its place among its cut's (8 bits)
  uint64_t live[kH];
  int nP, cuts;
  double R;
};

__device__ inline void vsync() {
  __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
  __builtin_amdgcn_wave_barrier();
  __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

// v of the lane a DPP control names, 0 where it names none
template <int kCtrl>
__device__ inline int dpp0(int v) {
  return __builtin_amdgcn_update_dpp(0, v, kCtrl, 0xf, 0xf, false);
}
// exclusive sum over the lanes
__device__ inline int vscan_excl(int v) {
  int x = v;
  x += dpp0<0x111>(x);
  x += dpp0<0x112>(x);
  x += dpp0<0x114>(x);
  x += dpp0<0x118>(x);
  x += __builtin_amdgcn_update_dpp(0, x, 0x142, 0xa, 0xf, false);  // into rows 1 and 3
  x += __builtin_amdgcn_update_dpp(0, x, 0x143, 0xc, 0xf, false);  // into rows 2 and 3
  return x - v;
}
// The reductions' steps: row_shr 1, 2, 4, 8, then row_bcast 15 and 31; the
// last lane holds the result.
template <int kCtrl>
__device__ inline double dpp_add(double v) {
  const int lo = dpp0<kCtrl>(__double2loint(v)), hi = dpp0<kCtrl>(__double2hiint(v));
  return v + __hiloint2double(hi, lo);
}
template <int kCtrl>
__device__ inline float dpp_max(float v) {  // v >= 0
  return fmaxf(v, __int_as_float(dpp0<kCtrl>(__float_as_int(v))));
}
__device__ inline double readlane_d(double v, int j) {
  return __hiloint2double(__builtin_amdgcn_readlane(__double2hiint(v), j),
                          __builtin_amdgcn_readlane(__double2loint(v), j));
}
__device__ inline double vsumd(double v) {
  // row_bcast adds a row's last lane to whole rows below: only lane 63's
  // chain is the full sum
  v = dpp_add<0x111>(v);
  v = dpp_add<0x112>(v);
  v = dpp_add<0x114>(v);
  v = dpp_add<0x118>(v);
  v = dpp_add<0x142>(v);
  v = dpp_add<0x143>(v);
  return readlane_d(v, 63);
}
template <int kCtrl>
__device__ inline double dpp_maxd(double v) {  // v >= 0
  const int lo = dpp0<kCtrl>(__double2loint(v)), hi = dpp0<kCtrl>(__double2hiint(v));
  return fmax(v, __hiloint2double(hi, lo));
}
__device__ inline double vmaxd(double v) {
  v = dpp_maxd<0x111>(v);
  v = dpp_maxd<0x112>(v);
  v = dpp_maxd<0x114>(v);
  v = dpp_maxd<0x118>(v);
  v = dpp_maxd<0x142>(v);
  v = dpp_maxd<0x143>(v);
  return readlane_d(v, 63);
}
__device__ inline float vmaxf(float v) {
  v = dpp_max<0x111>(v);
  v = dpp_max<0x112>(v);
  v = dpp_max<0x114>(v);
  v = dpp_max<0x118>(v);
  v = dpp_max<0x142>(v);
  v = dpp_max<0x143>(v);
  return __int_as_float(__builtin_amdgcn_readlane(__float_as_int(v), 63));
}

__device__ inline uint64_t ballot64(bool p) { return (uint64_t)__ballot(p); }
// set bits of m below this lane
__device__ inline int vrank(uint64_t m) {
  return (int)__builtin_amdgcn_mbcnt_hi((unsigned)(m >> 32), __builtin_amdgcn_mbcnt_lo((unsigned)m, 0u));
}
template <int kH>
__device__ inline bool vbit(const uint64_t (&m)[kH], int t) {
  uint64_t w = m[0];
#pragma unroll
  for (int h = 1; h < kH; ++h) w = (t >> 6) == h ? m[h] : w;
  return (w >> (t & 63)) & 1ull;
}

template <int kW, bool kO>
__device__ inline void vput(VorLds<kW> &L, const VorCell<kW, kO> &C, int h, int t) {
  L.vx[t] = C.x[h];
  L.vy[t] = C.y[h];
  L.vz[t] = C.z[h];
}
template <int kW>
__device__ inline void vlink(VorLds<kW> &L, uint32_t tri, int t) {
  const int a = tri & 0xff, b = (tri >> 8) & 0xff, c = (tri >> 16) & 0xff;
  L.T[a][b] = (uint8_t)t;
  L.T[b][c] = (uint8_t)t;
  L.T[c][a] = (uint8_t)t;
}
template <int kW, bool kO>
__device__ inline void vradius(VorCell<kW, kO> &C) {
  double r2 = C.x[0] * C.x[0] + C.y[0] * C.y[0] + C.z[0] * C.z[0];
#pragma unroll
  for (int h = 1; h < C.kH; ++h)
    if (C.live[h]) r2 = fmax(r2, C.x[h] * C.x[h] + C.y[h] * C.y[h] + C.z[h] * C.z[h]);
  if constexpr (kO) {
    C.R = sqrt(vmaxd(r2));
    return;
  }
  // rounded up throughout (the root is within 1 ulp)
  C.R = (double)(__builtin_amdgcn_sqrtf(vmaxf(__double2float_ru(r2))) * (1.0f + 0x1p-22f));
}

// Drop the planes no vertex lies on any more and renumber the rest.
template <int kW, bool kO>
__device__ void vcompact(VorLds<kW> &L, VorCell<kW, kO> &C, int lane) {
#pragma unroll
  for (int g = 0; g < kW; ++g) L.map[lane + 64 * g] = 0;
  vsync();
#pragma unroll
  for (int h = 0; h < C.kH; ++h)
    if ((C.live[h] >> lane) & 1ull) {
      L.map[C.tri[h] & 0xff] = 1;
      L.map[(C.tri[h] >> 8) & 0xff] = 1;
      L.map[(C.tri[h] >> 16) & 0xff] = 1;
    }
  vsync();
  int count = 0;
#pragma unroll
  for (int g = 0; g < kW; ++g) {  // a plane moves down, past planes already read
    const int q = lane + 64 * g;
    const bool used = q < C.nP && L.map[q];
    const uint64_t um = ballot64(used);
    const int to = count + vrank(um);
    count += __popcll(um);
    const int32_t id = L.pid[q];
    vsync();
    if (used) {
      L.map[q] = (uint8_t)to;
      L.pid[to] = id;
    }
    vsync();
  }
  C.nP = count;
#pragma unroll
  for (int h = 0; h < C.kH; ++h)
    if ((C.live[h] >> lane) & 1ull) {
      const uint32_t t = C.tri[h];
      C.tri[h] = (uint32_t)L.map[t & 0xff] | ((uint32_t)L.map[(t >> 8) & 0xff] << 8) |
                 ((uint32_t)L.map[(t >> 16) & 0xff] << 16);
      vlink(L, C.tri[h], lane + 64 * h);
    }
  vsync();
}

// Cut by n.x <= d (about the generator).  Returns false on an overflow
// (bit in err); R is refreshed after a cut.
template <int kW, bool kO>
__device__ bool vcut(VorLds<kW> &L, VorCell<kW, kO> &C, double nx, double ny, double nz, double d, int32_t id, double eps,
                     int lane, int &err) {
  constexpr int kH = VorCell<kW, kO>::kH;
  uint64_t m[kH], kept[kH];
  uint64_t any = 0ull;
#pragma unroll
  for (int h = 0; h < kH; ++h) {
    m[h] = 0ull;
    if (h == 0 || C.live[h]) m[h] = ballot64(nx * C.x[h] + ny * C.y[h] + nz * C.z[h] - d > eps) & C.live[h];
    kept[h] = C.live[h] & ~m[h];
    any |= m[h];
  }
  if (!any) return true;
  if (C.nP >= L.kP) vcompact(L, C, lane);
  if (C.nP >= L.kP) {
    err = kErrPlanes;
    return false;
  }
  const int p = C.nP;
  if (lane == 0) L.pid[p] = id;
  // each removed vertex names the new ones it hands to the cut: one per edge
  // whose twin is kept, where that cell edge crosses the plane
  int total = 0, room = 0;
  uint32_t mine[kO ? kH : 1] = {}, twin[kO ? kH : 1] = {};  // kO: which edges cross, and the twins
#pragma unroll
  for (int h = 0; h < kH; ++h) {
    room += __popcll(~kept[h]);
    if (!m[h]) continue;  // uniform
    const bool rm = (m[h] >> lane) & 1ull;
    const uint32_t tr = C.tri[h], rot = (tr >> 8) | (tr << 16);  // planes a, b, c and b, c, a
#pragma unroll
    for (int r = 0; r < 3; ++r) {
      const uint32_t u = (tr >> (8 * r)) & (L.kP - 1), v = (rot >> (8 * r)) & (L.kP - 1);
      const int t2 = rm ? L.T[v][u] & (L.kT - 1) : 0;
      const bool nv = rm && !vbit(m, t2);
      const uint64_t b = ballot64(nv);
      const int at = total + vrank(b);
      total += __popcll(b);
      if constexpr (kO) {
        mine[h] |= (uint32_t)nv << r;
        twin[h] |= (uint32_t)t2 << (8 * r);
        continue;
      }
      if (nv && at < L.kP)
        L.fresh[at] = make_uint2(u | (v << 8) | ((uint32_t)p << 16), (uint32_t)(lane + 64 * h) | ((uint32_t)t2 << 8));
    }
  }
  if (total > room || total > L.kP) {
    err = kErrVertices;
    return false;
  }
  if constexpr (kO) {
    // numbered as in a list of the vertices by age: its places 0-63, then
    // 64-127 beside them
    static_assert(kH == 2, "two slots a lane");
    uint32_t key[kH] = {C.age[0], C.age[1]};
    if (C.live[1]) {  // over 64 slots: the place itself
#pragma unroll
      for (int h = 0; h < kH; ++h)
        for (uint64_t w = m[h]; w; w &= w - 1) {
          const int l = __builtin_ctzll(w);
          const uint32_t al = (uint32_t)__builtin_amdgcn_readlane((int)C.age[h], l);
          const int place = __popcll(ballot64(C.age[0] < al) & C.live[0]) + __popcll(ballot64(C.age[1] < al) & C.live[1]);
          if (lane == l) key[h] = (uint32_t)((place & 63) * 2 + (place >> 6));
        }
    }
    int before[kH] = {0, 0};
#pragma unroll
    for (int h = 0; h < kH; ++h)
      for (uint64_t w = m[h]; w; w &= w - 1) {
        const int l = __builtin_ctzll(w);
        const uint32_t kl = (uint32_t)__builtin_amdgcn_readlane((int)key[h], l);
        const int nl = __popc((unsigned)__builtin_amdgcn_readlane((int)mine[h], l));
        before[0] += kl < key[0] ? nl : 0;
        before[1] += kl < key[1] ? nl : 0;
      }
#pragma unroll
    for (int h = 0; h < kH; ++h) {
      if (!m[h]) continue;  // uniform
      const uint32_t tr = C.tri[h], rot = (tr >> 8) | (tr << 16);
      int at = before[h];
#pragma unroll
      for (int r = 0; r < 3; ++r)
        if ((mine[h] >> r) & 1u) {
          const uint32_t u = (tr >> (8 * r)) & (L.kP - 1), v = (rot >> (8 * r)) & (L.kP - 1);
          L.fresh[at++] = make_uint2(u | (v << 8) | ((uint32_t)p << 16),
                                     (uint32_t)(lane + 64 * h) | (((twin[h] >> (8 * r)) & 0xffu) << 8));
        }
    }
  }
  vsync();
  // free slots take the new vertices in turn; a removed vertex whose slot
  // stays free moves to the generator, which no plane cuts
  bool take[kH];
  int before = 0;  // free slots of the halves before
#pragma unroll
  for (int h = 0; h < kH; ++h) {
    take[h] = false;
    const uint64_t fr = ~kept[h];
    const int k = before + vrank(fr);
    if (h == 0 || C.live[h] || total > before) {  // uniform
      take[h] = ((fr >> lane) & 1ull) && k < total;
      if (take[h]) {
        const uint2 f = L.fresh[k];
        const int t = f.y & 0xff, t2 = f.y >> 8;
        const double px = L.vx[t], py = L.vy[t], pz = L.vz[t];
        const double qx = L.vx[t2], qy = L.vy[t2], qz = L.vz[t2];
        const double s1 = nx * px + ny * py + nz * pz - d, s2 = nx * qx + ny * qy + nz * qz - d;
        const double w = fmin(fmax(s1 / (s1 - s2), 0.0), 1.0);
        C.x[h] = px + w * (qx - px);
        C.y[h] = py + w * (qy - py);
        C.z[h] = pz + w * (qz - pz);
        C.tri[h] = f.x;
        if constexpr (kO) C.age[h] = ((uint32_t)(C.cuts + 1) << 8) | (uint32_t)k;
      } else if ((m[h] >> lane) & 1ull) {
        C.x[h] = C.y[h] = C.z[h] = 0.0;
      }
    }
    before += __popcll(fr);
  }
  vsync();  // every end point is read before a slot is written
#pragma unroll
  for (int h = 0; h < kH; ++h) {
    const uint64_t tk = ballot64(take[h]);
    if (!(tk | m[h])) continue;  // uniform
    if (take[h] || ((m[h] >> lane) & 1ull)) vput(L, C, h, lane + 64 * h);
    if (take[h]) vlink(L, C.tri[h], lane + 64 * h);
    C.live[h] = kept[h] | tk;
  }
  C.nP = p + 1;
  ++C.cuts;
  vsync();
  vradius(C);
  return true;
}

// A grid's cell index of a coordinate.
__device__ inline int gcell(double x, double lo, double ics, int G) {
  int i = (int)floor((x - lo) * ics);
  return min(max(i, 0), G - 1);
}

// The slots that vertices have taken so far.
template <int kW, bool kO>
__device__ inline int vslots(const VorCell<kW, kO> &C) {
  int n = 64 - __builtin_clzll(C.live[0] | 1ull);
#pragma unroll
  for (int h = 1; h < C.kH; ++h)
    if (C.live[h]) n = 64 * h + 64 - __builtin_clzll(C.live[h]);
  return n;
}

__device__ inline int rcell(double x, double lo, double cs, int G) {
  int i = (int)floor((x - lo) / cs);
  return min(max(i, 0), G - 1);
}

// Cut by the bisectors of one batch of candidates (lane: the vector to the
// site, its distance and its index), nearest first.  With `test`, the planes
// are first tested against every vertex, one candidate per lane, so that the
// many sites that no longer cut cost no serial step (a plane that cuts no
// vertex cuts none of a smaller cell's).  Returns false on an error (bit in
// err).
template <int kW, bool kO>
__device__ bool vbatch(VorLds<kW> &L, VorCell<kW, kO> &C, bool cand, double ex, double ey, double ez, double dist,
                       int32_t id, bool test, double eps, int lane, int &err) {
  uint64_t cm = ballot64(cand);
  if (!cm) return true;
  if (ballot64(cand && !(dist > 0.0))) {
    err = kErrCoincident;
    return false;
  }
  double nx, ny, nz;
  if constexpr (kO) {
    nx = ex / dist, ny = ey / dist, nz = ez / dist;
  } else {
    const double inv = 1.0 / dist;
    nx = ex * inv, ny = ey * inv, nz = ez * inv;
  }
  const double dd = 0.5 * dist;
  if (test) {
    bool cuts = false;
    const int nT = vslots(C);
#pragma unroll 2
    for (int t = 0; t < nT; ++t) cuts |= nx * L.vx[t] + ny * L.vy[t] + nz * L.vz[t] - dd > eps;
    cand = cand && cuts;
    cm = ballot64(cand);
    if (!cm) return true;
  }
  const float key = (float)dist;
  int rank = 0;
  for (uint64_t m = cm; m; m &= m - 1) {
    const int l = __builtin_ctzll(m);
    const float kl = __int_as_float(__builtin_amdgcn_readlane(__float_as_int(key), l));
    rank += (kl < key || (kl == key && l < lane)) ? 1 : 0;
  }
  if (!cand) rank = -1;
  const int nc = __popcll(cm);
  for (int i = 0; i < nc; ++i) {
    const int l = __builtin_ctzll(ballot64(rank == i));
    const double dl = readlane_d(dd, l);
    if (dl > C.R + eps) break;
    if (!vcut(L, C, readlane_d(nx, l), readlane_d(ny, l), readlane_d(nz, l), dl, __builtin_amdgcn_readlane(id, l), eps,
              lane, err))
      return false;
  }
  return true;
}

// bits of v spread to every third place (v < 2^10)
__device__ inline uint32_t spread3(uint32_t v) {
  v = (v | (v << 16)) & 0x030000ffu;
  v = (v | (v << 8)) & 0x0300f00fu;
  v = (v | (v << 4)) & 0x030c30c3u;
  return (v | (v << 2)) & 0x09249249u;
}
// every third bit of v, gathered
__device__ inline uint32_t gather3(uint32_t v) {
  v &= 0x09249249u;
  v = (v | (v >> 2)) & 0x030c30c3u;
  v = (v | (v >> 4)) & 0x0300f00fu;
  v = (v | (v >> 8)) & 0x030000ffu;
  return (v | (v >> 16)) & 0x3ffu;
}

// Whether the box of half sizes (hx, hy, hz) about (mx, my, mz) meets the ball
// about some vertex through the generator: a site outside those balls is
// nearer to no vertex than the generator, and cuts nothing.
template <int kW, bool kO>
__device__ inline bool vballs(const VorLds<kW> &L, const VorCell<kW, kO> &C, double mx, double my, double mz, double hx,
                              double hy, double hz) {
  const int nT = vslots(C);
  bool in = false;
  for (int t = 0; t < nT; ++t) {
    const double vx = L.vx[t], vy = L.vy[t], vz = L.vz[t];
    const double bx = fmax(fabs(vx - mx) - hx, 0.0), by = fmax(fabs(vy - my) - hy, 0.0),
                 bz = fmax(fabs(vz - mz) - hz, 0.0);
    in |= bx * bx + by * by + bz * bz < (vx * vx + vy * vy + vz * vz) * (1.0 + 1e-9);
  }
  return in;
}

// The sites s0 .. s0 + cnt of a grid cell (ix, iy, iz) `sh` levels above the
// finest, if some point of it lies within rr of the generator and some
// beyond r0.
__device__ inline void vcell(const VorGrid &Gd, int64_t off, int sh, int ix, int iy, int iz, double gx, double gy,
                             double gz, double r0, double rr, int &s0, int &cnt) {
  const int gx_n = (Gd.G[0] + (1 << sh) - 1) >> sh, gy_n = (Gd.G[1] + (1 << sh) - 1) >> sh,
            gz_n = (Gd.G[2] + (1 << sh) - 1) >> sh;
  s0 = cnt = 0;
  if (ix < gx_n && iy < gy_n && iz < gz_n) {
    const double half = 0.5 * Gd.cs * (double)(1 << sh);
    const double mx = fabs(fma(2.0 * ix + 1.0, half, Gd.lo[0] - gx)), my = fabs(fma(2.0 * iy + 1.0, half, Gd.lo[1] - gy)),
                 mz = fabs(fma(2.0 * iz + 1.0, half, Gd.lo[2] - gz));
    const double bx = fmax(mx - half, 0.0), by = fmax(my - half, 0.0), bz = fmax(mz - half, 0.0);
    const double fx = mx + half, fy = my + half, fz = mz + half;
    const double far2 = fx * fx + fy * fy + fz * fz;
    if (bx * bx + by * by + bz * bz <= rr * rr * (1.0 + 1e-9) && (r0 < 0.0 || far2 * (1.0 + 1e-9) >= r0 * r0)) {
      const int64_t cell = off + ((int64_t)iz * gy_n + iy) * gx_n + ix;
      s0 = Gd.start[cell];
      cnt = Gd.end[cell] - s0;
    }
  }
}

// Cut by the sites of up to 64 grid cells (lane: sites s0 .. s0 + cnt).
template <int kW>
__device__ bool vsites(VorLds<kW> &L, VorCell<kW, false> &C, const VorGrid &Gd, int32_t self, double gx, double gy, double gz,
                       int s0, int cnt, double r0, double r1, bool test, double eps, int lane, int &err) {
  const int off = vscan_excl(cnt);
  const int tot = __builtin_amdgcn_readlane(off + cnt, 63);
  for (int w0 = 0; w0 < tot; w0 += 64) {
    const int e0 = max(0, w0 - off), e1 = min(cnt, w0 + 64 - off);
    for (int e = e0; e < e1; ++e) L.list[off + e - w0] = s0 + e;
    vsync();
    const int k = w0 + lane < tot ? L.list[lane] : -1;
    vsync();
    double ex = 0.0, ey = 0.0, ez = 0.0, dist = 0.0;
    bool cand = k >= 0 && k != self;
    if (cand) {
      ex = Gd.x[3 * (int64_t)k] - gx;
      ey = Gd.x[3 * (int64_t)k + 1] - gy;
      ez = Gd.x[3 * (int64_t)k + 2] - gz;
      dist = sqrt(ex * ex + ey * ey + ez * ez);
      cand = dist > r0 && dist <= r1 && 0.5 * dist <= C.R + eps;
    }
    if (!vbatch(L, C, cand, ex, ey, ez, dist, k, test, eps, lane, err)) return false;
    vsync();
  }
  return true;
}

// Cut by every site within r1 of the generator (and beyond r0), from the
// cells of one level.  Where these hold many sites (a lone site near a
// clump), the cells are descended into, and dropped when no vertex's ball
// meets them.
template <int kW>
__device__ bool vreach(VorLds<kW> &L, VorCell<kW, false> &C, const VorGrid &Gd, int32_t self, double gx, double gy, double gz,
                       double r0, double r1, bool test, double eps, int lane, int &err) {
  // the finest level whose cells are at least r1 wide: the sphere meets at
  // most four of them a side, one for each lane
  const double wide = r1 * Gd.ics;
  int sh = __builtin_amdgcn_frexp_exp(wide);
  if (__builtin_amdgcn_frexp_mant(wide) == 0.5) --sh;
  sh = __builtin_amdgcn_readfirstlane(min(max(sh, 0), Gd.L));
  const double rr = r1 * (1.0 + 1e-12) + eps;
  const int ix = (gcell(gx - rr, Gd.lo[0], Gd.ics, Gd.G[0]) >> sh) + (lane & 3);
  const int iy = (gcell(gy - rr, Gd.lo[1], Gd.ics, Gd.G[1]) >> sh) + ((lane >> 2) & 3);
  const int iz = (gcell(gz - rr, Gd.lo[2], Gd.ics, Gd.G[2]) >> sh) + (lane >> 4);
  int s0, cnt;
  vcell(Gd, L.off[Gd.L - sh], sh, ix, iy, iz, gx, gy, gz, r0, rr, s0, cnt);
  const int tot = __builtin_amdgcn_readlane(vscan_excl(cnt) + cnt, 63);
  if (tot <= kVMany || sh == 0)
    return vsites(L, C, Gd, self, gx, gy, gz, s0, cnt, r0, r1, test, eps, lane, err);
  uint64_t some = ballot64(cnt > 0);
  if (cnt > 0)
    L.stack[vrank(some)] =
        (1u << (3 * (Gd.L - sh))) | spread3((uint32_t)ix) | (spread3((uint32_t)iy) << 1) | (spread3((uint32_t)iz) << 2);
  int sp = __popcll(some);
  vsync();
  while (sp > 0) {
    const int take = min(sp, 8);
    sp -= take;
    s0 = cnt = 0;
    uint32_t code = 0;
    int l = 0;
    if ((lane >> 3) < take) {
      code = (L.stack[sp + (lane >> 3)] << 3) | (uint32_t)(lane & 7);
      l = (31 - __builtin_clz(code)) / 3;
      const uint32_t at = code ^ (1u << (3 * l));
      const int jx = (int)gather3(at), jy = (int)gather3(at >> 1), jz = (int)gather3(at >> 2);
      vcell(Gd, L.off[l], Gd.L - l, jx, jy, jz, gx, gy, gz, r0, rr, s0, cnt);
      if (cnt > 0) {
        const double half = 0.5 * Gd.cs * (double)(1 << (Gd.L - l)), hw = half + 8.0 * eps;
        const double mx = fma(2.0 * jx + 1.0, half, Gd.lo[0] - gx), my = fma(2.0 * jy + 1.0, half, Gd.lo[1] - gy),
                     mz = fma(2.0 * jz + 1.0, half, Gd.lo[2] - gz);
        if (!vballs(L, C, mx, my, mz, hw, hw, hw)) cnt = 0;
      }
    }
    // cells of many sites go back to be split further, while there is room
    bool deeper = cnt > kVLeaf && l < Gd.L;
    some = ballot64(deeper);
    if (sp + __popcll(some) > kVStack) {
      deeper = false;
      some = 0ull;
    }
    vsync();
    if (deeper) {
      L.stack[sp + vrank(some)] = code;
      cnt = 0;
    }
    sp += __popcll(some);
    vsync();
    if (ballot64(cnt > 0) && !vsites(L, C, Gd, self, gx, gy, gz, s0, cnt, r0, r1, true, eps, lane, err)) return false;
  }
  return true;
}

// The box about a site: planes x-, x+, y-, y+, z-, z+ and its eight corners.
template <int kW, bool kO>
__device__ inline void vbox(VorLds<kW> &L, VorCell<kW, kO> &C, const double (&lo)[3], const double (&hi)[3], double gx,
                            double gy, double gz, int lane) {
#pragma unroll
  for (int h = 0; h < C.kH; ++h) {
    C.x[h] = C.y[h] = C.z[h] = 0.0;
    C.tri[h] = 0;
    C.live[h] = 0ull;
    if constexpr (kO) C.age[h] = (uint32_t)lane;
  }
  if (lane < 6) L.pid[lane] = -1 - lane;
  if (lane < 8) {
    const int sx = lane & 1, sy = (lane >> 1) & 1, sz = (lane >> 2) & 1;
    const int px = sx ? 1 : 0, py = sy ? 3 : 2, pz = sz ? 5 : 4;
    // corner (+,+,+) is (x+, y+, z+); a reflection swaps the orientation
    const bool pos3 = (sx ? 1 : -1) * (sy ? 1 : -1) * (sz ? 1 : -1) > 0;
    C.tri[0] = (uint32_t)px | ((uint32_t)(pos3 ? py : pz) << 8) | ((uint32_t)(pos3 ? pz : py) << 16);
    C.x[0] = (sx ? hi[0] : lo[0]) - gx;
    C.y[0] = (sy ? hi[1] : lo[1]) - gy;
    C.z[0] = (sz ? hi[2] : lo[2]) - gz;
    vput(L, C, 0, lane);
    vlink(L, C.tri[0], lane);
  }
  C.live[0] = 0xffull;
  C.nP = 6;
  C.cuts = 0;
  vsync();
  vradius(C);
}

// The centroid of the cell of sorted site i.  Returns its error bits (0: done).
template <int kW>
__device__ int lloyd_cell(VorLds<kW> &L, const VorGrid &Gd, int64_t i, double eps, double *centroid, int lane) {
  const int32_t self = (int32_t)i;
  const int64_t c = Gd.id[i];
  const double gx = Gd.x[3 * i], gy = Gd.x[3 * i + 1], gz = Gd.x[3 * i + 2];
  VorCell<kW, false> C;
#pragma unroll
  for (int l = 0; l < kVLevels; ++l)
    if (lane == l) L.off[l] = Gd.off[l];
  vbox(L, C, Gd.lo, Gd.hi, gx, gy, gz, lane);
  // the first radius: the size of the finest own cell with three sites, less
  // where the finest level's own cell holds more than four
  double r1;
  {
    int cnt = 0;
    if (lane <= Gd.L) {
      const int sh = Gd.L - lane;
      const int64_t ix = gcell(gx, Gd.lo[0], Gd.ics, Gd.G[0]) >> sh, iy = gcell(gy, Gd.lo[1], Gd.ics, Gd.G[1]) >> sh,
                    iz = gcell(gz, Gd.lo[2], Gd.ics, Gd.G[2]) >> sh;
      const int64_t gx_n = (Gd.G[0] + (1 << sh) - 1) >> sh, gy_n = (Gd.G[1] + (1 << sh) - 1) >> sh;
      const int64_t cell = L.off[lane] + (iz * gy_n + iy) * gx_n + ix;
      cnt = Gd.end[cell] - Gd.start[cell];
    }
    const int l0 = 63 - __builtin_clzll(ballot64(cnt >= 3) | 1ull);
    const int own = __builtin_amdgcn_readlane(cnt, l0);
    r1 = Gd.cs * (double)(1 << (Gd.L - l0));
    if (own > 4) r1 *= (double)cbrtf(4.0f / (float)own);
  }
  double r0 = -1.0;
  for (int turn = 0; turn < 64; ++turn) {
    int err = 0;
    if (!vreach(L, C, Gd, self, gx, gy, gz, r0, r1, turn > 0, eps, lane, err)) return err;
    const double need = 2.0 * C.R + 2.0 * eps;
    if (r1 >= need) break;
    r0 = r1;
    r1 = fmin(2.0 * r1, need * (1.0 + 1e-12));
  }
  if (kW > 1) {  // the finished cell's limits
    vcompact(L, C, lane);
    int nv = 0;
#pragma unroll
    for (int h = 0; h < C.kH; ++h) nv += __popcll(C.live[h]);
    if (C.nP > kVP) return kErrPlanes;
    if (nv > kVT) return kErrVertices;
  }
  // volume and centroid: over every directed cell edge on face x, the
  // tetrahedron (g, foot of g on x, edge start, edge end)
  if (lane < C.nP) {  // (a finished cell has at most 64 planes)
    const int64_t q = L.pid[lane];
    double f[3];
#pragma unroll
    for (int a = 0; a < 3; ++a) {
      const double ga = a == 0 ? gx : (a == 1 ? gy : gz);
      // half way to the neighbour, or the box plane's foot point
      f[a] = q >= 0 ? 0.5 * (Gd.x[3 * q + a] - ga) : 0.0;
      if (q == -1 - 2 * a) f[a] = Gd.lo[a] - ga;
      if (q == -2 - 2 * a) f[a] = Gd.hi[a] - ga;
    }
    L.foot[lane][0] = f[0];
    L.foot[lane][1] = f[1];
    L.foot[lane][2] = f[2];
  }
  vsync();
  double V = 0.0, Sx = 0.0, Sy = 0.0, Sz = 0.0;
#pragma unroll
  for (int h = 0; h < C.kH; ++h) {
    if ((C.live[h] >> lane) & 1ull) {
      const double px = C.x[h], py = C.y[h], pz = C.z[h];
#pragma unroll
      for (int r = 0; r < 3; ++r) {
        const int x = (C.tri[h] >> (8 * r)) & 0xff, z = (C.tri[h] >> (8 * ((r + 2) % 3))) & 0xff;
        const int t2 = L.T[x][z] & (L.kT - 1);
        const double fx = L.foot[x][0], fy = L.foot[x][1], fz = L.foot[x][2];
        const double ux = L.vx[t2], uy = L.vy[t2], uz = L.vz[t2];
        const double cx = py * uz - pz * uy, cy = pz * ux - px * uz, cz = px * uy - py * ux;
        const double vol = (fx * cx + fy * cy + fz * cz) / 6.0;
        V += vol;
        Sx += vol * (fx + px + ux) / 4.0;
        Sy += vol * (fy + py + uy) / 4.0;
        Sz += vol * (fz + pz + uz) / 4.0;
      }
    }
  }
  V = vsumd(V);
  Sx = vsumd(Sx);
  Sy = vsumd(Sy);
  Sz = vsumd(Sz);
  if (lane == 0) {
    centroid[3 * c] = gx + Sx / V;
    centroid[3 * c + 1] = gy + Sy / V;
    centroid[3 * c + 2] = gz + Sz / V;
  }
  return 0;
}

// workgroups go to the eight XCDs in turn: each XCD takes a contiguous
// eighth of the sorted sites, whose neighbourhoods meet in its L2 (the grid
// is a multiple of eight workgroups)
__device__ inline int64_t xcd_cell(int w) {
  const int64_t per = gridDim.x / 8, b = blockIdx.x;
  return ((b & 7) * per + (b >> 3)) * kVWaves + w;
}

// Every cell's centroid; cells that outgrow the room are listed (wide_n of
// them, at most n) for k_lloyd_wide.
__global__ void __launch_bounds__(64 * kVWaves, 4) k_lloyd(VorGrid Gd, int64_t n, double eps, double *centroid,
                                                           int *err, int32_t *wide, int32_t *wide_n) {
  __shared__ VorLds<1> S[kVWaves];
  const int w = threadIdx.x >> 6, lane = threadIdx.x & 63;
  const int64_t i = xcd_cell(w);
  if (i >= n) return;
  const int e = lloyd_cell<1>(S[w], Gd, i, eps, centroid, lane);
  if (e && lane == 0) {
    if (e & (kErrPlanes | kErrVertices))
      wide[atomicAdd(wide_n, 1)] = (int32_t)i;
    else
      atomicOr(err, e);
  }
}

__global__ void __launch_bounds__(64) k_lloyd_wide(VorGrid Gd, double eps, double *centroid, int *err,
                                                   const int32_t *wide, const int32_t *wide_n) {
  __shared__ VorLds<kVWide> L;
  const int lane = threadIdx.x;
  const int m = *wide_n;
  for (int j = blockIdx.x; j < m; j += gridDim.x) {
    const int e = lloyd_cell<kVWide>(L, Gd, wide[j], eps, centroid, lane);
    if (e && lane == 0) atomicOr(err, e);
    vsync();
  }
}

// ------------------------------------------------------- the final grid
// The uniform grid of the fixed search order.
struct RingGrid {
  double lo[3], hi[3], cs[3];
  int G[3];
  const int32_t *start, *end;  // per grid cell, into sorted
  const int32_t *sorted;       // generator indices by grid cell
  const double *x;             // [n][3] their positions
  const double *gen;           // [n][3] positions by index
};

// Sort one 64-bit key per lane across the wave, ascending.
__device__ inline uint64_t vsort64(uint64_t key, int lane) {
#pragma unroll
  for (int kk = 2; kk <= 64; kk <<= 1)
#pragma unroll
    for (int jj = kk >> 1; jj > 0; jj >>= 1) {
      const uint64_t other = (uint64_t)__shfl_xor((long long)key, jj, 64);
      const bool up = (lane & kk) == 0, lower = (lane & jj) == 0;
      key = (lower == up) ? (key < other ? key : other) : (key > other ? key : other);
    }
  return key;
}

// Keep the 64 smallest of two ascending 64-lane lists, ascending.
__device__ inline uint64_t vmerge64(uint64_t best, uint64_t chunk, int lane) {
  const uint64_t rev = (uint64_t)__shfl((long long)chunk, 63 - lane, 64);
  uint64_t key = best < rev ? best : rev;  // bitonic: the 64 smallest of both
#pragma unroll
  for (int jj = 32; jj > 0; jj >>= 1) {
    const uint64_t other = (uint64_t)__shfl_xor((long long)key, jj, 64);
    const bool lower = (lane & jj) == 0;
    key = lower ? (key < other ? key : other) : (key > other ? key : other);
  }
  return key;
}

// Sites w0 .. w0 + 63 of a group of grid cells (lane: sites s0 .. s0 + cnt of
// the sorted array at offset off of the group's tot sites): this lane's, or -1.
__device__ inline int vwindow(VorLds<1> &L, int s0, int cnt, int off, int tot, int w0, int lane) {
  const int e0 = max(0, w0 - off), e1 = min(cnt, w0 + 64 - off);
  for (int e = e0; e < e1; ++e) L.list[off + e - w0] = s0 + e;
  vsync();
  const int k = w0 + lane < tot ? L.list[lane] : -1;
  vsync();
  return k;
}

// Cut by every site of a group (lane: a grid cell's sites, its centre about
// the generator and the squared distance of its nearest point).  With
// `nearest`, the 64 sites nearest to the generator cut first, so that the
// cell is close to its final shape before the rest are tested (far sites
// cutting a large cell first would leave many short-lived faces).  Windows
// of sites that cannot be among the nearest, or whose cells meet no vertex's
// ball, are passed over: the order of the others stays.
__device__ bool vgroup(VorLds<1> &L, VorCell<1, true> &C, const RingGrid &Gd, int32_t c, double gx, double gy,
                       double gz, int s0, int cnt, double mx, double my, double mz, double near2, bool nearest,
                       double eps, int lane, int &err) {
  const int off = vscan_excl(cnt);
  const int tot = __builtin_amdgcn_readlane(off + cnt, 63);
  if (nearest) {
    uint64_t best = ~0ull;
    // the home cell (lane 13 of the 27) first, for a tight bound
    const int home0 = __builtin_amdgcn_readlane(off, 13), home1 = home0 + __builtin_amdgcn_readlane(cnt, 13);
    for (int turn = 0; turn < 2; ++turn)
      for (int w0 = 0; w0 < tot; w0 += 64) {
        const bool home = w0 < home1 && w0 + 64 > home0;
        if (home != (turn == 0)) continue;
        const uint64_t last = (uint64_t)(uint32_t)__builtin_amdgcn_readlane((int)(uint32_t)best, 63) |
                              ((uint64_t)(uint32_t)__builtin_amdgcn_readlane((int)(uint32_t)(best >> 32), 63) << 32);
        if (last != ~0ull) {
          const double far = (double)__uint_as_float((uint32_t)(last >> 32)) * (1.0 + 1e-6);
          if (!ballot64(off < w0 + 64 && off + cnt > w0 && near2 <= far * far)) continue;
        }
        const int k = vwindow(L, s0, cnt, off, tot, w0, lane);
        uint64_t key = ~0ull;
        if (k >= 0) {
          const double ex = Gd.x[3 * (int64_t)k] - gx, ey = Gd.x[3 * (int64_t)k + 1] - gy,
                       ez = Gd.x[3 * (int64_t)k + 2] - gz;
          const int32_t j = Gd.sorted[k];
          if (j != c) key = ((uint64_t)__float_as_uint((float)sqrt(ex * ex + ey * ey + ez * ez)) << 32) | (uint32_t)j;
        }
        if (ballot64(key < last)) best = vmerge64(best, vsort64(key, lane), lane);
      }
    double ex = 0.0, ey = 0.0, ez = 0.0, dist = 0.0;
    const int32_t j = (int32_t)(best & 0xffffffffull);
    const bool some = best != ~0ull;
    if (some) {
      ex = Gd.gen[3 * (int64_t)j] - gx;
      ey = Gd.gen[3 * (int64_t)j + 1] - gy;
      ez = Gd.gen[3 * (int64_t)j + 2] - gz;
      dist = sqrt(ex * ex + ey * ey + ez * ez);
    }
    const int nb = __popcll(ballot64(some));
    if (ballot64(some && !(dist > 0.0))) {
      err = kErrCoincident;
      return false;
    }
    const double nx = ex / dist, ny = ey / dist, nz = ez / dist, dd = 0.5 * dist;
    for (int l = 0; l < nb; ++l) {
      const double dl = readlane_d(dd, l);
      if (dl > C.R + eps) break;
      if (!vcut(L, C, readlane_d(nx, l), readlane_d(ny, l), readlane_d(nz, l), dl, __builtin_amdgcn_readlane(j, l),
                eps, lane, err))
        return false;
    }
  }
  bool reach = cnt > 0;
  if (reach && tot > kVRing)
    reach = vballs(L, C, mx, my, mz, 0.5 * Gd.cs[0] + 8.0 * eps, 0.5 * Gd.cs[1] + 8.0 * eps, 0.5 * Gd.cs[2] + 8.0 * eps);
  for (int w0 = 0; w0 < tot; w0 += 64) {
    if (!ballot64(reach && off < w0 + 64 && off + cnt > w0)) continue;
    const int k = vwindow(L, s0, cnt, off, tot, w0, lane);
    double ex = 0.0, ey = 0.0, ez = 0.0, dist = 0.0;
    int32_t j = 0;
    bool cand = k >= 0;
    if (cand) {
      ex = Gd.x[3 * (int64_t)k] - gx;
      ey = Gd.x[3 * (int64_t)k + 1] - gy;
      ez = Gd.x[3 * (int64_t)k + 2] - gz;
      dist = sqrt(ex * ex + ey * ey + ez * ez);
      cand = 0.5 * dist <= C.R + eps;
      if (cand) {
        j = Gd.sorted[k];
        cand = j != c;
      }
    }
    if (!vbatch(L, C, cand, ex, ey, ez, dist, j, true, eps, lane, err)) return false;
    vsync();
  }
  return true;
}

// The cell of generator c, in the fixed order.
__device__ bool ring_cell(VorLds<1> &L, VorCell<1, true> &C, const RingGrid &Gd, int32_t c, double gx, double gy,
                          double gz, double eps, int lane, int &err) {
  vbox(L, C, Gd.lo, Gd.hi, gx, gy, gz, lane);
  const int hx = rcell(gx, Gd.lo[0], Gd.cs[0], Gd.G[0]);
  const int hy = rcell(gy, Gd.lo[1], Gd.cs[1], Gd.G[1]);
  const int hz = rcell(gz, Gd.lo[2], Gd.cs[2], Gd.G[2]);
  const double csmin = fmin(Gd.cs[0], fmin(Gd.cs[1], Gd.cs[2]));
  const int gmax = max(Gd.G[0], max(Gd.G[1], Gd.G[2]));
  // Candidates are gathered 64 grid cells at a time, one per lane; rings 0
  // and 1 form the first group, so the nearest sites cut first.
  for (int level = 0;; ++level) {
    const int r = level == 0 ? 1 : level + 1;
    if (level >= 1 && r > gmax - 1) break;
    if (level >= 1 && (r - 1) * csmin > 2.0 * C.R + eps) break;
    const int side = 2 * r + 1, ncube = side * side * side;
    for (int q0 = 0; q0 < ncube; q0 += 64) {
      const int q = q0 + lane;
      int cnt = 0, s0 = 0;
      double mx = 0.0, my = 0.0, mz = 0.0, near2 = 0.0;
      if (q < ncube) {
        const int cx = q % side - r, cy = (q / side) % side - r, cz = q / (side * side) - r;
        const bool shell = level == 0 || max(abs(cx), max(abs(cy), abs(cz))) == r;
        const int ix = hx + cx, iy = hy + cy, iz = hz + cz;
        if (shell && ix >= 0 && iy >= 0 && iz >= 0 && ix < Gd.G[0] && iy < Gd.G[1] && iz < Gd.G[2]) {
          // nearest point of the grid cell: nothing there can cut beyond 2R
          const double bx = fmax(fmax(Gd.lo[0] + ix * Gd.cs[0] - gx, gx - (Gd.lo[0] + (ix + 1) * Gd.cs[0])), 0.0);
          const double by = fmax(fmax(Gd.lo[1] + iy * Gd.cs[1] - gy, gy - (Gd.lo[1] + (iy + 1) * Gd.cs[1])), 0.0);
          const double bz = fmax(fmax(Gd.lo[2] + iz * Gd.cs[2] - gz, gz - (Gd.lo[2] + (iz + 1) * Gd.cs[2])), 0.0);
          near2 = bx * bx + by * by + bz * bz;
          if (sqrt(near2) <= 2.0 * C.R + eps) {
            const int64_t cell = ((int64_t)iz * Gd.G[1] + iy) * Gd.G[0] + ix;
            s0 = Gd.start[cell];
            cnt = Gd.end[cell] - s0;
            mx = fma(ix + 0.5, Gd.cs[0], Gd.lo[0] - gx);
            my = fma(iy + 0.5, Gd.cs[1], Gd.lo[1] - gy);
            mz = fma(iz + 0.5, Gd.cs[2], Gd.lo[2] - gz);
          }
        }
      }
      if (!ballot64(cnt > 0)) continue;
      if (!vgroup(L, C, Gd, c, gx, gy, gz, s0, cnt, mx, my, mz, near2, level == 0, eps, lane, err)) return false;
    }
  }
  return true;
}

// A finished cell kept between counting and the final arrays, when it fits
// (about 97% of a Voronoi grid's cells): building it again would cost as much
// as the first time.
struct VorKept {
  double v[40][3];
  int32_t nbr[24];
  uint8_t len[24], fv[128];  // faces' vertex counts, and their vertices by number
};
static_assert(sizeof(VorKept) % 8 == 0, "an array of them stays aligned");

// Mode 1: the counts of every cell, and each cell into `kept` or, where it
// does not fit, into the list (without `kept`: counts only).  Mode 2: the
// faces of the listed cells, or of every cell without a list; the counts
// are then the scanned ones.
template <int kMode>
__device__ void ring_build(VorLds<1> &L, const RingGrid &Gd, int64_t i, double eps, int64_t *cnt_f, int64_t *cnt_p,
                           int64_t *cnt_v, VorKept *kept, int32_t *list, int32_t *list_n, double *vert,
                           int64_t *cell_face_off, int64_t *face_vtx_off, int32_t *face_vtx, int32_t *face_nbr,
                           int *err, int lane) {
  const int32_t c = Gd.sorted[i];
  const double gx = Gd.x[3 * i], gy = Gd.x[3 * i + 1], gz = Gd.x[3 * i + 2];
  VorCell<1, true> C;
  {
    int e = 0;
    if (!ring_cell(L, C, Gd, c, gx, gy, gz, eps, lane, e)) {
      if (lane == 0) atomicOr(err, e);
      return;
    }
  }
  // the vertices' numbers: their places by age
  const int nT = __popcll(C.live[0]) + __popcll(C.live[1]);
  int place[2] = {0, 0};
#pragma unroll
  for (int h = 0; h < 2; ++h)
    for (uint64_t m = C.live[h]; m; m &= m - 1) {
      const uint32_t al = (uint32_t)__builtin_amdgcn_readlane((int)C.age[h], __builtin_ctzll(m));
      place[0] += al < C.age[0] ? 1 : 0;
      place[1] += al < C.age[1] ? 1 : 0;
    }
  L.out.first[lane] = 0u;
  vsync();
  // a face's cycle starts at its vertex of the upper half, then of the later
  // position (a, b, c), then of the higher place in its half
#pragma unroll
  for (int h = 0; h < 2; ++h)
    if ((C.live[h] >> lane) & 1ull) {
      const int t = lane + 64 * h;
      L.out.tri[t] = C.tri[h];
      L.out.rank[t] = (uint8_t)place[h];
      L.out.slot[place[h]] = (uint8_t)t;
#pragma unroll
      for (int r = 0; r < 3; ++r)
        atomicMax(&L.out.first[(C.tri[h] >> (8 * r)) & 0xff],
                  ((uint32_t)(place[h] >> 6) << 16) | ((uint32_t)(r + 1) << 8) | (uint32_t)(place[h] & 63));
    }
  vsync();
  // faces: one lane per plane; a plane is a face when a vertex lies on it
  auto next_of = [&](int t, int p) {  // the vertex after vertex t in plane p's cycle
    const uint32_t tr = L.out.tri[t];
    const int a = tr & 0xff, b = (tr >> 8) & 0xff, cc = (tr >> 16) & 0xff;
    const int nxt = a == p ? cc : (b == p ? a : b);  // the plane before p in (a, b, c)
    return (int)(L.T[p][nxt] & (kVT - 1));
  };
  const uint32_t fk = L.out.first[lane];
  const bool present = lane < C.nP && fk != 0u;
  int len = 0, t0 = 0;
  if (present) {
    t0 = L.out.slot[(fk >> 16) * 64 + (fk & 63)];
    int t = t0;
    do {
      t = next_of(t, lane);
      ++len;
    } while (t != t0 && len <= kVT);
  }
  if (ballot64(len > kVT)) {
    if (lane == 0) atomicOr(err, kErrCycle);
    return;
  }
  const uint64_t pm = ballot64(present);
  const int pi = vscan_excl(len);
  const int fi = vrank(pm);
  if (kMode == 1) {
    const int nf = __popcll(pm), fv = __builtin_amdgcn_readlane(pi + len, 63);
    if (lane == 0) {
      cnt_f[c] = nf;
      cnt_p[c] = fv;
      cnt_v[c] = nT;
    }
    if (!kept) return;
    if (nT > 40 || nf > 24 || fv > 128) {
      if (lane == 0) list[atomicAdd(list_n, 1)] = (int32_t)i;
      return;
    }
    VorKept &K = kept[c];
    if (present) {
      K.nbr[fi] = L.pid[lane];
      K.len[fi] = (uint8_t)len;
      int t = t0;
      for (int k = 0; k < len; ++k) {
        K.fv[pi + k] = L.out.rank[t];
        t = next_of(t, lane);
      }
    }
#pragma unroll
    for (int h = 0; h < 2; ++h)
      if ((C.live[h] >> lane) & 1ull) {
        K.v[place[h]][0] = gx + C.x[h];
        K.v[place[h]][1] = gy + C.y[h];
        K.v[place[h]][2] = gz + C.z[h];
      }
    return;
  }
  const int64_t f0 = cnt_f[c], p0 = cnt_p[c], v0 = cnt_v[c];  // the scanned counts
  if (lane == 0) cell_face_off[c] = f0;
  if (present) {
    face_vtx_off[f0 + fi] = p0 + pi;
    face_nbr[f0 + fi] = L.pid[lane];
    int t = t0, k = 0;
    do {
      face_vtx[p0 + pi + k] = (int32_t)(v0 + L.out.rank[t]);
      t = next_of(t, lane);
      ++k;
    } while (t != t0 && k < len);
  }
#pragma unroll
  for (int h = 0; h < 2; ++h)
    if ((C.live[h] >> lane) & 1ull) {
      const int64_t t = v0 + place[h];
      vert[3 * t] = gx + C.x[h];
      vert[3 * t + 1] = gy + C.y[h];
      vert[3 * t + 2] = gz + C.z[h];
    }
}

template <int kMode>
__global__ void __launch_bounds__(64 * kVWaves, 4) k_voronoi(RingGrid Gd, int64_t n, double eps, int64_t *cnt_f,
                                                             int64_t *cnt_p, int64_t *cnt_v, VorKept *kept,
                                                             int32_t *list, int32_t *list_n, double *vert,
                                                             int64_t *cell_face_off, int64_t *face_vtx_off,
                                                             int32_t *face_vtx, int32_t *face_nbr, int *err) {
  __shared__ VorLds<1> S[kVWaves];
  const int w = threadIdx.x >> 6, lane = threadIdx.x & 63;
  const bool listed = kMode == 2 && list;
  const int64_t m = listed ? (int64_t)*list_n : n;
  // with a list, fewer waves than there may be cells
  for (int64_t j = listed ? (int64_t)blockIdx.x * kVWaves + w : xcd_cell(w); j < m;
       j += listed ? (int64_t)gridDim.x * kVWaves : m) {
    ring_build<kMode>(S[w], Gd, listed ? list[j] : j, eps, cnt_f, cnt_p, cnt_v, kept, list, list_n, vert,
                      cell_face_off, face_vtx_off, face_vtx, face_nbr, err, lane);
    vsync();
  }
}

// The kept cells into the final arrays, one wavefront a cell.
__global__ void __launch_bounds__(256) k_vor_place(int64_t n, const int64_t *cf, const int64_t *cp, const int64_t *cv,
                                                   const int64_t *sf, const int64_t *sp, const int64_t *sv,
                                                   const VorKept *kept, double *vert, int64_t *cell_face_off,
                                                   int64_t *face_vtx_off, int32_t *face_vtx, int32_t *face_nbr) {
  const int lane = threadIdx.x & 63;
  const int64_t c = (int64_t)blockIdx.x * 4 + (threadIdx.x >> 6);
  if (c >= n) return;
  const int nf = (int)cf[c], fv = (int)cp[c], nT = (int)cv[c];
  if (nT > 40 || nf > 24 || fv > 128) return;  // listed
  const VorKept &K = kept[c];
  const int64_t f0 = sf[c], p0 = sp[c], v0 = sv[c];
  const int len = lane < nf ? K.len[lane] : 0;
  const int pi = vscan_excl(len);
  if (lane == 0) cell_face_off[c] = f0;
  if (lane < nf) {
    face_vtx_off[f0 + lane] = p0 + pi;
    face_nbr[f0 + lane] = K.nbr[lane];
  }
  for (int e = lane; e < fv; e += 64) face_vtx[p0 + e] = (int32_t)(v0 + K.fv[e]);
  const double *kv = &K.v[0][0];
  for (int e = lane; e < 3 * nT; e += 64) vert[3 * v0 + e] = kv[e];
}

__global__ void k_ring_keys(int64_t n, const double *g, RingGrid Gd, uint32_t *key, int32_t *idx, int *err) {
  const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= n) return;
  const double x = g[3 * i], y = g[3 * i + 1], z = g[3 * i + 2];
  const bool in = x >= Gd.lo[0] && x <= Gd.hi[0] && y >= Gd.lo[1] && y <= Gd.hi[1] && z >= Gd.lo[2] && z <= Gd.hi[2];
  if (!in) atomicOr(err, kErrOutside);
  if (i == 0) err[1] = 0;  // no cell listed yet
  const int ix = rcell(x, Gd.lo[0], Gd.cs[0], Gd.G[0]);
  const int iy = rcell(y, Gd.lo[1], Gd.cs[1], Gd.G[1]);
  const int iz = rcell(z, Gd.lo[2], Gd.cs[2], Gd.G[2]);
  key[i] = (uint32_t)(((int64_t)iz * Gd.G[1] + iy) * Gd.G[0] + ix);
  idx[i] = (int32_t)i;
}

__global__ void k_ring_bounds(int64_t n, const uint32_t *key, const double *g, const int32_t *sorted, double *x,
                              int32_t *start, int32_t *end) {
  const int64_t k = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (k >= n) return;
  const int64_t i = sorted[k];
  x[3 * k] = g[3 * i];
  x[3 * k + 1] = g[3 * i + 1];
  x[3 * k + 2] = g[3 * i + 2];
  const uint32_t c = key[k];
  if (k == 0 || key[k - 1] != c) start[c] = (int32_t)k;
  if (k == n - 1 || key[k + 1] != c) end[c] = (int32_t)(k + 1);
}

__global__ void k_vor_keys(int64_t n, const double *g, VorGrid Gd, uint32_t *key, int32_t *idx, int *err) {
  const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i == 0) err[1] = 0;  // no cell listed yet
  if (i >= n) return;
  const double x = g[3 * i], y = g[3 * i + 1], z = g[3 * i + 2];
  const bool in = x >= Gd.lo[0] && x <= Gd.hi[0] && y >= Gd.lo[1] && y <= Gd.hi[1] && z >= Gd.lo[2] && z <= Gd.hi[2];
  if (!in) atomicOr(err, kErrOutside);
  key[i] = spread3(gcell(x, Gd.lo[0], Gd.ics, Gd.G[0])) | (spread3(gcell(y, Gd.lo[1], Gd.ics, Gd.G[1])) << 1) |
           (spread3(gcell(z, Gd.lo[2], Gd.ics, Gd.G[2])) << 2);
  idx[i] = (int32_t)i;
}

// The sorted copy of the sites, and the runs of each level's cells.
__global__ void k_vor_bounds(int64_t n, const uint32_t *key, const double *g, VorGrid Gd, double *x, int32_t *start,
                             int32_t *end) {
  const int64_t k = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (k >= n) return;
  const int64_t i = Gd.id[k];
  x[3 * k] = g[3 * i];
  x[3 * k + 1] = g[3 * i + 1];
  x[3 * k + 2] = g[3 * i + 2];
  const uint32_t c = key[k];
  const uint32_t before = k > 0 ? key[k - 1] ^ c : ~0u, after = k < n - 1 ? key[k + 1] ^ c : ~0u;
  const uint32_t ix = gather3(c), iy = gather3(c >> 1), iz = gather3(c >> 2);
  for (int l = 0; l <= Gd.L; ++l) {
    const int sh = Gd.L - l;
    const int64_t gx_n = (Gd.G[0] + (1 << sh) - 1) >> sh, gy_n = (Gd.G[1] + (1 << sh) - 1) >> sh;
    const int64_t cell = Gd.off[l] + ((int64_t)(iz >> sh) * gy_n + (iy >> sh)) * gx_n + (ix >> sh);
    if (k == 0 || before >> (3 * sh)) start[cell] = (int32_t)k;
    if (k == n - 1 || after >> (3 * sh)) end[cell] = (int32_t)(k + 1);
  }
}

__global__ void k_vor_zero(int64_t m, int32_t *a, int32_t *b) {
  const int64_t k = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (k < m) {
    a[k] = 0;
    b[k] = 0;
  }
}

__global__ void k_vor_set(int64_t *a, int64_t va, int64_t *b, int64_t vb) {
  if (threadIdx.x == 0) {
    *a = va;
    *b = vb;
  }
}

void vor_check(Ctx &ctx, int *err, hipStream_t s) {
  int e = 0;
  SPH_HIP(hipMemcpyAsync(&e, err, sizeof(int), hipMemcpyDeviceToHost, s));
  SPH_HIP(hipStreamSynchronize(s));
  SPH_REQUIRE(!(e & kErrOutside), SPHMAP_EINVAL, "a generator lies outside the box");
  SPH_REQUIRE(!(e & kErrCoincident), SPHMAP_EINVAL, "two generators coincide");
  SPH_REQUIRE(!(e & kErrPlanes), SPHMAP_EGEOM, "a Voronoi cell has more than 58 neighbours");
  SPH_REQUIRE(!(e & kErrVertices), SPHMAP_EGEOM, "a Voronoi cell has more than 128 vertices");
  SPH_REQUIRE(!(e & kErrCycle), SPHMAP_EGEOM, "a Voronoi face did not close");
}

// the nested grids of the current generators
VorGrid vor_grid(Ctx &ctx, const double *g, int64_t n, const double lo[3], const double hi[3], int *err,
                 hipStream_t s) {
  Arena &ar = ctx.arena;
  VorGrid Gd;
  double size = 0.0;
  for (int a = 0; a < 3; ++a) {
    Gd.lo[a] = lo[a];
    Gd.hi[a] = hi[a];
    size = std::max(size, hi[a] - lo[a]);
  }
  // Cubic cells, the longest side split into 2^L, as fine as 256 bytes a
  // site hold (4 to 28 cells a site in a cube): a clump of a mixed set's
  // grid holds its sites in a 1e-3 of the box (35,000 sites: 2.0 ms a
  // construction with 28 bytes a site, 0.64 ms with 256; a log-normal cloud
  // gains nothing).  Under a workspace cap 28 bytes, which with the sorted
  // copy is what a call took before there were levels.
  auto cells_at = [&](int L, int l, int G[3]) {
    int64_t m = 1;
    for (int a = 0; a < 3; ++a) {
      const int fine = (int)std::min<double>(1 << L, std::max(1.0, ceil((hi[a] - lo[a]) / size * (1 << L))));
      G[a] = (fine + (1 << (L - l)) - 1) >> (L - l);
      m *= G[a];
    }
    return m;
  };
  int64_t cells = 1;
  Gd.L = 0;
  for (int L = 1; L < kVLevels; ++L) {
    int64_t m = 0;
    int G[3];
    for (int l = 0; l <= L; ++l) m += cells_at(L, l, G);
    if (8 * m > (ctx.ws.limit ? 28 : 256) * n) break;
    Gd.L = L;
    cells = m;
  }
  Gd.cs = size / (double)(1 << Gd.L);
  Gd.ics = 1.0 / Gd.cs;
  int64_t at = 0;
  for (int l = 0; l <= Gd.L; ++l) {
    Gd.off[l] = at;
    at += cells_at(Gd.L, l, Gd.G);
  }
  uint32_t *key = ar.get<uint32_t>("vo_key", n);
  int32_t *idx = ar.get<int32_t>("vo_idx", n);
  k_vor_keys<<<(unsigned)div_up(n, 256), 256, 0, s>>>(n, g, Gd, key, idx, err);
  SPH_LAUNCH_CHECK();
  if (Gd.L > 0) radix_sort_u32(ar, key, idx, n, 3 * Gd.L, s);
  int32_t *st = ar.get<int32_t>("vo_start", cells);
  int32_t *en = ar.get<int32_t>("vo_end", cells);
  double *x = ar.get<double>("vo_x", 3 * n);
  Gd.start = st;
  Gd.end = en;
  Gd.x = x;
  Gd.id = idx;
  k_vor_zero<<<(unsigned)div_up(cells, 256), 256, 0, s>>>(cells, st, en);
  SPH_LAUNCH_CHECK();
  k_vor_bounds<<<(unsigned)div_up(n, 256), 256, 0, s>>>(n, key, g, Gd, x, st, en);
  SPH_LAUNCH_CHECK();
  return Gd;
}

// the uniform grid of the final construction: about two generators a cell
RingGrid ring_grid(Ctx &ctx, const double *g, int64_t n, const double lo[3], const double hi[3], int *err,
                   hipStream_t s) {
  Arena &ar = ctx.arena;
  RingGrid Gd;
  double vol = 1.0;
  for (int a = 0; a < 3; ++a) {
    Gd.lo[a] = lo[a];
    Gd.hi[a] = hi[a];
    vol *= hi[a] - lo[a];
  }
  const double cs = cbrt(vol * 2.0 / (double)n);
  int64_t cells = 1;
  for (int a = 0; a < 3; ++a) {
    Gd.G[a] = (int)std::min<double>(1024.0, std::max(1.0, ceil((hi[a] - lo[a]) / cs)));
    Gd.cs[a] = (hi[a] - lo[a]) / Gd.G[a];
    cells *= Gd.G[a];
  }
  uint32_t *key = ar.get<uint32_t>("vo_key", n);
  int32_t *idx = ar.get<int32_t>("vo_idx", n);
  k_ring_keys<<<(unsigned)div_up(n, 256), 256, 0, s>>>(n, g, Gd, key, idx, err);
  SPH_LAUNCH_CHECK();
  int bits = 1;
  while (bits < 32 && ((int64_t)1 << bits) < cells) ++bits;
  radix_sort_u32(ar, key, idx, n, bits, s);
  int32_t *st = ar.get<int32_t>("vo_start", cells);
  int32_t *en = ar.get<int32_t>("vo_end", cells);
  double *x = ar.get<double>("vo_x", 3 * n);
  k_vor_zero<<<(unsigned)div_up(cells, 256), 256, 0, s>>>(cells, st, en);
  SPH_LAUNCH_CHECK();
  k_ring_bounds<<<(unsigned)div_up(n, 256), 256, 0, s>>>(n, key, g, idx, x, st, en);
  SPH_LAUNCH_CHECK();
  Gd.start = st;
  Gd.end = en;
  Gd.sorted = idx;
  Gd.x = x;
  Gd.gen = g;
  return Gd;
}

}  // namespace

void voronoi_build(Ctx &ctx, TessDev &t, int64_t n, const double *d_gen, const double lo[3], const double hi[3],
                   int n_lloyd, double *d_gen_out, hipStream_t s) {
  Arena &ar = ctx.arena;
  int *err = ar.get<int>("vo_err", 2);  // error bits; cells listed for the wide kernel
  SPH_HIP(hipMemsetAsync(err, 0, 2 * sizeof(int), s));
  double L = 0.0;
  for (int a = 0; a < 3; ++a) L = std::max(L, hi[a] - lo[a]);
  const double eps = 1e-13 * L;
  double *ga = ar.get<double>("vo_ga", 3 * n);
  double *gb = ar.get<double>("vo_gb", 3 * n);
  SPH_HIP(hipMemcpyAsync(ga, d_gen, 3 * n * sizeof(double), hipMemcpyDeviceToDevice, s));
  // a whole number of workgroups on each XCD
  const unsigned blocks = (unsigned)(8 * div_up(div_up(n, kVWaves), 8));
  for (int it = 0; it < n_lloyd; ++it) {
    VorGrid Gd = vor_grid(ctx, ga, n, lo, hi, err, s);
    KernelTimer kt(&ctx, "voronoi_lloyd", s);
    // the sort's keys are spent: the list of wide cells takes their place
    int32_t *wide = (int32_t *)ar.get<uint32_t>("vo_key", n);
    k_lloyd<<<blocks, 64 * kVWaves, 0, s>>>(Gd, n, eps, gb, err, wide, err + 1);
    SPH_LAUNCH_CHECK();
    k_lloyd_wide<<<256, 64, 0, s>>>(Gd, eps, gb, err, wide, err + 1);
    SPH_LAUNCH_CHECK();
    kt.done();
    vor_check(ctx, err, s);
    std::swap(ga, gb);
  }
  const RingGrid Gd = ring_grid(ctx, ga, n, lo, hi, err, s);
  int64_t *cf = ar.get<int64_t>("vo_cf", n + 1), *cp = ar.get<int64_t>("vo_cp", n + 1),
          *cv = ar.get<int64_t>("vo_cv", n + 1);
  int64_t *sf = ar.get<int64_t>("vo_sf", n + 1), *sp = ar.get<int64_t>("vo_sp", n + 1),
          *sv = ar.get<int64_t>("vo_sv", n + 1);
  // finished cells are kept from the count to the final arrays, but not under
  // a workspace cap (1.2 KB a cell, where a call takes 156 bytes without):
  // 3.1 ms less of a 131,071-cell grid's 6.2
  VorKept *kept = ctx.ws.limit ? nullptr : ar.get<VorKept>("vo_kept", n);
  int32_t *list = kept ? (int32_t *)ar.get<uint32_t>("vo_key", n) : nullptr;  // the sort's keys are spent
  {
    KernelTimer kt(&ctx, "voronoi_count", s);
    k_voronoi<1><<<blocks, 64 * kVWaves, 0, s>>>(Gd, n, eps, cf, cp, cv, kept, list, err + 1, nullptr, nullptr, nullptr,
                                                 nullptr, nullptr, err);
    SPH_LAUNCH_CHECK();
    kt.done();
  }
  vor_check(ctx, err, s);
  scan_exclusive_i64(ar, cf, sf, n, true, s);
  scan_exclusive_i64(ar, cp, sp, n, true, s);
  scan_exclusive_i64(ar, cv, sv, n, true, s);
  int64_t tot[3];
  SPH_HIP(hipMemcpyAsync(&tot[0], sf + n, sizeof(int64_t), hipMemcpyDeviceToHost, s));
  SPH_HIP(hipMemcpyAsync(&tot[1], sp + n, sizeof(int64_t), hipMemcpyDeviceToHost, s));
  SPH_HIP(hipMemcpyAsync(&tot[2], sv + n, sizeof(int64_t), hipMemcpyDeviceToHost, s));
  SPH_HIP(hipStreamSynchronize(s));
  const int64_t F = tot[0], FV = tot[1], V = tot[2];
  SPH_REQUIRE(F < ((int64_t)1 << 31) && FV < ((int64_t)1 << 31) && V < ((int64_t)1 << 31), SPHMAP_EINVAL,
              "grid too large");
  t.n_cells = n;
  t.n_faces = F;
  t.n_vertices = V;
  t.n_fv = FV;
  t.device = ctx.device;
  double size = 0.0;
  for (int a = 0; a < 3; ++a) {
    t.box_lo[a] = lo[a];
    size = std::max(size, hi[a] - lo[a]);
  }
  t.box_size = size * (1.0 + 1e-12);
  t.gen = t.mem.get<double>("gen", 3 * n);
  t.vert = t.mem.get<double>("vert", 3 * std::max<int64_t>(V, 1));
  t.cell_face_off = t.mem.get<int64_t>("cfo", n + 1);
  t.face_vtx_off = t.mem.get<int64_t>("fvo", F + 1);
  t.face_vtx = t.mem.get<int32_t>("fv", std::max<int64_t>(FV, 1));
  t.face_nbr = t.mem.get<int32_t>("fnbr", std::max<int64_t>(F, 1));
  {
    KernelTimer kt(&ctx, "voronoi_faces", s);
    if (kept) {
      k_vor_place<<<(unsigned)div_up(n, 4), 256, 0, s>>>(n, cf, cp, cv, sf, sp, sv, kept, t.vert, t.cell_face_off,
                                                         t.face_vtx_off, t.face_vtx, t.face_nbr);
      SPH_LAUNCH_CHECK();
    }
    k_voronoi<2><<<kept ? std::min(blocks, 1024u) : blocks, 64 * kVWaves, 0, s>>>(
        Gd, n, eps, sf, sp, sv, nullptr, list, err + 1, t.vert, t.cell_face_off, t.face_vtx_off, t.face_vtx,
        t.face_nbr, err);
    SPH_LAUNCH_CHECK();
    kt.done();
  }
  k_vor_set<<<1, 64, 0, s>>>(t.cell_face_off + n, F, t.face_vtx_off + F, FV);
  SPH_LAUNCH_CHECK();
  SPH_HIP(hipMemcpyAsync(t.gen, ga, 3 * n * sizeof(double), hipMemcpyDeviceToDevice, s));
  if (d_gen_out) SPH_HIP(hipMemcpyAsync(d_gen_out, ga, 3 * n * sizeof(double), hipMemcpyDeviceToDevice, s));
  vor_check(ctx, err, s);
  tess_prepare(ctx, t, s);
}

}  // namespace sphmap
