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
// (With the vertices compacted and T rebuilt after each cut, and shuffles
// for the scans and sums, 131,071 turbulent sites took 5.95 ms a
// construction; now 2.4 ms, about 8,400 wave instructions a cell at 0.61
// lane utilisation, most of them vector issue, of 64 lanes for about 25
// vertices.)
//
// Neighbours are found in a fixed order: a uniform grid of about two
// generators a cell, searched in rings of growing Chebyshev radius; the 64
// nearest sites of rings 0 and 1 first, then every site 64 at a time as the
// grid lists them, each batch nearest first.  A generator at distance D can
// cut only when D/2 does not exceed the largest vertex distance R of the
// current cell, so the search stops once the next ring lies beyond 2R (the
// security radius).  The order is kept because its results show: the final
// grid's faces and vertices are numbered by the cuts (sphmap_tess_export),
// the mixed path's rounding follows that numbering, and a site that moves by
// its last bit changes which of the mixed path's thresholds its faces meet
// (up to 1e-7 of a cell's mass).  Nested grids of Morton runs took the sites
// of a Lloyd iteration nearest first, 1.4 to 1.9 ms each instead of 2.6, but
// left sites that differ by an ulp; Lloyd iterations therefore share the fixed
// order, and add a cell's tetrahedra in the order of its vertices' numbers.
// Vertices carry their age (the cut that made them, and their place in it),
// so that slots reused in any order still give the numbering of a list that
// only closes up and grows.
//
// Outputs: centroids (Lloyd iterations); face, face vertex and vertex counts;
// the faces themselves (each face's vertex cycle walked through T) with the
// neighbour each one faces.
#include "common.hpp"

namespace sphmap {
namespace {

constexpr int kVP = 64;     // planes per cell: 6 box planes + neighbours
constexpr int kVT = 128;    // vertices per cell
// Cells per workgroup.  One, so that the room of a cell that is done goes to
// the next at once, whatever its neighbours still cut (131,071 sites with 5
// iterations: 19.6 ms with four, 19.2 with two, 18.1 with one).
constexpr int kVWaves = 1;
// Of the 64 nearest sites about 22 cut; the others cost a dependent step
// each.  After this many the rest are tested at once, one a lane (131,071
// sites with 5 iterations: 17.2 ms without, 16.9 at 12 or 16, 17.2 at 24).
constexpr int kVAhead = 12;
constexpr int kVRing = 128;  // sites in a group beyond which its grid cells are tested before them

// error bits
constexpr int kErrCoincident = 1;
constexpr int kErrPlanes = 2;
constexpr int kErrVertices = 4;
constexpr int kErrCycle = 8;
constexpr int kErrOutside = 16;

struct VorLds {  // 10,176 bytes: 16 workgroups of one wavefront a CU
  static constexpr int kP = kVP, kT = kVT;
  uint8_t T[kP][kP];              // vertex holding directed edge a -> b
  double vx[kT], vy[kT], vz[kT];  // vertex positions about the generator
  int32_t pid[kP];                // the neighbouring generator, or -1..-6 for box planes
  union {
    int32_t list[64];    // positions in the sorted order of the sites of one batch
    uint2 fresh[kP];   // the vertices a cut makes: planes; removed and kept end of the edge they lie on
    struct {             // at the end: the planes of each vertex, its number, a vertex on each plane
      uint32_t tri[kT];
      uint32_t first[kP];
      uint8_t rank[kT], slot[kT];
    } out;
    struct {             // or: unit normal and offset of each plane, and as above
      double n[kP][4];
      uint32_t tri[kT];
      uint8_t slot[kT];
    } cen;
  };
  uint8_t map[kP];
};

// One cell, spread over a wavefront: vertex lane + 64 h in x[h], y[h], z[h],
// tri[h] (planes a, b, c in bytes 0-2; a free slot has position 0, which no
// bisector cuts); uniform: the live vertex slots, the plane count, and a bound
// of the largest vertex distance.
struct VorCell {
  static constexpr int kH = 2;
  double x[kH], y[kH], z[kH];
  uint32_t tri[kH];
  uint32_t age[kH];  // cuts made before it, and its place among its cut's (8 bits)
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
__device__ inline double readlane_d(double v, int j) {
  return __hiloint2double(__builtin_amdgcn_readlane(__double2hiint(v), j),
                          __builtin_amdgcn_readlane(__double2loint(v), j));
}
// (a tree whose order Lloyd's sites are held to)
__device__ inline double vsumd(double v) {
#pragma unroll
  for (int o = 32; o > 0; o >>= 1) v += __shfl_xor(v, o, 64);
  return v;
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

__device__ inline void vput(VorLds &L, const VorCell &C, int h, int t) {
  L.vx[t] = C.x[h];
  L.vy[t] = C.y[h];
  L.vz[t] = C.z[h];
}
__device__ inline void vlink(VorLds &L, uint32_t tri, int t) {
  const int a = tri & 0xff, b = (tri >> 8) & 0xff, c = (tri >> 16) & 0xff;
  L.T[a][b] = (uint8_t)t;
  L.T[b][c] = (uint8_t)t;
  L.T[c][a] = (uint8_t)t;
}
// With room for the binary32 order of the sites: a bisector beyond R cuts
// nothing, and nor does any after it, whose binary32 distance may be equal and
// whose distance then up to 1.2e-7 smaller.
constexpr double kVSlack = 1.0 + 2e-7;
__device__ inline void vradius(VorCell &C) {
  double r2 = C.x[0] * C.x[0] + C.y[0] * C.y[0] + C.z[0] * C.z[0];
#pragma unroll
  for (int h = 1; h < C.kH; ++h)
    if (C.live[h]) r2 = fmax(r2, C.x[h] * C.x[h] + C.y[h] * C.y[h] + C.z[h] * C.z[h]);
  C.R = sqrt(vmaxd(r2)) * kVSlack;
}

// Drop the planes no vertex lies on any more and renumber the rest.
__device__ void vcompact(VorLds &L, VorCell &C, int lane) {
  L.map[lane] = 0;
  vsync();
#pragma unroll
  for (int h = 0; h < C.kH; ++h)
    if ((C.live[h] >> lane) & 1ull) {
      L.map[C.tri[h] & 0xff] = 1;
      L.map[(C.tri[h] >> 8) & 0xff] = 1;
      L.map[(C.tri[h] >> 16) & 0xff] = 1;
    }
  vsync();
  const bool used = lane < C.nP && L.map[lane];
  const uint64_t um = ballot64(used);
  const int to = vrank(um);
  const int32_t id = L.pid[lane];
  vsync();
  if (used) {  // a plane moves down, past planes already read
    L.map[lane] = (uint8_t)to;
    L.pid[to] = id;
  }
  vsync();
  C.nP = __popcll(um);
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
__device__ bool vcut(VorLds &L, VorCell &C, double nx, double ny, double nz, double d, int32_t id, double eps,
                     int lane, int &err) {
  constexpr int kH = VorCell::kH;
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
  uint32_t mine[kH] = {}, twin[kH] = {};  // which edges cross, and the twins
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
      total += __popcll(ballot64(nv));
      mine[h] |= (uint32_t)nv << r;
      twin[h] |= (uint32_t)t2 << (8 * r);
    }
  }
  if (total > room || total > L.kP) {
    err = kErrVertices;
    return false;
  }
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
  vsync();
  // free slots take the new vertices in turn; a removed vertex whose slot
  // stays free moves to the generator, which no plane cuts
  bool take[kH];
  int free_before = 0;  // free slots of the halves before
#pragma unroll
  for (int h = 0; h < kH; ++h) {
    take[h] = false;
    const uint64_t fr = ~kept[h];
    const int k = free_before + vrank(fr);
    if (h == 0 || C.live[h] || total > free_before) {  // uniform
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
        C.age[h] = ((uint32_t)(C.cuts + 1) << 8) | (uint32_t)k;
      } else if ((m[h] >> lane) & 1ull) {
        C.x[h] = C.y[h] = C.z[h] = 0.0;
      }
    }
    free_before += __popcll(fr);
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

// The slots that vertices have taken so far.
__device__ inline int vslots(const VorCell &C) {
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

// Whether the plane n.x <= d (a lane's) cuts any vertex.
__device__ inline bool vcuts(const VorLds &L, const VorCell &C, double nx, double ny, double nz, double d, double eps) {
  bool cuts = false;
  const int nT = vslots(C);
#pragma unroll 2
  for (int t = 0; t < nT; ++t) cuts |= nx * L.vx[t] + ny * L.vy[t] + nz * L.vz[t] - d > eps;
  return cuts;
}

// Cut by the bisectors of one batch of candidates (lane: the vector to the
// site, its distance and its index), nearest first.  The planes are first
// tested against every vertex, one candidate per lane, so that the many sites
// that no longer cut cost no serial step (a plane that cuts no vertex cuts none
// of a smaller cell's).  Returns false on an error (bit in err).
__device__ bool vbatch(VorLds &L, VorCell &C, bool cand, double ex, double ey, double ez, double dist,
                       int32_t id, double eps, int lane, int &err) {
  uint64_t cm = ballot64(cand);
  if (!cm) return true;
  if (ballot64(cand && !(dist > 0.0))) {
    err = kErrCoincident;
    return false;
  }
  const double nx = ex / dist, ny = ey / dist, nz = ez / dist;
  const double dd = 0.5 * dist;
  cand = vcuts(L, C, nx, ny, nz, dd, eps) && cand;
  cm = ballot64(cand);
  if (!cm) return true;
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

// Whether the box of half sizes (hx, hy, hz) about (mx, my, mz) meets the ball
// about some vertex through the generator: a site outside those balls is
// nearer to no vertex than the generator, and cuts nothing.
__device__ inline bool vballs(const VorLds &L, const VorCell &C, double mx, double my, double mz, double hx,
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

// The box about a site: planes x-, x+, y-, y+, z-, z+ and its eight corners.
__device__ inline void vbox(VorLds &L, VorCell &C, const double (&lo)[3], const double (&hi)[3], double gx,
                            double gy, double gz, int lane) {
#pragma unroll
  for (int h = 0; h < C.kH; ++h) {
    C.x[h] = C.y[h] = C.z[h] = 0.0;
    C.tri[h] = 0;
    C.live[h] = 0ull;
    C.age[h] = (uint32_t)lane;
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

// workgroups go to the eight XCDs in turn: each XCD takes a contiguous
// eighth of the sorted sites, whose neighbourhoods meet in its L2 (the grid
// is a multiple of eight workgroups)
__device__ inline int64_t xcd_cell(int w) {
  const int64_t per = gridDim.x / 8, b = blockIdx.x;
  return ((b & 7) * per + (b >> 3)) * kVWaves + w;
}

// ------------------------------------------------------- cells in the fixed order
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

// A site's distance and key: the binary32 distance, then the index.  Each in
// one place and in stated operations, so that a site's key is the same
// wherever it is formed.
__device__ __forceinline__ double vdist(double ex, double ey, double ez) {
  return sqrt(fma(ez, ez, fma(ex, ex, ey * ey)));
}
__device__ __forceinline__ uint64_t vkey(double dist, int32_t j) {
  return ((uint64_t)__float_as_uint((float)dist) << 32) | (uint32_t)j;
}

// Sites w0 .. w0 + 63 of a group of grid cells (lane: sites s0 .. s0 + cnt of
// the sorted array at offset off of the group's tot sites): this lane's, or -1.
__device__ inline int vwindow(VorLds &L, int s0, int cnt, int off, int tot, int w0, int lane) {
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
__device__ bool vgroup(VorLds &L, VorCell &C, const RingGrid &Gd, int32_t c, double gx, double gy,
                       double gz, int s0, int cnt, double mx, double my, double mz, double near2, bool nearest,
                       double eps, int lane, int &err) {
  const int off = vscan_excl(cnt);
  const int tot = __builtin_amdgcn_readlane(off + cnt, 63);
  uint64_t best = ~0ull;
  if (nearest) {
    // the home cell (lane 13 of the 27) first, for a tight bound
    const int home0 = __builtin_amdgcn_readlane(off, 13), home1 = home0 + __builtin_amdgcn_readlane(cnt, 13);
    for (int turn = 0; turn < 2; ++turn)
      for (int w0 = 0; w0 < tot; w0 += 64) {
        const bool home = w0 < home1 && w0 + 64 > home0;
        if (home != (turn == 0)) continue;
        const uint64_t last = (uint64_t)(uint32_t)__builtin_amdgcn_readlane((int)(uint32_t)best, 63) |
                              ((uint64_t)(uint32_t)__builtin_amdgcn_readlane((int)(uint32_t)(best >> 32), 63) << 32);
        if (last != ~0ull) {
          // (the cells' walls are rounded, by less than eps)
          const double far = (double)__uint_as_float((uint32_t)(last >> 32)) * (1.0 + 1e-6) + eps;
          if (!ballot64(off < w0 + 64 && off + cnt > w0 && near2 <= far * far)) continue;
        }
        const int k = vwindow(L, s0, cnt, off, tot, w0, lane);
        uint64_t key = ~0ull;
        if (k >= 0) {
          const double ex = Gd.x[3 * (int64_t)k] - gx, ey = Gd.x[3 * (int64_t)k + 1] - gy,
                       ez = Gd.x[3 * (int64_t)k + 2] - gz;
          const int32_t j = Gd.sorted[k];
          if (j != c) key = vkey(vdist(ex, ey, ez), j);
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
      dist = vdist(ex, ey, ez);
    }
    if (ballot64(some && !(dist > 0.0))) {
      err = kErrCoincident;
      return false;
    }
    const double nx = ex / dist, ny = ey / dist, nz = ez / dist, dd = 0.5 * dist;
    uint64_t todo = ballot64(some);
    for (int at = 0; todo; todo &= todo - 1, ++at) {
      if (at == kVAhead) {  // the rest at once: a plane that cuts no vertex cuts none of a smaller cell's
        todo &= ballot64(vcuts(L, C, nx, ny, nz, dd, eps));
        if (!todo) break;
      }
      const int l = __builtin_ctzll(todo);
      const double dl = readlane_d(dd, l);
      if (dl > C.R + eps) break;
      if (!vcut(L, C, readlane_d(nx, l), readlane_d(ny, l), readlane_d(nz, l), dl, __builtin_amdgcn_readlane(j, l),
                eps, lane, err))
        return false;
    }
  }
  // the nearest are done with: what they left cuts nothing a second time
  // (tested again with the others: 18.1 ms in place of 17.2)
  uint64_t upto = 0ull;
  if (nearest) {
    if (tot <= 64) return true;
    upto = (uint64_t)(uint32_t)__builtin_amdgcn_readlane((int)(uint32_t)best, 63) |
           ((uint64_t)(uint32_t)__builtin_amdgcn_readlane((int)(uint32_t)(best >> 32), 63) << 32);
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
      dist = vdist(ex, ey, ez);
      cand = 0.5 * dist <= C.R + eps;
      if (cand) {
        j = Gd.sorted[k];
        cand = j != c && vkey(dist, j) > upto;
      }
    }
    if (!vbatch(L, C, cand, ex, ey, ez, dist, j, eps, lane, err)) return false;
    vsync();
  }
  return true;
}

// The cell of generator c, in the fixed order.
__device__ bool ring_cell(VorLds &L, VorCell &C, const RingGrid &Gd, int32_t c, double gx, double gy,
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

// Each vertex's number: its place by age.
__device__ inline void vplaces(const VorCell &C, int (&place)[2]) {
  place[0] = place[1] = 0;
#pragma unroll
  for (int h = 0; h < 2; ++h)
    for (uint64_t m = C.live[h]; m; m &= m - 1) {
      const uint32_t al = (uint32_t)__builtin_amdgcn_readlane((int)C.age[h], __builtin_ctzll(m));
      place[0] += al < C.age[0] ? 1 : 0;
      place[1] += al < C.age[1] ? 1 : 0;
    }
}

// The centroid of the cell of sorted site i.
__device__ void ring_centroid(VorLds &L, const RingGrid &Gd, int64_t i, double eps, double *centroid, int *err,
                              int lane) {
  const int32_t c = Gd.sorted[i];
  const double gx = Gd.x[3 * i], gy = Gd.x[3 * i + 1], gz = Gd.x[3 * i + 2];
  VorCell C;
  {
    int e = 0;
    if (!ring_cell(L, C, Gd, c, gx, gy, gz, eps, lane, e)) {
      if (lane == 0) atomicOr(err, e);
      return;
    }
  }
  int place[2];
  vplaces(C, place);
  const int nT = __popcll(C.live[0]) + __popcll(C.live[1]);
  vsync();
#pragma unroll
  for (int h = 0; h < 2; ++h)
    if ((C.live[h] >> lane) & 1ull) {
      L.cen.tri[lane + 64 * h] = C.tri[h];
      L.cen.slot[place[h]] = (uint8_t)(lane + 64 * h);
    }
  if (lane < C.nP) {
    const int64_t q = L.pid[lane];
    double n[4];
    if (q >= 0) {
      const double ex = Gd.gen[3 * q] - gx, ey = Gd.gen[3 * q + 1] - gy, ez = Gd.gen[3 * q + 2] - gz;
      const double dist = sqrt(ex * ex + ey * ey + ez * ez);
      n[0] = ex / dist;
      n[1] = ey / dist;
      n[2] = ez / dist;
      n[3] = 0.5 * dist;
    } else {
      const int ax = (int)(-1 - q) >> 1;
      const bool up = (-1 - q) & 1;
      const double g = ax == 0 ? gx : (ax == 1 ? gy : gz);
      const double wl = ax == 0 ? Gd.lo[0] : (ax == 1 ? Gd.lo[1] : Gd.lo[2]);
      const double wh = ax == 0 ? Gd.hi[0] : (ax == 1 ? Gd.hi[1] : Gd.hi[2]);
      n[0] = ax == 0 ? (up ? 1.0 : -1.0) : 0.0;
      n[1] = ax == 1 ? (up ? 1.0 : -1.0) : 0.0;
      n[2] = ax == 2 ? (up ? 1.0 : -1.0) : 0.0;
      n[3] = up ? wh - g : g - wl;
    }
#pragma unroll
    for (int a = 0; a < 4; ++a) L.cen.n[lane][a] = n[a];
  }
  vsync();
  // over every directed cell edge on face x, the tetrahedron (g, foot of g
  // on x, edge start, edge end); lane l adds vertices l and l + 64
  double V = 0.0, Sx = 0.0, Sy = 0.0, Sz = 0.0;
#pragma unroll
  for (int h = 0; h < 2; ++h) {
    const int t = lane + 64 * h;
    if (t < nT) {
      const int s = L.cen.slot[t];
      const uint32_t tr = L.cen.tri[s];
      const int a = tr & 0xff, b = (tr >> 8) & 0xff, cc = (tr >> 16) & 0xff;
      const double px = L.vx[s], py = L.vy[s], pz = L.vz[s];
#pragma unroll
      for (int r = 0; r < 3; ++r) {
        const int x = r == 0 ? a : (r == 1 ? b : cc);
        const int z = r == 0 ? cc : (r == 1 ? a : b);
        const int t2 = L.T[x][z] & (kVT - 1);
        const double qd = L.cen.n[x][3];
        const double fx = qd * L.cen.n[x][0], fy = qd * L.cen.n[x][1], fz = qd * L.cen.n[x][2];
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
    centroid[3 * (int64_t)c] = gx + Sx / V;
    centroid[3 * (int64_t)c + 1] = gy + Sy / V;
    centroid[3 * (int64_t)c + 2] = gz + Sz / V;
  }
}

__global__ void __launch_bounds__(64 * kVWaves, 4) k_lloyd(RingGrid Gd, int64_t n, double eps, double *centroid,
                                                           int *err) {
  __shared__ VorLds S[kVWaves];
  const int w = threadIdx.x >> 6, lane = threadIdx.x & 63;
  const int64_t i = xcd_cell(w);
  if (i >= n) return;
  ring_centroid(S[w], Gd, i, eps, centroid, err, lane);
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
__device__ void ring_build(VorLds &L, const RingGrid &Gd, int64_t i, double eps, int64_t *cnt_f, int64_t *cnt_p,
                           int64_t *cnt_v, VorKept *kept, int32_t *list, int32_t *list_n, double *vert,
                           int64_t *cell_face_off, int64_t *face_vtx_off, int32_t *face_vtx, int32_t *face_nbr,
                           int *err, int lane) {
  const int32_t c = Gd.sorted[i];
  const double gx = Gd.x[3 * i], gy = Gd.x[3 * i + 1], gz = Gd.x[3 * i + 2];
  VorCell C;
  {
    int e = 0;
    if (!ring_cell(L, C, Gd, c, gx, gy, gz, eps, lane, e)) {
      if (lane == 0) atomicOr(err, e);
      return;
    }
  }
  const int nT = __popcll(C.live[0]) + __popcll(C.live[1]);
  int place[2];
  vplaces(C, place);
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
  __shared__ VorLds S[kVWaves];
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

// the uniform grid of the current generators: about two a cell
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
  int *err = ar.get<int>("vo_err", 2);  // error bits; cells listed by the count
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
    const RingGrid Gd = ring_grid(ctx, ga, n, lo, hi, err, s);
    KernelTimer kt(&ctx, "voronoi_lloyd", s);
    k_lloyd<<<blocks, 64 * kVWaves, 0, s>>>(Gd, n, eps, gb, err);
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
  // Finished cells are kept from the count to the final arrays: 3.1 ms less of
  // a 131,071-cell grid's 6.2.  They take 1.2 KB a cell where a call takes 156
  // bytes without, in a block of the context's pool that goes back to it here;
  // under a workspace cap, and where memory is short, every cell is built again.
  Arena keep;
  keep.pool = &ctx.pool;
  keep.close = true;
  VorKept *kept = ctx.ws.limit ? nullptr : keep.get_if<VorKept>("vo_kept", n);
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
  const auto arrays = [&] {
    t.gen = t.mem.get<double>("gen", 3 * n);
    t.vert = t.mem.get<double>("vert", 3 * std::max<int64_t>(V, 1));
    t.cell_face_off = t.mem.get<int64_t>("cfo", n + 1);
    t.face_vtx_off = t.mem.get<int64_t>("fvo", F + 1);
    t.face_vtx = t.mem.get<int32_t>("fv", std::max<int64_t>(FV, 1));
    t.face_nbr = t.mem.get<int32_t>("fnbr", std::max<int64_t>(F, 1));
  };
  try {
    arrays();
  } catch (const Error &e) {
    if (e.code != SPHMAP_ENOMEM || !kept) throw;
    keep.pool = nullptr;  // the kept cells' memory goes back to the device
    keep.release();
    kept = nullptr;
    list = nullptr;
    arrays();
  }
  {
    KernelTimer kt(&ctx, "voronoi_faces", s);
    if (kept) {
      k_vor_place<<<(unsigned)div_up(n, 4), 256, 0, s>>>(n, cf, cp, cv, sf, sp, sv, kept, t.vert, t.cell_face_off,
                                                         t.face_vtx_off, t.face_vtx, t.face_nbr);
      SPH_LAUNCH_CHECK();
    }
    // as many waves as the chip holds (the listed cells of the grids of a mixed
    // set of 167,000 and its 1,048,576 particles: 2.4 ms a grid, 3.4 with 1,024)
    k_voronoi<2><<<kept ? std::min(blocks, 4096u) : blocks, 64 * kVWaves, 0, s>>>(
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
  keep.release(true);  // s was waited for
  tess_prepare(ctx, t, s);
}

}  // namespace sphmap
