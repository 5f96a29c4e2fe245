// Per-particle values from the mixed set of real particles and pseudo-
// particles (Sec. 3.3: rather than giving every member of a pseudo-particle
// its node's value, each SPH particle is interpolated from the entries whose
// smoothing spheres reach it).
//
//   q_i = sum_j V_j W(r_ij, h_j) q_j / sum_j V_j W(r_ij, h_j)
//       = sum_j w(r_ij / h_j) q_j / sum_j w(r_ij / h_j)
//
// the Shepard-normalised SPH interpolant over the entries j with
// r_ij = |x_i - x_j| < 2 h_j, each entry standing for the volume
// V_j = (h_j / h_fact)^3 of the h-density relation (eq. h_node), so that
// only the dimensionless M4 kernel w remains.  A particle that is an entry
// itself keeps that entry's value; a particle no sphere reaches keeps its
// owner's value.
//
// Gather, not scatter: the entries are Morton-sorted under the ball
// hierarchy of the pair search, and every sum is formed by one lane over the
// entries in Morton order (no atomics; results repeat bit for bit, whatever
// particles share a walk).  Particles are taken in Morton order, so that the
// 64 of a wavefront lie close together and walk the hierarchy as one.
// Candidates pass a binary32 sphere test with the hierarchy's slack before
// the binary64 distance decides.
#include <mutex>

#include "ballsearch.hpp"

namespace sphmap {
namespace {

constexpr int kCompPass = 4;  // components accumulated per walk

__device__ inline double m4w(double q) {
#pragma clang fp contract(off)
  const double in = 1.0 - 1.5 * q * q + 0.75 * q * q * q, out = 0.25 * (2.0 - q) * (2.0 - q) * (2.0 - q);
  return q < 1.0 ? in : q < 2.0 ? out : 0.0;
}

__global__ void k_interp_check(int64_t n, const double *xyz, const int64_t *owner, int64_t ne, const double *exyz,
                               int *bad) {
  const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i < n) {
    const double *p = xyz + 3 * i;
    const bool in = p[0] >= 0.0 && p[0] < 1.0 && p[1] >= 0.0 && p[1] < 1.0 && p[2] >= 0.0 && p[2] < 1.0;
    if (!in) atomicOr(bad, 1);
    if (!(owner[i] >= 0 && owner[i] < ne)) atomicOr(bad, 2);
  }
  if (i < ne) {
    const double *p = exyz + 3 * i;
    const bool in = p[0] >= 0.0 && p[0] < 1.0 && p[1] >= 0.0 && p[1] < 1.0 && p[2] >= 0.0 && p[2] < 1.0;
    if (!in) atomicOr(bad, 4);
  }
}

__global__ void k_entry_prep(int64_t ne, const int32_t *sidx, const double *exyz, const double *eh, float4 *sx,
                             double4 *sd) {
  const int64_t k = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (k >= ne) return;
  const int64_t j = sidx[k];
  const double x = exyz[3 * j], y = exyz[3 * j + 1], z = exyz[3 * j + 2], h = eh[j];
  sx[k] = make_float4((float)x, (float)y, (float)z, (float)h);
  sd[k] = make_double4(x, y, z, h);
}

// Particles in Morton order, 8 bits an axis of [0,1): three digits of the
// sort.  All 10 bits (a fourth digit) cost more than closer wavefronts gave:
// 0.557 against 0.545 ms for 1,048,576 particles, 0.412 against 0.392 ms for
// 100,000 (MI355X).  Sending the particles that are entries themselves to the
// end brought far ones together in a wavefront: 0.68 ms.
constexpr int kPlaceBits = 24;
__device__ inline uint32_t spread10(double x) {  // bit b of the cell number at bit 3 b
  const uint32_t v = min((uint32_t)(x * 1024.0), 1023u);
  uint32_t r = 0;
#pragma unroll
  for (int b = 0; b < 10; ++b) r |= (v >> b & 1u) << (3 * b);
  return r;
}
__global__ void k_place_keys(int64_t n, const double *xyz, uint32_t *key, int32_t *idx) {
  const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= n) return;
  key[i] = (spread10(xyz[3 * i]) | spread10(xyz[3 * i + 1]) << 1 | spread10(xyz[3 * i + 2]) << 2) >> (30 - kPlaceBits);
  idx[i] = (int32_t)i;
}

__device__ __forceinline__ void wave_order() {  // orders a wave's LDS writes before its reads
  __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
  __builtin_amdgcn_wave_barrier();
  __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

__device__ __forceinline__ float readlane_f(float v, int k) {
  return __int_as_float(__builtin_amdgcn_readlane(__float_as_int(v), k));
}

// Wavefronts to which few particles are spread, a power of two each.  The fewer
// particles, the farther apart the 64 of a wavefront: its last walk then goes
// through most of the set.  64, 1,024 and 8,192 scattered particles of 84,000 to
// 93,000 entries took 0.95 to 2.2, 1.1 to 2.2 and 1.6 ms with 64 a wavefront
// (0.4 to 1.0, 0.8 to 1.4 and 1.3 to 1.5 with a walk a particle); now 0.2, 0.23
// and 0.31 (MI355X; 2,048 and 8,192 wavefronts are up to a third slower at
// 65,536 and at 100,000 particles).
constexpr int kInterpWaves = 4096;
constexpr int kTurn = 2;    // balls a lane sums at a time
constexpr int kGroups = 4;  // walks of a wave: the last takes all that is left
template <int kNc>
struct InterpWave {
  double4 ball[64];                 // x, y, z and a bound of 4 h^2
  double h[64];
  double val[64][kNc];
  int32_t list[128];                // candidates, ascending
  int32_t node[64];                 // groups of balls to look into
  uint32_t st[64 * kMaxLevels];     // node << 4 | level (a level-1 node index is below 2^27); 64 pushed a level
};

// One wavefront per `per` particles (64, fewer where that leaves less than
// kInterpWaves wavefronts), components [c0, c0 + kNc) of ncomp.  The particles
// around the first one left (within 2 h of its entry) share a walk: the boxes
// of four nodes, or 64 balls, at a time are tested against the group's box,
// boxes of balls also against its particles.  The balls that are left are
// gathered in LDS, 64 at a time; each lane marks those that reach its own
// particle and sums them.  The stack keeps boxes in ascending order,
// so each sum runs over the balls r < 2 h in Morton order.
// One thread a particle, with a walk and scattered loads of its own, took
// 1.6 ms of 2.02 ms for 1,048,576 particles in three components, this takes
// 0.33 of 0.52 ms (MI355X): bounded by instructions, about 100 binary64 ones
// for each ball that reaches a particle and as many for the walk, and for the
// last third by the wavefronts around few particles of many small entries.
template <int kNc>  // components of this pass
__global__ void __launch_bounds__(64) k_interp(Hier H, const double4 *sd, int64_t n, int per, const int32_t *qidx,
                                               const double *xyz, const int64_t *owner, const double *eh,
                                               const int32_t *ekind, const double *val, int ncomp, int c0, double *out,
                                               int *status) {
#pragma clang fp contract(off)
  __shared__ InterpWave<kNc> S;
  const int lane = threadIdx.x;
  const int64_t t = (int64_t)blockIdx.x * per + threadIdx.x;
  int64_t i = 0, o = 0;
  double px = 0.0, py = 0.0, pz = 0.0;
  bool left = lane < per && t < n;
  int bad = 0;
  if (left) {
    i = qidx[t];
    o = owner[i];
    if (ekind[o] == 0) {
      for (int k = 0; k < kNc; ++k) {
        const double v = val[(int64_t)ncomp * o + c0 + k];
        out[(int64_t)ncomp * i + c0 + k] = v;
        if (!isfinite(v)) bad = SPHMAP_STATUS_NONFINITE_VALUE;
      }
      left = false;
    } else {
      px = xyz[3 * i];
      py = xyz[3 * i + 1];
      pz = xyz[3 * i + 2];
    }
  }
  const uint64_t below = lane == 0 ? 0ull : (~0ull >> (64 - lane));
  const float r2box = H.margin_abs * H.margin_abs;
  const int top = H.levels;
  uint64_t rest = __ballot(left);
  for (int g = 0; rest; ++g) {
    const int lead = __builtin_ctzll(rest);
    bool mine = left && (rest >> lane & 1ull);
    if (g + 1 < kGroups) {
      const double r = 2.0 * __shfl(left ? eh[o] : 0.0, lead, 64);
      const double dx = px - __shfl(px, lead, 64), dy = py - __shfl(py, lead, 64), dz = pz - __shfl(pz, lead, 64);
      mine = mine && (lane == lead || fmax(fmax(fabs(dx), fabs(dy)), fabs(dz)) <= r);
    }
    rest &= ~__ballot(mine);
    // the group's box
    float lx = mine ? (float)px : 2.0f, ly = mine ? (float)py : 2.0f, lz = mine ? (float)pz : 2.0f;
    float hx = mine ? (float)px : -1.0f, hy = mine ? (float)py : -1.0f, hz = mine ? (float)pz : -1.0f;
#pragma unroll
    for (int d = 32; d > 0; d >>= 1) {
      lx = fminf(lx, __shfl_xor(lx, d, 64));
      ly = fminf(ly, __shfl_xor(ly, d, 64));
      lz = fminf(lz, __shfl_xor(lz, d, 64));
      hx = fmaxf(hx, __shfl_xor(hx, d, 64));
      hy = fmaxf(hy, __shfl_xor(hy, d, 64));
      hz = fmaxf(hz, __shfl_xor(hz, d, 64));
    }
    auto gap2 = [&](const float4 &lo, const float4 &hi) {  // squared distance to the group's box
      const float dx = fmaxf(fmaxf(lo.x - hx, lx - hi.x), 0.0f);
      const float dy = fmaxf(fmaxf(lo.y - hy, ly - hi.y), 0.0f);
      const float dz = fmaxf(fmaxf(lo.z - hz, lz - hi.z), 0.0f);
      return dx * dx + dy * dy + dz * dz;
    };
    const float4 at = make_float4((float)px, (float)py, (float)pz, 0.0f);
    double den = 0.0;
    double num[kNc] = {};
    auto take = [&](int cnt) {  // the first cnt <= 64 of the list
      if (lane < cnt) {
        const int32_t k = S.list[lane];
        const double4 b = sd[k];
        S.h[lane] = b.w;
        // no smaller than any r^2 rounded with r < 2 h
        S.ball[lane] = make_double4(b.x, b.y, b.z, 4.0 * b.w * b.w * (1.0 + 1e-9) + 1e-290);
        const double *v = val + (int64_t)ncomp * H.sidx[k] + c0;
        for (int c = 0; c < kNc; ++c) S.val[lane][c] = v[c];
      }
      wave_order();
      if (mine) {
        uint32_t near[2] = {0u, 0u};  // those that reach this lane's particle, but for rounding
#pragma unroll
        for (int w = 0; w < 2; ++w)
#pragma unroll 4
          for (int k = 0; k < 32; ++k) {
            const double4 b = S.ball[32 * w + k];
            const double ex = px - b.x, ey = py - b.y, ez = pz - b.z;
            near[w] |= ex * ex + ey * ey + ez * ez > b.w ? 0u : 1u << k;
          }
        uint64_t m = (uint64_t)near[1] << 32 | near[0];
        if (cnt < 64) m &= (1ull << cnt) - 1ull;
        while (m) {  // kTurn at a time: their terms do not wait for each other
          int kk[kTurn];
          bool on[kTurn];
          double W[kTurn];
#pragma unroll
          for (int q = 0; q < kTurn; ++q) {
            on[q] = m != 0ull;
            kk[q] = on[q] ? __builtin_ctzll(m) : 0;
            m &= m - 1ull;
            const double4 b = S.ball[kk[q]];
            const double ex = px - b.x, ey = py - b.y, ez = pz - b.z, h = S.h[kk[q]];
            const double r = sqrt(ex * ex + ey * ey + ez * ez);
            on[q] = on[q] && r < 2.0 * h;
            W[q] = m4w(r / h);
          }
#pragma unroll
          for (int q = 0; q < kTurn; ++q) {
            den = on[q] ? den + W[q] : den;
#pragma unroll
            for (int c = 0; c < kNc; ++c) num[c] = on[q] ? num[c] + W[q] * S.val[kk[q]][c] : num[c];
          }
        }
      }
      wave_order();
    };
    int sp = 0, cnt = 0;
    // level lc's boxes, one a lane (j; in: there is one): those near the group
    // are pushed, or, over balls, looked into if they are near a particle of it
    auto expand = [&](int lc, int64_t j, bool in) {
      float4 lo = {}, hi = {};
      if (in) {
        lo = H.lo[lc][j];
        hi = H.hi[lc][j];
      }
      uint64_t m = __ballot(in && gap2(lo, hi) <= r2box);
      if (lc > 1) {
        const int nh = __popcll(m);
        if (m >> lane & 1ull) S.st[sp + nh - 1 - __popcll(m & below)] = ((uint32_t)j << 4) | (uint32_t)lc;
        sp += nh;
        wave_order();
        return;
      }
      for (uint64_t a = m; a; a &= a - 1ull) {
        const int k = __builtin_ctzll(a);
        const float4 l = make_float4(readlane_f(lo.x, k), readlane_f(lo.y, k), readlane_f(lo.z, k), 0.0f);
        const float4 u = make_float4(readlane_f(hi.x, k), readlane_f(hi.y, k), readlane_f(hi.z, k), 0.0f);
        if (!__ballot(mine && box_hit(l, u, at, r2box))) m &= ~(1ull << k);
      }
      const int nh = __popcll(m);
      if (m >> lane & 1ull) S.node[__popcll(m & below)] = (int32_t)j;
      wave_order();
      auto ball_of = [&](int q) { return (int64_t)S.node[min(q + (lane >> 4), nh - 1)] * kFan + (lane & 15); };
      int64_t k = nh ? ball_of(0) : H.n[0];
      float4 next = k < H.n[0] ? H.sx[k] : make_float4(0.0f, 0.0f, 0.0f, 0.0f);
      for (int q = 0; q < nh; q += 4) {
        const float4 b = next;
        const int32_t id = (int32_t)k;
        const float rr = 2.0f * b.w * 1.00001f + H.margin_abs;
        const bool hit = q + (lane >> 4) < nh && k < H.n[0] && !(gap2(b, b) > rr * rr);
        if (q + 4 < nh) {
          k = ball_of(q + 4);
          if (k < H.n[0]) next = H.sx[k];
        }
        const uint64_t mb = __ballot(hit);
        if (hit) S.list[cnt + __popcll(mb & below)] = id;
        cnt += __popcll(mb);
        wave_order();
        if (cnt >= 64) {
          take(64);
          const int32_t k2 = S.list[64 + lane];
          wave_order();
          if (lane < cnt - 64) S.list[lane] = k2;
          cnt -= 64;
          wave_order();
        }
      }
    };
    expand(top, lane, lane < H.n[top]);
    while (sp > 0) {
      // the top boxes of the stack, up to four of one level
      const uint32_t x = S.st[max(sp - 1 - (lane >> 4), 0)];
      const int l = __builtin_amdgcn_readfirstlane((int)(x & 15u));
      const uint64_t other = __ballot(sp - 1 < (lane >> 4) || (int)(x & 15u) != l);
      const int nb = other ? __builtin_ctzll(other) >> 4 : 4;
      sp -= nb;
      wave_order();
      const int64_t j = (int64_t)(x >> 4) * kFan + (lane & 15);
      expand(l - 1, j, (lane >> 4) < nb && j < H.n[l - 1]);
    }
    take(cnt);
    if (mine) {
      for (int c = 0; c < kNc; ++c) {
        const double v = den > 0.0 ? num[c] / den : val[(int64_t)ncomp * o + c0 + c];
        out[(int64_t)ncomp * i + c0 + c] = v;
        if (!isfinite(v)) bad = SPHMAP_STATUS_NONFINITE_VALUE;
      }
    }
  }
  if (bad) atomicOr(status, bad);
}

}  // namespace

// ------------------------------------------------- fixed device scratch
// Device memory for callers that cannot allocate (the no-allocation
// interpolation entry point): each device holds one copy for the life of
// the process.  Host code must not pass `scratch` itself to a kernel -- on
// the host that name is a stand-in, not a device address -- but the address
// hipGetSymbolAddress returns on each device, looked up once per device.
constexpr size_t kNoAllocScratch = (size_t)64 << 20;
static __device__ __align__(256) unsigned char scratch[kNoAllocScratch];

namespace {
constexpr int kMaxDevices = 64;
std::mutex g_scratch_mu;
void *g_scratch_ptr[kMaxDevices] = {};
}  // namespace

// Look up this device's copy of the scratch (called with `device` current,
// by context creation).  Later lookups return the recorded address.
void *noalloc_scratch_init(int device) {
  SPH_REQUIRE(device >= 0 && device < kMaxDevices, SPHMAP_EINVAL, "device index out of range");
  std::lock_guard<std::mutex> lock(g_scratch_mu);
  if (!g_scratch_ptr[device]) {
    void *p = nullptr;
    SPH_HIP(hipGetSymbolAddress(&p, HIP_SYMBOL(scratch)));
    SPH_REQUIRE(p != nullptr, SPHMAP_EHIP, "no device address for the fixed scratch");
    g_scratch_ptr[device] = p;
  }
  return g_scratch_ptr[device];
}

size_t noalloc_scratch_bytes() { return kNoAllocScratch; }

// Upper bound of the scratch interpolate_particles carves for n particles
// and ne entries: Morton keys, index, sorted float4 and double4 copies and
// radix temporaries per entry; place keys, index and radix temporaries per
// particle; the search boxes; digit histograms and scan sums; and 256 bytes
// of alignment and padding for each of up to 64 named buffers.
size_t interp_scratch_bound(int64_t n, int64_t ne) {
  const double per_entry = 8 + 4 + 8 + 4 + 16 + 32 + 2.2 * 16;
  const double per_part = 4 + 4 + 4 + 4;
  const double hist = 4.0 * (16.0 * (double)(div_up(std::max(n, ne), 2048) + 1) * 8.0 + 64.0);
  return (size_t)(per_entry * (double)ne + per_part * (double)n + hist + 64.0 * 512.0 + 65536.0);
}

void interpolate_particles(Ctx &ctx, int64_t n, const double *xyz, const int64_t *owner, int64_t ne,
                           const double *exyz, const double *eh, const int32_t *ekind, const double *val, int ncomp,
                           double *out, hipStream_t s) {
  if (n <= 0) return;
  SPH_REQUIRE(ne > 0 && ne < ((int64_t)1 << 31), SPHMAP_EINVAL, "entry count out of range");
  SPH_REQUIRE(n < ((int64_t)1 << 31), SPHMAP_EINVAL, "particle count out of range");
  SPH_REQUIRE(ncomp >= 1, SPHMAP_EINVAL, "ncomp must be at least 1");
  Arena &ar = ctx.arena;
  int *bad = ar.get<int>("ip_bad", 1);
  SPH_HIP(hipMemsetAsync(bad, 0, sizeof(int), s));
  k_interp_check<<<(unsigned)div_up(std::max(n, ne), 256), 256, 0, s>>>(n, xyz, owner, ne, exyz, bad);
  SPH_LAUNCH_CHECK();
  int bad_h = 0;
  SPH_HIP(hipMemcpyAsync(&bad_h, bad, sizeof(int), hipMemcpyDeviceToHost, s));
  SPH_HIP(hipStreamSynchronize(s));
  SPH_REQUIRE(!(bad_h & 2), SPHMAP_EINVAL, "owner index outside [0, n_entries)");
  SPH_REQUIRE(!(bad_h & 5), SPHMAP_EINVAL, "particle or entry outside [0,1)^3");

  // entries in Morton order under the ball hierarchy
  uint64_t *keys = ar.get<uint64_t>("ip_keys", ne);
  int32_t *sidx = ar.get<int32_t>("ip_sidx", ne);
  morton_keys(exyz, 3, ne, 0.0, 0.0, 0.0, 1.0, keys, sidx, s);
  radix_sort_u64_range(ar, keys, sidx, ne, 33, 63, s);  // top 10 bits per axis
  float4 *sx = ar.get<float4>("ip_sx", ne);
  double4 *sd = ar.get<double4>("ip_sd", ne);
  k_entry_prep<<<(unsigned)div_up(ne, 256), 256, 0, s>>>(ne, sidx, exyz, eh, sx, sd);
  SPH_LAUNCH_CHECK();
  Hier H;
  H.sx = sx;
  H.sidx = sidx;
  build_hier(ar, sx, ne, 1e-6f, "ip", H, s);

  // particles grouped by place (no use where one batch holds every ball)
  int32_t *qidx = ar.get<int32_t>("ip_qidx", n);
  if (ne > 64) {
    uint32_t *pkey = ar.get<uint32_t>("ip_pkey", n);
    k_place_keys<<<(unsigned)div_up(n, 256), 256, 0, s>>>(n, xyz, pkey, qidx);
    SPH_LAUNCH_CHECK();
    radix_sort_u32(ar, pkey, qidx, n, kPlaceBits, s);
  } else {
    iota_i32(qidx, n, s);
  }

  int per = 64;
  while (per > 1 && div_up(n, per) < kInterpWaves) per /= 2;
  KernelTimer kt(&ctx, "interp", s);
  for (int c0 = 0; c0 < ncomp; c0 += kCompPass) {
    const int nc = std::min(kCompPass, ncomp - c0);
    const auto fn = nc == 1 ? k_interp<1> : nc == 2 ? k_interp<2> : nc == 3 ? k_interp<3> : k_interp<4>;
    fn<<<(unsigned)div_up(n, per), 64, 0, s>>>(H, sd, n, per, qidx, xyz, owner, eh, ekind, val, ncomp, c0, out,
                                              ctx.d_status);
    SPH_LAUNCH_CHECK();
  }
  kt.done();
}

// The same with every buffer carved from this device's fixed scratch: no
// device memory is allocated or freed.  Calls on one device share the
// scratch, so calls that overlap in time on one device race.
void interpolate_particles_noalloc(Ctx &ctx, int64_t n, const double *xyz, const int64_t *owner, int64_t ne,
                                   const double *exyz, const double *eh, const int32_t *ekind, const double *val,
                                   int ncomp, double *out, hipStream_t s) {
  SPH_REQUIRE(ne > 0 && ne < ((int64_t)1 << 31) && n >= 0 && n < ((int64_t)1 << 31), SPHMAP_EINVAL,
              "particle or entry count out of range");
  const size_t need = interp_scratch_bound(n, ne);
  SPH_REQUIRE(need <= kNoAllocScratch, SPHMAP_EINVAL,
              "n = " + std::to_string(n) + " particles and " + std::to_string(ne) + " entries need up to " +
                  std::to_string(need) + " bytes, more than the " + std::to_string(kNoAllocScratch) +
                  "-byte fixed scratch");
  void *base = g_scratch_ptr[ctx.device];
  SPH_REQUIRE(base != nullptr, SPHMAP_EHIP, "the fixed scratch of this device was not looked up");
  Arena region;
  region.region = (char *)base;
  region.region_cap = kNoAllocScratch;
  struct Swap {  // every request of the call goes to the region; timing off (no events)
    Ctx &c;
    bool timing;
    Swap(Ctx &cc, Arena *r) : c(cc), timing(cc.timing) {
      c.arena.redirect = r;
      c.timing = false;
    }
    ~Swap() {
      c.arena.redirect = nullptr;
      c.timing = timing;
    }
  } swap(ctx, &region);
  interpolate_particles(ctx, n, xyz, owner, ne, exyz, eh, ekind, val, ncomp, out, s);
}

}  // namespace sphmap
