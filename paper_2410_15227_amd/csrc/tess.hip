// Tessellation preprocessing (once per uploaded tessellation) and particle
// staging.
//
// Per face: the Newell area vector gives the plane; the face is oriented so
// that its normal points away from the cell's generation site (the site is
// strictly inside its Voronoi cell), its vertices are rewritten about the
// site in that orientation (counter-clockwise seen from outside), and a
// bounding sphere about the vertex centroid is kept for culling.  Per cell:
// the volume (sum of pyramids from the site) and the canonical binary32
// bounding radius used by the candidate-pair test.
#include "common.hpp"

namespace sphmap {
namespace {

__global__ void k_face_cell(const int64_t *cfo, int64_t C, int32_t *face_cell) {
  int64_t c = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (c >= C) return;
  for (int64_t f = cfo[c]; f < cfo[c + 1]; ++f) face_cell[f] = (int32_t)c;
}

// Canonical radius: smallest binary32 R with R*R >= max_v |v - g|^2 where
// the squared distance is (dx*dx + dy*dy) + dz*dz in binary64 without
// contraction.
__device__ float canonical_radius(double r2) {
  float R = (float)sqrt(r2);
  while ((double)R * (double)R < r2) R = nextafterf(R, INFINITY);
  while (R > 0.0f) {
    float Rm = nextafterf(R, 0.0f);
    if ((double)Rm * (double)Rm >= r2) R = Rm;
    else break;
  }
  return R;
}

struct TessOut {
  double4 *fplane, *fsphere;
  double *fvpos;
  float4 *fvpos32, *fplane32, *edgeA, *edgeE, *edgeM;
  double *volume;
  float *radius;
  float4 *gen32;
  int *bad;
};

struct FaceGeo {  // about the cell's site
  double cx, cy, cz, rad2;  // centroid of the vertices, squared radius about it
  double nx, ny, nz, off;   // outward unit normal, plane offset (<= 0: skip the face)
  bool rev;                 // the vertices come clockwise seen from outside
};

// pos(k, x, y, z): vertex k of the face about the site
template <class Pos>
__device__ inline FaceGeo face_geo(int nv, Pos pos, int *bad) {
  FaceGeo g;
  g.cx = g.cy = g.cz = 0;
  for (int k = 0; k < nv; ++k) {
    double x, y, z;
    pos(k, x, y, z);
    g.cx += x;
    g.cy += y;
    g.cz += z;
  }
  if (nv > 0) {
    g.cx /= nv;
    g.cy /= nv;
    g.cz /= nv;
  }
  double ax = 0, ay = 0, az = 0;
  g.rad2 = 0;
  for (int k = 0; k < nv; ++k) {
    double px, py, pz, qx, qy, qz;
    pos(k, px, py, pz);
    pos(k + 1 == nv ? 0 : k + 1, qx, qy, qz);
    px -= g.cx, py -= g.cy, pz -= g.cz;
    qx -= g.cx, qy -= g.cy, qz -= g.cz;
    ax += 0.5 * (py * qz - pz * qy);
    ay += 0.5 * (pz * qx - px * qz);
    az += 0.5 * (px * qy - py * qx);
    g.rad2 = fmax(g.rad2, px * px + py * py + pz * pz);
  }
  double an = sqrt(ax * ax + ay * ay + az * az);
  g.nx = g.ny = g.nz = 0;
  g.off = -1.0;
  g.rev = false;
  if (nv >= 3 && an > 0.0) {
    g.nx = ax / an;
    g.ny = ay / an;
    g.nz = az / an;
    g.off = g.nx * g.cx + g.ny * g.cy + g.nz * g.cz;
    if (g.off < 0.0) {
      g.rev = true;
      g.nx = -g.nx;
      g.ny = -g.ny;
      g.nz = -g.nz;
      g.off = -g.off;
    }
    if (!(g.off > 0.0)) {
      atomicAdd(bad, 1);  // generation site on the face plane: not a valid cell
      g.off = -1.0;
    }
  }
  return g;
}

__device__ inline void store_face(int64_t f, const FaceGeo &g, const TessOut &T) {
  T.fplane[f] = make_double4(g.nx, g.ny, g.nz, g.off);
  T.fplane32[f] = make_float4((float)g.nx, (float)g.ny, (float)g.nz, (float)g.off);
  T.fsphere[f] = make_double4(g.cx, g.cy, g.cz, sqrt(g.rad2));
}

// slot t: vertex A of the oriented polygon and the edge to its next vertex B
__device__ inline void store_slot(int64_t t, double Ax, double Ay, double Az, double Bx, double By, double Bz, double nx,
                                  double ny, double nz, const TessOut &T) {
  T.fvpos[3 * t + 0] = Ax;
  T.fvpos[3 * t + 1] = Ay;
  T.fvpos[3 * t + 2] = Az;
  T.fvpos32[t] = make_float4((float)Ax, (float)Ay, (float)Az, 0.0f);
  const double bx = Bx - Ax, by = By - Ay, bz = Bz - Az;
  const double len = sqrt(bx * bx + by * by + bz * bz);
  double ex = 0.0, ey = 0.0, ez = 0.0;
  if (len > 0.0) {
    ex = bx / len;
    ey = by / len;
    ez = bz / len;
  }
  const double mx = ny * ez - nz * ey, my = nz * ex - nx * ez, mz = nx * ey - ny * ex;
  T.edgeA[t] = make_float4((float)Ax, (float)Ay, (float)Az, (float)len);
  T.edgeE[t] = make_float4((float)ex, (float)ey, (float)ez, 0.0f);
  T.edgeM[t] = make_float4((float)mx, (float)my, (float)mz, 0.0f);
}

// squared distance of a vertex from the site, as the radius takes it
__device__ inline double site_dist2(double x, double y, double z) {
#pragma clang fp contract(off)
  return (x * x + y * y) + z * z;
}

// the face's pyramid from the site: plane offset times area over 3
template <class Pos>
__device__ inline double pyramid(int nv, Pos pos, double cx, double cy, double cz, double off) {
#pragma clang fp contract(off)
  double ax = 0, ay = 0, az = 0;
  for (int k = 0; k < nv; ++k) {
    double px, py, pz, qx, qy, qz;
    pos(k, px, py, pz);
    pos(k + 1 == nv ? 0 : k + 1, qx, qy, qz);
    px -= cx, py -= cy, pz -= cz;
    qx -= cx, qy -= cy, qz -= cz;
    ax += 0.5 * (py * qz - pz * qy);
    ay += 0.5 * (pz * qx - px * qz);
    az += 0.5 * (px * qy - py * qx);
  }
  return off * sqrt(ax * ax + ay * ay + az * az) / 3.0;
}

__device__ inline void store_cell(int64_t c, const double *gen, double vol, double r2, const TessOut &T) {
  T.volume[c] = vol;
  const float R = canonical_radius(r2);
  T.radius[c] = R;
  T.gen32[c] = make_float4((float)gen[3 * c], (float)gen[3 * c + 1], (float)gen[3 * c + 2], R);
}

// Planes, spheres, edges, volumes and radii.  A workgroup takes kPrepCells
// cells, whose faces and face-vertex slots are contiguous, and loads the
// slots' vertices into LDS once, a slot a thread; then a face a thread, then
// a slot a thread for what is stored per slot (112 bytes, contiguous), then a
// cell a thread, its faces' volumes added in their order.  Cells that do not
// fit (more than kPrepFaces faces or kPrepSlots slots) go the same way from
// global memory, a face and then a cell a thread.  Bounded by the gather
// of the vertices and the stores: 1.5 GB in 0.36 ms for 131,071 cells, where a
// face a thread and then a cell a thread, each from global memory, took 1.56
// ms (MI355X; 4 and 12 cells a workgroup 0.4 to 1 % of a build slower).
constexpr int kPrepThreads = 256;
constexpr int kPrepCells = 8;
constexpr int kPrepFaces = kPrepThreads;
constexpr int kPrepSlots = 1024;
constexpr int64_t kPrepBlocks = 1 << 16;  // workgroups of a launch: a grid of 2^27 cells is past what one takes

__global__ void __launch_bounds__(kPrepThreads) k_tess_prep(int64_t first, int64_t C, const double *gen,
                                                           const double *vert, const int64_t *cfo, const int64_t *fvo,
                                                           const int32_t *fv, TessOut T) {
  __shared__ double px[kPrepSlots], py[kPrepSlots], pz[kPrepSlots];
  __shared__ uint8_t slot_face[kPrepSlots];
  __shared__ double fn[3][kPrepFaces], fvol[kPrepFaces];
  __shared__ unsigned long long fr2[kPrepFaces];  // non-negative doubles order as their bits
  __shared__ int fs[kPrepFaces + 1];              // first slot of each face
  __shared__ bool frev[kPrepFaces];
  __shared__ uint8_t fcell[kPrepFaces];
  const int tid = threadIdx.x;
  const int64_t c0 = first + (int64_t)blockIdx.x * kPrepCells, c1 = min(C, c0 + kPrepCells);
  const int64_t f0 = cfo[c0], f1 = cfo[c1];
  const int64_t s0 = fvo[f0], s1 = fvo[f1];
  if (f1 - f0 <= kPrepFaces && s1 - s0 <= kPrepSlots) {
    const int nf = (int)(f1 - f0), ns = (int)(s1 - s0);
    for (int c = tid; c < (int)(c1 - c0); c += kPrepThreads)
      for (int64_t f = cfo[c0 + c]; f < cfo[c0 + c + 1]; ++f) fcell[f - f0] = (uint8_t)c;
    int a = 0, b = 0;  // this thread's face
    if (tid < nf) {
      a = (int)(fvo[f0 + tid] - s0);
      b = (int)(fvo[f0 + tid + 1] - s0);
      fs[tid] = a;
      fr2[tid] = 0ull;
      for (int k = a; k < b; ++k) slot_face[k] = (uint8_t)tid;
    }
    if (tid == 0) fs[nf] = ns;
    __syncthreads();
    for (int k = tid; k < ns; k += kPrepThreads) {
      const int j = slot_face[k];
      const double *g = gen + 3 * (c0 + fcell[j]);
      const double *v = vert + 3 * (int64_t)fv[s0 + k];
      const double x = v[0] - g[0], y = v[1] - g[1], z = v[2] - g[2];
      px[k] = x;
      py[k] = y;
      pz[k] = z;
      const double d2 = site_dist2(x, y, z);
      if (d2 > 0.0) atomicMax(&fr2[j], (unsigned long long)__double_as_longlong(d2));
    }
    __syncthreads();
    if (tid < nf) {
      const auto pos = [&](int k, double &x, double &y, double &z) {
        x = px[a + k];
        y = py[a + k];
        z = pz[a + k];
      };
      const FaceGeo g = face_geo(b - a, pos, T.bad);
      store_face(f0 + tid, g, T);
      fn[0][tid] = g.nx;
      fn[1][tid] = g.ny;
      fn[2][tid] = g.nz;
      frev[tid] = g.rev;
      fvol[tid] = g.off > 0.0 ? pyramid(b - a, pos, g.cx, g.cy, g.cz, g.off) : -1.0;
    }
    __syncthreads();
    for (int k = tid; k < ns; k += kPrepThreads) {
      const int j = slot_face[k], e = fs[j], nv = fs[j + 1] - e, q = k - e, q1 = q + 1 == nv ? 0 : q + 1;
      const int A = e + (frev[j] ? nv - 1 - q : q), B = e + (frev[j] ? nv - 1 - q1 : q1);
      store_slot(s0 + k, px[A], py[A], pz[A], px[B], py[B], pz[B], fn[0][j], fn[1][j], fn[2][j], T);
    }
    if (tid < (int)(c1 - c0)) {
      double vol = 0.0;
      unsigned long long r2 = 0ull;
      for (int64_t f = cfo[c0 + tid]; f < cfo[c0 + tid + 1]; ++f) {
        const int j = (int)(f - f0);
        if (!(fvol[j] < 0.0)) vol += fvol[j];
        if (fr2[j] > r2) r2 = fr2[j];
      }
      store_cell(c0 + tid, gen, vol, __longlong_as_double((long long)r2), T);
    }
    return;
  }
  for (int64_t c = c0; c < c1; ++c) {
    const double gx = gen[3 * c], gy = gen[3 * c + 1], gz = gen[3 * c + 2];
    for (int64_t f = cfo[c] + tid; f < cfo[c + 1]; f += kPrepThreads) {
      const int64_t e = fvo[f];
      const int nv = (int)(fvo[f + 1] - e);
      const auto pos = [&](int k, double &x, double &y, double &z) {
        const double *v = vert + 3 * (int64_t)fv[e + k];
        x = v[0] - gx;
        y = v[1] - gy;
        z = v[2] - gz;
      };
      const FaceGeo g = face_geo(nv, pos, T.bad);
      store_face(f, g, T);
      for (int k = 0; k < nv; ++k) {
        const int k1 = k + 1 == nv ? 0 : k + 1;
        double Ax, Ay, Az, Bx, By, Bz;
        pos(g.rev ? nv - 1 - k : k, Ax, Ay, Az);
        pos(g.rev ? nv - 1 - k1 : k1, Bx, By, Bz);
        store_slot(e + k, Ax, Ay, Az, Bx, By, Bz, g.nx, g.ny, g.nz, T);
      }
    }
  }
  __syncthreads();  // the faces' planes and spheres are read back
  for (int64_t c = c0 + tid; c < c1; c += kPrepThreads) {
    const double gx = gen[3 * c], gy = gen[3 * c + 1], gz = gen[3 * c + 2];
    double vol = 0.0, r2 = 0.0;
    for (int64_t f = cfo[c]; f < cfo[c + 1]; ++f) {
      const int64_t e = fvo[f];
      const int nv = (int)(fvo[f + 1] - e);
      const auto pos = [&](int k, double &x, double &y, double &z) {
        const double *v = vert + 3 * (int64_t)fv[e + k];
        x = v[0] - gx;
        y = v[1] - gy;
        z = v[2] - gz;
      };
      for (int k = 0; k < nv; ++k) {
        double x, y, z;
        pos(k, x, y, z);
        const double d2 = site_dist2(x, y, z);
        if (d2 > r2) r2 = d2;
      }
      const double4 pl = T.fplane[f], sp = T.fsphere[f];
      if (pl.w > 0.0) vol += pyramid(nv, pos, sp.x, sp.y, sp.z, pl.w);
    }
    store_cell(c, gen, vol, r2, T);
  }
}

// Twin of each face: a face is shared when the cell it names has a face
// naming it back, both planes are valid, the two bounding spheres agree
// (centres in absolute coordinates and radii, to 1e-9 of the larger radius)
// and the normals are opposite.  Such a face is one polygon seen from two
// cells: its share of the Exact sum is the same magnitude from both sides
// with opposite sign (Sec. 3 of the closed form: C_f depends only on the
// polygon and the particle, the sign on the side).  twin[f] is the other
// cell, or -1 (a wall, no declaration, or no match); twin_face[f] the
// matching face of that cell.
__global__ void k_face_twin(int64_t F, int64_t C, const int32_t *face_cell, const int64_t *cfo, const int32_t *nbr,
                            const double *gen, const double4 *fplane, const double4 *fsphere, int32_t *twin,
                            int32_t *twin_face) {
  const int64_t f = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (f >= F) return;
  int32_t tw = -1, tf = -1;
  const int64_t c = face_cell[f], n = nbr[f];
  const double4 pa = fplane[f];
  if (n >= 0 && n < C && n != c && pa.w > 0.0) {
    const double4 sa = fsphere[f];
    const double ax = gen[3 * c] + sa.x, ay = gen[3 * c + 1] + sa.y, az = gen[3 * c + 2] + sa.z;
    const int64_t g1 = cfo[n + 1];
    int64_t g = cfo[n];
    for (; g < g1; g += 4) {  // the first face that names c, four loads at a time
      int32_t m[4];
#pragma unroll
      for (int u = 0; u < 4; ++u) m[u] = nbr[min(g + u, g1 - 1)];
      const int u = m[0] == c ? 0 : m[1] == c ? 1 : m[2] == c ? 2 : m[3] == c ? 3 : 4;
      if (u < 4) {
        g += u;
        break;
      }
    }
    if (g < g1) {
      const double4 pb = fplane[g], sb = fsphere[g];
      const double bx = gen[3 * n] + sb.x, by = gen[3 * n + 1] + sb.y, bz = gen[3 * n + 2] + sb.z;
      const double tol = 1e-9 * fmax(sa.w, sb.w);
      const double dx = ax - bx, dy = ay - by, dz = az - bz;
      if (pb.w > 0.0 && dx * dx + dy * dy + dz * dz <= tol * tol && fabs(sa.w - sb.w) <= tol &&
          pa.x * pb.x + pa.y * pb.y + pa.z * pb.z < -1.0 + 1e-9) {
        tw = (int32_t)n;
        tf = (int32_t)g;
      }
    }
  }
  twin[f] = tw;
  twin_face[f] = tf;
}

// Per cell: its faces' roles in the mixed path -- code[f] = the face's slot
// among the cell's shared faces it evaluates (twin cell above it), -1 for a
// face evaluated for this cell only (wall or unshared) -- and the number of
// such slots.  A second pass gives each shared face the twin evaluates the
// code -2 - (its twin's slot).  The shared faces are counted here, one atomic
// a workgroup of at most kSlotBlocks: one a wavefront of faces, 31,000 on one
// address, made the twin search of 131,071 cells take 0.41 ms, 0.20 without.
constexpr int kSlotBlocks = 512;
__global__ void __launch_bounds__(256) k_face_slots(int64_t C, const int64_t *cfo, const int32_t *twin, int32_t *code,
                                                    int32_t *n_slots, unsigned long long *n_shared) {
  __shared__ unsigned long long part[256 / 64];
  unsigned long long shared = 0;
  for (int64_t c = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; c < C; c += (int64_t)gridDim.x * blockDim.x) {
    int32_t n = 0;
    for (int64_t f = cfo[c]; f < cfo[c + 1]; ++f) {
      const int32_t tw = twin[f];
      code[f] = tw < 0 ? -1 : (tw > c ? n++ : -2);
      shared += tw >= 0;
    }
    n_slots[c] = n;
  }
#pragma unroll
  for (int o = 32; o > 0; o >>= 1) shared += __shfl_xor(shared, o, 64);
  if ((threadIdx.x & 63) == 0) part[threadIdx.x >> 6] = shared;
  __syncthreads();
  if (threadIdx.x == 0 && part[0] + part[1] + part[2] + part[3])
    atomicAdd(n_shared, part[0] + part[1] + part[2] + part[3]);
}

__global__ void k_face_slots_in(int64_t F, const int32_t *twin_face, int32_t *code) {
  const int64_t f = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (f >= F || code[f] != -2) return;
  code[f] = -2 - code[twin_face[f]];  // the twin's code is a slot (>= 0)
}

__global__ void k_particles_prep(int64_t n, const double *xyz, const double *h, float4 *x32) {
  int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= n) return;
  x32[i] = make_float4((float)xyz[3 * i], (float)xyz[3 * i + 1], (float)xyz[3 * i + 2], (float)h[i]);
}

}  // namespace

void tess_prepare(Ctx &ctx, TessDev &t, hipStream_t s) {
  const int64_t C = t.n_cells, F = t.n_faces, FV = t.n_fv;
  t.face_cell = t.mem.get<int32_t>("face_cell", F);
  t.fplane = t.mem.get<double4>("fplane", F);
  t.fsphere = t.mem.get<double4>("fsphere", F);
  t.fplane32 = t.mem.get<float4>("fplane32", F);
  t.fvpos = t.mem.get<double>("fvpos", 3 * FV);
  t.fvpos32 = t.mem.get<float4>("fvpos32", FV);
  t.edgeA = t.mem.get<float4>("edgeA", FV);
  t.edgeE = t.mem.get<float4>("edgeE", FV);
  t.edgeM = t.mem.get<float4>("edgeM", FV);
  t.volume = t.mem.get<double>("volume", C);
  t.radius = t.mem.get<float>("radius", C);
  t.gen32 = t.mem.get<float4>("gen32", C);
  t.cell_order = t.mem.get<int32_t>("cell_order", C);
  int *bad = t.mem.get<int>("bad", 1);
  SPH_HIP(hipMemsetAsync(bad, 0, sizeof(int), s));
  k_face_cell<<<(unsigned)div_up(C, 256), 256, 0, s>>>(t.cell_face_off, C, t.face_cell);
  SPH_LAUNCH_CHECK();
  const TessOut to{t.fplane, t.fsphere, t.fvpos,  t.fvpos32, t.fplane32, t.edgeA,
                   t.edgeE,  t.edgeM,   t.volume, t.radius,  t.gen32,    bad};
  for (int64_t c = 0; c < C; c += kPrepBlocks * kPrepCells) {
    k_tess_prep<<<(unsigned)std::min(div_up(C - c, kPrepCells), kPrepBlocks), kPrepThreads, 0, s>>>(
        c, C, t.gen, t.vert, t.cell_face_off, t.face_vtx_off, t.face_vtx, to);
    SPH_LAUNCH_CHECK();
  }
  // cells in Morton order of their sites (locality of the pair search)
  uint64_t *keys = t.mem.get<uint64_t>("cell_keys", C);
  morton_keys(t.gen, 3, C, t.box_lo[0], t.box_lo[1], t.box_lo[2], t.box_size, keys, t.cell_order, s);
  radix_sort_u64(ctx.arena, keys, t.cell_order, C, 63, s);
  int bad_h = 0;
  SPH_HIP(hipMemcpyAsync(&bad_h, bad, sizeof(int), hipMemcpyDeviceToHost, s));
  SPH_HIP(hipStreamSynchronize(s));
  SPH_REQUIRE(bad_h == 0, SPHMAP_EGEOM,
              std::to_string(bad_h) + " face(s) have the generation site on their plane (site not strictly inside)");
  // a grid built here records the neighbour of every face
  if (t.face_nbr) tess_set_twins(ctx, t, t.face_nbr, s);
}

int64_t tess_set_twins(Ctx &ctx, TessDev &t, const int32_t *d_nbr, hipStream_t s) {
  (void)ctx;
  if (!d_nbr || t.n_faces == 0) {
    t.face_twin = t.twin_face = t.face_code = t.cell_slots = nullptr;
    return 0;
  }
  int32_t *tw = t.mem.get<int32_t>("ftwin", t.n_faces);
  int32_t *tf = t.mem.get<int32_t>("ftwinf", t.n_faces);
  int32_t *code = t.mem.get<int32_t>("fcode", t.n_faces);
  int32_t *ns = t.mem.get<int32_t>("cslots", t.n_cells);
  unsigned long long *cnt = t.mem.get<unsigned long long>("ftwin_n", 1);
  SPH_HIP(hipMemsetAsync(cnt, 0, sizeof(unsigned long long), s));
  k_face_twin<<<(unsigned)div_up(t.n_faces, 256), 256, 0, s>>>(t.n_faces, t.n_cells, t.face_cell, t.cell_face_off,
                                                               d_nbr, t.gen, t.fplane, t.fsphere, tw, tf);
  SPH_LAUNCH_CHECK();
  k_face_slots<<<(unsigned)std::min<int64_t>(div_up(t.n_cells, 256), kSlotBlocks), 256, 0, s>>>(
      t.n_cells, t.cell_face_off, tw, code, ns, cnt);
  SPH_LAUNCH_CHECK();
  k_face_slots_in<<<(unsigned)div_up(t.n_faces, 256), 256, 0, s>>>(t.n_faces, tf, code);
  SPH_LAUNCH_CHECK();
  unsigned long long n = 0;
  SPH_HIP(hipMemcpyAsync(&n, cnt, sizeof(n), hipMemcpyDeviceToHost, s));
  SPH_HIP(hipStreamSynchronize(s));
  if (n) {
    t.face_twin = tw;
    t.twin_face = tf;
    t.face_code = code;
    t.cell_slots = ns;
  } else {
    t.face_twin = t.twin_face = t.face_code = t.cell_slots = nullptr;
  }
  return (int64_t)n;
}

void particles_prepare(Ctx &ctx, PartDev &p, hipStream_t s) {
  (void)ctx;
  k_particles_prep<<<(unsigned)div_up(p.n, 256), 256, 0, s>>>(p.n, p.xyz, p.h, p.x32);
  SPH_LAUNCH_CHECK();
}

}  // namespace sphmap
