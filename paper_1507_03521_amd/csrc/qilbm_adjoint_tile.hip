// Adjoint step of small and medium lattices: a workgroup owns a tile of
// TX x TY nodes and applies every transposed stage to all its nodes at once,
// in the order of k_adj_fused (qilbm_adjoint.hip), whose row sweep is a serial
// chain of at least 24 row iterations of four barriers whatever the lattice's
// size (124 us per FP64 step at 512 x 512). Here a step is four barriers:
//   0   record planes phi, mu, p over the tile and four nodes around it
//   A'  collision transpose over the tile and three nodes around it (the
//       third ring only for its grad p cotangent, which needs no f)
//   B'  pressure cotangent and the macroscopic transposes over the tile and
//       two nodes around it; f cotangents of the tile out
//   C'  mu cotangent, then mu(phi), over the tile and one node around it
//   D'  phi cotangent, g cotangents of the tile out
// Fields that cross nodes live in LDS planes; a node's own cotangents and
// forward state stay in the registers of its thread from A' to D'. Threads:
// interior nodes first, then the two rings around them; the nodes of the
// third ring are shared out over all threads, those without an own node first.
#include "qilbm_adjoint.hpp"
#include "qilbm_adjoint_node.hpp"
#include "qilbm_internal.hpp"
#include "qilbm_tile.hpp"

namespace qilbm {

namespace {

// Post-collision cotangents of node k: population i at x + c_i, or opp(i) at
// the node itself when x + c_i lies beyond a wall. EDGE: the node may lie on
// a wall row.
template <typename T, bool EDGE, int KOFF, int I = 0>
__device__ __forceinline__ void tile_post(__amdgpu_buffer_rsrc_t rs, uint32_t ps,
                                          const TileNode& k, T v[9]) {
  if constexpr (I < 9) {
    constexpr int cx = CXS(I), cy = CYS(I);
    constexpr uint32_t size = (uint32_t)sizeof(T);
    const uint32_t off = (k.r[1 + cy] + k.c[1 + cx]) * size;
    if constexpr (EDGE && cy != 0) {
      const bool wall = cy > 0 ? k.hi : k.lo;
      const uint32_t own = (uint32_t)(KOFF + OPP(I)) * ps + (k.r[1] + k.c[1]) * size;
      v[I] = buf_ld<T>(rs, wall ? own : (uint32_t)(KOFF + I) * ps + off, 0);
    } else {
      v[I] = buf_ld<T>(rs, off, (uint32_t)(KOFF + I) * ps);
    }
    tile_post<T, EDGE, KOFF, I + 1>(rs, ps, k, v);
  }
}

// grad^T (vx, vy) at element e. The transposed stencil of a wall row drops
// the sources beyond the wall and adds, for the mirrored ghost, the row's own
// values with the sign of c_y turned: the same sum with the row beyond
// replaced by e's own and its vy negated.
template <typename T, int PX>
__device__ __forceinline__ T tile_gradT(const T* vx, const T* vy, int e, bool lo, bool hi) {
  const int em = lo ? e : e - PX, ep = hi ? e : e + PX;
  const T sm = lo ? T(-1) : T(1), sp = hi ? T(1) : T(-1);
  const T ax = (vx[e - 1] - vx[e + 1]) + fmad(sm, vy[em], sp * vy[ep]);
  const T dm = (vx[em - 1] - vx[em + 1]) + sm * (vy[em - 1] + vy[em + 1]);
  const T dp = (vx[ep - 1] - vx[ep + 1]) + sp * (vy[ep - 1] + vy[ep + 1]);
  return fmad(T(1.0 / 12.0), dm + dp, T(1.0 / 3.0) * ax);
}

// lap^T ws at element e (the Laplacian's weights are even in c, so the
// mirrored ghost is the row's own value).
template <typename T, int PX>
__device__ __forceinline__ T tile_lapT(const T* ws, int e, bool lo, bool hi) {
  const int em = lo ? e : e - PX, ep = hi ? e : e + PX;
  const T sa = (ws[e - 1] + ws[e + 1]) + (ws[em] + ws[ep]);
  const T sd = (ws[em - 1] + ws[em + 1]) + (ws[ep - 1] + ws[ep + 1]);
  return fmad(T(2.0 / 3.0), sa, fmad(T(1.0 / 6.0), sd, T(-10.0 / 3.0) * ws[e]));
}

// Adds the workgroup's four FP64 parameter sums to its slots: a fixed order
// for a fixed launch shape, so the totals are reproducible.
template <int NT>
__device__ __forceinline__ void block_add4(double (&v)[4], double* acc_part) {
  __shared__ double red[4][NT / 64];
#pragma unroll
  for (int q = 0; q < 4; ++q) {
#pragma unroll
    for (int off = 32; off > 0; off >>= 1) v[q] += __shfl_down(v[q], off, 64);
  }
  if ((threadIdx.x & 63) == 0) {
#pragma unroll
    for (int q = 0; q < 4; ++q) red[q][threadIdx.x >> 6] = v[q];
  }
  __syncthreads();
  if (threadIdx.x < 4) {
    double s = red[threadIdx.x][0];
#pragma unroll
    for (int w = 1; w < NT / 64; ++w) s += red[threadIdx.x][w];
    acc_part[4 * blockIdx.x + threadIdx.x] += s;
  }
}

// LDS planes of the tile and four nodes around it. The record's phi, mu and
// p are last read in A', the grad p cotangent in B', so later planes take
// their place.
template <typename T, int N>
struct AdjTileLds {
  T a[3][N];     // phi, mu, p; from B' on lambda D, grad mu x and y cotangents
  T gp[2][N];    // grad p cotangent; from C' on [0]: lap phi cotangent
  T gr[2][N];    // grad phi cotangent
};

template <typename T, int TX, int TY, int NT, bool EDGE>
__device__ __forceinline__ void adj_tile(__amdgpu_buffer_rsrc_t rrec, __amdgpu_buffer_rsrc_t rin,
                                         __amdgpu_buffer_rsrc_t rout, const Coef<T>& c,
                                         const Geom& g, int x0, int y0,
                                         AdjTileLds<T, (TX + 8) * (TY + 8)>& L,
                                         double (&acc)[4]) {
  constexpr int PX = TX + 8, PY = TY + 8;
  constexpr int NI = TX * TY, NP = (TX + 4) * (TY + 4);
  constexpr int NX = frame_count<TX + 4, TY + 4, 1>();
  constexpr uint32_t size = (uint32_t)sizeof(T);
  static_assert(NP <= NT, "one own node per thread");
  const uint32_t ps = (uint32_t)(g.Ns * (int64_t)sizeof(T));
  const int t = threadIdx.x;
  int lx = 0, ly = 0;
  if (t < NI) {
    ly = t / TX;
    lx = t - ly * TX;
  } else if (t < NP) {
    frame_pos<TX, TY, 2>(t - NI, lx, ly);
  }
  const int e = (ly + 4) * PX + lx + 4;
  const TileNode k = tile_node(x0 + lx, y0 + ly, g);
  const bool owns = t < NI && x0 + lx < g.nx && y0 + ly < g.ny;
  const uint32_t vo = (k.r[1] + k.c[1]) * size;
  T hf[9], hg[9], S = T(0), jx = T(0), jy = T(0);
  if (t < NP) {
    tile_post<T, EDGE, 0>(rin, ps, k, hf);
    tile_post<T, EDGE, 9>(rin, ps, k, hg);
    S = buf_ld<T>(rrec, vo, R_S * ps);
    jx = buf_ld<T>(rrec, vo, R_JX * ps);
    jy = buf_ld<T>(rrec, vo, R_JY * ps);
  }
  // 0
  for (int i = t; i < PX * PY; i += NT) {
    const int y = i / PX, x = i - y * PX;
    const TileNode ki = tile_node(x0 + x - 4, y0 + y - 4, g);
    const uint32_t v = (ki.r[1] + ki.c[1]) * size;
    L.a[0][i] = buf_ld<T>(rrec, v, R_PHI * ps);
    L.a[1][i] = buf_ld<T>(rrec, v, R_MU * ps);
    L.a[2][i] = buf_ld<T>(rrec, v, R_P * ps);
  }
  __syncthreads();
  // A'
  NodeBar<T> nb;
  Macro<T> m;
  T gmux = T(0), gmuy = T(0), lapmu = T(0), lapphi = T(0);
  if (t < NP) {
    T v[3][3], gphx, gphy, dpx, dpy, lapp;
    tile3x3<T, PX>(L.a[0], e, k.lo, k.hi, v);
    stencil(v, gphx, gphy, lapphi);
    const T ph = v[1][1];
    tile3x3<T, PX>(L.a[1], e, k.lo, k.hi, v);
    stencil(v, gmux, gmuy, lapmu);
    macro_node(ph, v[1][1], gphx, gphy, gmux, gmuy, lapmu, S, jx, jy, c, m);
    tile3x3<T, PX>(L.a[2], e, k.lo, k.hi, v);
    stencil(v, dpx, dpy, lapp);
    collide_node_T(hf, hg, m, dpx, dpy, c, nb);
    L.gp[0][e] = nb.dpx;
    L.gp[1][e] = nb.dpy;
  }
  for (int h = t >= NP ? t - NP : t + NT - NP; h < NX; h += NT) {
    int hx, hy;
    frame_pos<TX + 4, TY + 4, 1>(h, hx, hy);
    hx -= 2;
    hy -= 2;
    const int eh = (hy + 4) * PX + hx + 4;
    const TileNode kh = tile_node(x0 + hx, y0 + hy, g);
    const uint32_t vh = (kh.r[1] + kh.c[1]) * size;
    // grad p enters the collision only through Q = (c - u).(grad p - F),
    // whose cotangent does not depend on it: the f cotangents and grad p
    // itself reach only outputs that are not used here
    T gh[9], fh[9] = {};
    tile_post<T, EDGE, 9>(rin, ps, kh, gh);
    const T hjx = buf_ld<T>(rrec, vh, R_JX * ps), hjy = buf_ld<T>(rrec, vh, R_JY * ps);
    T v[3][3], ax, ay, al, bx, by, bl;
    tile3x3<T, PX>(L.a[0], eh, kh.lo, kh.hi, v);
    stencil(v, ax, ay, al);
    const T ph = v[1][1];
    tile3x3<T, PX>(L.a[1], eh, kh.lo, kh.hi, v);
    stencil(v, bx, by, bl);
    Macro<T> mh;
    macro_node(ph, v[1][1], ax, ay, bx, by, bl, T(0), hjx, hjy, c, mh);
    NodeBar<T> nh;
    collide_node_T(fh, gh, mh, T(0), T(0), c, nh);
    L.gp[0][eh] = nh.dpx;
    L.gp[1][eh] = nh.dpy;
  }
  __syncthreads();
  // B'
  T p2 = T(0);
  if (t < NP) {
    const T b_p = nb.p + tile_gradT<T, PX>(L.gp[0], L.gp[1], e, k.lo, k.hi);
    T b_rho = nb.rho, b_ux = nb.ux, b_uy = nb.uy;
    T b_Fx = nb.Fx, b_Fy = nb.Fy, b_drx = nb.drx, b_dry = nb.dry;
    T b_D = nb.D, b_phi = nb.phi;
    // p = S + (ux drx + uy dry - gamma rho D) / 6
    b_ux += b_p * m.drx * T(1.0 / 6.0);
    b_uy += b_p * m.dry * T(1.0 / 6.0);
    b_drx += b_p * m.ux * T(1.0 / 6.0);
    b_dry += b_p * m.uy * T(1.0 / 6.0);
    b_rho -= b_p * c.gamma * m.D * T(1.0 / 6.0);
    b_D -= b_p * c.gamma * m.rho * T(1.0 / 6.0);
    // u = (j + F / 6) * inv, inv = 3 / rho
    const T rinv = recip(m.rho);
    const T inv = T(3) * rinv;
    const T b_jx = b_ux * inv, b_jy = b_uy * inv;
    b_Fx += b_ux * inv * T(1.0 / 6.0);
    b_Fy += b_uy * inv * T(1.0 / 6.0);
    const T b_inv = b_ux * (jx + m.Fx * T(1.0 / 6.0)) + b_uy * (jy + m.Fy * T(1.0 / 6.0));
    b_rho -= b_inv * inv * rinv;
    // F = -phi grad mu + (rho - rho_ref) g
    b_phi -= b_Fx * gmux + b_Fy * gmuy;
    b_rho += b_Fx * c.gx + b_Fy * c.gy;
    // D = lambda lap mu; grad rho = drho grad phi; rho = rho_B + drho phi
    L.a[0][e] = c.lam * b_D;
    L.a[1][e] = -m.phi * b_Fx;
    L.a[2][e] = -m.phi * b_Fy;
    L.gr[0][e] = c.drho * b_drx;
    L.gr[1][e] = c.drho * b_dry;
    p2 = b_phi + c.drho * b_rho;
    if (owns) {
      fbar_out([&](int i, T v) { buf_st<T>(v, rout, vo, (uint32_t)i * ps); }, hf, b_p, b_jx, b_jy);
      acc[AP_ALPHA] += double(nb.alpha);
      acc[AP_LAMBDA] += double(b_D) * double(lapmu);
    }
  }
  __syncthreads();
  // C'
  T p3 = T(0);
  if (t < NP && lx >= -1 && lx <= TX && ly >= -1 && ly <= TY) {
    const T b_mu = nb.mu + tile_gradT<T, PX>(L.a[1], L.a[2], e, k.lo, k.hi) +
                   tile_lapT<T, PX>(L.a[0], e, k.lo, k.hi);
    const T ph = m.phi;
    const T dbulk = c.beta4 * (T(3) * ph * ph - T(3) * ph + T(0.5));
    p3 = p2 + b_mu * dbulk;
    L.gp[0][e] = -c.kappa * b_mu;
    if (owns) {
      acc[AP_BETA] += double(b_mu) * 4.0 * double((ph - T(1)) * ph * (ph - T(0.5)));
      acc[AP_KAPPA] -= double(b_mu) * double(lapphi);
    }
  }
  __syncthreads();
  // D'
  if (owns) {
    const T b_phi = p3 + tile_gradT<T, PX>(L.gr[0], L.gr[1], e, k.lo, k.hi) +
                    tile_lapT<T, PX>(L.gp[0], e, k.lo, k.hi);
#pragma unroll
    for (int i = 0; i < 9; ++i) buf_st<T>(hg[i] + b_phi, rout, vo, (uint32_t)(9 + i) * ps);
  }
}

// FP64: held to the 168 registers that three wavefronts per SIMD allow (192
// left to itself, nothing spilled: 512 x 512 38.1 us a step, 31.2 held; four
// wavefronts spill: 68.7). FP32 takes 92 to 102 by itself (80: 27.4 us
// against 20.6).
template <typename T, int TX, int TY, int NT>
__global__ __launch_bounds__(NT, sizeof(T) == 8 ? 3 : 1) void k_adj_tile(const T* __restrict__ rec,
                                                 const T* __restrict__ hin, T* __restrict__ hout,
                                                 double* acc_part, Coef<T> c, Geom g, int ntx) {
  __shared__ AdjTileLds<T, (TX + 8) * (TY + 8)> L;
  const int ps = (int)(g.Ns * (int64_t)sizeof(T));
  const __amdgpu_buffer_rsrc_t rrec = __builtin_amdgcn_make_buffer_rsrc((void*)rec, 0, 6 * ps, BUF_WORD3);
  const __amdgpu_buffer_rsrc_t rin = __builtin_amdgcn_make_buffer_rsrc((void*)hin, 0, 18 * ps, BUF_WORD3);
  const __amdgpu_buffer_rsrc_t rout = __builtin_amdgcn_make_buffer_rsrc((void*)hout, 0, 18 * ps, BUF_WORD3);
  double acc[4] = {0.0, 0.0, 0.0, 0.0};
  const int tile = xcd_tile(blockIdx.x, gridDim.x);
  const int ty = tile / ntx, tx = tile - ty * ntx;
  const int x0 = tx * TX, y0 = ty * TY;
  if (g.walls && (y0 - 4 <= 0 || y0 + TY + 4 >= g.ny))
    adj_tile<T, TX, TY, NT, true>(rrec, rin, rout, c, g, x0, y0, L, acc);
  else
    adj_tile<T, TX, TY, NT, false>(rrec, rin, rout, c, g, x0, y0, L, acc);
  block_add4<NT>(acc, acc_part);
}

template <typename T, int TX, int TY, int NT>
hipError_t launch(const void* rec, const void* hin, void* hout, double* part, const Coef<T>& c,
                  const Geom& g, hipStream_t s) {
  hipLaunchKernelGGL((k_adj_tile<T, TX, TY, NT>), dim3(tiles(g, TX, TY)), dim3(NT), 0, s,
                     (const T*)rec, (const T*)hin, (T*)hout, part, c, g, (g.nx + TX - 1) / TX);
  return hipGetLastError();
}

// Tile of a lattice: the smallest that covers it in one round of compute
// units, so that small lattices spread over all of them (fp64 64 x 64: 8 x 4
// 7.0 us, 16 x 4 7.3, 32 x 8 9.4; 128 x 128: 8.6, 7.6, 9.7; 256 x 256: 25.7,
// 16.3, 10.8). Beyond one round FP32 keeps 32 x 8 (512 x 512: 20.3 us; 16 x 8
// 20.7, 16 x 4 30.5) and FP64 takes 16 x 8 (31.2 us; 24 x 8 47.5, 12 x 8 36.4,
// 16 x 4 42.7).
enum Shape { T8x4, T16x4, T32x8, T16x8 };
template <typename T>
Shape shape(const Geom& g) {
  if (tiles(g, 8, 4) <= CUS) return T8x4;
  if (tiles(g, 16, 4) <= CUS) return T16x4;
  return sizeof(T) == 4 || tiles(g, 32, 8) <= CUS ? T32x8 : T16x8;
}

}  // namespace

// While both cotangent buffers and the record are about what the 256 MB
// Infinity Cache holds (us per step, tiles against the row sweep): fp64 490 k
// nodes (165 MB) 54 and 127, 810 k (272 MB) 92 and 130, 1.0 M (336 MB) 136 and 158,
// 1.2 M (407 MB) 177 and 169; fp32 934 k (157 MB) 60 and 83, 2.0 M (337 MB) 159 and
// 122. It also keeps the byte offsets in a buffer below 2^31.
template <typename T>
bool adj_tile_fits(const Geom& g) {
  return (2 * 18 + 6) * g.Ns * (int64_t)sizeof(T) <= (int64_t)(sizeof(T) == 8 ? 325 : 256) << 20;
}

// Of rows of more than 8192 columns, few fit, which give the row sweep short
// segments: it then has the shorter time where the tiles' lanes, idle ones
// included, exceed what its rounds of workgroups take (sweep and tiles: fp32
// 22 222 x 9 44 and 25, 66 666 x 9 54 and 63, 40 000 x 25 92 and 81, 52 000 x 25 92 and
// 104; fp64 35 294 x 17 106 and 77, 58 823 x 17 118 and 159).
template <typename T>
bool adj_tiles_beat_rows(const Geom& g, const AdjShape& sh) {
  const int64_t rounds = ((int64_t)sh.nstrips * sh.nseg + sh.resident - 1) / sh.resident;
  const int64_t lanes =
      sizeof(T) == 8 ? tiles(g, 16, 8) * (int64_t)128 : tiles(g, 32, 8) * (int64_t)256;
  return lanes <= (sizeof(T) == 8 ? 48000 : 74000) * rounds * (sh.seg + 3);
}

template <typename T>
int adj_tile_count(const Geom& g) {
  switch (shape<T>(g)) {
    case T8x4: return tiles(g, 8, 4);
    case T16x4: return tiles(g, 16, 4);
    case T32x8: return tiles(g, 32, 8);
    default: return tiles(g, 16, 8);
  }
}

template <typename T>
hipError_t launch_adj_tile(const void* rec, const void* hin, void* hout, double* part,
                           const Coef<T>& c, const Geom& g, hipStream_t s) {
  switch (shape<T>(g)) {
    case T8x4: return launch<T, 8, 4, 192>(rec, hin, hout, part, c, g, s);
    case T16x4: return launch<T, 16, 4, 256>(rec, hin, hout, part, c, g, s);
    case T32x8: return launch<T, 32, 8, sizeof(T) == 8 ? 512 : 448>(rec, hin, hout, part, c, g, s);
    default: break;
  }
  if constexpr (sizeof(T) == 8) return launch<T, 16, 8, 256>(rec, hin, hout, part, c, g, s);
  return hipErrorInvalidValue;
}

#define QILBM_INSTANTIATE(T)                                                                     \
  template bool adj_tile_fits<T>(const Geom&);                                                   \
  template bool adj_tiles_beat_rows<T>(const Geom&, const AdjShape&);                            \
  template int adj_tile_count<T>(const Geom&);                                                   \
  template hipError_t launch_adj_tile<T>(const void*, const void*, void*, double*,               \
                                         const Coef<T>&, const Geom&, hipStream_t);
QILBM_INSTANTIATE(double)
QILBM_INSTANTIATE(float)
#undef QILBM_INSTANTIATE

}  // namespace qilbm
