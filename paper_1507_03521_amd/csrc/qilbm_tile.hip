// Forward step of small and medium lattices: a workgroup owns a tile of
// TX x TY nodes and runs every stage of one step, or of two, over all its
// nodes at once, where the row-sweeping kernels (qilbm_kernels.hip) run a
// serial chain of row iterations.
//
// What bounds a small lattice is that chain: a row sweep of 16 rows and its
// warm-up takes 31 iterations of four barriers (98 us per two FP64 steps at
// 64 x 64, in four workgroups), while the lattice has work for a few
// microseconds. Here a step is four barriers:
//   A  phi over the tile and three nodes around it (pulled g),
//   B  mu over the tile and two nodes around it,
//   C  force, velocity, pressure over the tile and one node around it,
//   D  collision of the tile,
// with phi, mu and p in LDS planes and a node's populations in the registers
// of the thread that collides it. Two steps in one launch run the same
// stages twice, the first over the tile and four nodes around it; the words
// between the two steps stay in LDS, in the storage format.
//
// Threads: the first NI own the interior (the nodes that collide), the next
// NR the ring of one node around it, whose pressure needs pulled f; the
// nodes further out only need phi and mu and are shared out over all threads,
// those without an own node first, so that every stage is one round for most
// wavefronts.
#include "qilbm_internal.hpp"
#include "qilbm_rows.hpp"
#include "qilbm_tile.hpp"

namespace qilbm {

namespace {

// Byte layout of a population buffer (see Pop): offset of direction I's
// plane of f (G false) or g, its element size, and the byte of the element
// that the value starts at.
template <int P, bool G, int I>
struct PlaneOf {
  static constexpr uint32_t size = P == P_F64 ? 8 : (P == P_F32 ? 8 : (I == 0 ? (G ? 4 : 2) : 4));
  __device__ __forceinline__ static uint32_t at(uint32_t Ns) {
    if constexpr (P == P_F64) return (uint32_t)(G ? 9 + I : I) * 8u * Ns;
    else if constexpr (P == P_F32) return (uint32_t)I * 8u * Ns;
    else if constexpr (I == 0) return G ? 2u * Ns : 0u;
    else return 6u * Ns + (uint32_t)(I - 1) * 4u * Ns;
  }
};

// Reads direction I's word(s) of type S at the node's pull source, `part`
// bytes into the element. EDGE: the node may lie on a wall row, where the
// directions from beyond the wall take the node's own opposite population.
template <typename S, int P, bool G, bool EDGE, int I>
__device__ __forceinline__ S tile_pull(__amdgpu_buffer_rsrc_t rs, uint32_t Ns, const TileNode& k,
                                       uint32_t part = 0) {
  constexpr int cx = CXS(I), cy = CYS(I);
  constexpr uint32_t size = PlaneOf<P, G, I>::size;
  const uint32_t off = (k.r[1 - cy] + k.c[1 - cx]) * size + part;
  if constexpr (EDGE && cy != 0) {
    const bool wall = cy > 0 ? k.lo : k.hi;
    const uint32_t own = PlaneOf<P, G, OPP(I)>::at(Ns) + (k.r[1] + k.c[1]) * size + part;
    return buf_ld<S>(rs, wall ? own : PlaneOf<P, G, I>::at(Ns) + off, 0);
  } else {
    return buf_ld<S>(rs, off, PlaneOf<P, G, I>::at(Ns));
  }
}

// A node's whole row of words.
template <int P, bool EDGE, int I = 0>
__device__ __forceinline__ void tile_load_dirs(__amdgpu_buffer_rsrc_t rs, uint32_t Ns,
                                               const TileNode& k, Row<P>& row) {
  if constexpr (I < 9) {
    if constexpr (P == P_F64) {
      row.f[I] = tile_pull<double, P, false, EDGE, I>(rs, Ns, k);
      row.g[I] = tile_pull<double, P, true, EDGE, I>(rs, Ns, k);
    } else if constexpr (P == P_F16 && I == 0) {
      row.f0 = (uint32_t)__builtin_bit_cast(uint16_t,
                                            tile_pull<__half, P, false, EDGE, 0>(rs, Ns, k));
      row.w[0] = tile_pull<uint32_t, P, true, EDGE, 0>(rs, Ns, k);
    } else {
      row.w[I] = tile_pull<typename BufT<P>::R, P, true, EDGE, I>(rs, Ns, k);
    }
    tile_load_dirs<P, EDGE, I + 1>(rs, Ns, k, row);
  }
}

// A node's g words alone (FP32: the high word of a pair, FP16 storage: the
// high half), enough for phi.
template <int P> struct GWord { using T = double; };
template <> struct GWord<P_F32> { using T = int32_t; };
template <> struct GWord<P_F16> { using T = uint32_t; };

template <int P, bool EDGE, int I = 0>
__device__ __forceinline__ void tile_load_g(__amdgpu_buffer_rsrc_t rs, uint32_t Ns,
                                            const TileNode& k, typename GWord<P>::T w[9]) {
  if constexpr (I < 9) {
    if constexpr (P == P_F64) w[I] = tile_pull<double, P, true, EDGE, I>(rs, Ns, k);
    else if constexpr (P == P_F32) w[I] = tile_pull<int32_t, P, true, EDGE, I>(rs, Ns, k, 4);
    else w[I] = tile_pull<uint32_t, P, true, EDGE, I>(rs, Ns, k);
    tile_load_g<P, EDGE, I + 1>(rs, Ns, k, w);
  }
}

// FP64: a node's f.
template <bool EDGE, int I = 0>
__device__ __forceinline__ void tile_load_f(__amdgpu_buffer_rsrc_t rs, uint32_t Ns,
                                            const TileNode& k, double f[9]) {
  if constexpr (I < 9) {
    f[I] = tile_pull<double, P_F64, false, EDGE, I>(rs, Ns, k);
    tile_load_f<EDGE, I + 1>(rs, Ns, k, f);
  }
}

template <int P, int I = 0>
__device__ __forceinline__ int32_t g_words_q(const typename GWord<P>::T w[9]) {
  if constexpr (I < 9) {
    int32_t q;
    if constexpr (P == P_F32) q = w[I];
    else q = BufPop<P>::template q_g<I>(w[I]);
    return q + g_words_q<P, I + 1>(w);
  } else {
    return 0;
  }
}
template <int P>
__device__ __forceinline__ typename PrecT<P>::T g_words_phi(const typename GWord<P>::T w[9]) {
  using T = typename PrecT<P>::T;
  if constexpr (P == P_F64) return sum9(w);
  else return T(g_words_q<P>(w)) * T(GQI);
}

// phi as the moments and totals take it: the rounded sum of the stored values.
// FP16 storage sums its halves exactly (binary64), not as the truncated Q2.29
// contributions that a step conserves, which are up to 1.5e-8 below them.
template <int P, int I = 0>
__device__ __forceinline__ double g_words_sum(const typename GWord<P>::T w[9]) {
  if constexpr (I < 9) {
    double v;
    if constexpr (I == 0) v = double((int32_t)w[0]) * GQI_D;
    else v = double(BufPop<P>::template val_g<I>(w[I]));
    return v + g_words_sum<P, I + 1>(w);
  } else {
    return 0.0;
  }
}
template <int P>
__device__ __forceinline__ typename PrecT<P>::T moment_phi(const typename GWord<P>::T w[9]) {
  if constexpr (P == P_F16) return float(g_words_sum<P>(w));
  else return g_words_phi<P>(w);
}

// Stores a node's words at element n.
template <int P, int POL, int I = 0>
__device__ __forceinline__ void tile_store(__amdgpu_buffer_rsrc_t rs, uint32_t Ns, uint32_t n,
                                           const Row<P>& row) {
  if constexpr (I < 9) {
    if constexpr (P == P_F64) {
      buf_st<double, POL>(row.f[I], rs, n * 8u, PlaneOf<P, false, I>::at(Ns));
      buf_st<double, POL>(row.g[I], rs, n * 8u, PlaneOf<P, true, I>::at(Ns));
    } else if constexpr (P == P_F16 && I == 0) {
      buf_st<__half, POL>(__builtin_bit_cast(__half, (uint16_t)row.f0), rs, n * 2u, 0);
      buf_st<uint32_t, POL>(row.w[0], rs, n * 4u, PlaneOf<P, true, 0>::at(Ns));
    } else {
      buf_st<typename BufT<P>::R, POL>(row.w[I], rs, n * PlaneOf<P, true, I>::size,
                                  PlaneOf<P, true, I>::at(Ns));
    }
    tile_store<P, POL, I + 1>(rs, Ns, n, row);
  }
}

// Words between the two steps of a launch, direction-major over the first
// step's interior.
template <int P, int N> struct TileMid { typename BufT<P>::R w[9][N]; };
template <int N> struct TileMid<P_F64, N> { double f[9][N]; double g[9][N]; };

// Direction I's source in the intermediate words of node m (row pitch W):
// the element, and the direction whose plane holds it.
template <int P, int W, int N, bool EDGE, int I = 0>
__device__ __forceinline__ void mid_row(const TileMid<P, N>& M, int m, bool lo, bool hi,
                                        Row<P>& row) {
  if constexpr (I < 9) {
    constexpr int cx = CXS(I), cy = CYS(I);
    int e = I * N + m - cy * W - cx;
    if constexpr (EDGE && cy != 0) e = (cy > 0 ? lo : hi) ? OPP(I) * N + m : e;
    if constexpr (P == P_F64) {
      row.f[I] = (&M.f[0][0])[e];
      row.g[I] = (&M.g[0][0])[e];
    } else {
      row.w[I] = (&M.w[0][0])[e];
    }
    mid_row<P, W, N, EDGE, I + 1>(M, m, lo, hi, row);
  }
}
template <int P, int W, int N, bool EDGE, int I = 0>
__device__ __forceinline__ void mid_g(const TileMid<P, N>& M, int m, bool lo, bool hi,
                                      typename GWord<P>::T w[9]) {
  if constexpr (I < 9) {
    constexpr int cx = CXS(I), cy = CYS(I);
    int e = I * N + m - cy * W - cx;
    if constexpr (EDGE && cy != 0) e = (cy > 0 ? lo : hi) ? OPP(I) * N + m : e;
    if constexpr (P == P_F64) w[I] = (&M.g[0][0])[e];
    else w[I] = reinterpret_cast<const int32_t*>(&M.w[0][0])[2 * e + 1];
    mid_g<P, W, N, EDGE, I + 1>(M, m, lo, hi, w);
  }
}
template <int P, int N>
__device__ __forceinline__ void mid_put(TileMid<P, N>& M, int m, const Row<P>& row) {
#pragma unroll
  for (int i = 0; i < 9; ++i) {
    if constexpr (P == P_F64) {
      M.f[i][m] = row.f[i];
      M.g[i][m] = row.g[i];
    } else {
      M.w[i][m] = row.w[i];
    }
  }
}

// phi, mu and p of the largest stage, rows of PX nodes.
template <typename T, int PX, int PY>
struct TileRings {
  T phi[PY * PX];
  T mu[PY * PX];
  T p[PY * PX];
};

template <int K, int P, int N> struct MidOf { using T = TileMid<P, N>; };
template <int P, int N> struct MidOf<1, P, N> { struct T {}; };

// One step over an interior of IX x IY nodes whose corner is lattice node
// (bx, by). FROM_MID: the populations come from M (pitch and extent of the
// previous step's interior, four nodes larger on each side), else from `in`.
// TO_MID: the post-collision words go to M, else the nodes of the lattice
// (x < nx, y < ny) go to `out`. LDS element of interior node (lx, ly):
// (ly + 3) PX + lx + 3.
template <int P, int IX, int IY, int PX, int PY, int NT, int NM_, bool FROM_MID, bool TO_MID,
          bool EDGE, bool TRT, int POL, typename MID>
__device__ __forceinline__ void tile_phase(__amdgpu_buffer_rsrc_t rin, __amdgpu_buffer_rsrc_t rout,
                                           const Coef<typename PrecT<P>::T>& c, const Geom& g,
                                           int bx, int by, int ox, int TXr, int TYr,
                                           typename PrecT<P>::T* rec, bool rec_stream,
                                           TileRings<typename PrecT<P>::T, PX, PY>& L, MID& M) {
  using T = typename PrecT<P>::T;
  constexpr int NI = IX * IY, NR = frame_count<IX, IY, 1>(), NP = NI + NR;
  constexpr int NPHI = frame_count<IX + 2, IY + 2, 2>(), NMU = frame_count<IX + 2, IY + 2, 1>();
  constexpr int MW = IX + 8;          // pitch of M when FROM_MID
  static_assert(NP <= NT, "one own node per thread");
  // FP64, whose f has words of its own, loads it behind A's barrier where a
  // launch is one round of workgroups (two steps: 64 x 64 3.6 us a step, 3.45;
  // 256 x 256 6.1, 5.75): C is the first to need it, and ahead of the barrier it
  // kept phi waiting. With more workgroups to switch to, ahead is better
  // (512 x 512 15.2, 15.5).
  constexpr bool F_LATE = P == P_F64 && TO_MID;
  const int t = threadIdx.x;
  const uint32_t Ns = (uint32_t)g.Ns;
  const int slot = t >= NP ? t - NP : t + NT - NP;
  // own node
  int lx = 0, ly = 0;
  if (t < NI) {
    ly = t / IX;
    lx = t - ly * IX;
  } else if (t < NP) {
    frame_pos<IX, IY, 1>(t - NI, lx, ly);
  }
  const int e = (ly + 3) * PX + lx + 3;
  const TileNode k = tile_node(bx + lx, by + ly, g);
  const bool in_tile = t < NI && lx >= ox && lx < ox + TXr && ly >= ox && ly < ox + TYr;
  const bool owns = in_tile && bx + lx < g.nx && by + ly < g.ny;
  const int64_t n = (int64_t)k.r[1] + k.c[1];
  Row<P> row;
  T ph = T(0);
  int32_t phi_q = 0;
  // A
  if (t < NP) {
    if constexpr (FROM_MID) mid_row<P, MW, NM_, EDGE>(M, (ly + 4) * MW + lx + 4, k.lo, k.hi, row);
    else if constexpr (F_LATE) tile_load_g<P, EDGE>(rin, Ns, k, row.g);
    else tile_load_dirs<P, EDGE>(rin, Ns, k, row);
  }
  for (int h = slot; h < NPHI; h += NT) {
    int hx, hy;
    frame_pos<IX + 2, IY + 2, 2>(h, hx, hy);
    hx -= 1;
    hy -= 1;
    const TileNode kh = tile_node(bx + hx, by + hy, g);
    typename GWord<P>::T w[9];
    if constexpr (FROM_MID) mid_g<P, MW, NM_, EDGE>(M, (hy + 4) * MW + hx + 4, kh.lo, kh.hi, w);
    else tile_load_g<P, EDGE>(rin, Ns, kh, w);
    L.phi[(hy + 3) * PX + hx + 3] = g_words_phi<P>(w);
  }
  if (t < NP) {
    ph = row_phi<P>(row, phi_q);
    L.phi[e] = ph;
  }
  __syncthreads();
  if constexpr (F_LATE)
    if (t < NP) tile_load_f<EDGE>(rin, Ns, k, row.f);
  // B
  T mu = T(0);
  if (t < NP) {
    T v[3][3], gx, gy, lap;
    tile3x3<T, PX>(L.phi, e, k.lo, k.hi, v);
    stencil(v, gx, gy, lap);
    mu = mu_bulk(v[1][1], c) - c.kappa * lap;
    L.mu[e] = mu;
  }
  for (int h = slot; h < NMU; h += NT) {
    int hx, hy;
    frame_pos<IX + 2, IY + 2, 1>(h, hx, hy);
    hx -= 1;
    hy -= 1;
    const int y = by + hy;
    const int eh = (hy + 3) * PX + hx + 3;
    const bool lo = g.walls && y <= 0, hi = g.walls && y >= g.ny - 1;
    T v[3][3], gx, gy, lap;
    tile3x3<T, PX>(L.phi, eh, lo, hi, v);
    stencil(v, gx, gy, lap);
    L.mu[eh] = mu_bulk(v[1][1], c) - c.kappa * lap;
  }
  __syncthreads();
  // C
  Macro<T> m;
  T f[9], gg[9];
  if (t < NP) {
    row_unpack<P>(row, f, gg);
    T S, jx, jy;
    moments9(f, S, jx, jy);
    T v[3][3], gphx, gphy, lapphi, gmux, gmuy, lapmu;
    tile3x3<T, PX>(L.phi, e, k.lo, k.hi, v);
    stencil(v, gphx, gphy, lapphi);
    tile3x3<T, PX>(L.mu, e, k.lo, k.hi, v);
    stencil(v, gmux, gmuy, lapmu);
    macro_node(ph, mu, gphx, gphy, gmux, gmuy, lapmu, S, jx, jy, c, m);
    L.p[e] = m.p;
    if (rec && owns) {
      // two steps a launch, or stores written through: lattices too small for it
      if (POL == ST_BACK && !FROM_MID && !TO_MID && rec_stream) {
        const T v[6] = {ph, mu, m.p, S, jx, jy};
        const uint32_t pb = Ns * (uint32_t)sizeof(T);
        const __amdgpu_buffer_rsrc_t rr =
            __builtin_amdgcn_make_buffer_rsrc(rec, 0, (int)(6 * pb), BUF_WORD3);
#pragma unroll
        for (int q = 0; q < 6; ++q)
          buf_st<T, ST_STREAM>(v[q], rr, (uint32_t)n * (uint32_t)sizeof(T), q * pb);
      } else {
        rec[n] = ph;
        rec[g.Ns + n] = mu;
        rec[2 * g.Ns + n] = m.p;
        rec[3 * g.Ns + n] = S;
        rec[4 * g.Ns + n] = jx;
        rec[5 * g.Ns + n] = jy;
      }
    }
  }
  __syncthreads();
  // D
  if (t < NI) {
    T v[3][3], dpx, dpy, lapp;
    tile3x3<T, PX>(L.p, e, k.lo, k.hi, v);
    stencil(v, dpx, dpy, lapp);
    if constexpr (TRT) collide_node_trt(f, gg, m, dpx, dpy, c);
    else collide_node(f, gg, m, dpx, dpy, c);
    Row<P> o;
    row_pack<P>(f, gg, phi_q, o);
    if constexpr (TO_MID) mid_put<P, NM_>(M, ly * IX + lx, o);
    else if (owns) tile_store<P, POL>(rout, Ns, (uint32_t)n, o);
  }
}

// K steps of the lattice; tile (i, j) starts at node (i TX, j TY). Beyond the
// lattice's last column a tile goes on with the wrapped columns (computed,
// not stored); so it does beyond the last row when periodic.
// rec0, rec1: records of the states the steps start from, or null, stored as a
// stream with rec_stream. Whether and how they are written is a uniform branch and not a variant of the kernel: the
// compiler contracts multiply-adds per kernel, and a recording replay must
// reproduce the plain steps bit for bit.
template <int P, int K, int TX, int TY, int NT, bool TRT, int POL>
__global__ __launch_bounds__(NT) void k_tile(Pop<P> in, Pop<P> out, Coef<typename PrecT<P>::T> c,
                                             Geom g, int ntx, uint32_t bytes,
                                             typename PrecT<P>::T* rec0,
                                             typename PrecT<P>::T* rec1, bool rec_stream) {
  using T = typename PrecT<P>::T;
  static_assert(K == 1 || K == 2, "steps per launch");
  constexpr int O = 4 * (K - 1);                 // first step's interior beyond the tile
  constexpr int PX = TX + 2 * O + 6, PY = TY + 2 * O + 6;
  constexpr int NM_ = (TX + 2 * O) * (TY + 2 * O);
  __shared__ TileRings<T, PX, PY> L;
  __shared__ typename MidOf<K, P, NM_>::T M;
  const __amdgpu_buffer_rsrc_t rin = __builtin_amdgcn_make_buffer_rsrc(in.base, 0, (int)bytes, BUF_WORD3);
  const __amdgpu_buffer_rsrc_t rout = __builtin_amdgcn_make_buffer_rsrc(out.base, 0, (int)bytes, BUF_WORD3);
  // consecutive tiles, which share halo nodes, on one XCD
  const int tile = xcd_tile(blockIdx.x, gridDim.x);
  const int ty = tile / ntx, tx = tile - ty * ntx;
  const int x0 = tx * TX, y0 = ty * TY;
  // the wall rows are within reach of this tile's pulls (uniform)
  const bool edge = g.walls && (y0 - O - 3 <= 0 || y0 + TY + O + 3 >= g.ny);
  if constexpr (K == 2) {
    if (edge) {
      tile_phase<P, TX + 8, TY + 8, PX, PY, NT, NM_, false, true, true, TRT, POL>(
          rin, rout, c, g, x0 - 4, y0 - 4, 4, TX, TY, rec0, rec_stream, L, M);
      __syncthreads();
      tile_phase<P, TX, TY, PX, PY, NT, NM_, true, false, true, TRT, POL>(
          rin, rout, c, g, x0, y0, 0, TX, TY, rec1, rec_stream, L, M);
    } else {
      tile_phase<P, TX + 8, TY + 8, PX, PY, NT, NM_, false, true, false, TRT, POL>(
          rin, rout, c, g, x0 - 4, y0 - 4, 4, TX, TY, rec0, rec_stream, L, M);
      __syncthreads();
      tile_phase<P, TX, TY, PX, PY, NT, NM_, true, false, false, TRT, POL>(
          rin, rout, c, g, x0, y0, 0, TX, TY, rec1, rec_stream, L, M);
    }
  } else {
    if (edge)
      tile_phase<P, TX, TY, PX, PY, NT, NM_, false, false, true, TRT, POL>(
          rin, rout, c, g, x0, y0, 0, TX, TY, rec0, rec_stream, L, M);
    else
      tile_phase<P, TX, TY, PX, PY, NT, NM_, false, false, false, TRT, POL>(
          rin, rout, c, g, x0, y0, 0, TX, TY, rec0, rec_stream, L, M);
  }
}

// -------------------------------------------------- moments and totals
// State m of the thread's node of a TX x TY tile (one node per lane): phi
// over the tile and two nodes around it from the pulled g, mu over the tile
// and one node around it, force, velocity and pressure from the pulled f.
template <int P, int TX, int TY, bool EDGE>
__device__ __forceinline__ void tile_macro(__amdgpu_buffer_rsrc_t rin,
                                           const Coef<typename PrecT<P>::T>& c, const Geom& g,
                                           int x0, int y0, const TileNode& k, int lx, int ly,
                                           typename PrecT<P>::T* lphi,
                                           typename PrecT<P>::T* lmu, Row<P>& row,
                                           Macro<typename PrecT<P>::T>& m) {
  using T = typename PrecT<P>::T;
  constexpr int NT = TX * TY, PX = TX + 4;
  const int t = threadIdx.x, e = (ly + 2) * PX + lx + 2;
  const uint32_t Ns = (uint32_t)g.Ns;
  tile_load_dirs<P, EDGE>(rin, Ns, k, row);
  for (int h = t; h < frame_count<TX, TY, 2>(); h += NT) {
    int hx, hy;
    frame_pos<TX, TY, 2>(h, hx, hy);
    typename GWord<P>::T w[9];
    tile_load_g<P, EDGE>(rin, Ns, tile_node(x0 + hx, y0 + hy, g), w);
    lphi[(hy + 2) * PX + hx + 2] = moment_phi<P>(w);
  }
  int32_t phi_q = 0;
  T ph;
  if constexpr (P == P_F16) ph = moment_phi<P>(row.w);
  else ph = row_phi<P>(row, phi_q);
  lphi[e] = ph;
  __syncthreads();
  T v[3][3], gphx, gphy, lapphi, gmux, gmuy, lapmu;
  tile3x3<T, PX>(lphi, e, k.lo, k.hi, v);
  stencil(v, gphx, gphy, lapphi);
  const T mu = mu_bulk(ph, c) - c.kappa * lapphi;
  lmu[e] = mu;
  for (int h = t; h < frame_count<TX, TY, 1>(); h += NT) {
    int hx, hy;
    frame_pos<TX, TY, 1>(h, hx, hy);
    const int y = y0 + hy, eh = (hy + 2) * PX + hx + 2;
    T gx, gy, lap;
    tile3x3<T, PX>(lphi, eh, g.walls && y <= 0, g.walls && y >= g.ny - 1, v);
    stencil(v, gx, gy, lap);
    lmu[eh] = mu_bulk(v[1][1], c) - c.kappa * lap;
  }
  __syncthreads();
  T f[9], gg[9], S, jx, jy;
  row_unpack<P>(row, f, gg);
  moments9(f, S, jx, jy);
  tile3x3<T, PX>(lmu, e, k.lo, k.hi, v);
  stencil(v, gmux, gmuy, lapmu);
  macro_node(ph, mu, gphx, gphy, gmux, gmuy, lapmu, S, jx, jy, c, m);
}

// The requested moments in one pass over the populations (the three launches
// that form phi and mu as fields first read g, or its words' pairs, twice):
// with four fields 2048 x 8192 fp32 589 -> 333 us, 5.2 TB/s, fp64 732 -> 569, fp16
// 400 -> 276; on small lattices one launch instead of three.
template <int P, int TX, int TY>
__global__ __launch_bounds__(TX * TY) void k_tile_moments(Pop<P> in, MomentOut mo,
                                                          Coef<typename PrecT<P>::T> c, Geom g,
                                                          int ntx, uint32_t bytes) {
  using T = typename PrecT<P>::T;
  __shared__ T lphi[(TX + 4) * (TY + 4)];
  __shared__ T lmu[(TX + 4) * (TY + 4)];
  const __amdgpu_buffer_rsrc_t rin = __builtin_amdgcn_make_buffer_rsrc(in.base, 0, (int)bytes, BUF_WORD3);
  const int tile = xcd_tile(blockIdx.x, gridDim.x);
  const int ty = tile / ntx, tx = tile - ty * ntx;
  const int x0 = tx * TX, y0 = ty * TY;
  const int ly = threadIdx.x / TX, lx = threadIdx.x - ly * TX;
  const TileNode k = tile_node(x0 + lx, y0 + ly, g);
  Row<P> row;
  Macro<T> m;
  if (g.walls && (y0 - 2 <= 0 || y0 + TY + 2 >= g.ny))
    tile_macro<P, TX, TY, true>(rin, c, g, x0, y0, k, lx, ly, lphi, lmu, row, m);
  else
    tile_macro<P, TX, TY, false>(rin, c, g, x0, y0, k, lx, ly, lphi, lmu, row, m);
  if (x0 + lx >= g.nx || y0 + ly >= g.ny) return;
  const int64_t n = (int64_t)k.r[1] + k.c[1];
  if (mo.phi) mo.phi[n] = double(m.phi);
  if (mo.rho) mo.rho[n] = double(m.rho);
  if (mo.ux) mo.ux[n] = double(m.ux);
  if (mo.uy) mo.uy[n] = double(m.uy);
  if (mo.p) mo.p[n] = double(m.p);
  if (mo.mu) mo.mu[n] = double(m.mu);
}

// phi alone needs no neighbours: as an output (O double) or as the field that
// k_mu and k_macro read (O the compute type).
template <int P, typename O>
__global__ __launch_bounds__(256) void k_phi_out(Pop<P> in, O* __restrict__ phi, Geom g,
                                                 uint32_t bytes) {
  const __amdgpu_buffer_rsrc_t rin = __builtin_amdgcn_make_buffer_rsrc(in.base, 0, (int)bytes, BUF_WORD3);
  const int64_t n = (int64_t)xcd_tile(blockIdx.x, gridDim.x) * 256 + threadIdx.x;
  if (n >= g.N) return;
  const int y = (int)((uint32_t)n / (uint32_t)g.nx), x = (int)((uint32_t)n - (uint32_t)y * g.nx);
  typename GWord<P>::T w[9];
  tile_load_g<P, true>(rin, (uint32_t)g.Ns, tile_node(x, y, g), w);
  phi[n] = O(moment_phi<P>(w));
}

// phi of a node's words exactly, in binary64 (summed like pull_phi_exact).
template <int P, int I = 0>
__device__ __forceinline__ double row_phi_exact(const Row<P>& row) {
  if constexpr (I < 9) {
    double v;
    if constexpr (P == P_F64) v = row.g[I];
    else v = double(BufPop<P>::template q_g<I>(row.w[I])) * GQI_D;
    return v + row_phi_exact<P, I + 1>(row);
  } else {
    return 0.0;
  }
}

// Per-workgroup partials of (sum phi, sum rho, sum rho ux, sum rho uy), each
// over a contiguous share of the 32 x 8 tiles.
constexpr int MASS_TX = 32, MASS_TY = 8;
template <int P>
__global__ __launch_bounds__(256) void k_tile_mass(Pop<P> in, double* __restrict__ part,
                                                   Coef<typename PrecT<P>::T> c, double rho_B,
                                                   double drho, Geom g, int ntx, int ntiles,
                                                   uint32_t bytes) {
  using T = typename PrecT<P>::T;
  constexpr int TX = MASS_TX, TY = MASS_TY;
  __shared__ T lphi[(TX + 4) * (TY + 4)];
  __shared__ T lmu[(TX + 4) * (TY + 4)];
  const __amdgpu_buffer_rsrc_t rin = __builtin_amdgcn_make_buffer_rsrc(in.base, 0, (int)bytes, BUF_WORD3);
  const int b = xcd_tile(blockIdx.x, gridDim.x);
  const int t0 = (int)((int64_t)ntiles * b / gridDim.x);
  const int t1 = (int)((int64_t)ntiles * (b + 1) / gridDim.x);
  const int ly = threadIdx.x / TX, lx = threadIdx.x - ly * TX;
  double a[4] = {0.0, 0.0, 0.0, 0.0};
  for (int tile = t0; tile < t1; ++tile) {
    const int ty = tile / ntx, tx = tile - ty * ntx;
    const int x0 = tx * TX, y0 = ty * TY;
    const TileNode k = tile_node(x0 + lx, y0 + ly, g);
    Row<P> row;
    Macro<T> m;
    if (g.walls && (y0 - 2 <= 0 || y0 + TY + 2 >= g.ny))
      tile_macro<P, TX, TY, true>(rin, c, g, x0, y0, k, lx, ly, lphi, lmu, row, m);
    else
      tile_macro<P, TX, TY, false>(rin, c, g, x0, y0, k, lx, ly, lphi, lmu, row, m);
    if (x0 + lx < g.nx && y0 + ly < g.ny) {
      const double ph = row_phi_exact<P>(row);
      a[0] += ph;
      a[1] += rho_B + drho * ph;
      a[2] += double(m.rho) * double(m.ux);
      a[3] += double(m.rho) * double(m.uy);
    }
    __syncthreads();       // the next tile takes the LDS planes
  }
  block_sum4(a, part + 4 * blockIdx.x);
}

// Whether records are stored as a stream: where they and the two population
// buffers exceed what the Infinity Cache keeps, they would push the populations
// out of it, and a record is next read after a whole segment (us per recorded
// step, plain and as a stream: fp32 1143 x 1487 86 and 50, 1000 x 1300 44 and 39;
// fp16 1640 x 2134 132 and 81; fp64 1000 x 780 65 and 45). Below, the adjoint still
// finds them there (recorded and adjoint step, fp32 554 x 722 46 and 48).
template <int P>
bool records_stream(const Geom& g) {
  return 2 * pop_bytes(P, g.Ns) + 6 * g.Ns * (int64_t)sizeof(typename PrecT<P>::T) >
         (int64_t)190 << 20;
}

// ------------------------------------------------------------- dispatch
// Measured on MI355X (us per step, row-sweeping kernel -> tiles; fp64 / fp32
// at two steps per pass, fp16 storage at one):
//   64 x 64      49.4 -> 3.75   33.2 -> 3.17   34.3 -> 4.44
//   128 x 128    53.0 -> 4.27   35.2 -> 3.48   35.7 -> 4.52
//   256 x 256    52.8 -> 6.01   35.4 -> 4.31   35.3 -> 4.99
//   256 x 1024   53.1 -> 15.5   35.7 -> 9.0    36.1 -> 8.1
//   701 x 1333   42.1 -> 68.4   38.2 -> 25.3   39.1 -> 21.8
//   1001 x 2003  86.8 -> 182    53.1 -> 83.0   58.4 -> 43.7
// Two steps per launch pay while one round of workgroups covers the lattice:
// launches and loads are halved, and the second collision of the halo runs on
// compute units that would idle. The smallest tile that does it in one round
// is the fastest: 8 x 4 up to 64 x 128, 16 x 4 up to 128 x 128, 32 x 8 up to
// 256 x 256 (fp64, 64 x 64: 3.75, 3.96, 5.20 us; 128 x 128: 4.92, 4.27, 5.44;
// 256 x 256: 10.0, 11.2, 6.01). Beyond, the doubled halo costs more than a
// launch (256 x 1024, fp64: two steps 18.2, one 15.5) and a pair of steps is
// two launches.
template <int P, int K, int TX, int TY, int NT, bool TRT, int POL>
void launch_tile(const void* pin, void* pout, const Coef<typename PrecT<P>::T>& c, const Geom& g,
                 void* rec0, void* rec1, hipStream_t s) {
  using T = typename PrecT<P>::T;
  const Pop<P> i{(char*)pin, g.Ns}, o{(char*)pout, g.Ns};
  hipLaunchKernelGGL((k_tile<P, K, TX, TY, NT, TRT, POL>), dim3(tiles(g, TX, TY)), dim3(NT), 0, s,
                     i, o, c, g, (g.nx + TX - 1) / TX, (uint32_t)pop_bytes(P, g.Ns), (T*)rec0,
                     (T*)rec1, records_stream<P>(g));
}

// Whether the one-step kernel writes its results through. Lines that a kernel leaves
// dirty in the XCDs' L2 (4 MB each) are written back when it ends, with
// nothing to overlap that: written through, they leave as they are made (fp64
// 256 x 1024 17.1 us a step, 15.5 through; fp32 9.7, 9.0; 512 x 1024 28.6, 27.8;
// 640 x 1000 34.4 and 33.9 to 35.0: the end is a small part by then). A row that does not start on a 128-byte line has its tiles share
// lines, which then are written in parts, twice (fp64 1001 x 700 36.6, 40.0
// through; fp32 701 x 1333 25.9, 27.4), and still gains while the lattice is
// small (fp64 500 x 500 16.5, 15.0; 301 x 701 14.7, 14.3). FP16 storage, whose
// words take 4 and 2 bytes, has such rows at nx % 32 and % 64, and yet the same
// line: 560 x 560 10.2, 9.7; 400 x 1000 12.2, 11.5; 624 x 900 15.3, 15.0; 640 x 900
// 15.6, 15.1; 701 x 800 15.1, 15.4; 1333 x 400 15.1, 15.3.
bool tile_through(const Geom& g) {
  return g.N <= (g.nx % 16 == 0 ? 600000 : 300000);
}

template <int P, int K, int TX, int TY, int NT>
hipError_t launch_tile_variant(const void* pin, void* pout, const Coef<typename PrecT<P>::T>& c,
                               const Geom& g, void* rec0, void* rec1, hipStream_t s, bool trt) {
  if (trt && (rec0 || rec1)) return hipErrorInvalidValue;       // no recording TRT variant
  constexpr int THROUGH = K == 1 ? ST_THROUGH : ST_BACK;
  if (tile_through(g)) {
    if (trt) launch_tile<P, K, TX, TY, NT, true, THROUGH>(pin, pout, c, g, nullptr, nullptr, s);
    else launch_tile<P, K, TX, TY, NT, false, THROUGH>(pin, pout, c, g, rec0, rec1, s);
  } else {
    if (trt) launch_tile<P, K, TX, TY, NT, true, ST_BACK>(pin, pout, c, g, nullptr, nullptr, s);
    else launch_tile<P, K, TX, TY, NT, false, ST_BACK>(pin, pout, c, g, rec0, rec1, s);
  }
  return hipGetLastError();
}

}  // namespace

// Rows of more than 3072 columns (FP32 1.7 MB of populations in eight rows): the
// halo rows of a tile have left its XCD's L2 when the tiles below need them,
// and a lattice of few rows gives the sweep short segments, so it has the
// shorter time already at smaller sizes. The sweep takes (rows per segment +
// warm-up) for each round of its workgroups, the tiles a time by the lane,
// idle ones included; us per step, sweep and tiles: fp32 4095 x 290 44.5 and 39, x
// 341 44.6 and 45.1, x 424 45 and 55; 24 390 x 41 43 and 36, 31 707 x 41 43 and 46; 50 000 x 12 25 and 22,
// 83 333 x 12 29 and 35; 22 222 x 9 20 and 12, 66 666 x 9 24 and 26; fp16 4095 x 610
// 59 and 55; 83 333 x 12 36 and 30, 133 333 x 12 43 and 45; 200 000 x 3 20 and 30;
// fp64 40 000 x 5 21 and 18, 120 000 x 5 42 and 47, 50 000 x 12 37.5 and 37.7.
template <int P>
bool tiles_beat_rows(const Geom& g) {
  if (g.nx <= 3072) return true;
  if constexpr (P == P_F16) {
    const FusedShape sh = fused_shape<P>(g, 0, 0);
    const int64_t wgs = (int64_t)sh.nstrips * sh.nseg;
    return tiles(g, 32, 8) * (int64_t)256 <= 82000 * (sh.seg_rows + 2) * (860 + wgs) / 860;
  } else {
    constexpr int resident = P == P_F64 ? CUS : 2 * CUS;
    const FusedShape sh = fused2_shape<P>(g, 0, resident);
    const int64_t rounds = ((int64_t)sh.nstrips * sh.nseg + resident - 1) / resident;
    if constexpr (P == P_F64)
      return tiles(g, 32, 4) * (int64_t)128 <= 37000 * rounds * (sh.seg_rows + 4);
    return 2 * pop_bytes(P, g.Ns) <= (int64_t)205 << 20 &&
           tiles(g, 32, 8) * (int64_t)256 <= 66500 * rounds * (sh.seg_rows + 5);
  }
}

// Tiles while both population buffers together stay within the 256 MB
// Infinity Cache: a tile reads its halo again from L2 and beyond, which is
// cheap only there. Past it the row sweep, which moves the state once per two
// steps, is faster (us per step, row sweep against tiles): fp64 at 884 k nodes
// (254 MB) 40.1 and 44.0, at 810 k 39.8 and 40.4, at 750 k 39.6 and 38.2, at 640 k
// (184 MB) 39.4 and 33.1; fp32 pairs at 1.85 M nodes (266 MB) 44.5 and 46.4, at 1.6 M
// 44.1 and 41, single steps at 1.74 M 50 and 45; fp16 storage at 3.5 M nodes (266
// MB) 69 and 73, at 2.8 M 58 and 58, at 2.0 M 58 and 44. The limit also keeps
// every byte offset in a buffer below 2^31. steps: of a pass.
template <int P>
bool tile_fits(const Geom& g, int steps) {
  const int mib = P == P_F64 ? 220 : (P == P_F32 && steps == 1 ? 256 : 224);
  return 2 * pop_bytes(P, g.Ns) <= (int64_t)mib << 20 && tiles_beat_rows<P>(g);
}

template <int P>
int tile_steps(const Geom& g) {
  return tiles(g, 32, 8) <= CUS ? 2 : 1;
}

template <int P>
hipError_t launch_step_tile(const void* pin, void* pout, const Coef<typename PrecT<P>::T>& c,
                            const Geom& g, void* rec, hipStream_t s, bool trt) {
  // one step: small tiles spread a small lattice over more compute units;
  // a large one takes tiles with less halo. FP64 runs best in workgroups of
  // 256 (its 114 registers allow four of them per compute unit): 256 x 1024
  // 16.8 us in 32 x 4 tiles, 17.7 in 32 x 8
  if constexpr (P == P_F64) {
    if (tiles(g, 16, 4) <= CUS)
      return launch_tile_variant<P, 1, 16, 4, 128>(pin, pout, c, g, rec, nullptr, s, trt);
    return launch_tile_variant<P, 1, 32, 4, 256>(pin, pout, c, g, rec, nullptr, s, trt);
  } else {
    if (tiles(g, 16, 8) <= CUS)
      return launch_tile_variant<P, 1, 16, 8, 256>(pin, pout, c, g, rec, nullptr, s, trt);
    return launch_tile_variant<P, 1, 32, 8, 512>(pin, pout, c, g, rec, nullptr, s, trt);
  }
}

template <int P>
hipError_t launch_step2_tile(const void* pin, void* pout, const Coef<typename PrecT<P>::T>& c,
                             const Geom& g, void* rec0, void* rec1, hipStream_t s, bool trt) {
  if (tiles(g, 8, 4) <= CUS)
    return launch_tile_variant<P, 2, 8, 4, 256>(pin, pout, c, g, rec0, rec1, s, trt);
  if (tiles(g, 16, 4) <= CUS)
    return launch_tile_variant<P, 2, 16, 4, 384>(pin, pout, c, g, rec0, rec1, s, trt);
  return launch_tile_variant<P, 2, 32, 8, 832>(pin, pout, c, g, rec0, rec1, s, trt);
}

// All byte offsets of a population buffer in 32 bits.
template <int P>
bool moments_fit(const Geom& g) {
  return pop_bytes(P, g.Ns) <= (int64_t)UINT32_MAX;
}

// Tile of the moments: 64 wide ones of little halo where they are two rounds
// of workgroups and more (2048 x 8192, 64 x 16, 64 x 8, 32 x 8, 16 x 8: fp32
// 333, 358, 426, 515 us; fp64 596, 569, 631, 711), else small ones.
enum MomentShape { M16x8, M64x16, M64x8 };
template <int P>
MomentShape moment_shape(const Geom& g) {
  if (tiles(g, 64, 8) < 2 * CUS) return M16x8;
  return P == P_F32 ? M64x16 : M64x8;
}

// On a lattice of few columns most lanes of a tile have no node, and the
// kernels of a node per thread (launch_moment_fields, launch_macro) are the
// faster ones (us, tiles against them, 1 M nodes: fp64 nx = 3 247 and 41, 10 76
// and 41, 16 50 and 40, 20 41 and 41, 24 36 and 41; fp32 16 36 and 35; 200 k nodes:
// fp64 3 52 and 18, 10 18.5 and 17.5, 12 17 and 18). Up to a million lanes their
// three launches take longer than the idle lanes.
template <int P>
bool moments_tiled(const Geom& g, const MomentOut& mo) {
  if (!moments_fit<P>(g)) return false;
  if (mo.phi && !mo.rho && !mo.ux && !mo.uy && !mo.p && !mo.mu) return true;
  int64_t lanes;
  switch (moment_shape<P>(g)) {
    case M16x8: lanes = tiles(g, 16, 8) * (int64_t)128; break;
    case M64x16: lanes = tiles(g, 64, 16) * (int64_t)1024; break;
    default: lanes = tiles(g, 64, 8) * (int64_t)512; break;
  }
  return lanes <= 1200000 || 2 * lanes <= 7 * g.N;
}

template <int P, int TX, int TY>
void launch_moments_tile(const Pop<P>& in, const MomentOut& mo,
                         const Coef<typename PrecT<P>::T>& c, const Geom& g, hipStream_t s) {
  hipLaunchKernelGGL((k_tile_moments<P, TX, TY>), dim3(tiles(g, TX, TY)), dim3(TX * TY), 0, s, in,
                     mo, c, g, (g.nx + TX - 1) / TX, (uint32_t)pop_bytes(P, g.Ns));
}

template <int P, typename O>
hipError_t launch_phi(const void* pop, O* phi, const Geom& g, hipStream_t s) {
  hipLaunchKernelGGL((k_phi_out<P, O>), dim3((unsigned)((g.N + 255) / 256)), dim3(256), 0, s,
                     Pop<P>{(char*)pop, g.Ns}, phi, g, (uint32_t)pop_bytes(P, g.Ns));
  return hipGetLastError();
}

template <int P>
hipError_t launch_moments(const void* pop, const MomentOut& mo,
                          const Coef<typename PrecT<P>::T>& c, const Geom& g, hipStream_t s) {
  const Pop<P> in{(char*)pop, g.Ns};
  if (mo.phi && !mo.rho && !mo.ux && !mo.uy && !mo.p && !mo.mu)
    return launch_phi<P>(pop, mo.phi, g, s);
  switch (moment_shape<P>(g)) {
    case M16x8: launch_moments_tile<P, 16, 8>(in, mo, c, g, s); break;
    case M64x16: launch_moments_tile<P, 64, 16>(in, mo, c, g, s); break;
    default: launch_moments_tile<P, 64, 8>(in, mo, c, g, s); break;
  }
  return hipGetLastError();
}

// Totals likewise, from 400 thousand lanes on (us, tiles against a node per
// thread, fp64: 1 M nodes, nx = 3 158 and 70, 8 81 and 70, 10 71 and 70, 12 65
// and 70; 200 k, 3 58 and 40, 10 41 and 40; 40 k, 3 35 and 33, 4 32 and 35).
bool mass_tiled(const Geom& g) {
  const int64_t lanes = tiles(g, MASS_TX, MASS_TY) * (int64_t)(MASS_TX * MASS_TY);
  return lanes <= 400000 || lanes <= 3 * g.N;
}

// Workgroups of the totals kernel, one partial each.
int mass_blocks(const Geom& g) {
  const int64_t n = mass_tiled(g) ? tiles(g, MASS_TX, MASS_TY) : (g.N + 255) / 256;
  return n < MASS_BLOCKS ? (int)n : MASS_BLOCKS;
}

template <int P>
hipError_t launch_mass_tiles(const void* pop, double* part, const Coef<typename PrecT<P>::T>& c,
                             const Coef<double>& c64, const Geom& g, hipStream_t s) {
  const Pop<P> in{(char*)pop, g.Ns};
  hipLaunchKernelGGL(k_tile_mass<P>, dim3(mass_blocks(g)), dim3(256), 0, s, in, part, c, c64.rho_B,
                     c64.drho, g, (g.nx + MASS_TX - 1) / MASS_TX, tiles(g, MASS_TX, MASS_TY),
                     (uint32_t)pop_bytes(P, g.Ns));
  return hipGetLastError();
}

#define QILBM_INSTANTIATE(P)                                                                     \
  template bool tile_fits<P>(const Geom&, int);                                                  \
  template bool moments_fit<P>(const Geom&);                                                     \
  template bool moments_tiled<P>(const Geom&, const MomentOut&);                                 \
  template hipError_t launch_phi<P, PrecT<P>::T>(const void*, PrecT<P>::T*, const Geom&,         \
                                                 hipStream_t);                                   \
  template hipError_t launch_moments<P>(const void*, const MomentOut&,                           \
                                        const Coef<PrecT<P>::T>&, const Geom&, hipStream_t);     \
  template hipError_t launch_mass_tiles<P>(const void*, double*, const Coef<PrecT<P>::T>&,       \
                                           const Coef<double>&, const Geom&, hipStream_t);       \
  template hipError_t launch_step_tile<P>(const void*, void*, const Coef<PrecT<P>::T>&,          \
                                          const Geom&, void*, hipStream_t, bool);

QILBM_INSTANTIATE(P_F64)
QILBM_INSTANTIATE(P_F32)
QILBM_INSTANTIATE(P_F16)
#undef QILBM_INSTANTIATE

#define QILBM_INSTANTIATE2(P)                                                                    \
  template int tile_steps<P>(const Geom&);                                                       \
  template hipError_t launch_step2_tile<P>(const void*, void*, const Coef<PrecT<P>::T>&,         \
                                           const Geom&, void*, void*, hipStream_t, bool);

QILBM_INSTANTIATE2(P_F64)
QILBM_INSTANTIATE2(P_F32)
#undef QILBM_INSTANTIATE2

}  // namespace qilbm
