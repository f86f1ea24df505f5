// Kernels of the three-dimensional step over tiles of TX x TY x TZ nodes
// (included by qilbm3d.hip). One thread per node of the tile; the fields whose
// neighbours a stage needs are staged in LDS over the tile and the nodes
// around it.
//
// Three launches a step (every FP64 lattice but the smallest, FP32 ones that
// the z-sweep kernel has too few columns for): k3_tile_phi, k3_tile_f (mu, the
// pressure and f's collision), k3_tile_g. Each population set is pulled once
// for its collision, g once more for phi. Bound by memory (the Infinity Cache
// up to about 64^3 in FP64) at some 900 bytes a node in FP64: 64^3 44 us,
// 256^3 2.91 ms = 5.2 TB/s. The row-wave kernels that it replaces, which
// gathered every stencil through L1 and formed mu in a launch of its own,
// took 80 us and 3.17 ms, and 51 us against 16 at 32^3: there the mu launch
// was eight workgroups, 36 us.
//
// Small lattices are bound by launches and their latency, a few us each, so
// they take fewer: k3_tile_step makes the whole step, with phi from
// k3_tile_phi or, smaller still, pulled over the tile's halo as well.
#pragma once

namespace qilbm3 {

// One node's neighbourhood as byte offsets inside a plane of words of WS
// bytes: columns x - 1, x, x + 1, rows y - 1, y, y + 1 (periodic) and layers
// z - 1, z, z + 1 (periodic, or clamped to the wall layer); lo, hi: the layer
// below / above lies beyond a wall.
struct TNode {
  uint32_t xo[3], yo[3], zo[3];
  bool lo, hi;
};

// (x, y, z) may lie any number of periods outside the lattice; beyond a wall
// z is clamped to the wall layer.
template <int WS>
__device__ __forceinline__ TNode tnode(int x, int y, int z, const Geom3& g) {
  TNode k;
  const uint32_t row = (uint32_t)g.nx * WS, layer = row * (uint32_t)g.ny;
  x = wrapm(x, g.nx);
  y = wrapm(y, g.ny);
  z = g.walls ? min(max(z, 0), g.nz - 1) : wrapm(z, g.nz);
  const bool b = z == 0, t = z + 1 == g.nz;
  k.xo[0] = (uint32_t)(x == 0 ? g.nx - 1 : x - 1) * WS;
  k.xo[1] = (uint32_t)x * WS;
  k.xo[2] = (uint32_t)(x + 1 == g.nx ? 0 : x + 1) * WS;
  k.yo[0] = (uint32_t)(y == 0 ? g.ny - 1 : y - 1) * row;
  k.yo[1] = (uint32_t)y * row;
  k.yo[2] = (uint32_t)(y + 1 == g.ny ? 0 : y + 1) * row;
  k.lo = g.walls && b;
  k.hi = g.walls && t;
  k.zo[0] = (uint32_t)(b ? (g.walls ? 0 : g.nz - 1) : z - 1) * layer;
  k.zo[1] = (uint32_t)z * layer;
  k.zo[2] = (uint32_t)(t ? (g.walls ? z : 0) : z + 1) * layer;
  return k;
}

__device__ __forceinline__ uint32_t tself(const TNode& k) {
  return k.xo[1] + k.yo[1] + k.zo[1];
}

// The pre-collision word of population I at node k. EDGE: the node may lie on
// a wall layer, where the directions from beyond the wall take the node's own
// opposite population.
template <typename S, bool BIG, bool EDGE, int I>
__device__ __forceinline__ S tpull(const Planes<S, BIG>& v, const TNode& k) {
  constexpr int cz = CZ(I);
  S w = v.ldb(I, 0, k.xo[1 - CX(I)] + k.yo[1 - CY(I)] + k.zo[1 - cz]);
  if constexpr (EDGE && cz != 0) {
    if (cz > 0 ? k.lo : k.hi) w = v.ldb(OPP(I), 0, tself(k));
  }
  return w;
}

template <typename S, bool BIG, bool EDGE, int I = 0>
__device__ __forceinline__ void tpull_all(const Planes<S, BIG>& v, const TNode& k, S w[19]) {
  if constexpr (I < 19) {
    w[I] = tpull<S, BIG, EDGE, I>(v, k);
    tpull_all<S, BIG, EDGE, I + 1>(v, k, w);
  }
}

// phi of a node from its pulled g words (in direction order).
template <int P, bool BIG, bool EDGE>
__device__ __forceinline__ typename PrecT<P>::T tphi(const PopView<P, BIG>& v, const TNode& k) {
  using T = typename PrecT<P>::T;
  using GW = typename PopView<P, BIG>::GW;
  GW w[19];
  tpull_all<GW, BIG, EDGE>(v.g, k, w);
  GW s = w[0];
#pragma unroll
  for (int i = 1; i < 19; ++i) s += w[i];
  if constexpr (FixedG<P>::value) return T(s) * T(GQI);
  else return s;
}

// Tile (tx, ty, tz) of the launch. The launch of a BIG lattice has two dimensions
// (tile_grid) and may have workgroups beyond the last tile: theirs starts beyond
// the lattice (z0 >= nz).
struct TileAt {
  int x0, y0, z0;
};
template <bool BIG, int TX, int TY, int TZ>
__device__ __forceinline__ TileAt tile_at(const Geom3& g) {
  const int ntx = (g.nx + TX - 1) / TX, nty = (g.ny + TY - 1) / TY;
  // consecutive tiles, which share halo nodes, on one XCD
  int b, nb = (int)gridDim.x;
  if constexpr (BIG) {
    b = (int)(blockIdx.y * gridDim.x + blockIdx.x);
    nb *= (int)gridDim.y;
  } else {
    b = (int)blockIdx.x;
  }
  b = xcd_tile(b, nb);
  const int tz = b / (ntx * nty), r = b - tz * (ntx * nty);
  const int ty = r / ntx, tx = r - ty * ntx;
  return {tx * TX, ty * TY, tz * TZ};
}
template <int TX, int TY, int TZ>
inline int64_t tile_count(const Geom3& g) {
  return (int64_t)((g.nx + TX - 1) / TX) * ((g.ny + TY - 1) / TY) * ((g.nz + TZ - 1) / TZ);
}

// Grid of n workgroups of t lanes: a launch holds less than 2^32 lanes in a
// dimension, which a BIG lattice three nodes wide exceeds (13 idle lanes for
// three; FP32 3 x 5 x 34 million).
inline dim3 tile_grid(int64_t n, int t) {
  const int64_t rows = n * t / ((int64_t)1 << 31) + 1;
  return dim3((unsigned)((n + rows - 1) / rows), (unsigned)rows);
}

// A tile shape, with the addressing of populations beyond 4 GiB or without.
template <bool BIG, int TX, int TY, int TZ>
struct Tile3 {
  static constexpr bool big = BIG;
  static constexpr int x = TX, y = TY, z = TZ, n = TX * TY * TZ;
  static dim3 grid(const Geom3& g) {
    const int64_t c = tile_count<TX, TY, TZ>(g);
    return BIG ? tile_grid(c, n) : dim3((unsigned)c);
  }
};

// LDS region: the tile and H nodes around it.
template <int TX, int TY, int TZ, int H>
struct Reg3 {
  static constexpr int W = TX + 2 * H, HT = TY + 2 * H, D = TZ + 2 * H, A = W * HT * D;
  __device__ __forceinline__ static int at(int lx, int ly, int lz) {
    return ((lz + H) * HT + ly + H) * W + lx + H;
  }
  __device__ __forceinline__ static void pos(int r, int& lx, int& ly, int& lz) {
    lz = r / (W * HT);
    r -= lz * (W * HT);
    ly = r / W;
    lx = r - ly * W - H;
    ly -= H;
    lz -= H;
  }
};

// A wall layer is the tile's own or one of the H layers around it (uniform).
template <int TZ>
__device__ __forceinline__ bool tile_edge(const TileAt& o, int H, const Geom3& g) {
  return g.walls && (o.z0 <= H || o.z0 + TZ + H >= g.nz);
}

template <typename T>
__device__ __forceinline__ void moments19(const T f[19], T& S, T j[3]) {
  S = f[0];
  j[0] = j[1] = j[2] = T(0);
#pragma unroll
  for (int i = 1; i < 19; ++i) {
    S += f[i];
    if (CX(i) != 0) j[0] += T(CX(i)) * f[i];
    if (CY(i) != 0) j[1] += T(CY(i)) * f[i];
    if (CZ(i) != 0) j[2] += T(CZ(i)) * f[i];
  }
}

// Gradient and Laplacian at tile position (lx, ly, lz) of a staged region.
template <typename T, typename R>
__device__ __forceinline__ void tile_stencil(const T* q, int lx, int ly, int lz, T& c0, T gr[3],
                                             T& lap) {
  q += R::at(lx, ly, lz);
  lds_stencil<T, R::W>(q - R::W * R::HT, q, q + R::W * R::HT, 0, c0, gr[0], gr[1], gr[2], lap);
}

// mu at a tile position from the staged phi; beyond a wall that of the wall
// layer.
template <typename T, typename R>
__device__ __forceinline__ T tile_mu(const T* lphi, const TileAt& o, int hx, int hy, int hz,
                                     const Coef3<T>& c, const Geom3& g) {
  if (g.walls) hz = min(max(o.z0 + hz, 0), g.nz - 1) - o.z0;
  T c0, gr[3], lap;
  tile_stencil<T, R>(lphi, hx, hy, hz, c0, gr, lap);
  return mu_bulk(c0, c.c) - c.c.kappa * lap;
}

// The words of a node's g as values, and their Q2.29 sum (FP32).
template <int P, typename GW, typename T>
__device__ __forceinline__ int32_t g_values(const GW gw[19], T gg[19]) {
  int32_t q = 0;
#pragma unroll
  for (int i = 0; i < 19; ++i) {
    if constexpr (FixedG<P>::value) {
      q += gw[i];
      gg[i] = float(gw[i]) * GQI;
    } else {
      gg[i] = gw[i];
    }
  }
  return q;
}

// Stores a node's collided g; in FP32 g_0 closes the node's Q2.29 sum at the
// pulled total q.
template <int POL, int P, bool BIG, typename T>
__device__ __forceinline__ void g_store(const PopView<P, BIG>& w, uint32_t n, const T gg[19],
                                        int32_t q) {
  if constexpr (FixedG<P>::value) {
    int32_t rest = 0;
#pragma unroll
    for (int i = 1; i < 19; ++i) {
      const int32_t word = __float2int_rn(gg[i] * GQ);
      rest += word;
      w.g.template stb<POL>(i, 0, n, word);
    }
    w.g.template stb<POL>(0, 0, n, q - rest);
  } else {
#pragma unroll
    for (int i = 0; i < 19; ++i) w.g.template stb<POL>(i, 0, n, gg[i]);
  }
}

template <int POL, int P, bool BIG, typename T>
__device__ __forceinline__ void f_store(const PopView<P, BIG>& w, uint32_t n, const T f[19]) {
#pragma unroll
  for (int i = 0; i < 19; ++i) w.f.template stb<POL>(i, 0, n, f[i]);
}

// Order parameter over the tiles.
template <int P, bool BIG, int TX, int TY, int TZ>
__global__ __launch_bounds__(TX * TY * TZ) void k3_tile_phi(Pop3<P> in,
                                                            typename PrecT<P>::T* __restrict__ phi,
                                                            Geom3 g) {
  using T = typename PrecT<P>::T;
  constexpr int WS = sizeof(T);
  const PopView<P, BIG> v(in);
  const Planes<T, false> out(phi, g.Ns, 1);
  const TileAt o = tile_at<BIG, TX, TY, TZ>(g);
  const int t = threadIdx.x, lx = t % TX, ly = t / TX % TY, lz = t / (TX * TY);
  const int x = o.x0 + lx, y = o.y0 + ly, z = o.z0 + lz;
  if (x >= g.nx || y >= g.ny || z >= g.nz) return;
  const TNode k = tnode<WS>(x, y, z, g);
  T ph;
  if (tile_edge<TZ>(o, 0, g)) ph = tphi<P, BIG, true>(v, k);
  else ph = tphi<P, BIG, false>(v, k);
  out.stb(0, 0, tself(k), ph);
}

// phi over the tile and two nodes around it into lphi, mu over the tile and
// one node around it into lmu; then the state m of the thread's node k at
// tile position (lx, ly, lz) from its f and the stencils of both. f is pulled
// (pull) behind phi's staging: ahead of it, its 19 loads stood before phi's in
// the queue of the address unit (FP64 128^3 374 us a step, 360 behind; 256^3
// 2964, 2910; 65 x 130 x 130 244, 235).
template <int P, int TX, int TY, int TZ, typename PF>
__device__ __forceinline__ void tile_state(const PF& pull,
                                           const Planes<typename PrecT<P>::T, false>& phf,
                                           const TileAt& o, int lx, int ly, int lz,
                                           const Coef3<typename PrecT<P>::T>& c, const Geom3& g,
                                           typename PrecT<P>::T* lphi, typename PrecT<P>::T* lmu,
                                           typename PrecT<P>::T f[19],
                                           typename PrecT<P>::T j[3],
                                           Node3<typename PrecT<P>::T>& m) {
  using T = typename PrecT<P>::T;
  constexpr int NT = TX * TY * TZ;
  using R2 = Reg3<TX, TY, TZ, 2>;
  using R1 = Reg3<TX, TY, TZ, 1>;
#pragma unroll 2
  for (int r = threadIdx.x; r < R2::A; r += NT) {
    int hx, hy, hz;
    R2::pos(r, hx, hy, hz);
    lphi[r] = phf.ldb(0, 0, tself(tnode<sizeof(T)>(o.x0 + hx, o.y0 + hy, o.z0 + hz, g)));
  }
  __syncthreads();
  pull();
  for (int r = threadIdx.x; r < R1::A; r += NT) {
    int hx, hy, hz;
    R1::pos(r, hx, hy, hz);
    lmu[r] = tile_mu<T, R2>(lphi, o, hx, hy, hz, c, g);
  }
  __syncthreads();
  T S;
  moments19(f, S, j);
  T ph, m0, gph[3], gmu[3], lapphi, lapmu;
  tile_stencil<T, R2>(lphi, lx, ly, lz, ph, gph, lapphi);
  tile_stencil<T, R1>(lmu, lx, ly, lz, m0, gmu, lapmu);
  macro3<T>(ph, m0, gph, gmu, lapmu, S, j, c, m);
}

// Second launch of a step: force, velocity and pressure of the tile and f's
// collision, which needs no grad p. Writes f, mu, p and j, which the third
// launch needs. 117 registers in FP64: two 512-lane workgroups per CU.
template <int P, bool BIG, bool TRT, int POL, int TX, int TY, int TZ>
__global__ __launch_bounds__(TX * TY * TZ) void k3_tile_f(
    Pop3<P> in, Pop3<P> out, const typename PrecT<P>::T* __restrict__ phi,
    typename PrecT<P>::T* __restrict__ mu, typename PrecT<P>::T* __restrict__ p,
    typename PrecT<P>::T* __restrict__ jx, typename PrecT<P>::T* __restrict__ jy,
    typename PrecT<P>::T* __restrict__ jz, Coef3<typename PrecT<P>::T> c, Geom3 g) {
  using T = typename PrecT<P>::T;
  __shared__ T lphi[Reg3<TX, TY, TZ, 2>::A];
  __shared__ T lmu[Reg3<TX, TY, TZ, 1>::A];
  const PopView<P, BIG> v(in), w(out);
  const TileAt o = tile_at<BIG, TX, TY, TZ>(g);
  if (BIG && o.z0 >= g.nz) return;
  const int t = threadIdx.x, lx = t % TX, ly = t / TX % TY, lz = t / (TX * TY);
  const int x = o.x0 + lx, y = o.y0 + ly, z = o.z0 + lz;
  const TNode k = tnode<sizeof(T)>(x, y, z, g);
  T f[19], j[3];
  const auto pull = [&] {
    if (tile_edge<TZ>(o, 0, g)) tpull_all<T, BIG, true>(v.f, k, f);
    else tpull_all<T, BIG, false>(v.f, k, f);
  };
  Node3<T> m;
  tile_state<P, TX, TY, TZ>(pull, Planes<T, false>(phi, g.Ns, 1), o, lx, ly, lz, c, g, lphi, lmu, f, j,
                            m);
  if (x >= g.nx || y >= g.ny || z >= g.nz) return;
  const uint32_t n = tself(k);
  const Planes<T, false> mf(mu, g.Ns, 1), pf(p, g.Ns, 1);
  const Planes<T, false> jf[3] = {{jx, g.Ns, 1}, {jy, g.Ns, 1}, {jz, g.Ns, 1}};
  mf.stb(0, 0, n, m.mu);
  pf.stb(0, 0, n, m.p);
#pragma unroll
  for (int a = 0; a < 3; ++a) jf[a].stb(0, 0, n, j[a]);
  const T dp0[3] = {T(0), T(0), T(0)};
  T gd[19];
#pragma unroll
  for (int i = 0; i < 19; ++i) gd[i] = T(0);
  if constexpr (TRT) collide3_trt<T>(f, gd, m, dp0, c.c);
  else collide3<T>(f, gd, m, dp0, c.c);
  f_store<POL>(w, n, f);
}

// The requested moments (binary64 fields) of the tile.
template <int P, bool BIG, int TX, int TY, int TZ>
__global__ __launch_bounds__(TX * TY * TZ) void k3_tile_macro(
    Pop3<P> in, const typename PrecT<P>::T* __restrict__ phi, MomentOut3 mo,
    Coef3<typename PrecT<P>::T> c, Geom3 g) {
  using T = typename PrecT<P>::T;
  __shared__ T lphi[Reg3<TX, TY, TZ, 2>::A];
  __shared__ T lmu[Reg3<TX, TY, TZ, 1>::A];
  const PopView<P, BIG> v(in);
  const TileAt o = tile_at<BIG, TX, TY, TZ>(g);
  if (BIG && o.z0 >= g.nz) return;
  const int t = threadIdx.x, lx = t % TX, ly = t / TX % TY, lz = t / (TX * TY);
  const int x = o.x0 + lx, y = o.y0 + ly, z = o.z0 + lz;
  const TNode k = tnode<sizeof(T)>(x, y, z, g);
  T f[19], j[3];
  const auto pull = [&] {
    if (tile_edge<TZ>(o, 0, g)) tpull_all<T, BIG, true>(v.f, k, f);
    else tpull_all<T, BIG, false>(v.f, k, f);
  };
  Node3<T> m;
  tile_state<P, TX, TY, TZ>(pull, Planes<T, false>(phi, g.Ns, 1), o, lx, ly, lz, c, g, lphi, lmu, f, j,
                            m);
  if (x >= g.nx || y >= g.ny || z >= g.nz) return;
  const uint32_t n = tself(k) / sizeof(T);
  if (mo.phi) mo.phi[n] = double(m.phi);
  if (mo.rho) mo.rho[n] = double(m.rho);
  for (int a = 0; a < 3; ++a)
    if (mo.u[a]) mo.u[a][n] = double(m.u[a]);
  if (mo.p) mo.p[n] = double(m.p);
  if (mo.mu) mo.mu[n] = double(m.mu);
}

// Third launch of a step: collides g of the tile with grad p (p staged in LDS
// over the tile and one node around it, like mu), u and F re-formed from j
// and grad mu as the second launch formed them.
template <int P, bool BIG, int POL, int TX, int TY, int TZ>
__global__ __launch_bounds__(TX * TY * TZ) void k3_tile_g(
    Pop3<P> in, Pop3<P> out, const typename PrecT<P>::T* __restrict__ phi,
    const typename PrecT<P>::T* __restrict__ mu, const typename PrecT<P>::T* __restrict__ p,
    const typename PrecT<P>::T* __restrict__ jx, const typename PrecT<P>::T* __restrict__ jy,
    const typename PrecT<P>::T* __restrict__ jz, Coef3<typename PrecT<P>::T> c, Geom3 g) {
  using T = typename PrecT<P>::T;
  using GW = typename PopView<P, BIG>::GW;
  constexpr int WS = sizeof(T), NT = TX * TY * TZ;
  using R1 = Reg3<TX, TY, TZ, 1>;
  __shared__ T lmu[R1::A];
  __shared__ T lp[R1::A];
  const PopView<P, BIG> v(in), w(out);
  const Planes<T, false> phf(phi, g.Ns, 1), mf(mu, g.Ns, 1), pf(p, g.Ns, 1);
  const Planes<T, false> jf[3] = {{jx, g.Ns, 1}, {jy, g.Ns, 1}, {jz, g.Ns, 1}};
  const TileAt o = tile_at<BIG, TX, TY, TZ>(g);
  if (BIG && o.z0 >= g.nz) return;
  const int t = threadIdx.x, lx = t % TX, ly = t / TX % TY, lz = t / (TX * TY);
  const int x = o.x0 + lx, y = o.y0 + ly, z = o.z0 + lz;
  const bool owns = x < g.nx && y < g.ny && z < g.nz;
  const TNode k = tnode<WS>(x, y, z, g);
  const uint32_t n = tself(k);
  const bool edge = tile_edge<TZ>(o, 0, g);
  for (int r = t; r < R1::A; r += NT) {
    int hx, hy, hz;
    R1::pos(r, hx, hy, hz);
    const uint32_t h = tself(tnode<WS>(o.x0 + hx, o.y0 + hy, o.z0 + hz, g));
    lmu[r] = mf.ldb(0, 0, h);
    lp[r] = pf.ldb(0, 0, h);
  }
  GW gw[19];
  if (edge) tpull_all<GW, BIG, true>(v.g, k, gw);
  else tpull_all<GW, BIG, false>(v.g, k, gw);
  const T j[3] = {jf[0].ldb(0, 0, n), jf[1].ldb(0, 0, n), jf[2].ldb(0, 0, n)};
  const T ph = phf.ldb(0, 0, n);
  __syncthreads();
  if (!owns) return;
  T gg[19];
  const int32_t q = g_values<P>(gw, gg);
  T m0, gmu[3], lapmu, p0, dp[3], lapp;
  tile_stencil<T, R1>(lmu, lx, ly, lz, m0, gmu, lapmu);
  tile_stencil<T, R1>(lp, lx, ly, lz, p0, dp, lapp);
  // g's collision does not use grad phi, D and the pressure
  const T gph[3] = {T(0), T(0), T(0)};
  Node3<T> m;
  macro3<T>(ph, m0, gph, gmu, T(0), T(0), j, c, m);
  T fd[19];
#pragma unroll
  for (int i = 0; i < 19; ++i) fd[i] = T(0);
  collide3<T>(fd, gg, m, dp, c.c);
  g_store<POL>(w, n, gg, q);
}

// Position r of the shell of one node around the tile: the two layers below
// and above it, then the frames of its own layers.
template <int TX, int TY, int TZ>
__device__ __forceinline__ void shell_pos(int r, int& lx, int& ly, int& lz) {
  constexpr int W = TX + 2, HT = TY + 2, LAYER = W * HT, FRAME = 2 * W + 2 * TY;
  if (r < 2 * LAYER) {
    const int b = r >= LAYER ? 1 : 0;
    r -= b * LAYER;
    lz = b ? TZ : -1;
    ly = r / W;
    lx = r - ly * W - 1;
    ly -= 1;
  } else {
    r -= 2 * LAYER;
    lz = r / FRAME;
    r -= lz * FRAME;
    if (r < 2 * W) {
      const int b = r >= W ? 1 : 0;
      lx = r - b * W - 1;
      ly = b ? TY : -1;
    } else {
      r -= 2 * W;
      ly = r >> 1;
      lx = (r & 1) ? TX : -1;
    }
  }
}

// A whole step: phi over the tile and three nodes around it, mu over two, the
// pressure over one, then both collisions. PULL: phi is pulled over the halo,
// and the step is one launch; else it is read, and k3_tile_phi runs first.
// Bound by latency: pulled loads, three barriers, and in the halo of a
// 4 x 4 x 4 tile 15 times its own phi. 16^3 11.0 us a step in FP64 (three
// launches 15.8), 32^3 14.2 with k3_tile_phi (16.8).
template <int P, bool BIG, bool TRT, bool PULL, int TX, int TY, int TZ, int NT>
__global__ __launch_bounds__(NT) void k3_tile_step(
    Pop3<P> in, Pop3<P> out, const typename PrecT<P>::T* __restrict__ phi,
    Coef3<typename PrecT<P>::T> c, Geom3 g) {
  using T = typename PrecT<P>::T;
  using GW = typename PopView<P, BIG>::GW;
  constexpr int WS = sizeof(T), NI = TX * TY * TZ;
  using R3 = Reg3<TX, TY, TZ, 3>;
  using R2 = Reg3<TX, TY, TZ, 2>;
  using R1 = Reg3<TX, TY, TZ, 1>;
  static_assert(R1::A <= NT, "one node of the tile and its shell per thread");
  __shared__ T lphi[R3::A];
  __shared__ T lmu[R2::A];
  __shared__ T lp[R1::A];
  const PopView<P, BIG> v(in), w(out);
  const Planes<T, false> phf(phi, g.Ns, 1);
  const TileAt o = tile_at<BIG, TX, TY, TZ>(g);
  const int t = threadIdx.x;
  int lx = 0, ly = 0, lz = 0;
  if (t < NI) {
    lx = t % TX;
    ly = t / TX % TY;
    lz = t / (TX * TY);
  } else if (t < R1::A) {
    shell_pos<TX, TY, TZ>(t - NI, lx, ly, lz);
  }
  const TNode k = tnode<WS>(o.x0 + lx, o.y0 + ly, o.z0 + lz, g);
  const bool edge = tile_edge<TZ>(o, 3, g);
  T f[19];
  GW gw[19];
  if (t < R1::A) {
    if (edge) tpull_all<T, BIG, true>(v.f, k, f);
    else tpull_all<T, BIG, false>(v.f, k, f);
  }
  if (t < NI) {
    if (edge) tpull_all<GW, BIG, true>(v.g, k, gw);
    else tpull_all<GW, BIG, false>(v.g, k, gw);
  }
  for (int r = t; r < R3::A; r += NT) {
    int hx, hy, hz;
    R3::pos(r, hx, hy, hz);
    if (PULL && (unsigned)hx < TX && (unsigned)hy < TY && (unsigned)hz < TZ) continue;
    const TNode h = tnode<WS>(o.x0 + hx, o.y0 + hy, o.z0 + hz, g);
    if constexpr (!PULL) lphi[r] = phf.ldb(0, 0, tself(h));
    else if (edge) lphi[r] = tphi<P, BIG, true>(v, h);
    else lphi[r] = tphi<P, BIG, false>(v, h);
  }
  if (PULL && t < NI) {
    GW s = gw[0];
#pragma unroll
    for (int i = 1; i < 19; ++i) s += gw[i];
    if constexpr (FixedG<P>::value) lphi[R3::at(lx, ly, lz)] = T(s) * T(GQI);
    else lphi[R3::at(lx, ly, lz)] = s;
  }
  __syncthreads();
  for (int r = t; r < R2::A; r += NT) {
    int hx, hy, hz;
    R2::pos(r, hx, hy, hz);
    lmu[r] = tile_mu<T, R3>(lphi, o, hx, hy, hz, c, g);
  }
  __syncthreads();
  Node3<T> m;
  if (t < R1::A) {
    T S, j[3], ph, m0, gph[3], gmu[3], lapphi, lapmu;
    moments19(f, S, j);
    tile_stencil<T, R3>(lphi, lx, ly, lz, ph, gph, lapphi);
    tile_stencil<T, R2>(lmu, lx, ly, lz, m0, gmu, lapmu);
    macro3<T>(ph, m0, gph, gmu, lapmu, S, j, c, m);
    lp[R1::at(lx, ly, lz)] = m.p;
  }
  __syncthreads();
  const int x = o.x0 + lx, y = o.y0 + ly, z = o.z0 + lz;
  if (t >= NI || x >= g.nx || y >= g.ny || z >= g.nz) return;
  constexpr int LAYER = R1::W * R1::HT;
  const int e = R1::at(lx, ly, lz);
  T p0, dp[3], lapp;
  lds_stencil<T, R1::W>(lp + (k.lo ? 0 : -LAYER), lp, lp + (k.hi ? 0 : LAYER), e, p0, dp[0],
                        dp[1], dp[2], lapp);
  T gg[19];
  const int32_t q = g_values<P>(gw, gg);
  if constexpr (TRT) collide3_trt<T>(f, gg, m, dp, c.c);
  else collide3<T>(f, gg, m, dp, c.c);
  const uint32_t n = tself(k);
  f_store<ST_BACK>(w, n, f);
  g_store<ST_BACK>(w, n, gg, q);
}

}  // namespace qilbm3
