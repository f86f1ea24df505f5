// Node indexing of the tiled kernels of small lattices (forward and adjoint).
#pragma once

#include "qilbm_device.hpp"

namespace qilbm {

// Where one node's populations come from: element offsets of the rows
// y - 1, y, y + 1 and columns x - 1, x, x + 1 (periodic), and whether the
// node lies on the bottom (lo) or top (hi) wall row.
struct TileNode {
  uint32_t r[3], c[3];
  bool lo, hi;
};

// Node (x, y) given by coordinates that may lie up to 8 nodes outside the
// lattice (nx, ny >= 3). Columns wrap. Rows wrap when periodic; beyond a wall
// they are clamped to the wall row (such a node's values are never read).
__device__ __forceinline__ TileNode tile_node(int x, int y, const Geom& g) {
  TileNode k;
  const unsigned nx = (unsigned)g.nx, ny = (unsigned)g.ny;
  const unsigned xw = (unsigned)(x + 3 * g.nx) % nx;
  k.c[0] = xw == 0 ? nx - 1 : xw - 1;
  k.c[1] = xw;
  k.c[2] = xw == nx - 1 ? 0 : xw + 1;
  unsigned yw;
  if (g.walls) yw = (unsigned)(y < 0 ? 0 : (y >= g.ny ? g.ny - 1 : y));
  else yw = (unsigned)(y + 3 * g.ny) % ny;
  k.lo = g.walls && yw == 0;
  k.hi = g.walls && yw == ny - 1;
  k.r[0] = (yw == 0 ? ny - 1 : yw - 1) * nx;
  k.r[1] = yw * nx;
  k.r[2] = (yw == ny - 1 ? 0 : yw + 1) * nx;
  return k;
}

// Position h of the frame of D nodes around a W x H core: the D rows above,
// the D rows below, then D + D columns of the core's rows.
template <int W, int H, int D>
__device__ __forceinline__ void frame_pos(int h, int& lx, int& ly) {
  constexpr int RW = W + 2 * D, BAND = D * RW;
  if (h < 2 * BAND) {
    const int q = h / RW;
    lx = h - q * RW - D;
    ly = q < D ? q - D : H + q - D;
  } else {
    h -= 2 * BAND;
    ly = h / (2 * D);
    const int k = h - ly * (2 * D);
    lx = k < D ? k - D : W + k - D;
  }
}
template <int W, int H, int D>
__host__ __device__ constexpr int frame_count() {
  return (W + 2 * D) * (H + 2 * D) - W * H;
}

// 3x3 neighbourhood of element e; beyond a wall the mirrored row is e's own.
template <typename T, int PX>
__device__ __forceinline__ void tile3x3(const T* a, int e, bool lo, bool hi, T v[3][3]) {
  const int em = lo ? e : e - PX, ep = hi ? e : e + PX;
#pragma unroll
  for (int d = -1; d <= 1; ++d) {
    v[0][d + 1] = a[em + d];
    v[1][d + 1] = a[e + d];
    v[2][d + 1] = a[ep + d];
  }
}


// Tiles of tx x ty nodes that cover the lattice.
inline int tiles(const Geom& g, int tx, int ty) {
  const int64_t n = ((int64_t)(g.nx + tx - 1) / tx) * ((g.ny + ty - 1) / ty);
  return n > INT32_MAX ? INT32_MAX : (int)n;
}

}  // namespace qilbm
