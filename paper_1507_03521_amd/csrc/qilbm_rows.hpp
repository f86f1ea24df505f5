// Storage words of population rows and the buffer-resource access to them,
// shared by the forward kernels: raw word types, descriptors, decoding and
// packing of a node's nine f and nine g.
#pragma once

#include "qilbm_device.hpp"

namespace qilbm {

template <typename T>
__device__ __forceinline__ void moments9(const T f[9], T& S, T& jx, T& jy) {
  S = f[0];
#pragma unroll
  for (int i = 1; i < 9; ++i) S += f[i];
  jx = (f[1] - f[3]) + ((f[5] - f[6]) + (f[8] - f[7]));
  jy = (f[2] - f[4]) + ((f[5] + f[6]) - (f[7] + f[8]));
}

template <typename T>
__device__ __forceinline__ T sum9(const T v[9]) {
  T s = v[0];
#pragma unroll
  for (int i = 1; i < 9; ++i) s += v[i];
  return s;
}

// Population access of the fused kernel through buffer resources: one
// descriptor each for the f planes, the g_0 plane and the g_1..8 planes.
// The plane and row parts of an address are uniform over a wavefront and go
// into the scalar offset; the lane's column is one of three precomputed
// byte offsets (x - 1, x, x + 1). Loads beyond a descriptor's range return 0.
// Loads return the raw storage word (R), decoded only where the value is
// first used, so that a prefetched load is not waited for early.

template <int P> struct BufT;
template <> struct BufT<P_F64> { using F = double; using G0 = double; using GR = double; using R = double; };
// FP32: GR is the 64-bit word that holds f_i (low word, binary32) and g_i
// (high word, Q2.29), i = 0..8.
template <> struct BufT<P_F32> { using F = float; using G0 = int32_t; using GR = uint64_t; using R = uint64_t; };
// FP16 storage: F is the f_0 plane's binary16; GR the 32-bit word that holds
// f_i (low half) and g_i (high half), i >= 1.
template <> struct BufT<P_F16> { using F = __half; using G0 = int32_t; using GR = uint32_t; using R = uint32_t; };

// BIG: a group of population planes (f_0..8 or g_1..8) spans 4 GiB or more,
// beyond the 32-bit range of one descriptor (fused_big); every access then
// builds a descriptor for its own plane (scalar work only) and the scalar
// offset holds the row alone.
template <int P, bool BIG = false>
struct BufPop {
  using T = typename PrecT<P>::T;
  using F = typename BufT<P>::F;
  using G0 = typename BufT<P>::G0;
  using GR = typename BufT<P>::GR;
  using R = typename BufT<P>::R;
  // paired layouts: FP32 keeps (f_i, g_i) in one 64-bit word for i = 0..8,
  // FP16 storage in one 32-bit word for i = 1..8
  static constexpr bool PAIRED = P != P_F64;
  static constexpr int G_FIRST = P == P_F32 ? 0 : 1;   // first direction of the g group
  __amdgpu_buffer_rsrc_t rf, rg0, rgr;
  uint32_t pf, pg;     // plane strides (bytes) of the f and g (or pair) planes
  char *fp, *gp;       // first f plane and first g (or pair) plane

  __device__ __forceinline__ void init(const Pop<P>& p) {
    const int64_t Ns = p.Ns;
    char* b = p.base;
    char *f, *g0, *gr;
    if constexpr (P == P_F16) {
      f = b;
      g0 = b + 2 * Ns;
      gr = b + 6 * Ns;
    } else if constexpr (P == P_F32) {
      f = b;
      g0 = b;
      gr = b;
    } else {
      f = b;
      g0 = b + 9 * Ns * (int64_t)sizeof(T);
      gr = b + 10 * Ns * (int64_t)sizeof(T);
    }
    fp = f;
    gp = gr;
    pf = (uint32_t)(Ns * sizeof(F));
    pg = (uint32_t)(Ns * sizeof(GR));
    rg0 = __builtin_amdgcn_make_buffer_rsrc(g0, 0, (int)(Ns * sizeof(G0)), BUF_WORD3);
    if constexpr (!BIG) {
      rf = __builtin_amdgcn_make_buffer_rsrc(f, 0, (int)((P == P_F16 ? 1 : 9) * (int64_t)pf),
                                             BUF_WORD3);
      rgr = __builtin_amdgcn_make_buffer_rsrc(gr, 0, (int)((9 - G_FIRST) * (int64_t)pg), BUF_WORD3);
    }
  }
  template <typename S>
  __device__ __forceinline__ static R raw(S v) {
    if constexpr (sizeof(S) == 8) return v;
    else if constexpr (sizeof(S) == 4) return __builtin_bit_cast(uint32_t, v);
    else return (uint32_t)__builtin_bit_cast(uint16_t, v);
  }
  // descriptor and scalar offset of f_I / g_I (I >= 1) at element row elem_row
  template <int I>
  __device__ __forceinline__ __amdgpu_buffer_rsrc_t f_rsrc() const {
    if constexpr (BIG) return __builtin_amdgcn_make_buffer_rsrc(fp + (int64_t)I * pf, 0, (int)pf, BUF_WORD3);
    else return rf;
  }
  template <int I>
  __device__ __forceinline__ uint32_t f_soff(uint32_t elem_row) const {
    return (BIG ? 0u : I * pf) + elem_row * (uint32_t)sizeof(F);
  }
  template <int I>
  __device__ __forceinline__ __amdgpu_buffer_rsrc_t g_rsrc() const {
    if constexpr (BIG) return __builtin_amdgcn_make_buffer_rsrc(gp + (int64_t)(I - G_FIRST) * pg, 0, (int)pg, BUF_WORD3);
    else return rgr;
  }
  template <int I>
  __device__ __forceinline__ uint32_t g_soff(uint32_t elem_row) const {
    return (BIG ? 0u : (I - G_FIRST) * pg) + elem_row * (uint32_t)sizeof(GR);
  }
  // raw word of f_I (G = false) or g_I (G = true) at element (row, col[dx+1])
  template <bool G, int I>
  __device__ __forceinline__ R ld(uint32_t elem_row, const uint32_t col[3], int dx) const {
    if constexpr (P == P_F32 || (P == P_F16 && I >= 1)) {
      // the pair word of direction I (f_I low part, g_I high part)
      return buf_ld<GR>(g_rsrc<I>(), col[dx + 1] * (uint32_t)sizeof(GR), g_soff<I>(elem_row));
    } else if constexpr (!G) {
      return raw(buf_ld<F>(f_rsrc<I>(), col[dx + 1] * (uint32_t)sizeof(F), f_soff<I>(elem_row)));
    } else if constexpr (I == 0) {
      return raw(buf_ld<G0>(rg0, col[dx + 1] * (uint32_t)sizeof(G0),
                            elem_row * (uint32_t)sizeof(G0)));
    } else {
      return raw(buf_ld<GR>(g_rsrc<I>(), col[dx + 1] * (uint32_t)sizeof(GR), g_soff<I>(elem_row)));
    }
  }
  // decoded values of raw words
  template <int I>
  __device__ __forceinline__ static T val_f(R w) {
    if constexpr (P == P_F64) return w;
    else if constexpr (P == P_F32) return __builtin_bit_cast(float, (uint32_t)w);
    else return __half2float(__builtin_bit_cast(__half, (uint16_t)w)) * H_INV(I);
  }
  template <int I>
  __device__ __forceinline__ static T val_g(R w) {
    if constexpr (P == P_F64) return w;
    else if constexpr (P == P_F32) return float((int32_t)(uint32_t)(w >> 32)) * GQI;
    else if constexpr (I == 0) return float((int32_t)w) * GQI;
    else return __half2float(__builtin_bit_cast(__half, (uint16_t)(w >> 16))) * H_INV(I);
  }
  // Q2.29 contribution of a raw g word (fixed-point modes)
  template <int I>
  __device__ __forceinline__ static int32_t q_g(R w) {
    if constexpr (P == P_F32) return (int32_t)(uint32_t)(w >> 32);
    else if constexpr (I == 0) return (int32_t)w;
    else return q_half(__builtin_bit_cast(__half, (uint16_t)(w >> 16)), I);
  }
  template <int I>
  __device__ __forceinline__ void st_f(T v, uint32_t elem_row, uint32_t col) const {
    F w;
    if constexpr (P == P_F16) w = __float2half_rn(v * H_SCALE(I));
    else w = v;
    buf_st<F>(w, f_rsrc<I>(), col * (uint32_t)sizeof(F), f_soff<I>(elem_row));
  }
  // stores g_I (I >= 1); returns its Q2.29 contribution in the fixed-point modes
  template <int I>
  __device__ __forceinline__ int32_t st_g(T v, uint32_t elem_row, uint32_t col) const {
    const uint32_t so = g_soff<I>(elem_row);
    if constexpr (P == P_F64) {
      buf_st<GR>(v, g_rsrc<I>(), col * (uint32_t)sizeof(GR), so);
      return 0;
    } else if constexpr (P == P_F32) {
      const int32_t q = __float2int_rn(v * GQ);
      buf_st<GR>(q, g_rsrc<I>(), col * (uint32_t)sizeof(GR), so);
      return q;
    } else {
      const __half h = __float2half_rn(v * H_SCALE(I));
      buf_st<GR>(h, g_rsrc<I>(), col * (uint32_t)sizeof(GR), so);
      return q_half(h, I);
    }
  }
  // paired layouts: stores f_I and g_I as one word; returns the Q2.29
  // contribution of the stored g_I (FP32: I = 1..8; FP16 storage: I >= 1)
  template <int I>
  __device__ __forceinline__ int32_t st_pair(T fv, T gv, uint32_t elem_row, uint32_t col) const {
    if constexpr (P == P_F32) {
      const int32_t q = __float2int_rn(gv * GQ);
      st_pair_q<I>(fv, q, elem_row, col);
      return q;
    }
    const __half hf = __float2half_rn(fv * H_SCALE(I));
    const __half hg = __float2half_rn(gv * H_SCALE(I));
    const uint32_t w = (uint32_t)__builtin_bit_cast(uint16_t, hf) |
                       ((uint32_t)__builtin_bit_cast(uint16_t, hg) << 16);
    buf_st<GR>(w, g_rsrc<I>(), col * (uint32_t)sizeof(GR), g_soff<I>(elem_row));
    return q_half(hg, I);
  }
  // FP32: stores f_I and the Q2.29 word q of g_I as one 64-bit word
  template <int I>
  __device__ __forceinline__ void st_pair_q(T fv, int32_t q, uint32_t elem_row, uint32_t col) const {
    const uint64_t w = (uint64_t)__builtin_bit_cast(uint32_t, fv) | ((uint64_t)(uint32_t)q << 32);
    buf_st<GR>(w, g_rsrc<I>(), col * (uint32_t)sizeof(GR), g_soff<I>(elem_row));
  }
  __device__ __forceinline__ void st_g0(T v, int32_t q, uint32_t elem_row, uint32_t col) const {
    if constexpr (P == P_F64) buf_st<G0>(v, rg0, col * (uint32_t)sizeof(G0), elem_row * (uint32_t)sizeof(G0));
    else buf_st<G0>(q, rg0, col * (uint32_t)sizeof(G0), elem_row * (uint32_t)sizeof(G0));
  }
};

// FP16 storage: exact Q2.29 sum of a pulled row's g (raw words left intact)
template <int P, int I = 0>
__device__ __forceinline__ int32_t qsum_g(const typename BufT<P>::R w[9]) {
  if constexpr (I < 9) return BufPop<P>::template q_g<I>(w[I]) + qsum_g<P, I + 1>(w);
  else return 0;
}
// FP16 storage: f (low halves, f_0 from its own word) and g (high halves,
// g_0 Q2.29) of a pulled row
template <int P, int I = 0>
__device__ __forceinline__ void unpack_row(const typename BufT<P>::R w[9],
                                           typename BufT<P>::R f0w, typename PrecT<P>::T f[9],
                                           typename PrecT<P>::T g[9]) {
  if constexpr (I < 9) {
    f[I] = BufPop<P>::template val_f<I>((I == 0 && P == P_F16) ? f0w : w[I]);
    g[I] = BufPop<P>::template val_g<I>(w[I]);
    unpack_row<P, I + 1>(w, f0w, f, g);
  }
}

// The storage words of one row at one lane, as loaded from memory or pulled
// from the ring: FP32 the nine (f_i, g_i) pair words; FP16 storage the g_0
// word and the eight pair words, plus the f_0 half; FP64 the nine f and the
// nine g values.
template <int P> struct Row {
  typename BufT<P>::R w[9];
  typename BufT<P>::R f0;
};
template <> struct Row<P_F64> {
  double f[9];
  double g[9];
};

// Format of the state between the two steps: the storage format, except
// for FP16 storage, whose intermediate state stays in the FP32 format
// (binary32 f, Q2.29 g with the exact g_0 closure): the binary16
// conversions of a ring in the storage format made that kernel
// arithmetic-bound, and the state is rounded to binary16 once per pass.
template <int P> struct MidP { static constexpr int value = P; };
template <> struct MidP<P_F16> { static constexpr int value = P_F32; };

// Storage words of a node's post-collision populations (fixed-point modes):
// what store_row writes, g_0 closing the node's Q2.29 sum at phi_q.
template <int P>
__device__ __forceinline__ void pack_row(const typename PrecT<P>::T f[9],
                                         const typename PrecT<P>::T gg[9], int32_t phi_q,
                                         typename BufT<P>::R w[9], typename BufT<P>::R& f0w) {
  int32_t rest = 0;
  if constexpr (P == P_F32) {
#pragma unroll
    for (int i = 1; i < 9; ++i) {
      const int32_t q = __float2int_rn(gg[i] * GQ);
      rest += q;
      w[i] = (uint64_t)__builtin_bit_cast(uint32_t, f[i]) | ((uint64_t)(uint32_t)q << 32);
    }
    w[0] = (uint64_t)__builtin_bit_cast(uint32_t, f[0]) |
           ((uint64_t)(uint32_t)(phi_q - rest) << 32);
    f0w = 0;
  } else {
    f0w = (uint32_t)__builtin_bit_cast(uint16_t, __float2half_rn(f[0] * H_SCALE(0)));
#pragma unroll
    for (int i = 1; i < 9; ++i) {
      const __half hf = __float2half_rn(f[i] * H_SCALE(i));
      const __half hg = __float2half_rn(gg[i] * H_SCALE(i));
      rest += q_half(hg, i);
      w[i] = (uint32_t)__builtin_bit_cast(uint16_t, hf) |
             ((uint32_t)__builtin_bit_cast(uint16_t, hg) << 16);
    }
    w[0] = (uint32_t)(phi_q - rest);
  }
}

// phi of a row (and, in the fixed-point modes, its exact Q2.29 sum q), as
// the one-step kernel forms it.
template <int P>
__device__ __forceinline__ typename PrecT<P>::T row_phi(const Row<P>& row, int32_t& q) {
  using T = typename PrecT<P>::T;
  if constexpr (P == P_F64) {
    q = 0;
    return sum9(row.g);
  } else {
    q = qsum_g<P>(row.w);
    return T(q) * T(GQI);
  }
}

template <int P>
__device__ __forceinline__ void row_unpack(const Row<P>& row, typename PrecT<P>::T f[9],
                                           typename PrecT<P>::T g[9]) {
  if constexpr (P == P_F64) {
#pragma unroll
    for (int i = 0; i < 9; ++i) {
      f[i] = row.f[i];
      g[i] = row.g[i];
    }
  } else {
    unpack_row<P>(row.w, row.f0, f, g);
  }
}

template <int P>
__device__ __forceinline__ void row_pack(const typename PrecT<P>::T f[9],
                                         const typename PrecT<P>::T g[9], int32_t phi_q,
                                         Row<P>& row) {
  if constexpr (P == P_F64) {
#pragma unroll
    for (int i = 0; i < 9; ++i) {
      row.f[i] = f[i];
      row.g[i] = g[i];
    }
  } else {
    pack_row<P>(f, g, phi_q, row.w, row.f0);
  }
}

// Sum of a wave's values (lane 0), and of four values over a workgroup of 256
// lanes into out[0..3], in a fixed order.
__device__ __forceinline__ double wave_sum(double v) {
#pragma unroll
  for (int off = 32; off > 0; off >>= 1) v += __shfl_down(v, off, 64);
  return v;
}

__device__ __forceinline__ void block_sum4(double a[4], double* out) {
  __shared__ double red[4][4];
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
#pragma unroll
  for (int k = 0; k < 4; ++k) a[k] = wave_sum(a[k]);
  if (lane == 0) {
#pragma unroll
    for (int k = 0; k < 4; ++k) red[wave][k] = a[k];
  }
  __syncthreads();
  if (threadIdx.x < 4) {
    const int k = threadIdx.x;
    out[k] = (red[0][k] + red[1][k]) + (red[2][k] + red[3][k]);
  }
}

}  // namespace qilbm
