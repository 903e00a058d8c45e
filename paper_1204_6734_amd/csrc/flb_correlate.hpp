// flb_correlate.hpp — device helpers shared by the one-step and the
// several-step kernels: the collision constants of a slot and the correlator
// sums of one wavefront on the matrix cores.
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

#include "flb_device.hpp"
#include "flb_kernels.hpp"

namespace flb {

template <typename R>
__device__ __forceinline__ CollideConst<R> collide_const(const SlotDesc& sd);

template <>
__device__ __forceinline__ CollideConst<float> collide_const<float>(const SlotDesc& sd) {
  CollideConst<float> C;
  C.rho0 = sd.rho0f;
  C.ux0 = sd.ux0f;
  C.uy0 = sd.uy0f;
#pragma unroll
  for (int a = 0; a < 6; ++a) {
    C.rt[a] = sd.rtf[a];
    C.xc[a] = sd.xcf[a];
  }
  C.xc2 = sd.xc2f;
  C.one_tau = sd.one_tau;
  C.k0 = sd.k0;
  C.k1 = sd.k1;
  C.noise = sd.noise;
  return C;
}

template <>
__device__ __forceinline__ CollideConst<double> collide_const<double>(const SlotDesc& sd) {
  CollideConst<double> C;
  C.rho0 = sd.rho0;
  C.ux0 = sd.ux0;
  C.uy0 = sd.uy0;
#pragma unroll
  for (int a = 0; a < 6; ++a) {
    C.rt[a] = sd.rt[a];
    C.xc[a] = sd.xc[a];
  }
  C.xc2 = sd.xc2;
  C.one_tau = sd.one_tau;
  C.k0 = sd.k0;
  C.k1 = sd.k1;
  C.noise = sd.noise;
  return C;
}

typedef double double4_v __attribute__((ext_vector_type(4)));

// Position of statistic v in a wavefront's 16 x 16 result X^T X (row-major):
// the sum of df_i is entry (i, 9), the product df_i df_j (i <= j) entry (i, j).
struct StatPos {
  int pos[kNStat];
};
constexpr StatPos stat_positions() {
  StatPos p{};
  int q = 0;
  for (int i = 0; i < 9; ++i) p.pos[q++] = i * 16 + 9;
  for (int i = 0; i < 9; ++i)
    for (int j = i; j < 9; ++j) p.pos[q++] = i * 16 + j;
  return p;
}
static __constant__ StatPos kStatPos = stat_positions();

typedef __bf16 bf16x8_v __attribute__((ext_vector_type(8)));
typedef float float4_v __attribute__((ext_vector_type(4)));
typedef unsigned int u32x4_v __attribute__((ext_vector_type(4)));

// x = x1 + x2 + x3 exactly, each part a bfloat16 (returned as its 16 bits):
// x1 keeps the leading 8 significant bits of x (truncated), x2 the leading 8
// of what remains, x3 the rest, which has at most 8 significant bits left
// (an FP32 value has 24).  Both subtractions are exact.
__device__ __forceinline__ void split_bf16x3(float x, uint32_t p[3]) {
  const uint32_t b1 = __builtin_bit_cast(uint32_t, x) & 0xFFFF0000u;
  const float r1 = x - __builtin_bit_cast(float, b1);
  const uint32_t b2 = __builtin_bit_cast(uint32_t, r1) & 0xFFFF0000u;
  const float r2 = r1 - __builtin_bit_cast(float, b2);
  p[0] = b1 >> 16;
  p[1] = b2 >> 16;
  p[2] = __builtin_bit_cast(uint32_t, r2) >> 16;
}

// Correlator sums of df_i = f_i - f_i^0(rho0, u0) (= the stored h_i): 9
// first moments and the 45 products i <= j (row-major), added to this
// tile's open time-block partials.  For one wavefront (64 sites) these are
// the entries of X^T X, X the 64 x 10 matrix of the nine df_i and a
// constant 1 per site, a dense contraction over the sites done on the
// matrix cores; the wavefront stages its values in LDS first.
//   FP32 storage: every df_i is split exactly into three bfloat16 parts,
//   x = x1 + x2 + x3, so that x y = sum_{p,q} xp yq with every part product
//   exact in FP32; ten v_mfma_f32_16x16x32_bf16 (32 sites each; of the part
//   pairs p != q one product, returned transposed as well, the smallest pair
//   left out) accumulate the 16 x 16 result in FP32.  Operand layout:
//   lane l holds feature l % 16 of sites 8 (l / 16) .. + 7 of a group of 32
//   (the same registers serve as A and B); result row 4 (l / 16) + r,
//   column l % 16 in element r.  The products are exact and a wavefront's
//   sum of 64 sites has the rounding of FP32 additions (a few 1e-8
//   relative); all later sums are FP64.
//   FP64 storage: sixteen v_mfma_f64_16x16x4f64 (four sites each) on the
//   values themselves, lane l taking column l % 16 of site l / 16 of each
//   group of four; result row l / 16 + 4 r, column l % 16 in element r.
// The wavefront writes its 16 x 16 result (FP64) over its staged values;
// at the end of the step the four wavefronts of the tile add their results
// in a fixed order, so a tile's partial does not depend on the workgroup
// shape.
template <typename S>
constexpr int sample_wave_bytes() {
  // FP32: 3 parts x 10 values (the nine df_i and the constant) x 64 sites
  // of 2 bytes; FP64: 64 x 9 values; at least the 16 x 16 FP64 result
  return sizeof(S) == 4 ? 3 * 10 * kTileX * 2 : kTileX * 9 * 8;
}

// X^T X of one wavefront's sites.  Lane l brings the values h of the site at
// position pos of the 64 (a permutation of the lanes); lanes that are not
// `in` count as zeros, and so does every position from nsites (a multiple of
// four in effect) on.  Element r of out is row xtx_row(lane / 16, r), column
// lane % 16 of the result.  stage: sample_wave_bytes() of LDS that only this
// wavefront uses (no workgroup barrier).
template <typename S>
__device__ __forceinline__ int xtx_row(int grp, int r) {
  return sizeof(S) == 4 ? 4 * grp + r : grp + 4 * r;
}

template <typename S, typename R>
__device__ __forceinline__ void wave_xtx(const R h[9], bool in, int pos, int nsites, void* stage,
                                         double out[4]) {
  const int lane = threadIdx.x & 63;
  const int col = lane & 15, grp = lane >> 4;
  if constexpr (sizeof(S) == 4) {
    // staging [part 3][value 10][site 64] of bfloat16; value 9 is the
    // constant 1 = 1 + 0 + 0 (bfloat16 one is 0x3F80)
    unsigned short* xb = reinterpret_cast<unsigned short*>(stage);
#pragma unroll
    for (int i = 0; i < 9; ++i) {
      uint32_t pp[3];
      split_bf16x3(in ? (float)h[i] : 0.0f, pp);
#pragma unroll
      for (int q = 0; q < 3; ++q) xb[(q * 10 + i) * kTileX + pos] = (unsigned short)pp[q];
    }
    xb[9 * kTileX + lane] = 0x3F80;
    xb[19 * kTileX + lane] = 0;
    xb[29 * kTileX + lane] = 0;
    // the values come back from other lanes of the same wavefront, whose
    // LDS accesses complete in program order
    __builtin_amdgcn_wave_barrier();
    // rows 10..15 of the result are not used: those lanes read row 9
    const int colr = col < 10 ? col : 9;
    u32x4_v X[3][2];
#pragma unroll
    for (int q = 0; q < 3; ++q)
#pragma unroll
      for (int hh = 0; hh < 2; ++hh)
        X[q][hh] = *reinterpret_cast<const u32x4_v*>(xb + (q * 10 + colr) * kTileX + 32 * hh +
                                                     8 * grp);
    // B below is written over the staged values: every read above is
    // issued first (the compiler may not move the writes before them)
    asm volatile("" ::: "memory");
    // X^T X = sum over part pairs (p, q) of X_p^T X_q, and the (q, p) term is
    // the transpose of the (p, q) one: A holds the pairs p = q, B those with
    // p < q, and the sum is A + B + B^T.  The pair (2, 2) is left out: its
    // products are below 2^-30 of the others', under the rounding of the
    // FP32 accumulators.  Ten products per wavefront, in a fixed order.
    float4_v acc = {0.f, 0.f, 0.f, 0.f}, accb = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int hh = 0; hh < 2; ++hh) {
      const bf16x8_v x0 = __builtin_bit_cast(bf16x8_v, X[0][hh]);
      const bf16x8_v x1 = __builtin_bit_cast(bf16x8_v, X[1][hh]);
      const bf16x8_v x2 = __builtin_bit_cast(bf16x8_v, X[2][hh]);
      acc = __builtin_amdgcn_mfma_f32_16x16x32_bf16(x0, x0, acc, 0, 0, 0);
      accb = __builtin_amdgcn_mfma_f32_16x16x32_bf16(x0, x1, accb, 0, 0, 0);
      acc = __builtin_amdgcn_mfma_f32_16x16x32_bf16(x1, x1, acc, 0, 0, 0);
      accb = __builtin_amdgcn_mfma_f32_16x16x32_bf16(x0, x2, accb, 0, 0, 0);
      accb = __builtin_amdgcn_mfma_f32_16x16x32_bf16(x1, x2, accb, 0, 0, 0);
    }
    // B^T through LDS: B goes into the staging area past its first 2 KiB
    // (which the one-step kernel overwrites with the result) and comes back
    // transposed
    static_assert(sample_wave_bytes<S>() >= 2048 + 16 * 16 * (int)sizeof(float),
                  "B fits the staging area after the result");
    float* bt = reinterpret_cast<float*>(reinterpret_cast<char*>(stage) + 2048);
#pragma unroll
    for (int r = 0; r < 4; ++r) bt[(4 * grp + r) * 16 + col] = accb[r];
    __builtin_amdgcn_wave_barrier();
#pragma unroll
    for (int r = 0; r < 4; ++r)
      out[r] = (double)((acc[r] + accb[r]) + bt[col * 16 + 4 * grp + r]);
  } else {
    S* x = reinterpret_cast<S*>(stage);
#pragma unroll
    for (int i = 0; i < 9; ++i) x[pos * 9 + i] = in ? (S)h[i] : S(0);
    __builtin_amdgcn_wave_barrier();
    // columns 10..15 are zero and column 9 is the constant; every lane reads
    // an in-range element so that the sixteen reads issue back to back
    const int colr = col < 9 ? col : 8;
    const double pad = col == 9 ? 1.0 : 0.0;
    S xv[16];
#pragma unroll
    for (int q = 0; q < 16; ++q) xv[q] = x[(4 * q + grp) * 9 + colr];
    asm volatile("" ::: "memory");
    double4_v acc = {0.0, 0.0, 0.0, 0.0};
#pragma unroll
    for (int q = 0; q < 16; ++q) {
      // four sites that are all zeros add nothing (wave-uniform)
      if (4 * q < nsites) {
        const double val = col < 9 ? (double)xv[q] : pad;
        acc = __builtin_amdgcn_mfma_f64_16x16x4f64(val, val, acc, 0, 0, 0);
      }
    }
#pragma unroll
    for (int r = 0; r < 4; ++r) out[r] = acc[r];
  }
}

// Structure-factor fields of one site in the f-norm at (rho0, u0): d rho and
// dj~ = sqrt3 (j - u0 rho) = sqrt3 ((j - rho0 u0) - u0 (rho - rho0))  (eq. (34)),
// packed as z1 = d rho + i dj~_x, z2 = dj~_y in the storage precision.
template <typename S, typename R>
__device__ __forceinline__ void sk_fields(const R h[9], const SlotDesc& sd, uint32_t site) {
  using V = typename Cplx<S>::type;
  const uint32_t N = (uint32_t)sd.nx * (uint32_t)sd.ny;
  double hd[9];
#pragma unroll
  for (int i = 0; i < 9; ++i) hd[i] = (double)h[i];
  const Moments<double> m = hermite_moments(hd);
  V* z = reinterpret_cast<V*>(sd.skz);
  z[site] = V{(S)m.drho, (S)(1.7320508075688772935 * (m.jx - sd.ux0 * m.drho))};
  z[N + site] = V{(S)(1.7320508075688772935 * (m.jy - sd.uy0 * m.drho)), S(0)};
}

}  // namespace flb
