// flb_march.hip — two steps of large FP32 lattices in one pass over memory.
//
// On a lattice that does not fit the last-level cache the one-step kernel
// moves 72 bytes a site and step at the rate of a copy, under the board's
// power limit.  step_march_kernel reads the populations of an even time once
// and writes those two steps later: 36 bytes a site and step.  Each wavefront
// works alone, without LDS or barriers: its lanes hold 64 neighbouring columns
// and it walks down a strip of rows.  At each row it takes the first step of
// the row (site-local, on the loaded values) and, with what it kept of the two
// rows above, the second step of the row above: values that move along y wait
// in registers, values that move along x come from the neighbouring lane
// (DPP wave shifts).  The first and last lane and one row above and below the
// strip are computed for their neighbours' sake only and not stored: 64/62 and
// (H + 1)/H of the work.  The noise is keyed by (seed, step, site), so both
// copies of such a site agree and every population equals the one-step
// kernel's bit for bit.  Source and destination are two buffers, as in
// flb_multi.hip.
//
// Measured, us a step, one step per launch -> this kernel: f-norm basis 8192^2
// 845 -> 694 (79.4 -> 96.7 GLUPS), 4096^2 215 -> 183; Hermite basis 8192^2 826
// -> 507 (132 GLUPS), 4096^2 212 -> 135, 2048^2 43.8 -> 33.9, 1536^2 26.3 ->
// 18.4.  Bound by FP32 arithmetic in the f-norm basis (lattices that fit the
// cache reach 92.6 GLUPS in one step per launch); 101 vector registers leave
// four wavefronts a SIMD, five spill (8192^2: 883 us).  The row of loads for the
// next site is in flight while this one's two steps compute.  The barrier of
// each row gives 1 % there and 13 % in the Hermite basis (8192^2, 8 rows: 585 ->
// 507); workgroups of eight wavefronts gain 2 % more at 8192^2 in the Hermite
// basis and lose 5 % in the f-norm basis and below 2048^2.
#include <hip/hip_runtime.h>
#include <stdint.h>

#include "flb_buffer.hpp"
#include "flb_correlate.hpp"
#include "flb_device.hpp"
#include "flb_kernels.hpp"
#include "flb_multi.hpp"
#include "flb_runtime.hpp"

namespace flb {

// The value of the neighbouring lane: of lane l - 1 (a value moving along +x)
// or l + 1.  Lanes 0 and 63 keep their own (they are not stored).
__device__ __forceinline__ float from_left(float v) {
  const int x = __builtin_bit_cast(int, v);
  return __builtin_bit_cast(float, __builtin_amdgcn_update_dpp(x, x, 0x138, 0xF, 0xF, false));
}
__device__ __forceinline__ float from_right(float v) {
  const int x = __builtin_bit_cast(int, v);
  return __builtin_bit_cast(float, __builtin_amdgcn_update_dpp(x, x, 0x130, 0xF, 0xF, false));
}

struct MarchShape {
  int nx, ny;
  uint32_t pitch;
  int strips;                   // strips of columns
  int groups;                   // workgroups of one lattice
  uint32_t gr_magic, gr_shift;  // division by groups
  uint32_t st_magic, st_shift;  // and by strips
  int H;                        // rows of a wavefront
  int flip;                     // 1: pop2 -> pop
};

__device__ __forceinline__ void load_row(const void* src, uint32_t pitch, int y, uint32_t voff,
                                         float h[9]) {
  const __amdgpu_buffer_rsrc_t r = row_rsrc<float>(const_cast<void*>(src), pitch, y);
#pragma unroll
  for (int i = 0; i < 9; ++i) h[i] = buf_load(r, voff, (uint32_t)i * pitch * 4u, (float*)nullptr);
}

template <int BASIS>
__global__ __launch_bounds__(256) void step_march_kernel(const SlotDesc* __restrict__ slots,
                                                         const MarchShape M,
                                                         const uint64_t* __restrict__ clock,
                                                         uint32_t step_idx) {
  const uint32_t g = (uint32_t)xcd_tile(blockIdx.x, gridDim.x);
  const uint32_t slot = (uint32_t)(((uint64_t)g * M.gr_magic) >> M.gr_shift);
  // strips of one band of rows are consecutive wavefronts
  const uint32_t w = (g - slot * (uint32_t)M.groups) * 4u +
                     (uint32_t)__builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int band = (int)(((uint64_t)w * M.st_magic) >> M.st_shift);
  const int strip = (int)w - band * M.strips;
  const int nx = M.nx, ny = M.ny, y0 = band * M.H, H = min(M.H, ny - y0);
  const int rows = H > 0 ? H + 2 : 0;
  const SlotDesc& sd = slots[slot];
  const uint64_t t = sd.t0 + *clock + step_idx;
  const int lane = threadIdx.x & 63;
  // this lane's column, one to the left of the strip for lane 0, periodic;
  // lanes past the last one needed stay on it
  int x = strip * kMarchCols - 1 + lane;
  const bool stores = lane >= 1 && lane <= kMarchCols && x < nx;
  x = x < 0 ? x + nx : (x >= nx ? min(x - nx, 0) : x);
  const uint32_t voff = (uint32_t)x * 4u;
  const uint32_t vm = (uint32_t)(x == 0 ? nx - 1 : x - 1) * 4u;
  const uint32_t vp = (uint32_t)(x == nx - 1 ? 0 : x + 1) * 4u;
  const void* const src = M.flip ? sd.pop2 : sd.pop;
  void* const dst = M.flip ? sd.pop : sd.pop2;
  const CollideConst<float> C = collide_const<float>(sd);
  const uint32_t pe = M.pitch * 4u;

  int y = y0 == 0 ? ny - 1 : y0 - 1;
  float next[9];
  if (rows) load_row(src, M.pitch, y, voff, next);
  // what the first step left for rows above: of the row above (0, 1, 3) and of
  // the two above (2, 5, 6), each already moved along x
  float a0 = 0.f, a1 = 0.f, a3 = 0.f, b2 = 0.f, b5 = 0.f, b6 = 0.f, c2 = 0.f, c5 = 0.f, c6 = 0.f;
#pragma unroll 1
  for (int j = 0; j < M.H + 2; ++j) {
    // neighbouring strips in step (every wavefront of the workgroup comes here
    // M.H + 2 times; nothing is exchanged): their rows share cache lines at the
    // strips' edges, which leave the cache half written when one runs ahead
    __builtin_amdgcn_s_barrier();
    if (j >= rows) continue;
    float h[9];
#pragma unroll
    for (int i = 0; i < 9; ++i) h[i] = next[i];
    const int yn = y == ny - 1 ? 0 : y + 1;
    if (j < H + 1) load_row(src, M.pitch, yn, voff, next);
    // first step of row y
    {
      const uint32_t site = (uint32_t)y * (uint32_t)nx + (uint32_t)x;
      SiteDraw<float, false> draw;
      if (C.noise) site_draw<float, false>(C, site, t, draw);
      const int e = collide<float, BASIS>(h, C, draw);
      if (e) {
        atomicOr(sd.err, e);
        atomicMin(sd.err_step, (unsigned long long)t);
      }
    }
    const float s1 = from_left(h[1]), s5 = from_left(h[5]), s8 = from_left(h[8]);
    const float s3 = from_right(h[3]), s6 = from_right(h[6]), s7 = from_right(h[7]);
    if (j >= 2) {
      // second step of the row above
      const int Y = y == 0 ? ny - 1 : y - 1;
      const uint32_t site = (uint32_t)Y * (uint32_t)nx + (uint32_t)x;
      float f[9] = {a0, a1, c2, a3, h[4], c5, c6, s7, s8};
      SiteDraw<float, false> draw;
      if (C.noise) site_draw<float, false>(C, site, t + 1, draw);
      const int e = collide<float, BASIS>(f, C, draw);
      if (e && stores) {  // the outer lanes' second step has no neighbours' values
        atomicOr(sd.err, e);
        atomicMin(sd.err_step, (unsigned long long)(t + 1));
      }
      if (stores) {
        // the value of direction o goes to the site it moves to
        const __amdgpu_buffer_rsrc_t rc = row_rsrc<float>(dst, M.pitch, Y);
        const __amdgpu_buffer_rsrc_t rm = row_rsrc<float>(dst, M.pitch, Y == 0 ? ny - 1 : Y - 1);
        const __amdgpu_buffer_rsrc_t rp = row_rsrc<float>(dst, M.pitch, y);
#pragma unroll
        for (int o = 0; o < 9; ++o)
          buf_store(kVY[o] > 0 ? rp : (kVY[o] < 0 ? rm : rc),
                    kVX[o] > 0 ? vp : (kVX[o] < 0 ? vm : voff), (uint32_t)o * pe, f[o]);
      }
    }
    a0 = h[0];
    a1 = s1;
    a3 = s3;
    c2 = b2;
    c5 = b5;
    c6 = b6;
    b2 = h[2];
    b5 = s5;
    b6 = s6;
    y = yn;
  }
}

hipError_t launch_step_march(int basis, const SlotDesc* d_slots, int nslots, int nx, int ny,
                             int H, int flip, const uint64_t* d_clock, uint32_t step_idx,
                             hipStream_t st) {
  if (nslots <= 0) return hipSuccess;
  MarchShape M{};
  M.nx = nx;
  M.ny = ny;
  M.pitch = row_pitch(nx);
  M.strips = (nx + kMarchCols - 1) / kMarchCols;
  M.H = H;
  M.groups = (M.strips * ((ny + H - 1) / H) + 3) / 4;
  magic_div((uint32_t)M.groups, &M.gr_magic, &M.gr_shift);
  magic_div((uint32_t)M.strips, &M.st_magic, &M.st_shift);
  M.flip = flip;
  const dim3 g((unsigned)M.groups * nslots), b(256);
  switch (basis) {
    case kBasisFnormLocal:
      hipLaunchKernelGGL(step_march_kernel<kBasisFnormLocal>, g, b, 0, st, d_slots, M, d_clock,
                         step_idx);
      break;
    case kBasisHermite:
      hipLaunchKernelGGL(step_march_kernel<kBasisHermite>, g, b, 0, st, d_slots, M, d_clock,
                         step_idx);
      break;
    case kBasisFnormLut:
      hipLaunchKernelGGL(step_march_kernel<kBasisFnormLut>, g, b, 0, st, d_slots, M, d_clock,
                         step_idx);
      break;
    default:
      return hipErrorInvalidValue;
  }
  return hipGetLastError();
}

}  // namespace flb
