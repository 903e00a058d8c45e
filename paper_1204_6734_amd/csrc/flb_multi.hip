// flb_multi.hip — several steps of small lattices in one launch.
//
// A step of a small lattice takes about 3 us (21^2 to 256^2, FP32) of which
// the arithmetic is a third: the rest is the launch, the descriptor and
// population loads and the write-back at the kernel's end.  step_multi_kernel
// takes K steps (K even, starting at an even time) per launch: a workgroup
// loads its tiles with a halo of K - 1 sites, keeps the populations in LDS,
// and computes the halo redundantly, one site less per step, so that no two
// workgroups exchange anything in between.  The noise is keyed by (seed,
// step, site), so a halo site gets the same values as in the workgroup that
// owns it, and every population equals the one-step kernel's bit for bit.
//
// In LDS the populations follow the in-place two-phase pattern of the
// one-step kernel (even step: own nine values, written back reversed; odd
// step: reversed values of the neighbours, written forward), so a step needs
// one workgroup barrier and no second LDS buffer.  The first step takes its
// values straight from memory, the last (odd) one stores straight to memory,
// streamed.  Source and destination are two buffers (SlotDesc::pop, pop2):
// a workgroup still reads halo sites that another one has already finished.
#include <hip/hip_runtime.h>
#include <stdint.h>

#include <algorithm>

#include "flb_buffer.hpp"
#include "flb_correlate.hpp"
#include "flb_device.hpp"
#include "flb_kernels.hpp"
#include "flb_multi.hpp"
#include "flb_runtime.hpp"

namespace flb {

// Row stride of the LDS populations: 64 columns and up to three halo columns
// on each side.  Value i of (row, column) at ((9 row + i) kRS + column), so
// that the nine values and the neighbours' rows are immediate offsets of one
// of three addresses (columns x - 1, x, x + 1).
constexpr int kRS = kTileX + 2 * (kMultiMaxHalo);
constexpr int kXtxVals = 90;  // rows 0..8, columns 0..9 of a wavefront's X^T X

// Position of statistic v among those.
struct XtxPos {
  int pos[kNStat];
};
constexpr XtxPos xtx_positions() {
  XtxPos p{};
  int q = 0;
  for (int i = 0; i < 9; ++i) p.pos[q++] = i * 10 + 9;
  for (int i = 0; i < 9; ++i)
    for (int j = i; j < 9; ++j) p.pos[q++] = i * 10 + j;
  return p;
}
static __constant__ XtxPos kXtxPos = xtx_positions();

// The collision's constants, read again in each step by scalar loads (the
// empty asm keeps them from moving out of the loop): held through the loop
// they and its other scalars spilled into vector registers.
typedef const SlotDesc __attribute__((address_space(4))) * ConstSlot;
template <typename R>
__device__ __forceinline__ CollideConst<R> step_const(const SlotDesc* p) {
  asm volatile("" : "+s"(p));
  ConstSlot sd = (ConstSlot)p;
  CollideConst<R> C;
  constexpr bool f32 = sizeof(R) == 4;
  C.rho0 = f32 ? (R)sd->rho0f : (R)sd->rho0;
  C.ux0 = f32 ? (R)sd->ux0f : (R)sd->ux0;
  C.uy0 = f32 ? (R)sd->uy0f : (R)sd->uy0;
#pragma unroll
  for (int a = 0; a < 6; ++a) {
    C.rt[a] = f32 ? (R)sd->rtf[a] : (R)sd->rt[a];
    C.xc[a] = f32 ? (R)sd->xcf[a] : (R)sd->xc[a];
  }
  C.xc2 = f32 ? (R)sd->xc2f : (R)sd->xc2;
  C.one_tau = sd->one_tau;
  C.k0 = sd->k0;
  C.k1 = sd->k1;
  C.noise = sd->noise;
  return C;
}

// A site's Gaussian draw in LDS, value v at z[v plane]: as it is, or for the
// draws made in FP32 (an FP64 collision on FP32 storage) in FP32.  The
// collision reads it where it scales it, not before: held in registers from
// the start of a step it made the FP64 collision spill.
template <typename S, typename R>
struct LdsDraw {
  using type = R;
  static constexpr int n = 9;
  R* z;
  int plane;
  __device__ __forceinline__ void put(const SiteDraw<R, false>& d) const {
#pragma unroll
    for (int k = 0; k < 3; ++k) z[k * plane] = d.l[k];
#pragma unroll
    for (int k = 0; k < 6; ++k) z[(3 + k) * plane] = d.cs[k];
  }
  __device__ __forceinline__ SiteDraw<R, false> get() const {
    SiteDraw<R, false> d;
#pragma unroll
    for (int k = 0; k < 3; ++k) d.l[k] = z[k * plane];
#pragma unroll
    for (int k = 0; k < 6; ++k) d.cs[k] = z[(3 + k) * plane];
    return d;
  }
};
template <>
struct LdsDraw<float, double> {
  using type = float;
  static constexpr int n = 6;
  float* z;
  int plane;
  __device__ __forceinline__ void put(const SiteDraw<double, true>& d) const {
#pragma unroll
    for (int k = 0; k < 6; ++k) z[k * plane] = (float)d.n[k];
  }
  __device__ __forceinline__ SiteDraw<double, true> get() const {
    SiteDraw<double, true> d;
#pragma unroll
    for (int k = 0; k < 6; ++k) d.n[k] = (double)z[k * plane];
    return d;
  }
};
template <typename S, typename R>
__device__ __forceinline__ void scaled_noise(const LdsDraw<S, R>& d, R rho, R N[6]) {
  asm volatile("" ::: "memory");  // not earlier
  scaled_noise(d.get(), rho, N);
}

// What a launch's workgroups have in common, worked out on the host (divisions
// and a chain of dependent descriptor loads took 1300 cycles of every launch).
struct MultiShape {
  int nx, ny, tiles_x;
  uint32_t pitch;
  int groups;                    // workgroups of one lattice
  uint32_t gr_magic, gr_shift;   // division by groups
  uint32_t tx_magic, tx_shift;   // and by tiles_x
  int K;
  int ncw, nnw;                  // colliding and drawing wavefronts
  int rpw;                       // lattice rows of a wavefront (nx <= 64)
  uint32_t nx_magic;             // lane / nx = (lane nx_magic) >> 16
  uint32_t rpw_magic;            // row / rpw likewise
  int flip;                      // 1: pop2 -> pop
};

// Whether Gaussians are drawn by wavefronts of their own: in FP64, where they
// are two fifths of the arithmetic; in FP32 the exchange through LDS cost as
// much as it took off the chain (21 x 21: 1.99 us a step against 1.78).
template <typename R>
constexpr bool draws_apart() {
  return sizeof(R) == 8;
}

// Workgroup: one tile of 64 x 4 sites (all of the lattice's columns when nx <=
// 64, then without an x halo: the columns wrap in LDS).  FP64 collisions are
// taken on such lattices only.
// One thread per site of the region, fixed for all steps: on rows of more
// than 64 sites wavefront w < rows takes the 64 columns of region row w (the
// same 64 sites as a wavefront of the one-step kernel, so that the
// correlator sums come out alike) and the wavefronts after them the halo
// columns of all rows; on narrower lattices a wavefront takes 64 / nx rows.
// These wavefronts alone are one or two per SIMD, and a lone wavefront issues
// one instruction in about 8 cycles (two share the SIMD at full rate), so the
// work is spread over more of them: with FP64 collisions further wavefronts
// draw the Gaussians of step s + 1 into LDS while step s collides (the first
// step's are drawn by its own threads while the loads are in flight), and with
// SAMPLE one wavefront per tile row forms the correlator sums of step s during
// step s + 1, from the pre-collision values the others leave in LDS.
template <typename S, typename R, int BASIS, bool SAMPLE>
__global__ __launch_bounds__((multi_max_threads<R>())) void step_multi_kernel(
    const SlotDesc* __restrict__ slots, const MultiShape M, const uint64_t* __restrict__ clock,
    uint32_t step_idx) {
  extern __shared__ __attribute__((aligned(16))) unsigned char multi_lds[];
  const int K = M.K, ncw = M.ncw, H = K - 1, nx = M.nx, ny = M.ny;
  const uint32_t g = (uint32_t)xcd_tile(blockIdx.x, gridDim.x);
  const uint32_t slot = (uint32_t)(((uint64_t)g * M.gr_magic) >> M.gr_shift);
  const uint32_t lg = g - slot * (uint32_t)M.groups;
  const int gy = (int)(((uint64_t)lg * M.tx_magic) >> M.tx_shift);
  const int tx = (int)lg - gy * M.tiles_x;
  const SlotDesc& sd = slots[slot];
  const uint64_t t0 = sd.t0 + *clock + step_idx;
  const bool full = draws_apart<R>() || nx <= kTileX;
  const int x0 = tx * kTileX, y0 = gy * kTileY;
  const int TH = min(kTileY, ny - y0);
  const int W = min(kTileX, nx - x0);
  const int RH = TH + 2 * H;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int lane = threadIdx.x & 63;

  constexpr int NR = kTileY;
  const int nwaves = blockDim.x >> 6;
  // the wavefronts past the ncw colliding ones: the first nnw draw, the last
  // NR form the sums of a tile row each (some do both where both do not fit)
  const bool collides = wave < ncw;
  const bool draws = draws_apart<R>() && !collides && wave < ncw + M.nnw;
  const int srow = SAMPLE && !collides ? wave - (nwaves - NR) : -1;

  // this thread's site of the region: row, and column + H (bits 8..), kept in
  // one register; with FP64 collisions, which need every register, all else
  // is formed from it again in each step (the empty asm below)
  uint32_t where;
  int zslot = threadIdx.x;  // of a drawing thread: the colliding one of its site
  {
    int row, colh;
    bool valid;
    if (full) {
      const int rpw = M.rpw;
      const int rsub = (int)(((uint32_t)lane * M.nx_magic) >> 16);
      row = (draws ? wave - ncw : wave) * rpw + rsub + (draws ? 1 : 0);
      colh = lane - rsub * nx + H;
      valid = rsub < rpw && row < (draws ? RH - 1 : RH);
      if (draws) {
        const int cw = (int)(((uint32_t)row * M.rpw_magic) >> 16);
        zslot = cw * 64 + (row - cw * rpw) * nx + colh - H;
      }
    } else if (wave < RH) {
      row = wave;
      colh = lane + H;
      valid = lane < W;
    } else {
      const int idx = (wave - RH) * 64 + lane, w2 = 2 * H;
      row = idx / w2;
      const int c = idx - row * w2;
      colh = c < H ? c : W + c;
      valid = row < RH;
    }
    where = valid && (collides || draws) ? (uint32_t)row | (uint32_t)colh << 8 | 0x80000000u : 0u;
  }
  S* const pops = reinterpret_cast<S*>(multi_lds);
  // by the parity of the step: the pre-collision values of the tile rows
  // [2][row][value][64 sites]; the staging of the summing wavefronts; their
  // results [2][row][kXtxVals]; the tile's sums
  S* const raw = pops + (size_t)(NR + 2 * H) * 9 * kRS;
  unsigned char* const after = reinterpret_cast<unsigned char*>(raw + (size_t)2 * NR * 9 * kTileX);
  double* const red = reinterpret_cast<double*>(after + (size_t)NR * sample_wave_bytes<S>());
  double* const sums = red + (size_t)2 * NR * kXtxVals;
  // the draws, by the parity of the step: [2][value][colliding thread]
  using D = typename LdsDraw<S, R>::type;
  D* const drawn = SAMPLE ? reinterpret_cast<D*>(sums + 64)
                          : reinterpret_cast<D*>(pops + (size_t)(NR + 2 * H) * 9 * kRS);
  const int zplane = ncw * 64;

  constexpr bool kNoise32 = sizeof(S) < sizeof(R);

  // FP32 collisions hold their constants in scalar registers
  CollideConst<R> C;
  if constexpr (!draws_apart<R>()) C = collide_const<R>(sd);

  // statistic `lane` is kept by one thread of the first summing wavefront
  const bool keeps = SAMPLE && srow == 0 && lane < kNStat && sd.sample_every > 0;
  if (keeps) sums[lane] = sd.partials[((size_t)gy * M.tiles_x + tx) * kNStat + lane];
  // sites past the end of a row count as zeros
  if (srow >= 0 && lane >= W)
    for (int q = 0; q < 2 * 9; ++q)
      raw[((size_t)(q / 9 * NR + srow) * 9 + q % 9) * kTileX + lane] = S(0);
  // steps to the next sample, counted down from the first step's
  uint32_t to_sample = ~0u;
  if (SAMPLE && sd.sample_every > 0) {
    to_sample = 0;
    while (to_sample <= (uint32_t)K &&
           !multiple_of(t0 + to_sample, (uint32_t)sd.sample_every, sd.se_magic, sd.se_shift))
      ++to_sample;
  }
  bool was_due = false;

  // with SAMPLE one more turn, for the sums of the last step
#pragma unroll 1
  for (int s = 0; s < (SAMPLE ? K + 1 : K); ++s) {
    const uint64_t t = t0 + (uint64_t)s;
    const bool due = SAMPLE && to_sample == 0;
    if (SAMPLE && srow >= 0 && was_due && srow < TH) {
        const S* x = raw + (size_t)(((s - 1) & 1) * NR + srow) * 9 * kTileX + lane;
        R h[9];
#pragma unroll
        for (int i = 0; i < 9; ++i) h[i] = (R)x[i * kTileX];
        double a[4];
        wave_xtx<S, R>(h, true, lane, W, after + (size_t)srow * sample_wave_bytes<S>(), a);
        double* out = red + ((size_t)(s & 1) * NR + srow) * kXtxVals;
        const int xc = lane & 15;
#pragma unroll
        for (int q = 0; q < 4; ++q) {
          const int xr = xtx_row<S>(lane >> 4, q);
          if (xr < 9 && xc < 10) out[xr * 10 + xc] = a[q];
        }
    }
    if (s < (draws ? K - 1 : K)) {
      uint32_t w = where;
      if constexpr (draws_apart<R>()) asm volatile("" : "+v"(w));
      // a drawing wavefront is one step ahead
      const int sd_ = draws ? s + 1 : s;
      const int hs = H - sd_, row = (int)(w & 0xFFu), col = (int)((w >> 8) & 0xFFu) - H;
      const bool odd = (s & 1) != 0;
      const bool active = (int32_t)w < 0 && row >= sd_ && row < RH - sd_ &&
                          (full || (col >= -hs && col < W + hs));
      if (active) {
        // the site on the lattice (periodic; a halo may go round twice)
        int gxx = x0 + col, gyy = y0 - H + row;
        gxx = gxx < 0 ? gxx + nx : (gxx >= nx ? gxx - nx : gxx);
        if (gyy < 0) gyy += ny;
        if (gyy < 0) gyy += ny;
        if (gyy >= ny) gyy -= ny;
        if (gyy >= ny) gyy -= ny;
        const uint32_t site = (uint32_t)gyy * (uint32_t)nx + (uint32_t)gxx;
        if constexpr (draws_apart<R>()) C = step_const<R>(&sd);
        const LdsDraw<S, R> z{drawn + (sd_ & 1) * (LdsDraw<S, R>::n * zplane) + zslot, zplane};
        if (draws) {
          if (C.noise) {
            SiteDraw<R, kNoise32> d;
            site_draw<R, kNoise32>(C, site, t + 1, d);
            z.put(d);
          }
        } else {
        R h[9];
        if (s == 0) {
          const S* const src = reinterpret_cast<const S*>(M.flip ? sd.pop2 : sd.pop);
          const uint32_t e = (uint32_t)gyy * 9u * M.pitch + (uint32_t)gxx;
#pragma unroll
          for (int i = 0; i < 9; ++i) h[i] = (R)src[e + (uint32_t)i * M.pitch];
        }
        SiteDraw<R, kNoise32> draw;
        if (C.noise && (!draws_apart<R>() || s == 0)) {
          site_draw<R, kNoise32>(C, site, t, draw);
          if constexpr (draws_apart<R>()) z.put(draw);
        }
        // LDS element of value 0 at the three columns
        S* const lds_c = pops + row * 9 * kRS + (full ? col : col + H);
        S* const lds_m = full && col == 0 ? lds_c + (nx - 1) : lds_c - 1;
        S* const lds_p = full && col == nx - 1 ? lds_c - (nx - 1) : lds_c + 1;
        if (odd) {
#pragma unroll
          for (int i = 0; i < 9; ++i)
            h[i] = (R)(kVX[i] > 0 ? lds_m : (kVX[i] < 0 ? lds_p
                                                        : lds_c))[(kOpp[i] - 9 * kVY[i]) * kRS];
        } else if (s > 0) {
#pragma unroll
          for (int i = 0; i < 9; ++i) h[i] = (R)lds_c[i * kRS];
        }
        if (SAMPLE && row >= H && row < H + TH && col >= 0 && col < W) {
          if (due) {
            S* x = raw + (size_t)((s & 1) * NR + row - H) * 9 * kTileX + col;
#pragma unroll
            for (int i = 0; i < 9; ++i) x[i * kTileX] = (S)h[i];
          }
          if (s == 0 && sd.skz != nullptr && sd.sk_every > 0 &&
              multiple_of(t, (uint32_t)sd.sk_every, sd.sk_magic, sd.sk_shift))
            sk_fields<S, R>(h, sd, site);
        }
        int e;
        if constexpr (draws_apart<R>()) e = collide<R, BASIS>(h, C, z);
        else e = collide<R, BASIS>(h, C, draw);
        if (e) {
          atomicOr(sd.err, e);
          atomicMin(sd.err_step, (unsigned long long)t);
        }
        if (s == K - 1) {
          // the value of direction o goes to the site it moves to
          S* const dst = reinterpret_cast<S*>(M.flip ? sd.pop : sd.pop2);
          const uint32_t P = M.pitch;
          const uint32_t ym = gyy == 0 ? ny - 1 : gyy - 1, yp = gyy == ny - 1 ? 0 : gyy + 1;
          const uint32_t xm = gxx == 0 ? nx - 1 : gxx - 1, xp = gxx == nx - 1 ? 0 : gxx + 1;
          const uint32_t rc = (uint32_t)gyy * 9u * P, rm = ym * 9u * P, rp = yp * 9u * P;
#pragma unroll
          for (int o = 0; o < 9; ++o)
            dst[(kVY[o] > 0 ? rp : (kVY[o] < 0 ? rm : rc)) + (uint32_t)o * P +
                (kVX[o] > 0 ? xp : (kVX[o] < 0 ? xm : (uint32_t)gxx))] = (S)h[o];
        } else if (odd) {
#pragma unroll
          for (int i = 0; i < 9; ++i)
            (kVX[i] > 0 ? lds_m
                        : (kVX[i] < 0 ? lds_p : lds_c))[(kOpp[i] - 9 * kVY[i]) * kRS] =
                (S)h[kOpp[i]];
        } else {
#pragma unroll
          for (int i = 0; i < 9; ++i) lds_c[i * kRS] = (S)h[kOpp[i]];
        }
        }
      }
    }
    if (SAMPLE || s < K - 1) __syncthreads();
    if (was_due && keeps) {
      // rows past the lattice count as zeros; this result area is written
      // again two turns later, one barrier after these reads
      const double* r = red + (size_t)(s & 1) * NR * kXtxVals + kXtxPos.pos[lane];
      const double w0 = r[0], w1 = TH > 1 ? r[kXtxVals] : 0.0;
      const double w2 = TH > 2 ? r[2 * kXtxVals] : 0.0, w3 = TH > 3 ? r[3 * kXtxVals] : 0.0;
      sums[lane] += (w0 + w1) + (w2 + w3);
    }
    was_due = due;
    to_sample = due ? (uint32_t)sd.sample_every - 1 : to_sample - 1;
  }
  if (keeps) sd.partials[((size_t)gy * M.tiles_x + tx) * kNStat + lane] = sums[lane];
}

// ------------------------------------------------------------- shapes
static int colliding_waves(int nx, int K) {
  const int H = K - 1, RH = kTileY + 2 * H;
  if (nx > kTileX) return RH + (2 * H * RH + 63) / 64;
  const int rpw = kTileX / nx;
  return (RH + rpw - 1) / rpw;
}
static int drawing_waves(int compute, int nx, int K) {
  if (nx > kTileX || !(compute == 0 ? draws_apart<double>() : draws_apart<float>())) return 0;
  const int RH = kTileY + 2 * (K - 1), rpw = kTileX / nx;
  return (RH - 2 + rpw - 1) / rpw;
}
// All wavefronts of a workgroup: those that draw and those that sum are the
// same ones where they would not fit side by side.
int multi_waves(int compute, bool sample, int nx, int K) {
  const int most = (compute == 0 ? multi_max_threads<double>() : multi_max_threads<float>()) / 64;
  const int nc = colliding_waves(nx, K), nd = drawing_waves(compute, nx, K), ns = kTileY;
  if (!sample) return nc + nd;
  return nc + (nc + nd + ns <= most ? nd + ns : std::max(nd, ns));
}

static size_t multi_lds_bytes(int storage, int compute, bool sample, int nx, int K) {
  const int H = K - 1, RH = kTileY + 2 * H;
  const size_t es = storage == 0 ? 8 : 4, rows = kTileY;
  size_t b = (size_t)RH * 9 * kRS * es;
  if (sample)
    b += rows * (2 * 9 * kTileX * es + 2 * kXtxVals * sizeof(double) +
                 (storage == 0 ? sample_wave_bytes<double>() : sample_wave_bytes<float>())) +
         64 * sizeof(double);
  if (drawing_waves(compute, nx, K))
    b += 2 * (storage != compute ? 6 * sizeof(float) : 9 * es) * 64 *
         (size_t)colliding_waves(nx, K);
  return b;
}

bool multi_fits(int storage, int compute, bool sample, int nx, int K, size_t max_lds) {
  if (K < 2 || K > kMultiMaxSteps || (K & 1)) return false;
  // halo columns: as many as the row stride holds; FP64 collisions take none
  if (nx > kTileX && (K - 1 > kMultiMaxHalo || compute == 0)) return false;
  const int most = compute == 0 ? multi_max_threads<double>() : multi_max_threads<float>();
  return 64 * multi_waves(compute, sample, nx, K) <= most &&
         multi_lds_bytes(storage, compute, sample, nx, K) <= max_lds;
}

// Launches above 64 KiB of LDS have to be allowed, kernel by kernel.
template <typename S, typename R>
static hipError_t allow_lds(int basis, int bytes) {
  const void* k[3][2] = {{(const void*)step_multi_kernel<S, R, kBasisFnormLocal, false>,
                          (const void*)step_multi_kernel<S, R, kBasisFnormLocal, true>},
                         {(const void*)step_multi_kernel<S, R, kBasisHermite, false>,
                          (const void*)step_multi_kernel<S, R, kBasisHermite, true>},
                         {(const void*)step_multi_kernel<S, R, kBasisFnormLut, false>,
                          (const void*)step_multi_kernel<S, R, kBasisFnormLut, true>}};
  hipError_t e = hipSuccess;
  for (int s = 0; s < 2 && e == hipSuccess; ++s)
    e = hipFuncSetAttribute(k[basis][s], hipFuncAttributeMaxDynamicSharedMemorySize, bytes);
  return e;
}

hipError_t multi_prepare(int storage, int compute, int basis, int nx, int K, size_t max_lds) {
  if (multi_lds_bytes(storage, compute, true, nx, K) <= 65536) return hipSuccess;
  if (storage == 0) return allow_lds<double, double>(basis, (int)max_lds);
  if (compute == 0) return allow_lds<float, double>(basis, (int)max_lds);
  return allow_lds<float, float>(basis, (int)max_lds);
}

template <typename S, typename R, int BASIS>
static hipError_t launch_multi_t(bool sample, const SlotDesc* d_slots, int nslots, int nx, int ny,
                                 int K, int flip, const uint64_t* clk, uint32_t step_idx,
                                 hipStream_t st) {
  constexpr int storage = sizeof(S) == 8 ? 0 : 1, compute = sizeof(R) == 8 ? 0 : 1;
  MultiShape M{};
  M.nx = nx;
  M.ny = ny;
  M.tiles_x = (nx + kTileX - 1) / kTileX;
  M.pitch = (uint32_t)M.tiles_x * kTileX;
  M.groups = M.tiles_x * ((ny + kTileY - 1) / kTileY);
  magic_div((uint32_t)M.groups, &M.gr_magic, &M.gr_shift);
  magic_div((uint32_t)M.tiles_x, &M.tx_magic, &M.tx_shift);
  M.K = K;
  M.ncw = colliding_waves(nx, K);
  M.nnw = drawing_waves(compute, nx, K);
  M.rpw = nx > kTileX ? 1 : kTileX / nx;
  M.nx_magic = 65536u / (uint32_t)nx + 1;
  M.rpw_magic = 65536u / (uint32_t)M.rpw + 1;
  M.flip = flip;
  const dim3 grid((unsigned)M.groups * nslots), b(64 * multi_waves(compute, sample, nx, K));
  const size_t lds = multi_lds_bytes(storage, compute, sample, nx, K);
  if (sample)
    hipLaunchKernelGGL((step_multi_kernel<S, R, BASIS, true>), grid, b, lds, st, d_slots, M, clk,
                       step_idx);
  else
    hipLaunchKernelGGL((step_multi_kernel<S, R, BASIS, false>), grid, b, lds, st, d_slots, M, clk,
                       step_idx);
  return hipGetLastError();
}

template <typename S, typename R>
static hipError_t launch_multi_b(int basis, bool sample, const SlotDesc* d_slots, int nslots,
                                 int nx, int ny, int K, int flip, const uint64_t* clk,
                                 uint32_t k, hipStream_t st) {
  switch (basis) {
    case kBasisFnormLocal:
      return launch_multi_t<S, R, kBasisFnormLocal>(sample, d_slots, nslots, nx, ny, K, flip,
                                                    clk, k, st);
    case kBasisHermite:
      return launch_multi_t<S, R, kBasisHermite>(sample, d_slots, nslots, nx, ny, K, flip,
                                                 clk, k, st);
    case kBasisFnormLut:
      return launch_multi_t<S, R, kBasisFnormLut>(sample, d_slots, nslots, nx, ny, K, flip,
                                                  clk, k, st);
  }
  return hipErrorInvalidValue;
}

hipError_t launch_step_multi(int storage, int compute, int basis, bool sample,
                             const SlotDesc* d_slots, int nslots, int nx, int ny, int K, int flip,
                             const uint64_t* d_clock, uint32_t step_idx, hipStream_t st) {
  if (nslots <= 0) return hipSuccess;
  if (storage == 0)
    return launch_multi_b<double, double>(basis, sample, d_slots, nslots, nx, ny, K, flip,
                                          d_clock, step_idx, st);
  if (compute == 0)
    return launch_multi_b<float, double>(basis, sample, d_slots, nslots, nx, ny, K, flip,
                                         d_clock, step_idx, st);
  return launch_multi_b<float, float>(basis, sample, d_slots, nslots, nx, ny, K, flip, d_clock,
                                      step_idx, st);
}

}  // namespace flb
