// flb_multi.hpp — several steps of small lattices per launch (internal).
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

#include "flb_kernels.hpp"

namespace flb {

constexpr int kMultiMaxHalo = 3;       // halo columns on each side of a 64-site tile
constexpr int kMultiMaxSteps = 6;      // halo rows: at most five
// Threads of a workgroup: FP64 collisions are limited to 768, so that a thread
// may use 168 registers (128 spill).
template <typename R>
constexpr int multi_max_threads() {
  return sizeof(R) == 8 ? 768 : 1024;
}

// Whether K steps of a tile fit the kernel's limits.
bool multi_fits(int storage, int compute, bool sample, int nx, int K, size_t max_lds);
// Wavefronts of a workgroup that takes K steps.
int multi_waves(int compute, bool sample, int nx, int K);
// Allow the kernels the LDS that up to K steps take (before launches, outside a
// capture).
hipError_t multi_prepare(int storage, int compute, int basis, int nx, int K, size_t max_lds);
// K steps of nslots lattices of nx x ny sites (64 x 4 tiles, K even, the
// first step at an even time), pop -> pop2 (flip: pop2 -> pop), with the
// correlator sums of the steps that sample and, where the first step is a
// structure-factor step, its fields.
hipError_t launch_step_multi(int storage, int compute, int basis, bool sample,
                             const SlotDesc* d_slots, int nslots, int nx, int ny, int K, int flip,
                             const uint64_t* d_clock, uint32_t step_idx, hipStream_t st);

constexpr int kMarchCols = 62;  // columns a wavefront of step_march_kernel stores

// Two steps of nslots large lattices (FP32 storage and collision, no sums or
// fields due, the first step at an even time) in one pass over memory, H rows
// a wavefront, pop -> pop2 (flip: pop2 -> pop).
hipError_t launch_step_march(int basis, const SlotDesc* d_slots, int nslots, int nx, int ny,
                             int H, int flip, const uint64_t* d_clock, uint32_t step_idx,
                             hipStream_t st);

}  // namespace flb
