// flb_runtime.hpp — internal declarations shared by the host-side sources of
// libflb (runtime, lattice/ensemble, server).  Not part of the C ABI.
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

#include <vector>

#include "flb.h"
#include "flb_kernels.hpp"

namespace flb {

// Above this background speed the FP32-storage path builds the local basis
// in FP64 (the Schur complement loses digits as u approaches the edge of the
// validity region).
constexpr double kFp32BasisMaxSpeed = 0.25;


int set_error(int code, const char* fmt, ...);
int hip_fail(hipError_t e, const char* what);
int check_params(const flb_params* p);
int compute_precision(const flb_params* p);
// Whether this many tiles of independent lattices are stepped faster as two
// halves side by side (compute: 0 FP64, 1 FP32; the measurements are beside
// Group::graph_branches), alone on the device or beside other work.
inline bool two_branches(int compute, int tiles, bool alone) {
  const int least = alone ? 1024 : 8192;
  return tiles >= (compute == 0 ? least : 2 * least);
}
uint32_t row_pitch(int nx);
size_t population_elems(int nx, int ny);
void tile_shape(const flb_params& p, int* wide, int* tiles_x, int* ntiles);
void set_tiles(SlotDesc* d, int wide);
bool small_lattice_tiles(const flb_params& p);
void magic_div(uint32_t d, uint32_t* magic, uint32_t* shift);
void fill_slot(const flb_params* p, SlotDesc* d);
Shift9 slot_shift(const SlotDesc& d);
void hermite_rows(double m[81]);
double equilibrium(int i, double rho, double ux, double uy);
bool fnorm_rows(double ux, double uy, double mt[81]);

// Makes a device the calling thread's current one while it lives: events and
// streams belong to the device they are created on, and a thread may use a
// lattice of another device than its current one.
class OnDevice {
 public:
  explicit OnDevice(int device) {
    if (hipGetDevice(&was_) != hipSuccess || was_ == device) was_ = -1;
    else if (hipSetDevice(device) != hipSuccess) was_ = -1;
  }
  ~OnDevice() {
    if (was_ >= 0) (void)hipSetDevice(was_);
  }
  OnDevice(const OnDevice&) = delete;
  OnDevice& operator=(const OnDevice&) = delete;

 private:
  int was_ = -1;
};

// Whether a lattice, ensemble or server has work enqueued that the library has
// not waited for since, counted over the process by device: launches that pay
// only while nothing else fills the chip ask for others().  A program that
// waits by its own means (its stream's, the device's synchronisation) is taken
// to be at work until its next readout or sync.
class AtWork {
 public:
  AtWork() = default;
  ~AtWork() { end(); }
  AtWork(const AtWork&) = delete;
  AtWork& operator=(const AtWork&) = delete;
  void begin(int device);
  void end();
  bool begun() const { return on_ >= 0; }
  bool others(int device) const;

 private:
  int on_ = -1;  // the device, while at work
};

// A second population buffer's bytes, counted over the process by device while
// it lives; refused where the sum would exceed `most`.
class SecondBytes {
 public:
  SecondBytes() = default;
  ~SecondBytes() { give(); }
  SecondBytes(const SecondBytes&) = delete;
  SecondBytes& operator=(const SecondBytes&) = delete;
  bool take(int device, size_t bytes, size_t most);
  void give();

 private:
  int device_ = -1;  // while bytes are taken
  size_t bytes_ = 0;
};

// Readouts to caller-owned host memory go through page-locked staging: a copy
// of 14 MB straight into pageable memory takes 0.86 ms, through it 0.45, and
// every small piece 10 to 15 us.  The staging is the process's, held while any
// lattice or server exists (Staging members count them); a thread that finds
// it in use copies straight.
class Staging {
 public:
  Staging();
  ~Staging();
  Staging(const Staging&) = delete;
  Staging& operator=(const Staging&) = delete;
};
// One piece of a readout: bytes from device memory to the host.
struct HostPiece {
  void* dst;
  const void* src;
  size_t bytes;
};
// Copies the pieces behind the work already enqueued on st and waits for them.
// behind_steps: that work may be long (steps that nobody has waited for).
hipError_t copy_out(const HostPiece* pieces, int n, hipStream_t st, bool behind_steps = false);
inline hipError_t copy_out(void* dst, const void* src, size_t bytes, hipStream_t st) {
  const HostPiece p{dst, src, bytes};
  return copy_out(&p, 1, st);
}

struct Stats {
  uint64_t tb_len = 0, tb_fill = 0, nb = 0, nsamples = 0;
  int max_blocks = kMaxTimeBlocks;  // record capacity (even)
  std::vector<uint64_t> rec_len;    // samples (time steps) per closed record
  void reset(int block_steps);
  hipError_t after_sample(uint64_t nsites, double* d_partials, int ntiles, double* d_records,
                          hipStream_t st);
  // Whether the next sample closes a time block without first merging
  // records; then close_counted does that sample's bookkeeping and returns
  // the record index, and the caller closes the block on the device.
  bool plain_close_next() const;
  uint64_t close_counted(uint64_t nsites);
  uint64_t block_samples(uint64_t b) const;
};

int finish_covariance(const Stats& S, const std::vector<double>& rec, const double* open,
                      uint64_t sites, const double mt0[81], flb_cov* out);

// launchers (flb_kernels.hip)
hipError_t launch_step(int storage, int compute, int basis, bool sample, int odd,
                       const SlotDesc* d_slots, const int* d_prefix, int nslots,
                       int total_tiles, const uint64_t* d_clock, uint32_t step_idx,
                       LaunchCfg cfg, hipStream_t st);
hipError_t launch_tick(uint64_t* d_clock, uint64_t n, hipStream_t st);
hipError_t launch_write_state(int storage, void* pop, uint32_t P, const double* f, int nx, int ny,
                              int odd, const Shift9& sh, int y0, int rows, hipStream_t st);
hipError_t launch_read_state(int storage, const void* pop, uint32_t P, double* f, int nx, int ny,
                             int odd, const Shift9& sh, int y0, int rows, hipStream_t st);
hipError_t launch_raw_state(int storage, void* pop, uint32_t P, void* buf, int nx, int ny, int odd,
                            int to_buf, int y0, int rows, hipStream_t st);
hipError_t launch_init(int storage, void* pop, uint32_t P, const double* rho, const double* ux,
                       const double* uy, double rho0, double ux0, double uy0, const Shift9& sh,
                       int nx, int ny, double mu, uint32_t k0, uint32_t k1, int odd, int y0,
                       int rows, hipStream_t st);
hipError_t launch_moments(int storage, const void* pop, uint32_t P, const double* B, double* out,
                          int nx, int ny, int odd, double rho0, double ux0, double uy0,
                          const Shift9& sh, int* err, int y0, int rows, hipStream_t st);
// The Fourier-coefficient readback: a grid of gx blocks of 256 columns by
// gy row groups, gx * gy <= max_blocks (returned), one partial per block
// at blockIdx.y * gx + blockIdx.x.
int fourier_mode_grid(int nx, int ny, int max_blocks, int* gx, int* gy);
hipError_t launch_fourier_mode(int storage, const void* pop, uint32_t P, double2* partial,
                               int max_blocks, int nx, int ny, int odd, int which, int kx, int ky,
                               double ux0, double uy0, hipStream_t st);
hipError_t launch_close_block(double* partials, int ntiles, double* record, hipStream_t st);
// n lattices of ntiles tiles each at once (device arrays of their partials
// and record bases; the record written at records[k] + record_offset)
hipError_t launch_close_block_many(double* const* partials, double* const* records,
                                  size_t record_offset, int n, int ntiles, hipStream_t st);
// n lattices of any tile counts (host arrays)
hipError_t launch_close_block_list(double* const* partials, double* const* records,
                                   const int* ntiles, int n, hipStream_t st);
hipError_t launch_merge_blocks(double* rec, int nhalf, hipStream_t st);
// folds: kFoldRows rows of kNStat doubles of scratch
hipError_t launch_open_sum(const double* partials, int ntiles, double* out, double* folds,
                           hipStream_t st);
hipError_t launch_fill(double* p, size_t n, double v, hipStream_t st);
hipError_t launch_stream_copy(const void* in, void* out, size_t n4, hipStream_t st);
hipError_t launch_stream_probe(int storage, void* pop, int nx, int ny, uint32_t pitch, int wide,
                               int tiles_x, int ntiles, int odd, hipStream_t st);
// out[ky - ky0][kx] = norm acc[kx][ky] for rows ky0 .. ky0 + rows of the full
// plane, the half kx > nx/2 from its partner at -k (negated there for the
// imaginary part of the cross term)
hipError_t launch_sk_expand(const double* acc, double* out, int nx, int ny, int ky0, int rows,
                            double norm, int negate, hipStream_t st);
hipError_t sk_prepare(size_t max_lds);
hipError_t launch_sk_sample(int storage, void* z, void* zt, double* acc, int nx, int ny,
                            const void* twx, const void* twy, size_t max_lds, hipStream_t st);
// Whether rows of length n can be transformed (power of two that fits the
// LDS FFT, or short enough for the direct DFT).
int sk_transform_supported(int n, int storage, size_t max_lds);

// Bump allocator over one device allocation (256-byte aligned pieces).
struct Arena {
  char* base = nullptr;
  size_t used = 0, cap = 0;
  template <typename T>
  T* take(size_t count) {
    used = (used + 255) & ~(size_t)255;
    T* p = base ? reinterpret_cast<T*>(base + used) : nullptr;
    used += count * sizeof(T);
    return p;
  }
};

}  // namespace flb
