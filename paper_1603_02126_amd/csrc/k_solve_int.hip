// HIP kernels (gfx950): EPICal calibration solve of integer samples on the
// matrix cores.
#include <algorithm>
#include <cstddef>

#include "solve_int.h"

namespace epic {

// (the FP64 solve of a run's remaining intervals uses the same LDS)
constexpr int kSolveIntBytes = std::max(int(SolveSmem::BYTES), int(SolveIntSmem::BYTES));

// The intervals from n on, in FP64.  Called, not inlined, and with a pointer to
// the kernel's own arguments: inlined, or with a copy of them, it took the
// matrix-core loop's registers (0.2 to 0.5 us more per interval of 60 samples,
// 101 antennas).
typedef const __attribute__((address_space(4))) uint8_t* KernelArgs;
typedef __attribute__((address_space(3))) uint8_t* LdsPtr;   // (a generic one would be read by FLAT loads)
template <int FMT, int J>
__device__ __noinline__ void solve_rest(KernelArgs at, int f, LdsPtr lds, int n) {
  uint8_t* const smem = (uint8_t*)lds;
  SolveArgs a;
  __builtin_memcpy(&a, (const void*)at, sizeof(a));
  a = from_interval(uniform_copy(a), __builtin_amdgcn_readfirstlane(n));
  f = __builtin_amdgcn_readfirstlane(f);
  const int RB = FMT == kCI4 ? a.Na : 2 * a.Na;
  if (RB % 16 == 0) solve_channel_fmt<J, 16, FMT, kSolveMainThreads, true>(a, f, smem, nullptr, 0, true);
  else if (RB % 4 == 0) solve_channel_fmt<J, 4, FMT, kSolveMainThreads, true>(a, f, smem, nullptr, 0, true);
  else solve_channel_fmt<J, 1, FMT, kSolveMainThreads, true>(a, f, smem, nullptr, 0, true);
}

// A channel's whole run; `at`: byte offset of `a` in the kernel's arguments.
template <int FMT, int J>
__device__ __forceinline__ void solve_channel_int_alone(const SolveArgs& a, int f, uint8_t* smem, int at) {
  const int n = solve_channel_int<FMT, J, false>(a, f, smem);
  if (n < a.n_int) solve_rest<FMT, J>((KernelArgs)__builtin_amdgcn_kernarg_segment_ptr() + at, f, (LdsPtr)smem, n);
}

template <int FMT, int J>
__global__ __launch_bounds__(kSolveMainThreads) void k_solve_int(SolveArgs a) {
  __shared__ __align__(16) uint8_t smem[kSolveIntBytes];
  solve_channel_int_alone<FMT, J>(a, blockIdx.x, smem, 0);
}

// Integer samples, one tapped pixel, up to 1024 antennas (its LDS) and rows of
// at least one 16-byte piece, a chunk's rows within 32-bit offsets: the
// matrix-core solve.  Its steps per interval cost the same few microseconds
// however short the interval: 256 antennas of ci4, us per interval, FP64 FMAs
// against it, 2.4 / 3.3 at 8 samples, 3.5 / 3.6 at 25, 7.6 / 4.6 at 100.
bool solve_by_int(const SolveArgs& a) {
  const int64_t RB = int64_t(a.Na) * efmt_bytes(a.fmt);
  return std::min(a.t_cal, a.n_t) >= kSolveIntMinSamples && a.fmt != kCF32 && a.Na <= kSolveIntMaxAnt && RB >= 16 &&
         a.F * RB < (int64_t(1) << 24) && a.n_pix == 1 && !solve_by_wave(a);
}

bool solve_writes_u(const SolveArgs& a) { return solve_by_int(a); }

// Channels of several arrays: the variant by the workgroup's array.
__global__ __launch_bounds__(kSolveMainThreads) void k_solve_int_batch(BatchSolveArgs b) {
  __shared__ __align__(16) uint8_t smem[kSolveIntBytes];
  int i = 0;
  while (i + 1 < b.n_arrays && int(blockIdx.x) >= b.chan_off[i + 1]) ++i;
  const SolveArgs& a = b.arr[i];
  const int f = int(blockIdx.x) - b.chan_off[i];
  const bool one = a.Na <= kSolveMainThreads;
  const int at = int(offsetof(BatchSolveArgs, arr)) + i * int(sizeof(SolveArgs));
  if (a.fmt == kCI4 && one) solve_channel_int_alone<kCI4, 1>(a, f, smem, at);
  else if (a.fmt == kCI4) solve_channel_int_alone<kCI4, 2>(a, f, smem, at);
  else if (one) solve_channel_int_alone<kCI8, 1>(a, f, smem, at);
  else solve_channel_int_alone<kCI8, 2>(a, f, smem, at);
}

hipError_t launch_solve_int_batch(const BatchSolveArgs& b, hipStream_t s) {
  hipLaunchKernelGGL(k_solve_int_batch, dim3(b.chan_off[b.n_arrays]), dim3(kSolveMainThreads), 0, s, b);
  return hipGetLastError();
}

hipError_t launch_solve_int(const SolveArgs& a, hipStream_t s) {
  const dim3 grid(a.F), blk(kSolveMainThreads);
  const bool one = a.Na <= kSolveMainThreads;
  if (a.fmt == kCI4 && one) hipLaunchKernelGGL((k_solve_int<kCI4, 1>), grid, blk, 0, s, a);
  else if (a.fmt == kCI4) hipLaunchKernelGGL((k_solve_int<kCI4, 2>), grid, blk, 0, s, a);
  else if (one) hipLaunchKernelGGL((k_solve_int<kCI8, 1>), grid, blk, 0, s, a);
  else hipLaunchKernelGGL((k_solve_int<kCI8, 2>), grid, blk, 0, s, a);
  return hipGetLastError();
}

}  // namespace epic
