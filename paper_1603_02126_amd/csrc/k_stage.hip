// HIP kernels (gfx950) of the stage-wise calls: gridding to HBM, and
// transform + square + accumulate (+ tap) from HBM grids.
//
// Both are bound by the grids' bytes (8 N^2 per frame, written by the one and
// read by the other), so every global access is a run of consecutive cells
// over the lanes of a wave: rows are exchanged between lanes through LDS.
#include <algorithm>
#include <limits>

#include "image_fft.h"

namespace epic {

// E' = u E with the rounding fixed (which product the FMA takes exactly is
// otherwise the compiler's choice, and the gains of the stage-wise loop follow
// the tap of these grids).
__device__ __forceinline__ float2 calibrate(float2 e, float2 u) {
  return make_float2(fmaf(e.x, u.x, -(e.y * u.y)), fmaf(e.y, u.x, e.x * u.y));
}

// ---------------------------------------------------------------------------
// Gridding: one frame per lane group (N <= 32, and 64 x 64 arrays whose E'
// and half-frame schedule do not fit k_grid_half's LDS).
// ---------------------------------------------------------------------------
template <int N, int APL>
__global__ __launch_bounds__(256) void k_grid(GridArgs a) {
  using G = Geo<N>;
  __shared__ float2 lds[G::LDS];
  __shared__ float2 lds_e[G::SLOTS * APL * N];
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const int h = lane / N, lam = lane % N;
  const int slot = wave * G::FPW + h;
  const int64_t q = int64_t(blockIdx.x) * G::SLOTS + slot;  // frame = t * F + f
  const bool active = q < int64_t(a.nt) * a.F;
  float2* buf = lds + slot * G::FRAME;
  float2* epr = lds_e + slot * (APL * N);
  static_for<0, N>([&](auto xc) { buf[lam * G::PITCH + decltype(xc)::value] = make_float2(0.f, 0.f); });
  const int64_t t = active ? q / a.F : 0;
  const int f = active ? int(q % a.F) : 0;
  const int bpe = efmt_bytes(a.fmt);
  const uint8_t* row = a.efield + ((a.t0 + t) * a.F + f) * int64_t(a.Na) * bpe;
  for (int an = lam; an < a.Na; an += N)
    epr[an] = active ? calibrate(load_sample_global(row, an, a.fmt), gload(a.u + int64_t(f) * a.Na + an))
                     : make_float2(0.f, 0.f);
  wave_lds_sync();
  grid_frame(buf, epr, a.slots, a.n_slots, N, lam);
  wave_lds_sync();
  if (active) {
    float2* out = a.grid + q * (N * N);
    static_for<0, N>([&](auto yc) {
      constexpr int y = decltype(yc)::value;
      gstore(out + y * N + lam, buf[y * G::PITCH + lam]);
    });
  }
}

// ---------------------------------------------------------------------------
// Gridding at 64 x 64 through half a frame: eight waves, two per SIMD (a whole
// frame per wave leaves room for four), each gridding its own frames by the
// paired engine's half-frame schedules, which a workgroup copies to LDS once
// for all its frames.  The cells of a half are taken (and cleared) a pair per
// lane, so that a store instruction writes four runs of 256 bytes.
// Sums are those of k_grid, contribution by contribution.
// 64 channels x 100 samples of 200 antennas: 61 -> 37 us (210 MB written).
// ---------------------------------------------------------------------------
template <int APL>
__global__ __launch_bounds__(kPairThreads) void k_grid_half(GridArgs a) {
  constexpr int N = 64, W = kPairThreads / 64;
  using L = PairSmem<APL>;
  __shared__ __align__(16) uint8_t smem[L::BYTES];
  const int lam = threadIdx.x & 63, wave = wave_index();
  float2* H = reinterpret_cast<float2*>(smem) + wave * L::WAVE;
  float2* epr = H + L::HALF;
  uint2* stab = reinterpret_cast<uint2*>(smem + L::T_OFF);
  const int S0 = a.n_slots_h0, S1 = a.n_slots_h1;
  load_slot_table(stab, a.slots_h, S0 + S1, N);
  clear_half_row(H, lam);
  __syncthreads();
  const int bpe = efmt_bytes(a.fmt);
  const int64_t frames = int64_t(a.nt) * a.F;
  for (int64_t q = int64_t(blockIdx.x) * W + wave; q < frames; q += int64_t(gridDim.x) * W) {
    const int64_t t = q / a.F;
    const int f = int(q % a.F);
    const uint8_t* row = a.efield + ((a.t0 + t) * a.F + f) * int64_t(a.Na) * bpe;
    static_for<0, APL>([&](auto ic) {
      const int an = lam + N * decltype(ic)::value;
      if (an < a.Na) epr[an] = calibrate(load_sample_global(row, an, a.fmt), gload(a.u + int64_t(f) * a.Na + an));
    });
    wave_lds_sync();
    float2* out = a.grid + q * (N * N);
    static_for<0, 2>([&](auto hc) {
      constexpr int hf = decltype(hc)::value;
      grid_frame_fit(H, epr, stab + hf * S0 * N, hf ? S1 : S0, N, lam);
      wave_lds_sync();
      static_for<0, 16>([&](auto kc) {
        const int y = 4 * decltype(kc)::value + (lam >> 4), x = 2 * (lam & 15);
        const float2 c0 = lds_take(H + y * kHalfPitch + x), c1 = lds_take(H + y * kHalfPitch + x + 1);
        gstore(reinterpret_cast<float4*>(out + y * N + 32 * hf + x), make_float4(c0.x, c0.y, c1.x, c1.y));
      });
      wave_lds_sync();
    });
  }
}

// ---------------------------------------------------------------------------
// Transform + square + accumulate (+ tap).  The samples of a channel are
// divided over a.splits workgroups of eight waves (with one workgroup per
// channel an interval of 64 channels used a quarter of the CUs); with one
// split a workgroup adds its sum to the image itself, with several each
// writes a partial image and k_image_acc_add adds them.  The row transform
// runs first, then the column transform, as in the imaging engines.
// 64 channels x 100 samples at 64 x 64 (210 MB read): 281 -> 86 us.
// ---------------------------------------------------------------------------
constexpr int kAccThreads = 512;

// Sum (FP64) of the workgroup's accumulators (acc[y] of lane x per slot) through
// `red` ([slots][N][N] floats): added to the image, or a partial image.
template <int N, int SLOTS>
__device__ __forceinline__ void acc_reduce(const ImageAccArgs& a, int f, int s, const float (&acc)[N], float* red,
                                           int slot, int lam) {
  __syncthreads();
  static_for<0, N>([&](auto yc) {
    constexpr int y = decltype(yc)::value;
    red[(slot * N + y) * N + lam] = acc[y];
  });
  __syncthreads();
  const float s2 = a.inv_na * a.inv_na;
  for (int idx = threadIdx.x; idx < N * N; idx += kAccThreads) {
    double sum = 0.0;
#pragma unroll
    for (int q = 0; q < SLOTS; ++q) sum += double(red[q * N * N + idx]);
    if (a.splits > 1) a.partial[(int64_t(s) * a.F + f) * (N * N) + idx] = float(sum);
    else a.image[int64_t(f) * N * N + idx] += float(sum) * s2;
  }
}

template <int N>
__device__ __forceinline__ void acc_tap(const ImageAccArgs& a, int f, int t, const float2 (&v)[N], int lam, int kx0,
                                        int ky0) {
  if (a.tap && lam == kx0) {
    float2 p = make_float2(0.f, 0.f);
    static_for<0, N>([&](auto yc) {
      if (decltype(yc)::value == ky0) p = v[decltype(yc)::value];
    });
    a.tap[int64_t(t) * a.F + f] = cscale(p, a.inv_na);
  }
}

// N <= 32: a frame per lane group; lane x loads column x of each row (a run of
// consecutive cells over the lanes) and stores it to the frame's buffer, from
// which each lane takes its row.
template <int N>
__global__ __launch_bounds__(kAccThreads) void k_image_acc(ImageAccArgs a) {
  using G = Geo<N, kAccThreads / 64>;
  constexpr int P = G::PITCH;
  __shared__ float2 lds[G::LDS];
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const int slot = wave * G::FPW + lane / N, lam = lane % N;
  const int f = blockIdx.x % a.F, s = blockIdx.x / a.F;
  const int tb = int(int64_t(a.nt) * s / a.splits), te = int(int64_t(a.nt) * (s + 1) / a.splits);
  float2* buf = lds + slot * G::FRAME;
  const int kx0 = a.k0 ? a.k0[2 * f] : 0, ky0 = a.k0 ? a.k0[2 * f + 1] : 0;
  float acc[N];
  static_for<0, N>([&](auto yc) { acc[decltype(yc)::value] = 0.f; });
  const int iters = (te - tb + G::SLOTS - 1) / G::SLOTS;
  for (int it = 0; it < iters; ++it) {
    const int t = tb + it * G::SLOTS + slot;
    const bool active = t < te;
    const float2* in = a.grid + (int64_t(active ? t : tb) * a.F + f) * (N * N);
    float2 v[N];
    static_for<0, N>([&](auto yc) {
      constexpr int y = decltype(yc)::value;
      v[y] = active ? gload(in + y * N + lam) : make_float2(0.f, 0.f);
    });
    static_for<0, N>([&](auto yc) { buf[decltype(yc)::value * P + lam] = v[decltype(yc)::value]; });
    wave_lds_sync();
    static_for<0, N>([&](auto xc) { v[decltype(xc)::value] = buf[lam * P + decltype(xc)::value]; });
    fft_reg<N, +1>(v);
    wave_lds_sync();
    static_for<0, N>([&](auto xc) { buf[decltype(xc)::value * P + lam] = v[decltype(xc)::value]; });
    wave_lds_sync();
    static_for<0, N>([&](auto yc) { v[decltype(yc)::value] = buf[lam * P + decltype(yc)::value]; });
    wave_lds_sync();
    fft_reg<N, +1>(v);
    add_norms<N>(acc, v);
    if (active) acc_tap<N>(a, f, t, v, lam, kx0, ky0);
  }
  acc_reduce<N, G::SLOTS>(a, f, s, acc, reinterpret_cast<float*>(lds), slot, lam);
}

// 64 x 64: a frame per wave, transposed twice through the wave's staging area
// (xpose.h): lane x with column x -> lane y with row y -> lane kx.
__global__ __launch_bounds__(kAccThreads) void k_image_acc64(ImageAccArgs a) {
  constexpr int N = 64, W = kAccThreads / 64;
  __shared__ __align__(16) float2 lds[W * kXposeFloat2];
  static_assert(W * N * N * 4 <= W * kXposeFloat2 * 8, "the accumulator reduction reuses the staging areas");
  const int lam = threadIdx.x & 63, wave = wave_index();
  const int f = blockIdx.x % a.F, s = blockIdx.x / a.F;
  const int tb = int(int64_t(a.nt) * s / a.splits), te = int(int64_t(a.nt) * (s + 1) / a.splits);
  float2* T = lds + wave * kXposeFloat2;
  const int kx0 = a.k0 ? a.k0[2 * f] : 0, ky0 = a.k0 ? a.k0[2 * f + 1] : 0;
  float acc[N];
  static_for<0, N>([&](auto yc) { acc[decltype(yc)::value] = 0.f; });
  for (int t = tb + wave; t < te; t += W) {
    int lo = lam;                 // opaque copy: no per-row address held across the frame loop
    asm volatile("" : "+v"(lo));
    const float2* in = a.grid + (int64_t(t) * a.F + f) * (N * N) + lo;
    float2 v[N];
    static_for<0, N>([&](auto yc) { v[decltype(yc)::value] = gload(in + decltype(yc)::value * N); });
    transpose64(v, T, lam);
    fft_reg<N, +1>(v);
    transpose64(v, T, lam);
    fft_reg<N, +1>(v);
    add_norms<N>(acc, v);
    acc_tap<N>(a, f, t, v, lam, kx0, ky0);
  }
  acc_reduce<N, W>(a, f, s, acc, reinterpret_cast<float*>(lds), wave, lam);
}

// image += inv_na^2 sum_s partial (FP64 sum over splits)
__global__ __launch_bounds__(256) void k_image_acc_add(const float* partial, int splits, int64_t per_split,
                                                       float inv_na, float* image) {
  const int64_t i = int64_t(blockIdx.x) * 256 + threadIdx.x;
  if (i >= per_split) return;
  double s = 0.0;
  for (int k = 0; k < splits; ++k) s += double(partial[int64_t(k) * per_split + i]);
  image[i] = float(double(image[i]) + s * (double(inv_na) * double(inv_na)));
}

// ---------------------------------------------------------------------------
// launchers
// ---------------------------------------------------------------------------
template <int N, int APL>
struct LaunchGrid {
  static hipError_t run(const GridArgs& a, hipStream_t s) {
    const int64_t frames = int64_t(a.nt) * a.F;
    if constexpr (N == 64 && (APL == 2 || APL == 4)) {
      if (a.slots_h && a.n_slots_h0 + a.n_slots_h1 <= PairSmem<APL>::TAB_SLOTS) {
        // one workgroup per CU is resident; two frames per wave or more repay the table copy
        const int64_t blocks = std::min<int64_t>((frames + 7) / 8, a.n_cu);
        hipLaunchKernelGGL((k_grid_half<APL>), dim3(unsigned(blocks)), dim3(kPairThreads), 0, s, a);
        return hipGetLastError();
      }
    }
    const int slots = Geo<N>::SLOTS;
    hipLaunchKernelGGL((k_grid<N, APL>), dim3(unsigned((frames + slots - 1) / slots)), dim3(256), 0, s, a);
    return hipGetLastError();
  }
};

hipError_t launch_grid(int N, const GridArgs& a, hipStream_t s) {
  if (a.nt == 0) return hipSuccess;
  return dispatch_n<LaunchGrid>(N, a.Na, a, s);
}

// Time splits per channel: the split count with the fewest rounds of frames
// over the CUs (a workgroup takes `slots` frames at a time and its set-up and
// reduction cost about as much as one more), within the workspace.
int image_acc_splits(int N, int F, int nt, int n_cu) {
  const int slots = 8 * (64 / N);
  const int64_t resident = int64_t(n_cu) * (N == 16 ? 2 : 1);
  int best = 1;
  int64_t cost = std::numeric_limits<int64_t>::max();
  for (int s = 1; int64_t(s) * slots < int64_t(nt) + slots && (s == 1 || int64_t(s) * F <= kAccMaxPartials); ++s) {
    const int64_t rounds = (int64_t(F) * s + resident - 1) / resident;
    const int64_t steps = ((nt + s - 1) / s + slots - 1) / slots;
    if (rounds * (steps + 1) < cost) {
      cost = rounds * (steps + 1);
      best = s;
    }
  }
  return best;
}

hipError_t launch_image_acc(int N, const ImageAccArgs& a, hipStream_t s) {
  if (a.nt == 0) return hipSuccess;
  const dim3 grid(unsigned(a.F) * unsigned(a.splits)), block(kAccThreads);
  if (N == 16) hipLaunchKernelGGL((k_image_acc<16>), grid, block, 0, s, a);
  else if (N == 32) hipLaunchKernelGGL((k_image_acc<32>), grid, block, 0, s, a);
  else if (N == 64) hipLaunchKernelGGL(k_image_acc64, grid, block, 0, s, a);
  else return hipErrorInvalidValue;
  hipError_t e = hipGetLastError();
  if (e != hipSuccess || a.splits == 1) return e;
  const int64_t per = int64_t(a.F) * N * N;
  hipLaunchKernelGGL(k_image_acc_add, dim3(unsigned((per + 255) / 256)), dim3(256), 0, s, a.partial, a.splits, per,
                     a.inv_na, a.image);
  return hipGetLastError();
}

}  // namespace epic
