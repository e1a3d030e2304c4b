// HIP kernels (gfx950) for the EPIC direct-imaging loop with EPICal.
//
// Layout of the imaging engine ("one lane = one pencil"): a wave64 owns
// 64 / N frames of an N x N grid (N <= 64); lane lam of a frame owns grid row
// lam.  Per frame:
//   1. calibrate + grid (Sec. 2.1, E'_a = E_a / g_a and eq. gridding): each
//      lane stages antennas lam, lam + N, ... as E' in LDS, then sums the
//      contributions of the grid cells it owns (a fixed schedule built on the
//      host) and stores them into the frame's LDS buffer;
//   2. lane lam loads row lam into registers and runs an N-point FFT there;
//   3. the row spectrum is written transposed to LDS (lane-consecutive
//      addresses, conflict free) and lane lam reads back column lam (rows of
//      the buffer are padded by two complex values to spread banks), zeroing
//      the buffer for the next frame as it goes;
//   4. an N-point FFT over the other axis gives X(kx = lam, ky), whose |X|^2
//      is accumulated in registers over all frames of the wave (squaring and
//      time averaging, Sec. 2.1).
// Waves of one workgroup share a channel and split its samples; their
// accumulators are summed through LDS into one partial image per workgroup.
//
// The calibration solve runs in its own kernel before imaging: the tapped
// pixel of interval n only needs the gains of interval n, and its value
// X_t(k0) equals the beamformed sum (1/Na) sum_a A_a(k0) u_a E_a(t) (the
// transform of the gridded field evaluated at one pixel), so the feedback
// recursion costs O(Na) per sample and the O(Ng log Ng) imaging of every
// sample becomes independent work.
#include "image_cls.h"
#include "image_fft.h"
#include "image_small.h"

namespace epic {

// ---------------------------------------------------------------------------
// Fused imaging kernel
// ---------------------------------------------------------------------------
template <int N, int APL>
__global__ __launch_bounds__(256) void k_image(ImageArgs a) {
  __shared__ __align__(16) uint8_t smem[FftSmem<N, APL>::BYTES];
  image_item<N, APL>(a, blockIdx.x % a.F, blockIdx.x / a.F, smem);
}

template <int N, int APL, int FMT>
__global__ __launch_bounds__(64 * small_waves(N, APL)) void k_image_small(ImageArgs a) {
  constexpr int W = small_waves(N, APL);
  __shared__ __align__(16) uint8_t smem[SmallSmem<N, APL, W>::BYTES];
  image_item_small<N, APL, FMT, W>(a, blockIdx.x % a.F, blockIdx.x / a.F, smem);
}

template <int N, int APL, int FMT>
__global__ __launch_bounds__(64 * small_waves(N, APL)) void k_image_small_snap(ImageArgs a) {
  constexpr int W = small_waves(N, APL);
  __shared__ __align__(16) uint8_t smem[SmallSmem<N, APL, W>::BYTES];
  image_item_small_snap<N, APL, FMT, W>(a, blockIdx.x % a.F, blockIdx.x / a.F, smem);
}

template <int N, int APL, int FMT>
__global__ __launch_bounds__(64 * small_waves(N, APL)) void k_image_small_snap_group(ImageArgs a) {
  constexpr int W = small_waves(N, APL);
  __shared__ __align__(16) uint8_t smem[SmallSmem<N, APL, W>::BYTES];
  image_item_small_snap_group<N, APL, FMT, W>(a, blockIdx.x % a.F, blockIdx.x / a.F, smem);
}

template <int APL, int FMT>
__global__ __launch_bounds__(kPairThreads) void k_image_pair(ImageArgs a) {
  static_assert(APL == 2 || APL == 4, "instantiated for the register budget checked at two and four antennas per lane");
  __shared__ __align__(16) uint8_t smem[PairSmem<APL>::BYTES];
  image_item_pair<APL, FMT>(a, blockIdx.x % a.F, blockIdx.x / a.F, smem);
}

// Snapshot forms (one image per window of t_acc samples).
template <int N, int APL>
__global__ __launch_bounds__(256) void k_image_snap(ImageArgs a) {
  __shared__ __align__(16) uint8_t smem[FftSmem<N, APL>::BYTES];
  image_item_snap<N, APL>(a, blockIdx.x % a.F, blockIdx.x / a.F, smem);
}

template <int APL, int FMT>
__global__ __launch_bounds__(kPairThreads) void k_image_pair_snap(ImageArgs a) {
  static_assert(APL == 2 || APL == 4, "instantiated for the register budget checked at two and four antennas per lane");
  __shared__ __align__(16) uint8_t smem[PairSmem<APL>::BYTES];
  image_item_pair_snap<APL, FMT>(a, blockIdx.x % a.F, blockIdx.x / a.F, smem);
}

template <int APL, int FMT>
__global__ __launch_bounds__(kPairThreads) void k_image_pair_snap_group(ImageArgs a) {
  static_assert(APL == 2 || APL == 4, "instantiated for the register budget checked at two and four antennas per lane");
  __shared__ __align__(16) uint8_t smem[PairSmem<APL>::BYTES];
  image_item_pair_snap_group<APL, FMT>(a, blockIdx.x % a.F, blockIdx.x / a.F, smem);
}

template <int R, int FMT, bool DB>
__global__ __launch_bounds__(kClsPairThreads) void k_image_cls_pair(ImageArgs a) {
  __shared__ __align__(16) uint8_t smem[ClsPairSmem<R, DB>::BYTES];
  constexpr int CG = (R * R) / 4;
  const int rest = blockIdx.x / a.F;
  image_cls_pair_item<R, FMT, DB>(a, blockIdx.x % a.F, rest % CG, rest / CG, smem);
}

template <int R, int FMT, int GB>
__global__ __launch_bounds__(kClsDenseThreads) void k_image_cls_dense(ImageArgs a) {
  __shared__ __align__(16) uint8_t smem[ClsDenseSmem<R>::BYTES];
  constexpr int CG = (R * R) / ClsDenseSmem<R>::CPW;
  const int rest = blockIdx.x / a.F;
  image_cls_dense_item<R, FMT, GB>(a, blockIdx.x % a.F, rest % CG, rest / CG, smem);
}

template <int R>
__global__ __launch_bounds__(256) void k_image_cls_big(ImageArgs a) {
  __shared__ __align__(16) uint8_t smem[ClsBigSmem<R>::BYTES];
  constexpr int CG = (R * R) / 4;
  const int rest = blockIdx.x / a.F;
  image_cls_big_item<R>(a, blockIdx.x % a.F, rest % CG, rest / CG, smem);
}

// ---------------------------------------------------------------------------
// Partial-image reduction (FP64 sum over splits)
// ---------------------------------------------------------------------------
__global__ __launch_bounds__(256) void k_reduce(const float* partial, int splits, int64_t per_split,
                                                double scale, float* image) {
  const int64_t i = int64_t(blockIdx.x) * 256 + threadIdx.x;
  if (i >= per_split) return;
  image[i] = float(partial_sum(partial + i, splits, per_split) * scale);
}

// ---------------------------------------------------------------------------
// Integer E-field samples decoded by the imaging path's own unpacking
// (load_raw_global + unpack_raw), written as int16 (re, im) pairs
// ---------------------------------------------------------------------------
__global__ __launch_bounds__(256) void k_unpack(const uint8_t* efield, int64_t n, int fmt, short2* out) {
  const int64_t i = int64_t(blockIdx.x) * 256 + threadIdx.x;
  if (i >= n) return;
  const float2 v = unpack_raw(load_raw_global(efield + i * efmt_bytes(fmt), 0, fmt), fmt);
  out[i] = make_short2(short(v.x), short(v.y));
}


// ---------------------------------------------------------------------------
// launchers
// ---------------------------------------------------------------------------
hipError_t launch_unpack(const uint8_t* efield, int64_t n, int fmt, int16_t* out, hipStream_t s) {
  if (n == 0) return hipSuccess;
  if (fmt != kCI4 && fmt != kCI8) return hipErrorInvalidValue;
  hipLaunchKernelGGL(k_unpack, dim3(unsigned((n + 255) / 256)), dim3(256), 0, s, efield, n, fmt,
                     reinterpret_cast<short2*>(out));
  return hipGetLastError();
}

int grid_lanes(int N) { return N; }
int grid_pitch(int N) { return N + 2; }

bool image_supported(int N, int na, int n_slots) {
  if (N == 128 || N == 256) return na <= kClsMaxAntBig;
  if (!(N == 16 || N == 32 || N == 64) || na > 8 * N) return false;
  const int apl = apl_for(N, na);
  return apl != 0 && n_slots <= tab_slots_for(N, apl);
}

// The paired 64 x 64 engine: up to 256 antennas (two or four per lane: the
// register budget of two waves per SIMD is checked there), and a half-frame
// schedule that fits its LDS table.
bool pair_engine(const ImageArgs& a, int N) {
  const int apl = apl_for(N, a.Na);
  return N == 64 && (apl == 2 || apl == 4) && a.slots_h != nullptr &&
         a.n_slots_h0 + a.n_slots_h1 <= (apl == 2 ? PairSmem<2>::TAB_SLOTS : PairSmem<4>::TAB_SLOTS);
}

// The 16 x 16 / 32 x 32 engine: half-frame schedules that fit its LDS table
// (any but extreme layouts, dozens of antennas on one cell).
template <int N>
static int small_table_slots(int apl, int waves) {
  const bool own = waves == 0;
  switch (apl) {
    case 2: return own ? SmallSmem<N, 2, small_waves(N, 2)>::TAB_SLOTS : SmallSmem<N, 2, kSmallBodyWaves>::TAB_SLOTS;
    case 4: return own ? SmallSmem<N, 4, small_waves(N, 4)>::TAB_SLOTS : SmallSmem<N, 4, kSmallBodyWaves>::TAB_SLOTS;
    case 8: return own ? SmallSmem<N, 8, small_waves(N, 8)>::TAB_SLOTS : SmallSmem<N, 8, kSmallBodyWaves>::TAB_SLOTS;
    default: return 0;
  }
}

int small_apl(int N, int na) { return apl_for(N, na); }

bool small_engine(const ImageArgs& a, int N, int waves) {
  if (!(N == 16 || N == 32) || !a.slots_h) return false;
  const int apl = apl_for(N, a.Na);
  return a.n_slots_h0 + a.n_slots_h1 <= (N == 16 ? small_table_slots<16>(apl, waves) : small_table_slots<32>(apl, waves));
}

template <int N, int APL>
struct LaunchImage {
  static hipError_t run(const ImageArgs& a, hipStream_t s) {
    if constexpr (N <= 32) {
      if (small_engine(a, N)) {
        with_format(a.fmt, [&](auto fc) {
          hipLaunchKernelGGL((k_image_small<N, APL, decltype(fc)::value>), dim3(a.F * a.splits),
                             dim3(64 * small_waves(N, APL)), 0, s, a);
        });
        return hipGetLastError();
      }
    }
    if constexpr (N == 64 && (APL == 2 || APL == 4)) {
      if (pair_engine(a, N)) {
        with_format(a.fmt, [&](auto fc) {
          constexpr int FMT = decltype(fc)::value;
          hipLaunchKernelGGL((k_image_pair<APL, FMT>), dim3(a.F * a.splits), dim3(kPairThreads), 0, s, a);
        });
        return hipGetLastError();
      }
    }
    hipLaunchKernelGGL((k_image<N, APL>), dim3(a.F * a.splits), dim3(256), 0, s, a);
    return hipGetLastError();
  }
};

// The residue-class engine with two waves per SIMD: at most 512 antennas,
// half-frame schedules that fit its LDS table; with at most kClsPairMaxAntDB
// antennas and a table that still fits, its double-buffered form (one barrier
// per pair of samples).
bool cls_pair_db(const ImageArgs& a, int N) {
  const int cap = N == 128 ? ClsPairSmem<2, true>::TAB_SLOTS : ClsPairSmem<4, true>::TAB_SLOTS;
  return a.Na <= kClsPairMaxAntDB && a.n_slots_h0 + a.n_slots_h1 <= cap;
}

bool cls_pair_engine(const ImageArgs& a, int N) {
  if (!(N == 128 || N == 256) || a.Na > kClsMaxAnt || !a.slots_h || a.grid_batch != 0) return false;
  const int cap = N == 128 ? ClsPairSmem<2>::TAB_SLOTS : ClsPairSmem<4>::TAB_SLOTS;
  return a.n_slots_h0 + a.n_slots_h1 <= cap;
}

// The dense residue-class engine with two waves per SIMD: up to 2048 antennas
// at 256 x 256 and 1024 at 128 x 128 (its E' staging of one or two frames); by
// default the arrays the class-pair engine does not take, any of them when a
// gridding batch is chosen (grid_batch 2 or 4).
bool cls_dense_engine(const ImageArgs& a, int N) {
  if (!(N == 128 || N == 256) || !a.slots_m || cls_pair_engine(a, N)) return false;
  return a.Na <= (N == 256 ? ClsDenseSmem<4>::MAXA : ClsDenseSmem<2>::MAXA);
}

int cls_groups(const ImageArgs& a, int N) {
  if (N == 256) return cls_dense_engine(a, N) ? 16 / ClsDenseSmem<4>::CPW : 4;
  return 1;
}

// The residue-class engines (R = N / 64): the class-pair engine, the dense
// one, and for what neither takes (128 x 128 above 1024 antennas) the one-wave
// engine.
template <int R>
static hipError_t launch_image_cls(const ImageArgs& a, hipStream_t s) {
  constexpr int N = 64 * R;
  const dim3 grid(a.F * cls_groups(a, N) * a.splits);
  if (cls_dense_engine(a, N)) {
    with_format(a.fmt, [&](auto fc) {
      constexpr int FMT = decltype(fc)::value;
      if (a.grid_batch == 4) hipLaunchKernelGGL((k_image_cls_dense<R, FMT, 4>), grid, dim3(kClsDenseThreads), 0, s, a);
      else hipLaunchKernelGGL((k_image_cls_dense<R, FMT, 2>), grid, dim3(kClsDenseThreads), 0, s, a);
    });
  } else if (cls_pair_engine(a, N)) {
    with_format(a.fmt, [&](auto fc) {
      constexpr int FMT = decltype(fc)::value;
      if (cls_pair_db(a, N)) hipLaunchKernelGGL((k_image_cls_pair<R, FMT, true>), grid, dim3(kClsPairThreads), 0, s, a);
      else hipLaunchKernelGGL((k_image_cls_pair<R, FMT, false>), grid, dim3(kClsPairThreads), 0, s, a);
    });
  } else if constexpr (R == 2) {
    hipLaunchKernelGGL((k_image_cls_big<R>), grid, dim3(256), 0, s, a);
  } else {
    return hipErrorInvalidValue;
  }
  return hipGetLastError();
}

hipError_t launch_image(int N, const ImageArgs& a, hipStream_t s) {
  if (N == 128) return launch_image_cls<2>(a, s);
  if (N == 256) return launch_image_cls<4>(a, s);
  return dispatch_n<LaunchImage>(N, a.Na, a, s);
}

template <int N, int APL>
struct LaunchImageSnap {
  static hipError_t run(const ImageArgs& a, hipStream_t s) {
    if constexpr (N <= 32) {
      if (small_engine(a, N)) {
        with_format(a.fmt, [&](auto fc) {
          constexpr int FMT = decltype(fc)::value;
          const dim3 grid(a.F * a.splits), block(64 * small_waves(N, APL));
          if (a.snap_group) hipLaunchKernelGGL((k_image_small_snap_group<N, APL, FMT>), grid, block, 0, s, a);
          else hipLaunchKernelGGL((k_image_small_snap<N, APL, FMT>), grid, block, 0, s, a);
        });
        return hipGetLastError();
      }
    }
    if constexpr (N == 64 && (APL == 2 || APL == 4)) {
      if (pair_engine(a, N)) {
        const dim3 grid(a.F * a.splits), block(kPairThreads);
        with_format(a.fmt, [&](auto fc) {
          constexpr int FMT = decltype(fc)::value;
          if (a.snap_group) hipLaunchKernelGGL((k_image_pair_snap_group<APL, FMT>), grid, block, 0, s, a);
          else hipLaunchKernelGGL((k_image_pair_snap<APL, FMT>), grid, block, 0, s, a);
        });
        return hipGetLastError();
      }
    }
    hipLaunchKernelGGL((k_image_snap<N, APL>), dim3(a.F * a.splits), dim3(256), 0, s, a);
    return hipGetLastError();
  }
};

hipError_t launch_image_snap(int N, const ImageArgs& a, hipStream_t s) {
  if (N > 64 || a.t_acc < 1 || !a.snap || a.splits < 1) return hipErrorInvalidValue;
  return dispatch_n<LaunchImageSnap>(N, a.Na, a, s);
}

hipError_t launch_reduce(const float* partial, int splits, int64_t per_split, double scale, float* image,
                         hipStream_t s) {
  const int64_t blocks = (per_split + 255) / 256;
  hipLaunchKernelGGL(k_reduce, dim3(unsigned(blocks)), dim3(256), 0, s, partial, splits, per_split, scale,
                     image);
  return hipGetLastError();
}

}  // namespace epic
