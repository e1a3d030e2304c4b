// 16 x 16 and 32 x 32 FFT imaging engine (work-item body), shared by the
// per-array kernels, the batched persistent kernel and the fused run.
//
// A wave64 holds 64 / N frames at a time, consecutive samples, one per group of
// N lanes, lane lam of a group owning row lam.  As in the 64 x 64 paired
// engine a frame goes through half a frame of LDS: the columns 0..N/2-1 are
// gridded, each lane takes (and clears) its row's half, then the columns
// N/2..N-1; the row FFTs, a transpose through the same half frame one component
// at a time (which leaves it zero), the column FFTs, |X|^2 into registers.
// Waves never wait for each other inside the frame loop.
//
// What bounds it: vector issue and LDS traffic, half and half, once enough
// waves overlap their LDS phases with each other's FFTs.  Half frames let a
// workgroup hold small_waves() waves, three or four per SIMD, where whole frames
// (image_fft.h image_item) leave room for one or two.  Those are kept for
// schedules whose table does not fit here, and in the persistent kernels, whose
// eight waves are two per SIMD either way, for up to 64 antennas at 32 x 32
// (batch_body).
#pragma once
#include "engine.h"
#include "xpose.h"

namespace epic {

template <int N>
struct SmallGeo {
  static constexpr int FPW = 64 / N;          // frames per wave
  static constexpr int HC = N / 2;            // columns of a half frame
  static constexpr int HP = half_pitch(N);    // its pitch (complex values)
  static constexpr int HALF = N * HP;         // float2 per half frame
  static_assert(N * (N + 2) / 2 <= HALF, "the transpose staging reuses the half frame");
};

template <int N, int APL, int W>
struct SmallSmem {
  static constexpr int FRAME = SmallGeo<N>::HALF + APL * N;       // float2 per frame: half frame + E' staging
  static constexpr int WAVE = SmallGeo<N>::FPW * FRAME;
  static constexpr int T_OFF = W * WAVE * 8;                      // bytes: slot table
  static constexpr int TAB_SLOTS = (kLdsBytes - T_OFF) / (N * 8);
  static constexpr int BYTES = T_OFF + TAB_SLOTS * N * 8;
  static_assert(W * SmallGeo<N>::FPW * N * N * 4 <= T_OFF, "the accumulator reduction reuses the wave areas");
};

// Grid the staged frame and transform it: v[ky] = X(kx = lam, ky) Na.  The half
// frame H is zero on entry and on exit.
template <int N>
__device__ __forceinline__ void small_transform(float2 (&v)[N], float2* H, const float2* epr, const uint2* stab,
                                                int S0, int S1, int lam) {
  constexpr int HC = SmallGeo<N>::HC;
  grid_frame_fit(H, epr, stab, S0, N, lam);
  wave_lds_sync();
  take_half_row_n<N, 0>(v, H, lam);
  wave_lds_sync();
  grid_frame_fit(H, epr, stab + S0 * N, S1, N, lam);
  wave_lds_sync();
  take_half_row_n<N, HC>(v, H, lam);
  wave_lds_sync();
  fft_reg<N, +1>(v);
  transpose_lds<N>(v, H, lam);
  fft_reg<N, +1>(v);
}

// The samples t0 + h of a wave's lane groups h: row of the E-field stream
// (repeating the last sample past te).
template <int FMT>
__device__ __forceinline__ const uint8_t* small_row(const uint8_t* efield, int64_t t0, int64_t te, int h, int f, int F,
                                                    int Na) {
  constexpr int bpe = FMT == kCF32 ? 8 : FMT == kCI8 ? 2 : 1;
  const int64_t rowb = int64_t(Na) * bpe;
  const int left = int(min(te - 1 - t0, int64_t(63)));
  return efield + (t0 * F + f) * rowb + int64_t(min(h, left)) * (F * rowb);
}

// The frames [tb, te) of channel f shared by the workgroup's W waves, |X|^2
// added into acc (lane lam = kx, acc[y] = ky, one sum per lane group).
template <int N, int APL, int FMT, int W>
__device__ __forceinline__ void small_frames(const ImageArgs& a, int f, int64_t tb, int64_t te, float (&acc)[N],
                                             float2* H, const uint2* stab, int h, int lam, int wave) {
  using G = SmallGeo<N>;
  constexpr int STEP = W * G::FPW;
  float2* epr = H + G::HALF;
  const int S0 = a.n_slots_h0, S1 = a.n_slots_h1;
  Raw raw[APL];
  auto fetch_raw = [&](int64_t t0) {
    const uint8_t* row = small_row<FMT>(a.efield, t0, te, h, f, a.F, a.Na);
    static_for<0, APL>([&](auto ic) {
      raw[decltype(ic)::value] = load_raw_global(row, min(lam + N * decltype(ic)::value, a.Na - 1), FMT);
    });
  };
  IntervalCursor interval(a.t_cal);
  int64_t t0 = tb + wave * G::FPW;
  if (t0 < te) fetch_raw(t0);
  for (; t0 < te; t0 += STEP) {
    // u of each lane group's interval: the wave's first sample's, plus one per
    // interval end that lies between
    const int64_t n0 = interval.at(t0);
    const int to_end = int(min(interval.end - t0, int64_t(G::FPW))), tc = int(min(a.t_cal, int64_t(G::FPW)));
    int dn = 0;
    static_for<0, G::FPW - 1>([&](auto kc) { dn += h >= to_end + decltype(kc)::value * tc ? 1 : 0; });
    const bool active = t0 + h < te;
    if (!active) dn = 0;
    const float2* urow = a.u + (n0 * a.F + f) * int64_t(a.Na) + int64_t(dn) * (int64_t(a.F) * a.Na);
    float2 uu[APL];
    static_for<0, APL>([&](auto ic) {
      uu[decltype(ic)::value] = gload_at<float2>(urow, 8u * uint32_t(min(lam + N * decltype(ic)::value, a.Na - 1)));
    });
    static_for<0, APL>([&](auto ic) {
      constexpr int i = decltype(ic)::value;
      const float2 e = cmul(unpack_raw(raw[i], FMT), uu[i]);
      epr[lam + N * i] = active ? e : make_float2(0.f, 0.f);
    });
    wave_lds_sync();
    float2 v[N];
    small_transform<N>(v, H, epr, stab, S0, S1, lam);
    fetch_raw(t0 + STEP < te ? t0 + STEP : t0);
    add_norms<N>(acc, v);
  }
}

// Workgroup sum (FP64) of the lane groups' accumulators, times `scale`, into out[N * N];
// the accumulators are zeroed, the half frames left zero.
template <int N, int APL, int W>
__device__ __forceinline__ void small_reduce(float (&acc)[N], float* out, float scale, uint8_t* smem, float2* H, int h,
                                             int lam, int wave) {
  using G = SmallGeo<N>;
  __syncthreads();
  float* red = reinterpret_cast<float*>(smem);
  const int slot = wave * G::FPW + h;
  static_for<0, N>([&](auto yc) {
    red[(slot * N + decltype(yc)::value) * N + lam] = acc[decltype(yc)::value];
    acc[decltype(yc)::value] = 0.f;
  });
  __syncthreads();
  for (int idx = threadIdx.x; idx < N * N; idx += 64 * W) {
    double sum = 0.0;
#pragma unroll 8
    for (int q = 0; q < W * G::FPW; ++q) sum += double(red[q * N * N + idx]);
    gstore(out + idx, float(sum * scale));
  }
  __syncthreads();
  static_for<0, G::HP>([&](auto xc) { H[lam * G::HP + decltype(xc)::value] = make_float2(0.f, 0.f); });
}

// One work item: channel f, time split s; W waves.
template <int N, int APL, int FMT, int W>
__device__ __forceinline__ void image_item_small(const ImageArgs& a, int f, int s, uint8_t* smem) {
  using G = SmallGeo<N>;
  using L = SmallSmem<N, APL, W>;
  const int lane = threadIdx.x & 63, wave = wave_index();
  const int h = lane / N, lam = lane % N;
  float2* H = reinterpret_cast<float2*>(smem) + wave * L::WAVE + h * L::FRAME;
  uint2* stab = reinterpret_cast<uint2*>(smem + L::T_OFF);
  const int64_t tb = a.n_t * s / a.splits, te = a.n_t * (s + 1) / a.splits;
  load_slot_table(stab, a.slots_h, a.n_slots_h0 + a.n_slots_h1, N);
  static_for<0, G::HP>([&](auto xc) { H[lam * G::HP + decltype(xc)::value] = make_float2(0.f, 0.f); });
  __syncthreads();
  float acc[N];
  static_for<0, N>([&](auto yc) { acc[decltype(yc)::value] = 0.f; });
  small_frames<N, APL, FMT, W>(a, f, tb, te, acc, H, stab, h, lam, wave);
  small_reduce<N, APL, W>(acc, a.partial + (int64_t(s) * a.F + f) * (N * N), 1.f, smem, H, h, lam, wave);
  __syncthreads();
}

// Snapshots whose windows the workgroup's waves share, one after another.
template <int N, int APL, int FMT, int W>
__device__ __forceinline__ void image_item_small_snap_group(const ImageArgs& a, int f, int s, uint8_t* smem) {
  using G = SmallGeo<N>;
  using L = SmallSmem<N, APL, W>;
  const int lane = threadIdx.x & 63, wave = wave_index();
  const int h = lane / N, lam = lane % N;
  float2* H = reinterpret_cast<float2*>(smem) + wave * L::WAVE + h * L::FRAME;
  uint2* stab = reinterpret_cast<uint2*>(smem + L::T_OFF);
  const int64_t n_win = (a.n_t + a.t_acc - 1) / a.t_acc;
  const int64_t wb = n_win * s / a.splits, we = n_win * (s + 1) / a.splits;
  load_slot_table(stab, a.slots_h, a.n_slots_h0 + a.n_slots_h1, N);
  static_for<0, G::HP>([&](auto xc) { H[lam * G::HP + decltype(xc)::value] = make_float2(0.f, 0.f); });
  __syncthreads();
  float acc[N];
  static_for<0, N>([&](auto yc) { acc[decltype(yc)::value] = 0.f; });
  for (int64_t j = wb; j < we; ++j) {
    const int64_t t0 = j * a.t_acc, t1 = min(t0 + a.t_acc, a.n_t);
    small_frames<N, APL, FMT, W>(a, f, t0, t1, acc, H, stab, h, lam, wave);
    small_reduce<N, APL, W>(acc, a.snap + (j * a.F + f) * int64_t(N * N), float(a.snap_scale / double(t1 - t0)), smem, H,
                            h, lam, wave);
  }
}

// Snapshots: each lane group takes whole windows in turn (SnapCursor), as in
// the engines of image_fft.h.
template <int N, int APL, int FMT, int W>
__device__ __forceinline__ void image_item_small_snap(const ImageArgs& a, int f, int s, uint8_t* smem) {
  using G = SmallGeo<N>;
  using L = SmallSmem<N, APL, W>;
  constexpr int SLOTS = W * G::FPW;
  constexpr int bpe = FMT == kCF32 ? 8 : FMT == kCI8 ? 2 : 1;
  const int lane = threadIdx.x & 63, wave = wave_index();
  const int h = lane / N, lam = lane % N;
  float2* H = reinterpret_cast<float2*>(smem) + wave * L::WAVE + h * L::FRAME;
  float2* epr = H + G::HALF;
  uint2* stab = reinterpret_cast<uint2*>(smem + L::T_OFF);
  const int S0 = a.n_slots_h0, S1 = a.n_slots_h1;
  const int64_t n_win = (a.n_t + a.t_acc - 1) / a.t_acc;
  const int64_t wb = n_win * s / a.splits, we = n_win * (s + 1) / a.splits;

  load_slot_table(stab, a.slots_h, S0 + S1, N);
  static_for<0, G::HP>([&](auto xc) { H[lam * G::HP + decltype(xc)::value] = make_float2(0.f, 0.f); });
  __syncthreads();

  float acc[N];
  static_for<0, N>([&](auto yc) { acc[decltype(yc)::value] = 0.f; });
  // every lane group of a wave walks the same number of steps (frames past a
  // group's windows are empty)
  const int64_t steps = (max(int64_t(0), we - wb - wave * G::FPW) + SLOTS - 1) / SLOTS * a.t_acc;
  SnapCursor cur{wb + wave * G::FPW + h, 0, we, SLOTS, a.t_acc, a.n_t};
  Raw raw[APL];
  auto fetch_raw = [&](const SnapCursor& c) {
    const uint8_t* row = a.efield + ((c.valid() ? c.t() : 0) * a.F + f) * int64_t(a.Na) * bpe;
    static_for<0, APL>([&](auto ic) {
      raw[decltype(ic)::value] = load_raw_global(row, min(lam + N * decltype(ic)::value, a.Na - 1), FMT);
    });
  };
  IntervalCursor interval(a.t_cal);
  fetch_raw(cur);
  for (int64_t q = 0; q < steps; ++q) {
    const bool active = cur.valid();
    const float2* urow = a.u + ((active ? interval.at(cur.t()) : 0) * a.F + f) * int64_t(a.Na);
    float2 uu[APL];
    static_for<0, APL>([&](auto ic) {
      uu[decltype(ic)::value] = gload_at<float2>(urow, 8u * uint32_t(min(lam + N * decltype(ic)::value, a.Na - 1)));
    });
    static_for<0, APL>([&](auto ic) {
      constexpr int i = decltype(ic)::value;
      const float2 e = cmul(unpack_raw(raw[i], FMT), uu[i]);
      epr[lam + N * i] = active ? e : make_float2(0.f, 0.f);
    });
    wave_lds_sync();
    float2 v[N];
    small_transform<N>(v, H, epr, stab, S0, S1, lam);
    SnapCursor nxt = cur;
    nxt.next();
    fetch_raw(nxt);
    add_norms<N>(acc, v);
    if (active && cur.last()) snap_store<N>(a, f, cur.j, acc, lam);
    cur = nxt;
  }
  __syncthreads();
}

}  // namespace epic
