// EPICal calibration solve of one channel for integer E-fields (ci4, ci8; up to
// 1024 antennas) on the matrix cores.
//
// The tap P(t) = sum_a c_a E_a(t) and the correlation K_a = sum_t E_a(t) P(t)*
// are contractions of FP64 numbers with samples of at most eight bits.  Both
// run as exact integer products: the FP64 factor is scaled by the power of two
// that brings the largest of its kind (c over the antennas, P over the samples
// of a chunk) to 61 bits, rounded to a 64-bit integer and written as eight
// signed base-256 digits, and v_mfma_i32_16x16x64_i8 multiplies 16 digit rows
// (eight of the real, eight of the imaginary part) with the packed samples:
//   tap          rows = digits of (c_re, -c_im) and (c_im, c_re) interleaved as
//                the samples' (re, im) bytes are, contraction over the bytes of
//                a sample row, columns = 16 samples;
//   correlation  rows = digits of P_re and P_im, contraction over 64 samples,
//                columns = 16 bytes (two antennas in four lanes' columns).
// The digit sums are exact in int32 and meet in FP64 at the end, so a sum is
// rounded once where an FP64 sum rounds at every term.  Its factors are rounded
// to 2^-61 of the largest of them.  That is no less than FP64 keeps of a sum in
// which the largest takes part, but an antenna without a signal multiplies zeros
// only, while its c grows by 1 / gamma per interval (K = Q = 0, g' = gamma g) and
// would take every digit from the others' coefficients.  So an antenna whose
// samples of the last interval were all zero is left out (its term is zero), and if
// it has a sample after all, the interval is done again in FP64
// (solve_channel_fmt), as are all after it; likewise where the c of the antennas
// with a signal spread by more than 2^12 (kDigitSpan; a cold start of the HERA
// shape passes through 2^11), which bounds what an antenna that falls silent takes
// from the others in that interval.  (Keeping to 2^8 with all antennas in the scale
// sent a few channels of that start to FP64, its solve 0.31 -> 0.53 ms, and every
// run with a silent antenna, 100 intervals of 256 antennas ci4 450 -> 767 us.)
//   What remains per interval is latency: five barriers, the digits and the
// update.
// Largest error of P over the largest |P| against exact sums: 16 antennas 6.5e-17
// (FP64 sums 1.5e-16), 256 6.6e-17 (3.3e-16), 900 8.6e-17 (4.6e-16).
// 64 channels, 50 intervals, per interval, FP64 FMAs (four per sample in each
// contraction, after two conversions) against this:
//   intervals of 100: 256 antennas ci4 7.6 -> 4.6 us, 255 ci8 (rows of no
//   alignment) 28.5 -> 5.0, 350 ci8 19.1 -> 7.6, 900 ci8 51 -> 26;
//   of 25: 3.5 -> 3.6, 9.1 -> 4.1, 6.8 -> 4.2, 13.9 -> 7.7.
#pragma once
#include "solve.h"

namespace epic {

typedef int ivec4 __attribute__((ext_vector_type(4)));
typedef gvec4 gvec4_u __attribute__((aligned(1)));   // unaligned global load

constexpr int kSolveIntMaxAnt = 1024;
constexpr int64_t kSolveIntMinSamples = 20;   // of an interval
constexpr int kSolveIntRows = 128;          // samples of a chunk at most
constexpr int kRowBytes = 80;                // a block's row in the LDS: 64 bytes, padded
constexpr int kDigitSpan = 12;               // exponents of the c of an interval
constexpr uint32_t kStop = 0xffffffffu;      // in place of the largest |c| or |P| (abs_hi): not by this solve
constexpr int kDigitBlock = 16 * 16 + 16;   // bytes: 16 digit rows x 16 contraction entries, padded

struct SolveIntSmem {
  static constexpr int CH_BYTES = 8 * kSolveIntRows * kRowBytes;                // sample rows
  static constexpr int AD_OFF = CH_BYTES;                                       // digits of c
  static constexpr int PD_OFF = AD_OFF + 2 * kSolveIntMaxAnt / 16 * kDigitBlock;   // digits of P
  static constexpr int P_OFF = PD_OFF + kSolveIntRows / 16 * kDigitBlock;       // P [rows][2]
  static constexpr int K_OFF = P_OFF + kSolveIntRows * 16;                      // K [antennas]
  static constexpr int Q_OFF = K_OFF + kSolveIntMaxAnt * 16;                    // Q [antennas]
  static constexpr int MX_OFF = Q_OFF + kSolveIntMaxAnt * 8;                    // largest |c|, |P| per wave
  static constexpr int BYTES = MX_OFF + 64;
};

// Largest x over the wave, in lane 63.
__device__ __forceinline__ uint32_t wave_max63(uint32_t x) {
  auto dpp = [](uint32_t v, auto ctrl, auto mask) {
    return uint32_t(__builtin_amdgcn_update_dpp(0, int(v), decltype(ctrl)::value, decltype(mask)::value, 0xf, true));
  };
  using std::integral_constant;
  x = max(x, dpp(x, integral_constant<int, 0x111>{}, integral_constant<int, 0xf>{}));
  x = max(x, dpp(x, integral_constant<int, 0x112>{}, integral_constant<int, 0xf>{}));
  x = max(x, dpp(x, integral_constant<int, 0x114>{}, integral_constant<int, 0xf>{}));
  x = max(x, dpp(x, integral_constant<int, 0x118>{}, integral_constant<int, 0xf>{}));
  x = max(x, dpp(x, integral_constant<int, 0x142>{}, integral_constant<int, 0xa>{}));
  x = max(x, dpp(x, integral_constant<int, 0x143>{}, integral_constant<int, 0xc>{}));
  return x;
}

// High word of |x|: orders magnitudes, its exponent field in bits 20..30.
__device__ __forceinline__ uint32_t abs_hi(double x) { return uint32_t(__double_as_longlong(x) >> 32) & 0x7fffffffu; }

// The largest of the eight waves' entries.
__device__ __forceinline__ uint32_t max8(const uint32_t* mx) {
  const uint4 u = *reinterpret_cast<const uint4*>(mx), v = *reinterpret_cast<const uint4*>(mx + 4);
  return __builtin_amdgcn_readfirstlane(max(max(max(u.x, u.y), max(u.z, u.w)), max(max(v.x, v.y), max(v.z, v.w))));
}

// Scale exponent that brings values up to `hi` (abs_hi) to 61 bits.
__device__ __forceinline__ int digit_scale(uint32_t hi) { return 1083 - max(int(hi >> 20), 1); }

// x 2^sc rounded to an integer, and an integer as eight signed base-256 digits
// (byte i: digit i).
__device__ __forceinline__ long long fixed_point(double x, int sc) { return static_cast<long long>(rint(ldexp(x, sc))); }
__device__ __forceinline__ unsigned long long digits(long long i) {
  constexpr unsigned long long off = 0x8080808080808080ull;
  return (static_cast<unsigned long long>(i) + off) ^ off;
}

// Digit sums d[0..3] of a lane as sum_i d_i 256^i (exact: below 2^52).
__device__ __forceinline__ double digit_sum(ivec4 d) {
  return fma(fma(fma(double(d[3]), 256.0, double(d[2])), 256.0, double(d[1])), 256.0, double(d[0]));
}

// Returns the number of intervals solved: n_int, or fewer where the next one is
// left to the FP64 solve (the gains are then those at its start; its u is written).
template <int FMT, int J, bool PUBLISH>
__device__ __forceinline__ int solve_channel_int(const SolveArgs& a, int f, uint8_t* smem, int* progress = nullptr) {
  static_assert(FMT == kCI4 || FMT == kCI8, "integer samples");
  using L = SolveIntSmem;
  constexpr int T = kSolveMainThreads, W = T / 64;
  constexpr int NP = FMT == kCI4 ? 5 : 7;      // 16-byte pieces of a chunk per thread
  constexpr int XS = FMT == kCI4 ? 4 : 0;       // 4-bit samples are held as bytes times 16
  const int tid = threadIdx.x, lane = tid & 63, wave = wave_index();
  const int m16 = lane & 15, g16 = lane >> 4;
  const int Na = a.Na, RB = FMT == kCI4 ? Na : 2 * Na;
  const int nk = (2 * Na + 63) / 64;                                // blocks of 64 bytes (32 antennas)
  const int PR = (RB + 15) / 16;                                    // pieces per row
  const int RC = min(min(kSolveIntRows, L::CH_BYTES / (kRowBytes * nk)), NP * T / PR);   // rows of a chunk at most
  // The chunk lies block by block, a block row by row: with the rows' stride a
  // constant the correlation's sixteen row reads are immediate offsets from one
  // address.  It reads whole groups of 64 rows: what lies past the chunk's rows
  // is in the LDS and meets zero digits.
  const int BLK = RC * kRowBytes;
  uint8_t* const CH = smem;
  uint8_t* const AD = smem + L::AD_OFF;
  uint8_t* const PD = smem + L::PD_OFF;
  double* const P_l = reinterpret_cast<double*>(smem + L::P_OFF);
  double2* const K_l = reinterpret_cast<double2*>(smem + L::K_OFF);
  double* const Q_l = reinterpret_cast<double*>(smem + L::Q_OFF);
  uint32_t* const mx_c = reinterpret_cast<uint32_t*>(smem + L::MX_OFF);
  uint32_t* const mx_p = mx_c + 8;
  const int64_t rowstride = int64_t(a.F) * RB;
  const uint8_t* const ebase = a.efield + int64_t(f) * RB;

  // chunk copy: pieces tid + T k of the rows, requested a chunk ahead; offsets
  // in the stream (from the chunk's first row; ascending with the row) and in
  // the LDS
  gvec4 v[NP];
  uint32_t src_off[NP], dst_off[NP];
  static_for<0, NP>([&](auto kc) {
    constexpr int k = decltype(kc)::value;
    const int p = tid + T * k, r = int((float(p) + 0.5f) * (1.0f / float(PR))), c = p - r * PR;
    src_off[k] = r < RC ? uint32_t(r) * uint32_t(rowstride) + 16u * uint32_t(c) : 0xffffffffu;   // never a row's
    dst_off[k] = uint32_t(FMT == kCI4 ? c / 2 * BLK + r * kRowBytes + c % 2 * 32 : c / 4 * BLK + r * kRowBytes + c % 4 * 16);
  });
  // A row's last piece reads on into what follows the row in the stream (it
  // meets zero digits); at the stream's very end it is read `over` bytes early
  // and shifted when it is stored.  Pieces past the chunk's last read that one.
  const uint32_t over = uint32_t(16 * PR - RB);
  const int64_t stream = a.n_t * rowstride - int64_t(f) * RB - 16;    // last offset a piece may be read at
  auto last_piece = [&](int nr) { return uint32_t(nr - 1) * uint32_t(rowstride) + 16u * uint32_t(PR - 1); };
  auto request = [&](int64_t t_first, int nr) {
    const uint8_t* base = ebase + t_first * rowstride;
    const uint32_t lim = uint32_t(min(int64_t(last_piece(nr)), stream - t_first * rowstride));
    static_for<0, NP>([&](auto kc) {
      constexpr int k = decltype(kc)::value;
      v[k] = *(const __attribute__((address_space(1))) gvec4_u*)((const __attribute__((address_space(1))) uint8_t*)base +
                                                                 min(src_off[k], lim));
    });
  };
  auto store = [&](int64_t t_first, int nr) {
    const uint32_t end = uint32_t(nr) * uint32_t(rowstride), edge = last_piece(nr);
    if (int64_t(edge) > stream - t_first * rowstride) {     // uniform
      static_for<0, NP>([&](auto kc) {
        constexpr int k = decltype(kc)::value;
        if (src_off[k] == edge) {
          const uint64_t lo = uint64_t(v[k][1]) << 32 | v[k][0], hi = uint64_t(v[k][3]) << 32 | v[k][2];
          const int sh = 8 * int(over);          // 8 .. 120 bits
          const uint64_t l = sh < 64 ? lo >> sh | hi << (64 - sh) : hi >> (sh - 64), h = sh < 64 ? hi >> sh : 0;
          v[k] = gvec4{uint32_t(l), uint32_t(l >> 32), uint32_t(h), uint32_t(h >> 32)};
        }
      });
    }
    static_for<0, NP>([&](auto kc) {
      constexpr int k = decltype(kc)::value;
      if (src_off[k] < end) {
        if constexpr (FMT == kCI8) {
          *reinterpret_cast<gvec4*>(CH + dst_off[k]) = v[k];
        } else {
          uint32_t o[8];
          static_for<0, 4>([&](auto wc) {
            constexpr int w = decltype(wc)::value;
            const uint32_t re = v[k][w] & 0xf0f0f0f0u, im = (v[k][w] << 4) & 0xf0f0f0f0u;
            o[2 * w] = __builtin_amdgcn_perm(im, re, 0x05010400u);
            o[2 * w + 1] = __builtin_amdgcn_perm(im, re, 0x07030602u);
          });
          gvec4* d = reinterpret_cast<gvec4*>(CH + dst_off[k]);
          d[0] = gvec4{o[0], o[1], o[2], o[3]};
          d[1] = gvec4{o[4], o[5], o[6], o[7]};
        }
      }
    });
  };

  double2 g[J], A[J], invD[J];
  double2 At[J];                    // A in the tap: zero for silent antennas
  uint8_t hold[J];
  uint32_t st[J], st_was[J];
  uint32_t heard[J];                // the last interval's samples: 0 if all were zero
  static_for<0, J>([&](auto jc) {
    constexpr int j = decltype(jc)::value;
    const int an = tid + T * j;
    g[j] = A[j] = At[j] = invD[j] = make_double2(0.0, 0.0);
    hold[j] = 0;
    st[j] = st_was[j] = 0u;
    heard[j] = 1u;
    if (an < Na) {
      const int64_t ia = int64_t(f) * Na + an;
      g[j] = gload(a.gains + ia);
      At[j] = A[j] = gload(a.A + ia);
      const double2 D = gload(a.D + ia);
      const double d2 = D.x * D.x + D.y * D.y;
      invD[j] = make_double2(a.na_eff * D.x / d2, -a.na_eff * D.y / d2);
      hold[j] = gload(a.hold + ia);
      gstore(a.g_hist + ia, g[j]);
    }
  });
  // an interval's samples in chunks of as equal lengths as there are: the first
  // `rem` of them base + 1 rows, the others base
  struct Split {
    int len, nch, base, rem;
  };
  auto split = [&](int64_t len) {
    const int n = int(len), nch = (n + RC - 1) / RC;
    return Split{n, nch, n / nch, n % nch};
  };
  const Split last = split(a.n_t - int64_t(a.n_int - 1) * a.t_cal), full = a.n_int > 1 ? split(a.t_cal) : last;
  const double inv_full = 1.0 / double(full.len), inv_last = 1.0 / double(last.len);
  // entries past the last antenna's stay zero
  for (int i = tid; i < ((nk + 3) / 4 * 16 * kDigitBlock) / 4; i += T) reinterpret_cast<uint32_t*>(AD)[i] = 0u;
  const auto rows = [&](const Split& s, int i) { return s.base + (i < s.rem ? 1 : 0); };
  // chunk i of interval n: samples t .. t + nr - 1
  int n = 0, i = 0, nr = rows(a.n_int > 1 ? full : last, 0);
  int64_t t = 0;
  request(t, nr);
  store(t, nr);
  double rr[J];
  uint32_t hc = 0u;
  uint32_t redo = 0u;                    // kStop: an antenna left out of the last interval had a signal
  bool undo = false;
  // one loop over the chunks of all intervals: with a loop over an interval's
  // chunks inside, what the requests compute was hoisted to its front and ran
  // for every interval in the recurrence's way
  while (true) {
    const bool more = n + 1 < a.n_int, ends = i + 1 == (more ? full : last).nch;
    uint32_t mp = 0u;                          // largest |P|, or kStop
    if (i == 0) {
    // c_a = A_a u_a / Na = A_a conj(g_a) r_a, u_a = 1 / g_a (zero for flagged antennas)
    double2 c[J];
    uint32_t m[J], mx = redo;
    static_for<0, J>([&](auto jc) {
      constexpr int j = decltype(jc)::value;
      const int an = tid + T * j;
      rr[j] = recip_nr(a.na_eff * (g[j].x * g[j].x + g[j].y * g[j].y));
      c[j] = zmul(At[j], make_double2(g[j].x * rr[j], -g[j].y * rr[j]));
      if (an >= Na || (hold[j] & kHoldFlagged)) c[j] = make_double2(0.0, 0.0);
      m[j] = max(abs_hi(c[j].x), abs_hi(c[j].y));
      mx = max(mx, m[j]);
      if (an < Na) {
        const double s = a.na_eff * rr[j];   // 1 / |g|^2
        const float2 uf = hold[j] & kHoldFlagged ? make_float2(0.0f, 0.0f) : make_float2(float(g[j].x * s), float(-g[j].y * s));
        float2* up = a.u_hist + (int64_t(n) * a.F + f) * Na + an;
        if constexpr (PUBLISH)
          __hip_atomic_store((__attribute__((address_space(1))) uint64_t*)up, __builtin_bit_cast(uint64_t, uf),
                             __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        else
          gstore(up, uf);
      }
    });
    mx = wave_max63(mx);
    if (lane == 63) mx_c[wave] = mx;
    if constexpr (PUBLISH) asm volatile("s_waitcnt vmcnt(0)" ::: "memory");   // this wave's u stores are done
    __syncthreads();
    hc = max8(mx_c);
    mp = hc == kStop ? kStop : 0u;             // (left below, with the other reason to stop)
    if constexpr (PUBLISH) {
      if (tid == 0 && hc != kStop)
        __hip_atomic_store((__attribute__((address_space(1))) int*)(progress + f), n + 1, __ATOMIC_RELAXED,
                           __HIP_MEMORY_SCOPE_AGENT);
    }
    const bool finite = hc < 0x7ff00000u;      // uniform
    const int sc = digit_scale(hc);
    // a magnitude from 1 to `below` lies under the span
    const uint32_t below = finite && int(hc >> 20) > kDigitSpan ? (((hc >> 20) - kDigitSpan) << 20) - 1u : 0u;
    static_for<0, J>([&](auto jc) {
      constexpr int j = decltype(jc)::value;
      const int an = tid + T * j;
      if (an < Na) {
        if (m[j] - 1u < below) mp = kStop;
        const double x = finite ? c[j].x : 0.0, y = finite ? c[j].y : 0.0;
        const long long iy = fixed_point(y, sc);
        const unsigned long long dx = digits(fixed_point(x, sc)), dy = digits(iy), dn = digits(-iy);
        uint8_t* at = AD + (2 * an / 16) * kDigitBlock + (2 * an) % 16;
        static_for<0, 8>([&](auto ic) {
          constexpr int i = decltype(ic)::value;
          const uint32_t bx = uint32_t(dx >> (8 * i)) & 255u, by = uint32_t(dy >> (8 * i)) & 255u,
                         bn = uint32_t(dn >> (8 * i)) & 255u;
          *reinterpret_cast<uint16_t*>(at + 16 * i) = uint16_t(bx | bn << 8);
          *reinterpret_cast<uint16_t*>(at + 16 * (8 + i)) = uint16_t(by | bx << 8);
        });
      }
    });
    }
    __syncthreads();
    const bool finite = hc < 0x7ff00000u;
    const int sc = digit_scale(hc), nkk = (nr + 63) / 64;
    // the next chunk's samples arrive while this one is worked on
    const int nr_next = !ends ? rows(more ? full : last, i + 1) : more ? rows(n + 2 < a.n_int ? full : last, 0) : 0;
    if (nr_next) request(t + nr, nr_next);
    {
      // taps of 16 samples per wave
      for (int tile = wave; 16 * tile < nr; tile += W) {
        const int r = 16 * tile + m16;
        const uint8_t* bp = CH + r * kRowBytes + 16 * g16;
        const uint8_t* ap = AD + g16 * kDigitBlock + 16 * m16;
        // four products' operands at a time; past the row's end they meet zero digits
        ivec4 d0 = {0, 0, 0, 0}, d1 = {0, 0, 0, 0};
        for (int k0 = 0; k0 < nk; k0 += 4) {
          ivec4 x[4], y[4];
          static_for<0, 4>([&](auto qc) {
            constexpr int q = decltype(qc)::value;
            x[q] = *reinterpret_cast<const ivec4*>(ap + 4 * (k0 + q) * kDigitBlock);
            y[q] = *reinterpret_cast<const ivec4*>(bp + (k0 + q) * BLK);
          });
          d0 = __builtin_amdgcn_mfma_i32_16x16x64_i8(x[0], y[0], d0, 0, 0, 0);
          d1 = __builtin_amdgcn_mfma_i32_16x16x64_i8(x[1], y[1], d1, 0, 0, 0);
          d0 = __builtin_amdgcn_mfma_i32_16x16x64_i8(x[2], y[2], d0, 0, 0, 0);
          d1 = __builtin_amdgcn_mfma_i32_16x16x64_i8(x[3], y[3], d1, 0, 0, 0);
        }
        // lane groups 0..3: low and high digits of the real, of the imaginary part
        const double lo = digit_sum(d0 + d1), hi = __shfl_down(lo, 16);
        double p = ldexp(fma(hi, 4294967296.0, lo), -sc - XS);
        if (!finite) p = __builtin_nan("");
        if ((g16 & 1) == 0 && r < nr) {
          P_l[2 * r + (g16 >> 1)] = p;
          mp = max(mp, abs_hi(p));
        }
      }
      mp = wave_max63(mp);
      if (lane == 63) mx_p[wave] = mp;
      __syncthreads();
      const uint32_t hp = max8(mx_p);
      if (hp == kStop) {                       // uniform
        undo = hc == kStop;
        break;
      }
      const bool pfinite = hp < 0x7ff00000u;
      const int sp = digit_scale(hp);
      {
        // digits of P: four of one component of one sample per thread
        const int t = tid & 127, part = tid >> 7;
        if (t < 64 * nkk) {
          const double p = t < nr && pfinite ? P_l[2 * t + (part >> 1)] : 0.0;
          const uint32_t d = uint32_t(digits(fixed_point(p, sp)) >> (32 * (part & 1)));
          uint8_t* at = PD + (t / 64 * 4 + t / 4 % 4) * kDigitBlock + 64 * part + 4 * (t / 16 % 4) + t % 4;
          static_for<0, 4>([&](auto ic) { at[16 * decltype(ic)::value] = uint8_t(d >> (8 * decltype(ic)::value)); });
        }
      }
      __syncthreads();
      // correlation: 64 bytes (32 antennas) per wave at a time
      for (int cb = wave; cb < nk; cb += W) {
        ivec4 D[4] = {{0, 0, 0, 0}, {0, 0, 0, 0}, {0, 0, 0, 0}, {0, 0, 0, 0}};
        int q[4] = {0, 0, 0, 0};
        static_for<0, kSolveIntRows / 64>([&](auto kc) {
          constexpr int kk = decltype(kc)::value;
          if (kk >= nkk) return;
          const uint8_t* bp = CH + cb * BLK + 4 * g16 * kRowBytes + 4 * m16;
          uint32_t d[16];
          static_for<0, 16>([&](auto jc) {
            constexpr int j = decltype(jc)::value;
            d[j] = *reinterpret_cast<const uint32_t*>(bp + (64 * kk + j / 4 * 16 + j % 4) * kRowBytes);
          });
          const ivec4 pa = *reinterpret_cast<const ivec4*>(PD + (4 * kk + g16) * kDigitBlock + 16 * m16);
          // four rows' dwords to four columns' dwords
          ivec4 B[4];
          static_for<0, 4>([&](auto wc) {
            constexpr int w = decltype(wc)::value;
            const uint32_t l0 = __builtin_amdgcn_perm(d[4 * w + 1], d[4 * w], 0x05010400u),
                           l1 = __builtin_amdgcn_perm(d[4 * w + 3], d[4 * w + 2], 0x05010400u),
                           h0 = __builtin_amdgcn_perm(d[4 * w + 1], d[4 * w], 0x07030602u),
                           h1 = __builtin_amdgcn_perm(d[4 * w + 3], d[4 * w + 2], 0x07030602u);
            B[0][w] = int(__builtin_amdgcn_perm(l1, l0, 0x05040100u));
            B[1][w] = int(__builtin_amdgcn_perm(l1, l0, 0x07060302u));
            B[2][w] = int(__builtin_amdgcn_perm(h1, h0, 0x05040100u));
            B[3][w] = int(__builtin_amdgcn_perm(h1, h0, 0x07060302u));
          });
          if (64 * kk + 64 > nr) {   // uniform: rows past the chunk's do not count in |E|^2
            const int left = nr - (64 * kk + 4 * g16);
            static_for<0, 4>([&](auto wc) {
              constexpr int w = decltype(wc)::value;
              const int cnt = min(max(left - 16 * w, 0), 4);
              const int mask = cnt == 4 ? -1 : (1 << (8 * cnt)) - 1;
              static_for<0, 4>([&](auto ic) { B[decltype(ic)::value][w] &= mask; });
            });
          }
          static_for<0, 4>([&](auto ic) {
            constexpr int b = decltype(ic)::value;
            D[b] = __builtin_amdgcn_mfma_i32_16x16x64_i8(pa, B[b], D[b], 0, 0, 0);
            static_for<0, 4>([&](auto wc) {
              q[b] = __builtin_amdgcn_sdot4(B[b][decltype(wc)::value], B[b][decltype(wc)::value], q[b], false);
            });
          });
        });
        double S[4], Ti[4];
        static_for<0, 4>([&](auto ic) {
          constexpr int b = decltype(ic)::value;
          const double lo = digit_sum(D[b]), hi = __shfl_down(lo, 16);
          S[b] = fma(hi, 4294967296.0, lo);     // lane group 0: with P_re, group 2: with P_im
          Ti[b] = __shfl_down(S[b], 32);
        });
        int q0 = q[0] + q[1], q1 = q[2] + q[3];
        q0 += __shfl_xor(q0, 16);
        q1 += __shfl_xor(q1, 16);
        q0 += __shfl_xor(q0, 32);
        q1 += __shfl_xor(q1, 32);
        if (lane < 16) {
          // K = sum E conj(P): bytes (re, im) of antennas 32 cb + 2 lane, + 1
          const int an = 32 * cb + 2 * lane;
          double2 k0 = make_double2(ldexp(S[0] + Ti[1], -sp - XS), ldexp(S[1] - Ti[0], -sp - XS));
          double2 k1 = make_double2(ldexp(S[2] + Ti[3], -sp - XS), ldexp(S[3] - Ti[2], -sp - XS));
          if (!pfinite) k0 = k1 = make_double2(__builtin_nan(""), __builtin_nan(""));
          double s0 = double(q0) * (FMT == kCI4 ? 1.0 / 256 : 1.0), s1 = double(q1) * (FMT == kCI4 ? 1.0 / 256 : 1.0);
          if (i > 0) {
            const double2 p0 = K_l[an], p1 = K_l[an + 1];
            k0 = make_double2(k0.x + p0.x, k0.y + p0.y);
            k1 = make_double2(k1.x + p1.x, k1.y + p1.y);
            s0 += Q_l[an];
            s1 += Q_l[an + 1];
          }
          K_l[an] = k0;
          K_l[an + 1] = k1;
          Q_l[an] = s0;
          Q_l[an + 1] = s1;
        }
      }
      __syncthreads();
    }
    if (nr_next) store(t + nr, nr_next);
    if (ends) {
    const double inv_n = n + 1 < a.n_int ? inv_full : inv_last;
    static_for<0, J>([&](auto jc) {
      constexpr int j = decltype(jc)::value;
      const int an = tid + T * j;
      if (an < Na) {
        const double2 k = K_l[an];
        const double q = Q_l[an];
        const uint32_t now = abs_hi(q);
        if (heard[j] == 0u && now) redo = kStop;
        heard[j] = now;
        At[j] = now ? A[j] : make_double2(0.0, 0.0);
        st_was[j] = st[j];
        g[j] = epical_step_r(make_double2(k.x * inv_n, k.y * inv_n), q * inv_n, A[j], invD[j], g[j], rr[j], hold[j],
                             a.gamma, &st[j]);
        gstore(a.g_hist + (int64_t(n + 1) * a.F + f) * Na + an, g[j]);
      }
    });
    ++n;
    if (!more) break;
    }
    i = ends ? 0 : i + 1;
    t += nr;
    nr = nr_next;
  }
  if (n == a.n_int) {
    const bool any = __any(redo != 0u);
    if (lane == 63) mx_c[wave] = any;
    __syncthreads();
    undo = max8(mx_c) != 0u;
  }
  if (undo) --n;                         // the last update is void
  static_for<0, J>([&](auto jc) {
    constexpr int j = decltype(jc)::value;
    const int an = tid + T * j;
    if (an < Na) {
      if (undo) {
        g[j] = gload(a.g_hist + (int64_t(n) * a.F + f) * Na + an);
        st[j] = st_was[j];
      }
      gstore(a.gains + int64_t(f) * Na + an, g[j]);
      if (a.status) {
        uint32_t* sp = a.status + int64_t(f) * Na + an;
        gstore(sp, gload(sp) | st[j]);
      }
    }
  });
  __syncthreads();
  return n;
}

// A copy of uniform arguments in scalar registers, for functions that are called.
template <typename T>
__device__ __forceinline__ T uniform_copy(const T& a) {
  static_assert(sizeof(T) % 4 == 0, "word-wise copy");
  T r;
  uint32_t words[sizeof(T) / 4];
  __builtin_memcpy(words, &a, sizeof(T));
  static_for<0, int(sizeof(T) / 4)>([&](auto ic) {
    constexpr int i = decltype(ic)::value;
    words[i] = __builtin_amdgcn_readfirstlane(words[i]);
  });
  __builtin_memcpy(&r, words, sizeof(T));
  return r;
}

// The arguments of the run from interval n on.
__device__ __forceinline__ SolveArgs from_interval(SolveArgs a, int n) {
  const int64_t t = int64_t(n) * a.t_cal, per = int64_t(a.F) * a.Na;
  a.efield += t * per * (a.fmt == kCI4 ? 1 : a.fmt == kCI8 ? 2 : 8);
  a.n_t -= t;
  a.n_int -= n;
  a.u_hist += n * per;
  a.g_hist += n * per;
  return a;
}

}  // namespace epic
