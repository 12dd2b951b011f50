// L1 iteration-level detection over per-rank step times (paper section 6.1
// and Appendix B): sliding-window ratio-gated jitter detection with
// effective-width measurement, and full-scan change-point detection; the two
// together classify a rank's series as stable, jitter, regression or both.
//
// One 64-lane wavefront per rank. The series lives in LDS; per-point marks
// (covered by a candidate window, above the baseline) are 64-bit ballot
// words, so merged intervals and longest runs come from bit operations; the
// baseline median is a wavefront radix select. For the change point each lane
// walks a run of consecutive splits with running sums, and the squares are
// summed only for ranks where some split's ratio is large enough. Decisions
// are integer comparisons, by 128- and 256-bit products only where doubles
// cannot tell.
//
// What bounds it: instruction issue and LDS latency at four wavefronts per
// SIMD (10 KB of LDS each at 1,024 steps). With every prefix sum kept in LDS
// (42 KB) three wavefronts shared a CU: 10,240 ranks x 1,000 steps took 570 us,
// 110 us now (92 MB: 0.84 TB/s); 5,000 x 2,000 1,350 -> 165 us, 10,240 x 60
// 36 -> 21 us.
#include "argus_internal.h"

namespace argus {
namespace {

typedef unsigned __int128 u128;
constexpr int64_t kYLimit = (int64_t)1 << 40;

// a * b as a 256-bit (hi, lo) pair
__device__ __forceinline__ void mul_128x128(u128 a, u128 b, u128& hi, u128& lo) {
  const uint64_t a0 = (uint64_t)a, a1 = (uint64_t)(a >> 64), b0 = (uint64_t)b, b1 = (uint64_t)(b >> 64);
  const u128 p00 = (u128)a0 * b0, p01 = (u128)a0 * b1, p10 = (u128)a1 * b0, p11 = (u128)a1 * b1;
  const u128 mid = (p00 >> 64) + (uint64_t)p01 + (uint64_t)p10;
  lo = (u128)(uint64_t)p00 | (mid << 64);
  hi = p11 + (p01 >> 64) + (p10 >> 64) + (mid >> 64);
}

// sign of a*b - c*d
__device__ __forceinline__ int cmp_prod(u128 a, u128 b, u128 c, u128 d) {
  u128 h1, l1, h2, l2;
  mul_128x128(a, b, h1, l1);
  mul_128x128(c, d, h2, l2);
  if (h1 != h2) return h1 < h2 ? -1 : 1;
  if (l1 != l2) return l1 < l2 ? -1 : 1;
  return 0;
}

// Doubles below carry at most six roundings (relative error below 1e-15):
// where two products lie further apart than kBand they decide the comparison.
constexpr double kBand = 1e-13;

// sample (n-1) relative std <= cmax_pm / 1000, exactly (n >= 1)
__device__ __forceinline__ bool rel_std_ok(int64_t n, u128 s, u128 q, int32_t cmax_pm) {
  const u128 v = (u128)n * q - s * s;
  const double lhs = 1e6 * (double)n * u128_to_f64(v), sd = (double)(uint64_t)s;
  const double rhs = (double)cmax_pm * (double)cmax_pm * (double)(n - 1) * sd * sd;
  if (lhs < rhs * (1.0 - kBand)) return true;
  if (lhs > rhs * (1.0 + kBand)) return false;
  return cmp_prod((u128)1000000u * (u128)n, v, (u128)cmax_pm * (u128)cmax_pm * (u128)(n - 1), s * s) <= 0;
}

// inclusive prefix over the wavefront of a 128-bit value
__device__ __forceinline__ u128 wave_incl_scan128(u128 v) {
  const int lane = threadIdx.x & 63;
  for (int o = 1; o < 64; o <<= 1) {
    const uint64_t lo = __shfl_up((uint64_t)v, o, 64), hi = __shfl_up((uint64_t)(v >> 64), o, 64);
    if (lane >= o) v += ((u128)hi << 64) | lo;
  }
  return v;
}

struct Args {
  const int64_t* step_ns;
  int32_t R, S;
  argus_l1_params_t p;
  uint8_t* flags;
  uint8_t* cls;
  int32_t* eff_width;
  int32_t* cp;
  float* cp_ratio;
  int32_t* dev_status;
};

// Place of point i: one element of padding per 16, so that lanes that read
// runs of 16 consecutive points fall on different banks.
__device__ __forceinline__ int at(int i) { return i + (i >> 4); }

template <int SCAP>
struct L1Smem {
  uint64_t y[SCAP + SCAP / 16];
  uint64_t cov[SCAP / 64];  // bit i: point i covered by a candidate window
  uint64_t exc[SCAP / 64];  // bit i: point i above its interval's baseline
  uint32_t hist[256];
  uint32_t digit, before;
};

__device__ __forceinline__ uint64_t uniform64(uint64_t v) {
  return ((uint64_t)(uint32_t)__builtin_amdgcn_readfirstlane((int)(v >> 32)) << 32) |
         (uint32_t)__builtin_amdgcn_readfirstlane((int)v);
}

// Lower median (rank (m-1)/2) of y over the m points outside [ea, eb] (no
// exclusion when ea > eb), by MSD radix select over 8-bit digits of y
// (every y < 2^bits). Wavefront-wide.
template <int SCAP>
__device__ int64_t wave_lower_median(L1Smem<SCAP>& sm, int S, int ea, int eb, int bits) {
  const int lane = threadIdx.x & 63;
  const uint32_t m = (uint32_t)(S - (ea > eb ? 0 : eb - ea + 1));
  uint32_t k = (m - 1) / 2;
  uint64_t prefix = 0;
  const int top = (bits - 1) / 8 * 8;
  for (int shift = top; shift >= 0; shift -= 8) {
    for (int b = lane; b < 256; b += 64) sm.hist[b] = 0;
    lds_barrier();
    for (int i = lane; i < S; i += 64) {
      if (i >= ea && i <= eb) continue;
      const uint64_t v = sm.y[at(i)];
      if (shift == top || (v >> (shift + 8)) == prefix) atomicAdd(&sm.hist[(v >> shift) & 255u], 1u);
    }
    lds_barrier();
    // lane owns bins 4 lane .. 4 lane + 3
    uint32_t h[4], tot = 0;
    for (int j = 0; j < 4; ++j) {
      h[j] = sm.hist[4 * lane + j];
      tot += h[j];
    }
    uint32_t incl = tot;
    for (int o = 1; o < 64; o <<= 1) {
      const uint32_t n = __shfl_up(incl, o, 64);
      if (lane >= o) incl += n;
    }
    uint32_t run = incl - tot;
    for (int j = 0; j < 4; ++j) {
      if (run <= k && k < run + h[j]) {
        sm.digit = 4 * lane + j;
        sm.before = run;
      }
      run += h[j];
    }
    lds_barrier();
    prefix = (prefix << 8) | sm.digit;
    k -= sm.before;
    lds_barrier();
  }
  return (int64_t)prefix;
}

// Whether the window [t, t + w) has 1000 max > theta_pm min. T: the points'
// type (32 bits hold them and a product with a permille value fits 64).
template <typename T, int SCAP>
__device__ __forceinline__ bool candidate(const L1Smem<SCAP>& sm, int t, int w, int32_t theta_pm) {
  T mx = (T)sm.y[at(t)], mn = mx;
#pragma unroll 4
  for (int i = t + 1; i < t + w; ++i) {
    const T v = (T)sm.y[at(i)];
    mx = v > mx ? v : mx;
    mn = v < mn ? v : mn;
  }
  if constexpr (sizeof(T) == 4)
    return (uint64_t)1000u * mx > (uint64_t)(uint32_t)theta_pm * mn;
  else
    return (u128)1000u * (u128)mx > (u128)(uint32_t)theta_pm * (u128)mn;
}

template <int SCAP>
__global__ __launch_bounds__(64) void l1_kernel(Args a) {
  __shared__ L1Smem<SCAP> sm;
  const int lane = threadIdx.x;
  const int64_t r = blockIdx.x;
  const int S = a.S;
  if (S == 0) {
    if (lane == 0) {
      a.cls[r] = 0;
      a.eff_width[r] = 0;
      a.cp[r] = -1;
      if (a.cp_ratio) a.cp_ratio[r] = 0.0f;
    }
    return;
  }
  const int64_t* yr = a.step_ns + r * S;
  uint64_t any = 0;  // every set bit of the points; a negative point sets bit 63
#pragma unroll 4
  for (int i = lane; i < S; i += 64) {
    const uint64_t v = (uint64_t)yr[i];
    sm.y[at(i)] = v;
    any |= v;
  }
  for (int o = 32; o > 0; o >>= 1) any |= __shfl_xor(any, o, 64);
  any = uniform64(any);
  if (any >= (uint64_t)kYLimit) {
    for (int i = lane; i < S; i += 64) a.flags[r * S + i] = 0;
    if (lane == 0) {
      a.cls[r] = 0x80;
      a.eff_width[r] = 0;
      a.cp[r] = -1;
      if (a.cp_ratio) a.cp_ratio[r] = 0.0f;
      if (a.dev_status) atomicOr(a.dev_status, (int32_t)ARGUS_DEV_L1_DOMAIN);
    }
    return;
  }
  const bool narrow = any < (1ull << 32);
  lds_barrier();

  // sensitivity gating: window t = [t, t+w-1] is a candidate when its
  // max/min ratio exceeds theta; point i is covered when one of the windows
  // [i-w+1, i] is a candidate
  const int w = a.p.W < S ? a.p.W : S;
  const int nwin = S - w + 1;
  int last = -(1 << 30);  // last candidate before this word's points
  bool some = false;
  for (int i0 = 0; i0 < S; i0 += 64) {
    const int i = i0 + lane;
    bool c = false;
    if (i < nwin) c = narrow ? candidate<uint32_t>(sm, i, w, a.p.theta_pm) : candidate<uint64_t>(sm, i, w, a.p.theta_pm);
    const uint64_t word = __ballot(c), upto = word & (~0ull >> (63 - lane));
    const int mine = upto ? i0 + 63 - __builtin_clzll(upto) : last;
    const uint64_t covw = __ballot(i < S && mine >= i - w + 1);
    some = some || covw != 0;
    if (word) last = i0 + 63 - __builtin_clzll(word);
    if (lane == 0) {
      sm.cov[i0 >> 6] = covw;
      sm.exc[i0 >> 6] = 0;
    }
  }
  lds_barrier();
  // merged intervals: maximal runs of covered points (overlapping or
  // touching candidate windows merge), found by the whole wavefront alike
  int width = 0;
  for (int i = 0; some && i < S;) {
    const uint64_t rest0 = uniform64(sm.cov[i >> 6]) >> (i & 63);
    if (rest0 == 0) {
      i = ((i >> 6) + 1) << 6;
      continue;
    }
    const int ia = i + __builtin_ctzll(rest0);
    int j = ia;  // first uncovered point from ia on
    while (j < S) {
      const uint64_t ones = uniform64(sm.cov[j >> 6]) >> (j & 63);
      const int avail = 64 - (j & 63);
      int len = ~ones == 0 ? 64 : __builtin_ctzll(~ones);
      if (len > avail) len = avail;
      j += len;
      if (len < avail) break;
    }
    if (j > S) j = S;
    const int ib = j - 1;
    i = j;
    // baseline: lower median of the points outside [ia, ib], of all points
    // when none lie outside
    const bool all_inside = ia == 0 && ib == S - 1;
    const int bits = any ? 64 - __builtin_clzll(any) : 1;
    const int64_t base = all_inside ? wave_lower_median(sm, S, 1, 0, bits) : wave_lower_median(sm, S, ia, ib, bits);
    // 1000 y > beta_pm base: 1000 y < 2^50, so no point passes a larger limit
    const u128 limit = (u128)(uint32_t)a.p.beta_pm * (u128)(uint64_t)base;
    const uint64_t lim = limit >> 64 ? ~0ull : (uint64_t)limit;
    // points significantly above the baseline; the longest contiguous run
    // of them is the interval's effective width (wave-uniform bit scan)
    int run = 0;
    for (int wd = ia >> 6; wd <= ib >> 6; ++wd) {
      const int q = 64 * wd + lane;
      const uint64_t word = __ballot(q >= ia && q <= ib && 1000u * sm.y[at(q < S ? q : S - 1)] > lim);
      if (lane == 0) sm.exc[wd] |= word;
      int b = 0;
      while (b < 64) {
        const uint64_t rest = word >> b;
        if (rest & 1u) {
          int len = ~rest == 0 ? 64 - b : __builtin_ctzll(~rest);
          if (b + len > 64) len = 64 - b;
          run += len;
          width = run > width ? run : width;
          b += len;
        } else {
          run = 0;
          b = rest == 0 ? 64 : b + __builtin_ctzll(rest);
        }
      }
    }
  }

  // change point: each lane takes the splits at its run of consecutive
  // points. Sums stay below 2^52 and the cross products below 2^64.
  const int chunk = (S + 63) / 64;  // at most 64
  const int c0 = lane * chunk, c1 = c0 + chunk < S ? c0 + chunk : S;
  uint64_t ls = 0;
#pragma unroll 4
  for (int i = c0; i < c1; ++i) ls += sm.y[at(i)];
  uint64_t es = ls;
  for (int o = 1; o < 64; o <<= 1) {
    const uint64_t n = __shfl_up(es, o, 64);
    if (lane >= o) es += n;
  }
  const uint64_t total = __shfl(es, 63, 64);
  es -= ls;
  const int t_lo = a.p.min_seg > 1 ? a.p.min_seg : 1;
  const int64_t t_hi = (int64_t)S - a.p.min_seg;
  uint64_t pass = 0;  // bit i - c0: the means' ratio at split i reaches rho
  {
    uint64_t sl = es;
    for (int i = c0; i < c1; ++i) {
      const uint64_t sr = total - sl, num = sr * (uint64_t)i, den = sl * (uint64_t)(S - i);
      const double lhs = 1000.0 * (double)num, rhs = (double)a.p.rho_pm * (double)den;
      bool p = lhs > rhs * (1.0 + kBand);
      if (!p && lhs >= rhs * (1.0 - kBand)) p = (u128)1000u * num >= (u128)(uint32_t)a.p.rho_pm * den;
      // the ratio needs a positive left mean
      if (p && sl != 0 && i >= t_lo && i <= t_hi) pass |= 1ull << (i - c0);
      sl += sm.y[at(i)];
    }
  }
  int32_t bt = -1;
  uint64_t bn = 0, bd = 1;
  if (__ballot(pass != 0) != 0) {
    u128 lq = 0;
    for (int i = c0; i < c1; ++i) lq += (u128)sm.y[at(i)] * (u128)sm.y[at(i)];
    const u128 iq = wave_incl_scan128(lq);
    const u128 tq = ((u128)__shfl((uint64_t)(iq >> 64), 63, 64) << 64) | __shfl((uint64_t)iq, 63, 64);
    u128 ql = iq - lq;
    uint64_t sl = es;
    for (int i = c0; i < c1; ++i) {
      if ((pass >> (i - c0)) & 1u) {
        const uint64_t sr = total - sl, num = sr * (uint64_t)i, den = sl * (uint64_t)(S - i);
        if (rel_std_ok(i, sl, ql, a.p.cmax_pm) && rel_std_ok(S - i, sr, tq - ql, a.p.cmax_pm) &&
            (bt < 0 || (u128)num * bd > (u128)bn * den)) {
          bt = i;
          bn = num;
          bd = den;
        }
      }
      const uint64_t v = sm.y[at(i)];
      sl += v;
      ql += (u128)v * v;
    }
    // the largest ratio, the earliest split on ties (lanes hold ascending splits)
    for (int o = 32; o > 0; o >>= 1) {
      const int32_t t = __shfl_xor(bt, o, 64);
      const uint64_t n = __shfl_xor(bn, o, 64), d = __shfl_xor(bd, o, 64);
      if (t < 0) continue;
      const u128 x = (u128)n * bd, y = (u128)bn * d;
      if (bt < 0 || x > y || (x == y && t < bt)) {
        bt = t;
        bn = n;
        bd = d;
      }
    }
  }
  const int cpt = bt;
  if (lane == 0) {
    a.cp[r] = cpt;
    if (a.cp_ratio) a.cp_ratio[r] = cpt >= 0 ? (float)((double)bn / (double)bd) : 0.0f;
    a.eff_width[r] = width;
    a.cls[r] = (uint8_t)((width > 0 ? 1 : 0) | (cpt >= 0 ? 2 : 0));
  }
  lds_barrier();
  // flags: bit 0 covered, bit 1 above the baseline, bit 2 from the change point on
  for (int i = lane; i < S; i += 64) {
    const uint32_t c = (uint32_t)(sm.cov[i >> 6] >> (i & 63)) & 1u, e = (uint32_t)(sm.exc[i >> 6] >> (i & 63)) & 1u;
    a.flags[r * S + i] = (uint8_t)(c | (e << 1) | (cpt >= 0 && i >= cpt ? 4u : 0u));
  }
}

template <int SCAP>
hipError_t launch_t(const Args& args, hipStream_t st) {
  hipLaunchKernelGGL(l1_kernel<SCAP>, dim3(args.R), dim3(64), 0, st, args);
  return hipGetLastError();
}

}  // namespace

hipError_t launch_iter_windows(const IterWindowsLaunch& l, hipStream_t st) {
  Args a{l.step_ns, l.R, l.S, l.p, l.flags, l.cls, l.eff_width, l.cp, l.cp_ratio, l.dev_status};
  if (l.R == 0) return hipSuccess;
  if (l.S <= 64) return launch_t<64>(a, st);
  if (l.S <= 512) return launch_t<512>(a, st);
  if (l.S <= 1024) return launch_t<1024>(a, st);
  if (l.S <= 2048) return launch_t<2048>(a, st);
  return launch_t<ARGUS_MAX_L1_STEPS>(a, st);
}

}  // namespace argus
