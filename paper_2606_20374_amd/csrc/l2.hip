// Parallelism-group-aware L2 comparison (section 6.1 routing table; Appendix
// B, Eq. 5; the step-by-step definition is in include/argus.h).
//
// Launches, in order:
//   l2_init     default outputs: every cell z = 0, flags = 0; every (step,
//               event, group) not evaluated; ownership keys cleared.
//   l2_owner    one workgroup per (dimension, group): each listing (g, i) of
//               a rank m takes part in ownership by an atomic minimum of
//               g R + i, so the rank's first listing (lowest group, then
//               lowest position) is the one that counts; a second listing
//               or a malformed range raises a status bit.
//   l2_stats    the lanes are events of one dimension, listed per tile of 2048
//               event ids so that nearly all lanes have one; a wavefront takes
//               a small group, or the wavefronts of a workgroup share a large
//               one. Per lane the exact sums n, S = sum x, Q = sum x^2
//               (128-bit) give D = n Q - S^2; the CV class and the z threshold
//               are decided in double where that settles them and by exact
//               256-bit comparisons where it does not, the reported mean / std
//               / CV / z are one double operation each.
//   l2_each     instead, for up to kSmall ranks: a wavefront for every group
//               and 64 event ids.
// What bounds l2_stats: the latency of the scattered cell reads and writes (a
// wavefront's 64 events of one dimension span up to 430 event ids) and the
// double-precision divisions; 252 MB of cells are read once from HBM and up to
// four times, once per dimension, from the Infinity Cache. Cluster step
// (10,240 ranks x 2,048 events, TP / PP / DP / EP groups of 8 / 8 / 160 / 8):
// 996 us with one wavefront per group and 64 consecutive event ids, whose
// members were read one after another (four dependent loads each, twice) and
// whose 160-member groups were the tail; 339 us now, 1,014 -> 388 us per call.
// The loads are about 90 us of it, the z and flag stores 75 us, the group
// outputs 30 us, timed by leaving each out. The unrolled exact arithmetic of an earlier form (16,400
// instructions) did not fit the instruction cache and ran at half the speed.
#include "argus_internal.h"

namespace argus {
namespace {

typedef unsigned __int128 u128;

constexpr uint64_t kDomain = 1ull << 40;  // x at or above 2^40 ns is out of the domain
constexpr uint8_t kNotEvaluated = 0xFF;

struct L2Args {
  const uint32_t* count;
  const int64_t* sum;
  int32_t R, S, E;
  const uint8_t* route;
  const int32_t* off;  // [n_dims][max_groups + 1]
  const int32_t* mem;  // [n_dims][R]
  int32_t n_dims, max_groups;
  argus_l2_params_t p;
  argus_l2_out_t o;
  uint32_t* owner;  // workspace [n_dims][R]: first listing key g R + i
};

struct U256 {
  u128 hi, lo;
};

// Full 128 x 128 -> 256-bit product.
__device__ __forceinline__ U256 mul_wide(u128 a, u128 b) {
  const uint64_t a0 = (uint64_t)a, a1 = (uint64_t)(a >> 64), b0 = (uint64_t)b, b1 = (uint64_t)(b >> 64);
  const u128 p00 = (u128)a0 * b0, p01 = (u128)a0 * b1, p10 = (u128)a1 * b0, p11 = (u128)a1 * b1;
  const u128 mid = (p00 >> 64) + (uint64_t)p01 + (uint64_t)p10;
  return U256{p11 + (p01 >> 64) + (p10 >> 64) + (mid >> 64), (mid << 64) | (uint64_t)p00};
}

__device__ __forceinline__ bool less(const U256& a, const U256& b) {
  return a.hi < b.hi || (a.hi == b.hi && a.lo < b.lo);
}

__device__ __forceinline__ void raise(int32_t* st, int32_t bit) {
  if (st) atomicOr(st, bit);
}

// ------------------------------------------------------------------- init
__global__ __launch_bounds__(256) void l2_init(L2Args a, int64_t cells, int64_t gout, int64_t owners) {
  const int64_t stride = (int64_t)gridDim.x * 256;
  for (int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x; i < cells; i += stride) {
    a.o.z[i] = 0.0f;
    a.o.flags[i] = 0;
  }
  for (int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x; i < gout; i += stride) {
    a.o.n[i] = 0;
    a.o.mean_ns[i] = a.o.std_ns[i] = a.o.cv[i] = 0.0;
    a.o.cls[i] = kNotEvaluated;
    a.o.n_strag[i] = 0;
  }
  for (int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x; i < owners; i += stride) a.owner[i] = 0xFFFFFFFFu;
}

// ------------------------------------------------------------- membership
__global__ __launch_bounds__(256) void l2_owner(L2Args a) {
  const int g = blockIdx.x, d = blockIdx.y;
  const int32_t* off = a.off + (int64_t)d * (a.max_groups + 1);
  const int32_t lo = off[g], hi = off[g + 1];
  if (lo < 0 || hi < lo || hi > a.R) {
    if (threadIdx.x == 0) raise(a.o.dev_status, ARGUS_DEV_GROUPS_MALFORMED);
    return;
  }
  bool bad = false, dup = false;
  for (int32_t i = lo + (int32_t)threadIdx.x; i < hi; i += 256) {
    const int32_t m = a.mem[(int64_t)d * a.R + i];
    if (m < 0 || m >= a.R) {
      bad = true;
      continue;
    }
    const uint32_t old = atomicMin(&a.owner[(int64_t)d * a.R + m], (uint32_t)g * (uint32_t)a.R + (uint32_t)i);
    if (old != 0xFFFFFFFFu) dup = true;
  }
  if (__ballot(bad) != 0 && (threadIdx.x & 63) == 0) raise(a.o.dev_status, ARGUS_DEV_GROUPS_MALFORMED);
  if (__ballot(dup) != 0 && (threadIdx.x & 63) == 0) raise(a.o.dev_status, ARGUS_DEV_GROUPS_DUPLICATE);
}

// ----------------------------------------------------------------- stats
constexpr int kTile = 2048;  // event ids whose events of one dimension are listed together
constexpr int kSplit = 16;   // workgroups at most that share a tile's list, 64 events at a time
constexpr int kWaves = 8;    // wavefronts per workgroup: one small group each, or a share of a large one
constexpr int kSlots = 4;    // workgroups at most that share the large ones of kWaves groups
constexpr int kKeep = 24;    // members of a wavefront whose means stay in LDS between the two passes
constexpr int kSmall = 32;   // listed members up to which a group is small (one wavefront)
constexpr int kBatch = 8;    // members whose cells are loaded together
constexpr int kFew = 2;      // the same in l2_each: 8 take 92 registers and five wavefronts per SIMD, 2 take 68 and seven
constexpr double kBand = 1e-12;  // of the double comparisons below (their error is below 1e-14)
constexpr uint32_t kNoMean = 0xFFFFFFFFu;  // no mean that is kept: those lie below it

// x = floor(sum / n) for n >= 1 (sum read as uint64), or -1 when x is out of
// the domain. The double quotient is within x 2^-51 of the real one, so below
// the domain limit its floor is at most one off, which the remainder shows.
__device__ __forceinline__ int64_t mean_of(uint32_t n, uint64_t sum) {
  const double qd = (double)sum / (double)n;
  if (qd >= (double)(kDomain + 1)) return -1;
  uint64_t x = (uint64_t)qd;
  const int64_t r = (int64_t)(sum - x * n);
  x += r < 0 ? ~0ull : (r >= (int64_t)n ? 1ull : 0ull);
  return x < kDomain ? (int64_t)x : -1;
}

// One wavefront's share of a group: listings [lo, hi) of its dimension's
// member list. The lanes are events.
struct Part {
  const int32_t* mem;
  const uint32_t* own;
  uint32_t key0;
  int32_t lo, hi, s, e;

  // the members that count among the 64 listings from i0 on (first listings
  // of ranks in range); lane l gets listing i0 + l's rank
  __device__ __forceinline__ uint64_t at(const L2Args& a, int32_t i0, int32_t& m) const {
    const int32_t i = i0 + (int32_t)(threadIdx.x & 63);
    m = i < hi ? mem[i] : -1;
    const bool ok = m >= 0 && m < a.R && own[m] == key0 + (uint32_t)i;
    if (!ok) m = 0;
    return __ballot(ok);
  }

  // Up to B members from todo: their cells of this lane's event, every
  // load issued before the first is used. cnt = 0: no such member or an
  // absent cell.
  template <int B>
  __device__ __forceinline__ void load(const L2Args& a, uint64_t& todo, int32_t m, uint32_t (&row)[B],
                                       uint32_t (&cnt)[B], int64_t (&sm)[B]) const {
    const int nb = __popcll(todo);
#pragma unroll
    for (int u = 0; u < B; ++u) {
      if (u >= nb) {
        row[u] = 0;
        cnt[u] = 0;
        sm[u] = 0;
        continue;
      }
      const int l = __builtin_ctzll(todo);
      todo &= todo - 1;
      row[u] = (uint32_t)__builtin_amdgcn_readlane(m, l) * (uint32_t)a.S + (uint32_t)s;
      cnt[u] = (a.count + (uint64_t)row[u] * (uint32_t)a.E)[(uint32_t)e];
      sm[u] = (a.sum + (uint64_t)row[u] * (uint32_t)a.E)[(uint32_t)e];
    }
  }
};

struct Sums {
  uint32_t n;
  uint64_t S;
  u128 Q;
};

// Exact sums over a part's present members; their means go to keep (a row of
// 64 lanes per member, every 64 listings' rows from a multiple of B on)
// while they fit. Returns whether keep holds all of them.
template <int B>
__device__ __forceinline__ bool sum_part(const L2Args& a, const Part& p, Sums& t, uint32_t (*keep)[64], bool& dom) {
  const int lane = threadIdx.x & 63;
  t = Sums{0, 0, 0};
  bool kept = true;
  int at = 0;
  for (int32_t i0 = p.lo; i0 < p.hi; i0 += 64) {
    int32_t m;
    uint64_t todo = p.at(a, i0, m);
    while (todo) {
      uint32_t row[B], cnt[B];
      int64_t sm[B];
      p.load(a, todo, m, row, cnt, sm);
      // means below kNoMean of sums below 2^53: both operands are exact
      // doubles, so the floor of the rounded quotient is exact or one above,
      // and the squares fit 64 bits
      Sums q = t;
      bool wide = false;
      const bool room = at + B <= kKeep;
#pragma unroll
      for (int u = 0; u < B; ++u) {
        const double nd = (double)cnt[u], sd = (double)(uint64_t)sm[u], qd = sd / nd;
        wide = wide || (cnt[u] != 0 && !(sd < 0x1p53 && qd < (double)kNoMean));
        uint32_t x = (uint32_t)qd;
        x -= fma(-(double)x, nd, sd) < 0.0 ? 1u : 0u;
        x = cnt[u] ? x : 0u;
        q.n += cnt[u] ? 1u : 0u;
        q.S += x;
        q.Q += (uint64_t)x * x;
        if (room) keep[at + u][lane] = cnt[u] ? x : kNoMean;
      }
      if (__ballot(wide) == 0) {
        t = q;
        kept = kept && room;
      } else {
        kept = false;
#pragma unroll
        for (int u = 0; u < B; ++u) {
          if (cnt[u] == 0) continue;
          const int64_t x = mean_of(cnt[u], (uint64_t)sm[u]);
          if (x < 0) {
            dom = true;
            continue;
          }
          ++t.n;
          t.S += (uint64_t)x;
          t.Q += (u128)(uint64_t)x * (uint64_t)x;
        }
      }
      at += B;
    }
  }
  return kept;
}

// What a group reports for one event, and what its members are compared with.
// n <= 2^16 and x < 2^40, so n x and S stay within 2^56.
struct Group {
  bool eval;
  uint8_t cls;
  double mean, sd, cv;
  double rsd;          // 1 / sd
  double x_no, x_yes;  // x at or below x_no is no straggler, x at or above x_yes is one; decided exactly between
  uint64_t S;
  u128 D;
  uint32_t n;

  // n D 10^6 < cv_pm^2 (n - 1) S^2: in double, exactly where the two lie within kBand
  __device__ __forceinline__ bool below(double Dd, int32_t cv_pm) const {
    const double lhs = (double)n * 1e6 * Dd;
    const double rhs = (double)cv_pm * (double)cv_pm * (double)(n - 1) * (double)S * (double)S;
    if (lhs < rhs * (1.0 - kBand)) return true;
    if (lhs > rhs * (1.0 + kBand)) return false;
    return less(mul_wide((u128)n * 1000000u, D), mul_wide((u128)(uint32_t)cv_pm * (uint32_t)cv_pm * (n - 1), (u128)S * S));
  }

  __device__ __forceinline__ void set(const L2Args& a, const Sums& q) {
    n = q.n;
    S = q.S;
    eval = (int32_t)n >= a.p.min_group && n >= 2;
    cls = kNotEvaluated;
    mean = sd = cv = rsd = 0.0;
    x_no = x_yes = __builtin_inf();
    D = 0;
    if (!eval) return;
    D = (u128)n * q.Q - (u128)S * S;
    const double Dd = u128_to_f64(D);
    mean = (double)S / (double)n;
    sd = sqrt(Dd / ((double)n * (double)(n - 1)));
    cv = mean > 0.0 ? sd / mean : 0.0;
    uint8_t c = 0;
#pragma unroll 1
    for (; c < 2 && S != 0; ++c)
      if (below(Dd, c == 0 ? a.p.cv_mild_pm : a.p.cv_severe_pm)) break;
    cls = c;
    // equal members are no stragglers; otherwise (n x - S)^2 (n - 1) 10^6 >
    // z_pm^2 n D, n x > S turns at an x that doubles give to within 2^-8
    if (D == 0) return;
    rsd = 1.0 / sd;
    const double at = ((double)S + sqrt((double)n * Dd / ((double)(n - 1) * 1e6)) * (double)a.p.z_pm) / (double)n;
    x_no = at - 0.01;
    x_yes = at + 0.01;
  }

  __device__ __forceinline__ bool straggler(const L2Args& a, double xd, uint64_t x) const {
    if (xd >= x_yes) return true;
    if (xd <= x_no) return false;
    const uint64_t nx = (uint64_t)n * x;
    if (nx <= S) return false;
    return less(mul_wide((u128)(uint32_t)a.p.z_pm * (uint32_t)a.p.z_pm * n, D),
                mul_wide((u128)(nx - S) * (nx - S), (u128)(n - 1) * 1000000u));
  }

  // Correctly rounded v / sd: with rsd the rounded reciprocal of sd, q is
  // within an ulp of the quotient and the last step rounds it correctly
  // (Markstein's division theorem).
  __device__ __forceinline__ double over_sd(double v) const {
    const double q0 = v * rsd;
    const double q = fma(fma(-sd, q0, v), rsd, q0);
    return fma(fma(-sd, q, v), rsd, q);
  }

  // z and flags of one member
  __device__ __forceinline__ uint32_t write(const L2Args& a, uint32_t row, int e, double xd, uint64_t x) const {
    const bool f = straggler(a, xd, x);
    const uint64_t c = (uint64_t)row * (uint32_t)a.E;
    // + 0: sd 0 makes a mean that is rounded above x a negative zero, and no other quotient rounds to one
    (a.o.z + c)[(uint32_t)e] = (float)over_sd(xd - mean) + 0.0f;
    (a.o.flags + c)[(uint32_t)e] = f ? 3 : 1;
    return f ? 1u : 0u;
  }
};

// Second pass over a part: z and flags of its members (on: this lane's event
// is evaluated). Returns the number of stragglers.
template <int B>
__device__ __forceinline__ uint32_t write_part(const L2Args& a, const Part& p, const Group& g, bool on, bool kept,
                                               uint32_t (*keep)[64]) {
  const int lane = threadIdx.x & 63;
  uint32_t ns = 0;
  int at = 0;
  for (int32_t i0 = p.lo; i0 < p.hi; i0 += 64) {
    int32_t m;
    uint64_t todo = p.at(a, i0, m);
    if (kept) {
#pragma unroll 2
      for (; todo; todo &= todo - 1) {
        const uint32_t row = (uint32_t)__builtin_amdgcn_readlane(m, __builtin_ctzll(todo)) * (uint32_t)a.S + (uint32_t)p.s;
        const uint32_t x = keep[at++][lane];
        if (on && x != kNoMean) ns += g.write(a, row, p.e, (double)x, x);
      }
      at = (at + B - 1) / B * B;
    }
    while (todo) {
      uint32_t row[B], cnt[B];
      int64_t sm[B];
      p.load(a, todo, m, row, cnt, sm);
#pragma unroll
      for (int u = 0; u < B; ++u) {
        if (!on || cnt[u] == 0) continue;
        const int64_t x = mean_of(cnt[u], (uint64_t)sm[u]);
        if (x >= 0) ns += g.write(a, row[u], p.e, (double)x, (uint64_t)x);
      }
    }
  }
  return ns;
}

struct SmallOut {
  double mean[kWaves][65], sd[kWaves][65], cv[kWaves][65];
  uint32_t n[kWaves][65], ns[kWaves][65];
  uint8_t cls[kWaves][68];
};
struct LargePart {
  uint64_t S[kWaves][64], Qlo[kWaves][64], Qhi[kWaves][64];
  uint32_t n[kWaves][64];
};

// Workgroup (x, y, z): z names a step and a dimension d, y a span of kWaves
// groups of d and a slot, x a tile of event ids and a share of the tile's
// events of d. In slot 0 the small groups of the span take one wavefront
// each; its large groups go to the slots in turn, where the wavefronts share
// a group's members (one after another in one workgroup, the 8 large groups
// of a span ran 160 us on the cluster step; loads took a fifth of that).
// Dimensions differ in their group sizes, so workgroups with
// much and with little work would alternate with a fixed period if the
// dimension ran fastest, and the dispatcher's round over XCDs and shader
// engines would then load a few of them only; x has an odd extent for the
// same reason.
__global__ __launch_bounds__(64 * kWaves, 4) void l2_stats(L2Args a, int32_t tiles, int32_t split, int32_t n_span, int32_t slots) {
  __shared__ uint32_t keep_sh[kWaves][kKeep][64];
  __shared__ uint16_t ev[kTile];  // event ids from e0 on
  __shared__ int32_t wave_n[kWaves];
  __shared__ union {
    SmallOut small;
    LargePart large;
  } sh;
  // apart from the union: the first wavefront reads a large group's stragglers
  // while others may have gone on to the next events' small groups
  __shared__ uint32_t ns_sh[64];
  const int tid = threadIdx.x, lane = tid & 63, w = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int s = (int)(blockIdx.z / (uint32_t)a.n_dims), d = (int)(blockIdx.z % (uint32_t)a.n_dims);
  const int slot = (int)blockIdx.y / n_span, g0 = (int)blockIdx.y % n_span * kWaves;
  if (slot >= slots) return;
  // bit j: group g0 + j is a small / a large one of the dimension
  int32_t lo = 0, hi = 0;
  if (lane < kWaves && g0 + lane < a.max_groups) {
    const int32_t* off = a.off + (int64_t)d * (a.max_groups + 1) + g0 + lane;
    lo = off[0];
    hi = off[1];
  }
  const bool ok = lo >= 0 && hi > lo && hi <= a.R;
  const uint32_t some = (uint32_t)__ballot(ok && hi - lo <= kSmall && slot == 0);
  const uint32_t many = (uint32_t)__ballot(ok && hi - lo > kSmall && lane % slots == slot);
  if ((some | many) == 0) return;
  bool dom = false;
  const uint32_t items = (uint32_t)tiles * (uint32_t)split;
  for (uint32_t it = blockIdx.x; it < items; it += gridDim.x) {
    const int64_t e0 = (int64_t)(it % (uint32_t)tiles) * kTile;
    const int c0 = (int)(it / (uint32_t)tiles) * 64;
    // the tile's events of this dimension, in order
    constexpr int kSteps = kTile / 64 / kWaves;  // 64 event ids each, in turn
    uint64_t bal[kSteps];
    int n = 0;
#pragma unroll
    for (int h = 0; h < kSteps; ++h) {
      const int64_t e = e0 + (w * kSteps + h) * 64 + lane;
      bal[h] = __ballot(e < a.E && a.route[e] == d);
      n += __popcll(bal[h]);
    }
    if (lane == 0) wave_n[w] = n;
    lds_barrier();
    int M = 0, base = 0;
#pragma unroll
    for (int v = 0; v < kWaves; ++v) {
      base += v < w ? wave_n[v] : 0;
      M += wave_n[v];
    }
    M = __builtin_amdgcn_readfirstlane(M);
    if (c0 < M) {
#pragma unroll
      for (int h = 0; h < kSteps; ++h) {
        if ((bal[h] >> lane) & 1u)
          ev[base + __popcll(bal[h] & ((1ull << lane) - 1))] = (uint16_t)((w * kSteps + h) * 64 + lane);
        base += __popcll(bal[h]);
      }
    }
    lds_barrier();
    for (int c = c0; c < M; c += 64 * split) {
      const bool on = c + lane < M;
      Part p{a.mem + (int64_t)d * a.R, a.owner + (int64_t)d * a.R, 0, 0, 0, s, (int)e0 + ev[on ? c + lane : c]};
      // first the small groups together, then the large ones in turn
      uint32_t rest = many;
      bool large = some == 0;
      while (!large || rest != 0) {
        const int j = large ? __builtin_ctz(rest) : w;
        const bool busy = large || ((some >> j) & 1u) != 0;
        p.key0 = (uint32_t)(g0 + j) * (uint32_t)a.R;
        p.lo = __builtin_amdgcn_readlane(lo, j);
        p.hi = __builtin_amdgcn_readlane(hi, j);
        if (large) {
          const int64_t len = p.hi - p.lo, first = p.lo;
          p.lo = (int32_t)(first + len * w / kWaves);
          p.hi = (int32_t)(first + len * (w + 1) / kWaves);
        }
        Sums t{0, 0, 0};
        const bool kept = busy && sum_part<kBatch>(a, p, t, keep_sh[w], dom);
        if (large) {
          sh.large.n[w][lane] = t.n;
          sh.large.S[w][lane] = t.S;
          sh.large.Qlo[w][lane] = (uint64_t)t.Q;
          sh.large.Qhi[w][lane] = (uint64_t)(t.Q >> 64);
          if (w == 0) ns_sh[lane] = 0;
          lds_barrier();
          t = Sums{0, 0, 0};
#pragma unroll 1
          for (int v = 0; v < kWaves; ++v) {
            t.n += sh.large.n[v][lane];
            t.S += sh.large.S[v][lane];
            t.Q += ((u128)sh.large.Qhi[v][lane] << 64) | sh.large.Qlo[v][lane];
          }
        }
        if (busy) {
          Group gr;
          gr.set(a, t);
          const uint32_t ns = write_part<kBatch>(a, p, gr, on && gr.eval, kept, keep_sh[w]);
          if (large) {
            if (ns) atomicAdd(&ns_sh[lane], ns);
            lds_barrier();
            if (w == 0 && on) {
              const int64_t go = ((int64_t)s * a.E + p.e) * a.max_groups + g0 + j;
              a.o.n[go] = t.n;
              a.o.n_strag[go] = ns_sh[lane];
              a.o.mean_ns[go] = gr.mean;
              a.o.std_ns[go] = gr.sd;
              a.o.cv[go] = gr.cv;
              a.o.cls[go] = gr.cls;
            }
          } else {
            sh.small.ns[j][lane] = ns;
            sh.small.n[j][lane] = t.n;
            sh.small.mean[j][lane] = gr.mean;
            sh.small.sd[j][lane] = gr.sd;
            sh.small.cv[j][lane] = gr.cv;
            sh.small.cls[j][lane] = gr.cls;
          }
        }
        if (large) {
          rest &= rest - 1;
          continue;
        }
        large = true;
        // the outputs have the group as the fastest index: kWaves groups of an
        // event are written together
        lds_barrier();
        const int q = tid % kWaves, l = tid / kWaves;
        if (c + l < M && ((some >> q) & 1u)) {
          const int64_t go = ((int64_t)s * a.E + e0 + ev[c + l]) * a.max_groups + g0 + q;
          a.o.n[go] = sh.small.n[q][l];
          a.o.n_strag[go] = sh.small.ns[q][l];
          a.o.mean_ns[go] = sh.small.mean[q][l];
          a.o.std_ns[go] = sh.small.sd[q][l];
          a.o.cv[go] = sh.small.cv[q][l];
          a.o.cls[go] = sh.small.cls[q][l];
        }
        lds_barrier();
      }
    }
    lds_barrier();  // the event list is used to here
  }
  if (__ballot(dom) != 0 && lane == 0) raise(a.o.dev_status, ARGUS_DEV_L2_DOMAIN);
}

// A wavefront for every group and 64 event ids of a step and dimension, for
// so few ranks that no group is large. Its lanes are idle where an event has
// another dimension, but seven such wavefronts share a SIMD against four of
// l2_stats, and none waits for another: 16 ranks x 1,000 steps x 50 events 70 us
// with l2_stats, 52 us so; 32 x 200 x 200 103 and 67 us; 8 x 2,000 x 50 97 and
// 31 us.
__global__ __launch_bounds__(64) void l2_each(L2Args a) {
  __shared__ uint32_t keep[kKeep][64];
  const int lane = threadIdx.x, g = blockIdx.y;
  const int64_t e = (int64_t)blockIdx.x * 64 + lane;
  const int s = (int)(blockIdx.z / (uint32_t)a.n_dims), d = (int)(blockIdx.z % (uint32_t)a.n_dims);
  const int32_t* off = a.off + (int64_t)d * (a.max_groups + 1) + g;
  const int32_t lo = off[0], hi = off[1];
  const bool mine = e < a.E && a.route[e] == d;
  if (__ballot(mine) == 0 || lo < 0 || hi <= lo || hi > a.R) return;
  const Part p{a.mem + (int64_t)d * a.R, a.owner + (int64_t)d * a.R, (uint32_t)g * (uint32_t)a.R, lo, hi, s,
               (int)(e < a.E ? e : a.E - 1)};
  bool dom = false;
  Sums t;
  const bool kept = sum_part<kFew>(a, p, t, keep, dom);
  if (__ballot(dom && mine) != 0 && lane == 0) raise(a.o.dev_status, ARGUS_DEV_L2_DOMAIN);
  Group gr;
  gr.set(a, t);
  uint32_t ns = 0;
  if (__ballot(mine && gr.eval) != 0) ns = write_part<kFew>(a, p, gr, mine && gr.eval, kept, keep);
  if (!mine) return;
  const int64_t go = ((int64_t)s * a.E + e) * a.max_groups + g;
  a.o.n[go] = t.n;
  a.o.n_strag[go] = ns;
  a.o.mean_ns[go] = gr.mean;
  a.o.std_ns[go] = gr.sd;
  a.o.cv[go] = gr.cv;
  a.o.cls[go] = gr.cls;
}

}  // namespace

size_t l2_workspace_bytes(int32_t R, int32_t n_dims) {
  if (R < 0 || n_dims < 0) return 0;
  return (size_t)R * (size_t)n_dims * sizeof(uint32_t);
}

hipError_t launch_l2(const L2Launch& l, hipStream_t st) {
  L2Args a{l.count, l.sum_ns, l.R, l.S, l.E, l.g.route, l.g.group_off, l.g.members, l.g.n_dims, l.g.max_groups,
           l.p, l.o, static_cast<uint32_t*>(l.workspace)};
  const int64_t cells = (int64_t)l.R * l.S * l.E, gout = (int64_t)l.S * l.E * l.g.max_groups;
  const int64_t owners = (int64_t)l.g.n_dims * l.R;
  int64_t mx = cells > gout ? cells : gout;
  mx = mx > owners ? mx : owners;
  const int64_t blocks = (mx + 255) / 256;
  hipLaunchKernelGGL(l2_init, dim3((unsigned)(blocks < 65536 ? blocks : 65536)), dim3(256), 0, st, a, cells, gout,
                     owners);
  hipError_t e = hipGetLastError();
  if (e != hipSuccess) return e;
  hipLaunchKernelGGL(l2_owner, dim3(l.g.max_groups, l.g.n_dims), dim3(256), 0, st, a);
  e = hipGetLastError();
  if (e != hipSuccess) return e;
  const unsigned z = (unsigned)((int64_t)l.S * l.g.n_dims);
  if (l.R <= kSmall) {
    hipLaunchKernelGGL(l2_each, dim3((unsigned)(((int64_t)l.E + 63) / 64), l.g.max_groups, z), dim3(64), 0, st, a);
    return hipGetLastError();
  }
  // A workgroup that finds nothing to do costs 2.5 ns: no more shares of a tile
  // than it has 64 events, no more slots than the ranks make large groups, and
  // fewer shares where the grid is large and the steps keep the chip busy
  // without them (300 ranks x 60 steps x 1,000 events: 902 us with 16 shares,
  // 466 us with one; 64 x 200 x 130: 1,077 and 94 us with 16 shares x 4 slots
  // and without; 10,240 x 1 x 2,048: 382, 375 with 8, 436 with 4). The extents
  // are odd so that workgroups with work do not fall on a few shader engines
  // only (256 x 100 x 64, slot 0 of four at work: 252 us with 32 along y, 79
  // with 33).
  const int64_t tiles = ((int64_t)l.E + kTile - 1) / kTile;
  const int32_t groups = (l.g.max_groups + kWaves - 1) / kWaves;
  int32_t split = l.E < 64 * kSplit ? (l.E + 63) / 64 : kSplit;
  const int32_t large = l.R / (kSmall + 1), slots = large < kSlots ? large : kSlots;
  const unsigned y = (unsigned)(groups * slots) | 1u;
  unsigned x;
  for (;; split /= 2) {
    const int64_t items = tiles * split;
    x = (unsigned)(items < (1 << 20) ? items | 1 : (1 << 20) | 1);
    if (split == 1 || (int64_t)l.S * items * slots <= 64 || (int64_t)x * y * z <= 20000) break;
  }
  hipLaunchKernelGGL(l2_stats, dim3(x, y, z), dim3(64 * kWaves), 0, st, a, (int32_t)tiles, split, groups, slots);
  return hipGetLastError();
}

}  // namespace argus
