// Per-(rank, step, kernel id) summarization of raw kernel-event arrays.
//
// Paper: section 4.3 (kernel activity records: kernel, launch time,
// duration, stream) and section 5.2 (all raw events of each (kernel, stream,
// rank) in a time window are reduced to compact statistics; durations are
// log-transformed and evaluated on an equally spaced grid). A window here is
// one step, i.e. one seg_off segment; the grid is octaves of ns.
//
// Design (gfx950):
// * One 1024-thread workgroup owns one rank-step segment and streams its
//   structure-of-arrays events from HBM exactly once: 16-byte non-temporal
//   loads of four consecutive events per thread, software pipelined so the
//   next group is in flight while the current one is processed.
// * Per-kernel state is privatised in LDS: 64-bit sum, min and max, and a
//   WIN-bin window of the octave histogram (a lognormal mode spans two or
//   three octaves, a kernel whose positions run at 1x, 3x and 9x five or
//   six). In the dense layout the window has ten bins around the first
//   duration seen; where the map or table leaves room for fewer, eight or six,
//   bin b is counted at b mod 8 or 6 while the bins seen span at most so many
//   octaves, wherever the first lay. Bins outside the window go to a small
//   pool of full 32-bin records that a kernel claims on first need.
// * Keys (kernel ids, or (kernel id, stream) pairs as id * n_streams +
//   stream: section 5.2 groups per kernel and stream) map to LDS slots
//   directly when the key space fits (dense), through an LDS key->slot map
//   that hands out slots on first sight (mapped, up to 16,384 keys), or
//   through an LDS hash table of the keys seen (hashed, up to 65,536 keys),
//   so a large, sparse key space too is read once; keys past the table's slots
//   are noted and get slots by their rank in further passes.
// * Whenever the pool or the slots run out, the kernels concerned are
//   marked and redone exactly in another pass over the segment: the result
//   is exact for every input; typical traces need one pass.
// * Per-segment aggregates (valid/invalid counts, first start, last end,
//   busy time) are kept in registers and reduced once per segment; per-stream
//   busy time uses LDS atomics.
// * The flush writes each present cell once and the count of every cell
//   (0 for absent kernels); an absent cell's other fields are not written,
//   so a large, sparse key space costs 4 bytes per absent cell.
#include <atomic>
#include <type_traits>

#include "argus_internal.h"
#include "summarize_hash.h"

namespace argus {
namespace {

typedef int v4i __attribute__((ext_vector_type(4)));
typedef long long v2l __attribute__((ext_vector_type(2)));

constexpr int kThreads = 1024;
constexpr uint32_t kSpanMask = 0x3E00FFu;
constexpr uint32_t kSpanUnset = 0xFFu;  // first bin of a span: none seen yet
constexpr uint32_t kStNone = 0, kStBusy = 0xFE, kStPoison = 0xFF;
constexpr uint32_t kDone = 1u << 16;
constexpr int kMapIds = 16384;  // ids in mapped mode
// Bound on the iterations of one claim wait, and on the passes over one segment
// that may end with a wait cut short. A claim's owner publishes after
// a fixed number of its own instructions, so no wait comes near the bound
// unless the code around it is compiled wrongly; the bounds make the kernel
// exit (and report) in that case instead of hanging.
constexpr int kSpinCap = 1 << 16;
constexpr int kMaxStuckPasses = 4;
constexpr int kDense = 0, kMapped = 1, kHashed = 2;
constexpr uint32_t kMapEmpty = 0xFFFF, kMapBusy = 0xFFFE, kMapDefer = 0xFFFD, kMapDone = 0xFFFC;

// meta word of a slot: bits 0-7 first bin of the window's span (0xFF unset),
// bits 17-21 its width, last bin - first (not kept in dense mode: WIN - 1),
// bits 8-15 full-record state (0 none, 1..kPool record index + 1, 0xFE being
// claimed, 0xFF pool exhausted: redo in another pass), bit 16 already written.
//
// map entry (mapped mode, 16 bits, two per 32-bit word): a slot index, or
// empty / being claimed / deferred to another pass / already written.
// The hash table of hashed mode: summarize_hash.h.

template <int NSLOT, int WIN, int MODE>
struct Smem {
  unsigned long long sum[NSLOT];
  long long mm[NSLOT][2];  // min, max (one 16-byte read per event)
  uint32_t win[NSLOT][WIN];
  uint32_t meta[NSLOT];
  // full 32-bin records of a pass: in mapped mode as many as the LDS has room for
  static constexpr int kPool = MODE == kMapped ? 27 : 32;
  uint32_t pool[kPool][NB];
  unsigned long long stream_busy[ARGUS_MAX_STREAMS];
  alignas(16) uint32_t map[MODE == kMapped ? kMapIds / 2 : MODE == kHashed ? kHash : 1];
  uint32_t left[MODE == kHashed ? kHashIds / 32 : 1];  // hashed mode: bit per key that is left for another pass
  uint16_t slot_kid[MODE != kDense ? NSLOT : 1];
  unsigned long long red_busy, red_wire;
  long long red_first, red_last;
  uint32_t red_valid, red_invalid;
  uint32_t npool, poison, nslots, stuck;
};

struct Args {
  const int32_t* kernel_id;
  const int32_t* stream;
  const int64_t* start_ns;
  const int64_t* end_ns;
  const int64_t* seg_off;
  int64_t n_events;
  int32_t n_kernels, n_streams;
  int32_t key_ns;  // 0: cells keyed by kernel id; else n_streams: keyed by (kernel id, stream)
  int32_t n_keys;  // cells per segment: n_kernels, or n_kernels * n_streams
  int32_t vec_ok;  // event arrays 16-byte aligned: vector loads allowed
  int32_t n_seg;
  uint32_t* queue;  // next segment to take (zeroed before the launch)
  uint32_t* count;
  int64_t* sum_ns;
  int64_t* min_ns;
  int64_t* max_ns;
  uint32_t* hist;
  uint32_t* n_valid;
  uint32_t* n_invalid;
  int64_t* t_first;
  int64_t* t_last;
  int64_t* step_ns;
  int64_t* busy_ns;
  int64_t* stream_busy_ns;
  int64_t* wire_bytes;
  int32_t* dev_status;
};

template <int NSLOT, int WIN, int MODE>
struct Seg {
  using S = Smem<NSLOT, WIN, MODE>;
  S& sm;

  __device__ __forceinline__ uint16_t map_get(int lk) const {
    return reinterpret_cast<const uint16_t*>(sm.map)[lk];
  }
  __device__ __forceinline__ void map_set(int lk, uint16_t v) { reinterpret_cast<uint16_t*>(sm.map)[lk] = v; }

  // Slot of local id lk, claiming one on first sight (mapped mode); -1 when
  // the id is already written or deferred to another pass. Lanes of one
  // wavefront may race for the same claim; the loop exits only when no
  // active lane is still pending, so a winner's publish executes inside the
  // loop, before a waiting lane of its own wavefront re-reads the entry.
  __device__ int map_claim(int lk, uint32_t e) {
    uint32_t* w = &sm.map[lk >> 1];
    const int sh = (lk & 1) * 16;
    int res = -2;
    // the trip count is the same for every lane (the loop exits on __any):
    // the bound costs one scalar register
    for (int it = 0;; ++it) {
      if (res == -2 && it >= kSpinCap) {
        // the wait is cut short: this event is dropped and the pass redone
        lds_store(&sm.stuck, 1u);
        res = -1;
      }
      if (res == -2) {
        if (e < (uint32_t)NSLOT) {
          res = (int)e;
        } else if (e == kMapDone || e == kMapDefer) {
          res = -1;
        } else if (e == kMapEmpty) {
          const uint32_t word = lds_load(w);
          if (((word >> sh) & 0xFFFFu) == kMapEmpty) {
            const uint32_t want = (word & ~(0xFFFFu << sh)) | (kMapBusy << sh);
            if (atomicCAS(w, word, want) == word) {
              const uint32_t s = atomicAdd(&sm.nslots, 1u);
              uint32_t fin;
              if (s < (uint32_t)NSLOT) {
                sm.slot_kid[s] = (uint16_t)lk;
                fin = s;
                res = (int)s;
              } else {
                fin = kMapDefer;
                lds_store(&sm.poison, 1u);
                res = -1;
              }
              // our half is BUSY and only we change it: flip it to fin
              atomicXor(w, (kMapBusy ^ fin) << sh);
            }
          }
          if (res == -2) e = (lds_load(w) >> sh) & 0xFFFFu;
        } else {  // being claimed by another lane
          e = (lds_load(w) >> sh) & 0xFFFFu;
        }
      }
      if (!__any(res == -2)) break;
    }
    return res;
  }

  // Memory operations of hash_claim.
  struct LdsOps {
    __device__ __forceinline__ uint32_t load(const uint32_t* p) const { return lds_load(p); }
    __device__ __forceinline__ void store(uint32_t* p, uint32_t v) const { lds_store(p, v); }
    __device__ __forceinline__ uint32_t cas(uint32_t* p, uint32_t expect, uint32_t want) const {
      return atomicCAS(p, expect, want);
    }
    __device__ __forceinline__ uint32_t add(uint32_t* p, uint32_t v) const { return atomicAdd(p, v); }
    __device__ __forceinline__ void order() const { __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "workgroup", "local"); }
    __device__ __forceinline__ bool any(bool pending) const { return __any(pending); }
  };

  // Count bin b outside the inline window in a full pool record, claiming
  // one for the slot on first need (same exit discipline as map_claim).
  __device__ void pool_add(int slot, uint32_t m, int b) {
    bool pending = true;
    for (int it = 0;; ++it) {
      if (pending && it >= kSpinCap) {
        lds_store(&sm.stuck, 1u);
        pending = false;
      }
      if (pending) {
        const uint32_t st = (m >> 8) & 0xFFu;
        if (st == kStPoison) {
          pending = false;
        } else if (st != kStNone && st != kStBusy) {
          atomicAdd(&sm.pool[st - 1][b], 1u);
          pending = false;
        } else if (st == kStNone) {
          const uint32_t claim = (m & ~0xFF00u) | (kStBusy << 8);
          const uint32_t old = atomicCAS(&sm.meta[slot], m, claim);
          if (old == m) {
            const uint32_t idx = atomicAdd(&sm.npool, 1u);
            uint32_t fin;
            if (idx < (uint32_t)S::kPool) {
              atomicAdd(&sm.pool[idx][b], 1u);
              fin = (m & ~0xFF00u) | ((idx + 1u) << 8);
            } else {
              fin = (m & ~0xFF00u) | (kStPoison << 8);
              lds_store(&sm.poison, 1u);
            }
            // only the state field changes (it is ours while BUSY)
            atomicXor(&sm.meta[slot], (fin ^ claim) & 0xFF00u);
            pending = false;
          } else {
            m = old;
          }
        } else {
          m = lds_load(&sm.meta[slot]);
        }
      }
      if (!__any(pending)) break;
    }
  }

  // Span of the window in meta word m (its first bin set): first bin, width
  // (last bin - first), and the place of bin b of the span in the window.
  __device__ __forceinline__ static int span_lo(uint32_t m) { return (int)(m & 0xFFu); }
  __device__ __forceinline__ static uint32_t span_width(uint32_t m) {
    return MODE == kDense ? (uint32_t)WIN - 1 : (m >> 17) & 31u;
  }
  __device__ __forceinline__ static int win_at(uint32_t m, int b) {
    static_assert(MODE == kDense || WIN == 6 || WIN == 8, "b * 43 >> 8 is b / 6 up to 31");
    return MODE == kDense ? b - span_lo(m) : WIN == 8 ? b & 7 : b - WIN * ((b * 43) >> 8);
  }

  // Mapped and hashed modes: widen the span of slot's window to hold bin b
  // (m: its meta word, updated to the newest read); false when that would pass
  // WIN octaves. Spans only widen and a state changes at most twice, and a
  // failed swap means that another lane's succeeded, so the loop ends after a
  // bounded count.
  __device__ bool span_widen(int slot, uint32_t& m, int b) {
    while (true) {
      const bool unset = (m & 0xFFu) == kSpanUnset;
      const int lo = unset || b < span_lo(m) ? b : span_lo(m);
      const int last = span_lo(m) + (int)span_width(m), hi = unset || b > last ? b : last;
      if (hi - lo >= WIN) return false;
      const uint32_t want = (m & ~kSpanMask) | (uint32_t)lo | ((uint32_t)(hi - lo) << 17);
      if (want == m) return true;
      const uint32_t old = atomicCAS(&sm.meta[slot], m, want);
      if (old == m) {
        m = want;
        return true;
      }
      m = old;
    }
  }

  // mmv: min and max of the slot as read before this event (possibly stale:
  // min only falls and max only rises, so a stale read can only cause an
  // extra atomic, never a missed one)
  __device__ __forceinline__ void slot_add(int slot, uint32_t m, uint64_t d, const v2l& mmv) {
    if (m & kDone) return;
    const int b = octave_bin(d);
    bool in;
    if (MODE == kDense) {
      if ((m & 0xFFu) == kSpanUnset) {
        int base = b - WIN / 2 + 1;
        base = base < 0 ? 0 : (base > NB - WIN ? NB - WIN : base);
        const uint32_t want = (m & ~0xFFu) | (uint32_t)base;
        const uint32_t old = atomicCAS(&sm.meta[slot], m, want);
        m = (old == m) ? want : old;
      }
      in = (unsigned)(b - span_lo(m)) < (unsigned)WIN;
    } else {
      // unset: the first bin reads as 255 and the width as 0, so no bin lies in the span
      in = (uint32_t)(b - span_lo(m)) <= span_width(m) || span_widen(slot, m, b);
    }
    if (in)
      atomicAdd(&sm.win[slot][win_at(m, b)], 1u);
    else
      pool_add(slot, m, b);
    atomicAdd(&sm.sum[slot], (unsigned long long)d);
    if ((long long)d < mmv.x) atomicMin(&sm.mm[slot][0], (long long)d);
    if ((long long)d > mmv.y) atomicMax(&sm.mm[slot][1], (long long)d);
  }

  __device__ __forceinline__ void slot_reset(int s) {
    sm.sum[s] = 0;
    sm.mm[s][0] = INT64_MAX;
    sm.mm[s][1] = INT64_MIN;
#pragma unroll
    for (int w = 0; w < WIN; ++w) sm.win[s][w] = 0;
    sm.meta[s] = kSpanUnset;
  }
};

// Hashed mode, before a ranked pass: the first NSLOT of the keys left get the
// slots of their ranks. map[w]: rank of the first key left from word w on. An
// event outside these keys' range costs a comparison, one inside two four-byte
// LDS reads, and nothing is claimed. 256 segments of 400,000 events, 29,000 of
// 60,000 ids (15 passes, HBM bound): 8.0 ms with the table in every pass, 7.2
// so, 7.1 with one map range of 16,384 ids after another; 32,768 (kernel,
// stream) keys with Zipf kernels on every stream: 6.9, 6.5 and 11.5.
// A thread's keys past the last slot are counted by their words' set bits, not
// one by one (512 segments of 20,000 events, 32,768 keys: 859 -> 759 us).
template <typename S>
__device__ __forceinline__ void rank_left(S& sm, int tid) {
  constexpr int kWords = kHashIds / 32, kPer = kWords / kThreads, NSLOT = sizeof(sm.meta) / sizeof(sm.meta[0]);
  static_assert(kPer * kThreads == kWords && kWords + kThreads / 64 <= kHash, "words by thread, ranks in the map");
  uint32_t own = 0;
  for (int i = 0; i < kPer; ++i) own += (uint32_t)__popc(sm.left[tid * kPer + i]);
  uint32_t incl = own;
  for (int o = 1; o < 64; o <<= 1) {
    const uint32_t v = __shfl_up(incl, o, 64);
    if ((tid & 63) >= o) incl += v;
  }
  if ((tid & 63) == 63) sm.map[kWords + (tid >> 6)] = incl;
  lds_barrier();  // and the last use of the map before
  uint32_t rank = incl - own, all = 0;
  for (int w = 0; w < kThreads / 64; ++w) {
    const uint32_t n = sm.map[kWords + w];
    if (w < tid >> 6) rank += n;
    all += n;
  }
  for (int i = 0; i < kPer; ++i) {
    sm.map[tid * kPer + i] = rank;
    uint32_t bits = sm.left[tid * kPer + i], at = rank;
    rank += (uint32_t)__popc(bits);
    for (; bits && at < (uint32_t)NSLOT; bits &= bits - 1, ++at)
      sm.slot_kid[at] = (uint16_t)((tid * kPer + i) * 32 + __builtin_ctz(bits));
  }
  if (tid == 0) {
    sm.nslots = all < (uint32_t)NSLOT ? all : (uint32_t)NSLOT;
    sm.poison = all > (uint32_t)NSLOT ? 1u : 0u;
  }
}

// Four events of one thread: validity and per-segment aggregates, then the
// per-kernel updates. RANKED: hashed mode's later passes.
template <bool RANKED, int NSLOT, int WIN, int MODE>
__device__ __forceinline__ void process4(Seg<NSLOT, WIN, MODE>& sg, const Args& a, const int32_t (&kid)[4],
                                         const int32_t (&st)[4], const int64_t (&t0)[4], const int64_t (&t1)[4],
                                         int n, bool first_scan, uint32_t k_lo, uint32_t k_n, uint32_t& nv,
                                         uint32_t& ni, unsigned long long& busy, long long& tf, long long& tl) {
  uint64_t d[4];
  int lk[4];
#pragma unroll
  for (int j = 0; j < 4; ++j) {
    const bool valid =
        j < n && kid[j] >= 0 && kid[j] < a.n_kernels && st[j] >= 0 && st[j] < a.n_streams && t0[j] >= 0 && t1[j] >= t0[j];
    d[j] = (uint64_t)t1[j] - (uint64_t)t0[j];
    if (!RANKED && first_scan && j < n) {
      if (valid) {
        nv++;
        busy += d[j];
        tf = t0[j] < tf ? t0[j] : tf;
        tl = t1[j] > tl ? t1[j] : tl;
        atomicAdd(&sg.sm.stream_busy[st[j]], (unsigned long long)d[j]);
      } else {
        ni++;
      }
    }
    const uint32_t key = a.key_ns ? (uint32_t)kid[j] * (uint32_t)a.key_ns + (uint32_t)st[j] : (uint32_t)kid[j];
    lk[j] = valid && (!RANKED || key - k_lo < k_n) ? (int)key : -1;
  }
  // per-kernel updates two events at a time: their LDS lookups are issued
  // together, and the live register set stays small enough that nothing
  // spills around the scan loop
#pragma unroll
  for (int h = 0; h < 4; h += 2) {
    int slot[2];
    if (RANKED) {
      uint32_t w[2], first[2];
#pragma unroll
      for (int j = 0; j < 2; ++j) {
        w[j] = lk[h + j] >= 0 ? sg.sm.left[lk[h + j] >> 5] : 0u;
        first[j] = lk[h + j] >= 0 ? sg.sm.map[lk[h + j] >> 5] : 0u;
      }
#pragma unroll
      for (int j = 0; j < 2; ++j) {
        const uint32_t bit = 1u << (lk[h + j] & 31);
        slot[j] = w[j] & bit ? (int)(first[j] + (uint32_t)__popc(w[j] & (bit - 1))) : -1;
      }
    } else if (MODE == kHashed) {
      v4u e[2];
#pragma unroll
      for (int j = 0; j < 2; ++j)
        e[j] = *reinterpret_cast<const v4u*>(&sg.sm.map[hash_bucket(lk[h + j] >= 0 ? lk[h + j] : 0) * 4]);
#pragma unroll
      for (int j = 0; j < 2; ++j) {
        slot[j] = lk[h + j] >= 0 ? hash_find<NSLOT>(lk[h + j], e[j]) : -1;
        if (slot[j] == -2) {
          typename Seg<NSLOT, WIN, MODE>::LdsOps ops;
          slot[j] = hash_claim<NSLOT>(ops, sg.sm, lk[h + j], e[j], kSpinCap);
          if (slot[j] < 0) atomicOr(&sg.sm.left[lk[h + j] >> 5], 1u << (lk[h + j] & 31));
        }
      }
    } else if (MODE == kMapped) {
      uint32_t e[2];
#pragma unroll
      for (int j = 0; j < 2; ++j) e[j] = lk[h + j] >= 0 ? sg.map_get(lk[h + j]) : kMapDone;
#pragma unroll
      for (int j = 0; j < 2; ++j) {
        slot[j] = e[j] < (uint32_t)NSLOT ? (int)e[j] : -1;
        if (lk[h + j] >= 0 && e[j] >= (uint32_t)NSLOT && e[j] != kMapDone && e[j] != kMapDefer)
          slot[j] = sg.map_claim(lk[h + j], e[j]);
      }
    } else {
#pragma unroll
      for (int j = 0; j < 2; ++j) slot[j] = lk[h + j];
    }
    uint32_t m[2];
    v2l mmv[2];
#pragma unroll
    for (int j = 0; j < 2; ++j) {
      m[j] = slot[j] >= 0 ? sg.sm.meta[slot[j]] : 0u;
      mmv[j] = slot[j] >= 0 ? *reinterpret_cast<const v2l*>(&sg.sm.mm[slot[j]][0]) : v2l{0, 0};
    }
#pragma unroll
    for (int j = 0; j < 2; ++j)
      if (slot[j] >= 0) sg.slot_add(slot[j], m[j], d[h + j], mmv[j]);
  }
}

template <int NSLOT, int WIN, int MODE>
__global__ __launch_bounds__(kThreads) void summarize_kernel(Args a) {
  __shared__ Smem<NSLOT, WIN, MODE> sm;
  __shared__ int64_t g_next;
  Seg<NSLOT, WIN, MODE> sg{sm};
  const int tid = threadIdx.x;
  const int32_t K = a.n_keys, NS = a.n_streams;

  // Persistent workgroups pull segments from a queue, so the output stores
  // of one segment drain while the loads of the next are already in flight.
  // Threads share only LDS state, so every barrier orders LDS alone: no
  // barrier waits for the outputs' stores.
  while (true) {
  if (tid == 0) g_next = (int64_t)atomicAdd(a.queue, 1u);
  lds_barrier();
  // the segment index is wave-uniform: keep it (and what derives from it:
  // bounds, loop limits) in scalar registers
  const int64_t g = (int64_t)__builtin_amdgcn_readfirstlane((int)g_next);
  if (g >= a.n_seg) break;

  int64_t lo = a.seg_off[g], hi = a.seg_off[g + 1];
  const bool bad = !(lo >= 0 && lo <= hi && hi <= a.n_events && hi - lo <= (int64_t)UINT32_MAX);
  if (bad) {
    lo = hi = 0;
    if (tid == 0 && a.dev_status) atomicOr(a.dev_status, (int32_t)ARGUS_DEV_BAD_SEGMENT);
  }
  if (tid < NS) sm.stream_busy[tid] = 0;
  if (tid == 0) {
    sm.red_busy = 0;
    sm.red_wire = 0;
    sm.red_first = INT64_MAX;
    sm.red_last = INT64_MIN;
    sm.red_valid = 0;
    sm.red_invalid = 0;
  }

  // aligned part [a4, b4) in 4-event groups; head [lo, a4) and tail [b4, hi)
  int64_t a4 = lo, b4 = lo;
  if (a.vec_ok) {
    const int64_t up = (lo + 3) & ~(int64_t)3, dn = hi & ~(int64_t)3;
    a4 = up < hi ? up : hi;
    b4 = dn > a4 ? dn : a4;
  }
  const int64_t qa = a4 >> 2, qb = b4 >> 2;
  const v4i* K4 = reinterpret_cast<const v4i*>(a.kernel_id);
  const v4i* S4 = reinterpret_cast<const v4i*>(a.stream);
  const v2l* T0 = reinterpret_cast<const v2l*>(a.start_ns);
  const v2l* T1 = reinterpret_cast<const v2l*>(a.end_ns);

  uint32_t nv = 0, ni = 0;
  unsigned long long busy = 0, wire = 0;
  long long tf = INT64_MAX, tl = INT64_MIN;
  bool first_scan = true;
  int n_stuck = 0;  // passes of this segment that ended with a wait cut short

  if (MODE == kMapped)
    for (int i = tid; i < kMapIds / 2; i += kThreads) sm.map[i] = 0xFFFFFFFFu;
  else if (MODE == kDense)
    for (int s = tid; s < K; s += kThreads) sg.slot_reset(s);
  bool ranked = false;          // hashed mode: slots by rank among the keys left
  uint32_t k_lo = 0, k_n = 0;   // keys that a ranked pass looks at
  while (true) {
    // the mapped and hashed modes hand out slots afresh in every pass
    if (MODE == kHashed && !ranked) {
      for (int i = tid; i < kHash; i += kThreads) sm.map[i] = kHashEmpty;
      for (int i = tid; i < kHashIds / 32; i += kThreads) sm.left[i] = 0;
    }
    if (MODE != kDense)
      for (int s = tid; s < NSLOT; s += kThreads) sg.slot_reset(s);
    for (int i = tid; i < sm.kPool * NB; i += kThreads) (&sm.pool[0][0])[i] = 0;
    if (tid == 0) {
      sm.npool = 0;
      sm.poison = 0;
      sm.nslots = 0;
      sm.stuck = 0;
    }
    if (MODE == kHashed && ranked) rank_left(sm, tid);
    lds_barrier();
    if (MODE == kHashed && ranked) {
      k_lo = __builtin_amdgcn_readfirstlane(sm.slot_kid[0]);
      k_n = sm.nslots ? __builtin_amdgcn_readfirstlane(sm.slot_kid[sm.nslots - 1]) - k_lo + 1 : 0;
    }

    auto scan = [&](auto by_rank) __attribute__((always_inline)) {
      constexpr bool ranked_pass = decltype(by_rank)::value;
      // unaligned head and tail: at most 3 events each, on the first threads
      if (a.vec_ok) {
        int32_t kid[4], st[4];
        int64_t t0[4], t1[4];
        int n = 0;
        const int64_t h = a4 - lo, t = hi - b4;
        const int64_t i = tid < h ? lo + tid : (tid - h < t ? b4 + (tid - h) : -1);
        if (i >= 0) {
          kid[0] = a.kernel_id[i];
          st[0] = a.stream[i];
          t0[0] = a.start_ns[i];
          t1[0] = a.end_ns[i];
          n = 1;
        }
        for (int j = n; j < 4; ++j) {
          kid[j] = -1;
          st[j] = 0;
          t0[j] = t1[j] = 0;
        }
        if (n) process4<ranked_pass>(sg, a, kid, st, t0, t1, n, first_scan, k_lo, k_n, nv, ni, busy, tf, tl);
      }
      if (!a.vec_ok) {
        // scalar fallback for unaligned arrays: four strided events per thread
        for (int64_t i0 = lo + tid; i0 < hi; i0 += 4ll * kThreads) {
          int32_t kid[4], st[4];
          int64_t t0[4], t1[4];
          int n = 0;
#pragma unroll
          for (int j = 0; j < 4; ++j) {
            const int64_t i = i0 + (int64_t)j * kThreads;  // in range for a prefix of j
            const bool in = i < hi;
            kid[j] = in ? a.kernel_id[i] : -1;
            st[j] = in ? a.stream[i] : 0;
            t0[j] = in ? a.start_ns[i] : 0;
            t1[j] = in ? a.end_ns[i] : 0;
            n += in;
          }
          process4<ranked_pass>(sg, a, kid, st, t0, t1, n, first_scan, k_lo, k_n, nv, ni, busy, tf, tl);
        }
      }
      // aligned body: group q holds events 4q..4q+3; the next group's loads
      // are issued before the current group is processed
      {
        int64_t q = qa + tid;
        v4i nk4 = 0, ns4 = 0;
        v2l na0 = 0, na1 = 0, nb0 = 0, nb1 = 0;
        if (q < qb) {
          nk4 = __builtin_nontemporal_load(K4 + q);
          ns4 = __builtin_nontemporal_load(S4 + q);
          na0 = __builtin_nontemporal_load(T0 + 2 * q);
          na1 = __builtin_nontemporal_load(T0 + 2 * q + 1);
          nb0 = __builtin_nontemporal_load(T1 + 2 * q);
          nb1 = __builtin_nontemporal_load(T1 + 2 * q + 1);
        }
        while (q < qb) {
          const int32_t kid[4] = {nk4.x, nk4.y, nk4.z, nk4.w};
          const int32_t st[4] = {ns4.x, ns4.y, ns4.z, ns4.w};
          const int64_t t0[4] = {na0.x, na0.y, na1.x, na1.y};
          const int64_t t1[4] = {nb0.x, nb0.y, nb1.x, nb1.y};
          const int64_t qn = q + kThreads;
          if (qn < qb) {
            nk4 = __builtin_nontemporal_load(K4 + qn);
            ns4 = __builtin_nontemporal_load(S4 + qn);
            na0 = __builtin_nontemporal_load(T0 + 2 * qn);
            na1 = __builtin_nontemporal_load(T0 + 2 * qn + 1);
            nb0 = __builtin_nontemporal_load(T1 + 2 * qn);
            nb1 = __builtin_nontemporal_load(T1 + 2 * qn + 1);
          }
          process4<ranked_pass>(sg, a, kid, st, t0, t1, 4, first_scan, k_lo, k_n, nv, ni, busy, tf, tl);
          q = qn;
        }
      }
    };
    if (MODE == kHashed && ranked)
      scan(std::bool_constant<MODE == kHashed>{});
    else
      scan(std::false_type{});
    first_scan = false;
    lds_barrier();

    // A claim wait cut short dropped an update: every kernel of this pass is
    // redone (the per-segment aggregates were complete in the first scan).
    // After kMaxStuckPasses such passes the results are flushed as they are
    // and the condition is reported.
    const bool stuck = sm.stuck != 0;
    const bool redo_pass = stuck && n_stuck < kMaxStuckPasses;
    if (stuck) {
      if (!redo_pass && tid == 0 && a.dev_status) atomicOr(a.dev_status, (int32_t)ARGUS_DEV_SUMMARY_STALLED);
      ++n_stuck;
    }

    // flush: the count of every slot; sum, min, max and wire size of the
    // present ones
    const int nslot = MODE != kDense ? (int)(sm.nslots < (uint32_t)NSLOT ? sm.nslots : NSLOT) : (K < NSLOT ? K : NSLOT);
    for (int s = tid; s < (redo_pass ? 0 : nslot); s += kThreads) {
      const uint32_t m = sm.meta[s];
      const uint32_t pst = (m >> 8) & 0xFFu;
      if ((m & kDone) || pst == kStPoison) continue;
      uint32_t cnt = 0, nnz = 0;
#pragma unroll
      for (int w = 0; w < WIN; ++w) {
        cnt += sm.win[s][w];
        nnz += sm.win[s][w] != 0;
      }
      if (pst != kStNone) {
        for (int b = 0; b < NB; ++b) {
          cnt += sm.pool[pst - 1][b];
          nnz += sm.pool[pst - 1][b] != 0;
        }
      }
      const int64_t c = g * K + (MODE != kDense ? (int)sm.slot_kid[s] : s);
      a.count[c] = cnt;
      if (cnt) {
        a.sum_ns[c] = (int64_t)sm.sum[s];
        a.min_ns[c] = sm.mm[s][0];
        a.max_ns[c] = sm.mm[s][1];
        wire += 33u + 5u * nnz;
      }
    }
    // flush: histograms of the present slots (their span is set),
    // four bins per thread, 16-byte stores
    for (int it = tid; it < (redo_pass ? 0 : nslot) * (NB / 4); it += kThreads) {
      const int s = it >> 3, q = it & 7;
      const uint32_t m = sm.meta[s];
      const uint32_t pst = (m >> 8) & 0xFFu;
      if ((m & kDone) || pst == kStPoison || (m & 0xFFu) == kSpanUnset) continue;
      uint32_t v[4];
#pragma unroll
      for (int j = 0; j < 4; ++j) {
        const int b = 4 * q + j;
        v[j] = (uint32_t)(b - sg.span_lo(m)) <= sg.span_width(m) ? sm.win[s][sg.win_at(m, b)] : 0u;
        if (pst != kStNone) v[j] += sm.pool[pst - 1][b];
      }
      const int64_t c = g * K + (MODE != kDense ? (int)sm.slot_kid[s] : s);
      *reinterpret_cast<uint4*>(a.hist + c * NB + 4 * q) = make_uint4(v[0], v[1], v[2], v[3]);
    }
    if (MODE == kHashed && !ranked)
      for (int i = tid; i < kHashIds / 32; i += kThreads) sm.map[i] = 0;  // from here on: keys that had a slot
    lds_barrier();
    const bool again = sm.poison != 0 || redo_pass;
    // mark what was written; kernels that ran out of room start over
    for (int s = tid; s < nslot; s += kThreads) {
      const uint32_t m = sm.meta[s];
      if (m & kDone) continue;
      const bool redo = redo_pass || ((m >> 8) & 0xFFu) == kStPoison;
      if (MODE == kHashed) {
        const uint32_t k = sm.slot_kid[s], bit = 1u << (k & 31);
        if (ranked) {
          if (!redo) atomicAnd(&sm.left[k >> 5], ~bit);
        } else {
          atomicOr(&sm.map[k >> 5], bit);
          if (redo) atomicOr(&sm.left[k >> 5], bit);
        }
      } else if (MODE == kMapped) {
        sg.map_set(sm.slot_kid[s], redo ? (uint16_t)kMapEmpty : (uint16_t)kMapDone);
      } else if (redo) {
        sg.slot_reset(s);
      } else {
        sm.meta[s] = m | kDone;
      }
    }
    if (MODE == kMapped)
      for (int i = tid; i < K; i += kThreads)
        if (sg.map_get(i) == kMapDefer) sg.map_set(i, (uint16_t)kMapEmpty);
    lds_barrier();
    // keys that never occurred: count 0 (their other fields are not written)
    if (MODE == kHashed && !ranked && !redo_pass) {
      for (int i = tid; i < K; i += kThreads)
        if (!(((sm.map[i >> 5] | sm.left[i >> 5]) >> (i & 31)) & 1u)) a.count[g * K + i] = 0;
      ranked = true;
    }
    if (!again) break;
  }
  if (MODE == kMapped) {
    for (int i = tid; i < K; i += kThreads)
      if (sg.map_get(i) == kMapEmpty) a.count[g * K + i] = 0;
    lds_barrier();
  }

  // per-segment aggregates
  const unsigned long long wv = wave_sum_u64(nv), wi = wave_sum_u64(ni);
  const unsigned long long wb = wave_sum_u64(busy), ww = wave_sum_u64(wire);
  const long long wf = wave_min_i64(tf), wl = wave_max_i64(tl);
  if ((tid & 63) == 0) {
    atomicAdd(&sm.red_valid, (uint32_t)wv);
    atomicAdd(&sm.red_invalid, (uint32_t)wi);
    atomicAdd(&sm.red_busy, wb);
    atomicAdd(&sm.red_wire, ww);
    atomicMin(&sm.red_first, wf);
    atomicMax(&sm.red_last, wl);
  }
  lds_barrier();
  if (tid == 0) {
    a.n_valid[g] = sm.red_valid;
    a.n_invalid[g] = sm.red_invalid;
    a.t_first[g] = sm.red_first;
    a.t_last[g] = sm.red_last;
    a.step_ns[g] = sm.red_valid ? sm.red_last - sm.red_first : 0;
    a.busy_ns[g] = (int64_t)sm.red_busy;
    if (a.wire_bytes) a.wire_bytes[g] = (int64_t)sm.red_wire;
  }
  if (tid < NS) a.stream_busy_ns[g * NS + tid] = (int64_t)sm.stream_busy[tid];
  lds_barrier();
  }
}

// Workgroups resident at once (one per CU for the large tables): the grid
// of the persistent kernel. Cached per device and instantiation.
template <int NSLOT, int WIN, int MODE>
int resident_groups() {
  static std::atomic<int> cache[64];
  int dev = 0;
  if (hipGetDevice(&dev) != hipSuccess || dev < 0 || dev >= 64) return 0;
  int v = cache[dev].load(std::memory_order_relaxed);
  if (v == 0) {
    int cus = 0, per_cu = 0;
    if (hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess) return 0;
    if (hipOccupancyMaxActiveBlocksPerMultiprocessor(&per_cu, summarize_kernel<NSLOT, WIN, MODE>, kThreads, 0) !=
        hipSuccess)
      return 0;
    v = cus * (per_cu > 0 ? per_cu : 1);
    cache[dev].store(v, std::memory_order_relaxed);
  }
  return v;
}

template <int NSLOT, int WIN, int MODE>
hipError_t launch_t(const Args& args, int32_t n_seg, hipStream_t st) {
  const int groups = resident_groups<NSLOT, WIN, MODE>();
  if (groups <= 0) return hipErrorInvalidDevice;
  const int grid = n_seg < groups ? n_seg : groups;
  hipLaunchKernelGGL((summarize_kernel<NSLOT, WIN, MODE>), dim3(grid), dim3(kThreads), 0, st, args);
  return hipGetLastError();
}

bool aligned16(const void* p) { return (reinterpret_cast<uintptr_t>(p) & 15u) == 0; }

}  // namespace

hipError_t launch_summarize(const SummarizeLaunch& l, hipStream_t st) {
  const int32_t vec_ok =
      aligned16(l.kernel_id) && aligned16(l.stream) && aligned16(l.start_ns) && aligned16(l.end_ns) ? 1 : 0;
  const int32_t n_keys = l.keyed ? l.n_kernels * l.n_streams : l.n_kernels;
  Args a{l.kernel_id, l.stream, l.start_ns, l.end_ns, l.seg_off, l.n_events, l.n_kernels, l.n_streams,
         l.keyed ? l.n_streams : 0, n_keys, vec_ok, l.n_seg, l.queue, l.count, l.sum_ns, l.min_ns, l.max_ns, l.hist, l.n_valid, l.n_invalid, l.t_first, l.t_last,
         l.step_ns, l.busy_ns, l.stream_busy_ns, l.wire_bytes, l.dev_status};
  if (l.n_seg == 0) return hipSuccess;
  if (n_keys <= 64) return launch_t<64, 10, kDense>(a, l.n_seg, st);
  if (n_keys <= 512) return launch_t<512, 10, kDense>(a, l.n_seg, st);
  if (n_keys <= 2048) return launch_t<2048, 10, kDense>(a, l.n_seg, st);
  // Past the map's 16,384 entries the table of keys seen: with one map range
  // after another a segment is read once per range, and with windows fixed
  // around the first duration the full records ran out, each time for one
  // more read (512 segments of 400,000 events, 32,768 keys of which about
  // 1,900 occur, a third of them at 1x, 3x and 9x: 3.6 ms by ranges, 3.2 with
  // the table, 1.12 with the table and spans; the events read once take 0.8).
  // Up to 16,384 keys the map's one two-byte read is the cheaper lookup, with
  // room for windows of eight octaves: 4,096 segments of 200,000 events over
  // 8,200 ids, few of them wide, 4.38 ms (4.45 with six bins around the first
  // duration), 512 of 400,000 over 4,000 (kernel, stream) keys at up to three
  // scales 0.93 (2.11). A key space that fits the slots needs neither, and its
  // ten-bin window loses 4% to the span's extra instructions (2,048 keys: 3.55
  // against 3.66 ms).
  if (n_keys <= kMapIds) return launch_t<2048, 8, kMapped>(a, l.n_seg, st);
  return launch_t<2048, 6, kHashed>(a, l.n_seg, st);
}

}  // namespace argus
