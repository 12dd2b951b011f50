// The uploaded summary stream: dense per-(rank, step, key) summaries ->
// little-endian records of the present cells (section 5.2: only compact
// statistics leave the host; section 8.3 compares their size with the raw
// trace). The record layout is defined in include/argus.h.
//
// Launches, in order:
//   compact_clear   the segments' states and the ticket counter.
//   compact_kernel  one to eight wavefronts per segment, eight to a workgroup,
//                   in ticket order: each wavefront builds
//                   the records of a contiguous range of cells in its own LDS
//                   region, reading every summary field once; the
//                   segment's size is published, the sizes of the segments
//                   before it are added up (decoupled look-back), and the
//                   regions are copied to their final place with aligned
//                   4-byte stores (byte stores only at the two unaligned
//                   ends). Cells past a full region are only sized at first
//                   and read again once the place is known. A record is
//                   written only if it lies entirely inside the caller's
//                   buffer.
// 156 bytes of a present cell are read and 33 + 5 per nonzero bin written.
// Cluster step (10,240 x 2,048 cells, 4.0 GB): 1,755 us when the histograms
// were read once for sizes and once more for the records, a cell per thread;
// 1,290 us now (3.1 TB/s), of which the loads alone take 632 us, building the
// records 390 us (LDS: 5-byte entries at any alignment), the look-back 110 us
// and the copies 155 us, timed by leaving each out.
#include "argus_internal.h"

namespace argus {
namespace {

// Record bytes a wavefront stages: sixteen wavefronts share a CU's 160 KB.
constexpr int kRegion = 9856;
static_assert(8 * (33 + 5 * NB) <= kRegion, "a step of the largest records fits");
constexpr int kGroup = 8;                 // lanes per cell: four octave bins each
constexpr int64_t kMaxGrid = 1 << 20;     // workgroups per launch

// Segment state, one word: 2 bits of state above 62 bits of bytes.
constexpr uint64_t kSize = 1ull << 62;    // the segment's own bytes
constexpr uint64_t kPrefix = 2ull << 62;  // the bytes of all segments up to this one
constexpr uint64_t kBytes = kSize - 1;

struct CompactArgs {
  const uint32_t* count;
  const int64_t* sum;
  const int64_t* mn;
  const int64_t* mx;
  const uint32_t* hist;
  int32_t n_seg, n_cells, n_streams;
  uint8_t* out;
  int64_t cap;
  int64_t* seg_off;  // the last word is the ticket counter until the last segment writes the total there
  int32_t* dev_status;
  uint64_t* state;
};

__global__ __launch_bounds__(256) void compact_clear(CompactArgs a) {
  const int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x;
  if (i < a.n_seg) a.state[i] = 0;
  if (i == 0) {
    a.seg_off[a.n_seg] = 0;
    if (a.dev_status) *a.dev_status = 0;
  }
}

__device__ __forceinline__ void put4(uint8_t* p, uint32_t v) { __builtin_memcpy(p, &v, 4); }

__device__ __forceinline__ void wave_order() {
  __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
  __builtin_amdgcn_wave_barrier();
  __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

// Loaded steps of a wavefront: kGroup present cells each, kGroup lanes to a
// cell; lane sub of a cell holds four octave bins and, where records are
// built, one word of the record's head (sub 0: none).
constexpr int kSet = 4;
struct Steps {
  int cell[kSet];  // cell index in the segment, or -1
  uint4 h[kSet];
  uint32_t field[kSet];
};

// A place in a wavefront's cells: a window of kWindow cells and a step among
// its present cells.
constexpr int kWindow = 256;
struct Place {
  int c, step;
};

// Sizes the present cells from p up to cell c1 of the segment whose cell 0 is
// at row, adding to bytes. With kBuild their records are built in region while
// they fit; p is left at the first step that does not. Returns the bytes
// built. list: kWindow bytes of LDS of this wavefront. Two sets of steps
// alternate, so that one set's loads are in flight while the other's records
// are built.
template <bool kBuild>
__device__ __forceinline__ uint32_t take_cells(const CompactArgs& a, int64_t row, int c1, Place& p, uint8_t* region,
                                               uint8_t* list, uint64_t& bytes) {
  const int lane = threadIdx.x & 63, sub = lane & (kGroup - 1), grp = lane / kGroup;
  const uint64_t below = (1ull << lane) - 1;
  uint32_t at = 0;
  for (; p.c < c1; p.c += kWindow, p.step = 0) {
    const int c = p.c;
    uint32_t cnt[kWindow / 64];
#pragma unroll
    for (int q = 0; q < kWindow / 64; ++q) cnt[q] = c + 64 * q + lane < c1 ? a.count[row + c + 64 * q + lane] : 0u;
    int n = 0;
#pragma unroll
    for (int q = 0; q < kWindow / 64; ++q) {
      const uint64_t here = __ballot(cnt[q] != 0);
      if (cnt[q] != 0) list[n + __popcll(here & below)] = (uint8_t)(64 * q + lane);
      n += __popcll(here);
    }
    wave_order();
    const int steps = (n + kGroup - 1) / kGroup;
    auto load = [&](Steps& s, int first) {
#pragma unroll
      for (int u = 0; u < kSet; ++u) {
        const int i = (first + u) * kGroup + grp;
        s.cell[u] = i < n ? c + (int)list[i] : -1;
        s.h[u] = make_uint4(0, 0, 0, 0);
        s.field[u] = 0;
        if (s.cell[u] < 0) continue;
        const int64_t x = row + s.cell[u];
        s.h[u] = reinterpret_cast<const uint4*>(a.hist + x * NB)[sub];
        if (kBuild && sub != 0) {
          const uint32_t* f = reinterpret_cast<const uint32_t*>((sub < 4 ? a.sum : (sub < 6 ? a.mn : a.mx)) + x) + (sub & 1);
          s.field[u] = *(sub == 1 ? a.count + x : f);
        }
      }
    };
    // false: the region is full (p.step is the first step left)
    auto take = [&](const Steps& s, int first) -> bool {
#pragma unroll
      for (int u = 0; u < kSet; ++u) {
        if (first + u >= steps) break;
        // places from the nonzero bins of the lanes below
        const uint64_t b0 = __ballot(s.h[u].x != 0), b1 = __ballot(s.h[u].y != 0), b2 = __ballot(s.h[u].z != 0),
                       b3 = __ballot(s.h[u].w != 0);
        const int left = n - (first + u) * kGroup;
        const uint32_t nz = (uint32_t)(__popcll(b0) + __popcll(b1) + __popcll(b2) + __popcll(b3));
        const uint32_t len = 33u * (uint32_t)(left < kGroup ? left : kGroup) + 5u * nz;
        if (kBuild) {
          if (at + len > (uint32_t)kRegion) {
            p.step = first + u;
            return false;
          }
          uint32_t lower = 0;
          for (const uint64_t b : {b0, b1, b2, b3})
            lower = __builtin_amdgcn_mbcnt_hi((uint32_t)(b >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)b, lower));
          const uint32_t before = __shfl(lower, lane & ~(kGroup - 1), 64);  // those of the cells before this one
          if (s.cell[u] >= 0) {
            uint8_t* rec = region + at + 33u * (uint32_t)grp + 5u * before;
            uint32_t v = s.field[u];
            if (sub == 0)
              v = a.n_streams > 0
                      ? (uint32_t)(s.cell[u] / a.n_streams) | ((uint32_t)(s.cell[u] % a.n_streams) << 24)
                      : (uint32_t)s.cell[u];
            put4(rec + 4 * sub, v);
            uint8_t* e = rec + 33 + 5u * (lower - before);
            const uint32_t w[4] = {s.h[u].x, s.h[u].y, s.h[u].z, s.h[u].w};
#pragma unroll
            for (int q = 0; q < 4; ++q) {
              if (w[q] == 0) continue;
              e[0] = (uint8_t)(4 * sub + q);
              put4(e + 1, w[q]);
              e += 5;
            }
            // the last lane of the cell knows its number of nonzero bins
            if (sub == kGroup - 1) rec[32] = (uint8_t)((uint32_t)(e - rec - 33) / 5u);
          }
        }
        at += len;
        bytes += len;
      }
      return true;
    };
    Steps x, y;
    load(x, p.step);
    for (int s = p.step; s < steps; s += 2 * kSet) {
      load(y, s + kSet);
      if (!take(x, s)) return at;
      load(x, s + 2 * kSet);
      if (!take(y, s + kSet)) return at;
    }
    wave_order();  // the list is used to here
  }
  return at;
}

// region[0, len) to out[pos, pos + len): the whole wavefront.
__device__ __forceinline__ void copy_out(const CompactArgs& a, const uint8_t* region, uint32_t len, int64_t pos) {
  const int lane = threadIdx.x & 63;
  if (pos + (int64_t)len > a.cap) {
    // the records up to the first that does not fit
    uint32_t end = 0;
    while (end < len) {
      const uint32_t rec = 33u + 5u * region[end + 32];
      if (pos + (int64_t)(end + rec) > a.cap) break;
      end += rec;
    }
    len = end;
  }
  uint8_t* dst = a.out + pos;
  const uint32_t skew = (uint32_t)((0 - reinterpret_cast<uintptr_t>(dst)) & 3u);
  const uint32_t head = skew < len ? skew : len, words = (len - head) / 4, tail = (len - head) & 3u;
  const uint32_t* src = reinterpret_cast<const uint32_t*>(region);
  uint32_t* dw = reinterpret_cast<uint32_t*>(dst + head);
  for (uint32_t i = lane; i < words; i += 64) dw[i] = __builtin_amdgcn_alignbyte(src[i + 1], src[i], head);
  if ((uint32_t)lane < head) dst[lane] = region[lane];
  if ((uint32_t)lane < tail) dst[head + 4 * words + lane] = region[head + 4 * words + lane];
}

constexpr int kWaves = 8;  // wavefronts of a workgroup

// kShare wavefronts share a segment: a workgroup takes kWaves / kShare of them.
template <int kShare>
__global__ __launch_bounds__(64 * kWaves, 4) void compact_kernel(CompactArgs a, int64_t n_wg) {
  __shared__ alignas(16) uint8_t region_sh[kWaves][kRegion + 4];  // + a word that alignbyte may read past the end
  __shared__ uint8_t list_sh[kWaves][kWindow];
  __shared__ uint64_t wave_bytes[kWaves];
  __shared__ int64_t seg_sh, pos_sh;
  const int tid = threadIdx.x, lane = tid & 63, w = __builtin_amdgcn_readfirstlane(tid >> 6);
  // tickets number the segments in the order their workgroups started, so
  // every segment waited for below belongs to a workgroup that is running and
  // publishes its size without waiting for any other
  if (tid == 0) seg_sh = (int64_t)atomicAdd(reinterpret_cast<unsigned long long*>(a.seg_off + a.n_seg), 1ull);
  lds_barrier();
  const int64_t b = seg_sh;  // this workgroup's place: segments kWaves / kShare b on
  uint8_t* region = region_sh[w];
  const int64_t g = b * (kWaves / kShare) + w / kShare;
  const int64_t row = g * a.n_cells;
  const int per = kShare == 1 ? a.n_cells : ((a.n_cells + kShare - 1) / kShare + 15) / 16 * 16;
  const int64_t first = (int64_t)per * (w % kShare);
  const int c0 = g < a.n_seg && first < a.n_cells ? (int)first : a.n_cells;
  const int c1 = (int)((int64_t)c0 + per < a.n_cells ? (int64_t)c0 + per : a.n_cells);
  uint64_t bytes = 0;
  uint32_t staged = 0;
  Place p{c0, 0};
  int64_t pos = 0;
  for (bool placed = false;;) {
    if (a.cap > 0) staged = take_cells<true>(a, row, c1, p, region, list_sh[w], bytes);
    if (!placed) {
      placed = true;
      Place rest = p;
      take_cells<false>(a, row, c1, rest, region, list_sh[w], bytes);
      if (lane == 0) wave_bytes[w] = bytes;
      lds_barrier();
      uint64_t before = 0, all = 0;
#pragma unroll
      for (int v = 0; v < kWaves; ++v) {
        before += v < w ? wave_bytes[v] : 0;
        all += wave_bytes[v];
      }
      if (w == 0) {
        uint64_t excl = 0;
        if (b > 0) {
          if (lane == 0) __hip_atomic_store(&a.state[b], kSize | all, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
          // 64 predecessors at a time, nearest first, up to one whose prefix is known
          for (int64_t base = b - 1;;) {
            const int64_t i = base - lane;
            const uint64_t st = i >= 0 ? __hip_atomic_load(&a.state[i], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) : kPrefix;
            const uint64_t known = __ballot(st >> 62 == 2), none = __ballot(st >> 62 == 0);
            const int first = known ? __builtin_ctzll(known) : 63;
            if (none & (~0ull >> (63 - first))) {
              __builtin_amdgcn_s_sleep(1);
              continue;
            }
            excl += wave_sum_u64(lane <= first ? st & kBytes : 0ull);
            if (known) break;
            base -= 64;
          }
        }
        if (lane == 0) {
          __hip_atomic_store(&a.state[b], kPrefix | (excl + all), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
          pos_sh = (int64_t)excl;
          if (b == n_wg - 1) {  // every ticket has been taken
            a.seg_off[a.n_seg] = (int64_t)(excl + all);
            if ((int64_t)(excl + all) > a.cap && a.dev_status) atomicOr(a.dev_status, (int32_t)ARGUS_DEV_COMPACT_CAPACITY);
          }
        }
      }
      lds_barrier();
      pos = pos_sh + (int64_t)before;
      if (lane == 0 && g < a.n_seg && w % kShare == 0) a.seg_off[g] = pos;
    }
    if (staged == 0 || pos >= a.cap) break;
    copy_out(a, region, staged, pos);
    pos += staged;
    if (p.c >= c1) break;
    wave_order();
  }
}

}  // namespace

hipError_t launch_compact(const CompactLaunch& l, hipStream_t st) {
  CompactArgs a{l.count, l.sum_ns, l.min_ns, l.max_ns, l.hist, l.n_seg, l.n_cells, l.n_streams, l.out, l.capacity,
                l.seg_byte_off, l.dev_status, reinterpret_cast<uint64_t*>(l.sizes)};
  hipLaunchKernelGGL(compact_clear, dim3((unsigned)(((int64_t)l.n_seg + 255) / 256 + (l.n_seg == 0 ? 1 : 0))), dim3(256), 0,
                     st, a);
  hipError_t e = hipGetLastError();
  // Wavefronts to a segment: each takes about 64 cells one after another (0.1
  // us each), up to a workgroup's eight; fewer where the chain of places (about
  // 20 ns per workgroup) would then be the longer one, while a wavefront's
  // cells stay near what its region holds. With 1 / 2 / 4 / 8 of them, in us:
  // 100 segments of 512 cells 81 / 40 / 23 / 17, 1,024 of 128 cells 26 / 20 /
  // 24 / 38, 2,048 of 512 cells 97 / 73 / 82 / 96, 16,384 of 64 cells 97 / 139 /
  // 227 / 403.
  int share = 1;
  while (share < kWaves && share * 64 < l.n_cells) share *= 2;
  while (share > 1 && (int64_t)l.n_seg * share / kWaves > 6 * (int64_t)(l.n_cells / share) && l.n_cells / share * 2 <= 300)
    share /= 2;
  const int64_t n_wg = ((int64_t)l.n_seg * share + kWaves - 1) / kWaves;
  for (int64_t s = 0; s < n_wg && e == hipSuccess; s += kMaxGrid) {
    const dim3 n((unsigned)(n_wg - s < kMaxGrid ? n_wg - s : kMaxGrid)), t(64 * kWaves);
    if (share == 1) hipLaunchKernelGGL(compact_kernel<1>, n, t, 0, st, a, n_wg);
    else if (share == 2) hipLaunchKernelGGL(compact_kernel<2>, n, t, 0, st, a, n_wg);
    else if (share == 4) hipLaunchKernelGGL(compact_kernel<4>, n, t, 0, st, a, n_wg);
    else hipLaunchKernelGGL(compact_kernel<8>, n, t, 0, st, a, n_wg);
    e = hipGetLastError();
  }
  return e;
}

}  // namespace argus
