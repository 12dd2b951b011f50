// The hash table that hands out summarize's slots in large key spaces. Its
// memory operations come from a policy class, so that the same steps run on
// the GPU's LDS and, one at a time in every order, in a CPU test.
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

#include "../../include/argus.h"

namespace argus {

// 2,048 buckets of four entries (one 16-byte LDS read), at most a quarter
// full, so all but about 0.5% of the keys lie in their own bucket. An entry:
// key << 12 | slot index, or being claimed / deferred in the slot's place;
// empty is all ones. The table serves a segment's first pass; the keys that
// get no slot in it take theirs by rank in the passes after it.
constexpr int kHashIds = ARGUS_MAX_KERNELS;
constexpr int kHash = 8192, kBucketShift = 32 - 11;
constexpr uint32_t kHashEmpty = 0xFFFFFFFFu, kTagBits = 12, kTagMask = 0xFFF, kTagBusy = 0xFFE, kTagDefer = 0xFFD;

typedef uint32_t v4u __attribute__((ext_vector_type(4)));

__host__ __device__ inline int hash_bucket(int key) { return (int)(((uint32_t)key * 0x9E3779B1u) >> kBucketShift); }

// The slot of key if its own bucket, read as e, holds it; else -2.
template <int NSLOT>
__host__ __device__ inline int hash_find(int key, const v4u& e) {
  int r = -2;
#pragma unroll
  for (int i = 0; i < 4; ++i) {
    const uint32_t s = e[i] ^ ((uint32_t)key << kTagBits);  // below NSLOT only for the key's published entry
    r = s < (uint32_t)NSLOT ? (int)s : r;
  }
  return r;
}

// Slot of key, which its bucket (read as e0) does not hold with a slot:
// claims the first empty entry from the bucket on, or finds the key further
// on; -1 when the key has no slot in this pass.
//
// Entries only go from empty to claimed to published, so the stale read e0
// can only start the walk early. At most NSLOT keys and one more per thread
// are inserted, so the walk always meets an empty entry.
//
// An event may be dropped only if its key gets no slot in this pass: a key
// with a slot is written out and never looked at again. A claim takes the
// entry before it counts its slot, so once the count is seen full, every
// claim still to come is deferred; an entry read after that, and still
// empty, therefore holds no slot for the key. An empty entry read before the
// count shows nothing: another thread may have claimed it for the same key
// and taken the last slot in between.
//
// Lanes of one wavefront may race for the same claim; the loop exits only
// when no active lane is still pending, so a winner's publish executes inside
// the loop, before a waiting lane of its own wavefront re-reads the entry.
template <int NSLOT, typename M, typename S>
__host__ __device__ inline int hash_claim(M& m, S& sm, int key, const v4u& e0, int spin_cap) {
  int res = -2;
  const uint32_t mine = (uint32_t)key << kTagBits;
  int skip = 4;
#pragma unroll
  for (int i = 3; i >= 0; --i) skip = e0[i] == kHashEmpty || (e0[i] & ~kTagMask) == mine ? i : skip;
  int pos = (hash_bucket(key) * 4 + skip) & (kHash - 1);
  for (int it = 0;; ++it) {
    if (res == -2 && it >= spin_cap) {
      m.store(&sm.stuck, 1u);
      res = -1;
    }
    if (res == -2) {
      uint32_t e = m.load(&sm.map[pos]);
      if (e == kHashEmpty && m.load(&sm.nslots) >= (uint32_t)NSLOT) {
        m.order();
        e = m.load(&sm.map[pos]);
        if (e == kHashEmpty) {
          m.store(&sm.poison, 1u);
          res = -1;
        }
      } else if (e == kHashEmpty) {
        e = m.cas(&sm.map[pos], kHashEmpty, mine | kTagBusy);
        if (e == kHashEmpty) {
          const uint32_t s = m.add(&sm.nslots, 1u);
          uint32_t tag = kTagDefer;
          if (s < (uint32_t)NSLOT) {
            sm.slot_kid[s] = (uint16_t)key;
            tag = s;
            res = (int)s;
          } else {
            m.store(&sm.poison, 1u);
            res = -1;
          }
          m.store(&sm.map[pos], mine | tag);
        }
      }
      if (res == -2 && e != kHashEmpty) {
        if ((e & ~kTagMask) != mine) {
          pos = (pos + 1) & (kHash - 1);
        } else {
          const uint32_t tag = e & kTagMask;
          if (tag < (uint32_t)NSLOT)
            res = (int)tag;
          else if (tag == kTagDefer)
            res = -1;
        }
      }
    }
    if (!m.any(res == -2)) break;
  }
  return res;
}

}  // namespace argus
