// Test probe (not part of libargus; host code only): runs the claim of
// summarize's hash table (summarize_hash.h, the very function the kernel
// calls) on host memory, several threads of a workgroup as coroutines, one
// memory operation at a time in every order.
#include <stdint.h>
#include <ucontext.h>

#include <cstdlib>
#include <vector>

#include "../../paper_2606_20374_amd/csrc/summarize_hash.h"

namespace {

constexpr int kSlots = 4;       // slots of the table under test
constexpr int kMaxThreads = 4;  // coroutines
constexpr int kMaxRounds = 6;   // of a claim's loop; schedules that let one spin for longer are cut
constexpr size_t kStack = 1 << 16;

struct Table {
  uint32_t map[argus::kHash];
  uint16_t slot_kid[kSlots];
  uint32_t nslots, poison, stuck;
};

struct Run;

// Memory operations of one thread: each is a step that the schedule picks.
struct Ops {
  Run* run;
  int id, rounds;
  void step();
  uint32_t load(const uint32_t* p) { return step(), *p; }
  void store(uint32_t* p, uint32_t v) { step(), *p = v; }
  uint32_t cas(uint32_t* p, uint32_t expect, uint32_t want) {
    step();
    const uint32_t old = *p;
    if (old == expect) *p = want;
    return old;
  }
  uint32_t add(uint32_t* p, uint32_t v) {
    step();
    const uint32_t old = *p;
    *p += v;
    return old;
  }
  void order() {}
  bool any(bool pending);
};

struct Run {
  Table t;
  int n, key[kMaxThreads], res[kMaxThreads];
  bool over[kMaxThreads], cut;
  Ops ops[kMaxThreads];
  ucontext_t ctx[kMaxThreads], main_ctx;
  std::vector<char> stack[kMaxThreads];
};

void Ops::step() { swapcontext(&run->ctx[id], &run->main_ctx); }
bool Ops::any(bool pending) {
  if (pending && ++rounds >= kMaxRounds) {
    run->cut = true;
    step();  // never picked again
  }
  return pending;
}

void body(unsigned hi, unsigned lo, int id) {
  Run* r = reinterpret_cast<Run*>(((uintptr_t)hi << 32) | lo);
  Ops& o = r->ops[id];
  o.step();
  argus::v4u e;
  for (int i = 0; i < 4; ++i) e[i] = r->t.map[argus::hash_bucket(r->key[id]) * 4 + i];
  int s = argus::hash_find<kSlots>(r->key[id], e);
  if (s == -2) s = argus::hash_claim<kSlots>(o, r->t, r->key[id], e, 1 << 16);
  r->res[id] = s;
  r->over[id] = true;
  o.step();
}

// A workgroup's threads up to the end of a pass under one schedule: choice[i]
// is the i-th step's pick among the threads still running (grown with zeros),
// width[i] their number.
void play(Run& r, std::vector<int>& choice, std::vector<int>& width) {
  r.cut = false;
  width.clear();
  for (int i = 0; i < r.n; ++i) {
    r.over[i] = false;
    r.ops[i] = Ops{&r, i, 0};
    r.stack[i].resize(kStack);
    getcontext(&r.ctx[i]);
    r.ctx[i].uc_stack.ss_sp = r.stack[i].data();
    r.ctx[i].uc_stack.ss_size = kStack;
    r.ctx[i].uc_link = nullptr;
    const uintptr_t p = reinterpret_cast<uintptr_t>(&r);
    makecontext(&r.ctx[i], reinterpret_cast<void (*)()>(body), 3, (unsigned)(p >> 32), (unsigned)p, i);
  }
  for (size_t k = 0; !r.cut; ++k) {
    int alive[kMaxThreads], m = 0;
    for (int i = 0; i < r.n; ++i)
      if (!r.over[i]) alive[m++] = i;
    if (m == 0) break;
    width.push_back(m);
    if (k == choice.size()) choice.push_back(0);
    swapcontext(&r.main_ctx, &r.ctx[alive[choice[k] % m]]);
  }
}

// Whether the end state is one from which the kernel reports every event: a
// dropped event's key has no slot (the next pass takes it) and asks for that
// pass; equal keys share a slot and different ones do not.
bool sound(const Run& r) {
  for (int i = 0; i < r.n; ++i) {
    if (r.res[i] < -1 || r.res[i] >= kSlots || r.t.stuck) return false;
    if (r.res[i] >= 0 && r.t.slot_kid[r.res[i]] != r.key[i]) return false;
    if (r.res[i] < 0 && !r.t.poison) return false;
    for (int j = 0; j < r.n; ++j)
      if (r.key[i] == r.key[j] && r.res[i] != r.res[j]) return false;
  }
  return true;
}

}  // namespace

// Plays n threads with the given keys from a table that has handed out used
// slots (to keys 0 .. used - 1): every schedule if random is 0, else that many
// random ones. out: schedules played to their end, and those that lose events.
extern "C" int probe_hash_claim(const int32_t* keys, int32_t n, int32_t used, int64_t random, uint32_t seed,
                                int64_t* out) {
  if (n < 1 || n > kMaxThreads || used < 0 || used > kSlots) return -1;
  Run* r = new Run;
  static Table start;
  for (uint32_t& e : start.map) e = argus::kHashEmpty;
  for (int k = 0; k < used; ++k) {
    int p = argus::hash_bucket(k) * 4;
    while (start.map[p] != argus::kHashEmpty) p = (p + 1) & (argus::kHash - 1);
    start.map[p] = ((uint32_t)k << argus::kTagBits) | (uint32_t)k;
    start.slot_kid[k] = (uint16_t)k;
  }
  start.nslots = (uint32_t)used;
  r->n = n;
  for (int i = 0; i < n; ++i) r->key[i] = keys[i];
  out[0] = out[1] = 0;
  std::vector<int> choice, width;
  uint64_t x = seed * 2654435761ull + 88172645463325252ull;
  for (int64_t it = 0; random == 0 || it < random; ++it) {
    if (random) {
      choice.assign(64, 0);
      for (int& c : choice) {
        x ^= x << 13;
        x ^= x >> 7;
        x ^= x << 17;
        c = (int)((x >> 33) & 0xFF);
      }
    }
    // only what a claim may have written is put back
    for (int i = 0; i < n; ++i)
      for (int q = 0; q < 16; ++q) {
        const int p = (argus::hash_bucket(keys[i]) * 4 + q) & (argus::kHash - 1);
        r->t.map[p] = start.map[p];
      }
    if (it == 0) r->t = start;
    for (int s = 0; s < kSlots; ++s) r->t.slot_kid[s] = start.slot_kid[s];
    r->t.nslots = start.nslots;
    r->t.poison = r->t.stuck = 0;
    play(*r, choice, width);
    if (!r->cut) {
      ++out[0];
      out[1] += sound(*r) ? 0 : 1;
    }
    if (random) continue;
    // the next schedule in order: the last step with a thread left to pick
    choice.resize(width.size());
    while (!choice.empty() && choice.back() + 1 >= width[choice.size() - 1]) choice.pop_back();
    if (choice.empty()) break;
    ++choice.back();
  }
  delete r;
  return 0;
}
