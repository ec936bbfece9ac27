// Host-side rules of the library's kernels and launches, made callable for test_host_rules.py.
#include "dfisher_internal.h"

extern "C" __attribute__((visibility("default"))) int rules_row_records(int rows, int lds, int cols) {
  return dfi::row_records(rows, lds, cols);
}

#include "gram.hip"

extern "C" __attribute__((visibility("default"))) void rules_gram_plan(int64_t n, int64_t m, int64_t lds, int prec, int aligned,
                                                                       int q, int mode, int64_t* nslice, int64_t* kslice) {
  const dfi::GramPlan p = dfi::gram_plan(n, m, lds, prec, aligned != 0, q, mode);
  *nslice = p.nslice;
  *kslice = p.kslice;
}

#include "workspace.h"

// A device of `capacity` bytes that counts what it is asked for.
struct FakeMemory {
  size_t capacity, used = 0;
  std::vector<std::pair<void*, size_t>> blocks;
  int64_t allocs = 0, refusals = 0, frees = 0, syncs = 0;
  uintptr_t next = 0x1000;
  void* alloc(size_t b) {
    if (used + b > capacity) {
      ++refusals;
      return nullptr;
    }
    ++allocs;
    used += b;
    blocks.push_back({reinterpret_cast<void*>(next += 0x1000), b});
    return blocks.back().first;
  }
  void free(void* p) {
    ++frees;
    for (auto& b : blocks)
      if (b.first == p) {
        used -= b.second;
        b.second = 0;
      }
  }
  void sync() { ++syncs; }
  size_t available() { return capacity - used; }
};
struct FakeContext {
  FakeMemory mem;
  dfi::Workspace ws;
};

#define RULES extern "C" __attribute__((visibility("default")))
RULES FakeContext* rules_ws_new(size_t capacity) { return new FakeContext{FakeMemory{capacity}, {}}; }
RULES void rules_ws_set(FakeContext* c, size_t capacity, int frozen) {
  c->mem.capacity = capacity;
  c->ws.frozen = frozen != 0;
}
// the level taken, -1: none
RULES int rules_ws_levels(FakeContext* c, const size_t* need, int levels, int can_grow) {
  int at = -1;
  const bool ok = dfi::ws_levels(c->ws, levels, can_grow != 0, [&](int l) { return need[at = l]; }, c->mem);
  return ok && need[at] <= c->ws.bytes ? at : -1;
}
// bytes held, allocations, refusals, frees, synchronisations
RULES void rules_ws_counts(FakeContext* c, int64_t* out) {
  const int64_t v[5] = {(int64_t)c->ws.bytes, c->mem.allocs, c->mem.refusals, c->mem.frees, c->mem.syncs};
  for (int i = 0; i < 5; ++i) out[i] = v[i];
}
RULES void rules_ws_delete(FakeContext* c) { delete c; }

// the jobs that share a launch, in launch order; returns how many
RULES int rules_colpass_together(const int64_t* n, const int64_t* m, int count, int* out) {
  std::vector<dfi::ColJob> jobs((size_t)count);
  for (int k = 0; k < count; ++k) {
    jobs[(size_t)k].n = n[k];
    jobs[(size_t)k].m = m[k];
  }
  const std::vector<int> at = dfi::colpass_together(jobs.data(), count);
  std::copy(at.begin(), at.end(), out);
  return (int)at.size();
}

RULES int rules_gram_candidates(int64_t n, int64_t m, int* out) {
  int count = 0;
  dfi::gram_q_candidates(n, m, (size_t)4 << 30, out, &count, 16);
  return count;
}
