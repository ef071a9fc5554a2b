// barrier.h -- barrier instances of the redundant-barrier check over sorted
// keys (paper Sec. 4.2.3, the second loop of Alg. 5).
//
// After sorting, the records of one location and block form runs of equal
// epoch in epoch order, so the records that a block's barrier at boundary b
// separates on that location are two neighbouring runs: epoch b, then
// epoch b + 1.  The first element of an epoch run whose preceding run is
// the previous epoch of the same location and block marks one instance of
// that barrier (a visit-order change of the location it causes).  Both
// runs are summarised per action class by their smallest and largest thread,
// and the instance is racing when some pair across the two runs would race
// without the barrier: different threads, at least one write, not both
// atomic.
//
// Functions are usable from host and device code.
#pragma once
#include <stdint.h>

#include "keys.h"
#include "segstate.h"

#if defined(__HIPCC__)
#define SC_HDM __host__ __device__ __forceinline__
#else
#define SC_HDM inline
#endif

namespace sc {

// The records of one side of a barrier, per action class: the smallest and
// the largest thread (smallest above largest: none).
struct BarrierSide {
  uint32_t mn[3], mx[3];
  SC_HDM void clear() {
    for (int c = 0; c < 3; c++) {
      mn[c] = ~0u;
      mx[c] = 0;
    }
  }
  template <typename K>
  SC_HDM void add(const TraceLayout& L, K k) {
    add(action_class(k), key_ltid_t<K>(L, k));
  }
  SC_HDM void add(uint32_t c, uint32_t t) {
    for (uint32_t q = 0; q < 3; q++)
      if (c == q) {
        mn[q] = t < mn[q] ? t : mn[q];
        mx[q] = t > mx[q] ? t : mx[q];
      }
  }
  SC_HDM void merge(const BarrierSide& o) {
    for (int c = 0; c < 3; c++) {
      mn[c] = o.mn[c] < mn[c] ? o.mn[c] : mn[c];
      mx[c] = o.mx[c] > mx[c] ? o.mx[c] : mx[c];
    }
  }
  // fn(value, whether the smallest is wanted) over the lanes of a wave
  template <typename F>
  SC_HDM void reduce(F&& fn) {
    for (int c = 0; c < 3; c++) {
      mn[c] = fn(mn[c], true);
      mx[c] = fn(mx[c], false);
    }
  }
};

// Whether neighbouring keys w, x of a trace are the two epochs of an
// instance: the same location and block, and the next epoch (the epoch field
// lies at shift_e, below the location and block).
template <typename K>
SC_HD bool barrier_head(const TraceLayout& L, K w, K x) {
  const K rw = w >> L.shift_e, rx = x >> L.shift_e;
  return rx == rw + 1 && (rx >> L.eb) == (rw >> L.eb);
}

// Whether a thread of a's class i and a different one of b's class j exist.
SC_HD bool side_pair(const BarrierSide& a, int i, const BarrierSide& b, int j) {
  if (a.mn[i] > a.mx[i] || b.mn[j] > b.mx[j]) return false;
  return a.mn[i] != b.mx[j] || a.mx[i] != b.mn[j];
}

// A pair across the barrier that would race without it: not both reads and
// not both atomic.
SC_HD bool barrier_races(const BarrierSide& a, const BarrierSide& b) {
  bool r = false;
  for (int i = 0; i < 3; i++)
    for (int j = 0; j < 3; j++)
      if (i == CLS_W || j == CLS_W || i != j) r = r || side_pair(a, i, b, j);
  return r;
}

// Whether the element at position p of a trace's n sorted keys is the head
// of a barrier instance; then *boundary is the barrier's boundary (the
// epoch before it) and *racing whether the instance races.
template <typename K>
SC_HD bool barrier_instance(const TraceLayout& L, const K* keys, uint64_t n, uint64_t p, uint32_t* boundary,
                            bool* racing) {
  if (p == 0 || p >= n || !barrier_head<K>(L, keys[p - 1], keys[p])) return false;
  const K rw = keys[p - 1] >> L.shift_e, rx = keys[p] >> L.shift_e;
  BarrierSide before, after;
  before.clear();
  after.clear();
  for (uint64_t q = p; q > 0 && (keys[q - 1] >> L.shift_e) == rw; q--) before.add(L, keys[q - 1]);
  for (uint64_t q = p; q < n && (keys[q] >> L.shift_e) == rx; q++) after.add(L, keys[q]);
  *racing = barrier_races(before, after);
  *boundary = key_epoch_t<K>(L, keys[p - 1]);
  return true;
}

}  // namespace sc
