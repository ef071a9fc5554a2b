// filter.hip -- gfx950 kernels of the conflict filter (filter.h).
//
// The race check sorts 8-byte keys over five or six radix passes, about 150
// bytes of HBM traffic per record, although almost no record of a usual trace
// can race.  The filter reads every 16-byte record once and writes one 4-byte
// key, reads the keys once more, and leaves the full pipeline the few records
// that can: 24 bytes per record.
//   k_filter_begin  control words, tile -> trace and bucket -> trace tables
//   k_filter_part   per 16384-record tile: group hashes, the tile's keys
//                   ordered by hash bucket (writes and atomics of a bucket
//                   before its reads), bucket starts of the tile; record checks
//   k_filter_test   per bucket: LDS bitmaps of the bucket's groups, then an
//                   exact test of what they let through; survivors are marked
//                   in a bitmap over the call's records
//   k_filter_count / k_filter_scan / k_filter_gather  the marked records, in
//                   record order, and each trace's number of them
#include <hip/hip_runtime.h>

#include "filter.h"
#include "launch.h"
#include "wave.h"

namespace sc {

constexpr int FNT = 1024;              // threads of the partition and test kernels
constexpr int FNW = FNT / 64;
constexpr int FIT = FT / FNT;          // records per thread
constexpr uint32_t A_STRIDE = (1u << FILTER_SLOT_BITS) / 32;  // words of a stored bitmap
constexpr uint32_t HOT_READS = 1, HOT_WRITES = 2;
constexpr uint32_t SLOT_MASK = (1u << FILTER_SLOT_BITS) - 1;
static_assert(FT == 1u << FT_BITS && FILTER_SLOT_BITS + FT_BITS == 32, "a filter key is one 32-bit word");
static_assert(FILTER_SLOT_BITS + 1 + FILTER_MAX_LGB <= 32, "hash word: bucket bits, the write flag, slot bits");

// Block of a thread: a shift when threads per block is a power of two.
__device__ __forceinline__ uint32_t block_of(uint32_t tid, uint32_t tpb, uint32_t shift) {
  return shift < 32 ? tid >> shift : tid / tpb;
}
__device__ __forceinline__ uint32_t block_shift(uint32_t tpb) {
  return (tpb & (tpb - 1)) == 0 ? 31u - (uint32_t)__builtin_clz(tpb) : 32u;
}

__global__ __launch_bounds__(NT) void k_filter_begin(FilterBuffers f) {
  const uint32_t t = blockIdx.x;
  if (t == 0 && threadIdx.x == 0) {
    f.ctrl->pass_bits = 0;
    f.ctrl->error_flags = 0;
    f.ctrl->first_bad = ~0ull;
    f.ctrl->total_entries = 0;
    f.ctrl->wide_traces = 0;
    *f.n_hot = 0;
  }
  const FTrace T = f.tr[t];
  if (threadIdx.x == 0) f.trace_hot[(uint64_t)t * f.hot_stride] = 0;
  for (uint32_t i = threadIdx.x; i < T.ntiles; i += NT) f.tile_trace[T.tile0 + i] = t;
  if (T.ntiles)
    for (uint32_t i = threadIdx.x; i < 1u << T.lgb; i += NT) {
      f.bucket_trace[T.bucket0 + i] = t;
      f.hot[T.bucket0 + i] = 0;
    }
}

// ------------------------------------------------------- k_filter_part
// Bound by HBM: 16 bytes read and 4 written per record.  The order inside a
// bucket does not matter, so a key's place comes from one LDS atomic (its
// bucket's count of writes in the low half word, of reads in the high one)
// instead of a stable rank, and the tile is its own output range: no
// histogram pass and no offsets between tiles.  16384 records per tile make
// a tile's run of one bucket 32 keys (128 bytes) with 512 buckets; two
// workgroups of 1024 threads share a CU (72 KiB of LDS each; traces of more
// than 2^25 records take 4096 buckets and a workgroup per CU).
template <uint32_t LGB>
__global__ __launch_bounds__(FNT, LGB <= 11 ? 8 : 4) void k_filter_part(FilterBuffers f) {
  __shared__ uint32_t s_key[FT];
  __shared__ uint32_t s_cnt[1u << LGB];
  __shared__ uint32_t s_scan[FNW];
  const TileWalk tw = tile_walk(f.n_tiles, gridDim.x, blockIdx.x);
  if (tw.first >= tw.end) return;
  const uint32_t tile = tw.first, tx = threadIdx.x;
  const FTrace T = f.tr[f.tile_trace[tile]];
  const uint32_t local = tile - T.tile0;
  const uint64_t start = (uint64_t)local * FT;
  const uint32_t n_in = (uint32_t)min<uint64_t>((uint64_t)FT, T.n - start);
  const uint32_t B = 1u << T.lgb;
  const GRecords p = global_records((const char*)T.rec + start * 16);
  for (uint32_t k = tx; k < B; k += FNT) s_cnt[k] = 0;
  if (tx < (n_in + 31) / 32) f.survive[T.surv0 + local * (FT / 32) + tx] = 0;
  __syncthreads();
  const uint32_t shift = block_shift(T.tpb);
  uint32_t hv[FIT], rank[FIT / 2];  // ranks are 16-bit, two per word
  uint32_t bad = ~0u;
  constexpr int HALF = FIT / 4;  // records in flight per thread
#pragma unroll
  for (int half = 0; half < FIT / HALF; half++) {
    uint32_t tp = tx;
    asm volatile("" : "+v"(tp));  // per step: keeps the per-record indices and tests out of long-lived registers
    ulonglong2 v[HALF];
#pragma unroll
    for (int i = 0; i < HALF; i++) {
      const uint32_t j = tp + (half * HALF + i) * FNT;
      v[i] = j < n_in ? load_record(p, j) : ulonglong2{0ull, 0ull};
    }
#pragma unroll
    for (int i = 0; i < HALF; i++) {
      const int q = half * HALF + i;
      const uint32_t j = tp + q * FNT;
      const Rec x = unpack_rec(v[i]);
      const bool valid = j < n_in;
      if (valid && (x.action > 2 || x.space > 1)) bad = min(bad, j);
      const uint32_t h = filter_group(x.unit, block_of(x.tid, T.tpb, shift), x.epoch, x.space);
      const uint32_t w = x.action != 0 ? 1u : 0u;
      hv[q] = (h & ~(1u << FILTER_SLOT_BITS)) | (w << FILTER_SLOT_BITS);
      uint32_t rk = 0;
      if (T.lgb == 0) {  // one bucket: a count per wave, not 64 atomics on one word
        const uint64_t bw = __ballot(valid && w), br = __ballot(valid && !w);
        const uint64_t lt = (1ull << (tx & 63u)) - 1ull;
        uint32_t old = 0;
        if ((tx & 63u) == 0) old = atomicAdd(&s_cnt[0], (uint32_t)__popcll(bw) | ((uint32_t)__popcll(br) << 16));
        old = (uint32_t)__builtin_amdgcn_readfirstlane((int)old);
        rk = w ? (old & 0xFFFFu) + (uint32_t)__popcll(bw & lt) : (old >> 16) + (uint32_t)__popcll(br & lt);
      } else if (valid) {
        const uint32_t old = atomicAdd(&s_cnt[filter_bucket(h, T.lgb)], w ? 1u : 0x10000u);
        rk = w ? old & 0xFFFFu : old >> 16;
      }
      rank[q / 2] = (q & 1) ? rank[q / 2] | (rk << 16) : rk;
    }
  }
  if (bad != ~0u) {
    atomicOr(&f.ctrl->error_flags, LAYOUT_ERR_RECORD);
    atomicMin((unsigned long long*)&f.ctrl->first_bad, (unsigned long long)(T.off + start + bad));
  }
  __syncthreads();
  // bucket starts: thread t takes DPT consecutive buckets
  constexpr uint32_t DPT = (1u << LGB) / FNT;
  uint32_t c[DPT], sum = 0;
#pragma unroll
  for (uint32_t e = 0; e < DPT; e++) {
    const uint32_t b = tx * DPT + e;
    c[e] = b < B ? s_cnt[b] : 0u;
    sum += (c[e] & 0xFFFFu) + (c[e] >> 16);
  }
  uint32_t tot;
  uint32_t s0 = block_excl_sum_n<FNW>(sum, s_scan, &tot);
  uint32_t* row = f.rows + T.row0 + (uint64_t)local * (B + 1);
#pragma unroll
  for (uint32_t e = 0; e < DPT; e++) {
    const uint32_t b = tx * DPT + e;
    if (b < B) {
      const uint32_t pair = s0 | ((s0 + (c[e] & 0xFFFFu)) << 16);  // first write, first read
      s_cnt[b] = pair;
      row[b] = pair;
      // far more than a bucket's usual share: a hot word's reads, or writes
      // (few buckets, and each is flagged once or a few times).  Not where
      // the bucket is short all the same: another workgroup's worth or two
      // of reads is no delay among many.
      const uint32_t over = max(2 * (n_in >> T.lgb) + 16, 2 * FILTER_BUCKET / T.ntiles);
      const uint32_t hot = ((c[e] >> 16) > over ? HOT_READS : 0u) | ((c[e] & 0xFFFFu) > over ? HOT_WRITES : 0u);
      if (hot & ~f.hot[T.bucket0 + b]) atomicOr(&f.hot[T.bucket0 + b], hot);
      s0 += (c[e] & 0xFFFFu) + (c[e] >> 16);
    }
  }
  if (tx == 0) row[B] = n_in | (n_in << 16);
  __syncthreads();
#pragma unroll
  for (int q = 0; q < FIT; q++) {
    const uint32_t j = tx + q * FNT;
    if (j < n_in) {
      const uint32_t pair = s_cnt[filter_bucket(hv[q], T.lgb)];
      const uint32_t at = ((hv[q] >> FILTER_SLOT_BITS) & 1u ? pair & 0xFFFFu : pair >> 16) + ((q & 1) ? rank[q / 2] >> 16 : rank[q / 2] & 0xFFFFu);
      s_key[at] = ((hv[q] & SLOT_MASK) << FT_BITS) | j;
    }
  }
  __syncthreads();
  uint32_t* out = f.keys + T.off + start;
#pragma unroll
  for (int q = 0; q < FIT; q++) {
    const uint32_t j = tx + q * FNT;
    if (j < n_in) out[j] = s_key[j];
  }
}

// ------------------------------------------------------- k_filter_test
// One workgroup per bucket.  A bitmap over the slots of the bucket's groups
// marks where a write or atomic is (A), a second one, half as fine, where a
// write or atomic is not alone (D): another write's bit was set already, or a
// read's group has one.  Reads outside A and writes outside D cannot race.
// What is left, normally a few per cent, goes to a list and is tested on the
// records themselves: per group the smallest and largest thread (for a global
// word also the smallest and largest block) and the actions, in an LDS table,
// with a new hash each round.  Group hashes may collide: that keeps more
// records, never fewer.  A list that overflows is kept whole.
//
// Latency bounds it, not bytes (4 per record): a bucket's keys lie in one
// short run per tile, so the starts of many runs are read at once, and the
// keys of eight runs are in flight per thread.  Neighbouring buckets run at
// the same time on one XCD, so the lines their runs share are read once.
//
// A bucket with a hot word is taken apart: one workgroup would stream a
// million reads, and mark them with a million scattered atomics (c1: 94 of
// 160 us).  For hot reads it stores A, and k_filter_count, which has a
// workgroup per tile, tests the tile's run against it and sets the marks in
// LDS; all of the bucket's writes survive.  A bucket with hot writes survives
// whole, in the same way.


// Adds a bucket (b of its trace t) to the trace's list: its number, then
// (bucket << 2 | flags, place of A) pairs.  The place of its A, or ~0 when
// there is no room.
__device__ __forceinline__ uint32_t hot_place(const FilterBuffers& f, uint32_t t, uint32_t b, uint32_t flags) {
  uint32_t* const list = f.trace_hot + (uint64_t)t * f.hot_stride;
  uint32_t map = 0;
  if (!(flags & HOT_WRITES)) {
    map = atomicAdd(f.n_hot, 1u);
    if (map >= f.max_hot) return ~0u;
  }
  const uint32_t k = atomicAdd(&list[0], 1u);
  if (2 * k + 2 >= f.hot_stride) return ~0u;
  list[2 * k + 1] = (b << 2) | flags;
  list[2 * k + 2] = map;
  return map;
}

// The buckets the tiles have flagged.
__global__ __launch_bounds__(NT) void k_filter_plan(FilterBuffers f) {
  const uint32_t b = blockIdx.x * NT + threadIdx.x;
  if (b >= f.n_buckets) return;
  const uint32_t hot = f.hot[b];
  if (!hot) return;
  const uint32_t t = f.bucket_trace[b], place = hot_place(f, t, b - f.tr[t].bucket0, hot);
  f.hot[b] = place == ~0u ? 0u : (place << 2) | hot;  // (without room an ordinary bucket, if a slow one)
}

template <int NTH, uint32_t SB, uint32_t CAP, uint32_t CHUNK>
__global__ __launch_bounds__(NTH, 8) void k_filter_test(FilterBuffers f) {
  constexpr uint32_t A_WORDS = (1u << SB) / 32, D_WORDS = A_WORDS / 2;
  constexpr uint32_t X_SLOTS = (A_WORDS + D_WORDS) / 3;  // slots of the exact table: smallest, largest id, actions
  static_assert((X_SLOTS & (X_SLOTS - 1)) == 0, "the exact table is a power of two");
  constexpr int XPT = CAP / NTH;
  __shared__ __align__(16) uint32_t s_map[A_WORDS + D_WORDS];
  __shared__ uint32_t s_list[CAP];
  __shared__ uint32_t s_pair[CHUNK];
  __shared__ uint16_t s_end[CHUNK];
  __shared__ uint32_t s_n, s_any;
  const uint32_t tx = threadIdx.x;
  const TileWalk tw = tile_walk(f.n_buckets, gridDim.x, blockIdx.x);
  if (tw.first >= tw.end) return;
  const uint32_t bucket = tw.first, hot = f.hot[bucket];
  if (hot & HOT_WRITES) return;
  const FTrace T = f.tr[f.bucket_trace[bucket]];
  const uint32_t b = bucket - T.bucket0, B = 1u << T.lgb;
  const uint32_t sbits = min(T.sbits, SB), smask = (1u << sbits) - 1;  // (the host gives it SB at most)
  uint32_t* const A = s_map;
  uint32_t* const D = s_map + A_WORDS;
  const uint32_t a_words = 1u << (sbits - 5), d_words = a_words / 2;
  for (uint32_t k = 4 * tx; k < a_words; k += 4 * NTH) *(uint4*)(A + k) = make_uint4(0, 0, 0, 0);
  for (uint32_t k = 4 * tx; k < d_words; k += 4 * NTH) *(uint4*)(D + k) = make_uint4(0, 0, 0, 0);
  if (tx == 0) {
    s_n = 0;
    s_any = 0;
  }
  const uint32_t* rows = f.rows + T.row0 + b;
  // the starts and ends of the bucket's runs in tiles c0 .. c0 + n - 1
  auto load_runs = [&](uint32_t c0, uint32_t n) {
    __syncthreads();
    for (uint32_t i = tx; i < n; i += NTH) {
      const uint32_t* r = rows + (uint64_t)(c0 + i) * (B + 1);
      s_pair[i] = r[0];
      s_end[i] = (uint16_t)(r[1] & 0xFFFFu);
    }
    __syncthreads();
  };
  // The writes (or reads) of run i, from place `at` of its tile on: one key
  // per lane of a group and step, U steps at once; bit u of the result: k[u]
  // is a key.
  auto load_keys = [&](uint32_t c0, uint32_t i, bool writes, uint32_t skip, uint32_t lg, auto& k, bool* more) {
    constexpr uint32_t U = sizeof(k) / sizeof(k[0]);
    const uint32_t L = 1u << lg, pr = s_pair[i];
    const uint32_t at = (writes ? pr & 0xFFFFu : pr >> 16) + skip + (tx & (L - 1)), end = writes ? pr >> 16 : s_end[i];
    const uint32_t* p = f.keys + (T.off + (c0 + i) * FT);
    uint32_t live = 0;
#pragma unroll
    for (uint32_t u = 0; u < U; u++)
      if (at + u * L < end) {
        k[u] = p[at + u * L];
        live |= 1u << u;
      }
    *more = at + U * L < end;
    return live;
  };
  // fn(key, record index in the trace) for every write (or read) in runs
  // 0 .. n - 1 from tile c0 on, a run per group of 2^lg lanes
  auto for_runs = [&](uint32_t c0, uint32_t n, bool writes, uint32_t lg, auto&& fn) {
    constexpr uint32_t U = 8;
#pragma unroll 1
    for (uint32_t i = tx >> lg; i < n; i += NTH >> lg) {
      uint32_t skip = 0;
      bool more;
      do {
        uint32_t k[U];
        const uint32_t live = load_keys(c0, i, writes, skip, lg, k, &more);
#pragma unroll
        for (uint32_t u = 0; u < U; u++)
          if ((live >> u) & 1u) fn(k[u], (c0 + i) * FT + (k[u] & (FT - 1)));
        skip += U << lg;
      } while (more);
    }
  };
  // Lanes per run: with U keys per lane a group holds a run's usual length
  // and four deviations more, so few runs need a second step.
  auto lanes_for = [&](uint32_t len, uint32_t u) {
    const uint32_t want = (len + 4 * (uint32_t)__builtin_sqrtf((float)len) + u - 1) / u;
    return min(want <= 1 ? 0u : 32u - (uint32_t)__builtin_clz(want - 1), NTH == 1024 ? 10u : 9u);
  };
  constexpr uint32_t UW = 16;  // a thread's writes, when they stay in registers
  const uint32_t run = FT >> T.lgb;
  const uint32_t lg_r = lanes_for(run - run / 4, 8), lg_w = lanes_for(run / 4, UW);

  // ---- A and D from the writes.  (Bits are looked at before they are set:
  //      the atomics of a hot word's lanes would go one by one.)
  bool any = false;
  auto see_write = [&](uint32_t k) {
    const uint32_t s = (k >> FT_BITS) & smask, bit = 1u << (s & 31u), s2 = s >> 1, bit2 = 1u << (s2 & 31u);
    any = true;
    uint32_t old = A[s >> 5];
    if (!(old & bit)) old = atomicOr(&A[s >> 5], bit);
    if ((old & bit) && !(D[s2 >> 5] & bit2)) atomicOr(&D[s2 >> 5], bit2);
  };
  const bool one_chunk = T.ntiles <= CHUNK;
  const bool held = T.ntiles <= (uint32_t)NTH >> lg_w && one_chunk;  // a run per group: its writes stay in registers
  uint32_t kw[UW], w_live = 0;
  bool w_more = false;
  if (held) {
    load_runs(0, T.ntiles);  // (its barriers also follow the clears above)
    const uint32_t i = tx >> lg_w;
    if (i < T.ntiles) w_live = load_keys(0, i, true, 0, lg_w, kw, &w_more);
#pragma unroll
    for (uint32_t u = 0; u < UW; u++)
      if ((w_live >> u) & 1u) see_write(kw[u]);
    uint32_t skip = UW << lg_w;
    bool more = w_more;
    while (more) {
      uint32_t k[4];
      const uint32_t live = load_keys(0, i, true, skip, lg_w, k, &more);
#pragma unroll
      for (uint32_t u = 0; u < 4; u++)
        if ((live >> u) & 1u) see_write(k[u]);
      skip += 4u << lg_w;
    }
  } else {
    for (uint32_t c0 = 0; c0 < T.ntiles; c0 += CHUNK) {
      const uint32_t n = min(CHUNK, T.ntiles - c0);
      load_runs(c0, n);
      for_runs(c0, n, true, lg_w, [&](uint32_t k, uint32_t) { see_write(k); });
    }
  }
  if (hot) {
    __syncthreads();  // A is complete
    for (uint32_t k = tx; k < A_WORDS; k += NTH) f.hot_maps[(uint64_t)(hot >> 2) * A_STRIDE + k] = k < a_words ? A[k] : 0u;
    return;
  }
  if (any) s_any = 1;
  __syncthreads();
  if (!s_any) return;  // nothing but reads

  // ---- reads in A
  uint32_t* const surv = f.survive + T.surv0;
  auto mark = [&](uint32_t idx) { atomicOr(&surv[idx >> 5], 1u << (idx & 31u)); };
  auto keep = [&](uint32_t idx) {  // one LDS atomic for the lanes that are here together
    const uint64_t m = __ballot(true), before = m & ((1ull << __lane_id()) - 1ull);
    uint32_t pos = 0;
    if (before == 0) pos = atomicAdd(&s_n, (uint32_t)__popcll(m));
    pos = (uint32_t)__builtin_amdgcn_readfirstlane((int)pos) + (uint32_t)__popcll(before);
    if (pos < CAP) s_list[pos] = idx;
    return pos < CAP;
  };
  auto read_hits = [&](uint32_t k) {
    const uint32_t s = (k >> FT_BITS) & smask, s2 = s >> 1, bit2 = 1u << (s2 & 31u);
    if (!((A[s >> 5] >> (s & 31u)) & 1u)) return false;
    if (!(D[s2 >> 5] & bit2)) atomicOr(&D[s2 >> 5], bit2);
    return true;
  };
  for (uint32_t c0 = 0; c0 < T.ntiles; c0 += CHUNK) {
    const uint32_t n = min(CHUNK, T.ntiles - c0);
    if (!one_chunk) load_runs(c0, n);
    for_runs(c0, n, false, lg_r, [&](uint32_t k, uint32_t idx) {
      if (read_hits(k)) keep(idx);
    });
  }
  __syncthreads();  // D is complete
  if (s_n > CAP) {
    // a word too hot for the list but not for the tiles' flags: the bucket
    // goes the way of the flagged ones, if there is room
    if (tx == 0) s_any = hot_place(f, f.bucket_trace[bucket], b, HOT_READS);
    __syncthreads();
    const uint32_t place = s_any;
    if (place != ~0u) {
      for (uint32_t k = tx; k < A_WORDS; k += NTH) f.hot_maps[(uint64_t)place * A_STRIDE + k] = k < a_words ? A[k] : 0u;
      return;
    }
    for (uint32_t c0 = 0; c0 < T.ntiles; c0 += CHUNK) {
      const uint32_t n = min(CHUNK, T.ntiles - c0);
      if (!one_chunk) load_runs(c0, n);
      for_runs(c0, n, false, lg_r, [&](uint32_t k, uint32_t idx) {
        if (read_hits(k)) mark(idx);
      });
    }
  }

  // ---- writes in D
  auto keep_or_mark = [&](uint32_t idx) {
    if (!keep(idx)) mark(idx);
  };
  auto in_d = [&](uint32_t k) {
    const uint32_t s2 = ((k >> FT_BITS) & smask) >> 1;
    return ((D[s2 >> 5] >> (s2 & 31u)) & 1u) != 0;
  };
  if (held) {
    const uint32_t i = tx >> lg_w;
#pragma unroll
    for (uint32_t u = 0; u < UW; u++)
      if (((w_live >> u) & 1u) && in_d(kw[u])) keep_or_mark(i * FT + (kw[u] & (FT - 1)));
    uint32_t skip = UW << lg_w;
    bool more = w_more;
    while (more) {
      uint32_t k[4];
      const uint32_t live = load_keys(0, i, true, skip, lg_w, k, &more);
#pragma unroll
      for (uint32_t u = 0; u < 4; u++)
        if (((live >> u) & 1u) && in_d(k[u])) keep_or_mark(i * FT + (k[u] & (FT - 1)));
      skip += 4u << lg_w;
    }
  } else {
    for (uint32_t c0 = 0; c0 < T.ntiles; c0 += CHUNK) {
      const uint32_t n = min(CHUNK, T.ntiles - c0);
      if (!one_chunk) load_runs(c0, n);
      for_runs(c0, n, true, lg_w, [&](uint32_t k, uint32_t idx) {
        if (in_d(k)) keep_or_mark(idx);
      });
    }
  }
  __syncthreads();

  // ---- the exact test, on the records (the bitmaps' LDS holds the table
  //      now)
  uint32_t n = s_n;
  uint32_t* const mn = s_map;
  uint32_t* const mx = s_map + X_SLOTS;
  uint32_t* const act = s_map + 2 * X_SLOTS;
  if (n > 0 && n <= CAP) {
    const GRecords p = global_records(T.rec);
    const uint32_t shift = block_shift(T.tpb);
    Rec x[XPT];
    uint32_t idx[XPT];
    bool live[XPT];
#pragma unroll
    for (int q = 0; q < XPT; q++) {
      live[q] = tx + q * NTH < n;
      if (!live[q]) continue;
      idx[q] = s_list[tx + q * NTH];
      x[q] = unpack_rec(load_record(p, idx[q]));
    }
    uint32_t before = n;
#pragma unroll 1
    for (uint32_t round = 0; round < 3; round++) {
      __syncthreads();
      for (uint32_t k = 4 * tx; k < X_SLOTS; k += 4 * NTH) {
        *(uint4*)(mn + k) = make_uint4(~0u, ~0u, ~0u, ~0u);
        *(uint4*)(mx + k) = make_uint4(0, 0, 0, 0);
        *(uint4*)(act + k) = make_uint4(0, 0, 0, 0);
      }
      if (tx == 0) s_n = 0;
      __syncthreads();
      uint32_t se[XPT], sl[XPT];
#pragma unroll
      for (int q = 0; q < XPT; q++) {
        if (!live[q]) continue;
        const uint32_t blk = block_of(x[q].tid, T.tpb, shift), a = 1u << (x[q].action & 3u);
        // threads of one block's epoch; blocks of a global word
        se[q] = filter_exact_hash(x[q].unit, blk, x[q].epoch, 2 + x[q].space, round) & (X_SLOTS - 1);
        sl[q] = x[q].space ? se[q] : filter_exact_hash(x[q].unit, 0, 0, 1, round) & (X_SLOTS - 1);
        atomicMin(&mn[se[q]], x[q].tid);
        atomicMax(&mx[se[q]], x[q].tid);
        atomicOr(&act[se[q]], a);
        if (!x[q].space) {
          atomicMin(&mn[sl[q]], blk);
          atomicMax(&mx[sl[q]], blk);
          atomicOr(&act[sl[q]], a);
        }
      }
      __syncthreads();
#pragma unroll
      for (int q = 0; q < XPT; q++) {
        if (!live[q]) continue;
        auto races = [&](uint32_t s) {
          const uint32_t c = act[s];
          return mn[s] != mx[s] && ((c & 2u) || (c & 5u) == 5u);  // a write, or a read and an atomic
        };
        live[q] = races(se[q]) || races(sl[q]);
        const uint64_t m = __ballot(live[q]);
        if (live[q] && (m & ((1ull << __lane_id()) - 1ull)) == 0) atomicAdd(&s_n, (uint32_t)__popcll(m));
      }
      __syncthreads();
      const uint32_t left = s_n;
      if (left + (left >> 3) > before) break;  // a round that drops little is the last
      before = left;
    }
#pragma unroll
    for (int q = 0; q < XPT; q++)
      if (live[q]) mark(idx[q]);
  } else {
    for (uint32_t i = tx; i < min(n, CAP); i += NTH) mark(s_list[i]);
  }
}

// ---------------------------------------------- the surviving records

// Survivors per tile, with the marks of its trace's hot buckets.
__global__ __launch_bounds__(NT) void k_filter_count(FilterBuffers f) {
  __shared__ uint32_t s_map[FT / 32];
  __shared__ uint32_t s_sum[NWAVE];
  const uint32_t tile = blockIdx.x, tx = threadIdx.x;
  const uint32_t t = f.tile_trace[tile];
  const FTrace T = f.tr[t];
  const uint32_t local = tile - T.tile0, B = 1u << T.lgb;
  const uint64_t start = (uint64_t)local * FT;
  const uint32_t words = (uint32_t)((min<uint64_t>((uint64_t)FT, T.n - start) + 31) / 32);
  uint32_t* s = f.survive + T.surv0 + local * (FT / 32);
  const uint32_t* list = f.trace_hot + (uint64_t)t * f.hot_stride;
  const uint32_t n_hot = min(list[0], (f.hot_stride - 1) / 2);
  uint32_t c = 0;
  if (n_hot) {
    for (uint32_t k = tx; k < words; k += NT) s_map[k] = s[k];
    __syncthreads();
    const uint32_t smask = (1u << T.sbits) - 1;
    const uint32_t* keys = f.keys + (T.off + start);
    // 16 lanes per bucket, more where there are few; each group takes HU
    // buckets at a time, their loads in flight together
    constexpr uint32_t HU = 4;
    const uint32_t lg = n_hot >= 16 ? 4u : 8u - (n_hot > 1 ? 32u - (uint32_t)__builtin_clz(n_hot - 1) : 0u);
    const uint32_t L = 1u << lg, groups = NT >> lg;
    for (uint32_t h0 = tx >> lg; h0 < n_hot; h0 += HU * groups) {
      uint32_t at[HU], reads[HU], end[HU], flags[HU], k[HU];
      const uint32_t* A[HU];
#pragma unroll
      for (uint32_t u = 0; u < HU; u++) {
        const uint32_t h = h0 + u * groups;
        at[u] = end[u] = 0;
        if (h < n_hot) {
          const uint32_t w = list[2 * h + 1];
          const uint32_t* row = f.rows + T.row0 + (uint64_t)local * (B + 1) + (w >> 2);
          const uint32_t pair = row[0];
          flags[u] = w & 3u;
          A[u] = f.hot_maps + (uint64_t)list[2 * h + 2] * A_STRIDE;
          at[u] = (pair & 0xFFFFu) + (tx & (L - 1));
          reads[u] = pair >> 16;
          end[u] = row[1] & 0xFFFFu;
        }
      }
      bool more = true;
      while (more) {
        more = false;
#pragma unroll
        for (uint32_t u = 0; u < HU; u++)
          if (at[u] < end[u]) k[u] = keys[at[u]];
#pragma unroll
        for (uint32_t u = 0; u < HU; u++)
          if (at[u] < end[u]) {
            const uint32_t j = k[u] & (FT - 1), sl = (k[u] >> FT_BITS) & smask;
            if (at[u] < reads[u] || (flags[u] & HOT_WRITES) || ((A[u][sl >> 5] >> (sl & 31u)) & 1u))
              atomicOr(&s_map[j >> 5], 1u << (j & 31u));
            at[u] += L;
            more |= at[u] < end[u];
          }
      }
    }
    __syncthreads();
    for (uint32_t k = tx; k < words; k += NT) {
      s[k] = s_map[k];
      c += (uint32_t)__popc(s_map[k]);
    }
  } else {
    for (uint32_t k = tx; k < words; k += NT) c += (uint32_t)__popc(s[k]);
  }
  c = wave_reduce(c, 0u, [](uint32_t a, uint32_t d) { return a + d; });
  if ((tx & 63u) == 0) s_sum[tx >> 6] = c;
  __syncthreads();
  if (tx == 0) f.tile_cnt[tile] = s_sum[0] + s_sum[1] + s_sum[2] + s_sum[3];
}

// One workgroup: the tiles' exclusive prefix, in place, and each trace's
// first survivor (the call's total at the end).
__global__ __launch_bounds__(FNT) void k_filter_scan(FilterBuffers f) {
  __shared__ uint32_t s_scan[FNW];
  const uint32_t per = (f.n_tiles + FNT - 1) / FNT, t0 = min(f.n_tiles, threadIdx.x * per), t1 = min(f.n_tiles, t0 + per);
  uint32_t sum = 0;
#pragma unroll 8
  for (uint32_t t = t0; t < t1; t++) sum += f.tile_cnt[t];
  uint32_t tot;
  uint32_t run = block_excl_sum_n<FNW>(sum, s_scan, &tot);
  for (uint32_t t = t0; t < t1; t++) {
    const uint32_t c = f.tile_cnt[t];
    f.tile_cnt[t] = run;
    run += c;
  }
  __syncthreads();  // (one workgroup: its global stores are visible to it after a barrier)
  for (uint32_t i = threadIdx.x; i <= f.n_traces; i += FNT) {
    const uint32_t tile = i < f.n_traces ? f.tr[i].tile0 : f.n_tiles;
    f.trace_off[i] = tile < f.n_tiles ? f.tile_cnt[tile] : tot;
  }
}

// The marked records of a tile, in record order, to the survivors' array
// (unless it cannot hold them all; the host then takes the full path).
__global__ __launch_bounds__(NT) void k_filter_gather(FilterBuffers f) {
  __shared__ uint16_t s_idx[FT];
  __shared__ uint32_t s_scan[NWAVE];
  const uint32_t tile = blockIdx.x, tx = threadIdx.x;
  if (f.trace_off[f.n_traces] > f.out_cap) return;
  const FTrace T = f.tr[f.tile_trace[tile]];
  const uint32_t local = tile - T.tile0;
  const uint64_t start = (uint64_t)local * FT;
  const uint32_t words = (uint32_t)((min<uint64_t>((uint64_t)FT, T.n - start) + 31) / 32);
  const uint32_t* s = f.survive + T.surv0 + local * (FT / 32);
  static_assert(FT / 32 == 2 * NT, "two bitmap words per thread");
  uint32_t w0 = 2 * tx < words ? s[2 * tx] : 0u, w1 = 2 * tx + 1 < words ? s[2 * tx + 1] : 0u;
  uint32_t tot;
  uint32_t at = block_excl_sum((uint32_t)(__popc(w0) + __popc(w1)), s_scan, &tot);
  if (!tot) return;
  for (; w0; w0 &= w0 - 1) s_idx[at++] = (uint16_t)(64 * tx + (uint32_t)__builtin_ctz(w0));
  for (; w1; w1 &= w1 - 1) s_idx[at++] = (uint16_t)(64 * tx + 32 + (uint32_t)__builtin_ctz(w1));
  __syncthreads();
  const GRecords p = global_records((const char*)T.rec + start * 16);
  const uint32_t first = f.tile_cnt[tile];
  for (uint32_t i = tx; i < tot; i += NT) {
    const uint32_t j = s_idx[i];
    ((ulonglong2*)f.out)[first + i] = load_record(p, j);
    if (f.side) f.out_side[first + i] = f.side[T.off + start + j];
  }
}

// -------------------------------------------------------- launch wrappers

static inline uint32_t cdiv(uint64_t a, uint64_t b) { return (uint32_t)((a + b - 1) / b); }

hipError_t launch_filter_part(const FilterBuffers& f, hipStream_t s) {
  if (f.max_lgb > FILTER_MAX_LGB) return hipErrorInvalidValue;
  hipLaunchKernelGGL(k_filter_begin, dim3(f.n_traces), dim3(NT), 0, s, f);
  hipError_t e = hipGetLastError();
  if (e != hipSuccess) return e;
  // (the instantiation's counters hold every bucket of the call's traces)
  static_assert(FILTER_MAX_LGB == 12, "the larger instantiation");
  hipLaunchKernelGGL(f.max_lgb > 11 ? k_filter_part<12> : k_filter_part<11>, dim3(tile_grid(f.n_tiles, 0, 0)), dim3(FNT), 0, s, f);
  return hipGetLastError();
}
hipError_t launch_filter_test(const FilterBuffers& f, hipStream_t s) {
  hipLaunchKernelGGL(k_filter_plan, dim3(cdiv(f.n_buckets, NT)), dim3(NT), 0, s, f);
  hipError_t e = hipGetLastError();
  if (e != hipSuccess) return e;
  if (f.large)
    hipLaunchKernelGGL((k_filter_test<1024, 18, 4096, 1024>), dim3(tile_grid(f.n_buckets, 0, 0)), dim3(1024), 0, s, f);
  else
    hipLaunchKernelGGL((k_filter_test<512, 17, 2048, 512>), dim3(tile_grid(f.n_buckets, 0, 0)), dim3(512), 0, s, f);
  return hipGetLastError();
}
hipError_t launch_filter_out(const FilterBuffers& f, hipStream_t s) {
  hipLaunchKernelGGL(k_filter_count, dim3(f.n_tiles), dim3(NT), 0, s, f);
  hipError_t e = hipGetLastError();
  if (e != hipSuccess) return e;
  hipLaunchKernelGGL(k_filter_scan, dim3(1), dim3(FNT), 0, s, f);
  if ((e = hipGetLastError()) != hipSuccess) return e;
  hipLaunchKernelGGL(k_filter_gather, dim3(f.n_tiles), dim3(NT), 0, s, f);
  return hipGetLastError();
}

}  // namespace sc
