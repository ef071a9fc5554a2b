// filter.hip -- gfx950 kernels of the grouped race count (filter.h).
//
// The sorting race check moves about 150 bytes of HBM per record: 8-byte keys
// over five or six radix passes.  Here every 16-byte record is read once, a
// 4-byte key is written and read back, and only records that may race are
// looked at again: 24 bytes per record.  One trace of 2^24 records takes 61 us
// in k_filter_part (5.5 TB/s), 170 in k_filter_count, 19 in k_entries_sort; the
// sort took 707 for the whole call.  A call of 1279 records takes 12 us in one
// count kernel and one synchronisation, 35 us in all; sorting took 102.
//   k_filter_begin  control words, tile -> trace and bucket -> trace tables
//   k_filter_part   per 16384-record tile: group hashes, the tile's keys
//                   ordered by hash bucket (writes and atomics of a bucket
//                   before its reads), bucket starts of the tile; record checks
//   k_filter_plan   workgroups for buckets with hot words
//   k_filter_count  per bucket: bitmaps of its groups in LDS, then the pairs
//                   of the writes and atomics that may race, among themselves
//                   and with the reads; one entry per racing location.  A second
//                   launch counts the buckets that the first left for later
//   k_entries_place / k_entries_sort / k_entries_merge  the entries in order
#include <hip/hip_runtime.h>

#include <algorithm>
#include <type_traits>

#include "filter.h"
#include "launch.h"
#include "segstate.h"
#include "wave.h"

namespace sc {

constexpr int FNT = 1024;              // threads of the partition and test kernels
constexpr int FNW = FNT / 64;
constexpr int FIT = FT / FNT;          // records per thread
constexpr uint32_t SLOT_MASK = (1u << FILTER_SLOT_BITS) - 1;
static_assert(FT == 1u << FT_BITS && FILTER_SLOT_BITS + FT_BITS == 31, "a filter key is one 32-bit word");
static_assert(FILTER_SLOT_BITS + 2 + FILTER_MAX_LGB <= 32, "hash word: bucket bits, write and atomic flags, slot bits");
constexpr uint32_t HV_ACTION = 3u << FILTER_SLOT_BITS;  // 0 read, 1 write, 2 atomic

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
    f.cnt[FC_ENTRIES] = 0;
    f.cnt[FC_EXTRA] = 0;
    f.cnt[FC_MOST] = 0;
    f.cnt[FC_LATE] = 0;
    f.cnt[FC_ROUNDS] = 0;
    f.cnt[FC_EXTRA2] = 0;
  }
  const FTrace T = f.tr_src[t];
  if (threadIdx.x == 0) {
    if (f.tr_src != f.tr) f.tr[t] = T;
    f.trace_cnt[t] = 0;
    f.trace_fill[t] = 0;
  }
  for (uint32_t i = threadIdx.x; i < T.ntiles; i += NT) f.tile_trace[T.tile0 + i] = t;
  if (T.ntiles)
    for (uint32_t i = threadIdx.x; i < 1u << T.lgb; i += NT) {
      f.bucket_trace[T.bucket0 + i] = t;
      f.hot[T.bucket0 + i] = 0;
      f.hot_writes[T.bucket0 + i] = 0;
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
// than 2^25 records take up to 8192 buckets and a workgroup per CU).
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
      const uint32_t act = x.action <= 2 ? x.action : 0u;  // (a bad record's call fails)
      const bool w = act != 0;
      hv[q] = (h & ~HV_ACTION) | (act << FILTER_SLOT_BITS);
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
      asm volatile("" : "+v"(hv[q]), "+v"(rank[q / 2]));  // (kept packed: their parts would spill)
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
  const uint32_t usual = n_in >> T.lgb;
#pragma unroll
  for (uint32_t e = 0; e < DPT; e++) {
    const uint32_t b = tx * DPT + e;
    if (b < B) {
      const uint32_t pair = s0 | ((s0 + (c[e] & 0xFFFFu)) << 16);  // first write, first read
      s_cnt[b] = pair;
      row[b] = pair;
      // far more reads than a bucket's usual share: a hot word's (rare, so
      // these atomics are few)
      if ((c[e] >> 16) > usual + usual / 4 + 8) atomicAdd(&f.hot[T.bucket0 + b], c[e] >> 16);
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
      const uint32_t at = ((hv[q] & HV_ACTION) ? pair & 0xFFFFu : pair >> 16) + ((q & 1) ? rank[q / 2] >> 16 : rank[q / 2] & 0xFFFFu);
      s_key[at] = ((hv[q] << (30 - FILTER_SLOT_BITS)) & FILTER_ATOMIC) | ((hv[q] & SLOT_MASK) << FT_BITS) | j;
    }
  }
  __syncthreads();
  // far more writes than a bucket's usual share of all records (32 of the keys
  // tell them from atomics): the rest are a hot word's
#pragma unroll 1
  for (uint32_t b = tx * DPT; b < min((tx + 1) * DPT, B); b++) {
    const uint32_t pair = s_cnt[b], w0 = pair & 0xFFFFu, nw = (pair >> 16) - w0;
    if (nw <= usual + usual / 4 + 8) continue;
    uint32_t plain = 0;
#pragma unroll 8
    for (uint32_t k = 0; k < 32; k++) plain += (s_key[w0 + nw * k / 32] & FILTER_ATOMIC) ? 0u : 1u;
    const uint32_t writes = nw * plain / 32;
    if (writes > usual + usual / 4 + 8) atomicAdd(&f.hot_writes[T.bucket0 + b], writes - usual);
  }
  uint32_t* out = f.keys + T.off + start;
#pragma unroll
  for (int q = 0; q < FIT; q++) {
    const uint32_t j = tx + q * FNT;
    if (j < n_in) out[j] = s_key[j];
  }
}

// ------------------------------------------------------ k_filter_count
// One workgroup per bucket.  Bitmaps over the slots of the bucket's groups
// mark where a write is (W, one bit per slot) and where an atomic is (T, one
// per four), and then, in D (one per two), where one of them may have a
// partner: a second write, or a read whose slot is in W or T.  Reads outside W
// and T cannot race, nor can writes and atomics outside D, writes outside T
// and atomics outside W.  Those that are left, normally a few hundred, are
// loaded into LDS as records and chained by location; each is paired with
// those before it in its chain, and each read that is left with all of its
// location's.  Group hashes may collide: that only adds candidates, the pairs
// are tested on the records themselves.
//
// Where the chains get long, or the table of WCAP writes and atomics does not
// hold them, a later workgroup counts the bucket (see LATE_BUCKET), in rounds,
// by slot, if need be.  Where a few rounds do not hold them for the atomics among
// them (a hot atomic word whose slot holds an unrelated write or read by chance),
// it thins those out first: the bucket's writes and reads that are left are
// hashed anew into four maps, and atomics that do not meet one in all of them are
// dropped.  What still does not fit is for the sort.
//
// Latency bounds it, not bytes (4 per record): a bucket's keys lie in one
// short run per tile.  So each lane loads four keys at once and has four such
// loads in flight, of one run or of several, and the lists are filled by one
// LDS atomic per wave and step.  Neighbouring buckets run at the same time on
// one XCD, so the lines their runs share are read once.
//
// A bucket with a hot word's reads (as the tiles counted them) is split: each
// further workgroup takes a range of tiles' reads and all of the bucket's
// writes.  A read's pairs depend on the writes alone; pairs of writes are the
// first part's.  Entries of one location from several parts (or, for a shared
// word, from the buckets of several epochs) are added up by the host.

// Workgroups of hot buckets: item i is (bucket, part).  They come first in the
// grid, also those of one part: started among the others, a bucket that takes
// four times as long ends long after them (215 us for a trace of 2^24 records,
// 170 so).  Where the items run out, a bucket (of HOT_BIG parts at most) stays whole
// and in its place.
constexpr uint32_t NO_BUCKET = 0xFFFFFFFFu, HOT_ITEM = 1u << 31;
// Written words whose writes no table of the allowed rounds holds (estimated
// from samples, hence the quarter more) are for the sort, and the sooner the
// better: a flag that a quarter of 2^24 records write was found out by one
// workgroup's passes over its bucket and their records (172 ms, before the sort's
// one); the call takes 1163 us so, the sort alone 1041.
constexpr uint32_t TABLE = 1024;  // writes and atomics a late workgroup's table holds
__device__ __forceinline__ uint32_t hopeless(uint32_t rounds) { return rounds * TABLE + rounds * TABLE / 4; }
__global__ __launch_bounds__(NT) void k_filter_plan(FilterBuffers f) {
  const uint32_t b = blockIdx.x * NT + threadIdx.x;
  if (b >= f.n_buckets) return;
  if (f.hot_writes[b] > hopeless(f.max_rounds)) atomicOr(&f.ctrl->error_flags, ERR_GROUP_FULL);
  const uint32_t hot = f.hot[b], parts = min(f.tr[f.bucket_trace[b]].ntiles, 1u + hot / f.hot_part);
  uint32_t word = 1;
  if (hot > f.hot_part / 4) {
    const bool big = parts > HOT_BIG;
    const uint32_t lo = big ? 0u : f.extra_big, max = big ? f.extra_big : f.extra_max - f.extra_big;
    const uint32_t at = atomicAdd(&f.cnt[big ? FC_EXTRA : FC_EXTRA2], parts);
    const bool room = at < max && parts <= max - at;
    for (uint32_t k = 0; k < parts && at + k < max; k++) f.extra[lo + at + k] = make_uint2(room ? b : NO_BUCKET, k);
    if (room) word = parts | HOT_ITEM;
  }
  f.hot[b] = word;
}

// Four keys, or two row words, from any word on.
typedef uint32_t words4 __attribute__((ext_vector_type(4), aligned(4)));
typedef uint32_t words2 __attribute__((ext_vector_type(2), aligned(4)));
typedef const __attribute__((address_space(1))) uint32_t* GWords;
__device__ __forceinline__ words4 load_words4(GWords p) { return *(const __attribute__((address_space(1))) words4*)p; }
__device__ __forceinline__ words2 load_words2(GWords p) { return *(const __attribute__((address_space(1))) words2*)p; }

// A call of short traces needs no partition: MODE DIRECT_TRACE is a workgroup
// per trace, which reads the records itself, keeps their keys in record order
// and makes the passes over those.  A call of 1279 records took 12 us in
// k_filter_part and 12 here, and takes 12 so (47 and 36 us in all).
//
// LATE_BUCKET and LATE_TRACE count what the other two hand over: buckets or
// traces with more candidates than a table holds, with a word of many writers or
// with long chains.  The others walk the chains of their table's records by
// location, which costs least where nearly all have no partner or one, and stop
// at CHAIN steps (MANY_WRITERS where the bucket has many reads); the late ones count by group (filter.h,
// GROUP_LEVELS), one look-up per level and read however many wrote the word.
// (800 writers and 3276 readers of a word in a trace of 2^14 records took 3309 us
// by chains, 100 so.)  They take a CU each, with twice the registers.
//
// ROUNDS: as BY_BUCKET or DIRECT_TRACE, but up to four tables of candidates are
// filled one after another before a bucket is handed over.  Random words collide
// often enough for that where nearly all records write.  The loop costs registers
// (batch of 4096 traces: 4405 us with it, 4137 without), so a context takes it
// after a call where one bucket in 32 was such (in a small call, any): 2^24
// records that all write words of their own take 691 us with later workgroups,
// 395 so.
enum : int { BY_BUCKET = 0, LATE_BUCKET = 1, DIRECT_TRACE = 2, LATE_TRACE = 3, ROUNDS = 4 };
template <int MODE, bool WARP, uint32_t WCAP, uint32_t RCAP>
__global__ __launch_bounds__(FNT, (MODE & LATE_BUCKET) ? 4 : 8) void k_filter_count(FilterBuffers f) {
  constexpr bool LATE = MODE & LATE_BUCKET, DIRECT = MODE & DIRECT_TRACE, LOOP = MODE & ROUNDS;
  constexpr uint32_t NTH = FNT;
  constexpr uint32_t SB = FILTER_SLOT_BITS, W_WORDS = (1u << SB) / 32, D_WORDS = W_WORDS / 2, T_WORDS = W_WORDS / 4;
  constexpr uint32_t HN = 512, END = 0xFFFFu;  // chains of writes, and as many of atomics
  constexpr uint32_t MANY_WRITERS = 16, CHAIN = 64;
  constexpr uint32_t HT = 8192, NONE = 0xFFFFFFFFu;  // the table of groups: index | level << 16
  constexpr uint32_t LEVELS = WARP ? GROUP_LEVELS + 1 : GROUP_LEVELS, WARP_WALK = 64;
  static_assert(LEVELS * WCAP < HT, "a free place in the table");
  static_assert(WCAP <= NTH, "a thread per entry of the table");
  constexpr uint32_t CLASSES = 64;
  constexpr uint32_t MAPS = 4, L_BITS = 15, L_WORDS = (1u << L_BITS) / 32;  // of the thinning
  static_assert(MAPS * L_WORDS <= W_WORDS, "they take W's place");
  static_assert(!LATE || WCAP == TABLE, "");
  __shared__ __align__(16) uint32_t s_map[W_WORDS + D_WORDS + T_WORDS];
  __shared__ uint32_t s_read[RCAP];
  __shared__ uint4 s_w[WCAP];
  __shared__ uint32_t s_blk[WCAP];    // their blocks; before them their record indices
  __shared__ uint32_t s_side[WARP ? WCAP : 1];
  __shared__ uint32_t s_acc[5][WCAP]; // pairs by kind of the location whose first one this is
  __shared__ uint16_t s_lead[WCAP];   // the first one of its location
  __shared__ uint16_t s_next[WCAP];   // the next of its chain (late: of its warp's group)
  constexpr uint32_t LCAP = LATE ? WCAP : 1;
  __shared__ uint32_t s_cnt[LEVELS][LCAP];  // writes | atomics << 16 of the group whose first one this is
  __shared__ uint32_t s_whead[WARP ? LCAP : 1];  // undiverged members of a warp's group
  __shared__ uint32_t s_cls[2][CLASSES];  // candidates by the low bits of their slot: all, writes
  __shared__ __align__(16) uint32_t tab[LATE ? HT : 4];
  __shared__ uint32_t s_n, s_nw, s_any, s_base;
  const uint32_t tx = threadIdx.x;
  uint32_t bucket, part = 0, trace = 0, share = 1;
  const uint32_t flags = DIRECT ? 0u : f.ctrl->error_flags;
  if (LATE) {
    // few items: two or four workgroups each, with a share of the reads
    const uint32_t n = min(f.cnt[FC_LATE], f.late_max);  // (more of them: the call sorts)
    if (!DIRECT) share = n <= 64 ? 4u : (n <= 128 ? 2u : 1u);
    if (blockIdx.x >= n * share) return;
    const uint2 it = f.late[blockIdx.x / share];
    bucket = DIRECT ? 0u : it.x;
    trace = it.x;
    part = it.y;
  } else if (DIRECT) {
    if (!f.tr[blockIdx.x].n) return;
    bucket = 0;
    trace = blockIdx.x;
  } else if (blockIdx.x < f.extra_max) {
    const bool big = blockIdx.x < f.extra_big;
    if (blockIdx.x - (big ? 0u : f.extra_big) >= f.cnt[big ? FC_EXTRA : FC_EXTRA2]) return;
    const uint2 it = f.extra[blockIdx.x];
    if (it.x == NO_BUCKET) return;
    bucket = it.x;
    part = it.y;
  } else {
    const TileWalk tw = tile_walk(f.n_buckets, gridDim.x - f.extra_max, blockIdx.x - f.extra_max);
    if (tw.first >= tw.end) return;
    bucket = tw.first;
  }
  auto uniform = [](uint32_t x) { return (uint32_t)__builtin_amdgcn_readfirstlane((int)x); };
  bucket = uniform(bucket);
  part = uniform(part);
  const uint32_t item = uniform(f.extra_max && !DIRECT ? f.hot[bucket] : 1u), parts = (item & ~HOT_ITEM) * uniform(share);
  if (LATE) part = part * uniform(share) + blockIdx.x % uniform(share);
  if (!LATE && !DIRECT && (item & HOT_ITEM) && blockIdx.x >= f.extra_max) return;
  trace = uniform(DIRECT ? trace : f.bucket_trace[bucket]);
  FTrace T = f.tr[trace];
  T.rec = (const void*)readfirstlane((uint64_t)T.rec);
  T.n = readfirstlane(T.n);
  T.row0 = readfirstlane(T.row0);
  T.off = uniform(T.off);
  T.tpb = uniform(T.tpb);
  T.ntiles = uniform(T.ntiles);
  T.bucket0 = uniform(T.bucket0);
  T.lgb = uniform(T.lgb);
  T.sbits = uniform(T.sbits);
  const uint32_t b = bucket - T.bucket0, B = 1u << T.lgb;
  const uint32_t smask = (1u << T.sbits) - 1;
  uint32_t* const W = s_map;
  uint32_t* const D = s_map + W_WORDS;
  uint32_t* const A = D + D_WORDS;  // atomics (T)
  for (uint32_t k = 4 * tx; k < W_WORDS + D_WORDS + T_WORDS; k += 4 * NTH) {
    // (a bucket of fewer slots uses the front of each map)
    const uint32_t w = k < W_WORDS ? k : (k < W_WORDS + D_WORDS ? 2 * (k - W_WORDS) : 4 * (k - W_WORDS - D_WORDS));
    if (w < 1u << (T.sbits - 5)) *(uint4*)(s_map + k) = make_uint4(0, 0, 0, 0);
  }
  if (tx == 0) {
    s_n = 0;
    s_nw = 0;
    if (LOOP) s_cls[0][0] = s_cls[0][1] = s_cls[0][2] = s_cls[0][3] = 0;
    s_any = (flags & ERR_GROUP_FULL) ? 3u : 0u;
  }
  __syncthreads();
  if (!DIRECT && s_any == 3) return;  // the call sorts (one thread has looked: all of the workgroup leave, or none)
  auto bit = [](const uint32_t* map, uint32_t s) { return (map[s >> 5] >> (s & 31u)) & 1u; };
  auto set = [&](uint32_t* map, uint32_t s) { return atomicOr(&map[s >> 5], 1u << (s & 31u)); };
  // ---- a pass over the bucket's writes (or reads) of tiles lo .. hi - 1:
  //      fn(four keys, which of them are keys, first record of their tile).
  //      A run is a group of 2^lg lanes' (four keys a lane and load); with
  //      more runs than groups and short runs a lane loads of 2^ml runs at
  //      once.  All lanes of a wave call fn together.  (One copy of fn per
  //      pass: straight code for all sixteen keys took longer to fetch than
  //      to run.)
  const GWords rows = (GWords)(f.rows + T.row0 + b);
  const GWords keys = (GWords)(f.keys + T.off);
  const uint32_t run = (uint32_t)min<uint64_t>(FT >> T.lgb, T.n);  // usual length
  auto for_keys_n = [&](auto nv, bool writes, uint32_t lo, uint32_t hi, auto&& fn) {
    constexpr uint32_t NV = decltype(nv)::value;  // loads in flight
    if constexpr (DIRECT) {
      uint32_t to = threadIdx.x;
      asm volatile("" : "+v"(to));
      for (uint32_t i0 = 0; i0 < (uint32_t)T.n; i0 += 4 * NV * NTH) {
        words4 x[NV];
#pragma unroll
        for (uint32_t v = 0; v < NV; v++) {
          x[v] = words4{0, 0, 0, 0};
          if (i0 + 4 * (to + v * NTH) < (uint32_t)T.n) x[v] = load_words4(keys + (i0 + 4 * (to + v * NTH)));
        }
#pragma unroll 1
        for (uint32_t v = 0; v < NV; v++) {
          const uint32_t i = i0 + 4 * (to + v * NTH);
          if (!__any(i < (uint32_t)T.n)) break;
          uint32_t k[4] = {x[0].x, x[0].y, x[0].z, x[0].w}, live = 0;
#pragma unroll
          for (uint32_t u = 0; u < 4; u++) {
            const uint32_t act = k[u] & 3u;
            live |= (i + u < (uint32_t)T.n && (act != 0) == writes ? 1u : 0u) << u;
            k[u] = (k[u] & ~3u) | (act == 2 ? FILTER_ATOMIC : 0u) | (i + u);
          }
          fn(k, live, 0u);
#pragma unroll
          for (uint32_t q = 0; q + 1 < NV; q++) x[q] = x[q + 1];
        }
      }
      return;
    }
    const uint32_t len = writes ? run / 4 : run - run / 4;  // (a guess: it only sets how many lanes share a run)
    const uint32_t most = 31u - (uint32_t)__builtin_clz(NTH / min(NTH, hi - lo));  // with it every run has a group
    uint32_t lg = len > 16 ? 32u - (uint32_t)__builtin_clz((len - 1) / 16) : 0u;
    lg = min(lg, 10u);
    while (lg < most && ((4u << lg) < len || parts > 1)) lg++;
    const uint32_t step = NTH >> lg;
    uint32_t ml = NV == 1 ? 0u : (len <= 4u << lg ? 2u : (len <= 8u << lg ? 1u : 0u));
    while (ml && hi - lo <= step << (ml - 1)) ml--;
    uint32_t to = threadIdx.x;
    asm volatile("" : "+v"(to));  // (not hoisted over the passes)
    const uint32_t lane = to & ((1u << lg) - 1);
#pragma unroll 1
    for (uint32_t i0 = lo; i0 < hi; i0 += step << ml) {
      uint32_t at[NV];  // the lane's next key | the run's end << 16
      auto tile = [&](uint32_t v) { return i0 + (to >> lg) + ((v << ml) / NV) * step; };
#pragma unroll
      for (uint32_t v = 0; v < NV; v++) {
        if ((v & ((NV >> ml) - 1u)) == 0) {
          at[v] = 0;
          if (tile(v) < hi) {
            const words2 r = load_words2(rows + (uint64_t)tile(v) * (B + 1));
            at[v] = (writes ? r.x : (r.x >> 16) | (r.y << 16)) + 4 * lane;
          }
        } else {
          at[v] = at[v - 1] + (4u << lg);
        }
      }
      bool more;
      do {
        words4 x[NV];
        uint32_t live = 0;
        more = false;
#pragma unroll
        for (uint32_t v = 0; v < NV; v++) {
          const int left = (int)(at[v] >> 16) - (int)(at[v] & 0xFFFFu);
          if (left > 0) {
            x[v] = load_words4(keys + (tile(v) * FT + (at[v] & 0xFFFFu)));  // (may read on past the run, never past the buffer)
            live |= (left >= 4 ? 15u : (1u << left) - 1u) << (4 * v);
          }
          at[v] += left > 0 ? (4 * NV >> ml) << lg : 0u;
          more = more || left > (int)((4 * NV >> ml) << lg);
        }
#pragma unroll 1
        for (uint32_t v = 0; __any(live != 0); v++) {
          const uint32_t k[4] = {x[0].x, x[0].y, x[0].z, x[0].w};
          fn(k, live & 15u, tile(v) * FT);
#pragma unroll
          for (uint32_t q = 0; q + 1 < NV; q++) x[q] = x[q + 1];
          live >>= 4;
        }
      } while (__any(more));
    }
  };
  auto for_keys = [&](bool writes, uint32_t lo, uint32_t hi, auto&& fn) {
    for_keys_n(std::integral_constant<uint32_t, 4>(), writes, lo, hi, fn);
  };
  // ... where fn reads the keys' records: four of those are in flight instead
  auto for_keys_records = [&](bool writes, uint32_t lo, uint32_t hi, auto&& fn) {
    for_keys_n(std::integral_constant<uint32_t, 1>(), writes, lo, hi, fn);
  };
  auto slot_of = [&](uint32_t k) { return (k >> FT_BITS) & smask; };
  // Appends the indices of the keys in `pick` to a list (all lanes together).
  auto append = [&](const uint32_t(&k)[4], uint32_t pick, uint32_t base, uint32_t* list, uint32_t cap,
                    uint32_t* count) {
    if (!__any(pick != 0)) return;
    const uint32_t n = (uint32_t)__popc(pick), inc = wave_incl_scan(n, [](uint32_t a, uint32_t c) { return a + c; });
    const uint32_t all = readlane(inc, 63);
    uint32_t first = 0;
    if (__lane_id() == 0) first = atomicAdd(count, all);
    uint32_t pos = (uint32_t)__builtin_amdgcn_readfirstlane((int)first) + inc - n;
#pragma unroll
    for (uint32_t u = 0; u < 4; u++)
      if ((pick >> u) & 1u) {
        if (pos < cap) list[pos] = base + (k[u] & (FT - 1));
        pos++;
      }
  };

  // ---- W and T, and D from writes that meet another.  (Bits are looked at
  //      before they are set: a hot word's atomics would go one by one.)
  bool any = false;
  auto see_writes = [&](const uint32_t(&k)[4], uint32_t live, uint32_t) {
    any = any || live;
    uint32_t seen = 0;
#pragma unroll
    for (uint32_t u = 0; u < 4; u++)
      if ((live >> u) & 1u) {
        const uint32_t s = slot_of(k[u]);
        seen |= ((k[u] & FILTER_ATOMIC) ? bit(A, s >> 2) : bit(W, s)) << u;
      }
#pragma unroll
    for (uint32_t u = 0; u < 4; u++)
      if (((live & ~seen) >> u) & 1u) {
        const uint32_t s = slot_of(k[u]);
        if (k[u] & FILTER_ATOMIC) set(A, s >> 2);
        else seen |= ((set(W, s) >> (s & 31u)) & 1u) << u;
      }
#pragma unroll
    for (uint32_t u = 0; u < 4; u++)
      if (((live & seen) >> u) & 1u) {
        const uint32_t sd = slot_of(k[u]) >> 1;
        if (!(k[u] & FILTER_ATOMIC) && !bit(D, sd)) set(D, sd);
      }
  };
  if constexpr (DIRECT && !LATE) {  // the records: their keys (slot | action), and the writes among them
    constexpr uint32_t Q = 8;  // records in flight per thread
    const GRecords p = global_records(T.rec);
    const uint32_t shift = block_shift(T.tpb), n = (uint32_t)T.n;
    uint32_t bad = ~0u;
#pragma unroll 1
    for (uint32_t i0 = 0; i0 < n; i0 += Q * NTH) {
      ulonglong2 x[Q];
#pragma unroll
      for (uint32_t u = 0; u < Q; u++) {
        const uint32_t j = i0 + tx + u * NTH;
        x[u] = j < n ? load_record(p, j) : ulonglong2{0ull, 0ull};
      }
#pragma unroll 1
      for (uint32_t h = 0; h < Q && i0 + h * NTH < n; h += 4) {
        uint32_t k[4], live = 0;
#pragma unroll
        for (uint32_t u = 0; u < 4; u++) {
          const uint32_t j = i0 + tx + (h + u) * NTH;
          const Rec r = unpack_rec(x[u]);
          if (j < n && (r.action > 2 || r.space > 1)) bad = min(bad, j);
          const uint32_t act = r.action <= 2 ? r.action : 0u;  // (a bad record's call fails)
          k[u] = filter_slot(filter_group(r.unit, block_of(r.tid, T.tpb, shift), r.epoch, r.space)) << FT_BITS;
          if (j < n) f.keys[T.off + j] = k[u] | act;
          live |= (j < n && act ? 1u : 0u) << u;
          if (act == 2) k[u] |= FILTER_ATOMIC;
        }
        see_writes(k, live, 0u);
#pragma unroll
        for (uint32_t u = 0; u + 4 < Q; u++) x[u] = x[u + 4];
      }
    }
    if (bad != ~0u) {
      atomicOr(&f.ctrl->error_flags, LAYOUT_ERR_RECORD);
      atomicMin((unsigned long long*)&f.ctrl->first_bad, (unsigned long long)(T.off + (uint64_t)bad));
    }
  } else {
    for_keys(true, 0, T.ntiles, see_writes);
  }
  if (any) s_any = 1;
  __syncthreads();
  if (!s_any) return;  // nothing but reads

  // ---- reads in W or T; the first RCAP of them are remembered
  const uint32_t r0 = (uint32_t)((uint64_t)T.ntiles * part / parts), r1 = (uint32_t)((uint64_t)T.ntiles * (part + 1) / parts);
  for_keys(false, r0, r1, [&](const uint32_t(&k)[4], uint32_t live, uint32_t base) {
    uint32_t pick = 0;
#pragma unroll
    for (uint32_t u = 0; u < 4; u++)
      if ((live >> u) & 1u) pick |= (bit(W, slot_of(k[u])) | bit(A, slot_of(k[u]) >> 2)) << u;
#pragma unroll
    for (uint32_t u = 0; u < 4; u++)
      if ((pick >> u) & 1u) {
        const uint32_t sd = slot_of(k[u]) >> 1;
        if (!bit(D, sd)) set(D, sd);
      }
    append(k, pick, base, s_read, RCAP, &s_n);
  });
  __syncthreads();
  const uint32_t n_read = uniform(s_n);
  const GRecords p = global_records(T.rec);
  const uint32_t shift = block_shift(T.tpb);
  auto load_frec = [&](uint32_t idx) {
    const Rec x = unpack_rec(load_record(p, idx));
    return frec(x.unit, x.tid, x.epoch, x.action, x.space);
  };
  auto w_at = [&](uint32_t i) {
    const uint4 v = s_w[i];
    return FRec{v.x, v.y, v.z, v.w};
  };
  // The records of the keys in `pick`: fn(u, record, its index).
  auto for_records = [&](const uint32_t(&k)[4], uint32_t pick, uint32_t base, auto&& fn) {
    constexpr uint32_t IN = LATE ? 4 : 2;  // in flight
#pragma unroll 1
    for (uint32_t h = 0; h < 4; h += IN) {
      FRec x[IN];
      uint32_t at[IN];
#pragma unroll
      for (uint32_t u = 0; u < IN; u++) {
        at[u] = base + ((IN == 4 || h == 0 ? k[u] : k[(2 + u) & 3u]) & (FT - 1));
        if ((pick >> (h + u)) & 1u) x[u] = load_frec(at[u]);
      }
#pragma unroll 1
      for (uint32_t u = 0; u < IN; u++) {  // (one copy of fn)
        if ((pick >> (h + u)) & 1u) fn(h + u, x[0], at[0]);
#pragma unroll
        for (uint32_t q = 0; q + 1 < IN; q++) {
          x[q] = x[q + 1];
          at[q] = at[q + 1];
        }
      }
    }
  };

  // ---- the writes and atomics that are left: all of them, listed
  uint32_t rounds = 1;
  auto list_writes = [&](bool first, uint32_t round) {  // (the first time W and T tell them, then D alone)
    for_keys(true, 0, T.ntiles, [&](const uint32_t(&k)[4], uint32_t live, uint32_t base) {
      uint32_t pick = 0;
#pragma unroll
      for (uint32_t u = 0; u < 4; u++)
        if ((live >> u) & 1u) {
          const uint32_t s = slot_of(k[u]);
          uint32_t in_d = bit(D, s >> 1);
          if (first) {
            const uint32_t other = (k[u] & FILTER_ATOMIC) ? bit(W, s) : bit(A, s >> 2);
            if (other && !in_d) set(D, s >> 1);
            in_d |= other;
          }
          pick |= ((s & (rounds - 1)) == round ? in_d : 0u) << u;
        }
      append(k, pick, base, s_blk, WCAP, &s_nw);
      if (LOOP && !first && rounds == 1) {  // (by the low bits of the slot, for tables of them)
#pragma unroll
        for (uint32_t u = 0; u < 4; u++)
          if ((pick >> u) & 1u) atomicAdd(&s_cls[0][slot_of(k[u]) & 3u], 1u);
      }
    });
    __syncthreads();
    return uniform(s_nw);
  };
  auto to_late = [&]() {  // by one thread
    const uint32_t at = atomicAdd(&f.cnt[FC_LATE], 1u);
    if (at < f.late_max) f.late[at] = make_uint2(DIRECT ? trace : bucket, part);
    else atomicOr(&f.ctrl->error_flags, ERR_GROUP_FULL);
  };
  auto full = [&]() {
    if (tx == 0) atomicOr(&f.ctrl->error_flags, ERR_GROUP_FULL);
  };
  // a later workgroup's (but the sort's, where some of the bucket's entries are out)
  auto give_up = [&](uint32_t round) {
    if (round) return full();
    if (threadIdx.x == 0) to_late();
  };
  // the reads' pairs, summed per thread while the location stays the same (the
  // lanes' LDS atomics to a hot word's sums go one by one)
  uint32_t lead = 0, rw = 0, ar = 0, xb = 0;
  auto flush = [&]() {
    if (rw) atomicAdd(&s_acc[K_RW][lead], rw);
    if (ar) atomicAdd(&s_acc[K_AR][lead], ar);
    if (xb) atomicAdd(&s_acc[K_XB][lead], xb);
    rw = ar = xb = 0;
  };
  auto flush_wave = [&]() {
    const uint64_t has = __ballot((rw | ar) != 0);
    if (!has) return;
    const uint32_t l = readlane(lead, (int)__builtin_ctzll(has));
    if (__all((rw | ar) == 0 || lead == l)) {  // one location: one lane adds for the wave
      auto add = [](uint32_t a, uint32_t c) { return a + c; };
      rw = wave_reduce(rw, 0u, add);
      ar = wave_reduce(ar, 0u, add);
      xb = wave_reduce(xb, 0u, add);
      lead = l;
      if (__lane_id() == 0) flush();
      rw = ar = xb = 0;
    } else {
      flush();
    }
  };
  // an entry per location with pairs (all threads; the sums are complete, s_n is 0)
  auto paired = [&](uint32_t i) { return (s_acc[K_WW][i] | s_acc[K_RW][i] | s_acc[K_AW][i] | s_acc[K_AR][i]) != 0; };
  auto emit = [&](uint32_t nw) {
    const uint32_t i = threadIdx.x;
    const bool racing = i < nw && s_lead[i] == i && paired(i);
    const uint64_t mask = __ballot(racing);
    uint32_t pos = 0;
    if (mask) {
      if (__lane_id() == 0) pos = atomicAdd(&s_n, (uint32_t)__popcll(mask));
      pos = (uint32_t)__builtin_amdgcn_readfirstlane((int)pos) + __builtin_amdgcn_mbcnt_hi((uint32_t)(mask >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)mask, 0u));
    }
    __syncthreads();
    const uint32_t n_new = s_n;
    if (!n_new) return;
    if (i == 0) {
      s_base = atomicAdd(&f.cnt[FC_ENTRIES], n_new);
      if (s_base + n_new > f.entries_cap) atomicOr(&f.ctrl->error_flags, ERR_GROUP_FULL);
      const uint32_t in_trace = atomicAdd(&f.trace_cnt[trace], n_new) + n_new;
      if (in_trace > SORT_ALONE) atomicMax(&f.cnt[FC_MOST], in_trace);
      if (in_trace > GROUP_MAX_ENTRIES) atomicOr(&f.ctrl->error_flags, ERR_GROUP_FULL);
    }
    __syncthreads();
    if (racing && s_base + n_new <= f.entries_cap) {
      const FRec x = w_at(i);
      RaceOut e;
      e.trace = trace;
      e.space = (uint8_t)frec_space(x);
      e.kinds = (uint8_t)((s_acc[K_WW][i] ? 1 : 0) | (s_acc[K_RW][i] ? 2 : 0) | (s_acc[K_AW][i] ? 4 : 0) |
                          (s_acc[K_AR][i] ? 8 : 0) | (s_acc[K_XB][i] ? 16 : 0));
      e.reserved16 = 0;
      e.block = frec_space(x) ? block_of(x.tid, T.tpb, shift) : 0xFFFFFFFFu;
      e.reserved32 = 0;
      e.unit = ((uint64_t)x.uhi << 32) | x.ulo;
      e.ww = s_acc[K_WW][i];
      e.rw = s_acc[K_RW][i];
      e.aw = s_acc[K_AW][i];
      e.ar = s_acc[K_AR][i];
      e.xb = s_acc[K_XB][i];
      f.entries[s_base + pos] = e;
    }
  };
  // keys of D that are a round's
  auto in_round = [&](const uint32_t(&k)[4], uint32_t live, uint32_t round) {
    uint32_t pick = 0;
#pragma unroll
    for (uint32_t u = 0; u < 4; u++)
      if ((live >> u) & 1u) {
        const uint32_t s = slot_of(k[u]);
        pick |= (!LATE || (s & (rounds - 1)) == round ? bit(D, s >> 1) : 0u) << u;
      }
    return pick;
  };
  if constexpr (!LATE) {
    uint32_t round = 0;
#pragma unroll 1
    for (bool first = true;; first = false) {
      uint32_t tx = threadIdx.x;
      if (LOOP) asm volatile("" : "+v"(tx));  // keeps per-thread addresses out of registers across the passes
      const uint32_t nw = list_writes(first, round);
      if (nw > WCAP) {  // more than the table holds
        if (LOOP && rounds > 1) return give_up(round);
        if (nw > 4 * WCAP) {
          // by a sample, more writes than a late workgroup may take either
          const uint32_t plain = (uint32_t)__syncthreads_count(tx < WCAP && frec_action(load_frec(s_blk[min(tx, WCAP - 1)])) == 1u);
          if ((uint64_t)nw * plain > (uint64_t)hopeless(f.max_rounds) * WCAP) return full();
          return give_up(0);
        }
        if (tx == 0 && first) atomicAdd(&f.cnt[FC_ROUNDS], 1u);
        if (!LOOP) return give_up(0);
        // First once more, as D grew while they were listed, and counted by the low
        // bits of their slots; then in two or four tables that hold them.
        if (!first) {
          const uint32_t c0 = s_cls[0][0], c1 = s_cls[0][1], c2 = s_cls[0][2], c3 = s_cls[0][3];
          if (max(max(c0, c1), max(c2, c3)) > WCAP) return give_up(0);
          rounds = uniform(max(c0 + c2, c1 + c3) > WCAP ? 4u : 2u);
        }
        __syncthreads();
        if (tx == 0) s_nw = 0;
        __syncthreads();
        continue;
      }
      if (!LOOP && !nw) return;
      if (!pair_sums_fit(n_read, nw)) return full();  // sums of pairs are kept in 32 bits
      uint32_t* const head = W;  // chains of writes, and as many of atomics (W is free)
      // the latter's lengths, and which bits of a location's tag are set (low half)
      // or clear (high half) in some record of theirs: most reads that meet a hot
      // word's long chain by chance need not walk it
      uint32_t* const length = head + 2 * HN;
      uint32_t* const tags = head + 3 * HN;
      for (uint32_t k = tx; k < 4 * HN; k += NTH) head[k] = k < 2 * HN ? END : 0u;
      const uint32_t longest = n_read > RCAP ? MANY_WRITERS : CHAIN;
      __syncthreads();
      auto chain_of = [&](const FRec& x, uint32_t bx) { return location_hash(x, bx) & (HN - 1); };
      auto tag_of = [](uint32_t h) {  // (one bucket's hashes have their high bits in common)
        h *= 0x9E3779B1u;
        return h >> 16 | (~h & 0xFFFF0000u);
      };
      if (tx < nw) {
        const uint32_t i = tx, idx = s_blk[i];
        const FRec x = load_frec(idx);
        const uint32_t bx = block_of(x.tid, T.tpb, shift);
        if (WARP) s_side[i] = f.side[T.off + idx];
        s_w[i] = make_uint4(x.ulo, x.uhi, x.tid, x.meta);
        s_blk[i] = bx;
        const uint32_t h = location_hash(x, bx), c = h & (HN - 1), atomic = frec_action(x) == 2u;
        s_next[i] = (uint16_t)atomicExch(&head[c + (atomic ? HN : 0u)], i);
        if (atomic && n_read) {
          atomicAdd(&length[c], 1u);
          atomicOr(&tags[c], tag_of(h));
        }
#pragma unroll
        for (int q = 0; q < 5; q++) s_acc[q][i] = 0;
      }
      __syncthreads();
      // ---- a location's first write in the table (without one its first atomic),
      //      and the pairs of writes.  (A hot word's atomics meet no other atomic:
      //      where their chain is long, only reads of it would tell them apart, and
      //      those are for another path.)
      if (tx < nw) {
        const uint32_t i = tx;
        const FRec x = w_at(i);
        const uint32_t bx = s_blk[i], sx = WARP ? s_side[i] : 0u;
        const bool atomic = frec_action(x) == 2u;
        uint32_t first = i, ww = 0, aw = 0, xw = 0, left = longest;
#pragma unroll 1
        for (uint32_t j = head[chain_of(x, bx)]; j != END && left; j = s_next[j], left--) {
          if (!atomic && j >= i) continue;
          const FRec y = w_at(j);
          const uint32_t by = s_blk[j];
          if (!same_location(x, bx, y, by)) continue;
          first = first == i ? j : min(first, j);
          if (part == 0 && pair_races(x, bx, y, by, WARP, T.tpb, sx, WARP ? s_side[j] : 0u)) {
            if (atomic) aw++;
            else ww++;
            if (bx != by) xw++;
          }
        }
        if (atomic && n_read && first == i && length[chain_of(x, bx)] <= longest) {
#pragma unroll 1
          for (uint32_t j = head[chain_of(x, bx) + HN]; j != END; j = s_next[j])
            if (j < first && same_location(x, bx, w_at(j), s_blk[j])) first = j;
        }
        s_lead[i] = (uint16_t)first;
        if (!left) s_any = 2;
        if (ww) atomicAdd(&s_acc[K_WW][first], ww);
        if (aw) atomicAdd(&s_acc[K_AW][first], aw);
        if (xw) atomicAdd(&s_acc[K_XB][first], xw);
      }
      __syncthreads();
      if (s_any == 2) {  // long chains
        return give_up(round);
      }
      auto count_read = [&](const FRec& x, uint32_t idx) {
        const uint32_t bx = block_of(x.tid, T.tpb, shift);
        const uint32_t h = location_hash(x, bx), c = h & (HN - 1);
        uint32_t j = head[c], k = head[c + HN];
        if (k != END) {
          if (tag_of(h) & ~tags[c]) {  // none of its location
            k = END;
          } else if (length[c] > longest) {
            s_any = 2;
            return;
          }
        }
        if (j == END) {
          j = k;
          k = END;
        }
        if (j == END) return;
        const uint32_t sx = WARP ? f.side[T.off + idx] : 0u;
#pragma unroll 1
        for (uint32_t left = 2 * CHAIN; j != END && left; left--) {  // (or another path counts the bucket, see above)
          const uint32_t at = j;
          j = s_next[j];
          if (j == END) {  // the writes, then the atomics
            j = k;
            k = END;
          }
          const FRec y = w_at(at);
          const uint32_t by = s_blk[at];
          if (!same_location(x, bx, y, by) || !pair_races(x, bx, y, by, WARP, T.tpb, sx, WARP ? s_side[at] : 0u)) continue;
          const uint32_t l = s_lead[at];
          if (l != lead) flush();
          lead = l;
          if (frec_action(y) == 1u) rw++;
          else ar++;
          if (bx != by) xb++;
        }
      };
      if (n_read <= RCAP) {
#pragma unroll 1
        for (uint32_t i = tx; i < n_read; i += NTH) count_read(load_frec(s_read[i]), s_read[i]);
      } else if (n_read) {
        for_keys_records(false, r0, r1, [&](const uint32_t(&k)[4], uint32_t live, uint32_t base) {
          for_records(k, in_round(k, live, round), base, [&](uint32_t, const FRec& x, uint32_t idx) { count_read(x, idx); });
        });
      }
      flush_wave();
      if (tx == 0) s_n = 0;
      __syncthreads();
      if (s_any == 2) {  // reads of a word of many atomics
        return give_up(round);
      }
      emit(nw);
      if (!LOOP || ++round == rounds) return;
      __syncthreads();
      if (tx == 0) s_nw = 0;
      __syncthreads();
    }
  } else {
    const uint32_t n_left = list_writes(true, 0);
    bool thinned = false;
    static_assert(CLASSES == 64, "a lane per class");
    // a record's place in map m, and whether all of them hold it
    auto place = [&](const FRec& x, uint32_t bx, uint32_t m) { return filter_group2(x, bx, m) >> (32 - L_BITS); };
    auto kept = [&](const FRec& x) {
      const uint32_t bx = block_of(x.tid, T.tpb, shift);
      uint32_t all = 1;
      for (uint32_t m = 0; m < MAPS; m++) all &= bit(W + m * L_WORDS, place(x, bx, m));
      return all != 0;
    };
    auto atomics = [](const uint32_t(&k)[4]) {
      return k[0] >> 31 | k[1] >> 31 << 1 | k[2] >> 31 << 2 | k[3] >> 31 << 3;
    };
    auto keep_of = [&](const uint32_t(&k)[4], uint32_t pick, uint32_t base) {
      if (!thinned) return pick;
      uint32_t left = pick & ~atomics(k);
      for_records(k, pick & ~left, base, [&](uint32_t u, const FRec& x, uint32_t) { left |= kept(x) ? 1u << u : 0u; });
      return left;
    };
    const uint32_t most = f.max_rounds;
    bool listed = n_left <= WCAP;  // the list holds the candidates
    while (!listed) {
      uint32_t fit = 2 * CLASSES, fit_writes = 1;
      if (thinned || n_left <= most * WCAP) {  // the candidates that are left, listed and by class
        __syncthreads();
        if (tx < 2 * CLASSES) s_cls[tx / CLASSES][tx % CLASSES] = 0;
        if (tx == 0) s_nw = 0;
        __syncthreads();
        // (after a look at a sixteenth of the tiles: where that is too much
        // already, the rest need not be read)
        for (uint32_t lo = 0, hi = T.ntiles >= 32 ? T.ntiles / 16 : T.ntiles; lo < T.ntiles; lo = hi, hi = T.ntiles) {
          for_keys(true, lo, hi, [&](const uint32_t(&k)[4], uint32_t live, uint32_t base) {
            const uint32_t pick = keep_of(k, in_round(k, live, 0), base);
            append(k, pick, base, s_blk, WCAP, &s_nw);
#pragma unroll
            for (uint32_t u = 0; u < 4; u++)
              if ((pick >> u) & 1u) {
                const uint32_t c = slot_of(k[u]) & (CLASSES - 1);
                atomicAdd(&s_cls[0][c], 1u);
                if (!(k[u] & FILTER_ATOMIC)) atomicAdd(&s_cls[1][c], 1u);
              }
          });
          __syncthreads();
          // the fewest rounds that each fit: lane r adds up the classes of round r
          if (tx < 2 * CLASSES) {
            uint32_t sum = s_cls[tx / CLASSES][tx % CLASSES], r = CLASSES;
            if (__any(sum > WCAP)) r = 2 * CLASSES;
            while (r <= CLASSES && r > 1) {
              sum += __shfl_xor(sum, (int)(r / 2));
              if (__any(sum > WCAP)) break;
              r /= 2;
            }
            if (tx == 0) s_base = r;
            if (tx == CLASSES) s_n = r;
          }
          __syncthreads();
          fit = uniform(s_base);
          fit_writes = uniform(s_n);
          if (fit > most) break;
        }
        if (fit <= most) {
          rounds = fit;
          listed = uniform(s_nw) <= WCAP;
          break;
        }
      }
      if (fit_writes > most || thinned) return full();  // too many writes, or atomics that do meet one or a read
      // ---- the maps: where the writes and the reads are that an atomic may meet
      __syncthreads();
      for (uint32_t i = tx; i < MAPS * L_WORDS; i += NTH) W[i] = 0;
      __syncthreads();
      auto add = [&](const FRec& x) {
        const uint32_t bx = block_of(x.tid, T.tpb, shift);
        for (uint32_t m = 0; m < MAPS; m++) {
          const uint32_t s = place(x, bx, m);
          if (!bit(W + m * L_WORDS, s)) set(W + m * L_WORDS, s);
        }
      };
      for_keys(true, 0, T.ntiles, [&](const uint32_t(&k)[4], uint32_t live, uint32_t base) {
        for_records(k, in_round(k, live & ~atomics(k), 0), base, [&](uint32_t, const FRec& x, uint32_t) { add(x); });
      });
      if (n_read <= RCAP) {
        for (uint32_t i = tx; i < n_read; i += NTH) add(load_frec(s_read[i]));
      } else {
        for_keys_records(false, r0, r1, [&](const uint32_t(&k)[4], uint32_t live, uint32_t base) {
          for_records(k, in_round(k, live, 0), base, [&](uint32_t, const FRec& x, uint32_t) { add(x); });
        });
      }
      __syncthreads();
      thinned = true;
    }
#pragma unroll 1
    for (uint32_t round = 0; round < rounds; round++) {
      uint32_t tx = threadIdx.x;
      asm volatile("" : "+v"(tx));  // keeps per-thread addresses out of registers across the passes
      if (!listed) {                // this round's
        __syncthreads();
        if (tx == 0) s_nw = 0;
        __syncthreads();
        for_keys(true, 0, T.ntiles, [&](const uint32_t(&k)[4], uint32_t live, uint32_t base) {
          append(k, keep_of(k, in_round(k, live, round), base), base, s_blk, WCAP, &s_nw);
        });
      }
      for (uint32_t k = 4 * tx; k < HT; k += 4 * NTH) *(uint4*)(tab + k) = make_uint4(NONE, NONE, NONE, NONE);
      __syncthreads();
      const uint32_t nw = uniform(s_nw);  // (at most WCAP)
      if (!pair_sums_fit(n_read, nw)) return full();  // sums of pairs are kept in 32 bits
      if (!nw) continue;
      // Table entries of x's location (l0: its first record, or NONE) and of its
      // groups there: their first records.  Inside a location its first record
      // stands for it, in hashes and comparisons.
      auto is_group = [&](uint32_t level, uint32_t e, uint32_t l0, const FRec& x, uint32_t bx) {
        if (e >> 16 != level) return false;
        const uint32_t j = e & 0xFFFFu;
        if (level == 0) return same_location(w_at(j), s_blk[j], x, bx);
        if (s_lead[j] != l0 || s_blk[j] != bx) return false;
        if (level == 1) return true;
        const FRec y = w_at(j);
        if (((y.meta ^ x.meta) & 0xFFFFu) != 0) return false;
        return level == 2 || (level == 3 ? y.tid == x.tid : warp_of(y, bx, T.tpb) == warp_of(x, bx, T.tpb));
      };
      // (The high bits of a location's hash are those of its bucket, so the low ones
      // place it; a group's high ones.)
      static_assert(HT == 1u << 13, "places from a hash's high bits");
      auto place_of = [](uint32_t level, uint32_t h) { return level ? h >> (32 - 13) : h & (HT - 1); };
      auto find = [&](uint32_t level, uint32_t h, uint32_t l0, const FRec& x, uint32_t bx) {
        for (uint32_t at = place_of(level, h);; at = (at + 1) & (HT - 1)) {
          const uint32_t e = tab[at];
          if (e == NONE) return NONE;
          if (is_group(level, e, l0, x, bx)) return e & 0xFFFFu;
        }
      };
      // ... made record i's where there is none yet.  (A place is taken by one
      // compare-and-swap, and nobody waits: the records were stored before.)
      auto find_or_add = [&](uint32_t level, uint32_t h, uint32_t l0, const FRec& x, uint32_t bx, uint32_t i) {
        for (uint32_t at = place_of(level, h);; at = (at + 1) & (HT - 1)) {
          uint32_t e = __hip_atomic_load(&tab[at], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
          if (e == NONE) e = atomicCAS(&tab[at], NONE, level << 16 | i);
          if (e == NONE) return i;
          if (is_group(level, e, l0, x, bx)) return e & 0xFFFFu;
        }
      };
      auto level_hash = [&](uint32_t level, uint32_t l0, const FRec& x, uint32_t bx) {
        uint32_t h = groups_hash(l0);
        for (uint32_t l = 1; l <= level; l++)
          if (l != 3 || level == 3) h = group_hash(l, h, x, bx, T.tpb);
        return h;
      };
      auto several = [](uint32_t c) { return c != 1u && c != 0x10000u; };
      if (tx < nw) {
        const uint32_t idx = s_blk[tx];
        const FRec x = load_frec(idx);
        if (WARP) {
          s_side[WARP ? tx : 0] = f.side[T.off + idx];
          s_whead[WARP ? tx : 0] = NONE;
        }
        s_w[tx] = make_uint4(x.ulo, x.uhi, x.tid, x.meta);
        s_blk[tx] = block_of(x.tid, T.tpb, shift);
#pragma unroll
        for (uint32_t l = 0; l < LEVELS; l++) s_cnt[l][tx] = 0;
#pragma unroll
        for (int q = 0; q < 5; q++) s_acc[q][tx] = 0;
      }
      __syncthreads();
      if (tx < nw) {  // by location
        const FRec x = w_at(tx);
        const uint32_t bx = s_blk[tx], lead = find_or_add(0, location_hash(x, bx), 0u, x, bx, tx);
        s_lead[tx] = (uint16_t)lead;
        atomicAdd(&s_cnt[0][lead], group_one(x));
      }
      __syncthreads();
#pragma unroll 1
      for (uint32_t q = tx; q < (LEVELS - 1) * nw; q += NTH) {  // ... and, where it has several, by block, epoch and thread
        uint32_t l = 1, i = q;
        for (; i >= nw; l++) i -= nw;
        if (!several(s_cnt[0][s_lead[i]]) || (l == GROUP_WARP && (s_side[WARP ? i : 0] & SIDE_DIVERGED))) continue;
        const FRec x = w_at(i);
        const uint32_t bx = s_blk[i], l0 = s_lead[i];
        const uint32_t g = find_or_add(l, level_hash(l, l0, x, bx), l0, x, bx, i), before = atomicAdd(&s_cnt[l][g], group_one(x));
        if (WARP && l == GROUP_WARP) {
          s_next[i] = (uint16_t)atomicExch(&s_whead[WARP ? g : 0], i);
          if ((before & 0xFFFFu) + (before >> 16) >= WARP_WALK) s_any = 2;
        }
      }
      __syncthreads();
      if (WARP && s_any == 2) {  // a warp's records of one word are walked one by one: many of them are for the sort
        full();
        return;
      }
      // fn(an undiverged record of x's warp, epoch and word by another thread)
      auto for_warp = [&](uint32_t l0, const FRec& x, uint32_t bx, auto&& fn) {
        if constexpr (WARP) {
          const uint32_t g = find(GROUP_WARP, level_hash(GROUP_WARP, l0, x, bx), l0, x, bx);
          if (g == NONE) return;
#pragma unroll 1
          for (uint32_t j = s_whead[g] & END; j != END; j = s_next[j])
            if (s_w[j].z != x.tid) fn(j);
        }
      };
      if (part == 0 && tx < nw) {  // the pairs of writes and atomics
        const uint32_t lead = s_lead[tx];
        if (several(s_cnt[0][lead])) {
          uint32_t ww = 0, aw = 0, xb = 0;
#pragma unroll
          for (uint32_t l = 0; l < GROUP_LEVELS; l++) {  // (no record: the group's first one is another)
            const uint32_t c = s_cnt[l][tx], pw = c ? pairs_ww(c) : 0u, pa = pairs_aw(c);
            ww += (l & 1) ? 0u - pw : pw;
            aw += (l & 1) ? 0u - pa : pa;
            if (l < 2) xb += (l & 1) ? 0u - pw - pa : pw + pa;
          }
          if (WARP && !(s_side[WARP ? tx : 0] & SIDE_DIVERGED)) {
            const FRec x = w_at(tx);
            const uint32_t bx = s_blk[tx];
            for_warp(lead, x, bx, [&](uint32_t j) {  // ordered by lockstep, but two writes of one statement
              if (j >= tx) return;
              const FRec y = w_at(j);
              if (pair_races(x, bx, y, bx, true, T.tpb, s_side[WARP ? tx : 0], s_side[WARP ? j : 0])) return;
              if (frec_action(x) == 1u && frec_action(y) == 1u) ww--;
              else if (frec_action(x) != frec_action(y)) aw--;
            });
          }
          if (ww) atomicAdd(&s_acc[K_WW][lead], ww);
          if (aw) atomicAdd(&s_acc[K_AW][lead], aw);
          if (xb) atomicAdd(&s_acc[K_XB][lead], xb);
        }
      }
      uint32_t last = NONE;  // (a hot word's reads come one after another)
      auto count_read = [&](const FRec& x, uint32_t idx) {
        const uint32_t bx = block_of(x.tid, T.tpb, shift);
        uint32_t l0 = last;
        if (l0 == NONE || !same_location(w_at(l0), s_blk[l0], x, bx)) {
          l0 = find(0, location_hash(x, bx), 0u, x, bx);
          if (l0 == NONE) return;
          last = l0;
        }
        uint32_t left = s_cnt[0][l0], cross = left;
        if (!several(left)) {  // one record: the pair itself
          const uint32_t by = s_blk[l0];
          if (!pair_races(x, bx, w_at(l0), by, WARP, T.tpb, WARP ? f.side[T.off + idx] : 0u, WARP ? s_side[l0] : 0u)) return;
          if (bx == by) cross = 0;
        } else {
          uint32_t h = groups_hash(l0);
#pragma unroll 1
          for (uint32_t l = 1; l < GROUP_LEVELS; l++) {
            h = group_hash(l, h, x, bx, T.tpb);
            const uint32_t g = find(l, h, l0, x, bx);
            if (g == NONE) break;
            const uint32_t c = s_cnt[l][g];
            left += (l & 1) ? 0u - c : c;
            if (l == 1) cross = left;
            if (WARP && l == 2 && !(f.side[T.off + idx] & SIDE_DIVERGED))
              for_warp(l0, x, bx, [&](uint32_t j) { left -= group_one(w_at(j)); });
          }
        }
        if (!left) return;
        if (l0 != lead) flush();
        lead = l0;
        rw += left & 0xFFFFu;
        ar += left >> 16;
        xb += (cross & 0xFFFFu) + (cross >> 16);
      };
      if (n_read <= RCAP) {  // (in rounds, those of other slots meet no write here)
#pragma unroll 1
        for (uint32_t i = tx; i < n_read; i += NTH) count_read(load_frec(s_read[i]), s_read[i]);
      } else if (n_read) {
        for_keys_records(false, r0, r1, [&](const uint32_t(&k)[4], uint32_t live, uint32_t base) {
          for_records(k, in_round(k, live, round), base, [&](uint32_t, const FRec& x, uint32_t idx) { count_read(x, idx); });
        });
      }
      flush_wave();
      lead = 0;
      if (tx == 0) s_n = 0;
      __syncthreads();
      emit(nw);
    }
  }
}

// ------------------------------------------------------- entries in order
// The buckets' entries come in any order.  k_entries_place moves them to
// their trace's range; k_entries_sort sorts a trace's, SORT_CHUNK at a time;
// k_entries_merge puts the chunks of a trace with more together.
// Entries of one location end up next to each other.  A few entries go straight
// to the host's memory, with the counts, so that such a call downloads nothing.

struct EntryKey {
  uint64_t place;  // space, block
  uint64_t unit;
};
__device__ __forceinline__ EntryKey entry_key(const RaceOut& e) {
  return EntryKey{((uint64_t)e.space << 32) | e.block, e.unit};
}
__device__ __forceinline__ bool key_less(const EntryKey& a, const EntryKey& b) {
  return a.place < b.place || (a.place == b.place && a.unit < b.unit);
}
__device__ __forceinline__ void copy_entry(RaceOut* dst, const RaceOut* src) {
#pragma unroll
  for (int q = 0; q < 4; q++) ((ulonglong2*)dst)[q] = ((const ulonglong2*)src)[q];
}

__global__ __launch_bounds__(NT) void k_entries_place(FilterBuffers f) {
  __shared__ uint32_t s_first[GROUP_MAX_TRACES];
  __shared__ uint32_t s_scan[NWAVE];
  const uint32_t n = f.cnt[FC_ENTRIES], tx = threadIdx.x;
  if (f.ctrl->error_flags || (f.late_wait && f.cnt[FC_LATE])) return;
  const uint32_t per = (f.n_traces + NT - 1) / NT, t0 = min(f.n_traces, tx * per), t1 = min(f.n_traces, t0 + per);
  uint32_t sum = 0;
#pragma unroll 4
  for (uint32_t t = t0; t < t1; t++) {
    s_first[t] = f.trace_cnt[t];
    sum += s_first[t];
  }
  uint32_t tot;
  uint32_t base = block_excl_sum(sum, s_scan, &tot);
  for (uint32_t t = t0; t < t1; t++) {
    const uint32_t c = s_first[t];
    s_first[t] = base;
    if (blockIdx.x == 0) f.trace_first[t] = base;
    base += c;
  }
  __syncthreads();
  // (Entries of one trace tend to lie together: where a wave has many, a lane adds
  // for all of them, as atomics to one address take about 11 ns each: 60000
  // entries of one of two traces took 700 us one by one.)
  for (uint32_t i0 = blockIdx.x * NT; i0 < n; i0 += gridDim.x * NT) {
    const uint32_t i = i0 + tx;
    bool todo = i < n;
    const uint32_t t = todo ? f.entries[i].trace : 0u;
    uint32_t at = 0;
#pragma unroll 1
    for (uint32_t k = 0; k < 4; k++) {
      const uint64_t left = __ballot(todo);
      if (!left) break;
      const uint32_t first = (uint32_t)__builtin_ctzll(left), lt = readlane(t, (int)first);
      const uint64_t same = __ballot(todo && t == lt);
      if (__popcll(same) < 16) break;
      uint32_t base = 0;
      if (__lane_id() == first) base = atomicAdd(&f.trace_fill[lt], (uint32_t)__popcll(same));
      base = readlane(base, (int)first);
      if (todo && t == lt) {
        at = base + __builtin_amdgcn_mbcnt_hi((uint32_t)(same >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)same, 0u));
        todo = false;
      }
    }
    if (todo) at = atomicAdd(&f.trace_fill[t], 1u);
    if (i < n) copy_entry(f.placed + s_first[t] + at, f.entries + i);
  }
}

// An entry's place in its chunk is the number of entries before it there (of
// equal ones, those with a smaller index).  A workgroup holds a chunk's keys in
// LDS and places 16 of its entries, sixteen lanes to an entry (256, a lane each,
// where there are many): sorting 1677 entries in one
// workgroup's LDS took 68 us, 66 steps with a barrier each; this takes 17.
// Traces of one chunk (of SORT_ALONE entries, in a call of many traces) belong to the
// workgroups (trace, y); longer ones are shared out among all.  With one workgroup
// per trace, a call of 65 traces with 60000 entries in one of them took 52.7 ms, 0.5
// so (the sort 0.6); with 2048 entries in one of them, 1750 us and 140 (the sort 270).
__global__ __launch_bounds__(NT) void k_entries_sort(FilterBuffers f) {
  __shared__ uint64_t s_place[SORT_CHUNK], s_unit[SORT_CHUNK];
  __shared__ uint32_t s_long[NT], s_n;
  const uint32_t tx = threadIdx.x;
  const uint32_t total = f.cnt[FC_ENTRIES], err = f.ctrl->error_flags, late = f.cnt[FC_LATE], most = f.cnt[FC_MOST];
  const uint32_t own = blockIdx.x < f.n_traces ? f.trace_cnt[blockIdx.x] : 0u;
  if (blockIdx.x == 0 && blockIdx.y == 0 && tx == 0) {
    GroupHead h;
    h.entries = total;
    h.error_flags = err;
    h.late = late;
    h.rounds = f.cnt[FC_ROUNDS];
    h.first_bad = f.ctrl->first_bad;
    *f.head = h;
  }
  if (err || (f.late_wait && late)) return;
  const uint32_t all = gridDim.x * gridDim.y, me = blockIdx.y * gridDim.x + blockIdx.x;
  const uint32_t alone = gridDim.y > 1 ? SORT_CHUNK : SORT_ALONE;
  auto sort = [&](uint32_t t, uint32_t n, uint32_t from, uint32_t step) {
    if (!n) return;
    const uint32_t first = f.n_traces > 1 ? f.trace_first[t] : 0u;
    const RaceOut* src = (f.n_traces > 1 ? f.placed : f.entries) + first;
    RaceOut* dst = (n <= SORT_CHUNK ? (total <= f.host_cap ? f.host_entries : f.sorted)
                                    : (f.n_traces > 1 ? f.entries : f.placed)) + first;
    EntryKey* const mk = n > SORT_CHUNK ? (EntryKey*)f.merge_keys + first : nullptr;  // for the merge
    const uint32_t lanes = (gridDim.y > 1 ? n <= 32 * SORT_CHUNK : n > SORT_ALONE && total <= 64 * all) ? 16u : 1u, take = NT / lanes, per_chunk = SORT_CHUNK / take;
    for (uint32_t item = from;; item += step) {
      const uint32_t c0 = item / per_chunk * SORT_CHUNK, g0 = item % per_chunk * take;
      if (c0 >= n) break;
      const uint32_t m = min(SORT_CHUNK, n - c0);
      if (g0 >= m) continue;
      __syncthreads();
      for (uint32_t i0 = 0; i0 < m; i0 += 4 * NT) {
        EntryKey k[4];
#pragma unroll
        for (uint32_t u = 0; u < 4; u++)
          if (i0 + u * NT + tx < m) k[u] = entry_key(src[c0 + i0 + u * NT + tx]);
#pragma unroll
        for (uint32_t u = 0; u < 4; u++)
          if (i0 + u * NT + tx < m) {
            s_place[i0 + u * NT + tx] = k[u].place;
            s_unit[i0 + u * NT + tx] = k[u].unit;
          }
      }
      __syncthreads();
      const uint32_t e = g0 + tx / lanes, q = tx & (lanes - 1);
      uint32_t rank = 0;
      if (e < m) {
        const EntryKey k{s_place[e], s_unit[e]};
#pragma unroll 8
        for (uint32_t j = q; j < m; j += lanes) {
          const EntryKey o{s_place[j], s_unit[j]};
          rank += key_less(o, k) || (j < e && !key_less(k, o)) ? 1u : 0u;
        }
      }
      if (lanes == 16) {
        rank += __shfl_xor(rank, 1);
        rank += __shfl_xor(rank, 2);
        rank += __shfl_xor(rank, 4);
        rank += __shfl_xor(rank, 8);
        if (e < m && q < 4) ((ulonglong2*)(dst + c0 + rank))[q] = ((const ulonglong2*)(src + c0 + e))[q];
      } else if (e < m) {
        copy_entry(dst + c0 + rank, src + c0 + e);
      }
      if (mk && e < m && q == 0) mk[c0 + rank] = EntryKey{s_place[e], s_unit[e]};
    }
  };
  if (own <= alone) sort(blockIdx.x, own, blockIdx.y, gridDim.y);
  if (most <= alone) return;
  for (uint32_t t0 = 0; t0 < f.n_traces; t0 += NT) {
    __syncthreads();
    if (tx == 0) s_n = 0;
    __syncthreads();
    if (t0 + tx < f.n_traces && f.trace_cnt[t0 + tx] > alone) s_long[atomicAdd(&s_n, 1u)] = t0 + tx;
    __syncthreads();
    const uint32_t n_long = s_n;
    for (uint32_t k = 0; k < n_long; k++) {
      const uint32_t t = s_long[k];
      sort(t, f.trace_cnt[t], (me + t * 61u) % all, all);
    }
  }
}

// An entry's place among its trace's: its index in its chunk and, by binary
// search, the entries of the other chunks before it (equal ones of earlier
// chunks come first).  Bound by the chain of a search's loads, so four searches
// run at once, over keys of 16 bytes: 209713 entries took 520 us one after
// another over the entries themselves, 268 so.  It grows with the square of a
// trace's entries, hence GROUP_MAX_ENTRIES.
__global__ __launch_bounds__(NT) void k_entries_merge(FilterBuffers f) {
  if (f.ctrl->error_flags || (f.late_wait && f.cnt[FC_LATE]) || f.cnt[FC_MOST] <= SORT_CHUNK) return;
  const uint32_t total = f.cnt[FC_ENTRIES];
  const RaceOut* const all = f.n_traces > 1 ? f.entries : f.placed;
  for (uint32_t i = blockIdx.x * NT + threadIdx.x; i < total; i += gridDim.x * NT) {
    uint32_t t = 0;
    if (f.n_traces > 1) {  // the trace whose range holds i
      uint32_t hi = f.n_traces;
      while (hi - t > 1) {
        const uint32_t mid = (t + hi) / 2;
        if (f.trace_first[mid] <= i) t = mid;
        else hi = mid;
      }
    }
    const uint32_t n = f.trace_cnt[t], first = f.n_traces > 1 ? f.trace_first[t] : 0u;
    if (n <= SORT_CHUNK) continue;
    const EntryKey* const mk = (const EntryKey*)f.merge_keys + first;
    const uint32_t me = i - first, own = me / SORT_CHUNK;
    const EntryKey k = mk[me];
    uint32_t at = me % SORT_CHUNK;
    constexpr uint32_t U = 4;
#pragma unroll 1
    for (uint32_t c = 0; c * SORT_CHUNK < n; c += U) {
      uint32_t lo[U] = {0, 0, 0, 0};
#pragma unroll 1
      for (uint32_t step = SORT_CHUNK; step; step >>= 1) {
        EntryKey m[U];
#pragma unroll
        for (uint32_t u = 0; u < U; u++) {
          const uint32_t j = (c + u) * SORT_CHUNK + lo[u] + step - 1;
          m[u] = mk[min(j, n - 1)];
        }
#pragma unroll
        for (uint32_t u = 0; u < U; u++) {
          const uint32_t j = lo[u] + step - 1;
          if (j < SORT_CHUNK && (c + u) * SORT_CHUNK + j < n && c + u != own &&
              (c + u < own ? !key_less(k, m[u]) : key_less(m[u], k)))
            lo[u] += step;
        }
      }
      at += lo[0] + lo[1] + lo[2] + lo[3];
    }
    copy_entry((total <= f.host_cap ? f.host_entries : f.sorted) + first + at, all + i);
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
  static_assert(FILTER_MAX_LGB == 13, "the larger instantiation");
  if (f.direct) return hipSuccess;
  hipLaunchKernelGGL(f.max_lgb > 11 ? k_filter_part<13> : k_filter_part<11>, dim3(tile_grid(f.n_tiles, 0, 0)), dim3(FNT), 0,
                     s, f);
  return hipGetLastError();
}
hipError_t launch_filter_count(const FilterBuffers& f, hipStream_t s) {
  hipError_t e;
  if (f.extra_max) {
    hipLaunchKernelGGL(k_filter_plan, dim3(cdiv(f.n_buckets, NT)), dim3(NT), 0, s, f);
    if ((e = hipGetLastError()) != hipSuccess) return e;
  }
  const dim3 grid(f.extra_max + tile_grid(f.n_buckets, 0, 0));
  const bool warp = f.side != nullptr;
  auto count = [&](auto mode) {
    constexpr int M = decltype(mode)::value;
    hipLaunchKernelGGL((warp ? k_filter_count<M, true, 960, 1408> : k_filter_count<M, false, 1024, 1408>),
                       (M & DIRECT_TRACE) ? dim3(f.n_traces) : grid, dim3(FNT), 0, s, f);
  };
  if (f.direct && f.rounds) count(std::integral_constant<int, DIRECT_TRACE | ROUNDS>());
  else if (f.direct) count(std::integral_constant<int, DIRECT_TRACE>());
  else if (f.rounds) count(std::integral_constant<int, BY_BUCKET | ROUNDS>());
  else count(std::integral_constant<int, BY_BUCKET>());
  if ((e = hipGetLastError()) != hipSuccess || f.late_wait) return e;
  return launch_filter_late(f, f.late_max, s);
}
hipError_t launch_filter_late(const FilterBuffers& f, uint32_t n, hipStream_t s) {
  const bool warp = f.side != nullptr;
  n = std::min(n, f.late_max);
  if (f.direct)
    hipLaunchKernelGGL((warp ? k_filter_count<LATE_TRACE, true, 1024, 1408> : k_filter_count<LATE_TRACE, false, 1024, 1408>),
                       dim3(n), dim3(FNT), 0, s, f);
  else  // (room for up to 256 workgroups of a few items)
    hipLaunchKernelGGL((warp ? k_filter_count<LATE_BUCKET, true, 1024, 1408> : k_filter_count<LATE_BUCKET, false, 1024, 1408>),
                       dim3(std::max(n, std::min(4 * n, 256u))), dim3(FNT), 0, s, f);
  return hipGetLastError();
}
hipError_t launch_filter_out(const FilterBuffers& f, hipStream_t s) {
  hipError_t e;
  if (f.n_traces > 1) {
    hipLaunchKernelGGL(k_entries_place, dim3(std::min(1024u, cdiv(f.entries_cap, NT))), dim3(NT), 0, s, f);
    if ((e = hipGetLastError()) != hipSuccess) return e;
  }
  const uint32_t chunks = cdiv(f.entries_cap, SORT_CHUNK);
  // (many traces: a workgroup each, and as many as it takes for a long one among them)
  hipLaunchKernelGGL(k_entries_sort,
                     f.n_traces <= 64 ? dim3(f.n_traces, std::min(1024u / f.n_traces, cdiv(f.entries_cap, 16)))
                                      : dim3(std::max(f.n_traces, 512u)),
                     dim3(NT), 0, s, f);
  if ((e = hipGetLastError()) != hipSuccess || chunks <= 1) return e;
  hipLaunchKernelGGL(k_entries_merge, dim3(std::min(2048u, cdiv(f.entries_cap, NT))), dim3(NT), 0, s, f);
  return hipGetLastError();
}

}  // namespace sc
