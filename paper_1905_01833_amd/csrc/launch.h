// launch.h -- device data structures and kernel launch wrappers of the race
// check, shared by the kernels (kernels.hip) and the host runtime (api.cpp).
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

#include "filter.h"
#include "keys.h"
#include "tilewalk.h"

namespace sc {

constexpr int NT = 256;            // threads per workgroup
constexpr int ITEMS = 16;          // keys per thread
constexpr int TILE = NT * ITEMS;   // keys per tile (sort and scan)
constexpr int SW = 45;             // 32-bit words of a serialised segment State
constexpr int GROUP = 256;         // tiles per group of the output prefix
constexpr uint32_t MAX_HGROUP_SHIFT = 12; // histogram groups hold at most 4096 tiles

// kernel-side error flags beyond the per-trace layout errors of keys.h
// (ERR_GROUP_FULL: the grouped race count ran out of room; the call takes the
// sorting path)
enum : uint32_t { ERR_STAGE_OVERFLOW = 16, ERR_NEEDS_WIDE = 32, ERR_GROUP_FULL = 64 };

struct TraceDesc {   // one trace of a call (host-filled)
  uint64_t off;      // first record
  uint64_t n;        // records
  uint32_t tpb;      // threads per block
  uint32_t tile0;    // first tile
  uint32_t ntiles;
  uint32_t group0;   // first histogram group (runs of 2^gshift tiles of this trace)
  uint32_t ngroups;
  uint32_t gshift;   // log2 of the tiles per histogram group (about sqrt(ntiles))
  uint32_t pad[3];
};

struct TileRef {     // tile -> (trace, tile within trace), and where its records are
  uint32_t trace;
  uint32_t local;
  uint32_t first;    // call index of the tile's first record: its keys (a call holds < 2^32 records)
  uint32_t n_flags;  // records in the tile (bits 0..30); bit 31: the trace is sorted whole in LDS
  const void* rec;   // the tile's first record (device memory; the traces of a call need not be adjacent)
};
constexpr uint32_t TILE_SHORT = 1u << 31;

// Dedicated staging of a tile whose racing locations outgrow its slice of
// the idle key buffer: stage_ref[tile] = (first entry in `stage` <<
// STAGE_CAP_BITS) | capacity, or 0 for a tile that stages in its slice.
constexpr uint32_t STAGE_CAP_BITS = 16;
constexpr uint64_t STAGE_CAP_MASK = (1ull << STAGE_CAP_BITS) - 1;

struct GroupRef {    // histogram group -> trace, and its tiles
  uint32_t trace;
  uint32_t first;    // call index of the group's first tile
  uint32_t n_flags;  // tiles in the group (bits 0..30); bit 31 (TILE_SHORT): the trace is sorted whole in LDS
  uint32_t pad;
};

struct TileOut {     // per tile, from the tile scan
  uint32_t in_count; // racing locations that start and end inside the tile
  uint32_t owns;     // 1: the tile's last location continues into the next tile
};

struct Ctrl {               // per-call control block (device)
  uint32_t pass_bits;       // (most radix passes of a trace << 16) | the key bits that trace sorts
  uint32_t error_flags;     // LAYOUT_ERR_* / ERR_* of any trace or kernel
  uint64_t first_bad;       // smallest global index of an invalid record
  uint64_t total_entries;   // racing locations of the call
  uint32_t wide_traces;     // traces whose key needs two words
  uint32_t pad;
};
// Radix passes the call's traces need (all of them done: the scan may run).
SC_HD uint32_t ctrl_passes(uint32_t pass_bits) { return pass_bits >> 16; }

struct RaceOut {            // mirrors sim_race (64 bytes)
  uint32_t trace;
  uint8_t space, kinds;
  uint16_t reserved16;
  uint32_t block, reserved32;
  uint64_t unit, ww, rw, aw, ar, xb;
};

struct Buffers {            // device pointers of one call
  const TraceDesc* desc;
  const TileRef* tiles;
  TraceStats* stats_part;   // [tile]
  TraceLayout* layout;      // [trace]
  void* keys[2];             // uint64_t[] (one-word keys) or u128[] (two-word keys, `wide`)
  const GroupRef* groups;   // [group]
  uint32_t* thist;          // [tile][radix] the current pass's digit offsets within the tile's group
                            // (uint16_t when no group has more than 16 tiles, see kernels.hip)
  uint16_t* tcnt;           // [tile][radix] the current pass's digit counts (a tile holds 4096 keys)
  uint32_t* gtot;           // [group][radix] group totals
  uint64_t* gbase;          // [group][radix] absolute digit bases of the group
                            // (radix: 2^8 in pass 0, 2^digit_bits after it; rows of RADIX_MAX words at most)
  uint32_t* agg;            // [tile][SW]
  TileOut* tout;            // [tile]
  RaceOut* cross;           // [tile]
  uint32_t* cross_flag;     // [tile]
  uint32_t* group_sum;      // [group]
  RaceOut* stage;           // dedicated staging of the tiles stage_ref names (see STAGE_CAP_BITS)
  const uint64_t* stage_ref;// [tile], or nullptr: every tile stages in its slice of the idle key buffer
  Ctrl* ctrl;
  RaceOut* out;
  uint64_t out_cap;
  uint32_t n_traces;
  uint32_t n_tiles;
  uint32_t n_groups;        // histogram groups
  uint32_t grid_stream;     // workgroups of k_stats / k_keygen / k_upsweep (multiple of 8)
  uint32_t grid_sort;       // workgroups of k_scatter
  uint32_t scatter_nt;      // threads of a k_scatter workgroup: 256, or 512 (one-word keys)
  uint32_t grid_scan;       // workgroups of k_scan_tiles
  uint32_t max_group_tiles; // most tiles in one histogram group of the call
  uint32_t max_trace_groups;// most histogram groups in one trace of the call
  uint32_t fuse0;           // 1: digit 0 is tid mod 256 in every trace; k_stats builds its histograms
                            // and k_keygen_scatter does radix pass 0 (see kernels.hip)
  uint32_t wide;            // 1: two-word keys for every trace of the call
  const uint32_t* small_traces; // traces sorted whole in LDS: n_small1 of one tile, then
                            // n_small4 of two to four tiles (one-word keys only)
  uint32_t n_small1, n_small4;
  uint32_t small_max_tiles; // 4 with one-word keys, 1 with two-word keys
  uint32_t small_from;      // first radix pass done in LDS for those traces (pass 0 is
                            // k_keygen_scatter's when fuse0)
  uint32_t key_bytes;       // 8 or 16
  uint32_t fitness;         // 1: fitness keys (epoch and action dropped), for the EP fitness count
  const uint32_t* side;     // warp-aware check: one side word per record (call index), else nullptr
  uint32_t digit_bits;      // digit width of the radix passes after pass 0: RADIX_BITS or RADIX_WIDE_BITS
};

// Counters of a grouped call (FilterBuffers::cnt): entries found, items of the
// hottest buckets and of other hot ones, entries of the trace with most (where they exceed
// SORT_ALONE), buckets or traces for the later workgroups, those whose candidates
// fill two to four tables.
enum : uint32_t { FC_ENTRIES = 0, FC_EXTRA = 1, FC_MOST = 2, FC_LATE = 3, FC_ROUNDS = 4, FC_EXTRA2 = 5, FC_COUNT = 6 };
constexpr uint32_t SORT_CHUNK = 2048;         // entries sorted in one workgroup's LDS
constexpr uint32_t SORT_ALONE = 256;          // ... of which one workgroup places so many at once
// Entries of a trace, at most: beyond, merging its sorted chunks takes longer than
// sorting its records does.  (Grouped / sorted, in us: 262144 entries of 2^24
// records 1562 / 1822; of 2^22 records, 200000 1411 / 1118, 60000 512 / 624.)
constexpr uint32_t GROUP_MAX_ENTRIES = 1u << 18;
constexpr uint32_t GROUP_MAX_TRACES = 8192;   // traces of a grouped call

struct GroupHead {          // what the host needs of a grouped call besides its entries
  uint32_t entries, error_flags;
  uint64_t first_bad;
  uint32_t late;            // FC_LATE (with FilterBuffers::late_wait: still to be counted)
  uint32_t rounds;          // FC_ROUNDS
};
struct FilterBuffers {      // device pointers of a call's grouped race count (filter.h, filter.hip)
  FTrace* tr;
  const FTrace* tr_src;     // where k_filter_begin finds them: pinned host memory, or tr
  uint32_t n_traces, n_tiles, n_buckets;
  uint32_t direct;          // 1: every trace is counted by one workgroup from its records
  uint32_t* tile_trace;     // [tile] its trace
  uint32_t* bucket_trace;   // [bucket] its trace
  uint32_t* keys;           // [record] a tile's keys by bucket (filter.h)
  uint32_t* rows;           // [tile][buckets + 1] first write | first read << 16 of each bucket in the tile
  uint32_t* hot;            // [bucket] reads of hot words as the tiles counted them, then the bucket's parts
  uint32_t* hot_writes;     // [bucket] writes of hot words, estimated
  uint2* extra;             // the parts of split buckets: (bucket, part)
  uint32_t extra_max;       // room for them (a multiple of 8; 0: no bucket is split)
  uint32_t extra_big;       // ... of which for buckets of more than HOT_BIG parts (the first)
  uint32_t hot_part;        // hot reads per part
  uint2* late;              // buckets (traces, if direct) for the later workgroups, and their part
  uint32_t late_max;        // room for them
  uint32_t late_wait;       // 1: the host starts those workgroups, if there is work for them; until then nothing is put in order
  uint32_t rounds;          // 1: the first workgroups fill such tables themselves
  uint32_t max_rounds;      // tables a later workgroup may fill one after another, a power of two
  uint32_t max_lgb;         // the largest FTrace::lgb of the call
  const uint32_t* side;     // warp-aware check: one side word per record, else nullptr
  uint32_t* cnt;            // [FC_COUNT]
  uint32_t* trace_cnt;      // [trace] entries
  uint32_t* trace_fill;     // [trace] entries placed
  uint32_t* trace_first;    // [trace] first entry of its range
  RaceOut* entries;         // as the buckets found them
  RaceOut* placed;          // by trace
  RaceOut* sorted;          // in order
  void* merge_keys;         // 16 bytes per entry, of traces with more than SORT_CHUNK
  uint32_t entries_cap;     // entries each of the three holds
  GroupHead* head;          // pinned host memory
  RaceOut* host_entries;    // pinned host memory: the entries in order, if no more than
  uint32_t host_cap;        // this many
  Ctrl* ctrl;
};

// Barrier instances (per trace and boundary) of the redundant-barrier check:
// `copies` copies of every counter pair, spread over cache lines, summed by
// the host.  Trace i's boundaries start at bar_base[i].
struct BarrierCount {
  unsigned long long instances;
  unsigned long long racing;
};

// Kernel stages, in launch order.
enum Stage { ST_INIT = 0, ST_STATS, ST_LAYOUT, ST_KEYGEN, ST_UPSWEEP, ST_SORT, ST_SCAN, ST_CROSS, ST_OUT,
             ST_SORT_SMALL, ST_FILTER_PART, ST_FILTER_COUNT, ST_FILTER_OUT, ST_COUNT };

hipError_t launch_init(const Buffers& b, hipStream_t s);
hipError_t launch_stats(const Buffers& b, hipStream_t s);
hipError_t launch_layout(const Buffers& b, hipStream_t s);
hipError_t launch_keygen(const Buffers& b, hipStream_t s);  // with fuse0: keys + radix pass 0
hipError_t launch_upsweep(const Buffers& b, uint32_t pass, hipStream_t s);  // histograms and offsets
hipError_t launch_scatter(const Buffers& b, uint32_t pass, hipStream_t s);
hipError_t launch_sort_small(const Buffers& b, hipStream_t s);
hipError_t launch_scan_tiles(const Buffers& b, uint32_t passes_done, hipStream_t s);
hipError_t launch_scan_cross(const Buffers& b, uint32_t passes_done, hipStream_t s);
hipError_t launch_scan_out(const Buffers& b, uint32_t passes_done, hipStream_t s);
hipError_t launch_reset_errors(const Buffers& b, uint32_t mask, hipStream_t s);
// The grouped race count, in this order: keys by bucket and record checks; the
// pairs; the entries in order.
hipError_t launch_filter_part(const FilterBuffers& f, hipStream_t s);
hipError_t launch_filter_count(const FilterBuffers& f, hipStream_t s);
hipError_t launch_filter_late(const FilterBuffers& f, uint32_t n, hipStream_t s);  // (launch_filter_count does it without late_wait)
hipError_t launch_filter_out(const FilterBuffers& f, hipStream_t s);
// Redundant-barrier check over the sorted keys of a finished call: clears
// `table` (n_counts entries) and counts every trace's barrier instances.
hipError_t launch_barriers(const Buffers& b, const uint64_t* bar_base, BarrierCount* table, uint64_t n_counts,
                           uint32_t copies, hipStream_t s);

// EP fitness of one trace (mirrors sim_fitness, 48 bytes).
struct FitOut {
  uint64_t n_records, n_locations, n_location_threads, global_range, shared_range;
  double fitness;
};
// Over the sorted fitness keys of a finished call: every trace's row to out
// (device memory, n_traces rows).  Does nothing while fewer than the needed
// radix passes ran (the host runs them and launches again).
hipError_t launch_fitness(const Buffers& b, uint32_t passes_done, FitOut* out, hipStream_t s);

// Barrier divergence (Alg. 4): whole blocks of one trace per chunk.
struct DivChunk {
  uint64_t thread0;  // the chunk's first thread (index into the arrival counts)
  uint32_t trace;
  uint32_t block;    // the chunk's first block within its trace
  uint32_t n_blocks;
  uint32_t tpb;      // threads per block
  uint32_t block0;   // the chunk's first block among the call's blocks: its list's place
  uint32_t pad;
};
struct DivOut {      // mirrors sim_divergence (24 bytes): fewest and most arrivals, threads below the most
  uint32_t trace, block, lo, hi;
  uint64_t early;
};
constexpr uint32_t DIV_CHUNK_THREADS = TILE;  // threads per chunk (whole blocks, at least one)

// The chunks' lists of divergent blocks and their lengths (with the list's
// place), then the chunks' output offsets and the number of divergent blocks
// (*total) and the first host_cap of those in (trace, block) order: pinned host
// memory.  So is `chunks`.
hipError_t launch_divergence(const DivChunk* chunks, uint32_t n_chunks, const uint32_t* arrivals, DivOut* lists,
                             uint2* chunk_cnt, uint64_t* chunk_off, uint64_t* total, DivOut* host_out, uint32_t host_cap,
                             hipStream_t s);
// All of them, to out.
hipError_t launch_divergence_emit(uint32_t n_chunks, const DivOut* lists, const uint2* chunk_cnt, const uint64_t* chunk_off,
                                  DivOut* out, hipStream_t s);

// Warp-aware check (Theorem 1's warp clauses) after the plain check of a
// call whose keys carry the side field: the pairs lockstep execution
// orders are subtracted from the plain entries (n_entries of them, device
// memory, in key order; `removed` holds 4 counters per entry), and the
// entries left with a pair go to `out`, their number to *n_out (device).
hipError_t launch_warp_refine(const Buffers& b, const RaceOut* entries, uint64_t n_entries, unsigned long long* removed,
                              RaceOut* out, unsigned long long* n_out, hipStream_t s);

// Device memory of the no-allocation entry point: a file-scope array of
// SCRATCH_BYTES in the library's device code, one copy per GPU.
constexpr size_t SCRATCH_BYTES = (size_t)128 << 20;
// The array's address on `device` (which must be the current device), looked
// up once per device and remembered; the error of that lookup otherwise.
hipError_t scratch_address(int device, void** out);

}  // namespace sc
