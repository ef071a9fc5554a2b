// filter.h -- the grouped race count: a call's racing pairs counted without
// sorting its records.
//
// A record races only inside its group: the accesses of one shared word by
// one block in one epoch, or the accesses of one global word (where a pair is
// concurrent across blocks, or inside one block's epoch).  A group without a
// write or atomic holds no race, and in most traces almost every record is in
// such a group or alone in it.  Records are put into buckets by a hash of
// their group; bitmaps over a bucket's groups then leave the few writes and
// atomics that may have a partner, and the reads that may be one, and their
// pairs are counted one by one, or, for words of many writers, by group.
//
// Types and hash functions shared by the kernels (filter.hip), the host
// runtime (api.cpp) and the CPU tests.
#pragma once
#include <stdint.h>

#include "keys.h"

namespace sc {

constexpr uint32_t FT = 16384;            // records per filter tile
constexpr uint32_t FT_BITS = 14;
// A record's 4-byte key: its place in its tile (bits 0..13), its group's slot
// in the bucket (bits 14..30), whether it is atomic (bit 31).
constexpr uint32_t FILTER_SLOT_BITS = 17;
constexpr uint32_t FILTER_ATOMIC = 1u << 31;
constexpr uint32_t FILTER_MAX_LGB = 13;   // log2 of the most buckets of a trace
constexpr uint32_t FILTER_BUCKET = 16384; // records per bucket aimed at
constexpr uint64_t FILTER_MAX_RECORDS = 2ull * FILTER_BUCKET << FILTER_MAX_LGB;  // of one trace
constexpr uint32_t HOT_PART = 8192;      // hot reads per workgroup of a split bucket, at least: a part reads
                                         // all of its bucket's writes again (with 16384 the warp-aware check of
                                         // 2^22 records took 150 us, with 8192 142, with 5000 138 but 2^23 183
                                         // against 180)
constexpr uint32_t HOT_SHARE = 1024;     // ... and of a call's records, one in so many
// Room for the parts of hot buckets, from the parts that all records would make:
// those of more than HOT_BIG parts always find it (1 + n for n full parts), whatever
// the others take.  (With one room for both, of half as many, a bucket with half of
// 2^22 records was left whole on calls where others came first: 9.4 ms, 0.2 split.)
constexpr uint32_t HOT_BIG = 4;
SC_HD uint32_t hot_big_items(uint32_t full_parts) { return full_parts + full_parts / HOT_BIG + 1; }
SC_HD uint32_t hot_items(uint32_t full_parts) { return (hot_big_items(full_parts) + full_parts / 4 + 8 + 7) / 8 * 8; }

struct FTrace {       // one trace of a grouped call (host-filled)
  const void* rec;    // its first record
  uint64_t n;         // records
  uint64_t row0;      // its first bucket row word
  uint32_t off;       // call index of its first record
  uint32_t tpb;
  uint32_t tile0, ntiles;
  uint32_t bucket0;   // its first bucket
  uint32_t lgb;       // log2 of its buckets
  uint32_t sbits;     // slot bits its buckets use (10 .. FILTER_SLOT_BITS)
  uint32_t pad;
};

// log2 of the buckets of a trace of n records, and the slot bits of a bucket:
// eight slots and more per record of an average bucket (a quarter of them
// writes) keep chance hits to a few per cent.
SC_HD uint32_t filter_lgb(uint64_t n) {
  uint32_t k = 0;
  while (k < FILTER_MAX_LGB && (n >> k) > FILTER_BUCKET) k++;
  return k;
}
SC_HD uint32_t filter_sbits(uint64_t n, uint32_t lgb) {
  const uint32_t b = bits64(n >> lgb) + 4;
  return b < 10 ? 10u : (b > FILTER_SLOT_BITS ? FILTER_SLOT_BITS : b);
}

// 32-bit mixing of a word: lowbias32, the multiply and xor-shift hash with the
// constants that Chris Wellons published after a search for low bias.
SC_HD uint32_t mix32(uint32_t x) {
  x ^= x >> 16;
  x *= 0x7feb352du;
  x ^= x >> 15;
  x *= 0x846ca68bu;
  return x ^ (x >> 16);
}

// Hash of a record's group: one block's epoch of a shared word, or a global
// word.  Records of one group always get one value.
SC_HD uint32_t filter_group(uint64_t unit, uint32_t block, uint32_t epoch, uint32_t space) {
  uint32_t x = (uint32_t)unit * 0x9E3779B1u + (uint32_t)(unit >> 32) * 0x85EBCA77u;
  if (space) x ^= mix32(block * 0xC2B2AE3Du + epoch * 0x27D4EB2Fu + 0x165667B1u);
  return mix32(x);
}

// A record's bucket (the top bits of its group's hash) and its slot there.
SC_HD uint32_t filter_bucket(uint32_t h, uint32_t lgb) { return lgb ? h >> (32 - lgb) : 0u; }
SC_HD uint32_t filter_slot(uint32_t h) { return h & ((1u << FILTER_SLOT_BITS) - 1u); }

// A record in the form its pairs are counted from.
struct FRec {
  uint32_t ulo, uhi, tid;
  uint32_t meta;  // epoch | action << 16 | space << 18
};
SC_HD FRec frec(uint64_t unit, uint32_t tid, uint32_t epoch, uint32_t action, uint32_t space) {
  return FRec{(uint32_t)unit, (uint32_t)(unit >> 32), tid, epoch | (action & 3u) << 16 | (space & 1u) << 18};
}
SC_HD uint32_t frec_action(const FRec& a) { return (a.meta >> 16) & 3u; }
SC_HD uint32_t frec_space(const FRec& a) { return (a.meta >> 18) & 1u; }
// One location: the same word, and for shared words the same block.
SC_HD bool same_location(const FRec& a, uint32_t blk_a, const FRec& b, uint32_t blk_b) {
  return a.ulo == b.ulo && a.uhi == b.uhi && ((a.meta ^ b.meta) & (1u << 18)) == 0 && (frec_space(a) == 0 || blk_a == blk_b);
}
// A location's records fall into groups, each level's inside the one before: the
// location, its block's records, their epoch's, their thread's.  Two records race
// if their actions conflict and they share a group of level 0 but none of level 1,
// or one of level 2 but none of level 3; so counts per group give the pairs,
// signed + - + - over the levels, without a look at any pair.  GROUP_WARP: the
// records of one warp inside a group of level 2.
constexpr uint32_t GROUP_LEVELS = 4, GROUP_WARP = 4;
SC_HD uint32_t warp_of(const FRec& a, uint32_t blk, uint32_t tpb) { return (a.tid - blk * tpb) >> 5; }
SC_HD bool same_group(uint32_t level, const FRec& a, uint32_t blk_a, const FRec& b, uint32_t blk_b, uint32_t tpb) {
  if (!same_location(a, blk_a, b, blk_b)) return false;
  if (level >= 1 && blk_a != blk_b) return false;
  if (level >= 2 && ((a.meta ^ b.meta) & 0xFFFFu) != 0) return false;
  if (level == 3) return a.tid == b.tid;
  return level != GROUP_WARP || warp_of(a, blk_a, tpb) == warp_of(b, blk_b, tpb);
}
// Hashes: a record's location (of a global word that is filter_group's, so its high
// bits are the bucket's), and its groups inside a location (of which the high bits
// count) from that of the level they lie in (the one before; level 2 for GROUP_WARP),
// starting from groups_hash of the location's first record's index.
SC_HD uint32_t location_hash(const FRec& a, uint32_t blk) {
  return mix32(a.ulo * 0x9E3779B1u ^ mix32(a.uhi + (frec_space(a) ? blk * 0xC2B2AE3Du + 1u : 0u)));
}
SC_HD uint32_t groups_hash(uint32_t first) { return first * 0x85EBCA77u; }
SC_HD uint32_t group_hash(uint32_t level, uint32_t h, const FRec& a, uint32_t blk, uint32_t tpb) {
  const uint32_t v = level == 1 ? blk : (level == 2 ? a.meta & 0xFFFFu : (level == 3 ? a.tid : ~warp_of(a, blk, tpb)));
  h = (h ^ v) * 0x9E3779B1u + level;
  return h ^ (h >> 15);
}
// Writes and atomics of a group in one word, and the pairs among them.
SC_HD uint32_t group_one(const FRec& a) { return frec_action(a) == 1u ? 1u : 0x10000u; }
SC_HD uint32_t pairs_ww(uint32_t c) { return (c & 0xFFFFu) * ((c & 0xFFFFu) - 1u) / 2u; }
SC_HD uint32_t pairs_aw(uint32_t c) { return (c & 0xFFFFu) * (c >> 16); }

// Further hashes of a record's group, level 0, 1, ...: groups that share one
// or filter_group's need not share another.
SC_HD uint32_t filter_group2(const FRec& a, uint32_t blk, uint32_t level) {
  uint32_t x = mix32(a.ulo + (level + 1u) * 0x9E3779B9u);
  x = mix32(x ^ (a.uhi * 0xC2B2AE3Du));
  if (frec_space(a)) x = mix32(x + blk * 0x27D4EB2Fu + ((a.meta & 0xFFFFu) + 1u) * 0x165667B1u);
  return x;
}
// Whether two records of one location are concurrent, by different threads,
// not both reads and not both atomic.  warp: lockstep orders two threads of a
// warp unless one of them ran diverged or both are writes of one statement
// (side words; Theorem 1, clauses 1 to 3).
SC_HD bool pair_races(const FRec& a, uint32_t blk_a, const FRec& b, uint32_t blk_b, bool warp, uint32_t tpb,
                      uint32_t side_a, uint32_t side_b) {
  const uint32_t ca = frec_action(a), cb = frec_action(b);
  if (a.tid == b.tid || (ca == cb && ca != 1u)) return false;
  if (blk_a != blk_b) return true;
  if (((a.meta ^ b.meta) & 0xFFFFu) != 0) return false;
  if (!warp) return true;
  const uint32_t wa = (a.tid - blk_a * tpb) >> 5, wb = (b.tid - blk_b * tpb) >> 5;
  if (wa != wb || ((side_a | side_b) & SIDE_DIVERGED)) return true;
  return ca == 1u && cb == 1u && side_a == side_b;
}
// Whether every sum of pairs that a table of nw writes and atomics and n_read
// reads can give stays below 2^32: a location's pairs of all kinds together
// (the cross-block pairs hold them all) are the reads' with the table and the
// table's among themselves.
SC_HD bool pair_sums_fit(uint32_t n_read, uint32_t nw) { return ((uint64_t)n_read + nw) * nw < 1ull << 32; }

}  // namespace sc
