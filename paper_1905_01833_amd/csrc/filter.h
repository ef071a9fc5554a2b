// filter.h -- the conflict filter: which records of a call can be part of a
// racing pair at all.
//
// A record races only inside its group: the accesses of one shared word by
// one block in one epoch, or the accesses of one global word (where a pair is
// concurrent across blocks, or inside one block's epoch).  A group without a
// write or atomic, or touched by one thread only, holds no race, and in most
// traces almost every record is in such a group.  The filter keeps every
// record that could race (and some that do not), so the exact count over the
// kept records alone is the exact count of the trace.
//
// Types and hash functions shared by the kernels (filter.hip), the host
// runtime (api.cpp) and the CPU tests.
#pragma once
#include <stdint.h>

#include "keys.h"

namespace sc {

constexpr uint32_t FT = 16384;           // records per filter tile
constexpr uint32_t FT_BITS = 14;
constexpr uint32_t FILTER_SLOT_BITS = 18;  // slot bits of a filter key (the other 14 are the record's place in its tile)
constexpr uint32_t FILTER_MAX_LGB = 12;  // log2 of the most buckets of a trace
constexpr uint32_t FILTER_BUCKET = 16384; // records per bucket aimed at

struct FTrace {       // one trace of a filtered call (host-filled)
  const void* rec;    // its first record
  uint64_t n;         // records
  uint64_t row0;      // its first bucket row word
  uint32_t off;       // call index of its first record
  uint32_t tpb;
  uint32_t tile0, ntiles;
  uint32_t bucket0;   // its first bucket
  uint32_t lgb;       // log2 of its buckets
  uint32_t sbits;     // slot bits its buckets use (10 .. FILTER_SLOT_BITS)
  uint32_t surv0;     // its first word of the survivor bitmap
};

// log2 of the buckets of a trace of n records, and the slot bits of a bucket:
// about 16 slots per record of an average bucket (a quarter of them writes)
// keeps chance hits to a few per cent.
SC_HD uint32_t filter_lgb(uint64_t n) {
  uint32_t k = 0;
  while (k < FILTER_MAX_LGB && (n >> k) > FILTER_BUCKET) k++;
  return k;
}
SC_HD uint32_t filter_sbits(uint64_t n, uint32_t lgb) {
  const uint32_t b = bits64(n >> lgb) + 4;
  return b < 10 ? 10u : (b > FILTER_SLOT_BITS ? FILTER_SLOT_BITS : b);
}

// 32-bit mixing of a word (a published integer hash of the multiply and
// xor-shift kind: every input bit reaches every output bit).
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

// A record's bucket (top bits of its group's hash) and filter key.
SC_HD uint32_t filter_bucket(uint32_t h, uint32_t lgb) { return lgb ? h >> (32 - lgb) : 0u; }

// Second hash, of a record's (location, block, epoch) or of its location
// alone, for the exact test of the records the bitmaps let through.
SC_HD uint32_t filter_exact_hash(uint64_t unit, uint32_t block, uint32_t epoch, uint32_t kind, uint32_t round) {
  return mix32(mix32((uint32_t)unit + round * 0x68E31DA4u) ^
               mix32((uint32_t)(unit >> 32) * 0xB5297A4Du + block * 0x1B56C4E9u + epoch * 0x9E3779B1u + kind));
}

}  // namespace sc
