// Decode kernel families and the host rule that picks one per tensor.
#pragma once
#include <cstdint>
#include <initializer_list>

#include "../../include/entropack.h"

namespace ep {

enum DecodePath : uint32_t {
  kPathNone = 0,    // not a decodable tensor (never chosen for a blob that passes validation)
  kPathLut = 1,     // packed slot table in LDS: one 32-bit lookup per symbol
  kPathSearch = 2,  // cumulative table in LDS, branch-free binary search per symbol
  kPathWide = 3,    // packed slot table with a 10-bit coordinate field (wider ranges)
  kPathGlobal = 4,  // frequencies read from the blob in global memory, coarse cumulative index in LDS
};

// LDS bytes of the packed slot table (16 tables x 2^b slots x 4 B) and of the
// cumulative scratch it is built from.
constexpr uint32_t kLutMaxBits = 11;
constexpr int32_t kLutValueMin = -256;   // doubled coordinates whose integer part fits a signed byte
constexpr int32_t kLutValueMax = 255;
constexpr int32_t kWideValueMin = -1024; // ... a signed 10-bit field (wide entries)
constexpr int32_t kWideValueMax = 1023;
constexpr uint32_t kSearchLdsBytes = 128 * 1024;   // the payload rings take the other 32 KiB

// Search path: u16 cumulative tables plus, per table, 2^k + 1 u16 bucket
// bounds (bucket j starts at slot j * 2^(b-k)); k is the largest of
// min(b, 11) .. 8 whose tables fit, so that for b <= 11 and moderate table
// sizes every bucket is a single slot and no search remains.
constexpr uint32_t kBucketBitsMin = 8;
constexpr uint32_t kBucketBitsMax = 11;

struct SearchLayout {
  uint32_t bucket_bits;           // k (0 when no k fits)
  uint32_t bucket, meta, total;   // byte offsets of the buckets and metadata; bytes in all
};

constexpr SearchLayout search_layout_k(uint32_t sum_A, uint32_t k) {
  // u16 cumulative values: sum_A + one end value per table, padded to 4 bytes
  const uint32_t cum = (2 * (sum_A + 16) + 3) & ~3u;
  const uint32_t bucket = cum;
  const uint32_t meta = (bucket + 2 * 16 * ((1u << k) + 1) + 3) & ~3u;
  // the payload rings that follow are addressed as base | offset: 512-byte aligned
  const uint32_t total = (meta + 4 * 32 + 511) & ~511u;
  return SearchLayout{k, bucket, meta, total};
}

constexpr SearchLayout search_layout(uint32_t b, uint32_t sum_A) {
  for (uint32_t k = (b < kBucketBitsMax ? b : kBucketBitsMax); k >= kBucketBitsMin; k--) {
    const SearchLayout S = search_layout_k(sum_A, k);
    if (S.total <= kSearchLdsBytes) return S;
  }
  return SearchLayout{0, 0, 0, 0};
}

// Search path, compact form.  Tables of high-rate tensors are mostly gaps: at 8
// bits per weight a third of the symbols in a table's index range occur.  This
// form keeps only those, one u32 each (F | z << 16, z the integer part of the
// coordinate, 2m for field 8) and an end entry (F = 2^b) per table, and u16
// buckets of 2^k per table that hold the index of the symbol of their first slot
// (k = 11, or 10 when the symbols need the room).  A symbol is then one bucket
// read, one read of consecutive entries and, for b = 12, one compare: no metadata,
// no binary search (256 x 512 at b = 12: 82 -> 40 us, with the one-chain tasks it
// allows; 10240 x 3840 at 8 bits per weight: 150 -> 122 us).  Whether the symbols fit is known once they are counted, in
// the table build, which falls back to the cumulative form otherwise and says
// which form it chose in a word at the start of the area's last 512 bytes.
constexpr uint32_t kCompactBits = 11, kCompactBitsLow = 10;
constexpr uint32_t kCompactTail = 512;
constexpr int32_t kCompactValue = 65532;   // |doubled coordinate| whose z fits 16 bits

constexpr uint32_t compact_buckets(uint32_t area, uint32_t k) { return area - kCompactTail - (32u << k); }

// Bytes of the search path's table area; `compact`: the compact form may be tried.
// The one-chain rings that follow need 1024-byte alignment.
constexpr uint32_t search_area(uint32_t b, uint32_t sum_A, bool compact) {
  const uint32_t plain = search_layout(b, sum_A).total;
  if (!compact) return plain;
  uint32_t want = 4 * (sum_A + 18) + (32u << kCompactBits) + kCompactTail;
  if (sum_A > kSearchLdsBytes || want > kSearchLdsBytes) want = kSearchLdsBytes;
  if (want < plain + kCompactTail) want = plain + kCompactTail;
  return (want + 1023) & ~1023u;
}

// Whether the compact form may be tried: its z fit 16 bits and the cumulative
// form, should it be needed, leaves the form word free.
constexpr bool compact_possible(uint32_t b, uint32_t sum_A, int32_t coord2_min, int32_t coord2_max) {
  return coord2_min >= -kCompactValue && coord2_max <= kCompactValue &&
         ((search_layout(b, sum_A).total + kCompactTail + 1023) & ~1023u) <= kSearchLdsBytes;
}

// Whether the symbols are certain to fit (they are at most sum_A).
constexpr bool compact_certain(uint32_t sum_A) {
  return sum_A <= kSearchLdsBytes && 4 * (sum_A + 18) <= compact_buckets(kSearchLdsBytes, kCompactBitsLow);
}

// Global-table path (tables too large for the LDS paths; App. C.3 places the decode
// tables in shared or packed global memory by alphabet size).  The blob's own u16
// frequency arrays are read from global memory; LDS holds every G-th cumulative
// value of each table (G = 2^g), u16, n_t = ceil(A_t / G) entries per table, then
// u32 metadata for t < 16: the first coarse entry of the table, its min, n_t and
// the byte offset of its frequencies in the blob.  A symbol is found by a binary
// search over the coarse entries and a scan of at most G frequencies.
constexpr uint32_t kGlobalBitsMin = 3;
constexpr uint32_t kGlobalBitsMax = 6;

struct GlobalLayout {
  uint32_t g_bits;        // log2 G (0 when nothing fits)
  uint32_t meta, total;   // byte offset of the metadata; bytes in all (512-byte aligned)
};

inline GlobalLayout global_layout(const uint32_t* A) {
  for (uint32_t g = kGlobalBitsMin; g <= kGlobalBitsMax; g++) {
    uint64_t n = 0;
    for (int t = 0; t < 16; t++) n += (A[t] + (1u << g) - 1) >> g;
    const uint64_t meta = (2 * n + 3) & ~3ull;
    const uint64_t total = (meta + 4 * 64 + 511) & ~511ull;
    if (total <= kSearchLdsBytes) return GlobalLayout{g, (uint32_t)meta, (uint32_t)total};
  }
  return GlobalLayout{0, 0, 0};
}

// Whether path P can hold the tables of tensor I.
inline bool path_fits(uint32_t P, const ep_tensor_info& I) {
  switch (P) {
    case kPathLut:
      return I.prob_bits <= kLutMaxBits && I.coord2_min >= kLutValueMin && I.coord2_max <= kLutValueMax;
    case kPathWide:
      return I.prob_bits <= kLutMaxBits && I.coord2_min >= kWideValueMin && I.coord2_max <= kWideValueMax;
    case kPathSearch:
      return I.sum_alphabet <= 0xFFFF0u && search_layout(I.prob_bits, I.sum_alphabet).bucket_bits != 0;
    case kPathGlobal:
      return I.prob_bits >= 9 && I.prob_bits <= 15 && global_layout(I.table_A).g_bits != 0;
    default:
      return false;
  }
}

// The fastest path that holds the tables.  Every blob that passes validation (A <= 2^b
// <= 2^15 per table) fits the global-table path: 16 tables of at most 2^15 symbols
// need 2^16 coarse entries at G = 8 (128 KiB) or half that at G = 16.
inline uint32_t choose_path(const ep_tensor_info& I) {
  for (uint32_t P : {kPathLut, kPathWide, kPathSearch, kPathGlobal})
    if (path_fits(P, I)) return P;
  return kPathNone;
}

}  // namespace ep
