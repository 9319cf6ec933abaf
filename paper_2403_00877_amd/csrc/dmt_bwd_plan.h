// How the sparse update (dmt_bwd.hip) divides a call: sort blocks, reduce tiles, and where everything lies
// in the workspace.
#pragma once
#include <algorithm>

#include "dmt_internal.h"

namespace {

constexpr int kBlock = 256;
#ifndef DMT_SORT_ITEMS
#define DMT_SORT_ITEMS 8
#endif
#ifndef DMT_RADIX_BITS
#define DMT_RADIX_BITS 8
#endif
constexpr int kSortItems = DMT_SORT_ITEMS;
constexpr int kMaxRadixBits = DMT_RADIX_BITS;      // digit width of one sort pass
constexpr int kMaxRadix = 1 << kMaxRadixBits;
// A call of up to kWideNnz lookups is bound by its launches, not by bytes: it sorts in digits of up to
// 10 bits, and the scatter's blocks add up the digit counts of their table's other blocks themselves, so
// a pass is two launches instead of three and there are fewer passes (18 bits of row id: 4 launches
// instead of 9).  The counts a block reads grow with its table's blocks, which is what the limit is for:
// at kWideNnz lookups, all in one table, a block reads 256 lines of 4 KB.
constexpr int kWideRadixBits = 10;
constexpr int64_t kWideNnz = 1 << 19;
constexpr int kSortTile = kBlock * kSortItems;   // records per sort block, at most
static_assert(kSortItems < 16, "four bits of a sort block's entry");
// Records a thread of a sort block ranks, one after another, in calls that sort in wide digits.  Such a call
// does not fill the chip and is bound by that chain of ballots, so blocks are as small as two records a
// thread while a call has 256 of full tables, and a table 64 (table_items): a block reads the digit
// counts of all of its table's.  Whole update, us, blocks of 2048 / smaller ones: 8 tables of 16 K lookups
// 115.8 / 110.5 (1024 records), one of 32 K 50.2 / 45.4 (512), 4 of 32 K 112.3 / 111.6; past the line 2 of 123 K
// 119.3 / 123.1, one of 127 K 80.6 / 98.9.  A table's own length decides, not the mean of a call's tables, and
// only the kernels know it: 130 K lookups, 97 % of them in one of 8 tables, took 80.1 us in the blocks of 512 that
// the mean asks for, in blocks of 2048 65.5, and take 66.0; half of them in one table 67.4, 63.5 and 61.4.
constexpr int kTableBlocks = 64;
constexpr int64_t kWideBlocks = kWideNnz / kSortTile;
inline int wide_items(int64_t nnz) {     // the least of any table
  const int64_t items = (nnz + kBlock * kWideBlocks - 1) / (kBlock * kWideBlocks);
  return (int)std::min<int64_t>(kSortItems, std::max<int64_t>(2, items));
}
// Of a table of len lookups; least_items = kSortItems in narrow digits.  Never more blocks than
// least_items makes.
__host__ __device__ inline int table_items(uint32_t len, int least_items) {
  const uint32_t items = (len + kBlock * kTableBlocks - 1) / (kBlock * kTableBlocks);
  return items <= (uint32_t)least_items ? least_items : items < (uint32_t)kSortItems ? (int)items : kSortItems;
}
// A call of so few lookups, in tables of so few samples, sorts in one launch (bwd_sort_small).
constexpr int64_t kSmallNnz = 7168, kSmallBatch = 2048;
constexpr int kScanItems = 16;
constexpr int kScanTile = kBlock * kScanItems;   // records per head-scan block
// Sorted records per reduce tile (one wave walks one): 128, or down to 16 where a call is too small
// to fill the chip with tiles of 128.  A wave takes about 0.25 us per record, so 2300 records in
// tiles of 128 are 18 waves of 30 us (tiles of 16: 7.7); but every run that crosses a tile
// boundary costs a partial sum and a share of the fix-up, so tiles shrink only until there are
// fill_tiles of them (four waves per SIMD at 4096, eight at 8192).
constexpr int kReduceTile = 128, kMinReduceTile = 16;
inline int64_t fill_tiles(int max_dim) { return max_dim <= 128 ? 8192 : 4096; }
inline int reduce_tile(int64_t nnz, int max_dim) {
  int tile = kReduceTile;
  while (tile > kMinReduceTile && (nnz + tile / 2 - 1) / (tile / 2) <= fill_tiles(max_dim)) tile /= 2;
  return tile;
}
#ifndef DMT_RU
#define DMT_RU 4
#endif
constexpr int kReduceUnroll = DMT_RU;
constexpr uint32_t kInertBit = 0x80000000u;      // key flag of an id outside its table
constexpr int kScanThreads = 1024;               // block of the per-table offset scan
constexpr int kScanBatch = 16;                   // sort blocks whose counts it reads together

struct BwdWs {
  uint64_t* pk_a;
  uint64_t* pk_b;
  uint32_t* hist;         // [nblk_sort][kMaxRadix], or [nblk_sort][1 << kWideRadixBits]
  uint32_t* seg_begin;    // [F + 1] first record of each table (seg_begin[F] = nnz)
  uint32_t* seg_blk;      // [F + 1] first sort block of each table
  uint32_t* blk_table;    // [nblk_sort] table of each sort block, << 4 | its records per thread
  uint32_t* blk_heads;    // [nblk_scan]
  uint32_t* seg_off;      // [nnz + 1]
  uint32_t* num_unique;   // [1]
  float* partials;        // [2 * tiles][Dmax]
  size_t bytes;
  int64_t nblk_sort, nblk_scan, ntiles;
  int tile;               // records per reduce tile
  bool wide;              // sort in wide digits
  int least_items;        // records per thread of a sort block, at least (table_items)
};

BwdWs carve(const dmt_plan* p, int64_t nnz, void* base) {
  BwdWs w;
  const int64_t n = nnz > 0 ? nnz : 1;
  w.nblk_sort = (n + kSortTile - 1) / kSortTile + p->F;   // every table may end in a partial block
  w.nblk_scan = (n + kScanTile - 1) / kScanTile;
  w.tile = reduce_tile(n, p->max_dim);
  w.ntiles = (n + w.tile - 1) / w.tile;
  // partial slots for the tiles of this and of every smaller call (a workspace sized for the largest
  // serves all of them)
  const int64_t slots = std::max((n + kReduceTile - 1) / kReduceTile,
                                 std::min((n + kMinReduceTile - 1) / kMinReduceTile, fill_tiles(p->max_dim)));
  size_t off = 0;
  auto take = [&](size_t bytes) {
    size_t o = off;
    off = dmt_align_up(off + bytes, 256);
    return (char*)((uintptr_t)base + o);          // (base is null when only the size is wanted)
  };
  w.pk_a = (uint64_t*)take(sizeof(uint64_t) * n);
  w.pk_b = (uint64_t*)take(sizeof(uint64_t) * n);
  w.seg_begin = (uint32_t*)take(sizeof(uint32_t) * (p->F + 1));
  w.seg_blk = (uint32_t*)take(sizeof(uint32_t) * (p->F + 1));
  // (never less room for more lookups: a workspace sized for the largest call serves all of them)
  w.blk_table = (uint32_t*)take(sizeof(uint32_t) * std::max(w.nblk_sort, std::min((n + 2 * kBlock - 1) / (2 * kBlock), kWideBlocks + 1) + p->F));
  w.blk_heads = (uint32_t*)take(sizeof(uint32_t) * (w.nblk_scan + 1));
  w.num_unique = (uint32_t*)take(sizeof(uint32_t) * 64);
  // The sort is done with its counts before seg_off and partials are written, so wide counts may lie
  // over them.  That is room enough but for few lookups in narrow rows, whose counts get room of their
  // own unless the tables are many (then the digits stay narrow).  Never less room for more lookups: a
  // workspace sized for the largest call serves all of them.
  const size_t hist_at = off;
  int64_t counts = (int64_t)kMaxRadix * w.nblk_sort;
  if (p->F <= 64)
    counts = std::max(counts, (std::min<int64_t>(n, 8 * kSortTile) / kSortTile + 1 + p->F) << kWideRadixBits);
  w.hist = (uint32_t*)take(sizeof(uint32_t) * counts);
  w.seg_off = (uint32_t*)take(sizeof(uint32_t) * (n + 1));
  w.partials = (float*)take(sizeof(float) * 2 * slots * p->max_dim);
  w.bytes = off;
  w.wide = n <= kWideNnz && (sizeof(uint32_t) << kWideRadixBits) * w.nblk_sort <= off - hist_at;
  // smaller sort blocks as far as their counts have room
  w.least_items = kSortItems;
  for (int items = wide_items(n); w.wide && items < kSortItems; ++items) {
    const int64_t nblk = (n + items * kBlock - 1) / (items * kBlock) + p->F;
    if ((sizeof(uint32_t) << kWideRadixBits) * nblk > off - hist_at) continue;
    w.least_items = items;
    w.nblk_sort = nblk;
    break;
  }
  return w;
}

}  // namespace
