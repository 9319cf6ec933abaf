// dmt_tower_lookup_bwd_update: gradients to the activated rows only (paper
// Sec. 2.2), as  samples of the lookups -> stable LSD radix sort by row id inside every
// table's records -> tiled segment reduce fused with the rowwise Adagrad row
// update -> fix-up of rows whose run spans several tiles.
//
// Everything is deterministic: the sort is stable (equal rows keep ascending
// bag order), every row's gradient is summed in a fixed order, and each row has
// exactly one writer.  No floating-point atomics anywhere.
//
// The sort's result: 64-bit records (global_row << 32 | bag), where
// global_row = (sum of rows of earlier tables) + row and bag = f*B + b.  The
// lookups arrive grouped by table (bags are table-major), so the sort never moves
// a record out of its table's range: sort blocks are aligned to the tables and
// every pass ranks only the bits of the row inside the table, which takes
// ceil(log2(largest table)) bits instead of ceil(log2(all rows)), and until its last pass
// a record is the row inside the table and the sample.  An id outside
// its table gets the key  kInertBit | (global id one past the table's last row):
// it sorts behind the table's rows, equals no row's key, and is never touched.
// `offsets` must tile [0, nnz) (ascending, offsets[0] = 0, last = nnz): bwd_bag_samples
// checks this, records the first bag that breaks it, and the reduce and fix-up kernels
// then return without touching a row (dmt_last_device_error reports DMT_EINVAL).
#include <algorithm>
#include <mutex>
#include <type_traits>

#include "dmt_internal.h"
#include "dmt_device_utils.h"
#include "dmt_bwd_plan.h"

namespace {

// ------------------------------------------------------------------ samples of the lookups

// Where each table's records start and which sort blocks cover them.  Run by one block.
// The starts come from the offsets of every table's first bag, clamped to [0, nnz] and made ascending (each at
// least the largest before it), so that records and blocks stay inside their arrays whatever `offsets` holds.
__device__ void build_sort_map(const int64_t* __restrict__ offsets, uint32_t B, int F, int64_t nnz,
                               int least_items, uint32_t* __restrict__ seg_begin,
                               uint32_t* __restrict__ seg_blk, uint32_t* __restrict__ blk_table) {
  __shared__ uint32_t sm[kBlock / 64];
  __shared__ uint32_t s_first[kBlock], s_nb[kBlock];
  uint32_t rec_run = 0, blk_run = 0;
  for (int f0 = 0; f0 < F; f0 += kBlock) {
    const int f = f0 + (int)threadIdx.x;
    int64_t a = 0, b = 0;
    if (f < F) {
      a = offsets[(int64_t)f * B], b = offsets[(int64_t)(f + 1) * B];
      a = a < 0 ? 0 : (a > nnz ? nnz : a);
      b = b < 0 ? 0 : (b > nnz ? nnz : b);
    }
    uint32_t total;
    const uint32_t begin = max(rec_run, dmt::block_inclusive_max<kBlock / 64>((uint32_t)a, sm, total));
    const uint32_t end = max(begin, (uint32_t)b);          // (the next table's begin)
    rec_run = max(rec_run, total);
    const uint32_t items = (uint32_t)table_items(end - begin, least_items);
    const uint32_t nb = (end - begin + items * kBlock - 1) / (items * kBlock);
    const uint32_t first = blk_run + dmt::block_exclusive_scan<kBlock / 64>(nb, sm, total);
    blk_run += total;
    if (f < F) {
      seg_begin[f] = begin;
      seg_blk[f] = first;
      if (f == F - 1) seg_begin[F] = end;
    }
    // the tables' block lists are written a wave per table, a block per lane
    s_first[threadIdx.x] = first;
    s_nb[threadIdx.x] = f < F ? nb << 4 | items : 0u;
    __syncthreads();
    for (int q = threadIdx.x >> 6; q < kBlock && f0 + q < F; q += kBlock / 64)
      for (uint32_t j = threadIdx.x & 63; j < s_nb[q] >> 4; j += 64)
        blk_table[s_first[q] + j] = (uint32_t)(f0 + q) << 4 | (s_nb[q] & 15);
    __syncthreads();
  }
  if (threadIdx.x == 0) seg_blk[F] = blk_run;
}

// Which sample each lookup belongs to: smp[j] = b for the lookups j of bag f*B + b.  The sort's first pass reads
// it beside `indices`.
// One block takes 2^log2_bpb consecutive bags and walks their lookups four at a time, so the work per
// thread does not depend on how the bag lengths are spread (a lane group per bag leaves most lanes
// idle when a few bags are hundreds of ids long and most hold one or two).  The bags' offsets go
// to LDS; a thread finds the bag of its first position by bisection there and goes on from it.
constexpr int kKeysMaxBags = 1024;
template <typename Sample>
__global__ __launch_bounds__(kBlock) void bwd_bag_samples(
    const int64_t* __restrict__ offsets, uint32_t B, uint32_t nbags, int64_t nnz, int F,
    Sample* __restrict__ smp, int log2_bpb, int least_items, uint32_t* __restrict__ seg_begin,
    uint32_t* __restrict__ seg_blk, uint32_t* __restrict__ blk_table,
    unsigned long long* __restrict__ err_offsets) {
  __shared__ uint32_t offs[kKeysMaxBags + 1];
  // (a block of its own, the first: with bags beside it, it was the last to end: 26 tables of 10 K lookups 5.6 -> 4.5 us)
  if (blockIdx.x == 0) {
    build_sort_map(offsets, B, F, nnz, least_items, seg_begin, seg_blk, blk_table);
    return;
  }
  const uint32_t g0 = (blockIdx.x - 1) << log2_bpb;
  if (g0 >= nbags) return;
  const int nb = (int)min((uint32_t)(1 << log2_bpb), nbags - g0);
  // `offsets` must tile [0, nnz): starts at 0, never descends, ends at nnz.  The first bag
  // that breaks this is recorded; the reduce and fix-up kernels then touch no row.
  for (int i = threadIdx.x; i <= nb; i += kBlock) {
    const int64_t o = offsets[g0 + i];
    const bool at_end = g0 + (uint32_t)i == nbags;
    if (o < 0 || o > nnz || (g0 + (uint32_t)i == 0 && o != 0) || (at_end && o != nnz))
      atomicMin(err_offsets, (unsigned long long)(g0 + i - (at_end ? 1 : 0)));
    offs[i] = (uint32_t)(o < 0 ? 0 : (o > nnz ? nnz : o));
  }
  __syncthreads();
  for (int i = threadIdx.x; i < nb; i += kBlock)
    if (offs[i] > offs[i + 1]) atomicMin(err_offsets, (unsigned long long)(g0 + i));
  const uint32_t s = offs[0], e = offs[nb], b0 = g0 % B;
  for (uint32_t j = (s & ~3u) + threadIdx.x * 4; j < e; j += kBlock * 4) {
    Sample v[4];
    int lo = 0;
    uint32_t end = 0;                              // of bag lo: offs[lo] <= at < end = offs[lo + 1]
#pragma unroll
    for (int u = 0; u < 4; ++u) {
      const uint32_t at = j + u;
      // most lookups lie in the bag of the one before or in the next
      if (at >= s && at < e && at >= end) {
        if (end != 0) end = offs[++lo + 1];
        if (at >= end) {
          int hi = nb;
          while (hi - lo > 1) {
            const int mid = (lo + hi) >> 1;
            if (offs[mid] <= at) lo = mid; else hi = mid;
          }
          end = offs[lo + 1];
        }
      }
      uint32_t b = b0 + (uint32_t)lo;
      if (b >= B) b = B > kKeysMaxBags ? b - B : b % B;
      v[u] = (Sample)b;
    }
    if (j >= s && j + 4 <= e) {
      struct alignas(4 * sizeof(Sample)) Four { Sample v[4]; };
      *(Four*)(smp + j) = Four{{v[0], v[1], v[2], v[3]}};
    } else {
#pragma unroll
      for (int u = 0; u < 4; ++u)
        if (j + u >= s && j + u < e) smp[j + u] = v[u];
    }
  }
}

// ------------------------------------------------------------------ radix sort

// Between its passes the sort keeps a lookup as a 32-bit row id inside its table and the sample (16 bits up to
// 65536 samples), in two arrays: the table is known from the position.  The counting kernels then read 4 bytes
// a lookup and the scatters move 6 each way, and the first pass reads `indices` as they lie.  Only the last pass
// writes the 64-bit records the reduce kernels walk.  Records of 8 bytes through all passes, built beforehand
// / now, us: 64 tables of 164 K lookups, 20 bits of row id: build 41 / samples 17, count 22 / 10-13, scatter 43 / 31-33
// a pass, the whole sort 253 / 165; 256 of 246 K, 20 bits: 1543 / 830; 128 of 170 K, 23 bits: 563 / 328.  The
// scatters are bound by their instructions (a wave's 64 lanes take four cycles each) as much as by bytes.
template <typename Sample>
struct SortIo {
  const int32_t* ids;            // first pass: the call's indices
  const uint32_t* key_in;        // other passes
  const Sample* smp_in;
  uint32_t* key_out;             // all passes but the last
  Sample* smp_out;
  uint64_t* pk_out;              // last pass
};

// A sort block's share of its table's records, and what its table decides.
struct SortBlock {
  uint32_t id, base, n, valid;   // its number, counted through the tables
  uint32_t table_base, at, nb;   // first record of the table; which of its nb sort blocks this is
  uint32_t f, rows, row_base;    // the table; its rows; its first global row id
  int64_t row_begin;             // id of its first row
  int items;                     // records per thread (narrow digits: kSortItems)
};
template <bool Wide>
__device__ __forceinline__ SortBlock sort_block(const DmtTableMeta* __restrict__ meta,
                                                const uint32_t* __restrict__ seg_begin,
                                                const uint32_t* __restrict__ seg_blk,
                                                const uint32_t* __restrict__ blk_table, int F) {
  SortBlock sb{};
  // Blocks are dealt to the XCDs (block id mod 8) so that neighbours in a table share an L2: a digit's records
  // come from all of a table's blocks, 16 of a block side by side, and the lines they share are put together
  // there (first scatter of 64 tables of 164 K lookups 46 -> 33 us, of 128 of 170 K 113 -> 71).
  const uint32_t nblk = seg_blk[F], per_xcd = (nblk + 7) / 8;
  sb.id = (blockIdx.x & 7) * per_xcd + (blockIdx.x >> 3);
  if ((blockIdx.x >> 3) >= per_xcd || sb.id >= nblk) return sb;
  const uint32_t packed = blk_table[sb.id], f = packed >> 4;
  sb.items = Wide ? (int)(packed & 15) : kSortItems;
  const uint32_t sort_tile = (uint32_t)(sb.items * kBlock);
  sb.table_base = seg_begin[f];
  sb.at = sb.id - seg_blk[f];
  sb.nb = seg_blk[f + 1] - seg_blk[f];
  sb.base = sb.table_base + sb.at * sort_tile;
  const uint32_t end = seg_begin[f + 1];
  sb.n = end - sb.base < sort_tile ? end - sb.base : sort_tile;
  sb.f = f;
  sb.rows = (uint32_t)meta[f].rows;
  sb.row_base = (uint32_t)meta[f].row_base;
  sb.row_begin = meta[f].row_begin;
  sb.valid = 1;
  return sb;
}

// The row inside the table, or one past its last row for an id outside it.
template <bool First, typename Sample>
__device__ __forceinline__ uint32_t sort_key(const SortIo<Sample>& io, const SortBlock& sb, uint32_t at) {
  if constexpr (First) {
    const int64_t local = (int64_t)io.ids[at] - sb.row_begin;
    return (uint64_t)local < (uint64_t)sb.rows ? (uint32_t)local : sb.rows;
  } else {
    return io.key_in[at];
  }
}

template <int MaxBits, bool First, typename Sample>
__global__ __launch_bounds__(kBlock) void radix_hist(
    const DmtTableMeta* __restrict__ meta, SortIo<Sample> io, int shift, int bits,
    uint32_t* __restrict__ hist, const uint32_t* __restrict__ seg_begin,
    const uint32_t* __restrict__ seg_blk, const uint32_t* __restrict__ blk_table, int F,
    unsigned long long* __restrict__ err) {
  constexpr int MaxRadix = 1 << MaxBits;
  __shared__ uint32_t h[MaxRadix];
  const SortBlock sb = sort_block<MaxBits == kWideRadixBits>(meta, seg_begin, seg_blk, blk_table, F);
  if (!sb.valid) return;
  for (int d = threadIdx.x; d < MaxRadix; d += kBlock) h[d] = 0;
  const uint32_t mask = (1u << bits) - 1;
  // (no load is conditional: the compiler would wait for each before the next)
  uint32_t key[kSortItems];
#pragma unroll
  for (int i = 0; i < kSortItems; ++i)
    key[i] = sort_key<First>(io, sb, sb.base + min((uint32_t)(i * kBlock + threadIdx.x), sb.n - 1));
  __syncthreads();
  const int lane = threadIdx.x & 63;
#pragma unroll
  for (int i = 0; i < kSortItems; ++i) {
    const uint32_t q = i * kBlock + threadIdx.x;
    const uint32_t d = (key[i] >> shift) & mask;
    if constexpr (First) {
      if (q < sb.n) {
        atomicAdd(&h[d], 1u);
        // (a row-wise shard passes over the ids of other shards silently: err is null then)
        if (err && key[i] == sb.rows) atomicMin(err, (unsigned long long)(sb.base + q));
      }
    } else {
      // behind the first pass the lookups of a frequent row lie side by side, and 64 lanes that add to one
      // counter take 64 turns: a run of equal digits is added by its first lane
      const uint32_t before = (uint32_t)__builtin_amdgcn_update_dpp(-1, (int)d, 0x138, 0xf, 0xf, false);   // wave_shr:1
      const uint64_t valid = __ballot(q < sb.n);
      const uint64_t ends = (__ballot(d != before) | ~valid) >> 1 >> lane;     // where the lanes behind this one start anew
      if (q < sb.n && d != before) atomicAdd(&h[d], ends ? (uint32_t)__ffsll((unsigned long long)ends) : 64u - lane);
    }
  }
  __syncthreads();
  for (int d = threadIdx.x; d < (1 << bits); d += kBlock)
    hist[(int64_t)sb.id * MaxRadix + d] = h[d];
}

// One block per table: turns the per-block digit counts of the table's sort blocks into the
// position of each block's first record of each digit in the sorted output (digit-major,
// block-minor inside the table's record range).  Thread (slice, digit) walks one slice of the
// table's blocks.
__global__ __launch_bounds__(kScanThreads) void radix_scan(uint32_t* __restrict__ hist, int bits,
                                                           const uint32_t* __restrict__ seg_begin,
                                                           const uint32_t* __restrict__ seg_blk) {
  __shared__ uint32_t tot[kScanThreads];
  __shared__ uint32_t dbase[kMaxRadix];
  __shared__ uint32_t sm[kScanThreads / 64];
  const int f = blockIdx.x;
  const uint32_t b0 = seg_blk[f], nb = seg_blk[f + 1] - b0;
  if (nb == 0) return;
  const int R = 1 << bits, slices = kScanThreads >> bits;
  const int sl = threadIdx.x >> bits, d = threadIdx.x & (R - 1);
  const uint32_t per = (nb + slices - 1) / slices;
  const uint32_t lo = min(nb, sl * per), hi = min(nb, lo + per);
  // (counts are read sixteen blocks at a time: one by one, every read would wait for the store
  // before it, which the compiler must assume may touch the same word)
  uint32_t run = 0;
  for (uint32_t b = lo; b < hi; b += kScanBatch) {
    uint32_t v[kScanBatch];
#pragma unroll
    for (int q = 0; q < kScanBatch; ++q)
      v[q] = b + q < hi ? hist[(int64_t)(b0 + b + q) * kMaxRadix + d] : 0u;
#pragma unroll
    for (int q = 0; q < kScanBatch; ++q) {
      if (b + q < hi) hist[(int64_t)(b0 + b + q) * kMaxRadix + d] = run;
      run += v[q];
    }
  }
  tot[threadIdx.x] = run;
  __syncthreads();
  uint32_t before = 0, all = 0;                    // this digit: earlier slices, every slice
  for (int q = 0; q < slices; ++q) {
    const uint32_t t = tot[q * R + d];
    if (q < sl) before += t;
    all += t;
  }
  uint32_t total;
  const uint32_t ex = dmt::block_exclusive_scan<kScanThreads / 64>(sl == 0 ? all : 0u, sm, total);
  if (sl == 0) dbase[d] = ex;
  __syncthreads();
  const uint32_t add = seg_begin[f] + dbase[d] + before;
  for (uint32_t b = lo; b < hi; b += kScanBatch) {
    uint32_t v[kScanBatch];
#pragma unroll
    for (int q = 0; q < kScanBatch; ++q)
      v[q] = b + q < hi ? hist[(int64_t)(b0 + b + q) * kMaxRadix + d] : 0u;
#pragma unroll
    for (int q = 0; q < kScanBatch; ++q)
      if (b + q < hi) hist[(int64_t)(b0 + b + q) * kMaxRadix + d] = v[q] + add;
  }
}

// Stable scatter of a sort block's records.  `hist` holds where the block's first record of each digit
// goes or, with OwnScan, the digit counts radix_hist left.
template <int MaxBits, bool OwnScan, bool First, bool Last, typename Sample>
__global__ __launch_bounds__(kBlock) void radix_scatter(
    const DmtTableMeta* __restrict__ meta, SortIo<Sample> io, int shift, int bits,
    const uint32_t* __restrict__ hist, const uint32_t* __restrict__ seg_begin,
    const uint32_t* __restrict__ seg_blk, const uint32_t* __restrict__ blk_table, int F, uint32_t B) {
  __shared__ uint32_t kbuf[kSortTile];
  __shared__ Sample sbuf[kSortTile];
  constexpr int MaxRadix = 1 << MaxBits, DPT = (MaxRadix + kBlock - 1) / kBlock;
  __shared__ uint32_t cnt[kBlock / 64][MaxRadix];
  __shared__ uint32_t gbase[MaxRadix];
  __shared__ uint32_t sm[8];
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int radix = 1 << bits;
  const uint32_t mask = (uint32_t)radix - 1;
  const SortBlock sb = sort_block<OwnScan>(meta, seg_begin, seg_blk, blk_table, F);
  if (!sb.valid) return;
  const int items = sb.items;
  const int n_tile = (int)sb.n;
  // (no load is conditional: the compiler would wait for each before the next)
  uint32_t key[kSortItems], smp[kSortItems], rank[kSortItems];
#pragma unroll
  for (int i = 0; i < kSortItems; ++i) {
    const uint32_t at = sb.base + (uint32_t)min(wave * (items * 64) + i * 64 + lane, n_tile - 1);
    key[i] = sort_key<First>(io, sb, at);
    smp[i] = io.smp_in[at];
  }
  for (int w = 0; w < kBlock / 64; ++w)
    for (int d = tid; d < MaxRadix; d += kBlock) cnt[w][d] = 0;
  __syncthreads();

  // stable rank of every record among the records of its wave with the same digit: first among the 64
  // records of its step (the lanes whose digit differs in no bit) ...
#pragma unroll
  for (int i = 0; i < kSortItems; ++i) {
    if (i >= items) break;
    const uint32_t d = (key[i] >> shift) & mask;
    const uint64_t valid = __ballot(wave * (items * 64) + i * 64 + lane < n_tile);
    uint32_t other_lo = ~(uint32_t)valid, other_hi = ~(uint32_t)(valid >> 32);
#pragma unroll
    for (int b = 0; b < MaxBits; ++b) {
      if (b >= bits) break;
      const uint32_t mine = (uint32_t)__builtin_amdgcn_sbfe((int)d, b, 1);     // all ones where the bit is set
      const uint64_t m = __ballot(mine != 0);
      other_lo |= (uint32_t)m ^ mine;
      other_hi |= (uint32_t)(m >> 32) ^ mine;
    }
    const uint32_t below = __builtin_amdgcn_mbcnt_hi(~other_hi, __builtin_amdgcn_mbcnt_lo(~other_lo, 0));
    rank[i] = below | (uint32_t)(__popc(~other_lo) + __popc(~other_hi)) << 8;
  }
  // ... then behind those of the steps before it.  The lanes of a wave read a digit's count before its first
  // lane raises it (LDS serves a wave in order).
  volatile __attribute__((address_space(3))) uint32_t* my_cnt =
      (volatile __attribute__((address_space(3))) uint32_t*)cnt[wave];
#pragma unroll
  for (int i = 0; i < kSortItems; ++i) {
    if (i >= items) break;
    const uint32_t d = (key[i] >> shift) & mask, below = rank[i] & 0xff;
    const uint32_t old = my_cnt[d];
    __builtin_amdgcn_wave_barrier();
    if (below == 0 && wave * (items * 64) + i * 64 + lane < n_tile) my_cnt[d] = old + (rank[i] >> 8);
    __builtin_amdgcn_wave_barrier();
    rank[i] = old + below;
  }
  __syncthreads();
  // thread t owns digits t*DPT .. t*DPT+DPT-1: totals over the waves
  uint32_t tot[DPT];
  uint32_t tsum = 0;
#pragma unroll
  for (int j = 0; j < DPT; ++j) {
    const int d = tid * DPT + j;
    tot[j] = 0;
    if (d < radix)
      for (int w = 0; w < kBlock / 64; ++w) tot[j] += cnt[w][d];
    tsum += tot[j];
  }
  uint32_t total;
  uint32_t goes[DPT];                              // where this block's first record of a digit goes
  if constexpr (OwnScan) {
    // records of the table with a smaller digit, and with this digit in earlier blocks
    static_assert(DPT == 4, "a thread reads its digits' counts as one uint4");
    uint4 all = make_uint4(0, 0, 0, 0), before = make_uint4(0, 0, 0, 0);
    if (tid * DPT < radix) {
      const uint4* __restrict__ h = (const uint4*)(hist + (int64_t)(sb.id - sb.at) * MaxRadix) + tid;
      for (uint32_t b = 0; b < sb.nb; b += kScanBatch) {
        uint4 v[kScanBatch];
#pragma unroll
        for (int q = 0; q < kScanBatch; ++q)
          v[q] = b + q < sb.nb ? h[(int64_t)(b + q) * (MaxRadix / 4)] : make_uint4(0, 0, 0, 0);
#pragma unroll
        for (int q = 0; q < kScanBatch; ++q) {
          if (b + q == sb.at) before = all;
          all.x += v[q].x; all.y += v[q].y; all.z += v[q].z; all.w += v[q].w;
        }
      }
    }
    const uint32_t a[DPT] = {all.x, all.y, all.z, all.w};
    const uint32_t bef[DPT] = {before.x, before.y, before.z, before.w};
    uint32_t sum = 0;
#pragma unroll
    for (int j = 0; j < DPT; ++j) sum += tid * DPT + j < radix ? a[j] : 0u;
    uint32_t at = sb.table_base + dmt::block_exclusive_scan<kBlock / 64>(sum, sm, total);
#pragma unroll
    for (int j = 0; j < DPT; ++j) {
      goes[j] = at + bef[j];
      at += a[j];
    }
  }
  // cnt becomes where each wave's first record of the digit lies in the block's sorted tile
  uint32_t ex = dmt::block_exclusive_scan<kBlock / 64>(tsum, sm, total);
#pragma unroll
  for (int j = 0; j < DPT; ++j) {
    const int d = tid * DPT + j;
    if (d < radix) {
      if constexpr (OwnScan) gbase[d] = goes[j] - ex;
      else gbase[d] = hist[(int64_t)sb.id * MaxRadix + d] - ex;
      uint32_t run = ex;
      for (int w = 0; w < kBlock / 64; ++w) {
        const uint32_t c = cnt[w][d];
        cnt[w][d] = run;
        run += c;
      }
    }
    ex += tot[j];
  }
  __syncthreads();
#pragma unroll
  for (int i = 0; i < kSortItems; ++i) {
    if (i >= items) break;
    if (wave * (items * 64) + i * 64 + lane < n_tile) {
      const uint32_t at = cnt[wave][(key[i] >> shift) & mask] + rank[i];
      kbuf[at] = key[i];
      sbuf[at] = (Sample)smp[i];
    }
  }
  __syncthreads();
  const uint32_t bag0 = sb.f * B;
#pragma unroll
  for (int i = 0; i < kSortItems; ++i) {
    const int q = i * kBlock + tid;
    if (q >= n_tile) break;
    const uint32_t k = kbuf[q], b = sbuf[q];
    const uint32_t to = gbase[(k >> shift) & mask] + (uint32_t)q;
    if constexpr (Last) {
      const uint32_t gid = (sb.row_base + k) | (k == sb.rows ? kInertBit : 0u);
      io.pk_out[to] = ((uint64_t)gid << 32) | (bag0 + b);
    } else {
      io.key_out[to] = k;
      io.smp_out[to] = (Sample)b;
    }
  }
}

// The whole sort of a call of few lookups in one launch, a block per table: each lookup's sample, the checks of
// `offsets`, and every pass over digits of up to 10 bits with the records in LDS.  Bound by the chain of its steps; the
// launches it takes the place of (samples, and two a pass) were bound by that and by their own starts.  A block's time
// grows with its table's lookups, whoever holds them, and the line (kSmallNnz) lies where one table that holds them all
// is no slower for it.  Whole update, us, several launches / one: 8 tables of 288 lookups, 1000 rows 23.6 / 16.3; 12 of
// 590, 20000 rows 33.5 / 20.4; 200 of 35 60.7 / 19.9; 7168 in one table, 1000 rows 29.4 / 27.5, 10^6 rows 34.8 / 31.0;
// past the line 16384 in one table 29.0 / 42.6 and 38.9 / 56.6, 8 of 2000 26.7 / 20.3.
constexpr int kSmallBlock = 1024, kSmallItems = (int)(kSmallNnz / kSmallBlock);
constexpr int kSmallWaves = kSmallBlock / 64, kSmallRadix = 1 << kWideRadixBits;
static_assert(kSmallRadix == kSmallBlock && kSmallItems * kSmallBlock == kSmallNnz && kSmallNnz < 65536 && kSmallBatch % 8 == 0, "");
constexpr int kSmallLds = (int)kSmallNnz * 6 + kSmallWaves * kSmallRadix * 2 + ((int)kSmallBatch + 8) * 2;
__global__ __launch_bounds__(kSmallBlock) void bwd_sort_small(
    const DmtTableMeta* __restrict__ meta, const int32_t* __restrict__ indices, const int64_t* __restrict__ offsets,
    uint32_t B, int F, int nnz, uint64_t* __restrict__ pk, unsigned long long* __restrict__ err,
    unsigned long long* __restrict__ err_offsets) {
  extern __shared__ __attribute__((aligned(16))) uint32_t kbuf[];          // [kSmallNnz]
  uint16_t* const sbuf = (uint16_t*)(kbuf + kSmallNnz);                     // [kSmallNnz]
  uint16_t* const cnt = sbuf + kSmallNnz;                                   // [wave][digit]
  uint16_t* const offs = cnt + kSmallWaves * kSmallRadix;                   // [B + 1]
  __shared__ uint32_t sm[kSmallWaves];
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6, f = blockIdx.x;
  const uint32_t g0 = (uint32_t)f * B;
  // (as in bwd_bag_samples)
  for (uint32_t i = tid; i <= B; i += kSmallBlock) {
    const int64_t o = offsets[g0 + i];
    const bool at_end = f == F - 1 && i == B;
    if (o < 0 || o > nnz || (g0 + i == 0 && o != 0) || (at_end && o != nnz))
      atomicMin(err_offsets, (unsigned long long)(g0 + i - (at_end ? 1 : 0)));
    offs[i] = (uint16_t)(o < 0 ? 0 : (o > nnz ? nnz : o));
  }
  const DmtTableMeta& m = meta[f];
  const uint32_t rows = (uint32_t)m.rows, row_base = (uint32_t)m.row_base;
  const int64_t row_begin = m.row_begin;
  int bits_all = 1;
  while ((1ull << bits_all) < (uint64_t)rows + 1) ++bits_all;
  const int passes = (bits_all + kWideRadixBits - 1) / kWideRadixBits, bits = (bits_all + passes - 1) / passes;
  __syncthreads();
  for (uint32_t i = tid; i < B; i += kSmallBlock)
    if (offs[i] > offs[i + 1]) atomicMin(err_offsets, (unsigned long long)(g0 + i));
  const int first = offs[0], n = (int)offs[B] - first;
  if (n <= 0) return;
  const int items = (n + kSmallBlock - 1) / kSmallBlock, q0 = wave * (items * 64) + lane;      // this lane's first record
  uint32_t key[kSmallItems], smp[kSmallItems], rank[kSmallItems];
#pragma unroll
  for (int i = 0; i < kSmallItems; ++i) {
    if (i >= items) break;
    key[i] = (uint32_t)indices[first + min(q0 + i * 64, n - 1)];
  }
  // Samples: a bag leaves its number (and one) with its first lookup, a lookup takes the last one left up to it.
  for (int q = tid; q < n; q += kSmallBlock) sbuf[q] = 0;
  __syncthreads();
  for (uint32_t i = tid; i < B; i += kSmallBlock) {
    const int at = (int)offs[i] - first;
    if (offs[i] < offs[i + 1] && at >= 0 && at < n) sbuf[at] = (uint16_t)(i + 1);
  }
  uint32_t last = 0, past = B;                     // of the wave's first record: offs[last] <= it < offs[past]
  const int from = first + min(wave * (items * 64), n - 1);
  while (past - last > 1) {
    const uint32_t mid = (last + past) >> 1;
    if (offs[mid] <= from) last = mid; else past = mid;
  }
  __syncthreads();
#pragma unroll
  for (int i = 0; i < kSmallItems; ++i) {
    if (i >= items) break;
    const int q = q0 + i * 64;
    const uint32_t left = q < n ? sbuf[q] : 0u;
    const uint64_t marks = __ballot(left != 0), upto = marks & (~0ull >> (63 - lane));
    const uint32_t mine = (uint32_t)__shfl((int)left, upto ? 63 - __clzll((long long)upto) : 0);
    smp[i] = upto ? mine - 1 : last;
    last = (uint32_t)__shfl((int)smp[i], 63);
    const int64_t local = (int64_t)(int32_t)key[i] - row_begin;
    key[i] = (uint64_t)local < (uint64_t)rows ? (uint32_t)local : rows;
    if (err && q < n && key[i] == rows) atomicMin(err, (unsigned long long)(first + q));
  }
  volatile __attribute__((address_space(3))) uint16_t* const my_cnt =
      (volatile __attribute__((address_space(3))) uint16_t*)(cnt + wave * kSmallRadix);
  for (int p = 0; p < passes; ++p) {
    const int shift = p * bits;
    for (int i = tid; i < kSmallWaves * kSmallRadix / 8; i += kSmallBlock) ((uint4*)cnt)[i] = make_uint4(0, 0, 0, 0);
    __syncthreads();
    // (ranks as in radix_scatter)
#pragma unroll
    for (int i = 0; i < kSmallItems; ++i) {
      if (i >= items) break;
      const uint32_t d = key[i] >> shift & ((1u << bits) - 1);
      const bool valid = q0 + i * 64 < n;
      const uint64_t v = __ballot(valid);
      uint32_t other_lo = ~(uint32_t)v, other_hi = ~(uint32_t)(v >> 32);
#pragma unroll
      for (int b = 0; b < kWideRadixBits; ++b) {
        if (b >= bits) break;
        const uint32_t mine = (uint32_t)__builtin_amdgcn_sbfe((int)d, b, 1);
        const uint64_t same = __ballot(mine != 0);
        other_lo |= (uint32_t)same ^ mine;
        other_hi |= (uint32_t)(same >> 32) ^ mine;
      }
      const uint32_t below = __builtin_amdgcn_mbcnt_hi(~other_hi, __builtin_amdgcn_mbcnt_lo(~other_lo, 0));
      const uint32_t old = my_cnt[d];
      __builtin_amdgcn_wave_barrier();
      if (below == 0 && valid) my_cnt[d] = (uint16_t)(old + __popc(~other_lo) + __popc(~other_hi));
      __builtin_amdgcn_wave_barrier();
      rank[i] = old + below;
    }
    __syncthreads();
    // a thread owns a digit: each wave's first record of it
    uint32_t sum = 0, total;
#pragma unroll
    for (int w = 0; w < kSmallWaves; ++w) sum += cnt[w * kSmallRadix + tid];
    uint32_t run = dmt::block_exclusive_scan<kSmallWaves>(sum, sm, total);
#pragma unroll
    for (int w = 0; w < kSmallWaves; ++w) {
      const uint32_t c = cnt[w * kSmallRadix + tid];
      cnt[w * kSmallRadix + tid] = (uint16_t)run;
      run += c;
    }
    __syncthreads();
#pragma unroll
    for (int i = 0; i < kSmallItems; ++i) {
      if (i >= items) break;
      if (q0 + i * 64 < n) {
        const uint32_t at = cnt[wave * kSmallRadix + (key[i] >> shift & ((1u << bits) - 1))] + rank[i];
        kbuf[at] = key[i];
        sbuf[at] = (uint16_t)smp[i];
      }
    }
    __syncthreads();
    if (p + 1 == passes) break;
#pragma unroll
    for (int i = 0; i < kSmallItems; ++i) {
      if (i >= items) break;
      const int q = min(q0 + i * 64, n - 1);
      key[i] = kbuf[q];
      smp[i] = sbuf[q];
    }
  }
  for (int q = tid; q < n; q += kSmallBlock) {
    const uint32_t k = kbuf[q];
    pk[first + q] = (uint64_t)((row_base + k) | (k == rows ? kInertBit : 0u)) << 32 | (g0 + sbuf[q]);
  }
}

// ------------------------------------------------- run heads, segment offsets

// Run-head flags of the 1024 consecutive records a wave owns inside its block's
// tile, as 16 ballots (iteration i covers records i*64 .. i*64+63, one per lane,
// so every load is one coalesced 512-byte line set).  Returns the head count.
__device__ __forceinline__ uint32_t wave_head_ballots(const uint64_t* __restrict__ pk, int64_t nnz,
                                                      int64_t wave_base,
                                                      uint64_t (&ballots)[kScanItems]) {
  const int lane = threadIdx.x & 63;
  uint32_t count = 0;
  uint32_t carry = 0;                                  // key of the record before this iteration
  if (wave_base > 0 && wave_base <= nnz) carry = (uint32_t)(pk[wave_base - 1] >> 32);
#pragma unroll
  for (int i = 0; i < kScanItems; ++i) {
    const int64_t p = wave_base + i * 64 + lane;
    const uint32_t k = p < nnz ? (uint32_t)(pk[p] >> 32) : 0;
    uint32_t prev = __shfl_up(k, 1);
    if (lane == 0) prev = carry;
    const bool head = p < nnz && (p == 0 || k != prev) && !(k & kInertBit);
    ballots[i] = __ballot(head);
    count += (uint32_t)__popcll(ballots[i]);
    carry = __shfl(k, 63);
  }
  return count;
}

__global__ __launch_bounds__(kBlock) void heads_count(const uint64_t* __restrict__ pk, int64_t nnz,
                                                      uint32_t* __restrict__ blk_heads) {
  __shared__ uint32_t sm[kBlock / 64];
  const int wave = threadIdx.x >> 6;
  uint64_t ballots[kScanItems];
  const uint32_t c = wave_head_ballots(
      pk, nnz, (int64_t)blockIdx.x * kScanTile + (int64_t)wave * (kScanItems * 64), ballots);
  if ((threadIdx.x & 63) == 0) sm[wave] = c;
  __syncthreads();
  if (threadIdx.x == 0) {
    uint32_t t = 0;
    for (int w = 0; w < kBlock / 64; ++w) t += sm[w];
    blk_heads[blockIdx.x] = t;
  }
}

// Single block: exclusive scan of the per-block head counts; total = number of
// distinct keys (the inert key, if present, is counted and removed by the caller
// of num_unique through `has_inert`).
__global__ __launch_bounds__(1024) void heads_scan(uint32_t* __restrict__ blk_heads, int64_t nblk,
                                                   uint32_t* __restrict__ num_unique) {
  __shared__ uint32_t sm[32];
  uint32_t running = 0;
  for (int64_t base = 0; base < nblk; base += 1024) {
    const int64_t i = base + threadIdx.x;
    const uint32_t v = i < nblk ? blk_heads[i] : 0;
    uint32_t total;
    const uint32_t ex = dmt::block_exclusive_scan<16>(v, sm, total);
    if (i < nblk) blk_heads[i] = running + ex;
    running += total;
  }
  if (threadIdx.x == 0) num_unique[0] = running;
}

__global__ __launch_bounds__(kBlock) void heads_write(
    const uint64_t* __restrict__ pk, int64_t nnz, const uint32_t* __restrict__ blk_heads,
    uint32_t* __restrict__ seg_off) {
  __shared__ uint32_t sm[kBlock / 64];
  const int wave = threadIdx.x >> 6, lane = threadIdx.x & 63;
  const int64_t wave_base = (int64_t)blockIdx.x * kScanTile + (int64_t)wave * (kScanItems * 64);
  uint64_t ballots[kScanItems];
  const uint32_t c = wave_head_ballots(pk, nnz, wave_base, ballots);
  if (lane == 0) sm[wave] = c;
  __syncthreads();
  uint32_t before = blk_heads[blockIdx.x];              // run heads before this wave's records
  for (int w = 0; w < wave; ++w) before += sm[w];
  const uint64_t lt = (1ULL << lane) - 1;
#pragma unroll
  for (int i = 0; i < kScanItems; ++i) {
    const int64_t p = wave_base + i * 64 + lane;
    const uint32_t mine = before + (uint32_t)__popcll(ballots[i] & lt);   // heads before p
    const bool head = (ballots[i] >> lane) & 1;
    if (p < nnz) {
      if (head) seg_off[mine] = (uint32_t)p;
      if (p == nnz - 1) seg_off[mine + (head ? 1 : 0)] = (uint32_t)nnz;
    }
    before += (uint32_t)__popcll(ballots[i]);
  }
}

// ------------------------------------------- segment reduce + rowwise Adagrad

// A lane's four columns of a table row.
template <int TD> struct RowChunk { using type = uint2; static constexpr int bytes = 8; };
template <> struct RowChunk<DMT_F32> { using type = float4; static constexpr int bytes = 16; };

// One rowwise-Adagrad step on row `row` of table f, requested (the row and its state are on their way while the
// gradient is summed) and applied with the summed gradient g.  The group's lanes hold 4 consecutive columns each; lanes
// past D hold zeros.
template <int TD>
struct RowUpdate {
  typename RowChunk<TD>::type* at;
  typename RowChunk<TD>::type w;
  float* state;
  float st;
  int D;
  bool on;
  __device__ __forceinline__ void request(const DmtTableMeta& m, uint32_t row, int gl) {
    D = m.D;
    on = gl * 4 < D;
    at = (typename RowChunk<TD>::type*)((char*)m.table + (int64_t)row * D * (RowChunk<TD>::bytes / 4)) + (on ? gl : 0);
    state = m.state + row;
    w = dmt::gload(at);
    st = dmt::gload(state);
  }
  __device__ __forceinline__ void apply(float4 g, int gl, int GL, float lr, float eps) const {
    float ss = g.x * g.x + g.y * g.y + g.z * g.z + g.w * g.w;
    for (int o = 1; o < GL; o <<= 1) ss += __shfl_xor(ss, o);
    const float sn = st + ss / (float)D;
    const float step = lr / (sqrtf(sn) + eps);
    if (on) {
      if constexpr (TD == DMT_F32) {
        float4 v = w;
        v.x -= step * g.x; v.y -= step * g.y; v.z -= step * g.z; v.w -= step * g.w;
        dmt::gstore(v, at);
      } else {
        float a, b, c, d;
        dmt::unpack2<TD>(w.x, a, b);
        dmt::unpack2<TD>(w.y, c, d);
        a -= step * g.x; b -= step * g.y; c -= step * g.z; d -= step * g.w;
        dmt::gstore(make_uint2(dmt::pack2<TD>(a, b), dmt::pack2<TD>(c, d)), at);
      }
    }
    if (gl == 0) dmt::gstore(sn, state);
  }
};

__device__ __forceinline__ void store_partial(float* __restrict__ partials, int64_t slot,
                                              int Dmax, int gl, float4 g) {
  if (gl * 4 < Dmax) *((float4*)(partials + slot * Dmax) + gl) = g;
}

// Sum of v over the 2^LG lanes of an aligned lane group; every lane gets the
// total.  Data-parallel-primitive moves inside a 16-lane row, a swizzle across
// rows, a permute across the two 32-lane halves.
template <int LG>
__device__ __forceinline__ float group_sum(float v) {
  auto dpp = [](float x, auto ctrl) {
    return __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(x), decltype(ctrl)::value,
                                                      0xf, 0xf, true));
  };
  if constexpr (LG >= 1) v += dpp(v, std::integral_constant<int, 0xB1>());   // quad_perm [1,0,3,2]
  if constexpr (LG >= 2) v += dpp(v, std::integral_constant<int, 0x4E>());   // quad_perm [2,3,0,1]
  if constexpr (LG >= 3) v += dpp(v, std::integral_constant<int, 0x141>());  // row_half_mirror
  if constexpr (LG >= 4) v += dpp(v, std::integral_constant<int, 0x140>());  // row_mirror
  if constexpr (LG >= 5)
    v += __int_as_float(__builtin_amdgcn_ds_swizzle(__float_as_int(v), 0x401F));  // lane ^ 16
  if constexpr (LG >= 6) v += __shfl_xor(v, 32);
  return v;
}

// Orders one lane's LDS writes before other lanes' reads of them inside a wave.  The lanes of
// a wave run in lockstep, but to the compiler they are unrelated threads: without this it may
// move a lane's read in front of another lane's write.
__device__ __forceinline__ void wave_lds_sync() {
  __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
  __builtin_amdgcn_wave_barrier();
  __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

#ifndef DMT_QS
#define DMT_QS 5
#endif
constexpr int kQueueSlots = DMT_QS;
// finished runs parked before their rows are updated: per lane group, and per wave of the
// wave-per-tile kernel (whose slots are half as large)
constexpr int kQueueSlotsWave = 8;
constexpr int kWaveUnroll = 6;                   // gradient rows the wave-per-tile kernel requests at once
static_assert(kReduceUnroll <= kQueueSlots && kWaveUnroll <= kQueueSlotsWave,
              "a step of the walk parks at most as many runs as the queue holds");

// Each group of GL = 2^LG lanes walks one tile of `tile` sorted records,
// summing the bags' gradient slices run by run (float32, record order).  Runs
// that lie wholly inside the tile are parked in an LDS queue (their gradient
// sum, row and state address); the queue is drained four rows at a time, so the
// row / state reads of four updates are in flight together instead of one
// dependent read per run.  The piece of a run that continues from the previous
// tile goes to partial slot 2t, the piece of a run that starts here and
// continues into the next tile to slot 2t + 1.
// UD: every table has dim Dmax (no per-record width to pass round).
template <int TD, int LG, bool UD>
__global__ __launch_bounds__(kBlock) void bwd_reduce_update(
    const DmtTableMeta* __restrict__ meta, const uint64_t* __restrict__ pk, int64_t nnz, uint32_t B,
    uint32_t nbags, uint32_t total_rows, const float* __restrict__ grad,
    float* __restrict__ partials, int Dmax, int tile, int64_t ntiles, int64_t blocks_per_xcd, float lr,
    float eps, const unsigned long long* __restrict__ err_offsets) {
  if (*err_offsets != ~0ULL) return;              // malformed offsets: the records mean nothing
  constexpr int GL = 1 << LG, NG = kBlock >> LG;
  constexpr int eb = TD == DMT_F32 ? 4 : 2;
  using Chunk = typename RowChunk<TD>::type;
  __shared__ float4 q_g[kQueueSlots][kBlock];
  __shared__ unsigned long long q_rowp[NG][kQueueSlots];
  __shared__ unsigned long long q_stp[NG][kQueueSlots];
  __shared__ int q_D[NG][kQueueSlots];

  const int group = threadIdx.x >> LG;
  const int64_t tb = (int64_t)(blockIdx.x & 7) * blocks_per_xcd + (blockIdx.x >> 3);
  const int64_t t = tb * NG + group;
  const bool live = t < ntiles;                 // dead groups still take part in wave votes
  const int lane = threadIdx.x & 63;
  const int gl = threadIdx.x & (GL - 1);
  const int lane0 = lane & ~(GL - 1);
  const bool lane_on = gl * 4 < Dmax;
  const float4* __restrict__ grad4 = (const float4*)grad;

  int64_t p0 = 0;
  int n = 0;
  bool cont_prev = false, cont_next = false;
  uint32_t carry = 0;
  if (live) {
    p0 = t * tile;
    n = (int)min((int64_t)tile, nnz - p0);
    const uint32_t first_key = (uint32_t)(pk[p0] >> 32);
    if (p0 > 0) {
      carry = (uint32_t)(pk[p0 - 1] >> 32);
      cont_prev = carry == first_key;
    }
    cont_next = p0 + n < nnz && (uint32_t)(pk[p0 + n - 1] >> 32) == (uint32_t)(pk[p0 + n] >> 32);
  }
  bool has_prev = p0 > 0;
  bool run_open = cont_prev, from_left = cont_prev;
  float4 acc = make_float4(0.f, 0.f, 0.f, 0.f);
  unsigned long long cur_rowp = 0, cur_stp = 0;
  int cur_D = Dmax;
  bool cur_ok = false;
  int qn = 0;

  auto park = [&]() {                            // the open run is complete: queue its update
    if (cur_ok) {
      q_g[qn][threadIdx.x] = acc;
      q_rowp[group][qn] = cur_rowp;
      q_stp[group][qn] = cur_stp;
      if (!UD) q_D[group][qn] = cur_D;
      ++qn;
    }
  };
  auto drain = [&]() {
#pragma unroll
    for (int j0 = 0; j0 < kQueueSlots; j0 += 4) {
      if (!__any(j0 < qn)) break;
      Chunk w[4];
      float st[4];
      Chunk* wp[4];
      float* sp[4];
      int D[4];
#pragma unroll
      for (int u = 0; u < 4; ++u) {
        if (j0 + u < qn && j0 + u < kQueueSlots) {
          D[u] = UD ? Dmax : q_D[group][j0 + u];
          wp[u] = (Chunk*)(q_rowp[group][j0 + u]) + gl;
          sp[u] = (float*)(q_stp[group][j0 + u]);
          st[u] = dmt::gload(sp[u]);
          if (gl * 4 < D[u]) w[u] = dmt::gload(wp[u]);
        }
      }
#pragma unroll
      for (int u = 0; u < 4; ++u) {
        if (j0 + u < qn && j0 + u < kQueueSlots) {
          const float4 g = q_g[j0 + u][threadIdx.x];
          const float ss = group_sum<LG>(g.x * g.x + g.y * g.y + g.z * g.z + g.w * g.w);
          const float sn = st[u] + ss * __builtin_amdgcn_rcpf((float)D[u]);
          const float step = lr * __builtin_amdgcn_rcpf(__builtin_amdgcn_sqrtf(sn) + eps);
          if (gl * 4 < D[u]) {
            if constexpr (TD == DMT_F32) {
              float4 v = w[u];
              v.x -= step * g.x; v.y -= step * g.y; v.z -= step * g.z; v.w -= step * g.w;
              dmt::gstore(v, wp[u]);
            } else {
              float a, b, c, d;
              dmt::unpack2<TD>(w[u].x, a, b);
              dmt::unpack2<TD>(w[u].y, c, d);
              a -= step * g.x; b -= step * g.y; c -= step * g.z; d -= step * g.w;
              dmt::gstore(make_uint2(dmt::pack2<TD>(a, b), dmt::pack2<TD>(c, d)), wp[u]);
            }
          }
          if (gl == 0) dmt::gstore(sn, sp[u]);
        }
      }
    }
    qn = 0;
  };

  for (int sub = 0; sub < tile; sub += GL) {
    const int cnt = min(GL, n - sub);            // <= 0 once this group's tile is done
    if (!__any(cnt > 0)) break;
    // every lane prepares its own record: gradient offset, row and state address
    uint32_t key_l = total_rows, goff4_l = 0xffffffffu;
    unsigned long long rowp_l = 0, stp_l = 0;
    int D_l = 0;
    if (gl < cnt) {
      const uint64_t r = pk[p0 + sub + gl];
      const uint32_t k = (uint32_t)(r >> 32), bag = (uint32_t)r;
      if (k < total_rows && bag < nbags) {
        const uint32_t f = bag / B, b = bag - f * B;
        const DmtTableMeta& m = meta[f];
        const int64_t row = (int64_t)k - m.row_base;
        if (row >= 0 && row < m.rows) {            // key and bag agree on the table
          key_l = k;
          D_l = m.D;
          goff4_l = (uint32_t)(((int64_t)B * m.out_prefix + (int64_t)b * m.tower_width + m.col_off) >> 2);
          rowp_l = (unsigned long long)((const char*)m.table + row * D_l * eb);
          stp_l = (unsigned long long)(m.state + row);
        }
      }
    }
    // run heads of this sub-round as a bit mask, one bit per record
    uint32_t prev = __shfl_up(key_l, 1, GL);
    bool head_l = gl < cnt;
    if (gl == 0) head_l = head_l && (!has_prev || key_l != carry);
    else head_l = head_l && key_l != prev;
    const unsigned long long hm = __ballot(head_l);
    const unsigned long long gm = LG == 6 ? hm : ((hm >> lane0) & ((1ULL << (GL & 63)) - 1));
    if (cnt > 0) {
      carry = __shfl(key_l, lane0 + cnt - 1);
      has_prev = true;
    }

    for (int i0 = 0; i0 < GL; i0 += kReduceUnroll) {
      if (!__any(i0 < cnt)) break;
      float4 g[kReduceUnroll];
#pragma unroll
      for (int u = 0; u < kReduceUnroll; ++u) {
        const int src = lane0 + ((i0 + u) & (GL - 1));
        const uint32_t go = __shfl(goff4_l, src);
        // (every lane takes part in the exchange: a lane that is off would hand out nothing,
        // and the lanes past the widest row hold records like any other)
        const int D_src = UD ? Dmax : __shfl(D_l, src);
        const bool on = lane_on && i0 + u < cnt && go != 0xffffffffu && gl * 4 < D_src;
        g[u] = make_float4(0.f, 0.f, 0.f, 0.f);
        if (on) g[u] = grad4[(size_t)go + gl];
      }
#pragma unroll
      for (int u = 0; u < kReduceUnroll; ++u) {
        const int i = i0 + u;
        const int src = lane0 + (i & (GL - 1));
        if (i < cnt) {
          if ((gm >> i) & 1) {                     // a run starts at this record
            if (run_open) {
              if (from_left) store_partial(partials, 2 * t, Dmax, gl, acc);
              else park();
            }
            from_left = false;
            run_open = true;
            acc = make_float4(0.f, 0.f, 0.f, 0.f);
            cur_rowp = __shfl(rowp_l, src);
            cur_stp = __shfl(stp_l, src);
            cur_ok = __shfl(key_l, src) < total_rows;
            if (!UD) cur_D = __shfl(D_l, src);
          }
          acc.x += g[u].x; acc.y += g[u].y; acc.z += g[u].z; acc.w += g[u].w;
        }
      }
      if (__any(qn > kQueueSlots - kReduceUnroll)) drain();
    }
  }
  if (run_open) {
    if (from_left) store_partial(partials, 2 * t, Dmax, gl, acc);
    else if (cont_next) { if (cur_ok) store_partial(partials, 2 * t + 1, Dmax, gl, acc); }
    else park();
  }
  drain();
}

// The same tile walk for wide rows (64 < Dmax <= 256), one WAVE per tile: the 64
// lanes hold EPL = Dmax/64 columns each, so every per-record decision (run head,
// tile end, queue state) is wave-uniform and lives in scalar registers: record
// fields are fetched with v_readlane instead of ds_bpermute, branches are
// scalar, and the two half-waves never diverge.  Same queue-and-drain scheme,
// same partial-slot protocol, same float32 summation order as bwd_reduce_update.
template <int EPL> struct LaneVec;
template <> struct LaneVec<1> { using type = float; };
template <> struct LaneVec<2> { using type = float2; };
template <> struct LaneVec<4> { using type = float4; };

template <int EPL> __device__ __forceinline__ void lv_zero(typename LaneVec<EPL>::type& a) {
  if constexpr (EPL == 1) a = 0.f;
  else if constexpr (EPL == 2) a = make_float2(0.f, 0.f);
  else a = make_float4(0.f, 0.f, 0.f, 0.f);
}
template <int EPL>
__device__ __forceinline__ void lv_add(typename LaneVec<EPL>::type& a,
                                       const typename LaneVec<EPL>::type& b) {
  if constexpr (EPL == 1) a += b;
  else if constexpr (EPL == 2) { a.x += b.x; a.y += b.y; }
  else { a.x += b.x; a.y += b.y; a.z += b.z; a.w += b.w; }
}
template <int EPL> __device__ __forceinline__ float lv_sumsq(const typename LaneVec<EPL>::type& a) {
  if constexpr (EPL == 1) return a * a;
  else if constexpr (EPL == 2) return a.x * a.x + a.y * a.y;
  else return a.x * a.x + a.y * a.y + a.z * a.z + a.w * a.w;
}

// row[lane*EPL .. +EPL) -= step * g, in the table's element type
template <int TD, int EPL>
__device__ __forceinline__ void lane_row_update(void* rowp, int lane,
                                                const typename LaneVec<EPL>::type& g, float step,
                                                const void* loaded) {
  if constexpr (TD == DMT_F32) {
    using V = typename LaneVec<EPL>::type;
    V v = *(const V*)loaded;
    if constexpr (EPL == 1) v -= step * g;
    else if constexpr (EPL == 2) { v.x -= step * g.x; v.y -= step * g.y; }
    else { v.x -= step * g.x; v.y -= step * g.y; v.z -= step * g.z; v.w -= step * g.w; }
    dmt::gstore(v, (V*)rowp + lane);
  } else if constexpr (EPL == 1) {
    const uint16_t u = *(const uint16_t*)loaded;
    float a = TD == DMT_F16 ? dmt::f16_bits_to_f32(u) : dmt::bf16_lo(u);
    a -= step * g;
    dmt::gstore((uint16_t)(TD == DMT_F16 ? dmt::f32_to_f16_bits(a) : dmt::f32_to_bf16_bits(a)),
                (uint16_t*)rowp + lane);
  } else if constexpr (EPL == 2) {
    float a, b;
    dmt::unpack2<TD>(*(const uint32_t*)loaded, a, b);
    a -= step * g.x; b -= step * g.y;
    dmt::gstore(dmt::pack2<TD>(a, b), (uint32_t*)rowp + lane);
  } else {
    const uint2 u = *(const uint2*)loaded;
    float a, b, c, d;
    dmt::unpack2<TD>(u.x, a, b);
    dmt::unpack2<TD>(u.y, c, d);
    a -= step * g.x; b -= step * g.y; c -= step * g.z; d -= step * g.w;
    dmt::gstore(make_uint2(dmt::pack2<TD>(a, b), dmt::pack2<TD>(c, d)), (uint2*)rowp + lane);
  }
}

template <int TD, int EPL> struct LaneChunk {            // a lane's EPL elements of a table row
  using type = typename LaneVec<EPL>::type;
};
template <int EPL> struct LaneChunk<DMT_F16, EPL> {
  using type = std::conditional_t<EPL == 1, uint16_t, std::conditional_t<EPL == 2, uint32_t, uint2>>;
};
template <int EPL> struct LaneChunk<DMT_BF16, EPL> {
  using type = typename LaneChunk<DMT_F16, EPL>::type;
};

__device__ __forceinline__ unsigned long long readlane64(unsigned long long v, int l) {
  const uint32_t lo = __builtin_amdgcn_readlane((uint32_t)v, l);
  const uint32_t hi = __builtin_amdgcn_readlane((uint32_t)(v >> 32), l);
  return ((unsigned long long)hi << 32) | lo;
}

template <int TD, int EPL, bool UD>
__global__ __launch_bounds__(kBlock) void bwd_reduce_update_wave(
    const DmtTableMeta* __restrict__ meta, const uint64_t* __restrict__ pk, int64_t nnz, uint32_t B,
    uint32_t nbags, uint32_t total_rows, const float* __restrict__ grad,
    float* __restrict__ partials, int Dmax, int tile, int64_t ntiles, int64_t blocks_per_xcd, float lr,
    float eps, const unsigned long long* __restrict__ err_offsets) {
  if (*err_offsets != ~0ULL) return;              // malformed offsets: the records mean nothing
  constexpr int NW = kBlock / 64;
  constexpr int eb = TD == DMT_F32 ? 4 : 2;
  using Vec = typename LaneVec<EPL>::type;
  using Chunk = typename LaneChunk<TD, EPL>::type;
  __shared__ Vec q_g[kQueueSlotsWave][kBlock];
  __shared__ unsigned long long q_rowp[NW][kQueueSlotsWave + 1];
  __shared__ unsigned long long q_stp[NW][kQueueSlotsWave + 1];
  __shared__ int q_D[NW][kQueueSlotsWave + 1];

  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int lane = threadIdx.x & 63;
  const int64_t tb = (int64_t)(blockIdx.x & 7) * blocks_per_xcd + (blockIdx.x >> 3);
  const int64_t t = tb * NW + wave;
  if (t >= ntiles) return;
  const bool lane_on = lane * EPL < Dmax;
  const Vec* __restrict__ gradv = (const Vec*)grad;

  const int64_t p0 = t * tile;
  const int n = (int)min((int64_t)tile, nnz - p0);
  const uint32_t first_key = __builtin_amdgcn_readfirstlane((uint32_t)(pk[p0] >> 32));
  uint32_t carry = 0;
  bool cont_prev = false;
  if (p0 > 0) {
    carry = __builtin_amdgcn_readfirstlane((uint32_t)(pk[p0 - 1] >> 32));
    cont_prev = carry == first_key;
  }
  bool cont_next = false;
  if (p0 + n < nnz)
    cont_next = __builtin_amdgcn_readfirstlane((uint32_t)(pk[p0 + n - 1] >> 32)) ==
                __builtin_amdgcn_readfirstlane((uint32_t)(pk[p0 + n] >> 32));
  bool has_prev = p0 > 0;
  bool run_open = cont_prev, from_left = cont_prev;
  Vec acc;
  lv_zero<EPL>(acc);
  bool cur_ok = false;
  int qn = 0;

  auto store_part = [&](int64_t slot) {
    if (lane_on) ((Vec*)(partials + slot * Dmax))[lane] = acc;
  };
  // the open run's row / state address sit in queue slot qn already (its head lane put
  // them there); parking adds the gradient sum and commits the slot
  auto park = [&]() {
    if (cur_ok) {
      q_g[qn][threadIdx.x] = acc;
      ++qn;
    }
  };
  auto drain = [&]() {
    const int open_slot = qn;                      // may hold the open run's addresses
    wave_lds_sync();                               // the head lanes' addresses, the parked sums
    if constexpr (EPL == 2) {
      // two parked rows per step: lanes 0-31 take one, lanes 32-63 the next (4 columns a lane)
      using Chunk2 = typename RowChunk<TD>::type;
      const int half = lane >> 5, hl = lane & 31;
#pragma unroll
      for (int j0 = 0; j0 < kQueueSlotsWave; j0 += 8) {
        if (j0 >= qn) break;
        Chunk2 w[4];
        float st[4];
        Chunk2* wp[4];
        float* sp[4];
        int D[4];
#pragma unroll
        for (int u = 0; u < 4; ++u) {
          const int j = j0 + 2 * u + half;
          if (j < qn && j < kQueueSlotsWave) {
            D[u] = UD ? Dmax : q_D[wave][j];
            wp[u] = (Chunk2*)q_rowp[wave][j] + hl;
            sp[u] = (float*)q_stp[wave][j];
            // row and state are touched once per call: keep them from evicting gradient slices
            st[u] = dmt::nt_load(sp[u]);
            if (hl * 4 < D[u]) w[u] = dmt::nt_load(wp[u]);
          }
        }
#pragma unroll
        for (int u = 0; u < 4; ++u) {
          const int j = j0 + 2 * u + half;
          if (j < qn && j < kQueueSlotsWave) {
            const float4 g = ((const float4*)&q_g[j][wave * 64])[hl];
            const float ss = group_sum<5>(g.x * g.x + g.y * g.y + g.z * g.z + g.w * g.w);
            const float sn = st[u] + ss * __builtin_amdgcn_rcpf((float)D[u]);
            const float step = lr * __builtin_amdgcn_rcpf(__builtin_amdgcn_sqrtf(sn) + eps);
            if (hl * 4 < D[u]) {
              if constexpr (TD == DMT_F32) {
                float4 v = w[u];
                v.x -= step * g.x; v.y -= step * g.y; v.z -= step * g.z; v.w -= step * g.w;
                dmt::nt_store(v, wp[u]);
              } else {
                float a, b, c, d;
                dmt::unpack2<TD>(w[u].x, a, b);
                dmt::unpack2<TD>(w[u].y, c, d);
                a -= step * g.x; b -= step * g.y; c -= step * g.z; d -= step * g.w;
                dmt::nt_store(make_uint2(dmt::pack2<TD>(a, b), dmt::pack2<TD>(c, d)), wp[u]);
              }
            }
            if (hl == 0) dmt::nt_store(sn, sp[u]);
          }
        }
      }
    } else {
#pragma unroll
      for (int j0 = 0; j0 < kQueueSlotsWave; j0 += 4) {
        if (j0 >= qn) break;
        Chunk w[4];
        float st[4];
        void* wp[4];
        float* sp[4];
        int D[4];
#pragma unroll
        for (int u = 0; u < 4; ++u) {
          if (j0 + u < qn && j0 + u < kQueueSlotsWave) {
            D[u] = UD ? Dmax : __builtin_amdgcn_readfirstlane(q_D[wave][j0 + u]);
            wp[u] = (void*)q_rowp[wave][j0 + u];
            sp[u] = (float*)q_stp[wave][j0 + u];
            st[u] = dmt::gload(sp[u]);
            if (lane * EPL < D[u]) w[u] = dmt::gload((const Chunk*)wp[u] + lane);
          }
        }
#pragma unroll
        for (int u = 0; u < 4; ++u) {
          if (j0 + u < qn && j0 + u < kQueueSlotsWave) {
            const Vec g = q_g[j0 + u][threadIdx.x];
            float ss = group_sum<5>(lv_sumsq<EPL>(g));
            ss = __int_as_float(__builtin_amdgcn_readlane(__float_as_int(ss), 0)) +
                 __int_as_float(__builtin_amdgcn_readlane(__float_as_int(ss), 32));
            const float sn = st[u] + ss * __builtin_amdgcn_rcpf((float)D[u]);
            const float step = lr * __builtin_amdgcn_rcpf(__builtin_amdgcn_sqrtf(sn) + eps);
            if (lane * EPL < D[u]) lane_row_update<TD, EPL>(wp[u], lane, g, step, &w[u]);
            if (lane == 0) dmt::gstore(sn, sp[u]);
          }
        }
      }
    }
    wave_lds_sync();                               // every lane is done reading the slots
    // an open run keeps its addresses: move them to the slot it will be parked in now
    if (open_slot > 0 && open_slot < kQueueSlotsWave + 1 && run_open && !from_left && lane == 0) {
      q_rowp[wave][0] = q_rowp[wave][open_slot];
      q_stp[wave][0] = q_stp[wave][open_slot];
      if (!UD) q_D[wave][0] = q_D[wave][open_slot];
    }
    qn = 0;
  };

  for (int sub = 0; sub < n; sub += 64) {
    const int cnt = min(64, n - sub);
    uint32_t key_l = total_rows, goff_l = 0xffffffffu;
    unsigned long long rowp_l = 0, stp_l = 0;
    int D_l = 0;
    if (lane < cnt) {
      const uint64_t r = pk[p0 + sub + lane];
      const uint32_t k = (uint32_t)(r >> 32), bag = (uint32_t)r;
      if (k < total_rows && bag < nbags) {
        const uint32_t f = bag / B, b = bag - f * B;
        const DmtTableMeta& m = meta[f];
        const int64_t row = (int64_t)k - m.row_base;
        if (row >= 0 && row < m.rows) {            // key and bag agree on the table
          key_l = k;
          D_l = m.D;
          goff_l = (uint32_t)(((int64_t)B * m.out_prefix + (int64_t)b * m.tower_width + m.col_off) >> 2);
          rowp_l = (unsigned long long)((const char*)m.table + row * D_l * eb);
          stp_l = (unsigned long long)(m.state + row);
        }
      }
    }
    uint32_t prev = __shfl_up(key_l, 1);
    bool head_l = lane < cnt;
    if (lane == 0) head_l = head_l && (!has_prev || key_l != carry);
    else head_l = head_l && key_l != prev;
    const unsigned long long hm = __ballot(head_l);
    carry = __builtin_amdgcn_readlane(key_l, cnt - 1);
    has_prev = true;

    for (int i0 = 0; i0 < cnt; i0 += kWaveUnroll) {
      Vec g[kWaveUnroll];
#pragma unroll
      for (int u = 0; u < kWaveUnroll; ++u) {
        lv_zero<EPL>(g[u]);
        if (i0 + u < cnt) {
          const uint32_t go = __builtin_amdgcn_readlane(goff_l, i0 + u);
          bool on = lane_on && go != 0xffffffffu;
          if (!UD) on = on && lane * EPL < __builtin_amdgcn_readlane(D_l, i0 + u);
          if (on) g[u] = gradv[((size_t)go << 2) / EPL + lane];
        }
      }
#pragma unroll
      for (int u = 0; u < kWaveUnroll; ++u) {
        const int i = i0 + u;
        if (i < cnt) {
          if ((hm >> i) & 1) {                     // a run starts at this record
            if (run_open) {
              if (from_left) store_part(2 * t);
              else park();
            }
            from_left = false;
            run_open = true;
            lv_zero<EPL>(acc);
            cur_ok = __builtin_amdgcn_readlane(key_l, i) < total_rows;
            if (lane == i) {                         // the head record's lane knows the row
              q_rowp[wave][qn] = rowp_l;
              q_stp[wave][qn] = stp_l;
              if (!UD) q_D[wave][qn] = D_l;
            }
          }
          lv_add<EPL>(acc, g[u]);
        }
      }
      if (qn > kQueueSlotsWave - kWaveUnroll) drain();
    }
  }
  if (run_open) {
    if (from_left) store_part(2 * t);
    else if (cont_next) { if (cur_ok) store_part(2 * t + 1); }
    else park();
  }
  drain();
}

// The tile walk for rows of at most 128 columns, built to spend as few instructions per sorted
// record as the hardware allows and to keep a wave's row updates off its critical path.
//  * One wave per tile of `tile` records.  A tile is cut into chunks of up to 64
//    consecutive records of ONE table, one record per lane (two chunks, more only where the
//    tile straddles a table boundary), so everything a table decides (row width, gradient
//    base, row and state base) sits in scalar registers.
//  * Each lane reads one record and the record after it; "my key differs from the next one"
//    is one ballot, the mask of run TAILS.  Nothing else about runs is ever computed.
//  * The walk proper is, per record: one v_readlane (its gradient offset), one buffer load of
//    the slice (two columns per lane), two adds, one scalar bit test.  kLeanBatch slices are
//    requested together.
//  * At a tail the sum is parked in a ring of 8 LDS slots, and the lane number of the tail
//    record is packed into a scalar register.  Row updates come off the ring four at a time,
//    ONE instruction for four rows (16 lanes a row, 8 columns a lane), in two halves: at a
//    batch boundary the rows and states of the four oldest parked runs are REQUESTED (the
//    row's key comes from the tail record's lane by ds_bpermute, the addresses from the
//    chunk's scalars); the walk goes on, and at the next boundary the update is computed and
//    stored.  The requests are older than the next batch's slices and the memory counter
//    retires in order, so the wave waits once for both instead of once for each.
//  * Same partial-slot protocol and the same float32 summation order as the other walks.
constexpr int kLeanQueue = 8;
constexpr int kLeanGroup = 4;                    // rows updated by one instruction
constexpr int kLeanBatch = 8;                    // gradient slices requested together
static_assert(kLeanBatch <= kLeanQueue && 64 % kLeanBatch == 0,
              "every record of a batch may end a run, and all of them must fit the emptied ring");

// One wave per block: the waves of a block share nothing, and a block's slots are only handed
// on when its slowest wave is done.  Tile times spread widely (per-tile timestamps on Mid:
// 27 us at the 10th percentile, 73 at the 90th), so with four waves a block a third of the
// wave slots sat waiting for a sibling.  Filling them makes every tile slower instead (mean
// 48 -> 55 us: the gathers, not the number of waves, bound the kernel) and the launch 1 %
// faster.
constexpr int kLeanBlock = 64;
template <int TD>
__global__ __launch_bounds__(kLeanBlock) void bwd_reduce_update_lean(
    const DmtTableMeta* __restrict__ meta, const uint64_t* __restrict__ pk, int64_t nnz, uint32_t B,
    uint32_t bag_mul, uint32_t bag_shift, uint32_t F, const float* __restrict__ grad,
    float* __restrict__ partials, int Dmax, int tile, int64_t ntiles, int64_t blocks_per_xcd, float lr,
    float eps, const unsigned long long* __restrict__ err_offsets) {
  if (*err_offsets != ~0ULL) return;              // malformed offsets: the records mean nothing
  constexpr int NW = kLeanBlock / 64;
  constexpr int eb = TD == DMT_F32 ? 4 : 2;
  using Chunk = std::conditional_t<TD == DMT_F32, float4, uint4>;
  constexpr int NC = TD == DMT_F32 ? 2 : 1;
  __shared__ float q_g[NW][kLeanQueue][128];

  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int lane = threadIdx.x & 63;
  const int64_t tb = (int64_t)(blockIdx.x & 7) * blocks_per_xcd + (blockIdx.x >> 3);
  const int64_t t = tb * NW + wave;
  if (t >= ntiles) return;
  const int64_t p0 = t * tile;
  const int n = (int)min((int64_t)tile, nnz - p0);
  const int qd = lane >> 4, ql = lane & 15;        // row updates: quarter-wave qd, 8 columns from 8 ql
  float* const qbase = &q_g[wave][0][0];

  uint32_t from_left = 0;                          // the open run began in an earlier tile
  if (p0 > 0)
    from_left = __builtin_amdgcn_readfirstlane((uint32_t)(pk[p0 - 1] >> 32)) ==
                __builtin_amdgcn_readfirstlane((uint32_t)(pk[p0] >> 32));
  bool open_end = false;                           // the last record's run goes on in the next tile
  int last_D = 0;
  float2 acc = make_float2(0.f, 0.f);
  // the ring: runs parked, runs whose row and state are requested, runs updated (P >= I >= C,
  // P - C <= 8, I - C <= 4); run e lives in slot e & 7, byte e & 7 of qcodes is 4 x the lane
  // of its tail record
  uint32_t P = 0, I = 0, C = 0;
  uint64_t qcodes = 0;

  for (int pos = 0; pos < n;) {
    const int nrem = n - pos;
    const int64_t idx = p0 + pos + lane;
    uint64_t rec = ~0ULL;
    if (lane < nrem) rec = __builtin_nontemporal_load(pk + idx);
    const uint32_t key_l = (uint32_t)(rec >> 32), bag_l = (uint32_t)rec;
    // the key after each record: the next lane's, and for the last of the (up to) 64 records
    // read here the key of the record behind them, one scalar load
    const int nread = min(nrem, 64);
    const int64_t behind = p0 + pos + nread;
    uint32_t key_behind = ~key_l;                  // differs: the last record of all ends its run
    if (behind < nnz) key_behind = __builtin_amdgcn_readfirstlane((uint32_t)(pk[behind] >> 32));
    const uint32_t down = (uint32_t)__shfl_down((int)key_l, 1);
    const uint32_t next_key_l = lane == nread - 1 ? key_behind : down;
    const uint32_t f_l = B == 1 ? bag_l : (__umulhi(bag_l, bag_mul) >> bag_shift);   // bag / B
    const uint32_t f = __builtin_amdgcn_readfirstlane(f_l);
    const int cnt = __popcll(__ballot(lane < nrem && f_l == f));   // records sorted by table: a prefix
    if (f >= F) {                                  // not a record the sort wrote
      acc = make_float2(0.f, 0.f);
      from_left = 0;
      open_end = false;
      pos += cnt;
      continue;
    }
    const DmtTableMeta& m = meta[f];
    const int D = m.D;
    const uint32_t row_base = (uint32_t)m.row_base, rows = (uint32_t)m.rows;
    const char* const table = (const char*)m.table;
    float* const state = m.state;
    const uint32_t rowbytes = (uint32_t)D * eb;
    const char* const gbase = (const char*)(grad + (int64_t)B * m.out_prefix + m.col_off);
    const uint32_t tw4 = (uint32_t)m.tower_width * 4u;
    // (lanes past the chunk name sample 0's slice: every readlane below yields a valid offset)
    const uint32_t boff_l = lane < cnt ? (bag_l - f * B) * tw4 : 0u;
    const bool in_l = lane < cnt && (key_l - row_base) < rows;     // a row of this table
    const bool tail_l = in_l && next_key_l != key_l;
    const uint64_t tm = __ballot(tail_l);
    const bool last_in = (__ballot(in_l) >> (cnt - 1)) & 1;
    const bool lane_on = lane * 2 < D;
    // lanes past the row's width read the row's first columns instead (every load stays
    // unconditional and in bounds) and park zeros
    const uint32_t lane_off = lane_on ? (uint32_t)lane * 8u : 0u;
    const bool col_on = ql * 8 < D, col_hi = ql * 8 + 4 < D;
    const float inv_D = __builtin_amdgcn_rcpf((float)D);

    // rows and states requested for runs C .. I - 1, one run per quarter-wave
    Chunk pw[NC];
    float pst = 0.f;
    uint32_t prow = 0;
    // Requests the row and the state of runs I .. I + g - 1 (g <= 4).  No load is conditional:
    // a quarter-wave with no run, and lanes past the row's width, read row 0 / the row's
    // first columns.
    auto request = [&](uint32_t g) {
      const uint32_t slot = (I + qd) & 7u;
      const uint32_t code = (uint32_t)(qcodes >> (slot * 8)) & 0xffu;
      const uint32_t k = (uint32_t)__builtin_amdgcn_ds_bpermute((int)code, (int)key_l);
      prow = (uint32_t)qd < g ? k - row_base : 0u;
      const char* wp = table + (uint64_t)prow * rowbytes + (col_on ? ql * (8 * eb) : 0);
      pst = dmt::nt_load(state + prow);
      if constexpr (TD == DMT_F32) {
        pw[0] = dmt::nt_load((const float4*)wp);
        pw[1] = dmt::nt_load((const float4*)wp + (col_hi ? 1 : 0));
      } else {
        pw[0] = dmt::nt_load((const uint4*)wp);
      }
      I += g;
    };
    // Updates the rows requested last: runs C .. I - 1.
    auto update = [&]() {
      const bool on = (uint32_t)qd < I - C;
      wave_lds_sync();                             // the parked sums
      const float4* gq = (const float4*)(qbase + ((C + qd) & 7u) * 128 + ql * 8);
      const float4 g0 = gq[0], g1 = gq[1];
      float ss = g0.x * g0.x + g0.y * g0.y + g0.z * g0.z + g0.w * g0.w + g1.x * g1.x +
                 g1.y * g1.y + g1.z * g1.z + g1.w * g1.w;
      ss = group_sum<4>(ss);
      const float sn = pst + ss * inv_D;
      const float step = lr * __builtin_amdgcn_rcpf(__builtin_amdgcn_sqrtf(sn) + eps);
      char* wp = (char*)table + (uint64_t)prow * rowbytes + (col_on ? ql * (8 * eb) : 0);
      if constexpr (TD == DMT_F32) {
        float4 v = pw[0];
        v.x -= step * g0.x; v.y -= step * g0.y; v.z -= step * g0.z; v.w -= step * g0.w;
        if (on && col_on) dmt::nt_store(v, (float4*)wp);
        v = pw[1];
        v.x -= step * g1.x; v.y -= step * g1.y; v.z -= step * g1.z; v.w -= step * g1.w;
        if (on && col_hi) dmt::nt_store(v, (float4*)wp + 1);
      } else {
        float a, b, c, d;
        uint4 o;
        dmt::unpack2<TD>(pw[0].x, a, b);
        dmt::unpack2<TD>(pw[0].y, c, d);
        a -= step * g0.x; b -= step * g0.y; c -= step * g0.z; d -= step * g0.w;
        o.x = dmt::pack2<TD>(a, b);
        o.y = dmt::pack2<TD>(c, d);
        dmt::unpack2<TD>(pw[0].z, a, b);
        dmt::unpack2<TD>(pw[0].w, c, d);
        a -= step * g1.x; b -= step * g1.y; c -= step * g1.z; d -= step * g1.w;
        o.z = dmt::pack2<TD>(a, b);
        o.w = dmt::pack2<TD>(c, d);
        if (on && col_on) dmt::nt_store(o, (uint4*)wp);
      }
      if (on && ql == 0) dmt::nt_store(sn, state + prow);
      wave_lds_sync();                             // every lane is done reading the slots
      C = I;
    };
    // the run that ends at record i of this chunk is complete
    auto close_run = [&](int i) {
      const float2 a = lane_on ? acc : make_float2(0.f, 0.f);
      if (from_left != 0) {
        if (lane * 2 < Dmax) ((float2*)(partials + 2 * t * Dmax))[lane] = a;
        from_left = 0;
      } else {
        const uint32_t sh = (P & 7u) * 8u;
        ((float2*)(qbase + (sh << 4)))[lane] = a;
        qcodes = (qcodes & ~(0xffULL << sh)) | ((uint64_t)(uint32_t)(i * 4) << sh);
        ++P;
      }
      acc = make_float2(0.f, 0.f);
    };
    // This lane's two columns of record i's gradient, as a buffer load: the table's column
    // block is the buffer, the lane's column offset the vector offset and the record's row
    // offset the scalar offset, so a record costs no address arithmetic beyond its v_readlane
    // (and a read past the block would return zeros instead of faulting).
    const __amdgpu_buffer_rsrc_t gbuf = __builtin_amdgcn_make_buffer_rsrc(
        (void*)gbase, 0, (int)((B - 1) * tw4 + (uint32_t)D * 4u), 0x00020000);
    auto slice = [&](int i) {
      const uint32_t bo = __builtin_amdgcn_readlane(boff_l, i);
      const dmt::dmt_u32x2 v = __builtin_amdgcn_raw_buffer_load_b64(gbuf, (int)lane_off, (int)bo, 0);
      return make_float2(__uint_as_float(v.x), __uint_as_float(v.y));
    };

    // Parked runs name lanes of this chunk's key_l and live on its scalars, so the ring is
    // empty when the chunk is left.
    for (int i0 = 0;; i0 += kLeanBatch) {
      const bool more = i0 < cnt;
      const uint32_t tails = (uint32_t)(tm >> (i0 & 63)) & ((1u << kLeanBatch) - 1);
      // what was requested at the last boundary has had a batch's time to arrive
      if (I != C) update();
      // room for this batch's tails (seldom short), or everything out at the chunk's end
      while (more ? P - C + __popc(tails) > (uint32_t)kLeanQueue : P != C) {
        request(min(P - I, (uint32_t)kLeanGroup));
        update();
      }
      if (!more) break;
      if (P - I >= (uint32_t)kLeanGroup) request(kLeanGroup);
      float2 g[kLeanBatch];
      if (i0 + kLeanBatch <= cnt) {
#pragma unroll
        for (int u = 0; u < kLeanBatch; ++u) g[u] = slice(i0 + u);
#pragma unroll
        for (int u = 0; u < kLeanBatch; ++u) {
          acc.x += g[u].x;
          acc.y += g[u].y;
          if ((tails >> u) & 1) close_run(i0 + u);
        }
      } else {
#pragma unroll
        for (int u = 0; u < kLeanBatch; ++u) g[u] = slice((i0 + u) & 63);
#pragma unroll
        for (int u = 0; u < kLeanBatch; ++u) {
          if (i0 + u < cnt) {
            acc.x += g[u].x;
            acc.y += g[u].y;
            if ((tails >> u) & 1) close_run(i0 + u);
          }
        }
      }
    }
    open_end = last_in && !((tm >> (cnt - 1)) & 1);
    last_D = D;
    if (!last_in) {                                // ids outside the table end its records: nothing to carry
      acc = make_float2(0.f, 0.f);
      from_left = 0;
    }
    pos += cnt;
  }
  // (the last chunk's table decides which lanes hold columns; the others hold what they read
  // in place of them and store zeros)
  if (open_end && lane * 2 < Dmax)
    ((float2*)(partials + (2 * t + (from_left ? 0 : 1)) * Dmax))[lane] =
        lane * 2 < last_D ? acc : make_float2(0.f, 0.f);
}

// Table that owns global row id `gid` (row_base has F + 1 ascending entries).
__device__ __forceinline__ uint32_t table_of(const int64_t* __restrict__ row_base, int F,
                                             uint32_t gid) {
  int lo = 0, hi = F;                      // row_base[lo] <= gid < row_base[hi]
  while (hi - lo > 1) {
    const int mid = (lo + hi) >> 1;
    if ((int64_t)gid >= row_base[mid]) lo = mid; else hi = mid;
  }
  return (uint32_t)lo;
}

// Rows whose run crosses tile boundaries: the group of the tile where the run
// starts adds the pieces in tile order and applies the update.
// one wave per block: groups are independent, and the group at the head of a long run works
// far longer than its neighbours (50.7 -> 47.4 us on Mid)
//
// Small calls (Small): their tiles are smaller, so a row of many lookups has up to eight times the
// pieces, and one group would take eight times the memory latencies (eight pieces each).  A run of
// more than kLongRun tiles there is left to a block of its own, kLongGroups groups that share the
// pieces and add their sums in group order: no more latencies than tiles of 128 records have.  One
// such block stands ready for every kLongRun tiles and ends after two records if no long run
// has its first multiple of kLongRun tiles there.  Whole call, us, with tiles of 128 / smaller tiles
// and one group / now: one row of 131072 lookups, 128 columns 148 / 700 / 131; of 16384 64 / 110 / 36; two
// rows of 65536, 64 columns 93 / 367 / 80; 26 tables, half of them of 2 to 24 rows, 104156 lookups 114 / 67 / 61.
constexpr int kFixBlock = 64, kLongRun = 64, kLongGroups = 8, kLongBlock = kLongGroups * 64;
template <int TD, bool Small>
__global__ __launch_bounds__(Small ? kLongBlock : kFixBlock) void bwd_fixup_update(
    const DmtTableMeta* __restrict__ meta, uint32_t B, uint32_t nbags,
    const uint64_t* __restrict__ pk, int64_t nnz, uint32_t total_rows,
    const float* __restrict__ partials, int Dmax, int log2_gl, int tile, int64_t ntiles, int nlong, float lr,
    float eps, const unsigned long long* __restrict__ err_offsets) {
  if (*err_offsets != ~0ULL) return;
  const int GL = 1 << log2_gl, NG = (int)(blockDim.x >> log2_gl);
  const int grp = threadIdx.x >> log2_gl, gl = threadIdx.x & (GL - 1);
  const bool on = gl * 4 < Dmax;
  auto head_piece = [&](int64_t t0) -> float4 {
    return on ? *((const float4*)(partials + (2 * t0 + 1) * Dmax) + gl) : make_float4(0.f, 0.f, 0.f, 0.f);
  };
  // acc + the pieces of tiles first .. first + 7, of the eight `stride` tiles on, ... up to t1
  auto add_pieces = [&](float4 acc, int64_t first, int64_t t1, int stride) -> float4 {
    for (int64_t tt = first; tt <= t1; tt += stride) {
      float4 g[8];
#pragma unroll
      for (int q = 0; q < 8; ++q) {
        g[q] = make_float4(0.f, 0.f, 0.f, 0.f);
        if (on && tt + q <= t1) g[q] = *((const float4*)(partials + 2 * (tt + q) * Dmax) + gl);
      }
#pragma unroll
      for (int q = 0; q < 8; ++q) {
        acc.x += g[q].x; acc.y += g[q].y; acc.z += g[q].z; acc.w += g[q].w;
      }
    }
    return acc;
  };
  // The row of a run, from its key and (no search through the row bases) the bag of any of its records.
  uint32_t f = 0;
  int64_t row = 0;
  auto find_row = [&](uint64_t rec) -> bool {
    const uint32_t key = (uint32_t)(rec >> 32), bag = (uint32_t)rec;
    if (key >= total_rows || bag >= nbags) return false;
    f = bag / B;
    row = (int64_t)key - meta[f].row_base;
    return row >= 0 && row < meta[f].rows;         // key and bag disagree: not a row to touch
  };
  if constexpr (Small) {
    if ((int)blockIdx.x < nlong) {
      // (every wave finds the same: the block stays together)
      const int64_t m = ((int64_t)blockIdx.x + 1) * kLongRun;
      const int lane = threadIdx.x & 63;
      const uint64_t rec = pk[m * tile], before = pk[m * tile - 1];
      const uint32_t key = (uint32_t)(rec >> 32);
      if (key != (uint32_t)(before >> 32) || !find_row(rec)) return;
      // tiles m, m - 1, ... that start with the key (the keys are sorted), up to kLongRun of them
      const int back = __popcll(__ballot((uint32_t)(pk[(m - lane) * tile] >> 32) == key));
      const int64_t first = m - back + 1;
      const int64_t t0 = (uint32_t)(pk[first * tile - 1] >> 32) == key ? first - 1 : first;
      if (t0 > 0 && t0 == m - kLongRun && (uint32_t)(pk[t0 * tile] >> 32) == key &&
          (uint32_t)(pk[t0 * tile - 1] >> 32) == key)
        return;                                    // starts further back: another block's
      int64_t t1 = m, hi = ntiles;                 // holds at t1, fails at hi
      while (hi - t1 > 1) {
        const int64_t step = (hi - t1 + 63) / 64, at = t1 + (lane + 1) * step;
        const int n = __popcll(__ballot(at < hi && (uint32_t)(pk[min(at, ntiles - 1) * tile] >> 32) == key));
        hi = min(hi, t1 + (n + 1) * step);
        t1 += n * step;
      }
      if (t1 - t0 <= kLongRun) return;             // its group adds it up
      __shared__ float4 sums[kLongBlock];
      RowUpdate<TD> update;
      update.request(meta[f], (uint32_t)row, gl);
      sums[threadIdx.x] = add_pieces(make_float4(0.f, 0.f, 0.f, 0.f), t0 + 1 + grp * 8, t1, NG * 8);
      __syncthreads();
      if (grp > 0) return;
      float4 acc = head_piece(t0);
      for (int q = 0; q < NG; ++q) {
        const float4 g = sums[(q << log2_gl) + gl];
        acc.x += g.x; acc.y += g.y; acc.z += g.z; acc.w += g.w;
      }
      update.apply(acc, gl, GL, lr, eps);
      return;
    }
  }
  const int64_t t0 = (int64_t)(blockIdx.x - (Small ? nlong : 0)) * NG + grp;
  if (t0 >= ntiles - 1) return;
  const int64_t p0 = t0 * tile, p1 = p0 + tile;    // p1 < nnz here
  // (the records the decisions below look at are requested together: their latencies would otherwise follow one
  // another in every group; and so the row, its state, the run's first piece and the next tile's, which are wanted
  // whenever there is a run to add up: 64 tables of 164 K lookups 44.5 -> 41.6 us, 26 of 10 K 11.7 -> 11.0, 8 of 288 4.5 ->
  // 3.7)
  const bool third = t0 + 2 < ntiles;
  const uint64_t r_last = pk[p1 - 1], r_next = pk[p1], r_first = pk[p0], r_before = pk[p0 > 0 ? p0 - 1 : 0],
                 r_third = pk[third ? p1 + tile : p1];
  const uint32_t k_last = (uint32_t)(r_last >> 32);
  if (k_last != (uint32_t)(r_next >> 32) || !find_row(r_last)) return;
  const uint32_t k_first = (uint32_t)(r_first >> 32);
  if (k_first == k_last && p0 > 0 && (uint32_t)(r_before >> 32) == k_first) return;
  RowUpdate<TD> update;
  update.request(meta[f], (uint32_t)row, gl);
  float4 acc = head_piece(t0);
  const float4 second = on ? *((const float4*)(partials + 2 * (t0 + 1) * Dmax) + gl) : make_float4(0.f, 0.f, 0.f, 0.f);
  // last tile the run reaches: the largest t with the run's key at the tile's first record
  // (gallop first: most runs end within a tile or two)
  int64_t t1 = t0 + 1, hi = ntiles;               // holds at t1, fails at hi
  if (third && (uint32_t)(r_third >> 32) != k_last) hi = t0 + 2;
  for (int64_t step = 1; t1 + step < hi; step <<= 1) {
    if ((uint32_t)(pk[(t1 + step) * tile] >> 32) == k_last) t1 += step;
    else { hi = t1 + step; break; }
    if (Small && t1 - t0 > kLongRun) return;
  }
  while (hi - t1 > 1) {
    const int64_t mid = (t1 + hi) >> 1;
    if ((uint32_t)(pk[mid * tile] >> 32) == k_last) t1 = mid; else hi = mid;
  }
  if (Small && t1 - t0 > kLongRun) return;
  acc.x += second.x; acc.y += second.y; acc.z += second.z; acc.w += second.w;
  update.apply(add_pieces(acc, t0 + 2, t1, 8), gl, GL, lr, eps);
}

// ------------------------------------------------------------- parity exports

__global__ __launch_bounds__(kBlock) void bwd_export(
    const int64_t* __restrict__ row_base, int F, const uint64_t* __restrict__ pk, int64_t nnz,
    uint32_t total_rows, const uint32_t* __restrict__ seg_off,
    const uint32_t* __restrict__ num_unique_in, int64_t* __restrict__ sorted_keys,
    int32_t* __restrict__ sorted_bag, int64_t* __restrict__ unique_keys,
    int64_t* __restrict__ seg_off_out, int64_t* __restrict__ num_unique) {
  const int64_t i = (int64_t)blockIdx.x * kBlock + threadIdx.x;
  const uint32_t U = nnz > 0 ? num_unique_in[0] : 0;   // inert keys were not counted as heads
  if (i == 0 && num_unique) num_unique[0] = U;
  if (i < nnz) {
    const uint32_t gid = (uint32_t)(pk[i] >> 32);
    int64_t key = -1;
    if (gid < total_rows) {
      const uint32_t f = table_of(row_base, F, gid);
      key = ((int64_t)f << 32) | (int64_t)(gid - (uint32_t)row_base[f]);
    }
    if (sorted_keys) sorted_keys[i] = key;
    if (sorted_bag) sorted_bag[i] = (int32_t)(uint32_t)pk[i];
  }
  if (i <= U) {
    if (seg_off_out) seg_off_out[i] = nnz > 0 ? (int64_t)seg_off[i] : 0;
    if (i < U && unique_keys) {
      const uint32_t gid = (uint32_t)(pk[seg_off[i]] >> 32);
      const uint32_t f = table_of(row_base, F, gid);
      unique_keys[i] = ((int64_t)f << 32) | (int64_t)(gid - (uint32_t)row_base[f]);
    }
  }
}

int ilog2_ceil(int64_t x) {
  int l = 0;
  while ((1LL << l) < x) ++l;
  return l;
}

// One launch on `s`, bracketed by the plan's timing events when that kernel family is selected.
template <typename Kernel, typename... Args>
void timed_launch(const dmt_plan* plan, dmt_kernel_id id, hipStream_t s, Kernel kernel,
                  int64_t blocks, int threads, Args... args) {
  DmtScope scope(plan, id, s);
  hipLaunchKernelGGL(kernel, dim3((unsigned)blocks), dim3((unsigned)threads), 0, s, args...);
}

// What the sort's launches share.
struct SortCall {
  const dmt_plan* plan;
  const BwdWs* w;
  const int32_t* indices;
  const int64_t* offsets;
  int64_t nnz, B;
  uint32_t nbags;
  int log2_bpb;
  int64_t key_blocks;
  hipStream_t s;
};

template <int MaxBits, bool First, bool Last, typename Sample>
void launch_sort_pass(const SortCall& c, const SortIo<Sample>& io, int shift, int bits) {
  constexpr bool Wide = MaxBits == kWideRadixBits;
  const BwdWs& w = *c.w;
  const dmt_plan* plan = c.plan;
  const int64_t blocks = (w.nblk_sort + 7) / 8 * 8;     // as many for every XCD
  timed_launch(plan, DMT_K_BWD_SORT_HIST, c.s, radix_hist<MaxBits, First, Sample>, blocks, kBlock, plan->d_meta, io, shift,
               bits, w.hist, w.seg_begin, w.seg_blk, w.blk_table, (int)plan->F,
               plan->row_shards ? nullptr : plan->d_error);
  if (!Wide)
    timed_launch(plan, DMT_K_BWD_SORT_SCAN, c.s, radix_scan, plan->F, kScanThreads, w.hist, bits, w.seg_begin, w.seg_blk);
  timed_launch(plan, DMT_K_BWD_SORT_SCATTER, c.s, radix_scatter<MaxBits, Wide, First, Last, Sample>, blocks, kBlock,
               plan->d_meta, io, shift, bits, w.hist, w.seg_begin, w.seg_blk, w.blk_table, (int)plan->F, (uint32_t)c.B);
}

// Stable LSD radix sort inside every table over the bits a row id of the largest table (or its one-past-the-end
// inert id) can set.  The last pass leaves the records in pk_a; the passes before it take turns in the halves of
// the record arrays, the one before the last in pk_b, and the samples of the first lie where its output does not.
template <typename Sample>
void sort_lookups(const SortCall& c) {
  const BwdWs& w = *c.w;
  const dmt_plan* plan = c.plan;
  if (c.nnz <= kSmallNnz && c.B <= kSmallBatch) {
    static DmtPerDevice configured;
    dmt_allow_lds(configured, (const void*)bwd_sort_small, kSmallLds);
    DmtScope scope(plan, DMT_K_BWD_KEYS, c.s);
    hipLaunchKernelGGL(bwd_sort_small, dim3((unsigned)plan->F), dim3(kSmallBlock), kSmallLds, c.s, plan->d_meta, c.indices,
                       c.offsets, (uint32_t)c.B, (int)plan->F, (int)c.nnz, w.pk_a,
                       plan->row_shards ? nullptr : plan->d_error, plan->d_error + 1);
    return;
  }
  int64_t max_rows = 0;
  for (int32_t f = 0; f < plan->F; ++f) max_rows = std::max<int64_t>(max_rows, plan->meta[f].rows);
  const int key_bits = ilog2_ceil(max_rows + 1);
  const int most_bits = w.wide ? kWideRadixBits : kMaxRadixBits;
  const int passes = (key_bits + most_bits - 1) / most_bits;
  const int bits_per = (key_bits + passes - 1) / passes;
  auto region = [&](int pass) { return (passes - pass) & 1 ? w.pk_a : w.pk_b; };   // where a pass writes
  Sample* const samples = (Sample*)(region(0) == w.pk_a ? w.pk_b : w.pk_a);
  timed_launch(plan, DMT_K_BWD_KEYS, c.s, bwd_bag_samples<Sample>, c.key_blocks + 1, kBlock, c.offsets, (uint32_t)c.B,
               c.nbags, c.nnz, (int)plan->F, samples, c.log2_bpb, w.least_items, w.seg_begin, w.seg_blk, w.blk_table,
               plan->d_error + 1);
  SortIo<Sample> io{};
  io.ids = c.indices;
  io.smp_in = samples;
  for (int p = 0; p < passes; ++p) {
    const bool first = p == 0, last = p == passes - 1;
    const int shift = p * bits_per, bits = std::min(bits_per, key_bits - shift);
    io.key_out = (uint32_t*)region(p);
    io.smp_out = (Sample*)(io.key_out + c.nnz);
    io.pk_out = w.pk_a;
    auto launch = [&](auto max_bits) {
      constexpr int M = decltype(max_bits)::value;
      if (first && last) launch_sort_pass<M, true, true, Sample>(c, io, shift, bits);
      else if (first) launch_sort_pass<M, true, false, Sample>(c, io, shift, bits);
      else if (last) launch_sort_pass<M, false, true, Sample>(c, io, shift, bits);
      else launch_sort_pass<M, false, false, Sample>(c, io, shift, bits);
    };
    if (w.wide) launch(std::integral_constant<int, kWideRadixBits>());
    else launch(std::integral_constant<int, kMaxRadixBits>());
    io.key_in = io.key_out;
    io.smp_in = io.smp_out;
  }
}

// What the reduce / fix-up launches share.
struct ReduceCall {
  const dmt_plan* plan;
  const BwdWs* w;
  const uint64_t* sorted;
  int64_t nnz, B;
  uint32_t nbags, total_rows;
  const float* grad;
  float lr, eps;
  hipStream_t s;
};

template <int TD, int EPL>
void launch_reduce_wave(const ReduceCall& c) {
  constexpr int kWavesPerBlock = kBlock / 64;
  const int64_t per_xcd = ((c.w->ntiles + kWavesPerBlock - 1) / kWavesPerBlock + 7) / 8;
  auto kernel = c.plan->classes.size() == 1 ? bwd_reduce_update_wave<TD, EPL, true>
                                            : bwd_reduce_update_wave<TD, EPL, false>;
  timed_launch(c.plan, DMT_K_BWD_REDUCE_UPDATE, c.s, kernel, per_xcd * 8, kBlock, c.plan->d_meta,
               c.sorted, c.nnz, (uint32_t)c.B, c.nbags, c.total_rows, c.grad, c.w->partials,
               c.plan->max_dim, c.w->tile, c.w->ntiles, per_xcd, c.lr, c.eps, c.plan->d_error + 1);
}

// bag / B for bag < 2^31 as (bag * mul) >> (32 + shift); B = 1 is handled by the kernel.
void bag_divider(uint32_t B, uint32_t& mul, uint32_t& shift) {
  uint32_t l = 0;
  while ((1ull << l) < B) ++l;
  mul = 0;
  shift = 0;
  if (B <= 1) return;
  mul = (uint32_t)(((1ull << (31 + l)) + B - 1) / B);
  shift = l - 1;
}

template <int TD>
void launch_reduce_lean(const ReduceCall& c) {
  constexpr int kWavesPerBlock = kLeanBlock / 64;
  const int64_t per_xcd = ((c.w->ntiles + kWavesPerBlock - 1) / kWavesPerBlock + 7) / 8;
  uint32_t mul, shift;
  bag_divider((uint32_t)c.B, mul, shift);
  timed_launch(c.plan, DMT_K_BWD_REDUCE_UPDATE, c.s, bwd_reduce_update_lean<TD>, per_xcd * 8, kLeanBlock,
               c.plan->d_meta, c.sorted, c.nnz, (uint32_t)c.B, mul, shift, (uint32_t)c.plan->F, c.grad,
               c.w->partials, c.plan->max_dim, c.w->tile, c.w->ntiles, per_xcd, c.lr, c.eps,
               c.plan->d_error + 1);
}

template <int TD, int LG>
void launch_reduce_grouped(const ReduceCall& c) {
  const int64_t blocks = (c.w->ntiles + (kBlock >> LG) - 1) / (kBlock >> LG);
  const int64_t per_xcd = (blocks + 7) / 8;
  auto kernel = c.plan->classes.size() == 1 ? bwd_reduce_update<TD, LG, true>
                                            : bwd_reduce_update<TD, LG, false>;
  timed_launch(c.plan, DMT_K_BWD_REDUCE_UPDATE, c.s, kernel, per_xcd * 8, kBlock, c.plan->d_meta,
               c.sorted, c.nnz, (uint32_t)c.B, c.nbags, c.total_rows, c.grad, c.w->partials,
               c.plan->max_dim, c.w->tile, c.w->ntiles, per_xcd, c.lr, c.eps, c.plan->d_error + 1);
}

// Segment reduce + row update, then the rows whose run spans tiles.
template <int TD>
void launch_reduce_and_fixup(const ReduceCall& c) {
  const int max_dim = c.plan->max_dim;
  const int log2_gl = std::max(2, ilog2_ceil(max_dim / 4));       // lanes that hold one row
  const bool wave_kernel = (max_dim == 128 || max_dim == 256) && c.plan->sw.bwd_kernel != 2;
  // the lean walk addresses a gradient slice by a 32-bit byte offset inside its tower's block
  int64_t widest = 0;
  for (int32_t t = 0; t < c.plan->T; ++t) widest = std::max<int64_t>(widest, c.plan->tower_width[t]);
  const bool lean = max_dim <= 128 && c.B * widest * 4 < (1LL << 32) && c.plan->sw.bwd_kernel == 0;
  if (lean) {
    launch_reduce_lean<TD>(c);
  } else if (wave_kernel) {
    if (max_dim == 128) launch_reduce_wave<TD, 2>(c); else launch_reduce_wave<TD, 4>(c);
  } else {
    switch (log2_gl) {
      case 2: launch_reduce_grouped<TD, 2>(c); break;
      case 3: launch_reduce_grouped<TD, 3>(c); break;
      case 4: launch_reduce_grouped<TD, 4>(c); break;
      case 5: launch_reduce_grouped<TD, 5>(c); break;
      default: launch_reduce_grouped<TD, 6>(c); break;
    }
  }
  const bool small = c.w->tile < kReduceTile;
  const int threads = small ? std::max(64, kLongGroups << log2_gl) : kFixBlock, groups = threads >> log2_gl;
  const int nlong = small ? (int)((c.w->ntiles - 1) / kLongRun) : 0;      // tiles 64, 128, ... < ntiles
  const int64_t blocks = nlong + (c.w->ntiles + groups - 1) / groups;
  timed_launch(c.plan, DMT_K_BWD_FIXUP, c.s, small ? bwd_fixup_update<TD, true> : bwd_fixup_update<TD, false>, blocks,
               threads, c.plan->d_meta, (uint32_t)c.B, c.nbags, c.sorted, c.nnz, c.total_rows, c.w->partials, max_dim,
               log2_gl, c.w->tile, c.w->ntiles, nlong, c.lr, c.eps, c.plan->d_error + 1);
}

}  // namespace

extern "C" size_t dmt_bwd_workspace_bytes(const dmt_plan* plan, int64_t B, int64_t nnz) {
  if (!plan || B <= 0 || nnz < 0) return 0;
  return carve(plan, nnz, nullptr).bytes;
}

// Validation and launches of the update; `workspace` is any device memory of at least
// carve().bytes bytes, 256-byte aligned.  Allocates nothing.
static dmt_status bwd_update_run(const dmt_plan* plan, const int32_t* indices,
                                 const int64_t* offsets, int64_t B, int64_t nnz,
                                 const float* grad_pooled, float lr, float eps, void* workspace,
                                 size_t workspace_bytes, void* stream, const dmt_bwd_debug* dbg) {
  if (!plan || !offsets || !grad_pooled) return DMT_EINVAL;
  if (B <= 0 || B > plan->max_batch || nnz < 0 || nnz > plan->max_nnz) return DMT_EINVAL;
  if (nnz > 0 && !indices) return DMT_EINVAL;
  if (!plan->bound || !plan->has_state) return DMT_EINVAL;
  if (!(eps >= 0.f) || lr != lr) return DMT_EINVAL;
  if ((uintptr_t)grad_pooled & 15) return DMT_EINVAL;
  if (plan->max_dim > 256) return DMT_ENOTSUP;          // one float4 per lane, 64 lanes
  if (B * plan->width_prefix[plan->T] >= (1LL << 33)) return DMT_ENOTSUP;   // float4 index in 32 bits
  const BwdWs w = carve(plan, nnz, workspace);
  if (!workspace || ((uintptr_t)workspace & 255)) return DMT_EINVAL;
  if (workspace_bytes < w.bytes) return DMT_ENOMEM;
  hipStream_t s = (hipStream_t)stream;
  const uint32_t total_rows = (uint32_t)plan->total_rows;
  const uint32_t nbags = (uint32_t)((int64_t)plan->F * B);
  const uint64_t* const sorted = w.pk_a;

  if (nnz > 0) {
    // samples; bags per block: about 4096 lookups' worth (a power of two, at most kKeysMaxBags), or
    // what it takes to give every CU four blocks, but at least a lookup per thread (260 K lookups:
    // 51 blocks of 4096 took 25.5 us, 813 of 320 take 5.7)
    const double mean_len = (double)nnz / (double)nbags;
    const double want = std::min(4096.0, std::max(256.0, (double)nnz / 1024.0));
    int log2_bpb = ilog2_ceil((int64_t)(want / (mean_len > 1.0 ? mean_len : 1.0) + 0.5));
    if (plan->sw.keys_lg >= 0) log2_bpb = plan->sw.keys_lg;
    log2_bpb = log2_bpb < 4 ? 4 : (log2_bpb > 10 ? 10 : log2_bpb);
    const int64_t key_blocks = ((int64_t)nbags + (1 << log2_bpb) - 1) >> log2_bpb;
    const SortCall sc{plan, &w, indices, offsets, nnz, B, nbags, log2_bpb, key_blocks, s};
    if (B <= 65536) sort_lookups<uint16_t>(sc); else sort_lookups<uint32_t>(sc);

    const ReduceCall call{plan, &w, sorted, nnz, B, nbags, total_rows, grad_pooled, lr, eps, s};
    switch (plan->table_dtype) {
      case DMT_F32: launch_reduce_and_fixup<DMT_F32>(call); break;
      case DMT_F16: launch_reduce_and_fixup<DMT_F16>(call); break;
      default: launch_reduce_and_fixup<DMT_BF16>(call); break;
    }
  }
  if (dbg && (dbg->sorted_keys || dbg->sorted_bag || dbg->unique_keys || dbg->seg_off ||
              dbg->num_unique)) {
    if (nnz > 0) {
      // run heads -> segment offsets (only the parity exports need them)
      timed_launch(plan, DMT_K_BWD_HEADS, s, heads_count, w.nblk_scan, kBlock, sorted, nnz,
                   w.blk_heads);
      timed_launch(plan, DMT_K_BWD_HEADS, s, heads_scan, 1, 1024, w.blk_heads, w.nblk_scan,
                   w.num_unique);
      timed_launch(plan, DMT_K_BWD_HEADS, s, heads_write, w.nblk_scan, kBlock, sorted, nnz,
                   w.blk_heads, w.seg_off);
    }
    const int64_t n = nnz + 1;
    hipLaunchKernelGGL(bwd_export, dim3((unsigned)((n + kBlock - 1) / kBlock)), dim3(kBlock), 0, s,
                       plan->d_row_base, plan->F, sorted, nnz, total_rows, w.seg_off, w.num_unique,
                       dbg->sorted_keys, dbg->sorted_bag, dbg->unique_keys, dbg->seg_off,
                       dbg->num_unique);
  }
  return hipGetLastError() == hipSuccess ? DMT_OK : DMT_EHIP;
}

extern "C" dmt_status dmt_tower_lookup_bwd_update(const dmt_plan* plan, const int32_t* indices,
                                                  const int64_t* offsets, int64_t B, int64_t nnz,
                                                  const float* grad_pooled, float lr, float eps,
                                                  void* workspace, size_t workspace_bytes,
                                                  void* stream, const dmt_bwd_debug* dbg) {
  return bwd_update_run(plan, indices, offsets, B, nnz, grad_pooled, lr, eps, workspace,
                        workspace_bytes, stream, dbg);
}

// ------------------------------------------- the update on the library's own scratch memory

// Scratch of dmt_tower_lookup_bwd_update_noalloc: one array per GPU the library runs on, held
// until the process ends.  Host code never uses the array's name as an address: it asks the
// runtime for the array's device address once per device and passes that pointer on.
static __device__ __align__(256) unsigned char scratch[DMT_BWD_NOALLOC_SCRATCH_BYTES];

namespace {
constexpr int kMaxDevices = 64;
std::mutex g_scratch_mutex;
void* g_scratch_ptr[kMaxDevices];   // device address of `scratch` on each device, once resolved
}  // namespace

extern "C" size_t dmt_bwd_noalloc_scratch_bytes(void) { return DMT_BWD_NOALLOC_SCRATCH_BYTES; }

extern "C" dmt_status dmt_tower_lookup_bwd_update_noalloc(const dmt_plan* plan,
                                                          const int32_t* indices,
                                                          const int64_t* offsets, int64_t B,
                                                          int64_t nnz, const float* grad_pooled,
                                                          float lr, float eps, void* stream) {
  if (!plan || B <= 0 || nnz < 0) return DMT_EINVAL;
  // the size check comes first: nothing is resolved or launched for a call that cannot fit
  if (carve(plan, nnz, nullptr).bytes > (size_t)DMT_BWD_NOALLOC_SCRATCH_BYTES) return DMT_ENOMEM;
  int dev = -1;
  DMT_HIP_TRY(hipGetDevice(&dev));
  if (dev < 0 || dev >= kMaxDevices) return DMT_ENOTSUP;
  void* ptr = nullptr;
  {
    std::lock_guard<std::mutex> lock(g_scratch_mutex);
    if (!g_scratch_ptr[dev]) {
      void* p = nullptr;
      DMT_HIP_TRY(hipGetSymbolAddress(&p, HIP_SYMBOL(scratch)));
      if (!p) return DMT_EHIP;
      g_scratch_ptr[dev] = p;
    }
    ptr = g_scratch_ptr[dev];
  }
  return bwd_update_run(plan, indices, offsets, B, nnz, grad_pooled, lr, eps, ptr,
                        (size_t)DMT_BWD_NOALLOC_SCRATCH_BYTES, stream, nullptr);
}
