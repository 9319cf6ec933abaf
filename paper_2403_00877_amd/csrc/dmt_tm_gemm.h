// Grouped contractions of the Tower Module, shared by its forward and backward:
//   C = epilogue(A . W^T [+ b]), either operand contiguous along the reduction dimension or along
// its own, one launch for all towers of a stage (block id -> tower, tile).
// 16-bit types run on MFMA (v_mfma_f32_16x16x32, float32 accumulate); float32 has its own kernel
// (dmt_tm_f32.h).  Also the pairwise-dot (Gram tile) kernels and the projection-weight
// repack of the dot-product form.  Everything lives in an unnamed namespace: each
// translation unit that includes this header gets its own copy.
#pragma once
#include <algorithm>
#include <vector>

#include "dmt_internal.h"
#include "dmt_device_utils.h"

namespace {

typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef _Float16 halfx8 __attribute__((ext_vector_type(8)));
typedef float floatx4 __attribute__((ext_vector_type(4)));
typedef float floatx16 __attribute__((ext_vector_type(16)));

constexpr int kBlock = 256;              // threads of the small kernels' blocks
constexpr int BK = 64;                   // K step of the matrix kernels
constexpr int kMaxGroups = 16;

// EPI_F32 / EPI_F32_ADD: C is float32 whatever the operand type, no bias: C = acc / C += acc
// (gradients: the backward's accumulations stay in float32)
// EPI_CROSS_GRAD: a cross tower's gradient on its way down, acc being the data gradient of layer l or
// of the projection (l = the number of layers):
//   g_l = acc + g_{l+1}                       (float32; the sum without GN for the projection)
//   C = g_l                                   (where C is set: layers below need it)
//   DU = du_{l-1} = g_l * x0                  (rounded), DBP its column sums
//   ACC (+)= g_{l+1} * u_l [+ (g_1 * u_0 + g_1) where U0 is set, l = 1]
// (each product rounded to float32 before it is added, as in tmb_cross_prep: how the steps are shared
// out over kernels leaves grad_pooled as it is, to the last bit)
enum { EPI_BIAS = 0, EPI_BIAS_RELU = 1, EPI_CROSS = 2, EPI_F32 = 3, EPI_F32_ADD = 4, EPI_CROSS_GRAD = 5 };

// How an operand lies in memory: OP_ROW with its K columns contiguous ([M][ld], k in a row), or
// OP_COL with its row index contiguous ([K][ld]).  A data gradient contracts dz (OP_ROW) with the
// weights as they are (OP_COL), a weight gradient dz with x (both OP_COL): nothing is transposed.
enum { OP_ROW = 0, OP_COL = 1 };

// One contraction of a grouped launch, C[m][n] = sum over k of A(m, k) W(n, k).  K comes in two
// segments (the dot terms, then the pooled values); a plain contraction has K0 = 0.  Operand rows
// are multiples of 8 elements apart, the bases 16-byte aligned (W0 / W1: 4-byte aligned).
struct TmGroup {
  const void* A0;   // first K0 of the contraction
  const void* A1;   // next K1
  const void* W0;
  const void* W1;
  const void* bias; // [N] or NULL (no bias)
  const void* X0;   // EPI_CROSS: [M][ldx] (x0)
  const void* XL;   // EPI_CROSS: the x_l term, [M][ldxl]
  void* C;          // [M][ldc]
  // EPI_CROSS: when set, u = acc + bias (before the cross product) is also stored here, laid
  // out like C (what the backward needs of a cross layer).  A group whose dot terms are computed
  // in-kernel: when set, they are also stored here as [M][K0], zeros in the padding columns.
  void* U;
  int32_t lda0, K0, lda1, K1, ldw0, ldw1, ldc, ldx, ldxl, M, N, epi;
  int32_t nf, fdim;       // dot terms computed in-kernel: number of features and their dim
  // Split K (EPI_F32 with K0 = 0 only): ksplit > 1 cuts the K1 columns into slices of klen
  // (a multiple of BK); slice s is a contraction of its own whose result goes to
  // C + s * cstride floats, and the caller adds the slices up in a fixed order.
  int32_t ksplit, klen;
  int64_t cstride;
  // EPI_CROSS_GRAD: [M][ldc] float32 / 16-bit tensors, and the column sums of du, one row per 64 rows
  // of C
  const float* GN;        // g_{l+1} or NULL
  const void* UL;         // u_l (with GN)
  const void* U0;         // u_0 or NULL
  float* ACC;
  void* DU;
  float* DBP;             // [(M + 63) / 64][N]
  int32_t acc_first;      // ACC holds nothing yet
  // Two-level output rows: with rdiv > 0 row m of C starts at (m / rdiv) * ldc + (m % rdiv) * ldc2,
  // i.e. rdiv consecutive rows of the contraction share one row of the output tensor.
  int32_t rdiv, ldc2;
  // reps > 1 (no split K): so many contractions that differ in where A1, W0 (elements) and C (cstride
  // floats) start: a per-feature layer's.  They take the place of the slices.
  int32_t reps, a1_step, w0_step;
};

__host__ __device__ inline int tm_slices(const TmGroup& g) { return g.ksplit > 1 ? g.ksplit : g.reps > 1 ? g.reps : 1; }
// The first k behind the slice that starts at kofs < K1.  (kofs + klen may lie up to a K step per slice past
// K1, which itself may be next to 2^31.)
__host__ __device__ inline int tm_slice_end(int K1, int kofs, int klen) {
  return klen < K1 - kofs ? kofs + klen : K1;
}

struct TmLaunch {
  int32_t ngroups;
  int32_t super;                       // tiles of a super-tile (dealt to one XCD), at most
  int32_t cap;                         // block slots of a super-tile
  int32_t slots;                       // of an XCD
  int32_t step;                        // blocks of an XCD
  int32_t stagger;                     // how far apart the XCDs start, in sleeps of 4096 cycles
  int32_t tile_start[kMaxGroups + 1];  // first super-tile of each group
  TmGroup g[kMaxGroups];
};

template <int DT>
__device__ __forceinline__ floatx16 mfma32(uint4 a, uint4 b, floatx16 c) {
  if constexpr (DT == DMT_BF16)
    return __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(bf16x8, a),
                                                   __builtin_bit_cast(bf16x8, b), c, 0, 0, 0);
  else
    return __builtin_amdgcn_mfma_f32_32x32x16_f16(__builtin_bit_cast(halfx8, a),
                                                  __builtin_bit_cast(halfx8, b), c, 0, 0, 0);
}

template <int DT>
__device__ __forceinline__ floatx4 mfma16(uint4 a, uint4 b, floatx4 c) {
  if constexpr (DT == DMT_BF16)
    return __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8, a),
                                                   __builtin_bit_cast(bf16x8, b), c, 0, 0, 0);
  else
    return __builtin_amdgcn_mfma_f32_16x16x32_f16(__builtin_bit_cast(halfx8, a),
                                                  __builtin_bit_cast(halfx8, b), c, 0, 0, 0);
}

template <int DT> __device__ __forceinline__ float load_elt(const void* p, int64_t i) {
  if constexpr (DT == DMT_F32) return ((const float*)p)[i];
  else if constexpr (DT == DMT_F16) return dmt::f16_bits_to_f32(((const uint16_t*)p)[i]);
  else return dmt::bf16_lo(((const uint16_t*)p)[i]);
}

template <int DT> __device__ __forceinline__ void store_elt(void* p, int64_t i, float v) {
  if constexpr (DT == DMT_F32) ((float*)p)[i] = v;
  else if constexpr (DT == DMT_F16) ((uint16_t*)p)[i] = (uint16_t)dmt::f32_to_f16_bits(v);
  else ((uint16_t*)p)[i] = (uint16_t)dmt::f32_to_bf16_bits(v);
}

// a * b rounded to float32: never fused into an addition.
__device__ __forceinline__ float mul_rounded(float a, float b) {
#pragma clang fp contract(off)
  return a * b;
}

// ------------------------------------------------------------- MFMA grouped GEMM
//
// Two tilings of one kernel.  256 x 256 x 64, eight waves (two per SIMD) of 128 x 64, one block per
// CU: a 128 x 128 tile needs 1 byte from L2 per 64 FLOP, which caps the matrix cores at a fraction
// of their rate, and 256 x 256 halves that.  128 x 128 x 64, four waves of 64 x 64, two blocks per
// CU: for launches that would leave CUs without a 256 x 256 tile, and for outputs of at most 128
// rows or columns.
//
// 16 x 16 x 32 instructions rather than 32 x 32 x 16: the chip is power-limited on real data, and they
// take less of it for the same product (registers only, normal random operands: 1990 against 1730
// TFLOP/s; on zeros both reach 2430).  Within a row of them the W fragments go back and forth, so
// that neighbouring instructions share an operand (1990 against 1952).
//
// Operand tiles go from global memory straight into LDS (buffer_load_dwordx4 ... lds: a wave's 64
// lanes fill 1 KB of consecutive LDS, 16 bytes a lane), two stages deep: tile kt + 2 is requested
// into the stage tile kt is being read from, behind the barrier inside step kt, one request per row of
// MFMAs (in one burst they fill the memory pipe's queue, and the matrix instructions behind them
// wait), and every wave waits for its own requests before the next step's barrier.  The buffer's
// bounds stand in for all edges: rows past the operand's last, and chunks past the last k (their lanes
// ask for an offset that is never in bounds), arrive as zeros.  (The requests are inline assembly:
// told about them, the compiler makes every LDS read of the current tile wait for the next tile's
// requests, since it cannot tell the two stages apart.)
//
// The K steps of all the tiles a block works through are one stream: behind a tile's last step come the
// requests for the next tile's first, so that a tile starts with its operands in LDS; the epilogue in
// between has LDS of its own.
//
// OP_ROW tile: 128-byte rows (64 k) without padding; column chunk c (8 elements) of row r sits in
// slot c ^ (r / 2) % 8.  A fragment read (ds_read_b128, 16 lanes a cycle from 64 banks) touches 16
// rows: 2 r and 2 r + 1 lie in the two halves of one 256-byte bank row and share a slot, the eight
// pairs differ in it, so it is conflict-free.
// OP_COL tile: 64 rows of BM (BN) elements, one per k; chunk c of row k sits in slot
// c ^ 4 (k % 4) ^ 2 (k / 8 % 2).  Fragments come through ds_read_b64_tr_b16, which transposes 4 x 4
// blocks among 16 lanes: lane p of a group names row k + p / 4, elements 4 (p % 4) ..., and receives
// column p of the four rows.  The four rows of a group and those of the next (k + 8) lie on the same
// banks but for the slot, which spreads them.
//
// The MFMAs take the W fragment as their first operand, so the accumulators hold the tile
// transposed: a lane owns one row and four consecutive columns per tile of 16.

// TAG only marks the including source file in the kernel's name, so that a profile tells the
// forward's launches from the backward's.
#ifndef DMT_TM_TAG
#define DMT_TM_TAG 0
#endif

constexpr uint32_t kOobOffset = 0x80000000u;      // beyond any buffer (256 rows of a tile stay far below it)

// Buffer descriptor of `bytes` bytes from p (uniform).
__device__ __forceinline__ __amdgpu_buffer_rsrc_t tm_buffer(const void* p, uint32_t bytes) {
  // (all of it through scalar registers: the requests' assembly takes no others)
  const uint32_t lo = __builtin_amdgcn_readfirstlane((uint32_t)(uintptr_t)p), hi = __builtin_amdgcn_readfirstlane((uint32_t)((uintptr_t)p >> 32));
  return __builtin_amdgcn_make_buffer_rsrc((void*)((uintptr_t)hi << 32 | lo), 0, (int)__builtin_amdgcn_readfirstlane(bytes), 0x00020000);
}
// 64 lanes' 16-byte pieces of a buffer to 1 KB of LDS at byte address lds.
__device__ __forceinline__ void tm_request(uint32_t lds, __amdgpu_buffer_rsrc_t rsrc, uint32_t off) {
  asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tbuffer_load_dwordx4 %1, %2, 0 offen lds"
               :: "s"(__builtin_amdgcn_readfirstlane(lds)), "v"(off), "s"(rsrc) : "memory");
}

// 64 lanes' 4-byte pieces of a buffer to 256 bytes of LDS.
__device__ __forceinline__ void tm_touch(uint32_t lds, __amdgpu_buffer_rsrc_t rsrc, uint32_t off) {
  asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tbuffer_load_dword %1, %2, 0 offen lds"
               :: "s"(__builtin_amdgcn_readfirstlane(lds)), "v"(off), "s"(rsrc) : "memory");
}

// One operand's side of a block tile of R rows (A: R = BM, W: R = BN), staged by NW waves.
template <int LAY, int R, int NW>
struct TmStage {
  static constexpr int kInstr = R * BK * 2 / 1024 / NW;    // requests per wave and K step
  static_assert(NW % 2 == 0 && kInstr * NW * 1024 == R * BK * 2, "");
  uint32_t off, step;                              // this lane's byte offset from the tile's first element; a request's from the last
  int chunk;                                       // OP_ROW: this lane's column chunk (the same in every request)
  const uint16_t* base;                            // the tile's first element at the segment's first k
  int ld, rows;                                    // row pitch; operand rows in the tile

  // p: the operand, pitch ld_; row0: the tile's first row of rows_all; k0: the segment's first k.  (What
  // the requests need of the group is read here: behind a request, the compiler reads it anew.)
  __device__ __forceinline__ void init(const void* p, int ld_, int row0, int rows_all, int k0, int wave, int lane) {
    ld = ld_;
    rows = min(rows_all - row0, R);
    base = (const uint16_t*)p + (LAY == OP_ROW ? (int64_t)row0 * ld + k0 : (int64_t)k0 * ld + row0);
    chunk = LAY == OP_ROW ? (lane & 7) ^ (((wave & 1) << 2) | (lane >> 4)) : 0;
    if constexpr (LAY == OP_ROW) {
      off = ((uint32_t)(wave * 8 + (lane >> 3)) * (uint32_t)ld + chunk * 8) * 2u;
      step = NW * 8 * 2u * (uint32_t)ld;
    } else {
      constexpr int kRowLanes = R / 8;             // 16-byte slots of one k row
      static_assert(NW * (64 / kRowLanes) % 16 == 0, "requests 16 k apart share a slot");
      const int k = wave * (64 / kRowLanes) + lane / kRowLanes;
      const int c = (lane % kRowLanes) ^ ((k & 3) << 2) ^ ((k >> 2) & 2);
      off = c * 8 < rows ? ((uint32_t)k * (uint32_t)ld + c * 8) * 2u : kOobOffset;
      step = NW * (64 / kRowLanes) * 2u * (uint32_t)ld;
    }
  }
  // The segment's columns k .. k + 63 (from its first; kn are left), for request().  The buffer ends with
  // the tile's own last row and K step, so a step's descriptor is a few 32-bit scalar operations on
  // values that stay in registers.  Read and clamped from the group on every K step, it held up
  // the requests by a scalar load's latency: DCN training step 14.33 -> 13.94 ms, mid forward 308 -> 302 us.
  __device__ __forceinline__ __amdgpu_buffer_rsrc_t buffer(int k, int kn) const {
    // (The bounds check is by 4 bytes.  OP_ROW: the last row counts to the end of its last chunk, which
    // its pitch has room for.  OP_COL: to the end of the last element's 4 bytes and no further, since
    // the pitch may be less than whole chunks: with rows = ld = 12 the next k's first elements would
    // count as in bounds, and what lies past the tensor would meet the other operand's zeros.)
    const uint32_t left = (uint32_t)min(kn, BK);
    const uint32_t bytes = (LAY == OP_ROW ? (uint32_t)(rows - 1) * (uint32_t)ld + ((left + 7) & ~7u)
                                          : (left - 1) * (uint32_t)ld + ((uint32_t)(rows + 1) & ~1u)) * 2u;
    return tm_buffer(base + (LAY == OP_ROW ? (int64_t)k : (int64_t)k * ld), kn > 0 ? bytes : 0u);
  }
  // OP_ROW: zeros in columns k .. (k even) of the pieces of a landed tile that also hold columns before k
  // (each lane its own pieces).
  __device__ __forceinline__ void zero_from(uint16_t* tile, int k, int wave, int lane) const {
    if (!(k & 7) || chunk != k >> 3) return;
    uint4* const p = (uint4*)tile + wave * 64 + lane;
#pragma clang loop unroll(full)
    for (int j = 0; j < kInstr; ++j) {
      const uint4 v = p[j * NW * 64];
      p[j * NW * 64] = make_uint4(v.x, (k & 7) > 2 ? v.y : 0u, (k & 7) > 4 ? v.z : 0u, 0u);
    }
  }
  // This wave's j-th request of a step with kn columns left in the segment.
  __device__ __forceinline__ void request(uint32_t lds, __amdgpu_buffer_rsrc_t rsrc, int j, int wave, int kn) const {
    tm_request(lds + (j * NW + wave) * 1024, rsrc, LAY == OP_COL || chunk * 8 < kn ? off + j * step : kOobOffset);
  }
};

// One operand's fragment reads: fragment i is rows 16 i ... (from row `first`, a multiple of 64) x 32 k of a
// staged tile of R rows; lane l gets 8 consecutive k (8 (l / 16) ...) of its row l % 16.
template <int LAY, int R>
struct TmFrag {
  int at[LAY == OP_ROW ? BK / 32 : 1];
  __device__ __forceinline__ void init(int first, int lane) {
    if constexpr (LAY == OP_ROW) {
#pragma clang loop unroll(full)
      for (int kk = 0; kk < BK / 32; ++kk)
        at[kk] = (first + (lane & 15)) * BK + ((kk * 4 + (lane >> 4)) ^ ((lane >> 1) & 7)) * 8;
    } else {
      const int p = lane & 15, k = (lane >> 4) * 8 + (p >> 2);
      at[0] = k * R + (((first >> 3) + ((p & 3) >> 1)) ^ ((k & 3) << 2) ^ ((k >> 2) & 2)) * 8 + (p & 1) * 4;
    }
  }
  __device__ __forceinline__ uint4 read(const uint16_t* tile, int kk, int i) const {
    if constexpr (LAY == OP_ROW) {
      return *(const uint4*)(tile + at[kk] + i * 16 * BK);
    } else {
      typedef short short4v __attribute__((ext_vector_type(4)));
      typedef __attribute__((address_space(3))) short4v lds_short4;
      const uint16_t* q = tile + (at[0] ^ (i * 16)) + kk * 32 * R;
      const uint2 lo = __builtin_bit_cast(uint2, __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_short4*)q));
      const uint2 hi = __builtin_bit_cast(uint2, __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_short4*)(q + 4 * R)));
      return make_uint4(lo.x, lo.y, hi.x, hi.y);
    }
  }
};

// Whether a group's outputs, and what its epilogue reads, move in whole pieces of 16 bytes.  (EPI_CROSS_GRAD:
// N and ldc are a tower's width, the tensors the library's own or blocks of grad_pooled.)
__device__ __forceinline__ bool tm_whole(const TmGroup& g) {
  // (no short circuits: the fields are read together)
  const uint64_t c = (uint64_t)g.C, x = (uint64_t)g.X0 | (uint64_t)g.XL | (uint64_t)g.U;
  const bool f32 = ((g.N | g.ldc) & 3) == 0 & g.rdiv == 0 & (c & 15) == 0 & (tm_slices(g) <= 1 | (g.cstride & 3) == 0);
  const bool b16 = ((g.N | g.ldc | g.ldc2) & 7) == 0 & ((c | (uint64_t)g.bias) & 15) == 0;
  const bool cross = ((g.ldx | g.ldxl) & 7) == 0 & (x & 15) == 0;
  return g.epi == EPI_CROSS_GRAD | (g.epi >= EPI_F32 ? f32 : b16 & (g.epi != EPI_CROSS | cross));
}

// Orders a wave's LDS accesses: lanes read what other lanes wrote.  (A wave's LDS instructions execute in
// order; to the compiler its lanes are unrelated threads.)
__device__ __forceinline__ void wave_sync() {
  __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
  __builtin_amdgcn_wave_barrier();
  __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

// Sum over the four lanes l, l ^ 16, l ^ 32, l ^ 48; every lane gets it.
__device__ __forceinline__ float quarters_sum(float v) {
  v += __shfl_xor(v, 16);
  return v + __shfl_xor(v, 32);
}

// TILE: 256 or 128.  DOTS: the operand's first K0 (<= 64) columns are the tower's pairwise dot
// terms, which the block computes itself (Gram tiles, as in tm_dots_mfma) straight into the first
// LDS stage, so the dot terms never exist in global memory (unless KEEPZ: a training forward keeps
// them).
template <int TILE> struct TmTile {
  static constexpr int WM = 2, WN = TILE == 256 ? 4 : 2, kWaves = WM * WN, kThreads = kWaves * 64;
  static constexpr int MT = TILE / WM / 16, NT = TILE / WN / 16;     // MFMA tiles of a wave
  static constexpr int kStageBytes = 2 * TILE * BK * 2;              // A then W
  static constexpr int kHalf = TILE / WM;                            // rows a wave covers
  static constexpr int kLdsBytes = 2 * kStageBytes + kWaves * 4096;  // two stages, 4 KB a wave for the epilogue
  static_assert(NT == 4, "the epilogue takes 64 columns a wave");
};

constexpr int min_int(int a, int b) { return a < b ? a : b; }

// A block's work: one tile of one group (of one slice of its K).
struct TmWork {
  int gi, m0, n0, slice;
};

// What a launch's epilogues are: KIND_READS those that read as much as they write (EPI_CROSS,
// EPI_CROSS_GRAD), KIND_SUMS EPI_CROSS_GRAD of towers of three layers and more, whose gradients add to what the
// layers behind left in ACC, KIND_ADD EPI_F32_ADD, KIND_PLAIN all others.  (Kernels of their own: together they need
// more registers, and what an epilogue reads ahead behind a run-time condition is slow: data gradients of
// 16 towers of 2048 columns, batch 8192, added to a tensor 1303 us, in a kernel of their own 1090.)
enum { KIND_PLAIN = 0, KIND_READS = 1, KIND_ADD = 2, KIND_SUMS = 3 };
inline bool epi_sums(const TmGroup& g) { return g.epi == EPI_CROSS_GRAD && !g.acc_first && (g.GN || g.U0); }
inline int epi_kind(int epi) {           // (KIND_SUMS: a launch of KIND_READS of which any group is one)
  return epi == EPI_CROSS || epi == EPI_CROSS_GRAD ? KIND_READS : epi == EPI_F32_ADD ? KIND_ADD : KIND_PLAIN;
}

template <int DT, int TILE, int ALAY, int WLAY, int KIND = KIND_PLAIN, bool DOTS = false, bool KEEPZ = false, int TAG = DMT_TM_TAG>
__global__ __launch_bounds__(TmTile<TILE>::kThreads, TILE == 256 ? 1 : 2) void tm_gemm(const TmLaunch L) {
  using T = TmTile<TILE>;
  constexpr bool kForward = ALAY == OP_ROW && WLAY == OP_ROW;        // 16-bit outputs and x0; the others are gradients
  static_assert(!DOTS || kForward, "");
  extern __shared__ __attribute__((aligned(16))) uint16_t lds[];
  // XCD-aware rasterisation.  Consecutive block ids go to different XCDs, so block b belongs
  // to XCD b % 8 and is that XCD's (b / 8)-th block.  The launch's tiles are cut into
  // super-tiles of up to L.super tiles (a few tile rows x all tile columns of one group) that
  // are dealt to the XCDs in turn: the blocks resident on an XCD then share their A rows
  // and W columns in that XCD's L2 instead of every XCD pulling every A tile over the fabric.
  // A grid smaller than the launch's slots works through them a grid at a time, in the same order.
  int slot = blockIdx.x >> 3;
  auto locate = [&](TmWork& w) __attribute__((always_inline)) {      // this block's next tile, if there is one
    for (; slot < L.slots; slot += L.step) {
      const int gs = (slot / L.cap) * 8 + (blockIdx.x & 7), within = slot % L.cap;
      if (gs >= L.tile_start[L.ngroups]) continue;
      int gi = 0;
      while (gi + 1 < L.ngroups && gs >= L.tile_start[gi + 1]) ++gi;
      const TmGroup& G = L.g[gi];
      // (All lines of the group's arguments at once, and no others, the grid's size among them, before the first
      // request: a block's first read of each line goes to memory.  One after another as the code below needs them,
      // 512 blocks of two K steps each took 12.5 us, now 11.8; dot terms and 16 K steps, 128 blocks, 31.5, now 29.9.)
      const uint32_t* gp = (const uint32_t*)&G;
      static_assert(sizeof(TmGroup) > 192 && sizeof(TmGroup) <= 256, "the lines that are read");
      asm volatile("" :: "s"(gp[0]), "s"(gp[16]), "s"(gp[32]), "s"(gp[48]), "s"(gp[sizeof(TmGroup) / 4 - 1]));
      const int tiles_n = (G.N + TILE - 1) / TILE, tiles_m = (G.M + TILE - 1) / TILE;
      const int sm = tiles_n >= L.super ? 1 : L.super / tiles_n;     // tile rows per super-tile
      // a split K multiplies the tile rows: virtual row tmv = slice * tiles_m + tm
      const int tmv = (gs - L.tile_start[gi]) * sm + within / tiles_n;
      if (within >= sm * tiles_n || tmv >= tiles_m * tm_slices(G)) continue;
      w.gi = __builtin_amdgcn_readfirstlane(gi);
      w.slice = __builtin_amdgcn_readfirstlane(tmv / tiles_m);
      w.m0 = __builtin_amdgcn_readfirstlane(tmv % tiles_m * TILE);
      w.n0 = __builtin_amdgcn_readfirstlane(within % tiles_n * TILE);
      slot += L.step;
      return true;
    }
    return false;
  };
  // Blocks that work through several tiles of cross layers start a little apart, XCD by XCD: their epilogues,
  // bound by memory, then meet other XCDs' matrix work instead of one another's.  (Cross layer of 2048
  // columns with u kept, 16 towers, batch 8192: 1155 -> 1131 us, its gradient 1658 -> 1598; plain
  // epilogues gain nothing.)
  if constexpr (KIND != KIND_PLAIN)
    for (int q = (blockIdx.x & 7) * L.stagger; q > 0; --q) __builtin_amdgcn_s_sleep(64);
  TmWork work, ahead;                              // the tile being computed, the one being requested
  if (!locate(ahead)) return;
  work = ahead;

  const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int wm = wave / T::WN, wn = wave % T::WN;

  // ---- the requests
  TmStage<ALAY, TILE, T::kWaves> sa;
  TmStage<WLAY, TILE, T::kWaves> sw;
  constexpr int kReqs = 2 * TmStage<ALAY, TILE, T::kWaves>::kInstr;  // of a wave and K step: A and W in turn
  const uint32_t lds0 = (uint32_t)(size_t)(__attribute__((address_space(3))) uint16_t*)lds;
  __amdgpu_buffer_rsrc_t ba, bw;
  uint32_t to = 0;
  int k = 0, left = 0, kn = 0, stage = 0;          // of the next step: first k, columns left; of this one; its stage
  bool flat = false;                               // the second segment (pooled values) is being requested
  auto begin = [&](bool second) __attribute__((always_inline)) {
    const TmGroup& G = L.g[ahead.gi];
    flat = second;
    k = 0;
    if (second) {
      const int kofs = G.ksplit > 1 ? ahead.slice * G.klen : 0;
      left = (G.ksplit > 1 ? tm_slice_end(G.K1, kofs, G.klen) : G.K1) - kofs;
      sa.init((const uint16_t*)G.A1 + (int64_t)ahead.slice * G.a1_step, G.lda1, ahead.m0, G.M, kofs, wave, lane);
      sw.init(G.W1, G.ldw1, ahead.n0, G.N, kofs, wave, lane);
    } else {                                       // (in-kernel dot terms: A comes from the block itself)
      left = G.K0;
      if constexpr (!DOTS) sa.init(G.A0, G.lda0, ahead.m0, G.M, 0, wave, lane);
      sw.init((const uint16_t*)G.W0 + (int64_t)ahead.slice * G.w0_step, G.ldw0, ahead.n0, G.N, 0, wave, lane);
    }
  };
  // The next K step of the stream.  (The launch makes sure that a block with several tiles is never more
  // than one of them ahead: their K is two steps or more.)
  auto aim = [&]() __attribute__((always_inline)) {
    if (left <= 0) {
      if (!flat) begin(true);
      else if (locate(ahead)) begin(L.g[ahead.gi].K0 == 0);
    }
    bw = sw.buffer(k, left);
    ba = DOTS && !flat ? bw : sa.buffer(k, left);
    kn = left;
    to = lds0 + stage * T::kStageBytes;
    stage ^= 1;
    k += BK;
    left -= BK;
  };
  auto request = [&](int q) __attribute__((always_inline)) {
    if (q % 2 == 0) sa.request(to, ba, q / 2, wave, kn);
    else sw.request(to + TILE * BK * 2, bw, q / 2, wave, kn);
  };

  // ---- fragments: A's of a row of MFMAs are read three rows ahead, W's of a slice of 32 k a slice ahead
  TmFrag<ALAY, TILE> ra;
  TmFrag<WLAY, TILE> rw;
  ra.init(wm * T::MT * 16, lane);
  rw.init(wn * T::NT * 16, lane);
  constexpr int kRows = BK / 32 * T::MT, kAhead = 3;                 // rows of MFMAs in a K step
  // Requests per row, and how many the rows behind the barrier hold.  128 x 128 tiles: all of them right behind
  // it, ahead of the row's LDS reads.  Their K steps are half as long and their launches wait for memory: two per row,
  // a projection of 512 outputs on 8 towers, batch 3001, took 69.8 instead of 66.7 us.
  constexpr bool kBurst = TILE != 256;
  constexpr int kPerRow = kBurst ? kReqs : 1, kEarly = min_int(kReqs, kAhead * kPerRow);
  static_assert((kReqs - kEarly + kPerRow - 1) / kPerRow < kRows - kAhead - 2, "");
  uint4 fa[4], fw[2][T::NT];

  // what the K loop and the epilogue need of the tile being computed, read while requests are under way
  int nk, kl;                                      // K steps; columns of the second segment
  bool whole;
  auto measure = [&]() __attribute__((always_inline)) {
    const TmGroup& G = L.g[work.gi];
    const int kofs = G.ksplit > 1 ? work.slice * G.klen : 0;
    kl = (G.ksplit > 1 ? tm_slice_end(G.K1, kofs, G.klen) : G.K1) - kofs;
    nk = (G.K0 + BK - 1) / BK + (kl + BK - 1) / BK;
    whole = __builtin_amdgcn_readfirstlane(tm_whole(G));
  };

  begin(L.g[work.gi].K0 == 0);
  aim();
#pragma clang loop unroll(full)
  for (int q = DOTS ? 1 : 0; q < kReqs; q += DOTS ? 2 : 1) request(q);
  aim();
  if (kn > 0)
#pragma clang loop unroll(full)
    for (int q = 0; q < kEarly; ++q) request(q);
  {
    if constexpr (DOTS) {
      const TmGroup& G = L.g[work.gi];
      const int m0 = work.m0, M = G.M, K0 = G.K0;
      // pairwise dots of this block's samples into the first stage's A tile, zeros behind them: a
      // wave takes 32 / nf samples at a time, whose (sample, feature) rows are one Gram tile
#pragma clang loop unroll(full)
      for (int q = 0; q < TILE * BK * 2 / 16 / T::kThreads; ++q)
        *(uint4*)(lds + (q * T::kThreads + tid) * 8) = make_uint4(0, 0, 0, 0);
      __syncthreads();
      const int nf = G.nf, fd = G.fdim, spg = 32 / nf;
      const uint16_t* A = (const uint16_t*)G.A1;
      const int c = lane & 31, sc = c / nf, j = c % nf, h8 = (lane >> 5) * 8;
      const int np = nf * (nf - 1) / 2, npad = K0 - np;
      // the term each of this lane's 16 sums is (a byte each), kNoTerm: none
      constexpr int kNoTerm = 255;
      uint32_t terms[4] = {0, 0, 0, 0};
#pragma clang loop unroll(full)
      for (int v = 0; v < 16; ++v) {
        const int rr = (v >> 2) * 8 + (lane >> 5) * 4 + (v & 3), i = rr - sc * nf;
        terms[v >> 2] |= (uint32_t)(i >= 0 && i < j ? i * (2 * nf - i - 1) / 2 + (j - i - 1) : kNoTerm) << (v & 3) * 8;
      }
      // Sample groups a wave has under way together, and 16-column pieces of each it requests at once.  A
      // launch of 128 x 128 tiles leaves CUs short of blocks, and the terms take one load latency per step
      // (26 features of 128 columns on 4 towers, batch 2003: launch 38.5 -> 35.8 us); with 256 x 256 tiles
      // the loads of all CUs are at the memory's rate already, and more of them in flight is slower
      // (the phase 25.4 us on 64 features at batch 8192, 27.9 with two groups).
      constexpr int kGroups = TILE == 128 ? 2 : 1, kPieces = TILE == 128 ? 8 : 4;
      for (int s0 = wave * spg; s0 < TILE; s0 += kGroups * T::kWaves * spg) {
        bool on[kGroups];
        const uint16_t* xp[kGroups];
        floatx16 d[kGroups];
#pragma clang loop unroll(full)
        for (int g = 0; g < kGroups; ++g) {
          const int s = s0 + g * T::kWaves * spg + sc;
          on[g] = sc < spg && s < TILE && m0 + s < M;
          xp[g] = A + (on[g] ? (int64_t)(m0 + s) * G.lda1 + j * fd + h8 : 0);
#pragma clang loop unroll(full)
          for (int v = 0; v < 16; ++v) d[g][v] = 0.f;
        }
        for (int k = 0; k < fd; k += kPieces * 16) {
          uint4 a[kGroups][kPieces];
#pragma clang loop unroll(full)
          for (int g = 0; g < kGroups; ++g)
#pragma clang loop unroll(full)
            for (int u = 0; u < kPieces; ++u)       // (never past the tensor: what is not wanted reads its start)
              a[g][u] = dmt::gload((const uint4*)(on[g] && k + u * 16 + h8 < fd ? xp[g] + k + u * 16 : A));
#pragma clang loop unroll(full)
          for (int g = 0; g < kGroups; ++g)
#pragma clang loop unroll(full)
            for (int u = 0; u < kPieces; ++u) {
              if (!(on[g] && k + u * 16 + h8 < fd)) a[g][u] = make_uint4(0, 0, 0, 0);
              d[g] = mfma32<DT>(a[g][u], a[g][u], d[g]);
            }
        }
#pragma clang loop unroll(full)
        for (int g = 0; g < kGroups; ++g) {
          const int sg = s0 + g * T::kWaves * spg, s = sg + sc;
#pragma clang loop unroll(full)
          for (int v = 0; v < 16; ++v) {
            const int term = (terms[v >> 2] >> (v & 3) * 8) & 255;
            if (on[g] && term < kNoTerm) {
              store_elt<DT>(lds, s * BK + (((term >> 3) ^ ((s >> 1) & 7)) << 3) + (term & 7), d[g][v]);
              if constexpr (KEEPZ)
                if (G.U) store_elt<DT>(G.U, (int64_t)(m0 + s) * K0 + term, d[g][v]);
            }
          }
          if constexpr (KEEPZ) {
            if (G.U)
              for (int e = lane; e < spg * npad; e += 64) {
                const int row = sg + e / npad;
                if (row < TILE && m0 + row < M) store_elt<DT>(G.U, (int64_t)(m0 + row) * K0 + np + e % npad, 0.f);
              }
          }
        }
      }
    }
    if constexpr (DOTS) {
      // Weights that are read as they are: the pooled values' weights stand behind the terms' and
      // meet the zeros behind the terms.  They count as zeros (an infinite one would make NaN).
      const TmGroup& G = L.g[work.gi];
      asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
      const int np = G.nf * (G.nf - 1) / 2;
      if ((const uint16_t*)G.W0 + np == G.W1) sw.zero_from(lds + TILE * BK, np, wave, lane);
      measure();
    } else {
      measure();
      // vmcnt: this wave's requests of the first step have landed
      if (kn > 0) __builtin_amdgcn_s_waitcnt(0x0f70 + kEarly);
      else __builtin_amdgcn_s_waitcnt(0x0f70);
    }
    __syncthreads();
  }
  const uint16_t* tile = lds;                      // the stage being read, and the other one
  const uint16_t* next = lds + T::kStageBytes / 2;

  for (;;) {
    // (a tile's first fragments: the last step of the one before has read them too, but they would take
    // registers from its epilogue)
#pragma clang loop unroll(full)
    for (int i = 0; i < kAhead; ++i) fa[i] = ra.read(tile, 0, i);
#pragma clang loop unroll(full)
    for (int j = 0; j < T::NT; ++j) fw[0][j] = rw.read(tile + TILE * BK, 0, j);
    floatx4 acc[T::MT][T::NT];
#pragma clang loop unroll(full)
    for (int i = 0; i < T::MT; ++i)
#pragma clang loop unroll(full)
      for (int j = 0; j < T::NT; ++j)
#pragma clang loop unroll(full)
        for (int v = 0; v < 4; ++v) acc[i][j][v] = 0.f;

    // ---- K loop
    // Lines of the tile's operands kTouch steps ahead that this block brings to the XCD's L2 for itself and
    // the blocks it shares them with, a wave up to 64: an epilogue's traffic on other CUs makes misses too
    // slow for the two stages.  (The cross layer above 1304 -> 1246 us, others 1 %; weight gradients,
    // whose epilogues are few, lose 2 %.)  Not where the tile is as wide as the output: nobody shares its rows of A
    // then, and asking for them twice is all it does (4 towers of 6 and 7 features to 256 outputs, batch 20000,
    // 54.9 against 64.9 us; 4 towers of 1024 columns, batch 16384, 37.5 against 45.8).
    constexpr bool kTouches = TILE == 256 && ALAY == OP_ROW && !DOTS;
    constexpr int kTouch = 4;
    uint32_t touch = kOobOffset;
    bool touches = false;
    if constexpr (kTouches) {
      const TmGroup& G = L.g[work.gi];
      const int tiles_n = (G.N + TILE - 1) / TILE, sm = tiles_n >= L.super ? 1 : L.super / tiles_n;
      const int line = (wave & 3) * 64 + lane;
      const bool a = wave < 4;                     // four waves A's lines, four W's
      const int part = a ? work.n0 / TILE : work.m0 / TILE % sm, parts = a ? tiles_n : sm;
      if (line >= part * TILE / parts && line < (part + 1) * TILE / parts) {
        if (a || WLAY == OP_ROW) touch = line < (a ? sa.rows : sw.rows) ? (uint32_t)line * (uint32_t)(a ? sa.ld : sw.ld) * 2u : kOobOffset;
        else if ((line & 3) * 64 < sw.rows) touch = ((uint32_t)(line >> 2) * (uint32_t)sw.ld + (line & 3) * 64) * 2u;
      }
      touches = __builtin_amdgcn_readfirstlane(G.K0 == 0 && tiles_n > 1 && __any(touch != kOobOffset));
    }
    for (int kt = 0; kt < nk; ++kt) {
      // The barrier of a K step sits in front of its last three rows of MFMAs, by when every wave has
      // read all it needs of the stage: behind it come the first requests for tile kt + 2 and
      // the first reads of tile kt + 1, and those rows cover both.
#pragma clang loop unroll(full)
      for (int r = 0; r < kRows; ++r) {
        const int kk = r / T::MT, i = r % T::MT;
        if (r == kRows - kAhead) {
          if (kTouches && touches && kt + kTouch < nk) {
            const int k1 = (kt + kTouch) * BK;
            tm_touch(lds0 + 2 * T::kStageBytes + wave * 4096, wave < 4 ? sa.buffer(k1, kl - k1) : sw.buffer(k1, kl - k1), touch);
            __builtin_amdgcn_s_waitcnt(0x0f71);    // vmcnt: all but the touch
          } else {
            __builtin_amdgcn_s_waitcnt(0x0f70);
          }
          __syncthreads();
        }
        if (r == kRows - kAhead - 2) aim();
        auto requests = [&]() __attribute__((always_inline)) {
          if (kn > 0)
#pragma clang loop unroll(full)
            for (int q = 0; q < kReqs; ++q)
              if ((q < kEarly ? kRows - kAhead + q / kPerRow : (q - kEarly) / kPerRow) == r) request(q);
        };
        if (kBurst) requests();
        if (r + kAhead < kRows) {
          fa[(r + kAhead) % 4] = ra.read(tile, (r + kAhead) / T::MT, (r + kAhead) % T::MT);
        } else {
          fa[(r + kAhead) % 4] = ra.read(next, 0, r + kAhead - kRows);
#pragma clang loop unroll(full)
          for (int j = 0; j < T::NT; ++j)
            if (j * kAhead / T::NT == r + kAhead - kRows) fw[0][j] = rw.read(next + TILE * BK, 0, j);
        }
#pragma clang loop unroll(full)
        for (int j = 0; j < T::NT; ++j)
          if ((TILE == 256 ? j + 1 : j / 2) == r) fw[1][j] = rw.read(tile + TILE * BK, 1, j);
        if (!kBurst) requests();
#pragma clang loop unroll(full)
        for (int jj = 0; jj < T::NT; ++jj) {
          const int j = i & 1 ? T::NT - 1 - jj : jj;
          acc[i][j] = mfma16<DT>(fw[kk][j], fa[r % 4], acc[i][j]);
        }
        __builtin_amdgcn_sched_barrier(0);         // (left alone, reads end up right in front of their use)
      }
      const uint16_t* const was = tile;
      tile = next;
      next = was;
    }

    // ---- epilogue, 16 rows x 64 columns of the wave's accumulators at a time: they go through 4 KB of
    // LDS of its own, so that its loads and stores of global memory cover whole lines (straight from the
    // registers, 64 bytes of 16 rows each: data gradients 1257 against 1066 us).  Chunk c (four columns)
    // of row r lies in slot c ^ r: 16 lanes that write one chunk of 16 rows or read 16 chunks of one
    // touch all banks once.  No barrier: the next tile's operands are landing beside it.
    const TmGroup& G = L.g[work.gi];
    const int m0 = work.m0, n0 = work.n0, slice = work.slice, M = G.M, N = G.N, epi = G.epi;
    // (opaque: what the branches below work out from either would otherwise be worked out ahead of the
    // loop over tiles, and kept in registers)
    int ln = lane;
    asm volatile("" : "+v"(ln));
    floatx4* const turn = (floatx4*)(lds + T::kStageBytes) + wave * 256;
    auto put = [&](int i) __attribute__((always_inline)) {
      wave_sync();
#pragma clang loop unroll(full)
      for (int j = 0; j < T::NT; ++j) turn[(ln & 15) * 16 + ((j * 4 + (ln >> 4)) ^ (ln & 15))] = acc[i][j];
      wave_sync();
    };
    auto get = [&](int r, int c) __attribute__((always_inline)) { return turn[r * 16 + (c ^ r)]; };
    const int wrow = wm * T::kHalf, wcol = wn * 64;
    if (whole && epi < EPI_F32 && (kForward || KIND == KIND_PLAIN)) {
      // 16-bit outputs: eight rows at a time, eight columns a lane.  What the cross epilogue reads (x0 and
      // x_l) is requested kDeep pieces ahead: more is more registers than a wave has beside its
      // accumulators.
      constexpr int kAll = T::MT * 2, kDeep = 8;
      const int r8 = ln >> 3, c = wcol + (ln & 7) * 8;
      const bool on = n0 + c < N;
      // byte addresses: the tile's corner (uniform, 64 bits) + an offset inside the tile
      char* const cbase = (char*)G.C + ((int64_t)m0 * G.ldc + n0) * 2;
      char* const ubase = (char*)G.U + ((int64_t)m0 * G.ldc + n0) * 2;
      const char* const xbase = (const char*)G.X0 + ((int64_t)m0 * G.ldx + n0) * 2;
      const char* const lbase = (const char*)G.XL + ((int64_t)m0 * G.ldxl + n0) * 2;
      constexpr bool cross = KIND == KIND_READS;
      uint4 bias_raw = make_uint4(0, 0, 0, 0), pa[kDeep], pb[kDeep];
      if (G.bias && on) bias_raw = dmt::gload((const uint4*)((const uint16_t*)G.bias + n0 + c));
      auto pack8 = [](const float (&y)[8]) __attribute__((always_inline)) {
        return make_uint4(dmt::pack2<DT>(y[0], y[1]), dmt::pack2<DT>(y[2], y[3]), dmt::pack2<DT>(y[4], y[5]), dmt::pack2<DT>(y[6], y[7]));
      };
      auto fetch = [&](int e) __attribute__((always_inline)) {
        // (rows and columns past the edge read in bounds and are not stored)
        const uint32_t m = (uint32_t)min(wrow + e * 8 + r8, M - 1 - m0), cc = on ? (uint32_t)c : 0u;
        pa[e % kDeep] = dmt::gload((const uint4*)(xbase + (m * (uint32_t)G.ldx + cc) * 2u));
        pb[e % kDeep] = dmt::gload((const uint4*)(lbase + (m * (uint32_t)G.ldxl + cc) * 2u));
      };
      if (cross)
#pragma clang loop unroll(full)
        for (int e = 0; e < kDeep - 1; ++e) fetch(e);
#pragma clang loop unroll(full)
      for (int e = 0; e < kAll; ++e) {
        const int r = wrow + e * 8 + r8;
        if (cross && e + kDeep - 1 < kAll) fetch(e + kDeep - 1);
        if (e % 2 == 0) put(e / 2);
        const floatx4 s0 = get(e % 2 * 8 + r8, (ln & 7) * 2), s1 = get(e % 2 * 8 + r8, (ln & 7) * 2 + 1);
        float y[8] = {s0[0], s0[1], s0[2], s0[3], s1[0], s1[1], s1[2], s1[3]}, bv[8];
        dmt::decode_chunk<DT>(bv, bias_raw);
#pragma clang loop unroll(full)
        for (int q = 0; q < 8; ++q) y[q] += bv[q];
        if (m0 + r < M && on) {
          const uint32_t off = ((uint32_t)r * (uint32_t)G.ldc + (uint32_t)c) * 2u;
          char* out = cbase + off;
          if (G.rdiv > 0) {
            const int m = m0 + r;
            out = (char*)G.C + ((int64_t)(m / G.rdiv) * G.ldc + (int64_t)(m % G.rdiv) * G.ldc2 + n0 + c) * 2;
          }
          if (epi == EPI_BIAS_RELU) {
#pragma clang loop unroll(full)
            for (int q = 0; q < 8; ++q) y[q] = y[q] > 0.f ? y[q] : 0.f;
          } else if constexpr (cross) {
            float xv[8], lv[8];
            if (G.U) dmt::gstore(pack8(y), (uint4*)(ubase + off));
            dmt::decode_chunk<DT>(xv, pa[e % kDeep]);
            dmt::decode_chunk<DT>(lv, pb[e % kDeep]);
#pragma clang loop unroll(full)
            for (int q = 0; q < 8; ++q) y[q] = xv[q] * y[q] + lv[q];
          }
          dmt::gstore(pack8(y), (uint4*)out);
        }
        __builtin_amdgcn_sched_barrier(0);
      }
    } else if (!kForward && whole) {
      // float32 outputs: four rows at a time, four columns a lane.  What a piece reads is requested kDeep
      // pieces ahead.
      constexpr int kAll = T::MT * 4;
      const int r4 = ln >> 4, c = wcol + (ln & 15) * 4;
      const bool on = n0 + c < N;
      const int64_t corner = (int64_t)m0 * G.ldc + n0;
      char* const cbase = (char*)((float*)G.C + slice * G.cstride + corner);
      // (rows and columns past the edge read in bounds and are not stored)
      auto place = [&](int e) __attribute__((always_inline)) {
        return (uint32_t)min(wrow + e * 4 + r4, M - 1 - m0) * (uint32_t)G.ldc + (on ? (uint32_t)c : 0u);
      };
      if constexpr (KIND != KIND_READS && KIND != KIND_SUMS) {
        constexpr int kDeep = 4;
        constexpr bool add = KIND == KIND_ADD;
        float4 old[kDeep];
        if (add)
#pragma clang loop unroll(full)
          for (int e = 0; e < kDeep - 1; ++e) old[e] = dmt::gload((const float4*)(cbase + place(e) * 4u));
#pragma clang loop unroll(full)
        for (int e = 0; e < kAll; ++e) {
          if (add && e + kDeep - 1 < kAll) old[(e + kDeep - 1) % kDeep] = dmt::gload((const float4*)(cbase + place(e + kDeep - 1) * 4u));
          if (e % 4 == 0) put(e / 4);
          const floatx4 s = get(e % 4 * 4 + r4, ln & 15);
          float4 g = make_float4(s[0], s[1], s[2], s[3]);
          if (add) {
            const float4 o = old[e % kDeep];
            g.x += o.x; g.y += o.y; g.z += o.z; g.w += o.w;
          }
          if (m0 + wrow + e * 4 + r4 < M && on) dmt::gstore(g, (float4*)(cbase + place(e) * 4u));
          __builtin_amdgcn_sched_barrier(0);
        }
      } else {
        // (ACC is 16 bytes a lane and piece more; at five pieces ahead the 256 x 256 instance would spill.  Read
        // where it is added instead, a tower of four layers of 2048 columns, batch 500, took 266 us, now 259.)
        constexpr int kDeep = KIND == KIND_SUMS && TILE == 256 ? 4 : 5;
        const char *gn = (const char*)(G.GN + corner), *ul = (const char*)G.UL + corner * 2;
        const char *x0 = (const char*)G.X0 + corner * 2, *u0 = (const char*)G.U0 + corner * 2;
        char *a0 = (char*)(G.ACC + corner), *du = (char*)G.DU + corner * 2;
        const bool has_gn = G.GN, has_u0 = G.U0, has_c = G.C, acc_old = KIND == KIND_SUMS && !G.acc_first;
        float4 pg[kDeep], po[kDeep];
        uint2 px[kDeep], pu[kDeep], pv[kDeep];
        auto fetch = [&](int e) __attribute__((always_inline)) {
          const uint32_t at = place(e);
          px[e % kDeep] = dmt::gload((const uint2*)(x0 + at * 2u));
          if (has_gn) {
            pg[e % kDeep] = dmt::gload((const float4*)(gn + at * 4u));
            pu[e % kDeep] = dmt::gload((const uint2*)(ul + at * 2u));
          }
          if (has_u0) pv[e % kDeep] = dmt::gload((const uint2*)(u0 + at * 2u));
          if (acc_old) po[e % kDeep] = dmt::gload((const float4*)(a0 + at * 4u));
        };
        float4 sums = make_float4(0.f, 0.f, 0.f, 0.f);
#pragma clang loop unroll(full)
        for (int e = 0; e < kDeep - 1; ++e) fetch(e);
#pragma clang loop unroll(full)
        for (int e = 0; e < kAll; ++e) {
          const int b = e % kDeep;
          if (e + kDeep - 1 < kAll) fetch(e + kDeep - 1);
          if (e % 4 == 0) put(e / 4);
          const floatx4 s = get(e % 4 * 4 + r4, ln & 15);
          if (m0 + wrow + e * 4 + r4 < M && on) {
            const uint32_t at = place(e);
            float4 g = make_float4(s[0], s[1], s[2], s[3]);
            float v0, v1, v2, v3;
            if (has_gn || has_u0) {
              float4 t = make_float4(0.f, 0.f, 0.f, 0.f);
              if (acc_old) t = po[b];
              if (has_gn) {
                const float4 n = pg[b];
                g.x += n.x; g.y += n.y; g.z += n.z; g.w += n.w;
                dmt::unpack2<DT>(pu[b].x, v0, v1);
                dmt::unpack2<DT>(pu[b].y, v2, v3);
                t.x += mul_rounded(n.x, v0); t.y += mul_rounded(n.y, v1);
                t.z += mul_rounded(n.z, v2); t.w += mul_rounded(n.w, v3);
              }
              if (has_u0) {
                dmt::unpack2<DT>(pv[b].x, v0, v1);
                dmt::unpack2<DT>(pv[b].y, v2, v3);
                t.x += mul_rounded(g.x, v0) + g.x; t.y += mul_rounded(g.y, v1) + g.y;
                t.z += mul_rounded(g.z, v2) + g.z; t.w += mul_rounded(g.w, v3) + g.w;
              }
              dmt::gstore(t, (float4*)(a0 + at * 4u));
            }
            dmt::unpack2<DT>(px[b].x, v0, v1);
            dmt::unpack2<DT>(px[b].y, v2, v3);
            const uint2 d = make_uint2(dmt::pack2<DT>(g.x * v0, g.y * v1), dmt::pack2<DT>(g.z * v2, g.w * v3));
            dmt::gstore(d, (uint2*)(du + at * 2u));
            dmt::unpack2<DT>(d.x, v0, v1);         // the bias gradient sums the rounded values
            dmt::unpack2<DT>(d.y, v2, v3);
            sums.x += v0; sums.y += v1; sums.z += v2; sums.w += v3;
            if (has_c) dmt::gstore(g, (float4*)(cbase + at * 4u));
          }
          if (e % 16 == 15) {
            // column sums of 64 rows: 16 of a lane, then the four lanes of its columns
            sums = make_float4(quarters_sum(sums.x), quarters_sum(sums.y), quarters_sum(sums.z), quarters_sum(sums.w));
            const int block = (m0 + wrow) / 64 + e / 16;
            if (r4 == 0 && block * 64 < M && on) dmt::gstore(sums, (float4*)(G.DBP + (int64_t)block * N + n0 + c));
            sums = make_float4(0.f, 0.f, 0.f, 0.f);
          }
          __builtin_amdgcn_sched_barrier(0);
        }
      }
    } else {
      // odd widths, unaligned rows: a column a lane, element by element; four rows' values are read before the first
      // is stored, and the column's bias once.  (Row by row, bias and all, 4 towers of 2048 columns to 257 outputs, batch
      // 4999, took 54.8 us, now 43.8; to 100 44.3, now 33.5.)
      const int n = n0 + wcol + ln;
      const float bias = epi < EPI_F32 && G.bias && n < N ? load_elt<DT>(G.bias, n) : 0.f;
#pragma clang loop unroll(full)
      for (int i = 0; i < T::MT; ++i) {
        put(i);
        for (int r0 = 0; r0 < 16; r0 += 4) {
          float v[4];
#pragma clang loop unroll(full)
          for (int q = 0; q < 4; ++q) v[q] = ((const float*)(turn + (r0 + q) * 16 + ((ln >> 2) ^ (r0 + q))))[ln & 3];
#pragma clang loop unroll(full)
          for (int q = 0; q < 4; ++q) {
            const int m = m0 + wrow + i * 16 + r0 + q;
            if (m >= M || n >= N) continue;
            const int64_t row = !DOTS && G.rdiv > 0 ? (int64_t)(m / G.rdiv) * G.ldc + (int64_t)(m % G.rdiv) * G.ldc2 : (int64_t)m * G.ldc;
            float y = v[q];
            if (!kForward && epi >= EPI_F32) {
              float* c = (float*)G.C + slice * G.cstride + row + n;
              *c = KIND == KIND_ADD ? *c + y : y;
              continue;
            }
            if (G.bias) y += bias;
            if (epi == EPI_BIAS_RELU) y = y > 0.f ? y : 0.f;
            if (kForward && KIND == KIND_READS) {
              if (G.U) store_elt<DT>(G.U, row + n, y);
              y = load_elt<DT>(G.X0, (int64_t)m * G.ldx + n) * y + load_elt<DT>(G.XL, (int64_t)m * G.ldxl + n);
            }
            store_elt<DT>(G.C, row + n, y);
          }
        }
      }
    }
    // the requests are at the next tile's second step, if there is one
    if (kn <= 0) return;
    work = ahead;
    measure();
  }
}

// ------------------------------------------------ MFMA grouped GEMM, small launches
//
// For forward launches of few tiles (a serving batch): a 128 x 128 tile per block would leave most
// CUs idle and walk all of K in one block.  A block takes a 32 x 32 tile and its eight waves an
// eighth of K each; operands go from global memory straight into registers (a lane feeds the matrix
// core 8 consecutive k of one row), the waves' sums are added in wave order through LDS.  Bound by
// the latencies of one load batch, the exchange and, with in-kernel dot terms (DOTS, as in tm_gemm:
// every block computes its 32 samples' terms itself), the Gram tiles before them.  Batch 61, 8 towers
// of 8 x 128 + 28 terms to 256 outputs: 27 -> 10.5 us (25 -> 9.2 back to back).
constexpr int kSmallWaves = 8;

// 8 elements at p; VEC: p is 16-byte aligned (else the rows of unpacked weights: any even address).
template <bool VEC> __device__ __forceinline__ uint4 small_load(const uint16_t* p) {
  if constexpr (VEC) return *(const uint4*)p;
  uint4 v;
  __builtin_memcpy(&v, p, 16);
  return v;
}

template <int DT, bool DOTS, int TAG = DMT_TM_TAG>
__global__ __launch_bounds__(kSmallWaves * 64, 4) void tm_gemm_small(const TmLaunch L) {
  __shared__ __attribute__((aligned(16))) float red[kSmallWaves][16][64];
  constexpr int kZPitch = BK + 8;
  __shared__ __attribute__((aligned(16))) uint16_t z[DOTS ? 32 * kZPitch : 8];
  int gi = 0;
  while (gi + 1 < L.ngroups && (int)blockIdx.x >= L.tile_start[gi + 1]) ++gi;
  const TmGroup& G = L.g[gi];
  const int tile = blockIdx.x - L.tile_start[gi], tiles_n = (G.N + 31) / 32;
  const int m0 = tile / tiles_n * 32, n0 = tile % tiles_n * 32;
  const int M = G.M, N = G.N;
  const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int r = lane & 31, h8 = (lane >> 5) * 8;
  const int m = min(m0 + r, M - 1), n = min(n0 + r, N - 1);     // rows past the edge: the last row, not stored
  const uint16_t* A1 = (const uint16_t*)G.A1 + (int64_t)m * G.lda1 + h8;
  const uint16_t* W1 = (const uint16_t*)G.W1 + (int64_t)n * G.ldw1 + h8;
  // this wave's steps of 16 k (K1 is a multiple of 8: the last step may be half empty)
  const int S = (G.K1 + 15) / 16, lo = S * wave / kSmallWaves, hi = S * (wave + 1) / kSmallWaves;
  const bool vec = (((uintptr_t)G.W1 & 15) | (G.ldw1 & 7)) == 0;
  floatx16 acc;
#pragma unroll
  for (int v = 0; v < 16; ++v) acc[v] = 0.f;
  constexpr int U = 4;
  uint4 a[U], w[U];
  auto load = [&](int s) __attribute__((always_inline)) {
#pragma unroll
    for (int u = 0; u < U; ++u) {
      const int k = (s + u) * 16;
      a[u] = w[u] = make_uint4(0, 0, 0, 0);
      if (s + u < hi && k + h8 < G.K1) {
        a[u] = *(const uint4*)(A1 + k);
        w[u] = vec ? small_load<true>(W1 + k) : small_load<false>(W1 + k);
      }
    }
  };
  if constexpr (!DOTS) load(lo);
  if constexpr (DOTS) {
    const int nf = G.nf, fd = G.fdim, spg = 32 / nf, K0 = G.K0, np = nf * (nf - 1) / 2;
    for (int e = threadIdx.x; e < 32 * kZPitch / 8; e += kSmallWaves * 64) ((uint4*)z)[e] = make_uint4(0, 0, 0, 0);
    __syncthreads();
    const uint16_t* A = (const uint16_t*)G.A1;
    const int sc = r / nf, j = r % nf;
    for (int s0 = wave * spg; s0 < 32; s0 += kSmallWaves * spg) {
      const int s = s0 + sc;
      const bool on = sc < spg && s < 32 && m0 + s < M;
      const uint16_t* xp = A + (on ? (int64_t)(m0 + s) * G.lda1 + j * fd + h8 : 0);
      floatx16 d;
#pragma unroll
      for (int v = 0; v < 16; ++v) d[v] = 0.f;
      for (int k = 0; k < fd; k += 128) {
        uint4 x[8];
#pragma unroll
        for (int u = 0; u < 8; ++u) {
          x[u] = make_uint4(0, 0, 0, 0);
          if (on && k + u * 16 + h8 < fd) x[u] = *(const uint4*)(xp + k + u * 16);
        }
#pragma unroll
        for (int u = 0; u < 8; ++u)
          if (k + u * 16 < fd) d = mfma32<DT>(x[u], x[u], d);
      }
#pragma unroll
      for (int v = 0; v < 16; ++v) {
        const int rr = (v >> 2) * 8 + (lane >> 5) * 4 + (v & 3), i = rr - sc * nf;
        if (i >= 0 && i < j && on) store_elt<DT>(z, s * kZPitch + i * (2 * nf - i - 1) / 2 + (j - i - 1), d[v]);
      }
    }
    load(lo);
    __syncthreads();
    // the dot terms' own steps, one per wave from the last
    const int s0 = kSmallWaves - 1 - wave;
    if (s0 * 16 < K0) {
      const int k = s0 * 16 + h8;
      uint4 wz = make_uint4(0, 0, 0, 0);
      if (k < np) {
        wz = small_load<false>((const uint16_t*)G.W0 + (int64_t)n * G.ldw0 + k);
        // (behind the terms' weights stand the pooled values': zeros, as the terms there are)
        uint32_t* const q = (uint32_t*)&wz;
#pragma unroll
        for (int i = 0; i < 4; ++i) q[i] = k + 2 * i + 1 < np ? q[i] : k + 2 * i < np ? q[i] & 0xffffu : 0u;
      }
      acc = mfma32<DT>(*(const uint4*)(z + r * kZPitch + k), wz, acc);
    }
    if (G.U && n0 == 0)                            // a training forward keeps the terms, zeros behind them
      for (int e = threadIdx.x; e < 32 * K0; e += kSmallWaves * 64)
        if (m0 + e / K0 < M) ((uint16_t*)G.U)[(int64_t)(m0 + e / K0) * K0 + e % K0] = z[e / K0 * kZPitch + e % K0];
  }
  for (int s = lo; s < hi; s += U) {
    uint4 ca[U], cw[U];
#pragma unroll
    for (int u = 0; u < U; ++u) { ca[u] = a[u]; cw[u] = w[u]; }
    load(s + U);
#pragma unroll
    for (int u = 0; u < U; ++u)
      if (s + u < hi) acc = mfma32<DT>(ca[u], cw[u], acc);
  }
#pragma unroll
  for (int v = 0; v < 16; ++v) red[wave][v][lane] = acc[v];
  __syncthreads();
  // lane holds column n0 + lane % 32 of rows (v / 4) * 8 + (lane / 32) * 4 + v % 4; two v a wave
  const int nn = n0 + r;
  if (nn >= N) return;
  const float bias = G.bias ? load_elt<DT>(G.bias, nn) : 0.f;
#pragma unroll
  for (int q = 0; q < 16 / kSmallWaves; ++q) {
    const int v = wave * (16 / kSmallWaves) + q, mm = m0 + (v >> 2) * 8 + (lane >> 5) * 4 + (v & 3);
    if (mm >= M) continue;
    float y = red[0][v][lane];
#pragma unroll
    for (int p = 1; p < kSmallWaves; ++p) y += red[p][v][lane];
    y += bias;
    const int64_t row = G.rdiv > 0 ? (int64_t)(mm / G.rdiv) * G.ldc + (int64_t)(mm % G.rdiv) * G.ldc2 : (int64_t)mm * G.ldc;
    if (G.epi == EPI_BIAS_RELU) y = y > 0.f ? y : 0.f;
    if (G.epi == EPI_CROSS) {
      if (G.U) store_elt<DT>(G.U, row + nn, y);
      y = load_elt<DT>(G.X0, (int64_t)mm * G.ldx + nn) * y + load_elt<DT>(G.XL, (int64_t)mm * G.ldxl + nn);
    }
    store_elt<DT>(G.C, row + nn, y);
  }
}

// ------------------------------------------------------------ pairwise dot terms

// Per-tower work of a grouped auxiliary launch (dot terms or weight repack).
struct TmAuxItem {
  const void* src;
  void* dst;
  int32_t nf, n, np, np_pad;   // dots: features, dim, real and padded term count
  int32_t O, wt;               // pack: output rows, tower width
};

struct TmAuxLaunch {
  int32_t ngroups;
  int32_t block_start[kMaxGroups + 1];
  int64_t B;
  TmAuxItem g[kMaxGroups];
};

__device__ __forceinline__ int aux_group(const TmAuxLaunch& L) {
  int gi = 0;
  while (gi + 1 < L.ngroups && (int)blockIdx.x >= L.block_start[gi + 1]) ++gi;
  return gi;
}

// z[s][p(i,j)] = <x[s][i][:], x[s][j][:]>, i < j, p row-major; x is [B][nf][n] contiguous.
// A wave takes 32 / nf samples: their (sample, feature) rows are the rows of one 32 x 32 Gram
// tile, whose diagonal nf x nf blocks hold every sample's dots, so the operand is read once,
// straight from global memory, as both A and B (where nf does not divide 32 the last 32 % nf
// rows of the tile are idle).  Needs nf <= 32 and n a multiple of 8.  Columns np .. np_pad-1 of z
// are zeroed.  For 6 and 7 features of 128 columns, batch 2003, against one thread per (sample,
// term): 65.6 -> 7.2 us.
template <int DT>
__global__ __launch_bounds__(kBlock) void tm_dots_mfma(const TmAuxLaunch L) {
  const int gi = aux_group(L);
  const TmAuxItem& G = L.g[gi];
  const int64_t B = L.B;
  const int nf = G.nf, n = G.n, np = G.np, np_pad = G.np_pad;
  void* __restrict__ z = G.dst;
  const int lane = threadIdx.x & 63;
  const int64_t rg = (int64_t)(blockIdx.x - L.block_start[gi]) * (kBlock / 64) + (threadIdx.x >> 6);
  const int spg = 32 / nf;                         // samples per Gram tile
  const int64_t s0 = rg * spg;
  if (s0 >= B) return;
  const int c = lane & 31, sc = c / nf, j = c % nf;
  const bool on = sc < spg && s0 + sc < B;
  const int64_t row = on ? s0 * nf + c : 0;        // (idle rows read row 0 and count as zeros)
  floatx16 acc;
#pragma unroll
  for (int v = 0; v < 16; ++v) acc[v] = 0.f;
  if constexpr (DT == DMT_F32) {
    const float* xp = (const float*)G.src + row * n + (lane >> 5) * 4;
    for (int k = 0; k < n; k += 8) {
      float4 a = make_float4(0.f, 0.f, 0.f, 0.f);
      if (on) a = *(const float4*)(xp + k);
      acc = __builtin_amdgcn_mfma_f32_32x32x2f32(a.x, a.x, acc, 0, 0, 0);
      acc = __builtin_amdgcn_mfma_f32_32x32x2f32(a.y, a.y, acc, 0, 0, 0);
      acc = __builtin_amdgcn_mfma_f32_32x32x2f32(a.z, a.z, acc, 0, 0, 0);
      acc = __builtin_amdgcn_mfma_f32_32x32x2f32(a.w, a.w, acc, 0, 0, 0);
    }
  } else {
    const int h8 = (lane >> 5) * 8;
    const uint16_t* xp = (const uint16_t*)G.src + row * n + h8;
    for (int k = 0; k < n; k += 64) {
      uint4 a[4];
#pragma unroll
      for (int u = 0; u < 4; ++u) {
        a[u] = make_uint4(0, 0, 0, 0);
        if (on && k + u * 16 + h8 < n) a[u] = *(const uint4*)(xp + k + u * 16);
      }
#pragma unroll
      for (int u = 0; u < 4; ++u) acc = mfma32<DT>(a[u], a[u], acc);
    }
  }
#pragma unroll
  for (int v = 0; v < 16; ++v) {
    const int rr = (v >> 2) * 8 + (lane >> 5) * 4 + (v & 3), i = rr - sc * nf;
    if (i >= 0 && i < j && on)
      store_elt<DT>(z, (s0 + sc) * np_pad + (i * (2 * nf - i - 1) / 2 + (j - i - 1)), acc[v]);
  }
  // zeros behind the terms of the wave's samples (2 features: 16 samples x 7 columns, more than
  // one per lane)
  const int npad = np_pad - np;
  for (int e = lane; e < spg * npad; e += 64) {
    const int s = e / npad, q = e % npad;
    if (s0 + s < B) store_elt<DT>(z, (s0 + s) * np_pad + np + q, 0.f);
  }
}

// Whether tm_dots_mfma serves nf features of n columns, and the blocks it takes.
inline bool dots_mfma_ok(int nf, int n) { return nf >= 2 && nf <= 32 && n % 8 == 0; }
inline int64_t dots_mfma_blocks(int64_t B, int nf) {
  const int64_t waves = (B + 32 / nf - 1) / (32 / nf);
  return (waves + kBlock / 64 - 1) / (kBlock / 64);
}

// Any nf / n, any dtype: one thread per (sample, term).
template <int DT>
__global__ __launch_bounds__(kBlock) void tm_dots_simple(const TmAuxLaunch L) {
  const int gi = aux_group(L);
  const TmAuxItem& G = L.g[gi];
  const int nf = G.nf, n = G.n, np = G.np, np_pad = G.np_pad;
  const int64_t e = (int64_t)(blockIdx.x - L.block_start[gi]) * kBlock + threadIdx.x;
  if (e >= L.B * np_pad) return;
  const int64_t s = e / np_pad;
  const int p = (int)(e % np_pad);
  float d = 0.f;
  if (p < np) {
    int i = 0, rem = p;
    while (rem >= nf - 1 - i) { rem -= nf - 1 - i; ++i; }
    const int j = i + 1 + rem;
    const int64_t bi = (s * nf + i) * n, bj = (s * nf + j) * n;
    for (int k = 0; k < n; ++k) d += load_elt<DT>(G.src, bi + k) * load_elt<DT>(G.src, bj + k);
  }
  store_elt<DT>(G.dst, e, d);
}

// Projection weights [O][np + Wt] -> [O][np_pad + Wt] with zero columns after the
// dot terms, so both K segments start 16-byte aligned.  (Wt = 0: rows of np elements padded to np_pad.)
template <int DT>
__global__ __launch_bounds__(kBlock) void tm_pack_w(const TmAuxLaunch L) {
  const int gi = aux_group(L);
  const TmAuxItem& G = L.g[gi];
  const int np = G.np, np_pad = G.np_pad, wt = G.wt;
  const int64_t e = (int64_t)(blockIdx.x - L.block_start[gi]) * kBlock + threadIdx.x;
  const int kp = np_pad + wt;
  if (e >= (int64_t)G.O * kp) return;
  const int o = (int)(e / kp), k = (int)(e % kp);
  const int64_t src = (int64_t)o * (np + wt) + (k < np ? k : np + (k - np_pad));
  ((uint16_t*)G.dst)[e] = (k >= np && k < np_pad) ? (uint16_t)0 : ((const uint16_t*)G.src)[src];
}

// Whether a dot tower's projection weights ([O][np + wt], 16-bit) can be read as they are: both
// pieces of a row then start on a 4-byte boundary, which is what the straight-to-LDS loads need.
// Otherwise (an odd number of dot terms) they are repacked by tm_pack_w first.
inline bool dot_weights_as_is(const void* w_proj, int np) { return np % 2 == 0 && ((uintptr_t)w_proj & 3) == 0; }

// ---- The dot towers' data gradient in one kernel (tmb_dot_dgrad): its shape, and the towers that take it.
constexpr int kDotFeat = 8;                        // features, at most
constexpr int kDotTerms = kDotFeat * (kDotFeat - 1) / 2, kDotTermTiles = (kDotTerms + 15) / 16;
constexpr int kDotCols = 32;                       // columns of a feature that a block takes
constexpr int kDotTiles = kDotFeat * (kDotCols / 16) + kDotTermTiles;
constexpr int dot_rows(int S) { return 4 * 16 * S; }
// (32-bit byte offsets into a column block's weights)
inline bool dot_dgrad_ok(const dmt_plan* p, int nf, int n, int64_t O) {
  return p->sw.tm_fuse && nf >= 2 && nf <= kDotFeat && n % kDotCols == 0 && (O + 31) / 32 * kDotTiles * 1024 < (1LL << 31);
}
// The towers that it could serve, its blocks of 64 samples for all of them, their elements, and whether the call has
// other towers whose data gradients are plain contractions, dot towers among them.
struct DotDgrad {
  int towers = 0;
  int64_t blocks = 0, elements = 0;
  bool beside = false, beside_dots = false;
};
inline DotDgrad dot_dgrad_of(const dmt_plan* p, const dmt_tm_params* tp, int64_t B) {
  DotDgrad d;
  for (int32_t t = 0; t < p->T; ++t) {
    const bool dot = tp[t].kind == DMT_TM_DOT_LINEAR;
    if (dot && dot_dgrad_ok(p, p->tower_ntab[t], p->tower_uniform_dim[t], tp[t].out_dim)) {
      ++d.towers;
      d.blocks += (B + dot_rows(1) - 1) / dot_rows(1) * (p->tower_uniform_dim[t] / kDotCols);
      d.elements += B * p->tower_ntab[t] * p->tower_uniform_dim[t];
    } else if (tp[t].kind != DMT_TM_CROSS_LINEAR && tp[t].kind != DMT_TM_CROSS_LOWRANK_LINEAR) {
      d.beside = true;
      d.beside_dots = d.beside_dots || dot;
    }
  }
  return d;
}
// Whether it is the faster one for nf features to O outputs.  A step of 32 outputs takes a lone block longer than the
// contractions' tiles take, which costs more the longer it goes on and the fewer blocks there are.  Backward, us,
// separate kernels / this one: 4 towers of 8 features, 32 columns, 16 blocks, 64 outputs 24.0 / 21.8, 256 26.3 / 26.9, 2048
// 54.4 / 75.6; 64 blocks, 256 33.7 / 32.1, 512 38.4 / 41.4; 128 blocks, 512 45.5 / 43.7, 1024 62.7 / 66.0; 64 columns, 256
// blocks, 1024 73.9 / 73.0, 2048 107.9 / 118.4; 384 blocks, 2048 167 / 147 (128 columns 129 / 134); one tower, 4 blocks, 5
// features, 256 22.8 / 21.8, 700 27.9 / 31.3.  More towers than one launch of contractions holds with their dot terms
// take two: 12 of 2 and 7 features, 24 blocks, 700 50.1 / 41.0 and 59.2 / 54.3.
// Beside towers whose contractions are launched all the same (a cross tower's are a launch of their own) it is one launch
// more, beside other dot towers, which keep tmb_dot_bwd8, a longer one, and has to save that many bytes: 8 features of 32, 64
// and 128 columns beside a linear tower, 256 outputs, 2^20 elements 35.8 / 41.1, 37.3 / 41.9 and 37.4 / 43.5, 2^21 47.1 /
// 46.2, 43.7 / 42.4 and 41.8 / 44.5, 2^22 66.1 / 58.5, 62.7 / 55.0 and 51.9 / 47.2; beside 10 features 2^21 57.9 / 59.7,
// 53.0 / 57.6 and 48.2 / 55.4, 2^22 85.6 / 84.8, 75.8 / 79.0 and 67.6 / 71.2, 2^23 of 64 and 128 columns 141 / 114 and 119 / 100.
inline bool dot_dgrad_pays(const dmt_plan* p, int nf, int64_t O, const DotDgrad& all) {
  if (p->sw.tm_fuse == 2 || 2 * all.towers > kMaxGroups) return true;
  if (all.beside && all.elements < (all.beside_dots ? 4000000 : 1 << 21)) return false;
  return O <= std::max<int64_t>(6 * all.blocks, 1280 / nf);
}
// Of a dot tower t in a 16-bit type.
inline bool dot_one_kernel(const dmt_plan* p, int t, int64_t O, const DotDgrad& all) {
  return dot_dgrad_ok(p, p->tower_ntab[t], p->tower_uniform_dim[t], O) && dot_dgrad_pays(p, p->tower_ntab[t], O, all);
}

// What a training forward keeps for the backward: for every cross layer l of a cross tower
// (full-rank or low-rank), x_{l+1} and u_l = W_l x_l + b_l, each [B][W_t] in the compute type;
// for a dot-product tower its dot terms, [B][np_pad] (np_pad = the F (F - 1) / 2 terms rounded
// up to 8, zeros behind them), and, where its backward reads them so whatever their address (an odd number of terms,
// 16-bit types, not tmb_dot_dgrad), its projection weights with zero columns inserted to match, [O][np_pad + W_t].
// Offsets in bytes from a 256-byte-aligned base; towers of other kinds keep nothing (their backward needs only the pooled
// values).
struct TmKept {
  size_t x[DMT_MAX_CROSS_LAYERS] = {}, u[DMT_MAX_CROSS_LAYERS] = {};
  size_t z = 0, wp = 0;      // dot tower: dot terms, and the projection weights as repacked for them
  bool has_z = false, has_wp = false;
};

inline size_t plan_tm_kept(const dmt_plan* p, const dmt_tm_params* tp, int64_t B, int eb,
                           std::vector<TmKept>* kept) {
  size_t off = 0;
  kept->assign(p->T, TmKept());
  const DotDgrad dots = dot_dgrad_of(p, tp, B);
  for (int32_t t = 0; t < p->T; ++t) {
    if (tp[t].kind == DMT_TM_DOT_LINEAR) {
      const int nf = p->tower_ntab[t], np_pad = (nf * (nf - 1) / 2 + 7) / 8 * 8;
      if (np_pad > 0) {
        (*kept)[t].z = off;
        (*kept)[t].has_z = true;
        off += dmt_align_up((size_t)B * np_pad * eb, 256);
        (*kept)[t].has_wp = eb == 2 && nf * (nf - 1) / 2 % 2 == 1 && !dot_one_kernel(p, t, tp[t].out_dim, dots);
        (*kept)[t].wp = off;
        if ((*kept)[t].has_wp) off += dmt_align_up((size_t)tp[t].out_dim * (np_pad + p->tower_width[t]) * eb, 256);
      }
      continue;
    }
    if (tp[t].kind != DMT_TM_CROSS_LINEAR && tp[t].kind != DMT_TM_CROSS_LOWRANK_LINEAR) continue;
    const size_t bytes = dmt_align_up((size_t)B * p->tower_width[t] * eb, 256);
    for (int l = 0; l < tp[t].num_cross_layers && l < DMT_MAX_CROSS_LAYERS; ++l) {
      (*kept)[t].x[l] = off; off += bytes;
      (*kept)[t].u[l] = off; off += bytes;
    }
  }
  return off;
}

// Launches of tm_gemm.
template <int DT, int TILE, int ALAY, int WLAY, int KIND, bool DOTS, bool KEEPZ>
void launch_tiles(const TmLaunch& L, int64_t blocks, hipStream_t s) {
  constexpr int bytes = TmTile<TILE>::kLdsBytes;
  auto kernel = tm_gemm<DT, TILE, ALAY, WLAY, KIND, DOTS, KEEPZ>;
  static DmtPerDevice configured;
  dmt_allow_lds(configured, (const void*)kernel, bytes);
  hipLaunchKernelGGL(kernel, dim3((unsigned)blocks), dim3(TmTile<TILE>::kThreads), bytes, s, L);
}

inline int64_t tiles_of(const TmGroup& g, int tile) {
  return (int64_t)((g.M + tile - 1) / tile) * ((g.N + tile - 1) / tile) * tm_slices(g);
}

// Whether every tile of a launch has the same number of K steps, and two at least.
constexpr int kCUs = 256;
inline bool same_steps(const TmGroup* g, int n) {
  int64_t steps = 0;
  for (int i = 0; i < n; ++i) {
    const bool split = g[i].ksplit > 1;
    const int64_t first = split ? g[i].klen : g[i].K1, last = split ? g[i].K1 - (int64_t)(g[i].ksplit - 1) * g[i].klen : first;
    const int64_t k0 = (g[i].K0 + BK - 1) / BK, s = k0 + (first + BK - 1) / BK;
    if (k0 + (last + BK - 1) / BK < 2 || (steps != 0 && s != steps)) return false;
    steps = s;
  }
  return true;
}

// Whether a launch takes 256 x 256 tiles: when there are at least kBigTiles of them (three for every four CUs), or
// when 128 x 128 tiles of equal K would be more than the kMidSlots blocks that are resident together, and no group is
// so narrow that half of every tile would be empty.  Both sides measured (forward, 128 x 128 / 256 x 256 tiles, us): 4
// linear towers of 1024 columns, 448 mid tiles 22.1 / 30.9, 528 (132 big ones) 37.1 / 31.2, of 256 columns 11.3 / 16.5
// and 19.4 / 16.9; dots and K = 1052, 512 mid tiles 40.2 / 48.4, 528 77.2 / 49.1.  Cross layers' second round is
// short beside their epilogues: 4 towers of 2048 columns, 640 mid tiles (160 big ones) 156.3 / 162.9, from 192 big
// ones on 164.6 / 139.8; towers of unequal K even out better in the smaller tiles (3 to 20 tables, 576 mid tiles
// 30.2 / 38.0).
constexpr int kBigTiles = 192, kMidSlots = 512;
inline bool take_big(const dmt_plan* p, const TmGroup* g, int n) {
  if (p->sw.tm_big == 0) return false;
  int64_t tiles = 0, mid = 0;
  bool plain = true;
  for (int i = 0; i < n; ++i) {
    if (g[i].M <= 128 || g[i].N <= 128) return false;
    tiles += tiles_of(g[i], 256);
    mid += tiles_of(g[i], 128);
    plain = plain && (g[i].epi == EPI_BIAS || g[i].epi == EPI_BIAS_RELU);
  }
  return tiles >= kBigTiles || (plain && mid > kMidSlots && same_steps(g, n)) || p->sw.tm_big == 2;
}

// Whether a forward launch goes to tm_gemm_small: up to 512 tiles of 32 x 32, two for every CU; 768 of cross layers,
// 1024 with dot terms, which a 128 x 128 tile takes longer over.  Both sides measured (128 x 128 / 32 x 32 tiles, us):
// one segment, K = 1024, 512 tiles 13.7 / 12.0, 576 tiles 13.8 / 16.5, K = 2048 21.5 / 21.5 and 21.7 / 29.2, K = 512,
// 768 tiles 10.1 / 10.2; cross layers of 4 towers of 1024 columns, 768 tiles 46.5 / 42.5, 896 tiles 46.4 / 49.3; dots
// and K = 1052, 1024 tiles 30.2 / 28.6, 1152 tiles 30.1 / 32.9, 4 features of 32, 1024 tiles 14.4 / 11.5, 1152 tiles
// 14.4 / 14.4.
constexpr int kSmallTiles = 512;
inline bool take_small(const dmt_plan* p, const TmGroup* g, int n, bool dots) {
  if (p->sw.tm_big != 1) return p->sw.tm_big == 3;
  int64_t tiles = 0;
  bool cross = true;
  for (int i = 0; i < n; ++i) {
    tiles += tiles_of(g[i], 32);
    cross = cross && g[i].epi == EPI_CROSS;
  }
  return tiles <= (dots ? 1024 : cross ? 768 : kSmallTiles);
}

// Cuts a launch's groups into tiles and deals them out; how many blocks it takes.
inline int64_t tile_launch(const dmt_plan* p, TmLaunch& L, bool dots, int kind, bool* big_tiles) {
  const bool big = *big_tiles = take_big(p, L.g, L.ngroups);
  const int tile = big ? 256 : 128;
  int64_t tiles = 0;
  for (int i = 0; i < L.ngroups; ++i) tiles += tiles_of(L.g[i], tile);
  // super-tiles as large as an XCD's resident blocks, or an eighth of the launch where that is less
  const int resident = big ? 32 : 64;
  L.super = (int32_t)std::max<int64_t>(1, std::min<int64_t>(resident, (tiles + 7) / 8));
  L.cap = 1;
  int64_t nst = 0;
  for (int i = 0; i < L.ngroups; ++i) {
    L.tile_start[i] = (int32_t)nst;
    const int64_t tn = (L.g[i].N + tile - 1) / tile, tm = (int64_t)((L.g[i].M + tile - 1) / tile) * tm_slices(L.g[i]);
    const int64_t sm = tn >= L.super ? 1 : L.super / tn;
    L.cap = (int32_t)std::max<int64_t>(L.cap, std::min(sm, tm) * tn);
    nst += (tm + sm - 1) / sm;
  }
  L.tile_start[L.ngroups] = (int32_t)nst;
  int64_t blocks = (nst + 7) / 8 * 8 * L.cap;
  if (blocks == 0) return 0;
  L.slots = (int32_t)(blocks / 8);
  L.stagger = 0;
  // One block per CU works through a launch's 256 x 256 tiles where their K is equal (blocks that are handed out a
  // tile at a time even differences out) and two steps at least, so that the requests are never more than one tile
  // ahead, and where few slots are without a tile: they would leave their blocks idle.
  if (big && !dots && tiles > kCUs && nst * L.cap <= tiles + tiles / 16 && same_steps(L.g, L.ngroups)) {
    // (The last XCD starts 57 K cycles late: a third of a tile of 32 K steps, about a whole one of four.  Eight
    // rounds and more make up for that: cross layers of rank 256 and 128, 12 rounds, 1088 against 1082 us and 971
    // against 951 with none, 16 rounds 1284 / 1305 and 1148 / 1161, rank 512 and 1024 1 % less.)
    if (kind != KIND_PLAIN && tiles >= 8 * kCUs) L.stagger = 2;
    blocks = kCUs;
  }
  L.step = (int32_t)(blocks / 8);
  return blocks;
}

// All groups of the list, kMaxGroups to a launch.  dots: every group computes its dot terms itself.
template <int DT, int ALAY = OP_ROW, int WLAY = OP_ROW>
void launch_groups(const dmt_plan* p, std::vector<TmGroup>& groups, hipStream_t s, bool dots = false,
                   int kid = DMT_K_TM_GEMM) {
  // (towers of several forms may share a stage; their epilogues are kernels of their own)
  std::stable_sort(groups.begin(), groups.end(), [](const TmGroup& a, const TmGroup& b) { return epi_kind(a.epi) < epi_kind(b.epi); });
  for (size_t first = 0, end; first < groups.size(); first = end) {
    const int kind = epi_kind(groups[first].epi);
    for (end = first + 1; end < groups.size() && end < first + kMaxGroups && epi_kind(groups[end].epi) == kind; ++end) {}
    TmLaunch L;
    L.ngroups = (int32_t)(end - first);
    bool keepz = false;                           // a training forward keeps the dot terms
    for (int i = 0; i < L.ngroups; ++i) {
      L.g[i] = groups[first + i];
      keepz = keepz || (dots && L.g[i].U != nullptr);
    }
    if constexpr (ALAY == OP_ROW && WLAY == OP_ROW && DMT_TM_TAG == 0) {
      // (in-kernel dot terms, or one K segment)
      bool small = take_small(p, L.g, L.ngroups, dots);
      for (int i = 0; i < L.ngroups; ++i) small = small && (dots || L.g[i].K0 == 0);
      if (small) {
        int64_t blocks = 0;
        for (int i = 0; i < L.ngroups; ++i) {
          L.tile_start[i] = (int32_t)blocks;
          blocks += tiles_of(L.g[i], 32);
        }
        L.tile_start[L.ngroups] = (int32_t)blocks;
        DmtScope scope(p, kid, s);
        if (dots) hipLaunchKernelGGL((tm_gemm_small<DT, true>), dim3((unsigned)blocks), dim3(kSmallWaves * 64), 0, s, L);
        else hipLaunchKernelGGL((tm_gemm_small<DT, false>), dim3((unsigned)blocks), dim3(kSmallWaves * 64), 0, s, L);
        continue;
      }
    }
    bool big;
    const int64_t blocks = tile_launch(p, L, dots, kind, &big);
    if (blocks == 0) continue;
    DmtScope scope(p, kid, s);
    if constexpr (ALAY == OP_ROW && WLAY == OP_ROW && DMT_TM_TAG == 0) {
      if (dots && big && keepz) { launch_tiles<DT, 256, ALAY, WLAY, KIND_PLAIN, true, true>(L, blocks, s); continue; }
      if (dots && big) { launch_tiles<DT, 256, ALAY, WLAY, KIND_PLAIN, true, false>(L, blocks, s); continue; }
      if (dots && keepz) { launch_tiles<DT, 128, ALAY, WLAY, KIND_PLAIN, true, true>(L, blocks, s); continue; }
      if (dots) { launch_tiles<DT, 128, ALAY, WLAY, KIND_PLAIN, true, false>(L, blocks, s); continue; }
    }
    if constexpr (ALAY == OP_ROW && WLAY == OP_COL) {
      bool sums = false;
      for (int i = 0; i < L.ngroups; ++i) sums = sums || epi_sums(L.g[i]);
      if (sums && big) { launch_tiles<DT, 256, ALAY, WLAY, KIND_SUMS, false, false>(L, blocks, s); continue; }
      if (sums) { launch_tiles<DT, 128, ALAY, WLAY, KIND_SUMS, false, false>(L, blocks, s); continue; }
      if (kind == KIND_ADD && big) { launch_tiles<DT, 256, ALAY, WLAY, KIND_ADD, false, false>(L, blocks, s); continue; }
      if (kind == KIND_ADD) { launch_tiles<DT, 128, ALAY, WLAY, KIND_ADD, false, false>(L, blocks, s); continue; }
    }
    if constexpr (ALAY == OP_ROW) {
      if (kind == KIND_READS && big) { launch_tiles<DT, 256, ALAY, WLAY, KIND_READS, false, false>(L, blocks, s); continue; }
      if (kind == KIND_READS) { launch_tiles<DT, 128, ALAY, WLAY, KIND_READS, false, false>(L, blocks, s); continue; }
    }
    if (big) launch_tiles<DT, 256, ALAY, WLAY, KIND_PLAIN, false, false>(L, blocks, s);
    else launch_tiles<DT, 128, ALAY, WLAY, KIND_PLAIN, false, false>(L, blocks, s);
  }
  groups.clear();
}

// Grouped launch of the dot-term (which = 0: Gram tiles on MFMA, 1: plain FMA) or weight-repack
// (which = 2) kernels over `items`; nblocks[i] blocks serve items[i].
template <int DT>
void launch_aux(const dmt_plan* p, int64_t B, std::vector<TmAuxItem>& items,
                std::vector<int64_t>& nblocks, int which, hipStream_t s) {
  for (size_t first = 0; first < items.size(); first += kMaxGroups) {
    TmAuxLaunch L;
    L.B = B;
    L.ngroups = (int32_t)std::min<size_t>(kMaxGroups, items.size() - first);
    int32_t blocks = 0;
    for (int i = 0; i < L.ngroups; ++i) {
      L.g[i] = items[first + i];
      L.block_start[i] = blocks;
      blocks += (int32_t)nblocks[first + i];
    }
    L.block_start[L.ngroups] = blocks;
    if (blocks == 0) continue;
    if (which == 0) {
      DmtScope scope(p, DMT_K_TM_DOTS, s);
      hipLaunchKernelGGL((tm_dots_mfma<DT>), dim3(blocks), dim3(kBlock), 0, s, L);
    } else if (which == 1) {
      DmtScope scope(p, DMT_K_TM_DOTS, s);
      hipLaunchKernelGGL((tm_dots_simple<DT>), dim3(blocks), dim3(kBlock), 0, s, L);
    } else {
      DmtScope scope(p, DMT_K_TM_PACK, s);
      hipLaunchKernelGGL((tm_pack_w<DT>), dim3(blocks), dim3(kBlock), 0, s, L);
    }
  }
}

}  // namespace
