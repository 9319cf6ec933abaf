// Grouped contractions of the Tower Module, shared by its forward and backward:
//   C = epilogue(A . W^T [+ b]), either operand contiguous along the reduction dimension or along
// its own, one launch for all towers of a stage (block id -> tower, tile).
// 16-bit types run on MFMA (v_mfma_f32_32x32x16, float32 accumulate); float32 has its own kernel
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
  // EPI_CROSS_GRAD: [M][ldc] float32 / 16-bit tensors, and the column sums of du, one row per 128 rows
  // of C
  const float* GN;        // g_{l+1} or NULL
  const void* UL;         // u_l (with GN)
  const void* U0;         // u_0 or NULL
  float* ACC;
  void* DU;
  float* DBP;             // [(M + 127) / 128][N]
  int32_t acc_first;      // ACC holds nothing yet
  // Two-level output rows: with rdiv > 0 row m of C starts at (m / rdiv) * ldc + (m % rdiv) * ldc2,
  // i.e. rdiv consecutive rows of the contraction share one row of the output tensor.
  int32_t rdiv, ldc2;
};

__host__ __device__ inline int tm_slices(const TmGroup& g) { return g.ksplit > 1 ? g.ksplit : 1; }
// The first k behind the slice that starts at kofs < K1.  (kofs + klen may lie up to a K step per slice past
// K1, which itself may be next to 2^31.)
__host__ __device__ inline int tm_slice_end(int K1, int kofs, int klen) {
  return klen < K1 - kofs ? kofs + klen : K1;
}

struct TmLaunch {
  int32_t ngroups;
  int32_t super;                       // tiles of a super-tile (dealt to one XCD), at most
  int32_t cap;                         // block slots of a super-tile
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
// Operand tiles go from global memory straight into LDS (buffer_load_dwordx4 ... lds: a wave's 64
// lanes fill 1 KB of consecutive LDS, 16 bytes a lane), two stages deep: tile kt + 2 is requested
// into the stage tile kt is being read from, behind the barrier inside step kt, and every wave waits
// for its own requests before the next step's barrier.  The buffer's bounds stand in for all edges:
// rows past the operand's last, and chunks past the last k (their lanes ask for an offset that is
// never in bounds), arrive as zeros.  (The requests are inline assembly: told about them, the
// compiler makes every LDS read of the current tile wait for the next tile's requests, since it
// cannot tell the two stages apart.)
//
// OP_ROW tile: 128-byte rows (64 k) without padding; column chunk c (8 elements) of row r sits in
// slot c ^ (r / 2) % 8.  A fragment read (ds_read_b128, 16 lanes a cycle from 64 banks) touches 16
// rows: 2 r and 2 r + 1 lie in the two halves of one 256-byte bank row and share a slot, the eight
// pairs differ in it, so it is conflict-free.
// OP_COL tile: 64 rows of BM (BN) elements, one per k; chunk c of row k sits in slot
// c ^ 4 (k % 4).  Fragments come through ds_read_b64_tr_b16, which transposes 4 x 4 blocks among 16
// lanes: lane p of a group names row k + p / 4, elements 4 (p % 4) ..., and receives column p of the
// four rows.  The four rows of a group lie on the same banks but for the slot, which spreads them.
//
// The MFMAs take the W fragment as their first operand, so the accumulators hold the tile
// transposed: a lane owns one row and four consecutive columns per register quad, which the
// epilogue parks in LDS with 16-byte stores.

// TAG only marks the including source file in the kernel's name, so that a profile tells the
// forward's launches from the backward's.
#ifndef DMT_TM_TAG
#define DMT_TM_TAG 0
#endif

constexpr uint32_t kOobOffset = 0x80000000u;      // beyond any buffer (256 rows of a tile stay far below it)

// Buffer descriptor of `bytes` bytes from p (uniform).
__device__ __forceinline__ __amdgpu_buffer_rsrc_t tm_buffer(const void* p, uint32_t bytes) {
  return __builtin_amdgcn_make_buffer_rsrc((void*)p, 0, (int)bytes, 0x00020000);
}
// 64 lanes' 16-byte pieces of a buffer to 1 KB of LDS at byte address lds.
__device__ __forceinline__ void tm_request(uint32_t lds, __amdgpu_buffer_rsrc_t rsrc, uint32_t off) {
  asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tbuffer_load_dwordx4 %1, %2, 0 offen lds"
               :: "s"(__builtin_amdgcn_readfirstlane(lds)), "v"(off), "s"(rsrc) : "memory");
}

// One operand's side of a block tile of R rows (A: R = BM, W: R = BN), staged by NW waves.
template <int LAY, int R, int NW>
struct TmStage {
  static constexpr int kInstr = R * BK * 2 / 1024 / NW;    // requests per wave and K step
  static_assert(NW % 2 == 0 && kInstr * NW * 1024 == R * BK * 2, "");
  uint32_t off[kInstr];                            // this lane's byte offsets from the tile's first element
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
#pragma clang loop unroll(full)
    for (int j = 0; j < kInstr; ++j) {
      if constexpr (LAY == OP_ROW) {
        off[j] = ((uint32_t)((j * NW + wave) * 8 + (lane >> 3)) * (uint32_t)ld + chunk * 8) * 2u;
      } else {
        constexpr int kRowLanes = R / 8;           // 16-byte slots of one k row
        const int k = (j * NW + wave) * (64 / kRowLanes) + lane / kRowLanes;
        const int c = (lane % kRowLanes) ^ ((k & 3) << 2);
        off[j] = c * 8 < rows ? ((uint32_t)k * (uint32_t)ld + c * 8) * 2u : kOobOffset;
      }
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
    kn = min(kn, BK);
    return LAY == OP_ROW ? tm_buffer(base + k, ((uint32_t)(rows - 1) * (uint32_t)ld + ((kn + 7) & ~7)) * 2u)
                         : tm_buffer(base + (int64_t)k * ld, ((uint32_t)(kn - 1) * (uint32_t)ld + ((rows + 1) & ~1)) * 2u);
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
  // This wave's j-th request: of a whole step, or with kn columns left in the segment.
  __device__ __forceinline__ void request(uint32_t lds, __amdgpu_buffer_rsrc_t rsrc, int j, int wave) const {
    tm_request(lds + (j * NW + wave) * 1024, rsrc, off[j]);
  }
  __device__ __forceinline__ void request_tail(uint32_t lds, __amdgpu_buffer_rsrc_t rsrc, int j, int wave, int kn) const {
    tm_request(lds + (j * NW + wave) * 1024, rsrc, LAY == OP_COL || chunk * 8 < kn ? off[j] : kOobOffset);
  }
};

// One operand's fragment reads: NF fragments of 32 rows from row `first` (a multiple of 32 NF) of a
// staged tile of R rows.
template <int LAY, int R, int NF>
struct TmFrag {
  static constexpr int kReads = LAY == OP_ROW ? NF : 2 * NF;   // LDS instructions per K slice
  int at[LAY == OP_ROW ? BK / 16 : NF];
  __device__ __forceinline__ void init(int first, int lane) {
    if constexpr (LAY == OP_ROW) {
#pragma clang loop unroll(full)
      for (int kk = 0; kk < BK / 16; ++kk)
        at[kk] = (first + (lane & 31)) * BK + ((kk * 2 + (lane >> 5)) ^ ((lane >> 1) & 7)) * 8;
    } else {
      const int p = lane & 15;
#pragma clang loop unroll(full)
      for (int i = 0; i < NF; ++i) {
        const int c = (((first / 32 + i) ^ (p >> 2)) << 2) + ((lane >> 4) & 1) * 2 + ((p & 3) >> 1);
        at[i] = ((lane >> 5) * 8 + (p >> 2)) * R + c * 8 + (p & 1) * 4;
      }
    }
  }
  __device__ __forceinline__ void read(uint4 (&f)[NF], const uint16_t* tile, int kk) const {
    if constexpr (LAY == OP_ROW) {
#pragma clang loop unroll(full)
      for (int i = 0; i < NF; ++i) f[i] = *(const uint4*)(tile + at[kk] + i * 32 * BK);
    } else {
      typedef short short4v __attribute__((ext_vector_type(4)));
      typedef __attribute__((address_space(3))) short4v lds_short4;
#pragma clang loop unroll(full)
      for (int i = 0; i < NF; ++i) {
        const uint2 lo = __builtin_bit_cast(uint2, __builtin_amdgcn_ds_read_tr16_b64_v4i16(
                                                       (lds_short4*)(tile + at[i] + kk * 16 * R)));
        const uint2 hi = __builtin_bit_cast(uint2, __builtin_amdgcn_ds_read_tr16_b64_v4i16(
                                                       (lds_short4*)(tile + at[i] + (kk * 16 + 4) * R)));
        f[i] = make_uint4(lo.x, lo.y, hi.x, hi.y);
      }
    }
  }
};

// TILE: 256 or 128.  DOTS: the operand's first K0 (<= 64) columns are the tower's pairwise dot
// terms, which the block computes itself (Gram tiles, as in tm_dots_mfma) straight into the first
// LDS stage, so the dot terms never exist in global memory (unless KEEPZ: a training forward keeps
// them).
template <int TILE> struct TmTile {
  static constexpr int WM = 2, WN = TILE == 256 ? 4 : 2, kWaves = WM * WN, kThreads = kWaves * 64;
  static constexpr int MT = TILE / WM / 32, NT = TILE / WN / 32;     // MFMA tiles of a wave
  static constexpr int kStageBytes = 2 * TILE * BK * 2;              // A then W
  static constexpr int kHalf = TILE / WM;                            // rows the epilogue parks at a time
  static constexpr int kParkStride = TILE + 4;   // floats; rows 4 banks apart: 16 lanes' float4 stores spread over all 64
  static constexpr int kLdsBytes = 2 * kStageBytes > kHalf * kParkStride * 4 ? 2 * kStageBytes : kHalf * kParkStride * 4;
};

template <int DT, int TILE, int ALAY, int WLAY, bool DOTS = false, bool KEEPZ = false, int TAG = DMT_TM_TAG>
__global__ __launch_bounds__(TmTile<TILE>::kThreads, TILE == 256 ? 1 : 2) void tm_gemm(const TmLaunch L) {
  using T = TmTile<TILE>;
  static_assert(!DOTS || (ALAY == OP_ROW && WLAY == OP_ROW), "");
  extern __shared__ __attribute__((aligned(16))) uint16_t lds[];
  // XCD-aware rasterisation.  Consecutive block ids go to different XCDs, so block b belongs
  // to XCD b % 8 and is that XCD's (b / 8)-th block.  The launch's tiles are cut into
  // super-tiles of up to L.super tiles (a few tile rows x all tile columns of one group) that
  // are dealt to the XCDs in turn: the blocks resident on an XCD then share their A rows
  // and W columns in that XCD's L2 instead of every XCD pulling every A tile over the fabric.
  const int xcd = blockIdx.x & 7, idx = blockIdx.x >> 3;
  const int gs = (idx / L.cap) * 8 + xcd, within = idx % L.cap;
  if (gs >= L.tile_start[L.ngroups]) return;
  int gi = 0;
  while (gi + 1 < L.ngroups && gs >= L.tile_start[gi + 1]) ++gi;
  const TmGroup& G = L.g[gi];
  const int tiles_n = (G.N + TILE - 1) / TILE, tiles_m = (G.M + TILE - 1) / TILE;
  const int sm = tiles_n >= L.super ? 1 : L.super / tiles_n;     // tile rows per super-tile
  if (within >= sm * tiles_n) return;
  // a split K multiplies the tile rows: virtual row tmv = slice * tiles_m + tm
  const int tmv = (gs - L.tile_start[gi]) * sm + within / tiles_n, tn = within % tiles_n;
  if (tmv >= tiles_m * tm_slices(G)) return;
  const int slice = tmv / tiles_m, tm = tmv - slice * tiles_m;
  const int m0 = tm * TILE, n0 = tn * TILE;
  const int M = G.M, N = G.N, K0 = G.K0;
  const int kofs = G.ksplit > 1 ? slice * G.klen : 0, kend = G.ksplit > 1 ? tm_slice_end(G.K1, kofs, G.klen) : G.K1;

  const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int wm = wave / T::WN, wn = wave % T::WN;
  floatx16 acc[T::MT][T::NT];
#pragma clang loop unroll(full)
  for (int i = 0; i < T::MT; ++i)
#pragma clang loop unroll(full)
    for (int j = 0; j < T::NT; ++j)
#pragma clang loop unroll(full)
      for (int v = 0; v < 16; ++v) acc[i][j][v] = 0.f;

  // ---- K loop
  {
    TmStage<ALAY, TILE, T::kWaves> sa;
    TmStage<WLAY, TILE, T::kWaves> sw;
    sa.init(G.A1, G.lda1, m0, M, kofs, wave, lane);
    sw.init(G.W1, G.ldw1, n0, N, kofs, wave, lane);
    const int nk0 = (K0 + BK - 1) / BK, nk = nk0 + (kend - kofs + BK - 1) / BK;
    const uint32_t lds0 = (uint32_t)(size_t)(__attribute__((address_space(3))) uint16_t*)lds;
    auto request_tile = [&](int stage, int kt) __attribute__((always_inline)) {
      const uint32_t la = lds0 + stage * T::kStageBytes, lw = la + TILE * BK * 2;
      if (kt >= nk0) {
        const int k = (kt - nk0) * BK, kn = kend - kofs - k;
        const __amdgpu_buffer_rsrc_t ba = sa.buffer(k, kn), bw = sw.buffer(k, kn);
        if (kn >= BK) {
#pragma clang loop unroll(full)
          for (int j = 0; j < sa.kInstr; ++j) {
            sa.request(la, ba, j, wave);
            sw.request(lw, bw, j, wave);
          }
        } else {                                   // the segment's last, partial step
#pragma clang loop unroll(full)
          for (int j = 0; j < sa.kInstr; ++j) {
            sa.request_tail(la, ba, j, wave, kn);
            sw.request_tail(lw, bw, j, wave, kn);
          }
        }
      } else {                                     // (few steps: their offsets are not kept in registers)
        const int k = kt * BK;
        if constexpr (!DOTS) {
          TmStage<ALAY, TILE, T::kWaves> sa0;      // segment 0 has pitches of its own
          sa0.init(G.A0, G.lda0, m0, M, 0, wave, lane);
          const __amdgpu_buffer_rsrc_t b0 = sa0.buffer(k, K0 - k);
#pragma clang loop unroll(full)
          for (int j = 0; j < sa0.kInstr; ++j) sa0.request_tail(la, b0, j, wave, K0 - k);
        }
        TmStage<WLAY, TILE, T::kWaves> sw0;
        sw0.init(G.W0, G.ldw0, n0, N, 0, wave, lane);
        const __amdgpu_buffer_rsrc_t b0 = sw0.buffer(k, K0 - k);
#pragma clang loop unroll(full)
        for (int j = 0; j < sw0.kInstr; ++j) sw0.request_tail(lw, b0, j, wave, K0 - k);
      }
    };
    TmFrag<ALAY, TILE, T::MT> ra;
    TmFrag<WLAY, TILE, T::NT> rw;
    ra.init(wm * T::MT * 32, lane);
    rw.init(wn * T::NT * 32, lane);
    // Fragments are double-buffered in registers: the reads of K slice kk + 1 are issued before the
    // MFMAs of slice kk, so LDS latency hides behind matrix work of the same wave.  The barrier of
    // a K step sits in front of its last slice's MFMAs: behind it come the requests for tile
    // kt + 2 (every wave has read the whole current stage by then) and the first reads of tile
    // kt + 1, and the last slice's MFMAs cover both.
    uint4 fa[2][T::MT], fw[2][T::NT];
    auto read_frag = [&](int buf, int stage, int kk) __attribute__((always_inline)) {
      const uint16_t* t = lds + stage * (T::kStageBytes / 2);
      ra.read(fa[buf], t, kk);
      rw.read(fw[buf], t + TILE * BK, kk);
    };
    request_tile(0, 0);
    if constexpr (DOTS) {
      if (nk > 1) request_tile(1, 1);
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
              a[g][u] = *(const uint4*)(on[g] && k + u * 16 + h8 < fd ? xp[g] + k + u * 16 : A);
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
      asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
      const int np = G.nf * (G.nf - 1) / 2;
      if ((const uint16_t*)G.W0 + np == G.W1) sw.zero_from(lds + TILE * BK, np, wave, lane);
    } else {
      __builtin_amdgcn_s_waitcnt(0x0f70);          // vmcnt(0): this wave's requests have landed
    }
    __syncthreads();
    if (!DOTS && nk > 1) request_tile(1, 1);
    read_frag(0, 0, 0);
    for (int kt = 0; kt < nk; ++kt) {
      const int cur = kt & 1;
#pragma clang loop unroll(full)
      for (int kk = 0; kk < BK / 16; ++kk) {
        if (kk + 1 < BK / 16) {
          read_frag((kk + 1) & 1, cur, kk + 1);
        } else {
          __builtin_amdgcn_s_waitcnt(0x0f70);
          __syncthreads();
          if (kt + 2 < nk) request_tile(cur, kt + 2);
          if (kt + 1 < nk) read_frag(0, cur ^ 1, 0);
        }
#pragma clang loop unroll(full)
        for (int i = 0; i < T::MT; ++i)
#pragma clang loop unroll(full)
          for (int j = 0; j < T::NT; ++j) acc[i][j] = mfma32<DT>(fw[kk & 1][j], fa[kk & 1][i], acc[i][j]);
        // LDS reads and MFMAs alternately: left alone, the scheduler puts each read right in front
        // of the MFMA that needs it, to save registers
        if (kk + 1 < BK / 16) {
          constexpr int kReads = TmFrag<ALAY, TILE, T::MT>::kReads + TmFrag<WLAY, TILE, T::NT>::kReads;
          constexpr int kMfma = T::MT * T::NT, kPer = (kReads + kMfma - 1) / kMfma, kPairs = kReads / kPer;
#pragma clang loop unroll(full)
          for (int q = 0; q < kPairs; ++q) {
            __builtin_amdgcn_sched_group_barrier(0x100, kPer, 0);
            __builtin_amdgcn_sched_group_barrier(0x008, 1, 0);
          }
          if (kMfma > kPairs) __builtin_amdgcn_sched_group_barrier(0x008, kMfma - kPairs, 0);
        }
      }
    }
  }

  // ---- epilogue through LDS, the rows of one wave row at a time: the waves that own them park their
  // float32 accumulators (a lane holds four consecutive columns of one row per register quad: too
  // narrow for global memory), then all threads walk them in 8-column pieces, so bias, x0, x_l
  // and the output move as 16-byte accesses.
  const int epi = G.epi;
  float* park = (float*)lds;
  auto park_half = [&]() __attribute__((always_inline)) {
#pragma clang loop unroll(full)
    for (int j = 0; j < T::NT; ++j)
#pragma clang loop unroll(full)
      for (int i = 0; i < T::MT; ++i)
#pragma clang loop unroll(full)
        for (int g = 0; g < 4; ++g)
          *(float4*)(park + (i * 32 + (lane & 31)) * T::kParkStride + wn * T::NT * 32 + j * 32 + g * 8 + (lane >> 5) * 4) =
              make_float4(acc[i][j][g * 4], acc[i][j][g * 4 + 1], acc[i][j][g * 4 + 2], acc[i][j][g * 4 + 3]);
  };
  constexpr int kRowThreads = TILE / 8, kRowStep = T::kThreads / kRowThreads, kChunks = T::kHalf / kRowStep;
  constexpr int kAhead = 2, kBufs = TILE == 256 ? 3 : 4;     // pieces whose operands are requested together, batches of them
  static_assert(kChunks % kAhead == 0, "");
  const int r0 = tid / kRowThreads, cc = (tid % kRowThreads) * 8;
  constexpr bool kForward = ALAY == OP_ROW && WLAY == OP_ROW;        // 16-bit outputs and x0; the others are gradients
  if constexpr (!kForward) {
    // Float32 outputs, four columns a lane, so that a wave's store covers whole lines (eight columns a
    // lane, two stores of every other 16 bytes: 2.5 GB of data gradients took 715 us, now 644).
    constexpr int kRow4 = T::kThreads / (TILE / 4), kPieces = T::kHalf / kRow4;
    constexpr int kBatch = TILE == 256 ? 2 : 4, kBatchesHalf = kPieces / kBatch, kBatchesAll = T::WM * kBatchesHalf, kDeep = 2;
    const int r4 = tid / (TILE / 4), c4 = (tid % (TILE / 4)) * 4;
    const bool on = n0 + c4 < N;
    const int64_t corner = (int64_t)m0 * G.ldc + n0;
    char* const c = (char*)((float*)G.C + slice * G.cstride + corner);
    const bool grad = ALAY == OP_ROW && epi == EPI_CROSS_GRAD, add = epi == EPI_F32_ADD;
    if (grad || (epi >= EPI_F32 && N % 4 == 0 && G.ldc % 4 == 0 && G.rdiv == 0 && ((uintptr_t)c & 15) == 0)) {
      // What a piece reads is requested a batch of pieces ahead, the first before the accumulators are
      // parked: with one block per CU nothing else hides that latency.  EPI_CROSS_GRAD: whole
      // pieces only (N and ldc are a tower's width, the tensors the library's own or blocks of
      // grad_pooled).
      const char *gn = add ? c : (const char*)(G.GN + corner), *ul = (const char*)G.UL + corner * 2;
      const char *x0 = (const char*)G.X0 + corner * 2, *u0 = (const char*)G.U0 + corner * 2;
      char *a0 = (char*)(G.ACC + corner), *du = (char*)G.DU + corner * 2;
      const bool has_gn = add || (grad && G.GN), has_u0 = grad && G.U0, acc_old = grad && !G.acc_first && (G.GN || G.U0);
      float4 pg[kDeep][kBatch], po[kDeep][kBatch];
      uint2 px[kDeep][kBatch], pu[kDeep][kBatch], pv[kDeep][kBatch];
      auto request = [&](int buf, int b) __attribute__((always_inline)) {
#pragma clang loop unroll(full)
        for (int u = 0; u < kBatch; ++u) {
          // (rows and columns past the edge read in bounds and are not stored)
          const uint32_t m = (uint32_t)min(b / kBatchesHalf * T::kHalf + r4 + (b % kBatchesHalf * kBatch + u) * kRow4, M - 1 - m0);
          const uint32_t e = m * (uint32_t)G.ldc + (on ? (uint32_t)c4 : 0u);
          if (has_gn) pg[buf][u] = *(const float4*)(gn + e * 4u);
          if constexpr (ALAY == OP_ROW) {
            if (grad) {
              px[buf][u] = *(const uint2*)(x0 + e * 2u);
              if (G.GN) pu[buf][u] = *(const uint2*)(ul + e * 2u);
              if (has_u0) pv[buf][u] = *(const uint2*)(u0 + e * 2u);
              if (acc_old) po[buf][u] = *(const float4*)(a0 + e * 4u);
            }
          }
        }
      };
      float4 sums = make_float4(0.f, 0.f, 0.f, 0.f);
      if (has_gn || grad) request(0, 0);
#pragma clang loop unroll(full)
      for (int b = 0; b < kBatchesAll; ++b) {
        const int h = b / kBatchesHalf, buf = b % kDeep;
        if (b % kBatchesHalf == 0) {
          if (wm == h) park_half();
          __syncthreads();
        }
        if ((has_gn || grad) && b + 1 < kBatchesAll) request((b + 1) % kDeep, b + 1);
#pragma clang loop unroll(full)
        for (int u = 0; u < kBatch; ++u) {
          const int r = r4 + (b % kBatchesHalf * kBatch + u) * kRow4;
          if (m0 + h * T::kHalf + r >= M || !on) continue;
          const uint32_t e = (uint32_t)(h * T::kHalf + r) * (uint32_t)G.ldc + (uint32_t)c4;
          float4 g = *(const float4*)(park + r * T::kParkStride + c4);
          if (has_gn) {
            const float4 n = pg[buf][u];
            g.x += n.x; g.y += n.y; g.z += n.z; g.w += n.w;
          }
          if constexpr (ALAY == OP_ROW) {
            if (grad) {
              float v0, v1, v2, v3;
              if (G.GN || has_u0) {
                float4 t = make_float4(0.f, 0.f, 0.f, 0.f);
                if (acc_old) t = po[buf][u];
                if (G.GN) {
                  const float4 n = pg[buf][u];
                  dmt::unpack2<DT>(pu[buf][u].x, v0, v1);
                  dmt::unpack2<DT>(pu[buf][u].y, v2, v3);
                  t.x += mul_rounded(n.x, v0); t.y += mul_rounded(n.y, v1);
                  t.z += mul_rounded(n.z, v2); t.w += mul_rounded(n.w, v3);
                }
                if (has_u0) {
                  dmt::unpack2<DT>(pv[buf][u].x, v0, v1);
                  dmt::unpack2<DT>(pv[buf][u].y, v2, v3);
                  t.x += mul_rounded(g.x, v0) + g.x; t.y += mul_rounded(g.y, v1) + g.y;
                  t.z += mul_rounded(g.z, v2) + g.z; t.w += mul_rounded(g.w, v3) + g.w;
                }
                *(float4*)(a0 + e * 4u) = t;
              }
              dmt::unpack2<DT>(px[buf][u].x, v0, v1);
              dmt::unpack2<DT>(px[buf][u].y, v2, v3);
              const uint2 d = make_uint2(dmt::pack2<DT>(g.x * v0, g.y * v1), dmt::pack2<DT>(g.z * v2, g.w * v3));
              *(uint2*)(du + e * 2u) = d;
              dmt::unpack2<DT>(d.x, v0, v1);       // the bias gradient sums the rounded values
              dmt::unpack2<DT>(d.y, v2, v3);
              sums.x += v0; sums.y += v1; sums.z += v2; sums.w += v3;
              if (!G.C) continue;
            }
          }
          *(float4*)(c + e * 4u) = g;
        }
        if (b % kBatchesHalf == kBatchesHalf - 1) {
          __syncthreads();                         // the parked rows have been read
          if (grad && (TILE == 256 || h == T::WM - 1)) {
            // column sums of 128 rows: the row steps' sums, added in order
            *(float4*)(park + r4 * TILE + c4) = sums;
            sums = make_float4(0.f, 0.f, 0.f, 0.f);
            __syncthreads();
            const int block = (m0 + (TILE == 256 ? h * T::kHalf : 0)) / 128;
            if (tid < TILE && n0 + tid < N && block * 128 < M) {
              float y = 0.f;
#pragma clang loop unroll(full)
              for (int q = 0; q < kRow4; ++q) y += park[q * TILE + tid];
              G.DBP[(int64_t)block * N + n0 + tid] = y;
            }
            __syncthreads();
          }
        }
      }
      return;
    }
  }
  const bool f32out = epi >= EPI_F32;
  // byte addresses of the 16-bit tensors: the tile's corner (uniform, 64 bits) + an offset inside the tile
  char* const cbase = (char*)G.C + ((int64_t)m0 * G.ldc + n0) * 2;
  char* const ubase = (char*)G.U + ((int64_t)m0 * G.ldc + n0) * 2;
  const char* const xbase = (const char*)G.X0 + ((int64_t)m0 * G.ldx + n0) * 2;
  const char* const lbase = (const char*)G.XL + ((int64_t)m0 * G.ldxl + n0) * 2;
  // whole 16-byte pieces everywhere (all tiles of a group alike): N and the pitches multiples of 8
  bool fast = !f32out && G.N % 8 == 0 && G.ldc % 8 == 0 && G.ldc2 % 8 == 0 && (((uintptr_t)cbase | (uintptr_t)G.bias) & 15) == 0;
  if (epi == EPI_CROSS)
    fast = fast && G.ldx % 8 == 0 && G.ldxl % 8 == 0 && (((uintptr_t)xbase | (uintptr_t)lbase | (uintptr_t)ubase) & 15) == 0;
  const bool cols_on = n0 + cc < N;
  if (fast) {
    const bool pre_cross = kForward && epi == EPI_CROSS;
    const uint32_t la = (uint32_t)G.ldx * 2u, lb = (uint32_t)G.ldxl * 2u, col = cols_on ? (uint32_t)cc * 2u : 0u;
    // a thread's chunks all lie in one 8-column piece of the tile: one bias load serves them
    uint4 bias_raw = make_uint4(0, 0, 0, 0);
    if (G.bias && cols_on) bias_raw = *(const uint4*)((const uint16_t*)G.bias + n0 + cc);
    // The cross epilogue requests its operands (x0 and x_l) for two pieces together, kBufs - 1
    // batches ahead of the one being walked and the first before the accumulators are parked: with
    // one block per CU nothing else hides that latency, and more is more registers than a wave
    // has beside its accumulators.
    uint4 pa[kBufs][kAhead], pb[kBufs][kAhead];
    auto request = [&](int buf, int batch) __attribute__((always_inline)) {
      const int h = batch / (kChunks / kAhead), u1 = batch % (kChunks / kAhead) * kAhead;
#pragma clang loop unroll(full)
      for (int u = 0; u < kAhead; ++u) {
        const uint32_t m = (uint32_t)min(h * T::kHalf + r0 + (u1 + u) * kRowStep, M - 1 - m0);
        pa[buf][u] = *(const uint4*)(xbase + (m * la + col));
        pb[buf][u] = *(const uint4*)(lbase + (m * lb + col));
      }
    };
    constexpr int kBatches = T::WM * (kChunks / kAhead);
    if (pre_cross)
#pragma clang loop unroll(full)
      for (int q = 0; q < kBufs - 1 && q < kBatches; ++q) request(q, q);
#pragma clang loop unroll(full)
    for (int batch = 0; batch < kBatches; ++batch) {
      const int h = batch / (kChunks / kAhead), u1 = batch % (kChunks / kAhead) * kAhead, buf = batch % kBufs;
      if (u1 == 0) {
        if (wm == h) park_half();
        __syncthreads();
      }
      if (pre_cross && batch + kBufs - 1 < kBatches) request((batch + kBufs - 1) % kBufs, batch + kBufs - 1);
#pragma clang loop unroll(full)
      for (int u = 0; u < kAhead; ++u) {
        const int r = r0 + (u1 + u) * kRowStep;
        if (m0 + h * T::kHalf + r >= M || !cols_on) continue;
        const float4 s0 = *(const float4*)(park + r * T::kParkStride + cc);
        const float4 s1 = *(const float4*)(park + r * T::kParkStride + cc + 4);
        char* c = cbase + ((uint32_t)(h * T::kHalf + r) * (uint32_t)G.ldc + (uint32_t)cc) * 2u;
        if (G.rdiv > 0) {
          const int m = m0 + h * T::kHalf + r;
          c = (char*)G.C + ((int64_t)(m / G.rdiv) * G.ldc + (int64_t)(m % G.rdiv) * G.ldc2 + n0 + cc) * 2;
        }
        float y[8] = {s0.x, s0.y, s0.z, s0.w, s1.x, s1.y, s1.z, s1.w};
        float bv[8];
        dmt::decode_chunk<DT>(bv, bias_raw);
#pragma clang loop unroll(full)
        for (int q = 0; q < 8; ++q) y[q] += bv[q];
        if (epi == EPI_BIAS_RELU) {
#pragma clang loop unroll(full)
          for (int q = 0; q < 8; ++q) y[q] = y[q] > 0.f ? y[q] : 0.f;
        } else if (kForward && epi == EPI_CROSS) {
          float xv[8], lv[8];
          if (G.U) dmt::store_chunk<DT, 8>(ubase + ((uint32_t)(h * T::kHalf + r) * (uint32_t)G.ldc + (uint32_t)cc) * 2u, 0, y);
          dmt::decode_chunk<DT>(xv, pa[buf][u]);
          dmt::decode_chunk<DT>(lv, pb[buf][u]);
#pragma clang loop unroll(full)
          for (int q = 0; q < 8; ++q) y[q] = xv[q] * y[q] + lv[q];
        }
        dmt::store_chunk<DT, 8>(c, 0, y);
      }
      if (u1 + kAhead == kChunks && h + 1 < T::WM) __syncthreads();
    }
    return;
  }
  // odd widths, unaligned rows: the same, element by element
  for (int h = 0; h < T::WM; ++h) {
    if (wm == h) park_half();
    __syncthreads();
    for (int r = r0; r < T::kHalf; r += kRowStep) {
      const int m = m0 + h * T::kHalf + r;
      if (m >= M) break;
      const int64_t row = G.rdiv > 0 ? (int64_t)(m / G.rdiv) * G.ldc + (int64_t)(m % G.rdiv) * G.ldc2 : (int64_t)m * G.ldc;
      for (int q = 0; q < 8 && n0 + cc + q < N; ++q) {
        const int n = n0 + cc + q;
        float y = park[r * T::kParkStride + cc + q];
        if (f32out) {
          float* c = (float*)G.C + slice * G.cstride + row + n;
          *c = epi == EPI_F32_ADD ? *c + y : y;
          continue;
        }
        if (G.bias) y += load_elt<DT>(G.bias, n);
        if (epi == EPI_BIAS_RELU) y = y > 0.f ? y : 0.f;
        if (epi == EPI_CROSS) {
          if (G.U) store_elt<DT>(G.U, row + n, y);
          y = load_elt<DT>(G.X0, (int64_t)m * G.ldx + n) * y + load_elt<DT>(G.XL, (int64_t)m * G.ldxl + n);
        }
        store_elt<DT>(G.C, row + n, y);
      }
    }
    __syncthreads();
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

// What a training forward keeps for the backward: for every cross layer l of a cross tower
// (full-rank or low-rank), x_{l+1} and u_l = W_l x_l + b_l, each [B][W_t] in the compute type;
// for a dot-product tower its dot terms, [B][np_pad] (np_pad = the F (F - 1) / 2 terms rounded
// up to 8, zeros behind them), and, where they cannot be read as they are, its projection weights
// with zero columns inserted to match, [O][np_pad + W_t].  Offsets in bytes from a 256-byte-aligned base; towers of other
// kinds keep nothing (their backward needs only the pooled values).
struct TmKept {
  size_t x[DMT_MAX_CROSS_LAYERS] = {}, u[DMT_MAX_CROSS_LAYERS] = {};
  size_t z = 0, wp = 0;      // dot tower: dot terms, and the projection weights as repacked for them
  bool has_z = false;
};

inline size_t plan_tm_kept(const dmt_plan* p, const dmt_tm_params* tp, int64_t B, int eb,
                           std::vector<TmKept>* kept) {
  size_t off = 0;
  kept->assign(p->T, TmKept());
  for (int32_t t = 0; t < p->T; ++t) {
    if (tp[t].kind == DMT_TM_DOT_LINEAR) {
      const int nf = p->tower_ntab[t], np_pad = (nf * (nf - 1) / 2 + 7) / 8 * 8;
      if (np_pad > 0) {
        (*kept)[t].z = off;
        (*kept)[t].has_z = true;
        off += dmt_align_up((size_t)B * np_pad * eb, 256);
        (*kept)[t].wp = off;
        off += dmt_align_up((size_t)tp[t].out_dim * (np_pad + p->tower_width[t]) * eb, 256);
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
template <int DT, int TILE, int ALAY, int WLAY, bool DOTS, bool KEEPZ>
void launch_tiles(const TmLaunch& L, int64_t blocks, hipStream_t s) {
  constexpr int bytes = TmTile<TILE>::kLdsBytes;
  auto kernel = tm_gemm<DT, TILE, ALAY, WLAY, DOTS, KEEPZ>;
  static DmtPerDevice configured;
  int dev = -1;
  (void)hipGetDevice(&dev);
  if (configured.needed(dev) &&
      hipFuncSetAttribute((const void*)kernel, hipFuncAttributeMaxDynamicSharedMemorySize, bytes) == hipSuccess)
    configured.set(dev);
  hipLaunchKernelGGL(kernel, dim3((unsigned)blocks), dim3(TmTile<TILE>::kThreads), bytes, s, L);
}

inline int64_t tiles_of(const TmGroup& g, int tile) {
  return (int64_t)((g.M + tile - 1) / tile) * ((g.N + tile - 1) / tile) * tm_slices(g);
}

// Whether a launch takes 256 x 256 tiles: when there are at least kBigTiles of them (three for every
// four CUs) and no group is so narrow that half of every tile would be empty.  (A short K makes no
// difference: data gradients of K = 128 and 256, 720 against 715 and 108 against 102 us.)
constexpr int kBigTiles = 192;
inline bool take_big(const dmt_plan* p, const TmGroup* g, int n) {
  if (p->sw.tm_big == 0) return false;
  int64_t tiles = 0;
  for (int i = 0; i < n; ++i) {
    if (g[i].M <= 128 || g[i].N <= 128) return false;
    tiles += tiles_of(g[i], 256);
  }
  return tiles >= kBigTiles || p->sw.tm_big == 2;
}

// Whether a forward launch goes to tm_gemm_small: up to 768 tiles of 32 x 32, one and a half rounds of
// the blocks that are resident together.  Both sides measured (128 x 128 / 32 x 32 tiles, us): dots and
// K = 1052, 512 tiles 28.6 / 19.2, 832 tiles 28.0 / 30.3; K = 832, 704 tiles 31.9 / 27.2, 1024 tiles
// 31.5 / 34.1; two cross layers of 2048 columns, 1024 tiles each 85.8 / 84.2, 2048 tiles 87.8 / 149.
inline bool take_small(const dmt_plan* p, const TmGroup* g, int n) {
  if (p->sw.tm_big != 1) return p->sw.tm_big == 3;
  int64_t tiles = 0;
  for (int i = 0; i < n; ++i) tiles += tiles_of(g[i], 32);
  return tiles <= 768;
}

// All groups of the list, kMaxGroups to a launch.  dots: every group computes its dot terms itself.
template <int DT, int ALAY = OP_ROW, int WLAY = OP_ROW>
void launch_groups(const dmt_plan* p, std::vector<TmGroup>& groups, hipStream_t s, bool dots = false,
                   int kid = DMT_K_TM_GEMM) {
  for (size_t first = 0; first < groups.size(); first += kMaxGroups) {
    TmLaunch L;
    L.ngroups = (int32_t)std::min<size_t>(kMaxGroups, groups.size() - first);
    bool keepz = false;                           // a training forward keeps the dot terms
    for (int i = 0; i < L.ngroups; ++i) {
      L.g[i] = groups[first + i];
      keepz = keepz || (dots && L.g[i].U != nullptr);
    }
    if constexpr (ALAY == OP_ROW && WLAY == OP_ROW && DMT_TM_TAG == 0) {
      // (in-kernel dot terms, or one K segment)
      bool small = take_small(p, L.g, L.ngroups);
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
    const bool big = take_big(p, L.g, L.ngroups);
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
      L.cap = (int32_t)std::max<int64_t>(L.cap, sm * tn);
      nst += (tm + sm - 1) / sm;
    }
    L.tile_start[L.ngroups] = (int32_t)nst;
    const int64_t blocks = (nst + 7) / 8 * 8 * L.cap;
    if (blocks == 0) continue;
    DmtScope scope(p, kid, s);
    if constexpr (ALAY == OP_ROW && WLAY == OP_ROW && DMT_TM_TAG == 0) {
      if (dots && big && keepz) { launch_tiles<DT, 256, ALAY, WLAY, true, true>(L, blocks, s); continue; }
      if (dots && big) { launch_tiles<DT, 256, ALAY, WLAY, true, false>(L, blocks, s); continue; }
      if (dots && keepz) { launch_tiles<DT, 128, ALAY, WLAY, true, true>(L, blocks, s); continue; }
      if (dots) { launch_tiles<DT, 128, ALAY, WLAY, true, false>(L, blocks, s); continue; }
    }
    if (big) launch_tiles<DT, 256, ALAY, WLAY, false, false>(L, blocks, s);
    else launch_tiles<DT, 128, ALAY, WLAY, false, false>(L, blocks, s);
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
