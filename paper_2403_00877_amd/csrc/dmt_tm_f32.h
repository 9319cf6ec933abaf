// Grouped float32 contractions of the Tower Module, forward and backward:
//   C[m][n] = epilogue(sum over k of A(m, k) W(n, k) [+ bias[n]])
// on v_mfma_f32_32x32x2 (float32 products and sums).  Each operand is read where it lies, either
// with k contiguous (x, W of the forward; dy and W of a data gradient) or with its row index
// contiguous (W of a data gradient, dy and x of a weight gradient), so the backward needs no
// transposed copies; a ReLU mask and the bias gradient are taken on the way.
//
// Float32 towers are the small models, so the shape to serve is a few hundred tiles of a few dozen
// to a few thousand k: one wave owns a 32 x 32 tile (or, where tiles are few and k is long, an
// eighth to a half of its k; the waves' sums are added in wave order through LDS), and reads its
// operands straight into registers, thirty-two k ahead of the matrix instructions.  Nothing is
// staged: a lane may feed the matrix core any k it likes as long as both operands agree, so lane
// half h takes k + 4 h .. k + 4 h + 3 as one 16-byte load.  One thread per output, the plain
// kernel before this one, was bound by one dependent load pair per k; 26 features of 64 columns
// to 64 outputs, batch 2048: 394 -> 13 us forward, 1600 -> 26 us backward (with loads whose
// layout and guards were decided per load instead of per segment, so that each waited for the one
// before it, and a weight gradient's k left to one wave: 24 and 186 us).
#pragma once
#include <algorithm>
#include <cstdint>
#include <vector>

#include "dmt_tm_gemm.h"

namespace {

struct TmF32Group {
  const float* A0;    // first K0 columns of the operand (k contiguous)
  const float* A1;    // next K1 columns
  const float* W0;    // W(n, k) for k < K0
  const float* W1;    // ... and for the K1 columns behind
  const float* bias;  // [N] or null
  const float* mask;  // A1(m, k) counts only where mask, laid out like A1, is > 0 (wcol); or null
  const float* X0;    // EPI_CROSS, as in TmGroup
  const float* XL;
  float* C;
  float* U;
  float* db;          // [M] or null: sum over k of A(m, k)
  int32_t lda0, K0, lda1, K1, ldw0, ldw1, ldc, ldx, ldxl, M, N, epi;
  int32_t acol, wcol;     // 1: A1(m, k) is A1[k lda1 + m] (K0 = 0) / W(n, k) is W[k ldw + n]
  int32_t adiv, lda2;     // acol: row k of A1 starts at (k / adiv) lda1 + (k % adiv) lda2
  int32_t rdiv, ldc2;     // two-level rows of C, as in TmGroup
  int32_t log2_ks;        // 2^log2_ks waves share a tile's k
};

constexpr int kF32Groups = 16;
constexpr int kF32Waves = 16;
struct TmF32Launch {
  int32_t ngroups;
  int32_t block_start[kF32Groups + 1];
  TmF32Group g[kF32Groups];
};

// How an operand lies: k contiguous; its row index contiguous; the same with two-level k rows.
enum { F32_ROW = 0, F32_COL = 1, F32_COL2 = 2 };

// Four consecutive k of one operand row (`row` is clamped to a valid one): unguarded, and with
// zeros from K on.
template <int LAY, bool ANY>
__device__ __forceinline__ float4 f32_load4(const float* __restrict__ p, int64_t row, int k, int64_t ld, int div,
                                            int64_t ld2) {
  if constexpr (LAY == F32_ROW) {
    if constexpr (ANY) {                           // from any 4-byte boundary
      typedef float float4u __attribute__((ext_vector_type(4), aligned(4)));
      const float4u v = *(const float4u*)(p + row * ld + k);
      return make_float4(v.x, v.y, v.z, v.w);
    }
    return *(const float4*)(p + row * ld + k);
  }
  auto at = [&](int kk) {
    return row + (LAY == F32_COL2 ? (int64_t)(kk / div) * ld + (int64_t)(kk % div) * ld2 : kk * ld);
  };
  return make_float4(p[at(k)], p[at(k + 1)], p[at(k + 2)], p[at(k + 3)]);
}
template <int LAY>
__device__ __forceinline__ float4 f32_load4_edge(const float* __restrict__ p, int64_t row, int k, int K, int64_t ld,
                                                 int div, int64_t ld2) {
  auto at = [&](int kk) {
    if constexpr (LAY == F32_ROW) return row * ld + kk;
    else return row + (LAY == F32_COL2 ? (int64_t)(kk / div) * ld + (int64_t)(kk % div) * ld2 : kk * ld);
  };
  float4 v = make_float4(0.f, 0.f, 0.f, 0.f);
  if (k < K) v.x = p[at(k)];
  if (k + 1 < K) v.y = p[at(k + 1)];
  if (k + 2 < K) v.z = p[at(k + 2)];
  if (k + 3 < K) v.w = p[at(k + 3)];
  return v;
}

// One K segment of a wave's tile: steps lo .. hi - 1 of 8 k each.
struct F32Seg {
  const float *A, *W, *mask;
  int64_t lda, ldw, lda2;
  int K, div, lo, hi;
};
constexpr int kF32Unroll = 4;                      // steps whose operands are requested together

// Whether whole steps of a segment can be read 16 bytes at a time from 16-byte boundaries.
template <int ALAY, int WLAY, bool MASK>
__device__ __forceinline__ bool f32_aligned(const F32Seg& g) {
  return (ALAY != F32_ROW || (((uintptr_t)g.A | (MASK ? (uintptr_t)g.mask : 0)) & 15) + (g.lda & 3) == 0) &&
         (WLAY != F32_ROW || ((uintptr_t)g.W & 15) + (g.ldw & 3) == 0);
}

// ANY: rows may start on any 4-byte boundary.  (Otherwise those that are not aligned go step by step, each load behind
// a guard; one load for both kinds took the aligned ones 13.6 -> 15.1 us.)
template <int ALAY, int WLAY, bool MASK, bool ANY = false>
__device__ __forceinline__ void f32_segment(const F32Seg& g, int64_t m, int64_t n, int h4, floatx16& acc, float& db) {
  auto step = [&](float4 a, float4 w, float4 q) __attribute__((always_inline)) {
    if constexpr (MASK) {
      a.x = q.x > 0.f ? a.x : 0.f;
      a.y = q.y > 0.f ? a.y : 0.f;
      a.z = q.z > 0.f ? a.z : 0.f;
      a.w = q.w > 0.f ? a.w : 0.f;
    }
    acc = __builtin_amdgcn_mfma_f32_32x32x2f32(a.x, w.x, acc, 0, 0, 0);
    acc = __builtin_amdgcn_mfma_f32_32x32x2f32(a.y, w.y, acc, 0, 0, 0);
    acc = __builtin_amdgcn_mfma_f32_32x32x2f32(a.z, w.z, acc, 0, 0, 0);
    acc = __builtin_amdgcn_mfma_f32_32x32x2f32(a.w, w.w, acc, 0, 0, 0);
    db += (a.x + a.y) + (a.z + a.w);
  };
  // whole batches of steps, loads unconditional, a batch ahead of the matrix instructions (the
  // last prefetch reads the last batch once more)
  const int full = ANY || f32_aligned<ALAY, WLAY, MASK>(g) ? min(g.hi, g.K / 8) : g.lo;
  const int nb = (full - g.lo) / kF32Unroll;
  int s = g.lo;
  if (nb > 0) {
    float4 a[2][kF32Unroll], w[2][kF32Unroll], q[2][kF32Unroll];
    auto load = [&](int buf, int b) __attribute__((always_inline)) {
#pragma unroll
      for (int u = 0; u < kF32Unroll; ++u) {
        const int k = (g.lo + b * kF32Unroll + u) * 8 + h4;
        a[buf][u] = f32_load4<ALAY, ANY>(g.A, m, k, g.lda, g.div, g.lda2);
        w[buf][u] = f32_load4<WLAY, ANY>(g.W, n, k, g.ldw, 0, 0);
        if constexpr (MASK) q[buf][u] = f32_load4<ALAY, ANY>(g.mask, m, k, g.lda, g.div, g.lda2);
        else q[buf][u] = make_float4(0.f, 0.f, 0.f, 0.f);
      }
    };
    load(0, 0);
    for (int b = 0; b < nb; b += 2) {
      load(1, min(b + 1, nb - 1));
#pragma unroll
      for (int u = 0; u < kF32Unroll; ++u) step(a[0][u], w[0][u], q[0][u]);
      if (b + 1 >= nb) break;
      load(0, min(b + 2, nb - 1));
#pragma unroll
      for (int u = 0; u < kF32Unroll; ++u) step(a[1][u], w[1][u], q[1][u]);
    }
    s += nb * kF32Unroll;
  }
  for (; s < g.hi; ++s) {
    const int k = s * 8 + h4;
    float4 q = make_float4(0.f, 0.f, 0.f, 0.f);
    const float4 a = f32_load4_edge<ALAY>(g.A, m, k, g.K, g.lda, g.div, g.lda2);
    const float4 w = f32_load4_edge<WLAY>(g.W, n, k, g.K, g.ldw, 0, 0);
    if constexpr (MASK) q = f32_load4_edge<ALAY>(g.mask, m, k, g.K, g.lda, g.div, g.lda2);
    step(a, w, q);
  }
}

// First of a tile's `steps` that the wave `part` of 2^log2_ks takes.  (64 bits: a per-feature layer's weight
// gradient has up to 2^28 steps, times sixteen waves.)
__host__ __device__ inline int f32_first_step(int steps, int part, int log2_ks) {
  return (int)((int64_t)steps * part >> log2_ks);
}
// The forward's shares are whole batches of steps, since what is left of a batch goes step by step, each waiting for its
// loads (26 features of 64 columns to 64 outputs, batch 2048, shares of 6 and 7 steps / 4 and 8: 20.9 / 14.1 us, 13.6
// with the layouts that a forward does not have left out).  The backward's are single steps: an operand with its row
// index contiguous takes four loads a step, and a share of two batches loads three (the last prefetch), so it is the
// longest share that counts (per-feature layers of 6 and 7 features, batch 107, 81 steps to 16 waves, batches / steps:
// 48.1 / 38.6 us; 14 steps to two 11.8 / 11.4; 26 features of 64 columns, batch 2048, 16 steps a wave, the same).
__host__ __device__ inline int f32_share_begin(int steps, int part, int log2_ks, bool batches) {
  if (!batches) return f32_first_step(steps, part, log2_ks);
  const int first = f32_first_step((steps + kF32Unroll - 1) / kF32Unroll, part, log2_ks) * kF32Unroll;
  return first < steps ? first : steps;
}

template <int TAG = DMT_TM_TAG>
__global__ __launch_bounds__(kF32Waves * 64) void tm_gemm_f32(const TmF32Launch L) {
  __shared__ float red[kF32Waves][16][64];
  __shared__ float red_db[kF32Waves][32];
  int gi = 0;
  while (gi + 1 < L.ngroups && (int)blockIdx.x >= L.block_start[gi + 1]) ++gi;
  const TmF32Group& G = L.g[gi];
  const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int ks = 1 << G.log2_ks, part = wave & (ks - 1), first = wave - part;
  const int M = G.M, N = G.N;
  const int tiles_n = (N + 31) / 32, tiles = (M + 31) / 32 * tiles_n;
  const int tile = (int)(blockIdx.x - L.block_start[gi]) * (kF32Waves >> G.log2_ks) + (wave >> G.log2_ks);
  const bool live = tile < tiles;                  // (waves without a tile still meet the barrier)
  const int m0 = tile / tiles_n * 32, n0 = tile % tiles_n * 32;
  const int r = lane & 31, h4 = (lane >> 5) * 4;
  const int m = min(m0 + r, M - 1), n = min(n0 + r, N - 1);   // rows past the edge: the last row, not stored
  // this wave's share of the steps, cut into the two segments
  const int S0 = (G.K0 + 7) / 8, S = S0 + (G.K1 + 7) / 8;
  const int lo = live ? f32_share_begin(S, part, G.log2_ks, TAG == 0) : 0;
  const int hi = live ? f32_share_begin(S, part + 1, G.log2_ks, TAG == 0) : 0;
  floatx16 acc;
#pragma unroll
  for (int v = 0; v < 16; ++v) acc[v] = 0.f;
  float db = 0.f;
  // A dot tower's weights have rows of 78 terms and 208 columns, say, so few of them are aligned (13 features of 16
  // columns to 64 outputs, batch 107: 16.1 us step by step, 10.6).
  auto forward = [&](const F32Seg& g) __attribute__((always_inline)) {
    if (TAG != 0 || f32_aligned<F32_ROW, F32_ROW, false>(g)) f32_segment<F32_ROW, F32_ROW, false>(g, m, n, h4, acc, db);
    else f32_segment<F32_ROW, F32_ROW, false, true>(g, m, n, h4, acc, db);
  };
  if (lo < S0) {
    const F32Seg g0{G.A0, G.W0, nullptr, G.lda0, G.ldw0, 0, G.K0, 0, lo, min(hi, S0)};
    if (TAG != 0 && G.wcol) f32_segment<F32_ROW, F32_COL, false>(g0, m, n, h4, acc, db);
    else forward(g0);
  }
  if (hi > S0) {
    const F32Seg g1{G.A1, G.W1, G.mask, G.lda1, G.ldw1, G.lda2, G.K1, G.adiv, max(lo, S0) - S0, hi - S0};
    if (TAG == 0) {                                // (the forward's operands have k contiguous)
      forward(g1);
    } else if (!G.acol) {
      if (!G.wcol) f32_segment<F32_ROW, F32_ROW, false>(g1, m, n, h4, acc, db);
      else if (!G.mask) f32_segment<F32_ROW, F32_COL, false>(g1, m, n, h4, acc, db);
      else f32_segment<F32_ROW, F32_COL, true>(g1, m, n, h4, acc, db);
    } else {
      if (G.adiv) f32_segment<F32_COL2, F32_COL, false>(g1, m, n, h4, acc, db);
      else if (!G.mask) f32_segment<F32_COL, F32_COL, false>(g1, m, n, h4, acc, db);
      else f32_segment<F32_COL, F32_COL, true>(g1, m, n, h4, acc, db);
    }
  }
  const bool sums = G.db != nullptr && n0 == 0;    // (uniform) this tile's row sums of A are wanted
  db += __shfl_xor(db, 32);

  // lane holds column n0 + lane % 32 of rows (v / 4) * 8 + (lane / 32) * 4 + v % 4
  auto store = [&](int v, float y) {
    const int mm = m0 + (v >> 2) * 8 + (lane >> 5) * 4 + (v & 3), nn = n0 + r;
    if (mm >= M || nn >= N) return;
    const int64_t row = G.rdiv > 0 ? (int64_t)(mm / G.rdiv) * G.ldc + (int64_t)(mm % G.rdiv) * G.ldc2
                                   : (int64_t)mm * G.ldc;
    float* c = G.C + row + nn;
    if (G.epi == EPI_F32) { *c = y; return; }
    if (G.epi == EPI_F32_ADD) { *c += y; return; }
    if (G.bias) y += G.bias[nn];
    if (G.epi == EPI_BIAS_RELU) y = y > 0.f ? y : 0.f;
    if (G.epi == EPI_CROSS) {
      if (G.U) G.U[row + nn] = y;
      y = G.X0[(int64_t)mm * G.ldx + nn] * y + G.XL[(int64_t)mm * G.ldxl + nn];
    }
    *c = y;
  };
  if (ks == 1) {
    if (live) {
#pragma unroll
      for (int v = 0; v < 16; ++v) store(v, acc[v]);
      if (sums && lane < 32 && m0 + lane < M) G.db[m0 + lane] = db;
    }
    return;                                        // (uniform over the block: no barrier is skipped)
  }
#pragma unroll
  for (int v = 0; v < 16; ++v) red[wave][v][lane] = acc[v];
  if (sums && lane < 32) red_db[wave][lane] = db;
  __syncthreads();
  if (!live) return;
  const int per = 16 >> G.log2_ks;                 // accumulator registers this wave finishes
  for (int v = part * per; v < (part + 1) * per; ++v) {
    float y = red[first][v][lane];
    for (int q = 1; q < ks; ++q) y += red[first + q][v][lane];
    store(v, y);
  }
  if (sums && part == 0 && lane < 32 && m0 + lane < M) {
    float y = red_db[first][lane];
    for (int q = 1; q < ks; ++q) y += red_db[first + q][lane];
    G.db[m0 + lane] = y;
  }
}

// A forward-shaped group (both operands k contiguous).
inline TmF32Group f32_group(const TmGroup& g) {
  TmF32Group f{};
  f.A0 = (const float*)g.A0; f.lda0 = g.lda0; f.K0 = g.K0;
  f.A1 = (const float*)g.A1; f.lda1 = g.lda1; f.K1 = g.K1;
  f.W0 = (const float*)g.W0; f.ldw0 = g.ldw0;
  f.W1 = (const float*)g.W1; f.ldw1 = g.ldw1;
  f.bias = (const float*)g.bias;
  f.X0 = (const float*)g.X0; f.ldx = g.ldx;
  f.XL = (const float*)g.XL; f.ldxl = g.ldxl;
  f.C = (float*)g.C; f.ldc = g.ldc; f.rdiv = g.rdiv; f.ldc2 = g.ldc2;
  f.U = (float*)g.U;
  f.M = g.M; f.N = g.N; f.epi = g.epi;
  return f;
}

inline int64_t f32_tiles(const TmF32Group& g) { return (int64_t)((g.M + 31) / 32) * ((g.N + 31) / 32); }
inline int64_t f32_steps(const TmF32Group& g) { return (int64_t)((g.K0 + 7) / 8 + (g.K1 + 7) / 8); }

// Waves (2^log2_ks) for each of a launch's like tiles of `steps`, `before` waves of longer ones ahead of them; a wave
// keeps a batch of steps.  4096 waves are resident together, four to a SIMD.
// Forward: the least of  rounds of 4096 waves x (steps a wave + the start and end of a tile, about four steps, three of
// a cross layer, whose epilogue the waves share too).  A round and a half is as long as two: us, doubled up to 4096 waves /
// this: 20 cross towers of 64 columns, batch 6000 (6016 waves of 8 steps / 12032 of 4) 180 / 141; 2 dot towers of 13
// features of 16 columns (6016 of 4 and 8 / 3008 of 9) 26.8 / 24.8; per-feature layers on 4 towers 67 / 53.
// Backward: doubled up to 4096 waves, or 8192 while a wave keeps 32 steps: 2560 columns to 512 outputs, batch 512
// (2560 waves of 64 steps / 5120 of 32) 75 / 72 us; 4 data gradients of 8 steps (3328 tiles) beside weight gradients
// 26.3 us, as 6656 waves of 4 steps 29.6.
constexpr int64_t kF32Resident = 4096;
inline int f32_log2_ks(int64_t steps, int64_t tiles, int64_t before, bool forward, bool cross) {
  int best = 0;
  int64_t least = INT64_MAX;
  for (int l = 0; l <= 4 && (l == 0 || steps >> l >= kF32Unroll); ++l) {
    const int64_t waves = tiles << l;
    if (forward) {
      const int64_t cost = (before + waves + kF32Resident - 1) / kF32Resident * (((steps - 1) >> l) + 1 + (cross ? 3 : 4));
      if (cost < least) least = cost, best = l;
    } else if (waves <= kF32Resident || (waves <= 2 * kF32Resident && steps >> l >= 32)) {
      best = l;
    }
  }
  return best;
}

// The order of the groups, kF32Groups to a launch, and how many waves share a tile's k.  Waves are counted within a launch:
// counted group by group, the 26.3 us above were 29.6; over all of a stage's groups, 20 towers, which take two
// launches, got half the waves (192 columns to 64 outputs, batch 2048: 64 us, now 34; per-feature layers of 8 features on
// 8 towers, backward, 257 / 237).
inline void f32_arrange(std::vector<TmF32Group>& groups, bool forward) {
  auto longest_wave_first = [](const TmF32Group& a, const TmF32Group& b) { return f32_steps(a) >> a.log2_ks > f32_steps(b) >> b.log2_ks; };
  // which groups share a launch: those that would run about as long, each by itself
  for (TmF32Group& g : groups) g.log2_ks = f32_log2_ks(f32_steps(g), f32_tiles(g), 0, false, false);
  std::stable_sort(groups.begin(), groups.end(), longest_wave_first);
  for (size_t first = 0; first < groups.size(); first += kF32Groups) {
    const auto begin = groups.begin() + first, end = groups.begin() + std::min(groups.size(), first + kF32Groups);
    std::stable_sort(begin, end, [](const TmF32Group& a, const TmF32Group& b) { return f32_steps(a) > f32_steps(b); });
    int64_t before = 0;
    for (auto g = begin; g != end;) {              // groups of about as long a k, down to half of the longest
      const int64_t steps = f32_steps(*g);
      int64_t tiles = 0;
      auto past = g;
      for (; past != end && 2 * f32_steps(*past) >= steps; ++past) tiles += f32_tiles(*past);
      const int l = f32_log2_ks(steps, tiles, before, forward, g->epi == EPI_CROSS);
      before += tiles << l;
      for (; g != past; ++g)                       // (every wave keeps a batch: 8 and 4 steps in halves 9.1 us, 8 in halves 6.7)
        for (g->log2_ks = l; g->log2_ks > 0 && f32_steps(*g) >> g->log2_ks < kF32Unroll;) --g->log2_ks;
    }
    std::stable_sort(begin, end, longest_wave_first);
  }
}

// All groups in as few launches as they take (no group of the list may read what another writes).  Groups whose waves
// work longest go first.
inline void launch_f32(const dmt_plan* p, std::vector<TmF32Group>& groups, hipStream_t s, int kid) {
  f32_arrange(groups, DMT_TM_TAG == 0);
  for (size_t first = 0; first < groups.size(); first += kF32Groups) {
    TmF32Launch L;
    L.ngroups = (int32_t)std::min<size_t>(kF32Groups, groups.size() - first);
    int32_t blocks = 0;
    for (int i = 0; i < L.ngroups; ++i) {
      const TmF32Group& g = L.g[i] = groups[first + i];
      L.block_start[i] = blocks;
      const int per_block = kF32Waves >> g.log2_ks;
      blocks += (int32_t)((f32_tiles(g) + per_block - 1) / per_block);
    }
    L.block_start[L.ngroups] = blocks;
    if (blocks == 0) continue;
    DmtScope scope(p, kid, s);
    hipLaunchKernelGGL((tm_gemm_f32<DMT_TM_TAG>), dim3(blocks), dim3(kF32Waves * 64), 0, s, L);
  }
  groups.clear();
}

}  // namespace
