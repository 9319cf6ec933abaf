// dmt_tower_module_bwd: the chain rule through the Tower Module forms (paper
// Sec. 3.2, Sec. 4, Listings 1 and 2), from dL/d(tm_out) to dL/d(pooled) and the
// parameter gradients.
//
// Every contraction reads its operands where they lie:
//   data gradient    dX[B][Kin]  = dz[B][O] . W[O][Kin]        (W along its rows: OP_COL)
//   weight gradient  dW[O][Kin]  = dz[B][O]^T . x[B][Kin]      (both OP_COL)
// so nothing is transposed in memory: dy is rounded once to the compute type, and the tensors of
// the forward serve as they are.  Towers are grouped into one launch per stage like the forward's.
// The forward's intermediates are recomputed (dot terms; u_l and x_l of the cross layers) unless the
// caller hands over what a training forward kept.  A weight gradient has few output tiles and a
// long K (the batch): K is cut into slices that are contractions of their own and summed in slice
// order.  Bias gradients are fixed-order sums of the rounded gradient operand, taken where it is
// written.  A cross tower's elementwise steps run in the epilogues of the contractions above them
// (EPI_CROSS_GRAD).  The DLRM module's shared per-feature layer is the same machinery on rows
// (sample, feature) of the pooled block.
#include <type_traits>

#define DMT_TM_TAG 1          // this file's instances of the shared GEMM kernels
#include "dmt_tm_gemm.h"
#include "dmt_tm_f32.h"

namespace {

constexpr int kMaxItems = 32;

// One tower's share of a grouped launch of the small kernels below: block id ->
// (item, block within the item), like the grouped GEMM.  The meaning of the fields is
// each kernel's own.
struct TmbItem {
  const void* a;
  const void* b;
  const void* c;
  void* o0;
  void* o1;
  void* o2;
  int64_t n0, n1, n2;
  int32_t i0, i1, i2, i3, i4, i5;
  int32_t nbx;               // blocks along the first dimension (2-D kernels) or blocks of the item
};

struct TmbLaunch {
  int32_t n;
  int32_t block_start[kMaxItems + 1];
  TmbItem it[kMaxItems];
};

__device__ __forceinline__ int tmb_find(const TmbLaunch& L) {
  int i = 0;
  while (i + 1 < L.n && (int)blockIdx.x >= L.block_start[i + 1]) ++i;
  return i;
}

// ---------------------------------------------------------------- small kernels

__device__ __forceinline__ void load_f32x8(const float* p, int64_t e, float (&x)[8]) {
  const float4 a = *(const float4*)(p + e), b = *(const float4*)(p + e + 4);
  x[0] = a.x; x[1] = a.y; x[2] = a.z; x[3] = a.w; x[4] = b.x; x[5] = b.y; x[6] = b.z; x[7] = b.w;
}
__device__ __forceinline__ void store_f32x8(float* p, int64_t e, const float (&x)[8]) {
  *(float4*)(p + e) = make_float4(x[0], x[1], x[2], x[3]);
  *(float4*)(p + e + 4) = make_float4(x[4], x[5], x[6], x[7]);
}

__device__ __forceinline__ void pack_dot_weights(const TmbItem& G, int64_t e);

// dz[b][o] = dy[b][o] (zero where ReLU was off: y[b][o] <= 0), rounded to DT, with zero columns
// O .. Op-1, and the column sums of the rounded values over the rows of each block (the bias
// gradient's parts): dbp[block][o].  Row b of dy (and y) starts at element b * ldy, or, with
// rdiv > 0, at (b / rdiv) * ldy + (b % rdiv) * ld2: rdiv rows of the gradient operand lie side by
// side in one row of the output gradient (a per-feature layer).  One pass over dy, bound by its
// bytes; 2^tc threads take a row's (up to 256) columns, 8 each.
// a = dy, b = y, o0 = dz, o1 = dbp, n0 = rows, n1 = rows per block, n2 = ldy, i0 = O, i1 = Op,
// i2 = relu, i3 = rdiv, i4 = ld2, i5 = tc; nbx = blocks along the rows.  (Items with c set repack a dot tower's
// weights instead, pack_dot_weights.)
template <int DT>
__global__ __launch_bounds__(kBlock) void tmb_prep_dz(const TmbLaunch L) {
  __shared__ float red[kBlock][8];
  const int gi = tmb_find(L);
  const TmbItem& G = L.it[gi];
  const int lb = blockIdx.x - L.block_start[gi];
  if (G.c) {
    pack_dot_weights(G, (int64_t)lb * kBlock + threadIdx.x);
    return;
  }
  const float* __restrict__ dy = (const float*)G.a;
  const uint16_t* __restrict__ y = (const uint16_t*)G.b;
  uint16_t* __restrict__ dz = (uint16_t*)G.o0;
  const int64_t rows = G.n0;
  const int O = G.i0, Op = G.i1, relu = G.i2, tc = G.i5, rp = kBlock >> tc;
  const int o = (lb / G.nbx) * (8 << tc) + (threadIdx.x & ((1 << tc) - 1)) * 8, rr = threadIdx.x >> tc;
  const int64_t b0 = (int64_t)(lb % G.nbx) * G.n1, b1 = min(rows, b0 + G.n1);
  // whole 16-byte reads where every row allows them
  const bool vec = O % 8 == 0 && G.n2 % 4 == 0 && G.i4 % 4 == 0 && ((uintptr_t)dy & 15) == 0;
  const bool vec_y = vec && G.n2 % 8 == 0 && ((uintptr_t)y & 15) == 0;
  float s[8];
#pragma unroll
  for (int q = 0; q < 8; ++q) s[q] = 0.f;
  for (int64_t b = b0 + rr; b < b1; b += rp) {
    if (o >= Op) break;
    const int64_t at = (G.i3 > 0 ? (b / G.i3) * G.n2 + (b % G.i3) * G.i4 : b * G.n2) + o;
    float g[8], v[8];
    if (vec) load_f32x8(dy, at, g);
    else
#pragma unroll
      for (int q = 0; q < 8; ++q) g[q] = o + q < O ? dy[at + q] : 0.f;
    if (relu) {
      if (vec_y) dmt::decode_chunk<DT>(v, *(const uint4*)(y + at));
      else
#pragma unroll
        for (int q = 0; q < 8; ++q) v[q] = o + q < O ? load_elt<DT>(y, at + q) : 0.f;
#pragma unroll
      for (int q = 0; q < 8; ++q) g[q] = v[q] > 0.f ? g[q] : 0.f;
    }
    const uint4 d = make_uint4(dmt::pack2<DT>(g[0], g[1]), dmt::pack2<DT>(g[2], g[3]),
                               dmt::pack2<DT>(g[4], g[5]), dmt::pack2<DT>(g[6], g[7]));
    *(uint4*)(dz + b * Op + o) = d;
    dmt::accumulate_chunk<DT>(s, d);
  }
#pragma unroll
  for (int q = 0; q < 8; ++q) red[threadIdx.x][q] = s[q];
  for (int h = rp / 2; h > 0; h >>= 1) {
    __syncthreads();
    if (rr < h)
#pragma unroll
      for (int q = 0; q < 8; ++q) red[threadIdx.x][q] += red[threadIdx.x + (h << tc)][q];
  }
  if (rr == 0 && o < Op) store_f32x8((float*)G.o1 + (int64_t)(lb % G.nbx) * Op, o, red[threadIdx.x]);
}

// Dot-product tower: dx[b][i][c] = dZ[b][np_pad + i n + c]
//                                  + sum over j != i (ascending j) of dZ[b][p(i,j)] x[b][j][c]
// with p the row-major index of the pair {i, j}.  One thread per element of dx.
// a = x, b = dZ, o0 = dx, n0 = B, i0 = nf, i1 = n, i2 = np_pad, i3 = ldz.
template <int DT>
__global__ __launch_bounds__(kBlock) void tmb_dot_bwd(const TmbLaunch L) {
  const int gi = tmb_find(L);
  const TmbItem& G = L.it[gi];
  const int nf = G.i0, n = G.i1, np_pad = G.i2, ldz = G.i3;
  const int wt = nf * n;
  const int64_t e = (int64_t)(blockIdx.x - L.block_start[gi]) * kBlock + threadIdx.x;
  if (e >= G.n0 * wt) return;
  const int64_t b = e / wt;
  const int r = (int)(e % wt), i = r / n, c = r % n;
  const float* __restrict__ z = (const float*)G.b + b * ldz;
  float acc = z[np_pad + r];
  for (int j = 0; j < nf; ++j) {
    if (j == i) continue;
    const int lo = j < i ? j : i, hi = j < i ? i : j;
    acc += z[lo * (2 * nf - lo - 1) / 2 + (hi - lo - 1)] * load_elt<DT>(G.a, b * wt + j * n + c);
  }
  ((float*)G.o0)[e] = acc;
}

// The same for the 16-bit types with n a multiple of 8: one thread per 8 consecutive columns
// of one feature, 16-byte accesses.
template <int DT>
__global__ __launch_bounds__(kBlock) void tmb_dot_bwd8(const TmbLaunch L) {
  const int gi = tmb_find(L);
  const TmbItem& G = L.it[gi];
  const int nf = G.i0, n = G.i1, np_pad = G.i2, ldz = G.i3;
  const int wt = nf * n, w8 = wt / 8;
  const int64_t e = (int64_t)(blockIdx.x - L.block_start[gi]) * kBlock + threadIdx.x;
  if (e >= G.n0 * w8) return;
  const int64_t b = e / w8;
  const int r = (int)(e % w8) * 8, i = r / n, c = r % n;
  const float* __restrict__ z = (const float*)G.b + b * ldz;
  const uint16_t* __restrict__ x = (const uint16_t*)G.a + b * wt + c;
  float acc[8];
  load_f32x8(z, np_pad + r, acc);
  for (int j = 0; j < nf; ++j) {
    if (j == i) continue;
    const int lo = j < i ? j : i, hi = j < i ? i : j;
    const float g = z[lo * (2 * nf - lo - 1) / 2 + (hi - lo - 1)];
    float xv[8];
    dmt::decode_chunk<DT>(xv, *(const uint4*)(x + j * n));
#pragma unroll
    for (int q = 0; q < 8; ++q) acc[q] += g * xv[q];
  }
  store_f32x8((float*)G.o0, b * wt + r, acc);
}

// ---- Dot towers of 2 to 8 features of a multiple of 32 columns, 16-bit types: the whole data gradient,
//   dx[b][i][c] = sum over o of dz[b][o] W[o][np + i n + c] + sum over j != i of dZ[b][p(i,j)] x[b][j][c],
//   dZ[b][p] = sum over o of dz[b][o] W[o][p],
// in one kernel.  Bound by the bytes of x and dx: the two contractions and tmb_dot_bwd8 moved the flat part of dZ,
// as large as dx, through memory and back.  8 towers of 8 features of 128 columns, 256 outputs, batch 8192: 77 + 12 +
// 148 us, now 116 (0.44 GB at 3.8 TB/s; without the products 105, without the requests of weights and dz 96) and 8 more in
// tmb_prep_dz, which repacks the weights (22 -> 30); 4 of 6 and 7 features, batch 2003: 17 + 16 us, now 15 + 1.
// A wave owns 16 or 32 samples and the same 32 columns of EVERY feature, the weights as the first operand, so that a lane
// holds one sample's values of all features at four consecutive columns and the sum over j needs no other lane's
// (x comes in the accumulators' layout, 16 bytes a lane).  Four waves share the weights of their columns, which go
// through LDS in steps of 32 outputs, fragment by fragment as the repacked weights lie; behind them come the dot
// terms' rows, whose products, a few floats a sample, take the way through LDS to the sample's other lanes.
constexpr int kDotZPitch = kDotTermTiles * 16 + 4; // floats: 16 samples' pieces of 16 bytes on different banks
// Of 128 samples: up to here blocks of 64 (dot_rows).  8 features of 64 columns to 256 outputs on 4 towers, backward, us, 128
// / 64: 192 blocks of 128 44.4 / 40.6, 256 46.0 / 42.7, 384 59.1 / 62.4; of 128 columns, 512 blocks 65.0 / 67.7.
constexpr int64_t kDotFewBlocks = 256;
// Term of the pair {i, j}, i < j, whatever the number of features.
__host__ __device__ constexpr int dot_slot(int i, int j) { return i * (2 * kDotFeat - 1 - i) / 2 + j - i - 1; }
// Fragments (1 KB) of a tower's repacked weights.
inline int64_t dot_wt_frags(int nf, int n, int64_t O) {
  return (int64_t)(n / kDotCols) * ((O + 31) / 32) * (nf * (kDotCols / 16) + kDotTermTiles);
}

// The weights as tmb_dot_dgrad stages them: [column block][step of 32 outputs][fragment][lane][8], a lane's eight
// values one column's of outputs 8 (lane / 16) ... of the step; fragments of the features, two each, then of the
// terms (rows in dot_slot order); zeros past the last output.  One thread per lane's eight values.
// a = W [O][np + nf n], c = where to, i0 = nf, i1 = n, i2 = O.
__device__ __forceinline__ void pack_dot_weights(const TmbItem& G, int64_t e) {
  const int nf = G.i0, n = G.i1, O = G.i2, np = nf * (nf - 1) / 2, ld = np + nf * n;
  const int tiles = nf * (kDotCols / 16) + kDotTermTiles, steps = (O + 31) / 32;
  if (e >= (int64_t)(n / kDotCols) * steps * tiles * 64) return;
  const int lane = (int)(e & 63), m = lane & 15;
  const int64_t frag = e >> 6;
  const int tile = (int)(frag % tiles), step = (int)(frag / tiles % steps), cb = (int)(frag / ((int64_t)tiles * steps));
  int col = -1;
  if (tile < 2 * nf) {
    col = np + (tile >> 1) * n + cb * kDotCols + (m >> 2) * 8 + (tile & 1) * 4 + (m & 3);
  } else {
    const int slot = (tile - 2 * nf) * 16 + m;
    for (int i = 0; i + 1 < nf; ++i)
      if (slot >= dot_slot(i, i + 1) && slot <= dot_slot(i, nf - 1)) col = i * (2 * nf - 1 - i) / 2 + slot - dot_slot(i, i + 1);
  }
  const int o0 = step * 32 + (lane >> 4) * 8;
  const uint16_t* __restrict__ W = (const uint16_t*)G.a;
  uint32_t v[8];
#pragma unroll
  for (int q = 0; q < 8; ++q) v[q] = col >= 0 && o0 + q < O ? W[(int64_t)(o0 + q) * ld + col] : 0u;
  ((uint4*)G.c)[e] = make_uint4(v[0] | v[1] << 16, v[2] | v[3] << 16, v[4] | v[5] << 16, v[6] | v[7] << 16);
}

// Three stages in LDS, requested two steps ahead (a step is short: 36 instructions of 16 x 16 x 32 a wave); the
// wave's own dz goes the same way, so that the requests under way can be counted.  The x values are requested
// ahead of the last step.
// S sets of 16 samples a wave: two, or one where that makes more of the blocks that a launch is short of (2 towers of 8
// features, batch 822: 16.7 -> 11.3 us; 4 of 6 and 7, batch 2003: 18.0 -> 15.1).
constexpr int dot_stage(int S) { return kDotTiles * 1024 + 4 * S * 1024; }      // bytes: weights, then dz (a fragment a set)
constexpr int dot_lds(int S) { return 3 * dot_stage(S); }
static_assert(dot_lds(1) >= dot_rows(1) * kDotZPitch * 4 && dot_lds(2) >= dot_rows(2) * kDotZPitch * 4 && 2 * dot_lds(2) <= 160 * 1024,
              "two blocks per CU");

// a = dz [B][Op], b = repacked weights, c = x, o0 = dx, n0 = B, i0 = nf, i1 = n, i2 = O, i3 = Op.
template <int DT, int S>
__global__ __launch_bounds__(kBlock, 2) void tmb_dot_dgrad(const TmbLaunch L) {
  static_assert(kBlock == 256, "four waves");
  extern __shared__ __attribute__((aligned(16))) uint16_t lds[];
  // the column blocks of the same samples run side by side on one XCD: they share lines of x and dz
  const int q8 = gridDim.x >> 3, r8 = gridDim.x & 7, xcd = blockIdx.x & 7;
  const int id = xcd * q8 + min(xcd, r8) + (blockIdx.x >> 3);
  int gi = 0;
  while (gi + 1 < L.n && id >= L.block_start[gi + 1]) ++gi;
  const TmbItem& G = L.it[gi];
  const int nf = G.i0, n = G.i1, Op = G.i3, steps = (G.i2 + 31) / 32;
  const int ncb = n / kDotCols, cb = (id - L.block_start[gi]) % ncb;
  const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), m = lane & 15, h = lane >> 4;
  const int64_t B = G.n0, s0 = (int64_t)((id - L.block_start[gi]) / ncb) * dot_rows(S) + wave * (16 * S);
  const int tiles = 2 * nf + kDotTermTiles, per_wave = (tiles + 3) / 4;
  const int64_t wt = (int64_t)nf * n;

  // a step's requests, 1 KB each: per_wave of the weights (the last waves' past the end are the last fragment again)
  // and the wave's two of dz
  const uint32_t panel = (uint32_t)(steps * tiles) * 1024u;
  const __amdgpu_buffer_rsrc_t wbuf = tm_buffer((const char*)G.b + (int64_t)cb * panel, panel);
  const int64_t mine = min(max(B - s0, (int64_t)0), (int64_t)(16 * S));
  const __amdgpu_buffer_rsrc_t zbuf = tm_buffer((const uint16_t*)G.a + min(s0, B - 1) * Op, (uint32_t)mine * (uint32_t)Op * 2u);
  const uint32_t lds0 = (uint32_t)(size_t)(__attribute__((address_space(3))) uint16_t*)lds;
  auto request = [&](int step) {
    const uint32_t to = lds0 + (uint32_t)(step % 3) * dot_stage(S), from = (uint32_t)(step * tiles) * 1024u + lane * 16u;
    for (int r = 0; r < per_wave; ++r) {
      const uint32_t t = (uint32_t)min(wave + 4 * r, tiles - 1) * 1024u;
      tm_request(to + t, wbuf, from + t);
    }
    const int k = step * 32 + h * 8;
#pragma unroll
    for (int s = 0; s < S; ++s)
      tm_request(to + kDotTiles * 1024 + (wave * S + s) * 1024, zbuf, k < Op ? (uint32_t)((s * 16 + m) * Op + k) * 2u : kOobOffset);
  };
  floatx4 acc[S][kDotFeat][2], accz[S][kDotTermTiles];
#pragma unroll
  for (int s = 0; s < S; ++s) {
#pragma unroll
    for (int i = 0; i < kDotFeat; ++i) acc[s][i][0] = acc[s][i][1] = floatx4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int t = 0; t < kDotTermTiles; ++t) accz[s][t] = floatx4{0.f, 0.f, 0.f, 0.f};
  }
  auto multiply = [&](int step) {
    const uint4* w = (const uint4*)(lds + (step % 3) * (dot_stage(S) / 2)) + lane;
    uint4 d[S];
#pragma unroll
    for (int s = 0; s < S; ++s) d[s] = w[(kDotTiles + wave * S + s) * 64];
#pragma unroll
    for (int i = 0; i < kDotFeat; ++i)
      if (i < nf) {
        const uint4 w0 = w[(2 * i) * 64], w1 = w[(2 * i + 1) * 64];
#pragma unroll
        for (int s = 0; s < S; ++s) acc[s][i][0] = mfma16<DT>(w0, d[s], acc[s][i][0]);
#pragma unroll
        for (int s = S - 1; s >= 0; --s) acc[s][i][1] = mfma16<DT>(w1, d[s], acc[s][i][1]);
      }
#pragma unroll
    for (int t = 0; t < kDotTermTiles; ++t) {
      const uint4 wz = w[(2 * nf + t) * 64];
#pragma unroll
      for (int s = 0; s < S; ++s) accz[s][t] = mfma16<DT>(wz, d[s], accz[s][t]);
    }
  };
  request(0);
  if (steps > 1) request(1);
  for (int step = 0; step + 1 < steps; ++step) {
    // all of this wave's requests but the next step's have landed; behind the barrier everyone's, and the stage of
    // the step before is read no more
    switch (per_wave + S) {
      case 3: asm volatile("s_waitcnt vmcnt(3)" ::: "memory"); break;
      case 4: asm volatile("s_waitcnt vmcnt(4)" ::: "memory"); break;
      case 5: asm volatile("s_waitcnt vmcnt(5)" ::: "memory"); break;
      case 6: asm volatile("s_waitcnt vmcnt(6)" ::: "memory"); break;
      default: asm volatile("s_waitcnt vmcnt(7)" ::: "memory"); break;
    }
    __syncthreads();
    if (step + 2 < steps) request(step + 2);
    multiply(step);
  }
  asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
  __syncthreads();
  uint4 xr[S][kDotFeat];
#pragma unroll
  for (int s = 0; s < S; ++s) {
    const uint16_t* x = (const uint16_t*)G.c + min(s0 + s * 16 + m, B - 1) * wt + cb * kDotCols + h * 8;
#pragma unroll
    for (int j = 0; j < kDotFeat; ++j) xr[s][j] = *(const uint4*)(x + (j < nf ? j : 0) * n);
  }
  multiply(steps - 1);
  // the samples' dZ to all their lanes, over the stages
  __syncthreads();
  float* const z_of = (float*)lds + (wave * 16 * S + m) * kDotZPitch;
#pragma unroll
  for (int s = 0; s < S; ++s)
#pragma unroll
    for (int t = 0; t < kDotTermTiles; ++t) *(floatx4*)(z_of + s * 16 * kDotZPitch + t * 16 + h * 4) = accz[s][t];
  // (a wave reads what its own lanes wrote)
  __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
  __builtin_amdgcn_wave_barrier();
  __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
#pragma unroll
  for (int s = 0; s < S; ++s) {
    float z[kDotTermTiles * 16];
#pragma unroll
    for (int q = 0; q < (kDotTerms + 3) / 4; ++q) {
      const floatx4 v = *(const floatx4*)(z_of + s * 16 * kDotZPitch + q * 4);
#pragma unroll
      for (int r = 0; r < 4; ++r) z[q * 4 + r] = v[r];
    }
    // Two stores of whole lines for the 16 samples of a feature: lane m of the first eight stores its own first four
    // columns and those of lane m + 8, the others its second four and those of lane m - 8.
    float* const out = (float*)G.o0 + (s0 + s * 16 + (m & 7)) * wt + cb * kDotCols + h * 8 + (m < 8 ? 0 : 4);
    const bool on[2] = {s0 + s * 16 + (m & 7) < B, s0 + s * 16 + (m & 7) + 8 < B};
#pragma unroll
    for (int t = 0; t < 2; ++t) {
      float x[kDotFeat][4];
#pragma unroll
      for (int j = 0; j < kDotFeat; ++j) {
        dmt::unpack2<DT>(t == 0 ? xr[s][j].x : xr[s][j].z, x[j][0], x[j][1]);
        dmt::unpack2<DT>(t == 0 ? xr[s][j].y : xr[s][j].w, x[j][2], x[j][3]);
      }
#pragma unroll
      for (int i = 0; i < kDotFeat; ++i)
        if (i < nf) {
#pragma unroll
          for (int j = 0; j < kDotFeat; ++j)
            if (j != i && j < nf) {
              const float g = z[i < j ? dot_slot(i, j) : dot_slot(j, i)];
#pragma unroll
              for (int r = 0; r < 4; ++r) acc[s][i][t][r] += g * x[j][r];
            }
        }
    }
#pragma unroll
    for (int i = 0; i < kDotFeat; ++i)
      if (i < nf) {
        floatx4 st[2];
#pragma unroll
        for (int r = 0; r < 4; ++r) {
          // row_ror:8, written in the last eight lanes of 16 and in the first
          const int a = __float_as_int(acc[s][i][0][r]), c = __float_as_int(acc[s][i][1][r]);
          st[0][r] = __int_as_float(__builtin_amdgcn_update_dpp(a, c, 0x128, 0xf, 0xc, false));
          st[1][r] = __int_as_float(__builtin_amdgcn_update_dpp(c, a, 0x128, 0xf, 0x3, false));
        }
        // (nontemporal: dx is read again by the sparse update only, and x, which the weight gradients read next, stays
        // in the caches: those 51 -> 42 us on 8 towers of 8 features of 128 columns, batch 8192.  At any size: whole
        // passes, plain / nontemporal, 27 MB of dx 157.7 / 158.4 us, 160 MB 493 / 487, 218 MB 616 / 610, 25 passes of 7 to
        // 268 MB 0.2 % shorter together.)
        if (on[0]) __builtin_nontemporal_store(st[0], (floatx4*)(out + i * n));
        if (on[1]) __builtin_nontemporal_store(st[1], (floatx4*)(out + 8 * wt + i * n));
      }
  }
}

// dw[o][k] = sum over slices s (ascending) of part[s][o][k'], where k' = k for k < np and
// k - np + np_pad after: adds up a split contraction's slices and drops the padding columns
// between the dot terms and the flat part (np = np_pad = 0: plain rows).
// a = part, o0 = dw, n0 = slice stride in floats, i0 = O, i1 = np, i2 = np_pad, i3 = wt,
// i4 = slices, i5 = many parts of one row (nbx = its blocks).
// A thread takes four consecutive elements of the slices (whose rows are multiples of four) and requests eight slices'
// together; bound by the reads of part.  (A block to 1024 columns of a row, 4 bytes a load, left every second block of
// 28 + 1024 columns with 28: 8 towers of 256 x 1052 in 8 slices 31.4 -> 14.3 us, 12 of 128 x 192 to 1536 in 16 36 -> 16.6.)
__global__ __launch_bounds__(kBlock) void tmb_sum_slices(const TmbLaunch L) {
  const int gi = tmb_find(L);
  const TmbItem& G = L.it[gi];
  const int np = G.i1, np_pad = G.i2, wt = G.i3, ns = G.i4, kin = np + wt;
  const int lb = blockIdx.x - L.block_start[gi];
  const float* __restrict__ p = (const float*)G.a;
  if (G.i5) {
    // many parts of one short row (a bias gradient): 32 columns a block, eight thread groups each
    // adding every eighth part, then the group sums in order
    __shared__ float red[8][33];
    const int c = threadIdx.x & 31, g = threadIdx.x >> 5, k = lb * 32 + c;
    float s = 0.f;
    if (k < kin)
#pragma unroll 8
      for (int q = g; q < ns; q += 8) s += p[q * G.n0 + k];
    red[g][c] = s;
    __syncthreads();
    if (g == 0 && k < kin) {
#pragma unroll
      for (int q = 1; q < 8; ++q) s += red[q][c];
      ((float*)G.o0)[k] = s;
    }
    return;
  }
  const int64_t e = ((int64_t)lb * kBlock + threadIdx.x) * 4;
  if (e >= G.n0) return;
  float s[4] = {0.f, 0.f, 0.f, 0.f};
  int q = 0;
  auto add = [&](auto together) __attribute__((always_inline)) {
    constexpr int N = decltype(together)::value;
    float4 v[N];
#pragma unroll
    for (int u = 0; u < N; ++u) v[u] = *(const float4*)(p + (q + u) * G.n0 + e);
#pragma unroll
    for (int u = 0; u < N; ++u) s[0] += v[u].x, s[1] += v[u].y, s[2] += v[u].z, s[3] += v[u].w;
    q += N;
  };
  while (q + 8 <= ns) add(std::integral_constant<int, 8>());
  if (q + 4 <= ns) add(std::integral_constant<int, 4>());
  while (q < ns) add(std::integral_constant<int, 1>());
  const uint32_t pitch = (uint32_t)(np_pad + wt);
  const int64_t o = np_pad == 0 ? 0 : G.n0 < (1LL << 32) ? (int64_t)((uint32_t)e / pitch) : e / pitch;
  const int64_t k = e - o * pitch;                 // (plain rows: all of them as one)
  float* __restrict__ out = (float*)G.o0 + o * kin;
  if (k >= np_pad) {
    // (from any 4-byte boundary: rows of 78 + 1664 columns, say; four stores of 4 bytes took 2 towers of 256 of these 4.3 us,
    // now 3.9)
    typedef float float4u __attribute__((ext_vector_type(4), aligned(4)));
    *(float4u*)(out + (k - np_pad + np)) = float4u{s[0], s[1], s[2], s[3]};
    return;
  }
#pragma unroll
  for (int j = 0; j < 4; ++j)
    if (k + j < np) out[k + j] = s[j];
}

// Cross layer backward of a float32 tower, elementwise part: du = dxn * x0;
// dx0 = (first ? 0 : dx0) + dxn * u (+ dxn when `last`: the layer's data-gradient contraction
// then accumulates du W_l on top, which completes dx_0 + dx0 in place).
// a = dxn, b = x0, c = u, o0 = du, o1 = dx0, n0 = elements, i0 = first, i1 = last, nbx = blocks.
__global__ __launch_bounds__(kBlock) void tmb_cross_prep(const TmbLaunch L) {
  const int gi = tmb_find(L);
  const TmbItem& G = L.it[gi];
  const float* __restrict__ dxn = (const float*)G.a;
  const float* __restrict__ x0 = (const float*)G.b;
  const float* __restrict__ u = (const float*)G.c;
  float* __restrict__ du = (float*)G.o0;
  float* __restrict__ dx0 = (float*)G.o1;
  const float keep = G.i1 ? 1.f : 0.f;
  const int64_t stride = (int64_t)G.nbx * kBlock;
  for (int64_t e = (int64_t)(blockIdx.x - L.block_start[gi]) * kBlock + threadIdx.x; e < G.n0; e += stride) {
    const float g = dxn[e];
    float acc = G.i0 ? 0.f : dx0[e];
    acc += g * u[e] + keep * g;
    du[e] = x0[e] * g;
    dx0[e] = acc;
  }
}

// ----------------------------------------------------------------- host side

inline int64_t up8(int64_t v) { return (v + 7) / 8 * 8; }

inline bool is_cross(const dmt_tm_params& q) {
  return q.kind == DMT_TM_CROSS_LINEAR || q.kind == DMT_TM_CROSS_LOWRANK_LINEAR;
}

// Rows of dy per block of tmb_prep_dz: at most kPrepParts blocks along the rows, so that the bias
// gradient has few parts to add.
constexpr int kPrepParts = 128;
inline int64_t prep_rows(int64_t rows) {
  int64_t r = 16;
  while ((rows + r - 1) / r > kPrepParts) r *= 2;
  return r;
}

// Output tiles of the contractions of one launch (all towers), in both tile sizes.
struct TileCount {
  int64_t t128 = 0, t256 = 0;
  bool wide = true;            // no group is too narrow for 256 x 256 tiles
  void add(int64_t m, int64_t n) {
    t128 += ((m + 127) / 128) * ((n + 127) / 128);
    t256 += ((m + 255) / 256) * ((n + 255) / 256);
    wide = wide && m > 128 && n > 128;
  }
};

// Slices a weight-gradient contraction (K = batch) is cut into: so many that the launch's tiles
// fill the CUs once, as nearly as they can without a second, mostly empty round: 256 x 256 tiles
// (one to a CU) while a slice stays at least 1024 long, else 128 x 128 (two to a CU) and at least 512.
inline void choose_split(const dmt_plan* p, const TileCount& n, int64_t K, int* ksplit, int* klen) {
  // No slices where the 128 x 128 tiles alone are three for every four slots, but for two of 4096 and more, which
  // make enough 256 x 256 tiles: what these save then is more than adding the slices up takes.  Backward, 128 x 128 /
  // two slices, us: 12 towers of 1024 columns to 512 outputs (384 tiles), batch 4096 215.3 / 203.0, 8192 390.3 /
  // 356.0, 16384 722.8 / 643.7, 22 of them (704) 390.2 / 395.2, 691.4 / 671.4 and 1327 / 1254; 23 of 768 columns to 400 331.1 /
  // 359.0, 682.5 / 677.9 and 1213 / 1180; rank 512 beside 2048 columns, 8 towers, 737.2 / 745.2 and 1363 / 1323.
  int64_t ks = 1;
  const bool enough = n.wide ? n.t256 >= kBigTiles || n.t128 >= 384 : false;
  if (enough && n.t256 < kBigTiles && n.t256 * 2 >= kBigTiles && K >= 8192) ks = 2;
  if (n.wide && !enough) ks = std::min<int64_t>(16, 256 / std::max<int64_t>(n.t256, 1));
  if (!enough && (!n.wide || n.t256 * ks < kBigTiles || K / ks < 1024)) {
    ks = std::max<int64_t>(1, std::min<int64_t>(16, 512 / std::max<int64_t>(n.t128, 1)));
    while (ks > 1 && K / ks < 512) --ks;
  }
  // A long batch with few tiles (narrow outputs: the contraction is bound by memory latency)
  // measured faster in slices of about 4096 spread over several rounds (12 towers of 128 outputs,
  // batch 65536: 0.54 against 0.73 ms) than in one round of very long slices.
  if (!n.wide && n.t128 < 512 && K / ks > 4096) ks = std::min<int64_t>(16, (K + 4095) / 4096);
  const int forced = p->sw.tmb_ksplit;
  if (forced > 0 && K / forced >= 128) ks = forced;
  int len = (int)((K + ks - 1) / ks);
  len = (len + BK - 1) / BK * BK;
  *ksplit = (int)((K + len - 1) / len);
  *klen = len;
}

struct TowerBwdWs {
  int np = 0, np_pad = 0;
  bool packed = false;         // dot towers: the projection's weights are read from a repacked copy,
  int skip = 0;                // whose rows (or the weights' own) start with this many columns for the dot terms
  int kin = 0;                 // row length of dZ and of the weight gradient's slices (np_pad + wt for dots)
  int64_t Op = 0;
  size_t dz = 0, dbp = 0;      // dy rounded, [B][Op]; parts of its column sums
  size_t p = 0, wp = 0, dZ = 0;                                 // dot towers
  bool fused = false;          // dot towers: tmb_dot_dgrad, its weights in wp; dZ is not used
  bool dZ_behind = false;      // dot towers that tmb_dot_dgrad could serve: dZ lies behind all other pieces
  size_t xl[DMT_MAX_CROSS_LAYERS] = {}, u[DMT_MAX_CROSS_LAYERS] = {};   // cross towers
  size_t dxn = 0, du[2] = {0, 0}, dbc = 0;   // g_l, du of alternating layers, parts of its column sums
  // low-rank cross towers: t_l = V_l x_l per layer; dt (float32 towers), dt rounded
  size_t tl[DMT_MAX_CROSS_LAYERS] = {};
  size_t dtf = 0, dtq = 0;
  // DLRM towers: the shared per-feature layer's operands (rows = (sample, feature))
  int64_t Fp = 0;              // feat_out padded to 8
  size_t dz2 = 0, dbp2 = 0, part2 = 0;
  int ksplit2 = 1, klen2 = 0;
  size_t part = 0;             // weight-gradient slices (split K) / padded dW of a dot tower
  int ksplit = 1, klen = 0;    // of the projection's weight gradient
  int ksplit_c = 1, klen_c = 0;   // of the cross layers' weight gradients
};

dmt_status plan_tm_bwd(const dmt_plan* p, const dmt_tm_params* tp, int64_t B, int eb,
                       bool have_kept, std::vector<TowerBwdWs>* ws, size_t* bytes) {
  size_t off = 0;
  auto take = [&](size_t b) { size_t o = off; off = dmt_align_up(off + b, 256); return o; };
  ws->assign(p->T, TowerBwdWs());
  // output tiles of the weight-gradient launches (all towers together)
  TileCount tiles_proj, tiles_cross, tiles_feat;
  for (int32_t t = 0; t < p->T; ++t) {
    const dmt_tm_params& q = tp[t];
    const int64_t wt = p->tower_width[t];
    if (q.out_dim <= 0) return DMT_EINVAL;
    tiles_proj.add(q.out_dim, wt);
    if (q.kind == DMT_TM_CROSS_LINEAR) tiles_cross.add(wt, wt);
    if (q.kind == DMT_TM_CROSS_LOWRANK_LINEAR) tiles_cross.add(wt, q.feat_out);
    if (q.kind == DMT_TM_DLRM) tiles_feat.add(q.feat_out, p->tower_uniform_dim[t]);
  }
  const DotDgrad dots = dot_dgrad_of(p, tp, B);
  for (int32_t t = 0; t < p->T; ++t) {
    const dmt_tm_params& q = tp[t];
    const int64_t wt = p->tower_width[t];
    if (!q.w_proj || !q.b_proj) return DMT_EINVAL;
    if (((uintptr_t)q.w_proj & 15) && q.kind != DMT_TM_DOT_LINEAR) return DMT_EINVAL;
    TowerBwdWs& w = (*ws)[t];
    w.kin = (int)wt;
    if (eb == 2) {
      choose_split(p, tiles_proj, B, &w.ksplit, &w.klen);
      choose_split(p, tiles_cross, B, &w.ksplit_c, &w.klen_c);
    }
    switch (q.kind) {
      case DMT_TM_LINEAR:
      case DMT_TM_LINEAR_RELU:
        break;
      case DMT_TM_DOT_LINEAR: {
        const int nf = p->tower_ntab[t];
        if (p->tower_uniform_dim[t] == 0) return DMT_ENOTSUP;
        w.np = nf * (nf - 1) / 2;
        w.np_pad = (w.np + 7) / 8 * 8;
        const bool fusable = eb == 2 && dot_dgrad_ok(p, nf, p->tower_uniform_dim[t], q.out_dim);
        w.fused = fusable && dot_one_kernel(p, t, q.out_dim, dots);
        w.packed = !w.fused && !dot_weights_as_is(q.w_proj, w.np);
        w.skip = w.packed ? w.np_pad : w.np;
        w.kin = w.np_pad + (int)wt;
        w.p = take((size_t)B * w.np_pad * eb);
        // (room for either way, here and in dZ: a workspace sized for a larger batch serves a smaller one, which may go
        // the other)
        w.wp = take(std::max((size_t)q.out_dim * w.kin * eb,
                             fusable ? (size_t)dot_wt_frags(nf, p->tower_uniform_dim[t], q.out_dim) * 1024 : 0));
        if (!fusable) w.dZ = take((size_t)B * w.kin * 4);
        w.dZ_behind = fusable;
        break;
      }
      case DMT_TM_CROSS_LINEAR:
      case DMT_TM_CROSS_LOWRANK_LINEAR: {
        const bool low = q.kind == DMT_TM_CROSS_LOWRANK_LINEAR;
        const int L = q.num_cross_layers, r = q.feat_out, step = low ? 2 : 1;
        if (L < 1 || step * L > DMT_MAX_CROSS_LAYERS || (low && r < 1)) return DMT_EINVAL;
        if (low && eb == 2 && r % 8 != 0) return DMT_ENOTSUP;
        for (int l = 0; l < L; ++l) {
          if (!q.b_cross[l]) return DMT_EINVAL;
          for (int i = l * step; i < (l + 1) * step; ++i)
            if (!q.w_cross[i] || ((uintptr_t)q.w_cross[i] & 15)) return DMT_EINVAL;
        }
        for (int l = 0; l < L; ++l) {
          if (low) w.tl[l] = take((size_t)B * r * eb);
          if (have_kept) continue;                  // the forward kept them
          w.xl[l] = take((size_t)B * wt * eb);      // x_{l+1}
          w.u[l] = take((size_t)B * wt * eb);
        }
        w.dxn = take((size_t)B * wt * 4);
        w.du[0] = take((size_t)B * wt * eb);
        w.du[1] = take((size_t)B * wt * eb);
        w.dbc = take((size_t)((B + 63) / 64) * wt * 4);
        if (low) {
          w.dtf = take((size_t)B * r * 4);
          w.dtq = take((size_t)B * r * eb);
        }
        break;
      }
      case DMT_TM_DLRM: {
        const int nf = p->tower_ntab[t], n = p->tower_uniform_dim[t];
        if (n == 0) return DMT_ENOTSUP;
        if (q.feat_out < 1 || (int64_t)q.out_dim - (int64_t)nf * q.feat_out < 1) return DMT_EINVAL;
        if (!q.w_cross[0] || !q.b_cross[0] || ((uintptr_t)q.w_cross[0] & 15)) return DMT_EINVAL;
        if (B * nf >= (1LL << 31) - 128) return DMT_ENOTSUP;
        w.Fp = up8(q.feat_out);
        w.dz2 = take((size_t)B * nf * w.Fp * eb);
        w.dbp2 = take((size_t)kPrepParts * w.Fp * 4);
        if (eb == 2) choose_split(p, tiles_feat, B * nf, &w.ksplit2, &w.klen2);
        if (w.ksplit2 > 1) w.part2 = take((size_t)w.ksplit2 * q.feat_out * n * 4);
        break;
      }
      default:
        return DMT_EINVAL;
    }
    // rows of the projection's gradient operand: all outputs, or a DLRM tower's flat outputs
    const int64_t O1 = q.kind == DMT_TM_DLRM ? q.out_dim - p->tower_ntab[t] * q.feat_out : q.out_dim;
    w.Op = up8(O1);
    w.dz = take((size_t)B * w.Op * eb);
    w.dbp = take((size_t)kPrepParts * w.Op * 4);
    size_t part = 0;
    if (w.ksplit > 1 || q.kind == DMT_TM_DOT_LINEAR)
      part = (size_t)w.ksplit * O1 * w.kin * 4;
    if (q.kind == DMT_TM_CROSS_LINEAR && w.ksplit_c > 1)
      part = std::max(part, (size_t)w.ksplit_c * wt * wt * 4);
    if (q.kind == DMT_TM_CROSS_LOWRANK_LINEAR && w.ksplit_c > 1)
      part = std::max(part, (size_t)w.ksplit_c * wt * q.feat_out * 4);
    if (part) w.part = take(part);
  }
  // (tmb_dot_dgrad does without; between the pieces it uses, that room made 6 features of 128 columns, batch 16384, 163 ->
  // 171 us)
  for (TowerBwdWs& w : *ws)
    if (w.dZ_behind) w.dZ = take((size_t)B * w.kin * 4);
  *bytes = off;
  return DMT_OK;
}

// Items of one grouped launch of a small kernel, with each item's block count.
struct TmbBatch {
  std::vector<TmbItem> items;
  std::vector<int64_t> blocks;
  void add(const TmbItem& it, int64_t nblocks) {
    if (nblocks <= 0) return;
    items.push_back(it);
    blocks.push_back(nblocks);
  }
};

// False when an item alone exceeds the grid limit (nothing of it is launched).
template <typename Kernel>
bool launch_items(const dmt_plan* p, TmbBatch& batch, Kernel kernel, hipStream_t s, int lds = 0, int kid = DMT_K_TM_BWD_AUX) {
  bool ok = true;
  for (size_t first = 0; first < batch.items.size();) {
    TmbLaunch L;
    L.n = 0;
    int64_t blocks = 0;
    while (first < batch.items.size() && L.n < kMaxItems &&
           blocks + batch.blocks[first] < (1LL << 30)) {
      L.it[L.n] = batch.items[first];
      L.block_start[L.n] = (int32_t)blocks;
      blocks += batch.blocks[first];
      ++L.n;
      ++first;
    }
    if (L.n == 0) { ok = false; break; }
    L.block_start[L.n] = (int32_t)blocks;
    DmtScope sc_(p, kid, s);
    hipLaunchKernelGGL(kernel, dim3((unsigned)blocks), dim3(kBlock), lds, s, L);
  }
  batch.items.clear();
  batch.blocks.clear();
  return ok;
}

inline int64_t ew_blocks(int64_t count) { return std::min<int64_t>((count + kBlock - 1) / kBlock, 256 * 8); }

// One tower's rounded gradient operand and its column sums' parts.
template <int DT>
void add_prep(TmbBatch& b, TmbItem it) {
  it.n1 = prep_rows(it.n0);
  it.nbx = (int32_t)((it.n0 + it.n1 - 1) / it.n1);
  it.i5 = 0;
  while (it.i5 < 5 && (8 << it.i5) < it.i1) ++it.i5;
  b.add(it, (int64_t)it.nbx * ((it.i1 + (8 << it.i5) - 1) / (8 << it.i5)));
}

// A weight gradient's K slices: adds `slices` blocks of rows x (np_pad + cols) up.
void add_slices(TmbBatch& b, const void* part, int rows, int np, int np_pad, int cols, int slices, float* out) {
  TmbItem it{};
  it.a = part; it.o0 = out; it.n0 = (int64_t)rows * (np_pad + cols);
  it.i0 = rows; it.i1 = np; it.i2 = np_pad; it.i3 = cols; it.i4 = slices;
  b.add(it, (it.n0 / 4 + kBlock - 1) / kBlock);
}

// out[e] = sum over parts of part[q * stride + e], e < n.
void add_sum(TmbBatch& b, const void* part, int64_t stride, int64_t parts, float* out, int n) {
  TmbItem it{};
  it.a = part; it.o0 = out; it.n0 = stride; it.i0 = 1; it.i3 = n; it.i4 = (int32_t)parts;
  it.i5 = 1;
  it.nbx = (n + 31) / 32;
  b.add(it, it.nbx);
}

template <int DT>
dmt_status run_tm_bwd(const dmt_plan* p, const dmt_tm_params* tp, const std::vector<TowerBwdWs>& ws,
                      const void* pooled, const void* tm_out, int64_t B, const float* dy_all,
                      float* dx_all, const dmt_tm_grads* gr, const char* keptp, char* wsp,
                      hipStream_t s) {
  static_assert(DT != DMT_F32, "float32 towers: run_tm_bwd_f32");
  constexpr int eb = 2;
  const char* x_all = (const char*)pooled;
  std::vector<int64_t> out_prefix(p->T + 1, 0);
  for (int32_t t = 0; t < p->T; ++t) out_prefix[t + 1] = out_prefix[t] + tp[t].out_dim;
  auto x_of = [&](int t) { return (const void*)(x_all + (size_t)B * p->width_prefix[t] * eb); };
  auto dx_of = [&](int t) { return dx_all + (size_t)B * p->width_prefix[t]; };
  // x_l and u_l of a cross tower (x_0 is the pooled block itself): kept by the forward, or
  // recomputed below into the workspace
  std::vector<TmKept> kept;
  if (keptp) plan_tm_kept(p, tp, B, eb, &kept);
  auto xl_of = [&](int t, int l) -> const void* {
    if (l == 0) return x_of(t);
    return keptp ? (const void*)(keptp + kept[t].x[l - 1]) : (const void*)(wsp + ws[t].xl[l - 1]);
  };
  auto u_of = [&](int t, int l) -> const void* {
    return keptp ? (const void*)(keptp + kept[t].u[l]) : (const void*)(wsp + ws[t].u[l]);
  };
  int max_layers = 0;
  TmbBatch batch, batch2, batch3, groups_dot, dots_fused;
  bool ok = true;

  auto z_of = [&](int t) -> const char* {           // dot terms: kept by the forward, or recomputed
    return keptp && kept[t].has_z ? keptp + kept[t].z : (const char*)(wsp + ws[t].p);
  };
  // The projection's weights, repacked where they must be.  The forward has kept a repacked copy if the
  // terms are odd; if they are even, whether ITS weights were 4-byte aligned is more than the weights at hand tell.
  auto kept_wp = [&](int t) { return keptp && kept[t].has_wp; };
  auto wp_of = [&](int t) -> const char* {
    if (!ws[t].packed) return (const char*)tp[t].w_proj;
    return kept_wp(t) ? keptp + kept[t].wp : (const char*)(wsp + ws[t].wp);
  };
  // ---- recompute what the forward did not keep: dot terms (and the repacked weights)
  std::vector<TmAuxItem> dots_mfma, dots_simple, packs;
  std::vector<int64_t> nb_mfma, nb_simple, nb_pack;
  for (int32_t t = 0; t < p->T; ++t) {
    const dmt_tm_params& q = tp[t];
    if (is_cross(q)) max_layers = std::max(max_layers, q.num_cross_layers);
    if (q.kind != DMT_TM_DOT_LINEAR) continue;
    const TowerBwdWs& w = ws[t];
    TmAuxItem it{};
    it.nf = p->tower_ntab[t]; it.n = p->tower_uniform_dim[t]; it.np = w.np; it.np_pad = w.np_pad;
    it.O = q.out_dim; it.wt = p->tower_width[t];
    it.src = x_of(t);
    it.dst = wsp + w.p;
    if (w.np_pad > 0 && !(keptp && kept[t].has_z)) {
      if (dots_mfma_ok(it.nf, it.n)) {
        dots_mfma.push_back(it);
        nb_mfma.push_back(dots_mfma_blocks(B, it.nf));
      } else {
        dots_simple.push_back(it);
        nb_simple.push_back((B * w.np_pad + kBlock - 1) / kBlock);
      }
    }
    if (!w.packed || kept_wp(t)) continue;
    it.src = q.w_proj;
    it.dst = wsp + w.wp;
    packs.push_back(it);
    nb_pack.push_back(((int64_t)q.out_dim * w.kin + kBlock - 1) / kBlock);
  }
  launch_aux<DT>(p, B, dots_mfma, nb_mfma, 0, s);
  launch_aux<DT>(p, B, dots_simple, nb_simple, 1, s);
  launch_aux<DT>(p, B, packs, nb_pack, 2, s);

  auto group = [&](const void* A, int64_t lda, int64_t K, const void* W, int64_t ldw, int64_t M, int64_t N, void* C,
                   int64_t ldc, int epi) {
    TmGroup g{};
    g.A1 = A; g.lda1 = (int32_t)lda; g.K1 = (int32_t)K;
    g.W1 = W; g.ldw1 = (int32_t)ldw;
    g.M = (int32_t)M; g.N = (int32_t)N; g.C = C; g.ldc = (int32_t)ldc; g.epi = epi;
    return g;
  };
  constexpr int kid = DMT_K_TM_BWD_GEMM;

  // ---- ... and the cross layers' u_l = x_l W_l^T + b_l, x_{l+1} = x0 * u_l + x_l, both from one
  // contraction as in the training forward (low-rank layers: t_l = x_l V_l^T first, which the
  // backward needs whether or not the rest was kept, then u_l = t_l U_l^T + b_l)
  std::vector<TmGroup> groups, groups_t;
  for (int l = 0; l < max_layers; ++l) {
    for (int32_t t = 0; t < p->T; ++t) {
      const dmt_tm_params& q = tp[t];
      if (!is_cross(q) || l >= q.num_cross_layers) continue;
      const int wt = p->tower_width[t], r = q.feat_out;
      const bool low = q.kind == DMT_TM_CROSS_LOWRANK_LINEAR;
      if (low)
        groups_t.push_back(group(xl_of(t, l), wt, wt, q.w_cross[2 * l], wt, B, r, wsp + ws[t].tl[l], r, EPI_BIAS));
      if (keptp) continue;
      // exactly the training forward's contraction: x_{l+1} from the cross epilogue, u_l on the side
      TmGroup g = low ? group(wsp + ws[t].tl[l], r, r, q.w_cross[2 * l + 1], r, B, wt, wsp + ws[t].xl[l], wt, EPI_CROSS)
                      : group(xl_of(t, l), wt, wt, q.w_cross[l], wt, B, wt, wsp + ws[t].xl[l], wt, EPI_CROSS);
      g.bias = q.b_cross[l];
      g.X0 = x_of(t); g.ldx = wt; g.XL = xl_of(t, l); g.ldxl = wt;
      g.U = wsp + ws[t].u[l];
      groups.push_back(g);
    }
    launch_groups<DT>(p, groups_t, s, false, kid);
    launch_groups<DT>(p, groups, s, false, kid);
  }

  // The gradient of layer l of a cross tower (l = its number of layers: of the projection) out of the
  // contraction g: what its epilogue reads and leaves for the layer below.
  auto cross_grad = [&](TmGroup& g, int t, int l) {
    const dmt_tm_params& q = tp[t];
    const TowerBwdWs& w = ws[t];
    const int L = q.num_cross_layers, wt = p->tower_width[t];
    g.ldc = wt;
    if (l == 0) {
      g.epi = EPI_F32_ADD;
      g.C = dx_of(t);
      return;
    }
    g.epi = EPI_CROSS_GRAD;
    g.X0 = x_of(t); g.ldx = wt;
    if (l < L) { g.GN = (const float*)(wsp + w.dxn); g.UL = u_of(t, l); }
    if (l == 1) g.U0 = u_of(t, 0);
    g.C = l > 1 ? (void*)(wsp + w.dxn) : nullptr;
    g.ACC = dx_of(t);
    g.acc_first = l == L || l == L - 1;
    g.DU = wsp + w.du[(l - 1) & 1];
    g.DBP = (float*)(wsp + w.dbc);
  };
  const int64_t cross_parts = (B + 63) / 64;

  // ---- projections: gradient operands, then both contractions for all towers
  std::vector<TmGroup> dgrad, dgrad2, wgrad, wgrad2;
  for (int32_t t = 0; t < p->T; ++t) {
    const dmt_tm_params& q = tp[t];
    const TowerBwdWs& w = ws[t];
    const int wt = p->tower_width[t], nf = p->tower_ntab[t];
    const bool dot = q.kind == DMT_TM_DOT_LINEAR;
    const bool dlrm = q.kind == DMT_TM_DLRM;
    // outputs of the projection: all of the tower's, or a DLRM tower's flat ones
    const int O = dlrm ? q.out_dim - nf * q.feat_out : q.out_dim;
    const char* dz = wsp + w.dz;
    {
      TmbItem it{};
      it.a = dy_all + (size_t)B * out_prefix[t];
      it.i2 = q.kind == DMT_TM_LINEAR_RELU;
      it.b = it.i2 ? (const void*)((const char*)tm_out + (size_t)B * out_prefix[t] * eb) : nullptr;
      it.o0 = wsp + w.dz; it.o1 = wsp + w.dbp;
      it.n0 = B; it.n2 = q.out_dim; it.i0 = O; it.i1 = (int32_t)w.Op;
      add_prep<DT>(batch, it);
      add_sum(batch2, wsp + w.dbp, w.Op, (B + prep_rows(B) - 1) / prep_rows(B), gr[t].db_proj, O);
    }
    // weight gradient: x (or the last cross layer's output, or the dot terms and x) on dz
    const bool to_part = dot || w.ksplit > 1;
    float* dw = to_part ? (float*)(wsp + w.part) : gr[t].dw_proj;
    auto add_wgrad = [&](std::vector<TmGroup>& to, const void* z, int64_t ldz, int N, float* C) {
      TmGroup h = group(dz, w.Op, B, z, ldz, O, N, C, w.kin, EPI_F32);
      h.ksplit = w.ksplit; h.klen = w.klen; h.cstride = (int64_t)O * w.kin;
      to.push_back(h);
    };
    add_wgrad(wgrad, is_cross(q) ? xl_of(t, q.num_cross_layers) : x_of(t), wt, wt, dw + w.np_pad);
    if (w.np > 0) add_wgrad(wgrad2, z_of(t), w.np_pad, w.np_pad, dw);
    if (to_part) add_slices(batch2, wsp + w.part, O, w.np, w.np_pad, wt, w.ksplit, gr[t].dw_proj);
    // data gradient
    if (dot && w.fused) {
      const int n = p->tower_uniform_dim[t];
      TmbItem it{};
      it.a = q.w_proj; it.c = wsp + w.wp; it.i0 = nf; it.i1 = n; it.i2 = O;
      batch.add(it, (dot_wt_frags(nf, n, O) * 64 + kBlock - 1) / kBlock);
      it = TmbItem{};
      it.a = dz; it.b = wsp + w.wp; it.c = x_of(t); it.o0 = dx_of(t); it.n0 = B;
      it.i0 = nf; it.i1 = n; it.i2 = O; it.i3 = (int32_t)w.Op;
      dots_fused.add(it, (B + dot_rows(2) - 1) / dot_rows(2) * (n / kDotCols));
    } else if (dot) {
      const int64_t ldw = w.skip + wt;
      const char* W = wp_of(t);
      float* dZ = (float*)(wsp + w.dZ);
      // (the padding columns receive whatever weights follow the terms': nothing reads them)
      if (w.np > 0) dgrad2.push_back(group(dz, w.Op, O, W, ldw, B, w.np_pad, dZ, w.kin, EPI_F32));
      dgrad.push_back(group(dz, w.Op, O, W + (size_t)w.skip * eb, ldw, B, wt, dZ + w.np_pad, w.kin, EPI_F32));
      TmbItem it{};
      it.a = x_of(t); it.b = dZ; it.o0 = dx_of(t); it.n0 = B;
      it.i0 = nf; it.i1 = p->tower_uniform_dim[t]; it.i2 = w.np_pad; it.i3 = w.kin;
      if (it.i1 % 8 == 0) batch3.add(it, (B * (wt / 8) + kBlock - 1) / kBlock);
      else groups_dot.add(it, (B * wt + kBlock - 1) / kBlock);
    } else if (dlrm) {
      // the shared per-feature layer: rows (sample, feature)
      const int n = p->tower_uniform_dim[t], F = q.feat_out;
      const int64_t BF = B * nf;
      TmbItem it{};
      it.a = dy_all + (size_t)B * out_prefix[t] + O;
      it.o0 = wsp + w.dz2; it.o1 = wsp + w.dbp2;
      it.n0 = BF; it.n2 = q.out_dim; it.i0 = F; it.i1 = (int32_t)w.Fp;
      it.i3 = nf; it.i4 = F;
      add_prep<DT>(batch, it);
      add_sum(batch2, wsp + w.dbp2, w.Fp, (BF + prep_rows(BF) - 1) / prep_rows(BF), gr[t].db_cross[0], F);
      // data gradient, both layers in one contraction per feature f: the pooled block's columns
      // f n .. f n + n - 1 receive [dz1 | dz2 of feature f] . [W1 columns f n .. | W_f], so
      // grad_pooled is written once.  (A group per feature filled four launches of the 16 groups that
      // kernel arguments hold, where one does: 54 us for 8 towers of 8 features, batch 4096, now 48.)
      TmGroup g = group(wsp + w.dz2, nf * w.Fp, F, q.w_cross[0], n, B, n, dx_of(t), wt, EPI_F32);
      g.A0 = dz; g.lda0 = (int32_t)w.Op; g.K0 = O;
      g.W0 = q.w_proj; g.ldw0 = wt;
      g.reps = nf; g.a1_step = (int32_t)w.Fp; g.w0_step = n; g.cstride = n;
      dgrad2.push_back(g);
      TmGroup h = group(wsp + w.dz2, w.Fp, BF, x_of(t), n, F, n, w.ksplit2 > 1 ? (void*)(wsp + w.part2) : gr[t].dw_cross[0],
                        n, EPI_F32);
      h.ksplit = w.ksplit2; h.klen = w.klen2; h.cstride = (int64_t)F * n;
      wgrad2.push_back(h);
      if (w.ksplit2 > 1) add_slices(batch2, wsp + w.part2, F, 0, 0, n, w.ksplit2, gr[t].dw_cross[0]);
    } else {
      TmGroup g = group(dz, w.Op, O, q.w_proj, wt, B, wt, dx_of(t), wt, EPI_F32);
      if (is_cross(q)) cross_grad(g, t, q.num_cross_layers);
      dgrad.push_back(g);
    }
  }
  ok &= launch_items(p, batch, tmb_prep_dz<DT>, s);
  // (The dot terms' and the per-feature layers' contractions are narrow: where the flat ones take 128 x 128
  // tiles as well, both go into one launch.  6 and 7 features on 4 towers, batch 2003: data gradients
  // 18.9 + 8.1 us, now 18.8; weight gradients 17.4 + 11.7, now 15.2.)
  auto join = [&](std::vector<TmGroup>& wide, std::vector<TmGroup>& narrow) {
    if (wide.empty() || wide.size() + narrow.size() > kMaxGroups || take_big(p, wide.data(), (int)wide.size())) return;
    wide.insert(wide.end(), narrow.begin(), narrow.end());
    narrow.clear();
  };
  join(dgrad, dgrad2);
  join(wgrad, wgrad2);
  launch_groups<DT, OP_ROW, OP_COL>(p, dgrad, s, false, kid);
  launch_groups<DT, OP_ROW, OP_COL>(p, dgrad2, s, false, kid);
  if (!dots_fused.items.empty()) {
    int64_t blocks = 0;
    for (int64_t b : dots_fused.blocks) blocks += b;
    if (blocks <= kDotFewBlocks) {
      for (size_t i = 0; i < dots_fused.items.size(); ++i)
        dots_fused.blocks[i] = (B + dot_rows(1) - 1) / dot_rows(1) * (dots_fused.items[i].i1 / kDotCols);
      static DmtPerDevice configured;
      dmt_allow_lds(configured, (const void*)tmb_dot_dgrad<DT, 1>, dot_lds(1));
      ok &= launch_items(p, dots_fused, tmb_dot_dgrad<DT, 1>, s, dot_lds(1), kid);
    } else {
      static DmtPerDevice configured;
      dmt_allow_lds(configured, (const void*)tmb_dot_dgrad<DT, 2>, dot_lds(2));
      ok &= launch_items(p, dots_fused, tmb_dot_dgrad<DT, 2>, s, dot_lds(2), kid);
    }
  }
  launch_groups<DT, OP_COL, OP_COL>(p, wgrad, s, false, kid);
  launch_groups<DT, OP_COL, OP_COL>(p, wgrad2, s, false, kid);
  // ---- weight gradients: add up the slices, strip a dot tower's padding; dot towers: fold
  // the dot terms' gradients into dx
  ok &= launch_items(p, batch2, tmb_sum_slices, s);
  ok &= launch_items(p, groups_dot, tmb_dot_bwd<DT>, s);
  ok &= launch_items(p, batch3, tmb_dot_bwd8<DT>, s);

  // ---- cross towers: layers from the last to the first.  du_l and its column sums' parts were left by
  // the contraction above; grad_pooled accumulates along the way and the first layer's data
  // gradient lands on top of it.
  TmbBatch sums, sums2;
  for (int l = max_layers - 1; l >= 0; --l) {
    for (int32_t t = 0; t < p->T; ++t) {
      const dmt_tm_params& q = tp[t];
      if (!is_cross(q) || l >= q.num_cross_layers) continue;
      const TowerBwdWs& w = ws[t];
      const int wt = p->tower_width[t];
      const char* du = wsp + w.du[l & 1];
      const bool split = w.ksplit_c > 1;
      add_sum(sums, wsp + w.dbc, wt, cross_parts, gr[t].db_cross[l], wt);
      auto add_wgrad = [&](std::vector<TmGroup>& to, TmbBatch& sum, const void* d, int rows, const void* x, int cols, float* dw) {
        TmGroup h = group(d, rows, B, x, cols, rows, cols, split ? (void*)(wsp + w.part) : (void*)dw, cols, EPI_F32);
        h.ksplit = w.ksplit_c; h.klen = w.klen_c; h.cstride = (int64_t)rows * cols;
        to.push_back(h);
        if (split) add_slices(sum, wsp + w.part, rows, 0, 0, cols, w.ksplit_c, dw);
      };
      if (q.kind == DMT_TM_CROSS_LINEAR) {
        TmGroup g = group(du, wt, wt, q.w_cross[l], wt, B, wt, nullptr, wt, EPI_F32);
        cross_grad(g, t, l);
        dgrad.push_back(g);
        add_wgrad(wgrad, sums, du, wt, xl_of(t, l), wt, gr[t].dw_cross[l]);
        continue;
      }
      // low-rank, stage 1: dt = du U_l (rounded) and dU_l = du^T t_l; stage 2: dx_l = dt V_l + dx_{l+1}
      // and dV_l = dt^T x_l
      const int r = q.feat_out;
      dgrad2.push_back(group(du, wt, wt, q.w_cross[2 * l + 1], r, B, r, wsp + w.dtq, r, EPI_BIAS));
      TmGroup g = group(wsp + w.dtq, r, r, q.w_cross[2 * l], wt, B, wt, nullptr, wt, EPI_F32);
      cross_grad(g, t, l);
      dgrad.push_back(g);
      add_wgrad(wgrad, sums, du, wt, wsp + w.tl[l], r, gr[t].dw_cross[2 * l + 1]);
      add_wgrad(wgrad2, sums2, wsp + w.dtq, r, xl_of(t, l), wt, gr[t].dw_cross[2 * l]);
    }
    // (the column sums and a split weight gradient's slices are added up before the buffers they lie
    // in are written again)
    launch_groups<DT, OP_COL, OP_COL>(p, wgrad, s, false, kid);
    ok &= launch_items(p, sums, tmb_sum_slices, s);
    launch_groups<DT, OP_ROW, OP_COL>(p, dgrad2, s, false, kid);
    launch_groups<DT, OP_ROW, OP_COL>(p, dgrad, s, false, kid);
    launch_groups<DT, OP_COL, OP_COL>(p, wgrad2, s, false, kid);
    ok &= launch_items(p, sums2, tmb_sum_slices, s);
  }
  if (!ok) return DMT_ENOTSUP;
  return hipGetLastError() == hipSuccess ? DMT_OK : DMT_EHIP;
}

// Float32 towers: every operand is read where it lies (dmt_tm_f32.h), so a stage is one launch: the
// projections' data, weight and bias gradients of all towers, then, layer by layer, a cross
// tower's elementwise step and its contractions.
dmt_status run_tm_bwd_f32(const dmt_plan* p, const dmt_tm_params* tp, const std::vector<TowerBwdWs>& ws,
                          const float* x_all, const float* y_all, int64_t B, const float* dy_all,
                          float* dx_all, const dmt_tm_grads* gr, const char* keptp, char* wsp,
                          hipStream_t s) {
  std::vector<TmKept> kept;
  if (keptp) plan_tm_kept(p, tp, B, 4, &kept);
  auto x_of = [&](int t) { return x_all + B * p->width_prefix[t]; };
  auto dx_of = [&](int t) { return dx_all + B * p->width_prefix[t]; };
  auto at = [&](size_t off) { return (float*)(wsp + off); };
  auto xl_of = [&](int t, int l) -> const float* {
    if (l == 0) return x_of(t);
    return keptp ? (const float*)(keptp + kept[t].x[l - 1]) : at(ws[t].xl[l - 1]);
  };
  auto u_of = [&](int t, int l) -> const float* {
    return keptp ? (const float*)(keptp + kept[t].u[l]) : at(ws[t].u[l]);
  };
  auto z_of = [&](int t) -> const float* {
    return keptp && kept[t].has_z ? (const float*)(keptp + kept[t].z) : at(ws[t].p);
  };
  bool ok = true;
  int max_layers = 0;

  // ---- what the forward did not keep: dot terms, cross layers (low-rank: t_l in any case)
  std::vector<TmAuxItem> dots_mfma, dots_simple;
  std::vector<int64_t> nb_mfma, nb_simple;
  for (int32_t t = 0; t < p->T; ++t) {
    if (is_cross(tp[t])) max_layers = std::max(max_layers, tp[t].num_cross_layers);
    if (tp[t].kind != DMT_TM_DOT_LINEAR || ws[t].np_pad == 0 || (keptp && kept[t].has_z)) continue;
    TmAuxItem it{};
    it.nf = p->tower_ntab[t]; it.n = p->tower_uniform_dim[t]; it.np = ws[t].np; it.np_pad = ws[t].np_pad;
    it.src = x_of(t);
    it.dst = at(ws[t].p);
    if (dots_mfma_ok(it.nf, it.n)) {
      dots_mfma.push_back(it);
      nb_mfma.push_back(dots_mfma_blocks(B, it.nf));
    } else {
      dots_simple.push_back(it);
      nb_simple.push_back((B * it.np_pad + kBlock - 1) / kBlock);
    }
  }
  launch_aux<DMT_F32>(p, B, dots_mfma, nb_mfma, 0, s);
  launch_aux<DMT_F32>(p, B, dots_simple, nb_simple, 1, s);
  std::vector<TmF32Group> groups, groups2;
  auto group = [&](const float* A, int lda, int K, const float* W, int ldw, int M, int N, float* C, int ldc,
                   int epi) {
    TmF32Group g{};
    g.A1 = A; g.lda1 = lda; g.K1 = K; g.W1 = W; g.ldw1 = ldw;
    g.M = M; g.N = N; g.C = C; g.ldc = ldc; g.epi = epi;
    return g;
  };
  for (int l = 0; l < max_layers; ++l) {
    for (int32_t t = 0; t < p->T; ++t) {
      const dmt_tm_params& q = tp[t];
      if (!is_cross(q) || l >= q.num_cross_layers) continue;
      const int wt = p->tower_width[t], r = q.feat_out;
      const bool low = q.kind == DMT_TM_CROSS_LOWRANK_LINEAR;
      const float* xl = xl_of(t, l);
      if (low)
        groups.push_back(group(xl, wt, wt, (const float*)q.w_cross[2 * l], wt, (int)B, r, at(ws[t].tl[l]), r, EPI_BIAS));
      if (keptp) continue;
      TmF32Group g = low ? group(at(ws[t].tl[l]), r, r, (const float*)q.w_cross[2 * l + 1], r, (int)B, wt,
                                 at(ws[t].xl[l]), wt, EPI_CROSS)
                         : group(xl, wt, wt, (const float*)q.w_cross[l], wt, (int)B, wt, at(ws[t].xl[l]), wt,
                                 EPI_CROSS);
      g.bias = (const float*)q.b_cross[l];
      g.X0 = x_of(t); g.ldx = wt; g.XL = xl; g.ldxl = wt;
      g.U = at(ws[t].u[l]);
      groups2.push_back(g);
    }
    launch_f32(p, groups, s, DMT_K_TM_BWD_GEMM);
    launch_f32(p, groups2, s, DMT_K_TM_BWD_GEMM);
  }

  // ---- projections
  TmbBatch dots, prep;
  int64_t out_prefix = 0;
  for (int32_t t = 0; t < p->T; ++t) {
    const dmt_tm_params& q = tp[t];
    const TowerBwdWs& w = ws[t];
    const int wt = p->tower_width[t], nf = p->tower_ntab[t], ldy = q.out_dim;
    const float* dy = dy_all + B * out_prefix;
    const float* mask = q.kind == DMT_TM_LINEAR_RELU ? y_all + B * out_prefix : nullptr;
    out_prefix += q.out_dim;
    const float* W = (const float*)q.w_proj;
    const float* z = is_cross(q) ? xl_of(t, q.num_cross_layers) : x_of(t);
    const bool dot = q.kind == DMT_TM_DOT_LINEAR, dlrm = q.kind == DMT_TM_DLRM;
    const int F = dlrm ? q.feat_out : 0, O = ldy - nf * F, np = w.np, kin = np + wt;
    auto dgrad = [&](const float* Wk, int N, float* C, int ldc) {
      TmF32Group g = group(dy, ldy, O, Wk, kin, (int)B, N, C, ldc, EPI_F32);
      g.wcol = 1; g.mask = mask;
      groups.push_back(g);
    };
    auto wgrad = [&](const float* zk, int ldz, int N, float* C, float* db) {
      TmF32Group g = group(dy, ldy, (int)B, zk, ldz, O, N, C, kin, EPI_F32);
      g.acol = 1; g.wcol = 1; g.mask = mask; g.db = db;
      groups.push_back(g);
    };
    wgrad(z, wt, wt, gr[t].dw_proj + np, gr[t].db_proj);
    if (dot) {
      if (np > 0) {
        wgrad(z_of(t), w.np_pad, np, gr[t].dw_proj, nullptr);
        dgrad(W, np, at(w.dZ), w.kin);
      }
      dgrad(W + np, wt, at(w.dZ) + w.np_pad, w.kin);
      TmbItem it{};
      it.a = x_of(t); it.b = at(w.dZ); it.o0 = dx_of(t); it.n0 = B;
      it.i0 = nf; it.i1 = p->tower_uniform_dim[t]; it.i2 = w.np_pad; it.i3 = w.kin;
      dots.add(it, (B * wt + kBlock - 1) / kBlock);
    } else if (dlrm) {
      // feature f's slice of the pooled block: [dy flat | dy of feature f] . [W rows | shared W]
      const int n = p->tower_uniform_dim[t];
      const float* Wf = (const float*)q.w_cross[0];
      for (int f = 0; f < nf; ++f) {
        TmF32Group g = group(dy + O + f * F, ldy, F, Wf, n, (int)B, n, dx_of(t) + f * n, wt, EPI_F32);
        g.A0 = dy; g.lda0 = ldy; g.K0 = O; g.W0 = W + f * n; g.ldw0 = wt; g.wcol = 1;
        groups.push_back(g);
      }
      // the shared layer's weights: a sum over rows (sample, feature)
      TmF32Group g = group(dy + O, ldy, (int)(B * nf), x_of(t), n, F, n, gr[t].dw_cross[0], n, EPI_F32);
      g.acol = 1; g.wcol = 1; g.adiv = nf; g.lda2 = F; g.db = gr[t].db_cross[0];
      groups.push_back(g);
    } else {
      dgrad(W, wt, is_cross(q) ? at(w.dxn) : dx_of(t), wt);
    }
  }
  launch_f32(p, groups, s, DMT_K_TM_BWD_GEMM);
  ok &= launch_items(p, dots, tmb_dot_bwd<DMT_F32>, s);

  // ---- cross layers, last to first
  for (int l = max_layers - 1; l >= 0; --l) {
    for (int32_t t = 0; t < p->T; ++t) {
      const dmt_tm_params& q = tp[t];
      if (!is_cross(q) || l >= q.num_cross_layers) continue;
      const TowerBwdWs& w = ws[t];
      const int wt = p->tower_width[t];
      TmbItem it{};
      it.a = at(w.dxn); it.b = x_of(t); it.c = u_of(t, l); it.o0 = at(w.du[0]); it.o1 = dx_of(t);
      it.n0 = B * wt; it.i0 = l == q.num_cross_layers - 1; it.i1 = l == 0;
      it.nbx = (int32_t)ew_blocks(it.n0);
      prep.add(it, it.nbx);
      float* dx_l = l == 0 ? dx_of(t) : at(w.dxn);
      const float* du = at(w.du[0]);
      // dx_l += dv . V with V stored [K][wt]; dV = dv^T x_l
      auto pair = [&](std::vector<TmF32Group>& gs, const float* dv, int K, const void* V, float* dV, float* db) {
        TmF32Group g = group(dv, K, K, (const float*)V, wt, (int)B, wt, dx_l, wt, EPI_F32_ADD);
        g.wcol = 1;
        gs.push_back(g);
        g = group(dv, K, (int)B, xl_of(t, l), wt, K, wt, dV, wt, EPI_F32);
        g.acol = 1; g.wcol = 1; g.db = db;
        gs.push_back(g);
      };
      if (q.kind == DMT_TM_CROSS_LINEAR) {
        pair(groups, du, wt, q.w_cross[l], gr[t].dw_cross[l], gr[t].db_cross[l]);
        continue;
      }
      // low-rank: dt = du U_l and dU_l = du^T t_l, then the same with dt and V_l
      const int r = q.feat_out;
      TmF32Group g = group(du, wt, wt, (const float*)q.w_cross[2 * l + 1], r, (int)B, r, at(w.dtf), r, EPI_F32);
      g.wcol = 1;
      groups.push_back(g);
      g = group(du, wt, (int)B, at(w.tl[l]), r, wt, r, gr[t].dw_cross[2 * l + 1], r, EPI_F32);
      g.acol = 1; g.wcol = 1; g.db = gr[t].db_cross[l];
      groups.push_back(g);
      pair(groups2, at(w.dtf), r, q.w_cross[2 * l], gr[t].dw_cross[2 * l], nullptr);
    }
    ok &= launch_items(p, prep, tmb_cross_prep, s);
    launch_f32(p, groups, s, DMT_K_TM_BWD_GEMM);
    launch_f32(p, groups2, s, DMT_K_TM_BWD_GEMM);
  }
  if (!ok) return DMT_ENOTSUP;
  return hipGetLastError() == hipSuccess ? DMT_OK : DMT_EHIP;
}

}  // namespace

extern "C" size_t dmt_tm_bwd_workspace_bytes(const dmt_plan* plan, const dmt_tm_params* per_tower,
                                             int64_t B) {
  if (!plan || !per_tower || B <= 0) return 0;
  // enough for every dtype: the 16-bit layouts have smaller operands but may split K
  return dmt_guard_size([&]() -> size_t {
    std::vector<TowerBwdWs> ws;
    size_t b4 = 0, b2 = 0;
    if (plan_tm_bwd(plan, per_tower, B, 4, false, &ws, &b4) != DMT_OK) return 0;
    if (plan_tm_bwd(plan, per_tower, B, 2, false, &ws, &b2) != DMT_OK) b2 = 0;   // e.g. a rank no multiple of 8
    return std::max(b4, b2);
  });
}

extern "C" dmt_status dmt_tower_module_bwd(const dmt_plan* plan, const dmt_tm_params* per_tower,
                                           const void* pooled, const void* tm_out, int64_t B,
                                           const float* grad_tm_out, int32_t dtype_code,
                                           float* grad_pooled, const dmt_tm_grads* grads,
                                           const void* kept, size_t kept_bytes, void* workspace,
                                           size_t workspace_bytes, void* stream) {
  if (!plan || !per_tower || !pooled || !grad_tm_out || !grad_pooled || !grads) return DMT_EINVAL;
  if (B <= 0 || B > plan->max_batch || B >= (1LL << 31) - 128) return DMT_EINVAL;
  if (dtype_code != DMT_F32 && dtype_code != DMT_F16 && dtype_code != DMT_BF16) return DMT_EINVAL;
  const dmt_dtype dtype = (dmt_dtype)dtype_code;
  if (((uintptr_t)pooled & 15) || ((uintptr_t)tm_out & 15) || ((uintptr_t)grad_pooled & 15) ||
      ((uintptr_t)grad_tm_out & 3))
    return DMT_EINVAL;
  const int eb = dmt_elt_bytes(dtype);
  for (int32_t t = 0; t < plan->T; ++t) {
    if (plan->tower_width[t] % 8 != 0 && dtype != DMT_F32) return DMT_ENOTSUP;
    const dmt_tm_params& q = per_tower[t];
    if (q.kind == DMT_TM_LINEAR_RELU && !tm_out) return DMT_EINVAL;
    if (!grads[t].dw_proj || !grads[t].db_proj) return DMT_EINVAL;
    if (q.kind == DMT_TM_CROSS_LINEAR)
      for (int l = 0; l < q.num_cross_layers && l < DMT_MAX_CROSS_LAYERS; ++l)
        if (!grads[t].dw_cross[l] || !grads[t].db_cross[l]) return DMT_EINVAL;
    if (q.kind == DMT_TM_DLRM && (!grads[t].dw_cross[0] || !grads[t].db_cross[0])) return DMT_EINVAL;
    if (q.kind == DMT_TM_CROSS_LOWRANK_LINEAR)
      for (int l = 0; l < q.num_cross_layers && 2 * l + 1 < DMT_MAX_CROSS_LAYERS; ++l)
        if (!grads[t].dw_cross[2 * l] || !grads[t].dw_cross[2 * l + 1] || !grads[t].db_cross[l])
          return DMT_EINVAL;
  }
  return dmt_guard([&]() -> dmt_status {
  std::vector<TowerBwdWs> ws;
  size_t bytes = 0;
  const char* keptp = nullptr;
  if (kept) {
    std::vector<TmKept> k;
    const size_t need = plan_tm_kept(plan, per_tower, B, eb, &k);
    if ((uintptr_t)kept & 255) return DMT_EINVAL;
    if (kept_bytes < need) return DMT_ENOMEM;
    if (need > 0) keptp = (const char*)kept;
  }
  dmt_status st = plan_tm_bwd(plan, per_tower, B, eb, keptp != nullptr, &ws, &bytes);
  if (st != DMT_OK) return st;
  if (!workspace || ((uintptr_t)workspace & 255)) return DMT_EINVAL;
  if (workspace_bytes < bytes) return DMT_ENOMEM;
  hipStream_t s = (hipStream_t)stream;
  char* wsp = (char*)workspace;
  switch (dtype) {
    case DMT_F32:
      return run_tm_bwd_f32(plan, per_tower, ws, (const float*)pooled, (const float*)tm_out, B, grad_tm_out,
                            grad_pooled, grads, keptp, wsp, s);
    case DMT_F16:
      return run_tm_bwd<DMT_F16>(plan, per_tower, ws, pooled, tm_out, B, grad_tm_out, grad_pooled,
                                 grads, keptp, wsp, s);
    default:
      return run_tm_bwd<DMT_BF16>(plan, per_tower, ws, pooled, tm_out, B, grad_tm_out, grad_pooled,
                                  grads, keptp, wsp, s);
  }
  });
}
