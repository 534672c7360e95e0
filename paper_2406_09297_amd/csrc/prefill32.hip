// Prefill attention with 32 query rows a block (gfx950, wave64,
// v_mfma_f32_32x32x16_bf16), for the calls where it is the faster form; rows,
// units and results as in prefill.hip.
//
//   prefill_wide_kernel   head dim 128, large grids: 256 rows a workgroup
//   prefill_split_kernel  small grids: 32 rows a workgroup, its waves share
//                         out the tokens
//
//   S^T[32 tok][32 rows] = K Q^T   (D/16 products per tile)
//   O^T[D][32 rows] += V^T P^T     (D/32 x 2 products per tile)
// The key plane's chunk order gives lane l (row r = l % 32, half = l / 32) of
// the score product the tokens 16 a + 8 half + e, e = 0 .. 7, a = 0, 1: the
// k-slots it supplies to the value product, so nothing moves across lanes.
#include <hip/hip_ext.h>
#include <hip/hip_runtime.h>
#include <stdint.h>

#include "kernels.h"
#include "prefill.h"
#include "tile.h"

namespace mlkv {

namespace {

typedef float f32x16 __attribute__((ext_vector_type(16)));

__device__ __forceinline__ f32x16 mfma32(bf16x8 a, bf16x8 b, f32x16 c) {
  return __builtin_amdgcn_mfma_f32_32x32x16_bf16(a, b, c, 0, 0, 0);
}

__device__ __forceinline__ float max16(const f32x16& x) {
  const float a = fmaxf(fmaxf(fmaxf(x[0], x[1]), fmaxf(x[2], x[3])),
                        fmaxf(fmaxf(x[4], x[5]), fmaxf(x[6], x[7])));
  const float b = fmaxf(fmaxf(fmaxf(x[8], x[9]), fmaxf(x[10], x[11])),
                        fmaxf(fmaxf(x[12], x[13]), fmaxf(x[14], x[15])));
  return fmaxf(a, b);
}

// c + the eight weights' sum, from their bf16 values (the same rounded
// weights the value product takes).
__device__ __forceinline__ float sum8(bf16x8 w, float c) {
  typedef __bf16 bf16x2 __attribute__((ext_vector_type(2)));
  const bf16x2 one = {static_cast<__bf16>(1.f), static_cast<__bf16>(1.f)};
#pragma unroll
  for (int i = 0; i < 4; ++i)
    c = __builtin_amdgcn_fdot2_f32_bf16(bf16x2{w[2 * i], w[2 * i + 1]}, one, c, false);
  return c;
}

// Key/value tiles staged in LDS by direct global-to-LDS loads
// (global_load_lds_dwordx4: lane l of a wave writes its 16 bytes at the
// wave-uniform LDS address + 16 l), double-buffered, two tiles of 32 tokens a
// stage, shared by the workgroup's waves.  Key chunks keep the plane's order,
// in which a wave's operand reads are contiguous by sixteen lanes; the value
// chunk of channel c and 8-token part p sits at slot 4 c + (p ^ vswz(c)), so
// that the lanes reading channels c .. c + 15 at one part hit distinct banks.
__device__ __forceinline__ int vswz(int c) { return (c >> 2) & 3; }

// Pair p holds the tiles 2 p and 2 p + 1; it sits in buffer p & 1 of its plane.
template <int D, int NW>
struct PrefillRing {
  alignas(16) uint16_t k[2][2][kTile * D];
  alignas(16) uint16_t v[2][2][kTile * D];

  static constexpr int P = D / 16;  // 1 KB pieces per tile
  static constexpr int N = 2 * P;   // pieces of a pair, NW at a time

  // Requests a pair of tiles of a plane (indexes past the plane's last tile
  // read that one: their positions are masked).  off: this lane's byte offset
  // inside a 1 KB piece.
  __device__ __forceinline__ static void issue(uint16_t (&dst)[2][kTile * D], const uint16_t* base,
                                               int pair, int last_tile, unsigned off) {
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
#pragma unroll
    for (int u = 0; u < (N + NW - 1) / NW; ++u) {
      const int piece = u * NW + wave;
      if (N % NW != 0 && piece >= N) break;
      const int tt = piece / P, n = piece % P;
      const size_t at =
          static_cast<size_t>(min(2 * pair + tt, last_tile)) * (kTile * D * 2) + n * 1024;
      load_lds16(reinterpret_cast<const char*>(base) + at, off, &dst[tt][n * 512]);
    }
  }
  __device__ __forceinline__ void issue_k(const uint16_t* kbase, int pair, int last_tile) {
    issue(k[pair & 1], kbase, pair, last_tile, (threadIdx.x & 63) * 16);
  }
  // The value chunk of channel 16 n + lane / 4 (n the piece) goes to its swizzled part.
  __device__ __forceinline__ void issue_v(const uint16_t* vbase, int pair, int last_tile) {
    const unsigned lane = threadIdx.x & 63;
    issue(v[pair & 1], vbase, pair, last_tile,
          (lane >> 2) * 64 + (((lane & 3) ^ vswz(lane >> 2)) * 16));
  }

  // After its loads of value pair `pair` have landed: this wave's pieces with
  // positions at or past L (which may hold anything) become zero.
  __device__ __forceinline__ void clear_tail(int pair, int L) {
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    for (int piece = wave; piece < N; piece += NW) {
      const int tt = piece / P, q = (piece % P) * 64 + lane;
      const int part = (q & 3) ^ vswz(q >> 2);
      const int first = (2 * pair + tt) * kTile + part * 8;
      if (first + 8 > L) {
        u16x8* slot = reinterpret_cast<u16x8*>(&v[pair & 1][tt][q * 8]);
        u16x8 x = *slot;
#pragma unroll
        for (int e = 0; e < 8; ++e)
          if (first + e >= L) x[e] = 0;
        *slot = x;
      }
    }
  }
};

template <int D>
struct PrefillState {
  float m, den;        // reference (log2 units), this lane's part of the denominator
  f32x16 acc[D / 32];
};

// A row's weights against its reference, rounded to bf16, and their sum.
__device__ __forceinline__ float weights16(const f32x16& x, float scale_log2, float neg_m,
                                           bf16x8 (&p)[2]) {
  float sum[2];
#pragma unroll
  for (int a = 0; a < 2; ++a) {
    u16x8 bits;
#pragma unroll
    for (int e = 0; e < 8; ++e)
      bits[e] = f32_to_bf16_bits(
          fast_exp2(fmaf(x[8 * (e >> 2) + 4 * a + (e & 3)], scale_log2, neg_m)));
    p[a] = as_bf16(bits);
    sum[a] = sum8(p[a], 0.f);
  }
  return sum[0] + sum[1];
}

// The weights are taken against the reference at hand; only their sum, which
// is needed anyway, is looked at.  Where it passes kSumBar (or is not a
// number) the row's maximum becomes its reference.
constexpr float kSumBar = 4096.f;

// A reference below every score (a row none of whose attended positions has
// been seen): weights against it overflow, which raises it.
constexpr float kNoReference = -3e38f;

// Positions past `left` (counted from the tile's start + 8 half) take no weight.
__device__ __forceinline__ void mask_scores(f32x16& x, int left) {
#pragma unroll
  for (int i = 0; i < 16; ++i)
    if (16 * ((i >> 2) & 1) + 4 * (i >> 3) + (i & 3) > left) x[i] = -INFINITY;
}

// Moves the references of the rows whose maximum exceeds theirs up to it, and
// forms the tile's weights and their sum again.
template <int D>
__device__ __forceinline__ float raise_reference(PrefillState<D>& st, const f32x16& x,
                                                 float scale_log2, bf16x8 (&p)[2]) {
  float cm = max16(x);
  cm = fmaxf(cm, __shfl_xor(cm, 32)) * scale_log2;
  const float m_new = fmaxf(cm, st.m);
  const float alpha = fast_exp2(st.m - m_new);
  st.m = m_new;
  st.den *= alpha;
#pragma unroll
  for (int cb = 0; cb < D / 32; ++cb) st.acc[cb] *= alpha;
  return weights16(x, scale_log2, -st.m, p);
}

// A row's query operands (zero for rows past the end).
template <int D>
__device__ __forceinline__ void load_queries(bf16x8 (&qf)[D / 16], const uint16_t* q, bool valid,
                                             int half) {
#pragma unroll
  for (int ks = 0; ks < D / 16; ++ks) {
    const u16x8 v = load16(q + half * 8 + ks * 16);
    const u16x8 zero = {0, 0, 0, 0, 0, 0, 0, 0};
    qf[ks] = as_bf16(valid ? v : zero);
  }
}

// Scores of a tile: k its keys in LDS.
template <int D>
__device__ __forceinline__ f32x16 scores(const uint16_t (&k)[kTile * D],
                                         const bf16x8 (&qf)[D / 16], int koff) {
  f32x16 x = {0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f};
#pragma unroll
  for (int ks = 0; ks < D / 16; ++ks)
    x = mfma32(as_bf16(*reinterpret_cast<const u16x8*>(&k[(koff + (ks >> 1) * 64 + (ks & 1) * 32) * 8])),
               qf[ks], x);
  return x;
}

// Step i of a wave: the weights of tile i (scores x_cur, formed in step i - 1)
// beside the scores of tile i + 1 (-> x_next) and the value product of tile
// i - 1 (weights p_prev): the matrix cores and the vector units work on
// different tiles, so neither waits for the other inside a step.
template <int D>
__device__ __forceinline__ void prefill_step_tile(PrefillState<D>& st, const uint16_t (&k_next)[kTile * D],
                                                  const uint16_t (&v_prev)[kTile * D],
                                                  const bf16x8 (&qf)[D / 16], f32x16& x_cur,
                                                  f32x16& x_next, const bf16x8 (&p_prev)[2],
                                                  bf16x8 (&p_cur)[2], bool masked, int left,
                                                  int row, int half, int koff, float scale_log2) {
  if (masked) mask_scores(x_cur, left);
  x_next = scores<D>(k_next, qf, koff);
  float sum = weights16(x_cur, scale_log2, -st.m, p_cur);
#pragma unroll
  for (int a = 0; a < 2; ++a)
#pragma unroll
    for (int cb = 0; cb < D / 32; ++cb) {
      const int ch = cb * 32 + row;
      const bf16x8 vf = as_bf16(*reinterpret_cast<const u16x8*>(
          &v_prev[(ch * 4 + ((2 * a + half) ^ vswz(ch))) * 8]));
      st.acc[cb] = mfma32(vf, p_prev[a], st.acc[cb]);
    }
  if (__ballot(!(sum < kSumBar))) sum = raise_reference<D>(st, x_cur, scale_log2, p_cur);
  st.den += sum;
}

// 256 rows a workgroup, so that a staged byte serves twice the rows it does in
// prefill.hip's 16-row form, where head dim 128 is bound by LDS reads.  One
// layer of 32 heads, 2 x 2048 tokens: 92 us in a call with its append against
// 99; one prompt of 4096: 154 against 171.  Where it is slower than the 64-row
// workgroups of prefill.hip stands at prefill_form; head dim 64 gains nothing
// (744 against 708 us per 12-layer prompt).
template <int D, int NW>
__global__ __launch_bounds__(NW * 64) __attribute__((amdgpu_waves_per_eu(2)))
void prefill_wide_kernel(PrefillParams p) {
  constexpr int WAVE_ROWS = 32;
  __shared__ PrefillRing<D, NW> rg;
  const int lane = threadIdx.x & 63;
  const int wave = threadIdx.x >> 6;
  const int row = lane & 31;
  const int half = lane >> 5;
  const int unit = blockIdx.x;
  const int b = unit / p.n_groups;
  const int r = unit - b * p.n_groups;
  const int R = p.layers * p.G;           // rows per token
  const int rows = p.T * R;
  const int blk = gridDim.y - 1 - blockIdx.y;
  const int wg_row0 = blk * NW * WAVE_ROWS;  // < rows: the grid has no empty workgroup
  const int row0 = wg_row0 + wave * WAVE_ROWS;
  const bool active = row0 < rows;  // a wave past the end still stages tiles and syncs
  const int c0 = max(p.ctx[b], 0);
  const int L = min(c0 + p.T, p.S);  // filled positions of the sequence
  // Tiles of the workgroup (its last row's limit) and of this wave.
  const int wg_last = min(wg_row0 + NW * WAVE_ROWS - 1, rows - 1);
  const int n_wg = min(c0 + wg_last / R, p.S - 1) / kTile + 1;
  const int last_row = min(row0 + WAVE_ROWS - 1, rows - 1);
  const int lim_max = min(c0 + last_row / R, p.S - 1);
  const int lim_min = min(c0 + min(row0, rows - 1) / R, p.S - 1);
  const int n = active ? __builtin_amdgcn_readfirstlane(lim_max / kTile + 1) : 0;
  const int first_masked = __builtin_amdgcn_readfirstlane((lim_min + 1) / kTile);  // tiles before it lie under every limit
  const int last_tile = p.S / kTile - 1;

  const int kv = p.kv_begin + r;
  const int group = r / p.kv_per_layer;  // of layers
  const size_t seq = static_cast<size_t>(kv) * p.B + b;
  const uint16_t* kbase = p.k + seq * p.S * D;
  const uint16_t* vbase = p.v + seq * p.S * D;
  rg.issue_k(kbase, 0, last_tile);
  rg.issue_k(kbase, 1, last_tile);
  rg.issue_v(vbase, 0, last_tile);

  const RowPlace at = row_place(p, row0 + row, rows, b, group, r, D);
  const int left0 = min(c0 + at.tok, p.S - 1) - 8 * half;
  bf16x8 qf[D / 16];
  load_queries<D>(qf, p.q + at.offset, at.valid, half);
  PrefillState<D> st;
#pragma unroll
  for (int cb = 0; cb < D / 32; ++cb)
#pragma unroll
    for (int i = 0; i < 16; ++i) st.acc[cb][i] = 0.f;
  const int koff = (row >> 4) * (D / 32) * 64 + half * 16 + (row & 15);
  f32x16 xa, xb;
  bf16x8 pa[2], pb[2];

  // Tile 0: its scores set each row's reference (every row attends position 0).
  wait_loads();
  if (2 * kTile > L) rg.clear_tail(0, L);
  __syncthreads();
  xa = scores<D>(rg.k[0][0], qf, koff);
  if (first_masked == 0) mask_scores(xa, left0);
  xb = scores<D>(rg.k[0][1], qf, koff);
  {
    float cm = max16(xa);
    st.m = fmaxf(cm, __shfl_xor(cm, 32)) * p.scale_log2;
    st.den = weights16(xa, p.scale_log2, -st.m, pa);
  }
  // Steps 2 s + 1 and 2 s + 2 use the key pair s + 1 and the value pair s.  At
  // the barrier this wave's direct loads have landed, so every wave's part of
  // both is there, and every wave is done with key pair s and value pair
  // s - 1, whose buffers take the next pairs.  A wave's last step is n: it
  // has the value product of tile n - 1 (its own tile is masked entirely).
  for (int s = 0; 2 * s + 1 <= n_wg; ++s) {
    if (s > 0) {
      wait_loads();
      if ((2 * s + 2) * kTile > L) rg.clear_tail(s, L);
    }
    __syncthreads();
    if (2 * s + 3 <= n_wg) {
      rg.issue_k(kbase, s + 2, last_tile);
      rg.issue_v(vbase, s + 1, last_tile);
    }
    int i = 2 * s + 1;
    if (i > n) continue;
    prefill_step_tile<D>(st, rg.k[(s + 1) & 1][0], rg.v[s & 1][0], qf, xb, xa, pa, pb,
                         i >= first_masked, left0 - i * kTile, row, half, koff, p.scale_log2);
    if (++i > n) continue;
    prefill_step_tile<D>(st, rg.k[(s + 1) & 1][1], rg.v[s & 1][1], qf, xa, xb, pb, pa,
                         i >= first_masked, left0 - i * kTile, row, half, koff, p.scale_log2);
  }

  // Lane (row, half) holds channels 32 cb + 8 g + 4 half .. +3 of its row.
  const float inv = 1.f / (st.den + __shfl_xor(st.den, 32));
  if (!at.valid) return;
#pragma unroll
  for (int cb = 0; cb < D / 32; ++cb)
#pragma unroll
    for (int g = 0; g < 4; ++g)
      store4(p, at.offset + cb * 32 + 8 * g + 4 * half,
             f32x4{st.acc[cb][4 * g], st.acc[cb][4 * g + 1], st.acc[cb][4 * g + 2],
                   st.acc[cb][4 * g + 3]} * inv);
}

// ---------------------------------------------------------------------------
// For calls whose row blocks leave the device idle (few new tokens, long
// contexts; prefill_form): a workgroup of kSplitWaves waves takes 32 rows, wave
// w the tiles w, w + kSplitWaves, ..., straight from the planes to registers,
// and the waves' partial results are merged through LDS in wave order.  Every
// workgroup reads its whole context, and what a compute unit's load path
// delivers bounds it: 71 GB/s each in the first call below, vector issue 43 %
// of the busy cycles, matrix cores 21 %.  One layer, 257 new tokens on two
// contexts of 14000 (12 heads of 64 channels): 46 us against 217; 400 on 8000
// (32 heads of 128): 97 against 131.
// ---------------------------------------------------------------------------
constexpr int kSplitWaves = 8;

template <int D>
struct SplitShared {
  float acc[kSplitWaves][32][D + 4];
  float m[kSplitWaves][32], den[kSplitWaves][32];
  bf16x8 q[D / 16][64];  // the rows' query operands, read again for each tile
};

template <int D>
__device__ __forceinline__ void load_keys(u16x8 (&k)[D / 16], const uint16_t* kbase, int tile,
                                          int koff) {
  const uint16_t* src = kbase + static_cast<size_t>(tile) * (kTile * D) + koff * 8;
#pragma unroll
  for (int ks = 0; ks < D / 16; ++ks) k[ks] = load16(src + ((ks >> 1) * 64 + (ks & 1) * 32) * 8);
}

// Value operands of a tile.
template <int D>
__device__ __forceinline__ void load_values(u16x8 (&v)[D / 16], const uint16_t* vbase, int tile,
                                            int row, int half) {
  const uint16_t* src = vbase + static_cast<size_t>(tile) * (kTile * D) + row * kTile + half * 8;
#pragma unroll
  for (int u = 0; u < D / 16; ++u)
    v[u] = load16(src + (u % (D / 32)) * 32 * kTile + (u / (D / 32)) * 16);
}

template <int D>
__global__ __launch_bounds__(kSplitWaves * 64) __attribute__((amdgpu_waves_per_eu(2)))
void prefill_split_kernel(PrefillParams p) {
  __shared__ SplitShared<D> sm;
  const int lane = threadIdx.x & 63;
  const int wave = threadIdx.x >> 6;
  const int row = lane & 31;
  const int half = lane >> 5;
  const int unit = blockIdx.x;
  const int b = unit / p.n_groups;
  const int r = unit - b * p.n_groups;
  const int R = p.layers * p.G;  // rows per token
  const int rows = p.T * R;
  const int row0 = (gridDim.y - 1 - blockIdx.y) * 32;  // < rows
  const int c0 = max(p.ctx[b], 0);
  const int L = min(c0 + p.T, p.S);  // filled positions of the sequence
  const int n = min(c0 + min(row0 + 31, rows - 1) / R, p.S - 1) / kTile + 1;  // tiles
  const int first_masked = (min(c0 + row0 / R, p.S - 1) + 1) / kTile;
  const int kv = p.kv_begin + r;
  const int group = r / p.kv_per_layer;
  const size_t seq = static_cast<size_t>(kv) * p.B + b;
  const uint16_t* kbase = p.k + seq * p.S * D;
  const uint16_t* vbase = p.v + seq * p.S * D;
  const int koff = (row >> 4) * (D / 32) * 64 + half * 16 + (row & 15);
  u16x8 kc[D / 16], kn[D / 16], vc[D / 16], vn[D / 16];
  int it = wave;
  if (it < n) {
    load_keys<D>(kc, kbase, it, koff);
    load_values<D>(vc, vbase, it, row, half);
  }

  const RowPlace at = row_place(p, row0 + row, rows, b, group, r, D);
  const int left0 = min(c0 + at.tok, p.S - 1) - 8 * half;
  {
    bf16x8 qf[D / 16];
    load_queries<D>(qf, p.q + at.offset, at.valid, half);
    if (wave == 0) {
#pragma unroll
      for (int ks = 0; ks < D / 16; ++ks) sm.q[ks][lane] = qf[ks];
    }
    __syncthreads();
  }
  PrefillState<D> st;
  st.m = kNoReference;
  st.den = 0.f;
#pragma unroll
  for (int cb = 0; cb < D / 32; ++cb)
#pragma unroll
    for (int i = 0; i < 16; ++i) st.acc[cb][i] = 0.f;

  for (; it < n; it += kSplitWaves) {
    if (it + kSplitWaves < n) {
      load_keys<D>(kn, kbase, it + kSplitWaves, koff);
      load_values<D>(vn, vbase, it + kSplitWaves, row, half);
    }
    f32x16 x = {0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int ks = 0; ks < D / 16; ++ks) x = mfma32(as_bf16(kc[ks]), sm.q[ks][lane], x);
    if (it >= first_masked) mask_scores(x, left0 - it * kTile);
    bf16x8 pw[2];
    float sum = weights16(x, p.scale_log2, -st.m, pw);
    if (__ballot(!(sum < kSumBar))) sum = raise_reference<D>(st, x, p.scale_log2, pw);
    st.den += sum;
    if ((it + 1) * kTile > L) {
#pragma unroll
      for (int u = 0; u < D / 16; ++u)
#pragma unroll
        for (int e = 0; e < 8; ++e)
          if (it * kTile + 16 * (u / (D / 32)) + 8 * half + e >= L) vc[u][e] = 0;
    }
#pragma unroll
    for (int u = 0; u < D / 16; ++u)
      st.acc[u % (D / 32)] = mfma32(as_bf16(vc[u]), pw[u / (D / 32)], st.acc[u % (D / 32)]);
#pragma unroll
    for (int ks = 0; ks < D / 16; ++ks) {
      kc[ks] = kn[ks];
      vc[ks] = vn[ks];
    }
  }

  const float den = st.den + __shfl_xor(st.den, 32);
  if (half == 0) {
    sm.m[wave][row] = st.m;
    sm.den[wave][row] = den;
  }
#pragma unroll
  for (int cb = 0; cb < D / 32; ++cb)
#pragma unroll
    for (int g = 0; g < 4; ++g)
      *reinterpret_cast<f32x4*>(&sm.acc[wave][row][cb * 32 + 8 * g + 4 * half]) =
          f32x4{st.acc[cb][4 * g], st.acc[cb][4 * g + 1], st.acc[cb][4 * g + 2],
                st.acc[cb][4 * g + 3]};
  __syncthreads();
  constexpr int D4 = D / 4;
  for (int idx = threadIdx.x; idx < 32 * D4; idx += kSplitWaves * 64) {
    const int rr = idx / D4, d = (idx - rr * D4) * 4;
    const RowPlace to = row_place(p, row0 + rr, rows, b, group, r, D);
    if (!to.valid) continue;
    float M = sm.m[0][rr];
#pragma unroll
    for (int w = 1; w < kSplitWaves; ++w) M = fmaxf(M, sm.m[w][rr]);
    float total = 0.f;
    f32x4 o = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int w = 0; w < kSplitWaves; ++w) {
      const float f = fast_exp2(sm.m[w][rr] - M);
      total += f * sm.den[w][rr];
      o += f * *reinterpret_cast<const f32x4*>(&sm.acc[w][rr][d]);
    }
    store4(p, to.offset + d, o * (1.f / total));
  }
}

template <typename Kernel>
hipError_t launch(Kernel kernel, const PrefillParams& p, int rows_per_wg, int threads,
                  hipStream_t stream, hipEvent_t start, hipEvent_t stop) {
  const int blocks = (p.T * p.layers * p.G + rows_per_wg - 1) / rows_per_wg;
  const dim3 grid(p.B * p.n_groups, blocks);
  if (start || stop)
    hipExtLaunchKernelGGL(kernel, grid, dim3(threads), 0, stream, start, stop, 0, p);
  else
    hipLaunchKernelGGL(kernel, grid, dim3(threads), 0, stream, p);
  return hipGetLastError();
}

}  // namespace

hipError_t launch_prefill_wide(const PrefillParams& p, hipStream_t stream, hipEvent_t start,
                               hipEvent_t stop) {
  constexpr int NW = kPrefillWideRows / 32;
  return launch(prefill_wide_kernel<128, NW>, p, kPrefillWideRows, NW * 64, stream, start, stop);
}

hipError_t launch_prefill_split(const PrefillParams& p, int head_dim, hipStream_t stream,
                                hipEvent_t start, hipEvent_t stop) {
  auto kernel = head_dim == 64 ? prefill_split_kernel<64> : prefill_split_kernel<128>;
  return launch(kernel, p, kPrefillSplitRows, kSplitWaves * 64, stream, start, stop);
}

}  // namespace mlkv
