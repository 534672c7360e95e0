// Decode attention of a whole step in one launch, for CDNA4 (gfx950, wave64,
// MFMA).
//
// mlkv_decode_step is given every layer's queries at once, so nothing orders
// its layers but the owners' appends, and the layers of a group read the same
// KV heads (Section 3, Eqs. 13-17).  Here the query rows of every layer of
// the group that reads a KV head (layers-per-group x query heads per KV head)
// are the MFMA columns of one pass over that head's rows: a cached byte is
// read once per step instead of once per layer, and the step is one launch.
// The tile arithmetic is that of the one-layer kernel (tile.h).
//
// A unit is one (sequence, KV head).  Its rows are cut into `chunks` of at
// most 16*NB rows, its tiles into at most `runs` runs of equal length, taken
// from the sequence's own length; a workgroup is one run of one chunk.  The
// last run of a unit to finish merges its runs.
//
// What bounds it: HBM for large steps (a 7B-like step of 17.2 GB in 2.92 ms,
// 5.9 TB/s, where a plain streaming read reaches 6.0; one launch per layer
// took 11.6 ms), the first and last round trips for small ones (one sequence
// of 128 tokens 8.9 us against 46.8 us, 5.9 of them on the device).  128 ragged
// sequences of 12-layer MLKV-4: 43.5 us against 145 us; eight of 32768 tokens:
// 55 against 211 us.
// A third tile in flight per wave spills (184 us) and is no faster where it
// fits; eight waves on a unit shorten the stream of a lone workgroup but hold
// fewer workgroups per compute unit, so the host gives eight waves to grids of
// at most one workgroup per compute unit and to several rounds of long sequences.
#include <hip/hip_ext.h>
#include <hip/hip_runtime.h>
#include <stdint.h>

#include "decode.h"
#include "kernels.h"
#include "tile.h"

namespace mlkv {

namespace {

// One 32-token tile against the wave's NB blocks of 16 query rows; the tile's
// key and value registers serve every block.  Per block the arithmetic of
// process_tile, except for the reference of the weights: it follows the
// running maximum without slack, so that the largest weight of a row is
// rounded least (8 sequences of 32768 tokens, peaked scores: error against
// 64 bits 2.5e-4, with the slack of kLazyRescale 7.7e-4, layer by layer
// 5.8e-4).  It costs rescales, which the memory streams hide (128 ragged
// sequences 43.1 against 42.0 us, the other cases the same).  Whether a
// column has a new maximum is one wave-wide vote of every lane on its own
// eight scores, so a tile without one moves nothing across lanes.
template <int D, int NB, bool LAST>
__device__ __forceinline__ void step_tile(WaveState<D> (&st)[NB], Tile<D>& t,
                                          const bf16x8 (&qf)[NB][Tile<D>::KK], int t0, int L,
                                          int col, int grp, float scale_log2, int pos_new,
                                          const uint16_t* new_row) {
  constexpr int KK = Tile<D>::KK, DB = Tile<D>::DB;
  if (LAST && pos_new >= t0 && pos_new < t0 + kTile)
    take_new_row<D>(t, t0, col, grp, pos_new, new_row);
  const int first = t0 + grp * 8;
  if (LAST && t0 + kTile > L) {  // positions >= L take no value
#pragma unroll
    for (int e = 0; e < 8; ++e)
      if (first + e >= L) {
#pragma unroll
        for (int db = 0; db < DB; ++db) t.v[db][e] = 0;
      }
  }
#pragma unroll
  for (int c = 0; c < NB; ++c) {
    f32x4 s0 = {0.f, 0.f, 0.f, 0.f}, s1 = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int kk = 0; kk < KK; ++kk) {
      s0 = mfma_bf16(as_bf16(t.k[0][kk]), qf[c][kk], s0);
      s1 = mfma_bf16(as_bf16(t.k[1][kk]), qf[c][kk], s1);
    }
    float x[8];
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      x[i] = s0[i];
      x[4 + i] = s1[i];
    }
    if (LAST && t0 + kTile > L) {  // ... and no weight
#pragma unroll
      for (int e = 0; e < 8; ++e)
        if (first + e >= L) x[e] = -INFINITY;
    }
    float tmax = fmaxf(fmaxf(fmaxf(x[0], x[1]), fmaxf(x[2], x[3])),
                       fmaxf(fmaxf(x[4], x[5]), fmaxf(x[6], x[7])));
    if (__ballot(tmax * scale_log2 > st[c].m)) {
      tmax = fmaxf(tmax, __shfl_xor(tmax, 16));
      tmax = fmaxf(tmax, __shfl_xor(tmax, 32));
      tmax *= scale_log2;
      const float m_new = tmax > st[c].m ? tmax : st[c].m;
      const float alpha = fast_exp2(st[c].m - m_new);  // 0 on the first tile, 1 if unchanged
      st[c].m = m_new;
      st[c].den *= alpha;
#pragma unroll
      for (int db = 0; db < DB; ++db) st[c].acc[db] *= alpha;
    }
    u16x8 pbits;
    const float neg_m = -st[c].m;
#pragma unroll
    for (int e = 0; e < 8; ++e)
      pbits[e] = f32_to_bf16_bits(fast_exp2(fmaf(x[e], scale_log2, neg_m)));
    const bf16x8 pf = as_bf16(pbits);
    const u16x8 ones = {0x3F80, 0x3F80, 0x3F80, 0x3F80, 0x3F80, 0x3F80, 0x3F80, 0x3F80};
    st[c].den = mfma_bf16(as_bf16(ones), pf, st[c].den);
#pragma unroll
    for (int db = 0; db < DB; ++db) st[c].acc[db] = mfma_bf16(as_bf16(t.v[db]), pf, st[c].acc[db]);
  }
}

template <int D, int NB, int W>
struct alignas(16) StepShared {
  float acc[W][16 * NB][D + 4];  // the waves' merge
  float m[W][16 * NB];
  float l[W][16 * NB];
  alignas(16) uint16_t new_row[2 * D];  // newest token's key and value
  double2 rope[kMaxRopePairs];          // the sequence's rotary (cos, sin) pairs
  uint16_t rot_q[16 * NB][D + 8];       // rotated query channels
  int last;
};

// SPLIT: units may have several runs (p.runs > 1).
template <int D, int NB, int W, bool SPLIT>
__global__ __launch_bounds__(W * 64) __attribute__((amdgpu_waves_per_eu(2)))
void step_kernel(StepParams p) {
  constexpr int KK = Tile<D>::KK, DB = Tile<D>::DB;
  constexpr int NT = W * 64;
  constexpr int D4 = D / 4;
  __shared__ StepShared<D, NB, W> sm;
  const int lane = threadIdx.x & 63;
  const int wave = threadIdx.x >> 6;
  const int col = lane & 15;
  const int grp = lane >> 4;

  // Workgroups go round the eight XCDs: the chunks of one run, which read the
  // same rows, are eight apart, so that they share an XCD's L2.
  const unsigned per8 = 8u * static_cast<unsigned>(p.chunks);
  const unsigned x8 = blockIdx.x / per8, xr = blockIdx.x - x8 * per8;
  const int chunk = static_cast<int>(xr >> 3);
  const unsigned item = x8 * 8 + (xr & 7);
  if (item >= p.items) return;
  const unsigned unit = item / static_cast<unsigned>(p.runs);
  const int j = static_cast<int>(item - unit * static_cast<unsigned>(p.runs));
  const int b = static_cast<int>(unit / static_cast<unsigned>(p.n_kv));
  const int kv = static_cast<int>(unit - static_cast<unsigned>(b) * p.n_kv);
  const int group = kv / p.kv_per_layer;  // layer group; the head's place inside a layer:
  const int head0 = (kv - group * p.kv_per_layer) * p.G;
  const int layer0 = group * p.layers;
  const int row0 = chunk * p.chunk_rows;
  const int n_rows = min(p.chunk_rows, p.layers * p.G - row0);  // this workgroup's rows

  const int ctx = p.ctx[b];
  int L = ctx < 0 ? 0 : ctx == INT32_MAX ? ctx : ctx + 1;
  L = L > p.max_len ? p.max_len : L;
  const int tiles = (L + kTile - 1) / kTile;
  // Runs of this unit: at most p.runs, which bounds those of the longest, and
  // what its own tiles allow; none shorter than p.min_tiles unless it is the
  // only one.
  int nb = 1;
  if constexpr (SPLIT) {
    nb = tiles / p.min_tiles;
    nb = nb < 1 ? 1 : nb > p.runs ? p.runs : nb;
    nb = min(nb, step_run_bound(tiles));
    if (j >= nb) return;
  }
  const int k0 = static_cast<int>(static_cast<long>(tiles) * j / nb);
  const int k1 = static_cast<int>(static_cast<long>(tiles) * (j + 1) / nb);

  const size_t seq = static_cast<size_t>(kv) * p.B + b;
  const uint16_t* kbase = p.k + seq * p.S * D;
  const uint16_t* vbase = p.v + seq * p.S * D;
  // Row rho of the unit: layer layer0 + rho / G, query head head0 + rho % G;
  // its place in q and out, in rows of D.
  auto row_of = [&](int rho) -> size_t {
    const int layer = rho / p.G;
    return (static_cast<size_t>(layer0 + layer) * p.B + b) * p.h + head0 + (rho - layer * p.G);
  };

  Tile<D> ta, tb;
  int it = k0 + wave;
  if (it < k1) load_tile<D>(ta, kbase, vbase, it * kTile, col, grp);

  // Everything the prologue reads is requested now, behind the first tiles:
  // this lane's query chunks, the newest token's row (the unit's last run) and,
  // with rotation, the chunk of a query row that this thread turns.
  u16x8 qraw[NB][KK];
#pragma unroll
  for (int c = 0; c < NB; ++c) {
    const int rr = c * 16 + col;
    const uint16_t* qrow = p.q + row_of(row0 + (rr < n_rows ? rr : 0)) * D + grp * 8;
#pragma unroll
    for (int kk = 0; kk < KK; ++kk) qraw[c][kk] = load16(qrow + kk * 32);
  }
  const int rope_half = p.rope_half;
  const int d_new = threadIdx.x * 8;  // channels of the newest row this thread takes
  const bool appends = j == nb - 1 && ctx >= 0 && ctx < p.S;
  const bool takes_row = appends && threadIdx.x < D / 8;
  u16x8 nk, nv, nk_partner;
  if (takes_row) {
    const size_t src = (static_cast<size_t>(b) * p.n_kv + kv) * D;
    nk = load16(p.k_new + src + d_new);
    nv = load16(p.v_new + src + d_new);
    if (d_new < 2 * rope_half)
      nk_partner = load16(p.k_new + src + partner_chunk(d_new, rope_half));
  }
  // Rotation: each chunk of a row is turned by one thread of the workgroup and
  // shared through LDS.  Every wave turning every row, after a table launch and
  // a round trip for its entries, took (us, before and now; in brackets without
  // rotation) one sequence of 128 tokens 13.8 and 10.7 (10.5), 128 ragged
  // sequences 40.5 and 36.8 (35.2), GQA at batch 31 130.4 and 127.6 (125.9).
  auto cs_lds = [&](int jj) { return sm.rope[jj]; };
  if (rope_half) {
    const int per_row = rope_half / 4, n_rot = n_rows * per_row;
    int i = threadIdx.x, rr = i / per_row, c0 = (i - rr * per_row) * 8;
    u16x8 own, partner;
    auto request = [&]() {
      const uint16_t* qrow = p.q + row_of(row0 + rr) * D;
      own = load16(qrow + c0);
      partner = load16(qrow + partner_chunk(c0, rope_half));
    };
    if (i < n_rot) request();
    if (threadIdx.x < rope_half) {
      if (p.rope_cs) {
        sm.rope[threadIdx.x] = reinterpret_cast<const double2*>(
            p.rope_cs)[static_cast<size_t>(b) * rope_half + threadIdx.x];
      } else {
        double sn, cs;
        sincos(static_cast<double>(ctx) * p.inv_freq[threadIdx.x], &sn, &cs);
        sm.rope[threadIdx.x] = make_double2(cs, sn);
      }
    }
    __syncthreads();
    while (i < n_rot) {
      *reinterpret_cast<u16x8*>(&sm.rot_q[rr][c0]) =
          rotate_chunk(own, partner, c0, rope_half, cs_lds);
      i += NT;
      if (i >= n_rot) break;
      rr = i / per_row;
      c0 = (i - rr * per_row) * 8;
      request();
    }
    if (takes_row && d_new < 2 * rope_half)
      nk = rotate_chunk(nk, nk_partner, d_new, rope_half, cs_lds);
  }

  // The newest token's row: every chunk's last run takes it from LDS where it
  // is attended (the write below may not be seen by its tile loads); the
  // first chunk's writes it to the cache.
  if (takes_row) {
    if (chunk == 0) {
      uint16_t* kc = const_cast<uint16_t*>(kbase);  // the caller's cache, written here only
      uint16_t* vc = const_cast<uint16_t*>(vbase);
      *reinterpret_cast<u16x8*>(kc + static_cast<size_t>(ctx & ~(kTile - 1)) * D +
                                kchunk<D>(ctx & (kTile - 1), d_new / 8) * 8) = nk;
      uint16_t* vdst = vc + static_cast<size_t>(ctx & ~(kTile - 1)) * D + (ctx & (kTile - 1));
#pragma unroll
      for (int e = 0; e < 8; ++e) vdst[(d_new + e) * kTile] = nv[e];
    }
    *reinterpret_cast<u16x8*>(&sm.new_row[d_new]) = nk;
    *reinterpret_cast<u16x8*>(&sm.new_row[D + d_new]) = nv;
  }
  const int pos_new = appends && ctx == L - 1 ? ctx : -1;
  // The staged row and the rotated queries are visible to every wave.
  if (pos_new >= 0 || rope_half) __syncthreads();

  bf16x8 qf[NB][KK];
  WaveState<D> st[NB];
#pragma unroll
  for (int c = 0; c < NB; ++c) {
    const int rr = c * 16 + col;
#pragma unroll
    for (int kk = 0; kk < KK; ++kk) {
      const int c0 = grp * 8 + kk * 32;
      u16x8 v = qraw[c][kk];
      if (c0 < 2 * rope_half) v = *reinterpret_cast<const u16x8*>(&sm.rot_q[rr][c0]);
      const u16x8 zero = {0, 0, 0, 0, 0, 0, 0, 0};
      qf[c][kk] = as_bf16(rr < n_rows ? v : zero);  // padded rows score zero
    }
    st[c].den = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int db = 0; db < DB; ++db) st[c].acc[db] = f32x4{0.f, 0.f, 0.f, 0.f};
  }

  // The loads of tile it+W are issued before tile it is consumed; the wave's
  // last tile is processed after the loop, with the ragged-end mask and the
  // newest token.
  if (it < k1) {
    for (;;) {
      const int nxt = it + W;
      if (nxt >= k1) break;
      load_tile<D>(tb, kbase, vbase, nxt * kTile, col, grp);
      step_tile<D, NB, false>(st, ta, qf, it * kTile, L, col, grp, p.scale_log2, -1, nullptr);
      it = nxt;
      const int nx2 = it + W;
      if (nx2 >= k1) {
        ta = tb;
        break;
      }
      load_tile<D>(ta, kbase, vbase, nx2 * kTile, col, grp);
      step_tile<D, NB, false>(st, tb, qf, it * kTile, L, col, grp, p.scale_log2, -1, nullptr);
      it = nx2;
    }
    step_tile<D, NB, true>(st, ta, qf, it * kTile, L, col, grp, p.scale_log2, pos_new, sm.new_row);
  }

  // Merge the waves through LDS; a unit of one run is finished here, another
  // leaves a partial per run.
  const size_t uc = static_cast<size_t>(unit) * p.chunks + chunk;
  const int part_floats = p.chunk_rows * D;  // one run's partial outputs, [row][channel]
  float* const unit_acc = nb > 1 ? p.part_acc + uc * p.runs * part_floats : nullptr;
  float* const unit_ml = nb > 1 ? p.part_ml + uc * p.runs * p.chunk_rows * 2 : nullptr;
  const __amdgpu_buffer_rsrc_t rsrc =
      device_rsrc(unit_acc, nb > 1 ? static_cast<uint32_t>(nb * part_floats * 4) : 0u);
#pragma unroll
  for (int c = 0; c < NB; ++c) {
    if (grp == 0) {
      sm.m[wave][c * 16 + col] = st[c].m;
      sm.l[wave][c * 16 + col] = st[c].den[0];
    }
#pragma unroll
    for (int db = 0; db < DB; ++db)
      *reinterpret_cast<f32x4*>(&sm.acc[wave][c * 16 + col][db * 16 + grp * 4]) = st[c].acc[db];
  }
  __syncthreads();
  for (int idx = threadIdx.x; idx < n_rows * D4; idx += NT) {
    const int rr = idx / D4;  // row inside the chunk
    const int d = (idx - rr * D4) * 4;
    float mw[W];
    float M = -INFINITY;
#pragma unroll
    for (int w = 0; w < W; ++w) {
      mw[w] = sm.m[w][rr];
      M = fmaxf(M, mw[w]);
    }
    const float ref = merge_reference(M);
    float wsum = 0.f;
    f32x4 o = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int w = 0; w < W; ++w) {
      const float f = fast_exp2(mw[w] - ref);
      wsum += f * sm.l[w][rr];
      o += f * *reinterpret_cast<const f32x4*>(&sm.acc[w][rr][d]);
    }
    if (!SPLIT || nb == 1) {
      store4_as<D>(p.out, p.out_bf16, row_of(row0 + rr), d, normalize4(o, wsum));
    } else {
      store4_device(rsrc, (j * part_floats + rr * D + d) * 4, o);
      if (d == 0) {
        store_device(&unit_ml[(j * p.chunk_rows + rr) * 2 + 0], M);
        store_device(&unit_ml[(j * p.chunk_rows + rr) * 2 + 1], wsum);
      }
    }
  }
  if constexpr (!SPLIT) return;
  if (nb == 1) return;

  // The last run of the unit to finish merges its runs in run order
  // (deterministic).  Every other run bumped the counter after its partials
  // completed, so the device-scope loads below see them.
  wait_stores_complete();
  __syncthreads();
  if (threadIdx.x == 0)
    sm.last = __hip_atomic_fetch_add(&p.counters[uc], 1, __ATOMIC_RELAXED,
                                     __HIP_MEMORY_SCOPE_AGENT) == nb - 1;
  __syncthreads();
  if (!sm.last) return;
  // A thread merges IT four-channel pieces of rows, all of them U runs at a
  // time with every load in flight: one round trip for up to U runs.
  constexpr int IT = (16 * NB * D4 + NT - 1) / NT;
  constexpr int U = IT == 1 ? 16 : 8;
  float M[IT], den[IT];
  f32x4 o[IT];
#pragma unroll
  for (int i = 0; i < IT; ++i) {
    M[i] = -INFINITY;
    den[i] = 0.f;
    o[i] = f32x4{0.f, 0.f, 0.f, 0.f};
  }
  for (int s0 = 0; s0 < nb; s0 += U) {
    float m[U][IT], w[U][IT];
    f32x4 a[U][IT];
#pragma unroll
    for (int u = 0; u < U; ++u) {
#pragma unroll
      for (int i = 0; i < IT; ++i) {
        m[u][i] = -INFINITY;
        w[u][i] = 0.f;
        a[u][i] = f32x4{0.f, 0.f, 0.f, 0.f};
      }
      if (s0 + u < nb) {
#pragma unroll
        for (int i = 0; i < IT; ++i) {
          const int idx = min(static_cast<int>(threadIdx.x) + i * NT, n_rows * D4 - 1);
          const int rr = idx / D4;
          float* ml = &unit_ml[((s0 + u) * p.chunk_rows + rr) * 2];
          m[u][i] = load_device(ml);
          w[u][i] = load_device(ml + 1);
          a[u][i] = load4_device(rsrc, ((s0 + u) * part_floats + idx * 4) * 4);
        }
      }
    }
#pragma unroll
    for (int i = 0; i < IT; ++i) {
      float bm = M[i];
#pragma unroll
      for (int u = 0; u < U; ++u) bm = fmaxf(bm, m[u][i]);
      if (bm != -INFINITY) {
        const float sc = fast_exp2(M[i] - bm);  // 0 while nothing is accumulated
        den[i] *= sc;
        o[i] *= sc;
#pragma unroll
        for (int u = 0; u < U; ++u) {
          const float f = fast_exp2(m[u][i] - bm);
          den[i] += f * w[u][i];
          o[i] += f * a[u][i];
        }
        M[i] = bm;
      } else {  // no run so far has a score above -inf: their sums are zeros or NaN
#pragma unroll
        for (int u = 0; u < U; ++u) {
          den[i] += w[u][i];
          o[i] += a[u][i];
        }
      }
    }
  }
#pragma unroll
  for (int i = 0; i < IT; ++i) {
    const int idx = threadIdx.x + i * NT;
    if (idx < n_rows * D4) {
      const int rr = idx / D4;
      store4_as<D>(p.out, p.out_bf16, row_of(row0 + rr), (idx - rr * D4) * 4,
                   normalize4(o[i], den[i]));
    }
  }
  if (threadIdx.x == 0)  // ready for the next call on this workspace
    __hip_atomic_store(&p.counters[uc], 0, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

template <int D, int NB, int W>
hipError_t launch_step_w(const StepParams& p, hipStream_t stream, hipEvent_t start,
                         hipEvent_t stop) {
  const dim3 grid((p.items + 7) / 8 * 8 * static_cast<unsigned>(p.chunks));
  auto kernel = step_kernel<D, NB, W, false>;
  if (p.runs > 1) {  // the host splits units only on eight-wave workgroups
    if constexpr (W == kWideWaves)
      kernel = step_kernel<D, NB, W, true>;
    else
      return hipErrorInvalidValue;
  }
  if (start)
    hipExtLaunchKernelGGL(kernel, grid, dim3(W * 64), 0, stream, start, stop, 0, p);
  else
    hipLaunchKernelGGL(kernel, grid, dim3(W * 64), 0, stream, p);
  return hipGetLastError();
}

template <int D, int NB>
hipError_t launch_step_t(const StepParams& p, hipStream_t stream, hipEvent_t start,
                         hipEvent_t stop) {
  if (p.waves == kWideWaves) return launch_step_w<D, NB, kWideWaves>(p, stream, start, stop);
  return launch_step_w<D, NB, kWaves>(p, stream, start, stop);
}

}  // namespace

hipError_t launch_step(const StepParams& p, int head_dim, hipStream_t stream, hipEvent_t start,
                       hipEvent_t stop) {
  const int blocks = (p.chunk_rows + 15) / 16;
  if (head_dim == 64) {
    if (blocks == 1) return launch_step_t<64, 1>(p, stream, start, stop);
    if (blocks == 2) return launch_step_t<64, 2>(p, stream, start, stop);
    if (blocks == 3) return launch_step_t<64, 3>(p, stream, start, stop);
  } else {
    if (blocks == 1) return launch_step_t<128, 1>(p, stream, start, stop);
    if (blocks == 2) return launch_step_t<128, 2>(p, stream, start, stop);
  }
  return hipErrorInvalidValue;
}

}  // namespace mlkv
