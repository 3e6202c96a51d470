// Matmul over at most 64 rows in narrow column tiles: the streaming kernel.
//
// A short product (a few to 50 MB of weights) is over in 10 - 20 us, of which the stream is half: the rest
// is what comes after it, above all the meeting of the k splits (publish a partial tile, count, read all
// of them, run the epilogue).  That part grows with the tile, so here a workgroup owns 32 or 64 columns
// (128 where a normalised head of 128 has to stay whole) and its eight wavefronts share out its k range:
// each pulls its own run of the packed weights AND its own fragments of the activation panel straight to
// registers, D steps of 16 ahead, with no LDS and no barrier until the eight accumulators are added up.
// Both come through one ring of equal depth, because loads return in order: a wait for the panel is a
// wait for every weight requested before it.
//
// What bounds it: the panel is read once per 32 or 64 columns, so a CU draws 3 or 2 bytes per byte of weights
// over 32 rows, 5 or 3 over 64 ((2 * columns + 4 * rows) / (2 * columns)), at 60 - 70 GB/s; below 200 KB a workgroup the chain first data (2.2 us) - sum of the
// wavefronts (1 - 2) - publish and count (1 - 1.8) - read the splits (1.2 - 2.1) - epilogue (0.6 - 1.8).
// Over 60 rows, 128-column kernel -> this one: 2048 x 6144 22.5 -> 15.8 us, 2048 x 2048 14.3 -> 10.5,
// 4096 x 2048 (QKV) 19.5 -> 15.2, 4096 x 4096 18.6 -> 17.6; 1472-wide layers (23 blocks of 64) over 46
// rows: QKV 18.6 -> 14.6, down 17.1 -> 10.9, gate + up 16.3 -> 15.9.
//
// The accumulators are added up in fragment order (16-byte LDS accesses); partial tiles go to memory in
// the same order, so that the last workgroup to arrive adds its splits lane by lane and only the sum is
// turned into rows.
#include "gemm_tile.hpp"

namespace ts {

template <int MB, int NB, int D, int EPI>
__global__ __launch_bounds__(512) void k_gemm_stream(GemmArgs a) {
  constexpr int NT = 512, RB = MB * 32, TN = NB * 32, LD = TN + 4;
  constexpr int MG = MB * NB > 4 ? 4 / NB : MB;      // row blocks that go through LDS at a time
  constexpr int NQ = NB * MG * 4;                    // 1 KB accumulator fragments (4 registers x 64 lanes) of those
  constexpr int QW = (NQ + 7) / 8;                   // fragments that a wavefront adds up
  constexpr int LDS_BYTES = 8 * NQ * 1024 > RB * LD * 4 ? 8 * NQ * 1024 : RB * LD * 4;
  __shared__ __attribute__((aligned(16))) unsigned char lds[LDS_BYTES];
  f32x4 (*frag)[NQ][64] = (f32x4(*)[NQ][64])lds;     // accumulators of the eight wavefronts
  float *tl = (float *)lds;                          // then the reduced tile
  __shared__ float s_tmp[NT], s_rs[RB];
  __shared__ int s_last;

  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);   // scalar: addresses stay in scalar registers
  const int ln = lane & 31, g = lane >> 5;
  const int tile = blockIdx.x, split = blockIdx.y;
  const int kb_total = a.k >> 6;
  const int b0 = kb_total * split / a.n_splits, nb = kb_total * (split + 1) / a.n_splits - b0;   // 64-deep blocks
  const int wb = b0 + nb * wave / 8, ns = 4 * (b0 + nb * (wave + 1) / 8 - wb);                   // this wavefront's, in steps of 16
  const int first = min(wb, kb_total - 1), last = max(ns - 1, 0);

  // ---- the packed sub-tiles (32 columns each).  SWIGLU: gate sub-tiles, then the matching up
  // sub-tiles.  Sub-tiles past the end are clamped to the last one (their columns are never stored).
  const bf16 *wp[NB];
#pragma unroll
  for (int i = 0; i < NB; ++i) {
    int sidx = 0, sub;
    if (EPI == EPI_SWIGLU) {
      sidx = i >= NB / 2;
      sub = tile * (NB / 2) + i % (NB / 2);
    } else {
      int n0 = (tile * NB + i) * 32;
      if (EPI == EPI_QKV && NB == 2 && a.head_dim == 128) n0 = (4 * (tile >> 1) + (tile & 1) + 2 * i) * 32;
      if (a.n_seg > 1 && n0 >= a.seg[1].col0) sidx = 1;
      if (a.n_seg > 2 && n0 >= a.seg[2].col0) sidx = 2;
      sub = (n0 - (sidx == 0 ? a.seg[0].col0 : (sidx == 1 ? a.seg[1].col0 : a.seg[2].col0))) >> 5;
    }
    const bf16 *wseg = (const bf16 *)(sidx == 0 ? a.seg[0].w : (sidx == 1 ? a.seg[1].w : a.seg[2].w));
    const int seg_rows = sidx == 0 ? a.seg[0].n_rows : (sidx == 1 ? a.seg[1].n_rows : a.seg[2].n_rows);
    sub = min(max(sub, 0), ((seg_rows + 31) >> 5) - 1);
    wp[i] = wseg + ((size_t)sub * kb_total + first) * 2048;
  }
  const bf16 *xp = (const bf16 *)a.x + (size_t)first * 4 * MB * 2 * 512;

  RowScale<NT, RB> scale;
  if (a.n_splits == 1) scale.issue(a, 0);
  __builtin_amdgcn_sched_barrier(0);   // requested before the ring: loads come back in order

  f32x16 acc[NB][MB];
#pragma unroll
  for (int i = 0; i < NB; ++i)
#pragma unroll
    for (int m = 0; m < MB; ++m)
#pragma unroll
      for (int e = 0; e < 16; ++e) acc[i][m][e] = 0.f;

  bf16x8 w[D][NB], x[D][2 * MB];
  auto load = [&](int slot, int s) {
    const size_t c = (size_t)min(s, last);
#pragma unroll
    for (int i = 0; i < NB; ++i) w[slot][i] = __builtin_nontemporal_load((const bf16x8 *)(wp[i] + c * 512) + lane);
#pragma unroll
    for (int m = 0; m < 2 * MB; ++m) x[slot][m] = *((const bf16x8 *)(xp + (c * 2 * MB + m) * 512) + lane);
  };
  auto mul = [&](int slot) {
    // high parts, then low parts: consecutive instructions add to different accumulators
#pragma unroll
    for (int p = 0; p < 2; ++p)
#pragma unroll
      for (int i = 0; i < NB; ++i)
#pragma unroll
        for (int m = 0; m < MB; ++m)
          acc[i][m] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(x[slot][2 * m + p], w[slot][i], acc[i][m], 0, 0, 0);
  };
#pragma unroll
  for (int d = 0; d < D; ++d) load(d, d);
  __builtin_amdgcn_sched_barrier(0);
  if (a.n_splits == 1) scale.finish(a, 0, s_tmp, s_rs);
  int s0 = 0;
  for (; s0 + D < ns; s0 += D) {
#pragma unroll
    for (int d = 0; d < D; ++d) {
      mul(d);
      load(d, s0 + D + d);
      __builtin_amdgcn_sched_barrier(0);
    }
  }
#pragma unroll
  for (int d = 0; d < D; ++d)
    if (s0 + d < ns) mul(d);   // wave-uniform

  // ---- add the eight wavefronts up, in fragment order (16-byte accesses, no conflicts): wavefront w
  // takes fragments w * QW .. of every group, in ascending wavefront order
  f32x4 sum[MB / MG][QW];
#pragma unroll
  for (int mg = 0; mg < MB / MG; ++mg) {
    if (mg > 0) __syncthreads();
#pragma unroll
    for (int m = 0; m < MG; ++m)
#pragma unroll
      for (int i = 0; i < NB; ++i)
#pragma unroll
        for (int q = 0; q < 4; ++q) {
          const f32x16 &c = acc[i][mg * MG + m];
          frag[wave][(m * NB + i) * 4 + q][lane] = f32x4{c[4 * q], c[4 * q + 1], c[4 * q + 2], c[4 * q + 3]};
        }
    __syncthreads();
#pragma unroll
    for (int u = 0; u < QW; ++u) {
      const int f = wave * QW + u;
      if (NQ % 8 == 0 || f < NQ) {   // wave-uniform
        f32x4 v[8];
#pragma unroll
        for (int w8 = 0; w8 < 8; ++w8) v[w8] = frag[w8][f][lane];
#pragma unroll
        for (int w8 = 1; w8 < 8; ++w8) v[0] += v[w8];
        sum[mg][u] = v[0];
      }
    }
  }

  TileEpilogue<EPI == EPI_HEAD ? EPI_PLAIN : EPI, TN, NT, RB> epi;
  if (EPI != EPI_HEAD && a.n_splits > 1) {
    // partial tiles [split][tile][fragment][lane]: written through, and read by the last workgroup to
    // arrive with the same mapping (nobody reads them earlier in this launch, so no stale line exists)
    const size_t tile_elems = (size_t)RB * TN, stride = (size_t)a.n_tiles * tile_elems;
    float *p0 = a.part + (size_t)tile * tile_elems + (size_t)lane * 4;
    auto at = [&](int mg, int u) { return (size_t)((mg * NQ + wave * QW + u) * 256); };
#pragma unroll
    for (int mg = 0; mg < MB / MG; ++mg)
#pragma unroll
      for (int u = 0; u < QW; ++u)
        if (NQ % 8 == 0 || wave * QW + u < NQ) store_f32x4<true>(p0 + (size_t)split * stride + at(mg, u), sum[mg][u]);
    if (!publish_then_count(&a.counters[tile], a.n_splits, &s_last)) return;
    scale.issue(a, 0);
    epi.preload(a, tile, 0);
    constexpr int PER = MB / MG * QW, SG = PER >= 4 ? 4 : 8;   // splits requested side by side
    for (int s = 0; s < a.n_splits; s += SG) {
      f32x4 v[SG][PER];
#pragma unroll
      for (int q = 0; q < SG; ++q)
#pragma unroll
        for (int u = 0; u < PER; ++u)
          if (NQ % 8 == 0 || wave * QW + u % QW < NQ)
            v[q][u] = *(const f32x4 *)(p0 + (size_t)min(s + q, a.n_splits - 1) * stride + at(u / QW, u % QW));
#pragma unroll
      for (int q = 0; q < SG; ++q)
#pragma unroll
        for (int u = 0; u < PER; ++u) {
          if (s + q == 0) sum[u / QW][u % QW] = v[q][u];
          else if (s + q < a.n_splits) sum[u / QW][u % QW] += v[q][u];
        }
    }
    scale.finish(a, 0, s_tmp, s_rs);
  } else if constexpr (EPI != EPI_HEAD) {
    epi.preload(a, tile, 0);
  }
  // ---- the reduced tile, row by row
  __syncthreads();   // the fragments have been read
#pragma unroll
  for (int mg = 0; mg < MB / MG; ++mg)
#pragma unroll
    for (int u = 0; u < QW; ++u) {
      const int f = wave * QW + u;
      if (NQ % 8 == 0 || f < NQ) {
        const int m = f / (4 * NB), i = (f >> 2) % NB, q = f & 3;
#pragma unroll
        for (int e = 0; e < 4; ++e) tl[((mg * MG + m) * 32 + 8 * q + 4 * g + e) * LD + i * 32 + ln] = sum[mg][u][e];
      }
    }
  __syncthreads();
  if constexpr (EPI == EPI_HEAD)
    head_rows<TN, NT, RB, LD>(a, tl, s_rs, tile, 0);
  else
    epi.apply(a, [&](int lr, int c) { return *(const f32x4 *)(tl + lr * LD + c); }, s_rs, tile, 0);
}

template <int EPI>
static void dispatch_stream(hipStream_t st, const GemmArgs &a) {
  const dim3 grid(a.n_tiles, a.n_splits), block(512);
#define TS_LAUNCH(NB_, D1_, D2_)                                                              \
  do {                                                                                        \
    if (a.rows_pad == 32) hipLaunchKernelGGL((k_gemm_stream<1, NB_, D1_, EPI>), grid, block, 0, st, a); \
    else hipLaunchKernelGGL((k_gemm_stream<2, NB_, D2_, EPI>), grid, block, 0, st, a);        \
  } while (0)
  if constexpr (EPI == EPI_QKV || EPI == EPI_HEAD) {
    if (a.tile_n == 128) { TS_LAUNCH(4, 6, 3); return; }
  }
  if constexpr (EPI != EPI_HEAD) {
    if (a.tile_n == 64) { TS_LAUNCH(2, 10, 6); return; }
    if constexpr (EPI == EPI_RESID || EPI == EPI_PLAIN) TS_LAUNCH(1, 12, 8);
  }
#undef TS_LAUNCH
}

void launch_gemm_stream(hipStream_t st, const GemmArgs &a) {
  switch (a.epi) {
    case EPI_QKV: dispatch_stream<EPI_QKV>(st, a); break;
    case EPI_RESID: dispatch_stream<EPI_RESID>(st, a); break;
    case EPI_SWIGLU: dispatch_stream<EPI_SWIGLU>(st, a); break;
    case EPI_PLAIN: dispatch_stream<EPI_PLAIN>(st, a); break;
    default: dispatch_stream<EPI_HEAD>(st, a); break;
  }
}

}  // namespace ts
