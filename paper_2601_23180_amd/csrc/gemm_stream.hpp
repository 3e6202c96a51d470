// Matmul over at most 128 rows in narrow column tiles: the streaming kernel.
//
// A short product (a few to 250 MB of weights) is over in 6 - 60 us, and the stream is not all of it: the launch
// and the first memory round trip take 3 us, the meeting of the k splits 1 - 10.  So a workgroup owns a tile of 16 to 128
// columns, sized so that about every CU has one, and its wavefronts share out its k range: each pulls its own
// run of the packed weights AND its own fragments of the activation panel straight to registers, D steps of 32 ahead,
// with no LDS and no barrier until the accumulators are added up.
//
// Matrix instructions of 16 x 16 x 32: row blocks of 16, so that 9 rows read and multiply 16 and 37 rows 48, and
// column blocks of 16.  A tile holds whole rotation pairs (of a part of a head), or gate columns beside their up
// columns, in any multiple of 16 (QKV: 8 pairs).
//
// What bounds it: loads come back in order, so a CU's requests for the panel (from the L2) wait behind its requests
// for weights; it draws both together at 45 - 60 GB/s, 2 bytes a column and 64 a row block and k step.  Meeting
// the splits is bound by the size of the partial tile: it is written through to memory (32 KB a workgroup 1.7
// us; as 8-byte stores, which leave half lines, 3.3), counted, and read back by one CU, or by one a row block.  Without the stream's 3 us, meeting costs
// 3.5 us at 32 columns x 64 rows and 11 at 128.  The host weighs one against the other (plan_stream in plan.hpp).
// Measured, us, before (128-column kernel, or tiles of 32 and 64 columns in 32-row blocks) -> now.  9 rows: 4096 x 1024 (QKV) 10.5 -> 6.3,
// 1024 x 2048 8.9 -> 6.3, 6144 x 1024 (gate + up) 9.0 -> 6.5, 1024 x 3072 9.0 -> 6.8.  One row: 6144 x 4096 17.2 -> 15.9, 4096 x
// 4096 12.0 -> 10.6, 24576 x 4096 38.4 -> 33.1, 4096 x 12288 23.7 -> 20.1.  36 rows: 13.6 -> 8.1, 10.4 -> 7.4, 13.2 -> 8.4, 10.4 -> 8.5 at the
// widths of the 9 rows.  60 rows: 6144 x 4096 24.4 -> 23.2, 24576 x 4096 45.7 -> 43.3, 4096 x 2048 15.1 -> 12.2, 12288 x 2048 20.2
// -> 17.3, 4096 x 4096 and 4096 x 12288 even.  128 rows, two launches before (products and their finish): 24576 x 4096 70 -> 63.5, 111 rows:
// 2048 x 2048 16.3 -> 12.3, 12288 x 2048 29.4 -> 25.4, 2048 x 6144 22.2 -> 19.9.
//
// The accumulators are added up in fragment order (16-byte LDS accesses); partial tiles go to memory in the
// same order, so that whoever finishes a tile or a row block of it adds the splits lane by lane and only the sum is turned into rows.
#pragma once

#include "gemm_tile.hpp"
#include "meet.hpp"
#include "plan.hpp"

namespace ts {

// Wavefronts and the most steps in flight: 8 wavefronts of up to 256 registers, or 4 of up to 512 where the
// accumulators of a tile are large; a power of two of steps that fits beside the accumulators, with no more requests
// than a wavefront can have outstanding.
template <int RB, int CB>
struct StreamShape {
  static constexpr int kStep = CB + 2 * RB, kUsed = 4 * RB * CB + 44;
  static constexpr int NW = (256 - kUsed) / (4 * kStep) >= 2 ? 8 : 4;
  static constexpr int kRegs = ((NW == 8 ? 256 : 512) - kUsed) / (4 * kStep), kFit = kRegs < 60 / kStep ? kRegs : 60 / kStep;
  static constexpr int D = kFit >= 8 ? 8 : (kFit >= 4 ? 4 : 2);
  static_assert(kFit >= 2, "two steps in flight at least");
  // row blocks whose accumulators go through LDS at a time: at most 150 KB of them
  static constexpr int kBlk = NW * CB, MG = kBlk * RB <= 150 ? RB : (RB % 2 == 0 && kBlk * (RB / 2) <= 150 ? RB / 2 : (RB % 4 == 0 && kBlk * (RB / 4) <= 150 ? RB / 4 : 1));
};

// The arguments of k_gemm_stream, read again: what a rare path needs of them is not held in registers through the common one
__device__ __forceinline__ const GemmArgs &args_again() {
  auto p = (const __attribute__((address_space(4))) GemmArgs *)__builtin_amdgcn_kernarg_segment_ptr();
  asm volatile("" : "+s"(p));
  return *(const GemmArgs *)p;
}

// RB: 16-row blocks, CB: 16-column blocks of the tile, NW: wavefronts, D: steps in flight.  MEET: the workgroups of a tile finish it
// together (tile_meets in plan.hpp), in a kernel of its own: with both ways to finish in one, tiles that one workgroup
// finishes held what the other way needs (QKV, 48 rows x 16 columns: 96 -> 150 vector registers, 100 scalar ones spilt; 64 x 32: 20
// bytes of scratch a lane).
template <int RB, int CB, int NW, int D, int EPI, bool MEET>
__global__ __launch_bounds__(64 * NW) void k_gemm_stream(GemmArgs a) {
  constexpr int NT = 64 * NW, ROWS = RB * 16, TN = CB * 16, LD = TN + 4;
  // 32-row blocks of the activation panel: as many as the rows need, or the four of two row groups
  const int MBT = RB <= 2 ? 1 : (RB == 3 ? 2 : (RB > 4 ? 4 : a.rows_pad >> 5));
  constexpr int MG = StreamShape<RB, CB>::MG;                      // row blocks that go through LDS at a time
  constexpr int NQ = CB * MG;                                      // 1 KB accumulator fragments of those
  constexpr int QW = (NQ + NW - 1) / NW;                           // fragments that a wavefront adds up
  constexpr int LDS_BYTES = NW * NQ * 1024 > ROWS * LD * 4 ? NW * NQ * 1024 : ROWS * LD * 4;
  constexpr int SROWS = RB <= 2 ? ROWS : (RB <= 4 ? 64 : 128);
  __shared__ __attribute__((aligned(16))) unsigned char lds[LDS_BYTES];
  f32x4 (*frag)[NQ][64] = (f32x4(*)[NQ][64])lds;     // accumulators of the wavefronts
  float *tl = (float *)lds;                          // then the reduced tile
  __shared__ float s_tmp[NT], s_rs[SROWS];
  __shared__ int s_last;

  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);   // scalar: addresses stay in scalar registers
  const int lc = lane & 15, q4 = lane >> 4;
  const int tile = blockIdx.x, split = blockIdx.y, row0 = blockIdx.z * ROWS;   // row groups: panels of 128 rows with RB = 4
  const int kb_total = a.k >> 6, st_total = 2 * kb_total;      // 64-deep blocks, steps of 32
  const int b0 = st_total * split / a.n_splits, nb = st_total * (split + 1) / a.n_splits - b0;
  const int wb = b0 + nb * wave / NW, ns = b0 + nb * (wave + 1) / NW - wb;   // this wavefront's steps
  const int first = min(wb, st_total - 1), last = max(ns - 1, 0);

  // ---- the packed weights.  A column block has a scalar base (its matrix, its columns, this wavefront's run);
  // the lanes share one byte offset.  Fragment (64-deep block, j) of a 32-column sub-tile: lane half g holds
  // k = 32 g + 8 j ..; lane group q4 of the instruction takes (j, g) = (2 (step % 2) + q4 / 2, q4 % 2), here and
  // in the activations.  Blocks past the end are clamped to the last columns (never stored).
  constexpr bool kLanes = EPI == EPI_SWIGLU && CB % 2 != 0;   // blocks that straddle sub-tiles, one of them gate and up: a pointer per lane
  const char *wp[CB];
  uint32_t wo = (q4 >> 1) * 1024 + ((q4 & 1) * 32 + lc) * 16;
#pragma unroll
  for (int i = 0; i < CB; ++i) {
    const void *w = a.seg[0].w;
    int c0 = tile * TN + i * 16, c_end = a.n_total;
    if constexpr (kLanes) {
      const int c = i * 16 + lc;
      w = c >= TN / 2 ? a.seg[1].w : a.seg[0].w;
      c0 = min(tile * (TN / 2) + (c >= TN / 2 ? c - TN / 2 : c), a.ffn - 1);
    } else {
      if constexpr (EPI == EPI_SWIGLU) {
        if (i >= CB / 2) w = a.seg[1].w;
        c0 = tile * (TN / 2) + (i % (CB / 2)) * 16;
        c_end = a.ffn;
      } else if constexpr (EPI == EPI_QKV) {   // a block lies inside one head, and so inside one matrix
        c0 = min(qkv_column<TN>(tile, i * 16, a.head_dim), a.n_total - 16);
        if (c0 >= a.seg[2].col0) { w = a.seg[2].w; c0 -= a.seg[2].col0; c_end = a.seg[2].n_rows; }
        else if (c0 >= a.seg[1].col0) { w = a.seg[1].w; c0 -= a.seg[1].col0; c_end = a.seg[1].n_rows; }
      }
      c0 = min(c0, (c_end - 1) & ~15);
    }
    wp[i] = (const char *)w + ((size_t)(c0 >> 5) * st_total + first) * 2048 + (c0 & 31) * 16 - (kLanes ? lc * 16 : 0);
  }
  if constexpr (EPI == EPI_QKV && CB == 1) {   // 8 low features of a head, then their 8 high ones
    if (lc >= 8) wo += (uint32_t)(a.head_dim >> 6) * st_total * 2048u - 8 * 16;
  }
  const char *xp = (const char *)a.x + (size_t)first * (MBT * 4096) + (RB == 4 ? blockIdx.z * 4096 : 0);
  const uint32_t xo = (q4 >> 1) * (MBT * 2048) + ((q4 & 1) * 32 + lc) * 16;

  RowScale<NT, SROWS, (RB <= 4 ? 128 : 64) * SROWS / NT> scale;   // as many entries a row are requested ahead
  constexpr bool kScaleLate = RB > 4;   // no registers to spare: behind the stream
  if (!MEET && !kScaleLate && a.n_splits == 1) scale.issue(a, row0);
  __builtin_amdgcn_sched_barrier(0);   // requested before the ring: loads come back in order

  f32x4 acc[CB][RB];
#pragma unroll
  for (int i = 0; i < CB; ++i)
#pragma unroll
    for (int m = 0; m < RB; ++m) acc[i][m] = f32x4{0.f, 0.f, 0.f, 0.f};

  bf16x8 w[D][CB], x[D][2 * RB];
  // A run that is no whole number of rounds requests its last step again: no branch around any load, behind
  // which a wait would drain everything.  launch_ring picks D so that this is one step at most.
  auto load = [&](int slot, int s_) {
    const int s = min(s_, last);
#pragma unroll
    for (int i = 0; i < CB; ++i) w[slot][i] = __builtin_nontemporal_load((const bf16x8 *)(wp[i] + (size_t)s * 2048 + wo));
    const char *xs = xp + (size_t)s * (MBT * 4096);
#pragma unroll
    for (int m = 0; m < RB; ++m)
#pragma unroll
      for (int p = 0; p < 2; ++p) x[slot][2 * m + p] = *(const bf16x8 *)(xs + ((m >> 1) * 2 + p) * 1024 + (m & 1) * 256 + xo);
  };
  auto mul = [&](int slot) {
    // high parts, then low parts: consecutive instructions add to different accumulators
#pragma unroll
    for (int p = 0; p < 2; ++p)
#pragma unroll
      for (int i = 0; i < CB; ++i)
#pragma unroll
        for (int m = 0; m < RB; ++m)
          acc[i][m] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(x[slot][2 * m + p], w[slot][i], acc[i][m], 0, 0, 0);
  };
#pragma unroll
  for (int d = 0; d < D; ++d) load(d, d);
  __builtin_amdgcn_sched_barrier(0);
  if (!MEET && !kScaleLate && a.n_splits == 1) scale.partial(a, row0, s_tmp);
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

  if (!MEET && kScaleLate && a.n_splits == 1) {
    scale.issue(a, row0);
    scale.partial(a, row0, s_tmp);
  }
  // ---- add the wavefronts up, in fragment order (16-byte accesses, no conflicts): wavefront w takes
  // fragments w * QW .. of every group, in ascending wavefront order
  f32x4 sum[RB / MG][QW];
#pragma unroll
  for (int mg = 0; mg < RB / MG; ++mg) {
    if (mg > 0) __syncthreads();
#pragma unroll
    for (int m = 0; m < MG; ++m)
#pragma unroll
      for (int i = 0; i < CB; ++i) frag[wave][m * CB + i][lane] = acc[i][mg * MG + m];
    __syncthreads();
#pragma unroll
    for (int u = 0; u < QW; ++u) {
      const int f = wave * QW + u;
      if (NQ % NW == 0 || f < NQ) {   // wave-uniform
        f32x4 v[NW];
#pragma unroll
        for (int w8 = 0; w8 < NW; ++w8) v[w8] = frag[w8][f][lane];
#pragma unroll
        for (int w8 = 1; w8 < NW; ++w8) v[0] += v[w8];
        sum[mg][u] = v[0];
      }
    }
  }

  // The tile is finished by all its workgroups, a block of 16 rows each: one CU reading 32 KB a split back and finishing 64 rows
  // was the longest link of the chain behind the stream.  60 rows, us: 4096 x 12288 in 128 columns x 8 splits 30.9 -> 28.1 (31.6 in 64 x 4
  // before), 6144 x 4096 in 96 x 4 23.3 -> 21.7; 111 rows, two groups of 64: 4096 x 2048 21.6 -> 16.4.  The words they meet at are
  // 64 bytes apart: side by side, with all of them polled, the same took 2 - 4 us longer than one workgroup alone.
  if constexpr (MEET) {
    const int tl_id = blockIdx.z * a.n_tiles + tile;
    const size_t tile_elems = (size_t)ROWS * TN, stride = (size_t)gridDim.z * a.n_tiles * tile_elems;
    const ThroughBuffer mine(a.part + (size_t)split * stride + (size_t)tl_id * tile_elems, (uint32_t)tile_elems * 4);
#pragma unroll
    for (int mg = 0; mg < RB / MG; ++mg)
#pragma unroll
      for (int u = 0; u < QW; ++u)
        if (NQ % NW == 0 || wave * QW + u < NQ) mine.store((uint32_t)((mg * NQ + wave * QW + u) * 1024 + lane * 16), sum[mg][u]);
    if (split == 0)   // the words that the next launch meets at; the one before this has ended
      for (int i = tl_id + tid * (int)gridDim.z * a.n_tiles; i < a.n_counters; i += NT * (int)gridDim.z * a.n_tiles)
        __hip_atomic_store(&a.next_counters[i * kMeetStride], 0, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    __builtin_amdgcn_s_waitcnt(0);   // this thread's partial sums are acknowledged
    __syncthreads();
    // Row block `split` is this workgroup's, if there is one; what does not depend on the sums is requested before the wait
    const int n_blocks = min(RB, (a.rows - row0 + 15) >> 4);
    TileEpilogue<EPI, TN, NT, 16> bepi;
    RowScale<NT, 16> bscale;
    auto request = [&](const GemmArgs &g, int m) {
      bscale.issue(g, row0 + 16 * m);
      bepi.preload(g, tile, row0 + 16 * m);
    };
    auto finish_block = [&](const GemmArgs &g, int m) {
      constexpr int QB = (CB + NW - 1) / NW, SG = QB > 1 ? 4 : 8;   // fragments a wavefront, splits side by side
      f32x4 bsum[QB];
      for (int s = 0; s < g.n_splits; s += SG) {
        f32x4 v[SG][QB];
#pragma unroll
        for (int q = 0; q < SG; ++q)
#pragma unroll
          for (int u = 0; u < QB; ++u) {
            const int f = min(wave + u * NW, CB - 1);
            v[q][u] = *(const f32x4 *)(g.part + (size_t)min(s + q, g.n_splits - 1) * stride + (size_t)tl_id * tile_elems + (m * CB + f) * 256 + lane * 4);
          }
#pragma unroll
        for (int q = 0; q < SG; ++q)
#pragma unroll
          for (int u = 0; u < QB; ++u) {
            if (s + q == 0) bsum[u] = v[q][u];
            else if (s + q < g.n_splits) bsum[u] += v[q][u];
          }
      }
#pragma unroll
      for (int u = 0; u < QB; ++u) {
        const int f = wave + u * NW;
        if (CB % NW == 0 || f < CB)
#pragma unroll
          for (int e = 0; e < 4; ++e) tl[(4 * q4 + e) * LD + f * 16 + lc] = bsum[u][e];
      }
      bscale.finish(g, row0 + 16 * m, s_tmp, s_rs);   // ends with a barrier
      bepi.apply(g, [&](int lr, int c) { return *(const f32x4 *)(tl + lr * LD + c); }, s_rs, tile, row0 + 16 * m);
    };
    if (split < n_blocks) request(a, split);
    if (tid == 0) {
      MeetWord word{&a.counters[tl_id * kMeetStride], a.meet_ticks, 0};
      s_last = (int)meet_splits(word, a.n_splits, split, split < n_blocks);
    }
    __syncthreads();
    uint32_t take = s_last;
    if (split < n_blocks && (take >> split & 1u)) finish_block(a, split);
    for (take &= ~(1u << split); take != 0; take &= take - 1) {   // blocks of workgroups that have left
      const GemmArgs &again = args_again();
      __syncthreads();   // the block before has been read
      request(again, __builtin_ctz(take));
      finish_block(again, __builtin_ctz(take));
    }
    return;
  }
  TileEpilogue<EPI == EPI_HEAD ? EPI_PLAIN : EPI, TN, NT, ROWS> epi;
  constexpr bool kSplits = EPI != EPI_HEAD && EPI != EPI_SWIGLU;   // gate + up: tiles enough
  if (kSplits && a.n_splits > 1) {
    // partial tiles [split][tile][fragment][lane]: written through, and read by the last workgroup to
    // arrive with the same mapping (nobody reads them earlier in this launch, so no stale line exists)
    const int tl_id = blockIdx.z * a.n_tiles + tile;
    const size_t tile_elems = (size_t)ROWS * TN, stride = (size_t)gridDim.z * a.n_tiles * tile_elems;
    float *p0 = a.part + (size_t)tl_id * tile_elems + (size_t)lane * 4;
    auto at = [&](int mg, int u) { return (size_t)((mg * NQ + wave * QW + u) * 256); };
    const ThroughBuffer mine(a.part + (size_t)split * stride + (size_t)tl_id * tile_elems, (uint32_t)tile_elems * 4);
#pragma unroll
    for (int mg = 0; mg < RB / MG; ++mg)
#pragma unroll
      for (int u = 0; u < QW; ++u)
        if (NQ % NW == 0 || wave * QW + u < NQ) mine.store((uint32_t)(at(mg, u) * 4 + lane * 16), sum[mg][u]);
    if (!publish_then_count(&a.counters[tl_id], a.n_splits, &s_last)) return;
    scale.issue(a, row0);
    epi.preload(a, tile, row0);
    constexpr int PER = RB / MG * QW, SG = PER >= 16 ? 2 : (PER >= 4 ? 4 : 8);   // splits requested side by side
    for (int s = 0; s < a.n_splits; s += SG) {
      f32x4 v[SG][PER];
#pragma unroll
      for (int q = 0; q < SG; ++q)
#pragma unroll
        for (int u = 0; u < PER; ++u)
          if (NQ % NW == 0 || wave * QW + u % QW < NQ)
            v[q][u] = *(const f32x4 *)(p0 + (size_t)min(s + q, a.n_splits - 1) * stride + at(u / QW, u % QW));
#pragma unroll
      for (int q = 0; q < SG; ++q)
#pragma unroll
        for (int u = 0; u < PER; ++u) {
          if (s + q == 0) sum[u / QW][u % QW] = v[q][u];
          else if (s + q < a.n_splits) sum[u / QW][u % QW] += v[q][u];
        }
    }
    scale.finish(a, row0, s_tmp, s_rs);
  } else {
    scale.total(a, s_tmp, s_rs);   // the wavefronts have met since partial()
    if constexpr (EPI != EPI_HEAD) epi.preload(a, tile, row0);
  }
  // ---- the reduced tile, row by row
  __syncthreads();   // the fragments have been read
#pragma unroll
  for (int mg = 0; mg < RB / MG; ++mg)
#pragma unroll
    for (int u = 0; u < QW; ++u) {
      const int f = wave * QW + u;
      if (NQ % NW == 0 || f < NQ) {
        const int m = f / CB, i = f % CB;
#pragma unroll
        for (int e = 0; e < 4; ++e) tl[((mg * MG + m) * 16 + 4 * q4 + e) * LD + i * 16 + lc] = sum[mg][u][e];
      }
    }
  __syncthreads();
  if constexpr (EPI == EPI_HEAD)
    head_rows<TN, NT, ROWS, LD>(a, tl, s_rs, tile * TN, min((tile + 1) * TN, a.n_total), tile, row0);
  else
    epi.apply(a, [&](int lr, int c) { return *(const f32x4 *)(tl + lr * LD + c); }, s_rs, tile, row0);
}

template <int RB, int CB, int EPI, bool MEET>
void launch_ring(hipStream_t st, const GemmArgs &a) {
  using S = StreamShape<RB, CB>;
  const dim3 grid(a.n_tiles, a.n_splits, RB == 4 ? (a.rows + 63) / 64 : 1), block(64 * S::NW);
  // The deepest ring that divides the steps of a wavefront, for a ring deeper than the run requests its last step again
  // and again (2.5 us on a 6 us kernel).  Eight and four steps serve reductions that are powers of two, or three of them;
  // most others share out unevenly and have two in flight, with one step again at most.
  const int steps = a.k / 32, each = steps / (S::NW * a.n_splits);
  const int even = steps % (S::NW * a.n_splits) == 0 ? each : 2;
  if constexpr (S::D == 8) {
    if (even % 8 == 0) { hipLaunchKernelGGL((k_gemm_stream<RB, CB, S::NW, 8, EPI, MEET>), grid, block, 0, st, a); return; }
  }
  if constexpr (S::D >= 4) {
    if (even % 4 == 0) { hipLaunchKernelGGL((k_gemm_stream<RB, CB, S::NW, 4, EPI, MEET>), grid, block, 0, st, a); return; }
  }
  hipLaunchKernelGGL((k_gemm_stream<RB, CB, S::NW, 2, EPI, MEET>), grid, block, 0, st, a);
}
template <int RB, int CB, int EPI>
void launch_one(hipStream_t st, const GemmArgs &a) {
  if constexpr (tile_meets(EPI, RB, kMaxStreamSplits)) {
    if (tile_meets(EPI, RB, a.n_splits)) return launch_ring<RB, CB, EPI, true>(st, a);
  }
  launch_ring<RB, CB, EPI, false>(st, a);
}

// False, and nothing launched: not built
template <int RB, int EPI>
bool dispatch_cols(hipStream_t st, const GemmArgs &a) {
  auto built = [&](auto cb) {
    constexpr int CB = decltype(cb)::value;
    if constexpr (stream_built(EPI, CB * 16, RB)) launch_one<RB, CB, EPI>(st, a);
    return stream_built(EPI, CB * 16, RB);
  };
  switch (a.tile_n) {
    case 16: return built(IC<1>{});
    case 32: return built(IC<2>{});
    case 48: return built(IC<3>{});
    case 64: return built(IC<4>{});
    case 96: return built(IC<6>{});
    case 112: return built(IC<7>{});
    case 128: return built(IC<8>{});
    default: return false;
  }
}

template <int EPI>
bool dispatch_rows(hipStream_t st, const GemmArgs &a) {
  switch (row_blocks(a.rows)) {
    case 1: return dispatch_cols<1, EPI>(st, a);
    case 2: return dispatch_cols<2, EPI>(st, a);
    case 3: return dispatch_cols<3, EPI>(st, a);
    case 4: return dispatch_cols<4, EPI>(st, a);
    default:   // up to 128 rows; a head of 128 that stays whole: two groups of 64
      if (EPI == EPI_QKV && a.tile_n == 128) return dispatch_cols<4, EPI>(st, a);
      return row_blocks(a.rows) == 6 ? dispatch_cols<6, EPI>(st, a) : dispatch_cols<8, EPI>(st, a);
  }
}

}  // namespace ts
