// Matmul for panels of more than 128 activation rows (several sequences; for the LM head of a width that
// kernels_gemm.hip does not take, more than 64), where the
// matrix cores and not the weight stream set the time: 4 * rows * N * K flops for the high and low
// parts against 2 * N * K bytes cross at about 140 rows of one pass.
//
// A workgroup owns 128 rows x 256 columns or 128 x 128 of the product over one k split.  256 columns: four
// wavefronts with 128 x 64 accumulators, so that a weight fragment is multiplied with eight activation
// fragments and an activation fragment with two weight fragments: the LDS then delivers 64 bytes a
// clock at the full matrix rate, half of what it can.  128 columns: these tiles serve the smaller products, whose time
// is first data, waits and hand-over rather than matrix rate, so eight wavefronts of 64 x 32, two a SIMD, of which one works
// while the other waits; both rows of wavefronts read the same weights, the second out of the L1, hence without the
// non-temporal hint (40.3 -> 39.2, hinted 4096 x 14336 in 4 splits 77.7, plain 75.0).  Four wavefronts of 64 x 64 -> eight, 240 rows,
// us with the finishing launch: 1472 wide QKV 20.6 -> 18.6, O 15.5 -> 13.1, gate + up 28.3 -> 25.5, down 22.4 -> 20.0; 2048 wide 25.1 -> 24.0,
// 18.4 -> 17.0, 41.3 -> 40.1, 26.7 -> 25.3; 1024 wide 19.4 -> 18.6, 15.8 -> 14.5, 24.0 -> 21.7, 18.2 -> 16.6.  The 256-column tile with eight wavefronts
// of 64 x 64 is slower (28672 x 4096: 108 -> 120, 130 with the hint).
// Activations go global -> registers -> LDS in 64-deep chunks, double buffered; weights go straight
// to registers, two chunks ahead.
//
// The inner loop is written in fenced groups of two matrix instructions: without the fences the
// compiler moves every operand read down to the instruction that uses it and the wavefront waits
// for the LDS once per step (148 us for the 28672 x 4096 product over 256 rows; 105 us fenced, of
// which 7/8 of the chip is busy).  The reads of a step are issued one step ahead, across the chunk
// boundary too: the one barrier of a chunk sits before its last step, by which time every wavefront
// holds that step's operands in registers.
//
// Split K: the partial tiles go to memory with ordinary stores and k_gemm_finish, a second launch
// over the whole chip, adds them up and runs the epilogue.  At 256 rows a tile's partials are a
// megabyte: one workgroup reading them serially after the last arrival, as the narrow kernels do,
// took 15 - 20 us of a 77 us projection.
#include "gemm_tile.hpp"
#include "plan.hpp"

namespace ts {

template <int WR, int WC, int MBW, int NBW, int EPI, bool APART>
__global__ __launch_bounds__(WR * WC * 64) void k_gemm_wide(GemmArgs a) {
  static_assert(WR * MBW * 32 == kWideRows, "the wavefronts cover 128 rows");
  constexpr int NW = WR * WC, NT = NW * 64;
  constexpr int MB = WR * MBW;                   // 32-row blocks of the workgroup
  constexpr int TN = WC * NBW * 32;              // columns of the workgroup
  constexpr int FR = 4 * MB * 2, XV = FR / NW;    // 1 KB activation fragments per chunk, per wavefront
  constexpr int BUF = FR * 1024;
  constexpr int LD = TN + 4;                     // floats per row of the epilogue's LDS tile
  constexpr int EPI_BYTES = 32 * LD * 4, LDS_BYTES = 2 * BUF > EPI_BYTES ? 2 * BUF : EPI_BYTES;
  __shared__ __attribute__((aligned(1024))) unsigned char lds[LDS_BYTES];
  __shared__ float s_tmp[NT], s_rs[kWideRows];

  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int wr = wave / WC, wc = wave - wr * WC;
  const int ln = lane & 31, g = lane >> 5;
  // Workgroups go round-robin over the 8 XCDs: ids 8 apart are the row groups of one (tile, split), whose weights then
  // come through one L2 at about the same time (LM head 128256 x 4096 over 240 rows: 1187 MB into the L2s against 2187 for one group after the
  // other, 617 -> 546 us, 594 with the hint below).  Products of one round of workgroups, on the same buffers, against one group after the other: passes of
  // 81 models 1.5 % shorter (128 columns, at worst 0.2 % longer) and 0.4 % (256 columns, at worst 0.3 % longer).
  // APART: one row group after the other (wide_apart in plan.hpp).
  int tile, rg, split;
  if constexpr (APART) {
    tile = blockIdx.x; rg = blockIdx.y; split = blockIdx.z;
  } else {
    // no division: it is on the way to the first load (with three of them products of 8 - 15 us took 1 us more, passes of 81 models 1.4 %)
    static_assert(kMaxRows <= 2 * kWideRows, "one row group or two");
    const int n_tiles = (a.n_total + TN - 1) / TN, two = a.rows > kWideRows;
    const int item = (int)(blockIdx.x >> 3 >> two) * 8 + (blockIdx.x & 7);
    if (item >= n_tiles * a.n_splits) return;   // the last 8 are filled up
    rg = (int)(blockIdx.x >> 3) & two;
    split = a.n_splits == 1 ? 0 : wide_split(item, n_tiles, a.tiles_inv);
    tile = item - split * n_tiles;
  }
  const int mbt = a.rows_pad >> 5;
  const int kb_total = a.k >> 6;
  const int b0 = kb_total * split / a.n_splits, n = kb_total * (split + 1) / a.n_splits - b0;   // 64-deep blocks

  // ---- this wavefront's packed sub-tiles (32 columns each).  SWIGLU: the columns of the product
  // are 64 gate columns followed by their 64 up columns, 128 by 128.  Sub-tiles past the end are
  // clamped to the last one (their columns are never stored).
  const bf16 *wp[NBW];
#pragma unroll
  for (int i = 0; i < NBW; ++i) {
    const int vs = (tile * WC + wc) * NBW + i;   // sub-tile of the product
    int sidx, sub;
    if (EPI == EPI_SWIGLU) {
      sidx = (vs >> 1) & 1;
      sub = 2 * (vs >> 2) + (vs & 1);
    } else {
      const int n0 = vs * 32;
      sidx = 0;
      if (a.n_seg > 1 && n0 >= a.seg[1].col0) sidx = 1;
      if (a.n_seg > 2 && n0 >= a.seg[2].col0) sidx = 2;
      sub = (n0 - (sidx == 0 ? a.seg[0].col0 : (sidx == 1 ? a.seg[1].col0 : a.seg[2].col0))) >> 5;
    }
    const bf16 *wseg = (const bf16 *)(sidx == 0 ? a.seg[0].w : (sidx == 1 ? a.seg[1].w : a.seg[2].w));
    const int seg_rows = sidx == 0 ? a.seg[0].n_rows : (sidx == 1 ? a.seg[1].n_rows : a.seg[2].n_rows);
    sub = min(max(sub, 0), ((seg_rows + 31) >> 5) - 1);
    wp[i] = wseg + ((size_t)sub * kb_total + b0) * 2048;
  }
  const bf16 *xg = (const bf16 *)a.x + ((size_t)b0 * 4 * mbt + (size_t)rg * MB) * 1024;
  const unsigned lane_off = lane * 16;   // bases are scalar

  RowScale<NT, kWideRows> scale;
  if (a.n_splits == 1) scale.issue(a, rg * kWideRows);

  f32x16 acc[NBW][MBW];
#pragma unroll
  for (int i = 0; i < NBW; ++i)
#pragma unroll
    for (int m = 0; m < MBW; ++m)
#pragma unroll
      for (int e = 0; e < 16; ++e) acc[i][m][e] = 0.f;

  typedef unsigned int u32x4 __attribute__((ext_vector_type(4)));   // native vector: stays in registers
  bf16x8 w[2][4][NBW], xf[2][2 * MBW];
  u32x4 xr[XV];
  auto load_x1 = [&](int i, int c) {   // fragment i of this wavefront's share of chunk c
    const int f = wave * XV + i, j = f / (MB * 2), r = f % (MB * 2);
    xr[i] = *(const u32x4 *)((const char *)(xg + ((size_t)(c * 4 + j) * mbt * 2 + r) * 512) + lane_off);
  };
  auto store_x1 = [&](int i, int buf) { *(u32x4 *)(lds + buf * BUF + (wave * XV + i) * 1024 + lane * 16) = xr[i]; };
  auto load_w1 = [&](int set, int t, int i, int c) {
    const bf16x8 *p = (const bf16x8 *)((const char *)(wp[i] + (size_t)c * 2048 + 512 * t) + lane_off);
    w[set][t][i] = APART ? __builtin_nontemporal_load(p) : *p;   // no hint where other wavefronts or the other row group read it too
  };
  auto read_x1 = [&](int slot, int t, int buf, int m) {
    xf[slot][m] = *(const bf16x8 *)(lds + buf * BUF + (t * MB * 2 + wr * MBW * 2 + m) * 1024 + lane * 16);
  };
  constexpr int NR = 2 * MBW, NM = 2 * MBW * NBW, NG = NM / 2;   // operand reads, MFMAs and groups per step
  // One step (16 reduction elements): multiplies the operands in slot t & 1 and, spread over its
  // groups, reads the next step's operands (READ), writes the next chunk's activations to LDS (SX),
  // requests those of the chunk after it (LX) and refills the weight registers it has used (LW).
  auto step = [&](auto set_c, auto t_c, int nbuf, auto read_c, auto lw_c, int cw, auto sx_c, auto lx_c, int cx) {
    constexpr int set = decltype(set_c)::value, t = decltype(t_c)::value;
    constexpr bool READ = decltype(read_c)::value, LW = decltype(lw_c)::value, SX = decltype(sx_c)::value, LX = decltype(lx_c)::value;
#pragma unroll
    for (int q = 0; q < NG; ++q) {
      if (READ)
#pragma unroll
        for (int m = q * NR / NG; m < (q + 1) * NR / NG; ++m) read_x1((t + 1) & 1, (t + 1) & 3, nbuf, m);
      if (SX)
#pragma unroll
        for (int i = q * XV / NG; i < (q + 1) * XV / NG; ++i) store_x1(i, set ^ 1);
      if (LX)
#pragma unroll
        for (int i = q * XV / NG; i < (q + 1) * XV / NG; ++i) load_x1(i, min(cx, n - 1));
#pragma unroll
      for (int u = 0; u < 2; ++u) {   // consecutive instructions go to different accumulators
        const int e = q * 2 + u, p = e / (MBW * NBW), i = (e / MBW) % NBW, m = e % MBW;
        acc[i][m] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(xf[t & 1][2 * m + p], w[set][t][i], acc[i][m], 0, 0, 0);
      }
      if (LW && q >= NG - NBW) load_w1(set, t, q - (NG - NBW), min(cw, n - 1));
      __builtin_amdgcn_sched_barrier(0);
    }
  };
  // One chunk in LDS buffer / weight set `set`.  MORE: the next chunk (in xr) goes to the other buffer; FAR: chunk
  // c + 2 is requested.
  auto chunk = [&](auto set_c, int c, auto more_c, auto far_c) {
    constexpr bool MORE = decltype(more_c)::value, FAR = decltype(far_c)::value;
    constexpr int set = decltype(set_c)::value;
    step(IC<set>{}, IC<0>{}, set, IC<1>{}, IC<FAR>{}, c + 2, IC<MORE>{}, IC<0>{}, 0);
    step(IC<set>{}, IC<1>{}, set, IC<1>{}, IC<FAR>{}, c + 2, IC<0>{}, IC<FAR>{}, c + 2);
    step(IC<set>{}, IC<2>{}, set, IC<1>{}, IC<FAR>{}, c + 2, IC<0>{}, IC<0>{}, 0);
    if (MORE) __syncthreads();
    step(IC<set>{}, IC<3>{}, set ^ 1, IC<MORE>{}, IC<FAR>{}, c + 2, IC<0>{}, IC<0>{}, 0);
  };

#pragma unroll
  for (int i = 0; i < XV; ++i) load_x1(i, 0);
#pragma unroll
  for (int t = 0; t < 4; ++t)
#pragma unroll
    for (int i = 0; i < NBW; ++i) load_w1(0, t, i, 0);
  __builtin_amdgcn_sched_barrier(0);
#pragma unroll
  for (int i = 0; i < XV; ++i) store_x1(i, 0);
#pragma unroll
  for (int i = 0; i < XV; ++i) load_x1(i, min(1, n - 1));
  __builtin_amdgcn_sched_barrier(0);
#pragma unroll
  for (int t = 0; t < 4; ++t)
#pragma unroll
    for (int i = 0; i < NBW; ++i) load_w1(1, t, i, min(1, n - 1));
  __builtin_amdgcn_sched_barrier(0);
  if (a.n_splits == 1) scale.finish(a, rg * kWideRows, s_tmp, s_rs);   // ends with a barrier
  else __syncthreads();
#pragma unroll
  for (int m = 0; m < NR; ++m) read_x1(0, 0, 0, m);
  int c = 0;
  for (; c + 3 < n; c += 2) {
    chunk(IC<0>{}, c, IC<1>{}, IC<1>{});
    chunk(IC<1>{}, c + 1, IC<1>{}, IC<1>{});
  }
  // 1 to 3 chunks are left; surplus requests repeat the last one, into registers and an LDS buffer that nothing reads.  (As
  // three-way code without surplus the accumulators were in different registers on each way: 504 registers and
  // copies between them, now 338; 120 for eight wavefronts.)
  chunk(IC<0>{}, c, IC<1>{}, IC<1>{});
  if (c + 1 < n) chunk(IC<1>{}, c + 1, IC<1>{}, IC<0>{});
  if (c + 2 < n) chunk(IC<0>{}, c + 2, IC<0>{}, IC<0>{});

  if (a.n_splits > 1) {
    // partial tiles [split][128-column tile][row][128]; k_gemm_finish adds them up
    const int n_t128 = (a.n_total + 127) / 128;
#pragma unroll
    for (int i = 0; i < NBW; ++i) {
      const int col = ((tile * WC + wc) * NBW + i) * 32;
      if (col >= a.n_total) continue;   // wave-uniform
      float *o = a.part + ((size_t)split * n_t128 + (col >> 7)) * a.rows_pad * 128 + (col & 127) + ln;
#pragma unroll
      for (int m = 0; m < MBW; ++m)
#pragma unroll
        for (int e = 0; e < 16; ++e) {
          const int r = rg * kWideRows + (wr * MBW + m) * 32 + 8 * (e >> 2) + 4 * g + (e & 3);
          if (r < a.rows) o[(size_t)r * 128] = acc[i][m][e];
        }
    }
    return;
  }

  // one split: the epilogue, 32 rows at a time through LDS
  float *tl = (float *)lds;
  TileEpilogue<EPI == EPI_HEAD ? EPI_PLAIN : EPI, TN, NT, 32> epi;
#pragma unroll
  for (int mb = 0; mb < MB; ++mb) {
    const int row0 = rg * kWideRows + mb * 32;
    if (row0 >= a.rows) break;
    if constexpr (EPI != EPI_HEAD) epi.preload(a, tile, row0);
    __syncthreads();   // the last operand reads / the previous block's tile are done with
    if (wr == mb / MBW) {
#pragma unroll
      for (int i = 0; i < NBW; ++i)
#pragma unroll
        for (int e = 0; e < 16; ++e)
          tl[(8 * (e >> 2) + 4 * g + (e & 3)) * LD + (wc * NBW + i) * 32 + ln] = acc[i][mb % MBW][e];
    }
    __syncthreads();
    if constexpr (EPI == EPI_HEAD)
      head_rows<TN, NT, 32, LD>(a, tl, s_rs + mb * 32, tile * TN, min((tile + 1) * TN, a.n_total), tile, row0);
    else
      epi.apply(a, [&](int lr, int cc) { return *(const f32x4 *)(tl + lr * LD + cc); }, s_rs + mb * 32, tile, row0);
  }
}

// Adds up the split-K partial tiles of 32 rows x 128 columns, in ascending split order, and runs the
// epilogue on them.  Memory round trips set its time (about 5 us over the launch boundary): every
// partial of a thread, the epilogue's own operands and the sums of squares are requested at once.
template <int EPI>
__global__ __launch_bounds__(256) void k_gemm_finish(GemmArgs a) {
  constexpr int TN = 128, RB = 32, LD = TN + 4, PER = RB * TN / 4 / 256;
  __shared__ __attribute__((aligned(16))) float tl[RB * LD];
  __shared__ float s_tmp[256], s_rs[RB];
  const int tile = blockIdx.x, row0 = blockIdx.y * RB, tid = threadIdx.x;
  TileEpilogue<EPI, TN, 256, RB> epi;
  RowScale<256, RB> scale;
  const float *p0 = a.part + ((size_t)tile * a.rows_pad + row0) * TN + (size_t)tid * 4;
  const size_t stride = (size_t)((a.n_total + 127) / 128) * a.rows_pad * TN;
  constexpr int SG = 4;                // splits requested side by side
  f32x4 sum[PER];
  f32x4 v[SG][PER];
  auto request = [&](int s0) {
#pragma unroll
    for (int q = 0; q < SG; ++q)
#pragma unroll
      for (int u = 0; u < PER; ++u)
        if (s0 + q < a.n_splits) v[q][u] = *(const f32x4 *)(p0 + (size_t)(s0 + q) * stride + u * 1024);
  };
  request(0);
  scale.issue(a, row0);
  epi.preload(a, tile, row0);
#pragma unroll
  for (int u = 0; u < PER; ++u) sum[u] = v[0][u];
  for (int s0 = 0; s0 < a.n_splits; s0 += SG) {
    if (s0 > 0) request(s0);
#pragma unroll
    for (int q = 0; q < SG; ++q)
      if (s0 + q > 0 && s0 + q < a.n_splits)
#pragma unroll
        for (int u = 0; u < PER; ++u) sum[u] += v[q][u];
  }
#pragma unroll
  for (int u = 0; u < PER; ++u) {
    const int idx = tid + u * 256;
    *(f32x4 *)(tl + (idx >> 5) * LD + (idx & 31) * 4) = sum[u];
  }
  scale.finish(a, row0, s_tmp, s_rs);   // ends with a barrier
  epi.apply(a, [&](int lr, int cc) { return *(const f32x4 *)(tl + lr * LD + cc); }, s_rs, tile, row0);
}

template <int EPI>
static void dispatch_wide(hipStream_t st, GemmArgs a) {
  const int n_rg = (a.rows + kWideRows - 1) / kWideRows, wide = EPI == EPI_HEAD || a.tile_n == 256;   // the LM head always
  const int n_tiles = (a.n_total + (wide ? 255 : 127)) / (wide ? 256 : 128);
  const dim3 grid((n_tiles * a.n_splits + 7) / 8 * 8 * n_rg);
  a.tiles_inv = wide_tiles_inv(n_tiles);
  if constexpr (EPI == EPI_HEAD) {
    if (wide_apart(a.n_total, a.k, a.rows)) hipLaunchKernelGGL((k_gemm_wide<1, 4, 4, 2, EPI, true>), dim3(n_tiles, n_rg), dim3(256), 0, st, a);
    else hipLaunchKernelGGL((k_gemm_wide<1, 4, 4, 2, EPI, false>), grid, dim3(256), 0, st, a);
  } else if (wide) {
    hipLaunchKernelGGL((k_gemm_wide<1, 4, 4, 2, EPI, false>), grid, dim3(256), 0, st, a);
  } else {
    hipLaunchKernelGGL((k_gemm_wide<2, 4, 2, 1, EPI, false>), grid, dim3(512), 0, st, a);
  }
  if constexpr (EPI != EPI_HEAD) {
    if (a.n_splits > 1)
      hipLaunchKernelGGL(k_gemm_finish<EPI>, dim3((a.n_total + 127) / 128, (a.rows + 31) / 32), dim3(256), 0, st, a);
  }
}

void launch_gemm_wide(hipStream_t st, const GemmArgs &a) {
  switch (a.epi) {
    case EPI_QKV: dispatch_wide<EPI_QKV>(st, a); break;
    case EPI_RESID: dispatch_wide<EPI_RESID>(st, a); break;
    case EPI_SWIGLU: dispatch_wide<EPI_SWIGLU>(st, a); break;
    case EPI_PLAIN: dispatch_wide<EPI_PLAIN>(st, a); break;
    default: dispatch_wide<EPI_HEAD>(st, a); break;
  }
}

}  // namespace ts
