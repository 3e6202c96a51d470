// LM head over at most 128 rows: weight-streaming small-M matmul on the matrix cores (bf16 weights, fp32
// accumulate) with the vocabulary statistics fused in, and the one-time repack of the weights.
//
//   y[r][n] = rstd[r] * sum_k X[r][k] * W[n][k]        r < rows_pad <= 128
//
// At these row counts the product is bound by streaming W from HBM once, so the layout serves
// the W stream.  W is read from the PACKED copy made once by k_pack_weights: for every 32-row
// sub-tile s and 64-deep k block kb, one contiguous 4 KB block holding the four MFMA B-operand
// fragments of that (s, kb) in lane order.  A wavefront owns one sub-tile (32 output columns) and
// pulls its blocks straight from global memory into registers — every load instruction reads
// 1 KB contiguous (8 whole 128-byte lines), a sub-tile's k range is one contiguous run, W never
// passes through LDS and is never re-read.  (Reading row-major W with the same operand layout
// touches 32 rows x 32 bytes per instruction and reaches ~75 % of the contiguous rate.)
//
// The activation panel X (at most 128 rows; more rows: kernels_gemm_wide.hip) is what the four wavefronts of a workgroup share.
// It arrives as two bf16 panels, a high part and a low part (hi = round(v), lo = round(v - hi),
// written once by whichever kernel produced the activation — splitting it here would repeat the
// conversion in every one of the hundreds of workgroups and costs more issue slots than the
// MFMAs).  Each W fragment is multiplied by both parts, so the activations keep ~16 significant
// bits, the pass is a smooth function of its inputs, and W is still read exactly once.  X is
// stored in the operand layout (device_util.hpp: 1 KB fragments in consumption order), staged
// through LDS in chunks of KC reduction elements, double buffered, by plain contiguous copies;
// the 16-byte operand reads are conflict free.
// RMSNorm is fused around the matmul: the producer stores x * w_norm (the per-column weight) as
// the operand panels, and the per-row 1/rms multiplies the reduced sums in the epilogue here.
//
// MFMA 32x32x16: A = X fragment (row = activation row), B = W fragment (column = output
// column), so accumulator register e of lane (ln, g) holds y[8*(e/4) + 4*g + e%4][ln].  The k
// index inside a 64 block is permuted (lane half g owns k = 32g + 8j + 0..7 at MFMA step j)
// identically for both operands.
//
// A workgroup takes up to 128 output columns at a time over the whole reduction and leaves, per row, (largest
// logit, its column, second largest, sum of exp) of them; the probabilities are never materialised.
//
// Two workgroups run per CU (at most 256 registers a lane).  Over at most 32 rows a vocabulary of more tiles than that is
// shared out evenly in sub-tiles of 32: every workgroup makes the same number of passes over runs of neighbouring
// sub-tiles, and the chip has no last wave that is a third full (1187 tiles on 512 places).  151936 columns over 9
// rows of 1024 83 -> 66 us (one workgroup a CU and a tile each before), over one row of 4096 211 -> 206.  Over 60 rows the
// panel, drawn once per pass, outweighs that (256 -> 295 us): a tile each.  Over 65 to 128 rows the LDS delivers all it can (an
// operand fragment feeds one matrix instruction), and two workgroups a CU still beat the wide kernel's 256-column tiles, of
// which 594 leave a last wave a third full: 151936 x 2048 247 -> 215 us, 151936 x 4096 383 -> 367.
#include "gemm_tile.hpp"

namespace ts {

template <int MB, int KC, int DEPTH>
__global__ __launch_bounds__(256, MB == 2 ? 1 : 2) void k_gemm_head(GemmArgs a) {
  constexpr int KB = KC / 64;                 // 64-deep k blocks per chunk
  constexpr int FRAGS = KB * 4 * MB * 2;      // 1 KB operand fragments per chunk (operand layout)
  constexpr int BUF = FRAGS * 1024;           // one LDS stage
  constexpr int XV = FRAGS / 4;               // fragments (16 bytes per lane) per wavefront per chunk
  constexpr int EPI_BYTES = MB * 32 * (kGemmTileN + 4) * 4;   // the epilogue's fp32 tile reuses the stages
  constexpr int LDS_BYTES = 2 * BUF > EPI_BYTES ? 2 * BUF : EPI_BYTES;
  __shared__ __attribute__((aligned(1024))) unsigned char lds[LDS_BYTES];
  __shared__ float s_rs[kMaxRows];   // 1/rms of the rows of the matmul's input
  __shared__ float s_tmp[4 * kMaxRows];

  const int tid = threadIdx.x, lane = tid & 63;
  // scalar: the address of this wavefront's packed run stays in scalar registers
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int ln = lane & 31, g = lane >> 5;
  const int n_chunks = a.k / KC;   // whole, and a multiple of DEPTH (plan_head, launch_gemm_head)
  // Workgroups that run side by side start at different depths of their k range (and wrap
  // around), so that they do not all walk the memory channels in lockstep.  The order of the
  // additions is still a fixed function of the workgroup.
  const int rot = (int)((blockIdx.x * 11u) % (unsigned)n_chunks);
  auto rc = [&](int c) { const int cc = c + rot; return cc >= n_chunks ? cc - n_chunks : cc; };

  // ---- this workgroup's sub-tiles, and its passes over at most four of them
  const int n_sub = (a.seg[0].n_rows + 31) >> 5, n_pass = MB == 1 ? a.n_splits : 1;
  const int s_begin = (int)((long long)n_sub * blockIdx.x / gridDim.x), s_count = (int)((long long)n_sub * (blockIdx.x + 1) / gridDim.x) - s_begin;

  // ---- X staging: the chunk is a contiguous run of FRAGS fragments in operand layout; this
  // wavefront copies fragments wave*XV .. wave*XV + XV-1, 16 bytes per lane each
  const bf16 *xg = (const bf16 *)a.x + (size_t)wave * XV * 512 + lane * 8;

  // 1/rms of every row of the matmul's INPUT, requested ahead of everything else and finished with the
  // prologue: 64 or 128 entries a row come in one round trip; fetched after the stream they cost 4 us.
  RowScale<256, MB * 32> scale;
  scale.issue(a, 0);
  __builtin_amdgcn_sched_barrier(0);

  f32x16 acc[MB];
  const bf16 *wrow;   // this wavefront's packed sub-tile

  // The streaming loop is kept free of branches around loads: a load behind a branch makes the
  // wait-count analysis assume it may not have been issued, which turns every wait into "drain
  // everything" and serialises the stream.
  //
  // Per chunk c:
  //   1. X registers (chunk c+1, fetched during chunk c-1) -> LDS stage (c+1)&1
  //   2. issue the X loads of chunk c+2
  //   3. per 64-deep block: 4 x MB x 2 MFMAs on W set c % DEPTH, then refill that block of the
  //      set with chunk c+DEPTH — a W load has DEPTH chunks of compute to arrive, and a wavefront
  //      keeps about DEPTH * KC/64 * 4 KB in flight.  (HBM latency under load is several
  //      microseconds; at 8 wavefronts per CU it takes this much to keep the stream full.)
  //   4. workgroup barrier
  // sched_barrier pins the load issue points; the compiler would otherwise sink every load to
  // just before its first use and expose the whole memory latency once per chunk.
  bf16x8 w[DEPTH][KB][4];
  typedef unsigned int u32x4 __attribute__((ext_vector_type(4)));   // native vector: stays in registers
  // One register stage of the panel.  Loads come back in order, so the wait for it is also one for every
  // weight load before it.
  u32x4 xr[XV];

  auto load_w_block = [&](int set, int c, int kb) {
    const int k = rc(c) * KC + kb * 64;
    const bf16 *p = wrow + (size_t)(k >> 6) * 2048;
#pragma unroll
    for (int j = 0; j < 4; ++j) w[set][kb][j] = __builtin_nontemporal_load((const bf16x8 *)(p + 512 * j));
  };
  auto load_x = [&](int c) {
    const bf16 *src = xg + (size_t)rc(c) * FRAGS * 512;
#pragma unroll
    for (int i = 0; i < XV; ++i) xr[i] = *(const u32x4 *)(src + i * 512);
  };
  auto store_x = [&](int buf) {    // -> LDS stage buf (chunk parity)
    unsigned char *dst = lds + buf * BUF + (wave * XV) * 1024 + lane * 16;
#pragma unroll
    for (int i = 0; i < XV; ++i) *(u32x4 *)(dst + i * 1024) = xr[i];
  };
  // One chunk of MFMAs, software pipelined: step t = (k block, j) needs four A fragments
  // (row block 0/1 x hi/lo); they are read from LDS two steps ahead into a 2-slot register ring,
  // so the LDS latency hides behind the previous step's four MFMAs.  After the last step of a k
  // block, that block of the W set is refilled from chunk `c_next` (if LOADW).
  bf16x8 xf[2][2 * MB];
  auto read_frags = [&](int slot, int t, int buf) {
    const unsigned char *xp = lds + buf * BUF + (size_t)(t * MB * 2) * 1024 + lane * 16;   // t = kb*4 + j
#pragma unroll
    for (int mb = 0; mb < MB; ++mb) {
      xf[slot][2 * mb] = *(const bf16x8 *)(xp + (mb * 2) * 1024);
      xf[slot][2 * mb + 1] = *(const bf16x8 *)(xp + (mb * 2 + 1) * 1024);
    }
  };
  auto compute_chunk = [&](int set, int buf, int c_next, bool loadw) {
    constexpr int T = 4 * KB;
    read_frags(0, 0, buf);
    read_frags(1, 1, buf);
#pragma unroll
    for (int t = 0; t < T; ++t) {
      const int kb = t >> 2, j = t & 3;
      // high parts of every row block, then the low parts: a matrix instruction that adds to the
      // result of the one just before it would have to wait for it
#pragma unroll
      for (int mb = 0; mb < MB; ++mb)
        acc[mb] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(xf[t & 1][2 * mb], w[set][kb][j], acc[mb], 0, 0, 0);
#pragma unroll
      for (int mb = 0; mb < MB; ++mb)
        acc[mb] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(xf[t & 1][2 * mb + 1], w[set][kb][j], acc[mb], 0, 0, 0);
      if (t + 2 < T) read_frags(t & 1, t + 2, buf);
      if (j == 3 && loadw) load_w_block(set, c_next, kb);
      __builtin_amdgcn_sched_barrier(0);
    }
  };

  for (int pass = 0; pass < n_pass; ++pass) {
    const int s0 = s_begin + s_count * pass / n_pass, s1 = s_begin + s_count * (pass + 1) / n_pass;
    // one to four sub-tiles (head_passes in plan.hpp); wavefronts beyond them take the last one again (its lines are
    // on their way already), and their columns are not looked at
    wrow = (const bf16 *)a.seg[0].w + (size_t)min(s0 + wave, s1 - 1) * (a.k >> 6) * 2048 + lane * 8;
#pragma unroll
    for (int mb = 0; mb < MB; ++mb)
#pragma unroll
      for (int e = 0; e < 16; ++e) acc[mb][e] = 0.f;
    if (pass > 0) __syncthreads();   // the previous pass has read its logits
    // The prologue issues its loads in the order
    // the steady state does (X of a chunk before the W refill of the same step), so the wait
    // counts merged at the loop head are the steady-state ones.
    load_x(0);
#pragma unroll
    for (int kb = 0; kb < KB; ++kb) load_w_block(0, 0, kb);
    __builtin_amdgcn_sched_barrier(0);
    store_x(0);
    load_x(1);
    __builtin_amdgcn_sched_barrier(0);
#pragma unroll
    for (int d = 1; d < DEPTH; ++d)
#pragma unroll
      for (int kb = 0; kb < KB; ++kb) load_w_block(d, d, kb);
    __builtin_amdgcn_sched_barrier(0);
    if (pass == 0) scale.finish(a, 0, s_tmp, s_rs);   // ends with a barrier
    else __syncthreads();
    int c0 = 0;
    for (; c0 + DEPTH < n_chunks; c0 += DEPTH) {
#pragma unroll
      for (int d = 0; d < DEPTH; ++d) {
        store_x((d + 1) & 1);                                    // chunk c0+d+1
        load_x(min(c0 + d + 2, n_chunks - 1));   // clamped, never a branch
        __builtin_amdgcn_sched_barrier(0);
        compute_chunk(d, d & 1, c0 + d + DEPTH, true);
        __syncthreads();
      }
    }
    // last DEPTH chunks: nothing left to fetch from W
#pragma unroll
    for (int d = 0; d < DEPTH; ++d) {
      if (d + 1 < DEPTH) store_x((d + 1) & 1);
      if (d + 2 < DEPTH) load_x(c0 + d + 2);
      __builtin_amdgcn_sched_barrier(0);
      compute_chunk(d, d & 1, 0, false);
      if (d + 1 < DEPTH) __syncthreads();
    }

    // ---- per row, this tile's 128 logits to (l1, column, l2, sum exp)
    float *tl = (float *)lds;
    __syncthreads();   // every wavefront is done reading the last X stage
#pragma unroll
    for (int mb = 0; mb < MB; ++mb)
#pragma unroll
      for (int e = 0; e < 16; ++e) tl[(mb * 32 + 8 * (e >> 2) + 4 * g + (e & 3)) * (kGemmTileN + 4) + wave * 32 + ln] = acc[mb][e];
    __syncthreads();
    head_rows<kGemmTileN, 256, MB * 32, kGemmTileN + 4>(a, tl, s_rs, s0 * 32, min(s1 * 32, a.n_total), (int)blockIdx.x * n_pass + pass, 0);
  }
}

// One-time repack of a row-major [n_rows, k] bf16 matrix into the layout above.  One thread per
// 16-byte piece of the output: piece (s, kb, j, lane) = W[32 s + (lane & 31)][64 kb + 32 (lane >> 5) + 8 j .. + 8].
__global__ __launch_bounds__(256) void k_pack_weights(const bf16 *w, int n_rows, int k, uint4 *out,
                                                      size_t n_pieces) {
  const size_t p = (size_t)blockIdx.x * 256 + threadIdx.x;
  if (p >= n_pieces) return;
  const int lane = (int)(p & 63), j = (int)((p >> 6) & 3);
  const size_t blk = p >> 8;
  const int kblocks = k >> 6;
  const int kb = (int)(blk % kblocks);
  const int s = (int)(blk / kblocks);
  const int row = 32 * s + (lane & 31);
  const int col = 64 * kb + 32 * (lane >> 5) + 8 * j;
  uint4 v = make_uint4(0, 0, 0, 0);
  if (row < n_rows) v = *(const uint4 *)(w + (size_t)row * k + col);
  out[p] = v;
}

size_t packed_weight_bytes(int n_rows, int k) { return (size_t)((n_rows + 31) / 32) * (k / 64) * 4096; }

void launch_pack_weights(hipStream_t st, const void *w, int n_rows, int k, void *out) {
  const size_t n_pieces = packed_weight_bytes(n_rows, k) / 16;
  hipLaunchKernelGGL(k_pack_weights, dim3((unsigned)((n_pieces + 255) / 256)), dim3(256), 0, st,
                     (const bf16 *)w, n_rows, k, (uint4 *)out, n_pieces);
}

void launch_gemm_head(hipStream_t st, const GemmArgs &a) {
  const dim3 grid(a.n_tiles / a.n_splits), block(256);
  if (a.rows_pad == 128) hipLaunchKernelGGL((k_gemm_head<4, 64, 4>), grid, block, 0, st, a);
  else if (a.rows_pad == 32) hipLaunchKernelGGL((k_gemm_head<1, 128, 4>), grid, block, 0, st, a);
  else if (a.k % 512 == 0) hipLaunchKernelGGL((k_gemm_head<2, 128, 4>), grid, block, 0, st, a);
  else hipLaunchKernelGGL((k_gemm_head<2, 128, 2>), grid, block, 0, st, a);
}

}  // namespace ts
