// Epilogue of the layer kernel's matmuls (kernels_layer.hip): four wavefronts, a 32-column sub-tile each.
#pragma once

#include "gemm_tile.hpp"

namespace ts {

// 1/rms of every row of a matmul's INPUT, from the per-tile sums of squares its producer left.
// rstd_load only ISSUES loads (wavefront q of the workgroup takes tiles q, q+4, ...; a lane takes
// rows lane, lane+64, ...) and is called before the weight stream starts, so that nothing waits
// for them; rstd_finish, called after the stream, adds them up (plus the entries beyond the first
// 32: more than 4096 columns in entries of 128) and combines the wavefronts' sums through LDS.  The
// order of the additions is fixed, so the result does not depend on scheduling.
constexpr int kLayerWaves = 4, kLayerThreads = 64 * kLayerWaves;
template <int MB>
__device__ __forceinline__ void rstd_load(const GemmArgs &a, float (&x)[(MB + 1) / 2][8]) {
  constexpr int Q = kLayerWaves, RI = (MB + 1) / 2;
  const int q = threadIdx.x >> 6, r0 = threadIdx.x & 63;
  if (a.ss_in == nullptr) return;
#pragma unroll
  for (int i = 0; i < RI; ++i) {
    const int r = min(r0 + 64 * i, a.rows_pad - 1);
#pragma unroll
    for (int u = 0; u < 8; ++u) x[i][u] = a.ss_in[(size_t)min(q + Q * u, a.ss_tiles - 1) * a.rows_pad + r];
  }
}

// s_rsp: kLayerWaves * kMaxRows floats of LDS.  The caller synchronises the workgroup before s_rs is read.
template <int MB>
__device__ __forceinline__ void rstd_finish(const GemmArgs &a, const float (&x)[(MB + 1) / 2][8], float *s_rsp,
                                            float *s_rs) {
  constexpr int Q = kLayerWaves, RI = (MB + 1) / 2;
  const int q = threadIdx.x >> 6, r0 = threadIdx.x & 63;
  if (a.ss_in != nullptr) {
#pragma unroll
    for (int i = 0; i < RI; ++i) {
      float v = 0.f;
#pragma unroll
      for (int u = 0; u < 8; ++u) v += (q + Q * u < a.ss_tiles) ? x[i][u] : 0.f;
      const int r = min(r0 + 64 * i, a.rows_pad - 1);
      for (int t = q + Q * 8; t < a.ss_tiles; t += Q) v += a.ss_in[(size_t)t * a.rows_pad + r];
      s_rsp[q * kMaxRows + r0 + 64 * i] = v;
    }
  }
  __syncthreads();
  for (int r = threadIdx.x; r < a.rows; r += kLayerThreads) {
    float ss = 0.f;
#pragma unroll
    for (int qq = 0; qq < Q; ++qq) ss += s_rsp[qq * kMaxRows + r];
    s_rs[r] = a.ss_in != nullptr ? 1.0f / sqrtf(ss / (float)a.k + a.eps) : 1.0f;
  }
}

template <int N>
struct SplitGroup {
  static constexpr int value = N;
};

// Epilogue of one (tile, split).  A wavefront owns a 32-column sub-tile of the tile:
// acc[mb][e] of lane (ln, g) of wavefront `wave` holds y[mb*32 + 8*(e/4) + 4*g + e%4][wave*32 + ln].
// The reduced fp32 tile goes through LDS: at least MB*32*(TN+4)*4 bytes, free for reuse (every wavefront has
// passed a barrier after its last operand read).  s_rs: 1/rms per input row.  What a later phase of the same
// launch reads (residual stream, operand panels, sums of squares) is written through to memory.
template <int MB, int EPI>
__device__ __forceinline__ void gemm_epilogue(const GemmArgs &a, f32x16 (&acc)[MB], unsigned char *lds,
                                              int *s_last, const float *s_rs, int tile, int split) {
  constexpr int TN = kLayerWaves * 32, NT = kLayerThreads;
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int ln = lane & 31, g = lane >> 5;
  // ---- hand the tile to the epilogue, as an fp32 tile in LDS.  One split: straight from the
  // accumulators.  Several splits: write-through partial tiles part[split][tile][row][TN] + a
  // counter per tile; only the last workgroup to arrive goes on.
  constexpr int EPI_LD = TN + 4;       // floats per row of the LDS tile
  float *tl = (float *)lds;
  const bool single = a.n_splits == 1;
  const size_t tile_elems = (size_t)a.rows_pad * TN;
  __syncthreads();   // every wavefront is done reading the last X stage
  if (!single) {
    float *o = a.part + ((size_t)split * a.n_tiles + tile) * tile_elems + wave * 32 + ln;
#pragma unroll
    for (int mb = 0; mb < MB; ++mb)
#pragma unroll
      for (int e = 0; e < 16; ++e) {
        const int r = mb * 32 + 8 * (e >> 2) + 4 * g + (e & 3);
        if (r < a.rows) st_agent(o + (size_t)r * TN, acc[mb][e]);
      }
    if (!publish_then_count(&a.counters[tile], a.n_splits, s_last)) return;
  }

  // Loads of the epilogue that do not depend on the reduced tile (rotary tables; residual rows and
  // the next norm weight).  Issued together with the loads of the partial tiles: a memory round
  // trip costs more than everything else the epilogue does, so they must not follow each other.
  constexpr int QKV_PASSES = MB * 32 * (TN / 8) / NT;
  constexpr int RES_LPR = TN / 4, RES_RPP = NT / RES_LPR, RES_PASSES = MB * 32 / RES_RPP;
  constexpr int RES_UB = RES_PASSES < 8 ? RES_PASSES : 8;
  f32x4 pre_a[EPI == EPI_QKV ? QKV_PASSES : (EPI == EPI_RESID ? RES_UB : 1)];
  f32x4 pre_b[EPI == EPI_QKV ? QKV_PASSES : 1];
  bf16x4 pre_nw;

  // -- loads that do not depend on the tile
  if constexpr (EPI == EPI_QKV) {
    const int half = a.head_dim >> 1;
#pragma unroll
    for (int u = 0; u < QKV_PASSES; ++u) {
      const int t = tid + u * NT, r = min(t / (TN / 8), a.rows - 1), qi = t % (TN / 8);
      const int j = qi * 4 - ((qi * 4) / half) * half;
      pre_a[u] = *(const f32x4 *)(a.cos_t + r * half + j);
      pre_b[u] = *(const f32x4 *)(a.sin_t + r * half + j);
    }
  } else if constexpr (EPI == EPI_RESID) {
    const int col = tile * TN + (tid % RES_LPR) * 4, colc = col < a.n_total ? col : 0;
    pre_nw = *(const bf16x4 *)((const bf16 *)a.next_norm_w + colc);
#pragma unroll
    for (int u = 0; u < RES_UB; ++u)
      pre_a[u] = *(const f32x4 *)(a.x_resid + (size_t)min(tid / RES_LPR + u * RES_RPP, a.rows - 1) * a.n_total + colc);
  }
  // -- the reduced tile into LDS
  if (single) {
#pragma unroll
    for (int mb = 0; mb < MB; ++mb)
#pragma unroll
      for (int e = 0; e < 16; ++e)
        tl[(mb * 32 + 8 * (e >> 2) + 4 * g + (e & 3)) * EPI_LD + wave * 32 + ln] = acc[mb][e];
  } else {
    // Last workgroup of the tile: sum the splits, in ascending order.  The partial tiles were
    // written through to memory (st_agent) by workgroups anywhere on the chip and are read here
    // with plain vector loads, which may be served by this XCD's L2.  That is correct because a
    // line of the partial buffer cannot be in this L2 from before it was written: every launch
    // starts with the invalidation of the L2s that makes a kernel see its predecessors' results
    // at all on this multi-XCD chip, and inside one launch a partial line is read only here, by
    // the one workgroup that combines its tile, after the counter says all of it is written (a
    // launch that runs several matmuls gives each its own partial region for the same reason).
    // Agent-scope loads would not need that argument, but they exist only up to 8 bytes and,
    // measured, cost 0.15 ms per pass here.
    // Every load of up to SG splits (UB vectors each) is in flight before the first addition: the
    // reduction then costs one or two memory round trips, not one per pair of splits — it is the
    // longest link of the serial chain that ends a matmul.
    constexpr int PER = MB * 32 * (TN / 4) / NT;   // 4-column vectors per thread
    constexpr int UB = PER < 4 ? PER : 4;
    const float *p0 = a.part + (size_t)tile * tile_elems + (size_t)tid * 4;
    const size_t split_stride = (size_t)a.n_tiles * tile_elems;
    auto reduce_groups = [&](auto sg_c) {
      constexpr int SG = decltype(sg_c)::value;
#pragma unroll 1
      for (int ub = 0; ub < PER; ub += UB) {
        f32x4 sum[UB];
#pragma unroll 1
        for (int s0 = 0; s0 < a.n_splits; s0 += SG) {
          f32x4 v[SG][UB];
#pragma unroll
          for (int q = 0; q < SG; ++q) {
            const float *ps = p0 + (size_t)min(s0 + q, a.n_splits - 1) * split_stride;
#pragma unroll
            for (int u = 0; u < UB; ++u) v[q][u] = *(const f32x4 *)(ps + (size_t)(ub + u) * NT * 4);
          }
#pragma unroll
          for (int q = 0; q < SG; ++q)
#pragma unroll
            for (int u = 0; u < UB; ++u) {
              if (s0 + q == 0) sum[u] = v[q][u];
              else if (s0 + q < a.n_splits) sum[u] += v[q][u];
            }
        }
#pragma unroll
        for (int u = 0; u < UB; ++u) {
          const int idx = tid + (ub + u) * NT, r = idx / (TN / 4), c = (idx % (TN / 4)) * 4;
          *(f32x4 *)(tl + r * EPI_LD + c) = sum[u];
        }
      }
    };
    // the group size is the number of splits itself where that is small: no load is wasted on a
    // clamped duplicate (a 256-row partial tile is 128 KB per split)
    switch (a.n_splits) {
      case 2: reduce_groups(SplitGroup<2>{}); break;
      case 3: reduce_groups(SplitGroup<3>{}); break;
      case 4: reduce_groups(SplitGroup<4>{}); break;
      case 5: reduce_groups(SplitGroup<5>{}); break;
      case 6: reduce_groups(SplitGroup<6>{}); break;
      case 7: reduce_groups(SplitGroup<7>{}); break;
      default: reduce_groups(SplitGroup<8>{}); break;
    }
  }
  __syncthreads();
  auto reduced4 = [&](int r, int c) {   // 4 consecutive columns of row r of the reduced tile
    return *(const f32x4 *)(tl + r * EPI_LD + c);
  };

  if constexpr (EPI == EPI_QKV) {
    // a tile holds whole heads; thread = (row, 4 rotation pairs)
    const int d = a.head_dim, half = d >> 1;
    const int n_q = a.n_q_heads, n_kv = a.n_kv_heads;
    const bool paged = a.kv.page_table != nullptr;          // uniform: the contiguous cache's addresses stay plain arithmetic
    constexpr int quads = TN / 8;                           // 4-pair groups per row
#pragma unroll
    for (int u = 0; u < QKV_PASSES; ++u) {
      const int t = tid + u * NT;
      const int r = t / quads, qi = t - r * quads;
      const int hl = (qi * 4) / half, j = qi * 4 - hl * half;   // head within the tile, first pair
      const int c_lo = hl * d + j;                          // tile-local column of the low elements
      const int col = tile * TN + c_lo;                     // global column
      const bool live = r < a.rows && col < a.n_total;
      const int hh = col / d;                               // global head index (q heads, k heads, v heads)
      const float rsc = live ? s_rs[r] : 0.f;
      f32x4 lo = reduced4(r, c_lo) * rsc, hi = reduced4(r, c_lo + half) * rsc;
      if (a.q_norm_w != nullptr) {
        // RMSNorm of a query / key head over its d features: the half / 4 consecutive lanes that hold
        // the head add their sums of squares (every lane takes part: no early exit above)
        float ss = lo[0] * lo[0] + lo[1] * lo[1] + lo[2] * lo[2] + lo[3] * lo[3] + hi[0] * hi[0] + hi[1] * hi[1] +
                   hi[2] * hi[2] + hi[3] * hi[3];
        for (int o = 1; o < half / 4; o <<= 1) ss += __shfl_xor(ss, o, 64);
        if (live && hh < n_q + n_kv) {
          const float rn = 1.0f / sqrtf(ss / (float)d + a.eps);
          const bf16 *nw = (const bf16 *)(hh < n_q ? a.q_norm_w : a.k_norm_w);
          const bf16x4 wl = *(const bf16x4 *)(nw + j), wh = *(const bf16x4 *)(nw + j + half);
#pragma unroll
          for (int e = 0; e < 4; ++e) { lo[e] *= rn * (float)wl[e]; hi[e] *= rn * (float)wh[e]; }
        }
      }
      if (!live) continue;
      const int b = r / a.n_nodes, node = r - b * a.n_nodes;
      const int slot = a.ctx.v[b] + node;
      if (hh < n_q + n_kv) {
        const f32x4 rl = lo * pre_a[u] - hi * pre_b[u], rh = hi * pre_a[u] + lo * pre_b[u];
        lo = rl; hi = rh;
      }
      *(f32x4 *)(a.qkv_f32 + (size_t)r * a.n_total + col) = lo;
      *(f32x4 *)(a.qkv_f32 + (size_t)r * a.n_total + col + half) = hi;
      if (hh < n_q) {
        // matrix-core operand of the context attention: q * log2(e) / sqrt(d) as bf16 hi + lo, so
        // that the scores come out of the MFMA ready for exp2
        const float qs = 1.44269504088896f / sqrtf((float)d);
        bf16x4 lh, ll, hh4, hl4;
#pragma unroll
        for (int e = 0; e < 4; ++e) {
          const float ql_ = lo[e] * qs, qh_ = hi[e] * qs;
          lh[e] = (bf16)ql_; ll[e] = (bf16)(ql_ - (float)lh[e]);
          hh4[e] = (bf16)qh_; hl4[e] = (bf16)(qh_ - (float)hh4[e]);
        }
        bf16 *qo = (bf16 *)a.q_out + (size_t)r * n_q * d + col;
        *(bf16x4 *)qo = lh;
        *(bf16x4 *)(qo + a.q_panel) = ll;
        *(bf16x4 *)(qo + half) = hh4;
        *(bf16x4 *)(qo + half + a.q_panel) = hl4;
      }
      if (hh >= n_q && hh < n_q + n_kv) {
        bf16 *kc = (bf16 *)a.k_cache + (paged ? a.kv.k_row(b, hh - n_q, slot)
                                             : (((size_t)b * n_kv + (hh - n_q)) * a.kv.capacity + slot) * d);
        bf16x4 l4, h4;
#pragma unroll
        for (int e = 0; e < 4; ++e) { l4[e] = (bf16)lo[e]; h4[e] = (bf16)hi[e]; }
        *(bf16x4 *)(kc + j) = l4;
        *(bf16x4 *)(kc + j + half) = h4;
      } else if (hh >= n_q + n_kv) {
        bf16 *vc = (bf16 *)a.v_cache + (paged ? a.kv.v_col(b, hh - n_q - n_kv, slot)
                                             : ((size_t)b * n_kv + (hh - n_q - n_kv)) * d * a.kv.capacity + slot);
        const size_t vs = paged ? (size_t)kKvPage : (size_t)a.kv.capacity;
#pragma unroll
        for (int e = 0; e < 4; ++e) {
          vc[(size_t)(j + e) * vs] = (bf16)lo[e];
          vc[(size_t)(j + e + half) * vs] = (bf16)hi[e];
        }
      }
    }
  } else if constexpr (EPI == EPI_SWIGLU) {
    // columns [0, TN/2) of the tile are gate, [TN/2, TN) the matching up columns
    constexpr int FQ = TN / 8;   // float4 groups of features per row (TN/2 gate + TN/2 up columns)
    for (int t = tid; t < MB * 32 * FQ; t += NT) {
      const int r = t / FQ, f = (t % FQ) * 4;
      const int feat = tile * (TN / 2) + f;
      if (r >= a.rows || feat >= a.ffn) continue;
      const float rsc = s_rs[r];
      const f32x4 gt = reduced4(r, f) * rsc, up = reduced4(r, TN / 2 + f) * rsc;
      bf16x4 hi, lo;
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        const float o = gt[e] / (1.0f + expf(-gt[e])) * up[e];
        hi[e] = (bf16)o;
        lo[e] = (bf16)(o - (float)hi[e]);
      }
      bf16 *dst = (bf16 *)a.act_out;   // operand layout of the down projection (K = ffn)
      st_agent_bf16x4(dst + ol_offset(r, feat, 0, MB), hi);
      st_agent_bf16x4(dst + ol_offset(r, feat, 1, MB), lo);
    }
  } else {
    // ---- EPI_RESID: x += y; per-row sum of squares of the new x over this tile's columns.
    // TN/4 consecutive lanes (4 columns each) cover one row of the tile.
    constexpr int LPR = RES_LPR, RPP = RES_RPP;   // lanes per row, rows per pass
    constexpr int PASSES = RES_PASSES, UB = RES_UB;
    float *ssp = a.ss_part + (size_t)tile * a.rows_pad;
    const int c = (tid % LPR) * 4, col = tile * TN + c, r0 = tid / LPR;
    const bool col_ok = col < a.n_total;
    const int colc = col_ok ? col : 0;
    const bf16x4 nw = pre_nw;
#pragma unroll 1
    for (int ub = 0; ub < PASSES; ub += UB) {
      // the residual rows of UB passes at once (the first UB were fetched before the reduction)
      f32x4 xv[UB];
#pragma unroll
      for (int u = 0; u < UB; ++u) xv[u] = pre_a[u];
      if (ub > 0) {
#pragma unroll
        for (int u = 0; u < UB; ++u)
          xv[u] = *(const f32x4 *)(a.x_resid + (size_t)min(r0 + (ub + u) * RPP, a.rows - 1) * a.n_total + colc);
      }
      float ss[UB];
#pragma unroll
      for (int u = 0; u < UB; ++u) {
        const int r = r0 + (ub + u) * RPP;
        ss[u] = 0.f;
        if (r < a.rows && col_ok) {
          const f32x4 v = xv[u] + reduced4(r, c);
          st_agent_f32x4(a.x_resid_out + (size_t)r * a.n_total + col, v);
          ss[u] = v[0] * v[0] + v[1] * v[1] + v[2] * v[2] + v[3] * v[3];
          // operand of the next matmul: x * (next RMSNorm weight), as bf16 hi + lo
          bf16x4 hi, lo;
#pragma unroll
          for (int e = 0; e < 4; ++e) {
            const float o = v[e] * (float)nw[e];
            hi[e] = (bf16)o;
            lo[e] = (bf16)(o - (float)hi[e]);
          }
          bf16 *dst = (bf16 *)a.xw_out;   // operand layout of the next matmul (K = hidden)
          st_agent_bf16x4(dst + ol_offset(r, col, 0, MB), hi);
          st_agent_bf16x4(dst + ol_offset(r, col, 1, MB), lo);
        }
      }
      // the UB row sums are reduced side by side, so the exchanges of one hide behind the others'
#pragma unroll
      for (int o = LPR / 2; o > 0; o >>= 1)
#pragma unroll
        for (int u = 0; u < UB; ++u) ss[u] += __shfl_xor(ss[u], o, 64);
#pragma unroll
      for (int u = 0; u < UB; ++u) {
        const int r = r0 + (ub + u) * RPP;
        if (tid % LPR == 0 && r < a.rows) st_agent(ssp + r, ss[u]);   // read by the next matmul
      }
    }
  }
}

}  // namespace ts
