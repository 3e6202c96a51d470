// Element-wise half of the matmul epilogues, on a block of RB rows x TN columns of the reduced fp32
// product: rotary embedding + KV append, residual + next operand + norm statistics, SiLU * up, plain
// store, LM-head statistics.  Used by k_gemm_stream, k_gemm_wide and k_gemm_finish (which adds up split-K
// partial tiles); the LM-head statistics (head_rows) by k_gemm_head too.  The layer kernel finishes its tiles in
// gemm_epilogue.hpp, with the same arithmetic written for its layout: a change here belongs there too.
#pragma once

#include <type_traits>

#include "device_util.hpp"

namespace ts {

template <int N>
using IC = std::integral_constant<int, N>;

// Sums of squares of ROWS rows from the per-(tile, row) entries, in two parts: issue() requests the
// first entries, finish() adds everything up (ascending tiles within a thread, threads in ascending
// order) and leaves 1/rms in s_rs[0 .. ROWS).  s_tmp: NT floats.  Ends with a barrier.
template <int NT, int ROWS, int PRE = 16>
struct RowScale {
  static constexpr int Q = NT / ROWS;   // threads per row; each requests PRE entries ahead
  float x[PRE];
  __device__ __forceinline__ void issue(const GemmArgs &a, int row0) {
    if (a.ss_in == nullptr) return;
    const int r = min(row0 + (int)threadIdx.x % ROWS, a.rows_pad - 1), q = threadIdx.x / ROWS;
#pragma unroll
    for (int u = 0; u < PRE; ++u) x[u] = a.ss_in[(size_t)min(q + Q * u, a.ss_tiles - 1) * a.rows_pad + r];
  }
  // partial(): this thread's entries; total(), after a barrier: the threads of a row.  The caller synchronises
  // the workgroup before s_rs is read.
  __device__ __forceinline__ void partial(const GemmArgs &a, int row0, float *s_tmp) {
    if (a.ss_in == nullptr) return;
    const int tid = threadIdx.x, r = min(row0 + tid % ROWS, a.rows_pad - 1), q = tid / ROWS;
    float v = 0.f;
#pragma unroll
    for (int u = 0; u < PRE; ++u) v += (q + Q * u < a.ss_tiles) ? x[u] : 0.f;
    for (int t = q + Q * PRE; t < a.ss_tiles; t += Q) v += a.ss_in[(size_t)t * a.rows_pad + r];
    s_tmp[tid] = v;
  }
  __device__ __forceinline__ void total(const GemmArgs &a, const float *s_tmp, float *s_rs) {
    const int tid = threadIdx.x;
    if (tid < ROWS) {
      float ss = 0.f;
      if (a.ss_in != nullptr) {
#pragma unroll
        for (int q = 0; q < Q; ++q) ss += s_tmp[q * ROWS + tid];
      }
      s_rs[tid] = a.ss_in != nullptr ? 1.0f / sqrtf(ss / (float)a.k + a.eps) : 1.0f;
    }
  }
  __device__ __forceinline__ void finish(const GemmArgs &a, int row0, float *s_tmp, float *s_rs) {
    partial(a, row0, s_tmp);
    __syncthreads();
    total(a, s_tmp, s_rs);
    __syncthreads();
  }
};

// Columns that one entry of the per-(tile, row) sums of squares covers.
template <int TN>
constexpr int ss_width() { return TN < 128 ? TN : 128; }

// Column of the concatenated q, k, v projections that local column c of a QKV tile holds.  A tile of up to d
// columns takes TN / 2 consecutive rotation pairs of one head: their low features, then their high ones; a
// wider one whole heads.
template <int TN>
__device__ __forceinline__ int qkv_column(int tile, int c, int d) {
  const int half = d >> 1;
  if (TN / 2 > half) return tile * TN + c;
  const int up = c >= TN / 2, p = tile * (TN / 2) + (up ? c - TN / 2 : c), head = p / half;
  return head * d + p - head * half + (up ? half : 0);
}

// NT threads work on rows row0 .. row0 + RB - 1 and on columns tile * TN .. + TN of the product.
// preload() issues the loads that do not depend on the product (rotary tables; residual rows and the
// next norm weight), so that they travel together with whatever the caller still waits for; apply()
// reads the product through red(local row, local column) -> 4 consecutive columns.  rs[lr] is 1/rms
// of row row0 + lr of the matmul's input.
template <int EPI, int TN, int NT, int RB>
struct TileEpilogue {
  static constexpr int QG = TN / 8;                          // threads per row: 4 rotation pairs each
  static constexpr int QKV_PASSES = (RB * QG + NT - 1) / NT;
  static constexpr int LPR = TN / 4, RPP = NT / LPR;         // threads per row (4 columns each), rows per pass
  static constexpr int RES_PASSES = (RB + RPP - 1) / RPP;
  static constexpr int UB = RES_PASSES < 8 ? RES_PASSES : 8;
  f32x4 pre_a[EPI == EPI_QKV ? QKV_PASSES : (EPI == EPI_RESID ? UB : 1)];
  f32x4 pre_b[EPI == EPI_QKV ? QKV_PASSES : 1];
  bf16x4 pre_nw;

  // Where 4 rotation pairs sit: columns c_lo .. and c_lo + off .. of the tile, features j .. and
  // j + d/2 .. of head `head` of the concatenated q, k, v heads.
  struct Pair { int c_lo, off, j, head; };
  static __device__ __forceinline__ Pair qkv_pair(int tile, int qi, int d) {
    const int half = d >> 1, p = tile * (TN / 2) + qi * 4, head = p / half, j = p - head * half;
    if (TN / 2 <= half) return {qi * 4, TN / 2, j, head};
    return {(head * d - tile * TN) + j, half, j, head};
  }

  __device__ __forceinline__ void preload(const GemmArgs &a, int tile, int row0) {
    const int tid = threadIdx.x;
    if constexpr (EPI == EPI_QKV) {
      const int half = a.head_dim >> 1;
#pragma unroll
      for (int u = 0; u < QKV_PASSES; ++u) {
        const int t = tid + u * NT, r = min(row0 + t / QG, a.rows - 1), qi = t % QG;
        const int j = qkv_pair(tile, qi, a.head_dim).j;
        pre_a[u] = *(const f32x4 *)(a.cos_t + r * half + j);
        pre_b[u] = *(const f32x4 *)(a.sin_t + r * half + j);
      }
    } else if constexpr (EPI == EPI_RESID) {
      const int col = tile * TN + (tid % LPR) * 4, colc = col < a.n_total ? col : 0;
      pre_nw = *(const bf16x4 *)((const bf16 *)a.next_norm_w + colc);
#pragma unroll
      for (int u = 0; u < UB; ++u)
        pre_a[u] = *(const f32x4 *)(a.x_resid + (size_t)min(row0 + tid / LPR + u * RPP, a.rows - 1) * a.n_total + colc);
    }
  }

  template <class Red>
  __device__ __forceinline__ void apply(const GemmArgs &a, Red red, const float *rs, int tile, int row0) {
    const int tid = threadIdx.x;
    const int mb_count = a.rows_pad >> 5;
    if constexpr (EPI == EPI_QKV) {
      // thread = (row, 4 rotation pairs); a tile holds pairs of one or two heads, or whole heads (qkv_column), where
      // q and k have a norm of their own always the latter
      const int d = a.head_dim, half = d >> 1;
      const int n_q = a.n_q_heads, n_kv = a.n_kv_heads;
      const bool paged = a.kv.page_table != nullptr;          // uniform: the contiguous cache's addresses stay plain arithmetic
#pragma unroll
      for (int u = 0; u < QKV_PASSES; ++u) {
        const int t = tid + u * NT;
        const int lr = t / QG, qi = t - lr * QG, r = row0 + lr;
        const Pair pr = qkv_pair(tile, qi, d);
        const int j = pr.j, hh = pr.head;                     // first pair, head (q heads, k heads, v heads)
        const int col = hh * d + j;                           // global column
        const bool live = lr < RB && r < a.rows && col < a.n_total;
        const int lrc = lr < RB ? lr : 0;
        const float rsc = live ? rs[lrc] : 0.f;
        f32x4 lo = red(lrc, pr.c_lo) * rsc, hi = red(lrc, pr.c_lo + pr.off) * rsc;
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
      // every 128 columns of the product (all of them where the tile is narrower): the gate columns,
      // then as many matching up columns
      constexpr int FQ = TN / 8, H = TN < 128 ? TN / 2 : 64;   // groups of 4 features per row, gate columns in a row
      for (int t = tid; t < RB * FQ; t += NT) {
        const int lr = t / FQ, f = (t % FQ) * 4, r = row0 + lr;
        const int feat = tile * (TN / 2) + f, c = (f / H) * 2 * H + f % H;
        if (r >= a.rows || feat >= a.ffn) continue;
        const float rsc = rs[lr];
        const f32x4 gt = red(lr, c) * rsc, up = red(lr, c + H) * rsc;
        bf16x4 hi, lo;
#pragma unroll
        for (int e = 0; e < 4; ++e) {
          const float o = gt[e] / (1.0f + expf(-gt[e])) * up[e];
          hi[e] = (bf16)o;
          lo[e] = (bf16)(o - (float)hi[e]);
        }
        bf16 *dst = (bf16 *)a.act_out;   // operand layout of the down projection (K = ffn)
        *(bf16x4 *)(dst + ol_offset(r, feat, 0, mb_count)) = hi;
        *(bf16x4 *)(dst + ol_offset(r, feat, 1, mb_count)) = lo;
      }
    } else if constexpr (EPI == EPI_PLAIN) {
      // ---- y = (x W^T) / rms + bias, written as it is (the adapter on the exported features)
      for (int t = tid; t < RB * LPR; t += NT) {
        const int lr = t / LPR, c = (t % LPR) * 4, r = row0 + lr, col = tile * TN + c;
        if (r >= a.rows || col >= a.n_total) continue;
        f32x4 v = red(lr, c) * rs[lr];
        if (a.bias != nullptr) v += *(const f32x4 *)(a.bias + col);
        *(f32x4 *)(a.out + (size_t)r * a.n_total + col) = v;
      }
    } else {
      // ---- EPI_RESID: x += y; per-row sum of squares of the new x over ss_width columns, which
      // ss_width / 4 consecutive lanes hold
      constexpr int SSW = ss_width<TN>(), SSL = SSW / 4;
      const int c = (tid % LPR) * 4, col = tile * TN + c, r0 = tid / LPR;
      const bool col_ok = col < a.n_total;
      const int colc = col_ok ? col : 0;
      float *ssp = a.ss_part + (size_t)((tile * TN + c) / SSW) * a.rows_pad;
      const bf16x4 nw = pre_nw;
#pragma unroll 1
      for (int ub = 0; ub < RES_PASSES; ub += UB) {
        // the residual rows of UB passes at once (the first UB were fetched by preload)
        f32x4 xv[UB];
#pragma unroll
        for (int u = 0; u < UB; ++u) xv[u] = pre_a[u];
        if (ub > 0) {
#pragma unroll
          for (int u = 0; u < UB; ++u)
            xv[u] = *(const f32x4 *)(a.x_resid + (size_t)min(row0 + r0 + (ub + u) * RPP, a.rows - 1) * a.n_total + colc);
        }
        float ss[UB];
#pragma unroll
        for (int u = 0; u < UB; ++u) {
          const int lr = r0 + (ub + u) * RPP, r = row0 + lr;
          ss[u] = 0.f;
          if (lr < RB && r < a.rows && col_ok) {
            const f32x4 v = xv[u] + red(lr, c);
            *(f32x4 *)(a.x_resid_out + (size_t)r * a.n_total + col) = v;
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
            *(bf16x4 *)(dst + ol_offset(r, col, 0, mb_count)) = hi;
            *(bf16x4 *)(dst + ol_offset(r, col, 1, mb_count)) = lo;
          }
        }
        // the UB row sums are reduced side by side, so the exchanges of one hide behind the others'
#pragma unroll
        for (int o = SSL / 2; o > 0; o >>= 1)
#pragma unroll
          for (int u = 0; u < UB; ++u) ss[u] += __shfl_xor(ss[u], o, 64);
#pragma unroll
        for (int u = 0; u < UB; ++u) {
          const int lr = r0 + (ub + u) * RPP, r = row0 + lr;
          if (tid % SSL == 0 && lr < RB && r < a.rows && col_ok) ssp[r] = ss[u];   // read by the next matmul
        }
      }
    }
  }
};

// e^x for x <= 0: hardware exp2 with the rounding error of x * log2(e) put back (within 2 ulp, where
// exp2(x * log2(e)) alone would be off by |x| / 2 ulp).  Below -104 the result is 0; from -2.4e38 on x * log2(e)
// would overflow and its rounding error be a NaN.  A NaN stays one.  Confidences against fp64 on the same logits
// (2400 nodes, 151936 columns): 1.07e-7 rms relative, as with expf and a running maximum.
__device__ __forceinline__ float exp_neg(float x) {
  x = x < -104.f ? -104.f : x;
  const float L = 1.44269504088896341f, Llo = 1.92596299112661e-8f;
  const float t = x * L;
  const float r = __builtin_fmaf(x, Llo, __builtin_fmaf(x, L, -t));
  const float e = __builtin_amdgcn_exp2f(t);
  return __builtin_fmaf(e, r * 0.693147180559945f, e);
}

// LM head: rows row0 .. row0 + RB - 1 of the logits of columns col0 .. col_end - 1 (TN at most), in LDS as
// tl[lr * LD + column], to (largest logit, its column, second largest, sum of exp, sum of exp * distance) per
// row, entry `entry` of it; TN / 16 threads scan a row, 16 columns each.  rs[lr]: 1/rms of the row's input.
template <int TN, int NT, int RB, int LD>
__device__ __forceinline__ void head_rows(const GemmArgs &a, const float *tl, const float *rs, int col0, int col_end,
                                          int entry, int row0) {
  constexpr int PARTS = TN / 16, RP = NT / PARTS;
  const int tid = threadIdx.x, srow = tid / PARTS, part = tid % PARTS;
  if (a.debug_logits != nullptr) {   // materialised logits: consecutive threads write consecutive columns
    for (int i = tid; i < RB * TN; i += NT) {
      const int lr = i / TN, c = i % TN, r = row0 + lr, col = col0 + c;
      if (r < a.rows && col < col_end) a.debug_logits[(size_t)r * a.n_total + col] = tl[lr * LD + c] * rs[lr];
    }
  }
#pragma unroll
  for (int rp = 0; rp < RB; rp += RP) {
    const int lr = rp + srow, r = row0 + lr;
    const bool in = lr < RB;
    const float rsc = in && r < a.rows ? rs[lr] : 1.0f;
    const int cbase = col0 + part * 16;
    Top2 t = top2_empty();
    if (in) {
      f32x4 v[4];
#pragma unroll
      for (int q = 0; q < 4; ++q) v[q] = *(const f32x4 *)(tl + lr * LD + part * 16 + 4 * q);
#pragma unroll
      for (int c = 0; c < 16; ++c) {   // ascending: the lowest column of equal maxima stays
        const float x = cbase + c < col_end ? v[c >> 2][c & 3] * rsc : -INFINITY;
        v[c >> 2][c & 3] = x;
        const bool up = x > t.l1;
        t.l2 = up ? t.l1 : fmaxf(t.l2, x);   // a NaN is neither
        t.idx = up ? cbase + c : t.idx;
        t.l1 = up ? x : t.l1;
      }
      if (t.l1 != -INFINITY) {
#pragma unroll
        for (int c = 0; c < 16; ++c) {
          const float x = v[c >> 2][c & 3], dd = x - t.l1;
          if (x != -INFINITY && cbase + c != t.idx) {
            const float e = exp_neg(dd);
            t.s += e;
            t.t = __builtin_fmaf(e, dd, t.t);
          }
        }
        t.s += 1.f;   // the largest itself: x - l1 would be a NaN for +inf.  Last: the small terms add up first
      }
    }
#pragma unroll
    for (int o = 1; o < PARTS; o <<= 1) t = top2_merge(t, top2_shfl_xor(t, o));
    if (part == 0 && in && r < a.rows) {
      const size_t o = (size_t)r * a.hs.n_tiles + entry;
      a.hs.l1[o] = t.l1; a.hs.l2[o] = t.l2; a.hs.sumexp[o] = t.s; a.hs.ent[o] = t.t; a.hs.idx[o] = t.idx;
    }
  }
}

}  // namespace ts
