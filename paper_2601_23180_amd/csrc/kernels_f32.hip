// fp32 models: one matmul kernel with the layer's element-wise steps around it, so that a layer is five launches
// (QKV, attention, O, gate + up, down).  Such a pass is launches and memory round trips, nothing else: the toy model
// (256 wide, 2 layers, 9 nodes) takes 2 us of bytes; with norms, residuals, activation and rotation as launches of their own it
// took 94 us, now 65.
#include "device_util.hpp"

namespace ts {

// Sums over lanes of 2 N values a lane: lanes with bit O keep the upper N, the others the lower N, and so on, until every
// lane holds one value, summed over the lanes that differ from it in the bits used.
template <int N, int O, int M>
__device__ __forceinline__ void fold_lanes(float (&v)[M], int lane) {
  const bool up = (lane & O) != 0;
#pragma unroll
  for (int i = 0; i < N; ++i) v[i] = (up ? v[i + N] : v[i]) + __shfl_xor(up ? v[i] : v[i + N], O, 64);
  if constexpr (N > 1) fold_lanes<N / 2, O / 2>(v, lane);
}

// A wavefront takes two output columns - the two of a rotation pair (QKV), a gate column and its up column (SWIGLU),
// else neighbours - over R rows, its lanes the reduction, V elements at a time.  All loads of 2 (V = 4) or 8 steps, 512 reduction
// elements, are requested together and without a branch around any; the lanes' sums meet in a folding exchange, after
// which lane l holds row l / 4, column l / 2 % 2.  Rows are normalised on the way: x * w / rms(x), the sums of squares
// from the same loads, 1/rms on the finished sum.  9 rows, us, before (one column a wavefront, single elements, 8 rows
// at a time, the epilogue a launch of its own) -> now: 256 x 512 with the residual 4.9 + 2.9 -> 4.2, 1024 x 256 with the
// activation 5.4 + 2.3 -> 4.7, 512 x 256 with rotation and append 5.2 + 2.5 -> 5.1, 4096 x 256 11.1 -> 5.7.
// V = 4 needs k % 4 == 0 and matrices, rows and norm weight at multiples of 16 bytes (launch_gemm_f32).
template <int V, int R, int EPI>
__global__ __launch_bounds__(64) void k_gemm_f32(GemmArgs a) {
  typedef float vec __attribute__((ext_vector_type(V)));
  constexpr int U = 8 / V;
  const int lane = threadIdx.x, pair = blockIdx.x, r0 = blockIdx.y * R;
  const int row = r0 + (lane >> 2), c = (lane >> 1) & 1;   // of the finished sum that this lane holds
  const bool mine = (lane >> 2) < R && row < a.rows && (lane & 1) == 0;
  const int rowc = min(row, a.rows - 1);
  // ---- the two columns, and what the epilogue reads
  int col[2];
  const float *w[2];
  const int half = EPI == EPI_QKV ? a.head_dim >> 1 : 0, head = EPI == EPI_QKV ? pair / half : 0, j = EPI == EPI_QKV ? pair - head * half : 0;
  if constexpr (EPI == EPI_QKV) {
    col[0] = head * a.head_dim + j;
    col[1] = col[0] + half;
  } else if constexpr (EPI == EPI_SWIGLU) {
    col[0] = pair;
    col[1] = a.ffn + pair;
  } else {
    col[0] = 2 * pair;
    col[1] = min(2 * pair + 1, a.n_total - 1);
  }
#pragma unroll
  for (int i = 0; i < 2; ++i) {
    const void *m = a.seg[0].w;
    int at = a.seg[0].col0;
    if (a.n_seg > 1 && col[i] >= a.seg[1].col0) { m = a.seg[1].w; at = a.seg[1].col0; }
    if (a.n_seg > 2 && col[i] >= a.seg[2].col0) { m = a.seg[2].w; at = a.seg[2].col0; }
    w[i] = (const float *)m + (size_t)(col[i] - at) * a.k;
  }
  const int my_col = c ? col[1] : col[0];
  const bool live = mine && (EPI == EPI_QKV || EPI == EPI_SWIGLU || 2 * pair + c < a.n_total);
  float pre0 = 0.f, pre1 = 0.f;
  if constexpr (EPI == EPI_QKV) {
    pre0 = a.cos_t[rowc * half + j];
    pre1 = a.sin_t[rowc * half + j];
  } else if constexpr (EPI == EPI_RESID) {
    pre0 = a.x_resid[(size_t)rowc * a.n_total + my_col];
  } else if constexpr (EPI == EPI_PLAIN) {
    if (a.bias != nullptr) pre0 = a.bias[my_col];
  }

  const float *x[R];   // rows past the end repeat the last one; their sums are not stored
#pragma unroll
  for (int r = 0; r < R; ++r) x[r] = (const float *)a.x + (size_t)min(r0 + r, a.rows - 1) * a.k;
  const bool norm = a.norm_w != nullptr;   // uniform
  float v[32], ss[16];
#pragma unroll
  for (int i = 0; i < 32; ++i) v[i] = 0.f;
#pragma unroll
  for (int i = 0; i < 16; ++i) ss[i] = 0.f;
  for (int k0 = lane * V; k0 < a.k; k0 += 64 * V * U) {
    vec wv[U][2], nv[U], xv[U][R];
#pragma unroll
    for (int u = 0; u < U; ++u) {
      const int k = min(k0 + 64 * V * u, a.k - V);
      wv[u][0] = *(const vec *)(w[0] + k);
      wv[u][1] = *(const vec *)(w[1] + k);
      nv[u] = norm ? *(const vec *)(a.norm_w + k) : vec(1.f);
#pragma unroll
      for (int r = 0; r < R; ++r) xv[u][r] = *(const vec *)(x[r] + k);
    }
#pragma unroll
    for (int u = 0; u < U; ++u) {
      if (k0 + 64 * V * u >= a.k) continue;
#pragma unroll
      for (int r = 0; r < R; ++r)
#pragma unroll
        for (int e = 0; e < V; ++e) {
          const float xe = xv[u][r][e], xn = xe * nv[u][e];
          v[2 * r] += xn * wv[u][0][e];
          v[2 * r + 1] += xn * wv[u][1][e];
          ss[r] += xe * xe;
        }
    }
  }
  // ---- the lanes' sums: half of the values go to the other half of the lanes, until every lane has one
  fold_lanes<16, 32>(v, lane);
  float y = v[0] + __shfl_xor(v[0], 1, 64);
  if (norm) {
    fold_lanes<8, 32>(ss, lane);
    ss[0] += __shfl_xor(ss[0], 2, 64);
    ss[0] += __shfl_xor(ss[0], 1, 64);
    y *= 1.0f / sqrtf(ss[0] / (float)a.k + a.eps);
  }
  const float other = __shfl_xor(y, 2, 64);   // the pair's other column

  if (!live) return;
  if constexpr (EPI == EPI_QKV) {
    const int n_q = a.n_q_heads, n_kv = a.n_kv_heads, d = a.head_dim, f = c ? j + half : j;
    if (head < n_q + n_kv) y = c ? y * pre0 + other * pre1 : y * pre0 - other * pre1;
    const int b = row / a.n_nodes, slot = a.ctx.v[b] + row - b * a.n_nodes;
    if (head < n_q) ((float *)a.q_out)[((size_t)row * n_q + head) * d + f] = y;
    else if (head < n_q + n_kv) ((float *)a.k_cache)[a.kv.k_row(b, head - n_q, slot) + f] = y;
    else ((float *)a.v_cache)[a.kv.v_col(b, head - n_q - n_kv, slot) + (size_t)f * a.kv.v_stride()] = y;
  } else if constexpr (EPI == EPI_SWIGLU) {
    if (c == 0) ((float *)a.act_out)[(size_t)row * a.ffn + pair] = y / (1.0f + expf(-y)) * other;
  } else if constexpr (EPI == EPI_RESID) {
    a.x_resid_out[(size_t)row * a.n_total + my_col] = pre0 + y;
  } else {
    a.out[(size_t)row * a.n_total + my_col] = y + pre0;
  }
}

template <int V, int R>
static void launch_gemm_f32_epi(hipStream_t st, const GemmArgs &a, int groups) {
  const dim3 grid(a.epi == EPI_QKV || a.epi == EPI_SWIGLU ? a.n_total / 2 : (a.n_total + 1) / 2, groups), block(64);
  switch (a.epi) {
    case EPI_QKV: hipLaunchKernelGGL((k_gemm_f32<V, R, EPI_QKV>), grid, block, 0, st, a); break;
    case EPI_RESID: hipLaunchKernelGGL((k_gemm_f32<V, R, EPI_RESID>), grid, block, 0, st, a); break;
    case EPI_SWIGLU: hipLaunchKernelGGL((k_gemm_f32<V, R, EPI_SWIGLU>), grid, block, 0, st, a); break;
    default: hipLaunchKernelGGL((k_gemm_f32<V, R, EPI_PLAIN>), grid, block, 0, st, a); break;
  }
}
template <int V>
static void launch_gemm_f32_rows(hipStream_t st, const GemmArgs &a) {
  // up to 16 rows a wavefront, shared out evenly: the matrix is read once per group of rows
  const int groups = (a.rows + 15) / 16, per = (a.rows + groups - 1) / groups;
  if (per <= 4) launch_gemm_f32_epi<V, 4>(st, a, groups);
  else if (per <= 8) launch_gemm_f32_epi<V, 8>(st, a, (a.rows + 7) / 8);
  else if (per <= 12) launch_gemm_f32_epi<V, 12>(st, a, (a.rows + 11) / 12);
  else launch_gemm_f32_epi<V, 16>(st, a, groups);
}

void launch_gemm_f32(hipStream_t st, const GemmArgs &a) {
  uintptr_t at = (uintptr_t)a.x | (uintptr_t)a.norm_w;
  for (int i = 0; i < a.n_seg; ++i) at |= (uintptr_t)a.seg[i].w;
  if (a.k % 4 == 0 && at % 16 == 0) launch_gemm_f32_rows<4>(st, a);
  else launch_gemm_f32_rows<1>(st, a);
}

// One workgroup per (row, head), for models with per-head norms: norm and rotation of q and k heads (pair (j, j + d/2)), q to
// the attention's operand, k and v to cache slot ctx_len + node (v transposed).
__global__ void k_qkv_epilogue_f32(GemmArgs a, const float *qkv) {
  __shared__ float s_sq[64];
  const int r = blockIdx.x, hh = blockIdx.y, j = threadIdx.x;   // head_dim / 2 threads
  const int d = a.head_dim, half = d >> 1, n_q = a.n_q_heads, n_kv = a.n_kv_heads;
  const size_t off = (size_t)r * a.n_total + (size_t)hh * d + j;
  float lo = qkv[off], hi = qkv[off + half];
  if (hh < n_q + n_kv) {   // RMSNorm over the head (uniform branch)
    s_sq[j] = lo * lo + hi * hi;
    __syncthreads();
    float ss = 0.f;
    for (int i = 0; i < half; ++i) ss += s_sq[i];           // ascending: the same order in every thread
    const float rn = 1.0f / sqrtf(ss / (float)d + a.eps);
    const float *nw = (const float *)(hh < n_q ? a.q_norm_w : a.k_norm_w);
    lo *= rn * nw[j];
    hi *= rn * nw[j + half];
  }
  const int b = r / a.n_nodes, slot = a.ctx.v[b] + r - b * a.n_nodes;
  if (hh < n_q + n_kv) {
    const float c = a.cos_t[r * half + j], s = a.sin_t[r * half + j];
    const float rl = lo * c - hi * s, rh = hi * c + lo * s;
    lo = rl; hi = rh;
  }
  if (hh < n_q) {
    float *q = (float *)a.q_out + ((size_t)r * n_q + hh) * d;
    q[j] = lo;
    q[j + half] = hi;
  } else if (hh < n_q + n_kv) {
    float *k = (float *)a.k_cache + a.kv.k_row(b, hh - n_q, slot);
    k[j] = lo;
    k[j + half] = hi;
  } else {
    float *v = (float *)a.v_cache + a.kv.v_col(b, hh - n_q - n_kv, slot);
    v[(size_t)j * a.kv.v_stride()] = lo;
    v[(size_t)(j + half) * a.kv.v_stride()] = hi;
  }
}

void launch_qkv_epilogue_f32(hipStream_t st, const GemmArgs &a, const float *qkv) {
  hipLaunchKernelGGL(k_qkv_epilogue_f32, dim3(a.rows, a.n_q_heads + 2 * a.n_kv_heads), dim3(a.head_dim / 2), 0, st, a, qkv);
}

__global__ __launch_bounds__(256) void k_norm_rows_f32(const float *x, const float *w, int hidden, float eps, float *out) {
  __shared__ float red[4];
  const float *xr = x + (size_t)blockIdx.x * hidden;
  float ss = 0.f;
  for (int i = threadIdx.x; i < hidden; i += 256) ss += xr[i] * xr[i];
  ss = block_sum<4>(ss, red);
  const float rstd = 1.0f / sqrtf(ss / (float)hidden + eps);
  for (int i = threadIdx.x; i < hidden; i += 256) out[(size_t)blockIdx.x * hidden + i] = xr[i] * rstd * w[i];
}

void launch_norm_rows_f32(hipStream_t st, const float *x, const float *w, int rows, int hidden, float eps, float *out) {
  hipLaunchKernelGGL(k_norm_rows_f32, dim3(rows), dim3(256), 0, st, x, w, hidden, eps, out);
}

}  // namespace ts
