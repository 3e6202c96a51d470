// Tree-masked grouped-query attention of the draft nodes over (context cache + draft nodes).
//
// Node i of sequence b attends to cache slots [0, ctx_len_b) and to every draft node j on its
// root path (bit j of anc[i]).  K is cached [slot][d]; V is cached transposed [d][slot] so that
// both products read matrix-core operands with 16-byte loads.
//
// bf16 path.  Context: one workgroup per (context split, kv head, sequence) streams the cached K/V — no
// mask is needed there, every context key is visible to every node.  The draft nodes (masked to each
// row's root path) are taken in fp32 on this pass's unrounded q/k/v projections: the cache gets bf16
// copies for later rounds, but the pass itself never reads them back.  Where they are evaluated is up to
// the host (AttnArgs::draft_mode): in blocks of 32 by workgroups of the same launch, or by the merge
// kernel, which combines all partials of a row in ascending order.
#include <float.h>

#include "device_util.hpp"

namespace ts {

// ------------------------------------------------------------------ fp32 path (small models)
// One workgroup per (row, query head).  Scores of all allowed keys go to LDS, a thread a key, then a plain
// two-pass softmax and the value sum, a thread per output feature and share of the keys (whole runs of 64).  Keys and values
// come in 16-byte pieces, 16 of them requested at once, the first ones with the query: memory round trips and the pieces'
// scattered lines set its time (9 rows, 4 heads, 137 keys: 8.4 us with one wavefront -> 7.6).
constexpr int kAttnF32MaxKeys = 12288, kAttnF32Threads = 256;

__global__ __launch_bounds__(kAttnF32Threads) void k_attn_f32(AttnArgs a) {
  extern __shared__ __attribute__((aligned(16))) float sc[];   // n_keys scores, then zeros up to a multiple of 64
  constexpr int NT = kAttnF32Threads, NW = NT / 64;
  __shared__ __attribute__((aligned(16))) float s_q[128], s_o[NT], s_red[NW];
  const int r = blockIdx.x, head = blockIdx.y, tid = threadIdx.x;
  const int d = a.head_dim, group = a.n_q_heads / a.n_kv_heads, kvh = head / group;   // d is 64 or 128
  const int b = r / a.n_nodes, node = r - b * a.n_nodes;
  const int ctx = a.ctx.v[b];
  const int n_keys = ctx + a.n_nodes;
  const AncMask mask = a.anc[r];
  const float *kc = (const float *)a.k_cache, *vc = (const float *)a.v_cache;   // slots through a.kv
  const int j = tid % d, share = tid / d, shares = NT / d;   // output feature, share of the keys
  const int per = ((n_keys + shares - 1) / shares + 63) / 64 * 64, k_begin = share * per, k_end = min(n_keys, k_begin + per);
  const size_t vj = (size_t)j * a.kv.v_stride();
  // the first key's first 64 features and the first 64 values are requested with the query and the mask
  f32x4 k0[16], v0[16];
  {
    const float *kr = kc + a.kv.k_row(b, kvh, min(tid, n_keys - 1));
    const f32x4 *vp = (const f32x4 *)(vc + a.kv.v_col(b, kvh, k_begin < k_end ? k_begin : 0) + vj);
    const float q = tid < d ? ((const float *)a.q)[((size_t)r * a.n_q_heads + head) * d + tid] : 0.f;
#pragma unroll
    for (int i = 0; i < 16; ++i) k0[i] = *(const f32x4 *)(kr + 4 * i);
#pragma unroll
    for (int i = 0; i < 16; ++i) v0[i] = vp[i];
    __builtin_amdgcn_sched_barrier(0);
    if (tid < d) s_q[tid] = q;
  }
  __syncthreads();
  const float scale = 1.0f / sqrtf((float)d);
  float mx = -INFINITY;
  for (int k = tid; k < n_keys; k += NT) {
    const bool ok = (k < ctx) || mask.has(k - ctx);
    float s = -INFINITY;
    if (ok) {
      const float *kr = kc + a.kv.k_row(b, kvh, k);
      float acc = 0.f;
      for (int j0 = 0; j0 < d; j0 += 64) {
        if (k >= NT || j0 > 0) {
#pragma unroll
          for (int i = 0; i < 16; ++i) k0[i] = *(const f32x4 *)(kr + j0 + 4 * i);
        }
#pragma unroll
        for (int i = 0; i < 16; ++i) {
          const f32x4 q4 = *(const f32x4 *)(s_q + j0 + 4 * i);
#pragma unroll
          for (int e = 0; e < 4; ++e) acc += q4[e] * k0[i][e];
        }
      }
      s = acc * scale;
    }
    sc[k] = s;
    mx = fmaxf(mx, s);
  }
  mx = wave_max(mx);
  if ((tid & 63) == 0) s_red[tid >> 6] = mx;
  __syncthreads();
#pragma unroll
  for (int w = 0; w < NW; ++w) mx = fmaxf(mx, s_red[w]);
  float sum = 0.f;
  for (int k = tid; k < (n_keys + 63) / 64 * 64; k += NT) {
    const float p = (k >= n_keys || sc[k] == -INFINITY) ? 0.f : expf(sc[k] - mx);
    sc[k] = p;
    sum += p;
  }
  sum = block_sum<NW>(sum, s_red);   // its barriers also publish sc
  float acc = 0.f;
  for (int k = k_begin; k < k_end; k += 64) {   // 64 slots from a multiple of 64 lie side by side inside the cache, paged or not
    if (k > k_begin) {
      const f32x4 *vp = (const f32x4 *)(vc + a.kv.v_col(b, kvh, k) + vj);
#pragma unroll
      for (int i = 0; i < 16; ++i) v0[i] = vp[i];
    }
    const int left = n_keys - k;   // slots past the last key hold no value: their weight is 0, and a NaN is not to meet it
#pragma unroll
    for (int i = 0; i < 16; ++i) {
      const f32x4 p4 = *(const f32x4 *)(sc + k + 4 * i);
#pragma unroll
      for (int e = 0; e < 4; ++e) acc += p4[e] * (4 * i + e < left ? v0[i][e] : 0.f);
    }
  }
  s_o[tid] = acc;
  __syncthreads();
  if (tid >= d) return;
  for (int s = 1; s < shares; ++s) acc += s_o[s * d + tid];
  ((float *)a.out)[((size_t)r * a.n_q_heads + head) * d + tid] = acc / sum;
}

void launch_attn_f32(hipStream_t st, const AttnArgs &a) {
  int max_keys = 0;
  for (int b = 0; b < a.batch; ++b) max_keys = max(max_keys, a.ctx.v[b] + a.n_nodes);
  hipLaunchKernelGGL(k_attn_f32, dim3(a.batch * a.n_nodes, a.n_q_heads), dim3(kAttnF32Threads),
                     (size_t)((max_keys + 63) / 64 * 64) * sizeof(float), st, a);
}

// ------------------------------------------------------------------ bf16 path
// KT = keys per LDS tile
template <int D, int KT>
struct AttnLds {
  static constexpr int kStrideK = D * 2 + 16;     // bytes per key row of the K tile
  static constexpr int kStrideV = KT * 2 + 8;     // bytes per feature row of the V^T tile
  static constexpr int kBytesK = KT * kStrideK;
  static constexpr int kBytesV = D * kStrideV;
  static constexpr int kBuf = kBytesK + kBytesV;  // one stage
};

typedef __attribute__((ext_vector_type(2))) float f32x2;
typedef __attribute__((ext_vector_type(2))) __bf16 bf16x2;
// Elements e and e + 1 of the high and the low part of a probability operand: one conversion for two values.
__device__ __forceinline__ void split_pair(f32x2 p, bf16x8 &hi, bf16x8 &lo, int e) {
  const bf16x2 h = __builtin_convertvector(p, bf16x2);
  const f32x2 rest = {p[0] - (float)h[0], p[1] - (float)h[1]};
  const bf16x2 l = __builtin_convertvector(rest, bf16x2);
  hi[e] = h[0]; hi[e + 1] = h[1];
  lo[e] = l[0]; lo[e + 1] = l[1];
}

// Maximum, in natural-log units, that a partial is stored with.  -inf marks a partial without keys, which the
// merge skips without reading it; one whose scores are all NaN (fmaxf drops them) or all -inf has to be
// added up all the same, so that the NaN in its sums reaches the row: it is stored with the lowest finite value.
__device__ __forceinline__ float stored_max(float m_log2) { return fmaxf(m_log2 * 0.693147180559945f, -FLT_MAX); }

// Softmax partial of 32 query rows (one wavefront) over the draft nodes 32 kb .. 32 kb + 31: S^T = K Q^T
// and O^T = V^T P^T with fp32 matrix instructions (32x32x2), operands straight from the projections.
// Lane (ln, g) holds features g D/2 .. of key / query row ln for the first product; the scores come out
// with keys 8q + 4g + r in register 4q + r, which is the order in which the second product takes them.
// 128 instructions of 64 cycles, 3.5 us, beside context workgroups that run longer.  Evaluated by the
// merge kernel, where every row fetches its ancestors' keys and values for itself, a chain of 128 nodes
// with 32 heads takes 44 us a layer; the plain merge takes 8.4, the launch before it 18.6 instead of 16.1.
// s_p: 32 x 32 floats of LDS of this wavefront.
template <int D>
__device__ void draft_partial(const AttnArgs &a, int kb, int kvh, int b, int row_block, size_t part_base, float *s_p) {
  const int lane = threadIdx.x & 63, ln = lane & 31, g = lane >> 5;
  const int M = a.n_nodes, group = a.n_q_heads / a.n_kv_heads, p_rows = group * M;
  const int prow = row_block * 32 + ln;
  if (row_block * 32 >= p_rows) return;   // wave-uniform
  const int pc = min(prow, p_rows - 1), al = pc / M, node = pc - al * M;
  const AncMask mask = a.anc[b * M + node];
  const uint32_t mine = (uint32_t)((kb < 2 ? mask.lo : mask.hi) >> (32 * (kb & 1)));   // ancestors in this block
  const size_t pi = part_base * p_rows + prow;
  if (__builtin_amdgcn_ballot_w64(mine != 0) == 0) {   // none for any row
    if (prow < p_rows && g == 0) { a.part_m[pi] = -INFINITY; a.part_l[pi] = 0.f; }
    return;
  }
  const size_t n_total = (size_t)(a.n_q_heads + 2 * a.n_kv_heads) * D;
  const float *base = a.qkv + (size_t)b * M * n_total;
  const float *kp = base + min(kb * 32 + ln, M - 1) * n_total + (size_t)(a.n_q_heads + kvh) * D + g * (D / 2);
  const float *qp = base + node * n_total + (size_t)(kvh * group + al) * D + g * (D / 2);
  f32x16 s0, s1;
#pragma unroll
  for (int e = 0; e < 16; ++e) s0[e] = s1[e] = 0.f;
  {
    f32x4 kv[D / 8], qv[D / 8];
#pragma unroll
    for (int t = 0; t < D / 8; ++t) { kv[t] = *(const f32x4 *)(kp + 4 * t); qv[t] = *(const f32x4 *)(qp + 4 * t); }
#pragma unroll
    for (int t = 0; t < D / 8; ++t) {
      s0 = __builtin_amdgcn_mfma_f32_32x32x2f32(kv[t][0], qv[t][0], s0, 0, 0, 0);
      s1 = __builtin_amdgcn_mfma_f32_32x32x2f32(kv[t][1], qv[t][1], s1, 0, 0, 0);
      s0 = __builtin_amdgcn_mfma_f32_32x32x2f32(kv[t][2], qv[t][2], s0, 0, 0, 0);
      s1 = __builtin_amdgcn_mfma_f32_32x32x2f32(kv[t][3], qv[t][3], s1, 0, 0, 0);
    }
  }
  const float *vp = base + (size_t)(a.n_q_heads + a.n_kv_heads + kvh) * D;
  float v[16][D / 32];   // all values in one round trip, behind the softmax
#pragma unroll
  for (int e = 0; e < 16; ++e)
#pragma unroll
    for (int db = 0; db < D / 32; ++db)
      v[e][db] = vp[min(kb * 32 + 8 * (e >> 2) + 4 * g + (e & 3), M - 1) * n_total + db * 32 + ln];
  __builtin_amdgcn_sched_barrier(0);
  const float scale = 1.44269504088896f / sqrtf((float)D);
  float p[16], m = -INFINITY, l = 0.f;
#pragma unroll
  for (int e = 0; e < 16; ++e) {
    const int key = 8 * (e >> 2) + 4 * g + (e & 3);
    p[e] = (mine >> key) & 1u ? (s0[e] + s1[e]) * scale : -INFINITY;
    m = fmaxf(m, p[e]);
  }
  m = fmaxf(m, __shfl_xor(m, 32, 64));
  const float m_safe = m == -INFINITY ? 0.f : m;
#pragma unroll
  for (int e = 0; e < 16; ++e) {
    p[e] = __builtin_amdgcn_exp2f(p[e] - m_safe);   // 0 for other branches
    l += p[e];
  }
  l += __shfl_xor(l, 32, 64);
  f32x16 o[D / 32];
#pragma unroll
  for (int db = 0; db < D / 32; ++db)
#pragma unroll
    for (int e = 0; e < 16; ++e) o[db][e] = 0.f;
  float finite = 0.f;   // stays 0 while every value is finite
#pragma unroll
  for (int e = 0; e < 16; ++e)
#pragma unroll
    for (int db = 0; db < D / 32; ++db) {
      finite = __builtin_fmaf(v[e][db], 0.f, finite);
      o[db] = __builtin_amdgcn_mfma_f32_32x32x2f32(v[e][db], p[e], o[db], 0, 0, 0);
    }
  if (__builtin_amdgcn_ballot_w64(finite != 0.f) != 0) {
    // an infinity or NaN among the values: a weight of 0 would carry it into rows of other branches.
    // Row by row over the ancestors only.
#pragma unroll
    for (int e = 0; e < 16; ++e) s_p[(8 * (e >> 2) + 4 * g + (e & 3)) * 32 + ln] = p[e];
    __builtin_amdgcn_s_waitcnt(0);
    __builtin_amdgcn_wave_barrier();
#pragma unroll
    for (int db = 0; db < D / 32; ++db)
#pragma unroll
      for (int e = 0; e < 16; ++e) o[db][e] = 0.f;
#pragma unroll 1
    for (int k = 0; k < 32; ++k) {
      if (!((mine >> k) & 1u)) continue;
      const float w = s_p[k * 32 + ln];
      const float *vr = vp + (kb * 32 + k) * n_total + 4 * g;
#pragma unroll
      for (int db = 0; db < D / 32; ++db)
#pragma unroll
        for (int e = 0; e < 16; ++e) o[db][e] += w * vr[db * 32 + 8 * (e >> 2) + (e & 3)];
    }
  }
  if (prow >= p_rows) return;
  if (g == 0) {
    a.part_m[pi] = mine != 0 ? stored_max(m) : -INFINITY;
    a.part_l[pi] = l;
  }
  float *out = a.part_o + pi * D;
#pragma unroll
  for (int db = 0; db < D / 32; ++db)
#pragma unroll
    for (int q = 0; q < 4; ++q)
      *(f32x4 *)(out + db * 32 + 8 * q + 4 * g) = f32x4{o[db][4 * q], o[db][4 * q + 1], o[db][4 * q + 2], o[db][4 * q + 3]};
}

// NW wavefronts; KG groups of them take KT / KG keys of every tile each, the NW / KG wavefronts of a group a
// block of 32 query rows each; the groups' sums meet in LDS at the end.
// <KT 128, NW 4, KG 1>: 128 rows, one workgroup per CU.  <KT 64, NW 8, KG 1>: 256 rows share every staged K/V tile
// (trees of more than 128 rows read the cache once, not twice) and two waves per SIMD overlap
// one another's softmax arithmetic and matrix work.
// <KT 128, KG 2 or 4>: 128 rows, of which a quarter and more are missing: wavefronts that would have none take
// keys instead (launch_attn_bf16_d).
// DRAFT: some workgroups (splits from n_splits on) take a block of draft nodes each instead.
// PAGED: the cache is in pages of kKvPage slots (a multiple of KT, and every split starts at a
// multiple of KT, so a tile never straddles two pages): one scalar page lookup per tile.
template <int D, int KT, int NW, int KG, bool PAGED, bool DRAFT>
__global__ __launch_bounds__(64 * NW) void k_attn_bf16(AttnArgs a) {
  using L = AttnLds<D, KT>;
  constexpr int NT = 64 * NW, RB = NW / KG, KW = KT / KG;   // row blocks; keys of a tile that a wavefront takes
  constexpr bool LONG = KT == 64, SPARE = LONG || KG > 1;   // 256-row workgroups; two wavefronts a SIMD or few rows
  __shared__ __attribute__((aligned(16))) unsigned char lds[2 * L::kBuf];
  const int split = blockIdx.x, kvh = blockIdx.y;
  const int b = blockIdx.z / a.n_row_groups, rg = blockIdx.z - b * a.n_row_groups;   // sequence, group of query rows
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);   // scalar: branches on it are wave-uniform
  const int ln = lane & 31, g = lane >> 5, rb = wave % RB, kg = wave / RB;
  const int M = a.n_nodes, group = a.n_q_heads / a.n_kv_heads;
  const int p_rows = group * M;
  const int ctx = a.ctx.v[b];
  const int n_keys = ctx;            // context only
  const int k_begin = split * a.keys_per_split;
  const int k_end = min(n_keys, k_begin + a.keys_per_split);
  const size_t part_base = ((size_t)b * a.n_kv_heads + kvh) * (a.n_splits + a.n_draft) + split;
  if constexpr (DRAFT) {
    if (split >= a.n_splits) {
      if (kg == 0) draft_partial<D>(a, split - a.n_splits, kvh, b, rg * RB + rb, part_base, (float *)lds + wave * 1024);
      return;
    }
  }

  const int prow = (rg * RB + rb) * 32 + ln;   // this lane's query row
  const bool rows_here = (rg * RB + rb) * 32 < p_rows;   // wave-uniform

  if (k_begin >= k_end) {   // empty split: neutral partial
    if (prow < p_rows && g == 0 && kg == 0) {
      a.part_m[part_base * p_rows + prow] = -INFINITY;
      a.part_l[part_base * p_rows + prow] = 0.f;
    }
    return;
  }

  static_assert(kKvPage % KT == 0, "a tile must not straddle pages");
  const int cap = PAGED ? kKvPage : a.kv.capacity;   // slots behind kc / vc, and the V^T row stride
  const bf16 *kc0 = (const bf16 *)a.k_cache, *vc0 = (const bf16 *)a.v_cache;
  if (!PAGED) {
    kc0 += ((size_t)b * a.n_kv_heads + kvh) * a.kv.capacity * D;
    vc0 += ((size_t)b * a.n_kv_heads + kvh) * D * a.kv.capacity;
  }

  // ---- tile staging: K tile = KT rows of D*2 bytes (16-byte vectors), V^T tile = D rows of KT*2 bytes
  constexpr int KV_PER_T = KT * D * 2 / 16 / NT;   // 16-byte vectors per thread, each of K and V^T
  typedef unsigned int u32x4 __attribute__((ext_vector_type(4)));   // native vector: stays in registers
  typedef unsigned int u32x2 __attribute__((ext_vector_type(2)));
  u32x4 kreg[KV_PER_T], vreg[KV_PER_T];
  // load_tile only ISSUES loads — anything that looked at a loaded value here would make the
  // compiler wait for each load in turn; the slots past the context are zeroed in store_tile.
  auto load_tile = [&](int k0g) {
    // contiguous: k0 counts from the sequence's first slot; paged: from the first slot of the tile's page
    const bf16 *kc = kc0, *vc = vc0;
    int k0 = k0g;
    if (PAGED) {
      const int page = a.kv.page_of(b, k0g);
      kc += ((size_t)page * a.n_kv_heads + kvh) * kKvPage * D;
      vc += ((size_t)page * a.n_kv_heads + kvh) * D * kKvPage;
      k0 = k0g % kKvPage;
    }
#pragma unroll
    for (int i = 0; i < KV_PER_T; ++i) {
      const int v = tid + NT * i;
      {  // K: vector v -> key v / (D/8), 16-byte column v % (D/8)
        const int key = v / (D / 8), c = v % (D / 8);
        // rows past the context hold no token (their scores are masked); clamped into the cache
        kreg[i] = *(const u32x4 *)(kc + (size_t)min(k0 + key, cap - 1) * D + c * 8);
      }
      {  // V^T: vector v -> feature v / (KT/8), 8 keys starting at (v % (KT/8)) * 8
        const int f = v / (KT / 8), c = v % (KT / 8);
        vreg[i] = *(const u32x4 *)(vc + (size_t)f * cap + min(k0 + c * 8, cap - 8));
      }
    }
  };
  auto store_tile = [&](int buf, int k0) {
    unsigned char *base = lds + buf * L::kBuf;
    const bool ragged = k0 + KT > n_keys;   // uniform over the workgroup: the context ends inside this tile
#pragma unroll
    for (int i = 0; i < KV_PER_T; ++i) {
      const int v = tid + NT * i;
      {
        const int key = v / (D / 8), c = v % (D / 8);
        *(u32x4 *)(base + key * L::kStrideK + c * 16) = kreg[i];
      }
      {
        const int f = v / (KT / 8), c = v % (KT / 8);
        u32x4 t = vreg[i];
        if (ragged) {   // zero the values of slots that hold no token (two keys per 32-bit word)
          const int left = n_keys - (k0 + c * 8);   // keys of this vector inside the context
          auto keep = [&](uint32_t x, int e0) {
            return x & ((e0 < left ? 0x0000ffffu : 0u) | (e0 + 1 < left ? 0xffff0000u : 0u));
          };
          t = u32x4{keep(t.x, 0), keep(t.y, 2), keep(t.z, 4), keep(t.w, 6)};
        }
        u32x2 *dst = (u32x2 *)(base + L::kBytesK + f * L::kStrideV + c * 16);
        dst[0] = u32x2{t.x, t.y};
        dst[1] = u32x2{t.z, t.w};
      }
    }
  };

  // ---- running state: one query row per lane (both lane halves hold the same row)
  float m_run = -INFINITY, l_run = 0.f;
  f32x16 oacc[D / 32];
#pragma unroll
  for (int db = 0; db < D / 32; ++db)
#pragma unroll
    for (int e = 0; e < 16; ++e) oacc[db][e] = 0.f;

  const int n_tiles = (k_end - k_begin + KT - 1) / KT;
  load_tile(k_begin);
  // The query rows (as many bytes per workgroup as a tile) are requested after the first tile,
  // whose wait then does not include them, and without a branch (a row past the end reads the
  // last row: every lane's row is independent and such lanes store nothing).
  // rotated query as bf16 high part + bf16 low part (written by the QKV epilogue)
  bf16x8 qf[D / 16], ql[D / 16];
  {
    const int pc = min(prow, p_rows - 1);
    const int al = pc / M, node = pc - al * M;
    const int r = b * M + node;
    const bf16 *q = (const bf16 *)a.q + (size_t)r * a.n_q_heads * D + (size_t)(kvh * group + al) * D;
#pragma unroll
    for (int t = 0; t < D / 16; ++t) {
      qf[t] = *(const bf16x8 *)(q + 16 * t + 8 * g);
      ql[t] = *(const bf16x8 *)(q + a.q_panel + 16 * t + 8 * g);
    }
  }
  store_tile(0, k_begin);
  // Long loops: the query rows have arrived before them.  A wait for them inside the loop could not tell them from the
  // next tile's loads, which may or may not have been issued since, and would drain those in every step.
  if (SPARE) __builtin_amdgcn_s_waitcnt(0x0F70);   // vmcnt(0)
  __syncthreads();

  for (int t = 0; t < n_tiles; ++t) {
    const int k0 = k_begin + t * KT;
    const int buf = t & 1;
    if (t + 1 < n_tiles) load_tile(k0 + KT);
    const unsigned char *kb = lds + buf * L::kBuf;
    const unsigned char *vb = kb + L::kBytesK;
    const int kw = kg * KW;                          // this wavefront's keys of the tile
    const bool need_mask = (k0 + kw + KW > k_end);   // ragged end of the context or of this split

    if (rows_here) {
      // S^T[key][row] for the 32-key sub-tiles.  Consecutive matrix instructions go to different
      // accumulators: one that adds to the result of the instruction before it has to wait for it.
      f32x16 s[KW / 32];
#pragma unroll
      for (int ks = 0; ks < KW / 32; ++ks)
#pragma unroll
        for (int e = 0; e < 16; ++e) s[ks][e] = 0.f;
#pragma unroll
      for (int tt = 0; tt < D / 16; ++tt) {
        bf16x8 kf[KW / 32];
#pragma unroll
        for (int ks = 0; ks < KW / 32; ++ks)
          kf[ks] = *(const bf16x8 *)(kb + (kw + ks * 32 + ln) * L::kStrideK + (16 * tt + 8 * g) * 2);
#pragma unroll
        for (int ks = 0; ks < KW / 32; ++ks)
          s[ks] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(kf[ks], qf[tt], s[ks], 0, 0, 0);
#pragma unroll
        for (int ks = 0; ks < KW / 32; ++ks)
          s[ks] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(kf[ks], ql[tt], s[ks], 0, 0, 0);
      }
      // mask (only the tile in which the context or the split ends: a scalar branch), tile max;
      // the scores arrive scaled: q was pre-multiplied by log2(e) / sqrt(d).  The vector ALU, not
      // the matrix cores, sets the pace of a tile step, so every instruction saved here counts.
      if (need_mask) {
#pragma unroll
        for (int ks = 0; ks < KW / 32; ++ks)
#pragma unroll
          for (int e = 0; e < 16; ++e) {
            const int key = k0 + kw + ks * 32 + 8 * (e >> 2) + 4 * g + (e & 3);
            s[ks][e] = (key < k_end) ? s[ks][e] : -INFINITY;
          }
      }
      float tmax = -INFINITY;
#pragma unroll
      for (int ks = 0; ks < KW / 32; ++ks)
#pragma unroll
        for (int e = 0; e < 16; ++e) tmax = fmaxf(tmax, s[ks][e]);
      tmax = fmaxf(tmax, __shfl_xor(tmax, 32, 64));
      float alpha = 1.f, psum = 0.f;
      bf16x8 phi[KW / 16], plo[KW / 16];
      if constexpr (SPARE) {
        // Long loops, two wavefronts a SIMD: what the vector ALU does adds to the products' time, so two probabilities are
        // converted at a time.  (One group of four wavefronts and two or three tiles: it does not pay, 17.6 -> 17.9 us.)
        // The reference is the running maximum of each row, whatever the other rows do.  One that moves only when a
        // score outgrows it by 2^8 saves most of the multiplications below (4 x 60 nodes over 16384 keys 13.07 -> 12.98 ms
        // a pass), but the largest probability is then no longer exactly 1, high part 1 and low part 0: logits are off by up to
        // 4 % more on rows with few large probabilities, and a probability of 2^8 takes values beyond 1e36 out of range.
        if (__builtin_amdgcn_ballot_w64(tmax > m_run) != 0) {
          const float m_new = fmaxf(m_run, tmax);
          alpha = __builtin_amdgcn_exp2f(m_run - (m_new == -INFINITY ? 0.f : m_new));   // exp2(-inf) = 0
          m_run = m_new;
          if (t > 0) {
#pragma unroll
            for (int db = 0; db < D / 32; ++db)
#pragma unroll
              for (int e = 0; e < 16; ++e) oacc[db][e] *= alpha;
          }
        }
        const float m_safe = (m_run == -INFINITY) ? 0.f : m_run;
#pragma unroll
        for (int ks = 0; ks < KW / 32; ++ks)
#pragma unroll
          for (int e = 0; e < 16; e += 2) {
            const f32x2 p = {__builtin_amdgcn_exp2f(s[ks][e] - m_safe), __builtin_amdgcn_exp2f(s[ks][e + 1] - m_safe)};   // exp2(-inf) = 0 for masked keys
            psum += p[0];
            psum += p[1];
            split_pair(p, phi[ks * 2 + (e >> 3)], plo[ks * 2 + (e >> 3)], e & 7);
          }
        l_run = l_run * alpha + psum;
      } else {
        const float m_new = fmaxf(m_run, tmax);
        const float m_safe = (m_new == -INFINITY) ? 0.f : m_new;
        alpha = __builtin_amdgcn_exp2f(m_run - m_safe);   // exp2(-inf) = 0 on the first tile
        m_run = m_new;
#pragma unroll
        for (int ks = 0; ks < KW / 32; ++ks)
#pragma unroll
          for (int e = 0; e < 16; ++e) {
            const float p = __builtin_amdgcn_exp2f(s[ks][e] - m_safe);   // exp2(-inf) = 0 for masked keys
            psum += p;
            const bf16 hi = (bf16)p;
            const bf16 lo = (bf16)(p - (float)hi);
            phi[ks * 2 + (e >> 3)][e & 7] = hi;
            plo[ks * 2 + (e >> 3)][e & 7] = lo;
          }
        l_run = l_run * alpha + psum;
        if (__builtin_amdgcn_ballot_w64(alpha != 1.0f) != 0) {   // the running maximum of some row moved
#pragma unroll
          for (int db = 0; db < D / 32; ++db)
#pragma unroll
            for (int e = 0; e < 16; ++e) oacc[db][e] *= alpha;
        }
      }
      // O^T[feature][row] = alpha * O^T + V^T P^T, the feature blocks interleaved for the same reason
#pragma unroll
      for (int u = 0; u < KW / 16; ++u) {
        bf16x8 vf[D / 32];
#pragma unroll
        for (int db = 0; db < D / 32; ++db) {
          // key slots of lane half g at step u: 16u + 4g + {0..3} and 16u + 8 + 4g + {0..3}
          const unsigned char *vp = vb + (db * 32 + ln) * L::kStrideV + (kw + 16 * u + 4 * g) * 2;
          const u32x2 v0 = *(const u32x2 *)vp;
          const u32x2 v1 = *(const u32x2 *)(vp + 16);
          const u32x4 vv = u32x4{v0.x, v0.y, v1.x, v1.y};
          vf[db] = *(const bf16x8 *)&vv;
        }
#pragma unroll
        for (int db = 0; db < D / 32; ++db)
          oacc[db] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(vf[db], phi[u], oacc[db], 0, 0, 0);
#pragma unroll
        for (int db = 0; db < D / 32; ++db)
          oacc[db] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(vf[db], plo[u], oacc[db], 0, 0, 0);
      }
    }
    if (t + 1 < n_tiles) store_tile(buf ^ 1, k0 + KT);
    __syncthreads();
  }

  l_run += __shfl_xor(l_run, 32, 64);
  if constexpr (KG > 1) {
    // ---- the key groups of a row block: all but the first hand their sums over through LDS (the last barrier of
    // the loop has freed it), 16 bytes a lane, no conflicts
    constexpr int kSums = (KG - 1) * RB;
    static_assert(kSums * ((D / 8) * 1024 + 256) <= 2 * L::kBuf, "the sums fit where the tiles were");
    f32x4 (*so)[D / 8][64] = (f32x4(*)[D / 8][64])lds;
    float *sm = (float *)(lds + kSums * (D / 8) * 1024), *sl = sm + kSums * 32;
    if (kg > 0) {
      const int o = (kg - 1) * RB + rb;
#pragma unroll
      for (int db = 0; db < D / 32; ++db)
#pragma unroll
        for (int q = 0; q < 4; ++q)
          so[o][db * 4 + q][lane] = f32x4{oacc[db][4 * q], oacc[db][4 * q + 1], oacc[db][4 * q + 2], oacc[db][4 * q + 3]};
      if (g == 0) { sm[o * 32 + ln] = m_run; sl[o * 32 + ln] = l_run; }
    }
    __syncthreads();
    if (kg > 0) return;
    float m = m_run;
#pragma unroll
    for (int i = 1; i < KG; ++i) m = fmaxf(m, sm[((i - 1) * RB + rb) * 32 + ln]);
    const float m_safe = m == -INFINITY ? 0.f : m;
    const float w0 = __builtin_amdgcn_exp2f(m_run - m_safe);   // 0 without keys
    m_run = m;
    l_run *= w0;
#pragma unroll
    for (int db = 0; db < D / 32; ++db)
#pragma unroll
      for (int e = 0; e < 16; ++e) oacc[db][e] *= w0;
#pragma unroll 1
    for (int i = 1; i < KG; ++i) {   // in ascending order
      const int o = (i - 1) * RB + rb;
      const float w = __builtin_amdgcn_exp2f(sm[o * 32 + ln] - m_safe);
      l_run += sl[o * 32 + ln] * w;
#pragma unroll
      for (int db = 0; db < D / 32; ++db)
#pragma unroll
        for (int q = 0; q < 4; ++q) {
          const f32x4 o1 = so[o][db * 4 + q][lane];
#pragma unroll
          for (int e = 0; e < 4; ++e) oacc[db][4 * q + e] += o1[e] * w;
        }
    }
  }

  // ---- write the split's partial: O[row][feature] unnormalised, m, l
  if (prow >= p_rows) return;
  if (g == 0) {
    a.part_m[part_base * p_rows + prow] = stored_max(m_run);
    a.part_l[part_base * p_rows + prow] = l_run;
  }
  float *o = a.part_o + (part_base * p_rows + prow) * D;
#pragma unroll
  for (int db = 0; db < D / 32; ++db)
#pragma unroll
    for (int q4 = 0; q4 < 4; ++q4)
      *(f32x4 *)(o + db * 32 + 8 * q4 + 4 * g) = f32x4{oacc[db][4 * q4], oacc[db][4 * q4 + 1], oacc[db][4 * q4 + 2], oacc[db][4 * q4 + 3]};
}

// Context (and draft blocks) for at most 64 query rows per kv head: chains, short trees, single tokens.
// The kernel above would leave three of its four wavefronts without a row.  Here RB wavefronts side by
// side hold the row blocks and the KG = 4 / RB groups of them take 32 keys each of every 32 KG keys,
// operands straight from the cache to registers (a wavefront's keys are its own, so LDS would save
// nothing); the groups' partials are merged through LDS at the end.  A tile's registers are requested
// again as soon as it has been used.  What bounds it is one chain of memory round trips: rows and first
// keys, partials out.  Over the kernel above: 9 nodes, 16 heads on 8, 1000 keys 11.4 -> 7.6 us, 4096 keys
// 12.6 -> 10.6; 30 nodes, 2048 keys 12.7 -> 12.1; one node, 32 heads on 8, 1500 keys 11.2 -> 7.4.
template <int D, int RB, bool PAGED>
__global__ __launch_bounds__(256, 2) void k_attn_few(AttnArgs a) {
  constexpr int KG = 4 / RB, LD = 33, FW = D / KG / 2;   // key groups; LDS row; features per thread of the merge
  __shared__ __attribute__((aligned(16))) float s_o[4 * D * LD];
  __shared__ float s_m[KG][RB * 32], s_l[KG][RB * 32];
  const int split = blockIdx.x, kvh = blockIdx.y, b = blockIdx.z;
  const int lane = threadIdx.x & 63, ln = lane & 31, g = lane >> 5;
  const int wave = __builtin_amdgcn_readfirstlane((int)threadIdx.x >> 6), rb = wave % RB, kg = wave / RB;
  const int M = a.n_nodes, group = a.n_q_heads / a.n_kv_heads, p_rows = group * M;
  const size_t part_base = ((size_t)b * a.n_kv_heads + kvh) * (a.n_splits + a.n_draft) + split;
  if (split >= a.n_splits) {
    if (wave < RB) draft_partial<D>(a, split - a.n_splits, kvh, b, wave, part_base, s_o + wave * 1024);
    return;
  }
  const int ctx = a.ctx.v[b], k_begin = split * a.keys_per_split, k_end = min(ctx, k_begin + a.keys_per_split);
  const int prow = rb * 32 + ln;
  if (k_begin >= k_end) {   // empty split: neutral partial
    if (kg == 0 && g == 0 && prow < p_rows) {
      a.part_m[part_base * p_rows + prow] = -INFINITY;
      a.part_l[part_base * p_rows + prow] = 0.f;
    }
    return;
  }
  const int cap = PAGED ? kKvPage : a.kv.capacity;   // slots behind kc / vc, and the V^T row stride
  // Score register e of lane (ln, g) is row 8 (e / 4) + 4 g + e % 4 of S^T.  Row i gets the key that makes
  // a lane's keys of one second-product step (16 u + 8 g ..) adjacent: V^T then comes in 16-byte pieces.
  auto key_of = [](int i) { return (i & 0x13) | (i & 4) << 1 | (i & 8) >> 1; };   // bits 2 and 3 swapped
  auto key_at = [&](int e) { return 16 * (e >> 3) + 8 * g + (e & 7); };
  bf16x8 kf[D / 16], vf[D / 32][2];
  // the keys k0 .. k0 + 31; slots past the context hold no token: clamped into the cache here, masked below
  auto at = [&](const void *cache, int k0, int &slot) {
    const bf16 *c = (const bf16 *)cache;
    if (PAGED) {
      slot = k0 % kKvPage;
      return c + ((size_t)a.kv.page_of(b, k0) * a.n_kv_heads + kvh) * kKvPage * D;
    }
    slot = k0;
    return c + ((size_t)b * a.n_kv_heads + kvh) * a.kv.capacity * D;
  };
  auto load_k = [&](int k0) {
    int slot;
    const bf16 *kr = at(a.k_cache, k0, slot);
    kr += (size_t)min(slot + key_of(ln), cap - 1) * D + 8 * g;
#pragma unroll
    for (int t = 0; t < D / 16; ++t) kf[t] = *(const bf16x8 *)(kr + 16 * t);
  };
  auto load_v = [&](int k0) {
    int slot;
    const bf16 *vr = at(a.v_cache, k0, slot) + (size_t)ln * cap;
#pragma unroll
    for (int db = 0; db < D / 32; ++db)
#pragma unroll
      for (int u = 0; u < 2; ++u) vf[db][u] = *(const bf16x8 *)(vr + (size_t)db * 32 * cap + min(slot + 16 * u + 8 * g, cap - 8));
  };
  // past the end a group reads the split's last keys again and masks all of them
  auto clamped = [&](int k0) { return min(k0, (k_end - 1) & ~31); };
  const int first = k_begin + kg * 32;
  load_k(clamped(first));
  bf16x8 qf[D / 16], ql[D / 16];
  {
    const int pc = min(prow, p_rows - 1), al = pc / M, r = b * M + pc - al * M;
    const bf16 *q = (const bf16 *)a.q + (size_t)r * a.n_q_heads * D + (size_t)(kvh * group + al) * D + 8 * g;
#pragma unroll
    for (int t = 0; t < D / 16; ++t) {
      qf[t] = *(const bf16x8 *)(q + 16 * t);
      ql[t] = *(const bf16x8 *)(q + a.q_panel + 16 * t);
    }
  }
  load_v(clamped(first));
  float m_run = -INFINITY, l_run = 0.f;
  f32x16 o[D / 32];
#pragma unroll
  for (int db = 0; db < D / 32; ++db)
#pragma unroll
    for (int e = 0; e < 16; ++e) o[db][e] = 0.f;
  for (int k0 = first; k0 < k_end; k0 += 32 * KG) {
    f32x16 sh, sl;   // high and low part of the queries apart: two chains of matrix instructions
#pragma unroll
    for (int e = 0; e < 16; ++e) sh[e] = sl[e] = 0.f;
#pragma unroll
    for (int t = 0; t < D / 16; ++t) {
      sh = __builtin_amdgcn_mfma_f32_32x32x16_bf16(kf[t], qf[t], sh, 0, 0, 0);
      sl = __builtin_amdgcn_mfma_f32_32x32x16_bf16(kf[t], ql[t], sl, 0, 0, 0);
    }
    load_k(clamped(k0 + 32 * KG));
    float s[16], m_new = m_run;
#pragma unroll
    for (int e = 0; e < 16; ++e) s[e] = sh[e] + sl[e];
    if (k0 + 32 > k_end) {   // wave-uniform: the context ends in here
#pragma unroll
      for (int e = 0; e < 16; ++e)
        if (k0 + key_at(e) >= k_end) s[e] = -INFINITY;
#pragma unroll
      for (int db = 0; db < D / 32; ++db)
#pragma unroll
        for (int e = 0; e < 16; ++e)
          if (k0 + key_at(e) >= k_end) vf[db][e >> 3][e & 7] = (bf16)0.f;
    }
#pragma unroll
    for (int e = 0; e < 16; ++e) m_new = fmaxf(m_new, s[e]);
    m_new = fmaxf(m_new, __shfl_xor(m_new, 32, 64));
    const float m_safe = m_new == -INFINITY ? 0.f : m_new;
    const float alpha = __builtin_amdgcn_exp2f(m_run - m_safe);
    m_run = m_new;
    float psum = 0.f;
    bf16x8 ph[2], pl[2];
#pragma unroll
    for (int e = 0; e < 16; ++e) {
      const float p = __builtin_amdgcn_exp2f(s[e] - m_safe);
      psum += p;
      ph[e >> 3][e & 7] = (bf16)p;
      pl[e >> 3][e & 7] = (bf16)(p - (float)ph[e >> 3][e & 7]);
    }
    l_run = l_run * alpha + psum;
#pragma unroll
    for (int db = 0; db < D / 32; ++db)
#pragma unroll
      for (int e = 0; e < 16; ++e) o[db][e] *= alpha;
#pragma unroll
    for (int u = 0; u < 2; ++u) {
#pragma unroll
      for (int db = 0; db < D / 32; ++db) o[db] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(vf[db][u], ph[u], o[db], 0, 0, 0);
#pragma unroll
      for (int db = 0; db < D / 32; ++db) o[db] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(vf[db][u], pl[u], o[db], 0, 0, 0);
    }
    load_v(clamped(k0 + 32 * KG));
  }

  // ---- merge the key groups: O^T [wave][feature][row] through LDS, a thread then takes FW features of a row
  l_run += __shfl_xor(l_run, 32, 64);
  if (g == 0) { s_m[kg][prow] = m_run; s_l[kg][prow] = l_run; }
#pragma unroll
  for (int db = 0; db < D / 32; ++db)
#pragma unroll
    for (int e = 0; e < 16; ++e) s_o[(wave * D + db * 32 + 8 * (e >> 2) + 4 * g + (e & 3)) * LD + ln] = o[db][e];
  __syncthreads();
  if (prow >= p_rows) return;
  float m = -INFINITY, l = 0.f, w[KG];
#pragma unroll
  for (int i = 0; i < KG; ++i) m = fmaxf(m, s_m[i][prow]);
  const float m_safe = m == -INFINITY ? 0.f : m;
#pragma unroll
  for (int i = 0; i < KG; ++i) {
    w[i] = __builtin_amdgcn_exp2f(s_m[i][prow] - m_safe);   // 0 for a group without keys
    l += s_l[i][prow] * w[i];
  }
  const size_t pi = part_base * p_rows + prow;
  if (kg == 0 && g == 0) {
    a.part_m[pi] = stored_max(m);
    a.part_l[pi] = l;
  }
  const int f0 = (kg * 2 + g) * FW;
#pragma unroll
  for (int q = 0; q < FW / 4; ++q) {
    f32x4 v = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int i = 0; i < KG; ++i)
#pragma unroll
      for (int e = 0; e < 4; ++e) v[e] += w[i] * s_o[((i * RB + rb) * D + f0 + 4 * q + e) * LD + ln];
    *(f32x4 *)(a.part_o + pi * D + f0 + 4 * q) = v;
  }
}

// Combine the partials of one (row, kv head) — all `group` query heads that share the kv head: context
// splits, then draft blocks, in ascending order.  Memory round trips, not arithmetic, set its time: up to
// NB partials of a thread are requested at once, the smallest of 6, 12 and 20 that holds them all (a request beyond the
// last partial would fetch it again, and its registers cost wavefronts in flight: 128 nodes, 12 partials, 8.0 us
// with 20 requested, 6.8 with 12).  Block = group * d / 2 threads, two adjacent output features each.
constexpr int kMergeBatch = 20;   // 16 context splits and the draft blocks of 128 nodes
// e^x through the hardware exp2 (about 1e-7 |x| relative error; the arguments here are <= 0)
__device__ __forceinline__ float fast_exp(float x) { return __builtin_amdgcn_exp2f(x * 1.4426950408889634f); }

template <int D, int NB>
__global__ __launch_bounds__(512) void k_attn_merge(AttnArgs a) {
  const int r = blockIdx.x, kvh = blockIdx.y, tid = threadIdx.x;
  const int M = a.n_nodes, group = a.n_q_heads / a.n_kv_heads;
  const int b = r / M, node = r - b * M;
  const int p_rows = group * M, n = a.n_splits + a.n_draft;
  const size_t base = ((size_t)b * a.n_kv_heads + kvh) * n;
  const int al = tid / (D / 2), f = (tid - al * (D / 2)) * 2;   // head, first feature
  if (al >= group) return;
  const int p = al * M + node;
  float pm[NB], pl[NB];
  float2 po[NB];
  auto request = [&](int s0) {
#pragma unroll
    for (int i = 0; i < NB; ++i) {
      const size_t idx = (base + min(s0 + i, n - 1)) * p_rows + p;
      pm[i] = a.part_m[idx];
      pl[i] = a.part_l[idx];
      po[i] = *(const float2 *)(a.part_o + idx * D + f);
    }
  };
  request(0);
  float m_tot = -INFINITY;
#pragma unroll
  for (int i = 0; i < NB; ++i) m_tot = fmaxf(m_tot, i < n ? pm[i] : -INFINITY);
  for (int s0 = NB; s0 < n; s0 += 16) {   // long contexts only
    float t[16];
#pragma unroll
    for (int i = 0; i < 16; ++i) t[i] = a.part_m[(base + min(s0 + i, n - 1)) * p_rows + p];
#pragma unroll
    for (int i = 0; i < 16; ++i) m_tot = fmaxf(m_tot, t[i]);
  }
  float num0 = 0.f, num1 = 0.f, den = 0.f;
  for (int s0 = 0; s0 < n; s0 += NB) {
    if (s0 > 0) request(s0);
#pragma unroll
    for (int i = 0; i < NB; ++i) {
      if (s0 + i >= n || pm[i] == -INFINITY) continue;   // no key in it: its o was never written
      const float w = fast_exp(pm[i] - m_tot);
      num0 += po[i].x * w;
      num1 += po[i].y * w;
      den += pl[i] * w;
    }
  }
  const float o0 = num0 / den, o1 = num1 / den;
  const bf16 h0 = (bf16)o0, h1 = (bf16)o1;
  bf16 *dst = (bf16 *)a.out;   // operand layout of the O projection; out_panel = number of 32-row blocks
  const int kk = (kvh * group + al) * D + f;   // even: both features sit in the same 8-element run
  bf16 *d0 = dst + ol_offset(r, kk, 0, (int)a.out_panel), *d1 = dst + ol_offset(r, kk, 1, (int)a.out_panel);
  d0[0] = h0; d0[1] = h1;
  d1[0] = (bf16)(o0 - (float)h0); d1[1] = (bf16)(o1 - (float)h1);
}

// The other merge, where the draft nodes have no workgroups of their own: combine the context splits of
// one (row, kv head) — all `group` query heads that share the kv head — in ascending split order, with
// the draft-node part: for every ancestor-or-self j of the
// node, score = q . k_j / sqrt(d) and value v_j, all taken in fp32 from this pass's projections
// (a.qkv: [row][(nq + 2 nkv) * d], q and k already rotated).
// Memory round trips, not arithmetic, set this kernel's time: the ancestor mask (one word, quick
// to arrive) is requested first, the query rows and the first NB split partials right behind it, and the
// ancestors' keys and the first ancestors' values, whose addresses need the mask, while those are on their way
// (60 nodes, 32 heads: 10.3 us with the partials behind the mask's arrival, 9.7 now; 9 x 4 nodes 6.9 -> 6.1).
// NB: 8 where that holds every split, else 16 (4 x 60 nodes, 8 splits: 26.4 us with 16 requested, 21.7 with 8; 9 x 4 nodes
// 6.1 -> 5.4).  Block = group * d / 2 threads, two adjacent output features each;
// the ancestor list (at most 128 nodes) is scored by (slot x quarter of the features) threads.
constexpr int kMergePreV = 8;    // ancestors whose values are fetched ahead of the scores
template <int D, int NB>
__global__ __launch_bounds__(512) void k_attn_merge_tree(AttnArgs a) {
  __shared__ float s_q[kMaxGroup][D];
  __shared__ float s_sc[kMaxGroup][kMaxNodes];
  __shared__ int s_anc[kMaxNodes];
  const int r = blockIdx.x, kvh = blockIdx.y, tid = threadIdx.x, nt = blockDim.x;
  const int M = a.n_nodes, group = a.n_q_heads / a.n_kv_heads;
  const int b = r / M, node = r - b * M;
  const int p_rows = group * M;
  const size_t base = ((size_t)b * a.n_kv_heads + kvh) * a.n_splits;
  const int n_total = (a.n_q_heads + 2 * a.n_kv_heads) * D;
  const bool active = tid < group * D / 2;
  const int al = active ? tid / (D / 2) : 0, f = active ? (tid - al * (D / 2)) * 2 : 0;   // head, first feature
  const int p = al * M + node;

  // ---- the ancestor list first: one word per workgroup arrives quickly, and every address of
  // the second group of loads depends on it
  const AncMask mask = a.anc[r];           // bit j: node j is on the root path of this node (self included)
  // what does not depend on it follows at once: the query rows and the first NB split partials of this thread's outputs
  const float2 q2 = *(const float2 *)(a.qkv + (size_t)r * n_total + (size_t)(kvh * group + al) * D + f);
  float pm[NB], pl[NB];
  float2 po[NB];
#pragma unroll
  for (int i = 0; i < NB; ++i) {
    const size_t idx = (base + min(i, a.n_splits - 1)) * p_rows + p;
    pm[i] = a.part_m[idx];
    pl[i] = a.part_l[idx];
    po[i] = *(const float2 *)(a.part_o + idx * D + f);
  }
  __builtin_amdgcn_sched_barrier(0);
  const int n_anc = mask.count();          // >= 1
  for (int j = tid; j < kMaxNodes; j += nt)
    if (mask.has(j)) s_anc[mask.rank(j)] = j;
  __syncthreads();

  // ---- the values of the first ancestors and the keys of the first batch of ancestors
  const float *vbase = a.qkv + (size_t)(a.n_q_heads + a.n_kv_heads + kvh) * D + f;
  float2 vpre[kMergePreV];
#pragma unroll
  for (int i = 0; i < kMergePreV; ++i)
    vpre[i] = *(const float2 *)(vbase + (size_t)(b * M + s_anc[min(i, n_anc - 1)]) * n_total);
  const int qq = tid & 3;
  f32x4 kv4[D / 16];
  {
    const int j = s_anc[min(tid >> 2, n_anc - 1)];
    const float *kp = a.qkv + (size_t)(b * M + j) * n_total + (size_t)(a.n_q_heads + kvh) * D + qq * 4;   // four lanes: 64 bytes side by side
#pragma unroll
    for (int i = 0; i < D / 16; ++i) kv4[i] = *(const f32x4 *)(kp + 16 * i);
  }
  if (active) { s_q[al][f] = q2.x; s_q[al][f + 1] = q2.y; }
  __syncthreads();

  // ---- scores of the ancestors: (slot x quarter of the features) threads, nt / 4 slots per batch
  const float scale = 1.0f / sqrtf((float)D);
  for (int s0 = 0; s0 < n_anc; s0 += nt / 4) {
    const int slot = s0 + (tid >> 2);
    if (s0 > 0) {   // later batches (deep paths on small workgroups) fetch their keys here
      const int j = s_anc[min(slot, n_anc - 1)];
      const float *kp = a.qkv + (size_t)(b * M + j) * n_total + (size_t)(a.n_q_heads + kvh) * D + qq * 4;
#pragma unroll
      for (int i = 0; i < D / 16; ++i) kv4[i] = *(const f32x4 *)(kp + 16 * i);
    }
    for (int h = 0; h < group; ++h) {
      float acc = 0.f;
#pragma unroll
      for (int i = 0; i < D / 16; ++i)
#pragma unroll
        for (int e = 0; e < 4; ++e) acc += kv4[i][e] * s_q[h][16 * i + 4 * qq + e];
      acc += __shfl_xor(acc, 1, 64);
      acc += __shfl_xor(acc, 2, 64);
      if (qq == 0 && slot < n_anc) s_sc[h][slot] = acc * scale;
    }
  }
  __syncthreads();
  if (!active) return;

  float m_tot = -INFINITY;
  for (int i = 0; i < n_anc; ++i) m_tot = fmaxf(m_tot, s_sc[al][i]);
#pragma unroll
  for (int i = 0; i < NB; ++i) m_tot = fmaxf(m_tot, (i < a.n_splits) ? pm[i] : -INFINITY);
  for (int s0 = NB; s0 < a.n_splits; s0 += NB) {   // long contexts only
    float t[NB];
#pragma unroll
    for (int i = 0; i < NB; ++i) t[i] = (s0 + i < a.n_splits) ? a.part_m[(base + s0 + i) * p_rows + p] : -INFINITY;
#pragma unroll
    for (int i = 0; i < NB; ++i) m_tot = fmaxf(m_tot, t[i]);
  }
  float num0 = 0.f, num1 = 0.f, den = 0.f;
  for (int s0 = 0; s0 < a.n_splits; s0 += NB) {    // ascending split order
    if (s0 > 0) {
#pragma unroll
      for (int i = 0; i < NB; ++i) {
        const size_t idx = (base + min(s0 + i, a.n_splits - 1)) * p_rows + p;
        pm[i] = a.part_m[idx];
        pl[i] = a.part_l[idx];
        po[i] = *(const float2 *)(a.part_o + idx * D + f);
      }
    }
#pragma unroll
    for (int i = 0; i < NB; ++i) {
      if (s0 + i >= a.n_splits || pm[i] == -INFINITY) continue;   // empty split: its o / l were never written
      const float w = fast_exp(pm[i] - m_tot);
      num0 += po[i].x * w;
      num1 += po[i].y * w;
      den += pl[i] * w;
    }
  }
#pragma unroll
  for (int i = 0; i < kMergePreV; ++i)
    if (i < n_anc) {
      const float w = fast_exp(s_sc[al][i] - m_tot);
      num0 += w * vpre[i].x;
      num1 += w * vpre[i].y;
      den += w;
    }
  for (int i0 = kMergePreV; i0 < n_anc; i0 += 4) {
    float2 vv[4];
#pragma unroll
    for (int i = 0; i < 4; ++i)
      vv[i] = *(const float2 *)(vbase + (size_t)(b * M + s_anc[min(i0 + i, n_anc - 1)]) * n_total);
#pragma unroll
    for (int i = 0; i < 4; ++i)
      if (i0 + i < n_anc) {
        const float w = fast_exp(s_sc[al][i0 + i] - m_tot);
        num0 += w * vv[i].x;
        num1 += w * vv[i].y;
        den += w;
      }
  }
  const float o0 = num0 / den, o1 = num1 / den;
  const bf16 h0 = (bf16)o0, h1 = (bf16)o1;
  bf16 *dst = (bf16 *)a.out;   // operand layout of the O projection; out_panel = number of 32-row blocks
  const int kk = (kvh * group + al) * D + f;   // even: both features sit in the same 8-element run
  bf16 *d0 = dst + ol_offset(r, kk, 0, (int)a.out_panel), *d1 = dst + ol_offset(r, kk, 1, (int)a.out_panel);
  d0[0] = h0; d0[1] = h1;
  d1[0] = (bf16)(o0 - (float)h0); d1[1] = (bf16)(o1 - (float)h1);
}

template <int D>
static void launch_attn_bf16_d(hipStream_t st, const AttnArgs &a) {
  dim3 grid(a.n_splits + (a.draft_mode == kDraftOwnGroups ? a.n_draft : 0), a.n_kv_heads, a.batch * a.n_row_groups);
  const bool paged = a.kv.page_table != nullptr;
#define TS_ATTN(KT_, NW_, KG_, PAGED_)                                                                                       \
  do {                                                                                                                       \
    if (a.draft_mode == kDraftOwnGroups)                                                                                     \
      hipLaunchKernelGGL((k_attn_bf16<D, KT_, NW_, KG_, PAGED_, true>), grid, dim3(64 * NW_), 0, st, a);                            \
    else                                                                                                                     \
      hipLaunchKernelGGL((k_attn_bf16<D, KT_, NW_, KG_, PAGED_, false>), grid, dim3(64 * NW_), 0, st, a);                           \
  } while (0)
  if (a.few && a.rows_per_wg == 32) {
    if (paged) hipLaunchKernelGGL((k_attn_few<D, 1, true>), grid, dim3(256), 0, st, a);
    else hipLaunchKernelGGL((k_attn_few<D, 1, false>), grid, dim3(256), 0, st, a);
  } else if (a.few) {
    if (paged) hipLaunchKernelGGL((k_attn_few<D, 2, true>), grid, dim3(256), 0, st, a);
    else hipLaunchKernelGGL((k_attn_few<D, 2, false>), grid, dim3(256), 0, st, a);
  } else if (a.rows_per_wg == 64) {
    if (paged) TS_ATTN(128, 8, 4, true);
    else TS_ATTN(128, 8, 4, false);
  } else if (a.rows_per_wg == 256) {
    if (paged) TS_ATTN(64, 8, 1, true);
    else TS_ATTN(64, 8, 1, false);
  } else {
    // 128 rows; fewer: the wavefronts that would have none share the keys of a tile out.  us, one group -> KG: 18 rows
    // (8192 keys, KG 4 of 4 wavefronts) 15.4 -> 13.5, 32 rows (4 x 4096) 25.3 -> 19.7, 52 rows (12000, 4 of 8) 21.2 -> 17.9, 56 rows
    // (8192) 16.6 -> 15.9, 74 rows (3 x 3001, 2 of 8) 20.9 -> 19.3, 88 rows (8192) 18.4 -> 17.7.  With all four
    // row blocks it does not pay: 17.4 -> 19 for 120 rows over 256 keys a workgroup.
    const int p_rows = a.n_q_heads / a.n_kv_heads * a.n_nodes;
    if (p_rows <= 32) {
      if (paged) TS_ATTN(128, 4, 4, true);
      else TS_ATTN(128, 4, 4, false);
    } else if (p_rows <= 64) {
      if (paged) TS_ATTN(128, 8, 4, true);
      else TS_ATTN(128, 8, 4, false);
    } else if (p_rows <= 96) {
      if (paged) TS_ATTN(128, 8, 2, true);
      else TS_ATTN(128, 8, 2, false);
    } else {
      if (paged) TS_ATTN(128, 4, 1, true);
      else TS_ATTN(128, 4, 1, false);
    }
  }
#undef TS_ATTN
  const int group = a.n_q_heads / a.n_kv_heads;
  const int merge_threads = group * D / 2 < 64 ? 64 : group * D / 2;   // <= 512 (group <= 8, d <= 128)
  const dim3 mgrid(a.batch * a.n_nodes, a.n_kv_heads), mblock(merge_threads);
  const int n = a.n_splits + a.n_draft;
  if (a.draft_mode == kDraftInMerge) {
    if (n <= 8) hipLaunchKernelGGL((k_attn_merge_tree<D, 8>), mgrid, mblock, 0, st, a);
    else hipLaunchKernelGGL((k_attn_merge_tree<D, 16>), mgrid, mblock, 0, st, a);
  } else if (n <= 6) {
    hipLaunchKernelGGL((k_attn_merge<D, 6>), mgrid, mblock, 0, st, a);
  } else if (n <= 12) {
    hipLaunchKernelGGL((k_attn_merge<D, 12>), mgrid, mblock, 0, st, a);
  } else {
    hipLaunchKernelGGL((k_attn_merge<D, kMergeBatch>), mgrid, mblock, 0, st, a);
  }
}

void launch_attn_bf16(hipStream_t st, const AttnArgs &a) {
  if (a.head_dim == 128) launch_attn_bf16_d<128>(st, a);
  else launch_attn_bf16_d<64>(st, a);
}

}  // namespace ts
