// Small kernels of the verification pass: set-up, rotary table, embedding (+ first RMSNorm
// statistic), vocabulary statistics and the routing decision, feature export, commit of a path.
#include "device_util.hpp"

namespace ts {

// ------------------------------------------------------------------ set-up
// Also clears `zero[0 .. n_zero)`: the tile counters of the split-K matmuls and the barrier
// counters / abort word of the layer kernels, which must be zero when the pass starts.
__device__ __forceinline__ void setup_nodes(const NodeTable &tab, int rows, int n_nodes, AncMask *anc, int32_t *parent) {
  const int i = threadIdx.x;
  if (i < rows) {
    // root path of node i: walk up the parents (validated on the host: parent < node, root = -1)
    const int base = (i / n_nodes) * n_nodes;
    AncMask m;
    m.lo = m.hi = 0ull;
    for (int j = i - base, guard = 0; j >= 0 && guard < kMaxNodes; ++guard) {
      m.set(j);
      j = tab.parent[base + j];
    }
    anc[i] = m;
    parent[i] = tab.parent[i];
  }
}

__global__ void k_setup(NodeTable tab, int rows, int n_nodes, AncMask *anc, int32_t *parent) {
  setup_nodes(tab, rows, n_nodes, anc, parent);
}

void launch_setup(hipStream_t st, const NodeTable &tab, int rows, int n_nodes, AncMask *anc, int32_t *parent) {
  hipLaunchKernelGGL(k_setup, dim3(1), dim3(kMaxRows), 0, st, tab, rows, n_nodes, anc, parent);
}

__global__ void k_wait_probe(int32_t *counter, int expect, unsigned long long limit, int32_t *abort_word,
                             int32_t *status) {
  bar_wait(counter, expect, limit, abort_word, status);
}

void launch_wait_probe(hipStream_t st, int32_t *counter, int expect, unsigned long long limit,
                       int32_t *abort_word, int32_t *status) {
  hipLaunchKernelGGL(k_wait_probe, dim3(1), dim3(64), 0, st, counter, expect, limit, abort_word, status);
}

// angle[r][j] = position_r * base^(-2j/d), evaluated in fp64 so that large positions keep
// their phase; the table holds fp32 cos / sin.
__device__ __forceinline__ void rope_row(int r, const int32_t *positions, int head_dim, float base, float *cos_t,
                                         float *sin_t) {
  const int j = threadIdx.x;
  const int half = head_dim >> 1;
  if (j >= half) return;
  const double inv = pow((double)base, -2.0 * (double)j / (double)head_dim);
  const double ang = (double)positions[r] * inv;
  cos_t[r * half + j] = (float)cos(ang);
  sin_t[r * half + j] = (float)sin(ang);
}

// ------------------------------------------------------------------ embedding + first RMSNorm
// x[r] = E[token_r] (fp32 residual stream).  bf16 models also: the
// first matmul's operand panels h = x * w as bf16 hi + lo, and the row's sum of squares (that
// matmul's epilogue turns it into 1/rms).
template <typename AT>
__device__ __forceinline__ void embed_row(int r, const int32_t *tokens, const AT *embed, const AT *norm_w, int hidden,
                                          int vocab, float eps, float *x, void *h, size_t h_panel, float *ss_out) {
  __shared__ float red[4];
  int tok = tokens[r];
  if (tok < 0 || tok >= vocab) tok = 0;   // reported by the workgroup that sets the pass up
  const AT *e = embed + (size_t)tok * hidden;
  float *xr = x + (size_t)r * hidden;
  if constexpr (sizeof(AT) == 2) {
    // bf16 models (hidden is a multiple of 64): 8 elements = one 16-byte vector per step; a run of
    // 8 reduction indices is contiguous in the operand layout as well
    constexpr int MAXV = 4;                         // vectors per thread held in registers (hidden <= 8192)
    const int nv = hidden / 8;
    bf16x8 ev[MAXV], wv[MAXV];
#pragma unroll
    for (int u = 0; u < MAXV; ++u) {
      const int v = min((int)threadIdx.x + 256 * u, nv - 1);
      ev[u] = *(const bf16x8 *)(e + 8 * v);
      wv[u] = *(const bf16x8 *)(norm_w + 8 * v);
    }
    float ss = 0.f;
    for (int v0 = 0; v0 < nv; v0 += 256 * MAXV) {
#pragma unroll
      for (int u = 0; u < MAXV; ++u) {
        const int v = v0 + (int)threadIdx.x + 256 * u;
        if (v >= nv) continue;
        bf16x8 evv = ev[u], wvv = wv[u];
        if (v0 > 0) { evv = *(const bf16x8 *)(e + 8 * v); wvv = *(const bf16x8 *)(norm_w + 8 * v); }   // very wide models
        f32x4 x0, x1;
        bf16x8 hi, lo;
#pragma unroll
        for (int k = 0; k < 8; ++k) {
          const float xv = (float)evv[k];
          (k < 4 ? x0 : x1)[k & 3] = xv;
          ss += xv * xv;
          const float hv = xv * (float)wvv[k];
          hi[k] = (bf16)hv;
          lo[k] = (bf16)(hv - (float)hi[k]);
        }
        *(f32x4 *)(xr + 8 * v) = x0;
        *(f32x4 *)(xr + 8 * v + 4) = x1;
        bf16 *hp = (bf16 *)h;   // operand layout; h_panel carries the number of 32-row blocks
        *(bf16x8 *)(hp + ol_offset(r, 8 * v, 0, (int)h_panel)) = hi;
        *(bf16x8 *)(hp + ol_offset(r, 8 * v, 1, (int)h_panel)) = lo;
      }
    }
    ss = block_sum<4>(ss, red);
    if (threadIdx.x == 0) ss_out[r] = ss;
    (void)eps;
  } else {
    for (int i = threadIdx.x; i < hidden; i += 256) xr[i] = to_f32(e[i]);   // the consumers normalise
    (void)eps; (void)h; (void)h_panel; (void)ss_out; (void)norm_w;
  }
}

// Everything before the first matmul in one launch: workgroups 0 .. rows - 1 an embedding row each, rows ..
// 2 rows - 1 a row of the rotary table, the last one root paths, status word and counters.  Three
// launches took 14 us of a pass, nearly all of it launch and first memory round trip.
template <typename AT>
__global__ __launch_bounds__(256) void k_begin_pass(BeginArgs a) {
  static_assert(kMaxRows == 256, "a thread of the set-up workgroup per row");
  const int wg = blockIdx.x, i = threadIdx.x;
  if (wg < a.rows) {
    embed_row<AT>(wg, a.tokens, (const AT *)a.embed, (const AT *)a.norm_w, a.hidden, a.vocab, a.eps, a.x, a.h, a.h_panel,
                  a.ss_out);
  } else if (wg < 2 * a.rows) {
    rope_row(wg - a.rows, a.positions, a.head_dim, a.rope_base, a.cos_t, a.sin_t);
  } else {
    setup_nodes(a.tab, a.rows, a.n_nodes, a.anc, a.parent);
    const int bad = __syncthreads_or(i < a.rows && (a.tokens[i] < 0 || a.tokens[i] >= a.vocab));
    if (i == 0) *a.status = bad ? 1 : 0;
    for (int j = i; j < a.n_zero; j += 256) a.zero[j] = 0;
  }
}

void launch_begin_pass(hipStream_t st, int dtype, const BeginArgs &a) {
  const dim3 grid(2 * a.rows + 1);
  if (dtype == TRISPEC_F32) hipLaunchKernelGGL(k_begin_pass<float>, grid, dim3(256), 0, st, a);
  else hipLaunchKernelGGL(k_begin_pass<bf16>, grid, dim3(256), 0, st, a);
}

// One workgroup per node: count the vocabulary entries that precede the node's token in its
// parent's row of logits (exact integer sum: any order gives the same count).
__global__ __launch_bounds__(256) void k_draft_ranks(const float *logits, const int32_t *tokens, NodeTable tab,
                                                     int n_nodes, int vocab, int32_t *ranks) {
  __shared__ int red[4];
  const int r = blockIdx.x, tid = threadIdx.x;
  const int b = r / n_nodes, par = tab.parent[r], x = tokens[r];
  if (par < 0 || x < 0 || x >= vocab) {   // uniform over the workgroup
    if (tid == 0) ranks[r] = -1;
    return;
  }
  const float *row = logits + (size_t)(b * n_nodes + par) * vocab;
  const float lx = row[x];
  int n = 0;
  for (int c = tid; c < vocab; c += 256) {
    const float v = row[c];
    n += (v > lx) || (v == lx && c < x);
  }
#pragma unroll
  for (int o = 32; o > 0; o >>= 1) n += __shfl_xor(n, o, 64);
  if ((tid & 63) == 0) red[tid >> 6] = n;
  __syncthreads();
  if (tid == 0) ranks[r] = red[0] + red[1] + red[2] + red[3];
}

void launch_draft_ranks(hipStream_t st, const float *logits, const int32_t *tokens, const NodeTable &tab,
                        int batch, int n_nodes, int vocab, int32_t *ranks) {
  hipLaunchKernelGGL(k_draft_ranks, dim3(batch * n_nodes), dim3(256), 0, st, logits, tokens, tab, n_nodes, vocab, ranks);
}

// ------------------------------------------------------------------ decision
// Outputs of sequence b's nodes and its walk, by one workgroup of at least kMaxNodes threads.  At the current node test the
// trust predicate first (tau_a = tau_m is an escalation), then follow the lowest-numbered child whose draft token
// equals the verifier's argmax: one wavefront, two nodes a lane, so that a step is two ballots and not a search of the
// node table.
// AGENT: the statistics were written by other workgroups of this launch.
template <bool AGENT>
__device__ void decide_sequence(const DecideArgs &a, int b) {
  __shared__ int s_arg[kMaxNodes];
  const int i = threadIdx.x, M = a.n_nodes;
  auto ldf = [&](const float *p) { return AGENT ? ld_agent(p) : *p; };
  bool trusted = false;
  if (i < M) {
    const int r = b * M + i;
    const float l1 = ldf(a.node_l1 + r), l2 = ldf(a.node_l2 + r), sum = ldf(a.node_sum + r), ent = ldf(a.node_ent + r);
    const int arg = AGENT ? __hip_atomic_load(a.node_idx + r, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) : a.node_idx[r];
    // no logit above -inf (a row of NaN): the sum is empty, and 1 / 0 would pass every threshold
    const float s = l1 == -INFINITY ? NAN : sum;
    const float conf = 1.0f / s;                    // exp(l1 - l1) / sum
    const float margin = conf - expf(l2 - l1) / s;  // the second term is 0 when there is no second entry
    const float h = logf(s) - ent / s;              // ln sum e^d - sum e^d d / sum e^d
    s_arg[i] = arg;
    if (a.out.argmax) a.out.argmax[r] = arg;
    if (a.out.confidence) a.out.confidence[r] = conf;
    if (a.out.margin) a.out.margin[r] = margin;
    if (a.out.entropy) a.out.entropy[r] = h;
    // statistic on the right side of the threshold (a NaN statistic is never trusted)
    trusted = a.criterion == TRISPEC_CRIT_ENTROPY ? h <= a.threshold : (a.criterion == TRISPEC_CRIT_MARGIN ? margin : conf) >= a.threshold;
  }
  static_assert(kMaxNodes == 128, "the nodes are those of two wavefronts");
  __shared__ unsigned long long s_trust[2];
  const unsigned long long mine = __builtin_amdgcn_ballot_w64(trusted);
  if (i < kMaxNodes && (i & 63) == 0) s_trust[i >> 6] = mine;
  if (a.out.path && i < kMaxNodes) a.out.path[b * TRISPEC_PATH_STRIDE + i] = -1;
  __syncthreads();
  if (i >= 64) return;
  const bool relaxed = a.accept_top_k > 1 && a.draft_ranks != nullptr;
  int par[2], tok[2], rank[2];
#pragma unroll
  for (int w = 0; w < 2; ++w) {
    const int c = i + 64 * w, r = b * M + min(c, M - 1);
    par[w] = c < M ? a.parent[r] : -2;
    tok[w] = a.tokens[r];
    rank[w] = relaxed ? a.draft_ranks[r] : -1;
  }
  const unsigned long long trust0 = s_trust[0], trust1 = s_trust[1];
  int cur = a.n_forced - 1, acc = 0, token = -1, esc = 0;
  if (a.out.path && i == 0) a.out.path[b * TRISPEC_PATH_STRIDE] = cur;
  for (int step = 0; step <= M; ++step) {
    if (!(((cur < 64 ? trust0 : trust1) >> (cur & 63)) & 1ull)) { esc = 1; token = -1; break; }
    const int t = s_arg[cur];
    auto follows = [&](int w) { return par[w] == cur && (relaxed ? rank[w] >= 0 && rank[w] < a.accept_top_k : tok[w] == t); };
    const unsigned long long c0 = __builtin_amdgcn_ballot_w64(follows(0)), c1 = __builtin_amdgcn_ballot_w64(follows(1));
    if ((c0 | c1) == 0) { token = t; break; }
    cur = c0 != 0 ? __ffsll(c0) - 1 : 64 + __ffsll(c1) - 1;
    ++acc;
    if (a.out.path && i == 0) a.out.path[b * TRISPEC_PATH_STRIDE + acc] = cur;
  }
  if (i != 0) return;
  if (b == 0 && a.out.status) *a.out.status = *a.status_src;
  if (a.out.accepted_len) a.out.accepted_len[b] = acc;
  if (a.out.token) a.out.token[b] = token;
  if (a.out.escalate) a.out.escalate[b] = esc;
}

__global__ __launch_bounds__(kMaxNodes) void k_decide(DecideArgs a) { decide_sequence<false>(a, blockIdx.x); }

void launch_decide(hipStream_t st, const DecideArgs &a) {
  hipLaunchKernelGGL(k_decide, dim3(a.batch), dim3(kMaxNodes), 0, st, a);
}

// ------------------------------------------------------------------ vocabulary statistics
// Largest logit (its column, the second largest) of two sets; the lowest column of equal maxima
__device__ __forceinline__ void top2_win(float &l1, float &l2, int &idx, float ol1, float ol2, int oidx) {
  const bool up = ol1 > l1 || (ol1 == l1 && ol1 != -INFINITY && oidx < idx);
  l2 = up ? fmaxf(l1, ol2) : fmaxf(l2, ol1);
  l1 = up ? ol1 : l1;
  idx = up ? oidx : idx;
}
// The sums of a set whose largest logit is l1 at column idx, relative to the largest of all, m1 at column mi
__device__ __forceinline__ void top2_rescale(float l1, int idx, float m1, int mi, float &s, float &t) {
  if (idx == mi) return;   // the largest itself: l1 - m1 would be a NaN for +inf
  const float d = l1 == -INFINITY ? 0.f : l1 - m1, f = l1 == -INFINITY ? 0.f : expf(d);
  t = (t + s * d) * f;
  s *= f;
}
template <int U>
__device__ __forceinline__ void top2_absorb(Top2 &a, const Top2 (&b)[U]) {
  const float l0 = a.l1;
  const int i0 = a.idx;
#pragma unroll
  for (int u = 0; u < U; ++u) top2_win(a.l1, a.l2, a.idx, b[u].l1, b[u].l2, b[u].idx);
  top2_rescale(l0, i0, a.l1, a.idx, a.s, a.t);
#pragma unroll
  for (int u = 0; u < U; ++u) {
    float s = b[u].s, t = b[u].t;
    top2_rescale(b[u].l1, b[u].idx, a.l1, a.idx, s, t);
    a.s += s;
    a.t += t;
  }
}

// One workgroup per row: the per-tile statistics of the LM head (LOGITS: the row of logits itself, fp32 models) to the
// row's; the last workgroup of a sequence to finish takes its decision.  Threads stride the tiles, everything a thread
// reads is requested at once; then the largest of a wavefront is found first and every lane rescales its sums once, so that
// no exponential is on the chain of exchanges.  Orders are fixed: results do not depend on scheduling.
// Memory round trips set its time.  us, statistics (merged by pairs) and decision as launches of their own -> here: 1187 tiles,
// 60 nodes 9.8 + 7.6 -> 7.7, a chain of 128 9.6 + 12.3 -> 7.8, 512 entries and 9 nodes 9.5 + 4.0 -> 8.0; 4096 logits and 9 nodes
// 7.7 + 4.0 + 2.8 (three launches) -> 7.8.
constexpr int kStatsThreads = 256;
template <bool LOGITS>
__global__ __launch_bounds__(kStatsThreads) void k_stats_decide(HeadStats hs, const float *logits, int vocab, int32_t *done, DecideArgs d) {
  constexpr int NW = kStatsThreads / 64, U = LOGITS ? 16 : 5;
  static_assert(kStatsThreads >= kMaxNodes, "the workgroup takes a sequence's decision");
  __shared__ Top2 s_w[NW];
  __shared__ int s_last;
  const int r = blockIdx.x, tid = threadIdx.x, n = LOGITS ? vocab : hs.n_tiles;
  Top2 a = top2_empty();
  for (int i0 = tid; i0 < n; i0 += U * kStatsThreads) {
    Top2 b[U];
#pragma unroll
    for (int u = 0; u < U; ++u) {
      const int i = i0 + u * kStatsThreads;
      const size_t o = (size_t)r * n + min(i, n - 1);
      if constexpr (LOGITS) {
        const float v = logits[o];
        b[u].l1 = v; b[u].l2 = -INFINITY; b[u].s = v == -INFINITY ? 0.f : 1.f; b[u].t = 0.f; b[u].idx = i;
      } else {
        b[u].l1 = hs.l1[o]; b[u].l2 = hs.l2[o]; b[u].s = hs.sumexp[o]; b[u].t = hs.ent[o]; b[u].idx = hs.idx[o];
      }
    }
#pragma unroll
    for (int u = 0; u < U; ++u)
      if (i0 + u * kStatsThreads >= n) b[u] = top2_empty();
    top2_absorb(a, b);
  }
  {
    const float l1 = a.l1;
    const int idx = a.idx;
#pragma unroll
    for (int o = 1; o < 64; o <<= 1) {
      const float ol1 = __shfl_xor(a.l1, o, 64), ol2 = __shfl_xor(a.l2, o, 64);
      const int oi = __shfl_xor(a.idx, o, 64);
      top2_win(a.l1, a.l2, a.idx, ol1, ol2, oi);
    }
    top2_rescale(l1, idx, a.l1, a.idx, a.s, a.t);
#pragma unroll
    for (int o = 1; o < 64; o <<= 1) {
      a.s += __shfl_xor(a.s, o, 64);
      a.t += __shfl_xor(a.t, o, 64);
    }
  }
  if ((tid & 63) == 0) s_w[tid >> 6] = a;
  __syncthreads();
  if (tid == 0) {
    Top2 b[NW - 1];
    a = s_w[0];
#pragma unroll
    for (int w = 1; w < NW; ++w) b[w - 1] = s_w[w];
    top2_absorb(a, b);
    st_agent(d.node_l1 + r, a.l1); st_agent(d.node_l2 + r, a.l2); st_agent(d.node_sum + r, a.s); st_agent(d.node_ent + r, a.t);
    __hip_atomic_store(d.node_idx + r, a.idx, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
  }
  const int b = r / d.n_nodes;
  if (publish_then_count(done + b, d.n_nodes, &s_last)) decide_sequence<true>(d, b);
}

void launch_stats_decide(hipStream_t st, const HeadStats &hs, int rows, const float *logits, int vocab, int32_t *done, const DecideArgs &d) {
  if (logits != nullptr) hipLaunchKernelGGL(k_stats_decide<true>, dim3(rows), dim3(kStatsThreads), 0, st, hs, logits, vocab, done, d);
  else hipLaunchKernelGGL(k_stats_decide<false>, dim3(rows), dim3(kStatsThreads), 0, st, hs, logits, vocab, done, d);
}

// Plain streaming copy: grid-stride over blocks of 4 x 256 16-byte vectors, four independent
// loads in flight per thread before the stores.
__global__ __launch_bounds__(256) void k_copy_probe(uint4 *dst_, const uint4 *src_, size_t n) {
  typedef unsigned int u32x4 __attribute__((ext_vector_type(4)));
  u32x4 *dst = (u32x4 *)dst_;
  const u32x4 *src = (const u32x4 *)src_;
  const size_t stride = (size_t)gridDim.x * 1024;
  size_t i = (size_t)blockIdx.x * 1024 + threadIdx.x;
  for (; i + 768 < n; i += stride) {
    const u32x4 a = __builtin_nontemporal_load(src + i), b = __builtin_nontemporal_load(src + i + 256);
    const u32x4 c = __builtin_nontemporal_load(src + i + 512), d = __builtin_nontemporal_load(src + i + 768);
    __builtin_nontemporal_store(a, dst + i);
    __builtin_nontemporal_store(b, dst + i + 256);
    __builtin_nontemporal_store(c, dst + i + 512);
    __builtin_nontemporal_store(d, dst + i + 768);
  }
  for (; i < n; i += 256) dst[i] = src[i];   // ragged end of the last block
}

void launch_copy_probe(hipStream_t st, void *dst, const void *src, size_t bytes) {
  const size_t n = bytes / 16;
  size_t blocks = (n + 1023) / 1024;
  if (blocks > 256 * 16) blocks = 256 * 16;
  if (blocks < 1) blocks = 1;
  hipLaunchKernelGGL(k_copy_probe, dim3((unsigned)blocks), dim3(256), 0, st, (uint4 *)dst, (const uint4 *)src, n);
}

// Feature export: the final-norm output of every row in fp32.  One workgroup per row.
template <typename T>
__global__ __launch_bounds__(256) void k_export_hidden(const float *x, const T *w, const float *ss, int ss_tiles,
                                                        int rows_pad, int hidden, float eps, float *out) {
  const int r = blockIdx.x;
  float rstd = 1.f;
  if (ss != nullptr) {
    float s = 0.f;
    for (int t = 0; t < ss_tiles; ++t) s += ss[(size_t)t * rows_pad + r];   // ascending tile order
    rstd = 1.0f / sqrtf(s / (float)hidden + eps);
  }
  for (int c = threadIdx.x; c < hidden; c += 256) {
    const float v = x[(size_t)r * hidden + c];
    out[(size_t)r * hidden + c] = (ss != nullptr) ? v * rstd * to_f32(w[c]) : v;
  }
}

void launch_export_hidden(hipStream_t st, int dtype, const float *x, const void *norm_w, const float *ss,
                          int ss_tiles, int rows, int rows_pad, int hidden, float eps, float *out) {
  if (dtype == TRISPEC_F32)
    hipLaunchKernelGGL(k_export_hidden<float>, dim3(rows), dim3(256), 0, st, x, (const float *)norm_w, ss,
                       ss_tiles, rows_pad, hidden, eps, out);
  else
    hipLaunchKernelGGL(k_export_hidden<bf16>, dim3(rows), dim3(256), 0, st, x, (const bf16 *)norm_w, ss,
                       ss_tiles, rows_pad, hidden, eps, out);
}

// Commit of a verified path: per (kv head, sequence, layer) the K rows and the V^T columns of the
// path's nodes move from slot ctx + node[i] to slot ctx + i.  node[i] >= i, so a destination may
// be another row's source: everything is read into registers, then a barrier, then written.
template <typename T>
__global__ __launch_bounds__(256) void k_kv_commit(T *k_cache, T *v_cache, size_t layer_elems, KvMap kvm,
                                                    CommitTable t) {
  const int h = blockIdx.x, b = blockIdx.y, l = blockIdx.z, tid = threadIdx.x;
  const int n = t.n[b], ctx = t.ctx[b], d = kvm.d;
  if (n == 0) return;   // uniform over the workgroup
  T *kc = k_cache + (size_t)l * layer_elems;   // this layer; rows and columns through the slot map
  T *vc = v_cache + (size_t)l * layer_elems;
  const size_t vs = kvm.v_stride();
  constexpr int VEC = 16 / sizeof(T);                       // elements per 16-byte vector
  constexpr int MAXV = kMaxNodes * 128 / VEC / 256;         // vectors per thread at d = 128
  constexpr int MAXE = kMaxNodes * 128 / 256;               // V^T elements per thread at d = 128
  const int vec_per_row = d / VEC;
  typedef unsigned int u32x4 __attribute__((ext_vector_type(4)));   // native vector: stays in registers
  u32x4 kv[MAXV];
  T ve[MAXE];
#pragma unroll
  for (int u = 0; u < MAXV; ++u) {
    const int idx = tid + 256 * u, i = idx / vec_per_row, c = idx - i * vec_per_row;
    if (i < n) kv[u] = *(const u32x4 *)(kc + kvm.k_row(b, h, ctx + t.node[b][i]) + c * VEC);
  }
#pragma unroll
  for (int u = 0; u < MAXE; ++u) {
    const int idx = tid + 256 * u, f = idx / kMaxNodes, i = idx - f * kMaxNodes;   // 64 consecutive threads: one feature
    if (f < d && i < n) ve[u] = vc[kvm.v_col(b, h, ctx + t.node[b][i]) + (size_t)f * vs];
  }
  __syncthreads();
#pragma unroll
  for (int u = 0; u < MAXV; ++u) {
    const int idx = tid + 256 * u, i = idx / vec_per_row, c = idx - i * vec_per_row;
    if (i < n) *(u32x4 *)(kc + kvm.k_row(b, h, ctx + i) + c * VEC) = kv[u];
  }
#pragma unroll
  for (int u = 0; u < MAXE; ++u) {
    const int idx = tid + 256 * u, f = idx / kMaxNodes, i = idx - f * kMaxNodes;
    if (f < d && i < n) vc[kvm.v_col(b, h, ctx + i) + (size_t)f * vs] = ve[u];
  }
}

void launch_kv_commit(hipStream_t st, int dtype, void *k_cache, void *v_cache, int n_layers, size_t layer_elems,
                      int batch, const KvMap &kvm, const CommitTable &t) {
  dim3 grid(kvm.n_kv, batch, n_layers);
  if (dtype == TRISPEC_F32)
    hipLaunchKernelGGL(k_kv_commit<float>, grid, dim3(256), 0, st, (float *)k_cache, (float *)v_cache, layer_elems,
                       kvm, t);
  else
    hipLaunchKernelGGL(k_kv_commit<bf16>, grid, dim3(256), 0, st, (bf16 *)k_cache, (bf16 *)v_cache, layer_elems,
                       kvm, t);
}

}  // namespace ts
