// Verification, resampling and emission (Sec. 4.2; Alg. 1 inner while loop,
// resample line and "s <- s*"): accept scan over the draft block, token draw from
// the backbone row at the first rejected position, gather of that row's hidden
// state for the decoding heads, draws from the head distributions, and the
// length-only cache rollback.  One 256-thread workgroup per logits row; all
// reductions run in a fixed order so results do not depend on timing.
#include "xsm_device.h"
#include "xsm_internal.h"
#include "xsm_verify_device.h"

namespace xsm {

// Scratch words of a sequence in the step's tail, device-coherent: what its workgroups hand to the one
// that arrives last.  k_verify: token and verdict of row j at [2 j], [2 j + 1]; k_emit: token and near-tie
// bit of head k at [2 k], [2 k + 1], or the head's tree level at [8 k ..]: 4 tokens, 4 probabilities.
__device__ __forceinline__ void put_word(int32_t* p, int32_t v) {
  __hip_atomic_store(p, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
__device__ __forceinline__ int32_t get_word(const int32_t* p) {
  return __hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
// Called by every thread after the first wavefront has put its words: true for the workgroup that is
// the last of n to arrive at the counter (which returns to zero).
__device__ __forceinline__ bool last_of(uint32_t* ticket, int n, int* shared) {
  if (threadIdx.x == 0) {
    __builtin_amdgcn_s_waitcnt(0);                     // the words (all of this wavefront) have arrived
    const uint32_t old = __hip_atomic_fetch_add(ticket, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    *shared = old == (uint32_t)(n - 1);
    if (*shared) __hip_atomic_store(ticket, 0u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
  }
  __syncthreads();
  return *shared != 0;
}

// Accept scan, backbone draw and hidden-state gather, one workgroup per logits row: whether row j accepts
// candidate j + 1 and which token it would draw do not depend on the rows in front, so all rows are looked at
// side by side and the sequence's last workgroup to finish walks the verdicts.  (One workgroup per
// sequence, row after row, is a chain of up to R + 1 passes over a logits row, 2-4 us each.)
__global__ __launch_bounds__(256) void k_verify(const float* Z0, const float* Hf,
                                                const int32_t* block, const int32_t* eff_len,
                                                const int32_t* slot, xsm_verify_params vp,
                                                int32_t* acc, int32_t* y0, uint32_t* wflags, int32_t* row_index,
                                                int32_t* words, uint32_t* tickets,
                                                float* G, int R, int V, int d) {
  __shared__ RowScratch sm;
  __shared__ int last, sm_a;
  const int j = blockIdx.x, b = blockIdx.y;
  const int n = eff_len[b];
  if (n < 0) {
    if (j > 0) return;
    if (threadIdx.x == 0) { acc[b] = -1; y0[b] = 0; if (row_index) row_index[b] = b * R; }
    if (G) for (int i = threadIdx.x; i < d; i += 256) G[(size_t)b * d + i] = 0.f;
    return;
  }
  const float* z = Z0 + (size_t)(b * R + j) * V;
  bool near = false, ok = false;
  if (j + 1 < R) ok = row_accepts(z, V, block[b * R + j + 1], vp, sm, &near);
  uint32_t flag = 0;
  const int tok = row_sample(z, V, vp, (uint32_t)(n + j + 1), 0u, (uint32_t)slot[b], sm, &flag);
  int32_t* const w = words + (size_t)b * kTailWords;
  if (threadIdx.x == 0) {
    put_word(w + 2 * j, tok);
    put_word(w + 2 * j + 1, (ok ? 1 : 0) | (near ? 2 : 0) | (flag ? 4 : 0));
  }
  if (!last_of(tickets + b, R, &last)) return;
  if (threadIdx.x < 64) {
    // lane j: verdict of row j; the first row that refuses its candidate is the accepted count (row R - 1 has
    // none: it always ends the walk).  A near-tie counts up to there.
    const int lane = threadIdx.x;
    const int v = lane < R ? get_word(w + 2 * lane + 1) : 0;
    const uint64_t refuse = __ballot(!(v & 1)), ties = __ballot(v & 2), draws = __ballot(v & 4);
    const int a = __ffsll((unsigned long long)refuse) - 1;
    if (lane == 0) {
      const uint64_t upto = (2ull << a) - 1;
      acc[b] = a;
      y0[b] = get_word(w + 2 * a);
      if ((ties & upto) || (draws >> a & 1)) wflags[b] |= XSM_FLAG_NEAR_TIE;
      if (row_index) row_index[b] = b * R + a;
      sm_a = a;
    }
  }
  if (!G) return;
  __syncthreads();
  const float* h = Hf + (size_t)(b * R + sm_a) * d;
  for (int i = threadIdx.x; i < d; i += 256) G[(size_t)b * d + i] = h[i];
}
void launch_verify(const float* Z0, const float* Hf, const int32_t* block, const int32_t* eff_len,
                   const int32_t* slot, const xsm_verify_params& vp, int32_t* acc, int32_t* y0,
                   uint32_t* wflags, int32_t* row_index, int32_t* words, uint32_t* tickets, float* G, int n_seq,
                   int R, int V, int d, hipStream_t s) {
  TraceScope trace_("verify", s);
  hipLaunchKernelGGL(k_verify, dim3(R, n_seq), dim3(256), 0, s, Z0, Hf, block, eff_len, slot, vp, acc,
                     y0, wflags, row_index, words, tickets, G, R, V, d);
}

// r_k = g + SiLU(W_k g + b_k): Hh holds W_k g for all heads, [n_seq][K][d]
struct BiasPtrs { const void* p[16]; };
template <typename T>
__global__ void k_head_act(const float* G, const float* Hh, BiasPtrs bias, float* Rk, int K, int d,
                           long total) {
  const long idx = (long)blockIdx.x * blockDim.x + threadIdx.x;
  if (idx >= total) return;
  const int i = (int)(idx % d), k = (int)((idx / d) % K), b = (int)(idx / ((long)d * K));
  const float pre = Hh[idx] + ldf((const T*)bias.p[k] + i);
  Rk[idx] = G[(size_t)b * d + i] + pre / (1.0f + expf(-pre));
}
void launch_head_act(int dtype, const float* G, const float* Hh, const void* const* bias_ptrs,
                     float* Rk, int n_seq, int K, int d, hipStream_t s) {
  TraceScope trace_("head_act", s);
  BiasPtrs bp;
  for (int k = 0; k < 16; ++k) bp.p[k] = k < K ? bias_ptrs[k] : nullptr;
  const long total = (long)n_seq * K * d;
  const dim3 grid((unsigned)((total + 255) / 256)), blk(256);
  if (dtype == XSM_BF16)
    hipLaunchKernelGGL(k_head_act<bf16_t>, grid, blk, 0, s, G, Hh, bp, Rk, K, d, total);
  else
    hipLaunchKernelGGL(k_head_act<float>, grid, blk, 0, s, G, Hh, bp, Rk, K, d, total);
}

// Draws from the K head rows, one workgroup per (head, sequence): a token each, or a level each of the
// probability tree; the sequence's last workgroup to finish draws the tree's path and emits: accepted
// tokens, count, next block, new length.  (K = 0, a plain step: one workgroup per sequence emits.)
__global__ __launch_bounds__(256) void k_emit(const float* Zh, xsm_verify_params vp, int32_t* words, uint32_t* tickets,
                                              const int32_t* eff_len, const int32_t* slot,
                                              const int32_t* acc, const int32_t* y0,
                                              const uint32_t* wflags, int32_t* block,
                                              int32_t* kv_len, int32_t* out_tokens,
                                              int32_t* n_accepted, uint32_t* flags, int R, int K,
                                              int V) {
  __shared__ RowScratch sm;
  __shared__ TreeLevels lv;
  __shared__ int old_block[16];
  __shared__ int cand[17];
  __shared__ uint32_t tie;
  __shared__ int last;
  const int k = blockIdx.x, b = blockIdx.y;
  const int n = eff_len[b];
  if (n < 0) {
    if (k == 0 && threadIdx.x == 0) { n_accepted[b] = 0; flags[b] = wflags[b]; }
    return;
  }
  const int a = acc[b];
  if (threadIdx.x == 0) tie = 0;
  if (K > 0) {
    int32_t* const w = words + (size_t)b * kTailWords;
    const float* z = Zh + (size_t)(b * K + k) * V;
    const bool tree = vp.sample == 2;
    if (tree) {
      row_level(z, V, vp.top_ks, 1.0f / vp.temperature, sm, lv.idx[0], lv.p[0]);
      if (threadIdx.x < (unsigned)vp.top_ks) {
        put_word(w + 8 * k + threadIdx.x, lv.idx[0][threadIdx.x]);
        put_word(w + 8 * k + 4 + threadIdx.x, (int32_t)__float_as_uint(lv.p[0][threadIdx.x]));
      }
    } else {
      uint32_t flag = 0;
      const int t = row_sample(z, V, vp, (uint32_t)(n + a + 2 + k), (uint32_t)(k + 1), (uint32_t)slot[b], sm, &flag);
      if (threadIdx.x == 0) { put_word(w + 2 * k, t); put_word(w + 2 * k + 1, flag ? 1 : 0); }
    }
    if (!last_of(tickets + b, K, &last)) return;
    const int i = threadIdx.x;
    if (tree) {
      if (i < 8 * K && (i & 3) < vp.top_ks) {
        const int32_t v = get_word(w + i);
        if ((i & 7) < 4) lv.idx[i >> 3][i & 3] = v;
        else lv.p[i >> 3][i & 3] = __uint_as_float((uint32_t)v);
      }
      __syncthreads();
      const float u = philox_uniform(vp.seed, (uint32_t)(n + a + 1), 254u, (uint32_t)slot[b]);
      const bool near = pts_pick(lv, K, vp.top_ks, vp.pts_prune, u, sm, cand);
      if (i == 0 && near) tie = 1;
    } else if (i < 64) {
      const bool near = i < K && get_word(w + 2 * i + 1) != 0;
      if (i < K) cand[i + 1] = get_word(w + 2 * i);
      if (__ballot(near) && i == 0) tie = 1;
    }
  }
  if (threadIdx.x < (unsigned)R) old_block[threadIdx.x] = block[b * R + threadIdx.x];
  __syncthreads();
  if (threadIdx.x == 0) {
    for (int j = 0; j < a; ++j) out_tokens[b * R + j] = old_block[j + 1];
    out_tokens[b * R + a] = y0[b];
    for (int j = a + 1; j < R; ++j) out_tokens[b * R + j] = -1;
    block[b * R] = y0[b];
    for (int j = 1; j <= K; ++j) block[b * R + j] = cand[j];
    n_accepted[b] = a + 1;
    kv_len[b] = n + a + 1;
    flags[b] = wflags[b] | (tie ? XSM_FLAG_NEAR_TIE : 0u);
  }
}
void launch_emit(const float* Zh, const xsm_verify_params& vp, const int32_t* eff_len,
                 const int32_t* slot, const int32_t* acc, const int32_t* y0,
                 const uint32_t* wflags, int32_t* words, uint32_t* tickets, int32_t* block, int32_t* kv_len,
                 int32_t* out_tokens, int32_t* n_accepted, uint32_t* flags, int n_seq, int R, int K, int V,
                 hipStream_t s) {
  TraceScope trace_("emit", s);
  hipLaunchKernelGGL(k_emit, dim3(K > 0 ? K : 1, n_seq), dim3(256), 0, s, Zh, vp, words, tickets, eff_len, slot, acc, y0,
                     wflags, block, kv_len, out_tokens, n_accepted, flags, R, K, V);
}

}  // namespace xsm
