// All decoder layers of one pass as ONE persistent kernel, for passes of 17 to a few hundred rows
// (batched speculative and plain steps, short prefills); bf16, head_dim 64, F = 4 d.
//
// At these sizes a layer is five dependent stages (QKV, attention, O-projection, FFN-up, FFN-down;
// eight with cross-attention) of 1-3 us of work each, so what bounds it is what lies between
// them: a kernel boundary on gfx950 costs 2.5 us for an empty kernel and 4-5 us once the next one has
// to fetch what the last one wrote, and with separate kernels there were seven per layer (two of
// them RMSNorm passes).  Here 256 workgroups of 512 threads, one per compute unit, stay for
// the whole pass:
//   - A stage hands its output to the next one through memory with device-coherent (sc1) stores and
//     loads; "all tasks of the stage are done" is sixteen counters on lines of their own, added to by
//     the workgroups that finish a task and polled by one wavefront of each waiting workgroup
//     (1.4 us measured over 256 workgroups; one shared counter takes 3.8 us, release / acquire fences,
//     which write back and invalidate the 4 MB L2s, 20-60 us).
//   - Weights do not depend on activations: a workgroup requests all of its next task's weights
//     before it waits, so their HBM latency runs under the wait.
//   - RMSNorm is no pass of its own.  Whoever produces residual rows writes them as bf16 hi / lo
//     operand planes already multiplied by the next norm's gain, and one sum of squares per
//     (row, 16 columns); whoever consumes them multiplies its products by the row's 1 / rms.
//
// Projections.  A task is NT 16-row weight tiles x MT 16-row activation tiles over the whole
// contraction length.  The eight wavefronts split the contraction index; each holds its weight
// fragments in registers and streams its activation fragments straight from L2 (one contiguous KB
// per request; 125 GB/s per compute unit measured, 32 TB/s over the chip, against 8 TB/s when four
// wavefronts had four requests each in flight), and the eight partial tiles are summed through LDS
// in wavefront order.  The host picks (NT, MT) per projection so that there are about as many tasks
// as compute units and the bytes a task pulls from L2 are least (layers_tile).
//
// Attention.  The 64-key chunks of all (sequence, query tile, head) units form one list that is cut
// into 256 equal tasks and inside a task into eight equal wavefront ranges, whatever the
// sequences' lengths: a batch of ragged lengths keeps every compute unit busy to the end (one unit
// per workgroup left a third of the chip idle at lengths uniform on [n/2, n]).  A wavefront that
// holds a whole unit finishes it; pieces are merged in LDS, and pieces of different tasks by the
// last one to arrive, always in chunk order.
//
// Progress.  Tasks are numbered in stage order and claimed from sixteen queues by workgroups in
// dispatch order; a task waits only for lower-numbered ones.  The lowest unfinished task therefore
// always belongs to a running workgroup that waits for nothing, however few workgroups are resident
// (another stream's kernel may hold compute units), so the grid drains without needing to be
// co-resident.  Waits are bounded all the same: a workgroup that gives up marks every sequence
// as skipped (XSM_FLAG_DEVICE_TIMEOUT) and raises the error word of xsm_check_device; until that has
// reported it, every pass that starts finds the word and skips all of its sequences.
#include <type_traits>
#include "xsm_attn_device.h"
#include "xsm_internal.h"

namespace xsm {

namespace {

typedef unsigned u32x4 __attribute__((ext_vector_type(4)));
typedef unsigned u32x2 __attribute__((ext_vector_type(2)));

constexpr int kThreads = 512, kWaves = 8;
constexpr int kTasksPerAttn = 256;                  // equal shares of an attention stage
constexpr int kSlotFloats = (2 + 64) * 16;          // partial attention result: m[16], l[16], O^T fragments [4][64][4]
constexpr int kQueues = 16, kQueueStride = 32;      // claim queues and done counters, one 128-byte line each
constexpr int kClaimer = kThreads - 64;              // thread that claims tasks (the first wavefront polls)
constexpr int kMaxLayers = 48;
constexpr int kNoTask = 0x7fffffff;
constexpr int kMaxUnits = 1024, kMaxSeq = 1024;
constexpr uint64_t kWaitTicks = 200000000ull;       // 2 s of the 100 MHz clock

// ---- device-coherent accesses (sc1): what one workgroup wrote, another reads in the same launch ----
constexpr int kCoh = 16;
typedef __amdgpu_buffer_rsrc_t rsrc_t;
__device__ __forceinline__ rsrc_t make_rsrc(const void* p, size_t bytes) {
  return __builtin_amdgcn_make_buffer_rsrc(const_cast<void*>(p), 0, (int)bytes, 0x00020000);
}
__device__ __forceinline__ uint4 ldc16(rsrc_t r, unsigned off, unsigned uniform_off = 0) {
  return __builtin_bit_cast(uint4, __builtin_amdgcn_raw_buffer_load_b128(r, (int)off, (int)uniform_off, kCoh));
}
__device__ __forceinline__ void stc16(rsrc_t r, unsigned off, f32x4 v) {
  __builtin_amdgcn_raw_buffer_store_b128(__builtin_bit_cast(u32x4, v), r, (int)off, 0, kCoh);
}
__device__ __forceinline__ void stc8(rsrc_t r, unsigned off, uint2 v) {
  __builtin_amdgcn_raw_buffer_store_b64(u32x2{v.x, v.y}, r, (int)off, 0, kCoh);
}
template <typename P, typename T> __device__ __forceinline__ void st_coh(P p, T v) {
  __hip_atomic_store(p, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
template <typename T> __device__ __forceinline__ T ld_coh(const T* p) {
  return __hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
// The layer table is kept in LDS; a pointer from there has lost its address space, and an access
// through it would be a FLAT one, which waits for every other access in flight: say that it is global.
template <typename T> using gptr = __attribute__((address_space(1))) T*;
template <typename T> __device__ __forceinline__ gptr<T> glob(T* p) { return (gptr<T>)p; }
__device__ __forceinline__ uint4 ldg16(const void* p) { return __builtin_bit_cast(uint4, *(gptr<const u32x4>)p); }
__device__ __forceinline__ int uni(int x) { return __builtin_amdgcn_readfirstlane(x); }
// A value the compiler may not compute ahead: the stages of the task loop are different code, and
// what each derives from the thread index or the arguments would otherwise be hoisted in front of
// the loop and kept in registers through all of them.
__device__ __forceinline__ int fresh(int x) { asm volatile("" : "+v"(x)); return x; }
__device__ __forceinline__ const LayersArgs& fresh_args() {
  uint64_t p = (uint64_t)__builtin_amdgcn_kernarg_segment_ptr();
  asm volatile("" : "+s"(p));
  return *(const LayersArgs*)(const __attribute__((address_space(4))) LayersArgs*)p;
}

// four consecutive columns (n % 4 == 0) of row m -> hi / lo operand planes [rows][K] behind r
template <int K>
__device__ __forceinline__ void planes4(rsrc_t r, unsigned lo_bytes, int m, int n, float4 v) {
  uint2 hi, lo;
  split4(v, hi, lo);
  const unsigned o = (unsigned)plane_index(K, m, n) * 2u;
  stc8(r, o, hi);
  stc8(r, o + lo_bytes, lo);
}
__device__ __forceinline__ u32x2 gain_bits4(const uint16_t* g, int n) { return *(gptr<const u32x2>)(g + n); }
__device__ __forceinline__ float4 gain4(u32x2 x) {
  return float4{__uint_as_float(x.x << 16), __uint_as_float(x.x & 0xFFFF0000u), __uint_as_float(x.y << 16),
                __uint_as_float(x.y & 0xFFFF0000u)};
}
__device__ __forceinline__ float gelu_erf_f(float x) { return 0.5f * x * (1.0f + erff(x * 0.70710678118654752f)); }

// ---------------------------------------------------------------------------
// In front of the layers, one launch: input rows (token embeddings, or prefix embeddings in a
// prefill) as residual tiles, operand planes of the first norm and sums of squares; validation of
// the sequences (the step's prepare pass); the attention partition; cleared queues and counters.
// One workgroup per row, one more for the rest.
// ---------------------------------------------------------------------------
__device__ __forceinline__ uint32_t seq_flags(const LayersBegin& a, int b, int* len, int* slot) {
  uint32_t f = a.err && *a.err ? XSM_FLAG_DEVICE_TIMEOUT : 0;
  const int n = a.kv_len[b], sl = a.slot[b];
  if (n < 0 || n + a.R > a.max_ctx || n > a.bound) f |= XSM_FLAG_BAD_LEN;
  if (sl < 0 || sl >= a.max_batch) f |= XSM_FLAG_BAD_SLOT;
  for (int j = 0; j < a.R; ++j) {
    const int t = a.block[b * a.R + j];
    if (t < 0 || t >= a.vocab) f |= XSM_FLAG_BAD_TOKEN;
  }
  *len = n; *slot = (f & XSM_FLAG_BAD_SLOT) ? 0 : sl;
  return f;
}

__global__ __launch_bounds__(256) void k_layers_begin(const LayersBegin a) {
  const int M = a.n_seq * a.R, tid = threadIdx.x;
  if ((int)blockIdx.x < M) {
    const int m = blockIdx.x, b = m / a.R, j = m % a.R, D = a.d;
    bool live = true;
    const uint16_t* row;
    if (a.rows) {                                     // prefill: positions row0 + j of the prefix
      row = a.rows + ((size_t)b * a.rows_per_seq + a.row0 + j) * D;
    } else {
      int len, sl;
      live = seq_flags(a, b, &len, &sl) == 0;
      row = a.E + (size_t)(live ? a.block[m] : 0) * D;
    }
    const int Mp = (M + 15) & ~15;
    uint16_t* hp = reinterpret_cast<uint16_t*>(a.planes);
    for (int c = tid * 4; c < D; c += 1024) {
      float4 v = gain4(gain_bits4(row, c));                       // (four bf16 values)
      if (!live) v = float4{0.f, 0.f, 0.f, 0.f};
      const size_t tile = (size_t)(m >> 4) * (D >> 4) + (c >> 4);
      *reinterpret_cast<float4*>(a.x + (tile * 64 + (m & 15) + 16 * ((c >> 2) & 3)) * 4) = v;
      float ss = v.x * v.x + v.y * v.y + v.z * v.z + v.w * v.w;
      ss += lane_xor<1>(ss); ss += lane_xor<2>(ss);  // 16 columns = four neighbouring threads
      if ((tid & 3) == 0) a.ssq[(size_t)m * (D >> 4) + (c >> 4)] = ss;
      const float4 g = gain4(gain_bits4(a.gain, c));
      uint2 hi, lo;
      split4(float4{v.x * g.x, v.y * g.y, v.z * g.z, v.w * g.w}, hi, lo);
      const size_t o = plane_index(D, m, c);
      *reinterpret_cast<uint2*>(hp + o) = hi;
      *reinterpret_cast<uint2*>(hp + (size_t)Mp * D + o) = lo;
    }
    return;
  }
  __shared__ int cnt[kMaxUnits];
  const int QT = (a.R + 15) >> 4, NU = a.n_seq * QT;
  if (a.partition)
    for (int i = tid; i < 2 * kQueues * kQueueStride; i += 256) a.ctrl[i] = 0;
  for (int b = tid; b < a.n_seq; b += 256) {
    int len = a.err && *a.err ? -1 : a.row0, sl = 0;
    if (!a.rows) {
      const uint32_t f = seq_flags(a, b, &len, &sl);
      if (f) len = -1;
      a.slot_out[b] = sl;
      a.wflags[b] = f;
      a.arrived[b] = 0;
    }
    a.eff_len[b] = len;
    for (int qt = 0; a.partition && qt < QT; ++qt)
      cnt[b * QT + qt] = len < 0 ? 0 : (len + min(a.R, (qt + 1) * 16) + 63) >> 6;
  }
  if (!a.partition) return;
  __syncthreads();
  // exclusive prefix sums of the units' chunk counts: a run of units per thread, then over the runs
  __shared__ int tot[256];
  const int per = (NU + 255) / 256, u0 = min(NU, tid * per), u1 = min(NU, u0 + per);
  int s = 0;
  for (int u = u0; u < u1; ++u) s += cnt[u];
  tot[tid] = s;
  __syncthreads();
  int base = 0;
  for (int i = 0; i < tid; ++i) base += tot[i];
  __shared__ int pre[kMaxUnits + 1];
  for (int u = u0; u < u1; ++u) { a.unit_pre[u] = pre[u] = base; base += cnt[u]; }
  if (tid == 255) { a.unit_pre[NU] = pre[NU] = base; tot[0] = 0; }
  __syncthreads();
  // shares of whole units (thread t: share t): within 4 % of equal?
  const int total = pre[NU] * a.H;
  const int nsh = min(kTasksPerAttn, total);
  auto edge = [&](int t) {
    if (t >= nsh) return total;
    const int x = (int)((long)t * total / nsh);
    int lo = 0, hi = NU;                              // largest unit with pre * H <= x
    while (hi - lo > 1) { const int mid = (lo + hi) >> 1; if (pre[mid] * a.H <= x) lo = mid; else hi = mid; }
    const int NC = pre[lo + 1] - pre[lo], c = (x - pre[lo] * a.H) % NC;
    return x - c + (2 * c >= NC ? NC : 0);
  };
  if (tid < nsh) atomicMax(&tot[0], edge(tid + 1) - edge(tid));
  __syncthreads();
  if (tid == 0) a.unit_pre[NU + 1] = (long)tot[0] * nsh * 25 <= (long)total * 26;
}

// ---------------------------------------------------------------------------
struct Smem {
  union {
    float4 red[2 * kWaves * 8 * 64];                  // partial tiles of a projection, two groups
    float slots[kWaves * 2 * kSlotFloats];            // attention results: two per wavefront
  };
  float inv[64];                                      // 1 / rms of the task's rows
  int pre[kMaxUnits + 2];
  int eff[kMaxSeq], slot[kMaxSeq];
  int meta[kWaves * 2][4];                            // unit key, first chunk, end chunk
  int task, abort, last;
  uint4 junk[kWaves * 64];                            // target of requests that only warm the L2
  LayerWts wts[kMaxLayers];
};

// which stage a task number belongs to (a workgroup's tasks only ever go up)
struct TaskPos { int layer, st, idx; };
__device__ __forceinline__ TaskPos task_pos(const LayersArgs& a, int t, int from_layer) {
  TaskPos p;
  p.layer = from_layer;
  while (t >= (p.layer + 1) * a.per_layer) ++p.layer;
  const int r = t - p.layer * a.per_layer;
  p.st = 0;
#pragma unroll
  for (int s = 1; s < kMaxLayerStages; ++s)
    if (s < a.n_stages && r >= a.stage[s].base) p.st = s;
  p.idx = r - a.stage[p.st].base;
  return p;
}
// Position of a projection task: the slices of one weight group, then its row chunks follow each other
// on one XCD (task numbers go round the queues, queues round the XCDs), so an XCD's L2 sees a
// weight once.  Row groups mg0 .. mg1 - 1.
struct Tile { int ng, ks, mc, mg0, mg1; };
__device__ __forceinline__ bool tile_pos(const LayerStage& st, int idx, Tile* t) {
  if (idx >= st.NG * st.MC * st.KS) return false;     // (numbers that only fill a stage up to whole queues)
  const int x = idx & 7, i = idx >> 3, j = st.KS == 1 ? i : i >> 2, q = j / st.MC, mc = j - q * st.MC;
  t->ks = st.KS == 1 ? 0 : i & 3;
  t->ng = q * 8 + x;
  t->mc = mc;
  t->mg0 = mc * st.MG / st.MC;
  t->mg1 = (mc + 1) * st.MG / st.MC;
  return true;
}
__device__ __forceinline__ const uint4* stage_weights(int kind, const LayerWts* w) {
  switch (kind) {
    case kStQkv: return w->Wqkv;
    case kStO: return w->Wo;
    case kStCq: return w->Wcq;
    case kStCo: return w->Wco;
    case kStUp: return w->W1;
    default: return w->W2;
  }
}

// the weight fragments of a wavefront's share of a task: tiles nt0.., k-tiles kt0.. of KT
template <int NT, int KW, int NF>
__device__ __forceinline__ void load_weights(const uint4* W, int nt0, int KT, int kt0, int lane, uint4 (&w)[NF]) {
  const uint4* p = W + ((size_t)nt0 * KT + kt0) * 64 + lane;
#pragma unroll
  for (int t = 0; t < NT; ++t)
#pragma unroll
    for (int i = 0; i < KW; ++i) w[t * KW + i] = ldg16(p + ((size_t)t * KT + i) * 64);
}
__device__ __forceinline__ void lds_direct16(const void* gptr, void* lds) {
  __builtin_amdgcn_global_load_lds((const __attribute__((address_space(1))) void*)gptr,
                                   (__attribute__((address_space(3))) void*)lds, 16, 0, 0);
}
// The next stage's weights on their way into this XCD's L2 while this stage is worked on: each of
// the 32 workgroups of an XCD asks for its part of what the XCD's tasks will read.  The requests
// end in an LDS area nobody reads, so they take no registers.
template <int D>
__device__ __forceinline__ void warm_next(const LayersArgs& a, Smem& sm, int layer, int st_no, int wave, int lane) {
  const bool wrap = st_no + 1 == a.n_stages;
  if (wrap && layer + 1 == a.L) return;
  const LayerStage& st = a.stage[wrap ? 0 : st_no + 1];
  if (st.kind == kStAtt || st.kind == kStCatt) return;
  const uint4* W = stage_weights(st.kind, sm.wts + layer + (wrap ? 1 : 0));
  const int group = st.NT * (st.kind == kStDown ? 4 : 1) * (D / 32);          // fragments of one weight group
  const int per = (st.NG / 8 * group + 255) / 256;                            // of a wavefront's part
  const int xcd = blockIdx.x & 7, f0 = ((blockIdx.x >> 3) * kWaves + wave) * per;
  int q = f0 / group, o = f0 - q * group;
  for (int j = 0; j < per && q * 8 + xcd < st.NG; ++j) {
    lds_direct16(W + ((size_t)(q * 8 + xcd) * group + o) * 64 + lane, sm.junk + wave * 64);
    if (++o == group) { o = 0; ++q; }
  }
}

// QKV epilogue of four tile rows n0..n0+3 of activation row m: where they go, and their rotary factors
struct QkvPos { int sec, h, dim, pos; bool low, ok; size_t head; float4 c0, c1; };
template <int D>
__device__ __forceinline__ QkvPos qkv_pos(const LayersArgs& a, const Smem& sm, int n0, int m) {
  constexpr int TPS = D / 16, H = D / 64;
  const int nt = n0 >> 4, nrow = n0 & 15;
  QkvPos p;
  p.sec = nt / TPS;
  const int ts = nt - p.sec * TPS, tt = ts & 3;
  p.h = ts >> 2;
  p.low = nrow < 8;
  const int pi = tt * 8 + (nrow & 7);
  p.dim = p.sec < 2 ? (p.low ? pi : 32 + pi) : tt * 16 + nrow;
  p.ok = false; p.pos = 0; p.head = 0;
  if (m < a.M) {
    const int b = m / a.R, len = sm.eff[b];
    p.ok = len >= 0;
    p.pos = len + (m - b * a.R);
    p.head = (size_t)sm.slot[b] * H + p.h;
  }
  if (p.sec < 2) {
    const float4* rp = reinterpret_cast<const float4*>(a.rope + (size_t)(p.ok ? p.pos : 0) * 32 + pi);
    p.c0 = rp[0]; p.c1 = rp[1];
  }
  return p;
}
// v: the values, pr: those of the tile rows 8 further
template <int D>
__device__ __forceinline__ void qkv_out(const LayersArgs& a, const LayerWts* w, rsrc_t rq, const QkvPos& p, int m, f32x4 v, f32x4 pr) {
  if (!p.ok) return;
  f32x4 o = v;
  if (p.sec < 2) {
    const f32x4 co = {p.c0.x, p.c0.z, p.c1.x, p.c1.z}, si = {p.c0.y, p.c0.w, p.c1.y, p.c1.w};
    o = p.low ? v * co - pr * si : pr * si + v * co;
  }
  if (p.sec == 0) {
    stc16(rq, ((unsigned)m * D + p.h * 64 + p.dim) * 4u, o);
  } else if (p.sec == 1) {
    st_coh((gptr<uint64_t>)(w->Kc + p.head * a.cap * 64 + kfrag(p.pos, p.dim)),
           (uint64_t)f2bf_pair(o[0], o[1]) | ((uint64_t)f2bf_pair(o[2], o[3]) << 32));
  } else {
#pragma unroll
    for (int e = 0; e < 4; ++e) st_coh(glob(w->Vt + p.head * a.cap * 64 + vfrag(p.pos, p.dim) + e * 8), f2bf(o[e]));
  }
}

// A residual-add projection's four columns n0.. of row m: the new residual u, its operand planes for the
// next norm (gain g) and its square sum; or, at the end of the pass, the fp32 row.
template <int D>
__device__ __forceinline__ void add_out(const LayersArgs& a, int cur, bool last, int m, int n0, unsigned xoff, int lane, f32x4 u,
                                        float4 g) {
  constexpr int NP = D / 16;
  const int Mp = a.mtiles * 16;
  if (last) {
    if (m < a.M) *reinterpret_cast<f32x4*>(a.x_out + (size_t)m * D + n0) = u;
    return;
  }
  const rsrc_t ro = make_rsrc(a.x[cur ^ 1], (size_t)Mp * D * 4), rp = make_rsrc(a.P[cur ^ 1], (size_t)Mp * D * 4);
  stc16(ro, xoff, u);
  planes4<D>(rp, (unsigned)Mp * D * 2u, m, n0, float4{u[0] * g.x, u[1] * g.y, u[2] * g.z, u[3] * g.w});
  float s = u[0] * u[0] + u[1] * u[1] + u[2] * u[2] + u[3] * u[3];
  s += lane_xor<16>(s); s += lane_xor<32>(s);
  if (lane < 16) st_coh(a.ssq[cur ^ 1] + (size_t)m * NP + (n0 >> 4), s);
}

// largest ring of at most `most` k-tiles that divides a group's KW, so that a slot means the same k-tiles in every group
constexpr int ring_depth(int KW, int most) {
  int d = most < KW ? most : KW;
  while (KW % d) --d;
  return d;
}
// One projection task: its weights stay in registers while it goes through its row groups; while a
// group's partial tiles are summed and stored, the next group's first activations are on their
// way.  cur: which of the two residual / plane / square-sum buffers holds the rows.  SPLIT: the contraction in four slices
// (FFN-down); the last of a tile's four tasks to finish adds them up in slice order.
template <int D, int NT, int MT, int KW, bool SPLIT, typename Wait, typename Claim>
__device__ __forceinline__ bool gemm_task(Smem& sm, const Wait& wait, const Claim& claim, int layer, int st_no, const LayerWts* w,
                                          int cur, bool last, Tile tl) {
  static_assert(NT * MT <= kWaves && MT <= 2, "a wavefront finishes at most one tile; sixteen threads per row");
  constexpr int NP = D / 16;                          // square sums per row
  constexpr bool WHOLE = KW > D / 256;                // FFN-down in one piece: one row group per task
  constexpr int DEPTH = ring_depth(KW, (NT * KW > 16 && !WHOLE ? 4 : 8) / MT);   // k-tiles of activations in flight
  const LayersArgs& a = fresh_args();
  const LayerStage& st = a.stage[st_no];
  const int tid = fresh(threadIdx.x), wave = uni(tid >> 6), lane = tid & 63, kind = st.kind;
  const int KT = KW * kWaves * (SPLIT ? 4 : 1), MTT = a.mtiles, Mp = MTT * 16;
  const bool normed = !SPLIT && (kind == kStQkv || kind == kStUp || kind == kStCq);
  const bool add = SPLIT || kind == kStO || kind == kStCo || kind == kStDown;
  const uint16_t* gain = kind == kStDown ? w->g_next : (kind == kStO && a.n_cond > 0) ? w->gc : w->g2;
  const uint4* const W = stage_weights(kind, w);
  const void* in = kind == kStDown ? a.U : (kind == kStO || kind == kStCo) ? a.AO : a.P[cur];
  const unsigned in_lo = (unsigned)Mp * KT * 64u;     // bytes of one plane
  const rsrc_t rin = make_rsrc(in, (size_t)in_lo * 2), rx = make_rsrc(a.x[cur], (size_t)Mp * D * 4);
  // What the finishing threads will need: wavefront w finishes tile w of a group (n-tile t, row tile
  // q).  None of it comes from the stage in front, so it is requested before the wait too.  (What is
  // loaded stays as it is until it is used: arithmetic here would wait for the load here.)
  const int t_ = wave / MT, q_ = wave - t_ * MT, nt = tl.ng * NT + t_, n0 = nt * 16 + (lane >> 4) * 4;
  uint4 xin = uint4{0, 0, 0, 0};
  u32x2 gn = {0, 0};
  QkvPos qp{};
  bool fin;
  int m;
  unsigned xoff;
  auto fin_loads = [&](int mg) {
    const int mt = mg * MT + q_;
    fin = wave < NT * MT && mt < MTT;
    m = mt * 16 + (lane & 15);
    xoff = ((unsigned)(mt * NP + nt) * 64u + lane) * 16u;
    if (add && !SPLIT && fin) xin = ldc16(rx, xoff);
    if (!SPLIT && kind == kStQkv && fin) qp = qkv_pos<D>(a, sm, n0, m);
  };
  // The weights are requested before the wait.  Wavefront 0 does the polling and its loads return
  // in order, so it asks for its share afterwards (they are in the L2 by then).
  uint4 wf[NT * KW];                                  // the weight fragments of this wavefront's share of a task
  const int kt0 = (SPLIT ? tl.ks * (KW * kWaves) : 0) + wave * KW;
  auto early = [&]() {
    load_weights<NT, KW>(W, tl.ng * NT, KT, kt0, lane, wf);
    if (add && wave < NT * MT) gn = gain_bits4(gain, n0);
    fin_loads(tl.mg0);
  };
  if (wave != 0) early();
  if (!wait()) return false;
  if (wave == 0) early();
  uint4 rb[DEPTH][MT][2];
  unsigned boff[MT];
  auto request = [&](int i) {
#pragma unroll
    for (int q = 0; q < MT; ++q) {
      rb[i % DEPTH][q][0] = ldc16(rin, boff[q], (i % KW) * 1024u);
      rb[i % DEPTH][q][1] = ldc16(rin, boff[q], (i % KW) * 1024u + in_lo);
    }
  };
  auto aim = [&](int mg) {
#pragma unroll
    for (int q = 0; q < MT; ++q) boff[q] = (unsigned)((min(mg * MT + q, MTT - 1) * KT + kt0) * 64 + lane) * 16u;
  };
  // sixteen threads per row add up its square sums
  uint4 ssv[(NP + 63) / 64];
  const int srow = tid >> 4, sj = tid & 15;
  const rsrc_t rs = make_rsrc(a.ssq[cur], (size_t)Mp * NP * 4);
  const bool sums = normed && srow < MT * 16;
  auto sum_loads = [&](int mg) {
    const int mm = min(mg * (MT * 16) + srow, Mp - 1);
#pragma unroll
    for (int c = 0; c < NP; c += 64)
      if (NP - c >= 64 || sj * 4 < NP - c) ssv[c / 64] = ldc16(rs, (unsigned)(mm * NP + c + sj * 4) * 4u);
  };
  aim(tl.mg0);
#pragma unroll
  for (int i = 0; i < DEPTH; ++i) request(i);
  const int claimed = claim();                        // (behind the requests: its wavefront's loads return in order)
  if (sums) sum_loads(tl.mg0);
  warm_next<D>(a, sm, layer, st_no, wave, lane);      // (behind everything the first group waits for)

  f32x4 acc[NT][MT];
  // the products of one group; MORE: each slot of the ring is refilled for the following group
  auto products = [&](auto MORE, int mg) {
#pragma unroll
    for (int t = 0; t < NT; ++t)
#pragma unroll
      for (int q = 0; q < MT; ++q) acc[t][q] = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int i = 0; i < KW; ++i) {
#pragma unroll
      for (int q = 0; q < MT; ++q) {
        const bf16x8 bh = __builtin_bit_cast(bf16x8, rb[i % DEPTH][q][0]);
        const bf16x8 bl = __builtin_bit_cast(bf16x8, rb[i % DEPTH][q][1]);
#pragma unroll
        for (int t = 0; t < NT; ++t)
          acc[t][q] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8, wf[t * KW + i]), bl, acc[t][q], 0, 0, 0);
#pragma unroll
        for (int t = 0; t < NT; ++t)
          acc[t][q] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8, wf[t * KW + i]), bh, acc[t][q], 0, 0, 0);
      }
      if (decltype(MORE)::value && i + DEPTH == KW) aim(mg + 1);
      if (i + DEPTH < KW || decltype(MORE)::value) request(i + DEPTH);
    }
  };
  // Two sets of partial tiles, so that one barrier per group is enough: a wavefront that is through
  // with a group goes on with the next one's products while others still finish tiles.
  for (int mg = tl.mg0; mg < tl.mg1; ++mg) {
    const int par = (mg - tl.mg0) & 1;
    f32x4* const red = reinterpret_cast<f32x4*>(sm.red) + par * (kWaves * 8 * 64);
    const bool more = !WHOLE && mg + 1 < tl.mg1;
    if (more) products(std::true_type{}, mg); else products(std::false_type{}, mg);
#pragma unroll
    for (int t = 0; t < NT; ++t)
#pragma unroll
      for (int q = 0; q < MT; ++q) red[(wave * (NT * MT) + t * MT + q) * 64 + lane] = acc[t][q];
    if (sums) {
      float x = 0.f;
#pragma unroll
      for (int c = 0; c < NP; c += 64)
        if (NP - c >= 64 || sj * 4 < NP - c) {
          const float4 y = __builtin_bit_cast(float4, ssv[c / 64]);
          x += (y.x + y.y) + (y.z + y.w);
        }
      x += lane_xor<8>(x); x += lane_xor<4>(x); x += lane_xor<2>(x); x += lane_xor<1>(x);
      if (sj == 0) sm.inv[par * 32 + srow] = 1.0f / sqrtf(x / (float)D + a.eps);
    }
    if (tid == kClaimer) sm.task = claimed;
    __syncthreads();
    if (fin) {
      f32x4 u = red[wave * 64 + lane];
#pragma unroll
      for (int k = 1; k < kWaves; ++k) u += red[(k * (NT * MT) + wave) * 64 + lane];
      if (normed) u *= sm.inv[par * 32 + q_ * 16 + (lane & 15)];
      if (SPLIT) {
        stc16(make_rsrc(a.gpart, (size_t)Mp * D * 16), xoff + tl.ks * ((unsigned)Mp * D * 4u), u);
      } else if (kind == kStQkv) {
        f32x4 pr;
#pragma unroll
        for (int e = 0; e < 4; ++e) pr[e] = lane_xor<32>(u[e]);
        qkv_out<D>(a, w, make_rsrc(a.q, (size_t)a.M * D * 4), qp, m, u, pr);
      } else if (kind == kStCq) {
        if (m < a.M) stc16(make_rsrc(a.q, (size_t)a.M * D * 4), ((unsigned)m * D + n0) * 4u, u);
      } else if (kind == kStUp) {
        planes4<4 * D>(make_rsrc(a.U, (size_t)Mp * D * 16), (unsigned)Mp * D * 8u, m, n0,
                       float4{gelu_erf_f(u[0]), gelu_erf_f(u[1]), gelu_erf_f(u[2]), gelu_erf_f(u[3])});
      } else {
        add_out<D>(a, cur, last, m, n0, xoff, lane, u + __builtin_bit_cast(f32x4, xin), gain4(gn));
      }
    }
    if (more) {
      fin_loads(mg + 1);
      if (sums) sum_loads(mg + 1);
    }
  }
  if (SPLIT) {
    // the last of the four slices' tasks to get here adds them up, group by group
    const rsrc_t rp = make_rsrc(a.gpart, (size_t)Mp * D * 16);
    const unsigned pk = (unsigned)Mp * D * 4u;        // bytes of one slice
    __builtin_amdgcn_s_waitcnt(0x0F70);
    __syncthreads();
    if (tid == 0) {
      uint32_t* tk = a.gtickets + tl.ng * st.MC + tl.mc;
      const uint32_t old = __hip_atomic_fetch_add(tk, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
      sm.last = old == 3u;
      if (old == 3u) st_coh(tk, 0u);
    }
    __syncthreads();
    if (uni(sm.last) != 0 && wave < NT * MT) {
      constexpr int B = 2;                            // groups requested together
      for (int mg = tl.mg0; mg < tl.mg1; mg += B) {
        f32x4 s[B][5];
#pragma unroll
        for (int j = 0; j < B; ++j) {
          const int mt = min(min(mg + j, tl.mg1 - 1) * MT + q_, MTT - 1);
          const unsigned o = ((unsigned)(mt * NP + nt) * 64u + lane) * 16u;
#pragma unroll
          for (int k = 0; k < 4; ++k) s[j][k] = __builtin_bit_cast(f32x4, ldc16(rp, o, k * pk));
          s[j][4] = __builtin_bit_cast(f32x4, ldc16(rx, o));
        }
#pragma unroll
        for (int j = 0; j < B; ++j) {
          const int mt = (mg + j) * MT + q_;
          if (mg + j < tl.mg1 && mt < MTT)
            add_out<D>(a, cur, last, mt * 16 + (lane & 15), n0, ((unsigned)(mt * NP + nt) * 64u + lane) * 16u, lane,
                       (((s[j][0] + s[j][1]) + s[j][2]) + s[j][3]) + s[j][4], gain4(gn));
        }
      }
    }
  }
  return true;
}

// ---- attention --------------------------------------------------------------------
// one (sequence, query tile, head) unit and a chunk of it
struct Chunk { int u, h, c, NC; };
struct UnitRows { int n, R, row0, Ltot; size_t head; };

template <int D>
__device__ __forceinline__ UnitRows unit_rows(const LayersArgs& a, const Smem& sm, int u, int h, bool cross) {
  const int QT = (a.R + 15) >> 4, b = u / QT, qt = u - b * QT;
  UnitRows r;
  r.n = sm.eff[b] + qt * 16;
  r.R = min(16, a.R - qt * 16);
  r.row0 = b * a.R + qt * 16;
  r.Ltot = cross ? a.n_cond : r.n + r.R;
  r.head = (size_t)sm.slot[b] * (D / 64) + h;
  return r;
}

// finished rows of a unit (O^T fragments o, row sums l) -> operand planes of the projection that follows
template <int D>
__device__ __forceinline__ void attn_out(const LayersArgs& a, const UnitRows& ur, int h, int lane, float l, const f32x4 (&o)[4]) {
  const int r = lane & 15, g = lane >> 4;
  if (r >= ur.R) return;
  const rsrc_t ro = make_rsrc(a.AO, (size_t)a.mtiles * 16 * D * 4);
  const float inv = 1.0f / l;
#pragma unroll
  for (int dt = 0; dt < 4; ++dt)
    planes4<D>(ro, (unsigned)a.mtiles * 32u * D, ur.row0 + r, h * 64 + dt * 16 + g * 4,
               float4{o[dt][0] * inv, o[dt][1] * inv, o[dt][2] * inv, o[dt][3] * inv});
}

template <int D, typename Wait, typename Claim>
__device__ __forceinline__ bool attn_task(Smem& sm, const Wait& wait, const Claim& claim, const LayerWts* w, bool cross, int task) {
  constexpr int H = D / 64;
  const LayersArgs& a = fresh_args();
  const int tid = fresh(threadIdx.x), wave = uni(tid >> 6), lane = tid & 63, r = lane & 15, g = lane >> 4;
  const int QT = (a.R + 15) >> 4, NU = a.n_seq * QT, NCX = (a.n_cond + 63) >> 6;
  const int total = cross ? NU * NCX * H : sm.pre[NU] * H;
  auto start = [&](int x) {
    Chunk k;
    if (cross) {
      k.NC = NCX;
      k.u = x / (NCX * H);
      const int rem = x - k.u * (NCX * H);
      k.h = rem / NCX; k.c = rem - k.h * NCX;
    } else {
      int cnt = 0;
      for (int base = 0; base < NU; base += 64) {
        const int i = base + lane;
        cnt += __popcll(__ballot(i < NU && sm.pre[i] * H <= x));
      }
      k.u = uni(cnt - 1);
      const int p = uni(sm.pre[k.u]);
      k.NC = uni(sm.pre[k.u + 1]) - p;
      const int rem = x - p * H;
      k.h = rem / k.NC; k.c = rem - k.h * k.NC;
    }
    return k;
  };
  // Where whole units make shares that are as good as equal (many units, or few of equal length),
  // the shares begin and end at units and nothing has to be merged across tasks, which costs the
  // stage 4 us at its end.
  const bool whole = cross ? NU * H % kTasksPerAttn == 0 : sm.pre[NU + 1] != 0;
  const int nsh = min(kTasksPerAttn, total);          // (no empty share between two others)
  auto share = [&](int t) {
    if (t >= nsh) return total;
    const int x = (int)((long)t * total / nsh);
    if (!whole) return x;
    const Chunk k = start(x);
    return x - k.c + (2 * k.c >= k.NC ? k.NC : 0);
  };
  const int s0 = share(task), s1 = share(task + 1);
  const int x0 = s0 + (s1 - s0) * wave / kWaves, x1 = s0 + (s1 - s0) * (wave + 1) / kWaves;
  const uint16_t* Kb = cross ? w->Kx : w->Kc;
  const uint16_t* Vb = cross ? w->Vx : w->Vt;
  const int cap = cross ? a.cap_cross : a.cap;
  const rsrc_t rq = make_rsrc(a.q, (size_t)a.M * D * 4);
  float* slots = sm.slots;
  if (lane < 2) sm.meta[wave * 2 + lane][0] = -1;

  auto next = [&](const Chunk& k) {
    Chunk n = k;
    if (++n.c == n.NC) {
      n.c = 0;
      if (++n.h == H) {
        n.h = 0;
        ++n.u;
        if (!cross) {
          while (n.u + 1 < NU && uni(sm.pre[n.u + 1]) == uni(sm.pre[n.u])) ++n.u;
          n.NC = uni(sm.pre[n.u + 1]) - uni(sm.pre[n.u]);
        }
      }
    }
    return n;
  };

  // The first chunk is requested before the wait (by the wavefronts that do not poll), unless it
  // holds positions this very pass writes.
  const bool any = x0 < x1;
  Chunk cur{0, 0, 0, 1};
  UnitRows ur{};
  if (any) { cur = start(x0); ur = unit_rows<D>(a, sm, cur.u, cur.h, cross); }
  uint4 ka[4][2], va[4][2];
  const bool early = any && wave != 0 && (cross || (cur.c + 1) * 64 <= sm.eff[cur.u / QT]);

  auto load_kv = [&](const Chunk& k, const UnitRows& u, uint4 (&kf)[4][2], uint4 (&vf)[4][2]) {
    const size_t o = (u.head * (size_t)cap + (k.c << 6)) * 64 + lane * 8;
#pragma unroll
    for (int t = 0; t < 4; ++t)
#pragma unroll
      for (int j = 0; j < 2; ++j) {
        kf[t][j] = ldg16(Kb + o + (t * 2 + j) * 512);
        vf[t][j] = ldg16(Vb + o + (t * 2 + j) * 512);
      }
  };
  if (early) load_kv(cur, ur, ka, va);
  if (!wait()) return false;
  if (any && !early) load_kv(cur, ur, ka, va);
  const int claimed = claim();
  if (any) {
    bf16x8 qh[2], ql[2];
    auto queries = [&]() {
      float4 x[4];
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        const unsigned o = ((unsigned)(ur.row0 + min(r, ur.R - 1)) * D + cur.h * 64 + (i >> 1) * 32 + g * 8 + (i & 1) * 4) * 4u;
        x[i] = __builtin_bit_cast(float4, ldc16(rq, o));
      }
      split_queries(x, qh, ql);
    };
    float m_run = -INFINITY, l_run = 0.f;
    f32x4 o[4];
#pragma unroll
    for (int dt = 0; dt < 4; ++dt) o[dt] = f32x4{0.f, 0.f, 0.f, 0.f};
    int seg0 = cur.c, which = 0, x = x0;
    uint4 kb2[4][2], vb2[4][2];
    queries();
    // one chunk out of (kf, vf), the next one on its way into (kn, vn); false when the range is done
    auto step = [&](uint4 (&kf)[4][2], uint4 (&vf)[4][2], uint4 (&kn)[4][2], uint4 (&vn)[4][2]) {
      const bool more = x + 1 < x1;
      const Chunk nx = more ? next(cur) : cur;        // (at the end the same chunk again, so that no load sits behind a branch)
      const UnitRows un = unit_rows<D>(a, sm, nx.u, nx.h, cross);
      load_kv(nx, un, kn, vn);
      const int lim = r < ur.R ? (cross ? ur.Ltot : ur.n + r + 1) : 0;
      attn_chunk(kf, vf, qh, ql, cur.c << 6, g, r < ur.R, lim, cross ? ur.Ltot : ur.n + 1, ur.Ltot, a.scale_log2, m_run, l_run, o);
      if (!more || nx.u != cur.u || nx.h != cur.h) {  // this wavefront's piece of the unit ends here
        if (seg0 == 0 && cur.c + 1 == cur.NC) {
          attn_out<D>(a, ur, cur.h, lane, l_run, o);
        } else {
          const int sl = wave * 2 + which;
          float* p = slots + sl * kSlotFloats;
          if (g == 0) { p[r] = m_run; p[16 + r] = l_run; }
#pragma unroll
          for (int dt = 0; dt < 4; ++dt) *reinterpret_cast<f32x4*>(p + 32 + (dt * 64 + lane) * 4) = o[dt];
          if (lane == 0) { sm.meta[sl][1] = seg0; sm.meta[sl][2] = cur.c + 1; sm.meta[sl][0] = cur.u * H + cur.h; }
        }
        which = 1;                                    // (whole units in between need no slot)
        seg0 = 0; m_run = -INFINITY; l_run = 0.f;
#pragma unroll
        for (int dt = 0; dt < 4; ++dt) o[dt] = f32x4{0.f, 0.f, 0.f, 0.f};
        cur = nx; ur = un;
        if (more) queries();
      } else {
        cur = nx; ur = un;
      }
      ++x;
      return more;
    };
    while (true) {
      if (!step(ka, va, kb2, vb2)) break;
      if (!step(kb2, vb2, ka, va)) break;
    }
  }
  if (tid == kClaimer) sm.task = claimed;
  __syncthreads();
  // pieces of one unit lie in consecutive slots; group i of them is merged by wavefront i
  int grp = 0;
  for (int s = 0; s < kWaves * 2;) {
    const int key = uni(sm.meta[s][0]);
    if (key < 0) { ++s; continue; }
    int e = s + 1, last = s;                          // (slots of other wavefronts in between may be empty)
    while (e < kWaves * 2) {
      const int k2 = uni(sm.meta[e][0]);
      if (k2 >= 0 && k2 != key) break;
      if (k2 == key) last = e;
      ++e;
    }
    if (grp % kWaves == wave) {
      const int u = key / H, h = key - u * H;
      const UnitRows ur = unit_rows<D>(a, sm, u, h, cross);
      const int NC = cross ? NCX : uni(sm.pre[u + 1]) - uni(sm.pre[u]);
      const int c0 = uni(sm.meta[s][1]), c1 = uni(sm.meta[last][2]);
      float Mx = -INFINITY, L = 0.f;
      for (int i = s; i <= last; ++i)
        if (uni(sm.meta[i][0]) == key) Mx = fmaxf(Mx, slots[i * kSlotFloats + r]);
      f32x4 o[4];
#pragma unroll
      for (int dt = 0; dt < 4; ++dt) o[dt] = f32x4{0.f, 0.f, 0.f, 0.f};
      for (int i = s; i <= last; ++i)
        if (uni(sm.meta[i][0]) == key) {
          const float* p = slots + i * kSlotFloats;
          const float mi = p[r], f = mi == -INFINITY ? 0.f : exp2_hw(mi - Mx);
          L += p[16 + r] * f;
#pragma unroll
          for (int dt = 0; dt < 4; ++dt) o[dt] += *reinterpret_cast<const f32x4*>(p + 32 + (dt * 64 + lane) * 4) * f;
        }
      if (c0 == 0 && c1 == NC) {
        attn_out<D>(a, ur, h, lane, L, o);
      } else {
        // the unit spans tasks: leave the piece in memory, the last task to do so merges them.  A
        // task's piece of a unit that began in an earlier task is its piece 0, else its piece 1.
        const int first = (cross ? u * NCX : uni(sm.pre[u])) * H + h * NC;       // the unit's chunks in the list
        const int t0 = (int)((((long)first + 1) * nsh - 1) / total);
        const int t1 = (int)(((long)(first + NC) * nsh - 1) / total);
        const rsrc_t rp = make_rsrc(a.part, (size_t)kTasksPerAttn * 2 * kSlotFloats * 4);
        const unsigned pb = (unsigned)(task * 2 + (c0 == 0 ? 1 : 0)) * (kSlotFloats * 4u);
        if (g == 0) {
          __builtin_amdgcn_raw_buffer_store_b32(__float_as_uint(Mx), rp, (int)(pb + r * 4u), 0, kCoh);
          __builtin_amdgcn_raw_buffer_store_b32(__float_as_uint(L), rp, (int)(pb + 64u + r * 4u), 0, kCoh);
        }
#pragma unroll
        for (int dt = 0; dt < 4; ++dt) stc16(rp, pb + 128u + (dt * 64 + lane) * 16u, o[dt]);
        __builtin_amdgcn_s_waitcnt(0);
        uint32_t old = 0;
        if (lane == 0) {
          uint32_t* tk = a.tickets + key;
          old = __hip_atomic_fetch_add(tk, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
          if (old == (uint32_t)(t1 - t0)) st_coh(tk, 0u);
        }
        if (uni((int)old) == t1 - t0) {
          float Mg = -INFINITY, Lg = 0.f;
          f32x4 og[4];
#pragma unroll
          for (int dt = 0; dt < 4; ++dt) og[dt] = f32x4{0.f, 0.f, 0.f, 0.f};
          constexpr int B = 3;                        // pieces requested together
          for (int tb = t0; tb <= t1; tb += B) {
            float mi[B], li[B];
            f32x4 oi[B][4];
#pragma unroll
            for (int i = 0; i < B; ++i) {
              const int t = min(tb + i, t1);
              const unsigned p = (unsigned)(t * 2 + (t == t0 ? 1 : 0)) * (kSlotFloats * 4u);
              mi[i] = __uint_as_float(__builtin_amdgcn_raw_buffer_load_b32(rp, (int)(p + r * 4u), 0, kCoh));
              li[i] = __uint_as_float(__builtin_amdgcn_raw_buffer_load_b32(rp, (int)(p + 64u + r * 4u), 0, kCoh));
#pragma unroll
              for (int dt = 0; dt < 4; ++dt) oi[i][dt] = __builtin_bit_cast(f32x4, ldc16(rp, p + 128u + (dt * 64 + lane) * 16u));
            }
#pragma unroll
            for (int i = 0; i < B; ++i) {
              if (tb + i > t1) continue;
              const float mn = fmaxf(Mg, mi[i]), mu = mn == -INFINITY ? 0.f : mn;
              const float fo = exp2_hw(Mg - mu), fi = exp2_hw(mi[i] - mu);
              Lg = Lg * fo + li[i] * fi;
#pragma unroll
              for (int dt = 0; dt < 4; ++dt) og[dt] = og[dt] * fo + oi[i][dt] * fi;
              Mg = mn;
            }
          }
          attn_out<D>(a, ur, h, lane, Lg, og);
        }
      }
    }
    ++grp;
    s = last + 1;
  }
  return true;
}

static_assert(sizeof(Smem) <= 160 * 1024, "one compute unit's LDS");

// ---------------------------------------------------------------------------
template <int D>
__global__ __launch_bounds__(kThreads) void k_layers(const LayersArgs a) {
  constexpr int KW = D / 256, KWF = 4 * KW;
  extern __shared__ __align__(16) unsigned char raw[];
  Smem& sm = *reinterpret_cast<Smem*>(raw);
  const int tid = threadIdx.x, wave = uni(tid >> 6), lane = tid & 63;
  const int q = blockIdx.x & (kQueues - 1);
  uint32_t* const claim = a.ctrl + q * kQueueStride;
  uint32_t* const done = a.ctrl + (kQueues + q) * kQueueStride;
  const int n_tasks = a.kv_only ? a.per_layer * (a.L - 1) + a.stage[1].base : a.per_layer * a.L;
  auto claim_next = [&]() {
    return (int)__hip_atomic_fetch_add(claim, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) * kQueues + q;
  };
  if (tid == 0) { sm.task = claim_next(); sm.abort = 0; }
  {
    const int NU = a.n_seq * ((a.R + 15) >> 4);
    for (int i = tid; i <= NU + 1; i += kThreads) sm.pre[i] = a.unit_pre[i];
    for (int i = tid; i < a.n_seq; i += kThreads) { sm.eff[i] = a.eff_len[i]; sm.slot[i] = a.slot[i]; }
    for (int i = tid; i < (int)(a.L * sizeof(LayerWts) / 8); i += kThreads)
      reinterpret_cast<uint64_t*>(sm.wts)[i] = reinterpret_cast<const uint64_t*>(a.wts)[i];
  }
  __syncthreads();
  int task = uni(sm.task), ready = 0;
  TaskPos p = task_pos(a, task < n_tasks ? task : 0, 0);
  while (task < n_tasks) {
    const LayersArgs& a = fresh_args();
    const int lane = fresh(tid & 63);
    const LayerStage& st = a.stage[p.st];
    const int need = p.layer * a.per_layer + st.base;
    const bool att = st.kind == kStAtt || st.kind == kStCatt;
    Tile tl{};
    const bool real = att || tile_pos(st, p.idx, &tl);
    // every task of the stages in front is done?
    auto wait = [&]() {
      if (need > ready) {
        if (wave == 0) {
          uint64_t t0 = 0;
          for (int spin = 0;; ++spin) {
            int v = lane < kQueues ? (int)ld_coh(a.ctrl + (kQueues + lane) * kQueueStride) : 0;
            v += lane_xor<8>(v); v += lane_xor<4>(v); v += lane_xor<2>(v); v += lane_xor<1>(v);
            if (uni(v) >= need) break;
            if ((spin & 255) == 255) {
              const uint64_t now = __builtin_amdgcn_s_memrealtime();
              if (t0 == 0) t0 = now;
              else if (now - t0 > kWaitTicks) { if (lane == 0) sm.abort = 1; break; }
            }
          }
        }
        __syncthreads();
        ready = need;
      }
      return uni(sm.abort) == 0;
    };
    // The next claim comes only now, when every workgroup has finished the stage in front: each holds
    // one task ahead then, and a fast one cannot take a slow one's share of this stage.
    auto claim_now = [&]() { return tid == kClaimer ? claim_next() : 0; };
    const LayerWts* w = sm.wts + p.layer;
    const int cur = (p.layer * a.adds + st.adds_before) & 1;
    bool ok = true;
    if (att) {
      ok = attn_task<D>(sm, wait, claim_now, w, st.kind == kStCatt, p.idx);
    } else if (real) {
      const bool last = st.kind == kStDown && p.layer == a.L - 1;
#define XSM_GT(NT, MT, KWX, SPLIT) ok = gemm_task<D, NT, MT, KWX, SPLIT>(sm, wait, claim_now, p.layer, p.st, w, cur, last, tl)
      if (st.kind == kStDown && st.KS == 1) {
        if (st.MT == 1) XSM_GT(1, 1, KWF, false); else XSM_GT(1, 2, KWF, false);
      } else if (st.kind == kStDown) {
        if (st.NT == 2) XSM_GT(2, 2, KW, true); else if (st.MT == 1) XSM_GT(4, 1, KW, true); else XSM_GT(4, 2, KW, true);
      } else if (st.NT == 1) {
        if (st.MT == 1) XSM_GT(1, 1, KW, false); else XSM_GT(1, 2, KW, false);
      } else if (st.NT == 2) {
        if (st.MT == 1) XSM_GT(2, 1, KW, false); else XSM_GT(2, 2, KW, false);
      } else {
        if (st.MT == 1) XSM_GT(4, 1, KW, false); else XSM_GT(4, 2, KW, false);
      }
#undef XSM_GT
    } else {
      ok = wait();
      const int c = claim_now();
      if (tid == kClaimer) sm.task = c;
      __syncthreads();
    }
    if (!ok) break;
    __builtin_amdgcn_s_waitcnt(0x0F70);               // vmcnt(0): this wavefront's stores have arrived
    __syncthreads();
    if (tid == 0) __hip_atomic_fetch_add(done, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    task = uni(sm.task);
    if (task < n_tasks) p = task_pos(a, task, p.layer);
  }
  if (uni(sm.abort) && wave == 0) {                   // a wait gave up: nobody may use this pass
    for (int b = lane; b < a.n_seq; b += 64) {
      st_coh(a.eff_len_w + b, -1);
      if (a.wflags) st_coh(a.wflags + b, (uint32_t)XSM_FLAG_DEVICE_TIMEOUT);
    }
    if (lane == 0) {
      st_coh(a.err, 0x4C000000u | (uint32_t)task);
      if (a.err_small) st_coh(a.err_small, 0x4C000000u | (uint32_t)task);
    }
  }
}

// Tile sizes, slices and row chunks of one projection: least time by a model fitted to measured
// stages.  A stage costs its latency (request, partial-tile sum, store), and for every row group a
// task goes through the activation bytes it pulls through its compute unit's L2 port.
void layers_tile(int ntiles, int mtiles, int kbytes, bool down, LayerStage* st) {
  static const int cand[][3] = {{1, 1, 1}, {1, 2, 1}, {2, 1, 1}, {2, 2, 1}, {4, 1, 1}, {4, 2, 1}};
  static const int cand_down[][3] = {{1, 1, 1}, {1, 2, 1}, {2, 2, 4}, {4, 1, 4}, {4, 2, 4}};
  double best = 1e30;
  for (int i = 0; i < (down ? 5 : 6); ++i) {
    const int* c = down ? cand_down[i] : cand[i];
    const int nt = c[0], mt = c[1], ks = c[2];
    if (ntiles % (nt * 8)) continue;
    const int NG = ntiles / nt, MG = (mtiles + mt - 1) / mt;
    int MC = 256 / (NG * ks);                         // row chunks that still give one task per workgroup
    if (MC < 1) MC = 1;
    if (MC > MG || (down && ks == 1)) MC = MG;
    const int rounds = (NG * MC * ks + 255) / 256, groups = (MG + MC - 1) / MC;
    const double stream = (double)kbytes / ks * mt * 64 / 95e3 + 0.08 * nt * mt;
    const double us = rounds * (1.9 + groups * stream + (ks > 1 ? 2.0 + 0.5 * (groups - 1) : 0.0) + 0.4 * (groups - 1));
    if (us < best) { best = us; st->NT = nt; st->MT = mt; st->KS = ks; st->MC = MC; st->NG = NG; st->MG = MG; }
  }
}

}  // namespace

bool layers_supported(int D, int F, int L) { return L <= kMaxLayers && (D == 1024 || D == 1536) && F == 4 * D; }
bool layers_usable(int n_seq, int R) {
  const int M = n_seq * R;
  return M > 16 && M <= kLayersMaxRows && n_seq <= kMaxSeq && n_seq * ((R + 15) / 16) <= kMaxUnits;
}
size_t layers_ctrl_bytes() { return (size_t)2 * kQueues * kQueueStride * 4 + (size_t)(kMaxUnits + 64) * 4; }
size_t layers_part_bytes() { return (size_t)kTasksPerAttn * 2 * kSlotFloats * 4; }

void launch_layers_begin(const LayersBegin& b, hipStream_t s) {
  hipLaunchKernelGGL(k_layers_begin, dim3(b.n_seq * b.R + 1), dim3(256), 0, s, b);
}

void launch_layers(LayersBegin b, LayersArgs a, int D, hipStream_t s) {
  TraceScope trace_("fattn", s);               // (its kernel class: attention and everything between)
  const int M = b.n_seq * b.R;
  a.M = M; a.mtiles = (M + 15) / 16; a.n_seq = b.n_seq; a.R = b.R;
  b.d = D; b.H = D / 64; b.x = a.x[0]; b.planes = a.P[0]; b.ssq = a.ssq[0]; b.ctrl = a.ctrl; b.unit_pre = (int32_t*)(a.ctrl + 2 * kQueues * kQueueStride);
  a.unit_pre = b.unit_pre;
  int ns = 0, base = 0, adds = 0;
  auto gemm = [&](int kind, int ntiles, int kbytes) {
    LayerStage& st = a.stage[ns++];
    st.kind = kind;
    layers_tile(ntiles, a.mtiles, kbytes, kind == kStDown, &st);
    st.base = base; st.adds_before = adds;
    st.count = (st.NG * st.MC * st.KS + kQueues - 1) / kQueues * kQueues;
    base += st.count;
    if (kind == kStO || kind == kStCo || kind == kStDown) ++adds;
  };
  auto attn = [&](int kind) {
    LayerStage& st = a.stage[ns++];
    st = LayerStage{kind, 1, 1, 1, 1, 1, 1, base, kTasksPerAttn, adds};
    base += kTasksPerAttn;
  };
  gemm(kStQkv, 3 * D / 16, D); attn(kStAtt); gemm(kStO, D / 16, D);
  if (a.n_cond > 0) { gemm(kStCq, D / 16, D); attn(kStCatt); gemm(kStCo, D / 16, D); }
  gemm(kStUp, 4 * D / 16, D); gemm(kStDown, D / 16, 4 * D);
  a.n_stages = ns; a.per_layer = base; a.adds = adds;
  b.partition = 1;
  launch_layers_begin(b, s);
  auto go = [&](auto kfn) {
    allow_dynamic_lds((const void*)kfn, sizeof(Smem));
    hipLaunchKernelGGL(kfn, dim3(256), dim3(kThreads), sizeof(Smem), s, a);
  };
  if (D == 1024) go(k_layers<1024>); else go(k_layers<1536>);
}

}  // namespace xsm
