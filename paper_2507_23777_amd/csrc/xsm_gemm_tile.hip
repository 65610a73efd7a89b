// Projections of large passes (more rows than the persistent layers kernel takes: prefills of
// thousands of rows, very large batches) on bf16 MFMA (gfx950).
//
// Here a projection is matrix-core work: every fp32 activation enters as a bf16 hi + lo operand pair
// against the same weight fragment, so 8192 rows x 1024 x 4096 are 137 GFLOP of MFMA.  What bounded the
// kernel this one replaces was operand delivery: weight fragments went from L2 to registers once
// per pair of wavefronts, activations through registers into LDS, one stage ahead (200 us for that
// projection, 0.7 PFLOP/s issued).  Here
//   - a workgroup of eight wavefronts, two per SIMD, computes 256 (or 128) weight rows x 128
//     activation rows; a wavefront holds 4 x 4 (or 4 x 2) accumulator tiles, so a k-tile costs it 12 (8)
//     fragment reads from LDS for 32 (16) MFMAs.  (One wavefront per SIMD cannot keep the matrix
//     core busy: 16x16x32 MFMAs out of registers alone run at 1.26 PFLOP/s from four wavefronts
//     per compute unit and at 2.13 from eight.);
//   - both operands are stored in fragment order, so they go from L2 straight into LDS (1 KB per
//     request, no registers, no bank conflicts when read back), three k-tiles ahead in four
//     buffers; the fragments of the next k-tile are read while this one's are multiplied; one barrier
//     per k-tile;
//   - the buffers are separate LDS arrays and the loop is unrolled over them: the compiler can tell
//     then that a fragment read does not touch the requests in flight (out of one array it would
//     wait for all of them before every read).
// RMSNorm is folded into the neighbours as in xsm_layers.hip: a residual-add projection writes its
// rows as operand planes multiplied by the next norm's gain, with one square sum per row and 16
// columns; its consumer multiplies its products by the row's 1 / rms.  Projections with few blocks cut
// the contraction into slices whose partial tiles the last one to finish adds up in slice order.
#include "xsm_device.h"
#include "xsm_internal.h"

namespace xsm {

namespace {

typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef float f32x4 __attribute__((ext_vector_type(4)));

constexpr int kTileM = 128;                            // activation rows of a workgroup

__device__ __forceinline__ void lds_direct16(const void* gptr, void* lds) {
  __builtin_amdgcn_global_load_lds((const __attribute__((address_space(1))) void*)gptr,
                                   (__attribute__((address_space(3))) void*)lds, 16, 0, 0);
}
__device__ __forceinline__ float gelu_erf_f(float x) { return 0.5f * x * (1.0f + erff(x * 0.70710678118654752f)); }
__device__ __forceinline__ float4 gain4(const uint16_t* g, int n) {
  const uint2 x = *reinterpret_cast<const uint2*>(g + n);
  return float4{__uint_as_float(x.x << 16), __uint_as_float(x.x & 0xFFFF0000u), __uint_as_float(x.y << 16),
                __uint_as_float(x.y & 0xFFFF0000u)};
}

// the four buffers: weight fragments, then the hi and the lo fragments of the activations
__shared__ uint4 tile_s0[(16 + 16) * 64], tile_s1[(16 + 16) * 64], tile_s2[(16 + 16) * 64], tile_s3[(16 + 16) * 64];
__shared__ float tile_inv[kTileM];
__shared__ int tile_last;

// four columns n0.. of row m of a finished product v
__device__ __forceinline__ void tile_out(const TileGemm& g, int nt, int mt, int lane, f32x4 v) {
  const int n0 = nt * 16 + (lane >> 4) * 4, m = mt * 16 + (lane & 15);
  switch (g.kind) {
    case kTileQkv: {
      f32x4 pr;
#pragma unroll
      for (int e = 0; e < 4; ++e) pr[e] = lane_xor<32>(v[e]);     // tile rows +- 8
      const int tps = g.K / 16, sec = nt / tps, ts = nt - sec * tps, h = ts >> 2, tt = ts & 3, nrow = n0 & 15;
      if (m >= g.M) return;
      const int b = m / g.R, j = m - b * g.R, len = g.eff_len[b];
      if (len < 0) return;
      const int pos = len + j, pi = tt * 8 + (nrow & 7);
      const bool low = nrow < 8;
      const size_t head = ((size_t)g.slot[b] * g.H + h) * g.cap * 64;
      f32x4 o = v;
      if (sec < 2) {
        const float4* rp = reinterpret_cast<const float4*>(g.rope + (size_t)pos * 32 + pi);
        const float4 c0 = rp[0], c1 = rp[1];
        const f32x4 co = {c0.x, c0.z, c1.x, c1.z}, si = {c0.y, c0.w, c1.y, c1.w};
        o = low ? v * co - pr * si : pr * si + v * co;
        const int dim = low ? pi : 32 + pi;
        if (sec == 0) *reinterpret_cast<f32x4*>(g.Y + (size_t)m * g.K + h * 64 + dim) = o;
        else *reinterpret_cast<uint2*>(g.Kc + head + kfrag(pos, dim)) = uint2{f2bf_pair(o[0], o[1]), f2bf_pair(o[2], o[3])};
      } else {
        uint16_t* vp = g.Vc + head + vfrag(pos, tt * 16 + nrow);
#pragma unroll
        for (int e = 0; e < 4; ++e) vp[e * 8] = f2bf(o[e]);
      }
      return;
    }
    case kTileStore:
      if (m < g.M) *reinterpret_cast<f32x4*>(g.Y + (size_t)m * g.N + n0) = v;
      return;
    case kTileGelu:
      plane_store4(g.Y, g.M, g.N, m, n0, float4{gelu_erf_f(v[0]), gelu_erf_f(v[1]), gelu_erf_f(v[2]), gelu_erf_f(v[3])});
      return;
    default: {                                         // residual add: x in tile order, updated in place
      f32x4* x = reinterpret_cast<f32x4*>(g.x) + ((size_t)mt * (g.N / 16) + nt) * 64 + lane;
      const f32x4 u = *x + v;
      if (g.x_out) {                                   // the pass's result: fp32 rows
        if (m < g.M) *reinterpret_cast<f32x4*>(g.x_out + (size_t)m * g.N + n0) = u;
        return;
      }
      *x = u;
      const float4 gn = gain4(g.gain, n0);
      plane_store4(g.P, g.M, g.N, m, n0, float4{u[0] * gn.x, u[1] * gn.y, u[2] * gn.z, u[3] * gn.w});
      float s = u[0] * u[0] + u[1] * u[1] + u[2] * u[2] + u[3] * u[3];
      s += lane_xor<16>(s); s += lane_xor<32>(s);
      if (lane < 16) g.ssq_out[(size_t)m * (g.N / 16) + nt] = s;
    }
  }
}

// NWN wavefronts along the weight rows (four tiles each), 8 / NWN along the activation rows (WM tiles each)
template <int NWN>
__global__ __launch_bounds__(512) void k_gemm_tile(const TileGemm g) {
  constexpr int WN = 4, WM = NWN;                      // (8 / NWN wavefronts x WM tiles = eight row tiles)
  constexpr int NTB = NWN * WN, FR = NTB + 16, PW = FR / 8;    // weight tiles per block, fragments per k-tile, of a wavefront
  const int tid = threadIdx.x, wave = __builtin_amdgcn_readfirstlane(tid >> 6), lane = tid & 63;
  const int wn = wave % NWN, wm = wave / NWN;
  const int KT = g.K / 32, MTT = (g.M + 15) >> 4, NB = g.N / (16 * NTB), MB = (MTT + 7) >> 3, T = NB * MB;
  // An XCD's blocks are neighbours (workgroup ids go round the XCDs): eight row blocks by as many
  // column blocks as run together share their operands in its L2.
  int L = blockIdx.x / g.KS;
  const int ks = blockIdx.x - L * g.KS;
  if ((T & 7) == 0) L = (L & 7) * (T >> 3) + (L >> 3);
  const int gr = L / (8 * NB), rem = L - gr * 8 * NB, gw = min(8, MB - gr * 8);
  const int nb = rem / gw, mb = gr * 8 + rem - nb * gw;
  const int nt0 = nb * NTB, mt0 = mb * 8;
  const int steps = KT / g.KS, kt0 = ks * steps;

  // this wavefront's fragments of a k-tile: PW consecutive ones of {weights, hi rows, lo rows}
  const uint4* src[PW];
#pragma unroll
  for (int j = 0; j < PW; ++j) {
    const int f = wave * PW + j;
    if (f < NTB) src[j] = g.W + ((size_t)(nt0 + f) * KT + kt0) * 64;
    else {
      const int q = f - NTB, mt = min(mt0 + (q & 7), MTT - 1);
      src[j] = reinterpret_cast<const uint4*>(g.A) + (size_t)(q >> 3) * ((size_t)MTT * KT * 64) + ((size_t)mt * KT + kt0) * 64;
    }
  }
  auto request = [&](uint4* buf, int s) {
    const size_t o = (size_t)min(s, steps - 1) * 64 + lane;      // (past the end: the last k-tile again, into a buffer nobody reads)
#pragma unroll
    for (int j = 0; j < PW; ++j) lds_direct16(src[j] + o, buf + (wave * PW + j) * 64);
  };
  request(tile_s0, 0);
  request(tile_s1, 1);
  request(tile_s2, 2);
  if (g.ssq_in) {                                      // four threads per row add up its square sums
    const int NP = g.K / 16, m = min(mt0 * 16 + (tid >> 2), MTT * 16 - 1);
    const float* p = g.ssq_in + (size_t)m * NP + (tid & 3) * (NP / 4);
    float s = 0.f;
    for (int c = 0; c < NP / 4; c += 4) {
      const float4 v = *reinterpret_cast<const float4*>(p + c);
      s += (v.x + v.y) + (v.z + v.w);
    }
    s += lane_xor<1>(s); s += lane_xor<2>(s);
    if ((tid & 3) == 0) tile_inv[tid >> 2] = 1.0f / sqrtf(s / (float)g.K + g.eps);
  }

  f32x4 acc[WN][WM];
#pragma unroll
  for (int t = 0; t < WN; ++t)
#pragma unroll
    for (int q = 0; q < WM; ++q) acc[t][q] = f32x4{0.f, 0.f, 0.f, 0.f};
  struct Frags { uint4 w[WN], h[WM], l[WM]; };
  auto read = [&](const uint4* buf, Frags& f) {
#pragma unroll
    for (int q = 0; q < WM; ++q) f.l[q] = buf[(NTB + 8 + wm * WM + q) * 64 + lane];
#pragma unroll
    for (int t = 0; t < WN; ++t) f.w[t] = buf[(wn * WN + t) * 64 + lane];
#pragma unroll
    for (int q = 0; q < WM; ++q) f.h[q] = buf[(NTB + wm * WM + q) * 64 + lane];
  };
  constexpr int kWait = 0x0070 | (PW & 15) | ((PW >> 4) << 14);   // vmcnt(PW), lgkmcnt(0)
  // k-tile s out of cur; nxt <- k-tile s + 1 (in rd), k-tile s + 3 requested into wr
  auto step = [&](Frags& cur, Frags& nxt, const uint4* rd, uint4* wr, int s) {
    __builtin_amdgcn_s_waitcnt(kWait);                 // s + 1 has landed (s + 2 may be under way); cur has been read
    __builtin_amdgcn_s_barrier();                      // ... for every wavefront: rd is complete, wr is free
    asm volatile("" ::: "memory");
    request(wr, s + 3);
    read(rd, nxt);
#pragma unroll
    for (int q = 0; q < WM; ++q) {
#pragma unroll
      for (int t = 0; t < WN; ++t)
        acc[t][q] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8, cur.w[t]), __builtin_bit_cast(bf16x8, cur.l[q]), acc[t][q], 0, 0, 0);
    }
#pragma unroll
    for (int q = 0; q < WM; ++q) {
#pragma unroll
      for (int t = 0; t < WN; ++t)
        acc[t][q] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8, cur.w[t]), __builtin_bit_cast(bf16x8, cur.h[q]), acc[t][q], 0, 0, 0);
    }
    // the order asked of the scheduler: the next k-tile's reads and requests spread between the MFMAs
    // (left to itself it sinks every read to just in front of its use)
#pragma unroll
    for (int i = 0; i < WN + 2 * WM; ++i) {
      __builtin_amdgcn_sched_group_barrier(0x100, 1, 0);          // one LDS read
      __builtin_amdgcn_sched_group_barrier(0x008, 2, 0);          // two MFMAs
      if (i < PW) __builtin_amdgcn_sched_group_barrier(0x020, 1, 0);   // one request
    }
    __builtin_amdgcn_sched_group_barrier(0x008, 2 * WN * WM - 2 * (WN + 2 * WM), 0);
  };
  Frags f0, f1;
  __builtin_amdgcn_s_waitcnt(0x0F70 | (2 * PW & 15) | ((2 * PW >> 4) << 14));
  __builtin_amdgcn_s_barrier();
  asm volatile("" ::: "memory");
  read(tile_s0, f0);
  for (int s = 0; s < steps; s += 4) {
    step(f0, f1, tile_s1, tile_s3, s);
    step(f1, f0, tile_s2, tile_s0, s + 1);
    step(f0, f1, tile_s3, tile_s1, s + 2);
    step(f1, f0, tile_s0, tile_s2, s + 3);
  }
  __builtin_amdgcn_s_waitcnt(0);                       // (nothing may land in LDS after the workgroup has gone)
  __syncthreads();

  if (g.KS > 1) {
    // partial tiles, device-coherent; the last slice to arrive adds them all up in slice order
    const size_t slice = (size_t)MTT * (g.N / 16) * 64;
    auto at = [&](int t, int q) { return ((size_t)(mt0 + wm * WM + q) * (g.N / 16) + nt0 + wn * WN + t) * 64 + lane; };
#pragma unroll
    for (int t = 0; t < WN; ++t)
#pragma unroll
      for (int q = 0; q < WM; ++q)
        if (mt0 + wm * WM + q < MTT) {
          uint64_t* p = reinterpret_cast<uint64_t*>(g.part + (ks * slice + at(t, q)) * 4);
          __hip_atomic_store(p, (uint64_t)__float_as_uint(acc[t][q][0]) | ((uint64_t)__float_as_uint(acc[t][q][1]) << 32), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
          __hip_atomic_store(p + 1, (uint64_t)__float_as_uint(acc[t][q][2]) | ((uint64_t)__float_as_uint(acc[t][q][3]) << 32), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        }
    __builtin_amdgcn_s_waitcnt(0);
    __syncthreads();
    if (tid == 0) {
      uint32_t* tk = g.tickets + L;
      const uint32_t old = __hip_atomic_fetch_add(tk, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
      tile_last = old == (uint32_t)(g.KS - 1);
      if (tile_last) __hip_atomic_store(tk, 0u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    }
    __syncthreads();
    if (!tile_last) return;
#pragma unroll
    for (int t = 0; t < WN; ++t)
#pragma unroll
      for (int q = 0; q < WM; ++q) acc[t][q] = f32x4{0.f, 0.f, 0.f, 0.f};
    for (int k = 0; k < g.KS; ++k) {
#pragma unroll
      for (int t = 0; t < WN; ++t)
#pragma unroll
        for (int q = 0; q < WM; ++q)
          if (mt0 + wm * WM + q < MTT) {
            const uint64_t* p = reinterpret_cast<const uint64_t*>(g.part + (k * slice + at(t, q)) * 4);
            const uint64_t a = __hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT), b = __hip_atomic_load(p + 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            acc[t][q] += f32x4{__uint_as_float((uint32_t)a), __uint_as_float((uint32_t)(a >> 32)), __uint_as_float((uint32_t)b), __uint_as_float((uint32_t)(b >> 32))};
          }
    }
  }
#pragma unroll
  for (int q = 0; q < WM; ++q) {
    const int mt = mt0 + wm * WM + q;
    if (mt >= MTT) continue;
    const float inv = g.ssq_in ? tile_inv[(wm * WM + q) * 16 + (lane & 15)] : 1.0f;
#pragma unroll
    for (int t = 0; t < WN; ++t) tile_out(g, nt0 + wn * WN + t, mt, lane, acc[t][q] * inv);
  }
}

}  // namespace

bool tile_supported(int d, int F, int H) { return d % 256 == 0 && F % 256 == 0 && H * 64 == d; }

void launch_gemm_tile(TileGemm g, size_t part_floats, hipStream_t s) {
  TraceScope trace_("gemm_tile", s);
  // 256-wide blocks when they fill the chip, else 128-wide ones; a residual-add projection with fewer
  // than 200 of those in up to 8 slices of at least 8 k-tiles (that fit the partial buffer)
  const int MB = (g.M + kTileM - 1) / kTileM, wide = g.N / 256 * MB, narrow = g.N / 128 * MB;
  g.KS = 1;
  const bool add = g.kind == kTileAdd;
  const size_t slice = (size_t)((g.M + 15) / 16 * 16) * g.N;
  if (add)
    while (narrow * g.KS < 200 && g.KS < 8 && g.K / 32 % (g.KS * 2 * 4) == 0 && g.K / 32 / (g.KS * 2) >= 8 &&
           slice * g.KS * 2 <= part_floats && narrow <= (int)kWsTickets)
      g.KS *= 2;
  if (wide >= 200) hipLaunchKernelGGL(k_gemm_tile<4>, dim3(wide), dim3(512), 0, s, g);
  else hipLaunchKernelGGL(k_gemm_tile<2>, dim3(narrow * g.KS), dim3(512), 0, s, g);
}

}  // namespace xsm
