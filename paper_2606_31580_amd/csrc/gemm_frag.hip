// Projections of wide forwards (17 rows and more: probe chunks beside decode rows, prompt
// prefill) on operands that are already matrix-core fragments.
//
// The K-split and row-wave kernels read fp32 activations and split them into bf16 hi/lo inside
// every workgroup, so at several 16-row tiles the splitting, the LDS writes and the waits
// between them are most of their time.  Here the kernel that produces an activation matrix
// stores it once as fragments (frag_off): per 16-row tile and 32-column step 2 KB of hi and lo
// parts, as the 16x16x32 matrix-core operand takes them.  A projection is then
// nothing but a copy of 1 KB blocks (activations and tile-order weights) into an LDS ring,
// done by the load unit itself (global_load_lds), LDS reads without bank conflicts, and
// matrix-core instructions.
//
//   k_gemm_frag    W waves, WM x WN: wave (wm, wn) holds MTW tiles of 16 rows by NGW groups of
//                  16 weight rows.  The ring holds NS steps of 32 columns; a step's blocks are
//                  requested NS - 1 steps before they are multiplied.
// SwiGLU products need all of K in one workgroup; the residual projections and QKV may split it,
// and their K shares are added by the next kernel (k_resid_norm, k_qkv_slices_epi).
//   k_resid_norm   adds a residual projection's K shares to h and writes the next projection's
//                  activations: h * gain as fragments and the rows' 1 / rms, which the projection
//                  applies to its products (the first layer's h * gain, a product of two bf16
//                  values, is then exact in hi + lo).
#include <type_traits>

#include "device_common.hpp"
#include "gemm_common.hpp"
#include "kernels.hpp"

namespace laser {

template <int EPI, int MTW, int NGW, int WM, int WN, int NS>
__global__ __launch_bounds__(64 * WM * WN) void k_gemm_frag(GemmArgs a) {
  constexpr int W = WM * WN, MT = WM * MTW, NG = WN * NGW;
  constexpr int NB = 2 * MT + NG;          // 1 KB blocks of a step
  constexpr int LA = (2 * MT + W - 1) / W, LB = (NG + W - 1) / W;  // copies per wave and step (past the
  constexpr int LPW = LA + LB;                                     // end: the last block again)
  constexpr int SB = NB * 1024;
  constexpr int YB = EPI == EPI_SWIGLU ? NG * MT * 16 * 16 * 4 : 0;
  constexpr int SMEM = NS * SB > YB ? NS * SB : YB;
  __shared__ __align__(16) char smem[SMEM];
  const int tid = threadIdx.x, l = tid & 63;
  const int w = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int wm = w / WN, wn = w - wm * WN;
  // Block index -> (K share, row block, group block): K shares fastest, so that with 8 (4, 2)
  // shares an XCD reads one (two, four) K range(s) of the activations; then the row blocks of
  // one group block on the same XCD in a row, which read its weights from HBM once.
  const int ksplit = a.ksplit, mblocks = a.fr_mblocks;
  const int ks = blockIdx.x % ksplit, c = blockIdx.x / ksplit;
  const int per = 8 / ksplit;
  const int nblk = c / (per * mblocks) * per + c % per, mblk = c / per % mblocks;
  const int g0 = nblk * NG, t0 = mblk * MT;
  if (g0 >= a.n_groups) return;  // padding of the grid
  const int M = a.M, tiles = (M + 15) >> 4;
  const int nst = a.tsteps;
  const int s0 = nst * ks / ksplit, n = nst * (ks + 1) / ksplit - s0;  // this share's steps (n >= 1)

  // this wave's blocks of a step, where they come from: activations (2 KB per step and tile), then
  // weights (non-temporal: read once)
  const char* asrc[LA];
  const char* bsrc[LB];
#pragma unroll
  for (int u = 0; u < LA; ++u) {  // activation tiles past the last one read the last (unused)
    const int b = min(w + u * W, 2 * MT - 1), t = min(t0 + (b >> 1), tiles - 1);
    asrc[u] = a.afrag + ((size_t)t * nst + s0) * 2048 + (b & 1) * 1024 + 16 * l;
  }
  const bool tiled = a.wtile != nullptr;
  const int bstride = tiled ? 1024 : 64;
#pragma unroll
  for (int u = 0; u < LB; ++u) {
    const int g = min(g0 + min(w + u * W, NG - 1), a.n_groups - 1);
    bsrc[u] = tiled ? a.wtile + ((size_t)g * nst + s0) * 1024 + 16 * l
                    // the row-major tensors: 16 bytes of each of 16 rows, 4 times
                    : weight_row<bf16_t, EPI, 16>(a, g, l & 15) + (size_t)s0 * 64 + 16 * (l >> 4);
  }
  const unsigned ring = (unsigned)(size_t)(__attribute__((address_space(3))) char*)smem;
  unsigned slot = 0;  // ring slot of the next step to request
  auto request = [&]() {
#pragma unroll
    for (int u = 0; u < LB; ++u) {
      copy_to_lds16<true>(bsrc[u], ring + slot * SB + (2 * MT + min(w + u * W, NG - 1)) * 1024);
      bsrc[u] += bstride;
    }
#pragma unroll
    for (int u = 0; u < LA; ++u) {
      copy_to_lds16<false>(asrc[u], ring + slot * SB + min(w + u * W, 2 * MT - 1) * 1024);
      asrc[u] += 2048;
    }
    slot = slot + 1 == NS ? 0 : slot + 1;
  };
  f32x4 acc[NGW][MTW];
#pragma unroll
  for (int r = 0; r < NGW; ++r)
#pragma unroll
    for (int mt = 0; mt < MTW; ++mt) acc[r][mt] = f32x4{0.f, 0.f, 0.f, 0.f};
  unsigned cur = 0;  // ring slot of the step being multiplied
  const int ahi = (l & 15) * 128 + ((l >> 4) ^ ((l & 15) >> 1)) * 16;  // this lane's hi chunk (frag_off)
  auto multiply = [&]() {
    const char* sa = smem + cur * SB + wm * MTW * 2048;
    const char* sb = smem + cur * SB + 2 * MT * 1024 + wn * NGW * 1024 + 16 * l;
    bf16x8 b[NGW];
#pragma unroll
    for (int r = 0; r < NGW; ++r) b[r] = *(const bf16x8*)(sb + r * 1024);
    // every accumulator sums hi before lo; consecutive instructions feed different ones
#pragma unroll
    for (int mt = 0; mt < MTW; ++mt) {
      const bf16x8 hi = *(const bf16x8*)(sa + mt * 2048 + ahi);
      const bf16x8 lo = *(const bf16x8*)(sa + mt * 2048 + (ahi ^ 64));
#pragma unroll
      for (int r = 0; r < NGW; ++r) acc[r][mt] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(hi, b[r], acc[r][mt], 0, 0, 0);
#pragma unroll
      for (int r = 0; r < NGW; ++r) acc[r][mt] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(lo, b[r], acc[r][mt], 0, 0, 0);
    }
    cur = cur + 1 == NS ? 0 : cur + 1;
  };
  for (int i = 0; i < NS - 1 && i < n; ++i) request();
  // steady state: step i has landed (the NS - 2 later ones may be in flight) and every wave is
  // done with step i - 1, whose slot takes step i + NS - 1
  for (int i = 0; i + NS - 1 < n; ++i) {
    wait_copies<(NS - 2) * LPW>();
    wg_barrier();
    request();
    multiply();
  }
  static_for<NS - 1>([&](auto j) {  // the last steps: r later ones in flight
    constexpr int r = NS - 2 - decltype(j)::value;
    if (n - 1 - r >= 0) {
      wait_copies<r * LPW>();
      wg_barrier();
      multiply();
    }
  });

  // lane (n16, q = l / 16): acc[r][mt][i] = Y[row 16 mt + 4 q + i][weight row 16 r + n16] of the wave's part
  const int n16 = l & 15, q4 = 4 * (l >> 4);
  if (EPI != EPI_SWIGLU) {  // this K share's sums; k_resid_norm (k_qkv_slices_epi) adds the shares
#pragma unroll
    for (int r = 0; r < NGW; ++r) {
      const int g = g0 + wn * NGW + r;
      if (g < a.n_groups)
#pragma unroll
        for (int mt = 0; mt < MTW; ++mt)
#pragma unroll
          for (int i = 0; i < 4; ++i) {
            const int m = 16 * (t0 + wm * MTW + mt) + q4 + i;
            if (m < M) a.kpart[((size_t)ks * M + m) * a.N + 16 * g + n16] = acc[r][mt][i];
          }
    }
    return;
  }
  __syncthreads();  // the ring is free: Y[group][row][16], scaled by the rows' 1 / rms
  float* Y = (float*)smem;
  constexpr int YN = MT * 256;
  float sc[MTW][4];
#pragma unroll
  for (int mt = 0; mt < MTW; ++mt)
#pragma unroll
    for (int i = 0; i < 4; ++i) sc[mt][i] = a.row_scale[min(16 * (t0 + wm * MTW + mt) + q4 + i, M - 1)];
#pragma unroll
  for (int r = 0; r < NGW; ++r)
#pragma unroll
    for (int mt = 0; mt < MTW; ++mt)
#pragma unroll
      for (int i = 0; i < 4; ++i)
        Y[(wn * NGW + r) * YN + (16 * (wm * MTW + mt) + q4 + i) * 16 + n16] = acc[r][mt][i] * sc[mt][i];
  __syncthreads();
  const int rows = min(16 * MT, M - 16 * t0), ng = min(NG, a.n_groups - g0);
  // 8 consecutive outputs of a row: one 16-byte chunk of hi, one of lo
  const int fst = a.F >> 5;
  for (int idx = tid; idx < ng * rows; idx += 64 * W) {
    const int r = idx / rows, m = idx - r * rows;
    const float* y = Y + r * YN + m * 16;
    float v[8];
#pragma unroll
    for (int e = 0; e < 8; ++e) v[e] = y[e] / (1.f + expf(-y[e])) * y[8 + e];
    const size_t d = frag_off(16 * t0 + m, 8 * (g0 + r), fst);
    u32x4 hi, lo;
    split8(v, hi, lo);
    *(u32x4*)(a.frag_out + d) = hi;
    *(u32x4*)(a.frag_out + (d ^ 64)) = lo;
  }
}

// One workgroup per row: h += the K shares in order, then (gain given) the row's RMSNorm as
// fragments of the next projection.  One pass: the row stays in registers between the sum of
// squares and the scaling.
constexpr int kRnThreads = 512, kRnChunks = 4;  // 8 columns per chunk: rows of up to 16,384
template <int KS>
__global__ __launch_bounds__(kRnThreads) void k_resid_norm(float* h, const float* kpart, int M, int N,
                                                            const uint16_t* gain, float eps, char* xfrag,
                                                            float* row_scale) {
  __shared__ float s_sq[kRnThreads / 64];
  const int m = blockIdx.x, tid = threadIdx.x;
  const int nch = N >> 3;
  float4 v[kRnChunks][2];
  float sq = 0.f;
#pragma unroll
  for (int u = 0; u < kRnChunks; ++u) {
    const int ch = tid + u * kRnThreads;
    if (ch >= nch) break;
    float4* hp = (float4*)(h + (size_t)m * N + 8 * ch);
    float4 x0 = hp[0], x1 = hp[1];
    if (KS > 0) {
      float4 s0 = {0.f, 0.f, 0.f, 0.f}, s1 = s0;
#pragma unroll
      for (int k = 0; k < KS; ++k) {
        const float4* p = (const float4*)(kpart + ((size_t)k * M + m) * N + 8 * ch);
        const float4 p0 = p[0], p1 = p[1];
        s0.x += p0.x;
        s0.y += p0.y;
        s0.z += p0.z;
        s0.w += p0.w;
        s1.x += p1.x;
        s1.y += p1.y;
        s1.z += p1.z;
        s1.w += p1.w;
      }
      x0.x += s0.x;
      x0.y += s0.y;
      x0.z += s0.z;
      x0.w += s0.w;
      x1.x += s1.x;
      x1.y += s1.y;
      x1.z += s1.z;
      x1.w += s1.w;
      hp[0] = x0;
      hp[1] = x1;
    }
    v[u][0] = x0;
    v[u][1] = x1;
    sq = fmaf(x0.x, x0.x, fmaf(x0.y, x0.y, fmaf(x0.z, x0.z, fmaf(x0.w, x0.w, sq))));
    sq = fmaf(x1.x, x1.x, fmaf(x1.y, x1.y, fmaf(x1.z, x1.z, fmaf(x1.w, x1.w, sq))));
  }
  if (gain == nullptr) return;
  sq = wave_sum(sq);
  if ((tid & 63) == 0) s_sq[tid >> 6] = sq;
  __syncthreads();
  float tot = 0.f;
#pragma unroll
  for (int w = 0; w < kRnThreads / 64; ++w) tot += s_sq[w];
  if (tid == 0) row_scale[m] = rsqrtf(tot / (float)N + eps);
#pragma unroll
  for (int u = 0; u < kRnChunks; ++u) {
    const int ch = tid + u * kRnThreads;
    if (ch >= nch) break;
    float gf[8];
    unpack16<bf16_t>(*(const u32x4*)(gain + 8 * ch), gf);
    const float x[8] = {v[u][0].x, v[u][0].y, v[u][0].z, v[u][0].w, v[u][1].x, v[u][1].y, v[u][1].z, v[u][1].w};
    float y[8];
#pragma unroll
    for (int e = 0; e < 8; ++e) y[e] = x[e] * gf[e];
    u32x4 hi, lo;
    split8(y, hi, lo);
    const size_t d = frag_off(m, 8 * ch, N >> 5);
    *(u32x4*)(xfrag + d) = hi;
    *(u32x4*)(xfrag + (d ^ 64)) = lo;
  }
}

hipError_t launch_resid_norm(float* h, const float* kpart, int ksplit, int M, int N, const void* gain, float eps,
                             char* xfrag, float* row_scale, hipStream_t s) {
  if (N % 32 != 0 || N > 8 * kRnThreads * kRnChunks || M < 1) return hipErrorInvalidValue;
  auto go = [&](auto k) { return launch_k(k, dim3(M), dim3(kRnThreads), s, h, kpart, M, N, (const uint16_t*)gain, eps, xfrag, row_scale); };
  switch (ksplit) {
    case 0: return go(k_resid_norm<0>);
    case 1: return go(k_resid_norm<1>);
    case 2: return go(k_resid_norm<2>);
    case 4: return go(k_resid_norm<4>);
    case 8: return go(k_resid_norm<8>);
    default: return hipErrorInvalidValue;
  }
}

template <int MTW, int NGW, int WM, int WN, int NS>
static hipError_t launch_cfg(int epi, GemmArgs a, hipStream_t s) {
  const int tiles = (a.M + 15) / 16;
  a.fr_mblocks = (tiles + WM * MTW - 1) / (WM * MTW);
  const int per = 8 / a.ksplit;
  const int nblk = ((a.n_groups + WN * NGW - 1) / (WN * NGW) + per - 1) / per * per;
  const dim3 grid(nblk * a.fr_mblocks * a.ksplit), block(64 * WM * WN);
  switch (epi) {
    case EPI_QKV: return launch_k(k_gemm_frag<EPI_QKV, MTW, NGW, WM, WN, NS>, grid, block, s, a);
    case EPI_RESID: return launch_k(k_gemm_frag<EPI_RESID, MTW, NGW, WM, WN, NS>, grid, block, s, a);
    case EPI_SWIGLU: return launch_k(k_gemm_frag<EPI_SWIGLU, MTW, NGW, WM, WN, NS>, grid, block, s, a);
    default: return hipErrorInvalidValue;
  }
}

hipError_t launch_gemm_frag(int epi, int cfg, const GemmArgs& a, hipStream_t s) {
  if (a.afrag == nullptr || (epi != EPI_RESID && a.row_scale == nullptr) || a.K % 32 != 0 || a.tsteps != a.K / 32 ||
      a.M < 1 || a.M > kFragRows || (a.ksplit != 1 && a.ksplit != 2 && a.ksplit != 4 && a.ksplit != 8) ||
      a.tsteps < a.ksplit ||
      (epi == EPI_SWIGLU ? a.ksplit > 1 || a.frag_out == nullptr || a.F % 32 != 0 || a.n_groups * 8 != a.F
                         : a.kpart == nullptr || a.N != 16 * a.n_groups || a.ksplit * a.M > kFragPartRows))
    return hipErrorInvalidValue;
  switch (cfg) {
#define LASER_FRAG(MTW, NGW, WM, WN, NS) \
  case frag_cfg(MTW, NGW, WM, WN): return launch_cfg<MTW, NGW, WM, WN, NS>(epi, a, s);
    LASER_FRAG_SHAPES
#undef LASER_FRAG
    default: return hipErrorInvalidValue;
  }
}

}  // namespace laser
