// Weight addressing shared by the projection kernels.
#pragma once

#include "device_common.hpp"
#include "kernels.hpp"

namespace laser {

// One of three kernel-argument pointers chosen by flags, formed arithmetically: a select
// between argument loads would be folded into a load at a selected argument offset, which
// forces the whole argument block into scratch memory.
__device__ __forceinline__ const void* pick3(bool c0, bool c1, const void* p0, const void* p1, const void* p2) {
  const uint64_t u0 = (uint64_t)p0, u1 = (uint64_t)p1, u2 = (uint64_t)p2;
  const uint64_t f0 = c0, f1 = !c0 && c1, f2 = !c0 && !c1;
  return (const void*)(u0 * f0 + u1 * f1 + u2 * f2);
}

// Rotary pair gp of the QKV rows: pair (i, i + hd/2) of head h, heads numbered q, then k,
// then v.  A workgroup holds RW/2 consecutive pairs (they may span two heads).
struct QkvPair {
  int hh, i;  // head within q, k or v; pair index within the head
  bool isq, isk;
  const void* bias;
  const void* w;
};

__device__ __forceinline__ QkvPair qkv_pair(const GemmArgs& a, int gp) {
  QkvPair q;
  const int half = a.hd >> 1;
  const int h = gp / half;
  q.i = gp - h * half;
  q.isq = h < a.hq;
  q.isk = !q.isq && h < a.hq + a.hkv;
  q.hh = q.isq ? h : (q.isk ? h - a.hq : h - a.hq - a.hkv);
  q.bias = pick3(q.isq, q.isk, a.b0, a.b1, a.b2);
  q.w = pick3(q.isq, q.isk, a.w0, a.w1, a.w2);
  return q;
}

// Row j (< RW) of workgroup g: its weights.  QKV groups hold RW/2 rotary pairs, SwiGLU
// groups RW/2 gate rows and the matching up rows; rows past the matrix read row 0 (their
// results are discarded).
template <class WT, int EPI, int RW>
__device__ __forceinline__ const char* weight_row(const GemmArgs& a, int g, int j) {
  constexpr int P = RW / 2;
  const size_t rowbytes = (size_t)a.K * sizeof(WT);
  if (EPI == EPI_QKV) {
    const int jj = j < P ? j : j - P;
    int gp = P * g + jj;
    if (gp >= (a.hq + 2 * a.hkv) * (a.hd >> 1)) gp = 0;
    const QkvPair q = qkv_pair(a, gp);
    const int dim = j < P ? q.i : (a.hd >> 1) + q.i;
    return (const char*)q.w + (size_t)(q.hh * a.hd + dim) * rowbytes;
  } else if (EPI == EPI_SWIGLU) {
    int r = P * g + (j % P);
    if (r >= a.F) r = 0;
    return (const char*)pick3(j < P, true, a.w0, a.w1, a.w1) + (size_t)r * rowbytes;
  } else {
    int r = RW * g + j;
    if (r >= a.N) r = 0;
    return (const char*)a.w0 + (size_t)r * rowbytes;
  }
}

// Gain of 8 (bf16) or 4 (fp32) consecutive columns as floats.
template <class WT>
__device__ __forceinline__ void unpack16(const u32x4& raw, float* out) {
  if (sizeof(WT) == 2) {
#pragma unroll
    for (int q = 0; q < 4; ++q) {
      out[2 * q] = __uint_as_float(raw[q] << 16);
      out[2 * q + 1] = __uint_as_float(raw[q] & 0xffff0000u);
    }
  } else {
#pragma unroll
    for (int q = 0; q < 4; ++q) out[q] = __uint_as_float(raw[q]);
  }
}

}  // namespace laser
