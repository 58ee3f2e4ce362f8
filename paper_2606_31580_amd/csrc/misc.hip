// Small kernels of the forward: embedding gather (+ block-table updates), the LM head's
// softmax merge, KV-cache import/export between the paged layout and a dense one, and the
// probe's confidence mean.
#include <algorithm>
#include <cstddef>

#include "device_common.hpp"
#include "kernels.hpp"

namespace laser {

__device__ void apply_bt_updates(const Plan* plan, int* bt, int max_pps) {
  for (int i = threadIdx.x; i < plan->n_bt; i += blockDim.x) {
    const BtUpdate u = plan->bt[i];
    bt[(size_t)u.seq * max_pps + u.idx] = u.page;
  }
}

// grid (M, d/64), block 64: h[m][64g..64g+63] = embed[token(m)].
template <class WT>
__global__ __launch_bounds__(64) void k_embed(const Plan* plan, const void* embed, int d, int vocab, float* h, int* bt,
                                              int max_pps) {
  if (blockIdx.x == 0 && blockIdx.y == 0) apply_bt_updates(plan, bt, max_pps);
  const int m = blockIdx.x, g = blockIdx.y, j = threadIdx.x;
  const RowDesc rd = row_desc(plan, m);
  int tok = plan->io.tok_src[rd.tok_sel][rd.tok_off];
  if (tok < 0 || tok >= vocab) tok = 0;  // ids outside the vocabulary never index past the table
  h[(size_t)m * d + 64 * g + j] = ldw<WT>(embed, (size_t)tok * d + 64 * g + j);
}

// One workgroup per LM-head output row: merges the per-group softmax statistics into the
// greedy token (lowest index among equal maxima) and p_max = 1 / sum_j exp(l_j - l_max).
// Every thread loads all its groups at once (a 152k vocabulary at 8 rows per group is one
// round), then the maximum is reduced first (lanes, waves) and the sums are rescaled to it
// once, so no merge step needs an exponential of its own.  Indices are exact as floats
// (below 2^24), which lets the lowest index be a plain minimum reduction.
constexpr int kLmThreads = 1024;
constexpr int kLmPer = 20;  // groups per thread per round
__global__ __launch_bounds__(kLmThreads) void k_lm_reduce(const Plan* plan, const LmPart* part, int n_groups) {
  constexpr int NW = kLmThreads / 64;
  constexpr float kNoIdx = 3.0e38f;
  __shared__ float s_mx[NW], s_sum[NW], s_idx[NW];
  const int m = blockIdx.x, tid = threadIdx.x, lane = tid & 63, w = tid >> 6;
  const LmPart* row = part + (size_t)m * n_groups;
  float mx = -INFINITY, sum = 0.f, idx = kNoIdx;
  for (int g0 = tid; g0 < n_groups; g0 += kLmPer * kLmThreads) {
    LmPart pp[kLmPer];
#pragma unroll
    for (int u = 0; u < kLmPer; ++u) {
      const int g = g0 + u * kLmThreads;
      pp[u] = g < n_groups ? row[g] : LmPart{-INFINITY, 0.f, 0x7fffffff, 0};
    }
    float rm = mx;
#pragma unroll
    for (int u = 0; u < kLmPer; ++u) rm = fmaxf(rm, pp[u].mx);
    float rs = (mx == rm) ? sum : (mx == -INFINITY ? 0.f : sum * expf(mx - rm));
    float ri = (mx == rm) ? idx : kNoIdx;
#pragma unroll
    for (int u = 0; u < kLmPer; ++u) {
      if (pp[u].mx == rm) {
        rs += pp[u].sum;
        if (pp[u].idx != 0x7fffffff) ri = fminf(ri, (float)pp[u].idx);
      } else if (pp[u].mx != -INFINITY) {
        rs += pp[u].sum * expf(pp[u].mx - rm);
      }
    }
    mx = rm;
    sum = rs;
    idx = ri;
  }
  // maximum over the workgroup
  const float wm = wave_max(mx);
  if (lane == 0) s_mx[w] = wm;
  __syncthreads();
  float M = s_mx[0];
#pragma unroll
  for (int v = 1; v < NW; ++v) M = fmaxf(M, s_mx[v]);
  // sums rescaled to it; lowest index among the lanes at it
  const float mine = (mx == -INFINITY || M == -INFINITY) ? 0.f : (mx == M ? sum : sum * expf(mx - M));
  const float ws = wave_sum(mine);
  const float wi = wave_min(mx == M ? idx : kNoIdx);
  if (lane == 0) {
    s_sum[w] = ws;
    s_idx[w] = wi;
  }
  __syncthreads();
  if (tid == 0) {
    float tot = 0.f, best = kNoIdx;
    for (int v = 0; v < NW; ++v) {  // fixed order
      tot += s_sum[v];
      best = fminf(best, s_idx[v]);
    }
    const OutDesc od = plan->outs[m];
    plan->io.tok_dst[od.sel][od.off] = best >= kNoIdx ? 0 : (int)best;
    plan->io.p_dst[od.sel][od.off] = 1.f / tot;
  }
}

// Copies one sequence between the paged pools and dense [n_layers][len][hkv][hd] arrays in pieces of
// 8 elements (16 bytes of bf16; 8 of E4M3, 32 of fp32), for pools and dense arrays that are 16-byte
// aligned.  A thread moves 4 positions x 8 dims of K, of V, or (BOTH) of each: four 8-element loads
// (consecutive threads read consecutive bytes of a position), which in a page block are 32 consecutive
// elements: K chunks of 8 dims lie position by position, V as dims of 4 consecutive positions
// (transposed here in registers).  grid (4-position x 8-dim pieces of a layer / 256, layers, K and V).
// Long transfers are bounded by memory (6,001 positions of 8 layers x 4 heads x 128 in bf16, 98 MB:
// 98 us element by element, 36 us so), short ones by one thread's chain of page id, loads, stores.  So
// the last 1-3 positions take the same path with their absent neighbours left out (element by element
// they were a chain of up to 48 round trips: export of 63 positions, 4 layers x 4 heads x 128 in bf16,
// the call 10.0 us against 6.6; 3,003 positions of 2 layers x 2 heads x 64 in fp32 10.5 against 6.7), and
// the only division is by the head count, in 32 bits.
template <int ES>  // bytes per element
struct KvChunk {
  uint32_t w[2 * ES];  // 8 elements
};
template <int ES, bool TO_POOL, bool BOTH>
__global__ __launch_bounds__(256) void k_kv_copy16(void* kpool, void* vpool, const int* bt, int max_pps, int num_pages,
                                                   int hkv, int hd, int seq, int len, void* k_lin, void* v_lin) {
  using C = KvChunk<ES>;
  const unsigned idx = blockIdx.x * 256 + threadIdx.x;
  const int layer = blockIdx.y;
  const int ld8 = hd == 128 ? 4 : 3;  // log2 of a head's 8-dim pieces
  const int d8 = idx & ((1u << ld8) - 1);
  const unsigned r = idx >> ld8, pos4 = r / (unsigned)hkv;  // pos4: group of 4 positions
  const int kvh = r - pos4 * hkv, pg = pos4 >> 2, t4 = pos4 & 3;
  const int pos = 4 * (int)pos4, n = min(4, len - pos);
  if (n <= 0) return;
  const int page = bt[(size_t)seq * max_pps + pg];
  const size_t blk = (((size_t)layer * num_pages + page) * hkv + kvh) * (size_t)(16 * hd);
  const size_t lin = (((size_t)layer * len + pos) * hkv + kvh) * hd + 8 * d8, row = (size_t)hkv * hd;
  // a chunk is 8 ES bytes, loaded and stored as one or two vectors
  auto ld = [](const char* p) {
    C c;
    if constexpr (ES == 1) {
      const u32x2 v = ld_global<u32x2>(p);
      c.w[0] = v[0];
      c.w[1] = v[1];
    } else {
#pragma unroll
      for (int q = 0; q < ES / 2; ++q) {
        const u32x4 v = ld_global<u32x4>(p + 16 * q);
#pragma unroll
        for (int i = 0; i < 4; ++i) c.w[4 * q + i] = v[i];
      }
    }
    return c;
  };
  auto st = [](char* p, const C& c) {
    if constexpr (ES == 1) {
      *(u32x2*)p = u32x2{c.w[0], c.w[1]};
    } else {
#pragma unroll
      for (int q = 0; q < ES / 2; ++q) *(u32x4*)(p + 16 * q) = u32x4{c.w[4 * q], c.w[4 * q + 1], c.w[4 * q + 2], c.w[4 * q + 3]};
    }
  };
  auto get = [](const C& c, int e) -> uint32_t {  // element e
    if constexpr (ES == 4) return c.w[e];
    if constexpr (ES == 2) return (c.w[e >> 1] >> (16 * (e & 1))) & 0xffffu;
    return (c.w[e >> 2] >> (8 * (e & 3))) & 0xffu;
  };
  auto put = [](C& c, int e, uint32_t v) {
    if constexpr (ES == 4) c.w[e] = v;
    if constexpr (ES == 2) c.w[e >> 1] |= v << (16 * (e & 1));
    if constexpr (ES == 1) c.w[e >> 2] |= v << (8 * (e & 3));
  };
  // Positions past the length read the last one again (in a page: its own slots, which are there).
  auto load = [&](bool is_v, C* c) {
    const char* dense = (const char*)(is_v ? v_lin : k_lin) + lin * ES;
    const char* pool = (const char*)(is_v ? vpool : kpool) + (blk + (is_v ? v_block_off(4 * t4, 8 * d8) : k_block_off(4 * t4, 8 * d8))) * ES;
#pragma unroll
    for (int j = 0; j < 4; ++j) c[j] = ld(TO_POOL ? dense + min(j, n - 1) * row * ES : pool + j * 8 * ES);
  };
  auto store = [&](bool is_v, C* c) {
    char* dense = (char*)(is_v ? v_lin : k_lin) + lin * ES;
    char* pool = (char*)(is_v ? vpool : kpool) + (blk + (is_v ? v_block_off(4 * t4, 8 * d8) : k_block_off(4 * t4, 8 * d8))) * ES;
    if (is_v) {  // dense (position j, dim e) <-> page block: element 4 e + j of the 32
      if (TO_POOL && n < 4) {  // (slots past the length keep what they hold)
        using E = std::conditional_t<ES == 1, uint8_t, std::conditional_t<ES == 2, uint16_t, uint32_t>>;
#pragma unroll
        for (int j = 0; j < 3; ++j)
          if (j < n)
#pragma unroll
            for (int e = 0; e < 8; ++e) ((E*)pool)[4 * e + j] = (E)get(c[j], e);
        return;
      }
      C t[4] = {};
#pragma unroll
      for (int j = 0; j < 4; ++j)
#pragma unroll
        for (int e = 0; e < 8; ++e) {
          const int x = 4 * e + j;
          if constexpr (TO_POOL)
            put(t[x >> 3], x & 7, get(c[j], e));
          else
            put(t[j], e, get(c[x >> 3], x & 7));
        }
#pragma unroll
      for (int j = 0; j < 4; ++j) c[j] = t[j];
    }
#pragma unroll
    for (int j = 0; j < 4; ++j)
      if (j < n) st(TO_POOL ? pool + j * 8 * ES : dense + j * row * ES, c[j]);
  };
  C a[4], b[4];
  if constexpr (BOTH) {
    load(false, a);
    load(true, b);
    store(false, a);
    store(true, b);
  } else {
    load(blockIdx.z, a);
    store(blockIdx.z, a);
  }
}

// The same, one element per load and store, for any alignment.
template <class WT>
__global__ void k_kv_copy(int to_pool, void* kpool, void* vpool, const int* bt, int max_pps, int num_pages,
                          int n_layers, int hkv, int hd, int seq, int len, void* k_lin, void* v_lin) {
  const size_t total = (size_t)n_layers * len * hkv * hd;
  const size_t stride = (size_t)gridDim.x * blockDim.x;
  for (size_t e = (size_t)blockIdx.x * blockDim.x + threadIdx.x; e < total; e += stride) {
    const int d = (int)(e % hd);
    size_t r = e / hd;
    const int kvh = (int)(r % hkv);
    r /= hkv;
    const int pos = (int)(r % len);
    const int layer = (int)(r / len);
    const int page = bt[(size_t)seq * max_pps + (pos >> 4)];
    const size_t blk = (((size_t)layer * num_pages + page) * hkv + kvh) * (size_t)(16 * hd);
    const size_t ko = blk + k_block_off(pos & 15, d), vo = blk + v_block_off(pos & 15, d);
    if (to_pool) {
      ((WT*)kpool)[ko] = ((const WT*)k_lin)[e];
      ((WT*)vpool)[vo] = ((const WT*)v_lin)[e];
    } else {
      ((WT*)k_lin)[e] = ((const WT*)kpool)[ko];
      ((WT*)v_lin)[e] = ((const WT*)vpool)[vo];
    }
  }
}

// conf[r] = (p[r*T] + ... + p[r*T + T-1]) / T, summed in trial order.
__global__ void k_confidence(const float* p, int T, int n, float* conf) {
  const int r = blockIdx.x * blockDim.x + threadIdx.x;
  if (r >= n) return;
  float s = 0.f;
  for (int j = 0; j < T; ++j) s += p[r * T + j];
  conf[r] = s / (float)T;
}

// ATP cue detection: flags[i] = membership of tokens[i] in the bitmap set.
__global__ void k_atp_match(const int* tokens, int n, const unsigned* bitmap, int vocab, int* flags) {
  const int i = blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= n) return;
  const int t = tokens[i];
  flags[i] = (t >= 0 && t < vocab) ? (int)((bitmap[t >> 5] >> (t & 31)) & 1u) : 0;
}

// Copy of one page (every layer and kv head, K and V) from page src to page dst: grid
// (n_layers * hkv), 16-byte chunks of the 16 x hd block.
__global__ __launch_bounds__(256) void k_page_copy(void* kpool, void* vpool, int num_pages, int hkv, size_t blk_bytes,
                                                   int src, int dst) {
  const int layer = blockIdx.x / hkv, h = blockIdx.x - layer * hkv;
  const size_t s_off = (((size_t)layer * num_pages + src) * hkv + h) * blk_bytes;
  const size_t d_off = (((size_t)layer * num_pages + dst) * hkv + h) * blk_bytes;
  for (size_t c = threadIdx.x; c < blk_bytes / 16; c += blockDim.x) {
    *(u32x4*)((char*)kpool + d_off + 16 * c) = *(const u32x4*)((const char*)kpool + s_off + 16 * c);
    *(u32x4*)((char*)vpool + d_off + 16 * c) = *(const u32x4*)((const char*)vpool + s_off + 16 * c);
  }
}

hipError_t launch_page_copy(int kv_es, void* kpool, void* vpool, int num_pages, int n_layers, int hkv, int hd, int src,
                            int dst, hipStream_t s) {
  const size_t blk_bytes = (size_t)16 * hd * kv_es;
  return launch_k(k_page_copy, dim3(n_layers * hkv), dim3(256), s, kpool, vpool, num_pages, hkv, blk_bytes, src, dst);
}

hipError_t launch_embed(int dtype, const Plan* plan, int M, const void* embed, int d, int vocab, float* h, int* bt,
                        int max_pps, hipStream_t s) {
  const dim3 grid(M, d / 64);
  if (dtype == 1)
    return launch_k(k_embed<bf16_t>, grid, dim3(64), s, plan, embed, d, vocab, h, bt, max_pps);
  else
    return launch_k(k_embed<float>, grid, dim3(64), s, plan, embed, d, vocab, h, bt, max_pps);
}

hipError_t launch_lm_reduce(const Plan* plan, const LmPart* part, int n_groups, int n_out, hipStream_t s) {
  return launch_k(k_lm_reduce, dim3(n_out), dim3(kLmThreads), s, plan, part, n_groups);
}

// Copies the used part of a plan from its pinned host staging slot (fine-grained memory, read
// over the bus) to the device plan slot: the fixed head and the first work items in one round
// of loads (16 KB), then the rest of the items and the block-table updates, whose counts the
// head gives.  One workgroup; the next kernel of the forward sees the copy after the boundary.
constexpr int kFetchThreads = 1024;
__device__ __forceinline__ void plan_fetch(const Plan* src, Plan* dst) {
  const char* s = (const char*)src;
  char* d = (char*)dst;
  const int t = threadIdx.x;
  __shared__ int s_cnt[2];
  constexpr size_t R1 = 16 * kFetchThreads;
  static_assert(offsetof(Plan, n_items) < 32 && offsetof(Plan, n_bt) < 16, "counts in the first two chunks");
  static_assert(R1 <= offsetof(Plan, bt), "the first round stays inside the head and items");
  const u32x4 v = ld_global<u32x4>(s + 16 * t);
  *(u32x4*)(d + 16 * t) = v;
  if (t == 0) s_cnt[0] = (int)v[offsetof(Plan, n_bt) / 4];
  if (t == 1) s_cnt[1] = (int)v[(offsetof(Plan, n_items) - 16) / 4];
  __syncthreads();
  const int n_bt = min(max(s_cnt[0], 0), kMaxBt), n_items = min(max(s_cnt[1], 0), kMaxAttnItems);
  const size_t items_end = (offsetof(Plan, items) + sizeof(AttnItem) * (size_t)n_items + 15) & ~(size_t)15;
  for (size_t o = R1 + 16 * t; o < items_end; o += 4 * 16 * kFetchThreads) {
    u32x4 w[4];
#pragma unroll
    for (int u = 0; u < 4; ++u) {
      const size_t ou = o + (size_t)u * 16 * kFetchThreads;
      w[u] = ld_global<u32x4>(s + (ou < items_end ? ou : o));
    }
#pragma unroll
    for (int u = 0; u < 4; ++u) {
      const size_t ou = o + (size_t)u * 16 * kFetchThreads;
      if (ou < items_end) *(u32x4*)(d + ou) = w[u];
    }
  }
  // block-table updates: 12-byte entries from a 16-byte aligned start, whole chunks
  static_assert(offsetof(Plan, bt) % 16 == 0, "block-table updates 16-byte aligned");
  const size_t bt_end = offsetof(Plan, bt) + ((sizeof(BtUpdate) * (size_t)n_bt + 15) & ~(size_t)15);
  for (size_t o = offsetof(Plan, bt) + 16 * t; o < bt_end; o += 16 * kFetchThreads)
    *(u32x4*)(d + o) = ld_global<u32x4>(s + o);
}

__global__ __launch_bounds__(kFetchThreads) void k_plan_fetch(const Plan* src, Plan* dst) { plan_fetch(src, dst); }

// Block-table updates outside a forward (before an import, export, fork or the next forward), from
// the staging slot straight into the table: each thread reads the count and its own update in one
// round over the bus (entries past the count are stale but inside the slot, and unused).  Bounded by
// that round trip; as a plan copy and a second kernel on the copy it was three dependent memory
// rounds and a kernel boundary (an import of 6,001 positions at the 7B shape's heads, 8 layers: the
// call 63.2 us then, 60.2 us so).
__global__ __launch_bounds__(kMaxBt) void k_bt_upload(const Plan* src, int* bt, int max_pps) {
  const int i = threadIdx.x;
  const int n = ld_global<int>(&src->n_bt);
  const int* u = &src->bt[i].seq;
  const int seq = ld_global<int>(u), idx = ld_global<int>(u + 1), page = ld_global<int>(u + 2);
  if (i < n) bt[(size_t)seq * max_pps + idx] = page;
}

// The first kernel of a forward of up to kMaxRows rows: block 0 copies the plan as above and applies
// its block-table updates; block 1 + m gathers row m's embedding, its row descriptor and token
// pointers read from the staging slot like the plan itself (two reads over the bus in flight
// together), so the gather does not wait for the copy and a kernel boundary (copy 4.6 us, boundary,
// gather 4.8 us as two kernels).  With a gain (fragment path), the row's gain times h goes out as
// fragments and its 1 / rms too, as k_resid_norm would write them.
template <class WT>
__global__ __launch_bounds__(kFetchThreads) void k_fetch_embed(const Plan* src, Plan* dst, const void* embed, int d,
                                                                int vocab, float* h, int* bt, int max_pps,
                                                                const uint16_t* gain, float eps, char* xfrag,
                                                                float* row_scale) {
  const int tid = threadIdx.x;
  if (blockIdx.x == 0) {
    const int n_bt = min(max(ld_global<int>(&src->n_bt), 0), kMaxBt);  // in flight with the copy
    plan_fetch(src, dst);
    for (int i = tid; i < n_bt; i += kFetchThreads) {
      const int* u = &src->bt[i].seq;
      bt[(size_t)ld_global<int>(u) * max_pps + ld_global<int>(u + 1)] = ld_global<int>(u + 2);
    }
    return;
  }
  __shared__ int s_tok;
  __shared__ float s_sq[kFetchThreads / 64];
  const int m = blockIdx.x - 1;
  if (tid < 64) {  // wave 0: the descriptor and both token pointers, then the token
    const u32x2 rd = ld_global<u32x2>(&src->rows[m].tok_sel);  // tok_sel, tok_off
    const uint64_t p0 = ld_global<uint64_t>(&src->io.tok_src[0]), p1 = ld_global<uint64_t>(&src->io.tok_src[1]);
    int tok = ld_global<int>((const int*)(rd[0] ? p1 : p0) + (int)rd[1]);
    if (tok < 0 || tok >= vocab) tok = 0;  // ids outside the vocabulary never index past the table
    if (tid == 0) s_tok = tok;
  }
  __syncthreads();
  const size_t row = (size_t)s_tok * d;
  float sq = 0.f;
  for (int c = 8 * tid; c < d; c += 8 * kFetchThreads) {
    float v[8];
#pragma unroll
    for (int e = 0; e < 8; ++e) v[e] = ldw<WT>(embed, row + c + e);
    float4* hp = (float4*)(h + (size_t)m * d + c);
    hp[0] = make_float4(v[0], v[1], v[2], v[3]);
    hp[1] = make_float4(v[4], v[5], v[6], v[7]);
#pragma unroll
    for (int e = 0; e < 8; ++e) sq = fmaf(v[e], v[e], sq);
  }
  if (gain == nullptr) return;
  sq = wave_sum(sq);
  if ((tid & 63) == 0) s_sq[tid >> 6] = sq;
  __syncthreads();
  if (tid == 0) {
    float tot = 0.f;
    for (int w = 0; w < kFetchThreads / 64; ++w) tot += s_sq[w];
    row_scale[m] = rsqrtf(tot / (float)d + eps);
  }
  for (int c = 8 * tid; c < d; c += 8 * kFetchThreads) {
    float y[8];
#pragma unroll
    for (int e = 0; e < 8; ++e) y[e] = ldw<WT>(embed, row + c + e) * bf2f(ld_global<uint16_t>(gain + c + e));
    u32x4 hi, lo;
    split8(y, hi, lo);
    const size_t o = frag_off(m, c, d >> 5);
    *(u32x4*)(xfrag + o) = hi;
    *(u32x4*)(xfrag + (o ^ 64)) = lo;
  }
}

hipError_t launch_fetch_embed(int dtype, const FetchEmbedArgs& f, int M, hipStream_t s) {
  if (M < 1 || M > kMaxRows || f.d % 8 != 0 || (f.gain != nullptr && (dtype != 1 || f.d % 32 != 0))) return hipErrorInvalidValue;
  const dim3 grid(M + 1), block(kFetchThreads);
  const uint16_t* gain = (const uint16_t*)f.gain;
  if (dtype == 1)
    return launch_k(k_fetch_embed<bf16_t>, grid, block, s, f.src, f.dst, f.embed, f.d, f.vocab, f.h, f.bt, f.max_pps, gain,
                    f.eps, f.xfrag, f.row_scale);
  return launch_k(k_fetch_embed<float>, grid, block, s, f.src, f.dst, f.embed, f.d, f.vocab, f.h, f.bt, f.max_pps, gain,
                  f.eps, f.xfrag, f.row_scale);
}

// The kernel's arguments in order, for pointing a captured launch at the next staging slot.
void fetch_embed_params(FetchEmbedArgs& f, void* (&p)[12]) {
  void* a[12] = {&f.src, &f.dst, &f.embed, &f.d, &f.vocab, &f.h, &f.bt, &f.max_pps, &f.gain, &f.eps, &f.xfrag, &f.row_scale};
  for (int i = 0; i < 12; ++i) p[i] = a[i];
}

hipError_t launch_plan_fetch(const Plan* src, Plan* dst, hipStream_t s) {
  return launch_k(k_plan_fetch, dim3(1), dim3(kFetchThreads), s, src, dst);
}

const void* fetch_embed_kernel(int dtype) {
  return dtype == 1 ? (const void*)&k_fetch_embed<bf16_t> : (const void*)&k_fetch_embed<float>;
}

hipError_t launch_bt_upload(const Plan* src, int* bt, int max_pps, hipStream_t s) {
  return launch_k(k_bt_upload, dim3(1), dim3(kMaxBt), s, src, bt, max_pps);
}

hipError_t launch_kv_copy(int kv_es, int to_pool, void* kpool, void* vpool, const int* bt, int max_pps,
                          int num_pages, int n_layers, int hkv, int hd, int seq, int len, void* k_lin,
                          void* v_lin, hipStream_t s) {
  const size_t total = (size_t)n_layers * len * hkv * hd;
  if (total == 0) return hipSuccess;
  if ((((uintptr_t)k_lin | (uintptr_t)v_lin | (uintptr_t)kpool | (uintptr_t)vpool) & 15) == 0 && n_layers <= 65535) {
    // K and V on threads of their own but for imports past the 256 MB memory-side cache, whose writes
    // go out better together (read and written: 197 MB, 8 layers x 4 heads x 6,001 positions, 38.6 us
    // apart, 42.1 together; 574 MB, 5 layers x 8 heads x 14,001, 151 apart, 142 together; export 99 and 105)
    const bool both = to_pool && 4 * total * kv_es > ((size_t)256 << 20);
    const unsigned pieces = (unsigned)((len + 3) / 4) * hkv * (hd / 8);
    const dim3 grid((pieces + 255) / 256, n_layers, both ? 1 : 2);
    auto go = [&](auto k) {
      hipLaunchKernelGGL(k, grid, dim3(256), 0, s, kpool, vpool, bt, max_pps, num_pages, hkv, hd, seq, len, k_lin, v_lin);
      return hipGetLastError();
    };
    auto pick = [&](auto es) {
      constexpr int ES = decltype(es)::value;
      return !to_pool ? go(k_kv_copy16<ES, false, false>) : both ? go(k_kv_copy16<ES, true, true>) : go(k_kv_copy16<ES, true, false>);
    };
    if (kv_es == 1) return pick(std::integral_constant<int, 1>{});
    if (kv_es == 2) return pick(std::integral_constant<int, 2>{});
    return pick(std::integral_constant<int, 4>{});
  }
  size_t blocks = (total + 255) / 256;
  if (blocks > 65536) blocks = 65536;
  if (kv_es == 1)
    hipLaunchKernelGGL(k_kv_copy<uint8_t>, dim3((unsigned)blocks), dim3(256), 0, s, to_pool, kpool, vpool, bt,
                       max_pps, num_pages, n_layers, hkv, hd, seq, len, k_lin, v_lin);
  else if (kv_es == 2)
    hipLaunchKernelGGL(k_kv_copy<uint16_t>, dim3((unsigned)blocks), dim3(256), 0, s, to_pool, kpool, vpool, bt,
                       max_pps, num_pages, n_layers, hkv, hd, seq, len, k_lin, v_lin);
  else
    hipLaunchKernelGGL(k_kv_copy<float>, dim3((unsigned)blocks), dim3(256), 0, s, to_pool, kpool, vpool, bt, max_pps,
                       num_pages, n_layers, hkv, hd, seq, len, k_lin, v_lin);
  return hipGetLastError();
}

// p[0 .. n-1] = v (a kernel rather than a memset, so that a caller may capture it in a graph).
__global__ void k_fill_u32(unsigned* p, int n, unsigned v) {
  for (int i = blockIdx.x * blockDim.x + threadIdx.x; i < n; i += gridDim.x * blockDim.x) p[i] = v;
}

hipError_t launch_fill_u32(unsigned* p, int n, unsigned v, hipStream_t s) {
  if (n < 1) return hipSuccess;
  return launch_k(k_fill_u32, dim3(std::min((n + 255) / 256, 1024)), dim3(256), s, p, n, v);
}

hipError_t launch_confidence(const float* p, int T, int n, float* conf, hipStream_t s) {
  return launch_k(k_confidence, dim3((n + 63) / 64), dim3(64), s, p, T, n, conf);
}

hipError_t launch_atp_match(const int* tokens, int n, const unsigned* bitmap, int vocab, int* flags, hipStream_t s) {
  return launch_k(k_atp_match, dim3((n + 255) / 256), dim3(256), s, tokens, n, bitmap, vocab, flags);
}

}  // namespace laser
