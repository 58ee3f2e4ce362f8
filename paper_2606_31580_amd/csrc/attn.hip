// Paged grouped-query attention over the KV cache (decode rows and probe chunks).
//
// Work: grid (work item, kv head).  A row group is contiguous rows over one page range of one
// block table (the rows of a request in this forward, or of a request and its forks over
// their shared pages); its query columns are (row, query head of this kv head) pairs in
// 16-column tiles.  A work item is one tile of a group over one page split: each of the
// workgroup's 4 waves walks its own run of pages (split-K) and the waves merge (m, l, O) in
// one LDS round.  The host lists the tiles of one split 8 items apart: workgroups go to the
// 8 XCDs in turn, so these land on one XCD and each page comes from HBM once into that XCD's
// L2 for all of the group's columns.  Per page (16 positions):
//   S^T[t][c] = K[t][:] . Q[c][:]   v_mfma_f32_16x16x32_bf16, A = K page, B = Q^T (bf16 hi+lo)
//   online softmax over t per column (exp2 domain), causal mask t <= pos(c)
//   O^T[d][c] += V^T[d][t] P^T[t][c] v_mfma_f32_16x16x16_bf16, B = P^T taken straight from
//                                    the S^T accumulator layout (bf16 hi+lo)
// The KV page layout makes every operand load a contiguous 1 KB (K) / 512 B (V) per wave
// instruction.  A wave's query tile stays in registers and pages are taken in pairs, so the
// cross-lane max and sum reductions run once per 32 positions.  When a (group, kv head)
// spans several workgroups their fp32 partials are combined: for a one-row group (a decode
// row) by the group's last workgroup to finish, inside this kernel (the partials go out with
// device-scope stores, an arrival counter tells the last one; see the fused items below);
// otherwise by k_attn_merge, launched next.
#include <type_traits>

#include "device_common.hpp"
#include "kernels.hpp"

namespace laser {

__device__ __forceinline__ float safe_exp2(float x) { return x == -INFINITY ? 0.f : exp2f(x); }

// Uniform loads of data written by earlier kernels, through the scalar unit: they don't count
// against the vector-memory counter, which the page copies are waited for by.
typedef int i32x8 __attribute__((ext_vector_type(8), aligned(16)));
template <class T>
__device__ __forceinline__ T ld_scalar(const void* p) {
  return *(const __attribute__((address_space(4))) T*)(uint64_t)p;
}

// RING: runs of any length (see the page copies below); else every run has at most two pages
// (batch 1, 14k positions, 7B: 9.0 us; the ring's detour through LDS costs 0.4-0.8 us there).
// NT: 16-column query tiles per item (2: every page serves both from one load; RING only).
// WALK: runs of any length without the ring, for pools or a workspace that are not 16-byte aligned.
template <class KT, int HD, bool RING, int NT, bool WALK = false>
__global__ __launch_bounds__(64 * kAttnWaves) void k_attn(AttnArgs a) {
  constexpr int NS = HD / 32;  // QK k-steps
  constexpr int ND = HD / 16;  // PV d-tiles
  constexpr int NC = 16 * NT;  // query columns of the item
  static_assert(RING || NT == 1, "two tiles: long runs");
  constexpr int OS = HD + 4;   // merge-slot row stride (floats; padded so that 16 rows fall in different bank groups)
  constexpr int PB = 16 * HD * (int)sizeof(KT);  // bytes of a page's K (or V) block
  constexpr int RBYTES = 4 * PB;                 // a wave's two pages, K and V of each
  constexpr int QS = HD + 8;                     // query row stride (bf16 elements; padded likewise), short runs
  constexpr int QB = RING ? NC * HD * 4 : 4 * NC * QS;  // the tile's queries: fp32, or bf16 hi rows, then lo rows
  constexpr int MB = NT * 3 * 16 * OS * 4;       // merge slots of waves 1-3 (after the pages)
  constexpr int ML = NT * 3 * 16 * 2 * 4 + 16;   // their (m, l), the fused merge's ticket
  constexpr int USED = RING ? QB + kAttnWaves * RBYTES : QB;
  constexpr int SMEM = USED > MB + ML ? USED : MB + ML;
  __shared__ __align__(16) char smem[SMEM];
  float* s_m = (float*)(smem + MB);  // [tile][wave - 1][column]
  float* s_l = s_m + NT * 48;

  static_assert(sizeof(AttnItem) == 32, "one 32-byte load");
  AttnItem wi;
  if constexpr (RING)
    wi = __builtin_bit_cast(AttnItem, ld_scalar<i32x8>(&a.plan->items[blockIdx.x]));
  else
    wi = a.plan->items[blockIdx.x];
  if (wi.nrows == 0) return;  // padding item
  const int nrows = wi.nrows & 0xff;
  const int fuse_n = (wi.nrows >> 8) & 0xff;  // fused group: its split count (else 0)
  const int NQ = nrows * a.G;
  const int kvh = blockIdx.y;
  const int tid = threadIdx.x;
  const int w = __builtin_amdgcn_readfirstlane(tid >> 6), l = tid & 63;
  const int lc = l & 15, lg = l >> 4;
  const int col0 = (wi.info & 0xff) * NC;  // the item's first query column
  const bool two = NT == 2 && NQ - col0 > 16;  // it has a second tile
  const unsigned lds0 = (unsigned)(size_t)(__attribute__((address_space(3))) char*)smem;

  // Wave w walks its run of the item's pages for the tile's 16 columns, then the waves merge
  // through LDS.
  float m_run[NT], l_run[NT];
  f32x4 o[NT][ND];
#pragma unroll
  for (int u = 0; u < NT; ++u) {
    m_run[u] = -INFINITY;
    l_run[u] = 0.f;
#pragma unroll
    for (int dt = 0; dt < ND; ++dt) o[u][dt] = f32x4{0.f, 0.f, 0.f, 0.f};
  }

  const int p0 = wi.p0 + w * wi.pps;
  const int p1 = min(p0 + wi.pps, wi.pend);
  const int* btrow = a.bt + (size_t)wi.seq * a.max_pps;
  const size_t layer_base = (size_t)a.layer * a.num_pages;

  const int c = col0 + lc;           // this lane's query column (of the first tile)
  const int plast = max(p1 - 1, 0);  // clamped: a short run reads its last page again, unused
  int pidA, pidB, cpos[NT];          // the first pages; the columns' positions (-1 past the group's columns)
  // Short runs: the page ids and the queries load together (no page load waits behind another
  // page's data), then the pages, straight into registers.
  constexpr int Q4 = NC * HD / 4 / (64 * kAttnWaves);  // query float4 loads per thread
  static_assert(Q4 * 4 * 64 * kAttnWaves == NC * HD, "query tile");
  float4 qv[Q4];
  // Long runs: the queries go first, as they are, into LDS (they were just written by other XCDs:
  // behind the page traffic they would arrive last): chunk k (16 bytes) of column j at place k ^ j
  // of its row, so that the 16 columns a wave reads at once fall in 16 bank groups.  Columns past
  // the group's read its last one (masked by their position).
  constexpr int CPC = HD / 4, CPI = 64 / CPC;  // chunks per column, columns per copy
  if constexpr (RING) {
#pragma unroll
    for (int i = 0; i < NC / CPI / kAttnWaves; ++i) {
      const int j = (i * kAttnWaves + w) * CPI + l / CPC, k = (l % CPC) ^ (j & 15);
      const int q = min(col0 + j, NQ - 1);
      const float* src = a.q + ((size_t)(wi.row0 + q / a.G) * a.hq + kvh * a.G + q % a.G) * HD + 4 * k;
      copy_to_lds16<false>((const char*)src, lds0 + (i * kAttnWaves + w) * 1024);
    }
    pidA = ld_scalar<int>(btrow + min(p0, plast));
    pidB = ld_scalar<int>(btrow + min(p0 + 1, plast));
#pragma unroll
    for (int u = 0; u < NT; ++u) cpos[u] = row_desc(a.plan, wi.row0 + min(c + 16 * u, NQ - 1) / a.G).pos;
#pragma unroll
    for (int u = 0; u < NT; ++u) {
      asm volatile("" : "+v"(cpos[u]));  // waited for here, the queries too, before the page copies are in flight
      if (c + 16 * u >= NQ) cpos[u] = -1;
    }
  } else {
    // (vector loads: two scalar ones would wait for each other)
    const int pv = wi.p0 + (tid >> 6) * wi.pps, lv = max(min(pv + wi.pps, wi.pend) - 1, 0);
    pidA = btrow[min(pv, lv)];
    pidB = btrow[min(pv + 1, lv)];
#pragma unroll
    for (int i = 0; i < Q4; ++i) {
      const int idx = 4 * (tid + i * 64 * kAttnWaves);
      const int q = min(col0 + idx / HD, NQ - 1), d = idx % HD;
      qv[i] = *(const float4*)(a.q + ((size_t)(wi.row0 + q / a.G) * a.hq + kvh * a.G + q % a.G) * HD + d);
    }
    cpos[0] = row_desc(a.plan, wi.row0 + min(c, NQ - 1) / a.G).pos;
  }

  // Long runs: pages go by pairs through the wave's own LDS ring (K and V of two pages, copied as
  // they lie in memory): once a pair's operands are in registers the next pair's copies start, so a wave has
  // 16 KB (bf16, head dim 128) in flight all the time.
  const unsigned ring0 = lds0 + QB + w * RBYTES;
  const char* ring = smem + QB + w * RBYTES;
  auto copy_page = [&](int pid, int slot) {
    const size_t blk = ((layer_base + pid) * a.hkv + kvh) * (size_t)PB + 16 * l;
#pragma unroll
    for (int u = 0; u < PB / 1024; ++u) {
      copy_to_lds16<true>((const char*)a.kpool + blk + u * 1024, ring0 + slot * 2 * PB + u * 1024);
      copy_to_lds16<true>((const char*)a.vpool + blk + u * 1024, ring0 + slot * 2 * PB + PB + u * 1024);
    }
  };
  constexpr int KW = sizeof(KT) == 4 ? 2 : 1;  // 16-byte K reads per k-step (fp8: one 8-byte read)
  using KRaw = std::conditional_t<sizeof(KT) == 1, u32x2, u32x4>;
  using VRaw = std::conditional_t<sizeof(KT) == 1, uint32_t, std::conditional_t<sizeof(KT) == 2, u32x2, u32x4>>;
  KRaw kraw[2][NS][KW];
  VRaw vraw[2][ND];
  auto read_page = [&](auto bufc) {  // this lane's words of the page in a ring slot
    constexpr int buf = decltype(bufc)::value;
    const char* kb = ring + buf * 2 * PB;
    const char* vb = kb + PB;
#pragma unroll
    for (int s = 0; s < NS; ++s)
#pragma unroll
      for (int q = 0; q < KW; ++q) kraw[buf][s][q] = *(const KRaw*)(kb + (s * 512 + 8 * l) * sizeof(KT) + 16 * q);
#pragma unroll
    for (int dt = 0; dt < ND; ++dt) vraw[buf][dt] = *(const VRaw*)(vb + (dt * 256 + 4 * l) * sizeof(KT));
  };
  auto load_page = [&](int pid, auto bufc) {  // the same words straight from memory
    constexpr int buf = decltype(bufc)::value;
    const size_t blk = ((layer_base + pid) * a.hkv + kvh) * (size_t)PB;
    const char* kb = (const char*)a.kpool + blk;
    const char* vb = (const char*)a.vpool + blk;
#pragma unroll
    for (int s = 0; s < NS; ++s)
#pragma unroll
      for (int q = 0; q < KW; ++q)
        kraw[buf][s][q] = __builtin_nontemporal_load((global_ptr<KRaw>)(kb + (s * 512 + 8 * l) * sizeof(KT) + 16 * q));
#pragma unroll
    for (int dt = 0; dt < ND; ++dt)
      vraw[buf][dt] = __builtin_nontemporal_load((global_ptr<VRaw>)(vb + (dt * 256 + 4 * l) * sizeof(KT)));
  };
  // MFMA operands of one page.  K: lane l holds K[t = l%16][d = 32s + 8(l/16) + j];
  // V^T: V[t = 4(l/16) + j][d = 16dt + l%16].  Slots past the group's last position hold no
  // written value (possibly not even a finite one); P is zero there but 0 * NaN is not, so
  // those V entries are zeroed.
  struct PageOps {
    bf16x8 khi[NS], klo[NS];
    s16x4 vhi[ND], vlo[ND];
  };
  auto unpack = [&](int pg, auto cbc, PageOps& P) {
    constexpr int cb = decltype(cbc)::value;
    if constexpr (sizeof(KT) == 1) {  // E4M3 -> bf16 is exact: no lo part
#pragma unroll
      for (int s = 0; s < NS; ++s) {
        uint32_t w0, w1, w2, w3;
        fp8x4_to_bf16x4(kraw[cb][s][0][0], w0, w1);
        fp8x4_to_bf16x4(kraw[cb][s][0][1], w2, w3);
        P.khi[s] = __builtin_bit_cast(bf16x8, u32x4{w0, w1, w2, w3});
      }
#pragma unroll
      for (int dt = 0; dt < ND; ++dt) {
        uint32_t w0, w1;
        fp8x4_to_bf16x4(vraw[cb][dt], w0, w1);
        P.vhi[dt] = __builtin_bit_cast(s16x4, u32x2{w0, w1});
      }
    } else if constexpr (sizeof(KT) == 2) {
#pragma unroll
      for (int s = 0; s < NS; ++s) P.khi[s] = __builtin_bit_cast(bf16x8, kraw[cb][s][0]);
#pragma unroll
      for (int dt = 0; dt < ND; ++dt) P.vhi[dt] = __builtin_bit_cast(s16x4, vraw[cb][dt]);
    } else {
#pragma unroll
      for (int s = 0; s < NS; ++s) {
        const u32x4 x0 = kraw[cb][s][0], x1 = kraw[cb][s][KW - 1];
        u32x4 ph, pl;
#pragma unroll
        for (int q = 0; q < 4; ++q) {
          uint16_t h0, l0, h1, l1;
          const u32x4& src = q < 2 ? x0 : x1;
          split_bf16(__uint_as_float(src[(q & 1) * 2]), h0, l0);
          split_bf16(__uint_as_float(src[(q & 1) * 2 + 1]), h1, l1);
          ph[q] = (uint32_t)h0 | ((uint32_t)h1 << 16);
          pl[q] = (uint32_t)l0 | ((uint32_t)l1 << 16);
        }
        P.khi[s] = __builtin_bit_cast(bf16x8, ph);
        P.klo[s] = __builtin_bit_cast(bf16x8, pl);
      }
#pragma unroll
      for (int dt = 0; dt < ND; ++dt) {
        const u32x4 x = vraw[cb][dt];
        s16x4 h4, l4;
#pragma unroll
        for (int q = 0; q < 4; ++q) {
          uint16_t hh, ll;
          split_bf16(__uint_as_float(x[q]), hh, ll);
          h4[q] = (short)hh;
          l4[q] = (short)ll;
        }
        P.vhi[dt] = h4;
        P.vlo[dt] = l4;
      }
    }
    if (pg * 16 + 15 > wi.maxpos) {
#pragma unroll
      for (int dt = 0; dt < ND; ++dt)
#pragma unroll
        for (int j = 0; j < 4; ++j)
          if (pg * 16 + 4 * lg + j > wi.maxpos) {
            P.vhi[dt][j] = 0;
            if (sizeof(KT) == 4) P.vlo[dt][j] = 0;
          }
    }
  };
  // S^T tile of one page: lane (c = lc, lg) gets the scores of positions 16pg + 4lg + i.
  // (The hi and lo query parts accumulate in two chains, summed at the end, so that
  // consecutive matrix-core ops do not wait for each other's results.)
  auto scores = [&](const PageOps& P, const bf16x8* qh, const bf16x8* ql) {
    f32x4 shi = f32x4{0.f, 0.f, 0.f, 0.f}, slo = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int s = 0; s < NS; ++s) {
      shi = __builtin_amdgcn_mfma_f32_16x16x32_bf16(P.khi[s], qh[s], shi, 0, 0, 0);
      slo = __builtin_amdgcn_mfma_f32_16x16x32_bf16(P.khi[s], ql[s], slo, 0, 0, 0);
      if (sizeof(KT) == 4) slo = __builtin_amdgcn_mfma_f32_16x16x32_bf16(P.klo[s], qh[s], slo, 0, 0, 0);
    }
    return shi + slo;
  };
  // O^T += V^T P^T for one page; P^T comes straight from the score accumulator layout.
  auto accumulate = [&](const PageOps& P, const float* pv, f32x4* acc) {
    s16x4 phi, plo;
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      uint16_t hh, ll;
      split_bf16(pv[i], hh, ll);
      phi[i] = (short)hh;
      plo[i] = (short)ll;
    }
#pragma unroll
    for (int dt = 0; dt < ND; ++dt) {
      acc[dt] = __builtin_amdgcn_mfma_f32_16x16x16bf16_1k(P.vhi[dt], phi, acc[dt], 0, 0, 0);
      acc[dt] = __builtin_amdgcn_mfma_f32_16x16x16bf16_1k(P.vhi[dt], plo, acc[dt], 0, 0, 0);
      if (sizeof(KT) == 4) acc[dt] = __builtin_amdgcn_mfma_f32_16x16x16bf16_1k(P.vlo[dt], phi, acc[dt], 0, 0, 0);
    }
  };

  bf16x8 qh[NT][NS], ql[NT][NS];
  if constexpr (RING) {
    copy_page(pidA, 0);
    copy_page(pidB, 1);
    wg_barrier();  // every wave's query copies had arrived before its page copies started
#pragma unroll
    for (int u = 0; u < NT; ++u)
#pragma unroll
      for (int s = 0; s < NS; ++s) {
        const char* qr = smem + (16 * u + lc) * HD * 4;
        const f32x4 x0 = *(const f32x4*)(qr + (((8 * s + 2 * lg) ^ lc) & (CPC - 1)) * 16);
        const f32x4 x1 = *(const f32x4*)(qr + (((8 * s + 2 * lg + 1) ^ lc) & (CPC - 1)) * 16);
        const float v[8] = {x0[0], x0[1], x0[2], x0[3], x1[0], x1[1], x1[2], x1[3]};
        u32x4 hi, lo;
        split8(v, hi, lo);
        qh[u][s] = __builtin_bit_cast(bf16x8, hi);
        ql[u][s] = __builtin_bit_cast(bf16x8, lo);
      }
  } else {
    // Both pages load unconditionally: a branch here would make the wait for page 1's id also wait
    // for page 0's data.  The queries are split into bf16 hi/lo in LDS meanwhile.
    load_page(__builtin_amdgcn_readfirstlane(pidA), std::integral_constant<int, 0>{});
    load_page(__builtin_amdgcn_readfirstlane(pidB), std::integral_constant<int, 1>{});
    uint16_t* s_qh = (uint16_t*)smem;
    uint16_t* s_ql = s_qh + NC * QS;
#pragma unroll
    for (int i = 0; i < Q4; ++i) {
      const int idx = 4 * (tid + i * 64 * kAttnWaves);
      const float x[4] = {qv[i].x, qv[i].y, qv[i].z, qv[i].w};
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        uint16_t hi, lo;
        split_bf16(x[e], hi, lo);
        s_qh[(idx / HD) * QS + idx % HD + e] = hi;
        s_ql[(idx / HD) * QS + idx % HD + e] = lo;
      }
    }
    asm volatile("" : "+v"(cpos[0]));  // (issued ahead of the page loads, so it has arrived with the queries)
    if (c >= NQ) cpos[0] = -1;
    __syncthreads();
#pragma unroll
    for (int s = 0; s < NS; ++s) {
      qh[0][s] = *(const bf16x8*)(s_qh + lc * QS + 32 * s + 8 * lg);
      ql[0][s] = *(const bf16x8*)(s_ql + lc * QS + 32 * s + 8 * lg);
    }
  }
  auto pair = [&](int pgA, auto ca, auto cbB) {
    const int pgB = pgA + 1;
    const bool hasB = pgB < p1;  // wave-uniform
    PageOps A, B;
    f32x4 sat[NT], sbt[NT];
    unpack(pgA, ca, A);
    static_for<NT>([&](auto uc) {
      constexpr int u = decltype(uc)::value;
      sbt[u] = f32x4{0.f, 0.f, 0.f, 0.f};
      if (u == 0 || two) sat[u] = scores(A, qh[u], ql[u]);
    });
    if (hasB) {
      unpack(pgB, cbB, B);
      static_for<NT>([&](auto uc) {
        constexpr int u = decltype(uc)::value;
        if (u == 0 || two) sbt[u] = scores(B, qh[u], ql[u]);
      });
    }
    static_for<NT>([&](auto uc) {
      constexpr int u = decltype(uc)::value;
      if (u > 0 && !two) return;  // workgroup-uniform
      const f32x4 sa = sat[u], sb = sbt[u];
      float sv[8];
      float mloc = -INFINITY;
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        const int ta = pgA * 16 + 4 * lg + i, tb = pgB * 16 + 4 * lg + i;
        sv[i] = (ta <= cpos[u]) ? sa[i] * a.scale_log2 : -INFINITY;
        sv[4 + i] = (hasB && tb <= cpos[u]) ? sb[i] * a.scale_log2 : -INFINITY;
        mloc = fmaxf(mloc, fmaxf(sv[i], sv[4 + i]));
      }
      mloc = max_x16(mloc);
      mloc = max_x32(mloc);
      const float m_new = fmaxf(m_run[u], mloc);
      // o and l are still zero while m_run is -inf, so they need no rescale then
      const bool grow = m_run[u] != -INFINITY && m_new != m_run[u];
      const float alpha = grow ? __builtin_amdgcn_exp2f(m_run[u] - m_new) : 1.f;
      float pv[8], ls = 0.f;
#pragma unroll
      for (int i = 0; i < 8; ++i) {
        pv[i] = (sv[i] == -INFINITY) ? 0.f : __builtin_amdgcn_exp2f(sv[i] - m_new);
        ls += pv[i];
      }
      ls = sum_x16(ls);
      ls = sum_x32(ls);
      l_run[u] = l_run[u] * alpha + ls;
      m_run[u] = m_new;
      if (__builtin_amdgcn_read_exec() & __ballot(grow)) {  // any lane whose max moved
#pragma unroll
        for (int dt = 0; dt < ND; ++dt) o[u][dt] *= alpha;
      }
      accumulate(A, pv, o[u]);
      if (hasB) accumulate(B, pv + 4, o[u]);
    });
  };
  // pages in pairs: one max and one sum reduction across the lane groups per 32 positions
  using I0 = std::integral_constant<int, 0>;
  using I1 = std::integral_constant<int, 1>;
  if constexpr (RING) {
    for (int pg = p0; pg < p1; pg += 2) {
      const int nA = ld_scalar<int>(btrow + min(pg + 2, plast)), nB = ld_scalar<int>(btrow + min(pg + 3, plast));
      asm volatile("s_waitcnt vmcnt(0)" ::: "memory");  // the pair has landed
      read_page(I0{});
      read_page(I1{});
      asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
      if (pg + 2 < p1) {
        copy_page(nA, 0);
        copy_page(nB, 1);
      }
      pair(pg, I0{}, I1{});
    }
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");  // (a wave without pages: its copies are done too)
  } else {
    for (int pg = p0; pg < p1; pg += 2) {
      if (WALK && pg > p0) {
        load_page(__builtin_amdgcn_readfirstlane(btrow[pg]), I0{});
        load_page(__builtin_amdgcn_readfirstlane(btrow[min(pg + 1, plast)]), I1{});
      }
      pair(pg, I0{}, I1{});
      if (!WALK) break;  // (two pages at most)
    }
  }
  wg_barrier();  // the queries' and the rings' LDS is free: merge slots
  float* s_of = (float*)smem;

  // ---- one-round merge of the page-parallel waves: 1-3 publish, 0 absorbs in order
  if (w > 0) {
    static_for<NT>([&](auto uc) {
      constexpr int u = decltype(uc)::value;
      if (u > 0 && !two) return;
      const int slot = u * 3 + w - 1;
#pragma unroll
      for (int dt = 0; dt < ND; ++dt) *(f32x4*)(s_of + slot * 16 * OS + lc * OS + 16 * dt + 4 * lg) = o[u][dt];
      if (lg == 0) {
        s_m[slot * 16 + lc] = m_run[u];
        s_l[slot * 16 + lc] = l_run[u];
      }
    });
  }
  __syncthreads();
  if (w != 0 && fuse_n == 0) return;
  const size_t ncols = (size_t)a.max_rows * a.G;
  const __amdgpu_buffer_rsrc_t rpart = dev_rsrc(a.part, a.part_bytes), rml = dev_rsrc(a.ml, a.ml_bytes);
  if (w == 0) {
    static_for<NT>([&](auto uc) {
      constexpr int u = decltype(uc)::value;
      if (u > 0 && !two) return;
      float m = m_run[u], ls = l_run[u];
#pragma unroll
      for (int v = 0; v < 3; ++v) {
        const int slot = u * 3 + v;
        const float m2 = s_m[slot * 16 + lc], l2 = s_l[slot * 16 + lc];
        const float mm = fmaxf(m, m2);
        const float ca = (mm == -INFINITY) ? 0.f : __builtin_amdgcn_exp2f(m - mm);
        const float cb2 = (mm == -INFINITY) ? 0.f : __builtin_amdgcn_exp2f(m2 - mm);
        ls = ls * ca + l2 * cb2;
        m = mm;
#pragma unroll
        for (int dt = 0; dt < ND; ++dt) {
          const f32x4 x = *(const f32x4*)(s_of + slot * 16 * OS + lc * OS + 16 * dt + 4 * lg);
          o[u][dt] = o[u][dt] * ca + x * cb2;
        }
      }
      // ---- the tile's columns: the output (one workgroup) or the workgroup's partial
      const int cu = c + 16 * u;
      if (cu < NQ) {
        const int row = wi.row0 + cu / a.G, head = kvh * a.G + cu % a.G;
        const size_t col = ((size_t)kvh * a.max_wg + ((wi.info >> 8) & 0xffff)) * ncols + (size_t)wi.row0 * a.G + cu;
        if (wi.info & (1 << 24)) {
          const float inv = 1.f / ls;
          if (a.ofrag != nullptr) {
#pragma unroll
            for (int dt = 0; dt < ND; ++dt)
              st_frag4(a.ofrag, row, head * HD + 16 * dt + 4 * lg, a.hq * HD >> 5, o[u][dt] * inv);
          } else {
            float* out = a.o + ((size_t)row * a.hq + head) * HD;
#pragma unroll
            for (int dt = 0; dt < ND; ++dt) *(f32x4*)(out + 16 * dt + 4 * lg) = o[u][dt] * inv;
          }
        } else if (fuse_n) {  // device-scope stores: another XCD's workgroup may merge them
#pragma unroll
          for (int dt = 0; dt < ND; ++dt) st_dev16(rpart, (uint32_t)((col * HD + 16 * dt + 4 * lg) * 4), o[u][dt]);
          if (lg == 0) st_dev8(rml, (uint32_t)(col * 8), m, ls);
        } else {
#pragma unroll
          for (int dt = 0; dt < ND; ++dt) *(f32x4*)(a.part + col * HD + 16 * dt + 4 * lg) = o[u][dt];
          if (lg == 0) {
            a.ml[col * 2 + 0] = m;
            a.ml[col * 2 + 1] = ls;
          }
        }
      }
    });
  }
  if (fuse_n == 0) return;

  // ---- fused group: count this workgroup's arrival once its partial is stored; the last of
  // the group's fuse_n workgroups combines every split (slots 0 .. fuse_n-1, fixed order):
  // o = sum_s O_s 2^(m_s - M) / sum_s l_s 2^(m_s - M), then re-arms the counter.
  unsigned& s_tk = *(unsigned*)(s_l + NT * 48);
  unsigned* cnt = a.cnt + ((size_t)kvh * kMaxGroups + (wi.nrows >> 16)) * kAttnCntStride;
  if (w == 0) {
    wait_mem();
    if (l == 0) s_tk = __hip_atomic_fetch_add(cnt, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
  }
  __syncthreads();
  if (s_tk != (unsigned)(fuse_n - 1)) return;
  constexpr int CH = HD / 4;  // 4-dim chunks of a column
  // (a group size above 8 at head dim 128 is more chunks than threads)
  for (int ch = tid; ch < NQ * CH; ch += 64 * kAttnWaves) {
    const int cc = ch / CH, d4 = ch - cc * CH;
    const size_t colb = (size_t)wi.row0 * a.G + cc;
    float M = -INFINITY, Ls = 0.f;
    f32x4 acc = f32x4{0.f, 0.f, 0.f, 0.f};
    constexpr int B = 8;  // slots loaded together
    for (int s0 = 0; s0 < fuse_n; s0 += B) {
      f32x4 ov[B];
      i32x2 mv[B];
#pragma unroll
      for (int j = 0; j < B; ++j) {  // past the count: slot fuse_n - 1 again (ignored below)
        const size_t colx = ((size_t)kvh * a.max_wg + min(s0 + j, fuse_n - 1)) * ncols + colb;
        ov[j] = ld_dev16(rpart, (uint32_t)((colx * HD + 4 * d4) * 4));
        mv[j] = ld_dev8(rml, (uint32_t)(colx * 8));
      }
#pragma unroll
      for (int j = 0; j < B; ++j) {
        if (s0 + j < fuse_n) {
          const float ms = __int_as_float(mv[j][0]), ls = __int_as_float(mv[j][1]);
          const float mn = fmaxf(M, ms);
          const float ca = (M == -INFINITY) ? 0.f : __builtin_amdgcn_exp2f(M - mn);
          const float cb = (ms == -INFINITY) ? 0.f : __builtin_amdgcn_exp2f(ms - mn);
          Ls = Ls * ca + ls * cb;
          acc = acc * ca + ov[j] * cb;
          M = mn;
        }
      }
    }
    const int row = wi.row0 + cc / a.G, head = kvh * a.G + cc % a.G;
    if (a.ofrag != nullptr)
      st_frag4(a.ofrag, row, head * HD + 4 * d4, a.hq * HD >> 5, acc * (1.f / Ls));
    else
      *(f32x4*)(a.o + ((size_t)row * a.hq + head) * HD + 4 * d4) = acc * (1.f / Ls);
  }
  if (tid == 0) __hip_atomic_store(cnt, 0u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

// Combines the workgroup partials (m, l, O) of every (row, query head) whose group used
// more than one attention workgroup: o = sum_w O_w 2^(m_w - M) / sum_w l_w 2^(m_w - M),
// M = max_w m_w.  grid (rows, query heads), 8 waves.  A slot's HD floats are read by HD/4
// consecutive lanes with 16-byte loads, each lane also reading the slot's (m, l) pair, so
// one wave load covers 64/(HD/4) slots; a lane takes kAttnMaxWG/(kMergeWaves x that) slots, all its
// loads issued together before the plan lookup.  Each wave combines its slots across its
// lanes, then the waves are combined in LDS in fixed order.
constexpr int kMergeWaves = 8;
// FRAG: the output goes out as fragments (a.ofrag).
template <int HD, bool FRAG>
__global__ __launch_bounds__(64 * kMergeWaves) void k_attn_merge(AttnArgs a, int nslots) {
  constexpr int LPS = HD / 4;             // lanes per slot
  constexpr int SPW = 64 / LPS;           // slots per wave load
  constexpr int SPP = SPW * kMergeWaves;  // slots per workgroup pass
  constexpr int PER = kAttnMaxWG / SPP;   // slots per lane
  static_assert(PER * SPP == kAttnMaxWG, "slot passes");
  __shared__ float s_m[kMergeWaves], s_l[kMergeWaves];
  __shared__ __align__(16) float s_o[kMergeWaves][HD];
  const int row = blockIdx.x, head = blockIdx.y;
  const int v = threadIdx.x >> 6, l = threadIdx.x & 63;
  const int d4 = l % LPS, sl = l / LPS;
  const int kvh = head / a.G, gi = head - kvh * a.G;
  const size_t ncols = (size_t)a.max_rows * a.G;
  const size_t col = (size_t)row * a.G + gi;
  const int max_wg = FRAG ? a.max_wg : kAttnMaxWG;  // (only wide prefills have another layout)
  // Slots at or past nslots (the launch's bound on every group's count) read slot
  // nslots - 1 again, a cached line, instead of stale partials; slots past the row's own
  // count are replaced below, never combined.  The loads stay unconditional so none waits
  // for another.
  float mv[PER], lv[PER];
  f32x4 ov[PER];
#pragma unroll
  for (int i = 0; i < PER; ++i) {
    const int slot = min(SPP * i + SPW * v + sl, nslots - 1);
    const size_t sb = ((size_t)kvh * max_wg + slot) * ncols + col;
    const float2 ml = *(const float2*)(a.ml + sb * 2);
    mv[i] = ml.x;
    lv[i] = ml.y;
    ov[i] = *(const f32x4*)(a.part + sb * HD + 4 * d4);
  }
  const int nwg = !FRAG || row < kMaxRows ? a.plan->row_nslots[row] : a.plan->wide_nslots[row / kMaxRows];
  if (nwg <= 1) return;  // written directly by the attention kernel
#pragma unroll
  for (int i = 0; i < PER; ++i)
    if (SPP * i + SPW * v + sl >= nwg) {
      mv[i] = -INFINITY;
      lv[i] = 0.f;
      ov[i] = f32x4{0.f, 0.f, 0.f, 0.f};
    }
  float M = -INFINITY;
#pragma unroll
  for (int i = 0; i < PER; ++i) M = fmaxf(M, mv[i]);
  M = wave_max(M);  // over the wave's slots
  float L = 0.f;
  f32x4 O = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
  for (int i = 0; i < PER; ++i) {
    const float f = (M == -INFINITY) ? 0.f : safe_exp2(mv[i] - M);
    L += lv[i] * f;
    O += ov[i] * f;
  }
  // the wave's slot lanes (LPS apart) summed, so every lane holds the wave's totals
  if constexpr (SPW == 4) {
    L = sum_x16(L);
#pragma unroll
    for (int q = 0; q < 4; ++q) O[q] = sum_x16(O[q]);
  }
  L = sum_x32(L);
#pragma unroll
  for (int q = 0; q < 4; ++q) O[q] = sum_x32(O[q]);
  if (l < LPS) *(f32x4*)&s_o[v][4 * d4] = O;
  if (l == 0) {
    s_m[v] = M;
    s_l[v] = L;
  }
  __syncthreads();
  const int d = threadIdx.x;
  if (d < HD) {
    float Mt = -INFINITY;
#pragma unroll
    for (int u = 0; u < kMergeWaves; ++u) Mt = fmaxf(Mt, s_m[u]);
    float Lt = 0.f, Ot = 0.f;
#pragma unroll
    for (int u = 0; u < kMergeWaves; ++u) {
      const float f = (s_m[u] == -INFINITY) ? 0.f : safe_exp2(s_m[u] - Mt);
      Lt += s_l[u] * f;
      Ot += s_o[u][d] * f;
    }
    const float ov2 = Ot / Lt;
    if constexpr (!FRAG) {
      a.o[((size_t)row * a.hq + head) * HD + d] = ov2;
    } else {  // as fragments: even lanes store two columns' hi parts, odd lanes their lo parts
      uint16_t hi, lo;
      split_bf16(ov2, hi, lo);
      const uint32_t mine = (uint32_t)hi | ((uint32_t)lo << 16);
      const uint32_t other = __float_as_uint(dpp_f<kDppQuad1032>(__uint_as_float(mine)));
      const bool odd = d & 1;
      const uint32_t w2 = odd ? (other >> 16) | (mine & 0xffff0000u) : (mine & 0xffffu) | (other << 16);
      const int col = head * HD + (d & ~1);
      const size_t off = frag_off(row, col & ~7, a.hq * HD >> 5) + 2 * (col & 7);
      *(uint32_t*)(a.ofrag + (odd ? off ^ 64 : off)) = w2;
    }
  }
}

hipError_t launch_attn_merge(const AttnArgs& a, int M, int hd, int nslots, hipStream_t s) {
  if (nslots < 1 || nslots > a.max_wg) return hipErrorInvalidValue;
  const dim3 grid(M, a.hq), block(64 * kMergeWaves);
  if (hd == 128)
    return a.ofrag ? launch_k(k_attn_merge<128, true>, grid, block, s, a, nslots)
                   : launch_k(k_attn_merge<128, false>, grid, block, s, a, nslots);
  if (hd == 64)
    return a.ofrag ? launch_k(k_attn_merge<64, true>, grid, block, s, a, nslots)
                   : launch_k(k_attn_merge<64, false>, grid, block, s, a, nslots);
  return hipErrorInvalidValue;
}

template <class KT, int HD>
static hipError_t launch_hd(const AttnArgs& a, dim3 grid, hipStream_t s) {
  const dim3 block(64 * kAttnWaves);
  if (a.tiles == 2) {
    if constexpr (sizeof(KT) < 4) return launch_k(k_attn<KT, HD, true, 2>, grid, block, s, a);
    return hipErrorInvalidValue;  // (fp32 pools: one tile per item)
  }
  if (a.long_runs && !a.ring) return launch_k(k_attn<KT, HD, false, 1, true>, grid, block, s, a);
  return a.long_runs ? launch_k(k_attn<KT, HD, true, 1>, grid, block, s, a)
                     : launch_k(k_attn<KT, HD, false, 1>, grid, block, s, a);
}

hipError_t launch_attn(int dtype, int hd, const AttnArgs& a, dim3 grid, hipStream_t s) {
  if (dtype == 2) {
    if (hd == 128) return launch_hd<fp8_t, 128>(a, grid, s);
    if (hd == 64) return launch_hd<fp8_t, 64>(a, grid, s);
  } else if (dtype == 1) {
    if (hd == 128) return launch_hd<bf16_t, 128>(a, grid, s);
    if (hd == 64) return launch_hd<bf16_t, 64>(a, grid, s);
  } else {
    if (hd == 128) return launch_hd<float, 128>(a, grid, s);
    if (hd == 64) return launch_hd<float, 64>(a, grid, s);
  }
  return hipErrorInvalidValue;
}

}  // namespace laser
