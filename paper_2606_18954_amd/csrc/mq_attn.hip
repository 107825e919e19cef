// Multi-query (extend, prefill) segment attention for bf16 inputs: one work item = (segment chain,
// page chunk, row block of up to 128 query rows, kv-head), as in seg_attn.hip, with the work list,
// the descriptors, the partial rows and the merge shared with it.
//
// What bounds it.  With many queries per branch a page is read for a hundred rows and more, so the
// matrix cores, the softmax's vector instructions and LDS matter, and no one of them is full.  Counters
// over the kernel's time, 16-token extend | prefill (workloads below): matrix cores busy 39% | 43%,
// vector instructions 40% | 41% of the SIMDs' cycles, LDS active 22% | 25% with 0.1% | 3.5% of its
// cycles lost to conflicts.  Matrix and vector work together would fill 79% to 84% if they never
// overlapped, and with two waves per SIMD, each a chain of scores, softmax and products, they overlap
// little.  Per pair of pages and 32 rows (head_dim 128) the matrix cores need 16 x 32 cycles and the
// vector unit about 560 (16 exponentials, 91 others); two waves per SIMD that overlap perfectly would
// take 1,120 cycles for two such steps.  Measured: 1,950 to 1,990 (the same loop without copies 1,660,
// and alone on data in LDS 1,500), plus 2,100 before and 8,500 after the loop of a unit.  The kernel this
// one replaces (seg_attn.hip, 16-row tiles, three workgroups per CU) issued 6 vector instructions per
// matrix instruction of half the size; here it is 7 per instruction of twice the size.
//   16-token extend of the merged-DAG rollout, 1024 branches, 28/4 heads x 128, average of 50 steps,
//   other kernel | this one on one card: 1.38 | 1.30 ms (0.75 PFLOP/s); on a card with lower clocks 1.43.
//   Prefill of 32 prompts of 1024 to 2048 tokens: 1.58 | 0.61 ms, average of 40 passes, and no merge
//   (0.87 PFLOP/s; a plain 8192^3 bf16 matrix product reaches 1.23 on that card).
//
// Layout.  Four waves of one 32-row tile each; two pages (32 tokens) per step:
//   S^T = K Q^T    v_mfma_f32_32x32x16_bf16: a lane owns one row and half of its 32 scores
//   O^T += V^T P^T the same instruction, its B operand taken straight from S^T's registers: the
//                  contraction order is free, so slot (g, e) of step s stands for the token whose
//                  score the lane already holds, and V^T is read in that order
// K and V have rings of four slots of two pages each in LDS, filled by direct-to-LDS copies.  The
// 16-byte chunks of a token row are XOR-permuted with the token's low bits in the high chunk bits,
// so that both the K reads and the transposing V reads are free of bank conflicts (30% of the LDS
// cycles with the other kernel's permutation).  The scores of the next pair are computed while
// this pair's exponentials are (the order of issue is fixed by scheduling groups), with their K
// operands read from LDS an iteration ahead; so a K slot is free one iteration early and its ring
// runs two pairs ahead of V's.  A unit's page words sit in one register, a lane per pair, and one
// ballot says which iterations need the mask.  Pages that no row of the unit sees (causal units)
// are not visited: half of a prefill.  The next unit's first copies and queries are issued before
// this unit's rows are stored, and the rows leave through LDS, as whole lines.
#include "attn_dev.hpp"
#include "ga_internal.hpp"

#include <hip/hip_ext.h>

#include <type_traits>

namespace ga {
namespace {

typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef short s16x4 __attribute__((ext_vector_type(4)));
typedef float f32x16 __attribute__((ext_vector_type(16)));
typedef __attribute__((address_space(3))) s16x4 lds_s16x4;
typedef __attribute__((address_space(3))) const bf16x8 lds_bf16x8;
typedef __attribute__((address_space(3))) unsigned char lds_uchar;

template <int D>
struct MCfg {
  static constexpr int ROW = D * 2;                 // bytes of a token row of K or V
  static constexpr int CPR = ROW / 16;              // 16-byte chunks per token row
  static constexpr int KVB = 16 * ROW;              // bytes of a page's K (or V) block
  static constexpr int HALF = 2 * KVB;              // K (or V) of a pair of pages: one ring slot
  static constexpr int SLOTS = 4;                   // slots of the K ring and of the V ring
  static constexpr int CPW = HALF / 1024 / 4;       // 1 KiB copies per wave and slot
  static constexpr int KS = D / 16;                 // contraction steps of S^T = K Q^T
  static constexpr int NC = D / 32;                 // 32-column tiles of O^T
};

// XOR applied to the 16-byte chunk index of token tok's row.
template <int D>
__device__ __forceinline__ int fswz(int tok) {
  return D == 128 ? ((tok & 3) << 2) | ((tok >> 2) & 3) : (((tok >> 1) & 1) << 2) | ((tok >> 2) & 3);
}

template <int D>
__global__ __launch_bounds__(kAttnThreads, mq_wgs_per_cu(D)) void k_mq_attn(AttnArgs a) {
  using C = MCfg<D>;
  __shared__ __align__(1024) unsigned char smem[2 * C::SLOTS * C::HALF];   // K ring, V ring
  __shared__ __align__(1024) int s_desc[2][kDescMaxBytes / 4];
  __shared__ int s_next[2];

  const int tid = threadIdx.x;
  const int lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int r32 = lane & 31, g = lane >> 5, r16 = lane & 15;
  const int n_work = (int)(a.counters[0] * a.Hkv);
  const float NEG_INF = -__builtin_huge_valf();
  const unsigned char* pool = static_cast<const unsigned char*>(a.pool);
  const __bf16* qbase = static_cast<const __bf16*>(a.q);
  const unsigned lds_ring = (unsigned)(uintptr_t)(lds_uchar*)smem;
  const unsigned lds_desc =
      (unsigned)(uintptr_t)(__attribute__((address_space(3))) int*)&s_desc[0][0];
  const int dins = (a.desc_words * 4 + 1023) / 1024;
  const int br_word = kDescHead + a.chunk_pages;

  auto fetch_desc = [&](int v, int nb) {
    const bool ok = v < n_work;
    if (lane == 0) s_next[nb] = ok ? v : -1;
    if (ok) {
      const int* src = a.desc + (int64_t)(v / a.Hkv) * a.desc_words;
      const unsigned dst = lds_desc + nb * kDescMaxBytes;
      for (int i = 0; i < dins; ++i)
        dma16(1024 * i + 16 * lane, src, __builtin_amdgcn_readfirstlane(dst + 1024 * i));
    }
  };

  // The wave's copies of a slot: page wave / 2 of the pair, tokens 8 (wave mod 2) + 4 i .. + 3 (D =
  // 128, copies i = 0, 1) or all eight tokens (D = 64, one copy); this lane's token and chunk.
  const int c_pg = wave >> 1;
  int c_tok[C::CPW], c_chunk[C::CPW];
#pragma unroll
  for (int i = 0; i < C::CPW; ++i) {
    const int o = ((wave & 1) * C::CPW + i) * 1024 + lane * 16;
    c_tok[i] = o / C::ROW;
    c_chunk[i] = (((o % C::ROW) >> 4) ^ fswz<D>(c_tok[i])) << 4;
  }
  // LDS byte offsets of the operand reads inside a ring slot.  K: lane row r32 = token of the
  // pair (page r32 / 16), chunks 2 s + g.  V: the transposing reads' pieces of column tile n,
  // tokens 8 j + 4 g .. + 3 of a page.
  int koff[C::KS], voff[C::NC][2];
#pragma unroll
  for (int s = 0; s < C::KS; ++s)
    koff[s] = (r32 >> 4) * C::KVB + (r32 & 15) * C::ROW +
              (((2 * s + g) ^ fswz<D>(r32 & 15)) << 4);
#pragma unroll
  for (int n = 0; n < C::NC; ++n)
#pragma unroll
    for (int j = 0; j < 2; ++j) {
      const int tok = 8 * j + 4 * g + (r16 >> 2);
      const int ch = 4 * n + 2 * ((lane >> 4) & 1) + ((r16 & 3) >> 1);
      voff[n][j] = C::SLOTS * C::HALF + tok * C::ROW + ((ch ^ fswz<D>(tok)) << 4) + (r16 & 1) * 8;
    }

  const int ns = a.streams;
  const int per = a.Hkv / ns;
  const int n_str = (int)(a.counters[0] * per);
  int* heads = reinterpret_cast<int*>(a.counters + 4);
  auto gs = [&](int st) { return ((int)gridDim.x - st + ns - 1) / ns; };
  auto unit_of = [&](int j, int st) {
    return j < n_str ? (j / per) * a.Hkv + (j % per) * ns + st : n_work;
  };
  int cs = (int)blockIdx.x % ns;
  const int rank = (int)blockIdx.x / ns;
  if (wave == 0) {
    fetch_desc(unit_of(rank, cs), 0);
    wait_vmcnt(0);
  }
  __syncthreads();

  const int64_t blk_stride = (int64_t)a.Hkv * 2 * C::KVB;
  const unsigned dst_w = __builtin_amdgcn_readfirstlane(lds_ring + wave * C::CPW * 1024);
  const float rgroup = 1.f / (float)a.group;
  auto page_base = [&](const unsigned char* pool_h, int word) {
    return pool_h + (int64_t)(word & kPageIdMask) * blk_stride;
  };
  // The wave's part of a K slot, and of a V slot: a K row past the page's valid tokens may hold
  // anything (its scores are replaced by the mask), a V row must be finite (its probability is 0),
  // so those re-read the last valid token.
  auto copy_k = [&](const unsigned char* base, unsigned dst) {
#pragma unroll
    for (int i = 0; i < C::CPW; ++i)
      dma16_cached(c_tok[i] * C::ROW + c_chunk[i], base,
                   __builtin_amdgcn_readfirstlane(dst + i * 1024));
  };
  auto copy_v = [&](const unsigned char* base, int vm1, unsigned dst) {
#pragma unroll
    for (int i = 0; i < C::CPW; ++i)
      dma16_cached(min(c_tok[i], vm1) * C::ROW + c_chunk[i], base,
                   __builtin_amdgcn_readfirstlane(dst + i * 1024));
  };

  // A unit, read from its descriptor in LDS.
  struct Unit {
    int w, npe, n2, cw, row0, R, prow_base, kvh, j0;
    const unsigned char* pool_h;
  };
  // The first slots' copies of a unit: K of pairs 0 .. 2 and V of 0, 1 (start_unit), then K of pair
  // 3 and V of pair 2 (start_rest), into whose slots the wave's parts are free for the row stores'
  // staging until then.
  bf16x8 qop[C::KS];
  const unsigned char* vq[4];                     // V bases and valid tokens of the pairs whose K
  int vqm[4];                                      // was copied, by ring slot
  int pk = 0;                                      // lane t: word of the wave's page of pair t
  auto start_unit = [&](int b) {
    Unit u;
    u.w = __builtin_amdgcn_readfirstlane(s_next[b]);
    if (u.w < 0) return u;
    const int* dsc = &s_desc[b][0];
    u.kvh = u.w % a.Hkv;
    const int np = __builtin_amdgcn_readfirstlane(dsc[0]);
    u.cw = __builtin_amdgcn_readfirstlane(dsc[1]);
    const int cnt = __builtin_amdgcn_readfirstlane(dsc[3]);
    u.row0 = __builtin_amdgcn_readfirstlane(dsc[4]) * kRowsPerBlock;
    u.prow_base = __builtin_amdgcn_readfirstlane(dsc[7]);
    u.R = min(kRowsPerBlock, cnt * a.group - u.row0);
    u.j0 = u.row0 / a.group;
    // Pages that some row of the unit sees.
    u.npe = np;
    if (u.cw != kNoCausal)
      u.npe = max(0, min(np, (u.cw + (u.row0 + u.R - 1) / a.group + kPageTokens) / kPageTokens));
    u.n2 = (u.npe + 1) >> 1;
    u.pool_h = (const unsigned char*)uniform64(
        (int64_t)(uintptr_t)(pool + (int64_t)u.kvh * 2 * C::KVB));
    // (the second page of a last pair may not exist: its first page once more, masked)
    pk = dsc[kDescHead + max(0, min(2 * lane + c_pg, u.npe - 1))];
#pragma unroll
    for (int t = 0; t < 5; ++t) {
      const int word = __builtin_amdgcn_readlane(pk, t);
      const unsigned char* base = page_base(u.pool_h, word);
      const int vm1 = (int)((unsigned)word >> kPageValidShift);
      if (t < 3 && t < u.n2) {
        copy_k(base, dst_w + t * C::HALF);
        if (t < 2) copy_v(base + C::KVB, vm1, dst_w + (C::SLOTS + t) * C::HALF);
      }
      if (t > 0) {
        vq[t & 3] = base + C::KVB;
        vqm[t & 3] = vm1;
      }
    }
    return u;
  };
  auto start_rest = [&](const Unit& u) {
    if (3 < u.n2) copy_k(vq[3] - C::KVB, dst_w + 3 * C::HALF);
    if (2 < u.n2) copy_v(vq[2], vqm[2], dst_w + (C::SLOTS + 2) * C::HALF);
  };
  // Row of the wave's lane: group rank j (relative to the block's first) and q-head.
  auto row_of = [&](const Unit& u, int r, int& jl, int& h) {
    const int x = r + u.row0 - u.j0 * a.group;      // < 128 + group: the float quotient is exact
    jl = (int)(((float)x + 0.5f) * rgroup);
    h = u.kvh * a.group + x - jl * a.group;
  };
  auto load_q = [&](const Unit& u, int b) {
    const int r = 32 * wave + r32;
    const bool live = r < u.R;
    const __bf16* qp = qbase;
    if (live) {
      int jl, h;
      row_of(u, r, jl, h);
      qp = qbase + ((int64_t)s_desc[b][br_word + jl] * a.Hq + h) * D;
    }
#pragma unroll
    for (int s = 0; s < C::KS; ++s) {
      bf16x8 v = {};
      if (live) v = *reinterpret_cast<const bf16x8*>(qp + 16 * s + 8 * g);
      qop[s] = v;
    }
  };

  constexpr int kStores = 2 * (32 / (64 / (D / 16))) + 1;   // store instructions of a wave's rows
  Unit u = start_unit(0);
  if (u.w >= 0) {
    start_rest(u);
    load_q(u, 0);
  }
  bool first = true, stored = false;
  int claim = 0;
  for (int b = 0; u.w >= 0; b ^= 1) {
    const int* dsc = &s_desc[b][0];
    const int npe = u.npe, n2 = u.n2, cw = u.cw, row0 = u.row0, R = u.R;
    const bool live_wave = 32 * wave < R;
    const bool cm = cw != kNoCausal;
    // The first iteration (pair of pages) that holds a token some row of the wave does not see.
    const int itc = cm ? max(0, cw + (row0 + 32 * wave) / a.group + 1) >> 5 : 0x7fffffff;
    // A bit per iteration whose scores need the mask: a page with unused slots (or missing), or a
    // token some row of the wave does not see.
    auto short_page = [&](int p) {
      return p >= npe || ((unsigned)dsc[kDescHead + p] >> kPageValidShift) != kPageTokens - 1;
    };
    const uint64_t masked =
        __ballot(lane >= itc || short_page(2 * lane) || short_page(2 * lane + 1));

    // The first copies, the queries and the claim have landed; the row stores of the unit before,
    // issued after them, need not have.
    if (stored) wait_vmcnt_const<kStores>();
    else wait_vmcnt(0);
    asm volatile("" : "+v"(claim));
    wg_barrier();                       // every wave's first copies have landed, and its rows of
                                        // the unit before no longer need that unit's descriptor
    if (wave == 0) {
      int v;
      if (first) {
        v = unit_of(rank + gs(cs), cs);
      } else {
        int j = 2 * gs(cs) + __builtin_amdgcn_readfirstlane(claim);
        for (int t = 1; j >= n_str && t < ns; ++t) {
          cs = cs + 1 == ns ? 0 : cs + 1;
          int c = 0;
          if (lane == 0) c = atomicAdd(&heads[cs], 1);
          j = 2 * gs(cs) + __builtin_amdgcn_readfirstlane(c);
        }
        v = unit_of(j, cs);
      }
      fetch_desc(v, b ^ 1);
    }
    first = false;

    float m = NEG_INF, l = 0.f;
    f32x16 O[C::NC];
#pragma unroll
    for (int n = 0; n < C::NC; ++n)
#pragma unroll
      for (int i = 0; i < 16; ++i) O[n][i] = 0.f;
    f32x16 S;
    bf16x8 ka[C::KS];                   // the next scores' K operands, read an iteration ahead
    // The lane's row limit: it sees chunk token t only for t <= cl.
    const int cl = cm ? cw + (row0 + 32 * wave + r32) / a.group : 0x3fffffff;

    auto read_k = [&](auto slot, int s) {
      ka[s] = *(lds_bf16x8*)((const lds_uchar*)smem + (int)slot * C::HALF + koff[s]);
    };
    auto mask = [&](int it) {
      // Valid tokens of the pair's pages (a segment of the chain may end inside one).
      const int va0 = (int)((unsigned)__builtin_amdgcn_readfirstlane(dsc[kDescHead + 2 * it]) >>
                            kPageValidShift);
      const int va1 = 2 * it + 1 < npe
                          ? (int)((unsigned)__builtin_amdgcn_readfirstlane(
                                      dsc[kDescHead + 2 * it + 1]) >> kPageValidShift)
                          : -1;
      const int lim0 = min(va0, cl - 32 * it) - 4 * g;
      const int lim1 = min(va1, cl - 32 * it - 16) - 4 * g;
#pragma unroll
      for (int i = 0; i < 16; ++i)
        if (8 * ((i >> 2) & 1) + (i & 3) > (i < 8 ? lim0 : lim1)) S[i] = NEG_INF;
    };
    // One pair of pages: the softmax of its scores S, the next pair's scores, O += P V.  vslot /
    // kslot: ring slots of V of this pair and of K two pairs ahead.  The order of the issue is
    // fixed by hand: each matrix instruction of the next scores is followed by its share of the
    // softmax, V is read from LDS ahead of the products that use it, and the K operands of the
    // next iteration during them.
    auto body = [&](auto vslot, auto kslot, int it) {
      float lm = fmaxf(fmaxf(S[0], S[1]), S[2]);
#pragma unroll
      for (int i = 3; i < 15; i += 2) lm = fmaxf(fmaxf(lm, S[i]), S[i + 1]);
      lm = fmaxf(lm, S[15]) * a.scale_log2;
      if (__any(lm > m + kTau)) {
        const float mn = fmaxf(m, fmaxf(lm, __shfl_xor(lm, 32)));
        const float alpha = mn == NEG_INF ? 1.f : exp2_(m - mn);
        m = mn;
        l *= alpha;
#pragma unroll
        for (int n = 0; n < C::NC; ++n) O[n] *= alpha;
      }
      const float nm = m == NEG_INF ? 0.f : -m;
      const lds_uchar* vb = (const lds_uchar*)smem + (int)vslot * C::HALF;
      bf16x8 va[2][C::NC];
      auto read_v = [&](int s, int n) {
        const s16x4 v0 = __builtin_amdgcn_ds_read_tr16_b64_v4i16(
            (lds_s16x4*)(vb + s * C::KVB + voff[n][0]));
        const s16x4 v1 = __builtin_amdgcn_ds_read_tr16_b64_v4i16(
            (lds_s16x4*)(vb + s * C::KVB + voff[n][1]));
        va[s][n] = __builtin_bit_cast(bf16x8,
                                      __builtin_shufflevector(v0, v1, 0, 1, 2, 3, 4, 5, 6, 7));
      };
#pragma unroll
      for (int n = 0; n < C::NC; ++n) read_v(0, n);
      f32x16 Sn;
#pragma unroll
      for (int i = 0; i < 16; ++i) Sn[i] = 0.f;
      bf16x8 pb[2];
      constexpr int EPK = 16 / C::KS;               // scores handled per matrix instruction
      float ls = 0.f;
#pragma unroll
      for (int s = 0; s < C::KS; ++s) {
        Sn = __builtin_amdgcn_mfma_f32_32x32x16_bf16(ka[s], qop[s], Sn, 0, 0, 0);
        float ps = 0.f;
#pragma unroll
        for (int e = 0; e < EPK; e += 2) {
          const int i = EPK * s + e;
          const float p0 = exp2_(fmaf(S[i], a.scale_log2, nm));
          const float p1 = exp2_(fmaf(S[i + 1], a.scale_log2, nm));
          pb[i >> 3][i & 7] = (__bf16)p0;
          pb[i >> 3][(i & 7) + 1] = (__bf16)p1;
          ps += p0 + p1;
        }
        ls += ps;
        if (s == C::KS / 2 - 1) {
#pragma unroll
          for (int n = 0; n < C::NC; ++n) read_v(1, n);
        }
      }
      l += ls;
#pragma unroll
      for (int s = 0; s < 2; ++s) {
#pragma unroll
        for (int n = 0; n < C::NC; ++n) {
          O[n] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(va[s][n], pb[s], O[n], 0, 0, 0);
          read_k(kslot, s * C::NC + n);
        }
      }
      // The issue order (masks: 0x8 matrix, 0x2 vector, 0x400 transcendental, 0x100 LDS read).
#define GA_SGB(mask, n) __builtin_amdgcn_sched_group_barrier(mask, n, 0)
      GA_SGB(0x100, 2 * C::NC);
#pragma unroll
      for (int s = 0; s < C::KS; ++s) {
        GA_SGB(0x8, 1);
        GA_SGB(0x2, EPK);
        GA_SGB(0x400, EPK);
        GA_SGB(0x2, EPK + EPK / 2);
        if (s >= C::KS / 2) GA_SGB(0x100, 2 * C::NC / (C::KS / 2));
      }
#pragma unroll
      for (int s = 0; s < 2 * C::NC; ++s) {
        GA_SGB(0x8, 1);
        GA_SGB(0x100, 1);
      }
      S = Sn;
    };

    // One iteration: V of the pair three ahead and K of the pair five ahead are copied (the pair's
    // ring slots are compile-time, U = it mod 4).
    auto iteration = [&](auto live, auto ut, int it) {
      constexpr int U = decltype(ut)::value;
      if (it + 5 <= n2) {
        wait_vmcnt_const<4 * C::CPW>();
      } else {
        // (copies after those of K it + 2 and V it, with the unit's end near)
        wait_vmcnt(C::CPW * (max(0, min(2, n2 - it - 3)) + max(0, min(2, n2 - it - 1))));
      }
      lds_barrier();                               // (this wave's operand reads are done, too)
      if (it + 3 < n2)
        copy_v(vq[(U + 3) & 3], vqm[(U + 3) & 3], dst_w + (C::SLOTS + ((U + 3) & 3)) * C::HALF);
      if (it + 5 < n2) {
        const int word = __builtin_amdgcn_readlane(pk, it + 5);
        const unsigned char* base = page_base(u.pool_h, word);
        copy_k(base, dst_w + ((U + 1) & 3) * C::HALF);
        vq[(U + 1) & 3] = base + C::KVB;
        vqm[(U + 1) & 3] = (int)((unsigned)word >> kPageValidShift);
      }
      if constexpr (decltype(live)::value) {
        if ((masked >> it) & 1) mask(it);
        body(ut, std::integral_constant<int, (U + 2) & 3>{}, it);
      }
    };
    auto run = [&](auto live) {
      constexpr bool LIVE = decltype(live)::value;
      if (LIVE && n2 > 0) {
#pragma unroll
        for (int s = 0; s < C::KS; ++s) read_k(std::integral_constant<int, 0>{}, s);
#pragma unroll
        for (int i = 0; i < 16; ++i) S[i] = 0.f;
#pragma unroll
        for (int s = 0; s < C::KS; ++s)
          S = __builtin_amdgcn_mfma_f32_32x32x16_bf16(ka[s], qop[s], S, 0, 0, 0);
#pragma unroll
        for (int s = 0; s < C::KS; ++s) read_k(std::integral_constant<int, 1>{}, s);
      }
      lds_barrier();                               // the first two K slots are free
      if (n2 > 4) copy_k(vq[0] - C::KVB, dst_w);
      for (int it = 0; it < n2; it += 4) {
        iteration(live, std::integral_constant<int, 0>{}, it);
        if (it + 1 >= n2) break;
        iteration(live, std::integral_constant<int, 1>{}, it + 1);
        if (it + 2 >= n2) break;
        iteration(live, std::integral_constant<int, 2>{}, it + 2);
        if (it + 3 >= n2) break;
        iteration(live, std::integral_constant<int, 3>{}, it + 3);
      }
    };
    if (live_wave) run(std::true_type{});
    else run(std::false_type{});
    // Every wave is done with the rings; wave 0's copy of the next descriptor has landed.
    if (wave == 0) wait_vmcnt(0);
    lds_barrier();
    // The next unit's first copies and queries are on their way while this one's rows are stored.
    const Unit done = u;
    const float L = l + __shfl_xor(l, 32);
    u = start_unit(b ^ 1);
    if (u.w >= 0) load_q(u, b ^ 1);
    claim = 0;
    if (u.w >= 0 && wave == 0 && lane == 0) claim = atomicAdd(&heads[cs], 1);
    asm volatile("" ::: "memory");
    stored = live_wave;

    // Rows leave through LDS, so that each store instruction writes whole lines of few rows (a
    // lane holds 4 consecutive columns of a row at a time): D / 2 columns of the 32 rows per round,
    // rows 0 .. 15 in the wave's part of K slot 3 and 16 .. 31 in its part of V slot 2, 16-byte
    // chunks XOR-permuted by row.  Rows past the unit's end repeat its last one, so that every
    // wave that stores issues the same number of stores.
    constexpr int CB = D, NCH = CB / 16, RPI = 64 / NCH, NI = 32 / RPI;
    f16x8 st[2][NI];
    if (live_wave) {
      int g_e = g, r_e = r32, lane_e = lane;
      asm volatile("" : "+v"(g_e), "+v"(r_e), "+v"(lane_e));
      const float inv = L > 0.f ? 1.f / L : 0.f;
      float up = inv;
      int e = 0;
      if (!a.out) {
        float amax = 0.f;
#pragma unroll
        for (int n = 0; n < C::NC; ++n)
#pragma unroll
          for (int i = 0; i < 16; ++i) amax = fmaxf(amax, fabsf(O[n][i]));
        amax = fmaxf(amax, __shfl_xor(amax, 32)) * inv;
        e = max(__builtin_amdgcn_frexp_expf(amax), -100);
        up = __builtin_amdgcn_ldexpf(inv, kPartScaleBits - e);
      }
      auto piece = [&](int row) {
        return smem + ((row >> 4) ? (C::SLOTS + 2) * C::HALF : 3 * C::HALF) +
               wave * C::CPW * 1024 + (row & 15) * CB;
      };
      unsigned char* mine = piece(r_e);
#pragma unroll
      for (int p = 0; p < 2; ++p) {
#pragma unroll
        for (int t = 0; t < C::NC / 2; ++t) {
          const int n = p * (C::NC / 2) + t;
          if (!a.out) {
            // Column 32 n + 8 j + 4 g + i at position 32 n + 16 (j mod 2) + 8 g + 4 (j / 2) + i.
#pragma unroll
            for (int jl = 0; jl < 2; ++jl) {
              f16x8 v;
#pragma unroll
              for (int i = 0; i < 4; ++i) {
                v[i] = (_Float16)(O[n][4 * jl + i] * up);
                v[4 + i] = (_Float16)(O[n][4 * (jl + 2) + i] * up);
              }
              const int c = 4 * t + 2 * jl + g_e;
              *reinterpret_cast<f16x8*>(mine + ((c ^ (r_e & (NCH - 1))) << 4)) = v;
            }
          } else {
#pragma unroll
            for (int j = 0; j < 4; ++j) {
              s16x4 v;
#pragma unroll
              for (int i = 0; i < 4; ++i)
                v[i] = __builtin_bit_cast(short, (__bf16)(O[n][4 * j + i] * up));
              const int c = 4 * t + j;
              *reinterpret_cast<s16x4*>(mine + ((c ^ (r_e & (NCH - 1))) << 4) + 8 * g_e) = v;
            }
          }
        }
#pragma unroll
        for (int k = 0; k < NI; ++k) {
          const int row = min(k * RPI + lane_e / NCH, done.R - 1 - 32 * wave);
          st[p][k] = *reinterpret_cast<const f16x8*>(
              piece(row) + (((lane_e % NCH) ^ (row & (NCH - 1))) << 4));
        }
      }
      asm volatile("" ::: "memory");
      __builtin_amdgcn_s_waitcnt(0xC07F);          // the staged rows are in registers
      asm volatile("" ::: "memory");
      if (u.w >= 0) start_rest(u);
      // Rows of the stores: partial rows, or rows of the output itself.
      auto out_row = [&](int r) {
        int jl, h;
        row_of(done, r, jl, h);
        return a.out ? (int64_t)dsc[br_word + jl] * a.Hq + h
                     : ((int64_t)done.prow_base + done.j0 + jl) * a.Hq + h;
      };
      char* dst = static_cast<char*>(a.out ? a.out : a.po);
#pragma unroll
      for (int k = 0; k < NI; ++k) {
        const int row = min(k * RPI + lane_e / NCH, done.R - 1 - 32 * wave);
        char* rp = dst + out_row(32 * wave + row) * (2 * D) + (lane_e % NCH) * 16;
        *reinterpret_cast<f16x8*>(rp) = st[0][k];
        *reinterpret_cast<f16x8*>(rp + CB) = st[1][k];
      }
      if (g_e == 0 && 32 * wave + r_e < done.R) {
        const int64_t row = out_row(32 * wave + r_e);
        const float lam = m + log2_(L);
        if (a.out)
          a.lse[row] = lam * 0.69314718055994531f;
        else
          *reinterpret_cast<f32x2*>(a.plse + 2 * row) =
              f32x2{lam, __builtin_amdgcn_ldexpf(1.f, e - kPartScaleBits)};
      }
    } else if (u.w >= 0) {
      start_rest(u);
    }
  }
  // The work-stream heads are armed again by the merge, or, without one, by the last workgroup.
  if (a.out && tid == 0) {
    const int n_done = (int)__hip_atomic_fetch_add(reinterpret_cast<int*>(a.counters + 2), 1,
                                                   __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    if (n_done == (int)gridDim.x - 1) {
      for (int i = 0; i < kMaxStreams; ++i) heads[i] = 0;
      a.counters[2] = 0;
    }
  }
}

template <int D>
hipError_t launch_t(const AttnArgs& a, int grid, hipStream_t stream, hipEvent_t t0, hipEvent_t t1) {
  if (t0 || t1)
    hipExtLaunchKernelGGL(k_mq_attn<D>, dim3(grid), dim3(kAttnThreads), 0, stream, t0, t1, 0, a);
  else
    hipLaunchKernelGGL(k_mq_attn<D>, dim3(grid), dim3(kAttnThreads), 0, stream, a);
  return hipGetLastError();
}

}  // namespace

hipError_t launch_mq_attn(const AttnArgs& a, int head_dim, int grid, hipStream_t stream,
                          hipEvent_t t0, hipEvent_t t1) {
  if (head_dim == 64) return launch_t<64>(a, grid, stream, t0, t1);
  if (head_dim == 128) return launch_t<128>(a, grid, stream, t0, t1);
  return hipErrorInvalidValue;
}

}  // namespace ga
