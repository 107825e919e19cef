// Equivalence detection over rollout states and the graph suffix (Sec. 3.2, "Graph
// Construction"; Alg. S.1, Stage 1).
//
// Two states of one prompt's graph that are neither ancestor nor descendant of each other are
// compared by the cosine of their embeddings; pairs at or above kappa are linked, and the
// classes Q(v) are the connected components of the links.  The similarity is a dense
// contraction over the embedding width, so it runs on bf16 MFMA, the width streamed through an
// LDS ring in 32-wide stages that are copied straight from HBM; the squared norms are diagonals
// of the same products.  The epilogue tests every pair (u < v, not ancestor-related by the Euler
// intervals of the generation tree, z_u.z_v >= kappa |z_u| |z_v|) and links the qualifying ones at
// once with a lock-free union-find: the larger root is hooked under the smaller with a
// compare-and-swap, so every class's final root is its smallest state (a deterministic label,
// whatever order the links land in).
//
// Graph suffix: C_g(u) is u's direct successors plus those of the other members of Q(u) that lie
// deeper than u (shared edges only point deeper, so the graph stays acyclic).  One thread per
// state counts them over its prompt's states, and a second pass writes the CSR offsets and the
// lists in ascending state order.
#include "attn_dev.hpp"
#include "equiv_tiles.hpp"
#include "ga_internal.hpp"

#include <type_traits>

namespace ga {
namespace {

typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef float f32x4 __attribute__((ext_vector_type(4)));

__device__ __forceinline__ int load_rep(const int* rep, int x) {
  return __hip_atomic_load(rep + x, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

__device__ __forceinline__ int find_root(const int* rep, int x) {
  int p = load_rep(rep, x);
  while (p != x) {
    x = p;
    p = load_rep(rep, x);
  }
  return x;
}

// Links the classes of a and b: the larger root is hooked under the smaller one.  A failed
// compare-and-swap means another link changed that root first; the roots are looked up again.
__device__ void unite(int* rep, int a, int b) {
  while (true) {
    a = find_root(rep, a);
    b = find_root(rep, b);
    if (a == b) return;
    if (a > b) {
      const int t = a;
      a = b;
      b = t;
    }
    if (atomicCAS(rep + b, b, a) == b) return;
  }
}

// One prompt of at most 256 states in one workgroup (8 waves).  The prompt's embeddings stream
// through an LDS ring of 4 stages of 32 components (256 rows x 64 bytes each), 3 stages in
// flight, copied straight from HBM into LDS (global_load_lds_dwordx4: each lane moves 16 bytes,
// one wave instruction fills 1 KiB = 16 rows; 16-byte chunks are XOR-permuted by row pair so the
// MFMA operand reads are conflict-free).
//
// What bounds it: HBM (each embedding is read once), as long as LDS keeps up.  The upper triangle
// of 64 x 64 blocks goes to the waves as whole blocks: waves 0 to 5 the six blocks off the
// diagonal (16 tiles of 16 x 16 from 8 operand reads per stage), waves 6 and 7 two diagonal blocks
// each (20 tiles from 8 reads), so a stage costs 64 KiB of LDS reads where row strips of single
// tiles (17 tiles from 19 reads per wave) cost 152; and strips without states are not copied.  Both
// together took a pass over 512 prompts of 205 states and width 4096 from 194 to 182 us, the
// staggered start below to 165 us (5.2 TB/s).
// The squared norms are the diagonals of the diagonal tiles (the same fp32 sums as the dot
// products).  Links are made with a union-find in LDS and the labels written at the end.
constexpr int kPromptMax = 256;
constexpr int kPKC = 32;                        // components per stage: one MFMA k-step
constexpr int kPRow = kPKC * 2;                 // bytes of one state row in a stage
constexpr int kPStage = kPromptMax * kPRow;     // 16 KiB
constexpr int kPRing = 4;

// s_waitcnt vmcnt(n) for a runtime n in [0, 4].
__device__ __forceinline__ void wait_vm(int n) {
  asm volatile("" ::: "memory");
  switch (n) {
    case 0: __builtin_amdgcn_s_waitcnt(GA_VMCNT(0)); break;
    case 1: __builtin_amdgcn_s_waitcnt(GA_VMCNT(1)); break;
    case 2: __builtin_amdgcn_s_waitcnt(GA_VMCNT(2)); break;
    case 3: __builtin_amdgcn_s_waitcnt(GA_VMCNT(3)); break;
    default: __builtin_amdgcn_s_waitcnt(GA_VMCNT(4)); break;
  }
}

// The same for n copies of each of AHEAD pieces, n in [0, 4] (0: waits for all).
template <int AHEAD>
__device__ __forceinline__ void wait_stages(int n) {
  static_assert(4 * AHEAD < 64, "vmcnt counts to 63");
  asm volatile("" ::: "memory");
  switch (n) {
    case 0: __builtin_amdgcn_s_waitcnt(GA_VMCNT(0)); break;
    case 1: __builtin_amdgcn_s_waitcnt(GA_VMCNT(AHEAD)); break;
    case 2: __builtin_amdgcn_s_waitcnt(GA_VMCNT(2 * AHEAD)); break;
    case 3: __builtin_amdgcn_s_waitcnt(GA_VMCNT(3 * AHEAD)); break;
    default: __builtin_amdgcn_s_waitcnt(GA_VMCNT(4 * AHEAD)); break;
  }
}

__device__ __forceinline__ int poff(int row, int chunk) {
  return row * kPRow + ((chunk ^ ((row >> 1) & 3)) << 4);
}

__device__ __forceinline__ int lds_find(int* r, int x) {
  int p = __hip_atomic_load(r + x, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
  while (p != x) {
    x = p;
    p = __hip_atomic_load(r + x, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
  }
  return x;
}

__device__ void lds_unite(int* r, int a, int b) {
  while (true) {
    a = lds_find(r, a);
    b = lds_find(r, b);
    if (a == b) return;
    if (a > b) {
      const int t = a;
      a = b;
      b = t;
    }
    if (atomicCAS(r + b, b, a) == b) return;
  }
}

__global__ __launch_bounds__(512, 4) void k_prompt_classes(EquivArgs a) {
  __shared__ __align__(1024) unsigned char ring[kPRing * kPStage];
  __shared__ float s_inv[kPromptMax];
  __shared__ int s_tin[kPromptMax], s_tout[kPromptMax], s_rep[kPromptMax], s_par[kPromptMax];
  const int2 pr = a.prompts[blockIdx.x];          // (first state, states)
  const int s0 = pr.x, n = pr.y;
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int r16 = lane & 15, kg = lane >> 4;
  const int nt = (n + 15) >> 4;                   // 16-row tiles holding states
  unsigned mix = *reinterpret_cast<const unsigned*>(a.z + (int64_t)(s0 + min(lane, n - 1)) * a.dim) *
                 (2 * lane + 1);
  if (tid < kPromptMax) {
    s_rep[tid] = tid;
    s_tin[tid] = tid < n ? a.tin[s0 + tid] : 0;
    s_tout[tid] = tid < n ? a.tout[s0 + tid] : 0;
    s_par[tid] = tid < n ? a.parent[s0 + tid] - s0 : -1;   // prompt-local (< 0 for the root)
  }
#pragma unroll
  for (int o = 32; o > 0; o >>= 1) mix += __shfl_xor((int)mix, o);
  mix *= 2654435761u;
  __syncthreads();

  // Copies: wave w issues instructions q = 2w and 2w + 1 of every stage; instruction q fills rows
  // 16q .. 16q + 15, lane l the LDS chunk l % 4 of row 16q + l / 4 with the global chunk that
  // the permutation puts there.  Rows past the prompt re-read its last state (valid memory;
  // their products are never used).
  const void* pbase = (const void*)uniform64((int64_t)(uintptr_t)(a.z + (int64_t)s0 * a.dim));
  unsigned coff[2];
#pragma unroll
  for (int j = 0; j < 2; ++j) {
    const int row = 16 * (2 * wave + j) + (lane >> 2);
    const int chunk = (lane & 3) ^ ((row >> 1) & 3);
    coff[j] = (unsigned)(min(row, n - 1) * a.dim * 2 + chunk * 16);
  }
  const unsigned lds_ring = (unsigned)(uintptr_t)(__attribute__((address_space(3))) unsigned char*)ring;
  const int nst = a.dim / kPKC;
  // Workgroups start at different components and wrap around: rows of a power-of-two width lie on
  // one memory channel at a time, and all prompts at the same stage crowd onto few of them (182 us
  // with one start for all, 165 with 64).  The start follows from the prompt's own embeddings (the
  // first two components of its first 64 states), not from its place in the batch, so a prompt's
  // sums are taken in the same order, and have the same bits, wherever it stands.
  const int st0 = (int)((int64_t)(__builtin_amdgcn_readfirstlane((int)mix) >> 26 & 63) * nst >> 6);
  auto issue = [&](int st) {
    const int at = st0 + st < nst ? st0 + st : st0 + st - nst;
#pragma unroll
    for (int j = 0; j < 2; ++j)
      if (2 * wave + j < nt)                      // (strips without states are not copied)
        dma16_cached(coff[j] + (unsigned)(at * kPRow), pbase,
                     __builtin_amdgcn_readfirstlane(lds_ring + (st % kPRing) * kPStage +
                                                    (2 * wave + j) * 1024));
  };
  const int ncp = max(0, min(2, nt - 2 * wave));  // copies of this wave per stage
  auto next_stage = [&](int st) {
    wait_vm(ncp * min(nst - 1 - st, kPRing - 2)); // this wave's copies of stage st have landed
    lds_barrier();                                // ... and every wave's; stage st - 1 is done (its
                                                  // operand reads have returned)
    if (st + kPRing - 1 < nst) issue(st + kPRing - 1);
  };
  const int fo = poff(r16, kg);                   // this lane's chunk of a 16-row strip
  auto operand = [&](int st, int strip) {
    return *reinterpret_cast<const bf16x8*>(ring + (st % kPRing) * kPStage + strip * 16 * kPRow +
                                            fo);
  };
  // t[i] = z_u . z_v, u = 16 strip + 4 kg + i, v = 16 col + r16 (prompt-local): a bit per i whose
  // cosine reaches kappa.
  auto test_tile = [&](f32x4 t, int strip, int col) {
    asm volatile("" ::: "memory");                // (no tile's LDS reads move up into another's)
    const int v = col * 16 + r16;
    uint64_t hit = 0;
    if (v >= n) return hit;
    const float nv = s_inv[v];
    const int pv = a.edge_sim ? s_par[v] : -1;
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      const int u = strip * 16 + 4 * kg + i;
      if (u >= v) continue;
      const float cs = t[i] * s_inv[u] * nv;
      if (cs >= a.kappa) hit |= 1u << i;
      if (pv == u) a.edge_sim[s0 + v] = cs;
    }
    return hit;
  };
  auto link = [&](int u, int v) {
    const int tin_u = s_tin[u], tin_v = s_tin[v];
    const bool related =
        (tin_u <= tin_v && tin_v < s_tout[u]) || (tin_v <= tin_u && tin_u < s_tout[v]);
    if (!related) lds_unite(s_rep, u, v);
  };
  for (int st = 0; st < kPRing - 1 && st < nst; ++st) issue(st);
  // Blocks (bi, bj), bi < bj, of waves 0 .. 5; diagonal blocks bi and 3 - bi of waves 6 and 7.  A
  // wave whose (first) block has no states only copies; strips without states inside a block are
  // computed on whatever LDS holds, and their results not looked at.
  const int bi = wave < 3 ? 0 : wave < 5 ? 1 : wave < 6 ? 2 : wave - 6;
  const int bj = wave < 3 ? wave + 1 : wave < 5 ? wave - 1 : wave < 6 ? 3 : wave - 6;
  if (64 * bj >= n) {
    for (int st = 0; st < nst; ++st) next_stage(st);
    __syncthreads();                              // (the norms)
  } else if (wave < 6) {
    f32x4 acc[4][4];
#pragma unroll
    for (int x = 0; x < 4; ++x)
#pragma unroll
      for (int y = 0; y < 4; ++y) acc[x][y] = f32x4{0.f, 0.f, 0.f, 0.f};
    for (int st = 0; st < nst; ++st) {
      next_stage(st);
      bf16x8 av[4], bv[4];
#pragma unroll
      for (int x = 0; x < 4; ++x) {
        av[x] = operand(st, 4 * bi + x);
        bv[x] = operand(st, 4 * bj + x);
      }
#pragma unroll
      for (int x = 0; x < 4; ++x)
#pragma unroll
        for (int y = 0; y < 4; ++y)
          acc[x][y] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(av[x], bv[y], acc[x][y], 0, 0, 0);
    }
    __syncthreads();                              // the norms
    uint64_t hits = 0;                            // bit 16 x + 4 y + i
#pragma unroll
    for (int x = 0; x < 4; ++x)
#pragma unroll
      for (int y = 0; y < 4; ++y)
        hits |= test_tile(acc[x][y], 4 * bi + x, 4 * bj + y) << (16 * x + 4 * y);
    for (; hits; hits &= hits - 1) {
      const int k = __builtin_ctzll(hits);
      link(64 * bi + 16 * (k >> 4) + 4 * kg + (k & 3), 64 * bj + 16 * ((k >> 2) & 3) + r16);
    }
  } else {                                        // two blocks of the diagonal
    f32x4 acc[2][10];                             // tiles (x, y), x <= y, in row order
#pragma unroll
    for (int d = 0; d < 2; ++d)
#pragma unroll
      for (int k = 0; k < 10; ++k) acc[d][k] = f32x4{0.f, 0.f, 0.f, 0.f};
    for (int st = 0; st < nst; ++st) {
      next_stage(st);
#pragma unroll
      for (int d = 0; d < 2; ++d) {
        const int bd = d ? 3 - bi : bi;
        bf16x8 av[4];
#pragma unroll
        for (int x = 0; x < 4; ++x) av[x] = operand(st, 4 * bd + x);
        int k = 0;
#pragma unroll
        for (int x = 0; x < 4; ++x)
#pragma unroll
          for (int y = x; y < 4; ++y, ++k)
            acc[d][k] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(av[x], av[y], acc[d][k], 0, 0, 0);
      }
    }
    // Squared norms: row 16 strip + m of a diagonal tile sits in lane (r16 = m, kg = m / 4),
    // element m % 4.
#pragma unroll
    for (int d = 0; d < 2; ++d)
#pragma unroll
      for (int x = 0; x < 4; ++x)
#pragma unroll
        for (int i = 0; i < 4; ++i)
          if (4 * kg + i == r16) {
            const float q = acc[d][x * 4 - x * (x - 1) / 2][i];
            s_inv[64 * (d ? 3 - bi : bi) + 16 * x + r16] =
                q > 0.f ? 1.f / sqrtf(q) : __builtin_nanf("");
          }
    __syncthreads();
#pragma unroll
    for (int d = 0; d < 2; ++d) {
      const int bd = d ? 3 - bi : bi;
      if (64 * bd >= n) continue;
      uint64_t hits = 0;
      int t = 0;
#pragma unroll
      for (int x = 0; x < 4; ++x)
#pragma unroll
        for (int y = x; y < 4; ++y, ++t)
          hits |= test_tile(acc[d][t], 4 * bd + x, 4 * bd + y) << (16 * x + 4 * y);
      for (; hits; hits &= hits - 1) {
        const int k = __builtin_ctzll(hits);
        link(64 * bd + 16 * (k >> 4) + 4 * kg + (k & 3), 64 * bd + 16 * ((k >> 2) & 3) + r16);
      }
    }
  }
  __syncthreads();
  if (tid < n) {
    a.labels[s0 + tid] = s0 + lds_find(s_rep, tid);
    if (a.edge_sim && s_par[tid] < 0) a.edge_sim[s0 + tid] = 0.f;
  }
}

// Prompts of more than 256 states: tiles of their upper triangles, one workgroup each; 128 x 128, or
// 64 x 64 in batches of few tiles (the host's choice, equiv_tiles.hpp).
//
// What bounds it: with many tiles, no one unit (64 prompts of 517 states, width 4096: matrix cores busy
// 34% of the time, vector instructions 22%, LDS 15%, and 0.8 to 1.0 GB read past the L2s for 0.27
// GB of embeddings) but a barrier per 20 products and the second, partly filled round of tiles.  64 x 64
// tiles (16 flops per operand byte) staged through registers, after a pass of their own over the
// embeddings for the norms, took 322 + 42 us; 128 x 128 tiles take 165 us (590 TFLOP/s over whole
// tiles) and no pass before them.  With few, the chain
// of stages of one tile, each a barrier, the operand reads and the products one after another (about
// 1,200 cycles at 128 x 128 and 32 components): smaller tiles in stages of 64 components shorten it.
// One prompt of 300 states, us a call: 128 x 128 64, the register-staged tiles 37, 64 x 64 in stages of
// 32 components (ring of four) 37, in stages of 64 26; 8 of 517 67, 60, 43 and 35.  (More stages in
// flight change nothing: a ring of nine 128 x 128 stages 66.)
// Four waves hold a quadrant each (64 x 64: 16 tiles of 16 x 16 from 8 operand reads per 32
// components; 32 x 32: 4 from 4).  The ring (3 stages of 16 KiB with two in flight, or 2 with one)
// lets three or four workgroups share a CU.  The squared norms of a tile's rows and columns are the
// diagonals of more products per wave (a half of its quadrant's row strips and of its column strips:
// every wave orders its strips so that those come first), so no pass over the embeddings is needed
// for them.  A quadrant without states, or below the diagonal, only takes part in the copies and
// norms.  Both sizes sum in the same order, so a prompt's bits do not depend on the batch.  The host
// deals the tiles of a prompt to as few XCDs as the balance allows, whose L2s then serve all but the
// first read of a row.
template <int Q>                                  // 16-state strips along a quadrant: 4 or 2
struct TCfg {
  static constexpr int TILE = 32 * Q;
  static constexpr int KS = Q == 4 ? 1 : 2;       // pieces of 32 components of a stage
  static constexpr int HALF = TILE * kPRow;       // rows (then columns) of a piece
  static constexpr int PIECE = 2 * HALF;
  static constexpr int STAGE = KS * PIECE;        // 16 KiB
  static constexpr int RING = Q == 4 ? 3 : 2;
  static constexpr int WPC = Q == 4 ? 3 : 4;      // workgroups per CU
};

#pragma clang diagnostic push
#pragma clang diagnostic ignored "-Winline-asm"
// The same copy from a 64-bit address per lane (rows of any width).
__device__ __forceinline__ void dma16_at(const void* p, unsigned lds_base) {
  asm volatile("s_mov_b32 m0, %1\n\tglobal_load_lds_dwordx4 %0, off"
               :: "v"(p), "s"(lds_base) : "memory", "m0");
}
#pragma clang diagnostic pop

__global__ void k_rep_init(EquivArgs a) {
  const int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x;
  if (i < a.n_big) a.rep[a.big[i]] = a.big[i];
}

template <int Q>
__global__ __launch_bounds__(256, TCfg<Q>::WPC) void k_sim_union(EquivArgs a) {
  using C = TCfg<Q>;
  constexpr int H = Q / 2;                        // row (and column) strips a wave copies, and sums
                                                  // the norms of
  __shared__ __align__(1024) unsigned char ring[C::RING * C::STAGE];
  __shared__ float s_inv[2][C::TILE];
  const int4 it = a.items[blockIdx.x];            // (first row state, first column state, prompt end)
  const int i0 = it.x, j0 = it.y, pend = it.z;
  if (i0 >= pend) return;                         // (pads an XCD's list)
  const bool diag = i0 == j0;
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int r16 = lane & 15, kg = lane >> 4;
  const int wm = wave >> 1, wn = wave & 1;
  const int nst = a.dim / (kPKC * C::KS);         // (the width is a multiple of 64)
  // Copies: each wave fills row strips H w .. H w + H - 1 and, off the diagonal, the column strips of
  // those numbers; strips without states are left out, rows past the prompt re-read its last state.
  const unsigned short* src[Q];
  bool have[Q];
  int ncp = 0;
#pragma unroll
  for (int j = 0; j < Q; ++j) {
    const int first = (j < H ? i0 : j0) + 16 * (H * wave + j % H);
    const int row = min(first + (lane >> 2), pend - 1);
    const int chunk = (lane & 3) ^ ((lane >> 3) & 3);
    src[j] = a.z + (int64_t)row * a.dim + chunk * 8;
    have[j] = first < pend && (j < H || !diag);
    ncp += have[j];
  }
  const unsigned lds_ring = (unsigned)(uintptr_t)(__attribute__((address_space(3))) unsigned char*)ring;
  auto issue = [&](unsigned slot) {
#pragma unroll
    for (int j = 0; j < Q; ++j)
      if (have[j]) {
#pragma unroll
        for (int k = 0; k < C::KS; ++k) {
          dma16_at(src[j], __builtin_amdgcn_readfirstlane(lds_ring + slot + k * C::PIECE +
                                                          (j / H) * C::HALF +
                                                          (H * wave + j % H) * 1024));
          src[j] += kPKC;
        }
      }
  };
  // Strip x of the wave's rows and of its columns: those whose norms it computes come first.
  auto rstrip = [&](int x) { return Q * wm + (x ^ (H * wn)); };
  auto cstrip = [&](int y) { return Q * wn + (y ^ (H * wm)); };
  const int fo = poff(r16, kg), cbase = diag ? 0 : C::HALF;
  f32x4 acc[Q][Q], sa[H], sb[H];
#pragma unroll
  for (int x = 0; x < H; ++x) sa[x] = sb[x] = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
  for (int x = 0; x < Q; ++x) {
#pragma unroll
    for (int y = 0; y < Q; ++y) acc[x][y] = f32x4{0.f, 0.f, 0.f, 0.f};
  }
  auto stages = [&](auto quad) {
    constexpr int NS = decltype(quad)::value ? Q : H;
    unsigned slot = 0, fill = (C::RING - 1) * C::STAGE;
    // The norms' sums are all of one sign and lose most where a chain of products is long (3.9e-7
    // against 3.1e-7 of the similarities at width 4096), so they are taken over 128 components at
    // a time.
    for (int b0 = 0; b0 < nst; b0 += 4 / C::KS) {
      const int b1 = min(b0 + 4 / C::KS, nst);
      f32x4 qa[H], qb[H];
#pragma unroll
      for (int x = 0; x < H; ++x) qa[x] = qb[x] = f32x4{0.f, 0.f, 0.f, 0.f};
      for (int st = b0; st < b1; ++st) {
        // This wave's copies of the stage have landed ...
        wait_stages<C::KS * (C::RING - 2)>(st + C::RING - 2 < nst ? ncp : 0);
        lds_barrier();                            // ... and every wave's; the stage before is done
        if (st + C::RING - 1 < nst) issue(fill);
#pragma unroll
        for (int k = 0; k < C::KS; ++k) {
          bf16x8 av[NS], bv[NS];
#pragma unroll
          for (int x = 0; x < NS; ++x) {
            av[x] = *reinterpret_cast<const bf16x8*>(ring + slot + k * C::PIECE + rstrip(x) * 1024 + fo);
            bv[x] = *reinterpret_cast<const bf16x8*>(ring + slot + k * C::PIECE + cbase + cstrip(x) * 1024 + fo);
          }
#pragma unroll
          for (int x = 0; x < H; ++x) {
            qa[x] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(av[x], av[x], qa[x], 0, 0, 0);
            qb[x] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(bv[x], bv[x], qb[x], 0, 0, 0);
          }
          if constexpr (NS == Q) {
#pragma unroll
            for (int x = 0; x < Q; ++x)
#pragma unroll
              for (int y = 0; y < Q; ++y)
                acc[x][y] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(av[x], bv[y], acc[x][y], 0, 0, 0);
          }
        }
        fill = slot;
        slot = slot + C::STAGE == C::RING * C::STAGE ? 0 : slot + C::STAGE;
      }
#pragma unroll
      for (int x = 0; x < H; ++x) {
        sa[x] += qa[x];
        sb[x] += qb[x];
      }
    }
  };
  for (int st = 0; st < C::RING - 1 && st < nst; ++st) issue(st * C::STAGE);
  const bool quad = i0 + 16 * Q * wm < pend && j0 + 16 * Q * wn < pend && !(diag && wm > wn);
  if (quad) stages(std::true_type{});
  else stages(std::false_type{});
  // Squared norms: row m of a strip sits in lane (r16 = m, kg = m / 4), element m % 4.
#pragma unroll
  for (int x = 0; x < H; ++x)
#pragma unroll
    for (int i = 0; i < 4; ++i)
      if (4 * kg + i == r16) {
        const float p = sa[x][i], q = sb[x][i];
        s_inv[0][16 * rstrip(x) + r16] = p > 0.f ? 1.f / sqrtf(p) : __builtin_nanf("");
        s_inv[1][16 * cstrip(x) + r16] = q > 0.f ? 1.f / sqrtf(q) : __builtin_nanf("");
      }
  __syncthreads();
  if (!quad) return;
  // acc[x][y][i] = z_u . z_v with u the row state (4 kg + i of strip x), v the column state (r16 of
  // strip y): a bit (16 x + 4 y + i) per cosine that reaches kappa, then the links.
  uint64_t hits = 0;
#pragma unroll
  for (int y = 0; y < Q; ++y) {
    const int v = j0 + 16 * cstrip(y) + r16;
    if (v >= pend) continue;
    const float nv = s_inv[1][v - j0];
    const int pv = a.edge_sim ? a.parent[v] : -1;
#pragma unroll
    for (int x = 0; x < Q; ++x)
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        const int u = i0 + 16 * rstrip(x) + 4 * kg + i;
        if (u >= v) continue;
        const float cs = acc[x][y][i] * s_inv[0][u - i0] * nv;
        if (cs >= a.kappa) hits |= 1ull << (16 * x + 4 * y + i);
        if (pv == u) a.edge_sim[v] = cs;
      }
  }
  for (; hits; hits &= hits - 1) {
    const int k = __builtin_ctzll(hits);
    const int u = i0 + 16 * rstrip(k >> 4) + 4 * kg + (k & 3);
    const int v = j0 + 16 * cstrip((k >> 2) & 3) + r16;
    const int tin_u = a.tin[u], tin_v = a.tin[v];
    const bool related =
        (tin_u <= tin_v && tin_v < a.tout[u]) || (tin_v <= tin_u && tin_u < a.tout[v]);
    if (!related) unite(a.rep, u, v);
  }
}

// Final labels: every state's root (all links have landed: kernel boundary).
__global__ void k_labels(EquivArgs a) {
  const int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x;
  if (i >= a.n_big) return;
  const int v = a.big[i];
  a.labels[v] = find_root(a.rep, v);
  if (a.edge_sim && a.parent[v] < 0) a.edge_sim[v] = 0.f;
}

// Graph suffix, pass 1 (count into cnt[u], block totals into blk) or pass 2 (offsets and lists).
//
// What bounds it: the scan's LDS reads (a prompt's states, once per state of the prompt) and, for
// the small batches of a step, launches.  A state c belongs to C_g(u) exactly when its source p(c)
// carries u's label and c lies deeper than u (u's own successors among them), so one 8-byte word
// (label of p(c), depth of c) per state is staged, in pieces of the block's span, where three
// dependent reads per state took 37 us a pass on 512 prompts of 205 states (now 12 and 16).  Pass
// 2 adds the block totals before its own itself and writes offsets and lists only if the list fits
// the caller's buffer, so that the host need not wait for the total in between (five kernels, two
// copies and a wait before: 91 us of device work, now 28).
constexpr int kSufStage = 1024;
constexpr int kSufBlock = 256;
constexpr int64_t kSufDirect = 4096;             // block totals that every block adds up by itself

template <bool FILL>
__global__ __launch_bounds__(kSufBlock) void k_suffix(SuffixArgs a) {
  __shared__ int2 s_key[kSufStage + 8];
  __shared__ int64_t s_red[2][kSufBlock / 64];
  __shared__ int s_wsum[kSufBlock / 64];
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int64_t base = (int64_t)blockIdx.x * kSufBlock;
  const int64_t u = base + tid;
  const bool live = u < a.N;
  const int lo = a.pstart[base], hi = a.pend[min(base + kSufBlock, a.N) - 1];
  const int lu = live ? a.labels[u] : 0, du = live ? a.depth[u] : 0;
  const int c0 = live ? a.pstart[u] : 0, c1 = live ? a.pend[u] : 0;
  int64_t k = 0;
  bool fits = true;
  if (FILL) {
    int64_t total;
    if (a.nblk <= kSufDirect) {
      int64_t before = 0, all = 0;
      for (int64_t i = tid; i < a.nblk; i += kSufBlock) {
        const int64_t x = a.blk[i];
        all += x;
        if (i < (int64_t)blockIdx.x) before += x;
      }
#pragma unroll
      for (int o = 32; o > 0; o >>= 1) {
        before += __shfl_xor(before, o);
        all += __shfl_xor(all, o);
      }
      if (lane == 0) {
        s_red[0][wave] = before;
        s_red[1][wave] = all;
      }
      total = 0;
    } else {
      k = a.blk[blockIdx.x];                     // (scanned by k_suffix_blocks)
      total = a.blk[a.nblk];
    }
    const int n = live ? a.cnt[u] : 0;
    int x = n;
#pragma unroll
    for (int o = 1; o < 64; o <<= 1) {
      const int y = __shfl_up(x, o);
      if (lane >= o) x += y;
    }
    if (lane == 63) s_wsum[wave] = x;
    __syncthreads();
    if (a.nblk <= kSufDirect)
      for (int w = 0; w < kSufBlock / 64; ++w) {
        k += s_red[0][w];
        total += s_red[1][w];
      }
    for (int w = 0; w < wave; ++w) k += s_wsum[w];
    k += x - n;
    fits = total <= a.capacity && (total == 0 || a.states);
    if (blockIdx.x == 0 && tid == 0) *a.total = total;
    if (live && fits) {
      a.off[u] = k;
      if (u == a.N - 1) a.off[a.N] = total;
    }
  }
  if (fits) {
    for (int t0 = lo; t0 < hi; t0 += kSufStage) {
      const int m = min(kSufStage, hi - t0);
      __syncthreads();
      for (int i = tid; i < m; i += kSufBlock) {
        const int p = a.parent[t0 + i];
        s_key[i] = p >= 0 ? make_int2(a.labels[p], a.depth[t0 + i]) : make_int2(0, -1);
      }
      __syncthreads();
      const int e = min(c1 - t0, m);
      // Eight words are read before the first is looked at (the array ends in as many spare ones).
      for (int c = max(c0 - t0, 0); c < e; c += 8) {
        int2 key[8];
#pragma unroll
        for (int j = 0; j < 8; ++j) key[j] = s_key[c + j];
#pragma unroll
        for (int j = 0; j < 8; ++j)
          if (key[j].x == lu && key[j].y > du && c + j < e) {
            if (FILL) a.states[k] = t0 + c + j;
            ++k;
          }
      }
    }
  }
  if (!FILL) {
    if (live) a.cnt[u] = (int)k;
    int64_t x = k;
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) x += __shfl_xor(x, o);
    if (lane == 0) s_red[0][wave] = x;
    __syncthreads();
    if (tid == 0) {
      int64_t t = 0;
      for (int w = 0; w < kSufBlock / 64; ++w) t += s_red[0][w];
      a.blk[blockIdx.x] = t;
    }
  }
}

// Exclusive scan of the block totals in place, their sum behind them (large batches only).
__global__ __launch_bounds__(1024) void k_suffix_blocks(SuffixArgs a) {
  __shared__ int64_t s_wsum[16];
  const int t = threadIdx.x, lane = t & 63, w = t >> 6;
  int64_t carry = 0;
  for (int64_t b0 = 0; b0 < a.nblk; b0 += 1024) {
    const int64_t i = b0 + t;
    const int64_t v = i < a.nblk ? a.blk[i] : 0;
    int64_t x = v;
    for (int o = 1; o < 64; o <<= 1) {
      const int64_t y = __shfl_up(x, o);
      if (lane >= o) x += y;
    }
    if (lane == 63) s_wsum[w] = x;
    __syncthreads();
    int64_t before = carry;
    for (int k = 0; k < 16; ++k) {
      if (k < w) before += s_wsum[k];
      carry += s_wsum[k];
    }
    if (i < a.nblk) a.blk[i] = before + x - v;
    __syncthreads();
  }
  if (t == 0) a.blk[a.nblk] = carry;
}

}  // namespace

hipError_t launch_equivalence(const EquivArgs& a, hipStream_t stream) {
  if (a.n_prompts > 0)
    hipLaunchKernelGGL(k_prompt_classes, dim3((unsigned)a.n_prompts), dim3(512), 0, stream, a);
  if (a.n_big > 0) {
    hipLaunchKernelGGL(k_rep_init, dim3((unsigned)((a.n_big + 255) / 256)), dim3(256), 0, stream, a);
    if (a.n_items > 0 && a.tile == TCfg<4>::TILE)
      hipLaunchKernelGGL(k_sim_union<4>, dim3((unsigned)a.n_items), dim3(256), 0, stream, a);
    else if (a.n_items > 0)
      hipLaunchKernelGGL(k_sim_union<2>, dim3((unsigned)a.n_items), dim3(256), 0, stream, a);
    hipLaunchKernelGGL(k_labels, dim3((unsigned)((a.n_big + 255) / 256)), dim3(256), 0, stream, a);
  }
  return hipGetLastError();
}

hipError_t launch_suffix_count(const SuffixArgs& args, hipStream_t stream) {
  if (args.N == 0) return hipSuccess;
  SuffixArgs a = args;
  a.nblk = (a.N + kSufBlock - 1) / kSufBlock;
  hipLaunchKernelGGL(k_suffix<false>, dim3((unsigned)a.nblk), dim3(kSufBlock), 0, stream, a);
  if (a.nblk > kSufDirect) hipLaunchKernelGGL(k_suffix_blocks, dim3(1), dim3(1024), 0, stream, a);
  return hipGetLastError();
}

hipError_t launch_suffix_fill(const SuffixArgs& args, hipStream_t stream) {
  if (args.N == 0) return hipSuccess;
  SuffixArgs a = args;
  a.nblk = (a.N + kSufBlock - 1) / kSufBlock;
  hipLaunchKernelGGL(k_suffix<true>, dim3((unsigned)a.nblk), dim3(kSufBlock), 0, stream, a);
  return hipGetLastError();
}

}  // namespace ga
