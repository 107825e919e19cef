// Graph reward and dual-group advantage over the rollout states (Sec. 3.3-3.4; Alg. S.1,
// Stages 2-3), one pass per step over all states of a batch.
//
//   outcomes   c_own / t_own: sums over the terminal states of each state's subtree.  With the
//              states placed in Euler order (tin), a subtree is the contiguous range
//              [tin(v), tout(v)), so one prefix sum of the packed (R, 1) values of terminal states
//              gives every subtree's sums as a difference (integers: exact).
//   pooling    class totals by integer atomics (exact, so the order they land in is irrelevant);
//              S(v) = (c + w (C_Q - c)) / (t + w (T_Q - t)) in fp64, NaN without evidence.
//   step       r(v) = (S(v) - S(p(v))) (1 - max(0, sim(p(v), v))) on the edge into v.
//   correctness  the group of source u is E_cor(u) = {edges into C_g(u)}: u's successors plus
//              those of its class partners that lie deeper than u, found by one scan over the
//              prompt's states; mean and population std of the defined rewards; the edge into v
//              takes its z-score in the group of p(v) (0 without spread or reward; a spread of
//              at most kSpreadFloor is none: rewards equal by the definition differ by rounding).
//   efficiency per class of two or more (found by its smallest member): the deepest proper
//              ancestor a_Q of all members, route lengths l = d(v) - d(a_Q), z-scores of -l
//              gated by the class's mean defined score; every edge then sums, in a fixed order
//              (ascending state or Euler order), the values of the members in its subtree whose
//              anchor lies above it.
//   dual       A_dual = A_cor + lambda A_eff.
// Every value is computed in a fixed order, so the results are deterministic.
#include "ga_internal.hpp"

namespace ga {
namespace {

constexpr int kB = 256;
// Scores lie in [0, 1] and |r| <= 2: rewards equal by the definition differ by fp64 rounding
// (~1e-16) at most, unequal ones by far more, so a correctness group spread at or below this
// is taken as none (its z-scores are 0) rather than rounding blown up to order one.
constexpr double kSpreadFloor = 1e-12;

__device__ __forceinline__ int64_t gid() { return (int64_t)blockIdx.x * kB + threadIdx.x; }

__global__ void k_outcome_vals(RewardArgs a) {
  const int64_t v = gid();
  if (v >= a.N) return;
  // A label must name a state of the same prompt no later than v (the smallest member of v's
  // class); anything else is read as v itself, so no index leaves the prompt.
  const int l = a.labels[v];
  a.lab[v] = (l >= a.pstart[v] && l <= (int)v) ? l : (int)v;
  const int r = a.reward[v];
  a.euler[a.tin[v]] = r >= 0 ? (((int64_t)r << 32) | 1) : 0;
  a.ctot[v] = 0;                                  // class totals, indexed by label
}

// Exclusive scan of euler[0, N) into pre[0, N] over many workgroups (block totals first).
__global__ __launch_bounds__(1024) void k_pre_sums(RewardArgs a) {
  __shared__ int64_t red[16];
  const int64_t i = (int64_t)blockIdx.x * 1024 + threadIdx.x;
  int64_t v = i < a.N ? a.euler[i] : 0;
  for (int o = 32; o > 0; o >>= 1) v += __shfl_xor(v, o);
  if ((threadIdx.x & 63) == 0) red[threadIdx.x >> 6] = v;
  __syncthreads();
  if (threadIdx.x == 0) {
    int64_t t = 0;
    for (int w = 0; w < 16; ++w) t += red[w];
    a.blk[blockIdx.x] = t;
  }
}

__global__ __launch_bounds__(1024) void k_pre_apply(RewardArgs a) {
  __shared__ int64_t red[16], wsum[16];
  const int t = threadIdx.x, lane = t & 63, w = t >> 6;
  int64_t pre = 0;
  for (int k = t; k < (int)blockIdx.x; k += 1024) pre += a.blk[k];
  for (int o = 32; o > 0; o >>= 1) pre += __shfl_xor(pre, o);
  if (lane == 0) red[w] = pre;
  __syncthreads();
  int64_t base = 0;
  for (int k = 0; k < 16; ++k) base += red[k];
  const int64_t i = (int64_t)blockIdx.x * 1024 + t;
  const int64_t v = i < a.N ? a.euler[i] : 0;
  int64_t x = v;
  for (int o = 1; o < 64; o <<= 1) {
    const int64_t y = __shfl_up(x, o);
    if (lane >= o) x += y;
  }
  if (lane == 63) wsum[w] = x;
  __syncthreads();
  int64_t before = 0;
  for (int k = 0; k < w; ++k) before += wsum[k];
  if (i < a.N) a.pre[i] = base + before + x - v;
  if (i == a.N - 1) a.pre[a.N] = base + before + x;
}

// Own outcomes (packed: correct << 32 | terminal states) and their class totals.
__global__ void k_own(RewardArgs a) {
  const int64_t v = gid();
  if (v >= a.N) return;
  const int64_t own = a.pre[a.tout[v]] - a.pre[a.tin[v]];
  a.own[v] = own;
  atomicAdd(reinterpret_cast<unsigned long long*>(a.ctot + a.lab[v]), (unsigned long long)own);
}

__global__ void k_scores(RewardArgs a) {
  const int64_t v = gid();
  if (v >= a.N) return;
  const int64_t own = a.own[v], tot = a.ctot[a.lab[v]];
  const double c = (double)(own >> 32), t = (double)(own & 0xffffffffLL);
  const double C = (double)(tot >> 32), T = (double)(tot & 0xffffffffLL);
  const double num = c + a.w * (C - c), den = t + a.w * (T - t);
  a.score[v] = den > 0.0 ? num / den : __builtin_nan("");
  a.anchor[v] = -1;                               // set for class members by the next kernel
  a.aeff_node[v] = 0.0;
}

// Step rewards; and, for the smallest member of each class of two or more, the class's
// anchor, its members' efficiency values and their anchors.
__global__ void k_step_and_classes(RewardArgs a) {
  const int64_t v = gid();
  if (v >= a.N) return;
  const int p = a.parent[v];
  double r = __builtin_nan("");
  if (p >= 0) {
    const double s = fmax(0.0, (double)a.edge_sim[v]);
    r = (a.score[v] - a.score[p]) * (1.0 - s);
  }
  a.step[v] = r;
  if (a.lab[v] != (int)v) return;               // not the smallest member of its class
  const int lo = a.pstart[v], hi = a.pend[v];
  int m = 0, lca = -1;
  double ssum = 0.0;
  int sdef = 0;
  for (int x = (int)v; x < hi; ++x) {
    if (a.lab[x] != (int)v) continue;
    ++m;
    if (!isnan(a.score[x])) {
      ssum += a.score[x];
      ++sdef;
    }
    if (lca < 0) {
      lca = x;
      continue;
    }
    int y = x, z = lca;                            // lowest common ancestor by depth walking
    while (a.depth[y] > a.depth[z]) y = a.parent[y];
    while (a.depth[z] > a.depth[y]) z = a.parent[z];
    while (y != z) {
      y = a.parent[y];
      z = a.parent[z];
    }
    lca = y;
  }
  (void)lo;
  if (m < 2) return;
  const int anc = a.lab[lca] == (int)v ? a.parent[lca] : lca;   // a proper ancestor of all
  if (anc < 0) return;                             // a class holding its prompt's root
  const double gate = sdef > 0 ? ssum / sdef : 0.0;
  double lsum = 0.0;
  for (int x = (int)v; x < hi; ++x)
    if (a.lab[x] == (int)v) lsum += -(double)(a.depth[x] - a.depth[anc]);
  const double mean = lsum / m;
  double q = 0.0;
  for (int x = (int)v; x < hi; ++x)
    if (a.lab[x] == (int)v) {
      const double d = -(double)(a.depth[x] - a.depth[anc]) - mean;
      q += d * d;
    }
  const double sd = sqrt(q / m);
  for (int x = (int)v; x < hi; ++x)
    if (a.lab[x] == (int)v) {
      const double l = -(double)(a.depth[x] - a.depth[anc]);
      a.aeff_node[x] = sd > 0.0 ? gate * (l - mean) / sd : 0.0;
      a.anchor[x] = anc;
    }
}

// Correctness-group statistics of every source state u (over E_cor(u)), and the efficiency
// value of the edge into every state.
__global__ void k_groups_and_routes(RewardArgs a) {
  const int64_t u = gid();
  if (u >= a.N) return;
  const int lu = a.lab[u], du = a.depth[u], lo = a.pstart[u], hi = a.pend[u];
  int n = 0, members = 0;
  double s = 0.0;
  for (int c = lo; c < hi; ++c) {
    const int p = a.parent[c];
    if (p < 0 || !(p == (int)u || (a.lab[p] == lu && a.depth[c] > du))) continue;
    ++members;
    if (isnan(a.step[c])) continue;
    s += a.step[c];
    ++n;
  }
  double mean = 0.0, sd = 0.0;
  if (members > 1 && n > 0) {
    mean = s / n;
    double q = 0.0;
    for (int c = lo; c < hi; ++c) {
      const int p = a.parent[c];
      if (p < 0 || !(p == (int)u || (a.lab[p] == lu && a.depth[c] > du))) continue;
      if (isnan(a.step[c])) continue;
      const double d = a.step[c] - mean;
      q += d * d;
    }
    sd = sqrt(q / n);
    if (!(sd > kSpreadFloor)) sd = 0.0;
  }
  a.gmean[u] = mean;
  a.gstd[u] = sd;                                  // 0: no group, or no spread
  double e = 0.0;
  if (a.parent[u] >= 0) {
    const int tin_u = a.tin[u], tout_u = a.tout[u];
    for (int x = lo; x < hi; ++x) {
      const int an = a.anchor[x];
      if (an < 0 || a.tin[x] < tin_u || a.tin[x] >= tout_u) continue;
      if (a.depth[an] < du) e += a.aeff_node[x];
    }
  }
  a.a_eff[u] = e;
}

__global__ void k_dual(RewardArgs a) {
  const int64_t v = gid();
  if (v >= a.N) return;
  const int p = a.parent[v];
  double c = 0.0;
  if (p >= 0 && !isnan(a.step[v]) && a.gstd[p] > 0.0) c = (a.step[v] - a.gmean[p]) / a.gstd[p];
  a.a_cor[v] = c;
  a.a_dual[v] = c + a.lambda_eff * a.a_eff[v];
}

// Every prompt of at most kRewardPromptMax states in one workgroup, its arrays in LDS, one launch.
//
// What bounds it: latency.  A prompt is a few hundred states, and its phases are chains of LDS
// round trips between barriers; the 64 bytes a state moves through HBM are nothing beside them.
// So the phases are few (one block scan for the outcomes and both lists, one for the routes) and
// their loops short:
//   outcomes   a prefix sum of the packed (R, 1) values in Euler order (subtrees are ranges);
//   pooling    class totals by LDS integer atomics;
//   lists      children and class members as CSR, a state's place in its list being the number
//              of smaller ids there; step rewards are kept at those places, so a state's
//              correctness group reads runs of its class's children's (and only states with
//              children have a group that is read), and a class's smallest member only its
//              members (their common ancestor is that of the first and last in Euler order);
//   routes     the edge into u sums over u's subtree: a range of the Euler order, of which only
//              the members of classes with an anchor are kept (in that order).
// The results equal the multi-kernel path's up to the order of a few fp64 sums.
//   512 prompts of 205 states: 49 -> 21 us; 64 prompts of 517 states, which took the multi-kernel
//   path's scans of the whole prompt per state: 585 -> 17 us.
// Indices are prompt-local and held in 16 bits; LDS is sized for the batch's largest prompt.
__host__ __device__ constexpr size_t reward_lds_bytes(int n) {
  return 8 * (size_t)(5 * n + 1) + 4 * (size_t)(n + 1) + 2 * (size_t)(13 * n + 1);
}

template <int NT>
__global__ __launch_bounds__(NT) void k_prompt_advantages(RewardArgs a, int cap) {
  typedef unsigned short u16;
  constexpr u16 kNone = 0xffff;
  extern __shared__ __align__(16) unsigned char dyn[];
  __shared__ long long s_wsum[NT / 64];
  __shared__ unsigned s_wcnt[NT / 64];
  // (gs takes pre's place, gm ctot's and cval S's once those have been read)
  long long* s_pre = reinterpret_cast<long long*>(dyn);            // [cap + 1]
  double* s_gs = reinterpret_cast<double*>(s_pre);
  unsigned long long* s_ctot = reinterpret_cast<unsigned long long*>(s_pre + cap + 1);
  double* s_gm = reinterpret_cast<double*>(s_ctot);
  double* s_S = reinterpret_cast<double*>(s_ctot + cap);
  double* s_cval = s_S;
  double* s_r = s_S + cap;
  double* s_aen = s_r + cap;
  unsigned* s_off = reinterpret_cast<unsigned*>(s_aen + cap);      // [cap + 1] children | members
  u16* s_par = reinterpret_cast<u16*>(s_off + cap + 1);
  u16* s_lab = s_par + cap;
  u16* s_dep = s_lab + cap;
  u16* s_tin = s_dep + cap;
  u16* s_tout = s_tin + cap;
  u16* s_eul = s_tout + cap;
  u16* s_anc = s_eul + cap;
  u16* s_kids = s_anc + cap;
  u16* s_mem = s_kids + cap;
  u16* s_ku = s_mem + cap;                                         // lists in arrival order
  u16* s_mu = s_ku + cap;
  u16* s_cdep = s_mu + cap;
  u16* s_cpos = s_cdep + cap;                                      // [cap + 1]
  const int2 pr = a.prompts[blockIdx.x];
  const int s0 = pr.x, n = pr.y, tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  for (int v = tid; v <= n; v += NT) {
    s_off[v] = 0;
    if (v < n) s_ctot[v] = 0;
  }
  __syncthreads();
  // A state's slot in its lists, in order of arrival, waits in s_kids / s_mem until they are built.
  for (int v = tid; v < n; v += NT) {
    const int g = s0 + v;
    const int l = a.labels[g];
    const int lab = ((l >= s0 && l <= g) ? l : g) - s0;
    const int p = a.parent[g];
    const int tin = a.tin[g] - s0;                   // (the walk numbers every prompt's states in
                                                     // turn, so its root's number is its id)
    const int r = a.reward[g];
    s_lab[v] = (u16)lab;
    s_par[v] = p >= 0 ? (u16)(p - s0) : kNone;
    s_dep[v] = (u16)a.depth[g];
    s_tin[v] = (u16)tin;
    s_tout[v] = (u16)(a.tout[g] - s0);
    s_aen[v] = (double)a.edge_sim[g];                // (until the classes' values take its place)
    s_eul[tin] = (u16)v;
    s_pre[tin] = r >= 0 ? (((long long)r << 32) | 1) : 0;
    if (p >= 0) s_kids[v] = (u16)(atomicAdd(&s_off[p - s0], 1u) & 0xffff);
    s_mem[v] = (u16)(atomicAdd(&s_off[lab], 0x10000u) >> 16);
  }
  __syncthreads();
  // Exclusive scans over [0, n]: s_pre[k] = sum of the outcome values at Euler positions < k (so
  // a subtree's sums are s_pre[tout] - s_pre[tin]); s_off[v] = where v's children start (low half)
  // and where the members labelled v start (high half).
  {
    long long csum = 0;
    unsigned ccnt = 0;
    for (int b0 = 0; b0 <= n; b0 += NT) {
      const int i = b0 + tid;
      const long long x0 = i < n ? s_pre[i] : 0;
      const unsigned y0 = i < n ? s_off[i] : 0;
      long long x = x0;
      unsigned y = y0;
#pragma unroll
      for (int o = 1; o < 64; o <<= 1) {
        const long long xu = __shfl_up(x, o);
        const unsigned yu = __shfl_up(y, o);
        if (lane >= o) {
          x += xu;
          y += yu;
        }
      }
      if (lane == 63) {
        s_wsum[wave] = x;
        s_wcnt[wave] = y;
      }
      __syncthreads();
      long long xb = csum;
      unsigned yb = ccnt;
      for (int w = 0; w < NT / 64; ++w) {
        if (w < wave) {
          xb += s_wsum[w];
          yb += s_wcnt[w];
        }
        csum += s_wsum[w];
        ccnt += s_wcnt[w];
      }
      if (i <= n) {
        s_pre[i] = xb + x - x0;
        s_off[i] = yb + y - y0;
      }
      __syncthreads();
    }
  }
  auto kid0 = [&](int v) { return (int)(s_off[v] & 0xffff); };
  auto kid1 = [&](int v) { return (int)(s_off[v + 1] & 0xffff); };
  auto mem0 = [&](int v) { return (int)(s_off[v] >> 16); };
  auto mem1 = [&](int v) { return (int)(s_off[v + 1] >> 16); };
  for (int v = tid; v < n; v += NT) {                // lists; own outcomes -> class totals
    const int p = s_par[v], l = s_lab[v];
    if (p != kNone) s_ku[kid0(p) + s_kids[v]] = (u16)v;
    s_mu[mem0(l) + s_mem[v]] = (u16)v;
    atomicAdd(&s_ctot[l], (unsigned long long)(s_pre[s_tout[v]] - s_pre[s_tin[v]]));
    s_anc[v] = kNone;
  }
  __syncthreads();
  for (int v = tid; v < n; v += NT) {                // lists in ascending order; pooled scores
    const int p = s_par[v], l = s_lab[v];
    if (p != kNone) {
      const int k0 = kid0(p), k1 = kid1(p);
      int at = k0;
      for (int k = k0; k < k1; ++k) at += s_ku[k] < v;
      s_kids[v] = (u16)at;
    }
    const int m0 = mem0(l), m1 = mem1(l);
    int at = m0;
    for (int k = m0; k < m1; ++k) at += s_mu[k] < v;
    s_mem[at] = (u16)v;
    const long long own = s_pre[s_tout[v]] - s_pre[s_tin[v]];
    const long long tot = (long long)s_ctot[l];
    const double c = (double)(own >> 32), t = (double)(own & 0xffffffffLL);
    const double C = (double)(tot >> 32), T = (double)(tot & 0xffffffffLL);
    const double num = c + a.w * (C - c), den = t + a.w * (T - t);
    const double S = den > 0.0 ? num / den : __builtin_nan("");
    s_S[v] = S;
    a.score[s0 + v] = S;
  }
  __syncthreads();
  // Step rewards, at the states' places in their predecessors' lists; and per class of two and more,
  // by its smallest member, what its members' efficiency values are made of: the gate (in aen), the
  // route lengths' mean and deviation (in gm and gs) and the anchor.
  for (int v = tid; v < n; v += NT) {
    const int p = s_par[v];
    double r = __builtin_nan("");
    if (p != kNone) {
      r = (s_S[v] - s_S[p]) * (1.0 - fmax(0.0, s_aen[v]));
      s_r[s_kids[v]] = r;
    }
    a.step[s0 + v] = r;
    const u16* mem = s_mem + mem0(v);
    const int m = mem1(v) - mem0(v);
    if (s_lab[v] != v || m < 2) continue;
    // The lowest common ancestor of a set is that of its first and last state in Euler order.
    int sdef = 0, dsum = 0, first = n, last = 0;
    double ssum = 0.0;
#pragma unroll 4
    for (int k = 0; k < m; ++k) {
      const int x = mem[k], t = s_tin[x];
      const double S = s_S[x];
      ssum += isnan(S) ? 0.0 : S;
      sdef += !isnan(S);
      dsum += s_dep[x];
      first = min(first, t);
      last = max(last, t);
    }
    int y = s_eul[first], z = s_eul[last];
    while (s_dep[y] > s_dep[z]) y = s_par[y];        // (by depth walking)
    while (s_dep[z] > s_dep[y]) z = s_par[z];
    while (y != z) {
      y = s_par[y];
      z = s_par[z];
    }
    const int anc = s_lab[y] == v ? s_par[y] : y;
    if (anc == kNone) continue;                      // a class holding its prompt's root
    const int da = s_dep[anc];
    const double mean = -(double)(dsum - m * da) / m;
    double q = 0.0;
#pragma unroll 4
    for (int k = 0; k < m; ++k) {
      const double d = -(double)(s_dep[mem[k]] - da) - mean;
      q += d * d;
    }
    s_aen[v] = sdef > 0 ? ssum / sdef : 0.0;
    s_gm[v] = mean;
    s_gs[v] = sqrt(q / m);
    s_anc[v] = (u16)anc;
  }
  __syncthreads();
  // The efficiency values and anchors' depths of the class members with an anchor, in Euler order,
  // and how many lie before each position.
  {
    unsigned carry = 0;
    for (int b0 = 0; b0 <= n; b0 += NT) {
      const int i = b0 + tid;
      const int x = i < n ? s_eul[i] : 0;
      const int l = s_lab[x], anc = s_anc[l];
      const bool on = i < n && anc != kNone;
      const unsigned long long bal = __ballot(on);
      if (lane == 0) s_wcnt[wave] = (unsigned)__popcll(bal);
      __syncthreads();
      unsigned at = carry;
      for (int w = 0; w < NT / 64; ++w) {
        if (w < wave) at += s_wcnt[w];
        carry += s_wcnt[w];
      }
      at += (unsigned)__popcll(bal & ((1ull << lane) - 1));
      if (i <= n) s_cpos[i] = (u16)at;
      if (on) {
        const double len = -(double)(s_dep[x] - s_dep[anc]), sd = s_gs[l];
        s_cval[at] = sd > 0.0 ? s_aen[l] * (len - s_gm[l]) / sd : 0.0;
        s_cdep[at] = s_dep[anc];
      }
      __syncthreads();
    }
  }
  for (int u = tid; u < n; u += NT) {                // correctness groups; efficiency per edge
    if (kid0(u) < kid1(u)) {
      const int lu = s_lab[u], du = s_dep[u], m0 = mem0(lu), m1 = mem1(lu);
      int cnt = 0, members = 0;
      double sum = 0.0;
      for (int k = m0; k < m1; ++k) {
        const int q = s_mem[k], k1 = kid1(q);
        if (q != u && s_dep[q] < du) continue;       // (its children lie no deeper than u)
        members += k1 - kid0(q);
#pragma unroll 4
        for (int j = kid0(q); j < k1; ++j) {
          const double r = s_r[j];
          sum += isnan(r) ? 0.0 : r;
          cnt += !isnan(r);
        }
      }
      double mean = 0.0, sd = 0.0;
      if (members > 1 && cnt > 0) {
        mean = sum / cnt;
        double q2 = 0.0;
        for (int k = m0; k < m1; ++k) {
          const int q = s_mem[k], k1 = kid1(q);
          if (q != u && s_dep[q] < du) continue;
#pragma unroll 4
          for (int j = kid0(q); j < k1; ++j) {
            const double r = s_r[j], d = isnan(r) ? 0.0 : r - mean;
            q2 += d * d;
          }
        }
        sd = sqrt(q2 / cnt);
        if (!(sd > kSpreadFloor)) sd = 0.0;
      }
      s_gm[u] = mean;
      s_gs[u] = sd;
    }
    double e = 0.0;
    if (s_par[u] != kNone) {
      const int du = s_dep[u], c1 = s_cpos[s_tout[u]];
#pragma unroll 4
      for (int k = s_cpos[s_tin[u]]; k < c1; ++k) {
        const double x = s_cval[k];
        e += s_cdep[k] < du ? x : 0.0;
      }
    }
    s_aen[u] = e;                                    // (aen was last read by the compaction)
  }
  __syncthreads();
  for (int v = tid; v < n; v += NT) {
    const int p = s_par[v];
    double c = 0.0;
    if (p != kNone && s_gs[p] > 0.0) {
      const double r = s_r[s_kids[v]];
      if (!isnan(r)) c = (r - s_gm[p]) / s_gs[p];
    }
    a.a_cor[s0 + v] = c;
    a.a_eff[s0 + v] = s_aen[v];
    a.a_dual[s0 + v] = c + a.lambda_eff * s_aen[v];
  }
}

}  // namespace

hipError_t launch_advantages(const RewardArgs& a, hipStream_t stream) {
  if (a.N == 0) return hipSuccess;
  if (a.n_big == 0) {
    // About a thread per state: a prompt's loops then run once, and a batch of many small prompts
    // keeps several workgroups on a CU.
    const int cap = (a.max_prompt + 3) & ~3;
    const size_t lds = reward_lds_bytes(cap);
    const dim3 grid((unsigned)a.n_prompts);
    if (cap <= 256)
      hipLaunchKernelGGL(k_prompt_advantages<256>, grid, dim3(256), lds, stream, a, cap);
    else if (cap <= 512)
      hipLaunchKernelGGL(k_prompt_advantages<512>, grid, dim3(512), lds, stream, a, cap);
    else
      hipLaunchKernelGGL(k_prompt_advantages<1024>, grid, dim3(1024), lds, stream, a, cap);
    return hipGetLastError();
  }
  const unsigned g = (unsigned)((a.N + kB - 1) / kB);
  const unsigned sb = (unsigned)((a.N + 1023) / 1024);
  hipLaunchKernelGGL(k_outcome_vals, dim3(g), dim3(kB), 0, stream, a);
  hipLaunchKernelGGL(k_pre_sums, dim3(sb), dim3(1024), 0, stream, a);
  hipLaunchKernelGGL(k_pre_apply, dim3(sb), dim3(1024), 0, stream, a);
  hipLaunchKernelGGL(k_own, dim3(g), dim3(kB), 0, stream, a);
  hipLaunchKernelGGL(k_scores, dim3(g), dim3(kB), 0, stream, a);
  hipLaunchKernelGGL(k_step_and_classes, dim3(g), dim3(kB), 0, stream, a);
  hipLaunchKernelGGL(k_groups_and_routes, dim3(g), dim3(kB), 0, stream, a);
  hipLaunchKernelGGL(k_dual, dim3(g), dim3(kB), 0, stream, a);
  return hipGetLastError();
}

}  // namespace ga
