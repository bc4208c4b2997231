// Device side of routing (Sec. 3.3 error predictor; Sec. 3.4 router; inference-procedure
// steps 3-6 without a host round trip), for gfx950.  Compiled with floating-point
// contraction disabled: the router's fp64 operations are those of the host router, in the
// same order, so both give bit-identical routes.
//
//   error_predict_kernel  e(u, c) of the risk score from the probe's coverage and descriptors
//   route_kernel          the greedy latency-constrained solve, the tau step and the grouping,
//                         one workgroup
//   plan_kernel           per family, the work queues of the attention launch (query tiles of
//                         the units routed to the family, one queue per key/value bucket, longest
//                         first; block-sparse units of two heads with the same rows and key/value
//                         head share 64-row items), one workgroup per family and bucket
//
// Greedy on the device.  The host solve repeatedly applies the (unit, candidate)
// substitution of minimum ratio rho = (R(c) - R(cur)) / (t(cur) - t(c)) over strictly cheaper
// candidates, ties to the lowest unit and then the lowest candidate, until the unit-order
// total is within the budget.  A unit's next move depends only on its own current choice, so
// every unit's sequence of moves (its path) is fixed in advance; the solve merges the paths,
// always taking the smallest head.  That merge takes the moves in increasing order of
// (K, unit, position), K being the running maximum of rho along the unit's path: a move whose
// rho is below an earlier move of its unit is taken right after that move.  The kernel builds
// the paths (one lane per candidate), sorts the moves by that key, and finds the first prefix of
// the order after which the total (recomputed in unit order, non-increasing in the prefix
// length) is within the budget.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <string>
#include <vector>

#include "common.h"

namespace rs {

constexpr int kRouteMaxUnits = 2048;
constexpr int kRouteMaxMoves = 4096;
constexpr int kMaxCandR = 16;

// ---- error predictor ---------------------------------------------------------------------
struct EpArgs {
  int nunits, rmax, ncand;
  int fam[kMaxCandR];
  float w[4][4];
  const float *cov, *entropy, *local;
  const int *nsub;
  float *e;
};

__global__ void __launch_bounds__(64) error_predict_kernel(const EpArgs a) {
  const int u = blockIdx.x, lane = threadIdx.x;
  __shared__ double sHL[2];
  if (lane == 0) {
    const int nr = min(a.rmax, a.nsub[u * 3 + 0] + a.nsub[u * 3 + 1] + a.nsub[u * 3 + 2]);
    double h = 0.0, l = 0.0;
    for (int r = 0; r < nr; ++r) {
      h = h + (double)a.entropy[(long long)u * a.rmax + r];
      l = l + (double)a.local[(long long)u * a.rmax + r];
    }
    sHL[0] = nr > 0 ? h / (double)nr : 0.0;
    sHL[1] = nr > 0 ? l / (double)nr : 0.0;
  }
  __syncthreads();
  const int c = lane;
  if (c >= a.ncand) return;
  const int f = a.fam[c];
  float out = 0.f;
  if (f != RS_DENSE) {
    const float *cv = a.cov + ((long long)u * a.ncand + c) * 4;
    double vmax = 0.0, vmin = 0.0;
    int nv = 0;
    for (int s = 0; s < 3; ++s) {
      if (a.nsub[u * 3 + s] <= 0) continue;
      const double x = (double)cv[1 + s];
      if (nv == 0) {
        vmax = x;
        vmin = x;
      } else {
        vmax = vmax < x ? x : vmax;
        vmin = x < vmin ? x : vmin;
      }
      ++nv;
    }
    const double om = 1.0 - (double)cv[0];
    const double uu = nv <= 1 ? 0.0 : vmax - vmin;
    const double x[4] = {om, uu, om * sHL[0], om * (1.0 - sHL[1])};
    double acc = 0.0;
    for (int k = 0; k < 4; ++k) acc = acc + (double)a.w[f][k] * x[k];
    out = (float)acc;
  }
  a.e[(long long)u * a.ncand + c] = out;
}

// ---- router ------------------------------------------------------------------------------
struct RouteArgs {
  int U, C, nbucket, dense_c;
  int fam[kMaxCandR], brank[kMaxCandR];
  const float *cov, *e;
  const int *nsub, *s1, *bucket_edge;
  const double *t_table;
  double t_probe, T, tau, alpha, beta, delta_q;
  int *choice, *group_cand, *group_start, *group_units, *status;
  double *risk, *m_lower, *totals;
};

// Sum of x[0, n) in index order, onto `init` (fp64, LDS): one thread, values read ahead of the adds.
__device__ __forceinline__ double ordered_sum(const double *x, int n, double init) {
  double tot = init;
  int u = 0;
  for (; u + 16 <= n; u += 16) {
    double v[16];
#pragma unroll
    for (int k = 0; k < 16; ++k) v[k] = x[u + k];
#pragma unroll
    for (int k = 0; k < 16; ++k) tot = tot + v[k];
  }
  for (; u < n; ++u) tot = tot + x[u];
  return tot;
}

__device__ __forceinline__ double shfl_xor_f64(double v, int o) {
  const uint64_t b = __builtin_bit_cast(uint64_t, v);
  const uint32_t lo = (uint32_t)__shfl_xor((int)(uint32_t)b, o), hi = (uint32_t)__shfl_xor((int)(uint32_t)(b >> 32), o);
  return __builtin_bit_cast(double, (uint64_t)lo | ((uint64_t)hi << 32));
}
// One workgroup, bound by latency: times, risks, paths and ranks live in LDS (candidate-major, so
// that a thread per unit reads them without bank conflicts), only the moves that exist are sorted,
// with a workgroup barrier only for pairs 128 or more apart (a wave holds 128 consecutive elements),
// and the budget search narrows the range on sums taken in any order and then proves its answer on
// the two unit-order totals around it (the unit-order total is the route's definition; the bisection
// on it is kept for the case that the proof fails).  256 units x 9 candidates: 114 -> 56 us (the
// same steps over global arrays, with thirteen unit-order sums, before).
__global__ void __launch_bounds__(1024) route_kernel(const RouteArgs a) {
  const int U = a.U, C = a.C, W = C - 1;
  const int tid = threadIdx.x, NT = blockDim.x, lane = tid & 63, wave = tid >> 6;
  constexpr int NWV = 1024 / 64;
  __shared__ double sT[kRouteMaxMoves + kRouteMaxUnits];  // [C][U] latency
  __shared__ double sR[kRouteMaxMoves + kRouteMaxUnits];  // [C][U] risk
  __shared__ double sKey[kRouteMaxMoves];  // sort keys; later the per-unit times of a total
  __shared__ int sId[kRouteMaxMoves];
  __shared__ double sTot[2], sPart[3][NWV];
  __shared__ uint16_t sRank[kRouteMaxMoves];  // [U][W] position of each move in the merged order
  __shared__ uint8_t sPath[kRouteMaxMoves];   // [U][W] candidates along each unit's path
  __shared__ uint8_t sPlen[kRouteMaxUnits];   // moves on the unit's path
  __shared__ int sFb, sNvalid, sCnt[NWV][kMaxCandR], sStart[kMaxCandR + 1];
  if (tid == 0) {
    sFb = 0;
    sNvalid = 0;
  }

  // latency, risk and lower mass per (unit, candidate)
  for (int i = tid; i < U * C; i += NT) {
    const int u = i / C, c = i % C;
    const int s1 = a.s1[u];
    int b = a.nbucket - 1;
    for (int k0 = 0; k0 < a.nbucket; k0 += 8) {  // the first bucket whose edge reaches s1, else the last
      int e[8];
#pragma unroll
      for (int x = 0; x < 8; ++x) e[x] = a.bucket_edge[min(k0 + x, a.nbucket - 1)];
      int f = 8;
#pragma unroll
      for (int x = 7; x >= 0; --x) f = e[x] >= s1 ? x : f;
      if (f < 8) {
        b = min(k0 + f, a.nbucket - 1);
        break;
      }
    }
    double R = 0.0, ML = 1.0;
    if (a.fam[c] != RS_DENSE) {
      const float *cv = a.cov + (long long)i * 4;
      const float cm[4] = {cv[0], cv[1], cv[2], cv[3]};
      const int ns[3] = {a.nsub[u * 3], a.nsub[u * 3 + 1], a.nsub[u * 3 + 2]};
      const double e = a.e ? (double)a.e[i] : 0.0;
      const double mh = (double)cm[0];
      double vmax = 0.0, vmin = 0.0;
      int nv = 0;
#pragma unroll
      for (int s = 0; s < 3; ++s) {
        if (ns[s] <= 0) continue;
        const double x = (double)cm[1 + s];
        if (nv == 0) {
          vmax = x;
          vmin = x;
        } else {
          vmax = vmax < x ? x : vmax;
          vmin = x < vmin ? x : vmin;
        }
        ++nv;
      }
      const double uu = nv <= 1 ? 0.0 : vmax - vmin;
      R = (1.0 - mh) + a.alpha * uu + a.beta * e;
      const double lm = mh - a.delta_q;
      ML = 0.0 < lm ? lm : 0.0;
    }
    sT[c * U + u] = a.t_table[(long long)c * a.nbucket + b];
    sR[c * U + u] = R;
    a.risk[i] = R;
    a.m_lower[i] = ML;
  }
  __syncthreads();

  // each unit's path: from dense, repeatedly its best strictly cheaper candidate
  for (int u = tid; u < U; u += NT) {
    int cur = a.dense_c, len = 0;
    for (;;) {
      const double tc = sT[cur * U + u], rc = sR[cur * U + u];
      int bc = -1;
      double br = 0.0;
#pragma unroll 4
      for (int c = 0; c < C; ++c) {
        const double tn = sT[c * U + u];
        const double rho = (sR[c * U + u] - rc) / (tc - tn);
        const bool take = tn < tc && (bc < 0 || rho < br);
        br = take ? rho : br;
        bc = take ? c : bc;
      }
      if (bc < 0) break;
      sPath[u * W + len] = (uint8_t)bc;
      ++len;
      cur = bc;
    }
    sPlen[u] = (uint8_t)len;
    const int base = len > 0 ? atomicAdd(&sNvalid, len) : 0;
    cur = a.dense_c;
    double K = 0.0;
    for (int j = 0; j < len; ++j) {
      const int c = sPath[u * W + j];
      const double rho = (sR[c * U + u] - sR[cur * U + u]) / (sT[cur * U + u] - sT[c * U + u]);
      K = (j == 0 || rho > K) ? rho : K;
      // undefined ratios (NaN coverage) go last: with NaN keys the sort's outcome would depend on the
      // order in which the waves took their places in the list
      sKey[base + j] = K == K ? K : (double)INFINITY;
      sId[base + j] = u * W + j;
      cur = c;
    }
  }
  __syncthreads();
  const int nvalid = sNvalid;
  int Mp = 1;
  while (Mp < nvalid) Mp <<= 1;
  for (int i = nvalid + tid; i < Mp; i += NT) {
    sKey[i] = INFINITY;
    sId[i] = 0x7fffffff;
  }
  __syncthreads();

  // bitonic sort of the moves by (K, unit, position); unused slots sort last.  Pair p of a stage
  // at distance j is (i, i + j), i = 2 j (p / j) + p % j: for j <= 64 a wave's 64 pairs stay
  // within its own 128 elements.
  for (int k = 2; k <= Mp; k <<= 1)
    for (int lj = 31 - __builtin_clz(k >> 1); lj >= 0; --lj) {
      const int j = 1 << lj;
      for (int p = tid; p < (Mp >> 1); p += NT) {
        const int i = ((p >> lj) << (lj + 1)) | (p & (j - 1)), l = i + j;
        const bool up = (i & k) == 0;
        const double ki = sKey[i], kl = sKey[l];
        const int ii = sId[i], il = sId[l];
        const bool gt = ki > kl || (ki == kl && ii > il);
        if (gt == up) {
          sKey[i] = kl;
          sKey[l] = ki;
          sId[i] = il;
          sId[l] = ii;
        }
      }
      // the next stage crosses waves when it, or this one, pairs elements 128 or more apart
      if (j > 64 || (j == 1 && k >= 128)) {
        __syncthreads();
      } else {
        __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
        __builtin_amdgcn_wave_barrier();
        __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
      }
    }
  __syncthreads();
  for (int i = tid; i < Mp; i += NT) {
    const int id = sId[i];
    if (id != 0x7fffffff) sRank[id] = (uint16_t)i;
  }
  __syncthreads();

  // unit u's choice after the first k moves of the merged order, for NK values of k at once (a
  // rank past the path counts as a move never taken; reads stay inside the array)
  auto choice_after = [&](int u, auto &ks, auto &ch) {
    constexpr int NK = sizeof(ks) / sizeof(ks[0]);
    const int len = sPlen[u], o = u * W;
    int cnt[NK];
#pragma unroll
    for (int q = 0; q < NK; ++q) cnt[q] = 0;
    for (int j = 0; j < W; j += 8) {
      int r[8];
#pragma unroll
      for (int x = 0; x < 8; ++x) r[x] = (int)sRank[min(o + j + x, kRouteMaxMoves - 1)];
#pragma unroll
      for (int x = 0; x < 8; ++x)
#pragma unroll
        for (int q = 0; q < NK; ++q) cnt[q] += j + x < len && r[x] < ks[q];
    }
#pragma unroll
    for (int q = 0; q < NK; ++q) ch[q] = cnt[q] == 0 ? a.dense_c : (int)sPath[o + cnt[q] - 1];
  };
  // totals after ks[0], ks[1], ks[2] moves, summed in any order (every thread gets them)
  auto totals_near = [&](const int (&ks)[3], double (&tot)[3]) {
    double v[3] = {0.0, 0.0, 0.0};
    for (int u = tid; u < U; u += NT) {
      int ch[3];
      choice_after(u, ks, ch);
#pragma unroll
      for (int q = 0; q < 3; ++q) v[q] += sT[ch[q] * U + u];
    }
#pragma unroll
    for (int o = 32; o >= 1; o >>= 1)
#pragma unroll
      for (int q = 0; q < 3; ++q) v[q] += shfl_xor_f64(v[q], o);
    __syncthreads();
#pragma unroll
    for (int q = 0; q < 3; ++q)
      if (lane == 0) sPart[q][wave] = v[q];
    __syncthreads();
#pragma unroll
    for (int q = 0; q < 3; ++q) {
      tot[q] = a.t_probe;
      for (int w = 0; w < NWV; ++w) tot[q] += sPart[q][w];
    }
  };
  // unit-order totals after k0 and after k1 moves, into sTot[0] and sTot[1] (two waves in parallel)
  double *sTu = sKey;
  auto totals_after = [&](int k0, int k1) {
    __syncthreads();
    for (int u = tid; u < U; u += NT) {
      const int ks[2] = {k0, k1};
      int ch[2];
      choice_after(u, ks, ch);
      sTu[u] = sT[ch[0] * U + u];
      sTu[kRouteMaxUnits + u] = sT[ch[1] * U + u];
    }
    __syncthreads();
    if (tid == 0) sTot[0] = ordered_sum(sTu, U, a.t_probe);
    if (tid == 64) sTot[1] = ordered_sum(sTu + kRouteMaxUnits, U, a.t_probe);
    __syncthreads();
  };
  int kstar = 0;
  bool infeasible = false;
  // the first k whose total is within the budget, by sums in any order
  int guess = 0, above = nvalid;
  {
    double tn[3];
    const int k3[3] = {0, nvalid / 2, nvalid};
    totals_near(k3, tn);
    if (tn[0] > a.T) {
      guess = nvalid;
      if (nvalid > 0 && tn[2] <= a.T) {
        int lo = tn[1] > a.T ? k3[1] : 0, hi = tn[1] > a.T ? nvalid : max(k3[1], 1);
        while (hi - lo > 1) {  // three probes a step: a quarter of the range is left
          const int d = hi - lo;
          const int kq[3] = {lo + max(d / 4, 1), lo + max(d / 2, 1), lo + max((int)((3LL * d) / 4), 1)};
          totals_near(kq, tn);
          int nlo = lo, nhi = hi;
#pragma unroll
          for (int q = 0; q < 3; ++q) {
            if (tn[q] > a.T) nlo = max(nlo, kq[q]);
            else nhi = min(nhi, kq[q]);
          }
          if (nlo >= nhi) nlo = nhi - 1;  // sums in any order need not be monotone
          lo = nlo;
          hi = nhi;
        }
        guess = hi;
        above = hi - 1;
      }
    }
  }
  totals_after(guess, above);
  // total(k) never grows with k: a k within the budget whose predecessor is not is the first one
  const double tot_g = sTot[0], tot_a = sTot[1];
  if (guess == 0 && tot_g <= a.T) {
    kstar = 0;
  } else if (guess > above && tot_g <= a.T && tot_a > a.T) {
    kstar = guess;
  } else {
    totals_after(0, nvalid);
    const double tot_0 = sTot[0], tot_n = sTot[1];
    if (tot_0 > a.T) {
      if (tot_n > a.T) {
        kstar = nvalid;
        infeasible = true;
      } else {
        int lo = 0, hi = nvalid;  // total(lo) > T >= total(hi)
        while (hi - lo > 1) {
          const int mid = lo + (hi - lo) / 2;
          totals_after(mid, mid);
          const double tm = sTot[0];
          if (tm > a.T) lo = mid;
          else hi = mid;
        }
        kstar = hi;
      }
    }
  }
  __syncthreads();

  // the solve's choice, then expand or fall back: the next larger budget of its family that
  // reaches tau, else the cheapest sparse candidate that does, else dense
  for (int u = tid; u < U; u += NT) {
    const int ks[1] = {kstar};
    int cs[1];
    choice_after(u, ks, cs);
    int ch = cs[0];
    uint32_t reached = 0;  // sparse candidates whose lower mass reaches tau
    const double *ml = a.m_lower + (long long)u * C;
#pragma unroll 4
    for (int c2 = 0; c2 < C; ++c2) reached |= (a.fam[c2] != RS_DENSE && ml[c2] >= a.tau ? 1u : 0u) << c2;
    if (a.fam[ch] != RS_DENSE && !((reached >> ch) & 1u)) {
      int pick = -1;
      double best_t = 0.0;
      for (int c2 = 0; c2 < C && pick < 0; ++c2)  // budgets of a family rise in candidate order
        if (a.fam[c2] == a.fam[ch] && a.brank[c2] > a.brank[ch] && ((reached >> c2) & 1u)) pick = c2;
      if (pick < 0)
        for (int c2 = 0; c2 < C; ++c2) {
          if (!((reached >> c2) & 1u)) continue;
          const double tt = sT[c2 * U + u];
          if (pick < 0 || tt < best_t) {
            best_t = tt;
            pick = c2;
          }
        }
      if (pick < 0) {
        pick = a.dense_c;
        atomicAdd(&sFb, 1);
      }
      ch = pick;
    }
    a.choice[u] = ch;
    sId[u] = ch;                                  // the choice, for the grouping below
    sKey[u] = sT[ch * U + u];                     // its time
    sKey[kRouteMaxUnits + u] = sR[ch * U + u];    // its risk
  }
  // units per candidate: a wave's units by ballot, then over the waves in order
  for (int x = tid; x < NWV * kMaxCandR; x += NT) (&sCnt[0][0])[x] = 0;
  __syncthreads();
  if (tid == 0) sTot[0] = ordered_sum(sKey, U, a.t_probe);
  if (tid == 64) sTot[1] = ordered_sum(sKey + kRouteMaxUnits, U, 0.0);
  // wave w counts units [w P, (w + 1) P), P a multiple of 64
  const int P = ((U + NWV * 64 - 1) / (NWV * 64)) * 64;
  for (int u0 = wave * P; u0 < (wave + 1) * P; u0 += 64) {
    const int ch = u0 + lane < U ? sId[u0 + lane] : -1;
    for (int q = 0; q < C; ++q) {
      const int n = __popcll(__ballot(ch == q));
      if (lane == 0) sCnt[wave][q] += n;
    }
  }
  __syncthreads();
  if (tid == 0) {
    int ng = 0, pos = 0;
    for (int q = 0; q < C; ++q) {
      sStart[q] = pos;
      int n = 0;
      for (int w = 0; w < NWV; ++w) n += sCnt[w][q];
      if (n > 0) {
        a.group_cand[ng] = q;
        a.group_start[ng] = pos;
        ++ng;
      }
      pos += n;
    }
    a.group_start[ng] = pos;
    const double tot = sTot[0];
    a.status[0] = ng;
    a.status[1] = sFb;
    a.status[3] = infeasible ? 1 : 0;
    a.status[2] = (infeasible || tot > a.T) ? 1 : 0;
    a.totals[0] = tot;
    a.totals[1] = sTot[1];
  }
  __syncthreads();
  // group members in ascending unit order
  for (int q = 0; q < C; ++q) {
    int pos = sStart[q];
    for (int w = 0; w < wave; ++w) pos += sCnt[w][q];
    for (int u0 = wave * P; u0 < min(U, (wave + 1) * P); u0 += 64) {
      const uint64_t m = __ballot(u0 + lane < U && sId[u0 + lane] == q);
      if ((m >> lane) & 1ull) a.group_units[pos + __popcll(m & ((1ull << lane) - 1ull))] = u0 + lane;
      pos += __popcll(m);
    }
  }
}

// ---- work lists of the routed attention launches -------------------------------------------
struct PlanArgs {
  int U, C, group;
  int fam[kMaxCandR], cl[kMaxCandR], ca[kMaxCandR], cb[kMaxCandR];
  const rs_unit *units;
  const int *choice;
  DevUnit *dunits;  // [4][U]
  int *order;       // [4][max_items], bucket-major
  int max_items;
  int *qsize, *qoff, *qcount;  // [4][8] each
  int hq, d, n;
  int *items;  // split items (AttnParts::items), or NULL: no item is split
};

// Exclusive prefix sum over the workgroup (1024 threads) in thread order; *tot: the sum.
__device__ __forceinline__ int block_excl_scan(int v, int *sWave, int *tot) {
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  int x = v;
#pragma unroll
  for (int o = 1; o < 64; o <<= 1) {
    const int y = __shfl_up(x, o);
    if (lane >= o) x += y;
  }
  __syncthreads();  // sWave is free
  if (lane == 63) sWave[wave] = x;
  __syncthreads();
  int off = 0, all = 0;
  for (int w = 0; w < 16; ++w) {
    const int t = sWave[w];
    off += w < wave ? t : 0;
    all += t;
  }
  *tot = all;
  return off + x - v;
}

// One workgroup per (family, key/value bucket), each on its own queue: units compacted by scans,
// mates and item ranks searched among the bucket's units only.  Bound by latency; one workgroup
// per family with serial passes over the units took 233 us for 256 units of 128 tiles, this 21 us.
// Queue b of a family starts at the most items that the units of the buckets before it can have
// (whatever their families), so that no workgroup needs another's counts; dunits is indexed by
// the unit itself.
__global__ void __launch_bounds__(1024) plan_kernel(const PlanArgs a) {
  const int f = blockIdx.x >> 3, b = blockIdx.x & 7, tid = threadIdx.x, NT = blockDim.x;
  // units of this family and bucket in ascending order (mates not yet taken out)
  __shared__ int sU[kRouteMaxUnits], sHead[kRouteMaxUnits], sS0[kRouteMaxUnits], sS1[kRouteMaxUnits];
  __shared__ int sMate[kRouteMaxUnits];  // list position of the unit taken along, -2 taken along, -1
  __shared__ int sOff[kRouteMaxUnits];   // first flat item
  // items of a unit: n of them, the j-th starting at row 64 (k0 + (j << sh)); sh = 1 for 128-row
  // query tiles, 0 for the 64-row query blocks of a block-sparse unit with a mate
  // (each split into sp pieces, dense and vertical-slash)
  __shared__ uint32_t sIt[kRouteMaxUnits];  // k0 | n << 13 | sh << 26 | sp << 27
  __shared__ int sPb[kRouteMaxUnits];       // first partial slot of the unit
  __shared__ int sIb[kRouteMaxUnits];       // first entry of its query tiles among the items that may split
  __shared__ int sWave[16];
  const int U = a.U;
  int nl = 0, before = 0, slots = 0, mayb = 0;
  for (int u0 = 0; u0 < U; u0 += NT) {
    const int u = u0 + tid;
    bool mine = false, lost = false;
    int tiles = 0, ps = 0, nt = 0;
    rs_unit un{};
    if (u < U) {
      un = a.units[u];
      const int c = a.choice[u], bu = (un.head / a.group) & 7;
      const bool valid = c >= 0 && c < a.C;
      mine = bu == b && valid && a.fam[c] == f;
      lost = bu == b && !valid && f == RS_DENSE;  // not computed: none of its tiles is a split item
      // query tiles in the buckets before this one, as many times as any family may split them
      nt = ((un.s1 - 1) >> 7) - (un.s0 >> 7) + 1;
      if (a.items) ps = attn_split_slots(a.hq, a.d, a.n, un.s0, un.s1);
      tiles = bu < b ? max(nt, ps) : 0;
    }
    int tot, pb = 0, ib = 0;
    if (a.items) {
      pb = slots + block_excl_scan(ps, sWave, &tot);
      slots += tot;
      ib = mayb + block_excl_scan(ps > 0 ? nt : 0, sWave, &tot);
      mayb += tot;
      if (lost && ps > 0)
        for (int x = 0; x < nt; ++x) a.items[ib + x] = -1;
    }
    const int at = nl + block_excl_scan(mine ? 1 : 0, sWave, &tot);
    if (mine) {
      sU[at] = u;
      sHead[at] = un.head;
      sS0[at] = un.s0;
      sS1[at] = un.s1;
      sMate[at] = -1;
      sPb[at] = pb;
      sIb[at] = ps > 0 ? ib : -1;
    }
    nl += tot;
    block_excl_scan(tiles, sWave, &tot);
    before += tot;
  }
  __syncthreads();
  // block-sparse mates: the first unit of an even head h takes along the first unit of head
  // h + 1 with the same rows when both are routed here and read the same key/value head (and so
  // are in this bucket)
  if (f == RS_BSPARSE) {
    for (int x = tid; x < nl; x += NT) {
      const int h = sHead[x];
      if ((h & 1) || (h + 1) / a.group != h / a.group) continue;
      int v = -1;
      bool first = true;
      for (int y = 0; y < nl; ++y) {
        const int hy = sHead[y];
        if ((hy != h && hy != h + 1) || sS0[y] != sS0[x] || sS1[y] != sS1[x]) continue;
        if (hy == h && y < x) {
          first = false;
          break;
        }
        if (hy == h + 1 && v < 0) v = y;
      }
      if (first && v >= 0) {
        sMate[x] = v;
        sMate[v] = -2;
      }
    }
    __syncthreads();
  }
  int total = 0;
  DevUnit *dunits = a.dunits + (long long)f * U;
  for (int x0 = 0; x0 < nl; x0 += NT) {
    const int x = x0 + tid;
    int n = 0;
    if (x < nl) {
      const int u = sU[x], c = a.choice[u], m = sMate[x];
      const int sh = m >= 0 ? 0 : 1, lg = 6 + sh;  // log2 of an item's rows
      n = m == -2 ? 0 : ((sS1[x] - 1) >> lg) - (sS0[x] >> lg) + 1;
      const SplitRule sp = a.items ? attn_split(a.hq, a.d, a.n, sS0[x], sS1[x], f) : SplitRule{1, 1};
      sIt[x] = (uint32_t)((sS0[x] >> lg) << sh) | ((uint32_t)n << 13) | ((uint32_t)sh << 26) |
               ((uint32_t)sp.nsplit << 27);
      if (a.items && sIb[x] >= 0) {
        const int nt = ((sS1[x] - 1) >> 7) - (sS0[x] >> 7) + 1;
        for (int t = 0; t < nt; ++t) a.items[sIb[x] + t] = sp.nsplit > 1 ? ((f * U + u) << 16) | t : -1;
      }
      n *= sp.nsplit;
      if (n > 0)
        dunits[u] = DevUnit{sHead[x], sS0[x], sS1[x], a.cl[c], a.units[u].slot, f == RS_ASHAPE ? a.ca[c] : 0,
                            f == RS_ASHAPE ? a.cb[c] : 0, m >= 0 ? sHead[m] + 1 : 0,
                            m >= 0 ? a.cl[a.choice[sU[m]]] : 0, sp.nsplit, sp.ptiles, sPb[x]};
    }
    int tot;
    const int off = total + block_excl_scan(n, sWave, &tot);
    if (x < nl) sOff[x] = off;
    total += tot;
  }
  __syncthreads();
  if (tid == 0) {
    a.qsize[f * 8 + b] = total;
    a.qoff[f * 8 + b] = f * a.max_items + before;
    a.qcount[f * 8 + b] = 0;
  }
  int *order = a.order + (long long)f * a.max_items + before;
  for (int i = tid; i < total; i += NT) {
    int lo = 0, hi = nl - 1;  // list position of the unit holding flat item i: the last one with
    while (lo < hi) {         // items that starts at or before i
      const int mid = (lo + hi + 1) >> 1;
      if (sOff[mid] <= i) lo = mid;
      else hi = mid - 1;
    }
    const int spl = (int)(sIt[lo] >> 27), j = i - sOff[lo], t = spl == 1 ? j : j / spl, piece = j - t * spl;
    const int key = (int)(sIt[lo] & 0x1fffu) + (t << ((sIt[lo] >> 26) & 1u));  // first row / 64
    // rank in the bucket: later query rows first, then units ascending, then pieces
    int r = 0;
    for (int x = 0; x < nl; ++x) {
      const uint32_t it = sIt[x];
      const int n = (int)(it >> 13) & 0x1fff, sh = (int)(it >> 26) & 1, sp = (int)(it >> 27);
      const int d = key - (int)(it & 0x1fffu);
      const int below = d < 0 ? 0 : min(n, (d >> sh) + 1);  // items of x starting at or before key
      r += (n - below) * sp;
      r += (x < lo && d >= 0 && (d & sh) == 0 && (d >> sh) < n) ? sp : 0;
    }
    order[r + piece] = ((f * U + sU[lo]) << 16) | (piece << 12) | t;
  }
}

// ---- host launchers ----------------------------------------------------------------------
rs_status error_predict_launch(const rs_probe_out *p, const rs_candidate *grid, int32_t ncand,
                               const rs_error_model *m, float *e, hipStream_t st) {
  EpArgs a{};
  a.nunits = p->nunits;
  a.rmax = p->rmax;
  a.ncand = ncand;
  for (int c = 0; c < ncand; ++c) a.fam[c] = grid[c].fam;
  for (int f = 0; f < 4; ++f)
    for (int k = 0; k < 4; ++k) a.w[f][k] = m->w[f][k];
  a.cov = p->cov;
  a.entropy = p->entropy;
  a.local = p->local;
  a.nsub = p->nsub;
  a.e = e;
  if (p->nunits == 0) return RS_OK;
  hipLaunchKernelGGL(error_predict_kernel, dim3(p->nunits), dim3(64), 0, st, a);
  RS_HIP(hipGetLastError());
  return RS_OK;
}

// The router's scratch lives in LDS; the size a caller's workspace has to have is part of the
// interface (a smaller one is rejected) and stays what it was while the scratch was in memory.
size_t route_dev_ws_bytes(int32_t nunits, int32_t ncand) {
  Arena ar(nullptr, 0);
  ar.take<double>((size_t)nunits * ncand);
  ar.take<int>((size_t)nunits * (ncand > 1 ? ncand - 1 : 1));
  ar.take<int>((size_t)nunits * (ncand > 1 ? ncand - 1 : 1));
  ar.take<int>((size_t)nunits);
  return ar.off + 256;
}

static rs_status check_route_size(int U, int C) {
  if (U > kRouteMaxUnits || U * (C - 1) > kRouteMaxMoves)
    return fail(RS_ERR_UNSUPPORTED, "device routing supports nunits <= 2048 and nunits * (ncand - 1) <= 4096");
  return RS_OK;
}

static rs_status route_run(const rs_route_in *in, const rs_route_cfg *cfg, const rs_route_dev_out *out,
                           const int *fam, const int *brank, int dense_c, hipStream_t st) {
  const int U = in->nunits, C = in->ncand;
  RouteArgs a{};
  a.U = U;
  a.C = C;
  a.nbucket = in->nbucket;
  a.dense_c = dense_c;
  for (int c = 0; c < C; ++c) {
    a.fam[c] = fam[c];
    a.brank[c] = brank[c];
  }
  a.cov = in->cov;
  a.e = in->e;
  a.nsub = in->nsub;
  a.s1 = in->s1;
  a.bucket_edge = in->bucket_edge;
  a.t_table = in->t_table;
  a.t_probe = in->t_probe_us;
  a.T = cfg->T_layer_us;
  a.tau = cfg->tau;
  a.alpha = cfg->alpha;
  a.beta = cfg->beta;
  a.delta_q = cfg->delta_q;
  a.choice = out->choice;
  a.group_cand = out->group_cand;
  a.group_start = out->group_start;
  a.group_units = out->group_units;
  a.status = out->status;
  a.risk = out->risk;
  a.m_lower = out->m_lower;
  a.totals = out->totals;
  hipLaunchKernelGGL(route_kernel, dim3(1), dim3(1024), 0, st, a);
  RS_HIP(hipGetLastError());
  return RS_OK;
}

rs_status route_dev_launch(const rs_route_in *in, const rs_route_cfg *cfg, const rs_route_dev_out *out,
                           const int *fam, const int *brank, int dense_c, void *ws, size_t ws_bytes,
                           hipStream_t st) {
  rs_status s = check_route_size(in->nunits, in->ncand);
  if (s != RS_OK) return s;
  const size_t need = route_dev_ws_bytes(in->nunits, in->ncand);
  if (!ws || ws_bytes < need)
    return fail(RS_ERR_WORKSPACE, "device routing workspace too small: need " + std::to_string(need) + " bytes");
  return route_run(in, cfg, out, fam, brank, dense_c, st);
}

rs_status route_dev_launch_noalloc(const rs_route_in *in, const rs_route_cfg *cfg, const rs_route_dev_out *out,
                                   const int *fam, const int *brank, int dense_c, hipStream_t st) {
  rs_status s = check_route_size(in->nunits, in->ncand);
  if (s != RS_OK) return s;
  return route_run(in, cfg, out, fam, brank, dense_c, st);
}

// Bytes of the work lists for at most `items` items per family.
static size_t routed_list_bytes(int32_t nunits, size_t items) {
  Arena ar(nullptr, 0);
  ar.take<rs_unit>((size_t)nunits);
  ar.take<int>(3 * 32);
  ar.take<DevUnit>(4 * (size_t)nunits);
  ar.take<int>(4 * items);
  return ar.off + 256;  // (rounded down to 256 bytes: at or past the lists' end)
}

// Most items of a family, partial slots of the units and query tiles that may have pieces; split:
// items may be split along the keys.
struct RoutedCounts {
  size_t items = 0, slots = 0, mayb = 0;
};
static RoutedCounts routed_counts(const rs_qkv *qkv, const rs_unit *units, int32_t nunits, bool split) {
  RoutedCounts c;
  for (int i = 0; i < nunits; ++i) {
    const rs_unit &u = units[i];
    const int nt = (u.s1 - 1) / 128 - u.s0 / 128 + 1;
    const int s = split && qkv && qkv->hq > 0 && u.s0 >= 0 && u.s1 > u.s0
                      ? attn_split_slots(qkv->hq, qkv->d, qkv->n, u.s0, u.s1) : 0;
    c.items += (size_t)std::max(nt, s);
    c.slots += (size_t)s;
    if (s > 0) c.mayb += (size_t)nt;
  }
  return c;
}

size_t routed_attn_ws_bytes(const rs_qkv *qkv, const rs_unit *units, int32_t nunits) {
  const RoutedCounts c = routed_counts(qkv, units, nunits, true);
  return routed_list_bytes(nunits, c.items) + attn_parts_bytes(qkv ? qkv->d : 0, c.slots) +
         attn_cvt_bytes(qkv, units, nunits);
}

rs_status routed_attn_launch(const rs_qkv *qkv, float scale, const rs_unit *units, int32_t nunits,
                             const rs_candidate *grid, int32_t ncand, const rs_index_set *idx, const int32_t *choice,
                             void *o, int64_t so_h, int64_t so_t, float *lse, void *ws, size_t ws_bytes,
                             void *const *events, hipStream_t st) {
  if (nunits == 0) return RS_OK;
  if (nunits > kRouteMaxUnits) return fail(RS_ERR_UNSUPPORTED, "routed attention supports nunits <= 2048");
  RoutedCounts cn = routed_counts(qkv, units, nunits, true);
  size_t need = routed_list_bytes(nunits, cn.items);
  // items are split where the workspace holds their partial results
  if (cn.slots > 0 && (!ws || ((uintptr_t)ws & 15) || ws_bytes < need + attn_parts_bytes(qkv->d, cn.slots))) {
    cn = routed_counts(qkv, units, nunits, false);
    need = routed_list_bytes(nunits, cn.items);
  }
  const size_t items = cn.items, slots = cn.slots;
  if (!ws || ws_bytes < need)
    return fail(RS_ERR_WORKSPACE, "routed attention workspace too small: need " + std::to_string(need) + " bytes");
  AttnParts parts{};
  char *at = (char *)ws + need / 256 * 256;  // past the lists' end
  if (slots > 0) parts = attn_parts_at(at, qkv->d, slots);
  at += attn_parts_bytes(qkv->d, slots) / 256 * 256;
  const size_t used = (size_t)(at - (char *)ws);
  const rs_unit_table *tables = qkv->tables;
  rs_qkv conv;
  rs_status sc = attn_cvt_launch(qkv, units, nunits, grid, ncand, at, ws_bytes > used ? ws_bytes - used : 0, &conv, st);
  if (sc != RS_OK) return sc;
  qkv = &conv;
  Arena ar(ws, ws_bytes);
  rs_unit *d_units = ar.take<rs_unit>((size_t)nunits);
  int *d_q = ar.take<int>(3 * 32);
  PlanArgs p{};
  p.U = nunits;
  p.C = ncand;
  p.group = qkv->hq / qkv->hkv;
  bool present[4] = {false, false, false, false};
  int cnt[4] = {0, 0, 0, 0};
  for (int c = 0; c < ncand; ++c) {
    p.fam[c] = grid[c].fam;
    p.cl[c] = cnt[grid[c].fam]++;
    p.ca[c] = grid[c].a;
    p.cb[c] = grid[c].b;
    present[grid[c].fam] = true;
  }
  p.units = d_units;
  p.choice = choice;
  p.dunits = ar.take<DevUnit>(4 * (size_t)nunits);
  p.order = ar.take<int>(4 * items);
  p.max_items = (int)items;
  p.hq = qkv->hq;
  p.d = qkv->d;
  p.n = qkv->n;
  p.items = slots > 0 ? parts.items : nullptr;
  p.qsize = d_q;
  p.qoff = d_q + 32;
  p.qcount = d_q + 64;
  // the unit list: from the caller's unit table, else copied into the workspace (from the
  // caller's array, which the copy reads before hipMemcpyAsync returns)
  if (tables)
    p.units = unit_tab_units(tables);
  else
    RS_HIP(hipMemcpyAsync(d_units, units, (size_t)nunits * sizeof(rs_unit), hipMemcpyHostToDevice, st));
  hipLaunchKernelGGL(plan_kernel, dim3(32), dim3(1024), 0, st, p);
  RS_HIP(hipGetLastError());
  // persistent grids: two workgroups per compute unit (the kernel's occupancy), a multiple of 8
  int dev = 0, ncu = 0;
  RS_HIP(hipGetDevice(&dev));
  RS_HIP(hipDeviceGetAttribute(&ncu, hipDeviceAttributeMultiprocessorCount, dev));
  const int nblocks = std::min(((2 * ncu + 7) / 8) * 8, (((int)items + 7) / 8) * 8);
  const AttnQueues qs{p.qsize, p.qoff, p.qcount};
  if (!events) {  // every family in one launch
    rs_status s = attn_launch_queues(qkv, scale, -1, idx, p.dunits, p.order, qs, nblocks, parts, o, so_h, so_t, lse, st);
    if (s == RS_OK && slots > 0)
      s = attn_merge_launch(qkv, scale, p.dunits, parts, (int)cn.mayb, o, so_h, so_t, lse, st);
    return s;
  }
  // one launch per family, timed apart; dense first: its items are the longest
  const int fam_order[4] = {RS_DENSE, RS_VSLASH, RS_BSPARSE, RS_ASHAPE};
  RS_HIP(hipEventRecord((hipEvent_t)events[0], st));
  for (int k = 0; k < 4; ++k) {
    const int f = fam_order[k];
    if (present[f]) {
      rs_status s = attn_launch_queues(qkv, scale, f, idx, p.dunits, p.order, qs, nblocks, parts, o, so_h, so_t, lse, st);
      if (s != RS_OK) return s;
    }
    if (f == RS_VSLASH && slots > 0) {  // the two families with split items are launched
      rs_status s = attn_merge_launch(qkv, scale, p.dunits, parts, (int)cn.mayb, o, so_h, so_t, lse, st);
      if (s != RS_OK) return s;
    }
    RS_HIP(hipEventRecord((hipEvent_t)events[1 + k], st));
  }
  return RS_OK;
}

}  // namespace rs
