// Conditional Poisson (fixed-size) design: paper App. B "Fixed-size and
// exact-cost designs" (Hajek 1964 rejective sampling): exactly n of the G
// candidates continue, with first-order probabilities prescribed by the
// allocation and joint probabilities that do not factorise and are computed
// exactly from the design.
//
// With odds w, P(S) = prod_{i in S} w_i / e_n(w) over |S| = n, where e_k is
// the elementary symmetric polynomial, and
//     pi_i  = w_i e_{n-1}(w without i) / e_n(w),
//     pi_ij = w_i w_j e_{n-2}(w without i, j) / e_n(w)
//           = (w_j pi_i - w_i pi_j) / (w_j - w_i)          (w_i != w_j).
//
//  cps_fit_kernel   one wavefront per prompt, fp64.  Each iteration builds the
//                   prefix polynomials e_k(w_0..w_{m-1}) and the suffix
//                   polynomials e_k(w_{m+1}..w_{G-1}) for all m (lane k holds
//                   coefficient k; adding a unit is one whole-wave DPP shift
//                   and one multiply-add), and lane i gets the leave-one-out
//                   coefficient e_{n-1}(w without i) as the convolution
//                   sum_k prefix_i[k] suffix_i[n-1-k] (all terms positive);
//                   the log-odds then take a Newton step whose Hessian is
//                   the design covariance pi_ij - pi_i pi_j (solved by
//                   Gauss-Jordan elimination in registers, lane = row), halved until
//                   the concave objective rises, until every pi_i is within
//                   1e-12 of its target (3-8 evaluations where a plain
//                   fixed point w_i <- w_i pi_target_i / pi_i takes
//                   100-500).  The joint block uses the difference formula
//                   when the two odds differ by more than 1e-5 relative and
//                   the direct leave-two-out polynomial otherwise.
//  cps_draw_kernel  lane = replicate.  With E[i][k] = e_k(w_i .. w_{G-1}) (built from
//                   the last unit), each lane walks the units in order and
//                   selects unit i with probability
//                   w_i E[i+1][k-1] / E[i][k], k the units still to select,
//                   comparing the top 32 bits of Philox4x64-10 word (i & 3) at
//                   counter (replicate, prompt, i >> 2, 0) with that
//                   probability times 2^32.  The polynomials and the thresholds use
//                   unfused fp64 operations in a fixed order, so each draw is
//                   a deterministic function of (seed, replicate, prompt, w).
#include "common.hpp"
#include "launch.hpp"

namespace pair {

namespace {

constexpr int kMaxFitIter = 200;   // evaluations of pi(w), rejected steps included

// e_0..e_{KP-1} (only k <= n meaningful) of the units 0..g-1 excluding skip1
// and skip2, the units' odds taken from the wave (lane m holds w_m).
template <int KP>
__device__ __forceinline__ void esp_excl(double w, int g, int n, int skip1, int skip2,
                                         double (&e)[KP]) {
  e[0] = 1.0;
#pragma unroll
  for (int k = 1; k < KP; ++k) e[k] = 0.0;
  for (int m = 0; m < g; ++m) {
    const double wm0 = readlane_d(w, m);
    const double wm = (m == skip1 || m == skip2) ? 0.0 : wm0;
#pragma unroll
    for (int k = KP - 1; k >= 1; --k)
      if (k <= n) e[k] = __dadd_rn(e[k], __dmul_rn(wm, e[k - 1]));
  }
}

// Close pairs of a row of the joint block from which every lane's own polynomial
// is the faster: it costs all lanes g * KP steps whatever the number, a pair by
// the wave g steps of another kind.  Equal at 4.7, 6.7, 9.6 and 14.7 pairs for
// KP = 16, 32, 48, 64 (4.4, 13, 24 and 59 us a row against 0.9, 2.0, 2.5 and
// 4.0 a pair at G = KP, 512 prompts).
constexpr int many_close(int kp) { return kp / 5 + 1; }

// e_k of the units but two, in lane k.
__device__ __forceinline__ double esp_excl_wave(double w, int g, int lane, int skip1, int skip2) {
  double e = lane == 0 ? 1.0 : 0.0;
  for (int m = 0; m < g; ++m) {
    const double wm = (m == skip1 || m == skip2) ? 0.0 : readlane_d(w, m);
    e = __dadd_rn(e, __dmul_rn(wm, dpp_d<0x138>(e)));   // wave_shr:1
  }
  return e;
}

// e[k] for a run-time k, by an unrolled select (keeps e in registers).
template <int KP>
__device__ __forceinline__ double pick(const double (&e)[KP], int k) {
  double v = 0.0;
#pragma unroll
  for (int q = 0; q < KP; ++q) v = q == k ? e[q] : v;
  return v;
}

// Prefix rows Pf[m][k] = e_k(w_0 .. w_{m-1}), m = 0..g, and suffix rows
// Sf[m][k] = e_k(w_{m+1} .. w_{g-1}), m = 0..g-1, written to LDS with row
// stride kS (only k <= n is read).  Lane k carries coefficient k; adding unit m is
// e_k <- e_k + w_m e_{k-1}, where e_{k-1} arrives from lane k - 1 by a
// whole-wave DPP shift (lane 0 receives 0).
constexpr int kS = 65;

template <int KP>
__device__ __forceinline__ void esp_tables(double w, int g, int n, int lane, double* Pf,
                                           double* Sf) {
  // The two serial chains run side by side.
  double pre = lane == 0 ? 1.0 : 0.0, suf = pre;
  Pf[lane] = pre;
  Sf[(g - 1) * kS + lane] = suf;
  for (int m = 0; m < g - 1; ++m) {
    const int u = g - 1 - m;
    const double wp = readlane_d(w, m), ws = readlane_d(w, u);
    pre = __dadd_rn(pre, __dmul_rn(wp, dpp_d<0x138>(pre)));   // wave_shr:1
    suf = __dadd_rn(suf, __dmul_rn(ws, dpp_d<0x138>(suf)));
    Pf[(m + 1) * kS + lane] = pre;
    Sf[(u - 1) * kS + lane] = suf;
  }
  pre = __dadd_rn(pre, __dmul_rn(readlane_d(w, g - 1), dpp_d<0x138>(pre)));
  Pf[g * kS + lane] = pre;
  __syncthreads();
}

// 1 / x to rounding for normal x: the hardware's estimate and a step of third order.
__device__ __forceinline__ double recip_d(double x) {
  const double r = __builtin_amdgcn_rcp(x);
  const double e = fma(-x, r, 1.0);
  return fma(r, fma(e, e, e), r);
}

// Eight steps of the elimination of the Newton system, without pivoting (the
// matrix is symmetric positive definite), on the pivots k0 .. k0 + 7.  Lane i
// owns row i, shifted left by k0, of which W entries are left.  Every other
// row is cleared of the pivot column, rows above included (Gauss-Jordan: the
// lanes run anyway, and no back substitution is left).  The rows and columns
// from the pivot on stay symmetric, so the pivot row is the pivot column (entries
// of odds that agree to 1e-6 but form chains are symmetric to 1e-6 only, which
// moves the Newton direction by as much and not what it converges to): one
// store of it by all lanes, read back as broadcasts, kChunk entries in flight
// while the last ones are used.  One wave, whose LDS accesses keep their order:
// no waits but for the data.  Eight steps are unrolled, so that register indices
// are constants; all 64 took 55 KB of code and the same time.
constexpr int kChunk = 16;
constexpr int kPivots = 8;

template <int KP, int W>
__device__ __forceinline__ void eliminate(int k0, int lane, double (&a)[KP], double& x,
                                          double& inv_piv, double* buf) {
#pragma unroll
  for (int s = 0; s < kPivots; ++s) {
    double* v = buf + (s & 1) * (2 * kWave);   // upper half zero: columns past the wave
    v[lane] = a[s];
    wave_lds_order();
    const double* vk = v + k0;
    const int c0 = (s + 1) & ~1;   // pairs of entries, 16 bytes a load
    const int n = (W - c0 + kChunk - 1) / kChunk;
    double u[2][kChunk];
#pragma unroll
    for (int e = 0; e < kChunk; ++e)
      if (c0 + e < W) u[0][e] = vk[c0 + e];
    __builtin_amdgcn_sched_barrier(0);
    const double inv = recip_d(readlane_d(a[s], k0 + s));
    const double xk = readlane_d(x, k0 + s);
    const bool pivot = lane == k0 + s;
    const double m = pivot ? 0.0 : a[s] * inv;
    inv_piv = pivot ? inv : inv_piv;
    x = fma(-m, xk, x);
#pragma unroll
    for (int c = 0; c < n; ++c) {
#pragma unroll
      for (int e = 0; e < kChunk; ++e) {
        const int j = c0 + (c + 1) * kChunk + e;
        if (j < W) u[(c + 1) & 1][e] = vk[j];
      }
      __builtin_amdgcn_sched_barrier(0);
#pragma unroll
      for (int e = 0; e < kChunk; ++e) {
        const int j = c0 + c * kChunk + e;
        if (j > s && j < W) a[j] = fma(-m, u[c & 1][e], a[j]);
      }
    }
  }
#pragma unroll
  for (int j = 0; j < W; ++j) a[j] = j + kPivots < W ? a[j + kPivots] : 0.0;
}

template <int KP>
__global__ __launch_bounds__(kWave) void cps_fit_kernel(
    int64_t B, int64_t nv, int32_t gmax, const int64_t* __restrict__ offsets,
    const float* __restrict__ pi_target, double* __restrict__ w_out, int32_t* __restrict__ n_out,
    float* __restrict__ pi_joint, int32_t* __restrict__ iters, int32_t* d_status) {
  __shared__ double Pf[(KP + 1) * kS];
  __shared__ __attribute__((aligned(16))) double Sf[KP * kS];
  const int64_t b = blockIdx.x;
  const int lane = threadIdx.x;
  int64_t o0, g64;
  if (!prompt_bounds(offsets, b, nv, 2, gmax, &o0, &g64, d_status, lane == 0)) return;
  const int g = (int)g64;
  const bool unit = lane < g;
  double t = unit ? (double)pi_target[o0 + lane] : 0.0;
  const double sum = wave_sum_d(t);
  const int n = (int)rint(sum);
  bool bad = unit && !(t > 0.0 && t < 1.0);
  bad = __ballot(bad) != 0ull || n < 1 || n >= g || fabs(sum - (double)n) > 1e-4 * (double)n;
  if (!bad) {
    t = unit ? t * ((double)n / sum) : 0.0;
    bad = __ballot(unit && !(t < 1.0)) != 0ull;
  }
  if (bad) {
    if (lane == 0) {
      raise_status(d_status, PAIR_ST_P_RANGE);
      if (n_out != nullptr) n_out[b] = 0;
      if (iters != nullptr) iters[b] = 0;
    }
    if (unit) w_out[o0 + lane] = 0.0;
    return;
  }

  // Newton's method on the log-odds theta (mean zero, so the geometric mean
  // of the odds is 1).  The fitted odds maximise the concave
  //     F(theta) = sum_i t_i theta_i - log e_n(exp(theta)),
  // whose gradient is t - pi(theta) and whose negative Hessian is the
  // design's covariance H_ij = pi_ij - pi_i pi_j (H_ii = pi_i (1 - pi_i)).
  // H 1 = 0 (the odds are defined up to scale), so the step solves
  // (H + 1 1^T / g) d = t - pi, whose solution is orthogonal to 1.  A step
  // is kept when F rises by at least 1e-4 of the predicted amount or the
  // largest relative error falls; otherwise it is halved.
  // Wave reductions and lane reads run in uniform control flow: every lane
  // takes part, and lanes beyond the group contribute 0.
  double th = unit ? log(t / (1.0 - t)) : 0.0;
  const double mean0 = wave_sum_d(th) / (double)g;
  th = unit ? th - mean0 : 0.0;
  double w = 0.0, pi = 0.0, en_last = 1.0;
  double th0 = 0.0, d = 0.0, f0 = 0.0, err0 = 0.0, slope = 0.0, step = 1.0;
  bool have_base = false;
  int it = 0;
  bool converged = false;
  for (; it < kMaxFitIter; ++it) {
    w = unit ? exp(th) : 0.0;
    // pi_i(w) for every unit from the prefix and suffix polynomial tables.
    esp_tables<KP>(w, g, n, lane, Pf, Sf);
    const double en = Pf[g * kS + n];
    en_last = en;
    pi = 0.0;
    if (unit) {
      double e1 = 0.0;   // e_{n-1}(w without i) = sum_k Pf[i][k] Sf[i][n-1-k]
      // eight reads of each table in flight; terms past n add 0
      for (int k = 0; k < n; k += 8) {
        double pk[8], sk[8];
#pragma unroll
        for (int s = 0; s < 8; ++s) {
          const int kk = k + s < n ? k + s : n - 1;
          pk[s] = Pf[lane * kS + kk];
          sk[s] = Sf[lane * kS + (n - 1 - kk)];
        }
#pragma unroll
        for (int s = 0; s < 8; ++s)
          e1 = __dadd_rn(e1, k + s < n ? __dmul_rn(pk[s], sk[s]) : 0.0);
      }
      pi = w * e1 / en;
    }
    const double f = wave_sum_d(unit ? t * th : 0.0) - log(en);
    const double err = wave_max_d(unit ? fabs(pi / t - 1.0) : 0.0);
    __syncthreads();   // every lane has read the tables before the Newton system overwrites them
    if (have_base) {
      const bool ok = isfinite(f) && isfinite(err) &&
                      (f >= f0 + 1e-4 * step * slope || err < err0);
      if (!ok && step > 1e-9) {
        step *= 0.5;
        th = unit ? th0 + step * d : 0.0;
        continue;
      }
    }
    if (err <= 1e-12) {
      converged = true;
      break;
    }
    th0 = th;
    f0 = f;
    err0 = err;
    have_base = true;

    // Column `lane` of H + 1 1^T / g (it is symmetric), first in LDS: in
    // registers the loop over j would be unrolled KP times, twice, past the
    // instruction cache.  Off the diagonal pi_ij comes from the difference
    // formula; where two odds agree to 1e-6 it is numerically unreliable, and
    // those entries share what the row identity
    // sum_{j != i} pi_ij = (n - 1) pi_i leaves (exact for equal odds).
    const double inv_g = 1.0 / (double)g;
    double known = 0.0;
    int nclose = 0;
    for (int j0 = 0; j0 < g; j0 += 4) {
#pragma unroll
      for (int s = 0; s < 4; ++s) {
        const int j = j0 + s;
        const double wj = readlane_d(w, j), pj = readlane_d(pi, j);
        const bool off = unit && j < g && j != lane;
        const bool sep = fabs(wj - w) > 1e-6 * fmax(wj, w);
        // Formed in every lane and then selected: a branch per entry would
        // keep the entries from overlapping.
        double pij = (wj * pi - w * pj) * recip_d(wj - w);
        asm("" : "+v"(pij));
        pij = (off && sep) ? pij : 0.0;
        known += pij;
        nclose += (off && !sep) ? 1 : 0;
        double h = pij - pi * pj + inv_g, hd = pi * (1.0 - pi) + inv_g;
        asm("" : "+v"(h), "+v"(hd));
        h = (off && sep) ? h : 0.0;
        // the identity past the group: whole blocks of pivots are eliminated
        Pf[j * kS + lane] = j != lane ? h : (unit ? hd : 1.0);
      }
    }
    if (__ballot(nclose > 0) != 0ull) {
      const double share = nclose > 0 ? ((double)(n - 1) * pi - known) / (double)nclose : 0.0;
      for (int j = 0; j < g; ++j) {
        const double wj = readlane_d(w, j), pj = readlane_d(pi, j);
        const bool close = unit && j != lane && !(fabs(wj - w) > 1e-6 * fmax(wj, w));
        if (close) Pf[j * kS + lane] = share - pi * pj + inv_g;
      }
    }
    for (int j = (g + 3) & ~3; j < KP; ++j) Pf[j * kS + lane] = j == lane ? 1.0 : 0.0;
    double a[KP];   // a lane reads what it wrote
#pragma unroll
    for (int j = 0; j < KP; ++j) a[j] = Pf[j * kS + lane];
    double x = unit ? t - pi : 0.0, inv_piv = 0.0;
    Sf[kWave + lane] = Sf[3 * kWave + lane] = 0.0;
    int k0 = 0;
    if constexpr (KP > 32)
      for (; k0 < g && k0 < KP - 32; k0 += kPivots) eliminate<KP, KP>(k0, lane, a, x, inv_piv, Sf);
    if constexpr (KP > 16)
      for (; k0 < g && k0 < KP - 16; k0 += kPivots) eliminate<KP, 32>(k0, lane, a, x, inv_piv, Sf);
    for (; k0 < g; k0 += kPivots) eliminate<KP, 16>(k0, lane, a, x, inv_piv, Sf);
    x *= inv_piv;
    d = unit ? x : 0.0;
    slope = wave_sum_d(unit ? (t - pi) * d : 0.0);
    step = 1.0;
    th = unit ? th0 + d : 0.0;
    const double mean = wave_sum_d(th) / (double)g;
    th = unit ? th - mean : 0.0;
    __syncthreads();   // the tables are rebuilt by the next iteration
  }
  if (!converged && lane == 0) raise_status(d_status, PAIR_ST_P_RANGE);
  if (unit) w_out[o0 + lane] = w;
  if (lane == 0) {
    if (n_out != nullptr) n_out[b] = n;
    if (iters != nullptr) iters[b] = converged ? it : -it;
  }

  if (pi_joint != nullptr) {
    // Row j of the joint block at step j: lane i holds pi_ij = pi_ji, so the
    // wave stores a run (a row per lane would touch a line per lane).  It is
    // taken from the last evaluation's pi and
    // e_n(w).  The difference formula loses about eps / gap of relative
    // accuracy, so it is used where the two odds differ by more than 1e-5
    // (error below 1e-8, under the fp32 output's rounding); closer pairs
    // take the leave-two-out polynomial.
    // e_{n-2} of a few pairs is the wave's work, a lane per coefficient (the
    // same operations in the same order); from many_close() pairs in a row on
    // it is every lane's own polynomial.  Always the latter, a batch waited for
    // the one prompt with a close pair: 235 us for 512 prompts of 2..64, where
    // the fits take 115; now 136.  The former up to 32 pairs, 512 prompts with equal
    // targets took 223 us at G = 16 and 2005 at 32, always the latter 71 and 428.
    float* col = pi_joint + b * (int64_t)gmax * gmax + lane;
    for (int j = 0; j < gmax; ++j) {
      const double wj = readlane_d(w, j < g ? j : 0), pj = readlane_d(pi, j < g ? j : 0);
      const bool pair_ij = unit && j < g && j != lane;
      const bool sep = fabs(wj - w) > 1e-5 * fmax(wj, w);
      double diff = (wj * pi - w * pj) * recip_d(wj - w);
      asm("" : "+v"(diff));   // selected, not branched to
      double pij = (pair_ij && sep) ? diff : 0.0;
      pij = (unit && j == lane) ? pi : pij;
      const bool direct = pair_ij && !sep && n >= 2;
      uint64_t close = __ballot(direct);
      if (__popcll(close) >= many_close(KP)) {
        double e2[KP];
        esp_excl<KP>(w, g, n - 2, lane, j, e2);   // w of lane j is excluded too
        if (direct) pij = w * wj * pick<KP>(e2, n - 2) / en_last;
      } else {
        for (; close != 0ull; close &= close - 1ull) {
          const int i = __ffsll((unsigned long long)close) - 1;
          const double e2 = readlane_d(esp_excl_wave(w, g, lane, i, j), n - 2);
          if (lane == i) pij = w * wj * e2 / en_last;
        }
      }
      if (lane < gmax) col[(int64_t)j * gmax] = (float)pij;
    }
  }
}

// The draw of up to kDrawReps replicates of one prompt.  The selection
// probability depends on (unit, units still to select) alone, so wave 0 builds
// its thresholds once for the workgroup's replicates: lane k carries E[i][k] in a register (one
// whole-wave DPP shift per unit), and the division is beside that chain.  A
// replicate then costs one LDS read and one comparison per unit.  The taken units gather in
// a 64-bit mask per lane, and the wave stores its replicates' rows four bytes at a time,
// 16 lanes or fewer to a row, where a byte per lane and unit would touch a
// line per replicate each time.
// B = 512, G in 2..64, R = 256: 58 us with a division per unit and
// replicate, the table built per 64 replicates and byte stores; 29 us so.
constexpr int kDrawReps = 256;

template <int KP>
__global__ __launch_bounds__(kDrawReps) void cps_draw_kernel(
    int64_t B, int64_t nv, int32_t gmax, const int64_t* __restrict__ offsets,
    const double* __restrict__ w, const int32_t* __restrict__ n_in, uint64_t seed, int64_t rep0,
    int64_t R, int64_t nwg, uint8_t* __restrict__ mask, int32_t* __restrict__ edge_count,
    int32_t* d_status) {
  constexpr int S = KP + 1;
  __shared__ double thr[KP * S];   // [i][k]: 2^32 x the probability of taking unit i, k left
  const int64_t b = blockIdx.x / nwg;
  const int64_t chunk = blockIdx.x - b * nwg;
  const int tid = threadIdx.x;
  const int lane = tid & (kWave - 1);
  int64_t o0, g64;
  if (!prompt_bounds(offsets, b, nv, 1, gmax, &o0, &g64, d_status, chunk == 0 && tid == 0))
    return;
  const int g = (int)g64;
  const int n = n_in[b];
  // Every wave reads the odds: the decision to leave is the whole workgroup's.
  const double wv = lane < g ? w[o0 + lane] : 1.0;
  if (n < 0 || n > g || __ballot(!(wv > 0.0 && wv < 1e300)) != 0ull) {
    if (chunk == 0 && tid == 0) raise_status(d_status, PAIR_ST_P_RANGE);
    return;
  }
  const bool all_or_none = n == 0 || n == g;   // no randomness: the table is not needed
  if (!all_or_none) {
    if (tid < kWave) {
      double col = lane == 0 ? 1.0 : 0.0;   // E[i + 1][lane]
      for (int i = g - 1; i >= 0; --i) {
        const double num = __dmul_rn(readlane_d(wv, i), dpp_d<0x138>(col));   // wave_shr:1
        col = __dadd_rn(col, num);
        if (lane >= 1 && lane <= n)
          thr[i * S + lane] = __dmul_rn(__ddiv_rn(num, col), 4294967296.0);
        if (lane == 0) thr[i * S] = 0.0;   // none left: never taken
      }
    }
    __syncthreads();
  }

  const int64_t r0 = chunk * blockDim.x + (tid - lane);   // the wave's first replicate
  if (r0 >= R) return;
  const int nr = (int)(R - r0 < kWave ? R - r0 : kWave);
  uint64_t bits = n == g ? ~0ull : 0ull;
  if (!all_or_none) {
    const PhiloxRep pr = philox_rep((uint64_t)(rep0 + r0 + lane));
    int k = n;
    for (int i = 0; i < g; i += 4) {
      const Philox4x64 x = philox_quad(pr, (uint64_t)b, (uint64_t)(i >> 2), seed);
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        if (i + e < g) {
          const bool take = (double)(x.w[e] >> 32) < thr[(i + e) * S + k];
          bits |= (uint64_t)take << (i + e);
          k -= take ? 1 : 0;
        }
      }
    }
  }
  if (edge_count != nullptr && lane < nr) edge_count[(r0 + lane) * B + b] = n * (n - 1) / 2;
  // Row r of the mask: nq lanes of four units each, 64 / nq rows at a time.
  const int nq = (g + 3) >> 2;
  const int per = kWave / nq;
  const int row = lane / nq, q = lane - row * nq;
  const int units = g - 4 * q < 4 ? g - 4 * q : 4;
  uint8_t* m = mask + r0 * nv + o0 + 4 * q;
  for (int base = 0; base < nr; base += per) {
    const int r = base + row;
    const uint32_t lo = (uint32_t)__shfl((int)(uint32_t)bits, r & (kWave - 1), kWave);
    const uint32_t hi = (uint32_t)__shfl((int)(uint32_t)(bits >> 32), r & (kWave - 1), kWave);
    if (row >= per || r >= nr) continue;
    const uint32_t v = ((q < 8 ? lo : hi) >> (4 * (q & 7))) & 0xfu;
    const uint32_t bytes = (v & 1u) | (v & 2u) << 7 | (v & 4u) << 14 | (v & 8u) << 21;
    uint8_t* dst = m + (int64_t)r * nv;
    if (units == 4) {
      __builtin_memcpy(dst, &bytes, 4);
    } else {
      for (int e = 0; e < units; ++e) dst[e] = (uint8_t)(bytes >> (8 * e));
    }
  }
}

}  // namespace

int launch_cps_fit(int64_t B, int64_t nv, int32_t gmax, const int64_t* offsets,
                   const float* pi_target, double* w, int32_t* n_out, float* pi_joint,
                   int32_t* iters, int32_t* d_status, hipStream_t stream) {
  const int ks = (gmax + 15) / 16;
#define PAIR_CPS_FIT(KP_)                                                                        \
  hipLaunchKernelGGL(cps_fit_kernel<KP_>, dim3((unsigned)B), dim3(kWave), 0, stream, B, nv, gmax, \
                     offsets, pi_target, w, n_out, pi_joint, iters, d_status)
  switch (ks) {
    case 1: PAIR_CPS_FIT(16); break;
    case 2: PAIR_CPS_FIT(32); break;
    case 3: PAIR_CPS_FIT(48); break;
    default: PAIR_CPS_FIT(64); break;
  }
#undef PAIR_CPS_FIT
  return hipGetLastError() == hipSuccess ? PAIR_OK : PAIR_EHIP;
}

int launch_cps_draw(int64_t B, int64_t nv, int32_t gmax, const int64_t* offsets, const double* w,
                    const int32_t* n, uint64_t seed, int64_t rep0, int64_t R, uint8_t* mask,
                    int32_t* edge_count, int32_t* d_status, hipStream_t stream) {
  const int ks = (gmax + 15) / 16;
  // The range of a call is that of a workgroup per 64 replicates.
  if ((R + kWave - 1) / kWave > 0x7fffffffLL / B) return PAIR_ERANGE;
  // Replicates per workgroup: whole waves, no more of them than R needs.
  const int64_t reps = R < kDrawReps ? (R + kWave - 1) / kWave * kWave : kDrawReps;
  const int64_t nwg = (R + reps - 1) / reps;
  const int64_t grid = B * nwg;
#define PAIR_CPS_DRAW(KP_)                                                                     \
  hipLaunchKernelGGL(cps_draw_kernel<KP_>, dim3((unsigned)grid), dim3((unsigned)reps), 0, stream, B, nv, \
                     gmax, offsets, w, n, seed, rep0, R, nwg, mask, edge_count, d_status)
  switch (ks) {
    case 1: PAIR_CPS_DRAW(16); break;
    case 2: PAIR_CPS_DRAW(32); break;
    case 3: PAIR_CPS_DRAW(48); break;
    default: PAIR_CPS_DRAW(64); break;
  }
#undef PAIR_CPS_DRAW
  return hipGetLastError() == hipSuccess ? PAIR_OK : PAIR_EHIP;
}

}  // namespace pair
