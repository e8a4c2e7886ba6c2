// Graph-coupled probability design (paper Sec. 4.3-4.4): continuation
// probabilities from the prefix statistics, batched over prompts.
//
//   d_ij = p_i (1 - p_j) + (1 - p_i) p_j                 Eq. (disagreement)
//   a_ij = d_ij, or d_ij (m_i + m_j)^2 / 4               Eq. (edge-proxy)
//   b_i  = (sum_{j != i} sqrt(a_ij))^2 - sum_{j != i} a_ij
//   min  Phi = sum_{i<j} a_ij / (pi_i pi_j) + sum_i b_i / pi_i
//   s.t. sum_i c_i pi_i <= budget,  pi_min <= pi_i <= 1
// which is Eqs. (convex-objective)-(budget) in pi = e^{-x}.
//
// One 64-lane wavefront per prompt, lane i = vertex i, all arithmetic in
// fp64.  With A_i = sum_{j != i} a_ij / pi_j + b_i, the Lagrangian
// Phi + lam (c^T pi - budget) restricted to coordinate i is A_i / pi_i +
// lam c_i pi_i + const, minimised over the box exactly at
//     pi_i = clip( sqrt(A_i / (lam c_i)), pi_min, 1 ).
// For a fixed multiplier lam, cyclic coordinate descent with these exact
// updates converges to the minimiser of the (convex) Lagrangian; the spent
// budget c^T pi(lam) does not increase with lam, so lam is found by a
// safeguarded false-position search (Illinois) in log space between a
// multiplier that puts every vertex at pi_min and one that puts every vertex
// with positive A at 1, each inner solve warm-started from the previous one.
//
// Bound by one serial chain: a sweep is G dependent updates.  No update
// reduces over the wave or divides.  The state is y = 1 / pi, and lane j
// carries b_j + the partners' a_ij y_i in one accumulator: when vertex i gets its new y_i,
// every other lane adds a_ij y_i and lane i starts again from b_i, so at a
// lane's turn the accumulator holds the partners behind it from the previous sweep and
// those before it from this one -- A_j exactly as the sweep needs it, a sum of
// positive terms with nothing subtracted.  The update itself is y = rsqrt(A / (lam c)) from the
// hardware's reciprocal root and one third-order step.  a_ij is formed on the fly from p_j
// and the wave-uniform p_i, beside the chain, so nothing G x G is stored.
// B = 512, G in 2..64, half the full cost: 994 us with a wave reduction, a
// division and a square root per update, 328 us so.
//
// The pointwise comparison design is the same program with a = 0 and
// b_i = p_i (1 - p_i); the uniform design spends the budget with one
// probability.  Vertices whose A is identically zero (no contrast with any
// other vertex) take pi_min.
#include "common.hpp"
#include "launch.hpp"

namespace pair {

namespace {

constexpr int kMaxSweeps = 400;       // inner coordinate-descent sweeps per multiplier
constexpr int kMaxBisect = 200;       // multiplier search steps
constexpr int kDefaultCap = 10000;    // total sweeps of one prompt unless the caller caps them

__device__ __forceinline__ double wave_min_d(double v) {
#pragma unroll
  for (int m = 1; m < kWave; m <<= 1) v = fmin(v, __shfl_xor(v, m, kWave));
  return v;
}

// Edge proxy a_ij seen from lane j (vertex j) for a wave-uniform vertex i.
__device__ __forceinline__ double proxy(double pi_hat, double pj_hat, double mi, double mj,
                                        bool scaled) {
  double d = pi_hat * (1.0 - pj_hat) + (1.0 - pi_hat) * pj_hat;
  if (scaled) d *= 0.25 * (mi + mj) * (mi + mj);
  return d;
}

// 1 / sqrt(t) for t > 0, to rounding: the hardware's estimate (relative error
// below 2^-22) and one step of third order, whose error is 5/16 of the cube.
__device__ __forceinline__ double rsqrt_d(double t) {
  const double y = __builtin_amdgcn_rsq(t);
  const double e = fma(-t * y, y, 1.0);
  return fma(y * e, fma(e, 0.375, 0.5), y);
}

// Median of v over the lanes with `in` set (the mean of the two middle values
// for an even count), the same in every lane; 0 if no lane is set.  Ranks
// are counted per lane, ties broken by lane index.
__device__ double wave_median_d(double v, bool in, int g, int lane) {
  const uint64_t mask = __ballot(in);
  const int n = __popcll(mask);
  if (n == 0) return 0.0;
  int rank = 0;
  for (int j = 0; j < g; ++j) {
    const double vj = readlane_d(v, j);
    if (((mask >> j) & 1ull) && (vj < v || (vj == v && j < lane))) ++rank;
  }
  const int r1 = (n - 1) / 2, r2 = n / 2;
  const double lo = wave_sum_d((in && rank == r1) ? v : 0.0);
  const double hi = wave_sum_d((in && rank == r2) ? v : 0.0);
  return r1 == r2 ? lo : 0.5 * (lo + hi);
}

// EDGES: the program has the edge proxy's terms (the PAIR design, and the residual of
// the uniform one; the pointwise design has none).  SCALED: m_hat is given.
template <bool EDGES, bool SCALED>
__global__ __launch_bounds__(kWave) void alloc_kernel(
    int64_t B, int64_t nv, int32_t gmax, const int64_t* __restrict__ offsets,
    const float* __restrict__ p_hat, const float* __restrict__ c_hat,
    const float* __restrict__ m_hat, const float* __restrict__ budget, float pi_min_f,
    int32_t design, const float* __restrict__ pi_prev, int32_t cap,
    float* __restrict__ pi_out, double* __restrict__ objective, int32_t* __restrict__ iters,
    double* __restrict__ residual, int32_t* d_status) {
  const int64_t b = blockIdx.x;
  const int lane = threadIdx.x;
  int64_t o0, g;
  if (!prompt_bounds(offsets, b, nv, 1, gmax, &o0, &g, d_status, lane == 0)) return;
  const int gi = (int)g;
  const bool vert = lane < gi;
  const double pmin = (double)pi_min_f;
  const double p = vert ? (double)p_hat[o0 + lane] : 0.0;
  const double c = vert ? (double)c_hat[o0 + lane] : 0.0;
  const double m = (vert && SCALED) ? (double)m_hat[o0 + lane] : 0.0;
  const double bud = (double)budget[b];
  const bool bad_in = vert && !(p >= 0.0 && p <= 1.0 && c > 0.0 && c < 1e300 &&
                                (!SCALED || (m >= 0.0 && m < 1e300)));
  if (__ballot(bad_in) != 0ull || !(bud > 0.0) || !(pmin > 0.0 && pmin <= 1.0)) {
    if (lane == 0) raise_status(d_status, PAIR_ST_BUDGET);
    if (vert) pi_out[o0 + lane] = pi_min_f;
    return;
  }
  // a_ij of the proxy for the wave-uniform vertex i, in lane j (meaningless
  // where j = i or j is past the group).
  auto proxy_to = [&](int i) -> double {
    const double m_i = SCALED ? readlane_d(m, i) : 0.0;
    return proxy(readlane_d(p, i), p, m_i, m, SCALED);
  };
  auto edge_to = [&](int i) -> double { return EDGES ? proxy_to(i) : 0.0; };
  // Lane j's sums over its partners: a is symmetric, so no lane needs another's.
  auto vertex_term = [&](double* row) -> double {
    double s1 = 0.0, s2 = 0.0;
    for (int i = 0; i < gi; ++i) {
      const double a = lane != i ? proxy_to(i) : 0.0;
      s1 += sqrt(a);
      s2 += a;
    }
    *row = s2;
    return fmax(s1 * s1 - s2, 0.0);   // rounding: the exact value is >= 0 (Cauchy-Schwarz)
  };

  // Vertex term b_i (pointwise design: p (1 - p)); A_i's range over the box.
  double bv = p * (1.0 - p), arow = 0.0;
  if (EDGES) bv = vertex_term(&arow);
  if (!vert) bv = arow = 0.0;
  // A_i = sum_{j != i} a_ij / x_j + b_i of the program at probabilities x, in
  // lane i.
  auto a_vec = [&](double x) -> double {
    double out = bv;
    const double ix = 1.0 / x;
    for (int i = 0; i < gi; ++i) {
      const double a = lane != i ? edge_to(i) : 0.0;
      out = fma(a, readlane_d(ix, i), out);
    }
    return out;
  };

  const double csum = wave_sum_d(c);
  const double uni = fmin(fmax(bud / csum, pmin), 1.0);   // the uniform design's probability
  double pi = 1.0;
  int it = 0;
  bool failed = false;
  if (csum <= bud) {
    pi = 1.0;
  } else if (bud < pmin * csum * (1.0 - 1e-12)) {
    if (lane == 0) raise_status(d_status, PAIR_ST_BUDGET);
    pi = pmin;
  } else if (bud <= pmin * csum) {
    pi = pmin;
  } else if (design == PAIR_DESIGN_UNIFORM) {
    pi = uni;
  } else {
    // Multiplier bracket: at lam_hi every vertex sits at pi_min; at lam_lo
    // every vertex with A > 0 sits at 1.
    const double a_hi = arow / pmin + bv, a_lo = arow + bv;
    const double lam_hi = 2.0 * wave_max_d(vert ? a_hi / (c * pmin * pmin) : 0.0);
    const double lam_lo =
        0.5 * wave_min_d((vert && a_lo > 0.0) ? a_lo / c : 1e308);
    if (!(lam_hi > 0.0)) {
      pi = pmin;   // no contrast anywhere: the cheapest feasible design
    } else {
      // Root of f(t) = log(c^T pi(e^t)) - log(budget), nonincreasing in t,
      // by Illinois false position on a bracket [tlo, thi] with
      // f(tlo) >= 0 >= f(thi); when the same end is replaced twice in a row,
      // the other end's value is halved.  Each evaluation is an inner
      // coordinate descent at lam = e^t, warm-started from the previous
      // iterate; `inner_ok` records whether the last one converged.  Every
      // sweep counts against the prompt's cap.
      double spent = 0.0;
      bool inner_ok = false;
      const double ymax = 1.0 / pmin;
      double y = 1.0, acc = 0.0;
      // Takes the iterate from pi: the accumulators as a sweep leaves them.
      auto start_from_pi = [&]() {
        y = fmin(fmax(1.0 / pi, 1.0), ymax);
        acc = bv;
        for (int i = 0; i < gi; ++i)
          acc = fma(lane < i ? edge_to(i) : 0.0, readlane_d(y, i), acc);
      };
      auto solve_at = [&](double t) -> double {
        const double inv = 1.0 / (exp(t) * c);
        inner_ok = false;
        for (int sw = 0; sw < kMaxSweeps && it < cap; ++sw) {
          const double y_old = y;
          double a = edge_to(0);
          for (int i = 0; i < gi; ++i) {
            const double a_next = edge_to(i + 1 < gi ? i + 1 : i);
            // A / (lam c) = 0 (no contrast, or underflow) is pi_min; an
            // overflow gives NaN, which the clip turns into y = 1.
            const double q = acc * inv;
            double nw = fmin(fmax(rsqrt_d(q), 1.0), ymax);
            nw = q > 0.0 ? nw : ymax;
            const double y_i = readlane_d(nw, i);
            acc = fma(a, y_i, acc);
            acc = lane == i ? bv : acc;
            y = lane == i ? y_i : y;
            a = a_next;
          }
          ++it;
          // |pi_new - pi_old| / pi_old = |y_old - y| / y
          if (__ballot(vert && !(fabs(y_old - y) <= 1e-13 * y)) == 0ull) {
            inner_ok = true;
            break;
          }
        }
        pi = y >= ymax ? pmin : 1.0 / y;
        spent = wave_sum_d(vert ? c * pi : 0.0);
        return log(spent) - log(bud);
      };
      auto met = [&]() { return fabs(spent - bud) <= 1e-13 * bud; };
      const double tmin = log(fmin(lam_lo, lam_hi * 0.5)), tmax = log(lam_hi);
      double tlo = tmin, thi = tmax, flo = 0.0, fhi = 0.0;
      bool bracketed = false, done = false;
      double t0 = 0.0;
      bool warm = false;
      if (pi_prev != nullptr) {
        // Warm start: the previous probabilities (clipped to the box; NaN
        // reads as pi_min) and the multiplier their KKT conditions imply,
        // the median over interior vertices of A_i / (c_i pi_i^2).
        pi = vert ? fmin(fmax((double)pi_prev[o0 + lane], pmin), 1.0) : 1.0;
        const double A = a_vec(pi);
        start_from_pi();
        const bool interior = vert && pi > pmin * (1.0 + 1e-7) && pi < 1.0 - 1e-7;
        const double lam0 = wave_median_d(interior ? A / (c * pi * pi) : 0.0, interior, gi, lane);
        if (lam0 > 0.0) {
          warm = true;
          t0 = fmin(fmax(log(lam0), tmin), tmax);
        }
      }
      if (warm) {
        // Bracket the root by steps growing fourfold from t0, each solve
        // warm-started from the last.  d f / d t lies in [-1/2, 0] (an
        // interior pi_i moves as lam^(-1/2)), so the root is at least 2 |f0|
        // away and the first step is 4 |f0|.
        const double f0 = solve_at(t0);
        const double step0 = fmax(4.0 * fabs(f0), 1e-12);
        if (met()) {
          done = true;
        } else if (f0 > 0.0) {
          tlo = t0;
          flo = f0;
          for (double step = step0; it < cap; step *= 4.0) {
            const double t = fmin(tlo + step, tmax);
            const double ft = solve_at(t);
            if (met()) {
              done = true;
              break;
            }
            if (ft <= 0.0) {
              thi = t;
              fhi = ft;
              bracketed = true;
              break;
            }
            tlo = t;
            flo = ft;
            if (t >= tmax) break;
          }
        } else {
          thi = t0;
          fhi = f0;
          for (double step = step0; it < cap; step *= 4.0) {
            const double t = fmax(thi - step, tmin);
            const double ft = solve_at(t);
            if (met()) {
              done = true;
              break;
            }
            if (ft > 0.0) {
              tlo = t;
              flo = ft;
              bracketed = true;
              break;
            }
            thi = t;
            fhi = ft;
            if (t <= tmin) {   // every vertex with contrast at 1: the budget does not bind
              done = true;
              break;
            }
          }
        }
      } else {
        pi = 1.0;
        start_from_pi();
        flo = solve_at(tlo);
        if (flo > 0.0 && !met()) {   // otherwise the budget does not bind
          pi = pmin;
          start_from_pi();
          fhi = solve_at(thi);
          bracketed = fhi < 0.0 && !met();
          done = !bracketed;
        } else {
          done = true;
        }
      }
      if (bracketed) {
        int side = 0;
        for (int k = 0; k < kMaxBisect && it < cap; ++k) {
          double t = (tlo * fhi - thi * flo) / (fhi - flo);
          if (!(t > tlo && t < thi)) t = 0.5 * (tlo + thi);
          const double ft = solve_at(t);
          if (met()) {
            done = true;
            break;
          }
          if (ft > 0.0) {
            tlo = t;
            flo = ft;
            if (side == 1) fhi *= 0.5;
            side = 1;
          } else {
            thi = t;
            fhi = ft;
            if (side == -1) flo *= 0.5;
            side = -1;
          }
          if (thi - tlo <= 1e-15) {   // the multiplier is fixed to rounding
            done = true;
            break;
          }
        }
      }
      // Solver failure (App. C): the cap or a search limit reached before the
      // budget was met, or a last inner solve that did not converge.  The
      // prompt then gets the uniform design with the same expected cost.
      failed = !done || !inner_ok || !isfinite(pi);
      failed = __ballot(failed) != 0ull;
      if (failed) {
        pi = uni;
      } else {
        // The last multiplier may leave the budget overspent by a rounding
        // amount: keep the iterate of the feasible side.
        spent = wave_sum_d(vert ? c * pi : 0.0);
        if (spent > bud) pi = fmax(pmin, pi * (bud / spent));
      }
    }
  }
  if (failed && lane == 0) raise_status(d_status, PAIR_ST_SOLVER);

  if (vert) pi_out[o0 + lane] = (float)pi;
  if (objective != nullptr || iters != nullptr || residual != nullptr) {
    // Phi at the returned probabilities (the PAIR proxy for every design).
    double phi = 0.0;
    const double iy = 1.0 / pi;
    for (int i = 0; i < gi; ++i)
      phi = fma(lane > i ? proxy_to(i) : 0.0, readlane_d(iy, i), phi);
    // b of the PAIR proxy (for the pointwise design bv holds its own term).
    double unused;
    const double bp = EDGES ? bv : vertex_term(&unused);
    phi = vert ? (phi + bp) * iy : 0.0;
    phi = wave_sum_d(phi);
    // KKT residual of the design's program at the returned (fp32) probabilities
    // x, with the negative gradient g_i = A_i / x_i^2 and one budget
    // multiplier lam: interior vertices need g_i / c_i = lam, vertices at 1
    // need g_i / c_i >= lam, vertices at pi_min need g_i / c_i <= lam, and a
    // positive lam needs the budget spent.  lam is the median of g_i / c_i
    // over the interior vertices; with none, 0 if the budget is slack, else
    // the largest g_i / c_i at pi_min.  Violations are relative to the largest
    // g_i / c_i, the budget's to the budget.
    double res = 0.0;
    if (residual != nullptr) {
      const double x = vert ? (double)(float)pi : 1.0;
      const double ax = a_vec(x);   // wave reductions: every lane takes part
      const double gc = vert ? ax / (x * x) / c : 0.0;
      const double tol = 1e-7;
      const bool interior = vert && x > pmin * (1.0 + tol) && x < 1.0 - tol;
      const bool top = vert && x >= 1.0 - tol;
      const bool bot = vert && x <= pmin * (1.0 + tol);
      const double spent_x = wave_sum_d(vert ? c * x : 0.0);
      double lam;
      if (__ballot(interior) != 0ull)
        lam = wave_median_d(gc, interior, gi, lane);
      else if (spent_x < bud * (1.0 - 1e-9))
        lam = 0.0;
      else
        lam = fmax(wave_max_d(bot ? gc : 0.0), 0.0);
      const double scale = fmax(wave_max_d(vert ? gc : -1e308), 1e-300);
      double r = 0.0;
      if (interior) r = fabs(gc - lam) / scale;
      if (top) r = fmax(r, fmax(lam - gc, 0.0) / scale);
      if (bot) r = fmax(r, fmax(gc - lam, 0.0) / scale);
      res = wave_max_d(r);
      if (lam > 0.0) res = fmax(res, fabs(spent_x - bud) / bud);
      res = fmax(res, fmax(spent_x - bud, 0.0) / bud);
    }
    if (lane == 0) {
      if (objective != nullptr) objective[b] = phi;
      if (iters != nullptr) iters[b] = failed ? -it : it;
      if (residual != nullptr) residual[b] = res;
    }
  }
}

}  // namespace

int launch_alloc(int64_t B, int64_t nv, int32_t gmax, const int64_t* offsets, const float* p_hat,
                 const float* c_hat, const float* m_hat, const float* budget, float pi_min,
                 int32_t design, const float* pi_prev, int32_t max_sweeps, float* pi,
                 double* objective, int32_t* iters, double* residual, int32_t* d_status,
                 hipStream_t stream) {
  const int32_t cap = max_sweeps > 0 ? max_sweeps : kDefaultCap;
#define PAIR_ALLOC(EDGES_, SCALED_)                                                               \
  hipLaunchKernelGGL((alloc_kernel<EDGES_, SCALED_>), dim3((unsigned)B), dim3(kWave), 0, stream, B, \
                     nv, gmax, offsets, p_hat, c_hat, m_hat, budget, pi_min, design, pi_prev, cap, \
                     pi, objective, iters, residual, d_status)
  const bool edges = design != PAIR_DESIGN_POINTWISE, scaled = m_hat != nullptr;
  if (edges) {
    if (scaled) PAIR_ALLOC(true, true); else PAIR_ALLOC(true, false);
  } else {
    if (scaled) PAIR_ALLOC(false, true); else PAIR_ALLOC(false, false);
  }
#undef PAIR_ALLOC
  return hipGetLastError() == hipSuccess ? PAIR_OK : PAIR_EHIP;
}

}  // namespace pair
