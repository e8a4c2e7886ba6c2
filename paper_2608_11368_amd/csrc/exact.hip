// Exact design audit (paper Prop. 1; App. A "Design covariance"): the design
// bias and MSE of an estimator that is linear in the edge indicators, with no
// replicate draws.
//
// Such an estimator is g^ = (1/M) sum_e I_e v_e with edge vectors
//     v_ij = A_ij s_i + C_ij s_j,  A_ij = 1/2 (r_i - r_j) w_i,
//                                  C_ij = -1/2 (r_i - r_j) w_j
// (w from the edge-weight rule and the logged rho).  Under independent
// Bernoulli(p_i) vertices,
//     E g^ - t = sum_i beta_i s_i,
//         beta_i = (1/M) sum_{j != i} (p_i p_j A_ij - 1/2 (r_i - r_j)),
//     tr Cov g^ = (1/M^2) [ sum_{i<j} rho (1 - rho) <v_ij, v_ij>
//                 + sum_i sum_{j != k; j, k != i} p_i p_j p_k (1 - p_i) <v_ij, v_ik> ],
// and every inner product is a combination of entries of the Gram matrix
// K = S_b S_b^T.  So the audit is one G x G x D contraction per prompt on the
// matrix cores plus O(G^3) fp64 work:
//
//  1. gram_kernel    workgroup = (prompt, column slice): the slice's partial
//                    Gram matrix (gram.hpp), bound by HBM.
//  2. exact_final_kernel  workgroup per prompt: K in fp64 (slices summed in
//                    order), the rule's coefficients, beta^T K beta and the
//                    covariance trace with a fixed-order reduction.  The
//                    shared-vertex term of vertex i is
//                        | sum_j p_j v_ij |^2 - sum_j p_j^2 |v_ij|^2,
//                    and sum_j p_j v_ij = sum_j X_ij s_j, so all of them are
//                    one G x G x G product X K in place of a sum over ordered
//                    triples with four Gram entries each.
#include "common.hpp"
#include "gram.hpp"
#include "launch.hpp"

namespace pair {

namespace {

typedef double f64x4_t __attribute__((ext_vector_type(4)));

__host__ __device__ inline int64_t ceil_div(int64_t a, int64_t b) { return (a + b - 1) / b; }

struct ExactLayout {
  int ks, kp;
  int64_t nsl;     // column slices per prompt
  int64_t slice;   // columns per slice (whole rounds of a workgroup's waves)
  bool wide;       // slice partials in fp64
  size_t total;
};

ExactLayout exact_layout(int64_t B, int32_t gmax, int64_t D) {
  ExactLayout L;
  L.ks = (gmax + 15) / 16;
  L.kp = 16 * L.ks;
  // Slices of 4096 columns, 8192 for groups of at most 16, while 1024
  // workgroups remain (at B = 128, G in 2..64, D = 65536 their partials take the
  // two kernels 130 us with 2048 columns and 121 us with 4096), else 2048; at
  // most about 8192 workgroups over the batch.
  const int64_t round = kGramRoundCols;
  const int64_t longer = L.ks == 1 ? 4 : 2;
  int64_t nsl = ceil_div(D, longer * round);
  if (B * nsl < 1024) {
    int64_t more = ceil_div(1024, B);
    if (more > ceil_div(D, round)) more = ceil_div(D, round);
    // One workgroup adds a prompt's partials, 20 KB per slice of 64 rows: beyond
    // 64 slices that takes longer than the Gram itself.
    if (L.ks > 2 && more > 64) more = 64;
    if (more > nsl) nsl = more;
  }
  if (nsl > ceil_div(8192, B)) nsl = ceil_div(8192, B);
  L.slice = ceil_div(ceil_div(D, nsl), round) * round;
  L.nsl = ceil_div(D, L.slice);
  // The size callers are asked for also covers slices of 512 columns, about
  // 8192 of them over the batch, with whole KP x KP partials, as earlier
  // buffers do.
  int64_t old = ceil_div(8192, B);
  if (old > ceil_div(D, 512)) old = ceil_div(D, 512);
  old = ceil_div(D, ceil_div(ceil_div(D, old), 512) * 512);
  // fp64 partials where that size holds them, which is all but rows of fewer than
  // 1024 columns and batches of thousands of prompts; else fp32, a rounding of
  // 2^-25 per slice.
  const int64_t now = L.nsl * gram_tiles(L.ks) * 256;
  L.wide = 2 * now <= old * L.kp * L.kp;
  L.total = (size_t)B * (size_t)(old * L.kp * L.kp > now ? old * L.kp * L.kp : now) * sizeof(float);
  return L;
}

template <int KS, class Part>
__global__ __launch_bounds__(kGramThreads, gram_residency(KS)) void gram_kernel(
    int64_t nv, int32_t gmax, const int64_t* __restrict__ offsets, int64_t D,
    const uint16_t* __restrict__ scores, int64_t ld, int64_t nsl, int64_t slice,
    Part* __restrict__ part) {
  __shared__ __align__(16) uint16_t stage[gram_lds_elems(KS)];
  const int64_t b = blockIdx.x / nsl;
  const int64_t sl = blockIdx.x - b * nsl;
  int64_t o0, g;
  if (!prompt_bounds(offsets, b, nv, 2, gmax, &o0, &g, nullptr, false)) return;
  const int64_t c_lo = sl * slice;
  const int64_t c_hi = c_lo + slice < D ? c_lo + slice : D;
  gram_slice_of<KS>(scores + o0 * ld, ld, (int)g, c_lo, c_hi, stage, nullptr, false,
                    part + (b * nsl + sl) * (gram_tiles(KS) * 256), nullptr, nullptr,
                    [](int, int) {});
}

template <int T>
__device__ __forceinline__ double block_sum(double v, double* sh) {
  const int tid = threadIdx.x, lane = tid & (kWave - 1), wave = tid / kWave;
#pragma unroll
  for (int m = 1; m < kWave; m <<= 1) v += __shfl_xor(v, m, kWave);
  __syncthreads();
  if (lane == 0) sh[wave] = v;
  __syncthreads();
  double t = 0.0;
  for (int w = 0; w < T / kWave; ++w) t += sh[w];
  return t;
}

// T threads: 1024, or 256 for groups of at most 16 and few slices (4 prompts of 8 at
// D = 4096: 5.9 us with 1024, 4.6 us with 256; one prompt of 16 at D = 2^20, 512 slices:
// 62 us with 256 threads adding them, 20 us with all).
constexpr int64_t kFewSlices = 16;

template <int KS, class Part, int T>
__global__ __launch_bounds__(T) void exact_final_kernel(
    int64_t B, int64_t nv, int32_t gmax, const int64_t* __restrict__ offsets,
    const float* __restrict__ rewards, const float* __restrict__ p,
    const float* __restrict__ pi_w, int32_t rule, float wmax, int64_t nsl,
    const Part* __restrict__ part, double* __restrict__ mse, double* __restrict__ bias_norm,
    double* __restrict__ gram, int32_t* d_status) {
  constexpr int KP = 16 * KS;
  constexpr int kTiles = gram_tiles(KS);
  constexpr int kRow = KP + 1;   // row stride in LDS: column walks spread over the banks
  constexpr int kGroups = T / 256;
  constexpr int kOwn = (kTiles + kGroups - 1) / kGroups;
  constexpr int kSplit = kTiles == 1 ? kGroups : 1;   // groups that share a tile's slices
  constexpr int kFlight = kOwn == 1 ? 16 : 8;         // slices in flight
  __shared__ double K[KP * kRow];
  __shared__ double Ac[KP * kRow];   // A_ij: coefficient of s_i in v_ij; C_ij = A_ji
  __shared__ double X[KP * kRow];
  __shared__ double beta[KP], pd[KP], rd[KP];
  __shared__ double sh[T / kWave];
  __shared__ double split[kSplit > 1 ? kSplit - 1 : 1][256];
  const int64_t b = blockIdx.x;
  int64_t o0, g;
  if (!prompt_bounds(offsets, b, nv, 2, gmax, &o0, &g, d_status, threadIdx.x == 0)) return;
  const int tid = threadIdx.x;
  const int gi = (int)g;

  if (tid < KP) {
    pd[tid] = tid < gi ? (double)p[o0 + tid] : 1.0;
    rd[tid] = tid < gi ? (double)rewards[o0 + tid] : 0.0;
    if (tid < gi && !p_in_range(p[o0 + tid])) raise_status(d_status, PAIR_ST_P_RANGE);
  }
  bool nonfinite = false;
  // Slice partials added in slice order; thread e of a group of 256 holds
  // entry e of the group's tiles, kFlight slices of all of them in flight (one
  // tile after the other took 12 us longer at 64 rows and 32 slices).  A single
  // tile's slices are shared by the groups.
  const int e = tid & 255;
  double sum[kOwn];
#pragma unroll
  for (int u = 0; u < kOwn; ++u) sum[u] = 0.0;
  const Part* src = part + b * nsl * (kTiles * 256) + e;
  // Loads past the last slice or tile repeat it (a guarded load would wait for
  // its turn) and are not added.
  const int team = __builtin_amdgcn_readfirstlane(tid / 256);
  const int64_t s_lo = kSplit > 1 ? nsl * team / kSplit : 0;
  const int64_t s_hi = kSplit > 1 ? nsl * (team + 1) / kSplit : nsl;
  for (int64_t s0 = s_lo; s0 < s_hi; s0 += kFlight) {
    Part v[kOwn][kFlight];
#pragma unroll
    for (int u = 0; u < kOwn; ++u) {
      int t = kSplit > 1 ? 0 : team + u * kGroups;
      t = t < kTiles ? t : kTiles - 1;
#pragma unroll
      for (int q = 0; q < kFlight; ++q) {
        const int64_t sl = s0 + q < s_hi ? s0 + q : s_hi - 1;
        v[u][q] = src[(sl * kTiles + t) * 256];
      }
    }
#pragma unroll
    for (int u = 0; u < kOwn; ++u)
#pragma unroll
      for (int q = 0; q < kFlight; ++q) sum[u] += s0 + q < s_hi ? (double)v[u][q] : 0.0;
  }
  if (kSplit > 1) {
    if (team > 0) split[team - 1][e] = sum[0];
    __syncthreads();
    if (team == 0)
#pragma unroll
      for (int q = 1; q < kSplit; ++q) sum[0] += split[q - 1][e];
  }
#pragma unroll
  for (int u = 0; u < kOwn; ++u) {
    const int t = team + u * kGroups;
    if (t >= kTiles) continue;
    int ta = 0, tc = 0;
#pragma unroll
    for (int x = 0; x < KS; ++x)
#pragma unroll
      for (int y = x; y < KS; ++y)
        if (gram_tile(KS, x, y) == t) {
          ta = x;
          tc = y;
        }
    const int i = 16 * ta + 4 * (e >> 6) + (e & 3), j = 16 * tc + ((e >> 2) & 15);
    double k = 0.0;
    if (i < gi && j < gi) {   // tiles past the group's blocks were not written
      k = sum[u];
      if (!isfinite(k)) nonfinite = true;
      if (gram != nullptr) {
        gram[(b * gmax + i) * (int64_t)gmax + j] = k;
        if (ta != tc) gram[(b * gmax + j) * (int64_t)gmax + i] = k;
      }
    }
    K[i * kRow + j] = k;
    if (ta != tc) K[j * kRow + i] = k;
  }
  if (nonfinite) raise_status(d_status, PAIR_ST_NONFINITE);
  __syncthreads();

  // Rule coefficients of every ordered pair, weights from the logged rho.
  bool bad = false;
  for (int idx = tid; idx < KP * KP; idx += T) {
    const int i = idx / KP, j = idx - i * KP;
    double a = 0.0;
    if (i != j && i < gi && j < gi) {
      double rho = pd[i] * pd[j], pii = pd[i], pij = pd[j];
      if (pi_w != nullptr) {
        const float* blk = pi_w + b * (int64_t)gmax * gmax;
        const int lo = i < j ? i : j, hi = i < j ? j : i;
        rho = (double)blk[lo * gmax + hi];
        pii = (double)blk[i * gmax + i];
        pij = (double)blk[j * gmax + j];
      } else {
        rho = (double)(float)(pd[i] * pd[j]);   // the logged fl32(p_i p_j)
      }
      double wi = 1.0;
      if (rule == PAIR_RULE_MARGINAL) {
        if (!(pii > 0.0 && pii <= 1.0 && pij > 0.0 && pij <= 1.0)) bad = true;
        wi = 1.0 / pii;
      } else if (rule != PAIR_RULE_UNWEIGHTED) {
        if (!(rho > 0.0 && rho <= 1.0)) bad = true;
        wi = 1.0 / rho;
        if (rule == PAIR_RULE_CLIPPED && wi > (double)wmax) wi = (double)wmax;
      }
      a = 0.5 * (rd[i] - rd[j]) * wi;
    }
    Ac[i * kRow + j] = a;
  }
  if (bad) raise_status(d_status, PAIR_ST_RHO_RANGE);
  __syncthreads();

  // X_ij = p_j C_ij off the diagonal and X_ii = sum_j p_j A_ij, the
  // coefficients of sum_j p_j v_ij; the row sums by 16 lanes per row.
  const double M = 0.5 * (double)gi * (double)(gi - 1);
  for (int idx = tid; idx < KP * KP; idx += T) {
    const int i = idx / KP, j = idx - i * KP;
    if (i != j) X[i * kRow + j] = pd[j] * Ac[j * kRow + i];   // zero past the group
  }
  {
    const int i = tid / 16;
    double be = 0.0, d = 0.0;
    if (i < gi)
      for (int j = tid & 15; j < gi; j += 16) {
        const double a = Ac[i * kRow + j];   // zero for j = i
        be += pd[i] * pd[j] * a - 0.5 * (rd[i] - rd[j]);
        d += pd[j] * a;
      }
    be = row_sum_d(be);
    d = row_sum_d(d);
    if (i < KP && (tid & 15) == 0) {
      beta[i] = be / M;
      X[i * kRow + i] = d;
    }
  }
  __syncthreads();

  // beta^T K beta and the pair terms.
  double bk = 0.0, tr = 0.0;
  for (int idx = tid; idx < gi * gi; idx += T) {
    const int i = idx / gi, j = idx - i * gi;
    bk += beta[i] * beta[j] * K[i * kRow + j];
    if (j <= i) continue;
    const double aij = Ac[i * kRow + j], cij = Ac[j * kRow + i];
    const double rho = pd[i] * pd[j];
    const double nn = aij * aij * K[i * kRow + i] + 2.0 * aij * cij * K[i * kRow + j] +
                      cij * cij * K[j * kRow + j];
    // the pair's own term, less its share of both vertices' squares
    tr += (rho * (1.0 - rho) - pd[i] * (1.0 - pd[i]) * pd[j] * pd[j] -
           pd[j] * (1.0 - pd[j]) * pd[i] * pd[i]) * nn;
  }
  // The shared-vertex terms: Y = X K tile by tile on the fp64 matrix cores, a wave per 16 x 16 tile;
  // lane l holds rows 4 v + l / 16 and column l % 16 of it.  Rows and columns
  // past the group are zero.
  const int lane = tid & (kWave - 1), wave = tid / kWave;
  const int col = lane & 15, grp = lane >> 4;
  for (int t = wave; t < KS * KS; t += T / kWave) {
    const int r0 = 16 * (t / KS), c0 = 16 * (t % KS);
    f64x4_t y = {0.0, 0.0, 0.0, 0.0};
#pragma unroll
    for (int s = 0; s < KP / 4; ++s)
      y = __builtin_amdgcn_mfma_f64_16x16x4f64(X[(r0 + col) * kRow + 4 * s + grp],
                                               K[(4 * s + grp) * kRow + c0 + col], y, 0, 0, 0);
#pragma unroll
    for (int v = 0; v < 4; ++v) {
      const int i = r0 + 4 * v + grp;
      tr += pd[i] * (1.0 - pd[i]) * y[v] * X[i * kRow + c0 + col];
    }
  }
  const double bb = block_sum<T>(bk, sh);
  const double tt = block_sum<T>(tr, sh);
  if (tid == 0) {
    const double b2 = bb > 0.0 ? bb : 0.0;
    mse[b] = b2 + tt / (M * M);
    bias_norm[b] = sqrt(b2);
  }
}

}  // namespace

size_t exact_workspace_bytes(int64_t B, int32_t gmax, int64_t D) {
  return exact_layout(B, gmax, D).total;
}

int launch_audit_exact(int64_t B, int64_t nv, int32_t gmax, const int64_t* offsets, int64_t D,
                       const void* scores, int64_t ld, const float* rewards, const float* p,
                       const float* pi_w, int32_t rule, float wmax, double* mse,
                       double* bias_norm, double* gram, void* workspace, int32_t* d_status,
                       hipStream_t stream) {
  const ExactLayout L = exact_layout(B, gmax, D);
  const uint16_t* s = static_cast<const uint16_t*>(scores);
  const int64_t grid = B * L.nsl;
  if (grid > 0x7fffffffLL) return PAIR_ERANGE;
#define PAIR_GRAM(KS_, PART_)                                                                    \
  hipLaunchKernelGGL((gram_kernel<KS_, PART_>), dim3((unsigned)grid), dim3(kGramThreads), 0,      \
                     stream, nv, gmax, offsets, D, s, ld, L.nsl, L.slice,                        \
                     static_cast<PART_*>(workspace))
#define PAIR_FINAL(KS_, PART_)                                                                   \
  if (KS_ == 1 && L.nsl <= kFewSlices)                                                           \
    PAIR_FINAL_T(KS_, PART_, (KS_ == 1 ? 256 : 1024));                                           \
  else                                                                                           \
    PAIR_FINAL_T(KS_, PART_, 1024)
#define PAIR_FINAL_T(KS_, PART_, T_)                                                             \
  hipLaunchKernelGGL((exact_final_kernel<KS_, PART_, T_>), dim3((unsigned)B), dim3(T_), 0, stream, \
                     B, nv, gmax, offsets, rewards, p, pi_w, rule, wmax, L.nsl,                  \
                     static_cast<const PART_*>(workspace), mse, bias_norm, gram, d_status)
#define PAIR_OF(LAUNCH_, KS_) \
  if (L.wide) { LAUNCH_(KS_, double); } else { LAUNCH_(KS_, float); }
  switch (L.ks) {
    case 1: PAIR_OF(PAIR_GRAM, 1); break;
    case 2: PAIR_OF(PAIR_GRAM, 2); break;
    case 3: PAIR_OF(PAIR_GRAM, 3); break;
    default: PAIR_OF(PAIR_GRAM, 4); break;
  }
  if (hipGetLastError() != hipSuccess) return PAIR_EHIP;
  switch (L.ks) {
    case 1: PAIR_OF(PAIR_FINAL, 1); break;
    case 2: PAIR_OF(PAIR_FINAL, 2); break;
    case 3: PAIR_OF(PAIR_FINAL, 3); break;
    default: PAIR_OF(PAIR_FINAL, 4); break;
  }
#undef PAIR_OF
#undef PAIR_GRAM
#undef PAIR_FINAL_T
#undef PAIR_FINAL
  return hipGetLastError() == hipSuccess ? PAIR_OK : PAIR_EHIP;
}

}  // namespace pair
