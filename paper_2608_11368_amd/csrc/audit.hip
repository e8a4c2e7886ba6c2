// Frozen-population estimator audit (paper Sec. 6.2, Table 2; App. D
// metrics MSE = E||g^ - g_full||^2 and the bias norm) and its
// update-direction column.
//
// The complete-pair target of a prompt is itself a combination of its score
// rows, t = a S_b with a = (r_i - mean r)/(G - 1) (Theorem 1), and each
// replicate's HT estimate is g_r = u_r S_b with u_r = A~^(r) (Eq.
// pair-advantage).  With delta_r = u_r - a and the Gram matrix K = S_b S_b^T,
//     e_r   = ||g_r - t||^2 = delta_r K delta_r^T,
//     bias  = ||mean_r g_r - t|| = sqrt(delta_bar K delta_bar^T),
//     cos_r = <g_r, t> / (|g_r| |t|) = u_r K a / sqrt(u_r K u_r * a K a),
// so the score rows are needed once, for K, and a replicate costs G^2
// operations instead of 2 G D.  K is formed from exact bf16 products with
// fp32 sums of 128 columns, everything after it but the fold is fp64: e_r is
// within about 1e-7 of 64-bit arithmetic for score rows that do not nearly
// cancel in delta_r S_b, and the error grows with the square of that
// cancellation, |delta|.|s| over |delta S|.  Contracting delta_r S_b column by
// column on the fp16 matrix cores (the form before) gave 3e-4 and grew
// linearly, so it is behind until the rows cancel by a factor of 10^4; at
// B = 256, G = 16, D = 65536, R = 4096 it took 1.75 ms, bound by the
// matrix cores and the FP32 squares of their output.
//
// Pipeline (all on the caller's stream):
//  1. audit_stream  one workgroup per (prompt, column slice): the slice's
//                   partial Gram matrix, bound by HBM, and with the score
//                   loads in flight its share of the prompt's design draws,
//                   which are bound by the integer multiplies of Philox:
//                   J^(r) of each replicate as a 64-bit word.  Prompts whose
//                   rewards are all equal have delta_r = 0 in every
//                   replicate: their rows are not read.
//  2. audit_tables  workgroups per prompt: one per tile of K, the slice partials
//                   added in order (fp64), and one for the rule's edge table,
//                   the target's coefficients and the status checks.
//  3. audit_eval    64 replicates per wave: the fold of their indicators over
//                   the edge table (fp32 matrix instructions) and the
//                   quadratic form (fp64 matrix instructions).
//  4. audit_final   MSE, bias, or the mean cosine; prompts whose bias nearly
//                   cancels in K are taken from the score rows.
#include <type_traits>

#include "common.hpp"
#include "gram.hpp"
#include "launch.hpp"

namespace pair {

namespace {

constexpr int kEvalThreads = 256;
constexpr int kTableThreads = 1024;   // at most
constexpr int kFinalThreads = 256;
constexpr int64_t kFinalCols = 8 * kFinalThreads;   // columns of an audit_final step
constexpr int64_t kMaxSlices = 128;   // score-column slices per prompt at most
constexpr int64_t kMaxBiasSlices = 16;
constexpr int64_t kDrawRun = 512;     // replicates a stream workgroup draws at most, about

// Groups that may exceed 48: the fp64 sums of ten tiles leave no registers for
// the generator beside them, so the prompt's first workgroups draw and the others
// stream (128 prompts of 64, D = 65536, R = 500: 183 us, with both in one 203 us).
__host__ __device__ constexpr bool draws_apart(int ks) { return ks == 4; }

inline int64_t round_up(int64_t x, int64_t m) { return (x + m - 1) / m * m; }
inline int64_t ceil_div(int64_t a, int64_t b) { return (a + b - 1) / b; }

struct AuditLayout {
  int ks, kp;
  int64_t nsl;     // score-column slices per prompt
  int64_t slice;   // columns per slice
  int64_t slots;   // audit_stream workgroups per prompt: nsl slices, and those that only draw
  int64_t nchunk;  // audit_eval workgroups per prompt
  int rounds;      // and times 64 replicates each of their waves takes
  int64_t nbias;   // audit_final workgroups per prompt (column slices of the bias row)
  int64_t bslice;  // and columns of each
  size_t part_off, gex_off, k_off, w_off, v_off, a_off, flag_off, bits_off, epart_off, dpart_off,
      bpart_off, count_off, need;
};

// The slicing depends on gmax and D alone, so that a prompt's K, and with it
// e_r, is the same whatever batch or replicate range it is audited in.  A
// slice is 256 KB of scores where the batch's largest group fills its blocks of
// 16 rows: the partial it writes is under 5% of that.
AuditLayout audit_layout(int64_t B, int32_t gmax, int64_t D, int64_t R) {
  AuditLayout L;
  L.ks = (gmax + 15) / 16;
  L.kp = 16 * L.ks;
  int64_t nsl = ceil_div(D, (L.ks == 1 ? 4 : (L.ks == 2 ? 2 : 1)) * kGramRoundCols);
  if (nsl > kMaxSlices) nsl = kMaxSlices;
  L.slice = round_up(ceil_div(D, nsl), kGramRoundCols);
  L.nsl = ceil_div(D, L.slice);
  if (draws_apart(L.ks))
    L.slots = L.nsl + ceil_div(R, kDrawRun);
  else
    L.slots = L.nsl > ceil_div(R, kDrawRun) ? L.nsl : ceil_div(R, kDrawRun);
  // A wave's first 64 replicates cost the latency of its tables, so with many
  // it takes twice 64 (one round and two, us: B = 256, G = 16, R = 4096 29.4 and 28.9; B = 64,
  // G = 32 22.8 and 20.8; four rounds leave the last workgroups alone).  A few prompts
  // lose by it (B = 4: 5.4 and 7.0).  Groups above 32 have work enough in 64 (21 us
  // against 34 us at B = 64, G in 2..64, R = 1000).  By R and gmax alone: the sums'
  // order is the prompt's own.
  L.rounds = R >= 2048 && L.ks <= 2 ? 2 : 1;
  L.nchunk = ceil_div(R, (int64_t)L.rounds * kEvalThreads);
  const int64_t nbias = L.nsl < kMaxBiasSlices ? L.nsl : kMaxBiasSlices;
  L.bslice = round_up(ceil_div(D, nbias), kFinalCols);
  L.nbias = ceil_div(D, L.bslice);
  size_t off = 0;
  auto take = [&](int64_t bytes) {
    const size_t at = off;
    off += (size_t)round_up(bytes, 256);
    return at;
  };
  L.part_off = take(B * L.nsl * gram_tiles(L.ks) * 256 * 8);   // slice partials of K
  L.gex_off = take(B * L.nsl * (L.kp + 1) * 4);                // their row exponents
  L.k_off = take(B * L.kp * L.kp * 8);                         // K, fp64
  L.w_off = take(B * L.kp * L.kp * 4);                         // edge table
  L.v_off = take(B * L.kp * L.kp * 4);                         // 1/rho (self-normalised rule)
  L.a_off = take(B * L.kp * 8);                                // target coefficients
  L.flag_off = take(B * 4);                                    // 1: some rewards differ
  L.bits_off = take(B * R * 8);                                // indicators
  L.epart_off = take(B * L.nchunk * 8);                        // sums of e_r (of cos_r)
  L.dpart_off = take(B * L.nchunk * L.kp * 8);                 // sums of the deviations
  L.bpart_off = take(B * L.nbias * 8);                         // squared bias of the column slices
  L.count_off = take(B * 4);                                   // and how many are there
  L.need = off;
  return L;
}

// Complete-pair coefficient a_i of vertex `lane` (0 beyond the group): the
// fold with every vertex completed and rho = 1, centred over all G vertices
// (Theorem 1: (r_i - mean r) / (G - 1) in exact arithmetic).  The whole wave
// calls it; lane i holds r_i.
__device__ __forceinline__ float complete_pair_coeff(float r_i, int lane, int g) {
  const bool vert = lane < g;
  float cf = 0.0f;
  for (int j = 0; j < g; ++j) {
    const float r_j = lane_value(r_i, j);
    if (vert && j != lane) cf += r_i - r_j;
  }
  float a_full = vert ? cf / (float)(g * (g - 1)) : 0.0f;
  const float tot = wave_sum(a_full);
  return vert ? a_full - tot / (float)g : 0.0f;
}

// Some reward of the prompt differs from the first (a NaN counts as
// different).  The whole wave calls it.
__device__ __forceinline__ bool rewards_differ(const float* __restrict__ rewards, int g, int lane) {
  const float r_i = lane < g ? rewards[lane] : 0.0f;
  return __ballot(lane < g && !(r_i == lane_value(r_i, 0))) != 0ull;
}

// ---------------------------------------------------------------------------
// 1. Slice partials of K, and the design draws between their loads.
// ---------------------------------------------------------------------------
template <int KS>
__global__ __launch_bounds__(kGramThreads, gram_residency(KS)) void audit_stream_kernel(
    int64_t nv, int32_t gmax, const int64_t* __restrict__ offsets, int64_t D,
    const uint16_t* __restrict__ scores, int64_t ld, int nsl, int64_t slice, int slots,
    const float* __restrict__ rewards, const float* __restrict__ p, uint64_t seed, int64_t rep0,
    int64_t pbase, int64_t R, int skip_equal, int rescale, double* __restrict__ part,
    int32_t* __restrict__ gex, uint16_t* __restrict__ bits, int want_counts, int32_t* d_status) {
  constexpr int KP = 16 * KS;
  constexpr int kTiles = gram_tiles(KS);
  __shared__ __align__(16) uint16_t stage[gram_lds_elems(KS)];
  __shared__ int32_t ex[KP];
  __shared__ uint64_t threshold[KP];
  const int slot = (int)(blockIdx.x % (uint32_t)slots);
  const int64_t b = blockIdx.x / (uint32_t)slots;
  int64_t o0, g64;
  if (!prompt_bounds(offsets, b, nv, 2, gmax, &o0, &g64, nullptr, false)) return;
  const int g = (int)g64;
  const int tid = threadIdx.x, lane = tid & (kWave - 1);
  const int wave = __builtin_amdgcn_readfirstlane(tid / kWave);
  const bool wanted = !skip_equal || rewards_differ(rewards + o0, g, lane);
  if (!wanted && !want_counts) return;
  if (tid < KP) {
    const float pv = tid < g ? p[o0 + tid] : 0.0f;
    threshold[tid] = p_in_range(pv) ? inclusion_threshold(pv) : 0ull;
  }
  __syncthreads();

  // This wave's draws: items of 64 replicates (lane = replicate) and 16
  // vertices, dealt to the prompt's drawing waves in turn.  One unit is one Philox
  // block (four vertices) of one item; an item is 16 bits of the word.
  const int drawers = draws_apart(KS) ? slots - nsl : slots;
  const int slice_at = draws_apart(KS) ? slot - drawers : slot;
  const int ngrp = (g + 15) / 16;
  const int stride = drawers * kGramWaves;
  const int nitems = slot < drawers ? (int)((R + kWave - 1) / kWave) * ngrp : 0;
  int item = slot * kGramWaves + wave;
  const int units = item < nitems ? 4 * ((nitems - item + stride - 1) / stride) : 0;
  int done = 0;
  uint32_t word = 0;
  PhiloxRep rep;
  auto draw_until = [&](int target) {
    for (; done < target; ++done) {
      // item / ngrp for ngrp = 1 .. 4
      const int batch = ngrp == 3 ? (int)(__umulhi((uint32_t)item, 0xAAAAAAABu) >> 1)
                                  : item >> (ngrp >> 1);
      const int grp = item - batch * ngrp;
      const int64_t r = (int64_t)batch * kWave + lane;
      const int sub = done & 3, quad = 4 * grp + sub;
      if (sub == 0) {
        rep = philox_rep((uint64_t)(rep0 + r));
        word = 0;
      }
      if (4 * quad < g) {
        const Philox4x64 x = philox_quad(rep, (uint64_t)(pbase + b), (uint64_t)quad, seed);
#pragma unroll
        for (int q = 0; q < 4; ++q)   // the threshold is 0 past the group
          word |= (x.w[q] >> 32) < threshold[4 * quad + q] ? 1u << (4 * sub + q) : 0u;
      }
      if (sub == 3) {
        if (r < R) bits[(b * R + r) * 4 + grp] = (uint16_t)word;
        item += stride;
      }
    }
  };
  if (wanted && slice_at >= 0 && slice_at < nsl) {
    const int64_t c_lo = slice_at * slice;
    const int64_t c_hi = c_lo + slice < D ? c_lo + slice : D;
    gram_slice_of<KS>(scores + o0 * ld, ld, g, c_lo, c_hi, stage, ex, rescale != 0,
                      part + (b * nsl + slice_at) * (kTiles * 256),
                      gex + (b * nsl + slice_at) * (KP + 1), d_status, [&](int k, int n) {
                        if (draws_apart(KS)) return;
                        draw_until(k + 1 < n ? (int)((float)units * (float)(k + 1) / (float)n)
                                             : units);
                      });
    if (draws_apart(KS)) return;
  }
  draw_until(units);
}

// ---------------------------------------------------------------------------
// 2. Per-prompt tables: K, the edge table W_ij (the rule's weight times
//    r_i - r_j, zero on the diagonal and past G), 1/rho for the
//    self-normalised rule, the target's coefficients a, and for the cosine
//    K a and a K a.  The G x G tables are stored as the fragments that
//    audit_eval's matrix instructions take as their A operand (16 x 4: lane l
//    holds row l % 16 and column l / 16).  Step S of a row block covers the
//    columns 16 (S / 4) + 4 (l / 16) + S % 4, so that four consecutive
//    vertices of a lane group meet in four consecutive steps.
// ---------------------------------------------------------------------------
__device__ __forceinline__ int frag_column(int step, int lane) {
  return 16 * (step >> 2) + 4 * (lane >> 4) + (step & 3);
}

// The fp64 instruction leaves row 4 v + q of its result in accumulator v of
// lane group q, the fp32 one row 4 q + v: rows of K go in transposed, so that
// both leave vertex 4 q + v there.  It is its own inverse.
__device__ __forceinline__ int frag_row64(int row) { return 4 * (row & 3) + (row >> 2); }

// Place of K_ij in the fragments of a prompt.
__device__ __forceinline__ int frag_place64(int kp, int i, int j) {
  const int step = 4 * (j >> 4) + (j & 3), lane = 16 * ((j & 15) >> 2) + frag_row64(i & 15);
  return ((i >> 4) * (kp / 4) + step) * kWave + lane;
}

// One workgroup per prompt for the edge table and one per tile of K.  Rows of
// at least kTableSlices slices are summed in quarters, and the quarters in order, by 256
// threads one after the other, or by 1024 at once where the workgroups are few
// (one prompt of 16 at D = 2^20, 128 slices: 36 us with 256 threads, 9 us so; 128
// prompts of 64, 32 slices: 18 us with 256, 30 us with 1024).
constexpr int64_t kTableSlices = 64;

template <int KS>
__global__ __launch_bounds__(kTableThreads) void audit_tables_kernel(
    int64_t nv, int32_t gmax, const int64_t* __restrict__ offsets,
    const float* __restrict__ rewards, const float* __restrict__ p, const float* __restrict__ pi_w,
    int32_t rule, float wmax, int64_t nsl, int together, int skip_equal, const double* __restrict__ part,
    const int32_t* __restrict__ gex, double* __restrict__ K, float* __restrict__ wt,
    float* __restrict__ vt, double* __restrict__ a_out, int32_t* __restrict__ flag,
    int32_t* __restrict__ count, int32_t* d_status) {
  constexpr int KP = 16 * KS;
  constexpr int kTiles = gram_tiles(KS);
  __shared__ float pl[KP], rl[KP];
  __shared__ double quarter[kTableThreads / 256 - 1][256];
  const int64_t b = together ? blockIdx.x : blockIdx.x / (kTiles + 1);
  const int t = together ? 0 : (int)(blockIdx.x - b * (kTiles + 1)) - 1;
  const int tid = threadIdx.x, lane = tid & (kWave - 1), wave = tid / kWave;
  int64_t o0, g64;
  if (!prompt_bounds(offsets, b, nv, 2, gmax, &o0, &g64, d_status, (together || t < 0) && tid == 0))
    return;
  const int g = (int)g64;

  if (t >= 0 && !(skip_equal && !rewards_differ(rewards + o0, g, lane))) {
    // Thread e of a group holds entry e of the tile; the slices are added in
    // order, sixteen loads in flight.  The stream leaves no partials for a prompt
    // of equal rewards, and nothing reads its K.
    int a = 0, c = 0;
#pragma unroll
    for (int x = 0; x < KS; ++x)
#pragma unroll
      for (int y = x; y < KS; ++y)
        if (gram_tile(KS, x, y) == t) {
          a = x;
          c = y;
        }
    const int e = tid & 255, grp = __builtin_amdgcn_readfirstlane(tid >> 8);
    const int groups = (int)blockDim.x >> 8, parts = nsl >= kTableSlices ? 4 : 1;
    const int i = 16 * a + 4 * (e >> 6) + (e & 3), j = 16 * c + ((e >> 2) & 15);
    const double* src = part + (b * nsl * kTiles + t) * 256 + e;
    const int32_t* gx = gex + b * nsl * (KP + 1);
    double k = 0.0;
    const bool inside = 16 * c < g;   // uniform; entries past g inside a block are 0
    for (int u = grp; inside && u < parts; u += groups) {
      const int64_t s_lo = nsl * u / parts, s_hi = nsl * (u + 1) / parts;
      double sum = 0.0;
      // Loads past the last slice repeat it (a guarded load would wait for its
      // turn) and are not added.
      for (int64_t s0 = s_lo; s0 < s_hi; s0 += 16) {
        double v[16];
        int32_t scaled[16];
#pragma unroll
        for (int q = 0; q < 16; ++q) {
          const int64_t sl = s0 + q < s_hi ? s0 + q : s_hi - 1;
          v[q] = src[sl * (kTiles * 256)];
          scaled[q] = gx[sl * (KP + 1) + KP];
        }
#pragma unroll
        for (int q = 0; q < 16; ++q) {
          if (s0 + q >= s_hi) break;
          double x = v[q];
          if (skip_equal && scaled[q] != 0) {   // else the exponents were not written
            const int32_t* row = gx + (s0 + q) * (KP + 1);
            // rows past the prompt's own blocks have no exponent
            x = i < g && j < g ? ldexp(x, row[i] + row[j]) : 0.0;
          }
          sum += x;
        }
      }
      k += sum;
    }
    if (groups > 1) {
      if (grp > 0) quarter[grp - 1][e] = k;
      __syncthreads();
    }
    if (grp == 0) {
      for (int q = 1; q < groups; ++q) k += quarter[q - 1][e];
      if (!skip_equal && !isfinite(k)) raise_status(d_status, PAIR_ST_NONFINITE);
      K[b * (KP * KP) + frag_place64(KP, i, j)] = k;
      if (a != c) K[b * (KP * KP) + frag_place64(KP, j, i)] = k;
    }
  }
  if (t >= 0 && !together) return;

  if (wave == 0) {
    const bool vert = lane < g;
    const float r_i = vert ? rewards[o0 + lane] : 0.0f;
    const float p_i = vert ? p[o0 + lane] : 1.0f;
    if (vert && !p_in_range(p_i)) raise_status(d_status, PAIR_ST_P_RANGE);
    const float a_full = complete_pair_coeff(r_i, lane, g);
    if (lane < KP) {
      pl[lane] = p_i;
      rl[lane] = r_i;
      a_out[b * KP + lane] = (double)a_full;
    }
    const bool differ = __ballot(vert && !(r_i == lane_value(r_i, 0))) != 0ull;
    if (lane == 0) {
      flag[b] = differ ? 1 : 0;
      count[b] = 0;
    }
  }
  __syncthreads();
  bool bad_rho = false;
  for (int idx = tid; idx < KP * KP; idx += (int)blockDim.x) {
    const int fl = idx & (kWave - 1), blk = idx / kWave;
    const int i = 16 * (blk / (KP / 4)) + (fl & 15), j = frag_column(blk % (KP / 4), fl);
    float w = 0.0f, v = 0.0f;
    if (i != j && i < g && j < g) {
      float rho, pii = pl[i], pij = pl[j];
      if (pi_w != nullptr) {
        const float* blk_w = pi_w + b * (int64_t)gmax * gmax;
        const int lo = i < j ? i : j, hi = i < j ? j : i;
        rho = blk_w[lo * gmax + hi];
        pii = blk_w[i * gmax + i];
        pij = blk_w[j * gmax + j];
      } else {
        rho = pl[i] * pl[j];
      }
      float we;
      if (!rule_term(rule, wmax, rl[i] - rl[j], rho, pii, pij, &w, &we, &v)) {
        w = 0.0f;
        v = 0.0f;
        bad_rho = true;
      }
    }
    wt[b * (KP * KP) + idx] = w;
    if (rule == PAIR_RULE_SELFNORM) vt[b * (KP * KP) + idx] = v;
  }
  if (bad_rho) raise_status(d_status, PAIR_ST_RHO_RANGE);
}

// ---------------------------------------------------------------------------
// 3. Replicates: u_i = J_i (1/(2N)) sum_j J_j W_ij (fp32 products and sums),
//    then in fp64 the division, the centring over the completed vertices (not
//    for the marginal-only rule, whose fold is not antisymmetric), the target
//    and the quadratic form.  2N = G (G - 1), or k (k - 1) for the
//    observed-edge mean, or sum_{i, j observed} 1/rho_ij for the
//    self-normalised rule.  Fewer than two completed vertices: u = 0.
//
//    Both products are contractions: C = W J^T with v_mfma_f32_16x16x4_f32 and
//    Y = K x^T with v_mfma_f64_16x16x4_f64, whose rates are those of the
//    vector units but which need no broadcast of the tables.  Column l % 16 of a result is a replicate; lane l holds vertices
//    16 ib + 4 (l / 16) + v, v = 0..3, of it in both results, and that is also
//    the B operand of step 4 ib + v, so C becomes x and x meets Y in place.  One
//    lane per replicate with the tables in scalar registers took 31 us against
//    26 us here at B = 256, G = 16, R = 4096, and 123 us against 21 us at B = 64,
//    G in 2..64, R = 1000, where the 64 x 64 tables exceed the scalar cache.
//    Bound by the matrix and vector instructions together, which do not
//    overlap (of 32 us, the fp64 products took 8 and the fp32 ones 4).
// ---------------------------------------------------------------------------
typedef double f64x4_t __attribute__((ext_vector_type(4)));

// Sum over the four lane groups (rows of 16 lanes), the same in all of them.
__device__ __forceinline__ double group_sum_d(double v) {
  const uint64_t u = __builtin_bit_cast(uint64_t, v);
  auto lo = __builtin_amdgcn_permlane16_swap((uint32_t)u, (uint32_t)u, false, false);
  auto hi = __builtin_amdgcn_permlane16_swap((uint32_t)(u >> 32), (uint32_t)(u >> 32), false, false);
  v = __builtin_bit_cast(double, ((uint64_t)hi[0] << 32) | lo[0]) +
      __builtin_bit_cast(double, ((uint64_t)hi[1] << 32) | lo[1]);
  const uint64_t w = __builtin_bit_cast(uint64_t, v);
  lo = __builtin_amdgcn_permlane32_swap((uint32_t)w, (uint32_t)w, false, false);
  hi = __builtin_amdgcn_permlane32_swap((uint32_t)(w >> 32), (uint32_t)(w >> 32), false, false);
  return __builtin_bit_cast(double, ((uint64_t)hi[0] << 32) | lo[0]) +
         __builtin_bit_cast(double, ((uint64_t)hi[1] << 32) | lo[1]);
}

// All ones if bit v of a lane's four indicators is set, else 0.
__device__ __forceinline__ uint32_t vertex_mask(uint32_t nib, int v) {
  return (uint32_t)__builtin_amdgcn_sbfe((int)nib, v, 1);
}

__device__ __forceinline__ float masked(float x, uint32_t mask) {
  return __uint_as_float(__float_as_uint(x) & mask);
}

// Sum over the four lane groups, the same in all of them.
__device__ __forceinline__ float group_sum(float v) {
  auto s = __builtin_amdgcn_permlane16_swap(__float_as_uint(v), __float_as_uint(v), false, false);
  v = __uint_as_float(s[0]) + __uint_as_float(s[1]);
  s = __builtin_amdgcn_permlane32_swap(__float_as_uint(v), __float_as_uint(v), false, false);
  return __uint_as_float(s[0]) + __uint_as_float(s[1]);
}

// C[ib][cb] = table x J^T for NC blocks of 16 replicates.
template <int KS, int NC>
__device__ __forceinline__ void fold_table(const float* table, const uint32_t (&nib)[NC][KS],
                                           int nb, int lane, f32x4_t (&C)[KS][NC]) {
#pragma unroll
  for (int ib = 0; ib < KS; ++ib)
#pragma unroll
    for (int cb = 0; cb < NC; ++cb) C[ib][cb] = f32x4_t{0.0f, 0.0f, 0.0f, 0.0f};
#pragma unroll
  for (int jb = 0; jb < KS; ++jb)
    if (jb < nb) {
#pragma unroll
      for (int s = 0; s < 4; ++s) {
        float J[NC];   // 1 or 0
#pragma unroll
        for (int cb = 0; cb < NC; ++cb)
          J[cb] = __uint_as_float(vertex_mask(nib[cb][jb], s) & 0x3f800000u);
#pragma unroll
        for (int ib = 0; ib < KS; ++ib)
          if (ib < nb) {
            const float w = table[(ib * (4 * KS) + 4 * jb + s) * kWave + lane];
#pragma unroll
            for (int cb = 0; cb < NC; ++cb)
              C[ib][cb] = __builtin_amdgcn_mfma_f32_16x16x4f32(w, J[cb], C[ib][cb], 0, 0, 0);
          }
      }
    }
}

// T threads: kEvalThreads, one wave where groups of up to 16 have 64 replicates or fewer.
template <int KS, bool COS, int T>
__global__ __launch_bounds__(T) void audit_eval_kernel(
    int64_t nv, int32_t gmax, const int64_t* __restrict__ offsets, int32_t rule, int64_t R,
    int64_t nchunk, int rounds, const double* __restrict__ K, const float* __restrict__ wt,
    const float* __restrict__ vt, const double* __restrict__ a_full,
    const int32_t* __restrict__ flag, const uint64_t* __restrict__ bits,
    double* __restrict__ epart, double* __restrict__ dpart, float* __restrict__ rep_sqerr,
    int32_t* __restrict__ edge_count, double* __restrict__ target_norm) {
  constexpr int KP = 16 * KS;
  constexpr int NC = KS <= 2 ? 4 : 2;   // blocks of 16 replicates at once
  constexpr int kWaves = T / kWave;
  __shared__ __align__(16) double Ks[KP * KP];
  __shared__ __align__(16) float Ws[KP * KP];
  __shared__ __align__(16) float Vs[KP * KP];   // of the self-normalised rule
  __shared__ double wsum[kWaves][KP];
  __shared__ double red[kWaves];
  __shared__ double recip[PAIR_GMAX_LIMIT + 1];
  __shared__ float recip32[PAIR_GMAX_LIMIT + 1];
  const int64_t b = blockIdx.x / nchunk;
  const int64_t chunk = blockIdx.x - b * nchunk;
  const int tid = threadIdx.x, lane = tid & (kWave - 1), wave = tid / kWave;
  const int grp = lane >> 4;
  const int64_t first = (chunk * kWaves + wave) * rounds * kWave;   // this wave's replicates
  // Everything that depends on the prompt's number alone is asked for before
  // its size is known: one memory latency instead of four in a row.
  uint64_t next[NC];
  auto fetch = [&](int t) {
#pragma unroll
    for (int cb = 0; cb < NC; ++cb) {
      const int64_t r = first + (int64_t)t * (16 * NC) + 16 * cb + (lane & 15);
      next[cb] = r < R ? bits[b * R + r] : 0ull;
    }
  };
  fetch(0);
  double af[KS][4];
#pragma unroll
  for (int ib = 0; ib < KS; ++ib)
#pragma unroll
    for (int v = 0; v < 4; ++v) af[ib][v] = a_full[b * KP + 16 * ib + 4 * grp + v];
  const double* Kb = K + b * (KP * KP);
  for (int idx = 2 * tid; idx < KP * KP; idx += 2 * T)
    *reinterpret_cast<double2*>(Ks + idx) = *reinterpret_cast<const double2*>(Kb + idx);
  for (int idx = 4 * tid; idx < KP * KP; idx += 4 * T)
    *reinterpret_cast<float4*>(Ws + idx) =
        *reinterpret_cast<const float4*>(wt + b * (KP * KP) + idx);
  if (rule == PAIR_RULE_SELFNORM)
    for (int idx = 4 * tid; idx < KP * KP; idx += 4 * T)
      *reinterpret_cast<float4*>(Vs + idx) =
          *reinterpret_cast<const float4*>(vt + b * (KP * KP) + idx);
  const bool live = flag[b] != 0;
  int64_t o0, g64;
  if (!prompt_bounds(offsets, b, nv, 2, gmax, &o0, &g64, nullptr, false)) return;
  const int g = (int)g64;
  const int nb = KS == 1 ? 1 : (g + 15) / 16;
  const uint64_t group = g == 64 ? ~0ull : (1ull << g) - 1ull;   // bits the draws wrote
  if (COS && !live) {   // equal rewards: a = 0, no direction to compare with
    if (tid == 0) {
      epart[b * nchunk + chunk] = 0.0;
      if (chunk == 0) target_norm[b] = 0.0;
    }
    return;
  }
  if (!live) {   // equal rewards: every delta_r is exactly 0
    for (int t = 0; t < rounds; ++t) {
      const int64_t r = first + t * kWave + lane;
      if (r >= R) break;
      if (rep_sqerr != nullptr) rep_sqerr[b * R + r] = 0.0f;
      if (edge_count != nullptr) {
        const int k = __popcll(bits[b * R + r] & group);
        edge_count[b * R + r] = k * (k - 1) / 2;
      }
    }
    return;   // audit_final looks at the flag too
  }
  for (int k = tid; k <= PAIR_GMAX_LIMIT; k += T) {
    recip[k] = k > 0 ? 1.0 / (double)k : 0.0;
    recip32[k] = rule != PAIR_RULE_MARGINAL ? (float)recip[k] : 0.0f;   // not centred
  }
  __syncthreads();
  const double inv_pool = 1.0 / (double)(g * (g - 1));

  // x K x^T of the columns: off the diagonal blocks each pair of blocks counts
  // twice.
  auto quadratic = [&](const auto& x, auto& q) {
    constexpr int N = sizeof(q) / sizeof(q[0]);
#pragma unroll
    for (int cb = 0; cb < N; ++cb) q[cb] = 0.0;
#pragma unroll
    for (int ib = 0; ib < KS; ++ib)
      if (ib < nb) {
        f64x4_t Y[N], D[N];
#pragma unroll
        for (int cb = 0; cb < N; ++cb) Y[cb] = D[cb] = f64x4_t{0.0, 0.0, 0.0, 0.0};
#pragma unroll
        for (int jb = ib; jb < KS; ++jb)
          if (jb < nb) {
#pragma unroll
            for (int s = 0; s < 4; ++s) {
              const double kf = Ks[(ib * (4 * KS) + 4 * jb + s) * kWave + lane];
#pragma unroll
              for (int cb = 0; cb < N; ++cb) {
                if (jb == ib)
                  D[cb] = __builtin_amdgcn_mfma_f64_16x16x4f64(kf, x[jb][cb][s], D[cb], 0, 0, 0);
                else
                  Y[cb] = __builtin_amdgcn_mfma_f64_16x16x4f64(kf, x[jb][cb][s], Y[cb], 0, 0, 0);
              }
            }
          }
#pragma unroll
        for (int cb = 0; cb < N; ++cb)
#pragma unroll
          for (int v = 0; v < 4; ++v) {
            const double y = KS == 1 ? D[cb][v] : __builtin_fma(2.0, Y[cb][v], D[cb][v]);
            q[cb] = __builtin_fma(x[ib][cb][v], y, q[cb]);
          }
      }
  };

  // For the cosine: af becomes K a, and tt = a K a.
  double tt = 0.0;
  if (COS) {
    f64x4_t Y[KS];
#pragma unroll
    for (int ib = 0; ib < KS; ++ib) {
      Y[ib] = f64x4_t{0.0, 0.0, 0.0, 0.0};
      if (ib < nb) {
#pragma unroll
        for (int jb = 0; jb < KS; ++jb)
          if (jb < nb) {
#pragma unroll
            for (int s = 0; s < 4; ++s)
              Y[ib] = __builtin_amdgcn_mfma_f64_16x16x4f64(
                  Ks[(ib * (4 * KS) + 4 * jb + s) * kWave + lane], af[jb][s], Y[ib], 0, 0, 0);
          }
      }
    }
#pragma unroll
    for (int ib = 0; ib < KS; ++ib)
#pragma unroll
      for (int v = 0; v < 4; ++v) {
        tt = __builtin_fma(af[ib][v], Y[ib][v], tt);
        af[ib][v] = Y[ib][v];
      }
    tt = group_sum_d(tt);
    if (chunk == 0 && tid == 0) target_norm[b] = tt > 0.0 ? sqrt(tt) : 0.0;
  }

  // Sums of the deviations, in fp64: what cancels in them is sqrt(R) times
  // the mean.  (A factor instead of a branch: the blocks of replicates stay one
  // basic block, whose chains interleave.)
  double dsum[KS][4];
#pragma unroll
  for (int ib = 0; ib < KS; ++ib)
#pragma unroll
    for (int v = 0; v < 4; ++v) dsum[ib][v] = 0.0;
  double esum = 0.0;
  const int steps = first < R ? rounds * (4 / NC) : 0;   // waves past R have no replicates
#pragma unroll 1
  for (int t = 0; t < steps; ++t) {
    const int64_t r0 = first + (int64_t)t * (16 * NC) + (lane & 15);
    uint32_t nib[NC][KS];   // this lane's four indicators of each block of vertices
    int k[NC];
#pragma unroll
    for (int cb = 0; cb < NC; ++cb) {
      const uint64_t drawn = next[cb] & group;
      k[cb] = __popcll(drawn);
      const uint64_t word = k[cb] < 2 ? 0ull : drawn;
#pragma unroll
      for (int ib = 0; ib < KS; ++ib)
        nib[cb][ib] = (uint32_t)(word >> (32 * (ib / 2))) >> (16 * (ib % 2) + 4 * grp);
    }
    if (t + 1 < steps) fetch(t + 1);
    f32x4_t C[KS][NC];
    double inv[NC];
#pragma unroll
    for (int cb = 0; cb < NC; ++cb) inv[cb] = inv_pool;
    if (rule == PAIR_RULE_RATIO_KE) {
#pragma unroll
      for (int cb = 0; cb < NC; ++cb)
        inv[cb] = k[cb] >= 2 ? recip[k[cb]] * recip[k[cb] - 1] : 0.0;
    } else if (rule == PAIR_RULE_SELFNORM) {
      fold_table<KS, NC>(Vs, nib, nb, lane, C);
#pragma unroll
      for (int cb = 0; cb < NC; ++cb) {
        double n2 = 0.0;
#pragma unroll
        for (int ib = 0; ib < KS; ++ib)
#pragma unroll
          for (int v = 0; v < 4; ++v)
            n2 += (double)masked(C[ib][cb][v], vertex_mask(nib[cb][ib], v));
        n2 = group_sum_d(n2);
        inv[cb] = k[cb] >= 2 ? 1.0 / n2 : 0.0;
      }
    }
    fold_table<KS, NC>(Ws, nib, nb, lane, C);

    // The folds c_i = sum_j J_j W_ij of the completed vertices are centred in
    // fp32; the normaliser, whose rounding would be the same in every
    // replicate and so survive in their mean, is applied in fp64.
    double x[KS][NC][4];
#pragma unroll
    for (int cb = 0; cb < NC; ++cb) {
      float sum = 0.0f;
#pragma unroll
      for (int ib = 0; ib < KS; ++ib)
#pragma unroll
        for (int v = 0; v < 4; ++v) {
          C[ib][cb][v] = masked(C[ib][cb][v], vertex_mask(nib[cb][ib], v));
          sum += C[ib][cb][v];
        }
      const float mean = group_sum(sum) * recip32[k[cb]];
      const double counts = r0 + 16 * cb < R ? 1.0 : 0.0;   // replicates past R do not
#pragma unroll
      for (int ib = 0; ib < KS; ++ib)
#pragma unroll
        for (int v = 0; v < 4; ++v) {
          const float c = masked(C[ib][cb][v] - mean, vertex_mask(nib[cb][ib], v));
          if (COS) {
            x[ib][cb][v] = (double)c * inv[cb];
          } else {
            x[ib][cb][v] = __builtin_fma((double)c, inv[cb], -af[ib][v]);
            dsum[ib][v] = __builtin_fma(counts, x[ib][cb][v], dsum[ib][v]);
          }
        }
    }

    double q[NC];
    quadratic(x, q);

    double mine = 0.0;   // the replicate this lane stores: block grp
    int my_k = 0;
#pragma unroll
    for (int cb = 0; cb < NC; ++cb) {
      double e = group_sum_d(q[cb]);
      if (COS) {
        double uka = 0.0;
#pragma unroll
        for (int ib = 0; ib < KS; ++ib)
#pragma unroll
          for (int v = 0; v < 4; ++v) uka = __builtin_fma(x[ib][cb][v], af[ib][v], uka);
        uka = group_sum_d(uka);
        // 0 when either quadratic form is not positive (a draw with no observed
        // edge has u_r = 0 exactly; a prompt with equal rewards has a = 0).
        e = (r0 + 16 * cb < R && tt > 0.0 && e > 0.0) ? uka / sqrt(e * tt) : 0.0;
      } else {
        // rounding: the form is not negative; replicates past R count nothing
        e = (e < 0.0 || r0 + 16 * cb >= R) ? 0.0 : e;
      }
      if (grp == cb) {
        mine = e;
        my_k = k[cb];
      }
      esum += e;
    }
    if (!COS) {
      const int64_t r = r0 + 16 * grp;
      if (grp < NC && r < R) {
        if (rep_sqerr != nullptr) rep_sqerr[b * R + r] = (float)mine;
        if (edge_count != nullptr) edge_count[b * R + r] = my_k * (my_k - 1) / 2;
      }
    }
  }

  // Fixed-order sums over the replicates: the 16 columns, then the waves in order.
  esum = row_sum_d(esum);
  if (lane == 0) red[wave] = esum;
  if (!COS) {
#pragma unroll
    for (int ib = 0; ib < KS; ++ib)
#pragma unroll
      for (int v = 0; v < 4; ++v) {
        const double s = row_sum_d(dsum[ib][v]);
        if ((lane & 15) == 0) wsum[wave][16 * ib + 4 * grp + v] = s;
      }
  }
  __syncthreads();
  if (tid == 0) {
    double t = 0.0;
#pragma unroll
    for (int w = 0; w < kWaves; ++w) t += red[w];
    epart[b * nchunk + chunk] = t;
  }
  if (!COS && tid < KP) {
    double s = 0.0;
#pragma unroll
    for (int w = 0; w < kWaves; ++w) s += wsum[w][tid];
    dpart[(b * nchunk + chunk) * KP + tid] = s;
  }
}

// ---------------------------------------------------------------------------
// 4. Fixed-order reductions over the replicate chunks: the MSE (or the mean
//    cosine) and the bias norm |delta_bar S|.
//
//    The quadratic form delta_bar K delta_bar^T carries K's rounding (4e-9 of what
//    cancels in it) into the bias norm, so its relative error grows with the square of the
//    cancellation, where a sum per score column grows with its first power.  K
//    serves while the form is at least 1 / kCancel of sum_i delta_bar_i^2 K_ii (1e-7 at
//    the most); below that, as with a component that all rows of a prompt
//    share, the prompt's rows are read again and delta_bar S is summed column by
//    column in fp64.  Every workgroup of a prompt decides for itself (the
//    form takes it as long as asking another), and the last of them adds the slices in order.
//    G = 16, D = 4096, R = 1000, a common component of 100 times the rest: the form alone
//    is off by 1e-4 of the norm, so 1e-6.  64 registers, so that eight workgroups
//    share a CU: B = 256, G = 16, D = 65536, R = 4096 4.6 us (with 130 registers
//    6.6), 128 prompts of 64 with 16 slices 8.6 (32 slices and 130 registers: 18.5), and
//    190 us where every prompt of the former is read again.
// ---------------------------------------------------------------------------
constexpr double kCancel = 64.0;

template <bool COS>
__global__ __launch_bounds__(kFinalThreads, 8) void audit_final_kernel(
    int64_t nv, int32_t gmax, int kp, const int64_t* __restrict__ offsets, int64_t D,
    const uint16_t* __restrict__ scores, int64_t ld, int nbias, int64_t bslice, int64_t R,
    int64_t nchunk, const double* __restrict__ K, const int32_t* __restrict__ flag,
    const double* __restrict__ epart, const double* __restrict__ dpart, double* bpart,
    int32_t* count, double* __restrict__ first, double* __restrict__ bias_norm) {
  __shared__ double dl[kWave];
  __shared__ double form, sh[kFinalThreads / kWave];
  __shared__ int by_column;
  const int slot = (int)(blockIdx.x % (uint32_t)nbias);
  const int64_t b = blockIdx.x / (uint32_t)nbias;
  const int tid = threadIdx.x, lane = tid & (kWave - 1), wave = tid / kWave;
  int64_t o0, g64;
  if (!prompt_bounds(offsets, b, nv, 2, gmax, &o0, &g64, nullptr, false)) return;
  const int g = (int)g64;
  if (!COS && flag[b] == 0) {   // equal rewards: exact zeros
    if (slot == 0 && tid == 0) {
      first[b] = 0.0;
      bias_norm[b] = 0.0;
    }
    return;
  }
  if (wave == (COS ? 0 : 1) && slot == 0) {
    double t = 0.0;
    for (int64_t c = lane; c < nchunk; c += kWave) t += epart[b * nchunk + c];
    t = wave_sum_d(t);
    if (lane == 0) first[b] = t / (double)R;   // the MSE, or the mean cosine
  }
  if (COS) return;
  if (wave == 0) {
    double d = 0.0;
    if (lane < g) {
      int64_t c = 0;
      for (; c + 8 <= nchunk; c += 8) {   // eight loads in flight
        double v[8];
#pragma unroll
        for (int q = 0; q < 8; ++q) v[q] = dpart[(b * nchunk + c + q) * kp + lane];
#pragma unroll
        for (int q = 0; q < 8; ++q) d += v[q];
      }
      for (; c < nchunk; ++c) d += dpart[(b * nchunk + c) * kp + lane];
      d = d / (double)R;
    }
    const double* Kb = K + b * (kp * kp);
    const int row = lane < g ? lane : 0;   // lanes past the group read row 0
    const double kii = Kb[frag_place64(kp, row, row)];
    double y = 0.0;
    for (int j0 = 0; j0 < g; j0 += 16) {
      double v[16];
#pragma unroll
      for (int q = 0; q < 16; ++q) v[q] = Kb[frag_place64(kp, row, j0 + q)];
#pragma unroll
      for (int q = 0; q < 16; ++q) y = __builtin_fma(v[q], readlane_d(d, j0 + q), y);
    }
    const double q = wave_sum_d(d * y);   // d is 0 past the group
    const double own = wave_sum_d(d * d * kii);
    dl[lane] = d;
    if (lane == 0) {
      form = q;
      by_column = !(q * kCancel >= own) ? 1 : 0;
    }
  }
  __syncthreads();
  if (by_column == 0) {
    if (slot == 0 && tid == 0) bias_norm[b] = sqrt(form);
    return;
  }

  // Eight columns per thread and step, four rows in flight.  Rows past the
  // group repeat the last one, with the factor 0.
  const uint16_t* rows = scores + o0 * ld;
  const int64_t c_lo = slot * bslice, c_hi = c_lo + bslice < D ? c_lo + bslice : D;
  double sq = 0.0;
  for (int64_t c = c_lo + 8 * tid; c < c_hi; c += kFinalCols) {
    double y[8];
#pragma unroll
    for (int e = 0; e < 8; ++e) y[e] = 0.0;
    if (c + 8 <= c_hi) {
      for (int i0 = 0; i0 < g; i0 += 4) {
        uint4 v[4];
#pragma unroll
        for (int s = 0; s < 4; ++s) {
          const int i = i0 + s < g ? i0 + s : g - 1;
          v[s] = load_nt16(rows + (int64_t)i * ld + c);
        }
#pragma unroll
        for (int s = 0; s < 4; ++s) {
          const double f = dl[i0 + s];
          const uint32_t w[4] = {v[s].x, v[s].y, v[s].z, v[s].w};
#pragma unroll
          for (int e = 0; e < 4; ++e) {
            y[2 * e] = __builtin_fma(f, (double)bf16lo_to_f32(w[e]), y[2 * e]);
            y[2 * e + 1] = __builtin_fma(f, (double)bf16hi_to_f32(w[e]), y[2 * e + 1]);
          }
        }
      }
    } else {   // the row's last columns
      for (int i = 0; i < g; ++i)
#pragma unroll
        for (int e = 0; e < 8; ++e)
          if (c + e < c_hi)
            y[e] = __builtin_fma(dl[i], (double)bf16lo_to_f32(rows[(int64_t)i * ld + c + e]), y[e]);
    }
#pragma unroll
    for (int e = 0; e < 8; ++e) sq = __builtin_fma(y[e], y[e], sq);
  }
  sq = wave_sum_d(sq);
  if (lane == 0) sh[wave] = sq;
  __syncthreads();
  if (tid != 0) return;
  double t = 0.0;
#pragma unroll
  for (int w = 0; w < kFinalThreads / kWave; ++w) t += sh[w];
  // The slices' sums cross workgroups: stored and read past the caches of one XCD.
  __hip_atomic_store(bpart + b * nbias + slot, t, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
  if (__hip_atomic_fetch_add(count + b, 1, __ATOMIC_ACQ_REL, __HIP_MEMORY_SCOPE_AGENT) != nbias - 1)
    return;
  t = 0.0;
  for (int s = 0; s < nbias; ++s)
    t += __hip_atomic_load(bpart + b * nbias + s, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
  bias_norm[b] = sqrt(t);
}

struct AuditArgs {
  int64_t B, nv;
  int32_t gmax;
  const int64_t* offsets;
  int64_t D;
  const void* scores;
  int64_t ld;
  const float *rewards, *p, *pi_w;
  int32_t rule;
  float wmax;
  uint64_t seed;
  int64_t rep0, pbase, R;
  double *first, *second;   // mse and bias norm, or cosine and target norm
  float* rep_sqerr;
  int32_t* edge_count;
  void* workspace;
  int32_t* d_status;
  hipStream_t stream;
};

template <int KS, bool COS>
int run_audit(const AuditLayout& L, const AuditArgs& A) {
  unsigned char* ws = static_cast<unsigned char*>(A.workspace);
  double* part = reinterpret_cast<double*>(ws + L.part_off);
  int32_t* gex = reinterpret_cast<int32_t*>(ws + L.gex_off);
  double* K = reinterpret_cast<double*>(ws + L.k_off);
  float* wt = reinterpret_cast<float*>(ws + L.w_off);
  float* vt = reinterpret_cast<float*>(ws + L.v_off);
  double* a = reinterpret_cast<double*>(ws + L.a_off);
  int32_t* flag = reinterpret_cast<int32_t*>(ws + L.flag_off);
  uint64_t* bits = reinterpret_cast<uint64_t*>(ws + L.bits_off);
  double* epart = reinterpret_cast<double*>(ws + L.epart_off);
  double* dpart = reinterpret_cast<double*>(ws + L.dpart_off);
  double* bpart = reinterpret_cast<double*>(ws + L.bpart_off);
  int32_t* count = reinterpret_cast<int32_t*>(ws + L.count_off);
  const uint16_t* s = static_cast<const uint16_t*>(A.scores);

  // Every grid size is checked before the first launch.
  const int64_t stream_grid = A.B * L.slots, eval_grid = A.B * L.nchunk;
  const int64_t table_grid = A.B * (gram_tiles(KS) + 1);
  const int64_t nbias = COS ? 1 : L.nbias, final_grid = A.B * nbias;
  if (stream_grid > 0x7fffffffLL || eval_grid > 0x7fffffffLL || table_grid > 0x7fffffffLL ||
      final_grid > 0x7fffffffLL)
    return PAIR_ERANGE;
  // The cosine audit reports what its Gram matrix holds, so it reads every
  // prompt and leaves the products unscaled: an overflow is a non-finite entry.
  const int own = COS ? 0 : 1;
  hipLaunchKernelGGL((audit_stream_kernel<KS>), dim3((unsigned)stream_grid), dim3(kGramThreads), 0,
                     A.stream, A.nv, A.gmax, A.offsets, A.D, s, A.ld, (int)L.nsl, L.slice,
                     (int)L.slots, A.rewards, A.p, A.seed, A.rep0, A.pbase, A.R, own, own, part, gex,
                     reinterpret_cast<uint16_t*>(bits), A.edge_count != nullptr ? 1 : 0,
                     A.d_status);
  if (hipGetLastError() != hipSuccess) return PAIR_EHIP;
  // Groups of up to 16 have one tile: more prompts than the chip holds of both
  // kinds of workgroups at once take one workgroup for both (2000 prompts:
  // 12.9 us in two, 9.5 us in one; 256 prompts: 4.9 us in two).
  const bool together = KS == 1 && table_grid > 8 * (int64_t)device_cu_count();
  const bool few = L.nsl >= kTableSlices && table_grid <= 2 * (int64_t)device_cu_count();
  hipLaunchKernelGGL((audit_tables_kernel<KS>), dim3((unsigned)(together ? A.B : table_grid)),
                     dim3(few ? kTableThreads : 256), 0,
                     A.stream, A.nv, A.gmax, A.offsets, A.rewards, A.p, A.pi_w, A.rule, A.wmax,
                     L.nsl, together ? 1 : 0, own, part, gex, K, wt, vt, a, flag, count, A.d_status);
  if (hipGetLastError() != hipSuccess) return PAIR_EHIP;
  auto eval = [&](auto threads) {
    constexpr int T = decltype(threads)::value;
    hipLaunchKernelGGL((audit_eval_kernel<KS, COS, T>), dim3((unsigned)eval_grid), dim3(T), 0,
                       A.stream, A.nv, A.gmax, A.offsets, A.rule, A.R, L.nchunk, L.rounds, K, wt, vt,
                       a, flag, bits, epart, dpart, A.rep_sqerr, A.edge_count,
                       COS ? A.second : nullptr);
  };
  // A chunk of at most 64 replicates and small tables are one wave's (2000 prompts of 4,
  // R = 32: 13.5 us with four, 8.3 us with one).
  if (KS == 1 && A.R <= kWave)
    eval(std::integral_constant<int, KS == 1 ? kWave : kEvalThreads>{});
  else
    eval(std::integral_constant<int, kEvalThreads>{});
  if (hipGetLastError() != hipSuccess) return PAIR_EHIP;
  hipLaunchKernelGGL((audit_final_kernel<COS>), dim3((unsigned)final_grid), dim3(kFinalThreads), 0,
                     A.stream, A.nv, A.gmax, L.kp, A.offsets, A.D, s, A.ld, (int)nbias, L.bslice,
                     A.R, L.nchunk, K, flag, epart, dpart, bpart, count, A.first, A.second);
  return hipGetLastError() == hipSuccess ? PAIR_OK : PAIR_EHIP;
}

// Columns per slice of the column-by-column contraction.
int64_t contraction_cols(int64_t ks) { return ks == 1 ? 2048 : (ks == 2 ? 1024 : 512); }

// The range of a call is the one of that contraction, a workgroup per 256
// replicates and (but for the cosine) per slice; the grids here are smaller.
template <bool COS>
bool out_of_range(const AuditArgs& A) {
  const int64_t reps = ceil_div(COS ? A.R : A.R + 1, 256);
  const int64_t slices = COS ? 1 : ceil_div(A.D, contraction_cols((A.gmax + 15) / 16));
  return A.B * reps > 0x7fffffffLL || A.B * slices > 0x7fffffffLL;
}

template <bool COS>
int launch_any(const AuditArgs& A) {
  if (out_of_range<COS>(A)) return PAIR_ERANGE;
  const AuditLayout L = audit_layout(A.B, A.gmax, A.D, A.R);
  switch (L.ks) {
    case 1: return run_audit<1, COS>(L, A);
    case 2: return run_audit<2, COS>(L, A);
    case 3: return run_audit<3, COS>(L, A);
    default: return run_audit<4, COS>(L, A);
  }
}

}  // namespace

// The size a caller is asked for.  It is the one of the column-by-column
// contraction (fp32 deviations of every replicate and their per-slice sums),
// so that buffers sized by it, and the calls that pair_audit_noalloc's fixed
// scratch admits, stay what they were; what the audit writes (audit_need_bytes) is
// less except for a few replicates of wide groups, where it decides.
static size_t contraction_bytes(int64_t B, int32_t gmax, int64_t D, int64_t R, bool direction) {
  const int64_t ks = (gmax + 15) / 16, kp = 16 * ks;
  const int64_t rrows = round_up(R, 64) + 32, nwg = ceil_div(R, 256);
  const int64_t cols = contraction_cols(ks);
  size_t n = (size_t)round_up(B * rrows * kp * 4, 256) + (size_t)round_up(B * nwg * gmax * 4, 256);
  if (direction)
    return n + (size_t)round_up((int64_t)exact_workspace_bytes(B, gmax, D), 256) +
           (size_t)round_up(B * (int64_t)gmax * gmax * 8, 256) + (size_t)round_up(B * nwg * 8, 256);
  return n + (size_t)round_up(B * ceil_div(D, cols) * rrows * 4, 256) +
         (size_t)round_up(B * ceil_div(R + 1, 256) * 8, 256) + (size_t)round_up(B * 4, 256) +
         (size_t)round_up((2 * B + 1) * 4, 256);
}

size_t audit_need_bytes(int64_t B, int32_t gmax, int64_t D, int64_t R) {
  return audit_layout(B, gmax, D, R).need;
}

size_t audit_workspace_bytes(int64_t B, int32_t gmax, int64_t D, int64_t R) {
  const size_t a = contraction_bytes(B, gmax, D, R, false), n = audit_need_bytes(B, gmax, D, R);
  return a > n ? a : n;
}

size_t direction_workspace_bytes(int64_t B, int32_t gmax, int64_t D, int64_t R) {
  const size_t a = contraction_bytes(B, gmax, D, R, true), n = audit_need_bytes(B, gmax, D, R);
  return a > n ? a : n;
}

int launch_audit_direction(int64_t B, int64_t nv, int32_t gmax, const int64_t* offsets, int64_t D,
                           const void* scores, int64_t ld, const float* rewards, const float* p,
                           const float* pi_w, int32_t rule, float wmax, uint64_t seed,
                           int64_t rep0, int64_t R, double* cosine, double* target_norm,
                           void* workspace, int32_t* d_status, hipStream_t stream) {
  return launch_any<true>(AuditArgs{B, nv, gmax, offsets, D, scores, ld, rewards, p, pi_w, rule,
                                    wmax, seed, rep0, 0, R, cosine, target_norm, nullptr, nullptr,
                                    workspace, d_status, stream});
}

int launch_audit(int64_t B, int64_t nv, int32_t gmax, const int64_t* offsets, int64_t D,
                 const void* scores, int64_t ld, const float* rewards, const float* p,
                 const float* pi_w, int32_t rule, float wmax, uint64_t seed, int64_t rep0,
                 int64_t pbase, int64_t R, double* mse, double* bias_norm, float* rep_sqerr,
                 int32_t* edge_count, void* workspace, int32_t* d_status, hipStream_t stream) {
  return launch_any<false>(AuditArgs{B, nv, gmax, offsets, D, scores, ld, rewards, p, pi_w, rule,
                                     wmax, seed, rep0, pbase, R, mse, bias_norm, rep_sqerr,
                                     edge_count, workspace, d_status, stream});
}

}  // namespace pair
