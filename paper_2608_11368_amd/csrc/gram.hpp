// Streaming Gram partial K = S_b S_b^T of one prompt over one slice of score
// columns, shared by the audits (gfx950, wave64).
//
// Bound by HBM: a score row is read once (2 bytes per element against G
// multiply-adds on the matrix cores).  v_mfma_f32_16x16x32_bf16 takes its A
// fragment (rows of S) and B fragment (columns of S^T) from the same
// registers, so one 16-byte fragment per row block, lane and step serves
// both sides, and only the row-block pairs a <= c are multiplied.
//
// The four waves of a workgroup take the slice's chunks of 16 KS rows x kCols
// columns (16, 12 or 8 KB) in turn, each for itself: a wave loads a chunk in
// runs of 256 B to 1 KB per row, stages it in its own part of LDS (rows skewed
// by 16 bytes: conflict-free fragment reads) and, with the loads of its next
// chunk in flight, multiplies it.  No barrier is needed until the waves' sums
// are added at the end.  8 to 16 waves per CU keep 128 KB in flight.  The shape follows the prompt's own group size and not
// the batch's largest, so that small groups of a ragged batch stream in whole
// chunks too.
#pragma once

#include <type_traits>

#include "common.hpp"

namespace pair {

typedef __bf16 bf16x8_t __attribute__((ext_vector_type(8)));

constexpr int kGramThreads = 256;

// Workgroups per CU that gram_lds_elems() and the registers admit.
constexpr int gram_residency(int km) { return km <= 2 ? 4 : 2; }
constexpr int kGramWaves = kGramThreads / kWave;

constexpr int gram_tiles(int ks) { return ks * (ks + 1) / 2; }   // row-block pairs a <= c

// Index of the pair (a, c), a <= c: rows of the upper triangle in order.
__host__ __device__ constexpr int gram_tile(int ks, int a, int c) {
  return a * ks - a * (a - 1) / 2 + (c - a);
}

// Entry (i, j) of a tile sits where the matrix instruction leaves it: lane
// 16 (i / 4) + j, accumulator i % 4.
__device__ __forceinline__ int gram_entry(int i, int j) { return (16 * (i >> 2) + j) * 4 + (i & 3); }

// HALF (KS <= 2): chunks of 8 KB, for kernels whose largest shape is KS = 2:
// their LDS and registers then admit four workgroups per CU instead of two.
template <int KS, bool HALF>
struct GramShape {
  static constexpr int KP = 16 * KS;
  static constexpr int kCols = (KS == 1 ? 512 : (KS == 2 ? 256 : 128)) / (HALF ? 2 : 1);
  static constexpr int kRowLanes = kCols / 8;                           // lanes that load one row
  static constexpr int kRowsPerLoad = kWave / kRowLanes;
  static constexpr int kLoads = KP / kRowsPerLoad;                      // 16-byte loads per lane
  static constexpr int kStride = kCols + 8;                             // LDS row stride, elements
  static constexpr int kTiles = gram_tiles(KS);
  static constexpr int kWaveElems = KP * kStride;
  static constexpr int kLdsElems = kGramWaves * kWaveElems;
};

// Columns of a slice come in whole rounds of the four waves, for every shape.
constexpr int kGramRoundCols = 2048;

// bf16 pair times 2^ne per element, rounded back to bf16: exact down to
// bf16's subnormals.
__device__ __forceinline__ uint32_t scale_bf16_pair(uint32_t w, int ne) {
  const float lo = ldexpf(bf16lo_to_f32(w), ne), hi = ldexpf(bf16hi_to_f32(w), ne);
  return (__float_as_uint(lo) >> 16) | (__float_as_uint(hi) & 0xffff0000u);
}

// One pass of a wave over its chunks of columns [c_lo, c_hi) of the g rows at
// `rows`, 16 (KS - 1) < g <= 16 KS: adds to acc[tile].  SCALED: row i is
// multiplied by 2^-ex[i] first.  `between(k, n)` is called once per chunk k of
// n with the next chunk's loads in flight.  Rows past g are zero in the stage
// and never loaded.
//
// The loads of a whole chunk sit in straight-line code guarded by uniform
// branches only: with a per-lane guard, or with the partial last chunk merged
// into the same registers, the compiler waits for the loads where the paths
// meet, and nothing is in flight during the multiplication.
//
// The sums of every four matrix instructions move to fp64: their accumulation
// rounds with a bias, which grows with the length of a run (runs of 16 left
// 4e-8 in the exact audit's MSE, B = 128, G in 2..64, D = 65536; runs of 64, at
// G = 64 and D = 2^20, 4e-6 in the target norm of rows that share ten parts in
// eleven, where these leave 1e-7).
template <int KS, bool HALF>
struct GramAcc {
  f32x4_t f[GramShape<KS, HALF>::kTiles];
  double d[GramShape<KS, HALF>::kTiles][4];
};

template <int KS, bool HALF, bool SCALED, class Between>
__device__ __forceinline__ void gram_pass(const uint16_t* __restrict__ rows, int64_t ld, int g,
                                          int64_t c_lo, int64_t c_hi, uint16_t* stage, int wave,
                                          int lane, const int32_t* ex,
                                          GramAcc<KS, HALF>& acc, Between&& between) {
  using H = GramShape<KS, HALF>;
  const int rsub = lane / H::kRowLanes, csub = 8 * (lane % H::kRowLanes);
  const int64_t nwhole = (c_hi - c_lo) / H::kCols;                       // whole chunks
  const int n = (int)((nwhole - wave + kGramWaves - 1) / kGramWaves);    // this wave's
  const bool last = (c_hi - c_lo) % H::kCols != 0 && nwhole % kGramWaves == wave;
  uint16_t* put = stage + rsub * H::kStride + csub;
  auto put_at = [&](int t) { return reinterpret_cast<uint4*>(put + t * H::kRowsPerLoad * H::kStride); };
  for (int t = g / H::kRowsPerLoad; t < H::kLoads; ++t) *put_at(t) = make_uint4(0u, 0u, 0u, 0u);

  auto multiply = [&]() {
    if (SCALED) {
#pragma unroll 1
      for (int t = 0; t * H::kRowsPerLoad < g; ++t) {
        const int ne = -ex[t * H::kRowsPerLoad + rsub];
        uint4 x = *put_at(t);
        x.x = scale_bf16_pair(x.x, ne);
        x.y = scale_bf16_pair(x.y, ne);
        x.z = scale_bf16_pair(x.z, ne);
        x.w = scale_bf16_pair(x.w, ne);
        *put_at(t) = x;
      }
    }
    wave_lds_order();   // the rows are staged
    // Fragment of row block q, step s: row 16 q + l % 16, columns 32 s +
    // 8 (l / 16) .. + 7 (the order of the 32 products does not matter as
    // long as both operands share it).
    const uint16_t* frag = stage + (lane & 15) * H::kStride + 8 * (lane >> 4);
#pragma unroll
    for (int s = 0; s < H::kCols / 32; ++s) {
      bf16x8_t fr[KS];
#pragma unroll
      for (int q = 0; q < KS; ++q)
        fr[q] = __builtin_bit_cast(
            bf16x8_t, *reinterpret_cast<const uint4*>(frag + 16 * q * H::kStride + 32 * s));
#pragma unroll
      for (int a = 0; a < KS; ++a)
#pragma unroll
        for (int c = a; c < KS; ++c)
          acc.f[gram_tile(KS, a, c)] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(
              fr[a], fr[c], acc.f[gram_tile(KS, a, c)], 0, 0, 0);
      if (s % 4 == 3) {
#pragma unroll
        for (int i = 0; i < H::kTiles; ++i) {
#pragma unroll
          for (int v = 0; v < 4; ++v) acc.d[i][v] += (double)acc.f[i][v];
          acc.f[i] = f32x4_t{0.0f, 0.0f, 0.0f, 0.0f};
        }
      }
    }
    wave_lds_order();   // and read
  };

  uint4 v[H::kLoads];
  // A load slot that ends past row g reads row g - 1 again in its idle lanes.
  auto load = [&](int k) {
    const uint16_t* base =
        rows + c_lo + ((int64_t)k * kGramWaves + wave) * H::kCols + csub;
#pragma unroll
    for (int t = 0; t < H::kLoads; ++t) {
      if (t * H::kRowsPerLoad < 16 * (KS - 1) || t * H::kRowsPerLoad < g) {
        int row = t * H::kRowsPerLoad + rsub;
        row = row < g ? row : g - 1;
        v[t] = load_nt16(base + (int64_t)row * ld);
      }
    }
  };
  if (n > 0) load(0);
  for (int k = 0; k < n; ++k) {
#pragma unroll
    for (int t = 0; t < H::kLoads; ++t) {
      if (t * H::kRowsPerLoad < 16 * (KS - 1)) {
        *put_at(t) = v[t];
      } else if (t * H::kRowsPerLoad < g) {
        if (t * H::kRowsPerLoad + rsub < g) *put_at(t) = v[t];
      }
    }
    if (k + 1 < n) load(k + 1);
    between(k, n + (last ? 1 : 0));
    multiply();
  }
  if (last) {   // columns of the prompt's last chunk, past-the-end ones zero
    const int64_t col = c_lo + nwhole * H::kCols + csub;
#pragma unroll 1
    for (int t = 0; t * H::kRowsPerLoad < g; ++t) {
      const int row = t * H::kRowsPerLoad + rsub;
      if (row >= g) continue;
      const uint16_t* src = rows + (int64_t)row * ld + col;
      uint4 x = make_uint4(0u, 0u, 0u, 0u);
      if (col + 8 <= c_hi) {
        x = load_nt16(src);
      } else if (col < c_hi) {
        uint16_t h[8];
#pragma unroll
        for (int e = 0; e < 8; ++e) h[e] = (col + e < c_hi) ? src[e] : (uint16_t)0;
        x.x = (uint32_t)h[0] | ((uint32_t)h[1] << 16);
        x.y = (uint32_t)h[2] | ((uint32_t)h[3] << 16);
        x.z = (uint32_t)h[4] | ((uint32_t)h[5] << 16);
        x.w = (uint32_t)h[6] | ((uint32_t)h[7] << 16);
      }
      *put_at(t) = x;
    }
    between(n, n + 1);
    multiply();
  }
}

// Largest magnitude of one row within [c_lo, c_hi), as bf16 bits, in every lane.
__device__ __forceinline__ uint32_t row_magnitude(const uint16_t* __restrict__ row, int64_t c_lo,
                                                  int64_t c_hi, int lane) {
  uint32_t m = 0;
  for (int64_t c = c_lo + lane; c < c_hi; c += kWave) {
    const uint32_t h = row[c] & 0x7fffu;
    m = h > m ? h : m;
  }
#pragma unroll
  for (int o = 1; o < kWave; o <<= 1) {
    const uint32_t y = (uint32_t)__shfl_xor((int)m, o, kWave);
    m = y > m ? y : m;
  }
  return m;
}

// The slice partial of one workgroup, written to part[tile][256] (tiles
// numbered for KM row blocks, those past the prompt's KS not written) in the
// order of gram_entry(), the waves added in order in fp64, as many tiles at a
// time as the stage holds.  Part is double, or float where a caller's buffer
// has room for no more.  With `rescale`, a
// slice in which fp32 products could overflow or vanish (a row that is not
// all zero and whose sum of squares is below 2^-80, above 2^120 or not finite) is
// passed over again with every row divided by a power of two that brings its
// largest magnitude into [1, 2); gex[16 KM] is then 1 and gex[0 .. 16 KM) holds
// the exponents (gex[16 KM] is 0 otherwise), and a row that holds an infinity
// or NaN raises PAIR_ST_NONFINITE.
template <int KM, int KS, class Part, class Between>
__device__ __forceinline__ void gram_slice(const uint16_t* __restrict__ rows, int64_t ld, int g,
                                           int64_t c_lo, int64_t c_hi, uint16_t* stage_all,
                                           int32_t* ex, bool rescale, Part* __restrict__ part,
                                           int32_t* __restrict__ gex, int32_t* d_status,
                                           Between&& between) {
  constexpr bool HALF = KM <= 2;
  using H = GramShape<KS, HALF>;
  // Tiles whose wave sums fit the stage together.
  constexpr int kFit = H::kLdsElems * (int)sizeof(uint16_t) / (kGramWaves * 256 * (int)sizeof(double));
  constexpr int kRounds = (H::kTiles + kFit - 1) / kFit;
  constexpr int kSumTiles = (H::kTiles + kRounds - 1) / kRounds;
  const int tid = threadIdx.x, lane = tid & (kWave - 1);
  const int wave = __builtin_amdgcn_readfirstlane(tid / kWave);
  uint16_t* stage = stage_all + wave * H::kWaveElems;
  double* sums = reinterpret_cast<double*>(stage_all);   // [wave][tile][256], after the last chunk
  double tot[H::kTiles];
  // One pass over the columns and its sums, in tot.  The scaled one, which hardly
  // any slice needs, is a copy of its own: in one with the first it cost
  // registers (the audit of 128 prompts of 64, D = 65536, R = 500: 356 us against 255).
  auto pass = [&](auto scaled) {
    GramAcc<KS, HALF> acc;
#pragma unroll
    for (int i = 0; i < H::kTiles; ++i) {
      acc.f[i] = f32x4_t{0.0f, 0.0f, 0.0f, 0.0f};
#pragma unroll
      for (int v = 0; v < 4; ++v) acc.d[i][v] = 0.0;
    }
    gram_pass<KS, HALF, decltype(scaled)::value>(rows, ld, g, c_lo, c_hi, stage, wave, lane, ex, acc,
                                                 between);
#pragma unroll
    for (int i0 = 0; i0 < H::kTiles; i0 += kSumTiles) {
      __syncthreads();   // every wave is done with the stage, or with the last tiles' sums
#pragma unroll
      for (int i = i0; i < i0 + kSumTiles && i < H::kTiles; ++i)
#pragma unroll
        for (int v = 0; v < 4; ++v)
          sums[(wave * kSumTiles + i - i0) * 256 + 4 * lane + v] = acc.d[i][v];
      __syncthreads();
#pragma unroll
      for (int i = i0; i < i0 + kSumTiles && i < H::kTiles; ++i) {
        double s = 0.0;
#pragma unroll
        for (int w = 0; w < kGramWaves; ++w) s += sums[(w * kSumTiles + i - i0) * 256 + tid];
        tot[i] = s;
      }
    }
  };
  // Some row's products may leave fp32's range: this thread's entry of every tile is
  // (er, ec); the diagonal judges the rows (a row of zeros is looked through
  // before it costs a second pass).
  auto out_of_range = [&]() -> bool {
    bool odd = false;
    const int er = 4 * (tid >> 6) + (tid & 3), ec = (tid >> 2) & 15;
#pragma unroll
    for (int a = 0; a < KS; ++a) {
      const double d = tot[gram_tile(KS, a, a)];
      const bool o = !(d >= 0x1p-80 && d <= 0x1p120) && 16 * a + er < g;
      if (er == ec) {
        ex[16 * a + er] = o ? 1 : 0;
        odd = odd || o;
      }
    }
    if (!__syncthreads_or(odd ? 1 : 0)) return false;
    bool some = false;
    for (int row = wave; row < g; row += kGramWaves)
      if (ex[row] != 0)
        some = some || row_magnitude(rows + (int64_t)row * ld, c_lo, c_hi, lane) != 0u;
    return __syncthreads_or(some ? 1 : 0) != 0;
  };
  pass(std::false_type{});
  const bool again = rescale && out_of_range();
  if (again) {
    for (int row = wave; row < H::KP; row += kGramWaves) {
      const uint32_t m = row < g ? row_magnitude(rows + (int64_t)row * ld, c_lo, c_hi, lane) : 0u;
      if (lane == 0) {
        if (m >= 0x7f80u) raise_status(d_status, PAIR_ST_NONFINITE);
        ex[row] = (m == 0u || m >= 0x7f80u) ? 0 : (int32_t)(m >> 7) - 127;
      }
    }
    __syncthreads();
    pass(std::true_type{});
  }
#pragma unroll
  for (int a = 0; a < KS; ++a)
#pragma unroll
    for (int c = a; c < KS; ++c)
      part[gram_tile(KM, a, c) * 256 + tid] = (Part)tot[gram_tile(KS, a, c)];
  if (rescale) {
    if (tid == 0) gex[16 * KM] = again ? 1 : 0;
    if (again && tid < H::KP) gex[tid] = ex[tid];
  }
}

// LDS for any shape up to KM row blocks.
constexpr int gram_lds_elems(int km) {
  return km == 1 ? GramShape<1, true>::kLdsElems
                 : (km == 2 ? GramShape<2, true>::kLdsElems
                            : (km == 3 ? GramShape<2, false>::kLdsElems
                                       : GramShape<4, false>::kLdsElems));
}

// gram_slice in the shape of the prompt's group size.
template <int KM, class Part, class Between>
__device__ __forceinline__ void gram_slice_of(const uint16_t* __restrict__ rows, int64_t ld, int g,
                                              int64_t c_lo, int64_t c_hi, uint16_t* stage,
                                              int32_t* ex, bool rescale, Part* __restrict__ part,
                                              int32_t* __restrict__ gex, int32_t* d_status,
                                              Between&& between) {
  if (KM == 1 || g <= 16)
    gram_slice<KM, 1>(rows, ld, g, c_lo, c_hi, stage, ex, rescale, part, gex, d_status, between);
  else if (KM == 2 || g <= 32)
    gram_slice<KM, (KM < 2 ? KM : 2)>(rows, ld, g, c_lo, c_hi, stage, ex, rescale, part, gex,
                                      d_status, between);
  else if (KM == 3 || g <= 48)
    gram_slice<KM, (KM < 3 ? KM : 3)>(rows, ld, g, c_lo, c_hi, stage, ex, rescale, part, gex,
                                      d_status, between);
  else
    gram_slice<KM, (KM < 4 ? KM : 4)>(rows, ld, g, c_lo, c_hi, stage, ex, rescale, part, gex,
                                      d_status, between);
}

}  // namespace pair
