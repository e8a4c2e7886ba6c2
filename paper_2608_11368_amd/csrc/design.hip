// Design draw: independent Bernoulli continuation indicators and the logged
// joint inclusion probabilities (paper Sec. 3.3; the design draw of Algorithm
// 1, new for every step; rho_ij must be logged before rewards, Theorem 2).
//
// Vertex i of prompt b in replicate r is drawn from word i & 3 of
// Philox4x64-10 at counter (r, b, i >> 2, 0).
//
// design_kernel is bound by the generator's 64-bit products, so no lane repeats one: an item is one
// (replicate, quad of four vertices), a generator block.  A workgroup owns
// kPrompts consecutive prompts and rc replicates.  The prompts' quads are
// listed in LDS with their thresholds and the products that depend on the
// quad alone, the replicates with those that depend on the replicate alone
// (16 of 20 products are left per item), and the items run over
// (replicate, listed quad), so that lanes are full whatever the group sizes.
// A quad's four mask bytes are one (unaligned) store, and consecutive lanes
// write consecutive bytes of a replicate's row; counts gather in LDS and leave as runs
// of kPrompts integers.  The rho block goes to workgroups of its own ahead of the
// drawing ones in the same launch.
//
// design_wave_kernel, one wave per (replicate, prompt) with lane i = vertex
// i, evaluates each block in four lanes and writes the rho block with replicate 0's
// wave, but has no barrier: a small launch, where only that chain counts, is 1 us shorter.
// us for (B, G, R), wave against design_kernel: (128, 16, 1) 4.0 / 5.0,
// (128, 16, 64) 7.2 / 5.5, (512, 2..8, 8) 5.2 / 5.6, (512, 2..8, 16) 6.6 / 5.6,
// (512, 2..64, 1) 14.8 / 6.9, (512, 2..64, 1000) 231 / 48, (512, 64, 1024) 235 / 63.
// Without a rho block (512, 2..64, 1) 5.6 / 7.7, (512, 64, 8) 7.3 / 7.7,
// (64, 30..40, 64) 7.3 / 7.8, (512, 2..64, 64) 22.7 / 12.0.
// So it takes launches of at most kWaveUnits waves with gmax <= 16 (a rho
// block of at most four passes) or without a rho block.
#include "common.hpp"
#include "launch.hpp"

namespace pair {

namespace {

constexpr int64_t kWaveUnits = 4096;

__global__ __launch_bounds__(256) void design_wave_kernel(
    int64_t B, int64_t nv, int32_t gmax, const int64_t* __restrict__ offsets,
    const float* __restrict__ p, uint64_t seed, int64_t rep0, int64_t R, uint8_t* __restrict__ mask,
    float* __restrict__ pi, int32_t* __restrict__ edge_count, int32_t* __restrict__ completed,
    int32_t* d_status) {
  const int lane = threadIdx.x & (kWave - 1);
  const int64_t units = B * R;
  const int64_t waves_total = (int64_t)gridDim.x * (blockDim.x / kWave);
  const bool draws = mask != nullptr || edge_count != nullptr || completed != nullptr;
  for (int64_t u = (int64_t)blockIdx.x * (blockDim.x / kWave) + threadIdx.x / kWave; u < units;
       u += waves_total) {
    const int64_t r = u / B;  // replicate-major: consecutive waves share r
    const int64_t b = u - r * B;
    int64_t o0, g;
    const bool ok = prompt_bounds(offsets, b, nv, 2, gmax, &o0, &g, d_status, r == 0);
    const bool active = ok && lane < g;
    const float pv = active ? p[o0 + lane] : 1.0f;
    if (r == 0 && pi != nullptr) {
      // Logged rho block: fl32(p_i p_j) off the diagonal, p_i on it, zero
      // outside the G_b x G_b corner (all zero for a malformed prompt).
      // Whole-wave iterations so that every lane takes part in the shuffles
      // of p; only the store is guarded.
      float* blk = pi + b * (int64_t)gmax * gmax;
      for (int base = 0; base < gmax * gmax; base += kWave) {
        const int idx = base + lane;
        const int i = idx / gmax, j = idx - i * gmax;
        const float pa = __shfl(pv, i < kWave ? i : 0, kWave);
        const float pb = __shfl(pv, j, kWave);
        float v = 0.0f;
        if (ok && i < g && j < g) v = (i == j) ? pa : pa * pb;
        if (idx < gmax * gmax) blk[idx] = v;
      }
    }
    if (!ok || !draws) continue;
    int J = 0;
    if (active) {
      const Philox4x64 x = philox4x64_10((uint64_t)(rep0 + r), (uint64_t)b, (uint64_t)(lane >> 2),
                                         0ull, seed, 0ull);
      const uint64_t u32 = philox_word(x, lane & 3) >> 32;
      if (p_in_range(pv)) {
        J = u32 < inclusion_threshold(pv) ? 1 : 0;
      } else if (r == 0) {
        raise_status(d_status, PAIR_ST_P_RANGE);
      }
      if (mask != nullptr) mask[r * nv + o0 + lane] = (uint8_t)J;
    }
    const uint64_t bits = __ballot(J != 0);
    if (lane == 0) {
      const int32_t k = (int32_t)__popcll(bits);
      if (completed != nullptr) completed[r * B + b] = k;
      if (edge_count != nullptr) edge_count[r * B + b] = k * (k - 1) / 2;
    }
  }
}

constexpr int kPrompts = 16;
constexpr int kThreads = 256;
constexpr int kQuads = kPrompts * 16;   // 16 quads per prompt at most
constexpr int kMaxReps = 64;            // most replicates of a workgroup

struct alignas(16) QuadThr {
  uint32_t last[4];   // the largest draw that includes the vertex
};

__global__ __launch_bounds__(kThreads) void design_kernel(
    int64_t B, int64_t nv, int32_t gmax, const int64_t* __restrict__ offsets,
    const float* __restrict__ p, uint64_t seed, int64_t rep0, int64_t R, int32_t rc,
    int64_t pi_blocks, int64_t groups, uint8_t* __restrict__ mask, float* __restrict__ pi,
    int32_t* __restrict__ edge_count, int32_t* __restrict__ completed, int32_t* d_status) {
  __shared__ QuadThr thr[kQuads];
  __shared__ uint64_t qa[kQuads], qb[kQuads], qc[kQuads];   // quad's part of rounds 1 and 2
  __shared__ uint64_t ra[kMaxReps], rb[kMaxReps], rl[kMaxReps];   // the replicate's
  __shared__ int64_t dst[kQuads];       // first vertex of the quad, in packed rows
  __shared__ uint32_t code[kQuads];     // prompt << 16 | drawable vertices << 8 | vertices
  __shared__ float pl[kWave];
  __shared__ int64_t first[kPrompts];
  __shared__ int size[kPrompts];        // -1: malformed, or past the batch
  __shared__ int cnt[kMaxReps][kPrompts];
  const int tid = threadIdx.x;

  if (blockIdx.x < pi_blocks) {
    // Logged rho block: fl32(p_i p_j) off the diagonal, p_i on it, zero
    // outside the G_b x G_b corner (all zero for a malformed prompt).
    for (int64_t b = blockIdx.x; b < B; b += pi_blocks) {
      int64_t o0, g;
      prompt_bounds(offsets, b, nv, 2, gmax, &o0, &g, d_status, tid == 0);
      if (tid < kWave) pl[tid] = tid < g ? p[o0 + tid] : 0.0f;
      __syncthreads();
      float* blk = pi + b * (int64_t)gmax * gmax;
      for (int idx = tid; idx < gmax * gmax; idx += kThreads) {
        const int i = idx / gmax, j = idx - i * gmax;
        float v = 0.0f;
        if (i < g && j < g) v = (i == j) ? pl[i] : pl[i] * pl[j];
        blk[idx] = v;
      }
      __syncthreads();
    }
    return;
  }

  const bool count = edge_count != nullptr || completed != nullptr;
  const int64_t units = groups * ((R + rc - 1) / rc);
  for (int64_t unit = blockIdx.x - pi_blocks; unit < units; unit += gridDim.x - pi_blocks) {
    const int64_t chunk = unit / groups;
    const int64_t b0 = (unit - chunk * groups) * kPrompts;
    const int np = (int)(B - b0 < kPrompts ? B - b0 : kPrompts);
    const int64_t r0 = chunk * rc;
    const int nr = (int)(R - r0 < rc ? R - r0 : rc);
    if (tid < kPrompts) {
      int64_t o0 = 0, g = 0;
      const bool ok =
          tid < np && prompt_bounds(offsets, b0 + tid, nv, 2, gmax, &o0, &g, d_status, chunk == 0);
      first[tid] = o0;
      size[tid] = ok ? (int)g : -1;
    } else if (tid >= kWave && tid < kWave + nr) {
      const PhiloxRep pr = philox_rep((uint64_t)(rep0 + r0 + tid - kWave));
      ra[tid - kWave] = pr.hi1;
      rb[tid - kWave] = pr.lo1;
      rl[tid - kWave] = pr.lo0;
    }
    for (int i = tid; i < rc * kPrompts; i += kThreads) (&cnt[0][0])[i] = 0;
    __syncthreads();
    // Every thread is one (prompt, quad) slot; the quads that exist are listed
    // in order, a prompt's behind those of the prompts before it.
    int nq = 0;
    {
      const int bp = tid >> 4, q = tid & 15;
      int at = q;
#pragma unroll
      for (int w = 0; w < kPrompts; ++w) {
        const int c = size[w] < 0 ? 0 : (size[w] + 3) >> 2;
        at += w < bp ? c : 0;
        nq += c;
      }
      const int g = size[bp];
      if (4 * q < g) {
        const int n = g - 4 * q < 4 ? g - 4 * q : 4;
        uint32_t live = 0;
#pragma unroll
        for (int e = 0; e < 4; ++e) {
          const float pv = e < n ? p[first[bp] + 4 * q + e] : 1.0f;
          const uint64_t t = p_in_range(pv) ? inclusion_threshold(pv) : 0ull;
          thr[at].last[e] = (uint32_t)(t - 1ull);
          live |= (e < n && t != 0ull) ? 1u << e : 0u;
          if (!p_in_range(pv) && chunk == 0) raise_status(d_status, PAIR_ST_P_RANGE);
        }
        const PhiloxQuad pq = philox_quad_part((uint64_t)(b0 + bp), (uint64_t)q, seed);
        qa[at] = pq.c0;
        qb[at] = pq.c2;
        qc[at] = pq.c3;
        dst[at] = first[bp] + 4 * q;
        code[at] = (uint32_t)bp << 16 | live << 8 | (uint32_t)n;
      }
    }
    __syncthreads();

    if (nq > 0) {
      const int dr = kThreads / nq, dq = kThreads - dr * nq;
      int r = tid / nq, q = tid - r * nq;
      while (r < nr) {
        const uint32_t cd = code[q];
        const QuadThr t = thr[q];
        const Philox4x64 x = philox_rounds_3_10(ra[r] ^ qa[q], rb[r], qb[q] ^ rl[r], qc[q], seed);
        uint32_t bits = 0;
#pragma unroll
        for (int e = 0; e < 4; ++e)
          bits |= (uint32_t)(x.w[e] >> 32) <= t.last[e] ? 1u << e : 0u;
        bits &= cd >> 8;
        if (mask != nullptr) {
          uint8_t* m = mask + (r0 + r) * nv + dst[q];
          const int n = (int)(cd & 0xffu);
          const uint32_t bytes =
              (bits & 1u) | (bits & 2u) << 7 | (bits & 4u) << 14 | (bits & 8u) << 21;
          if (n == 4) {
            __builtin_memcpy(m, &bytes, 4);
          } else {
            for (int e = 0; e < n; ++e) m[e] = (uint8_t)(bytes >> (8 * e));
          }
        }
        if (count) atomicAdd(&cnt[r][cd >> 16], (int)__popc(bits));
        r += dr;
        q += dq;
        if (q >= nq) {
          q -= nq;
          ++r;
        }
      }
    }
    __syncthreads();
    if (count) {
      for (int i = tid; i < nr * kPrompts; i += kThreads) {
        const int r = i / kPrompts, w = i - r * kPrompts;
        if (size[w] < 0) continue;
        const int k = cnt[r][w];
        if (completed != nullptr) completed[(r0 + r) * B + b0 + w] = k;
        if (edge_count != nullptr) edge_count[(r0 + r) * B + b0 + w] = k * (k - 1) / 2;
      }
    }
    __syncthreads();   // the tables are rebuilt for the next unit
  }
}

}  // namespace

int launch_design(int64_t B, int64_t nv, int32_t gmax, const int64_t* offsets, const float* p,
                  uint64_t seed, int64_t rep0, int64_t R, uint8_t* mask, float* pi,
                  int32_t* edge_count, int32_t* completed, int32_t* d_status, hipStream_t stream) {
  const bool draws = mask != nullptr || edge_count != nullptr || completed != nullptr;
  if (!draws && pi == nullptr) return PAIR_OK;
  if ((gmax <= 16 || pi == nullptr) && B <= kWaveUnits && (!draws || R <= kWaveUnits / B)) {
    const int64_t waves = draws ? B * R : B;   // the rho block needs replicate 0 only
    hipLaunchKernelGGL(design_wave_kernel, dim3((unsigned)((waves + 3) / 4)), dim3(256), 0, stream,
                       B, nv, gmax, offsets, p, seed, rep0, draws ? R : 1, mask, pi, edge_count,
                       completed, d_status);
    return hipGetLastError() == hipSuccess ? PAIR_OK : PAIR_EHIP;
  }
  const int64_t groups = (B + kPrompts - 1) / kPrompts;
  // Replicates per workgroup: few while workgroups are fewer than CUs, then
  // enough that a workgroup has an item per thread, then as many as keep the
  // launch within 8 workgroups per CU (the waves that run at once).  Longer
  // launches loop: 64 workgroups per CU and 16 for the rho block at most.
  const int64_t cus = device_cu_count();
  const int64_t quads = nv / (4 * groups);
  int32_t rc = 1;
  for (; rc < kMaxReps; rc *= 2) {
    const int64_t wgs = groups * ((R + rc - 1) / rc);
    if (wgs <= 8 * cus && (wgs <= cus || rc * quads >= kThreads)) break;
  }
  const int64_t units = draws ? groups * ((R + rc - 1) / rc) : 0;
  const int64_t pi_blocks = pi == nullptr ? 0 : (B < 16 * cus ? B : 16 * cus);
  const int64_t grid = pi_blocks + (units < 64 * cus ? units : 64 * cus);
  hipLaunchKernelGGL(design_kernel, dim3((unsigned)grid), dim3(kThreads), 0, stream, B, nv, gmax,
                     offsets, p, seed, rep0, R, rc, pi_blocks, groups, mask, pi, edge_count,
                     completed, d_status);
  return hipGetLastError() == hipSuccess ? PAIR_OK : PAIR_EHIP;
}

}  // namespace pair
