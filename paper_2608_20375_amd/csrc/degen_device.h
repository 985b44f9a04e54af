// degen_device.h -- representation degeneration of the SABA decoding state (Sec.
// "State-Aware Budget Allocation", degen_t): the cosine similarity
//   r_d = <h_d, h_{d+1}> / (|h_d| |h_{d+1}|)
// of the drafter's hidden states at adjacent draft positions d, d + 1 of a
// sequence (0 when either state is the zero vector).  The budget stage turns
// them into degen = mean_d r_d + (r_{L-1} - r_1).
//
// One workgroup per (sequence, run of up to kPairs adjacent pairs), as extra
// workgroups of the logits pass's grid: they need nothing of it and fill the CUs
// that its last rows leave idle, where a kernel of their own cost its launch and
// 4 to 5 us (rounds with H = 4096: 16 sequences 47.3 -> 41.9 us, 64 75.2 ->
// 70.7, 128 257 -> 245).  A workgroup reads
// the kPairs + 1 hidden rows of its run once, 16 bytes a load, every load of a
// lane issued before any arithmetic; each lane keeps fp32 partial sums of the
// rows' squared norms and of the adjacent products over the vectors it owns; the
// partials are summed in fp64 across the wave (DPP) and across the waves (LDS).
#pragma once

#include "graft_internal.h"

namespace graft {

struct DegenArgs {
  unsigned first;            // first workgroup of the grid that takes a run
  const uint16_t *hidden;    // [B, L, H] bf16 bits
  int L, H, runs;            // runs per sequence
  float *adj_cos, *adj_cos_out;
};

constexpr int kDegenPairs = 4;                        // adjacent pairs per workgroup
constexpr int kDegenRows = kDegenPairs + 1;
constexpr int kDegenAcc = kDegenRows + kDegenPairs;   // norms, then adjacent products

// v > 0 for any bits, also in a file compiled without regard for NaNs.
__device__ __forceinline__ bool positive_f64(double v) {
  const long long b = __double_as_longlong(v);
  return b > 0 && b <= 0x7FF0000000000000ll;
}

// Run blk of a workgroup of W waves.
template <int W>
__device__ __forceinline__ void degen_run(const DegenArgs &a, int blk, double (*s_part)[kDegenAcc]) {
  typedef unsigned int u32x4 __attribute__((ext_vector_type(4)));
  constexpr int kThreads = W * kWave;
  constexpr int kVec = W <= 4 ? 2 : 1;                // 16-byte vectors per row per lane per step
  const int b = blk / a.runs;
  const int d0 = (blk % a.runs) * kDegenPairs;
  const int np = (a.L - 1 - d0) < kDegenPairs ? (a.L - 1 - d0) : kDegenPairs;   // pairs, >= 1
  const int nr = np + 1;
  const int tid = threadIdx.x, lane = lane_id(), wave = tid / kWave;
  const int64_t nv = a.H / 8;                                                   // vectors per row
  const u32x4 *base =
      reinterpret_cast<const u32x4 *>(a.hidden + (static_cast<int64_t>(b) * a.L + d0) * a.H);

  float acc[kDegenAcc];
#pragma unroll
  for (int k = 0; k < kDegenAcc; ++k) acc[k] = 0.f;
  for (int64_t v0 = 0; v0 < nv; v0 += kVec * kThreads) {
    u32x4 q[kVec][kDegenRows];
#pragma unroll
    for (int u = 0; u < kVec; ++u) {
      const int64_t v = v0 + u * kThreads + tid;
#pragma unroll
      for (int r = 0; r < kDegenRows; ++r) {
        q[u][r] = u32x4{0u, 0u, 0u, 0u};
        if (r < nr && v < nv) q[u][r] = __builtin_nontemporal_load(base + r * nv + v);
      }
    }
#pragma unroll
    for (int u = 0; u < kVec; ++u) {
#pragma unroll
      for (int e = 0; e < 8; ++e) {
        float x[kDegenRows];
#pragma unroll
        for (int r = 0; r < kDegenRows; ++r)
          x[r] = __uint_as_float(e & 1 ? q[u][r][e / 2] & 0xFFFF0000u : q[u][r][e / 2] << 16);
#pragma unroll
        for (int r = 0; r < kDegenRows; ++r) acc[r] = __builtin_fmaf(x[r], x[r], acc[r]);
#pragma unroll
        for (int p = 0; p < kDegenPairs; ++p)
          acc[kDegenRows + p] = __builtin_fmaf(x[p], x[p + 1], acc[kDegenRows + p]);
      }
    }
  }
  // rows past the run were loaded as zeros, so their sums are 0
#pragma unroll
  for (int k = 0; k < kDegenAcc; ++k) {
    double s = static_cast<double>(acc[k]);
#pragma unroll
    for (int o = 1; o < kWave; o <<= 1) s += xor_lane_f64(s, o);
    if (lane == 0) s_part[wave][k] = s;
  }
  __syncthreads();
  if (tid < np) {
    double n0 = 0.0, n1 = 0.0, dot = 0.0;
#pragma unroll
    for (int w = 0; w < W; ++w) {
      n0 += s_part[w][tid];
      n1 += s_part[w][tid + 1];
      dot += s_part[w][kDegenRows + tid];
    }
    const double r = positive_f64(n0) && positive_f64(n1) ? dot / sqrt(n0 * n1) : 0.0;
    const int64_t o = static_cast<int64_t>(b) * (a.L - 1) + d0 + tid;
    a.adj_cos[o] = static_cast<float>(r);
    if (a.adj_cos_out) a.adj_cos_out[o] = static_cast<float>(r);
  }
}

}  // namespace graft
