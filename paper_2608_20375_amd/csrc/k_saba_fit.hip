// k_saba_fit.hip -- SABA's gain and cost models fitted on a same-prefix
// budget-replay log (the paper's SABA section, eqs. saba-gain and saba-cost,
// fitted on held-out replays as its experimental setup describes).
//
// fit_kernel: one evaluation of the log per launch, with the Levenberg-Marquardt
// step in between on the device, so that a fit is a queue of launches with no
// host round trip.  Launch i
//   - adds launch i-1's block sums in a fixed order (every block, for itself) and
//     takes the step from them: accept or reject the trial, damp, solve the 4 x 4
//     system; at launch 1 also the 3 x 3 normal equations of the cost.  Every
//     block computes the same state; block 0 stores it for launch i+1;
//   - evaluates the log at the new trial: for every round G_j = 1 -
//     exp(-B_j / tau) with tau = max(phi . [1, s], tau_min), the round's best
//     scale A = sum_j a_j G_j / sum_j G_j^2, the residuals r_j = A G_j - a_j and
//     their derivatives by phi at that A (the gradient of the objective with A
//     eliminated), J_j = d_j [1, s], d_j = -A exp(-B_j / tau) B_j / tau^2 (0 when
//     tau is clamped), into the sum of squares, J^T J and J^T r.  Launch 0 adds
//     X^T X, X^T y and y^T y of the affine cost, X = [1, B, B prefix], launch 1
//     the fitted cost's residual sum of squares (the normal-equation form of it
//     cancels badly).
// Once the steps are done the remaining launches of the queue return at once.
//
// A quad of lanes takes one round, a lane every fourth budget: the five sums over
// budgets are two DPP steps each, and since a round's J^T J and J^T r are its
// scalars sum d^2 and sum d r times products of [1, s], each lane keeps four of
// the 15 sums.  Latency-bound: 20000 rounds of 31 budgets are 2.5 MB and about
// 0.1 GFLOP of fp64 an evaluation; a launch takes 8.7 us, of it 1.7 for the last
// launch's sums, 1.4 for the step, 2.7 for the rounds and 1.4 for the block's
// sums.  One wave a round with 25 sums a lane, a reducing kernel and the step on
// the host took 18.9 + 5.2 us and a round trip: that fit 3407 us, this one 890.
// (Rows of 16 lanes a round: 9.0 us a launch; blocks of four waves: 10.2.)
// With 33 to 64 budgets the first two launches spill registers, once a fit:
// 20000 rounds of 33, 48 and 64 budgets 8.6, 6.1 and 3.5 ms -> 2.3, 1.8 and 1.1.
#include <type_traits>

#include "graft_internal.h"

namespace graft {
namespace {

constexpr int kFitWaves = 8;
constexpr int kFitThreads = kFitWaves * kWave;
constexpr int kQuad = 4;                                   // lanes of a round
constexpr int kFitRounds = kFitThreads / kQuad;            // rounds a block takes at a time
constexpr int kSumLanes = kFitThreads / 32;               // sums a block adds at a time
constexpr int kGainSums = 15;                              // the others belong to the cost

struct FitArgs {
  int T, nb, max_iter;
  const float *state;       // [T, 3]
  const int32_t *prefix;    // [T]
  const float *accepted;    // [T, nb]
  const float *latency;     // [T, nb]
  double tau_min;
  double phi0[4];
  double *partial;          // [2][kFitSums][kFitMaxBlocks]
  FitState *slot;           // [2]
  int32_t budgets[kMaxGrid];
};

// Sum over a quad of lanes, in every lane of it (DPP steps).
__device__ __forceinline__ double quad_sum_f64(double v) {
  v += xor_lane_f64(v, 1);
  v += xor_lane_f64(v, 2);
  return v;
}

// Solves the N x N system M x = r by Gaussian elimination with partial pivoting;
// false when a pivot is not positive enough.  Fully unrolled: rows are swapped
// by selects, so everything stays in registers.  PLAIN: every operation rounded by
// itself and true divisions, so that a system of whole numbers whose columns are
// multiples of each other cancels to a zero pivot (with products by a reciprocal,
// or fused, a tiny one is left, and an x of 1e15); otherwise one division a pivot,
// since the step's chain is all latency.
template <int N, bool PLAIN>
__device__ __forceinline__ bool solve_small(double (&M)[N][N], double (&r)[N], double (&x)[N]) {
#pragma clang fp contract(off)
  bool ok = true;
  double inv[N];
#pragma unroll
  for (int c = 0; c < N; ++c) {
    double best = fabs(M[c][c]);
    int p = c;
#pragma unroll
    for (int i = c + 1; i < N; ++i) {
      const double v = fabs(M[i][c]);
      if (v > best) {
        best = v;
        p = i;
      }
    }
    ok = ok && best > 1e-300;
#pragma unroll
    for (int i = c + 1; i < N; ++i) {
      const bool sw = p == i;
#pragma unroll
      for (int j = 0; j < N; ++j) {
        const double a = M[c][j], b = M[i][j];
        M[c][j] = sw ? b : a;
        M[i][j] = sw ? a : b;
      }
      const double a = r[c], b = r[i];
      r[c] = sw ? b : a;
      r[i] = sw ? a : b;
    }
    if (!PLAIN) inv[c] = 1.0 / M[c][c];
#pragma unroll
    for (int i = c + 1; i < N; ++i) {
      const double f = PLAIN ? M[i][c] / M[c][c] : M[i][c] * inv[c];
#pragma unroll
      for (int j = c + 1; j < N; ++j) M[i][j] = PLAIN ? M[i][j] - f * M[c][j] : fma(-f, M[c][j], M[i][j]);
      r[i] = PLAIN ? r[i] - f * r[c] : fma(-f, r[c], r[i]);
    }
  }
#pragma unroll
  for (int c = N - 1; c >= 0; --c) {
    double v = r[c];
#pragma unroll
    for (int j = c + 1; j < N; ++j) v = PLAIN ? v - M[c][j] * x[j] : fma(-M[c][j], x[j], v);
    x[c] = PLAIN ? v / M[c][c] : v * inv[c];
    ok = ok && isfinite(x[c]);
  }
  return ok;
}

// Takes over the point the sums belong to.
__device__ __forceinline__ void adopt(FitState &s, const double *sums) {
  s.F = sums[0];
#pragma unroll
  for (int k = 0; k < 10; ++k) s.H[k] = sums[1 + k];
#pragma unroll
  for (int k = 0; k < 4; ++k) s.g[k] = sums[11 + k];
}

// The step after launch i-1's evaluation (one thread): Levenberg-Marquardt with
// Marquardt's diagonal scaling.
__device__ void fit_step(FitState &s, const double *sums, int i, int max_iter) {
  if (i == 1) {
    double M[3][3], r[3], c[3];
    int k = 15;
#pragma unroll
    for (int p = 0; p < 3; ++p) {
      r[p] = sums[21 + p];
#pragma unroll
      for (int q = p; q < 3; ++q) M[p][q] = M[q][p] = sums[k++];
    }
    s.cost_ok = solve_small<3, true>(M, r, c);
#pragma unroll
    for (int p = 0; p < 3; ++p) s.c[p] = s.cost_ok ? c[p] : 0.0;
    adopt(s, sums);
    s.lam = 1e-3;
  } else {
    if (i == 2) s.cost_sse = s.cost_ok ? sums[24] : 0.0;
    if (s.done) return;
    if (sums[0] < s.F) {
      const bool flat = s.F - sums[0] < 1e-15 * (s.F > 0.0 ? s.F : 1.0);
      double step = 0.0, size = 0.0;
#pragma unroll
      for (int k = 0; k < 4; ++k) {
        const double d = s.d[k];
        s.phi[k] = s.trial[k];
        step += d * d;
        size += s.phi[k] * s.phi[k];
      }
      adopt(s, sums);
      s.lam = s.lam / 10.0 > 1e-15 ? s.lam / 10.0 : 1e-15;
      if (flat || step <= 1e-24 * (1.0 + size)) s.converged = s.done = 1;
    } else {
      s.lam *= 10.0;
      if (s.lam > 1e16) s.converged = s.done = 1;   // no descent left at machine precision
    }
    if (s.done) return;
  }
  if (s.iters >= max_iter) {
    s.done = 1;
    return;
  }
  ++s.iters;
  double A[4][4], b[4], d[4];
  int k = 0;
#pragma unroll
  for (int p = 0; p < 4; ++p) {
    b[p] = -s.g[p];
#pragma unroll
    for (int q = p; q < 4; ++q) A[p][q] = A[q][p] = s.H[k++];
  }
#pragma unroll
  for (int p = 0; p < 4; ++p) A[p][p] += s.lam * (A[p][p] > 1e-300 ? A[p][p] : 1e-300);
  if (!solve_small<4, false>(A, b, d)) {   // singular: every tau clamped, or no data
    s.done = 1;
    return;
  }
#pragma unroll
  for (int p = 0; p < 4; ++p) {
    s.d[p] = d[p];
    s.trial[p] = s.phi[p] + d[p];
  }
}

// One replayed round as a quad of lanes holds it.
static_assert(kSumLanes >= kGainSums && 2 * kSumLanes >= kFitSums && kFitMaxBlocks % 32 == 0,
              "the sums of the last launch in one pass, in two with the cost's");

template <int NB>
struct Round {
  float a[NB], y[NB];
  float s[3];
  int32_t prefix;
};
template <int NB, bool COST>
__device__ __forceinline__ Round<NB> load_round(const FitArgs &a, int t, int l) {
  Round<NB> r;
  const int tc = t < a.T ? t : a.T - 1;
#pragma unroll
  for (int k = 0; k < 3; ++k) r.s[k] = a.state[static_cast<int64_t>(tc) * 3 + k];
  r.prefix = COST ? a.prefix[tc] : 0;
#pragma unroll
  for (int k = 0; k < NB; ++k) {
    const int j = l + k * kQuad < a.nb ? l + k * kQuad : a.nb - 1;
    r.a[k] = a.accepted[static_cast<int64_t>(tc) * a.nb + j];
    r.y[k] = COST ? a.latency[static_cast<int64_t>(tc) * a.nb + j] : 0.f;
  }
  return r;
}

// MODE 1: the cost's normal equations too; 2: its residual sum of squares; 0:
// the gain alone.  NB: budgets a lane holds, 4 NB >= nb.
template <int NB, int MODE>
__global__ void __launch_bounds__(kFitThreads) fit_kernel(FitArgs a, int launch) {
  __shared__ double s_sum[kFitSums];
  __shared__ double s_wave[kFitWaves][2 * 16];
  __shared__ FitState s_st;
  const int tid = threadIdx.x, lane = lane_id(), wave = tid / kWave;
  const int l = lane & (kQuad - 1);
  const double *prev = a.partial + ((launch + 1) & 1) * (kFitSums * kFitMaxBlocks);
  double *mine = a.partial + (launch & 1) * (kFitSums * kFitMaxBlocks);

  // the first round's loads are in flight while the step is taken
  int t = blockIdx.x * kFitRounds + tid / kQuad;
  Round<NB> cur = load_round<NB, MODE != 0>(a, t, l);
  if (launch == 0) {
    if (tid == 0) {
      FitState s{};
      for (int k = 0; k < 4; ++k) s.phi[k] = s.trial[k] = a.phi0[k];
      s_st = s;
    }
  } else {
    // block sums of the last launch, 32 lanes a value, and its state: every load
    // issued before any is used
    const FitState *from = a.slot + ((launch + 1) & 1);
    FitState s;
    if (tid == 0) s = *from;
    const int done = from->done;
    auto block_sums = [&](auto n) {   // sums [0, 16 n)
      constexpr int N = decltype(n)::value, kPer = kFitMaxBlocks / 32;
      double x[N][kPer];
#pragma unroll
      for (int j = 0; j < N; ++j)
#pragma unroll
        for (int i = 0; i < kPer; ++i) {
          const int b = i * 32 + (lane & 31), k = j * kSumLanes + (tid >> 5);
          x[j][i] = prev[(k < kFitSums ? k : 0) * kFitMaxBlocks +
                         (b < static_cast<int>(gridDim.x) ? b : 0)];
        }
#pragma unroll
      for (int j = 0; j < N; ++j) {
        const int k = j * kSumLanes + (tid >> 5);
        double v = 0.0;
#pragma unroll
        for (int i = 0; i < kPer; ++i)
          v += i * 32 + (lane & 31) < static_cast<int>(gridDim.x) ? x[j][i] : 0.0;
        v = quad_sum_f64(v);
        v += xor_lane_f64(v, 4);
        v += xor_lane_f64(v, 8);
        v += xor_lane_f64(v, 16);
        if ((lane & 31) == 0 && k < kFitSums) s_sum[k] = v;
      }
    };
    if (MODE == 0 && launch > 2)
      block_sums(std::integral_constant<int, 1>{});
    else
      block_sums(std::integral_constant<int, 2>{});
    if (done && launch > 2) {   // uniform over the grid
      if (blockIdx.x == 0 && tid == 0) a.slot[launch & 1] = s;
      return;
    }
    __syncthreads();
    if (tid == 0) {
      fit_step(s, s_sum, launch, a.max_iter);
      s_st = s;
    }
  }
  __syncthreads();
  if (blockIdx.x == 0 && tid == 0) a.slot[launch & 1] = s_st;
  if (MODE == 0 && s_st.done) return;

  const double p0 = s_st.trial[0], p1 = s_st.trial[1], p2 = s_st.trial[2], p3 = s_st.trial[3];
  const double c0 = s_st.c[0], c1 = s_st.c[1], c2 = s_st.c[2];
  double B[NB];
  bool on[NB];
  double S1 = 0.0, S2 = 0.0;   // sums of the budgets and their squares
#pragma unroll
  for (int k = 0; k < NB; ++k) {
    on[k] = l + k * kQuad < a.nb;
    B[k] = on[k] ? static_cast<double>(a.budgets[on[k] ? l + k * kQuad : 0]) : 0.0;
    S1 += B[k];
    S2 += B[k] * B[k];
  }
  if (MODE == 1) {
    S1 = quad_sum_f64(S1);
    S2 = quad_sum_f64(S2);
  }
  // sum 4 i + l of a lane: 0 r^2; 1..10 d^2 s_p s_q; 11..14 d r s_p
  constexpr int kP[16] = {0, 0, 0, 0, 0, 1, 1, 1, 2, 2, 3, 0, 1, 2, 3, 0};
  constexpr int kQ[16] = {0, 0, 1, 2, 3, 1, 2, 3, 2, 3, 3, 0, 0, 0, 0, 0};
  int lp[4], lq[4];
#pragma unroll
  for (int i = 0; i < 4; ++i) {
    lp[i] = l == 0 ? kP[4 * i] : l == 1 ? kP[4 * i + 1] : l == 2 ? kP[4 * i + 2] : kP[4 * i + 3];
    lq[i] = l == 0 ? kQ[4 * i] : l == 1 ? kQ[4 * i + 1] : l == 2 ? kQ[4 * i + 2] : kQ[4 * i + 3];
  }
  double acc[4] = {0.0, 0.0, 0.0, 0.0}, acc2[3] = {0.0, 0.0, 0.0};
  const int stride = static_cast<int>(gridDim.x) * kFitRounds;
  for (; t - tid / kQuad < a.T; t += stride) {   // uniform in the block
    const bool real = t < a.T;
    const double s1 = cur.s[0], s2 = cur.s[1], s3 = cur.s[2];
    const double lin = p0 + p1 * s1 + p2 * s2 + p3 * s3;
    const bool free_tau = lin > a.tau_min;
    const double inv = 1.0 / (free_tau ? lin : a.tau_min);
    double e[NB], sag = 0.0, sgg = 0.0;
#pragma unroll
    for (int k = 0; k < NB; ++k) {
      e[k] = on[k] ? exp(-B[k] * inv) : 1.0;
      const double G = 1.0 - e[k];
      sag += static_cast<double>(cur.a[k]) * G;   // G = 0 past the grid
      sgg += G * G;
    }
    sag = quad_sum_f64(sag);
    sgg = quad_sum_f64(sgg);
    const double A = sgg > 0.0 ? sag / sgg : 0.0;
    const double w = free_tau ? -A * inv * inv : 0.0;
    double rr = 0.0, dd = 0.0, dr = 0.0;
#pragma unroll
    for (int k = 0; k < NB; ++k) {
      const double r = on[k] ? A * (1.0 - e[k]) - static_cast<double>(cur.a[k]) : 0.0;
      const double d = w * e[k] * B[k];   // B = 0 past the grid
      rr += r * r;
      dd += d * d;
      dr += d * r;
    }
    rr = quad_sum_f64(rr);
    dd = quad_sum_f64(dd);
    dr = quad_sum_f64(dr);
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      const double sp = lp[i] == 0 ? 1.0 : lp[i] == 1 ? s1 : lp[i] == 2 ? s2 : s3;
      const double sq = lq[i] == 0 ? 1.0 : lq[i] == 1 ? s1 : lq[i] == 2 ? s2 : s3;
      const double x = 4 * i + l == 0 ? rr : 4 * i + l < 11 ? dd : dr;
      if (real) acc[i] += x * sp * sq;
    }
    if (MODE == 2) {
      const double pre = static_cast<double>(cur.prefix);
      double rc = 0.0;
#pragma unroll
      for (int k = 0; k < NB; ++k) {
        const double v = c0 + c1 * B[k] + c2 * B[k] * pre - static_cast<double>(cur.y[k]);
        rc += on[k] ? v * v : 0.0;
      }
      rc = quad_sum_f64(rc);
      if (real && l == 1) acc2[2] += rc;   // sum 9
    } else if (MODE == 1) {
      const double pre = static_cast<double>(cur.prefix);
      double y0 = 0.0, y1 = 0.0, y2 = 0.0;
#pragma unroll
      for (int k = 0; k < NB; ++k) {
        const double v = on[k] ? static_cast<double>(cur.y[k]) : 0.0;
        y0 += v;
        y1 += B[k] * v;
        y2 += v * v;
      }
      y0 = quad_sum_f64(y0);
      y1 = quad_sum_f64(y1);
      y2 = quad_sum_f64(y2);
      // sum 4 i + l: X^T X row by row, X^T y, y^T y
      const double x[12] = {static_cast<double>(a.nb), S1, S1 * pre, S2, S2 * pre, S2 * pre * pre,
                            y0, y1, y1 * pre, y2, 0.0, 0.0};
#pragma unroll
      for (int i = 0; i < 3; ++i) {
        const double v = l == 0 ? x[4 * i] : l == 1 ? x[4 * i + 1] : l == 2 ? x[4 * i + 2] : x[4 * i + 3];
        if (real) acc2[i] += v;
      }
    }
    if (t - tid / kQuad + stride < a.T) cur = load_round<NB, MODE != 0>(a, t + stride, l);
  }
  // the wave's quads, then the block's waves in order
#pragma unroll
  for (int o = kQuad; o < kWave; o <<= 1) {
#pragma unroll
    for (int i = 0; i < 4; ++i) acc[i] += xor_lane_f64(acc[i], o);
    if (MODE != 0) {
#pragma unroll
      for (int i = 0; i < 3; ++i) acc2[i] += xor_lane_f64(acc2[i], o);
    }
  }
  if (lane < kQuad) {
#pragma unroll
    for (int i = 0; i < 4; ++i) s_wave[wave][4 * i + l] = acc[i];
#pragma unroll
    for (int i = 0; i < 3; ++i) s_wave[wave][16 + 4 * i + l] = acc2[i];
  }
  __syncthreads();
  if (tid != kGainSums && tid < 16 + kFitSums - kGainSums) {
    const int k = tid < kGainSums ? tid : kGainSums + tid - 16;
    double v = 0.0;
#pragma unroll
    for (int w = 0; w < kFitWaves; ++w) v += s_wave[w][tid];
    if (k < kGainSums || MODE != 0) mine[k * kFitMaxBlocks + blockIdx.x] = v;
  }
}

template <int NB>
hipError_t launch_nb(const FitArgs &a, int blocks, int launch, hipStream_t stream) {
  const dim3 g(blocks), b(kFitThreads);
  if (launch == 0) hipLaunchKernelGGL((fit_kernel<NB, 1>), g, b, 0, stream, a, launch);
  else if (launch == 1) hipLaunchKernelGGL((fit_kernel<NB, 2>), g, b, 0, stream, a, launch);
  else hipLaunchKernelGGL((fit_kernel<NB, 0>), g, b, 0, stream, a, launch);
  return hipGetLastError();
}

}  // namespace

int64_t saba_fit_bytes() {
  return 2 * kFitSums * kFitMaxBlocks * static_cast<int64_t>(sizeof(double)) +
         2 * static_cast<int64_t>(sizeof(FitState));
}

hipError_t launch_saba_fit(const graft_saba_replay *log, const float *phi_init, int max_iter,
                           void *work, int launch, FitState **state, hipStream_t stream) {
  FitArgs a;
  a.T = log->n_rounds;
  a.nb = log->n_budgets;
  a.max_iter = max_iter;
  a.state = log->state;
  a.prefix = log->prefix;
  a.accepted = log->accepted;
  a.latency = log->latency;
  a.tau_min = log->tau_min;
  for (int k = 0; k < 4; ++k) a.phi0[k] = phi_init[k];
  a.partial = static_cast<double *>(work);
  a.slot = reinterpret_cast<FitState *>(a.partial + 2 * kFitSums * kFitMaxBlocks);
  for (int j = 0; j < kMaxGrid; ++j) a.budgets[j] = j < a.nb ? log->budgets[j] : 0;
  *state = a.slot + (launch & 1);
  // as few passes of the whole grid as kFitMaxBlocks allows, evenly filled
  const int passes = (a.T + kFitRounds * kFitMaxBlocks - 1) / (kFitRounds * kFitMaxBlocks);
  const int blocks = (a.T + kFitRounds * passes - 1) / (kFitRounds * passes);
  if (a.nb <= 4 * kQuad) return launch_nb<4>(a, blocks, launch, stream);
  if (a.nb <= 8 * kQuad) return launch_nb<8>(a, blocks, launch, stream);
  return launch_nb<16>(a, blocks, launch, stream);
}

}  // namespace graft
