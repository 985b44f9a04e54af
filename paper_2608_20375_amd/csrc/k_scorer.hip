// k_scorer.hip -- TDES edge scoring (Sec. "Target-Distilled Edge Scoring").
//
// projection_kernel: the cached projections g_p(e) = e^T G_p and g_c(e) =
//   e^T G_c of every vocabulary token, computed once per scorer; the paper notes
//   they depend only on the token id.  fp64 accumulation, fp32 storage.
// edge_kernel: for one (sequence, depth) it gathers the projections of the K
//   children and of the parents (the root token at depth 1, else the K
//   candidates of the previous depth) into LDS, forms every parent-child dot
//   product (eq. tdes-bitower), centers over the children of each parent when
//   asked (eq. tdes-center) and adds log q of the child (eq. tdes-score).
//   Selection's copy of the scores is indexed by token-id rank: row (depth,
//   rank of the parent's id) holds the K children in the order of their ids,
//   so selection appends a parent's children in canonical order by filtering
//   the row against its threshold, with no ranking; the exported table keeps
//   the candidates' logit-rank order.
// The K x m x K contraction of a (sequence, depth), at most 64 x 64 x 64, runs
// on fp32 matrix cores in 16 x 16 tiles (edge_tiles); the depth-1 block of
// each sequence also computes its SABA budget.
#include <type_traits>

#include "graft_internal.h"
#include "edge_mfma.h"
#include "saba_device.h"

namespace graft {
namespace {

__global__ void __launch_bounds__(256)
projection_kernel(const float *__restrict__ emb, const float *__restrict__ gp,
                  const float *__restrict__ gc, int64_t V, int E, int m,
                  float *__restrict__ P, float *__restrict__ Q) {
  const int64_t idx = static_cast<int64_t>(blockIdx.x) * blockDim.x + threadIdx.x;
  if (idx >= V * m) return;
  const int64_t v = idx / m;
  const int j = static_cast<int>(idx % m);
  const float *e = emb + v * E;
  double ap = 0.0, ac = 0.0;
  for (int i = 0; i < E; ++i) {
    const double x = static_cast<double>(e[i]);
    ap += x * static_cast<double>(gp[static_cast<int64_t>(i) * m + j]);
    ac += x * static_cast<double>(gc[static_cast<int64_t>(i) * m + j]);
  }
  P[idx] = static_cast<float>(ap);
  Q[idx] = static_cast<float>(ac);
}

constexpr int kGather = 8;         // projection loads (16 bytes) in flight per lane

// Division by a runtime divisor d <= 64 of numerators n below 2^26, without a
// branch: the high half of n * ceil(2^32 / d) in 64 bits.  Exact in that
// range: with ceil(2^32 / d) = (2^32 + e) / d, 0 <= e < d, the quotient is
// n / d plus n e / (d 2^32) < 2^-6 <= 1/d, which never reaches the next
// integer.
struct FastDiv {
  uint64_t m;
  __device__ __forceinline__ uint32_t div(uint32_t n) const {
    return static_cast<uint32_t>((static_cast<uint64_t>(n) * m) >> 32);
  }
};
FastDiv make_fastdiv(uint32_t d) { return FastDiv{((1ull << 32) + d - 1) / d}; }

// One block of WV waves per (sequence b, depth l): all gather, then each wave
// scores its share of the parents (a tile of 16 on matrix cores).  Dynamic
// LDS: parents [K][mp], children [K][mp] (rows of m floats, zeros up to 4 MK, the
// score dim rounded up to a multiple of 16, plus 4: 16-byte aligned rows that start
// on different banks), depth embedding [m], log q [K], token ids [K], their ranks
// by id [K], clamped child and parent ids [K], parent tokens [K] and their ranks by
// id [K].  The scores come from edge_tiles<MK, NT> (NT column tiles of 16
// children).  Latency-bound: ids, gathers, then a chain of tiles.
template <int MK, int NT, int WV, bool FULL>
__global__ void __launch_bounds__(WV * kWave)
edge_kernel(int L, int K, int m_arg, int64_t V, FastDiv mdiv, const int32_t *__restrict__ topk_ids,
            const float *__restrict__ topk_logq, const int32_t *__restrict__ root_token,
            const float *__restrict__ P, const float *__restrict__ Q,
            const float *__restrict__ depth_emb, ScorerParams sp,
            float *__restrict__ edge_rows, int32_t *__restrict__ cand_by_rank,
            uint8_t *__restrict__ positive,
            float *__restrict__ edge_out, uint32_t *__restrict__ error_flag, SabaArgs sa,
            SabaParams sp_saba) {
  constexpr int kEdgeThreads = WV * kWave;
  extern __shared__ float smem[];
  constexpr int mp = 4 * MK + 4;
  const int m = FULL ? 4 * MK : m_arg;
  float *s_par = smem;
  float *s_chd = s_par + K * mp;
  float *s_u = s_chd + K * mp;           // 16-byte aligned
  float *s_lq = s_u + m;
  int32_t *s_tok = reinterpret_cast<int32_t *>(s_lq + K);
  int32_t *s_idr = s_tok + K;
  int32_t *s_cid = s_idr + K;
  int32_t *s_pid = s_cid + K;
  int32_t *s_ptok = s_pid + K;     // parent tokens (depth >= 2)
  int32_t *s_pidr = s_ptok + K;    // rank of each parent's token id in its depth

  // depth-major blocks: with a batch that is a multiple of the 8 XCDs, every
  // depth of sequence b runs on the XCD that the select block of b (block b)
  // runs on, so selection's reads of the rows find them in that XCD's L2
  const int batch = static_cast<int>(gridDim.x) / L;
  const int b = blockIdx.x % batch;
  const int l = blockIdx.x / batch;
  const int n_par = (l == 0) ? 1 : K;
  const int64_t row = static_cast<int64_t>(b) * L + l;
  const int tid = threadIdx.x;
  const int wave = WV == 1 ? 0 : __builtin_amdgcn_readfirstlane(tid / kWave);
  // the depth-1 block (one parent, the lightest) also computes the budget, in its
  // last wave
  const bool saba_wave = l == 0 && wave == WV - 1;
  SabaIn saba_in{};
  if (saba_wave) saba_in = saba_load(sa, sp_saba, b, L);

  int32_t root = root_token[b];
  if (root < 0 || root >= V) {
    if (tid == 0) atomicOr(error_flag, 1u);
    root = 0;
  }
  // token ids (clamped copies for the gathers; ids fall outside [0, V) only
  // with non-finite logits), log q and the depth embedding
  if (tid < K) {
    const int32_t ct = topk_ids[row * K + tid];
    const int32_t pt = (l == 0) ? root : topk_ids[(row - 1) * K + tid];
    s_tok[tid] = ct;
    s_lq[tid] = topk_logq[row * K + tid];
    s_cid[tid] = (ct < 0 || ct >= V) ? 0 : ct;
    s_pid[tid] = (pt < 0 || pt >= V) ? 0 : pt;
    s_ptok[tid] = pt;
  }
  for (int j = tid; j < m; j += kEdgeThreads) s_u[j] = sp.has_depth_emb ? depth_emb[l * m + j] : 0.f;
  __syncthreads();
  // rank of each candidate's token id within the depth
  if (tid < K) {
    const int32_t tc = s_tok[tid];
    int r = 0;
#pragma unroll 8
    for (int c2 = 0; c2 < K; ++c2) r += s_tok[c2] < tc;
    s_idr[tid] = r;
    cand_by_rank[row * K + r] = tc;
    int rp = 0;
    if (l > 0) {
      const int32_t tp = s_ptok[tid];
#pragma unroll 8
      for (int c2 = 0; c2 < K; ++c2) rp += s_ptok[c2] < tp;
    }
    s_pidr[tid] = rp;
  }
  // projections of children and parents plus the depth embedding, 16 bytes a
  // load when m % 4 == 0; every load of a batch is issued before any store
  if (FULL || (m & 3) == 0) {
    const int m4 = m >> 2;
    const int nq = K * m4, total = nq + n_par * m4;
    for (int base = 0; base < total; base += kGather * kEdgeThreads) {
      // the batch's token ids first (LDS), then its projection loads
      int32_t tok[kGather], j4s[kGather];
      bool child[kGather];
#pragma unroll
      for (int k = 0; k < kGather; ++k) {
        int t = base + k * kEdgeThreads + tid;
        t = t < total ? t : total - 1;
        child[k] = t < nq;
        const int tt = child[k] ? t : t - nq;
        const int r = static_cast<int>(FULL ? tt / MK : mdiv.div(static_cast<uint32_t>(tt)));
        j4s[k] = tt - r * m4;
        tok[k] = child[k] ? s_cid[r] : s_pid[r];
      }
      float4 v[kGather];
#pragma unroll
      for (int k = 0; k < kGather; ++k) {
        const float *src = (child[k] ? Q : P) + static_cast<int64_t>(tok[k]) * m;
        v[k] = reinterpret_cast<const float4 *>(src)[j4s[k]];
      }
#pragma unroll
      for (int k = 0; k < kGather; ++k) {
        const int t = base + k * kEdgeThreads + tid;
        if (t >= total) continue;
        const int tt = t < nq ? t : t - nq;
        const int r = static_cast<int>(FULL ? tt / MK : mdiv.div(static_cast<uint32_t>(tt))), j4 = tt - r * m4;
        const float4 u = reinterpret_cast<const float4 *>(s_u)[j4];
        float4 *dst = reinterpret_cast<float4 *>((t < nq ? s_chd : s_par) + r * mp) + j4;
        *dst = make_float4(v[k].x + u.x, v[k].y + u.y, v[k].z + u.z, v[k].w + u.w);
      }
    }
  } else {
    const int nq = K * m, total = nq + n_par * m;
#pragma unroll 4
    for (int t = tid; t < total; t += kEdgeThreads) {
      const int tt = t < nq ? t : t - nq;
      const int r = static_cast<int>(mdiv.div(static_cast<uint32_t>(tt))), j = tt - r * m;
      const float *src = t < nq ? Q + static_cast<int64_t>(s_cid[r]) * m
                                : P + static_cast<int64_t>(s_pid[r]) * m;
      (t < nq ? s_chd : s_par)[r * mp + j] = src[j] + s_u[j];
    }
  }
  if (!FULL) {
    const int pad = 4 * MK - m;   // fewer than 16 columns
    for (int t = tid; t < 2 * K * 16; t += kEdgeThreads)
      if ((t & 15) < pad) smem[(t >> 4) * mp + m + (t & 15)] = 0.f;   // parents, then children
  }
  __syncthreads();

  const float fscale = sp.scale / sqrtf(static_cast<float>(m));
  const int64_t base = row * K * K;
  // selection's copy is indexed by token-id rank (parent row, child column);
  // the exported table keeps the candidates' rank order
  const int32_t *prank = l == 0 ? nullptr : s_pidr;
  float *out = edge_out ? edge_out + base : nullptr;
  bool pos = false;
  if (WV == 1 && n_par > 16) {
    // the parents in two halves of whole 16-row tiles, their chains interleaved
    const int h = ((n_par + 31) / 32) * 16;
    const EdgeJob job[2] = {{s_par, s_chd, h, s_lq, s_idr, prank, edge_rows + base, out},
                            {s_par + h * mp, s_chd, n_par - h, s_lq, s_idr, prank + h,
                             edge_rows + base, out ? out + h * K : nullptr}};
    pos = edge_tiles<MK, NT, 2>(job, mp, K, fscale, sp.beta, sp.center);
  } else if (wave * 16 < n_par) {
    const int p0 = wave * 16, np = n_par - p0 < 16 ? n_par - p0 : 16;
    const EdgeJob job[1] = {{s_par + p0 * mp, s_chd, np, s_lq, s_idr, prank ? prank + p0 : nullptr,
                             edge_rows + base, out ? out + p0 * K : nullptr}};
    pos = edge_tiles<MK, NT, 1>(job, mp, K, fscale, sp.beta, sp.center);
  }
  if (edge_out && l == 0)
    for (int i = K + tid; i < K * K; i += kEdgeThreads) edge_out[base + i] = 0.f;
  bool any_pos = __ballot(pos) != 0ull;
  if constexpr (WV > 1) {
    // the gathers are over: the clamped ids' slots hold the waves' flags
    __syncthreads();
    if ((tid & (kWave - 1)) == 0) s_cid[wave] = any_pos ? 1 : 0;
    __syncthreads();
    for (int w = 0; w < WV; ++w) any_pos |= s_cid[w] != 0;
  }
  if (tid == 0) positive[row] = any_pos ? 1 : 0;
  if (saba_wave) saba_budget(sa, sp_saba, b, L, saba_in);
}

}  // namespace

hipError_t launch_projection(graft_ctx *ctx, const graft_scorer_desc *d, hipStream_t stream) {
  const int64_t V = ctx->dims.vocab;
  const int m = d->score_dim;
  const int64_t n = V * m;
  const unsigned blocks = static_cast<unsigned>((n + 255) / 256);
  hipLaunchKernelGGL(projection_kernel, dim3(blocks), dim3(256), 0, stream, d->emb, d->g_parent,
                     d->g_child, V, d->emb_dim, m, ctx->proj_parent, ctx->proj_child);
  return hipGetLastError();
}

hipError_t launch_edge_scores(graft_ctx *ctx, const RoundScratch &ws, const graft_round_in *in,
                              const graft_tree_out *out, hipStream_t stream) {
  const graft_dims &d = ctx->dims;
  const int batch = in->batch;
  const int32_t *root_token = in->root_token;
  float *edge_out = out->edge_scores;
  const SabaArgs sa = saba_args(ctx, ws, in, out);
  const int K = d.top_k, m = ctx->scorer.score_dim;
  const int mk = (m + 15) / 16 * 4;   // matrix-core k-slots a lane: score dim 4 mk
  const size_t mp = 4 * mk + 4;
  const size_t lds = sizeof(float) * (2 * static_cast<size_t>(K) * mp + K + (m + 3) / 4 * 4) +
                     sizeof(int32_t) * 6 * K;
  const FastDiv mdiv = make_fastdiv(static_cast<uint32_t>(m % 4 == 0 ? m / 4 : m));
  const unsigned blocks = static_cast<unsigned>(batch * d.num_pos);
  auto run = [&](auto kernel, int waves) {
    hipLaunchKernelGGL(kernel, dim3(blocks), dim3(waves * kWave), lds, stream, d.num_pos, K, m,
                       static_cast<int64_t>(d.vocab), mdiv, ws.topk_ids, ws.topk_logq, root_token,
                       ctx->proj_parent, ctx->proj_child, ctx->depth_emb, ctx->scorer, ws.edge_rows,
                       ws.cand_by_rank, ws.positive, edge_out, ctx->error_flag, sa, ctx->saba);
  };
  // A wave for each tile of 16 parents while that still leaves a wave a SIMD or
  // less of blocks (512 blocks of K = m = 64: 13.0 us against 22.4 in one wave;
  // 1024 blocks: 23.6 against 23.9), else one wave with two tiles interleaved (4096
  // blocks of K = m = 32: 15.7 us against 18.4 in two waves).
  const bool spread = blocks <= 1024;
  auto by_k = [&](auto k_slots) {
    constexpr int MK = decltype(k_slots)::value;
    auto by_width = [&](auto full) {
      constexpr bool FULL = decltype(full)::value;
      if (K <= 16) run(edge_kernel<MK, 1, 1, FULL>, 1);
      else if (K <= 32 && spread) run(edge_kernel<MK, 2, 2, FULL>, 2);
      else if (K <= 32) run(edge_kernel<MK, 2, 1, FULL>, 1);
      else if (spread) run(edge_kernel<MK, 4, 4, FULL>, 4);
      else run(edge_kernel<MK, 4, 1, FULL>, 1);
    };
    if (m == 4 * MK) by_width(std::true_type{});
    else by_width(std::false_type{});
  };
  if (mk == 4) by_k(std::integral_constant<int, 4>{});
  else if (mk == 8) by_k(std::integral_constant<int, 8>{});
  else if (mk == 12) by_k(std::integral_constant<int, 12>{});
  else by_k(std::integral_constant<int, 16>{});
  return hipGetLastError();
}

}  // namespace graft
