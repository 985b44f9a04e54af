// k_verify.hip -- verifier-side consumers of a round (the step after emission
// and acceptance; the paper's Preliminaries: the target model verifies the
// tree under a tree-attention mask and commits the longest accepted path).
//
// bias_kernel: expands the ancestor bitset of every node into its row of the
//   draft block's additive attention bias (0 where the node may attend, -inf
//   elsewhere).  Write-bound: the bias is the only large stream.  The 16-byte
//   chunks (8 bf16 or 4 fp32 entries) of a sequence are dealt out to the lanes in
//   address order, several per thread with all their mask words loaded first.
//   64 x 512 x 512 bf16 (33.6 MB): 8.3 us = 4.0 TB/s; one row a
//   wave, one store a lane: 13.0 us
// commit_kernel: moves the key/value rows of the accepted nodes to
//   consecutive rows.  A thread owns one 16-byte column of one plane of a
//   sequence and loads it from up to 16 accepted rows before storing any, so a
//   compaction in place never overwrites a row it has still to read (accepted
//   node indices increase along the path and are >= their position).  The columns
//   of all planes are dealt out to full workgroups, and the path is read with one
//   load beside its length.  72 planes x 64 sequences x 4 rows of 2 KiB
//   (74 MB both ways): 17.1 us; a workgroup a plane, half of it idle on such rows,
//   29.8 us; with cached stores 25.1, with streaming loads instead 18.8, with both
//   21.9
#include "graft_internal.h"

namespace graft {
namespace {

constexpr int kBiasThreads = 256;
constexpr int kCommitThreads = 256;
constexpr int kCommitGroup = 16;   // accepted rows loaded before any store

typedef unsigned int u32x4 __attribute__((ext_vector_type(4)));

// Chunk t of a sequence is chunk t % per_row of row t / per_row; div =
// ceil(2^32 / per_row) divides exactly, t < 2^18 and per_row <= 256.
template <bool BF16, int PER>
__global__ void __launch_bounds__(kBiasThreads)
bias_kernel(int n_max, int words, int per_row, uint64_t div, int blocks_per_seq, const int32_t *__restrict__ n_nodes,
            const uint64_t *__restrict__ mask, void *__restrict__ bias, int64_t ld,
            int64_t batch_stride) {
  constexpr int kPer = BF16 ? 8 : 4;                 // entries per chunk
  const int b = blockIdx.x / blocks_per_seq, blk = blockIdx.x - b * blocks_per_seq;
  const int total = n_max * per_row;
  const uint64_t *mseq = mask + static_cast<int64_t>(b) * n_max * words;
  char *seq = static_cast<char *>(bias) + static_cast<int64_t>(b) * batch_stride * (BF16 ? 2 : 4);
  const int t0 = blk * (kBiasThreads * PER) + threadIdx.x;
  int row[PER], j0[PER];
  uint64_t word[PER];
#pragma unroll
  for (int k = 0; k < PER; ++k) {
    int t = t0 + k * kBiasThreads;
    t = t < total ? t : total - 1;
    row[k] = static_cast<int>((static_cast<uint64_t>(t) * div) >> 32);
    j0[k] = (t - row[k] * per_row) * kPer;
    word[k] = mseq[row[k] * words + (j0[k] >> 6)];
  }
  int n = n_nodes[b];
  n = n < 0 ? 0 : (n > n_max ? n_max : n);
#pragma unroll
  for (int k = 0; k < PER; ++k) {
    if (t0 + k * kBiasThreads >= total) break;
    uint32_t bits = static_cast<uint32_t>(word[k] >> (j0[k] & 63)) & ((1u << kPer) - 1u);
    const int left = n - j0[k];                      // entries below n_nodes
    bits = row[k] < n && left > 0 ? (left < kPer ? bits & ((1u << left) - 1u) : bits) : 0u;
    uint32_t v[kPer];
#pragma unroll
    for (int i = 0; i < kPer; ++i)
      v[i] = (bits >> i) & 1u ? 0u : (BF16 ? 0xFF80u : 0xFF800000u);
    char *out = seq + (static_cast<int64_t>(row[k]) * ld + j0[k]) * (BF16 ? 2 : 4);
    if (j0[k] + kPer <= n_max) {
      u32x4 q;
      if (BF16) {
        q = u32x4{v[0] | (v[1] << 16), v[2] | (v[3] << 16), v[4] | (v[5] << 16),
                  v[6] | (v[7] << 16)};
      } else {
        q = u32x4{v[0], v[1], v[2], v[3]};
      }
      *reinterpret_cast<u32x4 *>(out) = q;
    } else {
      // ragged tail of a row whose length is not a multiple of kPer
      for (int i = 0; i < kPer && j0[k] + i < n_max; ++i) {
        if (BF16)
          reinterpret_cast<uint16_t *>(out)[i] = static_cast<uint16_t>(v[i]);
        else
          reinterpret_cast<uint32_t *>(out)[i] = v[i];
      }
    }
  }
}

// cols: 16-byte columns of a row; column t of a sequence is column t % cols of
// plane t / cols.
__global__ void __launch_bounds__(kCommitThreads)
commit_kernel(int batch, int blocks_per_seq, int64_t cols, int64_t total, int L, int n_max,
              const int32_t *__restrict__ acc_len, const int32_t *__restrict__ acc_nodes,
              const char *src, char *dst, int64_t sp, int64_t sb, int64_t sr, int64_t dp,
              int64_t db, int64_t dr, uint32_t *__restrict__ error_flag) {
  const int b = blockIdx.x / blocks_per_seq, blk = blockIdx.x - b * blocks_per_seq;
  const int32_t *nodes = acc_nodes + static_cast<int64_t>(b) * L;
  const int lane = lane_id();
  // the path beside its length: at most 64 entries, one per lane
  const int32_t mine = nodes[lane < L ? lane : 0];
  int a = acc_len[b];
  a = a < 0 ? 0 : (a > L ? L : a);
  const int64_t t = static_cast<int64_t>(blk) * kCommitThreads + threadIdx.x;
  const bool active = t < total;
  const int64_t tc = active ? t : 0;
  const int64_t p = total < (int64_t{1} << 32)
                        ? static_cast<uint32_t>(tc) / static_cast<uint32_t>(cols)
                        : tc / cols;
  const int64_t col = (tc - p * cols) * 16;
  const char *s0 = src + p * sp + b * sb + col;
  char *d0 = dst + p * dp + b * db + col;
  if (blk == 0 && threadIdx.x < kWave && lane < a && (mine < 0 || mine >= n_max))
    atomicOr(error_flag, 4u);
  for (int g = 0; g < a; g += kCommitGroup) {
    u32x4 v[kCommitGroup];
    bool ok[kCommitGroup];
#pragma unroll
    for (int k = 0; k < kCommitGroup; ++k) {
      ok[k] = false;
      if (g + k < a) {
        const int r = __builtin_amdgcn_readlane(mine, g + k);
        ok[k] = r >= 0 && r < n_max;
        if (ok[k] && active) v[k] = *reinterpret_cast<const u32x4 *>(s0 + r * sr);
      }
    }
#pragma unroll
    for (int k = 0; k < kCommitGroup; ++k)
      if (ok[k] && active) __builtin_nontemporal_store(v[k], reinterpret_cast<u32x4 *>(d0 + (g + k) * dr));
  }
}

}  // namespace

hipError_t launch_mask_to_bias(graft_ctx *ctx, int batch, const int32_t *n_nodes,
                               const uint64_t *mask, void *bias, int dtype, int64_t ld,
                               int64_t batch_stride, hipStream_t stream) {
  const int n_max = ctx->dims.max_nodes, words = (n_max + 63) / 64;
  const int per_row = dtype == 1 ? (n_max + 7) / 8 : (n_max + 3) / 4;
  const uint64_t div = ((1ull << 32) + per_row - 1) / per_row;
  const int total = n_max * per_row;
  auto run = [&](auto kernel, int per) {
    const int per_seq = (total + kBiasThreads * per - 1) / (kBiasThreads * per);
    hipLaunchKernelGGL(kernel, dim3(static_cast<unsigned>(per_seq) * batch), dim3(kBiasThreads), 0,
                       stream, n_max, words, per_row, div, per_seq, n_nodes, mask, bias, ld,
                       batch_stride);
  };
  // eight chunks a thread where that still fills the chip, else one
  const bool many = static_cast<int64_t>(total) * batch >= int64_t{8} * kBiasThreads * 512;
  if (dtype == 1) {
    if (many) run(bias_kernel<true, 8>, 8);
    else run(bias_kernel<true, 1>, 1);
  } else {
    if (many) run(bias_kernel<false, 8>, 8);
    else run(bias_kernel<false, 1>, 1);
  }
  return hipGetLastError();
}

hipError_t launch_commit(graft_ctx *ctx, int batch, const int32_t *acc_len,
                         const int32_t *acc_nodes, const void *src, void *dst, int64_t row_bytes,
                         int n_planes, int64_t sp, int64_t sb, int64_t sr, int64_t dp,
                         int64_t db, int64_t dr, hipStream_t stream) {
  const int64_t cols = row_bytes / 16, total = cols * n_planes;
  const int64_t per_seq = (total + kCommitThreads - 1) / kCommitThreads;
  hipLaunchKernelGGL(commit_kernel, dim3(static_cast<unsigned>(per_seq * batch)),
                     dim3(kCommitThreads), 0, stream, batch, static_cast<int>(per_seq), cols, total,
                     ctx->dims.num_pos, ctx->dims.max_nodes, acc_len, acc_nodes,
                     static_cast<const char *>(src), static_cast<char *>(dst), sp, sb, sr, dp, db,
                     dr, ctx->error_flag);
  return hipGetLastError();
}

}  // namespace graft
