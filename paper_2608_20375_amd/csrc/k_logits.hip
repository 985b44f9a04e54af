// k_logits.hip -- the logits pass: log-softmax statistics and top-K candidates
// of every drafter row q_{t,d} (the paper's Preliminaries, "DFlash one-pass
// marginals"; candidates = the highest-probability tokens of each position, as
// in the DDTree paragraph; conf_t of the SABA decoding state uses the top-1
// probability).
//
// One pass over the bf16 logits, HBM-bound where there are rows to fill the chip
// and latency-bound below.  Each workgroup (4 or 8 waves) streams one row with
// 16-byte loads, 4 loads in flight per lane.  Each wave keeps an online softmax
// in log2 units: a wave-uniform offset mL (fp32, = max * log2 e) and per lane
// S = sum 2^y and T2 = sum 2^y * y with y = x * log2 e - mL, accumulated per tile
// in fp32 and across tiles in fp64.
// Top-K: every wave keeps a threshold (initially from the block's lane maxima
// over the first tiles, later raised from what the waves have buffered); a tile
// whose maximum falls below it costs one ballot; a group of 8 values whose
// maximum reaches it is copied raw to a per-wave LDS ring, whose elements are
// offered to the wave's candidate buffer (ballot/mbcnt appends, a wave bitonic
// sort of (value desc, id asc) keys when full) only when the ring fills and at
// the end.  Thresholds come from a radix selection over 16-bit ordered values
// (one ballot a bit), and the block's survivors are ranked by counting; with
// bitonic sorts in their place the pass issued 9.20 VALU instructions per element
// and lane instead of 8.07 (4096 rows of 151936, K = 32).
// Where few long rows leave the chip idle, a row is split over several
// workgroups whose partial results a second small kernel merges.
//
// Measured against four-wave blocks with sorted thresholds, rows split to reach
// 1024 blocks and a one-wave merge (rocprofv3, pass plus merge, us):
//   rows x V, K            before        now
//   8 x 32000, 4           7.6 + 4.3     9.0
//   16 x 151936, 8         10.3 + 13.3   8.0 + 4.6
//   60 x 70001, 13         12.3 + 9.4    13.7
//   256 x 151936, 8        22.8 + 4.4    20.4
//   512 x 151936, 64       45.7 + 5.4    39.1
//   1024 x 128256, 16      46.8          46.7
//   4096 x 151936, 32      202.5         197.9
#include <algorithm>
#include <type_traits>

#include "degen_device.h"
#include "graft_internal.h"

namespace graft {
namespace {

constexpr int kUnroll = 4;                        // 16-byte loads per lane per tile
constexpr int kTileVec = kWave * kUnroll;         // 256 vectors = 2048 elements
constexpr float kL2E = 1.44269504088896340736f;
constexpr double kLn2 = 0.693147180559945309417232121458;
constexpr double kLog2e = 1.44269504088896340735992468100;
constexpr float kNegBig = -1e30f;                 // offset of softmax sums without an element
constexpr int kCus = 256;                         // compute units of the chip
constexpr int kMinSplitVec = 1024;                // >= 8192 elements per split
constexpr int kMaxSplits = 32;                    // blocks a row may be split over
constexpr int kList = 256;                        // keys the end of a row ranks by counting
constexpr int kMergeThreads = 256;
constexpr int kMergePer = kMaxSplits * kMaxK / kMergeThreads;   // keys a merge thread loads
constexpr int kRing = 64;                         // deferred groups per wave

typedef unsigned int u32x4 __attribute__((ext_vector_type(4)));

struct LaneStats {
  float mx;      // wave-uniform: largest logit the wave has seen
  float mL;      // wave-uniform fp32 offset: fl(mx * log2 e)
  double S;      // per lane: sum 2^(x*log2e - mL)
  double T2;     // per lane: sum 2^y * y
};

__device__ __forceinline__ void stats_init(LaneStats &s) {
  s.mx = kNegBig;
  s.mL = kNegBig * kL2E;
  s.S = 0.0;
  s.T2 = 0.0;
}

// Moves the wave's offset to its new maximum when some lane's value exceeds
// the old one, and rescales every lane's S and T2.  The factor
// 2^(mL_old - mL_new) is one v_exp_f32 of an fp32 difference (exact for offsets
// within a factor two of each other, and 0 for the initial finite stand-in).
__device__ __forceinline__ void stats_raise(LaneStats &s, float v) {
  if (__ballot(v > s.mx) == 0ull) return;
  float m = v;
#pragma unroll
  for (int o = 1; o < kWave; o <<= 1) m = fmaxf(m, __uint_as_float(xor_lane(__float_as_uint(m), o)));
  m = __int_as_float(__builtin_amdgcn_readfirstlane(__float_as_int(m)));
  const float nL = m * kL2E;
  const float d = s.mL - nL;
  const double a = static_cast<double>(__builtin_amdgcn_exp2f(d));
  s.T2 = a * (s.T2 + static_cast<double>(d) * s.S);
  s.S = a * s.S;
  s.mL = nL;
  s.mx = m;
}

// The k-th largest (1 <= k <= 64) of one value per lane, all of them bf16 values
// (or masked out with a value no lane counts on): the ordered key's upper 16
// bits are built from the top, one ballot and one scalar count a bit.  16 VALU
// compares against the ~130 instructions of a 64-key sort.
__device__ __forceinline__ float wave_kth_bf16(uint32_t key16, int k) {
  uint32_t t = 0;
#pragma unroll
  for (int bit = 15; bit >= 0; --bit) {
    const uint32_t c = t | (1u << bit);
    if (__popcll(__ballot(key16 >= c)) >= k) t = c;
  }
  return __uint_as_float(__float_as_uint(unordered_f32(t << 16)) & 0xFFFF0000u);
}
// The same over N values per lane, 1 <= k <= 64 N.
template <int N>
__device__ __forceinline__ float wave_kth_bf16(const uint32_t (&key16)[N], int k) {
  uint32_t t = 0;
#pragma unroll
  for (int bit = 15; bit >= 0; --bit) {
    const uint32_t c = t | (1u << bit);
    int n = 0;
#pragma unroll
    for (int i = 0; i < N; ++i) n += __popcll(__ballot(key16[i] >= c));
    if (n >= k) t = c;
  }
  return __uint_as_float(__float_as_uint(unordered_f32(t << 16)) & 0xFFFF0000u);
}

template <int CAP>
struct WaveBuf {
  uint64_t *buf;   // LDS [CAP]
  int count;       // wave-uniform
  float thr;       // wave-uniform: a candidate needs value >= thr
  uint4 *rq;       // LDS [kRing]: deferred groups of 8 raw bf16 values
  uint32_t *rid;   // LDS [kRing]: element id of each group's first value
  int rcount;      // wave-uniform
  bool flushed;    // wave-uniform: the ring was emptied since the bound was updated
};

struct Compacted {
  int count;
  float thr;
};

// Sorts the first 64*E entries of a wave's buffer (count of them valid), keeps
// the best K keys and raises the threshold to the K-th value.  Out of line: it
// runs a few times per wave at most, and a single copy keeps the offer sites
// small.
template <int E>
__device__ __noinline__ Compacted compact_ool(uint64_t *buf, int count, float thr, int K) {
  const int lane = lane_id();
  uint64_t k[E];
#pragma unroll
  for (int e = 0; e < E; ++e) {
    const int i = e * kWave + lane;
    k[e] = (i < count) ? buf[i] : 0ull;
  }
  wave_sort_desc<E>(k);
#pragma unroll
  for (int e = 0; e < E; ++e) {
    const int i = e * kWave + lane;
    if (i < K) buf[i] = k[e];
  }
  count = count < K ? count : K;
  if (count >= K) {
    const int src_e = (K - 1) / kWave, src_l = (K - 1) % kWave;
    uint64_t kth = 0;
#pragma unroll
    for (int e = 0; e < E; ++e)
      if (e == src_e) kth = k[e];
    const uint32_t hi = __shfl(static_cast<uint32_t>(kth >> 32), src_l);
    const float t = unordered_f32(hi);
    thr = t > thr ? t : thr;
  }
  return {count, thr};
}

// Compaction sized to the number of buffered keys (K <= count rounded up).
template <int CAP>
__device__ __forceinline__ void wave_compact(WaveBuf<CAP> &w, int K) {
  const int need = w.count > K ? w.count : K;
  Compacted c;
  if (need <= kWave) c = compact_ool<1>(w.buf, w.count, w.thr, K);
  else if (need <= 2 * kWave || CAP == 2 * kWave) c = compact_ool<2>(w.buf, w.count, w.thr, K);
  else c = compact_ool<CAP / kWave>(w.buf, w.count, w.thr, K);
  // wave-uniform results: keep them in scalar registers
  w.count = __builtin_amdgcn_readfirstlane(c.count);
  w.thr = __int_as_float(__builtin_amdgcn_readfirstlane(__float_as_int(c.thr)));
}

// The j-th largest value in a wave's buffer (bf16 values), -inf with fewer.
template <int CAP>
__device__ __forceinline__ float wave_buf_jth(const WaveBuf<CAP> &w, int j) {
  const int lane = lane_id();
  if (w.count < j) return -INFINITY;
  uint32_t k[CAP / kWave];
#pragma unroll
  for (int e = 0; e < CAP / kWave; ++e) {
    const int i = e * kWave + lane;
    k[e] = i < w.count ? static_cast<uint32_t>(w.buf[i] >> 48) : 0u;
  }
  return w.count <= kWave ? wave_kth_bf16(k[0], j) : wave_kth_bf16<CAP / kWave>(k, j);
}

// The smallest of the waves' bounds: with ceil(K / W) distinct values of every
// wave at or above it, a lower bound of the block's K-th value.
template <int W>
__device__ __forceinline__ float min_bound(const uint32_t *bound) {
  uint32_t lo = __hip_atomic_load(&bound[0], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
#pragma unroll
  for (int i = 1; i < W; ++i) {
    const uint32_t v = __hip_atomic_load(&bound[i], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
    lo = v < lo ? v : lo;
  }
  return unordered_f32(__builtin_amdgcn_readfirstlane(lo));
}

// Offers one value per lane (valid lanes only) to the wave's buffer.
template <int CAP>
__device__ __forceinline__ void wave_offer(WaveBuf<CAP> &w, int K, float v, uint32_t id,
                                           bool valid) {
  bool pass = valid && v >= w.thr;
  uint64_t m = __ballot(pass);
  if (m == 0) return;
  int n = __popcll(m);
  if (w.count + n > CAP) {
    wave_compact<CAP>(w, K);
    pass = valid && v >= w.thr;
    m = __ballot(pass);
    if (m == 0) return;
    n = __popcll(m);
  }
  if (pass) w.buf[w.count + lanes_below(m)] = cand_key(v, id);
  w.count = __builtin_amdgcn_readfirstlane(w.count + n);
}

__device__ __forceinline__ void unpack8(const uint4 q, float (&v)[8]) {
  const uint32_t w[4] = {q.x, q.y, q.z, q.w};
#pragma unroll
  for (int i = 0; i < 4; ++i) {
    v[2 * i] = __uint_as_float(w[i] << 16);
    v[2 * i + 1] = __uint_as_float(w[i] & 0xFFFF0000u);
  }
}

// Offers the deferred groups (one per lane) against the current threshold.
// A group was deferred when its largest value reached the threshold of the
// time; the threshold only rises, so comparing now drops nothing that belongs
// to the top K.  Out of line, with the buffer state passed by value.
template <int CAP>
__device__ __noinline__ Compacted flush_ool(uint64_t *buf, int count, float thr, const uint4 *rq,
                                            const uint32_t *rid, int rcount, int K) {
  const int lane = lane_id();
  WaveBuf<CAP> w{buf, count, thr, nullptr, nullptr, 0, false};
  const bool have = lane < rcount;
  uint4 r = make_uint4(0, 0, 0, 0);
  uint32_t id0 = 0;
  if (have) {
    r = rq[lane];
    id0 = rid[lane];
  }
  float v[8];
  unpack8(r, v);
  float gm = fmaxf(fmaxf(fmaxf(v[0], v[1]), v[2]), v[3]);
  gm = fmaxf(fmaxf(fmaxf(gm, v[4]), v[5]), fmaxf(v[6], v[7]));
  // The K-th largest group maximum is a lower bound of the wave's K-th value
  // (K distinct groups reach it): raise the threshold before offering.
  if (rcount >= K) {
    const float tau = wave_kth_bf16(have ? ordered_f32(gm) >> 16 : 0u, K);
    if (tau > w.thr) w.thr = tau;
  }
  const bool live = have && gm >= w.thr;
  if (__ballot(live) != 0ull) {
#pragma unroll
    for (int e = 0; e < 8; ++e) wave_offer<CAP>(w, K, v[e], id0 + e, live);
  }
  return {w.count, w.thr};
}

// The largest threshold any wave of the block has published, as an ordered key
// in one LDS word (raised with atomic maxima, read without a barrier; relaxed
// atomics keep the LDS addressing).
__device__ __forceinline__ float block_thr(const uint32_t *s_thr) {
  const uint32_t k = __hip_atomic_load(s_thr, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
  return unordered_f32(__builtin_amdgcn_readfirstlane(k));
}
__device__ __forceinline__ void publish_thr(uint32_t *s_thr, float thr) {
  __hip_atomic_fetch_max(s_thr, ordered_f32(thr), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
}

// The last flush of a wave's ring, inlined so that every access stays an LDS
// access.  It first takes the largest threshold any wave of the block has
// published (each is a lower bound of the block's K-th value), then the K-th
// largest group maximum of the ring, and offers what survives both.
template <int CAP>
__device__ __forceinline__ void wave_flush_last(WaveBuf<CAP> &w, int K, const uint32_t *s_thr) {
  const int lane = lane_id();
  w.thr = fmaxf(w.thr, block_thr(s_thr));
  const bool have = lane < w.rcount;
  uint4 r = make_uint4(0, 0, 0, 0);
  uint32_t id0 = 0;
  if (have) {
    r = w.rq[lane];
    id0 = w.rid[lane];
  }
  float v[8];
  unpack8(r, v);
  float gm = fmaxf(fmaxf(fmaxf(v[0], v[1]), v[2]), v[3]);
  gm = fmaxf(fmaxf(fmaxf(gm, v[4]), v[5]), fmaxf(v[6], v[7]));
  if (w.rcount >= K) {
    const float tau = wave_kth_bf16(have ? ordered_f32(gm) >> 16 : 0u, K);
    if (tau > w.thr) w.thr = tau;
  }
  const bool live = have && gm >= w.thr;
  if (__ballot(live) != 0ull) {
#pragma unroll
    for (int e = 0; e < 8; ++e) wave_offer<CAP>(w, K, v[e], id0 + e, live);
  }
  w.rcount = 0;
}

// Empties the wave's ring of deferred groups into its candidate buffer.
template <int CAP>
__device__ __forceinline__ void wave_flush(WaveBuf<CAP> &w, int K) {
  const Compacted c = flush_ool<CAP>(w.buf, w.count, w.thr, w.rq, w.rid, w.rcount, K);
  w.count = __builtin_amdgcn_readfirstlane(c.count);
  w.thr = __int_as_float(__builtin_amdgcn_readfirstlane(__float_as_int(c.thr)));
  w.rcount = 0;
  w.flushed = true;
}

// Loads tile t: lane handles vectors t * kTileVec + u * 64 + lane, u < kUnroll.
__device__ __forceinline__ void load_tile(const u32x4 *__restrict__ vec, int t,
                                          uint4 (&q)[kUnroll]) {
  const u32x4 *p = vec + t * kTileVec + lane_id();
#pragma unroll
  for (int u = 0; u < kUnroll; ++u) {
    const u32x4 x = __builtin_nontemporal_load(p + u * kWave);
    q[u] = make_uint4(x.x, x.y, x.z, x.w);
  }
}

// Largest of a group of 8 values, as a chain of 3-input maxima (v_max3_f32).
__device__ __forceinline__ float group_max(const float (&v)[8]) {
  const float a = fmaxf(fmaxf(v[0], v[1]), v[2]);
  const float b = fmaxf(fmaxf(a, v[3]), v[4]);
  const float c = fmaxf(fmaxf(b, v[5]), v[6]);
  return fmaxf(c, v[7]);
}
__device__ __forceinline__ float group_max(const uint4 q) {
  float v[8];
  unpack8(q, v);
  return group_max(v);
}

// Defers a group of 8 per lane (first element id id0) whose largest value g
// reaches the threshold: it is copied raw to the wave's ring, which is offered
// element by element when it fills.
template <int CAP>
__device__ __forceinline__ void push_group(const uint4 q, float g, uint32_t id0, bool valid,
                                           WaveBuf<CAP> &w, int K) {
  const bool pass = valid && g >= w.thr;
  const uint64_t m = __ballot(pass);
  if (m == 0ull) return;
  const int n = __popcll(m);
  if (w.rcount + n > kRing) wave_flush<CAP>(w, K);
  if (pass) {
    const int slot = w.rcount + lanes_below(m);
    w.rq[slot] = q;
    w.rid[slot] = id0;
  }
  w.rcount = __builtin_amdgcn_readfirstlane(w.rcount + n);
}

// The groups of one tile; any wave's threshold bounds the block's K-th value.
template <int CAP>
__device__ __forceinline__ void push_tile(const uint4 (&q)[kUnroll], const float (&sub)[kUnroll],
                                          float tmax, int t, uint32_t elem0, WaveBuf<CAP> &w,
                                          int K) {
  if (__ballot(tmax >= w.thr) == 0ull) return;
#pragma unroll
  for (int u = 0; u < kUnroll; ++u)
    push_group<CAP>(q[u], sub[u],
                    elem0 + static_cast<uint32_t>(t * kTileVec + u * kWave + lane_id()) * 8, true, w,
                    K);
}

// Softmax sums of one tile against the wave's offset (already raised to it).
__device__ __forceinline__ void tile_stats(const float (&v)[kUnroll][8], LaneStats &st) {
  const float mL = st.mL;
  // all arguments, then all exponentials, then the sums: no exp result is
  // consumed by the instruction right after it
  float s[kUnroll], t[kUnroll];
#pragma unroll
  for (int u = 0; u < kUnroll; ++u) {
    float y[8], ex[8];
#pragma unroll
    for (int e = 0; e < 8; ++e) y[e] = __builtin_fmaf(v[u][e], kL2E, -mL);
#pragma unroll
    for (int e = 0; e < 8; ++e) ex[e] = __builtin_amdgcn_exp2f(y[e]);
    s[u] = ex[0];
    t[u] = ex[0] * y[0];
#pragma unroll
    for (int e = 1; e < 8; ++e) {
      s[u] += ex[e];
      t[u] = __builtin_fmaf(ex[e], y[e], t[u]);
    }
  }
  st.S += static_cast<double>((s[0] + s[1]) + (s[2] + s[3]));
  st.T2 += static_cast<double>((t[0] + t[1]) + (t[2] + t[3]));
}

// The same for one vector per lane, of the valid lanes.
__device__ __forceinline__ void vec_stats(const uint4 q, bool valid, LaneStats &st) {
  float v[8], s = 0.f, t = 0.f;
  unpack8(q, v);
#pragma unroll
  for (int e = 0; e < 8; ++e) {
    const float y = __builtin_fmaf(valid ? v[e] : kNegBig, kL2E, -st.mL);
    const float ex = valid ? __builtin_amdgcn_exp2f(y) : 0.f;
    s += ex;
    t = __builtin_fmaf(ex, y, t);
  }
  st.S += static_cast<double>(s);
  st.T2 += static_cast<double>(t);
}

// The wave's own bound from its buffer, for min_bound.
template <int CAP, int W>
__device__ __forceinline__ void update_bound(const WaveBuf<CAP> &w, int K, uint32_t *bound) {
  const float b = wave_buf_jth<CAP>(w, (K + W - 1) / W);
  if (lane_id() == 0)
    __hip_atomic_fetch_max(bound, ordered_f32(b), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
}

// One full tile: top-K candidates against the block-shared threshold, then the
// statistics.  A wave that had to empty its ring tightens its bound and, with
// the others', the block's threshold.
template <int CAP, int W>
__device__ __forceinline__ void step_tile(const uint4 (&q)[kUnroll], int t, uint32_t elem0,
                                          LaneStats &st, WaveBuf<CAP> &w, int K, uint32_t *s_thr,
                                          uint32_t *s_bound, int wave) {
  w.thr = fmaxf(w.thr, block_thr(s_thr));
  float v[kUnroll][8], sub[kUnroll];
#pragma unroll
  for (int u = 0; u < kUnroll; ++u) unpack8(q[u], v[u]);
#pragma unroll
  for (int u = 0; u < kUnroll; ++u) sub[u] = group_max(v[u]);
  const float tmax = fmaxf(fmaxf(fmaxf(sub[0], sub[1]), sub[2]), sub[3]);
  push_tile<CAP>(q, sub, tmax, t, elem0, w, K);
  stats_raise(st, tmax);
  tile_stats(v, st);
  if (w.flushed) {
    update_bound<CAP, W>(w, K, &s_bound[wave]);
    w.thr = fmaxf(w.thr, min_bound<W>(s_bound));
    if (lane_id() == 0) publish_thr(s_thr, w.thr);
    w.flushed = false;
  }
}

// Adds the lanes' sums inside each row of 16 lanes (DPP steps only; the rows of
// all waves are added once, in lanes_merge).
__device__ __forceinline__ void stats_row_reduce(LaneStats &st) {
#pragma unroll
  for (int o = 1; o < 16; o <<= 1) {
    st.S += xor_lane_f64(st.S, o);
    st.T2 += xor_lane_f64(st.T2, o);
  }
}

struct RowOut {
  int32_t *ids;      // workspace [rows, K]
  float *logq;       // workspace [rows, K]
  float *stats;      // workspace [rows, 3]
  int32_t *o_ids;    // optional caller outputs
  float *o_logq, *o_lse, *o_maxprob, *o_ent;
};

// Final results of a row: lse from its merged statistics, the candidate of
// rank r, and the row's statistics given the largest logit.
// S >= 1 (the maximum contributes 2^0); the hardware log2 and exp2 in fp32 are
// accurate to about 2^-22 relative, far inside what the outputs need.
__device__ __forceinline__ double row_log2s(double S) {
  return static_cast<double>(__builtin_amdgcn_logf(static_cast<float>(S)));
}
__device__ __forceinline__ void write_cand(const RowOut &o, int64_t row, int K, int r,
                                           uint64_t key, double lse) {
  const int32_t id = key ? cand_id(key) : -1;
  const float lq = key ? static_cast<float>(static_cast<double>(cand_value(key)) - lse)
                       : -INFINITY;
  o.ids[row * K + r] = id;
  o.logq[row * K + r] = lq;
  if (o.o_ids) o.o_ids[row * K + r] = id;
  if (o.o_logq) o.o_logq[row * K + r] = lq;
}
__device__ __forceinline__ void write_stats(const RowOut &o, int64_t row, double mx, float mL,
                                            double S, double T2) {
  const double l2s = row_log2s(S), lse2 = static_cast<double>(mL) + l2s;
  const float f_lse = static_cast<float>(lse2 * kLn2);
  const float f_mp = __builtin_amdgcn_exp2f(static_cast<float>(mx * kLog2e - lse2));
  const float f_ent = static_cast<float>(kLn2 * (l2s - T2 / S));
  o.stats[row * 3 + 0] = f_lse;
  o.stats[row * 3 + 1] = f_mp;
  o.stats[row * 3 + 2] = f_ent;
  if (o.o_lse) o.o_lse[row] = f_lse;
  if (o.o_maxprob) o.o_maxprob[row] = f_mp;
  if (o.o_ent) o.o_ent[row] = f_ent;
}

// Merges the (mL, S, T2) triples of each run of N lanes into all of them: the
// largest offset, then the rescaled sums added across lanes.  Lanes with on
// false add nothing.  Every lane of the wave gets a result.
template <int N>
__device__ __forceinline__ void lanes_merge(bool on, float &mL, double &S, double &T2) {
  float m = on ? mL : -INFINITY;
#pragma unroll
  for (int o = 1; o < N; o <<= 1)
    m = fmaxf(m, __uint_as_float(xor_lane(__float_as_uint(m), o)));
  const double d = on ? static_cast<double>(mL) - static_cast<double>(m) : 0.0;
  const double a = static_cast<double>(__builtin_amdgcn_exp2f(static_cast<float>(d)));
  T2 = on ? a * (T2 + d * S) : 0.0;
  S = on ? a * S : 0.0;
#pragma unroll
  for (int o = 1; o < N; o <<= 1) {
    S += xor_lane_f64(S, o);
    T2 += xor_lane_f64(T2, o);
  }
  mL = m;
}

// Sorts the first n <= 64*E keys of buf (LDS) and writes the best K back to
// the front.
template <int E>
__device__ __forceinline__ void sort_front(uint64_t *buf, int n, int K) {
  const int lane = lane_id();
  uint64_t k[E];
#pragma unroll
  for (int e = 0; e < E; ++e) {
    const int i = e * kWave + lane;
    k[e] = i < n ? buf[i] : 0ull;
  }
  wave_sort_desc<E>(k);
#pragma unroll
  for (int e = 0; e < E; ++e) {
    const int i = e * kWave + lane;
    if (i < K) buf[i] = k[e];
  }
}
// Moves the keys of buf[from, n) that are larger than `above` to buf[to, ...)
// in order (to <= from: nothing is overwritten before it is read) and returns
// the new end.
__device__ __forceinline__ int keep_above(uint64_t *buf, int from, int n, int to,
                                          uint64_t above) {
  const int lane = lane_id();
  for (int j0 = from; j0 < n; j0 += kWave) {
    const int j = j0 + lane;
    const uint64_t key = j < n ? buf[j] : 0ull;
    const bool keep = j < n && key > above;
    const uint64_t b = __ballot(keep);
    if (keep) buf[to + lanes_below(b)] = key;
    to += __popcll(b);
  }
  return to;
}

// Top K of the block by sorting (wave 0): the way out when more than kList keys
// reach the block's threshold th (long runs of equal logits).  Keys below th are
// dropped while the buffers are packed to the front of buf (a key never moves
// past an entry not yet read).  More than 256 survivors are cut down by sorting
// the first 256 and keeping only keys above the K-th of those, which removes at
// least 256 - K keys per pass.  On return buf[0..K) holds the block's top K in
// descending key order, 0 past the last candidate.
template <int CAP, int W>
__device__ __noinline__ void block_merge(uint64_t *buf, const int *cnt, float th, int K) {
  const int lane = lane_id();
  int m = 0;
  for (int wv = 0; wv < W; ++wv) {
    const int c = cnt[wv];
    for (int j0 = 0; j0 < c; j0 += kWave) {
      const int j = j0 + lane;
      const uint64_t key = j < c ? buf[wv * CAP + j] : 0ull;
      const bool keep = key != 0ull && cand_value(key) >= th;
      const uint64_t b = __ballot(keep);
      if (keep) buf[m + lanes_below(b)] = key;
      m += __popcll(b);
    }
  }
  while (m > 4 * kWave) {
    sort_front<4>(buf, 4 * kWave, K);
    m = keep_above(buf, 4 * kWave, m, K, buf[K - 1]);
  }
  sort_front<4>(buf, m, K);
  for (int i = m + lane; i < K; i += kWave) buf[i] = 0ull;
}

// Number of keys of list[0, m) larger than mine (keys are distinct): the key's
// rank.  Independent broadcast reads 16 at a time (the list is padded by 16), no
// chain: at the usual 20 to 100 keys cheaper than the 21 to 28 dependent steps
// of a sort.
__device__ __forceinline__ int rank_in(const uint64_t *list, int m, uint64_t mine) {
  int r = 0;
  for (int i = 0; i < m; i += 16) {
    uint64_t k[16];
#pragma unroll
    for (int j = 0; j < 16; ++j) k[j] = list[i + j];
#pragma unroll
    for (int j = 0; j < 16; ++j) r += (i + j < m) & (k[j] > mine);
  }
  return r;
}

template <int CAP, int W>
struct PassMem {
  uint64_t buf[W][CAP];
  uint4 rq[W][kRing];
  uint32_t rid[W][kRing];
  alignas(16) uint64_t list[kList + 16];
  double S[4 * W], T2[4 * W];   // per row of 16 lanes
  float mL[W];
  double fin[4];              // the chunk's mL, S, T2, and lse
  uint32_t lmax[W * kWave];   // lane maxima: all of a short chunk, a long one's first tiles
  uint32_t bound[W];          // per wave: ceil(K / W) of its values reach this (ordered key)
  uint32_t thr;               // largest published threshold, ordered key
  int cnt[W];
  int n_short, n_list;        // keys in list: of a short chunk, of the buffers
};

// A lower bound of the chunk's K-th largest value from the lanes' maxima (lmax,
// then a barrier): K distinct lanes reach the K-th largest of them.  Over the whole
// block, since words ordered by frequency put the largest logits of a row into one
// wave's share.  Where every lane holds elements (full), formed from the maxima of
// 256 groups of lanes across the waves, up to 16 candidates of 128, which takes
// fewer ballots; else the groups could be fewer than K.
// Against the smallest of the eight waves' own ceil(K / 8)-th maxima, which lets a
// hundred and more keys through on ordered words (us; logit = 2 normal -
// log(rank)): 16 rows of 8000, K = 8 11.9 -> 7.4, K = 64 25.4 -> 10.2, 512 rows of
// 32000, K = 64 34.1 -> 22.0; on exchangeable ones: 16 rows of 32000, K = 8 10.8 ->
// 10.4, 512 of 151936, K = 64 38.8 -> 39.0, one of 32000, K = 64 12.5 -> 12.8.
template <int CAP, int W>
__device__ __forceinline__ float lanes_kth(const PassMem<CAP, W> &s, int K, bool full) {
  const int lane = lane_id();
  uint32_t k[W];
#pragma unroll
  for (int i = 0; i < W; ++i) k[i] = s.lmax[i * kWave + lane];
  if (full) {
    uint32_t g[4];
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      g[i] = k[i];
#pragma unroll
      for (int j = i + 4; j < W; j += 4) g[i] = g[i] > k[j] ? g[i] : k[j];
    }
    if (K > 16) return wave_kth_bf16<4>(g, K);
    const uint32_t h[2] = {g[0] > g[2] ? g[0] : g[2], g[1] > g[3] ? g[1] : g[3]};
    return wave_kth_bf16<2>(h, K);
  }
  return wave_kth_bf16<W>(k, K);
}

template <int CAP, int W>
__device__ __forceinline__ void put_stats(PassMem<CAP, W> &s, LaneStats &st, int wave) {
  stats_row_reduce(st);
  const int lane = lane_id();
  if ((lane & 15) == 0) {
    s.S[4 * wave + (lane >> 4)] = st.S;
    s.T2[4 * wave + (lane >> 4)] = st.T2;
  }
  if (lane == 0) s.mL[wave] = st.mL;
}

// The chunk's statistics from the waves' (put_stats, then a barrier), by wave 0
// while the others list their keys: a split's partial goes out here, a row's is
// left in fin for write_ranked.
template <int CAP, int W>
__device__ __forceinline__ void merge_stats(PassMem<CAP, W> &s, int wave, int64_t slot, int splits,
                                            double *part_stats) {
  if (wave != 0) return;
  const int i = lane_id() & (4 * W - 1);
  float mL = s.mL[i >> 2];
  double S = s.S[i], T2 = s.T2[i];
  lanes_merge<4 * W>(true, mL, S, T2);
  if (lane_id() == 0) {
    double *to = splits > 1 ? part_stats + slot * 3 : s.fin;
    to[0] = static_cast<double>(mL);
    to[1] = S;
    to[2] = T2;
    if (splits == 1) s.fin[3] = (static_cast<double>(mL) + row_log2s(S)) * kLn2;
  }
}

// The block's results from the m <= kList keys of its list, every one at or
// above a lower bound of the chunk's K-th value: a key's rank is counted and the
// key written to its place.
template <int CAP, int W>
__device__ __forceinline__ void write_ranked(PassMem<CAP, W> &s, int m, int wave, int64_t row,
                                             int64_t slot, int splits, int K, uint64_t *part_keys,
                                             const RowOut &out) {
  const int n_rank = m > K ? m : K;                 // slots past m are empty
  for (int t = wave * kWave + lane_id(); t < n_rank; t += W * kWave) {
    const uint64_t key = t < m ? s.list[t] : 0ull;
    const int r = t < m ? rank_in(s.list, m, key) : t;
    if (r >= K) continue;
    if (splits > 1) {
      part_keys[slot * K + r] = key;
    } else {
      write_cand(out, row, K, r, key, s.fin[3]);
      if (r == 0)
        write_stats(out, row, static_cast<double>(cand_value(key)), static_cast<float>(s.fin[0]),
                    s.fin[1], s.fin[2]);
    }
  }
}

// The end of a block's chunk from the waves' buffers (rings flushed, statistics
// put): all waves drop their keys below the block's threshold into one list,
// whose keys are then ranked: two barriers and no sort.  More keys than the list
// holds (long runs of equal logits) are sorted by wave 0.
template <int CAP, int W>
__device__ __forceinline__ void finish_buffers(PassMem<CAP, W> &s, const WaveBuf<CAP> &w, int wave,
                                               int64_t row, int64_t slot, int splits, int K,
                                               double *part_stats, uint64_t *part_keys,
                                               const RowOut &out, bool with_stats) {
  const int lane = lane_id();
  update_bound<CAP, W>(w, K, &s.bound[wave]);
  if (lane == 0) {
    s.cnt[wave] = w.count;
    publish_thr(&s.thr, w.thr);
  }
  __syncthreads();
  const float th = fmaxf(block_thr(&s.thr), min_bound<W>(s.bound));
  if (with_stats) merge_stats<CAP, W>(s, wave, slot, splits, part_stats);
  for (int j0 = 0; j0 < w.count; j0 += kWave) {
    const int j = j0 + lane;
    const uint64_t key = j < w.count ? w.buf[j] : 0ull;
    const bool keep = key != 0ull && cand_value(key) >= th;
    const uint64_t b = __ballot(keep);
    const int n = __popcll(b);
    int at = 0;
    if (lane == 0 && n > 0) at = atomicAdd(&s.n_list, n);
    at = __builtin_amdgcn_readfirstlane(at) + lanes_below(b);
    if (keep && at < kList) s.list[at] = key;
  }
  __syncthreads();
  int m = s.n_list;
  if (m > kList) {
    if (wave == 0) {
      block_merge<CAP, W>(&s.buf[0][0], s.cnt, th, K);
      if (lane < K) s.list[lane] = s.buf[0][lane];
    }
    __syncthreads();
    m = K;   // at least K keys reach th
  }
  write_ranked<CAP, W>(s, m, wave, row, slot, splits, K, part_keys, out);
}

// The chunk of a row that a block reads.
struct Chunk {
  const uint16_t *rowp;
  const u32x4 *vec;     // its 16-byte aligned vectors
  int n_vec;
  uint32_t elem0;       // element id of vec[0]
  int a0, nv_row;       // the row's aligned body: elements [a0, a0 + 8 nv_row)
};
__device__ __forceinline__ Chunk chunk_of(const uint16_t *logits, int V, int64_t row, int split,
                                          int splits) {
  Chunk c;
  c.rowp = logits + row * V;
  c.a0 = (8 - static_cast<int>((row * V) & 7)) & 7;
  if (c.a0 > V) c.a0 = V;
  c.nv_row = (V - c.a0) / 8;
  const int per = (c.nv_row + splits - 1) / splits;
  const int begin = per * split < c.nv_row ? per * split : c.nv_row;
  c.n_vec = begin + per < c.nv_row ? per : c.nv_row - begin;
  c.elem0 = static_cast<uint32_t>(c.a0 + begin * 8);
  c.vec = reinterpret_cast<const u32x4 *>(c.rowp + c.a0) + begin;
  return c;
}
// The misaligned head [0, a0) and tail [a0 + 8 nv_row, V) of a row, fewer than
// 16 elements, go to one wave of split 0, one per lane: their number, and the
// element of a lane below it.
__device__ __forceinline__ int loose_count(const Chunk &c, int V) { return V - 8 * c.nv_row; }
__device__ __forceinline__ int loose_id(const Chunk &c, int lane) {
  return lane < c.a0 ? lane : 8 * c.nv_row + lane;
}
__device__ __forceinline__ float bf16_value(uint16_t h) {
  return __uint_as_float(static_cast<uint32_t>(h) << 16);
}
__device__ __forceinline__ void loose_stats(float x, bool valid, LaneStats &st) {
  const float y = __builtin_fmaf(x, kL2E, -st.mL);
  const float ex = valid ? __builtin_amdgcn_exp2f(y) : 0.f;
  st.S += static_cast<double>(ex);
  st.T2 += static_cast<double>(ex * y);
}

// A chunk of at most one tile a wave: divided evenly over the W waves, all of it
// loaded at once and kept in registers.  Latency-bound: the lanes' maxima and the
// waves' statistics meet at one barrier, then the few keys that reach the threshold go
// straight to the block's list and are ranked after a second one.
template <int CAP, int W>
__global__ void __launch_bounds__(W * kWave, 4)
short_pass_kernel(const uint16_t *__restrict__ logits, int V, int splits, int K,
                  double *__restrict__ part_stats, uint64_t *__restrict__ part_keys, RowOut out,
                  DegenArgs degen) {
  __shared__ PassMem<CAP, W> s;
  if (blockIdx.x >= degen.first) {   // a run of hidden-state cosines (degen_device.h)
    __shared__ double s_part[W][kDegenAcc];
    degen_run<W>(degen, blockIdx.x - degen.first, s_part);
    return;
  }
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x / kWave);
  const int lane = lane_id();
  const int64_t row = blockIdx.x / splits;
  const int split = blockIdx.x % splits;
  const Chunk c = chunk_of(logits, V, row, split, splits);

  const int pw = (c.n_vec + W - 1) / W;
  const int wb = pw * wave < c.n_vec ? pw * wave : c.n_vec;
  const int we = wb + pw < c.n_vec ? wb + pw : c.n_vec;
  const int nu = (we - wb + kWave - 1) / kWave;   // wave-uniform, <= kUnroll
  uint4 q[kUnroll];
#pragma unroll
  for (int u = 0; u < kUnroll; ++u) {
    q[u] = make_uint4(0, 0, 0, 0);
    const int vi = wb + u * kWave + lane;
    if (u < nu) {
      const u32x4 x = __builtin_nontemporal_load(c.vec + (vi < we ? vi : we - 1));
      q[u] = make_uint4(x.x, x.y, x.z, x.w);
    }
  }
  // wave 0 of split 0 takes the loose elements
  const int n_loose = split == 0 && wave == 0 ? loose_count(c, V) : 0;
  const bool lvalid = lane < n_loose;
  const int lid = lvalid ? loose_id(c, lane) : 0;
  float lx = kNegBig;
  if (n_loose > 0) lx = lvalid ? bf16_value(c.rowp[lid]) : kNegBig;
  LaneStats st;
  stats_init(st);
  if (threadIdx.x == 0) {
    s.thr = ordered_f32(-INFINITY);
    s.n_short = 0;
    s.n_list = 0;
  }

  // (-inf, no finite value, past the end: a masked logit may be as low as any)
  float g[kUnroll], own = -INFINITY;
#pragma unroll
  for (int u = 0; u < kUnroll; ++u) {
    g[u] = -INFINITY;
    if (u < nu && wb + u * kWave + lane < we) g[u] = group_max(q[u]);   // else past the end
    own = fmaxf(own, g[u]);
  }
  s.lmax[wave * kWave + lane] = ordered_f32(own) >> 16;
  if (lane == 0) s.bound[wave] = ordered_f32(-INFINITY);
  stats_raise(st, fmaxf(own, lx));
#pragma unroll
  for (int u = 0; u < kUnroll; ++u)
    if (u < nu) vec_stats(q[u], wb + u * kWave + lane < we, st);
  if (n_loose > 0) loose_stats(lx, lvalid, st);
  put_stats<CAP, W>(s, st, wave);
  __syncthreads();
  const float thr = lanes_kth<CAP, W>(s, K, c.n_vec >= W * kWave);   // -inf: fewer than K lanes
  const int64_t slot = row * splits + split;
  // a lane's elements that reach it, as bits u * 8 + e; one scan and one LDS
  // atomic place the wave's keys
  uint32_t hit = 0;
#pragma unroll
  for (int u = 0; u < kUnroll; ++u) {
    if (__ballot(g[u] >= thr) == 0ull) continue;   // nothing, or past the end
    float v[8];
    unpack8(q[u], v);
#pragma unroll
    for (int e = 0; e < 8; ++e) hit |= v[e] >= thr ? 1u << (u * 8 + e) : 0u;
    if (u >= nu || wb + u * kWave + lane >= we) hit &= ~(0xFFu << (u * 8));
  }
  const bool lhit = lvalid && lx >= thr;
  const int mine = __popc(hit) + (lhit ? 1 : 0);
  if (__ballot(mine > 0) != 0ull) {
    const int inc = wave_incl_scan(mine);
    int at = 0;
    if (lane == kWave - 1) at = atomicAdd(&s.n_short, inc);
    at = __builtin_amdgcn_readlane(at, kWave - 1) + inc - mine;
#pragma unroll
    for (int u = 0; u < kUnroll; ++u) {
      if (__ballot(((hit >> (u * 8)) & 0xFFu) != 0u) == 0ull) continue;
      const uint32_t id0 = c.elem0 + (wb + u * kWave + lane) * 8;
      float v[8];
      unpack8(q[u], v);
#pragma unroll
      for (int e = 0; e < 8; ++e)
        if ((hit >> (u * 8 + e)) & 1u) {
          if (at < kList) s.list[at] = cand_key(v[e], id0 + e);
          ++at;
        }
    }
    if (lhit && at < kList) s.list[at] = cand_key(lx, lid);
  }
  merge_stats<CAP, W>(s, wave, slot, splits, part_stats);
  __syncthreads();
  if (s.n_short <= kList) {
    write_ranked<CAP, W>(s, s.n_short, wave, row, slot, splits, K, part_keys, out);
    return;
  }
  // long runs of equal logits: through the waves' buffers
  WaveBuf<CAP> w{s.buf[wave], 0, thr, s.rq[wave], s.rid[wave], 0, false};
#pragma unroll
  for (int u = 0; u < kUnroll; ++u)
    if (u < nu) {
      const int vi = wb + u * kWave + lane;
      push_group<CAP>(q[u], g[u], c.elem0 + vi * 8, vi < we, w, K);
    }
  wave_offer<CAP>(w, K, lx, lid, lvalid);
  if (w.rcount > 0) wave_flush_last<CAP>(w, K, &s.thr);
  finish_buffers<CAP, W>(s, w, wave, row, slot, splits, K, part_stats, part_keys, out, false);
}

// A longer chunk, one block of W waves per row, or per split of a row (see
// logits_waves).
template <int CAP, int W>
__global__ void __launch_bounds__(W * kWave, 4)
logits_pass_kernel(const uint16_t *__restrict__ logits, int V, int splits, int K,
                   double *__restrict__ part_stats, uint64_t *__restrict__ part_keys,
                   RowOut out,
                  DegenArgs degen) {
  __shared__ PassMem<CAP, W> s;
  if (blockIdx.x >= degen.first) {   // a run of hidden-state cosines (degen_device.h)
    __shared__ double s_part[W][kDegenAcc];
    degen_run<W>(degen, blockIdx.x - degen.first, s_part);
    return;
  }

  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x / kWave);
  const int lane = lane_id();
  const int64_t row = blockIdx.x / splits;
  const int split = blockIdx.x % splits;
  const Chunk c = chunk_of(logits, V, row, split, splits);

  LaneStats st;
  stats_init(st);
  WaveBuf<CAP> w{s.buf[wave], 0, -INFINITY, s.rq[wave], s.rid[wave], 0, false};
  if (threadIdx.x == 0) {
    s.thr = ordered_f32(-INFINITY);
    s.n_list = 0;
  }

  // Tiles interleaved over the waves of the block; the next tile's loads are
  // issued before the current tile is processed.
  // At least one full tile; the last split of a row may have fewer than W, and
  // its surplus waves read the last one and skip it.
  const int n_full = c.n_vec / kTileVec;
  int t = wave;
  uint4 cur[kUnroll], nxt[kUnroll];
  const bool one = t < n_full, two = t + W < n_full;
  const int t0 = one ? t : n_full - 1;
  load_tile(c.vec, t0, cur);
  // The vectors past the full tiles (fewer than kTileVec) are spread over the
  // block, one per lane, and loaded with the first tiles; surplus lanes read
  // the last vector and are masked.
  const int pv = n_full * kTileVec + wave * kWave + lane;
  const bool partial = n_full * kTileVec + wave * kWave < c.n_vec;
  const bool pvalid = pv < c.n_vec;
  uint4 extra = make_uint4(0, 0, 0, 0);
  if (partial) {
    const u32x4 x = __builtin_nontemporal_load(c.vec + (pvalid ? pv : c.n_vec - 1));
    extra = make_uint4(x.x, x.y, x.z, x.w);
  }
  load_tile(c.vec, two ? t + W : t0, nxt);
  // Initial threshold, block wide, from the lanes' maxima over the first tile
  // (two tiles with 4 waves, whose first tiles hold few of the row).  A lane with
  // no element holds -inf, which every later bound exceeds (a finite stand-in would
  // pass for a logit in rows masked with large negative values).
  {
    float tm = -INFINITY;
#pragma unroll
    for (int u = 0; u < kUnroll; ++u) {
      if (one) tm = fmaxf(tm, group_max(cur[u]));
      if (W == 4 && two) tm = fmaxf(tm, group_max(nxt[u]));
    }
    if (partial && pvalid) tm = fmaxf(tm, group_max(extra));
    s.lmax[wave * kWave + lane] = ordered_f32(tm) >> 16;
    if (lane == 0) s.bound[wave] = ordered_f32(-INFINITY);
    __syncthreads();
    w.thr = lanes_kth<CAP, W>(s, K, n_full >= W);
  }
  if (partial) {
    const float g = pvalid ? group_max(extra) : kNegBig;
    push_group<CAP>(extra, g, c.elem0 + pv * 8, pvalid, w, K);
    stats_raise(st, g);
    vec_stats(extra, pvalid, st);
  }
  // ping-pong between two register buffers: the loads of tile t + W are in
  // flight while tile t is processed
  // The prefetch of tile t + W is issued on every step (past the last tile it
  // re-reads a valid one, a cache hit), so the wait before the current tile
  // covers only its own loads and never the prefetch.
  if (one) step_tile<CAP, W>(cur, t, c.elem0, st, w, K, &s.thr, s.bound, wave);
  for (;;) {
    t += W;
    if (t >= n_full) break;
    load_tile(c.vec, t + W < n_full ? t + W : n_full - 1, cur);
    step_tile<CAP, W>(nxt, t, c.elem0, st, w, K, &s.thr, s.bound, wave);
    t += W;
    if (t >= n_full) break;
    load_tile(c.vec, t + W < n_full ? t + W : n_full - 1, nxt);
    step_tile<CAP, W>(cur, t, c.elem0, st, w, K, &s.thr, s.bound, wave);
  }
  if (split == 0 && wave == 0 && loose_count(c, V) > 0) {
    const bool lvalid = lane < loose_count(c, V);
    const int lid = lvalid ? loose_id(c, lane) : 0;
    const float x = lvalid ? bf16_value(c.rowp[lid]) : kNegBig;
    wave_offer<CAP>(w, K, x, lid, lvalid);
    stats_raise(st, x);
    loose_stats(x, lvalid, st);
  }
  put_stats<CAP, W>(s, st, wave);
  if (w.rcount > 0) wave_flush_last<CAP>(w, K, &s.thr);
  const int64_t slot = row * splits + split;
  finish_buffers<CAP, W>(s, w, wave, row, slot, splits, K, part_stats, part_keys, out, true);
}

// One block per split row: merges the partial statistics and top-K lists (each
// in descending order, 0 past its end).  Latency-bound, so everything is loaded
// at once and nothing is sorted: with j = ceil(K / splits) and q = ceil(K / j),
// q lists whose j-th key is at least v hold K keys of at least v, so the q-th
// largest of the j-th values bounds the row's K-th from below, and so does the
// largest of the lists' K-th keys (the tight one where one split holds most of the
// row's largest logits: 16 rows of 151936 words ordered by frequency, K = 64, pass
// and merge 51.5 -> 17.5 us); the few keys that reach both are ranked by counting.
__global__ void __launch_bounds__(kMergeThreads)
merge_kernel(int splits, int K, const double *__restrict__ part_stats,
             const uint64_t *__restrict__ part_keys, RowOut out) {
  __shared__ alignas(16) uint64_t s_list[kMaxSplits * kMaxK + 16];
  __shared__ int s_n;
  const int64_t row = blockIdx.x;
  const int tid = threadIdx.x, lane = lane_id(), wave = tid / kWave;
  const uint64_t *pk = part_keys + row * splits * K;
  const int total = splits * K;
  uint64_t key[kMergePer];
#pragma unroll
  for (int i = 0; i < kMergePer; ++i) {
    const int t = i * kMergeThreads + tid;
    key[i] = pk[t < total ? t : 0];
    if (t >= total) key[i] = 0ull;
  }
  const int sl = lane & (kMaxSplits - 1);
  const bool has = sl < splits;
  const int j = (K + splits - 1) / splits, q = (K + j - 1) / j;
  const uint64_t jth = pk[(has ? sl : 0) * K + j - 1], last = pk[(has ? sl : 0) * K + K - 1];
  const double *ps = part_stats + row * splits * 3 + (has ? sl : 0) * 3;
  float mL = static_cast<float>(ps[0]);   // the offsets are fp32 values
  double S = ps[1], T2 = ps[2];
  if (tid == 0) s_n = 0;
  __syncthreads();
  const uint32_t jk = lane < splits ? static_cast<uint32_t>(jth >> 48) : 0u;   // bf16 values
  uint32_t th = 0;
#pragma unroll
  for (int bit = 15; bit >= 0; --bit) {
    const uint32_t c = th | (1u << bit);
    if (__popcll(__ballot(jk >= c)) >= q) th = c;
  }
  uint32_t lk = static_cast<uint32_t>(last >> 48);
#pragma unroll
  for (int o = 1; o < kMaxSplits; o <<= 1) {
    const uint32_t other = xor_lane(lk, o);
    lk = lk > other ? lk : other;
  }
  th = th > lk ? th : lk;   // lk: both halves of the wave hold the same lists
#pragma unroll
  for (int i = 0; i < kMergePer; ++i) {
    const bool keep = key[i] != 0ull && static_cast<uint32_t>(key[i] >> 48) >= th;
    const uint64_t b = __ballot(keep);
    if (b == 0ull) continue;
    int at = 0;
    if (lane == 0) at = atomicAdd(&s_n, __popcll(b));
    at = __builtin_amdgcn_readfirstlane(at) + lanes_below(b);
    if (keep) s_list[at] = key[i];
  }
  __syncthreads();
  const int m = s_n, n_rank = m > K ? m : K;
  if (wave * kWave >= n_rank) return;
  lanes_merge<kMaxSplits>(has, mL, S, T2);
  const double lse = (static_cast<double>(mL) + row_log2s(S)) * kLn2;
  for (int t = tid; t < n_rank; t += kMergeThreads) {
    const uint64_t k = t < m ? s_list[t] : 0ull;
    const int r = t < m ? rank_in(s_list, m, k) : t;
    if (r >= K) continue;
    write_cand(out, row, K, r, k, lse);
    if (r == 0) write_stats(out, row, static_cast<double>(cand_value(k)), mL, S, T2);
  }
}

}  // namespace

// Waves of a block.  Up to 512 rows eight: half as many rows in flight as with
// four, with half the work each (256 rows of 151936: 20.5 us against 21.6; 16
// rows of 32000: 9.9 against 10.5; at 512 rows within 4% of each other: 128256, K =
// 8 27.7 against 28.5, 151936, K = 32 35.7 against 35.1).  Above that four waves
// keep the chip as full and finish a row's end beside three other rows of the CU
// (640 rows of 128256: 34.8 us against 37.4; 1024: 46.0 against 49.2).  Sixteen lost
// everywhere (256 rows: 21.2; 512: 60 against 39).  Rows that four waves take in one
// tile each leave eight too little: above one row a CU they take four (512 rows of
// 4100, K = 8: 8.5 us against 9.1; 256 rows 7.8 against 8.0), and rows of one vector
// a lane at any number (one row of 1000, K = 16: 7.1 against 7.5; 512 rows, K = 64:
// 10.6 against 14.4).
static int logits_waves(int rows, int vocab, int splits) {
  if (rows > 2 * kCus || (rows > kCus && (splits > 1 || vocab <= 4 * 8 * kTileVec))) return 4;
  return vocab <= 4 * 8 * kWave ? 4 : 8;
}

// Blocks a row is split over.  A split shortens the longest share of a CU but its
// merge kernel costs about 5 us, so the words that it takes off that share have to
// be worth that.
//   up to 64 rows: one block a CU, for rows of more than six tiles a wave (16 rows of
// 151936: 12.5 us over 16 blocks, 19 over one; 64 rows: 16.1 over 4, 19 over one; of
// 32000, 65536 and 100277: 9.9, 11.5 and 13.8 over one block, 12.4, 11.7 and 12.0
// over many, with K = 32 12.1, 14.6 and 17.0 against 14.4, 15.9 and 17.3)
//   up to 128: the two or three blocks that give one a CU, where they take six tiles
// a wave off a block (K = 8, over one block and split: 85 rows of 151936 18.9 and
// 17.9 us, of 524288 38.3 and 26.9; 128 rows of 151936 18.7 and 19.7, of 200064
// 21.4 and 21.2, of 524288 39.2 and 32.1)
//   up to 170: three, two a CU, by the same line (170 rows of 262144 24.9 and 26.3,
// of 400000 32.7 and 32.4, 129 of 524288 38.7 and 35.5; 171 rows 39.6 and 47.4)
//   257 to 341: a second row goes to few CUs and the others wait for them.  Three
// blocks of four waves, four a CU, from 196608 words (300 rows of 200064 33.8 and
// 31.1 us, of 262144 40.7 and 37.4, with K = 64 48.2 and 48.3, of 524288 73.2 and
// 60.8)
//   up to 384: two, three a CU, from 393216 (342 rows of 262144, K = 64 48.8 and
// 50.1; of 400000, K = 8 58.6 and 53.9)
// Elsewhere a split gives no CU a smaller share, or costs more than it gives.
int logits_splits(const graft_dims &d, int rows) {
  const int64_t nv_row = d.vocab / 8, round = 8 * kTileVec;   // round: a tile for each of 8 waves
  if (rows <= kCus / 4) {
    if (nv_row <= 6 * round) return 1;
    const int64_t s = kCus / rows, max_s = nv_row / kMinSplitVec;   // max_s >= 12
    return static_cast<int>(std::min<int64_t>({s, max_s, kMaxSplits}));
  }
  if (rows <= kCus / 2) {
    const int s = kCus / rows;
    return nv_row * (s - 1) > 6 * round * s ? s : 1;
  }
  if (3 * rows <= 2 * kCus) return nv_row > 18 * round ? 3 : 1;
  if (rows <= kCus) return 1;
  if (3 * rows <= 4 * kCus) return nv_row > 12 * round ? 3 : 1;
  if (2 * rows <= 3 * kCus) return nv_row > 24 * round ? 2 : 1;
  return 1;
}

int logits_part_slots(const graft_dims &d) {
  int64_t best = 0;
  const int max_rows = d.max_batch * d.num_pos;
  for (int b = 1; b <= d.max_batch; ++b) {
    const int rows = b * d.num_pos;
    const int s = logits_splits(d, rows);
    if (s > 1 && static_cast<int64_t>(rows) * s > best) best = static_cast<int64_t>(rows) * s;
  }
  (void)max_rows;
  return static_cast<int>(best > 0 ? best : 1);
}

hipError_t launch_logits_pass(graft_ctx *ctx, const RoundScratch &ws, const graft_round_in *in,
                              const graft_tree_out *out, hipStream_t stream) {
  const int batch = in->batch;
  const uint16_t *logits = in->logits;
  const graft_dims &d = ctx->dims;
  const int rows = batch * d.num_pos;
  const int splits = logits_splits(d, rows);
  if (splits > 1 && static_cast<int64_t>(rows) * splits > ws.part_slots)
    return hipErrorInvalidValue;
  RowOut o;
  o.ids = ws.topk_ids;
  o.logq = ws.topk_logq;
  o.stats = ws.row_stats;
  o.o_ids = out ? out->topk_ids : nullptr;
  o.o_logq = out ? out->topk_logq : nullptr;
  o.o_lse = out ? out->row_lse : nullptr;
  o.o_maxprob = out ? out->row_maxprob : nullptr;
  o.o_ent = out ? out->row_entropy : nullptr;
  // the rows' blocks first, then the runs of hidden-state cosines
  DegenArgs dg{};
  dg.first = static_cast<unsigned>(rows * splits);
  unsigned extra = 0;
  if (in->hidden && d.num_pos > 1) {
    dg.hidden = in->hidden;
    dg.L = d.num_pos;
    dg.H = in->hidden_dim;
    dg.runs = (d.num_pos - 1 + kDegenPairs - 1) / kDegenPairs;
    dg.adj_cos = ws.adj_cos;
    dg.adj_cos_out = out ? out->adj_cos : nullptr;
    extra = static_cast<unsigned>(batch * dg.runs);
  }
  const dim3 grid(dg.first + extra);
  const int V = d.vocab;
  const int waves = logits_waves(rows, V, splits);
  auto pass = [&](auto kernel) {
    hipLaunchKernelGGL(kernel, grid, dim3(waves * kWave), 0, stream, logits, V, splits, d.top_k,
                       ws.part_stats, ws.part_keys, o, dg);
  };
  const bool brief = (V / 8 + splits - 1) / splits <= waves * kTileVec;
  auto by_waves = [&](auto cap) {
    constexpr int C = decltype(cap)::value;
    if (brief) {
      if (waves == 4) pass(short_pass_kernel<C, 4>);
      else pass(short_pass_kernel<C, 8>);
    } else {
      if (waves == 4) pass(logits_pass_kernel<C, 4>);
      else pass(logits_pass_kernel<C, 8>);
    }
  };
  if (d.top_k <= 32) by_waves(std::integral_constant<int, 128>{});
  else by_waves(std::integral_constant<int, 256>{});
  if (splits > 1)
    hipLaunchKernelGGL(merge_kernel, dim3(rows), dim3(kMergeThreads), 0, stream, splits, d.top_k,
                       ws.part_stats, ws.part_keys, o);
  return hipGetLastError();
}

}  // namespace graft
