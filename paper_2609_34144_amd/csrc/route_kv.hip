// Pooled chunk scores and TopK routing on gfx950 (Sec. 4.4 eq:pooled, eq:topk).
//
// route_means  HBM scan: one 8-wave block per (128-channel group, segment), where a
//              segment is an anchor frame of Q or a history chunk of K; fp32 sums of
//              16-byte coalesced bf16 loads, reduced in a fixed order to the pooled
//              means q_bar, k_bar.
// route_topk   one block per (anchor, head): scores s = scale * q_bar . k_bar for
//              all M chunks, then the k_eff best under (score descending, chunk index
//              ascending), written in ascending chunk order.  Above kOneLaunchM chunks
//              the scores (route_scores) and the selection (route_select) are two
//              launches.
// No atomics anywhere: results are bit-identical across runs.
#include "cast_common.h"
#include "topk_select.h"

namespace cast {

namespace {

typedef unsigned int u32x4 __attribute__((ext_vector_type(4)));

// Lane (row r = lane / 16, column = lane % 16) of a wave adds 8 consecutive bf16
// channels of the tokens t0 + r, t0 + r + 4, ... < t1 of a segment, so one load
// instruction reads 4 tokens x 256 contiguous bytes, kFlight of them in flight; then
// the 4 rows are summed by two lane exchanges (a fixed order, so runs are
// bit-identical).  base points at the segment's channel c = the lane's first one.
constexpr int kFlight = 8;   // loads in flight per lane
__device__ __forceinline__ void sum_tokens(const uint16_t* __restrict__ base, int t0, int t1, int row,
                                           int D, bool in, float (&acc)[8]) {
#pragma unroll
  for (int e = 0; e < 8; ++e) acc[e] = 0.0f;
  auto add = [&](const u32x4& v) {
    acc[0] += bf16lo(v.x); acc[1] += bf16hi(v.x);
    acc[2] += bf16lo(v.y); acc[3] += bf16hi(v.y);
    acc[4] += bf16lo(v.z); acc[5] += bf16hi(v.z);
    acc[6] += bf16lo(v.w); acc[7] += bf16hi(v.w);
  };
  if (in) {
    const long long step = (long long)D / 2;        // 4 tokens, in u32x4 units
    const u32x4* p = reinterpret_cast<const u32x4*>(base + (long long)(t0 + row) * D);
    int t = t0 + row;
    for (; t + 4 * (kFlight - 1) < t1; t += 4 * kFlight) {
      u32x4 v[kFlight];
#pragma unroll
      for (int u = 0; u < kFlight; ++u) v[u] = __builtin_nontemporal_load(p + u * step);
#pragma unroll
      for (int u = 0; u < kFlight; ++u) add(v[u]);
      p += kFlight * step;
    }
    for (; t < t1; t += 4) {
      add(__builtin_nontemporal_load(p));
      p += step;
    }
  }
#pragma unroll
  for (int e = 0; e < 8; ++e) {
    acc[e] += __shfl_xor(acc[e], 16);
    acc[e] += __shfl_xor(acc[e], 32);
  }
}

// The segments are the n_a anchor frames of q (S tokens each), then the M history
// chunks of k and (in coupled routing) those of v (Bv tokens each).  A block of
// kMeansWaves waves takes one group of kMeansCh channels of one anchor frame or of PACK
// chunks; kMeansWaves / PACK waves share a segment, wave w of them summing tokens
// [w T / n, (w + 1) T / n), and are added through LDS in wave order.
// HBM-bound: 6.0 TB/s on 32 chunks of 3520 tokens (779 MB).  Short chunks leave
// a wave one or two loads and the dispatcher one workgroup per 16 KB, so on long grids
// two chunks share a workgroup (launch_pool_means has the line).
template <int PACK>
__global__ __launch_bounds__(kMeansWaves * 64) void route_means_kernel(
    const uint16_t* __restrict__ q, const uint16_t* __restrict__ k, const uint16_t* __restrict__ v,
    int n_a, int M, int n_chunks, int S, int Bv, int D, float* __restrict__ means) {
  constexpr int NWC = kMeansWaves / PACK;
  __shared__ float red[kMeansWaves][kMeansCh];
  const int grp = blockIdx.x, y = blockIdx.y;
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const int col = lane & 15, row = lane >> 4;
  const int c = grp * kMeansCh + col * 8;
  const bool anchor = y < n_a;
  const int nw = anchor ? kMeansWaves : NWC;          // waves of this wave's segment
  const int m = (y - n_a) * PACK + wave / NWC;        // its chunk, past the anchors
  const int T = anchor ? S : Bv;
  const uint16_t* base = anchor ? q + (long long)y * S * D
                         : m < M ? k + (long long)m * Bv * D : v + (long long)(m - M) * Bv * D;
  const int w = anchor ? wave : wave % NWC;
  float acc[8];
  sum_tokens(base + c, (int)((long long)T * w / nw), (int)((long long)T * (w + 1) / nw), row, D,
                c < D && (anchor || m < n_chunks), acc);
  if (row == 0) {
#pragma unroll
    for (int e = 0; e < 8; ++e) red[wave][col * 8 + e] = acc[e];
  }
  __syncthreads();
  const int ch = grp * kMeansCh + (threadIdx.x & (kMeansCh - 1));
  const int part = threadIdx.x / kMeansCh;            // 4 x 128 threads
  if (ch >= D) return;
  if (anchor) {
    if (part > 0) return;
    float s = 0.0f;
#pragma unroll
    for (int x = 0; x < kMeansWaves; ++x) s += red[x][threadIdx.x];
    means[(long long)y * D + ch] = s / (float)T;
    return;
  }
  const int mo = (y - n_a) * PACK + part;
  if (part < PACK && mo < n_chunks) {
    float s = 0.0f;
#pragma unroll
    for (int x = 0; x < NWC; ++x) s += red[part * NWC + x][threadIdx.x & (kMeansCh - 1)];
    means[(long long)(n_a + mo) * D + ch] = s / (float)T;
  }
}

// Up to kOneLaunchM chunks: one block of four waves per (anchor i, head h) scores its
// chunks 64 at a time (score_tile, no barrier between the tiles) and its first wave
// selects (topk_words on one wave, KPT keys per lane): one launch, whose latency is
// what counts at this size.  KPT is the smallest that holds the chunks (8 keys per
// lane cost 100 chunks 1.1 us over 4).  The call at 200 chunks of 64 tokens: 34.3 us
// with a lane exchange per four chunks and a rank count over all keys, now 20.5.
template <int DH, int KPT>
__global__ __launch_bounds__(256) void route_topk_kernel(const float* __restrict__ means, int n_a,
                                                         int H, int M, int k_eff, float scale,
                                                         float* __restrict__ scores_out,
                                                         int32_t* __restrict__ idx_out) {
  __shared__ float sc[KPT * 64];
  __shared__ sel::Scratch scratch;
  const int i = blockIdx.x / H, h = blockIdx.x - (blockIdx.x / H) * H;
  const int D = H * DH;
  for (int m0 = 0; m0 < M; m0 += sel::kScoreBlock)
    sel::score_tile<DH, 1>(means, n_a, M, D, h, i, m0, scale, sc + m0, 0);
  __syncthreads();
  if (scores_out)
    for (int m = threadIdx.x; m < M; m += 256) scores_out[((long long)i * H + h) * M + m] = sc[m];
  if (threadIdx.x >= 64) return;
  uint32_t key[KPT];
  bool valid[KPT];
  unsigned long long win[KPT];
#pragma unroll
  for (int j = 0; j < KPT; ++j) {
    const int m = j * 64 + threadIdx.x;
    valid[j] = m < M;
    key[j] = valid[j] ? sel::order_key(sc[m]) : 0u;
  }
  int par = 0;
  sel::topk_words<1, KPT>(key, valid, k_eff, scratch, par, win);
  sel::write_indices<1, KPT>(win, scratch, par, idx_out + ((long long)i * H + h) * k_eff);
}

// More chunks: the scores come from a launch of their own, whose grid (head, 64
// chunks, four anchors) reads every k_bar row once per four anchors from all
// compute units, and one 16-wave block per (anchor, head) selects.  Bound by launch
// and load latency: 1760 chunks, 4 anchors, 24 heads of 128 take 16 us for both
// launches (one block per (anchor, head) that scored four chunks per wave at a time
// and sorted the keys in LDS took 266 us).  The line at kOneLaunchM: 512 chunks run
// 35.2 us a call in one launch and 38.9 in two (24 heads of 128), 300 chunks 18.4
// and 22.9; past it the one block's scoring loop grows by about 2 us per 64 chunks.
template <int DH>
__global__ __launch_bounds__(256) void route_scores_kernel(const float* __restrict__ means, int n_a,
                                                           int H, int M, float scale,
                                                           float* __restrict__ scores,
                                                           float* __restrict__ scores_out) {
  __shared__ float tile[4 * sel::kScoreBlock];
  const int h = blockIdx.x, m0 = blockIdx.y * sel::kScoreBlock, i0 = blockIdx.z * 4;
  const int na = min(4, n_a - i0);
  sel::score_tile<DH, 4>(means, n_a, M, H * DH, h, i0, m0, scale, tile, sel::kScoreBlock);
  __syncthreads();
  const int ii = threadIdx.x >> 6, m = m0 + (threadIdx.x & 63);
  if (ii < na && m < M) {
    const long long o = ((long long)(i0 + ii) * H + h) * M + m;
    const float v = tile[threadIdx.x];
    scores[o] = v;
    if (scores_out) scores_out[o] = v;
  }
}

constexpr int kSelectWaves = 16;
template <int KPT>
__global__ __launch_bounds__(kSelectWaves * 64) void route_select_kernel(
    const float* __restrict__ scores, int M, int k_eff, int32_t* __restrict__ idx_out) {
  __shared__ sel::Scratch scratch;
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const float* s = scores + (long long)blockIdx.x * M;
  uint32_t key[KPT];
  bool valid[KPT];
  unsigned long long win[KPT];
#pragma unroll
  for (int j = 0; j < KPT; ++j) {
    const int m = (wave * KPT + j) * 64 + lane;
    valid[j] = m < M;
    key[j] = valid[j] ? sel::order_key(s[m]) : 0u;
  }
  int par = 0;
  sel::clear_scratch(scratch);
  sel::topk_words<kSelectWaves, KPT>(key, valid, k_eff, scratch, par, win);
  sel::write_indices<kSelectWaves, KPT>(win, scratch, par, idx_out + (long long)blockIdx.x * k_eff);
}

template <int DH>
cast_status_t launch_topk(const float* means, int n_a, int H, int M, int k_eff, float scale,
                          float* scores_out, int32_t* idx_out, float* scores, hipStream_t stream) {
  if (M <= kOneLaunchM) {
    const auto fn = M <= 64 ? route_topk_kernel<DH, 1>
                            : (M <= 256 ? route_topk_kernel<DH, 4> : route_topk_kernel<DH, kOneLaunchM / 64>);
    hipLaunchKernelGGL(fn, dim3(n_a * H), dim3(256), 0, stream, means, n_a, H, M, k_eff, scale,
                       scores_out, idx_out);
    return check_launch("route_topk");
  }
  hipLaunchKernelGGL(route_scores_kernel<DH>,
                     dim3(H, (M + sel::kScoreBlock - 1) / sel::kScoreBlock, (n_a + 3) / 4), dim3(256), 0,
                     stream, means, n_a, H, M, scale, scores, scores_out);
  cast_status_t st = check_launch("route_scores");
  if (st != CAST_OK) return st;
  const dim3 grid(n_a * H), block(kSelectWaves * 64);
  if (M <= kSelectWaves * 64)
    hipLaunchKernelGGL(route_select_kernel<1>, grid, block, 0, stream, scores, M, k_eff, idx_out);
  else if (M <= kSelectWaves * 128)
    hipLaunchKernelGGL(route_select_kernel<2>, grid, block, 0, stream, scores, M, k_eff, idx_out);
  else
    hipLaunchKernelGGL(route_select_kernel<4>, grid, block, 0, stream, scores, M, k_eff, idx_out);
  return check_launch("route_select");
}

}  // namespace

RoutePlan plan_route(int n_a, int S, int H, int dh, int M, int Bv) {
  (void)S;
  (void)Bv;
  RoutePlan p{};
  p.D = H * dh;
  p.segs = n_a + M;
  p.off_means = 0;
  p.off_scores = align_up((size_t)p.segs * p.D * sizeof(float));
  p.total = p.off_scores + (M > kOneLaunchM ? align_up((size_t)n_a * H * M * sizeof(float)) : 0);
  return p;
}

cast_status_t launch_pool_means(const void* q, const void* k, const void* v, int n_a, int S, int M,
                                int Bv, int D, float* means, hipStream_t stream) {
  const int n_chunks = v != nullptr ? 2 * M : M;
  const int groups = (D + kMeansCh - 1) / kMeansCh;
  // Two chunks per workgroup where that is faster: chunks of up to 64 tokens on grids that
  // one workgroup per chunk makes longer than the chip holds at once (eight waves each,
  // about 1024 to 2048 workgroups).  Device times of a routing call, one and two chunks per
  // workgroup, by segments x groups: 64 tokens 1536 12.5 and 13.4 us, 2400 15.1 and 15.0,
  // 3072 18.5 and 17.8, 12288 47.0 and 44.2, 42240 148 and 137; 16 tokens 1536 11.4 and
  // 11.7; 33 tokens 2400 13.6 and 12.4, 12288 40.3 and 33.3.  Longer chunks lose at most
  // sizes (96 tokens 4680 30.9 and 32.0, 128 tokens 24000 136 and 139).
  constexpr int P = 2;
  const bool pack = Bv <= 64 && (long long)n_chunks * groups >= 2048;
  const int rows = n_a + (pack ? (n_chunks + P - 1) / P : n_chunks);
  hipLaunchKernelGGL((pack ? route_means_kernel<P> : route_means_kernel<1>), dim3(groups, rows),
                     dim3(kMeansWaves * 64), 0, stream, static_cast<const uint16_t*>(q),
                     static_cast<const uint16_t*>(k), static_cast<const uint16_t*>(v), n_a, M, n_chunks,
                     S, Bv, D, means);
  return check_launch("route_means");
}

cast_status_t launch_route(const void* q, const void* k, int n_a, int S, int H, int dh, int M,
                           int Bv, int k_eff, float scale, float* scores_out, int32_t* idx_out,
                           const RoutePlan& p, void* ws, hipStream_t stream) {
  float* means = reinterpret_cast<float*>(static_cast<char*>(ws) + p.off_means);
  cast_status_t st = launch_pool_means(q, k, nullptr, n_a, S, M, Bv, p.D, means, stream);
  if (st != CAST_OK) return st;
  float* scores = reinterpret_cast<float*>(static_cast<char*>(ws) + p.off_scores);
  switch (dh) {
    case 32: return launch_topk<32>(means, n_a, H, M, k_eff, scale, scores_out, idx_out, scores, stream);
    case 64: return launch_topk<64>(means, n_a, H, M, k_eff, scale, scores_out, idx_out, scores, stream);
    default: return launch_topk<128>(means, n_a, H, M, k_eff, scale, scores_out, idx_out, scores, stream);
  }
}

}  // namespace cast
