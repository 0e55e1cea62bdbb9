// Reconstruction-coupled historical routing on gfx950 (Sec. 4.4 eq:pooled,
// eq:omission, eq:abc, eq:risk, eq:objective, eq:topk; App. B eq:abcclosed,
// eq:boundarycoeff, eq:gain, eq:boundarygain, Algorithm 1).
//
// route_means (route_kv.hip)   token means of Q, K and V in one launch
// coupled_scores    grid (head, 64 chunks, four anchors): the scores of the tile
//                   and, per anchor, the tile's softmax maximum and sum and its part
//                   of o_bar (unnormalised), which the next launch merges
// coupled_omission  grid (anchor x head, 32 to 128 chunks): o_bar from the parts, then for
//                   each chunk of the range u = (pi/(1-pi+eps))^2 d^T G_h d with
//                   d = o_bar - v_bar[m] (G_h = P_h^T P_h, so ||P_h d||^2 costs dh^2,
//                   not D dh)
// coupled_refine    one workgroup per head (heads never interact): masks start as
//                   TopK(u), then Algorithm 1's directional passes; every lane keeps
//                   its chunks' values in registers and the TopK counts them down
//                   (topk_select.h); the head's objective J is kept up to date by the
//                   accepted gain differences
// wo_gram           G_h from the bf16 output projection (weights only, once per model)
// All reductions run in a fixed order and nothing is atomic: results are
// bit-identical across runs.
#include "cast_common.h"
#include "topk_select.h"

namespace cast {

namespace {

constexpr int kThreads = 256;
// chunks per omission workgroup: its four waves hold dh / 32 row blocks of G times
// 32 chunks each
constexpr int om_chunks(int dh) { return 32 * 4 / (dh / 32); }
typedef float f32x16 __attribute__((ext_vector_type(16)));
// LDS the solver may take besides its static 5 KB: with room, u of the head and its
// square roots (2 n_a M floats) are staged beside the masks
constexpr size_t kRefineLds = 59 * 1024;

struct CoupledArgs {
  const float* means;      // [n_a + 2 M, D]: q_bar rows, then k_bar rows, then v_bar rows
  const float* gram;       // [H, dh, dh]
  float* scores;           // [n_a, H, M] (workspace)
  float* part;             // [n_a, H, n_split, dh + 2]: o_bar part, maximum, sum
  float* u;                // [n_a, H, M] (workspace)
  float* u_out;            // optional copy of u
  int32_t* idx_out;        // [n_a, H, k_eff]
  int n_a, H, M, D, k_eff, n_frames, passes, n_split;
  float scale, l_anc, l_rec, tol, eps;
  short anchors[kCoupledMaxAnchors];
};

// Sum over the 64 lanes of a wave, the same on every lane, in a fixed order: row
// shifts and row broadcasts (DPP adds: no LDS round trip per step, which in the
// solver's serial chain cost as much as the rest of a step), lane 63 holds the total.
template <int CTRL, int ROWS>
__device__ __forceinline__ float dpp_add(float v) {
  return v + __builtin_bit_cast(float, __builtin_amdgcn_update_dpp(0, __builtin_bit_cast(int, v), CTRL, ROWS,
                                                                   0xf, true));
}
__device__ __forceinline__ float wave_sum(float v) {
  v = dpp_add<0x111, 0xf>(v);   // row_shr:1
  v = dpp_add<0x112, 0xf>(v);   // row_shr:2
  v = dpp_add<0x114, 0xf>(v);   // row_shr:4
  v = dpp_add<0x118, 0xf>(v);   // row_shr:8: lane 15 of each row holds the row's sum
  v = dpp_add<0x142, 0xa>(v);   // row_bcast:15 into rows 1 and 3
  v = dpp_add<0x143, 0xc>(v);   // row_bcast:31 into rows 2 and 3
  return __builtin_bit_cast(float, __builtin_amdgcn_readlane(__builtin_bit_cast(int, v), 63));
}
__device__ __forceinline__ float wave_max(float v) {
  for (int o = 32; o > 0; o >>= 1) v = fmaxf(v, __shfl_xor(v, o));
  return v;
}

// ---------------------------------------------------------------------------
// scores, softmax parts and o_bar parts (eq:pooled)
// ---------------------------------------------------------------------------
// Every k_bar and v_bar row is read once per four anchors, and the grid fills the
// chip (24 heads x 28 tiles at 1760 chunks); scoring all chunks again in every
// omission workgroup took 134 us at 390 chunks, 3 anchors and 12 heads of 128.
template <int DH>
__global__ __launch_bounds__(kThreads) void coupled_scores_kernel(CoupledArgs a) {
  constexpr int NP = kThreads / DH;              // parts of the tile's chunks in o_bar
  constexpr int CP = sel::kScoreBlock / NP;      // chunks per part
  __shared__ float tile[4 * sel::kScoreBlock];
  __shared__ float red[NP][4][DH];
  const int h = blockIdx.x, sp = blockIdx.y, m0 = sp * sel::kScoreBlock, i0 = blockIdx.z * 4;
  const int na = min(4, a.n_a - i0), nm = min(sel::kScoreBlock, a.M - m0);
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  sel::score_tile<DH, 4>(a.means, a.n_a, a.M, a.D, h, i0, m0, a.scale, tile, sel::kScoreBlock);
  __syncthreads();
  // wave w takes anchor i0 + w: maximum, unnormalised probabilities and their sum
  if (wave < na) {
    const long long ih = (long long)(i0 + wave) * a.H + h;
    const float sc = tile[tid];
    const bool in = lane < nm;
    if (in) a.scores[ih * a.M + m0 + lane] = sc;
    const float mx = wave_max(in ? sc : -INFINITY);
    // a score of -inf adds nothing, also where the tile has no other (-inf - mx would be
    // NaN there, and the tile's weight of 0 in the merge would not remove it)
    const float e = in && sc != -INFINITY ? expf(sc - mx) : 0.0f;
    const float sum = wave_sum(e);
    tile[tid] = e;
    if (lane == 0) {
      float* p = a.part + (ih * a.n_split + sp) * (DH + 2) + DH;
      p[0] = mx;
      p[1] = sum;
    }
  }
  __syncthreads();
  // thread -> (channel, part of the chunks), all four anchors; parts in a fixed order
  {
    const int d = tid % DH, part = tid / DH;
    const float* v = a.means + (long long)(a.n_a + a.M + m0) * a.D + h * DH + d;
    const int c0 = part * CP, c1 = min(c0 + CP, nm);
    float acc[4] = {0.0f, 0.0f, 0.0f, 0.0f};
#pragma unroll 8
    for (int c = c0; c < c1; ++c) {
      const float x = v[(long long)c * a.D];
#pragma unroll
      for (int ii = 0; ii < 4; ++ii) acc[ii] = fmaf(tile[ii * sel::kScoreBlock + c], x, acc[ii]);
    }
#pragma unroll
    for (int ii = 0; ii < 4; ++ii) red[part][ii][d] = acc[ii];
  }
  __syncthreads();
  for (int x = tid; x < na * DH; x += kThreads) {
    const int ii = x / DH, d = x - ii * DH;
    float o = 0.0f;
#pragma unroll
    for (int p = 0; p < NP; ++p) o += red[p][ii][d];
    a.part[(((long long)(i0 + ii) * a.H + h) * a.n_split + sp) * (DH + 2) + d] = o;
  }
}

// ---------------------------------------------------------------------------
// omission proxy u (eq:omission)
// ---------------------------------------------------------------------------
// y = G d for the range's difference vectors on the matrix cores in fp32
// (v_mfma_f32_32x32x2_f32, exact products and fp32 accumulation): wave w takes 32 rows
// of G (by symmetry its columns, so the loads coalesce) and 32 vectors, one vector per
// lane column, so d . y is the lane's own sum.  Its G operand (DH floats per lane) is
// loaded whole at the start, in flight during the o_bar merge.  Bound by that load and
// the launch at few chunks, by the fp32 MFMA rate at many.
template <int DH>
__global__ __launch_bounds__(kThreads) void coupled_omission_kernel(CoupledArgs a) {
  constexpr int RB = DH / 32;                    // 32-row blocks of G
  constexpr int NV = om_chunks(DH);              // vectors (chunks) of the workgroup
  constexpr int NP = kThreads / DH;
  constexpr int DS = NV + 4;                     // row stride of the transposed vectors
  constexpr int kMaxSplit = kRouteMaxM / sel::kScoreBlock;
  __shared__ float dt[DH * DS];                  // dt[c][vector]
  __shared__ float ob[DH], red[NP][DH], fac[kMaxSplit], norm[2], quad[RB][NV];
  const int ih = blockIdx.x, h = ih % a.H;
  const int m0 = blockIdx.y * NV;
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int l32 = lane & 31, hf = lane >> 5;
  const int r0 = (wave % RB) * 32, v0 = (wave / RB) * 32;
  // operand A of MFMA step t: row r0 + l32, column 2 t + hf
  float g[DH / 2];
  {
    const float* G = a.gram + (long long)h * DH * DH + hf * DH + r0 + l32;
#pragma unroll
    for (int t = 0; t < DH / 2; ++t) g[t] = G[2 * t * DH];
  }
  const float* part = a.part + (long long)ih * a.n_split * (DH + 2);
  // o_bar from the tiles' parts: weights exp(max_s - max) over the sum of all
  if (wave == 0) {
    const bool in = lane < a.n_split;
    const float mx = in ? part[lane * (DH + 2) + DH] : -INFINITY;
    const float sm = in ? part[lane * (DH + 2) + DH + 1] : 0.0f;
    const float smax = wave_max(mx);
    const float f = in ? expf(mx - smax) : 0.0f;
    const float ssum = wave_sum(f * sm);
    fac[lane] = f;
    if (lane == 0) {
      norm[0] = smax;
      norm[1] = ssum;
    }
  }
  __syncthreads();
  {
    const int d = tid % DH, p = tid / DH;
    float acc = 0.0f;
#pragma unroll 4
    for (int s = p; s < a.n_split; s += NP) acc = fmaf(fac[s], part[s * (DH + 2) + d], acc);
    red[p][d] = acc;
  }
  __syncthreads();
  const float smax = norm[0], ssum = norm[1];
  if (tid < DH) {
    float o = 0.0f;
#pragma unroll
    for (int p = 0; p < NP; ++p) o += red[p][tid];
    ob[tid] = o / ssum;
  }
  __syncthreads();
  const float* vm = a.means + (long long)(a.n_a + a.M) * a.D + h * DH;
#pragma unroll 8
  for (int x = tid; x < NV * DH; x += kThreads) {
    const int j = x / DH, c = x - j * DH;
    dt[c * DS + j] = ob[c] - vm[(long long)min(m0 + j, a.M - 1) * a.D + c];
  }
  __syncthreads();
  const float* dv = dt + v0 + l32;               // this lane's vector
  f32x16 y{};
#pragma unroll
  for (int t = 0; t < DH / 2; ++t)
    y = __builtin_amdgcn_mfma_f32_32x32x2f32(g[t], dv[(2 * t + hf) * DS], y, 0, 0, 0);
  // element e of the accumulator: row r0 + 8 (e / 4) + 4 hf + e % 4, the lane's vector
  float qs[4] = {0.0f, 0.0f, 0.0f, 0.0f};
#pragma unroll
  for (int e = 0; e < 16; ++e) qs[e % 4] = fmaf(dv[(r0 + 8 * (e / 4) + 4 * hf + e % 4) * DS], y[e], qs[e % 4]);
  float q = (qs[0] + qs[1]) + (qs[2] + qs[3]);
  q += __shfl_xor(q, 32);
  if (hf == 0) quad[wave % RB][v0 + l32] = q;
  __syncthreads();
  const int m = m0 + tid;
  if (tid < NV && m < a.M) {
    float d2 = 0.0f;
#pragma unroll
    for (int r = 0; r < RB; ++r) d2 += quad[r][tid];
    const long long o = (long long)ih * a.M + m;
    const float pi = expf(a.scores[o] - smax) / ssum;
    const float cf = pi / (1.0f - pi + a.eps);
    const float u = cf * cf * d2;
    a.u[o] = u;
    if (a.u_out) a.u_out[o] = u;
  }
}

// ---------------------------------------------------------------------------
// Algorithm 1 (eq:gain, eq:boundarygain, eq:topk)
// ---------------------------------------------------------------------------
struct Coeffs {
  // interval (rows j, j+1): A = B, C from the closed form of eq:abcclosed
  // boundary sides (eq:boundarycoeff): rows (ra, rb) and sums over their frames
  int has_l, has_r;
  float al, bl, cl, ar, br, cr;
};

// The solver is a serial chain of small selections and sums, bound by latency.  Lane
// l, slot j of wave w owns chunk m = ((w KPT) + j) 64 + l of every row, so gains,
// masks (one 64-bit word per row and slot) and u are touched only by their owner and
// the waves meet only in the sums and the selection's counts (refine_for chooses how
// many; a single wave runs without a barrier).  (Sorting the keys in LDS and editing the
// masks from one lane took 589 us at 390 chunks, 3 anchors, 78 kept; 52 us at 32
// chunks and 4 anchors.)
template <int NW, int KPT, bool CACHE_U>
__global__ __launch_bounds__(NW * 64) void coupled_refine_kernel(CoupledArgs a) {
  extern __shared__ unsigned long long xm[];          // [n_a][NW * KPT] retain words
  constexpr int WORDS = NW * KPT;
  const int M = a.M, n_a = a.n_a, k = a.k_eff, h = blockIdx.x;
  float* su = reinterpret_cast<float*>(xm + n_a * WORDS);   // [n_a][M] u of this head (CACHE_U)
  float* sq = su + (CACHE_U ? n_a * M : 0);                 // its square roots
  __shared__ Coeffs cf;
  __shared__ float pair_ab[kCoupledMaxAnchors], pair_c[kCoupledMaxAnchors];
  __shared__ sel::Scratch scratch;
  const int tid = threadIdx.x, lane = tid & 63, wave = NW == 1 ? 0 : tid >> 6;
  const int mb = wave * KPT * 64 + lane;              // this lane's chunks: mb + 64 j
  // slots past the last chunk read it and are masked out, so that a row's loads are
  // all in flight together
  bool valid[KPT];
  int mc[KPT];
#pragma unroll
  for (int j = 0; j < KPT; ++j) {
    valid[j] = mb + 64 * j < M;
    mc[j] = min(mb + 64 * j, M - 1);
  }
  const float* gu = a.u + (long long)h * M;
  const long long urow = (long long)a.H * M;
  if constexpr (CACHE_U)
    for (int i = 0; i < n_a; ++i)
#pragma unroll
      for (int j = 0; j < KPT; ++j)
        if (valid[j]) {
          const float x = gu[i * urow + mc[j]];
          su[i * M + mc[j]] = x;
          sq[i * M + mc[j]] = sqrtf(x);
        }
  auto U = [&](int i, int j) -> float {
    if constexpr (CACHE_U) return su[i * M + mc[j]];
    else return gu[i * urow + mc[j]];
  };
  auto R = [&](int i, int j) -> float {
    if constexpr (CACHE_U) return sq[i * M + mc[j]];
    else return sqrtf(gu[i * urow + mc[j]]);
  };
  auto X = [&](int i, int j) -> float {
    return (xm[i * WORDS + wave * KPT + j] >> lane) & 1ull ? 1.0f : 0.0f;
  };

  // ---- coefficients
  for (int j = tid; j + 1 < n_a; j += NW * 64) {
    const float n = (float)(a.anchors[j + 1] - a.anchors[j]);
    pair_ab[j] = (n - 1.0f) * (2.0f * n - 1.0f) / (6.0f * n);
    pair_c[j] = (n * n - 1.0f) / (6.0f * n);
  }
  if (tid == 0) {
    Coeffs c{};
    if (n_a >= 2) {
      const int a0 = a.anchors[0], a1 = a.anchors[1];
      const int b0 = a.anchors[n_a - 2], b1 = a.anchors[n_a - 1];
      for (int t = 0; t < a0; ++t) {
        const float al = (float)(t - a0) / (float)(a1 - a0);
        c.al += (1.0f - al) * (1.0f - al);
        c.bl += al * al;
        c.cl += fabsf(al * (1.0f - al));
      }
      for (int t = b1 + 1; t < a.n_frames; ++t) {
        const float al = (float)(t - b0) / (float)(b1 - b0);
        c.ar += (1.0f - al) * (1.0f - al);
        c.br += al * al;
        c.cr += fabsf(al * (1.0f - al));
      }
      c.has_l = a0 > 0;
      c.has_r = b1 < a.n_frames - 1;
    }
    cf = c;
  }
  sel::clear_scratch(scratch);

  int par = 0;
  // sums of two values over the workgroup, the same on every thread
  auto group_sum2 = [&](float& x, float& y) {
    x = wave_sum(x);
    y = wave_sum(y);
    if constexpr (NW > 1) {
      if (lane == 0) {
        scratch.sum[par & 1][wave][0] = x;
        scratch.sum[par & 1][wave][1] = y;
      }
      __syncthreads();
      x = scratch.sum[par & 1][lane % NW][0];
      y = scratch.sum[par & 1][lane % NW][1];
#pragma unroll
      for (int o = NW / 2; o > 0; o >>= 1) {
        x += __shfl_xor(x, o);
        y += __shfl_xor(y, o);
      }
      if (tid == 0) scratch.cnt[(par + 2) & 3] = 0ull;   // (keeps the ring's turn)
      ++par;
    }
  };
  auto store_words = [&](int i, const unsigned long long (&win)[KPT]) {
    if (lane == 0) {
#pragma unroll
      for (int j = 0; j < KPT; ++j) xm[i * WORDS + wave * KPT + j] = win[j];
    }
    // the owner wave alone reads these words back
    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
    __builtin_amdgcn_wave_barrier();
  };

  // ---- initial masks: TopK(u) per anchor
  uint32_t key[KPT];
  unsigned long long win[KPT];
  for (int i = 0; i < n_a; ++i) {
#pragma unroll
    for (int j = 0; j < KPT; ++j) key[j] = valid[j] ? sel::order_key(U(i, j)) : 0u;
    sel::topk_words<NW, KPT>(key, valid, k, scratch, par, win);
    store_words(i, win);
  }

  // ---- objective J of the head (eq:objective with eq:risk and eq:boundaryrisk)
  auto risk = [&](int ra, int rb, float A, float B, float C, int j) -> float {
    const float oa = 1.0f - X(ra, j), ob = 1.0f - X(rb, j);
    return A * oa * U(ra, j) + B * ob * U(rb, j) + 2.0f * C * oa * ob * R(ra, j) * R(rb, j);
  };
  float J = 0.0f;
  {
    float unused = 0.0f;
#pragma unroll
    for (int j = 0; j < KPT; ++j) {
      float anc = 0.0f, rec = 0.0f;
      for (int i = 0; i < n_a; ++i) anc += (1.0f - X(i, j)) * U(i, j);
      for (int p = 0; p + 1 < n_a; ++p) rec += risk(p, p + 1, pair_ab[p], pair_ab[p], pair_c[p], j);
      if (cf.has_l) rec += risk(0, 1, cf.al, cf.bl, cf.cl, j);
      if (cf.has_r) rec += risk(n_a - 2, n_a - 1, cf.ar, cf.br, cf.cr, j);
      J += valid[j] ? a.l_anc * anc + a.l_rec * rec : 0.0f;
    }
    group_sum2(J, unused);
  }

  // ---- directional passes
  for (int s = 0; s < a.passes && k < M; ++s) {
    bool changed = false;
    for (int v = 0; v < n_a; ++v) {
      const int i = (s % 2 == 0) ? v : n_a - 1 - v;
      float g[KPT];
      float g_old = 0.0f, g_new = 0.0f;
#pragma unroll
      for (int j = 0; j < KPT; ++j) {
        const float ui = U(i, j), si = R(i, j);
        float rec = 0.0f;
        if (i > 0) rec += pair_ab[i - 1] * ui + 2.0f * pair_c[i - 1] * (1.0f - X(i - 1, j)) * R(i - 1, j) * si;
        if (i + 1 < n_a) rec += pair_ab[i] * ui + 2.0f * pair_c[i] * (1.0f - X(i + 1, j)) * si * R(i + 1, j);
        if (cf.has_l) {
          if (i == 0) rec += cf.al * ui + 2.0f * cf.cl * (1.0f - X(1, j)) * si * R(1, j);
          if (i == 1) rec += cf.bl * ui + 2.0f * cf.cl * (1.0f - X(0, j)) * si * R(0, j);
        }
        if (cf.has_r) {
          if (i == n_a - 2) rec += cf.ar * ui + 2.0f * cf.cr * (1.0f - X(n_a - 1, j)) * si * R(n_a - 1, j);
          if (i == n_a - 1) rec += cf.br * ui + 2.0f * cf.cr * (1.0f - X(n_a - 2, j)) * si * R(n_a - 2, j);
        }
        g[j] = a.l_anc * ui + a.l_rec * rec;
        key[j] = valid[j] ? sel::order_key(g[j]) : 0u;
        g_old += (xm[i * WORDS + wave * KPT + j] >> lane) & 1ull ? g[j] : 0.0f;
      }
      sel::topk_words<NW, KPT>(key, valid, k, scratch, par, win);
#pragma unroll
      for (int j = 0; j < KPT; ++j) g_new += (win[j] >> lane) & 1ull ? g[j] : 0.0f;
      group_sum2(g_old, g_new);
      const float gain = g_new - g_old;
      if (gain > a.tol * fmaxf(J, 1e-8f)) {   // uniform: every thread holds the same sums
        store_words(i, win);
        J -= gain;
        changed = true;
      }
    }
    if (!changed) break;
  }

  // ---- ascending block indices of every mask
  for (int i = 0; i < n_a; ++i) {
#pragma unroll
    for (int j = 0; j < KPT; ++j) win[j] = xm[i * WORDS + wave * KPT + j];
    sel::write_indices<NW, KPT>(win, scratch, par, a.idx_out + ((long long)i * a.H + h) * k);
  }
}

typedef void (*RefineFn)(CoupledArgs);
template <int NW, int KPT>
RefineFn refine_fn(bool cache_u, int& waves, int& words) {
  waves = NW;
  words = NW * KPT;
  return cache_u ? coupled_refine_kernel<NW, KPT, true> : coupled_refine_kernel<NW, KPT, false>;
}
// The solver of M chunks.  Up to 128 chunks one wave (100 chunks, 3 anchors: 18 us,
// four waves 24); to 512 four waves of one or two chunks per lane (390 chunks, 78 kept,
// 3 anchors: 31 us, one wave with eight per lane 45); above, eight waves (1760 chunks,
// 352 kept, 4 anchors: 74 us, sixteen waves 76).
RefineFn refine_for(int M, bool cache_u, int& waves, int& words) {
  if (M <= 64) return refine_fn<1, 1>(cache_u, waves, words);
  if (M <= 128) return refine_fn<1, 2>(cache_u, waves, words);
  if (M <= 256) return refine_fn<4, 1>(cache_u, waves, words);
  if (M <= 512) return refine_fn<4, 2>(cache_u, waves, words);
  if (M <= 1024) return refine_fn<8, 2>(cache_u, waves, words);
  if (M <= 2048) return refine_fn<8, 4>(cache_u, waves, words);
  static_assert(kRouteMaxM <= 8 * 8 * 64, "the largest solver holds every chunk");
  return refine_fn<8, 8>(cache_u, waves, words);
}

// ---------------------------------------------------------------------------
// Gram matrices of the head slices of W_O
// ---------------------------------------------------------------------------
template <int DH>
__global__ __launch_bounds__(kThreads) void wo_gram_kernel(const uint16_t* __restrict__ w, int D,
                                                           float* __restrict__ gram) {
  constexpr int RB = 16;                 // G rows per workgroup
  constexpr int NB = DH * RB / kThreads; // outputs per thread
  constexpr int CH = 64;                 // W rows staged per step
  __shared__ float tile[CH][DH];
  const int h = blockIdx.x, rb = blockIdx.y, tid = threadIdx.x;
  const int ra = rb * RB + tid / (kThreads / RB);         // this thread's G row
  const int c0 = tid % (kThreads / RB);                   // first column, stride kThreads / RB
  float acc[NB];
#pragma unroll
  for (int j = 0; j < NB; ++j) acc[j] = 0.0f;
  for (int r0 = 0; r0 < D; r0 += CH) {
    for (int x = tid; x < CH * DH; x += kThreads) {
      const int rr = x / DH, cc = x - (x / DH) * DH;
      const int r = r0 + rr;
      tile[rr][cc] = r < D ? __uint_as_float((uint32_t)w[(long long)r * D + h * DH + cc] << 16) : 0.0f;
    }
    __syncthreads();
    for (int rr = 0; rr < CH; ++rr) {
      const float av = tile[rr][ra];
#pragma unroll
      for (int j = 0; j < NB; ++j) acc[j] = fmaf(av, tile[rr][c0 + j * (kThreads / RB)], acc[j]);
    }
    __syncthreads();
  }
#pragma unroll
  for (int j = 0; j < NB; ++j)
    gram[((long long)h * DH + ra) * DH + c0 + j * (kThreads / RB)] = acc[j];
}

}  // namespace

CoupledPlan plan_coupled(int n_a, int S, int H, int dh, int M, int Bv) {
  (void)S;
  (void)Bv;
  CoupledPlan p{};
  const size_t D = (size_t)H * dh, rows = (size_t)n_a * H;
  p.n_split = (M + sel::kScoreBlock - 1) / sel::kScoreBlock;
  p.off_means = 0;
  p.off_scores = align_up((n_a + 2 * (size_t)M) * D * sizeof(float));
  p.off_part = p.off_scores + align_up(rows * M * sizeof(float));
  p.off_u = p.off_part + align_up(rows * p.n_split * (dh + 2) * sizeof(float));
  p.total = p.off_u + align_up(rows * M * sizeof(float));
  return p;
}

cast_status_t launch_coupled(const void* q, const void* k, const void* v, const float* gram,
                             const int* anchors, int n_a, int n_frames, int S, int H, int dh,
                             int M, int Bv, int k_eff, float scale, const cast_coupled_params_t& prm,
                             float* u_out, int32_t* idx_out, const CoupledPlan& p, void* ws,
                             hipStream_t stream) {
  char* base = static_cast<char*>(ws);
  CoupledArgs a{};
  float* means = reinterpret_cast<float*>(base + p.off_means);
  a.means = means;
  a.gram = gram;
  a.scores = reinterpret_cast<float*>(base + p.off_scores);
  a.part = reinterpret_cast<float*>(base + p.off_part);
  a.n_split = p.n_split;
  a.u = reinterpret_cast<float*>(base + p.off_u);
  a.u_out = u_out;
  a.idx_out = idx_out;
  a.n_a = n_a;
  a.H = H;
  a.M = M;
  a.D = H * dh;
  a.k_eff = k_eff;
  a.n_frames = n_frames;
  a.passes = prm.passes;
  a.scale = scale;
  a.l_anc = prm.l_anc;
  a.l_rec = prm.l_rec;
  a.tol = prm.tol;
  a.eps = prm.eps;
  for (int j = 0; j < n_a; ++j) a.anchors[j] = (short)anchors[j];
  cast_status_t st = launch_pool_means(q, k, v, n_a, S, M, Bv, a.D, means, stream);
  if (st != CAST_OK) return st;
  const dim3 sgrid(H, p.n_split, (n_a + 3) / 4);
  const dim3 ogrid(n_a * H, (M + om_chunks(dh) - 1) / om_chunks(dh));
  switch (dh) {
    case 32:
      hipLaunchKernelGGL(coupled_scores_kernel<32>, sgrid, dim3(kThreads), 0, stream, a);
      hipLaunchKernelGGL(coupled_omission_kernel<32>, ogrid, dim3(kThreads), 0, stream, a);
      break;
    case 64:
      hipLaunchKernelGGL(coupled_scores_kernel<64>, sgrid, dim3(kThreads), 0, stream, a);
      hipLaunchKernelGGL(coupled_omission_kernel<64>, ogrid, dim3(kThreads), 0, stream, a);
      break;
    default:
      hipLaunchKernelGGL(coupled_scores_kernel<128>, sgrid, dim3(kThreads), 0, stream, a);
      hipLaunchKernelGGL(coupled_omission_kernel<128>, ogrid, dim3(kThreads), 0, stream, a);
      break;
  }
  st = check_launch("coupled_omission");
  if (st != CAST_OK) return st;
  int waves = 0, words = 0;
  RefineFn fn = refine_for(M, true, waves, words);
  size_t shm = (size_t)n_a * words * 8;
  if (shm + (size_t)n_a * M * 8 <= kRefineLds) shm += (size_t)n_a * M * 8;
  else fn = refine_for(M, false, waves, words);
  hipLaunchKernelGGL(fn, dim3(H), dim3(waves * 64), shm, stream, a);
  return check_launch("coupled_refine");
}

cast_status_t launch_wo_gram(const void* w_o, int D, int H, int dh, float* gram, hipStream_t stream) {
  const uint16_t* w = static_cast<const uint16_t*>(w_o);
  const dim3 grid(H, dh / 16);
  switch (dh) {
    case 32: hipLaunchKernelGGL(wo_gram_kernel<32>, grid, dim3(kThreads), 0, stream, w, D, gram); break;
    case 64: hipLaunchKernelGGL(wo_gram_kernel<64>, grid, dim3(kThreads), 0, stream, w, D, gram); break;
    default: hipLaunchKernelGGL(wo_gram_kernel<128>, grid, dim3(kThreads), 0, stream, w, D, gram); break;
  }
  return check_launch("wo_gram");
}

}  // namespace cast
