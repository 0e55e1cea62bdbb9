// TopK selection without a sort, shared by the routing and the coupled-routing
// kernels: the k largest of up to NW * 64 * KPT values under the total order (value
// descending, index ascending), as one winner bit per value.
//
// A group of NW waves holds the values in registers: wave w, lane l, slot j holds
// index ((w KPT) + j) 64 + l, so slot j's ballot is one 64-bit word of the winner
// mask and words follow each other in ascending index order.  The k-th largest key
// is found from its top bit down by counting the keys at or above a candidate
// (ballots and popcounts), and the walk ends early once a candidate keeps exactly k.
// One wave walks bit by bit with no barrier (up to kRankN values it ranks them instead);
// several waves take two bits per step, one LDS exchange of packed counts each.  Everything is integer work: results do
// not depend on the schedule.
#pragma once

#include "cast_common.h"

namespace cast {
namespace sel {

constexpr int kScoreBlock = 64;   // chunks per score workgroup

// Value key, monotone in v; -0 and +0 compare equal and get one key.
__device__ __forceinline__ uint32_t order_key(float v) {
  uint32_t b = __float_as_uint(v);
  if ((b << 1) == 0u) b = 0u;
  return (b & 0x80000000u) ? ~b : (b | 0x80000000u);
}

// LDS scratch of one group (NW > 1 only; clear_scratch before first use).  cnt is a
// ring of four packed-count slots: a step adds into slot r, meets at a barrier and
// reads it, and clears slot r + 2, which every wave has read before that barrier.
struct Scratch {
  unsigned long long cnt[4];
  float sum[2][16][2];
  int word[2][16];
};
__device__ __forceinline__ void clear_scratch(Scratch& s) {
  if (threadIdx.x < 4) s.cnt[threadIdx.x] = 0ull;
  __syncthreads();
}

template <int KPT>
__device__ __forceinline__ int count_ge(const uint32_t (&key)[KPT], uint32_t c) {
  int n = 0;
#pragma unroll
  for (int j = 0; j < KPT; ++j) n += __popcll(__ballot(key[j] >= c));
  return n;
}

// Number of set winner bits of the waves before this one, and of all waves.
template <int NW>
__device__ __forceinline__ void wave_prefix(int mine, Scratch& s, int& par, int& before, int& total) {
  if constexpr (NW == 1) {
    before = 0;
    total = mine;
  } else {
    const int wave = threadIdx.x >> 6;
    if ((threadIdx.x & 63) == 0) s.word[par & 1][wave] = mine;
    __syncthreads();
    before = total = 0;
#pragma unroll
    for (int w = 0; w < NW; ++w) {
      const int c = s.word[par & 1][w];
      before += w < wave ? c : 0;
      total += c;
    }
    if (threadIdx.x == 0) s.cnt[(par + 2) & 3] = 0ull;   // (keeps the ring's turn)
    ++par;
  }
}

// Few values in one wave, one per lane (lanes 0 .. n - 1): each lane counts the larger
// keys, and where equals straddle the k-th place the lower lanes take it.  A walk has the
// keys' common leading bits to pass first, and all 32 where equals straddle: routing's
// call over 2 chunks, 4 anchors, 12 heads of 128 7.3 us of device time ranked and 7.75
// walked, over 32 chunks 8.0 and 8.2, over 48 8.16 and 8.07, over 64 9.7 and 9.4; frame
// selection by age alone 2.1 and 3.5 us at 4 frames, 3.0 and 3.6 at 40.  Keeping every
// value, the walk ends at its first bit.
constexpr int kRankN = 40;
__device__ __forceinline__ void rank_word(uint32_t key, bool valid, int n, int k, unsigned long long& win) {
  int above = 0;
  for (int j = 0; j < n; j += 8) {   // (lanes past n hold key 0)
#pragma unroll
    for (int u = 0; u < 8; ++u) above += (uint32_t)__builtin_amdgcn_readlane((int)key, j + u) > key ? 1 : 0;
  }
  win = __ballot(valid && above < k);
  if (__popcll(win) <= k) return;
  int last = valid && above < k ? above : -1;   // the place of the equals
  for (int o = 32; o > 0; o >>= 1) last = max(last, __shfl_xor(last, o));
  const unsigned long long eq = __ballot(valid && above == last);
  const int lane = threadIdx.x & 63;
  const bool in = above < last || (above == last && __popcll(eq & ((1ull << lane) - 1ull)) < k - last);
  win = __ballot(valid && in);
}

// Winner words of this wave's slots: win[j] bit l set when the value at (wave, j, l)
// is among the k largest.  Slots past the n values carry key 0 and valid = false;
// 1 <= k <= n.  `par` counts the group's exchanges, which take their LDS
// buffers by it (start at 0, keep across calls).
template <int NW, int KPT>
__device__ __forceinline__ void topk_words(const uint32_t (&key)[KPT], const bool (&valid)[KPT], int k,
                                           Scratch& s, int& par, unsigned long long (&win)[KPT]) {
  if constexpr (NW == 1 && KPT == 1) {
    const int n = 64 - __clzll(__ballot(valid[0]));
    if (n <= kRankN && k < n) {
      rank_word(key[0], valid[0], n, k, win[0]);
      return;
    }
  }
  uint32_t t = 0;
  bool exact = false;
  int above = 0;   // values strictly above t once the walk ends without `exact`
  if constexpr (NW == 1) {
    for (int b = 31; b >= 0 && !exact; --b) {
      const uint32_t c = t | (1u << b);
      const int n = count_ge(key, c);
      if (n >= k) t = c;
      exact = n == k;
    }
  } else {
    for (int b = 30; b >= 0 && !exact; b -= 2) {
      const uint32_t c1 = t | (1u << b), c2 = t | (2u << b), c3 = t | (3u << b);
      const unsigned long long mine = (unsigned long long)count_ge(key, c1) |
                                      ((unsigned long long)count_ge(key, c2) << 16) |
                                      ((unsigned long long)count_ge(key, c3) << 32);
      // one integer add per wave, one read: 16 waves that each read 16 counts would
      // hold the LDS for longer than the rest of the step takes
      if ((threadIdx.x & 63) == 0) atomicAdd(&s.cnt[par & 3], mine);
      __syncthreads();
      const unsigned long long all = s.cnt[par & 3];
      if (threadIdx.x == 0) s.cnt[(par + 2) & 3] = 0ull;
      ++par;
      const int n1 = (int)(all & 0xffff), n2 = (int)((all >> 16) & 0xffff), n3 = (int)(all >> 32);
      if (n3 >= k) t = c3;
      else if (n2 >= k) t = c2;
      else if (n1 >= k) t = c1;
      exact = n3 == k || (n3 < k && n2 == k) || (n2 < k && n1 == k);
    }
  }
  if (exact) {
#pragma unroll
    for (int j = 0; j < KPT; ++j) win[j] = __ballot(valid[j] && key[j] >= t);
    return;
  }
  // t is the k-th largest key: all above it win, then its equals by ascending index
  unsigned long long eq[KPT];
  int gt = 0, neq = 0;
#pragma unroll
  for (int j = 0; j < KPT; ++j) {
    win[j] = __ballot(valid[j] && key[j] > t);
    eq[j] = __ballot(valid[j] && key[j] == t);
    gt += __popcll(win[j]);
    neq += __popcll(eq[j]);
  }
  int before, total;
  wave_prefix<NW>(gt, s, par, before, above);
  wave_prefix<NW>(neq, s, par, before, total);
  int room = k - above - before;   // equals this wave may still take
#pragma unroll
  for (int j = 0; j < KPT; ++j) {
    const int lane = threadIdx.x & 63;
    const int rank = __popcll(eq[j] & ((1ull << lane) - 1ull));
    win[j] |= __ballot(((eq[j] >> lane) & 1ull) && rank < room);
    room -= __popcll(eq[j]);
  }
}

// Writes the indices of the set winner bits in ascending order to dst, the first `most`.
template <int NW, int KPT>
__device__ __forceinline__ void write_indices(const unsigned long long (&win)[KPT], Scratch& s, int& par,
                                              int32_t* __restrict__ dst, int most = 1 << 30) {
  int mine = 0;
#pragma unroll
  for (int j = 0; j < KPT; ++j) mine += __popcll(win[j]);
  int pos, total;
  wave_prefix<NW>(mine, s, par, pos, total);
  const int lane = threadIdx.x & 63;
  const int wave = NW == 1 ? 0 : (int)(threadIdx.x >> 6);
#pragma unroll
  for (int j = 0; j < KPT; ++j) {
    const int at = pos + __popcll(win[j] & ((1ull << lane) - 1ull));
    if (((win[j] >> lane) & 1ull) && at < most) dst[at] = (wave * KPT + j) * 64 + lane;
    pos += __popcll(win[j]);
  }
}

// ---------------------------------------------------------------------------
// Pooled scores of kScoreBlock chunks against NA anchors of one head by a
// workgroup of four waves: s[ii stride + c] = scale * q_bar[i0 + ii] . k_bar[m0 + c].
// DH / 8 lanes share a chunk (8 channels each, two 16-byte loads), so a wave's 16
// chunks are all in flight together and the sum needs log2(DH / 8) lane exchanges.
// ---------------------------------------------------------------------------
template <int DH, int NA>
__device__ __forceinline__ void score_tile(const float* __restrict__ means, int n_a, int M, int D, int h,
                                           int i0, int m0, float scale, float* s, int stride) {
  constexpr int LPC = DH / 8, CPW = 64 / LPC, IT = 16 / CPW;
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const int c = h * DH + (lane % LPC) * 8, sub = lane / LPC;
  float4 k0[IT], k1[IT], q0[NA], q1[NA];
#pragma unroll
  for (int it = 0; it < IT; ++it) {
    const int m = min(m0 + wave * 16 + it * CPW + sub, M - 1);
    const float4* p = reinterpret_cast<const float4*>(means + (long long)(n_a + m) * D + c);
    k0[it] = p[0];
    k1[it] = p[1];
  }
#pragma unroll
  for (int ii = 0; ii < NA; ++ii) {   // (anchors past the last repeat it)
    const float4* p = reinterpret_cast<const float4*>(means + (long long)min(i0 + ii, n_a - 1) * D + c);
    q0[ii] = p[0];
    q1[ii] = p[1];
  }
#pragma unroll
  for (int ii = 0; ii < NA; ++ii) {
    float v[IT];
#pragma unroll
    for (int it = 0; it < IT; ++it) {
      float a = q0[ii].x * k0[it].x, b = q1[ii].x * k1[it].x;   // two chains, then pairwise
      a = fmaf(q0[ii].y, k0[it].y, a);
      b = fmaf(q1[ii].y, k1[it].y, b);
      a = fmaf(q0[ii].z, k0[it].z, a);
      b = fmaf(q1[ii].z, k1[it].z, b);
      a = fmaf(q0[ii].w, k0[it].w, a);
      b = fmaf(q1[ii].w, k1[it].w, b);
      v[it] = a + b;
    }
#pragma unroll
    for (int o = LPC / 2; o > 0; o >>= 1)
#pragma unroll
      for (int it = 0; it < IT; ++it) v[it] += __shfl_xor(v[it], o);
    if (lane % LPC == 0) {
#pragma unroll
      for (int it = 0; it < IT; ++it) s[ii * stride + wave * 16 + it * CPW + sub] = v[it] * scale;
    }
  }
}

}  // namespace sel
}  // namespace cast
