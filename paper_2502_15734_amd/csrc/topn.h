// Top-N selection of a segment, as a device function: a launch of its own (select.hip) or behind the second pass of the
// scores of the same segment (mfma_kernels.hip).
#pragma once

#include "device_util.h"

namespace cc {

// ---------------------------------------------------------------------------------------------
// Top-N per chunk.  One workgroup of NW wavefronts per segment.  score = mean over heads of the mass; the N-th
// largest score is found by building its bit pattern from the top down, two bits per round, then
// the tokens above it, and the lowest-index tokens equal to it, are written in ascending index
// order.  Equal scores go to the lower index, so the result is unique.
// Bound by its chain of rounds, not by bytes: the bits all keys of a chunk share are skipped, a
// round costs one barrier, the search ends as soon as exactly N keys lie above the threshold (about
// log2(n) + a few bits instead of 32), and a thread keeps its keys in registers (wavefront w owns a
// contiguous share of the chunk, so the final compaction needs one exchange of counts).
// ---------------------------------------------------------------------------------------------
constexpr int kTopnKeep = 16;               // keys a thread keeps in registers: chunks of up to 4096 tokens with four wavefronts

__device__ __forceinline__ uint32_t ordered_key(float v) {   // monotone float -> uint
  uint32_t u = __float_as_uint(v);
  return (u & 0x80000000u) ? ~u : (u | 0x80000000u);
}

// KEEP: the keys fit in registers (R <= kTopnKeep rounds of 64 tokens per wavefront); otherwise each
// thread reads its own keys back from key_buf.
template <bool KEEP, int NW>
__device__ __forceinline__ void topn_segment(
    const cc_segment& sg, const float* mass, int hq, bool given, const int32_t* __restrict__ block_tab,
    int32_t* __restrict__ sel_idx, int32_t* __restrict__ q_row, int32_t* __restrict__ q_pos,
    int32_t* __restrict__ slot_map, float* __restrict__ scores, uint32_t* key_buf) {
  __shared__ uint32_t all_and[NW], all_or[NW];
  __shared__ int counts[2][3][NW];
  const int n = sg.n_tokens, tid = threadIdx.x, lane = tid & 63, w = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int rounds = (n + 64 * NW - 1) / (64 * NW);          // of 64 tokens per wavefront
  const int first = w * rounds * 64 + lane;                          // token of round r: first + 64 r
  uint32_t held[KEEP ? kTopnKeep : 1];
  uint32_t* stored = key_buf + sg.tok_off;
  // visits (token, key); a token past the chunk's end has key 0 (below every candidate threshold)
  auto each = [&](auto&& f) __attribute__((always_inline)) {
    if constexpr (KEEP) {
#pragma unroll
      for (int r = 0; r < kTopnKeep; ++r)
        if (r < rounds) f(first + 64 * r, held[r]);
    } else {
      for (int r = 0; r < rounds; ++r) {
        const int i = first + 64 * r;
        f(i, i < n ? stored[i] : 0u);
      }
    }
  };
  // ---- scores and keys ----
  const float inv_h = 1.f / static_cast<float>(hq);
  uint32_t k_and = 0xffffffffu, k_or = 0u;
  auto make_key = [&](int i) __attribute__((always_inline)) {
    if (i >= n) return 0u;
    float sc = 0.f;
    if (given) {                            // scores supplied by the caller, one per token
      sc = mass[static_cast<size_t>(sg.tok_off) + i];
    } else if (sg.logical_start > 0) {
      // (summed head by head in index order whatever the load width, so the result does not
      //  depend on it)
      const float* mp = mass + (static_cast<size_t>(sg.tok_off) + i) * hq;
      if ((hq & 3) == 0) {
        const float4* mp4 = reinterpret_cast<const float4*>(mp);
#pragma unroll 8
        for (int h4 = 0; h4 < hq / 4; ++h4) {
          const float4 v = mp4[h4];
          sc += v.x; sc += v.y; sc += v.z; sc += v.w;
        }
      } else {
        for (int h = 0; h < hq; ++h) sc += mp[h];
      }
      sc *= inv_h;
    }
    if (scores) scores[sg.tok_off + i] = sc;
    const uint32_t k = ordered_key(sc);
    k_and &= k;
    k_or |= k;
    return k;
  };
  if constexpr (KEEP) {
#pragma unroll
    for (int r = 0; r < kTopnKeep; ++r)
      if (r < rounds) held[r] = make_key(first + 64 * r);
  } else {
    for (int r = 0; r < rounds; ++r) {
      const int i = first + 64 * r;
      const uint32_t k = make_key(i);
      if (i < n) stored[i] = k;
    }
  }
  const int n_sel = min(max(sg.n_select, 0), n);
  if (n_sel == 0) return;
  // ---- threshold: bits shared by all keys first ----
#pragma unroll
  for (int o = 32; o > 0; o >>= 1) {
    k_and &= __shfl_xor(k_and, o, 64);
    k_or |= __shfl_xor(k_or, o, 64);
  }
  if (lane == 0) { all_and[w] = k_and; all_or[w] = k_or; }
  __syncthreads();
#pragma unroll
  for (int i = 0; i < NW; ++i) { k_and &= all_and[i]; k_or |= all_or[i]; }
  const uint32_t differ = k_and ^ k_or;
  int bits = differ == 0 ? 0 : 32 - __builtin_clz(differ);           // low bits still open
  uint32_t thr = bits == 32 ? 0u : (k_and >> bits) << bits;
  int n_at = n;                                                      // keys >= thr
  for (int round = 0; bits > 0 && n_at != n_sel; ++round) {
    // two bits at a time: the largest of four candidates with at least n_sel keys at or above it
    // (an odd last bit: the step of the candidates is one bit)
    const int step = max(bits - 2, 0);
    const int n_cand = bits >= 2 ? 3 : 1;
    int cnt[3] = {0, 0, 0};
    each([&](int, uint32_t k) __attribute__((always_inline)) {
#pragma unroll
      for (int c = 0; c < 3; ++c) cnt[c] += __popcll(__ballot(k >= (thr | (static_cast<uint32_t>(c + 1) << step))));
    });
    int(*cell)[NW] = counts[round & 1];
    if (lane == 0) {
#pragma unroll
      for (int c = 0; c < 3; ++c) cell[c][w] = cnt[c];
    }
    __syncthreads();
    uint32_t take = 0;
#pragma unroll
    for (int c = 0; c < 3; ++c) {
      int all = 0;
#pragma unroll
      for (int i = 0; i < NW; ++i) all += cell[c][i];
      if (c < n_cand && all >= n_sel) { take = c + 1; n_at = all; }
    }
    thr |= take << step;
    bits = step;
  }
  // exactly n_sel keys at or above thr: all of them; else thr is the N-th key itself and of its
  // equals the first (lowest indices) are kept
  const bool ties = n_at != n_sel;
  int n_gt = 0, n_eq = 0;                                            // of this wavefront
  each([&](int i, uint32_t k) __attribute__((always_inline)) {
    n_gt += __popcll(__ballot(i < n && (ties ? k > thr : k >= thr)));
    n_eq += __popcll(__ballot(i < n && ties && k == thr));
  });
  __shared__ int wave_gt[NW], wave_eq[NW];
  if (lane == 0) { wave_gt[w] = n_gt; wave_eq[w] = n_eq; }
  __syncthreads();
  int gt_before = 0, eq_before = 0, gt_all = 0;
#pragma unroll
  for (int i = 0; i < NW; ++i) {
    if (i < w) { gt_before += wave_gt[i]; eq_before += wave_eq[i]; }
    gt_all += wave_gt[i];
  }
  const int n_eq_take = n_sel - gt_all;
  int pos0 = gt_before + min(eq_before, n_eq_take), eq0 = eq_before;
  const unsigned long long below = (1ull << lane) - 1ull;
  each([&](int i, uint32_t k) __attribute__((always_inline)) {
    const bool eq = i < n && ties && k == thr;
    const unsigned long long b_eq = __ballot(eq);
    const bool take = (i < n && (ties ? k > thr : k >= thr)) || (eq && eq0 + __popcll(b_eq & below) < n_eq_take);
    const unsigned long long b_tk = __ballot(take);
    if (take) {
      const int o = sg.sel_off + pos0 + __popcll(b_tk & below);
      sel_idx[o] = i;
      if (q_row) q_row[o] = sg.tok_off + i;
      if (q_pos) q_pos[o] = sg.logical_start + i;
      if (slot_map) slot_map[o] = block_tab[sg.tab_off + i / kBlock] * kBlock + i % kBlock;
    }
    pos0 += __popcll(b_tk);
    eq0 += __popcll(b_eq);
  });
}

template <int NW>
__device__ __forceinline__ void topn_block(
    int seg, const float* mass, int hq, bool given, const int32_t* __restrict__ block_tab,
    const cc_segment* __restrict__ segs, int32_t* __restrict__ sel_idx, int32_t* __restrict__ q_row,
    int32_t* __restrict__ q_pos, int32_t* __restrict__ slot_map, float* __restrict__ scores,
    uint32_t* key_buf) {
  const cc_segment sg = segs[seg];
  if (sg.kind != CC_SEG_CHUNK) {            // question: every token is a query
    for (int i = threadIdx.x; i < sg.n_tokens; i += 64 * NW) {
      const int o = sg.sel_off + i;
      sel_idx[o] = i;
      if (q_row) q_row[o] = sg.tok_off + i;
      if (q_pos) q_pos[o] = sg.logical_start + i;
      if (slot_map) slot_map[o] = block_tab[sg.tab_off + i / kBlock] * kBlock + i % kBlock;
    }
    return;
  }
  if (sg.n_tokens <= kTopnKeep * 64 * NW)
    topn_segment<true, NW>(sg, mass, hq, given, block_tab, sel_idx, q_row, q_pos, slot_map, scores, key_buf);
  else
    topn_segment<false, NW>(sg, mass, hq, given, block_tab, sel_idx, q_row, q_pos, slot_map, scores, key_buf);
}

}  // namespace cc
