// Rotate-and-scatter of recomputed K/V rows, as a device function: a launch of its own (prefill.hip) or beside the tile
// plan of the attention that follows (mfma_kernels.hip).
#pragma once

#include "device_util.h"

namespace cc {

// Rotate-and-scatter of the recomputed K/V rows into their cache slots.  Rows of the compact query
// list that fall into the same 16-token block are adjacent (the order cc_select emits) and form a
// run.  A workgroup looks at `rows` consecutive rows and handles every run that STARTS among them (a
// run may reach into the next workgroup's rows; it is still handled where it starts); its four
// wavefronts each take a quarter of the KV heads.
//   K rows are token-major and written directly, in 16-byte pieces.
//   The V block is dimension-major -- a token is one element in each of the block's d rows of 16
//   slots -- and isolated 2-byte stores cost a full memory write each, so every (head, dim) row
//   of the block is read, patched with the run's tokens in registers, and written back whole.
//   This needs all rows of a block to sit in ONE run.
// Bound by bytes (a page of values in and out per run) once enough runs are in flight, so nothing of
// a run passes through LDS and no wavefront waits for another: runs are found with one load and
// ballots, source rows and slots travel by lane permutes.
// Consecutive workgroups take rows 16 apart (first all spans' first rows, then their second ones, ...).  In the order of the rows the
// runs of a dense list begin in every fourth (or eighth, or sixteenth) workgroup, which the dispatcher deals to one or two of the
// eight XCDs: 40000 dense rows on 8 KV heads 164 -> 59 us, 16000 57 -> 22, 1000 14.4 -> 7.8; every seventh row of 40000 291 -> 284.
// Rows per workgroup: 4 on long lists, where fewer candidates start too many workgroups that find nothing on dense lists and
// eight or sixteen leave too few runs in flight on scattered ones.  Short lists: a run is a chain of four dependent loads,
// so that a workgroup should have one.  8 KV heads, d = 128, every seventh token / all of them, us with 4, 2, 1 rows: 230 rows 9.0,
// 6.4, 6.5 / 7.5, 7.3, 7.5; 1000: 11.4, 8.8, 9.4 / 7.9, 7.8, 7.9; 2000: 15.2, 13.2, 14.0 / 8.7, 8.7, 8.6; 4000: 24.0, 24.6, 24.6 /
// 9.4, 9.5, 9.4; 16000: 107, 108, 118 / 22, 24, 28.  With cold caches one row is ahead on the shortest: a whole decoder
// layer of 449 rows takes 3 of 320 us less than with two.
__host__ __device__ inline int scatter_rows(int n_rows) { return n_rows <= 1024 ? 1 : n_rows <= 2048 ? 2 : 4; }
inline int scatter_groups(int n_rows) { return (n_rows + kBlock - 1) / kBlock * (kBlock / scatter_rows(n_rows)); }      // workgroups

// (block: the workgroup's number among those that do this)
template <typename T, int D>
__device__ __forceinline__ void rope_scatter_rows(
    int block, int rows, const T* __restrict__ k_new, const T* __restrict__ v_new, const int32_t* __restrict__ q_pos,
    const int32_t* __restrict__ slot_map, int n_q_tot, int hkv, InvFreq inv_freq,
    T* __restrict__ k_pool, T* __restrict__ v_pool, int n_blocks, const int32_t* __restrict__ src_rows,
    const T* __restrict__ v_shared, int n_shared_blocks, int32_t* __restrict__ v_map) {
  const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int n_spans = (n_q_tot + kBlock - 1) / kBlock, base = block % n_spans * kBlock + block / n_spans * rows;
  // lane i looks at row base - 1 + i: the row before the first candidate, the candidates, and the
  // rows a run that starts at the last of them can still cover
  int slot = -1, row = 0, pos = 0;
  const int j = base - 1 + lane;
  if (lane < rows + kBlock && j >= 0 && j < n_q_tot) {
    slot = slot_map[j];
    row = src_rows != nullptr ? src_rows[j] : j;             // (row of k_new, v_new this list row reads)
    pos = q_pos[j];
    if (slot < 0 || slot >= n_blocks * kBlock) slot = -1;
  }
  const int my_blk = slot >= 0 ? slot / kBlock : -1;
  const int before = __shfl_up(my_blk, 1, 64);
  unsigned long long starts = __ballot(lane >= 1 && lane <= rows && my_blk >= 0 && before != my_blk);
  // this wavefront's KV heads
  const int per = (hkv + 3) / 4, h_first = wave * per;
  const int nh = max(min(per, hkv - h_first), 0);
  const size_t block_elems = static_cast<size_t>(hkv) * D * kBlock;
  unsigned long long pending = 0;        // runs whose page still had its values in the store

  while (starts != 0) {
    const int c = __builtin_ctzll(starts);                   // lane of the run's first row
    starts &= starts - 1;
    const int blk = __builtin_amdgcn_readlane(my_blk, c);
    const unsigned long long same = __ballot(my_blk == blk) >> c;
    const int n_run = min(__builtin_ctzll(~same), kBlock);
    // source of the page's values: the request's own block or - the first time a token of the page is
    // recomputed - the stored block the value map still points at (copy-on-write; the entry is cleared
    // once every wavefront has looked it up)
    const T* v_from = value_block<T>(v_pool, v_shared, n_shared_blocks, v_map, blk, block_elems);
    if (v_from != v_pool + static_cast<size_t>(blk) * block_elems) pending |= 1ull << c;
    // source row of every slot of the block (-1: not in the run), in scalar registers
    const bool in_run = lane >= c && lane < c + n_run;
    const int inv = __builtin_amdgcn_ds_permute((in_run ? slot % kBlock : 63) * 4, in_run ? row + 1 : 0);
    int src_of[kBlock];
#pragma unroll
    for (int k = 0; k < kBlock; ++k) src_of[k] = __builtin_amdgcn_readlane(inv, k) - 1;

    // ---- K: one (token, KV head, 16-byte piece of the head's first half) per lane and item, with the
    // matching piece of the second half: two 16-byte loads, kPer rotations, two 16-byte stores
    constexpr int kPer = 16 / sizeof(T), kPieces = D / 2 / kPer, kItems = 2;
    const int n_items = n_run * nh * kPieces;
    for (int i0 = lane; i0 - lane < n_items; i0 += 64 * kItems) {
      uint4 xv[kItems], yv[kItems];
      int p_[kItems], h_[kItems], pos_[kItems], slot_[kItems];
#pragma unroll
      for (int u = 0; u < kItems; ++u) {
        const int idx = min(i0 + 64 * u, n_items - 1);
        const int t = idx / (kPieces * nh);
        p_[u] = idx % kPieces;
        h_[u] = h_first + (idx / kPieces) % nh;
        const int r = __shfl(row, c + t, 64);
        pos_[u] = __shfl(pos, c + t, 64);
        slot_[u] = __shfl(slot, c + t, 64) % kBlock;
        const T* kp = k_new + (static_cast<size_t>(r) * hkv + h_[u]) * D + kPer * p_[u];
        xv[u] = *reinterpret_cast<const uint4*>(kp);
        yv[u] = *reinterpret_cast<const uint4*>(kp + D / 2);
      }
#pragma unroll
      for (int u = 0; u < kItems; ++u) {
        if (i0 + 64 * u < n_items) {
          T* ko = k_pool + ((static_cast<size_t>(blk) * hkv + h_[u]) * kBlock + slot_[u]) * D + kPer * p_[u];
          T x[kPer], y[kPer], ox[kPer], oy[kPer];
          *reinterpret_cast<uint4*>(x) = xv[u];
          *reinterpret_cast<uint4*>(y) = yv[u];
#pragma unroll
          for (int e = 0; e < kPer; ++e) {
            float cs, sn;
            if (sizeof(T) == 2) rot_cos_sin_fast(pos_[u], inv_freq.f[kPer * p_[u] + e], &cs, &sn);   // (the result is rounded to bf16)
            else rot_cos_sin(pos_[u], inv_freq.f[kPer * p_[u] + e], &cs, &sn);
            const float xf = to_float(x[e]), yf = to_float(y[e]);
            ox[e] = from_float<T>(xf * cs - yf * sn);
            oy[e] = from_float<T>(yf * cs + xf * sn);
          }
          *reinterpret_cast<uint4*>(ko) = *reinterpret_cast<uint4*>(ox);
          *reinterpret_cast<uint4*>(ko + D / 2) = *reinterpret_cast<uint4*>(oy);
        }
      }
    }

    // ---- V: (head, dim) rows of 16 slots, kRows per lane and step; the page's rows and the run's new
    // elements are all requested before the first is used
    constexpr int kVec = kBlock * sizeof(T) / 16;            // 16-byte vectors per row
    constexpr int kRows = 2;                                 // (4: 146 registers, 10 % slower on long lists; 1: twice as slow)
    T* v_page = v_pool + (static_cast<size_t>(blk) * hkv + h_first) * D * kBlock;
    const T* from_page = v_from + static_cast<size_t>(h_first) * D * kBlock;
    for (int i0 = lane; i0 - lane < nh * D; i0 += 64 * kRows) {
      uint4 e[kRows][kVec];
      T fresh[kRows][kBlock];
      if (n_run < kBlock) {
#pragma unroll
        for (int u = 0; u < kRows; ++u)
#pragma unroll
          for (int v = 0; v < kVec; ++v)
            e[u][v] = *reinterpret_cast<const uint4*>(from_page + static_cast<size_t>(min(i0 + 64 * u, nh * D - 1)) * kBlock + v * kPer);
      }
      const T* vcol = v_new + static_cast<size_t>(h_first) * D;
#pragma unroll
      for (int k = 0; k < kBlock; ++k)
        if (src_of[k] >= 0) {
#pragma unroll
          for (int u = 0; u < kRows; ++u)
            fresh[u][k] = vcol[static_cast<size_t>(src_of[k]) * hkv * D + min(i0 + 64 * u, nh * D - 1)];
        }
#pragma unroll
      for (int u = 0; u < kRows; ++u) {
        T out[kBlock];
#pragma unroll
        for (int v = 0; v < kVec; ++v) *reinterpret_cast<uint4*>(out + v * kPer) = e[u][v];
#pragma unroll
        for (int k = 0; k < kBlock; ++k)
          if (src_of[k] >= 0) out[k] = fresh[u][k];
        if (i0 + 64 * u < nh * D) {
#pragma unroll
          for (int v = 0; v < kVec; ++v)
            *reinterpret_cast<uint4*>(v_page + static_cast<size_t>(i0 + 64 * u) * kBlock + v * kPer) = *reinterpret_cast<uint4*>(out + v * kPer);
        }
      }
    }
  }
  if (pending != 0) {                    // (the same in all wavefronts: nobody clears an entry before this barrier)
    __syncthreads();
    if (wave == 0 && ((pending >> lane) & 1)) v_map[my_blk] = -1;
  }
}

}  // namespace cc
