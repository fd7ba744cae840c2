// MFMA (bf16, head_dim 128) kernels of cc_select's score stage and cc_sparse_prefill's attention.
//
// Both stages are "few queries against all earlier keys" (Sec. 4 "Selective Token Recomputation";
// per-token form of Eq. (1)).  One workgroup owns 32*QB query tokens of one request and one KV
// head; wavefront w owns query head kvh*G + w, so all G heads of the group share every K/V tile
// that is staged in LDS (grouped-query packing).  Key tiles are 64 keys (4 blocks of 16 tokens)
// and never straddle a segment, so block padding only shows up in a segment's last tile.
//
// Orientation: S^T = K Q^T and O^T = V^T P^T with v_mfma_f32_32x32x16_bf16.  In the 32x32 result
// a lane holds ONE query column (lane % 32) and 16 rows, so the softmax of a query (reference
// max, exponentials, sum, rescale of O) is lane-local; the two lane halves, which hold different
// keys of the same query, only talk when the reference max moves.  P^T feeds the second product
// straight from the accumulator registers: within a 32-key block the MFMA row m of S^T is
// assigned the key swap_bits_2_3(m), which makes the 8 values a lane-half contributes to one
// 16-key step the keys 8*half .. 8*half+7 of one 16-token block -- exactly one 16-byte row piece
// of the dimension-major V block.
//
// Softmax bookkeeping: the query is pre-multiplied by log2(e)/sqrt(d) before it is rounded to
// bf16, so S is in log2 units and p = exp2(S - m_ref).  The reference m_ref is fixed by the first
// block of the request -- 0 if that block's maximum is within +-2^24 of it (then the subtraction
// is skipped altogether), else that maximum -- and afterwards moves only when a block's sum of
// exponentials exceeds kBig (entries far above the reference); that block is then redone with the
// reference raised and the sums and O rescaled.  Until then p is merely "large": fp32 and bf16
// share the exponent range, so nothing is lost.
//
// LDS image of a tile (16-byte pieces; every MFMA operand read is one conflict-free 1 KiB run):
//   K piece (block b of 32 keys, k-step kk, half hh, row m):  (b*8+kk)*64 + hh*32 + (m ^ ((2kk+hh)&7))
//   V piece (page pg, 32-dim group db, half hh, dim n):       1024 + (pg*4+db)*64 + hh*32 + (n ^ 4hh)
// The XOR terms spread the *writes* of a coalesced global read over the LDS banks.
#include <type_traits>

#include "mfma_tile.h"
#include "scatter.h"
#include "topn.h"

namespace cc {

using namespace tile;

namespace {

// Small workgroups (64 or 128 threads; head groups of 1 or 2): the tile does not fit in registers,
// so it is copied piece by piece without prefetch.  Correct, not fast.
template <int NT, bool WITH_V>
__device__ __forceinline__ void stage_direct(uint4* lds, const bf16_t* __restrict__ k_pool,
                                             const bf16_t* __restrict__ v_pool, int n_blocks,
                                             const TileDesc& d, int hkv, int kvh, int tid,
                                             const bf16_t* __restrict__ v_shared, int n_shared_blocks,
                                             const int32_t* __restrict__ v_map) {
  const int nvalid = d.nvalid;
  constexpr int kPieces = WITH_V ? 2048 : 1024;
#pragma unroll 4
  for (int i = 0; i < kPieces / NT; ++i) {
    const int c = tid + NT * i;
    const bool is_v = WITH_V && c >= 1024;
    const int pg = (c & 1023) >> 8, cc_ = c & 255;
    const int nv = min(max(nvalid - kBlock * pg, 0), kBlock);
    const int blk = d.blk[pg];
    const bool ok = nv > 0 && blk >= 0 && blk < n_blocks;
    const size_t off = (static_cast<size_t>(ok ? blk : 0) * hkv + kvh) * (kBlock * kD) + cc_ * 8;
    uint4 val = make_uint4(0u, 0u, 0u, 0u);
    if (ok) {
      if (!is_v) {
        if ((cc_ >> 4) < nv) val = *reinterpret_cast<const uint4*>(k_pool + off);
      } else {
        const bf16_t* vb = value_block<bf16_t>(v_pool, v_shared, n_shared_blocks, v_map, blk,
                                               static_cast<size_t>(hkv) * (kBlock * kD));
        val = *reinterpret_cast<const uint4*>(vb + static_cast<size_t>(kvh) * (kBlock * kD) + cc_ * 8);
        if (nv < kBlock) val = zero_pad_slots(val, cc_ & 1, nv);
      }
    }
    lds[is_v ? v_piece_dst(pg, cc_) : k_piece_dst(pg, cc_)] = val;
  }
}

// SCORE = true : queries are 32*QB consecutive tokens of a chunk segment; result is the share of
//                the softmax mass that falls on keys of earlier segments (Eq. (2), Eq. (10)).
// SCORE = false: queries are 32*QB rows of the compact query list; result is the attention
//                output and log-sum-exp (Eq. (1)).
// REDO = true : second pass behind the wide kernels.  One workgroup per segment (score) or request
//                (attention) looks up, in parallel, which of its row tiles the wide kernel flagged
//                and walks those, one KV head after the other; without flags - the normal case -
//                it is gone after one round of loads, so the pass costs a few hundred short
//                workgroups instead of one per (tile, KV head).
// (item: the segment or request of this workgroup)
template <int G, bool SCORE, int QB, bool REDO>
__device__ __forceinline__ void sparse_qk(
    int y_item, const bf16_t* __restrict__ q, const int32_t* __restrict__ q_pos, const int32_t* __restrict__ cu_q,
    const bf16_t* __restrict__ k_pool, const bf16_t* __restrict__ v_pool, int n_blocks,
    const TileDesc* __restrict__ tiles, const int32_t* __restrict__ seg_tile_off, int max_tiles,
    const cc_segment* __restrict__ segs, const int32_t* __restrict__ req_seg_off, int hq, int hkv,
    int n_tiles_x, InvFreq inv_freq, bf16_t* __restrict__ out, float* __restrict__ lse,
    float* __restrict__ mass, const int32_t* __restrict__ redo, int redo_any, const int32_t* __restrict__ q_map,
    int map_pos, const bf16_t* __restrict__ v_shared, int n_shared_blocks, const int32_t* __restrict__ v_map) {
  constexpr int NT = 64 * G;
  constexpr int TQ = 32 * QB;                       // query tokens per workgroup
  constexpr bool kPrefetch = NT >= 256;
  constexpr int kImage = SCORE ? 1024 : 2048;       // 16-byte pieces per tile image
  // operand reads in flight ahead of the MFMAs (16 bytes per lane each)
  constexpr int kDepth = (QB == 2 || NT <= 256) ? 4 : 8;
  static_assert(16 % kDepth == 0, "ring slots must line up from one tile to the next");
  // attention: double-buffered.  score: three images, because the previous tile's image must stay
  // readable (repair path of its deferred block) while the next tile is being stored.
  constexpr int kBufs = SCORE ? 3 : 2;
  if constexpr (REDO) {
    if (redo[redo_any] == 0) return;                  // (normally: one load, and nothing that hangs on it)
  }
  __shared__ uint4 lds_all[kBufs * kImage];
  const int tid = threadIdx.x, lane = tid & 63, wave = uniform(tid >> 6);
  const int n = lane & 31, hh = lane >> 5;
  // ---- which row tiles ----------------------------------------------------------------------
  cc_segment sg_own = {};
  int q_first = 0, q_end = 0;
  if constexpr (SCORE) sg_own = segs[y_item];
  else { q_first = cu_q[y_item]; q_end = cu_q[y_item + 1]; }
  // is row tile t of this item flagged for the second pass?
  auto flagged = [&](int t) {
    if constexpr (SCORE) {
      const int t0 = t * TQ;
      if (sg_own.kind != CC_SEG_CHUNK || t0 >= sg_own.n_tokens || sg_own.logical_start == 0) return false;
      return (redo[(sg_own.tok_off + t0) >> 6] | redo[(sg_own.tok_off + min(t0 + TQ, sg_own.n_tokens) - 1) >> 6]) != 0;
    } else {
      if (q_first + t * TQ >= q_end) return false;
      return redo[redo_index(q_first + (t * TQ / 64) * 64)] != 0;
    }
  };
  __shared__ int todo[REDO ? NT : 1];
  __shared__ int n_todo;
  const int n_rounds = REDO ? (n_tiles_x + NT - 1) / NT : 1;
  for (int round = 0; round < n_rounds; ++round) {
  int n_work = 1;
  if constexpr (REDO) {
    __syncthreads();                                  // (the previous round's list has been walked)
    if (tid == 0) n_todo = 0;
    __syncthreads();
    const int t = round * NT + tid;
    if (t < n_tiles_x && flagged(t)) todo[atomicAdd(&n_todo, 1)] = t;
    __syncthreads();
    n_work = n_todo * hkv;
  }
  for (int work = 0; work < n_work; ++work) {
  if constexpr (REDO) __syncthreads();                // (LDS images of the previous tile are free)
  const int kvh = REDO ? work % hkv : blockIdx.x % hkv;
  const int tile = REDO ? todo[work / hkv] : n_tiles_x - 1 - blockIdx.x / hkv;       // late (long) tiles are dispatched first
  const int h = kvh * G + wave;

  // ---- which queries ------------------------------------------------------------------------
  // (attention with a row map: list row j takes its query from row q_map[j] of q - and, if
  // map_pos, its position from q_pos[q_map[j]]; results are always indexed by the list row)
  int row[QB], src_row[QB], p[QB], s_begin, s_end, s_self = -1;
  bool row_valid[QB];
  if constexpr (SCORE) {
    const int seg_id = y_item;
    const cc_segment sg = sg_own;
    const int t0 = tile * TQ;
    if (sg.kind != CC_SEG_CHUNK || t0 >= sg.n_tokens || sg.logical_start == 0) continue;
#pragma unroll
    for (int qb = 0; qb < QB; ++qb) {
      const int t = min(t0 + 32 * qb + n, sg.n_tokens - 1);
      row_valid[qb] = t0 + 32 * qb + n < sg.n_tokens;
      row[qb] = sg.tok_off + t;
      src_row[qb] = row[qb];
      p[qb] = sg.logical_start + t;
    }
    s_begin = req_seg_off[sg.req];
    s_self = seg_id;
    s_end = s_self + 1;
  } else {
    const int r = y_item;
    const int q0 = q_first + tile * TQ;
    if (q0 >= q_end) continue;
#pragma unroll
    for (int qb = 0; qb < QB; ++qb) {
      row[qb] = min(q0 + 32 * qb + n, q_end - 1);
      row_valid[qb] = q0 + 32 * qb + n < q_end;
      src_row[qb] = q_map != nullptr ? q_map[row[qb]] : row[qb];
      p[qb] = q_pos[map_pos ? src_row[qb] : row[qb]];
    }
    s_begin = req_seg_off[r];
    s_end = req_seg_off[r + 1];
  }
  int pmx = p[0], pmn = p[0];
#pragma unroll
  for (int qb = 1; qb < QB; ++qb) { pmx = max(pmx, p[qb]); pmn = min(pmn, p[qb]); }
  const int p_max = uniform(wave_max_i(pmx)), p_min = uniform(wave_min_i(pmn));

  // ---- load the query rows, rotate them to their positions, fold the softmax scale -------------
  // lane (n, hh) keeps, for k-step kk, dims 16kk + 8hh .. +7; dims < 64 pair with dims + 64.
  const float c2 = 0.08838834764831845f * kLog2e;           // log2(e) / sqrt(128)
  bf16x8 qreg[QB][8];
#pragma unroll
  for (int qb = 0; qb < QB; ++qb) {
    const bf16_t* qp = q + (static_cast<size_t>(src_row[qb]) * hq + h) * kD + 8 * hh;
#pragma unroll
    for (int kk = 0; kk < 4; ++kk) {
      bf16x8 xv = __builtin_bit_cast(bf16x8, *reinterpret_cast<const uint4*>(qp + 16 * kk));
      bf16x8 yv = __builtin_bit_cast(bf16x8, *reinterpret_cast<const uint4*>(qp + 16 * kk + 64));
#pragma unroll
      for (int j = 0; j < 8; ++j) {
        float c, s;
        rot_cos_sin_fast(p[qb], inv_freq.f[16 * kk + 8 * hh + j], &c, &s);
        c *= c2; s *= c2;
        const float x = static_cast<float>(xv[j]), y = static_cast<float>(yv[j]);
        xv[j] = static_cast<bf16_t>(x * c - y * s);
        yv[j] = static_cast<bf16_t>(y * c + x * s);
      }
      qreg[qb][kk] = xv;
      qreg[qb][kk + 4] = yv;
      __builtin_amdgcn_sched_barrier(0);     // keep the prologue's register footprint small
    }
  }

  // lane-dependent part of the operand addresses (pieces), constant over the whole loop
  int kx[4];
#pragma unroll
  for (int j = 0; j < 4; ++j) kx[j] = hh * 32 + (n ^ ((2 * j + hh) & 7));
  const int vx = 1024 + hh * 32 + (n ^ (4 * hh));

  float m_ref[QB], l_run[QB], l_prior[QB];
  f32x16 o[QB][SCORE ? 1 : 4];
  f32x16 sacc[QB][2];                 // S (then p) of the two 32-key blocks in flight
#pragma unroll
  for (int qb = 0; qb < QB; ++qb) {
    m_ref[qb] = 0.f; l_run[qb] = 0.f; l_prior[qb] = 0.f;
#pragma unroll
    for (int db = 0; db < (SCORE ? 1 : 4); ++db) o[qb][db] = splat16(0.f);
  }

  // ---- building blocks of the tile pipeline -----------------------------------------------------
  // S block b of the tile image `img`: 8 k-steps, operand reads kDepth steps ahead of the MFMAs;
  // `side(kk)` is VALU work of ANOTHER block that is slotted in after every k-step so that it runs
  // while the matrix pipe is busy.  raw = true ignores the reference (used by the repair path).
  // The MFMA operands of a tile form one stream of kSteps 16-byte pieces per lane (K pieces of S
  // block 0, S block 1, then the V pieces of the four pages); `ring` keeps kDepth of them in flight
  // ahead of the MFMA that consumes them, across the stages of the tile, so that LDS latency is
  // paid once per tile and not once per stage.
  constexpr int kSteps = SCORE ? 16 : 32;
  uint4 ring[kDepth];
  // step t of the current image; steps >= kSteps are the first K pieces of the next image `nimg`
  // (nullptr: there is no next tile, or it may not be read yet)
  auto issue = [&](const uint4* img, const uint4* nimg, int t) {   // t: compile-time step index
    if (t < kSteps) {
      ring[t % kDepth] = t < 16 ? img[t * 64 + kx[t & 3]] : img[(t - 16) * 64 + vx];
    } else if (nimg != nullptr) {
      const int t2 = t - kSteps;
      ring[t % kDepth] = nimg[t2 * 64 + kx[t2 & 3]];
    }
  };
  auto prime = [&](const uint4* img) {
#pragma unroll
    for (int t = 0; t < kDepth; ++t) issue(img, nullptr, t);
    __builtin_amdgcn_sched_barrier(0);
  };
  auto qk_block = [&](const uint4* img, const uint4* nimg, int b, auto&& side) {
#pragma unroll
    for (int kk = 0; kk < 8; ++kk) {
      const int t = b * 8 + kk;
      const bf16x8 a = __builtin_bit_cast(bf16x8, ring[t % kDepth]);
#pragma unroll
      for (int qb = 0; qb < QB; ++qb)
        sacc[qb][b] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(
            a, qreg[qb][kk], kk == 0 ? splat16(0.f) : sacc[qb][b], 0, 0, 0);
      issue(img, nimg, t + kDepth);
      side(kk);
      __builtin_amdgcn_sched_barrier(0);
    }
  };
  // repair path only: raw S of block b straight from the image (does not touch the ring)
  auto qk_block_raw = [&](const uint4* img, int b) {
#pragma unroll
    for (int kk = 0; kk < 8; ++kk) {
      const bf16x8 a = __builtin_bit_cast(bf16x8, img[(b * 8 + kk) * 64 + kx[kk & 3]]);
#pragma unroll
      for (int qb = 0; qb < QB; ++qb)
        sacc[qb][b] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(
            a, qreg[qb][kk], kk == 0 ? splat16(0.f) : sacc[qb][b], 0, 0, 0);
    }
  };
  // exponentials of elements 2kk, 2kk+1 of block b (all query blocks); sums go to lsum[]
  float lsum[QB];
  // While every query's reference is still exactly 0 (zero_ref: the first block's maximum was
  // small, which is the normal case for attention logits) the subtraction is skipped; the
  // accumulators always hold raw S, so switching between the two forms needs no fix-up.
  bool zero_ref = true;
  auto exp_pair = [&](auto zero, int b, int kk) {
    constexpr bool kZero = decltype(zero)::value;
#pragma unroll
    for (int qb = 0; qb < QB; ++qb)
#pragma unroll
      for (int e = 0; e < 2; ++e) {
        const int i = 2 * kk + e;
        const float v = __builtin_amdgcn_exp2f(kZero ? sacc[qb][b][i] : sacc[qb][b][i] - m_ref[qb]);
        sacc[qb][b][i] = v;
        lsum[qb] += v;
      }
  };
  using ZeroT = std::integral_constant<bool, true>;
  using SubT = std::integral_constant<bool, false>;
  auto no_side = [&](int) {};
  // padding / causal edge: entries of block b that the query must not see become -inf
  // (accumulator register i of block b holds key 32b + 16(i/8) + 8hh + i%8 of the tile)
  auto mask_block = [&](int b, int kpos0, int nvalid) {
#pragma unroll
    for (int qb = 0; qb < QB; ++qb) {
      int lim = min(nvalid - 1, p[qb] - kpos0) - 8 * hh - 32 * b;
      asm volatile("" : "+v"(lim));                        // keep the compares inside the branch
#pragma unroll
      for (int i = 0; i < 16; ++i)
        sacc[qb][b][i] = (16 * (i / 8) + (i % 8) <= lim) ? sacc[qb][b][i] : -INFINITY;
      asm volatile("" : "+v"(sacc[qb][b]));
    }
  };
  // move the reference of every query up to the maximum of block b (raw S); rescale what has been
  // summed so far.  init: first block of the request -- the reference stays 0 if every query's
  // maximum is within +-kZeroBand, else it becomes that maximum.
  auto raise_ref = [&](int b, bool init) {
    float t[QB];
    bool small = true;
#pragma unroll
    for (int qb = 0; qb < QB; ++qb) {
      t[qb] = max16(sacc[qb][b]);
      t[qb] = fmaxf(t[qb], __shfl_xor(t[qb], 32, 64));
      small = small && fabsf(t[qb]) <= kZeroBand;
    }
    if (init && __all(small)) return;
#pragma unroll
    for (int qb = 0; qb < QB; ++qb) {
      const float d = init ? t[qb] : fmaxf(t[qb] - m_ref[qb], 0.f);
      const float alpha = init ? 1.f : __builtin_amdgcn_exp2f(-d);
      l_run[qb] *= alpha;
      if constexpr (SCORE) l_prior[qb] *= alpha;
      else {
#pragma unroll
        for (int db = 0; db < 4; ++db)
#pragma unroll
          for (int i = 0; i < 16; ++i) o[qb][db][i] *= alpha;
      }
      m_ref[qb] += d;
    }
    zero_ref = false;
  };
  // close block b after its exponentials: normally just add the sums.  If a sum is huge or not
  // finite, entries ran far above the reference: recompute the block's S from the LDS image,
  // raise the reference (rescaling sums and O), and redo the exponentials.  Rare.
  auto close_block = [&](const uint4* img, int b, int kpos0, int nvalid, bool edge) {
    bool bad = false;
#pragma unroll
    for (int qb = 0; qb < QB; ++qb) bad = bad || !(lsum[qb] < kBig);
    if (__any(bad)) {
      asm volatile("" ::: "memory");
      qk_block_raw(img, b);
      if (edge) mask_block(b, kpos0, nvalid);
      raise_ref(b, false);
#pragma unroll
      for (int qb = 0; qb < QB; ++qb) {
        lsum[qb] = 0.f;
#pragma unroll
        for (int i = 0; i < 16; ++i) {
          const float v = __builtin_amdgcn_exp2f(sacc[qb][b][i] - m_ref[qb]);
          sacc[qb][b][i] = v;
          lsum[qb] += v;
        }
      }
    }
#pragma unroll
    for (int qb = 0; qb < QB; ++qb) { l_run[qb] += lsum[qb]; lsum[qb] = 0.f; }
  };
#pragma unroll
  for (int qb = 0; qb < QB; ++qb) lsum[qb] = 0.f;

  // ---- the tile loop ------------------------------------------------------------------------------
  // Tiles of the request are listed by the plan kernels; tile j is usable if j < j_end and its
  // first key is visible to some query of the workgroup.  Three things run ahead of the math of
  // tile t: the descriptor of tile t+3 (a broadcast vector load), the global loads of tile t+2
  // (into registers, issued right after the barrier), and the LDS image of tile t+1 (stored in the
  // middle of tile t).  The workgroup barrier sits before the last stage of a tile, whose operands
  // are already in registers, so that the first operand reads of the next image are in flight
  // while that stage's MFMAs run.
  const int j_begin = seg_tile_off[s_begin];
  const int j_end = min(seg_tile_off[s_end], max_tiles);
  const int j_own = SCORE ? seg_tile_off[s_self] : -1;
  auto usable = [&](const TileDesc& d, int j) { return j < j_end && uniform(d.kpos0) <= p_max; };

  Stager<kPrefetch ? NT : 256, !SCORE> stg;
  if constexpr (kPrefetch) stg.init(k_pool, v_pool, n_blocks, hkv, kvh, tid, v_shared, n_shared_blocks, v_map);
  auto stage_load = [&](const TileDesc& d) {            // global -> registers
    if constexpr (kPrefetch) stg.load(d);
  };
  auto stage_store = [&](const TileDesc& d, int b_) {   // registers (or global) -> LDS image b_
    if constexpr (kPrefetch) stg.store(lds_all + b_ * kImage);
    else stage_direct<NT, !SCORE>(lds_all + b_ * kImage, k_pool, v_pool, n_blocks, d, hkv, kvh, tid, v_shared,
                                  n_shared_blocks, v_map);
  };

  int j = j_begin;
  TileDesc d0 = to_scalar(fetch_desc(tiles, j, max_tiles));
  TileDesc d1 = to_scalar(fetch_desc(tiles, j + 1, max_tiles));
  TileDesc d2 = to_scalar(fetch_desc(tiles, j + 2, max_tiles));
  bool v0 = usable(d0, j), v1 = v0 && usable(d1, j + 1), v2 = v1 && usable(d2, j + 2);
  int buf = 0;
  if (v0) { stage_load(d0); stage_store(d0, 0); }
  if (v1) stage_load(d1);
  __syncthreads();
  if (v0) prime(lds_all);
  bool first = true;
  // SCORE: block 1 of the previous tile waits in sacc[*][1] for its exponentials, which are
  // slotted under the next tile's first S block
  bool pending = false;
  int prev_kpos0 = 0, prev_nvalid = 0;
  bool prev_edge = false;
  while (v0) {
    const bool enter_own = SCORE && j == j_own;
    const int kpos0 = uniform(d0.kpos0), nvalid = uniform(d0.nvalid);
    const bool edge = nvalid < kTile || kpos0 + kTile - 1 > p_min;   // padding or causal edge
    const int next_buf = (buf + 1) % kBufs;
    const uint4* img = lds_all + buf * kImage;
    const uint4* next_img = lds_all + next_buf * kImage;
    const uint4* prev_img = lds_all + ((buf + kBufs - 1) % kBufs) * kImage;
    TileDesc d3 = fetch_desc(tiles, j + 3, max_tiles);             // three tiles ahead
    TileDesc d3s;                                                  // ... made wave-uniform mid-tile

    // ---- stage 0: S block 0 ----------------------------------------------------------------------
    if constexpr (SCORE) {
      if (pending) {
        if (zero_ref) qk_block(img, nullptr, 0, [&](int kk) { exp_pair(ZeroT{}, 1, kk); });
        else qk_block(img, nullptr, 0, [&](int kk) { exp_pair(SubT{}, 1, kk); });
        close_block(prev_img, 1, prev_kpos0, prev_nvalid, prev_edge);
      } else {
        qk_block(img, nullptr, 0, no_side);
      }
      // entering the query's own segment: everything summed so far is prior-chunk mass
      if (enter_own) {
#pragma unroll
        for (int qb = 0; qb < QB; ++qb) { l_prior[qb] = l_run[qb]; l_run[qb] = 0.f; }
      }
    } else {
      qk_block(img, nullptr, 0, no_side);
    }
    if (edge) mask_block(0, kpos0, nvalid);
    if (first) {                       // key 0 of the request is in this block and visible to all
      raise_ref(0, true);
      first = false;
    }
    if constexpr (SCORE) {
      // all operand reads of this image are issued; publish the next image and meet
      if (v1) stage_store(d1, next_buf);
      __syncthreads();
      d3s = to_scalar(d3);             // its load is the only one in flight here: waiting is free
      if (v2) stage_load(d2);
      // ---- stage 1: S block 1, exponentials of block 0 underneath; first reads of the next image
      if (zero_ref) qk_block(img, v1 ? next_img : nullptr, 1, [&](int kk) { exp_pair(ZeroT{}, 0, kk); });
      else qk_block(img, v1 ? next_img : nullptr, 1, [&](int kk) { exp_pair(SubT{}, 0, kk); });
      if (edge) mask_block(1, kpos0, nvalid);
      close_block(img, 0, kpos0, nvalid, edge);
      pending = true; prev_kpos0 = kpos0; prev_nvalid = nvalid; prev_edge = edge;
    } else {
      // ---- stage 1: S block 1, exponentials of block 0 underneath -----------------------------------
      // (the attention kernel is bound by LDS operand reads, not by the VALU: one form is enough)
      qk_block(img, nullptr, 1, [&](int kk) { exp_pair(SubT{}, 0, kk); });
      if (edge) mask_block(1, kpos0, nvalid);
      close_block(img, 0, kpos0, nvalid, edge);
      if (v1) stage_store(d1, next_buf);
      // ---- stages 2, 3: O^T += V^T P^T, P^T straight from the accumulator registers ------------------
      // block b covers pages 2b, 2b+1 of the tile; step st = (u, db): page 2b+u, 32-dim group db
      auto pv_block = [&](const uint4* nimg, int b, auto&& side) {
        bf16x8 pb[QB];
#pragma unroll
        for (int st = 0; st < 8; ++st) {
          const int u = st >> 2, db = st & 3, t = 16 + b * 8 + st;
          if (db == 0) {
#pragma unroll
            for (int qb = 0; qb < QB; ++qb)
#pragma unroll
              for (int jj = 0; jj < 8; ++jj) pb[qb][jj] = static_cast<bf16_t>(sacc[qb][b][8 * u + jj]);
          }
          const bf16x8 a = __builtin_bit_cast(bf16x8, ring[t % kDepth]);
#pragma unroll
          for (int qb = 0; qb < QB; ++qb)
            o[qb][db] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a, pb[qb], o[qb][db], 0, 0, 0);
          issue(img, nimg, t + kDepth);
          side(st);
          __builtin_amdgcn_sched_barrier(0);
        }
      };
      pv_block(nullptr, 0, [&](int st) { exp_pair(SubT{}, 1, st); });
      close_block(img, 1, kpos0, nvalid, edge);
      // every read of this image has been issued; meet, then finish the tile out of registers
      // while the first operand reads of the next image are in flight
      __syncthreads();
      d3s = to_scalar(d3);             // its load is the only one in flight here: waiting is free
      if (v2) stage_load(d2);
      pv_block(v1 ? next_img : nullptr, 1, no_side);
    }
    ++j;
    d0 = d1; d1 = d2; d2 = d3s;
    v0 = v1; v1 = v2; v2 = v2 && usable(d2, j + 2);
    buf = next_buf;
  }
  if constexpr (SCORE) {
    if (pending) {                     // exponentials of the very last block
#pragma unroll
      for (int kk = 0; kk < 8; ++kk) exp_pair(SubT{}, 1, kk);
      close_block(lds_all + ((buf + kBufs - 1) % kBufs) * kImage, 1, prev_kpos0, prev_nvalid, prev_edge);
    }
  }

  // ---- epilogue ---------------------------------------------------------------------------------
#pragma unroll
  for (int qb = 0; qb < QB; ++qb) {
    const float l_tot = l_run[qb] + __shfl_xor(l_run[qb], 32, 64);
    if constexpr (SCORE) {
      const float lp = l_prior[qb] + __shfl_xor(l_prior[qb], 32, 64);
      if (row_valid[qb] && hh == 0) mass[static_cast<size_t>(row[qb]) * hq + h] = lp / (lp + l_tot);
    } else {
      const float inv = 1.f / l_tot;
      if (row_valid[qb]) {
        if (out != nullptr) {                // (a caller that only wants the log-sum-exp passes none)
          bf16_t* op = out + (static_cast<size_t>(row[qb]) * hq + h) * kD;
#pragma unroll
          for (int db = 0; db < 4; ++db)
#pragma unroll
            for (int g4 = 0; g4 < 4; ++g4) {
              bf16_t v4[4];
#pragma unroll
              for (int e = 0; e < 4; ++e) v4[e] = static_cast<bf16_t>(o[qb][db][4 * g4 + e] * inv);
              // accumulator register i holds output dim 32db + 8(i/4) + 4hh + i%4
              *reinterpret_cast<uint2*>(op + 32 * db + 8 * g4 + 4 * hh) = *reinterpret_cast<uint2*>(v4);
            }
        }
        if (lse != nullptr && hh == 0)
          lse[static_cast<size_t>(row[qb]) * hq + h] = kLn2 * (m_ref[qb] + __builtin_amdgcn_logf(l_tot));
      }
    }
  }
  }   // work items of the round
  }   // rounds
}

template <int G, bool SCORE, int QB, bool REDO>
__global__ __launch_bounds__(64 * G, 2) void sparse_qk_kernel(
    const bf16_t* __restrict__ q, const int32_t* __restrict__ q_pos, const int32_t* __restrict__ cu_q,
    const bf16_t* __restrict__ k_pool, const bf16_t* __restrict__ v_pool, int n_blocks,
    const TileDesc* __restrict__ tiles, const int32_t* __restrict__ seg_tile_off, int max_tiles,
    const int32_t* __restrict__ order, const cc_segment* __restrict__ segs, const int32_t* __restrict__ req_seg_off, int hq, int hkv,
    int n_tiles_x, InvFreq inv_freq, bf16_t* __restrict__ out, float* __restrict__ lse,
    float* __restrict__ mass, const int32_t* __restrict__ redo, int redo_any, const int32_t* __restrict__ q_map,
    int map_pos, const bf16_t* __restrict__ v_shared, int n_shared_blocks, const int32_t* __restrict__ v_map) {
  // segment (score; heaviest first) or request (attention; longest context first; second pass: any order)
  sparse_qk<G, SCORE, QB, REDO>(REDO ? static_cast<int>(blockIdx.y) : order[blockIdx.y], q, q_pos, cu_q, k_pool, v_pool, n_blocks, tiles, seg_tile_off, max_tiles, segs, req_seg_off, hq, hkv, n_tiles_x, inv_freq, out, lse, mass, redo, redo_any, q_map, map_pos, v_shared, n_shared_blocks, v_map);
}

// Behind the wide score kernel: a segment's workgroup redoes its flagged tokens (normally none) and then selects.  (As
// launches of their own the second pass, which mostly reads its flags and leaves, was 5 us of a single request's step.)
template <int G, int QB>
__global__ __launch_bounds__(64 * G, 2) void redo_topn_kernel(
    const bf16_t* __restrict__ q, const bf16_t* __restrict__ k_pool, int n_blocks, const TileDesc* __restrict__ tiles,
    const int32_t* __restrict__ seg_tile_off, int max_tiles, const cc_segment* __restrict__ segs,
    const int32_t* __restrict__ req_seg_off, int hq, int hkv, int n_tiles_x, InvFreq inv_freq, float* mass,
    const int32_t* __restrict__ redo, int redo_any, const int32_t* __restrict__ block_tab, int32_t* __restrict__ sel_idx,
    int32_t* __restrict__ q_row, int32_t* __restrict__ q_pos, int32_t* __restrict__ slot_map, float* __restrict__ scores,
    uint32_t* key_buf) {
  sparse_qk<G, true, QB, true>(blockIdx.x, q, nullptr, nullptr, k_pool, nullptr, n_blocks, tiles, seg_tile_off, max_tiles, segs,
                               req_seg_off, hq, hkv, n_tiles_x, inv_freq, nullptr, nullptr, mass, redo, redo_any, nullptr, 0, nullptr, 0,
                               nullptr);
  __syncthreads();                                    // (what it wrote is read by the other wavefronts)
  topn_block<G>(blockIdx.x, mass, hq, false, block_tab, segs, sel_idx, q_row, q_pos, slot_map, scores, key_buf);
}

// ---- LDS of the plan's parts (no workgroup runs two of them) ---------------------------------------
constexpr int kPlanFused = 1024;       // segments up to which the whole plan is one launch
constexpr int kListBuckets = 512;
struct PlanLds {
  int32_t seg_tile_off[kPlanFused + 1];
  int wsum[4], carry;
  union {
    int key[kMaxOrdered];              // dispatch order
    struct {                           // list of workgroups
      int off[kMaxSorted + 1], low[kMaxSorted], n_short[kMaxSorted], bucket[kListBuckets], longest, first_short;
      uint32_t seen[kMaxSortedTiles];  // of a row tile: its request << 16 | its bucket
    } list;
  };
};

// ---- plan: the key tiles of every segment, in prompt order ---------------------------------------
// seg_tile_off[s] = number of tiles before segment s (exclusive scan of ceil(n_tokens/64)); run by
// one whole workgroup of 256 threads, into global memory or into LDS.
__device__ __forceinline__ void plan_scan(const cc_segment* __restrict__ segs, int n_segs,
                                          int32_t* seg_tile_off, PlanLds& lds) {
  int (&wsum)[4] = lds.wsum;
  int& carry_s = lds.carry;
  const int tid = threadIdx.x, lane = tid & 63, w = tid >> 6;
  if (tid == 0) carry_s = 0;
  __syncthreads();
  for (int s0 = 0; s0 < n_segs; s0 += 256) {
    const int s = s0 + tid;
    const int nt = s < n_segs ? (max(segs[s].n_tokens, 0) + kTile - 1) / kTile : 0;
    int incl = nt;                                   // inclusive scan inside the wavefront
#pragma unroll
    for (int o = 1; o < 64; o <<= 1) {
      const int up = __shfl_up(incl, o, 64);
      if (lane >= o) incl += up;
    }
    if (lane == 63) wsum[w] = incl;
    __syncthreads();
    int base = carry_s;
    for (int ww = 0; ww < w; ++ww) base += wsum[ww];
    if (s < n_segs) seg_tile_off[s] = base + incl - nt;
    __syncthreads();
    if (tid == 255) carry_s = base + incl;
    __syncthreads();
  }
  if (tid == 0) seg_tile_off[n_segs] = carry_s;
  __syncthreads();
}

// (n_listed: count to begin at 0 for the list's workgroups, or null)
__global__ __launch_bounds__(256) void plan_scan_kernel(const cc_segment* __restrict__ segs, int n_segs,
                                                         int32_t* __restrict__ seg_tile_off, int32_t* __restrict__ n_listed) {
  __shared__ PlanLds lds;
  if (n_listed != nullptr && threadIdx.x == 0) *n_listed = 0;
  plan_scan(segs, n_segs, seg_tile_off, lds);
}

// descriptor of tile j (and the redo flags cleared, spread over the n_fill workgroups that do this)
__device__ __forceinline__ void plan_fill(const cc_segment* __restrict__ segs, int n_segs,
                                          const int32_t* seg_tile_off, const int32_t* __restrict__ block_tab,
                                          int n_blocks, int max_tiles, TileDesc* __restrict__ tiles,
                                          int32_t* __restrict__ redo, int n_redo, int j, int n_fill) {
  for (int i = j; i < n_redo; i += n_fill * 256) redo[i] = 0;
  if (j >= min(seg_tile_off[n_segs], max_tiles)) return;
  int lo = 0, hi = n_segs - 1;                       // last segment with seg_tile_off[s] <= j
  while (lo < hi) {
    const int mid = (lo + hi + 1) >> 1;
    if (seg_tile_off[mid] <= j) lo = mid; else hi = mid - 1;
  }
  const cc_segment sg = segs[lo];
  const int kt = j - seg_tile_off[lo];
  TileDesc d;
  d.kpos0 = sg.logical_start + kTile * kt;
  d.nvalid = min(kTile, sg.n_tokens - kTile * kt);
  for (int i = 0; i < 4; ++i) {
    int b = -1;
    if (kBlock * i < d.nvalid) b = block_tab[sg.tab_off + (kTile / kBlock) * kt + i];
    d.blk[i] = (b >= 0 && b < n_blocks) ? b : -1;
  }
  d.seg = lo;
  uint32_t* to = reinterpret_cast<uint32_t*>(tiles + j);      // (all but `work`, which is written by others)
  *reinterpret_cast<uint4*>(to) = make_uint4(d.kpos0, d.nvalid, d.blk[0], d.blk[1]);
  *reinterpret_cast<uint2*>(to + 4) = make_uint2(d.blk[2], d.blk[3]);
  to[6] = d.seg;
}

// Dispatch order of the grid's y index: items sorted by decreasing key-side work, so that the last
// workgroups to start are the short ones.  BY_REQUEST: item = request, key = end of its context;
// otherwise item = segment, key = end of the segment (0 for segments that are not scored).
// order[rank] = item; ties keep index order, so the result is always a permutation.  More than
// kMaxOrdered items: identity.
//
// Beside order[] a work item per request is written (attention), so that a workgroup of the
// wide kernel finds what it needs of a request with ONE load instead of a chain of dependent
// ones (request -> segments -> tile offsets).  Called by whole workgroups; `block` is the
// workgroup's index among those that do this.
template <bool BY_REQUEST>
__device__ __forceinline__ void plan_order(const cc_segment* __restrict__ segs,
                                           const int32_t* __restrict__ req_seg_off,
                                           const int32_t* __restrict__ cu_q,
                                           const int32_t* seg_tile_off, int n_items,
                                           int32_t* __restrict__ order, WorkItem* __restrict__ items, int block, PlanLds& lds) {
  int (&key)[kMaxOrdered] = lds.key;
  const int i = block * 256 + threadIdx.x;
  auto emit = [&](int rank, int item) {
    order[rank] = item;
    if constexpr (BY_REQUEST) {
      WorkItem w = {};
      w.row = cu_q[item]; w.n_rows = cu_q[item + 1] - cu_q[item];
      w.j_begin = seg_tile_off[req_seg_off[item]];
      w.j_end = seg_tile_off[req_seg_off[item + 1]];
      items[item] = w;
    }
  };
  if (n_items > kMaxOrdered) {
    if (i < n_items) emit(i, i);
    return;
  }
  for (int j = threadIdx.x; j < n_items; j += 256) {
    int kv = 0;
    if constexpr (BY_REQUEST) {
      const int s_last = req_seg_off[j + 1] - 1;
      if (s_last >= req_seg_off[j]) kv = segs[s_last].logical_start + segs[s_last].n_tokens;
    } else {
      const cc_segment sg = segs[j];
      if (sg.kind == CC_SEG_CHUNK && sg.logical_start > 0) kv = sg.logical_start + sg.n_tokens;
    }
    key[j] = kv;
  }
  __syncthreads();
  if (i >= n_items) return;
  const int mine = key[i];
  int rank = 0;
  for (int j = 0; j < n_items; ++j) {
    const int other = key[j];
    rank += (other > mine || (other == mine && j < i)) ? 1 : 0;
  }
  emit(rank, i);
}

// The list of workgroups (WorkList), by one whole workgroup of 256 threads, or several where it is not sorted (block: the
// workgroup's number among n_groups).  Row tiles are counted per request and
// numbered through; a tile's work is the number of key tiles it sees.  The list begins request by request, long tiles
// first: the workgroups that run at a time then walk the same keys, which an XCD's L2 holds once (all tiles in the order
// of their work instead: 8B batch of 32 requests 2077 -> 2243 us, 4 x 32 k tokens 8.1 -> 8.2 ms).  The shortest tiles of all requests
// come last, long before short: they fill what the long ones leave at the end.  They are as many as make up the longest
// tile's work on every place, but none longer than kShortest key tiles, whose keys and values (32 KiB a tile and KV head) would
// not fit an XCD's L2 either (8 requests of 10k tokens on 600 workgroups: none of them 505 us, as many as
// make up half of that work 481, this 452; 3 of 20k on 500: 784 and 664, without the limit 677).  (Which of two tiles of the same work comes first is left to
// chance: it decides when a workgroup starts, not what it computes.)
// (more requests than are sorted, plan in launches of its own: a workgroup per 256 segments)
inline int list_groups(int n_requests, int n_segs) { return n_requests > kMaxSorted && n_segs > kPlanFused ? (n_segs + 255) / 256 : 1; }

// inclusive sum over a workgroup's 256 threads; wsum: the wavefronts' sums
__device__ __forceinline__ int scan_256(int v, int (&wsum)[4]) {
  const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
  int incl = v;
#pragma unroll
  for (int o = 1; o < 64; o <<= 1) {
    const int up = __shfl_up(incl, o, 64);
    if (lane >= o) incl += up;
  }
  __syncthreads();
  if (lane == 63) wsum[w] = incl;
  __syncthreads();
  for (int ww = 0; ww < w; ++ww) incl += wsum[ww];
  return incl;
}

__device__ void plan_list(const WorkList& list, const cc_segment* __restrict__ segs, int n_segs,
                          const int32_t* __restrict__ req_seg_off, int n_requests, const int32_t* __restrict__ cu_q,
                          TileDesc* __restrict__ tiles, int max_tiles, int block, int n_groups, PlanLds& lds) {
  constexpr int kBuckets = kListBuckets, kShortest = 160;
  int (&off)[kMaxSorted + 1] = lds.list.off, (&low)[kMaxSorted] = lds.list.low, (&n_short)[kMaxSorted] = lds.list.n_short;
  int (&bucket)[kListBuckets] = lds.list.bucket, (&wsum)[4] = lds.wsum, &longest = lds.list.longest, &first_short = lds.list.first_short;
  uint32_t (&seen)[kMaxSortedTiles] = lds.list.seen;
  const int tid = threadIdx.x, lane = tid & 63, w = tid >> 6;
  const bool scored = list.kind == WorkList::kScored;
  auto is_scored = [&](const cc_segment& sg) { return sg.kind == CC_SEG_CHUNK && sg.logical_start > 0 && sg.n_tokens > 0; };
  auto entry = [&](int r, int k) { return static_cast<int32_t>(static_cast<uint32_t>(r) << list.tile_bits) | k; };
  if (n_requests > kMaxSorted) {
    // (scores only) request by request, by the thread that has its first segment.  Without gaps: the places of a list that begins
    // each request where its key tiles begin come in a pattern, which the dispatcher gives to some of the XCDs and shader
    // engines only (4 query heads, 2100 requests of 4 x 500 tokens: 12 of 32 places, 11.3 ms; 6.6 without).
    for (int s0 = 256 * block, base = 0; s0 < (n_groups > 1 ? min(256 * (block + 1), n_segs) : n_segs); s0 += 256) {
      const int s = s0 + tid;
      const cc_segment sg = segs[min(s, n_segs - 1)];
      const bool first = s < n_segs && sg.req >= 0 && sg.req < n_requests && (s == 0 || segs[s - 1].req != sg.req);
      const int cnt = s < n_segs && is_scored(sg) ? sg.n_tokens : 0;
      int rows = cnt;                                      // inclusive sum inside the wavefront, then the request's
#pragma unroll
      for (int o = 1; o < 64; o <<= 1) {
        const int up = __shfl_up(rows, o, 64);
        if (lane >= o) rows += up;
      }
      const uint64_t next = __ballot(first) & ~(~0ull >> (63 - lane));      // requests that begin behind this lane
      const int last = next != 0 ? __ffsll(static_cast<unsigned long long>(next)) - 2 : 63;
      rows = __shfl(rows, last, 64) - rows + cnt;
      if (first && next == 0)
        for (int t = s - lane + 64; t < n_segs && segs[t].req == sg.req; ++t) rows += is_scored(segs[t]) ? segs[t].n_tokens : 0;
      const int n = first ? (rows + list.rows - 1) / list.rows : 0, incl = scan_256(n, wsum);
      const int all = wsum[0] + wsum[1] + wsum[2] + wsum[3];
      if (n_groups > 1) {                                  // (places in any order of the workgroups)
        if (tid == 0) lds.carry = atomicAdd(&tiles[max_tiles - 1].work, all);
        __syncthreads();
        base = lds.carry;
      }
      for (int l = 0; l < 64; ++l) {
        const int at = base + __builtin_amdgcn_readlane(incl - n, l), n_l = __builtin_amdgcn_readlane(n, l), r = __builtin_amdgcn_readlane(sg.req, l);
        for (int k = lane; k < n_l && at + k < max_tiles - 1; k += 64) tiles[at + k].work = entry(r, n_l - 1 - k);
      }
      base += all;
      if (n_groups == 1 && tid == 0) tiles[max_tiles - 1].work = min(base, max_tiles - 1);
    }
    return;
  }
  // rows, then row tiles of every request; low: position of its first scored token
  for (int r = tid; r < n_requests; r += 256) { off[r] = scored ? 0 : max(cu_q[r + 1] - cu_q[r], 0); low[r] = 0x7fffffff; n_short[r] = 0; }
  for (int b = tid; b < kBuckets; b += 256) bucket[b] = 0;
  if (tid == 0) longest = 1;
  __syncthreads();
  for (int s = tid; s < n_segs; s += 256) {
    const cc_segment sg = segs[s];
    if (scored && is_scored(sg) && sg.req >= 0 && sg.req < n_requests) {
      atomicAdd(&off[sg.req], sg.n_tokens);
      atomicMin(&low[sg.req], sg.logical_start);
    }
    atomicMax(&longest, sg.logical_start + max(sg.n_tokens, 0));
  }
  __syncthreads();
  int carry = 0;
  for (int r0 = 0; r0 < n_requests; r0 += 256) {           // exclusive scan in place (off[n_requests]: all)
    const int r = r0 + tid, n = r < n_requests ? (off[r] + list.rows - 1) / list.rows : 0;
    int incl = n;
#pragma unroll
    for (int o = 1; o < 64; o <<= 1) {
      const int up = __shfl_up(incl, o, 64);
      if (lane >= o) incl += up;
    }
    if (lane == 63) wsum[w] = incl;
    __syncthreads();
    int base = carry;
    for (int ww = 0; ww < w; ++ww) base += wsum[ww];
    carry += wsum[0] + wsum[1] + wsum[2] + wsum[3];
    if (r < n_requests) off[r] = base + incl - n;
    __syncthreads();
  }
  if (tid == 0) off[n_requests] = carry;
  __syncthreads();
  const int total = min(carry, max_tiles - 1);
  if (tid == 0) tiles[max_tiles - 1].work = total;
  auto request_of = [&](int j) {                           // last request with off[r] <= j
    int lo = 0, hi = n_requests - 1;
    while (lo < hi) {
      const int mid = (lo + hi + 1) >> 1;
      if (off[mid] <= j) lo = mid; else hi = mid - 1;
    }
    return lo;
  };
  // one request, or all start at once, or too many to sort: request by request
  if (n_requests == 1 || total <= list.places || total > kMaxSortedTiles) {
    for (int j = tid; j < total; j += 256) {
      const int r = request_of(j), end = min(off[r + 1], total);
      tiles[off[r] + end - 1 - j].work = entry(r, j - off[r]);
    }
    return;
  }
  int shift = 0;
  while ((longest / kTile >> shift) >= kBuckets) ++shift;
  // (bucket 0 holds the longest)
  for (int j = tid; j < total; j += 256) {
    const int r = request_of(j), k = j - off[r];
    const int last = scored ? low[r] + list.rows * (k + 1) : list.q_pos[min(cu_q[r] + list.rows * (k + 1), cu_q[r + 1]) - 1];
    const int at = kBuckets - 1 - min(max(last / kTile >> shift, 0), kBuckets - 1);
    seen[j] = static_cast<uint32_t>(r) << 16 | static_cast<uint32_t>(at);
    atomicAdd(&bucket[at], 1);
  }
  const int cap = max(kBuckets - 1 - (kShortest >> shift), 0);      // (first bucket that may count as short)
  if (tid == 0) first_short = cap;
  __syncthreads();
  {
    // thread i has buckets 2 i, 2 i + 1; work behind them, in key tiles
    const int a = bucket[2 * tid] * (kBuckets - 2 * tid), b = bucket[2 * tid + 1] * (kBuckets - 1 - 2 * tid);
    const int incl = scan_256(a + b, wsum), all = wsum[0] + wsum[1] + wsum[2] + wsum[3];
    const int behind = all - incl, enough = list.places * ((longest / kTile >> shift) + 1);
    if (behind < enough && behind + b >= enough) first_short = max(2 * tid + 1, cap);
    else if (behind + b < enough && behind + b + a >= enough) first_short = max(2 * tid, cap);
    bucket[2 * tid] = bucket[2 * tid + 1] = 0;
  }
  __syncthreads();
  for (int j = tid; j < total; j += 256)
    if (static_cast<int>(seen[j] & 0xffff) >= first_short) atomicAdd(&n_short[seen[j] >> 16], 1);
  __syncthreads();
  // a request's first n_short tiles are the short ones (its rows are mostly in prompt order)
  for (int j = tid; j < total; j += 256) {
    const int r = seen[j] >> 16;
    if (j - off[r] < n_short[r]) atomicAdd(&bucket[seen[j] & 0xffff], 1);
  }
  __syncthreads();
  const int a = bucket[2 * tid], b = bucket[2 * tid + 1], incl = scan_256(a + b, wsum);
  const int n_long = total - (wsum[0] + wsum[1] + wsum[2] + wsum[3]);
  bucket[2 * tid] = incl - a - b;
  bucket[2 * tid + 1] = incl - b;
  int before = 0;                                          // long tiles of the requests in front
  for (int r0 = 0; r0 < n_requests; r0 += 256) {
    const int r = r0 + tid, first = r < n_requests ? min(off[r], total) : total, end = r < n_requests ? min(off[r + 1], total) : total;
    const int n = end - first - (r < n_requests ? n_short[r] : 0), upto = scan_256(n, wsum);
    if (r < n_requests) low[r] = before + upto - n;
    before += wsum[0] + wsum[1] + wsum[2] + wsum[3];
  }
  __syncthreads();
  for (int j = tid; j < total; j += 256) {
    const int r = seen[j] >> 16, k = j - off[r], n = min(off[r + 1], total) - off[r];
    const int at = k < n_short[r] ? n_long + atomicAdd(&bucket[seen[j] & 0xffff], 1) : low[r] + n - 1 - k;
    tiles[at].work = entry(r, k);
  }
}

// The whole plan in ONE launch: the first n_fill workgroups write descriptors, the next the
// dispatch order, and the last n_list the list of workgroups if there is to be one.  Up to kPlanFused segments every workgroup
// repeats the (tiny) scan into LDS, which saves a launch and a wait between dependent kernels: a single request's step is a dozen
// kernels of a few microseconds.  More segments: the scan is a launch in front.
struct PlanArgs {
  const cc_segment* segs;
  const int32_t *req_seg_off, *cu_q, *block_tab;
  int n_segs, n_items, n_requests, n_blocks, max_tiles, n_redo, n_fill, n_list, n_groups;      // n_groups: workgroups of the plan
  bool scanned;                      // seg_tile_off is there
  int32_t *seg_tile_off, *order, *redo;
  WorkItem* items;
  TileDesc* tiles;
  WorkList list;
};

template <bool BY_REQUEST>
__device__ __forceinline__ void plan_part(const PlanArgs& a, int block, PlanLds& lds) {
  const int32_t* seg_tile_off = a.seg_tile_off;
  if (!a.scanned) {
    plan_scan(a.segs, a.n_segs, lds.seg_tile_off, lds);
    if (block == 0)
      for (int s = threadIdx.x; s <= a.n_segs; s += 256) a.seg_tile_off[s] = lds.seg_tile_off[s];
    seg_tile_off = lds.seg_tile_off;
  }
  if (block < a.n_fill)
    plan_fill(a.segs, a.n_segs, seg_tile_off, a.block_tab, a.n_blocks, a.max_tiles, a.tiles, a.redo, a.n_redo,
              block * 256 + threadIdx.x, a.n_fill);
  else if (block < a.n_groups - a.n_list)
    plan_order<BY_REQUEST>(a.segs, a.req_seg_off, a.cu_q, seg_tile_off, a.n_items, a.order, a.items, block - a.n_fill, lds);
  else
    plan_list(a.list, a.segs, a.n_segs, a.req_seg_off, a.n_requests, a.cu_q, a.tiles, a.max_tiles,
              block - (a.n_groups - a.n_list), a.n_list, lds);
}

template <bool BY_REQUEST>
__global__ __launch_bounds__(256) void plan_fused_kernel(PlanArgs a) {
  __shared__ PlanLds lds;
  plan_part<BY_REQUEST>(a, blockIdx.x, lds);
}

// The attention's plan and the scatter in front of it need nothing of each other: its first workgroups make the plan, the
// others scatter.  (A plan launched behind the scatter: 4 us of one request's step, with a list 10 - 15 us of a batch's.)
__global__ __launch_bounds__(256) void scatter_plan_kernel(
    PlanArgs a, const bf16_t* __restrict__ k_new, const bf16_t* __restrict__ v_new, const int32_t* __restrict__ q_pos,
    const int32_t* __restrict__ slot_map, int n_q_tot, int hkv, InvFreq inv_freq, bf16_t* __restrict__ k_pool,
    bf16_t* __restrict__ v_pool, int n_blocks, const int32_t* __restrict__ src_rows, const bf16_t* __restrict__ v_shared,
    int n_shared_blocks, int32_t* __restrict__ v_map) {
  __shared__ PlanLds lds;
  const int block = blockIdx.x;
  if (block < a.n_groups)
    plan_part<true>(a, block, lds);
  else
    rope_scatter_rows<bf16_t, kD>(block - a.n_groups, scatter_rows(n_q_tot), k_new, v_new, q_pos, slot_map, n_q_tot, hkv, inv_freq, k_pool, v_pool,
                                  n_blocks, src_rows, v_shared, n_shared_blocks, v_map);
}

constexpr int kAttnQB = 1;     // 32 query tokens per workgroup in the attention kernel
constexpr int kScoreQB = 2;    // 64 in the score kernel (no O accumulator, so registers allow it)

template <int G>
void launch_attn_g(const cc_ctx* ctx, const void* q, const int32_t* q_pos, const int32_t* cu_q,
                   int max_q_per_req, const void* k_pool, const void* v_pool, int n_blocks,
                   const Plan& pl, const cc_segment* segs, const int32_t* req_seg_off,
                   int n_requests, void* out, float* lse, const int32_t* redo, const int32_t* q_map,
                   int map_pos, hipStream_t stream, const ValueSource& vs) {
  const int hkv = ctx->cfg.n_kv_heads, n_tiles = (max_q_per_req + 32 * kAttnQB - 1) / (32 * kAttnQB);
#define CC_KARGS static_cast<const bf16_t*>(q), q_pos, cu_q, static_cast<const bf16_t*>(k_pool),                 \
                 static_cast<const bf16_t*>(v_pool), n_blocks, pl.tiles, pl.seg_tile_off, pl.max_tiles,         \
                 pl.order, segs, req_seg_off, ctx->cfg.n_q_heads, hkv, n_tiles, ctx->inv_freq,                  \
                 static_cast<bf16_t*>(out), lse, static_cast<float*>(nullptr), redo, pl.redo_any, q_map, map_pos, \
                 static_cast<const bf16_t*>(vs.v_shared), vs.n_shared_blocks, static_cast<const int32_t*>(vs.v_map)
  if (redo != nullptr)
    hipLaunchKernelGGL((sparse_qk_kernel<G, false, kAttnQB, true>), dim3(1, n_requests), dim3(64 * G), 0, stream, CC_KARGS);
  else
    hipLaunchKernelGGL((sparse_qk_kernel<G, false, kAttnQB, false>), dim3(hkv * n_tiles, n_requests), dim3(64 * G), 0,
                       stream, CC_KARGS);
#undef CC_KARGS
}

// the narrow score kernel over everything, or - behind the wide one (redo) - over what that flagged; then the selection
template <int G>
void launch_select_g(const cc_ctx* ctx, const void* q, const void* k_pool, int n_blocks, const Plan& pl,
                     const int32_t* req_seg_off, int max_seg_tokens, float* mass, const int32_t* redo, const TopnJob& topn,
                     hipStream_t stream) {
  const int hkv = ctx->cfg.n_kv_heads, n_tiles = (max_seg_tokens + 32 * kScoreQB - 1) / (32 * kScoreQB);
  if constexpr (G % 4 == 0) {
    if (redo != nullptr) {
      hipLaunchKernelGGL((redo_topn_kernel<G, kScoreQB>), dim3(topn.n_segs), dim3(64 * G), 0, stream, static_cast<const bf16_t*>(q),
                         static_cast<const bf16_t*>(k_pool), n_blocks, pl.tiles, pl.seg_tile_off, pl.max_tiles, topn.segs,
                         req_seg_off, ctx->cfg.n_q_heads, hkv, n_tiles, ctx->inv_freq, mass, redo, pl.redo_any, topn.block_tab, topn.sel_idx,
                         topn.q_row, topn.q_pos, topn.slot_map, topn.scores, topn.key_buf);
      return;
    }
  }
  hipLaunchKernelGGL((sparse_qk_kernel<G, true, kScoreQB, false>), dim3(hkv * n_tiles, topn.n_segs), dim3(64 * G), 0, stream,
                     static_cast<const bf16_t*>(q), static_cast<const int32_t*>(nullptr),
                     static_cast<const int32_t*>(nullptr), static_cast<const bf16_t*>(k_pool),
                     static_cast<const bf16_t*>(nullptr), n_blocks, pl.tiles, pl.seg_tile_off, pl.max_tiles,
                     pl.order, topn.segs, req_seg_off, ctx->cfg.n_q_heads, hkv, n_tiles, ctx->inv_freq,
                     static_cast<bf16_t*>(nullptr), static_cast<float*>(nullptr), mass, redo, pl.redo_any,
                     static_cast<const int32_t*>(nullptr), 0, static_cast<const bf16_t*>(nullptr), 0,
                     static_cast<const int32_t*>(nullptr));
  launch_topn(ctx, mass, topn, false, stream);
}

bool group_supported(const cc_ctx* ctx) {
  if (ctx->cfg.dtype != CC_BF16 || ctx->cfg.head_dim != kD) return false;
  const int g = ctx->cfg.n_q_heads / ctx->cfg.n_kv_heads;
  return g == 1 || g == 2 || g == 4 || g == 8;
}

}  // namespace

// workspace: seg_tile_off[n_segs + 1] | order[n_segs] (requests never outnumber segments) |
//            items[n_segs] | tiles | redo flags
static size_t plan_ints_bytes(int n_segs) {
  return (static_cast<size_t>(2 * n_segs + 1) * sizeof(int32_t) + 255) / 256 * 256;
}
size_t plan_head_bytes(int n_segs) {
  return plan_ints_bytes(n_segs) + (static_cast<size_t>(n_segs) * sizeof(WorkItem) + 255) / 256 * 256;
}

static size_t plan_bytes_impl(int n_segs, int max_tiles) {
  return plan_head_bytes(n_segs) + static_cast<size_t>(max_tiles) * sizeof(TileDesc);
}

Plan run_plan(const cc_ctx* ctx, void* ws, const cc_segment* segs, int n_segs, const int32_t* req_seg_off, int n_requests, bool by_request,
              const int32_t* cu_q, const int32_t* block_tab, int n_blocks, int max_tiles, int n_redo, const WorkList& list,
              const ScatterJob* scatter, hipStream_t stream) {
  Plan pl;
  pl.seg_tile_off = static_cast<int32_t*>(ws);
  pl.order = pl.seg_tile_off + n_segs + 1;
  pl.items = reinterpret_cast<WorkItem*>(static_cast<char*>(ws) + plan_ints_bytes(n_segs));
  pl.tiles = reinterpret_cast<TileDesc*>(static_cast<char*>(ws) + plan_head_bytes(n_segs));
  pl.max_tiles = max_tiles;
  pl.redo_any = n_redo - 1;
  pl.redo = n_redo > 0 ? reinterpret_cast<int32_t*>(pl.tiles + max_tiles) : nullptr;
  const bool listed = list.kind != WorkList::kNone;
  const int n_items = by_request ? n_requests : n_segs, n_fill = (max_tiles + 255) / 256;
  const int n_order = listed && !by_request ? 0 : (n_items + 255) / 256;      // (the wide score kernel goes by the list alone)
  const int n_list = listed ? list_groups(n_requests, n_segs) : 0;
  const int n_groups = n_fill + n_order + n_list;
  const bool scanned = n_segs > kPlanFused;
  if (scanned)
    hipLaunchKernelGGL(plan_scan_kernel, dim3(1), dim3(256), 0, stream, segs, n_segs, pl.seg_tile_off, n_list > 1 ? &pl.tiles[max_tiles - 1].work : nullptr);
  const PlanArgs a{segs, req_seg_off, cu_q, block_tab, n_segs, n_items, n_requests, n_blocks, max_tiles, n_redo, n_fill, n_list, n_groups, scanned,
                   pl.seg_tile_off, pl.order, pl.redo, pl.items, pl.tiles, list};
  if (by_request && scatter != nullptr && scatter->n_rows > 0)
    hipLaunchKernelGGL(scatter_plan_kernel, dim3(n_groups + scatter_groups(scatter->n_rows)), dim3(256), 0, stream,
                       a, static_cast<const bf16_t*>(scatter->k_new), static_cast<const bf16_t*>(scatter->v_new),
                       scatter->q_pos, scatter->slot_map, scatter->n_rows, ctx->cfg.n_kv_heads, ctx->inv_freq,
                       static_cast<bf16_t*>(scatter->k_pool), static_cast<bf16_t*>(scatter->v_pool), scatter->n_blocks,
                       scatter->src_rows, static_cast<const bf16_t*>(scatter->vs.v_shared), scatter->vs.n_shared_blocks,
                       scatter->vs.v_map);
  else if (by_request)                                 // attention: the grid's y index walks requests
    hipLaunchKernelGGL(plan_fused_kernel<true>, dim3(n_groups), dim3(256), 0, stream, a);
  else                                                 // score without a list: it walks segments
    hipLaunchKernelGGL(plan_fused_kernel<false>, dim3(n_groups), dim3(256), 0, stream, a);
  return pl;
}

// Which SCORE kernel runs.  From one round of 128-token workgroups on (two per compute unit of an MI355X: kMinWideGrid) the wide one
// with four column blocks and one key stream.  Below, its small form (64 tokens, two key streams, one workgroup per
// compute unit) as long as its workgroups run in about one round, or in two with prompts long enough that the longest chain of
// tiles decides: it halves that chain.  In between the narrow kernel, of which two workgroups share a unit (later where a
// KV head has 8 query heads: a narrow workgroup takes all of them, so there are half as many, and the wide one's line is lower).  Whole
// cc_select call, narrow / wide, us, by the 128-token workgroups that the rule estimates and the chunks of the requests.  32 / 8
// heads: 288 (3 of 40 x 17-60) 135 / 154, 288 (12 of 3 x 160) 48 / 56, 320 (8 of 6 x 100) 53 / 57, 384 (6 of 3 x 440) 76 / 84,
// 448 (2 of 6 x 700) 182 / 201, 488 (12 x 700) 330 / 309, 552 (12 x 800) 419 / 377, 576 (12 of 20 x 17-60) 136 / 103.  8 heads per KV head: 276 (16 / 2, 12 x 800)
// 294 / 283, 312 (16 / 2, 6 of 40 x 17-60) 133 / 171, 368 (64 / 8, 30 x 100) 150 / 167, 368 (16 / 2, 4 of 5 x 700) 141 / 168, 512 (64 / 8, 4 of 10 x 100) 99 / 95,
// 552 (16 / 2, 2 of 12 x 800) 440 / 379.
// Narrow / small, by the 64-token workgroups that the rule estimates.  32 / 8
// heads: 130 (3 x 512) 49.5 / 37.2, 259 (5 x 512) 72.9 / 50.5, 306 (2 of 5 x 300) 55.4 / 49.6, 392 (3 of 3 x 512) 57.5 / 56.9,
// 421 (8 of 3 x 200) 37.4 / 48.6, 522 (4 of 3 x 512) 60.7 / 62.9, 603 (9 x 600) 164 / 156, 763 (4 of 6 x 300) 92.2 / 95.7.  64 / 8:
// 425 (4 of 5 x 100) 39.9 / 49.3, 612 (2 of 5 x 300) 75.3 / 80.3.  16 / 2: 301 (9 x 600) 177 / 91.3, 612 (8 of 5 x 300) 79.2 / 80.3,
// 706 (4 of 5 x 700) 141 / 131.
// The wide ATTENTION kernel is faster at every size measured, down to 64 workgroups (7-25 %), so it has no such limit.
constexpr int kMinWideGrid = 512, kMinWideGrid8 = 360;
constexpr int kOneRoundScore = 288, kTwoRoundScore = 540;

// (the chunks' lengths are on the device: the workgroups are estimated from the batch's tokens, taking a request's
// segments for equally long chunks and a short question; the first chunk is not scored)
static int64_t scored_tokens(int n_tok, int n_segs, int n_requests) {
  const int64_t per_req = std::max(n_segs / n_requests, 2), scored = per_req > 2 ? per_req - 2 : 1, chunks = scored + 1;
  return n_tok * scored / chunks;
}
static int64_t wide_score_groups(int n_q_heads, int n_tok, int n_segs, int n_requests) {
  const int64_t requests = std::min(n_requests, n_segs), per_request = scored_tokens(n_tok, n_segs, n_requests) / requests;
  return n_q_heads / 4 * requests * ((per_request + 127) / 128);
}
static bool wide_score_grid(int n_q_heads, int n_kv_heads, int n_tok, int n_segs, int n_requests) {
  return wide_score_groups(n_q_heads, n_tok, n_segs, n_requests) >= (n_q_heads / n_kv_heads > 4 ? kMinWideGrid8 : kMinWideGrid);
}
// Products of 16 columns where the call is long enough for the chip's power budget to hold its clock down: from about 0.1 TFLOP on (128-token workgroups x a
// request's tokens are 2^-16 of the flops), unless little more than one round of workgroups (512) leaves the chip half idle behind it, or chunks of a key tile or less
// put masks and their beginnings between the products; else 32 columns.  32 columns / 16, us, by
// workgroups and that product.  32 / 8 heads: 552 (1 of 12 x 800, 5.3 M) 377 / 382, 576 (12 of 20 x 17-60, 0.2 M) 103 / 111, 864 (9 of 3 x 743, 1.7 M)
// 171 / 161, 1280 (5 of 23 x 184, 4.7 M) 356 / 341, 3320 (5 of 23 x 477, 30 M) 1676 / 1610.  64 / 8: 512 (4 of 10 x 100, 0.5 M) 95 / 102, 5760 (5 of 23 x 414, 46 M) 2620 /
// 2558.  16 / 2: 480 (5 of 13 x 247, 1.3 M) 139 / 150, 896 (8 of 6 x 692, 3.2 M) 251 / 232, 1008 (36 of 3 x 413, 1.2 M) 134 / 135.  8 / 2: 646 (19 of 4 x 681, 1.5 M) 140 / 140,
// 1140 (57 of 5 x 247, 1.5 M) 131 / 128.  By tokens of a segment in the mean: 45 (64 / 8, 35 of 18 x 37-56, 3.9 M) 467 / 492, 66 (32 / 8, 22 of 20 x 49-74, 3.1 M) 282 / 289, 76 (33 of
// 27 x 58-87, 10.7 M) 1003 / 989.  (Over 150 calls of 1 to 64 requests this takes 0.03 % longer than the better of the two for each, 16 columns throughout 1 - 2 %.)
constexpr int64_t kPowerLine = 1400000, kPowerGrid = 680, kPowerSegment = 72;
static bool score_held_by_power(int n_q_heads, int n_tok, int n_segs, int n_requests) {
  const int64_t groups = wide_score_groups(n_q_heads, n_tok, n_segs, n_requests);
  return groups >= kPowerGrid && n_tok >= kPowerSegment * n_segs && groups * (n_tok / std::min(n_requests, n_segs)) >= kPowerLine;
}
static bool small_score_grid(int n_q_heads, int n_kv_heads, int n_tok, int n_segs, int n_requests) {
  const int64_t groups = n_q_heads / 4 * scored_tokens(n_tok, n_segs, n_requests) / 64;
  const int tokens_per_group = n_q_heads / n_kv_heads > 4 ? 4 : 7;
  return groups <= std::max(kOneRoundScore, std::min(n_tok / n_requests / tokens_per_group, kTwoRoundScore));
}

// Where there is a workgroup for every compute unit, but a request has one scored chunk (with the question three segments) and that
// fits a workgroup of the narrow kernel, a wide workgroup is as good as half empty and its longer prologue decides.  Whole call, wide /
// narrow, us, two chunks and a question.  64 / 8 heads: 100 requests, chunks of 20-30 tokens 91 / 72, 60-64 94 / 82, but
// 60-80 (two narrow workgroups a chunk) 109 / 134, and three chunks of 17-33 115 / 124.  32 / 8: 100 of 40-50 62 / 46.
// 16 / 2: 300 of 40-50 97 / 84.  The narrow kernel needs a dispatch order of the segments, which takes some 20 us beyond kPlanFused and only many heads
// outweigh: 1000 of 40-50 on 8 / 1 147 / 172, 16 / 2 225 / 233, 32 / 8 364 / 312, 64 / 8 680 / 630.  Nothing is scored of a chunk and a question
// (1000 on 32 / 8: 34 / 83).
static bool one_score_tile(int n_q_heads, int max_seg_tokens, int n_segs, int n_requests) {
  return static_cast<int64_t>(n_q_heads / 4) * n_requests >= 256 && max_seg_tokens <= 32 * kScoreQB && n_segs > 2 * static_cast<int64_t>(n_requests) &&
         n_segs <= 3 * static_cast<int64_t>(n_requests) && (n_segs <= kPlanFused || n_q_heads >= 32);
}

bool attn_mfma_supported(const cc_ctx* ctx) { return group_supported(ctx); }
bool score_mfma_supported(const cc_ctx* ctx) { return group_supported(ctx); }

size_t mfma_plan_bytes(int n_segs, int max_tiles, int n_q_max) {
  return plan_bytes_impl(n_segs, max_tiles) + redo_entries(n_q_max) * sizeof(int32_t);
}

void launch_attn_mfma(const cc_ctx* ctx, const void* q, const int32_t* q_pos, const int32_t* cu_q,
                      int n_q_tot, int max_q_per_req, const void* k_pool, const void* v_pool,
                      int n_blocks, const int32_t* block_tab, const cc_segment* segs, int n_segs,
                      const int32_t* req_seg_off, int n_requests, void* out, float* lse,
                      void* plan_ws, int max_tiles, const int32_t* q_map, int map_pos, hipStream_t stream,
                      const AttnByProduct* by, const ValueSource& vs, const ScatterJob* scatter) {
  // Wide kernel first where the head group allows it; the narrow kernel then redoes the 64-row
  // tiles the wide one flagged (normally none: its workgroups read one flag and exit).
  const bool wide = ctx->impl != CC_IMPL_MFMA_NARROW && attn_v2_supported(ctx);
  const int n_redo = wide ? static_cast<int>(redo_entries(n_q_tot)) : 0;
  WorkList list;
  if (wide) list = attn_v2_list(ctx, map_pos == 0 ? q_pos : nullptr, n_q_tot, max_q_per_req, n_requests, max_tiles);
  const Plan pl = run_plan(ctx, plan_ws, segs, n_segs, req_seg_off, n_requests, true, cu_q, block_tab, n_blocks, max_tiles, n_redo, list, scatter, stream);
  if (wide)
    launch_attn_v2(ctx, q, q_pos, n_q_tot, max_q_per_req, k_pool, v_pool, pl, req_seg_off, n_requests,
                   out, lse, pl.redo, q_map, map_pos, by != nullptr ? by->snap_index : nullptr,
                   by != nullptr ? by->cum : nullptr, by != nullptr ? by->s_max : 0, list, stream, vs);
  if (by != nullptr) {
    by->wide = wide;
    by->redo = pl.redo;
    by->redo_any = pl.redo_any;
  }
  const int32_t* redo = pl.redo;
#define CC_ARGS ctx, q, q_pos, cu_q, max_q_per_req, k_pool, v_pool, n_blocks, pl, segs, req_seg_off, n_requests, out, lse, redo, q_map, map_pos, stream, vs
  switch (ctx->cfg.n_q_heads / ctx->cfg.n_kv_heads) {
    case 1: launch_attn_g<1>(CC_ARGS); break;
    case 2: launch_attn_g<2>(CC_ARGS); break;
    case 4: launch_attn_g<4>(CC_ARGS); break;
    default: launch_attn_g<8>(CC_ARGS); break;
  }
#undef CC_ARGS
}

void launch_select_mfma(const cc_ctx* ctx, const void* q, const void* k_pool, int n_blocks,
                        const int32_t* req_seg_off, int n_requests, int max_seg_tokens, float* mass,
                        void* plan_ws, int max_tiles, int n_tok, const TopnJob& topn, hipStream_t stream) {
  const cc_segment* segs = topn.segs;
  const int32_t* block_tab = topn.block_tab;
  const int n_segs = topn.n_segs;
  // Wide kernel first where the head group and the grid allow it; the narrow kernel then
  // redoes the granules the wide one flagged (normally none: a segment's workgroup reads its flags and goes on to select).
  const int hq = ctx->cfg.n_q_heads, hkv = ctx->cfg.n_kv_heads;
  const bool forced = ctx->impl == CC_IMPL_MFMA_WIDE;
  const bool one_tile = !forced && one_score_tile(hq, max_seg_tokens, n_segs, n_requests);
  const bool big = forced || wide_score_grid(hq, hkv, n_tok, n_segs, n_requests);
  const bool small = !big && !one_tile && small_score_grid(hq, hkv, n_tok, n_segs, n_requests);
  const int rows = small ? 64 : 128;
  const bool wide = ctx->impl != CC_IMPL_MFMA_NARROW && score_v2_supported(ctx) && ((big && !one_tile) || small) &&
                    list_can_name(n_requests, n_tok / rows + 1);      // (empty requests count; a request may have all tokens)
  const int n_redo = wide ? static_cast<int>(score_redo_entries(n_tok)) : 0;
  WorkList list;
  if (wide) {
    list.kind = WorkList::kScored;
    list.rows = rows;
    list.tile_bits = list_tile_bits(n_requests);
    list.places = std::max((small ? 256 : 512) / (ctx->cfg.n_q_heads / 4), 1);
  }
  const Plan pl = run_plan(ctx, plan_ws, segs, n_segs, req_seg_off, n_requests, false, nullptr, block_tab, n_blocks, max_tiles, n_redo, list, nullptr, stream);
  // (CC_IMPL_MFMA_WIDE: the same sums at every size)
  const ScoreForm form = small ? ScoreForm::kSmall : forced || score_held_by_power(hq, n_tok, n_segs, n_requests) ? ScoreForm::kBig16 : ScoreForm::kBig;
  if (wide) launch_score_v2(ctx, q, k_pool, pl, segs, req_seg_off, n_requests, n_tok, mass, pl.redo, form, list, stream);
  const int32_t* redo = pl.redo;
#define CC_ARGS ctx, q, k_pool, n_blocks, pl, req_seg_off, max_seg_tokens, mass, redo, topn, stream
  switch (ctx->cfg.n_q_heads / ctx->cfg.n_kv_heads) {
    case 1: launch_select_g<1>(CC_ARGS); break;
    case 2: launch_select_g<2>(CC_ARGS); break;
    case 4: launch_select_g<4>(CC_ARGS); break;
    default: launch_select_g<8>(CC_ARGS); break;
  }
#undef CC_ARGS
}

}  // namespace cc
