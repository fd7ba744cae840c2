// cc_sparse_prefill's attention for head groups that are a multiple of 4 (bf16, head_dim 128):
// per-token form of Eq. (1); Sec. 4 "Selective Token Recomputation".
//
// One workgroup = 8 wavefronts, two per SIMD (up to 256 registers each), in one of two forms:
//   KS = 1: 4 query heads of one KV head x 64 query rows of the compact list; wavefront w owns head w % 4 and
//           rows 32 (w / 4) .. + 31, and all walk the same key tiles;
//   KS = 2: 4 query heads x 32 rows; wavefronts 0-3 walk the even key tiles, 4-7 the odd ones, and the two
//           halves of a (head, row) meet in LDS at the end.  Twice the workgroups with half the tiles each,
//           for grids that leave compute units idle.
// The running output (64 registers) and the rotated queries (32) sit in accumulation registers, two 32-key
// score blocks (32), the packed probabilities (16) and the operand ring (32) in vector registers.
// While one wavefront of a SIMD waits (for LDS, for its exponentials - a transcendental does not run beside a
// matrix instruction of its own wavefront) the other one keeps the matrix pipe busy.
//
// Orientation and key permutation are those of mfma_tile.h: S^T = K Q^T, O^T = V^T P^T with
// v_mfma_f32_32x32x16_bf16, a lane holds one query column, P^T goes from the accumulators to
// the second product without leaving the lane.
//
// Schedule.  A wavefront's keys advance in 32-key blocks b = 0, 1, 2, ... (two per 64-key tile).  Its matrix
// instructions are   S(b+1), PV(b), S(b+2), PV(b+1), ...   8 MFMAs each, and under every MFMA one exponential
// of a block whose S is already complete: the first half of exp(b) under PV(b-1), the second half
// under S(b+1).  Per element that is one v_exp_f32 and one add into the row sum: the reference is
// already subtracted (it enters through the C operand of the block's first MFMA).  The row sum
// takes the unrounded exponentials (summing the bf16 roundings instead - one v_dot2c_f32_bf16 per
// pair - was measured too: it biases the log-sum-exp by up to 1.4e-3 when the weights are nearly
// uniform, and saves nothing that shows).  The pack of a pair to bf16 and its two adds run one step
// late, in front of the next exponential, so that no instruction reads a transcendental result
// right behind its issue.
//
// Softmax reference: m_ref = maximum of the row's first 32-key block (of its key stream), for the whole row (fp32 and
// bf16 share the exponent range, so p = exp2(S - m_ref) may grow to 1e30 without loss).  Rows whose
// sum leaves the safe range are flagged and redone by the kernel that can move its reference
// (see the launcher).
//
// Staging: tile images in LDS (KS = 1: four of K and V; KS = 2: per key stream rings of five 32-key blocks of K and four of V), filled by
// loads that write LDS directly (global_load_lds, 16
// bytes per lane: lane L of an instruction fills piece base + L, so the image layout is chosen by
// the global address each lane is given).  KS = 1: wavefronts 0-3 bring the four K pages (16 tokens) of a tile,
// 4-7 the four V pages; KS = 2: the four wavefronts of a key stream bring half a page of K and of V each of every block of their own
// tiles.  A page is four instructions whose addresses are one scalar base + one per-lane constant + an
// immediate: no vector arithmetic per tile.  Image of a tile (16-byte pieces):
//   K piece (MFMA row m of 32-key block b, k-step kk, half hh):
//       ((b*2 + kk/4)*4 + m/8)*64 + ((kk%4)*2 + (hh ^ (m/8)%2))*8 + m%8
//     (an instruction = 8 token slots x 128 bytes: whole cache lines; with 64-byte runs per slot the
//     K loads cost three times what the V loads cost for the same bytes)
//   V piece (page pg, 32-dim group db, half hh, dim n):  1024 + (pg*4+db)*64 + hh*32 + n
// An MFMA operand read takes contiguous runs of 128 bytes that alternate between the two halves
// of the 256-byte bank sweep (K) or one contiguous KiB (V): no bank conflicts.  In iteration t the wavefronts
// read image t and (for S of the next tile's first block) image t+1.  KS = 1: they start the loads of image t+3
// and, before the iteration's barrier, wait for their loads of image t+2, one s_barrier per tile.  KS = 2: in half an iteration (one block) they
// start the loads of K five blocks and of V three blocks ahead, into the places the half before left, and at its end wait for what
// they started two halves ago; a barrier per half.  (Whole tiles, three images of K and two of V, had their loads half a tile ahead
// and waited for them: one request of 449 rows in a decoder layer 317 -> 306 us, 70B with 230 rows 592 -> 570.  With all its keys in the
// L2 a pair of tiles takes as long, 1.55 us on 120 workgroups, 1.2 of it the two wavefronts' MFMAs and exponentials.)
// Block padding: K padding never reaches a product (its S entries are masked by selection); V
// padding would, as 0 x garbage, so the wavefront that loaded a V page blanks the page's padding
// slots in LDS before the barrier, in a branch only a segment's last tile takes.
//
// What bounds it: long prompts, the two wavefronts' MFMAs and exponentials (32 x 32 clocks of matrix pipe and 32
// exponentials per wavefront and tile) at the clock the chip holds under them (1.75-1.85 GHz); short ones, the latency in
// front of and behind the loop.  Hence the
// prologue: the first pages and the query rows (whole rows each, regrouped in LDS) are on their way before the positions
// are known, a head computes a quarter of the angles and shares them, visible tiles are counted in the
// window; and the epilogue turns the output in LDS so that stores write whole rows.  Measured against a chain of
// dependent loads, each wavefront's own angles and 8-byte stores: one request of 2.6k tokens 65 -> 59 us (two
// streams: 44), the 8B batch of 32 1883 -> 1773, 4 x 32k tokens 3270 -> 3165 (1.2 PFLOP/s).
// Several requests: which workgroup takes which rows is in the plan's list (WorkList), because a grid of (row tiles) x (requests)
// starts the last request's long workgroups when nothing is left to run beside them: 70B on a quarter of the heads, 8
// requests of 10k tokens, cc_sparse_prefill and what is in front of it 514 -> 457 us; 6 requests of 3-6k tokens 318 -> 310.
// KS = 1: the rows of a sparse list lie far apart, so the first 32 see several tiles fewer than the second 32; their
// wavefronts stop multiplying there and only bring in their share of the tiles.
#include <algorithm>
#include <type_traits>

#include "mfma_tile.h"

namespace cc {

using namespace tile;

namespace {

typedef __attribute__((__vector_size__(4 * sizeof(uint32_t)))) uint32_t u32x4;

constexpr int kImage = 2048;    // 16-byte pieces per tile image (K: 1024, V: 1024)
constexpr int kBufs = 4;
// Two key streams up to this many 64-row workgroups.  A compute unit holds one workgroup; twice as many with half
// the tiles fill units that would idle and still run in one round, or nearly.  Up to 160 they are ahead whatever the
// batch; behind that it hangs on how unevenly its requests fill their last tiles, and what one or two requests would gain
// four lose.  cc_sparse_prefill, one stream / two, us: 40 workgroups 47 / 39 (4 requests of 1.2k, 8 / 2 heads), 64: 91 / 65 (1 of 3.6k, 64 / 8), 112: 50 / 44 (1 of 1.2k), 128: 54 / 46
// (4 of 1.2k), 96 / 72 (2 of 3.6k, 64 / 8), 136: 224 / 155 (1 of 10k), 160: 86 / 66 (1 of 3k), 54 / 54 (4 of 1.2k); 192: 225 / 167 (1 of 10k), 88 / 73
// (2 of 3k), 91 / 94 (4 of 3k), 224: 54 / 53 (2 of 1.2k), 54 / 61 (4 of 1.2k), 256: 95 / 109 (4 of 3k), 264: 237 / 207 (1 of 10k).
constexpr int kTwoStreamGrid = 160;
// KS = 2: blocks of 32 keys per stream: K in five places, V in four
constexpr int kHalf = 8192, kRingK = 5, kRingV = 4;
#ifndef CC_RING_DEPTH
#define CC_RING_DEPTH 8
#endif
constexpr int kDepth = CC_RING_DEPTH;       // operand reads in flight ahead of the MFMAs (even)
static_assert(kDepth % 2 == 0 && kDepth >= 4 && kDepth <= 8, "operand reads are issued in pairs");
// p = exp2(S - reference) may be large (fp32 and bf16 share the exponent range); a row sum
// beyond this leaves no headroom for O
constexpr float kSafeSum = 1.0e30f;

// MFMA forms with fixed register classes (the compiler's own choice shuffles accumulators between
// the two register files once a wavefront uses more than 256 registers): S accumulates in vector
// registers, where the vector ALU reads it; O accumulates in accumulation registers; the rotated
// query sits in accumulation registers as the B operand.  The matrix results are opaque to the
// compiler's hazard handling, so every vector-ALU read of them is either at least two MFMAs
// behind its producer (steady state) or behind mfma_result_wait().
__device__ __forceinline__ void mfma_s_zero(f32x16& d, const u32x4& a, const u32x4& b) {
  asm volatile("v_mfma_f32_32x32x16_bf16 %0, %1, %2, 0" : "=&v"(d) : "v"(a), "a"(b));
}
__device__ __forceinline__ void mfma_s_first(f32x16& d, const u32x4& a, const u32x4& b, const f32x16& c) {
  asm volatile("v_mfma_f32_32x32x16_bf16 %0, %1, %2, %3" : "=&v"(d) : "v"(a), "a"(b), "v"(c));
}
__device__ __forceinline__ void mfma_s_acc(f32x16& d, const u32x4& a, const u32x4& b) {
  asm volatile("v_mfma_f32_32x32x16_bf16 %0, %1, %2, %0" : "+v"(d) : "v"(a), "a"(b));
}
__device__ __forceinline__ void mfma_o_acc(f32x16& d, const u32x4& a, const u32x4& b) {
  asm volatile("v_mfma_f32_32x32x16_bf16 %0, %1, %2, %0" : "+a"(d) : "v"(a), "v"(b));
}
__device__ __forceinline__ void zero_acc(f32x16& d) {
#pragma unroll
  for (int i = 0; i < 16; ++i) asm volatile("v_accvgpr_write_b32 %0, 0" : "=a"(d[i]));
}
// 32 idle issue slots: longer than the 8 passes of the MFMA plus its write-back
__device__ __forceinline__ void mfma_result_wait() {
  asm volatile("s_nop 15\n\ts_nop 15" ::: "memory");
}
// Loads of 64 lanes x 16 bytes from global memory straight into LDS: lane L's 16 bytes land at
// M0 + immediate + 16 L, read from base + voff(L) + immediate (the immediate counts on both sides).
// Written as instructions the compiler does not model: it would otherwise drain every outstanding
// load before the next LDS read, because it cannot see that the image being filled is not the
// image being read.  Completion is counted by vmcnt.
template <int IMM>
__device__ __forceinline__ void dma_one(uint32_t voff, const char* base, uint32_t m0v) {
  asm volatile("s_mov_b32 m0, %2\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %0, %1 offset:%3"
               :: "v"(voff), "s"(base), "s"(m0v), "n"(IMM) : "memory", "m0");
}
template <int IMM0, int IMM1>
__device__ __forceinline__ void dma_two(uint32_t voff, const char* base, uint32_t m0v) {
  asm volatile("s_mov_b32 m0, %2\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %0, %1 offset:%3\n\t"
               "global_load_lds_dwordx4 %0, %1 offset:%4"
               :: "v"(voff), "s"(base), "s"(m0v), "n"(IMM0), "n"(IMM1) : "memory", "m0");
}
// The exponentials.  exp_only: t = exp2(s).  exp_behind_pack: first the pair that is still pending
// (e = its even element, v = its odd one) is packed to bf16 and both are added to the row sum, then
// e = exp2(s).  Written out so that each stays where it is placed, under one MFMA (the compiler
// otherwise lumps the exponentials of a block together or sinks them to their use).
__device__ __forceinline__ void exp_only(float& t, float s) {
  asm volatile("v_exp_f32 %0, %1" : "=v"(t) : "v"(s));
}
__device__ __forceinline__ void exp_behind_pack(uint32_t& pk, float& l, float& e, float v, float s) {
  asm volatile("v_cvt_pk_bf16_f32 %0, %2, %3\n\tv_add_f32 %1, %1, %2\n\tv_add_f32 %1, %1, %3\n\tv_exp_f32 %2, %4"
               : "=&v"(pk), "+v"(l), "+v"(e) : "v"(v), "v"(s));
}
// s_waitcnt with only the LDS counter set (vector-memory and export counters left alone)
template <int N>
__device__ __forceinline__ void wait_lds() {
  __builtin_amdgcn_s_waitcnt(15 | (3 << 14) | (7 << 4) | (N << 8));
}

// BY: with the by-product (see the tile loop).
template <int KS, bool BY>
__global__ __launch_bounds__(512, 1) void attn_v2_kernel(
    const bf16_t* __restrict__ q, const int32_t* __restrict__ q_pos,
    const bf16_t* __restrict__ k_pool, const bf16_t* __restrict__ v_pool,
    const TileDesc* __restrict__ tiles, int max_tiles, const WorkItem* __restrict__ items, const int32_t* __restrict__ order, int tile_bits,
    const int32_t* __restrict__ req_seg_off, int hq, int hkv, int n_sub, int n_tiles_x, InvFreq inv_freq, bf16_t* __restrict__ out, float* __restrict__ lse,
    int32_t* __restrict__ redo, int redo_any, const int32_t* __restrict__ q_map, int map_pos,
    const int32_t* __restrict__ snap_index, float* __restrict__ cum, int s_max,
    const bf16_t* __restrict__ v_shared, int n_shared_blocks, const int32_t* __restrict__ v_map) {
  constexpr int TQ = KS == 1 ? 64 : 32;     // query rows per workgroup
  // LDS: KS = 1: four images of K | V; KS = 2: per key stream a ring of five 32-key blocks of K and one of four of V, and what the streams
  // tell each other at a segment's end
  __shared__ uint4 lds_all[KS == 1 ? kBufs * kImage : 2 * (kRingK + kRingV) * (kHalf / 16) + 256];
  auto here = [&]() __attribute__((always_inline)) { int t = threadIdx.x; asm volatile("" : "+v"(t)); return t & 63; };
  const int tid = threadIdx.x, lane = tid & 63, wave = uniform(tid >> 6);
  const int n = lane & 31, hh = lane >> 5;
  const int whead = wave & 3, wgrp = wave >> 2;              // this wavefront's head of the four; row half or key stream
  const int ks = KS == 1 ? 0 : wgrp, wrows = KS == 1 ? 32 * wgrp : 0;
  const int per_tile = hkv * n_sub;
  const int rem = blockIdx.x % per_tile;
  const int kvh = rem % hkv, hsub = rem / hkv;
  const int h = kvh * (4 * n_sub) + hsub * 4 + whead;

  // ---- which queries ------------------------------------------------------------------------
  // (from the plan's list of workgroups, or where there is none from a grid of row tiles, long ones first, by requests
  // in the order of their length; tile_bits: of a list entry, 0: no list)
  int req, tile;
  if (tile_bits != 0) {
    const int at = blockIdx.x / per_tile, e = tiles[at].work;
    if (at >= uniform(tiles[max_tiles - 1].work)) return;
    req = uniform(static_cast<int>(static_cast<uint32_t>(e) >> tile_bits));
    tile = uniform(e & ((1u << tile_bits) - 1));
  } else {
    req = gridDim.y == 1 ? 0 : uniform(order[blockIdx.y]);      // (one load less on the way to the first tile)
    tile = n_tiles_x - 1 - blockIdx.x / per_tile;
  }
  const WorkItem item = items[req];
  const int q_first = uniform(item.row), q_end = q_first + uniform(item.n_rows);
  const int j_begin = uniform(item.j_begin), j_end = min(uniform(item.j_end), max_tiles);
  const int q0 = q_first + tile * TQ;
  if (q0 >= q_end) return;
  const int n_all = j_end - j_begin;
  if (n_all <= 0) return;
  const char* lds_bytes = reinterpret_cast<const char*>(lds_all);
  // ---- rows and positions: asked for first, whole rows each (see load_query_rows) ---------------------
  // (with a row map, list row j takes its query from row q_map[j] of q - and, if map_pos, its
  // position from q_pos[q_map[j]]; results are always indexed by the list row)
  int src_row, p, p_other = 0, snap_row = -1;      // (snap_row: the by-product's row, see there; -1: none)
  {
    const int row = min(q0 + wrows + n, q_end - 1);
    if (BY && q0 + wrows + n < q_end) snap_row = snap_index != nullptr ? snap_index[row] : row;      // (no index: every row is a snap row)
    src_row = q_map != nullptr ? q_map[row] : row;
    p = q_pos[map_pos ? src_row : row];
    if (KS == 1) {
      const int other = min(q0 + (32 - wrows) + n, q_end - 1);
      p_other = q_pos[map_pos ? (q_map != nullptr ? q_map[other] : other) : other];
    }
  }
  uint4 rows[8];

  // ---- descriptors and staging --------------------------------------------------------------------
  // What the loop needs of 64 consecutive tiles sits in vector registers, one tile per lane, and is
  // handed out with v_readlane: no memory access per tile.  The straight path reads the flags of tile t+2 and where this wavefront's pages of the tiles
  // ahead are (KS = 1: of tile t+3; KS = 2: keys of t+2 and t+3, values of t+1 and t+2, a block each); positions, key
  // counts and segments are read only inside the branches that need them.
  //   flag 1: the tile needs masking for some row (padding, or its last key lies behind p_min)
  //   flag 2: the tile has padding slots or missing pages
  //   flag 4: the next tile belongs to another segment
  int win_base = 0;
  // w_own: block of the page this wavefront brings in (-1: none); w_vown: where that page's values
  // are - the same block of v_pool, or (<= -2) block -2 - w_vown of v_shared while the value map
  // still points there (copy-on-write pending)
  // (KS = 2: a wavefront brings half a page of every 32-key block: w_own and w_vown for a tile's first block, w_own1 and w_vown1 for its second)
  int w_kpos0, w_nvalid, w_seg, w_seg_next, w_own, w_vown, w_own1 = 0, w_vown1 = 0, w_flags, w_pair = 0, w_seg_far = 0;
  auto fill_window = [&](int base) __attribute__((always_inline)) {
    const int jl = min(KS * (base + lane) + ks, n_all - 1);
    const TileDesc v = fetch_desc(tiles, j_begin + jl, max_tiles);
    const int b0 = v.blk[0], b1 = v.blk[1], b2 = v.blk[2], b3 = v.blk[3];
    w_kpos0 = v.kpos0; w_nvalid = v.nvalid; w_seg = v.seg;
    int jn = min(max(j_begin + min(jl + 1, n_all - 1), 0), max_tiles - 1);
    asm volatile("" : "+v"(jn));                   // (a vector load, like the descriptor itself: see fetch_desc)
    w_seg_next = tiles[jn].seg;
    if constexpr (KS == 2) {       // both streams' tiles (their loops and segment ends agree)
      int je = min(j_begin + min(2 * (base + lane), n_all - 1), max_tiles - 1);
      int jo = min(j_begin + min(2 * (base + lane) + 1, n_all - 1), max_tiles - 1);
      asm volatile("" : "+v"(je), "+v"(jo));
      w_pair = tiles[ks == 0 ? jo : je].kpos0;      // first key of the other stream's tile
      if constexpr (BY) {
        int jf = min(j_begin + min(2 * (base + lane) + 2, n_all - 1), max_tiles - 1);
        asm volatile("" : "+v"(jf));
        w_seg = tiles[je].seg; w_seg_next = tiles[jo].seg; w_seg_far = tiles[jf].seg;
      }
    }
    auto values_of = [&](int own) __attribute__((always_inline)) {
      int at = own;
      if (v_map != nullptr && own >= 0) {
        const int m = v_map[own];
        if (m >= 0 && m < n_shared_blocks) at = -2 - m;
      }
      return at;
    };
    if constexpr (KS == 1) {
      w_own = whead == 0 ? b0 : whead == 1 ? b1 : whead == 2 ? b2 : b3;
    } else {
      w_own = whead < 2 ? b0 : b1;
      w_own1 = whead < 2 ? b2 : b3;
      w_vown1 = values_of(w_own1);
    }
    w_vown = values_of(w_own);
    const bool edge = v.nvalid < kTile || (b0 | b1 | b2 | b3) < 0;
    w_flags = (edge ? 3 : 0) | (w_seg_next != w_seg ? 4 : 0) | (KS == 2 && BY && w_seg_far != w_seg_next ? 8 : 0);
  };
  fill_window(0);
  load_query_rows(rows, q, src_row, hq, h, lane);
  // KS = 1: byte offset of the image of tile t, K in front of V.  KS = 2: offset of the 32-key block b of K or V
  auto image = [&](int t) __attribute__((always_inline)) { return (t & (kBufs - 1)) * (kImage * 16); };
  auto k_block = [&](int b) __attribute__((always_inline)) { return ks * (kRingK + kRingV) * kHalf + (b % kRingK) * kHalf; };
  auto v_block = [&](int b) __attribute__((always_inline)) { return (ks * (kRingK + kRingV) + kRingK) * kHalf + (b % kRingV) * kHalf; };
  constexpr int kVPart = KS == 1 ? 16384 : 0;
  // Loads straight into LDS.  KS = 1: wavefront w brings page w % 4 of a tile, K (w < 4) or V.  KS = 2: of a 32-key block of K and of V
  // wavefront w brings half of page w / 2 % 2: eight rows of K, 64 dims of V.
  //   K: instruction (rg, kq) brings rows 8 rg .. 8 rg + 7 of the page (row r sits in token slot
  //      swap23(r)), 128 bytes each at dim 64 kq: lane L reads row 8 rg + L % 8, piece (L / 8) ^ rg
  //   V: lane (hh, n) reads slots 8hh.. of dim row 32 j + n
  const size_t blk_bytes = static_cast<size_t>(hkv) * (kBlock * kD) * sizeof(bf16_t);
  const char* k_head = reinterpret_cast<const char*>(k_pool) + static_cast<size_t>(kvh) * (kBlock * kD * sizeof(bf16_t));
  const char* v_head = reinterpret_cast<const char*>(v_pool) + static_cast<size_t>(kvh) * (kBlock * kD * sizeof(bf16_t));
  const char* v_head_shared = v_shared == nullptr ? v_head
      : reinterpret_cast<const char*>(v_shared) + static_cast<size_t>(kvh) * (kBlock * kD * sizeof(bf16_t));
  const uint32_t k_voff0 = swap23(lane & 7) * (kD * 2) + (lane >> 3) * 16;
  const uint32_t k_voff1 = swap23(8 + (lane & 7)) * (kD * 2) + ((lane >> 3) ^ 1) * 16;
  const uint32_t v_voff = n * 32 + hh * 16;
  typedef __attribute__((address_space(3))) const uint4 lds_piece;
  const uint32_t lds_base = uniform(static_cast<uint32_t>(reinterpret_cast<uintptr_t>((lds_piece*)lds_all)));   // LDS byte address
  const int page = KS == 1 ? whead : whead >> 1, part = whead & 1;              // (KS = 2: page of a 32-key block and half of it)
  const bool brings_k = wave < 4;                                              // (KS = 1)
  const uint32_t k_img = lds_base + (KS == 1 ? ((page >> 1) * 8 + (page & 1) * 2) * 1024 : (2 * page + part) * 1024);   // this wavefront's first K group in image 0
  const uint32_t v_img = lds_base + kVPart + 4 * page * 1024 + (KS == 1 ? 0 : 2048 * part);                   // ... and its V page
  const char* k_src = nullptr;                                                // page of the tile being loaded (scalar)
  const char* v_src = nullptr;
  uint32_t k_dst = 0, v_dst = 0;
  auto k_from = [&](int own, int to) __attribute__((always_inline)) {
    k_src = k_head + static_cast<size_t>(max(own, 0)) * blk_bytes;
    k_dst = k_img + to;
  };
  auto v_from = [&](int vown, int to) __attribute__((always_inline)) {
    v_src = vown <= -2 ? v_head_shared + static_cast<size_t>(-2 - vown) * blk_bytes
                       : v_head + static_cast<size_t>(max(vown, 0)) * blk_bytes;
    if (KS == 2) v_src += 2048 * part;
    v_dst = v_img + to;
  };
  // KS = 1: the tile in lane l of the window, into image offset `to`
  auto dma_begin = [&](int l, int to) __attribute__((always_inline)) {
    k_from(__builtin_amdgcn_readlane(w_own, l), to);
    v_from(__builtin_amdgcn_readlane(w_vown, l), to);
  };
  // (the two halves of a row are 4 KiB apart in the image and 128 bytes apart in memory; the two
  // row groups of a page are neighbours in the image)
  auto dma_k = [&](int j) __attribute__((always_inline)) {
    if (KS == 1 && !brings_k) return;
    const uint32_t voff = KS == 2 ? (part ? k_voff1 : k_voff0) : j < 2 ? k_voff0 : k_voff1;
    if (j == 0) dma_one<0>(voff, k_src, k_dst);
    else if (j == 1) dma_one<128>(voff, k_src, k_dst + (4096 - 128));
    else if (j == 2) dma_one<0>(voff, k_src, k_dst + 1024);
    else dma_one<128>(voff, k_src, k_dst + 1024 + (4096 - 128));
  };
  auto dma_v = [&](int half) __attribute__((always_inline)) {
    if (KS == 1 && brings_k) return;
    if (half == 0) dma_two<0, 1024>(v_voff, v_src, v_dst);
    else dma_two<2048, 3072>(v_voff, v_src, v_dst);
  };
  // blank the padding slots of the V page this wavefront loaded (rare; after its loads have landed).  l: the tile's lane of the window; KS = 2: second:
  // its second 32-key block
  auto blank_padding = [&](int l, int img, bool second) __attribute__((always_inline)) {
    const int nvalid = __builtin_amdgcn_readlane(w_nvalid, l), own = __builtin_amdgcn_readlane(KS == 2 && second ? w_own1 : w_own, l);
    const int nv = own < 0 ? 0 : min(max(nvalid - kBlock * (page + (KS == 2 && second ? 2 : 0)), 0), kBlock);
    if ((KS == 2 || !brings_k) && nv < kBlock) {
      const int ln = here();
      uint4* vp = reinterpret_cast<uint4*>(const_cast<char*>(lds_bytes) + img + kVPart + 4 * page * 1024 + (KS == 2 ? 2048 * part : 0) + ln * 16);
#pragma unroll
      for (int j = 0; j < 4 / KS; ++j) vp[j * 64] = zero_pad_slots(vp[j * 64], ln >> 5, nv);
      // (a rare branch leaves nothing pending, so that the code behind the join waits for no more
      // than the straight path does)
      wait_lds<0>();
    }
  };
  // wait until at most `newer` of this wavefront's vector-memory operations are outstanding
  auto wait_loads = [&](auto newer) __attribute__((always_inline)) {
    constexpr int kN = decltype(newer)::value;
    __builtin_amdgcn_s_waitcnt((kN & 15) | ((kN >> 4) << 14) | (7 << 4) | (15 << 8));
    asm volatile("" ::: "memory");
  };
  auto barrier = [&]() __attribute__((always_inline)) {
    asm volatile("" ::: "memory");
    __builtin_amdgcn_s_barrier();
    asm volatile("" ::: "memory");
  };

  // ---- first tiles: on their way before anything about the rows is known ------------------------------
  // (KS = 1: images 0, 1, image 2 when the queries are turned; KS = 2: K blocks 0, 1, 2 and V block 0, the next two of each when the queries are
  // turned.  Tiles no row sees are loaded in vain; past the request's last tile that tile is repeated.)
  const int n_av = (n_all - ks + KS - 1) / KS;                // tiles of the stream in the whole request
  auto first_lane = [&](int t) __attribute__((always_inline)) { return max(min(t, n_av - 1), 0); };
  auto first_tile = [&](int t) __attribute__((always_inline)) {         // KS = 1
    dma_begin(first_lane(t), image(t));
#pragma unroll
    for (int j = 0; j < 4; ++j) dma_k(j);
    dma_v(0);
    dma_v(1);
  };
  auto first_k = [&](int b, int l) __attribute__((always_inline)) {     // KS = 2: block b, of the tile in lane l of the window
    k_from(__builtin_amdgcn_readlane(b & 1 ? w_own1 : w_own, l), k_block(b));
    dma_k(0);
    dma_k(1);
  };
  auto first_v = [&](int b, int l) __attribute__((always_inline)) {
    v_from(__builtin_amdgcn_readlane(b & 1 ? w_vown1 : w_vown, l), v_block(b));
    dma_v(0);
  };
  if constexpr (KS == 1) {
    first_tile(0);
    first_tile(1);
  } else {
    first_k(0, first_lane(0));
    first_v(0, first_lane(0));
    first_k(1, first_lane(0));
    first_k(2, first_lane(1));
  }

  // first and last position over all rows of the workgroup (every wavefront walks the same tiles)
  const int p_mine = uniform(wave_max_i(p));
  const int p_max = KS == 1 ? max(p_mine, uniform(wave_max_i(p_other))) : p_mine;
  const int p_min = uniform(wave_min_i(KS == 1 ? min(p, p_other) : p));

  // ---- tiles of the request whose first key some query of the workgroup sees ------------------
  // (tiles are listed in prompt order, so these form a prefix)
  // (counted in the window; while all 64 are visible, those behind it are taken to be, until the window moves there)
  int n_odd = 0;                 // (tiles of the odd stream)
  // iterations of the workgroup; tiles of this wavefront's key stream (the odd one may have none); tiles it multiplies
  // (KS = 1: those its own 32 rows see)
  int n_it, n_loc, n_mine;
  auto see_window = [&]() __attribute__((always_inline)) {
    if (w_kpos0 + kTile - 1 > p_min) w_flags |= 1;
    const int jl = KS * (win_base + here()) + ks;
    const uint64_t seen = __ballot(jl < n_all && w_kpos0 <= p_max);
    n_loc = seen == ~0ull ? n_av : win_base + __popcll(seen);
    if constexpr (KS == 1) {
      n_loc = n_it = max(n_loc, 1);
      const uint64_t own = __ballot(jl < n_all && w_kpos0 <= p_mine);
      n_mine = own == ~0ull ? n_av : max(win_base + __popcll(own), 1);
    } else {
      const uint64_t pair = __ballot((jl ^ 1) < n_all && w_pair <= p_max);
      const int n_other = pair == ~0ull ? (n_all - (ks ^ 1) + 1) / 2 : win_base + __popcll(pair);
      n_it = max(max(n_loc, n_other), 1);
      if (BY) n_odd = min(n_loc, n_other);
      n_mine = n_it;
    }
  };
  see_window();
  auto lane_of = [&](int t) __attribute__((always_inline)) { return (KS == 1 ? min(t, n_loc - 1) : max(min(t, n_loc - 1), 0)) - win_base; };
  // ---- load the query rows, rotate them to their positions, fold the softmax scale -------------
  // lane (n, hh) keeps, for k-step kk, dims 16kk + 8hh .. +7; dims < 64 pair with dims + 64.
  const float c2 = 0.08838834764831845f * kLog2e;            // log2(e) / sqrt(128)
  u32x4 qreg[8];
  // The four heads share the angles (KS = 2: so do the two streams): a wavefront computes a quarter (an eighth) of them.
  auto load_queries = [&]() __attribute__((always_inline)) {
    char* lds_w = const_cast<char*>(lds_bytes);
    // scratch: KS = 1: images 2 and 3; KS = 2: the places of the streams' K block 4 and V blocks 1 to 3, for the angles those of K block 3 of both
    regroup_query_rows(rows, lds_w + (KS == 1 ? 2 * (kImage * 16) + wave * 8192 : whead == 0 ? k_block(4) : v_block(whead)), lane);
    barrier();
    char* turns_at = lds_w + (KS == 1 ? 2 * (kImage * 16) + wgrp * 16384 : 3 * kHalf) + lane * 16;
    auto turn_at = [&](int c) __attribute__((always_inline)) {
      return reinterpret_cast<float4*>(turns_at + c * 1024 + (KS == 2 && c >= 8 ? (kRingK + kRingV - 1) * kHalf : 0));
    };
#pragma unroll
    for (int i = 0; i < 4 / KS; ++i) {             // (float4 number c: rotation pairs 16 (c / 4) + 8 hh + 2 (c % 4), + 1)
      const int c = KS == 1 ? 4 * whead + i : 2 * wave + i;
      *turn_at(c) = query_turn(inv_freq, p, 16 * (c >> 2) + 2 * (c & 3), hh, c2);
    }
    wait_lds<0>();
    barrier();
#pragma unroll
    for (int kk = 0; kk < 4; ++kk) {
      u32x4 xv = __builtin_bit_cast(u32x4, rows[kk]), yv = __builtin_bit_cast(u32x4, rows[kk + 4]);
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        uint32_t x = xv[i], y = yv[i];
        turn_words(x, y, *turn_at(kk * 4 + i));
        xv[i] = x;
        yv[i] = y;
      }
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        asm volatile("v_accvgpr_write_b32 %0, %1" : "=a"(qreg[kk][i]) : "v"(xv[i]));
        asm volatile("v_accvgpr_write_b32 %0, %1" : "=a"(qreg[kk + 4][i]) : "v"(yv[i]));
      }
      __builtin_amdgcn_sched_barrier(0);
    }
  };

  // byte offsets of this lane's operand pieces inside an image (see the layout above)
  const int k_rd = (n >> 3) * 1024 + (hh ^ ((n >> 3) & 1)) * 128 + (n & 7) * 16;
  const int v_rd = kVPart + lane * 16;
  float m_ref, lsum, ev, vodd;
  f32x16 cinit;                   // -m_ref in all 16 registers: the C operand that opens an S block
  f32x16 o[4];                    // running output, accumulation registers for the whole loop
  f32x16 sacc[2];                 // S of the two 32-key blocks in flight (vector registers)
  uint32_t pk[2][2][4];           // P^T of [block parity][16-key half], packed bf16 pairs
  {
    m_ref = 0.f; lsum = 0.f; ev = 0.f; vodd = 0.f;
#pragma unroll
    for (int db = 0; db < 4; ++db) zero_acc(o[db]);
  }

  // ---- operand ring ---------------------------------------------------------------------------
  // Steps of one iteration (tile t):
  //    0.. 7  K pieces of the tile's second block      (S of that block)
  //    8..15  V pieces of the first block              (PV of the first block)
  //   16..23  K pieces of the next tile's first block  (S of that block)
  //   24..31  V pieces of the second block             (PV of the second block)
  //   32..39  = steps 0..7 of the next iteration
  // (behind the last tile the "next tile" is stale keys: that S block is masked as a whole)
  // Reads are issued two at a time behind every odd step (into the slots of the two pieces just
  // used), and one wait in front of every even step covers that step and the next.
  u32x4 ring[kDepth];
  struct Blocks { int k1, v0, k0_next, v1, k1_next; };      // where these blocks are
  auto k_piece = [&](int at, int kk) __attribute__((always_inline)) {
    return *reinterpret_cast<const u32x4*>(lds_bytes + at + k_rd + (kk >> 2) * 4096 + (kk & 3) * 256);
  };
  auto v_piece = [&](int at, int j) __attribute__((always_inline)) {      // j = page of the block * 4 + dim group
    return *reinterpret_cast<const u32x4*>(lds_bytes + at + v_rd + j * 1024);
  };
  auto issue = [&](const Blocks& at, int s) __attribute__((always_inline)) {   // s: compile-time
    if (s < 8) ring[s % kDepth] = k_piece(at.k1, s);
    else if (s < 16) ring[s % kDepth] = v_piece(at.v0, s - 8);
    else if (s < 24) ring[s % kDepth] = k_piece(at.k0_next, s - 16);
    else if (s < 32) ring[s % kDepth] = v_piece(at.v1, s - 24);
    else ring[s % kDepth] = k_piece(at.k1_next, s - 32);
  };

  // one exponential: element i (0..15) of block parity bp.  An even element first packs the pair
  // in front of it (element 0: the last pair of the block before, which has the other parity).
  auto exp_step = [&](int bp, int i) __attribute__((always_inline)) {
    const float s = sacc[bp][i];
    if (i & 1) exp_only(vodd, s);
    else if (i == 0) exp_behind_pack(pk[bp ^ 1][1][3], lsum, ev, vodd, s);
    else exp_behind_pack(pk[bp][(i - 2) >> 3][((i - 2) & 7) >> 1], lsum, ev, vodd, s);
  };
  // S block into parity bp from the ring; side(kk) runs after each MFMA
  auto s_slot = [&](const Blocks& at, int s0, int bp, auto&& side) __attribute__((always_inline)) {
#pragma unroll
    for (int kk = 0; kk < 8; ++kk) {
      if ((kk & 1) == 0) wait_lds<kDepth - 2>();
      {
        if (kk == 0) mfma_s_first(sacc[bp], ring[(s0 + kk) % kDepth], qreg[kk], cinit);
        else mfma_s_acc(sacc[bp], ring[(s0 + kk) % kDepth], qreg[kk]);
        if ((kk & 1)) {
          issue(at, s0 + kk - 1 + kDepth);
          issue(at, s0 + kk + kDepth);
        }
        side(kk);
        __builtin_amdgcn_sched_barrier(0);
      }
    }
  };
  // PV of block parity bp: step st = (u, db): 16-key half u (page), 32-dim group db
  auto pv_slot = [&](const Blocks& at, int s0, int bp, auto&& side) __attribute__((always_inline)) {
#pragma unroll
    for (int st = 0; st < 8; ++st) {
      const int u = st >> 2, db = st & 3;
      if ((st & 1) == 0) wait_lds<kDepth - 2>();
      {
        const u32x4 pw = {pk[bp][u][0], pk[bp][u][1], pk[bp][u][2], pk[bp][u][3]};
        mfma_o_acc(o[db], ring[(s0 + st) % kDepth], pw);
        if ((st & 1)) {
          issue(at, s0 + st - 1 + kDepth);
          issue(at, s0 + st + kDepth);
        }
        side(st);
        __builtin_amdgcn_sched_barrier(0);
      }
    }
  };

  // padding / causal edge: entries of block parity bp (tile block blk) the query must not see
  // become -inf (register i of block blk holds key 32 blk + 16(i/8) + 8hh + i%8 of the tile)
  auto mask_block = [&](int bp, int blk, int kpos0, int nvalid) __attribute__((always_inline)) {
    mfma_result_wait();
    {
      int lim = min(nvalid - 1, p - kpos0) - 8 * hh - 32 * blk;
      asm volatile("" : "+v"(lim));
#pragma unroll
      for (int i = 0; i < 16; ++i)
        sacc[bp][i] = (16 * (i / 8) + (i % 8) <= lim) ? sacc[bp][i] : -INFINITY;
      asm volatile("" : "+v"(sacc[bp]));
    }
  };

  auto mask_tile = [&](int bp, int blk, int t) __attribute__((always_inline)) {      // (a tile the stream does not have: all of it)
    const int l = lane_of(t);
    mask_block(bp, blk, __builtin_amdgcn_readlane(w_kpos0, l), t >= n_loc ? 0 : __builtin_amdgcn_readlane(w_nvalid, l));
  };

  // prologue: S of block 0 and the first half of its exponentials
  load_queries();
  wait_loads(std::integral_constant<int, 0>{});
#pragma unroll
  for (int t = 0; t < (KS == 1 ? 2 : 1); ++t) {
    const int l = first_lane(t);
    if (__builtin_amdgcn_readlane(w_flags, l) & 2) blank_padding(l, KS == 1 ? image(t) : v_block(0), false);
  }
  __syncthreads();
  if constexpr (KS == 1) {
    first_tile(2);
  } else {
    first_k(3, lane_of(1));
    first_v(1, lane_of(0));
    first_k(4, lane_of(2));
    first_v(2, lane_of(1));        // (values that are multiplied are those whose padding is blanked: of the last tile that is seen, not of one behind it)
  }
  int f_cur = __builtin_amdgcn_readlane(w_flags, lane_of(0));      // flags of tile t, t+1 (carried from tile to tile)
  int f_next = __builtin_amdgcn_readlane(w_flags, lane_of(1));
  {
    const Blocks at{KS == 1 ? image(0) + kHalf : k_block(1), 0, 0, 0, 0};
#pragma unroll
    for (int kk = 0; kk < 8; ++kk) {
      const u32x4 a = k_piece(KS == 1 ? image(0) : k_block(0), kk);
      {
        if (kk == 0) mfma_s_zero(sacc[0], a, qreg[kk]);
        else mfma_s_acc(sacc[0], a, qreg[kk]);
      }
    }
    if ((f_cur & 1) || (KS == 2 && n_loc == 0)) mask_tile(0, 0, 0);
    else mfma_result_wait();
    // the maximum of the stream's first block is the reference for the whole row.  KS = 1: it holds key 0 of the
    // request, which every query sees, so it is finite; KS = 2: a query may see no key of the odd stream at all
    // (then it sees none of its later tiles either, and its sum stays 0)
    {
      const float t = max16(sacc[0]);
      m_ref = fmaxf(t, __shfl_xor(t, 32, 64));
      if (KS == 2 && m_ref == -INFINITY) m_ref = 0.f;
#pragma unroll
      for (int i = 0; i < 16; ++i) {
        sacc[0][i] -= m_ref;
        cinit[i] = -m_ref;
      }
    }
    exp_only(ev, sacc[0][0]);
#pragma unroll
    for (int i = 1; i < 8; ++i)
exp_step(0, i);
#pragma unroll
    for (int s = 0; s < kDepth; ++s) issue(at, s);     // steps 0..kDepth-1 of iteration 0
    __builtin_amdgcn_sched_barrier(0);
    // (KS = 2: the first half-step brings K block 5 into block 0's place, which every wavefront of the stream has read by here)
    if constexpr (KS == 2) barrier();
  }

  // ---- the tile loop --------------------------------------------------------------------------------
  // on entry: parity 0 holds S of the tile's first block (masked) with the first half of its
  // exponentials done.  Every tile runs through the same straight-line body (the masking branches
  // apart): behind the last tile the "next tile" is a phantom whose S block is masked as a whole, so
  // that its exponentials are zeros.  (A peeled copy of the body for the last tile would save those
  // 16 MFMAs per workgroup; but the register allocator then settles the accumulators differently in
  // the two copies and moves them around between MFMAs it cannot see into, without the wait states
  // such moves need in front of a matrix instruction.)
  // By-product for rows that ask for it (snap_index >= 0: the question rows; or every row): when the tile that
  // has just been closed is the last one of its segment, the log-sum-exp over all keys up to here
  // goes to cum[snap row][head][segment's index in its request].  A stream's reference never moves in this
  // kernel, so with one stream these running sums subtract exactly; two streams' sums meet under the larger of
  // their references, which rounds each once.  (Rare: once per segment of the request.)
  const int seg_first = BY ? req_seg_off[req] : 0;
  // (segments without tokens have no tile: the value also stands for those between this tile's
  // segment and the next tile's; the row sum is taken with the pair that is still to be packed)
  // KS = 2: the even stream writes what a segment that ends with its tile leaves, the odd one likewise; each needs the
  // other's sum up to there, through LDS (rare as this is, it pays two
  // barriers).  prev: the odd stream's sum one tile ago.
  // (No load here: the compiler would wait for it and so for all loads of the tiles ahead, some of them just started.  The layer with the question's masses, 16 / 2
  // heads, 4 requests of 29 chunks of 66 tokens, one or two tiles each, 145 -> 140 us; 32 / 8, 1 of 5 x 512 85.2 -> 84.0.)
  float prev = 0.f;
  auto running = [&]() __attribute__((always_inline)) {
    const float mine = lsum + (ev + vodd);
    return mine + __shfl_xor(mine, 32, 64);
  };
  auto snapshot = [&](int t, float tot, int ends) __attribute__((always_inline)) {
    const int l = lane_of(t), pair = KS == 1 ? 0 : t - win_base;
    int seg = __builtin_amdgcn_readlane(w_seg, KS == 1 ? l : pair), seg_next = __builtin_amdgcn_readlane(w_seg_next, KS == 1 ? l : pair);
    const int ln = here();
    float m_all = m_ref;
    bool writes = true;
    if constexpr (KS == 2) {
      float4* meet = reinterpret_cast<float4*>(lds_all) + 2 * (kRingK + kRingV) * (kHalf / 16) + whead * 32 + (ln & 31);
      barrier();
      if (ln < 32) meet[ks * 128] = make_float4(m_ref, tot, prev, 0.f);
      wait_lds<0>();
      barrier();
      const float4 theirs = meet[(ks ^ 1) * 128];
      const float l_other = ks == 0 ? theirs.z : theirs.y;
      m_all = tot == 0.f ? theirs.x : l_other == 0.f ? m_ref : fmaxf(m_ref, theirs.x);
      tot = (tot == 0.f ? 0.f : tot * __builtin_amdgcn_exp2f(m_ref - m_all)) + (l_other == 0.f ? 0.f : l_other * __builtin_amdgcn_exp2f(theirs.x - m_all));
      if (ks == 1) { seg = seg_next; seg_next = __builtin_amdgcn_readlane(w_seg_far, pair); }
      writes = ks == 0 ? (ends & 4) != 0 : (ends & 8) != 0 && t < n_odd;
    }
    if (writes && ln < 32 && snap_row >= 0) {
      const float v = kLn2 * (m_all + __builtin_amdgcn_logf(tot));
      for (int sl = max(seg - seg_first, 0); sl < min(seg_next - seg_first, s_max); ++sl)
        cum[(static_cast<size_t>(snap_row) * hq + h) * s_max + sl] = v;
    }
    wait_lds<0>();                                 // (see blank_padding)
  };
  int f_far = 0;                                   // flags of tile t+2
  // next 64 descriptors, starting at tile t (rare)
  auto move_window = [&](int t) __attribute__((always_inline)) {
    if (min(t + 3, n_it - 1) - win_base >= 64) {
      win_base = t;
      fill_window(t);
      see_window();
      __builtin_amdgcn_s_waitcnt((7 << 4) | (15 << 8));      // vmcnt(0) here, so the hot path never waits for it
    }
  };
  // KS = 1: what the next iteration reads must be whole, image t+2 (loads started one iteration ago)
  auto end_tile = [&](int t) __attribute__((always_inline)) {
    wait_loads(std::integral_constant<int, 4>{});
    if (f_far & 2) blank_padding(lane_of(t + 2), image(t + 2), false);
    barrier();
    f_cur = f_next; f_next = f_far;
  };
  // KS = 2: half-step s (S(s + 1), PV(s)) reads V block s and K block s + 2, which must be whole; K block s + 5 and V block s + 3 are
  // started in it, into the places of K block s and V block s - 1, whose last operands left LDS in front of the barrier that opens it.  Of
  // the loads of the last two half-steps all eight may be out.
  auto end_half = [&](int t, bool pads, int b) __attribute__((always_inline)) {
    wait_loads(std::integral_constant<int, 8>{});
    if (pads) blank_padding(lane_of(t), v_block(b), b & 1);
    barrier();
  };
  int k_at = 2 * kHalf;          // KS = 2: place of K block 2 t + 2 in its ring
  auto k_place = [&](int blocks) __attribute__((always_inline)) {         // ... of the block so many behind it
    const int to = k_at + blocks * kHalf;
    return to >= kRingK * kHalf ? to - kRingK * kHalf : to;
  };
  int t = 0;
  // (Where the loop lies in the lines of the instruction cache shows: 70B on 8 requests of 10k tokens 1527 us with what is
  // behind this 0, 28 or 32 bytes behind a line of 64, 1550 with 16 or 20; with the by-product the layer of the 8B batch of 32 and a cache build are 0.4 - 0.9 %
  // slower 44 bytes behind a line than at its beginning, in five runs of five.  There 8 bytes of moves lie between this and the loop (an
  // alignment asked of the compiler for the loop itself has no effect); a test looks where the two loops begin.)
  if constexpr (KS == 1 && !BY) asm volatile(".p2align 6");
  if constexpr (KS == 1 && BY) asm volatile(".p2align 6\n\t.fill 14, 4, 0xbf800000");      // (14 s_nop)
  for (; t < n_mine; ++t) {
    Blocks at;
    if constexpr (KS == 1) at = Blocks{0, image(t), image(t + 1), image(t) + kHalf, image(t + 1) + kHalf};
    else at = Blocks{0, v_block(2 * t), k_block(0) + k_at, v_block(2 * t + 1), k_block(0) + k_place(1)};
    move_window(t);
    // slot 1: S of the tile's second block; second half of the first block's exponentials.
    // Underneath: the loads of the tiles ahead (past the last tile they repeat the last tile into an
    // image nobody reads), one instruction group per k-step.
    s_slot(at, 0, 1, [&](int kk) __attribute__((always_inline)) {
      exp_step(0, 8 + kk);
      if (kk == 0) {
        f_far = __builtin_amdgcn_readlane(w_flags, lane_of(t + 2));
        if constexpr (KS == 1) {
          dma_begin(lane_of(t + 3), image(t + 3));
        } else {
          k_from(__builtin_amdgcn_readlane(w_own1, lane_of(t + 2)), k_block(0) + k_place(3));
          v_from(__builtin_amdgcn_readlane(w_vown1, lane_of(t + 1)), v_block(2 * t + 3));
        }
      }
      if (kk >= 1 && kk <= 4 / KS) dma_k(kk - 1);
      if (kk == (KS == 1 ? 5 : 3)) dma_v(0);
      if (KS == 1 && kk == 6) dma_v(1);
    });
    if ((f_cur & 1) || (KS == 2 && t >= n_loc)) mask_tile(1, 1, t);
    // slot 2: PV of the first block; first half of the second block's exponentials
    pv_slot(at, 8, 0, [&](int st) __attribute__((always_inline)) { exp_step(1, st); });
    if constexpr (KS == 2) end_half(t, f_cur & 2, 2 * t + 1);
    // slot 3: S of the next tile's first block; second half of the second block's exponentials
    s_slot(at, 16, 0, [&](int kk) __attribute__((always_inline)) {
      exp_step(1, 8 + kk);
      if constexpr (KS == 2) {
        if (kk == 0) {
          k_from(__builtin_amdgcn_readlane(w_own, lane_of(t + 3)), k_block(0) + k_place(4));
          v_from(__builtin_amdgcn_readlane(w_vown, lane_of(t + 2)), v_block(2 * t));
        }
        if (kk == 1 || kk == 2) dma_k(kk - 1);
        if (kk == 3) dma_v(0);
      }
    });
    if constexpr (BY && KS == 1) {
      if (f_cur & 4) snapshot(t, running(), 0);       // tile t was the last of its segment
    } else if constexpr (BY) {                     // (both streams decide alike: one of the two tiles was)
      const int ends = __builtin_amdgcn_readlane(w_flags, t - win_base);
      const float tot = running();
      if ((ends & 4) || ((ends & 8) && t < n_odd)) snapshot(t, tot, ends);
      prev = tot;
    }
    if ((f_next & 1) || t + 1 >= (KS == 1 ? n_mine : n_loc)) mask_tile(0, 0, t + 1);
    // slot 4: PV of the second block; first half of the next block's exponentials
    pv_slot(at, 24, 1, [&](int st) __attribute__((always_inline)) { exp_step(0, st); });
    if constexpr (KS == 1) {
      end_tile(t);
    } else {
      end_half(t + 1, f_next & 2, 2 * t + 2);
      f_cur = f_next; f_next = f_far;
      k_at = k_place(2);
    }
  }
  // KS = 1: tiles that only the workgroup's other rows see: this wavefront brings in its share of the tiles ahead and
  // leaves the matrix pipe to the other half
  if constexpr (KS == 1) {
    for (; t < n_it; ++t) {
      move_window(t);
      f_far = __builtin_amdgcn_readlane(w_flags, lane_of(t + 2));
      dma_begin(lane_of(t + 3), image(t + 3));
#pragma unroll
      for (int j = 0; j < 4; ++j) dma_k(j);
      dma_v(0);
      dma_v(1);
      if constexpr (BY) {
        if (f_cur & 4) snapshot(t, running(), 0);
      }
      end_tile(t);
    }
  }
  // The output leaves the accumulation registers here, all at once and behind the last products.  (If its uses
  // further down may read them, the allocator parks some of the loop's own values there as well and moves them in
  // and out on every tile.)
  asm volatile("s_nop 15\n\ts_nop 15" : "+a"(o[0]), "+a"(o[1]), "+a"(o[2]), "+a"(o[3]));
#pragma unroll
  for (int db = 0; db < 4; ++db) asm volatile("" : "+v"(o[db]));

  // ---- epilogue ---------------------------------------------------------------------------------
  // (the images become scratch: no load may still be landing in them)
  wait_loads(std::integral_constant<int, 0>{});
  __syncthreads();
  const int ln = here(), en = ln & 31, eh = ln >> 5;
  float l_tot = lsum + __shfl_xor(lsum, 32, 64);
  float scale = 1.f / l_tot;
  bool overflow = !(l_tot > 0.f && l_tot < kSafeSum);        // the row's sum left the safe range (the sums only grow)
  float4* scratch = reinterpret_cast<float4*>(lds_all);
  float other[2][16];                                        // KS = 2: what the other stream has of this wavefront's two dim groups
  float w_other = 0.f, m_all = m_ref;
  bool none = false;                                         // KS = 2: the row sees no key of this stream
  if constexpr (KS == 2) {
    // stream 0 finishes dims 0 .. 63, stream 1 dims 64 .. 127: each hands the other half of its output over
    float2* ml = reinterpret_cast<float2*>(reinterpret_cast<char*>(lds_all) + 131072);
    if (eh == 0) ml[(ks * 4 + whead) * 32 + en] = make_float2(m_ref, l_tot);
    float4* give = scratch + ((ks ^ 1) * 4 + whead) * 512 + ln;
#pragma unroll
    for (int d = 0; d < 2; ++d)
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        float v[4];
#pragma unroll
        for (int e = 0; e < 4; ++e) v[e] = ks == 0 ? o[2 + d][4 * i + e] : o[d][4 * i + e];
        give[(d * 4 + i) * 64] = make_float4(v[0], v[1], v[2], v[3]);
      }
    __syncthreads();
    const float2 theirs = ml[((ks ^ 1) * 4 + whead) * 32 + en];
    const float4* take = scratch + (ks * 4 + whead) * 512 + ln;
#pragma unroll
    for (int d = 0; d < 2; ++d)
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        const float4 v = take[(d * 4 + i) * 64];
        other[d][4 * i] = v.x; other[d][4 * i + 1] = v.y; other[d][4 * i + 2] = v.z; other[d][4 * i + 3] = v.w;
      }
    // (a stream of which the row sees nothing has sum 0 and does not count.  By selection and not by a weight of 0: such a
    // stream may have multiplied values of a tile behind the workgroup's last position by its zeros, and these
    // need not be finite)
    none = l_tot == 0.f;
    if (theirs.y == 0.f) {
#pragma unroll
      for (int d = 0; d < 2; ++d)
#pragma unroll
        for (int i = 0; i < 16; ++i) other[d][i] = 0.f;
    }
    m_all = l_tot == 0.f ? theirs.x : theirs.y == 0.f ? m_ref : fmaxf(m_ref, theirs.x);
    const float a = l_tot == 0.f ? 0.f : __builtin_amdgcn_exp2f(m_ref - m_all);
    const float b = theirs.y == 0.f ? 0.f : __builtin_amdgcn_exp2f(theirs.x - m_all);
    const float z = l_tot * a + theirs.y * b;
    overflow = !(l_tot < kSafeSum && theirs.y < kSafeSum && z > 0.f);
    l_tot = z;
    scale = a / z;
    w_other = b / z;
  }
  // rows whose sums left the safe range are redone by the kernel that can move its reference
  const bool give_up = __any(overflow);
  if (give_up && ln == 0) redo[redo_index(q_first + (tile * TQ / 64) * 64)] = redo[redo_any] = 1;
  // The output tile goes through LDS so that a store instruction writes whole 256-byte rows of a head instead
  // of 8-byte pieces of 32 rows: row en of a head at 256 en, its 16-byte piece c at c ^ (en % 16).
  if (KS == 2) __syncthreads();                              // (both streams have taken what they need)
  if (out != nullptr) {                                      // (a caller that only wants the log-sum-exp passes none)
    char* rows = reinterpret_cast<char*>(lds_all) + (KS == 1 ? wave : whead) * 8192;
#pragma unroll
    for (int d = 0; d < (KS == 1 ? 4 : 2); ++d)
#pragma unroll
      for (int g4 = 0; g4 < 4; ++g4) {
        bf16_t v4[4];
#pragma unroll
        for (int e = 0; e < 4; ++e) {
          // accumulator register i holds output dim 32db + 8(i/4) + 4hh + i%4
          if constexpr (KS == 1) v4[e] = static_cast<bf16_t>(o[d][4 * g4 + e] * scale);
          else v4[e] = static_cast<bf16_t>((none ? 0.f : (ks == 0 ? o[d][4 * g4 + e] : o[2 + d][4 * g4 + e]) * scale) + other[d][4 * g4 + e] * w_other);
        }
        const int c = 4 * (KS == 1 ? d : 2 * ks + d) + g4;
        *reinterpret_cast<uint2*>(rows + en * 256 + ((c ^ (en & 15)) << 4) + 8 * eh) = *reinterpret_cast<uint2*>(v4);
      }
    if constexpr (KS == 2) __syncthreads();
    else wait_lds<0>();
    if (!give_up) {
      // KS = 1: the wavefront's own 32 rows; KS = 2: the two streams share the head's 32 rows
      constexpr int kRowsEach = 32 / KS;
#pragma unroll
      for (int i = 0; i < kRowsEach / 4; ++i) {
        const int rr = ks * kRowsEach + 4 * i + (ln >> 4), at = q0 + wrows + rr;
        const uint4 v = *reinterpret_cast<const uint4*>(rows + rr * 256 + (((ln & 15) ^ (rr & 15)) << 4));
        if (at < q_end) *reinterpret_cast<uint4*>(out + (static_cast<size_t>(at) * hq + h) * kD + (ln & 15) * 8) = v;
      }
    }
  }
  if (!give_up && lse != nullptr && q0 + wrows + en < q_end && eh == 0 && ks == 0)
    lse[static_cast<size_t>(q0 + wrows + en) * hq + h] = kLn2 * (m_all + __builtin_amdgcn_logf(l_tot));
}

}  // namespace

bool attn_v2_supported(const cc_ctx* ctx) {
  if (ctx->cfg.dtype != CC_BF16 || ctx->cfg.head_dim != kD) return false;
  return (ctx->cfg.n_q_heads / ctx->cfg.n_kv_heads) % 4 == 0;
}

// (CC_IMPL_MFMA_WIDE: the one-stream form at every size, as the score stage runs its 128-token form then)
static bool attn_two_streams(const cc_ctx* ctx, int n_q_tot, int max_q_per_req, int n_requests) {
  const int row_tiles = std::min((max_q_per_req + 63) / 64 * n_requests, n_q_tot / 64 + n_requests);
  return static_cast<int64_t>(row_tiles) * (ctx->cfg.n_q_heads / 4) <= kTwoStreamGrid && ctx->impl != CC_IMPL_MFMA_WIDE;
}

// A list pays from about one and a half rounds of workgroups on (a compute unit holds one), as soon as there are several
// requests: below, the second round is the short tiles of one request either way and the list's making (4 us) is lost.
// Grid / list, us: 320 workgroups 242 / 247 (2 requests of 8.1k tokens), 350: 176 / 180 (3), 480: 256 / 232 (4), 700: 387 /
// 359 (6), 1100: 516 / 487 (9), 1700: 733 / 727 (14).
// Beyond four rounds the tail is a small part, and prompts of more than kListedTiles key tiles (8 MiB of keys and values per KV head) lose more
// from short tiles of several requests side by side: 4 x 32k tokens on 1700 workgroups, the whole layer 7.72 / 7.77 ms; 8 x 20k on 6000
// the same; but 3 x 20k on 500 784 / 664 us, and the 8B batch of 32 x 5k on 5100 1 % faster listed.
// Nor for more requests than are sorted (with a list that began each request where its key tiles begin, the layer of 2000 requests of
// 2 x 17-60 tokens 1420 us without, 1752 with it, of 600 of 5-8 x 500-1000 on 8 / 2 heads 9.6 / 10.0 ms).
constexpr int kListedGrid = 400, kListedRounds = 1024, kListedTiles = 256;

WorkList attn_v2_list(const cc_ctx* ctx, const int32_t* q_pos, int n_q_tot, int max_q_per_req, int n_requests, int max_tiles) {
  WorkList list;
  const int heads = ctx->cfg.n_q_heads / 4, row_tiles = n_q_tot / 64 + n_requests;
  const int64_t grid = static_cast<int64_t>(row_tiles) * heads;
  // (a list must have room for every row tile, and one that cannot be sorted is worse than the order of the requests: 150 requests of
  // 7-9 x 200-500 tokens on 8 / 1 heads, 2200 row tiles, whole layer 1.28 / 1.22 ms)
  if (q_pos == nullptr || n_requests == 1 || n_requests > kMaxSorted || grid <= kListedGrid || row_tiles > std::min(max_tiles - 1, kMaxSortedTiles) ||
      (grid > kListedRounds && max_tiles / n_requests > kListedTiles) || !list_can_name(n_requests, (max_q_per_req + 63) / 64) || attn_two_streams(ctx, n_q_tot, max_q_per_req, n_requests))
    return list;
  list.kind = WorkList::kQueries;
  list.rows = 64;
  list.tile_bits = list_tile_bits(n_requests);
  list.places = std::max(256 / heads, 1);
  list.q_pos = q_pos;
  return list;
}

void launch_attn_v2(const cc_ctx* ctx, const void* q, const int32_t* q_pos,
                    int n_q_tot, int max_q_per_req, const void* k_pool, const void* v_pool,
                    const Plan& pl, const int32_t* req_seg_off, int n_requests, void* out, float* lse,
                    int32_t* redo, const int32_t* q_map, int map_pos, const int32_t* snap_index, float* cum,
                    int s_max, const WorkList& list, hipStream_t stream, const ValueSource& vs) {
  const int hkv = ctx->cfg.n_kv_heads, n_sub = ctx->cfg.n_q_heads / hkv / 4;
  const bool two_streams = attn_two_streams(ctx, n_q_tot, max_q_per_req, n_requests);
  // (how many rows a request has is on the device: the list is an upper bound, what is too much leaves at once)
  const int listed = list.kind != WorkList::kNone;
  const int entries = n_q_tot / 64 + n_requests;
#define CC_GO(KS, BY, TQ)                                                                                          \
  do {                                                                                                         \
    const int n_tiles = (max_q_per_req + TQ - 1) / TQ;                                                         \
    const dim3 grid = listed ? dim3(hkv * n_sub * entries) : dim3(hkv * n_sub * n_tiles, n_requests);          \
    hipLaunchKernelGGL((attn_v2_kernel<KS, BY>), grid, dim3(512), 0, stream,                                    \
                       static_cast<const bf16_t*>(q), q_pos, static_cast<const bf16_t*>(k_pool),               \
                       static_cast<const bf16_t*>(v_pool), pl.tiles, pl.max_tiles, pl.items, pl.order, list.tile_bits, \
                       req_seg_off, ctx->cfg.n_q_heads, hkv, n_sub, n_tiles, ctx->inv_freq,                    \
                       static_cast<bf16_t*>(out), lse, redo, pl.redo_any, q_map, map_pos, snap_index, cum, s_max, \
                       static_cast<const bf16_t*>(vs.v_shared), vs.n_shared_blocks,                            \
                       static_cast<const int32_t*>(vs.v_map));                                                 \
  } while (0)
  if (two_streams && cum != nullptr) CC_GO(2, true, 32);
  else if (two_streams) CC_GO(2, false, 32);
  else if (cum != nullptr) CC_GO(1, true, 64);
  else CC_GO(1, false, 64);
#undef CC_GO
}

}  // namespace cc
