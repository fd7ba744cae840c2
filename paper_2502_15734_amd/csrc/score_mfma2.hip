// cc_select's score stage for head groups that are a multiple of 4 (bf16, head_dim 128): share of a
// chunk token's softmax mass that falls on keys of earlier chunks (Eq. (2), block matrix below
// Eq. (3), Eq. (10)).
//
// One workgroup = 4 wavefronts = 4 query heads of one KV head x 128 consecutive scored tokens of a request;
// a wavefront owns one head and all 128 tokens (four column blocks of 32), so every K operand
// it reads from LDS is multiplied by 128 columns and one staged K tile serves 512 (token, head) columns.  The
// four rotated query blocks sit in accumulation registers (128), two S blocks (32) and the key block's eight K
// operands (32) in vector registers: 256 in all, so two workgroups share a compute unit.
//
// Schedule.  A 32-key block is walked column block by column block, in 16 MFMAs of 16 x 16 x 32 or eight of 32 x 32 x 16 into one S block, and
// underneath the exponentials and adds of the S block before.  (With all MFMAs of a block first and its 64
// exponentials behind them a wavefront's own chain was 2900 clocks a block, more than the two wavefronts
// of a SIMD need of the matrix pipe; now 2450 - 2600.)  A long call is then held by the clock that the chip's power budget leaves, 1.7 GHz
// with the pipe 77 % busy: hence 16 columns there, which move half the accumulator bytes per flop: 1.9 GHz, the pipe 70 % busy (this loop alone 1.44 -> 1.51 PFLOP/s; 4 x 32 k tokens 3 - 6 %
// faster, by the card, 12.70 -> 11.97 ms on one; the 8B batch of 32 2 - 3 %, 2.97 -> 2.87).  A call that is over before the clock falls waits for its
// own instructions, of which 32 columns need half as many: see score_held_by_power for the line between them.
//
// The tokens of a workgroup are numbered through the request's scored chunks: a workgroup per chunk and 128 tokens
// leaves columns empty in every chunk's last one.  Each column takes its prior chunks' mass where its own chunk
// begins (enter_chunk; once or twice per workgroup).  Which workgroup takes which tokens is in the plan's list,
// longest first and without gaps.  With a grid of (longest chunk) x (segments) the workgroups past a chunk's end
// left at once, and always in the same places: the dispatcher deals workgroups to the shader engines in turn, the
// engine that got every chunk's first tiles was busy while another idled, and of 512 places 400 were in
// use.  8B batch of 32 requests, chunks of 256 to 1024 tokens: 3.7 -> 3.15 ms for both; 2 requests of 9 x 600 tokens, 32
// heads, 465 -> 262 us.
//
// Orientation, key permutation and masking are those of mfma_tile.h: S^T = K Q^T, a lane holds
// elements of one token column (16-column MFMAs: of one in each half of a column block), the sums stay lane-local.  The query is
// pre-multiplied by log2(e)/sqrt(d), so p = exp2(S): no reference is subtracted.  That is exact as
// long as the sums stay in range; a workgroup whose sums leave the safe range (logits beyond about
// +-60) flags its tokens and the kernel that carries a movable reference redoes them (see the
// launcher).
//
// Small grids take a second form: 64 tokens per workgroup and eight wavefronts, two key streams (KS = 2: wavefronts 0-3 walk
// the even key tiles, 4-7 the odd ones, each stream with images of its own; the sums are just added at the end).
// With one workgroup per compute unit the four-wavefront form has nothing to put beside its exponentials;
// the second stream is that, and halves the chain of tiles.  It takes 32-column MFMAs (the loop of an 8B request of 2.6 k tokens 23.0 us, 24.0 with 16).
//
// Staging: four K-tile images in LDS (16 KiB each), filled by loads that write LDS directly
// (global_load_lds, lane L of an instruction fills piece base + L), whole 128-byte lines each:
//   K piece (row m of 32-key block b, 16-byte piece p of the row):
//       ((b*2 + p/8)*4 + m/8)*64 + (p%8 ^ x)*8 + m%8,  x = (m/8)%2 for 32-column MFMAs, 0 for 16-column ones
// (an operand read walks 32 rows at two neighbouring pieces, or 16 at four; ds_read_b128 takes lanes 0-3, 12-15, 20-23, 24-27 together and
// so on, and these meet no bank twice.  With x = (m/8)%2 the 16-row walk would: half the rate.)
// In iteration t the wavefronts read image t and, between its MFMAs, start the loads of image t+3; before the
// iteration's barrier each wavefront waits until its loads of image t+2 have landed.  Padding
// slots of K never reach a sum: their S entries are masked by selection.
#include <algorithm>
#include <type_traits>

#include "mfma_tile.h"

namespace cc {

using namespace tile;

namespace {

typedef __attribute__((__vector_size__(4 * sizeof(uint32_t)))) uint32_t u32x4;

constexpr int kBigQB = 4, kSmallQB = 2;   // 32-token column blocks per wavefront: big grids, small ones
constexpr int kImageK = 1024;     // 16-byte pieces per K tile image
constexpr int kBufs = 4;
// p = exp2(S) with no reference: sums outside this range leave too little headroom (above) or may
// have lost small terms to underflow (below)
constexpr float kSafeSum = 1.0e30f;
constexpr float kTinySum = 1.0e-18f;

// 64 lanes x 16 bytes from global memory straight into LDS: lane L's 16 bytes land at M0 + immediate + 16 L, read
// from base + voff(L) + immediate.  Written as an instruction the compiler does not model:
// it would otherwise drain every outstanding load before the next LDS read, because it cannot see
// that the image being filled is not the image being read.  Completion is counted by vmcnt.
template <int IMM>
__device__ __forceinline__ void load_to_lds(uint32_t voff, const char* base, uint32_t m0v) {
  asm volatile("s_mov_b32 m0, %2\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %0, %1 offset:%3"
               :: "v"(voff), "s"(base), "s"(m0v), "n"(IMM) : "memory", "m0");
}

// MFMA forms with fixed register classes (see attn_mfma2.hip): S accumulates in vector registers,
// the rotated query is the B operand out of accumulation registers.  The results are opaque to the
// compiler's hazard handling: the vector ALU reads them at least two MFMAs behind their producer or
// behind mfma_result_wait().
// A block of S, 32 keys x 32 tokens, in products of W columns (W 32: v_mfma_f32_32x32x16_bf16, W 16: v_mfma_f32_16x16x32_bf16).  Lane
// (c, g) = (lane % W, lane / W) of an operand holds dims (512 / W) k + 8 g .. + 7 of k-step k.  A lane's 16 elements i are in the order in which the
// exponentials take them: element i is that of token half i / (16 W / 32) and of key key(i) + lane_key(g).
template <int W> struct ScoreBlock;
template <> struct ScoreBlock<32> {
  static constexpr int kSteps = 8;                 // MFMAs of a block
  f32x16 s;
  // step st: K operand st, query operand st
  __device__ __forceinline__ void multiply(int st, const u32x4& k, const u32x4& q) {
    if (st == 0) asm volatile("v_mfma_f32_32x32x16_bf16 %0, %1, %2, 0" : "=&v"(s) : "v"(k), "a"(q));
    else asm volatile("v_mfma_f32_32x32x16_bf16 %0, %1, %2, %0" : "+v"(s) : "v"(k), "a"(q));
  }
  // exponentials of the block before under step st: first(st) .. first(st + 1) - 1 (none under the first: 2 2 2 2 3 2 3 under the others)
  static constexpr int first(int st) { return st < 1 ? 0 : st < 6 ? 2 * (st - 1) : st < 8 ? 2 * st - 1 : 16; }
  static constexpr int key(int i) { return 16 * (i / 8) + i % 8; }
  static __device__ __forceinline__ int lane_key(int g) { return 8 * g; }
  __device__ __forceinline__ float get(int i) const { return s[i]; }
  __device__ __forceinline__ void set(int i, float v) { s[i] = v; }
  __device__ __forceinline__ void pin() { asm volatile("" : "+v"(s)); }
};
template <> struct ScoreBlock<16> {
  static constexpr int kSteps = 16;
  f32x4 s[2][2];                                   // [16-key half][token half]
  // step st: k-step st / 4, 16-key half st / 2 % 2, token half st % 2: the same accumulator every fourth step, so that none waits for the one before
  __device__ __forceinline__ void multiply(int st, const u32x4& k, const u32x4& q) {
    f32x4& d = s[(st >> 1) & 1][st & 1];
    if (st < 4) asm volatile("v_mfma_f32_16x16x32_bf16 %0, %1, %2, 0" : "=&v"(d) : "v"(k), "a"(q));
    else asm volatile("v_mfma_f32_16x16x32_bf16 %0, %1, %2, %0" : "+v"(d) : "v"(k), "a"(q));
  }
  static constexpr int first(int st) { return st; }                  // (element st's last product lies four MFMAs back at least)
  static constexpr int key(int i) { return 16 * ((i >> 2) & 1) + (i & 3); }      // (row 4 g + e of a half is its key swap23(4 g + e))
  static __device__ __forceinline__ int lane_key(int g) { return 8 * (g & 1) + 4 * (g >> 1); }
  __device__ __forceinline__ float get(int i) const { return s[(i >> 2) & 1][i >> 3][i & 3]; }
  __device__ __forceinline__ void set(int i, float v) { s[(i >> 2) & 1][i >> 3][i & 3] = v; }
  __device__ __forceinline__ void pin() {
#pragma unroll
    for (int i = 0; i < 4; ++i) asm volatile("" : "+v"(s[i >> 1][i & 1]));
  }
};
__device__ __forceinline__ void mfma_result_wait() {
  asm volatile("s_nop 15\n\ts_nop 15" ::: "memory");
}
// l += e (the exponential taken two steps ago), then e = exp2(s): two such e in turn, so that an add never waits
// for the exponential it takes.  Written out so that it stays where it is placed, under one MFMA.
__device__ __forceinline__ void exp_step(float& l, float& e, float s) {
  asm volatile("v_add_f32 %0, %0, %1\n\tv_exp_f32 %1, %2" : "+v"(l), "+v"(e) : "v"(s));
}
// one 16-byte piece into accumulation registers
__device__ __forceinline__ u32x4 to_acc(const u32x4& v) {
  u32x4 r;
#pragma unroll
  for (int i = 0; i < 4; ++i) asm volatile("v_accvgpr_write_b32 %0, %1" : "=a"(r[i]) : "v"(v[i]));
  return r;
}

// Cosines and sines, times `scale`, of a position's angles of two rotation pairs
__device__ __forceinline__ float4 two_turns(const double (&freq)[2], int pos, float scale) {
  float4 t;
  rot_cos_sin_fast(pos, freq[0], &t.x, &t.y);
  rot_cos_sin_fast(pos, freq[1], &t.z, &t.w);
  t.x *= scale; t.y *= scale; t.z *= scale; t.w *= scale;
  return t;
}

// One workgroup = 128 (kQB = 4) or 64 (kQB = 2) consecutive scored tokens of a request, whatever chunks they lie in.
// Products of W columns.
template <int kQB, int KS, int W>
__global__ __launch_bounds__(256 * KS, 2) void score_v2_kernel(
    const bf16_t* __restrict__ q, const bf16_t* __restrict__ k_pool,
    const TileDesc* __restrict__ tiles, int max_tiles, int tile_bits, const cc_segment* __restrict__ segs,
    int n_requests, const int32_t* __restrict__ req_seg_off, const int32_t* __restrict__ seg_tile_off, int hq, int hkv, int n_sub,
    InvFreq inv_freq, float* __restrict__ mass, int32_t* __restrict__ redo, int redo_any) {
  constexpr int kTQ = 32 * kQB;               // tokens per workgroup
  constexpr int kTG = 32 / W, kKS = 8 / kTG;  // token halves of a block; k-steps
  static_assert(kQB % 2 == 0, "two S blocks in turn");
  __shared__ uint4 lds_all[KS * kBufs * kImageK];
  __shared__ int4 tokens[kTQ];                // what is rarely asked of a token: position, row, first key tile of its chunk
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = uniform(tid >> 6) & 3, ks = KS == 1 ? 0 : uniform(tid >> 8);      // head of the four; key stream
  const int n = lane & 31, c = lane & (W - 1), g = lane / W;      // token of a 32-token block; lane of an operand (ScoreBlock)
  const int per_tile = hkv * n_sub;
  const int entry = blockIdx.x / per_tile, rem = blockIdx.x % per_tile;
  const int kvh = rem % hkv, hsub = rem / hkv;
  const int h = kvh * (4 * n_sub) + hsub * 4 + wave;

  // ---- which tokens ---------------------------------------------------------------------------
  const int e = tiles[entry].work, n_list = tiles[max_tiles - 1].work;
  int seg_begin, seg_end;
  if (n_requests == 1) {                      // (a load that need not wait for the list's)
    seg_begin = req_seg_off[0];
    seg_end = req_seg_off[1];
  } else {
    if (entry >= uniform(n_list)) return;     // (what is behind the list names no request)
    const int req = uniform(static_cast<int>(static_cast<uint32_t>(e) >> tile_bits));
    seg_begin = req_seg_off[req];
    seg_end = req_seg_off[req + 1];
  }
  seg_begin = uniform(seg_begin);
  seg_end = uniform(seg_end);
  if (entry >= uniform(n_list)) return;
  const int u0 = uniform(e & ((1u << tile_bits) - 1)) * kTQ;
  const int j_begin = uniform(seg_tile_off[seg_begin]);
  // The scored tokens of the request are numbered through; this workgroup has u0 .. u0 + kTQ - 1.  A lane looks at one
  // segment; those that hold tokens of the workgroup (mostly one or two) are then walked.  Columns past the last
  // token repeat it; nothing of theirs is written.
  int row[kQB], pos[kQB], own[kQB], u_end = u0, t_last = -1;
#pragma unroll
  for (int qb = 0; qb < kQB; ++qb) row[qb] = pos[qb] = own[qb] = 0;
  for (int g0 = seg_begin, before = 0; g0 < seg_end && before < u0 + kTQ; g0 += 64) {
    const int s = min(g0 + lane, seg_end - 1);
    const cc_segment sg = segs[s];
    const int s_start = sg.logical_start, s_off = sg.tok_off, s_own = seg_tile_off[s] - j_begin;
    const int cnt = g0 + lane < seg_end && sg.kind == CC_SEG_CHUNK && s_start > 0 ? max(sg.n_tokens, 0) : 0;
    int incl = cnt;
#pragma unroll
    for (int o = 1; o < 64; o <<= 1) {
      const int up = __shfl_up(incl, o, 64);
      if (lane >= o) incl += up;
    }
    const int first = before + incl - cnt;
    for (uint64_t m = __ballot(cnt > 0 && first < u0 + kTQ && first + cnt > u0); m != 0; m &= m - 1) {
      const int l = __ffsll(static_cast<unsigned long long>(m)) - 1;
      const int c_first = __builtin_amdgcn_readlane(first, l), c_cnt = __builtin_amdgcn_readlane(cnt, l);
      const int c_start = __builtin_amdgcn_readlane(s_start, l), c_off = __builtin_amdgcn_readlane(s_off, l);
      const int c_own = __builtin_amdgcn_readlane(s_own, l);
      u_end = min(u0 + kTQ, c_first + c_cnt);
      t_last = max(t_last, c_own + (u_end - 1 - c_first) / kTile);
#pragma unroll
      for (int qb = 0; qb < kQB; ++qb) {
        const int u = u0 + 32 * qb + n, in = min(u, u_end - 1) - c_first;      // (columns behind the segment: its last token, for now)
        if (u >= c_first) { row[qb] = c_off + in; pos[qb] = c_start + in; own[qb] = c_own; }
      }
    }
    before += __builtin_amdgcn_readlane(incl, 63);
  }
  const int n_t = uniform(min(j_begin + t_last + 1, max_tiles) - j_begin);
  if (n_t <= 0) return;
  const int p_min = uniform(wave_min_i(pos[0]));
  if (wave == 0 && ks == 0 && lane < 32) {
#pragma unroll
    for (int qb = 0; qb < kQB; ++qb) tokens[32 * qb + n] = make_int4(pos[qb], row[qb], own[qb], 0);
  }
  // iterations; the one in which this wavefront's stream enters the chunk that begins with key tile t (n_it or more: never)
  const int n_it = (n_t + KS - 1) / KS;
  auto it_of = [&](int t) __attribute__((always_inline)) { return KS == 1 ? t : (t - ks + 1) >> 1; };

  // ---- query rows, two column blocks at a time -----------------
  // for token half tg of the block and k-step k a lane keeps 8 dims of token W tg + c (see ScoreBlock); dims < 64 pair with dims + 64.
  uint4 rows[2][8];
  auto load_rows = [&](int qb) __attribute__((always_inline)) {
    load_query_rows(rows[qb & 1], q, qb < 2 ? row[qb] : tokens[32 * qb + n].y, hq, h, lane);
  };

  // ---- descriptors and staging --------------------------------------------------------------------
  // What the loop needs of 64 consecutive tiles sits in vector registers, one tile per lane, and is handed out with
  // v_readlane: no memory access per tile.  w_own: block of the page this wavefront brings in; w_edge: the tile
  // needs masking for some token (padding, or its last key lies behind p_min).
  int win_base = 0;
  int w_kpos0, w_nvalid, w_own, w_edge;
  auto fill_window = [&](int base) __attribute__((always_inline)) {
    const int j = KS * (base + lane) + ks;
    const TileDesc d = fetch_desc(tiles, j_begin + min(j, n_t - 1), max_tiles);
    w_kpos0 = d.kpos0;
    w_nvalid = j >= n_t ? 0 : d.nvalid;                // (the odd stream may have one tile less: it is masked as a whole)
    w_own = wave == 0 ? d.blk[0] : wave == 1 ? d.blk[1] : wave == 2 ? d.blk[2] : d.blk[3];
    w_edge = w_nvalid < kTile || d.kpos0 + kTile - 1 > p_min;
  };
  fill_window(0);
  auto lane_of = [&](int t) __attribute__((always_inline)) { return min(t, n_it - 1) - win_base; };      // t in [win_base, win_base + 64)
  auto image_off = [&](int t) __attribute__((always_inline)) { return (ks * kBufs + (t & (kBufs - 1))) * (kImageK * 16); };   // bytes
  // Loads of one K tile: wavefront w brings page w.  Instruction j = 2 rg + kq brings rows 8 rg .. 8 rg + 7 of the
  // page (row r sits in token slot swap23(r)), 128 bytes each at dim 64 kq: lane L reads row 8 rg + L % 8,
  // piece L / 8 (32 columns: pieces of odd row groups with the lowest bit turned).  Addresses are a scalar base, a per-lane constant and an immediate.
  const size_t blk_bytes = static_cast<size_t>(hkv) * (kBlock * kD) * sizeof(bf16_t);
  const char* k_head = reinterpret_cast<const char*>(k_pool) + static_cast<size_t>(kvh) * (kBlock * kD * sizeof(bf16_t));
  constexpr int kSwizzle = W == 32 ? 1 : 0;
  const uint32_t k_voff0 = swap23(lane & 7) * (kD * 2) + (lane >> 3) * 16;
  const uint32_t k_voff1 = swap23(8 + (lane & 7)) * (kD * 2) + ((lane >> 3) ^ kSwizzle) * 16;
  typedef __attribute__((address_space(3))) const uint4 lds_piece;
  const uint32_t lds_base = uniform(static_cast<uint32_t>(reinterpret_cast<uintptr_t>((lds_piece*)lds_all)));   // LDS byte address
  const uint32_t k_img = lds_base + ((wave >> 1) * 8 + (wave & 1) * 2) * 1024;
  const char* k_src = nullptr;
  uint32_t k_dst = 0;
  auto dma_begin = [&](int t) __attribute__((always_inline)) {            // (past the last tile: that tile again, into an image nobody reads)
    const int own = __builtin_amdgcn_readlane(w_own, lane_of(t));
    const uint64_t src = reinterpret_cast<uint64_t>(k_head) + static_cast<size_t>(max(own, 0)) * blk_bytes;
    k_src = reinterpret_cast<const char*>(static_cast<uint64_t>(static_cast<uint32_t>(uniform(static_cast<int>(src >> 32)))) << 32 |
                                          static_cast<uint32_t>(uniform(static_cast<int>(src))));
    k_dst = k_img + image_off(t);
  };
  auto dma = [&](int j) __attribute__((always_inline)) {
    if (j == 0) load_to_lds<0>(k_voff0, k_src, k_dst);
    else if (j == 1) load_to_lds<128>(k_voff0, k_src, k_dst + (4096 - 128));
    else if (j == 2) load_to_lds<0>(k_voff1, k_src, k_dst + 1024);
    else load_to_lds<128>(k_voff1, k_src, k_dst + 1024 + (4096 - 128));
  };
  auto dma_tile = [&](int t) __attribute__((always_inline)) {
    dma_begin(t);
#pragma unroll
    for (int j = 0; j < 4; ++j) dma(j);
  };
  // wait until at most `newer` of this wavefront's vector-memory operations are outstanding
  auto wait_loads = [&](auto newer) __attribute__((always_inline)) {
    constexpr int kN = decltype(newer)::value;
    __builtin_amdgcn_s_waitcnt((kN & 15) | ((kN >> 4) << 14) | (7 << 4) | (15 << 8));
    asm volatile("" ::: "memory");
  };
  auto wait_lds = [&]() __attribute__((always_inline)) { __builtin_amdgcn_s_waitcnt(15 | (3 << 14) | (7 << 4)); };
  auto barrier = [&]() __attribute__((always_inline)) {
    asm volatile("" ::: "memory");
    __builtin_amdgcn_s_barrier();
    asm volatile("" ::: "memory");
  };
  load_rows(0);
  load_rows(1);
  // (images 2 and 3 are scratch until the queries are turned)
  dma_tile(0);
  dma_tile(1);

  // ---- rotate the queries to their positions, fold the softmax scale -----------------------------------
  // The four heads share the angles: a wavefront computes 8 / KS of a column block's 32 and reads the others'
  // from LDS, two column blocks at a time.
  const float c2 = 0.08838834764831845f * kLog2e;            // log2(e) / sqrt(128)
  char* lds_bytes = reinterpret_cast<char*>(lds_all);
  char* own_scratch = lds_bytes + (ks * kBufs + 2) * (kImageK * 16) + wave * 8192;
  u32x4 qreg[kQB][8];
  // A lane's angles of a block are 16 float4 (two rotation pairs each): number j is that of token half j / 4 / (kKS / 2), k-step
  // j / 4 % (kKS / 2) and the pairs 2 (j % 4), + 1 of its 8.  This wavefront makes the 4 / KS from here on.
  const int first = (4 / KS) * (KS == 1 ? wave : wave + 4 * ks);
#pragma unroll
  for (int qp = 0; qp < kQB; qp += 2) {
    if (qp > 0) barrier();                                  // (the angles before have been read)
#pragma unroll
    for (int u = 0; u < 2; ++u) regroup_query_rows<W>(rows[u], own_scratch, lane);
    double freq[4 / KS][2];                                 // (a lane's own: vector loads)
#pragma unroll
    for (int i = 0; i < 4 / KS; ++i)
#pragma unroll
      for (int j = 0; j < 2; ++j) freq[i][j] = inv_freq.f[512 / W * ((first >> 2) % (kKS / 2)) + 2 * ((first + i) & 3) + 8 * g + j];
    barrier();
    float4* turns[2];
#pragma unroll
    for (int u = 0; u < 2; ++u) {
      turns[u] = reinterpret_cast<float4*>(lds_bytes + (2 + u) * (kImageK * 16)) + lane;
      const int token = W * ((first >> 2) / (kKS / 2)) + c;
      const int at = qp == 0 ? (kTG == 1 ? pos[u] : __shfl(pos[u], token, 64)) : tokens[32 * (qp + u) + token].x;
#pragma unroll
      for (int i = 0; i < 4 / KS; ++i) turns[u][(first + i) * 64] = two_turns(freq[i], at, c2);
    }
    wait_lds();
    barrier();
#pragma unroll
    for (int u = 0; u < 2; ++u) {
#pragma unroll
      for (int j = 0; j < 4; ++j) {
        const int x_at = kKS * (j / (kKS / 2)) + j % (kKS / 2), y_at = x_at + kKS / 2;
        u32x4 xv = __builtin_bit_cast(u32x4, rows[u][x_at]), yv = __builtin_bit_cast(u32x4, rows[u][y_at]);
#pragma unroll
        for (int i = 0; i < 4; ++i) {
          uint32_t x = xv[i], y = yv[i];
          turn_words(x, y, turns[u][(j * 4 + i) * 64]);
          xv[i] = x;
          yv[i] = y;
        }
        qreg[qp + u][x_at] = to_acc(xv);
        qreg[qp + u][y_at] = to_acc(yv);
        __builtin_amdgcn_sched_barrier(0);
      }
      if (qp + 2 < kQB) load_rows(qp + 2 + u);
    }
  }

  // ---- one column block of a 32-key block: S, and underneath the exponentials of the column block before ----------
  const int k_rd = (c >> 3) * 1024 + (g ^ (kSwizzle & (c >> 3))) * 128 + (c & 7) * 16;      // this lane's operand pieces inside an image
  float l_run[kQB][kTG], l_prior[kQB][kTG], ev[2] = {0.f, 0.f};   // (of the lane's tokens in a column block)
  ScoreBlock<W> sacc[2];
  u32x4 ring[8];                               // K operands of the block, in the order of their use
#pragma unroll
  for (int i = 0; i < 16; ++i) { sacc[0].set(i, 0.f); sacc[1].set(i, -INFINITY); }
#pragma unroll
  for (int i = 0; i < kQB * kTG; ++i) l_run[i / kTG][i % kTG] = l_prior[i / kTG][i % kTG] = 0.f;
  // K operand j: k-step j / kTG, 16-key half j % kTG
  auto piece = [&](int img_off, int blk, int j) __attribute__((always_inline)) {
    const int p = 64 / W * (j / kTG);
    return *reinterpret_cast<const u32x4*>(lds_bytes + img_off + k_rd + blk * 8192 + (p >> 3) * 4096 + (j % kTG) * 2048 + (p & 7) * 128);
  };
  // element i of the S block of column block qb; the add is that of the element two steps ago
  auto exp_element = [&](int qb, int i) __attribute__((always_inline)) {
    exp_step(i < 2 ? l_run[(qb + kQB - 1) % kQB][kTG - 1] : l_run[qb][(i - 2) * kTG / 16], ev[i & 1], sacc[qb & 1].get(i));
  };
  // padding / causal edge: entries the token must not see become -inf
  auto mask = [&](int qb, int blk, int t) __attribute__((always_inline)) {
    mfma_result_wait();
    const int kpos0 = __builtin_amdgcn_readlane(w_kpos0, t - win_base), nvalid = __builtin_amdgcn_readlane(w_nvalid, t - win_base);
#pragma unroll
    for (int tg = 0; tg < kTG; ++tg) {
      int lim = min(nvalid - 1, tokens[32 * qb + W * tg + c].x - kpos0) - ScoreBlock<W>::lane_key(g) - 32 * blk;
      asm volatile("" : "+v"(lim));
#pragma unroll
      for (int i = 16 / kTG * tg; i < 16 / kTG * (tg + 1); ++i)
        sacc[qb & 1].set(i, ScoreBlock<W>::key(i) <= lim ? sacc[qb & 1].get(i) : -INFINITY);
    }
    sacc[qb & 1].pin();
  };
  // the last column block of a block is still to be summed when the next block begins: finish it
  auto drain = [&]() __attribute__((always_inline)) {
    mfma_result_wait();
#pragma unroll
    for (int i = 0; i < 16; ++i) exp_element(kQB - 1, i);
    asm volatile("s_nop 1\n\tv_add_f32 %0, %0, %1\n\tv_add_f32 %0, %0, %2" : "+v"(l_run[kQB - 1][kTG - 1]) : "v"(ev[0]), "v"(ev[1]));
    ev[0] = 0.f;
    ev[1] = 0.f;
#pragma unroll
    for (int i = 0; i < 16; ++i) sacc[1].set(i, -INFINITY);
    sacc[1].pin();
  };
  // tokens whose own chunk begins with iteration `from` or, up to `to`, later: all they have summed so far is prior-chunk mass.
  // Returns the next iteration in which a chunk of the workgroup's tokens begins.
  auto enter_chunk = [&](int from, int to) __attribute__((always_inline)) {
    int next = 0x7fffffff;
#pragma unroll
    for (int qb = 0; qb < kQB; ++qb)
#pragma unroll
      for (int tg = 0; tg < kTG; ++tg) {
        const int it = it_of(tokens[32 * qb + W * tg + c].z);
        const bool now = it >= from && it <= to;
        l_prior[qb][tg] = now ? l_run[qb][tg] : l_prior[qb][tg];
        l_run[qb][tg] = now ? 0.f : l_run[qb][tg];
        if (it > to) next = min(next, it);
      }
    return uniform(wave_min_i(next));
  };

  wait_loads(std::integral_constant<int, 0>{});
  __syncthreads();
  dma_tile(2);
#pragma unroll
  for (int j = 0; j < 8; ++j) ring[j] = piece(image_off(0), 0, j);
  int edge = __builtin_amdgcn_readlane(w_edge, 0);
  int it_enter = enter_chunk(0, -1);
  wait_lds();          // (whatever leads into the loop body leaves nothing pending there: the body's own reads could then not be waited for one by one)

  constexpr int kSteps = ScoreBlock<W>::kSteps;
  // ---- the tile loop --------------------------------------------------------------------------------
  for (int t = 0; t < n_it; ++t) {
    const int img = image_off(t), nimg = image_off(t + 1);      // (behind the last tile the next image holds stale keys nobody uses)
    if (min(t + 3, n_it - 1) - win_base >= 64) {                // next 64 descriptors, starting at tile t (rare)
      win_base = t;
      fill_window(t);
      __builtin_amdgcn_s_waitcnt((7 << 4) | (15 << 8));         // vmcnt(0) here, so the hot path never waits for it
    }
    if (t == it_enter) {                                        // a chunk with tokens of the workgroup begins (rare)
      drain();
      it_enter = enter_chunk(t, t);
      wait_lds();
    }
    int edge_next = 0;
#pragma unroll
    for (int blk = 0; blk < 2; ++blk) {
#pragma unroll
      for (int qb = 0; qb < kQB; ++qb) {
#pragma unroll
        for (int st = 0; st < kSteps; ++st) {
          const int j = st / kTG, tg = st % kTG;                 // K operand; token half
          sacc[qb & 1].multiply(st, ring[j], qreg[qb][kKS * tg + j / kTG]);
          if (qb == kQB - 1 && tg == kTG - 1) ring[j] = blk == 0 ? piece(img, 1, j) : piece(nimg, 0, j);
#pragma unroll
          for (int i = ScoreBlock<W>::first(st); i < ScoreBlock<W>::first(st + 1); ++i) exp_element((qb + kQB - 1) % kQB, i);
          // the loads of tile t+3, one instruction every quarter of the block
          if (blk == 0 && qb == 0 && st == 0) {
            dma_begin(t + 3);
            edge_next = __builtin_amdgcn_readlane(w_edge, lane_of(t + 1));
          }
          if (blk == 0 && qb == 0 && st % (kSteps / 4) == kSteps / 4 - 1) dma(st / (kSteps / 4));
          __builtin_amdgcn_sched_barrier(0);
        }
        if (edge) mask(qb, blk, t);
      }
    }
    // image t+2 (loads started one iteration ago) must be whole before anyone reads it
    wait_loads(std::integral_constant<int, 4>{});
    barrier();
    edge = edge_next;
  }
  drain();

  // ---- epilogue ---------------------------------------------------------------------------------
  wait_loads(std::integral_constant<int, 0>{});        // (nothing may still be landing when the LDS is given back or used)
  if constexpr (KS == 2) {
    enter_chunk(n_it, 0x7ffffffe);                       // (no tile of the chunk itself in this stream)
    __syncthreads();
    float2* share = reinterpret_cast<float2*>(lds_all) + wave * (kQB * kTG * 64) + lane;
    if (ks == 1) {
#pragma unroll
      for (int i = 0; i < kQB * kTG; ++i) share[i * 64] = make_float2(l_prior[i / kTG][i % kTG], l_run[i / kTG][i % kTG]);
    }
    __syncthreads();
    if (ks == 1) return;
#pragma unroll
    for (int i = 0; i < kQB * kTG; ++i) {
      const float2 o = share[i * 64];
      l_prior[i / kTG][i % kTG] += o.x;
      l_run[i / kTG][i % kTG] += o.y;
    }
  }
  bool bad = false;
  float lp[kQB][kTG], lt[kQB][kTG];
  auto over_keys = [&](float v) __attribute__((always_inline)) {      // (a token's keys are spread over 64 / W lanes)
#pragma unroll
    for (int o = W; o < 64; o <<= 1) v += __shfl_xor(v, o, 64);
    return v;
  };
#pragma unroll
  for (int i = 0; i < kQB * kTG; ++i) {
    float &t = lt[i / kTG][i % kTG], &p = lp[i / kTG][i % kTG];
    t = over_keys(l_run[i / kTG][i % kTG]);
    p = over_keys(l_prior[i / kTG][i % kTG]);
    bad = bad || !(p + t > kTinySum && p + t < kSafeSum);
  }
  // tokens whose sums left the safe range are redone by the kernel that carries a reference
  const bool give_up = __any(bad);
#pragma unroll
  for (int i = 0; i < kQB * kTG; ++i) {
    const int u = W * i + c;
    if (u0 + u >= u_end || g != 0) continue;
    const int at = tokens[u].y;
    const float t = lt[i / kTG][i % kTG], p = lp[i / kTG][i % kTG];
    if (give_up) redo[at >> 6] = redo[redo_any] = 1;
    else mass[static_cast<size_t>(at) * hq + h] = p / (p + t);
  }
}

}  // namespace

bool score_v2_supported(const cc_ctx* ctx) {
  if (ctx->cfg.dtype != CC_BF16 || ctx->cfg.head_dim != kD) return false;
  return (ctx->cfg.n_q_heads / ctx->cfg.n_kv_heads) % 4 == 0;
}

void launch_score_v2(const cc_ctx* ctx, const void* q, const void* k_pool, const Plan& pl, const cc_segment* segs,
                     const int32_t* req_seg_off, int n_requests, int n_tok, float* mass, int32_t* redo, ScoreForm form,
                     const WorkList& list, hipStream_t stream) {
  const int hkv = ctx->cfg.n_kv_heads, n_sub = ctx->cfg.n_q_heads / hkv / 4, per_tile = hkv * n_sub;
  // (the chunks' lengths are on the device: the grid is an upper bound, what is too much leaves at once)
  const bool small = form == ScoreForm::kSmall;
  const int rows = small ? 32 * kSmallQB : 32 * kBigQB;
  const int entries = std::min(n_tok / rows + n_requests, pl.max_tiles - 1);
#define CC_LAUNCH(...)                                                                                        \
  hipLaunchKernelGGL((score_v2_kernel<__VA_ARGS__>), dim3(per_tile * entries), dim3(small ? 512 : 256), 0, stream, static_cast<const bf16_t*>(q), \
                     static_cast<const bf16_t*>(k_pool), pl.tiles, pl.max_tiles, list.tile_bits, segs, n_requests, req_seg_off, pl.seg_tile_off,  \
                     ctx->cfg.n_q_heads, hkv, n_sub, ctx->inv_freq, mass, redo, pl.redo_any)
  if (small) CC_LAUNCH(kSmallQB, 2, 32);
  else if (form == ScoreForm::kBig) CC_LAUNCH(kBigQB, 1, 32);
  else CC_LAUNCH(kBigQB, 1, 16);
#undef CC_LAUNCH
}

}  // namespace cc
