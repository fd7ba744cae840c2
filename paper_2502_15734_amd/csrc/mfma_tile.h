// Shared pieces of the MFMA (bf16, head_dim 128) kernels: the 64-key tile descriptor written by the
// plan kernels, the LDS image layout of a staged K/V tile, and the register-prefetch stager.
//
// LDS image of a tile (16-byte pieces; every MFMA operand read is one conflict-free 1 KiB run):
//   K piece (block b of 32 keys, k-step kk, half hh, row m):  (b*8+kk)*64 + hh*32 + (m ^ ((2kk+hh)&7))
//   V piece (page pg, 32-dim group db, half hh, dim n):       1024 + (pg*4+db)*64 + hh*32 + (n ^ 4hh)
// The XOR terms spread the *writes* of a coalesced global read over the LDS banks.  Within a
// 32-key block the MFMA row m holds the key swap_bits_2_3(m), so that the 8 accumulator values a
// lane-half feeds to one 16-key step of the second product are slots 8*half..8*half+7 of one
// 16-token block -- one 16-byte piece of the dimension-major V block.
#pragma once

#include "device_util.h"

namespace cc {
namespace tile {

constexpr int kD = 128;
constexpr int kTile = 64;                      // keys per tile
constexpr float kLog2e = 1.4426950408889634f;
constexpr float kLn2 = 0.6931471805599453f;
constexpr float kBig = 1.0e12f;                // a tile sum above this moves the reference maximum
constexpr float kZeroBand = 24.f;              // first-block maxima within this keep the reference at 0

__device__ __forceinline__ int swap23(int m) { return (m & ~12) | ((m & 4) << 1) | ((m & 8) >> 1); }
__device__ __forceinline__ int uniform(int v) { return __builtin_amdgcn_readfirstlane(v); }

// One key tile as the plan kernels lay it out (32 bytes, read with two 16-byte loads).
struct TileDesc {
  int32_t kpos0;     // logical position of the tile's first key
  int32_t nvalid;    // keys of the tile that exist (1..64); the rest is block padding
  int32_t blk[4];    // physical block of each of the four 16-token pages (-1: none)
  int32_t seg;       // segment the tile belongs to
  int32_t work;      // (not of this tile) entry of the list of workgroups, see WorkList
};
static_assert(sizeof(TileDesc) == 32, "descriptor is read as two 16-byte vectors");

// a descriptor that came in through a (broadcast) vector load, moved to scalar registers
__device__ __forceinline__ TileDesc to_scalar(const TileDesc& v) {
  TileDesc d;
  d.kpos0 = __builtin_amdgcn_readfirstlane(v.kpos0);
  d.nvalid = __builtin_amdgcn_readfirstlane(v.nvalid);
#pragma unroll
  for (int i = 0; i < 4; ++i) d.blk[i] = __builtin_amdgcn_readfirstlane(v.blk[i]);
  d.seg = 0;
  d.work = 0;
  return d;
}

// The index is laundered through a vector register on purpose: a scalar (SMEM) load here would
// share the LDS operand reads' completion counter, return out of order, and force a full drain
// of the operand ring every tile; a broadcast vector load is counted with the global loads.
__device__ __forceinline__ TileDesc fetch_desc(const TileDesc* __restrict__ tiles, int j, int max_tiles) {
  int jj = min(max(j, 0), max_tiles - 1);
  asm volatile("" : "+v"(jj));
  const uint4* src = reinterpret_cast<const uint4*>(tiles + jj);
  union { uint4 v[2]; TileDesc d; } u;
  u.v[0] = src[0];
  u.v[1] = src[1];
  return u.d;
}

// LDS piece index of piece `cc_` (0..255, pool order) of page `pg` of the K / V tile image.
__device__ __forceinline__ int k_piece_dst(int pg, int cc_) {
  const int slot = cc_ >> 4, ch = cc_ & 15;
  // key a = 16*pg + slot of the tile -> block a/32, MFMA row swap23(a%32)
  return ((pg >> 1) * 8 + (ch >> 1)) * 64 + (ch & 1) * 32 + (((pg & 1) * 16 + swap23(slot)) ^ (ch & 7));
}
__device__ __forceinline__ int v_piece_dst(int pg, int cc_) {
  const int dcol = cc_ >> 1, hh = cc_ & 1;
  return 1024 + (pg * 4 + (dcol >> 5)) * 64 + hh * 32 + ((dcol & 31) ^ (4 * hh));
}
// V piece with the slots >= nv (padding of a partly filled block) zeroed.
__device__ __forceinline__ uint4 zero_pad_slots(uint4 val, int hh, int nv) {
  unsigned short e[8];
  *reinterpret_cast<uint4*>(e) = val;
#pragma unroll
  for (int j = 0; j < 8; ++j) if (8 * hh + j >= nv) e[j] = 0;
  return *reinterpret_cast<uint4*>(e);
}

// Staging of one key tile (and, if WITH_V, the value tile) of KV head `kvh` for workgroups of 256
// or 512 threads.  A thread owns the same 16-byte piece of every page it stages (thread t ->
// piece t % 256, so a wavefront instruction reads one contiguous KiB of a page); with 512 threads
// the lower half of the workgroup takes pages {0,1} and the upper half pages {2,3}.  Block ids
// come from the tile descriptor (already in registers), so all data loads are issued back to back
// with no memory access in between, one tile ahead of their use (load), and are written to the
// LDS image later (store).
// Slots past the segment's end are staged as zeros so that stale or non-finite padding can never
// reach a product.
template <int NT, bool WITH_V>
struct Stager {
  static_assert(NT == 256 || NT == 512, "register-prefetch staging needs 256 or 512 threads");
  static constexpr int kPagesPerThread = 1024 / NT;          // 4 or 2 pages of each pool
  static constexpr int PER = kPagesPerThread * (WITH_V ? 2 : 1);
  uint4 reg[PER];
  const bf16_t* k_src;   // pool + head offset + this thread's piece
  const bf16_t* v_src;
  const bf16_t* v_src_shared;   // the same piece of a block of the shared value pool
  const int32_t* v_map;         // see value_block()
  size_t blk_stride;     // elements per block (all heads)
  int n_blocks, n_shared_blocks, in_page, pg0;

  __device__ __forceinline__ void init(const bf16_t* k_pool, const bf16_t* v_pool, int n_blocks_,
                                       int hkv, int kvh, int tid, const bf16_t* v_shared = nullptr,
                                       int n_shared_blocks_ = 0, const int32_t* v_map_ = nullptr) {
    v_map = v_map_;
    n_shared_blocks = n_shared_blocks_;
    v_src_shared = (WITH_V && v_shared != nullptr)
                       ? v_shared + static_cast<size_t>(kvh) * (kBlock * kD) + (tid & 255) * 8 : nullptr;
    in_page = tid & 255;
    pg0 = NT == 512 ? uniform(tid >> 8) * 2 : 0;             // first page this thread stages
    k_src = k_pool + static_cast<size_t>(kvh) * (kBlock * kD) + in_page * 8;
    v_src = WITH_V ? v_pool + static_cast<size_t>(kvh) * (kBlock * kD) + in_page * 8 : nullptr;
    blk_stride = static_cast<size_t>(hkv) * (kBlock * kD);
    n_blocks = n_blocks_;
  }

  // this thread's piece of the values that belong to key block blk (a valid block id)
  __device__ __forceinline__ const bf16_t* value_piece(int blk) const {
    if (v_map != nullptr) {
      const int m = uniform(v_map[blk]);
      if (m >= 0 && m < n_shared_blocks) return v_src_shared + static_cast<size_t>(m) * blk_stride;
    }
    return v_src + static_cast<size_t>(blk) * blk_stride;
  }

  __device__ __forceinline__ void load(const TileDesc& d) {
    const int nvalid = uniform(d.nvalid);
    int blk[kPagesPerThread];
    bool all_ok = nvalid == kTile;
#pragma unroll
    for (int j = 0; j < kPagesPerThread; ++j) {
      blk[j] = uniform(NT == 512 ? (pg0 ? d.blk[2 + j] : d.blk[j]) : d.blk[j]);
      all_ok = all_ok && blk[j] >= 0 && blk[j] < n_blocks;
    }
    if (all_ok) {                                            // whole tile present (wave-uniform)
#pragma unroll
      for (int j = 0; j < kPagesPerThread; ++j) {
        reg[j] = *reinterpret_cast<const uint4*>(k_src + static_cast<size_t>(blk[j]) * blk_stride);
        if constexpr (WITH_V)
          reg[kPagesPerThread + j] = *reinterpret_cast<const uint4*>(value_piece(blk[j]));
      }
      return;
    }
#pragma unroll
    for (int j = 0; j < kPagesPerThread; ++j) {
      const int pg = pg0 + j;
      const int nv = min(max(nvalid - kBlock * pg, 0), kBlock);
      const bool ok = nv > 0 && blk[j] >= 0 && blk[j] < n_blocks;
      uint4 kv = make_uint4(0u, 0u, 0u, 0u), vv = make_uint4(0u, 0u, 0u, 0u);
      if (ok) {
        if ((in_page >> 4) < nv)                             // token slot of this K piece
          kv = *reinterpret_cast<const uint4*>(k_src + static_cast<size_t>(blk[j]) * blk_stride);
        if constexpr (WITH_V) {
          vv = *reinterpret_cast<const uint4*>(value_piece(blk[j]));
          if (nv < kBlock) vv = zero_pad_slots(vv, in_page & 1, nv);
        }
      }
      reg[j] = kv;
      if constexpr (WITH_V) reg[kPagesPerThread + j] = vv;
    }
  }

  __device__ __forceinline__ void store(uint4* lds) const {
#pragma unroll
    for (int j = 0; j < kPagesPerThread; ++j) {
      lds[k_piece_dst(pg0 + j, in_page)] = reg[j];
      if constexpr (WITH_V) lds[v_piece_dst(pg0 + j, in_page)] = reg[kPagesPerThread + j];
    }
  }
};

// Cosines and sines of a query position's angles, times `scale`: rotation pairs i, i + 1 for the lower half of the
// wavefront, i + 8, i + 9 for the upper one.  i is wave-uniform, so that the frequencies come with scalar loads.
__device__ __forceinline__ float4 query_turn(const InvFreq& inv_freq, int pos, int i, int hh, float scale) {
  const double lo0 = inv_freq.f[i], lo1 = inv_freq.f[i + 1], hi0 = inv_freq.f[i + 8], hi1 = inv_freq.f[i + 9];
  float4 t;
  rot_cos_sin_fast(pos, hh ? hi0 : lo0, &t.x, &t.y);
  rot_cos_sin_fast(pos, hh ? hi1 : lo1, &t.z, &t.w);
  t.x *= scale; t.y *= scale; t.z *= scale; t.w *= scale;
  return t;
}
// The 32 query rows of a wavefront (row: the row of column lane % 32; one head), on their way into the lanes that
// multiply them.  Loaded as whole 256-byte rows, 16 lanes each: in the operand layout an instruction would ask for 32
// bytes of 32 rows, and the lines it touches, not the bytes, are what such loads cost.
__device__ __forceinline__ void load_query_rows(uint4 (&raw)[8], const bf16_t* __restrict__ q, int row, int hq, int h, int lane) {
#pragma unroll
  for (int i = 0; i < 8; ++i) {
    const int r = __shfl(row, 4 * i + (lane >> 4), 64);
    raw[i] = *reinterpret_cast<const uint4*>(q + (static_cast<size_t>(r) * hq + h) * kD + (lane & 15) * 8);
  }
}
// ... and regrouped through 8 KiB of LDS of the wavefront's own into operands of W = 32 or 16 columns: afterwards raw[k] holds dims
// 16k + 8 (lane / 32) .. + 7 of column lane % 32, or dims 32 (k % 4) + 8 (lane / 16) .. + 7 of column 16 (k / 4) + lane % 16 (pieces
// of a row are permuted by its number, so that neither side meets a bank conflict)
template <int W = 32>
__device__ __forceinline__ void regroup_query_rows(uint4 (&raw)[8], char* own, int lane) {
#pragma unroll
  for (int i = 0; i < 8; ++i) {
    const int r = 4 * i + (lane >> 4);
    *reinterpret_cast<uint4*>(own + r * 256 + (((lane & 15) ^ (r & 15)) << 4)) = raw[i];
  }
  asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");        // (other lanes' pieces: an order the compiler does not see)
#pragma unroll
  for (int k = 0; k < 8; ++k) {
    const int r = W == 32 ? lane & 31 : 16 * (k >> 2) + (lane & 15), piece = W == 32 ? 2 * k + (lane >> 5) : 4 * (k & 3) + (lane >> 4);
    raw[k] = *reinterpret_cast<const uint4*>(own + r * 256 + ((piece ^ (r & 15)) << 4));
  }
  asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
}
// two bf16 pairs (x, y) packed in a word each, turned by the two angles of t
__device__ __forceinline__ void turn_words(uint32_t& x, uint32_t& y, const float4& t) {
  const float x0 = __uint_as_float(x << 16), x1 = __uint_as_float(x & 0xffff0000u);
  const float y0 = __uint_as_float(y << 16), y1 = __uint_as_float(y & 0xffff0000u);
  const float a0 = x0 * t.x - y0 * t.y, a1 = x1 * t.z - y1 * t.w, b0 = y0 * t.x + x0 * t.y, b1 = y1 * t.z + x1 * t.w;
  asm("v_cvt_pk_bf16_f32 %0, %1, %2" : "=v"(x) : "v"(a0), "v"(a1));
  asm("v_cvt_pk_bf16_f32 %0, %1, %2" : "=v"(y) : "v"(b0), "v"(b1));
}

__device__ __forceinline__ float max16(const f32x16& v) {
  float a = fmaxf(fmaxf(v[0], v[1]), fmaxf(v[2], v[3]));
  float b = fmaxf(fmaxf(v[4], v[5]), fmaxf(v[6], v[7]));
  float c = fmaxf(fmaxf(v[8], v[9]), fmaxf(v[10], v[11]));
  float d = fmaxf(fmaxf(v[12], v[13]), fmaxf(v[14], v[15]));
  return fmaxf(fmaxf(a, b), fmaxf(c, d));
}

__device__ __forceinline__ f32x16 splat16(float v) {
  f32x16 r;
#pragma unroll
  for (int i = 0; i < 16; ++i) r[i] = v;
  return r;
}


}  // namespace tile

// ---- tile plan (built by plan kernels on the stream, kept in the caller's workspace) ----------
// What a workgroup of the wide attention kernel needs of a request.
struct WorkItem {
  int32_t row, n_rows;       // its rows of the query list
  int32_t j_begin, j_end;    // its key tiles
  int32_t pad[4];
};
static_assert(sizeof(WorkItem) == 32, "room for two 16-byte vectors");

// List of workgroups in the order they start: entry i sits in tiles[i].work - request << tile_bits | row tile of it - and the
// number of entries in tiles[max_tiles - 1].work.  Rows: the scored tokens of a request (numbered through over its
// chunks) or its rows of the query list.
struct WorkList {
  enum Kind { kNone, kScored, kQueries } kind = kNone;
  int rows = 0;                     // rows of a workgroup
  int tile_bits = 0;                // bits of an entry that name the row tile
  int places = 0;                   // workgroups of one head group that run at a time
  const int32_t* q_pos = nullptr;   // kQueries: position of every row
};
constexpr int kMaxOrdered = 4096;      // segments or requests that are sorted for the dispatch order
constexpr int kMaxSorted = 512;       // requests whose workgroups are sorted (more: scores request by request, attention without a list)
constexpr int kMaxSortedTiles = 2048;  // row tiles that are sorted
// What the requests leave of an entry's 32 bits, and whether that names as many row tiles of one request.  (With half of the bits for
// each, calls of more than 4.2 M tokens had no list, however short their requests: 2100 of 4 x 500 tokens on 32 / 8 heads 40.9 ms, now 35.4.)
inline int list_tile_bits(int n_requests) {
  int bits = 31;
  while (bits > 0 && (n_requests - 1) >> (32 - bits) != 0) --bits;
  return bits;
}
inline bool list_can_name(int n_requests, int row_tiles) { return row_tiles <= static_cast<int64_t>(1) << list_tile_bits(n_requests); }
struct Plan { int32_t* seg_tile_off; int32_t* order; WorkItem* items; tile::TileDesc* tiles; int max_tiles; int32_t* redo; int redo_any; };      // redo[redo_any]: whether any flag is set
size_t plan_head_bytes(int n_segs);
// by_request: dispatch order over requests (attention; cu_q delimits their rows), else over segments (score; none where a list is made).
// list: the list of workgroups to build beside it.  scatter: a scatter to run beside it (attention), or null.
// n_redo > 0: the plan also holds n_redo redo flags (after the tiles), cleared by the plan kernels.
Plan run_plan(const cc_ctx* ctx, void* ws, const cc_segment* segs, int n_segs, const int32_t* req_seg_off, int n_requests, bool by_request,
              const int32_t* cu_q, const int32_t* block_tab, int n_blocks, int max_tiles, int n_redo, const WorkList& list,
              const ScatterJob* scatter, hipStream_t stream);

// The wide attention kernel (64 query rows per workgroup, 32 in two key streams) keeps one softmax reference per row; rows
// whose sums leave the safe range are flagged in redo[] and redone by the narrow kernel, which can
// move its reference.  q0 is the first row of the 64-row tile (the request's first row + 64 k);
// two tiles of different requests may share an entry, which only costs a spurious redo.
__host__ __device__ inline int redo_index(int q0) { return q0 >> 5; }
// (the last entry is no row's: it says whether any flag is set, so that a second pass with nothing to do reads one word and leaves)
inline size_t redo_entries(int n_q_tot) { return static_cast<size_t>(n_q_tot) / 32 + 2; }

void launch_attn_v2(const cc_ctx* ctx, const void* q, const int32_t* q_pos,
                    int n_q_tot, int max_q_per_req, const void* k_pool, const void* v_pool,
                    const Plan& pl, const int32_t* req_seg_off, int n_requests, void* out, float* lse,
                    int32_t* redo, const int32_t* q_map, int map_pos, const int32_t* snap_index, float* cum,
                    int s_max, const WorkList& list, hipStream_t stream, const ValueSource& vs);
// its list of workgroups (kNone where there is none); q_pos: by list row, or null
WorkList attn_v2_list(const cc_ctx* ctx, const int32_t* q_pos, int n_q_tot, int max_q_per_req, int n_requests, int max_tiles);

// The wide score kernel (128 tokens per wavefront, no softmax reference) flags 64-row granules of
// the per-token tensors whose sums left the safe range; the narrow kernel redoes them.
inline size_t score_redo_entries(int n_tok) { return static_cast<size_t>(n_tok) / 64 + 2; }
// 64 tokens and two key streams; 128 tokens in products of 32 columns; of 16
enum class ScoreForm { kSmall, kBig, kBig16 };
void launch_score_v2(const cc_ctx* ctx, const void* q, const void* k_pool, const Plan& pl, const cc_segment* segs,
                     const int32_t* req_seg_off, int n_requests, int n_tok, float* mass, int32_t* redo, ScoreForm form,
                     const WorkList& list, hipStream_t stream);

}  // namespace cc
