// cc_qkv_project: [q | k | v] = x W^T for the chosen tokens only (Sec. 3.4.3), and the other dense
// products of a decoder layer for the recomputed rows (Sec. 2.1, Sec. 3.4.3): y = x W^T (+ residual)
// and the feed-forward input silu(x W_gate^T) * (x W_up^T).
//
// x [n_rows][hidden], W [features][hidden]: both operands have the contraction index contiguous.
// bf16: MFMA GEMMs on the transposed product D^T = W x^T, in which a lane holds consecutive features of
// ONE token and writes 16-byte pieces of an output row; the products differ in their epilogue and in
// the rows of W a workgroup stages.  fp32 (and odd shapes): plain LDS-tiled kernels.
#include <type_traits>

#include "device_util.h"

namespace cc {

// what a GEMM kernel does with its accumulators
enum { kOutQkv = 0, kOutLinear = 1, kOutGated = 2 };
struct GemmOut {
  void *o0, *o1, *o2;          // qkv: q, k, v; linear / gated: y in o0
  const void* residual;        // linear: added to the product (may be y itself), or null
  int nq, nk;                  // qkv: widths of q and of k (= v)
  int width;                   // linear / gated: features of y
};

template <typename T>
__device__ __forceinline__ void store_qkv(float v, int row, int col, int nq, int nk, T* q, T* k, T* vv) {
  if (col < nq) q[static_cast<size_t>(row) * nq + col] = from_float<T>(v);
  else if (col < nq + nk) k[static_cast<size_t>(row) * nk + (col - nq)] = from_float<T>(v);
  else vv[static_cast<size_t>(row) * nk + (col - nq - nk)] = from_float<T>(v);
}

// ---- plain kernel (any dtype): 64x64 tile, 256 threads, 4x4 outputs per thread ----------------
template <typename T>
__global__ __launch_bounds__(256) void qkv_project_plain_kernel(
    const T* __restrict__ x, const T* __restrict__ w, int n_rows, int hidden, int n_cols, int nq,
    int nk, T* __restrict__ q, T* __restrict__ k, T* __restrict__ v) {
  __shared__ float xs[16][64 + 1];
  __shared__ float ws[16][64 + 1];
  const int tx = threadIdx.x % 16, ty = threadIdx.x / 16;
  const int row0 = blockIdx.y * 64, col0 = blockIdx.x * 64;
  float acc[4][4] = {};
  for (int k0 = 0; k0 < hidden; k0 += 16) {
    for (int i = threadIdx.x; i < 64 * 16; i += 256) {
      const int r = i / 16, kk = i % 16;
      xs[kk][r] = (row0 + r < n_rows) ? to_float(x[static_cast<size_t>(row0 + r) * hidden + k0 + kk]) : 0.f;
      ws[kk][r] = (col0 + r < n_cols) ? to_float(w[static_cast<size_t>(col0 + r) * hidden + k0 + kk]) : 0.f;
    }
    __syncthreads();
#pragma unroll
    for (int kk = 0; kk < 16; ++kk) {
      float a[4], b[4];
#pragma unroll
      for (int i = 0; i < 4; ++i) { a[i] = xs[kk][ty * 4 + i]; b[i] = ws[kk][tx * 4 + i]; }
#pragma unroll
      for (int i = 0; i < 4; ++i)
#pragma unroll
        for (int j = 0; j < 4; ++j) acc[i][j] += a[i] * b[j];
    }
    __syncthreads();
  }
  for (int i = 0; i < 4; ++i)
    for (int j = 0; j < 4; ++j) {
      const int r = row0 + ty * 4 + i, c = col0 + tx * 4 + j;
      if (r < n_rows && c < n_cols) store_qkv<T>(acc[i][j], r, c, nq, nk, q, k, v);
    }
}

// ---- plain kernels of y = x W^T (+ residual) and of the gated feed-forward input ------------------
template <typename T, bool GATED>
__global__ __launch_bounds__(256) void linear_plain_kernel(
    const T* __restrict__ x, const T* __restrict__ w, const T* __restrict__ w2, const T* residual,
    int n_rows, int n_in, int n_out, T* y) {                      // (residual may be y itself)
  __shared__ float xs[16][64 + 1];
  __shared__ float ws[16][64 + 1];
  __shared__ float us[GATED ? 16 : 1][64 + 1];
  const int tx = threadIdx.x % 16, ty = threadIdx.x / 16;
  const int row0 = blockIdx.y * 64, col0 = blockIdx.x * 64;
  float acc[4][4] = {}, acc2[4][4] = {};
  for (int k0 = 0; k0 < n_in; k0 += 16) {
    for (int i = threadIdx.x; i < 64 * 16; i += 256) {
      const int r = i / 16, kk = i % 16;
      const bool kin = k0 + kk < n_in;
      xs[kk][r] = (kin && row0 + r < n_rows) ? to_float(x[static_cast<size_t>(row0 + r) * n_in + k0 + kk]) : 0.f;
      ws[kk][r] = (kin && col0 + r < n_out) ? to_float(w[static_cast<size_t>(col0 + r) * n_in + k0 + kk]) : 0.f;
      if (GATED) us[kk][r] = (kin && col0 + r < n_out) ? to_float(w2[static_cast<size_t>(col0 + r) * n_in + k0 + kk]) : 0.f;
    }
    __syncthreads();
#pragma unroll
    for (int kk = 0; kk < 16; ++kk) {
      float a[4], b[4], c[4];
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        a[i] = xs[kk][ty * 4 + i];
        b[i] = ws[kk][tx * 4 + i];
        c[i] = GATED ? us[kk][tx * 4 + i] : 0.f;
      }
#pragma unroll
      for (int i = 0; i < 4; ++i)
#pragma unroll
        for (int j = 0; j < 4; ++j) {
          acc[i][j] += a[i] * b[j];
          if (GATED) acc2[i][j] += a[i] * c[j];
        }
    }
    __syncthreads();
  }
  for (int i = 0; i < 4; ++i)
    for (int j = 0; j < 4; ++j) {
      const int r = row0 + ty * 4 + i, c = col0 + tx * 4 + j;
      if (r >= n_rows || c >= n_out) continue;
      const size_t at = static_cast<size_t>(r) * n_out + c;
      float v = acc[i][j];
      if (GATED) v = v / (1.f + expf(-v)) * acc2[i][j];
      else if (residual != nullptr) v += to_float(residual[at]);
      y[at] = from_float<T>(v);
    }
}

// ---- MFMA kernel (bf16) -----------------------------------------------------------------------
namespace {

typedef __attribute__((__vector_size__(4 * sizeof(uint32_t)))) uint32_t u32x4;

// 64 lanes x 16 bytes from global memory straight into LDS: lane L's 16 bytes land at lds_addr + 16 L,
// read from base + voff(L)
__device__ __forceinline__ void gemm_load_to_lds(const char* base, uint32_t voff, uint32_t lds_addr) {
  asm volatile("s_mov_b32 m0, %2\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %0, %1" :: "v"(voff), "s"(base), "s"(lds_addr) : "memory", "m0");
}
__device__ __forceinline__ void gemm_mfma(f32x4& d, const u32x4& a, const u32x4& b) {
  asm volatile("v_mfma_f32_16x16x32_bf16 %0, %1, %2, %0" : "+a"(d) : "v"(a), "v"(b));
}

// Both GEMM kernels below share the following.
//
// v_mfma_f32_16x16x32_bf16, not 32x32x16: under matrix load the chip is held by its power budget, and this
// shape moves half the accumulator bytes per flop (MFMAs and barriers alone, everything else taken
// out of the loop: 1.9 PFLOP/s against 1.48; the whole product 1.30 against 1.17 at 4096 x 4096 x 14336).
//
// Operands go straight from global memory into LDS (global_load_lds: lane L of an instruction fills
// piece base + L), whole cache lines per load: a line of 128 bytes is 64 contraction indices of one row of W
// or x, 8 consecutive lanes share it (8 rows per instruction), and the image in LDS is row-major, 128 bytes
// per row.  Operand reads walk down 16 rows at one 16-byte piece, so piece c of row r is kept at
// c ^ swizzle(r), which spreads any such walk over all banks (0 conflicts); the permutation is
// applied on the global side (lane -> piece of the line), because the load fixes where a lane's bytes land.
//
// MFMA row m of the half i2 of a 32-feature block is feature 8 (m / 4) + 4 i2 + m % 4, so that the two halves give
// a lane 8 consecutive features of a token: one 16-byte store.
constexpr int kTK = 64;                               // contraction indices in a cache line
__device__ __forceinline__ int gemm_swz_w(int r) { return ((r >> 1) & 1) | ((r >> 2) & 6); }   // (rows 8 (m / 4) + m % 4)
__device__ __forceinline__ int gemm_swz_x(int r) { return (r >> 1) & 7; }                        // (rows m)

// gated: of a wavefront's FB 32-feature blocks the first half are rows of W_gate and the second half the SAME
// rows of W_up, so that a lane ends up holding both factors of an output

// the residual's 8 values that belong to 8 consecutive features of one token (asking for a 256 x
// 256 tile's residual ahead of its stores spills registers and gains nothing: all workgroups store at once, bound by bytes)
template <int MODE>
__device__ __forceinline__ uint4 gemm_residual8(const GemmOut& out, int row, int col) {
  if (MODE != kOutLinear || out.residual == nullptr) return make_uint4(0u, 0u, 0u, 0u);
  return *reinterpret_cast<const uint4*>(static_cast<const bf16_t*>(out.residual) + static_cast<size_t>(row) * out.width + col);
}

// stores 8 consecutive features of one token
template <int MODE>
__device__ __forceinline__ void gemm_store8(const f32x4& lo, const f32x4& hi, const f32x4& up_lo, const f32x4& up_hi,
                                            const uint4& residual, const GemmOut& out, int row, int col) {
  bf16_t* base;
  int c_in = col, width;                              // (32 features never straddle q | k | v)
  if (MODE != kOutQkv) { base = static_cast<bf16_t*>(out.o0); width = out.width; }
  else if (col < out.nq) { base = static_cast<bf16_t*>(out.o0); width = out.nq; }
  else if (col < out.nq + out.nk) { base = static_cast<bf16_t*>(out.o1); c_in = col - out.nq; width = out.nk; }
  else { base = static_cast<bf16_t*>(out.o2); c_in = col - out.nq - out.nk; width = out.nk; }
  const size_t at = static_cast<size_t>(row) * width + c_in;
  float v[8];
#pragma unroll
  for (int e = 0; e < 8; ++e) v[e] = e < 4 ? lo[e & 3] : hi[e & 3];
  if (MODE == kOutGated) {
#pragma unroll
    for (int e = 0; e < 8; ++e) v[e] = v[e] / (1.f + __expf(-v[e])) * (e < 4 ? up_lo[e & 3] : up_hi[e & 3]);
  }
  if (MODE == kOutLinear && out.residual != nullptr) {
    const bf16x8 r = __builtin_bit_cast(bf16x8, residual);
#pragma unroll
    for (int e = 0; e < 8; ++e) v[e] += static_cast<float>(r[e]);
  }
  bf16x8 o;
#pragma unroll
  for (int e = 0; e < 8; ++e) o[e] = static_cast<bf16_t>(v[e]);
  *reinterpret_cast<uint4*>(base + at) = __builtin_bit_cast(uint4, o);
}

// Which tile a workgroup takes: workgroups are handed to the 8 XCDs in turn, each XCD with an L2 of
// its own.  Workgroup L therefore takes entry (L % 8) * per_xcd + L / 8 of a tile order in which 32
// consecutive entries (what one XCD runs at a time) form a block of 4 feature tiles x 8 token tiles: the
// block's 32 workgroups ask their L2 for 12 different operand panels instead of up to 34.  (The plain order
// is 0 - 5 % slower, on gated products of 2 x 28672 features 25 %: 9000 rows 7.85 / 6.02 ms; 8 x 4 and 2 x 16 blocks
// measure the same.)
constexpr int kBlockN = 4, kBlockM = 8;
// With the contraction in parts the order runs through all tiles of a part before the next one.
__device__ __forceinline__ bool gemm_tile_of(int tiles_n, int tiles_m, int n_parts, int* tn, int* tm, int* part) {
  int entry = (blockIdx.x & 7) * (gridDim.x >> 3) + (blockIdx.x >> 3);
  if (entry >= tiles_n * tiles_m * n_parts) return false;  // (the grid is padded to a multiple of 8)
  *part = entry / (tiles_n * tiles_m);
  entry -= *part * (tiles_n * tiles_m);
  const int strip = min(entry / (kBlockN * tiles_m), (tiles_n - 1) / kBlockN);   // strip of up to 4 feature tiles
  const int strip_w = min(kBlockN, tiles_n - strip * kBlockN);
  const int in_strip = entry - strip * kBlockN * tiles_m;
  const int blk = in_strip / (strip_w * kBlockM), in_blk = in_strip - blk * strip_w * kBlockM;
  *tn = strip * kBlockN + in_blk % strip_w;
  *tm = blk * kBlockM + in_blk / strip_w;
  return true;
}

// A contraction in parts (SPLIT): the workgroups of a tile each take a range of its stages and write what their
// accumulators hold, in fp32 and in the accumulators' own order (a store instruction fills 1 KiB), to the caller's workspace;
// gemm_sum_kernel adds the parts in their order and does what the epilogue would have done.  Block (token block, feature
// block) of part p: 2 KiB at ((p n_tb + token block) n_fb + feature block).
struct GemmParts {
  f32x4* sums;                 // null: the contraction is not split
  int n, n_tb, n_fb;           // parts; 16-token blocks (of whole tiles) and 32-feature blocks of the product
};
__device__ __forceinline__ void gemm_store_part(const GemmParts& parts, int part, int tb, int fb, int lane, const f32x4& lo, const f32x4& hi) {
  f32x4* to = parts.sums + ((static_cast<size_t>(part) * parts.n_tb + tb) * parts.n_fb + fb) * 128;        // (wave-uniform)
  to[lane] = lo;
  to[64 + lane] = hi;
  __builtin_amdgcn_sched_barrier(0);                      // (one block's registers at a time)
}

template <int N>
__device__ __forceinline__ void gemm_wait_loads() {       // at most N of this wavefront's loads outstanding
  __builtin_amdgcn_s_waitcnt((N & 15) | ((N >> 4) << 14) | (7 << 4) | (15 << 8));
  asm volatile("" ::: "memory");
}
__device__ __forceinline__ void gemm_wait_lds() { __builtin_amdgcn_s_waitcnt(15 | (3 << 14) | (7 << 4) | (0 << 8)); }
__device__ __forceinline__ void gemm_barrier() {
  asm volatile("" ::: "memory");
  __builtin_amdgcn_s_barrier();
  asm volatile("" ::: "memory");
}

// The kernel for short lists and remainders: any tile of FB x TB blocks (32 features, 16 tokens) per
// wavefront, WF x WM wavefronts across the tile times WK along the contraction (each takes its share of a
// stage's k-steps and the partial sums meet in LDS at the end: more wavefronts per tile without more operand
// reads).  A stage is U cache lines of every row; NBUF stages are buffered, one barrier per stage, in front of
// its last k-step, whose operands are in registers by then: behind it the next stage is readable and this stage's
// buffer can be refilled.
// Bound by what a compute unit's L1 delivers: about half of its 64 bytes per clock with the 64 x 128 tile (the
// lines in flight are bounded, so the rate is that bound over the latency of the level the lines come
// from), whatever the number of buffers or wavefronts.  A list of 449 rows against the 256 x 256 tile:
// 4096 x 4096 101 -> 23 us, 4096 x 14336 354 -> 79 us, 6144 x 4096 106 -> 35 us.
template <int MODE, bool SPLIT, int FB, int TB, int WF, int WM, int WK, int U, int NBUF>
__global__ __launch_bounds__(64 * WF * WM * WK, (WF * WM * WK * 2 <= 8 && 2 * NBUF * U * (32 * FB * WF + 16 * TB * WM) * 128 <= 163840) ? 2 : 1) void gemm_tile_kernel(
    const bf16_t* __restrict__ x, const bf16_t* __restrict__ w, const bf16_t* __restrict__ w2, int n_rows,
    int hidden, int tiles_n, int tiles_m, GemmOut out, GemmParts parts) {
  constexpr int NW = WF * WM * WK;                    // wavefronts
  constexpr int F = 32 * FB * WF, M = 16 * TB * WM;   // features x tokens of the tile
  constexpr int PW = U * (F + M) / 8 / NW;            // load instructions of a wavefront per stage
  constexpr int kSub = (F + M) * kTK * 2, kStage = U * kSub;
  constexpr int S = 2 * U / WK;                       // 32-wide k-steps of a stage a wavefront multiplies
  static_assert((U * (F + M)) % (8 * NW) == 0 && (2 * U) % WK == 0, "stage must divide over the wavefronts");
  static_assert(MODE != kOutGated || FB % 2 == 0, "a wavefront holds gate and up rows of the same outputs");
  static_assert(!SPLIT || MODE == kOutLinear, "a part's epilogue knows no outputs; gated products are not split");
  __shared__ uint4 lds[NBUF * kStage / 16];
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int nl = lane & 15, g = lane >> 4;
  const int wk = wave % WK, wn = (wave / WK) % WF, wm = wave / (WK * WF);
  int n0, m0, part;
  if (!gemm_tile_of(tiles_n, tiles_m, SPLIT ? parts.n : 1, &n0, &m0, &part)) return;
  n0 *= F;
  m0 *= M;
  const int n_k_all = hidden / (kTK * U), k_first = SPLIT ? n_k_all * part / parts.n : 0;      // this part's stages: k_first .. + n_k - 1
  const int n_k = SPLIT ? n_k_all * (part + 1) / parts.n - k_first : n_k_all;
  __builtin_assume(!SPLIT || n_k > 0);

  // ---- staging: image rows 0..F-1 are W, F..F+M-1 are x; wavefront w brings groups PW w .. of 8 rows: lane L
  // -> row 8 j + L / 8, LDS piece L % 8 of that row
  const char* base[PW];                                    // (wave-uniform)
  uint32_t voff[PW];
#pragma unroll
  for (int j = 0; j < PW; ++j) {
    const int grp8 = PW * wave + j, sub = grp8 / ((F + M) / 8);
    const int r0 = 8 * (grp8 % ((F + M) / 8)), r = r0 + (lane >> 3);
    int off_row;
    if (r0 >= F) {
      base[j] = reinterpret_cast<const char*>(x + static_cast<size_t>(m0) * hidden);
      off_row = min(r - F, n_rows - 1 - m0);
    } else if (MODE != kOutGated) {
      base[j] = reinterpret_cast<const char*>(w + static_cast<size_t>(n0) * hidden);
      off_row = r;
    } else {
      const int blk = r0 >> 5, grp = blk / FB, in = blk % FB;
      base[j] = reinterpret_cast<const char*>((in >= FB / 2 ? w2 : w) + static_cast<size_t>(n0 / 2) * hidden);
      off_row = 32 * (grp * (FB / 2) + in % (FB / 2)) + (r & 31);
    }
    base[j] += (k_first * U + sub) * (kTK * 2);
    voff[j] = static_cast<uint32_t>(off_row) * static_cast<uint32_t>(hidden * 2) +
              16 * ((lane & 7) ^ (r0 >= F ? gemm_swz_x(r - F) : gemm_swz_w(r)));
  }
  typedef __attribute__((address_space(3))) const uint4 lds_piece;
  const uint32_t lds_base = __builtin_amdgcn_readfirstlane(static_cast<uint32_t>(reinterpret_cast<uintptr_t>((lds_piece*)lds)));
  // load j of stage t into buffer b (past the last stage: a harmless repeat into a buffer nobody reads any more)
  auto dma_one = [&](int t, int b, int j) __attribute__((always_inline)) {
    gemm_load_to_lds(base[j] + static_cast<size_t>(min(t, n_k - 1)) * (kTK * 2 * U), voff[j], lds_base + b * kStage + (PW * wave + j) * 1024);
  };

  // block (a, i2, b): features 32 a + 8 (m / 4) + 4 i2 + m % 4 of MFMA row m, tokens 16 b + n: a lane ends up with 8
  // consecutive features of a token in the two halves i2
  f32x4 acc[FB][2][TB];
#pragma unroll
  for (int a = 0; a < FB; ++a)
#pragma unroll
    for (int i2 = 0; i2 < 2; ++i2)
#pragma unroll
      for (int b = 0; b < TB; ++b)
#pragma unroll
        for (int i = 0; i < 4; ++i) asm volatile("v_accvgpr_write_b32 %0, 0" : "=a"(acc[a][i2][b][i]));

  const char* lds_bytes = reinterpret_cast<const char*>(lds);
  const int r_w = 8 * (nl >> 2) + (nl & 3), r_x = nl;      // (block bases are multiples of 32 / 16 rows; +4 leaves swz_w alone)
  const int row_w = (32 * FB * wn + r_w) * 128, row_x = (F + 16 * TB * wm + r_x) * 128;
  u32x4 opa[2][FB][2], opb[2][TB];
  auto read_step = [&](int set, int buf, int s) __attribute__((always_inline)) {       // s: the wavefront's step
    const int step = s * WK + wk, c = 4 * (step & 1) + g;
    const char* pw = lds_bytes + buf * kStage + (step >> 1) * kSub + row_w + ((c ^ gemm_swz_w(r_w)) << 4);
    const char* px = lds_bytes + buf * kStage + (step >> 1) * kSub + row_x + ((c ^ gemm_swz_x(r_x)) << 4);
#pragma unroll
    for (int b = 0; b < TB; ++b) opb[set][b] = *reinterpret_cast<const u32x4*>(px + b * 2048);
#pragma unroll
    for (int a = 0; a < FB; ++a)
#pragma unroll
      for (int i2 = 0; i2 < 2; ++i2) opa[set][a][i2] = *reinterpret_cast<const u32x4*>(pw + a * 4096 + i2 * 512);
  };

#pragma unroll
  for (int t = 0; t < NBUF; ++t)
#pragma unroll
    for (int j = 0; j < PW; ++j) dma_one(t, t, j);
  gemm_wait_loads<(NBUF - 1) * PW>();
  gemm_barrier();
  read_step(0, 0, 0);
  int buf = 0;
  // one stage; PAR: operand set of its first step
  auto stage = [&](int t, auto par) __attribute__((always_inline)) {
    constexpr int P0 = decltype(par)::value;
    const int nbuf = buf + 1 == NBUF ? 0 : buf + 1;
#pragma unroll
    for (int s = 0; s < S; ++s) {
      const int cur = (P0 + s) & 1, nxt = cur ^ 1;
      if (s == S - 1) {
        // this wavefront's last operands of the stage are in registers and its loads of stage t+1 have
        // landed; behind the barrier the whole stage t+1 can be read and buffer t refilled
        gemm_wait_loads<(NBUF - 2) * PW>();
        gemm_wait_lds();
        gemm_barrier();
        read_step(nxt, nbuf, 0);
      } else {
        read_step(nxt, buf, s + 1);
      }
      __builtin_amdgcn_sched_barrier(0);
      // (the refill's loads go out between the MFMAs of this step)
      constexpr int kSlots = FB * 2 * TB, kPer = (PW + kSlots - 1) / kSlots, kEvery = PW >= kSlots ? 1 : kSlots / PW;
#pragma unroll
      for (int a = 0; a < FB; ++a)
#pragma unroll
        for (int i2 = 0; i2 < 2; ++i2)
#pragma unroll
          for (int b = 0; b < TB; ++b) {
            gemm_mfma(acc[a][i2][b], opa[cur][a][i2], opb[cur][b]);
            if (s == S - 1) {
#pragma unroll
              for (int u = 0; u < kPer; ++u) {
                const int m = (a * 2 + i2) * TB + b, j = (m / kEvery) * kPer + u;
                if (m % kEvery == 0 && j < PW) dma_one(t + NBUF, buf, j);
              }
            }
          }
      __builtin_amdgcn_sched_barrier(0);
    }
    buf = nbuf;
  };
  if constexpr (S % 2 == 0) {
    for (int t = 0; t < n_k; ++t) stage(t, std::integral_constant<int, 0>{});
  } else {
    for (int t = 0; t < n_k; t += 2) {
      stage(t, std::integral_constant<int, 0>{});
      if (t + 1 < n_k) stage(t + 1, std::integral_constant<int, 1>{});
    }
  }
  gemm_wait_loads<0>();            // (nothing may still be landing when the LDS is given back)
  asm volatile("s_nop 15\n\ts_nop 15" ::: "memory");

  const int tok0 = m0 + 16 * TB * wm + nl;
  const int col0 = (MODE == kOutGated ? n0 / 2 + 32 * (FB / 2) * wn : n0 + 32 * FB * wn) + 8 * g;
  constexpr int FO = MODE == kOutGated ? FB / 2 : FB;      // 32-feature blocks of outputs
  if constexpr (WK > 1) {
    // the WK wavefronts of a tile hold partial sums over their k-steps: they exchange token blocks through LDS
    // and each finishes TB / WK of them
    constexpr int H = TB / WK, kBlk = FB * 2 * H;          // token blocks, 1 KiB pieces a wavefront gets from each other one
    static_assert(TB % WK == 0, "token blocks are shared out");
    static_assert(WF * WM * WK * WK * kBlk * 1024 <= NBUF * kStage, "partial sums must fit");
    __syncthreads();
    f32x4* share = reinterpret_cast<f32x4*>(lds) + (wave / WK) * (WK * WK * kBlk * 64) + lane;
#pragma unroll
    for (int k = 0; k < WK; ++k)
#pragma unroll
      for (int a = 0; a < FB; ++a)
#pragma unroll
        for (int i2 = 0; i2 < 2; ++i2)
#pragma unroll
          for (int b = 0; b < H; ++b)
            if (k != wk) share[((k * WK + wk) * kBlk + (a * 2 + i2) * H + b) * 64] = acc[a][i2][k * H + b];
    uint4 res[H][FO];
#pragma unroll
    for (int b = 0; b < H; ++b)
#pragma unroll
      for (int a = 0; a < FO; ++a) if (!SPLIT) res[b][a] = gemm_residual8<MODE>(out, min(tok0 + 16 * (wk * H + b), n_rows - 1), col0 + 32 * a);
    __syncthreads();
#pragma unroll
    for (int b = 0; b < H; ++b) {
      f32x4 sum[FB][2];
#pragma unroll
      for (int a = 0; a < FB; ++a)
#pragma unroll
        for (int i2 = 0; i2 < 2; ++i2) {
          f32x4 v = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
          for (int k = 0; k < WK; ++k) {                   // (summed in the order of k whatever the wavefront)
            f32x4 part;
            if (k == wk) {
              part = acc[a][i2][b];
#pragma unroll
              for (int o = 1; o < WK; ++o) if (wk == o) part = acc[a][i2][o * H + b];
            } else {
              part = share[((wk * WK + k) * kBlk + (a * 2 + i2) * H + b) * 64];
            }
            v += part;
          }
          sum[a][i2] = v;
        }
      if constexpr (SPLIT) {
#pragma unroll
        for (int a = 0; a < FB; ++a)
          gemm_store_part(parts, part, m0 / 16 + TB * wm + wk * H + b, n0 / 32 + FB * wn + a, lane, sum[a][0], sum[a][1]);
        continue;
      }
      const int row = tok0 + 16 * (wk * H + b);
      if (row < n_rows) {
#pragma unroll
        for (int a = 0; a < FO; ++a)
          gemm_store8<MODE>(sum[a][0], sum[a][1], sum[FB - FO + a][0], sum[FB - FO + a][1], res[b][a], out, row, col0 + 32 * a);
      }
    }
  } else if constexpr (SPLIT) {
#pragma unroll
    for (int b = 0; b < TB; ++b)
#pragma unroll
      for (int a = 0; a < FB; ++a)
        gemm_store_part(parts, part, m0 / 16 + TB * wm + b, n0 / 32 + FB * wn + a, lane, acc[a][0][b], acc[a][1][b]);
  } else {
#pragma unroll
    for (int b = 0; b < TB; ++b) {
      const int row = tok0 + 16 * b;
      if (row >= n_rows) continue;
#pragma unroll
      for (int a = 0; a < FO; ++a)
        gemm_store8<MODE>(acc[a][0][b], acc[a][1][b], acc[FB - FO + a][0][b], acc[FB - FO + a][1][b],
                          gemm_residual8<MODE>(out, row, col0 + 32 * a), out, row, col0 + 32 * a);
    }
  }
}

// The kernel for long lists: 256 features x 256 tokens, 8 wavefronts of 128 x 64 (two per SIMD), 12 operand reads
// feed 32 MFMAs.  A stage is one cache line of every row, W and x in buffers of 32 KiB each; five of them
// fill the LDS, so that W of stage t+2 starts landing when stage t begins (two stages ahead) and x of
// stage t+2 right behind the barrier that frees W of stage t (one stage ahead).  A wavefront keeps one set of
// W operands and rolls it: as soon as a half-block has met the step's four token blocks its registers take
// the next step's piece, which spreads the LDS reads over the MFMAs and leaves room for two wavefronts per SIMD.
// One barrier per stage, behind the first kMeet half-blocks of its second step.
// 1.37 - 1.40 PFLOP/s in full rounds of tiles (the 32x32x16 form with four wavefronts of 128 x 128: 1.15 - 1.24):
// 13 824 rows x 4096 x 14336 1.58 -> 1.28 ms, gated 4096 -> 2 x 14336 2.60 -> 2.37 ms.  What is left: loads from
// beyond the L2 cost 12 % (measured with the stages repeated), the loads themselves 10 %, operand reads 9 %.
template <int MODE, bool SPLIT>
__global__ __launch_bounds__(512, 2) void gemm_kernel(
    const bf16_t* __restrict__ x, const bf16_t* __restrict__ w, const bf16_t* __restrict__ w2, int n_rows,
    int hidden, int tiles_n, int tiles_m, GemmOut out, GemmParts parts) {
  constexpr int F = 256, M = 256, FB = 4, TB = 4, WF = 2;
  constexpr int kHalf = 32768, kSlots = 5;             // bytes and number of the half-stage buffers
  constexpr int kMeet = 2;                             // feature half-blocks of the second step in front of the barrier (1 or 3: the same)
  __shared__ uint4 lds[kSlots * kHalf / 16];
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int nl = lane & 15, g = lane >> 4;
  const int wn = wave % WF, wm = wave / WF;
  int n0, m0, part;
  if (!gemm_tile_of(tiles_n, tiles_m, SPLIT ? parts.n : 1, &n0, &m0, &part)) return;
  n0 *= F;
  m0 *= M;
  const int n_k_all = hidden / kTK, k_first = SPLIT ? n_k_all * part / parts.n : 0;            // this part's stages: k_first .. + n_k - 1
  const int n_k = SPLIT ? n_k_all * (part + 1) / parts.n - k_first : n_k_all;
  __builtin_assume(!SPLIT || n_k > 0);
  // wavefront w brings rows 32 w .. 32 w + 31 of W and of x, 8 rows per instruction
  uint32_t voff_w[4], voff_x[4];
  const char* base_w;
  const char* base_x = reinterpret_cast<const char*>(x + static_cast<size_t>(m0) * hidden) + k_first * (kTK * 2);
  if (MODE != kOutGated) base_w = reinterpret_cast<const char*>(w + static_cast<size_t>(n0) * hidden);
  else base_w = reinterpret_cast<const char*>(((wave % FB) >= FB / 2 ? w2 : w) + static_cast<size_t>(n0 / 2) * hidden);
  base_w += k_first * (kTK * 2);
#pragma unroll
  for (int j = 0; j < 4; ++j) {
    const int r = 32 * wave + 8 * j + (lane >> 3);
    const int rw = MODE != kOutGated ? r : 32 * ((wave / FB) * (FB / 2) + wave % (FB / 2)) + (r & 31);
    voff_w[j] = static_cast<uint32_t>(rw) * static_cast<uint32_t>(hidden * 2) + 16 * ((lane & 7) ^ gemm_swz_w(r));
    voff_x[j] = static_cast<uint32_t>(min(r, n_rows - 1 - m0)) * static_cast<uint32_t>(hidden * 2) + 16 * ((lane & 7) ^ gemm_swz_x(r));
  }
  typedef __attribute__((address_space(3))) const uint4 lds_piece;
  const uint32_t lds_base = __builtin_amdgcn_readfirstlane(static_cast<uint32_t>(reinterpret_cast<uintptr_t>((lds_piece*)lds))) + wave * 4096;
  auto dma_w = [&](int t, int slot, int j) __attribute__((always_inline)) {
    gemm_load_to_lds(base_w + static_cast<size_t>(min(t, n_k - 1)) * (kTK * 2), voff_w[j], lds_base + slot * kHalf + j * 1024);
  };
  auto dma_x = [&](int t, int slot, int j) __attribute__((always_inline)) {
    gemm_load_to_lds(base_x + static_cast<size_t>(min(t, n_k - 1)) * (kTK * 2), voff_x[j], lds_base + slot * kHalf + j * 1024);
  };
  f32x4 acc[FB][2][TB];
#pragma unroll
  for (int a = 0; a < FB; ++a)
#pragma unroll
    for (int i2 = 0; i2 < 2; ++i2)
#pragma unroll
      for (int b = 0; b < TB; ++b)
#pragma unroll
        for (int i = 0; i < 4; ++i) asm volatile("v_accvgpr_write_b32 %0, 0" : "=a"(acc[a][i2][b][i]));

  const char* lds_bytes = reinterpret_cast<const char*>(lds);
  const int r_w = 8 * (nl >> 2) + (nl & 3), r_x = nl;
  const int at_w0 = (32 * FB * wn + r_w) * 128 + ((g ^ gemm_swz_w(r_w)) << 4), at_w1 = (32 * FB * wn + r_w) * 128 + (((4 + g) ^ gemm_swz_w(r_w)) << 4);
  const int at_x0 = (16 * TB * wm + r_x) * 128 + ((g ^ gemm_swz_x(r_x)) << 4), at_x1 = (16 * TB * wm + r_x) * 128 + (((4 + g) ^ gemm_swz_x(r_x)) << 4);
  auto read_w = [&](int slot, int s, int i) __attribute__((always_inline)) {
    return *reinterpret_cast<const u32x4*>(lds_bytes + slot * kHalf + (s == 0 ? at_w0 : at_w1) + (i >> 1) * 4096 + (i & 1) * 512);
  };
  auto read_x = [&](int slot, int s, int b) __attribute__((always_inline)) {
    return *reinterpret_cast<const u32x4*>(lds_bytes + slot * kHalf + (s == 0 ? at_x0 : at_x1) + b * 2048);
  };
  u32x4 opw[8], opx[2][TB];

#pragma unroll
  for (int t = 0; t < 2; ++t) {
#pragma unroll
    for (int j = 0; j < 4; ++j) dma_w(t, 2 * t, j);
#pragma unroll
    for (int j = 0; j < 4; ++j) dma_x(t, 2 * t + 1, j);
  }
  gemm_wait_loads<8>();
  gemm_barrier();
#pragma unroll
  for (int b = 0; b < TB; ++b) opx[0][b] = read_x(1, 0, b);
#pragma unroll
  for (int i = 0; i < 8; ++i) opw[i] = read_w(0, 0, i);
  int sw = 0;                                              // slot of W of stage t; x sits in the next slot
  for (int t = 0; t < n_k; ++t) {
    const int sx = sw == 4 ? 0 : sw + 1, sp = sw == 0 ? 4 : sw - 1;
    const int sw1 = sw >= 3 ? sw - 3 : sw + 2, sx1 = sw1 == 4 ? 0 : sw1 + 1;
#pragma unroll
    for (int b = 0; b < TB; ++b) opx[1][b] = read_x(sx, 1, b);
    __builtin_amdgcn_sched_barrier(0);
#pragma unroll
    for (int i = 0; i < 8; ++i) {
#pragma unroll
      for (int b = 0; b < TB; ++b) gemm_mfma(acc[i >> 1][i & 1][b], opw[i], opx[0][b]);
      opw[i] = read_w(sw, 1, i);
      if (i & 1) dma_w(t + 2, sp, i >> 1);
      __builtin_amdgcn_sched_barrier(0);
    }
#pragma unroll
    for (int i = 0; i < 8; ++i) {
      if (i == kMeet) {
        gemm_wait_loads<4>();
        gemm_wait_lds();
        gemm_barrier();
#pragma unroll
        for (int k = 0; k < kMeet; ++k) opw[k] = read_w(sw1, 0, k);
#pragma unroll
        for (int b = 0; b < TB; ++b) opx[0][b] = read_x(sx1, 0, b);
        __builtin_amdgcn_sched_barrier(0);
      }
#pragma unroll
      for (int b = 0; b < TB; ++b) gemm_mfma(acc[i >> 1][i & 1][b], opw[i], opx[1][b]);
      if (i >= kMeet) opw[i] = read_w(sw1, 0, i);
      if (i >= kMeet && i < kMeet + 4) dma_x(t + 2, sw, i - kMeet);
      __builtin_amdgcn_sched_barrier(0);
    }
    sw = sw1;
  }
  gemm_wait_loads<0>();            // (nothing may still be landing when the LDS is given back)
  asm volatile("s_nop 15\n\ts_nop 15" ::: "memory");
  if constexpr (SPLIT) {
#pragma unroll
    for (int b = 0; b < TB; ++b)
#pragma unroll
      for (int a = 0; a < FB; ++a)
        gemm_store_part(parts, part, m0 / 16 + TB * wm + b, n0 / 32 + FB * wn + a, lane, acc[a][0][b], acc[a][1][b]);
    return;
  }
  const int tok0 = m0 + 16 * TB * wm + nl;
  const int col0 = (MODE == kOutGated ? n0 / 2 + 32 * (FB / 2) * wn : n0 + 32 * FB * wn) + 8 * g;
  constexpr int FO = MODE == kOutGated ? FB / 2 : FB;
#pragma unroll
  for (int b = 0; b < TB; ++b) {
    const int row = tok0 + 16 * b;
    if (row >= n_rows) continue;
#pragma unroll
    for (int a = 0; a < FO; ++a)
      gemm_store8<MODE>(acc[a][0][b], acc[a][1][b], acc[FB - FO + a][0][b], acc[FB - FO + a][1][b],
                        gemm_residual8<MODE>(out, row, col0 + 32 * a), out, row, col0 + 32 * a);
  }
}

// The sums of a contraction in parts: a wavefront per 32 features x 16 tokens adds the parts in their order and
// finishes the outputs as the kernels above do.  Bound by the parts' bytes (5 - 11 us at 230 rows x 8192 features x 4 parts to 1000 x
// 4096 x 4, start included).
template <int MODE>
__global__ __launch_bounds__(256) void gemm_sum_kernel(int n_rows, GemmOut out, GemmParts parts) {
  const int lane = threadIdx.x & 63;
  const int at = blockIdx.x * 4 + __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int tb = at / parts.n_fb, fb = at - tb * parts.n_fb;
  if (16 * tb >= n_rows) return;
  const int row = 16 * tb + (lane & 15), col = 32 * fb + 8 * (lane >> 4);
  const uint4 residual = gemm_residual8<MODE>(out, min(row, n_rows - 1), col);
  constexpr int kTogether = 4;                            // parts asked for at a time
  f32x4 lo = {0.f, 0.f, 0.f, 0.f}, hi = lo;
  for (int p0 = 0; p0 < parts.n; p0 += kTogether) {
    f32x4 v[kTogether][2];
#pragma unroll
    for (int i = 0; i < kTogether; ++i) {
      const f32x4* from = parts.sums + ((static_cast<size_t>(min(p0 + i, parts.n - 1)) * parts.n_tb + tb) * parts.n_fb + fb) * 128 + lane;
      v[i][0] = from[0];
      v[i][1] = from[64];
    }
#pragma unroll
    for (int i = 0; i < kTogether; ++i)
      if (p0 + i < parts.n) { lo += v[i][0]; hi += v[i][1]; }
  }
  if (row < n_rows) gemm_store8<MODE>(lo, hi, lo, hi, residual, out, row, col);
}

template <int MODE>
void launch_gemm_256(hipStream_t stream, const void* x, const void* w, const void* w2, int n_rows, int n_in, int n_features,
                      const GemmOut& out, const GemmParts& parts) {
  const int tiles_n = n_features / 256, tiles_m = (n_rows + 255) / 256;
#define CC_GO(M, SPLIT)                                                                                              \
  hipLaunchKernelGGL((gemm_kernel<M, SPLIT>), dim3((tiles_n * tiles_m * parts.n + 7) / 8 * 8), dim3(512), 0,            \
                     stream, static_cast<const bf16_t*>(x), static_cast<const bf16_t*>(w), static_cast<const bf16_t*>(w2), \
                     n_rows, n_in, tiles_n, tiles_m, out, parts)
  if (parts.sums == nullptr) CC_GO(MODE, false);
  else if constexpr (MODE != kOutGated) CC_GO(kOutLinear, true);
#undef CC_GO
}

template <int MODE, int FB, int TB, int WF, int WM, int WK, int U, int NBUF>
void launch_gemm_tile(hipStream_t stream, const void* x, const void* w, const void* w2, int n_rows, int n_in, int n_features,
                      const GemmOut& out, const GemmParts& parts) {
  const int tiles_n = n_features / (32 * FB * WF), tiles_m = (n_rows + 16 * TB * WM - 1) / (16 * TB * WM);
#define CC_GO(M, SPLIT)                                                                                              \
  hipLaunchKernelGGL((gemm_tile_kernel<M, SPLIT, FB, TB, WF, WM, WK, U, NBUF>), dim3((tiles_n * tiles_m * parts.n + 7) / 8 * 8), \
                     dim3(64 * WF * WM * WK), 0, stream, static_cast<const bf16_t*>(x), static_cast<const bf16_t*>(w),  \
                     static_cast<const bf16_t*>(w2), n_rows, n_in, tiles_n, tiles_m, out, parts)
  if (parts.sums == nullptr) CC_GO(MODE, false);
  else if constexpr (MODE != kOutGated) CC_GO(kOutLinear, true);
#undef CC_GO
}

// Tile shapes and what a stage of 64 contraction indices takes on a compute unit that runs one workgroup of
// that shape (us; measured over and over with the same weights, which the memory-side cache then holds.  In a decoder layer they come from HBM, and whole products of few rows take 10 to
// 30 % longer than these times say: 449 rows 4096 -> 6144 35 / 38, 4096 -> 4096 23 / 29, 230 rows 8192 -> 8192 46 / 58; products in parts, whose cost has a term for the
// weights, hardly: 230 rows 28672 -> 8192 118 / 123): big tiles do more flops per byte that passes a compute unit's L1, small
// ones give short lists enough workgroups.  A product takes the shape with the smallest
// (rounds of 256 workgroups) x (stage time).
struct GemmTile { int f, m, k; float stage_us; };
constexpr GemmTile kGemmTiles[] = {{256, 256, 64, 1.43f}, {128, 256, 64, 0.92f}, {128, 128, 64, 0.54f},
                                   {64, 128, 64, 0.36f},  {64, 64, 128, 0.27f},  {32, 64, 128, 0.21f}};
constexpr int kGemmUnits = 256;                       // compute units

inline bool gemm_tile_fits(int i, int n_features, int n_in, bool gated) {
  return n_features % kGemmTiles[i].f == 0 && n_in % kGemmTiles[i].k == 0 && !(gated && kGemmTiles[i].f < 64);
}
inline float gemm_tile_cost(int i, int n_features, int n_rows) {
  const GemmTile& t = kGemmTiles[i];
  const int64_t tiles = static_cast<int64_t>(n_features / t.f) * ((n_rows + t.m - 1) / t.m);
  return static_cast<float>((tiles + kGemmUnits - 1) / kGemmUnits) * t.stage_us;
}
inline int gemm_best_tile(int n_features, int n_in, int n_rows, bool gated) {
  int best = -1;
  for (int i = 0; i < 6; ++i)
    if (gemm_tile_fits(i, n_features, n_in, gated) &&
        (best < 0 || gemm_tile_cost(i, n_features, n_rows) < gemm_tile_cost(best, n_features, n_rows))) best = i;
  return best;
}

template <int MODE>
void launch_gemm_shape(int shape, hipStream_t stream, const void* x, const void* w, const void* w2, int n_rows, int n_in,
                       int n_features, const GemmOut& out, const GemmParts& parts) {
#define CC_TILE(...) launch_gemm_tile<MODE, __VA_ARGS__>(stream, x, w, w2, n_rows, n_in, n_features, out, parts)
  switch (shape) {
    case 0: launch_gemm_256<MODE>(stream, x, w, w2, n_rows, n_in, n_features, out, parts); break;
    case 1: CC_TILE(2, 4, 2, 4, 1, 1, 3); break;      // (128 x 256: 8 wavefronts of 64 x 64)
    case 2: CC_TILE(2, 4, 2, 2, 2, 1, 4); break;      // (128 x 128: 8 of 64 x 64, half the k-steps each)
    case 3: CC_TILE(2, 4, 1, 2, 2, 1, 5); break;      // (64 x 128: 4 of 64 x 64, half the k-steps each)
    case 4: CC_TILE(2, 4, 1, 1, 4, 2, 5); break;      // (64 x 64: 4, a quarter of the k-steps each)
    default: if constexpr (MODE != kOutGated) CC_TILE(1, 4, 1, 1, 4, 2, 5); break;   // (32 x 64: the same)
  }
#undef CC_TILE
  if constexpr (MODE != kOutGated)
    if (parts.sums != nullptr)
      hipLaunchKernelGGL((gemm_sum_kernel<MODE>), dim3(((n_rows + 15) / 16 * parts.n_fb + 3) / 4), dim3(256), 0, stream, n_rows, out, parts);
}

// How a range of rows is multiplied: the tile, the parts of the contraction, and what that is expected to take.
struct GemmChoice { int shape, parts; float us; };
inline int gemm_padded_rows(int shape, int n_rows) { return (n_rows + kGemmTiles[shape].m - 1) / kGemmTiles[shape].m * kGemmTiles[shape].m; }
inline size_t gemm_parts_bytes(const GemmChoice& c, int n_features, int n_rows) {
  return c.parts == 1 ? 0 : static_cast<size_t>(c.parts) * gemm_padded_rows(c.shape, n_rows) * n_features * sizeof(float);
}

// A short list has too few big tiles for 256 compute units, and small ones pass each weight line through an L1 with few tokens to
// multiply: parts of the contraction let big tiles fill the chip.  They cost their sums' way through memory
// (8 bytes per part and output at kPartsRate) and a launch; and nothing is faster than the weights arrive.  Whole / in parts, us:
// 28672 -> 8192 features, 60 rows 128 / 101, 230 rows 197 / 136, 449 250 / 208, 1000 414 / 372; 14336 -> 4096, 60 rows 50 / 29, 230
// 60 / 44, 449 78 / 66, 1000 127 / 110; 8192 -> 10240, 230 rows 73 / 55, 449 105 / 84; 4096 -> 6144, 449 rows 35 / 48: stays whole.
// (Over 204 products of these widths and 20 to 2300 rows the choice takes 1.6 % longer than the best of all tiles and
// parts, the choice without parts 10 %; none is slower than that.)  Gated products have enough tiles by themselves: 2 x 14336 features,
// 230 rows 66 / 79, 449 99 / 136.
constexpr int kMaxParts = 8;
constexpr size_t kMaxPartsBytes = size_t{256} << 20;
constexpr float kPartsUs = 6.f, kPartsRate = 5e6f, kWeightRate = 5.5e6f;       // a launch; bytes per us
inline GemmChoice gemm_choose(int n_features, int n_in, int n_rows, bool gated, size_t room) {
  GemmChoice c{gemm_best_tile(n_features, n_in, n_rows, gated), 1, 0.f};
  c.us = gemm_tile_cost(c.shape, n_features, n_rows) * n_in / kTK;
  if (gated) return c;
  const float weights_us = 2.f * n_features * n_in / kWeightRate;
  float whole = c.us > weights_us ? c.us : weights_us;
  for (int i = 0; i < 6; ++i) {
    if (!gemm_tile_fits(i, n_features, n_in, gated)) continue;
    const GemmTile& t = kGemmTiles[i];
    const int64_t tiles = static_cast<int64_t>(n_features / t.f) * ((n_rows + t.m - 1) / t.m);
    const int stages = n_in / t.k;
    for (int p = 2; p <= kMaxParts && p <= stages; ++p) {
      GemmChoice s{i, p, 0.f};
      const size_t bytes = gemm_parts_bytes(s, n_features, n_rows);
      if (bytes > room || bytes > kMaxPartsBytes) break;
      const float mul = static_cast<float>((tiles * p + kGemmUnits - 1) / kGemmUnits) * t.stage_us * ((stages + p - 1) / p) * (t.k / kTK);
      s.us = (mul > weights_us ? mul : weights_us) + kPartsUs + 2.f * bytes / kPartsRate;
      if (s.us < whole) { whole = s.us; c = s; }
    }
  }
  return c;
}

// A product of a few rounds of 256 x 256 tiles leaves most of the chip idle in its last one: then the first `full` rows (whole
// rounds) go to that kernel and the rest to what suits it, in a launch of its own (about 6 us more).
struct GemmPlan { int full; GemmChoice rest; };
inline GemmPlan gemm_plan(int n_features, int n_in, int n_rows, bool gated, size_t room) {
  GemmPlan plan{0, gemm_choose(n_features, n_in, n_rows, gated, room)};
  if (!gemm_tile_fits(0, n_features, n_in, gated)) return plan;
  const int tiles_n = n_features / 256, rounds = tiles_n * ((n_rows + 255) / 256) / kGemmUnits;
  const int rows_full = rounds * kGemmUnits / tiles_n * 256, rest = n_rows - rows_full;
  if (rows_full <= 0 || rest <= 0) return plan;
  const GemmChoice tail = gemm_choose(n_features, n_in, rest, gated, room);
  if (gemm_tile_cost(0, n_features, rows_full) * n_in / kTK + tail.us + 6.f < plan.rest.us) plan = GemmPlan{rows_full, tail};
  return plan;
}

template <int MODE>
void launch_gemm(hipStream_t stream, const void* x, const void* w, const void* w2, int n_rows, int n_in, int n_features,
                 const GemmOut& out, void* workspace, size_t room) {
  const GemmPlan plan = gemm_plan(n_features, n_in, n_rows, MODE == kOutGated, workspace != nullptr ? room : 0);
  auto shift = [&](const void* p, int width) { return p == nullptr ? nullptr : static_cast<const bf16_t*>(p) + static_cast<size_t>(plan.full) * width; };
  const GemmParts whole{nullptr, 1, 0, 0};
  if (plan.full > 0) launch_gemm_shape<MODE>(0, stream, x, w, w2, plan.full, n_in, n_features, out, whole);
  const int rest = n_rows - plan.full;
  GemmOut o = out;
  if (MODE == kOutQkv) {
    o.o0 = const_cast<bf16_t*>(shift(out.o0, out.nq)); o.o1 = const_cast<bf16_t*>(shift(out.o1, out.nk)); o.o2 = const_cast<bf16_t*>(shift(out.o2, out.nk));
  } else {
    o.o0 = const_cast<bf16_t*>(shift(out.o0, out.width)); o.residual = shift(out.residual, out.width);
  }
  const GemmParts parts = plan.rest.parts == 1 ? whole
      : GemmParts{static_cast<f32x4*>(workspace), plan.rest.parts, gemm_padded_rows(plan.rest.shape, rest) / 16, n_features / 32};
  launch_gemm_shape<MODE>(plan.rest.shape, stream, shift(x, n_in), w, w2, rest, n_in, n_features, o, parts);
}

// the MFMA GEMMs take outputs in tiles of at least 64 features and contraction lengths in whole cache lines
inline bool gemm_fits(const cc_ctx* ctx, int n_features, int n_in) {
  return ctx->cfg.dtype == CC_BF16 && ctx->impl != CC_IMPL_SCALAR && n_features % 64 == 0 && n_in % kTK == 0;
}

}  // namespace

// bytes that let a product of these sizes take the parts it would like to (0: it stays whole)
size_t gemm_workspace_bytes(const cc_ctx* ctx, int n_rows, int n_in, int n_features) {
  if (n_rows <= 0 || n_in <= 0 || n_features <= 0 || !gemm_fits(ctx, n_features, n_in)) return 0;
  const GemmPlan plan = gemm_plan(n_features, n_in, n_rows, false, kMaxPartsBytes);
  return gemm_parts_bytes(plan.rest, n_features, n_rows - plan.full);
}

void launch_qkv_project(const cc_ctx* ctx, const void* x, const void* w, int n_rows, int hidden,
                        void* q, void* k, void* v, void* workspace, size_t workspace_bytes, hipStream_t stream) {
  const int d = ctx->cfg.head_dim;
  const int nq = ctx->cfg.n_q_heads * d, nk = ctx->cfg.n_kv_heads * d, n_cols = nq + 2 * nk;
  if (gemm_fits(ctx, n_cols, hidden) && nq % 32 == 0 && nk % 32 == 0) {
    launch_gemm<kOutQkv>(stream, x, w, nullptr, n_rows, hidden, n_cols, GemmOut{q, k, v, nullptr, nq, nk, 0}, workspace, workspace_bytes);
    return;
  }
  dim3 grid((n_cols + 63) / 64, (n_rows + 63) / 64);
  if (ctx->cfg.dtype == CC_BF16)
    hipLaunchKernelGGL(qkv_project_plain_kernel<bf16_t>, grid, dim3(256), 0, stream,
                       static_cast<const bf16_t*>(x), static_cast<const bf16_t*>(w), n_rows, hidden,
                       n_cols, nq, nk, static_cast<bf16_t*>(q), static_cast<bf16_t*>(k),
                       static_cast<bf16_t*>(v));
  else
    hipLaunchKernelGGL(qkv_project_plain_kernel<float>, grid, dim3(256), 0, stream,
                       static_cast<const float*>(x), static_cast<const float*>(w), n_rows, hidden,
                       n_cols, nq, nk, static_cast<float*>(q), static_cast<float*>(k),
                       static_cast<float*>(v));
}

// y [n_rows][n_out] = x [n_rows][n_in] W^T (+ residual [n_rows][n_out]); W [n_out][n_in]
void launch_linear(const cc_ctx* ctx, const void* x, const void* w, const void* residual, int n_rows, int n_in,
                   int n_out, void* y, void* workspace, size_t workspace_bytes, hipStream_t stream) {
  const bool bf = ctx->cfg.dtype == CC_BF16;
  if (gemm_fits(ctx, n_out, n_in)) {
    launch_gemm<kOutLinear>(stream, x, w, nullptr, n_rows, n_in, n_out, GemmOut{y, nullptr, nullptr, residual, 0, 0, n_out}, workspace, workspace_bytes);
    return;
  }
  dim3 grid((n_out + 63) / 64, (n_rows + 63) / 64);
  if (bf)
    hipLaunchKernelGGL((linear_plain_kernel<bf16_t, false>), grid, dim3(256), 0, stream, static_cast<const bf16_t*>(x),
                       static_cast<const bf16_t*>(w), static_cast<const bf16_t*>(nullptr),
                       static_cast<const bf16_t*>(residual), n_rows, n_in, n_out, static_cast<bf16_t*>(y));
  else
    hipLaunchKernelGGL((linear_plain_kernel<float, false>), grid, dim3(256), 0, stream, static_cast<const float*>(x),
                       static_cast<const float*>(w), static_cast<const float*>(nullptr),
                       static_cast<const float*>(residual), n_rows, n_in, n_out, static_cast<float*>(y));
}

// y [n_rows][n_ffn] = silu(x W_gate^T) * (x W_up^T); both W [n_ffn][n_in]
void launch_gated_linear(const cc_ctx* ctx, const void* x, const void* w_gate, const void* w_up, int n_rows,
                         int n_in, int n_ffn, void* y, hipStream_t stream) {
  const bool bf = ctx->cfg.dtype == CC_BF16;
  if (gemm_fits(ctx, 2 * n_ffn, n_in)) {
    launch_gemm<kOutGated>(stream, x, w_gate, w_up, n_rows, n_in, 2 * n_ffn, GemmOut{y, nullptr, nullptr, nullptr, 0, 0, n_ffn}, nullptr, 0);
    return;
  }
  dim3 grid((n_ffn + 63) / 64, (n_rows + 63) / 64);
  if (bf)
    hipLaunchKernelGGL((linear_plain_kernel<bf16_t, true>), grid, dim3(256), 0, stream, static_cast<const bf16_t*>(x),
                       static_cast<const bf16_t*>(w_gate), static_cast<const bf16_t*>(w_up),
                       static_cast<const bf16_t*>(nullptr), n_rows, n_in, n_ffn, static_cast<bf16_t*>(y));
  else
    hipLaunchKernelGGL((linear_plain_kernel<float, true>), grid, dim3(256), 0, stream, static_cast<const float*>(x),
                       static_cast<const float*>(w_gate), static_cast<const float*>(w_up),
                       static_cast<const float*>(nullptr), n_rows, n_in, n_ffn, static_cast<float*>(y));
}

// ---- root-mean-square normalisation: y = x / sqrt(mean(x^2) + eps) * gain ---------------------------
// Rows of 256 to 1024 pieces of 16 bytes take a workgroup each (rms_norm_row_kernel), others a wavefront (four rows per
// workgroup).  A row stays in registers between the sum of squares and the scaling, so that it moves once in
// and once out of HBM; what a row has behind its first 1024 pieces is read a second time.
// the elements of a 16-byte piece as floats, and back, without taking the piece's address (which
// would move a register array to scratch memory)
__device__ __forceinline__ void piece_to_floats(const uint4& p, float (&f)[8], bf16_t*) {
  const uint32_t u[4] = {p.x, p.y, p.z, p.w};
#pragma unroll
  for (int i = 0; i < 4; ++i) {
    f[2 * i] = __uint_as_float(u[i] << 16);
    f[2 * i + 1] = __uint_as_float(u[i] & 0xffff0000u);
  }
}
__device__ __forceinline__ void piece_to_floats(const uint4& p, float (&f)[4], float*) {
  f[0] = __uint_as_float(p.x); f[1] = __uint_as_float(p.y); f[2] = __uint_as_float(p.z); f[3] = __uint_as_float(p.w);
}

// ss plus the squares of a piece, element by element; the first piece of a row that is kept whole begins with its second square,
// and every product goes into its sum unrounded.  (Written out because it decides the last bit of a sum in fp32, and that turns roundings to bf16
// which each product of a decoder layer passes on.)
template <int kPer>
__device__ __forceinline__ float add_squares(float ss, const float (&f)[kPer], bool first) {
  if (first) ss = fmaf(f[0], f[0], f[1] * f[1]);
#pragma unroll
  for (int e = 0; e < kPer; ++e)
    if (!first || e >= 2) ss = fmaf(f[e], f[e], ss);
  return ss;
}

// kKeep: 16-byte pieces a lane keeps.  4: whole rows (up to 256 pieces).  16: the first 1024 pieces of a long one, the others are read
// twice; without any kept, the rows in flight outgrow what is cached between the two reads.  fp32, none / these kept, us: 14000 x 8192
// 257 / 217, 2000 x 8192 37.5 / 31.0, 4000 x 12288 118 / 113, 14000 x 16384 552 / 504; bf16 449 x 16384 22.7 / 18.2.
template <typename T, int kKeep>
__global__ __launch_bounds__(256) void rms_norm_kernel(const T* x, const T* __restrict__ gain, float eps,
                                                       int n_rows, int hidden, T* y) {          // (y may be x)
  const int row = blockIdx.x * 4 + threadIdx.x / 64, lane = threadIdx.x % 64;
  if (row >= n_rows) return;
  constexpr int kPer = 16 / sizeof(T);                 // elements per 16-byte piece
  constexpr bool kWhole = kKeep == 4;
  const T* xr = x + static_cast<size_t>(row) * hidden;
  T* yr = y + static_cast<size_t>(row) * hidden;
  const int n_pieces = hidden / kPer;                  // (the call checks that hidden is a multiple of kPer)
  uint4 held[kKeep];
  auto piece = [&](int p) __attribute__((always_inline)) { return *reinterpret_cast<const uint4*>(xr + p * kPer); };
#pragma unroll
  for (int i = 0; i < kKeep; ++i) held[i] = lane + 64 * i < n_pieces ? piece(lane + 64 * i) : uint4{0, 0, 0, 0};
  float ss = 0.f;
  auto add = [&](const uint4& in, bool first) __attribute__((always_inline)) {
    float f[kPer];
    piece_to_floats(in, f, static_cast<T*>(nullptr));
    ss = add_squares(ss, f, first);
  };
#pragma unroll
  for (int i = 0; i < kKeep; ++i) add(held[i], kWhole && i == 0);
  if constexpr (!kWhole)
    for (int p = lane + 64 * kKeep; p < n_pieces; p += 64) add(piece(p), false);
  const float scale = rsqrtf(wave_sum(ss) / static_cast<float>(hidden) + eps);
  auto scaled = [&](const uint4& in, int p) __attribute__((always_inline)) {
    float f[kPer], g[kPer];
    T o[kPer];
    piece_to_floats(in, f, static_cast<T*>(nullptr));
    piece_to_floats(*reinterpret_cast<const uint4*>(gain + p * kPer), g, static_cast<T*>(nullptr));
#pragma unroll
    for (int e = 0; e < kPer; ++e) o[e] = from_float<T>(f[e] * scale * g[e]);
    *reinterpret_cast<uint4*>(yr + p * kPer) = *reinterpret_cast<uint4*>(o);
  };
#pragma unroll
  for (int i = 0; i < kKeep; ++i)
    if (lane + 64 * i < n_pieces) scaled(held[i], lane + 64 * i);
  if constexpr (!kWhole)
    for (int p = lane + 64 * kKeep; p < n_pieces; p += 64) scaled(piece(p), p);
}

// A workgroup of four wavefronts per row: with a wavefront per row a short list leaves most compute units without one, and a
// lane has four times as many pieces to wait for.  The sum of squares is that of the kernel above, bit for bit:
// lane l adds the elements of pieces l, l + 64, l + 128, ... in this order, so the wavefronts have consecutive shares of the
// pieces and hand the lanes' sums on, and the 64 sums meet in wave_sum.  bf16, a wavefront per row / this, us: 449 x 4096 in a decoder
// layer 7.4 / 5.3, 230 x 8192 10.8 / 5.2, 13824 x 4096 43 / 36 (6.3 TB/s), back to back 14000 x 8192 93 / 79, fp32 14000 x 4096 90 / 78.
template <typename T>
__global__ __launch_bounds__(256) void rms_norm_row_kernel(const T* x, const T* __restrict__ gain, float eps, int hidden, T* y) {   // (y may be x)
  constexpr int kPer = 16 / sizeof(T), kKeep = 4;      // elements per 16-byte piece; pieces a thread keeps
  __shared__ float sums[64];
  const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6), n_pieces = hidden / kPer;
  const int share = (n_pieces + 255) / 256, first = 64 * share * wave + lane;      // piece i of this thread: first + 64 i, i < share
  const T* xr = x + static_cast<size_t>(blockIdx.x) * hidden;
  T* yr = y + static_cast<size_t>(blockIdx.x) * hidden;
  uint4 held[kKeep], g[kKeep];
#pragma unroll
  for (int i = 0; i < kKeep; ++i) {
    const int p = first + 64 * i;
    const bool there = i < share && p < n_pieces;
    held[i] = there ? *reinterpret_cast<const uint4*>(xr + p * kPer) : uint4{0, 0, 0, 0};
    g[i] = there ? *reinterpret_cast<const uint4*>(gain + p * kPer) : uint4{0, 0, 0, 0};
  }
#pragma unroll
  for (int w = 0; w < 4; ++w) {
    if (wave == w) {
      float ss = w == 0 ? 0.f : sums[lane];
#pragma unroll
      for (int i = 0; i < kKeep; ++i) {
        if (i >= share) break;
        float f[kPer];
        piece_to_floats(held[i], f, static_cast<T*>(nullptr));
        ss = add_squares(ss, f, w == 0 && i == 0);
      }
      sums[lane] = ss;
    }
    __syncthreads();
  }
  const float scale = rsqrtf(wave_sum(sums[lane]) / static_cast<float>(hidden) + eps);
#pragma unroll
  for (int i = 0; i < kKeep; ++i) {
    const int p = first + 64 * i;
    if (i >= share || p >= n_pieces) continue;
    float f[kPer], w[kPer];
    T o[kPer];
    piece_to_floats(held[i], f, static_cast<T*>(nullptr));
    piece_to_floats(g[i], w, static_cast<T*>(nullptr));
#pragma unroll
    for (int e = 0; e < kPer; ++e) o[e] = from_float<T>(f[e] * scale * w[e]);
    *reinterpret_cast<uint4*>(yr + p * kPer) = *reinterpret_cast<uint4*>(o);
  }
}

void launch_rms_norm(const cc_ctx* ctx, const void* x, const void* gain, float eps, int n_rows, int hidden, void* y,
                     hipStream_t stream) {
  const bool bf = ctx->cfg.dtype == CC_BF16;
  const int n_pieces = hidden / (bf ? 8 : 4);
  const bool by_row = n_pieces >= 256 && n_pieces <= 256 * 4;
  const dim3 grid(by_row ? n_rows : (n_rows + 3) / 4);
#define CC_LAUNCH(T)                                                                                             \
  do {                                                                                                           \
    const T *xt = static_cast<const T*>(x), *gt = static_cast<const T*>(gain);                                   \
    if (by_row) hipLaunchKernelGGL(rms_norm_row_kernel<T>, grid, dim3(256), 0, stream, xt, gt, eps, hidden, static_cast<T*>(y)); \
    else if (n_pieces < 256) hipLaunchKernelGGL((rms_norm_kernel<T, 4>), grid, dim3(256), 0, stream, xt, gt, eps, n_rows, hidden, static_cast<T*>(y)); \
    else hipLaunchKernelGGL((rms_norm_kernel<T, 16>), grid, dim3(256), 0, stream, xt, gt, eps, n_rows, hidden, static_cast<T*>(y)); \
  } while (0)
  if (bf) CC_LAUNCH(bf16_t);
  else CC_LAUNCH(float);
#undef CC_LAUNCH
}

}  // namespace cc
