// cc_select's score stage and cc_sparse_prefill's attention in fp32 arithmetic on the matrix cores, for
// what the bf16 MFMA kernels do not take: fp32 tensors, head_dim 64, other head groups (per-token
// form of Eq. (1); Eq. (2), Eq. (10)).
//
// One workgroup = 16 query rows x one query head; its four wavefronts take the 16-token key blocks of the
// request in turn and merge their softmax statistics (and outputs) at the end.  These batches are
// small - a few thousand keys at most - and one wavefront per row with a cross-lane sum per key spent
// its time in that chain (three 64-token chunks, 4 heads of 64: 111 us to score, 137 us to attend,
// whatever the chip).  Here a block of 16 keys is D/4 + D/4 v_mfma_f32_16x16x4_f32 for 16 rows, and
// the chain is one block per wavefront at a time, with the next block's keys and values already loading.
//
// Layout: S^T = K Q^T and O^T = V^T P^T with lane = (n = lane % 16, g = lane / 16).  In step (c, e) of the
// first product lane (n, g) feeds dim 16 c + 4 g + e of key n and of query n: the contraction order is
// free as long as both operands agree, so a lane reads its operands as 16-byte pieces of a row.  S then
// holds, for query n, the keys 4 g + i in register i - and step e of the second product contracts
// exactly over the keys 4 g + e, so P goes from the result registers straight into the second
// product, and the value operand is a 16-byte piece (slots 4 g .. 4 g + 3) of a dimension-major V row.
// No operand passes through LDS.
//
// The softmax reference of a query is shared by the four lane groups and moves only when some logit
// is more than kSlack above it (the sums are fp32, exp(kSlack) leaves their precision alone).
#include "device_util.h"

namespace cc {

namespace {

constexpr int kRowsQ = 16;            // query rows per workgroup
constexpr int kWindow = 512;          // key blocks listed in LDS at a time
constexpr float kSlack = 8.f;

__device__ __forceinline__ f32x4 load4(const float* p) { return *reinterpret_cast<const f32x4*>(p); }
__device__ __forceinline__ f32x4 load4(const bf16_t* p) {
  const uint2 u = *reinterpret_cast<const uint2*>(p);
  f32x4 r;
  r[0] = __uint_as_float(u.x << 16); r[1] = __uint_as_float(u.x & 0xffff0000u);
  r[2] = __uint_as_float(u.y << 16); r[3] = __uint_as_float(u.y & 0xffff0000u);
  return r;
}

// SCORE: rows are consecutive tokens of a chunk segment, the result is the share of the softmax mass on
// keys of earlier segments.  Otherwise rows of the compact query list, the result is output + log-sum-exp.
// (two wavefronts per SIMD asked for: with half the registers the matrix results stay where the vector ALU reads them, which
// takes 8 % off the outputs' time at D = 128: 8 x 2k keys, 8 heads 305 -> 283 us)
template <typename T, int D, bool SCORE>
__global__ __launch_bounds__(256, SCORE ? 1 : 2) void qk_f32_kernel(
    const T* __restrict__ q, const int32_t* __restrict__ q_pos, const int32_t* __restrict__ cu_q,
    const T* __restrict__ k_pool, const T* __restrict__ v_pool, int n_blocks, const int32_t* __restrict__ block_tab,
    const cc_segment* __restrict__ segs, const int32_t* __restrict__ req_seg_off, int hq, int hkv, InvFreq inv_freq,
    T* __restrict__ out, float* __restrict__ lse, float* __restrict__ mass, const int32_t* __restrict__ q_map, int map_pos,
    const T* __restrict__ v_shared, int n_shared_blocks, const int32_t* __restrict__ v_map) {
  constexpr int kC = D / 16;           // 16-byte pieces of a row per lane; 16-dim groups of the output
  const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int n = lane & 15, g = lane >> 4;
  const int h = blockIdx.z, kvh = h / (hq / hkv);

  // ---- which rows ----
  int row, src, p, p_max, s_begin, s_end, s_self = -1;
  bool row_valid;
  if constexpr (SCORE) {
    const cc_segment sg = segs[blockIdx.y];
    const int t0 = blockIdx.x * kRowsQ;
    if (sg.kind != CC_SEG_CHUNK || t0 >= sg.n_tokens || sg.logical_start == 0) return;   // (no prior chunk: the top-N takes 0)
    const int t = min(t0 + n, sg.n_tokens - 1);
    row_valid = t0 + n < sg.n_tokens;
    row = src = sg.tok_off + t;
    p = sg.logical_start + t;
    p_max = sg.logical_start + min(t0 + kRowsQ, sg.n_tokens) - 1;
    s_begin = req_seg_off[sg.req];
    s_self = blockIdx.y;
    s_end = s_self + 1;
  } else {
    const int r = blockIdx.y;
    const int q0 = cu_q[r] + blockIdx.x * kRowsQ, q_end = cu_q[r + 1];
    if (q0 >= q_end) return;
    row = min(q0 + n, q_end - 1);
    row_valid = q0 + n < q_end;
    // (with a row map, list row j takes its query from row q_map[j] of q and, if map_pos, its position
    // from q_pos[q_map[j]])
    src = q_map != nullptr ? q_map[row] : row;
    p = q_pos[map_pos ? src : row];
    p_max = p;
#pragma unroll
    for (int o = 8; o > 0; o >>= 1) p_max = max(p_max, __shfl_xor(p_max, o, 64));
    s_begin = req_seg_off[r];
    s_end = req_seg_off[r + 1];
  }
  p_max = __builtin_amdgcn_readfirstlane(p_max);

  // ---- the query rows, rotated to their positions (dims < D/2 pair with dims + D/2: same lane) ----
  f32x4 qr[kC];
  {
    const T* qp = q + (static_cast<size_t>(src) * hq + h) * D + 4 * g;
#pragma unroll
    for (int c = 0; c < kC; ++c) qr[c] = load4(qp + 16 * c);
#pragma unroll
    for (int c = 0; c < kC / 2; ++c)
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        float cs, sn;
        rot_cos_sin(p, inv_freq.f[16 * c + 4 * g + e], &cs, &sn);
        const float x = qr[c][e], y = qr[c + kC / 2][e];
        qr[c][e] = x * cs - y * sn;
        qr[c + kC / 2][e] = y * cs + x * sn;
      }
  }

  // ---- key blocks of the request up to the last row's position, kWindow at a time in LDS ----
  struct BlockItem { int blk, kpos0, nvalid, own; };
  __shared__ BlockItem list[kWindow];
  const float scale = rsqrtf(static_cast<float>(D));
  float m = -INFINITY, l = 0.f, l_prior = 0.f;      // l: this lane's keys only; m: one value per query
  f32x4 o[SCORE ? 1 : kC];
#pragma unroll
  for (int c = 0; c < (SCORE ? 1 : kC); ++c) o[c] = f32x4{0.f, 0.f, 0.f, 0.f};
  const size_t block_elems = static_cast<size_t>(hkv) * kBlock * D;
  const size_t head_off = static_cast<size_t>(kvh) * kBlock * D;
  f32x4 kr[2][kC], vr[2][SCORE ? 1 : kC];

  auto load_block = [&](int b, const BlockItem& it) __attribute__((always_inline)) {
    const T* kp = k_pool + it.blk * block_elems + head_off + static_cast<size_t>(n) * D + 4 * g;
#pragma unroll
    for (int c = 0; c < kC; ++c) kr[b][c] = load4(kp + 16 * c);
    if constexpr (!SCORE) {
      const T* vp = value_block<T>(v_pool, v_shared, n_shared_blocks, v_map, it.blk, block_elems) + head_off + n * kBlock + 4 * g;
#pragma unroll
      for (int c = 0; c < kC; ++c) vr[b][c] = load4(vp + 16 * c * kBlock);
    }
  };
  // A row takes nothing from a key behind its position, but the product would give it 0 x value, and the value
  // need not be finite.  So in a block of which some row sees only a part, values that are not finite leave the
  // product; the rows that see their key (the first n_vis of the block) get them here.
  auto select_not_finite = [&](int b, const f32x4& w, int n_vis) __attribute__((always_inline)) {
    auto finite = [](float v) __attribute__((always_inline)) { return fabsf(v) < INFINITY; };
    bool all = true;
#pragma unroll
    for (int c = 0; c < (SCORE ? 0 : kC); ++c)
#pragma unroll
      for (int e = 0; e < 4; ++e) all = all && finite(vr[b][c][e]);
    if (__all(all)) return;
#pragma unroll 1
    for (int gk = 0; gk < 4; ++gk)                   // lanes (., gk) hold the values and weights of keys 4 gk + e
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        const float we = __shfl(w[e], n + 16 * gk, 64);
        const bool sees = 4 * gk + e < n_vis;
#pragma unroll
        for (int c = 0; c < (SCORE ? 0 : kC); ++c)
#pragma unroll
          for (int i = 0; i < 4; ++i) {
            const float v = __shfl(vr[b][c][e], 4 * g + i + 16 * gk, 64);
            if (sees && !finite(v)) o[c][i] += we * v;
          }
      }
#pragma unroll
    for (int c = 0; c < (SCORE ? 0 : kC); ++c)
#pragma unroll
      for (int e = 0; e < 4; ++e) vr[b][c][e] = finite(vr[b][c][e]) ? vr[b][c][e] : 0.f;
  };
  auto use_block = [&](int b, const BlockItem& it) __attribute__((always_inline)) {
    // A logit's absolute error is its weight's relative one, and a single chain of D fp32 additions makes the outputs of
    // short prompts worse than a cross-lane sum does: four chains for the outputs (the mass, a sum of many weights, needs none).
    // Relative error against 64 bits, cross-lane / one chain / four / all in a tree: D = 64, 56 keys 1.0e-7 / 1.5e-7 / 0.9e-7 /
    // 0.9e-7, D = 128, 2k keys 2.9e-7 / 2.9e-7 / 1.8e-7 / 1.6e-7.  The tree's additions cost 20 to 40 % of the time, four chains 2 %.
    constexpr int kChains = SCORE ? 1 : 4;
    f32x4 part[kChains];
#pragma unroll
    for (int i = 0; i < kChains; ++i) part[i] = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int c = 0; c < kC; ++c)
#pragma unroll
      for (int e = 0; e < 4; ++e) part[e % kChains] = __builtin_amdgcn_mfma_f32_16x16x4f32(kr[b][c][e], qr[c][e], part[e % kChains], 0, 0, 0);
    f32x4 s = part[0];
    if constexpr (kChains == 4) s = (part[0] + part[1]) + (part[2] + part[3]);
    const int lim = min(it.nvalid, p - it.kpos0 + 1) - 4 * g;
    float mx = -INFINITY;
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      s[i] = i < lim ? s[i] * scale : -INFINITY;
      mx = fmaxf(mx, s[i]);
    }
    if (__any(mx > m + kSlack)) {
      mx = fmaxf(mx, __shfl_xor(mx, 16, 64));
      mx = fmaxf(mx, __shfl_xor(mx, 32, 64));
      const float m_new = fmaxf(m, mx);
      const float a = m == -INFINITY ? 0.f : expf(m - m_new);
      l *= a;
      if constexpr (SCORE) l_prior *= a;
      else {
#pragma unroll
        for (int c = 0; c < kC; ++c) o[c] *= a;
      }
      m = m_new;
    }
    const float ref = m == -INFINITY ? 0.f : m;      // (no visible key yet: every s is -inf)
    float sum = 0.f;
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      s[i] = expf(s[i] - ref);
      sum += s[i];
    }
    l += sum;
    if constexpr (SCORE) l_prior += it.own ? 0.f : sum;
    else {
      if (it.nvalid < kBlock) {                      // padding slots of V: 0 x garbage would poison O
#pragma unroll
        for (int c = 0; c < kC; ++c)
#pragma unroll
          for (int i = 0; i < 4; ++i) vr[b][c][i] = 4 * g + i < it.nvalid ? vr[b][c][i] : 0.f;
      }
      if (__any(lim + 4 * g < it.nvalid)) select_not_finite(b, s, lim + 4 * g);
#pragma unroll
      for (int c = 0; c < kC; ++c)
#pragma unroll
        for (int e = 0; e < 4; ++e) o[c] = __builtin_amdgcn_mfma_f32_16x16x4f32(vr[b][c][e], s[e], o[c], 0, 0, 0);
    }
  };

  for (int w0 = 0;; w0 += kWindow) {
    __syncthreads();                                 // (the previous window has been walked)
    int n_all = 0;                                   // key blocks up to the last row's position
    for (int s = s_begin; s < s_end; ++s) {
      const cc_segment ks = segs[s];
      const int n_vis = min(ks.n_tokens, p_max - ks.logical_start + 1);
      const int nb = max((n_vis + kBlock - 1) / kBlock, 0);
      for (int i = max(w0 - n_all, 0) + tid; i < min(nb, w0 + kWindow - n_all); i += 256) {
        const int blk = block_tab[ks.tab_off + i];
        const bool ok = blk >= 0 && blk < n_blocks;          // (a block outside the pool holds no keys)
        list[n_all + i - w0] = BlockItem{ok ? blk : 0, ks.logical_start + kBlock * i,
                                         ok ? min(kBlock, ks.n_tokens - kBlock * i) : 0, s == s_self ? 1 : 0};
      }
      n_all += nb;
    }
    __syncthreads();
    const int n_here = min(n_all - w0, kWindow);
    // two register sets: block i + 4 is loading while block i is used
    if (wave < n_here) {
      BlockItem it0 = list[wave], it1;
      load_block(0, it0);
      for (int i = wave; i < n_here; i += 8) {
        if (i + 4 < n_here) { it1 = list[i + 4]; load_block(1, it1); }
        use_block(0, it0);
        if (i + 4 < n_here) {
          if (i + 8 < n_here) { it0 = list[i + 8]; load_block(0, it0); }
          use_block(1, it1);
        }
      }
    }
    if (w0 + kWindow >= n_all) break;
  }

  // ---- merge the four wavefronts ----
  l += __shfl_xor(l, 16, 64);
  l += __shfl_xor(l, 32, 64);
  l_prior += __shfl_xor(l_prior, 16, 64);
  l_prior += __shfl_xor(l_prior, 32, 64);
  __shared__ float part_m[4][kRowsQ], part_l[4][kRowsQ], part_prior[4][kRowsQ];
  __shared__ float part_o[SCORE ? 1 : 4][SCORE ? 1 : kRowsQ][SCORE ? 1 : D + 4];
  if (g == 0) { part_m[wave][n] = m; part_l[wave][n] = l; part_prior[wave][n] = l_prior; }
  if constexpr (!SCORE) {
#pragma unroll
    for (int c = 0; c < kC; ++c)                     // result register i: dim 16 c + 4 g + i of query n
      *reinterpret_cast<f32x4*>(&part_o[wave][n][16 * c + 4 * g]) = o[c];
  }
  __syncthreads();
  auto weight = [&](int w, int rr, float top) { return part_m[w][rr] == -INFINITY ? 0.f : expf(part_m[w][rr] - top); };
  auto top_of = [&](int rr) { return fmaxf(fmaxf(part_m[0][rr], part_m[1][rr]), fmaxf(part_m[2][rr], part_m[3][rr])); };
  if constexpr (SCORE) {
    if (wave == 0 && g == 0 && row_valid) {
      const float top = top_of(n);
      float z = 0.f, zp = 0.f;
      for (int w = 0; w < 4; ++w) {
        z += part_l[w][n] * weight(w, n, top);
        zp += part_prior[w][n] * weight(w, n, top);
      }
      mass[static_cast<size_t>(row) * hq + h] = zp / z;
    }
  } else {
    // thread -> (query, D/16 dims)
    const int rr = tid / 16, d0 = (tid % 16) * kC;
    const int q0 = cu_q[blockIdx.y] + blockIdx.x * kRowsQ;
    const float top = top_of(rr);
    float wt[4], z = 0.f;
#pragma unroll
    for (int w = 0; w < 4; ++w) { wt[w] = weight(w, rr, top); z += part_l[w][rr] * wt[w]; }
    if (q0 + rr < cu_q[blockIdx.y + 1]) {
      if (out != nullptr) {                          // (a caller that only wants the log-sum-exp passes none)
        T* op = out + (static_cast<size_t>(q0 + rr) * hq + h) * D + d0;
#pragma unroll
        for (int i = 0; i < kC; ++i) {
          float v = 0.f;
#pragma unroll
          for (int w = 0; w < 4; ++w) v += part_o[w][rr][d0 + i] * wt[w];
          op[i] = from_float<T>(v / z);
        }
      }
      if (lse != nullptr && d0 == 0) lse[static_cast<size_t>(q0 + rr) * hq + h] = top + logf(z);
    }
  }
}

}  // namespace

void launch_score_f32(const cc_ctx* ctx, const void* q, const void* k_pool, int n_blocks, const int32_t* block_tab,
                      const cc_segment* segs, int n_segs, const int32_t* req_seg_off, int max_seg_tokens, float* mass,
                      hipStream_t stream) {
  const bool bf = ctx->cfg.dtype == CC_BF16;
  const int d = ctx->cfg.head_dim, hq = ctx->cfg.n_q_heads, hkv = ctx->cfg.n_kv_heads;
  const dim3 grid((max_seg_tokens + kRowsQ - 1) / kRowsQ, n_segs, hq);
#define CC_LAUNCH(T, D)                                                                                     \
  hipLaunchKernelGGL((qk_f32_kernel<T, D, true>), grid, dim3(256), 0, stream, static_cast<const T*>(q),     \
                     static_cast<const int32_t*>(nullptr), static_cast<const int32_t*>(nullptr),            \
                     static_cast<const T*>(k_pool), static_cast<const T*>(nullptr), n_blocks, block_tab, segs, \
                     req_seg_off, hq, hkv, ctx->inv_freq, static_cast<T*>(nullptr), static_cast<float*>(nullptr), mass, \
                     static_cast<const int32_t*>(nullptr), 0, static_cast<const T*>(nullptr), 0, static_cast<const int32_t*>(nullptr))
  if (bf && d == 128) CC_LAUNCH(bf16_t, 128);
  else if (bf && d == 64) CC_LAUNCH(bf16_t, 64);
  else if (!bf && d == 128) CC_LAUNCH(float, 128);
  else CC_LAUNCH(float, 64);
#undef CC_LAUNCH
}

void launch_attn_f32(const cc_ctx* ctx, const void* q, const int32_t* q_pos, const int32_t* cu_q, int max_q_per_req,
                     const void* k_pool, const void* v_pool, int n_blocks, const int32_t* block_tab,
                     const cc_segment* segs, const int32_t* req_seg_off, int n_requests, void* out, float* lse,
                     const int32_t* q_map, int map_pos, hipStream_t stream, const ValueSource& vs) {
  const bool bf = ctx->cfg.dtype == CC_BF16;
  const int d = ctx->cfg.head_dim, hq = ctx->cfg.n_q_heads, hkv = ctx->cfg.n_kv_heads;
  const dim3 grid((max_q_per_req + kRowsQ - 1) / kRowsQ, n_requests, hq);
#define CC_LAUNCH(T, D)                                                                                     \
  hipLaunchKernelGGL((qk_f32_kernel<T, D, false>), grid, dim3(256), 0, stream, static_cast<const T*>(q), q_pos, cu_q, \
                     static_cast<const T*>(k_pool), static_cast<const T*>(v_pool), n_blocks, block_tab, segs, \
                     req_seg_off, hq, hkv, ctx->inv_freq, static_cast<T*>(out), lse, static_cast<float*>(nullptr), q_map, \
                     map_pos, static_cast<const T*>(vs.v_shared), vs.n_shared_blocks, static_cast<const int32_t*>(vs.v_map))
  if (bf && d == 128) CC_LAUNCH(bf16_t, 128);
  else if (bf && d == 64) CC_LAUNCH(bf16_t, 64);
  else if (!bf && d == 128) CC_LAUNCH(float, 128);
  else CC_LAUNCH(float, 64);
#undef CC_LAUNCH
}

}  // namespace cc
