// cc_sparse_prefill, plain kernels: row gather, rotate-and-scatter of the recomputed K/V into the
// paged cache ("fix", Sec. 3.4.3), and the scalar reference-grade attention (per-token form of
// Eq. (1)); Sec. 4 "Selective Token Recomputation".
#include "scatter.h"

namespace cc {

// dst[i] = src[row_idx[i]], 16 bytes per lane.
__global__ __launch_bounds__(256) void gather_rows_kernel(const uint4* __restrict__ src,
                                                          int n_src_rows,
                                                          const int32_t* __restrict__ row_idx,
                                                          int n_rows, int vec_per_row,
                                                          uint4* __restrict__ dst) {
  const int rows_per_block = max(1, 256 / vec_per_row);
  const int v_stride = (vec_per_row >= 256) ? 256 : vec_per_row;
  const int local_row = (vec_per_row >= 256) ? 0 : threadIdx.x / vec_per_row;
  const int v0 = (vec_per_row >= 256) ? threadIdx.x : threadIdx.x % vec_per_row;
  const int row = blockIdx.x * rows_per_block + local_row;
  if (row >= n_rows || local_row >= rows_per_block) return;
  const int s = row_idx[row];
  if (s < 0 || s >= n_src_rows) return;
  const uint4* sp = src + static_cast<size_t>(s) * vec_per_row;
  uint4* dp = dst + static_cast<size_t>(row) * vec_per_row;
  for (int v = v0; v < vec_per_row; v += v_stride) dp[v] = sp[v];
}

void launch_gather_rows(const void* src, int n_src_rows, const int32_t* row_idx, int n_rows,
                        size_t row_bytes, void* dst, hipStream_t stream) {
  const int vec_per_row = static_cast<int>(row_bytes / 16);
  const int rows_per_block = vec_per_row >= 256 ? 1 : 256 / vec_per_row;
  dim3 grid((n_rows + rows_per_block - 1) / rows_per_block);
  hipLaunchKernelGGL(gather_rows_kernel, grid, dim3(256), 0, stream,
                     static_cast<const uint4*>(src), n_src_rows, row_idx, n_rows, vec_per_row,
                     static_cast<uint4*>(dst));
}

template <typename T, int D>
__global__ __launch_bounds__(256) void rope_scatter_kernel(
    const T* __restrict__ k_new, const T* __restrict__ v_new, const int32_t* __restrict__ q_pos,
    const int32_t* __restrict__ slot_map, int n_q_tot, int hkv, InvFreq inv_freq,
    T* __restrict__ k_pool, T* __restrict__ v_pool, int n_blocks, const int32_t* __restrict__ src_rows,
    const T* __restrict__ v_shared, int n_shared_blocks, int32_t* __restrict__ v_map) {
  rope_scatter_rows<T, D>(blockIdx.x, scatter_rows(n_q_tot), k_new, v_new, q_pos, slot_map, n_q_tot, hkv, inv_freq, k_pool, v_pool, n_blocks, src_rows,
                          v_shared, n_shared_blocks, v_map);
}

// Check of the order the scatter relies on: the rows of a 16-token block must form ONE run of
// adjacent list rows.  mark[block] (-1 on entry) takes the first row of the first run that names
// the block; every further run that names it counts as a violation.
__global__ __launch_bounds__(256) void fill_int_kernel(int32_t* __restrict__ p, int n, int32_t v) {
  const int i = blockIdx.x * 256 + threadIdx.x;
  if (i < n) p[i] = v;
}
__global__ __launch_bounds__(256) void list_order_kernel(const int32_t* __restrict__ slot_map, int n_rows,
                                                          int n_blocks, int32_t* __restrict__ mark,
                                                          int32_t* __restrict__ n_violations) {
  const int j = blockIdx.x * 256 + threadIdx.x;
  if (j >= n_rows) return;
  const int slot = slot_map[j];
  if (slot < 0 || slot >= n_blocks * kBlock) return;            // (such rows are skipped by the scatter too)
  const int blk = slot / kBlock;
  if (j > 0) {
    const int prev = slot_map[j - 1];
    if (prev >= 0 && prev < n_blocks * kBlock && prev / kBlock == blk) return;   // not the first row of its run
  }
  if (atomicCAS(&mark[blk], -1, j) != -1) atomicAdd(n_violations, 1);
}

void launch_list_order_check(const int32_t* slot_map, int n_rows, int n_blocks, int32_t* mark,
                             int32_t* n_violations, hipStream_t stream) {
  hipLaunchKernelGGL(fill_int_kernel, dim3((n_blocks + 255) / 256), dim3(256), 0, stream, mark, n_blocks, -1);
  hipLaunchKernelGGL(fill_int_kernel, dim3(1), dim3(256), 0, stream, n_violations, 1, 0);
  if (n_rows > 0)
    hipLaunchKernelGGL(list_order_kernel, dim3((n_rows + 255) / 256), dim3(256), 0, stream, slot_map, n_rows,
                       n_blocks, mark, n_violations);
}

void launch_rope_scatter(const cc_ctx* ctx, const ScatterJob& job, hipStream_t stream) {
  if (job.n_rows <= 0) return;
  const bool bf = ctx->cfg.dtype == CC_BF16;
  const int d = ctx->cfg.head_dim, hkv = ctx->cfg.n_kv_heads;
#define CC_LAUNCH(T, D)                                                                          \
  hipLaunchKernelGGL((rope_scatter_kernel<T, D>), dim3(scatter_groups(job.n_rows)), dim3(256), 0, stream, \
                     static_cast<const T*>(job.k_new), static_cast<const T*>(job.v_new), job.q_pos, job.slot_map, \
                     job.n_rows, hkv, ctx->inv_freq, static_cast<T*>(job.k_pool), static_cast<T*>(job.v_pool),  \
                     job.n_blocks, job.src_rows, static_cast<const T*>(job.vs.v_shared), job.vs.n_shared_blocks, job.vs.v_map)
  if (bf && d == 128) CC_LAUNCH(bf16_t, 128);
  else if (bf && d == 64) CC_LAUNCH(bf16_t, 64);
  else if (!bf && d == 128) CC_LAUNCH(float, 128);
  else CC_LAUNCH(float, 64);
#undef CC_LAUNCH
}

// Scalar attention (CC_IMPL_SCALAR): one wavefront per (query row, query head).  Lane i owns rotation pair
// (i, i + d/2) of q and the same two output dimensions.
template <typename T, int D>
__global__ __launch_bounds__(64) void attn_scalar_kernel(
    const T* __restrict__ q, const int32_t* __restrict__ q_pos, const int32_t* __restrict__ cu_q,
    int n_requests, const T* __restrict__ k_pool, const T* __restrict__ v_pool, int n_blocks,
    const int32_t* __restrict__ block_tab, const cc_segment* __restrict__ segs,
    const int32_t* __restrict__ req_seg_off, int hq, int hkv, InvFreq inv_freq,
    T* __restrict__ out, float* __restrict__ lse, const int32_t* __restrict__ q_map, int map_pos,
    const T* __restrict__ v_shared, int n_shared_blocks, const int32_t* __restrict__ v_map) {
  const int j = blockIdx.x, h = blockIdx.y, lane = threadIdx.x;
  int r = 0;
  while (r + 1 < n_requests && cu_q[r + 1] <= j) ++r;
  if (j >= cu_q[n_requests]) return;                 // (the list may be shorter than its capacity)
  // with a row map, list row j takes its query from row q_map[j] of q (and, if map_pos, its
  // position from q_pos[q_map[j]])
  const int src = q_map != nullptr ? q_map[j] : j;
  const int p = q_pos[map_pos ? src : j];
  const int kvh = h / (hq / hkv);
  const bool own = lane < D / 2;
  float qx = 0.f, qy = 0.f;
  if (own) {
    const T* qp = q + (static_cast<size_t>(src) * hq + h) * D;
    float x = to_float(qp[lane]), y = to_float(qp[lane + D / 2]), c, s;
    rot_cos_sin(p, inv_freq.f[lane], &c, &s);
    qx = x * c - y * s;
    qy = y * c + x * s;
  }
  const float scale = rsqrtf(static_cast<float>(D));
  float m = -INFINITY, z = 0.f, ox = 0.f, oy = 0.f;
  for (int s = req_seg_off[r]; s < req_seg_off[r + 1]; ++s) {
    const cc_segment ks = segs[s];
    const int n_vis = min(ks.n_tokens, p - ks.logical_start + 1);
    for (int tk = 0; tk < n_vis; ++tk) {
      const int blk = block_tab[ks.tab_off + tk / kBlock];
      if (blk < 0 || blk >= n_blocks) continue;
      const size_t bh = static_cast<size_t>(blk) * hkv + kvh;
      const T* kp = k_pool + (bh * kBlock + tk % kBlock) * D;
      float part = own ? qx * to_float(kp[lane]) + qy * to_float(kp[lane + D / 2]) : 0.f;
      const float logit = wave_sum(part) * scale;
      if (logit > m) {
        const float a = expf(m - logit);
        z *= a; ox *= a; oy *= a;
        m = logit;
      }
      const float e = expf(logit - m);
      z += e;
      if (own) {
        const T* vp = value_block<T>(v_pool, v_shared, n_shared_blocks, v_map, blk, static_cast<size_t>(hkv) * D * kBlock) +
                      static_cast<size_t>(kvh) * D * kBlock + tk % kBlock;
        ox += e * to_float(vp[static_cast<size_t>(lane) * kBlock]);
        oy += e * to_float(vp[static_cast<size_t>(lane + D / 2) * kBlock]);
      }
    }
  }
  if (own && out != nullptr) {
    T* op = out + (static_cast<size_t>(j) * hq + h) * D;
    op[lane] = from_float<T>(ox / z);
    op[lane + D / 2] = from_float<T>(oy / z);
  }
  if (lse != nullptr && lane == 0) lse[static_cast<size_t>(j) * hq + h] = m + logf(z);
}

void launch_attn_plain(const cc_ctx* ctx, const void* q, const int32_t* q_pos, const int32_t* cu_q,
                        int n_q_tot, int max_q_per_req, const void* k_pool, const void* v_pool,
                        int n_blocks, const int32_t* block_tab, const cc_segment* segs,
                        const int32_t* req_seg_off, int n_requests, void* out, float* lse,
                        const int32_t* q_map, int map_pos, hipStream_t stream, const ValueSource& vs) {
  if (n_q_tot <= 0) return;
  if (ctx->impl != CC_IMPL_SCALAR) {
    launch_attn_f32(ctx, q, q_pos, cu_q, max_q_per_req, k_pool, v_pool, n_blocks, block_tab, segs, req_seg_off, n_requests,
                    out, lse, q_map, map_pos, stream, vs);
    return;
  }
  const bool bf = ctx->cfg.dtype == CC_BF16;
  const int d = ctx->cfg.head_dim, hq = ctx->cfg.n_q_heads, hkv = ctx->cfg.n_kv_heads;
#define CC_LAUNCH(T, D)                                                                         \
  hipLaunchKernelGGL((attn_scalar_kernel<T, D>), dim3(n_q_tot, hq), dim3(64), 0, stream,        \
                     static_cast<const T*>(q), q_pos, cu_q, n_requests,                         \
                     static_cast<const T*>(k_pool), static_cast<const T*>(v_pool), n_blocks,    \
                     block_tab, segs, req_seg_off, hq, hkv, ctx->inv_freq, static_cast<T*>(out), lse, q_map, map_pos, \
                     static_cast<const T*>(vs.v_shared), vs.n_shared_blocks, vs.v_map)
  if (bf && d == 128) CC_LAUNCH(bf16_t, 128);
  else if (bf && d == 64) CC_LAUNCH(bf16_t, 64);
  else if (!bf && d == 128) CC_LAUNCH(float, 128);
  else CC_LAUNCH(float, 64);
#undef CC_LAUNCH
}

}  // namespace cc
