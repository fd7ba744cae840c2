// cc_select, plain kernels: per-token prior-chunk attention mass (scalar reference-grade path)
// and the per-chunk top-N (Eq. (2), Eq. (10), Sec. 3.2.1).
#include "device_util.h"
#include "topn.h"

namespace cc {

// ---------------------------------------------------------------------------------------------
// Scalar score kernel: one wavefront per (chunk token, query head).  Lane i owns rotation pair
// (i, i + d/2) of the query; keys of the request are visited in logical order, each logit is a
// wavefront reduction.  Runs when CC_IMPL_SCALAR asks for it.
// ---------------------------------------------------------------------------------------------
template <typename T, int D>
__global__ __launch_bounds__(64) void score_scalar_kernel(
    const T* __restrict__ q, const T* __restrict__ k_pool, int n_blocks,
    const int32_t* __restrict__ block_tab, const cc_segment* __restrict__ segs,
    const int32_t* __restrict__ req_seg_off, int hq, int hkv, InvFreq inv_freq,
    float* __restrict__ mass) {
  const cc_segment sg = segs[blockIdx.y];
  const int t = blockIdx.x, h = blockIdx.z, lane = threadIdx.x;
  if (sg.kind != CC_SEG_CHUNK || t >= sg.n_tokens) return;
  const size_t row = static_cast<size_t>(sg.tok_off) + t;
  if (sg.logical_start == 0) {              // first chunk: no prior chunk to attend to
    if (lane == 0) mass[row * hq + h] = 0.f;
    return;
  }
  const int p = sg.logical_start + t;
  const int kvh = h / (hq / hkv);
  const bool own = lane < D / 2;
  float qx = 0.f, qy = 0.f;
  if (own) {
    const T* qp = q + (row * hq + h) * D;
    float x = to_float(qp[lane]), y = to_float(qp[lane + D / 2]), c, s;
    rot_cos_sin(p, inv_freq.f[lane], &c, &s);
    qx = x * c - y * s;
    qy = y * c + x * s;
  }
  const float scale = rsqrtf(static_cast<float>(D));
  float m = -INFINITY, z_prior = 0.f, z_all = 0.f;
  const int s_begin = req_seg_off[sg.req], s_self = blockIdx.y;
  for (int s = s_begin; s <= s_self; ++s) {
    const cc_segment ks = segs[s];
    const int n_vis = min(ks.n_tokens, p - ks.logical_start + 1);
    float z_seg = 0.f;
    for (int tk = 0; tk < n_vis; ++tk) {
      const int blk = block_tab[ks.tab_off + tk / kBlock];
      if (blk < 0 || blk >= n_blocks) continue;
      const T* kp = k_pool + ((static_cast<size_t>(blk) * hkv + kvh) * kBlock + tk % kBlock) * D;
      float part = own ? qx * to_float(kp[lane]) + qy * to_float(kp[lane + D / 2]) : 0.f;
      const float logit = wave_sum(part) * scale;
      if (logit > m) {                       // wave-uniform
        const float a = expf(m - logit);
        z_all *= a; z_seg *= a; z_prior *= a;
        m = logit;
      }
      const float e = expf(logit - m);
      z_all += e; z_seg += e;
    }
    if (s < s_self) z_prior += z_seg;
  }
  if (lane == 0) mass[row * hq + h] = z_prior / z_all;
}

template <typename T, int D>
static void launch_score_t(const cc_ctx* ctx, const void* q, const void* k_pool, int n_blocks,
                           const int32_t* block_tab, const cc_segment* segs, int n_segs,
                           const int32_t* req_seg_off, int max_seg_tokens, float* mass,
                           hipStream_t stream) {
  dim3 grid(max_seg_tokens, n_segs, ctx->cfg.n_q_heads);
  hipLaunchKernelGGL((score_scalar_kernel<T, D>), grid, dim3(64), 0, stream,
                     static_cast<const T*>(q), static_cast<const T*>(k_pool), n_blocks, block_tab,
                     segs, req_seg_off, ctx->cfg.n_q_heads, ctx->cfg.n_kv_heads, ctx->inv_freq, mass);
}

void launch_score_plain(const cc_ctx* ctx, const void* q, const void* k_pool, int n_blocks,
                         const int32_t* block_tab, const cc_segment* segs, int n_segs,
                         const int32_t* req_seg_off, int max_seg_tokens, float* mass,
                         hipStream_t stream) {
  const bool bf = ctx->cfg.dtype == CC_BF16;
  const int d = ctx->cfg.head_dim;
#define CC_ARGS ctx, q, k_pool, n_blocks, block_tab, segs, n_segs, req_seg_off, max_seg_tokens, mass, stream
  if (ctx->impl != CC_IMPL_SCALAR) launch_score_f32(CC_ARGS);
  else if (bf && d == 128) launch_score_t<bf16_t, 128>(CC_ARGS);
  else if (bf && d == 64) launch_score_t<bf16_t, 64>(CC_ARGS);
  else if (!bf && d == 128) launch_score_t<float, 128>(CC_ARGS);
  else launch_score_t<float, 64>(CC_ARGS);
#undef CC_ARGS
}

__global__ __launch_bounds__(256) void topn_kernel(
    const float* __restrict__ mass, int hq, bool given, const int32_t* __restrict__ block_tab,
    const cc_segment* __restrict__ segs, int32_t* __restrict__ sel_idx, int32_t* __restrict__ q_row,
    int32_t* __restrict__ q_pos, int32_t* __restrict__ slot_map, float* __restrict__ scores,
    uint32_t* key_buf) {
  topn_block<4>(blockIdx.x, mass, hq, given, block_tab, segs, sel_idx, q_row, q_pos, slot_map, scores, key_buf);
}

void launch_topn(const cc_ctx* ctx, const float* mass, const TopnJob& job, bool given, hipStream_t stream) {
  hipLaunchKernelGGL(topn_kernel, dim3(job.n_segs), dim3(256), 0, stream, mass, ctx->cfg.n_q_heads, given, job.block_tab,
                     job.segs, job.sel_idx, job.q_row, job.q_pos, job.slot_map, job.scores, job.key_buf);
}

}  // namespace cc
