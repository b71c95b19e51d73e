// Pieces of the FP32 path: LayerNorm rows, and per-query window attention for the
// windows that the FP32 matrix-core attention (k_train_attn.hip) does not hold.  The linears
// are in k_ops_gemm.hip.
#include "dr_device.h"
#include "dr_internal.h"

namespace dr {

// ------------------------------------------------------------------------------------------
// LayerNorm over C channels, biased variance, eps = 1e-5; one wavefront per row.
// Input row r is x[rows ? rows[r] : r]; output row r is compact.
// ------------------------------------------------------------------------------------------
// PER = C / 64 values per lane, fixed at compile time for the network widths, so that a row's
// loads are issued together.  `copy` (if given) receives the row as read.
template <int PER>
__global__ void __launch_bounds__(256) ln_kernel(const float* __restrict__ x, const int32_t* __restrict__ rows,
                                                 const int32_t* __restrict__ nrows_dev, int nrows_max, int C,
                                                 const float* __restrict__ g, const float* __restrict__ b,
                                                 float* __restrict__ y, float* __restrict__ copy) {
  const int lane = threadIdx.x & 63;
  const int r = blockIdx.x * 4 + (threadIdx.x >> 6);
  const int nrows = nrows_dev ? nrows_dev[0] : nrows_max;
  if (r >= nrows) return;
  const int src = rows ? rows[r] : r;
  const float* xr = x + (size_t)src * C;
  constexpr int MAXP = PER ? PER : 16;
  const int per = PER ? PER : C / 64;
  float v[MAXP];
  float s = 0.f;
#pragma unroll
  for (int e = 0; e < MAXP; ++e)
    if (e < per) v[e] = xr[lane + 64 * e];
#pragma unroll
  for (int e = 0; e < MAXP; ++e)
    if (e < per) {
      s += v[e];
      if (copy) copy[(size_t)r * C + lane + 64 * e] = v[e];
    }
  const float mean = wave_sum(s) / C;
  float q = 0.f;
#pragma unroll
  for (int e = 0; e < MAXP; ++e)
    if (e < per) {
      const float d = v[e] - mean;
      q = fmaf(d, d, q);
    }
  const float rstd = rsqrtf(wave_sum(q) / C + 1e-5f);
  float* yr = y + (size_t)r * C;
#pragma unroll
  for (int e = 0; e < MAXP; ++e)
    if (e < per) {
      const int c = lane + 64 * e;
      yr[c] = fmaf((v[e] - mean) * rstd, g[c], b[c]);
    }
}

void launch_ln_f32(const float* x, const int32_t* rows, const int32_t* nrows_dev, int nrows_max,
                   int C, const float* g, const float* b, float* y, hipStream_t s, float* copy) {
  if (nrows_max <= 0) return;
  const int grid = (nrows_max + 3) / 4;
  switch (C) {
    case 64: ln_kernel<1><<<grid, 256, 0, s>>>(x, rows, nrows_dev, nrows_max, C, g, b, y, copy); break;
    case 128: ln_kernel<2><<<grid, 256, 0, s>>>(x, rows, nrows_dev, nrows_max, C, g, b, y, copy); break;
    case 256: ln_kernel<4><<<grid, 256, 0, s>>>(x, rows, nrows_dev, nrows_max, C, g, b, y, copy); break;
    case 384: ln_kernel<6><<<grid, 256, 0, s>>>(x, rows, nrows_dev, nrows_max, C, g, b, y, copy); break;
    default: ln_kernel<0><<<grid, 256, 0, s>>>(x, rows, nrows_dev, nrows_max, C, g, b, y, copy); break;
  }
}

// ------------------------------------------------------------------------------------------
// Window attention, FP32: one wavefront per (window, head, query).  Scores over all S keys of
// the window, softmax with the row max subtracted, then O = P V.
//   q  : compact query rows [Nq, C]          (row woff[w] + j is window w's j-th query)
//   kv : all tokens [N, 2C] window-major     (K in columns [0, C), V in [C, 2C))
//   o  : compact [Nq, C]
// ------------------------------------------------------------------------------------------
__global__ void __launch_bounds__(256) attn_f32_kernel(Geo g, int C, int heads, const float* __restrict__ q,
                                                       const float* __restrict__ kv,
                                                       const int32_t* __restrict__ woff, float* __restrict__ o) {
  __shared__ float qs[4][64];
  __shared__ float ps[4][320];
  const int lane = threadIdx.x & 63, wv = threadIdx.x >> 6;
  const int w = blockIdx.x / heads, h = blockIdx.x - w * heads;
  const int j = blockIdx.y * 4 + wv;
  const int q0 = woff[w], nqw = woff[w + 1] - q0;
  if (j >= nqw) return;
  const int dh = C / heads;
  const int r = q0 + j;
  const float scale = rsqrtf((float)dh);
  if (lane < dh) qs[wv][lane] = q[(size_t)r * C + h * dh + lane];
  __builtin_amdgcn_wave_barrier();
  const float* kbase = kv + (size_t)w * g.S * 2 * C + h * dh;
  float mx = -INFINITY;
  for (int s = lane; s < g.S; s += 64) {
    const float* kr = kbase + (size_t)s * 2 * C;
    float d = 0.f;
    for (int e = 0; e < dh; ++e) d = fmaf(qs[wv][e], kr[e], d);
    d *= scale;
    ps[wv][s] = d;
    mx = fmaxf(mx, d);
  }
  mx = wave_max(mx);
  float sum = 0.f;
  for (int s = lane; s < g.S; s += 64) {
    const float e = expf(ps[wv][s] - mx);
    ps[wv][s] = e;
    sum += e;
  }
  sum = wave_sum(sum);
  __builtin_amdgcn_wave_barrier();
  if (lane < dh) {
    const float* vbase = kbase + C + lane;
    float acc = 0.f;
    for (int s = 0; s < g.S; ++s) acc = fmaf(ps[wv][s], vbase[(size_t)s * 2 * C], acc);
    o[(size_t)r * C + h * dh + lane] = acc / sum;
  }
}

void launch_attn_f32(const Geo& g, int C, int heads, const float* q, const float* kv,
                     const int32_t* woff, float* o, hipStream_t s) {
  dim3 grid(g.nwin * heads, (g.S + 3) / 4);
  attn_f32_kernel<<<grid, 256, 0, s>>>(g, C, heads, q, kv, woff, o);
}

}  // namespace dr
