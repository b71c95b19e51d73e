// Training kernels (FP32): the pieces of the hand-written reverse pass of the inpainting
// network.  Weight gradients are reductions over tokens; they are computed deterministically
// (fixed chunks of rows, then the chunk partials summed in order), so a gradient does not
// depend on launch timing or on which other clips share the batch.
#include <algorithm>

#include "dr_device.h"
#include "dr_internal.h"

namespace dr {

// ------------------------------------------------------------------------------------------
// Y[r, :] = X[rows[r], :] for r < *n (gather of residual rows)
// ------------------------------------------------------------------------------------------
__global__ void gather_rows_kernel(const float* __restrict__ X, const int32_t* __restrict__ rows,
                                   const int32_t* __restrict__ n_dev, int n_max, int C, float* __restrict__ Y) {
  const int n = n_dev ? n_dev[0] : n_max;
  for (size_t e = blockIdx.x * (size_t)blockDim.x + threadIdx.x; e < (size_t)n * C; e += (size_t)gridDim.x * blockDim.x) {
    const size_t r = e / C, c = e - r * C;
    Y[e] = X[(size_t)rows[r] * C + c];
  }
}

void launch_gather_rows(const float* X, const int32_t* rows, const int32_t* n_dev, int n_max, int C, float* Y,
                        hipStream_t s) {
  size_t grid = ((size_t)n_max * C + 255) / 256;
  if (grid > 8192) grid = 8192;
  if (grid) gather_rows_kernel<<<(unsigned)grid, 256, 0, s>>>(X, rows, n_dev, n_max, C, Y);
}

// X[rows[r], :] = Y[r, :] (scatter-replace)
__global__ void scatter_rows_kernel(const float* __restrict__ Y, const int32_t* __restrict__ rows,
                                    const int32_t* __restrict__ n_dev, int C, float* __restrict__ X) {
  const int n = n_dev[0];
  for (size_t e = blockIdx.x * (size_t)blockDim.x + threadIdx.x; e < (size_t)n * C; e += (size_t)gridDim.x * blockDim.x) {
    const size_t r = e / C, c = e - r * C;
    X[(size_t)rows[r] * C + c] = Y[e];
  }
}

void launch_scatter_rows(const float* Y, const int32_t* rows, const int32_t* n_dev, int n_max, int C, float* X,
                         hipStream_t s) {
  size_t grid = ((size_t)n_max * C + 255) / 256;
  if (grid > 8192) grid = 8192;
  if (grid) scatter_rows_kernel<<<(unsigned)grid, 256, 0, s>>>(Y, rows, n_dev, C, X);
}

// ------------------------------------------------------------------------------------------
// elementwise, four values per thread: a = GELU(h); and in the reverse pass d = d GELU'(h),
// GELU'(z) = Phi(z) + z phi(z), with a = GELU(h) again from the same error function (as two
// passes 35 + 58 us at 18,800 rows of 1,024; in the epilogue of the product that makes d, which
// its two blocks per CU do not hide, about 100 us)
// ------------------------------------------------------------------------------------------
__global__ void __launch_bounds__(256) gelu_fwd_kernel(const float* __restrict__ h, const int32_t* __restrict__ n_dev,
                                                       int R, float* __restrict__ a) {
  const size_t n = (size_t)n_dev[0] * R / 4;
  for (size_t e = blockIdx.x * (size_t)blockDim.x + threadIdx.x; e < n; e += (size_t)gridDim.x * blockDim.x) {
    const float4 z = reinterpret_cast<const float4*>(h)[e];
    reinterpret_cast<float4*>(a)[e] = make_float4(gelu_erf(z.x), gelu_erf(z.y), gelu_erf(z.z), gelu_erf(z.w));
  }
}

__device__ __forceinline__ void gelu_grad(float z, float& d, float& a) {
  const float e1 = 1.0f + erff(z * 0.70710678118654752f);
  a = 0.5f * z * e1;
  const float cdf = 0.5f * e1;
  const float pdf = 0.3989422804014327f * expf(-0.5f * z * z);
  d *= cdf + z * pdf;
}

__global__ void __launch_bounds__(256) gelu_bwd_kernel(const float* __restrict__ h, const int32_t* __restrict__ n_dev,
                                                       int R, float* __restrict__ d, float* __restrict__ a) {
  const size_t n = (size_t)n_dev[0] * R / 4;
  for (size_t e = blockIdx.x * (size_t)blockDim.x + threadIdx.x; e < n; e += (size_t)gridDim.x * blockDim.x) {
    const float4 z = reinterpret_cast<const float4*>(h)[e];
    float4 g = reinterpret_cast<const float4*>(d)[e], y;
    gelu_grad(z.x, g.x, y.x);
    gelu_grad(z.y, g.y, y.y);
    gelu_grad(z.z, g.z, y.z);
    gelu_grad(z.w, g.w, y.w);
    reinterpret_cast<float4*>(d)[e] = g;
    reinterpret_cast<float4*>(a)[e] = y;
  }
}

static unsigned gelu_grid(int n_max, int R) { return (unsigned)std::min<size_t>(((size_t)n_max * R / 4 + 255) / 256, 8192); }

void launch_gelu_fwd(const float* h, const int32_t* n_dev, int n_max, int R, float* a, hipStream_t s) {
  if (n_max > 0) gelu_fwd_kernel<<<gelu_grid(n_max, R), 256, 0, s>>>(h, n_dev, R, a);
}

void launch_gelu_bwd(const float* h, const int32_t* n_dev, int n_max, int R, float* d, float* a, hipStream_t s) {
  if (n_max > 0) gelu_bwd_kernel<<<gelu_grid(n_max, R), 256, 0, s>>>(h, n_dev, R, d, a);
}

// ------------------------------------------------------------------------------------------
// LayerNorm backward, one wavefront per row r < *n_dev (or n_max):
// dx[r] = (acc ? acc[r] : 0) + rstd * (dxh - mean(dxh) - xh * mean(dxh * xh)), dxh = dy * gamma
// (acc may be dx).  dgamma/dbeta partials per block of LNB_ROWS rows:
// part[blk][0..C) = sum dy*xh, part[blk][C..2C) = sum dy.  PER = C / 64 values per lane, fixed
// at compile time for the network widths so that a row's loads are issued together.
// ------------------------------------------------------------------------------------------
template <int PER>
__global__ void __launch_bounds__(256) ln_bwd_kernel(const float* __restrict__ x, const int32_t* __restrict__ n_dev,
                                                     int n_max, int C, const float* __restrict__ g,
                                                     const float* __restrict__ dy, const float* acc, float* dx,
                                                     float* __restrict__ part) {
  // every rounding is as written here, whatever the unrolling
#pragma clang fp contract(off)
  extern __shared__ float red[];  // [4][2C]
  const int lane = threadIdx.x & 63, wv = threadIdx.x >> 6;
  const int n = n_dev ? n_dev[0] : n_max;
  if (blockIdx.x * LNB_ROWS >= n) return;  // uniform per block
  constexpr int MAXP = PER ? PER : 16;
  const int per = PER ? PER : C / 64;
  float pg[MAXP], pb[MAXP], gm[MAXP];
#pragma unroll
  for (int e = 0; e < MAXP; ++e)
    if (e < per) {
      pg[e] = pb[e] = 0.f;
      gm[e] = g[lane + 64 * e];
    }
  for (int rr = 0; rr < LNB_ROWS / 4; ++rr) {
    const int r = blockIdx.x * LNB_ROWS + rr * 4 + wv;
    if (r >= n) break;
    const size_t at = (size_t)r * C + lane;
    float v[MAXP], d[MAXP], o[MAXP];
    float s = 0.f;
#pragma unroll
    for (int e = 0; e < MAXP; ++e)
      if (e < per) {
        v[e] = x[at + 64 * e];
        d[e] = dy[at + 64 * e];
        o[e] = acc ? acc[at + 64 * e] : 0.f;
      }
#pragma unroll
    for (int e = 0; e < MAXP; ++e)
      if (e < per) s += v[e];
    const float mean = wave_sum(s) / C;
    float q = 0.f;
#pragma unroll
    for (int e = 0; e < MAXP; ++e)
      if (e < per) {
        const float t = v[e] - mean;
        q = fmaf(t, t, q);
      }
    const float rstd = rsqrtf(wave_sum(q) / C + 1e-5f);
    float s1 = 0.f, s2 = 0.f;
#pragma unroll
    for (int e = 0; e < MAXP; ++e)
      if (e < per) {
        const float xh = (v[e] - mean) * rstd;
        const float dyv = d[e];
        d[e] = dyv * gm[e];
        s1 = fmaf(dyv, gm[e], s1);
        s2 = fmaf(d[e], xh, s2);
        pg[e] = fmaf(dyv, xh, pg[e]);
        pb[e] += dyv;
        v[e] = xh;
      }
    s1 = wave_sum(s1) / C;
    s2 = wave_sum(s2) / C;
#pragma unroll
    for (int e = 0; e < MAXP; ++e)
      if (e < per) {
        const float val = rstd * fmaf(-v[e], s2, d[e] - s1);
        dx[at + 64 * e] = acc ? o[e] + val : val;
      }
  }
  // fixed-order block reduction of the dgamma / dbeta partials
#pragma unroll
  for (int e = 0; e < MAXP; ++e)
    if (e < per) {
      red[wv * 2 * C + lane + 64 * e] = pg[e];
      red[wv * 2 * C + C + lane + 64 * e] = pb[e];
    }
  __syncthreads();
  for (int c = threadIdx.x; c < 2 * C; c += blockDim.x)
    part[(size_t)blockIdx.x * 2 * C + c] = red[c] + red[2 * C + c] + red[4 * C + c] + red[6 * C + c];
}

void launch_ln_bwd(const float* x, const int32_t* n_dev, int n_max, int C, const float* g, const float* dy,
                   const float* acc, float* dx, float* part, hipStream_t s) {
  const int blocks = ln_bwd_blocks(n_max);
  if (blocks <= 0) return;
  const size_t lds = 4 * 2 * C * sizeof(float);
  switch (C) {
    case 64: ln_bwd_kernel<1><<<blocks, 256, lds, s>>>(x, n_dev, n_max, C, g, dy, acc, dx, part); break;
    case 128: ln_bwd_kernel<2><<<blocks, 256, lds, s>>>(x, n_dev, n_max, C, g, dy, acc, dx, part); break;
    case 256: ln_bwd_kernel<4><<<blocks, 256, lds, s>>>(x, n_dev, n_max, C, g, dy, acc, dx, part); break;
    case 384: ln_bwd_kernel<6><<<blocks, 256, lds, s>>>(x, n_dev, n_max, C, g, dy, acc, dx, part); break;
    default: ln_bwd_kernel<0><<<blocks, 256, lds, s>>>(x, n_dev, n_max, C, g, dy, acc, dx, part); break;
  }
}

// out[c] = sum of part[b * stride + c] over the parts in use: all nparts, or with n_dev the first
// ceil(*n_dev / rows_per).  Four interleaved sums (part b of the first nparts / 4 * 4 in sum
// b mod 4, the rest in sum 0) combined in a fixed order, so the result depends on nothing but
// the values.  The four sums of a column run in four threads, each with eight loads in flight:
// as one chain per column this took 25 us on average in a 4-clip training step, mostly latency.
__global__ void __launch_bounds__(256) sum_parts_kernel(const float* __restrict__ part, int nparts,
                                                        size_t stride, const int32_t* __restrict__ n_dev, int rows_per,
                                                        int width, float* __restrict__ out) {
  __shared__ float sums[4][64];
  const int col = threadIdx.x & 63, q = threadIdx.x >> 6, c = blockIdx.x * 64 + col;
  const int used = n_dev ? min(nparts, (n_dev[0] + rows_per - 1) / rows_per) : nparts;
  const int n4 = nparts & ~3, end = min(used, n4);
  float a = 0.f;
  if (c < width) {
    const float* p = part + c;
    int b = q;
    for (; b + 28 < end; b += 32) {
      float v[8];
#pragma unroll
      for (int u = 0; u < 8; ++u) v[u] = p[(b + 4 * u) * stride];
#pragma unroll
      for (int u = 0; u < 8; ++u) a += v[u];
    }
    for (; b < end; b += 4) a += p[b * stride];
    if (q == 0)
      for (b = n4; b < used; ++b) a += p[b * stride];
  }
  sums[q][col] = a;
  __syncthreads();
  if (q == 0 && c < width) {
    out[c] = (sums[0][col] + sums[1][col]) + (sums[2][col] + sums[3][col]);
  }
}

void launch_sum_parts(const float* part, int nparts, size_t stride, const int32_t* n_dev, int rows_per, int width,
                      float* out, hipStream_t s) {
  if (width <= 0) return;
  sum_parts_kernel<<<(width + 63) / 64, 256, 0, s>>>(part, nparts, stride, n_dev, rows_per, width, out);
}

// ------------------------------------------------------------------------------------------
// Column sums: out[j] = sum_m B[m][j] over m < *M (or M_max), partials per TN_CHUNK rows.
// ------------------------------------------------------------------------------------------
// One block per (64 columns, chunk): 16 row groups of 64 lanes, each lane summing every 16th
// row of its column with 8 independent partial sums (loads in flight together), then a fixed
// order reduction of the groups in LDS (deterministic).
__global__ void __launch_bounds__(1024) colsum_partial_kernel(const float* __restrict__ B, int ldb,
                                                              const int32_t* __restrict__ M_dev, int M_max, int J,
                                                              float* __restrict__ part) {
  __shared__ float red[16][64];
  const int M = M_dev ? M_dev[0] : M_max;
  const int col = threadIdx.x & 63, grp = threadIdx.x >> 6;
  const int j = blockIdx.x * 64 + col;
  const int chunk = blockIdx.y;
  if (chunk * TN_CHUNK >= M) return;  // uniform per block
  const int m_begin = chunk * TN_CHUNK, m_end = min(M, m_begin + TN_CHUNK);
  float acc[8];
#pragma unroll
  for (int u = 0; u < 8; ++u) acc[u] = 0.f;
  if (j < J) {
    int m = m_begin + grp;
    for (; m + 7 * 16 < m_end; m += 8 * 16)
#pragma unroll
      for (int u = 0; u < 8; ++u) acc[u] += B[(size_t)(m + 16 * u) * ldb + j];
    for (; m < m_end; m += 16) acc[0] += B[(size_t)m * ldb + j];
  }
  red[grp][col] = ((acc[0] + acc[1]) + (acc[2] + acc[3])) + ((acc[4] + acc[5]) + (acc[6] + acc[7]));
  __syncthreads();
  if (grp == 0 && j < J) {
    float t = 0.f;
    for (int g = 0; g < 16; ++g) t += red[g][col];
    part[(size_t)chunk * J + j] = t;
  }
}

void launch_colsum_partial(const float* B, int ldb, const int32_t* M_dev, int M_max, int J, float* part,
                           hipStream_t s) {
  const int chunks = tn_chunks(M_max);
  if (chunks <= 0) return;
  colsum_partial_kernel<<<dim3((J + 63) / 64, chunks), 1024, 0, s>>>(B, ldb, M_dev, M_max, J, part);
}

// ------------------------------------------------------------------------------------------
// Pixel-side pieces.  Patches of the cut-out input [N][48] (k = (ky*4 + kx)*3 + c), and the
// decoder's pre-activation gradient per token: dyt[n][k] = dpred * pred * (1 - pred) at the
// token's pixels.  Also the full-frame decoder (all tokens) for the training forward:
// pred = sigmoid(z W_dec + b) written to every pixel.
// ------------------------------------------------------------------------------------------
__device__ __forceinline__ size_t tok_pixel(const Geo& g, int n) {
  int w = n / g.S, s = n - w * g.S;
  int v = w % g.nww;
  int r = w / g.nww;
  int u = r % g.nwh;
  r /= g.nwh;
  int nT = g.T / g.wt;
  int a = r % nT;
  int b = r / nT;
  int dj = s % g.ww;
  int q = s / g.ww;
  int di = q % g.wh;
  int dt = q / g.wh;
  int t = a * g.wt + dt, i = u * g.wh + di, j = v * g.ww + dj;
  return (((size_t)b * g.T + t) * g.H + (size_t)4 * i) * g.W + (size_t)4 * j;
}

__global__ void patches_kernel(Geo g, const float* __restrict__ frames, const uint8_t* __restrict__ masks,
                               float* __restrict__ P) {
  for (size_t e = blockIdx.x * (size_t)blockDim.x + threadIdx.x; e < (size_t)g.N * 48; e += (size_t)gridDim.x * blockDim.x) {
    const int n = (int)(e / 48), k = (int)(e % 48);
    const int pix = k / 3, c = k - 3 * pix, ky = pix >> 2, kx = pix & 3;
    const size_t px = tok_pixel(g, n) + (size_t)ky * g.W + kx;
    P[e] = masks[px] ? 0.f : frames[px * 3 + c];
  }
}

void launch_patches(const Geo& g, const float* frames, const uint8_t* masks, float* P, hipStream_t s) {
  size_t grid = ((size_t)g.N * 48 + 255) / 256;
  if (grid > 8192) grid = 8192;
  patches_kernel<<<(unsigned)grid, 256, 0, s>>>(g, frames, masks, P);
}

// Full-frame decoder: 48 threads (one per output of a token) x 4 groups of DEC_TOK tokens per
// block; z rows and the weight's 48 columns go through LDS in 64-channel slices, and a weight
// value serves DEC_TOK tokens (one output per thread, reading its row and column from memory,
// took 605 us at 129,600 tokens of 256).  Each output is one chain of fused multiply-adds over
// the channels in order.
constexpr int DEC_TOK = 8;
__global__ void __launch_bounds__(192) decoder_full_kernel(Geo g, int C, const float* __restrict__ z,
                                                           const float* __restrict__ dw, const float* __restrict__ db,
                                                           float* __restrict__ pred) {
  __shared__ __align__(16) float zs[4 * DEC_TOK][64];
  __shared__ float ws[64][48];
  const int t = threadIdx.x, grp = t / 48, k = t - 48 * grp;
  const int pix = k / 3, c = k - 3 * pix, ky = pix >> 2, kx = pix & 3;
  const int n0 = blockIdx.x * 4 * DEC_TOK;
  float acc[DEC_TOK];
#pragma unroll
  for (int u = 0; u < DEC_TOK; ++u) acc[u] = db[c];
  for (int i0 = 0; i0 < C; i0 += 64) {
    for (int e = t; e < 4 * DEC_TOK * 16; e += 192) {
      const int row = e >> 4, col = (e & 15) * 4;
      *reinterpret_cast<float4*>(&zs[row][col]) =
          *reinterpret_cast<const float4*>(z + (size_t)min(n0 + row, g.N - 1) * C + i0 + col);
    }
    for (int e = t; e < 64 * 48; e += 192) (&ws[0][0])[e] = dw[(size_t)i0 * 48 + e];
    __syncthreads();
#pragma unroll 4
    for (int i = 0; i < 64; i += 4) {
      float w[4];
#pragma unroll
      for (int e = 0; e < 4; ++e) w[e] = ws[i + e][k];
#pragma unroll
      for (int u = 0; u < DEC_TOK; ++u) {
        const float4 zv = *reinterpret_cast<const float4*>(&zs[grp * DEC_TOK + u][i]);
        acc[u] = fmaf(zv.x, w[0], acc[u]);
        acc[u] = fmaf(zv.y, w[1], acc[u]);
        acc[u] = fmaf(zv.z, w[2], acc[u]);
        acc[u] = fmaf(zv.w, w[3], acc[u]);
      }
    }
    __syncthreads();
  }
#pragma unroll
  for (int u = 0; u < DEC_TOK; ++u) {
    const int n = n0 + grp * DEC_TOK + u;
    if (n < g.N) {
      const size_t px = tok_pixel(g, n) + (size_t)ky * g.W + kx;
      pred[px * 3 + c] = 1.0f / (1.0f + expf(-acc[u]));
    }
  }
}

void launch_decoder_full(const Geo& g, int C, const float* z, const float* dw, const float* db, float* pred,
                         hipStream_t s) {
  if (g.N > 0) decoder_full_kernel<<<(g.N + 4 * DEC_TOK - 1) / (4 * DEC_TOK), 192, 0, s>>>(g, C, z, dw, db, pred);
}

__global__ void dec_grad_tok_kernel(Geo g, const float* __restrict__ pred, const float* __restrict__ dpred,
                                    float* __restrict__ dyt) {
  for (size_t e = blockIdx.x * (size_t)blockDim.x + threadIdx.x; e < (size_t)g.N * 48; e += (size_t)gridDim.x * blockDim.x) {
    const int n = (int)(e / 48), k = (int)(e % 48);
    const int pix = k / 3, c = k - 3 * pix, ky = pix >> 2, kx = pix & 3;
    const size_t i = (tok_pixel(g, n) + (size_t)ky * g.W + kx) * 3 + c;
    const float p = pred[i];
    dyt[e] = dpred[i] * p * (1.0f - p);
  }
}

void launch_dec_grad_tok(const Geo& g, const float* pred, const float* dpred, float* dyt, hipStream_t s) {
  size_t grid = ((size_t)g.N * 48 + 255) / 256;
  if (grid > 8192) grid = 8192;
  dec_grad_tok_kernel<<<(unsigned)grid, 256, 0, s>>>(g, pred, dpred, dyt);
}

// ------------------------------------------------------------------------------------------
// L1 training loss: L = w_in mean_{m!=0}|pred - gt| + w_out mean_{m==0}|pred - gt| over
// pixel-channel values, and dL/dpred = w * sign(pred - gt) / count (sign(0) = 0; an empty
// region contributes nothing).  Two passes: counts and partial sums per block (fixed order),
// then the gradient.  acc[0..3] = (sum_in, sum_out, n_in, n_out) after the reduction.
// ------------------------------------------------------------------------------------------
constexpr int L1_BLOCKS = 1024;

__global__ void l1_partial_kernel(const float* __restrict__ pred, const float* __restrict__ gt,
                                  const uint8_t* __restrict__ masks, size_t npix, float* __restrict__ part) {
  __shared__ float sh[4][256];
  float si = 0.f, so = 0.f, ni = 0.f, no = 0.f;
  for (size_t p = blockIdx.x * (size_t)blockDim.x + threadIdx.x; p < npix; p += (size_t)gridDim.x * blockDim.x) {
    const bool in = masks[p] != 0;
    float e = 0.f;
    for (int c = 0; c < 3; ++c) e += fabsf(pred[3 * p + c] - gt[3 * p + c]);
    if (in) {
      si += e;
      ni += 3.f;
    } else {
      so += e;
      no += 3.f;
    }
  }
  sh[0][threadIdx.x] = si;
  sh[1][threadIdx.x] = so;
  sh[2][threadIdx.x] = ni;
  sh[3][threadIdx.x] = no;
  __syncthreads();
  for (int st = 128; st > 0; st >>= 1) {
    if (threadIdx.x < st)
      for (int k = 0; k < 4; ++k) sh[k][threadIdx.x] += sh[k][threadIdx.x + st];
    __syncthreads();
  }
  if (threadIdx.x < 4) part[blockIdx.x * 4 + threadIdx.x] = sh[threadIdx.x][0];
}

__global__ void l1_final_kernel(const float* __restrict__ part, int nb, float w_in, float w_out,
                                float* __restrict__ acc, float* __restrict__ loss) {
  // the four sums run in four threads, over partials that the block has brought to LDS
  __shared__ float sh[4 * L1_BLOCKS];
  __shared__ double s[4];
  for (int e = threadIdx.x; e < 4 * nb; e += blockDim.x) sh[e] = part[e];
  __syncthreads();
  if (threadIdx.x < 4) {
    double t = 0;
#pragma unroll 16
    for (int b = 0; b < nb; ++b) t += sh[b * 4 + threadIdx.x];
    s[threadIdx.x] = t;
    acc[threadIdx.x] = (float)t;
  }
  __syncthreads();
  if (threadIdx.x != 0) return;
  double L = 0.0;
  if (s[2] > 0) L += w_in * s[0] / s[2];
  if (s[3] > 0) L += w_out * s[1] / s[3];
  loss[0] = (float)L;
}

__global__ void l1_grad_kernel(const float* __restrict__ pred, const float* __restrict__ gt,
                               const uint8_t* __restrict__ masks, size_t npix, float w_in, float w_out,
                               const float* __restrict__ acc, float* __restrict__ dpred) {
  const float gi = acc[2] > 0.f ? w_in / acc[2] : 0.f;
  const float go = acc[3] > 0.f ? w_out / acc[3] : 0.f;
  for (size_t e = blockIdx.x * (size_t)blockDim.x + threadIdx.x; e < 3 * npix; e += (size_t)gridDim.x * blockDim.x) {
    const float d = pred[e] - gt[e];
    const float sg = d > 0.f ? 1.f : (d < 0.f ? -1.f : 0.f);
    dpred[e] = sg * (masks[e / 3] ? gi : go);
  }
}

void launch_l1_loss(const float* pred, const float* gt, const uint8_t* masks, size_t npix, float w_in, float w_out,
                    float* part, float* acc, float* loss, float* dpred, hipStream_t s) {
  l1_partial_kernel<<<L1_BLOCKS, 256, 0, s>>>(pred, gt, masks, npix, part);
  l1_final_kernel<<<1, 256, 0, s>>>(part, L1_BLOCKS, w_in, w_out, acc, loss);
  if (dpred) {
    size_t grid = (3 * npix + 255) / 256;
    if (grid > 8192) grid = 8192;
    l1_grad_kernel<<<(unsigned)grid, 256, 0, s>>>(pred, gt, masks, npix, w_in, w_out, acc, dpred);
  }
}

}  // namespace dr
