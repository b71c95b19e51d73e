// Products of FP32 matrices on the bf16 matrix cores: the linears of the FP32 path and every
// weight product of the training passes (linears, input gradients, weight gradients).
//
// Two arithmetics share the kernels, by the number of bf16 planes NP an operand is split into:
//
//   NP = 3 (FP32): a = a1 + a2 + a3 exactly (8 + 8 + 8 significant bits: a1 the truncated
//     upper half of the float, a2 and a3 the rounded remainders), and
//     a w ~ a3 w1 + a2 w2 + a1 w3 + a2 w1 + a1 w2 + a1 w1, six v_mfma_f32_16x16x32_bf16 per
//     32-wide k step with FP32 accumulation, the small terms first.  The dropped terms are
//     below 2^-22 |a w|, under the rounding of one FP32 accumulation, and a k step rounds its
//     accumulator 6 times where a chain of FP32 fused multiply-adds rounds it 32 times.  Six
//     bf16 products cost 96 matrix cycles per 16 x 16 x 32 step where v_mfma_f32_16x16x4_f32
//     costs 256 (and the vector ALU as much).  A result that is not a number (an operand, or a sum, outside the finite
//     range) is recomputed by the fused multiply-adds, so infinities come out as they do there.
//   NP = 1 (mixed precision): operands rounded to bf16 to nearest even, one product.
//
// Block = 4 wavefronts (2 x 2), BM x BN outputs, k in steps of 32.  Operands are read from
// global memory into registers one step ahead, split there, and written to LDS as bf16 planes
// (the split is done once per block and element, not once per wavefront); two blocks per CU
// hide each other's barriers.  A row of 32 k values is 64 bytes, two rows share a 128-byte
// line, and the line's eight 16-byte chunks are XOR-swizzled by the line number, so the 16
// rows of an operand fragment fall on distinct banks.
#include "dr_device.h"
#include "dr_internal.h"
#include "gemm_core.h"

namespace dr {

template <int BM_, int BN_, int NP_>
struct OpsTile {
  static constexpr int BM = BM_, BN = BN_, NP = NP_, THREADS = 256;
  static constexpr int FM = BM / 32, FN = BN / 32;  // 16 x 16 fragments per wavefront
  static constexpr int SA = BM * 4 / THREADS, SW = BN * 4 / THREADS;  // 8-value chunks per thread and step
  static constexpr int PLANE = (BM + BN) * 32;      // bf16 elements
  static_assert(BM % 64 == 0 && BN % 64 == 0, "whole chunks and fragments per wavefront");
};

// LDS element offset of the 16-byte chunk c (k values 8c .. 8c + 7 of the step) of row r
__device__ __forceinline__ int ops_off(int r, int c) {
  const int line = r >> 1;
  return line * 64 + (((((r & 1) << 2) | c) ^ (line & 7)) << 3);
}

// 8 values -> their bf16 planes in LDS
template <class TL>
__device__ __forceinline__ void ops_put(bf16_t* lds, int off, const float (&v)[8]) {
  if constexpr (TL::NP == 1) {
    *reinterpret_cast<u32x4_t*>(lds + off) =
        u32x4_t{pack_bf2(v[0], v[1]), pack_bf2(v[2], v[3]), pack_bf2(v[4], v[5]), pack_bf2(v[6], v[7])};
  } else {
    u32x4_t p1, p2, p3;
    static_for<4>([&](auto h) {
      const uint32_t a = __float_as_uint(v[2 * h]), b = __float_as_uint(v[2 * h + 1]);
      p1[int(h)] = __builtin_amdgcn_perm(b, a, 0x07060302u);  // upper halves
      const float ra = v[2 * h] - __uint_as_float(a & 0xffff0000u), rb = v[2 * h + 1] - __uint_as_float(b & 0xffff0000u);
      const uint32_t q = pack_bf2(ra, rb);
      p2[int(h)] = q;
      p3[int(h)] = pack_bf2(ra - __uint_as_float(q << 16), rb - __uint_as_float(q & 0xffff0000u));
    });
    *reinterpret_cast<u32x4_t*>(lds + off) = p1;
    *reinterpret_cast<u32x4_t*>(lds + TL::PLANE + off) = p2;
    *reinterpret_cast<u32x4_t*>(lds + 2 * TL::PLANE + off) = p3;
  }
}

// acc += the tile's products over `steps` k steps.  la / lw: load(step, slot, v) reads the
// chunk (row, c) = la.at(slot) of the step (zeros outside the operand).
template <class TL, class LA, class LW>
__device__ __forceinline__ void ops_core(const LA& la, const LW& lw, int steps, bf16_t* lds,
                                         f32x4_t (&acc)[TL::FM][TL::FN]) {
  const int lane = threadIdx.x & 63, wv = threadIdx.x >> 6;
  const int wm = wv >> 1, wn = wv & 1, l16 = lane & 15, kg = lane >> 4;
  static_for<TL::FM>([&](auto i) {
    static_for<TL::FN>([&](auto j) { acc[i][j] = f32x4_t{0.f, 0.f, 0.f, 0.f}; });
  });
  if (steps <= 0) return;  // uniform per block
  int aoff[TL::SA], woff[TL::SW];
  static_for<TL::SA>([&](auto s) { aoff[s] = ops_off(la.row(s), la.chunk(s)); });
  static_for<TL::SW>([&](auto s) { woff[s] = ops_off(TL::BM + lw.row(s), lw.chunk(s)); });
  int afrag[TL::FM], wfrag[TL::FN];
  static_for<TL::FM>([&](auto i) { afrag[i] = ops_off(wm * 16 * TL::FM + 16 * i + l16, kg); });
  static_for<TL::FN>([&](auto j) { wfrag[j] = ops_off(TL::BM + wn * 16 * TL::FN + 16 * j + l16, kg); });
  float va[TL::SA][8], vw[TL::SW][8];
  auto load = [&](int step) {
    static_for<TL::SA>([&](auto s) { la.load(step, s, va[s]); });
    static_for<TL::SW>([&](auto s) { lw.load(step, s, vw[s]); });
  };
  load(0);
  for (int step = 0; step < steps; ++step) {
    static_for<TL::SA>([&](auto s) { ops_put<TL>(lds, aoff[s], va[s]); });
    static_for<TL::SW>([&](auto s) { ops_put<TL>(lds, woff[s], vw[s]); });
    lds_barrier();
    if (step + 1 < steps) load(step + 1);
    bf16x8_t af[TL::NP][TL::FM], wf[2][TL::NP];
    auto get = [&](int p, int off) { return *reinterpret_cast<const bf16x8_t*>(lds + p * TL::PLANE + off); };
    static_for<TL::NP>([&](auto p) { wf[0][p] = get(p, wfrag[0]); });
    static_for<TL::NP>([&](auto p) { static_for<TL::FM>([&](auto i) { af[p][i] = get(p, afrag[i]); }); });
    static_for<TL::FN>([&](auto j) {
      constexpr int b = j & 1;
      if constexpr (j + 1 < TL::FN) static_for<TL::NP>([&](auto p) { wf[b ^ 1][p] = get(p, wfrag[j + 1]); });
      auto product = [&](auto pw, auto pa) {
        static_for<TL::FM>([&](auto i) { acc[i][j] = mfma_bf16_16x16x32(wf[b][pw], af[pa][i], acc[i][j]); });
      };
      using I0 = std::integral_constant<int, 0>;
      mfma_fence_begin();
      if constexpr (TL::NP == 3) {
        using I1 = std::integral_constant<int, 1>;
        using I2 = std::integral_constant<int, 2>;
        product(I0{}, I2{});
        product(I1{}, I1{});
        product(I2{}, I0{});
        product(I0{}, I1{});
        product(I1{}, I0{});
      }
      product(I0{}, I0{});
      mfma_fence_end();
    });
    lds_barrier();
  }
}

// Non-finite results of the split: recomputed with fused multiply-adds over k in order.
// at(m, n) is the value of output (m, n) by that chain.
template <class TL, class F>
__device__ __forceinline__ void ops_mend(f32x4_t (&acc)[TL::FM][TL::FN], const F& at) {
  if constexpr (TL::NP == 3) {
    const int lane = threadIdx.x & 63, wv = threadIdx.x >> 6;
    const int wm = wv >> 1, wn = wv & 1, l16 = lane & 15, kg = lane >> 4;
    static_for<TL::FM>([&](auto i) {
      static_for<TL::FN>([&](auto j) {
        static_for<4>([&](auto e) {
          const float y = acc[i][j][int(e)];
          if (!(fabsf(y) < INFINITY))
            acc[i][j][int(e)] = at(wm * 16 * TL::FM + 16 * i + l16, wn * 16 * TL::FN + 16 * j + 4 * kg + e);
        });
      });
    });
  }
}

// ------------------------------------------------------------------------------------------
// Y[m, n] = sum_k A[arow(m), k] W[n, k] + bias[n], m < *m_dev (or m_max); K % 8 == 0,
// Nout % 4 == 0, rows of A, W and out 16-byte aligned
// ------------------------------------------------------------------------------------------
template <int SLOTS>
struct RowLoader {
  const float* p[SLOTS];
  int K;
  __device__ __forceinline__ static int row(int s) { return (threadIdx.x + 256 * s) >> 2; }
  __device__ __forceinline__ static int chunk(int) { return threadIdx.x & 3; }
  __device__ __forceinline__ void load(int step, int s, float (&v)[8]) const {
    const int k = step * 32 + 8 * (threadIdx.x & 3);
    float4 a = make_float4(0.f, 0.f, 0.f, 0.f), b = a;
    if (p[s] && k < K) {
      a = *reinterpret_cast<const float4*>(p[s] + k);
      b = *reinterpret_cast<const float4*>(p[s] + k + 4);
    }
    v[0] = a.x; v[1] = a.y; v[2] = a.z; v[3] = a.w;
    v[4] = b.x; v[5] = b.y; v[6] = b.z; v[7] = b.w;
  }
};

template <class TL>
__global__ void __launch_bounds__(TL::THREADS, 2) gemm_ops_kernel(const float* __restrict__ A, const int32_t* __restrict__ arows,
                                                               const int32_t* __restrict__ m_dev, int m_max, int K,
                                                               const float* __restrict__ W, const float* __restrict__ bias,
                                                               int Nout, int epi, float* __restrict__ out,
                                                               const int32_t* __restrict__ res_rows) {
  __shared__ __align__(16) bf16_t lds[TL::NP * TL::PLANE];
  const int M = m_dev ? m_dev[0] : m_max;
  const int mt = (M + TL::BM - 1) / TL::BM;
  int rt, ct;
  xcd_tile(blockIdx.x, (Nout + TL::BN - 1) / TL::BN, rt, ct);
  if (rt >= mt) return;  // uniform per block
  const int m0 = rt * TL::BM, n0 = ct * TL::BN;
  RowLoader<TL::SA> la;
  RowLoader<TL::SW> lw;
  la.K = lw.K = K;
  static_for<TL::SA>([&](auto s) {
    const int m = m0 + la.row(s);
    la.p[s] = m < M ? A + (size_t)(arows ? arows[m] : m) * K : nullptr;
  });
  static_for<TL::SW>([&](auto s) {
    const int n = n0 + lw.row(s);
    lw.p[s] = n < Nout ? W + (size_t)n * K : nullptr;
  });
  f32x4_t acc[TL::FM][TL::FN];
  ops_core<TL>(la, lw, (K + 31) / 32, lds, acc);
  ops_mend<TL>(acc, [&](int mr, int nr) {
    const int m = m0 + mr, n = n0 + nr;
    if (m >= M || n >= Nout) return 0.f;
    const float *a = A + (size_t)(arows ? arows[m] : m) * K, *w = W + (size_t)n * K;
    float y = 0.f;
    for (int k = 0; k < K; ++k) y = fmaf(a[k], w[k], y);
    return y;
  });
  // lane holds Y[m = .. + l16][n = .. + 4 kg + e]
  const int lane = threadIdx.x & 63, wv = threadIdx.x >> 6;
  const int wm = wv >> 1, wn = wv & 1, l16 = lane & 15, kg = lane >> 4;
  static_for<TL::FM>([&](auto i) {
    const int m = m0 + wm * 16 * TL::FM + 16 * i + l16;
    if (m >= M) return;
    const size_t dst = (size_t)(epi == EPI_RESID && res_rows ? res_rows[m] : m) * Nout;
    static_for<TL::FN>([&](auto j) {
      const int n = n0 + wn * 16 * TL::FN + 16 * j + 4 * kg;
      if (n >= Nout) return;
      const f32x4_t& a = acc[i][j];
      float4 y = make_float4(a[0] + bias[n], a[1] + bias[n + 1], a[2] + bias[n + 2], a[3] + bias[n + 3]);
      float4* p = reinterpret_cast<float4*>(out + dst + n);
      if (epi == EPI_GELU) {
        y = make_float4(gelu_erf(y.x), gelu_erf(y.y), gelu_erf(y.z), gelu_erf(y.w));
      } else if (epi == EPI_RESID) {
        const float4 x = *p;
        y = make_float4(x.x + y.x, x.y + y.y, x.z + y.z, x.w + y.w);
      }
      *p = y;
    });
  });
}

// Blocks below which the 64 x 64 tile is taken: 128 x 128 tiles run two per CU, so fewer than
// 512 of them leave CUs idle.  A row count known only on the device (the query rows) is taken
// as 0.4 of its bound, the most a clip's mask is expected to cover.
static bool ops_big(long long blocks, bool dev_rows) { return (dev_rows ? 2 * blocks / 5 : blocks) >= 512; }

template <int NP>
static void gemm_ops(const float* A, const int32_t* arows, const int32_t* m_dev, int m_max, int K, const float* W,
                     const float* bias, int Nout, int epi, float* out, const int32_t* res_rows, hipStream_t s) {
  if (m_max <= 0) return;
  auto run = [&](auto tl) {
    using TL = decltype(tl);
    const int grid = xcd_grid((m_max + TL::BM - 1) / TL::BM, (Nout + TL::BN - 1) / TL::BN);
    gemm_ops_kernel<TL><<<grid, TL::THREADS, 0, s>>>(A, arows, m_dev, m_max, K, W, bias, Nout, epi, out, res_rows);
  };
  const long long blocks = (long long)((m_max + 127) / 128) * ((Nout + 127) / 128);
  if (ops_big(blocks, m_dev != nullptr))
    run(OpsTile<128, 128, NP>());
  else
    run(OpsTile<64, 64, NP>());
}

void launch_gemm_f32(const float* A, const int32_t* arows, const int32_t* m_dev, int m_max, int K, const float* W,
                     const float* bias, int Nout, int epi, float* out, const int32_t* res_rows, hipStream_t s) {
  gemm_ops<3>(A, arows, m_dev, m_max, K, W, bias, Nout, epi, out, res_rows, s);
}

void launch_gemm_bf16ops(const float* A, const int32_t* arows, const int32_t* m_dev, int m_max, int K, const float* W,
                         const float* bias, int Nout, int epi, float* out, const int32_t* res_rows, hipStream_t s) {
  gemm_ops<1>(A, arows, m_dev, m_max, K, W, bias, Nout, epi, out, res_rows, s);
}

// ------------------------------------------------------------------------------------------
// Token reductions (weight gradients): part[chunk][i][j] = sum over the chunk's rows m of
// A[arow(m)][i] B[brow(m)][j], m < *M_dev (or M_max), TN_CHUNK rows per chunk, A row stride
// lda, B row stride ldb, i < I, j < J (J % 4 == 0).  Chunks past the last row write nothing
// (launch_sum_parts reads only the chunks in use).  The contraction runs over rows, so a
// thread reads 8 rows of one column (a wavefront reads 64 adjacent columns of a row at a time)
// and holds an operand chunk already transposed.
// ------------------------------------------------------------------------------------------
template <int ROWS, int SLOTS>
struct ColLoader {
  const float* X;
  const int32_t* rows;  // row table, or null
  int ld, col0, ncol, m_begin, m_end;
  __device__ __forceinline__ static int row(int s) { return (threadIdx.x + 256 * s) % ROWS; }
  __device__ __forceinline__ static int chunk(int s) { return (threadIdx.x + 256 * s) / ROWS; }
  __device__ __forceinline__ void load(int step, int s, float (&v)[8]) const {
    // every load is issued, from a row and column inside the operand; values outside become
    // zero afterwards (a condition around each load makes the compiler wait for them in turn:
    // 13,000 cycles per step against about 1,500)
    const int c = col0 + row(s), m = m_begin + 32 * step + 8 * chunk(s);
    const float* p = X + min(c, ncol - 1);
    int r[8];
    static_for<8>([&](auto e) { r[e] = min(m + e, m_end - 1); });
    if (rows) static_for<8>([&](auto e) { r[e] = rows[r[e]]; });  // uniform per launch
    static_for<8>([&](auto e) { v[e] = p[(size_t)r[e] * ld]; });
    static_for<8>([&](auto e) { v[e] = c < ncol && m + e < m_end ? v[e] : 0.f; });
  }
};

template <class TL>
__global__ void __launch_bounds__(TL::THREADS, 2) tn_ops_kernel(const float* __restrict__ A, const int32_t* __restrict__ arow,
                                                             int lda, const float* __restrict__ B,
                                                             const int32_t* __restrict__ brow, int ldb,
                                                             const int32_t* __restrict__ M_dev, int M_max, int I, int J,
                                                             float* __restrict__ part) {
  __shared__ __align__(16) bf16_t lds[TL::NP * TL::PLANE];
  const int M = M_dev ? M_dev[0] : M_max;
  // the tiles of a chunk run on one XCD (xcd_tile), so its rows enter that XCD's L2 once
  const int it = (I + TL::BM - 1) / TL::BM;
  int ch, tile;
  xcd_tile(blockIdx.x, it * ((J + TL::BN - 1) / TL::BN), ch, tile);
  const int m_begin = ch * TN_CHUNK, m_end = min(M, m_begin + TN_CHUNK);
  if (m_begin >= m_end) return;  // uniform per block
  const int i0 = (tile % it) * TL::BM, j0 = (tile / it) * TL::BN;
  const ColLoader<TL::BM, TL::SA> la{A, arow, lda, i0, I, m_begin, m_end};
  const ColLoader<TL::BN, TL::SW> lw{B, brow, ldb, j0, J, m_begin, m_end};
  f32x4_t acc[TL::FM][TL::FN];
  ops_core<TL>(la, lw, (m_end - m_begin + 31) / 32, lds, acc);
  ops_mend<TL>(acc, [&](int ir, int jr) {
    const int i = i0 + ir, j = j0 + jr;
    if (i >= I || j >= J) return 0.f;
    float y = 0.f;
    for (int m = m_begin; m < m_end; ++m)
      y = fmaf(A[(size_t)(arow ? arow[m] : m) * lda + i], B[(size_t)(brow ? brow[m] : m) * ldb + j], y);
    return y;
  });
  // lane holds P[i = .. + l16][j = .. + 4 kg + e]
  const int lane = threadIdx.x & 63, wv = threadIdx.x >> 6;
  const int wm = wv >> 1, wn = wv & 1, l16 = lane & 15, kg = lane >> 4;
  float* P = part + (size_t)ch * I * J;
  static_for<TL::FM>([&](auto fi) {
    const int i = i0 + wm * 16 * TL::FM + 16 * fi + l16;
    if (i >= I) return;
    static_for<TL::FN>([&](auto fj) {
      const int j = j0 + wn * 16 * TL::FN + 16 * fj + 4 * kg;
      if (j >= J) return;
      const f32x4_t& a = acc[fi][fj];
      *reinterpret_cast<float4*>(P + (size_t)i * J + j) = make_float4(a[0], a[1], a[2], a[3]);
    });
  });
}

// 64 x 64 tiles: a block's chunk is a serial chain of up to 64 steps, each waiting for rows
// from HBM, so many small blocks beat the halved operand traffic of 128 x 128 tiles (4 clips
// of 5 x 240 x 432, 256-wide, bf16 operands: 104 us a launch against 172 us).
template <int NP>
static void tn_ops(const float* A, const int32_t* arow, int lda, const float* B, const int32_t* brow, int ldb,
                   const int32_t* M_dev, int M_max, int I, int J, float* part, hipStream_t s) {
  using TL = OpsTile<64, 64, NP>;
  if (M_max <= 0) return;
  const int grid = xcd_grid(tn_chunks(M_max), ((I + TL::BM - 1) / TL::BM) * ((J + TL::BN - 1) / TL::BN));
  tn_ops_kernel<TL><<<grid, TL::THREADS, 0, s>>>(A, arow, lda, B, brow, ldb, M_dev, M_max, I, J, part);
}

void launch_tn_f32(const float* A, const int32_t* arow, int lda, const float* B, const int32_t* brow, int ldb,
                   const int32_t* M_dev, int M_max, int I, int J, float* part, hipStream_t s) {
  tn_ops<3>(A, arow, lda, B, brow, ldb, M_dev, M_max, I, J, part, s);
}

void launch_tn_bf16ops(const float* A, const int32_t* arow, int lda, const float* B, const int32_t* brow, int ldb,
                       const int32_t* M_dev, int M_max, int I, int J, float* part, hipStream_t s) {
  tn_ops<1>(A, arow, lda, B, brow, ldb, M_dev, M_max, I, J, part, s);
}

}  // namespace dr
