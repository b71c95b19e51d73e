// Products of FP32 matrices on the bf16 matrix cores: the linears of the FP32 path and every
// weight product of the training passes (linears, input gradients, weight gradients).
//
// Two arithmetics share the kernels, by the number of bf16 planes NP an operand is split into:
//
//   NP = 3 (FP32), the three-plane split of Henry, Tang and Heinecke ("Leveraging the bfloat16
//     Artificial Intelligence Datatype for Higher-Precision Computations", 2019):
//     a = a1 + a2 + a3 (8 + 8 + 8 significant bits: a1 the truncated upper half of the float,
//     a2 and a3 the rounded remainders), exactly from |a| = 2^-110 on; below, a3 falls under the
//     smallest bf16 and a loses at most 2^-134.
//     a w ~ a3 w1 + a2 w2 + a1 w3 + a2 w1 + a1 w2 + a1 w1, six v_mfma_f32_16x16x32_bf16 per
//     32-wide k step with FP32 accumulation, the small terms first.  The dropped a2 w3 + a3 w2 +
//     a3 w3 are at most 2^-22 |a w| (1.001 times that) and on average 0.4 x 2^-24 of it, but a k
//     step rounds its accumulator 6 times where a chain of FP32 fused multiply-adds rounds it 32
//     times: measured against 64 bits, the FP32 clip's and gradients' errors are not larger than
//     with the chain (1.21e-7 -> 1.17e-7, 2.6e-6 -> 0.95e-6).  Six bf16 products cost 96 matrix
//     cycles per 16 x 16 x 32 step where v_mfma_f32_16x16x4_f32 costs 256 (and the vector ALU as
//     much).  Where a result is not finite (an operand, or a sum, out of range) that of the fused
//     multiply-adds is taken, so infinities come out as they do there.
//   NP = 1 (mixed precision): operands rounded to bf16 to nearest even, one product.
//
// Block = 4 wavefronts (2 x 2), BM x BN outputs, k in steps of 32.  Operands of the linears
// (the weight gradients' are described with them) are read from
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

// put(p, plane p of 8 values)
template <int NP, class Put>
__device__ __forceinline__ void ops_split(const float (&v)[8], const Put& put) {
  using I0 = std::integral_constant<int, 0>;
  if constexpr (NP == 1) {
    put(I0{}, __builtin_bit_cast(bf16x8_t, u32x4_t{pack_bf2(v[0], v[1]), pack_bf2(v[2], v[3]), pack_bf2(v[4], v[5]),
                                                   pack_bf2(v[6], v[7])}));
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
    put(I0{}, __builtin_bit_cast(bf16x8_t, p1));
    put(std::integral_constant<int, 1>{}, __builtin_bit_cast(bf16x8_t, p2));
    put(std::integral_constant<int, 2>{}, __builtin_bit_cast(bf16x8_t, p3));
  }
}

// acc[..][j] += the products of the operand fragments af and wf (of column fragment j)
template <class TL, class J>
__device__ __forceinline__ void ops_products(const bf16x8_t (&af)[TL::NP][TL::FM], const bf16x8_t (&wf)[TL::NP],
                                             f32x4_t (&acc)[TL::FM][TL::FN], J j) {
  auto product = [&](auto pw, auto pa) {
    static_for<TL::FM>([&](auto i) { acc[i][j] = mfma_bf16_16x16x32(wf[pw], af[pa][i], acc[i][j]); });
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
}

// acc += the tile's products over `steps` k steps.  la / lw: load(step, slot, v) reads the
// chunk (row, c) = la.at(slot) of the step (zeros outside the operand).
template <class TL, class LA, class LW>
__device__ __forceinline__ void ops_core(const LA& la, const LW& lw, int steps, bf16_t* lds,
                                         f32x4_t (&acc)[TL::FM][TL::FN]) {
  static_for<TL::FM>([&](auto i) {
    static_for<TL::FN>([&](auto j) { acc[i][j] = f32x4_t{0.f, 0.f, 0.f, 0.f}; });
  });
  if (steps <= 0) return;  // uniform per block
  const int lane = threadIdx.x & 63, wv = threadIdx.x >> 6;
  const int wm = wv >> 1, wn = wv & 1, l16 = lane & 15, kg = lane >> 4;
  int afrag[TL::FM], wfrag[TL::FN], aoff[TL::SA], woff[TL::SW];
  static_for<TL::FM>([&](auto i) { afrag[i] = ops_off(wm * 16 * TL::FM + 16 * i + l16, kg); });
  static_for<TL::FN>([&](auto j) { wfrag[j] = ops_off(TL::BM + wn * 16 * TL::FN + 16 * j + l16, kg); });
  static_for<TL::SA>([&](auto s) { aoff[s] = ops_off(la.row(s), la.chunk(s)); });
  static_for<TL::SW>([&](auto s) { woff[s] = ops_off(TL::BM + lw.row(s), lw.chunk(s)); });
  float va[TL::SA][8], vw[TL::SW][8];
  auto load = [&](int step) {
    static_for<TL::SA>([&](auto s) { la.load(step, s, va[s]); });
    static_for<TL::SW>([&](auto s) { lw.load(step, s, vw[s]); });
  };
  auto put = [&](int off, const float(&v)[8]) {
    ops_split<TL::NP>(v, [&](auto p, bf16x8_t x) { *reinterpret_cast<bf16x8_t*>(lds + p * TL::PLANE + off) = x; });
  };
  bf16x8_t af[TL::NP][TL::FM], wf[2][TL::NP];
  auto get = [&](int p, int off) { return *reinterpret_cast<const bf16x8_t*>(lds + p * TL::PLANE + off); };
  load(0);
  for (int step = 0; step < steps; ++step) {
    static_for<TL::SA>([&](auto s) { put(aoff[s], va[s]); });
    static_for<TL::SW>([&](auto s) { put(woff[s], vw[s]); });
    lds_barrier();
    if (step + 1 < steps) load(step + 1);
    static_for<TL::NP>([&](auto p) { wf[0][p] = get(p, wfrag[0]); });
    static_for<TL::NP>([&](auto p) { static_for<TL::FM>([&](auto i) { af[p][i] = get(p, afrag[i]); }); });
    static_for<TL::FN>([&](auto j) {
      constexpr int b = j & 1;
      if constexpr (j + 1 < TL::FN) static_for<TL::NP>([&](auto p) { wf[b ^ 1][p] = get(p, wfrag[j + 1]); });
      ops_products<TL>(af, wf[b], acc, j);
    });
    lds_barrier();
  }
}

// Results of the split that are not finite (an operand, or a sum, out of range) are replaced by
// those of fused multiply-adds over k in order; the others keep their bits.  The block computes
// them for its whole tile, from FP32 operands in LDS: stage(step, As, Ws) writes a step's,
// As[32][BM] and Ws[32][BN].  (A 5 x 240 x 432 clip of a 256-wide network with a NaN weight takes
// 3.8 ms and one without 1.8; one result at a time it took 100.)
template <class TL, class Stage>
__device__ __forceinline__ void ops_mend(f32x4_t (&acc)[TL::FM][TL::FN], float* lds, int steps, const Stage& stage) {
  if constexpr (TL::NP == 3) {
    const int lane = threadIdx.x & 63, wv = threadIdx.x >> 6;
    const int wm = wv >> 1, wn = wv & 1, l16 = lane & 15, kg = lane >> 4;
    f32x4_t zero = {0.f, 0.f, 0.f, 0.f};  // NaN as soon as a result is not finite
    static_for<TL::FM>([&](auto i) {
      static_for<TL::FN>([&](auto j) {
        static_for<4>([&](auto e) { zero[int(e)] = fmaf(acc[i][j][int(e)], 0.f, zero[int(e)]); });
      });
    });
    const bool bad = __ballot(!((zero[0] + zero[1]) + (zero[2] + zero[3]) == 0.f)) != 0;
    if (lane == 0) lds[wv] = bad ? 1.f : 0.f;  // (every wavefront has read the last step)
    lds_barrier();
    if (lds[0] + lds[1] + lds[2] + lds[3] == 0.f) return;  // uniform per block
    f32x4_t y[TL::FM][TL::FN];
    static_for<TL::FM>([&](auto i) {
      static_for<TL::FN>([&](auto j) { y[i][j] = f32x4_t{0.f, 0.f, 0.f, 0.f}; });
    });
    float *As = lds, *Ws = lds + 32 * TL::BM;
    for (int step = 0; step < steps; ++step) {
      __syncthreads();
      stage(step, As, Ws);
      __syncthreads();
      for (int k = 0; k < 32; ++k) {
        float a[TL::FM];
        static_for<TL::FM>([&](auto i) { a[i] = As[k * TL::BM + wm * 16 * TL::FM + 16 * i + l16]; });
        static_for<TL::FN>([&](auto j) {
          const f32x4_t w = *reinterpret_cast<const f32x4_t*>(Ws + k * TL::BN + wn * 16 * TL::FN + 16 * j + 4 * kg);
          static_for<TL::FM>([&](auto i) {
            static_for<4>([&](auto e) { y[i][j][int(e)] = fmaf(a[i], w[int(e)], y[i][j][int(e)]); });
          });
        });
      }
    }
    static_for<TL::FM>([&](auto i) {
      static_for<TL::FN>([&](auto j) {
        static_for<4>([&](auto e) {
          if (!(fabsf(acc[i][j][int(e)]) < INFINITY)) acc[i][j][int(e)] = y[i][j][int(e)];
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
  ops_mend<TL>(acc, reinterpret_cast<float*>(lds), (K + 31) / 32, [&](int step, float* As, float* Ws) {
    auto put = [&](const auto& from, auto s, int rows, float* to) {
      float v[8];
      from.load(step, s, v);
      static_for<8>([&](auto e) { to[(8 * from.chunk(s) + e) * rows + from.row(s)] = v[e]; });
    };
    static_for<TL::SA>([&](auto s) { put(la, s, TL::BM, As); });
    static_for<TL::SW>([&](auto s) { put(lw, s, TL::BN, Ws); });
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
// A[m][i] B[brow(m)][j], m < *M_dev (or M_max), A row stride lda, B row stride ldb, i < I, j < J
// (multiples of 4; rows 16-byte aligned).  Chunks past the last row write nothing
// (launch_sum_parts reads only the chunks in use).  The contraction runs over rows: a thread
// reads 8 rows of one column back from LDS and holds an operand fragment already transposed.
// ------------------------------------------------------------------------------------------
// One operand: a step is 32 rows x COLS floats in LDS, the 16-byte chunk c of row r at
// c ^ 4 (r / 8 % 4), so the four row groups of a fragment read fall on distinct banks.
template <int COLS, bool TABLE>
struct ColDma {
  static constexpr int RPL = 256 / COLS;      // rows per 1 KB load
  static constexpr int LOADS = 32 / RPL / 4;  // per wavefront (4 wavefronts)
  const float* X;                             // column col0
  const int32_t* rows;                        // TABLE: the chunk's rows, in LDS
  int ld, ncol, m_begin, count;               // columns from col0 on; rows
  // row r of a step and its columns from col on: this lane's part of load i
  __device__ __forceinline__ static int first(int i) { return (4 * i + __builtin_amdgcn_readfirstlane(threadIdx.x >> 6)) * RPL; }
  __device__ __forceinline__ static int row(int i) { return first(i) + (threadIdx.x & 63) / (COLS / 4); }
  __device__ __forceinline__ int col(int i) const {  // past the last: repeated, its results are not stored
    return min(4 * (((threadIdx.x & 63) % (COLS / 4)) ^ (4 * (row(i) >> 3))), ncol - 4);
  }
  __device__ __forceinline__ void dma(int step, float* dst) const {
    static_for<LOADS>([&](auto i) {
      bf16_t* to = reinterpret_cast<bf16_t*>(dst + first(i) * COLS);
      if constexpr (TABLE) {
        const int m = min(32 * step + row(i), count - 1);
        const int r = lds_as_bf16<int>(rows + m);
        dma16(X + (size_t)r * ld + col(i), to);
      } else if (32 * step + 32 <= count) {  // a uniform base and a lane's offset, the same in every step
        dma16(X + (size_t)(m_begin + 32 * step) * ld + ((uint32_t)row(i) * ld + col(i)), to);
      } else {  // rows past the last repeat it: get() clears them
        dma16(X + (size_t)(m_begin + min(32 * step + row(i), count - 1)) * ld + col(i), to);
      }
    });
  }
  // rows 8 kg .. 8 kg + 7 of column c; unless the step is full, those past its first `left` as zeros
  template <class Full>
  __device__ __forceinline__ static void get(Full full, const float* src, int kg, int c, int left, float (&v)[8]) {
    static_for<8>([&](auto e) {
      const float x = lds_as_bf16<float>(src + (8 * kg + e) * COLS + (c ^ (16 * kg)));
      v[e] = full || 8 * kg + e < left ? x : 0.f;
    });
  }
};

template <class TL>
constexpr int TN_STAGE = (TL::BM + TL::BN) * 32;  // floats of a step

// acc += the tile's products over the chunk's rows.  Operands go to LDS as they are, by direct
// global->LDS loads two steps ahead, and each wavefront splits its own fragments.  What bounds
// it is the latency of a step's loads (the chunk is a serial chain and the shapes give one or
// two blocks per CU), so the loads in flight count and not the split being done twice.  A
// training step of 4 clips of 5 x 240 x 432 (256 wide, 8 blocks; bf16) and of 2 (FP32), all
// weight gradients: loads into registers one step ahead, split once into LDS, 64 x 64 tiles
// 5.2 and 5.5 ms; direct loads, split once through LDS 3.7 and 4.3 ms; this 3.5 and 3.3 ms.
template <class TL, class LA, class LW>
__device__ __forceinline__ void tn_core(const LA& la, const LW& lw, float* lds, f32x4_t (&acc)[TL::FM][TL::FN]) {
  const int lane = threadIdx.x & 63, wv = threadIdx.x >> 6;
  const int wm = wv >> 1, wn = wv & 1, l16 = lane & 15, kg = lane >> 4;
  const int steps = (la.count + 31) / 32;
  static_for<TL::FM>([&](auto i) {
    static_for<TL::FN>([&](auto j) { acc[i][j] = f32x4_t{0.f, 0.f, 0.f, 0.f}; });
  });
  auto issue = [&](int step) {
    float* dst = lds + (step & 1) * TN_STAGE<TL>;
    la.dma(step, dst);
    lw.dma(step, dst + TL::BM * 32);
  };
  auto multiply = [&](int step, auto full) {
    const float* src = lds + (step & 1) * TN_STAGE<TL>;
    const int left = la.count - 32 * step;
    bf16x8_t af[TL::NP][TL::FM], wf[TL::FN][TL::NP];
    static_for<TL::FM>([&](auto i) {
      float v[8];
      la.get(full, src, kg, wm * 16 * TL::FM + 16 * i + l16, left, v);
      ops_split<TL::NP>(v, [&](auto p, bf16x8_t x) { af[p][i] = x; });
    });
    static_for<TL::FN>([&](auto j) {
      float v[8];
      lw.get(full, src + TL::BM * 32, kg, wn * 16 * TL::FN + 16 * j + l16, left, v);
      ops_split<TL::NP>(v, [&](auto p, bf16x8_t x) { wf[j][p] = x; });
    });
    lds_barrier();  // every wavefront has read the step
    if (step + 2 < steps) issue(step + 2);
    static_for<TL::FN>([&](auto j) { ops_products<TL>(af, wf[j], acc, j); });
  };
  issue(0);
  if (steps > 1) issue(1);
  for (int step = 0; step + 1 < steps; ++step) {
    vm_wait_barrier<LA::LOADS + LW::LOADS>();  // this step has landed, the next is on its way
    multiply(step, std::true_type{});
  }
  vm_wait_barrier<0>();
  multiply(steps - 1, std::false_type{});
}

template <class TL, bool TABLE>
__global__ void __launch_bounds__(TL::THREADS, 2) tn_ops_kernel(const float* __restrict__ A, int lda, const float* __restrict__ B,
                                                             const int32_t* __restrict__ brow, int ldb,
                                                             const int32_t* __restrict__ M_dev, int M_max, int I, int J,
                                                             int chunk, float* __restrict__ part) {
  extern __shared__ __align__(16) float tn_lds[];
  const int M = M_dev ? M_dev[0] : M_max;
  // Each XCD (block b runs on b & 7) takes an eighth of the tiles that have rows, in the order
  // of the chunks: those of a chunk share its L2, and no XCD has a whole chunk more to do than
  // another (FP32, 64 x 64 tiles: 105 -> 99 us per call of the step below).
  const int it = (I + TL::BM - 1) / TL::BM, tiles = it * ((J + TL::BN - 1) / TL::BN);
  const int total = (M + chunk - 1) / chunk * tiles, per = (total + 7) / 8;
  const int k = blockIdx.x >> 3, idx = (blockIdx.x & 7) * per + k;
  if (k >= per || idx >= total) return;  // uniform per block
  const int ch = idx / tiles, tile = idx % tiles;
  const int m_begin = ch * chunk, m_end = min(M, m_begin + chunk);
  const int i0 = (tile % it) * TL::BM, j0 = (tile / it) * TL::BN;
  // a row table (B's) is brought to LDS first: a load that has to wait for its row number would
  // also wait for every load queued before it
  int32_t* table = reinterpret_cast<int32_t*>(tn_lds + 2 * TN_STAGE<TL>);
  if constexpr (TABLE) {
    for (int m = threadIdx.x; m < m_end - m_begin; m += TL::THREADS) table[m] = brow[m_begin + m];
    __syncthreads();
  }
  const ColDma<TL::BM, false> la{A + i0, nullptr, lda, I - i0, m_begin, m_end - m_begin};
  const ColDma<TL::BN, TABLE> lw{B + j0, table, ldb, J - j0, m_begin, m_end - m_begin};
  f32x4_t acc[TL::FM][TL::FN];
  tn_core<TL>(la, lw, tn_lds, acc);
  ops_mend<TL>(acc, tn_lds, (m_end - m_begin + 31) / 32, [&](int step, float* As, float* Ws) {
    auto put = [&](const float* X, int ld, const int32_t* rows, int c0, int ncol, int cols, float* to) {
      for (int e = threadIdx.x; e < 8 * cols; e += TL::THREADS) {
        const int r = e / (cols / 4), c = 4 * (e % (cols / 4)), m = m_begin + 32 * step + r;
        f32x4_t v = {0.f, 0.f, 0.f, 0.f};
        if (m < m_end && c0 + c < ncol) v = *reinterpret_cast<const f32x4_t*>(X + (size_t)(rows ? rows[m] : m) * ld + c0 + c);
        *reinterpret_cast<f32x4_t*>(to + r * cols + c) = v;
      }
    };
    put(A, lda, nullptr, i0, I, TL::BM, As);
    put(B, ldb, TABLE ? brow : nullptr, j0, J, TL::BN, Ws);
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

// 128 x 128 tiles halve the operand bytes where that leaves a block for every CU (a row count
// known only on the device is taken as 0.4 of its bound; the bf16 step above with 64 x 64 tiles
// alone: 4.7 ms, with both 3.7), else 64 x 64.  A row table takes the small tile: only the query
// weights' C x C gradients have one.
template <int NP>
static void tn_ops(const float* A, int lda, const float* B, const int32_t* brow, int ldb, const int32_t* M_dev,
                   int M_max, int I, int J, int chunk, float* part, hipStream_t s) {
  if (M_max <= 0) return;
  const int chunks = (M_max + chunk - 1) / chunk;
  auto run = [&](auto tl, auto has_table) {
    using TL = decltype(tl);
    constexpr bool TABLE = decltype(has_table)::value;
    static_assert(2 * TN_STAGE<TL> * 4 + (TABLE ? TN_CHUNK * 4 : 0) <= 65536, "more has to be asked for");
    const size_t bytes = 2 * TN_STAGE<TL> * 4 + (TABLE ? (size_t)chunk * 4 : 0);
    const int tiles = ((I + TL::BM - 1) / TL::BM) * ((J + TL::BN - 1) / TL::BN);
    const int grid = 8 * ((chunks * tiles + 7) / 8);
    tn_ops_kernel<TL, TABLE><<<grid, TL::THREADS, bytes, s>>>(A, lda, B, brow, ldb, M_dev, M_max, I, J, chunk, part);
  };
  const long long blocks = (long long)((I + 127) / 128) * ((J + 127) / 128) * chunks;
  const bool big = J > 64 && (M_dev ? 2 * blocks / 5 : blocks) >= 256;
  if (brow)
    run(OpsTile<64, 64, NP>(), std::true_type());
  else if (big)
    run(OpsTile<128, 128, NP>(), std::false_type());
  else
    run(OpsTile<64, 64, NP>(), std::false_type());
}

void launch_tn(bool bf16, const float* A, int lda, const float* B, const int32_t* brow, int ldb, const int32_t* M_dev,
               int M_max, int I, int J, float* part, hipStream_t s) {
  (bf16 ? tn_ops<1> : tn_ops<3>)(A, lda, B, brow, ldb, M_dev, M_max, I, J, tn_chunk(bf16), part, s);
}

}  // namespace dr
