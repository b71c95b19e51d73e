// BF16 linears of the transformer blocks on the direct-to-LDS MFMA core (gemm_core.h).
//
// The LayerNorms are split in two.  Their normalisation (x - mean) * rstd is applied by the
// kernel that produces the row -- the embedding for every token, the output projection and
// the second MLP linear for the updated tokens -- which stores the normalised row x^ in bf16
// next to the FP32 residual.  Their affine part is folded into the linear that follows:
// LN(x) W^T + b = x^ (W diag(g))^T + (b + W beta), so Q/K/V, the first MLP linear and the
// decoder read x^ directly.  In exact arithmetic this is the same network (the folded weights
// are derived on the device at load, in double precision).  The first MLP linear's folded
// weight and bias and the second's weight each also carry a factor 1/sqrt 2, so that the
// GELU epilogue evaluates x (1 + erf x) on x = z / sqrt 2 (gelu_scaled) without the two
// constant multiplications of 0.5 z (1 + erf(z / sqrt 2)).
//
//   qkv:   [Q | K | V] = x^ Wqkv'^T + bqkv'      all tokens of windows holding a query (K, V);
//                                                row tiles holding a flagged token (Q)
//   fc1:   h = GELU(u2 W1'^T + b1')              u2 = x^ of the flagged tokens after the
//                                                projection (compact rows)
//   proj:  x[idx[r]] += o W_o^T + b_o;  u2[r] = normalise(x[idx[r]])
//   fc2:   x[idx[r]] += h W_2^T + b_2;  x^[idx[r]] = normalise(x[idx[r]])
#include <algorithm>

#include "dr_internal.h"
#include "gemm_core.h"

namespace dr {

template <class K>
static void allow_lds(K kernel, size_t bytes) {
  if (bytes > 65536)
    (void)hipFuncSetAttribute(reinterpret_cast<const void*>(kernel), hipFuncAttributeMaxDynamicSharedMemorySize,
                              (int)bytes);
}

// Applies epi(m, n, acc[i][j]) to the fragments of rows m < M.
template <class TL, class Epi>
__device__ __forceinline__ void for_fragments(int M, int m0, int n0, f32x4_t (&acc)[TL::FM][TL::FN], const Epi& epi) {
  const int lane = threadIdx.x & 63, wv = threadIdx.x >> 6;
  const int wm = wv / TL::WN, wn = wv % TL::WN, l16 = lane & 15, kg = lane >> 4;
  static_for<TL::FM>([&](auto i) {
    const int m = m0 + wm * TL::TM + 16 * i + l16;
    if (m < M)
      static_for<TL::FN>([&](auto j) { epi(m, n0 + wn * TL::TN + 16 * j + 4 * kg, acc[i][j]); });
  });
}

// Row count from which the larger 8-wavefront tiles pay off (measured on the Q/K/V and first
// MLP linear shapes: from ~50k rows they run 13-17 % faster, at 16k rows 10 % slower).
constexpr int BIG_M = 32768;


// ------------------------------------------------------------------------------------------
// Q/K/V
// ------------------------------------------------------------------------------------------
// Columns [0, C) -> Q rows [N][C]; [C, 2C) -> K [win][head][Spad][dh]; [2C, 3C) -> V
// transposed, V^T [win][head][dh][spv] (keys contiguous, the layout the attention kernel
// stages as is).  A column tile lies inside one of the three parts (C % BN == 0); dh is a
// power of two (2^dsh).  Channel c of a part sits at head c >> dsh, lane c & (dh - 1), so K's
// offset is (c >> dsh) Spad dh + (c & (dh - 1)) and V^T's row is c itself.
struct QkvRow {
  bf16* base;  // token's Q row / K row of head 0 / V^T column of head 0, lane 0
  int part;    // 0 Q, 1 K, 2 V
};

__device__ __forceinline__ u32x4_t pack_bf8(const f32x4_t& a, const f32x4_t& b) {
  return u32x4_t{pack_bf2(a[0], a[1]), pack_bf2(a[2], a[3]), pack_bf2(b[0], b[1]), pack_bf2(b[2], b[3])};
}

struct QkvOut {
  const float* bias;
  bf16 *q, *k, *vt;
  int C, dsh, heads, Spad, S, spv;
  __device__ __forceinline__ QkvRow row(int m, int n0) const {
    const int part = n0 >= 2 * C ? 2 : n0 >= C ? 1 : 0;
    if (part == 0) return {q + (size_t)m * C, 0};
    const int w = m / S, s = m - w * S;
    if (part == 1) return {k + (((size_t)w * heads * Spad + s) << dsh), 1};
    return {vt + (((size_t)w * heads) << dsh) * spv + s, 2};
  }
  __device__ __forceinline__ int kstride() const { return Spad << dsh; }  // between heads of K
  __device__ __forceinline__ int vstride() const { return spv; }          // between channels of V^T
};

// Stream mode: Q rows into the batch buffer; K [win_f][head][S_f][dh] and V^T
// [win_f][head][dh][sfp] of every token into the current ring slot of its request's cache.
struct StreamQkvOut {
  const float* bias;
  bf16* q;
  StreamTable tab;
  int C, dsh, heads, Sf, nwin_f;
  __device__ __forceinline__ QkvRow row(int m, int n0) const {
    const int part = n0 >= 2 * C ? 2 : n0 >= C ? 1 : 0;
    if (part == 0) return {q + (size_t)m * C, 0};
    const int w = m / Sf, s = m - w * Sf;
    const int r = w / nwin_f, wl = w - r * nwin_f;
    const size_t slot = (size_t)pick(tab.head, r);
    if (part == 1) return {pick(tab.k, r) + slot * tab.slot_stride + (((size_t)wl * heads * Sf + s) << dsh), 1};
    return {pick(tab.v, r) + slot * tab.vslot_stride + (((size_t)wl * heads) << dsh) * tab.sfp + s, 2};
  }
  __device__ __forceinline__ int kstride() const { return Sf << dsh; }
  __device__ __forceinline__ int vstride() const { return tab.sfp; }
};

// Q/K/V tiles.  Clip mode runs only the row tiles listed with the window order (Q tiles
// holding a flagged token; K/V tiles touching a window with queries -- keys and values of a
// window without queries are never read); stream mode keeps K/V of every token (kv_all: later
// frames may query any window) and lists only the Q tiles.  A block tile is one or two listed
// row tiles (BM / ROW_TILE) by BN columns of one part.  Tiles are numbered Q column tiles
// first, then K/V (each part XCD-ordered as xcd_tile); block b runs tiles b, b + gridDim, ...
// (gridDim a multiple of 8, so they stay on its XCD).
//
// A block's tiles form one stream of 64-wide k stages through a 2-stage ring: the first two
// stages of the next tile are queued before this tile's epilogue, so that neither their
// latency nor the block start shows (one block per tile: 18,000 cycles at K = 384 for 6,100 of
// products, with 128 x 128 tiles two per CU).  Slices and barriers as in gemm_core.
// W's fragments follow lane8_row, so a lane's results are 8 consecutive channels of a token:
// Q and K rows are written 16 bytes per lane (8 bytes per lane: 19.2 us instead of 17.7 us at
// 32,400 rows of 256); V^T rows hold tokens and are written 2 bytes per lane, 16 lanes side by
// side (16 bytes of 8 tokens per lane measured slower wherever a run crosses a window: 17.7 ->
// 21.2 us at 225-token windows, 11.1 -> 16.9 us at 45).
template <class TL, class Out, int C>
__global__ void __launch_bounds__(TL::THREADS, TL::BM == ROW_TILE ? 6 : 2) qkv_kernel(int M, const bf16* __restrict__ xh,
                                                          const int32_t* __restrict__ tiles,
                                                          const int32_t* __restrict__ ntiles, int kv_all,
                                                          const bf16* __restrict__ W, Out out) {
  constexpr int SUB = TL::BM / ROW_TILE, NA = TL::BM / (8 * TL::NW), NB = TL::BN / (8 * TL::NW);
  constexpr bool ONE = SUB == 1;  // one tile per block (the grid covers them all)
  static_assert(SUB * ROW_TILE == TL::BM && SUB <= 2 && TL::ST == 2, "listed row tiles, 2-stage ring");
  static_assert(TL::BM % (8 * TL::NW) == 0 && TL::BN % (8 * TL::NW) == 0 && TL::FN % 2 == 0, "whole loads, fragment pairs");
  static_assert(C % TL::BN == 0 && (C % 128 == 0 || (C == 64 && ONE)), "whole column tiles; the ring half of a stage is fixed");
  extern __shared__ __align__(16) bf16 ring[];
  const int lane = threadIdx.x & 63, wv = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int wm = wv / TL::WN, wn = wv % TL::WN, l16 = lane & 15, kg = lane >> 4;
  const int mt = (M + ROW_TILE - 1) / ROW_TILE;
  const int nq = ntiles[0], nkv = kv_all ? mt : ntiles[1];
  const int ntq = C / TL::BN, gq = xcd_grid((nq + SUB - 1) / SUB, ntq);
  const int total = gq + xcd_grid((nkv + SUB - 1) / SUB, 2 * ntq);

  // the tile: tokens m0 .. and m1 .. (m1 = M: none), columns n0 ..
  struct Tile {
    int slot, m0, m1, n0;
  };
  auto find = [&](int slot) {  // the first slot from `slot` on that holds a tile, or total
    Tile t{total, 0, 0, 0};
    for (; slot < total; slot += gridDim.x) {
      const bool is_q = slot < gq;
      const int nt = is_q ? ntq : 2 * ntq;
      int i, ct;
      xcd_tile(is_q ? slot : slot - gq, nt, i, ct);
      // the column tiles of a row are rotated by about one per round of the grid, so that a
      // block's tiles are not all V tiles, whose epilogue is the longest (without it 173 us
      // instead of 93 us at 129,600 rows of 256)
      if (!ONE) ct = (ct + (i >> 3) * nt / (int)(gridDim.x >> 3)) % nt;
      const int n = is_q ? nq : nkv, first = i * SUB;
      if (first >= n) {
        if (ONE) break;
        continue;
      }
      const bool two = SUB == 2 && first + 1 < n;
      const int32_t* list = tiles + (is_q ? 0 : mt) + first;
      const bool listed = is_q || !kv_all;
      t = {slot, (listed ? list[0] : first) * ROW_TILE, two ? (listed ? list[1] : first + 1) * ROW_TILE : M,
           (is_q ? 0 : C) + ct * TL::BN};
      break;
    }
    return t;
  };
  auto token = [&](const Tile& t, int r) {  // token of tile row r, or one >= M
    return SUB == 1 || r < ROW_TILE ? t.m0 + r : t.m1 + r - ROW_TILE;
  };
  // a lane's sources, as byte offsets from uniform addresses
  const int lrow = wv * 8 + (lane >> 3);
  const uint32_t woff = lrow * C * 2 + ((lane & 7) ^ lane8_swz(lrow)) * 16;
  static_assert((8 * TL::NW) % 16 == 0, "lane8_swz repeats every 16 rows");
  uint32_t aoff[NA];
  const char *abase[SUB], *wbase;
  auto aim = [&](const Tile& t) {
    static_for<NA>([&](auto c) {
      constexpr int first = 8 * TL::NW * c;  // the tile row of lrow 0
      const int m0 = first < ROW_TILE ? t.m0 : t.m1, row = first % ROW_TILE + lrow;
      aoff[c] = min(row, max(M - 1 - m0, 0)) * C * 2 + ((lane & 7) ^ lds_swz(row)) * 16;
    });
    abase[0] = reinterpret_cast<const char*>(xh + (size_t)t.m0 * C);
    if constexpr (SUB == 2) abase[1] = reinterpret_cast<const char*>(xh + (size_t)(t.m1 < M ? t.m1 : 0) * C);
    wbase = reinterpret_cast<const char*>(W + (size_t)t.n0 * C);
  };
  auto issue = [&](int kt, int buf) {
    bf16* dst = ring + buf * TL::STAGE + wv * 512;
    static_for<NA>([&](auto c) {
      dma16(abase[8 * TL::NW * c / ROW_TILE] + kt * 128 + aoff[c], dst + 8 * TL::NW * c * 64);
    });
    static_for<NB>([&](auto c) {
      dma16(wbase + ((size_t)8 * TL::NW * c * C + kt * 64) * 2 + woff, dst + (TL::BM + 8 * TL::NW * c) * 64);
    });
  };
  bf16x8_t af[2][TL::FM], wf[2][TL::FN];
  auto read = [&](int buf, auto kk) {
    const bf16* sb = ring + buf * TL::STAGE;
    static_for<TL::FM>([&](auto i) {
      const int r = wm * TL::TM + 16 * i + l16;
      af[kk][i] = *reinterpret_cast<const bf16x8_t*>(sb + r * 64 + ((4 * kk + kg) ^ lds_swz(r)) * 8);
    });
    static_for<TL::FN>([&](auto j) {
      const int r = wn * TL::TN + lane8_row(j, l16);
      wf[kk][j] = *reinterpret_cast<const bf16x8_t*>(sb + (TL::BM + r) * 64 + ((4 * kk + kg) ^ lane8_swz(r)) * 8);
    });
  };
  f32x4_t acc[TL::FM][TL::FN];
  auto multiply = [&](auto kk, auto&& between) {
    mfma_fence_begin();
    bool first = true;
    static_for<TL::FM>([&](auto i) {
      static_for<TL::FN>([&](auto j) {
        acc[i][j] = mfma_bf16_16x16x32(wf[kk][j], af[kk][i], acc[i][j]);
        if (first) {
          first = false;
          mfma_fence_begin();
          between();
          mfma_fence_begin();
        }
      });
    });
    mfma_fence_end();
    asm volatile("" ::"v"(wf[kk][0]), "v"(af[kk][0]));  // not reallocated while in flight
  };
  using I0 = std::integral_constant<int, 0>;
  using I1 = std::integral_constant<int, 1>;

  constexpr int nk = C / 64;
  Tile t = find(blockIdx.x);
  if (t.slot >= total) return;
  aim(t);
  issue(0, 0);
  vm_wait_barrier<0>();
  lds_reads_done();
  read(0, I0{});
  mfma_fence_begin();
  if (nk > 1) issue(1, 1);
  for (;;) {
    const Tile nx = ONE ? Tile{total, 0, 0, 0} : find(t.slot + gridDim.x);
    const bool last = ONE || nx.slot >= total;
    const int part = t.n0 / C, c0 = t.n0 - part * C + wn * TL::TN + 8 * kg;
    f32x4_t bv[TL::FN];
    static_for<TL::FN>([&](auto j) {
      bv[j] = *reinterpret_cast<const f32x4_t*>(out.bias + part * C + c0 + 32 * (j / 2) + 4 * (j % 2));
    });
    static_for<TL::FM>([&](auto i) {
      static_for<TL::FN>([&](auto j) { acc[i][j] = f32x4_t{0.f, 0.f, 0.f, 0.f}; });
    });
    // Stage kt with its first slice read.  The stage two further on is queued once every
    // wavefront has read this one: stage kt + 2 of this tile, or of the next tile.
    auto stage = [&](int kt) {
      const int buf = kt & 1;  // its half of the ring (a tile has an even number of stages, or is the only one)
      const bool more = kt + 1 < nk || !last;
      multiply(I0{}, [&] { read(buf, I1{}); });
      if (more) {
        vm_wait_barrier<0>();
        lds_reads_done();
      }
      multiply(I1{}, [&] {
        if (more) {
          read(buf ^ 1, I0{});
          mfma_fence_begin();
          if (kt + 2 < nk) {
            issue(kt + 2, buf);
          } else if (!last) {
            if (kt + 2 == nk) aim(nx);
            issue(kt + 2 - nk, buf);
          }
        }
      });
    };
    static_for<nk>([&](auto kt) { stage(kt); });
    static_for<TL::FM>([&](auto f) {
      const int m = token(t, wm * TL::TM + 16 * f + l16);
      if (m < M) {
        const QkvRow rr = out.row(m, t.n0);
        static_for<TL::FN / 2>([&](auto p) {
          const f32x4_t y0 = acc[f][2 * p] + bv[2 * p], y1 = acc[f][2 * p + 1] + bv[2 * p + 1];
          const int c = c0 + 32 * p;
          if (part == 2) {
            const int vs = out.vstride();
            bf16* dst = rr.base + (size_t)c * vs;
            static_for<8>([&](auto e) { dst[(size_t)e * vs] = f2bf(e < 4 ? y0[int(e) % 4] : y1[int(e) % 4]); });
          } else {
            const int off = part == 0 ? c : (c >> out.dsh) * out.kstride() + (c & ((1 << out.dsh) - 1));
            *reinterpret_cast<u32x4_t*>(rr.base + off) = pack_bf8(y0, y1);
          }
        });
      }
    });
    if (last) return;
    t = nx;
  }
}

// Two-row-tile blocks run several tiles each, two blocks per CU; one-row-tile blocks, of which
// there are few rounds, run one tile each (with several each: 17.7 -> 20.9 us at 32,400 rows of
// 256, 11.1 -> 12.9 us at 6,480).
template <class TL, int C, class Out>
static void qkv_launch(int M, const bf16* xh, const int32_t* tiles, const int32_t* ntiles, int kv_all,
                       const bf16* w, const Out& out, hipStream_t s) {
  static bool attr = false;
  if (!attr) {
    allow_lds(qkv_kernel<TL, Out, C>, TL::LDS_BYTES);
    attr = true;
  }
  const int mt = (M + TL::BM - 1) / TL::BM;
  const int most = xcd_grid(mt, C / TL::BN) + xcd_grid(mt, 2 * C / TL::BN);
  const int grid = TL::BM == ROW_TILE || most < 512 ? most : 512;
  qkv_kernel<TL, Out, C><<<grid, TL::THREADS, TL::LDS_BYTES, s>>>(M, xh, tiles, ntiles, kv_all, w, out);
}

// One instantiation per network width, with the k loop unrolled (0.8 % per clip at
// 5 x 240 x 432 and 5 x 720 x 1280, timed back to back on one GPU).  BIG_M rows and more take two row tiles per block (4 wavefronts of 64 x 64 outputs:
// half the operand bytes from L2 and LDS per product), fewer rows one row tile on 8
// wavefronts, so that there are blocks for every CU.
template <class Out>
static void qkv_by_c(int M, int C, const bf16* xh, const int32_t* tiles, const int32_t* ntiles, int kv_all,
                     const bf16* w, const Out& out, hipStream_t s) {
  using Big = GemmTile<128, 128, 2, 2, 2>;
  using Small = GemmTile<64, 128, 2, 4, 2>;
  using Narrow = GemmTile<64, 64, 2, 2, 2>;
  const bool big = M >= BIG_M;
  switch (C) {
    case 64: return qkv_launch<Narrow, 64>(M, xh, tiles, ntiles, kv_all, w, out, s);
    case 128:
      return big ? qkv_launch<Big, 128>(M, xh, tiles, ntiles, kv_all, w, out, s)
                 : qkv_launch<Small, 128>(M, xh, tiles, ntiles, kv_all, w, out, s);
    case 256:
      return big ? qkv_launch<Big, 256>(M, xh, tiles, ntiles, kv_all, w, out, s)
                 : qkv_launch<Small, 256>(M, xh, tiles, ntiles, kv_all, w, out, s);
    case 384:
      return big ? qkv_launch<Big, 384>(M, xh, tiles, ntiles, kv_all, w, out, s)
                 : qkv_launch<Small, 384>(M, xh, tiles, ntiles, kv_all, w, out, s);
    default: return;  // rejected by the callers (resid_ln_supported)
  }
}

// log2 of a power of two (head widths 32 and 64 are the ones the attention kernels take)
static int log2_pow2(int v) {
  int k = 0;
  while ((1 << k) < v) ++k;
  return k;
}

void launch_qkv_bf16(const Geo& g, int C, int heads, int Spad, int spv, const bf16* xh, const int32_t* tiles,
                     const int32_t* ntiles, const bf16* w, const float* bias, bf16* q, bf16* k, bf16* vt,
                     hipStream_t s) {
  if (g.N <= 0) return;
  const QkvOut out{bias, q, k, vt, C, log2_pow2(C / heads), heads, Spad, g.S, spv};
  qkv_by_c(g.N, C, xh, tiles, ntiles, 0, w, out, s);
}

void launch_qkv_stream(const Geo& g, int C, int heads, const bf16* xh, const int32_t* tiles, const int32_t* ntiles,
                       const bf16* w, const float* bias, bf16* q, const StreamTable& tab, hipStream_t s) {
  if (g.N <= 0) return;
  const StreamQkvOut out{bias, q, tab, C, log2_pow2(C / heads), heads, g.S, g.nwh * g.nww};
  qkv_by_c(g.N, C, xh, tiles, ntiles, 1, w, out, s);
}

// ------------------------------------------------------------------------------------------
// First MLP linear + GELU over the compact query rows (the first *m_dev rows)
// ------------------------------------------------------------------------------------------
struct GeluOut {
  const float* bias;
  bf16* h;
  int R;
  __device__ __forceinline__ void operator()(int m, int n, const f32x4_t& a) const {
    const float4 b4 = *reinterpret_cast<const float4*>(bias + n);
    uint2 pk;
    // the first and second linears' weights carry GELU's constant factors (gelu_scaled)
    pk.x = pack_bf2(gelu_scaled(a[0] + b4.x), gelu_scaled(a[1] + b4.y));
    pk.y = pack_bf2(gelu_scaled(a[2] + b4.z), gelu_scaled(a[3] + b4.w));
    *reinterpret_cast<uint2*>(h + (size_t)m * R + n) = pk;
  }
};

template <class TL>
__global__ void __launch_bounds__(TL::THREADS) fc1_kernel(const int32_t* __restrict__ m_dev, int C, int R,
                                                  const bf16* __restrict__ u2, const bf16* __restrict__ W,
                                                  GeluOut out) {
  extern __shared__ __align__(16) bf16 ring[];
  const int M = m_dev[0];
  const int nt = R / TL::BN;
  const int mt = (M + TL::BM - 1) / TL::BM;
  // the grid covers the largest possible M (fixed for graph capture); surplus tiles exit
  int rt, ct;
  xcd_tile(blockIdx.x, nt, rt, ct);
  if (rt >= mt) return;
  const int m0 = rt * TL::BM, n0 = ct * TL::BN;
  f32x4_t acc[TL::FM][TL::FN];
  gemm_core<TL>(u2, M, m0, W, n0, C, ring, acc);
  for_fragments<TL>(M, m0, n0, acc, out);
}

template <class TL>
static void fc1_launch(int m_max, const int32_t* m_dev, int C, int R, const bf16* u2, const bf16* w,
                       const float* bias, bf16* h, hipStream_t s) {
  static bool attr = false;
  if (!attr) {
    allow_lds(fc1_kernel<TL>, TL::LDS_BYTES);
    attr = true;
  }
  const int grid = xcd_grid((m_max + TL::BM - 1) / TL::BM, R / TL::BN);
  fc1_kernel<TL><<<grid, TL::THREADS, TL::LDS_BYTES, s>>>(m_dev, C, R, u2, w, GeluOut{bias, h, R});
}

void launch_fc1_bf16(int m_max, const int32_t* m_dev, int C, int R, const bf16* u2, const bf16* w,
                     const float* bias, bf16* h, hipStream_t s) {
  if (m_max <= 0) return;
  if (m_max >= BIG_M && R % 256 == 0)
    fc1_launch<GemmTile<128, 256, 2, 4, 2>>(m_max, m_dev, C, R, u2, w, bias, h, s);
  else if (R % 128 == 0)
    fc1_launch<GemmTile<64, 128, 2, 2, 2>>(m_max, m_dev, C, R, u2, w, bias, h, s);
  else  // dim 64 with an odd MLP ratio
    fc1_launch<GemmTile<64, 64, 2, 2, 3>>(m_max, m_dev, C, R, u2, w, bias, h, s);
}

// ------------------------------------------------------------------------------------------
// Residual linears with the row normalisation in the epilogue.  Block tile 64 rows x the full
// width C (4 wavefronts side by side, each C/4 channels), so each row's statistics are
// complete inside the block: the wavefront sums go through LDS.  Two passes (mean, then the
// centred sum of squares), FP32, biased variance, eps 1e-5.
// ------------------------------------------------------------------------------------------
template <class TL>
__global__ void __launch_bounds__(TL::THREADS) resid_ln_kernel(const int32_t* __restrict__ m_dev, int K,
                                                       const bf16* __restrict__ A, const bf16* __restrict__ W,
                                                       const float* __restrict__ bias, float* __restrict__ x,
                                                       const int32_t* __restrict__ rows, bf16* __restrict__ xh,
                                                       const int32_t* __restrict__ hrows) {
  constexpr int C = TL::BN;
  extern __shared__ __align__(16) bf16 ring[];
  __shared__ float red[2][TL::WN][TL::BM];
  static_assert(TL::WN == 4, "row sums over four column wavefronts");
  const int M = m_dev[0];
  // row tile b: consecutive row tiles run on different XCDs
  const int m0 = blockIdx.x * TL::BM;
  if (m0 >= M) return;
  f32x4_t acc[TL::FM][TL::FN];
  gemm_core<TL>(A, M, m0, W, 0, K, ring, acc);

  const int lane = threadIdx.x & 63, wv = threadIdx.x >> 6;
  const int wm = wv / TL::WN, wn = wv % TL::WN;
  const int l16 = lane & 15, kg = lane >> 4;
  int dst[TL::FM];
  float part[TL::FM];
  static_for<TL::FM>([&](auto i) {
    const int m = m0 + wm * TL::TM + 16 * i + l16;
    const bool ok = m < M;
    dst[i] = ok ? rows[m] : -1;
    float sum = 0.f;
    static_for<TL::FN>([&](auto j) {
      const int n = wn * TL::TN + 16 * j + 4 * kg;
      const float4 b4 = *reinterpret_cast<const float4*>(bias + n);
      float4 xo = make_float4(0.f, 0.f, 0.f, 0.f);
      if (ok) xo = *reinterpret_cast<const float4*>(x + (size_t)dst[i] * C + n);
      f32x4_t& a = acc[i][j];
      a[0] += b4.x + xo.x;
      a[1] += b4.y + xo.y;
      a[2] += b4.z + xo.z;
      a[3] += b4.w + xo.w;
      if (ok) *reinterpret_cast<float4*>(x + (size_t)dst[i] * C + n) = make_float4(a[0], a[1], a[2], a[3]);
      sum += (a[0] + a[1]) + (a[2] + a[3]);
    });
    sum += __shfl_xor(sum, 16, 64);
    sum += __shfl_xor(sum, 32, 64);
    part[i] = sum;
  });
  if (kg == 0) static_for<TL::FM>([&](auto i) { red[0][wn][wm * TL::TM + 16 * i + l16] = part[i]; });
  __syncthreads();
  float mean[TL::FM];
  static_for<TL::FM>([&](auto i) {
    const int r = wm * TL::TM + 16 * i + l16;
    mean[i] = ((red[0][0][r] + red[0][1][r]) + (red[0][2][r] + red[0][3][r])) * (1.0f / C);
    float sq = 0.f;
    static_for<TL::FN>([&](auto j) {
      static_for<4>([&](auto e) {
        const float d = acc[i][j][int(e)] - mean[i];
        sq += d * d;
      });
    });
    sq += __shfl_xor(sq, 16, 64);
    sq += __shfl_xor(sq, 32, 64);
    part[i] = sq;
  });
  if (kg == 0) static_for<TL::FM>([&](auto i) { red[1][wn][wm * TL::TM + 16 * i + l16] = part[i]; });
  __syncthreads();
  static_for<TL::FM>([&](auto i) {
    const int r = wm * TL::TM + 16 * i + l16;
    const float var = ((red[1][0][r] + red[1][1][r]) + (red[1][2][r] + red[1][3][r])) * (1.0f / C);
    const float rstd = rsqrtf(var + 1e-5f);
    if (dst[i] >= 0) {
      const int hr = hrows ? hrows[m0 + r] : m0 + r;
      static_for<TL::FN>([&](auto j) {
        const int n = wn * TL::TN + 16 * j + 4 * kg;
        const f32x4_t& a = acc[i][j];
        uint2 pk;
        pk.x = pack_bf2((a[0] - mean[i]) * rstd, (a[1] - mean[i]) * rstd);
        pk.y = pack_bf2((a[2] - mean[i]) * rstd, (a[3] - mean[i]) * rstd);
        *reinterpret_cast<uint2*>(xh + (size_t)hr * C + n) = pk;
      });
    }
  });
}

template <class TL>
static void resid_ln_launch(int m_max, const int32_t* m_dev, int K, const bf16* A, const bf16* w, const float* bias,
                            float* x, const int32_t* rows, bf16* xh, const int32_t* hrows, hipStream_t s) {
  static bool attr = false;
  if (!attr) {
    allow_lds(resid_ln_kernel<TL>, TL::LDS_BYTES);
    attr = true;
  }
  resid_ln_kernel<TL><<<(m_max + TL::BM - 1) / TL::BM, TL::THREADS, TL::LDS_BYTES, s>>>(m_dev, K, A, w, bias, x, rows, xh, hrows);
}

bool resid_ln_supported(int C) { return C == 64 || C == 128 || C == 256 || C == 384; }

void launch_resid_ln_bf16(int m_max, const int32_t* m_dev, int C, int K, const bf16* A, const bf16* w,
                          const float* bias, float* x, const int32_t* rows, bf16* xh, const int32_t* hrows,
                          hipStream_t s) {
  if (m_max <= 0) return;
  switch (C) {
    case 64: resid_ln_launch<GemmTile<64, 64, 1, 4, 3>>(m_max, m_dev, K, A, w, bias, x, rows, xh, hrows, s); break;
    case 128: resid_ln_launch<GemmTile<64, 128, 1, 4, 3>>(m_max, m_dev, K, A, w, bias, x, rows, xh, hrows, s); break;
    case 256: resid_ln_launch<GemmTile<64, 256, 1, 4, 3>>(m_max, m_dev, K, A, w, bias, x, rows, xh, hrows, s); break;
    case 384: resid_ln_launch<GemmTile<64, 384, 2, 4, 2>>(m_max, m_dev, K, A, w, bias, x, rows, xh, hrows, s); break;
    default: break;  // rejected by the caller (resid_ln_supported)
  }
}

// ------------------------------------------------------------------------------------------
// Fused post-attention block over 64 (or 32) query rows (compact rows r, token idx[r]):
//   x1 = x + o W_o^T + b_o        u2 = normalise(x1)
//   h  = GELU(u2 W1'^T + b1')     (hidden chunks of HC columns)
//   x2 = x1 + h W_2^T + b_2       x^ = normalise(x2)
// u2 and h never leave LDS: the o rows are loaded once into a resident A tile that u2 then
// overwrites, each hidden chunk is written to LDS by the GELU epilogue and immediately
// consumed by the second linear.  Only the weights stream, through a 3-stage ring whose
// stages are, in order: the C/64 k-blocks of W_o; then per hidden chunk j the C/64 k-blocks
// of W1' rows [j*HC, (j+1)*HC) followed by the HC/64 k-blocks of W_2 columns of chunk j.
// Block = 512 threads = 8 wavefronts in 2 (rows) x 4 (columns): the block needs most of the
// LDS, so it runs alone on its CU, and two wavefronts per SIMD keep the matrix pipe fed
// while the other waits on LDS or the barrier.
// ------------------------------------------------------------------------------------------
constexpr int MLP_THREADS = 512;
// A block's chain of weight stages takes 28 us at dim 256 with 64 rows, however few blocks there
// are, and 21 us with 32 (half the products, fragment reads of rows and GELU per stage, the same
// weight stream).  So rows are split over 32-row blocks while every one of them has a CU of its
// own (one 5 x 240 x 432 stream, ~1,700 query rows: 465 -> 412 us per frame); beyond 256 of them
// a second turn (42 us) would cost more than 64-row blocks do (30 us).
constexpr int MLP_SMALL_BLOCKS = 256;

template <int C_, int HC_, int BM_ = 64, int ST_ = 3, int SR_ = 0>
struct MlpCfg {
  using Small = MlpCfg<C_, HC_, 32, ST_, SR_>;
  static constexpr int C = C_, HC = HC_, BM = BM_, R = 4 * C, ST = ST_;
  static constexpr int WM = 2, WN = 4, TM = BM / WM;   // wavefront grid; rows per wavefront
  static constexpr int FM = TM / 16;
  static constexpr int SLOT_ROWS = SR_ ? SR_ : (C > HC ? C : HC);
  static constexpr int SLOT = SLOT_ROWS * 64;          // bf16 elements per ring slot
  static constexpr int NKC = C / 64, NKH = HC / 64;    // k blocks of C- and HC-wide operands
  static constexpr int NCH = R / HC;                   // hidden chunks
  // a k block of a C-row weight (W_o, W_2) moves in NHALF stages of CS rows when a slot
  // holds fewer than C rows
  static constexpr int CS = C < SLOT_ROWS ? C : SLOT_ROWS, NHALF = C / CS;
  // k blocks of W1' per stage: as many HC-row blocks as a ring slot holds, so that every
  // stage moves a full slot (fewer stages, each with the same fixed wait + barrier cost)
  static constexpr int KB1 = (SLOT_ROWS / HC < NKC) ? SLOT_ROWS / HC : NKC;
  static constexpr int NW1 = NKC / KB1;                // W1' stages per hidden chunk
  static constexpr int PER_CHUNK = NW1 + NKH * NHALF;
  static constexpr int NSTAGE = NKC * NHALF + NCH * PER_CHUNK;
  static constexpr int FN_C = C / 64, FN_H = HC / 64;  // 16-wide fragments per wavefront
  static constexpr int FPH = FN_C / NHALF;             // of them per C-row stage
  static constexpr int NFW = FPH > KB1 * FN_H ? FPH : KB1 * FN_H;  // weight fragments per slice (half a stage)
  // stage s: of W1'; else its k block and half of W_2
  __device__ static constexpr bool is_w1(int s) {
    return s >= NKC * NHALF && (s - NKC * NHALF) % PER_CHUNK < NW1;
  }
  __device__ static constexpr int kb2(int s) { return ((s - NKC * NHALF) % PER_CHUNK - NW1) / NHALF; }
  __device__ static constexpr int half2(int s) { return ((s - NKC * NHALF) % PER_CHUNK - NW1) % NHALF; }
  // output column of wavefront wn's fragment j (lane group kg adds 4 kg): the wavefront's
  // columns are spread over the NHALF row ranges of a C-row stage, FPH fragments in each
  __device__ static constexpr int col(int wn, int j) { return (j / FPH) * CS + wn * 16 * FPH + 16 * (j % FPH); }
  static constexpr size_t RING = (size_t)ST * SLOT, ARES = (size_t)NKC * BM * 64, HRES = (size_t)NKH * BM * 64;
  static constexpr size_t FLOATS = 2 * (size_t)C + R + 2 * WN * BM + BM;  // b_o, b1', b_2, row sums, token rows
  static constexpr size_t LDS_BYTES = (RING + ARES + HRES) * 2 + FLOATS * 4;
  static_assert(C % 64 == 0 && HC % 64 == 0 && R % HC == 0 && NKC % KB1 == 0, "shapes");
  static_assert(C % CS == 0 && FN_C % NHALF == 0 && CS % (16 * WN) == 0 && SLOT_ROWS >= HC, "C-row stages");
  static_assert((BM == 32 || BM == 64) && (ST == 2 || ST == 3), "row tile and ring depth");
  // x1 (the residual after the projection) kept in registers for the second residual, rather
  // than stored to x and read back, where the registers allow it
  static constexpr bool X1_REGS = C <= 256 || BM == 32;
  static_assert(LDS_BYTES <= 160 * 1024, "LDS");
};

// A 16-row operand fragment (rows row0 + l % 16, k slice kk of a 64-wide k block) of a swizzled
// 64-column LDS tile.
__device__ __forceinline__ bf16x8_t lds_frag(const bf16* tile, int row0, int kk) {
  const int lane = threadIdx.x & 63, row = row0 + (lane & 15), kg = lane >> 4;
  return *reinterpret_cast<const bf16x8_t*>(tile + row * 64 + (((4 * kk + kg) ^ lds_swz(row)) * 8));
}

// Element offset of (row r, column c) in a resident [k block][BM rows][64] swizzled tile.
template <int BM = 64>
__device__ __forceinline__ int res_off(int r, int c) {
  return (c >> 6) * (BM * 64) + r * 64 + ((((c & 63) >> 3) ^ lds_swz(r)) << 3) + (c & 7);
}

// This thread's residual values x[row] for the [BM][C] accumulators: FM * FN_C loads of every
// wavefront, whatever its rows (the counted waits rely on that; of native vectors, since the
// compiler's vectoriser moves the four loads of a float4 struct to where they are used).
template <class MC>
__device__ __forceinline__ void load_resid(const float* __restrict__ x, const int (&row)[MC::FM],
                                           f32x4_t (&xo)[MC::FM][MC::FN_C]) {
  const int lane = threadIdx.x & 63, wv = threadIdx.x >> 6;
  const int wn = wv % MC::WN, kg = lane >> 4;
  static_for<MC::FM>([&](auto i) {
    static_for<MC::FN_C>([&](auto j) {
      const int n = MC::col(wn, j) + 4 * kg;
      xo[i][j] = *reinterpret_cast<const f32x4_t*>(x + (size_t)row[i] * MC::C + n);
    });
  });
}

// Residual + row normalisation for the [64][C] accumulators: acc += bias + xo (= x[dst]);
// x[dst] = acc; the row statistics come back through mean/rstd.  The four column
// wavefronts of a row group exchange partial sums through red[2][WN][BM].
template <class MC>
__device__ __forceinline__ void resid_rows(f32x4_t (&acc)[MC::FM][MC::FN_C], const float* sbias,
                                           float* __restrict__ x, const int (&dst)[MC::FM],
                                           const f32x4_t (&xo_in)[MC::FM][MC::FN_C], float (*red)[MC::WN][MC::BM],
                                           float (&mean)[MC::FM], float (&rstd)[MC::FM], bool store = true) {
  constexpr int C = MC::C, FN = MC::FN_C;
  // the thread index passes through an empty asm so that the column addresses below are
  // recomputed per call rather than kept live (or spilled) from an earlier call
  int tid = threadIdx.x;
  asm volatile("" : "+v"(tid));
  const int lane = tid & 63, wv = tid >> 6;
  const int wm = wv / MC::WN, wn = wv % MC::WN;
  const int l16 = lane & 15, kg = lane >> 4;
  float part[MC::FM];
  static_for<MC::FM>([&](auto i) {
    float sum = 0.f;
    static_for<FN>([&](auto j) {
      const int n = MC::col(wn, j) + 4 * kg;
      const f32x4_t xo = xo_in[i][j];
      f32x4_t& a = acc[i][j];
      a[0] += sbias[n] + xo[0];
      a[1] += sbias[n + 1] + xo[1];
      a[2] += sbias[n + 2] + xo[2];
      a[3] += sbias[n + 3] + xo[3];
      if (store && dst[i] >= 0)
        *reinterpret_cast<float4*>(x + (size_t)dst[i] * C + n) = make_float4(a[0], a[1], a[2], a[3]);
      sum += (a[0] + a[1]) + (a[2] + a[3]);
    });
    sum += __shfl_xor(sum, 16, 64);
    sum += __shfl_xor(sum, 32, 64);
    part[i] = sum;
  });
  if (kg == 0) static_for<MC::FM>([&](auto i) { red[0][wn][wm * MC::TM + 16 * i + l16] = part[i]; });
  lds_barrier();
  static_for<MC::FM>([&](auto i) {
    const int r = wm * MC::TM + 16 * i + l16;
    mean[i] = ((red[0][0][r] + red[0][1][r]) + (red[0][2][r] + red[0][3][r])) * (1.0f / C);
    float sq = 0.f;
    static_for<FN>([&](auto j) {
      static_for<4>([&](auto e) {
        const float d = acc[i][j][int(e)] - mean[i];
        sq += d * d;
      });
    });
    sq += __shfl_xor(sq, 16, 64);
    sq += __shfl_xor(sq, 32, 64);
    part[i] = sq;
  });
  if (kg == 0) static_for<MC::FM>([&](auto i) { red[1][wn][wm * MC::TM + 16 * i + l16] = part[i]; });
  lds_barrier();
  static_for<MC::FM>([&](auto i) {
    const int r = wm * MC::TM + 16 * i + l16;
    const float var = ((red[1][0][r] + red[1][1][r]) + (red[1][2][r] + red[1][3][r])) * (1.0f / C);
    rstd[i] = rsqrtf(var + 1e-5f);
  });
}

template <class MC>
__device__ __forceinline__ void mlp_block(int M, const bf16* __restrict__ o, const int32_t* __restrict__ rows,
                                          const bf16* __restrict__ Wo, const float* __restrict__ bo,
                                          const bf16* __restrict__ W1, const float* __restrict__ b1,
                                          const bf16* __restrict__ W2, const float* __restrict__ b2,
                                          float* __restrict__ x, bf16* __restrict__ xh) {
  constexpr int C = MC::C, HC = MC::HC, R = MC::R, BM = MC::BM, NW = MLP_THREADS / 64;
  extern __shared__ __align__(16) bf16 lds[];
  bf16* ring = lds;
  bf16* ares = lds + MC::RING;
  bf16* hres = ares + MC::ARES;
  float* sbo = reinterpret_cast<float*>(hres + MC::HRES);
  float* sb1 = sbo + C;
  float* sb2 = sb1 + R;
  float(*red)[MC::WN][MC::BM] = reinterpret_cast<float(*)[MC::WN][MC::BM]>(sb2 + C);
  int* sdst = reinterpret_cast<int*>(sb2 + C + 2 * MC::WN * BM);

  const int m0 = blockIdx.x * BM;
  if (m0 >= M) return;
  const int t = threadIdx.x, lane = t & 63, wv = t >> 6;
  const int wm = wv / MC::WN, wn = wv % MC::WN;
  const int l16 = lane & 15, kg = lane >> 4;

  // the rows' token indices first: the residual loads below need them
  int row[MC::FM];
  static_for<MC::FM>([&](auto i) { row[i] = rows[min(m0 + wm * MC::TM + 16 * i + l16, M - 1)]; });
  // the biases into registers now, into LDS after the loads below are queued: one round trip
  // for all of them instead of one per loop iteration
  constexpr int NBC = (C + MLP_THREADS - 1) / MLP_THREADS, NBR = (R + MLP_THREADS - 1) / MLP_THREADS;
  float vbo[NBC], vb2[NBC], vb1[NBR];
  static_for<NBC>([&](auto k) {
    const int i = min(t + MLP_THREADS * k, C - 1);
    vbo[k] = bo[i];
    vb2[k] = b2[i];
  });
  static_for<NBR>([&](auto k) { vb1[k] = b1[min(t + MLP_THREADS * k, R - 1)]; });
  const int uwv = __builtin_amdgcn_readfirstlane(wv);
  // o rows -> resident A tile (rows >= M read row M-1; their results are never stored):
  // 8 rows per load, BM / 8 row groups per k block, one group per wavefront
  if (BM == 8 * NW || uwv * 8 < BM)
    static_for<MC::NKC>([&](auto kb) {
      const int row = wv * 8 + (lane >> 3);
      const int m = min(m0 + row, M - 1);
      dma16(o + (size_t)m * C + 64 * kb + ((lane & 7) ^ lds_swz(row)) * 8, ares + kb * BM * 64 + wv * 512);
    });
  // weight stages: stage s holds rows [0, stage_rows(s)) of 64 k columns; a W1' stage holds
  // KB1 blocks of HC rows, k block b of the stage at rows [b HC, (b+1) HC)
  constexpr auto stage_rows = [](int s) {
    if (s < MC::NKC * MC::NHALF) return MC::CS;
    const int tt = (s - MC::NKC * MC::NHALF) % MC::PER_CHUNK;
    return tt < MC::NW1 ? HC * MC::KB1 : MC::CS;
  };
  // a lane's source: a byte offset in the stage's first 64 rows (row stride C or R) from a
  // uniform address, so a load needs no vector arithmetic and two registers serve every stage
  const int lrow = wv * 8 + (lane >> 3), lcol = ((lane & 7) ^ lds_swz(lrow)) * 16;
  const uint32_t off_c = lrow * C * 2 + lcol, off_r = lrow * R * 2 + lcol;
  auto issue = [&](auto s) {
    const bf16* base;
    constexpr bool w2 = s >= MC::NKC * MC::NHALF && !MC::is_w1(s);
    constexpr int ld = w2 ? R : C, blk_rows = MC::is_w1(s) ? HC : MC::CS;  // row stride; rows per k block in the slot
    static_assert(blk_rows % (8 * NW) == 0, "whole loads of 64 rows");
    if constexpr (s < MC::NKC * MC::NHALF) {
      base = Wo + (size_t)(s % MC::NHALF) * MC::CS * C + 64 * (s / MC::NHALF);
    } else {
      constexpr int j = (s - MC::NKC * MC::NHALF) / MC::PER_CHUNK, tt = (s - MC::NKC * MC::NHALF) % MC::PER_CHUNK;
      if constexpr (tt < MC::NW1)
        base = W1 + (size_t)j * HC * C + 64 * MC::KB1 * tt;
      else
        base = W2 + (size_t)MC::half2(s) * MC::CS * R + j * HC + 64 * MC::kb2(s);
    }
    bf16* dst = ring + (s % MC::ST) * MC::SLOT + uwv * 512;
    static_for<stage_rows(s) / (8 * NW)>([&](auto c) {
      constexpr int row = 8 * NW * c, b = row / blk_rows, rr = row % blk_rows;
      dma16(reinterpret_cast<const char*>(base + (size_t)rr * ld + 64 * b) + (w2 ? off_r : off_c), dst + row * 64);
    });
  };
  static_for<MC::ST - 1>([&](auto s0) {
    mfma_fence_begin();  // the loads are counted below in this order
    issue(s0);
  });
  mfma_fence_begin();
  // the residual rows for the projection's epilogue, requested now (after the first stages) so
  // that their latency hides behind the projection: the first two stage waits leave these NX
  // loads outstanding, the third covers them.  Every wavefront issues all of them: were they
  // guarded by dst, one whose rows are all past M would wait for too little.
  f32x4_t xo[MC::FM][MC::FN_C];
  // (the row numbers are first used here: in front of the stages these would wait for them)
#pragma unroll
  for (int i = 0; i < MC::FM; ++i) asm volatile("" : "+v"(row[i]));
  load_resid<MC>(x, row, xo);
  constexpr int NX = MC::FM * MC::FN_C;
  mfma_fence_begin();
  int dst[MC::FM];  // -1: a row past M, which repeats row M-1 and stores nothing
  static_for<MC::FM>([&](auto i) { dst[i] = m0 + wm * MC::TM + 16 * i + l16 < M ? row[i] : -1; });
  // (threads past the last value repeat it)
  static_for<NBC>([&](auto k) {
    const int i = min(t + MLP_THREADS * k, C - 1);
    sbo[i] = vbo[k];
    sb2[i] = vb2[k];
  });
  static_for<NBR>([&](auto k) { sb1[min(t + MLP_THREADS * k, R - 1)] = vb1[k]; });
  // the token rows wait in LDS for the last epilogue (in registers they would be spilled); the
  // wavefronts and lane groups that share a row write the same value
  static_for<MC::FM>([&](auto i) { sdst[wm * MC::TM + 16 * i + l16] = dst[i]; });
  f32x4_t acc[MC::FM][MC::FN_C], hacc[MC::FM][MC::FN_H];
  static_for<MC::FM>([&](auto i) {
    static_for<MC::FN_C>([&](auto j) { acc[i][j] = f32x4_t{0.f, 0.f, 0.f, 0.f}; });
    static_for<MC::FN_H>([&](auto j) { hacc[i][j] = f32x4_t{0.f, 0.f, 0.f, 0.f}; });  // set per chunk below
  });
  float mean[MC::FM], rstd[MC::FM];
  static_assert(MC::ST == 3, "the counted waits below assume a 3-stage ring");
  // Every stage is multiplied in two slices, and the fragments of slice n + 1 are read from LDS
  // among the products of slice n, also over the stage boundary: the wait and barrier that
  // make stage s + 1 visible come before the last products of stage s, so that the matrix
  // cores work while the wavefronts wait and read.  (After a direct global->LDS load the
  // compiler waits for all LDS reads before the first product that needs one, so the reads of
  // the next slice are issued after that product, not before it.)  (Reading both slices after the barrier and
  // then multiplying, every stage waited for all its reads: 1,100 + 360 cycles per stage for
  // 512 of matrix-core time.)  Fragments: of W_o and W_2, slice q holds the 32-wide k slice q
  // of the stage; of W1', KB1 of the stage's 2 KB1 (k block, slice) pairs.
  bf16x8_t fa[2][MC::FM], fw[2][MC::NFW];
  constexpr int S1 = MC::NKC * MC::NHALF;  // W_o stages
  bf16x8_t ua[MC::NKC][2][MC::FM];
  auto load_w = [&](auto s, auto q) {
    const bf16* ws = ring + (s % MC::ST) * MC::SLOT;
    if constexpr (MC::is_w1(s))
      static_for<MC::KB1>([&](auto p) {
        constexpr int pair = q * MC::KB1 + p, b = pair / 2, kk = pair % 2;
        static_for<MC::FN_H>([&](auto j) {
          fw[q][p * MC::FN_H + j] = lds_frag(ws + b * HC * 64, wn * 16 * MC::FN_H + 16 * j, kk);
        });
      });
    else
      static_for<MC::FPH>([&](auto j) { fw[q][j] = lds_frag(ws, wn * 16 * MC::FPH + 16 * j, q); });
  };
  auto load_a = [&](auto s, auto q) {  // rows of o (W_o stages) or of the H tile (W_2 stages)
    if constexpr (!MC::is_w1(s)) {
      const bf16* tile = s < S1 ? ares + (s / MC::NHALF) * BM * 64 : hres + MC::kb2(s) * BM * 64;
      static_for<MC::FM>([&](auto i) { fa[q][i] = lds_frag(tile, wm * MC::TM + 16 * i, q); });
    }
  };
  // The products of slice q of stage s; `between` runs after the first of them, whose operands
  // stay allocated to the end, so that nothing `between` writes shares a register that the
  // product in flight still reads.
  auto multiply = [&](auto s, auto q, auto&& between) {
    mfma_fence_begin();
    bool first = true;
    auto after_first = [&] {
      if (first) {
        first = false;
        mfma_fence_begin();
        between();
        mfma_fence_begin();
      }
    };
    if constexpr (MC::is_w1(s)) {
      constexpr int tt = (s - S1) % MC::PER_CHUNK;
      static_for<MC::KB1>([&](auto p) {
        constexpr int pair = q * MC::KB1 + p, kb = tt * MC::KB1 + pair / 2, kk = pair % 2;
        static_for<MC::FM>([&](auto i) {
          static_for<MC::FN_H>([&](auto j) {
            hacc[i][j] = mfma_bf16_16x16x32(fw[q][p * MC::FN_H + j], ua[kb][kk][i], hacc[i][j]);
            after_first();
          });
        });
      });
      mfma_fence_end();
      asm volatile("" ::"v"(fw[q][0]), "v"(ua[tt * MC::KB1 + q * MC::KB1 / 2][q * MC::KB1 % 2][0]));
    } else {
      constexpr int j0 = (s < S1 ? s % MC::NHALF : MC::half2(s)) * MC::FPH;
      static_for<MC::FM>([&](auto i) {
        static_for<MC::FPH>([&](auto j) {
          acc[i][j0 + j] = mfma_bf16_16x16x32(fw[q][j], fa[q][i], acc[i][j0 + j]);
          after_first();
        });
      });
      mfma_fence_end();
      asm volatile("" ::"v"(fw[q][0]), "v"(fa[q][0]));
    }
  };
  using I0 = std::integral_constant<int, 0>;
  using I1 = std::integral_constant<int, 1>;
  using INX = std::integral_constant<int, NX>;
  // Make stage s visible: wait for this wavefront's loads of it (at most the next stage's and
  // `more` other later vector-memory loads may be outstanding), then the block barrier; every
  // wavefront has then also finished reading stage s - 1, whose slot the loads of stage
  // s + ST - 1 overwrite.
  auto visible = [&](auto s, auto more) {
    constexpr int next = s + 1 < MC::NSTAGE ? stage_rows(s + 1) / (8 * NW) : 0;
    vm_wait_barrier<next + more>();
    lds_reads_done();
  };
  // read the first slice of stage s (visible) and queue stage s + ST - 1
  auto enter = [&](auto s, bool a_ready) {
    load_w(s, I0{});
    if (a_ready) load_a(s, I0{});
    mfma_fence_begin();
    if constexpr (s + MC::ST - 1 < MC::NSTAGE) issue(std::integral_constant<int, s + MC::ST - 1>{});
  };
  // Stage s with its first slice loaded; makes stage s + 1 visible before the last products.
  auto stage = [&](auto s, auto more, bool enter_next, bool a_ready) {
    constexpr bool last = s + 1 >= MC::NSTAGE;
    using Next = std::integral_constant<int, last ? s : s + 1>;
    multiply(s, I0{}, [&] {
      load_w(s, I1{});
      load_a(s, I1{});
    });
    if constexpr (!last)
      if (enter_next) visible(Next{}, more);
    multiply(s, I1{}, [&] {
      if constexpr (!last)
        if (enter_next) enter(Next{}, a_ready);
    });
  };
  // The x rows were requested after stages 0 and 1, so the first two waits leave them
  // outstanding and the third covers them.
  visible(I0{}, INX{});
  enter(I0{}, true);
  static_for<S1>([&](auto s) {
    if constexpr (s == 0)
      stage(s, INX{}, S1 > 1, true);
    else
      stage(s, I0{}, s + 1 < S1, true);
  });
  // x1 = x + o W_o^T + b_o; u2 = normalise(x1) into the resident tile (every wavefront has
  // finished reading o there: resid_rows passes two block barriers)
  // x1 stays in registers (xo) for the second residual (or goes to x and is read back)
  resid_rows<MC>(acc, sbo, x, dst, xo, red, mean, rstd, !MC::X1_REGS);
  if constexpr (MC::X1_REGS)
    static_for<MC::FM>([&](auto i) {
      static_for<MC::FN_C>([&](auto j) { xo[i][j] = acc[i][j]; });
    });
  static_for<MC::FM>([&](auto i) {
    const int r = wm * MC::TM + 16 * i + l16;
    static_for<MC::FN_C>([&](auto j) {
      const int n = MC::col(wn, j) + 4 * kg;
      const f32x4_t& a = acc[i][j];
      uint2 pk;
      pk.x = pack_bf2((a[0] - mean[i]) * rstd[i], (a[1] - mean[i]) * rstd[i]);
      pk.y = pack_bf2((a[2] - mean[i]) * rstd[i], (a[3] - mean[i]) * rstd[i]);
      *reinterpret_cast<uint2*>(ares + res_off<MC::BM>(r, n)) = pk;
      acc[i][j] = f32x4_t{0.f, 0.f, 0.f, 0.f};
    });
  });
  // this wavefront's u2 fragments stay in registers for every hidden chunk
  lds_barrier();
  static_for<MC::NKC>([&](auto kb) {
    static_for<2>([&](auto kk) {
      static_for<MC::FM>([&](auto i) { ua[kb][kk][i] = lds_frag(ares + kb * BM * 64, wm * MC::TM + 16 * i, kk); });
    });
  });
  // x was read (and written): wait for everything, the ring's two stages included
  vm_wait_barrier<0>();
  lds_reads_done();
  enter(std::integral_constant<int, S1>{}, true);
  // unrolled: every stage index, ring slot and wait count below is a constant (1.2 % per clip
  // at 5 x 240 x 432, timed back to back on one GPU)
  static_for<MC::NCH>([&](auto j) {
    // the chunk's accumulators start at its bias b1' (the GELU epilogue then adds nothing)
    static_for<MC::FN_H>([&](auto jj) {
      const f32x4_t b4 = lds_as_bf16<f32x4_t>(sb1 + j * HC + wn * 16 * MC::FN_H + 16 * jj + 4 * kg);
      static_for<MC::FM>([&](auto i) { hacc[i][jj] = b4; });
    });
    constexpr int s1 = S1 + j * MC::PER_CHUNK, s2 = s1 + MC::NW1;
    // (the last W1' stage enters the first W_2 stage, whose H rows do not exist yet)
    static_for<MC::NW1>([&](auto tt) { stage(std::integral_constant<int, s1 + tt>{}, I0{}, true, tt + 1 < MC::NW1); });
    // hidden chunk j: GELU into the H tile (its previous contents were consumed before this
    // stage's barrier); the weights carry GELU's constant factors (gelu_scaled)
    static_for<MC::FM>([&](auto i) {
      const int r = wm * MC::TM + 16 * i + l16;
      static_for<MC::FN_H>([&](auto jj) {
        const int c = wn * 16 * MC::FN_H + 16 * jj + 4 * kg;
        const f32x4_t& a = hacc[i][jj];
        *reinterpret_cast<bf16x4_t*>(hres + res_off<MC::BM>(r, c)) =
            bf16x4_t{(__bf16)gelu_scaled(a[0]), (__bf16)gelu_scaled(a[1]), (__bf16)gelu_scaled(a[2]), (__bf16)gelu_scaled(a[3])};
      });
    });
    lds_barrier();
    load_a(std::integral_constant<int, s2>{}, I0{});
    static_for<MC::NKH * MC::NHALF>([&](auto u) { stage(std::integral_constant<int, s2 + u>{}, I0{}, true, true); });
  });
  // x2 = x1 + h W_2^T + b_2; x^ = normalise(x2)
  static_for<MC::FM>([&](auto i) {
    dst[i] = sdst[wm * MC::TM + 16 * i + l16];
    row[i] = max(dst[i], 0);
  });
  if constexpr (!MC::X1_REGS) load_resid<MC>(x, row, xo);  // this thread's own stores, an L2 hit
  resid_rows<MC>(acc, sb2, x, dst, xo, red, mean, rstd);
  static_for<MC::FM>([&](auto i) {
    if (dst[i] >= 0)
      static_for<MC::FN_C>([&](auto j) {
        const int n = MC::col(wn, j) + 4 * kg;
        const f32x4_t& a = acc[i][j];
        uint2 pk;
        pk.x = pack_bf2((a[0] - mean[i]) * rstd[i], (a[1] - mean[i]) * rstd[i]);
        pk.y = pack_bf2((a[2] - mean[i]) * rstd[i], (a[3] - mean[i]) * rstd[i]);
        *reinterpret_cast<uint2*>(xh + (size_t)dst[i] * C + n) = pk;
      });
  });
}

// The row count is known on the device only, so the kernel holds both row tiles (MLP_SMALL_BLOCKS;
// next to a kernel with the larger one alone that costs the larger one at most 0.4 % of a clip).
template <class MC>
__global__ void __launch_bounds__(MLP_THREADS) mlp_block_kernel(const int32_t* __restrict__ m_dev,
                                                                const bf16* __restrict__ o,
                                                                const int32_t* __restrict__ rows,
                                                                const bf16* __restrict__ Wo, const float* __restrict__ bo,
                                                                const bf16* __restrict__ W1, const float* __restrict__ b1,
                                                                const bf16* __restrict__ W2, const float* __restrict__ b2,
                                                                float* __restrict__ x, bf16* __restrict__ xh) {
  const int M = m_dev[0];
  if (M <= 32 * MLP_SMALL_BLOCKS)
    mlp_block<typename MC::Small>(M, o, rows, Wo, bo, W1, b1, W2, b2, x, xh);
  else
    mlp_block<MC>(M, o, rows, Wo, bo, W1, b1, W2, b2, x, xh);
}

template <class MC>
static void mlp_launch(int m_max, const int32_t* m_dev, const bf16* o, const int32_t* rows, const bf16* wo,
                       const float* bo, const bf16* w1, const float* b1, const bf16* w2, const float* b2, float* x,
                       bf16* xh, hipStream_t s) {
  constexpr size_t bytes = std::max(MC::LDS_BYTES, MC::Small::LDS_BYTES);
  static bool attr = false;
  if (!attr) {
    allow_lds(mlp_block_kernel<MC>, bytes);
    attr = true;
  }
  const int grid = std::max((m_max + MC::BM - 1) / MC::BM, std::min((m_max + 31) / 32, MLP_SMALL_BLOCKS));
  mlp_block_kernel<MC><<<grid, MLP_THREADS, bytes, s>>>(m_dev, o, rows, wo, bo, w1, b1, w2, b2, x, xh);
}

bool mlp_block_supported(int C, int R) { return R == 4 * C && (C == 64 || C == 128 || C == 256 || C == 384); }

void launch_mlp_block_bf16(int m_max, const int32_t* m_dev, int C, const bf16* o, const int32_t* rows,
                           const bf16* wo, const float* bo, const bf16* w1, const float* b1, const bf16* w2,
                           const float* b2, float* x, bf16* xh, hipStream_t s) {
  if (m_max <= 0) return;
  switch (C) {
    case 64: mlp_launch<MlpCfg<64, 128>>(m_max, m_dev, o, rows, wo, bo, w1, b1, w2, b2, x, xh, s); break;
    case 128: mlp_launch<MlpCfg<128, 128>>(m_max, m_dev, o, rows, wo, bo, w1, b1, w2, b2, x, xh, s); break;
    case 256: mlp_launch<MlpCfg<256, 128>>(m_max, m_dev, o, rows, wo, bo, w1, b1, w2, b2, x, xh, s); break;
    // dim 384: 64-row tiles with 192-row weight slots (W_o and W_2 k blocks in two halves) and
    // 192-wide hidden chunks fit the LDS (155 KB)
    case 384: mlp_launch<MlpCfg<384, 192, 64, 3, 192>>(m_max, m_dev, o, rows, wo, bo, w1, b1, w2, b2, x, xh, s); break;
    default: break;  // rejected by the caller (mlp_block_supported)
  }
}

}  // namespace dr
