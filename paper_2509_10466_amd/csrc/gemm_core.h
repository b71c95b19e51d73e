// BF16 GEMM core for gfx950: C[m][n] = sum_k A[m][k] * W[n][k], FP32 accumulation on
// v_mfma_f32_16x16x32_bf16.
//
// Block = 64 WM WN threads (4 or 8 wavefronts) in a WM x WN grid; block tile BM tokens x BN
// output channels; K is consumed 64 at a time through an ST-stage ring in LDS.  Each stage holds the
// BM rows of A followed by the BN rows of W, 128 bytes (64 bf16) per row, and is filled by
// direct global->LDS loads (global_load_lds_dwordx4: each lane of a wavefront moves 16 bytes,
// lane i landing at byte 16*i of the wavefront's 1 KB destination, i.e. 8 rows per
// instruction) -- no VGPR staging, no LDS store instructions.  Stage kt+ST-1 is issued while
// stage kt is multiplied; a wavefront waits for its own loads of stage kt with an explicit
// vmcnt and the block barrier then makes every wavefront's loads visible.
//
// LDS layout: the 16-byte chunk c of row r sits at chunk position c ^ (r & 7).  The MFMA
// operand reads fetch 16 consecutive rows at one logical chunk; measured on gfx950 with the
// SQ_LDS_BANK_CONFLICT counter, this XOR pattern reads those 16 rows without bank conflicts
// (unswizzled 128-byte rows, 144-byte padded rows and an XOR with (r ^ (r >> 3)) & 7 all
// conflict).  The loads apply the same swizzle to the global addresses.
//
// MFMA operands: lane l supplies row (l % 16) of each operand with k values 8*(l/16)..+7 of
// the 32-wide k slice.  The W fragment is the MFMA's A operand, so result lane l holds output
// channels 4*(l/16)..+3 of token (l % 16) within the 16 x 16 fragment.  acc[i][j] covers
// tokens m0 + wm*TM + 16 i + (l % 16) and channels n0 + wn*TN + 16 j + 4 (l / 16) + e.
//
// Double-rate MFMA groups are fenced as everywhere in this library (scheduling barriers,
// then s_nop 7 after the group): a VALU write to a source VGPR of an in-flight
// v_mfma_f32_16x16x32_bf16 corrupts its product.
#pragma once

#include "dr_device.h"

namespace dr {

typedef uint16_t bf16_t;

__device__ __forceinline__ int lds_swz(int row) { return row & 7; }

__device__ __forceinline__ f32x4_t mfma_bf16_16x16x32(const bf16x8_t& a, const bf16x8_t& b, const f32x4_t& c) {
  return __builtin_amdgcn_mfma_f32_16x16x32_bf16(a, b, c, 0, 0, 0);
}

__device__ __forceinline__ void mfma_fence_begin() { __builtin_amdgcn_sched_barrier(0); }
__device__ __forceinline__ void mfma_fence_end() {
  __builtin_amdgcn_sched_barrier(0);
  asm volatile("s_nop 7" ::: "memory");
  __builtin_amdgcn_sched_barrier(0);
}

// Wait until at most N of this wavefront's vector-memory operations are outstanding and its
// LDS operations are done, then the block barrier.  Written as one asm statement with a
// memory clobber so that the compiler neither adds a full vmcnt(0) wait (as a fenced
// __syncthreads would) nor moves LDS accesses across the barrier.
template <int N>
__device__ __forceinline__ void vm_wait_barrier() {
  static_assert(N >= 0 && N < 64, "vmcnt range");
  asm volatile("s_waitcnt vmcnt(%0) lgkmcnt(0)\n\ts_barrier" ::"n"(N) : "memory");
}

// Tells the compiler what the lgkmcnt(0) of an asm wait above did (it does not read asm), so
// that it adds no wait of its own for the LDS reads before it.  gfx9 encoding: vmcnt 63,
// expcnt 7, lgkmcnt 0.
__device__ __forceinline__ void lds_reads_done() { __builtin_amdgcn_s_waitcnt(0xC07F); }

__device__ __forceinline__ void lds_barrier() { asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory"); }

__device__ __forceinline__ void dma16(const void* gsrc, bf16_t* lds_dst) {
  __builtin_amdgcn_global_load_lds(gsrc, (__attribute__((address_space(3))) void*)lds_dst, 16, 0, 0);
}

// A T (of 4 or 16 bytes) in LDS, read as __bf16 like the operand fragments.  Before a read that
// may alias the destination of a direct global->LDS load still in flight the compiler waits for
// all of them, which would undo the counted waits; destinations are bf16_t, and it holds __bf16
// apart from that (and from int and float).  By the language this is undefined, and it is right
// only because every such read stands behind the asm wait and barrier that make its data
// visible, whose memory clobbers the compiler keeps in order.
template <class T>
__device__ __forceinline__ T lds_as_bf16(const void* p) {
  typedef __bf16 raw_t __attribute__((ext_vector_type(sizeof(T) / 2)));
  return __builtin_bit_cast(T, *reinterpret_cast<const raw_t*>(p));
}

template <int BM_, int BN_, int WM_, int WN_, int ST_>
struct GemmTile {
  static constexpr int BM = BM_, BN = BN_, WM = WM_, WN = WN_, ST = ST_;
  static constexpr int NW = WM * WN, THREADS = 64 * NW;  // wavefronts, threads per block
  static constexpr int TM = BM / WM, TN = BN / WN;  // wavefront tile
  static constexpr int FM = TM / 16, FN = TN / 16;  // 16 x 16 fragments per wavefront
  static constexpr int ROWS = BM + BN;              // LDS rows per stage
  static constexpr int LOADS = ROWS / (8 * NW);     // 1 KB loads per wavefront per stage
  static constexpr int STAGE = ROWS * 64;           // bf16 elements per stage
  static constexpr size_t LDS_BYTES = (size_t)ST * STAGE * 2;
  static_assert(NW == 4 || NW == 8, "4 or 8 wavefronts");
  static_assert(BM % 32 == 0 && BN % 32 == 0, "whole 32-row groups of each operand");
  static_assert(TM % 16 == 0 && TN % 16 == 0 && BM % 16 == 0, "fragment multiples");
  static_assert(ROWS % (8 * NW) == 0, "whole loads");
  static_assert(ST >= 2 && (ST - 2) * LOADS < 64, "vmcnt range");
};

// One block tile.  A: [M][K] rows (rows >= M are read from row M-1 and must be ignored by the
// caller), W: [*][K] rows n0 .. n0+BN-1; K a multiple of 64, M >= 1.  `lds` holds
// GemmTile::LDS_BYTES.  On return every wavefront has finished reading LDS only after the
// caller's next barrier.
//
// A stage is multiplied in two 32-wide slices, and the fragments of the next slice are read
// from LDS right after the first product of the current one, also over the stage boundary:
// the wait and barrier that make stage kt + 1 visible come before the last products of stage
// kt.  (After a direct global->LDS load the compiler waits for every LDS read before the first
// product that needs one, so reads issued before the products would not overlap with them.)
template <class TL>
__device__ __forceinline__ void gemm_core(const bf16_t* __restrict__ A, int M, int m0,
                                          const bf16_t* __restrict__ W, int n0, int K, bf16_t* lds,
                                          f32x4_t (&acc)[TL::FM][TL::FN]) {
  const int t = threadIdx.x, lane = t & 63, wv = t >> 6;
  const int wm = wv / TL::WN, wn = wv % TL::WN;
  const int l16 = lane & 15, kg = lane >> 4;

  static_for<TL::FM>([&](auto i) {
    static_for<TL::FN>([&](auto j) { acc[i][j] = f32x4_t{0.f, 0.f, 0.f, 0.f}; });
  });

  // global source of each of this lane's loads (fixed over K; advanced by 64 per stage)
  const bf16_t* src[TL::LOADS];
  static_for<TL::LOADS>([&](auto c) {
    const int row = (wv + TL::NW * c) * 8 + (lane >> 3);
    const int chunk = (lane & 7) ^ lds_swz(row);
    const bf16_t* base;
    if (row < TL::BM)
      base = A + (size_t)min(m0 + row, M - 1) * K;
    else
      base = W + (size_t)(n0 + row - TL::BM) * K;
    src[c] = base + chunk * 8;
  });
  auto issue = [&](int kt, int buf) {
    bf16_t* dst = lds + buf * TL::STAGE;
    static_for<TL::LOADS>([&](auto c) { dma16(src[c] + kt * 64, dst + (wv + TL::NW * c) * 512); });
  };
  bf16x8_t af[2][TL::FM], wf[2][TL::FN];
  auto read = [&](int kt, auto kk) {  // the fragments of slice kk of stage kt
    const bf16_t* sb = lds + (kt % TL::ST) * TL::STAGE;
    static_for<TL::FM>([&](auto i) {
      const int r = wm * TL::TM + 16 * i + l16;
      af[kk][i] = *reinterpret_cast<const bf16x8_t*>(sb + r * 64 + ((4 * kk + kg) ^ lds_swz(r)) * 8);
    });
    static_for<TL::FN>([&](auto j) {
      const int r = TL::BM + wn * TL::TN + 16 * j + l16;
      wf[kk][j] = *reinterpret_cast<const bf16x8_t*>(sb + r * 64 + ((4 * kk + kg) ^ lds_swz(r)) * 8);
    });
  };
  // the products of slice kk; `between` runs after the first of them
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
    // the first product's operands stay allocated: nothing written in `between` may share
    // their registers while it is in flight
    asm volatile("" ::"v"(wf[kk][0]), "v"(af[kk][0]));
  };
  using I0 = std::integral_constant<int, 0>;
  using I1 = std::integral_constant<int, 1>;
  const int nk = K / 64;
  // stage kt landed (the later stages already queued may be outstanding) and, behind the
  // barrier, stage kt - 1 read by every wavefront
  auto visible = [&](int kt) {
    const int ahead = min(TL::ST - 2, nk - 1 - kt);
    static_for<TL::ST - 1>([&](auto a) {
      if (a == ahead) vm_wait_barrier<a * TL::LOADS>();
    });
    lds_reads_done();
  };
  auto enter = [&](int kt) {
    read(kt, I0{});
    mfma_fence_begin();
    if (kt + TL::ST - 1 < nk) issue(kt + TL::ST - 1, (kt + TL::ST - 1) % TL::ST);
  };
  auto stage = [&](int kt) {
    multiply(I0{}, [&] { read(kt, I1{}); });
    const bool more = kt + 1 < nk;
    if (more) visible(kt + 1);
    multiply(I1{}, [&] {
      if (more) enter(kt + 1);
    });
  };
  static_for<TL::ST - 1>([&](auto s) {
    if (s < nk) issue(s, s);
  });
  visible(0);
  enter(0);
  for (int kt = 0; kt < nk; ++kt) stage(kt);
}

// A lane's results of fragments 2p and 2p + 1 become 8 consecutive channels of its token (16-byte
// stores along a row) if W's fragment f takes row lane8_row(f, r) for lane row r, instead of
// 16 f + r.  These rows are 4 and 4 apart, so they are swizzled by lane8_swz, not by row & 7.
__device__ __forceinline__ int lane8_row(int f, int r) { return 32 * (f >> 1) + 8 * (r >> 2) + 4 * (f & 1) + (r & 3); }
__device__ __forceinline__ int lane8_swz(int row) { return (row & 3) | ((row >> 1) & 4); }

// Tile order: consecutive workgroups are dispatched round-robin over the 8 XCDs (each with
// its own L2).  Workgroup b runs on XCD b % 8; it is given row tile (k / nt) * 8 + b % 8 and
// column tile k % nt (k = b / 8), so each XCD owns every 8th row tile and computes all nt
// column tiles of a row tile back to back (its A rows are read into that XCD's L2 once), and
// the row tiles that exist for a data-dependent row count spread evenly over the XCDs.
// Grid: 8 * ceil(mt / 8) * nt workgroups; tiles with row >= mt exit.
__device__ __forceinline__ void xcd_tile(int b, int nt, int& rt, int& ct) {
  const int k = b >> 3;
  ct = k % nt;
  rt = (k / nt) * 8 + (b & 7);
}

__host__ __device__ constexpr int xcd_grid(int mt, int nt) { return 8 * ((mt + 7) / 8) * nt; }

}  // namespace dr
