// Numeric phases on gfx950 (MI355X): assembly of the shifted matrices, the
// supernodal LDL^T factorization, selected inversion, pole sums and inertia.
//
// Paper, Sec. II.A-II.B: for A = H - z S (complex symmetric) compute
// A = L D L^T (L unit lower, D diagonal) and then the entries of A^{-1} on
// the pattern of L; the factorization traverses the elimination tree from the
// leaves to the root and selected inversion from the root to the leaves, both
// as dense matrix products on supernodes.  Sec. II.C: for real shifts the
// number of negative d_k is the inertia count.
//
// Execution model: every launch covers all shifts of a batch (grid.y) and all
// tiles of one panel (a <= 64-column slice of a supernode).  The factorization
// issues supernodes leaves first (by height in the supernodal tree; within a
// height those whose scatters share no target together, then column order),
// panels left to right; SelInv runs root to leaves.  Within
// a launch, workgroups own disjoint outputs, so there are no atomics on matrix
// data, and every entry receives its updates in one fixed order, so results
// do not depend on scheduling or on the number of subtree streams.
//
// Per panel p of supernode J (row list E_J, own columns first), with
// B = rows of E_J below the panel's diagonal block:
//   factor:  k_diag   dense LDL^T of the wp x wp diagonal block in LDS; stores
//                     D on the diagonal and L_pp^{-1} below it
//            k_trsm   L_Bp = A_Bp L_pp^{-T} D_p^{-1}
//            k_update A_BB -= L_Bp D_p L_Bp^T, scattered through the maps into
//                     the later columns of J and into ancestor supernodes
//   selinv:  k_lhat   W = L_Bp L_pp^{-1}                       (workspace)
//            k_selinv_off   Z_Bp = -Z_BB W   (Z_BB gathered, symmetric)
//            k_selinv_diag_* Z_pp = L_pp^{-T} D_p^{-1} L_pp^{-1} - W^T Z_Bp
//            k_selinv_small  all of these for a panel with few rows below it
// The products run on FP64 MFMA (v_mfma_f64_16x16x4f64): a complex product is
// four real MFMAs on elements loaded straight into LDS.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <type_traits>
#include <cstdint>
#include <cstdio>
#include <new>
#include <vector>

#include "pxs_internal.h"
#include "numeric.h"

namespace pxs {

typedef double dbl4 __attribute__((ext_vector_type(4)));

constexpr int NT = 256;   // threads per workgroup (4 wave64)
constexpr int TM = 64;    // tile rows (m) and columns (n)

struct cplx {
  double re, im;
};

__device__ __forceinline__ cplx cmul(cplx a, cplx b) {
  return {a.re * b.re - a.im * b.im, a.re * b.im + a.im * b.re};
}
__device__ __forceinline__ cplx cinv(cplx a) {
  double d = a.re * a.re + a.im * a.im;
  return {a.re / d, -a.im / d};
}

template <bool CPLX>
__device__ __forceinline__ cplx ld_elem(const double* base, int64_t e) {
  if (CPLX) {
    const double2 v = *reinterpret_cast<const double2*>(base + 2 * e);
    return {v.x, v.y};
  }
  return {base[e], 0.0};
}
template <bool CPLX>
__device__ __forceinline__ void st_elem(double* base, int64_t e, cplx v) {
  if (CPLX) {
    *reinterpret_cast<double2*>(base + 2 * e) = make_double2(v.re, v.im);
  } else {
    base[e] = v.re;
  }
}

// What operand lanes outside their matrix read through a pointer of their own.
__device__ __align__(16) double kZeroElem[2] = {0.0, 0.0};   // never written

// --------------------------------------------------------------------------
// MFMA tiles: a 256-thread workgroup accumulates a 64 x NTILE tile
// P[m][n] = sum_k A[m][k] B[k][n] (NTILE = 64, 32 or 16).  The 4 waves are laid
// out WM x WN over the tile, each owning BM x BN blocks of 16 x 16.
// v_mfma_f64_16x16x4f64 lane layout (lane l, 0..63):
//   A operand: A[l % 16][l / 16];  B operand: B[l / 16][l % 16];
//   result register r: D[l / 16 + 4 r][l % 16].
// A complex block product is four real MFMAs: re += ar br - ai bi,
// im += ar bi + ai br.  The last argument of the f64 MFMA builtin holds the
// operand negation bits (bit 0 negates A), so -ai costs no instruction.
// --------------------------------------------------------------------------
// TALL (complex products of panels of at most 48 columns): 64 and 32 columns
// with the waves along n first, so that a panel's dead 16-row blocks are left
// out of every wave alike; the row blocks alternate between the two wave rows
// of a 32-column tile.
template <int NTILE, bool TALL = false>
struct Geo {
  static constexpr int WN = TALL ? (NTILE + 15) / 16 : NTILE < 32 ? 1 : NTILE / 32;   // waves along n
  static constexpr int WM = 4 / WN;            // waves along m
  static constexpr int BM = TALL ? (NTILE == 64 ? 3 : NTILE == 32 ? 2 : 1) : 64 / WM / 16;   // 16-blocks per wave along m
  static constexpr int BN = TALL || NTILE < 32 ? 1 : 2;    // 16-blocks per wave along n
};

template <bool CPLX, int NTILE, bool TALL = false>
struct Acc {
  static constexpr int BM = Geo<NTILE, TALL>::BM, BN = Geo<NTILE, TALL>::BN;
  dbl4 re[BM][BN];
  dbl4 im[CPLX ? BM : 1][CPLX ? BN : 1];
  __device__ void zero() {
#pragma unroll
    for (int a = 0; a < BM; ++a)
#pragma unroll
      for (int b = 0; b < BN; ++b) {
        re[a][b] = dbl4{0.0, 0.0, 0.0, 0.0};
        if (CPLX) im[a][b] = dbl4{0.0, 0.0, 0.0, 0.0};
      }
  }
};

// Row of the 16-row block a (column of the 16-column block b) of wave w:
// blocks in order, or, with bit 0 (bit 1) of SWZ on a 64 x 64 tile, the
// first wave row (column) taking blocks {0, 3} and the second {1, 2}, so that
// both skip equally many blocks of a triangle (products with a triangular
// operand or a symmetric result).
template <int NTILE, int SWZ, bool TALL = false>
__device__ __forceinline__ int block_row(int w, int a) {
  using G = Geo<NTILE, TALL>;
  if constexpr (TALL) {
    return 16 * (a * G::WM + w / G::WN);
  } else if constexpr ((SWZ & 1) != 0) {
    static_assert(G::BM == 2 && G::WM == 2, "block swizzle needs 2 x 2 waves of 2 blocks");
    const int wr = w / G::WN;
    return 16 * (a == 0 ? wr : 3 - wr);
  } else {
    return (w / G::WN) * (G::BM * 16) + a * 16;
  }
}
template <int NTILE, int SWZ, bool TALL = false>
__device__ __forceinline__ int block_col(int w, int b) {
  using G = Geo<NTILE, TALL>;
  if constexpr ((SWZ & 2) != 0) {
    static_assert(G::BN == 2 && G::WN == 2, "block swizzle needs 2 x 2 waves of 2 blocks");
    const int wc = w % G::WN;
    return 16 * (b == 0 ? wc : 3 - wc);
  } else {
    return (w % G::WN) * (G::BN * 16) + b * 16;
  }
}

// Visits every accumulator element as (m, n, value).
template <bool CPLX, int NTILE, int SWZ = 0, bool TALL = false, class F>
__device__ __forceinline__ void acc_foreach(const Acc<CPLX, NTILE, TALL>& acc, F f) {
  using G = Geo<NTILE, TALL>;
  const int lane = threadIdx.x & 63;
  const int w = threadIdx.x >> 6;
#pragma unroll
  for (int a = 0; a < G::BM; ++a)
#pragma unroll
    for (int b = 0; b < G::BN; ++b)
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        const int m = block_row<NTILE, SWZ, TALL>(w, a) + (lane >> 4) + 4 * r;
        const int n = block_col<NTILE, SWZ, TALL>(w, b) + (lane & 15);
        cplx v{acc.re[a][b][r], CPLX ? acc.im[a][b][r] : 0.0};
        f(m, n, v);
      }
}

// The idx-th accumulator element of the calling thread (the order in which
// acc_foreach visits them) and its tile coordinates.
template <int NTILE, bool TALL = false>
constexpr int acc_elems() { return Geo<NTILE, TALL>::BM * Geo<NTILE, TALL>::BN * 4; }

template <bool CPLX, int NTILE, bool TALL>
__device__ __forceinline__ void acc_at(const Acc<CPLX, NTILE, TALL>& acc, int idx, int& m, int& n, cplx& v) {
  using G = Geo<NTILE, TALL>;
  const int lane = threadIdx.x & 63;
  const int w = threadIdx.x >> 6;
  const int r = idx & 3, b = (idx >> 2) % G::BN, a = (idx >> 2) / G::BN;
  m = block_row<NTILE, 0, TALL>(w, a) + (lane >> 4) + 4 * r;
  n = block_col<NTILE, 0, TALL>(w, b) + (lane & 15);
  v = cplx{acc.re[a][b][r], CPLX ? acc.im[a][b][r] : 0.0};
}

// target[e] -= P for every accumulator element, in three passes so that a
// thread's memory operations overlap instead of running one element at a
// time: all target positions (addr(m, n, e) may read index maps; false
// skips the element, whose e must still be an in-bounds position of
// target), then all old values, then all stores.  Every target
// belongs to one element of one workgroup, so reordering the stores changes
// no result.
template <bool CPLX, int NTILE, bool TALL, class AF>
__device__ __forceinline__ void acc_sub_into(const Acc<CPLX, NTILE, TALL>& acc, double* target, AF addr) {
  constexpr int NE = acc_elems<NTILE, TALL>();
  // at most 8 elements at a time, so positions and old values fit
  // beside the accumulators in the 128 registers of four waves per SIMD
  constexpr int NH = NE > 8 ? (NE % 8 ? 4 : 8) : NE;
#pragma unroll
  for (int h = 0; h < NE; h += NH) {
    int64_t e[NH];
    bool ok[NH];
#pragma unroll
    for (int i = 0; i < NH; ++i) {
      int m, n;
      cplx v;
      acc_at(acc, h + i, m, n, v);
      ok[i] = addr(m, n, e[i]);
    }
    // addr returns an in-bounds position also for skipped elements, so the
    // old values load without branches
    cplx o[NH];
#pragma unroll
    for (int i = 0; i < NH; ++i) o[i] = ld_elem<CPLX>(target, e[i]);
#pragma unroll
    for (int i = 0; i < NH; ++i) {
      int m, n;
      cplx v;
      acc_at(acc, h + i, m, n, v);
      if (ok[i]) st_elem<CPLX>(target, e[i], cplx{o[i].re - v.re, o[i].im - v.im});
    }
  }
}

// XCD-aware tile order.  Workgroups are dispatched round-robin over the 8
// XCDs in linear-id order; this bijection gives each XCD a contiguous range
// of logical ids, so the tiles of one shift (which share the A operand) run
// on the same XCD and share its L2.  Returns the logical (x, y) of the
// caller in a grid of nx x ny.
constexpr int NXCD = 8;
__device__ __forceinline__ int xcd_logical(int b, int total) {
  const int xcd = b % NXCD, idx = b / NXCD;
  const int q = total / NXCD, r = total % NXCD;
  return (xcd < r) ? xcd * (q + 1) + idx : r * (q + 1) + (xcd - r) * q + idx;
}
__device__ __forceinline__ void xcd_remap(int& x, int& y) {
  const int nx = gridDim.x, ny = gridDim.y;
  const int logical = xcd_logical(blockIdx.x + nx * blockIdx.y, nx * ny);
  x = logical % nx;
  y = logical / nx;
}

// Which 16 x 16 blocks of a complex tile take part in the 16 columns c of the
// product: all, those of a triangular A operand that meet the columns in its
// nonzero triangle (LOWER: A[m][k] = 0 for k > m, else for k < m), or those on
// or above the diagonal of a symmetric result (cb: block column of the whole
// result).
struct AllBlocks {
  static constexpr bool kAll = true;
  static constexpr int kSwz = 0;
  __device__ bool operator()(int, int, int) const { return true; }
};
template <bool LOWER>
struct TriBlocks {
  static constexpr bool kAll = false;
  static constexpr int kSwz = 1;   // on 64 x 64 tiles the wave rows take blocks {0, 3} and {1, 2}
  __device__ bool operator()(int rb, int, int c) const { return LOWER ? c <= rb : c >= rb; }
};
struct UpperBlocks {
  static constexpr bool kAll = false;
  static constexpr int kSwz = 3;   // rows and columns
  int cb0;                         // the tile's first block column
  __device__ bool operator()(int rb, int cb, int) const { return cb0 + cb >= rb; }
};

// --------------------------------------------------------------------------
// Tile engine: the operands go straight from global memory into LDS.
//
// What bounds these products is the issue of everything that is not an MFMA:
// with the operands staged through registers (loads with 64-bit per-lane
// addresses, LDS stores, split re/im reads) the engine ran at 62 TFLOP/s on
// 64 x 4096 x 4096 x 32 shifts and the register staging held it to two
// workgroups per CU.  Here a stage of KD = 8 columns is moved by
// buffer_load_dwordx4 ... lds: the base is scalar and advances with k, the
// lane offset is constant, lanes outside the operand get an offset past the
// descriptor's range and read zeros.  An element stays one 16-byte (re, im)
// pair, read with one ds_read_b128.  No staging registers: four workgroups
// (16 waves) fit on a CU, which cover each other's barriers, so two stages
// are enough.  Measured on k_selinv_off's shape: 62.2 -> 69.0 TFLOP/s at
// 4096 rows x 32 shifts (74 with the loads taken out), 48.4 -> 54.4 at 884 x 60.
//
// Narrow tiles: a launch of T tiles of 64 columns takes ceil(T / 256) rounds
// over the CUs, so a few hundred tiles leave the chip partly idle (840 tiles:
// 3.3 rounds of work in 4).  32- and 16-column tiles cut the rounds finer:
// 884 rows x 60 shifts 54.4 -> 59.9 TFLOP/s with 32 columns, 452 x 40 33.3 ->
// 43.4 (32) and 47.8 (16), 130 x 40 13.7 -> 22.6 (32); on full launches they
// are slower (4096 x 32: 68.1 and 60.7), see pick_tile.
//
// LDS layouts of a stage of an operand with ROWS rows (slot = 16 bytes, a
// wave fills 64 slots in lane order per load):
//   rows fast  slot = k ROWS + row            (memory contiguous along rows)
//   k fast     slot = row 8 + (k ^ ((row / 2) % 8))   (contiguous along k)
// The 16 lanes of an MFMA operand row read 16 consecutive slots, or 16 slots
// that differ modulo 16 (the exclusive or sees to that): no bank conflicts.
//
// Real products (inertia) take stages of 16 columns, always rows fast.  Their
// 8-byte elements start at any multiple of 8, so they move as two 4-byte words
// by a lane pair each; on 64- and 32-row operands odd columns swap their 16-row
// halves, which keeps two columns read together on different banks.  An inertia
// of a sheet of N=7956 with 16 shifts took 12.15 ms with real tiles staged
// through registers (64 or 128 rows, 1 to 3 workgroups per CU), 11.5 so.
// --------------------------------------------------------------------------
typedef double dbl2 __attribute__((ext_vector_type(2)));
typedef __attribute__((address_space(3))) void* lds_ptr;
typedef const __attribute__((address_space(1))) void* glb_ptr;

constexpr int KD = 8, KR = 16;               // columns per stage, complex and real
constexpr unsigned LANE_OUT = 0x80000000u;   // lane offset past every descriptor's range: reads zeros
__device__ __align__(16) double kUnitElem[2] = {1.0, 0.0};   // never written

template <bool CPLX>
using elem_t = std::conditional_t<CPLX, dbl2, double>;
template <bool CPLX>
constexpr int kDepth = CPLX ? KD : KR;

template <bool CPLX, int NTILE, bool SCALE>
struct TileStage {
  static constexpr int D = kDepth<CPLX>;
  elem_t<CPLX> a[2][D * 64];
  elem_t<CPLX> b[2][D * NTILE];
  elem_t<CPLX> d[SCALE ? 2 : 1][SCALE ? D : 1];
};

// The wave's index and a pointer the compiler may not know to be uniform.
__device__ __forceinline__ int wave_id() { return __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6)); }
__device__ __forceinline__ const double* uniform(const double* p) {
  const uint64_t v = (uint64_t)p;
  const uint32_t lo = (uint32_t)__builtin_amdgcn_readfirstlane((int)(uint32_t)v);
  const uint32_t hi = (uint32_t)__builtin_amdgcn_readfirstlane((int)(uint32_t)(v >> 32));
  return (const double*)(((uint64_t)hi << 32) | lo);
}

// 16 bytes per lane into LDS at lds + 16 lane: from base + off (off < 2^31
// or LANE_OUT), or from a pointer per lane.
__device__ __forceinline__ void load_lds(const double* base, unsigned off, dbl2* lds) {
  const __amdgpu_buffer_rsrc_t r = __builtin_amdgcn_make_buffer_rsrc((void*)base, 0, LANE_OUT, 0x00020000);
  __builtin_amdgcn_raw_ptr_buffer_load_lds(r, (lds_ptr)lds, 16, off, 0, 0, 0);
}
__device__ __forceinline__ void load_lds_ptr(const double* p, dbl2* lds) {
  __builtin_amdgcn_global_load_lds((glb_ptr)p, (lds_ptr)lds, 16, 0, 0);
}
// 4 bytes per lane into LDS at lds + 4 lane
__device__ __forceinline__ void load_lds4(const double* base, unsigned off, double* lds) {
  const __amdgpu_buffer_rsrc_t r = __builtin_amdgcn_make_buffer_rsrc((void*)base, 0, LANE_OUT, 0x00020000);
  __builtin_amdgcn_raw_ptr_buffer_load_lds(r, (lds_ptr)lds, 4, off, 0, 0, 0);
}
__device__ __forceinline__ void load_lds4_ptr(const double* p, int half, double* lds) {
  __builtin_amdgcn_global_load_lds((glb_ptr)((const char*)p + 4 * half), (lds_ptr)lds, 4, 0, 0);
}

// Operand slot of lane `lane` in the wave load q of a stage: (row, k).
template <int ROWS>
__device__ __forceinline__ void slot_rows(int q, int lane, int& m, int& k) {
  m = lane % ROWS;
  k = q * (64 / ROWS) + lane / ROWS;
}
__device__ __forceinline__ void slot_k(int q, int lane, int& m, int& k) {
  m = q * 8 + (lane >> 3);
  k = (lane & 7) ^ ((m >> 1) & 7);
}

// The same of a real operand: 32 elements of a wave load, two lanes each.
template <int ROWS>
__device__ __forceinline__ int real_slot(int k, int row) {
  return k * ROWS + (ROWS >= 32 ? row ^ ((k & 1) << 4) : row);
}
template <int ROWS>
__device__ __forceinline__ void slot_real(int q, int lane, int& m, int& k) {
  const int e = q * 32 + (lane >> 1);
  k = e / ROWS;
  m = ROWS >= 32 ? (e % ROWS) ^ ((k & 1) << 4) : e % ROWS;
}

// Operands of gemm_lds.  issue(k0, lds) starts the loads of columns
// [k0, k0 + D) (k relative to the product's first column; columns from K on
// and rows from nrows on read zeros); fast(k0) is the layout it uses (true: k
// fast).  Wave w makes the loads q = w, w + 4, ...
template <bool CPLX, int ROWS>
struct LoadCount {
  static constexpr int N = CPLX ? KD * ROWS / 64 : KR * ROWS / 32, J = (N + 3) / 4;
};

// Element (row, k) at base + k ld + row.
template <bool CPLX, int ROWS>
struct ColsOp : LoadCount<CPLX, ROWS> {
  using LoadCount<CPLX, ROWS>::N;
  using LoadCount<CPLX, ROWS>::J;
  const double* base;
  int64_t ld;
  int K, w;
  unsigned v[J];
  int kk[J];
  __device__ __forceinline__ ColsOp(const double* b, int ld_, int nrows, int K_)
      : base(uniform(b)), ld(ld_), K(K_), w(wave_id()) {
    const int lane = threadIdx.x & 63;
#pragma unroll
    for (int j = 0; j < J; ++j) {
      int m;
      if (CPLX) slot_rows<ROWS>(w + 4 * j, lane, m, kk[j]);
      else slot_real<ROWS>(w + 4 * j, lane, m, kk[j]);
      const unsigned e = (unsigned)(kk[j] * ld_ + m);
      v[j] = m >= nrows ? LANE_OUT : CPLX ? e * 16u : e * 8u + 4u * (lane & 1);
    }
  }
  __device__ __forceinline__ void issue(int k0, elem_t<CPLX>* lds) const {
#pragma unroll
    for (int j = 0; j < J; ++j) {
      if (N < 4 && w >= N) continue;
      const unsigned o = k0 + kk[j] < K ? v[j] : LANE_OUT;
      if constexpr (CPLX) load_lds(base + 2 * (ld * k0), o, lds + (w + 4 * j) * 64);
      else load_lds4(base + ld * k0, o, lds + (w + 4 * j) * 32);
    }
  }
  __device__ __forceinline__ static constexpr bool fast(int) { return false; }
};

// Element (row, k) at base + row ld + k.
template <int ROWS>
struct RowsOp : LoadCount<true, ROWS> {
  using LoadCount<true, ROWS>::N;
  using LoadCount<true, ROWS>::J;
  const double* base;
  int K, w;
  int rows16;   // rows rounded up to blocks of 16: the slots behind them are never read
  unsigned v[J];
  int kk[J];
  __device__ __forceinline__ RowsOp(const double* b, int ld, int nrows, int K_)
      : base(uniform(b)), K(K_), w(wave_id()), rows16((nrows + 15) & ~15) {
#pragma unroll
    for (int j = 0; j < J; ++j) {
      int m;
      slot_k(w + 4 * j, threadIdx.x & 63, m, kk[j]);
      v[j] = m < nrows ? (unsigned)(m * ld + kk[j]) * 16u : LANE_OUT;
    }
  }
  __device__ __forceinline__ void issue(int k0, dbl2* lds) const {
#pragma unroll
    for (int j = 0; j < J; ++j) {
      if ((N < 4 && w >= N) || (w + 4 * j) * 8 >= rows16) continue;
      load_lds(base + 2 * (int64_t)k0, k0 + kk[j] < K ? v[j] : LANE_OUT, lds + (w + 4 * j) * 64);
    }
  }
  __device__ __forceinline__ static constexpr bool fast(int) { return true; }
};

// The unit lower triangular n x n block T (n <= 64; strict part stored, T(r,
// q) at base + q ld + r) as the A operand: A[m][k] = T[m][k], or T[k][m] when
// TRANS.
template <bool CPLX, bool TRANS>
struct TriOp : LoadCount<CPLX, 64> {
  static_assert(CPLX || !TRANS, "real operands are rows fast");
  using LoadCount<CPLX, 64>::J;
  const double* base;
  int ld, n, w;
  __device__ __forceinline__ TriOp(const double* b, int ld_, int n_) : base(b), ld(ld_), n(n_), w(wave_id()) {}
  __device__ __forceinline__ void issue(int k0, elem_t<CPLX>* lds) const {
    const int lane = threadIdx.x & 63;
#pragma unroll
    for (int j = 0; j < J; ++j) {
      int m, k;
      if (!CPLX) slot_real<64>(w + 4 * j, lane, m, k);
      else if (TRANS) slot_k(w + 4 * j, lane, m, k);
      else slot_rows<64>(w + 4 * j, lane, m, k);
      k += k0;
      const int r = TRANS ? k : m, q = TRANS ? m : k;
      const double* p = r == q ? kUnitElem : kZeroElem;
      if (r > q) p = base + (CPLX ? 2 : 1) * ((int64_t)q * ld + r);
      if (max(r, q) >= n) p = kZeroElem;
      if constexpr (CPLX) load_lds_ptr(p, lds + (w + 4 * j) * 64);
      else load_lds4_ptr(p, lane & 1, lds + (w + 4 * j) * 32);
    }
  }
  __device__ __forceinline__ static constexpr bool fast(int) { return TRANS; }
};

// Rows i0.. of the selected inverse Z_BB of a panel: element (row i, column
// k) sits at (row max, column min) of the lower triangle, which is stored in
// two parts: own (columns of the supernode itself: the first gw positions,
// leading dimension ld) and g (the rows below it, dense, leading dimension c,
// position gw first).  Both pointers are those of position (0, 0), for g the
// virtual one.  Chunks strictly below the block diagonal are read rows fast,
// strictly above it k fast (transposed), in both cases through one
// descriptor when the chunk's columns (or rows) lie in one part; a chunk that
// crosses the parts takes a pointer per lane.
// HERM: entries below the diagonal (row >= column of Z) come from one pair
// of arrays and those above it from another (utown / utg elements further);
// side 0 reads Z(i, k), side 1 Z(k, i).
template <int ROWS, bool HERM>
struct SymOp : LoadCount<true, ROWS> {
  using LoadCount<true, ROWS>::N;
  using LoadCount<true, ROWS>::J;
  const double *own, *g;
  int ld, c, gw, i0, nb, w, side;
  int64_t utown, utg;
  __device__ __forceinline__ SymOp(const double* own_, int ld_, const double* g_, int c_, int gw_, int i0_, int nb_,
                                   int side_ = 0, int64_t utown_ = 0, int64_t utg_ = 0)
      : own(uniform(own_)), g(uniform(g_)), ld(ld_), c(c_), gw(gw_), i0(i0_), nb(nb_), w(wave_id()), side(side_),
        utown(utown_), utg(utg_) {}
  __device__ __forceinline__ bool fast(int k0) const { return k0 + KD > i0; }
  __device__ __forceinline__ void issue(int k0, dbl2* lds) const {
    const bool low = !fast(k0), up = k0 >= i0 + ROWS;
    const int lo0 = min(k0, i0);                                     // smallest and largest column read
    const int lo1 = min(nb - 1, low ? k0 + KD - 1 : up ? i0 + ROWS - 1 : min(k0 + KD - 1, i0 + ROWS - 1));
    const bool from_own = lo1 < gw, from_g = lo0 >= gw;
    const int lane = threadIdx.x & 63;
    if ((from_own || from_g) && (low || up || !HERM)) {
      const int lz = from_own ? ld : c;
      const double* z = from_own ? own : g;
      if (HERM && low == (side == 1)) z += 2 * (from_own ? utown : utg);
      z += 2 * ((int64_t)lo0 * lz + (low ? i0 : up ? k0 : 0));
#pragma unroll
      for (int j = 0; j < J; ++j) {
        if (N < 4 && w >= N) continue;
        int n, k;
        unsigned v;
        if (low) {
          slot_rows<ROWS>(w + 4 * j, lane, n, k);
          v = __umul24(k, lz) + n;
        } else {
          slot_k(w + 4 * j, lane, n, k);
          if (up) {
            v = __umul24(n, lz) + k;
          } else {
            const int i = i0 + n, q = k0 + k;
            v = __umul24(min(i, q) - lo0, lz) + max(i, q);
          }
        }
        load_lds(z, i0 + n < nb && k0 + k < nb ? v * 16u : LANE_OUT, lds + (w + 4 * j) * 64);
      }
    } else {
#pragma unroll
      for (int j = 0; j < J; ++j) {
        if (N < 4 && w >= N) continue;
        int n, k;
        if (low) slot_rows<ROWS>(w + 4 * j, lane, n, k);
        else slot_k(w + 4 * j, lane, n, k);
        const int i = i0 + n, q = k0 + k;
        const int lo = min(i, q), hi = max(i, q);
        const bool og = lo >= gw;
        int64_t e = (int64_t)lo * (og ? c : ld) + hi;
        if (HERM && !(side ? q >= i : i >= q)) e += og ? utg : utown;
        const double* p = (og ? g : own) + 2 * e;
        load_lds_ptr(hi < nb ? p : kZeroElem, lds + (w + 4 * j) * 64);
      }
    }
  }
};

// Per-column factors of the A operand: d_k at base + k stride (elements).
template <bool CPLX>
struct DiagOp {
  const double* base;
  int64_t stride;
  int K;
  __device__ __forceinline__ DiagOp(const double* b, int64_t st, int K_) : base(uniform(b)), stride(st), K(K_) {}
  __device__ __forceinline__ void issue(int k0, elem_t<CPLX>* lds) const {
    if (threadIdx.x >= (CPLX ? KD : 2 * KR)) return;
    const int k = CPLX ? threadIdx.x : threadIdx.x >> 1;
    const unsigned e = (unsigned)(k * stride);
    const unsigned o = k0 + k >= K ? LANE_OUT : CPLX ? e * 16u : e * 8u + 4u * (threadIdx.x & 1);
    if constexpr (CPLX) load_lds(base + 2 * (stride * k0), o, lds);
    else load_lds4(base + stride * k0, o, lds);
  }
};
struct NoDiag {
  __device__ __forceinline__ void issue(int, dbl2*) const {}
  __device__ __forceinline__ void issue(int, double*) const {}
};

// One stage on the matrix cores.  MASKED: only the block pairs (a, b) with bit
// BN a + b of mask set (uniform over the wave; a branch per pair, one copy of
// the code: a copy per mask spilled registers at four waves per SIMD).
template <int NTILE, bool TALL, bool SCALE, bool MASKED, int SWZ>
__device__ __forceinline__ void mfma_stage(Acc<true, NTILE, TALL>& acc, const dbl2* as, bool afast, const dbl2* bs,
                                           bool bfast, const dbl2* ds, int mask) {
  using G = Geo<NTILE, TALL>;
  const int lane = threadIdx.x & 63;
  const int w = threadIdx.x >> 6;
  const int li = lane & 15, lk = lane >> 4;
#pragma unroll
  for (int ks = 0; ks < KD / 4; ++ks) {
    const int k = ks * 4 + lk;
    dbl2 av[G::BM], bv[G::BN];
#pragma unroll
    for (int t = 0; t < G::BM; ++t) {
      const int m = block_row<NTILE, SWZ, TALL>(w, t) + li;
      av[t] = as[afast ? m * 8 + (k ^ (li >> 1)) : k * 64 + m];
    }
#pragma unroll
    for (int t = 0; t < G::BN; ++t) {
      const int n = block_col<NTILE, SWZ, TALL>(w, t) + li;
      bv[t] = bs[bfast ? n * 8 + (k ^ (li >> 1)) : k * NTILE + n];
    }
    if constexpr (SCALE) {
      const dbl2 d = ds[k];
#pragma unroll
      for (int t = 0; t < G::BM; ++t) {
        const cplx v = cmul(cplx{d.x, d.y}, cplx{av[t].x, av[t].y});
        av[t] = dbl2{v.re, v.im};
      }
    }
    auto first = [&](int a, int b) {
      acc.re[a][b] = __builtin_amdgcn_mfma_f64_16x16x4f64(av[a].x, bv[b].x, acc.re[a][b], 0, 0, 0);
      acc.im[a][b] = __builtin_amdgcn_mfma_f64_16x16x4f64(av[a].x, bv[b].y, acc.im[a][b], 0, 0, 0);
    };
    auto second = [&](int a, int b) {
      acc.re[a][b] = __builtin_amdgcn_mfma_f64_16x16x4f64(av[a].y, bv[b].y, acc.re[a][b], 0, 0, 1);   // -ai bi
      acc.im[a][b] = __builtin_amdgcn_mfma_f64_16x16x4f64(av[a].y, bv[b].x, acc.im[a][b], 0, 0, 0);
    };
    if constexpr (MASKED) {
#pragma unroll
      for (int a = 0; a < G::BM; ++a)
#pragma unroll
        for (int b = 0; b < G::BN; ++b)
          if ((mask >> (G::BN * a + b)) & 1) {
            first(a, b);
            second(a, b);
          }
    } else {
#pragma unroll
      for (int a = 0; a < G::BM; ++a)
#pragma unroll
        for (int b = 0; b < G::BN; ++b) first(a, b);
#pragma unroll
      for (int a = 0; a < G::BM; ++a)
#pragma unroll
        for (int b = 0; b < G::BN; ++b) second(a, b);
    }
  }
}

template <int NTILE, bool TALL, bool SCALE, bool MASKED, int SWZ>
__device__ __forceinline__ void mfma_stage(Acc<false, NTILE, TALL>& acc, const double* as, bool, const double* bs, bool,
                                           const double* ds, int mask) {
  using G = Geo<NTILE, TALL>;
  const int lane = threadIdx.x & 63;
  const int w = threadIdx.x >> 6;
  const int li = lane & 15, lk = lane >> 4;
#pragma unroll
  for (int ks = 0; ks < KR / 4; ++ks) {
    const int k = ks * 4 + lk;
    double av[G::BM], bv[G::BN];
#pragma unroll
    for (int t = 0; t < G::BM; ++t) av[t] = as[real_slot<64>(k, block_row<NTILE, SWZ, TALL>(w, t) + li)];
#pragma unroll
    for (int t = 0; t < G::BN; ++t) bv[t] = bs[real_slot<NTILE>(k, block_col<NTILE, SWZ, TALL>(w, t) + li)];
    if constexpr (SCALE) {
      const double d = ds[k];
#pragma unroll
      for (int t = 0; t < G::BM; ++t) av[t] *= d;
    }
#pragma unroll
    for (int a = 0; a < G::BM; ++a)
#pragma unroll
      for (int b = 0; b < G::BN; ++b)
        if (!MASKED || ((mask >> (G::BN * a + b)) & 1))
          acc.re[a][b] = __builtin_amdgcn_mfma_f64_16x16x4f64(av[a], bv[b], acc.re[a][b], 0, 0, 0);
  }
}

// Waits for the caller's loads into LDS and its LDS reads, then for every
// wave of the workgroup.
__device__ __forceinline__ void stage_barrier() { asm volatile("s_waitcnt vmcnt(0) lgkmcnt(0)\n\ts_barrier" ::: "memory"); }

// P += A[:, k] B[k, :] over k in [0, K): two stages, one barrier per stage.
// A stage's loads start right after the barrier that ends the reads of its
// buffer and have the other stage's MFMAs (and three other workgroups') to
// land.  The result has mrows rows (64, or fewer: the blocks behind them are
// not multiplied).
template <class LV, bool CPLX, int NTILE, bool TALL, class OA, class OB, class OD>
__device__ __forceinline__ void gemm_lds(Acc<CPLX, NTILE, TALL>& acc,
                                         TileStage<CPLX, NTILE, !std::is_same<OD, NoDiag>::value>& s, int mrows, int K,
                                         const OA& oa, const OB& ob, const OD& od, LV lv) {
  constexpr bool SC = !std::is_same<OD, NoDiag>::value;
  constexpr int KD = kDepth<CPLX>;
  using G = Geo<NTILE, TALL>;
  constexpr int SWZ = NTILE == 64 && !TALL ? LV::kSwz : 0;
  constexpr bool MASKED = TALL || NTILE == 16 || !LV::kAll;
  if (K <= 0) return;
  const int nc = (K + KD - 1) / KD;
  const int w = wave_id();
  auto issue = [&](int c, int q) {
    oa.issue(c * KD, s.a[q]);
    ob.issue(c * KD, s.b[q]);
    od.issue(c * KD, s.d[SC ? q : 0]);
  };
  auto blocks = [&](int c) {   // the wave's live blocks in the 16 columns c
    int m = 0;
#pragma unroll
    for (int a = 0; a < G::BM; ++a)
#pragma unroll
      for (int b = 0; b < G::BN; ++b) {
        const int row = block_row<NTILE, SWZ, TALL>(w, a);
        if (row < mrows && lv(row / 16, block_col<NTILE, SWZ, TALL>(w, b) / 16, c)) m |= 1 << (G::BN * a + b);
      }
    return m;
  };
  issue(0, 0);
  int q = 0;
  int mask = LV::kAll && MASKED ? blocks(0) : 0;
  for (int c = 0; c < nc; ++c) {
    stage_barrier();
    if (c + 1 < nc) issue(c + 1, q ^ 1);
    const int k0 = c * KD;
    if (!LV::kAll) mask = blocks(k0 / 16);
    if (!MASKED || mask)
      mfma_stage<NTILE, TALL, SC, MASKED, SWZ>(acc, s.a[q], oa.fast(k0), s.b[q], ob.fast(k0), s.d[SC ? q : 0], mask);
    q ^= 1;
  }
}

// f(acc) with the accumulators of a tile of mrows rows: the square wave layout,
// or the tall one where at most three of the four 16-row blocks are live.  (16
// columns have one block per wave: one layout.)
template <bool CPLX, int NTILE, class F>
__device__ __forceinline__ void with_layout(int mrows, F f) {
  if (NTILE == 16 || mrows > 48) {
    Acc<CPLX, NTILE, false> acc;
    acc.zero();
    f(acc);
  } else if constexpr (NTILE != 16) {
    Acc<CPLX, NTILE, true> acc;
    acc.zero();
    f(acc);
  }
}
// the block swizzle gemm_lds uses for an accumulator type
template <class A>
struct AccLayout;
template <bool CPLX, int NTILE, bool TALL>
struct AccLayout<Acc<CPLX, NTILE, TALL>> {
  static constexpr bool kSquare64 = NTILE == 64 && !TALL;
};
template <class A, class LV>
constexpr int swz_of = AccLayout<std::decay_t<A>>::kSquare64 ? LV::kSwz : 0;

// --------------------------------------------------------------------------
// small kernels
// --------------------------------------------------------------------------
// p[0 .. n) = 0, p aligned to 16 bytes.  One 16-byte store per thread up to
// FILL_BLOCKS workgroups (32 GiB): 2 GiB fill at 6.8 TB/s so, and at 4.3 with
// 8192 workgroups that step through it (a wave's stores 32 MB apart).  An odd
// last double is one thread's 8-byte store.
constexpr int FILL_BLOCKS = 1 << 23;
__global__ void k_fill_zero(double* p, int64_t n) {
  const int64_t first = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  const int64_t stride = (int64_t)gridDim.x * blockDim.x;
  double2* p2 = (double2*)p;
  for (int64_t i = first; i < n / 2; i += stride) p2[i] = make_double2(0.0, 0.0);
  if (first == 0 && (n & 1)) p[n - 1] = 0.0;
}

// Real shifts eps_q as the complex shifts (eps_q, 0) of an inertia batch.
__global__ void k_real_shifts(const double* __restrict__ eps, double* __restrict__ shifts, int n) {
  const int q = blockIdx.x * blockDim.x + threadIdx.x;
  if (q < n) {
    shifts[2 * q] = eps[q];
    shifts[2 * q + 1] = 0.0;
  }
}

__global__ void k_zero_i64(int64_t* p, int n) {
  int i = blockIdx.x * blockDim.x + threadIdx.x;
  if (i < n) p[i] = 0;
}

// max |H| and max |S| (two-stage, deterministic)
__global__ void k_absmax_partial(const double* __restrict__ H, const double* __restrict__ S,
                                 int64_t nnz, double* partial) {
  __shared__ double sh[2][NT];
  double mh = 0.0, ms = 0.0;
  for (int64_t i = (int64_t)blockIdx.x * NT + threadIdx.x; i < nnz; i += (int64_t)gridDim.x * NT) {
    mh = fmax(mh, fabs(H[i]));
    ms = fmax(ms, fabs(S[i]));
  }
  sh[0][threadIdx.x] = mh;
  sh[1][threadIdx.x] = ms;
  __syncthreads();
  for (int s = NT / 2; s > 0; s >>= 1) {
    if (threadIdx.x < s) {
      sh[0][threadIdx.x] = fmax(sh[0][threadIdx.x], sh[0][threadIdx.x + s]);
      sh[1][threadIdx.x] = fmax(sh[1][threadIdx.x], sh[1][threadIdx.x + s]);
    }
    __syncthreads();
  }
  if (threadIdx.x == 0) {
    partial[2 * blockIdx.x] = sh[0][0];
    partial[2 * blockIdx.x + 1] = sh[1][0];
  }
}
// One wave per quantity (grid-wide partials of at most ABSMAX_BLOCKS blocks):
// a single thread over the 512 partials took 54 us.
__global__ void k_absmax_final(const double* partial, int nb, double* out) {
  const int q = threadIdx.x >> 6, lane = threadIdx.x & 63;   // q: 0 for H, 1 for S
  double m = 0.0;
  for (int b = lane; b < nb; b += 64) m = fmax(m, partial[2 * b + q]);
  for (int s = 32; s > 0; s >>= 1) m = fmax(m, __shfl_xor(m, s));
  if (lane == 0) out[q] = m;
}

// A_l = H - w_l S on the input pattern (the rest of the storage is zero).
template <bool CPLX>
__global__ void k_assemble(double* __restrict__ L, int64_t stride, const double* __restrict__ H,
                           const double* __restrict__ S, const int64_t* __restrict__ eoff,
                           int64_t nnz, const double* __restrict__ shifts) {
  const int sh = blockIdx.y;
  const double wr = shifts[2 * sh], wi = shifts[2 * sh + 1];
  double* Ls = L + (CPLX ? 2 : 1) * stride * sh;
  for (int64_t k = (int64_t)blockIdx.x * NT + threadIdx.x; k < nnz; k += (int64_t)gridDim.x * NT) {
    const double h = H[k], s = S[k];
    st_elem<CPLX>(Ls, eoff[k], cplx{h - wr * s, -wi * s});
  }
}

// --------------------------------------------------------------------------
// factor kernels
// --------------------------------------------------------------------------
struct PanelK {
  int64_t off;     // storage offset of the supernode
  int64_t cm;      // index of the supernode's row list in colmap/colseg
  int32_t ld;      // leading dimension of the supernode
  int32_t p0;      // panel's first column (position in the row list)
  int32_t wp;      // panel width
  int32_t nb;      // rows below the panel's diagonal block
  int32_t col0;    // new index of the panel's first column
  int32_t split;   // split-K pieces (SelInv diagonal update)
  int32_t w;       // width of the supernode
  int32_t c;       // rows below the supernode (ld - w)
  int32_t sh0;     // first shift of this launch (grid.y counts from it)
};

struct Common {
  double* L;               // factor storage of shift 0
  int64_t stride;          // elements per shift
  const int64_t* colmap;
  const int64_t* colseg;
  const int32_t* relpos;
  double* work;            // workspace base
  int64_t wps;             // workspace bytes per shift
  int64_t wfix;            // fixed workspace bytes
  const double* shifts;    // device, 2 doubles per shift
  const double* absmax;    // device, max|H|, max|S|
  int64_t* info;           // device, per shift
  int64_t* negc;           // device, per shift
  double pivtol;
  double* G;               // dense Z_CC of the current supernode, per shift of a chunk
  int64_t gstride;         // doubles per shift in G
  int64_t ut;              // Hermitian factorizations: elements from a shift's L region to its U^T region
};

template <bool CPLX>
__device__ __forceinline__ double* shift_base(const Common& c, int sh) {
  return c.L + (CPLX ? 2 : 1) * c.stride * sh;
}

// Where a workgroup finds its panel.  OnePanel: one panel of one system per
// launch (kernel argument), grid = (tiles, shifts).  PanelGroup: a table of
// panels of several systems launched as one grid of sum(tiles x shifts)
// workgroups (the fused execution of a batch of systems); each item's
// workgroups are a contiguous range of ids, with the XCD-aware order inside it.
struct OnePanel {
  Common c;
  PanelK p;
};

struct GroupItem {
  Common c;
  PanelK p;
  int64_t start;   // first logical workgroup of the item
  int32_t tiles;   // workgroups per shift
  int32_t nsh;     // shifts
};

struct PanelGroup {
  const GroupItem* items;
  int32_t n;
};

// LaneGroup: the same as PanelGroup for at most N panels of one system whose
// items travel in the kernel arguments (no device table, so a stream capture
// records them like any other launch): the fused launches of a tree of small
// supernodes.  Everything but the panel and the workspace views is common;
// starts sit in one array, which a workgroup reads as a whole.  A launch of one
// panel goes as OnePanel and one of up to FEW_ITEMS in the short form: reading
// 3.6 KB of arguments adds 2 us to every launch.
constexpr int MAX_ITEMS = 32, FEW_ITEMS = 8;
struct LaneItem {
  PanelK p;
  int64_t wfix;      // workspace views of the item (Common's fields)
  double* G;
  int64_t gstride;
  int32_t tiles;     // workgroups per shift
  int32_t nsh;       // shifts
};
template <int N>
struct LaneGroup {
  Common c;
  int32_t start[N];   // first logical workgroup of the item (INT32_MAX behind the last)
  LaneItem it[N];
};
static_assert(sizeof(LaneGroup<MAX_ITEMS>) <= 4096, "kernel arguments");

// remap: XCD-aware order (else the plain one); bx = tile, by = shift
__device__ __forceinline__ void locate(const OnePanel& src, Common& c, PanelK& p, int& bx, int& by, bool remap) {
  c = src.c;
  p = src.p;
  if (remap) {
    xcd_remap(bx, by);
  } else {
    bx = blockIdx.x;
    by = blockIdx.y;
  }
}

__device__ __forceinline__ void locate(const PanelGroup& src, Common& c, PanelK& p, int& bx, int& by, bool remap) {
  // the item by the plain id, the XCD-aware order within it: items differ in
  // the work of their tiles, and every XCD gets a share of each (a remap over
  // the whole grid gave whole items to an XCD: a sheet of N=7956 fused took
  // 236 ms against 214 panel by panel)
  const int64_t lid = blockIdx.x;
  int lo = 0, hi = src.n - 1;     // the last item starting at or before lid
  while (lo < hi) {
    const int mid = (lo + hi + 1) >> 1;
    if (src.items[mid].start <= lid) lo = mid;
    else hi = mid - 1;
  }
  const GroupItem& it = src.items[lo];
  c = it.c;
  p = it.p;
  int local = (int)(lid - it.start);
  if (remap) local = xcd_logical(local, it.tiles * it.nsh);
  bx = local % it.tiles;
  by = local / it.tiles;
}

template <int N>
__device__ __forceinline__ void locate(const LaneGroup<N>& src, Common& c, PanelK& p, int& bx, int& by, bool remap) {
  const int lx = (int)blockIdx.x;
  int i = -1;   // the last item starting at or before lx
#pragma unroll
  for (int q = 0; q < N; ++q) i += src.start[q] <= lx ? 1 : 0;
  const LaneItem& it = src.it[i];
  c = src.c;
  c.wfix = it.wfix;
  c.G = it.G;
  c.gstride = it.gstride;
  p = it.p;
  int local = lx - src.start[i];
  if (remap) local = xcd_logical(local, it.tiles * it.nsh);   // within the item, as for PanelGroup
  bx = local % it.tiles;
  by = local / it.tiles;
}

// Pivot report of a diagonal block: the smallest flagged column of a shift
// wins (0 = none yet), whatever the order in which independent subtrees run;
// negative pivots add up.
__device__ __forceinline__ void flag_pivots(const Common& c, int sh, int bad, int neg) {
  if (bad) {
    unsigned long long* q = (unsigned long long*)&c.info[sh];
    unsigned long long old = atomicCAS(q, 0ull, (unsigned long long)bad);
    while (old != 0ull && old > (unsigned long long)bad) {
      const unsigned long long seen = atomicCAS(q, old, (unsigned long long)bad);
      if (seen == old) break;
      old = seen;
    }
  }
  if (neg) atomicAdd((unsigned long long*)&c.negc[sh], (unsigned long long)neg);
}

// Dense LDL^T of the panel's wp x wp diagonal block in LDS with L_pp^{-1}.
//
// What bounds it is the chain of wp dependent column steps on one workgroup
// per shift.  With a barrier and a read-modify-write of the whole trailing
// block in LDS per column (512 threads) a step took 0.97 us: 62 us per launch
// of 64 columns x 60 shifts.  Here the block is cut into 16-column block
// columns:
//   panel(b)   wave 0, one row per lane, the 16 columns in registers: per
//              column the pivot and the multipliers of the 15 rows below are
//              broadcast by lane reads, no LDS and no barrier;
//   next(b)    block column b + 1 of the trailing matrix on the matrix cores
//              (waves 0-2), so panel(b + 1) can start;
//   rest(b)    beside panel(b + 1), waves 1-3: the other trailing blocks and
//              the inverse: X_bm = X_bb Y_bm for the columns m < b, Y_im -= L_ib
//              X_bm for the rows below (X = L^{-1}, Y its partial sums).  X_bb
//              comes from lanes of panel(b) that have no row.
// With at most SMALL_ROWS rows below the block it also computes them (L_Bp =
// A_Bp L_pp^{-T} D^{-1}, k_trsm's work): a launch less where a launch is what
// counts (a chain's k_trsm took 8 us beside 16 of this kernel).
// 26 us per launch of 64 complex columns x 60 shifts (real: 25), 14 for 16
// columns; of the 64-column time about 11 us are panels (one wave's issue of
// lane reads and fused multiply-adds), 4 the trailing products, the rest
// loads, stores and launch.  a[col][row] holds A, then L, in its
// lower triangle (block columns in place) and X transposed in the strict upper
// one, a[row][col] = X[row][col]: one array (66.5 KB of LDS), so a workgroup
// fits on a CU beside two of the matrix kernels.  Rows and columns from wp on
// are those of the identity.
constexpr int NTD = 256;
constexpr int SMALL_ROWS = 80;   // rows below a panel that k_diag and k_selinv_small take along
constexpr int LDD = 65;   // row stride of a[][]: 16-byte elements rotate over the banks

__device__ __forceinline__ cplx to_cplx(dbl2 v) { return {v.x, v.y}; }
__device__ __forceinline__ cplx to_cplx(double v) { return {v, 0.0}; }
template <bool CPLX>
__device__ __forceinline__ elem_t<CPLX> to_elem(cplx v) {
  if constexpr (CPLX) return dbl2{v.re, v.im};
  else return v.re;
}
// products that drop the imaginary part of real elements
template <bool CPLX>
__device__ __forceinline__ cplx mul(cplx a, cplx b) {
  if constexpr (CPLX) return cmul(a, b);
  else return {a.re * b.re, 0.0};
}
// x -= a b, one fused operation per product
template <bool CPLX>
__device__ __forceinline__ void sub_mul(cplx& x, cplx a, cplx b) {
  x.re = fma(-a.re, b.re, x.re);
  if constexpr (CPLX) {
    x.im = fma(-a.re, b.im, x.im);
    x.re = fma(a.im, b.im, x.re);
    x.im = fma(-a.im, b.re, x.im);
  }
}
template <bool CPLX>
__device__ __forceinline__ cplx inv_of(cplx d) {
  if constexpr (CPLX) return cinv(d);
  else return {1.0 / d.re, 0.0};
}
__device__ __forceinline__ double lane_read(double v, int lane) {
  const uint64_t u = __double_as_longlong(v);
  const uint32_t lo = (uint32_t)__builtin_amdgcn_readlane((int)(uint32_t)u, lane);
  const uint32_t hi = (uint32_t)__builtin_amdgcn_readlane((int)(uint32_t)(u >> 32), lane);
  return __longlong_as_double(((uint64_t)hi << 32) | lo);
}

// Orders the wave's LDS accesses before and after it (no instruction: a wave's
// LDS operations execute in order; it keeps the compiler from reusing values
// that other lanes have replaced).
__device__ __forceinline__ void wave_sync() {
  __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
  __builtin_amdgcn_wave_barrier();
}

// One 16 x 16 x 16 block product on the calling wave: fa(m, k) and fb(k, n)
// give the operands, out(m, n, value) takes P[m][n] (lanes run along n).
template <bool CPLX, class FA, class FB, class FO>
__device__ __forceinline__ void block_product(FA fa, FB fb, FO out) {
  const int lane = threadIdx.x & 63, li = lane & 15, lk = lane >> 4;
  dbl4 re{0.0, 0.0, 0.0, 0.0}, im{0.0, 0.0, 0.0, 0.0};
#pragma unroll
  for (int ks = 0; ks < 4; ++ks) {
    const int k = ks * 4 + lk;
    const cplx x = fa(li, k), y = fb(k, li);
    re = __builtin_amdgcn_mfma_f64_16x16x4f64(x.re, y.re, re, 0, 0, 0);
    if constexpr (CPLX) {
      im = __builtin_amdgcn_mfma_f64_16x16x4f64(x.re, y.im, im, 0, 0, 0);
      re = __builtin_amdgcn_mfma_f64_16x16x4f64(x.im, y.im, re, 0, 0, 1);
      im = __builtin_amdgcn_mfma_f64_16x16x4f64(x.im, y.re, im, 0, 0, 0);
    }
  }
#pragma unroll
  for (int r = 0; r < 4; ++r) out(lk + 4 * r, li, cplx{re[r], im[r]});
  __builtin_amdgcn_sched_barrier(0);
}

template <bool CPLX, class Src>
__global__ void __launch_bounds__(NTD, 2) k_diag(Src src) {
  using T = elem_t<CPLX>;
  __shared__ T a[64][LDD];
  __shared__ T pv[64];   // pivots d_k
  Common c;
  PanelK p;
  int bx, sh;
  locate(src, c, p, bx, sh, false);
  double* Ls = shift_base<CPLX>(c, sh);
  const int wp = p.wp;
  const int t = threadIdx.x;
  const int lane = t & 63, li = lane & 15, lk = lane >> 4;
  const int w = wave_id();
  const int nblk = (wp + 15) / 16;
  const int64_t dbase = p.off + (int64_t)p.p0 * p.ld + p.p0;
  {
    cplx v[16];
#pragma unroll
    for (int u = 0; u < 16; ++u) {
      const int cc = w + 4 * u;
      v[u] = cplx{lane == cc ? 1.0 : 0.0, 0.0};
      if (lane >= cc && lane < wp) v[u] = ld_elem<CPLX>(Ls, dbase + (int64_t)cc * p.ld + lane);
    }
#pragma unroll
    for (int u = 0; u < 16; ++u) {
      const int cc = w + 4 * u;
      if (lane >= cc) a[cc][lane] = to_elem<CPLX>(v[u]);
    }
  }
  auto L = [&](int r, int k) { return to_cplx(a[k][r]); };
  auto X = [&](int r, int k) { return to_cplx(a[r][k]); };
  // X_bb as an operand: unit diagonal, zero above it
  auto Xd = [&](int c0, int r, int k) {
    const cplx v = X(c0 + r, c0 + k);
    return r > k ? v : cplx{r == k ? 1.0 : 0.0, 0.0};
  };
  // A_ij -= L_ib D_b L_jb^T (block row i, block column j)
  auto trailing = [&](int b, int i, int j) {
    const int kb = 16 * b;
    block_product<CPLX>([&](int m, int k) { return mul<CPLX>(to_cplx(pv[kb + k]), L(16 * j + m, kb + k)); },
                        [&](int k, int n) { return L(16 * i + n, kb + k); },
                        [&](int m, int n, cplx v) {
                          if (i == j && n < m) return;
                          T& e = a[16 * j + m][16 * i + n];
                          const cplx o = to_cplx(e);
                          e = to_elem<CPLX>(cplx{o.re - v.re, o.im - v.im});
                        });
  };
  // X_00 by substitution (the panels of the later blocks have lanes to spare
  // for theirs): column li, rows lk, lk + 4, ... per lane; every wave computes
  // and stores the same values
  auto inverse_of_first = [&]() {
    cplx x[4];
#pragma unroll
    for (int u = 0; u < 4; ++u) x[u] = cplx{lk + 4 * u == li ? 1.0 : 0.0, 0.0};
#pragma unroll
    for (int k = 0; k < 15; ++k) {
      const int from = (k & 3) * 16 + li;   // the lane that holds X[k][li]
      const cplx xk{__shfl(x[k >> 2].re, from), CPLX ? __shfl(x[k >> 2].im, from) : 0.0};
#pragma unroll
      for (int u = k >> 2; u < 4; ++u) {
        const int r = lk + 4 * u;
        sub_mul<CPLX>(x[u], r > k ? L(r, k) : cplx{0.0, 0.0}, xk);
      }
    }
#pragma unroll
    for (int u = 0; u < 4; ++u)
      if (li < lk + 4 * u) a[lk + 4 * u][li] = to_elem<CPLX>(x[u]);
  };
  // the inverse's share of step b, column blocks m = q, q + nq, ...
  auto inverse = [&](int b, int q, int nq) {
    const int c0 = 16 * b;
    if (b == 0 && wp > 48) inverse_of_first();
    wave_sync();
    for (int m = q; m <= b; m += nq) {
      if (m < b)
        block_product<CPLX>([&](int r, int k) { return Xd(c0, r, k); }, [&](int k, int n) { return X(c0 + k, 16 * m + n); },
                            [&](int r, int n, cplx v) { a[c0 + r][16 * m + n] = to_elem<CPLX>(v); });
      wave_sync();
      for (int i = b + 1; i < nblk; ++i)
        block_product<CPLX>([&](int r, int k) { return L(16 * i + r, c0 + k); },
                            [&](int k, int n) { return m < b ? X(c0 + k, 16 * m + n) : Xd(c0, k, n); },
                            [&](int r, int n, cplx v) {
                              T& e = a[16 * i + r][16 * m + n];
                              const cplx o = m < b ? to_cplx(e) : cplx{0.0, 0.0};
                              e = to_elem<CPLX>(cplx{o.re - v.re, o.im - v.im});
                            });
    }
  };
  __syncthreads();
  for (int b = 0; b < nblk; ++b) {
    const int c0 = 16 * b;
    if (w == 0) {
      const int row = c0 + lane;
      // lanes without a row of A (LE and up, unless the first block column has
      // 64 rows) carry the rows of an identity below it: their entries before
      // the division are (I L_bb^{-T})[i][j] = X_bb[j][i]
      const int LE = b > 0 || wp <= 48 ? 48 : 64;
      const bool in = lane < LE && row < 64;
      cplx x[16];
#pragma unroll
      for (int k = 0; k < 16; ++k) x[k] = in ? to_cplx(a[c0 + k][row]) : cplx{lane - LE == k ? 1.0 : 0.0, 0.0};
      // one basic block: the next column is updated first and its pivot's
      // reciprocal runs beside the updates of the others
      cplx id = inv_of<CPLX>(cplx{lane_read(x[0].re, 0), CPLX ? lane_read(x[0].im, 0) : 0.0});
      auto column = [&](int j) {
        const cplx aj = x[j];   // A[row][j] before the division
        const cplx l = mul<CPLX>(aj, id);
#pragma unroll
        for (int k = j + 1; k < 16; ++k) {
          sub_mul<CPLX>(x[k], l, cplx{lane_read(aj.re, k), CPLX ? lane_read(aj.im, k) : 0.0});
          if (k == j + 1) id = inv_of<CPLX>(cplx{lane_read(x[k].re, k), CPLX ? lane_read(x[k].im, k) : 0.0});
        }
        const bool keep = lane == j || lane >= LE;
        x[j].re = keep ? aj.re : l.re;
        x[j].im = keep ? aj.im : l.im;
      };
#pragma unroll
      for (int j = 0; j < 8; ++j) column(j);
      if (c0 + 8 < wp) {   // else only identity columns follow, which stay as they are
#pragma unroll
        for (int j = 8; j < 16; ++j) column(j);
      }
#pragma unroll
      for (int k = 0; k < 16; ++k) {
        if (in && lane > k) a[c0 + k][row] = to_elem<CPLX>(x[k]);
        if (lane == k) pv[c0 + k] = to_elem<CPLX>(x[k]);
        // X_bb[k][i] from the identity row i
        if (lane >= LE && lane - LE < k) a[c0 + k][c0 + lane - LE] = to_elem<CPLX>(x[k]);
      }
    } else if (b > 0) {
      // the trailing blocks right of column b by step b - 1, then its inverse
      int q = 0;
      for (int j = b + 1; j < nblk; ++j)
        for (int i = j; i < nblk; ++i)
          if (q++ % 3 == w - 1) trailing(b - 1, i, j);
      inverse(b - 1, w - 1, 3);
    }
    __syncthreads();
    if (b + 1 < nblk && b + 1 + w < nblk) trailing(b, b + 1 + w, b + 1);
    __syncthreads();
  }
  // the rows below, block column w of 16 rows at a time
  const bool rows_too = p.nb > 0 && p.nb <= SMALL_ROWS;
  const int64_t rbase = dbase + wp;
  cplx f[16];
  auto load_rows = [&](int n) {
    const int i = 16 * n + li;
#pragma unroll
    for (int ks = 0; ks < 16; ++ks) {
      const int k = 4 * ks + lk;
      f[ks] = cplx{0.0, 0.0};
      if (i < p.nb && k < wp) f[ks] = ld_elem<CPLX>(Ls, rbase + (int64_t)k * p.ld + i);
    }
  };
  if (rows_too) load_rows(0);
  inverse(nblk - 1, w, 4);
  if (w == 0) {
    const double wabs = sqrt(c.shifts[2 * sh] * c.shifts[2 * sh] + c.shifts[2 * sh + 1] * c.shifts[2 * sh + 1]);
    const double thr = c.pivtol * (c.absmax[0] + (CPLX ? wabs : fabs(c.shifts[2 * sh])) * c.absmax[1]);
    const cplx d = to_cplx(pv[lane]);
    const double ad = CPLX ? sqrt(d.re * d.re + d.im * d.im) : fabs(d.re);
    const uint64_t tiny = __ballot(lane < wp && !(ad >= thr));
    const int neg = CPLX ? 0 : __popcll(__ballot(lane < wp && d.re < 0.0));
    if (lane == 0) flag_pivots(c, sh, tiny ? p.col0 + __ffsll((unsigned long long)tiny) : 0, neg);
  }
  __syncthreads();
#pragma unroll
  for (int u = 0; u < 16; ++u) {
    const int cc = w + 4 * u;
    if (lane < wp && lane >= cc)
      st_elem<CPLX>(Ls, dbase + (int64_t)cc * p.ld + lane, to_cplx(lane > cc ? a[lane][cc] : pv[cc]));
  }
  if (!rows_too) return;
  for (int n = 0; 16 * n < p.nb; ++n) {
    if (n > 0) load_rows(n);
    stage_barrier();   // every wave has read the rows that the others overwrite
    if (w >= nblk) continue;
    dbl4 re{0.0, 0.0, 0.0, 0.0}, im{0.0, 0.0, 0.0, 0.0};
#pragma unroll
    for (int ks = 0; ks < 16; ++ks) {
      if (ks / 4 > w) continue;   // X[c][k] = 0 for k > c
      const int r = 16 * w + li, k = 4 * ks + lk;
      const cplx x = r > k ? X(r, k) : cplx{r == k ? 1.0 : 0.0, 0.0};
      re = __builtin_amdgcn_mfma_f64_16x16x4f64(x.re, f[ks].re, re, 0, 0, 0);
      if constexpr (CPLX) {
        im = __builtin_amdgcn_mfma_f64_16x16x4f64(x.re, f[ks].im, im, 0, 0, 0);
        re = __builtin_amdgcn_mfma_f64_16x16x4f64(x.im, f[ks].im, re, 0, 0, 1);
        im = __builtin_amdgcn_mfma_f64_16x16x4f64(x.im, f[ks].re, im, 0, 0, 0);
      }
    }
#pragma unroll
    for (int r = 0; r < 4; ++r) {
      const int cc = 16 * w + lk + 4 * r, i = 16 * n + li;
      if (cc < wp && i < p.nb)
        st_elem<CPLX>(Ls, rbase + (int64_t)cc * p.ld + i, mul<CPLX>(cplx{re[r], im[r]}, inv_of<CPLX>(to_cplx(pv[cc]))));
    }
  }
}

// L_Bp = A_Bp L_pp^{-T} D^{-1}: P[c][i] = sum_k Linv[c][k] A[i][k], then / d_c.
// Panel products run on tiles of 64 x TN (TN = 64, 32 or 16 rows, pick_tile), at
// most 33 KB of LDS and 128 registers: four workgroups per CU.
#define PXS_LB __launch_bounds__(NT, 4)

template <bool CPLX, int TN, class Src>
__global__ void PXS_LB k_trsm(Src src) {
  __shared__ cplx dinv[64];
  Common c;
  PanelK p;
  int bx, by;
  locate(src, c, p, bx, by, true);
  const int sh = by;
  double* Ls = shift_base<CPLX>(c, sh);
  const int i0 = bx * TN;
  const int64_t dbase = p.off + (int64_t)p.p0 * p.ld + p.p0;   // (p0, p0)
  const int64_t rbase = dbase + p.wp;                          // first row below
  if (threadIdx.x < p.wp) {
    const cplx d = ld_elem<CPLX>(Ls, dbase + (int64_t)threadIdx.x * p.ld + threadIdx.x);
    dinv[threadIdx.x] = CPLX ? cinv(d) : cplx{1.0 / d.re, 0.0};
  }
  constexpr int E = CPLX ? 2 : 1;   // doubles per element
  // L^{-1} is lower triangular: the all-zero blocks of a stage are not
  // multiplied
  __shared__ TileStage<CPLX, TN, false> s;
  with_layout<CPLX, TN>(p.wp, [&](auto& acc) {
    gemm_lds(acc, s, p.wp, p.wp, TriOp<CPLX, false>(Ls + E * dbase, p.ld, p.wp),
             ColsOp<CPLX, TN>(Ls + E * (rbase + i0), p.ld, p.nb - i0, p.wp), NoDiag(), TriBlocks<true>());
    acc_foreach<CPLX, TN, swz_of<decltype(acc), TriBlocks<true>>>(acc, [&](int m, int n, cplx v) {
      const int ig = i0 + n;
      if (m < p.wp && ig < p.nb) st_elem<CPLX>(Ls, rbase + (int64_t)m * p.ld + ig, mul<CPLX>(v, dinv[m]));
    });
  });
}

// Left-looking update of panel p from the earlier columns of its own
// supernode: A[r][c] -= sum_{k < p0} L[r][k] d_k L[c][k] for rows r >= p0 of
// the row list and the panel's columns c.  P[c][r] = sum_k (d_k L[c][k]) L[r][k].
template <bool CPLX, int TN, class Src>
__global__ void PXS_LB k_int_update(Src src) {
  Common c;
  PanelK p;
  int bx, by;
  locate(src, c, p, bx, by, true);
  const int sh = by;
  double* Ls = shift_base<CPLX>(c, sh);
  const int r0 = bx * TN;            // rows p0 + r0 .. of the row list
  const int nrows = p.ld - p.p0;
  const int64_t cbase = p.off + p.p0;        // element (row p0, column 0)
  auto at = [&](int m, int n, int64_t& e) {
    const int rg = r0 + n;
    // clamped into the panel (in bounds for skipped elements)
    e = cbase + (int64_t)(p.p0 + min(m, p.wp - 1)) * p.ld + min(rg, nrows - 1);
    return m < p.wp && rg < nrows && rg >= m;
  };
  // A: L[p0 + c][k], scaled by d_k on the way to the MFMAs; B: L[p0 + r][k]
  constexpr int E = CPLX ? 2 : 1;
  __shared__ TileStage<CPLX, TN, true> s;
  with_layout<CPLX, TN>(p.wp, [&](auto& acc) {
    gemm_lds(acc, s, p.wp, p.p0, ColsOp<CPLX, 64>(Ls + E * cbase, p.ld, p.wp, p.p0),
             ColsOp<CPLX, TN>(Ls + E * (cbase + r0), p.ld, nrows - r0, p.p0),
             DiagOp<CPLX>(Ls + E * p.off, (int64_t)p.ld + 1, p.p0), AllBlocks());
    acc_sub_into(acc, Ls, at);
  });
}

__device__ __forceinline__ void tri_index(int b, int& ti, int& tj) {
  // b enumerates the pairs (ti >= tj) row by row: b = ti (ti + 1) / 2 + tj
  int x = (int)((sqrt(8.0 * (double)b + 1.0) - 1.0) * 0.5);
  while ((x + 1) * (x + 2) / 2 <= b) ++x;
  while (x * (x + 1) / 2 > b) --x;
  ti = x;
  tj = b - x * (x + 1) / 2;
}

// Update of the rows/columns below columns [p0, p0 + wp) of a supernode:
// A_BB -= L_B,K D_K L_B,K^T on lower tiles (ti >= tj), scattered through the
// maps (B = row-list positions from p0 + wp on).  Used once per supernode
// with K = all of its columns (p0 = 0, wp = w_J, B = the rows below it).
// P[j][i] = sum_k (d_k L[j][k]) L[i][k].
template <bool CPLX, int TN, class Src>
__global__ void PXS_LB k_update(Src src) {
  Common c;
  PanelK p;
  int bx, by;
  locate(src, c, p, bx, by, true);
  const int sh = by;
  double* Ls = shift_base<CPLX>(c, sh);
  // tiles: 64 columns j (m) by TN rows i (n); only tiles that reach the
  // lower triangle (some i >= some j) do work
  const int nti = (p.nb + TN - 1) / TN;
  const int tj = bx / nti, ti = bx % nti;
  const int i0 = ti * TN, j0 = tj * TM;
  if (i0 + TN - 1 < j0) return;
  const int base = p.p0 + p.wp;   // row-list position of the first row below
  const int64_t rbase = p.off + base;   // element (row base, column 0)
  const int kb = p.p0, ke = p.p0 + p.wp;
  const int64_t* cmap = c.colmap + p.cm;
  const int64_t* cseg = c.colseg + p.cm;
  auto at = [&](int m, int n, int64_t& e) {
    const int jg = j0 + m, ig = i0 + n;
    // branch-free, so the map loads of all elements are in flight together:
    // indices clamped into the supernode's row list with row >= column
    // (where relpos is defined); a skipped element reads a valid position
    // and is not stored
    const int jc = min(jg, p.nb - 1), ic = min(max(ig, jc), p.nb - 1);
    e = cmap[base + jc] + c.relpos[cseg[base + jc] + base + ic];
    return jg < p.nb && ig < p.nb && ig >= jg;
  };
  constexpr int E = CPLX ? 2 : 1;
  __shared__ TileStage<CPLX, TN, true> s;
  const int64_t k0 = rbase + (int64_t)kb * p.ld;
  with_layout<CPLX, TN>(min(64, p.nb - j0), [&](auto& acc) {
    gemm_lds(acc, s, p.nb - j0, ke - kb, ColsOp<CPLX, 64>(Ls + E * (k0 + j0), p.ld, p.nb - j0, ke - kb),
             ColsOp<CPLX, TN>(Ls + E * (k0 + i0), p.ld, p.nb - i0, ke - kb),
             DiagOp<CPLX>(Ls + E * (p.off + (int64_t)kb * (p.ld + 1)), (int64_t)p.ld + 1, ke - kb), AllBlocks());
    acc_sub_into(acc, Ls, at);
  });
}

// --------------------------------------------------------------------------
// selected inversion kernels (complex only)
// --------------------------------------------------------------------------
__device__ __forceinline__ double* wbase(const Common& c, int sh) {
  return (double*)((char*)c.work + c.wfix + c.wps * sh);
}

// W = L_Bp Linv: P[c][i] = sum_k Linv[k][c] L[i][k]; W stored W[c * nb + i].
template <int TN, class Src>
__global__ void PXS_LB k_lhat(Src src) {
  __shared__ TileStage<true, TN, false> s;
  Common c;
  PanelK p;
  int bx, by;
  locate(src, c, p, bx, by, true);
  const int sh = p.sh0 + by;
  double* Ls = shift_base<true>(c, sh);
  double* W = wbase(c, sh);
  const int i0 = bx * TN;
  const int64_t dbase = p.off + (int64_t)p.p0 * p.ld + p.p0;
  const int64_t rbase = dbase + p.wp;
  // A[m][k] = L^{-1}[k][m] vanishes for k < m (see k_trsm)
  with_layout<true, TN>(p.wp, [&](auto& acc) {
    gemm_lds(acc, s, p.wp, p.wp, TriOp<true, true>(Ls + 2 * dbase, p.ld, p.wp),
             ColsOp<true, TN>(Ls + 2 * (rbase + i0), p.ld, p.nb - i0, p.wp), NoDiag(), TriBlocks<false>());
    acc_foreach<true, TN, swz_of<decltype(acc), TriBlocks<false>>>(acc, [&](int m, int n, cplx v) {
      const int ig = i0 + n;
      if (m < p.wp && ig < p.nb) st_elem<true>(W, (int64_t)m * p.nb + ig, v);
    });
  });
}

// Z_Bp = -Z_BB W: P[c][i] = sum_k W[k][c] Z(k, i).  Z_BB is symmetric; its
// part inside the supernode's own columns is read from the supernode's
// storage (column min(i, k), row max(i, k)), the part in the rows below it
// from the dense copy G of Z_CC made by k_gather_cc.
template <int TN, class Src>
__global__ void PXS_LB k_selinv_off(Src src) {
  __shared__ TileStage<true, TN, false> s;
  Common c;
  PanelK p;
  int bx, by;
  locate(src, c, p, bx, by, true);
  const int sh = p.sh0 + by;
  double* Ls = shift_base<true>(c, sh);
  const double* W = wbase(c, sh);
  const double* G = c.G + c.gstride * by;
  const int i0 = bx * TN;
  const int base = p.p0 + p.wp;
  const int gw = p.w - base;   // rows of B inside the supernode
  const int64_t rbase = p.off + (int64_t)p.p0 * p.ld + base;
  with_layout<true, TN>(p.wp, [&](auto& acc) {
    gemm_lds(acc, s, p.wp, p.nb, RowsOp<64>(W, p.nb, p.wp, p.nb),
             SymOp<TN, false>(Ls + 2 * (p.off + (int64_t)base * (p.ld + 1)), p.ld, G - 2 * (int64_t)gw * (p.c + 1), p.c, gw,
                              i0, p.nb),
             NoDiag(), AllBlocks());
    acc_foreach<true, TN>(acc, [&](int m, int n, cplx v) {
      const int ig = i0 + n;
      if (m < p.wp && ig < p.nb) st_elem<true>(Ls, rbase + (int64_t)m * p.ld + ig, cplx{-v.re, -v.im});
    });
  });
}

// G = Z_CC, lower triangle: G[a + b c] = Z(w + a, w + b) for b <= a < c,
// gathered from the ancestors' storage through the maps.  Each thread moves
// 16 elements of a 64 x 64 tile: first all relative row positions, then all
// values, then the stores, so the loads of a thread are in flight together.
template <class Src>
__global__ void __launch_bounds__(NT) k_gather_cc(Src src) {
  Common c;
  PanelK p;
  int bx, by;
  locate(src, c, p, bx, by, false);
  const int sh = p.sh0 + by;
  const double* Ls = shift_base<true>(c, sh);
  double* G = c.G + c.gstride * by;
  int ta, tb;
  tri_index(bx, ta, tb);
  const int a0 = ta * TM, b0 = tb * TM;
  const int cc = p.c, w = p.w;
  const int64_t* cmap = c.colmap + p.cm;
  const int64_t* cseg = c.colseg + p.cm;
  const int t = threadIdx.x;
  const int a = a0 + (t & 63);
  int64_t e[16];
  bool ok[16];
  // branch-free, so all map and value loads of a thread are in flight
  // together: indices clamped into Z_CC with row >= column (where relpos is
  // defined); skipped elements read a valid position and are not stored
#pragma unroll
  for (int j = 0; j < 16; ++j) {
    const int b = b0 + (t >> 6) + 4 * j;
    ok[j] = (a < cc && b < cc && a >= b);
    const int bc = min(b, cc - 1), ac = min(max(a, bc), cc - 1);
    e[j] = cmap[w + bc] + c.relpos[cseg[w + bc] + w + ac];
  }
  cplx v[16];
#pragma unroll
  for (int j = 0; j < 16; ++j) v[j] = ld_elem<true>(Ls, e[j]);
#pragma unroll
  for (int j = 0; j < 16; ++j) {
    const int b = b0 + (t >> 6) + 4 * j;
    if (ok[j]) st_elem<true>(G, (int64_t)b * cc + a, v[j]);
  }
}

// Partial W^T Z_Bp over k in [split * SPLIT_ROWS, ...): P[c][r] = sum_k Z[k][c] W[k][r],
// in tiles of TN of its columns r (tile bx = split x columns).
template <int TN, class Src>
__global__ void PXS_LB k_selinv_diag_partial(Src src) {
  __shared__ TileStage<true, TN, false> s;
  Common c;
  PanelK p;
  int bx, by;
  locate(src, c, p, bx, by, true);
  const int sh = p.sh0 + by;
  const int nt = (p.wp + TN - 1) / TN;
  const int sp = bx / nt, n0 = (bx - sp * nt) * TN;
  double* Ls = shift_base<true>(c, sh);
  double* W = wbase(c, sh);
  double* part = W + 2 * (int64_t)p.nb * p.wp;   // after W: split x 64 x 64 complex
  const int base = p.p0 + p.wp;
  const int64_t rbase = p.off + (int64_t)p.p0 * p.ld + base;
  const int kb = sp * (int)SPLIT_ROWS, ke = min(p.nb, kb + (int)SPLIT_ROWS);
  double* out = part + 2 * (int64_t)sp * 64 * 64;
  // Z_pp is symmetric and stored by its lower triangle: only P[c][r], r >= c,
  // is summed by k_selinv_diag_final, so the blocks below that are skipped
  with_layout<true, TN>(p.wp, [&](auto& acc) {
    const UpperBlocks lv{n0 / 16};
    gemm_lds(acc, s, p.wp, ke - kb, RowsOp<64>(Ls + 2 * (rbase + kb), p.ld, p.wp, ke - kb),
             RowsOp<TN>(W + 2 * ((int64_t)n0 * p.nb + kb), p.nb, p.wp - n0, ke - kb), NoDiag(), lv);
    acc_foreach<true, TN, swz_of<decltype(acc), UpperBlocks>>(
        acc, [&](int m, int n, cplx v) { st_elem<true>(out, (int64_t)m * 64 + n0 + n, v); });
  });
}

// Z_pp = Linv^T D^{-1} Linv - sum of the partials, written over the diagonal block.
// One workgroup per shift (the block is overwritten in place, so it is read
// by the same workgroup that writes it).  Latency bound: the 16 x 16 blocks
// on and below the diagonal run on the matrix cores, one or two per wave, as
// Z_RC = sum over the block rows k >= R of X_kR^T D_k^{-1} X_kC (X = Linv), and
// the partials of a wave's blocks are summed while the block is on its way.
// Scalar dot products over the 64 rows in LDS took 22.7 us per launch at 60
// shifts.
constexpr int NTF = 512;
template <class Src>
__global__ void __launch_bounds__(NTF, 2) k_selinv_diag_final(Src src) {
  __shared__ dbl2 x[64][LDD];   // x[col][row] = Linv[row][col]
  __shared__ cplx dinv[64];
  Common c;
  PanelK p;
  int bx, by;
  locate(src, c, p, bx, by, false);
  const int sh = p.sh0 + by;
  double* Ls = shift_base<true>(c, sh);
  const double* W = wbase(c, sh);
  const double* part = W + 2 * (int64_t)p.nb * p.wp;
  const int wp = p.wp;
  const int lane = threadIdx.x & 63, li = lane & 15, lk = lane >> 4;
  const int w = wave_id();
  const int64_t dbase = p.off + (int64_t)p.p0 * p.ld + p.p0;
  cplx v[8];
#pragma unroll
  for (int u = 0; u < 8; ++u) {
    const int cc = w + 8 * u;
    v[u] = cplx{0.0, 0.0};
    if (lane >= cc && lane < wp) v[u] = ld_elem<true>(Ls, dbase + (int64_t)cc * p.ld + lane);
  }
  // the wave's blocks (R >= C) in the order of tri_index, the longest first;
  // the two last ones go to waves 6 and 7
  const int nsplit = (p.nb > 0) ? p.split : 0;
  cplx q[2][4];
#pragma unroll
  for (int b = 0; b < 2; ++b) {
    int R, C;
    tri_index(w + 2 * b, R, C);
#pragma unroll
    for (int r = 0; r < 4; ++r) q[b][r] = cplx{0.0, 0.0};
    if (16 * R >= wp || (b == 1 && w < 6)) continue;
    for (int sp = 0; sp < nsplit; ++sp)
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        // partial[m = cc][n = r] holds (W^T Z_Bp)[r][cc] for r >= cc
        const cplx e = ld_elem<true>(part + 2 * (int64_t)sp * 64 * 64, (int64_t)(16 * C + lk + 4 * r) * 64 + 16 * R + li);
        q[b][r].re += e.re;
        q[b][r].im += e.im;
      }
  }
#pragma unroll
  for (int u = 0; u < 8; ++u) {
    const int cc = w + 8 * u;
    if (lane == cc) {
      dinv[lane] = lane < wp ? cinv(v[u]) : cplx{0.0, 0.0};
      v[u] = cplx{lane < wp ? 1.0 : 0.0, 0.0};
    }
    x[cc][lane] = dbl2{v[u].re, v[u].im};
  }
  __syncthreads();
#pragma unroll
  for (int b = 0; b < 2; ++b) {
    int R, C;
    tri_index(w + 2 * b, R, C);
    if (16 * R >= wp || (b == 1 && w < 6)) continue;
    dbl4 re{0.0, 0.0, 0.0, 0.0}, im{0.0, 0.0, 0.0, 0.0};
    for (int kb = R; 16 * kb < wp; ++kb)
#pragma unroll
      for (int ks = 0; ks < 4; ++ks) {
        const int k = 16 * kb + ks * 4 + lk;
        const cplx f = cmul(to_cplx(x[16 * C + li][k]), dinv[k]), y = to_cplx(x[16 * R + li][k]);
        re = __builtin_amdgcn_mfma_f64_16x16x4f64(f.re, y.re, re, 0, 0, 0);
        im = __builtin_amdgcn_mfma_f64_16x16x4f64(f.re, y.im, im, 0, 0, 0);
        re = __builtin_amdgcn_mfma_f64_16x16x4f64(f.im, y.im, re, 0, 0, 1);
        im = __builtin_amdgcn_mfma_f64_16x16x4f64(f.im, y.re, im, 0, 0, 0);
      }
#pragma unroll
    for (int r = 0; r < 4; ++r) {
      const int cc = 16 * C + lk + 4 * r, row = 16 * R + li;
      // the diagonal block in global memory is no longer read (Linv and D sit in LDS)
      if (row >= cc && row < wp)
        st_elem<true>(Ls, dbase + (int64_t)cc * p.ld + row, cplx{re[r] - q[b][r].re, im[r] - q[b][r].im});
    }
  }
}

// The whole selected inversion of one panel with at most SMALL_ROWS rows below
// its diagonal block: W = L_Bp Linv, Z_Bp = -Z_BB W and Z_pp in one workgroup
// per shift, Z_BB read through the maps.  A tree of small supernodes (a 1D
// chain: 64 columns, 16 rows below) is bound by the latency of its launches; as
// five launches per level (Z_CC gather, W, Z_Bp, partials, final) it took 5.5 +
// 7.4 + 11.4 + 7.4 + 6.2 us with 8 lanes x 60 shifts, now 9.8 (8 panels x 40
// shifts; 26 with 64 rows below).  Per panel: all loads first (Linv, the first
// blocks of L_Bp and Z_BB), W in LDS, the diagonal product, Z_Bp over Linv's
// place in LDS, the second diagonal product.
//
// ROWS = 16 for panels of at most that many rows: 80 KB of LDS, two workgroups
// per CU.
template <int ROWS, class Src>
__global__ void __launch_bounds__(NT, ROWS <= 16 ? 2 : 1) k_selinv_small(Src src) {
  // all 160 KB of LDS (ROWS = 80): Linv (column, row) with D^{-1} on its
  // diagonal, then Z_Bp (row, column), and W (row, column); 64 slots a line,
  // permuted by the line so that 16 lines are read or written without bank
  // conflicts
  __shared__ dbl2 xs[(ROWS > 64 ? ROWS : 64) * 64], wl[ROWS * 64];
  auto at = [](int line, int q) { return line * 64 + (q ^ (line & 15)); };
  Common c;
  PanelK p;
  int bx, by;
  locate(src, c, p, bx, by, false);
  const int sh = p.sh0 + by;
  double* Ls = shift_base<true>(c, sh);
  const int wp = p.wp, nb = p.nb;
  const int lane = threadIdx.x & 63, li = lane & 15, lk = lane >> 4;
  const int w = wave_id();
  const int64_t dbase = p.off + (int64_t)p.p0 * p.ld + p.p0;
  const int64_t rbase = dbase + wp;
  const int base = p.p0 + wp;
  const int64_t* cmap = c.colmap + p.cm;
  const int64_t* cseg = c.colseg + p.cm;
  const int mbs = (wp + 15) / 16, nbs = (nb + 15) / 16;
  cplx v[16];
#pragma unroll
  for (int u = 0; u < 16; ++u) {
    const int cc = w + 4 * u;
    v[u] = cplx{0.0, 0.0};
    if (lane >= cc && lane < wp) v[u] = ld_elem<true>(Ls, dbase + (int64_t)cc * p.ld + lane);
  }
  // operand blocks of the rows 16 n..: L_Bp[i][k] (k < wp) and Z(k, i) (k < nb)
  auto load_l = [&](int n, cplx (&f)[16]) {
    const int i = 16 * n + li;
#pragma unroll
    for (int ks = 0; ks < 16; ++ks) {
      const int k = 4 * ks + lk;
      f[ks] = cplx{0.0, 0.0};
      if (i < nb && k < wp) f[ks] = ld_elem<true>(Ls, rbase + (int64_t)k * p.ld + i);
    }
  };
  constexpr int ZK = ROWS / 4;
  auto load_z = [&](int n, cplx (&f)[ZK]) {
    const int i = 16 * n + li;
    int64_t e[ZK];
#pragma unroll
    for (int ks = 0; ks < ZK; ++ks) {
      // branch-free over the maps: indices clamped into the row list
      const int k = 4 * ks + lk;
      const int q0 = base + min(i, nb - 1), q1 = base + min(k, nb - 1);
      const int lo = min(q0, q1), hi = max(q0, q1);
      e[ks] = lo < p.w ? p.off + (int64_t)lo * p.ld + hi : cmap[lo] + c.relpos[cseg[lo] + hi];
    }
#pragma unroll
    for (int ks = 0; ks < ZK; ++ks) {
      f[ks] = cplx{0.0, 0.0};
      if (i < nb && 4 * ks + lk < nb) f[ks] = ld_elem<true>(Ls, e[ks]);
    }
  };
  auto mac = [&](dbl4& re, dbl4& im, cplx a, cplx b) {
    re = __builtin_amdgcn_mfma_f64_16x16x4f64(a.re, b.re, re, 0, 0, 0);
    im = __builtin_amdgcn_mfma_f64_16x16x4f64(a.re, b.im, im, 0, 0, 0);
    re = __builtin_amdgcn_mfma_f64_16x16x4f64(a.im, b.im, re, 0, 0, 1);
    im = __builtin_amdgcn_mfma_f64_16x16x4f64(a.im, b.re, im, 0, 0, 0);
  };
  // the wave's block pairs (row block n, column block m): w, w + 4, ... of n mbs + m
  cplx f[16], z[ZK];
  if (w < mbs * nbs) {
    load_l(w / mbs, f);
    load_z(w / mbs, z);
  }
#pragma unroll
  for (int u = 0; u < 16; ++u) {
    const int cc = w + 4 * u;
    if (lane == cc && lane < wp) v[u] = cinv(v[u]);
    xs[at(cc, lane)] = dbl2{v[u].re, v[u].im};
  }
  __syncthreads();
  auto X = [&](int col, int row) {   // Linv[row][col] for row >= col - 15
    const cplx e = to_cplx(xs[at(col, row)]);
    return row == col ? cplx{col < wp ? 1.0 : 0.0, 0.0} : e;
  };
  // W[i][c] = sum_{k >= c} Linv[k][c] L[i][k]
  for (int q = w; q < mbs * nbs; q += 4) {
    const int n = q / mbs, m = q - n * mbs;
    if (q != w) load_l(n, f);
    dbl4 re{0.0, 0.0, 0.0, 0.0}, im{0.0, 0.0, 0.0, 0.0};
#pragma unroll
    for (int ks = 0; ks < 16; ++ks)
      if (ks / 4 >= m && ks / 4 < mbs) mac(re, im, X(16 * m + li, 4 * ks + lk), f[ks]);
#pragma unroll
    for (int r = 0; r < 4; ++r) wl[at(16 * n + li, 16 * m + lk + 4 * r)] = dbl2{re[r], im[r]};
  }
  // Z_pp's first term, the wave's blocks R >= C
  dbl4 re[3], im[3];
#pragma unroll
  for (int b = 0; b < 3; ++b) {
    int R, C;
    tri_index(w + 4 * b, R, C);
    re[b] = im[b] = dbl4{0.0, 0.0, 0.0, 0.0};
    for (int kb = R; kb < mbs && R < 4; ++kb)
#pragma unroll
      for (int ks = 0; ks < 4; ++ks) {
        const int k = 16 * kb + ks * 4 + lk;
        mac(re[b], im[b], cmul(X(16 * C + li, k), to_cplx(xs[at(k, k)])), X(16 * R + li, k));
      }
  }
  __syncthreads();
  // Z_Bp[i][c] = -sum_k W[k][c] Z(k, i)
  for (int q = w; q < mbs * nbs; q += 4) {
    const int n = q / mbs, m = q - n * mbs;
    if (q != w) load_z(n, z);
    dbl4 zr{0.0, 0.0, 0.0, 0.0}, zi{0.0, 0.0, 0.0, 0.0};
#pragma unroll
    for (int ks = 0; ks < ZK; ++ks)
      if (ks / 4 < nbs) mac(zr, zi, to_cplx(wl[at(4 * ks + lk, 16 * m + li)]), z[ks]);
#pragma unroll
    for (int r = 0; r < 4; ++r) {
      const int cc = 16 * m + lk + 4 * r, i = 16 * n + li;
      xs[at(i, cc)] = dbl2{-zr[r], -zi[r]};
      if (cc < wp && i < nb) st_elem<true>(Ls, rbase + (int64_t)cc * p.ld + i, cplx{-zr[r], -zi[r]});
    }
  }
  __syncthreads();
  // Z_pp[r][c] -= sum_k W[k][r] Z_Bp[k][c]
#pragma unroll
  for (int b = 0; b < 3; ++b) {
    int R, C;
    tri_index(w + 4 * b, R, C);
    if (R >= mbs) continue;
    dbl4 sr{0.0, 0.0, 0.0, 0.0}, si{0.0, 0.0, 0.0, 0.0};
    for (int k = lk; k < 16 * nbs; k += 4) mac(sr, si, to_cplx(xs[at(k, 16 * C + li)]), to_cplx(wl[at(k, 16 * R + li)]));
#pragma unroll
    for (int r = 0; r < 4; ++r) {
      const int cc = 16 * C + lk + 4 * r, row = 16 * R + li;
      if (row >= cc && row < wp)
        st_elem<true>(Ls, dbase + (int64_t)cc * p.ld + row, cplx{re[b][r] - sr[r], im[b][r] - si[r]});
    }
  }
}

// --------------------------------------------------------------------------
// pole sums, extraction
// --------------------------------------------------------------------------
// out[g][k] = sum_l Im(omega_{g,l} Z_l[k]); per-block partial traces.
constexpr int PS = 8;
__global__ void __launch_bounds__(NT) k_pole_sum(const double* __restrict__ L, int64_t stride,
                                                 int nshift, const double* __restrict__ wts,
                                                 int nsets, const int64_t* __restrict__ eoff,
                                                 const int32_t* __restrict__ ediag, int64_t nnz,
                                                 const double* __restrict__ H,
                                                 const double* __restrict__ S, double* out,
                                                 double* partial, int accumulate) {
  __shared__ double red[8][NT];
  double tr[8];
  for (int q = 0; q < 8; ++q) tr[q] = 0.0;
  for (int64_t k = (int64_t)blockIdx.x * NT + threadIdx.x; k < nnz; k += (int64_t)gridDim.x * NT) {
    const int64_t e = eoff[k];
    double acc[4] = {0.0, 0.0, 0.0, 0.0};
    // PS poles' values in flight (one at a time, a small system's sum took 40
    // dependent loads: 23 us for 2,640 entries)
    for (int l0 = 0; l0 < nshift; l0 += PS) {
      double2 z[PS];
#pragma unroll
      for (int i = 0; i < PS; ++i)
        z[i] = *reinterpret_cast<const double2*>(L + 2 * (stride * min(l0 + i, nshift - 1) + e));
#pragma unroll
      for (int i = 0; i < PS; ++i) {
        const int l = l0 + i;
        if (l >= nshift) break;
#pragma unroll
        for (int g = 0; g < 4; ++g) {
          if (g >= nsets) break;
          const double wr = wts[2 * (g * nshift + l)], wi = wts[2 * (g * nshift + l) + 1];
          acc[g] += wr * z[i].y + wi * z[i].x;
        }
      }
    }
    const double mult = ediag[k] == 1 ? 1.0 : 2.0;
    for (int g = 0; g < nsets; ++g) {
      // accumulate: add to the sums of earlier pole chunks (traces stay per chunk)
      out[(int64_t)g * nnz + k] = accumulate ? out[(int64_t)g * nnz + k] + acc[g] : acc[g];
      tr[2 * g] += mult * acc[g] * S[k];
      tr[2 * g + 1] += mult * acc[g] * H[k];
    }
  }
  for (int q = 0; q < 8; ++q) red[q][threadIdx.x] = tr[q];
  __syncthreads();
  for (int s2 = NT / 2; s2 > 0; s2 >>= 1) {
    if (threadIdx.x < s2)
      for (int q = 0; q < 8; ++q) red[q][threadIdx.x] += red[q][threadIdx.x + s2];
    __syncthreads();
  }
  if (threadIdx.x < 8) partial[8 * blockIdx.x + threadIdx.x] = red[threadIdx.x][0];
}

// The 8 sums over nb blocks' partials, one wave each: 64 strided sums, then
// halves in a fixed order.  (One thread per sum over 1024 partials took 153 us.)
__global__ void k_sum_partials(const double* partial, int nb, double* out) {
  const int q = threadIdx.x >> 6, lane = threadIdx.x & 63;
  double s = 0.0;
  for (int b = lane; b < nb; b += 64) s += partial[8 * b + q];
  for (int h = 32; h > 0; h >>= 1) s += __shfl_down(s, h);
  if (lane == 0) out[q] = s;
}

__global__ void k_gather(const double* __restrict__ L, const int64_t* __restrict__ eoff,
                         int64_t nnz, double2* out) {
  for (int64_t k = (int64_t)blockIdx.x * NT + threadIdx.x; k < nnz; k += (int64_t)gridDim.x * NT)
    out[k] = *reinterpret_cast<const double2*>(L + 2 * eoff[k]);
}

__global__ void k_get_diag(const double* __restrict__ L, const int64_t* __restrict__ diagoff, int n,
                           int cplx_elems, double2* out) {
  // diagoff[j] = element offset of the diagonal entry of new column j
  const int j = blockIdx.x * NT + threadIdx.x;
  if (j < n) {
    const int64_t e = diagoff[j];
    out[j] = cplx_elems ? *reinterpret_cast<const double2*>(L + 2 * e) : make_double2(L[e], 0.0);
  }
}

// --------------------------------------------------------------------------
// host orchestration
// --------------------------------------------------------------------------
namespace {

// Event pairs around the launches of one kernel class (benchmarks only).
struct Profiler {
  int kernel = KC_NONE;
  std::vector<hipEvent_t> ev;   // pool, reused across profiles
  size_t used = 0;
  int64_t launches = 0;
  double work = 0.0;    // algorithmic flops on the exact structure of L (bytes for the memory-bound classes)
  double bytes = 0.0;   // algorithmic HBM bytes: operands read once, results written once
  double stored = 0.0;  // flops on the stored (relaxed supernodal) structure
  int failed = 0;       // HIP error of an event create/record inside the profile, 0 if none
};
Profiler g_prof;

struct ProfScope {
  hipStream_t st;
  bool on;
  double w_, b_, s_;
  // work: exact algorithmic flops (bytes for the memory-bound classes);
  // stored: flops on the stored structure
  ProfScope(int kernel, hipStream_t s, double work, double bytes, double stored)
      : st(s), on(g_prof.kernel == kernel && kernel != KC_NONE), w_(work), b_(bytes), s_(stored) {
    if (!on) return;
    hipStreamCaptureStatus cs = hipStreamCaptureStatusNone;
    if (hipStreamIsCapturing(st, &cs) != hipSuccess || cs != hipStreamCaptureStatusNone) {
      on = false;   // no event nodes inside captured graphs
      return;
    }
    while (g_prof.ev.size() < g_prof.used + 2) {
      hipEvent_t e;
      const hipError_t ce = hipEventCreate(&e);
      if (ce != hipSuccess) { on = false; g_prof.failed = (int)ce; return; }
      g_prof.ev.push_back(e);
    }
    const hipError_t re = hipEventRecord(g_prof.ev[g_prof.used], st);
    if (re != hipSuccess) { on = false; g_prof.failed = (int)re; }
  }
  ~ProfScope() {
    if (!on) return;
    // a launch counts only with both of its events recorded
    const hipError_t re = hipEventRecord(g_prof.ev[g_prof.used + 1], st);
    if (re != hipSuccess) {
      g_prof.failed = (int)re;
      return;
    }
    g_prof.used += 2;
    g_prof.launches += 1;
    g_prof.work += w_;
    g_prof.bytes += b_;
    g_prof.stored += s_;
  }
};

inline int blocks_for(int64_t n, int cap) {
  int64_t b = (n + NT - 1) / NT;
  if (b < 1) b = 1;
  if (b > cap) b = cap;
  return (int)b;
}

PanelK panel_args(const Symbolic& S, const Panel& P) {
  PanelK k;
  k.off = S.off[P.J];
  k.cm = S.rowptr[P.J];
  k.ld = S.ld[P.J];
  k.p0 = P.p0;
  k.wp = P.wp;
  k.nb = P.nb_rows;
  k.col0 = S.sfirst[P.J] + P.p0;
  k.split = split_count(P.nb_rows);
  k.w = S.sfirst[P.J + 1] - S.sfirst[P.J];
  k.c = S.ld[P.J] - k.w;
  k.sh0 = 0;
  return k;
}

}  // namespace

Common make_common(const Symbolic& S, void* L, void* work) {
  Common c;
  c.L = (double*)L;
  c.stride = S.nnzL_store;
  const char* m = (const char*)S.dmaps;
  c.colmap = (const int64_t*)(m + S.o_colmap);
  c.colseg = (const int64_t*)(m + S.o_colseg);
  c.relpos = (const int32_t*)(m + S.o_relpos);
  c.work = (double*)work;
  c.wps = S.work_per_shift;
  c.wfix = S.work_fixed;
  char* w = (char*)work;
  c.absmax = (const double*)(w + WK_ABSMAX);
  c.shifts = (const double*)(w + WK_SHIFTS);
  c.info = (int64_t*)(w + WK_INFO);
  c.negc = (int64_t*)(w + WK_NEGC);
  c.pivtol = S.pivot_tol;
  c.G = nullptr;
  c.gstride = S.gather_per_shift / 8;
  c.ut = 0;
  return c;
}

// Tile width of a panel product: of 64, 32 and 16 columns the one
// whose rounds over the compute units take least time.  tiles(tn) is the
// number of workgroups at width tn.  A round of narrower tiles is shorter in
// proportion, but the operand loads weigh more: 69.0, 68.1 and 60.7 TFLOP/s
// on a full launch (4096 rows x 32 shifts), hence the rates.  At 884 rows x
// 60 shifts (4, 7 and 14 rounds) 54.4, 59.9 and 53.6 TFLOP/s, at 452 x 40 (2,
// 3, 5 rounds) 33.3, 43.4 and 47.8, at 130 x 40 (1, 1, 2) 13.7, 22.6 and 22.2.
//
// m: rows of the product (the panel's width): with b of its four 16-row blocks
// live a wave multiplies b blocks per 16 columns on 64-column tiles, (b + 1) / 2
// on 32- and one on 16-column ones (with_layout).
//
// The rates and rounds are those of a launch alone on the device.  On one stream
// the rule is worth 4.8% of a call (a sheet of N = 2,106 x 60 in a graph plan
// 22.27 ms with 64 columns throughout, 21.25 with the rule); in eager calls of
// large trees the subtree streams fill each other's last rounds and it makes no
// difference (64 columns throughout against the rule: sheets of N = 7,956 x 60
// 210.2 and 210.6 ms, N = 26,624 x 40 1016 and 1021, bulk of N = 7,488 x 40 548.9
// and 548.0; two runs of one side differ by 0.2 to 0.5%).
constexpr int NCU = 256;
template <class F>
int pick_tile(int m, F tiles) {
  const int b = std::min(4, (m + 15) / 16);
  const int width[3] = {64, 32, 16};
  const int work[3] = {b, (b + 1) / 2, 1};
  const double rate[3] = {1.0, 0.985, 0.88};
  int best = 64;
  double cost = 0.0;
  for (int q = 0; q < 3; ++q) {
    const int64_t rounds = ((int64_t)tiles(width[q]) + NCU - 1) / NCU;
    const double t = (double)rounds * work[q] / rate[q];
    if (q == 0 || t < cost) {
      best = width[q];
      cost = t;
    }
  }
  return best;
}
inline int tiles_of(int rows, int tn) { return (rows + tn - 1) / tn; }
// tiles of an ancestor update: 64 columns by tn rows, those in the lower part
inline int64_t update_tiles(int below, int tn) {
  int64_t n = 0;
  for (int j0 = 0; j0 < below; j0 += TM) n += tiles_of(below, tn) - j0 / tn;
  return n;
}

// f(std::integral_constant<int, tn>) for a width of pick_tile
template <class F>
void with_tile(int tn, F f) {
  if (tn == 16) f(std::integral_constant<int, 16>());
  else if (tn == 32) f(std::integral_constant<int, 32>());
  else f(std::integral_constant<int, 64>());
}
#define PXS_CHECK_LAUNCH()                         \
  do {                                             \
    hipError_t e_ = hipGetLastError();             \
    if (e_ != hipSuccess) return (int)e_;          \
  } while (0)

int profile_begin(int kernel) {
  g_prof.kernel = kernel;
  g_prof.used = 0;
  g_prof.launches = 0;
  g_prof.work = 0.0;
  g_prof.bytes = 0.0;
  g_prof.stored = 0.0;
  g_prof.failed = 0;
  return 0;
}

int profile_end(double* ms, int64_t* launches, double* work, double* bytes, double* stored) {
  if (g_prof.kernel == KC_NONE) return -1;   // no profile open
  if (g_prof.failed) {                        // totals would be partial
    const int f = g_prof.failed;
    g_prof.kernel = KC_NONE;
    g_prof.used = 0;
    return f;
  }
  double tot = 0.0;
  for (size_t i = 0; i + 1 < g_prof.used; i += 2) {
    hipError_t e = hipEventSynchronize(g_prof.ev[i + 1]);
    if (e != hipSuccess) return (int)e;
    float t = 0.0f;
    e = hipEventElapsedTime(&t, g_prof.ev[i], g_prof.ev[i + 1]);
    if (e != hipSuccess) return (int)e;
    tot += t;
  }
  *ms = tot;
  *launches = g_prof.launches;
  *work = g_prof.work;
  *bytes = g_prof.bytes;
  *stored = g_prof.stored;
  g_prof.kernel = KC_NONE;
  g_prof.used = 0;
  return 0;
}

int upload_shifts(int nshift, const double* shifts_host, void* work, hipStream_t st) {
  hipError_t e = hipMemcpyAsync((char*)work + WK_SHIFTS, shifts_host, sizeof(double) * 2 * nshift,
                                hipMemcpyHostToDevice, st);
  return (int)e;
}

int upload_shifts_device(int nshift, const double* shifts_dev, void* work, hipStream_t st) {
  return (int)hipMemcpyAsync((char*)work + WK_SHIFTS, shifts_dev, sizeof(double) * 2 * nshift,
                             hipMemcpyDeviceToDevice, st);
}

int upload_weights_device(int nshift, int nsets, const double* weights_dev, void* work, hipStream_t st) {
  return (int)hipMemcpyAsync((char*)work + WK_WEIGHTS, weights_dev, sizeof(double) * 2 * nsets * nshift,
                             hipMemcpyDeviceToDevice, st);
}

int upload_weights(int nshift, int nsets, const double* weights_host, void* work, hipStream_t st) {
  hipError_t e = hipMemcpyAsync((char*)work + WK_WEIGHTS, weights_host,
                                sizeof(double) * 2 * nsets * nshift, hipMemcpyHostToDevice, st);
  return (int)e;
}

template <bool CPLX>
int run_factor(const Symbolic& S, const double* H, const double* Sv, int nshift,
               const double* shifts_host, void* L, void* work, hipStream_t st, bool inorder) {
  int e = upload_shifts(nshift, shifts_host, work, st);
  if (e != 0) return e;
  return run_factor_kernels<CPLX>(S, H, Sv, nshift, L, work, st, inorder);
}

// Streams and events owned by the library for the subtree-parallel
// factorization and SelInv (created on first use on the current device,
// kept for the process).
struct StreamPool {
  int device = -1;
  std::vector<hipStream_t> streams;
  std::vector<hipEvent_t> events;
};
StreamPool g_pool;

int ensure_pool(int nstreams, int nevents) {
  int dev = 0;
  hipError_t e = hipGetDevice(&dev);
  if (e != hipSuccess) return (int)e;
  if (g_pool.device != dev) {
    g_pool.streams.clear();   // streams of another device are left alone
    g_pool.events.clear();
    g_pool.device = dev;
  }
  while ((int)g_pool.streams.size() < nstreams) {
    hipStream_t s;
    e = hipStreamCreateWithFlags(&s, hipStreamNonBlocking);
    if (e != hipSuccess) return (int)e;
    g_pool.streams.push_back(s);
  }
  while ((int)g_pool.events.size() < nevents) {
    hipEvent_t ev;
    e = hipEventCreateWithFlags(&ev, hipEventDisableTiming);
    if (e != hipSuccess) return (int)e;
    g_pool.events.push_back(ev);
  }
  return 0;
}

// Before the factorization: pivot flags and counts cleared, max|H|, max|S|
// for the pivot threshold, the factor storage zeroed and every shift's
// H - w_l S assembled into it.
template <bool CPLX>
int factor_prologue(const Symbolic& S, const double* H, const double* Sv, int nshift, void* L, void* work,
                    hipStream_t st) {
  char* w = (char*)work;
  hipLaunchKernelGGL(k_zero_i64, dim3((2 * MAX_SHIFTS + NT - 1) / NT), dim3(NT), 0, st,
                     (int64_t*)(w + WK_INFO), 2 * MAX_SHIFTS);
  PXS_CHECK_LAUNCH();
  const char* m = (const char*)S.dmaps;
  const int64_t* eoff = (const int64_t*)(m + S.o_entry_off);
  const int nbm = blocks_for(S.nnz_lower, ABSMAX_BLOCKS);
  hipLaunchKernelGGL(k_absmax_partial, dim3(nbm), dim3(NT), 0, st, H, Sv, S.nnz_lower,
                     (double*)(w + WK_ABSMAX_PART));
  hipLaunchKernelGGL(k_absmax_final, dim3(1), dim3(128), 0, st, (const double*)(w + WK_ABSMAX_PART),
                     nbm, (double*)(w + WK_ABSMAX));
  PXS_CHECK_LAUNCH();
  const int64_t total_d = (CPLX ? 2 : 1) * S.nnzL_store * (int64_t)nshift;   // doubles
  hipLaunchKernelGGL(k_fill_zero, dim3(blocks_for(total_d / 2, FILL_BLOCKS)), dim3(NT), 0, st, (double*)L, total_d);
  PXS_CHECK_LAUNCH();
  {
    // bytes: H, S, offsets read once per shift block; one element written per entry and shift
    const double ab = (double)S.nnz_lower * (24.0 + (CPLX ? 16.0 : 8.0) * nshift);
    ProfScope ps(KC_ASSEMBLE, st, ab, ab, ab);
    hipLaunchKernelGGL(k_assemble<CPLX>, dim3(blocks_for(S.nnz_lower, 2048), nshift), dim3(NT), 0, st,
                       (double*)L, S.nnzL_store, H, Sv, eoff, S.nnz_lower, (const double*)(w + WK_SHIFTS));
  }
  PXS_CHECK_LAUNCH();
  return 0;
}

// launch(group, grid) with a fused launch's items (nsh shifts each) in the
// shortest form that holds them; false without items.  A grid dimension holds
// fewer than 2^32 threads: more workgroups than GROUP_BLOCKS go as several
// launches (the items are independent), a single panel as tiles x shifts.
constexpr int64_t GROUP_BLOCKS = 1 << 22;
template <class F>
static bool with_group(const Common& c, const std::vector<LaneItem>& items, int nsh, F launch) {
  int64_t total = 0;
  for (const LaneItem& it : items) total += (int64_t)it.tiles * nsh;
  if (items.empty()) return false;
  if (items.size() > 1 && total > GROUP_BLOCKS) {
    const auto mid = items.begin() + items.size() / 2;
    return with_group(c, std::vector<LaneItem>(items.begin(), mid), nsh, launch) &&
           with_group(c, std::vector<LaneItem>(mid, items.end()), nsh, launch);
  }
  auto fill = [&](auto& g) {
    constexpr int N = sizeof(g.start) / sizeof(g.start[0]);
    g.c = c;
    int64_t at = 0;
    for (int q = 0; q < N; ++q) {
      g.start[q] = INT32_MAX;
      if (q >= (int)items.size()) continue;
      g.start[q] = (int32_t)at;
      g.it[q] = items[q];
      g.it[q].nsh = nsh;
      at += (int64_t)items[q].tiles * nsh;
    }
  };
  if (items.size() == 1) {
    OnePanel o{c, items[0].p};
    o.c.wfix = items[0].wfix;
    o.c.G = items[0].G;
    o.c.gstride = items[0].gstride;
    launch(o, dim3((unsigned)items[0].tiles, (unsigned)nsh));
  } else if (items.size() <= FEW_ITEMS) {
    LaneGroup<FEW_ITEMS> g;
    fill(g);
    launch(g, dim3((unsigned)total));
  } else {
    LaneGroup<MAX_ITEMS> g;
    fill(g);
    launch(g, dim3((unsigned)total));
  }
  return true;
}

template <bool CPLX>
int run_factor_kernels(const Symbolic& S, const double* H, const double* Sv, int nshift, void* L,
                       void* work, hipStream_t st, bool inorder) {
  {
    const int e = factor_prologue<CPLX>(S, H, Sv, nshift, L, work, st);
    if (e) return e;
  }
  Common c = make_common(S, L, work);
  const double fm = CPLX ? 8.0 : 2.0;   // flops per multiply-add
  const double eb = CPLX ? 16.0 : 8.0;  // bytes per element
  // tile width of a product over `rows` rows
  auto tile = [&](int rows, int m) {
    return pick_tile(m, [&](int tn) { return (int64_t)tiles_of(rows, tn) * nshift; });
  };
  // the panel work of one panel: left-looking update from the earlier
  // columns of its supernode, LDL^T of the diagonal block, the rows below
  auto panel_work = [&](const Panel& P, hipStream_t s) -> int {
    PanelK k = panel_args(S, P);
    const PanelMacs& xm = S.xm_panel[&P - S.panels.data()];
    if (k.p0 > 0) {
      const int nrows = k.ld - k.p0;
      ProfScope ps(KC_UPDATE, s, fm * nshift * xm.intu, eb * nshift * ((double)nrows * k.p0 + 2.0 * nrows * k.wp),
                   fm * nshift * ((double)nrows * k.wp - 0.5 * k.wp * (k.wp - 1)) * k.p0);
      with_tile(tile(nrows, k.wp), [&](auto t) {
        constexpr int TN = decltype(t)::value;
        hipLaunchKernelGGL((k_int_update<CPLX, TN, OnePanel>), dim3(tiles_of(nrows, TN), nshift), dim3(NT), 0, s,
                           OnePanel{c, k});
      });
    }
    {
      const double rows = k.nb <= SMALL_ROWS ? k.nb : 0.0;   // rows below done along
      ProfScope ps(KC_DIAG, s, fm * nshift * (xm.diag + (rows > 0.0 ? xm.trsm : 0.0)),
                   eb * nshift * ((double)k.wp * (k.wp + 1) + 2.0 * rows * k.wp),
                   fm * nshift * ((double)k.wp * k.wp * k.wp / 3.0 + rows * k.wp * (k.wp + 1) / 2.0));
      hipLaunchKernelGGL((k_diag<CPLX, OnePanel>), dim3(1, nshift), dim3(NTD), 0, s, OnePanel{c, k});
    }
    if (k.nb > SMALL_ROWS) {
      ProfScope ps(KC_TRSM, s, fm * nshift * xm.trsm, eb * nshift * (2.0 * k.nb * k.wp + 0.5 * k.wp * (k.wp + 1)),
                   fm * nshift * (double)k.nb * k.wp * (k.wp + 1) / 2.0);
      with_tile(tile(k.nb, k.wp), [&](auto t) {
        constexpr int TN = decltype(t)::value;
        hipLaunchKernelGGL((k_trsm<CPLX, TN, OnePanel>), dim3(tiles_of(k.nb, TN), nshift), dim3(NT), 0, s, OnePanel{c, k});
      });
    }
    PXS_CHECK_LAUNCH();
    return 0;
  };
  // right-looking: the whole supernode J updates its ancestors once (K = w),
  // scattered into their panels; J's last panel describes its row list
  auto scatter = [&](const Panel& P, hipStream_t s) -> int {
    const int32_t w = S.sfirst[P.J + 1] - S.sfirst[P.J];
    const int32_t below = S.ld[P.J] - w;
    if (below <= 0) return 0;
    PanelK u = panel_args(S, P);
    u.p0 = 0;
    u.wp = w;
    u.nb = below;
    const int tn = pick_tile(below, [&](int q) { return update_tiles(below, q) * nshift; });
    ProfScope ps(KC_UPDATE, s, fm * nshift * S.xm_update[P.J],
                 eb * nshift * ((double)below * w + (double)below * (below + 1)),
                 fm * nshift * (double)below * (below + 1) / 2.0 * w);
    with_tile(tn, [&](auto t) {
      constexpr int TN = decltype(t)::value;
      hipLaunchKernelGGL((k_update<CPLX, TN, OnePanel>), dim3(tiles_of(below, TM) * tiles_of(below, TN), nshift), dim3(NT), 0,
                         s, OnePanel{c, u});
    });
    PXS_CHECK_LAUNCH();
    return 0;
  };
  const size_t np = S.panels.size();
  const int ns = S.nsuper;
  const int NS = S.sel_nstreams;
  if ((int)S.fac_order.size() != ns || (int)S.fac_child.size() != ns) return (int)hipErrorInvalidValue;
  std::vector<int> pfirst(ns, -1), plast(ns, -1);
  for (size_t ip = 0; ip < np; ++ip) {
    const int J = S.panels[ip].J;
    if (pfirst[J] < 0) pfirst[J] = (int)ip;
    plast[J] = (int)ip;
  }
  // Supernodes are issued in fac_order on every path, so each entry receives
  // its scatters in the same order and the factors are bit-identical whether
  // the subtree streams are used or not.  Inside a stream capture, or with
  // one subtree stream, everything runs on the caller's stream.
  int err = 0;
  hipStreamCaptureStatus cap = hipStreamCaptureStatusNone;
  hipError_t he = hipStreamIsCapturing(st, &cap);
  if (he != hipSuccess) return (int)he;
  // Where the caller's stream is the only one, large trees run fused as well
  // (panel by panel a sheet of N=7956 x 60 shifts replays in 215 ms, fused in
  // 207.5); with the subtree streams they do not (208.8 ms against 211.1).
  const bool one_stream = cap != hipStreamCaptureStatusNone || inorder;
  if (NS > 1 && (S.fused_lanes || (S.fuse_one_stream && one_stream))) {
    // Fused launches (no library streams or events, so also on the in-order
    // paths): a launch takes the next panel operation of up to MAX_ITEMS
    // supernodes, of the kind that most of them wait for; a supernode is ready
    // once every scatter into it was in an earlier launch.  When no panel
    // operation is ready, one launch takes the scatters of finished supernodes
    // that share no target supernode with each other or with an earlier one
    // (in fac_order) that has not been scattered, so every entry receives its
    // scatters in the same order as on the other paths.  (One launch per
    // scatter and one lane per subtree stream took 52 launches of panel work
    // and scatters for a chain of 31 supernodes.)
    enum : int32_t { FK_INT, FK_DIAG, FK_TRSM, FK_UPD, FK_KINDS };
    struct FOp {
      int32_t kind;
      int32_t rows;   // rows of the product (its tiles follow from the launch's tile width)
      PanelK p;
      double work, bytes, stored;
    };
    if ((int)S.tgt_ptr.size() != ns + 1) return (int)hipErrorInvalidValue;
    std::vector<std::vector<FOp>> ops(ns);
    std::vector<int32_t> order;   // supernodes with panels, in fac_order
    std::vector<int32_t> need(ns, 0);   // scatters into J still to come
    for (int J : S.fac_order) {
      if (pfirst[J] < 0) continue;
      order.push_back(J);
      for (int64_t t = S.tgt_ptr[J]; t < S.tgt_ptr[J + 1]; ++t) ++need[S.tgt[t]];
      for (int ip = pfirst[J]; ip <= plast[J]; ++ip) {
        const PanelK k = panel_args(S, S.panels[ip]);
        const PanelMacs& xm = S.xm_panel[ip];
        if (k.p0 > 0) {
          const int nrows = k.ld - k.p0;
          ops[J].push_back(FOp{FK_INT, nrows, k, fm * nshift * xm.intu,
                               eb * nshift * ((double)nrows * k.p0 + 2.0 * nrows * k.wp),
                               fm * nshift * ((double)nrows * k.wp - 0.5 * k.wp * (k.wp - 1)) * k.p0});
        }
        const double rows = k.nb <= SMALL_ROWS ? k.nb : 0.0;   // rows below done along
        ops[J].push_back(FOp{FK_DIAG, 0, k, fm * nshift * (xm.diag + (rows > 0.0 ? xm.trsm : 0.0)),
                             eb * nshift * ((double)k.wp * (k.wp + 1) + 2.0 * rows * k.wp),
                             fm * nshift * ((double)k.wp * k.wp * k.wp / 3.0 + rows * k.wp * (k.wp + 1) / 2.0)});
        if (k.nb > SMALL_ROWS)
          ops[J].push_back(FOp{FK_TRSM, k.nb, k, fm * nshift * xm.trsm,
                               eb * nshift * (2.0 * k.nb * k.wp + 0.5 * k.wp * (k.wp + 1)),
                               fm * nshift * (double)k.nb * k.wp * (k.wp + 1) / 2.0});
      }
    }
    std::vector<size_t> pos(ns, 0);
    std::vector<uint8_t> scattered(ns, 0);
    std::vector<int64_t> mark(ns, -1);   // the launch whose scatters already claim this target
    size_t first = 0;                    // order[0 .. first) is finished
    int64_t nl = 0;
    std::vector<int32_t> take;
    std::vector<LaneItem> items;
    bool ok = true;
    for (;; ++nl) {
      while (first < order.size() && scattered[order[first]]) ++first;
      if (first == order.size()) break;
      int cnt[FK_KINDS] = {0, 0, 0, 0};
      for (size_t i = first; i < order.size(); ++i) {
        const int J = order[i];
        if (need[J] == 0 && pos[J] < ops[J].size()) ++cnt[ops[J][pos[J]].kind];
      }
      const int kind = (int)(std::max_element(cnt, cnt + FK_UPD) - cnt);
      take.clear();
      items.clear();
      int m = 0;
      double w = 0.0, b = 0.0, s = 0.0;
      if (cnt[kind] > 0) {
        for (size_t i = first; i < order.size() && (int)take.size() < MAX_ITEMS; ++i) {
          const int J = order[i];
          if (need[J] != 0 || pos[J] >= ops[J].size() || ops[J][pos[J]].kind != kind) continue;
          take.push_back(J);
          m = std::max(m, ops[J][pos[J]].p.wp);
        }
        auto rows = [&](int J) { return ops[J][pos[J]].rows; };
        const int tn = pick_tile(m, [&](int tq) {
          int64_t n = 0;
          for (int J : take) n += (int64_t)tiles_of(rows(J), tq) * nshift;
          return n;
        });
        for (size_t q = 0; q < take.size(); ++q) {
          const int J = take[q];
          const FOp& o = ops[J][pos[J]];
          items.push_back(LaneItem{o.p, c.wfix, c.G, c.gstride, kind == FK_DIAG ? 1 : tiles_of(o.rows, tn), 0});
          w += o.work;
          b += o.bytes;
          s += o.stored;
          // a root has no scatter: it is finished with its last operation
          if (++pos[J] == ops[J].size() && S.tgt_ptr[J] == S.tgt_ptr[J + 1]) scattered[J] = 1;
        }
        if (kind == FK_INT) {
          ProfScope ps(KC_UPDATE, st, w, b, s);
          with_tile(tn, [&](auto t) {
            constexpr int TN = decltype(t)::value;
            ok = with_group(c, items, nshift, [&](const auto& g, dim3 grid) {
              hipLaunchKernelGGL((k_int_update<CPLX, TN, std::decay_t<decltype(g)>>), grid, dim3(NT), 0, st, g);
            });
          });
        } else if (kind == FK_DIAG) {
          ProfScope ps(KC_DIAG, st, w, b, s);
          ok = with_group(c, items, nshift, [&](const auto& g, dim3 grid) {
            hipLaunchKernelGGL((k_diag<CPLX, std::decay_t<decltype(g)>>), grid, dim3(NTD), 0, st, g);
          });
        } else {
          ProfScope ps(KC_TRSM, st, w, b, s);
          with_tile(tn, [&](auto t) {
            constexpr int TN = decltype(t)::value;
            ok = with_group(c, items, nshift, [&](const auto& g, dim3 grid) {
              hipLaunchKernelGGL((k_trsm<CPLX, TN, std::decay_t<decltype(g)>>), grid, dim3(NT), 0, st, g);
            });
          });
        }
      } else {
        for (size_t i = first; i < order.size() && (int)take.size() < MAX_ITEMS; ++i) {
          const int J = order[i];
          if (scattered[J]) continue;
          bool may = need[J] == 0 && pos[J] == ops[J].size();
          for (int64_t t = S.tgt_ptr[J]; t < S.tgt_ptr[J + 1]; ++t) {
            may = may && mark[S.tgt[t]] != nl;
            mark[S.tgt[t]] = nl;
          }
          if (may) take.push_back(J);
        }
        if (take.empty()) return (int)hipErrorUnknown;   // unreachable: the first unscattered supernode is ready
        auto below = [&](int J) { return S.ld[J] - (S.sfirst[J + 1] - S.sfirst[J]); };
        for (int J : take) m = std::max(m, below(J));
        const int tn = pick_tile(m, [&](int tq) {
          int64_t n = 0;
          for (int J : take) n += update_tiles(below(J), tq) * nshift;
          return n;
        });
        for (size_t q = 0; q < take.size(); ++q) {
          const int J = take[q];
          items.push_back(LaneItem{panel_args(S, S.panels[plast[J]]), c.wfix, c.G, c.gstride, 0, 0});
          LaneItem& it = items.back();
          PanelK& u = it.p;
          const int32_t wj = S.sfirst[J + 1] - S.sfirst[J], bl = below(J);
          u.p0 = 0;
          u.wp = wj;
          u.nb = bl;
          it.tiles = tiles_of(bl, TM) * tiles_of(bl, tn);
          w += fm * nshift * S.xm_update[J];
          b += eb * nshift * ((double)bl * wj + (double)bl * (bl + 1));
          s += fm * nshift * (double)bl * (bl + 1) / 2.0 * wj;
          scattered[J] = 1;
          for (int64_t t = S.tgt_ptr[J]; t < S.tgt_ptr[J + 1]; ++t) --need[S.tgt[t]];
        }
        ProfScope ps(KC_UPDATE, st, w, b, s);
        with_tile(tn, [&](auto t) {
          constexpr int TN = decltype(t)::value;
          ok = with_group(c, items, nshift, [&](const auto& g, dim3 grid) {
            hipLaunchKernelGGL((k_update<CPLX, TN, std::decay_t<decltype(g)>>), grid, dim3(NT), 0, st, g);
          });
        });
      }
      if (!ok) return (int)hipErrorInvalidConfiguration;
      PXS_CHECK_LAUNCH();
    }
    return 0;
  }
  if (one_stream || NS <= 1) {
    for (int J : S.fac_order) {
      if (pfirst[J] < 0) continue;
      for (int ip = pfirst[J]; ip <= plast[J]; ++ip)
        if ((err = panel_work(S.panels[ip], st))) return err;
      if ((err = scatter(S.panels[plast[J]], st))) return err;
    }
    return 0;
  }
  // subtree streams: the panel work of J on pool stream sel_stream[J] once
  // the scatters into J are done (the scatter of fac_child[J] and, the
  // caller's stream being in order, every scatter issued before it); the
  // scatter of J on the caller's stream after J's panel work.  Scatters of
  // different supernodes write the same ancestor entries, so they stay on
  // the one stream, in fac_order.
  if ((err = ensure_pool(NS, 2 * ns + 1))) return err;
  hipEvent_t* evp = g_pool.events.data();   // evp[J]: panel work of J done
  hipEvent_t* evs = evp + ns;               // evs[J]: scatter of J done
  hipEvent_t evf = evp[2 * ns];             // assembly done
  if ((he = hipEventRecord(evf, st)) != hipSuccess) return (int)he;
  for (int J : S.fac_order) {
    if (pfirst[J] < 0) continue;
    hipStream_t sj = g_pool.streams[S.sel_stream[J]];
    const int ch = S.fac_child[J];
    if ((he = hipStreamWaitEvent(sj, ch >= 0 ? evs[ch] : evf, 0)) != hipSuccess) return (int)he;
    for (int ip = pfirst[J]; ip <= plast[J]; ++ip)
      if ((err = panel_work(S.panels[ip], sj))) return err;
    if ((he = hipEventRecord(evp[J], sj)) != hipSuccess) return (int)he;
    if (S.sparent[J] < 0) continue;   // a root: joined below
    if ((he = hipStreamWaitEvent(st, evp[J], 0)) != hipSuccess) return (int)he;
    if ((err = scatter(S.panels[plast[J]], st))) return err;
    if ((he = hipEventRecord(evs[J], st)) != hipSuccess) return (int)he;
  }
  for (int J = 0; J < ns; ++J)
    if (S.sparent[J] < 0 && pfirst[J] >= 0)
      if ((he = hipStreamWaitEvent(st, evp[J], 0)) != hipSuccess) return (int)he;
  return 0;
}

template int run_factor<true>(const Symbolic&, const double*, const double*, int, const double*, void*, void*,
                              hipStream_t, bool);
template int run_factor<false>(const Symbolic&, const double*, const double*, int, const double*, void*, void*,
                               hipStream_t, bool);
template int run_factor_kernels<true>(const Symbolic&, const double*, const double*, int, void*, void*, hipStream_t,
                                      bool);
template int run_factor_kernels<false>(const Symbolic&, const double*, const double*, int, void*, void*,
                                       hipStream_t, bool);

int64_t selinv_work_bytes(const Symbolic& S, int nshift) {
  const int chunk = (S.selinv_chunk > 0 && S.selinv_chunk < nshift) ? S.selinv_chunk : nshift;
  int64_t g = 0;
  for (int64_t b : S.gather_bytes) g += b;
  return S.work_fixed + (int64_t)nshift * S.sel_nstreams * S.work_per_shift + (int64_t)chunk * g;
}

int64_t selinv_work_bytes_inorder(const Symbolic& S, int nshift) {
  const int chunk = (S.selinv_chunk > 0 && S.selinv_chunk < nshift) ? S.selinv_chunk : nshift;
  return S.work_fixed + (int64_t)nshift * S.work_per_shift + (int64_t)chunk * S.gather_per_shift;
}

// Workspace of the allocation-free entry point (pxs_density_matrix_noalloc).
// Host code never passes this name to a kernel or a copy: it stands for a
// host-side shadow there; the device address comes from noalloc_scratch.
static __device__ __align__(256) char scratch[NOALLOC_SCRATCH_BYTES];

namespace {
constexpr int MAX_DEVICES = 64;
void* g_scratch_ptr[MAX_DEVICES] = {};
}  // namespace

int noalloc_scratch(void** ptr) {
  int dev = 0;
  hipError_t e = hipGetDevice(&dev);
  if (e != hipSuccess) return (int)e;
  if (dev < 0 || dev >= MAX_DEVICES) return (int)hipErrorInvalidDevice;
  if (!g_scratch_ptr[dev]) {
    void* p = nullptr;
    e = hipGetSymbolAddress(&p, HIP_SYMBOL(scratch));
    if (e != hipSuccess) return (int)e;
    if (!p) return (int)hipErrorInvalidSymbol;
    g_scratch_ptr[dev] = p;
  }
  *ptr = g_scratch_ptr[dev];
  return 0;
}

#define PXS_HIP(call)                      \
  do {                                     \
    hipError_t e_ = (call);                \
    if (e_ != hipSuccess) return (int)e_;  \
  } while (0)

int selinv_streams_ready(const Symbolic& S) {
  // streams are created here, never inside a stream capture
  return ensure_pool(S.sel_nstreams - 1, 0);
}

int selinv_event_count(const Symbolic& S) { return S.nsuper + S.sel_nstreams + 1; }

namespace {

// Selected inversion in fused launches (fused_lanes).  The operations of a
// supernode run in their order (per panel from the last: one operation for a
// panel of at most SMALL_ROWS rows below; for the others, after the Z_CC gather
// of the supernode, L-hat, off-diagonal product, diagonal partials, diagonal
// final); a launch on the caller's stream takes the next operation of up to
// MAX_ITEMS supernodes whose parent was finished by an earlier launch, of the
// kind that most of them wait for.  Operations that use the workspace take the
// region of the supernode's stream (sel_stream), which one supernode holds at a
// time.  Each panel operation computes what it computes on a stream of its own,
// so the results are the bits of the other paths.
enum LaneKind : int32_t { LK_GATHER, LK_LHAT, LK_OFF, LK_DPART, LK_DFIN, LK_SMALL, LK_SMALL16, LK_KINDS };

struct LaneOp {
  int32_t kind;
  int32_t rows;    // rows of an L-hat or off-diagonal product (its tiles follow from the launch's tile width), else 0
  int32_t tiles;   // workgroups per shift of the other kinds
  PanelK p;
  double work, bytes, stored;   // profile figures (ProfScope)
};

int lane_launch(int32_t kind, int tn, const Common& c, const std::vector<LaneItem>& items, int nsh, hipStream_t st) {
  bool ok = false;
  auto tiled = [&](auto launch) {   // launch(tile width, group, grid)
    with_tile(tn, [&](auto t) { ok = with_group(c, items, nsh, [&](const auto& g, dim3 grid) { launch(t, g, grid); }); });
  };
#define PXS_LANE_TILED(kernel)                                                                                  \
  tiled([&](auto t, const auto& g, dim3 grid) {                                                                 \
    hipLaunchKernelGGL((kernel<decltype(t)::value, std::decay_t<decltype(g)>>), grid, dim3(NT), 0, st, g);      \
  })
#define PXS_LANE(threads, ...)                                                                                  \
  ok = with_group(c, items, nsh, [&](const auto& g, dim3 grid) {                                                \
    hipLaunchKernelGGL((__VA_ARGS__ std::decay_t<decltype(g)>>), grid, dim3(threads), 0, st, g);                \
  })
  switch (kind) {
    case LK_GATHER: PXS_LANE(NT, k_gather_cc<); break;
    case LK_LHAT: PXS_LANE_TILED(k_lhat); break;
    case LK_OFF: PXS_LANE_TILED(k_selinv_off); break;
    case LK_DPART: PXS_LANE_TILED(k_selinv_diag_partial); break;
    case LK_DFIN: PXS_LANE(NTF, k_selinv_diag_final<); break;
    case LK_SMALL: PXS_LANE(NT, k_selinv_small<SMALL_ROWS,); break;
    case LK_SMALL16: PXS_LANE(NT, k_selinv_small<16,); break;
    default: return (int)hipErrorInvalidValue;
  }
#undef PXS_LANE
#undef PXS_LANE_TILED
  PXS_CHECK_LAUNCH();
  return ok ? 0 : (int)hipErrorInvalidConfiguration;
}

const int kLaneClass[LK_KINDS] = {KC_GATHER, KC_LHAT, KC_SELINV_OFF, KC_SELINV_DIAG, KC_NONE, KC_SELINV_OFF,
                                  KC_SELINV_OFF};

int run_selinv_lanes(const Symbolic& S, int nshift, void* L, void* work, hipStream_t st) {
  const int NL = S.sel_nstreams;
  const int ns = S.nsuper;
  const int chunk = (S.selinv_chunk > 0 && S.selinv_chunk < nshift) ? S.selinv_chunk : nshift;
  // workspace views as on NL streams (selinv_work_bytes)
  const Common c0 = make_common(S, L, work);
  std::vector<Common> cs(NL, c0);
  int64_t gofs = S.work_fixed + (int64_t)nshift * NL * S.work_per_shift;
  for (int q = 0; q < NL; ++q) {
    cs[q].wfix = S.work_fixed + (int64_t)q * nshift * S.work_per_shift;
    cs[q].G = (double*)((char*)work + gofs);
    cs[q].gstride = S.gather_bytes[q] / 8;
    gofs += (int64_t)chunk * S.gather_bytes[q];
  }
  std::vector<int> pfirst(ns, 0);
  for (int ip = (int)S.panels.size() - 1; ip >= 0; --ip) pfirst[S.panels[ip].J] = ip;
  std::vector<std::vector<LaneOp>> ops(ns);
  std::vector<size_t> pos(ns);
  std::vector<int32_t> holder(NL), ready, next, take;
  std::vector<LaneItem> items;
  std::vector<std::vector<int32_t>> kids(ns);
  for (int J = ns - 1; J >= 0; --J)
    if (S.sparent[J] >= 0) kids[S.sparent[J]].push_back(J);
  for (int sh0 = 0; sh0 < nshift; sh0 += chunk) {
    const int nsh = std::min(chunk, nshift - sh0);
    for (int J = 0; J < ns; ++J) {
      ops[J].clear();
      pos[J] = 0;
      auto add = [&](int32_t kind, const PanelK& k, int64_t tiles, double w, double b, double s) {
        ops[J].push_back(LaneOp{kind, (kind == LK_LHAT || kind == LK_OFF) ? k.nb : 0, (int32_t)tiles, k, w, b, s});
      };
      const int first = pfirst[J];
      int last = first;
      while (last + 1 < (int)S.panels.size() && S.panels[last + 1].J == J) ++last;
      bool gathered = false;
      for (int ip = last; ip >= first; --ip) {
        PanelK k = panel_args(S, S.panels[ip]);
        k.sh0 = sh0;
        const PanelMacs& xm = S.xm_panel[ip];
        if (k.nb <= SMALL_ROWS) {
          add(k.nb <= 16 ? LK_SMALL16 : LK_SMALL, k, 1, 8.0 * nsh * (xm.off + xm.sdiag),
              16.0 * nsh * (0.5 * k.nb * (k.nb + 1) + 2.0 * k.nb * k.wp + (double)k.wp * k.wp),
              8.0 * nsh * ((double)k.nb * k.nb * k.wp + (double)k.nb * k.wp * k.wp));
          continue;
        }
        if (k.c > 0 && !gathered) {
          gathered = true;
          const int64_t nt = (k.c + TM - 1) / TM;
          const double gb = (32.0 * nsh + 4.0) * 0.5 * k.c * (k.c + 1);
          add(LK_GATHER, k, nt * (nt + 1) / 2, gb, gb, gb);
        }
        add(LK_LHAT, k, 0, 0.0, 16.0 * nsh * (2.0 * k.nb * k.wp + 0.5 * k.wp * (k.wp + 1)),
            8.0 * nsh * (double)k.nb * k.wp * (k.wp + 1) / 2.0);
        add(LK_OFF, k, 0, 8.0 * nsh * xm.off, 16.0 * nsh * (0.5 * k.nb * (k.nb + 1) + 2.0 * k.nb * k.wp),
            8.0 * nsh * (double)k.nb * k.nb * k.wp);
        add(LK_DPART, k, k.split, 8.0 * nsh * xm.sdiag, 16.0 * nsh * (2.0 * k.nb * k.wp + (double)k.wp * k.wp),
            8.0 * nsh * (double)k.nb * k.wp * k.wp);
        add(LK_DFIN, k, 1, 0.0, 0.0, 0.0);
      }
    }
    std::fill(holder.begin(), holder.end(), -1);
    ready.clear();   // supernodes whose parent is finished, themselves not
    for (int J = ns - 1; J >= 0; --J)
      if (S.sparent[J] < 0) ready.push_back(J);
    while (!ready.empty()) {
      // may J's next operation run (one that uses the workspace needs the
      // region of its stream, or holds it already)
      auto runs = [&](int J) {
        const int h = holder[S.sel_stream[J]];
        return ops[J][pos[J]].kind >= LK_SMALL || h < 0 || h == J;
      };
      int cnt[LK_KINDS] = {};
      for (int J : ready)
        if (runs(J)) ++cnt[ops[J][pos[J]].kind];
      const int kind = (int)(std::max_element(cnt, cnt + LK_KINDS) - cnt);
      if (cnt[kind] == 0) return (int)hipErrorUnknown;   // unreachable: a region's holder can always go on
      take.clear();
      next.clear();
      int m = 0;
      for (int J : ready) {
        if ((int)take.size() < MAX_ITEMS && ops[J][pos[J]].kind == kind && runs(J)) {
          take.push_back(J);
          m = std::max(m, ops[J][pos[J]].p.wp);
          if (kind < LK_SMALL) holder[S.sel_stream[J]] = J;
        } else {
          next.push_back(J);
        }
      }
      auto tiles = [&](int J, int tn) {
        const LaneOp& o = ops[J][pos[J]];
        return o.rows > 0 ? tiles_of(o.rows, tn) : kind == LK_DPART ? o.tiles * tiles_of(o.p.wp, tn) : o.tiles;
      };
      const int tn = pick_tile(m, [&](int tq) {
        int64_t n = 0;
        for (int J : take) n += (int64_t)tiles(J, tq) * nsh;
        return n;
      });
      items.clear();
      double w = 0.0, b = 0.0, s = 0.0;
      for (size_t q = 0; q < take.size(); ++q) {
        const int J = take[q];
        const LaneOp& o = ops[J][pos[J]];
        const Common& cq = cs[S.sel_stream[J]];
        items.push_back(LaneItem{o.p, cq.wfix, cq.G, cq.gstride, tiles(J, tn), 0});
        w += o.work;
        b += o.bytes;
        s += o.stored;
      }
      for (int J : take) {
        ++pos[J];
        bool ws = false;   // workspace operations left
        for (size_t i = pos[J]; i < ops[J].size(); ++i) ws = ws || ops[J][i].kind < LK_SMALL;
        if (!ws && holder[S.sel_stream[J]] == J) holder[S.sel_stream[J]] = -1;
        if (pos[J] < ops[J].size()) next.push_back(J);
        else next.insert(next.end(), kids[J].begin(), kids[J].end());
      }
      {
        ProfScope ps(kLaneClass[kind], st, w, b, s);
        const int e = lane_launch(kind, tn, c0, items, nsh, st);
        if (e) return e;
      }
      ready.swap(next);
    }
  }
  return 0;
}

}  // namespace

int run_selinv(const Symbolic& S, int nshift, void* L, void* work, hipStream_t st,
               hipEvent_t* events, bool inorder) {
  // inside a stream capture everything runs on the capturing stream: the
  // subtree streams are used by eager runs only
  hipStreamCaptureStatus cap = hipStreamCaptureStatusNone;
  PXS_HIP(hipStreamIsCapturing(st, &cap));
  const bool fuse = S.fused_lanes || (S.fuse_one_stream && cap != hipStreamCaptureStatusNone);
  if (fuse && !inorder && S.sel_nstreams > 1) return run_selinv_lanes(S, nshift, L, work, st);
  const bool single = inorder || (cap != hipStreamCaptureStatusNone) || S.sel_nstreams == 1;
  const int NS = single ? 1 : S.sel_nstreams;
  const int ns = S.nsuper;
  // one stream needs no pool: the in-order path creates no streams or events
  int err = single ? 0 : ensure_pool(NS - 1, events ? 0 : selinv_event_count(S));
  if (err) return err;
  std::vector<hipStream_t> strm(NS);
  strm[0] = st;
  for (int q = 1; q < NS; ++q) strm[q] = g_pool.streams[q - 1];
  // events: the caller's (a graph plan keeps its own, since an event last
  // recorded inside a capture must not be waited on outside it) or the
  // pool's; none on one stream
  hipEvent_t* ev = single ? nullptr : (events ? events : g_pool.events.data());   // ev[J]: SelInv of J done
  hipEvent_t* ev_join = single ? nullptr : ev + ns;   // ev_join[q], q >= 1
  hipEvent_t ev_fork = single ? nullptr : ev[ns + NS];
  const int chunk = (S.selinv_chunk > 0 && S.selinv_chunk < nshift) ? S.selinv_chunk : nshift;
  // per-stream workspace views
  std::vector<Common> cs(NS, make_common(S, L, work));
  // workspace views (selinv_work_bytes): per-shift regions of all streams,
  // then the dense Z_CC regions of all streams; one stream alone uses one
  // per-shift region and a Z_CC area with the largest stride right after it
  // (selinv_work_bytes_inorder <= selinv_work_bytes)
  int64_t gofs = S.work_fixed + (int64_t)nshift * (single ? 1 : S.sel_nstreams) * S.work_per_shift;
  for (int q = 0; q < NS; ++q) {
    cs[q].wfix = S.work_fixed + (int64_t)q * nshift * S.work_per_shift;
    cs[q].G = (double*)((char*)work + gofs);
    cs[q].gstride = (single ? S.gather_per_shift : S.gather_bytes[q]) / 8;
    gofs += (int64_t)chunk * S.gather_bytes[q];
  }
  auto stream_of = [&](int J) { return single ? 0 : S.sel_stream[J]; };
  // first panel of every supernode (panels are grouped by supernode, in order)
  std::vector<int> pfirst(ns, 0);
  for (int ip = (int)S.panels.size() - 1; ip >= 0; --ip) pfirst[S.panels[ip].J] = ip;

  for (int sh0 = 0; sh0 < nshift; sh0 += chunk) {
    const int nsh = std::min(chunk, nshift - sh0);
    if (NS > 1) {
      PXS_HIP(hipEventRecord(ev_fork, st));
      for (int q = 1; q < NS; ++q) PXS_HIP(hipStreamWaitEvent(strm[q], ev_fork, 0));
    }
    // supernodes from the roots down; a child on another stream waits for
    // its parent's event
    for (int J = ns - 1; J >= 0; --J) {
      const int q = stream_of(J);
      hipStream_t sj = strm[q];
      const Common& c = cs[q];
      const int P = S.sparent[J];
      if (P >= 0 && stream_of(P) != q) PXS_HIP(hipStreamWaitEvent(sj, ev[P], 0));
      const int first = pfirst[J];
      int last = first;
      while (last + 1 < (int)S.panels.size() && S.panels[last + 1].J == J) ++last;
      PanelK g = panel_args(S, S.panels[last]);
      g.sh0 = sh0;
      // (the first panel has the most rows below: Z_CC is gathered if any has too many)
      if (g.c > 0 && S.panels[first].nb_rows > SMALL_ROWS) {
        const int nt = (g.c + TM - 1) / TM;
        // bytes: the lower triangle of Z_CC read from the ancestors and written to G, relative positions
        const double gb = (32.0 * nsh + 4.0) * 0.5 * g.c * (g.c + 1);
        ProfScope ps(KC_GATHER, sj, gb, gb, gb);
        hipLaunchKernelGGL(k_gather_cc<OnePanel>, dim3(nt * (nt + 1) / 2, nsh), dim3(NT), 0, sj, OnePanel{c, g});
      }
      for (int ip = last; ip >= first; --ip) {
        PanelK k = panel_args(S, S.panels[ip]);
        k.sh0 = sh0;
        const PanelMacs& xm = S.xm_panel[ip];
        if (k.nb <= SMALL_ROWS) {
          ProfScope ps(KC_SELINV_OFF, sj, 8.0 * nsh * (xm.off + xm.sdiag),
                       16.0 * nsh * (0.5 * k.nb * (k.nb + 1) + 2.0 * k.nb * k.wp + (double)k.wp * k.wp),
                       8.0 * nsh * ((double)k.nb * k.nb * k.wp + (double)k.nb * k.wp * k.wp));
          if (k.nb <= 16) hipLaunchKernelGGL((k_selinv_small<16, OnePanel>), dim3(1, nsh), dim3(NT), 0, sj, OnePanel{c, k});
          else hipLaunchKernelGGL((k_selinv_small<SMALL_ROWS, OnePanel>), dim3(1, nsh), dim3(NT), 0, sj, OnePanel{c, k});
          PXS_CHECK_LAUNCH();
          continue;
        }
        if (k.nb > 0) {
          const int tn = pick_tile(k.wp, [&](int q2) { return (int64_t)tiles_of(k.nb, q2) * nsh; });
          {
            // L-hat is a by-product of the blocked algorithm: no exact flops
            ProfScope ps(KC_LHAT, sj, 0.0, 16.0 * nsh * (2.0 * k.nb * k.wp + 0.5 * k.wp * (k.wp + 1)),
                         8.0 * nsh * (double)k.nb * k.wp * (k.wp + 1) / 2.0);
            with_tile(tn, [&](auto t) {
              constexpr int TN = decltype(t)::value;
              hipLaunchKernelGGL((k_lhat<TN, OnePanel>), dim3(tiles_of(k.nb, TN), nsh), dim3(NT), 0, sj, OnePanel{c, k});
            });
          }
          {
            // bytes: Z_BB (one triangle), L-hat read, Z_Bp written
            ProfScope ps(KC_SELINV_OFF, sj, 8.0 * nsh * xm.off,
                         16.0 * nsh * (0.5 * k.nb * (k.nb + 1) + 2.0 * k.nb * k.wp),
                         8.0 * nsh * (double)k.nb * k.nb * k.wp);
            with_tile(tn, [&](auto t) {
              constexpr int TN = decltype(t)::value;
              hipLaunchKernelGGL((k_selinv_off<TN, OnePanel>), dim3(tiles_of(k.nb, TN), nsh), dim3(NT), 0, sj,
                                 OnePanel{c, k});
            });
          }
          {
            ProfScope ps(KC_SELINV_DIAG, sj, 8.0 * nsh * xm.sdiag,
                         16.0 * nsh * (2.0 * k.nb * k.wp + (double)k.wp * k.wp),
                         8.0 * nsh * (double)k.nb * k.wp * k.wp);
            with_tile(pick_tile(k.wp, [&](int q2) { return (int64_t)k.split * tiles_of(k.wp, q2) * nsh; }), [&](auto t) {
              constexpr int TN = decltype(t)::value;
              hipLaunchKernelGGL((k_selinv_diag_partial<TN, OnePanel>), dim3(k.split * tiles_of(k.wp, TN), nsh), dim3(NT), 0,
                                 sj, OnePanel{c, k});
            });
          }
        }
        hipLaunchKernelGGL(k_selinv_diag_final<OnePanel>, dim3(1, nsh), dim3(NTF), 0, sj, OnePanel{c, k});
        PXS_CHECK_LAUNCH();
      }
      if (!single && S.cross_child[J]) PXS_HIP(hipEventRecord(ev[J], sj));
    }
    if (NS > 1) {
      for (int q = 1; q < NS; ++q) {
        PXS_HIP(hipEventRecord(ev_join[q], strm[q]));
        PXS_HIP(hipStreamWaitEvent(st, ev_join[q], 0));
      }
    }
  }
  return 0;
}

int run_inertia_async(const Symbolic& S, const double* H, const double* Sv, int nshift, const double* eps_dev,
                      void* L, void* work, int64_t* neg_dev, int64_t* info_dev, hipStream_t st) {
  char* w = (char*)work;
  hipLaunchKernelGGL(k_real_shifts, dim3((nshift + NT - 1) / NT), dim3(NT), 0, st, eps_dev,
                     (double*)(w + WK_SHIFTS), nshift);
  PXS_CHECK_LAUNCH();
  const int e = run_factor_kernels<false>(S, H, Sv, nshift, L, work, st, true);
  if (e) return e;
  PXS_HIP(hipMemcpyAsync(neg_dev, w + WK_NEGC, sizeof(int64_t) * nshift, hipMemcpyDeviceToDevice, st));
  PXS_HIP(hipMemcpyAsync(info_dev, w + WK_INFO, sizeof(int64_t) * nshift, hipMemcpyDeviceToDevice, st));
  return 0;
}

int run_pole_sum(const Symbolic& S, int nshift, const void* L, void* work, const double* H,
                 const double* Sv, int nsets, const double* weights_host, double* out,
                 hipStream_t st) {
  int e = upload_weights(nshift, nsets, weights_host, work, st);
  if (e != 0) return e;
  return run_pole_sum_kernels(S, nshift, L, work, H, Sv, nsets, out, 0, st);
}

int run_pole_sum_kernels(const Symbolic& S, int nshift, const void* L, void* work, const double* H,
                         const double* Sv, int nsets, double* out, int accumulate, hipStream_t st) {
  char* w = (char*)work;
  const char* m = (const char*)S.dmaps;
  const int nb = blocks_for(S.nnz_lower, POLESUM_BLOCKS);
  // bytes: one complex per entry and shift, offsets, flags, H, S, nsets outputs
  const double ab = (double)S.nnz_lower * (16.0 * nshift + 28.0 + 8.0 * nsets);
  ProfScope ps(KC_POLESUM, st, ab, ab, ab);
  hipLaunchKernelGGL(k_pole_sum, dim3(nb), dim3(NT), 0, st, (const double*)L, S.nnzL_store, nshift,
                     (const double*)(w + WK_WEIGHTS), nsets, (const int64_t*)(m + S.o_entry_off),
                     (const int32_t*)(m + S.o_entry_diag), S.nnz_lower, H, Sv, out,
                     (double*)(w + WK_POLESUM_PART), accumulate);
  hipLaunchKernelGGL(k_sum_partials, dim3(1), dim3(512), 0, st, (const double*)(w + WK_POLESUM_PART), nb,
                     (double*)(w + WK_TRACES));
  PXS_CHECK_LAUNCH();
  return 0;
}

int run_gather(const Symbolic& S, int shift, const void* L, void* out, hipStream_t st) {
  const char* m = (const char*)S.dmaps;
  const double* Ls = (const double*)L + 2 * S.nnzL_store * (int64_t)shift;
  hipLaunchKernelGGL(k_gather, dim3(blocks_for(S.nnz_lower, 4096)), dim3(NT), 0, st, Ls,
                     (const int64_t*)(m + S.o_entry_off), S.nnz_lower, (double2*)out);
  PXS_CHECK_LAUNCH();
  return 0;
}

int run_get_diag(const Symbolic& S, int shift, bool cplx, const void* L, void* out, hipStream_t st) {
  const char* m = (const char*)S.dmaps;
  const double* Ls = (const double*)L + (cplx ? 2 : 1) * S.nnzL_store * (int64_t)shift;
  hipLaunchKernelGGL(k_get_diag, dim3((S.n + NT - 1) / NT), dim3(NT), 0, st, Ls,
                     (const int64_t*)(m + S.o_diagoff), S.n, cplx ? 1 : 0, (double2*)out);
  PXS_CHECK_LAUNCH();
  return 0;
}

#include "hermitian.inc"
#include "batch.inc"

}  // namespace pxs
