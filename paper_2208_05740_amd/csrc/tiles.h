// Tile-level device code shared by the per-layer kernels (kernels.hip) and
// the persistent dataflow kernel (persist_kernels.hip): the tile GEMM with a
// fused epilogue on gfx950 MFMA, and the elementwise relaxation of a block
// of rows.
#pragma once
#include "gcp_internal.h"
#include "epilogues.h"

#include <hip/hip_runtime.h>

#include <type_traits>

namespace gcp {

// ------------------------------------------------------------------ tile GEMM
// C[M][N] = A[M][K] * Bt[N][K]^T on MFMA, epilogue per element, row partial
// sums reduced deterministically (lanes, then waves through LDS) into
// partial[r][slot0 + blockIdx.x].
// LDS of one tile: the A and B stages (16-byte row padding) and the per-wave
// row partials.
template <typename T, int BM, int BN, int WN, int BK>
struct TileLds {
  static constexpr int LD = BK + Op<T>::VEC;
  __attribute__((aligned(16))) T As[BM * LD];
  __attribute__((aligned(16))) T Bs[BN * LD];
  double red[WN][BM];
};

// One output tile (linear index vt, row panel major) of one GEMM problem,
// staged through the LDS block `sm`.
// OPAQUE: the thread id is made opaque to the optimiser, so that inside a
// persistent loop the values derived from it are recomputed per tile instead
// of held live across all of them (it costs the single-tile kernels
// registers, so they keep the plain id).
template <typename T, int BM, int BN, int WM, int WN, int BK, bool SIGN, class Epi, bool OPAQUE = false>
__device__ inline void gemm_tile_lds(const GemmArgs& g, const Epi& epi, int vt, TileLds<T, BM, BN, WN, BK>& sm) {
  constexpr int NT = WM * WN * 64;
  constexpr int VEC = Op<T>::VEC;
  constexpr int KC = Op<T>::KC;
  constexpr int LDS_LD = BK + VEC;          // 16-byte row padding
  constexpr int TM = BM / WM / 16;
  constexpr int TN = BN / WN / 16;
  constexpr int AV = BM * BK / VEC;         // 16-byte vectors per A stage
  constexpr int BV = BN * BK / VEC;
  constexpr int AIT = (AV + NT - 1) / NT;
  constexpr int BIT = (BV + NT - 1) / NT;
  static_assert(BK % KC == 0, "BK must be a multiple of the fragment K");

  T* As = sm.As;
  T* Bs = sm.Bs;
  auto& red = sm.red;

  int tid = threadIdx.x;
  if constexpr (OPAQUE) asm volatile("" : "+v"(tid));
  const int lane = tid & 63;
  const int wave = tid >> 6;
  const int wm = wave / WN, wn = wave % WN;
  const int n_col = (g.N + BN - 1) / BN;
  const int bx = vt % n_col, by = vt / n_col;
  const int m0 = by * BM, n0 = bx * BN;

  f4 acc[TM][TN];
#pragma unroll
  for (int i = 0; i < TM; ++i)
#pragma unroll
    for (int k = 0; k < TN; ++k) acc[i][k] = f4{0.f, 0.f, 0.f, 0.f};

  uint4 ra[AIT], rb[BIT];
  auto load_stage = [&](int k0) {
#pragma unroll
    for (int it = 0; it < AIT; ++it) {
      int v = tid + it * NT;
      uint4 val = {0u, 0u, 0u, 0u};
      if (v < AV) {
        int row = v / (BK / VEC), kk = (v % (BK / VEC)) * VEC;
        int gr = m0 + row, gk = k0 + kk;
        if (gr < g.M && gk < g.lda) {
          if constexpr (SIGN) {
            // VEC int8 signs in one load (the row pitch and gk are multiples of VEC)
            const int8_t* src = (const int8_t*)g.A + (size_t)gr * g.lda + gk;
            int8_t e[VEC];
            if constexpr (VEC == 8) *(uint2*)e = *(const uint2*)src;
            else *(uint32_t*)e = *(const uint32_t*)src;
            T tmp[VEC];
#pragma unroll
            for (int q = 0; q < VEC; ++q) tmp[q] = to_t<T>((float)e[q]);
            val = *(const uint4*)tmp;
          } else {
            val = *(const uint4*)((const T*)g.A + (size_t)gr * g.lda + gk);
          }
          if (gk + VEC > g.K) val = mask_tail<T>(val, g.K - gk);
        }
      }
      ra[it] = val;
    }
#pragma unroll
    for (int it = 0; it < BIT; ++it) {
      int v = tid + it * NT;
      uint4 val = {0u, 0u, 0u, 0u};
      if (v < BV) {
        int row = v / (BK / VEC), kk = (v % (BK / VEC)) * VEC;
        int gn = n0 + row, gk = k0 + kk;
        if (gn < g.N && gk < g.ldb) {
          val = *(const uint4*)((const T*)g.Bt + (size_t)gn * g.ldb + gk);
          if (gk + VEC > g.K) val = mask_tail<T>(val, g.K - gk);
        }
      }
      rb[it] = val;
    }
  };
  auto store_stage = [&]() {
#pragma unroll
    for (int it = 0; it < AIT; ++it) {
      int v = tid + it * NT;
      if (v < AV) {
        int row = v / (BK / VEC), kk = (v % (BK / VEC)) * VEC;
        *(uint4*)(As + row * LDS_LD + kk) = ra[it];
      }
    }
#pragma unroll
    for (int it = 0; it < BIT; ++it) {
      int v = tid + it * NT;
      if (v < BV) {
        int row = v / (BK / VEC), kk = (v % (BK / VEC)) * VEC;
        *(uint4*)(Bs + row * LDS_LD + kk) = rb[it];
      }
    }
  };

  const int arow = wm * (BM / WM) + (lane & 15);
  const int bcol = wn * (BN / WN) + (lane & 15);
  const int kq = (lane >> 4) * VEC;

  // output coordinates of this lane
  constexpr int R = TM * 4;
  LaneCoords<R, TN, false> lc;
  {
    const int row0 = m0 + wm * (BM / WM) + (lane >> 4) * 4;
    const int col0 = n0 + wn * (BN / WN) + (lane & 15);
#pragma unroll
    for (int i = 0; i < TM; ++i)
#pragma unroll
      for (int v = 0; v < 4; ++v) lc.r[i * 4 + v] = row0 + i * 16 + v;
#pragma unroll
    for (int k = 0; k < TN; ++k) lc.j[k][0] = col0 + k * 16;
  }
  ColPre<TN> pre;
  if constexpr (Epi::kColPre) {
    int col[TN];
#pragma unroll
    for (int k = 0; k < TN; ++k) col[k] = lc.j[k][0];
    col_prefetch<TN>(pre, epi.col_node(), epi.col_cuts(), col, g.N);
  }
  if (g.K > 0) load_stage(0);
  for (int k0 = 0; k0 < g.K; k0 += BK) {
    __syncthreads();
    store_stage();
    __syncthreads();
    if (k0 + BK < g.K) load_stage(k0 + BK);
#pragma unroll
    for (int kc = 0; kc < BK; kc += KC) {
      uint4 fa[TM], fb[TN];
#pragma unroll
      for (int i = 0; i < TM; ++i) fa[i] = *(const uint4*)(As + (arow + i * 16) * LDS_LD + kc + kq);
#pragma unroll
      for (int k = 0; k < TN; ++k) fb[k] = *(const uint4*)(Bs + (bcol + k * 16) * LDS_LD + kc + kq);
#pragma unroll
      for (int i = 0; i < TM; ++i)
#pragma unroll
        for (int k = 0; k < TN; ++k) Op<T>::mma(fa[i], fb[k], acc[i][k]);
    }
  }

  // Epilogue: lane holds rows 4*(lane/16)+v, column lane%16 of each 16x16 tile.
  // Its operands are fetched after the K loop: the K loops of these layers
  // are a few steps long, so prefetching them before the loop hid little
  // latency while keeping them live across it cost registers, and the
  // occupancy that buys back was worth more (measured: the adjoint kernel of
  // the 784-256x6 MLP at 1024 domains went from 41 to 36 us).
  typename Epi::template Frag<R, TN, false> fr;
  if constexpr (Epi::kColPre) epi.template load<R, TN, false>(fr, lc, g.M, g.N, &pre);
  else epi.template load<R, TN, false>(fr, lc, g.M, g.N);
  {
    double rs[R];
#pragma unroll
    for (int q = 0; q < R; ++q) rs[q] = 0.0;
    float val[TN][R];
#pragma unroll
    for (int k = 0; k < TN; ++k)
#pragma unroll
      for (int i = 0; i < TM; ++i)
#pragma unroll
        for (int v = 0; v < 4; ++v) val[k][i * 4 + v] = acc[i][k][v];
    epi.template apply<R, TN, false>(fr, lc, val, rs, g.M, g.N);
#pragma unroll
    for (int q = 0; q < R; ++q) {
      double t = wave_sum16(rs[q]);
      if ((lane & 15) == 0) red[wn][lc.r[q] - m0] = t;
    }
  }
  if (g.partial) {
    // row partials: one slot per 32 output columns, independent of the tile;
    // this block's sum goes to its first slot, zeros to the others it covers
    __syncthreads();
    const int nsl = (g.N + 31) / 32;
    const int s0 = bx * (BN / 32);
    for (int rl = tid; rl < BM; rl += NT) {
      int r = m0 + rl;
      if (r < g.M) {
        double s = 0.0;
#pragma unroll
        for (int w = 0; w < WN; ++w) s += red[w][rl];
#pragma unroll
        for (int t = 0; t < BN / 32; ++t)
          if (s0 + t < nsl) g.partial[(size_t)(g.slot0 + s0 + t) * g.mp + r] = t == 0 ? s : 0.0;
      }
    }
  }
}

// The same tile with its LDS block of its own.
template <typename T, int BM, int BN, int WM, int WN, int BK, bool SIGN, class Epi>
__device__ inline void gemm_tile(const GemmArgs& g, const Epi& epi, int vt) {
  __shared__ TileLds<T, BM, BN, WN, BK> sm;
  gemm_tile_lds<T, BM, BN, WM, WN, BK, SIGN, Epi>(g, epi, vt, sm);
}

// ------------------------------------------------------------------ layer tiles
// The per-layer launches' tile GEMM: WM x WN waves, each a (16 TM) x (16 TN)
// tile.  Two forms of the K loop:
//  - staged (D = 0, StagedLoop): A and B through LDS, 128 bytes of K at a
//    time.  For launches that fill the chip: each operand row is read once per
//    workgroup in whole cache lines.
//  - direct (D > 0): each wave reads its fragments from global memory in the
//    MFMA layout (lane i + 16 g: 16 bytes of row or column i at K offset
//    g VEC), D steps ahead in registers, no LDS and no barrier.  For launches
//    of a few workgroups, where latency is all: the 784-256x6 MLP's ascent at
//    9 rows 2195 -> 1570 us; at 9216 rows these reads (16 rows x 64 bytes
//    each) are bound by the L1 (10.1 -> 15.0 ms).
// A 9216 x 256 x 256 launch has nine waves per SIMD, so what bounds it is the
// sum of a wave's instructions and of the memory round trips that six to eight
// resident waves do not cover.  Hence the epilogue's rank-addressed operands
// (SubPre) are fetched before the K loop and arrive under it, two stages of
// the K loop are in flight, and nothing on the way carries a branch: with one,
// the compiler cannot count the loads in flight and every wait becomes a wait
// for all of them.  (Direct global-to-LDS loads have the same effect.)
// Measured there, all operands loaded after the K loop with 64-bit addresses
// -> now: relaxation 28.7 -> 24.1 us (bf16 18.0 -> 16.0), adjoint 38.4 -> 37.5
// (its alpha and moment traffic alone takes 12), adjoint from the sign matrix
// (K = 784) 70 -> 54, concretisation 51 -> 46.6.  Several tiles per workgroup
// with the next tile's loads ahead of the epilogue measured slower (three
// waves per SIMD, 43 us for the relaxation).  Both forms accumulate the
// fragments in the order of gemm_tile_lds, so the results are the same bits.
// Operand rows and epilogue windows have 32-bit offsets: launches that these do
// not reach run gemm_tile_lds (gemm_config_for).
template <typename T, int TM, int TN, int WM, int WN, int D>
struct LayerLds {
  static constexpr int BM = WM * TM * 16, BN = WN * TN * 16, BK = 128 / (int)sizeof(T), LD = BK + Op<T>::VEC;
  static constexpr int N = D > 0 ? 1 : 2;
  __attribute__((aligned(16))) T As[N][D > 0 ? 1 : BM * LD];
  __attribute__((aligned(16))) T Bs[N][D > 0 ? 1 : BN * LD];
  double red[WN][BM];
};

// 16 bytes of operand A (or the same number of sign bytes) as a fragment
template <typename T, bool SIGN> struct AFrag { typedef uint4 V; };
template <typename T> struct AFrag<T, true> {
  typedef typename std::conditional<Op<T>::VEC == 4, uint32_t, uint2>::type V;
};
template <typename T, bool SIGN>
__device__ inline uint4 as_frag(const typename AFrag<T, SIGN>::V& x) {
  if constexpr (SIGN) {
    T e[Op<T>::VEC];
    int8_t b[Op<T>::VEC];
    *(typename AFrag<T, SIGN>::V*)b = x;
#pragma unroll
    for (int q = 0; q < Op<T>::VEC; ++q) e[q] = to_t<T>((float)b[q]);
    return *(const uint4*)e;
  } else {
    return x;
  }
}

// The staged K loop of one workgroup: two stages in LDS (one multiplied, one
// written), two more in flight in registers.
template <typename T, int TM, int TN, int WM, int WN, bool SIGN>
struct StagedLoop {
  typedef LayerLds<T, TM, TN, WM, WN, 0> L;
  typedef typename AFrag<T, SIGN>::V AV;
  static constexpr int VEC = Op<T>::VEC, KC = Op<T>::KC, AB = SIGN ? 1 : (int)sizeof(T);
  static constexpr int BM = L::BM, BN = L::BN, BK = L::BK, LD = L::LD, NT = WM * WN * 64;
  static constexpr int CV = BK / VEC;                       // 16-byte vectors per staged row
  static constexpr int AIT = (BM * CV + NT - 1) / NT, BIT = (BN * CV + NT - 1) / NT;
  static_assert(BM * CV % NT == 0 || BM * CV < NT, "whole or single staging steps");
  static_assert(BN * CV % NT == 0 || BN * CV < NT, "whole or single staging steps");
  const char *Ab, *Bb;
  uint32_t oa[AIT], ob[BIT];
  int wa[AIT], wb[BIT], kk, arow, bcol, last;
  AV ra[2][AIT];
  uint4 rb[2][BIT];
  // this thread's vectors: row tid / CV (+ NT / CV per step), column tid % CV;
  // a thread past the tile's last row repeats it
  __device__ __forceinline__ void init(const GemmArgs& g, int tid, int wm, int wn, int li, int lg) {
    kk = tid % CV * VEC;
    last = (g.K + BK - 1) / BK - 1;
#pragma unroll
    for (int it = 0; it < AIT; ++it) wa[it] = min(tid / CV + it * (NT / CV), BM - 1) * LD + kk;
#pragma unroll
    for (int it = 0; it < BIT; ++it) wb[it] = min(tid / CV + it * (NT / CV), BN - 1) * LD + kk;
    // (computed here, not after the loads: there the address arithmetic could
    // take a register that a load in flight will write, and wait for it)
    arow = (wm * TM * 16 + li) * LD + lg * VEC;
    bcol = (wn * TN * 16 + li) * LD + lg * VEC;
    asm volatile("" : "+v"(arow), "+v"(bcol));
  }
  __device__ __forceinline__ void fetch(const GemmArgs& g, int st, int d) {
    const int k = st * BK + kk;         // (clamped to the row's last vector; the pitch is a multiple of VEC)
#pragma unroll
    for (int it = 0; it < AIT; ++it) ra[d][it] = ld_at<AV>(Ab, oa[it] + (uint32_t)min(k, g.lda - VEC) * AB);
#pragma unroll
    for (int it = 0; it < BIT; ++it) rb[d][it] = ld_at<uint4>(Bb, ob[it] + (uint32_t)min(k, g.ldb - VEC) * (uint32_t)sizeof(T));
  }
  // the first two stages of the tile at (m0, n0)
  __device__ __forceinline__ void start(const GemmArgs& g, int tid, int m0, int n0) {
    Ab = (const char*)g.A + (size_t)m0 * g.lda * AB;
    Bb = (const char*)g.Bt + (size_t)n0 * g.ldb * sizeof(T);
#pragma unroll
    for (int it = 0; it < AIT; ++it)
      oa[it] = (uint32_t)min(min(tid / CV + it * (NT / CV), BM - 1), g.M - 1 - m0) * ((uint32_t)g.lda * AB);
#pragma unroll
    for (int it = 0; it < BIT; ++it)
      ob[it] = (uint32_t)min(min(tid / CV + it * (NT / CV), BN - 1), g.N - 1 - n0) * ((uint32_t)g.ldb * (uint32_t)sizeof(T));
    fetch(g, 0, 0);
    fetch(g, min(1, last), 1);
  }
  __device__ __forceinline__ void put(const GemmArgs& g, L& sm, int st, int d) {
    T* A = sm.As[d];
    T* B = sm.Bs[d];
    const bool tail = (st + 1) * BK > g.K;      // columns past K hold no data of this precision
    const int keep = g.K - (st * BK + kk);
#pragma unroll
    for (int it = 0; it < AIT; ++it) {
      uint4 v = as_frag<T, SIGN>(ra[d][it]);
      if (tail) v = mask_tail<T>(v, keep);
      *(uint4*)(A + wa[it]) = v;
    }
#pragma unroll
    for (int it = 0; it < BIT; ++it) {
      uint4 v = rb[d][it];
      if (tail) v = mask_tail<T>(v, keep);
      *(uint4*)(B + wb[it]) = v;
    }
  }
  __device__ __forceinline__ void mul(const L& sm, int d, f4 (&acc)[TM][TN]) {
    const T* A = sm.As[d] + arow;
    const T* B = sm.Bs[d] + bcol;
#pragma unroll
    for (int kc = 0; kc < BK; kc += KC) {
      uint4 a[TM], b[TN];
#pragma unroll
      for (int i = 0; i < TM; ++i) a[i] = *(const uint4*)(A + i * 16 * LD + kc);
#pragma unroll
      for (int k = 0; k < TN; ++k) b[k] = *(const uint4*)(B + k * 16 * LD + kc);
#pragma unroll
      for (int i = 0; i < TM; ++i)
#pragma unroll
        for (int k = 0; k < TN; ++k) Op<T>::mma(a[i], b[k], acc[i][k]);
    }
  }
  // stage st is in LDS, st + 1 and st + 2 are in flight
  __device__ __forceinline__ void step(const GemmArgs& g, L& sm, int st, int d, f4 (&acc)[TM][TN]) {
    mul(sm, d, acc);
    put(g, sm, st + 1, d ^ 1);
    fetch(g, min(st + 3, last), d ^ 1);
    __syncthreads();
  }
  __device__ __forceinline__ void run(const GemmArgs& g, L& sm, f4 (&acc)[TM][TN]) {
#pragma unroll
    for (int i = 0; i < TM; ++i)
#pragma unroll
      for (int k = 0; k < TN; ++k) acc[i][k] = f4{0.f, 0.f, 0.f, 0.f};
    put(g, sm, 0, 0);
    fetch(g, min(2, last), 0);
    __syncthreads();
    int st = 0;
    for (; st + 2 <= last; st += 2) {
      step(g, sm, st, 0, acc);
      step(g, sm, st + 1, 1, acc);
    }
    if (st < last) {
      step(g, sm, st, 0, acc);
      mul(sm, 1, acc);
    } else if (last >= 0) {
      mul(sm, 0, acc);
    }
  }
};

// The neuron's words of column j: what the rank-addressed loads wait on.
template <class Epi>
__device__ inline void fetch_words(const Epi& epi, int j, int N, SubPre& p) {
  if constexpr (Epi::kColPre) {
    const int2* rng = epi.col_cuts().rng;
    const uint32_t col = (uint32_t)min(j, N - 1);
    p.kind = ld_at<int>(epi.col_node().kind, col * 4u);
    p.rng = make_int2(0, 0);
    if (rng) p.rng = ld_at<int2>(rng, col * 8u);
  }
}

// Epilogue of one 16x16 sub-tile in the MFMA layout (lane: rows 4 (lane / 16)
// + v, column lane % 16).
template <typename T, class Epi>
__device__ __forceinline__ void sub_epilogue(const GemmArgs& g, const Epi& epi, const TileLane& t, const SubPre& p,
                                             const f4& acc, double (&rs)[4]) {
  if constexpr (Epi::kPre > 0) {
    float sG[4], sH[4], sQ[4];
    tile_cuts(epi.a.cc, epi.a.rp, t, p, sG, sH, sQ);
    const float val[4] = {acc[0], acc[1], acc[2], acc[3]};
    const NodeDev& nd = epi.col_node();
    const uint32_t pitch = nd.ld * (uint32_t)sizeof(T), off = lane_off(t, t.jv, nd.ld, t.j, sizeof(T));
    const RowWin w = row_win(epi.out_base(), t.m0, t.rows, pitch);
    epi.tile(val, p, t, sG, sH, sQ, rs, g.partial != nullptr, [&](int q, T v) { win_st<T>(w, off + q * pitch, v); });
  } else {
    LaneCoords<4, 1, false> lc;
#pragma unroll
    for (int v = 0; v < 4; ++v) lc.r[v] = t.m0 + t.rl + v;
    lc.j[0][0] = t.j;
    const float val[1][4] = {{acc[0], acc[1], acc[2], acc[3]}};
    typename Epi::template Frag<4, 1, false> fr;
    if constexpr (Epi::kColPre) {
      ColPre<1> cp;
      cp.kind[0] = t.jv ? p.kind : 0;
      cp.rng[0] = t.jv ? p.rng : make_int2(0, 0);
      epi.template load<4, 1, false>(fr, lc, g.M, g.N, &cp);
    } else {
      epi.template load<4, 1, false>(fr, lc, g.M, g.N);
    }
    if (g.partial) {
      epi.template apply<4, 1, false>(fr, lc, val, rs, g.M, g.N);
    } else {                 // the row constants are not asked for: dead is never read
      double dead[4] = {0.0, 0.0, 0.0, 0.0};
      epi.template apply<4, 1, false>(fr, lc, val, dead, g.M, g.N);
    }
  }
}

// Row partials of a tile: one slot per 32 output columns, independent of the
// tile; the block's sum goes to its first slot, zeros to the others it covers.
template <int TM, int WN, int BM, int BN, int NT>
__device__ __forceinline__ void store_partials(const GemmArgs& g, double (&red)[WN][BM], const double (&rs)[TM][4], int m0,
                                               int bx, int wm, int wn, int li, int lg) {
#pragma unroll
  for (int i = 0; i < TM; ++i)
#pragma unroll
    for (int v = 0; v < 4; ++v) {
      const double t = wave_sum16(rs[i][v]);
      if (li == 0) red[wn][wm * TM * 16 + i * 16 + lg * 4 + v] = t;
    }
  __syncthreads();
  const int nsl = (g.N + 31) / 32;
  const int s0 = bx * (BN / 32);
  for (int rl = threadIdx.x; rl < BM; rl += NT) {
    const int r = m0 + rl;
    if (r < g.M) {
      double s = 0.0;
#pragma unroll
      for (int w = 0; w < WN; ++w) s += red[w][rl];
#pragma unroll
      for (int t = 0; t < BN / 32; ++t)
        if (s0 + t < nsl) g.partial[(size_t)(g.slot0 + s0 + t) * g.mp + r] = t == 0 ? s : 0.0;
    }
  }
}

template <typename T, int TM, int TN, int WM, int WN, int D, bool SIGN, class Epi>
__device__ __forceinline__ void layer_tile(const GemmArgs& g, const Epi& epi, int vt,
                                           LayerLds<T, TM, TN, WM, WN, D>& sm) {
  constexpr int VEC = Op<T>::VEC, KC = Op<T>::KC;
  constexpr int BM = WM * TM * 16, BN = WN * TN * 16, NT = WM * WN * 64;
  constexpr bool kEarly = TM * TN == 1;      // the register operands of one sub-tile are fetched before the K loop
  constexpr int AB = SIGN ? 1 : (int)sizeof(T);
  typedef typename AFrag<T, SIGN>::V AV;
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int wm = wave / WN, wn = wave % WN;
  const int n_col = (g.N + BN - 1) / BN;
  const int bx = vt % n_col, by = vt / n_col;
  const int m0 = by * BM, n0 = bx * BN;
  const int nw = n0 + wn * TN * 16;
  const int li = lane & 15, lg = lane >> 4;
  SubPre pre[TN];
#pragma unroll
  for (int k = 0; k < TN; ++k) fetch_words(epi, nw + k * 16 + li, g.N, pre[k]);
  f4 acc[TM][TN];
  // the lane's place in sub-tile (i, k)
  auto lane_at = [&](int i, int k) -> TileLane {
    const int j = nw + k * 16 + li;
    return TileLane{m0, min(BM, g.M - m0), (wm * TM + i) * 16 + lg * 4, j, min(j, g.N - 1), j < g.N};
  };
  auto early = [&](int i, int k) {
    if constexpr (Epi::kPre > 0) fetch_pre<T>(epi, lane_at(i, k), pre[k]);
  };
  if constexpr (D > 0) {
    const char* Ab = (const char*)g.A + (size_t)m0 * g.lda * AB;
    const char* Bb = (const char*)g.Bt + (size_t)n0 * g.ldb * sizeof(T);
#pragma unroll
    for (int i = 0; i < TM; ++i)
#pragma unroll
      for (int k = 0; k < TN; ++k) acc[i][k] = f4{0.f, 0.f, 0.f, 0.f};
    // operand rows of this lane (clamped: rows and columns past the edge only
    // feed outputs that are not stored)
    const int nfull = g.K / KC, last = max(nfull - 1, 0);
    uint32_t oa[TM], ob[TN];
#pragma unroll
    for (int i = 0; i < TM; ++i) oa[i] = (uint32_t)min((wm * TM + i) * 16 + li, g.M - 1 - m0) * (uint32_t)g.lda * AB;
#pragma unroll
    for (int k = 0; k < TN; ++k) ob[k] = (uint32_t)min((wn * TN + k) * 16 + li, g.N - 1 - n0) * (uint32_t)g.ldb * (uint32_t)sizeof(T);
    AV fa[D][TM];
    uint4 fb[D][TN];
    // K step s (lane offset ko elements) into slot d
    auto fetch = [&](int s, int d, int ko) {
#pragma unroll
      for (int i = 0; i < TM; ++i) fa[d][i] = ld_at<AV>(Ab, oa[i] + (uint32_t)((s * KC + ko) * AB));
#pragma unroll
      for (int k = 0; k < TN; ++k) fb[d][k] = ld_at<uint4>(Bb, ob[k] + (uint32_t)((s * KC + ko) * (int)sizeof(T)));
    };
    auto mul = [&](int d) {
      uint4 a[TM];
#pragma unroll
      for (int i = 0; i < TM; ++i) a[i] = as_frag<T, SIGN>(fa[d][i]);
#pragma unroll
      for (int i = 0; i < TM; ++i)
#pragma unroll
        for (int k = 0; k < TN; ++k) Op<T>::mma(a[i], fb[d][k], acc[i][k]);
    };
    // past the last full step the fetches repeat it (K < KC: every lane reads
    // its row's first elements, unused)
    const int ko = nfull > 0 ? lg * VEC : 0;
#pragma unroll
    for (int d = 0; d < D; ++d) fetch(min(d, last), d, ko);
    if constexpr (kEarly) early(0, 0);
    int s = 0;
    auto group = [&]() {
#pragma unroll
      for (int d = 0; d < D; ++d) {
        mul(d);
        fetch(min(s + d + D, last), d, ko);
        __builtin_amdgcn_sched_barrier(0);   // keep the fetches spread over the steps
      }
      s += D;
    };
    const int nmain = nfull - nfull % D;
    if (nmain > 0) {
      group();      // apart from the loop: its waits leave the epilogue's loads in flight
      while (s < nmain) group();
    }
#pragma unroll
    for (int d = 0; d < D - 1; ++d)
      if (d < nfull - nmain) mul(d);
    if (g.K % KC != 0) {       // the last step, masked (columns past K hold no data of this precision)
      const int keep = g.K - (nfull * KC + lg * VEC);
#pragma unroll
      for (int i = 0; i < TM; ++i) fa[0][i] = AV{};
#pragma unroll
      for (int k = 0; k < TN; ++k) fb[0][k] = uint4{0u, 0u, 0u, 0u};
      if (keep > 0) fetch(nfull, 0, lg * VEC);
      uint4 a[TM];
#pragma unroll
      for (int i = 0; i < TM; ++i) a[i] = mask_tail<T>(as_frag<T, SIGN>(fa[0][i]), keep);
#pragma unroll
      for (int k = 0; k < TN; ++k) fb[0][k] = mask_tail<T>(fb[0][k], keep);
#pragma unroll
      for (int i = 0; i < TM; ++i)
#pragma unroll
        for (int k = 0; k < TN; ++k) Op<T>::mma(a[i], fb[0][k], acc[i][k]);
    }
  } else {
    StagedLoop<T, TM, TN, WM, WN, SIGN> kl;
    kl.init(g, tid, wm, wn, li, lg);
    kl.start(g, tid, m0, n0);
    if constexpr (kEarly) early(0, 0);
    kl.run(g, sm, acc);
  }
  double rs[TM][4];
#pragma unroll
  for (int i = 0; i < TM; ++i)
#pragma unroll
    for (int v = 0; v < 4; ++v) rs[i][v] = 0.0;
#pragma unroll
  for (int i = 0; i < TM; ++i)
#pragma unroll
    for (int k = 0; k < TN; ++k) {
      if constexpr (!kEarly) early(i, k);
      sub_epilogue<T>(g, epi, lane_at(i, k), pre[k], acc[i][k], rs[i]);
    }
  if (g.partial) store_partials<TM, WN, BM, BN, NT>(g, sm.red, rs, m0, bx, wm, wn, li, lg);
}

// Elementwise relaxation (no GEMM: a_hat = bcast row + src): one block =
// kElemRows consecutive rows x 256 columns, each thread one column of those
// rows, so a neuron's data is read once for them and their loads are in
// flight together; one row partial per (row, column block), summed over the
// block in a fixed order.  PI selects the explicit-pi relaxation (a.rp.rho
// set); WIDE: arrays too large for the windows (windows_wide).
template <typename T, bool PI, bool OPAQUE = false, bool WIDE = false>
__device__ __forceinline__ void bound_elem_rows(const float* bcast, const void* src, const BoundEpiArgs& a, double* partial,
                                       int slot0, int r0, int cb) {
  constexpr int R = kElemRows;
  __shared__ double red[R][4];
  int tx = threadIdx.x;
  if constexpr (OPAQUE) asm volatile("" : "+v"(tx));   // as in gemm_tile_lds
  const int j = cb * 256 + tx;
  const int M = a.rp.M;
  BoundEpi<T, PI> epi{a};
  double rs[R];
#pragma unroll
  for (int q = 0; q < R; ++q) rs[q] = 0.0;
  if constexpr (!PI && !OPAQUE && !WIDE) {
    // as a layer tile of one column per lane (r0 is wave-uniform): bound by the
    // wave's instructions and its alpha and cut loads; with 64-bit addresses
    // and a division per row, 784-256x6 MLP: 9 rows 4.3 -> 3.4 us, 9216 rows
    // 16.2 -> 14.2, 36864 rows 53.6 -> 42.4
    static_assert(R == 4, "four rows, as BoundEpi::tile takes them");
    const TileLane t{r0, min(R, M - r0), 0, j, min(j, a.nd.size - 1), j < a.nd.size};
    SubPre p;
    fetch_words(epi, j, a.nd.size, p);
    const uint32_t pB = a.nd.ld * 4u, pT = a.nd.ld * (uint32_t)sizeof(T), oT = lane_off(t, t.jv, a.nd.ld, j, sizeof(T));
    const RowWin ws = row_win(src, r0, t.rows, pT);
    const uint32_t oB = lane_off(t, t.jv, a.nd.ld, j, 4);
    float val[R];
    int s = r0 % a.rp.S;
#pragma unroll
    for (int q = 0; q < R; ++q) {
      val[q] = 0.f;
      if (bcast) val[q] += win_ld<float>(row_win(bcast, s, 1, pB), oB);
      if (src) val[q] += from_t<T>(win_ld<T>(ws, oT + q * pT));
      s = s + 1 == a.rp.S ? 0 : s + 1;
    }
    fetch_pre<T>(epi, t, p);
    float sG[R], sH[R], sQ[R];
    tile_cuts(a.cc, a.rp, t, p, sG, sH, sQ);
    const RowWin w = row_win(a.lam_out, r0, t.rows, pT);
    epi.tile(val, p, t, sG, sH, sQ, rs, partial != nullptr, [&](int q, T v) { win_st<T>(w, oT + q * pT, v); });
    if (!partial) return;      // the row constants are not asked for
  } else {
    LaneCoords<R, 1, false> lc;
#pragma unroll
    for (int q = 0; q < R; ++q) lc.r[q] = r0 + q;
    lc.j[0][0] = j;
    float val[1][R];
#pragma unroll
    for (int q = 0; q < R; ++q) {
      const int r = r0 + q;
      float pre = 0.f;
      if (j < a.nd.size && r < M) {
        if (bcast) pre += bcast[(size_t)(r % a.rp.S) * a.nd.ld + j];
        if (src) pre += from_t<T>(((const T*)src)[(size_t)r * a.nd.ld + j]);
      }
      val[0][q] = pre;
    }
    typename BoundEpi<T, PI>::template Frag<R, 1, false> fr;
    epi.template load<R, 1, false>(fr, lc, M, a.nd.size);
    if (!partial) {            // the row constants are not asked for: rs is dead here
      epi.template apply<R, 1, false>(fr, lc, val, rs, M, a.nd.size);
      return;
    }
    epi.template apply<R, 1, false>(fr, lc, val, rs, M, a.nd.size);
  }
#pragma unroll
  for (int q = 0; q < R; ++q) {
    const double t = wave_sum64(rs[q]);
    if ((tx & 63) == 0) red[q][tx >> 6] = t;
  }
  __syncthreads();
  if (tx < R) {
    const int q = tx, r = r0 + q;
    if (r < M) partial[(size_t)(slot0 + cb) * a.rp.mp + r] = (red[q][0] + red[q][1]) + (red[q][2] + red[q][3]);
  }
}

}  // namespace gcp
