// Convolution edges of the GCP-CROWN passes as implicit GEMMs on MFMA.
//
// Bound direction (a_hat^(src) = Lambda^(node) A, A the conv's matrix): a
// transposed convolution.  Output position (y, x) of the source grid meets
// the node grid only through taps with ky = (y + pad) mod s (+ s a) and
// likewise for kx, so the positions split into s^2 phases; within a phase
// every tap is real and
//   a_hat[c][y][x] = sum_(o,a,b) Lambda[o][Yb - a][Xb - b] Wph[c][(o,a,b)],
//   Yb = (y + pad - ry) / s,  Xb = (x + pad - rx) / s.
// Adjoint direction (dLambda^(node) = A da_hat^(src)): a convolution,
//   out[o][y][x] = sum_(c,ky,kx) X[c][y s - pad + ky][x s - pad + kx] W[o][(c,ky,kx)].
//
// Both are "slab GEMMs": one workgroup takes four consecutive batch rows and
// one band of output rows.  The source rows the band reads go to LDS with the
// four batch rows innermost ("cells" of four values, zero halo, so the inner
// loop has no bounds checks): one 16-byte LDS read at base(position) +
// koff(k) is then the A operand of four MFMAs, one per batch row, which share
// the K offsets and the weight fragment.  B fragments (weights, K contiguous)
// are read from global memory, where the few KB of weights stay cached.  The
// accumulators stay in registers until every wave is done with the slab, and
// the band's results (cells again) take its place in LDS.
//
// Epilogue: most neurons of a convolutional node are stable under the root
// bounds and have no cut, so their relaxation is a copy or a zero.  The full
// epilogue therefore runs over the band's list of unstable (or cut) neurons
// only, one neuron of the four batch rows per lane, and leaves its results in
// LDS; a streaming pass then writes the whole band, four neurons of a row per
// 16-byte store.  The row constant of a band goes to one partial slot per
// batch row: slot0 + band.
//
// What bounds them: a workgroup's phases (slab, products, lists, streaming)
// follow one another and two workgroups per CU overlap them little, so their
// times add up.  Against the form with one batch row at a time (RB = 1, below),
// the CNN's kernels at 18432 rows in fp32: relaxation 670 -> 326 us, adjoint
// 745 -> 437, adjoint from the sign matrix 706 -> 312.
//
// The earlier form (one batch row in the slab at a time, element gathers of 4
// bytes, the full epilogue over every neuron) is kept as RB = 1 with the same
// epilogue, for convolutions whose rows are too wide for four slabs.
#include "gcp_internal.h"
#include "epilogues.h"

#include <hip/hip_runtime.h>

#include <algorithm>

namespace gcp {

namespace {
constexpr int kRows = 4;                 // batch rows per workgroup
constexpr int kItems = 16;               // MFMA items (16 positions x 16 channels) of a band, at most
constexpr int kIT = 2;                   // items whose accumulators a wave holds at once
// LDS of the slab or the results: two workgroups per CU (160 KB), else one.
// Higher bands re-read fewer halo rows and spread a workgroup's fixed costs:
// three workgroups per CU (52 KB) measured 11.3 ms against 9.95 ms for one
// gradient call of the 3x32x32 ResNet at 9216 rows (38.2 against 38.1 ms for
// the CNN's ascent), four (36 KB) 13.6.
constexpr int kSlabBudget[] = {78 * 1024, 150 * 1024};
constexpr int kRowBudget = 48 * 1024;    // the one-row plan: slab + result bands (4 bytes an element)
constexpr int kRowLds = 64 * 1024;       // and what it may use with its tables
constexpr int kLdsLimit = 160 * 1024;
constexpr int kDirNW = 4;                // waves per workgroup of the direct transposed conv
constexpr int kDirSlab = 24 * 1024;      // and the slab bytes it stages at a time
__host__ __device__ inline int align16(int b) { return (b + 15) & ~15; }

// e / d and the remainder through a float quotient (0 <= e < 2^24): within
// one of the result, then corrected
__device__ inline int div_rem(int e, int d, float inv, int* rem) {
  int n = (int)((float)e * inv), r = e - n * d;
  if (r < 0) { --n; r += d; } else if (r >= d) { ++n; r -= d; }
  *rem = r;
  return n;
}
}  // namespace

// Rows of phase ph inside band [yb0, yb1): source-side positions
// (yf + st*iy, xf + st*ix), iy < ny, ix < nx, st = s for the transposed
// direction (one phase per residue of y + pad and x + pad mod s), else 1.
__host__ __device__ inline void phase_rows(const ConvPlan& P, int ph, int yb0, int yb1, bool trans, int* yf, int* ny,
                                           int* xf, int* nx) {
  if (trans) {
    const int s = P.s, p = P.p, ry = ph / s, rx = ph % s;
    *yf = yb0 + (((ry - (yb0 + p)) % s) + s) % s;
    *ny = *yf < yb1 ? (yb1 - 1 - *yf) / s + 1 : 0;
    *xf = (((rx - p) % s) + s) % s;
    *nx = *xf < P.We ? (P.We - 1 - *xf) / s + 1 : 0;
  } else {
    *yf = yb0; *ny = yb1 - yb0; *xf = 0; *nx = P.We;
  }
}

static ConvPlan plan_dims(const ConvGeom& g, int trans) {
  ConvPlan P{};
  const int s = g.stride;
  P.s = s;
  P.p = g.pad;
  if (trans) {
    P.He = g.hi; P.We = g.wi; P.Nch = g.ci; P.Kch = g.co; P.hs = g.ho; P.ws = g.wo;
    P.A = (g.kh + s - 1) / s;
    P.Bn = (g.kw + s - 1) / s;
    P.n_phase = s * s;
    P.Kreal = g.co * P.A * P.Bn;
    P.xl = P.Bn - 1;
    const int xmax = (g.wi - 1 + g.pad) / s;           // largest Xb
    P.Wp = P.xl + std::max(xmax + 1, g.wo);
  } else {
    P.He = g.ho; P.We = g.wo; P.Nch = g.co; P.Kch = g.ci; P.hs = g.hi; P.ws = g.wi;
    P.A = g.kh;
    P.Bn = g.kw;
    P.n_phase = 1;
    P.Kreal = g.ci * g.kh * g.kw;
    P.xl = g.pad;
    P.Wp = P.xl + std::max(g.wi, (g.wo - 1) * s - g.pad + g.kw);
  }
  P.KP = (P.Kreal + 31) / 32 * 32;
  return P;
}

// Split the epilogue-side rows into bands of at most bh rows.
static void plan_bands(ConvPlan& P, int trans, int bh) {
  P.n_bands = (P.He + bh - 1) / bh;
  P.BH = (P.He + P.n_bands - 1) / P.n_bands;           // balance the bands
  P.rows_max = trans ? (P.BH - 1 + P.s - 1) / P.s + P.A : (P.BH - 1) * P.s + P.A;
  P.CHS = P.rows_max * P.Wp;
  P.OS = P.BH * P.We + 1;                              // odd: channel planes on different banks
  P.MT = 0;
  for (int b = 0; b < P.n_bands; ++b) {
    const int yb0 = b * P.BH, yb1 = std::min(P.He, yb0 + P.BH);
    int nt = 0;
    for (int ph = 0; ph < P.n_phase; ++ph) {
      int yf, ny, xf, nx;
      phase_rows(P, ph, yb0, yb1, trans != 0, &yf, &ny, &xf, &nx);
      nt += (ny * nx + 15) / 16;
    }
    P.MT = std::max(P.MT, nt);
  }
}

// What a slab launch's workgroup looks up, laid out once per net and band as
// it lies in LDS: the slab offset of each K index relative to a GEMM row's
// base [KP], base (low half) and result offset (high half, 0xffff: none) of
// each GEMM row [16 MT], phase of each 16-row tile [MT] and the number of
// tiles.  Made by every workgroup, with their integer divisions, these were
// part of what a workgroup costs apart from its data: the ascent of the
// 3x32x32 ResNet, 4608 rows in bf16, 72.1 -> 66.9 ms (with the lists walked as
// one, by the dense layers' branch-free loads).
__host__ __device__ static inline int table_words(const ConvPlan& P) { return P.KP + 16 * P.MT + (P.MT + 1 + 3) / 4 * 4; }
std::vector<int32_t> conv_tables(const ConvPlan& P, int trans) {
  const int words = table_words(P);
  std::vector<int32_t> all((size_t)words * P.n_bands, 0);
  const int s = P.s, p = P.p;
  const int safe_base = trans ? (P.A - 1) * P.Wp + P.Bn - 1 : 0;    // in-slab for every K offset
  for (int band = 0; band < P.n_bands; ++band) {
    int32_t *koff = all.data() + (size_t)band * words, *desc = koff + P.KP, *tph = desc + 16 * P.MT;
    for (int k = 0; k < P.Kreal; ++k) {
      const int ch = k / (P.A * P.Bn), a = (k / P.Bn) % P.A, b = k % P.Bn;
      koff[k] = trans ? ch * P.CHS - a * P.Wp - b : ch * P.CHS + a * P.Wp + b;
    }
    std::fill(desc, desc + 16 * P.MT, (int32_t)((uint32_t)safe_base | 0xffff0000u));
    const int yb0 = band * P.BH, yb1 = std::min(P.He, yb0 + P.BH);
    const int sy0 = trans ? (yb0 + p) / s - (P.A - 1) : yb0 * s - p;   // source row of slab row 0
    int ntile = 0;
    // GEMM rows of the band, phase by phase, each phase padded to whole tiles
    for (int ph = 0; ph < P.n_phase; ++ph) {
      int yf, ny, xf, nx;
      phase_rows(P, ph, yb0, yb1, trans != 0, &yf, &ny, &xf, &nx);
      const int npos = ny * nx, nt = (npos + 15) / 16, ry = ph / s, rx = ph % s;
      const int base0 = trans ? ((yf + p - ry) / s - sy0) * P.Wp + (xf + p - rx) / s + P.xl
                              : (yf * s - p - sy0) * P.Wp + xf * s - p + P.xl;
      const int rstep = trans ? P.Wp : s * P.Wp, cstep = trans ? 1 : s, st = trans ? s : 1;
      const int out0 = (yf - yb0) * P.We + xf;
      for (int i = 0; i < npos; ++i) {
        const int iy = i / nx, ix = i - iy * nx;
        desc[ntile * 16 + i] = (int32_t)((uint32_t)(base0 + iy * rstep + ix * cstep) |
                                         ((uint32_t)(out0 + iy * st * P.We + ix * st) << 16));
      }
      for (int i = 0; i < nt; ++i) tph[ntile + i] = ph;
      ntile += nt;
    }
    tph[P.MT] = ntile;
  }
  return all;
}

// The direct transposed conv: shapes it is built for, the 64-position chunks
// of a band (at most), and the channels it stages at a time.
static bool direct_shape(const ConvPlan& P) {
  return (P.A == 2 && P.Bn == 2 && P.s == 2) || (P.A == 3 && P.Bn == 3 && P.s == 1);
}
static int direct_chunks(const ConvPlan& P) {
  int most = 0;
  for (int b = 0; b < P.n_bands; ++b) {
    const int yb0 = b * P.BH, yb1 = std::min(P.He, yb0 + P.BH);
    int n = 0;
    for (int ph = 0; ph < P.n_phase; ++ph) {
      int yf, ny, xf, nx;
      phase_rows(P, ph, yb0, yb1, true, &yf, &ny, &xf, &nx);
      n += (ny * nx + 63) / 64;
    }
    most = std::max(most, n);
  }
  return most;
}
static int direct_kch(const ConvPlan& P) {
  return std::min(P.Kch, std::max(1, kDirSlab / (16 * P.CHS)));
}
static int conv_direct_lds_bytes(const ConvPlan& P) {   // reduction slots, the staged channels or the results
  return align16(kDirNW * 8 * kRows) + 16 * std::max(direct_kch(P) * P.CHS, P.Nch * P.OS);
}

static long slab_cells(const ConvPlan& P) { return (long)P.Kch * P.CHS; }
static long out_cells(const ConvPlan& P) { return (long)P.Nch * P.OS; }
static int plan_items(const ConvPlan& P) { return P.MT * ((P.Nch + 15) / 16); }

// Whether a launch of nw waves and tn column tiles per wave holds every item
// of a band in its accumulators, so that the results may replace the slab.
static bool conv_alias(const ConvPlan& P, int nw, int tn) {
  return P.rb == 4 && P.MT * ((P.Nch + 16 * tn - 1) / (16 * tn)) <= nw * kIT;
}

static int conv_lds_bytes(const ConvPlan& P, int esz, int nw, bool alias) {
  const int slab = align16(P.rb * (int)slab_cells(P) * esz), outs = align16((int)out_cells(P) * 16);
  return align16(nw * 8 * kRows) + table_words(P) * 4 +
         (alias ? std::max(slab, outs) : slab + outs);
}

// What a launch takes (every shape of workgroup asks for at most this much):
// its LDS within a workgroup's, at the operand's size, and the slab and result
// offsets in the halves of a descriptor (conv_tables).
bool conv_fits(const ConvPlan& P, int bf16) {
  const bool alias = conv_alias(P, 8, 1);
  return conv_lds_bytes(P, bf16 ? 2 : 4, P.rb == 1 ? 4 : 8, alias) <= kLdsLimit && P.CHS < 0xffff &&
         P.BH * P.We < 0xffff;
}

// The plan that holds one batch row in the slab.
static ConvPlan conv_plan_row(const ConvGeom& g, int trans) {
  ConvPlan P = plan_dims(g, trans);
  auto bytes_for = [&](int bh) {
    const long rows = trans ? (bh - 1) / P.s + 1 + P.A : (bh - 1) * P.s + P.A;   // (one more than is read, at times)
    return ((long)P.Kch * rows * P.Wp + (long)kRows * P.Nch * (bh * P.We + 1)) * 4;
  };
  int bh = P.He;
  while (bh > 1 && bytes_for(bh) > kRowBudget) --bh;
  plan_bands(P, trans, bh);
  P.rb = 1;
  return P;
}

// Bands as high as fit (a higher band re-reads fewer halo rows) with the
// slab of four batch rows within the budget of two workgroups per CU, then
// one, and its accumulators within two items per wave.  The budgets count four
// bytes an element for either operand type, so that both run the same bands;
// what a launch asks for beside the slab or the results, the tables above all
// (four bytes per K index), may still not fit: 320 -> 64 channels of 3x3 at
// 8x8 are 150 KB of slab and 11.8 KB of tables in fp32, which takes another
// plan, and half that slab in bf16, which keeps this one.
ConvPlan conv_plan(const ConvGeom& g, int trans, int bf16, bool* by_type) {
  ConvPlan P = plan_dims(g, trans);
  P.rb = 4;
  bool tight = false;
  auto fits = [&] {
    const bool ok = conv_fits(P, bf16);
    tight = tight || !ok;
    return ok;
  };
  auto pick = [&] {
    if (trans && P.Nch <= 4 && direct_shape(P))   // bands of the direct kernel: one 64-position chunk per wave
      for (int bh = P.He; bh >= 1; --bh) {
        plan_bands(P, trans, bh);
        if (direct_chunks(P) <= kDirNW && plan_items(P) <= kItems &&
            16 * std::max(slab_cells(P), out_cells(P)) <= kSlabBudget[1] && fits())
          return true;
      }
    for (long budget : kSlabBudget)
      for (int bh = P.He; bh >= 1; --bh) {
        plan_bands(P, trans, bh);
        if (plan_items(P) <= kItems && 16 * std::max(slab_cells(P), out_cells(P)) <= budget && fits()) return true;
      }
    plan_bands(P, trans, 1);   // more channels or positions than the waves hold: results beside the slab
    return 16 * (slab_cells(P) + out_cells(P)) <= kSlabBudget[1] && fits();
  };
  if (!pick()) P = conv_plan_row(g, trans);
  if (by_type) *by_type = tight;
  return P;
}

long conv_row_slab(const ConvGeom& g, int trans) {
  const ConvPlan P = conv_plan_row(g, trans);
  const long rows = trans ? (P.BH - 1) / P.s + 1 + P.A : P.rows_max;
  return (long)P.Kch * rows * P.Wp * 4;
}

int conv_ldb(const ConvGeom& g, int trans) { return plan_dims(g, trans).KP; }

void conv_pack_weights(const ConvGeom& g, int trans, const float* raw, float* out) {
  const ConvPlan P = plan_dims(g, trans);
  const int ldb = P.KP, s = g.stride;
  auto w = [&](int o, int c, int ky, int kx) { return raw[(((size_t)o * g.ci + c) * g.kh + ky) * g.kw + kx]; };
  if (!trans) {
    for (int o = 0; o < g.co; ++o)
      for (int k = 0; k < ldb; ++k) {
        float v = 0.f;
        if (k < P.Kreal) {
          const int c = k / (g.kh * g.kw), ky = (k / g.kw) % g.kh, kx = k % g.kw;
          v = w(o, c, ky, kx);
        }
        out[(size_t)o * ldb + k] = v;
      }
    return;
  }
  for (int ph = 0; ph < P.n_phase; ++ph) {
    const int ry = ph / s, rx = ph % s;
    for (int c = 0; c < g.ci; ++c)
      for (int k = 0; k < ldb; ++k) {
        float v = 0.f;
        if (k < P.Kreal) {
          const int o = k / (P.A * P.Bn), a = (k / P.Bn) % P.A, b = k % P.Bn;
          const int ky = ry + s * a, kx = rx + s * b;
          if (ky < g.kh && kx < g.kw) v = w(o, c, ky, kx);
        }
        out[((size_t)ph * g.ci + c) * ldb + k] = v;
      }
  }
}

// ---------------------------------------------------------------- slab fill
// V consecutive source elements of one batch row as fp32 values.
template <typename T, bool SIGN, int V>
__device__ inline void load_vals(const void* X, size_t off, float* d) {
  if constexpr (SIGN) {
    int8_t e[V];
    if constexpr (V == 4) *(uint32_t*)e = *(const uint32_t*)((const int8_t*)X + off);
    else e[0] = ((const int8_t*)X)[off];
#pragma unroll
    for (int q = 0; q < V; ++q) d[q] = (float)e[q];
  } else if constexpr (sizeof(T) == 4) {
    if constexpr (V == 4) *(float4*)d = *(const float4*)((const float*)X + off);
    else d[0] = ((const float*)X)[off];
  } else {
    if constexpr (V == 4) {
      const uint2 v = *(const uint2*)((const bf16*)X + off);
      d[0] = __uint_as_float(v.x << 16); d[1] = __uint_as_float(v.x & 0xffff0000u);
      d[2] = __uint_as_float(v.y << 16); d[3] = __uint_as_float(v.y & 0xffff0000u);
    } else {
      d[0] = (float)((const bf16*)X)[off];
    }
  }
}

// A slab cell: the values of RB batch rows at one source position, C the
// element type (the operand type, or fp32 in the direct kernel).
template <typename C, int RB> struct Cell;
template <> struct Cell<float, 4> {
  typedef float4 type;
  __device__ static inline type make(float a, float b, float c, float d) { return float4{a, b, c, d}; }
};
template <> struct Cell<bf16, 4> {
  typedef uint2 type;
  __device__ static inline type make(float a, float b, float c, float d) {
    bf16 e[4] = {(bf16)a, (bf16)b, (bf16)c, (bf16)d};
    return *(const uint2*)e;
  }
};
template <typename C> struct Cell<C, 1> {
  typedef C type;
  __device__ static inline type make(float a, float, float, float) { return (C)a; }
};

// Source rows sy0 .. sy0 + rows_max - 1 of channels c0 .. c0 + nch - 1 of
// batch rows r0 .. r0 + RB - 1 into the slab, zeros outside the source and
// past row M.
template <typename T, bool SIGN, typename C, int RB, int NT>
__device__ __forceinline__ void stage_slab(const ConvArgs& c, const ConvPlan& P, typename Cell<C, RB>::type* slab, int r0,
                                           int sy0, int c0, int nch) {
  const int tid = threadIdx.x;
  auto fill = [&](auto vc) {
    constexpr int V = decltype(vc)::value;
    const int nchunk = P.ws / V;
    const int total = nch * P.rows_max * nchunk;
    const float inv_c = 1.f / (float)nchunk, inv_r = 1.f / (float)P.rows_max;
    // two items per step, so that their loads are in flight together
    for (int v0 = tid; v0 < total; v0 += 2 * NT) {
      float d[2][4][V];
      int cell[2];
#pragma unroll
      for (int u = 0; u < 2; ++u) {
        const int v = v0 + u * NT;
        int xc, rho;
        const int ch = div_rem(div_rem(v, nchunk, inv_c, &xc), P.rows_max, inv_r, &rho);
        const int sy = sy0 + rho;
        cell[u] = ch * P.CHS + rho * P.Wp + P.xl + xc * V;
#pragma unroll
        for (int q = 0; q < 4; ++q)
#pragma unroll
          for (int e = 0; e < V; ++e) d[u][q][e] = 0.f;
        if (v < total && sy >= 0 && sy < P.hs) {
          const size_t src = (size_t)r0 * c.ldx + ((size_t)(c0 + ch) * P.hs + sy) * P.ws + (size_t)xc * V;
#pragma unroll
          for (int q = 0; q < RB; ++q)
            if (r0 + q < c.M) load_vals<T, SIGN, V>(c.X, src + (size_t)q * c.ldx, d[u][q]);
        }
      }
#pragma unroll
      for (int u = 0; u < 2; ++u) {
        if (v0 + u * NT >= total) break;
#pragma unroll
        for (int e = 0; e < V; ++e)
          slab[cell[u] + e] = Cell<C, RB>::make(d[u][0][e], d[u][1][e], d[u][2][e], d[u][3][e]);
      }
    }
  };
  if (P.ws % 4 == 0) fill(std::integral_constant<int, 4>{});
  else fill(std::integral_constant<int, 1>{});
  const int nh = P.Wp - P.ws;   // halo columns
  if (nh > 0) {
    const int total = nch * P.rows_max * nh;
    const float inv_h = 1.f / (float)nh;
    for (int v = tid; v < total; v += NT) {
      int hx;
      const int row = div_rem(v, nh, inv_h, &hx);   // ch * rows_max + rho; CHS = rows_max * Wp
      slab[row * P.Wp + (hx < P.xl ? hx : hx + P.ws)] = Cell<C, RB>::make(0.f, 0.f, 0.f, 0.f);
    }
  }
}

// The A fragments of RB batch rows: VEC consecutive K indices of a lane's
// GEMM row, gathered from the slab (uint4 in the MFMA operand layout).
template <typename T, int RB> struct Gather;
template <> struct Gather<float, 4> {
  __device__ static inline void get(const float4* slab, int base, const int* ko, uint4 (&fa)[4]) {
    const float4 k0 = slab[base + ko[0]], k1 = slab[base + ko[1]], k2 = slab[base + ko[2]], k3 = slab[base + ko[3]];
    fa[0] = uint4{__float_as_uint(k0.x), __float_as_uint(k1.x), __float_as_uint(k2.x), __float_as_uint(k3.x)};
    fa[1] = uint4{__float_as_uint(k0.y), __float_as_uint(k1.y), __float_as_uint(k2.y), __float_as_uint(k3.y)};
    fa[2] = uint4{__float_as_uint(k0.z), __float_as_uint(k1.z), __float_as_uint(k2.z), __float_as_uint(k3.z)};
    fa[3] = uint4{__float_as_uint(k0.w), __float_as_uint(k1.w), __float_as_uint(k2.w), __float_as_uint(k3.w)};
  }
};
template <> struct Gather<bf16, 4> {
  __device__ static inline void get(const uint2* slab, int base, const int* ko, uint4 (&fa)[4]) {
    uint32_t w[4][4];
#pragma unroll
    for (int p = 0; p < 4; ++p) {
      const uint2 a = slab[base + ko[2 * p]], b = slab[base + ko[2 * p + 1]];
      w[0][p] = __builtin_amdgcn_perm(b.x, a.x, 0x05040100u);
      w[1][p] = __builtin_amdgcn_perm(b.x, a.x, 0x07060302u);
      w[2][p] = __builtin_amdgcn_perm(b.y, a.y, 0x05040100u);
      w[3][p] = __builtin_amdgcn_perm(b.y, a.y, 0x07060302u);
    }
#pragma unroll
    for (int q = 0; q < 4; ++q) fa[q] = uint4{w[q][0], w[q][1], w[q][2], w[q][3]};
  }
};
template <> struct Gather<float, 1> {
  __device__ static inline void get(const float* slab, int base, const int* ko, uint4 (&fa)[1]) {
    const uint32_t* S = (const uint32_t*)slab;
    fa[0] = uint4{S[base + ko[0]], S[base + ko[1]], S[base + ko[2]], S[base + ko[3]]};
  }
};
template <> struct Gather<bf16, 1> {
  __device__ static inline void get(const bf16* slab, int base, const int* ko, uint4 (&fa)[1]) {
    const unsigned short* S = (const unsigned short*)slab;
    uint32_t w[4];
#pragma unroll
    for (int q = 0; q < 4; ++q)
      w[q] = (uint32_t)S[base + ko[2 * q]] | ((uint32_t)S[base + ko[2 * q + 1]] << 16);
    fa[0] = uint4{w[0], w[1], w[2], w[3]};
  }
};

// ---------------------------------------------------------------- band epilogue
// Where the full epilogue leaves its value of a listed neuron: the neuron's
// cell in the band's results.
template <typename T>
struct BandSink {
  float* cell;
  int r0;
  __device__ inline void operator()(size_t, int row, int, T v) const { cell[row - r0] = from_t<T>(v); }
};

// V values of one row as operand-type outputs at dst (16- or 8-byte aligned for V = 4)
template <typename T, int V>
__device__ inline void put(T* dst, const float (&v)[V]) {
  if constexpr (V == 4 && sizeof(T) == 4) {
    *(float4*)dst = float4{v[0], v[1], v[2], v[3]};
  } else if constexpr (V == 4 && sizeof(T) == 2) {
    T e[4] = {to_t<T>(v[0]), to_t<T>(v[1]), to_t<T>(v[2]), to_t<T>(v[3])};
    *(uint2*)dst = *(const uint2*)e;
  } else {
#pragma unroll
    for (int k = 0; k < V; ++k) dst[k] = to_t<T>(v[k]);
  }
}
template <int V>
__device__ inline void get_f32(const float* src, float (&v)[V]) {
  if constexpr (V == 4) *(float4*)v = *(const float4*)src;
  else v[0] = src[0];
}
// V accumulated values (fp32, or the operand type when acc_t)
template <typename T, int V>
__device__ inline void get_acc(const void* acc, int acc_t, size_t i, float (&v)[V]) {
  if (sizeof(T) == 2 && acc_t) load_vals<T, false, V>(acc, i, v);
  else get_f32<V>((const float*)acc + i, v);
}
// kind words of V neurons; the bit kListed is set for those the band's lists
// hold (their values in LDS are final)
constexpr int kListed = 1 << 30;
template <int V>
__device__ inline void get_kind(const NodeDev& nd, const CutCol& cc, int j, int (&kv)[V]) {
  if constexpr (V == 4) *(int4*)kv = *(const int4*)(nd.kind + j);
  else kv[0] = nd.kind[j];
#pragma unroll
  for (int k = 0; k < V; ++k) {
    if (kind_rank(kv[k]) >= 0) kv[k] |= kListed;
    else if (cc.stable && cc.stable[j + k]) kv[k] |= kListed;
  }
}

// What the epilogues do with a band: `run` handles one listed neuron of the
// four batch rows (its cell in LDS), `stream` V consecutive neurons j .. of
// the four rows, v[k][q] neuron k of row q.
template <class Epi> struct BandOps;

template <typename T, bool PI>
struct BandOps<BoundEpi<T, PI>> {
  static constexpr bool kLists = true, kStream = true;
  template <class LC, class Pre>
  __device__ static inline void run(const BoundEpi<T, PI>& e, const LC& lc, const Pre& pre, const float (&val)[1][kRows],
                                    float* cell, int r0, int M, int size, double (&rs)[kRows]) {
    typename BoundEpi<T, PI>::template Frag<kRows, 1, false> fr;
    e.template load<kRows, 1, false>(fr, lc, M, size, &pre);
    e.template apply_to<kRows, 1, false>(fr, lc, val, rs, M, size, BandSink<T>{cell, r0});
  }
  template <int V>
  __device__ static inline void stream(const BoundEpi<T, PI>& e, int j, const float (&v)[V][kRows], int r0, int M, bool want,
                                       double (&rs)[kRows]) {
    const NodeDev& nd = e.a.nd;
    int kv[V];
    float bj[V], pre[kRows][V];
    get_kind<V>(nd, e.a.cc, j, kv);
    if (want) get_f32<V>(nd.bias + j, bj);
    if (e.a.acc_in) {
#pragma unroll
      for (int q = 0; q < kRows; ++q)
        if (r0 + q < M) get_acc<T, V>(e.a.acc_in, e.a.acc_t, (size_t)(r0 + q) * nd.ld + j, pre[q]);
    }
#pragma unroll
    for (int q = 0; q < kRows; ++q) {
      if (r0 + q >= M) break;
      float o[V];
#pragma unroll
      for (int k = 0; k < V; ++k) {
        const float ah = v[k][q] + (e.a.acc_in ? pre[q][k] : 0.f);
        o[k] = kv[k] & kListed ? v[k][q] : (kind_cls(kv[k]) == ACTIVE ? ah : 0.f);
        if (want && !(kv[k] & kListed)) rs[q] += (double)o[k] * (double)bj[k];
      }
      put<T, V>((T*)e.a.lam_out + (size_t)(r0 + q) * nd.ld + j, o);
    }
  }
};

template <typename T>
struct BandOps<AhatEpi<T>> {
  static constexpr bool kLists = true, kStream = false;
  template <class LC, class Pre>
  __device__ static inline void run(const AhatEpi<T>& e, const LC& lc, const Pre& pre, const float (&val)[1][kRows],
                                    float*, int, int M, int size, double (&rs)[kRows]) {
    typename AhatEpi<T>::template Frag<kRows, 1, false> fr;
    e.template load<kRows, 1, false>(fr, lc, M, size, &pre);
    e.template apply<kRows, 1, false>(fr, lc, val, rs, M, size);
  }
};

template <typename T, bool PI>
struct BandOps<AdjEpi<T, PI>> {
  static constexpr bool kLists = true, kStream = true;
  template <class LC, class Pre>
  __device__ static inline void run(const AdjEpi<T, PI>& e, const LC& lc, const Pre& pre, const float (&val)[1][kRows],
                                    float* cell, int r0, int M, int size, double (&rs)[kRows]) {
    typename AdjEpi<T, PI>::template Frag<kRows, 1, false> fr;
    e.template load<kRows, 1, false>(fr, lc, M, size, &pre);
    e.template apply_to<kRows, 1, false>(fr, lc, val, rs, M, size, BandSink<T>{cell, r0});
  }
  template <int V>
  __device__ static inline void stream(const AdjEpi<T, PI>& e, int j, const float (&v)[V][kRows], int r0, int M, bool want,
                                       double (&rs)[kRows]) {
    if (!e.a.dahat_out) return;
    const NodeDev& nd = e.a.nd;
    int kv[V];
    float addj[V], pre[kRows][V];
    get_kind<V>(nd, e.a.cc, j, kv);
    get_f32<V>(e.a.add_vec + j, addj);
    if (e.a.acc_in) {
#pragma unroll
      for (int q = 0; q < kRows; ++q)
        if (r0 + q < M) get_acc<T, V>(e.a.acc_in, e.a.acc_t, (size_t)(r0 + q) * nd.ld + j, pre[q]);
    }
#pragma unroll
    for (int q = 0; q < kRows; ++q) {
      if (r0 + q >= M) break;
      float o[V];
#pragma unroll
      for (int k = 0; k < V; ++k) {
        const float dL = e.a.gemm_scale * v[k][q] + addj[k] + (e.a.acc_in ? pre[q][k] : 0.f);
        o[k] = kv[k] & kListed ? v[k][q] : (kind_cls(kv[k]) == ACTIVE ? dL : 0.f);
      }
      put<T, V>((T*)e.a.dahat_out + (size_t)(r0 + q) * nd.ld + j, o);
    }
  }
};

template <> struct BandOps<StoreEpi> {
  static constexpr bool kLists = false, kStream = true;
  template <int V>
  __device__ static inline void stream(const StoreEpi& e, int j, const float (&v)[V][kRows], int r0, int M, bool want,
                                       double (&rs)[kRows]) {
    float pre[kRows][V];
    if (e.a.acc_in) {
#pragma unroll
      for (int q = 0; q < kRows; ++q)
        if (r0 + q < M) get_f32<V>(e.a.acc_in + (size_t)(r0 + q) * e.a.ld + j, pre[q]);
    }
#pragma unroll
    for (int q = 0; q < kRows; ++q) {
      if (r0 + q >= M) break;
      float o[V];
#pragma unroll
      for (int k = 0; k < V; ++k) o[k] = e.a.scale * v[k][q] + (e.a.acc_in ? pre[q][k] : 0.f);
      put<float, V>(e.a.out + (size_t)(r0 + q) * e.a.ld + j, o);
    }
  }
};

// The input: the list holds the coordinates with cut entries, whose cell
// becomes v = GEMM + gamma^T G0.
template <> struct BandOps<ConcEpi> {
  static constexpr bool kLists = true, kStream = true;
  template <class LC, class Pre>
  __device__ static inline void run(const ConcEpi& e, const LC& lc, const Pre& pre, const float (&val)[1][kRows],
                                    float* cell, int r0, int M, int size, double (&)[kRows]) {
    int rr[kRows], rc[kRows], jq[kRows];
    bool rv[kRows], jv[kRows];
    lane_rows<kRows, false>(lc.r, M, e.a.rp.mp, rr, rc, rv);
    const int j = lc.j[0][0];
#pragma unroll
    for (int q = 0; q < kRows; ++q) { jq[q] = j; jv[q] = true; }
    float sG[kRows], sH[kRows], sQ[kRows];
    gather_cuts<kRows, false>(e.a.cc, e.a.rp.gammaT, e.a.rp.mp, jq, jv, rr, sG, sH, sQ, &pre.rng[0]);
    const double xj = e.a.x0[j];
#pragma unroll
    for (int q = 0; q < kRows; ++q) {
      const float v = val[0][q] + sG[q];
      cell[q] = v;
      if (!e.a.contrib || !rv[q]) continue;
      const float sg = (v > 0.f) ? 1.f : ((v < 0.f) ? -1.f : 0.f);
      const float dv = (float)(xj - e.a.eps * (double)sg);
      for (int i = pre.rng[0].x; i < pre.rng[0].y; ++i)
        e.a.contrib[(size_t)e.a.cc.pos[i] * e.a.rp.mp + rr[q]] = e.a.cc.ent[i].y * dv;
    }
  }
  template <int V>
  __device__ static inline void stream(const ConcEpi& e, int j, const float (&v)[V][kRows], int r0, int M, bool want,
                                       double (&rs)[kRows]) {
    double xj[V];
#pragma unroll
    for (int k = 0; k < V; ++k) xj[k] = want ? e.a.x0[j + k] : 0.0;
#pragma unroll
    for (int q = 0; q < kRows; ++q) {
      if (r0 + q >= M) break;
      int8_t sg[V];
#pragma unroll
      for (int k = 0; k < V; ++k) {
        const double vd = (double)v[k][q];
        if (want) rs[q] += xj[k] * vd - e.a.eps * fabs(vd);
        sg[k] = (v[k][q] > 0.f) ? 1 : ((v[k][q] < 0.f) ? -1 : 0);
      }
      if (!e.a.sign_out) continue;
      int8_t* dst = e.a.sign_out + (size_t)(r0 + q) * e.a.ld + j;
      if constexpr (V == 4) *(uint32_t*)dst = *(const uint32_t*)sg;
      else dst[0] = sg[0];
    }
  }
};

// An epilogue by its 64-bit form (arrays too large for the windows of
// fetch_pre: windows_wide).
template <class E> struct Wide : E {
  static constexpr int kPre = 0;
};
template <class E> struct BandOps<Wide<E>> : BandOps<E> {};

template <class Epi>
__device__ inline const CutCol& band_cuts(const Epi& e) { return e.a.cc; }

// The band's lists as one: the unstable neurons, then the stable ones with
// cut entries; entry i < n is {neuron, kind}.
struct BandList {
  const int2 *uns, *cut;
  int n_u, n;
  __device__ inline BandList(const ConvArgs& c, int band) {
    const int u0 = c.uns ? c.uns_off[band] : 0, c0 = c.cut ? c.cut_off[band] : 0;
    uns = c.uns + u0;
    cut = c.cut + c0;
    n_u = c.uns ? c.uns_off[band + 1] - u0 : 0;
    n = n_u + (c.cut ? c.cut_off[band + 1] - c0 : 0);
  }
  __device__ inline int2 at(int i) const { return i < n_u ? uns[i] : cut[i - n_u]; }
};

// Fused epilogue of one workgroup's band over the results of its kRows batch
// rows in LDS (cell n * OS + position of channel n; position (y - yb0) * We +
// x), then the row constant of each batch row into its partial slot slot0 +
// band.  (A thread's first list entry fetched ahead of the slab measured the
// same as here: two workgroups per CU cover these loads.)
template <typename T, int NW, class Epi>
__device__ __forceinline__ void band_epilogue(const ConvArgs& c, const ConvPlan& P, const Epi& epi, float4* outs,
                                              double* red, int r0, int band, int yb0, int yb1) {
  constexpr int NT = NW * 64;
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int HWe = P.He * P.We;
  const int size = P.Nch * HWe;
  const int j0 = yb0 * P.We;
  double rs[kRows];
#pragma unroll
  for (int q = 0; q < kRows; ++q) rs[q] = 0.0;
  if constexpr (BandOps<Epi>::kLists) {
    const float inv_hw = 1.f / (float)HWe;
    const BandList list(c, band);
    const int2* rng = band_cuts(epi).rng;
    for (int i = tid; i < list.n; i += NT) {
      const int2 e = list.at(i);
      int off;
      const int n = div_rem(e.x, HWe, inv_hw, &off);
      float4& cell = outs[n * P.OS + off - j0];
      const float4 v = cell;
      if constexpr (Epi::kPre > 0) {
        const TileLane t{r0, min(kRows, c.M - r0), 0, e.x, e.x, true};
        SubPre p;
        p.kind = e.y;
        p.rng = rng ? rng[e.x] : make_int2(0, 0);
        fetch_pre<T>(epi, t, p);
        float sG[4], sH[4], sQ[4];
        tile_cuts(epi.a.cc, epi.a.rp, t, p, sG, sH, sQ);
        const float val[4] = {v.x, v.y, v.z, v.w};
        epi.tile(val, p, t, sG, sH, sQ, rs, c.partial != nullptr, [&](int q, T o) { ((float*)&cell)[q] = from_t<T>(o); });
      } else {
        LaneCoords<kRows, 1, false> lc;
#pragma unroll
        for (int q = 0; q < kRows; ++q) lc.r[q] = r0 + q;
        lc.j[0][0] = e.x;
        ColPre<1> pre;
        pre.kind[0] = e.y;
        pre.rng[0] = rng ? rng[e.x] : make_int2(0, 0);
        const float val[1][kRows] = {{v.x, v.y, v.z, v.w}};
        BandOps<Epi>::run(epi, lc, pre, val, (float*)&cell, r0, c.M, size, rs);
      }
    }
    if constexpr (BandOps<Epi>::kStream) __syncthreads();
  }
  if constexpr (BandOps<Epi>::kStream) {
    const int per_ch = (yb1 - yb0) * P.We;
    auto walk = [&](auto vc) {
      constexpr int V = decltype(vc)::value;
      const int ng = per_ch / V, total = P.Nch * ng;
      const float inv_g = 1.f / (float)ng;
      for (int i = tid; i < total; i += NT) {
        int off;
        const int n = div_rem(i, ng, inv_g, &off);
        off *= V;
        float v[V][kRows];
#pragma unroll
        for (int k = 0; k < V; ++k) *(float4*)v[k] = outs[n * P.OS + off + k];
        BandOps<Epi>::template stream<V>(epi, n * HWe + j0 + off, v, r0, c.M, c.partial != nullptr, rs);
      }
    };
    if (per_ch % 4 == 0 && HWe % 4 == 0 && j0 % 4 == 0) walk(std::integral_constant<int, 4>{});
    else walk(std::integral_constant<int, 1>{});
  }
  if (c.partial) {
#pragma unroll
    for (int q = 0; q < kRows; ++q) {
      const double tsum = wave_sum64(rs[q]);
      if (lane == 0) red[wave * kRows + q] = tsum;
    }
    __syncthreads();
    if (tid < kRows && r0 + tid < c.M) {
      double sum = 0.0;
      for (int w = 0; w < NW; ++w) sum += red[w * kRows + tid];
      c.partial[(size_t)(c.slot0 + band) * c.mp + r0 + tid] = sum;
    }
  }
}

template <typename T, int NW, int TN, int RB, bool TRANS, bool SIGN, class Epi>
__global__ void __launch_bounds__(NW * 64) conv_slab_kernel(ConvArgs c, ConvPlan P, Epi epi, int alias) {
  constexpr int NT = NW * 64;
  constexpr int VEC = Op<T>::VEC;
  constexpr int KC = Op<T>::KC;
  typedef typename Cell<T, RB>::type CellT;
  extern __shared__ __attribute__((aligned(16))) unsigned char smem[];
  unsigned char* sp = smem;
  double* red = (double*)sp;      sp += align16(NW * 8 * kRows);
  // the band's tables (conv_tables): K index -> slab offset; per GEMM row: slab
  // base (low half), result offset (high half, 0xffff: none); per 16-row tile:
  // its phase, then the number of tiles
  const int words = table_words(P);
  int* koff = (int*)sp;           sp += words * 4;
  const uint32_t* desc = (const uint32_t*)(koff + P.KP);
  const int* tph = koff + P.KP + 16 * P.MT;
  CellT* slab = (CellT*)sp;
  float4* outs = (float4*)(alias ? sp : sp + align16(RB * P.Kch * P.CHS * (int)sizeof(T)));

  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int blk = xcd_tile(blockIdx.x, gridDim.x);     // the bands of a row group on one XCD: they share halo rows
  const int r0 = (blk / P.n_bands) * kRows, band = blk % P.n_bands;
  const int s = P.s, p = P.p;
  const int yb0 = band * P.BH, yb1 = min(P.He, yb0 + P.BH);
  const int sy0 = TRANS ? (yb0 + p) / s - (P.A - 1) : yb0 * s - p;   // source row of slab row 0
  const uint4* bt = (const uint4*)(c.tab + (size_t)band * words);
  for (int i = tid; i < words / 4; i += NT) ((uint4*)koff)[i] = bt[i];
  const int nck = (P.Nch + 16 * TN - 1) / (16 * TN);
  const int g = lane >> 4;
  const int KR = (P.Kreal + KC - 1) / KC * KC;
  for (int q0 = 0; q0 < kRows; q0 += RB) {
    if (q0 > 0 && r0 + q0 >= c.M) break;     // uniform
    if (q0 > 0) __syncthreads();             // the previous rows' MFMAs are done with the slab
    stage_slab<T, SIGN, T, RB, NT>(c, P, slab, r0 + q0, sy0, 0, P.Kch);
    __syncthreads();
    const int items = __builtin_amdgcn_readfirstlane(tph[P.MT]) * nck;
    // MFMA items: (16-row tile, column chunk of 16*TN channels), kIT per wave at a time
    for (int t0 = 0; t0 < items; t0 += NW * kIT) {
      f4 acc[kIT][RB][TN];
      auto gemm = [&](int t, f4 (&ac)[RB][TN]) {
        const int tt = nck == 1 ? t : t / nck, ck = nck == 1 ? 0 : t - tt * nck;
        const int ph = __builtin_amdgcn_readfirstlane(tph[tt]);
        const int base = desc[tt * 16 + (lane & 15)] & 0xffffu;
#pragma unroll
        for (int q = 0; q < RB; ++q)
#pragma unroll
          for (int k = 0; k < TN; ++k) ac[q][k] = f4{0.f, 0.f, 0.f, 0.f};
        const T* Bp = (const T*)c.Bt + (size_t)ph * P.Nch * c.ldb + VEC * g;
        const T* Bn[TN];
        bool bv[TN];
#pragma unroll
        for (int k = 0; k < TN; ++k) {
          const int nb = ck * 16 * TN + k * 16 + (lane & 15);
          bv[k] = nb < P.Nch;
          Bn[k] = Bp + (size_t)(bv[k] ? nb : 0) * c.ldb;
        }
        uint4 fb[TN];
#pragma unroll
        for (int k = 0; k < TN; ++k) fb[k] = bv[k] ? *(const uint4*)Bn[k] : uint4{0u, 0u, 0u, 0u};
        for (int k0 = 0; k0 < KR; k0 += KC) {
          uint4 fn[TN];                       // the next step's weights, in flight during this step
          const int kn = k0 + KC < KR ? k0 + KC : 0;
#pragma unroll
          for (int k = 0; k < TN; ++k) fn[k] = bv[k] ? *(const uint4*)(Bn[k] + kn) : uint4{0u, 0u, 0u, 0u};
          int ko[VEC];
          const int4* kp = (const int4*)(koff + k0 + VEC * g);
#pragma unroll
          for (int e = 0; e < VEC / 4; ++e) {
            const int4 t4 = kp[e];
            ko[4 * e] = t4.x; ko[4 * e + 1] = t4.y; ko[4 * e + 2] = t4.z; ko[4 * e + 3] = t4.w;
          }
          uint4 fa[RB];
          Gather<T, RB>::get(slab, base, ko, fa);
#pragma unroll
          for (int k = 0; k < TN; ++k)
            Op<T>::template mma_rows<RB, TN>(fa, fb[k], ac, k);
#pragma unroll
          for (int k = 0; k < TN; ++k) fb[k] = fn[k];
        }
      };
#pragma unroll
      for (int i = 0; i < kIT; ++i) {
        const int t = t0 + wave + i * NW;
        if (t < items) gemm(t, acc[i]);
      }
      if (alias) __syncthreads();            // every wave is done with the slab
#pragma unroll
      for (int i = 0; i < kIT; ++i) {
        const int t = t0 + wave + i * NW;
        if (t >= items) continue;
        const int tt = nck == 1 ? t : t / nck, ck = nck == 1 ? 0 : t - tt * nck;
#pragma unroll
        for (int v = 0; v < 4; ++v) {
          const uint32_t o = desc[tt * 16 + g * 4 + v] >> 16;
          if (o == 0xffffu) continue;
#pragma unroll
          for (int k = 0; k < TN; ++k) {
            const int nb = ck * 16 * TN + k * 16 + (lane & 15);
            if (nb >= P.Nch) continue;
            float4* dst = outs + nb * P.OS + o;
            if constexpr (RB == 4) *dst = float4{acc[i][0][k][v], acc[i][1][k][v], acc[i][2][k][v], acc[i][3][k][v]};
            else ((float*)dst)[q0] = acc[i][0][k][v];
          }
        }
      }
    }
  }
  __syncthreads();
  band_epilogue<T, NW>(c, P, epi, outs, red, r0, band, yb0, yb1);
}

// Transposed convolution into a source of at most four channels (the
// network's input image) on the vector ALUs.  An MFMA tile's 16 columns
// would carry NC real channels and padding, so here each lane computes all NC
// channels of one source position for the four batch rows: per tap, one
// 16-byte LDS read of a cell feeds 4 NC FMAs.  A wave takes 64 positions of
// one stride phase, so the phase's weights (taps TA x TB per phase, fp32 in
// the operand precision) are wave-uniform scalar loads; the stride ST is a
// template parameter.  Lambda's channels are staged kch at a time (fp32 for
// either operand type), so that high bands (few halo rows) leave LDS for
// several workgroups per CU, whose staging and FMA phases overlap.  Bands,
// results and epilogue are those of conv_slab_kernel.
template <typename T, int NC, int TA, int TB, int ST, class Epi>
__global__ void __launch_bounds__(kDirNW * 64) convT_direct_kernel(ConvArgs c, ConvPlan Pr, Epi epi, int kch) {
  ConvPlan P = Pr;
  P.s = ST;              // the stride as a constant: phase arithmetic without divisions
  constexpr int NT = kDirNW * 64;
  extern __shared__ __attribute__((aligned(16))) unsigned char smem[];
  double* red = (double*)smem;
  float4* slab = (float4*)(smem + align16(kDirNW * 8 * kRows));
  float4* outs = slab;

  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int blk = xcd_tile(blockIdx.x, gridDim.x);
  const int r0 = (blk / P.n_bands) * kRows, band = blk % P.n_bands;
  const int s = P.s, p = P.p;
  const int yb0 = band * P.BH, yb1 = min(P.He, yb0 + P.BH);
  const int sy0 = (yb0 + p) / s - (TA - 1);
  // this wave's 64 positions: chunk `wave` of the band's, phase by phase
  int tl = wave, ph = 0, yf = 0, ny = 0, xf = 0, nx = 0;
  for (; ph < P.n_phase; ++ph) {
    phase_rows(P, ph, yb0, yb1, true, &yf, &ny, &xf, &nx);
    const int nt = (ny * nx + 63) / 64;
    if (tl < nt) break;
    tl -= nt;
  }
  ph = __builtin_amdgcn_readfirstlane(ph);          // n_phase: no chunk
  const int i = tl * 64 + lane;
  const bool live = ph < P.n_phase && i < ny * nx;
  const int iy = live ? i / nx : 0, ix = live ? i - iy * nx : 0;
  const int ry = ph / s, rx = ph % s;
  const int base = live ? ((yf + p - ry) / s - sy0 + iy) * P.Wp + (xf + p - rx) / s + ix + P.xl
                        : (TA - 1) * P.Wp + TB - 1;  // in-slab for every tap
  const int coff = (yf - yb0 + iy * s) * P.We + xf + ix * s;
  f4 acc[NC];
#pragma unroll
  for (int ch = 0; ch < NC; ++ch) acc[ch] = f4{0.f, 0.f, 0.f, 0.f};
  for (int c0 = 0; c0 < P.Kch; c0 += kch) {
    const int nch = min(kch, P.Kch - c0);
    if (c0 > 0) __syncthreads();       // the previous channels' taps are read
    stage_slab<T, false, float, 4, NT>(c, P, slab, r0, sy0, c0, nch);
    __syncthreads();
    if (ph >= P.n_phase) continue;
    const GCP_CONSTANT_AS float* W = cst(c.Btf) + (size_t)ph * P.Nch * c.ldb + c0 * (TA * TB);
    const f4* cells = (const f4*)slab + base;
#pragma unroll 2
    for (int o = 0; o < nch; ++o) {
      const f4* so = cells + o * P.CHS;
      f4 v[TA][TB];
#pragma unroll
      for (int a = 0; a < TA; ++a)
#pragma unroll
        for (int b = 0; b < TB; ++b) v[a][b] = so[-a * P.Wp - b];
#pragma unroll
      for (int ch = 0; ch < NC; ++ch) {
        const GCP_CONSTANT_AS float* w = W + (size_t)ch * c.ldb + o * (TA * TB);
#pragma unroll
        for (int a = 0; a < TA; ++a)
#pragma unroll
          for (int b = 0; b < TB; ++b)
#pragma unroll
            for (int q = 0; q < kRows; ++q) acc[ch][q] = fmaf(v[a][b][q], w[a * TB + b], acc[ch][q]);
      }
    }
  }
  __syncthreads();       // every wave is done with the slab
  if (live) {
#pragma unroll
    for (int ch = 0; ch < NC; ++ch) *(f4*)(outs + ch * P.OS + coff) = acc[ch];
  }
  __syncthreads();
  band_epilogue<T, kDirNW>(c, P, epi, outs, red, r0, band, yb0, yb1);
}

// launch configurations: waves per workgroup x column tiles per wave
struct CCfg { int nw, tn; };
static const CCfg kConv[] = {{4, 1}, {4, 2}, {8, 1}, {8, 2}};
int conv_num_configs() { return (int)(sizeof(kConv) / sizeof(kConv[0])); }

template <typename T, int NW, int TN, int RB, bool TRANS, bool SIGN, class Epi>
static hipError_t conv_go(const ConvArgs& c, const ConvPlan& P, const Epi& epi, hipStream_t st) {
  const bool alias = conv_alias(P, NW, TN);
  const int lds = conv_lds_bytes(P, (int)sizeof(T), NW, alias);
  if (lds > kLdsLimit) return hipErrorInvalidValue;
  const long grid = (long)((c.M + kRows - 1) / kRows) * P.n_bands;
  if (grid <= 0 || grid > 0x7fffffffL) return hipErrorInvalidValue;
  hipLaunchKernelGGL((conv_slab_kernel<T, NW, TN, RB, TRANS, SIGN, Epi>), dim3((unsigned)grid), dim3(NW * 64),
                     (unsigned)lds, st, c, P, epi, alias ? 1 : 0);
  return hipGetLastError();
}

// Configurations that cannot hold the band's accumulators run as 8 waves x 1
// column tile.
template <typename T, bool TRANS, bool SIGN, class Epi>
static hipError_t conv_any(int cfg, const ConvArgs& c, const Epi& epi, hipStream_t st) {
  const ConvPlan& P = *c.plan;
  if (!c.tab || c.ldb < P.KP || c.ldb % 32 != 0 || !conv_fits(P, sizeof(T) == 2)) return hipErrorInvalidValue;
  if (P.rb == 1) return conv_go<T, 4, 1, 1, TRANS, SIGN>(c, P, epi, st);
  if (cfg >= 0 && cfg < conv_num_configs() && !conv_alias(P, kConv[cfg].nw, kConv[cfg].tn)) cfg = 2;
  switch (cfg) {
    case 0: return conv_go<T, 4, 1, 4, TRANS, SIGN>(c, P, epi, st);
    case 1: return conv_go<T, 4, 2, 4, TRANS, SIGN>(c, P, epi, st);
    case 3: return conv_go<T, 8, 2, 4, TRANS, SIGN>(c, P, epi, st);
    default: return conv_go<T, 8, 1, 4, TRANS, SIGN>(c, P, epi, st);
  }
}

template <typename T>
static hipError_t conv_typed(int cfg, EpiKind kind, const ConvArgs& c, const void* epi, hipStream_t st) {
  if (c.trans) {
    switch (kind) {
      case EPI_BOUND: return conv_any<T, true, false>(cfg, c, BoundEpi<T>{*(const BoundEpiArgs*)epi}, st);
      case EPI_AHAT: return conv_any<T, true, false>(cfg, c, AhatEpi<T>{*(const BoundEpiArgs*)epi}, st);
      case EPI_CONC: return conv_any<T, true, false>(cfg, c, ConcEpi{*(const ConcEpiArgs*)epi}, st);
      case EPI_STORE: return conv_any<T, true, false>(cfg, c, StoreEpi{*(const StoreEpiArgs*)epi}, st);
      default: return hipErrorInvalidValue;
    }
  }
  switch (kind) {
    case EPI_ADJ:
      if (c.x_is_sign) return conv_any<T, false, true>(cfg, c, AdjEpi<T>{*(const AdjEpiArgs*)epi}, st);
      return conv_any<T, false, false>(cfg, c, AdjEpi<T>{*(const AdjEpiArgs*)epi}, st);
    case EPI_STORE:
      if (c.x_is_sign) return conv_any<T, false, true>(cfg, c, StoreEpi{*(const StoreEpiArgs*)epi}, st);
      return conv_any<T, false, false>(cfg, c, StoreEpi{*(const StoreEpiArgs*)epi}, st);
    default: return hipErrorInvalidValue;
  }
}

// Explicit-pi epilogues (rho set) and those with 64-bit addresses:
// instantiated for one column tile per wave only, 4 or 8 waves; the other
// shapes run as 8 waves.
template <typename T, bool TRANS, bool SIGN, class Epi>
static hipError_t conv_few(int cfg, const ConvArgs& c, const Epi& epi, hipStream_t st) {
  const ConvPlan& P = *c.plan;
  if (!c.tab || c.ldb < P.KP || c.ldb % 32 != 0 || !conv_fits(P, sizeof(T) == 2)) return hipErrorInvalidValue;
  if (P.rb == 1) return conv_go<T, 4, 1, 1, TRANS, SIGN>(c, P, epi, st);
  if (cfg == 0 && conv_alias(P, 4, 1)) return conv_go<T, 4, 1, 4, TRANS, SIGN>(c, P, epi, st);
  return conv_go<T, 8, 1, 4, TRANS, SIGN>(c, P, epi, st);
}

template <typename T>
static hipError_t conv_typed_wide(int cfg, EpiKind kind, const ConvArgs& c, const void* epi, hipStream_t st) {
  if (c.trans)
    return kind == EPI_BOUND ? conv_few<T, true, false>(cfg, c, Wide<BoundEpi<T>>{{*(const BoundEpiArgs*)epi}}, st)
                             : hipErrorInvalidValue;
  if (kind != EPI_ADJ) return hipErrorInvalidValue;
  const Wide<AdjEpi<T>> e{{*(const AdjEpiArgs*)epi}};
  return c.x_is_sign ? conv_few<T, false, true>(cfg, c, e, st) : conv_few<T, false, false>(cfg, c, e, st);
}

template <typename T>
static hipError_t conv_typed_pi(int cfg, EpiKind kind, const ConvArgs& c, const void* epi, hipStream_t st) {
  if (c.trans)
    return kind == EPI_BOUND ? conv_few<T, true, false>(cfg, c, BoundEpi<T, true>{*(const BoundEpiArgs*)epi}, st)
                             : hipErrorInvalidValue;
  if (kind != EPI_ADJ) return hipErrorInvalidValue;
  if (c.x_is_sign) return conv_few<T, false, true>(cfg, c, AdjEpi<T, true>{*(const AdjEpiArgs*)epi}, st);
  return conv_few<T, false, false>(cfg, c, AdjEpi<T, true>{*(const AdjEpiArgs*)epi}, st);
}

bool conv_direct_ok(const ConvGeom& g, const ConvPlan& P, EpiKind kind) {
  if (kind != EPI_CONC || g.ci < 1 || g.ci > 4 || P.rb != 4 || !direct_shape(P)) return false;
  return direct_chunks(P) <= kDirNW && conv_direct_lds_bytes(P) <= kLdsLimit;
}

template <typename T, int NC, int TA, int TB, int ST, class Epi>
static hipError_t direct_go(const ConvArgs& c, const ConvPlan& P, const Epi& epi, hipStream_t st) {
  const long grid = (long)((c.M + kRows - 1) / kRows) * P.n_bands;
  if (grid <= 0 || grid > 0x7fffffffL) return hipErrorInvalidValue;
  hipLaunchKernelGGL((convT_direct_kernel<T, NC, TA, TB, ST, Epi>), dim3((unsigned)grid), dim3(kDirNW * 64),
                     (unsigned)conv_direct_lds_bytes(P), st, c, P, epi, direct_kch(P));
  return hipGetLastError();
}

template <typename T, int NC, class Epi>
static hipError_t direct_taps(const ConvArgs& c, const ConvPlan& P, const Epi& epi, hipStream_t st) {
  if (P.A == 2 && P.Bn == 2 && P.s == 2) return direct_go<T, NC, 2, 2, 2>(c, P, epi, st);
  if (P.A == 3 && P.Bn == 3 && P.s == 1) return direct_go<T, NC, 3, 3, 1>(c, P, epi, st);
  return hipErrorInvalidValue;
}

template <typename T>
static hipError_t conv_direct(const ConvArgs& c, const ConcEpi& epi, hipStream_t st) {
  const ConvPlan& P = *c.plan;
  if (!c.Btf || c.ldb < P.KP || c.ldb % 32 != 0) return hipErrorInvalidValue;
  switch (P.Nch) {
    case 1: return direct_taps<T, 1>(c, P, epi, st);
    case 2: return direct_taps<T, 2>(c, P, epi, st);
    case 3: return direct_taps<T, 3>(c, P, epi, st);
    case 4: return direct_taps<T, 4>(c, P, epi, st);
    default: return hipErrorInvalidValue;
  }
}

hipError_t launch_conv(int bf16_mode, int cfg, EpiKind kind, const ConvArgs& c, const void* epi, hipStream_t st) {
  if (c.M <= 0) return hipSuccess;
  if (!c.plan) return hipErrorInvalidValue;
  if (cfg == kConvDirectCfg) {
    if (!c.trans || !conv_direct_ok(c.cg, *c.plan, kind)) return hipErrorInvalidValue;
    const ConcEpi e{*(const ConcEpiArgs*)epi};
    return bf16_mode ? conv_direct<bf16>(c, e, st) : conv_direct<float>(c, e, st);
  }
  if (cfg < 0 || (cfg >= kConvDirectCfg && cfg != kConvWideCfg)) return hipErrorInvalidValue;
  if (fused_explicit_pi(kind, epi))
    return bf16_mode ? conv_typed_pi<bf16>(cfg, kind, c, epi, st) : conv_typed_pi<float>(cfg, kind, c, epi, st);
  if ((kind == EPI_BOUND || kind == EPI_ADJ) && (cfg == kConvWideCfg || epilogue_wide(kind, epi, kRows)))
    return bf16_mode ? conv_typed_wide<bf16>(cfg, kind, c, epi, st) : conv_typed_wide<float>(cfg, kind, c, epi, st);
  return bf16_mode ? conv_typed<bf16>(cfg, kind, c, epi, st) : conv_typed<float>(cfg, kind, c, epi, st);
}

}  // namespace gcp
