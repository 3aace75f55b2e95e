"""Host rules of the kernel launches at the edges of what they take, without a
device: a small C++ program linked against the built library asks them
(csrc/gcp_internal.h)."""
import os
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
PKG = os.path.join(ROOT, "paper_2208_05740_amd")
HIPCC = shutil.which("hipcc") or "/opt/rocm/bin/hipcc"

pytestmark = pytest.mark.skipif(not os.path.exists(HIPCC) or not os.path.exists(os.path.join(PKG, "libgcp.so")),
                                reason="hipcc or the built library not available")


def _run(tmp_path, source):
    """Lines that the program prints."""
    src, exe = tmp_path / "rules.cpp", tmp_path / "rules"
    src.write_text(source)
    cmd = [HIPCC, "-O2", "-std=c++17", "-I" + os.path.join(PKG, "csrc"), str(src), "-L" + PKG, "-lgcp",
           "-Wl,-rpath," + PKG, "-o", str(exe)]
    r = subprocess.run(cmd, capture_output=True, text=True)
    assert r.returncode == 0, r.stderr[-2000:]
    r = subprocess.run([str(exe)], capture_output=True, text=True, timeout=300)
    assert r.returncode == 0, (r.stdout + r.stderr)[-2000:]
    return r.stdout.splitlines()


# A workgroup once held one batch row of a band (48 KB with its results, at
# four bytes an element) and asked for its tables, that slab at the operand's
# size and the results: 64 KB of LDS at most, with eight waves.  Every conv
# that was taken then, in a net that can be created, has to be taken.
CONV_SWEEP = r"""
#include "gcp_internal.h"
#include <algorithm>
#include <cstdio>
using namespace gcp;
static int up16(int b) { return (b + 15) & ~15; }
struct Row { long slab; long lds[2]; };
static Row one_row(const ConvGeom& g, int t) {
  const int s = g.stride, He = t ? g.hi : g.ho, We = t ? g.wi : g.wo, Nch = t ? g.ci : g.co, Kch = t ? g.co : g.ci;
  const int A = t ? (g.kh + s - 1) / s : g.kh, Bn = t ? (g.kw + s - 1) / s : g.kw;
  const int Wp = t ? Bn - 1 + std::max((g.wi - 1 + g.pad) / s + 1, g.wo)
                   : g.pad + std::max(g.wi, (g.wo - 1) * s - g.pad + g.kw);
  const int KP = (Kch * A * Bn + 31) / 32 * 32;
  auto rows = [&](int bh) { return t ? (bh - 1) / s + 1 + A : (bh - 1) * s + g.kh; };
  int bh = He;
  while (bh > 1 && ((long)Kch * rows(bh) * Wp + 4l * Nch * (bh * We + 1)) * 4 > 48 * 1024) --bh;
  const int nb = (He + bh - 1) / bh, BH = (He + nb - 1) / nb;
  int MT = 0;
  for (int b = 0; b < nb; ++b) {
    const int y0 = b * BH, y1 = std::min(He, y0 + BH), np = t ? s : 1;
    int nt = 0;
    for (int ry = 0; ry < np; ++ry)
      for (int rx = 0; rx < np; ++rx) {
        int ny = 0, nx = 0;
        for (int y = y0; y < y1; ++y) ny += !t || (y + g.pad) % s == ry;
        for (int x = 0; x < We; ++x) nx += !t || (x + g.pad) % s == rx;
        nt += (ny * nx + 15) / 16;
      }
    MT = std::max(MT, nt);
  }
  const long cells = (long)Kch * rows(BH) * Wp;
  Row r{cells * 4, {}};
  for (int bf16 = 0; bf16 < 2; ++bf16)
    r.lds[bf16] = up16(KP * 4) + 8 * 8 * 4 + up16(MT * 4) + MT * 128 + up16((int)(cells * (bf16 ? 2 : 4))) +
                  4l * up16(Nch * (BH * We + 1) * 4);
  return r;
}
int main() {
  const int ch[] = {1, 2, 3, 5, 16, 24, 32, 64, 96, 128, 192, 256, 266, 320, 512, 640};
  const int hw[][2] = {{1, 1}, {2, 2}, {3, 3}, {4, 4}, {5, 5}, {5, 7}, {7, 5}, {6, 6}, {8, 8}, {10, 10}, {11, 13}, {12, 12},
                       {14, 14}, {16, 16}, {20, 20}, {24, 24}, {28, 28}, {32, 32}, {4, 64}, {64, 4}, {48, 48}, {64, 64}};
  long taken[2] = {0, 0}, lost[2] = {0, 0};
  for (int ci : ch) for (int co : ch) for (auto& d : hw) for (int k = 1; k <= 7; ++k) for (int s = 1; s <= 3; ++s)
    for (int p = 0; p <= 3; ++p) {
      const int ho = (d[0] + 2 * p - k) / s + 1, wo = (d[1] + 2 * p - k) / s + 1;
      if (p >= k || d[0] + 2 * p < k || d[1] + 2 * p < k) continue;
      const ConvGeom g{ci, d[0], d[1], co, ho, wo, k, k, s, p};
      const Row r[2] = {one_row(g, 0), one_row(g, 1)};
      bool made = true;
      for (int t = 0; t < 2; ++t) {
        if (r[t].slab != conv_row_slab(g, t)) return 1;
        made = made && r[t].slab <= 48 * 1024;
      }
      if (!made) continue;
      for (int t = 0; t < 2; ++t) {
        bool by_type;      // else bf16 runs fp32's plan
        const ConvPlan a = conv_plan(g, t, 0, &by_type), b = conv_plan(g, t, 1);
        if (!by_type && (a.BH != b.BH || a.rb != b.rb)) return 2;
      }
      for (int t = 0; t < 2; ++t)
        for (int bf16 = 0; bf16 < 2; ++bf16) {
          if (r[t].lds[bf16] > 64 * 1024) continue;
          ++taken[bf16];
          if (PLAN_FITS) continue;
          if (lost[bf16]++ < 20)
            printf("lost bf16=%d trans=%d %dx%dx%d -> %d, %dx%d stride %d pad %d\n", bf16, t, ci, d[0], d[1], co, k, k, s, p);
        }
    }
  printf("taken %ld %ld lost %ld %ld\n", taken[0], taken[1], lost[0], lost[1]);
}
"""


def _conv_sweep(tmp_path):
    *cases, last = _run(tmp_path, CONV_SWEEP.replace("PLAN_FITS", "conv_fits(conv_plan(g, t, bf16), bf16)"))
    words = last.split()
    taken, lost = [int(x) for x in words[1:3]], [int(x) for x in words[4:6]]
    assert min(taken) > 50000, last
    return lost, cases


def test_bf16_convs_that_one_row_slabs_took_are_taken(tmp_path):
    lost, cases = _conv_sweep(tmp_path)
    assert lost[1] == 0, (lost, [c for c in cases if "bf16=1" in c][:10])


def test_fp32_convs_that_one_row_slabs_took_are_taken(tmp_path):
    lost, cases = _conv_sweep(tmp_path)
    assert lost[0] == 0, (lost, cases[:10])


# Every offset that a layer tile forms in 32 bits, in 64: operand rows of the
# tile (those that exist) up to their last vector, and the windows of the
# epilogue, rows that do not exist included, below 2^31.
ADDRESSES = r"""
#include "gcp_internal.h"
#include <algorithm>
#include <cstdio>
using namespace gcp;
int main() {
  const long widths[] = {16, 784, 1 << 20, (1 << 23) - 16, 1 << 23, 1 << 24, 17039360, 17039376, (1 << 25) - 16, 1 << 25,
                         34078736, 1 << 26, (1 << 27) - 16, 1 << 27, 200000000};
  const EpiKind kinds[] = {EPI_STORE, EPI_BOUND, EPI_CONC, EPI_ADJ, EPI_AHAT};
  long n = 0, wide = 0, bad = 0, moved = 0;
  for (long kw : widths) for (long nw : widths) for (long ni : widths) for (EpiKind kind : kinds)
    for (int bf16 = 0; bf16 < 2; ++bf16) for (int sign = 0; sign < (kind == EPI_ADJ || kind == EPI_STORE ? 2 : 1); ++sign)
      for (int M : {1, 9, 37, 64, 36864}) for (int cfg = 0; cfg < 8; ++cfg) {
        GemmArgs g{};
        g.M = M; g.N = (int)nw; g.K = (int)kw; g.lda = (int)kw; g.ldb = (int)kw; g.a_is_sign = sign;
        BoundEpiArgs be{}; AdjEpiArgs ae{}; ConcEpiArgs ce{}; StoreEpiArgs se{};
        be.nd.ld = ae.nd.ld = (int)nw;
        be.rp.n_I = ae.rp.n_I = ce.rp.n_I = (int)ni;
        const void* epi = kind == EPI_ADJ ? (void*)&ae : kind == EPI_CONC ? (void*)&ce : kind == EPI_STORE ? (void*)&se : (void*)&be;
        const int run = gemm_config_for(cfg, kind, bf16, g, epi);
        ++n;
        int bm, bn;
        gemm_config_tile(run, &bm, &bn);
        if (run >= 8) {
          ++wide;
          if (std::max({kw, nw, kind == EPI_BOUND || kind == EPI_ADJ ? ni : 0}) < 1 << 23) ++moved;
          continue;
        }
        const long esz = bf16 ? 2 : 4, ab = sign ? 1 : esz;
        const long a = ((std::min(bm, M) - 1) * kw + kw) * ab - 1, b = ((std::min<long>(bn, nw) - 1) * kw + kw) * esz - 1;
        bool ok = run == cfg && a <= 0xffffffffl && b <= 0xffffffffl && nw * 16 - 1 <= 0xffffffffl;
        if (kind == EPI_BOUND || kind == EPI_ADJ)
          for (long p : {nw, ni}) ok = ok && bm * p * 4 < 0x80000000l && 0x80000000l + 3 * p * 4 <= 0xffffffffl;
        if (!ok && bad++ < 10) printf("cfg %d -> %d kind %d bf16 %d sign %d M %d N %ld K %ld n_I %ld\n", cfg, run, kind, bf16, sign, M, nw, kw, ni);
      }
  // four rows: the elementwise relaxation and the conv lists
  for (long p : widths)
    for (int swap = 0; swap < 2; ++swap) {
      NodeDev nd{}; RowParams rp{};
      nd.ld = (int)(swap ? 16 : p); rp.n_I = (int)(swap ? p : 16);
      const bool fits = 16 * p < 0x80000000l;
      if (windows_wide(nd, rp, 4) == fits) ++bad;
    }
  printf("%ld %ld %ld %ld\n", n, wide, bad, moved);
}
"""


def test_tiles_reach_their_rows_or_give_way_to_64_bit_tiles(tmp_path):
    *cases, last = _run(tmp_path, ADDRESSES)
    n, wide, bad, moved = [int(x) for x in last.split()]
    assert n > 100000 and wide > 1000 and bad == 0, (last, cases)
    assert moved == 0, last      # rows of up to 8 million keep the tile that was chosen


GRID = r"""
#include "gcp_internal.h"
#include <cstdio>
int main() {
  for (int n : {1, 2, 65535, 65536, 65537, 1 << 24, (1 << 24) + 1, 100000007, 0x7fff0000}) {
    const dim3 g = gcp::prep_grid(n);
    const unsigned long all = (unsigned long)g.x * g.y;
    printf("%d %d\n", n, g.x * 256ul < 1ul << 32 && g.y <= 65535 && g.z == 1 && all >= (unsigned long)n && all < (unsigned long)n + g.x &&
                              all <= 0x7fffffff);
  }
}
"""


def test_start_of_call_grid_is_launchable_and_covers_its_jobs(tmp_path):
    out = [line.split() for line in _run(tmp_path, GRID)]
    assert len(out) == 9 and all(ok == "1" for _, ok in out), out


def test_slack_grid_has_no_idle_workgroup(tmp_path):
    # 16 rows a workgroup
    out = _run(tmp_path, '''
#include "gcp_internal.h"
#include <cstdio>
int main() { for (int M : {1, 15, 16, 17, 333, 36864}) printf("%d %d\\n", M, gcp::slack_grid(M)); }
''')
    for M, g in (map(int, line.split()) for line in out):
        assert 16 * (g - 1) < M <= 16 * g, (M, g)
