"""The ILU(0) row form's layout as the library has it (IluLayout, called on
the host): every point has a place of its own within the arrays, runs have at
most RW rows, and the arrays stay within the bound that include/hh.h states.
And a model of the 25-point set's ring: the value of the row above is read from
the ring one step after another lane wrote it."""
import ctypes
import os
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
SRC = r"""
#include "hh_idr_kernels.hpp"
template <bool G> void layout(int nx, int ny, int64_t *o, int64_t *first, int64_t *w, int64_t *lo, int64_t *up)
{
    using S = hh::IluSet<G>;
    const hh::IluLayout<G> l(nx, ny);
    const int64_t head[] = {l.nb, l.DT, l.size(), l.chan_words(), S::M, S::RW, S::NLO, S::HR};
    for (int k = 0; k < 8; ++k) o[k] = head[k];
    for (int b = 0; b <= l.nb; ++b) first[b] = l.j0(b);
    for (int j = 0; j < ny; ++j) {
        const int b = l.band_of(j), r = j - l.j0(b);
        for (int i = 0; i < nx; ++i) {
            const int64_t dd = l.d0(b) + i + S::M * r, p = i + (int64_t)nx * j;
            w[p] = dd * S::RW + r;
            for (int k = 0; k < S::NLO; ++k) lo[p * S::NLO + k] = l.lo(dd, k, r);
            for (int k = 0; k <= S::NLO; ++k) up[p * (S::NLO + 1) + k] = l.up(dd, k, r);
        }
    }
}
extern "C" void layout_gal(int nx, int ny, int64_t *o, int64_t *f, int64_t *w, int64_t *lo, int64_t *up) { layout<true>(nx, ny, o, f, w, lo, up); }
extern "C" void layout_five(int nx, int ny, int64_t *o, int64_t *f, int64_t *w, int64_t *lo, int64_t *up) { layout<false>(nx, ny, o, f, w, lo, up); }
"""


@pytest.fixture(scope="module")
def lib(tmp_path_factory):
    if shutil.which("hipcc") is None:
        pytest.skip("hipcc not available")
    d = tmp_path_factory.mktemp("layout")
    (d / "layout.hip").write_text(SRC)
    from paper_0912_0180_amd import build as B
    cmd = ["hipcc", "-x", "hip", "--offload-arch=gfx950"] + B.FLAGS + ["-shared",
           "-I", os.path.join(ROOT, "paper_0912_0180_amd", "csrc"), str(d / "layout.hip"), "-o", str(d / "layout.so")]
    r = subprocess.run(cmd, capture_output=True, text=True, timeout=300)
    assert r.returncode == 0, r.stderr[-2000:]
    return ctypes.CDLL(str(d / "layout.so"))


@pytest.mark.parametrize("gal", [True, False])
@pytest.mark.parametrize("nx,ny", [(5, 5), (400, 10), (24, 24), (33, 33), (66, 66), (7, 31), (7, 32), (7, 33), (9, 64),
                                   (9, 65), (6, 129), (5, 700), (150, 97)])
def test_every_point_has_its_own_place(lib, nx, ny, gal):
    N, NLO = nx * ny, 12 if gal else 2
    o, first = (ctypes.c_int64 * 8)(), (ctypes.c_int64 * (ny + 2))()
    w, lo, up = (ctypes.c_int64 * N)(), (ctypes.c_int64 * (N * NLO))(), (ctypes.c_int64 * (N * (NLO + 1)))()
    (lib.layout_gal if gal else lib.layout_five)(nx, ny, o, first, w, lo, up)
    nb, DT, size, chan, M, RW, nlo, HR = o
    assert nlo == NLO and first[0] == 0 and first[nb] == ny
    rows = [first[b + 1] - first[b] for b in range(nb)]
    assert all(1 <= r <= RW for r in rows) and (nb == 1 or min(rows) >= max(HR, RW // 2))
    assert len(set(w)) == N and 0 <= min(w) and max(w) < DT * RW
    places = list(lo) + list(up)
    assert len(set(places)) == len(places) and 0 <= min(places) and max(places) < size
    # the bounds of the header: entries and work values, and the channel
    assert nb == -(-ny // RW) and size == DT * RW * (2 * NLO + 1)
    assert DT * RW <= N * (nb * RW / ny + M * RW / nx)
    assert chan == 1 + nb + 2 * (nb * nx * HR * 4)


def test_ring_reads_of_the_row_above():
    """25-point set: on step s of chunk c the solving wave reads row - 1's value
    of the step before from the ring (for row 0 the halo row that the channel
    filled).  Between a write and that read only the wave's own order stands
    (the same step's end) or a barrier (a chunk's), and no feeding wave touches
    the slot in the same chunk."""
    S, RW, HR, M, nx, R = 6, 32, 2, 3, 40, 32
    nd = nx + M * (R - 1)
    nch = (1 + -(-nd // S) + 2) // 3 * 3
    ring, writer = {}, {}
    for c in range(nch):
        # beside the solving wave: the channel's rows of chunk c + 1, and reads of chunk c - 1
        fed = {(((c + 1) % 3) * S + s, h) for s in range(S) for h in range(HR)}
        drained = {(((c - 1) % 3) * S + s, HR + r) for s in range(S) for r in range(RW)}
        for s in range(S):
            d = (c - 1) * S + s
            slot = (c % 3) * S + s - 1 if s else ((c + 2) % 3) * S + S - 1
            for row in range(RW):
                e = (slot, row + HR - 1)          # cur[(s - 1) ST + (row + 1) XE + part], one row up
                assert e not in fed
                if row and row - 1 < R:
                    want = d - 1 - M * (row - 1)  # row - 1's column on the step before
                    if 0 <= want < nx and c:
                        assert ring[e] == (row - 1, want)
                        assert writer[e] in ((c, s - 1), (c - 1, S - 1))
            cur = (c % 3) * S + s
            for row in range(RW):
                e = (cur, row + HR)
                assert e not in drained and e not in fed
                ring[e], writer[e] = (row, d - M * row), (c, s)
