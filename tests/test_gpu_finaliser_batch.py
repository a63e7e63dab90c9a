"""The finaliser's sums beyond the sizes of single small solves: a batch where
one problem has many partials and others few (all of them are then summed per
value first), and more partials than one lane per unit sum takes (above 2^24
unknowns).  The batch against its problems solved alone, bit for bit; the large
residual norms against a pairwise tree over the unknowns."""
import numpy as np
import pytest

from paper_0912_0180_amd import workloads as W

pytestmark = pytest.mark.gpu


def problem(n, levels, seed):
    h = 1.0 / 64
    lo = [-0.1] * len(n)
    hi = [lo[a] + h * n[a] for a in range(len(n))]
    d = W.base_desc(len(n), n, lo, hi, [0.0] * len(n), [v - 0.1 for v in hi], levels=levels)
    rng = np.random.default_rng(seed)
    N = int(np.prod(n))
    return d, 100.0 * (1 + 0.3 * rng.uniform(size=N)), rng.standard_normal(N) + 1j * rng.standard_normal(N)


# 5376 groups of 512 unknowns in the first problem, 4 and 15 in the others
@pytest.mark.parametrize("method,svals", [("bicgstab", (0, 0, 0)), ("idr", (4, 2, 3)), ("idr", (3, 8, 1))])
def test_large_and_small_problems_in_one_batch(method, svals):
    import ctypes
    import torch
    from paper_0912_0180_amd import hh
    print("case", method, svals, flush=True)
    sizes = [((1792, 1536), 7), ((48, 40), 3), ((96, 80), 3)]
    grids, bs, xs, opts, keep, refs = [], [], [], [], [], []
    for k, ((n, levels), s) in enumerate(zip(sizes, svals)):
        d, phi, b = problem(n, levels, 40 + k)
        g = hh.Grid(d, phi)
        bd = torch.from_numpy(b).cuda()
        kw = {"tol": 1e-30, "max_matvec": 13, "vcycle_prec": "c128"}
        if method == "idr":
            kw.update(s=s, P=hh.shadow_to_device(W.shadow_space(g.N, s, 60 + k)))
        x, i = g.solve(bd, method=method, **kw)
        refs.append((x.clone(), i))
        o, kp = hh.make_opts(method=method, **kw)
        grids.append(g)
        bs.append(bd)
        opts.append(o)
        keep.append((kp, kw))
        xs.append(torch.zeros_like(bd))
    O = (hh.SolveOpts * 3)(*opts)
    infos = (hh.SolveInfo * 3)()
    G = (ctypes.c_void_p * 3)(*[g.h.value for g in grids])
    B = (ctypes.c_void_p * 3)(*[b.data_ptr() for b in bs])
    X = (ctypes.c_void_p * 3)(*[x.data_ptr() for x in xs])
    st = hh.lib().hh_solve_batch(G, 3, O, B, X, infos, ctypes.c_void_p(torch.cuda.current_stream().cuda_stream))
    assert st in (hh.OK, -4)               # stopped at the matvec limit
    for q in range(3):
        assert infos[q].matvecs == refs[q][1]["matvecs"]
        assert infos[q].rel_res_recurrence == refs[q][1]["rel_res_recurrence"]
        assert torch.equal(xs[q], refs[q][0])


def pairwise_norm2(z):
    """||z||^2 by the pairwise tree over the zero-padded power-of-two length."""
    import torch
    v = torch.view_as_real(z)
    v = v[:, 0] * v[:, 0] + v[:, 1] * v[:, 1]
    m = 1 << (v.numel() - 1).bit_length()
    p = torch.zeros(m, dtype=torch.float64, device=v.device)
    p[: v.numel()] = v
    while p.numel() > 1:
        p = p[0::2] + p[1::2]
    return float(p[0])


# 64, 68 and 132 unit sums of 512 partials each: one, two and four per lane
@pytest.mark.parametrize("n,levels", [((4096, 4096), 10), ((4096, 4352), 9), ((6144, 5632), 9)])
def test_norms_of_many_unknowns(n, levels):
    import torch
    from paper_0912_0180_amd import hh
    print("case", n, flush=True)
    d, phi, b = problem(n, levels, 5)
    g = hh.Grid(d, phi)
    bd = torch.from_numpy(b).cuda()
    x, info = g.solve(bd, tol=1e-30, max_matvec=2, vcycle_prec="c128")
    r = bd - g.apply(x, "H")
    want = np.sqrt(pairwise_norm2(r)) / np.sqrt(pairwise_norm2(bd))
    assert info["rel_res_true"] == want
