"""The finaliser's sums at the edges of their paths, against the CPU oracle
value for value: an odd number of partials per value (their loads are then not
16-byte aligned), sums spread over workgroups (many partials) and not, IDR
passes built for 4 and for 8 columns, and mixed s in one batch."""
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


# 1001 groups of 512 unknowns: 17 (IDR(8)) x 1001 partials are spread, 9 x 1001 are not
@pytest.mark.parametrize("n,levels,method,s,mv", [((56, 88, 104), 4, "idr", 8, 12), ((56, 88, 104), 4, "idr", 4, 9),
                                                  ((56, 88, 104), 4, "bicgstab", 0, 4), ((48, 40), 3, "idr", 1, 9),
                                                  ((48, 40), 3, "idr", 3, 12), ((272, 240), 5, "idr", 5, 14)])
def test_first_matvecs_match_oracle(oracle_mod, n, levels, method, s, mv):
    import torch
    from paper_0912_0180_amd import hh
    print("case", n, method, s, flush=True)
    d, phi, b = problem(n, levels, 5)
    g, o = hh.Grid(d, phi), oracle_mod.Grid(d, phi)
    kw, okw = {}, {}
    if method == "idr":
        P = W.shadow_space(g.N, s, 6)
        kw, okw = {"s": s, "P": hh.shadow_to_device(P)}, {"s": s, "P": P}
    x, info = g.solve(torch.from_numpy(b).cuda(), method=method, tol=1e-30, max_matvec=mv, vcycle_prec="c128", history=True, **kw)
    xo, io = o.solve(b, method=method, tol=1e-30, max_matvec=mv, history=True, **okw)
    assert info["matvecs"] == io["matvecs"] and info["iterations"] == io["iterations"]
    assert np.array_equal(info["history"], io["history"])
    assert np.array_equal(x.cpu().numpy(), xo)


def test_mixed_s_in_a_batch(oracle_mod):
    import torch
    from paper_0912_0180_amd import hh
    cases = [((48, 40), 3, 2), ((64, 48), 3, 6)]
    grids, bs, opts, refs = [], [], [], []
    for k, (n, levels, s) in enumerate(cases):
        d, phi, b = problem(n, levels, 11 + k)
        g = hh.Grid(d, phi)
        P = hh.shadow_to_device(W.shadow_space(g.N, s, 20 + k))
        bd = torch.from_numpy(b).cuda()
        x, i = g.solve(bd, method="idr", s=s, P=P, tol=1e-8, vcycle_prec="c128")
        refs.append((x.clone(), i["matvecs"]))
        grids.append(g)
        bs.append(bd)
        opts.append(hh.make_opts(method="idr", s=s, P=P, tol=1e-8, vcycle_prec="c128"))
    import ctypes
    O = (hh.SolveOpts * 2)(*[o for o, _ in opts])
    infos = (hh.SolveInfo * 2)()
    xs = [torch.zeros_like(b) for b in bs]
    G = (ctypes.c_void_p * 2)(*[g.h.value for g in grids])
    B = (ctypes.c_void_p * 2)(*[b.data_ptr() for b in bs])
    X = (ctypes.c_void_p * 2)(*[x.data_ptr() for x in xs])
    hh.check(hh.lib().hh_solve_batch(G, 2, O, B, X, infos, ctypes.c_void_p(torch.cuda.current_stream().cuda_stream)))
    for q in range(2):
        assert infos[q].matvecs == refs[q][1] and torch.equal(xs[q], refs[q][0])
