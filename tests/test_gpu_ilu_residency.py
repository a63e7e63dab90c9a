"""The ILU(0) row form with one workgroup, with more than the device can run at
a time, and with cycles of several grids on streams beside each other."""
import numpy as np
import pytest

from paper_0912_0180_amd import workloads as W

pytestmark = pytest.mark.gpu


def problem(nx, ny, levels, coarse_op):
    h = 1.0 / 64
    hi = (-0.1 + nx * h, -0.1 + ny * h)
    d = W.base_desc(2, (nx, ny), (-0.1, -0.1), hi, (0.0, 0.0), (hi[0] - 0.04, hi[1] - 0.1), levels=levels, nu1=0,
                    omega=0.9, coarse_op=coarse_op, smoother=1)
    rng = np.random.default_rng(nx + 1000 * ny)
    return d, 36.0 * (1 + 0.3 * rng.uniform(size=nx * ny)), rng


@pytest.mark.parametrize("groups", [1, 2, 3, 1000])
@pytest.mark.parametrize("coarse_op", [0, 1])
def test_any_number_of_workgroups(oracle_mod, monkeypatch, coarse_op, groups):
    import torch
    from paper_0912_0180_amd import hh
    print("case", coarse_op, groups, flush=True)
    d, phi, rng = problem(28, 420, 3, coarse_op)     # 7 stages, then 4 (5-point) or 7 (25-point)
    g, o = hh.Grid(d, phi), oracle_mod.Grid(d, phi)
    monkeypatch.setenv("HH_ILU_GROUPS", str(groups))
    for k in range(3):
        f = rng.standard_normal(g.N) + 1j * rng.standard_normal(g.N)
        assert np.array_equal(g.vcycle(torch.from_numpy(f).cuda(), "c128").cpu().numpy(), o.vcycle(f)), k


def test_more_workgroups_than_compute_units(monkeypatch):
    """264 stages on the two finest levels, a workgroup for each."""
    import torch
    from paper_0912_0180_amd import hh
    assert torch.cuda.get_device_properties(0).multi_processor_count < 264
    d, phi, rng = problem(192, 16896, 7, 1)
    g = hh.Grid(d, phi)
    f = torch.from_numpy(rng.standard_normal(g.N) + 1j * rng.standard_normal(g.N)).cuda()
    ref = g.vcycle(f, "c128").clone()
    assert bool(torch.isfinite(torch.view_as_real(ref)).all())
    print("default number of workgroups done", flush=True)
    monkeypatch.setenv("HH_ILU_GROUPS", "264")
    for k in range(2):
        assert torch.equal(g.vcycle(f, "c128"), ref), k


def test_cycles_on_streams_beside_each_other():
    import torch
    from paper_0912_0180_amd import hh
    jobs = []
    for k in range(6):
        d, phi, rng = problem(96 + 8 * k, 384, 4, k % 2)
        g = hh.Grid(d, phi)
        f = torch.from_numpy(rng.standard_normal(g.N) + 1j * rng.standard_normal(g.N)).cuda()
        jobs.append((g, f, g.vcycle(f, "c128").clone(), torch.empty_like(f), torch.cuda.Stream()))
    torch.cuda.synchronize()
    for _ in range(5):
        for g, f, ref, u, s in jobs:
            with torch.cuda.stream(s):
                g.vcycle(f, "c128", out=u)
    torch.cuda.synchronize()
    for g, f, ref, u, s in jobs:
        assert torch.equal(u, ref)
