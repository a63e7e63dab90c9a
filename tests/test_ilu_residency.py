"""CPU model of how the ILU(0) row form hands out its stages (k_ilu_up_rows):
any number of workgroups may run at a time, in any order, the others starting
only as running ones end.  A stage waits for the stage before it (forward) or
after it (backward), nothing else."""
import os
import random
import re

import pytest

CSRC = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_0912_0180_amd", "csrc")


class Counter:
    """The kernel's rule: the next stage from a counter, the one before kept per stage."""

    def __init__(self, nb, G):
        self.nb, self.next, self.before = nb, 0, {}

    def start(self, g):
        return {"last": -1, "back": False}

    def take(self, w):
        if not w["back"]:
            b = self.next
            self.next += 1
            if b < self.nb:
                self.before[b] = w["last"]
                w["last"] = b
                return ("f", b)
            w["back"] = True
        b = w["last"]
        if b < 0:
            return None
        w["last"] = self.before[b]
        return ("b", b)


class Fixed:
    """Workgroup g takes stages g, g + G, ..., and the same ones backward."""

    def __init__(self, nb, G):
        self.nb, self.G = nb, G

    def start(self, g):
        mine = list(range(g, self.nb, self.G))
        return [("f", b) for b in mine] + [("b", b) for b in reversed(mine)]

    def take(self, w):
        return w.pop(0) if w else None


def finishes(rule, nb, G, resident, rng):
    """Whether the solves end with `resident` of G workgroups running at a time."""
    R = rule(nb, G)
    waiting = list(range(G))
    rng.shuffle(waiting)                 # the device may start them in any order
    running, done = [], set()
    while waiting or running:
        while waiting and len(running) < resident:
            w = R.start(waiting.pop())
            running.append([w, R.take(w)])
        moved = False
        for r in rng.sample(running, len(running)):
            job = r[1]
            if job is not None:
                k, b = job
                need = b - 1 if k == "f" else b + 1
                if 0 <= need < nb and (k, need) not in done:
                    continue
                if k == "b":
                    assert ("f", b) in done
                assert job not in done
                done.add(job)
                r[1] = R.take(r[0])
            moved = True
            if r[1] is None:
                running.remove(r)
        if not moved:
            return False
    assert len(done) == 2 * nb           # every stage once each way
    return True


@pytest.mark.parametrize("nb,G", [(1, 1), (2, 2), (7, 3), (20, 8), (33, 32), (64, 9), (5, 12)])
def test_solves_end_with_any_number_of_workgroups_running(nb, G):
    rng = random.Random(nb * 100 + G)
    for resident in range(1, G + 1):
        for _ in range(20):
            assert finishes(Counter, nb, G, resident, rng)


def test_fixed_stages_need_every_workgroup_resident():
    rng = random.Random(1)
    assert finishes(Fixed, 20, 8, 8, rng)
    assert not finishes(Fixed, 20, 8, 7, rng)


def test_kernel_takes_stages_by_counter():
    src = open(os.path.join(CSRC, "hh_kernels.hpp")).read()
    body = src[src.index("void k_ilu_up_rows("):]
    body = body[: body.index("\n}\n")]
    assert "__hip_atomic_fetch_add(a.chan, 1" in body
    assert not re.search(r"blockIdx|gridDim", body)
