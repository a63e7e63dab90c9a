"""CPU model of the ILU(0) row form's pipeline (k_ilu_up_rows, IluLayout),
written from its index arithmetic: stages of at most RW rows, chunks of S
steps between barriers, the LDS ring of three chunks with the rows of the
stage before in front, the register windows, the three chunk buffers filled
two chunks ahead and read one step ahead, and the channel by column.  Values are replaced by the
point they belong to, so every read is checked to be the neighbour that the
stencil asks for, and within a chunk nothing is written that another wave
reads."""
import pytest

GAL = {"M": 3, "RW": 32, "HR": 2, "S": 6, "NLO": 12, "lo": list(range(12)), "up": list(range(13, 25))}
FIVE = {"M": 1, "RW": 64, "HR": 1, "S": 6, "NLO": 2, "lo": [7, 11], "up": [13, 17]}


class Layout:
    def __init__(self, K, nx, ny):
        self.K, self.nx, self.ny = K, nx, ny
        self.nb = -(-ny // K["RW"])
        self.base, self.extra = ny // self.nb, ny % self.nb
        self.DT = self.nb * (nx - K["M"]) + K["M"] * ny

    def j0(self, b):
        return b * self.base + min(b, self.extra)

    def d0(self, b):
        return b * (self.nx - self.K["M"]) + self.K["M"] * self.j0(b)


def fetch(K, fwd, nd, c, NF):
    """The elements the 192 feeding threads load for chunk c, per LDS place of
    the buffer: (step, place within the step), or the clamped one."""
    S, RW = K["S"], K["RW"]
    d = max(min((c - 1) * S if fwd else nd - c * S, nd - 1), 1 - S)
    lo, hi = max(-d, 0), min(nd - d, S)
    out = []
    for e in range(S * NF * RW):
        x = d * NF * RW + min(max(e, lo * NF * RW), hi * NF * RW - 1)
        assert 0 <= x < nd * NF * RW
        out.append((x // (NF * RW), x % (NF * RW)))
    return out


def run_stage(K, lay, b, fwd, channel, solved):
    M, RW, HR, S = K["M"], K["RW"], K["HR"], K["S"]
    nx, R = lay.nx, lay.j0(b + 1) - lay.j0(b)
    nd = nx + M * (R - 1)
    assert HR <= R <= RW or lay.nb == 1
    nch = (1 + -(-nd // S) + 2) // 3 * 3
    first = b == 0 if fwd else b == lay.nb - 1
    NF = K["NLO"] + (0 if fwd else 1)
    j0 = lay.j0(b)

    def point(row, col):
        """Grid point of this stage's (mirrored) row and column; None outside."""
        i = col if fwd else nx - 1 - col
        j = j0 + row if fwd else j0 + R - 1 - row
        return (j, i) if 0 <= i < nx and 0 <= j < lay.ny else None

    ring = [[None] * (RW + HR) for _ in range(3 * S)]
    W1, W2, O = [[None] * 6 for _ in range(RW)], [[None] * 6 for _ in range(RW)], [[None, None] for _ in range(RW)]

    def poll(c):
        slots = set()
        for s in range(S):
            for h in range(HR):
                col = (c - 1) * S + s + M * (1 + h)
                v = channel[(fwd, b - 1 if fwd else b + 1, col, h)] if not first and 0 <= col < nx else None
                ring[(c % 3) * S + s][HR - 1 - h] = v
                slots.add(((c % 3) * S + s, HR - 1 - h))
        return slots

    def publish(c):
        slots = set()
        for s in range(S):
            for h in range(HR):
                row = R - 1 - h
                col = (c - 1) * S + s - M * row
                if 0 <= col < nx:
                    slots.add(((c % 3) * S + s, row + HR))
                    channel[(fwd, b, col, h)] = ring[(c % 3) * S + s][row + HR]
        return slots

    poll(0)
    bufs = [None, fetch(K, fwd, nd, 1, NF), None]
    for c in range(nch):
        # feeding waves, beside the solving wave
        polled = poll(c + 1)
        published = publish(c - 1) if c else set()
        reads, writes = set(), set()
        stored = {((c - 1) % 3 * S + s, row + HR) for s in range(S) for row in range(RW)}   # chunk c - 1 on its way to w
        for s in range(S):
            d = (c - 1) * S + s
            if s == 0:
                ahead = nxt if c else None     # step 0 was read at the end of the chunk before
            else:
                ahead = bufs[c % 3]
            if s == S - 1:
                nxt = bufs[(c + 1) % 3]
            vals = {}
            last = [O[row][(s + 1) & 1 if M == 3 else 0] for row in range(RW)]     # every row's value of step d - 1
            for row in range(RW):
                i = d - M * row
                act = 0 <= i < nx and row < R
                r1 = ((c % 3) * S + s - 1) if s >= 1 else (((c + 2) % 3) * S + S - 1)
                r2 = ((c % 3) * S + s - 4) if s >= 4 else (((c + 2) % 3) * S + S + s - 4)
                # row - 1's value of step d - 1 from the lane before, row -1's from the ring
                q1 = last[row - 1] if row else ring[r1][HR - 1]
                reads.add((r1, HR - 1))
                if M == 3:
                    W1[row][s], W2[row][s] = q1, ring[r2][row]
                    reads.add((r2, row))
                if act:
                    slot = s if fwd else S - 1 - s
                    rr = row if fwd else R - 1 - row
                    step, place = ahead[(slot * NF) * RW + rr]
                    assert (step, place) == ((d if fwd else nd - 1 - d), rr)
                    if M == 3:
                        o1, o2 = O[row][(s + 1) & 1], O[row][s & 1]
                        if fwd:
                            terms = [W2[row][(s + 2 + k) % 6] for k in range(5)] + [W1[row][(s + 2 + k) % 6] for k in range(5)] + [o2, o1]
                        else:
                            terms = [o1, o2] + [W1[row][(s + 6 - k) % 6] for k in range(5)] + [W2[row][(s + 6 - k) % 6] for k in range(5)]
                    else:
                        terms = [q1, O[row][0]] if fwd else [O[row][0], q1]
                    pj, pi = point(row, i)
                    for t, sk in zip(terms, K["lo"] if fwd else K["up"]):
                        qj, qi = pj + sk // 5 - 2, pi + sk % 5 - 2
                        want = (qj, qi) if 0 <= qi < nx and 0 <= qj < lay.ny else None
                        assert t == want, (b, d, row, sk, t, want)
                        assert want is None or (fwd, want) in solved
                vals[row] = point(row, i) if act else None
            for row in range(RW):
                k = (c % 3) * S + s
                ring[k][row + HR] = vals[row]
                writes.add((k, row + HR))
                if M == 3:
                    O[row][s & 1] = vals[row]
                else:
                    O[row][0] = vals[row]
                if vals[row]:
                    solved.add((fwd, vals[row]))
        assert not polled & (reads | writes | stored) and not (published | stored) & writes
        bufs[(c + 2) % 3] = fetch(K, fwd, nd, c + 2, NF)     # beside the solving wave: another buffer than c's and c + 1's
        fetch(K, fwd, nd, c + 5, NF)
    publish(nch - 1)


@pytest.mark.parametrize("name", ["gal", "five"])
def test_pipeline_reads_every_neighbour(name):
    K = GAL if name == "gal" else FIVE
    RW = K["RW"]
    for nx, ny in [(5, 5), (7, RW), (6, RW + 1), (13, 2 * RW + 1), (40, RW - 1), (9, 3 * RW), (31, 2 * RW)]:
        lay, channel, solved = Layout(K, nx, ny), {}, set()
        for b in range(lay.nb):              # a stage waits for the one before only
            run_stage(K, lay, b, True, channel, solved)
        assert len(solved) == nx * ny
        for b in reversed(range(lay.nb)):
            run_stage(K, lay, b, False, channel, solved)
        assert len(solved) == 2 * nx * ny


@pytest.mark.parametrize("name", ["gal", "five"])
def test_layout_positions_are_distinct_and_in_range(name):
    K = GAL if name == "gal" else FIVE
    M, RW, NLO = K["M"], K["RW"], K["NLO"]
    for nx in (5, 11, 70):
        for ny in (5, RW - 1, RW, RW + 1, 2 * RW + 1, 5 * RW - 3):
            lay = Layout(K, nx, ny)
            seen, steps = set(), 0
            for b in range(lay.nb):
                R = lay.j0(b + 1) - lay.j0(b)
                assert 1 <= R <= RW and (lay.nb == 1 or 2 * R >= RW) and lay.d0(b) == steps
                for r in range(R):
                    for i in range(nx):
                        seen.add((lay.d0(b) + i + M * r) * RW + r)
                steps += nx + M * (R - 1)
            assert steps == lay.DT and lay.j0(lay.nb) == ny
            assert len(seen) == nx * ny and max(seen) < lay.DT * RW


def test_workgroups_resident_and_in_order():
    """Stage b is run by workgroup b mod G, forward ascending and backward
    descending: each workgroup's next stage only ever waits for stages that
    come earlier in another workgroup's order."""
    for nb in range(1, 40):
        for G in range(1, min(nb, 32) + 1):
            order = []
            for g in range(G):
                mine = list(range(g, nb, G))
                order.append([("f", b) for b in mine] + [("b", b) for b in reversed(mine)])
            done, at = set(), [0] * G
            while any(at[g] < len(order[g]) for g in range(G)):
                moved = False
                for g in range(G):
                    while at[g] < len(order[g]):
                        k, b = order[g][at[g]]
                        need = (k, b - 1) if k == "f" else (k, b + 1)
                        if 0 <= need[1] < nb and need not in done:
                            break
                        done.add((k, b))
                        at[g] += 1
                        moved = True
                assert moved
