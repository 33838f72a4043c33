"""GPU parity of the batch kernel's instructions with few targets, records and tableaux against the
oracle bit for bit, in both widths: one, two and three targets, a single random one among many, T1/T2
instructions with no event, one and a few, at the sizes where the forms change."""
from __future__ import annotations

import numpy as np
import pytest

from oracle import oracle as O
from paper_2507_03092_amd import circuits as Cc

pytestmark = pytest.mark.gpu


def _few(n, seed):
    rng = np.random.default_rng((n, seed))
    c = Cc.Circuit(n=n)
    c.append(Cc.H, rng.permutation(n)[: (n + 1) // 2])
    if n > 1:
        c.append(Cc.CX, rng.permutation(n)[: n // 2 * 2])
    c.append(Cc.S, rng.permutation(n)[: (n + 2) // 3])
    for k in (1, 2, 3, 1, 2):
        for kind in (Cc.M, Cc.MR, Cc.R):
            t = rng.permutation(n)[: min(k, n)]
            c.append(kind, t)                         # right after another instruction
            c.append(Cc.H, rng.permutation(n)[: min(k, n)])
            c.append(kind, t)                         # after a gate pass
    c.append(Cc.M, rng.permutation(n))
    for kind in (Cc.M, Cc.MR, Cc.R):
        q = rng.permutation(n)
        c.append(Cc.H, q[:1])
        c.append(kind, q)                             # one random target, many that are not
        c.append(Cc.X, q[::2])
    for p in (0., 1.5 / n, 1. / (3 * n), 4. / n):
        t0 = min(int(min(p, 1.) * 2.0 ** 64), 2 ** 64 - 1)
        for _ in range(4):
            c.append(Cc.H, rng.permutation(n)[: (n + 3) // 4])
            c.append(Cc.T1T2, np.arange(n), (t0, min(2 * t0, 2 ** 64 - 1), 0))
    c.append(Cc.M, rng.permutation(n))
    return c


@pytest.mark.parametrize("tile", [8, 0x208])
@pytest.mark.parametrize("ns", [(1, 2, 3, 17, 64), (65, 256, 257, 300), (900,), (4100, 70)])
def test_few_targets(ns, tile):
    from paper_2507_03092_amd import stab

    print(f"case {ns} tile {tile:#x}", flush=True)
    circs = [_few(n, i) for n in ns for i in range(2)]
    tableau = max(ns) <= 1000
    b = stab.Batch([c.n for c in circs], seed=3)
    prog = b.compile(circs)
    prog.tile = tile
    got = b.execute(prog)
    for k, c in enumerate(circs):
        want = O.run(c, 1, 3, k, tableau)
        if tableau:
            want, (tx, tz, tr) = want
            x, z, r = b.get_tableau(k)
            assert np.array_equal(x, tx[0]) and np.array_equal(z, tz[0]) and np.array_equal(r, tr[0]), (k, c.n)
        assert np.array_equal(got[k], want[0]), (k, c.n)
    b.close()
