"""GPU parity of random measurements whose windows are cut for their row count (more than 4096 rows
with x at a window's targets), record and tableau against the oracle bit for bit: layers of less and
of more targets than an uncut window holds, and a second execution that knows its windows."""
from __future__ import annotations

import numpy as np
import pytest

from oracle import oracle as O
from paper_2507_03092_amd import circuits as Cc

pytestmark = pytest.mark.gpu


def _spread(n, targets, rng):
    """Every stabilizer has x at one of the targets, and a target at a few of them."""
    c = Cc.Circuit(n=n)
    q = rng.permutation(n)
    t, rest = q[:targets], q[targets:]
    c.append(Cc.H, np.arange(n))
    c.append(Cc.S, rng.permutation(n)[: n // 3])
    for i in range(0, len(rest), targets):
        r = rest[i: i + targets]
        c.append(Cc.CX, np.stack([r, t[: len(r)]], 1).reshape(-1))
    c.append(Cc.CX, np.stack([t[0:-1:2], t[1::2][: len(t[0:-1:2])]], 1).reshape(-1))
    c.append(Cc.S, rng.permutation(n)[: n // 3])
    return c, rng.permutation(t)


@pytest.mark.parametrize("n,targets,shots,windows", [(4200, 65, 2, 2), (6000, 130, 1, 2), (6000, 300, 2, 3)])
def test_cut_windows(n, targets, shots, windows):
    from paper_2507_03092_amd import stab

    rng = np.random.default_rng(n + targets)
    c, t = _spread(n, targets, rng)
    _, (tx, tz, tr) = O.run(c, 1, 7, want_tableau=True)
    # a window takes up to 256 targets, 64 where more than 4096 rows have x at one of those
    assert (tx[0][n:][:, t[:256]] != 0).any(1).sum() > 4096
    c.append(Cc.MR, t)
    c.append(Cc.H, rng.permutation(n)[: (n + 1) // 2])
    c.append(Cc.M, rng.permutation(n)[:targets])
    print(f"case n={n} targets={targets} shots={shots}", flush=True)
    want, (tx, tz, tr) = O.run(c, shots, 7, want_tableau=True)
    ctx = stab.Context(n, shots, seed=7)
    prog = ctx.compile(c)
    for i in range(2):
        ctx.reset(7)
        assert np.array_equal(ctx.execute(prog), want), i
        x, z, r = ctx.get_tableau(shots - 1)
        assert np.array_equal(x, tx[-1]) and np.array_equal(z, tz[-1]) and np.array_equal(r, tr[-1]), i
    # (two executions; the second layer takes one window at least)
    assert ctx.counters()[0] >= 2 * (windows + 1)
    ctx.close()
