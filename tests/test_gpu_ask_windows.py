"""GPU parity of executions that ask how many targets are pending (layers of more windows than are
launched without knowing): all random, few random and none, cut windows among them, from |0...0> and
going on, in a context and in the call that allocates nothing (which reads the count back)."""
from __future__ import annotations

import numpy as np
import pytest

from oracle import oracle as O
from paper_2507_03092_amd import circuits as Cc

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n,targets,shots,mode", [(1300, 1025, 3, "shared"), (1300, 1300, 2, "full"), (4200, 257, 1, "shared")])
def test_asked_windows(n, targets, shots, mode):
    from paper_2507_03092_amd import stab

    rng = np.random.default_rng(n)
    c = Cc.Circuit(n=n)
    c.append(Cc.H, rng.permutation(n)[: n // 2])
    c.append(Cc.CX, rng.permutation(n)[: n // 2 * 2])
    c.append(Cc.S, rng.permutation(n)[: n // 3])
    c.append(Cc.CX, rng.permutation(n)[: n // 2 * 2])
    t = rng.permutation(n)[:targets]
    c.append(Cc.M, t)                              # many random
    c.append(Cc.X, t[::3])
    c.append(Cc.MR, t)                             # none
    c.append(Cc.H, t[:5])
    c.append(Cc.M, t)                              # five
    ins, tg = c.arrays()
    twice = Cc.PackedCircuit(n, np.concatenate([ins, ins]), np.concatenate([tg, tg]))
    print(f"case n={n} targets={targets} shots={shots} {mode}", flush=True)
    want, (tx, tz, tr) = O.run(twice, shots, 5, want_tableau=True)
    ctx = stab.Context(n, shots, mode=mode, seed=5)
    got = [ctx.run(c), ctx.run(c)]
    assert np.array_equal(np.concatenate(got, axis=1), want)
    x, z, r = ctx.get_tableau(shots - 1)
    assert np.array_equal(x, tx[-1]) and np.array_equal(z, tz[-1]) and np.array_equal(r, tr[-1])
    ctx.close()
    if mode == "shared":
        assert np.array_equal(stab.sample_noalloc(c, shots, 5), want[:, : c.num_measurements()])
