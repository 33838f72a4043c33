"""GPU parity of graph replay where a measurement layer takes several windows of random targets:
replays from |0...0> with the known number of windows, and executions that go on from another state,
whose windows are not known, with eager work between them."""
from __future__ import annotations

import numpy as np
import pytest

from oracle import oracle as O
from paper_2507_03092_amd import circuits as Cc

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n,targets", [(130, 100), (600, 257), (700, 650)])
def test_graph_of_several_windows(n, targets):
    from paper_2507_03092_amd import stab

    c = Cc.random_layered_clifford(n, 9, (n, 4), meas_every=10)
    rng = np.random.default_rng(n)
    c.append(Cc.MR, rng.permutation(n)[:targets])
    c.append(Cc.H, rng.permutation(n)[: (n + 1) // 2])
    c.append(Cc.M, rng.permutation(n)[:targets])
    ins, tg = c.arrays()
    again = 3
    long = Cc.PackedCircuit(n, np.concatenate([ins] * again), np.concatenate([tg] * again))
    print(f"case n={n} targets={targets}", flush=True)
    want, (tx, tz, tr) = O.run(long, 3, 11, want_tableau=True)
    ctx = stab.Context(n, 3, seed=11)
    prog = ctx.compile(c)
    ctx.set_graph(True)
    for i in range(4):
        ctx.reset(11)
        got = [ctx.execute(prog) for _ in range(again)]
        assert np.array_equal(np.concatenate(got, axis=1), want), i
        x, z, r = ctx.get_tableau(2)
        assert np.array_equal(x, tx[-1]) and np.array_equal(z, tz[-1]) and np.array_equal(r, tr[-1]), i
    # the same program from |0...0> again and again
    for i in range(3):
        ctx.reset(11)
        assert np.array_equal(ctx.execute(prog), want[:, : c.num_measurements()]), i
    ctx.close()
