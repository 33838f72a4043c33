"""GPU parity of the windowed random measurements (k_plan, k_snap, k_apply) at the sizes where
their forms change, record and tableau against the oracle bit for bit: one word of rows, more than
one 64-target chunk, more than one window and more than one word of shots, more rows than one
wave eliminates, and windows cut for their row count (n > 4096, dense)."""
from __future__ import annotations

import numpy as np
import pytest

from oracle import oracle as O
from paper_2507_03092_amd import circuits as Cc

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n,layers,targets,shots,mode", [
    (1, 4, 1, 3, "shared"), (64, 8, 64, 65, "shared"), (65, 9, 65, 3, "full"), (130, 10, 129, 5, "full"),
    (300, 12, 290, 130, "shared"), (600, 12, 600, 2, "shared"), (1100, 14, 80, 2, "shared"),
    (4200, 16, 130, 1, "shared")])
def test_windows_of_random_targets(n, layers, targets, shots, mode):
    from paper_2507_03092_amd import stab

    c = Cc.random_layered_clifford(n, layers, (n, 1), meas_every=layers + 1)
    rng = np.random.default_rng(n)
    c.append(Cc.MR, rng.permutation(n)[:targets])
    c.append(Cc.H, rng.permutation(n)[: (n + 1) // 2])
    c.append(Cc.M, rng.permutation(n)[:targets])
    print(f"case n={n} targets={targets} shots={shots} {mode}", flush=True)
    want, (tx, tz, tr) = O.run(c, shots, 7, want_tableau=True)
    ctx = stab.Context(n, shots, mode=mode, seed=7)
    got = ctx.run(c)
    assert np.array_equal(got, want)
    x, z, r = ctx.get_tableau(shots - 1)
    assert np.array_equal(x, tx[-1]) and np.array_equal(z, tz[-1]) and np.array_equal(r, tr[-1])
    ctx.close()
