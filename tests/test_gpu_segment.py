"""GPU parity of the segment kernel where its item lists change form, records and tableaux against the
oracle bit for bit: layers of every kind mix and odd gate counts, more gates (2048, above 4096
qubits 4096) or events (1024, 2048) in a layer than are loaded ahead, more layers than keep their
descriptors in LDS, and tiles of odd and even width."""
from __future__ import annotations

import numpy as np
import pytest

from oracle import oracle as O
from paper_2507_03092_amd import circuits as Cc

pytestmark = pytest.mark.gpu

KINDS = (Cc.H, Cc.S, Cc.X, Cc.Y, Cc.Z)


def _layers(n, layers, noise, seed):
    rng = np.random.default_rng(seed)
    c = Cc.Circuit(n=n)
    for k in range(layers):
        q = rng.permutation(n)
        m = int(rng.integers(0, n // 2 + 1)) if k % 3 else 0      # CX gates; none in every third layer
        for j in range(m):
            c.append(Cc.CX, q[2 * j: 2 * j + 2])
        rest = q[2 * m:]
        which = rng.integers(0, 5, len(rest)) if k % 3 != 2 else np.zeros(len(rest), dtype=int)
        for s, kind in enumerate(KINDS):
            if (which == s).any():
                c.append(kind, rest[which == s])
        if noise and k % 2:
            c.dep1(noise, np.arange(n))
    c.append(Cc.M, rng.permutation(n)[: min(n, 70)])
    return c


@pytest.mark.parametrize("n,layers,noise,shots,mode", [
    (1, 5, .5, 3, "shared"), (2, 9, .3, 65, "full"), (64, 140, .05, 3, "shared"), (65, 70, 0., 2, "shared"),
    (129, 12, .5, 64, "shared"), (190, 12, .9, 40, "full"), (2111, 9, 0., 1, "shared"), (4230, 6, .6, 2, "shared")])
def test_segment_lists(n, layers, noise, shots, mode):
    from paper_2507_03092_amd import stab

    c = _layers(n, layers, noise, n)
    print(f"case n={n} layers={layers} noise={noise} shots={shots} {mode}", flush=True)
    want, (tx, tz, tr) = O.run(c, shots, 5, want_tableau=True)
    ctx = stab.Context(n, shots, mode=mode, seed=5)
    got = ctx.run(c)
    assert np.array_equal(got, want)
    x, z, r = ctx.get_tableau(shots - 1)
    assert np.array_equal(x, tx[-1]) and np.array_equal(z, tz[-1]) and np.array_equal(r, tr[-1])
    ctx.close()
