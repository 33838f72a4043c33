"""GPU parity of the batch kernel where its forms change, records and tableaux against the oracle bit
for bit, in both widths: windows of 64 (32 above 4096 qubits) random targets and their remainders,
targets an earlier one of the instruction decides, few needed columns (gathered) and many (a band
pass), T1/T2 instructions with few events, many and only events, and runs with more noise layers or
errors than are listed."""
from __future__ import annotations

import numpy as np
import pytest

from oracle import oracle as O
from paper_2507_03092_amd import circuits as Cc

pytestmark = pytest.mark.gpu


def _append(c, parts):
    for p in parts:
        ins, tg = p.arrays()
        off = 0
        for q in ins:
            k = int(q["ntargets"])
            c.append(int(q["kind"]), tg[off: off + k])
            off += k


def _windows(n, targets, seed):
    rng = np.random.default_rng(seed)
    c = Cc.Circuit(n=n)
    _append(c, [Cc.random_layered_clifford(n, 8, (seed, n), meas_every=9)])
    for kind in (Cc.MR, Cc.M, Cc.R, Cc.M):
        c.append(kind, rng.permutation(n)[:targets])
        c.append(Cc.H, rng.permutation(n)[: (n + 1) // 2])
    c.append(Cc.M, rng.permutation(n))
    return c


def _relax(n, p_reset, seed):
    c = _windows(n, n, seed)
    for p in (p_reset, p_reset / 3):
        t0 = int(p * 2.0 ** 64) if p < 1 else 2 ** 64 - 1
        c.append(Cc.T1T2, np.arange(n), (t0, min(2 ** 64 - 1, t0 + (1 << 60)), 0))
        c.append(Cc.H, np.arange(0, n, 2))
        c.append(Cc.MR, np.arange(0, n, 3))
    c.append(Cc.M, np.arange(n))
    return c


def _noise(n, layers, p, seed):
    c = _windows(n, (n + 1) // 2, seed)
    for k in range(layers):
        c.dep1(p, np.arange(n))
        if k == layers // 2:
            c.append(Cc.H, np.arange(n))
    c.append(Cc.M, np.arange(n))
    return c


CASES = {
    "one": lambda: [_windows(n, n, 3) for n in (1, 2, 63, 64)],
    "remainders": lambda: [_windows(n, k, 4) for n, k in ((65, 65), (130, 129), (200, 60), (200, 61), (300, 193), (700, 320))],
    "above_4096": lambda: [_windows(4100, 70, 5), _windows(90, 90, 5)],
    "relax": lambda: [_relax(n, p, 6) for n, p in ((5, .5), (70, .02), (130, .3), (300, 1.), (520, .1))],
    "noise": lambda: [_noise(n, k, p, 7) for n, k, p in ((70, 40, .05), (300, 3, .9), (130, 30, .02), (65, 31, .3))],
}


@pytest.mark.parametrize("tile", [8, 0x208])
@pytest.mark.parametrize("name", sorted(CASES))
def test_batch_forms(name, tile):
    from paper_2507_03092_amd import stab

    print(f"case {name} tile {tile:#x}", flush=True)
    circs = CASES[name]()
    tableau = name != "above_4096"
    b = stab.Batch(np.array([c.n for c in circs], dtype=np.int32), seed=9)
    prog = b.compile(circs)
    prog.tile = tile
    got = b.execute(prog)
    for k, c in enumerate(circs):
        want = O.run(c, 1, 9, k, tableau)
        if tableau:
            want, (tx, tz, tr) = want
            x, z, r = b.get_tableau(k)
            assert np.array_equal(x, tx[0]) and np.array_equal(z, tz[0]) and np.array_equal(r, tr[0]), (k, c.n)
        assert np.array_equal(got[k], want[0]), (k, c.n)
    b.close()
