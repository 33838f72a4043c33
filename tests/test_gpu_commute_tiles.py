"""GPU parity of stab_commute at the edges of its tiles, against the oracle's matrices: 32- and 64-string
tiles, 256 strings a block, rows of more than 16 result words, passes of 256 qubits and strings past
the span that is counted at once, with every pair conflicting on every qubit among them."""
from __future__ import annotations

import numpy as np
import pytest

from oracle import commute as OC
from paper_2507_03092_amd import circuits as Cc

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("na,nb,n", [(1, 1, 3), (31, 33, 128), (65, 32, 192), (257, 1100, 256), (255, 1025, 257),
                                     (64, 700, 449), (2, 3, (1 << 22) + 300)])
def test_commute_tiles(na, nb, n):
    from paper_2507_03092_amd import stab

    print(f"commute na={na} nb={nb} n={n}", flush=True)
    ax, az = Cc.random_paulis(na, n, (7, na))
    bx, bz = Cc.random_paulis(nb, n, (8, nb))
    ax[-1], az[-1] = 1, 0            # X...X against Z...Z and Y...Y: n conflicts
    bx[-1], bz[-1] = 0, 1
    if nb > 1:
        bx[0], bz[0] = 1, 1
    gc, qwc = stab.commute(stab.pack_paulis(ax, az), stab.pack_paulis(bx, bz), n)
    wg, wq = OC.commute_matrix(ax, az, bx, bz)
    assert np.array_equal(gc, wg) and np.array_equal(qwc, wq)
