"""Bosons whose rings hardly exchange: every row of the recursion is carried by
one term (the particle's own ring), whose weight is 1 to the last bit, and so are
the products of such weights down the rows.  The oracle's recursion says that all
other links together stay below a rounding of 1, so the exact probabilities are
those of the identity; within two roundings of 1 (2^-52)."""
import numpy as np
import pytest

import oracle

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("N,P", [(64, 32), (256, 16), (500, 32)])
def test_link_probabilities_without_exchange(N, P):
    from paper_2602_13553_amd import inputs, pimd
    s = inputs.lj_bosons(n_atoms=N, n_beads=P, seed=11)
    wn = P * s.kB * s.temp / s.hbar
    k, bn = 0.5 * s.mass[0] * s.mvv2e * wn * wn, 1.0 / (P * s.kB * s.temp)
    print("case weak exchange N=%d P=%d" % (N, P), flush=True)
    prob = pimd.boson_spring(s.x0, k, bn, box=s.box)[3].cpu().numpy()
    want = oracle.boson_spring(s.x0, k, bn, box=s.box)[2]
    off = want - np.diag(np.diag(want))
    assert off.sum() < 2.0 ** -54, "the input exchanges"
    assert np.abs(prob - np.eye(N)).max() <= 2.0 ** -52, np.abs(prob - np.eye(N)).max()
