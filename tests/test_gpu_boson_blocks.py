"""The blocked solve of the bosonic exchange recursion at the sizes where its
64 x 64 tiles begin and end, over the range of link energies that its
(mantissa, exponent) pairs carry, and past that range, where the call goes
through the recursion in log space.  Against the oracle's recursion in
extended precision, at the exchange springs' bar (tests/test_gpu_boson.py):
1e-12 of V_B, EV_B, of the largest force, and absolute for probabilities."""
import sys

import numpy as np
import pytest

import oracle

pytestmark = pytest.mark.gpu

BAR = 1e-12


def _compare(x, k, b, box=None):
    from paper_2602_13553_amd import pimd
    v, ev, f, prob = pimd.boson_spring(x, k, b, box=box)
    f, prob = f.cpu().numpy(), prob.cpu().numpy()
    vo, fo, po, evo = oracle.boson_spring(x, k, b, with_ev=True, box=box)
    ef = np.abs(f - fo).max() / max(np.abs(fo).max(), 1e-300)
    ep = np.abs(prob - po).max()
    print("  V %.15e / %.15e  EV %.15e / %.15e  f rel %.3e  prob %.3e"
          % (v, vo, ev, evo, ef, ep), flush=True)
    assert abs(v - vo) <= BAR * max(1.0, abs(vo)), (v, vo)
    assert abs(ev - evo) <= BAR * max(1.0, abs(evo)), (ev, evo)
    assert ef <= BAR and ep <= BAR, (ef, ep)


@pytest.mark.parametrize("N,P", [(63, 3), (65, 1), (127, 2), (128, 5), (129, 2), (193, 4),
                                 (448, 2), (449, 3), (1023, 1)])
def test_tile_edges(N, P):
    """One row or column short of a tile, whole tiles, one past; two, three and
    more blocks (the columns summed ahead start with the third)."""
    rng = np.random.default_rng(N * 17 + P)
    print("case tiles N=%d P=%d" % (N, P), flush=True)
    sys.stdout.flush()
    _compare(rng.normal(0, 0.4, (P, N, 3)) + rng.normal(0, 1.2, (1, N, 3)), 1.1, 0.9)


@pytest.mark.parametrize("N,spread,k", [(130, 0.0, 1.1), (130, 30.0, 5.0), (97, 100.0, 1.0),
                                        (70, 500.0, 1.0)])
def test_link_range(N, spread, k):
    """Coincident rings (every term alike), links of thousands and of tens of
    thousands of kT (factors far below the smallest double), and links beyond
    the blocked solve's range."""
    rng = np.random.default_rng(int(N + spread + k))
    print("case links N=%d spread=%g k=%g" % (N, spread, k), flush=True)
    x = rng.normal(0, 0.01 if spread == 0.0 else 0.4, (4, N, 3)) + spread * rng.normal(0, 1, (1, N, 3))
    _compare(x, k, 1.0)


def test_stretched_rings():
    """Rings stretched by hundreds of kT in a row of far clusters: the terms
    that count are not the ones with the smallest closing link."""
    rng = np.random.default_rng(5)
    N = 140
    x = rng.normal(0, 0.3, (3, N, 3)) + 20.0 * (np.arange(N) % 3)[None, :, None]
    x[2] += rng.normal(0, 12.0, (N, 3))
    print("case stretched N=%d" % N, flush=True)
    _compare(x, 1.0, 1.0)
