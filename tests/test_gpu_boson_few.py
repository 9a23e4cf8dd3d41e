"""Exchange springs and the bosonic step of very few particles, on both sides of
the number up to which the recursion runs in log space instead of the blocked
solve.  Against the oracle at the exchange springs' bar (tests/test_gpu_boson.py):
1e-12 of V_B, EV_B, of the largest force, and absolute for probabilities."""
import numpy as np
import pytest

from test_gpu_boson import _boson_pair, _check_boson
from test_gpu_boson_blocks import _compare

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("N", [1, 2, 3, 5, 6, 7])
@pytest.mark.parametrize("P", [1, 4, 33])
def test_springs(N, P):
    rng = np.random.default_rng(N * 100 + P)
    print("case few N=%d P=%d" % (N, P), flush=True)
    x = rng.normal(0, 0.4, (P, N, 3)) + rng.normal(0, 1.2, (1, N, 3))
    _compare(x, 1.1, 0.9)
    _compare(x, 1.1, 0.9, box=[2.5, 0.0, 3.0])


@pytest.mark.parametrize("N,integrator", [(2, 0), (5, 1), (6, 0)])
def test_steps(N, integrator):
    from paper_2602_13553_amd import inputs
    spec = inputs.trapped_bosons(n_atoms=N, n_beads=8, integrator=integrator, seed=N)
    _check_boson(_boson_pair(spec, 40, chunks=[32, 8]))
