"""LJ with a sigma whose square underflows (a switched-off potential): no force, no
energy, and a free ring polymer's step."""
import numpy as np
import pytest

import oracle
from test_gpu_parity import TOL

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("sigma", [1e-156, 1e-170])
def test_vanishing_sigma(sigma):
    from paper_2602_13553_amd import inputs, pimd
    spec = inputs.lj_liquid(n_atoms=64, n_beads=4, seed=2)
    spec.lj_sigma = sigma
    print("case sigma %g" % sigma, flush=True)
    ctx = pimd.Context.from_spec(spec)
    ctx.set_state(spec.x0, spec.v0, 0)
    ctx.step(3)
    x, p, _ = ctx.get_state()
    e = ctx.estimators()
    ctx.close()
    st = oracle.State.from_spec(spec)
    st.step(3)
    assert e["epot"] == 0.0
    assert np.abs(x - st.x).max() <= TOL * np.abs(st.x).max()
    assert np.abs(p - st.p).max() <= TOL * np.abs(st.p).max()
