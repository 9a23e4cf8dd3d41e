"""The conversions between the caller's layout [P][N][3] and the device layout
[N][3][P] at the edges of their tiles of 8, 16 and 32 atoms, for beads below,
at and past one wave, and through the internal atom order (LJ-active atoms
first).  Positions come back bit for bit; momenta are m M^T (M v), two
transforms of P terms: 4 P eps of the largest momentum, under 2e-13."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("N,P", [(1, 1), (7, 3), (9, 64), (8, 65), (33, 128), (16383, 5), (16384, 2),
                                 (16385, 64), (16401, 65), (0, 8)])
def test_state_round_trip(N, P):
    import torch
    from paper_2602_13553_amd import inputs, pimd
    if N:
        spec = inputs.free_ring_polymer(n_atoms=N, n_beads=P, seed=N + P)
    else:
        spec = inputs.water(n_atoms=648, n_beads=P, seed=3)
    print("case layout N=%d P=%d" % (spec.n_atoms, P), flush=True)
    ctx = pimd.Context.from_spec(spec)
    ctx.set_state(spec.x0, spec.v0, 5)
    xd = torch.full((P, spec.n_atoms, 3), -1.0, dtype=torch.float64, device="cuda")
    ctx.get_positions(xd)
    x, p, step = ctx.get_state()
    ctx.close()
    assert step == 5
    assert np.array_equal(x, spec.x0) and np.array_equal(xd.cpu().numpy(), spec.x0)
    want = spec.mass[None, :, None] * spec.v0
    assert np.abs(p - want).max() <= 4 * P * 2.3e-16 * np.abs(want).max()
