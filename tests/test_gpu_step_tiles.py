"""The step, closing and estimator passes with a tile per block and, past the
grid, several tiles per block: at P = 128 a tile is two atoms and the card runs
256 of its blocks, so 512 atoms are the last that fit; 513 and 771 take the
loop, with a ragged last tile.  Against the oracle, within the bounds of the
other step tests (rounding of the same sums in another order)."""
import pytest

from test_gpu_parity import check_states, run_pair

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("kind,N,fixcom,obabo", [
    ("harmonic", 512, 0, 0), ("harmonic", 513, 1, 1), ("harmonic", 771, 0, 1),
    ("lj", 512, 1, 0), ("lj", 513, 0, 0), ("lj", 513, 1, 1)])
def test_step_passes_around_the_grid(kind, N, fixcom, obabo):
    from paper_2602_13553_amd import inputs, pimd
    make = inputs.harmonic_tiny if kind == "harmonic" else inputs.lj_liquid
    spec = make(n_atoms=N, n_beads=128, seed=N)
    spec.fixcom = fixcom
    spec.integrator = pimd.PIMD_OBABO if obabo else pimd.PIMD_BAOAB
    g, o = run_pair(spec, 3, chunks=[1, 2])
    check_states(g, o)
