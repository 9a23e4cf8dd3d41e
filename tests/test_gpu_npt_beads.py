"""The barostat's passes at the bead counts where their mode matrix is the last
to be staged in LDS (64) and the first read in place (65, 96, 128), and with
more blocks than one batch of the finalizes' reads holds (N = 700 at P = 64: 175
blocks of 4 atoms, against 128 rows; the anisotropic barostat's at 64), both
splittings.  Against the oracle within the bounds of the other barostat tests."""
import pytest

from paper_2602_13553_amd import inputs
from test_gpu_npt import _aniso, _barostat, _stretch, check, run_both

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("N,P,aniso,integrator", [
    (64, 64, 0, 0), (64, 65, 0, 1), (65, 96, 1, 0), (64, 128, 1, 1), (700, 64, 0, 1), (270, 64, 1, 0)])
def test_barostat_bead_counts(N, P, aniso, integrator):
    spec = inputs.lj_liquid(n_atoms=N, n_beads=P, seed=70 + P)
    if aniso:
        spec = _aniso(_stretch(spec, (1.05, 1.0, 0.97)), 2, 1.0, 0.3, integrator)
    else:
        spec = _barostat(spec, 2, 1.0, 0.3, integrator)
    g, st = run_both(spec, [1, 3])
    check(g, st)
