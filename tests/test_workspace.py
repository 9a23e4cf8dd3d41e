"""Device memory of a context (no GPU): admission counts on the state arrays that a
system cannot do without (positions, their modes, velocities, forces where they
are stored, and one staging array for states handed in and out); small systems
may stage positions and momenta side by side, for at most 1 MB more."""
import ctypes as C

import numpy as np
import pytest

from paper_2602_13553_amd import inputs, pimd


@pytest.mark.parametrize("kind,N,P,arrays", [("trap", 256, 8, 4), ("trap", 5461, 8, 4), ("trap", 4000, 16, 4), ("trap", 4000, 64, 4), ("trap", 20000, 64, 4),
                                             ("external", 4000, 32, 5)])
def test_state_arrays(kind, N, P, arrays):
    spec = inputs.harmonic_tiny(n_atoms=N, n_beads=P)
    if kind == "external":
        spec.potential = pimd.PIMD_POT_EXTERNAL
    p = pimd.params_from_spec(spec)
    n = C.c_size_t()
    mass = np.ascontiguousarray(spec.mass)
    assert pimd.load().pimd_workspace_bytes(C.byref(p), pimd._dp(mass), None, C.byref(n)) == 0
    # tables and sums: under 160 B an atom, a 128 B line per block of at least
    # two atoms, the matrices
    rest = 160 * N + 128 * (N // 2 + 2) + 16 * P * P + 65536
    arr = N * 3 * P * 8
    assert n.value <= (arrays + (arr <= 2 ** 20)) * arr + rest, n.value
