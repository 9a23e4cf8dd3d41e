"""Bonds: the minimum image at half a box and the force's rounding.

A bond of half a box's length has two nearest images; the one taken is the one
of d - L rint(d / L) with the quotient rounded as a division, as in the oracle
(the other reverses the force).  With r0 = 0 and a power of two for the force
constant K, the force -2 K (r - r0) / r is -2 K to the last bit wherever r is
exact, and then so are the virial and the pressure of a state at rest.  Atoms on
one point: the energy K r0^2 stands, the forces have no value."""
import numpy as np
import pytest

import oracle

pytestmark = pytest.mark.gpu


def _pairs(sep, box, k, r0):
    """One bond of vector sep per pair; no LJ, unit masses, one bead, at rest."""
    from paper_2602_13553_amd import inputs
    n = len(sep)
    x = np.zeros((1, 2 * n, 3))
    x[0, 1::2] = sep
    bonds = np.stack([2 * np.arange(n), 2 * np.arange(n) + 1], 1).astype(np.int32)
    return inputs.SystemSpec(
        name="bonds %d" % n, n_atoms=2 * n, n_beads=1, temp=1.0, kB=1.0, hbar=1.0, mvv2e=1.0, dt=2.0 ** -10,
        tau=1.0, tau_scale=1.0, ensemble=inputs.NVE, box=tuple(box), seed=1, potential=inputs.POT_WATER,
        mass=np.ones(2 * n), x0=x, v0=np.zeros_like(x), lj_eps=0.0, lj_sigma=1.0, lj_rc=min(box) / 4,
        bond_k=k, bond_r0=r0, skin=0.0, lj_active=np.zeros(2 * n, np.int32), bonds=bonds)


def _half_boxes():
    """Boxes L and distances d = (n + 1/2) L that d (1/L) puts at another image
    than d / L does."""
    found = []
    for q in range(200):
        L = 7.0 + q / 16.0 + 1.0 / 3.0
        for n in (-2.5, -1.5, 1.5, 2.5):
            for d in (np.nextafter(n * L, 0.0), n * L, np.nextafter(n * L, 100.0)):
                if np.rint(d * (1.0 / L)) != np.rint(d / L):
                    found.append((L, d))
    return found


def test_half_box_image():
    from paper_2602_13553_amd import pimd
    cases = _half_boxes()
    assert len(cases) >= 4
    for L, d in cases[:8]:
        print("case half box L=%r d=%r" % (L, d), flush=True)
        spec = _pairs([[d, 0.3, -0.2]], (L, L, L), 4.0, 0.96)
        ctx = pimd.Context.from_spec(spec)
        ctx.set_state(spec.x0, spec.v0, 0)
        ctx.step(1)
        x, p, _ = ctx.get_state()
        ctx.close()
        st = oracle.State.from_spec(spec)
        st.step(1)
        assert np.abs(p - st.p).max() <= 1e-12 * np.abs(st.p).max(), (L, d, p, st.p)
        assert np.abs(x - st.x).max() <= 1e-12 * np.abs(st.x).max()


def test_force_is_rounded_once():
    from paper_2602_13553_amd import pimd
    print("case bond force", flush=True)
    box, k = (16.0, 16.0, 16.0), 8.0
    off = []
    for q in range(96):
        r = (601 + 37 * q) * 2.0 ** -10       # r and r^2 exact
        spec = _pairs([[0.0, r, 0.0]], box, k, 0.0)
        ctx = pimd.Context.from_spec(spec)
        ctx.set_state(spec.x0, spec.v0, 0)
        e = ctx.estimators()
        ctx.close()
        assert e["epot"] == k * r * r
        off.append(e["pmd"] != (-2.0 * k * r * r) * (1.0 / (3.0 * 16.0 ** 3)))
    assert not any(off), "%d of %d bonds" % (sum(off), len(off))


def test_coincident_atoms():
    from paper_2602_13553_amd import pimd
    print("case coincident", flush=True)
    spec = _pairs([[0.0, 0.0, 0.0], [0.5, 0.0, 0.0]], (16.0,) * 3, 8.0, 0.75)
    ctx = pimd.Context.from_spec(spec)
    ctx.set_state(spec.x0, spec.v0, 0)
    assert ctx.estimators(check=False)["epot"] == 8.0 * (0.75 ** 2 + 0.25 ** 2)
    ctx.step(1)
    with pytest.raises(pimd.PimdError) as e:
        ctx.estimators()
    ctx.close()
    assert e.value.code == pimd.PIMD_ERR_NONFINITE
