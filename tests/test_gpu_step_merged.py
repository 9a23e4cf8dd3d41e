"""A small system's force pass, which takes the rebuild decision and carries the
step's finalize as one of its blocks, against the pass and the finalize as
launches of their own (profiled steps): bit for bit, through rebuilds, for one
and two atoms' worth of blocks, at the last size that does so (512 step-pass
blocks) and the first that does not, with fixcom, bonds, a box of several
images, and non-power-of-two beads."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("kind,N,P,fixcom,obabo", [
    ("lj", 30, 4, 0, 0), ("lj", 257, 7, 0, 0), ("lj", 1021, 8, 1, 0), ("lj", 1100, 16, 1, 1),
    ("lj", 2048, 64, 0, 0), ("lj", 2052, 64, 0, 1), ("water", 387, 8, 0, 0), ("water", 1536, 33, 1, 1)])
def test_step_equals_separate_finalize(kind, N, P, fixcom, obabo):
    from paper_2602_13553_amd import inputs, pimd
    make = inputs.lj_liquid if kind == "lj" else inputs.water
    spec = make(n_atoms=N, n_beads=P, seed=N)
    spec.fixcom = fixcom
    spec.integrator = pimd.PIMD_OBABO if obabo else pimd.PIMD_BAOAB
    spec.skin = 0.05 if kind == "lj" else spec.skin   # rebuilds every few steps
    print("case merged %s N=%d P=%d" % (kind, N, P), flush=True)
    res = []
    for profiled in (False, True):
        ctx = pimd.Context.from_spec(spec, flags=pimd.PIMD_FLAG_VALU_TRANSFORMS)
        ctx.set_state(spec.x0, spec.v0, 0)
        if profiled:
            ctx.profile_begin()
        for n in (1, 70, 3):
            ctx.step(n)
        if profiled:
            ctx.profile_end()
        res.append((ctx.get_state(), ctx.estimators()))
        ctx.close()
    (xa, pa, sa), ea = res[0]
    (xb, pb, sb), eb = res[1]
    assert sa == sb == 74
    assert np.array_equal(xa, xb) and np.array_equal(pa, pb)
    assert ea == eb
