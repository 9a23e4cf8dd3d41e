"""More contexts at once than the 64 pinned control blocks of a process: the
rest read theirs through pageable memory, freed blocks are taken again, and all
read the same values (identical systems, so to the bit)."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu


def test_more_contexts_than_pinned_blocks():
    from paper_2602_13553_amd import inputs, pimd
    spec = inputs.harmonic_tiny()

    def run(ctx):
        ctx.set_state(spec.x0, spec.v0, 0)
        ctx.step(3)
        return ctx.estimators()

    ctxs = [pimd.Context.from_spec(spec) for _ in range(66)]
    est = [run(c) for c in ctxs]
    for c in ctxs[:40]:
        c.close()
    again = [pimd.Context.from_spec(spec) for _ in range(3)]
    est += [run(c) for c in again]
    states = [c.get_state()[0] for c in ctxs[40:] + again]
    for c in ctxs[40:] + again:
        c.close()
    assert all(e == est[0] for e in est)
    assert all(np.array_equal(x, states[0]) for x in states)
