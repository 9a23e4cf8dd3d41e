"""Neighbor lists built by testing every listed atom, 64 at a time and four such
chunks in flight: atom counts around the chunks' edges, lane groups of any size
(P = 3, 5, 7 do not divide a wave), the last size without centroid cells and the
first with them, and an odd number of listed atoms among others.  Against the
oracle, within the bounds of the other force tests."""
import pytest

from test_gpu_parity import check_states, run_pair

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("kind,N,P", [("lj", 255, 3), ("lj", 256, 5), ("lj", 257, 7), ("lj", 320, 1),
                                      ("lj", 4096, 2), ("lj", 4097, 2), ("water", 975, 4)])
def test_lists_match_oracle(kind, N, P):
    from paper_2602_13553_amd import inputs, pimd
    make = inputs.lj_liquid if kind == "lj" else inputs.water
    spec = make(n_atoms=N, n_beads=P, seed=N + P)
    ctx = pimd.Context.from_spec(spec)
    assert (ctx.launch_info()["cells"] > 0) == (N > 4096)
    ctx.close()
    g, o = run_pair(spec, 4, chunks=[1, 3])
    check_states(g, o)
