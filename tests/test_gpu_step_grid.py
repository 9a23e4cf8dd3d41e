"""Blocks of the vector-ALU step pass: a tile per block as long as all are resident
at once, and past that a grid that loops, of blocks that are resident together (the
looping kernel's registers allow two per CU) and no second round of them.  Results
on both sides of the change against the oracle, within the bounds of the other step
tests."""
import pytest

from test_gpu_parity import check_states, run_pair

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("P,fixcom,obabo", [(8, 0, 0), (8, 1, 1), (24, 0, 1), (48, 1, 0), (64, 0, 0)])
def test_looping_grid_is_resident(P, fixcom, obabo):
    import torch
    from paper_2602_13553_amd import inputs, pimd
    cus = torch.cuda.get_device_properties(0).multi_processor_count
    tile = 256 // P
    for blocks in (cus, 5 * cus + 1):          # (no CU holds five: 96 VGPRs at least)
        spec = inputs.harmonic_tiny(n_atoms=tile * blocks, n_beads=P, seed=P)
        spec.fixcom, spec.integrator = fixcom, obabo
        ctx = pimd.Context.from_spec(spec, flags=pimd.PIMD_FLAG_VALU_TRANSFORMS)
        info = ctx.launch_info()
        ctx.close()
        print("case grid P=%d tiles=%d blocks=%d" % (P, blocks, info["fused_blocks"]), flush=True)
        assert info["transforms"] == 0
        assert info["fused_blocks"] == (blocks if blocks == cus else 2 * cus)
        g, o = run_pair(spec, 3, chunks=[1, 2], flags=pimd.PIMD_FLAG_VALU_TRANSFORMS)
        check_states(g, o)
