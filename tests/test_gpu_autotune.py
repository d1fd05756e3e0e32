"""The pass-1 tuner against the choice by system size: in a small system, where
the kernel of every model size is clearly the fastest (8.9 against 14.6 us at
1,000 atoms), tuning leaves that choice in place; an explicit shape overrides
it.  The kernels sum in different orders, so the forces' bits tell them apart."""
import pytest

from paper_2107_08119_amd import inputs as I

pytestmark = pytest.mark.gpu


def test_tuning_a_small_system_keeps_the_choice_by_size():
    import torch
    from paper_2107_08119_amd import nep
    pos, box = I.diamond_supercell(5, 5, 5)
    ctx = nep.Context(0)
    ctx.load_params(nep.hyper(), I.random_parameters(931, 3))
    p = nep.soa(pos + 0.02 * pos[:, ::-1] % 0.3)
    ctx.build_neighbors(p, box, skin=0.5, max_neighbors=96)
    by_size = ctx.compute(p)["F"]
    lanes, ms = ctx.autotune(p, reps=50)
    assert lanes in (2, 4, 8) and len(ms) == 3
    assert torch.equal(ctx.compute(p)["F"], by_size)
    ctx.set_tile(lanes)
    assert not torch.equal(ctx.compute(p)["F"], by_size)
    ctx.synchronize()
