"""One context used for several systems in turn: what a build keeps for the next
one (cleared cell counters, grown buffers) must not reach another system's
lists.  Lists are whole numbers and equal a fresh context's."""
import numpy as np
import pytest

from paper_2107_08119_amd import inputs as I

pytestmark = pytest.mark.gpu


def crystal(k):
    return I.diamond_supercell(k, k, k)


def gas(n, edge):
    return edge * np.random.default_rng(n).random((n, 3)), edge * np.eye(3)


# bulk crystals sorted by several kernels with few cells, between them systems
# sorted by one block whose cells are more (dilute gases) or fewer, or none (a
# cell thinner than three list cutoffs)
@pytest.mark.parametrize("order", [
    [crystal(8), gas(1000, 60.0), crystal(8)],                     # 343, 1,000, 343 cells
    [crystal(10), gas(2000, 80.0), crystal(10), gas(4000, 90.0)],  # 729, 2,744, 729, 4,096
    [crystal(8), crystal(5), crystal(8), crystal(2), crystal(8)],  # 343, 64, 343, thin, 343
    [gas(3072, 85.0), crystal(8), gas(3073, 85.0)],
])
def test_lists_do_not_depend_on_earlier_systems(order):
    from paper_2107_08119_amd import nep
    z = I.random_parameters(931, 3)
    ctx = nep.Context(0)
    ctx.load_params(nep.hyper(), z)
    for pos, box in order:
        alone = nep.Context(0)
        alone.load_params(nep.hyper(), z)
        got, want = [], []
        for c, out in ((ctx, got), (alone, want)):
            c.build_neighbors(nep.soa(pos), box, skin=0.5, max_neighbors=64)
            out.append({k: v.cpu().numpy() for k, v in c.get_neighbors().items()})
            c.synchronize()
        assert want[0]["cnt_radial"].sum() > 0
        for key in want[0]:
            np.testing.assert_array_equal(got[0][key], want[0][key], err_msg=key)
