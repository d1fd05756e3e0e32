"""The population kernels choose their shape by the sizes of the set and of the
population (column tiles per block, individuals per wave).  An individual's loss
must not depend on it: its products are the same, the force and virial sums are
integers, so equal bit for bit."""
import numpy as np
import pytest

from paper_2107_08119_amd import inputs as I

pytestmark = pytest.mark.gpu


def unlabelled(n_struct, n_min, n_max):
    st = I.training_structures(n_struct, n_min, n_max, 11)
    rng = np.random.default_rng(5)
    n = np.array([len(s.pos) for s in st], np.int32)
    return I.LabelledSet(n, np.stack([s.box.reshape(9) for s in st]), np.concatenate([s.pos for s in st]),
                         -4.0 * n, rng.standard_normal((int(n.sum()), 3)), rng.standard_normal((n_struct, 6)),
                         (np.arange(n_struct) % 3 > 0).astype(np.uint8))


@pytest.mark.parametrize("n_struct,n_min,n_max", [(3, 8, 20), (100, 40, 140), (300, 90, 120), (5, 300, 1100)])
def test_losses_do_not_depend_on_the_shape(n_struct, n_min, n_max):
    """From 1 to 67 individuals the four sets reach blocks of one to four column
    tiles; a structure of more than 845 atoms leaves room for fewer than 16."""
    import torch
    from paper_2107_08119_amd import nep
    rng = np.random.default_rng(1)
    Z = torch.from_numpy((0.1 * rng.standard_normal((67, 931))).astype(np.float32)).cuda()
    ctx = nep.Context(0)
    ctx.load_params(nep.hyper(), Z[0].cpu().numpy())
    ds = ctx.dataset_create(unlabelled(n_struct, n_min, n_max), 96)
    full = ctx.eval_population(ds, Z)
    for first, last in ((0, 1), (1, 16), (0, 16), (3, 20), (10, 43), (0, 50), (17, 67)):
        part = ctx.eval_population(ds, Z[first:last].contiguous())
        assert torch.equal(part, full[first:last]), (first, last)
    assert bool(torch.isfinite(full).all())
    ctx.synchronize()
