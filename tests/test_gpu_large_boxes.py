"""Lists of a few atoms in boxes of more cells than the scan of the cell counts
serves (2^20), against the oracle's float64 predicate, and the static
evaluation on one of them."""
import numpy as np
import pytest

import oracle as O
from paper_2107_08119_amd import inputs as I

pytestmark = pytest.mark.gpu


def droplets(n, edges, seed):
    """Atoms in droplets at places all over the box, some across its faces."""
    rng = np.random.default_rng(seed)
    centre = rng.random((20, 3))
    centre[:4] = [[0, 0, 0], [0.999, 0.5, 0.001], [0.5, 0.999, 0.5], [0.3, 0.4, 1.0]]
    pos = centre[rng.integers(0, 20, n)] * edges + rng.uniform(-7.0, 7.0, (n, 3))
    return pos, np.diag(edges)


@pytest.mark.parametrize("n,edges", [(3500, (570.0, 560.0, 565.0)),      # 103 x 101 x 102 cells of 5.5 A
                                     (3500, (1200.0, 900.0, 1000.0)),
                                     (4000, (20.0, 17.0, 700000.0)), (500, (900.0, 901.0, 902.0))])
def test_lists_match_oracle(n, edges):
    from paper_2107_08119_amd import nep
    pos, box = droplets(n, np.array(edges), n)
    cap = 256
    ctx = nep.Context(0)
    ctx.load_params(nep.hyper(), I.random_parameters(931, 3))
    ctx.build_neighbors(nep.soa(pos), box, skin=0.5, max_neighbors=cap)
    nb = {k: v.cpu().numpy() for k, v in ctx.get_neighbors().items()}
    ctx.synchronize()
    for rc, which in ((5.5, "cnt_radial"), (4.5, "cnt_angular")):
        cnt, jl, img = O.neighbor_arrays(pos, box, rc, cap=cap)
        np.testing.assert_array_equal(nb[which], cnt)
        for i in range(0, n, 17):
            c = cnt[i]
            want = sorted(zip(jl[i, :c].tolist(), map(tuple, img[i, :c].tolist())))
            got = sorted(zip(nb["nbr"][:c, i].tolist(), map(tuple, nb["img"][:c, i].tolist())))
            assert got == want


def test_static_evaluation_of_a_large_box():
    import torch
    from paper_2107_08119_amd import nep
    pos, box = droplets(1500, np.array([600.0, 650.0, 640.0]), 5)
    ctx = nep.Context(0)
    ctx.load_params(nep.hyper(), I.random_parameters(931, 3))
    p = nep.soa(pos)
    ctx.build_neighbors(p, box, skin=0.5, max_neighbors=96)
    want = ctx.compute(p)
    got = {"F": torch.empty_like(want["F"]), "U": torch.empty_like(want["U"])}
    ctx.evaluate_static(p, box, got, max_neighbors=96)
    ctx.synchronize()
    assert torch.equal(got["F"], want["F"]) and torch.equal(got["U"], want["U"])
