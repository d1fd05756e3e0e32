"""Parameter gradient at atom counts around the contraction's steps (16 atoms
per wave, 64 per block, blocks striding over more): against the oracle's
float64 gradient to 1e-5, the bound of the other gradient tests (float32 terms
per atom, float64 sums)."""
import numpy as np
import pytest

import oracle as O
from paper_2107_08119_amd import inputs as I

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("sizes", [[1], [15], [16], [17], [64], [65], [47, 1, 90]])
@pytest.mark.parametrize("parts", ["energy", "both"])
def test_gradient_matches_oracle(sizes, parts):
    import torch
    from paper_2107_08119_amd import nep
    rng = np.random.default_rng(sum(sizes))
    pos, boxes = [], []
    for n in sizes:
        cells = I.smallest_supercell(n)
        p, box = I.diamond_supercell(*cells)
        pos.append(p[:n] + 0.1 * rng.standard_normal((n, 3)))
        boxes.append(box.reshape(9))
    S, N = len(sizes), sum(sizes)
    ls = I.LabelledSet(np.array(sizes, np.int32), np.array(boxes), np.concatenate(pos), np.zeros(S),
                       np.zeros((N, 3)), np.zeros((S, 6)), np.zeros(S, np.uint8))
    z = I.random_parameters(931, 5)
    gE = rng.standard_normal(S)
    gF = rng.standard_normal((N, 3)).astype(np.float32) * (parts == "both")
    ctx = nep.Context(0)
    ctx.load_params(nep.hyper(), z)
    ds = ctx.dataset_create(ls, 200)
    zt = torch.from_numpy(z).cuda()
    gF_dev = torch.from_numpy(np.ascontiguousarray(gF.T)).cuda() if parts == "both" else None
    F = ctx.dataset_compute(ds, zt)["F"]
    g = ctx.dataset_backward(ds, zt, torch.from_numpy(gE).cuda(), gF_dev, F, want_pos=True)
    ctx.synchronize()
    ref = O.grad_params(O.hyper(), z, ls, gE, gF.astype(np.float64), cap=200)
    got = g["z"].cpu().numpy()
    assert np.linalg.norm(got - ref) < 1e-5 * np.linalg.norm(ref)
    struct = np.repeat(np.arange(S), sizes)
    np.testing.assert_array_equal(g["pos"].cpu().numpy(), -gE[struct] * F.cpu().numpy().astype(np.float64))
