"""Gradient paths chosen by what is asked for and by the neighbour count: the
position gradient alone (no parameter gradient), an output that the objective
does not use, and atoms with fewer and more neighbours than the backward pass
keeps in LDS (40), against the oracle's float64 gradient to 1e-5, the bound of
the other gradient tests (float32 terms per atom, float64 sums)."""
import numpy as np
import pytest

import oracle as O
from paper_2107_08119_amd import inputs as I

pytestmark = pytest.mark.gpu


def scaled_set(sizes, scale, seed):
    rng = np.random.default_rng(seed)
    pos, boxes = [], []
    for n in sizes:
        p, box = I.diamond_supercell(*I.smallest_supercell(n))
        pos.append(scale * (p[:n] + 0.1 * rng.standard_normal((n, 3))))
        boxes.append(scale * box.reshape(9))
    S, N = len(sizes), sum(sizes)
    return I.LabelledSet(np.array(sizes, np.int32), np.array(boxes), np.concatenate(pos), np.zeros(S),
                         np.zeros((N, 3)), np.zeros((S, 6)), np.zeros(S, np.uint8))


def setup(ls, z):
    import torch
    from paper_2107_08119_amd import nep
    ctx = nep.Context(0)
    ctx.load_params(nep.hyper(), z)
    return ctx, ctx.dataset_create(ls, 200), torch.from_numpy(z).cuda()


@pytest.mark.parametrize("scale,least,most", [(1.0, 1, 40), (0.88, 30, 60), (0.8, 41, 100)])
def test_gradient_by_neighbour_count(scale, least, most):
    import torch
    ls = scaled_set([64, 8, 33], scale, 7)
    z = I.random_parameters(931, 6)
    ctx, ds, zt = setup(ls, z)
    mean = ds.pairs()[0] / ds.n_atoms
    assert least <= mean <= most
    rng = np.random.default_rng(8)
    gE = rng.standard_normal(3)
    gF = rng.standard_normal((ds.n_atoms, 3)).astype(np.float32)
    g = ctx.dataset_backward(ds, zt, torch.from_numpy(gE).cuda(),
                             torch.from_numpy(np.ascontiguousarray(gF.T)).cuda())
    ref = O.grad_params(O.hyper(), z, ls, gE, gF.astype(np.float64), cap=200)
    got = g["z"].cpu().numpy()
    assert np.linalg.norm(got - ref) < 1e-5 * np.linalg.norm(ref)


@pytest.mark.parametrize("pos_grad,z_grad", [(True, False), (False, True), (True, True)])
def test_gradients_asked_for(pos_grad, z_grad):
    import torch
    from paper_2107_08119_amd import nep
    ls = scaled_set([64, 1, 17], 1.0, 9)
    ctx, ds, z0 = setup(ls, I.random_parameters(931, 11))
    pairs = ds.pairs()
    w = torch.tensor([1.5, -2.0, 0.25], dtype=torch.float64, device="cuda")
    pos = ctx.dataset_positions(ds).clone().requires_grad_(pos_grad)
    z = z0.clone().requires_grad_(z_grad)
    E, F = nep.NEPEnergy.apply(pos, z, ctx, ds)
    (w * E).sum().backward()
    want = ctx.dataset_backward(ds, z0, w, torch.zeros_like(F), F.detach(), want_pos=True)
    assert (pos.grad is not None) == pos_grad and (z.grad is not None) == z_grad
    if pos_grad:
        assert torch.equal(pos.grad, want["pos"])
    if z_grad:
        assert torch.equal(z.grad, want["z32"])
    if not pos_grad:  # the energies unused
        z.grad = None
        v = torch.randn_like(F)
        (v * nep.NEPEnergy.apply(pos, z, ctx, ds)[1]).sum().backward()
        assert torch.equal(z.grad, ctx.dataset_backward(ds, z0, None, v)["z32"])
    ctx.dataset_set_positions(ds, ctx.dataset_positions(ds))
    assert ds.pairs() == pairs
    with pytest.raises(ValueError):
        ctx._position_gradient(ds, w, F.detach()[:2])
