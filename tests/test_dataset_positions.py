"""Which positions a differentiable dataset evaluation uses (no GPU needed): the
binding around a stand-in library that keeps the positions it is handed and
returns their sums, so that a result from an earlier call's positions shows."""
import numpy as np
import pytest
import torch

from paper_2107_08119_amd import nep

N = 20000  # large enough that the allocator hands a freed block out again


class _Lib:
    """Energies are the sums of the positions held; status of the next upload."""

    def __init__(self):
        self.pos, self.status, self.uploads = torch.empty((3, N), dtype=torch.float64), 0, 0

    def nep_dataset_set_positions(self, h, d, pos):
        self.pos.copy_(pos)
        self.uploads += 1
        status, self.status = self.status, 0
        return status

    def nep_dataset_compute(self, h, d, z, E, F, W):
        E.fill_(self.pos.sum())
        F.copy_(-self.pos)
        return 0

    def nep_dataset_backward(self, h, d, z, gE, gF, F, gpos, gz, gz32):
        gz.fill_(self.pos.sum() * gE.sum())
        gz32.copy_(gz)
        if gpos is not None:
            gpos.copy_(-gE.sum() * F)
        return 0

    def nep_md_step(self, h, steps, dt, every, mass, pos, vel, thermo, W, J):
        pos.numpy()[:] += 1.0  # unseen by the version counter, as a kernel's writes
        return 0

    def nep_last_error(self, h):
        return b"list overflow"


@pytest.fixture
def held(monkeypatch):
    monkeypatch.setattr(nep, "_ptr", lambda t: t)
    ctx = nep.Context.__new__(nep.Context)
    ctx._lib, ctx._h, ctx.device, ctx.hyper = _Lib(), None, "cpu", nep.hyper()
    ds = nep.Dataset(ctx, None, 2, N)
    monkeypatch.setattr(ctx, "dataset_positions", lambda ds: ctx._lib.pos.clone(), raising=False)
    z = torch.zeros(nep.num_params(ctx.hyper))
    yield ctx, ds, z


def base():
    return torch.from_numpy(np.random.default_rng(1).random((3, N)))


def energy(pos, z, ctx, ds):
    return float(nep.NEPEnergy.apply(pos, z, ctx, ds)[0][0].detach())


def test_temporary_positions(held):
    # a temporary freed after each call: the allocator hands its address out again
    ctx, ds, z = held
    p = base()
    wants = [float((p + k).sum()) for k in range(50)]
    for k, want in enumerate(wants):
        assert energy((p + k).requires_grad_(), z, ctx, ds) == want


def test_positions_set_directly_or_in_place(held):
    ctx, ds, z = held
    p = base().requires_grad_()
    first = energy(p, z, ctx, ds)
    ctx.dataset_set_positions(ds, base() + 1.0)
    assert energy(p, z, ctx, ds) == first
    with torch.no_grad():
        p.add_(2.0)
    assert energy(p, z, ctx, ds) == float(p.detach().sum())


def test_positions_moved_by_md(held):
    ctx, ds, z = held
    ctx.n = N
    p = base()
    energy(p, z, ctx, ds)
    ctx.md_step(2, 1.0, 10, 28.0, p, torch.zeros_like(p))
    assert energy(p, z, ctx, ds) == float(p.sum())


def test_failed_upload_is_not_taken_for_the_one_before(held):
    ctx, ds, z = held
    p, q = base(), base() + 3.0
    first = energy(p, z, ctx, ds)
    ctx._lib.status = nep.NEP_EOVERFLOW
    with pytest.raises(nep.NepError):
        energy(q, z, ctx, ds)
    assert energy(p, z, ctx, ds) == first


def test_unchanged_positions_are_uploaded_once(held):
    ctx, ds, z = held
    p = base().requires_grad_()
    for view in (p, p, p.detach(), p.view(3, N)):
        energy(view, z, ctx, ds)
    assert ctx._lib.uploads == 1
    with pytest.raises(ValueError):
        energy(p.detach().view(N, 3), z, ctx, ds)


@pytest.mark.parametrize("later", ["frame", "set", "back"])
def test_parameter_gradient_at_the_positions_of_its_call(held, later):
    ctx, ds, z = held
    z.requires_grad_()
    p, q = base(), base() + 2.0
    E = nep.NEPEnergy.apply(p, z, ctx, ds)[0]
    if later == "set":
        ctx.dataset_set_positions(ds, q)
    else:  # "back": another frame and the first one again
        for frame in ((q,) if later == "frame" else (q, p)):
            nep.NEPEnergy.apply(frame, z, ctx, ds)
    now = ctx._lib.pos.clone()
    E.sum().backward()
    assert float(z.grad[0]) == float((p.sum() * len(E)).float())
    assert torch.equal(ctx._lib.pos, now)  # the dataset is left as it was


def test_parameter_gradient_of_positions_that_are_gone(held):
    ctx, ds, z = held
    z.requires_grad_()
    p = base()
    E = nep.NEPEnergy.apply(p, z, ctx, ds)[0]
    want = float((p.sum() * len(E)).float())
    p.add_(1.0)
    E.sum().backward(retain_graph=True)  # the dataset still has the first ones
    assert float(z.grad[0]) == want
    nep.NEPEnergy.apply(p, z, ctx, ds)
    with pytest.raises(RuntimeError, match="in place"):
        E.sum().backward()
