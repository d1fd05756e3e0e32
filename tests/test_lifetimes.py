"""What the binding keeps alive, and in which order it lets go (no GPU needed, a
stand-in library): datasets and correlations are freed before their context,
whatever the order in which Python gives them up, and the tensors of an MD call
stay while the library knows their addresses."""
import ctypes
import gc

import pytest
import torch

from paper_2107_08119_amd import nep


class _Lib:
    def __init__(self):
        self.freed = []

    def nep_vvcf_create(self, h, n, lags, out):
        out._obj.value = 77
        return 0

    def __getattr__(self, name):
        def call(handle):
            self.freed.append((name, handle.value))
        return call


def things():
    ctx = nep.Context.__new__(nep.Context)
    lib = _Lib()
    ctx._lib, ctx._h = lib, ctypes.c_void_p(1)
    sets = [nep.Dataset(ctx, ctypes.c_void_p(k), 1, 8) for k in (11, 12)]
    return lib, ctx, sets, nep.Correlation(ctx, 8, 4)


WANT = [("nep_dataset_destroy", 11), ("nep_dataset_destroy", 12), ("nep_vvcf_destroy", 77)]


@pytest.mark.parametrize("first", [0, 1, 2, 3])
def test_reference_cycle(first):
    lib, ctx, sets, corr = things()
    order = [ctx, sets[0], sets[1], corr]
    order = order[first:] + order[:first]
    order.append(order)  # one cycle that holds them all, as a traceback does
    ctx.cycle = order
    del ctx, sets, corr, order
    gc.collect()
    assert sorted(lib.freed[:-1]) == WANT and lib.freed[-1] == ("nep_destroy", 1)


def test_context_closed_first_or_last():
    lib, ctx, sets, corr = things()
    sets[0].close()
    ctx.close()
    assert not sets[1]._h and not corr._h  # no dangling handles
    for x in (*sets, corr, ctx):
        x.close()
    assert sorted(lib.freed[:-1]) == WANT and lib.freed[-1] == ("nep_destroy", 1)
    lib, ctx, sets, corr = things()
    for x in (corr, *sets, ctx):
        x.close()
    assert sorted(lib.freed[:-1]) == WANT and lib.freed[-1] == ("nep_destroy", 1)


def test_md_tensors_stay_while_their_addresses_count(monkeypatch):
    monkeypatch.setattr(nep, "_ptr", lambda t: t)
    ctx = nep.Context.__new__(nep.Context)
    ctx.device, ctx.n, ctx.cap, ctx._h = 0, 20000, 16, None

    class Lib:
        def __getattr__(self, name):
            return lambda *a: 0

    ctx._lib = Lib()

    def state():
        return torch.zeros((3, ctx.n), dtype=torch.float64)

    taken = set()
    for _ in range(20):  # each call on new tensors: none may lie where one before it did
        p, v = state(), state()
        here = {p.data_ptr(), v.data_ptr()}
        assert not here & taken
        ctx.md_step(1, 1.0, 10, 28.0, p, v)
        taken = here
        del p, v
    ctx.build_neighbors(state(), torch.eye(3).numpy(), 0.5, 16)
    assert ctx._md_buffers is None
