"""Datasets and correlations are freed before their context, whatever the order
in which Python gives them up (no GPU needed): a stand-in library records the
calls that free them."""
import ctypes
import gc

import pytest

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
    for x in (*sets, corr, ctx):
        x.close()
    assert sorted(lib.freed[:-1]) == WANT and lib.freed[-1] == ("nep_destroy", 1)
    lib, ctx, sets, corr = things()
    for x in (corr, *sets, ctx):
        x.close()
    assert sorted(lib.freed[:-1]) == WANT and lib.freed[-1] == ("nep_destroy", 1)
