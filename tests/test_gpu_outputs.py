"""Results of one evaluation do not depend on which of them are asked for, at
atom counts around the copy kernel's blocks; the static call gives the same.
Every result is copied or summed once in a fixed order: equal bit for bit."""
import numpy as np
import pytest

from paper_2107_08119_amd import inputs as I

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n", [1, 255, 256, 257, 1000])
def test_outputs_do_not_depend_on_the_others(n):
    import torch
    from paper_2107_08119_amd import nep
    rng = np.random.default_rng(n)
    pos, box = I.diamond_supercell(*I.smallest_supercell(n)) if n > 1 else I.diamond_supercell(3, 3, 3)
    p = nep.soa(pos[rng.permutation(len(pos))[:n]] + 0.05 * rng.standard_normal((n, 3)))
    v = nep.soa(0.01 * rng.standard_normal((n, 3)))
    ctx = nep.Context(0)
    ctx.load_params(nep.hyper(), I.random_parameters(931, 3))
    ctx.build_neighbors(p, box, max_neighbors=64)
    full = {k: t.clone() for k, t in ctx.compute(p, v).items()}
    blank = lambda keys: {k: torch.full_like(full[k], float("nan")) for k in keys}  # noqa: E731
    for keys in (["F"], ["F", "U"], ["F", "W"], ["F", "J"], ["F", "U", "totals"], ["F", "W", "J", "totals"]):
        out = ctx.compute(p, v, out=blank(keys))
        assert all(torch.equal(out[k], full[k]) for k in keys), keys
    out = ctx.evaluate_static(p, box, blank(["F", "U", "W", "J", "totals"]), v, max_neighbors=64)
    assert all(torch.equal(out[k], full[k]) for k in full)
    ctx.synchronize()
