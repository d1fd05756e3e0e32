"""The force kernel of every model size where its tiles have remainders: atom
counts around a block (4 and 16 atoms), list lengths around its staged slots
(48 and 64), angular pair counts around its 4, 8 and 16 pairs per product,
runtime-sized models down to one radial function and one neuron; one and two
species.  Against the float64 oracle at 1e-5 relative (norm over all
components), the bound of the other force tests."""
import numpy as np
import pytest

import oracle as O
from paper_2107_08119_amd import inputs as I

pytestmark = pytest.mark.gpu
TOL = 1e-5

MODELS = {  # r_c^R, r_c^A, n_max^R, n_max^A, l_max, N_neu
    "si_80_50_1": (5.0, 5.0, 15, 15, 4, 50),
    "pbte_41_40_1": (8.0, 4.0, 12, 6, 4, 40),
    "wide": (9.0, 6.0, 9, 8, 3, 64),     # about 180 slots and 45 angular pairs
    "odd": (6.5, 4.5, 3, 9, 2, 17),
    "least": (5.0, 2.9, 0, 0, 1, 1),     # 4-5 angular pairs
}


def rel(a, b):
    a, b = np.asarray(a, np.float64), np.asarray(b, np.float64)
    return float(np.linalg.norm(a - b) / np.linalg.norm(b))


@pytest.mark.parametrize("species", [False, True])
@pytest.mark.parametrize("n", [1, 15, 16, 17, 33])
@pytest.mark.parametrize("model", list(MODELS))
def test_tiles_match_oracle(model, n, species):
    from paper_2107_08119_amd import nep
    rng = np.random.default_rng(n)
    edge = max((n / 0.05) ** (1.0 / 3.0), 0.55 * (MODELS[model][0] + 0.5))
    grid = int(np.ceil(n ** (1.0 / 3.0)))
    sites = np.array(np.unravel_index(rng.permutation(grid ** 3)[:n], (grid,) * 3)).T
    pos = (sites + 0.5) * edge / grid + 0.15 * rng.standard_normal((n, 3))
    box = np.diag(edge * np.array([1.0, 1.02, 1.05]))
    vel = 0.01 * rng.standard_normal((n, 3))
    h, oh = nep.hyper(*MODELS[model]), O.hyper(*MODELS[model])
    z = I.random_parameters(nep.num_params(h), 7, std=0.03)
    Z = rng.choice([14, 32], n).astype(np.int32) if species else None
    if species:  # O(1) pre-activations, as in a trained model
        z[:h.n_neuron * nep.num_descriptors(h)] *= np.float32(1.0 / 100.0)
    ctx = nep.Context(0)
    ctx.load_params(h, z)
    ctx.set_tile(64)
    p = nep.soa(pos)
    ctx.build_neighbors(p, box, skin=0.5, max_neighbors=400)
    if species:
        ctx.set_species(Z)
    out = ctx.compute(p, nep.soa(vel))
    ctx.synchronize()
    ref = O.nep_eval(oh, z, pos, box, vel=vel, cap=400, Z=Z)
    assert rel(out["U"].cpu().numpy(), ref["U"]) < TOL
    if n > 1:  # one atom: the forces of its images cancel
        assert rel(nep.aos(out["F"]), ref["F"]) < TOL
    assert rel(nep.aos(out["W"]).reshape(-1, 3, 3), ref["W"]) < TOL
    assert rel(nep.aos(out["J"]), ref["J"]) < TOL


@pytest.mark.parametrize("model,n", [("si_80_50_1", 2048), ("si_80_50_1", 2049), ("si_80_50_1", 2063),
                                     ("pbte_41_40_1", 2064), ("wide", 2065), ("odd", 2063),
                                     ("si_29_30_1", 2049), ("si_29_30_1", 4096), ("si_29_30_1", 4097),
                                     ("si_29_30_1", 8192), ("si_29_30_1", 8193)])
def test_shapes_chosen_by_size_match_oracle(model, n):
    """Around the sizes where the kernel's shape changes: the first, last and
    some other atoms of a jittered lattice with vacancies."""
    from paper_2107_08119_amd import nep
    rng = np.random.default_rng(n)
    cells = int(np.ceil((n / 8) ** (1.0 / 3.0)))
    if model == "pbte_41_40_1":
        pos, box, Z, _ = I.rocksalt_supercell(cells, cells, cells)
    else:
        pos, box = I.diamond_supercell(cells, cells, cells)
        Z = None
    keep = np.sort(rng.permutation(len(pos))[:n])
    pos = pos[keep] + 0.08 * rng.standard_normal((n, 3))
    Z = None if Z is None else Z[keep]
    vel = 0.01 * rng.standard_normal((n, 3))
    sizes = MODELS.get(model, (5.0, 4.0, 8, 4, 4, 30))
    h, oh = nep.hyper(*sizes), O.hyper(*sizes)
    z = I.random_parameters(nep.num_params(h), 7, std=0.03)
    if Z is not None:
        z[:h.n_neuron * nep.num_descriptors(h)] *= np.float32(1.0 / 300.0)
    ctx = nep.Context(0)
    ctx.load_params(h, z)
    p = nep.soa(pos)
    ctx.build_neighbors(p, box, skin=0.5, max_neighbors=256)
    if Z is not None:
        ctx.set_species(Z)
    out = ctx.compute(p, nep.soa(vel))
    ctx.synchronize()
    sel = np.unique(np.concatenate([[0, 1, n - 2, n - 1], rng.integers(0, n, 60)])).astype(np.int32)
    ref = O.nep_eval(oh, z, pos, box, vel=vel, sel=sel, Z=Z)
    assert rel(out["U"].cpu().numpy()[sel], ref["U"]) < TOL
    assert rel(nep.aos(out["F"])[sel], ref["F"]) < TOL
    assert rel(nep.aos(out["W"]).reshape(-1, 3, 3)[sel], ref["W"]) < TOL
    assert rel(nep.aos(out["J"])[sel], ref["J"]) < TOL
