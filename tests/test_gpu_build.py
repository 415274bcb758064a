"""The neighbour build where its kernels can go wrong: rows whose candidates exceed the kept hit
words (measured again by the fill), more slots than are walked together, sizes at the scan's
tile and one-block limits, single atoms.  Lists are compared bit for bit with the oracle's;
energies and forces of many-element systems in FP64 at the FP64 path's bounds (1e-12, 1e-10)."""
import numpy as np
import pytest

from synth import models, systems

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def rn():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2505_06711_amd as rn
    return rn


@pytest.fixture(scope="module")
def ctx(rn):
    return rn.Context(0)


def clump(n=600, far=9, seed=11):
    """A dense ball in a large open box: far more candidates per row than the mean."""
    rng = np.random.default_rng(seed)
    d = rng.normal(size=(n, 3))
    ball = d / np.linalg.norm(d, axis=1, keepdims=True) * 4.0 * rng.uniform(size=(n, 1)) ** (1 / 3)
    pos = np.concatenate([ball, rng.uniform(-90, 90, (far, 3))])
    return dict(pos=pos, species=np.zeros(len(pos), np.int32), cell=np.diag([1.0, 1.0, 1.0]),
                pbc=np.zeros(3, np.int32), elements=["Cu"])


def few(n, pbc, seed=12):
    rng = np.random.default_rng(seed)
    return dict(pos=rng.uniform(0, 9, (n, 3)), species=np.zeros(n, np.int32), cell=np.diag([9.0, 8.0, 10.0]),
                pbc=np.full(3, pbc, np.int32), elements=["Cu"])


CASES = {
    "clump": (clump, 6.0, 1.0, (1, 1, 1)),
    "one_open": (lambda: few(1, 0), 5.0, 0.5, (1, 1, 1)),
    "one_periodic": (lambda: few(1, 1), 5.0, 0.5, (1, 1, 1)),
    "two_open": (lambda: few(2, 0), 5.0, 0.5, (1, 1, 1)),
    "33_split": (lambda: few(33, 1), 3.0, 0.5, (2, 1, 2)),
    "scan_tile_4096": (lambda: systems.fcc_crystal((16, 16, 4), seed=13), 4.0, 0.5, (1, 1, 1)),
    "scan_one_block_16384": (lambda: systems.fcc_crystal((16, 16, 16), seed=14), 4.0, 0.5, (2, 2, 1)),
    "scan_three_launches": (lambda: systems.fcc_crystal((17, 16, 17), seed=15), 4.0, 0.5, (1, 1, 1)),
}


@pytest.mark.parametrize("case", list(CASES))
def test_list_bit_exact(rn, ctx, oracle_lib, case):
    make, r_c, skin, dec = CASES[case]
    s = make()
    print("case", case, len(s["pos"]), flush=True)
    got = rn.build_neighbors(ctx, s, r_c, skin, dec).export()
    want = oracle_lib.neighbors(s, r_c + skin, dec)
    for a, b in zip(got, want):
        np.testing.assert_array_equal(a, b)


@pytest.mark.parametrize("n_elements,decomp,exchange", [(2, (1, 1, 1), "messages"), (3, (2, 1, 1), "node_features"),
                                                        (7, (1, 1, 1), "messages"), (7, (2, 2, 1), "node_features")])
def test_many_elements(rn, ctx, oracle_lib, n_elements, decomp, exchange):
    """Slots (elements and the ghosts') walked in several batches."""
    el = ["E%d" % k for k in range(n_elements)]
    m = models.make_model(el, L=1, K=4, r_c=4.0, n_hidden=1, hidden=64, T_max=2, seed=16, bias_std=0.5,
                          ang_scale=0.25)
    s = systems.fcc_crystal((5, 4, 4), seed=16)
    s["species"] = np.random.default_rng(16).integers(0, n_elements, len(s["pos"])).astype(np.int32)
    s["elements"] = el
    print("elements", n_elements, decomp, exchange, flush=True)
    E, F, W = rn.energy_forces(ctx, rn.Model(m), s, T=2, precision="fp64", skin=0.5, decomp=decomp, exchange=exchange)
    ref = oracle_lib.evaluate(m, s, T=2)
    assert abs(E - ref["energy"]) <= 1e-12 * max(abs(ref["energy"]), np.abs(ref["atom_energy"]).sum())
    assert np.abs(F - ref["forces"]).max() <= 1e-10 * np.abs(ref["forces"]).max()
    assert np.abs(W - ref["virial"]).max() <= 1e-10 * np.abs(ref["virial"]).max()
