"""The FP64 NN kernels against the FP64 oracle at the FP64 path's bounds (1e-12 of the summed atomic energies,
1e-10 of the largest force and virial component): row counts at the edges of their 16-row tiles,
every (L, K) and width they are compiled for with one to four hidden layers, the launch's segments
and ghosts' rows, and the evaluation that may not allocate, which runs layer by layer until a plan has
packed the operands."""
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


def check(out, ref):
    E, F, W = out
    assert abs(E - ref["energy"]) <= 1e-12 * max(abs(ref["energy"]), np.abs(ref["atom_energy"]).sum())
    assert np.abs(F - ref["forces"]).max() <= 1e-10 * np.abs(ref["forces"]).max()
    assert np.abs(W - ref["virial"]).max() <= 1e-10 * np.abs(ref["virial"]).max()


@pytest.mark.parametrize("hidden,n", [(128, 2), (128, 15), (128, 16), (128, 17), (64, 33), (64, 48)])
def test_row_counts(rn, ctx, oracle_lib, hidden, n):
    print("rows", n, hidden, flush=True)
    m = models.make_model(["Cu"], L=2, K=12, r_c=4.0, n_hidden=3, hidden=hidden, T_max=2, seed=31, bias_std=1.0,
                          ang_scale=0.25)
    s = systems.fcc_crystal((4, 4, 4), seed=31)
    order = np.argsort((s["pos"] ** 2).sum(1), kind="stable")[:n]   # an open cluster
    s = dict(s, pos=s["pos"][order], species=s["species"][order], pbc=np.zeros(3, np.int32))
    check(rn.energy_forces(ctx, rn.Model(m), s, T=2, precision="fp64", skin=0.3), oracle_lib.evaluate(m, s, T=2))


@pytest.mark.parametrize("L,K", [(2, 12), (2, 8), (2, 4), (1, 4), (0, 12), (0, 8)])
@pytest.mark.parametrize("hidden,nh", [(64, 1), (64, 4), (128, 1), (128, 2)])
def test_shapes(rn, ctx, oracle_lib, L, K, hidden, nh):
    print("shape", L, K, hidden, nh, flush=True)
    m = models.make_model(["H", "O"], L=L, K=K, r_c=4.0, n_hidden=nh, hidden=hidden, T_max=3, seed=32, bias_std=1.0,
                          ang_scale=0.25, energy_scale=1.2, form="radial" if L == 0 else "reann")
    s = systems.water_box(seed=32)
    check(rn.energy_forces(ctx, rn.Model(m), s, T=3, precision="fp64", skin=0.5, decomp=(2, 1, 1)),
          oracle_lib.evaluate(m, s, T=3, skin=0.5))


@pytest.mark.parametrize("exchange", ["messages", "node_features"])
def test_many_elements(rn, ctx, oracle_lib, exchange):
    """Five elements: more segments than one launch takes (kFuseMaxSeg = 4)."""
    m = models.make_model(["H", "O", "Cu", "C", "N"], L=1, K=4, r_c=4.0, n_hidden=2, hidden=64, T_max=3, seed=33,
                          bias_std=1.0, ang_scale=0.25)
    s = systems.water_box(seed=33)
    s = dict(s, species=(np.arange(len(s["species"])) * 7 % 5).astype(np.int32))
    check(rn.energy_forces(ctx, rn.Model(m), s, T=3, precision="fp64", skin=0.5, decomp=(2, 1, 1), exchange=exchange),
          oracle_lib.evaluate(m, s, T=3, skin=0.5))


def test_noalloc_before_and_after_a_plan(rn, oracle_lib):
    m = models.water_model(T_max=2, seed=34)
    s = systems.water_box(seed=34)
    ref = oracle_lib.evaluate(m, s, T=2, skin=0.5)
    ctx, model = rn.Context(0), rn.Model(m)
    rn.energy_forces(ctx, model, s, T=2, precision="fp32", skin=0.5)   # the weights, not the packed operands
    check(rn.energy_forces(ctx, model, s, T=2, precision="fp64", skin=0.5, noalloc=True), ref)
    check(rn.energy_forces(ctx, model, s, T=2, precision="fp64", skin=0.5), ref)
    check(rn.energy_forces(ctx, model, s, T=2, precision="fp64", skin=0.5, noalloc=True), ref)
