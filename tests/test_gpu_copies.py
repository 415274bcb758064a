"""Message exchange in cells shorter than the cutoff: systems below and above the number of ghost
copies an atom from which a gather launch writes the ghosts' messages, instead of the message NN's
launch, against the oracle at the FP64 path's bounds (1e-12 of the summed atomic energies, 1e-10 of
the largest force and virial component, or of 1 where the lattice cancels them)."""
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


def one(edge):
    return dict(pos=np.array([[0.3, 0.4, 0.5]]), species=np.zeros(1, np.int32), cell=np.eye(3) * edge,
                pbc=np.ones(3, np.int32), elements=["Cu"])


@pytest.mark.parametrize("form", ["reann", "radial"])
@pytest.mark.parametrize("case", ["1_atom", "1x1x1", "2x1x1", "2x2x2", "3x3x3", "1x1x9_split"])
def test_short_cells(rn, oracle_lib, form, case):
    r_c, skin = 4.0, 0.5
    m = models.make_model(["Cu"], L=0 if form == "radial" else 2, K=8, r_c=r_c, n_hidden=2, hidden=64, T_max=3, seed=5,
                          bias_std=1.0, ang_scale=1 / r_c, form=form)
    s = one(2.6) if case == "1_atom" else systems.fcc_crystal(tuple(map(int, case.split("_")[0].split("x"))), seed=5)
    decomp = (1, 1, 2) if case.endswith("split") else (1, 1, 1)
    ghosts = rn.build_neighbors(rn.Context(0), s, r_c, skin, decomp).info()["n_ghosts"]
    print("copies", case, form, ghosts / len(s["pos"]), flush=True)
    assert (ghosts > 16 * len(s["pos"])) == (case not in ("2x2x2", "3x3x3"))   # both sides of the rule
    ctx, model = rn.Context(0), rn.Model(m)
    E, F, W = rn.energy_forces(ctx, model, s, T=3, precision="fp64", skin=skin, decomp=decomp)
    ref = oracle_lib.evaluate(m, s, T=3, skin=skin)
    assert abs(E - ref["energy"]) <= 1e-12 * max(abs(ref["energy"]), np.abs(ref["atom_energy"]).sum())
    assert np.abs(F - ref["forces"]).max() <= 1e-10 * max(np.abs(ref["forces"]).max(), 1.0)
    assert np.abs(W - ref["virial"]).max() <= 1e-10 * max(np.abs(ref["virial"]).max(), 1.0)
