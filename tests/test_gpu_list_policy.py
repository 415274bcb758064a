"""When a forward asks about its list before it runs: after an unrelated frame, not after a
trajectory's rebuild.  Told from the launches and phase times of the plan; energies against the oracle
at the FP64 path's bound (1e-12 of the summed atomic energies; a shifted crystal keeps its energy)."""
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


@pytest.mark.parametrize("T", [1, 2])
def test_asks_first_after_an_unrelated_frame_only(rn, oracle_lib, T):
    import torch
    skin = 1.0
    s, m = systems.water_box(seed=64), models.water_model(T_max=2, seed=64)
    ref = oracle_lib.evaluate(m, s, T=T)
    tol = 1e-12 * max(abs(ref["energy"]), np.abs(ref["atom_energy"]).sum())
    plan = rn.Plan(rn.Context(0), rn.Model(m), s, T=T, precision="fp64", skin=skin)
    plan.set_timing(True)
    pos = torch.tensor(s["pos"], device="cuda")
    E = torch.empty((), dtype=torch.float64, device="cuda")

    def forward(shift):
        """(forwards run, lists built, whether the forward waited for the list check first)"""
        plan.forward(pos + shift * skin, E)
        t = plan.timing()
        assert abs(float(E) - ref["energy"]) <= tol
        runs, builds = t["launches"]["edge_fwd"] // T, t["launches"]["nlist"]
        return runs, builds, runs == 1 and t["ms"]["nlist"] > 0.0

    x = torch.tensor([1.0, 0.0, 0.0], dtype=torch.float64, device="cuda")
    assert forward(0 * x) == (1, 1, True)        # the first list
    assert forward(0.1 * x) == (1, 0, False)
    assert forward(0.55 * x) == (2, 1, False)    # a step past the bound
    assert forward(0.6 * x) == (1, 0, False)     # the trajectory goes on
    assert forward(1.15 * x) == (2, 1, False)
    assert forward(1.2 * x) == (1, 0, False)
    assert forward(4.0 * x) == (2, 1, False)     # another frame
    assert forward(7.0 * x) == (1, 1, True)      # and another
    assert forward(7.1 * x) == (1, 0, True)
    assert forward(7.2 * x) == (1, 0, False)
