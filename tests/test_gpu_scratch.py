"""The allocation-free evaluation near the size of its static scratch: open clusters that fit with
every buffer at the size it needs (a few more atoms do not), at sixteen layers, where a row kept per
layer and block costs the most.  Results against the allocating call, which shares the kernels: bit
for bit, whatever was evaluated before."""
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


@pytest.mark.parametrize("K,r_c,hidden,nh,precision,n", [(12, 6.0, 128, 4, "fp32", 1390), (12, 6.0, 128, 4, "bf16", 1390),
                                                         (8, 5.0, 64, 2, "fp32", 3710), (4, 5.0, 32, 1, "fp64", 3381)])
def test_cluster_that_just_fits(rn, K, r_c, hidden, nh, precision, n):
    print("scratch", K, hidden, nh, precision, n, flush=True)
    m = models.make_model(["Cu"], L=2, K=K, r_c=r_c, n_hidden=nh, hidden=hidden, T_max=16, seed=1, ang_scale=1 / r_c)
    s = systems.fcc_crystal((24, 24, 24), seed=1)
    order = np.argsort(((s["pos"] - s["pos"].mean(0)) ** 2).sum(1), kind="stable")[:n]
    s = dict(s, pos=s["pos"][order], species=s["species"][order], pbc=np.zeros(3, np.int32))
    ctx, model = rn.Context(0), rn.Model(m)
    want = rn.energy_forces(ctx, model, s, T=16, precision=precision, skin=0.5)
    got = rn.energy_forces(ctx, model, s, T=16, precision=precision, skin=0.5, noalloc=True)
    assert got[0] == want[0]
    np.testing.assert_array_equal(got[1], want[1])
    np.testing.assert_array_equal(got[2], want[2])


@pytest.mark.parametrize("form", ["reann", "radial"])
def test_fp64_bits_do_not_depend_on_what_ran_before(rn, form):
    """The FP64 evaluation that may not allocate, with only an FP32 call before it and after an FP64 one."""
    m = (models.water_model if form == "reann" else models.water_model_radial)(T_max=3, seed=2)
    s = systems.water_box(seed=2)
    ctx, model = rn.Context(0), rn.Model(m)
    rn.energy_forces(ctx, model, s, T=3, precision="fp32", skin=0.5)   # the model's device copies
    first = rn.energy_forces(ctx, model, s, T=3, precision="fp64", skin=0.5, noalloc=True)
    want = rn.energy_forces(ctx, model, s, T=3, precision="fp64", skin=0.5)
    again = rn.energy_forces(ctx, model, s, T=3, precision="fp64", skin=0.5, noalloc=True)
    for got in (first, again):
        assert got[0] == want[0]
        np.testing.assert_array_equal(got[1], want[1])
        np.testing.assert_array_equal(got[2], want[2])
