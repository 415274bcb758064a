"""The edge records of the FP32 adjoint on both sides of the size from which they are written past the
caches (300 MiB of list slots, 64 bytes each at K = 12, the rows of ghosts included), for launches of 16
lanes a row, against the FP64 path (itself held to the oracle) within the FP32 path's bounds for forces:
1e-5 of their RMS and of max|F|."""
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


@pytest.mark.parametrize("dims,streamed", [((20, 20, 20), False), ((20, 21, 21), True)])
def test_records_below_and_above_the_limit(rn, dims, streamed):
    m = models.cu_model(T_max=3, seed=42)
    s = systems.fcc_crystal(dims, seed=42)
    slots = rn.build_neighbors(rn.Context(0), s, m.r_c, 1.0).info()["n_pairs"]
    print("records", dims, slots * 64 / 2 ** 20, "MiB", flush=True)
    assert (slots * 64 > 300 * 2 ** 20) == streamed
    ctx, model = rn.Context(0), rn.Model(m)
    _, F, _ = rn.energy_forces(ctx, model, s, T=3, precision="fp32", skin=1.0)
    _, F64, _ = rn.energy_forces(ctx, model, s, T=3, precision="fp64", skin=1.0)
    assert np.sqrt(((F - F64) ** 2).mean()) <= 1e-5 * np.sqrt((F64 ** 2).mean())
    assert np.abs(F - F64).max() <= 1e-5 * np.abs(F64).max()
