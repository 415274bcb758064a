"""The edge records of the FP32 adjoint: written through the caches or past them (record buffers above
and below 300 MiB), and across the boundary of a row's local and ghost neighbours, against the FP64 path
(itself held to the oracle) within the FP32 path's bounds for forces: 1e-5 of their RMS and of max|F|."""
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


# list entries x 64 bytes with skin 1 (119 or so a row): 42 MB, 304 MB, 477 MB
@pytest.mark.parametrize("dims,decomp", [((11, 11, 11), (2, 1, 2)), ((21, 22, 22), (1, 1, 1)), ((25, 25, 25), (1, 2, 1))])
def test_records_fp32_against_fp64(rn, dims, decomp):
    print("records", dims, decomp, flush=True)
    m = models.cu_model(T_max=3, seed=41)
    s = systems.fcc_crystal(dims, seed=41)
    ctx, model = rn.Context(0), rn.Model(m)
    _, F, _ = rn.energy_forces(ctx, model, s, T=3, precision="fp32", skin=1.0, decomp=decomp)
    _, F64, _ = rn.energy_forces(ctx, model, s, T=3, precision="fp64", skin=1.0, decomp=decomp)
    assert np.sqrt(((F - F64) ** 2).mean()) <= 1e-5 * np.sqrt((F64 ** 2).mean())
    assert np.abs(F - F64).max() <= 1e-5 * np.abs(F64).max()
