"""Row counts where the launches of the evaluation change shape, in FP32 and BF16: the fused NN kernels'
16- and 32-row tiles (edges of a tile, a single row, both sides of the rule between them) and the
lanes that share a row in the edge adjoint (64, 32 or 16).

FP32 within the FP32 path's bounds (1e-6 energy, 1e-5 of the force RMS and of max|F|) against the
FP64 oracle; BF16 as a layout check (1% energy and 2% force RMSE per hidden layer and MP layer: the
rounding is 2^-9 per operand, a misplaced operand or tile gives errors of order one)."""
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


def crystal(n, seed):
    """The first n atoms of a jittered crystal, as an open cluster."""
    s = systems.fcc_crystal((24, 24, 24), seed=seed) if n > 9000 else systems.fcc_crystal((14, 14, 14), seed=seed)
    order = np.argsort((s["pos"] ** 2).sum(1), kind="stable")[:n]
    return dict(s, pos=s["pos"][order], species=s["species"][order], pbc=np.zeros(3, np.int32))


# rows: one; tile edges of 16 and 32; forward rule at 256 tiles of 16 rows (H = 128) and 512 (H = 64);
# adjoint rule at 1,024 (H = 128) and 2,048 (H = 64); edge adjoint at 1,536 and 4,096 rows
@pytest.mark.parametrize("hidden,n", [(128, 1), (128, 15), (128, 17), (128, 33), (128, 1536), (128, 1537), (128, 4096), (128, 4097), (128, 16384),
                                      (128, 16385), (64, 31), (64, 8192), (64, 8193), (64, 32768), (64, 32769)])
@pytest.mark.parametrize("prec", ["fp32", "bf16"])
def test_row_counts(rn, ctx, oracle_lib, hidden, n, prec):
    print("rows", n, hidden, prec, flush=True)
    m = models.make_model(["Cu"], L=1, K=4, r_c=3.2, n_hidden=2, hidden=hidden, T_max=2, seed=21, bias_std=1.0,
                          ang_scale=1.0 / 3.2)
    s = crystal(n, 21)
    E, F, W = rn.energy_forces(ctx, rn.Model(m), s, T=2, precision=prec, skin=0.3)
    ref = oracle_lib.evaluate(m, s, T=2)
    den = max(abs(ref["energy"]), np.abs(ref["atom_energy"]).sum())
    rms = np.sqrt((ref["forces"] ** 2).mean())
    rf = np.sqrt(((F - ref["forces"]) ** 2).mean())
    tol_e, tol_f = (1e-6, 1e-5) if prec == "fp32" else (0.04, 0.08)
    assert abs(E - ref["energy"]) <= tol_e * den
    assert rf <= tol_f * rms if rms > 0 else np.abs(F).max() == 0.0
    if prec == "fp32":
        assert np.abs(F - ref["forces"]).max() <= 1e-5 * np.abs(ref["forces"]).max()
