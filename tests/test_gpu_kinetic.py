"""The kick and the kinetic energy of a velocity-Verlet step at the sizes where their kernel changes: in one
block of 1,024 threads up to 2,048 atoms (one, several and unequal components a thread), in two
launches above.  The kinetic energy the server reports is half the sum of m v^2 of the velocities it
returns; both are FP64 sums of at most 3 n terms, so they agree to 1e-12."""
import time

import numpy as np
import pytest

from synth import models, systems

pytestmark = pytest.mark.gpu

ELEMENTS = ["H", "O", "Cu"]
MASSES = [systems.MASS_AMU[e] for e in ELEMENTS]
KACCEL = 9.648533212e-3     # (eV/A) / amu in A/fs^2


@pytest.fixture(scope="module")
def rn():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2505_06711_amd as rn
    return rn


@pytest.mark.parametrize("n", [5, 342, 683, 2048, 2049])
def test_kinetic_energy(rn, n):
    print("atoms", n, flush=True)
    s = systems.remap_species(systems.water_box(grid=(9, 9, 9), spacing=systems.WATER_BOX_L / 4, seed=82), ELEMENTS)
    s = dict(s, pos=s["pos"][:n], species=s["species"][:n], pbc=np.zeros(3, np.int32))   # an open cluster
    m = models.serving_model(T_max=2, seed=3)
    srv = rn.Server(rn.Model(m), T=2, precision="fp32", skin=0.5, use_graph=True)
    srv.set_masses(MASSES)
    v0 = systems.maxwell_boltzmann(s["species"], ELEMENTS, 300.0, seed=10)
    sid = srv.add_system(s, v0)
    ticket, t0, r = srv.submit_vv(sid, 0.5), time.time(), None
    while r is None:
        assert time.time() - t0 < 60.0
        r = srv.poll(ticket, sid, velocities=True)
        time.sleep(0.0002)
    srv.close()
    mass = np.array([MASSES[k] for k in s["species"]])[:, None]
    K = 0.5 * (mass * r["velocities"] ** 2).sum() / KACCEL
    assert abs(r["kinetic"] - K) <= 1e-12 * K
    assert np.abs(r["velocities"] - v0).max() > 0.0
