"""GPU parity of the reciprocal part at the largest (x, y) planes that its own transforms take and
just above them (96 x 96 goes to the FFT library), on row blocks halved to fit in LDS, and for
batches on grids with odd sizes and planes at the limit.

FP64: 1e-12 relative RMS on forces, 1e-12 relative on the energy and 1e-11 on the virial, as for
the other grids."""

import numpy as np
import pytest

import nbtest_util as U
from oracle import pme as PO
from paper_0902_0827_amd import nbhip as H
from paper_0902_0827_amd import systems as S

torch = pytest.importorskip("torch")
pytestmark = [pytest.mark.gpu,
              pytest.mark.skipif(not torch.cuda.is_available(), reason="needs a GPU")]


@pytest.mark.parametrize("systems", [1, 3])
@pytest.mark.parametrize("grid", [(90, 90, 20), (81, 112, 16), (90, 96, 12), (96, 96, 12), (16, 80, 1024), (27, 25, 21)])
def test_reciprocal_at_the_limits(grid, systems):
    boxes = [S.solvated_chain(19.0 + 0.4 * k, 25, 700 + 31 * k, seed=41 + k, cutoff=9.0, beta=0.34)
             for k in range(systems)]
    print(f"[case] pme-limits grid={grid} systems={systems}", flush=True)
    b = H.device_batch(boxes, dtype=torch.float64)
    p = H.make_params(9.0, 0.34, H.NB_FP64)
    ws = H.alloc_pme_workspace(b, grid)
    force = torch.full((b.n_atoms, 3), 7.0, dtype=torch.float64, device="cuda")
    energy = torch.full((systems,), 7.0, dtype=torch.float64, device="cuda")
    vir = torch.full((systems, 3, 3), 7.0, dtype=torch.float64, device="cuda")
    H.pme_reciprocal(b, p, grid, ws, force, energy, vir)
    torch.cuda.synchronize()
    force, energy, vir = force.cpu().numpy(), energy.cpu().numpy(), vir.cpu().numpy()
    at = 0
    for k, s in enumerate(boxes):
        ref = PO.spme_reciprocal(s.pos, s.charge, s.box, s.beta, grid)
        assert U.rel_rms(force[at:at + s.n], ref["force"]) <= 1e-12, k
        assert abs(energy[k] - ref["energy"]) <= 1e-12 * abs(ref["energy"]), k
        assert np.linalg.norm(vir[k] - ref["virial"]) <= 1e-11 * np.linalg.norm(ref["virial"]), k
        at += s.n
