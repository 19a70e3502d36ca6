"""FP64 half shell with atoms whose raw coordinates lie whole boxes away from the others (any
real coordinate is accepted): such an atom's rounding stays with its own pairs.  Every other
pair is evaluated from the same two coordinates as without the shift, and the accumulators are
fixed point, so the forces on atoms that no shifted atom reaches are the same bits.  (The
scattered atoms are, some of them, the first of their cluster, beside atoms out of their
reach.)"""

import numpy as np
import pytest

import nbtest_util as U
from paper_0902_0827_amd import nbhip as H

torch = pytest.importorskip("torch")
pytestmark = [pytest.mark.gpu,
              pytest.mark.skipif(not torch.cuda.is_available(), reason="needs a GPU")]


@pytest.mark.parametrize("kernel", ["half8", "half4_dynamic"])
@pytest.mark.parametrize("boxes", [1, -1, 10, 1000, 10_000_000])
def test_a_shifted_atom_changes_only_its_own_pairs(boxes, kernel):
    s = U.lattice_system((36.0, 38.0, 44.0), 2.6, seed=29)
    box = np.asarray(s.box)
    print(f"[case] far-atoms boxes={boxes} kernel={kernel} n={s.n}", flush=True)
    base = U.gpu_eval(s, H.NB_FP64, kernel=kernel, energy_call=True)
    moved = np.random.default_rng(5).choice(s.n, 14, replace=False)
    d = s.pos[:, None, :] - s.pos[None, moved, :]
    d -= box * np.rint(d / box)
    clear = np.sqrt((d * d).sum(-1)).min(1) > s.cutoff + 0.01
    assert clear.sum() > 1000
    s.pos = s.pos.copy()
    s.pos[moved] += boxes * box
    out = U.gpu_eval(s, H.NB_FP64, kernel=kernel, energy_call=True)
    assert out["status"] == 0
    assert np.array_equal(out["force"][clear], base["force"][clear])
    assert np.array_equal(out["atom_energy"][clear], base["atom_energy"][clear])
