"""Workspace sizes: a workspace sized for a batch serves every smaller one.  The size never falls
as atoms are added or as a box shrinks around the same atoms, through every change of the rules
that depend on the size (parts of small systems' gradients, the fused build), and so does that of
the MD workspace, which holds a nonbonded one; the gradients' room depends on the batch alone."""

import ctypes

import numpy as np
import pytest

from paper_0902_0827_amd import nbhip as H
from test_abi_cpu import fake_system, ws_bytes

SIZES = sorted({round(x) for x in np.geomspace(100, 60_000, 400)})


def _md_bytes(s, p):
    md = H.make_md_params(0.002)
    n = ctypes.c_size_t()
    assert H.load_library().nb_md_workspace_bytes(ctypes.byref(s), ctypes.byref(p), ctypes.byref(md),
                                                  ctypes.byref(n)) == H.NB_OK
    return n.value


def _side(n):
    return max((n / 0.1) ** (1 / 3), 18.1)


@pytest.mark.parametrize("precision", [H.NB_MIXED, H.NB_FP64])
@pytest.mark.parametrize("types", [1, 64])
def test_size_never_falls_as_atoms_are_added(precision, types):
    p = H.make_params(9.0, 0.34, precision)
    last = last_md = 0
    for n in SIZES:
        s = fake_system((n,), L=_side(n))
        s.n_types = types
        code, size = ws_bytes(s, p)
        assert code == H.NB_OK and size >= last, n
        last = size
        s.pos_is_f64 = 1
        md = _md_bytes(s, p)
        assert md >= last_md, n
        last_md = md


@pytest.mark.parametrize("precision", [H.NB_MIXED, H.NB_FP64])
@pytest.mark.parametrize("n", [648, 7_581, 15_500, 23_600, 30_500, 48_000])
def test_size_never_grows_as_the_box_shrinks(precision, n):
    p = H.make_params(9.0, 0.34, precision)
    last = None
    for f in np.linspace(1.5, 0.7, 200):
        code, size = ws_bytes(fake_system((n,), L=max(_side(n) * f, 18.1)), p)
        assert code == H.NB_OK and (last is None or size <= last), f
        last = size


@pytest.mark.parametrize("n", [648, 7_581, 23_600, 100_000])
def test_gradient_room_depends_on_the_batch_alone(n):
    """The options that turn the parts off do not change the size, and precision, kernel and
    cluster size change it by what their own arrays take."""
    s = fake_system((n,), L=_side(n))
    for prec in (H.NB_MIXED, H.NB_FP64):
        size = ws_bytes(s, H.make_params(9.0, 0.34, prec))[1]
        assert ws_bytes(s, H.make_params(9.0, 0.34, prec, split=1))[1] == size
        assert ws_bytes(s, H.make_params(9.0, 0.34, prec, schedule=H.NB_SCHED_DYNAMIC))[1] == size
    limb = (32 * n + 255) // 256 * 256
    two = (64 * n + 255) // 256 * 256
    mixed = ws_bytes(s, H.make_params(9.0, 0.34, H.NB_MIXED))[1]
    assert ws_bytes(s, H.make_params(9.0, 0.34, H.NB_FP64))[1] - mixed == two - limb
