"""The binding's packed structures against ctypes structures filled field by field."""
import ctypes as C

import numpy as np
import pytest

from paper_2604_07980_amd import ocsr, synth


@pytest.mark.parametrize("n", [1, 16])
@pytest.mark.parametrize("width", [1, 4096, 2**31 - 1, 2**32 + 9, -(2**40) - 3])
def test_frame_array(n, width):
    rows = [(0x7F0000000000 + k, 3 * k, width, k + 1, width, 40 * k, 40, 0) for k in range(n)]
    want = (ocsr.Frame * n)()
    for k, r in enumerate(rows):
        want[k] = ocsr.Frame(*r)
    assert bytes(ocsr._frame_array(rows)) == bytes(want)


def test_frame_array_refuses_fractions():
    with pytest.raises(TypeError):
        ocsr._frame_array([(0, 0, 1.5, 2, 3, 0, 4, 0)])


@pytest.mark.parametrize("form", ["lists", "fortran", "float32"])
def test_point_params(form):
    g = synth.point_geometry(1921, 1203, synth.base_params())
    conv = {"lists": lambda a: a, "fortran": lambda a: np.asfortranarray(np.asarray(a, np.float64)),
            "float32": lambda a: np.asarray(a, np.float32)}[form]
    Q = conv((np.arange(16.0).reshape(4, 4) / 4).tolist())
    R, t = conv(g["R"]), conv(g["t"])
    pp = ocsr.point_params(dict(g, Q=Q, R=R, t=t))
    want = ocsr.PointParams()
    want.width, want.height = 1921, 1203
    for name, v in (("Q", Q), ("R", R), ("t", t)):
        getattr(want, name)[:] = [float(x) for x in np.asarray(v).reshape(-1)]
    for name in ("focal_px", "baseline_m", "var_d", "var_x", "var_y"):
        setattr(want, name, g[name])
    assert C.sizeof(pp) == C.sizeof(want) and bytes(pp) == bytes(want)
    with pytest.raises(ValueError):
        ocsr.point_params(dict(g, t=[1.0, 2.0]))
