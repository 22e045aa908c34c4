"""The C structures filled from a caller's objects (no GPU)."""
import ctypes as C
import warnings

import numpy as np
import pytest

from paper_2608_27735_amd import _lib
from paper_2608_27735_amd.camera import look_at


def _camera_element_by_element(cam):
    """camera_struct's arrays, one float() an element."""
    R = [float(x) for row in cam.R for x in row] if hasattr(cam.R[0], "__len__") else list(cam.R)
    f = lambda a, n: [C.c_float(float(a[i])).value for i in range(n)]
    return f(R, 9), f(cam.t, 3), f(cam.campos, 3)


_NINE = [0.1 * k - 0.37 for k in range(9)]


@pytest.mark.parametrize("field", ["R", "t", "campos"])
@pytest.mark.parametrize("form", [
    "list", "tuple", "flat", "nested", "float16", "float64", "int32", "bool", "str", "object", "complex",
    "row", "column", "deep", "longer", "shorter", "strided", "reversed", "masked", "tensor"])
def test_camera_arrays_as_element_by_element(field, form):
    """The arrays of a camera in every form that a caller may hold them in: accepted
    with the same numbers, or refused, as element by element."""
    import torch
    n = 9 if field == "R" else 3
    v = _NINE[:n]
    a = np.array(v, np.float32)
    x = dict(list=v, tuple=tuple(v), flat=a, nested=a.reshape(-1, 3), float16=a.astype(np.float16),
             float64=np.array(v), int32=np.arange(n, dtype=np.int32), bool=a > 0,
             str=np.array([str(k) for k in v]), object=np.array(v, object), complex=a.astype(np.complex64),
             row=a.reshape(1, n), column=a.reshape(n, 1), deep=a.reshape(1, -1, 3),
             longer=np.concatenate([a, a]), shorter=a[:-1], strided=np.repeat(a, 2)[::2],
             reversed=a[::-1], masked=np.ma.array(a, mask=False), tensor=torch.tensor(v))[form]
    cam = look_at((0.0, -3.0, 0.5), (0, 0, 0), 32, 16)
    setattr(cam, field, x)

    def outcome(f):
        with warnings.catch_warnings():
            warnings.simplefilter("ignore")
            try:
                return f(cam)
            except (TypeError, ValueError, IndexError) as e:
                return "refused"

    got = outcome(lambda c: (lambda s: (list(s.R), list(s.t), list(s.campos)))(_lib.camera_struct(c)))
    assert got == outcome(_camera_element_by_element)
