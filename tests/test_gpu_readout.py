"""Field reads: chunks in pinned slots, several threads, and only the selected planes.  The full read is
compared with the oracle elsewhere; here any selection must be those planes' bits, in any split."""
import ctypes

import numpy as np
import pytest

from paper_2209_14889_amd import lb
from paper_2209_14889_amd import workload as wl

pytestmark = pytest.mark.gpu

SELECTIONS = [["rho"], ["sxy"], ["Px", "Py"], ["vx", "vy"], ["fpx"], ["rho", "vy", "sxx", "fpy"], ["Py", "rho"]]


# one slot less than full, slots ended by ragged planes, one site short of two slots' worth
@pytest.mark.parametrize("nx,ny", [(64, 64), (517, 413), (229, 229), (1024, 103)])
@pytest.mark.parametrize("precision", [0, 1])
def test_selected_planes_are_the_full_reads(nx, ny, precision):
    w = wl.small_case(3, nx, ny, n_bodies=1, radius=8.0)
    g = lb.Sim(w, lb.make_options(precision=precision))
    g.step(5)
    N = nx * ny
    every = np.empty(10 * N)
    dp = ctypes.POINTER(ctypes.c_double)
    lb.check(lb.lib().lb_read_fields(g.h, 0, 0x3FF, every.ctypes.data_as(dp), every.size))
    ref = {f: every[i * N:(i + 1) * N].reshape(ny, nx) for i, f in enumerate(lb.FIELDS)}
    assert all(np.isfinite(v).all() for v in ref.values()) and abs(ref["rho"].mean() - 1.0) < 1e-3
    for names in [list(lb.FIELDS), *SELECTIONS]:
        got = g.fields(names=names)
        assert list(got) == [f for f in lb.FIELDS if f in names]
        for f, v in got.items():
            assert v.shape == (ny, nx) and v.flags.owndata
            np.testing.assert_array_equal(v, ref[f], err_msg=f)
    g.close()


def test_read_planes_rejects_what_is_no_plane():
    g = lb.Sim(wl.small_case(3, 48, 40))
    dp = ctypes.POINTER(ctypes.c_double)
    a = np.empty(48 * 40)
    read = lb.lib().lb_read_planes
    one = (dp * 2)(a.ctypes.data_as(dp), dp())
    assert read(g.h, 0, lb.F_NODES, one) == lb.LB_EINVAL
    assert read(g.h, 0, 0x3, one) == lb.LB_EINVAL       # the second plane is NULL
    assert read(g.h, 1, 0x1, one) == lb.LB_ERANGE
    assert read(g.h, 0, 0x1, None) == lb.LB_EINVAL
    assert read(None, 0, 0x1, one) == lb.LB_EINVAL
    assert read(g.h, 0, 0x1, one) == lb.LB_OK and read(g.h, 0, 0x0, one) == lb.LB_OK
    g.close()
