"""Short work items as tiles (all rows of a tile at once) against items that march down their rows: the
same arithmetic at every site, so the same bits."""
import ctypes

import numpy as np
import pytest

from paper_2209_14889_amd import lb
from paper_2209_14889_amd import workload as wl

pytestmark = pytest.mark.gpu

FE = dict(alpha=-1.8e-3, beta=2e-3, kappa=2e-6)


def run(spec, opt, steps=9):
    g = lb.Sim([spec], opt)
    g.step(steps)
    out = g.fields(), g.nodes(), g.launch_shape()
    g.close()
    return out


def same(a, b, what):
    for k in lb.FIELDS:
        assert np.array_equal(a[0][k], b[0][k]), (what, k)
    for x, y in zip(a[1], b[1]):
        assert np.array_equal(x, y), (what, "nodes")


# lattices at and beside whole numbers of tiles, narrower than a tile with its halo, and ragged; 39 rows of
# any work-group size are more than a tile takes, so they march
@pytest.mark.parametrize("nx,ny", [(32, 32), (33, 31), (8, 9), (130, 47)])
@pytest.mark.parametrize("walls,precision,polar", [(0, 0, 1), (0, 1, 1), (1, 0, 0), (2, 1, 1), (2, 0, 1)])
def test_tiles_agree_with_marching_items_bitwise(nx, ny, walls, precision, polar):
    bodies = 1 if min(nx, ny) > 30 else 0
    w = wl.small_case(81, nx, ny, n_bodies=bodies, radius=4.5, pull=2e-4, walls=walls, gx=1e-6, **(FE if walls else {}))
    s = w.sims[0]
    if not polar:
        s.P0 = np.zeros_like(s.P0)
    ref = run(s, lb.make_options(precision=precision, fused_threads=64, seg_rows=39))
    for T, rows in ((64, 4), (64, 7), (64, 8), (128, 5), (128, 8), (256, 4), (256, 9), (256, 16)):
        print(f"case tiles {nx}x{ny} walls {walls} precision {precision} threads {T} rows {rows}", flush=True)
        same(run(s, lb.make_options(precision=precision, fused_threads=T, seg_rows=rows)), ref, (T, rows))
    same(run(s, lb.make_options(precision=precision)), ref, "default")


def test_arena_without_room_for_tiles():
    """An arena of the size that the marching items alone need is accepted, and gives the same bits."""
    s = wl.small_case(82, 96, 80, n_bodies=1, radius=6.0).sims[0]
    opt = lb.make_options()
    g = lb.Sim([s], opt)
    a = g.launch_shape()
    g.step(20)
    f = g.fields()
    lb.check(lb.lib().lb_destroy(g.h))
    m = lb._Marshal([s])
    table = 32 * max(-(-96 // (T // max(8, r))) * -(-80 // r) for T in (64, 128, 256)
                     for r in range(4, (16 if T == 256 else 8) + 1))
    h = ctypes.c_void_p()
    lb.check(lb.lib().lb_create(m.params, 1, ctypes.byref(opt), ctypes.c_void_p(g.arena.data_ptr()),
                                ctypes.c_size_t(g.arena.numel() - table), ctypes.c_void_p(g.stream.cuda_stream),
                                ctypes.byref(h)))
    g.h = h
    b = g.launch_shape()
    assert a["seg_rows"] == 4 and a["n_items"] != b["n_items"]
    g.step(20)
    f2 = g.fields()
    for k in lb.FIELDS:
        assert np.array_equal(f[k], f2[k]), k
    g.close()


@pytest.mark.parametrize("walls", [0, 1, 2])
@pytest.mark.parametrize("precision", [0, 1])
def test_marching_items_of_three_rows(walls, precision):
    """The shortest marching items that the launch model takes (the last ones of two and three rows of 91)
    against long ones; a grid of one work-group per item keeps both from being tiles."""
    w = wl.small_case(21, 150, 91, n_bodies=1, radius=8.0, walls=walls)
    want = None
    for threads, seg in ((256, 91), (256, 3), (128, 3)):
        g = lb.Sim(w, lb.make_options(precision=precision, fused_threads=threads, seg_rows=seg, grid=1 << 20))
        g.step(9)
        f = g.fields()
        want = f if want is None else want
        for k in lb.FIELDS:
            np.testing.assert_array_equal(f[k], want[k], err_msg=f"{threads} {seg} {k}")
        g.close()


@pytest.mark.parametrize("nx,threads", [(24, 0), (56, 0), (57, 64), (112, 64), (113, 128), (240, 256)])
def test_the_model_fits_the_item_table(nx, threads):
    """Widths whose strips fill the item table at four rows an item: the chosen shape must fit and step."""
    w = wl.small_case(21, nx, 90, n_bodies=0)
    one = lb.Sim(w)
    g = lb.Sim(w, lb.make_options(fused_threads=threads, grid=1 << 20))
    one.step(5)
    g.step(5)
    a, b = one.fields(), g.fields()
    for k in lb.FIELDS:
        np.testing.assert_array_equal(a[k], b[k], err_msg=k)
    one.close()
    g.close()


@pytest.mark.parametrize("polar", [0, 1])
@pytest.mark.parametrize("threads,nx", [(64, 64), (128, 100), (256, 300)])
def test_a_lattice_without_bodies_beside_one_with(threads, nx, polar):
    """A launch without bodies takes a variant of the marching kernel of its own; beside a lattice with a
    body, the same lattice takes the other one.  The same bits."""
    alone = wl.small_case(83, nx, 45).sims[0]
    alone.bodies = []
    other = wl.small_case(84, 70, 50, radius=6.0, pull=2e-4).sims[0]
    if not polar:
        for s in (alone, other):
            s.P0 = np.zeros_like(s.P0)
    opt = lb.make_options(fused_threads=threads, seg_rows=23)
    a, b = lb.Sim([alone], opt), lb.Sim([alone, other], opt)
    a.step(9)
    b.step(9)
    x, y = a.fields(), b.fields(0)
    for k in lb.FIELDS:
        np.testing.assert_array_equal(x[k], y[k], err_msg=k)
    a.close()
    b.close()


@pytest.mark.parametrize("nx,ny,k,precision,polar,tiles,rows", [
    (64, 64, 128, 0, 1, 0, 4), (100, 100, 40, 0, 0, 0, 4), (128, 128, 30, 0, 1, 0, 4), (640, 640, 1, 0, 1, 0, 4),
    (250, 250, 8, 1, 1, 0, 4), (128, 128, 30, 1, 0, 0, 4), (700, 700, 1, 0, 1, 0, 3), (250, 250, 6, 0, 1, 1, 8)])
def test_launch_model_without_bodies(nx, ny, k, precision, polar, tiles, rows):
    """Lattices without bodies on 256 compute units: tiles up to six a unit, and three marching rows only
    where they do not put a further wave on a SIMD.  The lattices beyond were slower than in four rows."""
    s = wl.small_case(85, nx, ny, n_bodies=0, random_dirs=False).sims[0]
    if not polar:
        s.P0 = np.zeros_like(s.P0)
    g = lb.Sim([s] * k, lb.make_options(precision=precision))
    if g._torch.cuda.get_device_properties(0).multi_processor_count != 256:
        pytest.skip("the sizes are those of 256 compute units")
    shape = g.launch_shape()
    across = -(-nx // 32) if tiles else 1 if nx <= 256 else -(-nx // 248)
    assert shape["seg_rows"] == rows and shape["n_items"] == k * across * -(-ny // rows), shape
    g.close()
