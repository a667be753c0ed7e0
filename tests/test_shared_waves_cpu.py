"""The query of a local search's shared layout: arguments that are refused, and the
empty call, before any device work."""
import ctypes as C

from paper_2410_10447_amd import dock


def test_shared_waves_arguments():
    L = dock.lib()
    n = C.c_int32(-1)
    o = dock.LsOpts(iterations=10, rho=0.8, eps=1e-2, variant=0, threads_per_ind=0, flags=1)
    items = (dock.LsItem * 1)()
    assert L.dock_ls_shared_waves(items, 0, C.byref(o), None, None) == dock.DOCK_EINVAL
    assert L.dock_ls_shared_waves(None, 1, C.byref(o), None, C.byref(n)) == dock.DOCK_EINVAL
    assert L.dock_ls_shared_waves(items, 1, C.byref(o), None, C.byref(n)) == dock.DOCK_EINVAL   # no handles
    assert L.dock_ls_shared_waves(items, 0, None, None, C.byref(n)) == dock.DOCK_EINVAL
    assert n.value == -1
    assert L.dock_ls_shared_waves(items, 0, C.byref(o), None, C.byref(n)) == dock.DOCK_OK and n.value == 0
