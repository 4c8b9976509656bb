"""Workspace queries never shrink as the problem grows, so that a workspace for a larger one always serves a
smaller one (CPU only: the queries make no HIP call)."""
import ctypes as C

import pytest

# around every size at which a sort, a scan or a numbering changes its form
SIZES = sorted({s + d for s in [1 << k for k in range(8, 29)] + [3 * 256 << 10, 8_388_608, 4_300_000, 12_000_000]
                for d in (-4097, -1025, -257, -1, 0, 1, 255, 1024, 4097) if s + d > 0} | set(range(1, 40)))


def queries():
    from paper_2604_12942_amd import _abi
    L = _abi.load()
    out = {k: (lambda f: lambda n: int(f(n)))(getattr(L, "gsr_%s_workspace" % k))
           for k in ("row_order", "prune", "gicp", "voxel_pca", "visible_list")}
    out["proximity map"] = lambda n: int(L.gsr_proximity_workspace(n, 1000))
    out["proximity new"] = lambda n: int(L.gsr_proximity_workspace(1000, n))
    r = _abi.Raster(1920, 1080, 16, 16)
    out["bin_sort rows"] = lambda n: int(L.gsr_bin_sort_workspace(n, 1, 1000, C.byref(r)))
    out["bin_sort instances"] = lambda n: int(L.gsr_bin_sort_workspace(1000, 1, n, C.byref(r)))
    out["render_fwd_sliced"] = lambda n: int(L.gsr_render_fwd_sliced_workspace(1, C.byref(r), n))
    out["render_step"] = lambda n: int(L.gsr_render_step_workspace(1, C.byref(r), n))
    out["project_bwd"] = lambda n: int(L.gsr_project_bwd_workspace(n, 2))
    return out


@pytest.mark.parametrize("name", ["row_order", "prune", "gicp", "voxel_pca", "visible_list", "proximity map", "proximity new",
                                  "bin_sort rows", "bin_sort instances", "render_fwd_sliced", "render_step", "project_bwd"])
def test_workspace_never_shrinks(name):
    f = queries()[name]
    got = [f(n) for n in SIZES]
    down = [(a, b, x, y) for a, b, x, y in zip(SIZES, SIZES[1:], got, got[1:]) if y < x]
    assert not down, down[:3]
