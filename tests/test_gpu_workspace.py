"""Workspaces without the parts that only faster routes need are still taken, with
the same results, and the static workspace still holds the largest lattice that
its size allows."""
import ctypes

import numpy as np
import pytest

from paper_1409_5645_amd import workloads as W

pytestmark = pytest.mark.gpu

STATIC = 64 << 20
LINE = 256


@pytest.fixture(scope="module")
def fs():
    from paper_1409_5645_amd import fslbm
    return fslbm


def up(n):
    return (n + LINE - 1) // LINE * LINE


def least(n, precision, static=False, kappa=False):
    """Bytes that every context needs: collision values of the interface cells, marks, lists, counters,
    scalars, extents, wall terms and (not in FP16, not static) the interface-first buffers."""
    o = up(32 * n) + 11 * up(4 * n) + up(64) + up(80) + up(65 * 128) + up(8 * 6 * 19)
    if kappa:
        o += up(8 * n)
    if precision != "fp16s" and not static:
        s = 8 if precision == "fp64" else 4
        o += up(4 * n) + up(19 * s * (n if n <= 32768 else max(32768, n // 8)))
    return o


def with_workspace(fs, monkeypatch, w, precision, nbytes):
    """A context whose workspace has nbytes (None: as fslbm_workspace_size says)."""
    with monkeypatch.context() as m:
        if nbytes is not None:
            def fake(params, out):
                out._obj.value = nbytes
                return 0
            m.setattr(fs.lib(), "fslbm_workspace_size", fake)
        return fs.Sim.from_workload(w, precision=precision)


def full_size(fs, w, precision):
    cp, ws = fs.make_params(w.params, fs.PRECISIONS[precision]), ctypes.c_size_t()
    assert fs.lib().fslbm_workspace_size(ctypes.byref(cp), ctypes.byref(ws)) == 0
    return ws.value


def tank(nx, ny, nz):
    return W.sloshing(nx, ny, nz, depth=0.55 * ny, amp=0.1 * ny, seed=3, gy=-2e-4, tau=0.6, amp_z=0.04 * ny)


@pytest.mark.parametrize("precision", ["fp64", "fp32", "fp16s"])
@pytest.mark.parametrize("size", [(8, 48, 8), (31, 25, 17), (61, 45, 37)])
def test_least_workspace(fs, monkeypatch, size, precision):
    print(f"case least workspace {size} {precision}", flush=True)
    w = tank(*size)
    n = w.params.n_cells
    need = least(n, precision)
    assert need < full_size(fs, w, precision)
    with pytest.raises(fs.FslbmError, match="workspace too small"):
        with_workspace(fs, monkeypatch, w, precision, need - 1)
    out = []
    for nbytes in (None, need):
        s = with_workspace(fs, monkeypatch, w, precision, nbytes)
        for k in (1, 3, 12, 40):
            s.step(k, 1)
        out.append((s.fields(("f", "flags", "mass", "phi")), s.conversions()))
        s.close()
    (a, ca), (b, cb) = out
    act = a["flags"] != W.GAS
    assert np.array_equal(a["flags"], b["flags"])
    for k in ("f", "mass", "phi"):
        assert np.array_equal(a[k][..., act], b[k][..., act]), k
    for k in ca:
        np.testing.assert_array_equal(ca[k], cb[k], err_msg=k)


@pytest.mark.parametrize("precision,nz", [("fp64", 180), ("fp32", 350)])
def test_workspace_without_the_third_buffer(fs, monkeypatch, precision, nz):
    import torch
    print(f"case third buffer {precision}", flush=True)
    w = W.sloshing(128, 96, nz, depth=58.0, amp=4.0, seed=2, gy=-2e-5, tau=0.56, amp_z=2.0)
    third = up(19 * w.params.n_cells * (8 if precision == "fp64" else 4))
    size = full_size(fs, w, precision)
    assert size == least(w.params.n_cells, precision) + third + LINE  # the kept list's length
    out = []
    for nbytes in (size, size - 1, size - third):
        s = with_workspace(fs, monkeypatch, w, precision, nbytes)
        s.step(5, 1)
        s.step(12, 1)
        out.append(s.fields(("f", "flags", "mass", "phi"), device=True))
        s.close()
    act = (out[0]["flags"] == W.LIQUID) | (out[0]["flags"] == W.INTERFACE)
    for g in out[1:]:
        assert torch.equal(g["flags"], out[0]["flags"])
        for k in ("f", "mass", "phi"):
            assert torch.equal(g[k][..., act], out[0][k][..., act]), k


def test_static_workspace_to_its_last_bytes(fs):
    n = next(k for k in range(STATIC // 76, 0, -1) if least(k, "fp64", static=True) <= STATIC)
    assert STATIC - least(n, "fp64", static=True) < 2 * LINE  # nothing to spare
    for cells, ok in ((n, True), (n + 4 * LINE, False)):
        p = W.Params(nx=cells, ny=1, nz=1)
        if not ok:
            with pytest.raises(fs.FslbmError, match="static workspace") as e:
                fs.Sim(p, np.zeros(cells, np.uint8), static_workspace=True)
            assert e.value.status == 6
            continue
        s = fs.Sim(p, np.full(cells, W.LIQUID, np.uint8), static_workspace=True)
        s.set_equilibrium(np.ones(cells), np.zeros((3, cells)), np.ones(cells))
        s.step(3, 1)
        assert s.stats()["liquid"] == cells
        s.close()
