"""Two steps at once below the surface, on lattices thinner than a tile or of one
to three planes whose faces wrap (the loads' ranges are checked on the CPU by
test_deep_index.py), and with the rules that reach furthest below the surface:
the same bits as one step after the other."""
import dataclasses

import numpy as np
import pytest

from paper_1409_5645_amd import workloads as W

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def fs():
    from paper_1409_5645_amd import fslbm
    return fslbm


def compare(fs, monkeypatch, w, precision, rule):
    import torch
    assert 19 * w.params.n_cells * (8 if precision == "fp64" else 4) >= 300e6
    out = []
    for deep in ("0", "1"):
        monkeypatch.setenv("FSLBM_DEEP", deep)
        s = fs.Sim.from_workload(w, precision=precision)
        got = []
        for n in (3, 7, 12):
            s.step(n, rule)
            got.append((s.fields(("f", "flags", "mass", "phi"), device=True), s.conversions()))
        out.append(got)
        s.close()
    for (a, ca), (b, cb) in zip(*out):
        act = (a["flags"] == W.LIQUID) | (a["flags"] == W.INTERFACE)
        assert torch.equal(a["flags"], b["flags"])
        for k in ("f", "mass", "phi"):
            assert torch.equal(a[k][..., act], b[k][..., act]), k
        for k in ca:
            np.testing.assert_array_equal(ca[k], cb[k], err_msg=k)


def tank(nx, ny, nz, periodic=(0, 0, 0), gy=-2e-5):
    return W.sloshing(nx, ny, nz, depth=0.6 * ny, amp=4.0, seed=2, gy=gy, tau=0.56, periodic=periodic, amp_z=2.0)


def full(nx, ny, nz, periodic):
    w = W.pool(nx=nx, ny=ny, nz=nz, level=2.0 * ny, gy=0.0)
    u = 1e-3 * np.random.default_rng(5).standard_normal((3, w.params.n_cells))  # nothing looks like its neighbour
    return dataclasses.replace(w, u=u, params=dataclasses.replace(w.params, periodic=periodic))


# sizes (FP64, FP32); buffers of 19 N values just past the smallest that take it
THIN = {
    "one plane": lambda k: tank(2048 * k, 1024, 1, periodic=(0, 0, 1)),
    "one plane, all wrap": lambda k: tank(1999 * k, 1024, 1, periodic=(1, 0, 1)),
    "two planes": lambda k: tank(1023 * k, 1024, 2, periodic=(0, 0, 1)),
    "three planes": lambda k: tank(701 * k, 1000, 3, periodic=(1, 0, 1)),
    "four columns": lambda k: tank(4, 1024, 512 * k, periodic=(1, 0, 0)),
    "one column, all liquid": lambda k: full(1, 1024, 2048 * k, (1, 0, 0)),
    "columns of less than half a tile, all liquid": lambda k: full(8 * k, 512, 512, (1, 0, 1)),
}


@pytest.mark.parametrize("precision", ["fp64", "fp32"])
@pytest.mark.parametrize("name", list(THIN))
def test_thin_lattices(fs, monkeypatch, name, precision):
    print(f"case thin {name} {precision}", flush=True)
    compare(fs, monkeypatch, THIN[name](1 if precision == "fp64" else 2), precision, 1)


@pytest.mark.parametrize("precision,nz", [("fp64", 180), ("fp32", 350)])
@pytest.mark.parametrize("rule", [2, 3, 4, 5])
@pytest.mark.parametrize("gy", [-2e-5, -3e-4])
def test_rules_with_a_boundary_shear(fs, monkeypatch, precision, nz, rule, gy):
    print(f"case deep rule {rule} {precision} gy {gy}", flush=True)
    compare(fs, monkeypatch, tank(120, 100, nz, gy=gy), precision, rule)
