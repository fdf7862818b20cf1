"""Two steps at once below the surface (k_deep): the same bits as one step after
the other, for the FP64 and FP32 forms, over ragged tiles, walls and periodic faces, options
that act near the surface, solids in the liquid, and a moving row limit."""
import numpy as np
import pytest

from paper_1409_5645_amd import workloads as W

pytestmark = pytest.mark.gpu

ROWS = 24  # fewest rows the two-step kernel takes (csrc/fslbm_internal.hpp)


@pytest.fixture(scope="module")
def fs():
    from paper_1409_5645_amd import fslbm
    return fslbm


def tank(nx, ny, nz, periodic=(0, 0, 0), gy=-2e-5, **kw):
    w = W.sloshing(nx, ny, nz, depth=0.6 * ny, amp=4.0, seed=2, gy=gy, tau=0.56, periodic=periodic, amp_z=2.0)
    if kw:
        import dataclasses
        w = dataclasses.replace(w, params=dataclasses.replace(w.params, **kw))
    return w


def with_solid(w, y0, y1):
    """A solid block well inside the liquid, walls halfway."""
    p = w.params
    cls = w.flags.reshape(p.nz, p.ny, p.nx).copy()
    cls[p.nz // 3:p.nz // 2, y0:y1, p.nx // 3:p.nx // 2] = W.SOLID
    solid = cls == W.SOLID
    near = W._shift_any(solid, p.periodic) & ~solid
    cells = np.nonzero(near.reshape(-1))[0].astype(np.int32)
    w.flags = cls.reshape(-1)
    w.fill = np.where(solid.reshape(-1), 0.0, w.fill)
    w.walls = {"cells": cells, "delta": np.full((19, cells.size), 0.5), "uw": np.zeros((3, 19, cells.size))}
    return w


# sizes by the form: the buffers of 19 N values are just past the smallest that take it
NZ = {"fp64": 180, "fp32": 350}
CASES = {
    "tank": lambda nz: tank(128, 96, nz),
    "ragged": lambda nz: tank(133, 101, nz - 3),
    "periodic": lambda nz: tank(96, 128, nz, periodic=(1, 0, 1)),
    "periodic ragged": lambda nz: tank(101, 125, nz + 1, periodic=(1, 0, 1)),
    "falling surface": lambda nz: tank(120, 100, nz, gy=-3e-4),
    "narrow": lambda nz: tank(30, 420, nz),
    "tension": lambda nz: tank(128, 96, nz, sigma=1e-4, plic=2),
    "solid": lambda nz: with_solid(tank(128, 96, nz), 40, 46),
    "all liquid": lambda nz: W.pool(nx=128, ny=96, nz=nz, level=150.0),
}


@pytest.mark.parametrize("precision", ["fp64", "fp32"])
@pytest.mark.parametrize("name", list(CASES))
def test_two_steps_at_once_are_bit_identical(fs, monkeypatch, name, precision):
    print(f"case deep {name} {precision}", flush=True)
    import torch
    w = CASES[name](NZ[precision])
    rows = w.flags.reshape(w.params.nz, w.params.ny, w.params.nx).transpose(1, 0, 2).reshape(w.params.ny, -1)
    other = np.nonzero((rows != W.LIQUID).any(axis=1))[0]
    assert (other[0] if other.size else w.params.ny) >= ROWS + 14  # rows for it up to the last step's age
    assert 19 * w.params.n_cells * (8 if precision == "fp64" else 4) >= 300e6
    out = []
    for deep in ("0", "1"):
        monkeypatch.setenv("FSLBM_DEEP", deep)
        s = fs.Sim.from_workload(w, precision=precision)
        got = []
        for n in (3, 7, 12, 1, 16):  # odd and even runs from states whose extent has arrived
            s.step(n, 1)
            got.append((s.fields(("f", "flags", "mass", "phi"), device=True), s.conversions()))
        st = s.fields(("f", "mass", "phi"), device=True)
        s.set_state(st["f"], st["mass"], st["phi"])  # forgets the extent; a third buffer holds nothing of use
        s.step(2, 0)
        s.stats()
        s.step(5, 0)
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
