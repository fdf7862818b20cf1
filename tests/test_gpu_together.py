"""The interface cells and the sweep of a step in one launch, from a list that
the conversions keep: rows of one wavefront, of a block and beyond, odd rows in
FP16 storage, steps across the list's renewal, many conversions, cells that
leave the surface and come back.  FP64 bit for bit with the oracle; every form
bit for bit with the three kernels of a step (the operations are the same)."""
import numpy as np
import pytest

from paper_1409_5645_amd import workloads as W

pytestmark = pytest.mark.gpu
NAMES = ("f", "flags", "mass", "phi")


@pytest.fixture(scope="module")
def fs():
    from paper_1409_5645_amd import fslbm
    return fslbm


def _run(fs, monkeypatch, w, together, precision, rule, parts):
    monkeypatch.setenv("FSLBM_RESIDENT", "0")
    monkeypatch.setenv("FSLBM_TOGETHER", together)
    s = fs.Sim.from_workload(w, precision=precision)
    for n in parts:
        s.step(n, rule)
    g = s.fields(NAMES)
    s.close()
    return g


def _same(a, b):
    act = a["flags"] != W.GAS
    it = a["flags"] == W.INTERFACE
    return (np.array_equal(a["flags"], b["flags"]) and np.array_equal(a["f"][:, act], b["f"][:, act])
            and np.array_equal(a["mass"][it], b["mass"][it]) and np.array_equal(a["phi"][it], b["phi"][it]))


@pytest.mark.parametrize("nx", [3, 61, 64, 65, 130, 259])
@pytest.mark.parametrize("rule", [0, 1, 3])
def test_one_launch_for_surface_and_sweep(fs, oracle_mod, monkeypatch, nx, rule):
    print(f"case together nx={nx} rule={rule}", flush=True)
    w = W.sloshing(nx, 20, 6, depth=9.0, amp=3.0, seed=4, gy=-4e-4, tau=0.6, wavelength=40.0)
    parts = (8, 3, 90)  # three steps the other way; 90 steps see the list renewed
    g = _run(fs, monkeypatch, w, "1", "fp64", rule, parts)
    o = oracle_mod.Oracle.from_workload(w)
    o.step(sum(parts), rule)
    act = o.flags() != W.GAS
    it = o.flags() == W.INTERFACE
    assert np.array_equal(g["flags"], o.flags())
    assert np.array_equal(g["f"][:, act], o.populations()[:, act])
    assert np.array_equal(g["phi"][it], o.phi()[it])
    for precision in ("fp32", "fp16s"):
        print(precision, flush=True)
        assert _same(_run(fs, monkeypatch, w, "1", precision, rule, parts),
                     _run(fs, monkeypatch, w, "0", precision, rule, parts)), precision


@pytest.mark.parametrize("precision", ["fp64", "fp32", "fp16s"])
def test_conversion_burst(fs, monkeypatch, precision):
    """A falling blob: hundreds of conversions a step, cells that return."""
    w = W.droplet(n=28, radius=8.0, sigma=0.0)
    import dataclasses
    w = dataclasses.replace(w, params=dataclasses.replace(w.params, g=(0.0, -2e-3, 0.0)))
    print(f"case together burst {precision}", flush=True)
    assert _same(_run(fs, monkeypatch, w, "1", precision, 1, (150,)), _run(fs, monkeypatch, w, "0", precision, 1, (150,)))
