"""The interface list over rows of one wavefront, of a block's four, and of more
than a block (one reservation per block): FP64 against the oracle, bit for bit;
the FP16 forms against the list of the classes."""
import numpy as np
import pytest

from paper_1409_5645_amd import workloads as W

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def fs():
    from paper_1409_5645_amd import fslbm
    return fslbm


@pytest.mark.parametrize("nx", [64, 65, 128, 130, 256, 257, 512, 514])
def test_rows_of_every_block_shape(fs, oracle_mod, monkeypatch, nx):
    print(f"case list nx={nx}", flush=True)
    monkeypatch.setenv("FSLBM_RESIDENT", "0")
    w = W.sloshing(nx, 18, 4, depth=9.0, amp=3.0, seed=4, gy=-4e-4, tau=0.6, wavelength=40.0)
    o = oracle_mod.Oracle.from_workload(w)
    o.step(12, 1)
    act = o.flags() != W.GAS
    s = fs.Sim.from_workload(w)
    s.step(12, 1)
    g = s.fields(("f", "flags"))
    s.close()
    assert np.array_equal(g["flags"], o.flags())
    assert np.array_equal(g["f"][:, act], o.populations()[:, act])
    for pairs in ("0", "1"):  # every interface cell of an FP16 step is on the list: its fill is the new one
        monkeypatch.setenv("FSLBM_FP16_PAIRS", pairs)
        s = fs.Sim.from_workload(w, precision="fp16s")
        s.step(1, 1)
        g = s.fields(("flags", "phi", "mass", "rho_c"))
        s.close()
        it = g["flags"] == W.INTERFACE
        assert np.array_equal(g["phi"][it], g["mass"][it] / g["rho_c"][it])
