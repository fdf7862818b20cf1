"""Runs of steps in one launch (the resident step of small lattices): the same
bits as the step-by-step kernels and, in FP64, as the serial oracle."""
import numpy as np
import pytest

from paper_1409_5645_amd import workloads as W

pytestmark = pytest.mark.gpu

LIMIT = 32768  # cells of the largest resident lattice (csrc/fslbm_internal.hpp)


@pytest.fixture(scope="module")
def fs():
    from paper_1409_5645_amd import fslbm
    return fslbm


def run(fs, monkeypatch, w, precision, rule, chunks, resident, **kw):
    monkeypatch.setenv("FSLBM_RESIDENT", "1" if resident else "0")
    s = fs.Sim.from_workload(w, precision=precision, **kw)
    out = []
    for n in chunks:
        s.step(n, rule)
        g = s.fields(("f", "flags", "mass", "phi", "rho_c", "u_c"))
        st = s.stats()
        # sums by atomics in an order of their own
        assert abs(st["total_mass"] - (out[0][2]["total_mass"] if out else st["total_mass"])) < 1e-3 * st["total_mass"]
        out.append((g, s.conversions(), st))
    s.close()
    return out


def slosh(nx, ny, nz, amp=None, gy=-4e-4, periodic=(0, 0, 0)):
    amp = 0.16 * ny if amp is None else amp
    return W.sloshing(nx, ny, nz, depth=0.55 * ny, amp=amp, seed=3, gy=gy, tau=0.6, periodic=periodic,
                      amp_z=0.4 * amp)


CASES = {
    "one cell": (lambda: W.channel(h=0.5, nx=1, ny=1, nz=1), (1, 3)),
    "film": (lambda: W.channel(nx=4, ny=80, nz=4, h=54.5), (1, 2, 300)),       # longer than one launch's run
    "list made anew": (lambda: slosh(6, 8, 3, amp=3.5, gy=-2e-3), (250, 20)),  # its entries pass the cell count
    "conversions": (lambda: slosh(31, 25, 17), (1, 7, 60)),
    "periodic": (lambda: slosh(48, 22, 10, periodic=(1, 0, 1)), (1, 50)),
    "largest": (lambda: slosh(32, 32, 32), (1, 30)),
    "past the limit": (lambda: slosh(33, 31, 33), (1, 10)),
}


@pytest.mark.parametrize("precision,rule", [("fp64", 0), ("fp64", 1), ("fp64", 3), ("fp64", 4), ("fp64", 5),
                                            ("fp32", 0), ("fp32", 1), ("fp32", 2), ("fp32", 5)])
@pytest.mark.parametrize("name", list(CASES))
def test_resident_is_bit_identical(fs, monkeypatch, name, precision, rule):
    print(f"case resident {name} {precision} rule={rule}", flush=True)
    make, chunks = CASES[name]
    w = make()
    assert (w.params.n_cells <= LIMIT) == (name != "past the limit")
    kw = {"check_every": 7} if name == "conversions" else {}
    a = run(fs, monkeypatch, w, precision, rule, chunks, False, **kw)
    b = run(fs, monkeypatch, w, precision, rule, chunks, True, **kw)
    for (ga, ca, sa), (gb, cb, sb) in zip(a, b):
        act = ga["flags"] != W.GAS
        assert np.array_equal(ga["flags"], gb["flags"])
        for k in ("f", "mass", "phi", "rho_c"):
            assert np.array_equal(ga[k][..., act], gb[k][..., act]), k
        act[np.concatenate((ca["NI"], ca["NL"]))] = False  # not collided as interface cells yet: no u_c
        assert np.array_equal(ga["u_c"][:, act], gb["u_c"][:, act])
        for k in ca:
            np.testing.assert_array_equal(ca[k], cb[k], err_msg=k)
        assert all(sa[k] == sb[k] for k in sa if k not in ("total_mass", "reservoir"))


def test_resident_matches_oracle_and_list_is_remade(fs, oracle_mod):
    w = CASES["list made anew"][0]()
    o = oracle_mod.Oracle.from_workload(w)
    s = fs.Sim.from_workload(w)
    entries = int((w.flags == W.INTERFACE).sum())
    for _ in range(250):
        o.step(1, 1)
        lists = o.lists()
        entries += len(lists["NI"]) + len(lists["NL"])
    assert entries > w.params.n_cells  # in one launch the list outgrows the lattice
    s.step(250, 1)
    g = s.fields(("f", "flags"))
    act = g["flags"] != W.GAS
    assert np.array_equal(g["flags"], o.flags())
    assert np.array_equal(g["f"][:, act], o.populations()[:, act])
    s.close()


def test_resident_contexts_on_two_streams(fs):
    """Two contexts on streams of their own, steps enqueued in turn, against the same steps alone."""
    import torch
    w = slosh(31, 25, 17)
    alone = fs.Sim.from_workload(w)
    alone.step(60, 1)
    ref = alone.fields(("f", "flags"))
    sims = [fs.Sim.from_workload(w, stream=torch.cuda.Stream()) for _ in range(2)]
    for _ in range(6):
        for s in sims:
            s.step(10, 1)
    act = ref["flags"] != W.GAS
    for s in sims:
        g = s.fields(("f", "flags"))
        assert np.array_equal(g["flags"], ref["flags"])
        assert np.array_equal(g["f"][:, act], ref["f"][:, act])
        s.close()
    alone.close()
