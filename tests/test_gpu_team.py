"""Kernels whose workgroups wait for one another go on with those that are on the
device: teams of every small size (one workgroup alone included) and teams
closed at once give the same bits as a full one, in the resident steps and in
the conversions."""
import numpy as np
import pytest

from paper_1409_5645_amd import workloads as W

pytestmark = pytest.mark.gpu

TEAMS = [{"FSLBM_TEAM": "1"}, {"FSLBM_TEAM": "2"}, {"FSLBM_TEAM": "3"}, {"FSLBM_TEAM": "7"}, {"FSLBM_TEAM_WAIT": "0"}]


@pytest.fixture(scope="module")
def fs():
    from paper_1409_5645_amd import fslbm
    return fslbm


def slosh(nx, ny, nz, gy=-4e-4):
    return W.sloshing(nx, ny, nz, depth=0.55 * ny, amp=0.16 * ny, seed=3, gy=gy, tau=0.6, amp_z=0.06 * ny)


def run(fs, monkeypatch, w, precision, rule, chunks, env):
    for k in ("FSLBM_TEAM", "FSLBM_TEAM_WAIT", "FSLBM_RESIDENT"):
        monkeypatch.delenv(k, raising=False)
    for k, v in env.items():
        monkeypatch.setenv(k, v)
    s = fs.Sim.from_workload(w, precision=precision)
    out = []
    for n in chunks:
        s.step(n, rule)
        out.append((s.fields(("f", "flags", "mass", "phi")), s.conversions()))
    s.close()
    return out


def same(a, b):
    for (ga, ca), (gb, cb) in zip(a, b):
        act = ga["flags"] != W.GAS
        assert np.array_equal(ga["flags"], gb["flags"])
        for k in ("f", "mass", "phi"):
            assert np.array_equal(ga[k][..., act], gb[k][..., act]), k
        for k in ca:
            np.testing.assert_array_equal(ca[k], cb[k], err_msg=k)


@pytest.mark.parametrize("precision,rule", [("fp64", 1), ("fp64", 3), ("fp32", 1), ("fp32", 2)])
@pytest.mark.parametrize("env", TEAMS, ids=lambda e: "-".join(f"{k[6:]}{v}" for k, v in e.items()))
def test_resident_steps_of_a_part_of_the_grid(fs, monkeypatch, precision, rule, env):
    print(f"case team resident {precision} rule {rule} {env}", flush=True)
    w = slosh(31, 25, 17, gy=-1.2e-3)
    ref = run(fs, monkeypatch, w, precision, rule, (1, 6, 30, 3), {"FSLBM_RESIDENT": "0"})
    same(ref, run(fs, monkeypatch, w, precision, rule, (1, 6, 30, 3), {"FSLBM_RESIDENT": "1", **env}))
    assert any(sum(v.size for v in c.values()) > 0 for _, c in ref)


@pytest.mark.parametrize("precision", ["fp64", "fp32", "fp16s"])
@pytest.mark.parametrize("env", [{}] + TEAMS, ids=lambda e: "-".join(f"{k[6:]}{v}" for k, v in e.items()) or "full")
@pytest.mark.parametrize("converted", [9, 60, 700])
def test_conversions_of_a_part_of_the_grid(fs, oracle_mod, monkeypatch, precision, env, converted):
    """A flat surface of which some cells fill and some empty in the first step:
    the first step's lists as the oracle's, the rest the same bits as with
    the full team."""
    print(f"case team conversions {precision} {env} {converted}", flush=True)
    w = W.pool(nx=61, ny=20, nz=47, level=11.5, gy=0.0)
    cells = np.random.default_rng(7).permutation(np.nonzero(w.flags == W.INTERFACE)[0])[:converted]
    w.fill[cells] = np.where(np.arange(converted) % 3 == 0, -0.01, 1.01)
    ref = run(fs, monkeypatch, w, precision, 1, (1, 10), {})
    got = run(fs, monkeypatch, w, precision, 1, (1, 10), env)
    same(ref, got)
    o = oracle_mod.Oracle.from_workload(w)
    o.step(1, 1)
    lists = o.lists()
    assert len(lists["F"]) + len(lists["E"]) == converted
    for k in lists:
        np.testing.assert_array_equal(got[0][1][k], np.sort(lists[k]), err_msg=k)
    if precision == "fp64":
        g = got[0][0]
        act = g["flags"] != W.GAS
        assert np.array_equal(g["flags"], o.flags())
        assert np.array_equal(g["f"][:, act], o.populations()[:, act])


def test_eight_contexts_share_the_device(fs, monkeypatch):
    """Resident steps whose workgroups take a compute unit each (FP64, boundary shear from the bulk) and
    conversions of larger lattices, on eight streams at once: each as alone."""
    import torch
    for k in ("FSLBM_TEAM", "FSLBM_TEAM_WAIT"):
        monkeypatch.delenv(k, raising=False)
    monkeypatch.setenv("FSLBM_RESIDENT", "1")
    loads = [(slosh(31, 25, 17, gy=-1.2e-3), 3), (slosh(48, 40, 44, gy=-6e-4), 1)]
    refs = []
    for w, rule in loads:
        s = fs.Sim.from_workload(w)
        s.step(60, rule)
        refs.append(s.fields(("f", "flags")))
        s.close()
    sims = [(i % 2, fs.Sim.from_workload(loads[i % 2][0], stream=torch.cuda.Stream())) for i in range(8)]
    for _ in range(6):
        for k, s in sims:
            s.step(10, loads[k][1])
    for k, s in sims:
        g = s.fields(("f", "flags"))
        act = refs[k]["flags"] != W.GAS
        assert np.array_equal(g["flags"], refs[k]["flags"])
        assert np.array_equal(g["f"][:, act], refs[k]["f"][:, act])
        s.close()
