"""Steps in which a surface converts as a whole: counts of converted cells around
the widths of the team that does them (32, 96 and up to 256 workgroups of 16
cells), against the serial oracle: FP64 bit for bit, the lists in every form."""
import numpy as np
import pytest

from paper_1409_5645_amd import workloads as W

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def fs():
    from paper_1409_5645_amd import fslbm
    return fslbm


@pytest.fixture(scope="module")
def stepped(oracle_mod):
    """The workload and the oracle's state after its first step and the next."""
    made = {}

    def get(converted, kind):
        if (converted, kind) not in made:
            w = W.pool(nx=129, ny=16, nz=128, level=8.5, gy=0.0)
            it = np.nonzero(w.flags == W.INTERFACE)[0]
            c = np.random.default_rng(3).permutation(it)[:converted]
            full = np.ones(c.size, bool) if kind == "fill" else (np.zeros(c.size, bool) if kind == "empty"
                                                                 else np.arange(c.size) % 2 == 0)
            w.fill[c] = np.where(full, 1.01, -0.01)
            o = oracle_mod.Oracle.from_workload(w)
            out = []
            for _ in range(2):
                o.step(1, 0)
                out.append((o.flags().copy(), o.populations().copy(), o.mass().copy(), o.phi().copy(), o.lists()))
            made[converted, kind] = (w, out)
        return made[converted, kind]
    return get


@pytest.mark.parametrize("precision", ["fp64", "fp32", "fp16s"])
@pytest.mark.parametrize("kind", ["fill", "empty", "both"])
@pytest.mark.parametrize("converted", [127, 129, 1919, 1921, 5200, 16512])
def test_surface_that_converts_as_a_whole(fs, stepped, converted, kind, precision):
    print(f"case wide {converted} {kind} {precision}", flush=True)
    w, want = stepped(converted, kind)
    s = fs.Sim.from_workload(w, precision=precision)
    for flags, f, mass, phi, lists in want if precision == "fp64" else want[:1]:
        s.step(1, 0)
        g, got = s.fields(("f", "flags", "mass", "phi")), s.conversions()
        assert np.array_equal(g["flags"], flags)
        for k in lists:
            np.testing.assert_array_equal(got[k], np.sort(lists[k]), err_msg=k)
        if precision == "fp64":
            act, it = flags != W.GAS, flags == W.INTERFACE
            assert np.array_equal(g["f"][:, act], f[:, act])
            assert np.array_equal(g["mass"][it], mass[it])
            assert np.array_equal(g["phi"][it], phi[it])
    assert len(want[0][4]["F"]) + len(want[0][4]["E"]) == converted
    s.close()
