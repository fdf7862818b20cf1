"""The conversion passes (one kernel; a few converted cells in one workgroup,
more over the grid) against the serial FP64 oracle: steps with every count of
converted cells around the limit between the two, at walls and periodic faces."""
import numpy as np
import pytest

from paper_1409_5645_amd import workloads as W

pytestmark = pytest.mark.gpu

SOLO_CELLS = 8  # converted cells up to which one workgroup does them (csrc/fslbm_internal.hpp)


@pytest.fixture(scope="module")
def fs():
    from paper_1409_5645_amd import fslbm
    return fslbm


def same_state(s, o):
    """Classes, lists, populations, mass and fill equal to the oracle's, bit for bit (the FP64 form
    has the oracle's expression order)."""
    g = s.fields(("f", "flags", "mass", "phi"))
    fl = o.flags()
    act, it = fl != W.GAS, fl == W.INTERFACE
    assert np.array_equal(g["flags"], fl)
    assert np.array_equal(g["f"][:, act], o.populations()[:, act])
    assert np.array_equal(g["mass"][it], o.mass()[it])
    assert np.array_equal(g["phi"][it], o.phi()[it])
    lg, lo = s.conversions(), o.lists()
    for k in lo:
        np.testing.assert_array_equal(lg[k], lo[k], err_msg=k)
    return len(lo["F"]) + len(lo["E"])


@pytest.mark.parametrize("periodic", [(0, 0, 0), (1, 0, 1)])
@pytest.mark.parametrize("size,amp,few", [((31, 25, 17), 4.0, True), ((64, 40, 40), 8.0, False)])
def test_conversion_counts_around_the_solo_limit(fs, oracle_mod, size, amp, few, periodic):
    print(f"case conversions {size} periodic={periodic}", flush=True)
    nx, ny, nz = size
    w = W.sloshing(nx, ny, nz, depth=0.55 * ny, amp=amp, seed=3, gy=-4e-4, tau=0.6, periodic=periodic,
                   amp_z=0.5 * amp)
    o = oracle_mod.Oracle.from_workload(w)
    s = fs.Sim.from_workload(w)
    seen = []
    for _ in range(60):
        o.step(1, 1)
        s.step(1, 1)
        seen.append(same_state(s, o))
    s.close()
    assert any(n > SOLO_CELLS for n in seen), sorted(set(seen))
    assert not few or set(range(1, SOLO_CELLS + 1)) <= set(seen), sorted(set(seen))
