"""GPU: the reverse steps of the adjoint in two kernels (large grids, and two
passes of two rows) against the one kernel of grids in the cache, and beyond
the cache against the oracle."""
import numpy as np
import pytest

import oracle as O
from paper_0809_1547_amd import inputs as I

pytestmark = pytest.mark.gpu


def _run(n, bc, precision, schedule, nsteps, K, frozen=False, source=True):
    from paper_0809_1547_amd import mbf
    eps, gain = I.voxelize(I.rsa_pack(n, seed=4, count=1, radius=0.3 * min(n)))
    sim = mbf.Sim(n, boundary=bc, precision=precision, seed=9, realization=2, E_sp=1e-2, absorb_cells=2, frozen_pop=frozen)
    sim.set_tuning(*schedule)
    sim.set_material(eps, gain)
    sim.set_pump(3e24)
    if source:
        sim.set_source(1, n[0] // 2, n[1] // 2, n[2] // 2, amp=0.3, tau_p=2e-16, t0=4e-16)
    sim.set_loss_box((0, 0, 0), (max(2, n[0] - 1), max(2, n[1] - 2), n[2]))
    out = sim.adjoint_run(nsteps, K=K)
    sim.close()
    return out


@pytest.mark.parametrize("n", [(2, 2, 2), (15, 3, 5), (17, 5, 6), (64, 9, 7), (65, 7, 9), (130, 6, 3), (33, 21, 18)])
@pytest.mark.parametrize("bc", ["pec", "absorb", ("absorb", "pec", "absorb")])
@pytest.mark.parametrize("precision,nsteps,K", [("fp32", 41, 7), ("fp32", 40, 40), ("fp64", 24, 6)])
def test_two_reverse_kernels_equal_one(n, bc, precision, nsteps, K):
    if n == (2, 2, 2) and bc != "pec":
        n = (8, 6, 7)                                 # room for the layers
    La, ga, na = _run(n, bc, precision, ("two_pass", 4, 2), nsteps, K)
    Lb, gb, nb = _run(n, bc, precision, ("two_pass", 2, 2), nsteps, K)
    assert np.any(ga != 0.0)
    assert np.array_equal(ga, gb)
    # the same terms in other partial sums
    assert Lb == pytest.approx(La, rel=1e-12)
    assert nb == pytest.approx(na, rel=1e-9)


@pytest.mark.parametrize("source", [True, False])
def test_frozen_populations(source):
    ra, rb = (_run((33, 21, 18), "absorb", "fp32", ("two_pass", ty, 2), 25, 10, True, source) for ty in (4, 2))
    assert np.array_equal(ra[1], rb[1])


@pytest.mark.parametrize("bc", ["pec", "absorb"])
def test_beyond_the_cache_matches_oracle(bc):
    # 290 MB of reverse state: two kernels by default, as the N_a gradient's bits
    # show; bounds of the small grids' test (FP64 against FP64)
    from paper_0809_1547_amd import mbf
    n, nsteps = (96, 92, 90), 6
    eps, gain = I.voxelize(I.rsa_pack(n, seed=4, count=1, radius=9.0))
    box = ((30, 30, 30), (60, 62, 58))
    got = []
    for schedule in (None, ("two_pass", 2, 4)):
        sim = mbf.Sim(n, boundary=bc, precision="fp64", seed=3, realization=1, E_sp=1e-2, absorb_cells=5)
        if schedule:
            sim.set_tuning(*schedule)
        sim.set_material(eps, gain)
        sim.set_pump(3e24)
        sim.set_source(2, 45, 44, 43, amp=0.3, tau_p=2e-16, t0=4e-16)
        sim.set_loss_box(*box)
        got.append(sim.adjoint_run(nsteps, K=4))
        sim.close()
    assert np.array_equal(got[0][1], got[1][1]) and got[0][2] == got[1][2]
    kind = {"pec": O.PEC, "absorb": O.ABSORB}[bc]
    ora = O.Oracle(O.default_params(n, bc=(kind,) * 3, round_f32=False, seed=3, realization=1, E_sp=1e-2,
                                    absorb_cells=5))
    ora.set_material(eps, gain)
    ora.set_pump(3e24, O.PREPUMPED)
    ora.set_source(2, 45, 44, 43, amp=0.3, tau_p=2e-16, t0=4e-16)
    ora.set_loss_box(*box)
    Lo, go, no = ora.adjoint_run(nsteps)
    ora.close()
    L, g, gna = got[0]
    rel = float(np.linalg.norm(g - go) / np.linalg.norm(go))
    print(bc, "L", L, Lo, "g_eps rel", rel, "g_Na", gna, no)
    assert L == pytest.approx(Lo, rel=1e-12)
    assert rel <= 1e-10
    assert gna == pytest.approx(no, rel=1e-10)
