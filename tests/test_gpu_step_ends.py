"""GPU: the end of a step with many partial sums (narrow workgroups, one-plane
segments), whose waves are summed one by one and added a launch later: the
energy of every step, the loss, the probes and the fields against steps that
one workgroup ends, and its cost beside the step's kernels."""
import time

import numpy as np
import pytest

from paper_0809_1547_amd import inputs as I

pytestmark = pytest.mark.gpu

STEPS = 70


def _sim(n, variant, tile_y, zseg, precision="fp32", box=True, decim=0, sim=None):
    from paper_0809_1547_amd import mbf
    eps = np.full(n[::-1], 2.25, dtype=np.float32)
    gain = np.zeros(n[::-1], dtype=np.uint8)
    gain[:, :, 5:33] = 1
    if sim is None:
        sim = mbf.Sim(n, boundary="absorb", precision=precision, seed=3, E_sp=1e-2, energy_history=STEPS)
        sim.set_tuning(variant, tile_y=tile_y, zseg=zseg)
    sim.set_material(eps, gain)
    sim.set_pump(2e24)
    sim.set_source(2, 20, 10, 12, amp=0.3)
    if box:
        sim.set_loss_box((3, 3, 3), (n[0] - 4, n[1] - 3, n[2] - 5))
    if decim:
        sim.set_probes(I.select_probes(eps, gain, 9, seed=1), [2e15, 3e15, 4e15], decim=decim)
    return sim


def _results(sim, decim=0):
    return [np.array(sim.energy()), np.array(sim.loss()), sim.energy_history()] + [sim.field(q) for q in (2, 5, 8, 13)] + (
        [sim.spectrum()] if decim else [])


# 2560 (two rows) to 19200 (sixteen) partials: more than one workgroup sums at
# the front of a launch, few enough for one in a launch of its own
@pytest.mark.parametrize("n,variant,tile_y", [((64, 40, 32), "two_pass", 2), ((64, 40, 32), "two_pass_split", 2),
                                              ((64, 40, 32), "fused", 2), ((70, 64, 65), "two_pass_split", 4),
                                              ((70, 64, 65), "fused", 4), ((128, 64, 70), "two_pass_split", 8),
                                              ((128, 96, 100), "fused", 16)])
@pytest.mark.parametrize("precision,box,decim", [("fp32", True, 0), ("fp32", False, 5), ("fp64", True, 40)])
def test_many_partials_keep_their_sums(n, variant, tile_y, precision, box, decim):
    from paper_0809_1547_amd import mbf
    one = _sim(n, variant, tile_y, 1, precision, box, decim)
    one.step_timed(STEPS)
    ref = _results(one, decim)
    one.close()
    sim = _sim(n, variant, tile_y, 1, precision, box, decim)
    for part in (1, 2, 33, 34):
        sim.step(part)
    for q, (a, b) in enumerate(zip(ref, _results(sim, decim))):
        assert np.array_equal(a, b), q
    sim.close()
    # a batch whose other member has no loss box and few partials
    batch = mbf.Batch([mbf.make_config(n, boundary="absorb", precision=precision, seed=3, E_sp=1e-2, energy_history=STEPS),
                       mbf.make_config((40, 24, 20), boundary="absorb", precision=precision, seed=4)])
    batch.set_tuning(variant, tile_y=tile_y, zseg=1)
    _sim(n, None, None, None, box=box, decim=decim, sim=batch[0])
    _sim((40, 24, 20), None, None, None, box=False, sim=batch[1])
    batch.step(STEPS)
    for q, (a, b) in enumerate(zip(ref, _results(batch[0], decim))):
        assert np.array_equal(a, b), ("batch", q)
    batch.close()


# 67600 partials: by units in a launch of their own as well; against one
# workgroup's sums of the 34320 partials that workgroups of four rows leave (the
# same lanes' shares, added up in FP64 in another order: 1e-12)
@pytest.mark.parametrize("variant", ["two_pass", "fused_lds"])
def test_most_partials(variant):
    n = (64, 130, 260)
    res = []
    for parts in ((STEPS,), (1,) * 6 + (STEPS - 6,)):
        sim = _sim(n, variant, 2, 1)
        for p in parts:
            sim.step(p)
        res.append(_results(sim))
        sim.close()
    for a, b in zip(res[0], res[1]):
        assert np.array_equal(a, b)
    one = _sim(n, "two_pass_split", 4, 1)
    one.step_timed(STEPS)
    ref = _results(one)
    one.close()
    for q in range(3):
        np.testing.assert_allclose(res[0][q], ref[q], rtol=1e-12)
    for a, b in zip(res[0][3:], ref[3:]):
        assert np.array_equal(a, b)


@pytest.mark.parametrize("variant", ["two_pass", "two_pass_split", "fused"])
def test_the_end_of_a_step_stays_beside_its_kernels(variant):
    # a sequence's time a step within 1.4 times that of its field kernels (it was
    # 1.9 times and more while one workgroup summed a member's partials)
    sim = _sim((160, 160, 160), variant, 2, 1)
    sim.step(64)
    sim.sync()
    kernels = 1e30
    for _ in range(3):
        ms, steps = sim.step_timed(16)
        kernels = min(kernels, sum(ms) / steps)
    t = []
    for _ in range(3):
        t0 = time.perf_counter()
        sim.step(64)
        sim.sync()
        t.append((time.perf_counter() - t0) / 64 * 1e3)
    print(f"{variant}: {min(t) * 1e3:.1f} us a step, kernels {kernels * 1e3:.1f}")
    sim.close()
    assert min(t) <= 1.4 * kernels
