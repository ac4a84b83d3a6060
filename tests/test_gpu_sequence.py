"""GPU: steps queued as sequences (each step ended in the next one's launch)
against the same steps one by one (each with a launch to end it): fields,
spectra, source, loss and the energy of every step bit for bit, at sequence
lengths around their longest (32), probe decimations that split them, and
workgroups of 2, 4, 8 and 16 rows."""
import numpy as np
import pytest

from paper_0809_1547_amd import inputs as I

pytestmark = pytest.mark.gpu

N = (37, 22, 19)
STEPS = 101


def _configure(sim, decim, source):
    from paper_0809_1547_amd import mbf
    eps, gain = I.voxelize(I.rsa_pack(N, seed=3, count=1, radius=5.0))
    sim.set_material(eps, gain)
    sim.set_pump(2e24)
    if source:
        sim.set_source(1, 9, 11, 8, amp=0.3, tau_p=2e-16, t0=6e-16)
    sim.set_loss_box((1, 2, 3), (30, 17, 15))
    if decim:
        dt = sim.coefficients()[mbf.MBF_C_DT]
        sim.set_probes(I.select_probes(eps, gain, 70, seed=1), I.dft_omegas(450e-9, 800e-9, 400, dt)[:9], decim=decim)


def _results(sim, decim):
    return [sim.field(q) for q in range(21)] + [np.array(sim.energy()), np.array(sim.loss()), sim.energy_history()] + (
        [sim.spectrum()] if decim else [])


@pytest.mark.parametrize("variant,tile_y", [("two_pass", 4), ("two_pass", 2), ("two_pass_split", 8), ("fused", 2),
                                            ("fused", 16), ("fused_lds", 4), ("fused_persistent", 8)])
@pytest.mark.parametrize("precision,decim,source", [("fp32", 0, True), ("fp32", 40, True), ("fp64", 7, False)])
def test_sequences_equal_single_steps(variant, tile_y, precision, decim, source):
    from paper_0809_1547_amd import mbf
    kw = dict(boundary=("mur", "pec", "absorb"), precision=precision, seed=5, E_sp=1e-2, energy_history=STEPS)
    one = mbf.Sim(N, **kw)
    one.set_tuning(variant, tile_y=tile_y, zseg=2)
    _configure(one, decim, source)
    one.step_timed(STEPS)                        # a launch ends each step
    ref = _results(one, decim)
    one.close()
    # graphs and remainders; sequences of 1, 31, 32 and 33 steps; a batch whose
    # other member has other probes
    for parts in ((STEPS,), (1, 31, 32, 33, 4)):
        sim = mbf.Sim(N, **kw)
        sim.set_tuning(variant, tile_y=tile_y, zseg=2)
        _configure(sim, decim, source)
        for p in parts:
            sim.step(p)
        for q, (a, b) in enumerate(zip(ref, _results(sim, decim))):
            assert np.array_equal(a, b), (parts, q)
        sim.close()
    batch = mbf.Batch([mbf.make_config(N, **kw), mbf.make_config(N, **kw)])
    batch.set_tuning(variant, tile_y=tile_y, zseg=2)
    _configure(batch[0], decim, source)
    _configure(batch[1], 12, source)
    batch.step(STEPS)
    for q, (a, b) in enumerate(zip(ref, _results(batch[0], decim))):
        assert np.array_equal(a, b), ("batch", q)
    batch.close()
