"""GPU: the two whole passes where the two-pass schedule takes them: at two rows
always (in FP64 and at any size), and at more rows between the cache and the
split passes; against other kernels, fields bit for bit."""
import numpy as np
import pytest

from paper_0809_1547_amd import inputs as I

pytestmark = pytest.mark.gpu


def _run(n, bc, precision, schedule, steps, columns=None):
    from paper_0809_1547_amd import mbf
    if columns is None:
        eps, gain = I.voxelize(I.rsa_pack(n, seed=3, count=1, radius=0.3 * min(n)))
    else:
        eps = np.full(n[::-1], 2.25, dtype=np.float32)
        gain = np.zeros(n[::-1], dtype=np.uint8)
        gain[:, :, 5:5 + columns] = 1
    sim = mbf.Sim(n, boundary=bc, precision=precision, seed=7, E_sp=1e-2, energy_history=steps)
    sim.set_tuning(*schedule)
    sim.set_material(eps, gain)
    sim.set_pump(2e24)
    sim.set_source(2, n[0] // 2, n[1] // 2, n[2] // 2, amp=0.5)
    sim.set_loss_box((0, 0, 0), (max(1, n[0] - 1), n[1], n[2]))
    two = sim.step_bytes()[2] > 0.0
    sim.step(steps)
    fields = [sim.field(q) for q in (range(21) if columns is None else (0, 1, 2, 3, 4, 5, 6, 13, 20))]
    sums = [np.array(sim.energy()), np.array(sim.loss()), sim.energy_history()]
    sim.close()
    return fields, sums, two


@pytest.mark.parametrize("n", [(2, 2, 2), (15, 3, 5), (63, 8, 4), (65, 7, 9), (130, 6, 3)])
@pytest.mark.parametrize("bc,precision", [("pec", "fp64"), ("absorb", "fp64"), (("mur", "pec", "absorb"), "fp64"),
                                          (("mur", "pec", "absorb"), "fp32")])
def test_whole_passes_of_two_rows_equal_tiles(n, bc, precision):
    a, _, two = _run(n, bc, precision, ("two_pass", 2, 2), 37)
    assert two
    b, _, two = _run(n, bc, precision, ("fused", 4, 2), 37)
    assert not two
    for x, y in zip(a, b):
        assert np.array_equal(x, y)


# 275 MB of state: between the cache (250) and the split passes (300)
@pytest.mark.parametrize("tile_y", [4, 8, 16])
def test_whole_passes_between_cache_and_split(tile_y):
    n = (128, 142, 150)
    a, sa, two = _run(n, "absorb", "fp32", ("two_pass", tile_y, 4), 33, columns=83)
    assert two
    b, sb, _ = _run(n, "absorb", "fp32", ("fused", tile_y, 4), 33, columns=83)
    for x, y in zip(a + sa, b + sb):
        assert np.array_equal(x, y)


# beyond 300 MB: at two rows whole, as the caller asked
@pytest.mark.parametrize("n,precision", [((128, 150, 160), "fp32"), ((112, 116, 114), "fp64")])
def test_two_rows_stay_whole_beyond_the_cache(n, precision):
    a, sa, two = _run(n, "absorb", precision, ("two_pass", 2, 4), 33, columns=100)
    assert two
    for schedule in (("two_pass_split", 2, 4), ("fused", 4, 4)):
        b, sb, _ = _run(n, "absorb", precision, schedule, 33, columns=100)
        for x, y in zip(a, b):
            assert np.array_equal(x, y)
        if schedule[0] == "two_pass_split":
            for x, y in zip(sa, sb):
                assert np.array_equal(x, y)
