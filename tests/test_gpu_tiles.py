"""The single-pass tile kernel (16 x 4 columns a wave) at the edges of its
tiles, rows and segments: fields against the two passes bit for bit, and the
energy and loss sums, whose partials do not follow a kernel's workgroups."""
import numpy as np
import pytest

from paper_0809_1547_amd import inputs as I

pytestmark = pytest.mark.gpu


def _run(n, bc, precision, variant, tile_y, zseg, steps=37):
    from paper_0809_1547_amd import mbf
    eps, gain = I.voxelize(I.rsa_pack(n, seed=3, count=1, radius=0.3 * min(n)))
    sim = mbf.Sim(n, boundary=bc, precision=precision, seed=7, E_sp=1e-2, energy_history=steps)
    sim.set_tuning(variant, tile_y=tile_y, zseg=zseg, xcd_remap=2)
    sim.set_material(eps, gain)
    sim.set_pump(2e24)
    sim.set_source(2, n[0] // 2, n[1] // 2, n[2] // 2, amp=0.5)
    sim.set_loss_box((0, 0, 0), (max(1, n[0] - 1), n[1], n[2]))
    sim.set_plane_monitor(n[2] // 2)
    f = I.random_fields(n, seed=5, amplitude=1e-2)
    for c in range(3):
        sim.set_field(c, f[c])
    sim.step(steps)
    out = [sim.field(q) for q in range(21)]
    sums = [np.array(sim.energy()), np.array(sim.loss()), sim.energy_history(), sim.plane_monitor()[0]]
    one_kernel = sim.step_bytes()[2] == 0.0
    sim.close()
    return out, sums, one_kernel


# sides around the tile (16, 4), the workgroup (64) and the segment (zseg)
@pytest.mark.parametrize("n", [(2, 2, 2), (15, 3, 5), (16, 4, 2), (17, 5, 3), (63, 8, 4), (64, 9, 7), (65, 7, 9), (130, 6, 3)])
@pytest.mark.parametrize("bc,precision", [("pec", "fp32"), ("absorb", "fp32"), (("mur", "pec", "absorb"), "fp32"),
                                          ("absorb", "fp64")])
def test_tile_kernel_equals_the_two_passes(n, bc, precision):
    ref, ref_sums, one = _run(n, bc, precision, "two_pass_split", 4, 2)
    assert not one
    for variant, tile_y, zseg, same_sums in (("two_pass", 4, 2, True), ("fused", 8, 2, True), ("fused", 2, 2, True),
                                             ("fused_persistent", 16, 2, True), ("two_pass", 16, 3, False),
                                             ("fused", 4, 1, False)):
        got, sums, one = _run(n, bc, precision, variant, tile_y, zseg)
        assert one
        for q, (a, b) in enumerate(zip(ref, got)):
            assert np.array_equal(a, b), (variant, tile_y, zseg, q)
        assert np.array_equal(ref_sums[3], sums[3])
        if same_sums:
            for a, b in zip(ref_sums, sums):
                assert np.array_equal(a, b), (variant, tile_y, zseg)


def test_two_pass_schedule_leaves_the_tile_kernel_beyond_the_cache():
    # 136^3 (240 MB of state) takes one kernel, 144^3 (280 MB) two
    from paper_0809_1547_amd import mbf
    for n, want in ((136, True), (144, False)):
        eps, gain = I.homogeneous(n, 1.0, 1)
        gain[:, :, : int(0.4 * n)] = 0
        sim = mbf.Sim(n)
        sim.set_tuning("two_pass", tile_y=4, zseg=4)
        sim.set_material(eps, gain)
        sim.set_pump(2e24)
        assert (sim.step_bytes()[2] == 0.0) == want
        sim.set_tuning("two_pass", tile_y=2, zseg=4)
        assert sim.step_bytes()[2] > 0.0
        sim.step(2)
        sim.sync()
        sim.close()


# beyond the last-level cache: FP64 (one kernel), FP32 rows that fill 72 of 128
# lanes (one), rows that fill all of theirs (two, split from 300 MB on), a plane
# above 640 KB (two)
@pytest.mark.parametrize("n,precision,one", [((112, 116, 114), "fp64", True), ((72, 70, 1040), "fp32", True),
                                             ((64, 62, 1700), "fp32", False), ((140, 126, 290), "fp32", False)])
def test_two_pass_schedule_beyond_the_cache(n, precision, one):
    from paper_0809_1547_amd import mbf
    eps = np.full(n[::-1], 2.25, dtype=np.float32)
    gain = np.zeros(n[::-1], dtype=np.uint8)
    gain[:, :, 5:33] = 1
    res = []
    for variant in ("two_pass", "two_pass_split"):
        sim = mbf.Sim(n, boundary="absorb", precision=precision, seed=3, E_sp=1e-2, energy_history=33)
        sim.set_tuning(variant, tile_y=4, zseg=4)
        sim.set_material(eps, gain)
        sim.set_pump(2e24)
        sim.set_loss_box((3, 3, 3), (60, 50, 100))
        assert (sim.step_bytes()[2] == 0.0) == (one and variant == "two_pass")
        sim.step(33)
        res.append([sim.field(q) for q in (0, 1, 2, 3, 4, 5, 6, 13, 20)] + [sim.energy_history(), np.array(sim.loss())])
        sim.close()
    for a, b in zip(*res):
        assert np.array_equal(a, b)


# marches of several segments (grids that make 1800 waves at two and four planes,
# a last march and a last segment cut short): the sums stay the segments'
@pytest.mark.parametrize("n,precision", [((64, 48, 80), "fp64"), ((64, 64, 63), "fp32"), ((130, 90, 37), "fp32")])
@pytest.mark.parametrize("zseg", [1, 2, 3])
def test_marches_keep_the_segments_sums(n, precision, zseg):
    ref, ref_sums, _ = _run(n, "absorb", precision, "two_pass_split", 4, zseg, steps=9)
    got, sums, one = _run(n, "absorb", precision, "two_pass", 4, zseg, steps=9)
    assert one
    for a, b in zip(ref + ref_sums, got + sums):
        assert np.array_equal(a, b)
