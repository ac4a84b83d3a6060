"""GPU: packing steps whose cells hold as many centres as the two read paths of
a list meet at (eight, nine) and the most a cell may hold (32), against the
oracle's all-pairs forces."""
import numpy as np
import pytest

import oracle as O

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("per_cell", [1, 7, 8, 9, 32])
def test_crowded_cells_match_oracle(per_cell):
    from paper_0809_1547_amd import mbf
    # one sphere of diameter 10 makes cells 10 wide; small ones crowd four of them
    rng = np.random.default_rng(per_cell)
    box = np.array([40.0, 30.0, 20.0])
    x = [np.array([[35.0, 25.0, 15.0]])]
    for corner in ((0, 0, 0), (10, 0, 0), (0, 10, 0), (10, 10, 10)):
        x.append(np.array(corner) + 2.0 + 6.0 * rng.random((per_cell, 3)))
    x = np.concatenate(x)
    x = np.concatenate([x[:1], x[1:][rng.permutation(len(x) - 1)]])
    d = np.concatenate([[10.0], 1.5 + rng.random(len(x) - 1)])
    kw = dict(s0=0.8, stages=2, iters=2, final_iters=4, eta=0.05)
    got, U, ov = mbf.mbf_pack_md(box, d, x, **kw)
    want = O.pack_md(box, d, x, **kw)
    Uo, ovo = O.pack_energy(box, d, want)
    # eight steps of rounding-sized differences at coordinates of order the box
    assert np.max(np.abs(got - want)) <= 1e-12 * 40.0
    assert abs(U - Uo) <= 1e-9 * max(Uo, 1e-300) and abs(ov - ovo) <= 1e-9 * max(ovo, 1e-300)
    again, U2, _ = mbf.mbf_pack_md(box, d, x, **kw)
    assert np.array_equal(got, again) and U == U2
