"""GPU: the Gross-Pitaevskii solver at the ends of its row layouts (4, 8 and
16 rows a lane, whole and partly filled lanes, fewer rows than lanes) and of
its spectrum tiles (64 frequencies, eight solutions), against the oracle."""
import numpy as np
import pytest

from oracle import gp as OG

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("M,n_nu", [(3, 1), (5, 63), (64, 64), (65, 65), (255, 128), (256, 129), (257, 40), (511, 64),
                                    (512, 64), (513, 64), (1009, 64), (1023, 64)])
def test_row_layouts_match_oracle(M, n_nu):
    from paper_0809_1547_amd import mbf
    L = 4.0 if M < 16 else 9.0
    # three bound states spread over 33 solutions (a whole tile and one more)
    Es = [[1.3, 2.5, 6.0][q % 3] if M >= 16 else [9.0, 11.0, 15.0][q % 3] for q in range(33)]
    g = mbf.mbf_gp_solve(Es, M=M, L=L, n_nu=n_nu, dnu=0.03)
    for q in range(3):
        o = OG.gp_solve(Es[q], M, L, n_nu, 0.03)
        scale = float(np.max(np.abs(o["phi"])))
        for r in range(q, 33, 3):
            assert g["converged"][r] == 1.0
            assert np.max(np.abs(g["phi"][r] - o["phi"])) <= 1e-9 * scale
            assert np.max(np.abs(g["spec"][r] - o["spec"])) <= 1e-9 * float(np.max(o["spec"]))
            # equal inputs, equal bits wherever they lie in the batch
            assert np.array_equal(g["phi"][r], g["phi"][q]) and np.array_equal(g["spec"][r], g["spec"][q])
            for key in ("N", "peak", "phi_max"):
                assert g[key][r] == pytest.approx(o[key], rel=1e-9)
