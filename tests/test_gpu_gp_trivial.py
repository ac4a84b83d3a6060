"""GPU: eigenvalues below the lowest one of the box, which has only the trivial
state then: zero, and converged."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("M", [3, 33, 64, 101, 255, 600, 1023])
@pytest.mark.parametrize("L,E", [(0.3, [5.0, 12.0]), (1.0, [1.00001, 1.05, 1.5]), (2.0, [1.00001, 1.05])])
def test_no_bound_state_in_the_box(M, L, E):
    from paper_0809_1547_amd import mbf
    h = 2 * L / (M + 1)
    tau = -L + h * np.arange(1, M + 1)
    A = np.diag(2 / h ** 2 + tau * tau) - np.diag(np.full(M - 1, 1 / h ** 2), 1) - np.diag(np.full(M - 1, 1 / h ** 2), -1)
    E = [e for e in E if e < np.linalg.eigvalsh(A)[0]]
    if not E:
        pytest.skip("the coarse box has a bound state")
    g = mbf.mbf_gp_solve(E, M=M, L=L, n_nu=5, dnu=0.1)
    assert np.all(g["converged"] == 1.0) and np.all(g["phi"] == 0.0) and np.all(g["N"] == 0.0) and np.all(g["spec"] == 0.0)


@pytest.mark.parametrize("M,L", [(101, 8.0), (255, 14.0), (1023, 30.0)])
def test_a_missed_bound_state_is_not_called_converged(M, L):
    # just above threshold the flow from the Gaussian may decay although the box
    # has a bound state
    from paper_0809_1547_amd import mbf
    g = mbf.mbf_gp_solve([1.00001, 3.0], M=M, L=L, n_nu=5, dnu=0.1)
    assert g["converged"][0] == 0.0 or g["phi_max"][0] > 1e-6
    assert g["converged"][1] == 1.0 and g["phi_max"][1] > 1.0
