"""The expectation workspace a state keeps: calls of growing and shrinking
term counts (beyond one launch's 4096 too) between changes of the state."""
import numpy as np
import pytest

import qsynth

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("dtype,tol", [(0, 1e-5), (1, 1e-12)])
def test_kept_workspace(oracle, dtype, tol):
    from paper_2509_04955_amd import qsim as Q

    n = 9
    st = Q.State(n, dtype)
    for i, terms in enumerate((3, 5000, 1, 300)):
        psi = qsynth.random_state(n, seed=i)
        ham = qsynth.random_pauli_sum(n, terms, seed=(i, 2))
        st.load(psi)
        e, t = st.expect(ham, with_terms=True)
        ref = np.array([oracle.expect_pauli_sum(psi, n, ham.x[k:k + 1], ham.z[k:k + 1], np.ones(1))
                        for k in range(0, terms, 17)])
        assert np.max(np.abs(t[::17] - ref)) <= tol
        assert abs(e - float(ham.coeff @ t)) <= 1e-12 * max(1.0, float(np.abs(ham.coeff) @ np.abs(t)))
    st.close()
