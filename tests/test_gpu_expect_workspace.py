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


@pytest.mark.parametrize("dtype", [0, 1])
def test_threads_read_one_state(dtype):
    """Threads that read energies of one state at once, each with its own
    Hamiltonian and with sums that make the workspace grow between theirs, get
    what one thread alone gets, bit for bit."""
    import threading

    import torch

    from paper_2509_04955_amd import qsim as Q

    n = 15
    st = Q.State(n, dtype)
    st.load(qsynth.random_state(n, seed=3))
    hams = [[qsynth.random_pauli_sum(n, terms, seed=(w, terms)) for terms in (5 + w, 90 + 40 * w, 700 + 900 * w)]
            for w in range(3)]
    ref = Q.State(n, dtype)
    ref.load(qsynth.random_state(n, seed=3))
    want = [[ref.expect(h, with_terms=True) for h in hs] for hs in hams]
    wrong = []

    def read(w):
        torch.cuda.set_device(0)
        for _ in range(10):
            for h, (e0, t0) in zip(hams[w], want[w]):
                e, t = st.expect(h, with_terms=True)
                if e != e0 or not np.array_equal(t, t0):
                    wrong.append((w, len(h.coeff), e, e0))

    threads = [threading.Thread(target=read, args=(w,)) for w in range(3)]
    for t in threads:
        t.start()
    for t in threads:
        t.join()
    st.close()
    ref.close()
    assert not wrong, wrong[:4]
