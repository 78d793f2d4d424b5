"""Tile passes at the edges of their launch choices: one tile, a workgroup per
tile up to the resident count, more tiles than that, and norms summed by the
next pass or by a reduction of their own."""
import numpy as np
import pytest

import qsynth

pytestmark = pytest.mark.gpu

TOL = {0: 1e-5, 1: 1e-12}   # as for every parity test


@pytest.fixture(scope="module")
def Q():
    import torch

    from paper_2509_04955_amd import qsim

    assert torch.cuda.is_available()
    qsim.lib()
    return qsim


@pytest.mark.parametrize("renorm", [0, 1])
@pytest.mark.parametrize("dtype,n,k,t", [
    (0, 6, 3, 13), (0, 13, 5, 13), (0, 14, 5, 13), (0, 15, 4, 14), (0, 14, 6, 12), (0, 12, 2, 4), (0, 17, 3, 8),
    (0, 20, 3, 9), (0, 21, 3, 9), (0, 22, 4, 13), (0, 23, 4, 13),
    (1, 6, 3, 12), (1, 13, 5, 12), (1, 13, 3, 12), (1, 14, 5, 11), (1, 16, 2, 7), (1, 20, 3, 8), (1, 21, 3, 12),
    (1, 22, 3, 12),
    # staged passes: lean (blocks of up to 3 or 4 qubits at 2^12) and general ones, resident and not
    (0, 18, 3, 12), (0, 18, 4, 12), (0, 18, 5, 12), (0, 23, 3, 12), (0, 16, 5, 11), (0, 21, 5, 13),
    (1, 18, 3, 12), (1, 16, 4, 11), (1, 16, 5, 12),
])
def test_pass_chain(Q, oracle, dtype, n, k, t, renorm):
    """A plan applied twice to a random state of norm 3 (renorm: the chain of
    scales brings it to norm 1) against the oracle's state."""
    c = qsynth.random_u3_cnot(n, 2, seed=n)
    psi0 = qsynth.random_state(n, 5)
    plan = Q.qs_contract(n, Q.GateList(c), Q.opts(k_max=k, tile_qubits=t, low_qubits=3, dtype=dtype, renorm=renorm))
    assert Q.qs_plan_info_get(plan).n_passes > (0 if t >= n else 1)
    st = Q.State(n, dtype)
    st.load(3.0 * psi0)
    st.apply_plan(plan)
    st.apply_plan(plan)
    got = st.amplitudes()
    norm = st.norm()
    st.close()
    Q.qs_plan_destroy(plan)
    ref = oracle.run(c, oracle.run(c, psi0)) * (1.0 if renorm else 3.0)
    assert oracle.max_abs(ref, got) <= TOL[dtype] * (1 if renorm else 3)
    assert abs(norm - (1.0 if renorm else 9.0)) <= 100 * TOL[dtype]


@pytest.mark.parametrize("k,low", [(3, 4), (4, 6)])
def test_staged_passes_light_and_heavy(Q, oracle, k, low):
    """Staged complex64 passes on more tiles than fit at once, where the
    number of blocks picks the variant: plans with passes on both sides."""
    n = 23
    c = qsynth.brickwork(n, 4, seed=k)
    plan = Q.qs_contract(n, Q.GateList(c), Q.opts(k_max=k, tile_qubits=12, low_qubits=low, dtype=0))
    counts = [Q.qs_plan_pass(plan, i)[3] for i in range(Q.qs_plan_info_get(plan).n_passes)]
    assert min(counts) < 4 and (k == 4 or max(counts) > 4)
    psi0 = qsynth.random_state(n, 5)
    st = Q.State(n, 0)
    st.load(psi0)
    st.apply_plan(plan)
    got = st.amplitudes()
    st.close()
    Q.qs_plan_destroy(plan)
    assert oracle.max_abs(oracle.run(c, psi0), got) <= TOL[0]


def test_captured_small_plan_replays(Q):
    """A plan whose passes give every tile a workgroup draws no tickets, so a
    captured launch can be replayed: each replay, with eager work between,
    equals an eager call bit for bit."""
    import torch

    n = 16
    gl = Q.GateList(qsynth.hea(n, 3, seed=(1, n)))
    s = torch.cuda.Stream()
    with torch.cuda.stream(s):
        st, ref = Q.State(n, 0), Q.State(n, 0)
        plan = Q.qs_contract(n, gl, Q.opts(k_max=4, tile_qubits=12, low_qubits=4))
        ref.apply_plan(plan)   # uploads the plan and sizes ref's partials
        st.apply_plan(plan)
        g = torch.cuda.CUDAGraph()
        with torch.cuda.graph(g, stream=s):
            st.apply_plan(plan)
        for _ in range(3):
            g.replay()
            ref.apply_plan(plan)
            s.synchronize()
            assert torch.equal(torch.view_as_real(st.tensor), torch.view_as_real(ref.tensor))
    st.close()
    ref.close()
    Q.qs_plan_destroy(plan)
