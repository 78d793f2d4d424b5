"""Gate lists (qs_apply_gates) at the edges of their runs: tile and state
sizes, controls inside and outside a tile, gates that take sweeps of their own,
full record and stage tables, and capture."""
import numpy as np
import pytest

import qsynth

pytestmark = pytest.mark.gpu

TOL = {0: 1e-5, 1: 1e-12}   # as for every parity test: rounding of a few hundred updates


@pytest.fixture(scope="module")
def Q():
    import torch

    from paper_2509_04955_amd import qsim

    assert torch.cuda.is_available()
    qsim.lib()
    return qsim


def _check(Q, oracle, c, dtype, seed=1):
    psi0 = qsynth.random_state(c.n, seed)
    st = Q.State(c.n, dtype)
    st.load(psi0)
    st.apply_gates(Q.GateList(c))
    got = st.amplitudes()
    st.close()
    ref = oracle.run(c, psi0)
    assert oracle.max_abs(ref, got) <= TOL[dtype], c.n


@pytest.mark.parametrize("dtype", [0, 1])
@pytest.mark.parametrize("n,gates", [(2, 20), (3, 40), (4, 120), (5, 300), (9, 200), (10, 200), (11, 250), (13, 250),
                                     (16, 200), (20, 60), (21, 50), (22, 40)])
def test_lists_of_every_kind(Q, oracle, n, gates, dtype):
    """Every gate kind, dense gates of up to three qubits between them, at
    state sizes on both sides of each tile and register choice."""
    _check(Q, oracle, qsynth.random_circuit(n, gates, seed=n, max_dense=min(3, n)), dtype)


@pytest.mark.parametrize("dtype", [0, 1])
@pytest.mark.parametrize("n", [6, 12])
def test_full_tables(Q, oracle, n, dtype):
    """More gates than a run's records hold, and more stages than its table
    (a SWAP fills a two-qubit stage by itself): the rest goes to later runs."""
    _check(Q, oracle, qsynth.random_circuit(n, 300, seed=3, kinds=["swap", "h"]), dtype)
    _check(Q, oracle, qsynth.random_circuit(n, 300, seed=4, kinds=["u3", "cu"]), dtype)


def test_identity_and_far_controls(Q, oracle):
    """Identity phases vanish; controls and phases on the highest qubits with
    targets on the lowest lie outside every tile."""
    n = 16
    c = qsynth.Circuit(n)
    for q in range(4):
        c.add("h", (q,))
    for q in range(12, 16):
        c.add("ry", (q,), (0.3 + q,))
    for q in range(4):
        c.add("p", (q,), (0.0,)).add("cx", (12 + q, q)).add("cp", (15 - q, q), (0.7,)).add("cz", (12 + q, 15 - q) if
                                                                                           q in (0, 1) else (q, 14))
        c.add("rz", (12 + q,), (0.2 * q + 0.1,)).add("cu", (q, 12 + q), (0.4, 0.5, 0.6))
    for dtype in (0, 1):
        _check(Q, oracle, c, dtype)


def test_captured_list_replays(Q):
    """A gate list captured on the state's stream, replayed with eager work
    between the replays, gives what eager calls give, bit for bit."""
    import torch

    c = qsynth.random_circuit(13, 150, seed=8)
    gl = Q.GateList(c)
    s = torch.cuda.Stream()
    with torch.cuda.stream(s):
        st, ref = Q.State(13, 0), Q.State(13, 0)
        g = torch.cuda.CUDAGraph()
        with torch.cuda.graph(g, stream=s):
            st.apply_gates(gl)
        st.set_basis(5)
        ref.set_basis(5)
        for _ in range(3):
            g.replay()
            ref.apply_gates(gl)
            s.synchronize()
            assert torch.equal(torch.view_as_real(st.tensor), torch.view_as_real(ref.tensor))
    st.close()
    ref.close()


@pytest.mark.parametrize("dtype", [0, 1])
@pytest.mark.parametrize("n", [21, 22, 23])
def test_two_light_gates(Q, oracle, n, dtype):
    """Lists of two to four gates that move half of the state or less each: as
    sweeps or as a run, on near and far qubits."""
    for kinds in (("swap", "swap"), ("swap", "cx"), ("p", "cu"), ("cz",) * 4):
        for b in (0, n - 8):
            c = qsynth.Circuit(n)
            for i, k in enumerate(kinds):
                q = (b + 2 * i, b + 2 * i + 1)
                c.add(k, q if k != "p" else q[:1], {"p": (0.4,), "cu": (0.1, 0.2, 0.3)}.get(k, ()))
            _check(Q, oracle, c, dtype, seed=n)
