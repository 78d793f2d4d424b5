"""Plans whose tile and low qubits are left to the library: every size, width
and dtype gives a valid plan, and any fixed low-qubit count that fits the
largest tile is accepted with it (host only)."""
import pytest

import qsynth
from paper_2509_04955_amd import qsim as Q


def _passes(n, gl, o):
    p = Q.qs_contract(n, gl, o)
    info = Q.qs_plan_info_get(p)
    blocks = [Q.qs_plan_block(p, b, with_matrix=False)[0] for b in range(info.n_blocks)]
    members = sum(len(Q.qs_plan_block(p, b, with_matrix=False)[2]) for b in range(info.n_blocks))
    passes = [Q.qs_plan_pass(p, i) for i in range(info.n_passes)]
    Q.qs_plan_destroy(p)
    for t, tile, first, count in passes:
        assert t == len(tile) <= n and tile[0] == 0
        assert all(set(blocks[b]) <= set(tile) for b in range(first, first + count))
    return members, passes


@pytest.mark.parametrize("dtype,cap", [(Q.QS_C64, 13), (Q.QS_C128, 12)])
@pytest.mark.parametrize("n", list(range(1, 27)) + [30, 33, 40])
def test_auto_shapes(n, dtype, cap):
    c = qsynth.random_circuit(n, 60, seed=n)
    if n >= 6:   # the widest dense gate a complex64 plan takes (complex128: 5)
        w = 6 if dtype == Q.QS_C64 else 5
        c.gates += [g for g in qsynth.random_circuit(n, 40, seed=1, max_dense=w).gates if g.name == "dense"]
    gl = Q.GateList(c)
    for k in (0, 1, 2, 3, 4, 5):
        members, passes = _passes(n, gl, Q.opts(k_max=k, dtype=dtype))
        assert members == len(c)
        assert all(t <= cap for t, *_ in passes)
    for low in range(1, cap + 1):
        members, _ = _passes(n, gl, Q.opts(k_max=3, low_qubits=low, dtype=dtype))
        assert members == len(c)
    with pytest.raises(Q.QsimError):
        Q.qs_contract(n, gl, Q.opts(low_qubits=cap + 1, dtype=dtype))


def _shape(n, gl, **kw):
    p = Q.qs_contract(n, gl, Q.opts(**kw))
    t, tile, _, _ = Q.qs_plan_pass(p, 0)
    Q.qs_plan_destroy(p)
    return t, tile


@pytest.mark.parametrize("dtype,cap", [(Q.QS_C64, 13), (Q.QS_C128, 12)])
@pytest.mark.parametrize("n", [8, 12, 13, 14, 16, 18, 20, 23, 26])
def test_given_low_qubits_take_the_usual_tile(n, dtype, cap):
    """With the low qubits given, an open tile has 13 qubits (complex128: 12),
    whatever the size of the state."""
    gl = Q.GateList(qsynth.hea(n, 2, seed=(1, n)))
    for low in range(1, 9):
        for k in (0, 3, 4):
            t, tile = _shape(n, gl, k_max=k, low_qubits=low, dtype=dtype)
            assert t == min(cap, n)
            assert list(tile[:min(low, t - (k or 5))]) == list(range(min(low, t - (k or 5))))


@pytest.mark.parametrize("dtype,one", [(Q.QS_C64, 13), (Q.QS_C128, 12)])
def test_open_shapes_follow_the_plan(dtype, one):
    """Plans of rotations keep small states in one tile and complex128 states of
    24 qubits in 2^12 tiles, where 5-qubit blocks and single gates take 2^11;
    the rotation strategy on a circuit without such rotations is a plan of
    blocks."""
    c64 = dtype == Q.QS_C64
    for n in range(9, one + 1):
        gl = Q.GateList(qsynth.ucc(n, n_exp=6, wmax=min(8, n), seed=n)[0])
        assert _shape(n, gl, strategy=Q.STRATEGY_PAULI, dtype=dtype)[0] == n
    gl = Q.GateList(qsynth.ucc(24, n_exp=6, wmax=8, seed=24)[0])
    assert _shape(24, gl, strategy=Q.STRATEGY_PAULI, dtype=dtype)[0] == (13 if c64 else 12)
    for strategy in (Q.STRATEGY_NONE, Q.STRATEGY_GREEDY):
        assert _shape(24, gl, strategy=strategy, dtype=dtype)[0] == (13 if c64 else 11)
    for n in (13, 24):
        gl = Q.GateList(qsynth.qaoa_maxcut(n, 2, seed=(1, n)))
        assert (_shape(n, gl, strategy=Q.STRATEGY_PAULI, dtype=dtype)[0] == _shape(n, gl, dtype=dtype)[0]
                == {13: 10, 24: 13 if c64 else 11}[n])
