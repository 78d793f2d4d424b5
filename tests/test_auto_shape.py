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
