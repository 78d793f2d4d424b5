"""GPU parity of the batched path (one hipGraph launch): every
state's energy and amplitudes against the FP64 oracle, for uneven qubit
counts, repeated launches (determinism) and the autotuned plan choice."""
import numpy as np
import pytest

import qsynth

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def Q():
    import torch

    from paper_2509_04955_amd import qsim

    assert torch.cuda.is_available()
    qsim.lib()
    return qsim


def _oracle_energy(oracle, c, h):
    psi = oracle.run(c)
    return psi, oracle.expect_pauli_sum(psi, c.n, h.x, h.z, h.coeff)


@pytest.mark.parametrize("dtype,tol", [(0, 1e-6), (1, 1e-12)])
def test_batch_small_uneven(Q, oracle, dtype, tol):
    """24 HEA states with 3..15 qubits (several passes for the larger ones
    at a 10-qubit tile), 8 layers RY/RZ + CZ ring, 30-term Pauli sums."""
    circuits, hams = qsynth.hea_batch(24, 3, 15, layers=8, n_terms=30, seed=7)
    b = Q.Batch(circuits, hams, Q.opts(k_max=3, tile_qubits=10, dtype=dtype))
    E1 = b.run()
    E2 = b.run()
    assert np.array_equal(E1, E2), "repeated launches must agree bitwise"
    for i, (c, h) in enumerate(zip(circuits, hams)):
        psi, e = _oracle_energy(oracle, c, h)
        assert abs(E1[i] - e) <= tol * max(1, abs(e)), (i, c.n, E1[i], e)
        amps = b.amplitudes(i)
        assert oracle.max_abs(psi, amps) <= (1e-5 if dtype == 0 else 1e-12)
    b.close()


def test_batch_mixed_block_kinds(Q, oracle):
    """k_max = 5 (MFMA blocks) and monomial blocks together in one batch."""
    circuits = [qsynth.random_circuit(n, 120, seed=n, max_dense=2) for n in (6, 9, 12, 14, 16)]
    hams = [qsynth.random_pauli_sum(c.n, 12, seed=(3, c.n)) for c in circuits]
    b = Q.Batch(circuits, hams, Q.opts(k_max=5, tile_qubits=11))
    E = b.run()
    for i, (c, h) in enumerate(zip(circuits, hams)):
        psi, e = _oracle_energy(oracle, c, h)
        assert abs(E[i] - e) <= 1e-5
        assert 1 - oracle.fidelity(psi, b.amplitudes(i)) <= 1e-6
    b.close()


@pytest.mark.parametrize("dtype,tol", [(0, 1e-5), (1, 1e-12)])
def test_batch_pauli_rotation_plans(Q, oracle, dtype, tol):
    """UCC states of 10..16 qubits under the Pauli-rotation contraction in the
    batch kernel: rotation blocks, grouped rotations and their per-tile signs
    (Z parts outside the tile) go through the same block dispatch."""
    circuits = [qsynth.ucc(n, n_exp=25, seed=40 + n)[0] for n in (10, 12, 13, 16)]
    hams = [qsynth.random_pauli_sum(c.n, 16, seed=(5, c.n)) for c in circuits]
    b = Q.Batch(circuits, hams, Q.opts(k_max=4, tile_qubits=10, dtype=dtype, strategy=Q.STRATEGY_PAULI))
    E = b.run()
    for i, (c, h) in enumerate(zip(circuits, hams)):
        psi, e = _oracle_energy(oracle, c, h)
        assert abs(E[i] - e) <= tol * max(1, abs(e)), (i, c.n, E[i], e)
        assert oracle.max_abs(psi, b.amplitudes(i)) <= tol
    b.close()


def test_batch_autotuned(Q, oracle):
    """k_max = 0 asks the autotuner for every distinct qubit count."""
    circuits, hams = qsynth.hea_batch(10, 12, 17, layers=8, n_terms=20, seed=9)
    b = Q.Batch(circuits, hams, Q.opts(k_max=0, tile_qubits=0))
    E = b.run()
    for i, (c, h) in enumerate(zip(circuits, hams)):
        _, e = _oracle_energy(oracle, c, h)
        assert abs(E[i] - e) <= 1e-5
    b.close()


def test_autotune_returns_valid_choice(Q):
    c = qsynth.brickwork(16, depth=6, seed=1)
    gl = Q.GateList(c)
    best = Q.qs_autotune(16, Q.QS_C64, gl)
    assert 2 <= best.k_max <= 5 and 11 <= best.tile_qubits <= 13
    again = Q.qs_autotune(16, Q.QS_C64, gl)
    assert (again.k_max, again.tile_qubits) == (best.k_max, best.tile_qubits)


def test_batch_rejects_bad_input(Q):
    c = qsynth.hea(5, 1, seed=(1, 1))
    h = qsynth.random_pauli_sum(6, 3, seed=(1, 2))  # acts on qubit 5 of a 5-qubit state
    with pytest.raises(Q.QsimError):
        Q.Batch([c], [h], Q.opts(k_max=2, tile_qubits=5))


@pytest.mark.parametrize("dtype,tol", [(0, 1e-6), (1, 1e-12)])
def test_batch_item_and_coset_edges(Q, oracle, dtype, tol):
    """Levels and energy items at their edges: one-qubit states, states just
    below and at a full expectation coset (14 qubits complex64, 13 complex128),
    and a pass of 2^13 four-qubit tiles, whose items hold several tiles.
    Tolerances as for the uneven batch above."""
    ns = (1, 2, 5, 12, 13, 14, 15, 17)
    circuits = [qsynth.random_circuit(n, 40, seed=60 + n) for n in ns]
    hams = [qsynth.random_pauli_sum(n, 1 + 5 * i, seed=(6, n)) for i, n in enumerate(ns)]
    b = Q.Batch(circuits, hams, Q.opts(k_max=2, tile_qubits=4, low_qubits=2, dtype=dtype))
    E = b.run()
    assert np.array_equal(E, b.run())
    for i, (c, h) in enumerate(zip(circuits, hams)):
        psi, e = _oracle_energy(oracle, c, h)
        assert abs(E[i] - e) <= tol * max(1, abs(e)), (i, c.n, E[i], e)
        assert oracle.max_abs(psi, b.amplitudes(i)) <= (1e-5 if dtype == 0 else 1e-12)
    b.close()


def test_batch_more_energy_items_than_one_grid(Q):
    """A 26-qubit complex128 state with 65536 terms has 2^22 energy items and
    more, of 1024 threads each, where a grid holds fewer than 2^32 threads.
    The state is a product of RY rotations and the terms have X and Z letters,
    so every expectation is a product of sines and cosines.  Rounding: 2^26
    summands of at most 2^-26 in FP64 give each term to about 1e-14."""
    n, terms = 26, 65536
    rng = np.random.default_rng(12)
    theta = rng.uniform(0.5, 1.0, size=n)
    c = qsynth.Circuit(n)
    for q in range(n):
        c.add("ry", (q,), (theta[q],))
    letters = rng.integers(0, 3, size=(terms, n))   # I, X, Z
    bits = (np.uint64(1) << np.arange(n, dtype=np.uint64))
    x = ((letters == 1) * bits).sum(axis=1, dtype=np.uint64)
    z = ((letters == 2) * bits).sum(axis=1, dtype=np.uint64)
    want = np.prod(np.where(letters == 1, np.sin(theta), np.where(letters == 2, np.cos(theta), 1.0)), axis=1)
    coeff = rng.normal(size=terms)
    b = Q.Batch([c], [qsynth.PauliSum(n, x, z, coeff)], Q.opts(k_max=3, tile_qubits=12, low_qubits=4, dtype=1))
    e = b.run()[0]
    b.close()
    assert abs(e - coeff @ want) <= 1e-13 * np.abs(coeff).sum()


def test_batch_more_pass_items_than_one_launch(Q):
    """600 states of 19 qubits in four-qubit tiles: 2048 items each, more in a
    level than one launch takes."""
    n, states = 19, 600
    theta = np.linspace(0.2, 2.9, states)
    circuits = [qsynth.Circuit(n).add("ry", (i % n,), (theta[i],)) for i in range(states)]
    hams = [qsynth.PauliSum(n, np.zeros(1, np.uint64), np.array([1 << (i % n)], np.uint64), np.ones(1))
            for i in range(states)]
    b = Q.Batch(circuits, hams, Q.opts(k_max=1, tile_qubits=4, low_qubits=2))
    e = b.run()
    assert np.max(np.abs(e - np.cos(theta))) <= 1e-6
    for i in (0, 511, 512, states - 1):
        want = np.zeros(1 << n, dtype=np.complex128)
        want[0], want[1 << (i % n)] = np.cos(theta[i] / 2), np.sin(theta[i] / 2)
        assert np.max(np.abs(b.amplitudes(i) - want)) <= 1e-6
    b.close()


def test_batch_tiles_of_several_sizes(Q, oracle):
    """A batch keeps its LDS room when one with smaller tiles is made after it."""
    circuits = [qsynth.hea(n, 3, seed=(8, n)) for n in (14, 15)]
    hams = [qsynth.random_pauli_sum(c.n, 10, seed=(8, c.n)) for c in circuits]
    batches = [Q.Batch(circuits, hams, Q.opts(k_max=3, tile_qubits=t, low_qubits=4)) for t in (14, 13, 10)]
    want = [_oracle_energy(oracle, c, h)[1] for c, h in zip(circuits, hams)]
    for b in batches:
        assert np.max(np.abs(b.run() - want)) <= 1e-5
        b.close()


def test_batch_holds_its_operands_once(Q):
    """Device memory of a batch: one copy of the operands of all plans.  40
    six-qubit dense gates in each of 20 states are 800 blocks of 64 KiB (the
    128 x 128 real form), 52 MB; the states and tables are below 4 MB."""
    import torch

    rng = np.random.default_rng(3)
    u, _ = np.linalg.qr(rng.normal(size=(64, 64)) + 1j * rng.normal(size=(64, 64)))
    n, states, gates = 11, 20, 40
    circuits = []
    for i in range(states):
        c = qsynth.Circuit(n)
        for _ in range(gates):
            c.add("dense", tuple(int(q) for q in rng.permutation(n)[:6]), matrix=u)
        circuits.append(c)
    hams = [qsynth.random_pauli_sum(n, 2, seed=(4, i)) for i in range(states)]
    o = Q.opts(k_max=6, tile_qubits=11, low_qubits=2, strategy=Q.STRATEGY_NONE)
    Q.Batch(circuits[:1], hams[:1], o).close()   # the first use of the kernels
    free0, _ = torch.cuda.mem_get_info()
    b = Q.Batch(circuits, hams, o)
    used = free0 - torch.cuda.mem_get_info()[0]
    b.close()
    one = states * gates * 128 * 128 * 4
    assert used <= 1.5 * one, (used, one)   # less where the driver reuses chunks freed before


@pytest.mark.parametrize("dtype,tol", [(0, 1e-6), (1, 1e-12)])
def test_batch_long_items(Q, oracle, dtype, tol):
    """Items of several tiles and of several cosets: four 19-qubit states in
    64-amplitude tiles are more than 48 tiles per CU in a level, and 400 terms
    on each give more than 16 full cosets per CU; beside them a state of one
    full coset (14 qubits complex64, 13 complex128) and one of two.
    Tolerances as for the uneven batch above."""
    cus, _, _ = Q.qs_device_query()
    one = 14 if dtype == 0 else 13
    ns = (one, one + 1, 19, 19, 19, 19)
    assert 4 * 2 ** (19 - 6) >= 2 * 24 * cus and 4 * (400 // 9) * 2 ** (19 - one) >= 2 * 8 * cus
    circuits = [qsynth.random_circuit(n, 25, seed=70 + i) for i, n in enumerate(ns)]
    hams = [qsynth.random_pauli_sum(n, 400 if n == 19 else 30, seed=(7, i)) for i, n in enumerate(ns)]
    b = Q.Batch(circuits, hams, Q.opts(k_max=3, tile_qubits=6, low_qubits=2, dtype=dtype))
    E = b.run()
    assert np.array_equal(E, b.run())
    for i, (c, h) in enumerate(zip(circuits, hams)):
        psi, e = _oracle_energy(oracle, c, h)
        assert abs(E[i] - e) <= tol * max(1, abs(e)), (i, c.n, E[i], e)
        assert oracle.max_abs(psi, b.amplitudes(i)) <= (1e-5 if dtype == 0 else 1e-12)
    b.close()
