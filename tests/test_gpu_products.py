"""H times a state through the row kernels, at row lengths around their launch
shapes, against the oracle.

Tolerances: energies 1e-10 Ha, adjoint gradients 1e-9, as for every product
path (sums of at most a few thousand terms of unit-norm states)."""

import numpy as np
import pytest

from oracle import sector
from workloads import random_problem
from tests.gpu_helpers import dense_from_sector, oracle_energy_grad, say

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def fsv(gpu):
    import paper_2405_11567_amd as m
    m.load()
    return m


def _problem(m, na, nb, rank, seed):
    p = random_problem(2 * m, 2 * nb, 6, seed=seed, theta_std=0.4, replace=True, ordering=seed % 2)
    # na differs from nb: operators are drawn again for the actual counts
    from workloads import uccsd_pool
    rng = np.random.default_rng(seed)
    pool = uccsd_pool(m, na, nb)
    p.n_alpha, p.n_beta = na, nb
    p.ops = np.ascontiguousarray(pool[rng.integers(0, len(pool), 6)])
    p.theta = rng.normal(0, 0.4, 6)
    p.e_core = 0.25
    if rank:
        f = np.stack([(lambda l: l + l.T)(rng.normal(0, 0.05, (m, m))) for _ in range(rank)]).reshape(rank, m * m)
        p.g = (f.T @ f).reshape(m, m, m, m)
    return p


# rows of 2, 3, 10, 84, 126, 210 (odd pairs), 462, 715 (odd), 924, 1287, 1716 and
# 3003 columns; then few columns under 1287 and 3003 alpha strings
@pytest.mark.parametrize("m,na,nb,rank", [
    (2, 1, 1, 0), (3, 1, 1, 0), (5, 2, 2, 0), (9, 1, 3, 0), (9, 2, 4, 0), (10, 1, 4, 0), (11, 1, 5, 0),
    (13, 1, 4, 0), (12, 1, 6, 0), (13, 1, 5, 0), (13, 1, 6, 0), (14, 1, 6, 0), (13, 5, 1, 0), (14, 6, 1, 0),
    (3, 1, 1, 6), (5, 2, 2, 15), (9, 1, 3, 20), (9, 2, 4, 45), (11, 1, 5, 30), (13, 1, 4, 40), (12, 1, 6, 78),
    (13, 1, 5, 30), (14, 1, 6, 20)])
def test_row_products(fsv, m, na, nb, rank):
    import torch
    p = _problem(m, na, nb, rank, seed=900 + 17 * m + nb)
    say("row products", m, na, nb, rank)
    plan = fsv.Plan(p)
    e, g = plan.energy_grad(p.theta)
    e_ref, g_ref = oracle_energy_grad(p)
    assert abs(e - e_ref) < 1e-10 and np.abs(g - g_ref).max() < 1e-9
    psi = plan.ansatz_apply(p.theta)
    assert abs(plan.energy(psi) - e_ref) < 1e-10
    # a complex state, and a real one again after it
    rng = np.random.default_rng(m)
    d = sector.dim(m, na, nb)
    vec = rng.normal(size=d) + 1j * rng.normal(size=d)
    vec /= np.linalg.norm(vec)
    full, _ = dense_from_sector(vec, p)
    t = torch.from_numpy(full).to(plan.device)
    assert abs(plan.energy(t) - sector.energy(vec, p.h, p.g, p.e_core, na, nb, p.ordering)) < 1e-10
    assert abs(plan.energy(psi) - e_ref) < 1e-10


# general integrals: rows of 126, 210, 252, 330, 495, 1001, 1716 and 2002 columns
# (either side of each launch shape); 1, 4, 5, 9 and 13 sources (a step of four
# and its remainders, no excitation at all), 6, 10 and more orbital pairs (a
# chunk of 16 and its remainder)
@pytest.mark.parametrize("m,na,nb,rank", [
    (3, 3, 1, 6), (4, 4, 2, 10), (9, 8, 4, 20), (10, 9, 4, 20), (10, 10, 5, 20), (11, 1, 4, 30), (12, 2, 4, 12),
    (14, 1, 4, 20), (13, 12, 6, 20), (14, 13, 5, 12)])
def test_general_rows(fsv, m, na, nb, rank):
    test_row_products(fsv, m, na, nb, rank)


# dense same-spin products of 36 to 495 strings (tiles with a remainder on every
# side), few and many columns, either side of 1024 tiles, accumulated (general
# integrals) and not
@pytest.mark.parametrize("m,na,nb,rank", [
    (9, 2, 4, 0), (8, 4, 4, 0), (8, 4, 4, 20), (9, 4, 5, 20), (10, 3, 5, 0), (12, 2, 5, 20), (12, 5, 2, 20),
    (12, 4, 4, 0), (12, 4, 5, 0)])
def test_same_spin_tiles(fsv, m, na, nb, rank):
    test_row_products(fsv, m, na, nb, rank)


# dense images smaller than, equal to and larger than a chunk of 1024 amplitudes,
# both orderings and types, chunks without a sector amplitude
@pytest.mark.parametrize("precision", [0, 1])
@pytest.mark.parametrize("ordering", [0, 1])
@pytest.mark.parametrize("m,na,nb", [(2, 1, 1), (5, 2, 3), (6, 5, 1), (8, 1, 7), (10, 3, 2)])
def test_dense_image(fsv, m, na, nb, ordering, precision):
    p = _problem(m, na, nb, 0, seed=30 + m)
    p.ordering = ordering
    say("dense image", m, na, nb, ordering, precision)
    plan = fsv.Plan(p, precision=precision)
    psi = plan.new_state()
    psi.fill_(7.0)  # every amplitude is written
    got = plan.ansatz_apply(p.theta, psi).cpu().numpy()
    want, _ = dense_from_sector(sector.ansatz(m, na, nb, p.ops, p.theta, ordering, 0), p)
    # a few rotations of a unit-norm state
    assert np.abs(got - want).max() < (1e-13 if precision == 0 else 1e-6)
    assert (got[want == 0] == 0).sum() >= (1 << 2 * m) - sector.dim(m, na, nb)


# 1-RDMs of a real and of a complex state: no excitation between strings, one to
# 30 of them per row, rows shorter and longer than a wavefront
@pytest.mark.parametrize("m,na,nb", [
    (2, 1, 1), (4, 4, 2), (4, 4, 3), (6, 3, 1), (9, 8, 4), (10, 5, 5), (11, 1, 4), (11, 5, 10), (12, 1, 6)])
def test_rdm_rows(fsv, m, na, nb):
    import torch
    p = _problem(m, na, nb, 0, seed=60 + m)
    say("rdm rows", m, na, nb)
    plan = fsv.Plan(p)
    rng = np.random.default_rng(m)
    d = sector.dim(m, na, nb)
    for vec in (rng.normal(size=d) + 1j * rng.normal(size=d), rng.normal(size=d) + 0j):
        vec /= np.linalg.norm(vec)
        full, _ = dense_from_sector(vec, p)
        gam = plan.rdm1(torch.from_numpy(full).to(plan.device))
        # sums of at most a few thousand terms of a unit-norm state
        assert np.abs(gam - sector.rdm1(vec, m, na, nb, p.ordering)).max() < 1e-12


# rows of 2, 21 (odd), 126, 462 and 924 columns; sectors whose row pairs leave
# remainders of the workgroups' share; one operator, repeated ones, a whole pool
@pytest.mark.parametrize("m,na,nb,excitation,ordering,precision", [
    (2, 1, 1, 0, 0, 0), (7, 2, 2, 1, 0, 0), (9, 4, 4, 0, 1, 0), (9, 3, 4, 1, 1, 0), (11, 3, 5, 1, 0, 0),
    (12, 2, 6, 0, 0, 0), (12, 6, 2, 1, 0, 0), (9, 4, 4, 1, 0, 1)])
def test_pool_rows(fsv, m, na, nb, excitation, ordering, precision):
    from workloads import uccsd_pool
    p = _problem(m, na, nb, 0, seed=700 + 11 * m + na)
    p.ordering, p.excitation = ordering, excitation
    full = np.asarray(uccsd_pool(m, na, nb), dtype=np.int32)
    rng = np.random.default_rng(m)
    some = full[rng.integers(0, len(full), min(len(full), 70))]  # repeats
    say("pool rows", m, na, nb, excitation, ordering, precision)
    psi = sector.ansatz(m, na, nb, p.ops, p.theta, ordering, excitation)
    ref = sector.pool_gradients(psi, p.h, p.g, p.e_core, full, na, nb, ordering, excitation)
    at = {tuple(o): t for t, o in enumerate(full)}
    plan = fsv.Plan(p, precision=precision)
    tol = 1e-9 if precision == 0 else 1e-4  # FP32 states: as the FP32 energies
    for ops in (full, full[-1:], some):
        _, g = plan.pool(ops).gradients(p.theta)
        want = ref[[at[tuple(o)] for o in ops]]
        assert np.abs(g - want).max() < tol


# whole sweeps in one workgroup (states of at most 8192 amplitudes): 1 operator,
# 16 and 17 (a block of steps and its remainder), operators of one pair and of
# several steps; 8281 amplitudes: packets either way
@pytest.mark.parametrize("m,na,nb,k,precision", [
    (2, 1, 1, 1, 0), (4, 2, 2, 16, 0), (4, 2, 2, 17, 1), (6, 1, 3, 33, 0), (9, 3, 3, 17, 0), (9, 3, 3, 40, 1),
    (13, 2, 2, 16, 0), (14, 2, 2, 17, 0)])
def test_whole_sweeps(fsv, m, na, nb, k, precision, monkeypatch):
    import dataclasses
    from workloads import uccsd_pool
    from tests.gpu_helpers import random_dets
    p = _problem(m, na, nb, 0, seed=500 + m)
    pool = uccsd_pool(m, na, nb)
    rng = np.random.default_rng(m + k)
    p = dataclasses.replace(p, ops=np.ascontiguousarray(pool[rng.integers(0, len(pool), k)]),
                            theta=rng.normal(0, 0.3, k))
    say("whole sweeps", m, na, nb, k, precision)
    plan = fsv.Plan(p, precision=precision)
    dim = sector.dim(m, na, nb)
    if dim <= 8192:
        assert all((r == 0).all() and (t == 1).all() for r, t in (plan.runs(), plan.runs(adjoint=True)))
    monkeypatch.setenv("FSV_FUSE", "packets")
    ref = fsv.Plan(p, precision=precision)
    e_ref, g_ref = oracle_energy_grad(p)
    tol_e, tol_g = (1e-10, 1e-9) if precision == 0 else (1e-4, 1e-4)
    for warm in (False, True):
        if warm:
            dets, coef = random_dets(p, min(5, dim), seed=k)
            plan.set_initial_state(dets, coef)
            ref.set_initial_state(dets, coef)
        for _ in range(2):
            e, g = plan.energy_grad(p.theta)
            e2, g2 = ref.energy_grad(p.theta)
            # the same rotations in the same order; gradient terms of a unit-norm
            # state summed in another order
            assert abs(e - e2) < 1e-12 and np.abs(g - g2).max() < 1e-11
            if not warm:
                assert abs(e - e_ref) < tol_e and np.abs(g - g_ref).max() < tol_g


# operators without a pair in the sector (an alpha-alpha double on one alpha
# electron): first, in the middle, behind whole blocks of 16 steps, last, two in
# a row, and nothing else
@pytest.mark.parametrize("precision", [0, 1])
@pytest.mark.parametrize("before,empty,after", [(0, 1, 3), (2, 1, 2), (4, 2, 1), (3, 1, 0), (16, 1, 17), (0, 1, 0), (0, 3, 0)])
def test_whole_sweeps_without_pairs(fsv, before, empty, after, precision):
    import dataclasses
    from workloads import uccsd_pool
    from tests.gpu_helpers import random_dets
    m, na, nb = 4, 1, 1
    p = _problem(m, na, nb, 0, seed=541)
    pool = uccsd_pool(m, na, nb)
    rng = np.random.default_rng(before + 31 * after)
    some = pool[rng.integers(0, len(pool), before + after)].reshape(-1, 4)
    ops = np.concatenate([some[:before], np.tile([[4, 6, 2, 0]], (empty, 1)), some[before:]]).astype(np.int32)
    k = len(ops)
    p = dataclasses.replace(p, ops=np.ascontiguousarray(ops), theta=rng.normal(0, 0.3, k))
    say("whole sweeps without pairs", before, empty, after, precision)
    plan = fsv.Plan(p, precision=precision)
    assert all((r == 0).all() and (t == 1).all() for r, t in (plan.runs(), plan.runs(adjoint=True)))
    e_ref, g_ref = oracle_energy_grad(p)
    tol_e, tol_g = (1e-10, 1e-9) if precision == 0 else (1e-4, 1e-4)
    for _ in range(2):
        e, g = plan.energy_grad(p.theta)
        assert abs(e - e_ref) < tol_e and np.abs(g - g_ref).max() < tol_g
        assert (g[before:before + empty] == 0.0).all()
    dets, coef = random_dets(p, 5, seed=k)
    plan.set_initial_state(dets, coef)
    e, g = plan.energy_grad(p.theta)
    keep = np.r_[:before, before + empty:k]
    ref = fsv.Plan(dataclasses.replace(p, ops=np.ascontiguousarray(ops[keep]), theta=p.theta[keep]), precision=precision)
    ref.set_initial_state(dets, coef)
    # the same rotations and sums: the operators left out change no amplitude
    e2, g2 = ref.energy_grad(p.theta[keep])
    assert abs(e - e2) < 1e-12 and np.abs(g[keep] - g2).max(initial=0.0) < 1e-11
    assert (g[before:before + empty] == 0.0).all()


# rows of 5005 columns (30 qubits): the longest launch shape of general integrals,
# and factorised ones
@pytest.mark.parametrize("rank", [20, 0])
def test_long_rows(fsv, rank):
    p = _problem(15, 1, 6, rank, seed=931)
    say("long rows", rank)
    e, g = fsv.Plan(p).energy_grad(p.theta)
    e_ref, g_ref = oracle_energy_grad(p)
    assert abs(e - e_ref) < 1e-10 and np.abs(g - g_ref).max() < 1e-9


# screening with three, two and one row pair per workgroup, in both precisions,
# with a remainder of row pairs: FP64 rows of 792 and 1287 columns, FP32 rows of
# 1287, 1716 and 3003
@pytest.mark.parametrize("m,na,nb,precision", [(12, 2, 5, 0), (13, 2, 5, 0), (13, 2, 5, 1), (13, 2, 6, 1), (14, 1, 6, 1)])
def test_pool_long_rows(fsv, m, na, nb, precision, monkeypatch):
    monkeypatch.setenv("FSV_POOL", "rows")
    from workloads import uccsd_pool
    p = _problem(m, na, nb, 0, seed=700 + 11 * m + nb)
    full = np.asarray(uccsd_pool(m, na, nb), dtype=np.int32)
    ops = np.ascontiguousarray(full[np.random.default_rng(m).permutation(len(full))[:40]])
    say("pool long rows", m, na, nb, precision)
    psi = sector.ansatz(m, na, nb, p.ops, p.theta, p.ordering, p.excitation)
    want = sector.pool_gradients(psi, p.h, p.g, p.e_core, ops, na, nb, p.ordering, 0)
    _, g = fsv.Plan(p, precision=precision).pool(ops).gradients(p.theta)
    assert np.abs(g - want).max() < (1e-9 if precision == 0 else 1e-4)  # as test_pool_rows


# the cases of test_pool_rows through each of the two screening kernels (pools
# of these sizes take pairs by themselves), and nothing to screen: operators
# without a pair in the sector
@pytest.mark.parametrize("mode", ["rows", "pairs"])
@pytest.mark.parametrize("m,na,nb,excitation,ordering,precision", [
    (2, 1, 1, 0, 0, 0), (7, 2, 2, 1, 0, 0), (9, 4, 4, 0, 1, 0), (9, 3, 4, 1, 1, 0), (11, 3, 5, 1, 0, 0),
    (12, 2, 6, 0, 0, 0), (12, 6, 2, 1, 0, 0), (9, 4, 4, 1, 0, 1)])
def test_pool_both_ways(fsv, mode, m, na, nb, excitation, ordering, precision, monkeypatch):
    monkeypatch.setenv("FSV_POOL", mode)
    test_pool_rows(fsv, m, na, nb, excitation, ordering, precision)


@pytest.mark.parametrize("mode", ["rows", "pairs", ""])
def test_pool_without_pairs(fsv, mode, monkeypatch):
    monkeypatch.setenv("FSV_POOL", mode)
    p = _problem(4, 1, 1, 0, seed=551)
    say("pool without pairs", mode)
    ops = np.array([[4, 6, 2, 0], [5, 7, 3, 1]], dtype=np.int32)
    _, g = fsv.Plan(p).pool(ops).gradients(p.theta)
    assert (g == 0.0).all()


# the choice between the two, by sizes: the whole pool at 24 qubits is screened
# by rows, 50 of its operators and a 22-qubit pool pair by pair; both agree
# (sums of the same products in another order)
@pytest.mark.parametrize("m,na,nb,k", [(12, 6, 6, 0), (12, 6, 6, 50), (11, 5, 5, 400)])
def test_pool_choice(fsv, m, na, nb, k, monkeypatch):
    from workloads import uccsd_pool
    p = _problem(m, na, nb, 0, seed=560 + m)
    full = np.asarray(uccsd_pool(m, na, nb), dtype=np.int32)
    ops = np.ascontiguousarray(full[np.random.default_rng(k).permutation(len(full))[:k or len(full)]])
    say("pool choice", m, na, nb, k)
    plan = fsv.Plan(p)
    got = []
    for mode in ("", "rows", "pairs"):
        monkeypatch.setenv("FSV_POOL", mode)
        got.append(plan.pool(ops).gradients(p.theta)[1])
    assert np.array_equal(got[0], got[1 if k == 0 else 2])
    assert np.abs(got[1] - got[2]).max() < 1e-12


# rows whose orbital pairs are shared by groups of wavefronts (few rows of at most
# 128 or of 257 to 384 columns) and rows that are not (792 rows, two planes; 715
# rows); pairs and source rows that leave a rest
@pytest.mark.parametrize("m,na,nb", [
    (8, 1, 2), (8, 7, 2), (8, 3, 4), (9, 4, 2), (11, 1, 2), (12, 4, 2), (12, 5, 2), (13, 1, 3), (13, 4, 3), (14, 2, 3)])
def test_row_groups(fsv, m, na, nb):
    test_row_products(fsv, m, na, nb, 0)
