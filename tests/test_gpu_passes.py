"""Kernels of the passes at the edges of their work splits (gpu)."""
import numpy as np
import pytest
import torch

from oracle import Oracle, Problem

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def ci():
    import paper_1412_5989_amd as m

    return m


# neutron keys of 1, a few, 15..17 and more determinants; one block, more than 64 blocks
@pytest.mark.parametrize("p", [(1, 1, 0, 0, 1), (6, 1, 2, 1, -1), (1, 6, 2, 1, -1), (3, 3, 4, 2, 1), (2, 2, 6, 0, 1),
                               (2, 3, 5, 1, -1)])
def test_count_groups(ci, p):
    b = ci.ci_basis_build([p, (2, 2, 2, 0, 1), p])
    o = Oracle(Problem(*p))
    rows = np.arange(o.dim)
    for count, ref in ((ci.ci_hamiltonian_count, o.row_counts(rows)), (ci.ci_hamiltonian_count_full, o.rows_full(rows, values=False)[0])):
        rp, nnz = count(b)
        for k in (0, 2):
            r = b.row_ptr_slice(rp, k).cpu().numpy()
            assert np.array_equal(np.diff(r), ref), (p, k)
            assert nnz[k] == ref.sum() and r[0] == sum(nnz[:k])


# one to four words per determinant; no nucleons of one kind; one nucleon; more
# determinants than one window of the bit mask (52949 neutron determinants)
@pytest.mark.parametrize("p", [(3, 4, 2, 1, -1), (3, 0, 4, 1, -1), (1, 1, 4, 2, 1), (2, 2, 6, 0, 1), (3, 3, 6, 2, 1),
                               (0, 6, 6, 0, 1)])
def test_partner_lists(ci, p):
    b = ci.ci_basis_build([p])
    o = Oracle(Problem(*p))
    rng = np.random.default_rng(3)
    rows = np.unique(np.concatenate([rng.integers(0, o.dim, 150), np.arange(32766, 32771), [0, o.dim - 1]]))
    rows = rows[rows < o.dim]
    rp, nnz = ci.ci_hamiltonian_count(b)
    col, _ = ci.ci_hamiltonian_fill(b, torch.zeros(b.n_tbme, device="cuda"), rp)
    r = rp.cpu().numpy()
    assert np.array_equal(np.diff(r)[rows], o.row_counts(rows)), p
    got = np.concatenate([col[r[i]:r[i + 1]].cpu().numpy() for i in rows])
    assert np.array_equal(got, o.rows(rows, values=False)[1]), p


# one-nucleon differences of more than 64 terms (A - 1, plus the kinetic term),
# which no round of lanes holds at once: the walking adjoint against the one
# from stored words (another evaluation of the same terms), and the fill against
# the adjoint through <G, H(t) - H(0)> = <H^T G, t>
@pytest.mark.parametrize("p", [(40, 39, 0, 1, -1), (39, 40, 0, 3, -1), (40, 26, 0, 18, 1)])
@pytest.mark.parametrize("kinetic", [0, 1])
def test_many_nucleons(ci, p, kinetic):
    b = ci.ci_basis_build([p + (15.0, kinetic)])
    rp, nnz = ci.ci_hamiltonian_count(b)
    assert b.info[0]["dim"] > 1 and sum(nnz) > b.info[0]["dim"]
    g = torch.Generator(device="cuda").manual_seed(11)
    t = torch.randn(b.n_tbme, device="cuda", generator=g)
    col, h0 = ci.ci_hamiltonian_fill(b, torch.zeros_like(t), rp)
    col, h, keys = ci.ci_hamiltonian_fill_keys(b, t, rp)
    G = torch.randn(sum(nnz), device="cuda", generator=g)
    b.tuning = {"adj_rows": 32, "adj_tile_n": 8, "adjk_rows": 32, "adjk_tile_n": 8}
    walk = ci.ci_hamiltonian_vjp(b, rp, G)
    stored = ci.ci_hamiltonian_vjp_keys(b, rp, keys, G)
    assert torch.equal(walk, stored)
    lhs = float((G.double() * (h.double() - h0.double())).sum())
    rhs = float((walk.double() * t.double()).sum())
    # h and h0 are rounded to FP32; a gradient element is rounded to FP32 and
    # sums at most dim contributions on a grid of spacing 2^-24 max |G|
    tol = float((G.abs().double() * (h.abs() + h0.abs()).double()).sum()) * 2.0**-24
    tol += float((t.abs().double() * (walk.abs().double() * 2.0**-24 + b.info[0]["dim"] * 2.0**-25 * float(G.abs().max()))).sum())
    assert abs(lhs - rhs) <= tol


# the lanes that a row of a group gets: each power of two, and sizes on both sides of it
def test_count_group_sizes(ci):
    sizes = set()
    for p in ((5, 1, 4, 0, 1), (2, 1, 4, 1, 1), (1, 2, 4, 1, 1), (2, 2, 4, 0, 1), (1, 3, 4, 2, 1)):
        o = Oracle(Problem(*p))
        n = np.diff(o.keys()["nkey_off"])
        groups = (n + 15) // 16
        rows = (n + groups - 1) // groups  # rows of a key's groups, fewer in its last one
        sizes |= set(rows) | set(n - (groups - 1) * rows)
        b = ci.ci_basis_build([p])
        every = np.arange(o.dim)
        for count, ref in ((ci.ci_hamiltonian_count, o.row_counts(every)),
                           (ci.ci_hamiltonian_count_full, o.rows_full(every, values=False)[0])):
            assert np.array_equal(np.diff(count(b)[0].cpu().numpy()), ref), p
    assert sizes >= {1, 2, 3, 4, 5, 7, 8, 10, 15, 16} and max(sizes) == 16, sizes


# one determinant table as the neutrons of one problem and the protons of another
@pytest.mark.parametrize("ps", [[(1, 4, 2, 1, -1), (4, 1, 2, 1, -1)], [(4, 1, 2, 1, -1), (1, 4, 2, 1, -1)],
                                [(4, 1, 2, 1, -1)], [(4, 0, 4, 0, 1), (2, 4, 2, 0, 1)]])
def test_count_of_shared_species(ci, ps):
    b = ci.ci_basis_build(ps)
    for k, p in enumerate(ps):
        o = Oracle(Problem(*p))
        rows = np.arange(o.dim)
        for count, ref in ((ci.ci_hamiltonian_count, o.row_counts(rows)),
                           (ci.ci_hamiltonian_count_full, o.rows_full(rows, values=False)[0])):
            assert np.array_equal(np.diff(b.row_ptr_slice(count(b)[0], k).cpu().numpy()), ref), p
