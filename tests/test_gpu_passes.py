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
