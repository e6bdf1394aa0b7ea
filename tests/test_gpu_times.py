"""Times of one pass against another on the same GPU (gpu): paths that were
once slower than what they replaced.  Each time is the smallest of many, the
two taken in turn, and the bound lies well between the two ratios measured."""
import pytest
import torch

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def ci():
    import paper_1412_5989_amd as m

    return m


def ratio(f, g, reps=12):
    """Smallest time of f over smallest time of g."""
    a, e = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
    best = [float("inf"), float("inf")]
    for _ in range(reps):
        for k, h in enumerate((f, g)):
            a.record()
            h()
            e.record()
            e.synchronize()
            best[k] = min(best[k], a.elapsed_time(e))
    print("times (us)", [round(1e3 * t, 1) for t in best], flush=True)
    return best[0] / best[1]


def problem(ci, p):
    """Basis, row_ptr, two-body table, upstream gradient."""
    b = ci.ci_basis_build([p])
    rp, nnz = ci.ci_hamiltonian_count(b)
    gen = torch.Generator(device="cuda").manual_seed(3)
    t = torch.randn(b.n_tbme, device="cuda", generator=gen)
    G = torch.randn(sum(nnz), device="cuda", generator=gen)
    return b, rp, t, G


# 80 nucleons: sums of 79 terms and of 3160 pairs (8.2 times the fill of 8Be
# with twice the entries when one lane summed them and neighbouring lanes read
# far-apart words, 5.4 now)
def test_fill_of_many_nucleons(ci):
    f = []
    for p in ((40, 40, 2, 0, 1), (4, 4, 4, 0, 1)):
        b, rp, t, G = problem(ci, p)
        col, val = ci.ci_hamiltonian_fill(b, t, rp)
        f.append(lambda b=b, rp=rp, t=t, col=col, val=val: ci.ci_hamiltonian_fill(b, t, rp, col, val))
    assert ratio(*f) < 6.8


# a neutron-only basis: tiles of 64 x 8 hold 8 rows.  Untuned against 64 x 32
# tiles with tile records: 2.1 times with 64 x 8, 1.2 with the untuned 64 x 32.
def test_untuned_adjoint_of_few_proton_determinants(ci):
    b, rp, t, G = problem(ci, (0, 10, 4, 0, 1))
    c, _, _, _ = problem(ci, (0, 10, 4, 0, 1))
    c.tuning = {"adj_rows": 64, "adj_tile_n": 32, "adj_wide": 1, "adj_flush": 0, "adj_persistent": 0}
    work = torch.empty(max(b.vjp_work_bytes(), c.vjp_work_bytes()), dtype=torch.uint8, device="cuda")
    g = [torch.empty_like(t), torch.empty_like(t)]
    r = ratio(lambda: ci.ci_hamiltonian_vjp(b, rp, G, g[0], work), lambda: ci.ci_hamiltonian_vjp(c, rp, G, g[1], work))
    assert torch.equal(*g)  # the same 64 rows: the same fixed-point grid
    assert r < 1.6


# the tuner's choice against the untuned shapes: 1.27 and 1.46 times when those
# were not among its candidates
# (an energy of their own: the choice is kept for later handles of the problem)
@pytest.mark.parametrize("p", [(4, 5, 4, 1, 1, 15.5), (2, 2, 6, 0, 1, 15.5)])
def test_tuned_adjoint_is_not_slower_than_untuned(ci, p):
    b, rp, t, G = problem(ci, p)
    untuned = b.tuning
    room = b.vjp_work_bytes()
    col, val = ci.ci_hamiltonian_fill(b, t, rp)
    keys = torch.empty_like(col)
    print("tuned", ci.ci_hamiltonian_tune(b, t, rp, col, val, G, reps=3, keys=keys), flush=True)
    assert b.vjp_work_bytes() <= room
    c, _, _, _ = problem(ci, p)
    c.tuning = untuned
    work = torch.empty(room, dtype=torch.uint8, device="cuda")
    g = torch.empty_like(t)
    assert ratio(lambda: ci.ci_hamiltonian_vjp(b, rp, G, g, work), lambda: ci.ci_hamiltonian_vjp(c, rp, G, g, work)) < 1.12
    assert ratio(lambda: ci.ci_hamiltonian_vjp_keys(b, rp, keys, G, g, work),
                 lambda: ci.ci_hamiltonian_vjp_keys(c, rp, keys, G, g, work)) < 1.2


# one neutron: groups of one to five rows.  The full count against the upper
# triangle's: 1.17 times with 16 lanes for each row of a group of any size, 0.89 now.
def test_full_count_of_few_neutron_determinants(ci):
    b = ci.ci_basis_build([(6, 1, 6, 1, 1)])
    assert ratio(lambda: ci.ci_hamiltonian_count_full(b), lambda: ci.ci_hamiltonian_count(b)) < 1.05
