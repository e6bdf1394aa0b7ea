"""A batch of more rows, groups of rows and adjoint tiles than one launch can
hold in threads (gpu; about 60 GB of device memory)."""
import pytest
import torch

pytestmark = pytest.mark.gpu


def test_more_rows_than_one_launch_holds():
    import paper_1412_5989_amd as ci

    p, copies = (3, 3, 2, 0, 1), 84000
    one = ci.ci_basis_build([p])
    rp1, (nnz1,) = ci.ci_hamiltonian_count(one)
    gen = torch.Generator(device="cuda").manual_seed(3)
    t1 = torch.randn(one.n_tbme, device="cuda", generator=gen)
    G1 = torch.randn(nnz1, device="cuda", generator=gen)
    col1, val1 = ci.ci_hamiltonian_fill(one, t1, rp1)
    D = one.info[0]["dim"]
    print("build", flush=True)
    b = ci.ci_basis_build([p] * copies)
    assert D * copies * 64 > 2**32 and b.tuning["row_grab"] == 0
    print("count", flush=True)
    rp, nnz = ci.ci_hamiltonian_count(b)
    assert nnz == [nnz1] * copies
    want = torch.arange(copies, device="cuda")[:, None] * nnz1 + rp1
    assert torch.equal(rp.view(copies, D + 1), want)
    del want
    print("fill", flush=True)
    col = torch.full((nnz1 * copies,), -1, dtype=torch.int32, device="cuda")
    val = torch.full((nnz1 * copies,), float("nan"), device="cuda")
    ci.ci_hamiltonian_fill(b, t1.repeat(copies), rp, col, val)
    for k in range(0, copies, 1000):  # every basis as the one alone
        n = min(1000, copies - k)
        assert torch.equal(col[k * nnz1:(k + n) * nnz1], col1.repeat(n)), k
        assert torch.equal(val[k * nnz1:(k + n) * nnz1], val1.repeat(n)), k
    del col, val
    print("adjoint", flush=True)
    b.tuning = {"adj_rows": 8, "adj_tile_n": 8, "adj_persistent": 0}
    one.tuning = b.tuning
    assert D * copies // 8 * 1024 > 2**32
    g1 = ci.ci_hamiltonian_vjp(one, rp1, G1)
    g = ci.ci_hamiltonian_vjp(b, rp, G1.repeat(copies)).view(copies, -1)
    assert torch.equal(g, g1.expand_as(g))
