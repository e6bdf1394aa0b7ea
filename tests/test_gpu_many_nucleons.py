"""Fill of bases with many nucleons, at the edges of its two ways of summing
the terms of a one-nucleon difference (gpu)."""
import numpy as np
import pytest
import torch

import seeded_inputs as si

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def ci():
    import paper_1412_5989_amd as m

    return m


class Reference:
    """Elements of rows by the Slater-Condon rules in FP64, from the states and
    the two-body keys (the oracle's enumeration is too slow for this many nucleons)."""

    def __init__(self, ci, p, kinetic, b, tb):
        self.n = b.info[0]["n_sps"]
        self.hw, self.kinetic = ci.HW_MEV, kinetic
        self.v = {tuple(k): float(x) for k, x in zip(ci.ci_tbme_keys(p).tolist(), tb)}
        self.orb = [(N, l, j, m) for N in range(b.info[0]["shell_max"] + 1) for l in range(N % 2, N + 1, 2)
                    for j in (2 * l - 1, 2 * l + 1) if j > 0 for m in range(-j, j + 1, 2)]
        assert len(self.orb) == self.n
        W = b.info[0]["n_words"]
        s = b.states().cpu().numpy().view(np.uint8).reshape(b.info[0]["dim"], 2, W * 8)
        self.bits = np.unpackbits(s, axis=2, bitorder="little")[:, :, :self.n].reshape(-1, 2 * self.n)

    def two(self, a, b, c, d):
        sign = 1.0
        if a > b:
            a, b, sign = b, a, -sign
        if c > d:
            c, d, sign = d, c, -sign
        x = self.v.get((a, b, c, d))
        return sign * (self.v[(c, d, a, b)] if x is None else x)

    def one(self, p, h):
        (N, l, j, m), (M, k, i, q) = self.orb[p % self.n], self.orb[h % self.n]
        if p == h:
            return (N + 1.5) * self.hw * (0.5 if self.kinetic else 1.0)
        if not self.kinetic or (l, j, m) != (k, i, q) or abs(N - M) != 2:
            return 0.0
        r = (min(N, M) - l) // 2
        return 0.5 * self.hw * np.sqrt((r + 1) * (r + l + 1.5))

    def element(self, i, j):
        x, y = self.bits[i], self.bits[j]
        occ = np.flatnonzero(x).tolist()
        new, gone = np.flatnonzero(x & ~y & 1).tolist(), np.flatnonzero(y & ~x & 1).tolist()
        if not new:
            return sum(self.one(a, a) for a in occ) + sum(self.two(a, b, a, b) for t, b in enumerate(occ) for a in occ[:t])
        if len(new) > 1:
            return None
        p, h = new[0], gone[0]
        sign = (-1.0) ** int(x[min(p, h) + 1:max(p, h)].sum())
        return sign * (self.one(p, h) + sum(self.two(p, s, h, s) for s in occ if s != p))


# A - 1 terms, one more with the kinetic term: 31..33, 39, 63..65, 78..80
@pytest.mark.parametrize("kinetic", [0, 1])
@pytest.mark.parametrize("p", [(20, 12, 0, 0, 1), (20, 13, 0, 1, 1), (12, 20, 2, 12, -1), (40, 24, 0, 0, 1),
                               (25, 40, 1, 1, -1), (40, 39, 1, 1, 1), (40, 40, 1, 0, -1)])
def test_fill_values(ci, p, kinetic):
    b = ci.ci_basis_build([p + (ci.HW_MEV, kinetic)])
    rp, nnz = ci.ci_hamiltonian_count(b)
    tb = si.tbme_f32(17, b.n_tbme)
    t = torch.from_numpy(tb).cuda()
    col, val = ci.ci_hamiltonian_fill(b, t, rp)
    col2, val2, _ = ci.ci_hamiltonian_fill_keys(b, t, rp)
    assert torch.equal(col, col2) and torch.equal(val, val2)
    ref = Reference(ci, p, kinetic, b, tb)
    r, c, v = rp.cpu().numpy(), col.cpu().numpy(), val.cpu().numpy().astype(np.float64)
    A = p[0] + p[1]
    # one rounding to FP32, and an FP64 sum of up to A (A + 1) / 2 terms in another order
    top = A * A * (np.abs(tb).max() + 8 * ci.HW_MEV)
    seen = [0, 0]
    for i in np.unique(np.concatenate([np.random.default_rng(5).integers(0, b.info[0]["dim"], 12), [0]])):
        for e in range(r[i], r[i + 1]):
            x = ref.element(i, c[e])
            if x is not None:
                seen[int(c[e] != i)] += 1
                assert abs(v[e] - x) <= 2.0**-24 * abs(x) + A * A * top * 2.0**-53, (p, i, c[e], v[e], x)
    assert seen[0] and seen[1], seen
