"""The sums that the last block of a product takes, at the edges of its ticket groups (32 blocks) and of
the rule that hands many partials to a launch of their own, and the scalars of a CG solve at the edges
of the chunks the host waits for."""

import numpy as np
import pytest
import torch

from oracle import hamiltonian as oh
from synth import lattices as L
from synth.configs import BasisDesc
from synth.vectors import device_uniform, uniform_vectors

pytestmark = pytest.mark.gpu

import paper_1703_03637_amd as hp  # noqa: E402


@pytest.fixture(scope="module", autouse=True)
def _need_gpu():
    assert torch.cuda.is_available(), "GPU tests need an MI355X"


@pytest.mark.parametrize("bits,nvec", [(1, 1), (6, 1), (8, 1), (12, 1), (13, 1), (14, 1), (18, 1), (21, 1), (13, 4), (12, 16),
                                       (14, 16), (16, 16), (18, 16)])
def test_product_sums(bits, nvec):
    """The four sums equal FP64 sums over the product's own output, call after call and in a graph."""
    print(f"[gpu] product sums {bits} bits nvec={nvec}", flush=True)
    terms = [L.heisenberg_bond(i, (i + 1) % bits) for i in range(bits)] if bits > 2 else [L.Term(L.SPIN_FIELD, 0, -1, (0.3, 0.0, 0.7))]
    ham = hp.hphi_ham_build(hp.hphi_basis_build(BasisDesc("spin", bits)), terms)
    red = torch.empty(4 * nvec, dtype=torch.float64, device="cuda")
    u = None
    for seed in (1, 2):
        x = device_uniform(ham.dim, 0 if nvec == 1 else nvec, seed, True, torch.complex128)
        u = hp.hphi_hv(ham, x, u, reduce=red)
        xs, us = x.reshape(ham.dim, nvec), u.reshape(ham.dim, nvec)
        want = torch.stack([(xs.conj() * xs).real.sum(0), (xs.conj() * us).real.sum(0), (us.conj() * us).real.sum(0),
                            (us.conj() * us).real.sum(0)])
        size = torch.stack([want[0], (xs.abs() * us.abs()).sum(0), want[2], want[3]])
        first = red.clone()
        assert torch.all((red.reshape(4, nvec) - want).abs() <= 1e-12 * size)
    out = torch.empty_like(u)
    s = torch.cuda.Stream()
    s.wait_stream(torch.cuda.current_stream())
    g = torch.cuda.CUDAGraph()
    with torch.cuda.graph(g, stream=s):
        hp.hphi_hv(ham, x, out, reduce=red)
    for _ in range(3):
        red.zero_()
        g.replay()
        torch.cuda.synchronize()
        assert torch.equal(red, first) and torch.equal(out, u)
        hp.hphi_hv(ham, x, out)


@pytest.mark.parametrize("n_iter", [1, 7, 8, 9, 24, 25])
def test_cg_stops_where_asked(n_iter):
    """A CG solve of n_iter steps equals the literal recurrence (1e-12 of the vector's size)."""
    print(f"[gpu] cg {n_iter} steps", flush=True)
    desc = BasisDesc("spin", 10, "sz", two_sz=0)
    terms = [L.heisenberg_bond(i, (i + 1) % 10) for i in range(10)]
    H = oh.sparse_h(desc, terms).real.tocsr()
    y = uniform_vectors(H.shape[0], [5], False)[:, 0]
    y /= np.linalg.norm(y)
    ham = hp.hphi_ham_build(hp.hphi_basis_build(desc), terms)
    x = torch.from_numpy(y.copy()).cuda()
    r = hp.hphi_cg_refine(ham, x, -6.0, shift=1e-6, n_inverse=1, cg_max_iter=n_iter, cg_tol=1e-300)
    assert r["cg_iters"] == n_iter and r["info"] == 2
    e = -6.0 + 1e-6
    xs = y.copy()
    res = y - (H @ xs - e * xs)
    p, rr = res.copy(), res @ res
    for _ in range(n_iter):
        q = H @ p - e * p
        a = rr / (p @ q)
        xs += a * p
        res -= a * q
        rn = res @ res
        p = res + rn / rr * p
        rr = rn
    xs /= np.linalg.norm(xs)
    assert np.max(abs(x.cpu().numpy() - xs)) <= 1e-12
    # a tolerance that the first step meets, and one that the start meets
    x = torch.from_numpy(y.copy()).cuda()
    assert hp.hphi_cg_refine(ham, x, -6.0, n_inverse=1, cg_max_iter=n_iter, cg_tol=1e3)["cg_iters"] == 0
