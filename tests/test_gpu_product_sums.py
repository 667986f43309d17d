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


@pytest.mark.parametrize("n_steps", [2, 512, 513, 545])
def test_long_runs_replay_the_same_steps(n_steps):
    """TPQ runs around the length from which a graph of 32 steps is replayed: bit for bit the eager run."""
    print(f"[gpu] tpq run {n_steps} steps", flush=True)
    ham = hp.hphi_ham_build(hp.hphi_basis_build(BasisDesc("spin", 8, "sz", two_sz=0)),
                            [L.heisenberg_bond(i, (i + 1) % 8) for i in range(8)])
    psi = torch.from_numpy(uniform_vectors(ham.dim, [1, 2], True)).cuda()
    out = []
    for graph in (True, False):
        a, b = psi.clone(), torch.empty_like(psi)
        log = hp.hphi_tpq_run(ham, a, b, 1.5, 1, n_steps, use_graph=graph)
        out.append((log.clone(), (a if n_steps % 2 == 0 else b).clone()))
    assert torch.equal(out[0][0], out[1][0]) and torch.equal(out[0][1], out[1][1])
    lz = [hp.hphi_lanczos([ham], [psi[:, 0].contiguous()], 20, use_graph=g)[0] for g in (True, False)]
    assert np.array_equal(lz[0]["alpha"], lz[1]["alpha"])


@pytest.mark.parametrize("bits", [9, 14, 17, 19])
def test_sums_of_every_launch_are_its_own(bits):
    """2,000 products that alternate between two inputs: every launch's sums are those of its input,
    bit for bit (a last block that read a partial of the launch before would mix the two)."""
    print(f"[gpu] sums of alternating products {bits} bits", flush=True)
    ham = hp.hphi_ham_build(hp.hphi_basis_build(BasisDesc("spin", bits)), [L.heisenberg_bond(i, (i + 1) % bits) for i in range(bits)])
    n = 2000
    xs = [device_uniform(ham.dim, 0, seed, False, torch.float64) for seed in (1, 2)]
    xs[1] *= 3.0
    log = torch.empty((n, 4), dtype=torch.float64, device="cuda")
    for k in range(n):
        hp.hphi_hv(ham, xs[k & 1], reduce=log[k], write=False)
    torch.cuda.synchronize()
    assert torch.equal(log[0::2], log[0].expand(n // 2, 4)) and torch.equal(log[1::2], log[1].expand(n // 2, 4))
    x = xs[0].double()
    assert abs(float(log[0, 0]) - float((x * x).sum())) <= 1e-12 * float((x * x).sum())


def test_cg_solves_repeat_bit_for_bit():
    """200 CG solves from fresh workspaces give the same bits."""
    print("[gpu] repeated cg", flush=True)
    ham = hp.hphi_ham_build(hp.hphi_basis_build(BasisDesc("spin", 18, "sz", two_sz=0)), [L.heisenberg_bond(i, (i + 1) % 18) for i in range(18)])
    y = device_uniform(ham.dim, 0, 4, False, torch.float64)
    y /= torch.linalg.vector_norm(y)
    first = None
    for _ in range(200):
        x = y.clone()
        r = hp.hphi_cg_refine(ham, x, -10.0, n_inverse=1, cg_max_iter=12, cg_tol=1e-300)
        got = (r["e_refined"], r["cg_iters"], x)
        if first is None:
            first = got
        assert got[0] == first[0] and got[1] == 12 and torch.equal(x, first[2])
