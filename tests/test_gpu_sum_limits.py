"""The sums of a product at the numbers of partials where they move from the kernel's last block to a
launch of their own, in each product kernel, alone and with the scalar step of a TPQ step."""

import pytest
import torch

from synth import lattices as L
from synth.configs import BasisDesc
from synth.vectors import device_uniform

pytestmark = pytest.mark.gpu

import paper_1703_03637_amd as hp  # noqa: E402


@pytest.fixture(scope="module", autouse=True)
def _need_gpu():
    assert torch.cuda.is_available(), "GPU tests need an MI355X"


def _chain(n, z=0.0):
    # z: a Dzyaloshinskii-Moriya part, which makes the Hamiltonian complex
    return [L.Term(L.SPIN_BOND, i, (i + 1) % n, (1.0, z, 0, -z, 1.0, 0, 0, 0, 1.0)) for i in range(n)]


# per-tile, class-blocked and windowed kernel; rows from one block to the persistent grid's limit, so that the
# partials (4 x vectors x blocks) pass 1,024, 4,096 and 16,384
CASES = [(k, n, nvec) for k, sizes in (("tiles", (12, 16, 18, 20, 22)), ("classes", (12, 16, 18, 20, 22)),
                                       ("windowed", (9, 12, 14, 16, 18))) for n in sizes for nvec in (1, 4, 16)]


@pytest.mark.parametrize("kernel,n,nvec", CASES)
def test_sums_at_the_limits(kernel, n, nvec):
    """The four sums are FP64 sums over the product's own output (1e-12 of the sum of sizes), the same bits call
    after call and in a replayed graph; without an output vector too, up to the order of a windowed product's
    passes (there is one); a TPQ step's numbers follow from them."""
    print(f"[gpu] sum limits {kernel} {n} sites nvec={nvec}", flush=True)
    desc = BasisDesc("spin", n) if kernel == "windowed" else BasisDesc("spin", n, "sz", two_sz=0)
    ham = hp.hphi_ham_build(hp.hphi_basis_build(desc), _chain(n, 0.3 if kernel == "tiles" else 0.0))
    x = device_uniform(ham.dim, 0 if nvec == 1 else nvec, 11, True, torch.complex128)
    red = torch.full((4 * nvec,), -1.0, dtype=torch.float64, device="cuda")
    u = hp.hphi_hv(ham, x, reduce=red)
    xs, us = x.reshape(ham.dim, nvec), u.reshape(ham.dim, nvec)
    xx, xu, uu = (xs.conj() * xs).real.sum(0), (xs.conj() * us).real.sum(0), (us.conj() * us).real.sum(0)
    size = torch.stack([xx, (xs.abs() * us.abs()).sum(0), uu, uu])
    assert torch.all((red.reshape(4, nvec) - torch.stack([xx, xu, uu, uu])).abs() <= 1e-12 * size)
    first = red.clone()
    out = torch.empty_like(u)
    s = torch.cuda.Stream()
    s.wait_stream(torch.cuda.current_stream())
    g = torch.cuda.CUDAGraph()
    with torch.cuda.graph(g, stream=s):
        hp.hphi_hv(ham, x, out, reduce=red)
    for k in range(3):
        red.fill_(-1.0)
        g.replay()
        torch.cuda.synchronize()
        assert torch.equal(red, first) and torch.equal(out, u)
        red.fill_(-1.0)
        hp.hphi_hv(ham, x, reduce=red, write=False)
        assert torch.equal(red, first) or (kernel == "windowed" and
                                           torch.all((red - first).abs().reshape(4, nvec) <= 1e-12 * size))
    l, k, obs = 1.5, 3, torch.empty((1, 4, nvec), dtype=torch.float64, device="cuda")
    scale = 1.0 / torch.sqrt(xx)
    phi = torch.empty_like(x)
    hp.hphi_tpq_step(ham, x, phi, l, k, scale, obs)
    e = xu / xx / n
    pp = phi.reshape(ham.dim, nvec)
    want = torch.stack([e, uu / xx / n ** 2, 2.0 * (k - 1) / n / (l - e), 1.0 / torch.sqrt((pp.conj() * pp).real.sum(0))])
    # e is a small difference of large terms: its error is relative to |x| |Hx| / |x|^2
    bound = 1e-11 * torch.stack([torch.sqrt(uu / xx), uu / xx, torch.sqrt(uu / xx), want[3]]).clamp(min=1.0)
    assert torch.all((obs[0] - want).abs() <= bound)
