"""The class-blocked sector product (one low-half decode for several high halves) against the oracle
and the per-tile kernel: charge classes shorter and longer than a tile, partial groups of high halves,
both particle kinds, every storage type and batch, and the calls that stay with the per-tile kernel."""

import numpy as np
import pytest
import torch

from oracle import basis as ob
from oracle import hamiltonian as oh
from synth import lattices as L
from synth.configs import BasisDesc
from synth.vectors import uniform_vectors

pytestmark = pytest.mark.gpu

import paper_1703_03637_amd as hp  # noqa: E402


@pytest.fixture(scope="module", autouse=True)
def _need_gpu():
    assert torch.cuda.is_available(), "GPU tests need an MI355X"


CASES = {
    # low classes up to 252 rows (tiles of 64 and a remainder), 9-bit high half
    "spin19": (BasisDesc("spin", 19, "sz", two_sz=1, split_bits=10),
               lambda: [L.heisenberg_bond(i, (i + 1) % 19, 1.0 + 0.1 * i) for i in range(19)]),
    # random XXZ couplings and fields: diagonal terms of every kind, one element per operator
    "spin_random": (BasisDesc("spin", 13, "sz", two_sz=-1, split_bits=7),
                    lambda: L.random_spin_terms(13, 30, 71, conserve_sz=True, fields=True, real=True)),
    # one low bit, one high half per class
    "spin_split1": (BasisDesc("spin", 8, "sz", two_sz=0, split_bits=1),
                    lambda: [L.heisenberg_bond(i, (i + 3) % 8) for i in range(8)]),
    # everything in the low half
    "spin_split_all": (BasisDesc("spin", 9, "sz", two_sz=1, split_bits=9),
                       lambda: [L.heisenberg_bond(i, (i + 1) % 9) for i in range(9)]),
    # fermion signs inside each half and across, densities across, U and mu
    "ferm_nupndn": (BasisDesc("fermion", 7, "nupndn", n_up=3, n_dn=4),
                    lambda: L.random_fermion_terms(7, 24, 72, conserve_spin=True, n_dens=9, with_mu=True)),
    "ferm_ntot": (BasisDesc("fermion", 5, "ntot", n_tot=4),
                  lambda: L.random_fermion_terms(5, 18, 73, conserve_spin=False, n_dens=5, with_mu=True)),
    "hubbard_4x2": (BasisDesc("fermion", 8, "nupndn", n_up=4, n_dn=3, split_bits=10),
                    lambda: L.hubbard_terms(L.rect_bonds(4, 2), 8, t=1.0, U=8.0)),
}
DT = {"f64": torch.float64, "f32": torch.float32, "c128": torch.complex128, "c64": torch.complex64}


def _problem(name):
    desc, mk = CASES[name]
    terms = mk()
    st = ob.states(desc)
    return desc, terms, st, hp.hphi_ham_build(hp.hphi_basis_build(desc), terms)


@pytest.mark.parametrize("k", [1, 2, 4, 8])
@pytest.mark.parametrize("name", list(CASES))
def test_class_blocked_matches_oracle(monkeypatch, name, k):
    """FP64 products within 1e-12 per element of |H||v|; the four sums within 1e-12."""
    print(f"[gpu] class-blocked {name} k={k}", flush=True)
    monkeypatch.setenv("HPHI_GROUP_K", str(k))
    desc, terms, st, ham = _problem(name)
    H = oh.sparse_h(desc, terms).real
    Ha = abs(H)
    for dt, nvec in (("f64", 1), ("c128", 1), ("f64", 2), ("c128", 4), ("f64", 16), ("c128", 16)):
        v = uniform_vectors(len(st), list(range(nvec)), dt[0] == "c")
        red = torch.empty(4 * nvec, dtype=torch.float64, device="cuda")
        scale = torch.linspace(0.5, 1.5, nvec, dtype=torch.float64, device="cuda")
        vd = torch.from_numpy(v).cuda()
        u = hp.hphi_hv(ham, vd if nvec > 1 else vd.reshape(-1), a=-0.3, b=0.7, in_scale=scale, reduce=red)
        x = v * scale.cpu().numpy()
        h = H @ x
        w = -0.3 * h + 0.7 * x
        bound = 1e-12 * (Ha @ abs(x) + abs(x))
        assert np.all(abs(u.cpu().numpy().reshape(len(st), nvec) - w) <= bound), (dt, nvec)
        want = [np.sum(abs(x) ** 2, 0), np.sum((x.conj() * h).real, 0), np.sum(abs(h) ** 2, 0), np.sum(abs(w) ** 2, 0)]
        size = [want[0], np.sum(abs(x) * (Ha @ abs(x)), 0), want[2], want[3]]
        for q in range(4):
            assert np.all(abs(red.cpu().numpy().reshape(4, nvec)[q] - want[q]) <= 1e-12 * size[q])


@pytest.mark.parametrize("nvec", [1, 2, 4, 8, 16])
@pytest.mark.parametrize("dt", list(DT))
def test_class_blocked_storage_types_match_per_tile(monkeypatch, dt, nvec):
    """Every storage type and batch: the per-tile kernel's result up to one rounding of the stored
    value and the order of an FP64 sum (2^-24 resp. 1e-13 of |H||v|), reduce-only sums too."""
    print(f"[gpu] class-blocked vs per-tile {dt} nvec={nvec}", flush=True)
    eps = 2.0 ** -23 if dt in ("f32", "c64") else 1e-13
    for name in ("spin19", "hubbard_4x2"):
        desc, terms, st, ham = _problem(name)
        v = torch.from_numpy(uniform_vectors(len(st), list(range(3, 3 + nvec)), dt[0] == "c")).to(DT[dt]).cuda()
        v = v if nvec > 1 else v.reshape(-1).contiguous()
        out = {}
        for mode in ("2", "0"):
            monkeypatch.setenv("HPHI_SECTOR_BLOCKS", mode)
            red = torch.empty(4 * nvec, dtype=torch.float64, device="cuda")
            only = torch.empty_like(red)
            u = hp.hphi_hv(ham, v, reduce=red)
            hp.hphi_hv(ham, v, reduce=only, write=False)
            # without an output vector the last sum is that of the rounded-free result
            assert torch.equal(red, only)
            out[mode] = (u.cpu().numpy().reshape(len(st), nvec), red.cpu().numpy())
        bound = abs(oh.sparse_h(desc, terms)) @ abs(v.cpu().numpy().reshape(len(st), nvec).astype(np.complex128))
        assert np.all(abs(out["2"][0] - out["0"][0]) <= eps * bound + 1e-300)
        assert np.allclose(out["2"][1], out["0"][1], rtol=1e-11, atol=1e-11 * np.max(abs(out["0"][1])))


def test_class_blocked_declines_what_it_cannot_take():
    """Complex elements, row conditions and tables larger than the vector stay with the per-tile kernel:
    same results as the oracle."""
    print("[gpu] class-blocked declines", flush=True)
    n = 24   # 20 low bits: lists of 2^20 low halves for 276 rows
    for desc, terms in (
            (BasisDesc("spin", 10, "sz", two_sz=0), L.random_spin_terms(10, 14, 75, conserve_sz=True, real=False)),
            (BasisDesc("fermion", 5, "nupndn", n_up=2, n_dn=2), [L.green2_term(0, 2, 5, 7)] + L.hubbard_terms(L.rect_bonds(5, 1), 5, 1.0, 4.0)),
            (BasisDesc("spin", n, "sz", two_sz=n - 4, split_bits=20), [L.heisenberg_bond(i, (i + 1) % n) for i in range(n)])):
        st = ob.states(desc)
        v = uniform_vectors(len(st), [9], True)
        ham = hp.hphi_ham_build(hp.hphi_basis_build(desc), terms)
        u = hp.hphi_hv(ham, torch.from_numpy(v[:, 0].copy()).cuda()).cpu().numpy()
        ref = oh.apply_h(desc, terms, v, st)[:, 0]
        assert np.linalg.norm(u - ref) <= 1e-12 * np.linalg.norm(ref)


@pytest.mark.parametrize("k", [1, 2, 4, 8])
@pytest.mark.parametrize("name", list(CASES))
def test_class_blocked_reads_only_the_vector(monkeypatch, name, k):
    """NaN on both sides of the input vector (and in the output beforehand) does not reach the result."""
    print(f"[gpu] class-blocked stays inside {name} k={k}", flush=True)
    monkeypatch.setenv("HPHI_GROUP_K", str(k))
    desc, terms, st, ham = _problem(name)
    for dt in DT.values():
        for nvec in (1, 4):
            pad = 4096
            n = len(st) * nvec
            buf = torch.full((n + 2 * pad,), float("nan"), dtype=dt, device="cuda")
            x = torch.from_numpy(uniform_vectors(len(st), list(range(nvec)), dt.is_complex)).to(dt).cuda()
            v = buf[pad:pad + n]
            v.copy_(x.reshape(-1))
            v = v.reshape(len(st), nvec) if nvec > 1 else v
            u = hp.hphi_hv(ham, v, torch.full_like(v, float("nan")))
            red = torch.empty(4 * nvec, dtype=torch.float64, device="cuda")
            hp.hphi_hv(ham, v, reduce=red, write=False)
            assert torch.isfinite(torch.view_as_real(u) if dt.is_complex else u).all() and torch.isfinite(red).all()
            assert torch.equal(u, hp.hphi_hv(ham, x if nvec > 1 else x.reshape(-1)))
