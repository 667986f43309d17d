"""Element lists of sector products in windows of rows."""

import numpy as np
import pytest
import torch

from oracle import basis as ob
from oracle import hamiltonian as oh
from synth import lattices as L
from synth.configs import BasisDesc

pytestmark = pytest.mark.gpu

import paper_1703_03637_amd as hp  # noqa: E402


@pytest.fixture(scope="module", autouse=True)
def _need_gpu():
    assert torch.cuda.is_available(), "GPU tests need an MI355X"


SECTORS = {
    "spin": (BasisDesc("spin", 14, "sz", two_sz=2), lambda: L.random_spin_terms(14, 26, 31, conserve_sz=True, fields=True, real=True)),
    "spin_split4": (BasisDesc("spin", 12, "sz", two_sz=0, split_bits=4), lambda: [L.heisenberg_bond(i, (i + 1) % 12) for i in range(12)]),
    "nupndn": (BasisDesc("fermion", 7, "nupndn", n_up=3, n_dn=4),
               lambda: L.random_fermion_terms(7, 20, 32, conserve_spin=True, n_dens=7, with_mu=True)),
    "ntot": (BasisDesc("fermion", 6, "ntot", n_tot=5), lambda: L.random_fermion_terms(6, 18, 33, conserve_spin=False, n_dens=5, with_mu=True)),
}


def _lists(ham, row0, nrows, nvec=1):
    cols, re, im, term, cnt = (t.cpu().numpy() for t in hp.hphi_hv_elements(ham, row0, nrows, 64, nvec=nvec))
    out = []
    for r in range(nrows):
        n = cnt[r]
        assert n <= 64 and not im[r, :n].any()
        out.append((cols[r, :n].tolist(), re[r, :n].tolist(), term[r, :n].tolist()))
    return out


def _same_as_matrix(lists, H, row0):
    for r, (cols, re, _) in enumerate(lists):
        got = np.zeros(H.shape[0])
        np.add.at(got, cols, re)
        assert np.max(abs(got - H[row0 + r].toarray().ravel())) <= 1e-13


@pytest.mark.parametrize("name", list(SECTORS))
def test_windows_of_rows_are_parts_of_the_whole_list(monkeypatch, name):
    """Windows at the ends, across high halves and of one row hold the whole list's entries; the list is the
    oracle's matrix, and the per-tile kernel's list up to the last bits of the diagonal."""
    print(f"[gpu] element windows {name}", flush=True)
    desc, mk = SECTORS[name]
    terms = mk()
    H = oh.sparse_h(desc, terms).real.tocsr()
    ham = hp.hphi_ham_build(hp.hphi_basis_build(desc), terms)
    dim = ham.dim
    whole = _lists(ham, 0, dim)
    _same_as_matrix(whole, H, 0)
    for row0, n in ((0, 1), (0, 65), (dim // 3, 200), (dim // 2 - 7, 64), (dim - 130, 130), (dim - 1, 1)):
        assert _lists(ham, row0, n) == whole[row0:row0 + n]
    monkeypatch.setenv("HPHI_SECTOR_BLOCKS", "0")
    tiles = _lists(hp.hphi_ham_build(hp.hphi_basis_build(desc), terms), 0, dim)
    for a, b in zip(whole, tiles):
        assert a[0] == b[0] and a[2] == b[2] and np.allclose(a[1], b[1], rtol=0, atol=1e-13)


def test_batched_launches_follow_the_blocks_per_cu(monkeypatch):
    """HPHI_BLOCKS_PER_CU reaches the batched class-blocked launch: the block sums are added in another order,
    so the last bits of alpha change, and nothing else."""
    print("[gpu] batched lanczos, blocks per CU", flush=True)
    terms = [L.heisenberg_bond(i, (i + 1) % 20) for i in range(20)]
    hams = [hp.hphi_ham_build(hp.hphi_basis_build(BasisDesc("spin", 20, "sz", two_sz=m)), terms) for m in (0, 2)]
    g = torch.Generator(device="cuda")
    g.manual_seed(3)
    v = [torch.empty(h.dim, dtype=torch.float64, device="cuda").normal_(generator=g) for h in hams]
    wide = hp.hphi_lanczos(hams, v, 8, refine=False)
    monkeypatch.setenv("HPHI_BLOCKS_PER_CU", "1")
    narrow = hp.hphi_lanczos(hams, v, 8, refine=False)
    for a, b in zip(wide, narrow):
        assert np.allclose(a["alpha"], b["alpha"], rtol=0, atol=1e-11)
    assert any(not np.array_equal(a["alpha"], b["alpha"]) for a, b in zip(wide, narrow))
