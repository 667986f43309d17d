"""Element lists of sector products in windows of rows, batched launches, and the per-tile kernel's own paths
where the class-blocked kernel is the default: exports by table placement and lanes, batched recurrences."""

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


@pytest.mark.parametrize("stage", ["0", "1", "2"])
@pytest.mark.parametrize("lpr,nvec", [("1", 1), ("1", 2), ("2", 2), ("4", 4), ("2", 8), ("8", 8), ("4", 16)])
@pytest.mark.parametrize("name", list(SECTORS))
def test_per_tile_kernel_by_tables_and_lanes(monkeypatch, name, lpr, nvec, stage):
    """The per-tile kernel of real sector Hamiltonians with its tables in LDS or in memory and each split of a
    row: its element list and its product are the oracle's (1e-12 of |H||v| per element)."""
    print(f"[gpu] per-tile {name} lanes={lpr} nvec={nvec} tables={stage}", flush=True)
    for k, v in (("HPHI_SECTOR_BLOCKS", "0"), ("HPHI_LPR", lpr), ("HPHI_STAGE_TABLES", stage)):
        monkeypatch.setenv(k, v)
    desc, mk = SECTORS[name]
    terms = mk()
    H = oh.sparse_h(desc, terms).real.tocsr()
    ham = hp.hphi_ham_build(hp.hphi_basis_build(desc), terms)
    _same_as_matrix(_lists(ham, ham.dim // 4, 150, nvec), H, ham.dim // 4)
    for cplx in (False, True):
        v = uniform_vectors(ham.dim, list(range(nvec)), cplx)
        x = torch.from_numpy(v).cuda()
        red = torch.empty(4 * nvec, dtype=torch.float64, device="cuda")
        u = hp.hphi_hv(ham, x if nvec > 1 else x.reshape(-1), reduce=red).cpu().numpy().reshape(v.shape)
        assert np.all(abs(u - H @ v) <= 1e-12 * (abs(H) @ abs(v) + 1e-300))
        want = np.concatenate([np.sum(abs(v) ** 2, 0), np.sum((v.conj() * (H @ v)).real, 0), np.sum(abs(H @ v) ** 2, 0)])
        assert np.all(abs(red.cpu().numpy()[:3 * nvec] - want) <= 1e-11 * np.sum((abs(H) @ abs(v)) ** 2 + abs(v) ** 2))


@pytest.mark.parametrize("dt", ["f64", "c64"])
def test_batched_per_tile_recurrence(monkeypatch, dt):
    """Several real sectors in one batched recurrence of the per-tile kernel: the problems run one by one
    (rounding of 10 steps: 1e-10 in FP64, 1e-4 in FP32 storage, of energies up to 10)."""
    print(f"[gpu] batched per-tile lanczos {dt}", flush=True)
    monkeypatch.setenv("HPHI_SECTOR_BLOCKS", "0")
    terms = [L.heisenberg_bond(i, j) for i, j in L.triangular_bonds(4, 3)]
    hams = [hp.hphi_ham_build(hp.hphi_basis_build(BasisDesc("spin", 12, "sz", two_sz=m)), terms) for m in (0, 2, 6)]
    tdt = {"f64": torch.float64, "c64": torch.complex64}[dt]
    v = [torch.from_numpy(uniform_vectors(h.dim, [i], tdt.is_complex)[:, 0].copy()).to(tdt).cuda() for i, h in enumerate(hams)]
    batch = hp.hphi_lanczos(hams, v, 10)
    tol = 10 * (1e-10 if dt == "f64" else 1e-4)
    for h, x, b in zip(hams, v, batch):
        one = hp.hphi_lanczos([h], [x], 10)[0]
        assert np.allclose(b["alpha"], one["alpha"], rtol=0, atol=tol) and np.allclose(b["beta"], one["beta"], rtol=0, atol=tol)
        assert abs(b["e0_refined"] - one["e0_refined"]) <= tol


def test_a_batch_of_unlike_tables_runs_per_tile():
    """A batch in which one problem has no class-blocked tables (20 low bits for 276 rows): each problem's
    energies as by itself."""
    print("[gpu] batched lanczos, one problem without tables", flush=True)
    hams = [hp.hphi_ham_build(hp.hphi_basis_build(BasisDesc("spin", 14, "sz", two_sz=0)), [L.heisenberg_bond(i, (i + 1) % 14) for i in range(14)]),
            hp.hphi_ham_build(hp.hphi_basis_build(BasisDesc("spin", 24, "sz", two_sz=20, split_bits=20)),
                              [L.heisenberg_bond(i, (i + 1) % 24) for i in range(24)])]
    v = [torch.from_numpy(uniform_vectors(h.dim, [i], False)[:, 0].copy()).cuda() for i, h in enumerate(hams)]
    batch = hp.hphi_lanczos(hams, v, 12)
    for h, x, b in zip(hams, v, batch):
        one = hp.hphi_lanczos([h], [x], 12)[0]
        assert np.allclose(b["alpha"], one["alpha"], rtol=0, atol=1e-9) and abs(b["e0_refined"] - one["e0_refined"]) <= 1e-9


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
