"""Edges of the class-blocked sector product: values that are not finite beside its padding, and the
groups of high halves and lanes per row it is launched with."""

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

DT = {"f64": torch.float64, "f32": torch.float32, "c128": torch.complex128, "c64": torch.complex64}


@pytest.fixture(scope="module", autouse=True)
def _need_gpu():
    assert torch.cuda.is_available(), "GPU tests need an MI355X"


# lists inside the high half of unequal length: a chain leaves 1 to 8 of 9 operators live there
CHAIN = (BasisDesc("spin", 19, "sz", two_sz=1, split_bits=10),
         [L.heisenberg_bond(i, (i + 1) % 19, 1.0 + 0.1 * i) for i in range(19)])
HUBBARD = (BasisDesc("fermion", 8, "nupndn", n_up=4, n_dn=3, split_bits=8),
           L.hubbard_terms(L.rect_bonds(4, 2), 8, t=1.0, U=8.0))


@pytest.mark.parametrize("k", [1, 2, 4, 8])
@pytest.mark.parametrize("dt,nvec", [("f64", 1), ("f32", 2), ("c128", 1), ("c64", 4), ("f32", 16), ("c128", 16)])
@pytest.mark.parametrize("problem", [CHAIN, HUBBARD], ids=["chain19", "hubbard4x2"])
def test_infinite_entries_give_the_oracle_s_rows(monkeypatch, problem, dt, nvec, k):
    """Inf entries: H v, row by row, is what the row's own elements make of them -- infinite where one
    infinite partner has a nonzero element, not NaN because a padded list read it with a zero one."""
    print(f"[gpu] infinite entries {dt} nvec={nvec} k={k}", flush=True)
    monkeypatch.setenv("HPHI_GROUP_K", str(k))
    desc, terms = problem
    st = ob.states(desc)
    H = oh.sparse_h(desc, terms, st).real.tocsr()
    dim = len(st)
    v = uniform_vectors(dim, list(range(nvec)), False)
    bad = [dim // 7, dim // 2, dim - 1]
    v[bad] = np.inf
    x = torch.from_numpy(v).cuda().to(DT[dt])       # real parts only: complex rows carry zero imaginary parts
    if x.dtype.is_complex:
        x = torch.complex(torch.from_numpy(v), torch.zeros(v.shape, dtype=torch.float64)).to(DT[dt]).cuda()
    ham = hp.hphi_ham_build(hp.hphi_basis_build(desc), terms)
    # a = 1, b = 2: no 0 * Inf in the update itself
    u = hp.hphi_hv(ham, x if nvec > 1 else x.reshape(-1), a=1.0, b=2.0)
    got = (torch.view_as_real(u)[..., 0] if u.dtype.is_complex else u).cpu().numpy().reshape(dim, nvec)
    want = np.zeros((dim, nvec))
    with np.errstate(invalid="ignore"):
        for r in range(dim):
            c = H.indices[H.indptr[r]:H.indptr[r + 1]]
            e = H.data[H.indptr[r]:H.indptr[r + 1]]
            live = e != 0
            h = (e[live, None] * v[c[live]]).sum(0)
            if r in bad and not np.any(live & (c == r)):
                h = h + np.nan                       # the diagonal is always taken: 0 * Inf
            want[r] = h + 2.0 * v[r]
    assert np.array_equal(np.isnan(got), np.isnan(want))
    assert np.array_equal(np.isinf(got), np.isinf(want)) and np.array_equal(got[np.isinf(got)], want[np.isinf(want)])


def _vectors(dim, nvec, dt, seed=3):
    x = torch.from_numpy(uniform_vectors(dim, list(range(seed, seed + nvec)), dt[0] == "c")).to(DT[dt]).cuda()
    return x if nvec > 1 else x.reshape(-1).contiguous()


@pytest.mark.parametrize("k", [1, 2, 4, 8])
@pytest.mark.parametrize("nvec", [1, 2, 4, 8, 16])
@pytest.mark.parametrize("dt", list(DT))
@pytest.mark.parametrize("problem", [CHAIN, HUBBARD], ids=["chain19", "hubbard4x2"])
def test_every_group_size_matches_the_per_tile_kernel(monkeypatch, problem, dt, nvec, k):
    """Each storage type, batch and number of high halves: the per-tile kernel's result up to one rounding of
    each stored value (two of 2^-24 in FP32) and the order of an FP64 sum (1e-13), times |H||v|."""
    print(f"[gpu] group size {k} {dt} nvec={nvec}", flush=True)
    desc, terms = problem
    ham = hp.hphi_ham_build(hp.hphi_basis_build(desc), terms)
    v = _vectors(ham.dim, nvec, dt)
    out = []
    for mode, group in (("2", str(k)), ("0", "")):
        monkeypatch.setenv("HPHI_SECTOR_BLOCKS", mode)
        monkeypatch.setenv("HPHI_GROUP_K", group)
        out.append(hp.hphi_hv(ham, v, a=-0.4, b=0.3).cpu().numpy().reshape(ham.dim, nvec))
    a = abs(v.cpu().numpy().reshape(ham.dim, nvec).astype(np.complex128))
    bound = (2.0 ** -23 if dt in ("f32", "c64") else 1e-13) * (0.4 * abs(oh.sparse_h(desc, terms)) @ a + 0.3 * a)
    assert np.all(abs(out[0] - out[1]) <= bound)


def _torus(lx, ly, up):
    n = lx * ly
    return BasisDesc("spin", n, "sz", two_sz=2 * up - n), [L.heisenberg_bond(i, j) for i, j in L.triangular_bonds(lx, ly)]


# the shapes the default chooses: twice the lanes per row (3,280 wavefront items), two high halves of
# four scalars, one, and eight lanes per row
@pytest.mark.parametrize("lx,ly,up", [(5, 4, 10), (5, 4, 7), (6, 3, 9), (5, 5, 5)])
@pytest.mark.parametrize("dt,nvec", [("f64", 4), ("f64", 8), ("c128", 4), ("f64", 16), ("c128", 8), ("c64", 16), ("c128", 16), ("f32", 1)])
def test_default_shapes_match_the_per_tile_kernel(monkeypatch, lx, ly, up, dt, nvec):
    """The default's product and sums on sectors around the limits of the shape rule (bounds as above; sums 1e-12)."""
    print(f"[gpu] default shape {lx}x{ly} up={up} {dt} nvec={nvec}", flush=True)
    desc, terms = _torus(lx, ly, up)
    ham = hp.hphi_ham_build(hp.hphi_basis_build(desc), terms)
    v = _vectors(ham.dim, nvec, dt)
    out = []
    for mode in ("2", "0"):
        monkeypatch.setenv("HPHI_SECTOR_BLOCKS", mode)
        red = torch.empty(4 * nvec, dtype=torch.float64, device="cuda")
        out.append((hp.hphi_hv(ham, v, reduce=red).cpu().numpy().reshape(ham.dim, nvec), red.cpu().numpy()))
    # every |H| element is 1/4 or 1/2, at most 3 per site each
    bound = (2.0 ** -23 if dt in ("f32", "c64") else 1e-13) * 0.75 * 3 * lx * ly
    assert np.max(abs(out[0][0] - out[1][0])) <= bound * float(v.abs().max())
    assert np.all(abs(out[0][1] - out[1][1]) <= 1e-12 * (0.75 * 3 * lx * ly) ** 2 * out[1][1][:nvec].max())


@pytest.mark.parametrize("desc_terms,dt,nvec", [
    (_torus(5, 4, 10), "c64", 4),
    ((BasisDesc("spin", 24, "sz", two_sz=0), [L.heisenberg_bond(i, j) for i, j in L.kagome_bonds(4, 2)]), "f64", 8),
], ids=["triangular20_c64x4", "kagome24_f64x8"])
def test_dense_sectors_of_wide_rows_keep_the_per_tile_kernel(monkeypatch, desc_terms, dt, nvec):
    """Sectors that the default leaves to the per-tile kernel: its bits, and they are not the other kernel's."""
    print(f"[gpu] dense sector {dt} nvec={nvec}", flush=True)
    desc, terms = desc_terms
    ham = hp.hphi_ham_build(hp.hphi_basis_build(desc), terms)
    g = torch.Generator(device="cuda")
    g.manual_seed(7)
    v = torch.empty((ham.dim, nvec), dtype=DT[dt], device="cuda")
    (torch.view_as_real(v) if v.dtype.is_complex else v).normal_(generator=g)
    out = {}
    for mode in ("", "0", "2"):
        monkeypatch.setenv("HPHI_SECTOR_BLOCKS", mode)
        red = torch.empty(4 * nvec, dtype=torch.float64, device="cuda")
        out[mode] = (hp.hphi_hv(ham, v, reduce=red), red)
    assert torch.equal(out[""][0], out["0"][0]) and torch.equal(out[""][1], out["0"][1])
    assert not torch.equal(out["2"][1], out["0"][1])


@pytest.mark.parametrize("k", [2, 4, 8])
@pytest.mark.parametrize("dt", ["f64", "c64"])
def test_batched_fermion_lanczos_matches_single_problems(monkeypatch, dt, k):
    """Several fermion sectors in one batched recurrence, at each number of high halves: alpha, beta and energies
    of the problems run one by one (rounding of 12 steps: 1e-10 in FP64, 1e-4 in FP32 storage)."""
    print(f"[gpu] batched fermion lanczos {dt} k={k}", flush=True)
    monkeypatch.setenv("HPHI_GROUP_K", str(k))
    terms = L.hubbard_terms(L.rect_bonds(4, 2), 8, t=1.0, U=8.0)
    hams = [hp.hphi_ham_build(hp.hphi_basis_build(BasisDesc("fermion", 8, "nupndn", n_up=u, n_dn=d)), terms)
            for u, d in ((4, 4), (3, 4), (2, 3))]
    v = [_vectors(h.dim, 1, dt, 20 + i) for i, h in enumerate(hams)]
    batch = hp.hphi_lanczos(hams, v, 12)
    for h, x, b in zip(hams, v, batch):
        one = hp.hphi_lanczos([h], [x], 12)[0]
        tol = 1e-10 if dt == "f64" else 1e-4
        assert np.allclose(b["alpha"], one["alpha"], rtol=0, atol=tol * 40) and np.allclose(b["beta"], one["beta"], rtol=0, atol=tol * 40)
        assert abs(b["e0_refined"] - one["e0_refined"]) <= tol * 40


@pytest.mark.parametrize("two_sz,split,blocked", [(-12, 8, True), (-10, 8, False)])
def test_tables_are_counted_as_they_are_allocated(monkeypatch, two_sz, split, blocked):
    """26 spins with 18 high bits: the partner lists take 8 bytes per operator inside the high half, 16 MB with
    the rest at 7 up (657,800 rows).  Counted at 16 bytes the space would be left to the per-tile kernel.  The rows
    differ from that kernel's in the last bits only (1e-13 of sums of up to 26 elements of 0.5 and a diagonal).
    At 8 up the tables are 27 MB, more than half of the 12 MB vector, and the per-tile kernel stays."""
    print(f"[gpu] class-blocked table rule 2Sz={two_sz} split={split}", flush=True)
    desc = BasisDesc("spin", 26, "sz", two_sz=two_sz, split_bits=split)
    terms = [L.heisenberg_bond(i, (i + 1) % 26) for i in range(26)]
    out = []
    for blocks in (None, "0"):
        if blocks:
            monkeypatch.setenv("HPHI_SECTOR_BLOCKS", blocks)
        ham = hp.hphi_ham_build(hp.hphi_basis_build(desc), terms)
        g = torch.Generator(device="cuda")
        g.manual_seed(5)
        v = torch.empty(ham.dim, dtype=torch.float64, device="cuda").normal_(generator=g)
        out.append(hp.hphi_hv(ham, v))
    assert float((out[0] - out[1]).abs().max()) <= 1e-13 * 26 * float(v.abs().max())
    assert torch.equal(out[0], out[1]) != blocked


SPARSE = {
    "triangular24_up6": _torus(6, 4, 6), "triangular25_up5": _torus(5, 5, 5),
    "hubbard4x3_3_3": (BasisDesc("fermion", 12, "nupndn", n_up=3, n_dn=3), L.hubbard_terms(L.rect_bonds(4, 3), 12, t=1.0, U=8.0)),
    "hubbard7x2_2_2": (BasisDesc("fermion", 14, "nupndn", n_up=2, n_dn=2),
                       L.hubbard_terms([b for b in L.rect_bonds(7, 2) if b[0] != b[1]], 14, t=1.0, U=8.0)),
}


@pytest.mark.parametrize("dt,nvec", [("c128", 2), ("f64", 8), ("c128", 8), ("c128", 16)])
@pytest.mark.parametrize("name", list(SPARSE))
def test_default_shapes_of_sparse_sectors_match_the_per_tile_kernel(monkeypatch, name, dt, nvec):
    """Sectors with few rows to a tile have shapes of their own (1e-13 of the row sums of |H|: 0.75 per spin bond; for
    fermions at most 4 hops of 1 per particle and U = 8 on at most 3 sites)."""
    print(f"[gpu] sparse default shape {name} {dt} nvec={nvec}", flush=True)
    desc, terms = SPARSE[name]
    ham = hp.hphi_ham_build(hp.hphi_basis_build(desc), terms)
    v = _vectors(ham.dim, nvec, dt)
    out = []
    for mode in ("2", "0"):
        monkeypatch.setenv("HPHI_SECTOR_BLOCKS", mode)
        red = torch.empty(4 * nvec, dtype=torch.float64, device="cuda")
        out.append((hp.hphi_hv(ham, v, reduce=red).cpu().numpy().reshape(ham.dim, nvec), red.cpu().numpy()))
    row = 0.75 * 75 if desc.particle == "spin" else 4 * 6 + 8 * 3
    assert np.max(abs(out[0][0] - out[1][0])) <= 1e-13 * row * float(v.abs().max())
    assert np.all(abs(out[0][1] - out[1][1]) <= 1e-12 * row ** 2 * out[1][1][:nvec].max())
