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
