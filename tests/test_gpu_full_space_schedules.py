"""The default schedules of full-space products, by row width, size and how far the operators reach: the
single-pass kernel's result."""

import pytest
import torch

from synth import lattices as L
from synth.configs import BasisDesc, kh_honeycomb_terms
from synth.vectors import device_uniform

pytestmark = pytest.mark.gpu

import paper_1703_03637_amd as hp  # noqa: E402

DT = {"f32": torch.float32, "f64": torch.float64, "c64": torch.complex64, "c128": torch.complex128}


@pytest.fixture(scope="module", autouse=True)
def _need_gpu():
    assert torch.cuda.is_available(), "GPU tests need an MI355X"


def _xyz(bonds):
    return [L.Term(L.SPIN_BOND, i, j, (1.0, 0, 0, 0, 0.7, 0, 0, 0, 0.4)) for i, j in bonds]


CASES = {
    # live in every row, many operators beyond a window: three passes of 2 MB, one pass below 16 MB
    "xyz_triangular20": (BasisDesc("spin", 20), lambda: _xyz(L.triangular_bonds(5, 4))),
    "xyz_triangular18": (BasisDesc("spin", 18), lambda: _xyz(L.triangular_bonds(6, 3))),
    "kitaev20": (BasisDesc("spin", 20), lambda: kh_honeycomb_terms(lx=2, ly=5)),
    # conserving: one pass in and beyond the memory-side cache
    "chain20": (BasisDesc("spin", 20), lambda: [L.heisenberg_bond(i, j) for i, j in L.chain_bonds(20)]),
    "hubbard11": (BasisDesc("fermion", 11), lambda: L.hubbard_terms(L.rect_bonds(11, 1), 11, t=1.0, U=8.0)),
    # single flips (fields) beside the bonds
    "ising19": (BasisDesc("spin", 19), lambda: [L.xxz_bond(i, (i + 1) % 19, 0.0, 1.0) for i in range(19)]
                + [L.Term(L.SPIN_FIELD, i, -1, (0.6, 0.0, 0.1)) for i in range(19)]),
}


@pytest.mark.parametrize("dt,nvec", [("f64", 1), ("c128", 2), ("c64", 4), ("f64", 8), ("c64", 16), ("f32", 8)])
@pytest.mark.parametrize("name", list(CASES))
def test_default_schedule_matches_single_pass(monkeypatch, name, dt, nvec):
    """Outputs and sums up to rounding: FP64 1e-13, FP32 storage two roundings and one of each partial sum that
    passes hand on (4 * 2^-24), times the row sums of |H| (under 60) and the largest entry."""
    print(f"[gpu] default schedule {name} {dt} nvec={nvec}", flush=True)
    desc, mk = CASES[name]
    if name == "hubbard11" and nvec > 4:
        nvec = 4
    ham = hp.hphi_ham_build(hp.hphi_basis_build(desc), mk())
    x = device_uniform(ham.dim, 0 if nvec == 1 else nvec, 5, DT[dt].is_complex, DT[dt])
    red = [torch.empty(4 * nvec, dtype=torch.float64, device="cuda") for _ in range(2)]
    a = hp.hphi_hv(ham, x, a=-0.1, b=1.5, reduce=red[0])
    monkeypatch.setenv("HPHI_WINDOWED", "0")
    b = hp.hphi_hv(ham, x, a=-0.1, b=1.5, reduce=red[1])
    eps = 4 * 2.0 ** -24 if dt in ("f32", "c64") else 1e-13
    top = float((torch.view_as_real(x) if x.dtype.is_complex else x).abs().max())
    assert float((a - b).abs().max()) <= eps * (0.1 * 60 + 1.5) * 2 * top
    xx = float(red[1][:nvec].max())
    assert float((red[0] - red[1]).abs().max()) <= max(eps, 1e-12) * 60 ** 2 * xx
