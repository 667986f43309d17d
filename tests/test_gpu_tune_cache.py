"""Lines of a tune cache: those written before a sector Hamiltonian could run the class-blocked kernel do
not keep it from that kernel; newer ones, and those of other spaces, are used as they stand."""

import pytest
import torch

from synth import lattices as L
from synth.configs import BasisDesc

pytestmark = pytest.mark.gpu

import paper_1703_03637_amd as hp  # noqa: E402


@pytest.fixture(scope="module", autouse=True)
def _need_gpu():
    assert torch.cuda.is_available(), "GPU tests need an MI355X"


def _normal(n):
    # entries of full precision: row sums in another order differ in their last bits
    g = torch.Generator(device="cuda")
    g.manual_seed(1)
    return torch.empty(n, dtype=torch.float64, device="cuda").normal_(generator=g)


def _product(desc, terms, v):
    """H v: the last bits of its rows tell the kernels and schedules apart."""
    return hp.hphi_hv(hp.hphi_ham_build(hp.hphi_basis_build(desc), terms), v)


@pytest.mark.parametrize("line,kernel", [
    ("{key} 0 2048 1 1 0 1 0 123.45", "2"),          # seven fields: before the block-staged kernel
    ("{key} 0 2048 1 1 0 1 0 0 123.45", "2"),        # eight: per-tile, the class-blocked kernel was no candidate
    ("{key} 0 2048 1 1 0 1 0 2 123.45", "2"),        # eight, class-blocked
    ("{key} 0 2048 1 1 0 1 0 0 123.45 k2", "0"),     # per-tile, chosen beside the class-blocked kernel
    ("{key} 0 2048 1 1 0 1 0 2 123.45 k2", "2"),
])
def test_old_lines_do_not_pin_the_per_tile_kernel(monkeypatch, tmp_path, line, kernel):
    print(f"[gpu] tune cache line {line}", flush=True)
    desc = BasisDesc("spin", 18, "sz", two_sz=0)
    terms = [L.heisenberg_bond(i, (i + 1) % 18, 1.0 + 0.1 * i) for i in range(18)]
    want, v = {}, _normal(48620)
    for mode in ("0", "2"):
        monkeypatch.setenv("HPHI_SECTOR_BLOCKS", mode)
        want[mode] = _product(desc, terms, v)
    monkeypatch.delenv("HPHI_SECTOR_BLOCKS")
    assert not torch.equal(want["0"], want["2"])
    cache = tmp_path / "tune"
    monkeypatch.setenv("HPHI_TUNE_CACHE", str(cache))
    ham = hp.hphi_ham_build(hp.hphi_basis_build(desc), terms)
    hp.hphi_hv_tune(ham, v, torch.empty_like(v))
    written = cache.read_text().split()
    assert written[-1] == "k2"
    cache.write_text(line.format(key=written[0]) + "\n")
    assert torch.equal(_product(desc, terms, v), want[kernel])


def test_lines_of_full_spaces_are_used_as_they_stand(monkeypatch, tmp_path):
    """An old line of a full space: the two passes of 8 kB windows it names, not the default's one pass."""
    print("[gpu] tune cache full space", flush=True)
    desc = BasisDesc("spin", 14)
    terms = [L.kitaev_heisenberg_bond(i, (i + 1) % 14, i % 3, -1.0, 0.1) for i in range(14)]
    v = _normal(1 << 14)
    default = _product(desc, terms, v)
    monkeypatch.setenv("HPHI_L2_WINDOW_KB", "8")
    monkeypatch.setenv("HPHI_PASSES", "2")
    windows = _product(desc, terms, v)
    monkeypatch.delenv("HPHI_L2_WINDOW_KB")
    monkeypatch.delenv("HPHI_PASSES")
    cache = tmp_path / "tune"
    monkeypatch.setenv("HPHI_TUNE_CACHE", str(cache))
    ham = hp.hphi_ham_build(hp.hphi_basis_build(desc), terms)
    hp.hphi_hv_tune(ham, v, torch.empty_like(v))
    key = cache.read_text().split()[0]
    cache.write_text(f"{key} 1 8 2 1 0 1 0 0 50.00\n")
    assert not torch.equal(windows, default) and torch.equal(_product(desc, terms, v), windows)
