"""Runs long enough to replay a captured graph of 32 steps (from 513 steps on): step for step the same bits
as the runs that launch every step, with a remainder behind the last replay, and the progress lines of both."""

import re

import numpy as np
import pytest
import torch

from synth import lattices as L
from synth.configs import BasisDesc
from synth.vectors import uniform_vectors

pytestmark = pytest.mark.gpu

import paper_1703_03637_amd as hp  # noqa: E402


@pytest.fixture(scope="module", autouse=True)
def _need_gpu():
    assert torch.cuda.is_available(), "GPU tests need an MI355X"


def _chain(n, z=0.0):
    return [L.Term(L.SPIN_BOND, i, (i + 1) % n, (1.0, z, 0, -z, 1.0, 0, 0, 0, 1.0)) for i in range(n)]


def _sz(n, m2):
    return BasisDesc("spin", n, "sz", two_sz=m2)


HUB = L.hubbard_terms(L.rect_bonds(4, 2), 8, t=1.0, U=4.0)
# class-blocked, per-tile (complex elements), windowed
SINGLE = {"classes": (_sz(16, 0), _chain(16), torch.float64), "classes_f32": (_sz(14, 0), _chain(14), torch.float32),
          "tiles": (_sz(14, 0), _chain(14, 0.3), torch.complex128), "windowed": (BasisDesc("spin", 12), _chain(12), torch.float64),
          "hubbard": (BasisDesc("fermion", 8, "nupndn", n_up=4, n_dn=4), HUB, torch.complex128)}


def _start(ham, dt, seed):
    return torch.from_numpy(uniform_vectors(ham.dim, [seed], dt.is_complex)[:, 0].copy()).to(dt).cuda()


def _same(a, b):
    assert np.array_equal(a["alpha"], b["alpha"]) and np.array_equal(a["beta"], b["beta"])
    assert a["e0_refined"] == b["e0_refined"] and torch.equal(a["x"], b["x"])


@pytest.mark.parametrize("n_iter", [512, 513, 545, 578])
@pytest.mark.parametrize("name", list(SINGLE))
def test_long_lanczos_replays_the_same_steps(name, n_iter):
    """alpha, beta, the refined energy and the eigenvector of the replayed run are those of the launched one.
    (The recurrence goes on: a tiny breakdown tolerance, and rounding keeps beta above it.)"""
    print(f"[gpu] long lanczos {name} {n_iter}", flush=True)
    desc, terms, dt = SINGLE[name]
    ham = hp.hphi_ham_build(hp.hphi_basis_build(desc), terms)
    v = _start(ham, dt, 3)
    runs = [hp.hphi_lanczos([ham], [v], n_iter, use_graph=g, breakdown_tol=1e-300)[0] for g in (True, False, True)]
    assert len(runs[0]["alpha"]) >= min(n_iter, 513)
    _same(runs[0], runs[1])
    _same(runs[0], runs[2])


@pytest.mark.parametrize("kind", ["classes", "tiles", "mixed"])
def test_long_batched_lanczos_replays_the_same_steps(kind):
    """A batched recurrence of 545 steps whose smallest problem ends inside the first replay (its space has 20
    rows): all problems as in the launched run.  mixed: only some have the class-blocked tables, so the
    batch runs on the per-tile kernel."""
    print(f"[gpu] long batched lanczos {kind}", flush=True)
    z = 0.3 if kind == "tiles" else 0.0
    dt = torch.complex128 if z else torch.float64
    descs = [(_sz(14, 0), 14), (_sz(6, 0), 6), (_sz(13, 1), 13)]
    if kind == "mixed":      # 20 low bits: tables of 2^20 low halves for 276 rows are not built
        descs[2] = (BasisDesc("spin", 24, "sz", two_sz=20, split_bits=20), 24)
    hams = [hp.hphi_ham_build(hp.hphi_basis_build(d), _chain(n, z)) for d, n in descs]
    v = [_start(h, dt, 5 + i) for i, h in enumerate(hams)]
    a, b = (hp.hphi_lanczos(hams, v, 545, use_graph=g, breakdown_tol=1e-300) for g in (True, False))
    for x, y, h in zip(a, b, hams):
        assert len(x["alpha"]) <= h.dim
        _same(x, y)
    assert len(a[0]["alpha"]) >= 513 and len(a[1]["alpha"]) <= 20


@pytest.mark.parametrize("use_graph", [False, True])
def test_progress_lines_come_every_n_steps(monkeypatch, capfd, use_graph):
    """HPHI_PROGRESS=N: a line at every Nth step of a launched run, and at the first replay's end behind it of a
    replayed one; never more often."""
    print(f"[gpu] progress use_graph={use_graph}", flush=True)
    ham = hp.hphi_ham_build(hp.hphi_basis_build(_sz(14, 0)), _chain(14))
    v = _start(ham, torch.float64, 1)

    def steps(n_iter, every):
        monkeypatch.setenv("HPHI_PROGRESS", str(every))
        capfd.readouterr()
        hp.hphi_lanczos([ham], [v], n_iter, use_graph=use_graph, refine=False, breakdown_tol=1e-300)
        return [int(k) for k in re.findall(r"step (\d+) of", capfd.readouterr().err)]

    assert steps(40, 7) == [7, 14, 21, 28, 35]
    assert steps(41, 1) == list(range(2, 42))      # the first step is launched before the loop
    long = steps(600, 150)
    if use_graph:
        assert len(long) == 4 and all(150 * (i + 1) <= k < 150 * (i + 1) + 32 for i, k in enumerate(long))
    else:
        assert long == [150, 300, 450, 600]
