"""Performance cases: the calls that programs make of this library, over the range of sizes they make them at.

A case is a plain dict.  ``model``/``lattice``/``lx``/``ly`` name the Hamiltonian, ``two_sz`` or ``n_up``/``n_dn`` the
sector (absent: the full space), ``dtype`` and ``nvec`` the stored vectors, ``kind`` the entry point that is called.
Handles are used as built (no tuning), which is what a program gets that only follows the README.
"""

import math

import numpy as np
import torch

import paper_1703_03637_amd as hp
from synth import lattices as L
from synth.configs import BasisDesc, kh_honeycomb_terms

DTYPES = {"f32": torch.float32, "f64": torch.float64, "c64": torch.complex64, "c128": torch.complex128}


def listed():
    return [
        # 8-site Hubbard cluster compared with full diagonalization: 16 samples of 4,900 rows, launch latency only
        dict(name="hubbard8_tpq_step", kind="tpq_step", model="hubbard", lattice="super", lx=2, ly=2, n_up=4, n_dn=4,
             dtype="c128", nvec=16),
        # Heisenberg chain, full 2^16 space: a short FP64 Lanczos with its second pass, microseconds per step
        dict(name="heis_chain16_lanczos", kind="lanczos", model="heis", lattice="chain", lx=16, ly=1, dtype="c128",
             n_iter=24),
        # open 4x3 Hubbard cluster at half filling (853,776 rows): a ground state with its second pass
        dict(name="hubbard4x3_lanczos", kind="lanczos", model="hubbard", lattice="rect", lx=4, ly=3, n_up=6, n_dn=6,
             dtype="c128", n_iter=24),
        # the same cluster: measuring a list of one- and two-body correlations in a state that is at hand
        dict(name="hubbard4x3_expect", kind="expect", model="hubbard", lattice="rect", lx=4, ly=3, n_up=6, n_dn=6,
             dtype="c128", nvec=1, n_obs=12),
        # the same cluster: inverse iteration of an approximate eigenvector (a fixed number of CG steps)
        dict(name="hubbard4x3_cg", kind="cg", model="hubbard", lattice="rect", lx=4, ly=3, n_up=6, n_dn=6,
             dtype="f64", n_iter=24, e_approx=-5.4),
        # 18-site Kitaev-Heisenberg honeycomb, 4 samples: a stretch of a TPQ trajectory replayed as graphs
        dict(name="kh18_tpq_run", kind="tpq_run", model="kh", lattice="honeycomb", lx=3, ly=3, dtype="c64", nvec=4,
             n_iter=40),
        # 24-site Kitaev-Heisenberg honeycomb: the batched mixed-precision TPQ step of 16 samples
        dict(name="kh24_tpq_b16_c64", kind="tpq_step", model="kh", lattice="honeycomb", lx=3, ly=4, dtype="c64", nvec=16),
        # and the plain FP64 step of one sample
        dict(name="kh24_tpq_c128", kind="tpq_step", model="kh", lattice="honeycomb", lx=3, ly=4, dtype="c128", nvec=1),
        # 24-site triangular torus: the Sz sectors 0 to 10 (2,704,156 rows down to 276; the last two are smaller than the
        # recurrence is long) as one batched FP32 Lanczos
        dict(name="tri24_allsz_lanczos", kind="lanczos", model="heis", lattice="tri", lx=6, ly=4, sectors=11, dtype="f32",
             n_iter=16),
        # 27-site kagome torus at Sz = 1/2 (20,058,300 rows, an odd number of bits): one FP64 product with its sums
        dict(name="kagome27_hv_f64", kind="hv", model="heis", lattice="kagome", lx=3, ly=3, two_sz=1, dtype="f64", nvec=1),
        # 36-site kagome torus in a magnetized sector (1,251,677,700 rows, 36-bit configurations): one FP32 product
        dict(name="kagome36_sz6_hv_f32", kind="hv", model="heis", lattice="kagome", lx=3, ly=4, two_sz=12, dtype="f32",
             nvec=1),
        # 18-site Hubbard cluster away from half filling (344,622,096 rows): four complex64 samples in one TPQ step
        dict(name="hubbard18_tpq_b4_c64", kind="tpq_step", model="hubbard", lattice="super", lx=3, ly=3, n_up=6, n_dn=6,
             dtype="c64", nvec=4),
    ]


def draw(rng):
    """One more case of these ranges: another lattice, sector, storage type, batch and entry point."""
    while True:
        c = _draw(rng)
        dim = sum(_dims(c))
        words = dim * c.get("nvec", 1) * torch.empty(0, dtype=DTYPES[c["dtype"]]).element_size() // 4
        passes = 2 * c.get("n_iter", 1) if c["kind"] != "tpq_run" else c["n_iter"]
        if c["kind"] in ("hv", "tpq_step", "expect"):
            passes = max(1, c.get("n_obs", 1))
        # a short recurrence on a space of few distinct energies ends in rounding noise: those have a few thousand rows
        few = 2000 if c["kind"] in ("lanczos", "cg") else 2
        if dim >= few and words * passes <= 600_000_000 and words <= 500_000_000:
            return c


def _draw(rng):
    model = rng.choice(("heis", "heis", "hubbard", "hubbard", "kh"))
    dtype = rng.choice(("f32", "f64", "c64", "c128"))
    nvec = rng.choice((1, 1, 1, 2, 4, 8, 16))
    if model == "kh":
        n = int(round(2 ** rng.uniform(math.log2(8), math.log2(26)))) // 2 * 2
        shapes = [(a, n // 2 // a) for a in (1, 2, 3, 4) if (n // 2) % a == 0 and n // 2 // a >= 1]
        lx, ly = rng.choice(shapes)
        c = dict(model="kh", lattice="honeycomb", lx=lx, ly=ly)
        bits = n
    elif model == "heis":
        lattice = rng.choice(("chain", "tri", "kagome"))
        if lattice == "chain":
            lx, ly = int(round(2 ** rng.uniform(3, math.log2(34)))), 1
        elif lattice == "tri":
            lx, ly = rng.choice(((3, 3), (4, 3), (5, 3), (4, 4), (6, 3), (5, 4), (7, 3), (6, 4), (5, 5), (9, 3), (7, 4), (6, 5)))
        else:
            lx, ly = rng.choice(((3, 1), (2, 2), (5, 1), (3, 2), (7, 1), (4, 2), (3, 3), (5, 2), (11, 1), (3, 4)))
        c = dict(model="heis", lattice=lattice, lx=lx, ly=ly)
        bits = _n_sites(c)
        if bits > 20 or rng.random() < 0.8:
            up = rng.randint(1, bits // 2)
            c["two_sz"] = bits - 2 * up
    else:
        lx, ly = rng.choice(((4, 1), (5, 1), (3, 2), (7, 1), (4, 2), (3, 3), (5, 2), (11, 1), (4, 3), (13, 1), (7, 2), (5, 3),
                             (4, 4), (6, 3)))
        n = lx * ly
        c = dict(model="hubbard", lattice="rect", lx=lx, ly=ly, n_up=rng.randint(1, (n + 1) // 2), n_dn=rng.randint(1, n // 2))
        bits = 2 * n
    c["dtype"] = dtype
    kind = rng.choice(("hv", "hv", "tpq_step", "lanczos", "tpq_run", "expect", "cg"))
    if bits > 32:
        nvec = min(nvec, 4)
    if kind in ("lanczos", "cg"):
        c.update(kind=kind, n_iter=rng.randint(8, 20))
        if kind == "cg" and dtype in ("f32", "c64"):
            c["dtype"] = "f64" if dtype == "f32" else "c128"
    elif kind == "tpq_run":
        c.update(kind=kind, nvec=nvec, n_iter=rng.randint(8, 40))
    elif kind == "expect":
        c.update(kind=kind, nvec=nvec, n_obs=rng.randint(2, 12))
    else:
        c.update(kind=kind, nvec=nvec)
    return c


# ---------------------------------------------------------------- Hamiltonians and spaces

def _n_sites(c):
    if c["lattice"] == "kagome":
        return 3 * c["lx"] * c["ly"]
    if c["lattice"] == "honeycomb":
        return 2 * c["lx"] * c["ly"]
    if c["lattice"] == "super":
        return L.square_supercell((c["lx"], c["ly"]), (-c["lx"], c["ly"]))[0]
    return c["lx"] * c["ly"]


def _terms(c):
    lx, ly, n = c["lx"], c["ly"], _n_sites(c)
    if c["model"] == "kh":
        return kh_honeycomb_terms(lx=lx, ly=ly) if lx > 1 and ly > 1 else \
            [L.kitaev_heisenberg_bond(a, b, g, -1.0, 0.1) for a, b, g in L.honeycomb_links(lx, ly)]
    bonds = {"chain": lambda: L.chain_bonds(n), "rect": lambda: L.rect_bonds(lx, ly),
             "tri": lambda: L.triangular_bonds(lx, ly), "kagome": lambda: L.kagome_bonds(lx, ly),
             "super": lambda: L.square_supercell((lx, ly), (-lx, ly))[1]}[c["lattice"]]()
    bonds = [(i, j) for i, j in bonds if i != j]
    if c["model"] == "hubbard":
        return L.hubbard_terms(bonds, n, t=1.0, U=8.0)
    return [L.heisenberg_bond(i, j, 1.0) for i, j in bonds]


def _bases(c):
    n = _n_sites(c)
    if c["model"] == "hubbard":
        return [BasisDesc("fermion", n, "nupndn", n_up=c["n_up"], n_dn=c["n_dn"])]
    if "sectors" in c:
        return [BasisDesc("spin", n, "sz", two_sz=2 * m) for m in range(c["sectors"])]
    if "two_sz" in c:
        return [BasisDesc("spin", n, "sz", two_sz=c["two_sz"])]
    return [BasisDesc("spin", n)]


def _dims(c):
    out = []
    for b in _bases(c):
        if b.sector == "none":
            out.append(2 ** b.n_bits)
        elif b.sector == "sz":
            out.append(math.comb(b.n_sites, (b.n_sites + b.two_sz) // 2))
        else:
            out.append(math.comb(b.n_sites, b.n_up) * math.comb(b.n_sites, b.n_dn))
    return out


def _shift(c):
    """The TPQ shift l: above the largest energy per site."""
    return 8.5 if c["model"] == "hubbard" else 1.5


def _observables(c):
    """Term lists of n_obs Hermitian observables: densities, hops and two-body correlations at growing distance."""
    n, out = _n_sites(c), []
    for k in range(c["n_obs"]):
        d = 1 + (k // 4) % (n - 1)
        if c["model"] == "hubbard":
            out.append([L.Term(L.HOP, 0, 2 * d, (1.0, 0.0))] if k % 4 == 0 else
                       [L.Term(L.DENS, 0, 2 * d + 1, (1.0,))] if k % 4 == 1 else
                       [L.Term(L.HUBBARD_U, i, -1, (1.0,)) for i in range(d + 1)] if k % 4 == 2 else
                       [L.green2_term(0, 2 * d, 2 * d + 1, 1)])
        else:
            out.append([L.heisenberg_bond(0, d)] if k % 4 == 0 else
                       [L.xxz_bond(0, d, 0.0, 1.0)] if k % 4 == 1 else
                       [L.xxz_bond(i, i + 1, 1.0, 0.0) for i in range(d)] if k % 4 == 2 else _terms(c))
    return out


# ---------------------------------------------------------------- what a program has in hand, and the call

def _vectors(c, seed, dims):
    """Start vectors as the solvers take them: i.i.d. N(0, 1) entries."""
    dt = DTYPES[c["dtype"]]
    g = torch.Generator(device="cuda")
    g.manual_seed(seed)
    out = []
    for d in dims:
        shape = (d,) if c.get("nvec", 1) == 1 else (d, c["nvec"])
        x = torch.empty(shape, dtype=dt, device="cuda")
        (torch.view_as_real(x) if dt.is_complex else x).normal_(generator=g)
        out.append(x)
    return out


def prepare(case, seed):
    c, kind = case, case["kind"]
    bases = [hp.hphi_basis_build(b) for b in _bases(c)]
    vecs = _vectors(c, seed, [b.dim for b in bases])
    st = dict(case=c, bases=bases, v=vecs)
    nvec = c.get("nvec", 1)
    if kind == "expect":
        st["obs"] = [hp.hphi_ham_build(bases[0], t) for t in _observables(c)]
        return st
    st["hams"] = [hp.hphi_ham_build(b, _terms(c)) for b in bases]
    if kind == "hv":
        st["u"] = torch.empty_like(vecs[0])
        st["red"] = torch.empty(4 * nvec, dtype=torch.float64, device="cuda")
    elif kind in ("tpq_step", "tpq_run"):
        st["u"] = torch.empty_like(vecs[0])
        st["scale"] = 1.0 / torch.sqrt(sum(torch.linalg.vector_norm(p, dim=0, dtype=None).reshape(-1).double() ** 2
                                           for p in vecs[0].split(1 << 26)))
        st["obs"] = torch.empty((c.get("n_iter", 1), 4, nvec), dtype=torch.float64, device="cuda")
        if kind == "tpq_run":
            st["a"] = torch.empty_like(vecs[0])
    elif kind == "lanczos":
        dt = DTYPES[c["dtype"]]
        xdt = torch.complex128 if dt.is_complex else torch.float64
        st["work"] = [torch.empty(2 * b.dim, dtype=dt, device="cuda") for b in bases]
        st["x"] = [torch.empty(b.dim, dtype=xdt, device="cuda") for b in bases]
    elif kind == "cg":
        st["x"] = torch.empty_like(vecs[0])
        st["work"] = torch.empty(3 * bases[0].dim, dtype=vecs[0].dtype, device="cuda")
        st["v"][0] /= torch.linalg.vector_norm(vecs[0])
    return st


def _e_approx(c):
    """The energy that the inverse iteration starts from (by default one below the spectrum, where the solve is definite)."""
    return c.get("e_approx", -0.8 * sum(1 for t in _terms(c) if t.kind in (L.SPIN_BOND, L.HOP)))


def run(state):
    c = state["case"]
    kind, v = c["kind"], state["v"]
    if kind == "hv":
        # the product of a solver's step, with the sums that its recurrence reads
        hp.hphi_hv(state["hams"][0], v[0], state["u"], reduce=state["red"])
        return dict(u=state["u"], red=state["red"])
    if kind == "tpq_step":
        hp.hphi_tpq_step(state["hams"][0], v[0], state["u"], _shift(c), 2, state["scale"], state["obs"])
        return dict(psi=state["u"], obs=state["obs"])
    if kind == "tpq_run":
        state["a"].copy_(v[0])
        log = hp.hphi_tpq_run(state["hams"][0], state["a"], state["u"], _shift(c), 1, c["n_iter"], state["scale"], state["obs"])
        return dict(psi=state["a"] if c["n_iter"] % 2 == 0 else state["u"], obs=log)
    if kind == "lanczos":
        res = hp.hphi_lanczos(state["hams"], v, c["n_iter"], work=state["work"], x_out=state["x"])
        return [dict(alpha=r["alpha"], beta=r["beta"], e=r["e0_refined"], x=r["x"]) for r in res]
    if kind == "expect":
        return dict(o=[hp.hphi_expect(o, v[0]) for o in state["obs"]])
    state["x"].copy_(v[0])
    r = hp.hphi_cg_refine(state["hams"][0], state["x"], _e_approx(c), n_inverse=1, cg_max_iter=c["n_iter"], cg_tol=1e-300,
                          work=state["work"])
    return dict(x=state["x"], e=r["e_refined"], iters=r["cg_iters"])


# ---------------------------------------------------------------- compulsory work

def work(case):
    """Each input vector read once and each output vector written once per pass over the space; the flops are one
    multiply-add per stored real number and off-diagonal operator (half of a conserving operator's rows are live)."""
    c = case
    dims, nvec = _dims(c), c.get("nvec", 1)
    e = torch.empty(0, dtype=DTYPES[c["dtype"]]).element_size()
    reals = 2 if c["dtype"][0] == "c" else 1
    off = sum(1 for t in _terms(c) if t.kind in (L.SPIN_BOND, L.HOP))
    live = 1.0 if c["model"] == "kh" else 0.5
    byts = flops = 0
    for d in dims:
        vec, prod = d * nvec * e, 2 * live * off * d * nvec * reals
        if c["kind"] in ("hv", "tpq_step"):
            byts, flops = byts + 2 * vec, flops + prod
        elif c["kind"] == "tpq_run":
            byts, flops = byts + 2 * vec * c["n_iter"], flops + prod * c["n_iter"]
        elif c["kind"] == "lanczos":
            # a step: read v_k and v_{k-1}, write w; read w and v_k, write w; the second pass also updates x in FP64
            n = min(c["n_iter"], d)
            byts, flops = byts + n * (12 * vec + 16 * reals * d), flops + 2 * n * prod
        elif c["kind"] == "expect":
            byts, flops = byts + vec * c["n_obs"], flops + vec // e * reals * c["n_obs"] * 4
        else:
            # a CG step: the product (read p, write q), x, r and p updated from p, q and r
            byts, flops = byts + c["n_iter"] * 10 * vec, flops + c["n_iter"] * prod
    return {"bytes": byts, "flops": flops}


# ---------------------------------------------------------------- the same in 64 bits, in plain torch

def _states(b):
    n = b.n_bits
    if b.sector == "none":
        return torch.arange(1 << n, dtype=torch.int64, device="cuda")
    def combos(bits, k):
        # ascending bit strings over the given (ascending) bit positions with k set
        cur = {0: torch.zeros(1, dtype=torch.int64, device="cuda")}
        for p in bits:
            nxt = dict(cur)
            for q, s in cur.items():
                if q < k:
                    up = s | (1 << p)
                    nxt[q + 1] = torch.cat([cur[q + 1], up]) if q + 1 in cur else up
            cur = nxt
        return cur.get(k, torch.zeros(0, dtype=torch.int64, device="cuda"))
    if b.sector == "sz":
        return torch.sort(combos(range(n), (b.n_sites + b.two_sz) // 2))[0]
    up, dn = combos(range(0, n, 2), b.n_up), combos(range(1, n, 2), b.n_dn)
    return torch.sort((up[:, None] | dn[None, :]).reshape(-1))[0]


def _parity(x):
    for k in (32, 16, 8, 4, 2, 1):
        x = x ^ (x >> k)
    return x & 1


def _elements(t, s):
    """The pulled elements of one term in rows s: a list of (flip mask, complex coefficient per row)."""
    if t.kind == L.SPIN_BOND:
        up, z = np.array([[0, 0], [1, 0]]), np.diag([-0.5, 0.5])
        spin = ((up + up.T) / 2, (up - up.T) / 2j, z)   # index 0: down, 1: up
        m = np.zeros((4, 4), dtype=complex)
        for a in range(3):
            for b in range(3):
                m += t.c[3 * a + b] * np.kron(spin[b], spin[a])   # local index: bit i + 2 * bit j
        p = ((s >> t.i) & 1) | (((s >> t.j) & 1) << 1)
        out = []
        for x in range(4):
            row = np.array([m[q, q ^ x] for q in range(4)])
            if np.any(row != 0):
                tab = torch.tensor(row, device="cuda")
                out.append((((x & 1) << t.i) | ((x >> 1) << t.j), tab[p]))
        return out
    if t.kind == L.HOP:
        a, b = t.i, t.j
        lo, hi = min(a, b), max(a, b)
        between = (1 << hi) - (1 << (lo + 1))
        ba, bb = (s >> a) & 1, (s >> b) & 1
        sign = 1.0 - 2.0 * _parity(s & between).double()
        co = torch.complex((ba != bb).double() * t.c[0], (ba - bb).double() * t.c[1]) * sign
        return [((1 << a) | (1 << b), co)]
    if t.kind == L.HUBBARD_U:
        return [(0, (((s >> (2 * t.i)) & (s >> (2 * t.i + 1)) & 1).double() * t.c[0]).to(torch.complex128))]
    if t.kind == L.DENS:
        return [(0, (((s >> t.i) & (s >> t.j) & 1).double() * t.c[0]).to(torch.complex128))]
    return None


def _apply(b, terms, s, x, chunk=1 << 21):
    """H x in 64 bits (x: (dim, nvec)), a chunk of rows at a time."""
    u = torch.zeros_like(x)
    full = b.sector == "none"
    for r0 in range(0, s.numel(), chunk):
        rows = s[r0:r0 + chunk]
        acc = torch.zeros_like(x[r0:r0 + chunk])
        for t in terms:
            for mask, co in _elements(t, rows):
                co = co if x.dtype.is_complex else co.real
                tgt = rows ^ mask
                at = tgt if full else torch.searchsorted(s, tgt).clamp_(max=s.numel() - 1)
                acc += torch.where(co[:, None] != 0, co[:, None] * x[at], torch.zeros((), dtype=x.dtype, device="cuda"))
        u[r0:r0 + chunk] = acc
    return u


def exact(case, seed):
    c, dims = case, _dims(case)
    nvec = c.get("nvec", 1)
    reals = 2 if c["dtype"][0] == "c" else 1
    terms = _terms(c)
    steps = {"lanczos": c.get("n_iter", 1), "tpq_run": c.get("n_iter", 1), "cg": c.get("n_iter", 1) + 2}.get(c["kind"], 1)
    if sum(dims) * len(terms) * (nvec * reals + 4) * steps > 6e10:
        return None
    bases = _bases(c)
    wide = torch.complex128 if reals == 2 else torch.float64
    vecs = [v.to(wide).reshape(d, nvec) for v, d in zip(_vectors(c, seed, dims), dims)]

    def ip(x, y):
        return torch.sum(x.real * y.real + x.imag * y.imag if reals == 2 else x * y, dim=0)

    def shaped(x):
        return x.reshape(-1) if nvec == 1 else x
    if c["kind"] == "expect":
        s, x = _states(bases[0]), vecs[0]
        rows = []
        for obs in _observables(c):
            rows.append(None if any(t.kind == L.GREEN2 for t in obs) else
                        ip(x, _apply(bases[0], obs, s, x)) / ip(x, x))
        return dict(o=rows)
    if c["kind"] == "hv":
        s, x = _states(bases[0]), vecs[0]
        h = _apply(bases[0], terms, s, x)
        return dict(u=shaped(h), red=torch.cat([ip(x, x), ip(x, h), ip(h, h), ip(h, h)]))
    ns = _n_sites(c)
    if c["kind"] in ("tpq_step", "tpq_run"):
        s, x, l = _states(bases[0]), vecs[0], _shift(c)
        x = x / torch.sqrt(ip(x, x))
        logs, phi = [], None
        for j in range(c.get("n_iter", 1)):
            k = j + 1 if c["kind"] == "tpq_run" else 2
            h = _apply(bases[0], terms, s, x)
            xx = ip(x, x)
            u = ip(x, h) / xx / ns
            phi = l * x - h / ns
            scale = 1.0 / torch.sqrt(ip(phi, phi))
            logs.append(torch.stack([u, ip(h, h) / xx / ns ** 2, 2.0 * (k - 1) / ns / (l - u), scale]))
            x = phi * scale
        return dict(psi=shaped(phi), obs=torch.stack(logs))
    if c["kind"] == "lanczos":
        out = []
        for b, v in zip(bases, vecs):
            s = _states(b)
            x, prev, beta = v / torch.sqrt(ip(v, v)), torch.zeros_like(v), 0.0
            al, be = [], []
            n = min(c["n_iter"], b.n_bits and s.numel())
            for k in range(n):
                w = _apply(b, terms, s, x) - beta * prev
                a = float(ip(x, w))
                w = w - a * x
                beta = float(torch.sqrt(ip(w, w)))
                al.append(a)
                be.append(beta)
                if k + 1 == n or beta <= 1e-13:
                    break
                prev, x = x, w / beta
            if len(al) < c["n_iter"] or min(be[:-1], default=1.0) < 1e-6:
                out.append(None)     # the recurrence ends inside the space: what follows is rounding
                continue
            out.append(dict(alpha=np.array(al), beta=np.array(be), e=None, x=None))
        return out
    return None
