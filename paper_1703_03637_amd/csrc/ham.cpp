// Term validation and packing for the on-the-fly product (Sec. 2.3 models,
// Sec. 3.3 matrix elements generated by bit test, XOR and parity).
#include <algorithm>
#include <cmath>
#include <complex>
#include <cstring>
#include <new>
#include <vector>

#include "group.h"
#include "hphi_internal.h"

using namespace hphi;
using cplx = std::complex<double>;

namespace {

// 2x2 spin-1/2 operators in the basis (bit 0 = down, bit 1 = up):
// S^z = diag(-1/2, 1/2), S^+ maps bit 0 to bit 1; S^x, S^y from S^+ and S^-.
// spin_elem(a, row_bit, col_bit) = <row|S^a|col>.
cplx spin_elem(int a, int r, int c) {
    if (a == 2) return r == c ? cplx(r ? 0.5 : -0.5, 0.0) : cplx(0, 0);
    if (r == c) return cplx(0, 0);
    const double sp = (r == 1 && c == 0) ? 1.0 : 0.0;   // <r|S^+|c>
    const double sm = (r == 0 && c == 1) ? 1.0 : 0.0;   // <r|S^-|c>
    if (a == 0) return cplx((sp + sm) / 2.0, 0.0);
    return cplx(0.0, -(sp - sm) / 2.0);                  // (S^+ - S^-)/(2i)
}

DevOp blank_op(uint32_t bi, uint32_t bj, int term) {
    DevOp o{};
    o.bi = bi;
    o.bj = bj;
    o.term = term;
    return o;
}

void set_off(DevOp& o, int p, cplx c) {
    o.cr[p] = c.real();
    o.ci[p] = c.imag();
    if (c != cplx(0, 0)) o.has_off = 1;
}

// t c+_a c_b c+_c c_d + h.c. on orbitals orb[0..3] (Sec. 3.3 sign rule, each
// operator applied in turn): for every occupation pattern P of the distinct
// orbitals involved, the four operators map P to P' with a sign from the
// occupied involved orbitals below each one, and the orbitals outside the
// set contribute the parity of s & M, M the XOR of the four below-masks.
// Row patterns R are selected by the two lowest involved orbitals (the
// operator's pattern bits) and, for the others, a row condition.
int pack_green2(const int orb[4], cplx t, int term, std::vector<DevOp>& ops) {
    std::vector<int> D;
    for (int k = 0; k < 4; ++k)
        if (std::find(D.begin(), D.end(), orb[k]) == D.end()) D.push_back(orb[k]);
    std::sort(D.begin(), D.end());
    const int m = int(D.size());
    uint64_t dmask = 0;
    for (int x : D) dmask |= uint64_t(1) << x;
    auto loc = [&](int x) { return int(std::find(D.begin(), D.end(), x) - D.begin()); };
    // operators right to left: c_d, c+_c, c_b, c+_a
    const int seq[4] = {orb[3], orb[2], orb[1], orb[0]};
    const bool cre[4] = {false, true, false, true};
    uint64_t outmask = 0;
    for (int k = 0; k < 4; ++k) outmask ^= ((uint64_t(1) << seq[k]) - 1) & ~dmask;
    std::vector<DevOp> local;
    auto op_for = [&](uint64_t xm, uint64_t cm, uint64_t cv) -> DevOp& {
        for (DevOp& o : local)
            if (o.xmask == xm && o.cmask == cm && o.cval == cv) return o;
        DevOp o = blank_op(uint32_t(D[0]), uint32_t(m > 1 ? D[1] : D[0]), term);
        o.xmask = xm;
        o.smask = xm ? outmask : 0;
        o.cmask = cm;
        o.cval = cv;
        local.push_back(o);
        return local.back();
    };
    // the kernel's pattern index of a row pattern R (bits of D[0], D[1]) and its condition
    auto pat = [&](int R) { return m == 1 ? ((R & 1) ? 3 : 0) : (R & 3); };
    auto cond = [&](int R, uint64_t& cm, uint64_t& cv) {
        cm = cv = 0;
        for (int k = 2; k < m; ++k) {
            cm |= uint64_t(1) << D[k];
            if ((R >> k) & 1) cv |= uint64_t(1) << D[k];
        }
    };
    auto bits_of = [&](int F) {
        uint64_t x = 0;
        for (int k = 0; k < m; ++k)
            if ((F >> k) & 1) x |= uint64_t(1) << D[k];
        return x;
    };
    for (int P = 0; P < (1 << m); ++P) {
        int st = P;
        double sign = 1.0;
        bool ok = true;
        for (int k = 0; k < 4 && ok; ++k) {
            const int j = loc(seq[k]);
            const bool occ = (st >> j) & 1;
            if (occ == cre[k]) {
                ok = false;
                break;
            }
            // involved orbitals below this one that are occupied now
            int below = 0;
            for (int q = 0; q < m; ++q)
                if (D[q] < seq[k] && ((st >> q) & 1)) ++below;
            if (below & 1) sign = -sign;
            st ^= 1 << j;
        }
        if (!ok) continue;
        const cplx c = t * sign;
        const int F = P ^ st;
        uint64_t cm, cv;
        if (F == 0) {
            // diagonal: t sign + conj(t sign) on rows with pattern P (the outside signs cancel)
            cond(P, cm, cv);
            op_for(0, cm, cv).d[pat(P)] += 2.0 * c.real();
            continue;
        }
        // rows with pattern st pull from P through T; rows with pattern P pull from st through T^dagger
        cond(st, cm, cv);
        DevOp& o1 = op_for(bits_of(F), cm, cv);
        set_off(o1, pat(st), cplx(o1.cr[pat(st)], o1.ci[pat(st)]) + c);
        cond(P, cm, cv);
        DevOp& o2 = op_for(bits_of(F), cm, cv);
        set_off(o2, pat(P), cplx(o2.cr[pat(P)], o2.ci[pat(P)]) + std::conj(c));
    }
    for (DevOp& o : local) {
        if (!o.has_off) o.xmask = 0;
        ops.push_back(o);
    }
    return HPHI_OK;
}

}  // namespace

extern "C" int hphi_ham_build(const hphi_basis* basis, const hphi_term* terms, int64_t n_terms,
                              hphi_ham** out) {
    if (!basis || !out || n_terms < 0 || (n_terms > 0 && !terms))
        return set_error(HPHI_EINVAL, "hphi_ham_build: bad argument");
    *out = nullptr;
    const int particle = basis->desc.particle;
    const int ns = basis->desc.n_sites;
    const int nbits = basis->nbits;
    std::vector<DevOp> ops;

    for (int64_t t = 0; t < n_terms; ++t) {
        const hphi_term& T = terms[t];
        for (int k = 0; k < 9; ++k)
            if (!std::isfinite(T.c[k])) return set_error(HPHI_EINVAL, "term %lld: non-finite coefficient", (long long)t);
        const bool spin_kind = T.kind == HPHI_TERM_SPIN_BOND || T.kind == HPHI_TERM_SPIN_FIELD;
        const bool ferm_kind = T.kind >= HPHI_TERM_HOP && T.kind <= HPHI_TERM_GREEN2;
        if (!spin_kind && !ferm_kind) return set_error(HPHI_EINVAL, "term %lld: unknown kind %d", (long long)t, T.kind);
        if (spin_kind && particle != HPHI_SPIN_HALF)
            return set_error(HPHI_EINVAL, "term %lld: spin term on a fermion basis", (long long)t);
        if (ferm_kind && particle != HPHI_FERMION)
            return set_error(HPHI_EINVAL, "term %lld: fermion term on a spin basis", (long long)t);

        switch (T.kind) {
            case HPHI_TERM_SPIN_BOND: {
                if (T.i < 0 || T.j < 0 || T.i >= ns || T.j >= ns || T.i == T.j)
                    return set_error(HPHI_EINVAL, "term %lld: bad bond sites (%d, %d)", (long long)t, T.i, T.j);
                // M[p][q] = <p| sum_ab J^ab S_i^a S_j^b |q>, p = bit_i | bit_j << 1
                cplx M[4][4];
                for (int p = 0; p < 4; ++p)
                    for (int q = 0; q < 4; ++q) {
                        cplx acc(0, 0);
                        for (int a = 0; a < 3; ++a)
                            for (int b = 0; b < 3; ++b) {
                                const double J = T.c[3 * a + b];
                                if (J == 0.0) continue;
                                acc += J * spin_elem(a, p & 1, q & 1) * spin_elem(b, p >> 1, q >> 1);
                            }
                        M[p][q] = acc;
                    }
                // one operator per flip pattern f (1: bit i, 2: bit j, 3: both);
                // the diagonal rides on the first emitted operator
                bool diag_done = false;
                for (int f = 3; f >= 1; --f) {
                    DevOp o = blank_op(uint32_t(T.i), uint32_t(T.j), int(t));
                    o.xmask = ((f & 1) ? (uint64_t(1) << T.i) : 0) | ((f & 2) ? (uint64_t(1) << T.j) : 0);
                    for (int p = 0; p < 4; ++p) set_off(o, p, M[p][p ^ f]);
                    if (!o.has_off) continue;
                    if (!diag_done) {
                        for (int p = 0; p < 4; ++p) o.d[p] = M[p][p].real();
                        diag_done = true;
                    }
                    ops.push_back(o);
                }
                if (!diag_done) {
                    DevOp o = blank_op(uint32_t(T.i), uint32_t(T.j), int(t));
                    for (int p = 0; p < 4; ++p) o.d[p] = M[p][p].real();
                    ops.push_back(o);
                }
                break;
            }
            case HPHI_TERM_SPIN_FIELD: {
                if (T.i < 0 || T.i >= ns) return set_error(HPHI_EINVAL, "term %lld: bad site %d", (long long)t, T.i);
                // pattern p in {0, 3} (bi == bj): bit value b = p & 1
                cplx M[2][2];
                for (int r = 0; r < 2; ++r)
                    for (int c = 0; c < 2; ++c) {
                        cplx acc(0, 0);
                        for (int a = 0; a < 3; ++a)
                            if (T.c[a] != 0.0) acc += T.c[a] * spin_elem(a, r, c);
                        M[r][c] = acc;
                    }
                DevOp o = blank_op(uint32_t(T.i), uint32_t(T.i), int(t));
                o.d[0] = M[0][0].real();
                o.d[3] = M[1][1].real();
                o.xmask = uint64_t(1) << T.i;
                set_off(o, 0, M[0][1]);
                set_off(o, 3, M[1][0]);
                if (!o.has_off) o.xmask = 0;
                ops.push_back(o);
                break;
            }
            case HPHI_TERM_HOP: {
                const int a = T.i, b = T.j;
                if (a < 0 || b < 0 || a >= nbits || b >= nbits || a == b)
                    return set_error(HPHI_EINVAL, "term %lld: bad hop orbitals (%d, %d)", (long long)t, a, b);
                DevOp o = blank_op(uint32_t(a), uint32_t(b), int(t));
                o.xmask = (uint64_t(1) << a) | (uint64_t(1) << b);
                const int lo = a < b ? a : b, hi = a < b ? b : a;
                // orbitals strictly between the two ends
                o.smask = ((uint64_t(1) << hi) - 1) & ~((uint64_t(2) << lo) - 1);
                const cplx tt(T.c[0], T.c[1]);
                // row s with n_a = 1, n_b = 0 (p = 1) pulls from t = s ^ xmask via t c+_a c_b;
                // row s with n_a = 0, n_b = 1 (p = 2) pulls via conj(t) c+_b c_a
                set_off(o, 1, tt);
                set_off(o, 2, std::conj(tt));
                if (!o.has_off) o.xmask = 0;
                ops.push_back(o);
                break;
            }
            case HPHI_TERM_DENS: {
                const int a = T.i, b = T.j;
                if (a < 0 || b < 0 || a >= nbits || b >= nbits || a == b)
                    return set_error(HPHI_EINVAL, "term %lld: bad orbitals (%d, %d)", (long long)t, a, b);
                DevOp o = blank_op(uint32_t(a), uint32_t(b), int(t));
                o.d[3] = T.c[0];
                ops.push_back(o);
                break;
            }
            case HPHI_TERM_NUM: {
                const int a = T.i;
                if (a < 0 || a >= nbits) return set_error(HPHI_EINVAL, "term %lld: bad orbital %d", (long long)t, a);
                DevOp o = blank_op(uint32_t(a), uint32_t(a), int(t));
                o.d[3] = T.c[0];
                ops.push_back(o);
                break;
            }
            case HPHI_TERM_HUBBARD_U: {
                if (T.i < 0 || T.i >= ns) return set_error(HPHI_EINVAL, "term %lld: bad site %d", (long long)t, T.i);
                DevOp o = blank_op(uint32_t(2 * T.i), uint32_t(2 * T.i + 1), int(t));
                o.d[3] = T.c[0];
                ops.push_back(o);
                break;
            }
            case HPHI_TERM_GREEN2: {
                const int orb[4] = {T.i, T.j, int(T.c[2]), int(T.c[3])};
                for (int k = 0; k < 4; ++k)
                    if (orb[k] < 0 || orb[k] >= nbits || (k >= 2 && double(orb[k]) != T.c[k]))
                        return set_error(HPHI_EINVAL, "term %lld: bad Green's-function orbital", (long long)t);
                if (int rc = pack_green2(orb, cplx(T.c[0], T.c[1]), int(t), ops)) return rc;
                break;
            }
        }
    }


    // ---- sector check: every nonzero off-diagonal element must conserve the charge
    const int sector = basis->desc.sector;
    bool is_complex = false;
    for (const DevOp& o : ops) {
        for (int p = 0; p < 4; ++p) {
            if (o.ci[p] != 0.0) is_complex = true;
            if (!o.xmask || (o.cr[p] == 0.0 && o.ci[p] == 0.0)) continue;
            if (sector == HPHI_SECTOR_NONE) continue;
            // charge change of the flip: the row's bits come from the pattern
            // (bi, bj) and, for conditional operators, from cval
            int d_all = 0, d_even = 0, d_odd = 0;
            for (int x = 0; x < 64; ++x) {
                if (!((o.xmask >> x) & 1)) continue;
                int bit;
                if (uint32_t(x) == o.bi) bit = p & 1;
                else if (uint32_t(x) == o.bj) bit = (p >> 1) & 1;
                else bit = int((o.cval >> x) & 1);
                const int dq = bit ? -1 : 1;
                d_all += dq;
                (x & 1 ? d_odd : d_even) += dq;
            }
            const bool ok = sector == HPHI_SECTOR_NUP_NDN ? (d_even == 0 && d_odd == 0) : d_all == 0;
            if (!ok)
                return set_error(HPHI_ESECTOR, "term %d leaves the sector (flip 0x%llx, pattern %d)", o.term,
                                 (unsigned long long)o.xmask, p);
        }
    }

    hphi_ham* H = alloc_fails() ? nullptr : new (std::nothrow) hphi_ham();
    if (!H) return set_error(HPHI_ENOMEM, "hphi_ham_build: host allocation");
    H->basis = basis;
    H->n_sites = ns;
    H->is_complex = is_complex;
    H->ops = ops;
    for (const DevOp& o : ops) H->has_cond = H->has_cond || o.cmask != 0;
    // device copies padded with inert operators to a multiple of 4 (at
    // least 4): the product kernels decode operators four at a time
    const int n_pad = ops.empty() ? 4 : int((ops.size() + 3) / 4 * 4);
    H->n_ops_pad = n_pad;
    std::vector<DevOp> padded(ops);
    padded.resize(size_t(n_pad), blank_op(0, 0, -1));
    // pattern table: entry (o, p) = {Re c[p], Im c[p], d[p], 0}
    std::vector<double> ptab(size_t(n_pad) * 16, 0.0);
    for (int o = 0; o < n_pad; ++o)
        for (int q = 0; q < 4; ++q) {
            ptab[size_t(o) * 16 + q * 4 + 0] = padded[o].has_off ? padded[o].cr[q] : 0.0;
            ptab[size_t(o) * 16 + q * 4 + 1] = padded[o].has_off ? padded[o].ci[q] : 0.0;
            ptab[size_t(o) * 16 + q * 4 + 2] = padded[o].d[q];
        }
    // One allocation: reduction partials, reductions and the non-finite flag
    // word, then what is uploaded (operators, pattern table and, for the
    // class-blocked sector product, its operator lists), then that product's
    // tables, filled by a kernel.
    GroupHost gh;
    const bool grouped = group_analyse(basis, ops, is_complex, H->has_cond, gh);
    size_t off = 0;
    auto take = [&](size_t bytes) {
        const size_t at = off;
        off += (bytes + 255) / 256 * 256;
        return at;
    };
    const size_t o_part = take(size_t(kMaxGrid) * kNQ * kMaxNvec * sizeof(double));
    const size_t o_up = off;
    const size_t o_red = take(size_t(kNQ) * kMaxNvec * sizeof(double) + 256);
    const size_t o_tick = take(size_t(kTickets) * 4);
    const size_t o_ops = take(padded.size() * sizeof(DevOp));
    const size_t o_ptab = take(ptab.size() * sizeof(double));
    const size_t base_bytes = off;
    const size_t n_slot = size_t(basis->grp.n_slot);
    const size_t n_low = size_t(1) << basis->b_lo;
    const size_t n_hh = gh.hh.size(), n_lh = gh.lh.size(), n_ci = gh.ci.size(), n_ll = gh.ll.size(), n_col = gh.col.size();
    const size_t stride = group_ent_stride(gh);
    const size_t ll_rows = size_t(group_rows(int(n_ll)));
    const size_t o_ll = take(n_ll * sizeof(GLow)), o_coef = take(gh.coef.size() * 8), o_col = take(n_col * sizeof(GColumn)),
                 o_lh = take((n_lh + kGroupPad) * sizeof(GCross)), o_ci = take(n_ci * 4), o_bhh = take(n_hh * sizeof(GBuildOp)),
                 o_blh = take(n_lh * sizeof(GBuildOp)), o_dlo = take(gh.dlo.size() * sizeof(GBuildDiag)),
                 o_dhi = take(gh.dhi.size() * sizeof(GBuildDiag)), o_dx = take(gh.dx.size() * sizeof(GBuildDiag));
    const size_t up_end = off;
    const size_t o_row = take(n_slot * 8), o_hv = take(n_slot * 4), o_ne = take(n_slot * 4), o_dh = take(n_slot * 8),
                 o_hh = take(n_slot * stride * 8), o_lhe = take(n_lh * n_slot * 8),
                 o_w = take(n_ci * n_slot * sizeof(double)),
                 o_dl = take(n_low * sizeof(double)), o_nbr = take(ll_rows * n_low * 4), o_xnb = take(std::max<size_t>(n_col, 1) * n_low * 4);
    bool group = grouped;
    if (alloc_fails()) {
        hphi_ham_free(H);
        return set_error(HPHI_ENOMEM, "hphi_ham_build: device allocation failed (injected)");
    }
    hipError_t e = hipMalloc(&H->d_mem, group ? off : base_bytes);
    if (e == hipErrorOutOfMemory && group) {   // without the class-blocked tables
        (void)hipGetLastError();
        group = false;
        e = hipMalloc(&H->d_mem, base_bytes);
    }
    if (e != hipSuccess) {
        H->d_mem = nullptr;
        (void)hipGetLastError();
        hphi_ham_free(H);
        return set_error(e == hipErrorOutOfMemory ? HPHI_ENOMEM : HPHI_EDEVICE, "hphi_ham_build: device allocation of %zu bytes: %s",
                         base_bytes, hipGetErrorString(e));
    }
    char* const m = static_cast<char*>(H->d_mem);
    H->d_partials = reinterpret_cast<double*>(m + o_part);
    H->d_red = reinterpret_cast<double*>(m + o_red);
    H->d_flag = reinterpret_cast<int32_t*>(H->d_red + kNQ * kMaxNvec);
    H->d_tickets = reinterpret_cast<uint32_t*>(m + o_tick);
    H->d_ops = reinterpret_cast<DevOp*>(m + o_ops);
    H->d_ptab = reinterpret_cast<double*>(m + o_ptab);
    const size_t up_bytes = (group ? up_end : base_bytes) - o_up;
    std::vector<char> up(up_bytes, 0);         // the reductions, the flag and the tickets start at zero
    auto fill = [&](size_t at, const void* src, size_t bytes) {
        if (bytes) std::memcpy(up.data() + (at - o_up), src, bytes);
    };
    fill(o_ops, padded.data(), padded.size() * sizeof(DevOp));
    fill(o_ptab, ptab.data(), ptab.size() * sizeof(double));
    if (group) {
        fill(o_ll, gh.ll.data(), n_ll * sizeof(GLow));
        fill(o_coef, gh.coef.data(), gh.coef.size() * 8);
        fill(o_col, gh.col.data(), n_col * sizeof(GColumn));
        fill(o_lh, gh.lh.data(), n_lh * sizeof(GCross));
        fill(o_ci, gh.ci.data(), n_ci * 4);
        fill(o_bhh, gh.hh.data(), n_hh * sizeof(GBuildOp));
        fill(o_blh, gh.lh_build.data(), n_lh * sizeof(GBuildOp));
        fill(o_dlo, gh.dlo.data(), gh.dlo.size() * sizeof(GBuildDiag));
        fill(o_dhi, gh.dhi.data(), gh.dhi.size() * sizeof(GBuildDiag));
        fill(o_dx, gh.dx.data(), gh.dx.size() * sizeof(GBuildDiag));
    }
    e = hipMemcpy(m + o_up, up.data(), up_bytes, hipMemcpyHostToDevice);
    if (e != hipSuccess) {
        hphi_ham_free(H);
        return check_hip(e, "hphi_ham_build: upload");
    }
    if (group) {
        GroupBuild G{};
        G.op_hh = reinterpret_cast<const GBuildOp*>(m + o_bhh);
        G.op_lh = reinterpret_cast<const GBuildOp*>(m + o_blh);
        G.dlo_ops = reinterpret_cast<const GBuildDiag*>(m + o_dlo);
        G.dhi = reinterpret_cast<const GBuildDiag*>(m + o_dhi);
        G.dx = reinterpret_cast<const GBuildDiag*>(m + o_dx);
        G.n_hh = int(n_hh);
        G.n_lh = int(n_lh);
        G.n_dlo = int(gh.dlo.size());
        G.n_dhi = int(gh.dhi.size());
        G.n_x = int(gh.dx.size());
        G.n_ci = int(n_ci);
        G.hh_stride = int(stride);
        G.n_ll = int(n_ll);
        G.n_col = int(n_col);
        G.ll = reinterpret_cast<const GLow*>(m + o_ll);
        G.col = reinterpret_cast<const GColumn*>(m + o_col);
        G.row0 = reinterpret_cast<int64_t*>(m + o_row);
        G.hval = reinterpret_cast<uint32_t*>(m + o_hv);
        G.n_ent = reinterpret_cast<uint32_t*>(m + o_ne);
        G.dhi_out = reinterpret_cast<double*>(m + o_dh);
        G.hh = reinterpret_cast<uint64_t*>(m + o_hh);
        G.lhe = reinterpret_cast<int64_t*>(m + o_lhe);
        G.w = reinterpret_cast<double*>(m + o_w);
        G.dlo = reinterpret_cast<double*>(m + o_dl);
        G.nbr = reinterpret_cast<uint32_t*>(m + o_nbr);
        G.xnb = reinterpret_cast<uint32_t*>(m + o_xnb);
        H->grp = new (std::nothrow) GroupPlan();
        const int rc = H->grp ? group_build(basis, G) : set_error(HPHI_ENOMEM, "hphi_ham_build: host allocation");
        if (rc) {
            hphi_ham_free(H);
            return rc;
        }
        GroupPlan& P = *H->grp;
        P.n_ll = int(n_ll);
        P.n_lh = int(n_lh);
        P.n_col = int(n_col);
        P.n_ci = int(n_ci);
        P.n_hh = int(n_hh);
        P.n_coef = int(gh.coef.size());
        P.hh_stride = int(stride);
        P.n_slot = uint32_t(n_slot);
        P.n_low = uint32_t(n_low);
        P.row0 = G.row0;
        P.hval = G.hval;
        P.n_ent = G.n_ent;
        P.dhi = G.dhi_out;
        P.hh = G.hh;
        P.lhe = G.lhe;
        P.w = G.w;
        P.ci = reinterpret_cast<const uint32_t*>(m + o_ci);
        P.dlo = G.dlo;
        P.nbr = G.nbr;
        P.xnb = G.xnb;
        P.coef = reinterpret_cast<const double*>(m + o_coef);
        P.lh = reinterpret_cast<const GCross*>(m + o_lh);
        P.ll_ops = G.ll;
        P.hh_ops = G.op_hh;
    }
    // persistent grid: enough waves to cover the tiles, at most kMaxGrid blocks,
    // a multiple of 8 so every XCD gets the same number of blocks
    const int64_t tiles = basis->dev.n_tiles;
    int64_t g = (tiles + kWavesPerBlock - 1) / kWavesPerBlock;
    if (g > kMaxGrid) g = kMaxGrid;
    g = ((g + 7) / 8) * 8;
    H->grid = int(g);
    *out = H;
    return HPHI_OK;
}

extern "C" int hphi_ham_is_complex(const hphi_ham* h, int32_t* is_complex) {
    if (!h || !is_complex) return set_error(HPHI_EINVAL, "hphi_ham_is_complex: null argument");
    *is_complex = h->is_complex ? 1 : 0;
    return HPHI_OK;
}

hphi_ham::~hphi_ham() {
    if (d_mem) (void)hipFree(d_mem);
    delete grp;
    for (PassPlan* p : plans) {
        if (p->d_ops) (void)hipFree(p->d_ops);
        if (p->d_perm) (void)hipFree(p->d_perm);
        if (p->d_kop64) (void)hipFree(p->d_kop64);
        if (p->d_kopq) (void)hipFree(p->d_kopq);
        if (p->d_inv) (void)hipFree(p->d_inv);
        delete p;
    }
    for (void* b : d_stage)
        if (b) (void)hipFree(b);
    for (CmaPlan* p : cma_plans) {
        if (p->d_hf) (void)hipFree(p->d_hf);
        if (p->d_hd) (void)hipFree(p->d_hd);
        if (p->d_bits) (void)hipFree(p->d_bits);
        delete p;
    }
}

extern "C" void hphi_ham_free(hphi_ham* h) { delete h; }
