// Class-blocked sector product (group.h): the tables of a Hamiltonian, and the
// choice of a kernel.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <cmath>
#include <cstdlib>

#include "group.h"
#include "hphi_internal.h"

namespace hphi {

int launch_hvg_f32(HvgArgs& A, const HvLaunch& L, int ns, int k, int lanes, bool sign, int cap, int cus, hipStream_t st,
                   int* g);
int launch_hvg_f64(HvgArgs& A, const HvLaunch& L, int ns, int k, int lanes, bool sign, int cap, int cus, hipStream_t st,
                   int* g);
int launch_hvg_multi_f32(const HvgArgs* d_args, const int* d_begin, int n, int ns, int k, bool sign, int grid, int* occ,
                         hipStream_t st);
int launch_hvg_multi_f64(const HvgArgs* d_args, const int* d_begin, int n, int ns, int k, bool sign, int grid, int* occ,
                         hipStream_t st);

// rows from which only groups of four and more high halves are used
static constexpr int64_t kGroupLarge = int64_t(1) << 22;

namespace {

// a sum with its rounding errors carried along (Knuth's two-sum)
struct TwoSum {
    double s = 0.0, e = 0.0;
    __device__ void add(double x) {
        const double t = s + x, b = t - s;
        e += (s - (t - b)) + (x - b);
        s = t;
    }
    __device__ double value() const { return s + e; }
};

// One thread per slot: its first row, the diagonal of the
// high half, the partner blocks of the operators inside it, and per cross
// operator the partner block and the signed element.
__global__ __launch_bounds__(256) void group_high_kernel(GroupBuild G, BasisDev bs, const uint32_t* __restrict__ hord,
                                                          uint32_t n_slot) {
    const uint32_t p = blockIdx.x * 256u + threadIdx.x;
    if (p >= n_slot) return;
    const uint32_t k = hord[p];
    const uint64_t h = bs.h_val[k];
    const int64_t row0 = bs.h_row[k];
    G.row0[p] = row0;
    G.hval[p] = uint32_t(h);
    TwoSum dhi;
    for (int i = 0; i < G.n_dhi; ++i) {
        const GBuildDiag& d = G.dhi[i];
        const int bj = int((h >> (d.bj - bs.b_lo)) & 1);
        const int bi = d.bi >= bs.b_lo ? int((h >> (d.bi - bs.b_lo)) & 1) : 0;
        dhi.add(d.d[bi | (bj << 1)]);
    }
    G.dhi_out[p] = dhi.value();
    uint32_t n = 0;
    uint64_t* hh = G.hh + size_t(p) * size_t(G.hh_stride);
    for (int o = 0; o < G.n_hh; ++o) {
        const GBuildOp& op = G.op_hh[o];
        const uint64_t x = h & op.m_hi;
        if (x == 0 || x == op.m_hi) continue;
        const uint64_t c = uint64_t((__popcll(h & op.sm_hi) & 1) ? op.neg : op.pos);
        hh[n++] = uint64_t(bs.j_hi[h ^ op.m_hi]) | (c << 48);
    }
    G.n_ent[p] = n;
    for (; n < uint32_t(G.hh_stride); ++n) hh[n] = uint64_t(row0);
    for (int o = 0; o < G.n_lh; ++o) {
        const GBuildOp& op = G.op_lh[o];
        const int64_t t = bs.j_hi[h ^ op.m_hi];
        // no sector state has the target high half: then no row of h is live
        const uint64_t sg = uint64_t(__popcll(h & op.sm_hi) & 1) << 63;
        G.lhe[size_t(o) * n_slot + p] = int64_t(uint64_t(t >= 0 ? t : row0) | sg);
    }
    for (int c = 0; c < G.n_ci; ++c) {
        TwoSum w;
        for (int i = 0; i < G.n_x; ++i) {
            if (G.dx[i].ci != c) continue;
            const bool up = ((h >> (G.dx[i].bj - bs.b_lo)) & 1) != 0;
            if (up) w.add(G.dx[i].d[3]);
            else if (G.dx[i].spin) w.add(-G.dx[i].d[3]);
        }
        G.w[size_t(c) * n_slot + p] = w.value();
    }
}

// one thread per low half: its diagonal, its partner list and the partners of
// its single flips
__global__ __launch_bounds__(256) void group_low_kernel(GroupBuild G, BasisDev bs) {
    const uint32_t i = blockIdx.x * 256u + threadIdx.x;
    const uint32_t n_low = 1u << bs.b_lo;
    if (i >= n_low) return;
    const uint32_t l = bs.lows[i];
    TwoSum s;
    for (int k = 0; k < G.n_dlo; ++k) {
        const GBuildDiag& d = G.dlo_ops[k];
        const int bi = int((l >> d.bi) & 1u);
        const int bj = d.bj < bs.b_lo ? int((l >> d.bj) & 1u) : 0;
        s.add(d.d[bi | (bj << 1)]);
    }
    G.dlo[i] = s.value();
    for (int o = 0; o < G.n_ll; ++o) {
        const GLow op = G.ll[o];
        const uint32_t x = l & op.m;
        const uint32_t ci = uint32_t((__popc(l & op.sm) & 1) ? op.neg : op.pos);
        G.nbr[size_t(o) * n_low + i] = x == 0 || x == op.m ? bs.j_lo[l] : bs.j_lo[l ^ op.m] | (ci << 24);
    }
    const int rows = group_rows(G.n_ll);
    for (int o = G.n_ll; o < rows; ++o) G.nbr[size_t(o) * n_low + i] = bs.j_lo[l];
    for (int k = 0; k < G.n_col; ++k) {
        const GColumn col = G.col[k];
        const uint32_t sg = uint32_t(__popc(l & col.sm) & 1) << 30, bit = (l & col.mi) ? 0x80000000u : 0u;
        G.xnb[size_t(k) * n_low + i] = bs.j_lo[l ^ col.mi] | sg | bit;
    }
}

// Element export of the class-blocked product: the partners and elements that it
// takes from its tables, row by row, under their operators.  A block takes whole
// groups, and of these only the rows in the range, a row per lane.
__global__ __launch_bounds__(kBlock) void hvg_export_kernel(HvgArgs A) {
    const GroupPlan& P = A.plan;
    const int64_t first = A.ex.row0, end = A.ex.row0 + A.ex.nrows;
    for (uint32_t g = blockIdx.x; g < A.grp.begin[8]; g += gridDim.x) {
        const GGroup grp = A.grp.groups[g];
        const GClass cls = A.cls[grp.cls];       // (a closing entry has no slots)
        for (uint32_t p = grp.p0; p < grp.p0 + grp.n; ++p) {
            const int64_t row0 = P.row0[p];
            if (row0 >= end || row0 + int64_t(cls.n_l) <= first) continue;
            const uint32_t hval = P.hval[p];
            // ranks of the rows in the range
            const uint32_t r1 = uint32_t(std::min<int64_t>(cls.n_l, end - row0));
            const uint32_t r0 = uint32_t(std::max<int64_t>(0, first - row0));
            for (uint32_t r = r0 + blockIdx.y * kBlock + threadIdx.x; r < r1; r += gridDim.y * kBlock) {
                const uint32_t li = cls.l_off + r, l = A.lows[li];
                const int64_t row = row0 + int64_t(r) - first;
                auto put = [&](int op, int64_t col, double c) {
                    A.ex.col[size_t(row) * size_t(A.ex.n_slots) + size_t(op)] = col;
                    A.ex.cr[size_t(row) * size_t(A.ex.n_slots) + size_t(op)] = c;
                };
                for (int o = 0; o < P.n_ll; ++o) {
                    const uint32_t ent = P.nbr[size_t(o) * P.n_low + li];
                    if (ent >> 24) put(P.ll_ops[o].op, row0 + int64_t(ent & kGroupRank), P.coef[ent >> 24]);
                }
                uint32_t e = 0;
                for (int o = 0; o < P.n_hh; ++o) {
                    const uint32_t m = uint32_t(P.hh_ops[o].m_hi), x = hval & m;
                    if (x == 0 || x == m) continue;
                    const uint64_t t = P.hh[size_t(p) * size_t(P.hh_stride) + e++];
                    put(P.hh_ops[o].op, int64_t((t << 16) >> 16) + int64_t(r), P.coef[t >> 48]);
                }
                for (int o = 0; o < P.n_lh; ++o) {
                    if (P.lh[o].op < 0) continue;
                    const uint32_t ent = P.xnb[size_t(P.lh[o].col) * P.n_low + li];
                    if ((ent >> 31) == ((hval >> P.lh[o].j) & 1u)) continue;
                    const int64_t t = P.lhe[size_t(o) * P.n_slot + p];
                    const bool minus = ((ent & (1u << 30)) != 0) != (t < 0);
                    put(P.lh[o].op, (t & INT64_MAX) + int64_t(ent & kGroupRank), minus ? -P.lh[o].c : P.lh[o].c);
                }
                // the diagonal as the product adds it up
                double dd = P.dlo[li] + P.dhi[p];
                for (int i = 0; i < P.n_ci; ++i) {
                    const uint32_t bit = P.ci[i];
                    const double b = (l >> (bit & 31u)) & 1u ? 1.0 : ((bit & 32u) ? -1.0 : 0.0);
                    dd += b * P.w[size_t(i) * P.n_slot + p];
                }
                A.ex.diag[size_t(row) * size_t(A.ex.n_pass)] = dd;
            }
        }
    }
}

int cu_count() {
    static const int n = [] {
        int dev = 0, ncu = 0;
        (void)hipGetDevice(&dev);
        if (hipDeviceGetAttribute(&ncu, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess || ncu < 1) ncu = 256;
        return ncu;
    }();
    return n;
}

}  // namespace

// Sort the operators of a Hamiltonian by the halves they touch.  Operators
// that are not a real symmetric flip of two bits with the charge kept (complex
// elements, row conditions, a sign mask that mixes a one-half flip with the
// other half) leave the whole Hamiltonian to the per-tile kernel.
bool group_analyse(const hphi_basis* B, const std::vector<DevOp>& ops, bool is_complex, bool has_cond, GroupHost& out) {
    if (B->dev.sector == 0 || !B->grp.d_hord || is_complex || has_cond) return false;
    const int b_lo = B->b_lo;
    const uint64_t ml = (uint64_t(1) << b_lo) - 1;
    struct Cross {
        uint32_t mi, sm;
        int j;
        GBuildOp b;
        double c;
    };
    std::vector<Cross> lh;
    out.coef.assign(1, 0.0);
    auto coef_at = [&](double c) {
        for (size_t k = 0; k < out.coef.size(); ++k)
            if (out.coef[k] == c) return int32_t(k);
        out.coef.push_back(c);
        return int32_t(out.coef.size() - 1);
    };
    for (size_t o = 0; o < ops.size(); ++o) {
        const DevOp& op = ops[o];
        if (op.has_off) {
            if (op.bi == op.bj || op.xmask != ((uint64_t(1) << op.bi) | (uint64_t(1) << op.bj))) return false;
            if (op.cr[0] != 0.0 || op.cr[3] != 0.0 || op.cr[1] != op.cr[2]) return false;
            const uint64_t xl = op.xmask & ml, xh = op.xmask >> b_lo, sl = op.smask & ml, sh = op.smask >> b_lo;
            if (xh == 0) {
                if (sh) return false;
                out.ll.push_back(GLow{uint32_t(xl), uint32_t(sl), coef_at(op.cr[1]), coef_at(-op.cr[1]), int32_t(o), 0});
            } else if (xl == 0) {
                if (sl) return false;
                out.hh.push_back(GBuildOp{xh, sh, coef_at(op.cr[1]), coef_at(-op.cr[1]), int32_t(o), 0});
            } else {
                lh.push_back({uint32_t(xl), uint32_t(sl), __builtin_ctzll(xh), GBuildOp{xh, sh, 0, 0, int32_t(o), 0}, op.cr[1]});
            }
        }
        if (op.d[0] == 0.0 && op.d[1] == 0.0 && op.d[2] == 0.0 && op.d[3] == 0.0) continue;
        GBuildDiag d{int(op.bi), int(op.bj), -1, 0, {op.d[0], op.d[1], op.d[2], op.d[3]}};
        const bool li = int(op.bi) < b_lo, lj = int(op.bj) < b_lo;
        if (li && lj) out.dlo.push_back(d);
        else if (!li && !lj) out.dhi.push_back(d);
        else {
            if (!li) {   // the low bit first
                std::swap(d.bi, d.bj);
                std::swap(d.d[1], d.d[2]);
            }
            // split into parts of one bit each and a product term.  Where the
            // two bits enter as spins (d0 == d3, d1 == d2) the product of the
            // signs +-1 carries all but a constant, so no large parts cancel:
            //   d = (d0 + d1) / 2 + (d0 - d1) / 2 * (2 bi - 1) (2 bj - 1);
            // otherwise
            //   d = d0 + (d1 - d0) bi + (d2 - d0) bj + (d3 - d2 - d1 + d0) bi bj
            const double d0 = d.d[0], d1 = d.d[1], d2 = d.d[2], d3 = d.d[3];
            const bool spin = d0 == d3 && d1 == d2;
            double dx = (d3 - d2) - (d1 - d0);
            if (spin) {
                dx = 0.5 * (d0 - d1);
                const double c0 = 0.5 * (d0 + d1);
                if (c0 != 0.0) out.dhi.push_back(GBuildDiag{d.bj, d.bj, -1, 0, {c0, 0.0, 0.0, c0}});
            } else {
                out.dlo.push_back(GBuildDiag{d.bi, d.bi, -1, 0, {0.0, 0.0, 0.0, d1 - d0}});
                out.dhi.push_back(GBuildDiag{d.bj, d.bj, -1, 0, {d0, 0.0, 0.0, d2}});
            }
            if (dx != 0.0) {
                const uint32_t key = uint32_t(d.bi) | (spin ? 32u : 0u);
                int col = -1;
                for (size_t q = 0; q < out.ci.size(); ++q)
                    if (out.ci[q] == key) col = int(q);
                if (col < 0) {
                    col = int(out.ci.size());
                    out.ci.push_back(key);
                }
                out.dx.push_back(GBuildDiag{d.bi, d.bj, col, spin ? 1 : 0, {0.0, 0.0, 0.0, dx}});
            }
        }
    }
    if (out.coef.size() > size_t(kGroupCoef)) return false;
    // one column per low bit and sign mask, its operators next to each other
    std::vector<char> done(lh.size(), 0);
    for (size_t a = 0; a < lh.size(); ++a) {
        if (done[a]) continue;
        for (size_t b = a; b < lh.size(); ++b) {
            if (done[b] || lh[b].mi != lh[a].mi || lh[b].sm != lh[a].sm) continue;
            done[b] = 1;
            out.lh.push_back(GCross{lh[b].j, int32_t(out.col.size()), lh[b].b.op, 0, lh[b].c});
            out.lh_build.push_back(lh[b].b);
        }
        out.col.push_back(GColumn{lh[a].mi, lh[a].sm});
    }
    // Padding is never live, so it reads nothing: its column flips and holds no
    // bit, and bit 31 of a high half (26 bits at most) is zero.  A test in the
    // kernel instead costs 5% where the rows are wide: 18-site Hubbard, 3.4e8
    // rows of four complex64 79.0 -> 83.3 ms.
    if (out.lh.size() % size_t(kGroupPad)) out.col.push_back(GColumn{0, 0});
    while (out.lh.size() % size_t(kGroupPad)) {
        out.lh.push_back(GCross{31, int32_t(out.col.size()) - 1, -1, 0, 0.0});
        out.lh_build.push_back(GBuildOp{0, 0, 0, 0, -1, 0});
    }
    // the tables stay below half of an 8-byte vector, or small
    const size_t bytes = group_table_bytes(size_t(B->grp.n_slot), size_t(1) << b_lo, out);
    if (bytes > (size_t(16) << 20) && bytes > size_t(B->dim) * 4) return false;
    return true;
}

// Order the high halves and deal their groups to the XCDs.  The top bits of
// the high half come first: a segment of them holds at most about 96 MB of an
// 8-byte vector, so the partner blocks of the operators on the other bits stay
// in the 256 MB memory-side cache while the eight XCDs sweep the segment
// together.  The order is one for all row widths: with rows of 32 bytes a segment
// is 384 MB and only part of it stays there.  Inside it the charge classes, and inside a class ascending high
// halves in groups of K.  A group goes to the XCD with the fewest items so far,
// whole, so that the blocks of a group are read through one L2.
void group_order(const hphi_basis* B, const std::vector<uint64_t>& h_val, const std::vector<uint32_t>& h_lobase,
                 const std::vector<uint32_t>& cls_off, const std::vector<uint32_t>& cls_count, GroupBasis& gb,
                 std::vector<char>& image) {
    const int ncls = int(cls_count.size());
    const size_t n_high = h_val.size();
    int seg = 0;
    while (seg < 12 && seg < B->b_hi - 8 && ((B->dim * 8) >> seg) > (int64_t(96) << 20)) ++seg;
    const int shift = B->b_hi - seg;
    std::vector<int> cls_of(size_t(cls_off[size_t(ncls)]) + 1, 0);
    for (int c = 0; c < ncls; ++c)
        if (cls_count[size_t(c)]) cls_of[cls_off[size_t(c)]] = c;
    std::vector<GClass> cls;
    std::vector<int> slot(size_t(ncls), -1);
    std::vector<char> used(size_t(ncls), 0);
    for (size_t k = 0; k < n_high; ++k) used[size_t(cls_of[h_lobase[k]])] = 1;
    for (int c = 0; c < ncls; ++c) {
        if (!used[size_t(c)]) continue;
        slot[size_t(c)] = int(cls.size());
        const uint32_t nt = (cls_count[size_t(c)] + 63) / 64;
        cls.push_back(GClass{cls_off[size_t(c)], cls_count[size_t(c)], nt, 0});
    }
    gb.n_cls = int(cls.size());
    // segments of equal top bits are contiguous (h_val ascends)
    struct Run {
        uint32_t p0, n, cls;
    };
    std::vector<Run> runs;
    std::vector<uint32_t> hord;
    hord.reserve(n_high + n_high / 8);
    std::vector<std::vector<uint32_t>> of_cls(cls.size());
    for (size_t a = 0; a < n_high;) {
        size_t b = a;
        for (; b < n_high && (h_val[b] >> shift) == (h_val[a] >> shift); ++b)
            of_cls[size_t(slot[size_t(cls_of[h_lobase[b]])])].push_back(uint32_t(b));
        for (size_t c = 0; c < cls.size(); ++c) {
            std::vector<uint32_t>& o = of_cls[c];
            if (o.empty()) continue;
            runs.push_back(Run{uint32_t(hord.size()), uint32_t(o.size()), uint32_t(c)});
            hord.insert(hord.end(), o.begin(), o.end());
            while (hord.size() % size_t(kGroupSlots)) hord.push_back(o.back());
            o.clear();
        }
        a = b;
    }
    gb.n_slot = uint32_t(hord.size());
    for (const Run& r : runs) gb.n_item += int64_t(r.n) * cls[r.cls].n_tile;
    auto put = [&](const void* src, size_t bytes) {
        const size_t o = image.size();
        image.resize(o + (bytes + 255) / 256 * 256);
        std::copy_n(static_cast<const char*>(src), bytes, image.data() + o);
        return o;
    };
    put(hord.data(), hord.size() * 4);
    gb.cls_at = put(cls.data(), cls.size() * sizeof(GClass));
    for (int i = B->dim >= kGroupLarge ? 2 : 0; i < 4; ++i) {
        const uint32_t K = 1u << i;
        std::vector<GGroup> of[8];
        uint32_t items[8] = {};
        for (const Run& r : runs)
            for (uint32_t k = 0; k < r.n; k += K) {
                const int x = int(std::min_element(items, items + 8) - items);
                of[x].push_back(GGroup{items[x], r.p0 + k, r.cls, std::min(K, r.n - k)});
                items[x] += cls[r.cls].n_tile;
            }
        std::vector<GGroup> all;
        for (int x = 0; x < 8; ++x) {
            gb.begin[i][x] = uint32_t(all.size());
            gb.items[i][x] = items[x];
            all.insert(all.end(), of[x].begin(), of[x].end());
            all.push_back(GGroup{items[x], 0, 0, 0});
        }
        gb.begin[i][8] = uint32_t(all.size());
        gb.groups_at[i] = put(all.data(), all.size() * sizeof(GGroup));
    }
}

int group_build(const hphi_basis* B, const GroupBuild& G) {
    const uint32_t n_slot = B->grp.n_slot;
    group_high_kernel<<<(n_slot + 255) / 256, 256, 0, nullptr>>>(G, B->dev, B->grp.d_hord, n_slot);
    int rc = check_hip(hipGetLastError(), "group_high launch");
    if (rc) return rc;
    group_low_kernel<<<((1u << B->b_lo) + 255) / 256, 256, 0, nullptr>>>(G, B->dev);
    rc = check_hip(hipGetLastError(), "group_low launch");
    return rc ? rc : check_hip(hipStreamSynchronize(nullptr), "hphi_ham_build: sector tables");
}

// High halves per wavefront and lanes per row, from the wavefronts there are at
// one high half each (items of a tile of at most 64 low halves, times the lanes
// per row): more high halves share one decode and put more gathers in flight,
// but leave fewer wavefronts for the 1,024 SIMDs.  Microseconds at K = 1 / 2 / 4 / 8:
//   rows of one or two scalars: 48,620 FP32 rows (932 wavefronts) 14 / 19 / 23 / 33;
//     46,376 (3,693) 14.8 / 13.9 / 16.4 / 20; 376,740 (11,142) 22.5 / 18.4 / 17.1 /
//     20.6; from 4,194,304 rows on 8: 20,058,300 FP64 rows 1,030 / 630 / 590 / 570
//   rows of four: 48,620 complex128 x 2 20 / 24 / 34; 184,756 (3,280) 37.4 / 40.3 /
//     49.9; 376,740 39 / 35 / 31; 853,776 (15,196 wavefronts) 76 / 72 / 83; 2,704,156
//     133 / 126 / 131
//   wider rows: 63,504 complex64 x 8 (5,696) 25 / 19.5 / 26; 376,740 x 4 (22,284)
//     51 / 47 / 40; 184,756 x 4 (6,560) 23.6 / 24.6 / 20.3
// FP64 rows of 8 or 16 scalars have twice the lanes between 3,072 and 16,384
// items, where four high halves leave a SIMD a wavefront or two of them (352,716
// rows of 8 FP64 104 -> 79 us in the triangular, 72 -> 59 in the kagome lattice;
// above, 2,035,800 rows lose, 439 -> 473 us).
// Sparse FP64 sectors, at most 50 rows to an item, have short classes that leave part
// of a tile idle:
//   spins, 8 or 16 scalars, from 4,096 items: four at the plain lanes (134,596 rows of
//     8 FP64, triangular lattice 67.5 -> 55.8; 296,010 146 -> 124; kagome 40 -> 34.7;
//     3 of 28 sectors lose, by 3 to 8%).  Fermions hold the signs of each high half as
//     well and lose 4 to 19% by it.
//   spins, 8 scalars, 2,700 to 3,072 items, at most 25 rows each: one (53,130 rows 45.8
//     -> 38.0; with 41 rows each two, 48 against 59).
//   fermions, 16 and 32 scalars, from 2,048 items: two where full tiles take four
//     (48,400 rows of 16 complex128 68 -> 56, of 8 44.7 -> 36.6; 218,400 of 16 205 -> 179);
//     below, with at most 14 rows each, one (8,281 rows of 16 28 -> 20).
struct GroupShape {
    int k, lanes;
};

static GroupShape group_shape(int ns, bool f64, bool sign, int64_t items, int64_t rows) {
    GroupShape s{1, group_lanes(ns)};
    const int64_t waves = items * s.lanes;
    const bool large = rows >= kGroupLarge, mid = f64 && ns >= 8 && ns <= 16 && items < 16384, sparse = f64 && rows <= 50 * items;
    if (const char* e = std::getenv("HPHI_GROUP_K")) {
        const int k = std::atoi(e);
        if (((k == 1 || k == 2) && !large) || k == 4 || (k == 8 && ns <= 2)) {
            s.k = k;
            return s;
        }
    }
    if (large) s.k = ns <= 2 ? 8 : 4;
    else if (waves < (ns < 4 ? 3584 : ns == 4 && !f64 ? 3200 : 4096)) s.k = 1;
    else if (ns <= 2) s.k = waves < 9216 ? 2 : 4;
    else if (ns == 4) s.k = 2;
    else if (mid && sparse && !sign && items >= 4096) s.k = 4;
    else if (mid && items >= 3072) s = GroupShape{4, 2 * s.lanes};
    else if (mid && !sign && ns == 8 && rows <= 25 * items && items >= 2700) s.k = 1;
    else if (sparse && sign && ns >= 16 && items >= 2048 && (ns > 16 || items < 4096)) s.k = 2;
    else if (sign && f64 && ns >= 16 && rows <= 14 * items && items < 2048) s.k = 1;
    else s.k = waves < 6144 ? 2 : 4;
    return s;
}

// Spaces that hold a large part of all configurations, with many operators per
// bit: there the ascending order of the per-tile kernel keeps a partner's rows in
// the L2 by itself, and the class order, which spreads neighbouring high halves
// over the XCDs, re-reads wide rows (2,704,156 rows of 8 FP64, triangular lattice:
// per tile 619 us, class-blocked 729; kagome 431 against 507; two operators fewer
// per bit, chain: 249 against 256).  Sparser spaces, narrower rows and fewer
// operators gain from the shared decode throughout.
bool group_prefers_tiles(const hphi_ham* H, int nvec, int dtype) {
    const hphi_basis* B = H->basis;
    if (!H->grp) return false;
    const bool f64 = dtype == HPHI_F64 || dtype == HPHI_C128;
    const int ns = nvec * (dtype_complex(dtype) ? 2 : 1);
    const size_t row = size_t(nvec) * dtype_size(dtype);
    int n_off = 0;
    for (const DevOp& o : H->ops) n_off += o.has_off ? 1 : 0;
    const double fill = std::ldexp(double(B->dim), -B->nbits), per_bit = double(n_off) / B->nbits;
    const int64_t items = B->grp.n_item;
    if (f64 && row >= 64 && items >= 16384 &&
        ((fill > 1.0 / 11 && per_bit >= 1.5 && B->dim < kGroupLarge) || (row == 64 && fill > 1.0 / 30 && per_bit >= 2.5)))
        return true;
    // 352,716 rows of 4 complex64, triangular lattice: 74 us per tile, 96 class-blocked
    return !f64 && ns == 8 && fill > 1.0 / 11 && per_bit >= 2.5 && items >= 3072 && items < 16384;
}

static void group_args(const hphi_ham* H, int k, bool cplx, HvgArgs& A) {
    const GroupBasis& g = H->basis->grp;
    const int i = k == 8 ? 3 : k == 4 ? 2 : k == 2 ? 1 : 0;
    A.plan = *H->grp;
    A.grp.groups = g.d_groups[i];
    for (int x = 0; x < 9; ++x) A.grp.begin[x] = g.begin[i][x];
    for (int x = 0; x < 8; ++x) A.grp.items[x] = g.items[i][x];
    A.cls = g.d_cls;
    A.lows = H->basis->dev.lows;
    A.cshift = cplx ? 1 : 0;
}

int try_launch_hvg(const HvLaunch& L, const Schedule& sc, hipStream_t st) {
    const hphi_ham* H = L.ham;
    const hphi_basis* B = H->basis;
    if (!H->grp || sc.sector_blocks != 2 || (B->nbits > 32 && L.nvec > 4)) return 1;
    const bool cplx = dtype_complex(L.dtype), f64 = L.dtype == HPHI_F64 || L.dtype == HPHI_C128;
    if (L.ex && !cplx) return 1;
    const int ns = L.nvec * (cplx ? 2 : 1);
    const GroupShape g = group_shape(ns, f64, B->desc.particle == HPHI_FERMION, B->grp.n_item, B->dim);
    HvgArgs A{};
    group_args(H, g.k, cplx, A);
    A.v = L.v;
    A.u = L.u;
    A.y = L.y;
    A.cy = L.cy;
    A.sx = L.sx;
    A.a = L.a;
    A.b = L.b;
    A.stop = L.stop;
    A.partials = H->d_partials;
    A.tail = L.tail;
    if (L.ex) {
        A.ex = *L.ex;
        const int64_t most = std::min<int64_t>(L.ex->nrows, A.plan.n_low);   // rows of one block in the range
        const dim3 blocks(std::min<uint32_t>(A.grp.begin[8], 16384u), uint32_t(std::clamp<int64_t>((most + kBlock - 1) / kBlock, 1, 8)));
        hvg_export_kernel<<<blocks, kBlock, 0, st>>>(A);
        return check_hip(hipGetLastError(), "hvg_export launch");
    }
    int grid = 0;
    const bool sign = B->desc.particle == HPHI_FERMION;
    const int rc = f64 ? launch_hvg_f64(A, L, ns, g.k, g.lanes, sign, sc.blocks_per_cu, cu_count(), st, &grid)
                       : launch_hvg_f32(A, L, ns, g.k, g.lanes, sign, sc.blocks_per_cu, cu_count(), st, &grid);
    return rc ? rc : launch_product_tail(L, grid, group_sums_max(grid), st);
}

// Several problems that all have the class-blocked tables: the problems share
// the grid in proportion to their wavefront items.
int group_multi_prepare(const HvLaunch* Ls, int n, MultiPlan* out) {
    const int dtype = Ls[0].dtype;
    for (int p = 0; p < n; ++p)
        if (!Ls[p].ham->grp || schedule_for(Ls[p].ham, 1, dtype).sector_blocks != 2) return 1;
    const bool cplx = dtype_complex(dtype), f64 = dtype == HPHI_F64 || dtype == HPHI_C128;
    const int ns = cplx ? 2 : 1;
    MultiPlan P;
    P.n = n;
    P.dtype = dtype;
    int64_t rows = 0, n_item = 0;
    for (int p = 0; p < n; ++p) {
        rows += Ls[p].ham->basis->dim;
        n_item += Ls[p].ham->basis->grp.n_item;
    }
    P.group_k = std::max(2, group_shape(ns, f64, false, n_item, rows).k);
    P.cc = false;
    std::vector<HvgArgs> args(n, HvgArgs{});
    std::vector<int64_t> items(n);
    for (int p = 0; p < n; ++p) {
        const HvLaunch& L = Ls[p];
        HvgArgs& A = args[p];
        group_args(L.ham, P.group_k, cplx, A);
        items[p] = 0;
        for (int x = 0; x < 8; ++x) items[p] += A.grp.items[x];
        P.sign = P.sign || L.ham->basis->desc.particle == HPHI_FERMION;
        A.v = L.v;
        A.u = L.u;
        A.y = L.y;
        A.cy = L.cy;
        A.sx = L.sx;
        A.a = L.a;
        A.b = L.b;
        A.stop = L.stop;
    }
    int occ = 1;
    if (int rc = f64 ? launch_hvg_multi_f64(nullptr, nullptr, n, ns, P.group_k, P.sign, 0, &occ, nullptr)
                     : launch_hvg_multi_f32(nullptr, nullptr, n, ns, P.group_k, P.sign, 0, &occ, nullptr))
        return rc;
    const int cap = schedule_for(Ls[0].ham, 1, dtype).blocks_per_cu;   // as for the per-tile batch: the first problem's
    if (cap > 0 && cap < occ) occ = cap;
    const std::vector<int> begin = deal_blocks(items, int64_t(std::max(1, occ)) * cu_count() / 8);
    P.grid = begin[n];
    const size_t a_bytes = size_t(n) * sizeof(HvgArgs);
    const size_t b_off = (a_bytes + 255) / 256 * 256;
    const size_t p_off = b_off + (size_t(n + 1) * 4 + 255) / 256 * 256;
    const size_t total = p_off + size_t(P.grid) * kNQ * sizeof(double);
    char* mem = nullptr;
    if (int rc = dev_alloc((void**)&mem, total, "hv_multi_prepare")) return rc;
    double* partials = reinterpret_cast<double*>(mem + p_off);
    for (int p = 0; p < n; ++p) {
        args[p].partials = partials + size_t(begin[p]) * kNQ;
        args[p].tail = Ls[p].tail;
        args[p].tail.flag = Ls[p].ham->d_flag;
    }
    hipError_t e = hipMemcpy(mem, args.data(), a_bytes, hipMemcpyHostToDevice);
    if (e == hipSuccess) e = hipMemcpy(mem + b_off, begin.data(), size_t(n + 1) * 4, hipMemcpyHostToDevice);
    if (e != hipSuccess) {
        (void)hipFree(mem);
        return check_hip(e, "hv_multi_prepare: upload");
    }
    P.mem = mem;
    P.d_args = mem;
    P.d_begin = reinterpret_cast<const int*>(mem + b_off);
    *out = P;
    return HPHI_OK;
}

int group_multi_launch(const MultiPlan& P, hipStream_t st) {
    const HvgArgs* a = static_cast<const HvgArgs*>(P.d_args);
    const int ns = dtype_complex(P.dtype) ? 2 : 1;
    return P.dtype == HPHI_F64 || P.dtype == HPHI_C128
               ? launch_hvg_multi_f64(a, P.d_begin, P.n, ns, P.group_k, P.sign, P.grid, nullptr, st)
               : launch_hvg_multi_f32(a, P.d_begin, P.n, ns, P.group_k, P.sign, P.grid, nullptr, st);
}

}  // namespace hphi
