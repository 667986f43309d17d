// Class-blocked product on sector bases: tables shared by the host code and
// the gfx950 kernels.
//
// The rows of a sector basis with high half h are the low halves of one charge
// class, the same list for every h that needs that class.  So an operator that
// touches the low half picks the same partner ranks, the same live rows and the
// same low-half sign in all of them, and an operator that leaves the low half
// alone picks one partner block and one coefficient for all rows of h.  A
// wavefront therefore takes 64 low halves of one class together with K high
// halves that need it: the partners of a low half come from a list that is read
// once for the K blocks, and what depends on the high half alone is read as
// scalars.  The tables are built once per Hamiltonian on the device.
#pragma once

#include <cstdint>
#include <vector>

#include "hphi_internal.h"

namespace hphi {

constexpr int kGroupPad = 8;   // lists are padded to a multiple of it
constexpr int kGroupEnt = 4;             // and the partner blocks of a high half to a multiple of it
constexpr int kGroupSlots = 8;           // high halves of one class are padded to a multiple of it
constexpr int kGroupCoef = 256;          // signed elements a low-half list can name (one byte)
constexpr uint32_t kGroupRank = 0xFFFFFFu;   // rank bits of a list entry

// Lanes per row of ns scalars: at most 16 bytes of an FP32 row and 32 of an FP64
// row to a lane.  Four lanes for rows of 32 scalars leave each lane twice that,
// one gather in flight and K times 8 sums: 2,220,075 rows of 16 complex64 take
// 1,260 us in the per-tile kernel, 1,690 with four lanes, 1,085 with eight.
constexpr int group_lanes(int ns) { return ns <= 4 ? 1 : ns <= 8 ? 2 : ns <= 16 ? 4 : 8; }

// partials up to which plain sums stay in a launch of `grid` blocks
constexpr int group_sums_max(int grid) { return grid <= 256 ? kSumsMaxShort : kSumsMax; }

// one charge class of the low half
struct GClass {
    uint32_t l_off, n_l;      // its low halves in `lows`
    uint32_t n_tile, pad;     // its 64-row tiles
};

// K slots p0 .. p0 + K - 1 of one class, the first n of them its own high halves
// and the rest repeats of one: items item0 .. item0 + n_tile - 1 of its XCD
struct GGroup {
    uint32_t item0;
    uint32_t p0;
    uint32_t cls;
    uint32_t n;
};

// the groups of one K: XCD x owns groups[begin[x]] .. groups[begin[x + 1]] (the
// last one closes its item range)
struct GGroups {
    const GGroup* groups;
    uint32_t begin[9];
    uint32_t items[8];
};

// operator inside the low half: flips m (two bits), sign parity of l & sm;
// pos/neg: its element and its negative in the coefficient list
struct GLow {
    uint32_t m, sm;
    int32_t pos, neg;
    int32_t op, pad;
};

// low side of the operators with one bit in each half: flips mi, sign parity
// of l & sm
struct GColumn {
    uint32_t mi, sm;
};

// an operator with one bit in each half: bit j of the high half, its column and
// its element (padding: op -1, element 0)
struct GCross {
    int32_t j, col, op, pad;
    double c;
};

// operator as the table builder reads it
struct GBuildOp {
    uint64_t m_hi, sm_hi;     // flip and sign masks in the high half
    int32_t pos, neg;         // its element and its negative in the coefficient list
    int32_t op, pad;
};

// diagonal term of the low half, the high half or of both: d[p] over bits (bi, bj)
struct GBuildDiag {
    int32_t bi, bj;           // bit positions in the configuration
    int32_t ci;               // >= 0: column of a cross term
    int32_t spin;             // 1: the bits enter as signs +-1
    double d[4];
};

// rows of a padded list: the batches of a kernel and one of reading ahead
constexpr int group_rows(int n) { return (n + kGroupPad - 1) / kGroupPad * kGroupPad + kGroupPad; }

struct GroupPlan {
    int n_ll = 0, n_lh = 0, n_col = 0, n_ci = 0, n_hh = 0, hh_stride = 0, n_coef = 0;
    uint32_t n_slot = 0, n_low = 0;
    // per slot: first row, configuration, entries of the operators inside the
    // high half, diagonal part of the high half
    const int64_t* row0 = nullptr;
    const uint32_t* hval = nullptr;
    const uint32_t* n_ent = nullptr;
    const double* dhi = nullptr;
    const uint64_t* hh = nullptr;    // [n_slot][hh_stride] first row of the partner block | coefficient << 48 (0: padding)
    const int64_t* lhe = nullptr;    // [n_lh][n_slot] first row of the partner block | high-half sign << 63
    const double* w = nullptr;       // [n_ci][n_slot]
    const uint32_t* ci = nullptr;    // [n_ci] low bit of each cross-diagonal column; + 32: it enters as a sign
    const double* dlo = nullptr;     // [n_low], the order of `lows`
    const uint32_t* nbr = nullptr;   // [n_ll, padded twice][n_low]: partner rank | coefficient << 24 (0: row not touched)
    const uint32_t* xnb = nullptr;   // [n_col][n_low]: rank of l ^ mi | (sign << 30) | (bit of l << 31)
    const double* coef = nullptr;    // [n_coef], coef[0] = 0
    const GCross* lh = nullptr;      // [n_lh], padded; one padding more
    // element export
    const GLow* ll_ops = nullptr;    // [n_ll]
    const GBuildOp* hh_ops = nullptr;
};

// the operators of a Hamiltonian sorted by the halves they touch (host)
struct GroupHost {
    std::vector<GLow> ll;
    std::vector<double> coef;
    std::vector<GColumn> col;
    std::vector<GCross> lh;
    std::vector<GBuildOp> hh, lh_build;
    std::vector<GBuildDiag> dlo, dhi, dx;
    std::vector<uint32_t> ci;
};

// partner blocks of a high half, padded to whole batches
inline size_t group_ent_stride(const GroupHost& g) { return (g.hh.size() + kGroupEnt - 1) / kGroupEnt * kGroupEnt; }

// bytes of the tables, the padding of the lists of low halves left out: per slot the
// first row, the configuration, the entries, the diagonal part and 8 bytes per
// operator; per low half 8 and 4 per operator
inline size_t group_table_bytes(size_t n_slot, size_t n_low, const GroupHost& g) {
    return n_slot * (24 + 8 * (group_ent_stride(g) + g.lh.size() + g.ci.size())) +
           n_low * (8 + 4 * (g.ll.size() + g.col.size()));
}

// what the table builder reads and writes (device)
struct GroupBuild {
    const GBuildOp* op_hh;
    const GBuildOp* op_lh;
    const GBuildDiag* dlo_ops;
    const GBuildDiag* dhi;
    const GBuildDiag* dx;
    const GLow* ll;
    const GColumn* col;
    int n_hh, n_lh, n_dlo, n_dhi, n_x, n_ci, hh_stride, n_ll, n_col;
    int64_t* row0;
    uint32_t* hval;
    uint32_t* n_ent;
    double* dhi_out;
    uint64_t* hh;
    int64_t* lhe;
    double* w;
    double* dlo;
    uint32_t* nbr;
    uint32_t* xnb;
};

// the groups of a basis and their device image (group.hip)
void group_order(const hphi_basis* B, const std::vector<uint64_t>& h_val, const std::vector<uint32_t>& h_lobase,
                 const std::vector<uint32_t>& cls_off, const std::vector<uint32_t>& cls_count, GroupBasis& gb,
                 std::vector<char>& image);

bool group_analyse(const hphi_basis* B, const std::vector<DevOp>& ops, bool is_complex, bool has_cond, GroupHost& out);
int group_build(const hphi_basis* B, const GroupBuild& G);
// arguments of one class-blocked product
struct HvgArgs {
    GroupPlan plan;
    GGroups grp;
    const GClass* cls;
    const uint32_t* lows;
    int32_t cshift, pad;             // cshift 1: complex vectors (two columns per vector)
    const void* v;
    void* u;
    const void* y;
    const double* cy;
    const double* sx;
    double a, b;
    const int* stop;
    double* partials;
    Tail tail;
    ExportArgs ex;
};

}  // namespace hphi
