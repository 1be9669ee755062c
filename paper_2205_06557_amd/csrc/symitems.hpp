// symitems.hpp -- the work item of the symmetric all-pairs sum, shared by the
// kernels (pairsym.hpp, mesh.hpp) and the host code that builds the item lists
// (worksplit.hpp).  Plain C++: constexpr functions serve both.
#pragma once

namespace odk {

// Target tile rows that share one pass over the sources (sym_rows).
constexpr int kSymRows = 3;

// rows == 1: target tile row I against source tiles [J0, J1) (sym_item), of
// each source tile only the 64-ion sub-tiles [st0, st1) (0..4: the whole
// tile); rows == kSymRows: target tile rows I .. I + kSymRows - 1 together
// (sym_rows), whole tiles.
struct SymItem {
    int I, J0, J1, rows, st0, st1;
};

// All items of one system of T tiles: groups of `rows` target tile rows, each
// group with runs of C source tiles from its first row on; rows left over at
// the end alone, with all their sources.
struct SymRuns {
    int T, rows, C;
};

// A place among them: the first row of a group, and the items before it.
struct SymPlace {
    int I, before;
};

// Item k, searched from `at` on (place {0, 0}, or where an earlier call with a
// smaller k left it).  False: there are no more.
constexpr bool sym_item_at(const SymRuns& s, int k, SymPlace& at, SymItem& it)
{
    while (at.I < s.T) {
        const bool group = at.I + s.rows <= s.T;
        const int n = group ? (s.T - at.I + s.C - 1) / s.C : 1;
        if (k < at.before + n) {
            const int J0 = group ? at.I + (k - at.before) * s.C : at.I;
            it = {at.I, J0, group && J0 + s.C < s.T ? J0 + s.C : s.T, group ? s.rows : 1, 0, 4};
            return true;
        }
        at.before += n;
        at.I += group ? s.rows : 1;
    }
    return false;
}

}  // namespace odk
