// Host-only look at the order in which the solve tiles' one launch may read b and write x, built with
// AddressSanitizer and UndefinedBehaviorSanitizer by tests/test_solve_tiles.py: reads a CSR system
// from a binary file (int64 n, int64 nnz, double tau, int32 ordering, int32 ref_lds, int64 sol_lds,
// int64 sol_dense_lds; then rowptr, colidx, values), runs the analysis (one argument more:
// its list_max) and prints
// tiles=<solve tiles> longest=<entries of the refactorization tiles' longest list> offdiag=<pivots off the diagonal>
// early=<entries of x that a U tile may write before the L tile that reads the same entry of b has
// started: that L task is not among those the U task waits for, directly or not>
// same=, shifted=, apart=<what may_overwrite answers for x = b, for x one entry after b and for
// x behind b>
// dense=<dense ranges> mixed=<those with rows of several elimination trees>.
#include <algorithm>
#include <cstdio>
#include <cstdint>
#include <string>
#include <utility>
#include <vector>

#include "../../paper_2401_13926_amd/csrc/analysis.hpp"

namespace {

int64_t early_writes(const kkt::Analysis &a) {
    const kkt::SolveTiles &t = a.sol;
    const int64_t nt = t.tiles();
    std::vector<int32_t> tile_of(a.n), reader(a.n);  // by position; by entry of b
    for (int64_t k = 0; k < nt; ++k) {
        const int32_t *d = t.desc.data() + kkt::kSolDesc * k;
        for (int32_t r = 0; r < d[1]; ++r) {
            tile_of.at(d[0] + r) = (int32_t)k;
            reader.at(a.prow.at(t.node_l.at(d[0] + r))) = (int32_t)k;
        }
    }
    // L tasks that are done when L task k, U task k have what they wait for (k itself among them)
    std::vector<std::vector<bool>> lower(nt), upper(nt);
    for (int64_t k = 0; k < nt; ++k) {
        lower[k].assign(nt, false);
        lower[k][k] = true;
        const int32_t *e = t.desc.data() + kkt::kSolDesc * k + 2;
        for (int32_t x = 0; x < e[5]; ++x) {
            const int32_t o = tile_of.at(t.ext_l.at(e[4] + x));
            for (int64_t q = 0; q < nt; ++q)
                if (lower.at(o)[q]) lower[k][q] = true;
        }
    }
    int64_t early = 0;
    for (int64_t k = nt - 1; k >= 0; --k) {
        upper[k] = lower[k];
        const int32_t *d = t.desc.data() + kkt::kSolDesc * k, *e = d + 2 + kkt::kSolSweep;
        for (int32_t x = 0; x < e[5]; ++x) {
            const int32_t o = tile_of.at(t.ext_u.at(e[4] + x));
            for (int64_t q = 0; q < nt; ++q)
                if (upper.at(o)[q]) upper[k][q] = true;
        }
        for (int32_t r = 0; r < d[1]; ++r) early += !upper[k][reader.at(a.q.at(t.node_u.at(d[0] + r)))];
    }
    return early;
}

// Dense ranges (first) and those that mix trees (second).
std::pair<int64_t, int64_t> dense_ranges(const kkt::Analysis &a) {
    std::vector<int32_t> tree(a.n);
    for (int64_t m = a.n - 1; m >= 0; --m) {
        const int64_t p = a.fp[m] + a.fdiag[m] + 1;
        tree[m] = p < a.fp[m + 1] ? tree.at(a.fi[p]) : (int32_t)m;
    }
    std::pair<int64_t, int64_t> c{0, 0};
    for (int64_t k = 0; k < 2 * a.sol.tiles(); ++k) {
        const int32_t *d = a.sol.desc.data() + kkt::kSolDesc * (k / 2);
        const int32_t *e = d + 2 + (k & 1) * kkt::kSolSweep;
        const std::vector<int32_t> &node = k & 1 ? a.sol.node_u : a.sol.node_l;
        c.first += e[7] > 0;
        for (int32_t r = 1; r < e[7]; ++r)
            if (tree[node.at(d[0] + e[6] + r)] != tree[node.at(d[0] + e[6])]) {
                ++c.second;
                break;
            }
    }
    return c;
}

}  // namespace

int main(int argc, char **argv) {
    if (argc != 2 && argc != 3) return 2;
    std::FILE *f = std::fopen(argv[1], "rb");
    if (!f) return 2;
    int64_t n = 0, nnz = 0, lds[2] = {};
    double tau = 0.0;
    int32_t opt2[2] = {};
    bool ok = std::fread(&n, 8, 1, f) == 1 && std::fread(&nnz, 8, 1, f) == 1 && std::fread(&tau, 8, 1, f) == 1 &&
              std::fread(opt2, 4, 2, f) == 2 && std::fread(lds, 8, 2, f) == 2;
    std::vector<int64_t> rp(ok ? n + 1 : 0);
    std::vector<int32_t> ci(ok ? nnz : 0);
    std::vector<double> v(ok ? nnz : 0);
    ok = ok && std::fread(rp.data(), 8, rp.size(), f) == rp.size() &&
         std::fread(ci.data(), 4, ci.size(), f) == ci.size() && std::fread(v.data(), 8, v.size(), f) == v.size();
    std::fclose(f);
    if (!ok) return 2;
    kkt::AnalysisOptions opt;
    opt.ordering = opt2[0];
    opt.pivot_tau = tau;
    opt.ref_lds = opt2[1];
    opt.sol_lds = lds[0];
    opt.sol_dense_lds = lds[1];
    if (argc == 3) opt.list_max = std::stoll(argv[2]);
    kkt::Analysis a;
    std::string msg;
    if (kkt::analyze(opt, n, rp.data(), ci.data(), v.data(), a, &msg) != kkt::AN_OK) return 3;
    std::vector<double> b(2 * n + 1);
    const size_t longest =
        std::max(std::max(a.ref.upd.size(), a.ref.item.size() / 2), std::max(a.ref.ext.size(), a.ref.src.size()));
    std::printf("tiles=%lld longest=%lld offdiag=%lld early=%lld same=%d shifted=%d apart=%d dense=%lld mixed=%lld\n", (long long)a.sol.tiles(), (long long)longest,
                (long long)a.offdiag_pivots, (long long)early_writes(a),
                (int)kkt::may_overwrite(a, b.data(), b.data()),
                (int)kkt::may_overwrite(a, b.data(), b.data() + 1),
                (int)kkt::may_overwrite(a, b.data(), b.data() + n), (long long)dense_ranges(a).first,
                (long long)dense_ranges(a).second);
    return 0;
}
