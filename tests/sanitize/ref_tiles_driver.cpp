// Host-only replay of the tile schedules of the refactorization (RefTiles) and of the solves
// (SolveTiles), built with AddressSanitizer and UndefinedBehaviorSanitizer by
// tests/test_ref_tiles.py: reads a CSR system
// from a binary file (int64 n, int64 nnz, double tau, int32 ordering, int32 ref_lds; then rowptr,
// colidx, values of system 1, values of system 2), runs the analysis and refactors system 2 as
// the tile kernel does: tiles in hand-out order, entries and externals in slots, segments of
// items (each entry read before it is final, each export read before it is written, and each
// solve-layout position written twice or never is an error), the pivot guard with column
// maxima gathered from the tile's own entries and its extras.  Writes L and U in exchange
// layout and prints tiles=<count> layers=<count> refactor=<ok or the first violated property>.
// Both sweeps are replayed with the factors of system 2 the same way (tasks in hand-out order,
// chunks from slots; a value read before it is written, a place read out of range, a row solved
// twice or never is an error) and compared with plain substitution: solve=ok:<relative difference>.
#include <cmath>
#include <cstdio>
#include <cstdint>
#include <limits>
#include <string>
#include <vector>

#include "../../paper_2401_13926_amd/csrc/analysis.hpp"

namespace {

const double kNaN = std::numeric_limits<double>::quiet_NaN();

std::string replay(const kkt::Analysis &a, int64_t budget, const std::vector<double> &vals, std::vector<double> &lx,
                   std::vector<double> &ux, int64_t &guarded) {
    const kkt::RefTiles &t = a.ref;
    std::vector<double> kval(a.ksrc.size()), tv(a.t_size, 0.0), X(t.exp.size(), kNaN);
    for (size_t k = 0; k < kval.size(); ++k) kval[k] = vals[a.ksrc[k]];
    std::vector<int> written(a.t_size, 0);
    guarded = 0;
    int64_t entries = 0, nodes = 0;
    for (int64_t ti = 0; ti < t.tiles(); ++ti) {
        const int32_t *d = t.desc.data() + kkt::kRefDesc * ti;
        const int32_t ns = d[1], ne = d[3], ni = d[5], nu = d[7], nl = d[9], nx = d[13], nn = d[14];
        entries += ne;
        nodes += nn;
        if (kkt::ref_lds_bytes(ne, nx, nn, nu, ni, nl) > budget) return "lds_budget";
        std::vector<double> xs(ne + nx), cm(nn, 0.0);
        for (int32_t e = 0; e < ne; ++e) {
            const int32_t s = t.src.at(d[2] + e);
            xs[e] = s >= 0 ? kval.at(s) : 0.0;
            const uint16_t c = t.col.at(d[2] + e);
            if (c != 0xFFFF) cm.at(c) = std::fmax(cm[c], std::fabs(xs[e]));
        }
        for (int32_t k = 0; k < d[16]; ++k) {
            double &c = cm.at(t.cmx_node.at(d[15] + k));
            c = std::fmax(c, std::fabs(kval.at(t.cmx_src.at(d[15] + k))));
        }
        for (int32_t k = 0; k < nx; ++k) {
            xs[ne + k] = X.at(t.ext.at(d[12] + k));
            if (std::isnan(xs[ne + k])) return "external_not_final";
        }
        std::vector<uint8_t> final_(ne + nx, 0);
        for (int32_t k = 0; k < nx; ++k) final_[ne + k] = 1;
        int32_t i0 = 0, n0 = 0, q0 = 0;
        for (int32_t g = 0; g < ns; ++g) {
            const uint32_t w0 = t.seg.at(2 * (d[0] + g)), w1 = t.seg.at(2 * (d[0] + g) + 1);
            const int32_t i1 = w0 & 0xFFFF, sl0 = w0 >> 16, n1 = w1 & 0xFFFF, q1 = w1 >> 16;
            const int32_t nd = n1 - n0, nq = q1 - q0, nlq = nq - nd;
            if (nd < 1 || nlq < 0 || sl0 + nq > ne) return "segment_shape";
            std::vector<uint8_t> touched(ne, 0);
            for (int32_t i = i0; i < i1; ++i) {
                const uint32_t ia = t.item.at(2 * (d[4] + i)), ie = t.item.at(2 * (d[4] + i + 1));
                const uint32_t s = (ia & 0xFFFF) / 8;
                if ((ia & 7) || (int32_t)s >= ne || final_[s] || touched[s]++) return "item_target";
                if ((ie >> 16) < (ia >> 16) || (int32_t)(ie >> 16) > nu) return "item_updates";
                for (int64_t u = -1; u < (int64_t)(ie >> 16) - (int64_t)(ia >> 16); ++u) {
                    const uint32_t p = u < 0 ? t.item.at(2 * (d[4] + i) + 1) : t.upd.at(d[6] + (ia >> 16) + u);
                    const uint32_t l = (p & 0xFFFF) / 8, f = (p >> 16) / 8;
                    if ((p & 7) || (p >> 16 & 7) || !final_.at(l) || !final_.at(f)) return "factor_not_final";
                    const double prod = xs[l] * xs[f];
                    xs[s] = xs[s] - prod;
                }
            }
            for (int32_t k = 0; k < nd; ++k) {
                double &p = xs[sl0 + nlq + k];
                const double c = cm.at(n0 + k) > 0.0 ? cm[n0 + k] : 1.0;
                if (!(std::fabs(p) > 0x1p-53 * c) || !std::isfinite(p)) {
                    p = (p < 0.0 ? -1.0 : 1.0) * 0x1p-53 * c;
                    ++guarded;
                }
                final_[sl0 + nlq + k] = 1;
            }
            for (int32_t q = 0; q < nq; ++q) {
                const int32_t piv = t.lq.at(d[8] + q0 + q) / 8, e = sl0 + q;
                if ((t.lq[d[8] + q0 + q] & 7) || piv < sl0 + nlq || piv >= sl0 + nq || (q >= nlq && piv != e)) return "pivot";
                if (q >= nlq) continue;
                xs[e] = xs[e] / xs[piv];
                final_[e] = 1;
            }
            // the rest of the segment's slots are its nodes' U entries
            const int32_t end = g + 1 < ns ? (int32_t)(t.seg.at(2 * (d[0] + g + 1)) >> 16) : ne;
            for (int32_t e = sl0 + nq; e < end; ++e) final_[e] = 1;
            i0 = i1;
            n0 = n1;
            q0 = q1;
        }
        if (i0 != ni || n0 != nn || q0 != nl) return "segment_totals";
        for (int32_t k = 0; k < d[11]; ++k) {
            const uint16_t e = t.exp.at(d[10] + k);
            if (e >= ne) return "export_slot";
            X.at(d[10] + k) = xs[e];
        }
        for (int32_t e = 0; e < ne; ++e) {
            const int32_t pos = t.out_pos.at(d[2] + e);
            if (e && pos <= t.out_pos[d[2] + e - 1]) return "out_order";
            if (written.at(pos)++) return "written_twice";
            tv[pos] = xs.at(t.out_slot.at(d[2] + e));
        }
    }
    if (entries != a.nnz_f() || nodes != a.n) return "entries_lost";
    lx.resize(a.nnz_l());
    ux.resize(a.nnz_u());
    for (size_t p = 0; p < lx.size(); ++p) lx[p] = tv.at(a.f2t.at(a.l2f[p]));
    for (size_t p = 0; p < ux.size(); ++p) ux[p] = tv.at(a.f2t.at(a.u2f[p]));
    return "ok";
}

std::string replay_solve(const kkt::Analysis &a, const std::vector<double> &lx, const std::vector<double> &ux) {
    const kkt::SolveTiles &t = a.sol;
    const int64_t n = a.n;
    std::vector<double> tv(a.t_size, 0.0), b(n), ref(n);
    for (size_t p = 0; p < lx.size(); ++p) tv.at(a.f2t.at(a.l2f[p])) = lx[p];
    for (size_t p = 0; p < ux.size(); ++p) tv.at(a.f2t.at(a.u2f[p])) = ux[p];
    for (int64_t i = 0; i < n; ++i) b[i] = std::sin(1.0 + 0.7 * (double)i);
    // plain substitution in step space from the exchange layout (li holds original rows)
    for (int64_t k = 0; k < n; ++k) ref[k] = b[a.prow[k]];
    for (int64_t k = 0; k < n; ++k)
        for (int64_t p = a.lp[k]; p < a.lp[k + 1]; ++p) ref[a.pinv[a.li[p]]] -= lx[p] * ref[k];
    for (int64_t k = n - 1; k >= 0; --k) {
        ref[k] /= ux[a.up[k + 1] - 1];
        for (int64_t p = a.up[k]; p < a.up[k + 1] - 1; ++p) ref[a.ui[p]] -= ux[p] * ref[k];
    }
    const int64_t ub = (int64_t)t.ref_l.size(), db = ub + (int64_t)t.ref_u.size();
    if (db + n != a.t_size) return "solve_layout_size";
    std::vector<double> y(n, kNaN), z(n, kNaN);
    for (int64_t w = 0; w < 2 * t.tiles(); ++w) {
        const bool up = w >= t.tiles();
        const int32_t *d = t.desc.data() + kkt::kSolDesc * (up ? 2 * t.tiles() - 1 - w : w);
        const int32_t *e = d + (up ? 2 + kkt::kSolSweep : 2);
        const int32_t base = d[0], nr = d[1], nc = e[1], np = e[3], nx = e[5];
        const auto &chunk = up ? t.chunk_u : t.chunk_l;
        const auto &ref16 = up ? t.ref_u : t.ref_l;
        const auto &ext = up ? t.ext_u : t.ext_l;
        std::vector<double> &out = up ? z : y;
        if (kkt::sol_lds_bytes(nr, nx, np, e[7]) > t.lds || (np & 1) || (e[2] & 1) || (e[8] & 1)) return "solve_lds";
        if (e[7] && (e[7] > 64 || e[6] + e[7] > nr || (up ? e[9] > nc : e[9] != nc))) return "dense_shape";
        std::vector<double> xs(nr + nx + 1, 0.0);
        std::vector<uint8_t> fin(nr + nx + 1, 0);  // 0 not final, 1 for wavefront 0 only, 2 for all
        for (int32_t r = 0; r < nr; ++r) xs[r] = up ? y.at(t.pos_u.at(base + r)) : b[a.prow[t.node_l.at(base + r)]];
        for (int32_t k = 0; k <= nx; ++k) fin[nr + k] = 2;
        for (int32_t k = 0; k < nx; ++k) xs[nr + k] = out.at(ext.at(e[4] + k));
        for (double v : xs)
            if (std::isnan(v)) return "solve_input_not_final";
        std::vector<double> res(nr, kNaN);
        // rows of L without entries need no chunk: their slots hold the solution from the start
        for (int32_t r = 0; r < nr && !up; ++r) {
            const int32_t k = t.node_l[base + r];
            if (a.lrp[k] == a.lrp[k + 1] && !(e[7] && r >= e[6] && r < e[6] + e[7])) {
                res[r] = xs[r];
                fin[r] = 2;
            }
        }
        std::vector<int32_t> fresh;  // rows of the segment under way: final only after it
        std::vector<int32_t> seen0;  // rows with fin = 1
        bool one_wave = true;
        auto barrier = [&]() {
            for (int32_t r : fresh) fin[r] = 2;
            for (int32_t r : seen0) fin[r] = 2;
            fresh.clear();
            seen0.clear();
            one_wave = true;
        };
        std::vector<uint8_t> raw(nr, 0);
        auto sweep = [&]() -> std::string {
            const int32_t m = e[7], r0 = e[6];
            std::vector<double> tri(m * (m - 1) / 2 + 1, 0.0);
            for (int32_t k = 0; k < e[8]; ++k)
                tri.at(ref16.at(e[2] + np + k)) = tv.at((up ? ub : 0) + e[2] + np + k);
            barrier();
            for (int32_t c = 0; c < m; ++c) {
                if (!raw[r0 + c] && !std::isnan(res[r0 + c])) return "dense_row";
                double x = xs[r0 + c];
                if (up) x /= tv.at(db + base + r0 + c);
                for (int32_t l = c + 1; l < m; ++l) xs[r0 + l] -= tri[c * m - c * (c + 1) / 2 + (l - c - 1)] * x;
                xs[r0 + c] = res[r0 + c] = x;
                fresh.push_back(r0 + c);
            }
            return "";
        };
        for (int32_t c = 0; c < nc; ++c) {
            if (up && e[7] && c == e[9]) {
                const std::string s = sweep();
                if (!s.empty()) return s;
            }
            const uint32_t w0 = chunk.at(2 * (e[0] + c)), w1 = chunk.at(2 * (e[0] + c) + 1);
            const int32_t r0 = w0 & 0x1FFF, cnt = (w0 >> 13) & 0x7F, lg = (w0 >> 20) & 7, half = (w0 >> 23) & 0xFF;
            const int32_t off = w1 & 0x0FFFFFFF, wave = w1 >> 30;
            if ((w1 >> 28 & 1) && (half != 2 || wave != 0 || (w0 >> 31) || (w1 >> 29 & 1))) return "short_chunk";
            const bool rw = (w1 >> 29) & 1;
            // rows become final at a barrier, or at the next chunk while only wavefront 0 works
            if (w0 >> 31) barrier();
            if (one_wave && wave == 0) {
                for (int32_t r : fresh) fin[r] = 1;
                seen0.insert(seen0.end(), fresh.begin(), fresh.end());
                fresh.clear();
            }
            one_wave = one_wave && wave == 0;
            if (cnt < 1 || (cnt << lg) > 64 || lg > 6 || off % 2 || off + (cnt << lg) * 2 * half > np) return "chunk_shape";
            for (int32_t q = 0; q < cnt; ++q) {
                double acc = 0.0;
                for (int32_t k = 0; k < (1 << lg) * 2 * half; ++k) {
                    const int64_t at = e[2] + off + (int64_t)(q << lg) * 2 * half + k;
                    const uint16_t s = ref16.at(at);
                    if (s % 8 || fin.at(s / 8) < (wave == 0 ? 1 : 2)) return "solve_ref_not_final";
                    acc += tv.at((up ? ub : 0) + at) * xs[s / 8];
                }
                const int32_t row = r0 + q;
                if (row >= nr || !std::isnan(res[row])) return "solve_row";
                res[row] = xs[row] - acc;
                if (up && !rw) res[row] /= tv.at(db + base + row);
                raw[row] = rw;
                if (!rw) fresh.push_back(row);
                if (rw != (e[7] && row >= e[6] && row < e[6] + e[7])) return "dense_flag";
                xs[row] = res[row];
            }
        }
        if (e[7] && e[9] == nc) {
            const std::string s = sweep();
            if (!s.empty()) return s;
        }
        for (int32_t r = 0; r < nr; ++r) {
            if (std::isnan(res[r]) || !std::isnan(out.at(base + r))) return "solve_row_lost";
            out[base + r] = res[r];
        }
    }
    double diff = 0.0, scale = 0.0;
    for (int64_t p = 0; p < n; ++p) {
        diff = std::fmax(diff, std::fabs(z[p] - ref[t.node_u[p]]));
        scale = std::fmax(scale, std::fabs(ref[t.node_u[p]]));
    }
    char buf[64];
    std::snprintf(buf, sizeof buf, "ok:%.3e", diff / scale);
    return buf;
}

}  // namespace

int main(int argc, char **argv) {
    if (argc != 3) return 2;
    std::FILE *f = std::fopen(argv[1], "rb");
    if (!f) return 2;
    int64_t n = 0, nnz = 0;
    double tau = 0.0;
    int32_t ordering = 0, lds = 0;
    bool ok = std::fread(&n, 8, 1, f) == 1 && std::fread(&nnz, 8, 1, f) == 1 && std::fread(&tau, 8, 1, f) == 1 &&
              std::fread(&ordering, 4, 1, f) == 1 && std::fread(&lds, 4, 1, f) == 1;
    std::vector<int64_t> rp(ok ? n + 1 : 0);
    std::vector<int32_t> ci(ok ? nnz : 0);
    std::vector<double> v(ok ? nnz : 0), v2(ok ? nnz : 0);
    ok = ok && std::fread(rp.data(), 8, rp.size(), f) == rp.size() && std::fread(ci.data(), 4, ci.size(), f) == ci.size() &&
         std::fread(v.data(), 8, v.size(), f) == v.size() && std::fread(v2.data(), 8, v2.size(), f) == v2.size();
    std::fclose(f);
    if (!ok) return 2;
    kkt::AnalysisOptions opt;
    opt.ordering = ordering;
    opt.pivot_tau = tau;
    opt.ref_lds = lds;
    kkt::Analysis a;
    std::string msg;
    const int rc = kkt::analyze(opt, n, rp.data(), ci.data(), v.data(), a, &msg);
    if (rc != kkt::AN_OK) return 3;
    std::printf("tiles=%lld layers=%lld ", (long long)a.ref.tiles(), (long long)a.ref.layers);
    if (a.ref.tiles() > 0) {
        std::vector<double> lx, ux;
        int64_t guarded = 0;
        const std::string r = replay(a, lds, v2, lx, ux, guarded);
        std::printf("refactor=%s guarded=%lld", r.c_str(), (long long)guarded);
        if (r == "ok") {
            std::printf(" solve=%s", replay_solve(a, lx, ux).c_str());
            std::FILE *o = std::fopen(argv[2], "wb");
            if (!o) return 2;
            const bool w = std::fwrite(lx.data(), 8, lx.size(), o) == lx.size() &&
                           std::fwrite(ux.data(), 8, ux.size(), o) == ux.size();
            std::fclose(o);
            if (!w) return 2;
        }
    }
    std::printf("\n");
    return 0;
}
