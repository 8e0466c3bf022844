// Host check of the factorisation's launch lists in either order (test infrastructure, built by the tests only).
//
// Builds the plan with the library's own host code (ordering.hip) in the natural or a nested-dissection order, checks
// that each level's panel entries are exactly its columns' tile rows, a column's entries together ((k, -1) for a
// column without any), and that the update tasks are those of a plain enumeration, in its order; then runs the
// factorisation on the CPU as the device launches it: per level one launch over the panel entries (every entry
// factors its column's diagonal block for itself; the column's first writes W and, in a nested-dissection order, the
// forward step), one over the update tasks.  A launch reads the state before it: its writes are applied at its end,
// and no two workgroups of it may write one place.  Entries outside the pattern are NaN.
//
// argv[1]: natural | nd.  stdin, stdout as nd_plan_check.cpp: int32 np, ne, ne pairs, int32 n0, anchor, float64
// lambda, H, b -> float64 dx.  Exit status 3 when a check fails.
#include "pba_internal.h"
#include <algorithm>
#include <chrono>
#include <cmath>
#include <cstdio>
#include <cstdlib>
#include <cstring>
#include <map>
#include <set>
using namespace pba;
static const int NB = 64;
#define CHECK(c) do { if (!(c)) { fprintf(stderr, "CHECK failed line %d: %s\n", __LINE__, #c); exit(3); } } while (0)

struct Mem {   // a buffer whose writes take effect at the end of a launch
    std::vector<double> v;
    std::map<long, double> pend;
    double rd(long i) const { CHECK(i >= 0 && i < (long)v.size()); return v[i]; }
    void wr(long i, double x) { CHECK(i >= 0 && i < (long)v.size()); CHECK(pend.emplace(i, x).second); }
    void end() { for (auto &p : pend) v[p.first] = p.second; pend.clear(); }
};

static std::vector<int> tasks_by_enumeration(const TilePattern &tp, int l, std::vector<int> &contrib)
{
    std::map<std::pair<int, int>, std::vector<int>> of;
    for (int k = 0; k < tp.nt; ++k)
        if (tp.level[k] == l)
            for (int x : tp.rows[k])
                for (int y : tp.rows[k])
                    if (y <= x) of[{x, y}].push_back(k);
    std::vector<std::pair<std::pair<int, int>, std::vector<int>>> list(of.begin(), of.end());
    std::stable_sort(list.begin(), list.end(), [](const auto &a, const auto &b) { return a.second.size() > b.second.size(); });
    std::vector<int> t;
    for (auto &e : list) {
        t.insert(t.end(), {e.first.first, e.first.second, (int)contrib.size(), (int)e.second.size()});
        contrib.insert(contrib.end(), e.second.begin(), e.second.end());
    }
    return t;
}

int main(int argc, char **argv)
{
    const bool nd = argc > 1 && !strcmp(argv[1], "nd");
    int np, ne, n0, anchor;
    double lam;
    CHECK(fread(&np, 4, 1, stdin) == 1 && fread(&ne, 4, 1, stdin) == 1);
    std::vector<std::pair<int, int>> edges(ne);
    for (auto &e : edges) { int st[2]; CHECK(fread(st, 4, 2, stdin) == 2); e = {st[0], st[1]}; }
    CHECK(fread(&n0, 4, 1, stdin) == 1 && fread(&anchor, 4, 1, stdin) == 1 && fread(&lam, 8, 1, stdin) == 1);
    const bool lists_only = n0 == 0;   // the lists alone, no system: for graphs too large to factor here
    std::vector<double> H((size_t)n0 * n0), b(n0);
    CHECK(fread(H.data(), 8, H.size(), stdin) == H.size() && fread(b.data(), 8, n0, stdin) == (size_t)n0);
    int n = 6 * np;
    std::vector<int> pos(np);
    for (int v = 0; v < np; ++v) pos[v] = 6 * v;
    if (nd) pos = nd_positions(np, nd_blocks(np, edges, 20), n);
    auto now = [] { return std::chrono::steady_clock::now(); };
    auto ms = [](auto d) { return std::chrono::duration<double>(d).count() * 1e3; };
    const auto t0 = now();
    const TilePattern tp = tile_pattern(n, pos, edges);
    const auto t1 = now();
    const NdArrays a = nd_arrays(tp, pos);
    const auto t2 = now();
    const int nt = tp.nt, nlev = tp.nlev;
    fprintf(stderr, "n %d nt %d levels %d tasks %zu panels %zu pattern_ms %.4f lists_ms %.4f\n", n, nt, nlev,
            a.tasks.size() / 4, a.panels.size() / 2, ms(t1 - t0), ms(t2 - t1));
    // the lists
    CHECK((int)a.pbeg.size() == nlev && (int)a.pcnt.size() == nlev && (int)a.tbeg.size() == nlev && (int)a.tcnt.size() == nlev);
    std::vector<int> contrib, tasks;
    int np_seen = 0;
    for (int l = 0; l < nlev; ++l) {
        CHECK(a.pbeg[l] == np_seen);
        std::vector<int> want;
        for (int k = 0; k < nt; ++k)
            if (tp.level[k] == l) {
                if (tp.rows[k].empty()) want.insert(want.end(), {k, -1});
                for (int i : tp.rows[k]) want.insert(want.end(), {k, i});
            }
        CHECK((int)want.size() == 2 * a.pcnt[l] && std::equal(want.begin(), want.end(), a.panels.begin() + 2 * a.pbeg[l]));
        np_seen += a.pcnt[l];
        CHECK(a.tbeg[l] == (int)tasks.size() / 4);
        const std::vector<int> t = tasks_by_enumeration(tp, l, contrib);
        CHECK((int)t.size() == 4 * a.tcnt[l]);
        tasks.insert(tasks.end(), t.begin(), t.end());
    }
    CHECK((int)a.panels.size() == 2 * np_seen);
    CHECK(std::equal(tasks.begin(), tasks.end(), a.tasks.begin(), a.tasks.end()));
    CHECK(std::equal(contrib.begin(), contrib.end(), a.contrib.begin(), a.contrib.end()));
    if (lists_only) return 0;

    // the damped, gauge-fixed system: pattern tiles in a nested-dissection order, everything in the natural one
    const double NaN = std::nan("");
    Mem A{std::vector<double>((size_t)n * n, NaN), {}}, L = A, LT = A, W{std::vector<double>((size_t)nt * NB * NB, NaN), {}};
    Mem x{std::vector<double>(n, NaN), {}};
    const int a0 = 6 * anchor, a1 = a0 + 6;
    std::set<std::pair<int, int>> tiles;
    for (size_t e = 0; e < a.dtiles.size(); e += 2) tiles.insert({a.dtiles[e], a.dtiles[e + 1]});
    for (int R = 0; R < n; ++R)
        for (int C = 0; C < n; ++C) {
            const int o = a.perm[R], oc = a.perm[C];
            double v = (o >= 0 && oc >= 0) ? H[(size_t)o * n0 + oc] : 0.0;
            if (o < 0 || oc < 0 || (o >= a0 && o < a1) || (oc >= a0 && oc < a1)) v = R == C ? 1.0 : 0.0;
            if (R == C) v += lam * v;
            if (tiles.count({R / NB, C / NB})) A.v[(size_t)R * n + C] = v;
            else if (C <= R) CHECK(v == 0.0);
        }
    for (int R = 0; R < n; ++R) x.v[R] = (a.perm[R] < 0 || (a.perm[R] >= a0 && a.perm[R] < a1)) ? 0.0 : -b[a.perm[R]];

    for (int l = 0; l < nlev; ++l) {
        for (int e = 0; e < a.pcnt[l]; ++e) {   // the panel launch: workgroup e
            const int32_t *p = &a.panels[2 * (a.pbeg[l] + e)];
            const int k0 = p[0] * NB, ra = p[1] * NB, nb = std::min(NB, n - k0);
            const bool first = e == 0 || p[-2] != p[0];
            double Lk[NB][NB] = {}, Wk[NB][NB] = {};
            for (int i = 0; i < NB; ++i)
                for (int j = 0; j <= i; ++j) {
                    double s = i < nb ? A.rd((long)(k0 + i) * n + k0 + j) : (i == j);
                    for (int m = 0; m < j; ++m) s -= Lk[i][m] * Lk[j][m];
                    if (i == j) { CHECK(s > 0); Lk[i][i] = std::sqrt(s); } else Lk[i][j] = s / Lk[j][j];
                }
            for (int c = 0; c < NB; ++c)
                for (int i = 0; i < NB; ++i) {
                    double s = i == c;
                    for (int m = 0; m < i; ++m) s -= Lk[i][m] * Wk[m][c];
                    Wk[i][c] = s / Lk[i][i];
                }
            if (first) {
                for (int i = 0; i < NB; ++i)
                    for (int j = 0; j < NB; ++j) W.wr(((long)p[0] * NB + i) * NB + j, i < nb && j < nb ? Wk[i][j] : 0.0);
                for (int i = 0; nd && i < NB; ++i) {
                    double y = 0;
                    for (int j = 0; j <= i; ++j) y += Wk[i][j] * x.rd(k0 + j);
                    x.wr(k0 + i, y);
                }
            }
            if (p[1] < 0) continue;
            CHECK(nb == NB);
            for (int i = 0; i < NB && ra + i < n; ++i)
                for (int j = 0; j < NB; ++j) {
                    double s = 0;
                    for (int m = 0; m <= j; ++m) s += A.rd((long)(ra + i) * n + k0 + m) * Wk[j][m];
                    L.wr((long)(ra + i) * n + k0 + j, s);
                    LT.wr((long)(k0 + j) * n + ra + i, s);
                }
        }
        L.end(); LT.end(); W.end(); x.end();
        for (int t = a.tbeg[l]; t < a.tbeg[l] + a.tcnt[l]; ++t)   // the update launch: four workgroups a task
            for (int q = 0; q < 4; ++q) {
                const int qi = q >> 1, qj = q & 1, ta = a.tasks[4 * t], tb = a.tasks[4 * t + 1];
                const int ri = ta * NB + 32 * qi, rj = tb * NB + 32 * qj;
                const bool diag = ta == tb;
                if ((diag && qj > qi) || ri >= n) continue;
                for (int i = 0; i < 32 && ri + i < n; ++i) {
                    for (int j = 0; j < 32 && rj + j < n; ++j) {
                        if (diag && 32 * qj + j > 32 * qi + i) continue;
                        double s = 0;
                        for (int e = 0; e < a.tasks[4 * t + 3]; ++e) {
                            const int k0 = a.contrib[a.tasks[4 * t + 2] + e] * NB;
                            for (int m = 0; m < NB; ++m) s += L.rd((long)(ri + i) * n + k0 + m) * L.rd((long)(rj + j) * n + k0 + m);
                        }
                        A.wr((long)(ri + i) * n + rj + j, A.rd((long)(ri + i) * n + rj + j) - s);
                    }
                    if (nd && diag && qj == 0) {
                        double z = 0;
                        for (int e = 0; e < a.tasks[4 * t + 3]; ++e) {
                            const int k0 = a.contrib[a.tasks[4 * t + 2] + e] * NB;
                            for (int m = 0; m < NB; ++m) z += L.rd((long)(ri + i) * n + k0 + m) * x.rd(k0 + m);
                        }
                        x.wr(ri + i, x.rd(ri + i) - z);
                    }
                }
            }
        A.end(); x.end();
    }
    // the triangular solves: forward over the block columns (the natural order; the other one's is done), backward
    std::vector<double> &v = x.v;
    auto times_w = [&](int k, bool t) {
        double u[NB] = {};
        const int nb = std::min(NB, n - k * NB);
        for (int i = 0; i < nb; ++i)
            for (int j = 0; j < nb; ++j) u[i] += W.rd(((long)k * NB + (t ? j : i)) * NB + (t ? i : j)) * v[k * NB + j];
        for (int i = 0; i < nb; ++i) v[k * NB + i] = u[i];
    };
    for (int k = 0; !nd && k < nt; ++k) {
        times_w(k, false);
        for (int i : tp.rows[k])
            for (int r = i * NB; r < std::min(n, (i + 1) * NB); ++r)
                for (int j = 0; j < NB; ++j) v[r] -= L.rd((long)r * n + k * NB + j) * v[k * NB + j];
    }
    for (int k = nt - 1; k >= 0; --k) {
        for (int i : tp.rows[k])
            for (int j = 0; j < NB; ++j)
                for (int r = i * NB; r < std::min(n, (i + 1) * NB); ++r) v[k * NB + j] -= LT.rd((long)(k * NB + j) * n + r) * v[r];
        times_w(k, true);
    }
    std::vector<double> out(n0);
    for (int p = 0; p < np; ++p)
        for (int i = 0; i < 6; ++i) out[6 * p + i] = v[pos[p] + i];
    fwrite(out.data(), 8, n0, stdout);
    return 0;
}
