// Host check of how a pass's work is cut into items (ItemCut in engine.hpp), no
// GPU: whatever the cut, every target must meet exactly the sources it met
// before, through the items' own slots and the fold; no item may be empty; and
// an item holds at most the sources the cut allows.  Exits non-zero on a failed
// check.
#include <cstdio>
#include <map>
#include <random>
#include <vector>

#include "../../paper_2012_06925_amd/csrc/engine.hpp"

using namespace bldtt;

namespace {

int failures = 0;

void check(bool ok, const char* what, long long a = 0, long long b = 0) {
    if (!ok) {
        std::fprintf(stderr, "FAILED: %s (%lld, %lld)\n", what, a, b);
        ++failures;
    }
}

int64_t cube3(int d) { return (int64_t)(d + 1) * (d + 1) * (d + 1); }

// Sum over the sources each output meets of the source's weight (its position
// + 1): equal sums for the same sources, and a missing or doubled one shows.
double weight(int64_t pos) { return (double)(pos + 1); }

struct Made {
    std::vector<double> out;        // per particle, or per cluster and proxy
    int64_t items = 0, most = 0;    // items, sources of the largest
};

Made apply(const Tree& T, const std::vector<Item>& items, const std::vector<Entry>& entries, bool proxies, int degree,
           const SymFold& f) {
    Made m;
    const int64_t P = cube3(degree);
    m.out.assign(proxies ? T.size() * P : T.n_particles, 0.0);
    m.items = (int64_t)items.size();
    std::vector<double> slots(f.nslots, 0.0);
    std::vector<int> written(f.nslots, 0);
    for (size_t i = 0; i < items.size(); ++i) {
        const Item& it = items[i];
        int64_t o = f.ibase[i];
        double src = 0.0, tgt = 0.0;
        int64_t n = 0;
        for (int32_t e = it.eb; e < it.ee; ++e) {
            const int64_t c = proxies ? P : (entries[e].b & kCountMask);
            for (int64_t k = 0; k < c; ++k) src += weight(proxies ? entries[e].a * P + k : entries[e].a + k);
            n += c;
        }
        check(n > 0 && it.tn > 0, "empty item", (long long)i, it.tn);
        m.most = std::max(m.most, n);
        for (int32_t r = 0; r < it.tn; ++r) tgt += weight(proxies ? (int64_t)it.cluster * P + it.t0 + r : it.t0 + r);
        for (int32_t r = 0; r < it.tn; ++r, ++o) {
            slots[o] = src;
            written[o]++;
        }
        for (int64_t k = 0; k < n; ++k, ++o) {
            slots[o] = tgt;
            written[o]++;
        }
    }
    for (int64_t k = 0; k < f.nslots; ++k) check(written[k] == 1, "slot written once", k, written[k]);
    for (const FoldSeg& sg : f.segs)
        for (int32_t q = sg.pb; q < sg.pe; ++q)
            for (int32_t k = 0; k < f.parts[q].len; ++k) m.out[sg.off + f.parts[q].lo + k] += slots[f.parts[q].slot + k];
    return m;
}

void run(int64_t n, int64_t leaf, int degree, double theta, bool gauss, bool separate_guarded, int tile, ItemCut cut) {
    std::mt19937_64 rng(n * 31 + leaf);
    std::uniform_real_distribution<double> u(-1.0, 1.0);
    std::normal_distribution<double> g(0.0, 0.25);
    std::vector<double> x[3], s[3];
    for (auto& v : x) {
        v.resize(n);
        for (double& a : v) a = gauss ? g(rng) : u(rng);
    }
    Tree T;
    build_tree(n, x[0].data(), x[1].data(), x[2].data(), leaf, T, s[0], s[1], s[2]);
    Lists L, rest, rest0;
    traverse(T, T, theta, degree, kSchemeDtt, L);
    SymWork whole, parts;
    whole.guard_near = parts.guard_near = separate_guarded;
    split_symmetric(T, L, degree, true, true, rest0, whole, {}, separate_guarded, false, tile);
    split_symmetric(T, L, degree, true, true, rest, parts, {}, separate_guarded, false, tile, cut);
    for (SymWork* w : {&whole, &parts}) fold_parts(T, w->pp_items, w->pp_entries, false, w->pp_fold);
    check(whole.pp_evaluations == parts.pp_evaluations && whole.cc_evaluations == parts.cc_evaluations, "terms");
    for (int k = 0; k < 4; ++k) check(rest.tc[k] == rest0.tc[k] && rest.sc[k] == rest0.sc[k], "rest lists", k);
    const Made a = apply(T, whole.pp_items, whole.pp_entries, false, degree, whole.pp_fold);
    const Made b = apply(T, parts.pp_items, parts.pp_entries, false, degree, parts.pp_fold);
    const Made c = apply(T, whole.cc_items, whole.cc_entries, true, degree, whole.cc_fold);
    const Made d = apply(T, parts.cc_items, parts.cc_entries, true, degree, parts.cc_fold);
    check(a.out == b.out, "particle sums of the cut items");
    check(c.out == d.out, "proxy sums of the cut items");
    for (size_t i = 0; i < parts.pp_items.size(); ++i) {       // guarded ranges stay apart from plain ones
        const Item& it = parts.pp_items[i];
        for (int32_t e = it.eb; e < it.ee && separate_guarded; ++e)
            check(((uint32_t)parts.pp_entries[e].b >> 29 == SRC_RANGE_GUARD) == ((int64_t)i >= parts.pp_plain), "guard", (long long)i);
    }
    std::printf("n %lld leaf %lld: PP %lld -> %lld items (most sources %lld -> %lld), CC %lld -> %lld\n", (long long)n,
                (long long)leaf, (long long)a.items, (long long)b.items, (long long)a.most, (long long)b.most,
                (long long)c.items, (long long)d.items);
    check(b.items >= a.items && d.items >= c.items, "a cut makes items, never fewer", b.items, a.items);
}

// One-way items: what the pieces give every output, the first of an item
// directly and the others through slots and the fold, equals the whole items'.
void run_one_way(int64_t m, int64_t n, int64_t leaf, int degree, double theta, int scheme, ItemCut cut) {
    std::mt19937_64 rng(m * 7 + n);
    std::normal_distribution<double> g(0.0, 0.4);
    std::vector<double> x[3], y[3], sx[3], sy[3];
    for (int d = 0; d < 3; ++d) {
        x[d].resize(m);
        y[d].resize(n);
        for (double& a : x[d]) a = g(rng);
        for (double& a : y[d]) a = g(rng);
    }
    Tree T, S;
    build_tree(m, x[0].data(), x[1].data(), x[2].data(), leaf, T, sx[0], sx[1], sx[2]);
    build_tree(n, y[0].data(), y[1].data(), y[2].data(), leaf, S, sy[0], sy[1], sy[2]);
    Lists L;
    traverse(T, S, theta, degree, scheme, L);
    Work w;
    pack_work(T, S, L, degree, 512, 512, w);
    for (bool proxies : {false, true}) {
        std::vector<Entry>& entries = proxies ? w.qentries : w.pentries;
        const std::vector<Item>& items = proxies ? w.qitems : w.pitems;
        const int64_t P = cube3(degree), nout = proxies ? T.size() * P : m;
        auto sum = [&](const Item& it) {
            double v = 0.0;
            for (int32_t e = it.eb; e < it.ee; ++e) {
                const int64_t low = entries[e].b & kCountMask;
                const bool grid = (uint32_t)entries[e].b >> 29 == SRC_PROXY;
                for (int64_t k = 0; k < (grid ? cube3((int)low) : low); ++k)
                    v += weight(grid ? (1 << 20) + entries[e].a * 1000 + k : entries[e].a + k);
            }
            return v;
        };
        auto at = [&](const Item& it) { return proxies ? it.slot * P + it.t0 : (int64_t)it.slot; };
        std::vector<double> want(nout, 0.0), got(nout, 0.0);
        for (const Item& it : items)
            for (int32_t r = 0; r < it.tn; ++r) want[at(it) + r] = sum(it);
        CutItems c;
        cut_items(items, entries, proxies, cut, c);
        if (c.items.empty()) {
            std::printf("  nothing to cut\n");
            continue;
        }
        check(c.items.size() == c.fold.ibase.size(), "a base per piece");
        std::vector<double> slots(c.fold.nslots, 0.0);
        std::vector<int> direct(nout, 0);
        int64_t empty = 0, whole_empty = 0;
        for (size_t i = 0; i < c.items.size(); ++i) {
            const Item& it = c.items[i];
            empty += it.ee == it.eb;
            for (int32_t r = 0; r < it.tn; ++r) {
                if (c.fold.ibase[i] >= 0) slots[c.fold.ibase[i] + r] = sum(it);
                else {
                    got[at(it) + r] = sum(it);
                    direct[at(it) + r]++;
                }
            }
        }
        for (const Item& it : items) whole_empty += it.ee == it.eb;
        check(empty == whole_empty, "pieces hold sources", empty, whole_empty);
        for (const FoldSeg& sg : c.fold.segs)
            for (int32_t q = sg.pb; q < sg.pe; ++q)
                for (int32_t k = 0; k < c.fold.parts[q].len; ++k)
                    got[sg.off + c.fold.parts[q].lo + k] += slots[c.fold.parts[q].slot + k];
        check(got == want, "one-way sums of the pieces", proxies);
        for (const Item& it : items)
            for (int32_t r = 0; r < it.tn; ++r) check(direct[at(it) + r] == 1, "one piece writes each output", it.slot, r);
        std::printf("one-way m %lld n %lld proxies %d: %zu -> %zu items\n", (long long)m, (long long)n, proxies,
                    items.size(), c.items.size());
    }
}

// PC/CP pairs once for both: with proxy_tiles some become items over proxy tiles
// with particle ranges.  Through their slots and the two folds, every particle
// must meet the same proxies and every proxy the same particles as without, and
// no pair may come twice.
void run_pc(int64_t n, int64_t leaf, int degree, double theta, ItemCut cut) {
    std::mt19937_64 rng(n * 13 + leaf);
    std::normal_distribution<double> g(0.0, 0.25);
    std::vector<double> x[3], s[3];
    for (auto& v : x) {
        v.resize(n);
        for (double& a : v) a = g(rng);
    }
    Tree T;
    build_tree(n, x[0].data(), x[1].data(), x[2].data(), leaf, T, s[0], s[1], s[2]);
    Lists L;
    traverse(T, T, theta, degree, kSchemeDtt, L);
    const int64_t P = cube3(degree);
    std::vector<double> pout[2], cout[2];
    double evals[2];
    int64_t rest[2];
    size_t cp = 0, pc = 0;
    for (int k = 0; k < 2; ++k) {
        Lists r;
        SymWork w;
        cut.proxy_tiles = k == 1;
        split_symmetric(T, L, degree, true, true, r, w, {}, false, true, 256, cut);
        build_pc_folds(T, w);
        rest[k] = (int64_t)(r.tc[PC].size() + r.tc[CP].size());
        evals[k] = w.pc_evaluations;
        if (k == 0) check(w.cp_items.empty() && w.cp_entries.empty(), "no proxy tiles unless asked for");
        cp = w.cp_items.size();
        pc = w.pc_items.size();
        std::vector<double> ps(w.pc_fold.nslots, 0.0), cs(w.cc_fold.nslots, 0.0);
        std::vector<int> pw(ps.size(), 0), cw(cs.size(), 0);
        // the CC items' own slots are not under test: no values, marked as written
        const int64_t c0 = w.pc_items.empty() ? (w.cp_items.empty() ? w.cc_fold.nslots : w.cp_tbase[0]) : w.pc_sbase[0];
        for (int64_t i = 0; i < c0; ++i) cw[i] = 1;
        auto span = [&](int64_t a, int64_t c) {
            double v = 0.0;
            for (int64_t i = 0; i < c; ++i) v += weight(a + i);
            return v;
        };
        auto put = [&](std::vector<double>& sl, std::vector<int>& wr, int64_t o, int64_t c, double v) {
            for (int64_t i = o; i < o + c; ++i) {
                sl[i] = v;
                wr[i]++;
            }
        };
        for (size_t i = 0; i < w.pc_items.size(); ++i) {
            const Item& it = w.pc_items[i];
            double src = 0.0;
            for (int32_t e = it.eb; e < it.ee; ++e) {
                const int64_t b = w.pc_entries[e].a;
                src += span(b * P, P);
                put(cs, cw, w.pc_sbase[i] + (e - it.eb) * P, P, span(it.t0, it.tn));
            }
            put(ps, pw, w.pc_fold.ibase[i], it.tn, src);
        }
        for (size_t i = 0; i < w.cp_items.size(); ++i) {
            const Item& it = w.cp_items[i];
            const double tgt = span(it.cluster * P + it.t0, it.tn);
            double src = 0.0;
            int64_t o = w.cp_sbase[i];
            check(it.ee > it.eb && it.tn > 0 && it.tn <= 256 && it.t0 + it.tn <= P, "proxy tile", (long long)i);
            for (int32_t e = it.eb; e < it.ee; ++e) {
                const int64_t c = w.cp_entries[e].b & kCountMask;
                src += span(w.cp_entries[e].a, c);
                put(ps, pw, o, c, tgt);
                o += c;
            }
            put(cs, cw, w.cp_tbase[i], it.tn, src);
        }
        for (size_t i = 0; i < pw.size(); ++i) check(pw[i] == 1, "particle slot written once", (long long)i, pw[i]);
        for (size_t i = 0; i < cw.size(); ++i) check(cw[i] == 1, "proxy slot written once", (long long)i, cw[i]);
        auto fold = [](const SymFold& f, const std::vector<double>& sl, std::vector<double>& out) {
            for (const FoldSeg& sg : f.segs)
                for (int32_t q = sg.pb; q < sg.pe; ++q)
                    for (int32_t i = 0; i < f.parts[q].len; ++i)
                        out[sg.off + f.parts[q].lo + i] += sl[f.parts[q].slot + i];
        };
        pout[k].assign(n, 0.0);
        cout[k].assign(T.size() * P, 0.0);
        fold(w.pc_fold, ps, pout[k]);
        fold(w.cc_fold, cs, cout[k]);
    }
    check(evals[0] == evals[1] && rest[0] == rest[1], "PC/CP terms");
    check(pout[0] == pout[1], "particle sums of the PC/CP items");
    check(cout[0] == cout[1], "proxy sums of the PC/CP items");
    std::printf("PC/CP n %lld leaf %lld degree %d: %zu particle items, %zu proxy items\n", (long long)n, (long long)leaf,
                degree, pc, cp);
}

// Symmetric items (pairs of particles, of proxies, and both kinds of PC/CP items)
// cut by cost: every target and every source meets what it met before, no piece is
// empty, and a piece costs at most the cap, rounded up to whole rounds and grids.
void run_cut_symmetric(int64_t n, int64_t leaf, int degree, double theta, double cap) {
    std::mt19937_64 rng(n * 17 + leaf);
    std::normal_distribution<double> g(0.0, 0.25);
    std::vector<double> x[3], s[3];
    for (auto& v : x) {
        v.resize(n);
        for (double& a : v) a = g(rng);
    }
    Tree T;
    build_tree(n, x[0].data(), x[1].data(), x[2].data(), leaf, T, s[0], s[1], s[2]);
    Lists L, r;
    traverse(T, T, theta, degree, kSchemeDtt, L);
    SymWork w;
    split_symmetric(T, L, degree, true, true, r, w, {}, false, true, 256, ItemCut{0, 1, true});
    const int64_t P = cube3(degree);
    struct Kind {
        std::vector<Item>* items;
        std::vector<Entry>* entries;
        bool proxy_tgt, proxy_src;
    };
    for (const Kind& k : {Kind{&w.pp_items, &w.pp_entries, false, false}, Kind{&w.cc_items, &w.cc_entries, true, true},
                          Kind{&w.pc_items, &w.pc_entries, false, true}, Kind{&w.cp_items, &w.cp_entries, true, false}}) {
        auto sums = [&] {
            std::vector<double> out[2];            // what particles and proxies meet
            out[0].assign(n, 0.0);
            out[1].assign(T.size() * P, 0.0);
            for (const Item& it : *k.items) {
                const int64_t t0 = k.proxy_tgt ? it.cluster * P + it.t0 : it.t0;
                double tgt = 0.0, src = 0.0;
                for (int64_t i = 0; i < it.tn; ++i) tgt += weight(t0 + i);
                for (int32_t e = it.eb; e < it.ee; ++e) {
                    const Entry& en = (*k.entries)[e];
                    const int64_t c = k.proxy_src ? P : (en.b & kCountMask), a = k.proxy_src ? en.a * P : en.a;
                    for (int64_t i = a; i < a + c; ++i) {
                        src += weight(i);
                        out[k.proxy_src][i] += tgt;
                    }
                }
                for (int64_t i = 0; i < it.tn; ++i) out[k.proxy_tgt][t0 + i] += src;
            }
            return std::make_pair(out[0], out[1]);
        };
        const auto want = sums();
        const size_t before = k.items->size();
        size_t most = 0;
        for (const Item& it : *k.items) most += (size_t)(item_cost(it, *k.entries) / cap) + 1;
        cut_symmetric(*k.items, *k.entries, cap);
        check(sums() == want, "sums of the pieces", k.proxy_tgt, k.proxy_src);
        check(k.items->size() >= before && k.items->size() <= most, "pieces", (long long)k.items->size(), (long long)most);
        for (const Item& it : *k.items) {
            const double lanes = (it.tn + 63) / 64, c = item_cost(it, *k.entries);
            check(it.ee > it.eb, "a piece holds sources");
            check(c <= cap + lanes * (256 + (k.proxy_src ? P : 0)), "cost of a piece", (long long)c, (long long)cap);
        }
        std::printf("cut %d%d n %lld cap %g: %zu -> %zu items\n", k.proxy_tgt, k.proxy_src, (long long)n, cap, before,
                    k.items->size());
    }
}

// pc_slots_bound covers what the PC/CP items take, for every tile.
void run_pc_bound(int64_t n, int64_t leaf, int degree, double theta, ItemCut cut) {
    std::mt19937_64 rng(n * 19 + leaf);
    std::normal_distribution<double> g(0.0, 0.25);
    std::vector<double> x[3], s[3];
    for (auto& v : x) {
        v.resize(n);
        for (double& a : v) a = g(rng);
    }
    Tree T;
    build_tree(n, x[0].data(), x[1].data(), x[2].data(), leaf, T, s[0], s[1], s[2]);
    Lists L;
    traverse(T, T, theta, degree, kSchemeDtt, L);
    for (bool proxy_tiles : {false, true})
        for (int tile : {256, 512, 1024}) {
            Lists r;
            SymWork w;
            cut.proxy_tiles = proxy_tiles;
            split_symmetric(T, L, degree, true, true, r, w, {}, false, true, tile, cut);
            build_pc_folds(T, w);
            std::vector<std::vector<int64_t>> b;
            const int64_t cc = fold_group_bases({{&w.cc_items, &w.cc_entries, FoldGroup::kProxyBoth}}, b);
            const double took = (double)(w.pc_fold.nslots + w.cc_fold.nslots - cc);
            const double bound = pc_slots_bound(T, L, degree, tile, proxy_tiles);
            check(took > 0 && took <= bound, "slots within the bound", (long long)took, (long long)bound);
            std::printf("PC/CP n %lld degree %d tile %d grids %d: %.0f slots, bound %.0f\n", (long long)n, degree, tile,
                        proxy_tiles, took, bound);
        }
}

// A large problem's lists do not stay with the thread, whatever their types (a
// particle-cluster treecode lists PC pairs, a cluster-particle one CP pairs); a
// small one's do.
void run_kept(int scheme, int64_t m, int64_t n, int64_t leaf, double theta, bool symmetric) {
    std::mt19937_64 rng(11);
    std::uniform_real_distribution<double> u(-1.0, 1.0);
    std::vector<double> x[3], y[3], sx[3], sy[3];
    for (int d = 0; d < 3; ++d) {
        x[d].resize(m);
        y[d].resize(n);
        for (double& a : x[d]) a = u(rng);
        for (double& a : y[d]) a = u(rng);
    }
    Tree T, S;
    build_tree(m, x[0].data(), x[1].data(), x[2].data(), leaf, T, sx[0], sx[1], sx[2]);
    build_tree(n, y[0].data(), y[1].data(), y[2].data(), leaf, S, sy[0], sy[1], sy[2]);
    Lists L;
    size_t listed = 0;
    if (symmetric) {
        Lists r;
        SymWork w;
        traverse(T, T, theta, 1, scheme, L);
        split_symmetric(T, L, 1, true, true, r, w, {}, false, true, 256, ItemCut{4096, 256, true});
    } else {
        traverse(T, S, theta, 1, scheme, L);
    }
    for (int k = 0; k < 4; ++k) listed += L.tc[k].size();
    const size_t kept = kept_host_bytes();
    check(kept <= (size_t)256 << 20, "kept lists are bounded", (long long)kept, (long long)listed);
    check(listed < 100000 || listed > 8000000, "sizes of the check", (long long)listed);
    check(listed > 8000000 ? kept < 17 * listed / 2 : kept > 0, "a large problem's lists are given back", (long long)kept, (long long)listed);
    std::printf("kept: %zu pairs listed, %zu bytes\n", listed, kept);
}

}  // namespace

int main() {
    run_kept(kSchemeDtt, 2000, 2000, 100, 0.8, true);
    run_kept(kSchemeBltc, 100000, 100000, 4, 0.6, false);
    run_kept(kSchemeCpBltc, 100000, 100000, 4, 0.6, false);
    run_kept(kSchemeDtt, 60000, 10, 4, 0.4, true);
    run_pc_bound(30000, 300, 6, 0.8, ItemCut{4096, 256});
    run_pc_bound(40000, 700, 8, 0.9, ItemCut{4096, 256});
    run_pc_bound(60000, 1500, 12, 0.9, ItemCut{100, 256});
    run_pc_bound(9000, 70, 5, 0.8, ItemCut{1000000, 1});
    run_cut_symmetric(6000, 100, 5, 0.8, 3000.0);
    run_cut_symmetric(9000, 300, 4, 0.9, 1.0);
    run_cut_symmetric(20000, 70, 3, 0.8, 700.0);
    run_cut_symmetric(30000, 1500, 6, 0.9, 1e9);
    run_pc(4000, 40, 3, 0.8, ItemCut{4096, 256});
    run_pc(6000, 100, 5, 0.8, ItemCut{2048, 256});
    run_pc(9000, 70, 6, 0.8, ItemCut{0, 1});
    run_pc(9000, 300, 8, 0.9, ItemCut{1000000, 1});
    run_pc(30000, 1500, 9, 0.9, ItemCut{4096, 256});
    run_pc(300, 500, 3, 0.7, ItemCut{4096, 256});
    run_one_way(3000, 9000, 200, 3, 0.7, kSchemeDtt, ItemCut{4096, 256});
    run_one_way(700, 20000, 1000, 5, 0.8, kSchemeBltc, ItemCut{4096, 256});
    run_one_way(20000, 700, 300, 4, 0.8, kSchemeCpBltc, ItemCut{4096, 256});
    run_one_way(10, 5000, 60, 2, 0.9, kSchemeDtt, ItemCut{1000000, 1});
    run_one_way(5, 7, 60, 2, 0.9, kSchemeDtt, ItemCut{4096, 256});
    for (bool guarded : {false, true}) {
        run(4000, 60, 2, 0.7, false, guarded, 256, ItemCut{4096, 256});
        run(6000, 700, 3, 0.8, true, guarded, 256, ItemCut{100, 256});
        run(9000, 300, 2, 0.9, false, guarded, 512, ItemCut{1000000, 1});
        run(5000, 2000, 4, 0.8, true, guarded, 1024, ItemCut{64, 512});
        run(300, 500, 3, 0.7, false, guarded, 256, ItemCut{4096, 256});
    }
    if (failures) std::fprintf(stderr, "%d check(s) failed\n", failures);
    return failures != 0;
}
