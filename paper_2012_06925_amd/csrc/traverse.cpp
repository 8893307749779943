// traverse.cpp -- dual tree traversal (Algorithm 2) and packing of the four
// interaction lists into device work items.
//
// MAC (Sec. 2.6): clusters are well separated when (r_t + r_s) / R < theta,
// r = half the box diagonal, R = distance of the box midpoints; R == 0 never
// separates.  Separated pairs interact by CC when both clusters hold more
// than n_p = (n+1)^3 particles, by CP when only the target does, by PC when
// only the source does, and by PP otherwise.  A pair that is not separated
// interacts by PP when both are leaves; otherwise the traversal recurses into
// the children of the target when the source is a leaf, of the source when
// the target is a leaf, and else of the larger cluster by particle count,
// descending into the source on a tie.
//
// The two treecodes the paper compares with build their lists from the same
// MAC.  BLTC (Sec. 2.8): each target leaf (a batch) starts at the source root;
// a separated source cluster interacts by PC when it holds more than n_p
// particles and by PP otherwise, a source leaf that is not separated by PP,
// and any other source cluster passes the batch to its children.  CP-BLTC
// (Sec. 4.5) is the same walk with the roles exchanged: each source leaf
// starts at the target root, and separated target clusters with more than n_p
// particles receive it by CP.
#include <algorithm>
#include <array>
#include <cmath>
#include <numeric>

#include "bldtt.h"
#include "engine.hpp"

namespace bldtt {

int separated_type(int64_t ct, int64_t cs, int d, bool pp_cc_only) {
    const int64_t np = (int64_t)(d + 1) * (d + 1) * (d + 1);
    if (ct > np && cs > np) return CC;
    if (pp_cc_only) return PP;
    if (ct > np) return CP;
    if (cs > np) return PC;
    return PP;
}

namespace {

constexpr int kSeparated = 4;   // step() result: separated pair, type deferred

struct Ctx {
    const Tree& T;
    const Tree& S;
    double theta;
    int degree;
    int scheme;
    bool defer;
};

int scheme_type(const Ctx& x, int64_t ct, int64_t cs) {
    const int64_t np = (int64_t)(x.degree + 1) * (x.degree + 1) * (x.degree + 1);
    switch (x.scheme) {
    case kSchemeBltc: return cs > np ? PC : PP;
    case kSchemeCpBltc: return ct > np ? CP : PP;
    default: return separated_type(ct, cs, x.degree, x.scheme == kSchemePpCc);
    }
}

// One step of Algorithm 2.  Returns the list type for a terminal pair
// (kSeparated when the choice is deferred), or -1 after passing the child
// pairs to push_pair.
template <class Push>
int step(const Ctx& x, int64_t t, int64_t s, Push&& push_pair) {
    const Tree& T = x.T;
    const Tree& S = x.S;
    double dx = T.center[3 * t] - S.center[3 * s];
    double dy = T.center[3 * t + 1] - S.center[3 * s + 1];
    double dz = T.center[3 * t + 2] - S.center[3 * s + 2];
    double R = std::sqrt((dx * dx + dy * dy) + dz * dz);
    bool sep = R > 0.0 && (T.radius[t] + S.radius[s]) / R < x.theta;
    int64_t ct = T.count[t], cs = S.count[s];
    if (sep) return x.defer ? kSeparated : scheme_type(x, ct, cs);
    bool tl = T.is_leaf(t), sl = S.is_leaf(s);
    bool into_target;
    if (x.scheme == kSchemeBltc) {              // the batch t stays; the source side is refined
        if (sl) return PP;
        into_target = false;
    } else if (x.scheme == kSchemeCpBltc) {     // the batch s stays; the target side is refined
        if (tl) return PP;
        into_target = true;
    } else {
        if (tl && sl) return PP;
        into_target = sl ? true : (tl ? false : (cs < ct));
    }
    if (into_target) {
        for (int k = 0; k < T.nchild[t]; ++k) push_pair(T.child[8 * t + k], s);
    } else {
        for (int k = 0; k < S.nchild[s]; ++k) push_pair(t, S.child[8 * s + k]);
    }
    return -1;
}

void record(Lists& out, int ty, int64_t t, int64_t s, int degree) {
    if (ty == kSeparated) {
        out.sep_tc.push_back(t);
        out.sep_sc.push_back(s);
    } else {
        out.push(ty, t, s, degree);
    }
}

void recurse(const Ctx& x, int64_t t, int64_t s, Lists& out) {
    int ty = step(x, t, s, [&](int64_t a, int64_t b) { recurse(x, a, b, out); });
    if (ty >= 0) record(out, ty, t, s, x.degree);
}

}  // namespace

int scheme_of(uint32_t flags) {
    if (flags & BLDTT_BLTC) return kSchemeBltc;
    if (flags & BLDTT_CP_BLTC) return kSchemeCpBltc;
    return (flags & BLDTT_PP_CC_ONLY) ? kSchemePpCc : kSchemeDtt;
}

std::vector<std::pair<int64_t, int64_t>> walk_roots(const Tree& T, const Tree& S, int scheme) {
    std::vector<std::pair<int64_t, int64_t>> roots;
    if (scheme == kSchemeBltc) {                // every target batch from the source root
        for (int64_t b = 0; b < T.size(); ++b)
            if (T.is_leaf(b)) roots.emplace_back(b, 0);
    } else if (scheme == kSchemeCpBltc) {       // every source batch from the target root
        for (int64_t b = 0; b < S.size(); ++b)
            if (S.is_leaf(b)) roots.emplace_back(0, b);
    } else {
        roots.emplace_back(0, 0);
    }
    return roots;
}

void traverse(const Tree& T, const Tree& S, double theta, int degree, int scheme, Lists& out,
              bool defer_separated) {
    traverse_roots(T, S, walk_roots(T, S, scheme), theta, degree, scheme, out, defer_separated);
}

int64_t append_tree(Tree& f, const Tree& t, int64_t pos0, int64_t caller0) {
    const int64_t c0 = f.size(), n = t.size();
    f.lo.insert(f.lo.end(), t.lo.begin(), t.lo.end());
    f.hi.insert(f.hi.end(), t.hi.begin(), t.hi.end());
    f.center.insert(f.center.end(), t.center.begin(), t.center.end());
    f.radius.insert(f.radius.end(), t.radius.begin(), t.radius.end());
    f.level.insert(f.level.end(), t.level.begin(), t.level.end());
    f.nchild.insert(f.nchild.end(), t.nchild.begin(), t.nchild.end());
    for (int64_t c = 0; c < n; ++c) {
        f.begin.push_back(t.begin[c] + pos0);
        f.count.push_back(t.count[c]);
        f.parent.push_back(t.parent[c] < 0 ? -1 : t.parent[c] + c0);
        for (int k = 0; k < 8; ++k) f.child.push_back(t.child[8 * c + k] < 0 ? -1 : t.child[8 * c + k] + c0);
    }
    for (int64_t p = 0; p < t.n_particles; ++p) f.perm.push_back(t.perm[p] + caller0);
    f.n_particles += t.n_particles;
    f.depth = std::max(f.depth, t.depth);
    return c0;
}

namespace {

// What a calling thread keeps between computes, so that a plan repacked every
// compute touches no fresh pages: at most kKeptBytes each for the walk's lists and
// for the packing's (1E7 particles in the cube: 24 and 26 MB).
constexpr size_t kKeptBytes = (size_t)128 << 20;
thread_local std::vector<Lists> kept_walk;

template <class V>
size_t held(const V& v) { return v.capacity() * sizeof(v[0]); }

size_t walk_bytes() {
    size_t n = held(kept_walk);
    for (const Lists& p : kept_walk) {
        for (int k = 0; k < 4; ++k) n += held(p.tc[k]) + held(p.sc[k]) + held(p.deg[k]);
        n += held(p.sep_tc) + held(p.sep_sc);
    }
    return n;
}

}  // namespace

void traverse_roots(const Tree& T, const Tree& S, const std::vector<std::pair<int64_t, int64_t>>& roots,
                    double theta, int degree, int scheme, Lists& out, bool defer_separated) {
    Ctx x{T, S, theta, degree, scheme, defer_separated};
    out.clear();
    // Breadth-first expansion until there is enough independent work, then
    // depth-first recursion on all threads, the frontier in as many runs as keep
    // the threads even.  The runs' lists (kept per calling thread: no fresh pages
    // per compute) are concatenated in frontier order, so the output is
    // deterministic.
    std::vector<std::pair<int64_t, int64_t>> cur(roots), nxt;
    const size_t want = (size_t)16 * num_threads();
    const bool small = T.size() + S.size() < 128;         // some thousand pairs: not worth waking threads
    while (!small && !cur.empty() && cur.size() < want) {
        nxt.clear();
        for (auto& pr : cur) {
            int ty = step(x, pr.first, pr.second, [&](int64_t a, int64_t b) { nxt.emplace_back(a, b); });
            if (ty >= 0) record(out, ty, pr.first, pr.second, degree);
        }
        cur.swap(nxt);
    }
    const int64_t runs = small ? 1 : std::min<int64_t>((int64_t)cur.size(), (int64_t)8 * num_threads());
    std::vector<Lists>& part = kept_walk;
    if ((int64_t)part.size() < runs) part.resize(runs);
    parallel_run(runs, [&](int64_t r) {
        part[r].clear();
        for (int64_t i = (int64_t)cur.size() * r / runs; i < (int64_t)cur.size() * (r + 1) / runs; ++i)
            recurse(x, cur[i].first, cur[i].second, part[r]);
    });
    // list k of run r goes to [at[r][k], at[r][k] + its size); list 4: the deferred pairs
    std::vector<std::array<size_t, 5>> at(runs + 1);
    for (int k = 0; k < 4; ++k) at[0][k] = out.tc[k].size();
    at[0][4] = out.sep_tc.size();
    for (int64_t r = 0; r < runs; ++r) {
        for (int k = 0; k < 4; ++k) at[r + 1][k] = at[r][k] + part[r].tc[k].size();
        at[r + 1][4] = at[r][4] + part[r].sep_tc.size();
    }
    for (int k = 0; k < 4; ++k) {
        out.tc[k].resize(at[runs][k]);
        out.sc[k].resize(at[runs][k]);
        out.deg[k].resize(at[runs][k]);
    }
    out.sep_tc.resize(at[runs][4]);
    out.sep_sc.resize(at[runs][4]);
    parallel_run(runs, [&](int64_t r) {
        const Lists& p = part[r];
        for (int k = 0; k < 4; ++k) {
            std::copy(p.tc[k].begin(), p.tc[k].end(), out.tc[k].begin() + at[r][k]);
            std::copy(p.sc[k].begin(), p.sc[k].end(), out.sc[k].begin() + at[r][k]);
            std::copy(p.deg[k].begin(), p.deg[k].end(), out.deg[k].begin() + at[r][k]);
        }
        std::copy(p.sep_tc.begin(), p.sep_tc.end(), out.sep_tc.begin() + at[r][4]);
        std::copy(p.sep_sc.begin(), p.sep_sc.end(), out.sep_sc.begin() + at[r][4]);
    });
    if (walk_bytes() > kKeptBytes) std::vector<Lists>().swap(part);      // a large problem's lists are not kept
}

namespace {

// CSR of the entries of some types, grouped by target cluster in list order.
struct ByTarget {
    std::vector<int64_t> off;      // n_clusters + 1
    std::vector<int64_t> sc;       // source cluster
    std::vector<int8_t> type, deg;
};

// Parallel counting sort over the concatenated lists t0..t1: chunk k counts
// its entries per cluster, and its entries land after those of chunks < k, so
// the order within a cluster is the list order.
ByTarget group(const Tree& T, const Lists& L, int t0, int t1, int degree) {
    ByTarget g;
    const int64_t nc = T.size();
    std::vector<int64_t> base{0};
    for (int ty = t0; ty <= t1; ++ty) base.push_back(base.back() + (int64_t)L.tc[ty].size());
    const int64_t E = base.back();
    auto at = [&](int64_t i, int& ty, int64_t& e) {
        ty = t0;
        while (i >= base[ty - t0 + 1]) ++ty;
        e = i - base[ty - t0];
    };
    const int64_t nch = std::max<int64_t>(1, std::min<int64_t>(4 * num_threads(), E / 4096 + 1));
    const int64_t per = (E + nch - 1) / nch;
    std::vector<int64_t> cnt(nch * nc, 0);
    parallel_run(nch, [&](int64_t k) {
        int64_t* c = cnt.data() + k * nc;
        for (int64_t i = k * per; i < std::min(E, (k + 1) * per); ++i) {
            int ty;
            int64_t e;
            at(i, ty, e);
            c[L.tc[ty][e]]++;
        }
    });
    g.off.assign(nc + 1, 0);
    for (int64_t c = 0; c < nc; ++c) {
        int64_t run = g.off[c];
        for (int64_t k = 0; k < nch; ++k) {
            int64_t n = cnt[k * nc + c];
            cnt[k * nc + c] = run;             // start of chunk k's entries of cluster c
            run += n;
        }
        g.off[c + 1] = run;
    }
    g.sc.resize(E);
    g.type.resize(E);
    g.deg.resize(E);
    parallel_run(nch, [&](int64_t k) {
        int64_t* fill = cnt.data() + k * nc;
        for (int64_t i = k * per; i < std::min(E, (k + 1) * per); ++i) {
            int ty;
            int64_t e;
            at(i, ty, e);
            int64_t to = fill[L.tc[ty][e]]++;
            g.sc[to] = L.sc[ty][e];
            g.type[to] = (int8_t)ty;
            g.deg[to] = L.deg[ty].empty() ? (int8_t)degree : L.deg[ty][e];
        }
    });
    return g;
}

// Guarded particle ranges.  FP64 needs the guard only where the boxes touch
// (the two sets may share a point: r^2 == 0).  The FP32 forms also guard near
// ranges (range_guarded): the boxes touch, or their gap g is small against the distance R from t's box centre
// to the farthest corner of either box, g^2 <= 2^-23 R^2.  Pairs of unguarded
// ranges then lie farther apart than 2^-11.5 R, so in coordinates relative to
// that centre r^2 > 2^-24 (|x|^2 + |y|^2): the FP64 expansion |x|^2 - 2 x.y +
// |y|^2 of the FP32 matrix-core passes keeps a relative error below 2^-25 there.
bool boxes_touch(const Tree& T, int64_t t, const Tree& S, int64_t s) {
    for (int d = 0; d < 3; ++d)
        if (T.hi[3 * t + d] < S.lo[3 * s + d] || S.hi[3 * s + d] < T.lo[3 * t + d]) return false;
    return true;
}

bool range_guarded(const Tree& T, int64_t t, const Tree& S, int64_t s) {
    double g2 = 0.0, R2 = 0.0;
    for (int d = 0; d < 3; ++d) {
        const double tlo = T.lo[3 * t + d], thi = T.hi[3 * t + d], slo = S.lo[3 * s + d], shi = S.hi[3 * s + d];
        const double gap = std::max({slo - thi, tlo - shi, 0.0});
        const double c = 0.5 * (tlo + thi);
        const double far = std::max({c - tlo, thi - c, std::fabs(slo - c), std::fabs(shi - c)});
        g2 += gap * gap;
        R2 += far * far;
    }
    return g2 <= 0x1p-23 * R2;
}

// Particle ranges of one work group: sort by start and merge neighbours that
// touch and share the guard flag.  Summation order is free (any order of the
// same terms is a valid evaluation of the sum).
void emit_ranges(std::vector<std::pair<int64_t, int64_t>>& rng_plain, std::vector<std::pair<int64_t, int64_t>>& rng_guard,
                 std::vector<Entry>& out) {
    for (int g = 0; g < 2; ++g) {
        auto& v = g ? rng_guard : rng_plain;
        std::sort(v.begin(), v.end());
        size_t i = 0;
        while (i < v.size()) {
            int64_t b = v[i].first, e = v[i].first + v[i].second;
            size_t j = i + 1;
            while (j < v.size() && v[j].first == e && e - b + v[j].second <= kCountMask) {
                e += v[j].second;
                ++j;
            }
            out.push_back(Entry{(int32_t)b, (int32_t)((uint32_t)(g ? SRC_RANGE_GUARD : SRC_RANGE) << 29 | (uint32_t)(e - b))});
            i = j;
        }
        v.clear();
    }
}

inline int64_t cube(int d) { return (int64_t)(d + 1) * (d + 1) * (d + 1); }

inline Entry proxy_entry(int64_t sc, int d) {
    return Entry{(int32_t)sc, (int32_t)((uint32_t)SRC_PROXY << 29 | (uint32_t)d)};
}

// Output of one block of target clusters, concatenated in block order.
struct Block {
    std::vector<Entry> entries;
    std::vector<std::pair<double, Item>> items;      // eb, ee relative to this block's entries
    std::vector<Item> prolong;
};

void append_blocks(std::vector<Block>& blocks, std::vector<Entry>& entries, std::vector<std::pair<double, Item>>& items,
                   std::vector<Item>* prolong) {
    size_t ne = 0, ni = 0;
    for (auto& b : blocks) {
        ne += b.entries.size();
        ni += b.items.size();
    }
    entries.reserve(ne);
    items.reserve(ni);
    for (auto& b : blocks) {
        const int32_t shift = (int32_t)entries.size();
        entries.insert(entries.end(), b.entries.begin(), b.entries.end());
        for (auto& it : b.items) {
            it.second.eb += shift;
            it.second.ee += shift;
            items.push_back(it);
        }
        if (prolong) prolong->insert(prolong->end(), b.prolong.begin(), b.prolong.end());
        b = Block();
    }
}

void sort_items(const std::vector<std::pair<double, Item>>& items, std::vector<Item>& out) {
    // Longest items first: the tail of the grid is then made of short items.
    // A stable counting sort on the cost's exponent and top three mantissa
    // bits (eighth-octave classes, descending): linear time, and the order
    // among items of one class is their input order.
    constexpr int kClasses = 2048;
    auto code = [](double c) { return c > 0.0 ? (int64_t)(__builtin_bit_cast(uint64_t, c) >> 49) : (int64_t)0; };
    int64_t top = 0;
    for (auto& it : items) top = std::max(top, code(it.first));
    auto cls = [&](double c) { return (int)std::min<int64_t>(kClasses - 1, top - code(c)); };
    std::vector<int64_t> start(kClasses + 1, 0);
    for (auto& it : items) start[cls(it.first) + 1]++;
    for (int k = 0; k < kClasses; ++k) start[k + 1] += start[k];
    const size_t o = out.size();
    out.resize(o + items.size());
    for (auto& it : items) out[o + start[cls(it.first)]++] = it.second;
}

}  // namespace

void Work::clear() {
    pentries.clear();
    pitems.clear();
    qentries.clear();
    qitems.clear();
    leaf_has_far.clear();
    prolong.clear();
    src_degrees = tgt_degrees = 0;
    down_degree = 0;
    for (double& v : interactions) v = 0.0;
}

void pack_work(const Tree& T, const Tree& S, const Lists& L, int degree, int tile, int ptile, Work& w,
               const std::vector<uint32_t>* extra) {
    w.clear();
    auto deg_of = [&](int ty, size_t e) { return L.deg[ty].empty() ? degree : (int)L.deg[ty][e]; };
    for (int ty = 0; ty < 4; ++ty) {
        const int64_t n = (int64_t)L.tc[ty].size();
        const int64_t nch = std::max<int64_t>(1, std::min<int64_t>(4 * num_threads(), n / 4096 + 1));
        const int64_t per = (n + nch - 1) / nch;
        std::vector<double> acc(nch, 0.0);
        std::vector<uint32_t> sd(nch, 0), td(nch, 0);
        parallel_run(nch, [&](int64_t k) {
            double a = 0.0;
            uint32_t s = 0, t = 0;
            for (int64_t e = k * per; e < std::min(n, (k + 1) * per); ++e) {
                const int d = deg_of(ty, e);
                double np = (double)cube(d);
                double ct = ty == PP || ty == PC ? (double)T.count[L.tc[ty][e]] : np;
                double cs = ty == PP || ty == CP ? (double)S.count[L.sc[ty][e]] : np;
                a += ct * cs;                        // integers below 2^53: exact in any order
                if (ty == PC || ty == CC) s |= 1u << d;
                if (ty == CP || ty == CC) t |= 1u << d;
            }
            acc[k] = a;
            sd[k] = s;
            td[k] = t;
        });
        for (int64_t k = 0; k < nch; ++k) {
            w.interactions[ty] += acc[k];
            w.src_degrees |= sd[k];
            w.tgt_degrees |= td[k];
        }
    }
    if (extra)
        for (uint32_t m : *extra) {
            w.src_degrees |= m;
            w.tgt_degrees |= m;
        }
    // Downward degree: the largest degree of any proxy potential (lower degrees
    // are lifted to it exactly), or the base degree when there are none.
    w.down_degree = degree;
    for (int d = kMaxDegree; d >= 0; --d)
        if (w.tgt_degrees >> d & 1) {
            w.down_degree = d;
            break;
        }

    ByTarget part = group(T, L, PP, PC, degree);
    ByTarget prox = group(T, L, CP, CC, degree);
    const int64_t nc = T.size();
    constexpr int64_t kBlockClusters = 64;
    const int64_t nblk = (nc + kBlockClusters - 1) / kBlockClusters;

    // Particle targets: per target leaf, the PP/PC entries of the leaf and of
    // every ancestor (each leaf owns its targets, so no two items share an output).
    w.leaf_has_far.assign(nc, 0);
    std::vector<Block> blocks(nblk);
    parallel_run(nblk, [&](int64_t bi) {
        Block& B = blocks[bi];
        std::vector<std::pair<int64_t, int64_t>> rp, rg;
        for (int64_t leaf = bi * kBlockClusters; leaf < std::min(nc, (bi + 1) * kBlockClusters); ++leaf) {
            if (!T.is_leaf(leaf)) continue;
            int64_t eb = (int64_t)B.entries.size();
            double src = 0.0;
            bool far = false;
            for (int64_t c = leaf; c >= 0; c = T.parent[c]) {
                if (prox.off[c + 1] > prox.off[c] || (extra && (*extra)[c])) far = true;
                for (int64_t e = part.off[c]; e < part.off[c + 1]; ++e) {
                    int64_t sc = part.sc[e];
                    if (part.type[e] == PC) {
                        B.entries.push_back(proxy_entry(sc, part.deg[e]));
                        src += (double)cube(part.deg[e]);
                    } else {
                        ((w.guard_near ? range_guarded(T, leaf, S, sc) : boxes_touch(T, leaf, S, sc)) ? rg : rp)
                            .emplace_back(S.begin[sc], S.count[sc]);
                        src += (double)S.count[sc];
                    }
                }
            }
            emit_ranges(rp, rg, B.entries);
            w.leaf_has_far[leaf] = far;
            int64_t ee = (int64_t)B.entries.size();
            for (int64_t tb = T.begin[leaf]; tb < T.begin[leaf] + T.count[leaf]; tb += tile) {
                int64_t tn = std::min<int64_t>(tile, T.begin[leaf] + T.count[leaf] - tb);
                B.items.push_back({src * (double)tn, Item{(int32_t)tb, (int32_t)tn, (int32_t)eb, (int32_t)ee,
                                                          (int32_t)leaf, (int32_t)w.down_degree, (int32_t)tb}});
            }
        }
    });
    std::vector<std::pair<double, Item>> items;
    append_blocks(blocks, w.pentries, items, nullptr);
    sort_items(items, w.pitems);

    // Proxy targets: per (target cluster, degree) with CP/CC entries, tiles of its proxies.
    items.clear();
    blocks.assign(nblk, Block());
    const int down = w.down_degree;
    parallel_run(nblk, [&](int64_t bi) {
        Block& B = blocks[bi];
        std::vector<std::pair<int64_t, int64_t>> rp, rg;
        for (int64_t c = bi * kBlockClusters; c < std::min(nc, (bi + 1) * kBlockClusters); ++c) {
            const uint32_t more = extra ? (*extra)[c] : 0u;
            if (prox.off[c + 1] == prox.off[c] && !more) continue;
            uint32_t used = 0;
            for (int64_t e = prox.off[c]; e < prox.off[c + 1]; ++e) used |= 1u << prox.deg[e];
            for (int d = 0; d <= kMaxDegree; ++d) {
                if (!(used >> d & 1)) continue;
                int64_t eb = (int64_t)B.entries.size();
                double src = 0.0;
                for (int64_t e = prox.off[c]; e < prox.off[c + 1]; ++e) {
                    if (prox.deg[e] != d) continue;
                    int64_t sc = prox.sc[e];
                    if (prox.type[e] == CC) {
                        B.entries.push_back(proxy_entry(sc, d));
                        src += (double)cube(d);
                    } else {
                        rp.emplace_back(S.begin[sc], S.count[sc]);     // separated: never r = 0
                        src += (double)S.count[sc];
                    }
                }
                emit_ranges(rp, rg, B.entries);
                int64_t ee = (int64_t)B.entries.size();
                const int64_t np = cube(d);
                for (int64_t lb = 0; lb < np; lb += ptile) {
                    int64_t ln = std::min<int64_t>(ptile, np - lb);
                    B.items.push_back({src * (double)ln, Item{(int32_t)lb, (int32_t)ln, (int32_t)eb, (int32_t)ee,
                                                              (int32_t)c, (int32_t)d, (int32_t)c}});
                }
            }
            // degrees of this cluster's proxy potentials that are lifted to the downward degree
            uint32_t lift = (used | more) & ~(1u << down);
            if (lift) B.prolong.push_back(Item{0, 0, 0, 0, (int32_t)c, (int32_t)lift, (int32_t)c});
        }
    });
    append_blocks(blocks, w.qentries, items, &w.prolong);
    sort_items(items, w.qitems);
}

namespace {

int64_t entry_sources(const Entry& e) {
    const int low = e.b & kCountMask;
    return (uint32_t)e.b >> 29 == SRC_PROXY ? cube(low) : (int64_t)low;
}

}  // namespace

double item_cost(const Item& it, const std::vector<Entry>& entries) {
    int64_t n = 0;
    for (int32_t e = it.eb; e < it.ee; ++e) n += entry_sources(entries[e]);
    return (double)n * (double)((it.tn + 63) / 64);
}

void cut_items(const std::vector<Item>& items, std::vector<Entry>& entries, bool proxies, const ItemCut& cut,
               CutItems& out) {
    out.clear();
    // lanes of an item: its targets in whole waves
    auto lanes_of = [](const Item& it) { return (int64_t)(it.tn + 63) / 64 * 64; };
    std::vector<int64_t> src(items.size(), 0);
    double total = 0.0;
    for (size_t i = 0; i < items.size(); ++i) {
        for (int32_t e = items[i].eb; e < items[i].ee; ++e) src[i] += entry_sources(entries[e]);
        total += (double)src[i] * (double)lanes_of(items[i]);
    }
    const double cap = std::max(1.0, total / (double)std::max<int64_t>(1, cut.want));
    std::vector<std::pair<double, Item>> cost;
    std::vector<int64_t> base;                            // slot base per item of `cost`, -1: the outputs
    bool any = false;
    cost.reserve(items.size());
    for (size_t i = 0; i < items.size(); ++i) {
        const Item& it = items[i];
        const int64_t lanes = lanes_of(it);
        const int64_t chunk = std::max((int64_t)std::min(cap / (double)lanes, 1e15), cut.min_src);
        // no cut for less than half a chunk more than one
        if (2 * src[i] < 3 * chunk) {
            cost.push_back({(double)src[i] * (double)lanes, it});
            base.push_back(-1);
            continue;
        }
        any = true;
        const int64_t pieces = (src[i] + chunk - 1) / chunk;
        const int64_t each = ((src[i] + pieces - 1) / pieces + 255) / 256 * 256;   // whole rounds of the matrix-core pass
        FoldSeg sg;
        sg.off = proxies ? (int64_t)it.slot * cube(it.degree) + it.t0 : (int64_t)it.slot;
        sg.n = it.tn;
        sg.deg = proxies ? it.degree : -1;
        sg.pb = (int32_t)out.fold.parts.size();
        int32_t at = (int32_t)entries.size();
        int64_t have = 0;
        bool first = true;
        auto close = [&] {
            Item piece = it;
            piece.eb = at;
            piece.ee = at = (int32_t)entries.size();
            cost.push_back({(double)have * (double)lanes, piece});
            if (first) {
                base.push_back(-1);
                first = false;
            } else {
                base.push_back(out.fold.nslots);
                out.fold.parts.push_back(FoldPart{out.fold.nslots, 0, it.tn});
                out.fold.nslots += it.tn;
            }
            have = 0;
        };
        for (int32_t e = it.eb; e < it.ee; ++e) {
            const Entry en = entries[e];                   // by value: entries grows below
            if ((uint32_t)en.b >> 29 == SRC_PROXY) {       // a grid stays whole
                entries.push_back(en);
                have += entry_sources(en);
                if (have >= each) close();
                continue;
            }
            const uint32_t kind = (uint32_t)en.b & ~(uint32_t)kCountMask;
            for (int64_t a = en.a, n = en.b & kCountMask; n > 0;) {
                const int64_t m = std::min(n, each - have);
                entries.push_back(Entry{(int32_t)a, (int32_t)(kind | (uint32_t)m)});
                a += m;
                n -= m;
                have += m;
                if (have >= each) close();
            }
        }
        if (have > 0) close();
        sg.pe = (int32_t)out.fold.parts.size();
        if (sg.pe > sg.pb) out.fold.segs.push_back(sg);
    }
    if (!any) return;
    // longest first; the slot bases follow their items
    std::vector<size_t> order(cost.size());
    std::iota(order.begin(), order.end(), (size_t)0);
    std::stable_sort(order.begin(), order.end(), [&](size_t x, size_t y) { return cost[x].first > cost[y].first; });
    out.items.reserve(order.size());
    out.fold.ibase.reserve(order.size());
    for (size_t k : order) {
        out.items.push_back(cost[k].second);
        out.fold.ibase.push_back(base[k]);
    }
}

void cut_symmetric(std::vector<Item>& items, std::vector<Entry>& entries, double cap) {
    bool any = false;
    for (const Item& it : items) any = any || item_cost(it, entries) > cap;
    if (!any) return;
    std::vector<std::pair<double, Item>> cost;
    cost.reserve(items.size());
    for (const Item& it : items) {
        const double c = item_cost(it, entries), lanes = (double)((it.tn + 63) / 64);
        // pieces of equal size, in whole rounds of the symmetric kernels (a grid stays whole)
        const int64_t pieces = c > cap ? (int64_t)std::ceil(c / cap) : 1;
        const int64_t each = ((int64_t)(c / lanes) / pieces + 256) / 256 * 256;
        if (pieces == 1 || (double)each * lanes >= c) {
            cost.push_back({c, it});
            continue;
        }
        Item piece = it;
        piece.eb = (int32_t)entries.size();
        int64_t have = 0;
        auto close = [&] {
            piece.ee = (int32_t)entries.size();
            cost.push_back({(double)have * lanes, piece});
            piece.eb = piece.ee;
            have = 0;
        };
        for (int32_t e = it.eb; e < it.ee; ++e) {
            const Entry en = entries[e];                   // by value: entries grows below
            if ((uint32_t)en.b >> 29 == SRC_PROXY) {
                entries.push_back(en);
                have += entry_sources(en);
                if (have >= each) close();
                continue;
            }
            const uint32_t kind = (uint32_t)en.b & ~(uint32_t)kCountMask;
            for (int64_t a = en.a, n = en.b & kCountMask; n > 0;) {
                const int64_t m = std::min(n, each - have);
                entries.push_back(Entry{(int32_t)a, (int32_t)(kind | (uint32_t)m)});
                a += m;
                n -= m;
                have += m;
                if (have >= each) close();
            }
        }
        if (have > 0) close();
    }
    items.clear();
    sort_items(cost, items);
}

namespace {

// Pairs of one type as CSR by target cluster: partners sorted by (source
// cluster, degree) per target, only pairs accepted by `take`, each with its
// list position and a flag, set by mirror(), that its mirror is listed too.
struct PairIndex {
    struct Rec {
        int64_t key;                 // source cluster << 4 | degree
        int64_t e;                   // position in the list
        bool operator<(const Rec& o) const { return key < o.key; }
        int64_t sc() const { return key >> 4; }
        int deg() const { return (int)(key & 15); }
    };
    std::vector<int64_t> off, cnt;
    int64_t kBlk = 32;               // clusters per task
    std::vector<Rec> part;
    std::vector<uint8_t> both;       // per Rec
    template <class F>
    void build(int64_t nc, const std::vector<int64_t>& tc, const std::vector<int64_t>& sc, const std::vector<int8_t>& dg,
               int degree, F take) {
        // counting sort by target with per-chunk counts (see group); the order
        // within a target is fixed by the sort below
        const int64_t n = (int64_t)tc.size();
        kBlk = n < 4096 ? std::max<int64_t>(1, nc) : 32;
        const int64_t nch = std::max<int64_t>(1, std::min<int64_t>(4 * num_threads(), n / 4096 + 1));
        const int64_t per = (n + nch - 1) / nch;
        cnt.assign(nch * nc, 0);
        parallel_run(nch, [&](int64_t k) {
            int64_t* c = cnt.data() + k * nc;
            for (int64_t e = k * per; e < std::min(n, (k + 1) * per); ++e)
                if (take(tc[e], sc[e])) c[tc[e]]++;
        });
        off.assign(nc + 1, 0);
        for (int64_t c = 0; c < nc; ++c) {
            int64_t run = off[c];
            for (int64_t k = 0; k < nch; ++k) {
                const int64_t m = cnt[k * nc + c];
                cnt[k * nc + c] = run;
                run += m;
            }
            off[c + 1] = run;
        }
        part.resize(off[nc]);
        both.assign(off[nc], 0);
        parallel_run(nch, [&](int64_t k) {
            int64_t* fill = cnt.data() + k * nc;
            for (int64_t e = k * per; e < std::min(n, (k + 1) * per); ++e)
                if (take(tc[e], sc[e])) part[fill[tc[e]]++] = Rec{sc[e] << 4 | (dg.empty() ? degree : (int)dg[e]), e};
        });
        parallel_run((nc + kBlk - 1) / kBlk, [&](int64_t b) {
            for (int64_t c = b * kBlk; c < std::min(nc, (b + 1) * kBlk); ++c)
                std::sort(part.begin() + off[c], part.begin() + off[c + 1]);
        });
    }
    // Flags every pair (a, b, d) here with (b, a, d) in `other`, on both sides, and
    // clears their entries of `keep` (this list's) and `other_keep`.  One search per
    // pair, by the smaller cluster when the two indexes are the same one: no two
    // threads write one flag.
    void mirror(PairIndex& other, std::vector<uint8_t>& keep, std::vector<uint8_t>& other_keep) {
        const int64_t nc = (int64_t)off.size() - 1;
        const bool same = &other == this;
        parallel_run((nc + kBlk - 1) / kBlk, [&](int64_t blk) {
            for (int64_t a = blk * kBlk; a < std::min(nc, (blk + 1) * kBlk); ++a)
                for (int64_t k = off[a]; k < off[a + 1]; ++k) {
                    const int64_t b = part[k].sc();
                    if (same && b <= a) continue;
                    const Rec want{a << 4 | part[k].deg(), 0};
                    const auto end = other.part.begin() + other.off[b + 1];
                    const auto it = std::lower_bound(other.part.begin() + other.off[b], end, want);
                    if (it == end || it->key != want.key) continue;
                    both[k] = 1;
                    other.both[it - other.part.begin()] = 1;
                    keep[part[k].e] = 0;
                    other_keep[it->e] = 0;
                }
        });
    }
};

struct SymBlock {
    std::vector<Entry> entries;
    std::vector<std::pair<double, Item>> items, gitems;    // items without / with guarded ranges
    double evals = 0.0;
    void clear() {
        entries.clear();
        items.clear();
        gitems.clear();
        evals = 0.0;
    }
};

// The particle-range entries [at, end) of E cut at every multiple of `chunk`
// sources (the order of the sources stays); first[c] is the entry chunk c
// starts with, first.back() the end.
void chunk_ranges(std::vector<Entry>& E, int64_t at, int64_t chunk, std::vector<int32_t>& first) {
    static thread_local std::vector<Entry> in;
    in.assign(E.begin() + at, E.end());
    E.resize(at);
    first.assign(1, (int32_t)at);
    int64_t have = 0;                                      // sources in the open chunk
    for (const Entry& e : in) {
        const uint32_t kind = (uint32_t)e.b & ~(uint32_t)kCountMask;
        for (int64_t a = e.a, n = e.b & kCountMask; n > 0;) {
            if (have == chunk) {
                first.push_back((int32_t)E.size());
                have = 0;
            }
            const int64_t m = std::min(n, chunk - have);
            E.push_back(Entry{(int32_t)a, (int32_t)(kind | (uint32_t)m)});
            a += m;
            n -= m;
            have += m;
        }
    }
    first.push_back((int32_t)E.size());
}

// Sources per chunk of items with up to `targets` targets that cost at most
// about `cap` each, in whole rounds: the symmetric kernels stage 64, 128 or 256
// sources at a time.
int64_t chunk_sources(int64_t targets, double cap, int64_t min_src) {
    const double by_cost = std::min(cap / (double)targets, 1e15);
    return (std::max((int64_t)by_cost, min_src) + 255) / 256 * 256;
}

// The share of its lanes' time that a tile's targets use: whole tiles of 256 at four
// per lane, and a tail at two per lane (128 lanes' worth, a tenth slower) or one
// (64, half as fast: a source read per pair).
double lane_use(int64_t n) {
    const int64_t tail = n % 256;
    const double lanes = (double)(n - tail) + (tail == 0 ? 0.0 : (tail <= 64 ? 100.0 : (tail <= 128 ? 140.0 : 256.0)));
    return (double)n / lanes;
}

// A PC/CP pair of a cluster of `count` particles is tiled over the proxy grid of
// degree d (in tiles of kGridTile) where that fills the lanes better.
constexpr int64_t kGridTile = 256;
bool tiles_the_grid(int64_t count, int d) { return lane_use(count) < lane_use(cube(d)); }

// What split_symmetric keeps per calling thread (see kKeptBytes).
struct KeptPack {
    PairIndex ipp, icc, ipc, icp;
    std::vector<uint8_t> keep[4];
    std::vector<SymBlock> blks[2];
    std::vector<std::pair<double, Item>> items, gitems;
    size_t bytes() const {
        size_t n = held(items) + held(gitems);
        for (const PairIndex* x : {&ipp, &icc, &ipc, &icp}) n += held(x->off) + held(x->cnt) + held(x->part) + held(x->both);
        for (const auto& k : keep) n += held(k);
        for (const auto& v : blks) {
            n += held(v);
            for (const SymBlock& b : v) n += held(b.entries) + held(b.items) + held(b.gitems);
        }
        return n;
    }
};
thread_local KeptPack kept_pack;

// The blocks' entries concatenated; their items sorted longest first, those
// without guarded ranges ahead of those with (n_plain of them).
void gather(std::vector<SymBlock>& blks, std::vector<Entry>& entries, std::vector<Item>& out, double& evals,
            int64_t* n_plain = nullptr) {
    auto &items = kept_pack.items, &gitems = kept_pack.gitems;
    items.clear();
    gitems.clear();
    for (auto& B : blks) {
        const int32_t shift = (int32_t)entries.size();
        entries.insert(entries.end(), B.entries.begin(), B.entries.end());
        for (auto* v : {&B.items, &B.gitems})
            for (auto& it : *v) {
                it.second.eb += shift;
                it.second.ee += shift;
                (v == &B.items ? items : gitems).push_back(it);
            }
        evals += B.evals;
    }
    sort_items(items, out);
    if (n_plain) *n_plain = (int64_t)out.size();
    sort_items(gitems, out);
}

}  // namespace

std::vector<uint32_t> sym_cc_degrees(const Tree& T, const SymWork& sw) {
    std::vector<uint32_t> m(T.size(), 0u);
    for (const Item& it : sw.cc_items) m[it.cluster] |= 1u << it.degree;
    for (const Entry& e : sw.cc_entries) m[e.a] |= 1u << (e.b & kCountMask);
    for (const Entry& e : sw.pc_entries) m[e.a] |= 1u << (e.b & kCountMask);
    for (const Item& it : sw.cp_items) m[it.cluster] |= 1u << it.degree;
    return m;
}

void split_symmetric(const Tree& T, const Lists& L, int degree, bool pp, bool cc, Lists& rest, SymWork& sw,
                     const std::function<void()>& pp_ready, bool separate_guarded, bool pc, int tile,
                     const ItemCut& cut) {
    sw.clear();
    const int64_t nc = T.size();
    // small problems stay on this thread: their regions cost more than they do
    size_t listed = 0;
    for (int k = 0; k < 4; ++k) listed += L.tc[k].size();
    const int64_t kBlk = listed < 4096 ? std::max<int64_t>(1, nc) : 32;
    const int64_t kTile = tile;
    const int64_t nblk = (nc + kBlk - 1) / kBlk;
    // the workers reach the caller's copies through these references
    PairIndex &ipp = kept_pack.ipp, &icc = kept_pack.icc, &ipc = kept_pack.ipc, &icp = kept_pack.icp;
    std::vector<uint8_t>* keep = kept_pack.keep; // per entry: not one of a pair evaluated once for both
    struct Trim {
        ~Trim() {
            if (kept_pack.bytes() > kKeptBytes) kept_pack = KeptPack();
        }
    } trim;
    for (int k = 0; k < 4; ++k) keep[k].assign(L.tc[k].size(), 1);
    const std::vector<int8_t> no_degrees;        // PP pairs are matched without their degree
    if (pp) {
        ipp.build(nc, L.tc[PP], L.sc[PP], no_degrees, 0,
                  [&](int64_t a, int64_t b) { return a != b && T.is_leaf(a) && T.is_leaf(b); });
        ipp.mirror(ipp, keep[PP], keep[PP]);
    }
    // the indexes of CC, PC and CP pairs are formed after pp_ready, below
    // the blocks of one list type at a time, kept like the indexes
    std::vector<SymBlock>* all_blks = kept_pack.blks;
    auto blocks = [&](int which = 0) -> std::vector<SymBlock>& {
        std::vector<SymBlock>& v = all_blks[which];
        if ((int64_t)v.size() > 4 * nblk + 1024) v.clear();      // a much larger problem's
        v.resize(nblk);
        for (SymBlock& b : v) b.clear();
        return v;
    };
    // the most one item may cost, from the symmetric pairs' kernel values
    auto cost_cap = [&](const std::vector<int64_t>& tc, const std::vector<int64_t>& sc, auto&& values) {
        if (cut.want <= 0) return 1e300;
        const int64_t n = (int64_t)tc.size();
        const int64_t nch = std::max<int64_t>(1, std::min<int64_t>(4 * num_threads(), n / 4096 + 1));
        const int64_t per = (n + nch - 1) / nch;
        std::vector<double> part(nch, 0.0);
        parallel_run(nch, [&](int64_t k) {
            for (int64_t e = k * per; e < std::min(n, (k + 1) * per); ++e) part[k] += values(e, tc[e], sc[e]);
        });
        double v = 0.0;
        for (double x : part) v += x;
        return std::max(1.0, v / (double)cut.want);
    };
    if (pp) {
        const double cap = cost_cap(L.tc[PP], L.sc[PP], [&](int64_t, int64_t a, int64_t b) {
            return a != b && T.is_leaf(a) && T.is_leaf(b) ? 0.5 * (double)T.count[a] * (double)T.count[b] : 0.0;
        });
        // per leaf A: the partners B > A as merged particle ranges, tiles of A's particles
        std::vector<SymBlock>& blks = blocks();
        parallel_run(nblk, [&](int64_t bi) {
            SymBlock& B = blks[bi];
            std::vector<std::pair<int64_t, int64_t>> rp, rg, none;
            std::vector<int32_t> first, gfirst;
            for (int64_t a = bi * kBlk; a < std::min(nc, (bi + 1) * kBlk); ++a) {
                if (!T.is_leaf(a)) continue;
                double src = 0.0;
                for (int64_t k = ipp.off[a]; k < ipp.off[a + 1]; ++k) {
                    const int64_t b = ipp.part[k].sc();
                    if (b > a && ipp.both[k]) {
                        ((sw.guard_near ? range_guarded(T, a, T, b) : boxes_touch(T, a, T, b)) ? rg : rp)
                            .emplace_back(T.begin[b], T.count[b]);
                        src += (double)T.count[b];
                    }
                }
                if (rp.empty() && rg.empty()) continue;
                double src_g = 0.0;
                for (auto& r : rg) src_g += (double)r.second;
                // the ranges, plain then guarded, cut into the chunks of a full tile
                const int64_t full = std::min(kTile, T.count[a]);
                const double src_all = separate_guarded ? src - src_g : src;
                const int64_t eb = (int64_t)B.entries.size();
                emit_ranges(rp, none, B.entries);
                if (!separate_guarded) emit_ranges(none, rg, B.entries);
                const int64_t chunk = chunk_sources(full, cap, cut.min_src);
                if ((int64_t)src_all > chunk) chunk_ranges(B.entries, eb, chunk, first);
                else first = {(int32_t)eb, (int32_t)B.entries.size()};
                const int64_t em = (int64_t)B.entries.size();
                if (separate_guarded) {
                    emit_ranges(none, rg, B.entries);
                    if ((int64_t)src_g > chunk) chunk_ranges(B.entries, em, chunk, gfirst);
                    else gfirst = {(int32_t)em, (int32_t)B.entries.size()};
                }
                B.evals += 2.0 * (double)T.count[a] * src;
                // items of one tile over the chunks first[0..]: a tile of few
                // targets (whole waves of 64) takes several chunks, half as many
                // as would make it cost what a full one does (its rounds of 256
                // sources wait longer for their loads than they compute)
                auto put = [&](std::vector<std::pair<double, Item>>& items, const std::vector<int32_t>& at, double sources,
                               int64_t tb, int64_t tn) {
                    const int64_t nch = (int64_t)at.size() - 1;
                    const int64_t g = std::max<int64_t>(1, std::min(nch, full / (2 * ((tn + 63) / 64 * 64))));
                    for (int64_t c = 0; c < nch; c += g) {
                        const int64_t d = std::min(nch, c + g);
                        if (at[d] == at[c]) continue;
                        items.push_back({sources * (double)tn * (double)(d - c) / (double)nch,
                                         Item{(int32_t)tb, (int32_t)tn, at[c], at[d], (int32_t)a, 0, (int32_t)tb}});
                    }
                };
                // tiles of A's particles: items over every range, or over the
                // plain ranges and over the guarded ranges apart
                for (int64_t tb = T.begin[a]; tb < T.begin[a] + T.count[a]; tb += kTile) {
                    const int64_t tn = std::min<int64_t>(kTile, T.begin[a] + T.count[a] - tb);
                    put(B.items, first, src_all, tb, tn);
                    if (separate_guarded) put(B.gitems, gfirst, src_g, tb, tn);
                }
            }
        });
        gather(blks, sw.pp_entries, sw.pp_items, sw.pp_evaluations, &sw.pp_plain);
        fold_bases(sw.pp_items, sw.pp_entries, false, sw.pp_fold);
    }
    if (pp_ready) pp_ready();
    if (cc) {
        icc.build(nc, L.tc[CC], L.sc[CC], L.deg[CC], degree, [](int64_t a, int64_t b) { return a != b; });
        icc.mirror(icc, keep[CC], keep[CC]);
    }
    if (pc) {
        // PC (a, b) listed with its mirror CP (b, a) at the same degree
        auto all = [](int64_t, int64_t) { return true; };
        ipc.build(nc, L.tc[PC], L.sc[PC], L.deg[PC], degree, all);        // particles of a <- proxies of b
        icp.build(nc, L.tc[CP], L.sc[CP], L.deg[CP], degree, all);        // proxies of a <- particles of b
        ipc.mirror(icp, keep[PC], keep[CP]);
    }
    // the rest: every entry except both directions of the symmetric pairs,
    // in list order (per-chunk compaction on all threads)
    for (int k = 0; k < 4; ++k) {
        const bool typed = !L.deg[k].empty();
        const int64_t n = (int64_t)L.tc[k].size();
        const bool filter = (k == PP && pp) || (k == CC && cc) || ((k == PC || k == CP) && pc);
        if (!filter) {
            rest.tc[k] = L.tc[k];
            rest.sc[k] = L.sc[k];
            rest.deg[k] = L.deg[k];
            continue;
        }
        const uint8_t* kp = keep[k].data();
        const int64_t nch = std::max<int64_t>(1, std::min<int64_t>(4 * num_threads(), n / 4096 + 1));
        const int64_t per = (n + nch - 1) / nch;
        std::vector<int64_t> kept(nch + 1, 0);
        parallel_run(nch, [&](int64_t c) {
            int64_t m = 0;
            for (int64_t e = c * per; e < std::min(n, (c + 1) * per); ++e) m += kp[e];
            kept[c + 1] = m;
        });
        for (int64_t c = 0; c < nch; ++c) kept[c + 1] += kept[c];
        rest.tc[k].resize(kept[nch]);
        rest.sc[k].resize(kept[nch]);
        rest.deg[k].resize(typed ? kept[nch] : 0);
        parallel_run(nch, [&](int64_t c) {
            int64_t o = kept[c];
            for (int64_t e = c * per; e < std::min(n, (c + 1) * per); ++e) {
                if (!kp[e]) continue;
                rest.tc[k][o] = L.tc[k][e];
                rest.sc[k][o] = L.sc[k][e];
                if (typed) rest.deg[k][o] = L.deg[k][e];
                ++o;
            }
        });
    }
    rest.sep_tc.clear();
    rest.sep_sc.clear();
    if (cc) {
        const double cap = cost_cap(L.tc[CC], L.sc[CC], [&](int64_t e, int64_t a, int64_t b) {
            const double np = (double)cube(L.deg[CC].empty() ? degree : (int)L.deg[CC][e]);
            return a != b ? 0.5 * np * np : 0.0;
        });
        // per (cluster A, degree d): the partners B > A at d, tiles of A's
        // proxies, as many partners per item as the cap allows
        std::vector<SymBlock>& blks = blocks();
        parallel_run(nblk, [&](int64_t bi) {
            SymBlock& B = blks[bi];
            for (int64_t a = bi * kBlk; a < std::min(nc, (bi + 1) * kBlk); ++a) {
                uint32_t used = 0;
                for (int64_t q = icc.off[a]; q < icc.off[a + 1]; ++q) used |= icc.both[q] ? 1u << icc.part[q].deg() : 0u;
                for (int d = 0; d <= kMaxDegree; ++d) {
                    if (!(used >> d & 1)) continue;
                    const int64_t eb = (int64_t)B.entries.size();
                    for (int64_t q = icc.off[a]; q < icc.off[a + 1]; ++q) {
                        const int64_t b = icc.part[q].sc();
                        if (icc.part[q].deg() == d && b > a && icc.both[q])
                            B.entries.push_back(Entry{(int32_t)b, (int32_t)((uint32_t)SRC_PROXY << 29 | (uint32_t)d)});
                    }
                    const int64_t ee = (int64_t)B.entries.size();
                    if (ee == eb) continue;
                    const int64_t np = (int64_t)(d + 1) * (d + 1) * (d + 1);
                    B.evals += 2.0 * (double)np * (double)np * (double)(ee - eb);
                    for (int64_t lb = 0; lb < np; lb += kTile) {
                        const int64_t ln = std::min<int64_t>(kTile, np - lb);
                        const int64_t n = std::max<int64_t>(1, std::min<int64_t>(
                            ee - eb, (int64_t)std::ceil(std::min((double)(np * (ee - eb) * ln) / cap, 1e9))));
                        for (int64_t c = 0; c < n; ++c) {
                            const int64_t e0 = eb + (ee - eb) * c / n, e1 = eb + (ee - eb) * (c + 1) / n;
                            B.items.push_back({(double)np * (double)(e1 - e0) * (double)ln,
                                               Item{(int32_t)lb, (int32_t)ln, (int32_t)e0, (int32_t)e1, (int32_t)a,
                                                    (int32_t)d, (int32_t)a}});
                        }
                    }
                }
            }
        });
        gather(blks, sw.cc_entries, sw.cc_items, sw.cc_evaluations);
        if (!pc) build_fold(T, sw.cc_items, sw.cc_entries, true, sw.cc_fold);
    }
    if (pc) {
        const double cap = cost_cap(L.tc[PC], L.sc[PC], [&](int64_t e, int64_t a, int64_t) {
            return (double)T.count[a] * (double)cube(L.deg[PC].empty() ? degree : (int)L.deg[PC][e]);
        });
        auto by_proxies = [&](int64_t a, int d) { return cut.proxy_tiles && tiles_the_grid(T.count[a], d); };
        // per (cluster A, degree d): the partners B whose PC and CP pairs with A
        // are both listed at d, as proxy entries; tiles of A's particles.  Then
        // per (cluster B, degree d) the partners A of the other pairs, as merged
        // particle ranges cut into chunks; tiles of B's proxies.
        std::vector<SymBlock>&blks = blocks(), &cblks = blocks(1);
        parallel_run(nblk, [&](int64_t bi) {
            SymBlock& B = blks[bi];
            for (int64_t a = bi * kBlk; a < std::min(nc, (bi + 1) * kBlk); ++a) {
                uint32_t used = 0;
                for (int64_t q = ipc.off[a]; q < ipc.off[a + 1]; ++q) used |= ipc.both[q] ? 1u << ipc.part[q].deg() : 0u;
                for (int d = 0; d <= kMaxDegree; ++d) {
                    if (!(used >> d & 1) || by_proxies(a, d)) continue;
                    const int64_t eb = (int64_t)B.entries.size();
                    for (int64_t q = ipc.off[a]; q < ipc.off[a + 1]; ++q) {
                        const int64_t b = ipc.part[q].sc();
                        if (ipc.part[q].deg() == d && ipc.both[q])
                            B.entries.push_back(Entry{(int32_t)b, (int32_t)((uint32_t)SRC_PROXY << 29 | (uint32_t)d)});
                    }
                    const int64_t ee = (int64_t)B.entries.size();
                    if (ee == eb) continue;
                    const double np = (double)cube(d) * (double)(ee - eb);
                    B.evals += 2.0 * (double)T.count[a] * np;
                    for (int64_t tb = T.begin[a]; tb < T.begin[a] + T.count[a]; tb += kTile) {
                        const int64_t tn = std::min<int64_t>(kTile, T.begin[a] + T.count[a] - tb);
                        const int64_t n = std::max<int64_t>(
                            1, std::min<int64_t>(ee - eb, (int64_t)std::ceil(std::min(np * (double)tn / cap, 1e9))));
                        for (int64_t c = 0; c < n; ++c) {
                            const int64_t e0 = eb + (ee - eb) * c / n, e1 = eb + (ee - eb) * (c + 1) / n;
                            B.items.push_back({(double)cube(d) * (double)(e1 - e0) * (double)tn,
                                               Item{(int32_t)tb, (int32_t)tn, (int32_t)e0, (int32_t)e1, (int32_t)a,
                                                    (int32_t)d, (int32_t)tb}});
                        }
                    }
                }
            }
            if (!cut.proxy_tiles) return;
            SymBlock& C = cblks[bi];
            std::vector<std::pair<int64_t, int64_t>> rp, none;
            std::vector<int32_t> first;
            for (int64_t b = bi * kBlk; b < std::min(nc, (bi + 1) * kBlk); ++b) {
                uint32_t used = 0;
                for (int64_t q = icp.off[b]; q < icp.off[b + 1]; ++q) used |= icp.both[q] ? 1u << icp.part[q].deg() : 0u;
                for (int d = 0; d <= kMaxDegree; ++d) {
                    if (!(used >> d & 1)) continue;
                    int64_t src = 0;
                    for (int64_t q = icp.off[b]; q < icp.off[b + 1]; ++q) {
                        const int64_t a = icp.part[q].sc();
                        if (icp.part[q].deg() != d || !icp.both[q] || !by_proxies(a, d)) continue;
                        rp.emplace_back(T.begin[a], T.count[a]);       // separated: never r = 0
                        src += T.count[a];
                    }
                    if (rp.empty()) continue;
                    const int64_t eb = (int64_t)C.entries.size(), np = cube(d);
                    emit_ranges(rp, none, C.entries);
                    const int64_t chunk = chunk_sources(std::min(kGridTile, np), cap, std::max<int64_t>(1, cut.min_src));
                    if (src > chunk) chunk_ranges(C.entries, eb, chunk, first);
                    else first = {(int32_t)eb, (int32_t)C.entries.size()};
                    C.evals += 2.0 * (double)np * (double)src;
                    for (int64_t lb = 0; lb < np; lb += kGridTile) {
                        const int64_t ln = std::min(kGridTile, np - lb);
                        for (size_t c = 0; c + 1 < first.size(); ++c)
                            C.items.push_back({(double)ln * (double)std::min(chunk, src - (int64_t)c * chunk),
                                               Item{(int32_t)lb, (int32_t)ln, first[c], first[c + 1], (int32_t)b,
                                                    (int32_t)d, (int32_t)b}});
                    }
                }
            }
        });
        gather(blks, sw.pc_entries, sw.pc_items, sw.pc_evaluations);
        if (cut.proxy_tiles) gather(cblks, sw.cp_entries, sw.cp_items, sw.pc_evaluations);
    }
}

void build_fold(const Tree& T, const std::vector<Item>& items, const std::vector<Entry>& entries, bool proxies,
                SymFold& f) {
    fold_bases(items, entries, proxies, f);
    fold_parts(T, items, entries, proxies, f);
}

namespace {

// Slots of one item of a fold group: its targets, its sources, or both.
int64_t group_item_slots(const FoldGroup& g, const Item& it) {
    int64_t n = 0;
    if (g.kind != FoldGroup::kProxySources && g.kind != FoldGroup::kParticleSources) n += it.tn;
    if (g.kind == FoldGroup::kParticleTargets || g.kind == FoldGroup::kProxyTargets) return n;
    if (g.kind == FoldGroup::kProxyBoth || g.kind == FoldGroup::kProxySources)
        return n + cube(it.degree) * (int64_t)(it.ee - it.eb);
    for (int32_t e = it.eb; e < it.ee; ++e) n += (int64_t)((*g.entries)[e].b & kCountMask);
    return n;
}

}  // namespace

int64_t fold_group_bases(const std::vector<FoldGroup>& groups, std::vector<std::vector<int64_t>>& bases) {
    bases.assign(groups.size(), {});
    int64_t slots = 0;
    for (size_t g = 0; g < groups.size(); ++g) {
        const std::vector<Item>& items = *groups[g].items;
        bases[g].resize(items.size());
        for (size_t i = 0; i < items.size(); ++i) {
            bases[g][i] = slots;
            slots += group_item_slots(groups[g], items[i]);
        }
    }
    return slots;
}

void fold_group_parts(const Tree& T, bool proxies, const std::vector<FoldGroup>& groups,
                      const std::vector<std::vector<int64_t>>& bases, SymFold& f) {
    f.segs.clear();
    f.parts.clear();
    const int64_t nc = T.size();
    constexpr int D = kMaxDegree + 1;
    // segments: every leaf in cluster order (particles), or every (cluster,
    // degree) an item or an entry names, by degree then cluster (proxies)
    std::vector<int32_t> seg_of;
    std::vector<int64_t> leaf_begin, leaf_id;
    if (!proxies) {
        seg_of.assign(nc, -1);
        for (int64_t c = 0; c < nc; ++c)
            if (T.is_leaf(c)) {
                seg_of[c] = (int32_t)f.segs.size();
                f.segs.push_back(FoldSeg{T.begin[c], (int32_t)T.count[c], -1, 0, 0});
                leaf_begin.push_back(T.begin[c]);
                leaf_id.push_back(c);
            }
    } else {
        std::vector<uint8_t> used(nc * D, 0);
        for (const FoldGroup& g : groups)
            for (const Item& it : *g.items) {
                if (g.kind == FoldGroup::kProxyBoth || g.kind == FoldGroup::kProxyTargets)
                    used[it.degree * nc + it.cluster] = 1;
                for (int32_t e = it.eb; e < it.ee && g.kind != FoldGroup::kProxyTargets; ++e) used[it.degree * nc + (*g.entries)[e].a] = 1;
            }
        seg_of.assign(nc * D, -1);
        for (int d = 0; d < D; ++d)
            for (int64_t c = 0; c < nc; ++c)
                if (used[d * nc + c]) {
                    seg_of[d * nc + c] = (int32_t)f.segs.size();
                    f.segs.push_back(FoldSeg{c * cube(d), (int32_t)cube(d), d, 0, 0});
                }
    }
    auto leaf_at = [&](int64_t pos) {
        return (size_t)(std::upper_bound(leaf_begin.begin(), leaf_begin.end(), pos) - leaf_begin.begin()) - 1;
    };
    // parts of a particle range [a, a + len) whose slots start at o, split at leaf boundaries
    auto range_parts = [&](int64_t a, int64_t len, int64_t o, auto&& put) {
        size_t k = leaf_at(a);
        for (int64_t pos = a; pos < a + len; ++k) {
            const int64_t L = leaf_id[k];
            const int64_t end = std::min(a + len, T.begin[L] + T.count[L]);
            put(seg_of[L], FoldPart{o + (pos - a), (int32_t)(pos - T.begin[L]), (int32_t)(end - pos)});
            pos = end;
        }
    };
    // the items of all groups one after another; one item's parts in order:
    // its target tile, then its sources entry by entry
    std::vector<int64_t> first(groups.size() + 1, 0);
    for (size_t g = 0; g < groups.size(); ++g) first[g + 1] = first[g] + (int64_t)groups[g].items->size();
    const int64_t ni = first[groups.size()];
    auto emit = [&](int64_t vi, auto&& put) {
        const size_t g = (size_t)(std::upper_bound(first.begin(), first.end(), vi) - first.begin()) - 1;
        const FoldGroup& G = groups[g];
        const Item& it = (*G.items)[vi - first[g]];
        const std::vector<Entry>& entries = *G.entries;
        int64_t o = bases[g][vi - first[g]];
        switch (G.kind) {
        case FoldGroup::kProxyBoth:
        case FoldGroup::kProxySources: {
            const int64_t P = cube(it.degree);
            if (G.kind == FoldGroup::kProxyBoth) {
                put(seg_of[it.degree * nc + it.cluster], FoldPart{o, it.t0, it.tn});
                o += it.tn;
            }
            for (int32_t e = it.eb; e < it.ee; ++e, o += P)
                put(seg_of[it.degree * nc + entries[e].a], FoldPart{o, 0, (int32_t)P});
            return;
        }
        case FoldGroup::kParticleTargets:
            range_parts(it.t0, it.tn, o, put);
            return;
        case FoldGroup::kProxyTargets:
            put(seg_of[it.degree * nc + it.cluster], FoldPart{o, it.t0, it.tn});
            return;
        default:
            if (G.kind == FoldGroup::kParticleBoth) {
                put(seg_of[it.cluster], FoldPart{o, (int32_t)(it.t0 - T.begin[it.cluster]), it.tn});
                o += it.tn;
            }
            for (int32_t e = it.eb; e < it.ee; ++e) {
                const int64_t len = entries[e].b & kCountMask;
                range_parts(entries[e].a, len, o, put);
                o += len;
            }
        }
    };
    // parts grouped by segment, chunks of items in order (a parallel counting
    // sort: chunk k's parts of a segment follow those of chunks < k)
    const int64_t ns = (int64_t)f.segs.size();
    int64_t work = ni;
    for (const FoldGroup& g : groups) work += (int64_t)g.entries->size();
    const int64_t nch = std::max<int64_t>(1, std::min<int64_t>(num_threads(), work / 512 + 1));
    const int64_t per = (ni + nch - 1) / nch;
    std::vector<int32_t> cnt(nch * ns, 0);
    parallel_run(nch, [&](int64_t k) {
        int32_t* c = cnt.data() + k * ns;
        for (int64_t i = k * per; i < std::min(ni, (k + 1) * per); ++i) emit(i, [&](int32_t sg, const FoldPart&) { c[sg]++; });
    });
    int32_t run = 0;
    for (int64_t sg = 0; sg < ns; ++sg) {
        f.segs[sg].pb = run;
        for (int64_t k = 0; k < nch; ++k) {
            const int32_t n = cnt[k * ns + sg];
            cnt[k * ns + sg] = run;
            run += n;
        }
        f.segs[sg].pe = run;
    }
    f.parts.resize(run);
    parallel_run(nch, [&](int64_t k) {
        int32_t* fill = cnt.data() + k * ns;
        for (int64_t i = k * per; i < std::min(ni, (k + 1) * per); ++i)
            emit(i, [&](int32_t sg, const FoldPart& pt) { f.parts[fill[sg]++] = pt; });
    });
}

void build_pc_folds(const Tree& T, SymWork& sw) {
    std::vector<std::vector<int64_t>> pb, cb;
    const std::vector<FoldGroup> pg{{&sw.pc_items, &sw.pc_entries, FoldGroup::kParticleTargets},
                                    {&sw.cp_items, &sw.cp_entries, FoldGroup::kParticleSources}};
    const std::vector<FoldGroup> cg{{&sw.cc_items, &sw.cc_entries, FoldGroup::kProxyBoth},
                                    {&sw.pc_items, &sw.pc_entries, FoldGroup::kProxySources},
                                    {&sw.cp_items, &sw.cp_entries, FoldGroup::kProxyTargets}};
    sw.pc_fold.clear();
    sw.cc_fold.clear();
    sw.pc_fold.nslots = fold_group_bases(pg, pb);
    sw.cc_fold.nslots = fold_group_bases(cg, cb);
    fold_group_parts(T, false, pg, pb, sw.pc_fold);
    fold_group_parts(T, true, cg, cb, sw.cc_fold);
    sw.pc_fold.ibase = std::move(pb[0]);
    sw.cp_sbase = std::move(pb[1]);
    sw.cc_fold.ibase = std::move(cb[0]);
    sw.pc_sbase = std::move(cb[1]);
    sw.cp_tbase = std::move(cb[2]);
}

double pc_slots_bound(const Tree& T, const Lists& L, int degree, int tile, bool proxy_tiles) {
    // pairs tiled over the grid: their particles per (grid, degree), whose chunks of at
    // least 256 each take the grid's target slots
    std::vector<int64_t> by_grid(proxy_tiles ? T.size() * (kMaxDegree + 1) : 0, 0);
    double n = 0.0;
    for (size_t e = 0; e < L.tc[PC].size(); ++e) {
        const int d = L.deg[PC].empty() ? degree : (int)L.deg[PC][e];
        const int64_t P = cube(d), c = T.count[L.tc[PC][e]];
        if (proxy_tiles && tiles_the_grid(c, d)) {
            n += (double)(c * ((P + kGridTile - 1) / kGridTile));
            by_grid[L.sc[PC][e] * (kMaxDegree + 1) + d] += c;
        } else {
            n += (double)(P * ((c + tile - 1) / tile) + c);
        }
    }
    for (size_t k = 0; k < by_grid.size(); ++k)
        n += (double)(cube((int)(k % (kMaxDegree + 1))) * ((by_grid[k] + 255) / 256));
    return n;
}

size_t kept_host_bytes() { return walk_bytes() + kept_pack.bytes(); }

void fold_bases(const std::vector<Item>& items, const std::vector<Entry>& entries, bool proxies, SymFold& f) {
    f.clear();
    std::vector<std::vector<int64_t>> bases;
    const FoldGroup g{&items, &entries, proxies ? FoldGroup::kProxyBoth : FoldGroup::kParticleBoth};
    f.nslots = fold_group_bases({g}, bases);
    f.ibase = std::move(bases[0]);
}

void fold_parts(const Tree& T, const std::vector<Item>& items, const std::vector<Entry>& entries, bool proxies,
                SymFold& f) {
    const FoldGroup g{&items, &entries, proxies ? FoldGroup::kProxyBoth : FoldGroup::kParticleBoth};
    fold_group_parts(T, proxies, {g}, {f.ibase}, f);
}

}  // namespace bldtt
