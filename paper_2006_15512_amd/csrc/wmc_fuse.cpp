// The fused program of a plan: runs of consecutive contractions
//   F_i[.] = sum_{kappa_i} F_{i-1} * G_i      (i = 1 .. L)
// along a tree path, each taking the previous one's output as its larger
// operand, become one chain whose intermediates F_1 .. F_{L-1} stay in LDS
// (wmc_chain.h).  A node-by-node launch list writes every intermediate to
// memory and reads it back, and pays one launch per tree level.

// Pricing a chain counts bits throughout; every host that takes this card has
// the instruction.
#pragma GCC target("popcnt")
#include <algorithm>
#include <cmath>
#include <cstring>
#include <map>
#include <numeric>

#include "wmc_internal.h"

namespace {

// Cost of a launch's work, used only to choose between fused and separate
// contractions: seconds per launch, bytes/s of the streaming kernels, and
// products/s of the register-tiled ones.
const double kLaunch = 5e-6, kBytes = 4.6e12, kProducts = 4e12;
// A workgroup's tile of a chain of many tiles, fitted to measured launches
// with a third on top, so that a chain is taken only where it clearly saves:
// its fixed part, each stage, each round of outputs of a stage; workgroups
// running at once.  Then a short chain's tile, and products/s of it.
const double kTile = 1.3e-6, kStage = 0.5e-6, kRound = 0.8e-6, kRunning = 768;
const double kTileProducts = 12e9;
const double kShortTile = 3e-6, kShortStage = 0.4e-6;

// A vector of bounded length without allocations: planning prices hundreds
// of chains even for a small formula.
template <typename X, int N>
struct Few {
    X v[N];
    int n = 0;
    void push_back(X x) { v[n++] = x; }
    void clear() { n = 0; }
    size_t size() const { return (size_t)n; }
    bool empty() const { return n == 0; }
    X &operator[](size_t i) { return v[i]; }
    const X &operator[](size_t i) const { return v[i]; }
    const X &back() const { return v[n - 1]; }
    const X &front() const { return v[0]; }
    const X *begin() const { return v; }
    const X *end() const { return v + n; }
};

// The variables around one chain, as bits of 64-bit masks.
struct Chain {
    Few<int32_t, WMC_CHAIN_MAX> nodes, gs;
    int32_t f = -1;
    Few<int32_t, 64> local;                          // local id -> variable
    uint64_t vf = 0;
    Few<uint64_t, WMC_CHAIN_MAX> vc, vg, kap;        // per stage
    uint64_t inner = 0, outer = 0;
    Few<int, WMC_CHAIN_MAX> ebits;                   // per stage: log2 of the tile's outputs
    // LDS entries: the outputs of odd and of even stages, the copies of F_0
    // (-1: read from memory) and of the G_i, and all of them (place_lds)
    int odd = 0, even = 0, fcopy = -1, lds = 0;
    int gcopy[WMC_CHAIN_MAX] = {};
    double bytes = 0, products = 0;
    bool big = false;                          // many tiles: runs alone, register-tiled
};

int bits(uint64_t m) { return __builtin_popcountll(m); }
// 2^n, 0 <= n < 1024
double power(int n) {
    const uint64_t u = (uint64_t)(n + 1023) << 52;
    double x;
    std::memcpy(&x, &u, sizeof x);
    return x;
}

// A chain with more products, or more tiles, runs alone (wmc_chain.h).
const double kShort = 1048576.0;

struct Fuser {
    wmc_plan_t &P;
    const std::vector<TNode> &T;
    const int elem;
    double slices = 1, level = kLaunch;
    double total = 0;  // seconds of the plan's bytes at the streaming rate
    std::vector<int32_t> nk;       // summed variables per internal tensor
    std::vector<int32_t> id_of;    // variable -> local id while a chain is built
    std::vector<int32_t> stamp;
    int32_t now = 0;

    explicit Fuser(wmc_plan_t &p) : P(p), T(p.T), elem(p.elem) {
        nk.assign(T.size(), 0);
        double bytes = 0;
        for (const NodeDesc &d : P.nodes) {
            nk[(size_t)d.tc] = d.nk;
            bytes += (double)elem * (std::ldexp(1.0, rank(d.ta)) + std::ldexp(1.0, rank(d.tb)) + std::ldexp(1.0, d.rc));
        }
        slices = (double)P.group;
        total = slices * bytes / kBytes;
        if (total > 1e-3) level = 1e-6;
        id_of.assign((size_t)P.n + 1, -1);
        stamp.assign((size_t)P.n + 1, 0);
    }

    int rank(int32_t t) const { return (int)T[(size_t)t].layout.size(); }
    int32_t big(int32_t c) const {
        const TNode &C = T[(size_t)c];
        return rank(C.a) >= rank(C.b) ? C.a : C.b;
    }
    int32_t other(int32_t c, int32_t x) const { return T[(size_t)c].a == x ? T[(size_t)c].b : T[(size_t)c].a; }
    bool fits(int32_t c) const {
        return T[(size_t)c].cls != WMC_CLASS_GEMM && nk[(size_t)c] <= WMC_CHAIN_NK && rank(c) <= 31 &&
               rank(T[(size_t)c].a) <= 31 && rank(T[(size_t)c].b) <= 31;
    }

    // Local ids of a tensor's variables; false past 64 variables.
    bool mask_of(Chain &h, int32_t t, uint64_t *m) {
        *m = 0;
        for (int32_t v : T[(size_t)t].layout) {
            if (stamp[(size_t)v] != now) {
                if (h.local.size() >= 64) return false;
                stamp[(size_t)v] = now;
                id_of[(size_t)v] = (int32_t)h.local.size();
                h.local.push_back(v);
            }
            *m |= 1ull << id_of[(size_t)v];
        }
        return true;
    }

    bool begin(Chain &h, int32_t c) {
        ++now;
        h.f = big(c);
        return mask_of(h, h.f, &h.vf) && extend(h, c);
    }

    bool extend(Chain &h, int32_t c) {
        const int32_t prev = h.nodes.empty() ? h.f : h.nodes.back();
        const uint64_t vp = h.nodes.empty() ? h.vf : h.vc.back();
        uint64_t vc = 0, vg = 0;
        const int32_t g = other(c, prev);
        if (!mask_of(h, g, &vg) || !mask_of(h, c, &vc)) return false;
        h.nodes.push_back(c);
        h.gs.push_back(g);
        h.vc.push_back(vc);
        h.vg.push_back(vg);
        h.kap.push_back((vp | vg) & ~vc);
        return true;
    }

    // LDS entries of the chain with the given inner variables (copy_f,
    // copy_g: with copies of F_0 and of the G_i) by region, and whether they
    // fit.  F_0's copy shares the even stages' region, which stage 2 is the
    // first to write.
    bool lds_fits(const Chain &h, uint64_t inner, bool copy_f, bool copy_g, int *odd_even = nullptr) const {
        const size_t L = h.nodes.size();
        int odd = 0, even = 0;
        long long total = 0;
        for (size_t i = 0; i < L; ++i) {
            const int eb = bits(inner & h.vc[i]);
            if (eb > WMC_CHAIN_BITS) return false;
            if (i + 1 < L) (i % 2 ? even : odd) = std::max(i % 2 ? even : odd, 1 << eb);
            if (!copy_g) continue;
            const int gb = bits(h.vg[i] & (inner | h.kap[i]));
            if (gb > WMC_CHAIN_BITS) return false;
            total += 1 << gb;
        }
        if (copy_f) {
            const int fb = bits(h.vf & (inner | h.kap[0]));
            if (fb > WMC_CHAIN_BITS) return false;
            even = std::max(even, 1 << fb);
        }
        total += odd + even;
        // the words of a short chain are read from LDS, too
        const long long words =
            CH_WORDS + (long long)L * CS_WORDS + (long long)(L + 2) * WMC_CHAIN_TILE_BITS + (long long)(L + 1) * WMC_CHAIN_BITS;
        if (total * elem + (copy_g ? words * 4 + 1024 : 0) > (copy_g ? WMC_CHAIN_LDS_SHORT : WMC_CHAIN_LDS)) return false;
        if (odd_even) {
            odd_even[0] = odd;
            odd_even[1] = even;
        }
        return true;
    }

    // Places the regions of an evaluated chain: every one is a power of two of
    // entries, so that in descending order each starts at a multiple of its
    // size (addresses combine by XOR).
    void place_lds(Chain &h) const {
        const size_t L = h.nodes.size();
        int oe[2] = {0, 0};
        const bool copy_f = !h.big && lds_fits(h, h.inner, true, true, oe);
        if (!copy_f) lds_fits(h, h.inner, false, !h.big, oe);
        std::vector<std::pair<int, int>> r = {{oe[0], -1}, {oe[1], -2}};
        for (size_t i = 0; i < L; ++i) r.push_back({h.big ? 0 : 1 << bits(h.vg[i] & (h.inner | h.kap[i])), (int)i});
        std::stable_sort(r.begin(), r.end(), [](auto &x, auto &y) { return x.first > y.first; });
        int at = 0;
        for (auto &x : r) {
            (x.second == -1 ? h.odd : x.second == -2 ? h.even : h.gcopy[x.second]) = at;
            at += x.first;
        }
        h.fcopy = copy_f ? h.even : -1;
        h.lds = at;
    }

    // Chooses the inner variables of the chain and prices it; false if the
    // tiles do not fit the LDS.  Short chains copy their operands to LDS; for
    // chains of many tiles the tile size of the least cost is taken.
    bool evaluate(Chain &h) {
        Chain best;
        if (evaluate_to(h, false, best) && h.products <= kShort && bits(h.outer) <= WMC_CHAIN_TILE_BITS) return true;
        evaluate_to(h, true, best);
        if (best.nodes.empty()) return false;
        h = best;
        return true;
    }

    // The largest tiles of a short chain into h; of a chain of many tiles the
    // least dear of those that first reach 2^8 ... 2^WMC_CHAIN_BITS outputs of
    // a stage, into best.
    bool evaluate_to(Chain &h, bool big, Chain &best) {
        const size_t L = h.nodes.size();
        h.big = big;
        const std::vector<int32_t> &out = T[(size_t)h.nodes.back()].layout;
        const uint64_t vl = h.vc.back();
        // every variable summed after stage 1, and the lowest of the
        // output's order, so that its stores cover whole 128-byte lines
        uint64_t in = 0;
        for (size_t i = 1; i < L; ++i) in |= h.kap[i];
        const size_t low = elem == 8 ? 4 : 5;
        for (size_t q = 0; q < out.size() && q < low; ++q) in |= 1ull << id_of[(size_t)out[q]];
        if (!lds_fits(h, in, false, !big)) return false;
        auto take = [&](uint64_t b) {
            if (!lds_fits(h, in | b, false, !big)) return false;
            in |= b;
            return true;
        };
        // a variable that only a later stage brings in repeats the stages
        // before it once per value unless it is inside the tile
        for (size_t i = 1; i < L; ++i) {
            uint64_t late = h.vc[i] & ~h.vc[i - 1] & vl & ~in;
            while (late) {
                const uint64_t b = late & -late;
                late ^= b;
                take(b);
            }
        }
        // tiles of at least one entry per thread, larger ones while enough
        // tiles remain to fill the device
        int reached = 7;
        auto offer = [&] {
            if (measure(h, in) && (best.nodes.empty() || price(h) < price(best))) best = h;
        };
        for (int32_t v : out) {
            const uint64_t b = 1ull << id_of[(size_t)v];
            if (in & b) continue;
            int t = 0;
            for (size_t i = 0; i < L; ++i) t = std::max(t, bits(in & h.vc[i]));
            if (big && t > reached) {
                reached = t;
                offer();
            }
            if (t >= WMC_CHAIN_BITS || (t >= WMC_CHAIN_LANE_BIG && bits(vl & ~in) <= 10)) break;
            if (!take(b)) break;
        }
        if (big) offer();
        return measure(h, in);
    }

    bool measure(Chain &h, uint64_t in) const {
        const size_t L = h.nodes.size();
        const uint64_t vl = h.vc.back();
        h.inner = in;
        h.outer = vl & ~in;
        h.ebits.clear();
        h.products = 0;
        h.bytes = (double)elem * (power(bits(h.vf) + bits(h.outer & ~h.vf)) + power(bits(vl)));
        for (size_t i = 0; i < L; ++i) {
            h.ebits.push_back(bits(in & h.vc[i]));
            h.products += power(bits(h.outer) + h.ebits.back() + bits(h.kap[i]));
            h.bytes += (double)elem * power(bits(h.vg[i]));
        }
        return bits(h.outer) <= 28;
    }

    // Seconds of a launch, for all slices it runs side by side.
    double price(const Chain &h) const {
        const double L = (double)h.nodes.size(), tiles = std::ldexp(slices, bits(h.outer));
        const double rounds = std::max(1.0, tiles / kRunning);
        if (!h.big) return kLaunch + rounds * (kShortTile + kShortStage * L + slices * h.products / tiles / kTileProducts);
        double tile = kTile + kStage * L;
        for (int eb : h.ebits) tile += kRound * std::ldexp(1.0, std::max(0, eb - WMC_CHAIN_LANE_BIG - 2));
        return kLaunch + std::max(1.3 * slices * h.bytes / kBytes, (rounds + 1.0) * tile);
    }
    // The same for a contraction apart.  Small nodes share their launch with
    // the others of their level: in a plan of large tensors a level more or
    // less is nothing, in a small one it is what the time goes to.
    double price_node(int32_t c) const {
        return (T[(size_t)c].cls == WMC_CLASS_SMALL ? level : kLaunch) + slices * node_bytes(c) / kBytes;
    }
    double node_bytes(int32_t c) const {
        const TNode &C = T[(size_t)c];
        return (double)elem * (std::ldexp(1.0, rank(C.a)) + std::ldexp(1.0, rank(C.b)) + std::ldexp(1.0, rank(c)));
    }

    int lift(const Chain &h) const {
        int summed = 0;
        for (uint64_t k : h.kap) summed += bits(k);
        return top(h.nodes.back()) - summed;
    }
    // Bound of the stored magnitudes of a chain that ends at `out`.
    int top(int32_t out) const {
        const int32_t up = T[(size_t)out].parent;
        if (elem == 8) return WMC_CHAIN_TOP_FP64;
        return up >= 0 && nk[(size_t)up] >= 4 ? WMC_CHAIN_TOP_FP32_MATRIX : WMC_CHAIN_TOP_FP32;
    }

    // The chain's words.  Positions: the entry index of stage i's output
    // tile numbers its inner variables in F_i's storage order (F_i stores
    // [kappa_{i+1} | F_{i+1}'s order], so the summed entries of the next
    // stage are contiguous and every tile is read and written in runs).
    void emit(const Chain &h, FusedProgram &F, ChainTask &t) {
        const size_t L = h.nodes.size();
        ++now;
        for (size_t q = 0; q < h.local.size(); ++q) {
            stamp[(size_t)h.local[q]] = now;
            id_of[(size_t)h.local[q]] = (int32_t)q;
        }
        auto bit = [&](int32_t v) { return 1ull << id_of[(size_t)v]; };
        auto place = [&](int32_t tensor) {
            std::vector<int> p(h.local.size(), -1);
            const std::vector<int32_t> &lay = T[(size_t)tensor].layout;
            for (size_t q = 0; q < lay.size(); ++q) p[(size_t)id_of[(size_t)lay[q]]] = (int)q;
            return p;
        };
        auto offset = [](int p) { return p < 0 ? 0u : 1u << p; };
        while (F.words.size() % 4) F.words.push_back(0);
        t.nodes.assign(h.nodes.begin(), h.nodes.end());
        t.g.assign(h.gs.begin(), h.gs.end());
        t.f = h.f;
        t.desc = (unsigned)F.words.size();
        t.tile_bits = bits(h.outer);
        t.lds = h.lds;
        t.big = h.big;
        t.work = h.products;
        std::vector<unsigned> w(CH_WORDS, 0u);
        w[CH_STAGES] = (unsigned)L;
        w[CH_TILE_BITS] = (unsigned)t.tile_bits;
        w[CH_TF] = (unsigned)h.f;
        w[CH_TC] = (unsigned)h.nodes.back();
        w[CH_MASK] = (unsigned)h.nodes.front();
        w[CH_NT] = rank(h.nodes.back()) >= 23 ? 1u : 0u;
        // tile index bits: variables F_0 does not have first (tiles that
        // read the same F_0 entries run together), then the others in order
        std::vector<int32_t> tv;
        for (int pass = 0; pass < 2; ++pass)
            for (int32_t v : T[(size_t)h.nodes.back()].layout)
                if ((h.outer & bit(v)) && ((h.vf & bit(v)) != 0) == (pass == 1)) tv.push_back(v);
        const std::vector<int> pf = place(h.f), pl = place(h.nodes.back());
        // an operand's copy: its variables summed at the stage or inside the
        // tile, in storage order; returns their bit positions in the copy
        std::vector<std::pair<size_t, std::vector<unsigned>>> lists;
        auto copy = [&](size_t x, int32_t tensor, uint64_t vars, int lds) {
            std::vector<int> at(h.local.size(), -1);
            const std::vector<int32_t> &lay = T[(size_t)tensor].layout;
            std::vector<unsigned> off;
            unsigned low = 0;
            for (size_t q = 0; q < lay.size(); ++q) {
                if (!(vars & bit(lay[q]))) continue;
                at[(size_t)id_of[(size_t)lay[q]]] = (int)off.size();
                if (low == off.size() && q == off.size()) ++low;
                off.push_back(1u << q);
            }
            w[x + CX_BITS] = (unsigned)off.size();
            w[x + CX_LOW] = low;
            w[x + CX_LDS] = (unsigned)lds;
            if (low < off.size()) lists.push_back({x, std::vector<unsigned>(off.begin() + low, off.end())});
            return at;
        };
        std::vector<int> src = pf;  // bit positions in the stage's source
        w[CH_FCOPY] = h.fcopy >= 0 ? 1u : 0u;
        if (h.fcopy >= 0) src = copy(CH_X, h.f, h.vf & (h.inner | h.kap[0]), h.fcopy);
        for (size_t i = 0; i < L; ++i) {
            const uint64_t vp = i ? h.vc[i - 1] : h.vf;
            const bool last = i + 1 == L;
            // entry bits of the output tile, in F_i's storage order
            std::vector<int32_t> ev;
            for (int32_t v : T[(size_t)h.nodes[i]].layout)
                if (h.inner & bit(v)) ev.push_back(v);
            std::vector<int> dst(h.local.size(), -1);
            for (size_t q = 0; q < ev.size(); ++q)
                dst[(size_t)id_of[(size_t)ev[q]]] = last ? pl[(size_t)id_of[(size_t)ev[q]]] : (int)q;
            // register bits (chains of many tiles): the highest one-operand
            // entry bits, as long as every thread keeps an entry; one of each kind first (a G row
            // is then used twice and a source row twice)
            int budget = h.big ? std::min(2, std::max(0, (int)ev.size() - WMC_CHAIN_LANE_BIG)) : 0;
            std::vector<int32_t> pb, qb;
            auto pick = [&](bool p) {
                for (size_t q = ev.size(); q-- > 0;) {
                    const uint64_t b = bit(ev[q]);
                    const bool only = p ? ((vp & b) && !(h.vg[i] & b)) : ((h.vg[i] & b) && !(vp & b));
                    if (only && std::find(pb.begin(), pb.end(), ev[q]) == pb.end() &&
                        std::find(qb.begin(), qb.end(), ev[q]) == qb.end()) {
                        (p ? pb : qb).push_back(ev[q]);
                        --budget;
                        return true;
                    }
                }
                return false;
            };
            if (budget > 0) pick(true);
            if (budget > 0) pick(false);
            while (budget > 0 && (pick(true) || pick(false))) {
            }
            std::vector<int32_t> tb;
            for (int32_t v : ev)
                if (std::find(pb.begin(), pb.end(), v) == pb.end() && std::find(qb.begin(), qb.end(), v) == qb.end())
                    tb.push_back(v);
            const size_t s = w.size();
            w.resize(s + (size_t)(h.big ? CS_WORDS_BIG : CS_WORDS), 0u);
            w[s + CS_SHAPE] = (unsigned)bits(h.kap[i]) | ((unsigned)pb.size() << 8) | ((unsigned)qb.size() << 16);
            w[s + CS_TBITS] = (unsigned)tb.size();
            w[s + CS_TG] = (unsigned)h.gs[i];
            w[s + CS_SRC] = (unsigned)(i ? (i % 2 ? h.odd : h.even) : std::max(h.fcopy, 0));
            w[s + CS_DST] = (unsigned)(last ? 0 : i % 2 ? h.even : h.odd);
            if (i == 0) w[s + CS_LIFT] = (unsigned)lift(h);
            const std::vector<int> pg =
                h.big ? place(h.gs[i]) : copy(s + CS_X, h.gs[i], h.vg[i] & (h.inner | h.kap[i]), h.gcopy[i]);
            auto S = [&](int32_t v) { return (vp & bit(v)) ? offset(src[(size_t)id_of[(size_t)v]]) : 0u; };
            auto G = [&](int32_t v) { return offset(pg[(size_t)id_of[(size_t)v]]); };
            auto D = [&](int32_t v) { return offset(dst[(size_t)id_of[(size_t)v]]); };
            for (size_t q = 0; q < tb.size(); ++q) {
                if (h.big) {
                    w[s + CS_BIT_S + q] = S(tb[q]);
                    w[s + CS_BIT_G + q] = G(tb[q]);
                    w[s + CS_BIT_O + q] = D(tb[q]);
                    continue;
                }
                const bool memory = i == 0 && h.fcopy < 0;
                w[s + CS_BIT_SG + q] = (memory ? 0u : S(tb[q])) | (G(tb[q]) << 16);
                if (memory) w[CH_SRC + q] = S(tb[q]);
                if (last) w[CH_OUT + q] = D(tb[q]);
            }
            for (size_t q = 0; q < pb.size(); ++q) {
                w[s + CS_PS + q] = S(pb[q]);
                w[s + CS_PO + q] = D(pb[q]);
            }
            for (size_t q = 0; q < qb.size(); ++q) {
                w[s + CS_QG + q] = G(qb[q]);
                w[s + CS_QO + q] = D(qb[q]);
            }
            src = dst;
        }
        w[CH_TILES] = (unsigned)w.size();
        for (int32_t v : tv) w.push_back(offset(pf[(size_t)id_of[(size_t)v]]));
        for (int32_t v : tv) w.push_back(offset(pl[(size_t)id_of[(size_t)v]]));
        for (size_t i = 0; i < L; ++i) {
            const std::vector<int> pg = place(h.gs[i]);
            for (int32_t v : tv) w.push_back(offset(pg[(size_t)id_of[(size_t)v]]));
        }
        for (const auto &l : lists) {
            w[l.first + CX_LIST] = (unsigned)w.size();
            w.insert(w.end(), l.second.begin(), l.second.end());
        }
        F.words.insert(F.words.end(), w.begin(), w.end());
    }
};

}  // namespace

void wmc_fuse(wmc_plan_t &P, uint64_t max_arena) {
    FusedProgram &F = P.fused;
    F = FusedProgram();
    if (P.root < 0 || P.nodes.empty()) return;
    const size_t NT = P.T.size();
    Fuser fu(P);
    // Along each path on which every contraction takes the one below as its
    // larger operand: the partition into chains and single contractions of
    // the least cost.
    std::vector<Chain> chains;
    std::vector<int32_t> chain_of(NT, -1);
    double saved = 0;
    for (int32_t c0 : P.node_order) {
        const int32_t below = fu.big(c0);
        if (!fu.fits(c0) || (P.T[(size_t)below].kind == 2 && fu.fits(below))) continue;
        std::vector<int32_t> path = {c0};
        for (int32_t up = P.T[(size_t)c0].parent; up >= 0 && fu.big(up) == path.back() && fu.fits(up);
             up = P.T[(size_t)up].parent)
            path.push_back(up);
        const size_t m = path.size();
        std::vector<double> cost(m + 1, 0.0);  // of the first q contractions
        std::vector<int> from(m + 1, -1);      // where the last part of that partition starts
        for (size_t q = 0; q < m; ++q) cost[q + 1] = HUGE_VAL;
        for (size_t i = 0; i < m; ++i) {
            const double one = cost[i] + fu.price_node(path[i]);
            if (one < cost[i + 1]) {
                cost[i + 1] = one;
                from[i + 1] = (int)i;
            }
            // no chain costs less than a short one of one tile: where even that
            // would be no gain, none is built
            auto gains = [&](size_t j) {
                return cost[i] + kLaunch + kShortTile + kShortStage * (double)(j - i + 1) < cost[j + 1];
            };
            size_t end = std::min(m, i + WMC_CHAIN_MAX);
            while (end > i + 1 && !gains(end - 1)) --end;
            Chain h;
            if (end == i + 1 || !fu.begin(h, path[i])) continue;
            int most = fu.rank(path[i]);
            for (size_t j = i + 1; j < end; ++j) {
                if (!fu.extend(h, path[j])) break;
                most = std::max(most, fu.rank(path[j]));
                if (most < 6) continue;  // a handful of entries: left to the batched small nodes
                if (!gains(j)) continue;
                if (!fu.evaluate(h)) break;
                const double c = cost[i] + fu.price(h);
                if (c < cost[j + 1]) {
                    cost[j + 1] = c;
                    from[j + 1] = (int)i;
                }
            }
        }
        for (int32_t q : path) saved += fu.price_node(q);
        saved -= cost[m];
        for (size_t j = m; j > 0; j = (size_t)from[j]) {
            const size_t i = (size_t)from[j];
            if (j - i < 2) continue;
            Chain h;
            bool ok = fu.begin(h, path[i]);
            for (size_t q = i + 1; q < j && ok; ++q) ok = fu.extend(h, path[q]);
            if (!ok || !fu.evaluate(h)) continue;
            fu.place_lds(h);
            for (int32_t q : h.nodes) chain_of[(size_t)q] = (int32_t)chains.size();
            chains.push_back(std::move(h));
        }
    }
    // A plan whose time goes to nodes that no chain takes (K >= 16) keeps its
    // launch list: fusing only its small ends made the row-major 24x24 lattice
    // 0.6% and the banded 300-variable formula 0.3% slower (FP64; the larger
    // image), while plans that gain save over a tenth (min-fill lattice 50%).
    if (chains.empty() || (fu.total > 1e-3 && saved < 0.05 * fu.total)) return;

    // items: a chain or a single node, in launch order of their last node;
    // all ready small ones share a launch, big ones run alone
    struct Item {
        int32_t chain = -1, node = -1, pending = 0;
        bool small = false;
    };
    std::vector<int32_t> node_at(NT, -1);
    for (size_t q = 0; q < P.nodes.size(); ++q) node_at[(size_t)P.nodes[q].tc] = (int32_t)q;
    std::vector<Item> items;
    std::vector<int32_t> item_of(NT, -1);
    for (size_t q = 0; q < chains.size(); ++q) {
        Item it;
        it.chain = (int32_t)q;
        it.small = !chains[q].big;
        for (int32_t t : chains[q].nodes) item_of[(size_t)t] = (int32_t)items.size();
        items.push_back(it);
    }
    for (int32_t c : P.node_order)
        if (chain_of[(size_t)c] < 0) {
            Item it;
            it.node = c;
            it.small = P.T[(size_t)c].cls == WMC_CLASS_SMALL;
            item_of[(size_t)c] = (int32_t)items.size();
            items.push_back(it);
        }
    auto inputs = [&](const Item &it, std::vector<int32_t> &in) {
        in.clear();
        if (it.chain >= 0) {
            const Chain &h = chains[(size_t)it.chain];
            in.assign(h.gs.begin(), h.gs.end());
            in.push_back(h.f);
        } else {
            in.push_back(P.T[(size_t)it.node].a);
            in.push_back(P.T[(size_t)it.node].b);
        }
    };
    std::vector<int32_t> in, ready_small, ready_big;
    auto out_of = [&](const Item &it) { return it.chain >= 0 ? chains[(size_t)it.chain].nodes.back() : it.node; };
    for (size_t q = 0; q < items.size(); ++q) {
        inputs(items[q], in);
        for (int32_t t : in) items[q].pending += P.T[(size_t)t].kind == 2;
        if (!items[q].pending) (items[q].small ? ready_small : ready_big).push_back((int32_t)q);
    }
    std::vector<std::vector<int32_t>> steps;
    size_t done = 0;
    while (done < items.size()) {
        std::vector<int32_t> step;
        auto by_node = [&](int32_t a, int32_t b) { return out_of(items[(size_t)a]) < out_of(items[(size_t)b]); };
        if (!ready_small.empty()) {
            step.swap(ready_small);
            std::sort(step.begin(), step.end(), by_node);
        } else if (!ready_big.empty()) {
            auto it = std::min_element(ready_big.begin(), ready_big.end(), by_node);
            step.push_back(*it);
            ready_big.erase(it);
        } else {
            return;  // not a tree: keep the node-by-node form
        }
        done += step.size();
        for (int32_t q : step) {
            const int32_t up = P.T[(size_t)out_of(items[(size_t)q])].parent;
            if (up < 0) continue;
            Item &it = items[(size_t)item_of[(size_t)up]];
            if (--it.pending == 0) (it.small ? ready_small : ready_big).push_back(item_of[(size_t)up]);
        }
        steps.push_back(std::move(step));
    }

    // A small plan keeps its launch list, too, if chains neither save a tenth of
    // its launches, nor eight, nor a twentieth of its time in bytes: the larger
    // image then costs more than they save.  Row-by-row lattices in blocks of 5
    // and 6 that saved 0 to 3 launches of 23 to 96 ran at 0.96 to 1.00 of the
    // list's speed; those in blocks of 3 that saved 10 and more of 82 to 131 at
    // 1.04 to 1.06, and plans of a dozen launches that saved two at 1.01 to 1.06.
    if (fu.total <= 1e-3) {
        const double n = (double)(P.launches.size() - 1), less = n - (double)steps.size();
        double bytes = 0;
        for (const Chain &h : chains) {
            for (int32_t c : h.nodes) bytes += fu.node_bytes(c);
            bytes -= h.bytes;
        }
        if (less < 0.1 * n && less < 8 && fu.slices * bytes / kBytes < 0.05 * (n * kLaunch + fu.total)) return;
    }

    // placement: a tensor lives from its writer's launch to its reader's
    const int32_t NL = (int32_t)steps.size() + 1;
    std::vector<int32_t> at(items.size(), 0);
    for (size_t k = 0; k < steps.size(); ++k)
        for (int32_t q : steps[k]) at[(size_t)q] = (int32_t)k + 1;
    std::vector<int32_t> stored, birth, death;
    std::vector<uint64_t> elems;
    const uint64_t align = 256 / (uint64_t)P.elem;
    for (size_t t = 0; t < NT; ++t) {
        const bool internal = P.T[t].kind == 2;
        if (internal && out_of(items[(size_t)item_of[t]]) != (int32_t)t) continue;  // only in LDS
        stored.push_back((int32_t)t);
        birth.push_back(internal ? at[(size_t)item_of[t]] : 0);
        const int32_t up = P.T[t].parent;
        death.push_back(up < 0 ? NL : at[(size_t)item_of[(size_t)up]]);
        elems.push_back((((uint64_t)1 << fu.rank((int32_t)t)) + align - 1) / align * align);
    }
    std::vector<int64_t> offs;
    const uint64_t arena_bytes = wmc_place(birth, death, elems, &offs) * (uint64_t)P.elem;
    if (arena_bytes > max_arena) return;
    F.arena_bytes = arena_bytes;
    F.off.assign(NT, -1);
    for (size_t q = 0; q < stored.size(); ++q) F.off[(size_t)stored[q]] = offs[q];

    // descriptors
    auto off = [&](int32_t t) { return (long long)F.off[(size_t)t]; };
    F.leaves = P.leaves;
    for (LeafDesc &d : F.leaves) d.out = off(d.tensor);
    if (F.leaves.size() > 1) {
        F.leaf_tab = 0;
        F.tabs.assign((size_t)(P.leaf_work / WMC_WAVE), 0);
        for (size_t q = 0; q < F.leaves.size(); ++q)
            for (int64_t x = 0; x < (int64_t)(((1ull << F.leaves[q].rank) + WMC_WAVE - 1) / WMC_WAVE); ++x)
                F.tabs[(size_t)(F.leaves[q].work_begin / WMC_WAVE + x)] = (int32_t)q;
    }
    for (const std::vector<int32_t> &step : steps) {
        FusedLaunch L;
        L.node_first = (int32_t)F.nodes.size();
        L.chain_first = (int32_t)F.chains.size();
        L.rec_first = (int32_t)F.recs.size();
        for (int32_t q : step) {
            const Item &it = items[(size_t)q];
            if (it.chain >= 0) {
                ChainTask t;
                fu.emit(chains[(size_t)it.chain], F, t);
                unsigned *w = F.words.data() + t.desc;
                auto put = [&](unsigned at_word, long long v) {
                    w[at_word] = (unsigned)(unsigned long long)v;
                    w[at_word + 1] = (unsigned)((unsigned long long)v >> 32);
                };
                put(CH_F, off(t.f));
                put(CH_C, off(t.nodes.back()));
                for (size_t s = 0; s < t.g.size(); ++s) put((unsigned)(CH_WORDS + s * (t.big ? CS_WORDS_BIG : CS_WORDS)) + CS_G, off(t.g[s]));
                if (t.nodes.size() > 1) F.masks.push_back(t.nodes.front());
                L.lds = std::max(L.lds, t.lds + (t.big ? 0 : ((int)(F.words.size() - t.desc) * 4 + 1023) / 1024 * 1024 / P.elem));
                if (t.big) L.type = FUSED_CHAIN;
                // workgroups: one tile each up to the launch's share of the
                // device, then equal runs of consecutive tiles; dealt so
                // that each XCD (workgroup index modulo 8) walks one slab.
                // The share: about 2^11 workgroups over all slices of a group
                // fill the device and leave each several tiles to spread its
                // start over.  Min-fill 24x24 lattice FP64, ms at 2^7 / 2^8 /
                // 2^10 / 2^11 / 2^12 workgroups per slice: 1 slice 165 / 101 /
                // 75.2 / 73.5 / 75.8, 4 slices 55.6 / 53.5 / 50.7 / 51.2 / 54.3,
                // 16 slices 44.6 / 43.1 / 43.5 / 48.2 / 48.0, 64 slices 41.4 /
                // 40.4 / 41.4 / 42.7 / 46.0
                const int cap_bits = P.group >= 8 ? 8 : P.group >= 2 ? 10 : 11;
                const int jb = t.big ? std::max(0, t.tile_bits - cap_bits) : 0;
                const unsigned n = 1u << (t.tile_bits - jb);
                for (unsigned b = 0; b < n; ++b)
                    F.recs.push_back({t.desc, n % 8 ? b : (b % 8) * (n / 8) + b / 8, (unsigned)jb,
                                      (unsigned)F.words.size() - t.desc});
                F.chains.push_back(std::move(t));
                continue;
            }
            const int32_t nd = node_at[(size_t)it.node];
            NodeDesc d = P.nodes[(size_t)nd];
            d.a = off(d.ta);
            d.b = off(d.tb);
            d.c = off(d.tc);
            if (P.T[(size_t)it.node].cls == WMC_CLASS_GEMM) {
                for (GemmDesc g : P.gemms)
                    if (g.tc == it.node) {
                        g.a = off(g.ta);
                        g.b = off(g.tb);
                        g.c = off(g.tc);
                        L.type = FUSED_GEMM;
                        L.gemm = (int32_t)F.gemms.size();
                        F.gemms.push_back(g);
                        break;
                    }
            } else if (!it.small) {
                L.type = FUSED_NODE;
            }
            d.work_begin = L.node_work;
            L.node_work += (int64_t)(((1ull << d.rc) + WMC_WAVE - 1) / WMC_WAVE * WMC_WAVE);
            F.nodes.push_back(d);
        }
        L.node_count = (int32_t)F.nodes.size() - L.node_first;
        L.chain_count = (int32_t)F.chains.size() - L.chain_first;
        L.rec_count = (int32_t)F.recs.size() - L.rec_first;
        if (L.type == FUSED_STEP && L.node_count > 1) {
            L.tab = (int64_t)F.tabs.size();
            F.tabs.resize(F.tabs.size() + (size_t)(L.node_work / WMC_WAVE), 0);
            for (int32_t q = 0; q < L.node_count; ++q) {
                const NodeDesc &d = F.nodes[(size_t)(L.node_first + q)];
                for (int64_t x = 0; x < (int64_t)(((1ull << d.rc) + WMC_WAVE - 1) / WMC_WAVE); ++x)
                    F.tabs[(size_t)(L.tab + d.work_begin / WMC_WAVE + x)] = q;
            }
        }
        F.launches.push_back(L);
    }

    // image
    uint64_t o = 0;
    auto part = [&](uint64_t &at_byte, size_t bytes) {
        at_byte = o;
        o = (o + std::max<size_t>(bytes, 1) + 255) / 256 * 256;
    };
    part(F.o_leaf, sizeof(LeafDesc) * F.leaves.size());
    part(F.o_node, sizeof(NodeDesc) * F.nodes.size());
    part(F.o_gemm, sizeof(GemmDesc) * F.gemms.size());
    part(F.o_words, sizeof(unsigned) * F.words.size());
    part(F.o_recs, sizeof(ChainRec) * F.recs.size());
    part(F.o_tab, sizeof(int32_t) * F.tabs.size());
    part(F.o_masks, sizeof(int32_t) * F.masks.size());
    F.image.assign((size_t)o, 0);
    auto fill = [&](uint64_t at_byte, const void *src, size_t bytes) {
        if (bytes) std::memcpy(F.image.data() + at_byte, src, bytes);
    };
    fill(F.o_leaf, F.leaves.data(), sizeof(LeafDesc) * F.leaves.size());
    fill(F.o_node, F.nodes.data(), sizeof(NodeDesc) * F.nodes.size());
    fill(F.o_gemm, F.gemms.data(), sizeof(GemmDesc) * F.gemms.size());
    fill(F.o_words, F.words.data(), sizeof(unsigned) * F.words.size());
    fill(F.o_recs, F.recs.data(), sizeof(ChainRec) * F.recs.size());
    fill(F.o_tab, F.tabs.data(), sizeof(int32_t) * F.tabs.size());
    fill(F.o_masks, F.masks.data(), sizeof(int32_t) * F.masks.size());
    F.on = true;
}

FusedProgram wmc_program_of(const wmc_plan_t &P, bool fused) {
    if (fused && P.fused.on) return P.fused;
    FusedProgram F;
    F.leaves = P.leaves;
    F.nodes = P.nodes;
    F.gemms = P.gemms;
    for (const TNode &t : P.T) F.off.push_back(t.off);
    for (size_t k = 1; k < P.launches.size(); ++k) {
        const Launch &Ln = P.launches[k];
        FusedLaunch L;
        L.type = Ln.type == LAUNCH_GEMM ? FUSED_GEMM
                 : Ln.count == 1 && P.nodes[(size_t)Ln.first].cls != WMC_CLASS_SMALL ? FUSED_NODE : FUSED_STEP;
        L.node_first = Ln.first;
        L.node_count = Ln.count;
        L.node_work = Ln.work;
        L.gemm = Ln.type == LAUNCH_GEMM ? Ln.pad : -1;
        F.launches.push_back(L);
    }
    return F;
}

double wmc_fused_busy_us(const wmc_plan_t &P) {
    const FusedProgram &F = P.fused;
    auto size = [&](int32_t t) { return std::ldexp(1.0, (int)P.T[(size_t)t].layout.size()); };
    double bytes = 0, stages = 0, products = 0, big_stages = 0;
    for (const NodeDesc &d : F.nodes) bytes += (double)P.elem * (size(d.ta) + size(d.tb) + size(d.tc));
    for (const ChainTask &t : F.chains) {
        const double st = std::ldexp((double)t.nodes.size(), t.tile_bits);
        if (t.big) big_stages += st;
        else stages += st, products += t.work;
    }
    return wmc_chain_busy_us(bytes, stages, products, big_stages);
}

unsigned wmc_shift_chain(const FusedProgram &F, const ChainTask &t, unsigned words, long long abase, int mbase,
                         std::vector<unsigned> &out) {
    while (out.size() % 4) out.push_back(0);
    const size_t at = out.size();
    out.insert(out.end(), F.words.begin() + t.desc, F.words.begin() + t.desc + words);
    unsigned *w = out.data() + at;
    auto shift = [&](size_t q) {
        const unsigned long long v = (((unsigned long long)w[q + 1] << 32) | w[q]) + (unsigned long long)abase;
        w[q] = (unsigned)v;
        w[q + 1] = (unsigned)(v >> 32);
    };
    shift(CH_F);
    shift(CH_C);
    for (int q : {(int)CH_TF, (int)CH_TC, (int)CH_MASK}) w[q] += (unsigned)mbase;
    for (unsigned s = 0; s < w[CH_STAGES]; ++s) {
        const size_t q = CH_WORDS + (size_t)s * (t.big ? CS_WORDS_BIG : CS_WORDS);
        shift(q + CS_G);
        w[q + CS_TG] += (unsigned)mbase;
    }
    return (unsigned)at;
}

// Bounds of the fused program: every tensor inside the arena, and for every
// stage of every chain the largest address its index bits can form (the OR
// of all of them) inside the tensor or LDS region it reads or writes.
bool wmc_validate_fused(const wmc_plan_t &P, std::string *why) {
    const FusedProgram &F = P.fused;
    if (!F.on) return true;
    auto fail = [&](const char *what) {
        *why = std::string("fused program: ") + what;
        return false;
    };
    auto rank = [&](int32_t t) { return (int)P.T[(size_t)t].layout.size(); };
    const uint64_t arena = std::max(P.arena_bytes, F.arena_bytes) / (uint64_t)P.elem;
    for (size_t t = 0; t < F.off.size(); ++t)
        if (F.off[t] >= 0 && (uint64_t)F.off[t] + (1ull << rank((int32_t)t)) > arena) return fail("tensor outside the arena");
    std::map<unsigned, unsigned> used;  // words of the chain at a word
    for (const ChainTask &t : F.chains) {
        const unsigned *w = F.words.data() + t.desc;
        if (t.desc + (uint64_t)CH_WORDS > F.words.size()) return fail("chain header");
        const uint64_t have = F.words.size() - t.desc;
        const unsigned L = w[CH_STAGES], ob = w[CH_TILE_BITS];
        if (L < 1 || L > WMC_CHAIN_MAX || L != t.nodes.size() || (int)w[CH_TC] != t.nodes.back() || (int)w[CH_TF] != t.f)
            return fail("chain header");
        if (F.off[(size_t)t.f] < 0 || F.off[(size_t)t.nodes.back()] < 0) return fail("chain operand is not stored");
        const unsigned stride = t.big ? CS_WORDS_BIG : CS_WORDS;
        const unsigned *tiles = w + w[CH_TILES];
        if (w[CH_TILES] != CH_WORDS + L * stride || ob > 28 || w[CH_TILES] + (L + 2) * ob > have) return fail("tile lists");
        unsigned &words = used[t.desc];
        words = w[CH_TILES] + (L + 2) * ob;
        unsigned long long of = 0, oc = 0;
        for (unsigned b = 0; b < ob; ++b) {
            of |= tiles[b];
            oc |= tiles[ob + b];
        }
        // LDS regions: [start, end) of what a stage writes and of the copies
        auto inside = [&](unsigned start, unsigned long long top, unsigned *end) {
            unsigned size = 1;
            while (size <= top) size *= 2;
            *end = start + size;
            return start % size == 0 && *end <= (unsigned)t.lds;
        };
        auto copied = [&](const unsigned *x, unsigned long long tiles_or, int tensor, unsigned *end) {
            unsigned long long all = tiles_or;
            if (x[CX_BITS] > WMC_CHAIN_BITS || x[CX_LOW] > x[CX_BITS]) return false;
            all |= (1ull << x[CX_LOW]) - 1ull;
            if (x[CX_LOW] < x[CX_BITS]) {
                const uint64_t last = (uint64_t)x[CX_LIST] + x[CX_BITS] - x[CX_LOW];
                if (x[CX_LIST] < w[CH_TILES] + (L + 2) * ob || last > have) return false;
                words = std::max(words, (unsigned)last);
            }
            for (unsigned b = x[CX_LOW]; b < x[CX_BITS]; ++b) all |= w[x[CX_LIST] + b - x[CX_LOW]];
            return (all >> rank(tensor)) == 0 && inside(x[CX_LDS], (1ull << x[CX_BITS]) - 1ull, end);
        };
        unsigned fe = 0, lo = 0, hi = 0;
        const bool fcopy = w[CH_FCOPY] != 0;
        if (fcopy && !copied(w + CH_X, of, t.f, &fe)) return fail("copy of the first operand");
        if (t.lds * P.elem > (t.big ? WMC_CHAIN_LDS : WMC_CHAIN_LDS_SHORT)) return fail("LDS size");
        std::vector<std::pair<unsigned, unsigned>> gr;
        unsigned summed = 0;
        for (unsigned i = 0; i < L; ++i) summed += w[CH_WORDS + i * stride + CS_SHAPE] & 255u;
        if (w[CH_WORDS + CS_LIFT] + summed > (unsigned)(P.elem == 8 ? WMC_CHAIN_TOP_FP64 : WMC_CHAIN_TOP_FP32))
            return fail("lift");
        for (unsigned i = 0; i < L; ++i) {
            const unsigned *s = w + CH_WORDS + i * stride;
            unsigned long long og = 0;
            for (unsigned b = 0; b < ob; ++b) og |= tiles[(2 + i) * ob + b];
            unsigned e = 0;
            if ((int)s[CS_TG] != t.g[i] || F.off[(size_t)t.g[i]] < 0) return fail("stage operand is not stored");
            if (t.big) {
                unsigned long long g = og | ((1ull << (s[CS_SHAPE] & 255u)) - 1ull) | s[CS_QG] | s[CS_QG + 1];
                for (unsigned q = 0; q < WMC_CHAIN_BITS; ++q) g |= s[CS_BIT_G + q];
                if (g >> rank(t.g[i])) return fail("second operand");
                continue;
            }
            if (!copied(s + CS_X, og, t.g[i], &e)) return fail("copy of the second operand");
            for (const auto &r : gr)
                if (r.first < e && s[CS_X + CX_LDS] < r.second) return fail("copies overlap");
            if (fcopy && w[CH_X + CX_LDS] < e && s[CS_X + CX_LDS] < fe) return fail("copies overlap");
            gr.push_back({s[CS_X + CX_LDS], e});
        }
        for (unsigned i = 0; i < L; ++i) {
            const unsigned *s = w + CH_WORDS + i * stride;
            const unsigned nk = s[CS_SHAPE] & 255u, np = (s[CS_SHAPE] >> 8) & 255u, nq = s[CS_SHAPE] >> 16;
            const unsigned tb = s[CS_TBITS];
            if (nk > WMC_CHAIN_NK || np + nq > 2 || (!t.big && np + nq) || tb + np + nq > WMC_CHAIN_BITS)
                return fail("stage shape");
            unsigned long long src = 0, g = 0, out = 0;
            for (unsigned q = 0; q < 2; ++q) {
                if (!t.big) break;
                src |= s[CS_PS + q];
                out |= s[CS_PO + q] | s[CS_QO + q];
                g |= s[CS_QG + q];
            }
            for (unsigned q = 0; q < WMC_CHAIN_BITS; ++q) {
                src |= t.big ? s[CS_BIT_S + q] : i == 0 && !fcopy ? w[CH_SRC + q] : s[CS_BIT_SG + q] & 0xFFFFu;
                g |= t.big ? s[CS_BIT_G + q] : s[CS_BIT_SG + q] >> 16;
                out |= t.big ? s[CS_BIT_O + q] : i + 1 == L ? w[CH_OUT + q] : q < tb ? 1u << q : 0u;
            }
            const unsigned long long row = (1ull << nk) - 1ull;
            if ((src & row) || (g & row)) return fail("summed entries of a row are not contiguous");
            if (!t.big && ((g | row) >> s[CS_X + CX_BITS])) return fail("second operand");
            if (i == 0) {
                if (fcopy ? ((src | row) >> w[CH_X + CX_BITS]) != 0 || s[CS_SRC] != w[CH_X + CX_LDS]
                          : ((src | of | row) >> rank(t.f)) != 0)
                    return fail("first operand");
            } else if (s[CS_SRC] != lo || lo + (src | row) >= hi) {
                return fail("LDS source");
            }
            if (i + 1 == L) {
                if ((out | oc) >> rank(t.nodes.back())) return fail("output");
                continue;
            }
            const unsigned from = i ? lo : fcopy ? w[CH_X + CX_LDS] : 0u, to = i ? hi : fcopy ? fe : 0u;
            lo = s[CS_DST];
            if (!inside(lo, out, &hi)) return fail("LDS output");
            if (from < hi && lo < to) return fail("LDS regions overlap");
            for (const auto &r : gr)
                if (r.first < hi && lo < r.second) return fail("LDS output over a copy");
        }
    }
    for (const ChainRec &r : F.recs) {
        // the chain's words end before the next chain's begin
        const auto at = used.find(r.desc);
        if (at == used.end()) return fail("workgroup record");
        const auto next = std::next(at);
        const uint64_t end = next == used.end() ? F.words.size() : next->first;
        const unsigned ob = F.words[r.desc + CH_TILE_BITS];
        if (r.jbits > ob || r.blk >> (ob - r.jbits) || r.words < at->second || r.words > 3u << WMC_CHAIN_LANE ||
            r.desc + (uint64_t)r.words > end)
            return fail("workgroup record");
    }
    return true;
}

// Raw image of the fused program, for tools and tests:
// [LeafDesc][NodeDesc][GemmDesc][chain words u32][ChainRec][per launch: type,
// node_first, node_count, chain_first, chain_count, gemm, rec_first, rec_count
// (int32)][per chain: first word u32][tensor offsets int64, -1: never stored];
// info[] = {n_leaves, n_nodes, n_gemms, n_words, n_recs, n_launches, n_chains,
//           n_tensors, arena_elems}.  An empty program (n_launches 0) means
// that wmc_contract runs the plan's launch list as it is.
extern "C" wmc_status wmc_plan_program(const wmc_plan_t *plan, void *dst, uint64_t dst_bytes, uint64_t *needed,
                                       int64_t *info) {
    if (!plan) {
        wmc_set_error("wmc_plan_program: plan is NULL");
        return WMC_ERR_INVALID_ARGUMENT;
    }
    static const FusedProgram none;
    const FusedProgram &F = plan->fused.on ? plan->fused : none;
    const uint64_t need = sizeof(LeafDesc) * F.leaves.size() + sizeof(NodeDesc) * F.nodes.size() +
                          sizeof(GemmDesc) * F.gemms.size() + sizeof(unsigned) * F.words.size() +
                          sizeof(ChainRec) * F.recs.size() + 8 * sizeof(int32_t) * F.launches.size() +
                          sizeof(unsigned) * F.chains.size() + sizeof(int64_t) * F.off.size();
    if (needed) *needed = need;
    if (info) {
        const int64_t v[9] = {(int64_t)F.leaves.size(), (int64_t)F.nodes.size(),    (int64_t)F.gemms.size(),
                              (int64_t)F.words.size(),  (int64_t)F.recs.size(),     (int64_t)F.launches.size(),
                              (int64_t)F.chains.size(), (int64_t)plan->T.size(), (int64_t)(plan->arena_stride / (uint64_t)plan->elem)};
        std::memcpy(info, v, sizeof v);
    }
    if (!dst) return WMC_OK;
    if (dst_bytes < need) {
        wmc_set_error("wmc_plan_program: buffer too small");
        return WMC_ERR_OUT_OF_MEMORY;
    }
    char *p = (char *)dst;
    auto put = [&](const void *src, size_t bytes) {
        if (bytes) std::memcpy(p, src, bytes);
        p += bytes;
    };
    put(F.leaves.data(), sizeof(LeafDesc) * F.leaves.size());
    put(F.nodes.data(), sizeof(NodeDesc) * F.nodes.size());
    put(F.gemms.data(), sizeof(GemmDesc) * F.gemms.size());
    put(F.words.data(), sizeof(unsigned) * F.words.size());
    put(F.recs.data(), sizeof(ChainRec) * F.recs.size());
    for (const FusedLaunch &L : F.launches) {
        const int32_t row[8] = {L.type,        L.node_first, L.node_count, L.chain_first,
                                L.chain_count, L.gemm,       L.rec_first,  L.rec_count};
        put(row, sizeof row);
    }
    for (const ChainTask &t : F.chains) put(&t.desc, sizeof t.desc);
    put(F.off.data(), sizeof(int64_t) * F.off.size());
    return WMC_OK;
}
