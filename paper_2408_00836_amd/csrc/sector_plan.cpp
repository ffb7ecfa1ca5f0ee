// sector_plan.cpp -- clusters, orbits and LDS slots of the particle-number
// sector form.  Host only; no GPU calls.
#include <algorithm>
#include <cmath>
#include <string>

#include "sector_plan.hpp"

namespace hv {
namespace sec {

namespace {

int popc(uint32_t x) { return __builtin_popcount(x); }

struct Hop {
    int bond, i, j, slot;
};

// Hops of `todo` (in order) that a cluster can apply as two matchings: both
// sites inside, no earlier hop that shares a site left behind, and at most
// one earlier hop of the cluster on either site.  which: their indices and
// matchings (1, 2).
int closure(const std::vector<Hop> &todo, uint32_t S, std::vector<std::array<int, 2>> *which)
{
    uint32_t blocked = 0, used[2] = {0, 0};
    int cnt = 0;
    for (size_t h = 0; h < todo.size(); ++h) {
        const uint32_t b = (1u << todo[h].i) | (1u << todo[h].j);
        if ((b & ~S) || (b & blocked) || (b & used[1])) {
            blocked |= b;
            continue;
        }
        const int stage = (b & used[0]) ? 1 : 0;
        used[stage] |= b;
        if (stage == 1)
            used[0] |= b;
        ++cnt;
        if (which)
            which->push_back({(int)h, stage + 1});
    }
    return cnt;
}

// Phases of one layer's hops: repeatedly the four-site cluster that applies
// the most hops, among equals (the first kTies of them) the one that leaves
// the best next cluster.
void plan_clusters(const Model &m, SectorPlan &P)
{
    constexpr int kTies = 16;
    std::vector<Hop> todo;
    for (int s = 1; s <= m.ngroups; ++s)
        for (int k = 0; k < m.nb; ++k)
            if (m.slot[k] == s)
                todo.push_back({k, std::min(m.bi[k], m.bj[k]), std::max(m.bi[k], m.bj[k]), s});
    const int N = std::max(m.ns, 4);   // sites >= ns are never occupied
    std::vector<uint32_t> sets;
    for (int a = 0; a < N; ++a)
        for (int b = a + 1; b < N; ++b)
            for (int c = b + 1; c < N; ++c)
                for (int d = c + 1; d < N; ++d)
                    sets.push_back((1u << a) | (1u << b) | (1u << c) | (1u << d));
    auto best_of = [&](const std::vector<Hop> &t) {
        int best = 0;
        for (uint32_t S : sets)
            best = std::max(best, closure(t, S, nullptr));
        return best;
    };
    do {
        int best = -1;
        std::vector<uint32_t> ties;
        for (uint32_t S : sets) {
            const int c = closure(todo, S, nullptr);
            if (c > best) {
                best = c;
                ties.clear();
            }
            if (c == best && (int)ties.size() < kTies)
                ties.push_back(S);
        }
        auto without = [&](const std::vector<std::array<int, 2>> &w) {
            std::vector<Hop> left;
            for (size_t h = 0, k = 0; h < todo.size(); ++h)
                if (k < w.size() && w[k][0] == (int)h)
                    ++k;
                else
                    left.push_back(todo[h]);
            return left;
        };
        uint32_t pick = ties[0];
        int pick_next = -1;
        for (uint32_t S : ties) {
            std::vector<std::array<int, 2>> w;
            closure(todo, S, &w);
            const std::vector<Hop> left = without(w);
            const int nx = left.empty() ? 1 << 20 : best_of(left);
            if (nx > pick_next) {
                pick_next = nx;
                pick = S;
            }
        }
        std::vector<std::array<int, 2>> w;
        closure(todo, pick, &w);
        // name the sites so that the matchings are {01, 23} and {02, 13}
        std::array<int, 4> sites;
        for (int q = 0, k = 0; q < N; ++q)
            if ((pick >> q) & 1u)
                sites[k++] = q;
        std::array<int, 4> order = {0, 1, 2, 3}, bond = {-1, -1, -1, -1};
        for (bool found = false;; std::next_permutation(order.begin(), order.end())) {
            bond = {-1, -1, -1, -1};
            found = true;
            for (const auto &g : w) {
                int q = 2 * (g[1] - 1);
                const int end = q + 2;
                for (; q < end; ++q) {
                    const int a = sites[order[kPosA[q]]], b = sites[order[kPosB[q]]];
                    if (std::min(a, b) == todo[g[0]].i && std::max(a, b) == todo[g[0]].j)
                        break;
                }
                if (q == end) {
                    found = false;
                    break;
                }
                bond[q] = todo[g[0]].bond;
            }
            if (found)
                break;
        }
        P.sites.push_back({sites[order[0]], sites[order[1]], sites[order[2]], sites[order[3]]});
        P.bond.push_back(bond);
        // a position without a hop takes the slot of a hop of its phase; in the
        // one phase of a model without bonds there is none: slot 0, which is a
        // parameter (the layer has no other) but no group's, and nothing reduced
        int slot = 0;
        for (int q = 0; q < kPositions; ++q)
            if (bond[q] >= 0)
                slot = m.slot[bond[q]];
        for (int q = kPositions - 1; q >= 0; --q) {
            SecGate g{};
            if (bond[q] >= 0)
                slot = m.slot[bond[q]];
            g.slot = slot;
            g.t = bond[q] >= 0 ? m.t[bond[q]] : 0.0;
            P.gates.push_back(g);
        }
        std::reverse(P.gates.end() - kPositions, P.gates.end());
        for (int q = 0; q < kPositions; ++q) {
            SecGate *g = &P.gates[P.gates.size() - kPositions + q];
            g->last = g->slot > 0 && (q == 0 || g[-1].slot != g->slot);
        }
        todo = without(w);
    } while (!todo.empty());
}

// Orbits of a cluster with k electrons on it: the patterns outside it.
std::vector<uint32_t> orbits(const SpinPlan &S, int ns, const std::array<int, 4> &sites, int k)
{
    uint32_t cl = 0, low = 0;
    int real = 0;
    for (int q : sites)
        if (q < ns) {
            cl |= 1u << q;
            if (real++ < k)
                low |= 1u << q;
        }
    std::vector<uint32_t> out;
    if (k > real || S.n_el < k)
        return out;
    // every rest pattern appears once among the patterns whose k cluster
    // electrons sit on the same k sites
    for (uint32_t p : S.pat)
        if ((p & cl) == low)
            out.push_back(p & ~cl);
    return out;
}

// LDS bank class of a pattern: XOR of a per-site vector over its electrons.
// Linear, so that patterns that differ by a fixed set of sites differ by a
// fixed class: lanes whose orbits have different classes stay apart in every
// element of the orbit.
uint32_t class_of(uint32_t p, const uint32_t *v)
{
    uint32_t c = 0;
    for (; p; p &= p - 1u)
        c ^= v[__builtin_ctz(p)];
    return c;
}

// Deal a list into lanes so that every aligned group of M lanes holds M
// different classes as long as the classes last.
std::vector<uint32_t> deal(const std::vector<uint32_t> &list, int M, const uint32_t *v)
{
    std::vector<std::vector<uint32_t>> by(M);
    for (uint32_t r : list)
        by[class_of(r, v)].push_back(r);
    std::vector<size_t> at(M, 0);
    std::vector<uint32_t> out;
    for (size_t i = 0; i < list.size(); ++i) {
        int c = (int)(i % M);
        if (at[c] == by[c].size())
            for (int q = 0; q < M; ++q)
                if (by[q].size() - at[q] > by[c].size() - at[c])
                    c = q;
        out.push_back(by[c][at[c]++]);
    }
    return out;
}

// Rows of a workgroup (log2), threads and bank classes of short rows.
//   rows: as many as leave >= kMinGroups workgroups, at most kMaxWgT lanes per
//   list and kRowsLds bytes of rows (two workgroups per CU); at least one.
constexpr int kMinGroups = 60;
constexpr int kMaxWgT = 512;
constexpr int kRowsLds = 72 * 1024;

void shape(SpinPlan &S, int n_rows, int longest_list)
{
    S.lr = 0;
    while (S.lr < 4 && (n_rows >> (S.lr + 1)) >= kMinGroups &&
           (longest_list << (S.lr + 1)) <= kMaxWgT && ((S.n * 16) << (S.lr + 1)) <= kRowsLds)
        ++S.lr;
    const int lanes = std::max(1, longest_list << S.lr);
    S.threads = 2 * ((lanes + 63) / 64 * 64);   // a half for the orbits of six, one for the others
    S.classes = std::max(1, 16 >> S.lr);
}

void build_spin(const Model &m, SectorPlan &P, int s, int n_rows)
{
    SpinPlan &S = P.spin[s];
    const int ns = m.ns;
    S.is_long = S.n > kShortRow;
    int longest = 0;
    for (const auto &c : P.sites)
        for (int k = 1; k <= 3; ++k)
            longest = std::max(longest, (int)orbits(S, ns, c, k).size());
    if (S.is_long) {
        S.threads = kLongT;
        S.classes = 32;
    } else {
        shape(S, n_rows, longest);
    }
    const int M = S.classes;
    // class vectors: the best of a few pseudo-random choices (fewest slots,
    // then the most even orbit lists)
    uint32_t v[16], best_v[16] = {0};
    long best_score = -1;
    uint64_t rng = 0x9E3779B97F4A7C15ull;
    for (int tries = 0; tries < (M == 1 ? 1 : 24); ++tries) {
        for (int i = 0; i < 16; ++i) {
            rng = rng * 6364136223846793005ull + 1442695040888963407ull;
            v[i] = (uint32_t)(rng >> 40) & (uint32_t)(M - 1);
        }
        std::vector<int> cnt(M, 0);
        for (uint32_t p : S.pat)
            ++cnt[class_of(p, v)];
        long score = 64l * *std::max_element(cnt.begin(), cnt.end());
        for (const auto &c : P.sites)
            for (int k = 1; k <= 3; ++k) {
                const std::vector<uint32_t> o = orbits(S, ns, c, k);
                std::fill(cnt.begin(), cnt.end(), 0);
                for (uint32_t r : o)
                    ++cnt[class_of(r, v)];
                for (int q : cnt)
                    score += std::max(0, q - ((int)o.size() + M - 1) / M);
            }
        if (best_score < 0 || score < best_score) {
            best_score = score;
            std::copy(v, v + 16, best_v);
        }
    }
    // slots: class + M * (position within the class)
    std::vector<int> used(M, 0);
    std::vector<int> slot((size_t)S.n);
    for (int r = 0; r < S.n; ++r) {
        const int c = (int)class_of(S.pat[r], best_v);
        slot[r] = c + M * used[c]++;
    }
    S.nslots = M * *std::max_element(used.begin(), used.end());
    S.patslot.assign((size_t)S.nslots, 0);
    S.baseslot.assign((size_t)S.nslots, 0.0);
    std::vector<int> rank_at((size_t)S.nslots, -1);
    for (int r = 0; r < S.n; ++r) {
        S.patslot[slot[r]] = (uint16_t)S.pat[r];
        S.baseslot[slot[r]] = S.base[r];
        rank_at[slot[r]] = r;
    }
    if (S.is_long) {
        S.colslot.assign((size_t)2 * kLongT * 8, 0);
        for (int t = 0; t < kLongT; ++t)
            for (int j = 0; j < 16; ++j) {
                const int r = t + j * kLongT;
                S.colslot[long_index(t, j)] =
                    (uint16_t)(r < S.n ? slot[r] : S.nslots + t % kLongDummy);
            }
    } else {
        S.colslot.assign(slot.begin(), slot.end());
    }
    auto slot_of = [&](uint32_t p) -> int {   // -1: the pattern occupies a missing site
        return (p >> ns) ? -1 : slot[S.rank_of[p]];
    };
    static const int kPair[6][2] = {{0, 1}, {0, 2}, {0, 3}, {1, 2}, {1, 3}, {2, 3}};
    for (size_t ph = 0; ph < P.sites.size(); ++ph) {
        const std::array<int, 4> &c = P.sites[ph];
        uint32_t bit[4];
        for (int a = 0; a < 4; ++a)
            bit[a] = 1u << c[a];
        const uint32_t all = bit[0] | bit[1] | bit[2] | bit[3];
        auto flags = [&](int k, uint32_t r) {
            uint32_t f = 0;
            for (int q = 0; q < kPositions; ++q) {
                const int a = kPosA[q], b = kPosB[q];
                const uint32_t lo = std::min(bit[a], bit[b]), hi = std::max(bit[a], bit[b]);
                const uint32_t between = (hi - 1u) & ~(2u * lo - 1u);
                uint32_t others = 0;   // the two spectators
                for (int e = 0, i = 0; e < 4; ++e) {
                    if (e == a || e == b)
                        continue;
                    others |= bit[e];
                    if (k == 2)
                        f |= (uint32_t)(popc((r | bit[e]) & between) & 1) << (31 - (2 * q + i));
                    ++i;
                }
                if (k == 1)
                    f |= (uint32_t)(popc(r & between) & 1) << (23 - q);
                if (k == 3)
                    f |= (uint32_t)(popc((r | others) & between) & 1) << (19 - q);
            }
            return f;
        };
        auto element = [&](int k, uint32_t r, int e) -> uint32_t {
            return k == 2 ? (r | bit[kPair[e][0]] | bit[kPair[e][1]])
                          : (k == 1 ? (r | bit[e]) : (r | (all & ~bit[e])));
        };
        SecPhase D{};
        static const int kOrder[3] = {2, 1, 3};
        if (!S.is_long) {
            for (int l = 0; l < 3; ++l) {
                const int k = kOrder[l];
                const std::vector<uint32_t> o = deal(orbits(S, ns, c, k), M, best_v);
                D.n[l] = (int)o.size();
                for (uint32_t r : o) {
                    uint16_t e[8] = {0};
                    for (int i = 0; i < (k == 2 ? 6 : 4); ++i) {
                        const int sl = slot_of(element(k, r, i));
                        e[i] = (uint16_t)((sl < 0 ? S.nslots : sl) << S.lr);
                    }
                    Rec R;
                    for (int i = 0; i < 4; ++i)
                        R.w[i] = (uint32_t)e[2 * i] | ((uint32_t)e[2 * i + 1] << 16);
                    R.w[k == 2 ? 3 : 2] = flags(k, r) | 1u;
                    S.recs.push_back(R);
                }
                // the lanes without an orbit read the zero slot
                const uint32_t z = (uint32_t)(S.nslots << S.lr);
                Rec none = {{z | z << 16, z | z << 16, k == 2 ? z | z << 16 : 0, 0}};
                for (int i = D.n[l]; i < (S.threads / 2) >> S.lr; ++i)
                    S.recs.push_back(none);
            }
        } else {
            const size_t at = S.lcode.size();
            S.lcode.resize(at + (size_t)kLongT * 8);
            std::vector<uint16_t> el((size_t)kLongT * 16);
            std::vector<uint16_t> pt((size_t)kLongT * 16, 0);
            for (int t = 0; t < kLongT; ++t)
                for (int j = 0; j < 16; ++j)
                    el[(size_t)t * 16 + j] =
                        (uint16_t)(j < kOrbitElems ? S.nslots + t % kLongDummy : 0);
            static const int kAt[3] = {0, 6, 10};
            for (int l = 0; l < 3; ++l) {
                const int k = kOrder[l];
                const std::vector<uint32_t> o = deal(orbits(S, ns, c, k), M, best_v);
                D.n[l] = (int)o.size();
                for (size_t t = 0; t < o.size(); ++t) {
                    el[t * 16 + 15] |= (uint16_t)(flags(k, o[t]) >> 16);
                    for (int i = 0; i < (k == 2 ? 6 : 4); ++i) {
                        const uint32_t p = element(k, o[t], i);
                        el[t * 16 + kAt[l] + i] = (uint16_t)slot_of(p);
                        pt[t * 16 + kAt[l] + i] = (uint16_t)p;
                    }
                }
            }
            std::vector<uint32_t> one = orbits(S, ns, c, 0);   // singles: all empty, all full
            for (uint32_t r : orbits(S, ns, c, 4))
                one.push_back(r | all);
            one = deal(one, M, best_v);
            for (size_t t = 0; t < one.size(); ++t) {
                el[t * 16 + 14] = (uint16_t)slot_of(one[t]);
                pt[t * 16 + 14] = (uint16_t)one[t];
            }
            for (int t = 0; t < kLongT; ++t)
                for (int i = 0; i < 8; ++i)
                    S.lcode[at + (size_t)t * 8 + i] =
                        (uint32_t)el[(size_t)t * 16 + 2 * i] |
                        ((uint32_t)el[(size_t)t * 16 + 2 * i + 1] << 16);
            if (ph == 0) {
                S.lpat.resize((size_t)kLongT * 8);
                S.lbase.assign((size_t)kOrbitElems * kLongT, 0.0);
                for (int t = 0; t < kLongT; ++t) {
                    for (int i = 0; i < 8; ++i)
                        S.lpat[(size_t)t * 8 + i] =
                            (uint32_t)pt[(size_t)t * 16 + 2 * i] |
                            ((uint32_t)pt[(size_t)t * 16 + 2 * i + 1] << 16);
                    for (int j = 0; j < kOrbitElems; ++j) {
                        const int sl = el[(size_t)t * 16 + j];
                        S.lbase[(size_t)j * kLongT + t] = sl < S.nslots ? S.baseslot[sl] : 0.0;
                    }
                }
            }
        }
        S.phases.push_back(D);
    }
    // H: for every bond the slot of the partner pattern and the hop's sign
    // (an inactive element: the zero slot nslots).  Short rows: per rank,
    // ham_bonds(nb) codes; long rows: per bond, element t + j kLongT counted
    // by slots, at long_index, the signs apart: bit 31 - j of the dword that
    // the thread's codes 14 and 15 make.
    const int hb = ham_bonds(m.nb);
    auto code = [&](int r, int k) -> uint16_t {
        if (r < 0)
            return (uint16_t)S.nslots;
        const int i = std::min(m.bi[k], m.bj[k]), j = std::max(m.bi[k], m.bj[k]);
        const uint32_t p = S.pat[r];
        if (!(((p >> i) ^ (p >> j)) & 1u))
            return (uint16_t)S.nslots;
        const uint32_t between = ((1u << j) - 1u) & ~((2u << i) - 1u);
        return (uint16_t)(slot[S.rank_of[p ^ ((1u << i) | (1u << j))]] |
                          ((popc(p & between) & 1) << 15));
    };
    if (!S.is_long) {
        S.hcode.assign((size_t)S.n * hb, (uint16_t)S.nslots);
        for (int r = 0; r < S.n; ++r)
            for (int k = 0; k < m.nb; ++k)
                S.hcode[(size_t)r * hb + k] = code(r, k);
    } else {
        const size_t per = (size_t)2 * kLongT * 8;
        S.hcode.assign(per * std::max(1, m.nb), (uint16_t)S.nslots);
        for (int k = 0; k < m.nb; ++k)
            for (int t = 0; t < kLongT; ++t) {
                uint32_t signs = 0;
                for (int j = 0; j < kLongElems; ++j) {
                    const int e = t + j * kLongT;
                    if (e < S.nslots) {
                        const uint16_t c = code(rank_at[e], P.ham_order[k]);
                        S.hcode[per * k + long_index(t, j)] = c & 0x7FFFu;
                        signs |= (uint32_t)(c >> 15) << (31 - j);
                    }
                }
                S.hcode[per * k + long_index(t, 14)] = (uint16_t)signs;
                S.hcode[per * k + long_index(t, 15)] = (uint16_t)(signs >> 16);
            }
    }
}

// m of the reverse sweep's vectors chi = lambda / m -+ i m psi: a power of two
// near the square root of |H psi| / |psi|.  The rounding of <chi2|G|chi2> -
// <chi1|G|chi1> grows with |lambda|^2 / m^2 + m^2 |psi|^2, which is least there.
// |H psi|^2 of an evenly filled state: t^2 for every bond and spin that moves an
// electron, and the sector's mean of D^2.  (The mean of D in D^2's place vanishes
// for a staggered potential and for eps against U: m = 2 instead of 32 for eps =
// +-1000, and the gradient's error was ten to thirty times that of Im
// <lambda|G|psi> summed directly; with D^2 the two are alike.)
double mix_scale(const Model &m, const SectorPlan &P)
{
    const SpinPlan &X = P.spin[0], &Y = P.spin[1];
    const int ns = m.ns;
    // the probability that two sites hold two electrons, or one
    auto two = [ns](double n) { return ns > 1 ? n * (n - 1.0) / (ns * (ns - 1.0)) : 0.0; };
    auto one = [ns](double n) { return ns > 1 ? 2.0 * n * (ns - n) / (ns * (ns - 1.0)) : 0.0; };
    double norm2 = 0.0;
    for (int k = 0; k < m.nb; ++k)
        norm2 += m.t[k] * m.t[k] * (one(X.n_el) + one(Y.n_el));
    // D = A(p) + A(q) + sum_j p_j w_j(q), p and q the two spins' patterns: the mean
    // over p of the square from A's and the p_j's moments, then over q
    double a1 = 0.0, a2 = 0.0, ap[16] = {0.0};
    for (int r = 0; r < X.n; ++r) {
        a1 += X.base[r] / X.n;
        a2 += X.base[r] * X.base[r] / X.n;
        for (int i = 0; i < ns; ++i)
            ap[i] += (X.pat[r] >> i) & 1u ? X.base[r] / X.n : 0.0;
    }
    const double p1 = (double)X.n_el / ns, p2 = two(X.n_el);
    for (int r = 0; r < Y.n; ++r) {
        const double b = Y.base[r];
        double sum = 0.0, sq = 0.0, aw = 0.0;
        for (int i = 0; i < ns; ++i) {
            const double w = m.general ? Y.wrow[(size_t)r * 16 + i]
                                       : ((Y.pat[r] >> i) & 1u ? m.U : 0.0);
            sum += w;
            sq += w * w;
            aw += w * ap[i];
        }
        norm2 += (a2 + b * b + sq * p1 + (sum * sum - sq) * p2 +
                  2.0 * (a1 * b + aw + b * sum * p1)) / Y.n;
    }
    const double norm = std::sqrt(norm2);
    if (!(norm > 0.0) || !std::isfinite(norm))
        return 1.0;
    return std::ldexp(1.0, std::max(-64, std::min(64, (int)std::lround(0.5 * std::log2(norm)))));
}

}  // namespace

std::string plan_sector(const Model &m, SectorPlan &P)
{
    const int ns = m.ns;
    const uint32_t smask = (1u << ns) - 1u;
    const uint32_t start[2] = {(uint32_t)m.neel & smask, (uint32_t)(m.neel >> ns) & smask};
    for (int s = 0; s < 2; ++s) {
        SpinPlan &S = P.spin[s];
        S.n_el = popc(start[s]);
        S.rank_of.assign((size_t)1 << ns, -1);
        for (uint32_t p = 0; p <= smask; ++p) {
            if (popc(p) != S.n_el)
                continue;
            S.rank_of[p] = (int32_t)S.pat.size();
            S.pat.push_back(p);
            double b = 0.0;
            for (int i = 0; i < ns; ++i)
                if ((p >> i) & 1u)
                    b += m.eps[i];
            for (int k = 0; k < m.nb; ++k)
                if (((p >> m.bi[k]) & 1u) && ((p >> m.bj[k]) & 1u))
                    b += m.V[k];
            S.base.push_back(b);
            if (m.general) {
                double w[16] = {0.0};
                for (int i = 0; i < ns; ++i)
                    if ((p >> i) & 1u)
                        w[i] += m.U;
                for (int k = 0; k < m.nb; ++k) {
                    if ((p >> m.bi[k]) & 1u)
                        w[m.bj[k]] += m.V[k];
                    if ((p >> m.bj[k]) & 1u)
                        w[m.bi[k]] += m.V[k];
                }
                S.wrow.insert(S.wrow.end(), w, w + 16);
            }
        }
        S.n = (int)S.pat.size();
        if (S.n > kMaxRows)
            return "sector rows longer than 13 x 1024";
    }
    plan_clusters(m, P);
    for (int k = 0; k < m.nb; ++k)
        P.ham_order.push_back(k);
    if (P.spin[0].n > kShortRow)
        P.n_flat = (int)(std::stable_partition(P.ham_order.begin(), P.ham_order.end(),
                                               [&](int k) {
                                                   return std::abs(m.bi[k] - m.bj[k]) == 1;
                                               }) -
                         P.ham_order.begin());
    for (int s = 0; s < 2; ++s) {
        if (s == 1 && P.spin[1].n_el == P.spin[0].n_el) {   // the same rows
            P.spin[1] = P.spin[0];
            break;
        }
        build_spin(m, P, s, P.spin[1 - s].n);
        SpinPlan &S = P.spin[s];
        if (S.is_long && S.nslots > kMaxRows)
            return "sector row slots exceed 13 x 1024";
    }
    P.mix = mix_scale(m, P);
    return "";
}

}  // namespace sec
}  // namespace hv
