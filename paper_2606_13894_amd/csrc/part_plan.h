// Plan of block inference (Sec. 5.1, Alg. 2): which sums of z = log(g^2 + eps) each divisor
// p of a tensor's n elements is formed from. Plain C++ with no HIP types, so that a host
// test can run every plan on the CPU.
//
// S(p) needs the n / p sums of z over blocks of p. A divisor's sums are sums of a smaller
// divisor's sums, so z is not evaluated once per divisor:
//  - the base pass reads the gradient once, chunk by chunk of at most kPartChunkMax elements,
//    chunks being whole blocks of one divisor L of n, and forms the sums of every divisor of
//    L in LDS (each from its largest proper divisor), their contrasts inside the chunk and
//    first and last sum of the workgroup's run of chunks for the contrasts across runs. It
//    stores the sums that later nodes read. The work on a chunk is cut into units of one
//    wave, in phases with a barrier between: phase d forms the sums of the divisors of d
//    prime factors and takes the contrasts of those of d - 1;
//  - a node forms the sums of a divisor p that does not divide L from those of gcd(p, L)
//    when that is at least kPartDirectGcd, else from p / (smallest prime of p); when that is
//    1, from the gradient itself (a prime of n that L lacks): up to kPartDirectMax all in one
//    second pass, which takes a span of elements and two blocks beyond into LDS, as z, and
//    sums and contrasts there the blocks that begin in the span. A sum over more than kPartSub
//    terms goes through sub-sums of kPartSub terms, so that a huge block spreads over many
//    workgroups;
//  - a node's contrasts are taken one launch later, when its sums are complete.
// L is the divisor with the least left to do (part_base). The launches are numbered: 0 the
// base pass and the nodes read from the gradient, then each node after its source.
//
// Memory. Stored sums are 8 / p bytes an element, so those of small divisors exceed the
// gradient itself. A plan's stored sums stay within part_budget, a fraction of what the
// optimizer's state takes anyway: a tensor that would exceed it alone gets a least divisor
// `least` whose sums may be stored; smaller ones that then have no stored source join the
// second pass. `least` is 1 wherever everything fits. Tensors that fit one by one but not
// together go into several plans, run one after another in the same memory (part_plans).
// (All sums of all tensors at once took 2.9 GB for the 1.5e9 elements of a model with
// 128256 x 2048 embeddings, twice its optimizer state.)
#pragma once

#include <stdint.h>

#include <algorithm>
#include <bitset>
#include <limits>
#include <map>
#include <numeric>
#include <vector>

namespace gefen {

constexpr int kPartThreads = 512;       // base pass
constexpr int kPartChunkMax = 2048;     // elements of a base chunk, and the largest L
constexpr int kPartMaxEntry = 40;       // most divisors of a number up to kPartChunkMax (1680)
constexpr int kPartRun = 8;             // most chunks of one workgroup of the base pass
constexpr int64_t kPartGroups = 4096;   // workgroups below which runs are shorter
constexpr int kPartUnit = 512;          // sums (or contrasts) of one unit
constexpr int kPartMaxUnit = 160;       // most units of a tensor (1680: 126)
constexpr int kPartMaxPhase = 16;       // most phases (2048: 11 prime factors, 13 phases)
constexpr int64_t kPartDirectGcd = 32;
constexpr int64_t kPartSub = 4096;      // terms of one sub-sum
constexpr int64_t kPartItem = 4096;     // terms one node work item adds, if its blocks are short
constexpr int64_t kPartPairs = 2048;    // contrasts per work item
constexpr int kPartSpan = 4096;         // elements of a direct item
constexpr int64_t kPartDirectMax = 1023;   // largest direct divisor
constexpr int64_t kPartLeastMax = 512;  // largest `least`
constexpr int kPartDirectThreads = 512;
constexpr int64_t kPartBudgetMin = int64_t(64) << 20;

// A unit of a chunk's work. The sums of an entry (a divisor of L) lie at one place of the
// chunk's LDS, `n` of them in a whole chunk (len / p in a tensor's last one).
//  PART_ADD   sums i0 .. of divisor p at dst, q consecutive ones at src each
//  PART_GAP   contrasts of the sums at src from i0 on; with i0 = 0 also the run's first and
//             last sum of entry `entry`. `slot` numbers the GAP units.
//  PART_KEEP  the sums from i0 on to the sums buffer, at the place keep[slot]
enum : uint16_t { PART_ADD = 0, PART_GAP = 1, PART_KEEP = 2 };
struct PartUnit {
    uint16_t kind, p, q, src, dst, i0, n, slot;
};
static_assert(sizeof(PartUnit) == 16, "PartUnit layout");

// A tensor in the base pass: nchunk chunks of `chunk` elements, `run` to a workgroup,
// workgroups ngroup from group0 on. Its units run from unit0 in nphase phases, phase f ends
// before unit phase_end[phase0 + f]. GAP unit s of workgroup w writes its contrasts to
// part[out0 + s * ngroup + w]; entry e's first sum goes to part[out0 + (ngap + e) * ngroup +
// w], its last one nentry * ngroup further on.
struct PartTensor {
    const void* grad;
    int64_t n;
    int64_t group0, nchunk, ngroup, out0;
    int32_t gdtype, chunk, run, unit0, nunit, phase0, nphase, keep0, ngap, nentry;
};

// The direct divisors of a tensor (formed in the second pass), direct[first .. first + count)
// rising: item it takes the blocks that begin in the elements [it kPartSpan, + kPartSpan) and
// writes the contrasts with the block after each, of divisor d, to part[out + d * n_items +
// it], and the sums to the place store[store0 + d] (-1: nowhere).
struct PartSpan {
    int64_t item0, n_items, out;
    int32_t tensor, first, count, store0;
};

// Work of one launch. SUM: block i = the sum of terms [i q, (i + 1) q) of the source, item
// it takes blocks [it per, + per). SUB: sub-sums, item it = block it / sub, terms from
// (it % sub) kPartSub on. DIFF: contrasts of the sums at src, item it takes the pairs
// [it per, + per) and writes part[dst + it].
enum : int32_t { PART_SUM = 0, PART_SUB = 1, PART_DIFF = 2 };
struct PartJob {
    int64_t item0, n_items;
    int64_t src;          // in the sums buffer; -1: z of tensor `tensor`
    int64_t dst;
    int64_t q, count;     // terms per block; blocks (SUM, SUB) or sums (DIFF)
    int64_t per;
    int32_t kind, tensor, sub, pad;
};

// The score of one (tensor, divisor), in tensor order, divisors rising: the contrasts at
// part[out .. out + terms), and those across `runs` runs, whose first and last sums are at
// `firsts` and `lasts`.
struct PartScore {
    int64_t p, nb, out, terms, runs, firsts, lasts;
};

// What depends on n alone, shared by the tensors of one size: the divisors, L, the base
// pass's units (in the plan's tables) and how each divisor's sums are formed.
struct PartShape {
    struct Div {
        int64_t p, nb;           // nb: its blocks, n / p
        int32_t spf, parent;     // indices of its smallest prime and of p over that
        int32_t source;          // index of the divisor its sums are formed from (-1: gradient)
        int32_t entry;           // index among the divisors of L, or -1
        int32_t gap0, gaps;      // entry: its GAP units
        int32_t keep;            // entry: its KEEP slot, or -1
        int32_t direct;          // index among the direct divisors, or -1
    };
    std::vector<Div> divs;
    int64_t L = 1, least = 1;
    int64_t stored = 0;              // doubles of a tensor's sums
    int32_t direct0 = 0, ndirect = 0;
    int32_t chunk = 0, unit0 = 0, nunit = 0, phase0 = 0, nphase = 0, ngap = 0, nentry = 0,
            nkeep = 0;
};

struct PartPlan {
    std::map<int64_t, PartShape> shapes;   // by n
    std::vector<PartTensor> tensors;
    std::vector<PartUnit> units;
    std::vector<int32_t> phase_end;
    std::vector<int64_t> keep;
    std::vector<int32_t> direct;
    std::vector<PartSpan> spans;
    std::vector<int64_t> store;
    std::vector<std::vector<PartJob>> launches;   // [0] runs beside the base pass
    std::vector<PartScore> scores;
    std::vector<int32_t> first, count;            // per tensor: its scores
    int64_t groups = 0, sums = 0, parts = 0, span_items = 0;
    int32_t lds_doubles = 0, direct_max = 0;      // the largest direct divisor
};

inline std::vector<int64_t> part_divisors(int64_t n)
{
    std::vector<int64_t> lo, hi;
    for (int64_t d = 1; d <= n / d; ++d) {
        if (n % d == 0) {
            lo.push_back(d);
            if (d != n / d) hi.push_back(n / d);
        }
    }
    for (auto it = hi.rbegin(); it != hi.rend(); ++it) lo.push_back(*it);
    return lo;
}

// Bytes that a plan over `total` elements may store: half a byte an element, what the state's
// 4-bit codes take afterwards, and 64 MiB (no size up to 4e6 elements needs more with
// everything stored).
inline int64_t part_budget(int64_t total) { return kPartBudgetMin + total / 2; }

// The divisor whose sums those of d (not a divisor of L; g = gcd(d.p, L)) are formed from; 1:
// the gradient.
inline int64_t part_source(const PartShape::Div& d, int64_t g, int64_t least, int64_t parent)
{
    if (g >= std::max(kPartDirectGcd, least)) return g;
    return d.spf && parent >= least ? parent : 1;
}

// What base divisor L and `least` come to: the doubles that a tensor stores (the sums of the
// sources among L's divisors and of the nodes, with sub-sums) and the cost in terms an
// element, those that the nodes add, a term read from the gradient (a float64 logarithm)
// counting as eight and a direct divisor's, in LDS, as a half. False as soon as they exceed
// `most` or reach `limit` (the small divisors, first, take most of both).
inline bool part_price(const std::vector<PartShape::Div>& divs, int64_t L, int64_t least,
                       int64_t most, double limit, int64_t& stored, double& cost,
                       std::vector<uint32_t>& gcd)
{
    const int64_t n = divs.back().p;
    const uint32_t l = static_cast<uint32_t>(L);
    std::bitset<kPartChunkMax + 1> kept;
    bool direct = false;
    stored = 0;
    cost = 0.0;
    gcd.resize(divs.size());
    gcd[0] = 1;
    for (size_t i = 1; i + 1 < divs.size(); ++i) {
        const PartShape::Div& d = divs[i];
        // gcd(q p', L), q prime, from gcd(p', L)
        const int64_t q = divs[d.spf].p;
        uint32_t g = gcd[d.parent];
        if (q <= L && l / g % static_cast<uint32_t>(q) == 0) g *= static_cast<uint32_t>(q);
        gcd[i] = g;
        if (g == d.p) continue;   // a divisor of L
        const int64_t src = part_source(d, g, least, divs[d.parent].p);
        const bool entry = src > 1 && (src == g || gcd[d.parent] == src);
        if (entry && !kept[src]) {
            kept[src] = true;
            stored += n / src;
        }
        if (src > 1 || d.p >= least) stored += d.nb;
        if (d.p > kPartSub * src)
            stored += d.nb * ((d.p / src + kPartSub - 1) / kPartSub);
        if (src == 1 && d.p <= kPartDirectMax) {
            cost += direct ? 0.5 : 8.5;
            direct = true;
        } else {
            cost += (src == 1 ? 8.0 : 1.0) / static_cast<double>(src);
        }
        if (stored > most || cost >= limit) return false;
    }
    return stored <= most && cost < limit;
}

// L: the divisor up to kPartChunkMax with the lowest cost, ties the largest, of those whose
// sums fit `budget` and that cost less than `cost`, which becomes theirs; 0 if there is none.
inline int64_t part_base(const std::vector<PartShape::Div>& divs, int64_t least, int64_t budget,
                         double& cost, int64_t& stored)
{
    std::vector<uint32_t> gcd;
    int64_t best = 0;
    for (size_t li = divs.size(); li-- > 0;) {
        double c;
        int64_t s;
        if (divs[li].p > kPartChunkMax ||
            !part_price(divs, divs[li].p, least, budget / 8, cost, s, c, gcd))
            continue;
        best = divs[li].p;
        cost = c;
        stored = s;
    }
    return best;
}

// `budget`: bytes that a tensor may store.
inline const PartShape& part_shape(PartPlan& P, int64_t n, int64_t budget)
{
    auto it = P.shapes.find(n);
    if (it != P.shapes.end()) return it->second;
    PartShape& s = P.shapes[n];
    for (int64_t p : part_divisors(n)) s.divs.push_back(PartShape::Div{p, n / p, 0, 0, -1, -1, 0, 0, -1, -1});
    auto index = [&](int64_t p) {
        auto f = std::lower_bound(s.divs.begin(), s.divs.end(), p,
                                  [](const PartShape::Div& d, int64_t v) { return d.p < v; });
        return static_cast<int32_t>(f - s.divs.begin());
    };
    for (PartShape::Div& d : s.divs)   // the smallest divisor of n above 1 that divides p
        if (d.p > 1) {
            for (d.spf = 1; d.p % s.divs[d.spf].p; ++d.spf) {}
            d.parent = index(d.p / s.divs[d.spf].p);
        }
    constexpr double kNone = std::numeric_limits<double>::infinity();
    double cost = kNone;
    s.L = part_base(s.divs, 1, INT64_MAX, cost, s.stored);
    if (8 * s.stored > budget) {
        cost = kNone;
        for (int64_t least = 1; least <= kPartLeastMax; least = std::max(4 * least, kPartDirectGcd)) {
            double c = 0.95 * cost;   // (one that saves little makes longer chains of nodes)
            int64_t stored;
            const int64_t L = part_base(s.divs, least, budget, c, stored);
            if (!L) continue;
            s.L = L;
            s.least = least;
            s.stored = stored;
            cost = c;
        }
        if (cost == kNone) {   // nothing fits: store as little as there is
            s.least = kPartLeastMax;
            s.L = part_base(s.divs, s.least, INT64_MAX, cost, s.stored);
        }
    }
    s.chunk = static_cast<int32_t>(s.L * std::max<int64_t>(1, kPartChunkMax / s.L));
    // the entries: the divisors of L below n (n = 1: 1)
    struct Entry {
        int32_t div, depth, lds, n;
    };
    std::vector<Entry> entries;
    int32_t lds = 0, deepest = 0;
    for (size_t i = 0; i < s.divs.size(); ++i) {
        PartShape::Div& d = s.divs[i];
        if (s.L % d.p || (d.p == n && n > 1)) continue;
        Entry e{static_cast<int32_t>(i), 0, lds, static_cast<int32_t>(s.chunk / d.p)};
        if (d.p > 1) e.depth = entries[s.divs[d.parent].entry].depth + 1;
        d.entry = static_cast<int32_t>(entries.size());
        lds += e.n;
        deepest = std::max(deepest, e.depth);
        entries.push_back(e);
    }
    P.lds_doubles = std::max(P.lds_doubles, lds);
    s.nentry = static_cast<int32_t>(entries.size());
    for (PartShape::Div& d : s.divs) {   // the nodes' sources; the entries they read are kept
        if (d.p == n || d.entry >= 0) continue;
        const int64_t src = part_source(d, std::gcd(d.p, s.L), s.least, s.divs[d.parent].p);
        if (src == 1 && d.p <= kPartDirectMax) {
            if (!s.ndirect) s.direct0 = static_cast<int32_t>(P.direct.size());
            d.direct = s.ndirect++;
            P.direct.push_back(static_cast<int32_t>(d.p));
            P.direct_max = std::max(P.direct_max, static_cast<int32_t>(d.p));
        }
        if (src == 1) continue;
        d.source = index(src);
        PartShape::Div& e = s.divs[d.source];
        if (e.entry >= 0 && e.keep < 0) e.keep = s.nkeep++;
    }
    s.unit0 = static_cast<int32_t>(P.units.size());
    s.phase0 = static_cast<int32_t>(P.phase_end.size());
    s.nphase = deepest + 2;   // phase 0 is empty: the logarithms
    for (int32_t f = 0; f < s.nphase; ++f) {
        for (const Entry& e : entries) {
            PartShape::Div& d = s.divs[e.div];
            PartUnit u{};
            u.p = static_cast<uint16_t>(d.p);
            u.n = static_cast<uint16_t>(e.n);
            if (d.p > 1 && e.depth == f) {
                u.kind = PART_ADD;
                u.q = static_cast<uint16_t>(s.divs[d.spf].p);
                u.src = static_cast<uint16_t>(entries[s.divs[d.parent].entry].lds);
                u.dst = static_cast<uint16_t>(e.lds);
                for (int32_t i = 0; i < e.n; i += kPartUnit) {
                    u.i0 = static_cast<uint16_t>(i);
                    P.units.push_back(u);
                }
            }
            if (e.depth != f - 1) continue;
            u.kind = PART_GAP;
            u.src = static_cast<uint16_t>(e.lds);
            u.dst = static_cast<uint16_t>(d.entry);
            d.gap0 = s.ngap;
            for (int32_t i = 0; i + 1 < std::max(e.n, 2); i += kPartUnit) {
                u.i0 = static_cast<uint16_t>(i);
                u.slot = static_cast<uint16_t>(s.ngap++);
                P.units.push_back(u);
            }
            d.gaps = s.ngap - d.gap0;
            if (d.keep < 0) continue;
            u.kind = PART_KEEP;
            u.slot = static_cast<uint16_t>(d.keep);
            for (int32_t i = 0; i < e.n; i += kPartUnit) {
                u.i0 = static_cast<uint16_t>(i);
                P.units.push_back(u);
            }
        }
        P.phase_end.push_back(static_cast<int32_t>(P.units.size()) - s.unit0);
    }
    s.nunit = static_cast<int32_t>(P.units.size()) - s.unit0;
    return s;
}

// Adds one tensor; `total`: the elements of all the plan's tensors, `budget`: bytes that they
// may store.
inline void part_add(PartPlan& P, const void* grad, int64_t n, int32_t gdtype, int64_t total,
                     int64_t budget)
{
    const PartShape& s = part_shape(P, n, budget);
    const int32_t tensor = static_cast<int32_t>(P.tensors.size());
    auto take = [&](int64_t count) {   // room for `count` sums
        const int64_t a = P.sums;
        P.sums += count;
        return a;
    };
    PartTensor t{};
    t.grad = grad;
    t.n = n;
    t.gdtype = gdtype;
    t.chunk = s.chunk;
    t.run = static_cast<int32_t>(std::max<int64_t>(
        1, std::min<int64_t>(kPartRun, total / t.chunk / kPartGroups)));
    t.nchunk = (n + t.chunk - 1) / t.chunk;
    t.group0 = P.groups;
    t.ngroup = (t.nchunk + t.run - 1) / t.run;
    P.groups += t.ngroup;
    t.unit0 = s.unit0;
    t.nunit = s.nunit;
    t.phase0 = s.phase0;
    t.nphase = s.nphase;
    t.ngap = s.ngap;
    t.nentry = s.nentry;
    t.keep0 = static_cast<int32_t>(P.keep.size());
    P.keep.resize(P.keep.size() + s.nkeep);
    for (const PartShape::Div& d : s.divs)
        if (d.keep >= 0) P.keep[t.keep0 + d.keep] = take(n / d.p);
    t.out0 = P.parts;
    P.parts += (t.ngap + 2 * t.nentry) * t.ngroup;
    P.tensors.push_back(t);

    PartSpan span{};
    if (s.ndirect) {
        span.item0 = P.span_items;
        span.n_items = (n + kPartSpan - 1) / kPartSpan;
        span.out = P.parts;
        span.tensor = tensor;
        span.first = s.direct0;
        span.count = s.ndirect;
        span.store0 = static_cast<int32_t>(P.store.size());
        P.span_items += span.n_items;
        P.parts += s.ndirect * span.n_items;
        P.spans.push_back(span);
    }

    // per divisor: where its stored sums are and which launch completes them
    struct Node {
        int64_t at;
        int32_t ready;
    };
    std::vector<Node> nodes(s.divs.size(), Node{0, 0});
    auto job = [&](int32_t launch, const PartJob& j) {
        if (static_cast<int32_t>(P.launches.size()) <= launch) P.launches.resize(launch + 1);
        P.launches[launch].push_back(j);
    };
    P.first.push_back(static_cast<int32_t>(P.scores.size()));
    P.count.push_back(static_cast<int32_t>(s.divs.size()));
    for (size_t i = 0; i < s.divs.size(); ++i) {
        const PartShape::Div& d = s.divs[i];
        const int64_t p = d.p, nb = n / p;
        PartScore sc{p, nb, 0, 0, 0, 0, 0};
        if (p == n) {
            P.scores.push_back(sc);   // one block: 0 by definition
            continue;
        }
        if (d.entry >= 0) {
            sc.out = t.out0 + d.gap0 * t.ngroup;
            sc.terms = d.gaps * t.ngroup;
            sc.runs = t.ngroup;
            sc.firsts = t.out0 + (t.ngap + d.entry) * t.ngroup;
            sc.lasts = sc.firsts + t.nentry * t.ngroup;
            P.scores.push_back(sc);
            if (d.keep >= 0) nodes[i] = Node{P.keep[t.keep0 + d.keep], 0};
            continue;
        }
        if (d.direct >= 0) {
            P.store.push_back(p < s.least ? -1 : take(nb));
            nodes[i] = Node{P.store.back(), 0};
            sc.out = span.out + d.direct * span.n_items;
            sc.terms = span.n_items;
            P.scores.push_back(sc);
            continue;
        }
        PartJob j{};
        j.tensor = tensor;
        j.src = d.source < 0 ? -1 : nodes[d.source].at;
        j.q = d.source < 0 ? p : p / s.divs[d.source].p;
        j.count = nb;
        int32_t launch = d.source < 0 ? 0 : nodes[d.source].ready + 1;
        if (j.q > kPartSub) {   // sub-sums first
            j.kind = PART_SUB;
            j.sub = static_cast<int32_t>((j.q + kPartSub - 1) / kPartSub);
            j.n_items = nb * j.sub;
            j.dst = take(j.n_items);
            j.per = 1;
            job(launch, j);
            PartJob c{};
            c.tensor = tensor;
            c.src = j.dst;
            c.q = j.sub;
            c.count = nb;
            j = c;
            ++launch;
        }
        j.kind = PART_SUM;
        j.dst = take(nb);
        j.per = std::max<int64_t>(1, kPartItem / j.q);
        j.n_items = (nb + j.per - 1) / j.per;
        job(launch, j);
        nodes[i] = Node{j.dst, launch};
        PartJob f{};
        f.tensor = tensor;
        f.kind = PART_DIFF;
        f.src = j.dst;
        f.count = nb;
        f.per = kPartPairs;
        f.n_items = (nb - 1 + f.per - 1) / f.per;
        f.dst = P.parts;
        P.parts += f.n_items;
        job(launch + 1, f);
        sc.out = f.dst;
        sc.terms = f.n_items;
        P.scores.push_back(sc);
    }
}

// Numbers the work items of every launch (after the last part_add).
inline void part_finish(PartPlan& P)
{
    for (auto& l : P.launches) {
        int64_t items = 0;
        for (PartJob& j : l) {
            j.item0 = items;
            items += j.n_items;
        }
    }
}

// The plans of a list of tensors, in their order: one if the budget holds all their sums.
struct PartInput {
    const void* grad;
    int64_t n;
    int32_t gdtype;
};

inline std::vector<PartPlan> part_plans(const std::vector<PartInput>& in, int64_t budget)
{
    PartPlan shapes;   // the tables that all plans share
    for (const PartInput& t : in) part_shape(shapes, t.n, budget);
    std::vector<PartPlan> plans;
    for (size_t a = 0, b = 0; a < in.size(); a = b) {
        int64_t stored = 0, elems = 0;
        for (; b < in.size(); ++b) {
            stored += 8 * shapes.shapes.at(in[b].n).stored;
            if (b > a && stored > budget) break;
            elems += in[b].n;
        }
        PartPlan P = a == 0 && b == in.size() ? std::move(shapes) : shapes;
        for (size_t i = a; i < b; ++i)
            part_add(P, in[i].grad, in[i].n, in[i].gdtype, elems, budget);
        part_finish(P);
        plans.push_back(std::move(P));
    }
    return plans;
}

}  // namespace gefen
