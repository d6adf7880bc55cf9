// Runs the plan of block inference (part_plan.h) on the CPU, term by term as the kernels
// index it, and compares every score with the definition (z evaluated once per divisor).
// Usage: part_plan_check n [n ...]   -- one plan over tensors of these sizes; with PART_BUDGET
// the plans that store at most so many bytes at a time.
#include <cmath>
#include <cstdio>
#include <cstdlib>
#include <random>

#include "part_plan.h"

using namespace gefen;

// Plan P over tensors whose z are `z`.
int check(const PartPlan& P, const std::vector<std::vector<double>>& z)
{
    const double unset = std::nan("");
    std::vector<double> sums(P.sums, unset), part(P.parts, unset);
    int64_t written = 0;
    auto put = [&](std::vector<double>& v, int64_t i, double x) {
        if (!std::isnan(v.at(i))) std::printf("slot %lld written twice\n", (long long)i), std::exit(1);
        if (std::isnan(x)) std::printf("slot %lld: a term was not ready\n", (long long)i), std::exit(1);
        v.at(i) = x;
        ++written;
    };
    // the base pass
    int64_t groups = 0;
    for (size_t ti = 0; ti < P.tensors.size(); ++ti) {
        const PartTensor& t = P.tensors[ti];
        if (t.group0 != groups || t.chunk > kPartChunkMax || t.nentry > kPartMaxEntry ||
            t.nunit > kPartMaxUnit || t.nphase > kPartMaxPhase || t.run < 1 || t.run > kPartRun)
            return std::puts("limits"), 1;
        groups += t.ngroup;
        if (t.ngroup != (t.nchunk + t.run - 1) / t.run) return std::puts("runs"), 1;
        if (P.phase_end.at(t.phase0) != 0 || P.phase_end.at(t.phase0 + t.nphase - 1) != t.nunit)
            return std::puts("phases"), 1;
        std::vector<double> gap, edge;
        for (int64_t c = 0; c < t.nchunk; ++c) {
            const int64_t g = c / t.run, c0 = g * t.run, c1 = std::min(c0 + t.run, t.nchunk);
            if (c == c0) gap.assign(t.ngap, 0.0), edge.assign(t.nentry, unset);
            const int64_t start = c * t.chunk, len = std::min<int64_t>(t.chunk, t.n - start);
            std::vector<double> S(P.lds_doubles, unset);
            for (int64_t i = 0; i < len; ++i) S.at(i) = z[ti].at(start + i);
            for (int32_t f = 1; f < t.nphase; ++f) {
                std::vector<std::pair<int64_t, double>> out;   // a phase reads nothing it writes
                for (int32_t u = P.phase_end.at(t.phase0 + f - 1); u < P.phase_end.at(t.phase0 + f); ++u) {
                    const PartUnit w = P.units.at(t.unit0 + u);
                    const int64_t cnt = len / w.p;
                    if (len % w.p || (len == t.chunk && cnt != w.n)) return std::puts("unit size"), 1;
                    if (w.kind == PART_ADD) {
                        for (int64_t i = w.i0; i < std::min<int64_t>(w.i0 + kPartUnit, cnt); ++i) {
                            double s = 0.0;
                            for (int32_t k = 0; k < w.q; ++k) s += S.at(w.src + i * w.q + k);
                            out.push_back({w.dst + i, s});
                        }
                    } else if (w.kind == PART_GAP) {
                        double acc = 0.0;
                        for (int64_t i = w.i0; i < std::min<int64_t>(w.i0 + kPartUnit, cnt - 1); ++i)
                            acc += std::fabs(S.at(w.src + i + 1) - S.at(w.src + i));
                        if (w.i0 == 0) {
                            const int64_t o = t.out0 + (t.ngap + w.dst) * t.ngroup + g;
                            if (c == c0) put(part, o, S.at(w.src));
                            else acc += std::fabs(S.at(w.src) - edge.at(w.dst));
                            edge.at(w.dst) = S.at(w.src + cnt - 1);
                            if (c + 1 == c1) put(part, o + t.nentry * t.ngroup, S.at(w.src + cnt - 1));
                        }
                        gap.at(w.slot) += acc;
                        if (c + 1 == c1) put(part, t.out0 + w.slot * t.ngroup + g, gap.at(w.slot));
                    } else {
                        for (int64_t i = w.i0; i < std::min<int64_t>(w.i0 + kPartUnit, cnt); ++i)
                            put(sums, P.keep.at(t.keep0 + w.slot) + start / w.p + i, S.at(w.src + i));
                    }
                }
                for (auto& o : out) {
                    if (!std::isnan(S.at(o.first)) || std::isnan(o.second)) return std::puts("LDS slot"), 1;
                    S.at(o.first) = o.second;
                }
            }
        }
    }
    if (groups != P.groups) return std::puts("group count"), 1;
    int64_t span_items = 0;   // the direct divisors
    for (const PartSpan& sp : P.spans) {
        const int64_t n = P.tensors.at(sp.tensor).n;
        if (sp.item0 != span_items || sp.count < 1) return std::puts("span items"), 1;
        span_items += sp.n_items;
        for (int64_t it = 0; it < sp.n_items; ++it) {
            const int64_t e0 = it * kPartSpan, e1 = std::min(e0 + kPartSpan, n);
            const int64_t top = P.direct.at(sp.first + sp.count - 1);
            if (top > P.direct_max || top > kPartDirectMax) return std::puts("direct divisor"), 1;
            const int64_t end = std::min(e1 + 2 * top, n);   // elements in LDS
            for (int64_t d = 0; d < sp.count; ++d) {
                const int64_t p = P.direct.at(sp.first + d), nb = n / p;
                const int64_t first = (e0 + p - 1) / p, last = std::min((e1 + p - 1) / p, nb - 1);
                const int64_t at = P.store.at(sp.store0 + d), own = (e1 + p - 1) / p;
                double acc = 0.0, prev = 0.0;
                for (int64_t i = first; i <= last || i < own; ++i) {
                    if (i * p < e0 || (i + 1) * p > end) return std::puts("block outside the span"), 1;
                    double s = 0.0;
                    for (int64_t k = i * p; k < (i + 1) * p; ++k) s += z[sp.tensor].at(k);
                    if (i > first && i <= last) acc += std::fabs(s - prev);
                    prev = s;
                    if (at >= 0 && i < own) put(sums, at + i, s);
                }
                put(part, sp.out + d * sp.n_items + it, acc);
            }
        }
    }
    if (span_items != P.span_items) return std::puts("span count"), 1;
    for (const auto& l : P.launches) {
        int64_t items = 0;
        std::vector<std::pair<int64_t, double>> out;   // a launch reads nothing it writes
        for (const PartJob& j : l) {
            if (j.item0 != items || j.n_items < 1) return std::puts("items"), 1;
            items += j.n_items;
            auto term = [&](int64_t i) { return j.src >= 0 ? sums.at(j.src + i) : z[j.tensor].at(i); };
            for (int64_t it = 0; it < j.n_items; ++it) {
                if (j.kind == PART_DIFF) {
                    double acc = 0.0;
                    for (int64_t i = it * j.per; i < std::min(it * j.per + j.per, j.count - 1); ++i)
                        acc += std::fabs(sums.at(j.src + i + 1) - sums.at(j.src + i));
                    put(part, j.dst + it, acc);
                } else if (j.kind == PART_SUB) {
                    const int64_t b = it / j.sub, a = b * j.q + (it % j.sub) * kPartSub;
                    double s = 0.0;
                    for (int64_t i = a; i < std::min(a + kPartSub, (b + 1) * j.q); ++i) s += term(i);
                    out.push_back({j.dst + it, s});
                } else {
                    for (int64_t b = it * j.per; b < std::min(it * j.per + j.per, j.count); ++b) {
                        double s = 0.0;
                        for (int64_t i = b * j.q; i < (b + 1) * j.q; ++i) s += term(i);
                        out.push_back({j.dst + b, s});
                    }
                }
            }
        }
        for (auto& o : out) put(sums, o.first, o.second);
    }
    if (written != P.sums + P.parts) return std::puts("slots never written"), 1;
    // scores
    double worst = 0.0;
    for (size_t ti = 0; ti < P.tensors.size(); ++ti) {
        const int64_t n = P.tensors[ti].n;
        const std::vector<int64_t> divs = part_divisors(n);
        if (P.count.at(ti) != (int32_t)divs.size()) return std::puts("divisor count"), 1;
        for (size_t i = 0; i < divs.size(); ++i) {
            const PartScore& s = P.scores.at(P.first.at(ti) + i);
            if (s.p != divs[i] || s.nb != n / s.p) return std::puts("score order"), 1;
            if (s.nb < 2) continue;
            double acc = 0.0;
            for (int64_t k = 0; k < s.terms; ++k) acc += part.at(s.out + k);
            for (int64_t k = 0; k + 1 < s.runs; ++k)
                acc += std::fabs(part.at(s.firsts + k + 1) - part.at(s.lasts + k));
            const double got = acc / double(s.p) / double(s.nb - 1);
            double ref = 0.0, prev = 0.0;
            for (int64_t b = 0; b < s.nb; ++b) {
                double m = 0.0;
                for (int64_t k = 0; k < s.p; ++k) m += z[ti][b * s.p + k];
                m /= double(s.p);
                if (b) ref += std::fabs(m - prev);
                prev = m;
            }
            ref /= double(s.nb - 1);
            worst = std::max(worst, std::fabs(got - ref) / std::max(std::fabs(ref), 1e-300));
        }
    }
    std::printf("largest relative difference %.3g\n", worst);
    return worst < 1e-9 ? 0 : 1;
}

int main(int argc, char** argv)
{
    // PART_SCALE: as if the plan held that many times the elements (longer runs)
    const int64_t scale = std::getenv("PART_SCALE") ? std::atoll(std::getenv("PART_SCALE")) : 1;
    const char* limit = std::getenv("PART_BUDGET");
    std::vector<std::vector<double>> z;   // z of every tensor
    std::vector<PartInput> in;
    std::mt19937_64 gen(17);
    int64_t total = 0;
    for (int a = 1; a < argc; ++a) {
        const int64_t n = std::atoll(argv[a]);
        z.emplace_back(n);
        std::normal_distribution<double> d(0.0, 1.0);
        for (double& v : z.back()) v = std::log(std::pow(d(gen), 2) + 1e-8);
        in.push_back(PartInput{nullptr, n, 0});
        total += n;
    }
    if (!limit) {
        PartPlan P;
        for (const PartInput& t : in) part_add(P, nullptr, t.n, 0, total * scale, part_budget(total * scale));
        part_finish(P);
        return check(P, z);
    }
    const int64_t budget = std::atoll(limit);
    size_t at = 0;
    for (const PartPlan& P : part_plans(in, budget)) {
        const size_t n = P.tensors.size();
        int64_t least = 0;
        for (size_t i = 0; i < n; ++i) least = std::max(least, P.shapes.at(P.tensors[i].n).least);
        std::printf("%zu tensors from %zu: %lld bytes stored, least %lld\n", n, at,
                    (long long)(8 * P.sums), (long long)least);
        if (at + n > z.size() || !n) return std::puts("plan's tensors"), 1;
        if (8 * P.sums > budget && (n > 1 || least < kPartLeastMax))
            return std::puts("over the budget"), 1;
        if (check(P, {z.begin() + at, z.begin() + at + n})) return 1;
        at += n;
    }
    return at == z.size() ? 0 : 1;
}
