// Third form of the plan-specialized matvec ("window form"): the same map as the two forms of jit.cpp (target-driven
// gather, Sec. II; digits by Eq. decode; channels by Eqs. src_digit_two_site / sourceoffset; ladder factors of App. A,
// App. B, App. C), for plans with real term weights, built for registers and for the L2.
//
// Index space.  The sites are taken in an order of their own, most significant first: uniform sites (digits fixed for
// a super-tile), unrolled sites (P_U copies per thread) and inner sites (T rows, one per thread).  The order need not
// be that of the index: a row's memory offset is the sum of its digits times their strides, a 32-bit register for the
// inner sites, a constant for a copy and a scalar for the super-tile.  So a super-tile, and the run of super-tiles
// that one XCD sweeps, can span any set of sites.
//
// Registers.  The masked and the list form hold every copy's rows and coefficients at once (150 to 330 registers on
// the named lattices, one or two waves per SIMD).  Here the copies run one after the other out of LDS, where the
// super-tile's x is staged, and a coefficient is a scalar wherever the operators' nonzero factors are all equal (spins
// up to 1, most bonds): what a row may not read is decided by its address instead, a zero row in LDS or an
// out-of-range buffer offset, so a masked lane adds k * 0.  Two channels of one coefficient that exclude each other
// (the S+S- and S-S+ of a bond with a spin 1/2) share one read, at the address of whichever applies.  Channels that
// leave the super-tile are skipped by a scalar branch where their uniform digits do not admit them, and the gathers of
// a copy are issued before the LDS part of the copy ahead of them is done.  Diagonal terms and factors of the uniform
// digits come from small tables in LDS, theta included, which every block fills once.
//
// Passes.  One launch may leave out terms, add to y instead of overwriting it, or do half a Chebyshev step, so that
// the terms of the most significant sites can be applied by a second pass whose order makes them near neighbours.
#include <algorithm>
#include <map>
#include <set>
#include <sstream>

#include "gen_util.h"
#include "mrmf_internal.h"
#include "window.h"

namespace mrmf {
namespace {

constexpr int kPairMax = 256;      // largest d_a d_b tabulated for a pair of uniform sites

struct WinGen {
    const mrmf_plan_t* p;
    const WindowPass& w;
    const bool f32;
    const int N;
    std::vector<int> pos;       // position of a site in the order
    std::vector<int64_t> vs;    // stride of a site within its group (rows, copies or super-tiles)
    int64_t T = 1, PU = 1, n_st = 1;
    int SZ;

    WinGen(const mrmf_plan_t* plan, const WindowPass& pass)
        : p(plan), w(pass), f32(pass.f32), N(plan->N), pos(plan->N), vs(plan->N, 1), SZ(pass.f32 ? 8 : 16) {
        for (int i = 0; i < N; ++i) pos[w.ord[i]] = i;
        auto strides = [&](int lo, int hi) {
            int64_t m = 1;
            for (int i = hi - 1; i >= lo; --i) {
                vs[w.ord[i]] = m;
                m *= p->d[w.ord[i]];
            }
            return m;
        };
        n_st = strides(0, w.n_uni);
        PU = strides(w.n_uni, w.n_uni + w.n_unr);
        T = strides(w.n_uni + w.n_unr, N);
    }

    bool uni(int s) const { return s >= 0 && pos[s] < w.n_uni; }
    bool unr(int s) const { return s >= 0 && pos[s] >= w.n_uni && pos[s] < w.n_uni + w.n_unr; }
    bool inner(int s) const { return s >= 0 && pos[s] >= w.n_uni + w.n_unr; }
    int udigit(int s, int64_t j) const { return static_cast<int>((j / vs[s]) % p->d[s]); }
    int64_t copy_rows(int64_t j) const {
        int64_t o = 0;
        for (int i = w.n_uni; i < w.n_uni + w.n_unr; ++i) o += udigit(w.ord[i], j) * p->M[w.ord[i]];
        return o;
    }
    // the copy that copy j's channel reads, -1 when an unrolled source digit is out of range
    int64_t copy_source(int64_t j, const DevChan& c) const {
        int64_t s = j;
        for (auto so : {std::make_pair(c.a, c.qa), std::make_pair(c.b, c.qb)})
            if (unr(so.first)) {
                const int n = udigit(so.first, j) - so.second;
                if (n < 0 || n >= p->d[so.first]) return -1;
                s -= so.second * vs[so.first];
            }
        return s;
    }

    // ---------------------------------------------------------------- constants
    std::vector<double> pool;  // factor tables looked up by a lane's digit
    std::map<std::pair<int, int>, size_t> pool_at;
    size_t table(int s, int op) {
        auto it = pool_at.find({s, op});
        if (it != pool_at.end()) return it->second;
        const size_t at = pool.size();
        for (double v : op_table(p, s, op)) pool.push_back(v);
        pool_at[{s, op}] = at;
        return at;
    }
    // whether the table's entry at digit variable n is nonzero; "" always, "false" never
    std::string nonzero(int s, int op, const std::string& n) {
        const std::vector<double> t = op_table(p, s, op);
        const int d = static_cast<int>(t.size());
        int lo = d, hi = -1, cnt = 0;
        uint32_t bits = 0;
        for (int i = 0; i < d; ++i)
            if (t[i] != 0.0) {
                lo = std::min(lo, i);
                hi = i;
                ++cnt;
                if (i < 32) bits |= 1u << i;
            }
        if (cnt == d) return "";
        if (cnt == 0) return "false";
        if (cnt == hi - lo + 1) {
            if (lo == 0) return n + " <= " + std::to_string(hi) + "u";
            if (hi == d - 1) return n + " >= " + std::to_string(lo) + "u";
            return n + " - " + std::to_string(lo) + "u <= " + std::to_string(hi - lo) + "u";
        }
        if (d <= 32) return "((" + std::to_string(bits) + "u >> " + n + ") & 1u) != 0u";
        return name("K") + "[" + std::to_string(table(s, op)) + "u + " + n + "] != (R)0";
    }
    // the common nonzero value of a table; false when it has several (or none)
    bool one_value(int s, int op, double* v) const {
        *v = 0.0;
        for (double t : op_table(p, s, op)) {
            if (t == 0.0) continue;
            if (*v != 0.0 && t != *v) return false;
            *v = t;
        }
        return *v != 0.0;
    }
    std::string name(const std::string& n) const { return n + w.tag; }
    static std::string num(int64_t v) { return std::to_string(v); }

    // ---------------------------------------------------------------- lane functions (inner sites)
    // The factor of a term's inner sites at a row: mask (where it is nonzero) and value.
    using InnerOps = std::vector<std::pair<int, int>>;  // (site, op)
    struct Lane {
        bool masked = false, konst = false;
        double value = 1.0;  // of a konst function where the mask holds
        bool have_value = false;
    };
    std::map<InnerOps, int> lane_at;
    std::vector<Lane> lanes;
    std::set<int> lane_sites, params;
    std::ostringstream head;  // per-thread values computed once
    InnerOps inner_ops(int a, int opa, int b, int opb) const {
        InnerOps k;
        if (inner(a)) k.push_back({a, opa});
        if (inner(b)) k.push_back({b, opb});
        std::sort(k.begin(), k.end());
        return k;
    }
    int lane(const InnerOps& k) {
        if (k.empty()) return -1;
        auto it = lane_at.find(k);
        if (it != lane_at.end()) return it->second;
        const int i = static_cast<int>(lanes.size());
        Lane L;
        std::string m;
        L.konst = true;
        for (const auto& so : k) {
            lane_sites.insert(so.first);
            const std::string c = nonzero(so.first, so.second, "n" + num(so.first));
            if (!c.empty()) m += (m.empty() ? "" : " && ") + ("(" + c + ")");
            double v;
            if (one_value(so.first, so.second, &v))
                L.value *= v;
            else
                L.konst = false;
        }
        L.masked = !m.empty();
        head << "  const bool m" << i << " = act" << (m.empty() ? "" : " && " + m) << ";\n";
        lanes.push_back(L);
        lane_at[k] = i;
        return i;
    }
    std::string mask(int lf) const { return lf < 0 ? "act" : "m" + num(lf); }
    // register with the value of lane function lf (0 where masked)
    std::string value(const InnerOps& k, int lf) {
        Lane& L = lanes[lf];
        const std::string v = "f" + num(lf);
        if (!L.have_value) {
            L.have_value = true;
            std::string e;
            if (L.konst) {
                e = lit(L.value, f32);
            } else {
                for (const auto& so : k)
                    e += (e.empty() ? "" : " * ") + name("K") + "[" + num(table(so.first, so.second)) + "u + n" +
                         num(so.first) + "]";
            }
            head << "  const R " << v << " = m" << lf << " ? " << e << " : (R)0;\n";
        }
        return v;
    }

    // ---------------------------------------------------------------- registries of emitted values
    std::map<std::pair<int, double>, std::string> uk;  // uniform coefficient theta[param] * value
    std::string ucoef(int param, double v) {
        auto it = uk.find({param, v});
        if (it != uk.end()) return it->second;
        params.insert(param);
        const std::string n = "u" + num(uk.size());
        head << "  const R " << n << " = uniform_of(th" << param << " * " << lit(v, f32) << ");\n";
        return uk[{param, v}] = n;
    }
    std::map<std::tuple<int, double, int>, std::string> lk;  // theta[param] * value * lane function
    std::string lcoef(int param, double v, const InnerOps& k, int lf) {
        auto it = lk.find({param, v, lf});
        if (it != lk.end()) return it->second;
        params.insert(param);
        const std::string n = "l" + num(lk.size()), f = value(k, lf);
        head << "  const R " << n << " = th" << param << " * " << lit(v, f32) << " * " << f << ";\n";
        return lk[{param, v, lf}] = n;
    }
    std::map<std::string, std::string> exprs;  // expression of a per-thread register -> its name
    std::string reg(const std::string& type, const std::string& prefix, const std::string& e) {
        auto it = exprs.find(e);
        if (it != exprs.end()) return it->second;
        const std::string n = prefix + num(exprs.size());
        head << "  const " << type << " " << n << " = " << e << ";\n";
        return exprs[e] = n;
    }
    // Tables over the digits of one or two uniform sites: entry (n_a, n_b) is the sum of theta[param] * value over
    // its list, filled into LDS by every block, read once per super-tile.
    struct Tab {
        int a, b;
        size_t at;
    };
    std::vector<std::vector<std::pair<int, double>>> entries;
    std::vector<Tab> tabs;
    bool too_big = false;
    int new_tab(int a, int b) {
        const size_t n = size_t(p->d[a]) * (b >= 0 ? p->d[b] : 1);
        if (entries.size() + n > size_t(kWindowTab)) {
            too_big = true;
            return -1;
        }
        tabs.push_back({a, b, entries.size()});
        entries.resize(entries.size() + n);
        return static_cast<int>(tabs.size()) - 1;
    }
    std::set<int> uni_sites;  // uniform sites whose digit the kernel needs
    // adds theta[param] * v * f_a(n_a) f_b(n_b) to a table of a superset of the sites
    void tab_add(int t, int param, double v, int a, int opa, int b, int opb) {
        const Tab& q = tabs[t];
        const int da = p->d[q.a], db = q.b >= 0 ? p->d[q.b] : 1;
        const std::vector<double> fa = op_table(p, a, opa);
        const std::vector<double> fb = b >= 0 ? op_table(p, b, opb) : std::vector<double>{};
        for (int i = 0; i < da; ++i)
            for (int k = 0; k < db; ++k) {
                auto dig = [&](int s) { return s == q.a ? i : k; };
                const double x = v * fa[dig(a)] * (b >= 0 ? fb[dig(b)] : 1.0);
                if (x != 0.0) entries[q.at + size_t(i) * db + k].push_back({param, x});
            }
        uni_sites.insert(q.a);
        if (q.b >= 0) uni_sites.insert(q.b);
    }
    std::string tab_read(int t) const {
        const Tab& q = tabs[t];
        std::string i = "n" + num(q.a);
        if (q.b >= 0) i += " * " + num(p->d[q.b]) + "u + n" + num(q.b);
        return "ut[" + num(q.at) + "u + " + i + "]";
    }

    // scalar byte offset of a copy's rows shifted by -delta from super-tile base b
    std::string soff(const std::string& b, int64_t j, int64_t delta) const {
        const int64_t o = (copy_rows(j) - delta) * SZ;
        if (w.wide) return b + " + (unsigned long long)(" + num(o) + "ll)";
        return b + " + " + std::to_string(static_cast<uint32_t>(static_cast<uint64_t>(o))) + "u";
    }

    std::string source(WindowCost* cost);
};

std::string WinGen::source(WindowCost* cost) {
    const mrmf_plan_t& P = *p;
    const int block = static_cast<int>(round_up(T, 64));
    const bool cheb = w.mode >= kPassCheb;
    int64_t dmax = 0;
    for (const auto& c : P.chans) dmax = std::max<int64_t>(dmax, c.delta);
    const int64_t shift = (dmax + T) * SZ, nrec = (P.D + dmax + T) * SZ;
    const int64_t CS = T + 1;  // rows of a copy in LDS: its T rows and a zero row

    // ---------------------------------------------------------------- channels
    struct Stat {
        std::string addr, coef;
        int64_t src;
        int chan, lf;
        InnerOps ops;
        int64_t di;
    };
    // a channel that reads outside the super-tile: scalar condition ("": always), lanes, offset, coefficient
    struct Glob {
        std::string cond, coef;
        int64_t delta;
        int chan, lf;
        bool varying, tabled;  // as a gather's
    };
    // a gather: per-lane byte offset, offset of its scalar base, coefficient; `branch`: scalar condition of a gather
    // that is rare enough to be issued and used in a branch of its own
    struct Load {
        std::string off, coef, branch;
        int64_t delta;
        bool varying = false, tabled = false;  // the coefficient differs between rows or super-tiles; comes from a table
    };
    std::vector<std::vector<Stat>> stat(PU);
    std::vector<std::vector<Glob>> glob(PU);
    std::vector<std::vector<Load>> load(PU);
    std::map<std::string, std::string> tile_bools;  // per super-tile: condition -> name
    std::ostringstream tile;                        // per super-tile scalars
    std::map<int, std::string> tab_names;
    auto tab_value = [&](int t) {
        auto it = tab_names.find(t);
        if (it != tab_names.end()) return it->second;
        const std::string n = "t" + num(t);
        tile << "    const R " << n << " = " << tab_read(t) << ";\n";
        return tab_names[t] = n;
    };
    bool any_static = false;
    for (int ci : w.chans) {
        const DevChan& c = P.chans[ci];
        const InnerOps ops = inner_ops(c.a, c.opa, c.b, c.opb);
        const bool global = uni(c.a) || uni(c.b);
        // scalar admissibility of the uniform sites and whether their factors are constants there
        std::string cond;
        double uconst = 1.0;
        bool utab = false, never = false;
        // the lower site first, however the term lists them: the conditions are sorted by their text, and in the other
        // order the scalars of many bonds spill (all pairs of 16 spins 1/2, 164 instead of 16)
        const std::pair<int, int> sa(c.a, c.opa), sb(c.b, c.opb);
        for (auto so : {std::min(sa, sb), std::max(sa, sb)})
            if (uni(so.first)) {
                const std::string e = nonzero(so.first, so.second, "n" + num(so.first));
                if (e == "false") never = true;
                if (!e.empty()) {
                    cond += (cond.empty() ? "" : " && ") + ("(" + e + ")");
                    uni_sites.insert(so.first);
                }
                double v;
                if (one_value(so.first, so.second, &v))
                    uconst *= v;
                else
                    utab = true;
            }
        for (auto so : {std::make_pair(c.a, c.opa), std::make_pair(c.b, c.opb)})
            if (inner(so.first) && nonzero(so.first, so.second, "n") == "false") never = true;
        if (never) continue;
        int64_t di = 0;  // inner part of the offset, in rows of a copy
        if (inner(c.a)) di += c.qa * vs[c.a];
        if (inner(c.b)) di += c.qb * vs[c.b];
        const int lf = lane(ops);
        const bool lconst = lf < 0 || lanes[lf].konst;
        std::string gcond, ut;
        if (global) {
            if (!cond.empty()) {
                auto it = tile_bools.find(cond);
                if (it == tile_bools.end()) it = tile_bools.emplace(cond, "q" + num(tile_bools.size())).first;
                gcond = it->second;
            }
            if (utab) {  // theta w f_a f_b (and a constant lane factor) of the uniform digits, from a table
                const bool ua = uni(c.a), ub = uni(c.b);
                if (ua && ub && P.d[c.a] * P.d[c.b] > kPairMax) return "";
                const int t = new_tab(ua ? c.a : c.b, ua && ub ? c.b : -1);
                if (t < 0) return "";
                const double v = c.wr * (lf >= 0 && lconst ? lanes[lf].value : 1.0);
                params.insert(c.param);
                if (ua)
                    tab_add(t, c.param, v, c.a, c.opa, ub ? c.b : -1, c.opb);
                else
                    tab_add(t, c.param, v, c.b, c.opb, -1, 0);
                ut = tab_value(t);
            }
        }
        for (int64_t j = 0; j < PU; ++j) {
            double uf = 1.0;
            if (unr(c.a)) uf *= op_table(p, c.a, c.opa)[udigit(c.a, j)];
            if (unr(c.b)) uf *= op_table(p, c.b, c.opb)[udigit(c.b, j)];
            if (uf == 0.0) continue;
            const double v = c.wr * uf * uconst * (lf >= 0 && lconst ? lanes[lf].value : 1.0);
            if (global) {
                Glob g;
                g.cond = gcond;
                g.delta = c.delta;
                g.chan = ci;
                g.lf = lf;
                g.tabled = !ut.empty();
                g.varying = !lconst || g.tabled;
                if (!ut.empty()) {
                    g.coef = ut + (uf != 1.0 ? " * " + lit(uf, f32) : std::string(""));
                    if (!lconst) g.coef += " * " + value(ops, lf);
                } else {
                    g.coef = lconst ? ucoef(c.param, v) : lcoef(c.param, c.wr * uf * uconst, ops, lf);
                }
                glob[j].push_back(g);
                continue;
            }
            Stat s;
            s.src = copy_source(j, c);
            if (s.src < 0) continue;
            s.chan = ci;
            s.lf = lf;
            s.ops = ops;
            s.di = di;
            s.coef = lconst ? ucoef(c.param, v) : lcoef(c.param, c.wr * uf, ops, lf);
            stat[j].push_back(s);
            any_static = true;
        }
    }
    // static channels of one copy with the same coefficient whose lanes exclude each other share a read
    auto disjoint = [&](const InnerOps& x, const InnerOps& y) {
        std::vector<int> sites;
        for (const auto& so : x) sites.push_back(so.first);
        for (const auto& so : y) sites.push_back(so.first);
        std::sort(sites.begin(), sites.end());
        sites.erase(std::unique(sites.begin(), sites.end()), sites.end());
        if (sites.size() > 2) return false;
        const int da = p->d[sites[0]], db = sites.size() > 1 ? p->d[sites[1]] : 1;
        for (int i = 0; i < da; ++i)
            for (int k = 0; k < db; ++k) {
                auto on = [&](const InnerOps& z) {
                    for (const auto& so : z)
                        if (op_table(p, so.first, so.second)[so.first == sites[0] ? i : k] == 0.0) return false;
                    return true;
                };
                if (on(x) && on(y)) return false;
            }
        return true;
    };
    std::map<std::pair<InnerOps, InnerOps>, bool> disjoint_at;
    for (int64_t j = 0; j < PU; ++j) {
        std::vector<Stat> out;
        std::vector<char> used(stat[j].size(), 0);
        for (size_t i = 0; i < stat[j].size(); ++i) {
            if (used[i]) continue;
            Stat s = stat[j][i];
            std::string e = mask(s.lf) + " ? r - (unsigned)(" + num(s.di) + ") : " + num(T) + "u";
            const bool konst = s.lf >= 0 && lanes[s.lf].konst && lanes[s.lf].masked;
            for (size_t k = i + 1; konst && k < stat[j].size(); ++k) {
                const Stat& q = stat[j][k];
                if (used[k] || q.src != s.src || q.coef != s.coef || q.lf < 0 || !lanes[q.lf].konst) continue;
                const auto key = std::make_pair(s.ops, q.ops);
                auto it = disjoint_at.find(key);
                if (it == disjoint_at.end()) it = disjoint_at.emplace(key, disjoint(s.ops, q.ops)).first;
                if (!it->second) continue;
                e = mask(s.lf) + " ? r - (unsigned)(" + num(s.di) + ") : " + mask(q.lf) + " ? r - (unsigned)(" + num(q.di) +
                    ") : " + num(T) + "u";
                used[k] = 1;
                break;
            }
            s.addr = s.lf < 0 ? "ra" : reg("unsigned", "ad", e);
            out.push_back(s);
        }
        stat[j] = out;
    }

    // Gathers.  Two channels on the same sites that exclude each other share one, at the offset of whichever applies;
    // two on uniform sites that do not (spins of 1 and more) share one for either and have a rare second one for both.
    std::map<std::string, std::string> tile_regs;  // per super-tile: expression of a lane offset or coefficient -> name
    std::ostringstream tile_off;
    auto tile_reg = [&](const std::string& type, const std::string& prefix, const std::string& e) {
        auto it = tile_regs.find(e);
        if (it != tile_regs.end()) return it->second;
        const std::string n = prefix + num(tile_regs.size());
        tile_off << "    const " << type << " " << n << " = " << e << ";\n";
        return tile_regs[e] = n;
    };
    auto both = [&](const DevChan& x, const DevChan& y) {  // share of the digits of their (uniform or inner) sites that admit both
        const int sa = x.a, sb = x.b;
        const int da = p->d[sa], db = sb >= 0 ? p->d[sb] : 1;
        int n = 0;
        for (int i = 0; i < da; ++i)
            for (int k = 0; k < db; ++k) {
                auto on = [&](const DevChan& c) {
                    for (auto so : {std::make_pair(c.a, c.opa), std::make_pair(c.b, c.opb)})
                        if (so.first >= 0 && !unr(so.first) && op_table(p, so.first, so.second)[so.first == sa ? i : k] == 0.0)
                            return false;
                    return true;
                };
                if (on(x) && on(y)) ++n;
            }
        return double(n) / double(da * db);
    };
    // The second gather of a pair gets a branch where at most this share of the digits admits both: two spins 1 (1/9), whose
    // branch is mostly skipped (4 x 4 lattice 1.33 ms either way).  Above it a masked load for every lane costs less than
    // the waits around a branch that is often taken: ring of 12 spins 3/2 (1/4) 434 -> 301 us, chain 328 -> 284 us,
    // chain of 13 spins 1 and 3/2 363 -> 337 us, in c64 222 -> 195 us.
    constexpr double kRareShare = 0.125;
    int64_t span = 0;  // largest lane offset of a row in its copy
    for (int i = w.n_uni + w.n_unr; i < N; ++i) span += (P.d[w.ord[i]] - 1) * P.M[w.ord[i]];
    std::map<std::pair<int, int>, double> both_at;
    for (int64_t j = 0; j < PU; ++j) {
        std::vector<char> used(glob[j].size(), 0);
        for (size_t i = 0; i < glob[j].size(); ++i) {
            if (used[i]) continue;
            const Glob& one = glob[j][i];
            bool paired = false;
            for (size_t k = i + 1; k < glob[j].size() && !paired; ++k) {
                const Glob& two = glob[j][k];
                if (used[k] || two.delta == one.delta) continue;
                const DevChan &x = P.chans[one.chan], &y = P.chans[two.chan];
                if (!((x.a == y.a && x.b == y.b) || (x.a == y.b && x.b == y.a))) continue;
                const bool scalar = one.lf < 0 && two.lf < 0;  // no inner site
                if (one.coef != two.coef && !scalar) continue;
                const auto key = std::make_pair(one.chan, two.chan);
                auto it = both_at.find(key);
                if (it == both_at.end()) it = both_at.emplace(key, both(x, y)).first;
                const double share = it->second;
                if (share > 0.0 && !(scalar && !one.cond.empty() && !two.cond.empty())) continue;
                if (share > 0.0 && one.cond == two.cond) continue;
                // h's rows are ahead of the gather's base, which is g's: never negative
                const Glob &g = one.delta > two.delta ? one : two, &h = one.delta > two.delta ? two : one;
                if ((g.delta - h.delta + span) * SZ >= (int64_t(1) << 31)) break;
                auto on = [&](const Glob& q) {
                    std::string e = q.cond;
                    if (q.lf >= 0 && lanes[q.lf].masked) e += (e.empty() ? "" : " && ") + mask(q.lf);
                    return e.empty() ? std::string("act") : e;
                };
                const std::string ahead = num((g.delta - h.delta) * SZ) + "u";
                const std::string og = on(g), oh = on(h);
                if (og == "act" || oh == "act") break;
                Load l;
                l.delta = g.delta;
                l.varying = g.varying || h.varying;
                l.tabled = g.tabled || h.tabled;
                // voff + ahead of an inactive lane stays out of range: 2^31 + ahead < 2^32
                l.off = tile_reg("unsigned", "o", "(" + og + ") ? voff : (" + oh + ") ? voff + " + ahead + " : OOB");
                l.coef = g.coef == h.coef ? g.coef : tile_reg("R", "c", "(" + og + ") ? " + g.coef + " : " + h.coef);
                load[j].push_back(l);
                if (share > 0.0) {  // both: the second one of the pair
                    Load r;
                    r.delta = h.delta;
                    r.varying = h.varying;
                    r.tabled = h.tabled;
                    r.off = "voff";
                    r.coef = h.coef;
                    r.branch = g.cond + " && " + h.cond;
                    if (share > kRareShare) {
                        r.off = tile_reg("unsigned", "o", "(" + r.branch + ") ? voff : OOB");
                        r.branch.clear();
                    }
                    load[j].push_back(r);
                }
                used[k] = 1;
                paired = true;
            }
            if (paired) continue;
            Load l;
            l.delta = one.delta;
            l.varying = one.varying;
            l.tabled = one.tabled;
            l.coef = one.coef;
            const std::string lane_off =
                one.lf < 0 || !lanes[one.lf].masked ? "voff" : reg("unsigned", "vo", mask(one.lf) + " ? voff : OOB");
            l.off = one.cond.empty() ? lane_off : tile_reg("unsigned", "o", "(" + one.cond + ") ? " + lane_off + " : OOB");
            load[j].push_back(l);
        }
        // the gathers in branches of their own last
        std::stable_sort(load[j].begin(), load[j].end(), [](const Load& x, const Load& y) { return x.branch.empty() > y.branch.empty(); });
    }

    // ---------------------------------------------------------------- diagonal terms
    std::vector<std::string> dj(PU);  // per copy: terms added to its weight
    std::string d_lane;               // inner sites only: one register
    std::vector<std::string> d_tile;  // uniform sites only: one scalar per super-tile
    std::string d_mixed;              // uniform and inner sites: summed per lane once per super-tile
    {
        std::map<std::pair<int, int>, int> utabs;
        std::vector<std::map<int, double>> cc(PU);  // unrolled sites only: sum over params of theta * value
        std::vector<int> order(w.diags.begin(), w.diags.end());
        std::stable_sort(order.begin(), order.end(), [&](int x, int y) { return (P.diags[x].b >= 0) > (P.diags[y].b >= 0); });
        for (int gi : order) {
            const DevDiag& g = P.diags[gi];
            const bool ua = uni(g.a), ub = uni(g.b);
            const InnerOps ops = inner_ops(g.a, g.opa, g.b, g.opb);
            const bool un = unr(g.a) || unr(g.b);
            if (ua && (ub || g.b < 0)) {  // uniform only: one table per pair, a one-site term joins a pair of its site
                if (ub && P.d[g.a] * P.d[g.b] > kPairMax) return "";
                int t = -1;
                if (g.b < 0)
                    for (const auto& kv : utabs)
                        if (kv.first.first == g.a || kv.first.second == g.a) t = kv.second;
                if (t < 0) {
                    const std::pair<int, int> key(g.a, ub ? g.b : -1);
                    auto it = utabs.find(key);
                    if (it == utabs.end()) {
                        t = new_tab(key.first, key.second);
                        if (t < 0) return "";
                        utabs[key] = t;
                        d_tile.push_back(tab_value(t));
                    } else {
                        t = it->second;
                    }
                }
                params.insert(g.param);
                tab_add(t, g.param, g.wr, g.a, g.opa, ub ? g.b : -1, g.opb);
                continue;
            }
            if (!ua && !ub) {
                if (ops.empty()) {  // unrolled only
                    for (int64_t j = 0; j < PU; ++j) {
                        double v = g.wr * op_table(p, g.a, g.opa)[udigit(g.a, j)];
                        if (g.b >= 0) v *= op_table(p, g.b, g.opb)[udigit(g.b, j)];
                        cc[j][g.param] += v;
                    }
                    params.insert(g.param);
                    continue;
                }
                const int lf = lane(ops);
                const std::string f = value(ops, lf);
                if (!un) {
                    params.insert(g.param);
                    d_lane += (d_lane.empty() ? "" : " + ") + ("th" + num(g.param) + " * " + lit(g.wr, f32) + " * " + f);
                    continue;
                }
                const int us = unr(g.a) ? g.a : g.b, uo = unr(g.a) ? g.opa : g.opb;
                for (int64_t j = 0; j < PU; ++j) {
                    const double z = op_table(p, us, uo)[udigit(us, j)];
                    if (z != 0.0) dj[j] += " + " + ucoef(g.param, g.wr * z) + " * " + f;
                }
                continue;
            }
            // one uniform site and one of the super-tile
            const int us = ua ? g.a : g.b, uo = ua ? g.opa : g.opb;
            const int ts = ua ? g.b : g.a, to = ua ? g.opb : g.opa;
            const int t = new_tab(us, -1);
            if (t < 0) return "";
            params.insert(g.param);
            tab_add(t, g.param, g.wr, us, uo, -1, 0);
            const std::string tv = tab_value(t);
            if (inner(ts)) {
                const std::string f = value(ops, lane(ops));
                d_mixed += " + " + tv + " * " + f;
            } else {
                for (int64_t j = 0; j < PU; ++j) {
                    const double z = op_table(p, ts, to)[udigit(ts, j)];
                    if (z != 0.0) dj[j] += " + " + tv + " * " + lit(z, f32);
                }
            }
        }
        for (int64_t j = 0; j < PU; ++j) {
            std::string e;
            for (const auto& kv : cc[j])
                if (kv.second != 0.0) e += (e.empty() ? "" : " + ") + ("th" + num(kv.first) + " * " + lit(kv.second, f32));
            if (!e.empty()) dj[j] += " + " + reg("R", "cc", "uniform_of(" + e + ")");
        }
        if (!d_lane.empty()) head << "  const R dI = " << d_lane << ";\n";
    }
    if (too_big) return "";
    const bool has_diag = !w.diags.empty();
    const bool need_x = has_diag || (cheb);  // the row's own x

    // ---------------------------------------------------------------- kernel
    std::ostringstream o;
    const size_t ne = entries.size();
    cost->coefs = static_cast<int>(uk.size());
    cost->fills = static_cast<int>((ne + block - 1) / block);
    cost->gathers = static_cast<int>(load[0].size());
    for (const Load& l : load[0]) {
        cost->varying += l.varying;
        cost->tabled += l.tabled;
    }
    // the couplings and values of an entry's addend u at [u * ne + entry]; -1: it has fewer
    size_t width = 0;
    for (const auto& e : entries) width = std::max(width, e.size());
    std::ostringstream cp, cv;
    for (size_t u = 0; u < width; ++u)
        for (size_t e = 0; e < ne; ++e) {
            const bool in = u < entries[e].size();
            cp << (u + e ? ", " : "") << (in ? entries[e][u].first : -1);
            cv << (u + e ? ", " : "") << lit(in ? entries[e][u].second : 0.0, f32);
        }
    if (width > 0)
        o << "__constant__ int " << name("CP") << "[" << width * ne << "] = {" << cp.str() << "};\n"
          << "__constant__ R " << name("CV") << "[" << width * ne << "] = {" << cv.str() << "};\n";
    std::ostringstream body;
    const bool use_lds = any_static || need_x;
    const bool dbuf = use_lds && 2 * PU * CS * SZ <= w.dbuf_bytes;
    if ((use_lds ? (dbuf ? 2 : 1) * PU * CS * SZ : 0) + int64_t(ne) * (f32 ? 4 : 8) > kWindowLds) return "";
    body << "extern \"C\" __global__ __launch_bounds__(" << block << ") ";
    if (w.waves > 0) body << "__attribute__((amdgpu_waves_per_eu(" << w.waves << "))) ";
    body << "void " << w.name << "(const R* __restrict__ theta,\n    const C* __restrict__ x, C* __restrict__ y, ";
    if (cheb) body << "C* __restrict__ acc, R ea, R eb, R eg, R ecr, R eci, ";
    body << "const int* __restrict__ skip) {\n  if (skip != nullptr && *skip != 0) return;\n";
    if (use_lds) body << "  __shared__ C xl[" << (dbuf ? 2 : 1) * PU * CS << "];\n";
    if (ne > 0) body << "  __shared__ R ut[" << ne << "];\n";
    body << "  const unsigned tid = threadIdx.x;\n"
         << "  const bool act = tid < " << T << "u;\n"
         << "  const unsigned r = act ? tid : 0u;\n"
         << "  const unsigned ra = act ? tid : " << T << "u;\n"
         << "  const unsigned OOB = 0x80000000u;\n";
    // The tables.  A thread works all its entries out before it stores the first, so their loads are in flight together: one
    // entry after another, a chain of three loads each, was what a short launch waited for (8 spins 3/2 in a chain of
    // different couplings, four rounds of 64 threads: 4.8 -> 4.0 us in c128, 4.7 -> 3.8 in c64; a chain of 12 spins 1/2, one
    // round: 3.5 -> 3.2; from 10^7 rows up no difference).
    if (ne > 0) {
        body << "  R us[" << cost->fills << "];\n#pragma unroll\n  for (unsigned i = 0; i < " << cost->fills << "u; ++i) {\n"
             << "    const unsigned k = tid + i * " << block << "u < " << ne << "u ? tid + i * " << block << "u : " << ne - 1
             << "u;\n    (void)k;\n    R s = (R)0;\n";
        if (width > 0)
            body << "#pragma unroll " << kWindowSum << "\n    for (unsigned u = 0; u < " << width * ne << "u; u += " << ne
                 << "u) { const int p = " << name("CP") << "[u + k]; const R t = theta[p < 0 ? 0 : p] * " << name("CV")
                 << "[u + k]; s = p < 0 ? s : s + t; }\n";
        body << "    us[i] = s;\n  }\n#pragma unroll\n  for (unsigned i = 0; i < " << cost->fills << "u; ++i)\n    if (tid + i * " << block
             << "u < " << ne << "u) ut[tid + i * " << block << "u] = us[i];\n";
    }
    if (use_lds)
        body << "  for (unsigned i = tid; i < " << (dbuf ? 2 : 1) * PU << "u; i += " << block << "u) { const C z = {(R)0, (R)0}; xl[i * "
             << CS << "u + " << T << "u] = z; }\n";
    // the row's digits and its offset in memory
    bool contiguous = true;
    std::string vo;
    for (int i = w.n_uni + w.n_unr; i < N; ++i) {
        const int s = w.ord[i];
        contiguous &= p->M[s] == vs[s];
    }
    if (!contiguous)
        for (int i = w.n_uni + w.n_unr; i < N; ++i) lane_sites.insert(w.ord[i]);
    for (int s : lane_sites) body << "  const unsigned n" << s << " = (r / " << vs[s] << "u) % " << P.d[s] << "u;\n";
    if (contiguous) {
        vo = "r * " + num(SZ) + "u";
    } else {
        for (int i = w.n_uni + w.n_unr; i < N; ++i) {
            const int s = w.ord[i];
            vo += (vo.empty() ? "" : " + ") + ("n" + num(s) + " * " + num(p->M[s] * SZ) + "u");
        }
    }
    body << "  const unsigned voff = act ? " << vo << " : OOB;\n";
    for (int q : params) body << "  const R th" << q << " = theta[" << q << "];\n";
    body << head.str();
    if (w.wide) {
        body << "  const char* const xs = (const char*)x;\n  char* const ys = (char*)y;\n";
        if (w.mode == kPassCheb) body << "  char* const as = (char*)acc;\n";
    } else {
        auto rs = [&](const char* n, const std::string& ptr) {
            body << "  const __amdgpu_buffer_rsrc_t " << n << " = __builtin_amdgcn_make_buffer_rsrc((void*)((char*)" << ptr << " - "
                 << shift << "ll), (short)0, " << nrec << ", 0x00020000);\n";
        };
        rs("xs", "x");
        rs("ys", "y");
        if (w.mode == kPassCheb) rs("as", "acc");
    }
    // sweep: windows of G super-tiles, or one contiguous eighth per XCD (blocks b mod 8), its blocks side by side
    body << "  const unsigned G = gridDim.x, b = blockIdx.x;\n  unsigned par = 0u;\n  (void)par;\n";
    if (w.sched == MRMF_SCHED_XCD_CHUNK)
        body << "  const unsigned nx = (G % 8u == 0u) ? 8u : 1u, xcd = b % nx, t_step = G / nx;\n"
             << "  const unsigned Cx = (" << n_st << "u + nx - 1u) / nx;\n"
             << "  const unsigned t_end = (xcd + 1u) * Cx < " << n_st << "u ? (xcd + 1u) * Cx : " << n_st << "u;\n"
             << "  unsigned t = xcd * Cx + b / nx;\n";
    else if (w.sched == MRMF_SCHED_BLOCK_RUN)
        body << "  const unsigned v = (G % 8u == 0u) ? (b % 8u) * (G / 8u) + b / 8u : b;\n"
             << "  const unsigned t_end = (unsigned)(((unsigned long long)(v + 1u) * " << n_st << "ull) / G), t_step = 1u;\n"
             << "  unsigned t = (unsigned)(((unsigned long long)v * " << n_st << "ull) / G);\n";
    else
        body << "  const unsigned t_end = " << n_st << "u, t_step = G;\n"
             << "  unsigned t = (G % 8u == 0u) ? (b % 8u) * (G / 8u) + b / 8u : b;\n";
    // base of super-tile `t`
    bool natural = true;
    for (int i = 0; i < w.n_uni; ++i) natural &= P.M[w.ord[i]] == vs[w.ord[i]] * (w.n_uni > 0 ? P.M[w.ord[w.n_uni - 1]] : 1);
    auto base = [&](const std::string& b, const std::string& t) {
        std::string e;
        const char* ty = w.wide ? "unsigned long long" : "unsigned";
        if (w.n_uni == 0) {
            e = "0";
        } else if (natural) {
            e = std::string("(") + ty + ")(" + t + ") * " + num(P.M[w.ord[w.n_uni - 1]] * SZ) + "u";
        } else {
            for (int i = 0; i < w.n_uni; ++i) {
                const int s = w.ord[i];
                e += (e.empty() ? "" : " + ") + std::string("(") + ty + ")(((" + t + ") / " + num(vs[s]) + "u) % " + num(P.d[s]) +
                     "u) * " + (w.wide ? num(P.M[s] * SZ) + "ull" : num(P.M[s] * SZ) + "u");
            }
        }
        return std::string("const ") + ty + " " + b + " = " + e + (w.wide ? "" : " + " + num(shift) + "u") + ";";
    };
    const bool stage = use_lds;
    if (stage && w.prefetch) {
        for (int64_t j = 0; j < PU; ++j) body << "  C xn" << j << " = {(R)0, (R)0};\n";
        body << "  if (t < t_end) {\n    " << base("Fn", "t") << "\n";
        for (int64_t j = 0; j < PU; ++j) body << "    xn" << j << " = LD(xs, voff, " << soff("Fn", j, 0) << ");\n";
        body << "  }\n";
    }
    body << "  __syncthreads();\n"
         << "  for (; t < t_end; t += t_step) {\n    " << base("F0", "t") << "\n";
    if (stage) {
        body << "    C* const lb = xl" << (dbuf ? " + par * " + num(PU * CS) + "u" : std::string("")) << ";\n";
        if (!w.prefetch)
            for (int64_t j = 0; j < PU; ++j) body << "    const C xn" << j << " = LD(xs, voff, " << soff("F0", j, 0) << ");\n";
        body << "    if (act) {\n";
        for (int64_t j = 0; j < PU; ++j) body << "      lb[" << j * CS << "u + r] = xn" << j << ";\n";
        body << "    }\n";
    }
    for (int s : uni_sites) body << "    const unsigned n" << s << " = (t / " << vs[s] << "u) % " << P.d[s] << "u;\n";
    for (const auto& kv : tile_bools) body << "    const bool " << kv.second << " = " << kv.first << ";\n";
    if (stage) body << "    __syncthreads();\n";
    // the rows of the next super-tile, requested behind the last gathers (loads return in order)
    auto prefetch = [&]() {
        if (!stage || !w.prefetch) return;
        body << "    if (t + t_step < t_end) {\n      " << base("Fn", "t + t_step") << "\n";
        for (int64_t j = 0; j < PU; ++j) body << "      xn" << j << " = LD(xs, voff, " << soff("Fn", j, 0) << ");\n";
        body << "    }\n";
    };
    body << tile.str() << tile_off.str();
    const bool d_common = !d_tile.empty() || !d_lane.empty() || !d_mixed.empty();
    if (d_common) {
        body << "    const R dU = " << (d_lane.empty() ? "(R)0" : "dI");
        for (const auto& t : d_tile) body << " + " << t;
        body << d_mixed << ";\n";
    }
    struct Unit {
        int64_t j;
        size_t lo, hi;
        bool first, last;
    };
    std::vector<Unit> units;
    const size_t GS = static_cast<size_t>(w.group);
    std::vector<size_t> plain(PU);  // gathers that are not in a branch
    for (int64_t j = 0; j < PU; ++j) {
        size_t n = 0, lo = 0;
        while (n < load[j].size() && load[j][n].branch.empty()) ++n;
        plain[j] = n;
        do {
            const size_t hi = std::min(n, lo + GS);
            units.push_back({j, lo, hi, lo == 0, hi == n});
            lo = hi;
        } while (lo < n);
    }
    auto loads = [&](const Unit& u) {
        const std::string J = num(u.j);
        for (size_t i = u.lo; i < u.hi; ++i) {
            const Load& g = load[u.j][i];
            body << "    const C s" << J << "_" << num(i) << " = LD(xs, " << g.off << ", " << soff("F0", u.j, g.delta) << ");\n";
        }
        if (u.first) {
            const std::string so = soff("F0", u.j, 0);
            if (w.mode == kPassAdd || cheb) body << "    const C yv" << J << " = LD(ys, voff, " << so << ");\n";
            if (w.mode == kPassCheb) body << "    const C av" << J << " = LD(as, voff, " << so << ");\n";
        }
    };
    loads(units[0]);
    if (units.size() == 1) prefetch();
    for (size_t ui = 0; ui < units.size(); ++ui) {
        const Unit& u = units[ui];
        const std::string J = num(u.j), ar = "a" + J + "r", ai = "a" + J + "i";
        // Without it the compiler turns the conditional accumulations into selects and sinks them all below the last
        // gather, so that every gather of the super-tile is live at once.
        auto fence = [&]() { body << "    MRMF_GROUP_FENCE(" << ar << ", " << ai << ");\n"; };
        if (ui + 1 < units.size()) {
            loads(units[ui + 1]);
            if (ui + 2 == units.size()) prefetch();
        }
        if (u.first) {
            if (need_x) body << "    const C x" << J << " = lb[ra + " << u.j * CS << "u];\n";
            if (has_diag) {
                const std::string d = d_common ? "dU" : "(R)0";
                body << "    R " << ar << ", " << ai << ";\n    { const R d = " << d << dj[u.j] << "; " << ar << " = d * x" << J
                     << ".x; " << ai << " = d * x" << J << ".y; }\n";
            } else {
                body << "    R " << ar << " = (R)0, " << ai << " = (R)0;\n";
            }
            int n = 0;
            for (const Stat& s : stat[u.j]) {
                if (n && n % w.group == 0) fence();
                ++n;
                body << "    { const C s = lb[" << s.addr << " + " << s.src * CS << "u]; " << ar << " += " << s.coef << " * s.x; "
                     << ai << " += " << s.coef << " * s.y; }\n";
            }
            fence();
        }
        for (size_t i = u.lo; i < u.hi; ++i) {
            const std::string s = "s" + J + "_" + num(i);
            body << "    { const R k = " << load[u.j][i].coef << "; " << ar << " += k * " << s << ".x; " << ai << " += k * " << s
                 << ".y; }\n";
        }
        if (u.hi > u.lo) fence();
        if (!u.last) continue;
        for (size_t i = plain[u.j]; i < load[u.j].size(); ++i) {
            const Load& g = load[u.j][i];
            body << "    if (" << g.branch << ") { const C s = LD(xs, " << g.off << ", " << soff("F0", u.j, g.delta) << "); const R k = "
                 << g.coef << "; " << ar << " += k * s.x; " << ai << " += k * s.y; }\n";
        }
        const std::string so = soff("F0", u.j, 0);
        if (w.mode == kPassSet || w.mode == kPassAdd) {
            const std::string add = w.mode == kPassAdd ? "yv" + J : "";
            body << "    { C out; out.x = " << ar << (add.empty() ? "" : " + " + add + ".x") << "; out.y = " << ai
                 << (add.empty() ? "" : " + " + add + ".y") << "; ST(out, ys, voff, " << so << "); }\n";
        } else {
            body << "    { C np; np.x = ea * " << ar << " + eb * x" << J << ".x + eg * yv" << J << ".x; np.y = ea * " << ai << " + eb * x"
                 << J << ".y + eg * yv" << J << ".y;\n      ST(np, ys, voff, " << so << ");\n";
            if (w.mode == kPassCheb)
                body << "      C na; na.x = av" << J << ".x + ecr * np.x - eci * np.y; na.y = av" << J
                     << ".y + ecr * np.y + eci * np.x;\n      ST(na, as, voff, " << so << ");\n";
            body << "    }\n";
        }
    }
    if (stage && !dbuf) body << "    __syncthreads();\n";
    body << "    par ^= 1u;\n  }\n}\n";

    std::ostringstream full;
    full << "// generated (window form): " << N << " sites, " << w.chans.size() << " channels, " << w.diags.size()
         << " diagonal terms; " << T << " rows per block, " << PU << " unrolled copies, " << n_st << " super-tiles\n";
    full << "__constant__ R " << name("K") << "[" << std::max<size_t>(1, pool.size()) << "] = {";
    if (pool.empty()) full << "0";
    for (size_t i = 0; i < pool.size(); ++i) full << (i ? ", " : "") << lit(pool[i], f32);
    full << "};\n" << o.str() << body.str();
    return full.str();
}

}  // namespace

bool window_real(const mrmf_plan_t* p) {
    for (const auto& c : p->chans)
        if (c.wi != 0.0) return false;
    for (const auto& g : p->diags)
        if (g.wi != 0.0) return false;
    return true;
}

std::string window_prelude(bool f32, bool wide) {
    std::ostringstream o;
    const char* bits = f32 ? "64" : "128";
    o << "typedef " << (f32 ? "float" : "double") << " R;\ntypedef " << (f32 ? "float" : "double")
      << " C __attribute__((ext_vector_type(2)));\n"
      << "typedef unsigned U __attribute__((ext_vector_type(" << (f32 ? 2 : 4) << ")));\n";
    if (wide) {
        // a buffer resource per access, based at the super-tile's byte offset (scalar arithmetic only)
        o << "#define RS(p) __builtin_amdgcn_make_buffer_rsrc((void*)(p), (short)0, 0x7fffffff, 0x00020000)\n"
          << "#define LD(rs, vo, so) __builtin_bit_cast(C, __builtin_amdgcn_raw_buffer_load_b" << bits
          << "(RS((rs) + (so)), (int)(vo), 0, 0))\n"
          << "#define ST(v, rs, vo, so) __builtin_amdgcn_raw_buffer_store_b" << bits
          << "(__builtin_bit_cast(U, (v)), RS((rs) + (so)), (int)(vo), 0, 2)\n";
    } else {
        // the store's offset goes into the VGPR operand and its scalar offset is the constant 0: with a register
        // scalar offset the compiler inserts no wait state between a 128-bit store and a following VALU write of its
        // data registers, and the stored value was then observed to be overwritten
        o << "#define LD(rs, vo, so) __builtin_bit_cast(C, __builtin_amdgcn_raw_buffer_load_b" << bits
          << "((rs), (int)(vo), (int)(so), 0))\n"
          << "#define ST(v, rs, vo, so) __builtin_amdgcn_raw_buffer_store_b" << bits
          << "(__builtin_bit_cast(U, (v)), (rs), (int)((unsigned)(vo) + (unsigned)(so)), 0, 2)\n";
    }
    o << "#ifndef MRMF_GROUP_FENCE\n"
      << "#define MRMF_GROUP_FENCE(a, b) __asm__ __volatile__(\"\" : \"+v\"(a), \"+v\"(b) : : \"memory\")\n"
      << "#endif\n"
      << "__device__ __forceinline__ R uniform_of(R v) {\n";
    if (f32)
        o << "  return __builtin_bit_cast(R, __builtin_amdgcn_readfirstlane(__builtin_bit_cast(int, v)));\n}\n";
    else
        o << "  const unsigned long long u = __builtin_bit_cast(unsigned long long, v);\n"
          << "  const unsigned lo = (unsigned)__builtin_amdgcn_readfirstlane((int)(unsigned)u);\n"
          << "  const unsigned hi = (unsigned)__builtin_amdgcn_readfirstlane((int)(unsigned)(u >> 32));\n"
          << "  return __builtin_bit_cast(R, ((unsigned long long)hi << 32) | lo);\n}\n";
    return o.str();
}

std::string window_pass(const mrmf_plan_t* p, const WindowPass& w, int64_t* n_tiles, int64_t* rows, WindowCost* cost) {
    WinGen g(p, w);
    *n_tiles = g.n_st;
    *rows = g.T;
    return g.source(cost);
}

}  // namespace mrmf
