// Factorised form of the contraction program (used by gen_contract.cpp).
//
// A connected graph is evaluated by contracting its moments two tensors at a
// time: every connected node subset S of a graph is an intermediate tensor
// whose open legs are the index slots of its nodes that no edge of S takes.
// Two subsets with isomorphic labelled multigraphs are the same tensor, so
// intermediates are shared between graphs (and, inside one, between equal
// branches).  The expanded polynomials multiply every monomial out instead:
// 285 k flops per neighborhood at level 24 against 21 k here, 39.4 k against
// 7.2 k at level 20, 5.3 k against 2.2 k at level 16 (four clusters; the
// basis functions' walk included).
//
// A tensor keeps one component per orbit of its symmetries: the open legs of
// one node are interchangeable, and so are nodes exchanged by an automorphism
// of the subset.
//
// The basis functions split at half the level: a graph above L / 2 ("high")
// occurs in a basis function at most once and only beside low graphs, so
//   V = Z(low) + sum_H g_H Y_H(low),  Y_H = sum_p xi_{H p} p,
// p running over the products of low graphs (1 included) that fit beside H.
// dV/dg_H = Y_H needs the low graphs' values alone, so a high graph goes
// forward, gets its dV/dg and comes back in one piece, and what the low graphs
// need of the high ones are the few sums X_p = sum_H xi_{H p} g_H: neither
// graph values nor dV/dg are exchanged between wavefronts or kept.
#pragma once

#include <algorithm>
#include <array>
#include <cmath>
#include <functional>
#include <map>
#include <set>
#include <sstream>
#include <stdexcept>
#include <string>
#include <tuple>
#include <vector>

#include "basis.hpp"

namespace mtp {
namespace dag {

using Multi = std::array<int, 3>;   // exponents of x, y, z

inline const std::vector<Multi> &sym_multis(int o) {   // the multi-indices of degree o, in component order
    static std::vector<std::vector<Multi>> all;
    while ((int)all.size() <= o) {
        const int d = (int)all.size();
        std::vector<Multi> v;
        for (int a = d; a >= 0; --a)
            for (int b = d - a; b >= 0; --b) v.push_back({a, b, d - a - b});
        all.push_back(v);
    }
    return all[o];
}
inline int sym_index(const Multi &m) {
    const auto &v = sym_multis(m[0] + m[1] + m[2]);
    return (int)(std::find(v.begin(), v.end(), m) - v.begin());
}

struct Key {
    std::vector<Label> labels;
    std::vector<int> edges;   // canonical, upper triangle row-major
    bool operator<(const Key &o) const { return labels < o.labels || (labels == o.labels && edges < o.edges); }
};

struct Tensor {
    Key key;
    std::vector<int> open;    // open legs per canonical node
    std::vector<int> radix;   // components per canonical node
    int full = 1;             // product of radix
    std::vector<int> rep;     // full component -> stored component
    std::vector<std::vector<Multi>> reps;   // stored component -> multi-index per canonical node
    int n_store() const { return (int)reps.size(); }
    int first_comp = -1;      // single node: its first moment component
    int index(const std::vector<Multi> &m) const {
        int f = 0;
        for (size_t v = 0; v < open.size(); ++v) f = f * radix[v] + sym_index(m[v]);
        return rep[f];
    }
};

struct Term {
    int c, a, b;
    long coef;
};

struct Split {                // a node subset as the product of two
    int s1, s2;               // masks
    int t1, t2;               // tensors
    std::vector<Term> terms;
    long cost = 0;            // forward and reverse multiply-adds
};

// every connected subset of a graph's nodes, its tensor and its splits
struct Host {
    int n = 0;
    std::vector<int> tensor;                  // by mask, -1: not connected
    std::vector<std::vector<int>> order;      // canonical position -> node
    std::vector<std::vector<Split>> splits;   // by mask
    std::vector<int> by_size;                 // connected masks, small first
};

struct Op {                   // how a tensor is formed in a cluster
    int c, a, b;              // tensors
    std::vector<Term> terms;
    long cost;
};

struct Cluster {
    std::vector<int> graphs;
    std::map<int, Op> ops;    // tensor -> op
    long cost = 0;
    std::vector<int> comps;   // moment components read and whose dV/dM is added to
    std::vector<int> prods;   // products p whose sum X_p is added to
    std::vector<int> rows(int nc) const {   // the sums a cluster adds to: components, then nc + p
        std::vector<int> r = comps;
        for (int p : prods) r.push_back(nc + p);
        return r;
    }
};

class Factorised {
  public:
    const Basis &B;
    std::vector<Tensor> tensors;
    std::map<Key, int> by_key;
    std::vector<Host> hosts;
    std::vector<int> low, high;                        // graph numbers
    std::vector<std::vector<int>> prods;               // p: factors (low graph numbers), prods[0] = {}
    std::map<std::vector<int>, int> prod_id;
    std::map<std::vector<int>, int> func_id;           // basis function by factors

    explicit Factorised(const Basis &b) : B(b) {
        for (size_t f = 0; f < B.funcs.size(); ++f) func_id[B.funcs[f]] = (int)f;
        int min_high = 1 << 20;
        for (size_t G = 0; G < B.graphs.size(); ++G) {
            const int lv = B.graphs[G].level();
            (2 * lv > B.level ? high : low).push_back((int)G);
            if (2 * lv > B.level) min_high = std::min(min_high, lv);
        }
        prods.push_back({});
        if (!high.empty())
            for (auto &f : B.funcs) {
                int lv = 0;
                bool ok = true;
                for (int g : f) {
                    lv += B.graphs[g].level();
                    ok = ok && 2 * B.graphs[g].level() <= B.level;
                }
                if (ok && lv + min_high <= B.level) prods.push_back(f);
            }
        for (size_t p = 0; p < prods.size(); ++p) prod_id[prods[p]] = (int)p;
        for (auto &f : B.funcs) {   // every prefix of a function is a function: products are formed along it
            int nh = 0;
            for (int g : f) nh += 2 * B.graphs[g].level() > B.level;
            if (nh > 1) throw std::runtime_error("two high graphs in one basis function");
            if (nh == 1 && !prod_id.count(std::vector<int>(f.begin(), f.end() - 1)))
                throw std::runtime_error("high graph beside an unlisted product");
        }
        hosts.resize(B.graphs.size());
        for (size_t G = 0; G < B.graphs.size(); ++G) build_host((int)G);
    }

    // the cluster of the given graphs: contraction orders chosen graph by
    // graph with what is already formed at no cost, then improved by
    // re-choosing every graph's order against the others' tensors
    Cluster make_cluster(const std::vector<int> &graphs) const {
        std::vector<std::map<int, Op>> ops(graphs.size());
        auto available = [&](size_t skip) {
            std::map<int, Op> av;
            for (size_t k = 0; k < graphs.size(); ++k)
                if (k != skip) av.insert(ops[k].begin(), ops[k].end());
            return av;
        };
        std::vector<size_t> by_size(graphs.size());
        for (size_t k = 0; k < graphs.size(); ++k) by_size[k] = k;
        std::stable_sort(by_size.begin(), by_size.end(), [&](size_t x, size_t y) {
            return B.graphs[graphs[x]].n() < B.graphs[graphs[y]].n();
        });
        long best_total = -1;
        std::map<int, Op> best_ops;
        for (int round = 0; round < 4; ++round) {
            for (size_t k : by_size) {
                const std::map<int, Op> av = available(k);
                ops[k] = plan(graphs[k], av);
            }
            // one op per tensor, and only those that are reached
            std::map<int, Op> all = available((size_t)-1), live;
            std::function<void(int)> need = [&](int t) {
                if (tensors[t].key.labels.size() == 1 || live.count(t)) return;
                const Op &o = all.at(t);
                live[t] = o;
                need(o.a);
                need(o.b);
            };
            for (int G : graphs) need(top(G));
            long total = 0;
            for (auto &kv : live) total += kv.second.cost;
            if (best_total < 0 || total < best_total) {
                best_total = total;
                best_ops = live;
            }
        }
        Cluster cl;
        cl.graphs = graphs;
        cl.ops = best_ops;
        cl.cost = std::max<long>(best_total, 0);
        std::set<int> cs;
        for (int G : graphs)
            for (auto &l : B.graphs[G].labels) {
                const Tensor &t = tensors[by_key.at(Key{{l}, {}})];
                for (int q = 0; q < t.n_store(); ++q) cs.insert(t.first_comp + q);
            }
        cl.comps.assign(cs.begin(), cs.end());
        std::set<int> ps;
        for (int G : graphs)
            if (2 * B.graphs[G].level() > B.level)
                for (size_t p = 0; p < prods.size(); ++p)
                    if (function_of((int)p, G) >= 0) ps.insert((int)p);
        cl.prods.assign(ps.begin(), ps.end());
        return cl;
    }

    // Graphs into nc clusters: largest first, each to the cluster it adds the
    // least work and the fewest sums (moment components, X_p) to, among those whose work
    // stays near the mean (cluster nc - 1 has last_extra to do besides).
    std::vector<Cluster> clusters(const std::vector<int> &graphs, int nc, int comp_weight, long last_extra) const {
        std::vector<std::vector<int>> part(nc);
        std::vector<Cluster> cl(nc);
        const long whole = make_cluster(graphs).cost;
        std::vector<int> order = graphs;
        std::map<int, long> alone;
        for (int G : graphs) alone[G] = make_cluster({G}).cost;
        std::stable_sort(order.begin(), order.end(), [&](int a, int b) { return alone[a] > alone[b]; });
        for (int G : order) {
            int best = -1;
            double bs = 0;
            Cluster bc;
            for (int q = 0; q < nc; ++q) {
                std::vector<int> gl = part[q];
                gl.push_back(G);
                const Cluster c = make_cluster(gl);
                const double grow = (double)(c.cost - cl[q].cost) +
                                    comp_weight * (double)((long)(c.comps.size() + c.prods.size()) -
                                                           (long)(cl[q].comps.size() + cl[q].prods.size()));
                // past the mean load, what a cluster already holds counts against it
                const double load = (double)c.cost + (q == nc - 1 ? (double)last_extra : 0.0);
                const double over = std::max(0.0, load - 1.12 * (double)(whole + last_extra) / nc);
                const double score = grow + 2.0 * over;
                if (best < 0 || score < bs) {
                    best = q;
                    bs = score;
                    bc = c;
                }
            }
            part[best].push_back(G);
            cl[best] = bc;
        }
        for (int q = 0; q < nc; ++q) {
            std::sort(part[q].begin(), part[q].end());
            cl[q] = make_cluster(part[q]);
        }
        return cl;
    }

    int top(int G) const { return hosts[G].tensor[(1 << hosts[G].n) - 1]; }
    int function_of(int p, int G) const {   // basis function: product p times graph G, or -1
        std::vector<int> f = prods[p];
        f.push_back(G);
        auto it = func_id.find(f);
        return it == func_id.end() ? -1 : it->second;
    }
    int n_low_functions() const {
        int n = 0;
        for (auto &f : B.funcs) n += 2 * B.graphs[f.back()].level() <= B.level;
        return n;
    }
    int n_prods() const { return (int)prods.size(); }

    // ---- code ------------------------------------------------------------------
    // cmul(c, x) and cfma(c, x, y) multiply by a constant or a coefficient
    // that carries no tangent when T is a dual number.

    // Cluster `cl`, forward and back: reads M[k] and the products p[], writes
    // B_alpha of its functions (WB) and its share of the sums it adds to (in the
    // order of cl.rows) to d[].
    std::string emit_cluster(const Cluster &cl, long &fl) const {
        Writer w{*this, cl, fl};
        std::vector<bool> xset(prods.size(), false);
        std::vector<int> left = cl.graphs;
        while (!left.empty()) {
            size_t best = 0;
            long bl = -1;
            for (size_t k = 0; k < left.size(); ++k) {   // the graph that leaves the fewest tensors waiting
                const long l = w.live_after(left[k]);
                if (bl < 0 || l < bl) {
                    bl = l;
                    best = k;
                }
            }
            const int G = left[best];
            left.erase(left.begin() + (long)best);
            w.os << "    // " << B.graphs[G].str() << "\n";
            w.forward(top(G));
            const std::string g = "g" + std::to_string(G), y = "y" + std::to_string(G);
            w.os << "    const T " << g << " = " << w.value(top(G), 0) << ";\n";
            for (size_t q = 0; q < cl.prods.size(); ++q) {
                const int p = cl.prods[q], f = function_of(p, G);
                if (f < 0) continue;
                const std::string al = "xi[" + std::to_string(f) + "]", pv = "p[" + std::to_string(p) + "]",
                                  x = "d[" + std::to_string(cl.comps.size() + q) + "]";
                w.os << "    if (WB) Bout[" << f << "] = " << (p ? pv + " * " + g : g) << ";\n";
                if (p == 0)
                    w.os << "    T " << y << " = T(" << al << ");\n";
                else
                    w.os << "    " << y << " = cfma(" << al << ", " << pv << ", " << y << ");\n";
                w.os << "    " << x << " = " << (xset[p] ? "cfma(" : "cmul(") << al << ", " << g
                     << (xset[p] ? ", " + x : std::string()) << ");\n";
                fl += (p ? 2 : 0) + (xset[p] ? 2 : 1);
                xset[p] = true;
            }
            w.reverse(top(G), y);
            w.os << "    MTP_FACT_SCHED();\n";
        }
        for (size_t k = 0; k < cl.comps.size(); ++k)
            if (!w.dset[k]) w.os << "    d[" << k << "] = T(0);\n";
        return w.os.str();
    }

    // gl[] of the low graphs (cluster `cl`) and the products p[] (p[0], the empty one, is not written)
    std::string emit_low_values(const Cluster &cl, long &fl) const {
        Writer w{*this, cl, fl};
        for (size_t k = 0; k < cl.graphs.size(); ++k) {
            w.forward(top(cl.graphs[k]));
            w.os << "    gl[" << k << "] = " << w.value(top(cl.graphs[k]), 0) << ";\n";
        }
        for (size_t p = 1; p < prods.size(); ++p) {
            const std::vector<int> &f = prods[p];
            const std::string last = "gl[" + std::to_string(low_pos(f.back())) + "]";
            if (f.size() == 1)
                w.os << "    p[" << p << "] = " << last << ";\n";
            else {
                w.os << "    p[" << p << "] = p[" << prod_id.at({f.begin(), f.end() - 1}) << "] * " << last << ";\n";
                fl += 1;
            }
        }
        return w.os.str();
    }

    // Z: the basis functions of low graphs alone, V and dz[] = dV/dg of the
    // low graphs by a nested walk over the trie of their factor sequences
    std::string emit_low_functions(long &fl) const {
        std::ostringstream os;
        std::vector<bool> set(low.size(), false);
        os << "    T w0 = T(0);\n";
        std::function<void(const std::vector<int> &, const std::string &)> visit = [&](const std::vector<int> &pre,
                                                                                        const std::string &ind) {
            const int d = (int)pre.size();
            const std::string bd = "b" + std::to_string(d), b1 = "b" + std::to_string(d + 1),
                              wd = "w" + std::to_string(d), w1 = "w" + std::to_string(d + 1);
            for (size_t k = pre.empty() ? 0 : (size_t)low_pos(pre.back()); k < low.size(); ++k) {
                std::vector<int> f = pre;
                f.push_back(low[k]);
                auto it = func_id.find(f);
                if (it == func_id.end()) continue;
                const std::string g = "gl[" + std::to_string(k) + "]", dg = "dz[" + std::to_string(k) + "]";
                os << ind << "{\n" << ind << "  const T " << b1 << " = " << (d ? bd + " * " + g : g) << ";\n";
                os << ind << "  if (WB) Bout[" << it->second << "] = " << b1 << ";\n";
                os << ind << "  T " << w1 << " = T(xi[" << it->second << "]);\n";
                visit(f, ind + "  ");
                if (d == 0)
                    os << ind << "  " << dg << (set[k] ? " += " : " = ") << w1 << ";\n";
                else
                    os << ind << "  " << dg << " = " << (set[k] ? "fma(" + bd + ", " + w1 + ", " + dg + ")" : bd + " * " + w1)
                       << ";\n";
                set[k] = true;
                os << ind << "  " << wd << " = fma(" << g << ", " << w1 << ", " << wd << ");\n" << ind << "}\n";
                fl += (d ? 1 : 0) + (d ? 2 : 1) + 2;
            }
        };
        visit({}, "    ");
        os << "    V = w0;\n";
        for (size_t k = 0; k < low.size(); ++k)
            if (!set[k]) os << "    dz[" << k << "] = T(0);\n";
        return os.str();
    }

    // the coupling of the low graphs to the sums X_p: V += sum_p X_p p, dz += sum_p X_p dp/dg
    std::string emit_coupling(long &fl) const {
        std::ostringstream os;
        os << "    V = V + X[0];\n";
        fl += 1;
        // w(p) = X_p + sum over p g of g w(p g); dz[g] += p w(p g) along the products' trie, longest first
        std::vector<size_t> order;
        for (size_t p = 1; p < prods.size(); ++p) order.push_back(p);
        std::stable_sort(order.begin(), order.end(),
                         [&](size_t a, size_t b) { return prods[a].size() > prods[b].size(); });
        for (size_t p : order) os << "    T w" << p << " = X[" << p << "];\n";
        for (size_t p : order) {
            const std::vector<int> &f = prods[p];
            const int par = prod_id.at({f.begin(), f.end() - 1});
            const std::string g = "gl[" + std::to_string(low_pos(f.back())) + "]",
                              dg = "dz[" + std::to_string(low_pos(f.back())) + "]", w = "w" + std::to_string(p);
            if (par == 0) {
                os << "    " << dg << " = " << dg << " + " << w << ";\n    V = fma(" << g << ", " << w << ", V);\n";
                fl += 3;
            } else {
                os << "    " << dg << " = fma(p[" << par << "], " << w << ", " << dg << ");\n    w" << par << " = fma(" << g
                   << ", " << w << ", w" << par << ");\n";
                fl += 4;
            }
        }
        return os.str();
    }

    // dV/dM of the low graphs (cluster `cl`) from dz[]
    std::string emit_low_reverse(const Cluster &cl, long &fl) const {
        Writer w{*this, cl, fl};
        for (int G : cl.graphs) w.forward(top(G));
        for (size_t k = 0; k < cl.graphs.size(); ++k) w.reverse(top(cl.graphs[k]), "dz[" + std::to_string(k) + "]");
        for (size_t k = 0; k < cl.comps.size(); ++k)
            if (!w.dset[k]) w.os << "    d[" << k << "] = T(0);\n";
        return w.os.str();
    }

  private:
    int low_pos(int G) const { return (int)(std::find(low.begin(), low.end(), G) - low.begin()); }

    // writes the straight-line code of one cluster; every emitted multiply or
    // add counts into fl (a multiply-add as two)
    struct Writer {
        const Factorised &F;
        const Cluster &cl;
        long &fl;
        std::ostringstream os;
        std::set<int> formed;
        std::map<int, int> waiting;                 // tensor -> consumer ops not yet reversed
        std::map<int, std::vector<bool>> aset;      // tensor -> adjoint component assigned
        std::vector<bool> dset;
        Writer(const Factorised &f, const Cluster &c, long &n) : F(f), cl(c), fl(n), dset(c.comps.size(), false) {
            for (auto &kv : cl.ops) {
                ++waiting[kv.second.a];
                if (kv.second.b != kv.second.a) ++waiting[kv.second.b];
            }
        }
        bool single(int t) const { return F.tensors[t].key.labels.size() == 1; }
        std::string value(int t, int c) const {
            if (single(t)) return "M[" + std::to_string(F.tensors[t].first_comp + c) + "]";
            return "t" + std::to_string(t) + "_" + std::to_string(c);
        }
        static std::string scaled(long c, const std::string &x) {
            return c == 1 ? x : "cmul(" + std::to_string(c) + ", " + x + ")";
        }
        void forward(int t) {
            if (single(t) || formed.count(t)) return;
            formed.insert(t);
            const Op &o = cl.ops.at(t);
            forward(o.a);
            forward(o.b);
            std::vector<bool> set(F.tensors[t].n_store(), false);
            for (auto &x : o.terms) {
                const std::string a = scaled(x.coef, value(o.a, x.a)), b = value(o.b, x.b), c = value(t, x.c);
                if (!set[x.c])
                    os << "    T " << c << " = " << a << " * " << b << ";\n";
                else
                    os << "    " << c << " = fma(" << a << ", " << b << ", " << c << ");\n";
                fl += (set[x.c] ? 2 : 1) + (x.coef != 1);
                set[x.c] = true;
            }
        }
        // adjoint component c of tensor t gets x * y
        void add(int t, int c, const std::string &x, const std::string &y) {
            std::string n;
            bool had, decl = false;
            if (single(t)) {
                const int k = F.tensors[t].first_comp + c;
                const size_t at = std::find(cl.comps.begin(), cl.comps.end(), k) - cl.comps.begin();
                n = "d[" + std::to_string(at) + "]";
                had = dset[at];
                dset[at] = true;
            } else {
                auto &s = aset[t];
                if (s.empty()) s.assign(F.tensors[t].n_store(), false);
                n = "a" + std::to_string(t) + "_" + std::to_string(c);
                had = s[c];
                decl = !had;
                s[c] = true;
            }
            if (had)
                os << "    " << n << (y.empty() ? " = " + n + " + " + x : " = fma(" + x + ", " + y + ", " + n + ")") << ";\n";
            else
                os << "    " << (decl ? "T " : "") << n << " = " << x << (y.empty() ? "" : " * " + y) << ";\n";
            fl += (had ? 1 : 0) + (y.empty() ? 0 : 1);
        }
        // back through the op of t, whose adjoint is complete (seed: the
        // adjoint of a graph value), then through what that completes
        void reverse(int t, const std::string &seed = "") {
            if (single(t)) {
                if (!seed.empty()) add(t, 0, seed, "");
                return;
            }
            const Op &o = cl.ops.at(t);
            for (auto &x : o.terms) {
                if (seed.empty() && (aset[t].empty() || !aset[t][x.c])) continue;
                const std::string c = scaled(x.coef, seed.empty() ? "a" + std::to_string(t) + "_" + std::to_string(x.c) : seed);
                if (o.a == o.b && x.a == x.b) {
                    add(o.a, x.a, scaled(2, c), value(o.a, x.a));
                    ++fl;
                    continue;
                }
                add(o.a, x.a, c, value(o.b, x.b));
                add(o.b, x.b, c, value(o.a, x.a));
                fl += x.coef != 1;
            }
            if (--waiting[o.a] == 0) reverse(o.a);
            if (o.b != o.a && --waiting[o.b] == 0) reverse(o.b);
        }
        // stored components waiting for their adjoint once G is done
        long live_after(int G) const {
            std::set<int> f = formed;
            std::function<void(int)> need = [&](int t) {
                if (single(t) || !f.insert(t).second) return;
                const Op &o = cl.ops.at(t);
                need(o.a);
                need(o.b);
            };
            need(F.top(G));
            std::map<int, int> wt = waiting;
            std::function<void(int)> back = [&](int t) {
                if (single(t)) return;
                f.erase(t);
                const Op &o = cl.ops.at(t);
                if (--wt[o.a] == 0) back(o.a);
                if (o.b != o.a && --wt[o.b] == 0) back(o.b);
            };
            back(F.top(G));
            long n = 0;
            for (int t : f)
                if (wt[t] > 0) n += F.tensors[t].n_store();
            return n;
        }
    };

    // the tensor of the nodes `nodes` of a graph with edge matrix m; order
    // receives the canonical order of the nodes
    int tensor_of(const CGraph &g, const std::vector<std::vector<int>> &m, std::vector<int> nodes,
                  std::vector<int> &order) {
        std::stable_sort(nodes.begin(), nodes.end(), [&](int a, int b) { return g.labels[a] < g.labels[b]; });
        const int n = (int)nodes.size();
        std::vector<std::vector<int>> perms;
        std::vector<int> cur(nodes);
        std::function<void(int)> rec = [&](int at) {
            if (at == n) {
                perms.push_back(cur);
                return;
            }
            int e = at;
            while (e < n && g.labels[nodes[e]] == g.labels[nodes[at]]) ++e;
            std::vector<int> grp(nodes.begin() + at, nodes.begin() + e);
            std::sort(grp.begin(), grp.end());
            do {
                std::copy(grp.begin(), grp.end(), cur.begin() + at);
                rec(e);
            } while (std::next_permutation(grp.begin(), grp.end()));
        };
        rec(0);
        auto upper = [&](const std::vector<int> &o) {
            std::vector<int> v;
            for (int p = 0; p < n; ++p)
                for (int q = p + 1; q < n; ++q) v.push_back(m[o[p]][o[q]]);
            return v;
        };
        std::vector<int> best;
        for (auto &o : perms) {
            auto v = upper(o);
            if (order.empty() || v < best) {
                best = v;
                order = o;
            }
        }
        Key k;
        for (int v : order) k.labels.push_back(g.labels[v]);
        k.edges = best;
        auto it = by_key.find(k);
        if (it != by_key.end()) return it->second;
        Tensor t;
        t.key = k;
        for (int p = 0; p < n; ++p) {
            int o = g.labels[order[p]].nu;
            for (int q = 0; q < n; ++q) o -= q == p ? 0 : m[order[p]][order[q]];
            t.open.push_back(o);
            t.radix.push_back((int)sym_multis(o).size());
            t.full *= t.radix.back();
        }
        // automorphisms as permutations of the canonical positions
        std::vector<std::vector<int>> autos;
        for (auto &o : perms) {
            if (upper(o) != best) continue;
            std::vector<int> a(n);
            for (int p = 0; p < n; ++p) a[p] = (int)(std::find(order.begin(), order.end(), o[p]) - order.begin());
            autos.push_back(a);
        }
        auto decode = [&](int f) {
            std::vector<Multi> r(n);
            for (int p = n - 1; p >= 0; --p) {
                r[p] = sym_multis(t.open[p])[f % t.radix[p]];
                f /= t.radix[p];
            }
            return r;
        };
        t.rep.assign(t.full, -1);
        for (int f = 0; f < t.full; ++f) {
            if (t.rep[f] >= 0) continue;
            const auto mi = decode(f);
            const int id = (int)t.reps.size();
            t.reps.push_back(mi);
            for (auto &a : autos) {
                int ff = 0;
                for (int p = 0; p < n; ++p) ff = ff * t.radix[p] + sym_index(mi[a[p]]);
                t.rep[ff] = id;
            }
        }
        if (n == 1) {
            for (size_t c = 0; c < B.comps.size(); ++c)
                if (B.comps[c].mu == k.labels[0].mu && B.comps[c].nu == k.labels[0].nu) {
                    t.first_comp = (int)c;
                    break;
                }
        }
        tensors.push_back(t);
        by_key[k] = (int)tensors.size() - 1;
        return (int)tensors.size() - 1;
    }

    void build_host(int G) {
        const CGraph &g = B.graphs[G];
        Host &h = hosts[G];
        h.n = g.n();
        const int n = h.n;
        std::vector<std::vector<int>> m(n, std::vector<int>(n, 0));
        int k = 0;
        for (int p = 0; p < n; ++p)
            for (int q = p + 1; q < n; ++q, ++k) m[p][q] = m[q][p] = g.edges[k];
        h.tensor.assign(1 << n, -1);
        h.order.resize(1 << n);
        h.splits.resize(1 << n);
        for (int s = 1; s < (1 << n); ++s) {
            int seen = s & -s;
            for (bool more = true; more;) {
                more = false;
                for (int p = 0; p < n; ++p)
                    if ((s >> p & 1) && !(seen >> p & 1))
                        for (int q = 0; q < n; ++q)
                            if ((seen >> q & 1) && m[p][q]) {
                                seen |= 1 << p;
                                more = true;
                                break;
                            }
            }
            if (seen != s) continue;
            std::vector<int> nodes;
            for (int p = 0; p < n; ++p)
                if (s >> p & 1) nodes.push_back(p);
            h.tensor[s] = tensor_of(g, m, nodes, h.order[s]);
            h.by_size.push_back(s);
        }
        std::stable_sort(h.by_size.begin(), h.by_size.end(),
                         [](int a, int b) { return __builtin_popcount(a) < __builtin_popcount(b); });
        for (int s : h.by_size) {
            const int lowbit = s & -s, rest = s ^ lowbit;
            if (!rest) continue;
            for (int sub = (rest - 1) & rest;; sub = (sub - 1) & rest) {   // proper subsets of rest, with the lowest node
                const int s1 = sub | lowbit, s2 = s ^ s1;
                if (h.tensor[s1] >= 0 && h.tensor[s2] >= 0) {
                    Split sp{s1, s2, h.tensor[s1], h.tensor[s2], {}, 0};
                    contract(h, m, s, sp);
                    h.splits[s].push_back(sp);
                }
                if (sub == 0) break;
            }
        }
    }

    void contract(const Host &h, const std::vector<std::vector<int>> &m, int s, Split &sp) const {
        const Tensor &C = tensors[h.tensor[s]], &T1 = tensors[sp.t1], &T2 = tensors[sp.t2];
        const std::vector<int> &oc = h.order[s], &o1 = h.order[sp.s1], &o2 = h.order[sp.s2];
        std::vector<std::pair<int, int>> cross;
        for (int u : o1)
            for (int v : o2)
                for (int e = 0; e < m[u][v]; ++e) cross.push_back({u, v});
        long total = 1;
        for (size_t e = 0; e < cross.size(); ++e) total *= 3;
        for (int c = 0; c < C.n_store(); ++c) {
            std::vector<Multi> base(h.n, Multi{0, 0, 0});
            for (size_t p = 0; p < oc.size(); ++p) base[oc[p]] = C.reps[c][p];
            std::map<std::pair<int, int>, long> acc;
            for (long code = 0; code < total; ++code) {
                std::vector<Multi> x = base;
                long r = code;
                for (auto &e : cross) {
                    x[e.first][r % 3]++;
                    x[e.second][r % 3]++;
                    r /= 3;
                }
                std::vector<Multi> m1, m2;
                for (int v : o1) m1.push_back(x[v]);
                for (int v : o2) m2.push_back(x[v]);
                int a = T1.index(m1), b = T2.index(m2);
                if (sp.t1 == sp.t2 && a > b) std::swap(a, b);
                acc[{a, b}] += 1;
            }
            for (auto &kv : acc) sp.terms.push_back({c, kv.first.first, kv.first.second, kv.second});
        }
        sp.cost = 0;
        for (auto &t : sp.terms) sp.cost += 3 + (t.coef != 1);
    }

    // the cheapest contraction order of a graph when the tensors of `av` cost nothing
    std::map<int, Op> plan(int G, const std::map<int, Op> &av) const {
        const Host &h = hosts[G];
        const int full = (1 << h.n) - 1;
        std::vector<long> cost(full + 1, -1);
        std::vector<int> pick(full + 1, -1);
        for (int s : h.by_size) {
            if (!(s & (s - 1)) || (s != full && av.count(h.tensor[s]))) {
                cost[s] = 0;
                continue;
            }
            for (size_t k = 0; k < h.splits[s].size(); ++k) {
                const Split &sp = h.splits[s][k];
                // equal halves are formed once
                const long c = sp.cost + cost[sp.s1] + (sp.t1 == sp.t2 ? 0 : cost[sp.s2]);
                if (cost[s] < 0 || c < cost[s]) {
                    cost[s] = c;
                    pick[s] = (int)k;
                }
            }
        }
        std::map<int, Op> out;
        std::function<void(int)> take = [&](int s) {
            const int t = h.tensor[s];
            if (!(s & (s - 1)) || out.count(t)) return;
            auto it = av.find(t);
            if (s != full && it != av.end()) {   // formed for another graph: kept with its own order
                out[t] = it->second;
                std::function<void(int)> follow = [&](int u) {
                    if (tensors[u].key.labels.size() == 1 || out.count(u)) return;
                    const Op &o = av.at(u);
                    out[u] = o;
                    follow(o.a);
                    follow(o.b);
                };
                follow(it->second.a);
                follow(it->second.b);
                return;
            }
            const Split &sp = h.splits[s][pick[s]];
            out[t] = Op{t, sp.t1, sp.t2, sp.terms, sp.cost};
            take(sp.s1);
            take(sp.s2);
        };
        take(full);
        return out;
    }
};

}  // namespace dag
}  // namespace mtp
