// Source generator of the run-time specialized evaluator: writes the
// diagram's evaluation tables (leaves, denominators, groups, terms and
// momentum lines, built by build_tables) out as straight-line device code for
// the kernels of jit_kernel.hpp.  Sums over coefficients keep the order of the
// table-driven evaluators (index order, first term as +v or -v) and products
// their left-to-right association; every fused multiply-add of the values
// is written out (the code is compiled without contraction, which only the
// reverse sweep's functions turn on), so the forward and adjoint kernels of a
// diagram compute the same values bit for bit.
#include <algorithm>
#include <cstdio>
#include <cstdlib>
#include <cstring>
#include <map>
#include <mutex>
#include <sstream>
#include <string>
#include <tuple>
#include <unordered_map>
#include <vector>

#include "ami_internal.hpp"
#include "jit.hpp"

namespace ami {

namespace {

// The reverse sweep (cotangents and their scatters) lets the compiler fuse
// its multiply-add pairs; the forward values are computed outside it, with
// every fused multiply-add written out, so they do not change.
const char *const kReverseContract = "#pragma clang fp contract(fast)\n";

// First statement of every function that reaches the workspace: the lane's
// byte offset through an empty asm in the accesses' own basic block, where the
// compiler sees its zero extension and takes it as the 32-bit offset of a
// scalar base (else each load adds a 64-bit vector address).
const char *const kOffsetHere = "  AMI_OPAQUE(off);\n";

std::string num(double v) {
    char b[40];
    std::snprintf(b, sizeof(b), "%.17g", v);
    std::string s(b);
    if (s.find_first_of(".eEn") == std::string::npos) s += ".0";
    return s;
}

// A sum of signed products of leaves, sum_t c_t prod_{l in t} F_l, written as
// nested multiply-adds (a greedy multivariate Horner scheme): the leaf a that
// occurs in the most terms (the lowest index among equals) is factored out,
// F_a * (the terms holding a, one a removed) + (the other terms), and both
// parts are nested the same way.  Each step is one fma (a mul or an add where
// a part is zero or a unit constant); terms with equal leaf multisets merge,
// and a sub-sum met again (or its negative) reuses the node that holds it.
// The nodes are built first (horner_build), then written out (horner_emit:
// const double h<k> of the enclosing block).
// Nesting is most of what generating a large solution's source costs (2804 terms:
// ordered maps of printed keys, merging anew at every step, took 12 ms for all
// group sums, this form 2), so leaf lists are u16strings (up to seven
// leaves without an allocation) and the keys of sub-sums their bits.
struct HornerTerm {
    double c;
    std::u16string leaves;   // a multiset (a leaf may repeat)
};

bool leaves_less(const HornerTerm &x, const HornerTerm &y) { return x.leaves < y.leaves; }

// The terms with their leaf multisets sorted, equal multisets merged and
// zero coefficients dropped.
std::vector<HornerTerm> merged_terms(std::vector<HornerTerm> ts) {
    for (HornerTerm &t : ts) std::sort(t.leaves.begin(), t.leaves.end());
    std::sort(ts.begin(), ts.end(), leaves_less);
    std::vector<HornerTerm> m;
    m.reserve(ts.size());
    for (HornerTerm &t : ts) {
        if (!m.empty() && m.back().leaves == t.leaves) m.back().c += t.c;
        else m.push_back(std::move(t));
    }
    m.erase(std::remove_if(m.begin(), m.end(), [](const HornerTerm &t) { return t.c == 0.0; }), m.end());
    return m;
}

// The merged sum's key up to sign (`flip`: its first coefficient is negative
// and the key is that of the negated sum): every coefficient's bits, the number
// of leaves and the leaves.
std::u16string sum_key(const std::vector<HornerTerm> &m, bool &flip) {
    flip = m[0].c < 0.0;
    std::u16string key;
    key.reserve(m.size() * (5 + m[0].leaves.size()));
    for (const HornerTerm &t : m) {
        const double c = flip ? -t.c : t.c;
        char16_t bits[4];
        std::memcpy(bits, &c, sizeof(c));
        key.append(bits, 4);
        key.push_back(static_cast<char16_t>(t.leaves.size()));
        key += t.leaves;
    }
    return key;
}

// The sub-sums of one nesting met so far (up to sign), and its counts per leaf
// (zero between uses).
template <typename Value>
struct NestMemo {
    std::unordered_map<std::u16string, Value> found;
    std::vector<int> count;
};

// One step of the nesting of merged terms: the leaf in the most terms (the lowest
// index among equals) and the terms split into those holding it (one occurrence
// removed, sorted again) and the others.  Both parts are merged: terms that
// differ still differ without one leaf.
int split_on_shared_leaf(std::vector<HornerTerm> m, std::vector<int> &count, std::vector<HornerTerm> &with,
                         std::vector<HornerTerm> &without) {
    int a = -1, best = 0;
    for (const HornerTerm &t : m)
        for (size_t j = 0; j < t.leaves.size(); ++j) {
            if (j > 0 && t.leaves[j] == t.leaves[j - 1]) continue;
            const int l = t.leaves[j];
            if (static_cast<size_t>(l) >= count.size()) count.resize(static_cast<size_t>(l) + 1, 0);
            const int n = ++count[l];               // terms holding l
            if (n > best || (n == best && l < a)) {
                a = l;
                best = n;
            }
        }
    for (HornerTerm &t : m)
        for (char16_t l : t.leaves) count[l] = 0;
    with.reserve(static_cast<size_t>(best));
    without.reserve(m.size() - static_cast<size_t>(best));
    for (HornerTerm &t : m) {
        const size_t at = t.leaves.find(static_cast<char16_t>(a));
        if (at == std::u16string::npos) {
            without.push_back(std::move(t));
        } else {
            t.leaves.erase(at, 1);
            with.push_back(std::move(t));
        }
    }
    std::sort(with.begin(), with.end(), leaves_less);
    return a;
}

// A value of the nesting: zero, a number, a leaf or a node, with a sign.
struct HRef {
    enum Kind { ZERO, CONST, LEAF, NODE } kind = ZERO;
    double c = 0.0;   // CONST
    int idx = -1;     // LEAF: the leaf; NODE: the node
    bool neg = false;
};

// Node k holds F_a * w + u (w not zero).
struct HNode {
    int a;
    HRef w, u;
};

HRef href_negated(HRef r) {
    if (r.kind == HRef::CONST) r.c = -r.c;
    else if (r.kind != HRef::ZERO) r.neg = !r.neg;
    return r;
}

// The nodes of the merged terms m.
HRef horner_nodes(std::vector<HornerTerm> m, std::vector<HNode> &nodes, NestMemo<HRef> &memo) {
    HRef r;
    if (m.empty()) return r;
    if (m.size() == 1 && m[0].leaves.empty()) {
        r.kind = HRef::CONST;
        r.c = m[0].c;
        return r;
    }
    bool flip;
    std::u16string key = sum_key(m, flip);
    if (const auto it = memo.found.find(key); it != memo.found.end())
        return flip ? href_negated(it->second) : it->second;
    std::vector<HornerTerm> with, without;
    const int a = split_on_shared_leaf(std::move(m), memo.count, with, without);
    const HRef w = horner_nodes(std::move(with), nodes, memo);
    const HRef u = horner_nodes(std::move(without), nodes, memo);
    if (w.kind == HRef::ZERO) {
        r = u;
    } else if (w.kind == HRef::CONST && (w.c == 1.0 || w.c == -1.0) && u.kind == HRef::ZERO) {
        r.kind = HRef::LEAF;           // +-F_a itself
        r.idx = a;
        r.neg = w.c < 0.0;
    } else {
        nodes.push_back(HNode{a, w, u});
        r.kind = HRef::NODE;
        r.idx = static_cast<int>(nodes.size()) - 1;
    }
    memo.found.emplace(std::move(key), flip ? href_negated(r) : r);
    return r;
}

// The nesting of sum_t c_t prod F over the given terms: its nodes and value.
HRef horner_build(std::vector<HornerTerm> ts, std::vector<HNode> &nodes) {
    NestMemo<HRef> memo;
    return horner_nodes(merged_terms(std::move(ts)), nodes, memo);
}

template <typename LeafName>
std::string href_name(const HRef &r, const LeafName &leaf_name) {   // without its sign
    if (r.kind == HRef::LEAF) return leaf_name(r.idx);
    if (r.kind == HRef::NODE) return "h" + std::to_string(r.idx);
    return r.kind == HRef::CONST ? num(r.c) : std::string("0.0");
}

template <typename LeafName>
std::string href_expr(const HRef &r, const LeafName &leaf_name) {
    if (r.kind == HRef::CONST || r.kind == HRef::ZERO) return href_name(r, leaf_name);
    return r.neg ? "(-" + href_name(r, leaf_name) + ")" : href_name(r, leaf_name);
}

// The nodes as "const double h<k> = ...;" (one fma, mul or add each).
template <typename LeafName>
void horner_emit(const std::vector<HNode> &nodes, const LeafName &leaf_name, std::ostream &o) {
    for (size_t k = 0; k < nodes.size(); ++k) {
        const HNode &n = nodes[k];
        const std::string fa = leaf_name(n.a);
        std::string rhs;
        if (n.w.kind == HRef::CONST) {
            if (n.w.c == 1.0 || n.w.c == -1.0) rhs = href_expr(n.u, leaf_name) + (n.w.c < 0 ? " - " : " + ") + fa;
            else if (n.u.kind == HRef::ZERO) rhs = num(n.w.c) + " * " + fa;
            else rhs = "fma(" + num(n.w.c) + ", " + fa + ", " + href_expr(n.u, leaf_name) + ")";
        } else {
            const std::string sfa = n.w.neg ? "-" + fa : fa;
            const std::string wn = href_name(n.w, leaf_name);
            if (n.u.kind == HRef::ZERO) rhs = (n.w.neg ? "(-" + fa + ")" : fa) + " * " + wn;
            else rhs = "fma(" + sfa + ", " + wn + ", " + href_expr(n.u, leaf_name) + ")";
        }
        o << "    const double h" << k << " = " << rhs << ";\n";
    }
}

// The same greedy nesting for a sum of products whose factors may be complex:
// sum_g prod_{k in g} z_k with complex reciprocals z_k and one real factor
// per product (its group sum, read from memory).  Values are zero, a number,
// a real or a complex pair of expressions; each step L * W + U is written out
// with fma and the kinds of its operands (a complex product fused into the
// addend: re = fma(lr, wr, fma(-li, wi, ur))).
struct CVal {
    enum Kind { ZERO, CONST, REAL, CPLX } kind = ZERO;
    double c = 0.0;
    std::string re, im;   // expressions: a name, "(-name)" or a number
};

std::string neg_expr(const std::string &e) {
    if (e.size() > 3 && e.compare(0, 2, "(-") == 0 && e.back() == ')') return e.substr(2, e.size() - 3);
    return "(-" + e + ")";
}

CVal cnegated(CVal v) {
    if (v.kind == CVal::CONST) v.c = -v.c;
    if (v.kind == CVal::REAL || v.kind == CVal::CPLX) v.re = neg_expr(v.re);
    if (v.kind == CVal::CPLX) v.im = neg_expr(v.im);
    return v;
}

// products (sign, x, y) added to an addend: nested fma, or a product alone
std::string fused(const std::vector<std::tuple<bool, std::string, std::string>> &prods, const std::string &addend) {
    std::string acc = addend;
    for (auto it = prods.rbegin(); it != prods.rend(); ++it) {
        const auto &[negp, x, y] = *it;
        const std::string xs = negp ? neg_expr(x) : x;
        acc = acc.empty() ? xs + " * " + y : "fma(" + xs + ", " + y + ", " + acc + ")";
    }
    return acc;
}

using CMemo = NestMemo<CVal>;

// leaf(a) gives the value of factor a (a REAL or CPLX CVal of names); the terms
// m are merged
template <typename Leaf>
CVal horner_c_merged(std::vector<HornerTerm> m, const Leaf &leaf, std::ostream &o, int &temps, CMemo &memo) {
    CVal r;
    if (m.empty()) return r;
    if (m.size() == 1 && m[0].leaves.empty()) {
        r.kind = CVal::CONST;
        r.c = m[0].c;
        return r;
    }
    bool flip;
    std::u16string key = sum_key(m, flip);
    if (const auto it = memo.found.find(key); it != memo.found.end()) return flip ? cnegated(it->second) : it->second;
    std::vector<HornerTerm> with, without;
    const int a = split_on_shared_leaf(std::move(m), memo.count, with, without);
    const CVal w = horner_c_merged(std::move(with), leaf, o, temps, memo);
    const CVal u = horner_c_merged(std::move(without), leaf, o, temps, memo);
    const CVal L = leaf(a);
    if (w.kind == CVal::ZERO) {
        r = u;
    } else {
        // the product L * w as real and imaginary lists of (sign, x, y), or a
        // plain (signed) expression where w is a unit
        using Prods = std::vector<std::tuple<bool, std::string, std::string>>;
        Prods pre, pim;
        std::string plain_re, plain_im;
        const bool lc = L.kind == CVal::CPLX;
        bool cplx = lc;
        if (w.kind == CVal::CONST) {
            if (w.c == 1.0 || w.c == -1.0) {
                plain_re = w.c < 0 ? neg_expr(L.re) : L.re;
                if (lc) plain_im = w.c < 0 ? neg_expr(L.im) : L.im;
            } else {
                pre.emplace_back(false, num(w.c), L.re);
                if (lc) pim.emplace_back(false, num(w.c), L.im);
            }
        } else if (w.kind == CVal::REAL) {
            pre.emplace_back(false, L.re, w.re);
            if (lc) pim.emplace_back(false, L.im, w.re);
        } else {
            cplx = true;
            if (lc) {
                pre.emplace_back(false, L.re, w.re);
                pre.emplace_back(true, L.im, w.im);
                pim.emplace_back(false, L.re, w.im);
                pim.emplace_back(false, L.im, w.re);
            } else {
                pre.emplace_back(false, L.re, w.re);
                pim.emplace_back(false, L.re, w.im);
            }
        }
        cplx = cplx || u.kind == CVal::CPLX;
        std::string ure, uim;
        if (u.kind == CVal::CONST) ure = num(u.c);
        if (u.kind == CVal::REAL || u.kind == CVal::CPLX) ure = u.re;
        if (u.kind == CVal::CPLX) uim = u.im;
        auto part = [&](const Prods &pr, const std::string &plain, const std::string &add) -> std::string {
            if (!pr.empty()) return fused(pr, add);
            if (plain.empty()) return add;                    // nothing of L * w here
            if (add.empty()) return plain;
            return add + " + " + plain;
        };
        const std::string ere = part(pre, plain_re, ure);
        const std::string eim = cplx ? part(pim, plain_im, uim) : std::string();
        auto temp = [&](const std::string &e) {
            if (e.empty()) return std::string("0.0");
            const bool simple = e.find_first_of(" (") == std::string::npos || (e.compare(0, 2, "(-") == 0 &&
                                                                               e.find(' ') == std::string::npos);
            if (simple) return e;                              // a name or a negated name
            const std::string n = "c" + std::to_string(temps++);
            o << "    const double " << n << " = " << e << ";\n";
            return n;
        };
        r.kind = cplx ? CVal::CPLX : CVal::REAL;
        r.re = temp(ere);
        if (cplx) r.im = temp(eim);
    }
    memo.found.emplace(std::move(key), flip ? cnegated(r) : r);
    return r;
}

template <typename Leaf>
CVal horner_c(std::vector<HornerTerm> ts, const Leaf &leaf, std::ostream &o, int &temps, CMemo &memo) {
    return horner_c_merged(merged_terms(std::move(ts)), leaf, o, temps, memo);
}

// sum_i c_i v[i] over the non-zero coefficients, in index order: "+-v" for
// unit coefficients, fma for others; "0.0" when every coefficient is zero.
struct Lin {
    std::string expr;
    void add(double c, const std::string &v) {
        if (c == 0.0) return;
        if (expr.empty()) {
            if (c == 1.0) expr = v;
            else if (c == -1.0) expr = "(-" + v + ")";
            else expr = "(" + num(c) + " * " + v + ")";
        } else {
            if (c == 1.0) expr = "(" + expr + " + " + v + ")";
            else if (c == -1.0) expr = "(" + expr + " - " + v + ")";
            else expr = "fma(" + num(c) + ", " + v + ", " + expr + ")";
        }
    }
    std::string str() const { return expr.empty() ? "0.0" : expr; }
};

std::string idx(const char *a, int i) { return std::string(a) + "[" + std::to_string(i) + "]"; }

// Groups per chunk of the adjoint's frequency pass for large solutions (the
// cotangents of a chunk's denominators are gathered in registers).
constexpr int kAdjChunkGroups = 2;
// Whether each chunk forms the reciprocals of its own denominators (else all
// of them are formed once per frequency row and held through the chunks).
constexpr bool kAdjChunkOwnDens = true;
// Terms per nested part of a group in the adjoint's leaf pass, and parts
// between scheduling fences.
constexpr int kAdjLeafPartTerms = 32;
constexpr int kAdjLeafFenceParts = 1;
// Terms per nested part of a group in the block adjoint's leaf sweep.
constexpr int kBlockPartTerms = 32;
// The block adjoints' waves for one frequency row and for several are copies apart
// above this many terms: the rows' cotangents of group sums overflow the registers
// there, and one copy for both spills in the one-row path too (2804 terms, 2 10^5
// samples: one row 189 us apart and 204 in one, four rows 607 and 658).  Below,
// one copy takes two thirds of the compilation (560 terms at complex energies 11
// -> 6 s) and of the code, and no more time (560 terms: 77 and 77 us, four rows 136
// and 134; complex 137 and 135, 217 and 204; 264 terms complex 105 and 98).
constexpr int kBlockRowsApartTerms = 1024;
// Groups of a wave above which the real block adjoint for several rows takes eight
// waves for four: their cotangents stay in registers through the rows, beside four
// values for each denominator (2804 terms, 31 groups of a wave, 10^5 samples: two
// rows 214 us with four waves, 170 with eight, 16 rows 1075 and 555, where the passes
// take 861; 21 groups: four rows 181 and 166, 2054 terms 174 and 178).
constexpr int kBlockRowGroups = 24;

// Values a row of the one-pass forwards holds (group sums and reciprocals with
// their arguments), up to which it takes two rows at a time.  Two rows' values
// cost registers: at complex energies 264 terms (168 values) fell from two waves
// per SIMD to one (252 -> 292 VGPRs; 16 rows of 2 10^5 samples 88 us a row at a time,
// 100 two), and nothing above these sizes gained.  Below, 16 rows of 10^6 order-2
// samples 57.4 us and 54.8.
constexpr int kPairRowsValues = 40, kPairRowsValuesC = 64;

}  // namespace

bool jit_prefers_two_pass(const AmiTerms *t) {
    const Tables &tb = t->tab;
    return tb.T > kJitMaxTerms || 2 * tb.G + 4 * tb.D > 128;
}

bool jit_prefers_block_adjoint(const AmiTerms *t) {
    const Tables &tb = t->tab;
    return tb.T > kJitAutoAdjointTerms || tb.L + 4 * tb.G + 4 * tb.D + 2 * t->n_eps > 100;
}

bool jit_prefers_complex_block(const AmiTerms *t, bool one_row) {
    const Tables &tb = t->tab;
    if (tb.T <= kJitAutoComplexBlockTermsOneRow) return false;
    return one_row || tb.T > kJitAutoComplexBlockTerms ||
           (tb.T <= kJitAutoAdjointTerms && 4 * tb.G + 6 * tb.D > 80);
}

bool jit_supported(const AmiTerms *t, bool hub, std::string *why, bool two_pass) {
    const Tables &tb = t->tab;
    auto no = [&](const std::string &m) {
        if (why) *why = m;
        return false;
    };
    if (tb.L < 1 || tb.G < 1) return no("solution without leaves");
    if (t->n_eps > kMaxEpsDev) return no("more than 16 energies");
    if (t->n_ext > kMaxExt) return no("more than 4 external slots");
    if (hub && t->n_g != t->n_eps) return no("momentum input needs one energy per line");
    const int max_terms = two_pass ? kJitTwoPassMaxTerms : kJitMaxTerms;
    if (tb.T > max_terms) return no("more than " + std::to_string(max_terms) + " terms");
    return true;
}

bool jit_adjoint_passes_supported(const AmiTerms *t, bool hub, std::string *why) {
    return jit_supported(t, hub, why, true);
}

namespace {

// Adjoint values parked in LDS instead of registers: the momentum chain
// rule's 3 per line, and the leaf derivatives while both fit in 40 doubles
// per lane (two resident blocks of 256 lanes per CU).
constexpr int kParkBudget = 40;
int park_chain(const AmiTerms *t, bool hub) { return hub ? 3 * t->n_g : 0; }
bool park_dv(const AmiTerms *t, bool hub) {
    if (const char *e = std::getenv("AMIGPU_JIT_PARK_DV")) return std::atoi(e) != 0;   // tuning override
    for (int o : t->tab.leaf_order)
        if (o > 0) return false;              // Taylor-coefficient leaves: their slopes stay in registers
    return park_chain(t, hub) + t->tab.L <= kParkBudget;
}
int park_cols(const AmiTerms *t, bool hub) { return park_chain(t, hub) + (park_dv(t, hub) ? t->tab.L : 0); }

// occupancy floor of the one-pass adjoint (waves per SIMD; 0: none),
// AMIGPU_JIT_ADJ_WAVES overriding the default of two: an adjoint that would
// take more than 256 VGPRs runs at two waves with a few spills rather than at
// one (order-4 topologies of 40-52 terms: 0.099-0.105 -> 0.081-0.086 ms per
// 10^6-sample step)
// Terms per nested part in the complex adjoint's leaf pass (each node holds
// a complex value and a complex cotangent); AMIGPU_JIT_CADJ_PART overrides.
int cadj_part_terms() {
    const char *e = std::getenv("AMIGPU_JIT_CADJ_PART");
    const int v = e ? std::atoi(e) : 0;
    return v >= 1 && v <= 64 ? v : 64;
}

// occupancy floor of the complex adjoint's leaf pass (one wave: its spills
// at two cost more than the occupancy, 196 terms 1.73 -> 1.25 ms, 560 terms
// 2.63 -> 1.90 ms per 10^6-sample step); AMIGPU_JIT_CADJL_WAVES overrides
int cadjl_waves() {
    const char *e = std::getenv("AMIGPU_JIT_CADJL_WAVES");
    const int v = e ? std::atoi(e) : -1;
    return v >= 0 && v <= 8 ? v : 1;
}

}  // namespace

// Terms per part of the one-pass adjoint's nested leaf-cotangent sweep when
// AMIGPU_JIT_NESTED_COTANGENTS names it (0: per-term products), else -1.
int jit_nested_override() {
    const char *e = std::getenv("AMIGPU_JIT_NESTED_COTANGENTS");
    if (!e) return -1;
    const int v = std::atoi(e);
    return v >= 0 && v <= 64 ? v : 0;
}

namespace {
// ---- block adjoint: a block's waves split the work of 64 samples -----------
//
// The split of a solution over the waves of a block: wave w takes the groups
// [first[w], first[w + 1]) (consecutive in canonical order, so that a wave's
// groups share denominators), balanced by the operations of their nested sums,
// their reverse sweep and their products.
struct BlockPlan {
    int waves = 0;                        // 0: no split worth having
    std::vector<int> first;
    int max_groups = 0;
    double imbalance = 1.0;               // largest wave's cost over the mean
    // the wave that forms every value whole, as the forward does (-1: each wave
    // its groups' part, added up at the end of a row)
    int value_wave = -1;
    // reduction of the leaf cotangents over the waves, in rounds: round r holds
    // the leaves [round[r], round[r + 1]); slot[l][w] is wave w's column of leaf l
    // in its round (-1: the wave does not read the leaf)
    std::vector<int> round;
    std::vector<std::vector<int>> slot;
    // LDS columns (64 doubles each): energies, a row's sums, slopes (-1: formed
    // again where they are needed), then a region that holds leaves and group
    // sums (-1: in the wave's registers), then the reductions
    int c_e = 0, c_acc = 0, c_slope = -1, c_union = 0, c_leaf = 0, c_group = -1, columns = 0;
};

// Columns of LDS of one of two blocks on a CU, and of a block alone (160 KB
// less a margin).
constexpr int kBlockHalfColumns = 158;
constexpr int kBlockMaxColumns = 316;
// Groups whose sums and cotangents a wave holds in registers at most.
constexpr int kBlockRegisterGroups = 12;

// Consecutive ranges of groups for `waves` waves (first[w] .. first[w + 1]) with
// the smallest largest cost.
bool split_groups(const std::vector<double> &cost, int waves, std::vector<int> &out) {
    const int G = static_cast<int>(cost.size());
    double total = 0.0;
    for (double c : cost) total += c;
    // the smallest bound under which consecutive ranges fit `waves` waves
    auto ranges = [&](double bound, std::vector<int> &first) {
        first.assign(1, 0);
        double c = 0.0;
        for (int g = 0; g < G; ++g) {
            const int left_waves = waves - static_cast<int>(first.size());
            if (g > first.back() && (c + cost[g] > bound || G - g <= left_waves)) {
                if (left_waves == 0) return false;
                first.push_back(g);
                c = 0.0;
            }
            c += cost[g];
        }
        while (static_cast<int>(first.size()) < waves) first.push_back(G);
        first.push_back(G);
        return c <= bound;
    };
    double lo = total / waves, hi = total;
    std::vector<int> first;
    for (int it = 0; it < 40; ++it) {
        const double mid = 0.5 * (lo + hi);
        if (ranges(mid, first)) hi = mid;
        else lo = mid;
    }
    return ranges(hi, out);
}

// Nodes of each group's nested sum, what its share of a wave's work is judged by;
// counted once per handle (every plan and every block kernel's source asks).
const std::vector<int> &group_nest_sizes(const AmiTerms *t) {
    std::call_once(t->nest_once, [t] {
        const Tables &tb = t->tab;
        for (int g = 0; g < tb.G; ++g) {
            std::vector<HornerTerm> ts;
            for (int ti = tb.group_start[g]; ti < tb.group_start[g + 1]; ++ti) {
                HornerTerm h{tb.term_sign[ti], {}};
                for (int j = 0; j < t->n_int; ++j)
                    h.leaves.push_back(tb.term_leaf[static_cast<size_t>(ti) * t->n_int + j]);
                ts.push_back(std::move(h));
            }
            std::vector<HNode> nodes;
            horner_build(std::move(ts), nodes);
            t->nest_sizes.push_back(static_cast<int>(nodes.size()));
        }
    });
    return t->nest_sizes;
}

BlockPlan block_plan(const AmiTerms *t, bool hub, bool cplx, int waves) {
    const Tables &tb = t->tab;
    const int G = tb.G, L = tb.L, ni = t->n_int, ne = t->n_eps, nx = t->n_ext;
    const int cw = cplx ? 2 : 1;          // columns of a value
    BlockPlan p;
    if (waves < 2 || G < waves) return p;
    std::vector<double> cost(static_cast<size_t>(G));
    double total = 0.0;
    const std::vector<int> &nest_sizes = group_nest_sizes(t);
    for (int g = 0; g < G; ++g) {
        const int dens = tb.group_den_start[g + 1] - tb.group_den_start[g];
        cost[g] = 3.6 * (cplx ? 3.5 : 1.0) * static_cast<double>(nest_sizes[g]) + 3.0 * dens + 8.0;
        total += cost[g];
    }
    if (!split_groups(cost, waves, p.first)) return p;
    double most = 0.0;
    for (int w = 0; w < waves; ++w) {
        double c = 0.0;
        for (int g = p.first[w]; g < p.first[w + 1]; ++g) c += cost[g];
        most = std::max(most, c);
        p.max_groups = std::max(p.max_groups, p.first[w + 1] - p.first[w]);
    }
    p.imbalance = most * waves / total;
    // Real solutions whose forward adds the values group by group (up to the
    // one-pass adjoint's automatic size): the values are the forward's bit for bit,
    // formed by one wave from every group's sum in its column (its own groups'
    // products it has anyway), the wave with the least work of its own.  76 terms, a
    // step of 2 10^5 momenta: 39.0 us with the values added up from the waves'
    // parts, 39.7 this way (four rows 59.0 and 60.4).
    const bool exact = !cplx && tb.T <= kJitAutoAdjointTerms;
    if (exact) {
        if (p.max_groups > kBlockRegisterGroups) return p;
        double least = total;
        for (int w = 0; w < waves; ++w) {
            double c = 0.0;
            for (int g = p.first[w]; g < p.first[w + 1]; ++g) c += cost[g];
            if (c < least) {
                least = c;
                p.value_wave = w;
            }
        }
    }
    // Two blocks per CU hide each other's barriers and start, so four waves in
    // half the LDS where the solution fits there, else eight in all of it.
    // Columns that are optional, in the order of what they save: the group sums
    // (a wave with many groups spills without them), the slopes.
    const int limit = waves <= 4 ? kBlockHalfColumns : kBlockMaxColumns;
    bool fits = false;
    for (int option = 3; option >= 0 && !fits; --option) {
        const bool group = option & 2, slope = option & 1;
        if (!group && (exact || p.max_groups > kBlockRegisterGroups)) continue;
        p.c_e = 0;
        p.c_acc = cw * ne;
        p.c_slope = slope ? p.c_acc + (2 + 2 * nx) * waves : -1;
        p.c_union = p.c_acc + (2 + 2 * nx) * waves + (slope ? cw * L : 0);
        p.c_leaf = p.c_union;
        p.c_group = group ? p.c_leaf + cw * L : -1;
        p.columns = p.c_leaf + cw * L + (group ? cw * G : 0);
        // the reduction of the energies' cotangents, on the momentum input
        // beside the lines'; the staged gradient rows lie over the first columns
        p.columns = std::max(p.columns, p.c_union + (cw * ne + 1) * waves + (hub ? 2 * ne + 2 * waves : 0));
        p.columns = std::max(p.columns, hub ? 2 * ni + 1 : cw * ne + 1);
        fits = p.columns <= limit;
    }
    if (!fits) return p;
    // rounds of the leaf reduction within the columns there are
    std::vector<std::vector<char>> reads(static_cast<size_t>(L), std::vector<char>(static_cast<size_t>(waves), 0));
    for (int w = 0; w < waves; ++w)
        for (int g = p.first[w]; g < p.first[w + 1]; ++g)
            for (int ti = tb.group_start[g]; ti < tb.group_start[g + 1]; ++ti)
                for (int j = 0; j < ni; ++j) reads[tb.term_leaf[static_cast<size_t>(ti) * ni + j]][w] = 1;
    {
        p.round.assign(1, 0);
        p.slot.assign(static_cast<size_t>(L), std::vector<int>(static_cast<size_t>(waves), -1));
        int used = 0, top = 0;
        for (int l = 0; l < L; ++l) {
            int n = 0;
            for (int w = 0; w < waves; ++w) n += reads[l][w] ? cw : 0;
            if (used > 0 && p.c_union + used + n > limit) {
                p.round.push_back(l);
                used = 0;
            }
            for (int w = 0; w < waves; ++w)
                if (reads[l][w]) {
                    p.slot[l][w] = used;
                    used += cw;
                }
            top = std::max(top, used);
        }
        p.round.push_back(L);
        p.columns = std::max(p.columns, p.c_union + top);
    }
    if (p.columns > limit) return p;
    p.waves = waves;
    return p;
}

}  // namespace

// Waves per block of the block forward: four, two blocks per CU, where energies,
// leaves and group sums fit half the LDS, else eight in all of it.
int jit_block_forward_waves(const AmiTerms *t) {
    for (int o : t->tab.leaf_order)
        if (o > 0) return 0;              // Taylor-coefficient leaves: the two passes over a workspace
    if (t->tab.T > kJitTwoPassMaxTerms) return 0;
    const int columns = t->n_eps + t->tab.L + t->tab.G;
    const int waves = columns <= kBlockHalfColumns ? 4 : columns <= kBlockMaxColumns ? 8 : 0;
    return t->tab.G >= 2 * waves ? waves : 0;
}

// Waves per block of the block adjoint (AMIGPU_JIT_BLOCK_WAVES overrides): as
// few as leave each wave a part that, with one row, fits its registers, since every
// wave more is another partner at each barrier.  Real energies: two up to 200 terms (76
// terms, 2 10^5 samples: 38.8 us a step, four waves 40.8; 136 terms 41.6 and
// 50.4; 264 terms at four rows and 5 10^4 samples: 38.0 and 35.8), else four (560
// terms 78.7, 76.9 and with eight 119; 2804 terms 233, 190 and 233).  Complex
// energies, whose parts are twice as large: four (136 terms 78.7 and 65.8, 560
// terms 168, 134 and with eight 172).  Eight, alone on its CU, where the columns
// of four do not fit half its LDS.
static int choose_block_waves(const AmiTerms *t, bool hub, bool cplx) {
    for (int o : t->tab.leaf_order)
        if (o > 0) return 0;              // Taylor-coefficient leaves: the passes over a workspace
    if (t->tab.T > kJitTwoPassMaxTerms) return 0;
    if (const char *e = std::getenv("AMIGPU_JIT_BLOCK_WAVES")) {
        const int v = std::atoi(e);
        return v == 2 || v == 4 || v == 8 ? block_plan(t, hub, cplx, v).waves : 0;
    }
    for (int w : {2, 4, 8}) {
        if (w == 2 && (cplx || t->tab.T > 200)) continue;
        const BlockPlan p = block_plan(t, hub, cplx, w);
        if (p.waves > 0 && p.imbalance <= 1.6) return w;
    }
    return 0;
}

bool jit_block_rows_apart(const AmiTerms *t) { return t->tab.T > kBlockRowsApartTerms; }

int jit_block_waves(const AmiTerms *t, bool hub, bool cplx, bool several) {
    std::lock_guard<std::mutex> lock(t->plan_mu);
    int &w = t->block_waves[cplx ? 2 : hub ? 1 : 0];
    if (w < 0) w = choose_block_waves(t, hub, cplx);
    if (cplx || !several || w != 4 || !jit_block_rows_apart(t)) return w;
    int &s = t->block_waves[hub ? 4 : 3];
    if (s < 0 && std::getenv("AMIGPU_JIT_BLOCK_WAVES")) s = w;
    if (s < 0)
        s = block_plan(t, hub, false, 4).max_groups > kBlockRowGroups && block_plan(t, hub, false, 8).waves > 0 ? 8 : 4;
    return s;
}

namespace {

int adj_waves() {
    const char *e = std::getenv("AMIGPU_JIT_ADJ_WAVES");
    if (!e) return 2;
    const int v = std::atoi(e);
    return (v >= 0 && v <= 8) ? v : 2;
}

}  // namespace

// 256 lanes while the adjoint's parked columns fit in 80 KB per block (two
// blocks per CU), else 128
int jit_block(const AmiTerms *t, bool hub) { return park_cols(t, hub) * 256 * 8 <= 80 * 1024 ? 256 : 128; }

std::string jit_source(const AmiTerms *t, bool hub, int kernels, int nested_part) {
    if (nested_part < 0) nested_part = std::max(0, jit_nested_override());
    const Tables &tb = t->tab;
    const int ne = t->n_eps, ni = t->n_int, ng = t->n_g, nx = t->n_ext, nf = t->n_freq;
    // a solution whose terms hold no denominators gets one phantom
    // denominator equal to 1 (no group uses it), so no array is empty
    const int L = tb.L, D = std::max(tb.D, 1), G = tb.G;
    auto gbegin = [&](int g) { return tb.group_den_start[g]; };
    auto gend = [&](int g) { return tb.group_den_start[g + 1]; };
    const int nc = ne + nx;
    std::ostringstream o;
    o << "// generated: specialized AMI evaluator, " << tb.T << " terms, " << L << " leaves, " << D
      << " denominators, " << G << " groups\n";
    o << "#define AMI_JIT_HUB " << (hub ? "true" : "false") << "\n";
    o << "#define AMI_JIT_KERNELS " << kernels << "\n";
    o << "#define AMI_JIT_BLOCK " << jit_block(t, hub) << "\n";
    o << "#define AMI_JIT_PARK_DV " << (park_dv(t, hub) ? "true" : "false") << "\n";
    o << "#define AMI_JIT_ADJ_WAVES " << adj_waves() << "\n";
    // the complex adjoint (one pass at every size): the same floor up to the
    // one-pass adjoint's automatic size; above it the spills of a two-wave
    // floor cost more than the lost occupancy (196 terms: 1.11 -> 0.86 ms,
    // 560 terms: 6.8 -> 5.7 ms per 10^6-sample step at one wave)
    o << "#define AMI_JIT_CADJ_WAVES " << (tb.T <= kJitAutoAdjointTerms ? adj_waves() : 1) << "\n";
    // the leaf pass of the complex adjoint in passes (its values per leaf and
    // node are complex, twice the real pass's)
    o << "#define AMI_JIT_CADJL_WAVES " << cadjl_waves() << "\n";
    o << "#include \"kargs.hpp\"\n";
    o << "namespace amijit {\n";
    o << "constexpr int NE = " << ne << ", NI = " << ni << ", NG = " << ng << ", NX = " << nx << ";\n";
    o << "constexpr int L = " << L << ", D = " << D << ", G = " << G << ";\n";
    // the forward values from sum_g FT_g R_g nested over the reciprocals
    // (groups_combine) above the adjoint's automatic size, group by group below
    const bool nested_groups = tb.T > kJitAutoAdjointTerms;
    if (kernels & (1 | 8))
        o << "constexpr bool kPairRows = " << (2 * G + 4 * D <= kPairRowsValues ? "true" : "false")
          << ", kPairRowsC = " << (4 * G + 6 * D <= kPairRowsValuesC ? "true" : "false") << ";\n";
    o << "constexpr bool kNestedGroups = " << (nested_groups ? "true" : "false") << ";\n";
    o << "constexpr bool kBose[L] = {";
    for (int l = 0; l < L; ++l) o << (l ? ", " : "") << (tb.leaf_sigma[l] < 0 ? "true" : "false");
    o << "};\n";
    const std::string NXA = "(NX > 0 ? NX : 1)", NIA = "(NI > 0 ? NI : 1)", NGA = "(NG > 0 ? NG : 1)";

    // momentum lines: K_j = sum_l alpha_jl k_l over the loops, then + q of the external slots
    o << "__device__ __forceinline__ void lines(const double (&kx)[" << NIA << "], const double (&ky)[" << NIA
      << "], const double *q, double (&Kx)[" << NGA << "], double (&Ky)[" << NGA << "]) {\n";
    if (hub) {
        for (int j = 0; j < ng; ++j) {
            Lin ax, ay;
            for (int l = 0; l < ni; ++l) {
                const double a = tb.line_alpha[static_cast<size_t>(j) * nf + l];
                ax.add(a, idx("kx", l));
                ay.add(a, idx("ky", l));
            }
            for (int x = 0; x < nx; ++x) {
                const double a = tb.line_alpha[static_cast<size_t>(j) * nf + ni + x];
                ax.add(a, idx("q", 2 * x));
                ay.add(a, idx("q", 2 * x + 1));
            }
            o << "  Kx[" << j << "] = " << ax.str() << ";\n  Ky[" << j << "] = " << ay.str() << ";\n";
        }
    }
    o << "}\n";

    // sin and cos of the line momenta from those of the loop momenta and of
    // q (adjoint): K_j = sum of +-k_l (+-q), folded term by term with
    // sin(A +- b) = sin A cos b +- cos A sin b, cos(A +- b) = cos A cos b -+ sin A sin b
    o << "__device__ __forceinline__ void line_trig(const double (&sx)[" << NIA << "], const double (&cx)[" << NIA
      << "], const double (&sy)[" << NIA << "], const double (&cy)[" << NIA
      << "], const double *qs, const double *qc, double (&Sx)[" << NGA << "], double (&Cx)[" << NGA
      << "], double (&Sy)[" << NGA << "], double (&Cy)[" << NGA << "]) {\n";
    if (hub) {
        o << "  double nS;\n";
        for (int j = 0; j < ng; ++j)
            for (int comp = 0; comp < 2; ++comp) {
                std::vector<std::pair<int, std::pair<std::string, std::string>>> terms;
                for (int l = 0; l < ni; ++l) {
                    const int a = static_cast<int>(tb.line_alpha[static_cast<size_t>(j) * nf + l]);
                    if (a) terms.push_back({a, {idx(comp ? "sy" : "sx", l), idx(comp ? "cy" : "cx", l)}});
                }
                for (int x = 0; x < nx; ++x) {
                    const int a = static_cast<int>(tb.line_alpha[static_cast<size_t>(j) * nf + ni + x]);
                    if (a) terms.push_back({a, {idx("qs", 2 * x + comp), idx("qc", 2 * x + comp)}});
                }
                const std::string S = idx(comp ? "Sy" : "Sx", j), C = idx(comp ? "Cy" : "Cx", j);
                if (terms.empty()) {
                    o << "  " << S << " = 0.0; " << C << " = 1.0;\n";
                    continue;
                }
                for (size_t k = 0; k < terms.size(); ++k) {
                    const int sg = terms[k].first;
                    const std::string &sb = terms[k].second.first, &cb = terms[k].second.second;
                    if (k == 0) {
                        o << "  " << S << " = " << (sg > 0 ? "" : "-") << sb << "; " << C << " = " << cb << ";\n";
                    } else if (sg > 0) {
                        o << "  nS = fma(" << S << ", " << cb << ", " << C << " * " << sb << "); " << C << " = fma("
                          << C << ", " << cb << ", -(" << S << " * " << sb << ")); " << S << " = nS;\n";
                    } else {
                        o << "  nS = fma(" << S << ", " << cb << ", -(" << C << " * " << sb << ")); " << C
                          << " = fma(" << C << ", " << cb << ", " << S << " * " << sb << "); " << S << " = nS;\n";
                    }
                }
            }
        o << "  (void)nS;\n";
    }
    o << "  (void)sx; (void)cx; (void)sy; (void)cy; (void)qs; (void)qc; (void)Sx; (void)Cx; (void)Sy; (void)Cy;\n}\n";

    // leaf arguments x_l = sum_i c_li E_i
    o << "__device__ __forceinline__ void leaf_args(const double (&E)[NE], double (&x)[L]) {\n";
    for (int l = 0; l < L; ++l) {
        Lin s;
        for (int i = 0; i < ne; ++i) s.add(tb.leaf_coef[static_cast<size_t>(l) * ne + i], idx("E", i));
        o << "  x[" << l << "] = " << s.str() << ";\n";
    }
    o << "}\n";

    // group sums FT_g = sum_t s_t prod f, each group in the nested form of
    // horner()
    // leaf names: F[l], or a group's own copy f<l> (opaque copies)
    std::string leaf_prefix = "F[", leaf_suffix = "]";
    auto leaf_name = [&](int l) { return leaf_prefix + std::to_string(l) + leaf_suffix; };
    // the one-pass kernels' functions (and the adjoint's) are emitted when one
    // of those kernels is asked for, or for any solution small enough for them
    // (the host checks compile them); a two-pass source of a large solution
    // holds only what its two kernels use
    const bool small = tb.T <= kJitMaxTerms;
    const bool one_pass = (kernels & (15 | 256)) != 0;
    const bool adj_fns = (kernels & (2 | 256)) || ((kernels & 1) && small);
    // With `opaque`, every group first takes copies of the leaves it reads
    // through an empty asm (no instruction): the compiler then cannot merge
    // equal products of different groups, which for large solutions would
    // keep hundreds of shared products live across the whole function; equal
    // products within a group are still merged.
    auto group_sums_body = [&](const std::string &sink_prefix, const std::string &sink_suffix, bool opaque) {
    for (int g = 0; g < G; ++g) {
        o << "  { double ft;\n";
        leaf_prefix = opaque ? "f" : "F[";
        leaf_suffix = opaque ? "" : "]";
        if (opaque) {
            std::vector<int> used;
            for (int ti = tb.group_start[g]; ti < tb.group_start[g + 1]; ++ti)
                for (int j = 0; j < ni; ++j) used.push_back(tb.term_leaf[static_cast<size_t>(ti) * ni + j]);
            std::sort(used.begin(), used.end());
            used.erase(std::unique(used.begin(), used.end()), used.end());
            for (int l : used)
                o << "    double f" << l << " = F[" << l << "]; AMI_OPAQUE(f" << l << ");\n";
        }
        std::vector<HornerTerm> ts;
        for (int ti = tb.group_start[g]; ti < tb.group_start[g + 1]; ++ti) {
            HornerTerm h{tb.term_sign[ti], {}};
            for (int j = 0; j < ni; ++j) h.leaves.push_back(tb.term_leaf[static_cast<size_t>(ti) * ni + j]);
            ts.push_back(std::move(h));
        }
        std::vector<HNode> nodes;
        const HRef v = horner_build(std::move(ts), nodes);
        horner_emit(nodes, leaf_name, o);
        o << "    ft = " << href_expr(v, leaf_name) << ";\n";
        if (sink_suffix.find("ft)") != std::string::npos) o << "    " << sink_prefix << g << sink_suffix << "; }\n";
        else o << "    " << sink_prefix << g << sink_suffix << " = ft; }\n";
    }
    };
    if (one_pass) {
        o << "__device__ __forceinline__ void group_sums(const double (&F)[L], double (&FT)[G]) {\n";
        group_sums_body("FT[", "]", false);
        o << "}\n";
    }
    // two-pass forward, first pass: each group sum stored as soon as it is formed
    if (kernels & 16) {
        o << "__device__ __forceinline__ void group_sums_store(const double (&F)[L], double *ws, int64_t ld, "
             "uint32_t off) {\n";
        o << kOffsetHere;
        group_sums_body("ami::ws_store(ws, ld, ", ", off, ft)", true);
        o << "}\n";
    }

    // complex group sums (complex energies): each group's sum nested as the
    // real group sums, in complex arithmetic; `store`: each stored to the
    // workspace as soon as it is formed (real part in column g, imaginary part
    // in column G + g; the two-pass complex forward's first pass), the leaves
    // a group reads taken through opaque copies as in group_sums_store
    auto group_sums_c_body = [&](bool store) {
        for (int g = 0; g < G; ++g) {
            o << "  {\n";
            std::vector<HornerTerm> ts;
            for (int ti = tb.group_start[g]; ti < tb.group_start[g + 1]; ++ti) {
                HornerTerm h{tb.term_sign[ti], {}};
                for (int j = 0; j < ni; ++j) h.leaves.push_back(tb.term_leaf[static_cast<size_t>(ti) * ni + j]);
                ts.push_back(std::move(h));
            }
            if (store) {
                std::vector<int> used;
                for (const HornerTerm &h : ts) used.insert(used.end(), h.leaves.begin(), h.leaves.end());
                std::sort(used.begin(), used.end());
                used.erase(std::unique(used.begin(), used.end()), used.end());
                for (int l : used)
                    o << "    double fr" << l << " = Fr[" << l << "], fi" << l << " = Fi[" << l << "]; AMI_OPAQUE(fr" << l
                      << "); AMI_OPAQUE(fi" << l << ");\n";
            }
            auto leaf = [&](int l) {
                CVal v;
                v.kind = CVal::CPLX;
                v.re = store ? "fr" + std::to_string(l) : "Fr[" + std::to_string(l) + "]";
                v.im = store ? "fi" + std::to_string(l) : "Fi[" + std::to_string(l) + "]";
                return v;
            };
            int temps = 0;
            CMemo memo;
            const CVal v = horner_c(ts, leaf, o, temps, memo);
            const std::string re = v.kind == CVal::ZERO ? "0.0" : v.kind == CVal::CONST ? num(v.c) : v.re;
            const std::string im = v.kind == CVal::CPLX ? v.im : "0.0";
            if (store)
                o << "    ami::ws_store(ws, ld, " << g << ", off, " << re << "); ami::ws_store(ws, ld, " << G + g
                  << ", off, " << im << "); }\n";
            else
                o << "    FTr[" << g << "] = " << re << "; FTi[" << g << "] = " << im << "; }\n";
        }
    };
    if (kernels & (8 | 256)) {
        o << "__device__ __forceinline__ void group_sums_c(const double (&Fr)[L], const double (&Fi)[L], double "
             "(&FTr)[G], double (&FTi)[G]) {\n";
        group_sums_c_body(false);
        o << "}\n";
    }
    if (kernels & 512) {
        o << "__device__ __forceinline__ void group_sums_c_store(const double (&Fr)[L], const double (&Fi)[L], "
             "double *ws, int64_t ld, uint32_t off) {\n";
        o << kOffsetHere;
        group_sums_c_body(true);
        o << "}\n";
    }

    // Taylor-coefficient leaves (poles of higher order): T_j = beta^j f^(j) / j!,
    // f^(j) as a polynomial in f and fm = f(-y) (f' = -f fm, fm' = f fm);
    // taylor_expr writes statements that leave T_j of the values named f and m
    // in `dst` (j = 0: f itself)
    auto taylor_expr = [&](int jo, const std::string &dst, const std::string &pad) {
        if (jo == 0) return pad + dst + " = f;\n";
        std::map<std::pair<int, int>, long long> poly{{{1, 0}, 1}};
        for (int step = 0; step < jo; ++step) {
            std::map<std::pair<int, int>, long long> nxt;
            for (const auto &kv : poly) {
                const int a = kv.first.first, b = kv.first.second;
                if (a) nxt[{a, b + 1}] -= a * kv.second;
                if (b) nxt[{a + 1, b}] += b * kv.second;
            }
            poly.clear();
            for (const auto &kv : nxt)
                if (kv.second) poly.insert(kv);
        }
        double fact = 1.0;
        for (int i = 2; i <= jo; ++i) fact *= i;
        std::string scale = "beta";
        for (int i = 1; i < jo; ++i) scale += " * beta";
        std::string out = pad + "{ double acc = 0.0;\n";
        for (const auto &kv : poly) {
            std::string mono;
            for (int i = 0; i < kv.first.first; ++i) mono += (mono.empty() ? "f" : " * f");
            for (int i = 0; i < kv.first.second; ++i) mono += (mono.empty() ? "m" : " * m");
            out += pad + "  acc = fma(" + num(static_cast<double>(kv.second)) + ", " + mono + ", acc);\n";
        }
        out += pad + "  " + dst + " = acc * (" + scale + ") * " + num(1.0 / fact) + "; }\n";
        return out;
    };
    bool taylor = false;
    for (int l = 0; l < L; ++l) taylor = taylor || tb.leaf_order[l] > 0;
    o << "constexpr bool kTaylor = " << (taylor ? "true" : "false") << ";\n";
    o << "__device__ __forceinline__ void taylor_leaves(double (&F)[L], const double (&FM)[L], double beta) {\n";
    for (int l = 0; l < L; ++l) {
        const int jo = tb.leaf_order[l];
        if (jo == 0) continue;
        o << "  { const double f = F[" << l << "], m = FM[" << l << "];\n";
        o << taylor_expr(jo, "F[" + std::to_string(l) + "]", "    ");
        o << "  }\n";
    }
    o << "  (void)FM; (void)beta;\n}\n";
    // the adjoint's derivatives of the leaves of a solution with Taylor
    // coefficients: DX = dT_j/dx = (j + 1) T_(j+1), DB = dT_j/dbeta =
    // (j T_j + x DX) / beta, from the plain leaf pair (f, fm) at x
    o << "__device__ __forceinline__ void taylor_slopes(const double (&F)[L], const double (&FM)[L], const double "
         "(&X)[L], double beta, double (&DX)[L], double (&DB)[L]) {\n";
    if (taylor)
        for (int l = 0; l < L; ++l) {
            const int jo = tb.leaf_order[l];
            o << "  { const double f = F[" << l << "], m = FM[" << l << "]; double tj = 0.0, tn = 0.0;\n";
            o << taylor_expr(jo, "tj", "    ") << taylor_expr(jo + 1, "tn", "    ");
            o << "    DX[" << l << "] = " << num(static_cast<double>(jo + 1)) << " * tn;\n";
            o << "    DB[" << l << "] = fma(" << num(static_cast<double>(jo)) << ", tj, X[" << l << "] * DX[" << l
              << "]) / beta; }\n";
        }
    o << "  (void)F; (void)FM; (void)X; (void)beta; (void)DX; (void)DB;\n}\n";

    // denominators D_k = e_k . E + a_k . w
    o << "__device__ __forceinline__ void den_args(const double (&E)[NE], const double (&wr)[" << NXA
      << "], const double (&wi)[" << NXA << "], double (&dr)[D], double (&di)[D]) {\n";
    if (tb.D == 0) o << "  (void)E; (void)wr; (void)wi;\n  dr[0] = 1.0;\n  di[0] = 0.0;\n";
    for (int k = 0; k < tb.D; ++k) {
        Lin re, im;
        for (int i = 0; i < ne; ++i) re.add(tb.den_coef[static_cast<size_t>(k) * nc + i], idx("E", i));
        for (int x = 0; x < nx; ++x) {
            const double a = tb.den_coef[static_cast<size_t>(k) * nc + ne + x];
            re.add(a, idx("wr", x));
            im.add(a, idx("wi", x));
        }
        o << "  dr[" << k << "] = " << re.str() << ";\n  di[" << k << "] = " << im.str() << ";\n";
    }
    o << "}\n";

    // group products R_g = prod rho_k (complex), left to right
    auto group_product = [&](int g) {
        o << "  { double rr = 1.0, ri = 0.0, nr = 0.0;\n";
        for (int j = 0; j < gend(g) - gbegin(g); ++j) {
            const std::string k = std::to_string(tb.group_den_list[gbegin(g) + j]);
            if (j == 0) {
                o << "    rr = xr[" << k << "]; ri = xi[" << k << "];\n";
            } else {
                o << "    nr = fma(rr, xr[" << k << "], -ri * xi[" << k << "]); ri = fma(rr, xi[" << k
                  << "], ri * xr[" << k << "]); rr = nr;\n";
            }
        }
    };
    if (one_pass) {
        o << "__device__ __forceinline__ void group_products(const double (&xr)[D], const double (&xi)[D], "
             "double (&Rr)[G], double (&Ri)[G]) {\n";
        for (int g = 0; g < G; ++g) {
            group_product(g);
            o << "    (void)nr; Rr[" << g << "] = rr; Ri[" << g << "] = ri; }\n";
        }
        o << "}\n";
    }
    // the one-pass kernels' values sum_g FT_g R_g: nested over the reciprocals
    // (as the two-pass frequency pass) for solutions above the adjoint's
    // automatic size, else group by group from the products R_g (the
    // adjoint's own accumulation, so both kernels give the same bits)
    if (one_pass) {
        o << "__device__ __forceinline__ void groups_combine(const double (&xr)[D], const double (&xi)[D], "
             "const double (&FT)[G], double &acc_re, double &acc_im) {\n";
        if (nested_groups) {
            std::vector<HornerTerm> ts;
            for (int g = 0; g < G; ++g) {
                HornerTerm h{1.0, {}};
                for (int j = gbegin(g); j < gend(g); ++j) h.leaves.push_back(tb.group_den_list[j]);
                h.leaves.push_back(D + g);
                ts.push_back(std::move(h));
            }
            auto leaf = [&](int k) {
                CVal v;
                if (k < D) {
                    v.kind = CVal::CPLX;
                    v.re = "xr[" + std::to_string(k) + "]";
                    v.im = "xi[" + std::to_string(k) + "]";
                } else {
                    v.kind = CVal::REAL;
                    v.re = "FT[" + std::to_string(k - D) + "]";
                }
                return v;
            };
            int temps = 0;
            CMemo memo;
            const CVal v = horner_c(ts, leaf, o, temps, memo);
            const bool z = v.kind == CVal::ZERO;
            o << "    acc_re = " << (z ? "0.0" : v.kind == CVal::CONST ? num(v.c) : v.re) << ";\n";
            o << "    acc_im = " << (v.kind == CVal::CPLX ? v.im : "0.0") << ";\n";
        } else {
            o << "  double Rr[G], Ri[G];\n  group_products(xr, xi, Rr, Ri);\n  acc_re = 0.0;\n  acc_im = 0.0;\n";
            for (int g = 0; g < G; ++g)
                o << "  acc_re = fma(FT[" << g << "], Rr[" << g << "], acc_re);\n  acc_im = fma(FT[" << g << "], Ri[" << g
                  << "], acc_im);\n";
        }
        o << "}\n";
    }
    // two-pass forward, second pass: sum_g FT_g R_g nested over the
    // reciprocals, each stored group sum read where the nesting needs it
    if (kernels & 32) {
        o << "__device__ __forceinline__ void group_accumulate(const double (&xr)[D], const double (&xi)[D], "
             "const double *ws, int64_t ld, uint32_t off, double &acc_re, double &acc_im) {\n";
        o << kOffsetHere;
        // sum_g FT_g R_g nested over the reciprocals (factor k < D: z_k; factor
        // D + g: the stored FT_g, read where the nesting first needs it)
        std::vector<HornerTerm> ts;
        for (int g = 0; g < G; ++g) {
            HornerTerm h{1.0, {}};
            for (int j = gbegin(g); j < gend(g); ++j) h.leaves.push_back(tb.group_den_list[j]);
            h.leaves.push_back(D + g);
            ts.push_back(std::move(h));
        }
        std::vector<bool> loaded(static_cast<size_t>(G), false);
        auto leaf = [&](int k) {
            CVal v;
            if (k < D) {
                v.kind = CVal::CPLX;
                v.re = "xr[" + std::to_string(k) + "]";
                v.im = "xi[" + std::to_string(k) + "]";
            } else {
                const int g = k - D;
                if (!loaded[static_cast<size_t>(g)]) {
                    o << "    const double ft" << g << " = ami::ws_load(ws, ld, " << g << ", off);\n";
                    loaded[static_cast<size_t>(g)] = true;
                }
                v.kind = CVal::REAL;
                v.re = "ft" + std::to_string(g);
            }
            return v;
        };
        int temps = 0;
        CMemo memo;
        const CVal v = horner_c(ts, leaf, o, temps, memo);
        auto comp = [&](bool imag) {
            if (v.kind == CVal::ZERO) return std::string("0.0");
            if (v.kind == CVal::CONST) return imag ? std::string("0.0") : num(v.c);
            if (v.kind == CVal::REAL) return imag ? std::string("0.0") : v.re;
            return imag ? v.im : v.re;
        };
        o << "    acc_re += " << comp(false) << ";\n    acc_im += " << comp(true) << ";\n";
        o << "}\n";
    }

    // the second pass of the two-pass complex forward: as group_accumulate,
    // with each stored FT_g complex (columns g and G + g)
    if (kernels & 1024) {
        o << "__device__ __forceinline__ void group_accumulate_c(const double (&xr)[D], const double (&xi)[D], "
             "const double *ws, int64_t ld, uint32_t off, double &acc_re, double &acc_im) {\n";
        o << kOffsetHere;
        std::vector<HornerTerm> ts;
        for (int g = 0; g < G; ++g) {
            HornerTerm h{1.0, {}};
            for (int j = gbegin(g); j < gend(g); ++j) h.leaves.push_back(tb.group_den_list[j]);
            h.leaves.push_back(D + g);
            ts.push_back(std::move(h));
        }
        std::vector<bool> loaded(static_cast<size_t>(G), false);
        auto leaf = [&](int k) {
            CVal v;
            v.kind = CVal::CPLX;
            if (k < D) {
                v.re = "xr[" + std::to_string(k) + "]";
                v.im = "xi[" + std::to_string(k) + "]";
            } else {
                const int g = k - D;
                if (!loaded[static_cast<size_t>(g)]) {
                    o << "    const double ftr" << g << " = ami::ws_load(ws, ld, " << g << ", off), fti" << g
                      << " = ami::ws_load(ws, ld, " << G + g << ", off);\n";
                    loaded[static_cast<size_t>(g)] = true;
                }
                v.re = "ftr" + std::to_string(g);
                v.im = "fti" + std::to_string(g);
            }
            return v;
        };
        int temps = 0;
        CMemo memo;
        const CVal v = horner_c(ts, leaf, o, temps, memo);
        auto comp = [&](bool imag) {
            if (v.kind == CVal::ZERO) return std::string("0.0");
            if (v.kind == CVal::CONST) return imag ? std::string("0.0") : num(v.c);
            if (v.kind == CVal::REAL) return imag ? std::string("0.0") : v.re;
            return imag ? v.im : v.re;
        };
        o << "    acc_re += " << comp(false) << ";\n    acc_im += " << comp(true) << ";\n";
        o << "}\n";
    }

    // The adjoint of large solutions in passes (after the two-pass forward's
    // first pass has stored every FT_g and E_j in the workspace [column][sample]:
    // columns 0..G-1 FT_g, G..G+NE-1 E_j, then NE columns of the energy
    // cotangents gathered from the denominators, then G columns of the group-sum
    // cotangents FTB_g).
    const std::string ftb0 = "(G + 2 * NE)";
    if (kernels & 64) {
        // frequency pass, one frequency row: every reciprocal, then per chunk
        // of groups (scheduled apart, so that only one chunk's values are live
        // at a time) each group's R_g, the value FT_g R_g, FTB_g +=
        // Re(conj(c) R_g) (stored; added to the stored value after the first
        // row) and u_g = -FT_g conj(c) R_g summed per denominator of the
        // chunk, then per such denominator the scatter of U_k rho_k
        // FIRST: the first frequency row (FTB_g stored, not added to the stored value)
        o << "template <bool FIRST>\n__device__ __forceinline__ void adj_freq_row(const double (&E)[NE], const double (&wr)["
          << NXA << "], const double (&wi)[" << NXA << "], double cr, double ci, double *ws, int64_t ld, uint32_t off, "
             "double &acc_re, double &acc_im, double (&gE)[NE], double (&gwr)["
          << NXA << "], double (&gwi)[" << NXA << "]) {\n";
        o << kOffsetHere;
        const bool own = kAdjChunkOwnDens;
        if (!own)
            o << "  double xr[D], xi[D];\n  { double dr[D], di[D];\n    den_args(E, wr, wi, dr, di);\n"
                 "#pragma unroll\n    for (int k = 0; k < D; ++k) {\n"
                 "      const double inv = ami::rcp_nr(fma(dr[k], dr[k], di[k] * di[k]));\n"
                 "      xr[k] = dr[k] * inv;\n      xi[k] = -di[k] * inv;\n    } }\n";
        for (int g0 = 0; g0 < G; g0 += kAdjChunkGroups) {
            const int g1 = std::min(G, g0 + kAdjChunkGroups);
            std::vector<int> ks;
            for (int g = g0; g < g1; ++g)
                for (int j = gbegin(g); j < gend(g); ++j) ks.push_back(tb.group_den_list[j]);
            std::sort(ks.begin(), ks.end());
            ks.erase(std::unique(ks.begin(), ks.end()), ks.end());
            o << "  {\n";
            if (own) {
                // the chunk's own reciprocals
                o << "    double xr[D], xi[D];\n";
                for (int k : ks) {
                    Lin re, im;
                    for (int i = 0; i < ne; ++i) re.add(tb.den_coef[static_cast<size_t>(k) * nc + i], idx("E", i));
                    for (int x = 0; x < nx; ++x) {
                        const double a = tb.den_coef[static_cast<size_t>(k) * nc + ne + x];
                        re.add(a, idx("wr", x));
                        im.add(a, idx("wi", x));
                    }
                    o << "    { const double dr = " << re.str() << ", di = " << im.str()
                      << ";\n      const double inv = ami::rcp_nr(fma(dr, dr, di * di));\n      xr[" << k
                      << "] = dr * inv;\n      xi[" << k << "] = -di * inv; }\n";
                }
            }
            for (int k : ks) o << "    double Ur" << k << " = 0.0, Ui" << k << " = 0.0;\n";
            for (int g = g0; g < g1; ++g) {
                o << "    { const double ft = ami::ws_load(ws, ld, " << g << ", off);\n";
                o << "      double rr = 1.0, ri = 0.0, nr = 0.0;\n";
                for (int j = gbegin(g); j < gend(g); ++j) {
                    const std::string k = std::to_string(tb.group_den_list[j]);
                    if (j == gbegin(g)) o << "      rr = xr[" << k << "]; ri = xi[" << k << "];\n";
                    else
                        o << "      nr = fma(rr, xr[" << k << "], -ri * xi[" << k << "]); ri = fma(rr, xi[" << k
                          << "], ri * xr[" << k << "]); rr = nr;\n";
                }
                o << "      (void)nr;\n";
                o << "      acc_re = fma(ft, rr, acc_re);\n      acc_im = fma(ft, ri, acc_im);\n";
                o << "      const double tb = fma(cr, rr, ci * ri);\n";
                o << "      if constexpr (FIRST) ami::ws_store(ws, ld, " << ftb0 << " + " << g << ", off, tb);\n"
                  << "      else ami::ws_store(ws, ld, " << ftb0 << " + " << g << ", off, ami::ws_load(ws, ld, " << ftb0
                  << " + " << g << ", off) + tb);\n";
                o << "      const double qr = ft * cr, qi = -ft * ci;\n";
                o << "      const double ur = -fma(qr, rr, -qi * ri), ui = -fma(qr, ri, qi * rr);\n";
                for (int j = gbegin(g); j < gend(g); ++j) {
                    const std::string k = std::to_string(tb.group_den_list[j]);
                    o << "      Ur" << k << " += ur; Ui" << k << " += ui;\n";
                }
                o << "    }\n";
            }
            for (int k : ks) {
                o << "    { const double dR = fma(Ur" << k << ", xr[" << k << "], -Ui" << k << " * xi[" << k
                  << "]), dI = fma(Ur" << k << ", xi[" << k << "], Ui" << k << " * xr[" << k << "]);\n";
                for (int i = 0; i < ne; ++i) {
                    const double c = tb.den_coef[static_cast<size_t>(k) * nc + i];
                    if (c == 1.0) o << "      gE[" << i << "] += dR;\n";
                    else if (c == -1.0) o << "      gE[" << i << "] -= dR;\n";
                    else if (c != 0.0) o << "      gE[" << i << "] = fma(" << num(c) << ", dR, gE[" << i << "]);\n";
                }
                for (int x = 0; x < nx; ++x) {
                    const double a = tb.den_coef[static_cast<size_t>(k) * nc + ne + x];
                    if (a == 0.0) continue;
                    o << "      gwr[" << x << "] = fma(" << num(a) << ", dR, gwr[" << x << "]);\n";
                    o << "      gwi[" << x << "] = fma(" << num(a) << ", dI, gwi[" << x << "]);\n";
                }
                o << "    }\n";
            }
            o << "  }\n";
            if (g1 < G) o << "  AMI_SCHED_FENCE();\n";
        }
        o << "}\n";
    }
    // The leaf passes' parts: each group's terms nested in parts of at most
    // kAdjLeafPartTerms (consecutive in canonical order), with the leaves
    // each part reads and the first and last part that reads each leaf.
    struct Part {
        int g;
        std::vector<HNode> nodes;
        HRef root;
        std::vector<int> leaves;
    };
    auto build_parts = [&](std::vector<Part> &parts, std::vector<int> &first_use, std::vector<int> &last_use,
                           int part_terms) {
        for (int g = 0; g < G; ++g) {
            for (int t0 = tb.group_start[g]; t0 < tb.group_start[g + 1]; t0 += part_terms) {
                const int t1 = std::min(tb.group_start[g + 1], t0 + part_terms);
                std::vector<HornerTerm> ts;
                for (int ti = t0; ti < t1; ++ti) {
                    HornerTerm h{tb.term_sign[ti], {}};
                    for (int j = 0; j < ni; ++j) h.leaves.push_back(tb.term_leaf[static_cast<size_t>(ti) * ni + j]);
                    ts.push_back(std::move(h));
                }
                Part pt;
                pt.g = g;
                pt.root = horner_build(std::move(ts), pt.nodes);
                std::vector<int> used;
                auto note = [&](const HRef &r) {
                    if (r.kind == HRef::LEAF) used.push_back(r.idx);
                };
                note(pt.root);
                for (const HNode &n : pt.nodes) {
                    used.push_back(n.a);
                    note(n.w);
                    note(n.u);
                }
                std::sort(used.begin(), used.end());
                used.erase(std::unique(used.begin(), used.end()), used.end());
                pt.leaves = used;
                parts.push_back(std::move(pt));
            }
        }
        first_use.assign(static_cast<size_t>(L), -1);
        last_use.assign(static_cast<size_t>(L), -1);
        for (size_t p = 0; p < parts.size(); ++p)
            for (int l : parts[p].leaves) {
                if (first_use[l] < 0) first_use[l] = static_cast<int>(p);
                last_use[l] = static_cast<int>(p);
            }
    };
    if (kernels & 128) {
        // leaf pass: FB_l = sum_g FTB_g dFT_g/dF_l by a reverse sweep of each
        // group's nested sum (the nodes recomputed, then their cotangents in
        // reverse order: node h = F_a w + u passes h' w to F_a, h' F_a to w and
        // h' to u).  A group's terms are nested in parts of at most
        // kAdjLeafPartTerms (consecutive in canonical order), which bounds the
        // node values live in a sweep; each leaf is formed just before the
        // first part that reads it and its cotangent is scattered to the
        // energies and to beta just after the last one.
        std::vector<Part> parts;
        std::vector<int> first_use, last_use;
        build_parts(parts, first_use, last_use, kAdjLeafPartTerms);
        o << "__device__ __forceinline__ void leaf_pass(const double (&E)[NE], double beta, double e_reg, const double "
             "*ws, int64_t ld, uint32_t off, double (&gE)[NE], double &gbeta) {\n";
        o << kReverseContract;
        o << kOffsetHere;
        o << "  (void)e_reg;\n";
        // with Taylor-coefficient leaves DV holds dT/dx and DB dT/dbeta
        for (int l = 0; l < L; ++l)
            o << "  double F" << l << ", FB" << l << ", DV" << l << (taylor ? ", DB" + std::to_string(l) : "") << ";\n";
        auto leaf_arg = [&](int l) {
            Lin x;
            for (int i = 0; i < ne; ++i) x.add(tb.leaf_coef[static_cast<size_t>(l) * ne + i], idx("E", i));
            return x.str() + (tb.leaf_sigma[l] < 0 ? " + e_reg" : "");
        };
        auto fname = [](int l) { return "F" + std::to_string(l); };
        for (size_t p = 0; p < parts.size(); ++p) {
            const Part &pt = parts[p];
            for (int l : pt.leaves) {
                if (first_use[l] != static_cast<int>(p)) continue;
                if (taylor) {
                    const int jo = tb.leaf_order[l];
                    o << "  { const double x = " << leaf_arg(l) << ";\n    double f, m, tn = 0.0;\n    ami::leaf_pair("
                      << (tb.leaf_sigma[l] < 0 ? "true" : "false") << ", beta * x, f, m);\n";
                    o << taylor_expr(jo, "F" + std::to_string(l), "    ") << taylor_expr(jo + 1, "tn", "    ");
                    o << "    DV" << l << " = " << num(static_cast<double>(jo + 1)) << " * tn;\n    DB" << l << " = fma("
                      << num(static_cast<double>(jo)) << ", F" << l << ", x * DV" << l << ") / beta; }\n  FB" << l
                      << " = 0.0;\n";
                } else {
                    o << "  ami::leaf_and_slope(" << (tb.leaf_sigma[l] < 0 ? "true" : "false") << ", beta * ("
                      << leaf_arg(l) << "), F" << l << ", DV" << l << ");\n  FB" << l << " = 0.0;\n";
                }
            }
            o << "  { const double tb = ami::ws_load(ws, ld, " << ftb0 << " + " << pt.g << ", off);\n";
            horner_emit(pt.nodes, fname, o);
            const size_t nn = pt.nodes.size();
            for (size_t k = 0; k < nn; ++k) o << "    double hb" << k << " = 0.0;\n";
            // a cotangent c passed to reference r: hb += c (node) or FB += c (leaf)
            auto pass = [&](const HRef &r, const std::string &c) {
                if (r.kind == HRef::NODE) o << "    hb" << r.idx << (r.neg ? " -= " : " += ") << c << ";\n";
                else if (r.kind == HRef::LEAF) o << "    FB" << r.idx << (r.neg ? " -= " : " += ") << c << ";\n";
            };
            pass(pt.root, "tb");
            for (size_t kk = nn; kk-- > 0;) {
                const HNode &n = pt.nodes[kk];
                const std::string hb = "hb" + std::to_string(kk), fa = fname(n.a), fb = "FB" + std::to_string(n.a);
                if (n.w.kind == HRef::CONST) {
                    if (n.w.c == 1.0) o << "    " << fb << " += " << hb << ";\n";
                    else if (n.w.c == -1.0) o << "    " << fb << " -= " << hb << ";\n";
                    else o << "    " << fb << " = fma(" << num(n.w.c) << ", " << hb << ", " << fb << ");\n";
                } else {
                    const std::string wn = href_name(n.w, fname);
                    o << "    " << fb << " = fma(" << (n.w.neg ? "-" : "") << wn << ", " << hb << ", " << fb << ");\n";
                    pass(n.w, fa + " * " + hb);
                }
                pass(n.u, hb);
            }
            o << "  }\n";
            for (int l : pt.leaves) {
                if (last_use[l] != static_cast<int>(p)) continue;
                if (taylor)
                    o << "  { gbeta = fma(FB" << l << ", DB" << l << ", gbeta);\n    const double v = FB" << l << " * DV"
                      << l << ";\n";
                else
                    o << "  { const double fb = FB" << l << " * DV" << l << ";\n    gbeta = fma(fb, " << leaf_arg(l)
                      << ", gbeta);\n    const double v = fb * beta;\n";
                for (int i = 0; i < ne; ++i) {
                    const double c = tb.leaf_coef[static_cast<size_t>(l) * ne + i];
                    if (c == 1.0) o << "    gE[" << i << "] += v;\n";
                    else if (c == -1.0) o << "    gE[" << i << "] -= v;\n";
                    else if (c != 0.0) o << "    gE[" << i << "] = fma(" << num(c) << ", v, gE[" << i << "]);\n";
                }
                o << "  }\n";
            }
            if ((p + 1) % kAdjLeafFenceParts == 0 && p + 1 < parts.size()) o << "  AMI_SCHED_FENCE();\n";
        }
        o << "}\n";
    }

    // Shared by the block adjoints: the plan's constants, per-wave functions
    // (wave WV of a block), a range of terms, and the reads of a range's leaves.
    const bool blk_cplx = (kernels & 16384) != 0;
    BlockPlan bp;
    if (kernels & (8192 | 65536 | 16384))
        bp = block_plan(t, hub, blk_cplx, jit_block_waves(t, hub, blk_cplx, (kernels & 65536) != 0));
    auto wave_fn = [&](const std::string &name, const std::string &args, bool reverse, const auto &body) {
        o << "template <int WV" << (name == "blk_freq" ? ", bool ONE" : "") << "> __device__ __forceinline__ void " << name << "(" << args << ") {\n";
        if (reverse) o << kReverseContract;
        for (int w = 0; w < bp.waves; ++w) {
            o << "  if constexpr (WV == " << w << ") {\n";
            body(w);
            o << "  }\n";
        }
        o << "}\n";
    };
    auto terms_of = [&](int t0, int t1) {
        std::vector<HornerTerm> ts;
        for (int ti = t0; ti < t1; ++ti) {
            HornerTerm h{tb.term_sign[ti], {}};
            for (int j = 0; j < ni; ++j) h.leaves.push_back(tb.term_leaf[static_cast<size_t>(ti) * ni + j]);
            ts.push_back(std::move(h));
        }
        return ts;
    };
    auto leaves_of = [&](int t0, int t1) {
        std::vector<int> used;
        for (int ti = t0; ti < t1; ++ti)
            for (int j = 0; j < ni; ++j) used.push_back(tb.term_leaf[static_cast<size_t>(ti) * ni + j]);
        std::sort(used.begin(), used.end());
        used.erase(std::unique(used.begin(), used.end()), used.end());
        return used;
    };
    auto dens_of = [&](int w) {
        std::vector<int> ks;
        for (int g = bp.first[w]; g < bp.first[w + 1]; ++g)
            for (int j = gbegin(g); j < gend(g); ++j) ks.push_back(tb.group_den_list[j]);
        std::sort(ks.begin(), ks.end());
        ks.erase(std::unique(ks.begin(), ks.end()), ks.end());
        return ks;
    };
    if (kernels & 16384)
        // f(y) and conj(f'(y)) = -conj(f(y) f(-y))
        o << "__device__ __forceinline__ void blk_cleaf(bool bose, double yr, double yi, double &fr, double &fi, double "
             "&Sr, double &Si) {\n  double mr, mi;\n  ami::leaf_complex_pair(bose, yr, yi, fr, fi, mr, mi);\n"
             "  Sr = -fma(fr, mr, -fi * mi);\n  Si = fma(fr, mi, fi * mr);\n}\n";
    if (kernels & (8192 | 65536 | 16384)) {
        o << "constexpr int NW = " << bp.waves << ", GW = " << bp.max_groups << ", kRounds = " << bp.round.size() - 1
          << ", kBlockCols = " << bp.columns << ";\n";
        o << "constexpr bool kRowsApart = " << (jit_block_rows_apart(t) ? "true" : "false") << ";\n";
        if (!blk_cplx) o << "constexpr int kValueWave = " << bp.value_wave << ";\n";
        o << "constexpr int kBE = " << bp.c_e << ", kBS = " << bp.c_slope << ", kBU = " << bp.c_union << ", kBF = "
          << bp.c_leaf << ", kBT = " << bp.c_group << ", kBA = " << bp.c_acc << ";\n";
        o << "__device__ __forceinline__ void blk_rho(double dr, double di, double &xr, double &xi) {\n"
             "  const double inv = ami::rcp_nr(fma(dr, dr, di * di));\n  xr = dr * inv;\n  xi = -di * inv;\n}\n";
    }
    if (kernels & (8192 | 65536)) {
        // The block adjoint's per-wave functions (wave WV of a block of NW
        // waves that share 64 samples; LDS columns are passed as the address
        // of the lane's element in the first column of a region, column c of
        // it at [64 c]).
        const int W = bp.waves;
        const bool group_cols = bp.c_group >= 0, slope_cols = bp.c_slope >= 0;
        // the group sums' columns serve the cotangents too, unless the value
        // wave may still read them
        const bool exact = bp.value_wave >= 0, keep_cols = group_cols && !exact;
        // group g's sum of wave w
        auto gsum = [&](int w, int g, const char *reg) {
            return group_cols ? "sT[" + std::to_string(64 * g) + "]" : idx(reg, g - bp.first[w]);
        };
        // the leaves that terms [t0, t1) read, as "const double f<l>" from the
        // columns of a pointer taken through an empty asm (so that the compiler
        // loads them again here instead of holding every leaf)
        auto load_leaves = [&](int t0, int t1) {
            const std::vector<int> used = leaves_of(t0, t1);
            o << "    ami::clds p = sF; AMI_OPAQUE(p);\n   ";
            for (int l : used) o << " const double f" << l << " = p[" << 64 * l << "];";
            o << "\n";
        };
        auto fname = [](int l) { return "f" + std::to_string(l); };
        // group sums of the wave's groups
        wave_fn("blk_sums", "ami::clds sF, ami::lds sT, double (&ft)[GW]", false, [&](int w) {
            o << "    (void)sT; (void)ft;\n";
            for (int g = bp.first[w]; g < bp.first[w + 1]; ++g) {
                if (g > bp.first[w]) o << "  AMI_SCHED_FENCE();\n";
                o << "  {\n";
                load_leaves(tb.group_start[g], tb.group_start[g + 1]);
                std::vector<HNode> nodes;
                const HRef v = horner_build(terms_of(tb.group_start[g], tb.group_start[g + 1]), nodes);
                horner_emit(nodes, fname, o);
                o << "    " << gsum(w, g, "ft") << " = " << href_expr(v, fname) << "; }\n";
            }
        });
        if (exact)
            for (int k = 0; k < tb.D; ++k) {
                Lin re, im;
                for (int i = 0; i < ne; ++i) re.add(tb.den_coef[static_cast<size_t>(k) * nc + i], idx("E", i));
                for (int x = 0; x < nx; ++x) {
                    const double a = tb.den_coef[static_cast<size_t>(k) * nc + ne + x];
                    re.add(a, idx("wr", x));
                    im.add(a, idx("wi", x));
                }
                o << "__device__ __forceinline__ void blk_den" << k << "(const double (&E)[NE], const double (&wr)[" << NXA
                  << "], const double (&wi)[" << NXA << "], double &xr, double &xi) {\n  blk_rho(" << re.str() << ", "
                  << im.str() << ", xr, xi);\n}\n";
            }
        // one frequency row of the wave's groups: the reciprocals of their
        // denominators, R_g, the value's part sum FT_g R_g, FTB_g +=
        // Re(conj(c) R_g), and per denominator -conj(c) rho_k sum FT_g R_g,
        // scattered to the energies and frequencies
        // ONE: the only row, whose FTB_g takes FT_g's column at once
        wave_fn("blk_freq",
                "ami::clds sE, const double (&wr)[" + NXA + "], const double (&wi)[" + NXA +
                    "], ami::lds sT, const double (&ft)[GW], double cr, double ci, double (&ftb)[GW], double &acc_re, "
                    "double &acc_im, double (&gE)[NE], double (&gwr)[" + NXA + "], double (&gwi)[" + NXA + "]",
                true, [&](int w) {
            const std::vector<int> ks = dens_of(w);
            const bool all = w == bp.value_wave;      // the other waves' groups too, for the values
            // the columns through an empty asm: the sums are read here, not
            // held in registers since they were written
            o << "    AMI_OPAQUE(sT); (void)ft; (void)ftb;\n    double E[NE];\n#pragma unroll\n    for (int i = 0; i < NE; ++i) E[i] = sE[64 * i];\n";
            if (exact) {
                // the forward's reciprocals, formed outside this function's contraction
                if (all)
                    for (int k = 0; k < tb.D; ++k)
                        if (!std::binary_search(ks.begin(), ks.end(), k))
                            o << "    double xr" << k << ", xi" << k << ";\n    blk_den" << k << "(E, wr, wi, xr" << k
                              << ", xi" << k << ");\n";
                for (int k : ks)
                    o << "    double xr" << k << ", xi" << k << ", Ur" << k << " = 0.0, Ui" << k << " = 0.0;\n    blk_den"
                      << k << "(E, wr, wi, xr" << k << ", xi" << k << ");\n";
            }
            for (int k : ks) {
                if (exact) break;
                Lin re, im;
                for (int i = 0; i < ne; ++i) re.add(tb.den_coef[static_cast<size_t>(k) * nc + i], idx("E", i));
                for (int x = 0; x < nx; ++x) {
                    const double a = tb.den_coef[static_cast<size_t>(k) * nc + ne + x];
                    re.add(a, idx("wr", x));
                    im.add(a, idx("wi", x));
                }
                o << "    double xr" << k << ", xi" << k << ", Ur" << k << " = 0.0, Ui" << k << " = 0.0;\n    blk_rho("
                  << re.str() << ", " << im.str() << ", xr" << k << ", xi" << k << ");\n";
            }
            for (int g = all ? 0 : bp.first[w]; g < (all ? G : bp.first[w + 1]); ++g) {
                const bool own = g >= bp.first[w] && g < bp.first[w + 1];
                const std::string j0 = std::to_string(g - bp.first[w]);
                o << "    { double rr = 1.0, ri = 0.0, nr = 0.0;\n";
                for (int j = gbegin(g); j < gend(g); ++j) {
                    const std::string k = std::to_string(tb.group_den_list[j]);
                    if (j == gbegin(g)) o << "      rr = xr" << k << "; ri = xi" << k << ";\n";
                    else
                        o << "      nr = fma(rr, xr" << k << ", -ri * xi" << k << "); ri = fma(rr, xi" << k << ", ri * xr"
                          << k << "); rr = nr;\n";
                }
                if (all)
                    o << "      acc_re = fma(sT[" << 64 * g << "], rr, acc_re); acc_im = fma(sT[" << 64 * g
                      << "], ri, acc_im);\n";
                if (!own) {
                    o << "      (void)nr;\n    }\n";
                    continue;
                }
                o << "      (void)nr;\n      const double t = " << gsum(w, g, "ft")
                  << ", qr = t * rr, qi = t * ri, tb = fma(cr, rr, ci * ri);\n";
                if (keep_cols) o << "      if constexpr (ONE) sT[" << 64 * g << "] = tb;\n      else ";
                o << "ftb[" << j0 << "] += tb;\n";
                if (!exact) o << "      acc_re += qr; acc_im += qi;\n";
                for (int j = gbegin(g); j < gend(g); ++j) {
                    const std::string k = std::to_string(tb.group_den_list[j]);
                    o << "      Ur" << k << " += qr; Ui" << k << " += qi;\n";
                }
                o << "    }\n";
            }
            for (int k : ks) {
                const std::string K = std::to_string(k);
                o << "    { const double vr = -fma(Ur" << K << ", cr, Ui" << K << " * ci), vi = -fma(Ui" << K << ", cr, -Ur"
                  << K << " * ci);\n      const double dR = fma(vr, xr" << K << ", -vi * xi" << K << "), dI = fma(vr, xi"
                  << K << ", vi * xr" << K << ");\n      (void)dI;\n";
                for (int i = 0; i < ne; ++i) {
                    const double c = tb.den_coef[static_cast<size_t>(k) * nc + i];
                    if (c == 1.0) o << "      gE[" << i << "] += dR;\n";
                    else if (c == -1.0) o << "      gE[" << i << "] -= dR;\n";
                    else if (c != 0.0) o << "      gE[" << i << "] = fma(" << num(c) << ", dR, gE[" << i << "]);\n";
                }
                for (int x = 0; x < nx; ++x) {
                    const double a = tb.den_coef[static_cast<size_t>(k) * nc + ne + x];
                    if (a == 0.0) continue;
                    o << "      gwr[" << x << "] = fma(" << num(a) << ", dR, gwr[" << x << "]);\n";
                    o << "      gwi[" << x << "] = fma(" << num(a) << ", dI, gwi[" << x << "]);\n";
                }
                o << "    }\n";
            }
        });
        // leaf cotangents of the wave's groups by the reverse sweep of each
        // group's nested sum, in parts of at most kBlockPartTerms terms
        if (keep_cols)
            wave_fn("blk_keep", "ami::lds sT, const double (&ftb)[GW]", false, [&](int w) {
                for (int g = bp.first[w]; g < bp.first[w + 1]; ++g)
                    o << "    sT[" << 64 * g << "] = ftb[" << g - bp.first[w] << "];\n";
            });
        else
            wave_fn("blk_keep", "ami::lds, const double (&)[GW]", false, [&](int) {});
        wave_fn("blk_leaf", "ami::clds sF, ami::clds sT, const double (&ftb)[GW], double (&FB)[L]", true, [&](int w) {
            o << "    (void)sT; (void)ftb;\n";
            for (int g = bp.first[w]; g < bp.first[w + 1]; ++g)
                for (int t0 = tb.group_start[g]; t0 < tb.group_start[g + 1]; t0 += kBlockPartTerms) {
                    const int t1 = std::min(tb.group_start[g + 1], t0 + kBlockPartTerms);
                    std::vector<HNode> nodes;
                    const HRef root = horner_build(terms_of(t0, t1), nodes);
                    if (g > bp.first[w] || t0 > tb.group_start[g]) o << "  AMI_SCHED_FENCE();\n";
                    o << "  {\n";
                    load_leaves(t0, t1);
                    horner_emit(nodes, fname, o);
                    const size_t nn = nodes.size();
                    for (size_t k = 0; k < nn; ++k) o << "    double hb" << k << " = 0.0;\n";
                    auto pass = [&](const HRef &r, const std::string &c) {
                        if (r.kind == HRef::NODE) o << "    hb" << r.idx << (r.neg ? " -= " : " += ") << c << ";\n";
                        else if (r.kind == HRef::LEAF)
                            o << "    FB[" << r.idx << "]" << (r.neg ? " -= " : " += ") << c << ";\n";
                    };
                    pass(root, keep_cols ? gsum(w, g, "ftb") : idx("ftb", g - bp.first[w]));
                    for (size_t kk = nn; kk-- > 0;) {
                        const HNode &n = nodes[kk];
                        const std::string hb = "hb" + std::to_string(kk), fa = fname(n.a),
                                          fb = "FB[" + std::to_string(n.a) + "]";
                        if (n.w.kind == HRef::CONST) {
                            if (n.w.c == 1.0) o << "    " << fb << " += " << hb << ";\n";
                            else if (n.w.c == -1.0) o << "    " << fb << " -= " << hb << ";\n";
                            else o << "    " << fb << " = fma(" << num(n.w.c) << ", " << hb << ", " << fb << ");\n";
                        } else {
                            o << "    " << fb << " = fma(" << (n.w.neg ? "-" : "") << href_name(n.w, fname) << ", " << hb
                              << ", " << fb << ");\n";
                            pass(n.w, fa + " * " + hb);
                        }
                        pass(n.u, hb);
                    }
                    o << "  }\n";
                }
        });
        // the reduction of the leaf cotangents: round r's leaves of the wave to
        // their columns; then each leaf's sum over the waves (in their order)
        // by wave l mod NW: times the leaf's slope, to beta and the energies
        for (size_t r = 0; r + 1 < bp.round.size(); ++r) {
            const std::string R = std::to_string(r);
            wave_fn("blk_put" + R, "const double (&FB)[L], ami::lds sR", false, [&](int w) {
                for (int l = bp.round[r]; l < bp.round[r + 1]; ++l)
                    if (bp.slot[l][w] >= 0) o << "    sR[" << 64 * bp.slot[l][w] << "] = FB[" << l << "];\n";
            });
            wave_fn("blk_take" + R,
                    "double beta, double e_reg, ami::clds sE, ami::clds sR, ami::clds sS, double (&gE)[NE], double &gbeta",
                    true, [&](int w) {
                o << "    (void)e_reg; (void)sS;\n";
                for (int l = bp.round[r]; l < bp.round[r + 1]; ++l) {
                    if (l % W != w) continue;
                    Lin sum;
                    for (int v = 0; v < W; ++v)
                        if (bp.slot[l][v] >= 0) sum.add(1.0, "sR[" + std::to_string(64 * bp.slot[l][v]) + "]");
                    Lin x;
                    for (int i = 0; i < ne; ++i)
                        x.add(tb.leaf_coef[static_cast<size_t>(l) * ne + i], "sE[" + std::to_string(64 * i) + "]");
                    o << "    { const double x = " << x.str() << (tb.leaf_sigma[l] < 0 ? " + e_reg" : "") << ";\n";
                    if (slope_cols) {
                        o << "      const double dv = sS[" << 64 * l << "];\n";
                    } else {
                        o << "      double f, dv;\n      ami::leaf_and_slope(" << (tb.leaf_sigma[l] < 0 ? "true" : "false")
                          << ", beta * x, f, dv);\n";
                    }
                    o << "      const double fb = " << sum.str()
                      << " * dv, v = fb * beta;\n      gbeta = fma(fb, x, gbeta);\n";
                    for (int i = 0; i < ne; ++i) {
                        const double c = tb.leaf_coef[static_cast<size_t>(l) * ne + i];
                        if (c == 1.0) o << "      gE[" << i << "] += v;\n";
                        else if (c == -1.0) o << "      gE[" << i << "] -= v;\n";
                        else if (c != 0.0) o << "      gE[" << i << "] = fma(" << num(c) << ", v, gE[" << i << "]);\n";
                    }
                    o << "    }\n";
                }
            });
        }
        // the rounds, each between two barriers that every wave passes
        o << "template <int WV> __device__ __forceinline__ void blk_rounds(const double (&FB)[L], double beta, double "
             "e_reg, ami::clds sE, ami::lds sR, ami::clds sS, double (&gE)[NE], double &gbeta) {\n";
        for (size_t r = 0; r + 1 < bp.round.size(); ++r)
            o << "  __syncthreads();\n  blk_put" << r << "<WV>(FB, sR);\n  __syncthreads();\n  blk_take" << r
              << "<WV>(beta, e_reg, sE, sR, sS, gE, gbeta);\n";
        o << "}\n";
    }

    if (kernels & 16384) {
        // The block adjoint at complex energies: the same split, every value of
        // a leaf, a group sum or an energy two columns (real, imaginary) or two
        // registers; cotangents Xbar = dL/dRe X + i dL/dIm X.
        const int W = bp.waves;
        const bool group_cols = bp.c_group >= 0, slope_cols = bp.c_slope >= 0;
        auto gsum = [&](int w, int g, int im, const char *reg) {
            return group_cols ? "sT[" + std::to_string(64 * (2 * g + im)) + "]"
                              : std::string(reg) + (im ? "i[" : "r[") + std::to_string(g - bp.first[w]) + "]";
        };
        auto load_leaves = [&](int t0, int t1) {
            o << "    ami::clds p = sF; AMI_OPAQUE(p);\n   ";
            for (int l : leaves_of(t0, t1))
                o << " const double fr" << l << " = p[" << 128 * l << "], fi" << l << " = p[" << 128 * l + 64 << "];";
            o << "\n";
        };
        auto scatter2 = [&](const double *coef, const std::string &vr, const std::string &vi, double sr, double si) {
            for (int i = 0; i < ne; ++i) {
                const double c = coef[i];
                if (c == 0.0) continue;
                o << "      gEr[" << i << "] = fma(" << num(sr * c) << ", " << vr << ", gEr[" << i << "]); gEi[" << i
                  << "] = fma(" << num(si * c) << ", " << vi << ", gEi[" << i << "]);\n";
            }
        };
        wave_fn("blk_sums", "ami::clds sF, ami::lds sT, double (&ftr)[GW], double (&fti)[GW]", false, [&](int w) {
            o << "    (void)sT; (void)ftr; (void)fti;\n";
            for (int g = bp.first[w]; g < bp.first[w + 1]; ++g) {
                if (g > bp.first[w]) o << "  AMI_SCHED_FENCE();\n";
                o << "  {\n";
                load_leaves(tb.group_start[g], tb.group_start[g + 1]);
                auto leaf = [&](int l) {
                    CVal v;
                    v.kind = CVal::CPLX;
                    v.re = "fr" + std::to_string(l);
                    v.im = "fi" + std::to_string(l);
                    return v;
                };
                int temps = 0;
                CMemo memo;
                const CVal v = horner_c(terms_of(tb.group_start[g], tb.group_start[g + 1]), leaf, o, temps, memo);
                const std::string re = v.kind == CVal::ZERO ? "0.0" : v.kind == CVal::CONST ? num(v.c) : v.re;
                o << "    " << gsum(w, g, 0, "ft") << " = " << re << "; " << gsum(w, g, 1, "ft") << " = "
                  << (v.kind == CVal::CPLX ? v.im : "0.0") << "; }\n";
            }
        });
        wave_fn("blk_freq",
                "ami::clds sE, const double (&wr)[" + NXA + "], const double (&wi)[" + NXA +
                    "], ami::lds sT, const double (&ftr)[GW], const double (&fti)[GW], double cr, double ci, double "
                    "(&ftbr)[GW], double (&ftbi)[GW], double &acc_re, double &acc_im, double (&gEr)[NE], double "
                    "(&gEi)[NE], double (&gwr)[" + NXA + "], double (&gwi)[" + NXA + "]",
                true, [&](int w) {
            const std::vector<int> ks = dens_of(w);
            o << "    AMI_OPAQUE(sT); (void)ftr; (void)fti; (void)ftbr; (void)ftbi;\n    double Er[NE], Ei[NE];\n"
                 "#pragma unroll\n    for (int i = 0; i < NE; ++i) {\n      Er[i] = sE[64 * i];\n      Ei[i] = sE[64 * (NE + "
                 "i)];\n    }\n";
            for (int k : ks) {
                Lin re, im;
                for (int i = 0; i < ne; ++i) {
                    re.add(tb.den_coef[static_cast<size_t>(k) * nc + i], idx("Er", i));
                    im.add(tb.den_coef[static_cast<size_t>(k) * nc + i], idx("Ei", i));
                }
                for (int x = 0; x < nx; ++x) {
                    const double a = tb.den_coef[static_cast<size_t>(k) * nc + ne + x];
                    re.add(a, idx("wr", x));
                    im.add(a, idx("wi", x));
                }
                o << "    double xr" << k << ", xi" << k << ", Ur" << k << " = 0.0, Ui" << k << " = 0.0;\n    blk_rho("
                  << re.str() << ", " << im.str() << ", xr" << k << ", xi" << k << ");\n";
            }
            for (int g = bp.first[w]; g < bp.first[w + 1]; ++g) {
                const std::string j0 = std::to_string(g - bp.first[w]);
                o << "    { double rr = 1.0, ri = 0.0, nr = 0.0;\n";
                for (int j = gbegin(g); j < gend(g); ++j) {
                    const std::string k = std::to_string(tb.group_den_list[j]);
                    if (j == gbegin(g)) o << "      rr = xr" << k << "; ri = xi" << k << ";\n";
                    else
                        o << "      nr = fma(rr, xr" << k << ", -ri * xi" << k << "); ri = fma(rr, xi" << k << ", ri * xr"
                          << k << "); rr = nr;\n";
                }
                o << "      (void)nr;\n      const double tr = " << gsum(w, g, 0, "ft") << ", ti = " << gsum(w, g, 1, "ft")
                  << ";\n      const double qr = fma(tr, rr, -ti * ri), qi = fma(tr, ri, ti * rr);\n"
                     "      const double tbr = fma(cr, rr, ci * ri), tbi = fma(ci, rr, -cr * ri);\n";
                if (group_cols)
                    o << "      if constexpr (ONE) { sT[" << 128 * g << "] = tbr; sT[" << 128 * g + 64
                      << "] = tbi; }\n      else ";
                o << "{ ftbr[" << j0 << "] += tbr; ftbi[" << j0 << "] += tbi; }\n      acc_re += qr; acc_im += qi;\n";
                for (int j = gbegin(g); j < gend(g); ++j) {
                    const std::string k = std::to_string(tb.group_den_list[j]);
                    o << "      Ur" << k << " += qr; Ui" << k << " += qi;\n";
                }
                o << "    }\n";
            }
            for (int k : ks) {
                const std::string K = std::to_string(k);
                o << "    { const double vr = -fma(Ur" << K << ", cr, Ui" << K << " * ci), vi = -fma(Ui" << K << ", cr, -Ur"
                  << K << " * ci);\n      const double dR = fma(vr, xr" << K << ", -vi * xi" << K << "), dI = fma(vr, xi"
                  << K << ", vi * xr" << K << ");\n      (void)dI;\n";
                scatter2(&tb.den_coef[static_cast<size_t>(k) * nc], "dR", "dI", 1.0, -1.0);
                for (int x = 0; x < nx; ++x) {
                    const double a = tb.den_coef[static_cast<size_t>(k) * nc + ne + x];
                    if (a == 0.0) continue;
                    o << "      gwr[" << x << "] = fma(" << num(a) << ", dR, gwr[" << x << "]);\n";
                    o << "      gwi[" << x << "] = fma(" << num(a) << ", dI, gwi[" << x << "]);\n";
                }
                o << "    }\n";
            }
        });
        if (group_cols)
            wave_fn("blk_keep", "ami::lds sT, const double (&ftbr)[GW], const double (&ftbi)[GW]", false, [&](int w) {
                for (int g = bp.first[w]; g < bp.first[w + 1]; ++g)
                    o << "    sT[" << 128 * g << "] = ftbr[" << g - bp.first[w] << "]; sT[" << 128 * g + 64 << "] = ftbi["
                      << g - bp.first[w] << "];\n";
            });
        else
            wave_fn("blk_keep", "ami::lds, const double (&)[GW], const double (&)[GW]", false, [&](int) {});
        // a node h = F_a w + u passes hbar conj(w) to F_a, hbar conj(F_a) to w
        // and hbar to u
        wave_fn("blk_leaf",
                "ami::clds sF, ami::clds sT, const double (&ftbr)[GW], const double (&ftbi)[GW], double (&FBr)[L], double "
                "(&FBi)[L]",
                true, [&](int w) {
            o << "    (void)sT; (void)ftbr; (void)ftbi;\n";
            auto vre = [&](const HRef &r) -> std::string {
                if (r.kind == HRef::LEAF) return "fr" + std::to_string(r.idx);
                if (r.kind == HRef::NODE) return "h" + std::to_string(r.idx) + "r";
                return r.kind == HRef::CONST ? num(r.c) : std::string("0.0");
            };
            auto vim = [&](const HRef &r) -> std::string {
                if (r.kind == HRef::LEAF) return "fi" + std::to_string(r.idx);
                if (r.kind == HRef::NODE) return "h" + std::to_string(r.idx) + "i";
                return std::string("0.0");
            };
            auto sg = [](const HRef &r, const std::string &e) { return r.neg ? "(-" + e + ")" : e; };
            for (int g = bp.first[w]; g < bp.first[w + 1]; ++g)
                for (int t0 = tb.group_start[g]; t0 < tb.group_start[g + 1]; t0 += kBlockPartTerms) {
                    const int t1 = std::min(tb.group_start[g + 1], t0 + kBlockPartTerms);
                    std::vector<HNode> nodes;
                    const HRef root = horner_build(terms_of(t0, t1), nodes);
                    if (g > bp.first[w] || t0 > tb.group_start[g]) o << "  AMI_SCHED_FENCE();\n";
                    o << "  {\n";
                    load_leaves(t0, t1);
                    const size_t nn = nodes.size();
                    for (size_t k = 0; k < nn; ++k) {
                        const HNode &n = nodes[k];
                        const std::string far = "fr" + std::to_string(n.a), fai = "fi" + std::to_string(n.a);
                        std::string ur, ui;
                        if (n.u.kind == HRef::CONST) {
                            ur = num(n.u.c);
                        } else if (n.u.kind != HRef::ZERO) {
                            ur = sg(n.u, vre(n.u));
                            ui = sg(n.u, vim(n.u));
                        }
                        std::string hr, hi;
                        if (n.w.kind == HRef::CONST) {
                            hr = fused({{false, num(n.w.c), far}}, ur);
                            hi = fused({{false, num(n.w.c), fai}}, ui);
                        } else {
                            const std::string wr = sg(n.w, vre(n.w)), wi = sg(n.w, vim(n.w));
                            hr = fused({{false, far, wr}, {true, fai, wi}}, ur);
                            hi = fused({{false, far, wi}, {false, fai, wr}}, ui);
                        }
                        o << "    const double h" << k << "r = " << hr << ", h" << k << "i = " << hi << ";\n";
                    }
                    for (size_t k = 0; k < nn; ++k) o << "    double hb" << k << "r = 0.0, hb" << k << "i = 0.0;\n";
                    auto pass = [&](const HRef &r, const std::string &cr, const std::string &ci) {
                        const char *op = r.neg ? " -= " : " += ";
                        if (r.kind == HRef::NODE)
                            o << "    hb" << r.idx << "r" << op << cr << "; hb" << r.idx << "i" << op << ci << ";\n";
                        else if (r.kind == HRef::LEAF)
                            o << "    FBr[" << r.idx << "]" << op << cr << "; FBi[" << r.idx << "]" << op << ci << ";\n";
                    };
                    pass(root, gsum(w, g, 0, "ftb"), gsum(w, g, 1, "ftb"));
                    for (size_t kk = nn; kk-- > 0;) {
                        const HNode &n = nodes[kk];
                        const std::string A = std::to_string(n.a);
                        const std::string br = "hb" + std::to_string(kk) + "r", bi = "hb" + std::to_string(kk) + "i";
                        const std::string far = "fr" + A, fai = "fi" + A, fbr = "FBr[" + A + "]", fbi = "FBi[" + A + "]";
                        if (n.w.kind == HRef::CONST) {
                            o << "    " << fbr << " = fma(" << num(n.w.c) << ", " << br << ", " << fbr << "); " << fbi
                              << " = fma(" << num(n.w.c) << ", " << bi << ", " << fbi << ");\n";
                        } else {
                            const std::string wr = sg(n.w, vre(n.w)), wi = sg(n.w, vim(n.w));
                            o << "    " << fbr << " = fma(" << br << ", " << wr << ", fma(" << bi << ", " << wi << ", " << fbr
                              << ")); " << fbi << " = fma(" << bi << ", " << wr << ", fma(-" << br << ", " << wi << ", "
                              << fbi << "));\n";
                            pass(n.w, "fma(" + br + ", " + far + ", " + bi + " * " + fai + ")",
                                 "fma(" + bi + ", " + far + ", -" + br + " * " + fai + ")");
                        }
                        pass(n.u, br, bi);
                    }
                    o << "  }\n";
                }
        });
        for (size_t r = 0; r + 1 < bp.round.size(); ++r) {
            const std::string R = std::to_string(r);
            wave_fn("blk_put" + R, "const double (&FBr)[L], const double (&FBi)[L], ami::lds sR", false, [&](int w) {
                for (int l = bp.round[r]; l < bp.round[r + 1]; ++l)
                    if (bp.slot[l][w] >= 0)
                        o << "    sR[" << 64 * bp.slot[l][w] << "] = FBr[" << l << "]; sR[" << 64 * bp.slot[l][w] + 64
                          << "] = FBi[" << l << "];\n";
            });
            wave_fn("blk_take" + R,
                    "double beta, double e_reg, ami::clds sE, ami::clds sR, ami::clds sS, double (&gEr)[NE], double "
                    "(&gEi)[NE], double &gbeta",
                    true, [&](int w) {
                o << "    (void)e_reg; (void)sS;\n";
                for (int l = bp.round[r]; l < bp.round[r + 1]; ++l) {
                    if (l % W != w) continue;
                    Lin sr, si, xr, xi;
                    for (int v = 0; v < W; ++v)
                        if (bp.slot[l][v] >= 0) {
                            sr.add(1.0, "sR[" + std::to_string(64 * bp.slot[l][v]) + "]");
                            si.add(1.0, "sR[" + std::to_string(64 * bp.slot[l][v] + 64) + "]");
                        }
                    for (int i = 0; i < ne; ++i) {
                        xr.add(tb.leaf_coef[static_cast<size_t>(l) * ne + i], "sE[" + std::to_string(64 * i) + "]");
                        xi.add(tb.leaf_coef[static_cast<size_t>(l) * ne + i], "sE[" + std::to_string(64 * (ne + i)) + "]");
                    }
                    const bool bose = tb.leaf_sigma[l] < 0;
                    o << "    { const double xr = " << xr.str() << (bose ? " + e_reg" : "") << ", xi = " << xi.str() << ";\n";
                    if (slope_cols)
                        o << "      const double Sr = sS[" << 128 * l << "], Si = sS[" << 128 * l + 64 << "];\n";
                    else
                        o << "      double Sr, Si, fr, fi;\n      blk_cleaf(" << (bose ? "true" : "false")
                          << ", beta * xr, beta * xi, fr, fi, Sr, Si);\n";
                    o << "      const double br = " << sr.str() << ", bi = " << si.str()
                      << ";\n      const double Vr = fma(br, Sr, -bi * Si), Vi = fma(br, Si, bi * Sr);\n"
                         "      gbeta = fma(Vr, xr, fma(Vi, xi, gbeta));\n      const double vr = Vr * beta, vi = Vi * beta;\n";
                    scatter2(&tb.leaf_coef[static_cast<size_t>(l) * ne], "vr", "vi", 1.0, 1.0);
                    o << "    }\n";
                }
            });
        }
        o << "template <int WV> __device__ __forceinline__ void blk_rounds(const double (&FBr)[L], const double (&FBi)[L], "
             "double beta, double e_reg, ami::clds sE, ami::lds sR, ami::clds sS, double (&gEr)[NE], double (&gEi)[NE], "
             "double &gbeta) {\n";
        for (size_t r = 0; r + 1 < bp.round.size(); ++r)
            o << "  __syncthreads();\n  blk_put" << r << "<WV>(FBr, FBi, sR);\n  __syncthreads();\n  blk_take" << r
              << "<WV>(beta, e_reg, sE, sR, sS, gEr, gEi, gbeta);\n";
        o << "}\n";
    }

    if (kernels & 32768) {
        // The block forward of large solutions: as the block adjoint, the
        // leaves' columns shared by the block's waves, each wave the sums of its
        // own groups into theirs; then every wave takes whole frequency rows.
        const int W = jit_block_forward_waves(t);
        std::vector<double> cost(static_cast<size_t>(G));
        for (int g = 0; g < G; ++g) cost[g] = static_cast<double>(group_nest_sizes(t)[g]) + 4.0;
        bp = BlockPlan();
        bp.waves = W;
        (void)split_groups(cost, W, bp.first);
        o << "constexpr int NW = " << W << ", kBlockCols = NE + L + G;\n";
        auto fname = [](int l) { return "f" + std::to_string(l); };
        wave_fn("blk_sums", "ami::clds sF, ami::lds sT", false, [&](int w) {
            for (int g = bp.first[w]; g < bp.first[w + 1]; ++g) {
                if (g > bp.first[w]) o << "  AMI_SCHED_FENCE();\n";
                o << "  { ami::clds p = sF; AMI_OPAQUE(p);\n   ";
                for (int l : leaves_of(tb.group_start[g], tb.group_start[g + 1]))
                    o << " const double f" << l << " = p[" << 64 * l << "];";
                o << "\n";
                std::vector<HNode> nodes;
                const HRef v = horner_build(terms_of(tb.group_start[g], tb.group_start[g + 1]), nodes);
                horner_emit(nodes, fname, o);
                o << "    sT[" << 64 * g << "] = " << href_expr(v, fname) << "; }\n";
            }
        });
        o << "__device__ __forceinline__ void blk_row(ami::clds sT, const double (&xr)[D], const double (&xi)[D], double "
             "&acc_re, double &acc_im) {\n";
        std::vector<HornerTerm> ts;
        for (int g = 0; g < G; ++g) {
            HornerTerm h{1.0, {}};
            for (int j = gbegin(g); j < gend(g); ++j) h.leaves.push_back(tb.group_den_list[j]);
            h.leaves.push_back(D + g);
            ts.push_back(std::move(h));
        }
        auto leaf = [&](int k) {
            CVal v;
            if (k < D) {
                v.kind = CVal::CPLX;
                v.re = "xr[" + std::to_string(k) + "]";
                v.im = "xi[" + std::to_string(k) + "]";
            } else {
                v.kind = CVal::REAL;
                v.re = "sT[" + std::to_string(64 * (k - D)) + "]";
            }
            return v;
        };
        int temps = 0;
        CMemo memo;
        const CVal v = horner_c(ts, leaf, o, temps, memo);
        o << "    acc_re = " << (v.kind == CVal::ZERO ? "0.0" : v.kind == CVal::CONST ? num(v.c) : v.re)
          << ";\n    acc_im = " << (v.kind == CVal::CPLX ? v.im : "0.0") << ";\n}\n";
    }

    // The adjoint at complex energies in passes (after the complex two-pass
    // forward's first pass stored FT_g and E_j, both complex, in the
    // workspace: columns [0, G) Re FT, [G, 2G) Im FT, [2G, 2G + NE) Re E,
    // [2G + NE, 2G + 2NE) Im E, then the denominators' energy cotangents
    // (re NE, im NE) and the group-sum cotangents FTB_g (re G, im G)).  The
    // cotangents are complex, Xbar = dL/dRe X + i dL/dIm X.
    const std::string cge0 = "(2 * G + 2 * NE)", cftb0 = "(2 * G + 4 * NE)";
    if (kernels & 2048) {
        // frequency pass, one frequency row: per chunk of groups its own
        // reciprocals (the energies' imaginary parts in the denominators),
        // each group's R_g, the value FT_g R_g, FTB_g += c conj(R_g) (stored;
        // added to the stored value after the first row), u_g = -FT_g conj(c)
        // R_g summed per denominator, then U_k rho_k = conj(Dbar_k) scattered:
        // its real part to Re Ebar and the frequencies, minus its imaginary
        // part to Im Ebar
        o << "template <bool FIRST>\n__device__ __forceinline__ void cadj_freq_row(const double (&Er)[NE], const double "
             "(&Ei)[NE], const double (&wr)["
          << NXA << "], const double (&wi)[" << NXA << "], double cr, double ci, double *ws, int64_t ld, uint32_t off, "
             "double &acc_re, double &acc_im, double (&gEr)[NE], double (&gEi)[NE], double (&gwr)["
          << NXA << "], double (&gwi)[" << NXA << "]) {\n";
        o << kOffsetHere;
        for (int g0 = 0; g0 < G; g0 += kAdjChunkGroups) {
            const int g1 = std::min(G, g0 + kAdjChunkGroups);
            std::vector<int> ks;
            for (int g = g0; g < g1; ++g)
                for (int j = gbegin(g); j < gend(g); ++j) ks.push_back(tb.group_den_list[j]);
            std::sort(ks.begin(), ks.end());
            ks.erase(std::unique(ks.begin(), ks.end()), ks.end());
            o << "  {\n    double xr[D], xi[D];\n";
            for (int k : ks) {
                Lin re, im;
                for (int i = 0; i < ne; ++i) {
                    re.add(tb.den_coef[static_cast<size_t>(k) * nc + i], idx("Er", i));
                    im.add(tb.den_coef[static_cast<size_t>(k) * nc + i], idx("Ei", i));
                }
                for (int x = 0; x < nx; ++x) {
                    const double a = tb.den_coef[static_cast<size_t>(k) * nc + ne + x];
                    re.add(a, idx("wr", x));
                    im.add(a, idx("wi", x));
                }
                o << "    { const double dr = " << re.str() << ", di = " << im.str()
                  << ";\n      const double inv = ami::rcp_nr(fma(dr, dr, di * di));\n      xr[" << k
                  << "] = dr * inv;\n      xi[" << k << "] = -di * inv; }\n";
            }
            for (int k : ks) o << "    double Ur" << k << " = 0.0, Ui" << k << " = 0.0;\n";
            for (int g = g0; g < g1; ++g) {
                o << "    { const double ftr = ami::ws_load(ws, ld, " << g << ", off), fti = ami::ws_load(ws, ld, "
                  << G + g << ", off);\n";
                o << "      double rr = 1.0, ri = 0.0, nr = 0.0;\n";
                for (int j = gbegin(g); j < gend(g); ++j) {
                    const std::string k = std::to_string(tb.group_den_list[j]);
                    if (j == gbegin(g)) o << "      rr = xr[" << k << "]; ri = xi[" << k << "];\n";
                    else
                        o << "      nr = fma(rr, xr[" << k << "], -ri * xi[" << k << "]); ri = fma(rr, xi[" << k
                          << "], ri * xr[" << k << "]); rr = nr;\n";
                }
                o << "      (void)nr;\n";
                o << "      acc_re = fma(ftr, rr, fma(-fti, ri, acc_re));\n"
                     "      acc_im = fma(ftr, ri, fma(fti, rr, acc_im));\n";
                o << "      const double tbr = fma(cr, rr, ci * ri), tbi = fma(ci, rr, -cr * ri);\n";
                const std::string cr_ = cftb0 + " + " + std::to_string(g), ci_ = cftb0 + " + " + std::to_string(G + g);
                o << "      if constexpr (FIRST) {\n        ami::ws_store(ws, ld, " << cr_ << ", off, tbr);\n"
                  << "        ami::ws_store(ws, ld, " << ci_ << ", off, tbi);\n      } else {\n"
                  << "        ami::ws_store(ws, ld, " << cr_ << ", off, ami::ws_load(ws, ld, " << cr_ << ", off) + tbr);\n"
                  << "        ami::ws_store(ws, ld, " << ci_ << ", off, ami::ws_load(ws, ld, " << ci_
                  << ", off) + tbi);\n      }\n";
                o << "      const double qr = fma(ftr, cr, fti * ci), qi = fma(fti, cr, -ftr * ci);\n";
                o << "      const double ur = -fma(qr, rr, -qi * ri), ui = -fma(qr, ri, qi * rr);\n";
                for (int j = gbegin(g); j < gend(g); ++j) {
                    const std::string k = std::to_string(tb.group_den_list[j]);
                    o << "      Ur" << k << " += ur; Ui" << k << " += ui;\n";
                }
                o << "    }\n";
            }
            for (int k : ks) {
                o << "    { const double dR = fma(Ur" << k << ", xr[" << k << "], -Ui" << k << " * xi[" << k
                  << "]), dI = fma(Ur" << k << ", xi[" << k << "], Ui" << k << " * xr[" << k << "]);\n";
                for (int i = 0; i < ne; ++i) {
                    const double c = tb.den_coef[static_cast<size_t>(k) * nc + i];
                    if (c == 1.0) o << "      gEr[" << i << "] += dR; gEi[" << i << "] -= dI;\n";
                    else if (c == -1.0) o << "      gEr[" << i << "] -= dR; gEi[" << i << "] += dI;\n";
                    else if (c != 0.0)
                        o << "      gEr[" << i << "] = fma(" << num(c) << ", dR, gEr[" << i << "]); gEi[" << i
                          << "] = fma(" << num(-c) << ", dI, gEi[" << i << "]);\n";
                }
                for (int x = 0; x < nx; ++x) {
                    const double a = tb.den_coef[static_cast<size_t>(k) * nc + ne + x];
                    if (a == 0.0) continue;
                    o << "      gwr[" << x << "] = fma(" << num(a) << ", dR, gwr[" << x << "]);\n";
                    o << "      gwi[" << x << "] = fma(" << num(a) << ", dI, gwi[" << x << "]);\n";
                }
                o << "    }\n";
            }
            o << "  }\n";
            if (g1 < G) o << "  AMI_SCHED_FENCE();\n";
        }
        o << "}\n";
    }
    if (kernels & 4096) {
        // leaf pass at complex energies: the reverse sweep of each part of a
        // group's nested sum in complex arithmetic; a node h = F_a w + u
        // passes hbar conj(w) to F_a, hbar conj(F_a) to w and hbar to u.
        // Each leaf is formed just before the first part that reads it; after
        // the last one its pair again gives S = conj(f'(y)) = -conj(f(y) f(-y)),
        // and V = Fbar S gives xbar = beta V to the energies and
        // Re(conj(V) x) to beta.
        std::vector<Part> parts;
        std::vector<int> first_use, last_use;
        build_parts(parts, first_use, last_use, cadj_part_terms());
        o << "__device__ __forceinline__ void cleaf_pass(const double (&Er)[NE], const double (&Ei)[NE], double beta, "
             "double e_reg, const double *ws, int64_t ld, uint32_t off, double (&gEr)[NE], double (&gEi)[NE], "
             "double &gbeta) {\n";
        o << kReverseContract;
        o << kOffsetHere;
        o << "  (void)e_reg;\n";
        for (int l = 0; l < L; ++l)
            o << "  double Fr" << l << ", Fi" << l << ", FBr" << l << ", FBi" << l << ";\n";
        auto arg = [&](int l, bool imag) {
            Lin x;
            for (int i = 0; i < ne; ++i) x.add(tb.leaf_coef[static_cast<size_t>(l) * ne + i], idx(imag ? "Ei" : "Er", i));
            return x.str() + (!imag && tb.leaf_sigma[l] < 0 ? " + e_reg" : "");
        };
        // names of a reference's value: real and imaginary part (without its sign)
        auto vre = [&](const HRef &r) -> std::string {
            if (r.kind == HRef::LEAF) return "Fr" + std::to_string(r.idx);
            if (r.kind == HRef::NODE) return "h" + std::to_string(r.idx) + "r";
            return r.kind == HRef::CONST ? num(r.c) : std::string("0.0");
        };
        auto vim = [&](const HRef &r) -> std::string {
            if (r.kind == HRef::LEAF) return "Fi" + std::to_string(r.idx);
            if (r.kind == HRef::NODE) return "h" + std::to_string(r.idx) + "i";
            return std::string("0.0");
        };
        auto sg = [](const HRef &r, const std::string &e) { return r.neg ? "(-" + e + ")" : e; };
        for (size_t p = 0; p < parts.size(); ++p) {
            const Part &pt = parts[p];
            for (int l : pt.leaves) {
                if (first_use[l] != static_cast<int>(p)) continue;
                o << "  ami::leaf_complex(" << (tb.leaf_sigma[l] < 0 ? "true" : "false") << ", beta * ("
                  << arg(l, false) << "), beta * (" << arg(l, true) << "), Fr" << l << ", Fi" << l << ");\n  FBr" << l
                  << " = 0.0; FBi" << l << " = 0.0;\n";
            }
            o << "  { const double tbr = ami::ws_load(ws, ld, " << cftb0 << " + " << pt.g
              << ", off), tbi = ami::ws_load(ws, ld, " << cftb0 << " + " << G + pt.g << ", off);\n";
            // forward: node values
            const size_t nn = pt.nodes.size();
            for (size_t k = 0; k < nn; ++k) {
                const HNode &n = pt.nodes[k];
                const std::string far = "Fr" + std::to_string(n.a), fai = "Fi" + std::to_string(n.a);
                // u's parts (signed)
                std::string ur = "0.0", ui = "0.0";
                if (n.u.kind == HRef::CONST) ur = num(n.u.c);
                else if (n.u.kind != HRef::ZERO) {
                    ur = sg(n.u, vre(n.u));
                    ui = sg(n.u, vim(n.u));
                }
                std::string hr, hi;
                if (n.w.kind == HRef::CONST) {
                    hr = "fma(" + num(n.w.c) + ", " + far + ", " + ur + ")";
                    hi = "fma(" + num(n.w.c) + ", " + fai + ", " + ui + ")";
                } else {
                    const std::string wr = sg(n.w, vre(n.w)), wi = sg(n.w, vim(n.w));
                    hr = "fma(" + far + ", " + wr + ", fma(-" + fai + ", " + wi + ", " + ur + "))";
                    hi = "fma(" + far + ", " + wi + ", fma(" + fai + ", " + wr + ", " + ui + "))";
                }
                o << "    const double h" << k << "r = " << hr << ", h" << k << "i = " << hi << ";\n";
            }
            for (size_t k = 0; k < nn; ++k) o << "    double hb" << k << "r = 0.0, hb" << k << "i = 0.0;\n";
            // a cotangent (cr, ci) passed to reference r
            auto pass = [&](const HRef &r, const std::string &cr, const std::string &ci) {
                const char *op = r.neg ? " -= " : " += ";
                if (r.kind == HRef::NODE)
                    o << "    hb" << r.idx << "r" << op << cr << "; hb" << r.idx << "i" << op << ci << ";\n";
                else if (r.kind == HRef::LEAF)
                    o << "    FBr" << r.idx << op << cr << "; FBi" << r.idx << op << ci << ";\n";
            };
            pass(pt.root, "tbr", "tbi");
            for (size_t kk = nn; kk-- > 0;) {
                const HNode &n = pt.nodes[kk];
                const std::string br = "hb" + std::to_string(kk) + "r", bi = "hb" + std::to_string(kk) + "i";
                const std::string far = "Fr" + std::to_string(n.a), fai = "Fi" + std::to_string(n.a);
                const std::string fbr = "FBr" + std::to_string(n.a), fbi = "FBi" + std::to_string(n.a);
                if (n.w.kind == HRef::CONST) {
                    o << "    " << fbr << " = fma(" << num(n.w.c) << ", " << br << ", " << fbr << "); " << fbi
                      << " = fma(" << num(n.w.c) << ", " << bi << ", " << fbi << ");\n";
                } else {
                    // F_a += hbar conj(w) (w with its sign); w += hbar conj(F_a) (sign applied by pass)
                    const std::string wr = sg(n.w, vre(n.w)), wi = sg(n.w, vim(n.w));
                    o << "    " << fbr << " = fma(" << br << ", " << wr << ", fma(" << bi << ", " << wi << ", " << fbr
                      << ")); " << fbi << " = fma(" << bi << ", " << wr << ", fma(-" << br << ", " << wi << ", " << fbi
                      << "));\n";
                    pass(n.w, "fma(" + br + ", " + far + ", " + bi + " * " + fai + ")",
                         "fma(" + bi + ", " + far + ", -" + br + " * " + fai + ")");
                }
                pass(n.u, br, bi);
            }
            o << "  }\n";
            for (int l : pt.leaves) {
                if (last_use[l] != static_cast<int>(p)) continue;
                // the slope from the leaf pair formed again, from opaque copies of
                // its argument (else the compiler merges it with the first
                // evaluation and keeps that one's values live through the sweep)
                const std::string L_ = std::to_string(l);
                o << "  { double yr = beta * (" << arg(l, false) << "), yi = beta * (" << arg(l, true)
                  << ");\n    AMI_OPAQUE(yr); AMI_OPAQUE(yi);\n    double fr, fi, mr, mi;\n    ami::leaf_complex_pair("
                  << (tb.leaf_sigma[l] < 0 ? "true" : "false")
                  << ", yr, yi, fr, fi, mr, mi);\n    const double Sr = -fma(fr, mr, -fi * mi), Si = fma(fr, mi, fi * mr);\n";
                o << "    const double Vr = fma(FBr" << L_ << ", Sr, -FBi" << L_ << " * Si), Vi = fma(FBr" << L_
                  << ", Si, FBi" << L_ << " * Sr);\n";
                o << "    gbeta = fma(Vr, " << arg(l, false) << ", fma(Vi, " << arg(l, true) << ", gbeta));\n";
                o << "    const double vr = Vr * beta, vi = Vi * beta;\n";
                for (int i = 0; i < ne; ++i) {
                    const double c = tb.leaf_coef[static_cast<size_t>(l) * ne + i];
                    if (c == 1.0) o << "    gEr[" << i << "] += vr; gEi[" << i << "] += vi;\n";
                    else if (c == -1.0) o << "    gEr[" << i << "] -= vr; gEi[" << i << "] -= vi;\n";
                    else if (c != 0.0)
                        o << "    gEr[" << i << "] = fma(" << num(c) << ", vr, gEr[" << i << "]); gEi[" << i << "] = fma("
                          << num(c) << ", vi, gEi[" << i << "]);\n";
                }
                o << "  }\n";
            }
            if ((p + 1) % kAdjLeafFenceParts == 0 && p + 1 < parts.size()) o << "  AMI_SCHED_FENCE();\n";
        }
        o << "}\n";
    }

    if (adj_fns) {
    // U_k = sum over the occurrences of k in the groups of u_g
    std::vector<std::vector<int>> occ(D);
    for (int g = 0; g < G; ++g)
        for (int j = gbegin(g); j < gend(g); ++j) occ[tb.group_den_list[j]].push_back(g);
    o << "__device__ __forceinline__ void den_cotangents(const double (&ur)[G], const double (&ui)[G], double "
         "(&Ur)[D], double (&Ui)[D]) {\n";
    o << kReverseContract;
    for (int k = 0; k < D; ++k) {
        Lin r, i;
        for (int g : occ[k]) {
            r.add(1.0, idx("ur", g));
            i.add(1.0, idx("ui", g));
        }
        o << "  Ur[" << k << "] = " << r.str() << ";\n  Ui[" << k << "] = " << i.str() << ";\n";
    }
    o << "}\n";

    // dL/dE_i += e_ki dR_k ; dL/dw_x += a_kx (dR_k, dI_k)
    auto scatter = [&](std::ostream &os, double c, const std::string &dst, const std::string &v) {
        if (c == 0.0) return;
        if (c == 1.0) os << "  " << dst << " += " << v << ";\n";
        else if (c == -1.0) os << "  " << dst << " -= " << v << ";\n";
        else os << "  " << dst << " = fma(" << num(c) << ", " << v << ", " << dst << ");\n";
    };
    o << "__device__ __forceinline__ void den_scatter(const double (&dR)[D], const double (&dI)[D], double (&gE)[NE], "
         "double (&gwr)["
      << NXA << "], double (&gwi)[" << NXA << "]) {\n";
    o << kReverseContract;
    o << "  (void)dR; (void)dI; (void)gE; (void)gwr; (void)gwi;\n";
    for (int k = 0; k < tb.D; ++k) {
        for (int i = 0; i < ne; ++i) scatter(o, tb.den_coef[static_cast<size_t>(k) * nc + i], idx("gE", i), idx("dR", k));
        for (int x = 0; x < nx; ++x) {
            const double a = tb.den_coef[static_cast<size_t>(k) * nc + ne + x];
            scatter(o, a, idx("gwr", x), idx("dR", k));
            scatter(o, a, idx("gwi", x), idx("dI", k));
        }
    }
    o << "}\n";

    // leaf cotangents: by a reverse sweep of each group's nested sum (parts of
    // at most kAdjLeafPartTerms terms, as the leaf pass of the adjoint in
    // passes), or by prefix/suffix products over each term's leaves
    o << "__device__ __forceinline__ void leaf_cotangents(const double (&F)[L], const double (&FTB)[G], double "
         "(&FB)[L]) {\n";
    o << kReverseContract;
    if (nested_part > 0) {
        std::vector<Part> parts;
        std::vector<int> first_use, last_use;
        build_parts(parts, first_use, last_use, nested_part);
        auto fname = [](int l) { return "F[" + std::to_string(l) + "]"; };
        for (size_t p = 0; p < parts.size(); ++p) {
            const Part &pt = parts[p];
            if (p > 0) o << "  AMI_SCHED_FENCE();\n";
            o << "  {\n";
            horner_emit(pt.nodes, fname, o);
            const size_t nn = pt.nodes.size();
            for (size_t k = 0; k < nn; ++k) o << "    double hb" << k << " = 0.0;\n";
            auto pass = [&](const HRef &r, const std::string &c) {
                if (r.kind == HRef::NODE) o << "    hb" << r.idx << (r.neg ? " -= " : " += ") << c << ";\n";
                else if (r.kind == HRef::LEAF) o << "    FB[" << r.idx << "]" << (r.neg ? " -= " : " += ") << c << ";\n";
            };
            pass(pt.root, "FTB[" + std::to_string(pt.g) + "]");
            for (size_t kk = nn; kk-- > 0;) {
                const HNode &n = pt.nodes[kk];
                const std::string hb = "hb" + std::to_string(kk), fa = fname(n.a),
                                  fb = "FB[" + std::to_string(n.a) + "]";
                if (n.w.kind == HRef::CONST) {
                    if (n.w.c == 1.0) o << "    " << fb << " += " << hb << ";\n";
                    else if (n.w.c == -1.0) o << "    " << fb << " -= " << hb << ";\n";
                    else o << "    " << fb << " = fma(" << num(n.w.c) << ", " << hb << ", " << fb << ");\n";
                } else {
                    const std::string wn = href_name(n.w, fname);
                    o << "    " << fb << " = fma(" << (n.w.neg ? "-" : "") << wn << ", " << hb << ", " << fb << ");\n";
                    pass(n.w, fa + " * " + hb);
                }
                pass(n.u, hb);
            }
            o << "  }\n";
        }
        o << "}\n";
    } else {
    for (int g = 0; g < G; ++g) {
        for (int ti = tb.group_start[g]; ti < tb.group_start[g + 1]; ++ti) {
            const double s = tb.term_sign[ti];
            std::vector<int> lv(ni);
            for (int j = 0; j < ni; ++j) lv[j] = tb.term_leaf[static_cast<size_t>(ti) * ni + j];
            // a unit sign goes into the update (a free negation), so that terms
            // sharing leading leaves share their prefix products
            const bool unit = s == 1.0 || s == -1.0;
            const char *sg = s == -1.0 ? "-" : "";
            o << "  { const double p0 = ";
            if (unit) o << "FTB[" << g << "]";
            else o << "FTB[" << g << "] * " << num(s);
            o << ";\n";
            for (int j = 1; j < ni; ++j)
                o << "    const double p" << j << " = p" << j - 1 << " * F[" << lv[j - 1] << "];\n";
            o << "    double q = 1.0;\n";
            for (int j = ni - 1; j >= 0; --j) {
                if (j == ni - 1) o << "    FB[" << lv[j] << "] " << (s == -1.0 ? "-=" : "+=") << " p" << j << ";\n";
                else o << "    FB[" << lv[j] << "] = fma(" << sg << "p" << j << ", q, FB[" << lv[j] << "]);\n";
                if (j > 0) {
                    if (j == ni - 1) o << "    q = F[" << lv[j] << "];\n";
                    else o << "    q *= F[" << lv[j] << "];\n";
                }
            }
            o << "    (void)q; }\n";
        }
    }
    o << "}\n";
    }

    // the same at complex energies: FB_l += sum over the terms holding l of
    // s FTB_g prod_(others) F, in complex arithmetic (the caller passes
    // conj(F), which makes the update FTB_g conj(dFT_g/dF_l))
    if (kernels & 256) {
    o << "__device__ __forceinline__ void leaf_cotangents_c(const double (&Fr)[L], const double (&Fi)[L], const double "
         "(&FTBr)[G], const double (&FTBi)[G], double (&FBr)[L], double (&FBi)[L]) {\n";
    o << kReverseContract;
    if (nested_part > 0) {
        // the reverse sweep of each group's nested sum at the given conj(F):
        // its node values are the conjugates of the true ones (real
        // coefficients), so a node h = F_a w + u passes hbar w to F_a and
        // hbar F_a to w as plain complex products
        std::vector<Part> parts;
        std::vector<int> first_use, last_use;
        build_parts(parts, first_use, last_use, nested_part);
        auto vre = [&](const HRef &r) -> std::string {
            if (r.kind == HRef::LEAF) return "Fr[" + std::to_string(r.idx) + "]";
            if (r.kind == HRef::NODE) return "h" + std::to_string(r.idx) + "r";
            return r.kind == HRef::CONST ? num(r.c) : std::string("0.0");
        };
        auto vim = [&](const HRef &r) -> std::string {
            if (r.kind == HRef::LEAF) return "Fi[" + std::to_string(r.idx) + "]";
            if (r.kind == HRef::NODE) return "h" + std::to_string(r.idx) + "i";
            return std::string("0.0");
        };
        auto sg = [](const HRef &r, const std::string &e) { return r.neg ? "(-" + e + ")" : e; };
        for (size_t p = 0; p < parts.size(); ++p) {
            const Part &pt = parts[p];
            if (p > 0) o << "  AMI_SCHED_FENCE();\n";
            o << "  {\n";
            const size_t nn = pt.nodes.size();
            for (size_t k = 0; k < nn; ++k) {
                const HNode &n = pt.nodes[k];
                const std::string far = "Fr[" + std::to_string(n.a) + "]", fai = "Fi[" + std::to_string(n.a) + "]";
                std::string ur = "0.0", ui = "0.0";
                if (n.u.kind == HRef::CONST) ur = num(n.u.c);
                else if (n.u.kind != HRef::ZERO) {
                    ur = sg(n.u, vre(n.u));
                    ui = sg(n.u, vim(n.u));
                }
                std::string hr, hi;
                if (n.w.kind == HRef::CONST) {
                    hr = "fma(" + num(n.w.c) + ", " + far + ", " + ur + ")";
                    hi = "fma(" + num(n.w.c) + ", " + fai + ", " + ui + ")";
                } else {
                    const std::string wr = sg(n.w, vre(n.w)), wi = sg(n.w, vim(n.w));
                    hr = "fma(" + far + ", " + wr + ", fma(-" + fai + ", " + wi + ", " + ur + "))";
                    hi = "fma(" + far + ", " + wi + ", fma(" + fai + ", " + wr + ", " + ui + "))";
                }
                o << "    const double h" << k << "r = " << hr << ", h" << k << "i = " << hi << ";\n";
            }
            for (size_t k = 0; k < nn; ++k) o << "    double hb" << k << "r = 0.0, hb" << k << "i = 0.0;\n";
            auto pass = [&](const HRef &r, const std::string &cr, const std::string &ci) {
                const char *op = r.neg ? " -= " : " += ";
                if (r.kind == HRef::NODE)
                    o << "    hb" << r.idx << "r" << op << cr << "; hb" << r.idx << "i" << op << ci << ";\n";
                else if (r.kind == HRef::LEAF)
                    o << "    FBr[" << r.idx << "]" << op << cr << "; FBi[" << r.idx << "]" << op << ci << ";\n";
            };
            pass(pt.root, "FTBr[" + std::to_string(pt.g) + "]", "FTBi[" + std::to_string(pt.g) + "]");
            for (size_t kk = nn; kk-- > 0;) {
                const HNode &n = pt.nodes[kk];
                const std::string br = "hb" + std::to_string(kk) + "r", bi = "hb" + std::to_string(kk) + "i";
                const std::string far = "Fr[" + std::to_string(n.a) + "]", fai = "Fi[" + std::to_string(n.a) + "]";
                const std::string fbr = "FBr[" + std::to_string(n.a) + "]", fbi = "FBi[" + std::to_string(n.a) + "]";
                if (n.w.kind == HRef::CONST) {
                    o << "    " << fbr << " = fma(" << num(n.w.c) << ", " << br << ", " << fbr << "); " << fbi
                      << " = fma(" << num(n.w.c) << ", " << bi << ", " << fbi << ");\n";
                } else {
                    const std::string wr = sg(n.w, vre(n.w)), wi = sg(n.w, vim(n.w));
                    o << "    " << fbr << " = fma(" << br << ", " << wr << ", fma(-" << bi << ", " << wi << ", " << fbr
                      << ")); " << fbi << " = fma(" << br << ", " << wi << ", fma(" << bi << ", " << wr << ", " << fbi
                      << "));\n";
                    pass(n.w, "fma(" + br + ", " + far + ", -" + bi + " * " + fai + ")",
                         "fma(" + br + ", " + fai + ", " + bi + " * " + far + ")");
                }
                pass(n.u, br, bi);
            }
            o << "  }\n";
        }
        o << "}\n";
    } else {
    for (int g = 0; g < G; ++g) {
        for (int ti = tb.group_start[g]; ti < tb.group_start[g + 1]; ++ti) {
            const double s = tb.term_sign[ti];
            std::vector<int> lv(ni);
            for (int j = 0; j < ni; ++j) lv[j] = tb.term_leaf[static_cast<size_t>(ti) * ni + j];
            const bool unit = s == 1.0 || s == -1.0;
            const std::string sg = s == -1.0 ? "-" : "";
            auto F = [&](const char *part, int j) { return std::string(part) + "[" + std::to_string(lv[j]) + "]"; };
            o << "  { const double p0r = FTBr[" << g << "]" << (unit ? "" : " * " + num(s)) << ", p0i = FTBi[" << g
              << "]" << (unit ? "" : " * " + num(s)) << ";\n";
            for (int j = 1; j < ni; ++j) {
                const std::string pr = "p" + std::to_string(j - 1) + "r", pi = "p" + std::to_string(j - 1) + "i";
                o << "    const double p" << j << "r = fma(" << pr << ", " << F("Fr", j - 1) << ", -" << pi << " * "
                  << F("Fi", j - 1) << "), p" << j << "i = fma(" << pr << ", " << F("Fi", j - 1) << ", " << pi
                  << " * " << F("Fr", j - 1) << ");\n";
            }
            o << "    double qr = 1.0, qi = 0.0;\n";
            for (int j = ni - 1; j >= 0; --j) {
                const std::string pr = "p" + std::to_string(j) + "r", pi = "p" + std::to_string(j) + "i";
                const std::string fbr = F("FBr", j), fbi = F("FBi", j);
                if (j == ni - 1) {
                    o << "    " << fbr << (s == -1.0 ? " -= " : " += ") << pr << ";\n";
                    o << "    " << fbi << (s == -1.0 ? " -= " : " += ") << pi << ";\n";
                } else {
                    o << "    " << fbr << " = fma(" << sg << pr << ", qr, fma(" << (s == -1.0 ? "" : "-") << pi
                      << ", qi, " << fbr << "));\n";
                    o << "    " << fbi << " = fma(" << sg << pr << ", qi, fma(" << sg << pi << ", qr, " << fbi
                      << "));\n";
                }
                if (j > 0) {
                    if (j == ni - 1) {
                        o << "    qr = " << F("Fr", j) << "; qi = " << F("Fi", j) << ";\n";
                    } else {
                        o << "    { const double tr = fma(qr, " << F("Fr", j) << ", -qi * " << F("Fi", j)
                          << "); qi = fma(qr, " << F("Fi", j) << ", qi * " << F("Fr", j) << "); qr = tr; }\n";
                    }
                }
            }
            o << "    (void)qr; (void)qi; }\n";
        }
    }
    o << "}\n";
    }
    }
    }  // adj_fns

    // the leaves' and lines' scatters: every adjoint kernel (one pass, or the
    // leaf pass of large solutions)
    if (adj_fns || (kernels & (128 | 8192 | 65536))) {
    auto scatter = [&](std::ostream &os, double c, const std::string &dst, const std::string &v) {
        if (c == 0.0) return;
        if (c == 1.0) os << "  " << dst << " += " << v << ";\n";
        else if (c == -1.0) os << "  " << dst << " -= " << v << ";\n";
        else os << "  " << dst << " = fma(" << num(c) << ", " << v << ", " << dst << ");\n";
    };
    // dL/dE_i += sum_l c_li v_l
    o << "__device__ __forceinline__ void leaf_scatter(const double (&v)[L], double (&gE)[NE]) {\n";
    o << kReverseContract;
    for (int l = 0; l < L; ++l)
        for (int i = 0; i < ne; ++i) scatter(o, tb.leaf_coef[static_cast<size_t>(l) * ne + i], idx("gE", i), idx("v", l));
    o << "}\n";

    // dL/dk_l += sum_j alpha_jl dL/dK_j
    o << "__device__ __forceinline__ void line_scatter(const double (&gx)[" << NGA << "], const double (&gy)[" << NGA
      << "], double (&gkx)[" << NIA << "], double (&gky)[" << NIA << "]) {\n";
    o << kReverseContract;
    if (hub) {
        for (int j = 0; j < ng; ++j)
            for (int l = 0; l < ni; ++l) {
                const double a = tb.line_alpha[static_cast<size_t>(j) * nf + l];
                scatter(o, a, idx("gkx", l), idx("gx", j));
                scatter(o, a, idx("gky", l), idx("gy", j));
            }
    }
    o << "}\n";
    }  // adjoint scatters
    o << "}  // namespace amijit\n";
    o << "#include \"jit_kernel.hpp\"\n";
    return o.str();
}

std::string jit_batch_source(const std::vector<const AmiTerms *> &items, const std::vector<int> &two_pass,
                             const std::vector<int> &one_row, bool hub, int block, int phases,
                             const std::vector<int> &labels, bool claim_ahead, int waves) {
    std::ostringstream o;
    o << "// generated: persistent batch of " << items.size() << " specialized evaluators\n";
    o << "#include \"kargs.hpp\"\n";
    // the tile functions read the argument blocks through the constant address space
    o << "#define AMI_JIT_ARGS const __attribute__((address_space(4))) ami::KArgs\n";
    const char *const kSettings[] = {"AMI_JIT_HUB", "AMI_JIT_KERNELS", "AMI_JIT_BLOCK", "AMI_JIT_PARK_DV",
                                     "AMI_JIT_ADJ_WAVES", "AMI_JIT_CADJ_WAVES", "AMI_JIT_CADJL_WAVES"};
    bool any_two = false;
    for (size_t j = 0; j < items.size(); ++j) {
        any_two = any_two || two_pass[j];
        std::string src = jit_source(items[j], hub, two_pass[j] ? (16 | 32) : 1);
        // the diagram's functions in a namespace of its own, with its settings
        // and the block of the batch, followed by the tile functions
        std::istringstream in(src);
        std::string line;
        for (const char *m : kSettings) o << "#undef " << m << "\n";
        o << "#define amijit amijit_b" << j << "\n";
        while (std::getline(in, line)) {
            if (line == "#include \"kargs.hpp\"" || line == "#include \"jit_kernel.hpp\"") continue;
            if (line.rfind("#define AMI_JIT_BLOCK ", 0) == 0) line = "#define AMI_JIT_BLOCK " + std::to_string(block);
            o << line << "\n";
        }
        o << "#include \"jit_tiles.hpp\"\n#undef amijit\n";
    }
    // the persistent kernels: every block takes work items (item, first tile,
    // tile count, first frequency row, row count) from its counter until the
    // list is done (every wave sees the counter pass n_work and exits) and runs
    // the item's own tile function on each tile (and row); the first kernel
    // runs the one-pass forward tiles and the two-pass items' first pass, the
    // second their frequency pass.  With claim_ahead the claim of the next
    // work item is issued before the current one runs, so that its round trip
    // overlaps the work.
    o << "namespace amibatch {\n"
         "struct Work {\n  int32_t item, ntiles;\n  int64_t tile0;\n  int32_t f, nf;\n};\n"
         "typedef const __attribute__((address_space(4))) Work *cwork;\n"
         "typedef const __attribute__((address_space(4))) ami::KArgs *cargs;\n"
         "}  // namespace amibatch\n";
    const std::string stride = std::to_string(kBatchCounterStride);
    for (int phase = 1; phase <= 2; ++phase) {
        if (!(phases & phase) || (phase == 2 && !any_two)) continue;
        // eight work lists, one per XCD (xoff[x] .. xoff[x + 1] of work, with
        // their counters kBatchCounterStride apart): a block drains the list
        // of its own XCD first (block b runs on XCD b mod 8), then the others
        // in turn, so every block has tried every list before it exits
        if (waves > 0) o << "__attribute__((amdgpu_waves_per_eu(" << waves << ")))\n";
        o << "extern \"C\" __global__ __launch_bounds__(" << block << ") void ami_batch_p" << phase
          << "(const ami::KArgs *args, const amibatch::Work *work, const int *xoff, unsigned int *counter) {\n"
             "  __shared__ int next;\n"
             "  const amibatch::cwork cw = (amibatch::cwork)(work);\n"
             "  const amibatch::cargs ca = (amibatch::cargs)(args);\n"
             "  const int x0 = static_cast<int>(blockIdx.x & 7u);\n"
             "  for (int k = 0; k < 8; ++k) {\n"
             "   const int x = (x0 + k) & 7, begin = xoff[x], n_work = xoff[x + 1] - begin;\n"
             "   unsigned int *const ctr = counter + " << stride << " * x;\n"
             "   if (threadIdx.x == 0) next = static_cast<int>(atomicAdd(ctr, 1u));\n"
             "   __syncthreads();\n"
             "   int wj = __builtin_amdgcn_readfirstlane(next);\n"
             "   __syncthreads();\n"
             "   while (wj < n_work) {\n";
        if (claim_ahead)
            o << "    unsigned int claim = 0u;\n"
                 "    if (threadIdx.x == 0) claim = atomicAdd(ctr, 1u);\n";
        o << "    const int wi = begin + wj;\n"
             "    const int item = cw[wi].item, ntiles = cw[wi].ntiles, f = cw[wi].f, nf = cw[wi].nf;\n"
             "    const int64_t tile0 = cw[wi].tile0;\n"
             "    const __attribute__((address_space(4))) ami::KArgs &a = ca[item];\n"
             "    (void)f;\n"
             "    (void)nf;\n"
             "    switch (item) {\n";
        for (size_t j = 0; j < items.size(); ++j) {
            const std::string ns = "amijit_b" + std::to_string(j);
            const std::string h = hub ? "true" : "false";
            const int label = labels.empty() ? static_cast<int>(j) : labels[j];
            if (phase == 1) {
                o << "    case " << label << ":\n      for (int64_t t = tile0; t < tile0 + ntiles; ++t) {\n"
                  << "        asm volatile(\"\" ::: \"memory\");   // each tile loads its own inputs\n        ";
                if (two_pass[j]) o << ns << "::sums_tile<" << h << ">(a, t);\n";
                else o << ns << "::fwd_tile<" << h << ", " << (one_row[j] ? "true" : "false")
                       << ">(a, t, 0, a.n_f);\n";
                o << "      }\n      break;\n";
            } else if (two_pass[j]) {
                o << "    case " << label << ":\n      for (int64_t t = tile0; t < tile0 + ntiles; ++t)\n"
                  << "        for (int r = f; r < f + nf; ++r) {\n"
                  << "          asm volatile(\"\" ::: \"memory\");   // each row loads its own inputs\n"
                  << "          " << ns << "::freq_tile(a, t, r);\n        }\n      break;\n";
            }
        }
        o << "    default: break;\n    }\n";
        o << (claim_ahead ? "    if (threadIdx.x == 0) next = static_cast<int>(claim);\n"
                          : "    if (threadIdx.x == 0) next = static_cast<int>(atomicAdd(ctr, 1u));\n");
        o << "    __syncthreads();\n"
             "    wj = __builtin_amdgcn_readfirstlane(next);\n"
             "    __syncthreads();\n"
             "   }\n  }\n}\n";
    }
    return o.str();
}

}  // namespace ami

extern "C" AmiStatus amiBatchSource(AmiTerms *const *terms, int32_t n, const int64_t *n_f, int32_t momentum,
                                    int32_t compile, char *buf, int64_t cap, int64_t *len) {
    using namespace ami;
    clear_error();
    if (!terms || !n_f || !len || n < 1) return fail(AMI_E_ARG, "NULL argument or no items");
    const bool hub = momentum != 0;
    std::vector<const AmiTerms *> ts;
    std::vector<int> two, one;
    for (int i = 0; i < n; ++i) {
        if (!terms[i]) return fail(AMI_E_ARG, "terms[" + std::to_string(i) + "] is NULL");
        two.push_back(jit_prefers_two_pass(terms[i]) ? 1 : 0);
        std::string why;
        if (!jit_supported(terms[i], hub, &why, two.back() != 0))
            return fail(AMI_E_UNSUPPORTED, "item " + std::to_string(i) + ": no specialized kernel: " + why);
        ts.push_back(terms[i]);
        one.push_back(n_f[i] == 1 ? 1 : 0);
    }
    const std::string src = jit_batch_source(ts, two, one, hub, 256, 3, {});
    if (compile) {
        std::vector<char> code;
        std::string err;
        const AmiStatus st = code_from_source(src, code, err);
        if (st != AMI_OK) return fail(st, err);
    }
    *len = static_cast<int64_t>(src.size()) + 1;
    if (!buf) return AMI_OK;
    if (cap < *len) return fail(AMI_E_ARG, "buffer too small");
    std::memcpy(buf, src.c_str(), src.size() + 1);
    return AMI_OK;
}

extern "C" AmiStatus amiTermsSource(const AmiTerms *t, int32_t momentum, char *buf, int64_t cap, int64_t *len) {
    using namespace ami;
    clear_error();
    if (!t || !len) return fail(AMI_E_ARG, "NULL argument");
    if (momentum < 0 || momentum > 3) return fail(AMI_E_ARG, "momentum must be 0..3");
    const bool hub = (momentum & 1) != 0, two_pass = (momentum & 2) != 0;
    std::string why;
    if (!jit_supported(t, hub, &why, two_pass)) return fail(AMI_E_UNSUPPORTED, "no specialized kernel: " + why);
    int kernels = two_pass ? (hub ? 48 | 64 | 128 : 48 | 64 | 128 | 512 | 1024 | 2048 | 4096) : hub ? 7 : 11 | 256;
    for (int o : t->tab.leaf_order)
        if (o > 0) kernels &= ~(8 | 256 | 512 | 1024 | 2048 | 4096);   // Taylor-coefficient leaves: no complex energies
    const std::string src = jit_source(t, hub, kernels);
    *len = static_cast<int64_t>(src.size()) + 1;
    if (!buf) return AMI_OK;
    if (cap < *len) return fail(AMI_E_ARG, "buffer too small");
    std::memcpy(buf, src.c_str(), src.size() + 1);
    return AMI_OK;
}
