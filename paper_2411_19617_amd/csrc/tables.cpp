// Host-side constant tables of the descriptor kernels.
//
// Clebsch-Gordan coefficients <j1 m1 j2 m2 | j m> are built by coupling:
// the stretched state |j1+j2, j1+j2> = |j1 j1>|j2 j2> is lowered with
// J- = J1- + J2-; each lower j starts from the vector of the M = j subspace
// orthogonal to all states of larger j (Gram-Schmidt), with the
// Condon-Shortley phase <j1 j1, j2 (j-j1) | j j> > 0, and is lowered in turn.
// This is a different route from the closed Racah sum.
//
// Table layout per descriptor triple, in its contraction orientation
// (A, B -> C) (doubled): a dense (A+1) x (C+1) block
// c[ma1*(C+1) + ma] = <a m1 b m2 | c m> with ma1 = a + m1, ma = c + m,
// m2 = m - m1 (zero where m2 is out of range).
#include <math.h>
#include <string.h>

#include <algorithm>
#include <array>
#include <vector>

#include "ace.h"
#include "mala_internal.h"
#include "snap_core.h"

namespace mala {

namespace {

// coupled[J][ma][ma1] for fixed (J1, J2): coefficient of |ma1, ma2 = ma - ma1 + (J1+J2-J)/2>
struct Coupling {
    int J1, J2;
    // index (J, ma, ma1, ma2) flattened over the product basis
    std::vector<std::vector<std::vector<double>>> vec;  // [Jidx][ma] -> product-basis vector
};

inline int pidx(int J2, int a1, int a2) { return a1 * (J2 + 1) + a2; }

Coupling couple(int J1, int J2) {
    Coupling c;
    c.J1 = J1;
    c.J2 = J2;
    const int dim = (J1 + 1) * (J2 + 1);
    const int nJ = std::min(J1, J2) + 1;   // J = J1+J2, J1+J2-2, ..., |J1-J2|
    c.vec.assign(nJ, {});
    // lowering: J-|j,m> = sqrt((j+m)(j-m+1)) |j,m-1>; doubled: ma = j+m, so
    // (j+m)(j-m+1) = ma * (J - ma + 1) with J doubled.
    auto lower = [&](const std::vector<double>& v) {
        std::vector<double> out(dim, 0.0);
        for (int a1 = 0; a1 <= J1; ++a1)
            for (int a2 = 0; a2 <= J2; ++a2) {
                const double x = v[pidx(J2, a1, a2)];
                if (x == 0.0) continue;
                if (a1 >= 1) out[pidx(J2, a1 - 1, a2)] += x * sqrt((double)a1 * (J1 - a1 + 1));
                if (a2 >= 1) out[pidx(J2, a1, a2 - 1)] += x * sqrt((double)a2 * (J2 - a2 + 1));
            }
        return out;
    };
    for (int t = 0; t < nJ; ++t) {
        const int J = J1 + J2 - 2 * t;
        // top state: M = J/2, i.e. a1 + a2 = (J + J1 + J2)/2
        const int S = (J + J1 + J2) / 2;
        std::vector<double> top(dim, 0.0);
        // start from the product state with a1 = J1 (m1 = j1), orthogonalise
        top[pidx(J2, J1, S - J1)] = 1.0;
        for (int u = 0; u < t; ++u) {
            const int Ju = J1 + J2 - 2 * u;
            const std::vector<double>& w = c.vec[u][(Ju + J) / 2];   // |Ju, M = J/2>: ma = Ju/2 + J/2
            double dot = 0.0;
            for (int i = 0; i < dim; ++i) dot += w[i] * top[i];
            for (int i = 0; i < dim; ++i) top[i] -= dot * w[i];
        }
        double nrm = 0.0;
        for (int i = 0; i < dim; ++i) nrm += top[i] * top[i];
        nrm = sqrt(nrm);
        for (int i = 0; i < dim; ++i) top[i] /= nrm;
        if (top[pidx(J2, J1, S - J1)] < 0)
            for (int i = 0; i < dim; ++i) top[i] = -top[i];
        c.vec[t].assign(J + 1, std::vector<double>());
        c.vec[t][J] = top;
        for (int ma = J; ma >= 1; --ma) {
            std::vector<double> v = lower(c.vec[t][ma]);
            const double f = sqrt((double)ma * (J - ma + 1));
            for (int i = 0; i < dim; ++i) v[i] /= f;
            c.vec[t][ma - 1] = v;
        }
    }
    return c;
}

}  // namespace

// Returns the number of floats written, or -1 if cap is too small.  Triple t
// gets the block of its contraction orientation (A, B -> C) of zb_perm.
int build_cg_table(int twojmax, float* table, int* offsets, int cap) {
    int n = 0;
    std::vector<Coupling> cache((twojmax + 1) * (twojmax + 1));
    std::vector<bool> have(cache.size(), false);
    for (int t = 0; t < n_triples(twojmax); ++t) {
        const ZbPerm p = zb_perm(twojmax, t);
        const int A = p.a, B = p.b, C = p.c;
        const int key = A * (twojmax + 1) + B;
        if (!have[key]) {
            cache[key] = couple(A, B);
            have[key] = true;
        }
        const Coupling& c = cache[key];
        const int D = (A + B - C) / 2;       // also the index of C in the coupling's list
        offsets[t] = n;
        const int sz = (A + 1) * (C + 1);
        if (n + sz > cap) return -1;
        for (int ma1 = 0; ma1 <= A; ++ma1)
            for (int ma = 0; ma <= C; ++ma) {
                const int ma2 = ma - ma1 + D;
                double v = 0.0;
                if (ma2 >= 0 && ma2 <= B) v = c.vec[D][ma][pidx(B, ma1, ma2)];
                table[n + ma1 * (C + 1) + ma] = (float)v;
            }
        n += sz;
    }
    return n;
}

// The same blocks for every coupled pair (A, B -> C) of the descriptor
// adjoint (combo_of order).
int build_cg_table_adjoint(int twojmax, float* table, int* offsets, int cap) {
    int n = 0;
    std::vector<Coupling> cache((twojmax + 1) * (twojmax + 1));
    std::vector<bool> have(cache.size(), false);
    for (int k = 0; k < n_combos(twojmax); ++k) {
        const Combo cb = combo_of(twojmax, k);
        const int A = cb.a, B = cb.b, C = cb.c;
        const int key = A * (twojmax + 1) + B;
        if (!have[key]) {
            cache[key] = couple(A, B);
            have[key] = true;
        }
        const Coupling& c = cache[key];
        const int D = (A + B - C) / 2;
        offsets[k] = n;
        const int sz = (A + 1) * (C + 1);
        if (n + sz > cap) return -1;
        for (int ma1 = 0; ma1 <= A; ++ma1)
            for (int ma = 0; ma <= C; ++ma) {
                const int ma2 = ma - ma1 + D;
                double v = 0.0;
                if (ma2 >= 0 && ma2 <= B) v = c.vec[D][ma][pidx(B, ma1, ma2)];
                table[n + ma1 * (C + 1) + ma] = (float)v;
            }
        n += sz;
    }
    return n;
}

// Work units of the adjoint contraction: output level C (c_lo..c_hi) and
// column mb, each summing Z^C(A, B)[., mb] over the coupled pairs of C.
// Assigned to the waves of a block by longest processing time; wave_units[w*stride] = count,
// followed by the units (C * 32 + mb).
void plan_y_units(int twojmax, int c_lo, int c_hi, int n_waves, int* wave_units, int stride) {
    std::vector<std::pair<double, int>> jobs;
    for (int C = c_lo; C <= c_hi; ++C)
        for (int mb = 0; mb <= C; ++mb) {
            double cost = 0.0;
            for (int k = combo_first(twojmax, C); k < n_combos(twojmax) && combo_of(twojmax, k).c == C; ++k) {
                const Combo cb = combo_of(twojmax, k);
                const int A = cb.a, B = cb.b, D = (A + B - C) / 2, HR = C / 2;
                int t = 0;
                for (int ma = 0; ma <= HR; ++ma)
                    for (int ma1 = 0; ma1 <= A; ++ma1)
                        if (zb_pair_ok(A, B, C, ma, ma1) && (C % 2 || ma < HR || mb <= HR)) ++t;
                const int lo = mb + D - B > 0 ? mb + D - B : 0, hi = A < mb + D ? A : mb + D;
                cost += (hi - lo + 1) * (4.0 * t + zy_scale_ops(A, B, C) + 6.0) + 2.0 * t + 4.0;
            }
            jobs.push_back({cost, C * 32 + mb});
        }
    std::stable_sort(jobs.begin(), jobs.end(),
                     [](const std::pair<double, int>& a, const std::pair<double, int>& b) {
                         return a.first > b.first;
                     });
    std::vector<double> load(n_waves, 0.0);
    std::vector<std::vector<int>> lists(n_waves);
    for (auto& jb : jobs) {
        int w = (int)(std::min_element(load.begin(), load.end()) - load.begin());
        load[w] += jb.first;
        lists[w].push_back(jb.second);
    }
    for (int w = 0; w < n_waves; ++w) {
        wave_units[w * stride] = (int)lists[w].size();
        for (size_t i = 0; i < lists[w].size(); ++i) wave_units[w * stride + 1 + i] = lists[w][i];
    }
}

// Rank-3 descriptors: multisets of three (n, l) that obey the triangle rule, with an even l-sum.
int ace_count_rank3(int nmax, int lmax) {
    const int nl = lmax + 1, np = nmax * nl;
    int nd = 0;
    for (int p1 = 0; p1 < np; ++p1)
        for (int p2 = p1; p2 < np; ++p2)
            for (int p3 = p2; p3 < np; ++p3) {
                const int l1 = p1 % nl, l2 = p2 % nl, l3 = p3 % nl;
                nd += l3 >= abs(l1 - l2) && l3 <= l1 + l2 && (l1 + l2 + l3) % 2 == 0;
            }
    return nd;
}

// Plan of ranks 1-3 (layout in ace.h).  Rank-3 columns follow the order
// p1 <= p2 <= p3 of the keys p = n (lmax+1) + l.  The pairs of one (l1, l2), those
// whose later key has the largest n first so that a round's outputs start at as
// high an n3 as they can, fill rounds; runs of rounds go to the waves by cost
// (VALU instructions), longest first to the least loaded.
void build_ace_plan(int nmax, int lmax, int groups, std::vector<int>& plan) {
    const int nl = lmax + 1, np = nmax * nl;
    std::vector<int> col(np * np, 0);                // first column of (p1, p2)
    int next = ace_count_ranks12(nmax, lmax);
    for (int p1 = 0; p1 < np; ++p1)
        for (int p2 = p1; p2 < np; ++p2) {
            col[p1 * np + p2] = next;
            const int l1 = p1 % nl, l2 = p2 % nl;
            for (int p3 = p2; p3 < np; ++p3) {
                const int l3 = p3 % nl;
                next += l3 >= abs(l1 - l2) && l3 <= l1 + l2 && (l1 + l2 + l3) % 2 == 0;
            }
        }
    struct Run { long cost; std::vector<int> rounds; };
    struct Pair { int n1, n2, later, first, col; };  // later: n of the later key
    std::vector<Run> runs;
    // one run: the pairs in rounds; set up once, `each` per round, `third` per n3 a round forms
    auto add = [&](int kind, const std::vector<Pair>& pairs, long setup, long each, long third) {
        Run r{setup, {}};
        for (size_t i = 0; i < pairs.size(); i += groups) {
            int lo = nmax;
            std::vector<int> entry(groups, 15 << 4);
            for (size_t g = 0; g < (size_t)groups && i + g < pairs.size(); ++g) {
                const Pair& p = pairs[i + g];
                lo = std::min(lo, p.later);
                entry[g] = p.n1 | p.n2 << 2 | p.first << 4 | p.col << 8;
            }
            r.rounds.push_back(kind | lo << 8);
            r.rounds.insert(r.rounds.end(), entry.begin(), entry.end());
            r.cost += each + third * (nmax - lo);
        }
        if (!r.rounds.empty()) runs.push_back(r);
    };
    std::vector<Pair> pairs;
    for (int n = 0; n < nmax; ++n) pairs.push_back({n, 0, 0, 0, n});
    add(kAceRank1, pairs, 10, 15, 0);
    for (int l = 0; l <= lmax; ++l) {
        pairs.clear();
        int c = nmax + l * nmax * (nmax + 1) / 2;
        for (int n1 = 0; n1 < nmax; ++n1)
            for (int n2 = n1; n2 < nmax; ++n2) pairs.push_back({n1, n2, 0, 0, c++});
        add(kAceRank2 + l, pairs, 10, 20 + 4 * l, 0);
    }
    for (int l1 = 0; l1 <= lmax; ++l1)
        for (int l2 = l1; l2 <= lmax; ++l2) {
            long each = 30, third = 0, reads = 0;
            int below1 = 0, below2 = 0, n_l3 = 0;    // of the l3: below l1, below l2, all
            for (int l3 = l2 - l1; l3 <= l1 + l2 && l3 <= lmax; l3 += 2) {
                below1 += l3 < l1;
                below2 += l3 < l2;
                ++n_l3;
            }
            for (int M = 0; M <= l1 + l2; ++M) {
                int terms = 0, nl3 = 0;
                for (int m = -l1; m <= l1; ++m) terms += abs(M - m) <= l2;
                for (int l3 = l2 - l1; l3 <= l1 + l2 && l3 <= lmax; l3 += 2) nl3 += l3 >= M;
                if (nl3 == 0) continue;
                each += M ? terms * (4 + 2 * nl3) : (terms + 1) / 2 * (2 + nl3);
                third += nl3 * (M ? 2 : 1);
                reads += nl3;
            }
            third += 3 * n_l3;
            pairs.clear();
            for (int later = nmax - 1; later >= 0; --later)
                for (int n = 0; n <= later; ++n) {
                    // (n l1) (later l2), and, other than for one l, (n l2) (later l1) with n < later
                    const int f2 = later * n_l3 + below2, f1 = later * n_l3 + below1;
                    if (f2 < nmax * n_l3) pairs.push_back({n, later, later, f2, col[(n * nl + l1) * np + later * nl + l2]});
                    if (l1 < l2 && n < later && f1 < nmax * n_l3)
                        pairs.push_back({later, n, later, f1, col[(n * nl + l2) * np + later * nl + l1]});
                }
            add(l1 * (kAceMaxL + 1) + l2, pairs, 60 + 8 * reads, each, third);
        }
    std::stable_sort(runs.begin(), runs.end(), [](const Run& a, const Run& b) { return a.cost > b.cost; });
    std::vector<long> load(kAce3Waves, 0);
    std::vector<std::vector<int>> lists(kAce3Waves);
    for (const Run& x : runs) {
        const int w = (int)(std::min_element(load.begin(), load.end()) - load.begin());
        load[w] += x.cost;
        lists[w].insert(lists[w].end(), x.rounds.begin(), x.rounds.end());
    }
    plan.assign(kAce3Waves + 1, 0);
    for (int w = 0; w < kAce3Waves; ++w) {
        plan[w] = (int)plan.size();
        plan.insert(plan.end(), lists[w].begin(), lists[w].end());
    }
    plan[kAce3Waves] = (int)plan.size();
}

// Rank-4 grid ACE (Eq. ace_grid with four factors, one intermediate
// coupling L): for keys p = n (lmax4+1) + l,
//   B(p1 p2 p3 p4; L) = sum over m of <l1 m1 l2 m2 | L M> <l3 m3 l4 m4 | L -M>
//                       (-1)^(L-M)/sqrt(2L+1) A_p1 A_p2 A_p3 A_p4.
// The set: multisets p1 <= p2 <= p3 <= p4 with an even l-sum; for each, the
// couplings L (in increasing order) whose coefficients, summed over the
// permutations that exchange equal keys, are linearly independent of those
// kept before.  Without equal keys every L is; an equal pair inside (p1 p2) or
// (p3 p4) leaves the even L; where p2 = p3 the first L are, as many as the
// symmetric states allow (a count, no coefficients: Gram-Schmidt on the
// coefficient tensors gives the same set and took 4.9 ms at nmax4 = lmax4 = 3,
// this takes 2 us, and a caller that sizes its output asks on every call).
// Evaluation: with the coupled pairs P_a(M) = sum_m1 <l1 m1 l2 m2|L M>
// A_p1,m1 A_p2,m2 (a = (p1 p2), m2 = M - m1) and A_{l,-m} = (-1)^m conj A_{l,m},
// P_a(-M) = (-1)^(l1+l2-L+M) conj P_a(M); for an even l-sum the descriptor is
//   B = (-1)^(l3+l4-L) (-1)^L / sqrt(2L+1)
//       [Re P_a(0) conj P_b(0) + 2 sum_{M>=1} Re P_a(M) conj P_b(M)],
// so only M >= 0 of every pair is formed.  Tables per L: pair units
// (coefficient block, (l1, l2, L) combination, LDS slot of P_a(0), storage
// bases of the two keys), one Clebsch-Gordan block per combination, and
// descriptors (slot of P_a(0), slot of P_b(0), output position, factor).
namespace {

struct Ace4Cg {
    std::vector<Coupling> cache = std::vector<Coupling>(25 * 25);
    std::vector<bool> have = std::vector<bool>(25 * 25, false);
    // <l1 m1 l2 m2 | L M> from the coupled states of couple()
    double operator()(int l1, int m1, int l2, int m2, int L, int M) {
        if (m1 + m2 != M || abs(m1) > l1 || abs(m2) > l2 || abs(M) > L || L < abs(l1 - l2) || L > l1 + l2)
            return 0.0;
        const int key = 2 * l1 * 25 + 2 * l2;
        if (!have[key]) {
            cache[key] = couple(2 * l1, 2 * l2);
            have[key] = true;
        }
        return cache[key].vec[l1 + l2 - L][L + M][pidx(2 * l2, l1 + m1, l2 + m2)];
    }
};

}  // namespace

namespace {

// Multiplicity of the angular momentum `total` in the symmetric product of k
// equal momenta l: the symmetric states of sum M = total less those of total + 1.
int sym_multiplicity(int l, int k, int total) {
    // ways[s]: multisets of k values from 0..2l of sum s (m + l each)
    std::array<std::array<int, 4 * 2 * kAce4MaxL + 1>, 5> ways{};
    ways[0][0] = 1;
    for (int m = 0; m <= 2 * l; ++m)
        for (int j = 1; j <= k; ++j)
            for (int s = m; s <= 2 * l * k; ++s) ways[j][s] += ways[j - 1][s - m];
    const int at = total + k * l;
    return at > 2 * l * k ? 0 : ways[k][at] - (at + 1 > 2 * l * k ? 0 : ways[k][at + 1]);
}

// How many couplings L of (l1 l2)(l3 l4) are independent after symmetrising
// over equal keys, where the second and third key are equal.
int ace4_independent(int l1, int l, int l4, bool eq12, bool eq34) {
    if (eq12 && eq34) return sym_multiplicity(l, 4, 0);
    if (eq12) return sym_multiplicity(l, 3, l4);
    if (eq34) return sym_multiplicity(l, 3, l1);
    int n = 0;                                       // even couplings of (l2 l3) that reach (l1 l4)
    for (int L = 0; L <= 2 * l; L += 2) n += L >= abs(l1 - l4) && L <= l1 + l4;
    return n;
}

}  // namespace

int ace4_descriptor_set(int nmax4, int lmax4, std::vector<int>& desc) {
    desc.clear();
    const int nl = lmax4 + 1, np = nmax4 * nl;
    desc.reserve((size_t)5 * 1024);
    for (int p1 = 0; p1 < np; ++p1)
        for (int p2 = p1; p2 < np; ++p2)
            for (int p3 = p2; p3 < np; ++p3)
                for (int p4 = p3; p4 < np; ++p4) {
                    const int l1 = p1 % nl, l2 = p2 % nl, l3 = p3 % nl, l4 = p4 % nl;
                    if ((l1 + l2 + l3 + l4) % 2) continue;
                    const bool eq12 = p1 == p2, eq34 = p3 == p4;
                    // (l l) of equal keys couples to even L only
                    const int step = eq12 || eq34 ? 2 : 1;
                    int L = std::max(abs(l1 - l2), abs(l3 - l4));
                    const int hi = std::min(l1 + l2, l3 + l4);
                    if (step == 2) L += L & 1;
                    int left = p2 == p3 ? ace4_independent(l1, l2, l4, eq12, eq34) : hi + 1;
                    for (; L <= hi && left > 0; L += step, --left) {
                        const int d[5] = {p1, p2, p3, p4, L};
                        desc.insert(desc.end(), d, d + 5);
                    }
                }
    return (int)(desc.size() / 5);
}

int build_ace4_tables(int nmax4, int lmax4, std::vector<int>& l_units, std::vector<int4>& units,
                      std::vector<float>& coef, std::vector<int>& l_descs, std::vector<int4>& descs,
                      int& max_slots) {
    std::vector<int> set;
    const int n4 = ace4_descriptor_set(nmax4, lmax4, set);
    Ace4Cg cg;
    const int nl = lmax4 + 1;
    l_units.assign(1, 0);
    l_descs.assign(1, 0);
    units.clear();
    coef.clear();
    descs.clear();
    max_slots = 0;
    // per L: the pairs it needs, in first-use order, each with L+1 slots,
    // and its descriptors (first pair slot, second pair slot, output, l3+l4)
    struct LPart {
        std::vector<std::pair<int, int>> pairs;
        std::vector<std::array<int, 4>> dl;
        int slots() const { return (int)pairs.size(); }
    };
    std::vector<LPart> part(2 * lmax4 + 1);
    for (int L = 0; L <= 2 * lmax4; ++L) {
        LPart& P = part[L];
        auto slot_of = [&](int pa, int pb) {
            for (size_t i = 0; i < P.pairs.size(); ++i)
                if (P.pairs[i].first == pa && P.pairs[i].second == pb) return (int)i * (L + 1);
            P.pairs.push_back({pa, pb});
            return (int)(P.pairs.size() - 1) * (L + 1);
        };
        for (int k = 0; k < n4; ++k) {
            const int* d = &set[5 * k];
            if (d[4] != L) continue;
            P.dl.push_back({slot_of(d[0], d[1]), slot_of(d[2], d[3]), k, (d[2] % nl + d[3] % nl)});
        }
    }
    // phases: several L share one pass (one pair formation, one evaluation,
    // two barriers) while their slots fit the LDS budget and their entries
    // the staged table; first fit, largest L first
    const int slot_cap = (int)(kAce4LdsBudget / (sizeof(float) * 2 * 64));
    std::vector<int> order;
    for (int L = 0; L <= 2 * lmax4; ++L)
        if (!part[L].dl.empty()) order.push_back(L);
    auto slots_of = [&](int L) { return part[L].slots() * (L + 1); };
    std::stable_sort(order.begin(), order.end(), [&](int a, int b) { return slots_of(a) > slots_of(b); });
    std::vector<std::vector<int>> phases;
    std::vector<int> ph_slots, ph_descs;
    for (int L : order) {
        size_t i = 0;
        for (; i < phases.size(); ++i)
            if (ph_slots[i] + slots_of(L) <= slot_cap && ph_descs[i] + (int)part[L].dl.size() <= kAce4MaxDescsL)
                break;
        if (i == phases.size()) {
            phases.push_back({});
            ph_slots.push_back(0);
            ph_descs.push_back(0);
        }
        phases[i].push_back(L);
        ph_slots[i] += slots_of(L);
        ph_descs[i] += (int)part[L].dl.size();
    }
    std::vector<int> block_of(4 * 4 * 7, -1);        // (l1, l2, L) with l <= 3, L <= 6
    for (auto& ph : phases) {
        std::sort(ph.begin(), ph.end());
        std::vector<std::array<int, 5>> dl;           // slot a, slot b, output, l3+l4, L
        int base = 0;
        for (int L : ph) {
            const LPart& P = part[L];
            for (const auto& x : P.dl) dl.push_back({x[0] + base, x[1] + base, x[2], x[3], L});
            // one unit per pair: P_a(M) for M = 0..L by code specialised for
            // (l1, l2, L), with the Clebsch-Gordan coefficients of that
            // combination in one block, ordered M = 0..L, m1 = -l1..l1 with
            // |M - m1| <= l2 (zeros included)
            for (size_t i = 0; i < P.pairs.size(); ++i) {
                const int pa = P.pairs[i].first, pb = P.pairs[i].second;
                const int n1 = pa / nl, l1 = pa % nl, n2 = pb / nl, l2 = pb % nl;
                const int combo = (l1 * 4 + l2) * 7 + L;
                if (block_of[combo] < 0) {
                    block_of[combo] = (int)coef.size();
                    for (int M = 0; M <= L; ++M)
                        for (int m1 = -l1; m1 <= l1; ++m1) {
                            const int m2 = M - m1;
                            if (abs(m2) > l2) continue;
                            coef.push_back((float)cg(l1, m1, l2, m2, L, M));
                        }
                }
                const int base1 = n1 * 15 + l1 * (l1 + 1) / 2, base2 = n2 * 15 + l2 * (l2 + 1) / 2;
                units.push_back(make_int4(block_of[combo], combo, base + (int)i * (L + 1), base1 | (base2 << 8)));
            }
            base += slots_of(L);
        }
        // descriptors sharing their first pair next to each other
        std::stable_sort(dl.begin(), dl.end(), [](const std::array<int, 5>& x, const std::array<int, 5>& y) {
            return x[0] < y[0];
        });
        for (const auto& x : dl) {
            const double f = ((x[3] & 1) ? -1.0 : 1.0) / sqrt(2.0 * x[4] + 1.0);   // (-1)^(l3+l4-L) (-1)^L
            float ff = (float)f;
            int fb;
            memcpy(&fb, &ff, 4);
            descs.push_back(make_int4(x[0] | (x[4] << 16), x[1], x[2], fb));
        }
        max_slots = std::max(max_slots, base);
        l_units.push_back((int)units.size());
        l_descs.push_back((int)descs.size());
    }
    return n4;
}

// Plan of the point-major rank-4 kernel (layout in ace.h).  The pair (p1, p2) with
// l1 > l2 is formed as (p2, p1): <l2 m2 l1 m1|L M> = (-1)^(l1+l2-L) <l1 m1 l2 m2|L M>
// goes into the descriptors' signs.
void build_ace4_rows_plan(int nmax4, int lmax4, std::vector<int>& plan, int& n_slots) {
    constexpr int G = kTile / kAce4RowPoints, W = kAce4RowWaves;
    std::vector<int> set;
    const int n4 = ace4_descriptor_set(nmax4, lmax4, set);
    const int nl = lmax4 + 1, np = nmax4 * nl, nL = 2 * kAce4MaxL + 1;
    std::vector<int> slot((size_t)np * np * nL, -1);
    n_slots = 0;
    struct Desc { int L, sa, sb, out, neg; };
    std::vector<Desc> descs;
    for (int k = 0; k < n4; ++k) {
        const int* d = &set[5 * k];
        const int L = d[4];
        int s[2], neg = (d[2] % nl + d[3] % nl) & 1;             // (-1)^(l3+l4-L) (-1)^L
        for (int h = 0; h < 2; ++h) {
            const int pa = d[2 * h], pb = d[2 * h + 1], la = pa % nl, lb = pb % nl;
            int& at = slot[((size_t)pa * np + pb) * nL + L];
            if (at < 0) {
                at = n_slots;
                n_slots += L + 1;
            }
            s[h] = at;
            if (la > lb) neg ^= (la + lb - L) & 1;
        }
        descs.push_back({L, s[0], s[1], k, neg});
    }
    const int spare = n_slots;
    n_slots += nL;
    std::stable_sort(descs.begin(), descs.end(), [](const Desc& x, const Desc& y) {
        return x.L != y.L ? x.L < y.L : x.sa < y.sa;
    });
    // rounds of pairs of one (l1, l2), dealt by cost, longest first to the least loaded
    std::vector<std::pair<long, std::vector<int>>> rounds;
    for (int l1 = 0; l1 <= lmax4; ++l1)
        for (int l2 = l1; l2 <= lmax4; ++l2) {
            long cost = 30;
            for (int M = 0; M <= l1 + l2; ++M)
                for (int m = -l1; m <= l1; ++m)
                    if (abs(M - m) <= l2) cost += 4 + 2 * (l1 + l2 - std::max(M, l2 - l1) + 1);
            std::vector<std::array<int, kAce4PairInts>> pairs;
            for (int pa = 0; pa < np; ++pa)
                for (int pb = pa; pb < np; ++pb) {
                    const int la = pa % nl, lb = pb % nl;
                    if (std::min(la, lb) != l1 || std::max(la, lb) != l2) continue;
                    std::array<int, kAce4PairInts> e{};
                    e[0] = la <= lb ? pa / nl | pb / nl << 2 : pb / nl | pa / nl << 2;
                    bool used = false;
                    for (int i = 0; i <= 2 * l1; ++i) {
                        const int at = slot[((size_t)pa * np + pb) * nL + l2 - l1 + i];
                        used = used || at >= 0;
                        e[1 + i / 3] |= (at < 0 ? spare : at) << (10 * (i % 3));
                    }
                    if (used) pairs.push_back(e);
                }
            std::array<int, kAce4PairInts> none{};
            for (int i = 0; i <= 2 * l1; ++i) none[1 + i / 3] |= spare << (10 * (i % 3));
            for (size_t i = 0; i < pairs.size(); i += G) {
                std::vector<int> r(1, l1 * (kAce4MaxL + 1) + l2);
                for (size_t g = 0; g < (size_t)G; ++g) {
                    const auto& e = i + g < pairs.size() ? pairs[i + g] : none;
                    r.insert(r.end(), e.begin(), e.end());
                }
                rounds.push_back({cost, r});
            }
        }
    std::stable_sort(rounds.begin(), rounds.end(), [](const auto& a, const auto& b) { return a.first > b.first; });
    std::vector<long> load(W, 0);
    std::vector<std::vector<int>> lists(W);
    for (const auto& x : rounds) {
        const int w = (int)(std::min_element(load.begin(), load.end()) - load.begin());
        load[w] += x.first;
        lists[w].insert(lists[w].end(), x.second.begin(), x.second.end());
    }
    plan.assign(W + 1 + nL + 1, 0);
    for (int w = 0; w < W; ++w) {
        plan[w] = (int)plan.size();
        plan.insert(plan.end(), lists[w].begin(), lists[w].end());
    }
    plan[W] = (int)plan.size();
    const int d0 = (int)plan.size();
    for (int L = 0, k = 0; L <= nL; ++L) {
        while (k < n4 && descs[k].L < L) ++k;
        plan[W + 1 + L] = d0 + k;
    }
    for (const Desc& d : descs)
        plan.push_back((int)((unsigned)d.sa | (unsigned)d.sb << 10 | (unsigned)d.out << 20 | (unsigned)d.neg << 31));
}

// Longest-processing-time assignment of triples to the waves of a block.
// wave_triples[w*stride] = count, followed by the triple indices.
void plan_zb_waves(int twojmax, int n_waves, int* wave_triples, int stride) {
    std::vector<std::pair<double, int>> jobs;
    for (int t = 0; t < n_triples(twojmax); ++t) {
        const ZbPerm p = zb_perm(twojmax, t);
        jobs.push_back({zb_cost(p.a, p.b, p.c), t});
    }
    std::stable_sort(jobs.begin(), jobs.end(),
                     [](const std::pair<double, int>& a, const std::pair<double, int>& b) {
                         return a.first > b.first;
                     });
    std::vector<double> load(n_waves, 0.0);
    std::vector<std::vector<int>> lists(n_waves);
    for (auto& jb : jobs) {
        int w = (int)(std::min_element(load.begin(), load.end()) - load.begin());
        load[w] += jb.first;
        lists[w].push_back(jb.second);
    }
    for (int w = 0; w < n_waves; ++w) {
        std::sort(lists[w].begin(), lists[w].end());
        wave_triples[w * stride] = (int)lists[w].size();
        for (size_t i = 0; i < lists[w].size(); ++i) wave_triples[w * stride + 1 + i] = lists[w][i];
    }
}

}  // namespace mala
