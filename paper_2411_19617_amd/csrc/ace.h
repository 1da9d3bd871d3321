// Host interface of the grid ACE descriptor kernel (ace.hip) and its
// rank-3 term tables (tables.cpp).
#pragma once
#include <vector>
#include "mala_internal.h"

namespace mala {

constexpr int kAceMaxN = 4;      // radial functions
constexpr int kAceMaxL = 4;      // angular momentum

inline int ace_count_ranks12(int nmax, int lmax) { return nmax + (lmax + 1) * nmax * (nmax + 1) / 2; }
int ace_count_rank3(int nmax, int lmax);         // descriptors of the rank-3 set
// Plan of ranks 1-3 for kAce3Waves waves whose lanes form `groups` groups: the
// starts of the waves' lists (kAce3Waves + 1 ints), then rounds of
// groups + 1 ints: kind | first n3 << 8, and per lane group its pair
// n1 | n2 << 2 | place of its first value << 4 | that value's output column << 8
// (place 15: no pair).  Kind l1 (kAceMaxL + 1) + l2, l1 <= l2, is rank 3 of pairs
// (n1 l1), (n2 l2): a value's place counts (n3, l3) from n3 = 0, and the pair's
// values are those from its later key on.  kAceRank2 + l is rank 2, kAceRank1 rank 1.
constexpr int kAceRank2 = (kAceMaxL + 1) * (kAceMaxL + 1), kAceRank1 = kAceRank2 + kAceMaxL + 1;
constexpr int kAce3Waves = 8;
constexpr int kAceRowPoints = 16;               // points per block, point-major
constexpr int kAceMaxPairCols = 3 * kAceMaxN;    // three l3 at most couple with (l1, l2)
void build_ace_plan(int nmax, int lmax, int groups, std::vector<int>& plan);
// rank 4: descriptor set (p1, p2, p3, p4, L per entry) and its evaluation tables
constexpr int kAce4MaxN = 3;
constexpr int kAce4MaxL = 3;
constexpr size_t kAce4LdsBudget = 96 * 1024;     // dynamic LDS of the pair vectors of one L
constexpr int kAce4MaxDescsL = 1024;              // descriptors of one phase (364 for L = 2 at nmax4 = lmax4 = 3)
// Point-major rank 4: the plan of k_ace4_rows.  kAce4RowWaves + 1 starts of the
// waves' lists of pair rounds; 8 bounds of the descriptors of L = 0..6; the rounds
// (kind l1 (kAce4MaxL + 1) + l2, l1 <= l2, then kAce4PairInts per lane group:
// n1 | n2 << 2, and the slots of L = l2 - l1.., three of ten bits to a word); the
// descriptors by L and first pair: slot | slot << 10 | column << 20, sign bit.
// Slots count float2 vectors of the block's points; a pair and L it does not need
// has the spare slots at the end.  n_slots, spare ones included.
constexpr int kAce4RowPoints = 8, kAce4RowWaves = 8;
constexpr int kAce4PairInts = 4;
constexpr int kAce4ARows = kAce4MaxN * 15;       // of A, those of n < kAce4MaxN
constexpr size_t kAce4RowsLds = 160 * 1024;
inline size_t ace4_rows_lds(size_t plan_ints, size_t n_slots, size_t n4) {
    return sizeof(float2) * kAce4RowPoints * (kAce4ARows + n_slots) + sizeof(float) * (kAce4RowPoints * n4 + 64) +
           sizeof(int) * plan_ints;
}
void build_ace4_rows_plan(int nmax4, int lmax4, std::vector<int>& plan, int& n_slots);
int ace4_descriptor_set(int nmax4, int lmax4, std::vector<int>& desc);
// The evaluation runs in phases, each one or more couplings L whose pair
// slots fit the LDS budget together: l_units / l_descs are offsets per
// phase; a descriptor entry is (first pair slot | L << 16, second pair slot,
// output, factor bits), slots counted within the phase.
int build_ace4_tables(int nmax4, int lmax4, std::vector<int>& l_units, std::vector<int4>& units,
                      std::vector<float>& coef, std::vector<int>& l_descs, std::vector<int4>& descs,
                      int& max_slots);
// A of every point of a chunk (n < 4, l <= 4, m >= 0: 60 complex per point),
// laid out [tile][60][64 lanes], written by the projection kernel and read by
// the contraction kernels.
constexpr int kAceAPerPoint = kAceMaxN * 15;
hipError_t launch_ace_proj(hipStream_t s, const BinState& bins, const int N[3], double rcut, int64_t pt_begin,
                           int64_t n_pts, float2* Ag, int* err);
hipError_t launch_ace4(hipStream_t s, const float2* Ag, int lmax4, int n_phases, int64_t n_pts, const int* l_units,
                       const int4* units, const float* coef, const int* l_descs, const int4* descs, int max_slots,
                       int n4, float* out, int64_t ds);   // descriptor k of point p at out[p + k ds]
hipError_t launch_ace4_rows(hipStream_t s, const float2* Ag, int64_t n_pts, const int* plan, int plan_ints, int n_slots,
                            int n4, float* out);      // out[p n4 + k]
// point-major rows of n_desc (rows, plan for kTile / kAceRowPoints groups) or one
// plane of ds values per descriptor (plan for one group)
hipError_t launch_ace(hipStream_t s, const float2* Ag, int nmax, int lmax, int64_t n_pts, const int* plan,
                      int plan_ints, bool rows, int n_desc, float* out, int64_t ds);

}  // namespace mala
