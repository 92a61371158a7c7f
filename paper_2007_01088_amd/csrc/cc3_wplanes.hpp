// The segments (operand products) of the planes of the W build, shared by its FP64 / FP32
// wave-tile form (kern_triples.hip, where the planes are explained) and its LDS-tile
// form (kern_wlp.hip).
#pragma once
#include <stdint.h>

#include <initializer_list>

#include "cc3_internal.hpp"

namespace cc3 {

// The segments of a plane, in order: 6 bits each, the permutation of perm_pqr that names
// the term (bits 0-2), l sum (bit 3), amplitude operand on the columns instead of the
// rows (bit 4), operand rows one slab apart (bit 5: Gw for a d sum, t2N for an l sum).
constexpr uint64_t wseg(int pi, int lsum, int col, int strided) {
  return (uint64_t)(pi | lsum << 3 | col << 4 | strided << 5);
}
constexpr uint64_t wsegs(std::initializer_list<uint64_t> l) {
  uint64_t v = 0;
  int at = 0;
  for (uint64_t x : l) { v |= x << at; at += 6; }
  return v;
}
// perm_pqr: 0 ijk, 1 jik, 2 kji, 3 ikj, 4 jki, 5 kij
constexpr uint64_t kSegsA = wsegs({wseg(0, 0, 0, 0), wseg(3, 0, 0, 1), wseg(2, 0, 1, 0),
                                   wseg(5, 0, 1, 1), wseg(0, 1, 0, 0), wseg(2, 1, 1, 0),
                                   wseg(4, 1, 1, 1)});
constexpr uint64_t kSegsAij = wsegs({wseg(0, 0, 0, 0), wseg(3, 0, 0, 1), wseg(2, 0, 1, 0),
                                     wseg(0, 1, 0, 0), wseg(2, 1, 1, 0), wseg(4, 1, 1, 1)});
constexpr uint64_t kSegsAjk = wsegs({wseg(0, 0, 0, 0), wseg(2, 0, 1, 0), wseg(5, 0, 1, 1),
                                     wseg(0, 1, 0, 0), wseg(2, 1, 1, 0), wseg(1, 1, 0, 1)});
constexpr uint64_t kSegsB = wsegs({wseg(1, 0, 0, 0), wseg(4, 0, 0, 1), wseg(1, 1, 0, 0),
                                   wseg(5, 1, 1, 0), wseg(3, 1, 1, 1)});

// the two planes (0: PA, 1: PB) of a triple of this kind, and their number of d sums (the l
// sums follow them and are three)
__device__ inline uint64_t wplane_segs(int plane, int kind) {
  return plane ? kSegsB
         : kind == TRI_DISTINCT ? kSegsA
         : kind == TRI_IJ ? kSegsAij : kSegsAjk;
}
__device__ inline int wplane_dsums(int plane, int kind) {
  return plane ? 2 : kind == TRI_DISTINCT ? 4 : 3;
}

// Whether the pieces of this segment's operands are paired with those of the columns first:
// where the three planes below have the operand on the rows that this segment has on the
// columns (of a triple with i == j or j == k they hold a term jki or kij as the transpose of
// ikj or jik)
__device__ inline bool wseg_swap(int code, int kind) {
  const int cols = kind == TRI_DISTINCT ? 0x34 : 0x04;  // permutations with t2 on the columns
  return ((code >> 4) & 1) != ((cols >> (code & 7)) & 1);
}

// The three planes of the BF16x3 build, whose FP32 accumulator runs over the d sum and then
// the l sum of one term: two terms per plane at fixed b, a and c,
//   P0[b][a][c] = ijk + kji,  P1[a][b][c] = jik + kij,  P2[c][a][b] = ikj + jki,
// each term's d sum and l sum in turn.
constexpr uint64_t kSegs3[3] = {
    wsegs({wseg(0, 0, 0, 0), wseg(0, 1, 0, 0), wseg(2, 0, 1, 0), wseg(2, 1, 1, 0)}),
    wsegs({wseg(1, 0, 0, 0), wseg(1, 1, 0, 0), wseg(5, 0, 1, 0), wseg(5, 1, 1, 0)}),
    wsegs({wseg(3, 0, 0, 0), wseg(3, 1, 0, 0), wseg(4, 0, 1, 0), wseg(4, 1, 1, 0)})};

}  // namespace cc3
