// Host-side declarations of the transition-density loop (Algorithm 3): the
// kernel launchers of kern_density.hip and the loop itself.
#pragma once
#include <hip/hip_runtime.h>

#include <algorithm>

#include "cc3_internal.hpp"

namespace cc3 {

constexpr int D3_MAXB = 64;  // most triples of a batch (the reductions' lists)

// Doubles of the partial slabs of any launch: batches of up to maxt triples, Gram launches
// of npair pairs.
size_t d3_partial_doubles(int no, int nv, int maxt, int npair);

void launch_build_density_blocks(const CholeskyScratch& cs, double* Gw, double* Go, double* Jo,
                                 double* Go3, double* Gl, double* tmp, int no, int nv, int nJ,
                                 hipStream_t st);
// The contractions of a batch of nt triples (cubes tau and lc, one per triple, in order):
// D_cd; Y' (Y'[l][r][p][c] = Y^o[c][l][p][r]) and D_kc, all added to.  P: partial slabs.
void launch_d3_cd(const double* tau, const double* lc, const int* tri, int nt, double* P,
                  double* Dcd, int nv, hipStream_t st);
void launch_d3_vec(const double* tau, const double* lc, const int* tri, int nt, const double* t2,
                   const double* E, double* P, double* Y, double* Dkc, int no, int nv,
                   hipStream_t st);
// The Gram matrices of pairs pair0 .. pair0 + npair - 1 (pair i (i + 1) / 2 + j) into D_lk;
// resident: one cube per unordered triple in lexicographic order, all-equal ones
// included; otherwise (npair = 1) the no cubes (i, j, k) of the pair.
void launch_d3_gram(const double* tau, const double* lc, bool resident, int pair0, int npair,
                    double* P, double* Dlk, int no, int nv, hipStream_t st);
void launch_d3_ld(const double* Y, const double* t2, double* P, double* Dld, int no, int nv,
                  hipStream_t st);
void launch_d3_yout(const double* Y, double* Yo, int no, int nv, bool accumulate, hipStream_t st);
// l2M[r][y][x][l] = -l2[l][r][x][y] (the W build's operand) and E (see kern_density.hip)
void launch_d3_l2(const double* l2, double* l2M, double* E, int no, int nv, hipStream_t st);

}  // namespace cc3
