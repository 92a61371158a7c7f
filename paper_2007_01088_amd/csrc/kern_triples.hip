// The triple loop of Algorithm 1 (CC3 ground-state equations) on gfx950.
//
// For a batch of unordered occupied triples i >= j >= k (not all equal):
//
//  k_wbuild  (FP64 MFMA)  the six terms B_pqr[x,y,z] = sum_d t2[p][q][x][d] g_{ydzr}
//            - sum_l t2[p][l][x][y] g_{lqzr} of the permutation operator, summed into
//            two planes so that X = P B = PA[b][a][c] + PB[a][b][c] (see there).
//            With two equal occupied indices three of the six terms repeat: PB is not
//            built and PA appears twice in X.
//  k_mix     (LDS)  per S3-orbit of 8x8x8 virtual blocks: X, the denominator
//            division tau = -X / eps^{abc}_{ijk}, and the contravariant
//            tau~ = 4 tau^{abc} - 2 tau^{acb} - 2 tau^{cba} - 2 tau^{bac} + tau^{bca} + tau^{cab},
//            written as tau~[a][b][c] (and, for the Jacobian preparation, its transpose
//            tau~T[a][c][b]).
//  k_omega   (FP64 MFMA)  for each distinct occupied permutation (p,q,r), with
//            U = tau~_{pqr} a view of tau~, one long-K GEMM over K = (b, c):
//              Ot2[p][q][a][d] += sum_bc U[a,b,c] g_{dbrc}    (columns d < nv)
//              Ot1[p][a]       += sum_bc U[a,b,c] g_{qbrc}    (column nv)
//            split over K into per-(triple, permutation, chunk) partial slabs;
//  k_reduce  adds the slabs into Ot1/Ot2 in a fixed order (deterministic, no atomics);
//  k_omega_oo (FP64 MFMA, output-stationary)  the oo and Fock terms
//              Ot2[p][l][a][b] += sum_c U[a,b,c] (delta_lq F_rc - g_{qlrc}),
//            four of the six permutations kept transposed, OtT[p][l][b][a], so that
//            their stores run along a.
#include <algorithm>

#include "cc3.h"
#include "cc3_device.hpp"
#include "cc3_internal.hpp"
#include "cc3_wplanes.hpp"

namespace cc3 {

static inline unsigned nblk(int64_t n, int b) { return (unsigned)((n + b - 1) / b); }

enum { SLOT_PA = SLOT_P0, SLOT_PB = SLOT_P1 };

// ---------------------------------------------------------------------------
// W build
// ---------------------------------------------------------------------------
// Every term is a product of an amplitude operand and an integral operand, both rows of
// contiguous k.  The d sum of B_pqr[x,y,z] multiplies t2[p][q] (rows x) by Gw[r] (rows
// (y, z)): it is a matrix product in x and z at fixed y, and, with the Gw rows taken one
// slab apart, in x and y at fixed z.  The l sum multiplies t2N[p] (rows (y, x)) by
// Go[q][r] (rows z): a product in x and z at fixed y, and in y and z at fixed x.  So the
// terms of two planes suffice, PA at fixed b and PB at fixed a (ijk: B_ijk[a,b,c], ikj:
// B_ikj[a,c,b], ... as in the permutation operator):
//   PA[b][a][c] = d sums of ijk, ikj, kji, kij + l sums of ijk, kji, jki,
//   PB[a][b][c] = d sums of jik, jki           + l sums of jik, kij, ikj,
// and X = PA[b][a][c] + PB[a][b][c].  With i == j the terms pair up under a <-> b, with
// j == k under b <-> c, and one of each pair is enough:
//   i == j: PA = d sums of ijk, ikj, kji + l sums of ijk, kji, jki; X = PA[b][a][c] + PA[a][b][c]
//   j == k: PA = d sums of ijk, kji, kij + l sums of ijk, kji, jik; X = PA[b][a][c] + PA[c][a][b].
// Two planes instead of one per value of the fixed index of each pair of terms (three):
// a third less written here and read by the mix, and up to 4 nv + 3 no of K per plane.
//
// One wavefront per FM x FN blocks of 16 x 16 outputs of a plane, without LDS and
// without barriers: it loads its own MFMA fragments, 8 k at a time (lane: two
// consecutive k of one row), two such units in flight.  FP64 MFMA takes 64 cycles per
// block and 4 k, so at 4 x 4 blocks a wavefront loads 16 B per cycle and CU, which L1 and
// L2 sustain; what a shared 128 x 128 LDS tile saves in loads it lost to barriers and,
// unless nv fills whole tiles, to padding.  Measured in isolation, 8 distinct triples,
// no = 10 (LDS tile -> this): nv = 93 1.30 -> 0.73 ms (4x the triples), 150 5.33 -> 2.6
// (2x), 250 7.35 -> 6.9, 400 65.8 -> 40.1 ms (70 TFLOP/s of MFMA, 89% of peak).
//
// MODE 0: the t3 terms (t2, t2N, Gw, Go as named).  MODE 1: the L3 terms of
// Algorithm 3, C_pqr[x,y,z] = sum_d L^{xd}_{qr} g_{pydz} - sum_l L^{xy}_{lr} g_{plqz}
// (+ outer products added by the density mix), with t2 <- l2, t2N <- l2M
// (l2M[r][y][x][l] = -l2[l][r][x][y]), Gw <- Gl (Gl[p][y][z][d] = g_{pydz}) and
// Go <- Go3 (Go3[p][q][z][l] = g_{plqz}): the same products with the roles of the
// occupied indices permuted.

// Operand element types.  double: the arrays themselves, K = nv and no, the k past K of a
// segment's last unit zeroed in registers.  float (CC3_FP32): FP32 copies whose rows are
// padded with zeros to a multiple of 32 k; every 32 k are summed on the MFMA in FP32 from
// zero and added into FP64 accumulators.  A unit of loads is 64 bytes of each row: lane
// group kq = lane / 16 holds the KL consecutive k from KL kq on, and feeds its t-th to
// MFMA step t.
template <class E>
struct WElem;
template <>
struct WElem<double> {
  static constexpr int KL = 2, UK = 8;
  typedef d2v Frag;
  typedef d4v Acc;
  static __device__ Acc mfma(double a, double b, Acc c) {
    return __builtin_amdgcn_mfma_f64_16x16x4f64(a, b, c, 0, 0, 0);
  }
  static __device__ int row(int kq, int r) { return kq + 4 * r; }
};
template <>
struct WElem<float> {
  static constexpr int KL = 4, UK = 16;
  typedef float Frag __attribute__((ext_vector_type(4)));
  typedef float Acc __attribute__((ext_vector_type(4)));
  static __device__ Acc mfma(float a, float b, Acc c) {
    return __builtin_amdgcn_mfma_f32_16x16x4f32(a, b, c, 0, 0, 0);
  }
  static __device__ int row(int kq, int r) { return 4 * kq + r; }
};
// strides of the operands, in elements: rows of K = nv and K = no (rv, ro), their K
// (padded for float), slabs of Gw and of t2N
struct WDims {
  int rv, ro, kv, ko;
  int64_t gy, ty;
};
template <class E>
__host__ __device__ inline WDims wdims(int no, int nv) {
  WDims d;
  if (sizeof(E) == 8) {
    d.rv = d.kv = nv;
    d.ro = d.ko = no;
    d.gy = gw_pitch(nv);
    d.ty = t2n_pitch(no, nv);
  } else {
    d.rv = d.kv = (int)kpad32(nv);
    d.ro = d.ko = (int)kpad32(no);
    d.gy = lp_slab(nv, nv, 4);
    d.ty = lp_slab(nv, no, 4);
  }
  return d;
}

// `item`: the wave tile, tiles of a plane fastest, then the fixed index y, plane, triple
template <class E, int MODE, int FM, int FN>
__device__ __forceinline__ void wbuild_body(const E* __restrict__ t2, const E* __restrict__ t2N,
                                            const E* __restrict__ Gw, const E* __restrict__ Go,
                                            const int* __restrict__ tri, int ntri,
                                            double* __restrict__ cubes, int64_t zs, int64_t ss,
                                            int pitch, int no, int nv, int tiles_m, int tiles_n,
                                            int all_terms, unsigned item) {
  typedef WElem<E> T;
  constexpr int KL = T::KL, UK = T::UK;
  constexpr bool F64 = sizeof(E) == 8;
  const unsigned tpp = (unsigned)(tiles_m * tiles_n);
  const int tile = (int)(item % tpp);
  item /= tpp;
  const int y = (int)(item % (unsigned)nv);
  item /= (unsigned)nv;
  const int plane = (int)(item & 1u), z = (int)(item >> 1);
  if (z >= ntri) return;
  const int i = tri[3 * z], j = tri[3 * z + 1], k = tri[3 * z + 2];
  const int kind = all_terms ? TRI_DISTINCT : tri_kind(i, j, k);
  if (kind != TRI_DISTINCT && plane == 1) return;
  const uint64_t segs = wplane_segs(plane, kind);
  const int nd = wplane_dsums(plane, kind), nseg = nd + 3;  // the l sums are three
  const WDims D = wdims<E>(no, nv);
  const int units = nd * ((D.kv + UK - 1) / UK) + 3 * ((D.ko + UK - 1) / UK);
  const int m0 = (tile / tiles_n) * (FM * 16), n0 = (tile % tiles_n) * (FN * 16);
  const int lane = threadIdx.x & 63, r16 = lane & 15, kq = lane >> 4;
  const int64_t xm = (int64_t)nv * D.rv, hm = (int64_t)nv * D.ro;  // one matrix of t2, of Go

  // the segment being loaded: resources at row m0 / n0, row strides, K, and the next k
  BufRsrc ra, rb;
  int seg = 0, lda, ldb, K, kk;
  unsigned va, vb;
  auto open = [&](int s) {
    const int code = (int)(segs >> (6 * s)) & 63;
    const bool lsum = code & 8, col = code & 16, strided = code & 32;
    int p, q, r;
    perm_pqr(code & 7, i, j, k, p, q, r);
    const int am0 = col ? n0 : m0, in0 = col ? m0 : n0;  // first rows of the two operands
    const E *amp, *in;
    int64_t an, inn;  // elements left in their arrays
    int la, li;
    if (!lsum) {
      la = D.rv;
      const int64_t ao = (MODE ? q * no + r : p * no + q) * xm + (int64_t)am0 * la;
      amp = t2 + ao;
      an = no * no * xm - ao;
      li = strided ? (int)D.gy : D.rv;
      const int64_t go = (MODE ? p : r) * nv * D.gy + (strided ? (int64_t)y * D.rv : y * D.gy) +
                         (int64_t)in0 * li;
      in = Gw + go;
      inn = no * nv * D.gy - go;
      K = D.kv;
    } else {
      la = strided ? (int)D.ty : D.ro;
      const int64_t ao = (MODE ? r : p) * nv * D.ty + (strided ? (int64_t)y * D.ro : y * D.ty) +
                         (int64_t)am0 * la;
      amp = t2N + ao;
      an = no * nv * D.ty - ao;
      li = D.ro;
      const int64_t go = (MODE ? p * no + q : q * no + r) * hm + (int64_t)in0 * li;
      in = Go + go;
      inn = no * no * hm - go;
      K = D.ko;
    }
    ra = buf_rsrc_n(col ? in : amp, col ? inn : an);
    rb = buf_rsrc_n(col ? amp : in, col ? an : inn);
    lda = (col ? li : la) * (int)sizeof(E);
    ldb = (col ? la : li) * (int)sizeof(E);
    va = (unsigned)(r16 * lda + kq * 16);
    vb = (unsigned)(r16 * ldb + kq * 16);
    kk = 0;
  };
  typename T::Frag a[2][FM], b[2][FN];
  int kn[2];  // k left in the segment at each unit (uniform); below UK the unit is partial
  auto fetch = [&](typename T::Frag (&fa)[FM], typename T::Frag (&fb)[FN], int& n) {
#pragma unroll
    for (int f = 0; f < FM; ++f) fa[f] = buf_load_16<typename T::Frag>(ra, va, (unsigned)(f * 16 * lda));
#pragma unroll
    for (int f = 0; f < FN; ++f) fb[f] = buf_load_16<typename T::Frag>(rb, vb, (unsigned)(f * 16 * ldb));
    n = K - kk;
    kk += UK;
    va += 64u;
    vb += 64u;
    // past the last segment the loads go on along its rows and are not used
    if (kk >= K && seg + 1 < nseg) open(++seg);
  };
  typename T::Acc acc[FM][FN];
  d4v accd[FM][FN];  // float: the 32-k stages summed in FP64
#pragma unroll
  for (int fm = 0; fm < FM; ++fm)
#pragma unroll
    for (int fn = 0; fn < FN; ++fn) {
      acc[fm][fn] = typename T::Acc{0, 0, 0, 0};
      accd[fm][fn] = d4v{0.0, 0.0, 0.0, 0.0};
    }
  open(0);
  fetch(a[0], b[0], kn[0]);
  fetch(a[1], b[1], kn[1]);
  for (int u = 0; u < units; u += 2) {
#pragma unroll
    for (int d = 0; d < 2; ++d) {
      if (u + d < units) {
        if constexpr (F64) {
          if (kn[d] < 8) {  // zero the k past K in both operands
            const bool i0 = 2 * kq < kn[d], i1 = 2 * kq + 1 < kn[d];
#pragma unroll
            for (int f = 0; f < FM; ++f) a[d][f] = d2v{i0 ? a[d][f][0] : 0.0, i1 ? a[d][f][1] : 0.0};
#pragma unroll
            for (int f = 0; f < FN; ++f) b[d][f] = d2v{i0 ? b[d][f][0] : 0.0, i1 ? b[d][f][1] : 0.0};
          }
        }
        // lane supplies A[m = l%16][k] and B[k][n = l%16], k = KL (l/16) + t of the unit
#pragma unroll
        for (int t = 0; t < KL; ++t)
#pragma unroll
          for (int fm = 0; fm < FM; ++fm)
#pragma unroll
            for (int fn = 0; fn < FN; ++fn)
              acc[fm][fn] = T::mfma(a[d][fm][t], b[d][fn][t], acc[fm][fn]);
      }
      fetch(a[d], b[d], kn[d]);
    }
    if constexpr (!F64) {  // both units of a 32-k stage (units are even in every segment)
#pragma unroll
      for (int fm = 0; fm < FM; ++fm)
#pragma unroll
        for (int fn = 0; fn < FN; ++fn) {
#pragma unroll
          for (int r = 0; r < 4; ++r) accd[fm][fn][r] += (double)acc[fm][fn][r];
          acc[fm][fn] = typename T::Acc{0, 0, 0, 0};
        }
    }
  }

  double* out = cubes + (int64_t)z * zs + (int64_t)plane * ss + (int64_t)y * nv * pitch;
#pragma unroll
  for (int fm = 0; fm < FM; ++fm)
#pragma unroll
    for (int fn = 0; fn < FN; ++fn)
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        const int m = m0 + fm * 16 + T::row(kq, r), n = n0 + fn * 16 + r16;
        if (m < nv && n < nv)
          out[(int64_t)m * pitch + n] = F64 ? (double)acc[fm][fn][r] : accd[fm][fn][r];
      }
}

// The shape with the least MFMA work, padding included, weighted by the loads per MFMA:
// relative time per block measured at nv = 150 to 400 about 1 + 0.7 (1/FM + 1/FN - 1/2)
// (3 x 3 1.04 to 1.2, 5 x 2 1.16 to 1.26, 4 x 3 1.0 to 1.09, 5 x 4 0.98 to 1.05 of 4 x 4).
// The item loop of the packed kernels takes registers that 5 x 4 and 5 x 2 do not leave.
static double shape_cost(int s, int64_t M, int64_t N) {
  const double fm = kShapes[s].fm, fn = kShapes[s].fn;
  int tm, tn;
  shape_tiles(s, M, N, &tm, &tn);
  return tm * fm * tn * fn * (0.65 + 0.7 * (1.0 / fm + 1.0 / fn));
}
int pick_shape(int64_t M, int64_t N, bool packed, int most) {
  int best = 0;
  double cost = 0.0;
  for (int s = 0; s < NSHAPE; ++s) {
    const int blocks = kShapes[s].fm * kShapes[s].fn;
    if (blocks > most || (packed && (blocks == 20 || blocks == 10))) continue;
    const double c = shape_cost(s, M, N);
    if (cost == 0.0 || c < cost) { best = s; cost = c; }
  }
  return best;
}

void shape_tiles(int shape, int64_t M, int64_t N, int* tm, int* tn) {
  *tm = (int)((M + 16 * kShapes[shape].fm - 1) / (16 * kShapes[shape].fm));
  *tn = (int)((N + 16 * kShapes[shape].fn - 1) / (16 * kShapes[shape].fn));
}

// Wavefronts per SIMD of the FP32 form: 12 accumulator registers per block and lane
// instead of 8.
template <class E>
constexpr int wbuild_waves(int fm, int fn) {
  return sizeof(E) == 8 ? shape_waves(fm, fn) : fm * fn <= 4 ? 4 : fm * fn <= 6 ? 3 : 2;
}

template <class E, int MODE, int FM, int FN>
__global__ __launch_bounds__(WNT, wbuild_waves<E>(FM, FN)) void k_wbuild(
    const E* __restrict__ t2, const E* __restrict__ t2N, const E* __restrict__ Gw,
    const E* __restrict__ Go, const int* __restrict__ tri, int ntri, double* __restrict__ cubes,
    int64_t zs, int64_t ss, int pitch, int no, int nv, int tiles_m, int tiles_n, int all_terms) {
  // runs of four planes per XCD: the tiles of a plane share its operand rows in one L2
  // (the 3 x 3 shape at nv = 250: 49 -> 57 TFLOP/s of MFMA)
  const unsigned wg = xcd_item(blockIdx.x, gridDim.x, (unsigned)(tiles_m * tiles_n));
  const unsigned wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  wbuild_body<E, MODE, FM, FN>(t2, t2N, Gw, Go, tri, ntri, cubes, zs, ss, pitch, no, nv, tiles_m,
                               tiles_n, all_terms, wg * 4 + wave);
}

// wave tiles of a W launch: tiles per plane x nv x two planes x triples, four to a workgroup
static unsigned wbuild_wgs(int nv, int ntri, int shape) {
  int tm, tn;
  shape_tiles(shape, nv, nv, &tm, &tn);
  return (unsigned)(((int64_t)tm * tn * nv * 2 * ntri + 3) / 4);
}

// FP32 runs on wave tiles where the 128 x 128 LDS tiles of kern_wlp.hip would be less than
// 85% outputs: the FP64 sums of its stages leave a wavefront 4 x 3 blocks at most, and where
// the LDS tiles are filled they load less.  MEASURED, whole calls, wave tiles / LDS tiles:
// nv = 93: 3.31 / 3.84 ms, 140: 17.0 / 20.2, 180: 37.8 / 40.7, 400: 172 / 182 (fill 51 to
// 61%); 120: 9.91 / 9.63, 250: 469 / 447 (88 and 95%).
bool fp32_wave_tiles(int nv) {
  const double f = nv / (128.0 * ((nv + 127) / 128));
  return f * f < 0.85;
}

// The FP32 form takes the shapes up to 4 x 3 (its accumulators: 144 registers).
static int wbuild_shape(int prec, int nv, bool packed) {
  return pick_shape(nv, nv, packed, prec == CC3_FP32 ? 12 : 20);
}

void launch_wbuild_ex(int mode, const double* X, const double* XN, const double* G, const double* H,
                      const int* tri, int ntri, double* cubes, int64_t zs, int64_t ss, int pitch,
                      int no, int nv, bool all_terms, hipStream_t st) {
  if (ntri <= 0) return;
  const int shape = wbuild_shape(CC3_FP64, nv, false);
  int tm, tn;
  shape_tiles(shape, nv, nv, &tm, &tn);
  const dim3 grid(wbuild_wgs(nv, ntri, shape)), block(WNT);
  with_shape(shape, [&](auto fm, auto fn) {
    constexpr int FM = decltype(fm)::value, FN = decltype(fn)::value;
    if (mode == 0)
      hipLaunchKernelGGL((k_wbuild<double, 0, FM, FN>), grid, block, 0, st, X, XN, G, H, tri, ntri,
                         cubes, zs, ss, pitch, no, nv, tm, tn, all_terms ? 1 : 0);
    else
      hipLaunchKernelGGL((k_wbuild<double, 1, FM, FN>), grid, block, 0, st, X, XN, G, H, tri, ntri,
                         cubes, zs, ss, pitch, no, nv, tm, tn, all_terms ? 1 : 0);
  });
}

void launch_wbuild(const double* t2, const double* t2N, const Blocks& b, const int* tri, int ntri,
                   double* cubes, int no, int nv, bool all_terms, hipStream_t st) {
  const int64_t cs = cube_slot(nv);
  launch_wbuild_ex(0, t2, t2N, b.Gw, b.Go, tri, ntri, cubes, NSLOT * cs, cs, cube_pitch(nv), no,
                   nv, all_terms, st);
}

void launch_wbuild_f32(const LpOperands& lp, const int* tri, int ntri, double* cubes, int no, int nv,
                       bool all_terms, hipStream_t st) {
  if (ntri <= 0) return;
  const int shape = wbuild_shape(CC3_FP32, nv, false);
  const int64_t cs = cube_slot(nv);
  int tm, tn;
  shape_tiles(shape, nv, nv, &tm, &tn);
  with_shape(shape, [&](auto fm, auto fn) {
    constexpr int FM = decltype(fm)::value, FN = decltype(fn)::value;
    if constexpr (FM * FN <= 12)
      hipLaunchKernelGGL((k_wbuild<float, 0, FM, FN>), dim3(wbuild_wgs(nv, ntri, shape)), dim3(WNT),
                         0, st, (const float*)lp.t2, (const float*)lp.t2N, (const float*)lp.GwT,
                         (const float*)lp.GoT, tri, ntri, cubes, NSLOT * cs, cs, cube_pitch(nv), no,
                         nv, tm, tn, all_terms ? 1 : 0);
  });
}

// ---------------------------------------------------------------------------
// Mix: X, tau, tau~ on the S3 orbit of an 8x8x8 block triple (A <= B <= C).
// ---------------------------------------------------------------------------
#define MT 8
#define MT3 (MT * MT * MT)
// padded LDS position of tile element (u, v, w): strides 73 and 9 keep every
// permuted access pattern of the orbit conflict-free across 8 lanes
#define TP(u, v, w) ((u) * 73 + (v) * 9 + (w))
#define TSZ 584

// the six orientations of a block triple, as positions into (A, B, C)
__host__ __device__ inline void orient(int o, int& p0, int& p1, int& p2) {
  switch (o) {
    case 0: p0 = 0; p1 = 1; p2 = 2; break;
    case 1: p0 = 0; p1 = 2; p2 = 1; break;
    case 2: p0 = 1; p1 = 0; p2 = 2; break;
    case 3: p0 = 1; p1 = 2; p2 = 0; break;
    case 4: p0 = 2; p1 = 0; p2 = 1; break;
    default: p0 = 2; p1 = 1; p2 = 0; break;
  }
}

__device__ inline int orient_of(int p0, int p1) {
  // the orientation index whose first two positions are (p0, p1)
  return p0 == 0 ? (p1 == 1 ? 0 : 1) : (p0 == 1 ? (p1 == 0 ? 2 : 3) : (p1 == 0 ? 4 : 5));
}

__device__ inline void decode_block_triple(int idx, int& A, int& B, int& C) {
  // lexicographic (C, B, A) with A <= B <= C
  int c = 0;
  while ((c + 1) * (c + 2) * (c + 3) / 6 <= idx) ++c;
  idx -= c * (c + 1) * (c + 2) / 6;
  int b = 0;
  while ((b + 1) * (b + 2) / 2 <= idx) ++b;
  idx -= b * (b + 1) / 2;
  A = idx; B = b; C = c;
}

// X of a triple whose six terms were all built (kind TRI_DISTINCT)
template <bool TWO>
__device__ inline double xval(const double* __restrict__ cz, int64_t nv, int a, int b, int c) {
  const int64_t rp = cube_pitch((int)nv), pl = nv * rp, cs = cube_slot((int)nv);
  const double* P0 = cz + SLOT_P0 * cs;
  const double* P1 = cz + SLOT_P1 * cs;
  double x = P0[b * pl + a * rp + c] + P1[a * pl + b * rp + c];
  if (!TWO) x += cz[SLOT_P2 * cs + c * pl + a * rp + b];
  return x;
}

// The split-BF16 copies of one orientation tile of tau~ (block A, B, C; values in T): form
// 0 or 1 of yl_piece, P pieces, each a run of 1 KB, 16 bytes per lane.
template <int P>
__device__ __forceinline__ void yl_put(char* Y, int form, const double* T, int A, int B, int C,
                                       int nv, int lane) {
  const int x0 = lane >> 3, x1 = lane & 7;
  const int64_t nb = (nv + 7) / 8;
  uint32_t w[P][4];
#pragma unroll
  for (int h = 0; h < 4; ++h) {
    uint16_t p0[P], p1[P];
    split_bf16<P>(form ? T[TP(x0, 2 * h, x1)] : T[TP(x0, x1, 2 * h)], p0);
    split_bf16<P>(form ? T[TP(x0, 2 * h + 1, x1)] : T[TP(x0, x1, 2 * h + 1)], p1);
#pragma unroll
    for (int pc = 0; pc < P; ++pc) w[pc][h] = p0[pc] | (uint32_t)p1[pc] << 16;
  }
  char* at = Y + form * P * yl_piece(nv) + ((A * nb + (form ? C : B)) * nb + (form ? B : C)) * 1024 +
             lane * 16;
#pragma unroll
  for (int pc = 0; pc < P; ++pc)
    *(uint4*)(at + pc * yl_piece(nv)) = make_uint4(w[pc][0], w[pc][1], w[pc][2], w[pc][3]);
}

// Mixed-all copies: cubesF (nullable), FP32 tau~ and tau~T, [triple][2][nv^3]; LP: YL, the
// split-BF16 blocks of the split-BF16 Omega GEMM (yl_piece), in lpP pieces.  TWO: the two
// planes of the W build, X = PA[b][a][c] + PB[a][b][c] (for i == j PA[a][b][c], for j == k
// PA[c][a][b] in the place of PB); otherwise the three planes of the BF16x3 build,
// X = P0[b][a][c] + P1[a][b][c] + P2[c][a][b], where for i == j P1 = P0 and P2 is
// symmetrised over (a, b), and for j == k P2 = P0 and P1 is symmetrised over (b, c).
template <bool TWO, bool LP>
__device__ __forceinline__ void mix_body(const double* __restrict__ eps,
                                         const int* __restrict__ tri, double* __restrict__ cubes,
                                         float* __restrict__ cubesF, char* __restrict__ YL, int lpP,
                                         int transposed, int no, int nv, int bx, int by) {
  __shared__ double Xs[6 * TSZ];
  const int z = by, ob = bx;
  const int i = tri[3 * z], j = tri[3 * z + 1], k = tri[3 * z + 2];
  const int kind = tri_kind(i, j, k);
  const int64_t nvl = nv, nv3 = nvl * nvl * nvl;
  // the padded cube rows: pitch rp, plane pl, slot cs
  const int64_t rp = cube_pitch(nv), pl = nvl * rp, cs = cube_slot(nv);
  double* cz = cubes + (int64_t)z * NSLOT * cs;
  int blk[3];
  decode_block_triple(ob, blk[0], blk[1], blk[2]);
  // With equal blocks some orientations repeat an earlier one: canon[o] is the
  // first orientation with the same block triple.  Repeats are neither loaded,
  // combined nor written; reads of a repeated tile go to its first copy.
  int canon[6];
#pragma unroll
  for (int o = 0; o < 6; ++o) {
    int q0, q1, q2;
    orient(o, q0, q1, q2);
    canon[o] = o;
#pragma unroll
    for (int o2 = 4; o2 >= 0; --o2) {
      if (o2 >= o) continue;
      int r0, r1, r2;
      orient(o2, r0, r1, r2);
      if (blk[r0] == blk[q0] && blk[r1] == blk[q1] && blk[r2] == blk[q2]) canon[o] = o2;
    }
  }
  const double eijk = eps[i] + eps[j] + eps[k];
  const double* P0 = cz + SLOT_P0 * cs;
  const double* P1 = cz + SLOT_P1 * cs;
  const double* P2 = cz + SLOT_P2 * cs;
  const int t = threadIdx.x;
  // 1. X on the orbit.  Each orientation tile is summed in up to three passes
  //    whose thread mapping makes the contiguous index of the cubes read in
  //    that pass the fastest one (c, b, then a).
#pragma unroll
  for (int o = 0; o < 6; ++o) {
    if (canon[o] != o) continue;
    int q0, q1, q2;
    orient(o, q0, q1, q2);
    const int A0 = blk[q0] * MT, B0 = blk[q1] * MT, C0 = blk[q2] * MT;
    const int u = t >> 6, v = (t >> 3) & 7, w = t & 7;  // pass 0: c fastest
    const int a = A0 + u, b = B0 + v, c = C0 + w;
    double x = 0.0;
    if (a < nv && b < nv && c < nv)
      x = TWO && kind == TRI_JK
              ? P0[b * pl + a * rp + c]
              : P0[b * pl + a * rp + c] + (kind == TRI_IJ ? P0 : P1)[a * pl + b * rp + c];
    Xs[o * TSZ + TP(u, v, w)] = x;
  }
  if (!TWO || kind == TRI_JK) {
    __syncthreads();
#pragma unroll
    for (int o = 0; o < 6; ++o) {
      if (canon[o] != o) continue;
      int q0, q1, q2;
      orient(o, q0, q1, q2);
      const int A0 = blk[q0] * MT, B0 = blk[q1] * MT, C0 = blk[q2] * MT;
      const int u = t >> 6, w = (t >> 3) & 7, v = t & 7;  // pass 1: b fastest
      const int a = A0 + u, b = B0 + v, c = C0 + w;
      if (a < nv && b < nv && c < nv) {
        double x;
        if (TWO) x = P0[c * pl + a * rp + b];
        else if (kind == TRI_JK) x = P1[a * pl + c * rp + b] + P0[c * pl + a * rp + b];
        else x = P2[c * pl + a * rp + b];
        Xs[o * TSZ + TP(u, v, w)] += x;
      }
    }
  }
  if (!TWO && kind == TRI_IJ) {
    __syncthreads();
#pragma unroll
    for (int o = 0; o < 6; ++o) {
      if (canon[o] != o) continue;
      int q0, q1, q2;
      orient(o, q0, q1, q2);
      const int A0 = blk[q0] * MT, B0 = blk[q1] * MT, C0 = blk[q2] * MT;
      const int v = t >> 6, w = (t >> 3) & 7, u = t & 7;  // pass 2: a fastest
      const int a = A0 + u, b = B0 + v, c = C0 + w;
      if (a < nv && b < nv && c < nv) Xs[o * TSZ + TP(u, v, w)] += P2[c * pl + b * rp + a];
    }
  }
  __syncthreads();
  // 2. tau~ on the orbit, in registers
  double tt[6];
#pragma unroll
  for (int o = 0; o < 6; ++o) {
    if (canon[o] != o) continue;
    int q0, q1, q2;
    orient(o, q0, q1, q2);
    const int A0 = blk[q0] * MT, B0 = blk[q1] * MT, C0 = blk[q2] * MT;
    const int o_acb = canon[orient_of(q0, q2)], o_cba = canon[orient_of(q2, q1)];
    const int o_bac = canon[orient_of(q1, q0)], o_bca = canon[orient_of(q1, q2)];
    const int o_cab = canon[orient_of(q2, q0)];
    const int u = t >> 6, v = (t >> 3) & 7, w = t & 7;
    const int a = A0 + u, b = B0 + v, c = C0 + w;
    double val = 0.0;
    if (a < nv && b < nv && c < nv) {
      // X at permuted virtual labels: (a,c,b), (c,b,a), (b,a,c), (b,c,a), (c,a,b)
      const double x_abc = Xs[o * TSZ + TP(u, v, w)];
      const double x_acb = Xs[o_acb * TSZ + TP(u, w, v)];
      const double x_cba = Xs[o_cba * TSZ + TP(w, v, u)];
      const double x_bac = Xs[o_bac * TSZ + TP(v, u, w)];
      const double x_bca = Xs[o_bca * TSZ + TP(v, w, u)];
      const double x_cab = Xs[o_cab * TSZ + TP(w, u, v)];
      const double D = eps[no + a] + eps[no + b] + eps[no + c] - eijk;
      val = -(4.0 * x_abc - 2.0 * x_acb - 2.0 * x_cba - 2.0 * x_bac + x_bca + x_cab) / D;
    }
    tt[o] = val;
  }
  // 3. write tau~[a][b][c], with zeros in the padding columns c >= nv, and its FP32
  //    copy of the same order, straight from the registers
  double* TT = cz + SLOT_TT * cs;
#pragma unroll
  for (int o = 0; o < 6; ++o) {
    if (canon[o] != o) continue;
    int q0, q1, q2;
    orient(o, q0, q1, q2);
    const int A0 = blk[q0] * MT, B0 = blk[q1] * MT, C0 = blk[q2] * MT;
    const int u = t >> 6, v = (t >> 3) & 7, w = t & 7;
    const int a = A0 + u, b = B0 + v, c = C0 + w;
    if (a < nv && b < nv) {
      const double x = tt[o];
      TT[(a * nvl + b) * rp + c] = x;
      if (cubesF && c < nv) cubesF[(int64_t)z * 2 * nv3 + (a * nvl + b) * nvl + c] = (float)x;
    }
  }
  // 4. the copies with a and b, or c and b, exchanged: through LDS, b fastest
  if (!LP && !transposed && !cubesF) return;
  __syncthreads();
#pragma unroll
  for (int o = 0; o < 6; ++o) {
    if (canon[o] != o) continue;
    Xs[o * TSZ + TP(t >> 6, (t >> 3) & 7, t & 7)] = tt[o];
  }
  __syncthreads();
  if constexpr (LP) {  // two wavefronts per orientation, one form each
    int alive = 0;
#pragma unroll
    for (int o = 0; o < 6; ++o) alive |= (canon[o] == o) << o;
    const int wave = __builtin_amdgcn_readfirstlane(t >> 6);
    char* Y = YL + (int64_t)z * 2 * lpP * yl_piece(nv);
    for (int o = wave >> 1; o < 6; o += 4) {
      if (!(alive >> o & 1)) continue;
      int q0, q1, q2;
      orient(o, q0, q1, q2);
      const int A = q0 == 0 ? blk[0] : q0 == 1 ? blk[1] : blk[2];
      const int B = q1 == 0 ? blk[0] : q1 == 1 ? blk[1] : blk[2];
      const int C = q2 == 0 ? blk[0] : q2 == 1 ? blk[1] : blk[2];
      if (lpP == 2) yl_put<2>(Y, wave & 1, Xs + o * TSZ, A, B, C, nv, t & 63);
      else yl_put<3>(Y, wave & 1, Xs + o * TSZ, A, B, C, nv, t & 63);
    }
  }
  if (!transposed && !cubesF) return;
  double* TTT = cz + SLOT_TTT * cs;
#pragma unroll
  for (int o = 0; o < 6; ++o) {
    if (canon[o] != o) continue;
    int q0, q1, q2;
    orient(o, q0, q1, q2);
    const int A0 = blk[q0] * MT, B0 = blk[q1] * MT, C0 = blk[q2] * MT;
    const int u = t >> 6, w = (t >> 3) & 7, v = t & 7;
    const int a = A0 + u, b = B0 + v, c = C0 + w;
    if (a < nv && b < nv && c < nv) {
      const double x = Xs[o * TSZ + TP(u, v, w)];
      if (transposed) TTT[(a * nvl + c) * rp + b] = x;
      if (cubesF) cubesF[((int64_t)z * 2 + 1) * nv3 + (a * nvl + c) * nvl + b] = (float)x;
    }
  }
}

template <bool TWO, bool LP>
__global__ __launch_bounds__(512, LP ? 6 : 8) void k_mix(const double* __restrict__ eps,
                                             const int* __restrict__ tri,
                                             double* __restrict__ cubes, float* __restrict__ cubesF,
                                             char* __restrict__ YL, int lpP, int transposed, int no,
                                             int nv) {
  mix_body<TWO, LP>(eps, tri, cubes, cubesF, YL, lpP, transposed, no, nv, blockIdx.x, blockIdx.y);
}

void launch_mix(bool two_planes, const double* eps, const int* tri, int ntri, double* cubes,
                float* cubesF, void* YL, int lpP, bool transposed, int no, int nv, hipStream_t st) {
  const int nb = (nv + MT - 1) / MT;
  const int nbt = nb * (nb + 1) * (nb + 2) / 6;
  auto run = [&](auto* kernel) {
    hipLaunchKernelGGL(kernel, dim3(nbt, ntri), dim3(512), 0, st, eps, tri, cubes, cubesF, (char*)YL,
                       lpP, transposed ? 1 : 0, no, nv);
  };
  if (two_planes && YL) run(k_mix<true, true>);
  else if (two_planes) run(k_mix<true, false>);
  else if (YL) run(k_mix<false, true>);
  else run(k_mix<false, false>);
}

// ---------------------------------------------------------------------------
// Mix of the transition-density loop (Algorithm 3).  LMODE false: tau = -X/eps from the t3
// planes (PA, PB).  LMODE true: from the L3 planes plus the outer-product terms of the L3
// statement,
//   sum over the six simultaneous permutations (p,q,r; x,y,z) of (i,j,k; a,b,c) of
//   L^x_p g_{qyrz} + L^{xy}_{pq} F_{rz},
// L = X / (omega - eps) and its contravariant L~.  Same S3-orbit tiling of 8^3 virtual
// blocks as k_mix; outputs are written in [a][b][c] order straight from the orientation
// tiles.  The six terms are equal in pairs (g_{qyrz} = g_{rzqy}, L^{xy}_{pq} = L^{yx}_{qp}),
// so three of each are loaded and doubled: the loads of the outer products, and not the
// cubes, had set the time of this form (374 against 210 us per 12 triples at nv = 120).
// ---------------------------------------------------------------------------
__device__ inline double l3_outer(const double* __restrict__ l1, const double* __restrict__ l2,
                                  const double* __restrict__ Jo, const double* __restrict__ F,
                                  int no, int64_t nv, int i, int j, int k, int a, int b, int c) {
  auto term = [&](int p, int q, int r, int x, int y, int z) {  // p, x outside; (q, y), (r, z) inside
    const int64_t at = (((int64_t)q * no + r) * nv + y) * nv + z;
    return l1[p * nv + x] * Jo[at] + F[p * nv + x] * l2[at];
  };
  return 2.0 * (term(i, j, k, a, b, c) + term(j, i, k, b, a, c) + term(k, i, j, c, a, b));
}

template <bool LMODE>
__global__ __launch_bounds__(512) void k_mix3(const double* __restrict__ eps,
                                             const int* __restrict__ tri,
                                             const double* __restrict__ planesA,
                                             const double* __restrict__ planesB,
                                             double* __restrict__ cubes, double omega,
                                             const double* __restrict__ l1,
                                             const double* __restrict__ l2,
                                             const double* __restrict__ Jo,
                                             const double* __restrict__ F, int no, int nv) {
  __shared__ double Xs[6 * TSZ];
  const int z = blockIdx.y, ob = blockIdx.x;
  const int i = tri[3 * z], j = tri[3 * z + 1], k = tri[3 * z + 2];
  const int kind = tri_kind(i, j, k);
  const int64_t nvl = nv;
  // the padded cube rows: pitch rp, plane pl, cube cs
  const int64_t rp = cube_pitch(nv), pl = nvl * rp, cs = cube_slot(nv);
  const double* PA = planesA + (int64_t)z * cs;
  const double* PB = planesB + (int64_t)z * cs;
  int blk[3];
  decode_block_triple(ob, blk[0], blk[1], blk[2]);
  int canon[6];
#pragma unroll
  for (int o = 0; o < 6; ++o) {
    int q0, q1, q2;
    orient(o, q0, q1, q2);
    canon[o] = o;
#pragma unroll
    for (int o2 = 4; o2 >= 0; --o2) {
      if (o2 >= o) continue;
      int r0, r1, r2;
      orient(o2, r0, r1, r2);
      if (blk[r0] == blk[q0] && blk[r1] == blk[q1] && blk[r2] == blk[q2]) canon[o] = o2;
    }
  }
  const int t = threadIdx.x;
  const int u = t >> 6, v = (t >> 3) & 7, w = t & 7;
  // X on the orbit: the two-plane sum of k_mix (c, then b fastest), plus the outer
  // products in the L3 form
#pragma unroll
  for (int o = 0; o < 6; ++o) {
    if (canon[o] != o) continue;
    int q0, q1, q2;
    orient(o, q0, q1, q2);
    const int a = blk[q0] * MT + u, b = blk[q1] * MT + v, c = blk[q2] * MT + w;
    double x = 0.0;
    if (a < nv && b < nv && c < nv) {
      x = PA[b * pl + a * rp + c];
      if (kind != TRI_JK) x += (kind == TRI_IJ ? PA : PB)[a * pl + b * rp + c];
      if (LMODE) x += l3_outer(l1, l2, Jo, F, no, nvl, i, j, k, a, b, c);
    }
    Xs[o * TSZ + TP(u, v, w)] = x;
  }
  if (kind == TRI_JK) {
    __syncthreads();
#pragma unroll
    for (int o = 0; o < 6; ++o) {
      if (canon[o] != o) continue;
      int q0, q1, q2;
      orient(o, q0, q1, q2);
      const int uu = t >> 6, ww = (t >> 3) & 7, vv = t & 7;  // b fastest
      const int a = blk[q0] * MT + uu, b = blk[q1] * MT + vv, c = blk[q2] * MT + ww;
      if (a < nv && b < nv && c < nv)
        Xs[o * TSZ + TP(uu, vv, ww)] += PA[c * pl + a * rp + b];
    }
  }
  __syncthreads();
  // the denominators and the contravariant combination; outputs in [a][b][c] order,
  // with zeros in the padding columns c >= nv of each row (c < rp: the blocks cover
  // exactly rp values)
  const double eijk = eps[i] + eps[j] + eps[k];
  double* out = cubes + (int64_t)z * cs;
#pragma unroll
  for (int o = 0; o < 6; ++o) {
    if (canon[o] != o) continue;
    int q0, q1, q2;
    orient(o, q0, q1, q2);
    const int a = blk[q0] * MT + u, b = blk[q1] * MT + v, c = blk[q2] * MT + w;
    if (!(a < nv && b < nv)) continue;
    const int64_t e = (a * nvl + b) * rp + c;
    if (c >= nv) {
      out[e] = 0.0;
      continue;
    }
    const double x_abc = Xs[o * TSZ + TP(u, v, w)];
    const double D = eps[no + a] + eps[no + b] + eps[no + c] - eijk - (LMODE ? omega : 0.0);
    if (!LMODE) {
      out[e] = -x_abc / D;
      continue;
    }
    const int o_acb = canon[orient_of(q0, q2)], o_cba = canon[orient_of(q2, q1)];
    const int o_bac = canon[orient_of(q1, q0)], o_bca = canon[orient_of(q1, q2)];
    const int o_cab = canon[orient_of(q2, q0)];
    const double x_acb = Xs[o_acb * TSZ + TP(u, w, v)];
    const double x_cba = Xs[o_cba * TSZ + TP(w, v, u)];
    const double x_bac = Xs[o_bac * TSZ + TP(v, u, w)];
    const double x_bca = Xs[o_bca * TSZ + TP(v, w, u)];
    const double x_cab = Xs[o_cab * TSZ + TP(w, u, v)];
    out[e] = -(4.0 * x_abc - 2.0 * x_acb - 2.0 * x_cba - 2.0 * x_bac + x_bca + x_cab) / D;
  }
}

void launch_mix3(bool lmode, const double* eps, const int* tri, int ntri, const double* PA,
                 const double* PB, double* out, double omega, const double* l1, const double* l2,
                 const double* Jo, const double* F, int no, int nv, hipStream_t st) {
  if (ntri <= 0) return;
  const int nb = (nv + MT - 1) / MT;
  const int nbt = nb * (nb + 1) * (nb + 2) / 6;
  if (lmode)
    hipLaunchKernelGGL(k_mix3<true>, dim3(nbt, ntri), dim3(512), 0, st, eps, tri, PA, PB, out,
                       omega, l1, l2, Jo, F, no, nv);
  else
    hipLaunchKernelGGL(k_mix3<false>, dim3(nbt, ntri), dim3(512), 0, st, eps, tri, PA, PB, out, 0.0,
                       l1, l2, Jo, F, no, nv);
}

// tau^{abc}_{ijk} = -X / eps^{abc}_{ijk} for one ordered triple whose six terms were all built
template <bool TWO>
__global__ void k_tau_export(const double* __restrict__ eps, const int* __restrict__ tri,
                             const double* __restrict__ cubes, double* __restrict__ tau, int no,
                             int nv) {
  const int64_t nvl = nv, nv3 = nvl * nvl * nvl;
  const int64_t e = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (e >= nv3) return;
  const int a = (int)(e / (nvl * nvl)), b = (int)((e / nvl) % nvl), c = (int)(e % nvl);
  const int i = tri[0], j = tri[1], k = tri[2];
  const double X = xval<TWO>(cubes, nvl, a, b, c);
  tau[e] = -X / (eps[no + a] + eps[no + b] + eps[no + c] - eps[i] - eps[j] - eps[k]);
}

void launch_tau_export(bool two_planes, const double* eps, const int* tri, const double* cubes,
                       double* tau, int no, int nv, hipStream_t st) {
  const int64_t nv3 = (int64_t)nv * nv * nv;
  if (two_planes)
    hipLaunchKernelGGL(k_tau_export<true>, dim3(nblk(nv3, 256)), dim3(256), 0, st, eps, tri, cubes,
                       tau, no, nv);
  else
    hipLaunchKernelGGL(k_tau_export<false>, dim3(nblk(nv3, 256)), dim3(256), 0, st, eps, tri, cubes,
                       tau, no, nv);
}

// ---------------------------------------------------------------------------
// Omega contraction: the vv term and Omega1
// ---------------------------------------------------------------------------
// One (triple, permutation) GEMM over the flattened K = (b, c), K = nv^2:
//   columns n < nv : Ot2[p][q][a][n] += sum_bc U[a,b,c] g_{nbrc}
//   column  n = nv : Ot1[p][a]       += sum_bc U[a,b,c] g_{qbrc}
// Both column kinds are rows of one block G[r][n'][.][.] (n' < nv: g_{n'brc};
// n' = nv + l: g_{lbrc}), stored once with K in (b, c) order (Gbc) and once in
// (c, b) order (Gcb).  With the K order of each permutation chosen to match, the six
// views U_pi of tau~ are three operands of the one cube TT[x][y][z] = tau~[x][y][z]:
//   rows TT[a][x][y]: pi 0 = tau~[a][b][c] by Gbc, pi 3 = tau~[a][c][b] by Gcb
//   rows TT[x][a][y]: pi 1 = tau~[b][a][c] by Gbc, pi 4 = tau~[c][a][b] by Gcb
//   rows TT[x][y][a]: pi 5 = tau~[b][c][a] by Gbc, pi 2 = tau~[c][b][a] by Gcb
// with K = (x, y) and y contiguous in the first two, a in the third.  K runs over the
// padded rows of y (zeros in G, and in tau~ where it is read along y), so that every unit
// of 8 k has one x.  K is split into chunks of whole units; each chunk writes a partial
// slab Pvv[z][pi][chunk][a][n] (n <= nv) that k_reduce sums in a fixed order.
//
// Wave tiles as in the W build: no LDS, two units of 8 k in flight.  The waves of one
// (triple, operand, chunk, permutation) are neighbours on one XCD and share the rows of tau~ and
// of G in its L2; the operand's second permutation follows and finds part of tau~ there.  Bound
// by MFMA and by the loads' way through L1 and L2 (16 B per cycle and CU at 4 x 4 blocks).  Per
// launch, 128 x 128 LDS tiles -> this, before the order of items at omega_body: 23/250, 8 triples
// 6.14 -> 5.81 ms; 8/400, 8 triples 49.0 -> 36.2; 7/93 1.91 -> 1.07; 6/45 0.137 -> 0.032 ms.
// From nv = 448 on: omega_lds.
template <bool ROWS, int FM, int FN>
__device__ __forceinline__ void omega_tile(const double* __restrict__ U, int64_t un, unsigned va0,
                                           unsigned bs, unsigned us, int64_t xs, BufRsrc rb,
                                           unsigned vb, unsigned gs, unsigned dq, int u0, int u1,
                                           int ux, double* __restrict__ pvv, int m0, int n0,
                                           int nv) {
  const int lane = threadIdx.x & 63, r16 = lane & 15, kq = lane >> 4;
  // U, un: tau~ at the tile's first row and x = 0, and the doubles left in its slot.
  // Unit u is at x = u / ux, y = 8 (u % ux): the resource moves to each x (offsets over
  // all of K would not fit 32 bits), va by us bytes per unit within it; ks = us / 8 is
  // the byte step of one k where a is contiguous.
  const int x0 = u0 / ux;
  const double* pa = U + x0 * xs;
  int64_t na = un - x0 * xs;
  int yu = u0 - x0 * ux;
  BufRsrc ra = buf_rsrc_n(pa, na);
  unsigned va = va0 + (unsigned)yu * us;
  // B: row r16 of each block, gs bytes between the blocks; the lane of column nv reads dq
  // bytes further on (the Omega1 row)
  vb += (unsigned)u0 * 64u;
  const int fq = (nv - n0) >> 4;  // the block of column nv (outside [0, FN): another tile's)
  const unsigned dv = r16 == (nv & 15) ? dq : 0u;
  double a[2][FM][2];
  d2v b[2][FN];
  auto fetch = [&](double (&fa)[FM][2], d2v (&fb)[FN]) {
    frag_load<ROWS, FM>(ra, va, bs, us / 8u, fa);
#pragma unroll
    for (int f = 0; f < FN; ++f)
      fb[f] = buf_load_2f64(rb, f == fq ? vb + dv : vb, (unsigned)f * gs);
    vb += 64u;
    va += us;
    if (++yu == ux) {
      yu = 0;
      va = va0;
      pa += xs;
      na = na > xs ? na - xs : 0;
      ra = buf_rsrc_n(pa, na);
    }
  };
  d4v acc[FM][FN];
#pragma unroll
  for (int fm = 0; fm < FM; ++fm)
#pragma unroll
    for (int fn = 0; fn < FN; ++fn) acc[fm][fn] = d4v{0.0, 0.0, 0.0, 0.0};
  fetch(a[0], b[0]);
  fetch(a[1], b[1]);
  for (int u = u0; u < u1; u += 2) {
#pragma unroll
    for (int d = 0; d < 2; ++d) {
      if (u + d < u1) {
#pragma unroll
        for (int t = 0; t < 2; ++t)
#pragma unroll
          for (int fm = 0; fm < FM; ++fm)
#pragma unroll
            for (int fn = 0; fn < FN; ++fn)
              acc[fm][fn] = __builtin_amdgcn_mfma_f64_16x16x4f64(a[d][fm][t], b[d][fn][t],
                                                                 acc[fm][fn], 0, 0, 0);
      }
      fetch(a[d], b[d]);
    }
  }
  const int NV1 = nv + 1;
#pragma unroll
  for (int fm = 0; fm < FM; ++fm)
#pragma unroll
    for (int fn = 0; fn < FN; ++fn)
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        const int m = m0 + frag_row<ROWS, FM>(fm, kq, r), n = n0 + fn * 16 + r16;
        if (m < nv && n <= nv) pvv[(int64_t)m * NV1 + n] = acc[fm][fn][r];
      }
}

// `item`: the wave tile, column tiles fastest, then row tiles, the permutation of the operand's
// two, the K chunk, the operand and the triple.  One permutation after the other: with the two in
// turn per row tile, and only one of them distinct (two equal occupied indices), every other
// four wave tiles end at once and those that stay hold the rows of twice the groups in an L2.
// MEASURED, in turn / one after the other, FP64 launches of one triple with two equal indices
// and of 8 distinct or not: nv = 250 0.74 / 0.44 and 5.07 / 4.72 ms, 384 3.39 / 2.80 and 37.6 /
// 34.8, 432 4.95 / 4.29 and 56.7 / 55.7.
template <int FM, int FN>
__device__ __forceinline__ void omega_body(const double* __restrict__ cubes,
                                           const double* __restrict__ Gbc,
                                           const double* __restrict__ Gcb,
                                           const int* __restrict__ tri, int ntri,
                                           double* __restrict__ Pvv, int no, int nv, int nchunks,
                                           int tiles_m, int tiles_n, unsigned item) {
  const int tn = (int)(item % (unsigned)tiles_n);
  item /= (unsigned)tiles_n;
  const int tm = (int)(item % (unsigned)tiles_m);
  item /= (unsigned)tiles_m;
  const bool cb = item & 1u;  // the permutation that takes Gcb
  item >>= 1;
  const int ch = (int)(item % (unsigned)nchunks);
  item /= (unsigned)nchunks;
  const int op = (int)(item % 3u), z = (int)(item / 3u);
  if (z >= ntri) return;
  const int i = tri[3 * z], j = tri[3 * z + 1], k = tri[3 * z + 2];
  const int pi = op == 0 ? (cb ? 3 : 0) : op == 1 ? (cb ? 4 : 1) : (cb ? 2 : 5);
  if (!perm_active(tri_kind(i, j, k), pi)) return;
  int p, q, r;
  perm_pqr(pi, i, j, k, p, q, r);
  const int rp = cube_pitch(nv), ux = rp / 8, units = nv * ux;
  const int u0 = (int)((int64_t)ch * units / nchunks), u1 = (int)((int64_t)(ch + 1) * units / nchunks);
  const int m0 = tm * (FM * 16), n0 = tn * (FN * 16);
  const int lane = threadIdx.x & 63, r16 = lane & 15, kq = lane >> 4;
  const int64_t pl = (int64_t)nv * rp, css = cube_slot(nv), gp = g_pitch(nv);
  // B rows n < nv are rows n of G; the Omega1 column n = nv reads row nv + q (columns past
  // it read some row or zeros and are not stored)
  const int64_t go = ((int64_t)r * (nv + no) + n0) * gp;
  const BufRsrc rb = buf_rsrc_n((cb ? Gcb : Gbc) + go, (int64_t)no * (nv + no) * gp - go);
  const unsigned vb = (unsigned)(r16 * gp + 2 * kq) * 8u;
  const unsigned gs = (unsigned)(gp * 128), dq = (unsigned)(q * gp * 8);
  const double* TT = cubes + ((int64_t)z * NSLOT + SLOT_TT) * css;
  double* pvv = Pvv + (((int64_t)z * 6 + pi) * nchunks + ch) * nv * (int64_t)(nv + 1);
  if (op == 2) {
    omega_tile<false, FM, FN>(TT + m0, css - m0, (unsigned)(2 * kq * rp + 2 * r16) * 8u, 0u,
                              (unsigned)rp * 64u, pl, rb, vb, gs, dq, u0, u1, ux, pvv, m0, n0,
                              nv);
  } else {
    const int64_t rs = op == 0 ? pl : rp;  // row stride
    omega_tile<true, FM, FN>(TT + m0 * rs, css - m0 * rs, (unsigned)(r16 * rs + 2 * kq) * 8u,
                             (unsigned)(rs * 128), 64u, op == 0 ? rp : pl, rb, vb, gs, dq, u0, u1, ux,
                             pvv, m0, n0, nv);
  }
}

template <int FM, int FN>
__global__ __launch_bounds__(WNT, shape_waves(FM, FN)) void k_omega(
    const double* __restrict__ cubes, const double* __restrict__ Gbc,
    const double* __restrict__ Gcb, const int* __restrict__ tri, int ntri,
    double* __restrict__ Pvv, int no, int nv, int nchunks, int tiles_m, int tiles_n) {
  // one (triple, operand, chunk) per run and XCD: 2 tiles_m tiles_n wave tiles
  const unsigned wg = xcd_item(blockIdx.x, gridDim.x, (unsigned)(tiles_m * tiles_n + 1) / 2u);
  const unsigned wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  omega_body<FM, FN>(cubes, Gbc, Gcb, tri, ntri, Pvv, no, nv, nchunks, tiles_m, tiles_n,
                     wg * 4 + wave);
}

// The FP32 mixed-all form: the same products on FP32 MFMA over FP32 copies of tau~,
// tau~T (TTT[x][y][z] = tau~[x][z][y], which makes every view affine in K with the K order
// of G below) and of Gbc, Gcb, none of them padded; the products of each K chunk are
// summed in FP32 and the chunks in FP64 by k_reduce.
//   pi 0: tau~[a][b][c] = TT[a][(b,c)], pi 3: tau~[a][c][b] = TTT[a][(b,c)]  (k contiguous)
//   pi 1: tau~[b][a][c] = TTT[(b,c)][a], pi 5: tau~[b][c][a] = TT[(b,c)][a]  (a contiguous)
//   pi 2: tau~[c][b][a] = TT[(c,b)][a], pi 4: tau~[c][a][b] = TTT[(c,b)][a]  (K = (c, b))
// 128 x 128 tiles on 8 wavefronts of 32 x 64 through LDS, 16 k per stage.
typedef TileCfg<4, 2, 2, 4, 16> OCfg;
typedef float f4v_ __attribute__((ext_vector_type(4)));

// The FP64 form for large nv (omega_lds): the products of k_omega, with its views, K and
// slabs, on 128 x 128 tiles of 8 wavefronts through LDS, 16 k (two units of 8) per stage.
// From nv = 448 on the rows of both operands are 1.6 MB and more apart. A wave tile touches
// 64 bytes of each of 128 rows per unit, and what its neighbours share has left the caches by
// then; the LDS tile touches 128 bytes of each of 256 rows for four times the outputs.
// U: tau~ at the tile's first row; AMAJ: a contiguous (rs = 1), else y.  xs, ys, rs: doubles
// between x, y and rows.  Elements outside K or past y = nv load a valid element, and their
// zero is applied at the LDS store, so that the loads stay in flight over the current stage's
// MFMAs.  Rows past nv repeat row nv - 1 (their outputs are never stored).
template <bool AMAJ>
__device__ __forceinline__ void omega_lds_tile(const double* __restrict__ U,
                                               const double* __restrict__ G, int64_t xs, int ys,
                                               int64_t rs, int64_t gp, int rows, int brow, int nv,
                                               int s0, int s1, double* lds,
                                               d4v (&acc)[OCfg::FM][OCfg::FN]) {
  typedef OCfg T;
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int wm = wave % T::WM, wn = wave / T::WM;
  const int ux = cube_pitch(nv) / 8, units = nv * ux;
  // element e: rows xt + 32 e at k = kt; with AMAJ, A's row am at k = ak + 4 e.  Offsets stay
  // below 191 rows of 8 nv (nv + 7) bytes, below 2^31.
  const int kt = tid % T::BK, xt = tid / T::BK, am = tid % T::BM, ak = tid / T::BM;
  static_assert(T::NT / T::BK == 32 && T::NT / T::BM == 4 && T::EA == 4 && T::EB == 4, "mapping");
  unsigned aoff[AMAJ ? 1 : 4], boff[4];
#pragma unroll
  for (int e = 0; e < 4; ++e) {
    if (!AMAJ) aoff[e] = (unsigned)(min(xt + 32 * e, rows - 1) * rs + (kt & 7)) * 8u;
    // rows n >= nv of B (only in the last column tile) read the Omega1 row
    const int n = xt + 32 * e;
    boff[e] = ((unsigned)(n < brow >> 6 ? n : (brow >> 6) + (brow & 63)) * (unsigned)gp + (unsigned)kt) * 8u;
  }
  if (AMAJ) aoff[0] = (unsigned)(min(am, rows - 1) + ak * ys) * 8u;
  double ra[4], rb[4];
  unsigned amask = 0u;  // bit e (AMAJ), or bit 0: element inside K
  bool inb = true;
  int x0 = 2 * s0 / ux, y0 = 2 * s0 % ux;  // the stage's first unit: x, and y / 8
  auto fetch = [&](int s) __attribute__((always_inline)) {
    const bool two = 2 * s + 1 < units;  // the last stage may hold one unit
    const bool wrap = y0 + 1 == ux;
    const int64_t at = x0 * xs + (int64_t)y0 * 8 * ys;
    const int64_t step = wrap ? xs - (int64_t)y0 * 8 * ys : 8 * (int64_t)ys;  // to the second
    const BufRsrc sa = buf_rsrc(U + at), sb = buf_rsrc(G + (int64_t)s * T::BK);
    if constexpr (AMAJ) {
      // rows y >= nv hold the next x, or end the array
      const int left0 = nv - y0 * 8, left1 = !two ? 0 : wrap ? nv : left0 - 8;
      amask = 0u;
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        const bool in = ak + 4 * (e & 1) < (e < 2 ? left0 : left1);
        ra[e] = buf_load_f64(sa, in ? aoff[0] + (unsigned)((e < 2 ? 0 : step) + (e & 1) * 4 * ys) * 8u
                                    : 0u);
        amask |= in ? 1u << e : 0u;
      }
    } else {
      const unsigned h = kt < 8 ? 0u : two ? (unsigned)step * 8u : 0u;
#pragma unroll
      for (int e = 0; e < 4; ++e) ra[e] = buf_load_f64(sa, aoff[e] + h);
    }
    inb = kt < 8 || two;
    const unsigned kb = inb ? 0u : 64u;
#pragma unroll
    for (int e = 0; e < 4; ++e) rb[e] = buf_load_f64(sb, boff[e] - kb);
    y0 += 2;
    while (y0 >= ux) { y0 -= ux; ++x0; }
  };
  // lds_idx: row k at k LDA, the column XOR-ed by k
  double* wa = lds + (AMAJ ? ak * T::LDA : kt * T::LDA + (xt ^ kt));
  double* wb = lds + T::BK * T::LDA + kt * T::LDB + (xt ^ kt);
  auto store = [&](int o) __attribute__((always_inline)) {
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      if constexpr (AMAJ)
        wa[o + 4 * e * T::LDA + (am ^ (ak + 4 * e))] = ((amask >> e) & 1u) ? ra[e] : 0.0;
      else
        wa[o + 32 * e] = inb ? ra[e] : 0.0;
      wb[o + 32 * e] = inb ? rb[e] : 0.0;
    }
  };
  fetch(s0);
  store(0);
  __syncthreads();
  for (int s = s0; s < s1; ++s) {
    const int cur = ((s - s0) & 1) * T::STAGE;
    const bool more = s + 1 < s1;
    if (more) fetch(s + 1);
    mfma_stage<T>(lds + cur, lds + cur + T::BK * T::LDA, acc, lane, wm, wn);
    if (more) store(T::STAGE - cur);
    __syncthreads();
  }
}

__global__ __launch_bounds__(OCfg::NT, 4) void k_omega_lds(const double* __restrict__ cubes,
                                                           const double* __restrict__ Gbc,
                                                           const double* __restrict__ Gcb,
                                                           const int* __restrict__ tri,
                                                           double* __restrict__ Pvv, int no, int nv,
                                                           int nchunks, int tiles_n) {
  typedef OCfg T;
  __shared__ double lds[T::LDS_DOUBLES];
  const int pi = blockIdx.y, z = blockIdx.z;
  const int i = tri[3 * z], j = tri[3 * z + 1], k = tri[3 * z + 2];
  if (!perm_active(tri_kind(i, j, k), pi)) return;
  int p, q, r;
  perm_pqr(pi, i, j, k, p, q, r);
  const int ch = blockIdx.x % nchunks, tile = blockIdx.x / nchunks;
  const int m0 = (tile / tiles_n) * T::BM, n0 = (tile % tiles_n) * T::BN;
  const int rp = cube_pitch(nv), S = (nv * (rp / 8) + 1) / 2;
  const int s0 = (int)((int64_t)ch * S / nchunks), s1 = (int)((int64_t)(ch + 1) * S / nchunks);
  if (s0 >= s1) return;  // nchunks <= S, so never taken
  const int64_t pl = (int64_t)nv * rp, gp = g_pitch(nv);
  const double* U = cubes + ((int64_t)z * NSLOT + SLOT_TT) * cube_slot(nv);
  const double* G = (pi >= 2 && pi <= 4 ? Gcb : Gbc) + ((int64_t)r * (nv + no) + n0) * gp;
  const int brow = (nv - n0) << 6 | q;  // rows of B in the tile, and from there to the Omega1 row
  d4v acc[T::FM][T::FN];
  zero_acc<T>(acc);
  if (pi == 2 || pi == 5) {  // rows TT[x][y][a]
    omega_lds_tile<true>(U + m0, G, pl, rp, 1, gp, nv - m0, brow, nv, s0, s1, lds, acc);
  } else {  // TT[x][a][y], or TT[a][x][y]
    const bool mid = pi == 1 || pi == 4;
    const int64_t rs = mid ? rp : pl;
    omega_lds_tile<false>(U + m0 * rs, G, mid ? pl : rp, 1, rs, gp, nv - m0, brow, nv, s0, s1, lds, acc);
  }
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const int wm = wave % T::WM, wn = wave / T::WM;
  const int NV1 = nv + 1;
  double* pvv = Pvv + (((int64_t)z * 6 + pi) * nchunks + ch) * nv * (int64_t)NV1;
#pragma unroll
  for (int fm = 0; fm < T::FM; ++fm)
#pragma unroll
    for (int fn = 0; fn < T::FN; ++fn)
#pragma unroll
      for (int rr = 0; rr < 4; ++rr) {
        const int a = m0 + acc_row<T>(wm, fm, lane, rr), n = n0 + acc_col<T>(wn, fn, lane);
        if (a < nv && n <= nv) pvv[(int64_t)a * NV1 + n] = acc[fm][fn][rr];
      }
}

// cubes: TT and TTT of each triple
__global__ __launch_bounds__(OCfg::NT) void k_omega_f32(const float* __restrict__ cubes,
                                                        const float* __restrict__ Gbc,
                                                        const float* __restrict__ Gcb,
                                                        const int* __restrict__ tri,
                                                        double* __restrict__ Pvv, int no, int nv,
                                                        int nchunks, int tiles_n) {
  typedef OCfg T;
  constexpr unsigned ES = sizeof(float);
  __shared__ float lds[T::LDS_DOUBLES];
  const int pi = blockIdx.y, z = blockIdx.z;
  const int i = tri[3 * z], j = tri[3 * z + 1], k = tri[3 * z + 2];
  if (!perm_active(tri_kind(i, j, k), pi)) return;
  int p, q, r;
  perm_pqr(pi, i, j, k, p, q, r);
  const int ch = blockIdx.x % nchunks, tile = blockIdx.x / nchunks;
  const int m0 = (tile / tiles_n) * T::BM, n0 = (tile % tiles_n) * T::BN;
  const int64_t nvl = nv, nv2 = nvl * nvl, nv3 = nv2 * nvl;
  const int K = nv * nv;
  const int S = (K + T::BK - 1) / T::BK;
  const int s0 = (int)((int64_t)ch * S / nchunks), s1 = (int)((int64_t)(ch + 1) * S / nchunks);
  if (s0 >= s1) return;  // nchunks <= S, so never taken
  const bool cb = (pi == 2 || pi == 4);
  const bool amaj = !(pi == 0 || pi == 3);  // a contiguous, k stride nv
  const int ttt = (pi == 1 || pi == 3 || pi == 4) ? 1 : 0;
  const float* U = cubes + ((int64_t)z * 2 + ttt) * nv3;
  const float* G = (cb ? Gcb : Gbc) + (int64_t)r * (nv + no) * nv2;
  const int ask = amaj ? nv : 1;  // k stride of A in elements
  // tile origins (k = 0) of the two operands
  const float* A0 = amaj ? U + m0 : U + (int64_t)m0 * K;
  const float* B0 = G + (int64_t)n0 * K;

  // Per-thread part of every stage.  A: element e at (row/column x_e, k_e) of the
  // stage, global byte offset aoff[e] plus that of k_e from the stage origin, LDS slot
  // alds[e].  Rows past nv repeat row nv - 1 (their outputs are never stored).
  // B rows n < nv are G rows n; rows n >= nv (only in the last column tile) read the
  // Omega1 row nv + q.  Offsets are relative to the tile origin: below 191 rows of
  // stride nv^2 <= 2^20, so below 2^31 bytes.
  const int tid = threadIdx.x;
  constexpr int RP = T::NT / T::BK;  // k-fast mapping: 32 rows per element step
  constexpr int KP = T::NT / T::BM;  // a-fast mapping: 4 k per element step
  unsigned aoff[T::EA], boff[T::EB];
  int ak[T::EA], alds[T::EA], blds[T::EB];
  const int kt = tid % T::BK, xt = tid / T::BK;
  if (amaj) {
    const int x = tid % T::BM, k0t = tid / T::BM;
    const unsigned xc = (unsigned)(min(m0 + x, nv - 1) - m0);
#pragma unroll
    for (int e = 0; e < T::EA; ++e) {
      ak[e] = k0t + e * KP;
      aoff[e] = xc * ES;
      alds[e] = lds_idx<T::BK>(ak[e], x, T::LDA);
    }
  } else {
#pragma unroll
    for (int e = 0; e < T::EA; ++e) {
      ak[e] = kt;
      aoff[e] = (unsigned)(min(m0 + xt + e * RP, nv - 1) - m0) * (unsigned)K * ES;
      alds[e] = lds_idx<T::BK>(kt, xt + e * RP, T::LDA);
    }
  }
#pragma unroll
  for (int e = 0; e < T::EB; ++e) {
    const int n = n0 + xt + e * RP;
    boff[e] = (unsigned)((n < nv ? n : nv + q) - n0) * (unsigned)K * ES;
    blds[e] = T::BK * T::LDA + lds_idx<T::BK>(kt, xt + e * RP, T::LDB);
  }
  const unsigned ask8 = (unsigned)ask * ES;
  float ra[T::EA], rb[T::EB];
  // which loaded elements lie inside K (bit e for A, one flag for B); the zero of the
  // others is applied at the LDS store, after the current stage's MFMAs, so that the
  // loads stay in flight during them
  unsigned amask = ~0u;
  bool inb = true;
  auto fetch = [&](int s) {
    const int k0 = s * T::BK;
    const BufRsrc sb = buf_rsrc(B0 + k0);
    const int kl = K - 1 - k0;  // last valid k of this stage (only the last stage is partial)
    amask = 0u;
    if (amaj) {
      const BufRsrc sa = buf_rsrc(A0 + (int64_t)k0 * ask);
#pragma unroll
      for (int e = 0; e < T::EA; ++e) {
        const bool in = ak[e] <= kl;
        const int kc = in ? ak[e] : kl;  // k past K reads a valid element
        ra[e] = buf_load_f32(sa, aoff[e] + (unsigned)kc * ask8);
        amask |= in ? (1u << e) : 0u;
      }
    } else {
      const BufRsrc sa = buf_rsrc(A0 + k0);
      const bool in = kt <= kl;
      const unsigned ko = (unsigned)(in ? kt : kl) * ES;  // k past K reads a valid element
#pragma unroll
      for (int e = 0; e < T::EA; ++e) {
        ra[e] = buf_load_f32(sa, aoff[e] + ko);
        amask |= in ? (1u << e) : 0u;
      }
    }
    inb = kt <= kl;
    const unsigned kb = (unsigned)(inb ? kt : kl) * ES;
#pragma unroll
    for (int e = 0; e < T::EB; ++e) rb[e] = buf_load_f32(sb, boff[e] + kb);
  };
  auto store = [&](float* st) {
#pragma unroll
    for (int e = 0; e < T::EA; ++e) st[alds[e]] = ((amask >> e) & 1u) ? ra[e] : 0.f;
#pragma unroll
    for (int e = 0; e < T::EB; ++e) st[blds[e]] = inb ? rb[e] : 0.f;
  };
  f4v_ acc[T::FM][T::FN];
#pragma unroll
  for (int fm = 0; fm < T::FM; ++fm)
#pragma unroll
    for (int fn = 0; fn < T::FN; ++fn) acc[fm][fn] = f4v_{0, 0, 0, 0};
  const int lane = tid & 63, wave = tid >> 6;
  const int wm = wave % T::WM, wn = wave / T::WM;
  fetch(s0);
  store(lds);
  __syncthreads();
  for (int s = s0; s < s1; ++s) {
    float* cur = lds + ((s - s0) & 1) * T::STAGE;
    float* nxt = lds + ((s - s0 + 1) & 1) * T::STAGE;
    const bool more = s + 1 < s1;
    if (more) fetch(s + 1);
    // lane supplies A[m = l%16][k = l/16] and B[k = l/16][n = l%16] to each MFMA
#pragma unroll
    for (int kk = 0; kk < T::BK / 4; ++kk) {
      const int kr = kk * 4 + (lane >> 4);
      const int sw = (lane & 15) ^ lds_swz<T::BK>(kr);
      float a[T::FM], b[T::FN];
#pragma unroll
      for (int fm = 0; fm < T::FM; ++fm) a[fm] = cur[kr * T::LDA + (wm * T::FM + fm) * 16 + sw];
#pragma unroll
      for (int fn = 0; fn < T::FN; ++fn)
        b[fn] = cur[T::BK * T::LDA + kr * T::LDB + (wn * T::FN + fn) * 16 + sw];
#pragma unroll
      for (int fm = 0; fm < T::FM; ++fm)
#pragma unroll
        for (int fn = 0; fn < T::FN; ++fn)
          acc[fm][fn] = __builtin_amdgcn_mfma_f32_16x16x4f32(a[fm], b[fn], acc[fm][fn], 0, 0, 0);
    }
    if (more) store(nxt);
    __syncthreads();
  }
  const int NV1 = nv + 1;
  double* pvv = Pvv + (((int64_t)z * 6 + pi) * nchunks + ch) * nvl * NV1;
#pragma unroll
  for (int fm = 0; fm < T::FM; ++fm)
#pragma unroll
    for (int fn = 0; fn < T::FN; ++fn)
#pragma unroll
      for (int rr = 0; rr < 4; ++rr) {
        const int a = m0 + (wm * T::FM + fm) * 16 + 4 * (lane >> 4) + rr;  // FP32 16x16x4 MFMA rows
        const int n = n0 + acc_col<T>(wn, fn, lane);
        if (a < nv && n <= nv) pvv[(int64_t)a * NV1 + n] = (double)acc[fm][fn][rr];
      }
}

// The (triple, permutation) pairs of a batch with first occupied index p, second index q
// (any with q < 0) and permutation in the mask `perms`, in batch order (triple, then
// permutation): lz = 6 z + pi, lqr = q no + r; at most two per triple and p, so at most
// 2 * MAX_BATCH.  Every thread of the workgroup (256 or more, whole wavefronts) calls it; it
// holds barriers.  One candidate per thread and round, placed by ballots; cz is LDS scratch
// of one int per wavefront.  Returns the count.
#define PLIST_MAX (2 * MAX_BATCH)
__device__ inline int list_pairs(const int* __restrict__ tri, int ntri, int p, int q,
                                 unsigned perms, int no, int* lz, int* lqr, int* cz) {
  const int nt = (int)blockDim.x, lane = threadIdx.x & 63, wave = threadIdx.x >> 6, nw = nt >> 6;
  int base = 0;
  for (int e0 = 0; e0 < 6 * ntri; e0 += nt) {
    const int e = e0 + (int)threadIdx.x;
    bool in = false;
    int qr = 0;
    if (e < 6 * ntri) {
      const int z = e / 6, pi = e - 6 * z;
      const int i = tri[3 * z], j = tri[3 * z + 1], k = tri[3 * z + 2];
      int pp, qq, rr;
      perm_pqr(pi, i, j, k, pp, qq, rr);
      in = pp == p && (q < 0 || qq == q) && ((perms >> pi) & 1u) &&
           perm_active(tri_kind(i, j, k), pi);
      qr = qq * no + rr;
    }
    const unsigned long long hit = __ballot(in);
    if (lane == 0) cz[wave] = __popcll(hit);
    __syncthreads();
    int at = base;
    for (int w = 0; w < nw; ++w) {
      const int c = cz[w];
      if (w < wave) at += c;
      base += c;
    }
    at += __popcll(hit & ((1ull << lane) - 1ull));
    if (in && at < PLIST_MAX) {
      lz[at] = e;
      lqr[at] = qr;
    }
    __syncthreads();
  }
  return base < PLIST_MAX ? base : PLIST_MAX;
}
#define LIST_SCRATCH 16

// The view of U_pi[a, b, c] at fixed b as a strided (a, c) matrix: base + b * sbb, (sm, sk)
// (k_zv, for which the mix writes tau~T too), in the cubes [x][y][z] with the row pitch rp (x
// stride nv rp, y stride rp).
__device__ inline void u_view(int pi, int nv, int rp, int& slot, int& sbb, int& sm, int& sk) {
  const int pl = nv * rp;
  switch (pi) {
    case 0: slot = SLOT_TT; sbb = rp; sm = pl; sk = 1; break;    // tau~[a][b][c]
    case 1: slot = SLOT_TT; sbb = pl; sm = rp; sk = 1; break;    // tau~[b][a][c]
    case 2: slot = SLOT_TT; sbb = rp; sm = 1; sk = pl; break;    // tau~[c][b][a]
    case 3: slot = SLOT_TTT; sbb = rp; sm = pl; sk = 1; break;   // tau~T[a][b][c]
    case 4: slot = SLOT_TTT; sbb = rp; sm = 1; sk = pl; break;   // tau~T[c][b][a]
    default: slot = SLOT_TT; sbb = pl; sm = 1; sk = rp; break;   // tau~[b][c][a]
  }
}

// ---------------------------------------------------------------------------
// Omega contraction: the oo and Fock terms, output-stationary
// ---------------------------------------------------------------------------
// One workgroup of 4 wavefronts per (p, form, pair of b, 64-wide tile of a) sums, over
// the batch's pairs with that p in batch order,
//   Out[p][l][b][a] += sum_c Hs[q][r][c][l] U[a,b,c]      (l < no)
// (Hs[q][r][c][l] = delta_lq F_rc - g_{qlrc}) and adds the sum into Out
// (read-modify-write; successive batches are ordered by the caller).  Form 0 takes the
// permutations whose view of tau~ has a or c contiguous (pi 0, 1, 2, 5) and Out = OtT;
// form 1 those with b contiguous (pi 3, 4), with the roles of a and b exchanged and
// Out = Ot2: both load rows of the one cube, and no transposed copy of it is needed.
// Wavefront w owns the 16 columns a0 = tile + 16 w of both b and every row l (FNO blocks
// of 16), as D[l][a] of the FP64 MFMA with A = Hs, B = U.  The kernel streams U once
// per pair and is bound by the memory pipeline, so there are no workgroup
// barriers in the loop: the next step's loads are in flight during the current
// step's MFMAs, and the Hs fragments serve both b.  Within a 16-c step, lane
// group kq = lane / 16 feeds c = c0 + 4 kq + t to MFMA t (the same order on both
// operands, which leaves the sum unchanged).  Views with a contiguous are loaded
// in the MFMA layout directly (16 consecutive a per row of c); views with c
// contiguous are loaded along c (4 rows of 16 consecutive c per instruction) and
// transposed through a wavefront-private LDS tile.
// SHARES: of the workgroup's 4 WS wavefronts 1, 2 or 4 (oo_waves_a) lie side by side over a
// and the others take shares of the (pair, step) loop, added in share order.
// the view of U_pi as (column m, fixed index b, contracted c) in TT[x][y][z]
__device__ inline void oo_view(int pi, int nv, int rp, int& sbb, int& sm, int& sk) {
  const int pl = nv * rp;
  switch (pi) {
    case 0: sbb = rp; sm = pl; sk = 1; break;   // TT[a][b][c]
    case 1: sbb = pl; sm = rp; sk = 1; break;   // TT[b][a][c]
    case 2: sbb = rp; sm = 1; sk = pl; break;   // TT[c][b][a]
    case 3: sbb = pl; sm = 1; sk = rp; break;   // TT[a][c][b], m = b, fixed a
    case 4: sbb = rp; sm = 1; sk = pl; break;   // TT[c][a][b], m = b, fixed a
    default: sbb = pl; sm = 1; sk = rp; break;  // TT[b][c][a]
  }
}
// wavefronts side by side over a in the form with shares, and its shares (1: the other form).
// no <= 16, where 16 wavefronts have the registers: shares where fewer than 640 workgroups
// run, since a small launch is one chain of loads per wavefront.  MEASURED, calls with /
// without: 4/20 (80) 84 / 99 us, 5/30 (150) 130 / 156, 6/45 (276) 461 / 506, 8/64 (512) 1593 /
// 1633, 12/60 (720) 3.82 / 3.79 ms, 3/140 (1260) 1.459 / 1.436.
// Above, 4 wavefronts: shares up to nv = 32, where 2 or 3 of them would have no columns.
// MEASURED, BF16x3 mixed-all calls with / without: 63/8 27.1 / 32.6 ms, 63/16 47.2 / 57.5,
// 40/12 6.6 / 7.9, 48/24 27.5 / 31.7, 30/20 4.7 / 5.7, 20/32 2.65 / 2.87.
__host__ __device__ inline int oo_waves_a(int nv) { return nv <= 16 ? 1 : nv <= 32 ? 2 : 4; }
__host__ __device__ inline int oo_shares(int no, int nv) {
  if (no > 16) return 4 / oo_waves_a(nv);
  return ((nv + 1) / 2) * ((nv + 63) / 64) * no * 2 < 640 ? 16 / oo_waves_a(nv) : 1;
}
// SEQ: the packed form, where a wavefront takes the shares in turn: the sums of the call alone.
template <int FNO, int WS, bool SHARES, bool SEQ>
__device__ __forceinline__ void omega_oo_body(const double* __restrict__ cubes,
                                              const double* __restrict__ Hs,
                                              const int* __restrict__ tri, int ntri,
                                              double* __restrict__ Ot2,
                                              double* __restrict__ OtT, int no, int nv,
                                              int tiles_a, int bx, int by, int form) {
  constexpr int NB = 2;
  // per wavefront: 16 rows a x 16 c (+1 pad) of each b; with SHARES its share's sums
  constexpr int LT = SHARES && NB * FNO * 256 > NB * 16 * 17 ? NB * FNO * 256 : NB * 16 * 17;
  __shared__ double lts[4 * WS][LT];
  __shared__ int lz[PLIST_MAX], lqr[PLIST_MAX], cz[LIST_SCRATCH];
  double* __restrict__ Out = form ? Ot2 : OtT;
  const int p = by;
  const int bp = bx / tiles_a;
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const int wa = SHARES ? oo_waves_a(nv) : 4;  // wavefronts over a
  const int share = wave / wa;
  const int shares = SHARES ? 4 * WS / wa : SEQ ? oo_shares(no, nv) : 1;
  const int a0 = (bx % tiles_a) * 16 * wa + 16 * (wave % wa);
  double (*lt)[16][17] = (double (*)[16][17])lts[wave];
  const int n = list_pairs(tri, ntri, p, -1, form ? 0x18u : 0x27u, no, lz, lqr, cz);
  if (n == 0 || (!SHARES && a0 >= nv)) return;  // no workgroup barrier follows
  const int m = lane & 15, kq = lane >> 4;
  int bb[NB];
#pragma unroll
  for (int j = 0; j < NB; ++j) bb[j] = min(NB * bp + j, nv - 1);
  const int64_t nvl = nv, nv2 = nvl * nvl;
  d4v acc[NB][FNO];
#pragma unroll
  for (int j = 0; j < NB; ++j)
#pragma unroll
    for (int f = 0; f < FNO; ++f) acc[j][f] = d4v{0.0, 0.0, 0.0, 0.0};
  // flattened (pair, 16-c step) loop with the next step's loads issued before
  // the current step's MFMAs
  const int cs = (nv + 15) / 16;
  // Elements with c past nv load a valid element (c clamped) and are zeroed when they
  // are used (cm: bit i or tt set for c < nv), so that the next step's loads stay in
  // flight over the current step's MFMAs.
  double u[2][NB][4], h[2][FNO][4];
  bool cc1[2];
  unsigned cm1[2];
  auto load = [&](int it, double (&uu)[NB][4], double (&hh)[FNO][4], bool& ccont,
                  unsigned& cm) {
    const int t = it / cs, c0 = (it - t * cs) * 16;
    const int zp = lz[t], zz = zp / 6, pi = zp % 6;
    int sbb, sm, sk;
    oo_view(pi, nv, cube_pitch(nv), sbb, sm, sk);
    const double* ub = cubes + ((int64_t)zz * NSLOT + SLOT_TT) * cube_slot(nv);
    ccont = (sk == 1);
    if (ccont) {  // element i: row a0 + 4 i + kq, c = c0 + m
      const int c = c0 + m;
      const int cc = min(c, nv - 1);
      cm = c < nv ? 15u : 0u;
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        const int row = min(a0 + 4 * i + kq, nv - 1);
#pragma unroll
        for (int j = 0; j < NB; ++j) uu[j][i] = ub[(int64_t)row * sm + (int64_t)bb[j] * sbb + cc];
      }
    } else {  // element tt: row a0 + m, c = c0 + 4 kq + tt
      const int64_t ra = (int64_t)min(a0 + m, nv - 1);
      cm = 0u;
#pragma unroll
      for (int tt = 0; tt < 4; ++tt) {
        const int c = c0 + 4 * kq + tt;
        const int cc = min(c, nv - 1);
        cm |= c < nv ? 1u << tt : 0u;
#pragma unroll
        for (int j = 0; j < NB; ++j) uu[j][tt] = ub[ra + (int64_t)bb[j] * sbb + (int64_t)cc * sk];
      }
    }
    const double* hb = Hs + (int64_t)lqr[t] * no * nvl;
#pragma unroll
    for (int tt = 0; tt < 4; ++tt) {
      const int cc = min(c0 + 4 * kq + tt, nv - 1);
#pragma unroll
      for (int f = 0; f < FNO; ++f) hh[f][tt] = hb[(int64_t)cc * no + min(16 * f + m, no - 1)];
    }
  };
  auto mma = [&](const double (&uu)[NB][4], const double (&hh)[FNO][4], bool ccont, unsigned cm) {
    double x[NB][4];
    if (ccont) {  // transpose through this wavefront's LDS tile
#pragma unroll
      for (int j = 0; j < NB; ++j)
#pragma unroll
        for (int i = 0; i < 4; ++i) lt[j][4 * i + kq][m] = cm ? uu[j][i] : 0.0;
      __builtin_amdgcn_wave_barrier();
#pragma unroll
      for (int j = 0; j < NB; ++j)
#pragma unroll
        for (int tt = 0; tt < 4; ++tt) x[j][tt] = lt[j][m][4 * kq + tt];
      __builtin_amdgcn_wave_barrier();
    } else {
#pragma unroll
      for (int j = 0; j < NB; ++j)
#pragma unroll
        for (int tt = 0; tt < 4; ++tt) x[j][tt] = ((cm >> tt) & 1u) ? uu[j][tt] : 0.0;
    }
#pragma unroll
    for (int tt = 0; tt < 4; ++tt)
#pragma unroll
      for (int j = 0; j < NB; ++j)
#pragma unroll
        for (int f = 0; f < FNO; ++f)
          acc[j][f] = __builtin_amdgcn_mfma_f64_16x16x4f64(hh[f][tt], x[j][tt], acc[j][f], 0, 0, 0);
  };
  auto run = [&](int sh) __attribute__((always_inline)) {  // one share of the loop into acc
    const int it0 = n * cs * sh / shares, nit = n * cs * (sh + 1) / shares;
    if (it0 < nit) load(it0, u[0], h[0], cc1[0], cm1[0]);
    for (int it = it0; it < nit; it += 2) {
      if (it + 1 < nit) load(it + 1, u[1], h[1], cc1[1], cm1[1]);
      mma(u[0], h[0], cc1[0], cm1[0]);
      if (it + 1 < nit) {
        if (it + 2 < nit) load(it + 2, u[0], h[0], cc1[0], cm1[0]);
        mma(u[1], h[1], cc1[1], cm1[1]);
      }
    }
  };
  if constexpr (!SEQ) {
    if (a0 < nv) run(SHARES ? share : 0);
  } else {
    d4v tot[NB][FNO];
    for (int sh = 0; sh < shares; ++sh) {
      run(sh);
#pragma unroll
      for (int j = 0; j < NB; ++j)
#pragma unroll
        for (int f = 0; f < FNO; ++f) {
          tot[j][f] = sh == 0 ? acc[j][f] : tot[j][f] + acc[j][f];
          acc[j][f] = d4v{0.0, 0.0, 0.0, 0.0};
        }
    }
#pragma unroll
    for (int j = 0; j < NB; ++j)
#pragma unroll
      for (int f = 0; f < FNO; ++f) acc[j][f] = tot[j][f];
  }
  if constexpr (SHARES) {
    if (share > 0) {
#pragma unroll
      for (int j = 0; j < NB; ++j)
#pragma unroll
        for (int f = 0; f < FNO; ++f)
#pragma unroll
          for (int rr = 0; rr < 4; ++rr) lts[wave][((j * FNO + f) * 4 + rr) * 64 + lane] = acc[j][f][rr];
    }
    __syncthreads();
    if (share > 0) return;
    for (int h = 1; h < shares; ++h)
#pragma unroll
      for (int j = 0; j < NB; ++j)
#pragma unroll
        for (int f = 0; f < FNO; ++f)
#pragma unroll
          for (int rr = 0; rr < 4; ++rr)
            acc[j][f][rr] += lts[wave + h * wa][((j * FNO + f) * 4 + rr) * 64 + lane];
  }
  const int ac = a0 + m;
#pragma unroll
  for (int j = 0; j < NB; ++j) {
    const int b = NB * bp + j;
#pragma unroll
    for (int f = 0; f < FNO; ++f)
#pragma unroll
      for (int rr = 0; rr < 4; ++rr) {
        const int l = 16 * f + kq + 4 * rr;
        if (l < no && ac < nv && b < nv)
          Out[(((int64_t)p * no + l) * nvl + b) * nvl + ac] += acc[j][f][rr];
      }
  }
}

template <int FNO, int WS, bool SHARES>
__global__ __launch_bounds__(256 * WS) void k_omega_oo(const double* __restrict__ cubes,
                                                       const double* __restrict__ Hs,
                                                       const int* __restrict__ tri, int ntri,
                                                       double* __restrict__ Ot2,
                                                       double* __restrict__ OtT, int no, int nv,
                                                       int tiles_a) {
  omega_oo_body<FNO, WS, SHARES, false>(cubes, Hs, tri, ntri, Ot2, OtT, no, nv, tiles_a, blockIdx.x,
                                        blockIdx.y, blockIdx.z);
}

// For output block (p, x):
//   Ot2[p][x][a][d] += sum of Pvv[z][pi][chunk][a][d] over the batch's (triple,
//                      permutation) pairs with that p and q == x, and chunks;
//   Ot1[p][a]       += column nv of Pvv over the pairs with that p (block x == no).
// 256 threads as 256 / slices elements by `slices` shares of the (pair, chunk) slabs (every
// slices-th, in order), which are added in share order: a fixed order, no atomics.  One
// share streams best where there are many blocks; a few blocks with many slabs each are a
// chain of dependent adds, so small launches take more shares (reduce_slices), and the few
// elements of Ot1 always 16 (at 6/45, 17 triples and 32 chunks the one-share form took 91 us).
constexpr int OT1_SLICES = 16;
__device__ __forceinline__ void reduce_body(const int* __restrict__ tri, int ntri,
                                            const double* __restrict__ Pvv,
                                            double* __restrict__ Ot1, double* __restrict__ Ot2,
                                            int no, int nv, int nchunks, int slices, int bx, int by,
                                            int bz) {
  __shared__ int lz[PLIST_MAX], lqr[PLIST_MAX], cz[LIST_SCRATCH];
  __shared__ double part[256];
  const int p = bz, x = by;
  const bool one = x == no;  // Ot1
  if (one) slices = OT1_SLICES;
  const int els = 256 / slices;
  const int n = one ? nv : nv * nv;
  if (bx * els >= n) return;
  const int cnt = list_pairs(tri, ntri, p, one ? -1 : x, 0x3fu, no, lz, lqr, cz);
  if (cnt == 0) return;  // a block without pairs leaves its output as it is
  const int64_t nvl = nv;
  const int NV1 = nv + 1;
  const int64_t pvs = nvl * NV1;  // one chunk slab
  const int share = threadIdx.x / els, el = threadIdx.x % els;
  const int e = bx * els + el;
  double s = 0.0;
  if (e < n) {
    const int64_t off = one ? (int64_t)e * NV1 + nv : (int64_t)(e / nv) * NV1 + e % nv;
    for (int t = 0; t < cnt; ++t) {
      const double* pv = Pvv + (int64_t)lz[t] * nchunks * pvs + off;
      // chunk c of pair t is slab t nchunks + c of the list
      int c = (share - t * nchunks) % slices;
      if (c < 0) c += slices;
#pragma unroll 16
      for (; c < nchunks; c += slices) s += pv[c * pvs];
    }
  }
  if (slices > 1) {
    part[threadIdx.x] = s;
    __syncthreads();
    if (share == 0)
      for (int h = 1; h < slices; ++h) s += part[h * els + el];
  }
  if (share == 0 && e < n) {
    if (one) Ot1[(int64_t)p * nvl + e] += s;
    else Ot2[((int64_t)p * no + x) * nvl * nvl + e] += s;
  }
}

__global__ __launch_bounds__(256) void k_reduce(const int* __restrict__ tri, int ntri,
                                                const double* __restrict__ Pvv,
                                                double* __restrict__ Ot1, double* __restrict__ Ot2,
                                                int no, int nv, int nchunks, int slices) {
  reduce_body(tri, ntri, Pvv, Ot1, Ot2, no, nv, nchunks, slices, blockIdx.x, blockIdx.y,
              blockIdx.z);
}

// Shares of k_reduce: enough workgroups for two per CU, at most 16 shares.
static int reduce_slices(int no, int nv) {
  int sl = 1;
  while (sl < 16 && (int64_t)nblk((int64_t)nv * nv, 256 / sl) * no * no < 512) sl *= 4;
  return sl;
}
// its grid: element blocks (at least those of Ot1), second index and Ot1, first index
static dim3 reduce_grid(int no, int nv) {
  const unsigned gx = std::max(nblk((int64_t)nv * nv, 256 / reduce_slices(no, nv)),
                               nblk(nv, 256 / OT1_SLICES));
  return dim3(gx, no + 1, no);
}

// ---------------------------------------------------------------------------
// Preparation for the Jacobian transformations (Algorithm 2): for each distinct
// occupied permutation (p,q,r) of a triple, with U = tau~_{pqr},
//   Zv[a][b][p][d] -= sum_c    U[a,b,c] g_{qdrc}     (g_{qdrc} = Jo[q][r][d][c])
//   Zo[a][q][p][l] += sum_{bc} U[a,b,c] g_{lbrc}     (g_{lbrc} = Jo[l][r][b][c])
// ---------------------------------------------------------------------------

// Zv, output-stationary on wave tiles: one wavefront per (p, b, FM x FN blocks of (a, d))
// sums the batch's (triple, permutation) pairs with that p, in batch order, over c and
// subtracts the sum from Zv (read-modify-write; the batches run in order).  Units of 8 c, two
// in flight, no LDS; lane (r16, kq) holds c = 2 kq + h of row r16 of each block, loaded 8 bytes
// at a time from the views of U, which have c or a contiguous (one form for both: a loop for
// each kind doubled the registers), and 16 bytes from the rows of Jo.  Past c = nv the U
// operand is zero (an offset outside the resource); the unpadded rows of Jo go on in the next.
// Bound by the FP64 MFMAs.  Against 128 x 128 tiles through LDS with a barrier per 16 c, at
// 12/120: 2.42 -> 1.91 ms per batch of 32 triples (beside the other stream's kernels; 1.1 ms of
// MFMA), the call 43.5 -> 40.8 ms; with k_zo, 20/64 60.7 -> 21.5 ms.
template <int FM, int FN>
__global__ __launch_bounds__(WNT, shape_waves(FM, FN)) void k_zv(
    const double* __restrict__ cubes, const double* __restrict__ Jo, const int* __restrict__ tri,
    int ntri, double* __restrict__ Zv, int no, int nv, int tiles_m, int tiles_n) {
  __shared__ int lz[PLIST_MAX], lqr[PLIST_MAX], cz[LIST_SCRATCH];
  // the wave tiles of one p: column tiles fastest, then row tiles, then b
  const int per = nv * tiles_m * tiles_n, wgs = (per + 3) / 4;
  const unsigned wg = xcd_item(blockIdx.x, gridDim.x, (unsigned)(tiles_m * tiles_n));
  const int p = (int)(wg / (unsigned)wgs);
  const int n = __builtin_amdgcn_readfirstlane(list_pairs(tri, ntri, p, -1, 0x3fu, no, lz, lqr, cz));
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int item = (int)(wg % (unsigned)wgs) * 4 + wave;
  if (n == 0 || item >= per) return;  // no barrier follows
  const int n0 = item % tiles_n * (FN * 16), m0 = item / tiles_n % tiles_m * (FM * 16);
  const int b = item / (tiles_n * tiles_m);
  const int lane = threadIdx.x & 63, r16 = lane & 15, kq = lane >> 4;
  const int rp = cube_pitch(nv), ux = rp / 8;
  const int64_t css = cube_slot(nv), nv2 = (int64_t)nv * nv, nj = (int64_t)no * no * nv2;
  // the pair being loaded: its operands at the next unit, elements left in their arrays
  const double *pa, *pb;
  int64_t na, nb;
  int sm, sk, t = 0, uu = 0;
  auto open = [&](int at) {
    const int zp = __builtin_amdgcn_readfirstlane(lz[at]);
    const int qr = __builtin_amdgcn_readfirstlane(lqr[at]);
    int slot, sbb;
    u_view(zp % 6, nv, rp, slot, sbb, sm, sk);
    const int64_t off = (int64_t)b * sbb + (int64_t)m0 * sm;
    pa = cubes + ((int64_t)(zp / 6) * NSLOT + slot) * css + off;
    na = css - off;
    const int64_t jo = qr * nv2 + (int64_t)n0 * nv;
    pb = Jo + jo;
    nb = nj - jo;
    uu = 0;
  };
  const unsigned vb = (unsigned)(r16 * nv + 2 * kq) * 8u, bs = (unsigned)nv * 128u;
  auto fetch = [&](double (&a)[FM][2], double (&bb)[FN][2]) __attribute__((always_inline)) {
    const BufRsrc ra = buf_rsrc_n(pa, na), rb = buf_rsrc_n(pb, nb);
#pragma unroll
    for (int h = 0; h < 2; ++h) {
      const int c = 2 * kq + h;
      const unsigned va = uu * 8 + c < nv ? (unsigned)(c * sk + r16 * sm) * 8u : 0x80000000u;
#pragma unroll
      for (int f = 0; f < FM; ++f) a[f][h] = buf_load_f64_at(ra, va, (unsigned)(f * sm) * 128u);
    }
#pragma unroll
    for (int f = 0; f < FN; ++f) {
      const d2v v = buf_load_2f64(rb, vb, (unsigned)f * bs);
      bb[f][0] = v[0];
      bb[f][1] = v[1];
    }
    pa += 8 * sk;
    na = na > 8 * sk ? na - 8 * sk : 0;
    pb += 8;
    nb = nb > 8 ? nb - 8 : 0;
    if (++uu == ux) open(t = min(t + 1, n - 1));  // past the last pair: loads that nothing uses
  };
  d4v acc[FM][FN];
#pragma unroll
  for (int fm = 0; fm < FM; ++fm)
#pragma unroll
    for (int fn = 0; fn < FN; ++fn) acc[fm][fn] = d4v{0.0, 0.0, 0.0, 0.0};
  double a[2][FM][2], bb[2][FN][2];
  open(0);
  fetch(a[0], bb[0]);
  fetch(a[1], bb[1]);
  const int nu = n * ux;
  for (int u = 0; u < nu; u += 2) {
#pragma unroll
    for (int d = 0; d < 2; ++d) {
      if (u + d < nu) {
#pragma unroll
        for (int h = 0; h < 2; ++h)
#pragma unroll
          for (int fm = 0; fm < FM; ++fm)
#pragma unroll
            for (int fn = 0; fn < FN; ++fn)
              acc[fm][fn] = __builtin_amdgcn_mfma_f64_16x16x4f64(a[d][fm][h], bb[d][fn][h],
                                                                 acc[fm][fn], 0, 0, 0);
      }
      fetch(a[d], bb[d]);
    }
  }
#pragma unroll
  for (int fm = 0; fm < FM; ++fm)
#pragma unroll
    for (int fn = 0; fn < FN; ++fn)
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        const int a = m0 + frag_row<true, FM>(fm, kq, r), d = n0 + fn * 16 + r16;
        if (a < nv && d < nv) Zv[(((int64_t)a * nv + b) * no + p) * nv + d] -= acc[fm][fn][r];
      }
}

// Zo partials on wave tiles: per (triple, permutation, chunk of K)
//   Pzo[z][pi][chunk][a][l] = sum_{(x, y) in chunk} T[a,x,y] J_l[x][y]   (l < no)
// As in k_omega, two permutations share each view T of tau~ (rows a over its first, second or
// third index): (0, 3), (1, 4), (5, 2), the first with (b, c) = (x, y) and J_l = Jo[l][r], the
// second with (c, b) = (x, y) and J_l = Jo[r][l] (g_{lbrc} = g_{rclb}).  One wavefront per
// (triple, view, FM blocks of a, chunk) and both permutations, FN blocks of l each; units of 8
// y, two in flight, no LDS.  Past y = nv the U operand is zero (the padding of its rows, or an
// offset outside the resource) and the J operand repeats y = nv - 1.
// Bound by the cubes that it streams (1.3 GB a batch at 12/120).  Against 128 x 16 tiles
// through LDS, one permutation each and the transposed cube for two of them: 1.03 -> 0.72 ms a
// batch (beside the other stream's kernels), the call 40.8 -> 39.4 ms.
template <bool ROWS, int FM, int FN>
__device__ __forceinline__ void zo_tile(const double* ta, int64_t na, int sm, int sx, int sk,
                                        const double* const (&jb)[2][FN], int u0, int u1, int ux,
                                        int nv, d4v (&acc)[2][FM][FN]) {
  const int lane = threadIdx.x & 63, r16 = lane & 15, kq = lane >> 4;
  int x = u0 / ux, yu = u0 - x * ux;
  auto fetch = [&](double (&a)[FM][2], double (&b)[2][FN][2]) __attribute__((always_inline)) {
    const int64_t off = (int64_t)x * sx + (int64_t)yu * 8 * sk;
    const BufRsrc ra = buf_rsrc_n(ta + off, na > off ? na - off : 0);
    const int y = yu * 8 + 2 * kq;
    if constexpr (ROWS) {
      const unsigned va = (unsigned)(r16 * sm + 2 * kq) * 8u;
#pragma unroll
      for (int f = 0; f < FM; ++f) {
        const d2v v = buf_load_2f64(ra, va, (unsigned)(f * sm) * 128u);
        a[f][0] = v[0];
        a[f][1] = v[1];
      }
    } else {
#pragma unroll
      for (int h = 0; h < 2; ++h) {
        const unsigned va = y + h < nv ? (unsigned)((2 * kq + h) * sk + 2 * r16) * 8u : 0x80000000u;
#pragma unroll
        for (int f = 0; f < FM; f += 2) {
          const d2v v = buf_load_2f64(ra, va, (unsigned)f * 128u);
          a[f][h] = v[0];
          a[f + 1][h] = v[1];
        }
      }
    }
#pragma unroll
    for (int h = 0; h < 2; ++h) {
      const int64_t jo = (int64_t)x * nv + min(y + h, nv - 1);
#pragma unroll
      for (int e = 0; e < 2; ++e)
#pragma unroll
        for (int f = 0; f < FN; ++f) b[e][f][h] = jb[e][f][jo];
    }
    if (++yu == ux) {
      yu = 0;
      x = min(x + 1, nv - 1);  // past the last unit: loads that nothing uses
    }
  };
  double a[2][FM][2], b[2][2][FN][2];
  fetch(a[0], b[0]);
  fetch(a[1], b[1]);
  for (int u = u0; u < u1; u += 2) {
#pragma unroll
    for (int d = 0; d < 2; ++d) {
      if (u + d < u1) {
#pragma unroll
        for (int h = 0; h < 2; ++h)
#pragma unroll
          for (int e = 0; e < 2; ++e)
#pragma unroll
            for (int fm = 0; fm < FM; ++fm)
#pragma unroll
              for (int f = 0; f < FN; ++f)
                acc[e][fm][f] = __builtin_amdgcn_mfma_f64_16x16x4f64(a[d][fm][h], b[d][e][f][h],
                                                                     acc[e][fm][f], 0, 0, 0);
      }
      fetch(a[d], b[d]);
    }
  }
}

template <int FM, int FN>
__global__ __launch_bounds__(WNT) void k_zo(const double* __restrict__ cubes,
                                            const double* __restrict__ Jo,
                                            const int* __restrict__ tri, int ntri,
                                            double* __restrict__ Pzo, int no, int nv, int nchunks,
                                            int tiles_m) {
  static_assert(FM % 2 == 0, "pairs of row blocks");
  unsigned item = xcd_item(blockIdx.x, gridDim.x, 1) * 4 +
                  __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int m0 = (int)(item % (unsigned)tiles_m) * (FM * 16);
  item /= (unsigned)tiles_m;
  const int ch = (int)(item % (unsigned)nchunks);
  item /= (unsigned)nchunks;
  const int op = (int)(item % 3u), z = (int)(item / 3u);
  if (z >= ntri) return;
  const int i = tri[3 * z], j = tri[3 * z + 1], k = tri[3 * z + 2];
  const int kind = tri_kind(i, j, k);
  const int pis[2] = {op == 0 ? 0 : op == 1 ? 1 : 5, op == 0 ? 3 : op == 1 ? 4 : 2};
  const bool on[2] = {perm_active(kind, pis[0]), perm_active(kind, pis[1])};
  if (!on[0] && !on[1]) return;
  const int rp = cube_pitch(nv), ux = rp / 8, units = nv * ux;
  const int u0 = (int)((int64_t)ch * units / nchunks), u1 = (int)((int64_t)(ch + 1) * units / nchunks);
  const int lane = threadIdx.x & 63, r16 = lane & 15, kq = lane >> 4;
  const int64_t nvl = nv, nv2 = nvl * nvl, css = cube_slot(nv);
  const int pl = nv * rp;
  const double* jb[2][FN];
#pragma unroll
  for (int e = 0; e < 2; ++e) {
    int p, q, r;
    perm_pqr(pis[e], i, j, k, p, q, r);
#pragma unroll
    for (int f = 0; f < FN; ++f) {
      const int64_t l = min(f * 16 + r16, no - 1);
      jb[e][f] = Jo + (e ? r * (int64_t)no + l : l * no + r) * nv2;
    }
  }
  d4v acc[2][FM][FN];
#pragma unroll
  for (int e = 0; e < 2; ++e)
#pragma unroll
    for (int fm = 0; fm < FM; ++fm)
#pragma unroll
      for (int f = 0; f < FN; ++f) acc[e][fm][f] = d4v{0.0, 0.0, 0.0, 0.0};
  const double* TT = cubes + ((int64_t)z * NSLOT + SLOT_TT) * css;
  const int sm = op == 0 ? pl : op == 1 ? rp : 1;
  const double* ta = TT + (int64_t)m0 * sm;
  const int64_t na = css - (int64_t)m0 * sm;
  if (op == 2) zo_tile<false, FM, FN>(ta, na, 1, pl, rp, jb, u0, u1, ux, nv, acc);
  else zo_tile<true, FM, FN>(ta, na, sm, op == 0 ? rp : pl, 1, jb, u0, u1, ux, nv, acc);
#pragma unroll
  for (int e = 0; e < 2; ++e) {
    if (!on[e]) continue;
    double* out = Pzo + (((int64_t)z * 6 + pis[e]) * nchunks + ch) * nvl * no;
#pragma unroll
    for (int fm = 0; fm < FM; ++fm)
#pragma unroll
      for (int f = 0; f < FN; ++f)
#pragma unroll
        for (int r = 0; r < 4; ++r) {
          const int a = m0 + (op == 2 ? frag_row<false, FM>(fm, kq, r) : frag_row<true, FM>(fm, kq, r));
          const int l = f * 16 + r16;
          if (a < nv && l < no) out[(int64_t)a * no + l] = acc[e][fm][f][r];
        }
  }
}

// Zo[a][q][p][l] += the chunk sums of the batch's pairs with that (p, q), in batch order.
__global__ __launch_bounds__(256) void k_zo_reduce(const int* __restrict__ tri, int ntri,
                                                   const double* __restrict__ Pzo,
                                                   double* __restrict__ Zo, int no, int nv,
                                                   int nbchunks) {
  __shared__ int lz[PLIST_MAX], lqr[PLIST_MAX], cz[LIST_SCRATCH];
  const int q = blockIdx.y, p = blockIdx.z;
  const int n = list_pairs(tri, ntri, p, q, 0x3fu, no, lz, lqr, cz);
  const int64_t e = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (n == 0 || e >= (int64_t)nv * no) return;
  const int a = (int)(e / no), l = (int)(e % no);
  const int64_t slab = (int64_t)nv * no;
  double s = 0.0;
  for (int t = 0; t < n; ++t) {
    const double* pz = Pzo + (int64_t)lz[t] * nbchunks * slab + e;
    for (int c = 0; c < nbchunks; ++c) s += pz[c * slab];
  }
  Zo[(((int64_t)a * no + q) * no + p) * no + l] += s;
}

void launch_zv(const double* cubes, const Blocks& b, const int* tri, int ntri, double* Zv, int no,
               int nv, hipStream_t st) {
  const int shape = pick_shape(nv, nv);
  int tm, tn;
  shape_tiles(shape, nv, nv, &tm, &tn);
  const unsigned wgs = nblk((int64_t)nv * tm * tn, 4) * (unsigned)no;
  with_shape(shape, [&](auto fm, auto fn) {
    constexpr int FM = decltype(fm)::value, FN = decltype(fn)::value;
    hipLaunchKernelGGL((k_zv<FM, FN>), dim3(wgs), dim3(WNT), 0, st, cubes, b.Jo, tri, ntri, Zv, no, nv,
                       tm, tn);
  });
}

void launch_zo(const double* cubes, const Blocks& b, const int* tri, int ntri, double* Pzo,
               double* Zo, int no, int nv, hipStream_t st, bool reduce) {
  const int nbc = zo_nbchunks(nv, ntri);
  if (reduce) {
    hipLaunchKernelGGL(k_zo_reduce, dim3(nblk((int64_t)nv * no, 256), no, no), dim3(256), 0, st,
                       tri, ntri, Pzo, Zo, no, nv, nbc);
    return;
  }
  auto run = [&](auto* kernel, int fm) {
    const int tm = (int)nblk(nv, 16 * fm);
    hipLaunchKernelGGL(kernel, dim3(nblk((int64_t)tm * nbc * 3 * ntri, 4)), dim3(WNT), 0, st, cubes,
                       b.Jo, tri, ntri, Pzo, no, nv, nbc, tm);
  };
  if (no <= 16) run(k_zo<4, 1>, 4);
  else if (no <= 32) run(k_zo<4, 2>, 4);
  else if (no <= 48) run(k_zo<2, 3>, 2);
  else run(k_zo<2, 4>, 2);
}

double zprep_flops(int no, int nv, const int* kinds, int n) {
  const double v = nv, o = no;
  double perms = 0;
  for (int t = 0; t < n; ++t) perms += (kinds[t] == 0) ? 6 : 3;
  return perms * (2.0 * v * v * v * v + 2.0 * v * v * v * o);
}

// K chunks that make about 2048 workgroups of 128 x 128 tiles per launch, six products per
// triple; a multiple of 8 beyond 8.  (The Zo partials below, and the limit of the cube budget.)
int chunks_2048(int nv, int ntri) {
  const int t = (nv + 127) / 128;
  const int per = 6 * t * t * (ntri > 0 ? ntri : 1);
  int nbc = (2048 + per - 1) / per;
  if (nbc > 8) nbc = (nbc + 7) / 8 * 8;
  if (nbc > nv) nbc = nv;
  return nbc < 1 ? 1 : nbc;
}

// K chunks of the Zo partials per (triple, permutation pair, rows of a): chunks_2048, or where
// that leaves fewer than 2048 wavefronts of 64 rows (two per SIMD), as many as make 4096, of at
// least 64 units of 8 k.  MEASURED, k_zv and k_zo of a call with chunks_2048 alone / so raised:
// 8/187 34.3 / 32.8 ms, 4/250 11.9 / 11.4, 2/512 20.5 / 18.9, 2/896 186 / 160, 2/1024 359 / 305
// (from 288 wavefronts); 4096 at 12/120, which has 3072: 19.9 / 20.5.
int zo_nbchunks(int nv, int ntri) {
  const int n = chunks_2048(nv, ntri), per = 3 * (int)nblk(nv, 64) * (ntri > 0 ? ntri : 1);
  if (n * per >= 2048) return n;
  return std::max(n, std::min((4096 + per - 1) / per, nv * (cube_pitch(nv) / 8) / 64));
}

// The LDS form of the FP64 Omega GEMM: from nv = 448 on, unless its 128 x 128 tiles are so
// much emptier than the wave tiles that a 1.19 times higher rate per block does not make up for
// it.  MEASURED, LDS / wave tiles, ms per launch of 8 triples: 416 46.4 / 40.7, 448 54.4 / 52.6,
// 464 58.6 / 58.7, 480 62.9 / 60.6, 500 70.3 / 73.7, 512 97 / 122; of 3: 448 20.2 / 22.4, 530 41.0 /
// 34.0, 576 48.8 / 45.0, 644 84.0 / 80.4, 700 98.4 / 91.1, 768 121 / 148; of one: 576 14.1 / 15.1,
// 600 15.3 / 17.4, 772 58.7 / 47.3, 832 68.8 / 69.7, 900 92 / 95, 960 107 / 118, 1000 118 / 139, 1024
// 152 / 168.  (Rows a power of two of lines apart, as at 512, 768 and 1024, cost the wave tiles
// most.)
bool omega_lds(int nv) {
  const int t = OCfg::BM;
  return nv >= 448 && (double)nblk(nv, t) * nblk(nv + 1, t) * (t / 16) * (t / 16) <
                          1.19 * shape_cost(pick_shape(nv, nv + 1), nv, nv + 1);
}

// K chunks of the Omega GEMM of one (triple, permutation, tile).
// FP64: enough wave tiles for six rounds of the 2048 that are resident at two per SIMD
// (4096, 8192, 12288, 24576 tiles: 23/250 CVS list 585, 562, 548, 552 ms per call, 12/120
// 40.5, 39.6, 39.5, 40.6), as long as a chunk keeps 64 units of 8 k; small products are split
// further, down to 8 units per chunk, while there are fewer than 3072 wave tiles (CC3_OMEGA_WG in
// the environment sets the larger target instead).
// 128 x 128 LDS tiles (omega_lds, and fp32acc, the mixed-all forms): about 2048 workgroups, as a
// multiple of 8 beyond 8 so that the tiles of one (triple, permutation, chunk) are
// dispatched to the same XCD; at least 16 stages of 16 k per chunk and, with fp32acc, at most
// 4096 k, which the MFMA sums in FP32, so that their rounding does not grow with the batch (the
// split-BF16 form's K is the blocked lp_kb_len(nv) >= nv^2).
struct OmegaSplit {
  int64_t per, units;  // tiles of one triple (wave tiles, or LDS tiles), units (stages) of K
  int target, need;    // tiles of a launch; chunks that hold fp32acc's K to 4096
  bool lds;
};
static OmegaSplit omega_split(int nv, bool fp32acc) {
  static const int env = [] {
    const char* e = getenv("CC3_OMEGA_WG");
    return e ? atoi(e) : 0;
  }();
  OmegaSplit s;
  int tm, tn;
  s.lds = fp32acc || omega_lds(nv);
  if (!s.lds) {
    shape_tiles(pick_shape(nv, nv + 1), nv, nv + 1, &tm, &tn);
    s.units = (int64_t)nv * (cube_pitch(nv) / 8);
  } else {
    tm = (nv + OCfg::BM - 1) / OCfg::BM;
    tn = (nv + 1 + OCfg::BN - 1) / OCfg::BN;
    s.units = ((int64_t)nv * (fp32acc ? nv : cube_pitch(nv)) + OCfg::BK - 1) / OCfg::BK;
  }
  s.per = 6ll * tm * tn;
  s.target = env > 0 ? env : s.lds ? 2048 : 12288;
  s.need = fp32acc ? (int)((lp_kb_len(nv) + 4095) / 4096) : 1;
  return s;
}
static int omega_chunks(const OmegaSplit& s, int ntri) {
  const int64_t per = s.per * (ntri > 0 ? ntri : 1), big = (s.target + per - 1) / per;
  if (!s.lds) {
    const int64_t small = (3072 + per - 1) / per;
    return (int)std::max<int64_t>(1, std::max(std::min(big, s.units / 64), std::min(small, s.units / 8)));
  }
  auto eights = [](int64_t n) { return n > 8 ? (n + 7) / 8 * 8 : n; };
  const int64_t nch = std::min(eights(big), std::max<int64_t>(1, s.units / 16));
  return (int)(nch < s.need ? eights(s.need) : nch);
}

int omega_kchunks(int nv, int ntri, bool fp32acc) {
  return omega_chunks(omega_split(nv, fp32acc), ntri);
}

size_t omega_slabs(int nv, int batch, bool fp32acc) {
  const OmegaSplit s = omega_split(nv, fp32acc);
  size_t most = 1;
  for (int nb = 1; nb <= batch; ++nb)
    most = std::max(most, (size_t)nb * omega_chunks(s, nb));
  return most;
}

size_t zo_slabs(int nv, int batch) {
  size_t most = 1;
  for (int nb = 1; nb <= batch; ++nb) most = std::max(most, (size_t)nb * zo_nbchunks(nv, nb));
  return most;
}

int batch_within(int nv, int least, int most, size_t doubles) {
  const OmegaSplit s = omega_split(nv, false);
  const size_t cube = (size_t)cube_slot(nv), slab = 6 * (size_t)nv * (nv + 1);
  size_t slabs = 1;
  int best = least;
  for (int nb = 1; nb <= most; ++nb) {
    slabs = std::max(slabs, (size_t)nb * omega_chunks(s, nb));
    if (nb > best && NSLOT * nb * cube + slabs * slab <= doubles) best = nb;
  }
  return best;
}

static unsigned omega_wgs(int nv, int ntri, int nch, int shape) {
  int tm, tn;
  shape_tiles(shape, nv, nv + 1, &tm, &tn);
  return (unsigned)(((int64_t)tm * tn * 6 * nch * ntri + 3) / 4);
}

void launch_omega(const double* cubes, const Blocks& b, const int* tri, int ntri, double* Pvv,
                  int no, int nv, hipStream_t st) {
  const int nch = omega_kchunks(nv, ntri);
  int tm, tn;
  if (omega_lds(nv)) {
    typedef OCfg T;
    tm = (nv + T::BM - 1) / T::BM, tn = (nv + 1 + T::BN - 1) / T::BN;
    hipLaunchKernelGGL(k_omega_lds, dim3(nch * tm * tn, 6, ntri), dim3(T::NT), 0, st, cubes, b.Gbc,
                       b.Gcb, tri, Pvv, no, nv, nch, tn);
    return;
  }
  const int shape = pick_shape(nv, nv + 1);
  shape_tiles(shape, nv, nv + 1, &tm, &tn);
  with_shape(shape, [&](auto fm, auto fn) {
    hipLaunchKernelGGL((k_omega<decltype(fm)::value, decltype(fn)::value>),
                       dim3(omega_wgs(nv, ntri, nch, shape)), dim3(WNT), 0, st, cubes, b.Gbc, b.Gcb,
                       tri, ntri, Pvv, no, nv, nch, tm, tn);
  });
}

void launch_omega_f32(const float* cubesF, const float* GbcF, const float* GcbF, const int* tri,
                      int ntri, double* Pvv, int no, int nv, hipStream_t st) {
  typedef OCfg T;
  const int tm = (nv + T::BM - 1) / T::BM, tn = (nv + 1 + T::BN - 1) / T::BN;
  const int nch = omega_kchunks(nv, ntri, true);
  hipLaunchKernelGGL(k_omega_f32, dim3(nch * tm * tn, 6, ntri), dim3(T::NT), 0, st, cubesF, GbcF,
                     GcbF, tri, Pvv, no, nv, nch, tn);
}

__global__ void k_g_to_f32(const double* __restrict__ src, float* __restrict__ dst, int64_t rows,
                           int nv) {
  const int64_t nv2 = (int64_t)nv * nv, gp = g_pitch(nv), n = rows * nv2;
  const int rp = cube_pitch(nv);
  for (int64_t e = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; e < n;
       e += (int64_t)gridDim.x * blockDim.x) {
    const int xy = (int)(e % nv2);
    dst[e] = (float)src[e / nv2 * gp + (int64_t)(xy / nv) * rp + xy % nv];
  }
}

void launch_g_to_f32(const double* src, float* dst, int64_t rows, int nv, hipStream_t st) {
  unsigned g = nblk(rows * nv * nv, 256);
  if (g > 65536) g = 65536;
  hipLaunchKernelGGL(k_g_to_f32, dim3(g), dim3(256), 0, st, src, dst, rows, nv);
}

void launch_omega_oo(const double* cubes, const Blocks& b, const int* tri, int ntri, double* Ot2,
                     double* OtT, int no, int nv, hipStream_t st) {
  const int ta = (nv + 63) / 64;
  const dim3 grid(((nv + 1) / 2) * ta, no, 2);
  auto run = [&](auto* kernel, unsigned threads) {
    hipLaunchKernelGGL(kernel, grid, dim3(threads), 0, st, cubes, b.Hs, tri, ntri, Ot2, OtT, no, nv,
                       ta);
  };
  const bool sh = oo_shares(no, nv) > 1;
  if (no <= 16) sh ? run(k_omega_oo<1, 4, true>, 1024) : run(k_omega_oo<1, 1, false>, 256);
  else if (no <= 32) run(sh ? k_omega_oo<2, 1, true> : k_omega_oo<2, 1, false>, 256);
  else if (no <= 48) run(sh ? k_omega_oo<3, 1, true> : k_omega_oo<3, 1, false>, 256);
  else run(sh ? k_omega_oo<4, 1, true> : k_omega_oo<4, 1, false>, 256);
}

void launch_reduce(const int* tri, int ntri, const double* Pvv, double* Ot1, double* Ot2, int no,
                   int nv, bool fp32acc, hipStream_t st) {
  const int nch = omega_kchunks(nv, ntri, fp32acc);
  hipLaunchKernelGGL(k_reduce, reduce_grid(no, nv), dim3(256), 0, st, tri, ntri, Pvv, Ot1, Ot2, no,
                     nv, nch, reduce_slices(no, nv));
}

// ---------------------------------------------------------------------------
// Packed persistent launches of the triple loop (serving): each workgroup takes
// work items blockIdx.x, blockIdx.x + gridDim.x, ... of the union of the jobs'
// unpacked grids and runs the same body on the job's operands, so each job's
// arithmetic is exactly that of its own launch.
// ---------------------------------------------------------------------------
__device__ inline int pack_job(const PackJob* __restrict__ jobs, int njobs, int kind,
                               unsigned item) {
  int r = 0;
  while (r + 1 < njobs && item >= jobs[r + 1].first[kind]) ++r;
  return r;
}

template <class E, int FM, int FN>
__global__ __launch_bounds__(WNT, wbuild_waves<E>(FM, FN)) void k_pack_wbuild(
    const PackJob* __restrict__ jobs, int njobs, unsigned total) {
  for (unsigned item = blockIdx.x; item < total; item += gridDim.x) {
    const PackJob& J = jobs[pack_job(jobs, njobs, PK_W, item)];
    const unsigned local = item - J.first[PK_W];
    const int tm = (J.nv + 16 * FM - 1) / (16 * FM), tn = (J.nv + 16 * FN - 1) / (16 * FN);
    const int64_t cs = cube_slot(J.nv);
    const unsigned wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const void *t2 = J.t2, *t2N = J.t2N, *Gw = J.Gw, *Go = J.Go;
    if (sizeof(E) == 4) { t2 = J.lpt2; t2N = J.lpt2N; Gw = J.lpGwT; Go = J.lpGoT; }
    wbuild_body<E, 0, FM, FN>((const E*)t2, (const E*)t2N, (const E*)Gw, (const E*)Go, J.tri, J.ntri,
                              J.cubes, NSLOT * cs, cs, cube_pitch(J.nv), J.no, J.nv, tm, tn, 0,
                              local * 4 + wave);
  }
}

template <bool TWO>
__global__ __launch_bounds__(512) void k_pack_mix(const PackJob* __restrict__ jobs, int njobs,
                                                  unsigned total) {
  for (unsigned item = blockIdx.x; item < total; item += gridDim.x) {
    const PackJob& J = jobs[pack_job(jobs, njobs, PK_MIX, item)];
    const unsigned local = item - J.first[PK_MIX];
    const int nb = (J.nv + MT - 1) / MT;
    const unsigned nbt = (unsigned)(nb * (nb + 1) * (nb + 2) / 6);
    mix_body<TWO, false>(J.eps, J.tri, J.cubes, nullptr, nullptr, 0, 0, J.no, J.nv, (int)(local % nbt),
                  (int)(local / nbt));
    __syncthreads();
  }
}

template <int FM, int FN>
__global__ __launch_bounds__(WNT, shape_waves(FM, FN)) void k_pack_omega(
    const PackJob* __restrict__ jobs, int njobs, unsigned total) {
  for (unsigned item = blockIdx.x; item < total; item += gridDim.x) {
    const PackJob& J = jobs[pack_job(jobs, njobs, PK_OMEGA, item)];
    const unsigned local = item - J.first[PK_OMEGA];
    const int tm = (J.nv + 16 * FM - 1) / (16 * FM), tn = (J.nv + 16 * FN) / (16 * FN);
    const unsigned wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    omega_body<FM, FN>(J.cubes, J.Gbc, J.Gcb, J.tri, J.ntri, J.Pvv, J.no, J.nv, J.nch, tm, tn,
                       local * 4 + wave);
  }
}

template <int FNO>
__global__ __launch_bounds__(256) void k_pack_omega_oo(const PackJob* __restrict__ jobs, int njobs,
                                                       unsigned total) {
  for (unsigned item = blockIdx.x; item < total; item += gridDim.x) {
    const PackJob& J = jobs[pack_job(jobs, njobs, PK_OO, item)];
    const unsigned local = item - J.first[PK_OO];
    const int ta = (J.nv + 63) / 64;
    const unsigned gx = (unsigned)((J.nv + 1) / 2) * ta;
    omega_oo_body<FNO, 1, false, true>(J.cubes, J.Hs, J.tri, J.ntri, J.Ot2, J.OtT, J.no, J.nv, ta,
                       (int)(local % gx), (int)((local / gx) % J.no), (int)(local / (gx * J.no)));
    __syncthreads();
  }
}

__global__ __launch_bounds__(256) void k_pack_reduce(const PackJob* __restrict__ jobs, int njobs,
                                                     unsigned total) {
  for (unsigned item = blockIdx.x; item < total; item += gridDim.x) {
    const PackJob& J = jobs[pack_job(jobs, njobs, PK_RED, item)];
    const unsigned local = item - J.first[PK_RED];
    const unsigned gx = J.rgx;
    reduce_body(J.tri, J.ntri, J.Pvv, J.Ot1, J.Ot2, J.no, J.nv, J.nch, J.rslices,
                (int)(local % gx), (int)((local / gx) % (J.no + 1)), (int)(local / (gx * (J.no + 1))));
    __syncthreads();
  }
}

// The packed tile shapes for a member of nv: wave tiles (below NSHAPE) or, for the W build,
// NSHAPE plus the wavefronts of an LDS tile.
void pack_shapes(int prec, int nv, int* wshape, int* oshape) {
  *wshape = prec == CC3_FP64 || (prec == CC3_FP32 && fp32_wave_tiles(nv))
                ? wbuild_shape(prec, nv, true)
                : NSHAPE + (prec == CC3_FP32 ? 8 : lp_tile_waves(nv, nv));
  *oshape = pick_shape(nv, nv + 1, true);
}

void pack_items(PackJob& j, int prec, unsigned (&items)[PK_N]) {
  const int no = j.no, nv = j.nv, nt = j.ntri;
  items[PK_W] = prec == CC3_FP64 || (prec == CC3_FP32 && j.wshape < NSHAPE)
                    ? wbuild_wgs(nv, nt, j.wshape)
                    : wbuild_lp_wgs(prec, nv, nt, j.wshape - NSHAPE);
  const int nb = (nv + MT - 1) / MT;
  items[PK_MIX] = (unsigned)(nb * (nb + 1) * (nb + 2) / 6) * nt;
  items[PK_OMEGA] = omega_wgs(nv, nt, j.nch, j.oshape);
  items[PK_OO] = (unsigned)((nv + 1) / 2) * ((nv + 63) / 64) * no * 2u;
  const dim3 rg = reduce_grid(no, nv);
  j.rgx = rg.x;
  j.rslices = reduce_slices(no, nv);
  items[PK_RED] = rg.x * rg.y * rg.z;
}

// persistent grids: a few rounds of resident workgroups, never more than the items
static unsigned pack_grid(unsigned total, unsigned cap) { return total < cap ? total : cap; }

void launch_packed_step(const PackJob* dev_jobs, const PackJob* host_jobs, int njobs, int prec,
                        hipStream_t st) {
  if (njobs <= 0) return;
  unsigned total[PK_N] = {0, 0, 0, 0, 0};
  int max_no = 1;
  for (int r = 0; r < njobs; ++r) {
    PackJob j = host_jobs[r];
    unsigned it[PK_N];
    pack_items(j, prec, it);
    for (int k = 0; k < PK_N; ++k) total[k] += it[k];
    max_no = std::max(max_no, host_jobs[r].no);
  }
  const dim3 gmix(pack_grid(total[PK_MIX], 4096));
  if (host_jobs[0].wshape < NSHAPE) {
    const dim3 gw(pack_grid(total[PK_W], 4096));
    with_shape(host_jobs[0].wshape, [&](auto fm, auto fn) {
      constexpr int FM = decltype(fm)::value, FN = decltype(fn)::value;
      if constexpr (FM * FN != 20 && FM * FN != 10) {  // see pick_shape
        if (prec == CC3_FP64)
          hipLaunchKernelGGL((k_pack_wbuild<double, FM, FN>), gw, dim3(WNT), 0, st, dev_jobs, njobs,
                             total[PK_W]);
        else if constexpr (FM * FN <= 12)
          hipLaunchKernelGGL((k_pack_wbuild<float, FM, FN>), gw, dim3(WNT), 0, st, dev_jobs, njobs,
                             total[PK_W]);
      }
    });
  } else {
    launch_wbuild_lp_packed(dev_jobs, njobs, total[PK_W], prec, host_jobs[0].wshape - NSHAPE, st);
  }
  if (two_planes(prec))
    hipLaunchKernelGGL(k_pack_mix<true>, gmix, dim3(512), 0, st, dev_jobs, njobs, total[PK_MIX]);
  else
    hipLaunchKernelGGL(k_pack_mix<false>, gmix, dim3(512), 0, st, dev_jobs, njobs, total[PK_MIX]);
  with_shape(host_jobs[0].oshape, [&](auto fm, auto fn) {
    constexpr int FM = decltype(fm)::value, FN = decltype(fn)::value;
    if constexpr (FM * FN != 20 && FM * FN != 10)
      hipLaunchKernelGGL((k_pack_omega<FM, FN>), dim3(pack_grid(total[PK_OMEGA], 4096)), dim3(WNT),
                         0, st, dev_jobs, njobs, total[PK_OMEGA]);
  });
  const dim3 goo(pack_grid(total[PK_OO], 8192));
  if (max_no <= 16)
    hipLaunchKernelGGL(k_pack_omega_oo<1>, goo, dim3(256), 0, st, dev_jobs, njobs, total[PK_OO]);
  else if (max_no <= 32)
    hipLaunchKernelGGL(k_pack_omega_oo<2>, goo, dim3(256), 0, st, dev_jobs, njobs, total[PK_OO]);
  else if (max_no <= 48)
    hipLaunchKernelGGL(k_pack_omega_oo<3>, goo, dim3(256), 0, st, dev_jobs, njobs, total[PK_OO]);
  else
    hipLaunchKernelGGL(k_pack_omega_oo<4>, goo, dim3(256), 0, st, dev_jobs, njobs, total[PK_OO]);
  hipLaunchKernelGGL(k_pack_reduce, dim3(pack_grid(total[PK_RED], 16384)), dim3(256), 0, st,
                     dev_jobs, njobs, total[PK_RED]);
}

// FLOP of the dominant contractions and their companions, padding excluded.
double wbuild_flops(int no, int nv, const int* kinds, int n) {
  const double v = nv, o = no;
  const double term = 2.0 * v * v * v * v + 2.0 * v * v * v * o;
  double f = 0.0;
  for (int t = 0; t < n; ++t) f += (kinds[t] == TRI_DISTINCT ? 6.0 : 3.0) * term;
  return f;
}

// k_omega: the vv term (2 nv^4) and Omega1 (2 nv^3) per permutation
double omega_flops(int no, int nv, const int* kinds, int n) {
  const double v = nv;
  const double perm = 2.0 * v * v * v * v + 2.0 * v * v * v;
  double f = 0.0;
  for (int t = 0; t < n; ++t) f += (kinds[t] == TRI_DISTINCT ? 6.0 : 3.0) * perm;
  (void)no;
  return f;
}

// k_omega_oo: the oo and Fock terms (2 nv^3 no) per permutation
double omega_oo_flops(int no, int nv, const int* kinds, int n) {
  const double v = nv, o = no;
  double f = 0.0;
  for (int t = 0; t < n; ++t) f += (kinds[t] == TRI_DISTINCT ? 6.0 : 3.0) * 2.0 * v * v * v * o;
  return f;
}

}  // namespace cc3
