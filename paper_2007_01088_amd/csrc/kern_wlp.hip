// Low-precision W build (the t3-building contractions of Algorithm 1's first
// statement) on gfx950 MFMA, with FP32 accumulation:
//   CC3_FP32   : v_mfma_f32_16x16x4f32 on FP32 copies of the operands;
//   CC3_BF16X3 : v_mfma_f32_16x16x32_bf16 on a 2-piece split x = hi + lo,
//                products hi*hi + hi*lo + lo*hi;
//   CC3_BF16X6 : 3-piece split x = hi + mid + lo, products hi*hi + hi*mid +
//                mid*hi + hi*lo + mid*mid + lo*hi.
// FP32 and BF16x6 convert every 32-k partial sum and add it in FP64, BF16x3 each term
// after its whole K range; the planes are stored in FP64, so the
// permutation sum, the denominator division, the contravariant combination
// and the Omega accumulation downstream stay FP64.
//
// The operands are re-laid out once per call so that the contracted index is
// contiguous and zero-padded to a multiple of 32 (tiles load as 16-byte
// chunks into row-major LDS rows, and the K loop needs no bounds checks):
//   t2L [piece][p][q][x][dk]  = t2[p][q][x][d]
//   t2NL[piece][p][y][x][lk]  = -t2[p][l][x][y]
//   GwTL[piece][r][y][z][dk]  = Gw[r][y][z][d]   (= g_{ydzr})
//   GoTL[piece][q][r][z][lk]  = Go[q][r][z][l]   (= g_{lqzr})
#include <hip/hip_bf16.h>

#include "cc3.h"
#include "cc3_device.hpp"
#include "cc3_internal.hpp"
#include "cc3_wplanes.hpp"

namespace cc3 {

static inline unsigned nblk(int64_t n, int b) { return (unsigned)((n + b - 1) / b); }

typedef float f4v __attribute__((ext_vector_type(4)));
typedef __bf16 bf8v __attribute__((ext_vector_type(8)));
typedef unsigned u4v __attribute__((ext_vector_type(4)));  // a 16-byte chunk (kept in registers)

__host__ __device__ inline int kpad(int k) { return (k + 31) / 32 * 32; }

// ---------------------------------------------------------------------------
// Operand conversion: FP64 value -> pieces
// ---------------------------------------------------------------------------
// Generic re-layout: out[piece][outer][x][kk] (kk < K padded) from an FP64
// source element (outer, x, k) at src[outer * so + x * sx + k * sk] * sign; `slab`: elements
// of the copy between outer indices.
// `piece_stride` is the element distance between pieces of the whole array.
template <int MODE>  // 0: FP32, 2: BF16 2-piece, 3: BF16 3-piece
__global__ void k_lp_copy(const double* __restrict__ src, int64_t so, int64_t sx, int64_t sk,
                          double sign, int nouter, int nx, int K, int64_t slab,
                          void* __restrict__ dst, int64_t piece_stride) {
  const int Kp = kpad(K);
  const int64_t n = (int64_t)nouter * nx * Kp;
  const int64_t e = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (e >= n) return;
  const int kk = (int)(e % Kp);
  const int x = (int)((e / Kp) % nx);
  const int64_t o = e / ((int64_t)Kp * nx);
  const double v = (kk < K) ? sign * src[o * so + (int64_t)x * sx + (int64_t)kk * sk] : 0.0;
  const int64_t at = o * slab + (int64_t)x * Kp + kk;
  if constexpr (MODE == 0) {
    ((float*)dst)[at] = (float)v;
  } else {
    constexpr int P = MODE;
    uint16_t pc[P];
    split_bf16<P>(v, pc);
#pragma unroll
    for (int i = 0; i < P; ++i) ((uint16_t*)dst)[i * piece_stride + at] = pc[i];
  }
}

static int mode_of(int prec) { return prec == CC3_FP32 ? 0 : prec == CC3_BF16X3 ? 2 : 3; }

size_t lp_operand_bytes(int prec, int no, int nv) {
  if (prec == CC3_FP64) return 0;
  const size_t o = no, v = nv, dk = kpad(nv), lk = kpad(no);
  const size_t esz = prec == CC3_FP32 ? 4 : 2;
  const size_t gs = lp_slab(nv, nv, (int)esz), ns = lp_slab(nv, no, (int)esz);
  const size_t elems = o * o * v * dk + o * v * ns + o * v * gs + o * o * v * lk;
  const size_t pieces = prec == CC3_FP32 ? 1 : prec == CC3_BF16X3 ? 2 : 3;
  return elems * esz * pieces + 4 * 256;
}

void lp_operand_ptrs(int prec, int no, int nv, void* base, LpOperands& lp) {
  const size_t o = no, v = nv, dk = kpad(nv), lk = kpad(no);
  const size_t esz = prec == CC3_FP32 ? 4 : 2;
  const size_t pieces = prec == CC3_FP32 ? 1 : prec == CC3_BF16X3 ? 2 : 3;
  const size_t gs = lp_slab(nv, nv, (int)esz), ns = lp_slab(nv, no, (int)esz);
  auto al = [](size_t x) { return (x + 255) & ~(size_t)255; };
  char* b = (char*)base;
  lp.t2 = b;
  b += al(o * o * v * dk * esz * pieces);
  lp.t2N = b;
  b += al(o * v * ns * esz * pieces);
  lp.GwT = b;
  b += al(o * v * gs * esz * pieces);
  lp.GoT = b;
  lp.prec = prec;
}

template <int MODE>
static void lp_copy(const double* src, int64_t so, int64_t sx, int64_t sk, double sign, int nouter,
                    int nx, int K, int64_t slab, void* dst, int64_t piece_stride, hipStream_t st) {
  const int64_t n = (int64_t)nouter * nx * kpad(K);
  hipLaunchKernelGGL(k_lp_copy<MODE>, dim3(nblk(n, 256)), dim3(256), 0, st, src, so, sx, sk, sign,
                     nouter, nx, K, slab, dst, piece_stride);
}

void launch_lp_convert(const double* t2, const Blocks& b, int no, int nv, const LpOperands& lp,
                       hipStream_t st) {
  const int64_t v = nv, o = no, dk = kpad(nv), lk = kpad(no);
  auto run = [&](auto mode_tag) {
    constexpr int M = decltype(mode_tag)::value;
    constexpr int64_t esz = (M == 0 ? 4 : 2);
    const int64_t gs = lp_slab(nv, nv, (int)esz), ns = lp_slab(nv, no, (int)esz);
    // t2L[p][q][x][d] = t2[p][q][x][d]
    lp_copy<M>(t2, v * v, v, 1, 1.0, no * no, nv, nv, v * dk, lp.t2, o * o * v * dk, st);
    // t2NL[p][y][x][l] = -t2[p][l][x][y]: for each p, outer = y, x = x, k = l
    for (int p = 0; p < no; ++p)
      lp_copy<M>(t2 + (int64_t)p * o * v * v, 1, v, v * v, -1.0, nv, nv, no, ns,
                 (char*)lp.t2N + (size_t)p * v * ns * esz, o * v * ns, st);
    // GwTL[r][y][z][d] = Gw[r][y][z][d]: outer = (r, y), x = z, k = d
    lp_copy<M>(b.Gw, gw_pitch(nv), v, 1, 1.0, no * nv, nv, nv, gs, lp.GwT, o * v * gs,
               st);
    // GoTL[q][r][z][l] = Go[q][r][z][l]: outer = (q, r), x = z, k = l
    lp_copy<M>(b.Go, o * v, o, 1, 1.0, no * no, nv, no, v * lk, lp.GoT, o * o * v * lk, st);
  };
  const int m = mode_of(lp.prec);
  if (m == 0) run(std::integral_constant<int, 0>());
  else if (m == 2) run(std::integral_constant<int, 2>());
  else run(std::integral_constant<int, 3>());
}

// ---------------------------------------------------------------------------
// W build in low precision
// ---------------------------------------------------------------------------
// Tiles of 16 NW x 16 NW outputs on NW wavefronts (4 to 8), each FM x FN blocks of 16 x 16.
// The edge that costs least with its padding is taken (lp_tile_waves).
template <int NW>
struct LpGeo {
  static constexpr int WM = NW == 8 ? 4 : NW == 6 ? 3 : NW == 4 ? 2 : NW;
  static constexpr int WN = NW / WM, FM = NW / WM, FN = NW / WN;
  static constexpr int NT = 64 * NW, BM = 16 * NW;
  static_assert(WM * FM == NW && WN * FN == NW, "square tile");
};

// Engine traits.  FLUSH: each LDS stage (32 k) is accumulated in FP32 from zero
// and then added into an FP64 accumulator, so the FP32 rounding of the MFMA
// outputs applies to 32-term partial sums rather than to the running sum over
// the whole K range.  Used where the split is fine enough for that rounding to
// dominate the error (FP32 and the 3-piece BF16 split); the 2-piece split is
// limited by its operands and keeps one FP32 accumulator per term.
// MINW: waves per SIMD the W kernel is built for (4: two workgroups of 8 wavefronts per CU).
// ns: LDS stage buffers of the ring (ns - 1 stages of loads in flight): two where they let
// two workgroups share a CU (BF16x6 on 6 wavefronts, nv = 187: 70.4 -> 69.5 ms a call).
struct EngF32 {
  static constexpr int BK = 32, P = 1, NPROD = 1, ESZ = 4;
  static constexpr bool FLUSH = true;
  static constexpr int MINW = 4;
  static constexpr int ns(int) { return 2; }
};
template <int P_>
struct EngBF16 {
  static constexpr int BK = 32, P = P_, NPROD = (P_ == 2 ? 3 : 6), ESZ = 2;
  static constexpr bool FLUSH = (P_ == 3);
  static constexpr int MINW = (P_ == 2 ? 4 : 2);
  static constexpr int ns(int nw) { return P_ == 2 || nw <= 6 ? 2 : 3; }
};

// the piece pairs of the split products, in the order of their sum
__device__ inline void prod_pair(int P, int t, int& pa, int& pb) {
  if (P == 2) {
    const int a[3] = {0, 0, 1}, b[3] = {0, 1, 0};
    pa = a[t]; pb = b[t];
  } else {
    const int a[6] = {0, 0, 1, 0, 1, 2}, b[6] = {0, 1, 0, 2, 1, 0};
    pa = a[t]; pb = b[t];
  }
}

// ---------------------------------------------------------------------------
// The tile engine.  Operands are row-major (row, k) with k contiguous and
// zero-padded to a multiple of 32, in P pieces.  A stage holds 32 k of the
// A rows and B rows of the tile, every piece.  It goes from global memory to LDS
// directly: a buffer load with the LDS flag writes 16 bytes per lane at
// consecutive LDS addresses (1 KB per instruction), so the tile needs no
// staging registers and no LDS stores.  Each LDS row holds the RB bytes of one
// row and one stage as 16-byte chunks, XOR-swizzled by the row (lp_chunk) so
// that the 16 rows of one fragment read fall in different banks; the lane that
// fills LDS slot s loads the global chunk that the swizzle puts there.  A ring of NS
// stage buffers, one barrier per stage: the loads of stage s + NS - 1 are issued
// before the MFMAs of stage s.
// ---------------------------------------------------------------------------
template <class E, int NW>
struct LpTile : LpGeo<NW> {
  typedef LpGeo<NW> G;
  static constexpr int P = E::P, ESZ = E::ESZ;
  static constexpr int RB = E::BK * ESZ;         // bytes of one row in one stage
  static constexpr int CPR = RB / 16;            // 16-byte chunks per row (8 or 4)
  static constexpr int TILEB = G::BM * RB;       // one operand piece of one stage
  static constexpr int NI = RB / 64;             // loads per lane per operand piece
  static constexpr int STAGEB = 2 * P * TILEB;
  static constexpr int NS = E::ns(NW);               // stage buffers
  static constexpr int LPS = 2 * P * NI;         // direct loads per lane per stage
  static_assert(NI * G::NT * 16 == TILEB, "tile shape");
  static_assert(NS >= 2 && (NS - 2) * LPS <= 63, "vmcnt range");
};

// LDS chunk of logical chunk c of row `row` (an involution in c).  Both forms
// measured free of bank conflicts (SQ_LDS_BANK_CONFLICT = 0) for the fragment
// reads, 16 rows by one chunk column per lane group; XOR with (row >> 2) & 3
// for 64-byte rows, or no swizzle, gives two-way conflicts.
template <class E>
__device__ inline int lp_chunk(int row, int c) {
  if constexpr (E::BK * E::ESZ == 128) return c ^ ((row >> 1) & 7);
  else return c ^ ((row >> 1) & 3);
}

typedef __attribute__((address_space(3))) void* lds_ptr_t;

// One K segment of a product: piece-0 operand origins (row 0, k = 0), piece
// strides and row strides in bytes, and its number of stages.
struct LpSeg {
  const char *a, *b;
  int64_t aps, bps;
  unsigned ars, brs;
  int nst;
};

// The rows this lane loads: for load i of an operand piece, LDS slot
// s = (NW i + wave) 64 + lane holds row s / CPR and the swizzled chunk of s % CPR.
template <class E, int NW>
struct LpLanes {
  int row[LpTile<E, NW>::NI];
  unsigned cb[LpTile<E, NW>::NI];  // byte offset of the chunk within the row's stage
  __device__ LpLanes(int wave, int lane) {
    typedef LpTile<E, NW> L;
#pragma unroll
    for (int i = 0; i < L::NI; ++i) {
      const int s = (NW * i + wave) * 64 + lane;
      row[i] = s / L::CPR;
      cb[i] = (unsigned)lp_chunk<E>(row[i], s % L::CPR) * 16u;
    }
  }
};

// Issue the direct loads of one stage into the stage buffer `buf`: a, b, the operands'
// piece 0 at the stage, aps and bps their piece strides, ao(i), bo(i) this lane's byte offsets
template <class E, int NW, class A, class B>
__device__ __forceinline__ void lp_load_stage(const char* a, const char* b, int64_t aps,
                                              int64_t bps, char* buf, A ao, B bo, int wave) {
  typedef LpTile<E, NW> L;
#pragma unroll
  for (int pc = 0; pc < L::P; ++pc) {
    const BufRsrc ra = buf_rsrc(a + pc * aps), rb = buf_rsrc(b + pc * bps);
#pragma unroll
    for (int i = 0; i < L::NI; ++i) {
      char* la = buf + pc * L::TILEB + (NW * i + wave) * 1024;
      char* lb = buf + (L::P + pc) * L::TILEB + (NW * i + wave) * 1024;
      __builtin_amdgcn_raw_ptr_buffer_load_lds(ra, (lds_ptr_t)la, 16, ao(i), 0, 0, 0);
      __builtin_amdgcn_raw_ptr_buffer_load_lds(rb, (lds_ptr_t)lb, 16, bo(i), 0, 0, 0);
    }
  }
}

// The oldest stage in flight has reached LDS for every lane: this lane waits until at
// most `later` stages of its loads are outstanding (they return in order), then the
// workgroup barrier.  The barrier also ends every wave's reads of the previous stage,
// whose buffer the next loads overwrite.
template <int N>
__device__ __forceinline__ void lp_vmcnt() {
  asm volatile("s_waitcnt vmcnt(%0)" ::"n"(N) : "memory");
}
template <class E, int NW>
__device__ __forceinline__ void lp_stage_ready(int later) {
  typedef LpTile<E, NW> L;
  if constexpr (L::NS >= 3) {
    if (later >= 1) {
      if constexpr (L::NS >= 4) {
        if (later >= 2) {
          lp_vmcnt<2 * L::LPS>();
          __syncthreads();
          return;
        }
      }
      lp_vmcnt<L::LPS>();
      __syncthreads();
      return;
    }
  }
  lp_vmcnt<0>();
  __syncthreads();
}

// acc += A B over one LDS stage.  BF16: one k = 32 MFMA per product; lane
// supplies A[m = l%16][k = 8 (l/16) .. + 7] (chunk l/16 of its row).  FP32: the
// lane reads chunk 4 h + l/16 (four consecutive k) of its row and supplies its
// element j to the k-step (h, j) of the 16x16x4 MFMA; A and B use the same k
// assignment, so the eight k-steps cover the stage's 32 k once each.
// SWAP: A and B change places in the order of the piece products.
template <class E, int NW, bool SWAP = false>
__device__ __forceinline__ void lp_mfma_stage(const char* buf,
                                              f4v (&acc)[LpGeo<NW>::FM][LpGeo<NW>::FN], int lane,
                                              int wm, int wn) {
  typedef LpTile<E, NW> L;
  constexpr int LFM = L::FM, LFN = L::FN;
  const int g = lane >> 4, r16 = lane & 15;
  // Fragment rows are 16 R + r16, and lp_chunk's XOR depends on bits 1-3 of the row
  // only, that is on r16: the lane's byte offset within a fragment's rows is one value
  // per chunk column, and the fragment's own offset (16 R RB) is a constant.
  auto lane_off = [&](int c) __attribute__((always_inline)) {
    return r16 * L::RB + lp_chunk<E>(r16, c) * 16;
  };
  const char* ab = buf + wm * LFM * 16 * L::RB;             // this wave's A rows
  const char* bb = buf + L::P * L::TILEB + wn * LFN * 16 * L::RB;  // and B rows
  if constexpr (E::P == 1) {
#pragma unroll
    for (int h = 0; h < 2; ++h) {
      const int lo = lane_off(4 * h + g);
      f4v a[LFM];
#pragma unroll
      for (int fm = 0; fm < LFM; ++fm) a[fm] = *(const f4v*)(ab + fm * 16 * L::RB + lo);
      // one B fragment at a time (registers: the FP64 accumulator of FLUSH is large)
#pragma unroll
      for (int fn = 0; fn < LFN; ++fn) {
        const f4v b = *(const f4v*)(bb + fn * 16 * L::RB + lo);
#pragma unroll
        for (int j = 0; j < 4; ++j)
#pragma unroll
          for (int fm = 0; fm < LFM; ++fm)
            acc[fm][fn] = __builtin_amdgcn_mfma_f32_16x16x4f32(a[fm][j], b[j], acc[fm][fn], 0, 0, 0);
      }
    }
  } else {
    const int lo = lane_off(g);
    bf8v a[L::P][LFM], b[L::P][LFN];
#pragma unroll
    for (int pc = 0; pc < L::P; ++pc) {
#pragma unroll
      for (int fm = 0; fm < LFM; ++fm)
        a[pc][fm] = *(const bf8v*)(ab + pc * L::TILEB + fm * 16 * L::RB + lo);
#pragma unroll
      for (int fn = 0; fn < LFN; ++fn)
        b[pc][fn] = *(const bf8v*)(bb + pc * L::TILEB + fn * 16 * L::RB + lo);
    }
#pragma unroll
    for (int t = 0; t < E::NPROD; ++t) {
      int pa, pb;
      if constexpr (SWAP) prod_pair(L::P, t, pb, pa);
      else prod_pair(L::P, t, pa, pb);
#pragma unroll
      for (int fm = 0; fm < LFM; ++fm)
#pragma unroll
        for (int fn = 0; fn < LFN; ++fn)
          acc[fm][fn] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(a[pa][fm], b[pb][fn], acc[fm][fn], 0, 0, 0);
    }
  }
}

template <int FM, int FN>
__device__ __forceinline__ void lp_zero(f4v (&acc)[FM][FN]) {
#pragma unroll
  for (int fm = 0; fm < FM; ++fm)
#pragma unroll
    for (int fn = 0; fn < FN; ++fn) acc[fm][fn] = f4v{0.f, 0.f, 0.f, 0.f};
}
template <int FM, int FN>
__device__ __forceinline__ void lp_flush(f4v (&acc)[FM][FN], d4v (&accd)[FM][FN]) {
#pragma unroll
  for (int fm = 0; fm < FM; ++fm)
#pragma unroll
    for (int fn = 0; fn < FN; ++fn) {
#pragma unroll
      for (int r = 0; r < 4; ++r) accd[fm][fn][r] += (double)acc[fm][fn][r];
      acc[fm][fn] = f4v{0.f, 0.f, 0.f, 0.f};
    }
}

// ---------------------------------------------------------------------------
// W build in low precision
// ---------------------------------------------------------------------------
// One workgroup per (triple, plane, y, tile).  Bound by the MFMAs (BF16x6: 0.76 of 1.34
// PFLOP/s at nv = 187) and, BF16x3, by the planes that it stores (at nv = 210 8 triples are
// 1.8 GB, 0.41 of the 1.0 ms).  FP32 and BF16x6 add every stage into FP64, so
// the order of their segments is free and they build the two planes of the FP64 form; the
// running FP32 sum of BF16x3 goes over the d sum and then the l sum of a term, which keeps
// those together and needs the three planes.  (Segments: cc3_wplanes.hpp.)  The pieces of a
// product are paired in one order per permutation in both (wseg_swap), so the FP32 sums of a
// stage do not depend on the planes.
template <class E, int NW>
__device__ __forceinline__ void wbuild_lp_body(
    const char* __restrict__ t2L, const char* __restrict__ t2NL, const char* __restrict__ GwTL,
    const char* __restrict__ GoTL, const int* __restrict__ tri, double* __restrict__ cubes, int no,
    int nv, int tiles, int all_terms, int bx, int by, int bz) {
  typedef LpTile<E, NW> L;
  constexpr int ESZ = E::ESZ, FM = L::FM, FN = L::FN;
  constexpr bool TWO = E::FLUSH;
  __shared__ __attribute__((aligned(16))) char lds[L::NS * L::STAGEB];
  const int y = bx / (tiles * tiles);
  const int tile = bx % (tiles * tiles);
  const int m0 = (tile / tiles) * L::BM, n0 = (tile % tiles) * L::BM;
  const int plane = by;
  const int z = bz;
  const int i = tri[3 * z], j = tri[3 * z + 1], k = tri[3 * z + 2];
  const int kind = all_terms ? TRI_DISTINCT : tri_kind(i, j, k);
  if (TWO ? kind != TRI_DISTINCT && plane == 1
          : (kind == TRI_IJ && plane == 1) || (kind == TRI_JK && plane == 2))
    return;
  const bool two = kind == TRI_DISTINCT || plane == 0;  // three planes: both terms
  const uint64_t segs = TWO ? wplane_segs(plane, kind) : kSegs3[plane];
  const int64_t dk = kpad(nv), lk = kpad(no), v = nv, o = no;
  const int64_t gy = lp_slab(nv, nv, ESZ), ty = lp_slab(nv, no, ESZ);
  const int sv = (int)(dk / 32), so = (int)(lk / 32);  // stages of a d sum and of an l sum
  int nsteps;
  if (TWO) nsteps = wplane_dsums(plane, kind) * sv + 3 * so;
  else nsteps = (two ? 2 : 1) * (sv + so);
  // the segment being loaded and its next stage
  LpSeg sg;
  int seg = 0, st = 0;
  auto open = [&](int s) {
    const int code = (int)(segs >> (6 * s)) & 63;
    const bool lsum = code & 8, col = code & 16, strided = code & 32;
    int p, q, r;
    perm_pqr(code & 7, i, j, k, p, q, r);
    const char *amp, *in;
    int64_t ap, ip;   // piece strides (bytes)
    unsigned ar, ir;  // row strides (bytes)
    if (!lsum) {
      amp = t2L + (p * o + q) * v * dk * ESZ;
      ap = o * o * v * dk * ESZ;
      ar = (unsigned)(dk * ESZ);
      in = GwTL + (r * v * gy + (strided ? y * dk : y * gy)) * ESZ;
      ip = o * v * gy * ESZ;
      ir = (unsigned)((strided ? gy : dk) * ESZ);
      sg.nst = sv;
    } else {
      amp = t2NL + (p * v * ty + (strided ? y * lk : y * ty)) * ESZ;
      ap = o * v * ty * ESZ;
      ar = (unsigned)((strided ? ty : lk) * ESZ);
      in = GoTL + (q * o + r) * v * lk * ESZ;
      ip = o * o * v * lk * ESZ;
      ir = (unsigned)(lk * ESZ);
      sg.nst = so;
    }
    sg.aps = col ? ip : ap;
    sg.bps = col ? ap : ip;
    sg.ars = col ? ir : ar;
    sg.brs = col ? ar : ir;
    // the tile's first rows: the lanes' offsets from them stay below 2 GiB at every nv (a row
    // stride of one slab is 4 nv^2 bytes)
    sg.a = (col ? in : amp) + (int64_t)m0 * sg.ars;
    sg.b = (col ? amp : in) + (int64_t)n0 * sg.brs;
    st = 0;
  };

  const int tid = threadIdx.x;
  const int lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int wm = wave % L::WM, wn = wave / L::WM;
  const LpLanes<E, NW> ln(wave, lane);
  // rows past nv repeat row nv - 1 (their outputs are never stored)
  int ar[L::NI], br[L::NI];
#pragma unroll
  for (int e = 0; e < L::NI; ++e) {
    ar[e] = min(ln.row[e], nv - 1 - m0);
    br[e] = min(ln.row[e], nv - 1 - n0);
  }
  auto load = [&](int t) {  // stage t of the plane, in order
    const int64_t ko = (int64_t)st * L::RB;
    lp_load_stage<E, NW>(
        sg.a + ko, sg.b + ko, sg.aps, sg.bps, lds + (t % L::NS) * L::STAGEB,
        [&](int e) { return (unsigned)ar[e] * sg.ars + ln.cb[e]; },
        [&](int e) { return (unsigned)br[e] * sg.brs + ln.cb[e]; }, wave);
    if (++st == sg.nst && t + 1 < nsteps) open(++seg);
  };
  f4v acc1[FM][FN], acc2[FM][FN];
  d4v accd[FM][FN];
  lp_zero(acc1);
  lp_zero(acc2);
#pragma unroll
  for (int fm = 0; fm < FM; ++fm)
#pragma unroll
    for (int fn = 0; fn < FN; ++fn) accd[fm][fn] = d4v{0.0, 0.0, 0.0, 0.0};
  // stages [sb, se) into acc (with FLUSH into accd), the loads NS - 1 stages ahead
  auto run = [&](auto swap, int sb, int se, f4v (&acc)[FM][FN]) __attribute__((always_inline)) {
    for (int s = sb; s < se; ++s) {
      lp_stage_ready<E, NW>(min(L::NS - 2, nsteps - 1 - s));
      if (s + L::NS - 1 < nsteps) load(s + L::NS - 1);
      lp_mfma_stage<E, NW, decltype(swap)::value>(lds + (s % L::NS) * L::STAGEB, acc, lane, wm, wn);
      if constexpr (E::FLUSH) lp_flush(acc, accd);
    }
  };
  open(0);
#pragma unroll
  for (int t = 0; t < L::NS - 1; ++t)
    if (t < nsteps) load(t);
  if constexpr (!TWO) {  // term 1, then term 2 in an accumulator of its own
    run(std::false_type(), 0, sv + so, acc1);
    if (two) run(std::false_type(), sv + so, nsteps, acc2);
  } else if constexpr (L::P == 1) {
    run(std::false_type(), 0, nsteps, acc1);
  } else {
    const int nd = wplane_dsums(plane, kind);
    for (int g = 0, s = 0; g < nd + 3; ++g) {
      const int se = s + (g < nd ? sv : so);
      if (wseg_swap((int)(segs >> (6 * g)) & 63, kind)) run(std::true_type(), s, se, acc1);
      else run(std::false_type(), s, se, acc1);
      s = se;
    }
  }

  // the FP32/BF16 MFMA leaves D[row = 4 (lane/16) + r][col = lane%16] in register r
  const int64_t rp = cube_pitch(nv);
  double* dst = cubes + ((int64_t)z * NSLOT + plane) * cube_slot(nv) + (int64_t)y * nv * rp;
#pragma unroll
  for (int fm = 0; fm < FM; ++fm)
#pragma unroll
    for (int fn = 0; fn < FN; ++fn)
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        const int m = m0 + (wm * FM + fm) * 16 + 4 * (lane >> 4) + r;
        const int n = n0 + (wn * FN + fn) * 16 + (lane & 15);
        if (m < nv && n < nv)
          dst[(int64_t)m * rp + n] = accd[fm][fn][r] + ((double)acc1[fm][fn][r] + (double)acc2[fm][fn][r]);
      }
}

template <class E, int NW>
__global__ __launch_bounds__(LpGeo<NW>::NT, E::MINW) void k_wbuild_lp(
    const char* __restrict__ t2L, const char* __restrict__ t2NL, const char* __restrict__ GwTL,
    const char* __restrict__ GoTL, const int* __restrict__ tri, double* __restrict__ cubes, int no,
    int nv, int tiles, int all_terms) {
  wbuild_lp_body<E, NW>(t2L, t2NL, GwTL, GoTL, tri, cubes, no, nv, tiles, all_terms, blockIdx.x,
                        blockIdx.y, blockIdx.z);
}

// Wavefronts (tile edge 16 NW) that cover an M x N product with the least work: the outputs
// computed, padding included, weighted by the time per output of the W build's launches relative
// to NW = 8 (nv = 150 to 900: 4 1.4 to 2.3, 5 1.4 to 1.7, 6 1.4 to 1.7, 7 1.1 to 1.3).
// MEASURED, whole calls of 9 occupied orbitals at NW = 4 / 5 / 6 / 7 / 8 (the rule's choice
// is the fastest in each): BF16x6, nv = 112: 13.1 / 16.0 / 16.9 / 12.1 / 12.3 ms, 150: 38.8 /
// 37.0 / 38.6 / 40.9 / 42.2, 187: 72.6 / 85.0 / 69.5 / 72.7 / 75.3, 240: 177 / 184 / 187 / 198 /
// 168; BF16x3, 150: 36.1 / 33.7 / 34.5 / 35.8 / 36.1, 180: 62.9 / 64.6 / 59.8 / 61.4 / 63.0,
// 210: 123 / 120 / 122 / 116 / 116.  The W build of 8 triples in BF16x3 and x6: 400 12.3 / 10.0 /
// 10.6 / 9.2 / 10.3 and 24.0 / 19.1 / 19.5 / 15.8 / 17.4, 450 14.9 / 13.2 / 12.7 / 13.4 / 10.4 and
// 22.9 / 26.6 / 22.0 / 23.8 / 18.3; of one, 900: 35.6 / 22.5 / 21.6 / 22.8 / 17.3 and 65.2 / 44.7 /
// 37.5 / 36.1 / 32.6.  Instead, 128 x 128 tiles whose empty blocks are skipped: 73.7 ms for
// BF16x6 at 187, and the same as 7 wavefronts for BF16x3 at 210.
int lp_tile_waves(int64_t M, int64_t N) {
  constexpr double weight[] = {1.5, 1.6, 1.42, 1.2, 1.0};  // NW = 4 to 8
  int best = 8;
  double cost = 0.0;
  for (int nw = 8; nw >= 4; --nw) {
    const double t = 16.0 * nw;
    const double c = (double)nblk(M, 16 * nw) * nblk(N, 16 * nw) * t * t * weight[nw - 4];
    if (nw == 8 || c < cost) { best = nw; cost = c; }
  }
  return best;
}

// Calls f with the tile's wavefront count as an integral constant.
template <class F>
static void with_waves(int nw, F f) {
  if (nw == 4) f(std::integral_constant<int, 4>());
  else if (nw == 5) f(std::integral_constant<int, 5>());
  else if (nw == 6) f(std::integral_constant<int, 6>());
  else if (nw == 7) f(std::integral_constant<int, 7>());
  else f(std::integral_constant<int, 8>());
}

// ---------------------------------------------------------------------------
// Mixed-all Omega contraction (the vv term and Omega1) on split-BF16 MFMA
// ---------------------------------------------------------------------------
// The long-K GEMM of k_omega per (triple, permutation, 128 x 128 tile, K chunk):
//   Pvv[z][pi][chunk][a][n] = sum_{kk in chunk} Y_v(pi)[a][kk] G[r][n'][kk],
// with K = (x, y) in 8 x 8 blocks (lp_kb), so that a stage is half a block: four x, eight
// consecutive y each.  The six permutations need four views of tau~: rows a with
// K = (b, c) (pi 0), b with (a, c) (1, 4), c with (a, b) (2, 5) and a with (c, b) (3); the two
// forms of YL (yl_piece) hold all four, the rows being their first or second index.  B:
//   GL[piece][r][n'][kk]: Gbc (or Gcb for pi 2, 4) rows, n' = n for n < nv and
//     nv + q (the Omega1 row) for n >= nv.
// Against one k-major copy per view, written value by value: the mix of 8 triples of nv = 210
// 1.21 -> 0.84 ms (40 B per element at 3.5 TB/s), this kernel 0.85 -> 0.78 (its MFMAs at 0.72
// PFLOP/s: one barrier per stage and the loads behind it, not the 32 KB that a stage moves).
// Each chunk sums in FP32 on the MFMA (with FLUSH, stage by stage into FP64);
// k_reduce sums the chunks in FP64.  The tile engine is that of k_wbuild_lp.
template <class E, int NW>
__global__ __launch_bounds__(LpGeo<NW>::NT) void k_omega_lp(const char* __restrict__ YL,
                                                            const char* __restrict__ GbcL,
                                                            const char* __restrict__ GcbL,
                                                            const int* __restrict__ tri,
                                                            double* __restrict__ Pvv, int no,
                                                            int nv, int nchunks, int tiles_n) {
  typedef LpTile<E, NW> L;
  constexpr int ESZ = E::ESZ, LFM = L::FM, LFN = L::FN, LBM = L::BM, LBN = L::BM, LWM = L::WM;
  __shared__ __attribute__((aligned(16))) char lds[L::NS * L::STAGEB];
  const int pi = blockIdx.y, z = blockIdx.z;
  const int i = tri[3 * z], j = tri[3 * z + 1], k = tri[3 * z + 2];
  if (!perm_active(tri_kind(i, j, k), pi)) return;
  int p, q, r;
  perm_pqr(pi, i, j, k, p, q, r);
  const int ch = blockIdx.x % nchunks, tile = blockIdx.x / nchunks;
  const int m0 = (tile / tiles_n) * LBM, n0 = (tile % tiles_n) * LBN;
  const int S = (int)(lp_kb_len(nv) / E::BK);
  const int s0 = (int)((int64_t)ch * S / nchunks), s1 = (int)((int64_t)(ch + 1) * S / nchunks);
  if (s0 >= s1) return;
  const int form = pi == 2 || pi == 3 || pi == 5;
  const bool second = pi != 0 && pi != 3;  // rows: the form's second index
  const bool cb = (pi == 2 || pi == 4);
  const unsigned nb = (unsigned)(nv + 7) / 8;
  const unsigned rs = (unsigned)(lp_kb_pitch(nv) * ESZ);         // row stride of GL, bytes
  const int64_t y_ps = yl_piece(nv), g_ps = (int64_t)no * (nv + no) * rs;  // piece strides
  // from the tile's first rows, as in the W build (m0 is a multiple of 8)
  const int64_t m8 = (int64_t)(m0 >> 3) * nb * 1024;
  const char* ga = YL + ((int64_t)z * 2 + form) * E::P * y_ps + (second ? m8 : m8 * nb);
  const char* gb = (cb ? GcbL : GbcL) + ((int64_t)r * (nv + no) + n0) * rs;

  const int tid = threadIdx.x;
  const int lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int wm = wave % LWM, wn = wave / LWM;
  const LpLanes<E, NW> ln(wave, lane);
  // rows past nv repeat row nv - 1 (outputs never stored); B rows n >= nv read the
  // Omega1 row nv + q
  unsigned ao[L::NI], bo[L::NI];
#pragma unroll
  for (int e = 0; e < L::NI; ++e) {
    const unsigned m = (unsigned)min(ln.row[e], nv - 1 - m0);
    ao[e] = second ? (m >> 3) * nb * 1024 + (m & 7) * 16 + ln.cb[e] * 8
                   : (m >> 3) * nb * nb * 1024 + (m & 7) * 128 + ln.cb[e];
    bo[e] = (unsigned)(n0 + ln.row[e] < nv ? ln.row[e] : nv + q - n0) * rs + ln.cb[e];
  }
  f4v acc[LFM][LFN];
  d4v accd[LFM][LFN];  // FLUSH: each stage's FP32 sum added in FP64
  lp_zero(acc);
#pragma unroll
  for (int fm = 0; fm < LFM; ++fm)
#pragma unroll
    for (int fn = 0; fn < LFN; ++fn) accd[fm][fn] = d4v{0.0, 0.0, 0.0, 0.0};
  // the loads run NS - 1 stages ahead in the ring of NS stage buffers
  auto load = [&](int t) {
    const unsigned blk = (unsigned)(s0 + t) >> 1, half = (unsigned)(s0 + t) & 1;  // of K
    const int64_t ko = second ? ((int64_t)(blk / nb) * nb * nb + blk % nb) * 1024 + half * 512
                              : (int64_t)blk * 1024 + half * 64;
    lp_load_stage<E, NW>(
        ga + ko, gb + (int64_t)(s0 + t) * L::RB, y_ps, g_ps, lds + (t % L::NS) * L::STAGEB,
        [&](int e) { return ao[e]; }, [&](int e) { return bo[e]; }, wave);
  };
#pragma unroll
  for (int t = 0; t < L::NS - 1; ++t)
    if (s0 + t < s1) load(t);
  for (int s = s0; s < s1; ++s) {
    lp_stage_ready<E, NW>(min(L::NS - 2, s1 - 1 - s));
    const int ahead = s - s0 + L::NS - 1;
    if (s0 + ahead < s1) load(ahead);
    lp_mfma_stage<E, NW>(lds + ((s - s0) % L::NS) * L::STAGEB, acc, lane, wm, wn);
    if constexpr (E::FLUSH) lp_flush(acc, accd);
  }
  // the BF16 MFMA leaves D[row = 4 (lane/16) + r][col = lane%16] in register r
  const int NV1 = nv + 1;
  double* pvv = Pvv + (((int64_t)z * 6 + pi) * nchunks + ch) * (int64_t)nv * NV1;
#pragma unroll
  for (int fm = 0; fm < LFM; ++fm)
#pragma unroll
    for (int fn = 0; fn < LFN; ++fn)
#pragma unroll
      for (int rr = 0; rr < 4; ++rr) {
        const int a = m0 + (wm * LFM + fm) * 16 + 4 * (lane >> 4) + rr;
        const int n = n0 + (wn * LFN + fn) * 16 + (lane & 15);
        if (a < nv && n <= nv) pvv[(int64_t)a * NV1 + n] = accd[fm][fn][rr] + (double)acc[fm][fn][rr];
      }
}

size_t lp_contract_g_bytes(int prec, int no, int nv) {
  const int P = prec == CC3_BF16X3 ? 2 : 3;
  return (size_t)P * no * (nv + no) * (size_t)lp_kb_pitch(nv) * 2;  // one of Gbc, Gcb
}
size_t lp_contract_cube_bytes(int prec, int nv) {
  const int P = prec == CC3_BF16X3 ? 2 : 3;
  return (size_t)2 * P * (size_t)yl_piece(nv);  // per triple
}

// Split-BF16 pieces of the rows of Gbc or Gcb with K = (x, y) (padded rows in the source)
// in the blocked order lp_kb: dst[piece][row][kb] at row pitch lp_kb_pitch, zero where x
// or y is past nv (the pitch's tail is never read).
template <int P>
__global__ void k_lp_copy_blocked(const double* __restrict__ src, int64_t rows, int nv,
                                  uint16_t* __restrict__ dst, int64_t piece_stride) {
  const int64_t Kb = lp_kb_len(nv), Kr = lp_kb_pitch(nv), gp = g_pitch(nv);
  const int rp = cube_pitch(nv);
  const int nb = (nv + 7) / 8;
  const int64_t e = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (e >= rows * Kb) return;
  const int64_t row = e / Kb;
  const int kb = (int)(e % Kb);
  const int blk = kb >> 6, x = (blk / nb) * 8 + ((kb >> 3) & 7), y = (blk % nb) * 8 + (kb & 7);
  const double v = (x < nv && y < nv) ? src[row * gp + (int64_t)x * rp + y] : 0.0;
  uint16_t pc[P];
  split_bf16<P>(v, pc);
#pragma unroll
  for (int i = 0; i < P; ++i) dst[i * piece_stride + row * Kr + kb] = pc[i];
}

void launch_lp_contract_convert(const Blocks& b, int prec, int no, int nv, void* GbcL, void* GcbL,
                                hipStream_t st) {
  const int64_t rows = (int64_t)no * (nv + no), n = rows * lp_kb_len(nv);
  const int64_t ps = rows * lp_kb_pitch(nv);  // piece stride (elements)
  const unsigned g = nblk(n, 256);
  if (prec == CC3_BF16X3) {
    hipLaunchKernelGGL(k_lp_copy_blocked<2>, dim3(g), dim3(256), 0, st, b.Gbc, rows, nv,
                       (uint16_t*)GbcL, ps);
    hipLaunchKernelGGL(k_lp_copy_blocked<2>, dim3(g), dim3(256), 0, st, b.Gcb, rows, nv,
                       (uint16_t*)GcbL, ps);
  } else {
    hipLaunchKernelGGL(k_lp_copy_blocked<3>, dim3(g), dim3(256), 0, st, b.Gbc, rows, nv,
                       (uint16_t*)GbcL, ps);
    hipLaunchKernelGGL(k_lp_copy_blocked<3>, dim3(g), dim3(256), 0, st, b.Gcb, rows, nv,
                       (uint16_t*)GcbL, ps);
  }
}

void launch_omega_lp(int prec, const void* YL, const void* GbcL, const void* GcbL, const int* tri,
                     int ntri, double* Pvv, int no, int nv, hipStream_t st) {
  const int nch = omega_kchunks(nv, ntri, true);
  const char *y = (const char*)YL, *gb = (const char*)GbcL, *gc = (const char*)GcbL;
  with_waves(lp_tile_waves(nv, nv + 1), [&](auto nw) {
    constexpr int NW = decltype(nw)::value;
    const int tm = (int)nblk(nv, 16 * NW), tn = (int)nblk(nv + 1, 16 * NW);
    const dim3 grid(nch * tm * tn, 6, ntri), block(64 * NW);
    if (prec == CC3_BF16X3)
      hipLaunchKernelGGL((k_omega_lp<EngBF16<2>, NW>), grid, block, 0, st, y, gb, gc, tri, Pvv, no, nv,
                         nch, tn);
    else
      hipLaunchKernelGGL((k_omega_lp<EngBF16<3>, NW>), grid, block, 0, st, y, gb, gc, tri, Pvv, no, nv,
                         nch, tn);
  });
}

// Packed persistent form of the W build (serving), as k_pack_wbuild.
template <class E, int NW>
__global__ __launch_bounds__(LpGeo<NW>::NT) void k_pack_wbuild_lp(const PackJob* __restrict__ jobs,
                                                                  int njobs, unsigned total) {
  constexpr unsigned planes = E::FLUSH ? 2u : 3u;
  for (unsigned item = blockIdx.x; item < total; item += gridDim.x) {
    int r = 0;
    while (r + 1 < njobs && item >= jobs[r + 1].first[PK_W]) ++r;
    const PackJob& J = jobs[r];
    const unsigned local = item - J.first[PK_W];
    const int t = (J.nv + 16 * NW - 1) / (16 * NW);
    const unsigned gx = (unsigned)J.nv * t * t;
    wbuild_lp_body<E, NW>((const char*)J.lpt2, (const char*)J.lpt2N, (const char*)J.lpGwT,
                          (const char*)J.lpGoT, J.tri, J.cubes, J.no, J.nv, t, 0,
                          (int)(local % gx), (int)((local / gx) % planes),
                          (int)(local / (gx * planes)));
    __syncthreads();
  }
}

unsigned wbuild_lp_wgs(int prec, int nv, int ntri, int nw) {
  const unsigned t = nblk(nv, 16 * nw);
  return (unsigned)nv * t * t * (two_planes(prec) ? 2u : 3u) * (unsigned)ntri;
}

void launch_wbuild_lp_packed(const PackJob* jobs, int njobs, unsigned total, int prec, int nw,
                             hipStream_t st) {
  const dim3 grid(total < 2048 ? total : 2048);
  if (prec == CC3_FP32) {
    hipLaunchKernelGGL((k_pack_wbuild_lp<EngF32, 8>), grid, dim3(512), 0, st, jobs, njobs, total);
    return;
  }
  with_waves(nw, [&](auto n) {
    constexpr int NW = decltype(n)::value;
    if (prec == CC3_BF16X3)
      hipLaunchKernelGGL((k_pack_wbuild_lp<EngBF16<2>, NW>), grid, dim3(64 * NW), 0, st, jobs, njobs,
                         total);
    else
      hipLaunchKernelGGL((k_pack_wbuild_lp<EngBF16<3>, NW>), grid, dim3(64 * NW), 0, st, jobs, njobs,
                         total);
  });
}

void launch_wbuild_lp(const LpOperands& lp, const int* tri, int ntri, double* cubes, int no, int nv,
                      bool all_terms, hipStream_t st) {
  const char *a = (const char*)lp.t2, *b = (const char*)lp.t2N, *c = (const char*)lp.GwT,
             *d = (const char*)lp.GoT;
  const int at = all_terms ? 1 : 0;
  const unsigned planes = two_planes(lp.prec) ? 2 : 3;
  if (lp.prec == CC3_FP32) {
    const int t = (int)nblk(nv, 128);
    hipLaunchKernelGGL((k_wbuild_lp<EngF32, 8>), dim3(nv * t * t, planes, ntri), dim3(512), 0, st, a, b,
                       c, d, tri, cubes, no, nv, t, at);
    return;
  }
  with_waves(lp_tile_waves(nv, nv), [&](auto n) {
    constexpr int NW = decltype(n)::value;
    const int t = (int)nblk(nv, 16 * NW);
    const dim3 grid(nv * t * t, planes, ntri), block(64 * NW);
    if (lp.prec == CC3_BF16X3)
      hipLaunchKernelGGL((k_wbuild_lp<EngBF16<2>, NW>), grid, block, 0, st, a, b, c, d, tri, cubes, no,
                         nv, t, at);
    else
      hipLaunchKernelGGL((k_wbuild_lp<EngBF16<3>, NW>), grid, block, 0, st, a, b, c, d, tri, cubes, no,
                         nv, t, at);
  });
}

}  // namespace cc3
