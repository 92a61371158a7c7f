// Contractions of the transition-density loop (Algorithm 3, the triples
// contributions to D^{m,0}) on gfx950, after the t3 and L3 builds and their mix.
//
// The cubes of a batch of triples are tau_t and L~_t (t3 and the contravariant
// left-state triples), [a][b][c] of the triple's own order (i, j, k), rows at the padded
// pitch with zeros in the padding.  Every unordered triple i >= j >= k, not all equal,
// contributes once, with all six formal orderings (p,q,r) of (i,j,k) at weight 1, or 1/2
// with two equal indices (each distinct ordering then appears twice):
//   D_cd[c][d]      += 1/2 sum_ab L~_{pqr}[a,b,c] tau_{pqr}[a,b,d]
//   Y^o[c][l][p][r] += sum_ab L~_{pqr}[a,b,c] t2[l][q][a][b]
//   D_kc[r][c]      += sum_ab l2[p][q][a][b] tau~_{pqr}[a,b,c]
// The orderings pair up into three mode contractions, one per cube axis m holding the
// free index, K = (x, y) over the other two axes u < v.  With s, U, V the occupied indices
// of the axes m, u, v:
//   D_cd: sum over modes of G_m[c][d] = sum_K L~ tau with c, d on axis m;
//   Y^o:  p = U, q = V: columns l of t2[l][V][x][y]; p = V, q = U: columns l of
//         t2[l][U][y][x] = t2[U][l][x][y]; both to r = s;
//   D_kc: with tau~ written out in permuted tau and E[p][q][x][y] = 2 l2[p][q][x][y]
//         - l2[p][q][y][x] (which has the pair symmetry of l2), mode m of tau gives
//         r = s: 4 E[U][V], r = V: -2 E[U][s], r = U: -2 E[s][V], each [x][y]
//         contracted with tau over K; tau~ is not needed as a cube.
// The occupied-occupied block, for which the paper runs a loop over virtual triples, is
// D_lk = -1/2 sum_{ij} sum_{abc} L~^{abc}_{ijk} tau^{abc}_{ijl}; per pair it is the Gram
// matrix M_ij[k][l] = <L~_{ijk}, tau_{ijl}>, and M_ji = M_ij (the simultaneous relabelling
// of (a,i) and (b,j)), so D_lk -= 1/2 w_ij M_ij with w_ij = 2 for i > j, 1 for i == j.
// After the loop  D_ld = - sum_{cik} Y^o[c][l][i][k] t2[k][i][c][d].
// Every contraction goes to partial slabs reduced in a fixed order (no atomics).
#include "cc3_density.hpp"
#include "cc3_device.hpp"

namespace cc3 {

static inline unsigned nblk(int64_t n, int b) { return (unsigned)((n + b - 1) / b); }

typedef TileCfg<2, 2, 1, 1, 16> GrCfg;   // 32 x 32 tiles (D_ld)

// weight of a triple of the mode contractions (0: all equal, it does not contribute)
__device__ inline double d3_weight(int i, int j, int k) {
  return (i == j && j == k) ? 0.0 : (i == j || j == k || i == k) ? 0.5 : 1.0;
}

// ---------------------------------------------------------------------------
// D_cd: the mode contractions of a batch, K = (triple, x, y), in chunks of whole (triple, x)
// slices; one wavefront per (tile, chunk, mode), without LDS (as the W build), each writing
// one slab of its mode: the K of the whole batch goes through one accumulator, so the
// slabs number 3 nch and not three per triple and chunk (their reduction had taken three
// times the contraction: 492 against 178 us per occupied pair at 12/120).
// ---------------------------------------------------------------------------
template <bool ROWS, int FM, int FN>
__device__ __forceinline__ void cd_tile(const double* __restrict__ tau,
                                        const double* __restrict__ lc, const int* __restrict__ tri,
                                        int g0, int g1, int64_t sm, int64_t su, int m0, int n0,
                                        int nv, double* __restrict__ out) {
  const int lane = threadIdx.x & 63, r16 = lane & 15, kq = lane >> 4;
  const int rp = cube_pitch(nv), ux = rp / 8;
  const int64_t cs = cube_slot(nv);
  // ROWS: rows at stride sm, y contiguous; else rows contiguous, y at the pitch
  const unsigned v0 = ROWS ? (unsigned)(r16 * sm + 2 * kq) * 8u : (unsigned)(2 * kq * rp + 2 * r16) * 8u;
  const unsigned us = ROWS ? 64u : (unsigned)rp * 64u, ks = (unsigned)rp * 8u;
  const unsigned bs = (unsigned)(sm * 128);
  int g = g0, yu = 0;
  unsigned vo = v0;
  double w = 0.0;
  BufRsrc ra = buf_rsrc_n(lc, 0), rb = ra;
  auto open = [&]() {  // the next slice of a contributing triple
    int t = 0;
    while (g < g1) {
      t = g / nv;
      w = d3_weight(tri[3 * t], tri[3 * t + 1], tri[3 * t + 2]);
      if (w != 0.0) break;
      g = (t + 1) * nv;
    }
    if (g >= g1) return;
    const int64_t xo = (int64_t)(g - t * nv) * su;
    ra = buf_rsrc_n(lc + t * cs + xo + m0 * sm, cs - xo - m0 * sm);
    rb = buf_rsrc_n(tau + t * cs + xo + n0 * sm, cs - xo - n0 * sm);
    yu = 0;
    vo = v0;
  };
  double a[2][FM][2], b[2][FN][2];
  int left[2];     // y values left in the slice at this unit; 0: no unit
  double wt[2];
  auto fetch = [&](double (&fa)[FM][2], double (&fb)[FN][2], int& n, double& fw) {
    // past the last slice the loads go on (unused), so that every path has the same count
    // in flight
    frag_load<ROWS, FM>(ra, vo, bs, ks, fa);
    frag_load<ROWS, FN>(rb, vo, bs, ks, fb);
    n = g < g1 ? nv - 8 * yu : 0;
    fw = w;
    vo += us;
    if (++yu == ux && g < g1) {
      ++g;
      open();
    }
  };
  d4v acc[FM][FN];
#pragma unroll
  for (int fm = 0; fm < FM; ++fm)
#pragma unroll
    for (int fn = 0; fn < FN; ++fn) acc[fm][fn] = d4v{0.0, 0.0, 0.0, 0.0};
  open();
  fetch(a[0], b[0], left[0], wt[0]);
  fetch(a[1], b[1], left[1], wt[1]);
  while (left[0] > 0) {
#pragma unroll
    for (int d = 0; d < 2; ++d) {
      if (left[d] > 0) {
        if (!ROWS && left[d] < 8) {  // rows y >= nv of the other order hold the next x
          const bool i0 = 2 * kq < left[d], i1 = 2 * kq + 1 < left[d];
#pragma unroll
          for (int f = 0; f < FM; ++f) {
            a[d][f][0] = i0 ? a[d][f][0] : 0.0;
            a[d][f][1] = i1 ? a[d][f][1] : 0.0;
          }
#pragma unroll
          for (int f = 0; f < FN; ++f) {
            b[d][f][0] = i0 ? b[d][f][0] : 0.0;
            b[d][f][1] = i1 ? b[d][f][1] : 0.0;
          }
        }
        if (wt[d] != 1.0) {
#pragma unroll
          for (int f = 0; f < FM; ++f) {
            a[d][f][0] *= wt[d];
            a[d][f][1] *= wt[d];
          }
        }
#pragma unroll
        for (int t = 0; t < 2; ++t)
#pragma unroll
          for (int fm = 0; fm < FM; ++fm)
#pragma unroll
            for (int fn = 0; fn < FN; ++fn)
              acc[fm][fn] = __builtin_amdgcn_mfma_f64_16x16x4f64(a[d][fm][t], b[d][fn][t],
                                                                 acc[fm][fn], 0, 0, 0);
        fetch(a[d], b[d], left[d], wt[d]);
      }
    }
  }
#pragma unroll
  for (int fm = 0; fm < FM; ++fm)
#pragma unroll
    for (int fn = 0; fn < FN; ++fn)
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        const int c = m0 + frag_row<ROWS, FM>(fm, kq, r), d = n0 + frag_col<ROWS, FN>(fn, r16);
        if (c < nv && d < nv) out[(int64_t)c * nv + d] = acc[fm][fn][r];
      }
}

template <int FM, int FN>
__global__ __launch_bounds__(WNT, shape_waves(FM, FN)) void k_d3_cd(
    const double* __restrict__ tau, const double* __restrict__ lc, const int* __restrict__ tri,
    int nt, double* __restrict__ P, int nv, int nch, int tiles_m, int tiles_n) {
  const unsigned tpp = (unsigned)(tiles_m * tiles_n);
  unsigned item = xcd_item(blockIdx.x, gridDim.x, (tpp + 3) / 4) * 4u +
                  __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int tile = (int)(item % tpp);
  item /= tpp;
  const int ch = (int)(item % (unsigned)nch), m = (int)(item / (unsigned)nch);
  if (m >= 3) return;
  const int m0 = tile / tiles_n * (16 * FM), n0 = tile % tiles_n * (16 * FN);
  const int64_t n = (int64_t)nt * nv;
  const int g0 = (int)(ch * n / nch), g1 = (int)((ch + 1) * n / nch);
  const int64_t rp = cube_pitch(nv), pl = nv * rp;
  double* out = P + ((int64_t)m * nch + ch) * nv * nv;
  if (m == 2) cd_tile<false, FM, FN>(tau, lc, tri, g0, g1, 1, pl, m0, n0, nv, out);
  else cd_tile<true, FM, FN>(tau, lc, tri, g0, g1, m == 0 ? pl : rp, m == 0 ? rp : pl, m0, n0, nv, out);
}

// D[e] += the sum of the nslab slabs of n values: 16 shares of the slabs, then the shares in
// order.
__global__ __launch_bounds__(256) void k_d3_sum(const double* __restrict__ P, int nslab, int64_t n,
                                                double* __restrict__ D) {
  __shared__ double part[256];
  const int el = threadIdx.x & 15, share = threadIdx.x >> 4;
  const int64_t e = (int64_t)blockIdx.x * 16 + el;
  double s = 0.0;
  if (e < n) {
#pragma unroll 8
    for (int q = share; q < nslab; q += 16) s += P[q * n + e];
  }
  part[threadIdx.x] = s;
  __syncthreads();
  if (share == 0 && e < n) {
    for (int h = 1; h < 16; ++h) s += part[h * 16 + el];
    D[e] += s;
  }
}

// ---------------------------------------------------------------------------
// Y^o and D_kc: per (triple, mode), rows of axis m, columns the 2 no rows of t2 (KC 0, the
// cube is L~) or the three rows of E (KC 1, the cube is tau), K = (x, y) split over x.
// Bound by reading the cube once per mode and column tile.
// ---------------------------------------------------------------------------
typedef double d2u __attribute__((ext_vector_type(2), aligned(8)));

template <int KC, bool ROWS, int FM, int FN>
__device__ __forceinline__ void vec_tile(const double* __restrict__ cube, int64_t sm, int64_t su,
                                         const double* const (&col)[FN], int x0, int x1, int m0,
                                         int n0, int ncol, int nv, double* __restrict__ out) {
  const int lane = threadIdx.x & 63, r16 = lane & 15, kq = lane >> 4;
  const int rp = cube_pitch(nv), ux = rp / 8;
  const int64_t cs = cube_slot(nv);
  const unsigned v0 = ROWS ? (unsigned)(r16 * sm + 2 * kq) * 8u : (unsigned)(2 * kq * rp + 2 * r16) * 8u;
  const unsigned us = ROWS ? 64u : (unsigned)rp * 64u, ks = (unsigned)rp * 8u;
  const unsigned bs = (unsigned)(sm * 128);
  int x = x0, yu = 0;
  unsigned vo = v0;
  BufRsrc ra = buf_rsrc_n(cube + x * su + m0 * sm, cs - x * su - m0 * sm);
  double a[2][FM][2], b[2][FN][2];
  int left[2];
  auto fetch = [&](double (&fa)[FM][2], double (&fb)[FN][2], int& n) {
    // past x1 the loads repeat the last slice's (unused)
    frag_load<ROWS, FM>(ra, vo, bs, ks, fa);
    const int y = 8 * yu + 2 * kq, ny = nv - 8 * yu;
    const int64_t xo = (int64_t)min(x, x1 - 1) * nv;
    n = x < x1 ? ny : 0;
    if (ny >= 8) {
#pragma unroll
      for (int f = 0; f < FN; ++f) {
        const d2u v = *(const d2u*)(col[f] + xo + y);
        fb[f][0] = v[0];
        fb[f][1] = v[1];
      }
    } else {  // the row's end: clamped loads, zeroed below
#pragma unroll
      for (int f = 0; f < FN; ++f) {
        fb[f][0] = col[f][xo + min(y, nv - 1)];
        fb[f][1] = col[f][xo + min(y + 1, nv - 1)];
      }
    }
    vo += us;
    if (++yu == ux) {
      yu = 0;
      vo = v0;
      ++x;
      if (x < x1) ra = buf_rsrc_n(cube + x * su + m0 * sm, cs - x * su - m0 * sm);
    }
  };
  d4v acc[FM][FN];
#pragma unroll
  for (int fm = 0; fm < FM; ++fm)
#pragma unroll
    for (int fn = 0; fn < FN; ++fn) acc[fm][fn] = d4v{0.0, 0.0, 0.0, 0.0};
  fetch(a[0], b[0], left[0]);
  fetch(a[1], b[1], left[1]);
  while (left[0] > 0) {
#pragma unroll
    for (int d = 0; d < 2; ++d) {
      if (left[d] > 0) {
        if (left[d] < 8) {
          const bool i0 = 2 * kq < left[d], i1 = 2 * kq + 1 < left[d];
#pragma unroll
          for (int f = 0; f < FM; ++f) {
            a[d][f][0] = i0 ? a[d][f][0] : 0.0;
            a[d][f][1] = i1 ? a[d][f][1] : 0.0;
          }
#pragma unroll
          for (int f = 0; f < FN; ++f) {
            b[d][f][0] = i0 ? b[d][f][0] : 0.0;
            b[d][f][1] = i1 ? b[d][f][1] : 0.0;
          }
        }
#pragma unroll
        for (int t = 0; t < 2; ++t)
#pragma unroll
          for (int fm = 0; fm < FM; ++fm)
#pragma unroll
            for (int fn = 0; fn < FN; ++fn)
              acc[fm][fn] = __builtin_amdgcn_mfma_f64_16x16x4f64(a[d][fm][t], b[d][fn][t],
                                                                 acc[fm][fn], 0, 0, 0);
        fetch(a[d], b[d], left[d]);
      }
    }
  }
#pragma unroll
  for (int fm = 0; fm < FM; ++fm)
#pragma unroll
    for (int fn = 0; fn < FN; ++fn)
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        const int c = m0 + frag_row<ROWS, FM>(fm, kq, r), n = n0 + fn * 16 + r16;
        if (c < nv && n < ncol) out[(int64_t)c * ncol + n] = acc[fm][fn][r];
      }
}

constexpr int VFM = 4;  // 64 rows per wavefront; 32 columns of Y^o, 16 (three used) of D_kc

template <int KC>
__global__ __launch_bounds__(WNT, 2) void k_d3_vec(const double* __restrict__ cubes,
                                                   const int* __restrict__ tri, int nt,
                                                   const double* __restrict__ X,
                                                   double* __restrict__ P, int no, int nv, int nch,
                                                   int tiles_m, int tiles_n) {
  constexpr int FN = KC ? 1 : 2;
  unsigned item = blockIdx.x * 4u + __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int tn = (int)(item % (unsigned)tiles_n);
  item /= (unsigned)tiles_n;
  const int tm = (int)(item % (unsigned)tiles_m);
  item /= (unsigned)tiles_m;
  const int ch = (int)(item % (unsigned)nch);
  item /= (unsigned)nch;
  const int m = (int)(item % 3u), t = (int)(item / 3u);
  if (t >= nt) return;
  const int o[3] = {tri[3 * t], tri[3 * t + 1], tri[3 * t + 2]};
  if (o[0] == o[1] && o[1] == o[2]) return;
  const int s = m == 0 ? o[0] : m == 1 ? o[1] : o[2];
  const int U = m == 0 ? o[1] : o[0], V = m == 2 ? o[1] : o[2];
  const int ncol = KC ? 3 : 2 * no, n0 = tn * 16 * FN, m0 = tm * 16 * VFM;
  const double* col[FN];
#pragma unroll
  for (int f = 0; f < FN; ++f) {
    const int n = min(n0 + f * 16 + (int)(threadIdx.x & 15), ncol - 1);
    int p, q;  // the matrix [x][y] of X[p][q]
    if (KC) { p = n == 2 ? s : U; q = n == 1 ? s : V; }
    else if (n < no) { p = n; q = V; }
    else { p = U; q = n - no; }
    col[f] = X + ((int64_t)p * no + q) * nv * nv;
  }
  const int x0 = (int)((int64_t)ch * nv / nch), x1 = (int)((int64_t)(ch + 1) * nv / nch);
  const int64_t rp = cube_pitch(nv), pl = nv * rp;
  const double* cube = cubes + t * cube_slot(nv);
  double* out = P + (((int64_t)t * 3 + m) * nch + ch) * nv * ncol;
  if (m == 2)
    vec_tile<KC, false, VFM, FN>(cube, 1, pl, col, x0, x1, m0, n0, ncol, nv, out);
  else
    vec_tile<KC, true, VFM, FN>(cube, m == 0 ? pl : rp, m == 0 ? rp : pl, col, x0, x1, m0, n0, ncol,
                                nv, out);
}

// The candidates e < n for which `match` holds, in order, into list[] (at most `cap`), by
// ballots; every thread of the 256 calls it.
template <class M>
__device__ inline int d3_list(int n, int cap, int* list, int* cz, M match) {
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  int base = 0;
  for (int e0 = 0; e0 < n; e0 += 256) {
    const int e = e0 + (int)threadIdx.x;
    const bool in = e < n && match(e);
    const unsigned long long hit = __ballot(in);
    if (lane == 0) cz[wave] = __popcll(hit);
    __syncthreads();
    int at = base;
    for (int w = 0; w < 4; ++w) {
      const int c = cz[w];
      if (w < wave) at += c;
      base += c;
    }
    at += __popcll(hit & ((1ull << lane) - 1ull));
    if (in && at < cap) list[at] = e;
    __syncthreads();
  }
  return base < cap ? base : cap;
}

// Y'[l][r][p][c] (= Y^o[c][l][p][r]) += the weighted chunk sums of the (triple, mode, half)
// products with that (p, r), in that order; one block of (c, l) per (p, r).
__global__ __launch_bounds__(256) void k_d3_red_y(const int* __restrict__ tri, int nt,
                                                  const double* __restrict__ P,
                                                  double* __restrict__ Y, int no, int nv, int nch) {
  __shared__ int list[6 * D3_MAXB], cz[4];
  const int p = blockIdx.y / no, r = blockIdx.y % no;
  const int cnt = d3_list(6 * nt, 6 * D3_MAXB, list, cz, [&](int e) {
    const int t = e / 6, m = (e % 6) >> 1, h = e & 1;
    const int* o = tri + 3 * t;
    if (o[0] == o[1] && o[1] == o[2]) return false;
    const int U = m == 0 ? o[1] : o[0], V = m == 2 ? o[1] : o[2];
    return o[m] == r && (h ? V : U) == p;
  });
  const int64_t e = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;  // c * no + l
  if (cnt == 0 || e >= (int64_t)nv * no) return;
  const int c = (int)(e / no), l = (int)(e % no);
  const int64_t slab = (int64_t)nv * 2 * no;
  double s = 0.0;
  for (int q = 0; q < cnt; ++q) {
    const int t = list[q] / 6, m = (list[q] % 6) >> 1, h = list[q] & 1;
    const double* pp = P + ((int64_t)t * 3 + m) * nch * slab + (int64_t)c * 2 * no + h * no + l;
    double st = 0.0;
#pragma unroll 8
    for (int ch = 0; ch < nch; ++ch) st += pp[ch * slab];
    s += d3_weight(tri[3 * t], tri[3 * t + 1], tri[3 * t + 2]) * st;
  }
  Y[(((int64_t)l * no + r) * no + p) * nv + c] += s;
}

// D_kc[r][c] += the weighted sums of the triples that hold r: 16 c per workgroup, 16 shares
// of the triples added in order.  The columns of one mode are summed first, then the modes of
// one triple: where tau~ vanishes (nv = 1) they cancel exactly.
__global__ __launch_bounds__(256) void k_d3_red_kc(const int* __restrict__ tri, int nt,
                                                   const double* __restrict__ P,
                                                   double* __restrict__ D, int no, int nv,
                                                   int nch) {
  __shared__ int list[D3_MAXB], cz[4];
  __shared__ double part[256];
  const int r = blockIdx.y;
  const int cnt = d3_list(nt, D3_MAXB, list, cz, [&](int t) {
    const int* o = tri + 3 * t;
    return !(o[0] == o[1] && o[1] == o[2]) && (o[0] == r || o[1] == r || o[2] == r);
  });
  const int el = threadIdx.x & 15, share = threadIdx.x >> 4;
  const int c = blockIdx.x * 16 + el;
  const int64_t slab = (int64_t)nv * 3;
  double s = 0.0;
  if (c < nv)
    for (int q = share; q < cnt; q += 16) {
      const int* o = tri + 3 * list[q];
      double sq = 0.0;
      for (int m = 0; m < 3; ++m) {
        const int U = m == 0 ? o[1] : o[0], V = m == 2 ? o[1] : o[2];
        double sm = 0.0;
        for (int n = 0; n < 3; ++n) {
          if ((n == 0 ? o[m] : n == 1 ? V : U) != r) continue;
          const double* pp = P + ((int64_t)list[q] * 3 + m) * nch * slab + (int64_t)c * 3 + n;
          double st = 0.0;
#pragma unroll 8
          for (int ch = 0; ch < nch; ++ch) st += pp[ch * slab];
          sm += (n == 0 ? 4.0 : -2.0) * st;
        }
        sq += sm;
      }
      s += d3_weight(o[0], o[1], o[2]) * sq;
    }
  part[threadIdx.x] = s;
  __syncthreads();
  if (share == 0 && c < nv) {
    for (int h = 1; h < 16; ++h) s += part[h * 16 + el];
    D[(int64_t)r * nv + c] += s;
  }
}

// ---------------------------------------------------------------------------
// Gram matrices of pairs: M[k][l] = <L~_{ijk}, tau_{ijl}> over the whole cube
// ---------------------------------------------------------------------------
// The cube of (i, j, k) is that of its sorted triple, whose axes hold (a, b, c) as
//   k <= j: [a][b][c],   j < k <= i: [a][c][b],   k > i: [c][a][b]
// (resident cubes, one per unordered triple), or the k-th cube of a batch in its own
// order.  A workgroup runs over (a, 16 x 16 of (b, c)) patches: every row of the patch is
// read as whole 128-byte segments along its contiguous index, put into LDS in the common
// order (b, c), and the patch's 256 k go through the MFMA, 64 to each of the four
// wavefronts.  Bound by reading each cube once per pair.
constexpr int GRS = 276;  // doubles of an LDS row: 16 x 17 (conflict-free in both orders) + 4

template <int RT>
__global__ __launch_bounds__(256) void k_d3_gram(const double* __restrict__ tau,
                                                 const double* __restrict__ lc, int resident,
                                                 int pair0, double* __restrict__ P, int no, int nv,
                                                 int nch, int tiles) {
  constexpr int NB = RT / 16;
  __shared__ double lds[2 * RT * GRS];
  __shared__ int64_t rbase[2 * RT];
  __shared__ int rcls[2 * RT];
  const int ch = blockIdx.x, pr = blockIdx.y;
  const int k0 = (int)blockIdx.z / tiles * RT, l0 = (int)blockIdx.z % tiles * RT;
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6, r16 = lane & 15, kq = lane >> 4;
  const int64_t rp = cube_pitch(nv), pl = nv * rp, cs = cube_slot(nv);
  if (tid < 2 * RT) {
    const int k = tid < RT ? k0 + tid : l0 + tid - RT;
    int64_t at = -1;
    int cls = 0;
    if (k < no) {
      at = k;
      if (resident) {
        int i = 0;  // pair index = i (i + 1) / 2 + j
        while ((i + 1) * (i + 2) / 2 <= pair0 + pr) ++i;
        const int j = pair0 + pr - i * (i + 1) / 2;
        cls = k <= j ? 0 : k <= i ? 1 : 2;
        const int A = k > i ? k : i, C = k <= j ? k : j, B = i + j + k - A - C;
        at = (int64_t)A * (A + 1) * (A + 2) / 6 + B * (B + 1) / 2 + C;
      }
      at *= cs;
    }
    rbase[tid] = at;
    rcls[tid] = cls;
  }
  __syncthreads();
  const int nb = (nv + 15) / 16, npatch = nv * nb * nb;
  const int u = tid >> 4, v = tid & 15;
  d4v acc[NB][NB];
#pragma unroll
  for (int f = 0; f < NB; ++f)
#pragma unroll
    for (int g = 0; g < NB; ++g) acc[f][g] = d4v{0.0, 0.0, 0.0, 0.0};
  for (int pt = ch; pt < npatch; pt += nch) {
    const int a = pt / (nb * nb), b0 = pt / nb % nb * 16, c0 = pt % nb * 16;
    // class 0: (b, c) = (u, v); classes 1 and 2: (u, v) exchanged
    const bool in0 = b0 + u < nv && c0 + v < nv, in1 = b0 + v < nv && c0 + u < nv;
    const int64_t e0 = in0 ? a * pl + (b0 + u) * rp + c0 + v : 0;
    const int64_t e1 = in1 ? a * pl + (c0 + u) * rp + b0 + v : 0;
    const int64_t e2 = in1 ? (c0 + u) * pl + a * rp + b0 + v : 0;
    // eight rows in flight; rows past no and elements past nv load a valid element
#pragma unroll
    for (int r0 = 0; r0 < 2 * RT; r0 += 8) {
      double x[8];
#pragma unroll
      for (int h = 0; h < 8; ++h) {
        const int64_t base = rbase[r0 + h];
        const int cls = rcls[r0 + h];
        x[h] = ((r0 < RT ? lc : tau) + (base >= 0 ? base : 0))[cls == 0 ? e0 : cls == 1 ? e1 : e2];
      }
#pragma unroll
      for (int h = 0; h < 8; ++h) {
        const int cls = rcls[r0 + h];
        const bool in = rbase[r0 + h] >= 0 && (cls == 0 ? in0 : in1);
        lds[(r0 + h) * GRS + (cls == 0 ? u * 17 + v : v * 17 + u)] = in ? x[h] : 0.0;
      }
    }
    __syncthreads();
#pragma unroll 4
    for (int s = 0; s < 16; ++s) {  // k-step: four c of one b
      const int ks = wave * 16 + s, at = (ks >> 2) * 17 + (ks & 3) * 4 + kq;
      double x[NB], y[NB];
#pragma unroll
      for (int f = 0; f < NB; ++f) {
        x[f] = lds[(f * 16 + r16) * GRS + at];
        y[f] = lds[(RT + f * 16 + r16) * GRS + at];
      }
#pragma unroll
      for (int f = 0; f < NB; ++f)
#pragma unroll
        for (int g = 0; g < NB; ++g)
          acc[f][g] = __builtin_amdgcn_mfma_f64_16x16x4f64(x[f], y[g], acc[f][g], 0, 0, 0);
    }
    __syncthreads();
  }
  double* out = P + (((int64_t)pr * nch + ch) * 4 + wave) * no * no;
#pragma unroll
  for (int f = 0; f < NB; ++f)
#pragma unroll
    for (int g = 0; g < NB; ++g)
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        const int k = k0 + f * 16 + kq + 4 * r, l = l0 + g * 16 + r16;
        if (k < no && l < no) out[k * no + l] = acc[f][g][r];
      }
}

// D_lk[l][k] -= w_ij / 2 M_ij[k][l] over the pairs: one workgroup per element, thread t
// sums the slabs t, t + 256, ... in order, then a fixed binary tree.
__global__ __launch_bounds__(256) void k_d3_red_lk(const double* __restrict__ P,
                                                   double* __restrict__ D, int pair0, int npair,
                                                   int no, int nch) {
  __shared__ double part[256];
  const int e = blockIdx.x;
  const int l = e / no, k = e % no;
  const int per = 4 * nch;
  double s = 0.0;
  for (int64_t q = threadIdx.x; q < (int64_t)npair * per; q += 256) {
    const int pr = pair0 + (int)(q / per);
    int i = 0;
    while ((i + 1) * (i + 2) / 2 <= pr) ++i;
    s += (pr == i * (i + 1) / 2 + i ? -0.5 : -1.0) * P[q * no * no + (int64_t)k * no + l];
  }
  part[threadIdx.x] = s;
  __syncthreads();
  for (int w = 128; w > 0; w >>= 1) {
    if (threadIdx.x < w) part[threadIdx.x] += part[threadIdx.x + w];
    __syncthreads();
  }
  if (threadIdx.x == 0) D[e] += part[0];
}

// ---------------------------------------------------------------------------
// D_ld = - sum_{k,i,c} Y'[l][k][i][c] t2[k][i][c][d]: rows l, columns d, K = (k,i,c)
// ---------------------------------------------------------------------------
__global__ __launch_bounds__(GrCfg::NT) void k_d3_ld(const double* __restrict__ Y,
                                                     const double* __restrict__ t2,
                                                     double* __restrict__ P, int no, int nv,
                                                     int nch, int tiles_n) {
  typedef GrCfg T;
  __shared__ double lds[T::LDS_DOUBLES];
  const int ch = blockIdx.x % nch, tile = blockIdx.x / nch;
  const int m0 = (tile / tiles_n) * T::BM, n0 = (tile % tiles_n) * T::BN;
  const int K = no * no * nv;
  const int S = (K + T::BK - 1) / T::BK;
  const int s0 = (int)((int64_t)ch * S / nch), s1 = (int)((int64_t)(ch + 1) * S / nch);
  auto ops = [&](int s, Opnd& A, Opnd& B, int& k0) {
    k0 = (s0 + s) * T::BK;
    A = make_opnd(Y, K, 1, no, K, false);
    B = make_opnd(t2, 1, nv, nv, K, true);
  };
  d4v acc[T::FM][T::FN];
  zero_acc<T>(acc);
  k_loop<T>(s1 - s0, m0, n0, ops, acc, lds);
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const int wm = wave % T::WM, wn = wave / T::WM;
  double* out = P + (int64_t)ch * no * nv;
#pragma unroll
  for (int fm = 0; fm < T::FM; ++fm)
#pragma unroll
    for (int fn = 0; fn < T::FN; ++fn)
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        const int l = m0 + acc_row<T>(wm, fm, lane, r), d = n0 + acc_col<T>(wn, fn, lane);
        if (l < no && d < nv) out[(int64_t)l * nv + d] = acc[fm][fn][r];
      }
}

__global__ void k_d3_red_ld(const double* __restrict__ P, double* __restrict__ D, int no, int nv,
                            int nch) {
  const int64_t e = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (e >= (int64_t)no * nv) return;
  double s = 0.0;
  for (int ch = 0; ch < nch; ++ch) s += P[(int64_t)ch * no * nv + e];
  D[e] -= s;
}

// Y^o[c][l][i][k] (+)= Y'[l][k][i][c]
__global__ void k_d3_yout(const double* __restrict__ Y, double* __restrict__ Yo, int no, int nv,
                          int accumulate) {
  const int64_t n = (int64_t)nv * no * no * no;
  const int64_t e = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (e >= n) return;
  const int k = (int)(e % no), i = (int)((e / no) % no), l = (int)((e / (no * no)) % no);
  const int c = (int)(e / ((int64_t)no * no * no));
  const double v = Y[(((int64_t)l * no + k) * no + i) * nv + c];
  Yo[e] = accumulate ? Yo[e] + v : v;
}

// l2M[r][y][x][l] = -l2[l][r][x][y], each (r, y) slab at the pitch t2n_pitch
__global__ void k_d3_l2m(const double* __restrict__ l2, double* __restrict__ l2M, int no, int nv) {
  const int64_t nvl = nv, n = (int64_t)no * no * nvl * nvl;
  const int64_t e = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (e >= n) return;
  const int l = (int)(e % no), x = (int)((e / no) % nvl), y = (int)((e / (no * nvl)) % nvl);
  const int r = (int)(e / (no * nvl * nvl));
  l2M[((int64_t)r * nvl + y) * t2n_pitch(no, nv) + (int64_t)x * no + l] = -l2[(((int64_t)l * no + r) * nvl + x) * nvl + y];
}

// E[p][q][x][y] = 2 l2[p][q][x][y] - l2[p][q][y][x]
__global__ void k_d3_e(const double* __restrict__ l2, double* __restrict__ E, int64_t n, int nv) {
  const int64_t nv2 = (int64_t)nv * nv;
  const int64_t e = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (e >= n) return;
  const int xy = (int)(e % nv2);
  E[e] = 2.0 * l2[e] - l2[e - xy + (int64_t)(xy % nv) * nv + xy / nv];
}

// ---------------------------------------------------------------------------
// launchers
// ---------------------------------------------------------------------------
// K chunks: about 2048 wave tiles per launch (one round of the resident ones), the slabs
// read back by the reductions being in proportion.
static int cd_chunks(int nv, int nt) {
  int tm, tn;
  shape_tiles(pick_shape(nv, nv), nv, nv, &tm, &tn);
  const int64_t n = (2048 + 3 * tm * tn - 1) / (3 * tm * tn), most = (int64_t)(nt > 0 ? nt : 1) * nv;
  return (int)(n < 1 ? 1 : n > most ? most : n);
}
static int vec_chunks(int nv, int nt, int ncol) {
  const int t = (int)nblk(nv, 16 * VFM) * (int)nblk(ncol, ncol > 16 ? 32 : 16) * 3;
  const int n = (2048 + t * nt - 1) / (t * (nt > 0 ? nt : 1));
  return n < 1 ? 1 : (n > nv ? nv : n);
}
static int gram_tiles(int no) { return no <= 16 ? 1 : (int)nblk(no, 32); }
static int gram_chunks(int no, int nv, int npair) {
  const int nb = (nv + 15) / 16, t = gram_tiles(no);
  const int64_t np = (int64_t)nv * nb * nb;
  int64_t n = (4096 + (int64_t)npair * t * t - 1) / ((int64_t)npair * t * t);
  if (n > 1024) n = 1024;
  return (int)(n > np ? np : n);
}
static int ld_chunks(int no, int nv) {
  const int t = ((no + GrCfg::BM - 1) / GrCfg::BM) * ((nv + GrCfg::BN - 1) / GrCfg::BN);
  const int S = (no * no * nv + GrCfg::BK - 1) / GrCfg::BK;
  int n = (1024 + t - 1) / t;
  return n > S ? S : n;
}

size_t d3_partial_doubles(int no, int nv, int maxt, int npair) {
  size_t m = 0;
  const size_t v = nv, o = no;
  for (int nt = 1; nt <= maxt; ++nt) {
    m = std::max(m, 3 * (size_t)cd_chunks(nv, nt) * v * v);
    m = std::max(m, (size_t)nt * 3 * vec_chunks(nv, nt, 2 * no) * v * 2 * o);
    m = std::max(m, (size_t)nt * 3 * vec_chunks(nv, nt, 3) * v * 3);
  }
  m = std::max(m, (size_t)npair * gram_chunks(no, nv, npair) * 4 * o * o);
  return std::max(m, (size_t)ld_chunks(no, nv) * o * v);
}

void launch_d3_cd(const double* tau, const double* lc, const int* tri, int nt, double* P,
                  double* Dcd, int nv, hipStream_t st) {
  if (nt <= 0) return;
  const int shape = pick_shape(nv, nv), nch = cd_chunks(nv, nt);
  int tm, tn;
  shape_tiles(shape, nv, nv, &tm, &tn);
  with_shape(shape, [&](auto fm, auto fn) {
    hipLaunchKernelGGL((k_d3_cd<decltype(fm)::value, decltype(fn)::value>),
                       dim3(nblk((int64_t)tm * tn * nch * 3, 4)), dim3(WNT), 0, st, tau, lc, tri, nt,
                       P, nv, nch, tm, tn);
  });
  const int64_t n = (int64_t)nv * nv;
  hipLaunchKernelGGL(k_d3_sum, dim3(nblk(n, 16)), dim3(256), 0, st, P, 3 * nch, n, Dcd);
}

void launch_d3_vec(const double* tau, const double* lc, const int* tri, int nt, const double* t2,
                   const double* E, double* P, double* Y, double* Dkc, int no, int nv,
                   hipStream_t st) {
  if (nt <= 0) return;
  const int tm = (int)nblk(nv, 16 * VFM);
  {
    const int tn = (int)nblk(2 * no, 32), nch = vec_chunks(nv, nt, 2 * no);
    hipLaunchKernelGGL(k_d3_vec<0>, dim3(nblk((int64_t)tm * tn * nch * 3 * nt, 4)), dim3(WNT), 0, st,
                       lc, tri, nt, t2, P, no, nv, nch, tm, tn);
    hipLaunchKernelGGL(k_d3_red_y, dim3(nblk((int64_t)nv * no, 256), no * no), dim3(256), 0, st, tri,
                       nt, P, Y, no, nv, nch);
  }
  {
    const int nch = vec_chunks(nv, nt, 3);
    hipLaunchKernelGGL(k_d3_vec<1>, dim3(nblk((int64_t)tm * nch * 3 * nt, 4)), dim3(WNT), 0, st, tau,
                       tri, nt, E, P, no, nv, nch, tm, 1);
    hipLaunchKernelGGL(k_d3_red_kc, dim3(nblk(nv, 16), no), dim3(256), 0, st, tri, nt, P, Dkc, no, nv,
                       nch);
  }
}

void launch_d3_gram(const double* tau, const double* lc, bool resident, int pair0, int npair,
                    double* P, double* Dlk, int no, int nv, hipStream_t st) {
  const int t = gram_tiles(no), nch = gram_chunks(no, nv, npair);
  const dim3 grid(nch, npair, t * t);
  if (no <= 16)
    hipLaunchKernelGGL(k_d3_gram<16>, grid, dim3(256), 0, st, tau, lc,
                       resident ? 1 : 0, pair0, P, no, nv, nch, t);
  else
    hipLaunchKernelGGL(k_d3_gram<32>, grid, dim3(256), 0, st, tau, lc,
                       resident ? 1 : 0, pair0, P, no, nv, nch, t);
  hipLaunchKernelGGL(k_d3_red_lk, dim3(no * no), dim3(256), 0, st, P, Dlk, pair0, npair, no, nch);
}

void launch_d3_ld(const double* Y, const double* t2, double* P, double* Dld, int no, int nv,
                  hipStream_t st) {
  typedef GrCfg T;
  const int tm = (no + T::BM - 1) / T::BM, tn = (nv + T::BN - 1) / T::BN;
  const int nch = ld_chunks(no, nv);
  hipLaunchKernelGGL(k_d3_ld, dim3(tm * tn * nch), dim3(T::NT), 0, st, Y, t2, P, no, nv, nch, tn);
  hipLaunchKernelGGL(k_d3_red_ld, dim3(nblk((int64_t)no * nv, 256)), dim3(256), 0, st, P, Dld, no,
                     nv, nch);
}

void launch_d3_yout(const double* Y, double* Yo, int no, int nv, bool accumulate, hipStream_t st) {
  const int64_t n = (int64_t)nv * no * no * no;
  hipLaunchKernelGGL(k_d3_yout, dim3(nblk(n, 256)), dim3(256), 0, st, Y, Yo, no, nv,
                     accumulate ? 1 : 0);
}

void launch_d3_l2(const double* l2, double* l2M, double* E, int no, int nv, hipStream_t st) {
  const int64_t n = (int64_t)no * no * nv * nv;
  hipLaunchKernelGGL(k_d3_l2m, dim3(nblk(n, 256)), dim3(256), 0, st, l2, l2M, no, nv);
  hipLaunchKernelGGL(k_d3_e, dim3(nblk(n, 256)), dim3(256), 0, st, l2, E, n, nv);
}

}  // namespace cc3
