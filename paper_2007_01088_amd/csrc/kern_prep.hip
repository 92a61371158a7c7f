// Preparation kernels run once per residual call, before the triple loop:
// the T1 transformation of the Cholesky vectors, the Fock ov block, the
// integral-block build (FP64 MFMA GEMMs over the Cholesky index, writing the
// internal layouts the triple loop streams), the re-layout of caller-given
// blocks, the triple table, and the covariant back-transformation after it.
#include <algorithm>

#include "cc3_device.hpp"
#include "cc3_internal.hpp"

namespace cc3 {

static inline unsigned nblk(int64_t n, int b) { return (unsigned)((n + b - 1) / b); }

__global__ void k_fill(double* __restrict__ p, int64_t n, double v) {
  int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  const int64_t stride = (int64_t)gridDim.x * blockDim.x;
  for (; i < n; i += stride) p[i] = v;
}

void launch_fill(double* p, int64_t n, double v, hipStream_t st) {
  if (n <= 0) return;
  unsigned g = nblk(n, 256);
  if (g > 65536u) g = 65536u;
  hipLaunchKernelGGL(k_fill, dim3(g), dim3(256), 0, st, p, n, v);
}

__global__ void k_add(double* __restrict__ y, const double* __restrict__ x, int64_t n) {
  int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  const int64_t stride = (int64_t)gridDim.x * blockDim.x;
  for (; i < n; i += stride) y[i] += x[i];
}

void launch_add(double* y, const double* x, int64_t n, hipStream_t st) {
  if (n <= 0) return;
  unsigned g = nblk(n, 256);
  if (g > 65536u) g = 65536u;
  hipLaunchKernelGGL(k_add, dim3(g), dim3(256), 0, st, y, x, n);
}

// ---------------------------------------------------------------------------
// T1 transformation (exp(-T1) H exp(T1)):  Lt = (1 - t) L (1 + t), t[no+a][i] = t1[i][a].
//   Lt_bd = L_bd - sum_l t1[l][b] L_ld        Lt_lj = L_lj + sum_d L_ld t1[j][d]
//   Lt_ck = L_ck + sum_d L_cd t1[k][d] - sum_l t1[l][c] Lt_lk      Lt_kc = L_kc
// ---------------------------------------------------------------------------
// First launch, one grid row per J: blocks of the vv part, blocks of the oo part (with the
// copy of the ov block), and one for the sums of the Fock block,
//   s_J = sum_ld t1[l][d] L_ld,  M_J[k][l] = sum_d L_kd t1[l][d].
__device__ __forceinline__ void t1_vv(const double* __restrict__ LJ, const double* __restrict__ t1,
                                      double* __restrict__ Lvv, int J, int bx, int no, int nv) {
  const int64_t idx = (int64_t)bx * blockDim.x + threadIdx.x;
  if (idx >= (int64_t)nv * nv) return;
  const int b = (int)(idx / nv), d = (int)(idx % nv);
  const int nmo = no + nv;
  double v = LJ[(int64_t)(no + b) * nmo + no + d];
  for (int l = 0; l < no; ++l) v -= t1[(int64_t)l * nv + b] * LJ[(int64_t)l * nmo + no + d];
  Lvv[(int64_t)J * nv * nv + idx] = v;
}

__device__ __forceinline__ void t1_oo(const double* __restrict__ LJ, const double* __restrict__ t1,
                                      double* __restrict__ Loo, double* __restrict__ LooT,
                                      double* __restrict__ Lov, int J, int bx, int nblocks, int no,
                                      int nv) {
  const int nmo = no + nv;
  const int idx = bx * blockDim.x + threadIdx.x;
  if (idx < no * no) {
    const int l = idx / no, j = idx % no;
    double v = LJ[(int64_t)l * nmo + j];
    for (int d = 0; d < nv; ++d) v += LJ[(int64_t)l * nmo + no + d] * t1[(int64_t)j * nv + d];
    Loo[(int64_t)J * no * no + (int64_t)l * no + j] = v;
    LooT[(int64_t)J * no * no + (int64_t)j * no + l] = v;
  }
  // untransformed ov block, Lov[J][k][c] = L_{k, no+c}
  for (int e = idx; e < no * nv; e += nblocks * blockDim.x) {
    const int k = e / nv, c = e % nv;
    Lov[(int64_t)J * no * nv + e] = LJ[(int64_t)k * nmo + no + c];
  }
}

__device__ __forceinline__ void fock_sm(const double* __restrict__ LJ,
                                        const double* __restrict__ t1, double* __restrict__ s,
                                        double* __restrict__ M, int J, int no, int nv) {
  const int nmo = no + nv;
  __shared__ double red[256];
  double acc = 0.0;
  for (int e = threadIdx.x; e < no * nv; e += blockDim.x)
    acc += t1[e] * LJ[(int64_t)(e / nv) * nmo + no + e % nv];
  red[threadIdx.x] = acc;
  __syncthreads();
  for (int w = blockDim.x / 2; w > 0; w >>= 1) {
    if ((int)threadIdx.x < w) red[threadIdx.x] += red[threadIdx.x + w];
    __syncthreads();
  }
  if (threadIdx.x == 0) s[J] = red[0];
  for (int e = threadIdx.x; e < no * no; e += blockDim.x) {
    const int k = e / no, l = e % no;
    double v = 0.0;
    for (int d = 0; d < nv; ++d) v += LJ[(int64_t)k * nmo + no + d] * t1[(int64_t)l * nv + d];
    M[(int64_t)J * no * no + e] = v;
  }
}

__global__ __launch_bounds__(256) void k_t1_first(const double* __restrict__ L,
                                                  const double* __restrict__ t1,
                                                  CholeskyScratch cs, int nvv, int noo, int no,
                                                  int nv) {
  const int J = blockIdx.y, bx = blockIdx.x;
  const double* LJ = L + (int64_t)J * (no + nv) * (no + nv);
  if (bx < nvv) t1_vv(LJ, t1, cs.Lvv, J, bx, no, nv);
  else if (bx < nvv + noo) t1_oo(LJ, t1, cs.Loo, cs.LooT, cs.Lov, J, bx - nvv, noo, no, nv);
  else fock_sm(LJ, t1, cs.s, cs.M, J, no, nv);
}

// LvoT[J][k][c] for 16 consecutive c of one J.  The rows L_{no+c, no+d} and t1
// pass through LDS in chunks of 64 d, so every global read is a row segment;
// each sum keeps the order of the formula above (d ascending, then l).
constexpr int VO_RC = 16, VO_DC = 64;
__device__ __forceinline__ void t1_vo(const double* __restrict__ L, const double* __restrict__ t1,
                                      const double* __restrict__ Loo, double* __restrict__ LvoT,
                                      double (&Ls)[VO_RC][VO_DC + 1], double (&Ts)[64][VO_DC + 1],
                                      int J, int bx, int no, int nv) {
  constexpr int RC = VO_RC, DC = VO_DC;
  const int c0 = bx * RC, tid = threadIdx.x;
  const int nmo = no + nv;
  const double* LJ = L + (int64_t)J * nmo * nmo;
  const int ci = tid % RC, k = tid / RC, c = c0 + ci;  // no <= 63: one sum per thread
  double v = (k < no && c < nv) ? LJ[(int64_t)(no + c) * nmo + k] : 0.0;
  for (int d0 = 0; d0 < nv; d0 += DC) {
    const int dn = min(DC, nv - d0);
    for (int e = tid; e < RC * DC; e += 1024) {
      const int r = e / DC, dd = e % DC;
      Ls[r][dd] = (c0 + r < nv && dd < dn) ? LJ[(int64_t)(no + c0 + r) * nmo + no + d0 + dd] : 0.0;
    }
    for (int e = tid; e < no * DC; e += 1024) {
      const int r = e / DC, dd = e % DC;
      Ts[r][dd] = dd < dn ? t1[(int64_t)r * nv + d0 + dd] : 0.0;
    }
    __syncthreads();
    if (k < no)
      for (int dd = 0; dd < dn; ++dd) v += Ls[ci][dd] * Ts[k][dd];
    __syncthreads();
  }
  const double* LooJ = Loo + (int64_t)J * no * no;
  if (k >= no || c >= nv) return;
  for (int l = 0; l < no; ++l) v -= t1[(int64_t)l * nv + c] * LooJ[(int64_t)l * no + k];
  LvoT[(int64_t)J * no * nv + (int64_t)k * nv + c] = v;
}

// ---------------------------------------------------------------------------
// Fock ov block of the T1-transformed Hamiltonian (canonical reference):
//   F_kc = sum_ld t1[l][d] (2 g_kcld - g_kdlc),  g_kcld = sum_J L_kc L_ld
//        = sum_J [ 2 s_J L_kc - sum_l M_J[k][l] L_lc ],
//   s_J = sum_ld t1[l][d] L_ld,  M_J[k][l] = sum_d L_kd t1[l][d].
// ---------------------------------------------------------------------------
// F[k][c] for 64 consecutive c of one k; sixteen slices of the Cholesky index
// summed through LDS in a fixed order.
__device__ __forceinline__ void fock(const double* __restrict__ Lov, const double* __restrict__ s,
                                     const double* __restrict__ M, double* __restrict__ F,
                                     double* __restrict__ red, int k, int by, int no, int nv,
                                     int nJ) {
  constexpr int NS = 16;
  const int c = by * 64 + (threadIdx.x & 63);
  const int js = threadIdx.x >> 6;
  double v = 0.0;
  if (c < nv) {
    for (int J = js; J < nJ; J += NS) {
      const double* LJ = Lov + (int64_t)J * no * nv;
      double w = 2.0 * s[J] * LJ[(int64_t)k * nv + c];
      const double* MJ = M + (int64_t)J * no * no + (int64_t)k * no;
      for (int l = 0; l < no; ++l) w -= MJ[l] * LJ[(int64_t)l * nv + c];
      v += w;
    }
  }
  red[threadIdx.x] = v;
  __syncthreads();
  for (int h = NS / 2; h >= 1; h >>= 1) {
    if (js < h) red[threadIdx.x] += red[threadIdx.x + 64 * h];
    __syncthreads();
  }
  if (js == 0 && c < nv) F[(int64_t)k * nv + c] = red[threadIdx.x];
}

// Second launch: the Fock blocks first (they sum over J), then LvoT.  Two launches instead of
// five, since each is a few microseconds of latency at 4/20 (MEASURED, with the one-launch
// start of the triple loop and a single batch on the caller's stream: 166 -> 99 us a call).
__global__ __launch_bounds__(1024) void k_t1_second(const double* __restrict__ L,
                                                    const double* __restrict__ t1,
                                                    CholeskyScratch cs, double* __restrict__ F,
                                                    int no, int nv, int nJ) {
  __shared__ double Ls[VO_RC][VO_DC + 1];
  __shared__ double Ts[64][VO_DC + 1];
  const int nf = no * ((nv + 63) / 64), nc = (nv + VO_RC - 1) / VO_RC;
  const int bx = blockIdx.x;
  if (bx < nf) fock(cs.Lov, cs.s, cs.M, F, &Ls[0][0], bx % no, bx / no, no, nv, nJ);
  else t1_vo(L, t1, cs.Loo, cs.LvoT, Ls, Ts, (bx - nf) / nc, (bx - nf) % nc, no, nv);
}
static_assert(VO_RC * (VO_DC + 1) >= 64 * 16, "the Fock sums use Ls");

void launch_t1_fock(const double* L, const double* t1, const CholeskyScratch& cs, double* F, int no,
                    int nv, int nJ, hipStream_t st) {
  const int nvv = (int)nblk((int64_t)nv * nv, 256);
  const int noo = (int)nblk(no * std::max(no, nv), 256);
  hipLaunchKernelGGL(k_t1_first, dim3(nvv + noo + 1, nJ), dim3(256), 0, st, L, t1, cs, nvv, noo, no,
                     nv);
  hipLaunchKernelGGL(k_t1_second, dim3(no * nblk(nv, 64) + nblk(nv, VO_RC) * nJ), dim3(1024), 0, st,
                     L, t1, cs, F, no, nv, nJ);
}

// ---------------------------------------------------------------------------
// Integral-block build: C[m][n] = sum_J A(m, J) B(J, n) on FP64 MFMA, with an output
// map per block kind:
//   BUILD_PLAIN  C[m][n]
//   BUILD_JO     m = q nv + b, n = r nv + c -> Jo[q][r][b][c]
//   BUILD_HS     m = q no + l, n = r nv + c -> Hs[q][r][c][l] = delta_lq F[r][c] - value
//   BUILD_GO     m = q no + l, n = r nv + z -> Go[q][r][z][l]
//   BUILD_GW     m = z, n = y nv + d        -> Gw[y][z][d] (batch r)
//   BUILD_GBC    m = n' nv + b, n = c       -> G[n'][b][c], zeros in the padding of c
enum BuildKind {
  BUILD_PLAIN = 0, BUILD_JO = 1, BUILD_HS = 2, BUILD_GO = 3, BUILD_GW = 4, BUILD_GBC = 5
};

// One product of a grouped build launch: C_z = A_z B_z for z < batch, with
// A(m, J) at A[z * a_bs + m + J * a_sk], B(J, n) at B[z * b_bs + J * b_sk + n], both
// with J < K rows in all.
struct BuildProb {
  const double* A;
  const double* B;
  double* C;
  int64_t a_sk, a_bs, b_sk, b_bs, c_bs;
  int M, N, kind, batch;
};
enum { MAX_BUILD_PROBS = 6 };
// The products of one launch, all with the same K; wave tiles first0[p] ..
// first0[p + 1] - 1 are those of product p.
struct BuildSet {
  BuildProb p[MAX_BUILD_PROBS];
  unsigned first0[MAX_BUILD_PROBS + 1];
  int n, K, no, nv;
  const double* F;
};

// One wavefront per FM x FN blocks of 16 x 16 outputs, without LDS, as in the W build: 8 k
// (rows J of both operands) per unit, two units in flight.  Rows m and columns n are the
// contiguous ones here: per k the A rows load as pairs (block 2 f the even rows and block
// 2 f + 1 the odd rows of 32), the B columns 16 in a row, so that the stores run along n.
// Rows J >= K lie past the resources, which give zeros.  Bound by the loads (per MFMA as in
// the W build, both operands streamed) and by the writes of the blocks, no nv^3 twice.
// 128 x 128 LDS tiles before -> now: 28.1 -> 23.4 ms at 23/250/800, 61.7 -> 43.0 at
// 8/400/1200, 8.1 -> 4.6 at 9/187/588, 23 -> 10 us at 4/20/60.
template <int FM, int FN>
__global__ __launch_bounds__(256, FM * FN <= 4 ? 4 : FM * FN <= 9 ? 3 : 2) void k_build(
    const BuildSet set) {
  const unsigned item = xcd_item(blockIdx.x, gridDim.x, 4u) * 4u +
                        __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  if (item >= set.first0[set.n]) return;
  int pi = 0;
  while (pi + 1 < set.n && item >= set.first0[pi + 1]) ++pi;
  const BuildProb& pr = set.p[pi];
  const int M = pr.M, N = pr.N, K = set.K, kind = pr.kind, no = set.no, nv = set.nv;
  const unsigned mt = (unsigned)(M + 16 * FM - 1) / (16 * FM), nt = (unsigned)(N + 16 * FN - 1) / (16 * FN);
  const unsigned local = item - set.first0[pi], z = local / (mt * nt), t = local % (mt * nt);
  // the shorter dimension fastest: neighbours share the rows of the longer one
  const int m0 = (int)(mt <= nt ? t % mt : t / nt) * (16 * FM);
  const int n0 = (int)(mt <= nt ? t / mt : t % nt) * (16 * FN);
  const int lane = threadIdx.x & 63, r16 = lane & 15, kq = lane >> 4;
  const double* pa = pr.A + z * pr.a_bs + m0;
  const double* pb = pr.B + z * pr.b_bs + n0;
  int64_t na = K * pr.a_sk - (int64_t)z * pr.a_bs - m0, nb = K * pr.b_sk - (int64_t)z * pr.b_bs - n0;
  const int64_t sa = 8 * pr.a_sk, sb = 8 * pr.b_sk;  // doubles per unit
  const unsigned ka = (unsigned)pr.a_sk * 8u, kb = (unsigned)pr.b_sk * 8u;  // bytes per k
  const unsigned va = (unsigned)(2 * kq) * ka + (unsigned)r16 * 16u;
  const unsigned va1 = (unsigned)(2 * kq) * ka + (unsigned)r16 * 8u;  // an odd last block
  const unsigned vb = (unsigned)(2 * kq) * kb + (unsigned)r16 * 8u;
  double a[2][FM][2], b[2][FN][2];
  auto fetch = [&](double (&fa)[FM][2], double (&fb)[FN][2]) {
    const BufRsrc ra = buf_rsrc_n(pa, na > 0 ? na : 0), rb = buf_rsrc_n(pb, nb > 0 ? nb : 0);
#pragma unroll
    for (int t = 0; t < 2; ++t) {
#pragma unroll
      for (int f = 0; f + 1 < FM; f += 2) {
        const d2v v = buf_load_2f64(ra, va + (unsigned)t * ka, (unsigned)f * 128u);
        fa[f][t] = v[0];
        fa[f + 1][t] = v[1];
      }
      if constexpr (FM & 1) fa[FM - 1][t] = buf_load_f64(ra, va1 + (unsigned)t * ka + (FM - 1) * 128u);
#pragma unroll
      for (int f = 0; f < FN; ++f) fb[f][t] = buf_load_f64(rb, vb + (unsigned)t * kb + f * 128u);
    }
    pa += sa;
    pb += sb;
    na -= sa;
    nb -= sb;
  };
  d4v acc[FM][FN];
#pragma unroll
  for (int fm = 0; fm < FM; ++fm)
#pragma unroll
    for (int fn = 0; fn < FN; ++fn) acc[fm][fn] = d4v{0.0, 0.0, 0.0, 0.0};
  const int units = (K + 7) / 8;
  fetch(a[0], b[0]);
  fetch(a[1], b[1]);
  for (int u = 0; u < units; u += 2) {
#pragma unroll
    for (int d = 0; d < 2; ++d) {
      if (u + d < units) {
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
  // output (m, n) of every kind is at row(m) + col(n)
  double* Cz = pr.C + z * pr.c_bs;
  const int rp = cube_pitch(nv), nlim = kind == BUILD_GBC ? rp : N;
  int64_t col[FN];
#pragma unroll
  for (int fn = 0; fn < FN; ++fn) {
    const int n = n0 + fn * 16 + r16;
    col[fn] = n;                                                       // [..][n]
    if (kind == BUILD_JO) col[fn] = n / nv * (int64_t)nv * nv + n % nv;  // n = r nv + c
    else if (kind == BUILD_HS || kind == BUILD_GO) col[fn] = (int64_t)n * no;  // [r][c][l]
    else if (kind == BUILD_GW) col[fn] = n / nv * gw_pitch(nv) + n % nv;  // n = y nv + d
  }
#pragma unroll
  for (int fm = 0; fm < FM; ++fm)
#pragma unroll
    for (int r = 0; r < 4; ++r) {
      const int m = m0 + ((FM & 1) && fm == FM - 1
                              ? fm * 16 + kq + 4 * r
                              : (fm & ~1) * 16 + 2 * (kq + 4 * r) + (fm & 1));
      int64_t row = (int64_t)m * N;             // BUILD_PLAIN: C[m][n]
      if (kind == BUILD_GBC) row = m / nv * g_pitch(nv) + (int64_t)(m % nv) * rp;  // m = n' nv + b
      else if (kind == BUILD_JO) row = (m / nv * (int64_t)no * nv + m % nv) * nv;  // m = q nv + b
      else if (kind == BUILD_HS || kind == BUILD_GO)
        row = m / no * (int64_t)no * nv * no + m % no;                             // m = q no + l
      else if (kind == BUILD_GW) row = (int64_t)m * nv;                            // m = z
      const bool diag = kind == BUILD_HS && m / no == m % no;
#pragma unroll
      for (int fn = 0; fn < FN; ++fn) {
        const int n = n0 + fn * 16 + r16;
        double v = n < N ? acc[fm][fn][r] : 0.0;  // zeros in the padding of BUILD_GBC
        if (kind == BUILD_HS) v = (diag && m < M && n < N ? set.F[n] : 0.0) - v;
        if (m < M && n < nlim) Cz[row + col[fn]] = v;
      }
    }
}

static void add_build(BuildSet& set, const double* A, int64_t a_sk, int64_t a_bs, const double* B,
                      int64_t b_sk, int64_t b_bs, int M, int N, double* C, int64_t c_bs, int batch,
                      int kind) {
  BuildProb& p = set.p[set.n++];
  p.A = A; p.a_sk = a_sk; p.a_bs = a_bs;
  p.B = B; p.b_sk = b_sk; p.b_bs = b_bs;
  p.C = C; p.c_bs = c_bs;
  p.M = M; p.N = N; p.kind = kind; p.batch = batch;
}

template <int FM, int FN>
static void launch_build_shape(BuildSet& set, hipStream_t st) {
  if (set.n == 0) return;
  set.first0[0] = 0;
  for (int i = 0; i < set.n; ++i) {
    const BuildProb& p = set.p[i];
    set.first0[i + 1] = set.first0[i] + nblk(p.M, 16 * FM) * nblk(p.N, 16 * FN) * (unsigned)p.batch;
  }
  hipLaunchKernelGGL((k_build<FM, FN>), dim3(nblk(set.first0[set.n], 4)), dim3(256), 0, st, set);
}

// Blocks of 16 along nv per wave tile: 2, 3, 4 or 5, the least blocks in all, weighted by
// the loads per MFMA as the wave-tile shapes of the W build.
static int build_blocks_nv(int nv) {
  int best = 4;
  double cost = 0.0;
  for (int f = 2; f <= 5; ++f) {
    const double c = (double)nblk(nv, 16 * f) * f * (0.65 + 0.7 * (1.0 / f + (f == 2 ? 0.5 : f == 3 ? 1.0 / 3 : 0.25)));
    if (f == 2 || c < cost) { best = f; cost = c; }
  }
  return best;
}

// The products of `set`: square wave tiles and one launch for 2, 3 and 4 blocks along nv;
// for 5 the products with nv rows (5 x 4) and those with nv columns (4 x 5) in two.
static void launch_build_set(const BuildSet& set, hipStream_t st) {
  const int f = build_blocks_nv(set.nv);
  BuildSet rows = set, cols = set;
  rows.n = cols.n = 0;
  for (int i = 0; i < set.n; ++i) {
    BuildSet& to = f == 5 && set.p[i].M <= set.p[i].N ? rows : cols;
    to.p[to.n++] = set.p[i];
  }
  if (f == 2) launch_build_shape<2, 2>(cols, st);
  else if (f == 4) launch_build_shape<4, 4>(cols, st);
  else if (f == 3) launch_build_shape<3, 3>(cols, st);
  else {
    launch_build_shape<5, 4>(rows, st);
    launch_build_shape<4, 5>(cols, st);
  }
}

// Gcb[r][n][c][b] = Gbc[r][n][b][c]: nv x nv transposes, one per (r, n), through
// padded 32 x 32 LDS tiles; ss and ds: doubles between the slabs, rs and rd: between the
// rows of a slab (past nv, the rows of dst are filled with zeros).
__global__ __launch_bounds__(256) void k_gcb(const double* __restrict__ Gbc,
                                             double* __restrict__ Gcb, int nv, int64_t ss,
                                             int64_t ds, int rs, int rd) {
  __shared__ double t[32][33];
  const int tn = (nv + 31) / 32;
  const int64_t slab = blockIdx.x / (tn * tn);  // r * (nv + no) + n
  const int tile = blockIdx.x % (tn * tn);
  const int b0 = (tile / tn) * 32, c0 = (tile % tn) * 32;
  const double* src = Gbc + slab * ss;
  double* dst = Gcb + slab * ds;
  const int tx = threadIdx.x & 31, ty = threadIdx.x >> 5;
  for (int y = ty; y < 32; y += 8) {
    const int b = b0 + y, c = c0 + tx;
    if (b < nv && c < nv) t[y][tx] = src[(int64_t)b * rs + c];
  }
  __syncthreads();
  for (int y = ty; y < 32; y += 8) {
    const int c = c0 + y, b = b0 + tx;
    if (b < rd && c < nv) dst[(int64_t)c * rd + b] = b < nv ? t[tx][y] : 0.0;
  }
}

void launch_gcb(const Blocks& bl, int no, int nv, hipStream_t st) {
  const unsigned t = nblk(nv, 32);
  hipLaunchKernelGGL(k_gcb, dim3(t * t * no * (nv + no)), dim3(256), 0, st, bl.Gbc, bl.Gcb, nv,
                     g_pitch(nv), g_pitch(nv), cube_pitch(nv), cube_pitch(nv));
}

void launch_build_blocks(const CholeskyScratch& cs, const Blocks& bl, int no, int nv, int nJ,
                         hipStream_t st) {
  const int64_t nv2 = (int64_t)nv * nv, onv = (int64_t)no * nv;
  const int64_t gs = (nv + no) * g_pitch(nv);  // one r slab of Gbc / Gcb
  // all six products share K = nJ
  BuildSet set = {};
  set.K = nJ; set.no = no; set.nv = nv; set.F = bl.F;
  // Gw[r][y][z][d] = sum_J LvoT[J][r][z] Lvv[J][(y,d)]   (rows z, columns (y,d), batch r)
  add_build(set, cs.LvoT, onv, nv, cs.Lvv, nv2, 0, nv, (int)nv2, bl.Gw, nv * gw_pitch(nv), no,
            BUILD_GW);
  // Gbc[r][(d,b)][c] = sum_J Lvv[J][(d,b)] Lov[J][r][c]            (rows n = d < nv)
  add_build(set, cs.Lvv, nv2, 0, cs.Lov, onv, nv, (int)nv2, nv, bl.Gbc, gs, no, BUILD_GBC);
  // Gbc[r][nv + (l,b)][c] = sum_J Lov[J][(l,b)] Lov[J][r][c]      (rows n = nv + l)
  add_build(set, cs.Lov, onv, 0, cs.Lov, onv, nv, (int)onv, nv, bl.Gbc + nv * g_pitch(nv), gs, no,
            BUILD_GBC);
  // Jo[q][r][b][c] = sum_J Lov[J][q][b] Lov[J][r][c]
  add_build(set, cs.Lov, onv, 0, cs.Lov, onv, 0, (int)onv, (int)onv, bl.Jo, 0, 1, BUILD_JO);
  // Hs[q][r][c][l] = delta_lq F[r][c] - sum_J Loo[J][q][l] Lov[J][r][c]
  add_build(set, cs.Loo, (int64_t)no * no, 0, cs.Lov, onv, 0, no * no, (int)onv, bl.Hs, 0, 1,
            BUILD_HS);
  // Go[q][r][z][l] = sum_J LooT[J][q][l] LvoT[J][r][z]   (LooT[J][q][l] = Lt_lq)
  add_build(set, cs.LooT, (int64_t)no * no, 0, cs.LvoT, onv, 0, no * no, (int)onv, bl.Go, 0, 1,
            BUILD_GO);
  launch_build_set(set, st);
  launch_gcb(bl, no, nv, st);
}

// The blocks of the transition-density loop (Algorithm 3), in one grouped launch:
// Gw, Go and Jo as for the residual; Go3[p][q][z][l] = g_{plqz} = sum_J Lt_pl L_qz;
// Gl[p][y][z][d] = g_{pydz} = sum_J L_py Lt_dz, built as [p][y][d][z] into `tmp`
// (no nv^3 doubles) and transposed per (p, y) slab (Gl at the slab pitch of Gw).
void launch_build_density_blocks(const CholeskyScratch& cs, double* Gw, double* Go, double* Jo,
                                 double* Go3, double* Gl, double* tmp, int no, int nv, int nJ,
                                 hipStream_t st) {
  const int64_t nv2 = (int64_t)nv * nv, onv = (int64_t)no * nv;
  BuildSet set = {};
  set.K = nJ; set.no = no; set.nv = nv; set.F = nullptr;
  add_build(set, cs.LvoT, onv, nv, cs.Lvv, nv2, 0, nv, (int)nv2, Gw, nv * gw_pitch(nv), no, BUILD_GW);
  // tmp[(p,y)][(d,z)] = sum_J Lov[J][p][y] Lvv[J][d][z]
  add_build(set, cs.Lov, onv, 0, cs.Lvv, nv2, 0, (int)onv, (int)nv2, tmp, 0, 1, BUILD_PLAIN);
  add_build(set, cs.Lov, onv, 0, cs.Lov, onv, 0, (int)onv, (int)onv, Jo, 0, 1, BUILD_JO);
  add_build(set, cs.LooT, (int64_t)no * no, 0, cs.LvoT, onv, 0, no * no, (int)onv, Go, 0, 1,
            BUILD_GO);
  // Go3: m = p*no + l (Loo[J][p][l] = Lt_pl), n = q*nv + z (Lov[J][q][z] = L_qz)
  add_build(set, cs.Loo, (int64_t)no * no, 0, cs.Lov, onv, 0, no * no, (int)onv, Go3, 0, 1,
            BUILD_GO);
  launch_build_set(set, st);
  const unsigned t = nblk(nv, 32);
  hipLaunchKernelGGL(k_gcb, dim3(t * t * no * nv), dim3(256), 0, st, tmp, Gl, nv, nv2,
                     gw_pitch(nv), nv, nv);
}

// ---------------------------------------------------------------------------
// Integral blocks given in the paper's index order -> internal layouts.
// ---------------------------------------------------------------------------
__global__ void k_relayout_vv(const double* __restrict__ g_vvvo_y, const double* __restrict__ g_vvov_y,
                              double* __restrict__ Gw, double* __restrict__ Gbc, int no, int nv,
                              int y0, int ny) {
  // output index (r, y, d, z) of an nv^3 slab, z fastest, for y in [y0, y0 + ny);
  // the inputs start at first index y0
  const int64_t nv2 = (int64_t)nv * nv;
  const int64_t e = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  const int r = blockIdx.y;
  if (e >= (int64_t)ny * nv2) return;
  const int yl = (int)(e / nv2), d = (int)((e / nv) % nv), z = (int)(e % nv);
  // Gw[r][y][u][w] = g_vvvo[y][w][u][r]  (u = d, w = z: the contracted index w fastest)
  Gw[((int64_t)r * nv + y0 + yl) * gw_pitch(nv) + e % nv2] = g_vvvo_y[(((int64_t)yl * nv + z) * nv + d) * no + r];
  // Gbc[r][n=y][b=d][c=z] = g_vvov[n][b][r][c]
  double* gr = Gbc + ((int64_t)r * (nv + no) + y0 + yl) * g_pitch(nv) + (int64_t)d * cube_pitch(nv);
  if (z == nv - 1)
    for (int c = nv; c < cube_pitch(nv); ++c) gr[c] = 0.0;
  gr[z] = g_vvov_y[(((int64_t)yl * nv + d) * no + r) * nv + z];
}

__global__ void k_relayout_small(const double* __restrict__ g_oovo, const double* __restrict__ g_ovov,
                                 const double* __restrict__ g_ooov, const double* __restrict__ F_ov,
                                 double* __restrict__ Go, double* __restrict__ Jo,
                                 double* __restrict__ Gbc, double* __restrict__ Hs,
                                 double* __restrict__ F, int no, int nv) {
  const int q = blockIdx.y / no, r = blockIdx.y % no;
  const int64_t nv2 = (int64_t)nv * nv;
  for (int e = blockIdx.x * blockDim.x + threadIdx.x; e < nv * nv; e += gridDim.x * blockDim.x) {
    const int b = e / nv, c = e % nv;  // Jo[q][r][b][c] = Gbc[r][nv + q][b][c] = g_ovov[q][b][r][c]
    const double g = g_ovov[(((int64_t)q * nv + b) * no + r) * nv + c];
    Jo[((int64_t)q * no + r) * nv2 + e] = g;
    double* gr = Gbc + ((int64_t)r * (nv + no) + nv + q) * g_pitch(nv) + (int64_t)b * cube_pitch(nv);
    gr[c] = g;
    if (c == nv - 1)
      for (int p = nv; p < cube_pitch(nv); ++p) gr[p] = 0.0;
  }
  for (int e = blockIdx.x * blockDim.x + threadIdx.x; e < no * nv; e += gridDim.x * blockDim.x) {
    const int l = e / nv, c = e % nv;
    // Go[q][r][z][l] = g_oovo[l][q][z][r]
    Go[(((int64_t)q * no + r) * nv + c) * no + l] = g_oovo[(((int64_t)l * no + q) * nv + c) * no + r];
    // Hs[q][r][c][l] = delta_lq F[r][c] - g_ooov[q][l][r][c]
    Hs[(((int64_t)q * no + r) * nv + c) * no + l] =
        (l == q ? F_ov[(int64_t)r * nv + c] : 0.0) - g_ooov[(((int64_t)q * no + l) * no + r) * nv + c];
  }
  if (blockIdx.y == 0)
    for (int e = blockIdx.x * blockDim.x + threadIdx.x; e < no * nv; e += gridDim.x * blockDim.x)
      F[e] = F_ov[e];
}

void launch_relayout_small(const double* g_oovo, const double* g_ovov, const double* g_ooov,
                           const double* F_ov, const Blocks& b, int no, int nv, hipStream_t st) {
  unsigned gx = nblk((int64_t)nv * nv, 256);
  if (gx > 64) gx = 64;
  hipLaunchKernelGGL(k_relayout_small, dim3(gx, no * no), dim3(256), 0, st, g_oovo, g_ovov,
                     g_ooov, F_ov, b.Go, b.Jo, b.Gbc, b.Hs, b.F, no, nv);
}

void launch_relayout_vv(const double* g_vvvo_y, const double* g_vvov_y, int y0, int ny,
                        const Blocks& b, int no, int nv, hipStream_t st) {
  const int64_t n = (int64_t)ny * nv * nv;
  hipLaunchKernelGGL(k_relayout_vv, dim3(nblk(n, 256), no), dim3(256), 0, st, g_vvvo_y, g_vvov_y,
                     b.Gw, b.Gbc, no, nv, y0, ny);
}

// ---------------------------------------------------------------------------
// Triple table: the restricted loop i >= j >= k without the i == j == k triples,
// lexicographic rank L = C(i+2,3) + j(j+1)/2 + k - i, dealt round-robin over the
// nbatch batches: position = start of group L mod nbatch + L / nbatch.  Each
// batch then samples the whole loop, so that the (triple, permutation) pairs of
// a batch spread evenly over the first occupied index, which the
// output-stationary kernels are parallel over.
// ---------------------------------------------------------------------------
__device__ __forceinline__ void triple_entry(int* __restrict__ tri, int e, int no, int nbatch) {
  const int i = e / (no * no), j = (e / no) % no, k = e % no;
  if (!(i >= j && j >= k) || (i == j && j == k)) return;
  const int n = no * (no + 1) * (no + 2) / 6 - no;
  const int L = i * (i + 1) * (i + 2) / 6 + j * (j + 1) / 2 + k - i;
  const int g = L % nbatch;
  const int pos = g * (n / nbatch) + min(g, n % nbatch) + L / nbatch;
  tri[3 * pos + 0] = i;
  tri[3 * pos + 1] = j;
  tri[3 * pos + 2] = k;
}

// What a triple loop starts from, in one launch: the triple table (tri, unless null), zeros
// (n of them at Z) and t2N[p][y][x][l] = -t2[p][l][x][y], the slab (p, y) at t2n_pitch.
__global__ void k_loop_begin(int* __restrict__ tri, int nbatch, double* __restrict__ Z, int64_t n,
                             const double* __restrict__ t2, double* __restrict__ t2N, int no,
                             int nv) {
  const int64_t nvl = nv, n2 = (int64_t)no * no * nvl * nvl, stride = (int64_t)gridDim.x * blockDim.x;
  const int64_t e0 = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (tri && e0 < no * no * no) triple_entry(tri, (int)e0, no, nbatch);
  for (int64_t e = e0; e < n2; e += stride) {
    const int l = (int)(e % no), x = (int)((e / no) % nvl), y = (int)((e / (no * nvl)) % nvl);
    const int p = (int)(e / (no * nvl * nvl));
    t2N[((int64_t)p * nvl + y) * t2n_pitch(no, nv) + (int64_t)x * no + l] =
        -t2[(((int64_t)p * no + l) * nvl + x) * nvl + y];
  }
  for (int64_t e = e0; e < n; e += stride) Z[e] = 0.0;
}

void launch_loop_begin(int* tri, int nbatch, double* Z, int64_t n, const double* t2, double* t2N,
                       int no, int nv, hipStream_t st) {
  const int64_t m = std::max((int64_t)no * no * nv * nv, (int64_t)no * no * no);
  hipLaunchKernelGGL(k_loop_begin, dim3(nblk(m, 256)), dim3(256), 0, st, tri, nbatch < 1 ? 1 : nbatch,
                     Z, n, t2, t2N, no, nv);
}

void launch_set_triples(int* tri_dev, const int* host_tri, int n, hipStream_t st) {
  hipMemcpyAsync(tri_dev, host_tri, sizeof(int) * 3 * (size_t)n, hipMemcpyHostToDevice, st);
}

// ---------------------------------------------------------------------------
// Covariant back-transformation.  The contravariant doubles residual is held
// in two parts, Ot~[i][j][a][b] = Ot2[i][j][a][b] + OtT[i][j][b][a]; then
//   Omega^a_i = Ot^a_i
//   Omega^{ab}_{ij} = 1/3 [(2 Ot~^{ab}_{ij} + Ot~^{ba}_{ij}) + (2 Ot~^{ba}_{ji} + Ot~^{ab}_{ji})]
// ---------------------------------------------------------------------------
__device__ inline double ot2(const double* __restrict__ Ot2, const double* __restrict__ OtT,
                             int64_t ij, int64_t nv, int a, int b) {
  return Ot2[(ij + a) * nv + b] + OtT[(ij + b) * nv + a];
}

__global__ void k_back(const double* __restrict__ Ot1, const double* __restrict__ Ot2,
                       const double* __restrict__ OtT, double* __restrict__ O1,
                       double* __restrict__ O2, int no, int nv, int acc) {
  const int64_t nvl = nv, n2 = (int64_t)no * no * nvl * nvl;
  const int64_t e = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (e < n2) {
    const int b = (int)(e % nvl), a = (int)((e / nvl) % nvl);
    const int j = (int)((e / (nvl * nvl)) % no), i = (int)(e / (nvl * nvl * no));
    const int64_t ij = ((int64_t)i * no + j) * nvl, ji = ((int64_t)j * no + i) * nvl;
    const double v = (2.0 * ot2(Ot2, OtT, ij, nvl, a, b) + ot2(Ot2, OtT, ij, nvl, b, a) +
                      2.0 * ot2(Ot2, OtT, ji, nvl, b, a) + ot2(Ot2, OtT, ji, nvl, a, b)) / 3.0;
    O2[e] = acc ? O2[e] + v : v;
  }
  if (e < (int64_t)no * nv) O1[e] = acc ? O1[e] + Ot1[e] : Ot1[e];
}

void launch_back_transform(const double* Ot1, const double* Ot2, const double* OtT, double* O1,
                           double* O2, int no, int nv, bool accumulate, hipStream_t st) {
  const int64_t n2 = (int64_t)no * no * nv * nv;
  hipLaunchKernelGGL(k_back, dim3(nblk(n2, 256)), dim3(256), 0, st, Ot1, Ot2, OtT, O1, O2, no, nv,
                     accumulate ? 1 : 0);
}

__global__ void k_combine(const double* __restrict__ Ot1, const double* __restrict__ Ot2,
                          const double* __restrict__ OtT, double* __restrict__ O1,
                          double* __restrict__ O2, int no, int nv) {
  const int64_t nvl = nv, n2 = (int64_t)no * no * nvl * nvl;
  const int64_t e = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (e < n2) {
    const int b = (int)(e % nvl), a = (int)((e / nvl) % nvl);
    O2[e] = ot2(Ot2, OtT, (e / (nvl * nvl)) * nvl, nvl, a, b);
  }
  if (e < (int64_t)no * nv) O1[e] = Ot1[e];
}

void launch_combine(const double* Ot1, const double* Ot2, const double* OtT, double* O1,
                    double* O2, int no, int nv, hipStream_t st) {
  const int64_t n2 = (int64_t)no * no * nv * nv;
  hipLaunchKernelGGL(k_combine, dim3(nblk(n2, 256)), dim3(256), 0, st, Ot1, Ot2, OtT, O1, O2, no,
                     nv);
}

// ---------------------------------------------------------------------------
// Input checks (CC3_CHECK): pair symmetry of t2, symmetry of L in (p, q), and
// positive denominators (3 min e_vir - 3 max e_occ > 0).  Sets bits of *flag.
// ---------------------------------------------------------------------------
__device__ inline bool differs(double x, double y) {
  const double s = fmax(fabs(x), fabs(y));
  return fabs(x - y) > 1e-12 * s;
}

__global__ void k_check(const double* __restrict__ eps, const double* __restrict__ L,
                        const double* __restrict__ t2, int no, int nv, int nJ, int* flag) {
  const int64_t stride = (int64_t)gridDim.x * blockDim.x;
  const int64_t e0 = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  const int64_t nvl = nv, n2 = (int64_t)no * no * nvl * nvl;
  int bits = 0;
  for (int64_t e = e0; e < n2; e += stride) {
    const int b = (int)(e % nvl), a = (int)((e / nvl) % nvl);
    const int j = (int)((e / (nvl * nvl)) % no), i = (int)(e / (nvl * nvl * no));
    if (differs(t2[e], t2[(((int64_t)j * no + i) * nvl + b) * nvl + a])) bits |= 1;
  }
  if (L) {
    const int64_t nmo = no + nv, nl = (int64_t)nJ * nmo * nmo;
    for (int64_t e = e0; e < nl; e += stride) {
      const int64_t q = e % nmo, pp = (e / nmo) % nmo, J = e / (nmo * nmo);
      if (differs(L[e], L[(J * nmo + q) * nmo + pp])) bits |= 2;
    }
  }
  if (e0 == 0) {
    double emax = eps[0], vmin = eps[no];
    for (int i = 1; i < no; ++i) emax = fmax(emax, eps[i]);
    for (int a = 1; a < nv; ++a) vmin = fmin(vmin, eps[no + a]);
    if (!(3.0 * vmin - 3.0 * emax > 0.0)) bits |= 4;
  }
  if (bits) atomicOr(flag, bits);
}

__global__ void k_zero_int(int* p) { *p = 0; }

void launch_check(const double* eps, const double* L, const double* t2, int no, int nv, int nJ,
                  int* flag, hipStream_t st) {
  hipLaunchKernelGGL(k_zero_int, dim3(1), dim3(1), 0, st, flag);
  hipLaunchKernelGGL(k_check, dim3(1024), dim3(256), 0, st, eps, L, t2, no, nv, nJ, flag);
}

}  // namespace cc3
