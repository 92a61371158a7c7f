// The transition-density loop (Algorithm 3, the triples contributions to
// D^{m,0}) on the caller's stream: workspace plan, the batched loop, and its C-ABI entry
// points.
//
// Each triple's t3 (W build, mix) and left-state L3 (the same engine with the L3
// operands, the mix with the outer products and the (omega - eps) denominator) feed the
// contractions of kern_density.hip.  Two loops:
//  - resident: the unordered triples in batches, every cube of tau and L~ kept, then the
//    Gram matrices of every occupied pair for D_lk from the kept cubes.  Each triple is
//    built once.
//  - by pairs: each pair (i, j), i >= j, is one batch holding the ordered triples
//    (i, j, k) for every k and contributes its Gram matrix at once; each unordered triple
//    is sorted in exactly one pair and contributes its D_cd, Y^o and D_kc terms there, but
//    is built in each of its up to three pairs.
// The resident loop needs no (no + 1) (no + 2) / 3 cubes.  It is taken where they fit the
// cube budget (64 GiB, two of the residual's buffer sets) and the caller's workspace;
// a smaller workspace, down to that of the loop by pairs, takes the latter.  At 12/120/400
// (10 GB of cubes) the resident loop builds 364 triples where the loop by pairs builds 936.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <cstdlib>
#include <vector>

#include "cc3_density.hpp"
#include "cc3_host.hpp"

using namespace cc3;

namespace {

size_t a256(size_t x) { return (x + 255) & ~(size_t)255; }

struct DPlan {
  int no, nv, nchol, npairs;
  bool resident;
  int nall;     // triples of the loop's table
  int batch;    // most triples of a batch
  size_t cube;  // doubles per cube (cube_slot: nv x nv rows at the padded pitch)
  size_t off_Gw, off_Gl, off_Go, off_Go3, off_Jo, off_F, off_t2N, off_l2M, off_E, off_Y;
  size_t off_part, off_tri, off_planes, off_tau, off_lc, off_cubes;
  size_t chol_bytes;
  size_t total;
  std::vector<int> htri;  // [triple][3]: unordered, lexicographic, or [pair][k]
};

size_t cube_budget() {
  const char* e = getenv("CC3_CUBE_BUDGET_MB");  // per buffer set, as for the residual
  const long v = e ? atol(e) : 0;
  return (size_t)(v > 0 ? v : 32768) << 21;
}

void make_dplan(int no, int nv, int nchol, bool resident, DPlan* p) {
  const size_t o = no, v = nv, J = nchol;
  p->no = no; p->nv = nv; p->nchol = nchol;
  p->cube = (size_t)cube_slot(nv);  // one padded cube
  p->npairs = no * (no + 1) / 2;
  p->resident = resident;
  p->htri.clear();
  for (int i = 0; i < no; ++i)
    for (int j = 0; j <= i; ++j)
      for (int k = 0; k < (resident ? j + 1 : no); ++k) {
        p->htri.push_back(i); p->htri.push_back(j); p->htri.push_back(k);
      }
  p->nall = (int)p->htri.size() / 3;
  if (resident) {
    // about 16384 wave tiles of the W build per launch (eight rounds), the planes of a
    // batch within 4 GiB
    int tm, tn;
    shape_tiles(pick_shape(nv, nv), nv, nv, &tm, &tn);
    const int64_t per = 2ll * nv * tm * tn;
    int64_t b = std::min<int64_t>(D3_MAXB, (16384 + per - 1) / per);
    b = std::min<int64_t>(std::max<int64_t>(b, 4), ((size_t)4 << 30) / (16 * p->cube));
    b = std::max<int64_t>(1, std::min<int64_t>(b, p->nall));
    const int64_t nb = (p->nall + b - 1) / b;  // balanced
    p->batch = (int)((p->nall + nb - 1) / nb);
  } else {
    p->batch = no;
  }
  size_t off = 0;
  auto take = [&](size_t bytes) { size_t at = off; off = a256(off + bytes); return at; };
  p->off_Gw = take(o * v * gw_pitch(nv) * 8);
  p->off_Gl = take(o * v * gw_pitch(nv) * 8);
  p->off_Go = take(o * o * o * v * 8);
  p->off_Go3 = take(o * o * o * v * 8);
  p->off_Jo = take(o * o * v * v * 8);
  p->off_F = take(o * v * 8);
  p->off_t2N = take(o * v * t2n_pitch(no, nv) * 8);
  p->off_l2M = take(o * v * t2n_pitch(no, nv) * 8);
  p->off_E = take(o * o * v * v * 8);
  p->off_Y = take(o * o * o * v * 8);
  p->off_part = take(d3_partial_doubles(no, nv, p->batch, resident ? p->npairs : 1) * 8);
  p->off_tri = take(p->htri.size() * sizeof(int));
  // the planes (PA, then PB) of a batch, then the cubes of tau and L~; before the loop
  // the Cholesky scratch and the build's temporary (vv|ov) block use the same region
  p->chol_bytes = a256(J * v * v * 8) + a256(J * o * o * 8) * 2 + a256(J * o * v * 8) * 2 +
                  a256(J * 8) + a256(J * o * o * 8);
  const size_t kept = resident ? (size_t)p->nall : o, cb = p->cube * 8;
  const size_t planes = a256(2 * (size_t)p->batch * cb), one = a256(kept * cb);
  p->off_cubes = take(std::max(planes + 2 * one, p->chol_bytes + a256(o * v * v * v * 8)));
  p->off_planes = p->off_cubes;
  p->off_tau = p->off_cubes + planes;
  p->off_lc = p->off_tau + one;
  p->total = off;
}

// Whether the resident loop's cubes fit the budget.  (no = 1 has no triple to share between
// pairs, and the loop by pairs skips the contractions of its one, all-equal triple.)
bool resident_fits(int no, int nv) {
  if (no == 1) return false;
  const size_t n = (size_t)no * (no + 1) * (no + 2) / 6;
  return 2 * n * (size_t)cube_slot(nv) * 8 <= cube_budget();
}

int check_density_sizes(int no, int nv, int nchol) {
  int rc = check_sizes(no, nv, nchol, CC3_FP64);
  if (rc) return rc;
  if (nchol < 1) return fail(CC3_E_INVAL, "nchol must be >= 1 (got %d)", nchol);
  if (nv > 400)
    return fail(CC3_E_INVAL, "the transition-density loop supports nv <= 400 (got %d)", nv);
  return CC3_OK;
}

}  // namespace

extern "C" int cc3_transition_density_workspace_size(int no, int nv, int nchol, size_t* bytes) {
  if (!bytes) return fail(CC3_E_INVAL, "cc3_transition_density_workspace_size: bytes is NULL");
  int rc = check_density_sizes(no, nv, nchol);
  if (rc) return rc;
  DPlan p;
  make_dplan(no, nv, nchol, false, &p);
  *bytes = p.total;
  if (resident_fits(no, nv)) {
    make_dplan(no, nv, nchol, true, &p);
    *bytes = std::max(*bytes, p.total);
  }
  return CC3_OK;
}

extern "C" int cc3_transition_density_workspace_min(int no, int nv, int nchol, size_t* bytes) {
  if (!bytes) return fail(CC3_E_INVAL, "cc3_transition_density_workspace_min: bytes is NULL");
  int rc = check_density_sizes(no, nv, nchol);
  if (rc) return rc;
  DPlan p;
  make_dplan(no, nv, nchol, false, &p);
  *bytes = p.total;
  if (resident_fits(no, nv)) {
    make_dplan(no, nv, nchol, true, &p);
    *bytes = std::min(*bytes, p.total);
  }
  return CC3_OK;
}

extern "C" int cc3_transition_density(cc3_ctx* c, int no, int nv, int nchol, const double* eps,
                                      const double* L, const double* t1, const double* t2,
                                      const double* l1, const double* l2, double omega,
                                      double* D_cd, double* D_kc, double* D_ld, double* D_lk,
                                      double* Yo, unsigned flags, void* ws, size_t ws_bytes,
                                      cc3_stream_t stream) {
  if (!c) return fail(CC3_E_INVAL, "ctx is NULL");
  int rc = check_density_sizes(no, nv, nchol);
  if (rc) return rc;
  if (flags & ~(unsigned)(CC3_ACCUMULATE | CC3_DETERMINISTIC))
    return fail(CC3_E_INVAL, "flags 0x%x: cc3_transition_density accepts CC3_ACCUMULATE and "
                "CC3_DETERMINISTIC", flags);
  HIPCHK(hipSetDevice(c->device));
  const void* ptrs[] = {eps, L, t1, t2, l1, l2, D_cd, D_kc, D_ld, D_lk, ws};
  const char* names[] = {"eps", "L", "t1", "t2", "l1", "l2", "D_cd", "D_kc", "D_ld", "D_lk",
                         "workspace"};
  for (int i = 0; i < 11; ++i)
    if ((rc = check_dev_ptr(ptrs[i], names[i]))) return rc;
  if (Yo && (rc = check_dev_ptr(Yo, "Yo"))) return rc;
  if (((uintptr_t)ws) & 255) return fail(CC3_E_INVAL, "workspace must be 256-byte aligned");
  DPlan p;
  p.total = (size_t)-1;
  if (resident_fits(no, nv)) make_dplan(no, nv, nchol, true, &p);
  if (ws_bytes < p.total) make_dplan(no, nv, nchol, false, &p);
  if (ws_bytes < p.total)
    return fail(CC3_E_NOMEM, "workspace too small: %zu bytes given, %zu needed", ws_bytes, p.total);
  const bool acc = (flags & CC3_ACCUMULATE) != 0;
  hipStream_t st = (hipStream_t)stream;
  char* base = (char*)ws;
  double* Gw = (double*)(base + p.off_Gw);
  double* Gl = (double*)(base + p.off_Gl);
  double* Go = (double*)(base + p.off_Go);
  double* Go3 = (double*)(base + p.off_Go3);
  double* Jo = (double*)(base + p.off_Jo);
  double* F = (double*)(base + p.off_F);
  double* t2N = (double*)(base + p.off_t2N);
  double* l2M = (double*)(base + p.off_l2M);
  double* Y = (double*)(base + p.off_Y);
  double* E = (double*)(base + p.off_E);
  double* Ppart = (double*)(base + p.off_part);
  int* dtri = (int*)(base + p.off_tri);
  double* planes = (double*)(base + p.off_planes);
  double* tau = (double*)(base + p.off_tau);
  double* lc = (double*)(base + p.off_lc);
  // the Cholesky scratch, then the temporary (vv|ov) block, in the cube region
  const size_t o = no, v = nv, J = nchol;
  CholeskyScratch cs;
  {
    char* cr = base + p.off_cubes;
    size_t at = 0;
    auto take = [&](size_t bytes) { double* q = (double*)(cr + at); at = a256(at + bytes); return q; };
    cs.Lvv = take(J * v * v * 8);
    cs.Loo = take(J * o * o * 8);
    cs.LooT = take(J * o * o * 8);
    cs.LvoT = take(J * o * v * 8);
    cs.Lov = take(J * o * v * 8);
    cs.s = take(J * 8);
    cs.M = take(J * o * o * 8);
  }
  double* gtmp = (double*)(base + p.off_cubes + p.chol_bytes);
  const int64_t csl = (int64_t)p.cube;
  std::lock_guard<std::mutex> g(c->mu);
  Profiler* pf = &c->prof;
  HIPCHK(hipMemcpyAsync(dtri, p.htri.data(), p.htri.size() * sizeof(int), hipMemcpyHostToDevice,
                        st));
  HIPCHK(hipStreamSynchronize(st));  // the host table may go out of scope
  {
    Timer tm(pf, st, FAM_T1, 0.0, 0.0);
    launch_t1_fock(L, t1, cs, F, no, nv, nchol, st);
  }
  {
    const double fl = 2.0 * J * (2.0 * v * v * v * o + o * o * v * v + 2.0 * o * o * o * v);
    Timer tm(pf, st, FAM_BUILD, fl, 0.0);
    launch_build_density_blocks(cs, Gw, Go, Jo, Go3, Gl, gtmp, no, nv, nchol, st);
  }
  launch_loop_begin(nullptr, 1, nullptr, 0, t2, t2N, no, nv, st);
  launch_d3_l2(l2, l2M, E, no, nv, st);
  launch_fill(Y, (int64_t)o * o * o * v, 0.0, st);
  if (!acc) {
    launch_fill(D_cd, (int64_t)v * v, 0.0, st);
    launch_fill(D_kc, (int64_t)o * v, 0.0, st);
    launch_fill(D_ld, (int64_t)o * v, 0.0, st);
    launch_fill(D_lk, (int64_t)o * o, 0.0, st);
  }
  std::vector<int> kinds;
  const int ngroups = p.resident ? (p.nall + p.batch - 1) / p.batch : p.npairs;
  for (int g = 0; g < ngroups; ++g) {
    const int t0 = g * p.batch, nb = std::min(p.batch, p.nall - t0);
    const int* tb = dtri + (size_t)t0 * 3;
    const int* hb = p.htri.data() + (size_t)t0 * 3;
    double* bt = p.resident ? tau + t0 * csl : tau;
    double* bl = p.resident ? lc + t0 * csl : lc;
    double* PB = planes + nb * csl;
    kinds.resize(nb);
    for (int t = 0; t < nb; ++t) kinds[t] = tri_kind(hb[3 * t], hb[3 * t + 1], hb[3 * t + 2]);
    const double wfl = wbuild_flops(no, nv, kinds.data(), nb);
    {
      Timer tm(pf, st, FAM_W, wfl, 0.0);
      launch_wbuild_ex(0, t2, t2N, Gw, Go, tb, nb, planes, csl, nb * csl, cube_pitch(nv), no, nv,
                       false, st);
    }
    {
      Timer tm(pf, st, FAM_MIX, 0.0, 0.0);
      launch_mix3(false, eps, tb, nb, planes, PB, bt, 0.0, l1, l2, Jo, F, no, nv, st);
    }
    {
      Timer tm(pf, st, FAM_L3, wfl, 0.0);
      launch_wbuild_ex(1, l2, l2M, Gl, Go3, tb, nb, planes, csl, nb * csl, cube_pitch(nv), no, nv,
                       false, st);
    }
    {
      Timer tm(pf, st, FAM_MIX, 0.0, 0.0);
      launch_mix3(true, eps, tb, nb, planes, PB, bl, omega, l1, l2, Jo, F, no, nv, st);
    }
    // the triples that contribute to D_cd, Y^o and D_kc: all of a batch of unordered
    // triples; of a pair (i, j) the sorted ones, k <= j
    const int nown = p.resident ? nb : (hb[0] == hb[1] ? hb[1] : hb[1] + 1);
    double dfl = 0.0;
    for (int t = 0; t < nown; ++t) {
      if (hb[3 * t] == hb[3 * t + 2]) continue;
      dfl += 6.0 * v * v * v * v + (kinds[t] == TRI_DISTINCT ? 6.0 : 3.0) * 2.0 * v * v * v * (o + 1);
    }
    if (!p.resident) dfl += 2.0 * o * o * v * v * v;
    {
      Timer tm(pf, st, FAM_DENSITY, dfl, 0.0);
      launch_d3_cd(bt, bl, tb, nown, Ppart, D_cd, nv, st);
      launch_d3_vec(bt, bl, tb, nown, t2, E, Ppart, Y, D_kc, no, nv, st);
      if (!p.resident) launch_d3_gram(tau, lc, false, g, 1, Ppart, D_lk, no, nv, st);
    }
    HIPCHK(hipGetLastError());
  }
  if (p.resident) {
    Timer tm(pf, st, FAM_DENSITY, p.npairs * 2.0 * o * o * v * v * v, 0.0);
    launch_d3_gram(tau, lc, true, 0, p.npairs, Ppart, D_lk, no, nv, st);
  }
  {
    Timer tm(pf, st, FAM_DENSITY, 2.0 * o * v * o * o * v, 0.0);
    launch_d3_ld(Y, t2, Ppart, D_ld, no, nv, st);
    if (Yo) launch_d3_yout(Y, Yo, no, nv, acc, st);
  }
  HIPCHK(hipGetLastError());
  return CC3_OK;
}
