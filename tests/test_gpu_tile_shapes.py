"""Forms of the wave-tile and LDS-tile kernels that the other parity tests do not reach: the
5 x 2 and 5 x 4 wave tiles of the Jacobian preparation and of the transition density, the
Jacobian preparation and the mixed-all contraction in reduced precision at tile edges, and
packed groups whose members take different tiles alone.

Bars: FP64 1e-11, that of the parity tests.  A partial sum of 32 terms rounded to FP32 is off by
at most 32 x 6e-8 of its terms (FP32 and BF16x6: 2e-6); the products that the two-piece split
leaves out are 2^-16 of a term, and its sums run over K (BF16x3: 1e-4); a chunk of 4096 terms
summed in FP32, rounding errors of random sign, is off by 64 x 6e-8 of them (FP32 mixed-all: five
times that, 2e-5)."""
import numpy as np
import pytest
import torch

from oracle import cc3_oracle as O
from paper_2007_01088_amd import cc3
from paper_2007_01088_amd.synth import make_inputs, make_left_inputs, sample_triples

pytestmark = pytest.mark.gpu
TOL = 1e-11


def rel(x, ref):
    return np.linalg.norm(x - ref) / max(np.linalg.norm(ref), 1e-300)


def cuda(*arrays):
    return [torch.from_numpy(np.ascontiguousarray(a)).cuda() for a in arrays]


def density_oracle(d, lf):
    no = d["no"]
    blk = O.IntegralBlocks(O.t1_transform(d["L"], d["t1"]), no, full=True)
    return O.transition_density_occupied(d["eps"], d["t2"], lf["l1"], lf["l2"], lf["omega"], blk,
                                         O.fock_ov(d["L"], d["t1"]))


@pytest.mark.parametrize("no,nv0,nv", [(2, 150, 150), (3, 24, 155), (3, 24, 290), (2, 40, 320),
                                       (2, 40, 400)])
def test_five_block_tiles(no, nv0, nv):
    """A problem of nv0 virtuals spread at random over nv, the others decoupled (zero Cholesky
    rows and columns, zero amplitudes): the oracle's values in place, exact zeros elsewhere."""
    print(f"five-block tiles no={no} nv={nv0} in {nv}", flush=True)
    d, lf = make_inputs(no, nv0, 24, tag=61), make_left_inputs(no, nv0, tag=61)
    at = np.sort(np.random.default_rng(nv).choice(nv, nv0, replace=False))
    mo = np.concatenate([np.arange(no), no + at])
    eps = np.full(no + nv, 10.0)
    eps[mo] = d["eps"]
    L = np.zeros((24, no + nv, no + nv))
    L[np.ix_(range(24), mo, mo)] = d["L"]

    def spread(x, axes):
        out = np.zeros([nv if a in axes else n for a, n in enumerate(x.shape)])
        out[np.ix_(*[at if a in axes else range(n) for a, n in enumerate(x.shape)])] = x
        return out
    g = cuda(eps, L, spread(d["t1"], (1,)), spread(d["t2"], (2, 3)))
    left = cuda(spread(lf["l1"], (1,)), spread(lf["l2"], (2, 3)))
    ctx = cc3.Context(0)
    zv, zo = ctx.jacobian_prep(*g)
    rv, ro = O.jacobian_prep(d["eps"], d["L"], d["t1"], d["t2"])
    dcd, dkc, dld, _, yo = ctx.transition_density(*g, *left, lf["omega"], want_yo=True)
    pcd, pkc, pld, py = density_oracle(d, lf)
    for name, got, ref, axes in (("Zv", zv, rv, (0, 1, 3)), ("Zo", zo, ro, (0,)),
                                 ("D_cd", dcd, pcd, (0, 1)), ("D_kc", dkc, pkc, (1,)),
                                 ("D_ld", dld, pld, (1,)), ("Y^o", yo, py, (0,))):
        got = got.cpu().numpy()
        ix = np.ix_(*[at if a in axes else range(n) for a, n in enumerate(ref.shape)])
        assert rel(got[ix], ref) < TOL, name
        got[ix] = 0.0
        assert not got.any(), name
    ctx.close()


@pytest.mark.parametrize("prec,bar", [(cc3.FP32, 2e-6), (cc3.BF16X6, 2e-6), (cc3.BF16X3, 1e-4)])
@pytest.mark.parametrize("no,nv", [(3, 15), (3, 63), (2, 81), (3, 97), (2, 117), (3, 118), (2, 129)])
def test_reduced_precision_jacobian_at_tile_edges(no, nv, prec, bar):
    d = make_inputs(no, nv, 2 * (no + nv), tag=62)
    ctx = cc3.Context(0)
    zv, zo = ctx.jacobian_prep(*cuda(d["eps"], d["L"], d["t1"], d["t2"]), prec=prec)
    rv, ro = O.jacobian_prep(d["eps"], d["L"], d["t1"], d["t2"])
    assert rel(zv.cpu().numpy(), rv) < bar
    assert rel(zo.cpu().numpy(), ro) < bar


@pytest.mark.parametrize("prec,bar", [(cc3.FP32, 2e-5), (cc3.BF16X6, 2e-6)])
@pytest.mark.parametrize("no,nv", [(3, 1), (2, 15), (3, 17), (3, 65), (2, 81), (3, 97), (2, 112),
                                   (3, 113), (2, 129)])
def test_mixed_all_at_tile_edges(no, nv, prec, bar):
    d = make_inputs(no, nv, 2 * (no + nv), tag=63)
    ctx = cc3.Context(0)
    o1, o2 = ctx.triples_residual(*cuda(d["eps"], d["L"], d["t1"], d["t2"]), prec=prec,
                                  flags=cc3.LOWP_CONTRACT)
    r1, r2 = O.triples_residual(d["eps"], d["L"], d["t1"], d["t2"])
    assert rel(o1.cpu().numpy(), r1) < bar
    assert rel(o2.cpu().numpy(), r2) < bar


# groups of (no, nv): FP32 on either side of nv = 118, where LDS tiles take over from wave
# tiles, led by a member on each; BF16 with tiles of 64 to 128 in one group
GROUPS = [(cc3.FP32, [(6, 150), (5, 120), (4, 93), (3, 118), (3, 117)]),
          (cc3.FP32, [(9, 120), (4, 145), (5, 64), (3, 128)]),
          (cc3.BF16X6, [(7, 113), (5, 63), (4, 81), (3, 97), (2, 130)]),
          (cc3.BF16X3, [(7, 81), (5, 64), (4, 113), (3, 97), (2, 33)]),
          (cc3.FP64, [(17, 30), (20, 12), (9, 40), (33, 16), (18, 33)])]


@pytest.mark.parametrize("prec,members", GROUPS)
def test_packed_group_of_mixed_tiles_equals_alone(prec, members):
    arena = torch.empty(8 << 30, dtype=torch.uint8, device="cuda")
    srv = cc3.Server(arena, max_inflight=1)
    srv.set_packing(8, 2e12)
    big = make_inputs(10, 170, 300, tag=64)  # holds the slot while the group queues; not packed
    ds = [big] + [make_inputs(no, nv, 3 * (no + nv), tag=65) for no, nv in members]
    gs = [cuda(d["eps"], d["L"], d["t1"], d["t2"]) for d in ds]
    ms = [srv.register(d["no"], d["nv"], *g[:3]) for d, g in zip(ds, gs)]
    tks = [srv.submit(m, g[3], prec=prec) for m, g in zip(ms, gs)]
    packed = [srv.wait(t, mol=m) for t, m in zip(tks, ms)][1:]
    assert srv.stats()["packed"] >= 2, srv.stats()
    srv.set_packing(1, 0)
    for m, g, (p1, p2, _) in list(zip(ms, gs, [None] + packed))[1:]:
        a1, a2, _ = srv.wait(srv.submit(m, g[3], prec=prec), mol=m)
        assert torch.equal(a1, p1) and torch.equal(a2, p2)
    srv.close()


@pytest.mark.parametrize("no,nv", [(17, 1), (17, 16), (20, 5), (18, 17), (21, 32), (18, 33), (33, 7),
                                   (34, 17), (49, 3), (63, 16)])
def test_oo_terms_in_shares_above_16_occupied(no, nv):
    """Wavefronts without columns of their own (nv <= 32) take shares of the oo terms: each
    count of row blocks, one and two wavefronts side by side, and the next size up."""
    d = make_inputs(no, nv, 20, tag=66)
    tri = np.unique(np.concatenate([sample_triples(no, 150, seed=no),
                                    [[no - 1, no - 1, 0], [no - 1, 0, 0]]]), axis=0).astype(np.int32)
    ctx = cc3.Context(0)
    g = cuda(d["eps"], d["L"], d["t1"], d["t2"])
    o1, o2 = ctx.triples_residual_subset(*g, tri)
    r1, r2 = O.omega_tilde_subset(d["eps"], d["L"], d["t1"], d["t2"], tri)
    assert rel(o1.cpu().numpy(), r1) < TOL
    assert rel(o2.cpu().numpy(), r2) < TOL


@pytest.mark.parametrize("nv", [448, 451, 465, 500, 512, 513, 576, 601, 641])
def test_omega_on_lds_tiles_at_large_nv(nv):
    """The LDS form of the Omega GEMM (448 and more virtuals; 513 stays on wave tiles): 24
    virtuals spread over nv against the oracle, zeros elsewhere.  Odd and even counts of units
    of 8 k, rows with and without padding, the column of Omega1 in a tile of its own."""
    no, nv0 = 3, 24
    print(f"omega on LDS tiles nv={nv}", flush=True)
    d = make_inputs(no, nv0, 12, tag=67)
    at = np.sort(np.random.default_rng(nv).choice(nv, nv0, replace=False))
    mo = np.concatenate([np.arange(no), no + at])
    eps = np.full(no + nv, 10.0)
    eps[mo] = d["eps"]
    L, t1, t2 = np.zeros((12, no + nv, no + nv)), np.zeros((no, nv)), np.zeros((no, no, nv, nv))
    L[np.ix_(range(12), mo, mo)] = d["L"]
    t1[:, at] = d["t1"]
    t2[np.ix_(range(no), range(no), at, at)] = d["t2"]
    ctx = cc3.Context(0)
    o1, o2 = (x.cpu().numpy() for x in ctx.triples_residual(*cuda(eps, L, t1, t2)))
    r1, r2 = O.triples_residual(d["eps"], d["L"], d["t1"], d["t2"])
    ix = np.ix_(range(no), range(no), at, at)
    assert rel(o1[:, at], r1) < TOL and rel(o2[ix], r2) < TOL
    o1[:, at] = 0.0
    o2[ix] = 0.0
    assert not o1.any() and not o2.any()
    ctx.close()


@pytest.mark.parametrize("no,nv", [(2, 451), (3, 500)])
def test_omega_on_lds_tiles_dense(no, nv):
    """Every value in use: against the split-BF16 W build and contraction, which is another
    kernel on other operands (BF16x6: 2e-6)."""
    print(f"omega on LDS tiles, dense no={no} nv={nv}", flush=True)
    d = make_inputs(no, nv, 24, tag=68)
    ctx = cc3.Context(0)
    g = cuda(d["eps"], d["L"], d["t1"], d["t2"])
    o1, o2 = ctx.triples_residual(*g)
    r1, r2 = ctx.triples_residual(*g, prec=cc3.BF16X6, flags=cc3.LOWP_CONTRACT)
    assert float((o1 - r1).norm()) < 2e-6 * float(r1.norm())
    assert float((o2 - r2).norm()) < 2e-6 * float(r2.norm())
    ctx.close()


def test_lds_tile_requests_are_not_packed():
    """Requests whose Omega GEMM runs on LDS tiles stay out of packed groups, whose form is
    another, and give the bits of the same request alone."""
    arena = torch.empty(40 << 30, dtype=torch.uint8, device="cuda")
    srv = cc3.Server(arena, max_inflight=1)
    srv.set_packing(8, 1e13)
    ds = [make_inputs(2, 448, 24, tag=69 + t) for t in range(3)]
    gs = [cuda(d["eps"], d["L"], d["t1"], d["t2"]) for d in ds]
    ms = [srv.register(2, 448, *g[:3]) for g in gs]
    tks = [srv.submit(m, g[3]) for m, g in zip(ms, gs)]
    got = [srv.wait(t, mol=m) for t, m in zip(tks, ms)]
    assert srv.stats()["packed"] == 0
    for m, g, (p1, p2, _) in zip(ms, gs, got):
        a1, a2, _ = srv.wait(srv.submit(m, g[3]), mol=m)
        assert torch.equal(a1, p1) and torch.equal(a2, p2)
    srv.close()
