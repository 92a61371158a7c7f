"""The FP64 GEMMs at the edges of their wave tiles: virtual sizes around multiples of 16
(blocks) and around the changes of the wave-tile shape, with distinct triples and both
kinds of equal pairs, and occupied sizes around the 8-k load unit.  Each whole call is
compared with the CPU oracle at the FP64 bar of the parity tests, 1e-11 (products and sums
of K < 1e5 random terms in FP64 stay below 1e-13)."""
import numpy as np
import pytest
import torch

from oracle import cc3_oracle as O
from paper_2007_01088_amd import cc3
from paper_2007_01088_amd.synth import make_inputs

pytestmark = pytest.mark.gpu
TOL = 1e-11


def rel(x, ref):
    return np.linalg.norm(x - ref) / max(np.linalg.norm(ref), 1e-300)


@pytest.mark.parametrize("no,nv", [
    (3, 1), (2, 15), (3, 16), (3, 17), (4, 31), (3, 32), (3, 33), (7, 47), (8, 48), (9, 49),
    (3, 64), (3, 65), (2, 80), (3, 81), (3, 96), (2, 97), (3, 127), (3, 129), (3, 145), (2, 160),
    (2, 161), (2, 193)])
def test_residual_at_tile_edges(no, nv):
    d = make_inputs(no, nv, 2 * (no + nv), tag=21)
    ctx = cc3.Context(0)
    g = {k: torch.from_numpy(d[k]).cuda() for k in ("eps", "L", "t1", "t2")}
    o1, o2 = ctx.triples_residual(g["eps"], g["L"], g["t1"], g["t2"])
    r1, r2 = O.triples_residual(d["eps"], d["L"], d["t1"], d["t2"])
    assert rel(o1.cpu().numpy(), r1) < TOL
    assert rel(o2.cpu().numpy(), r2) < TOL


# W (and the contraction) in reduced precision at the edges of its tiles (multiples of 16 from 64 to 128, and the
# change of FP32 from wave tiles to LDS tiles at 118).  Bars: a partial sum of 32 terms rounded
# to FP32 is off by at most 32 x 6e-8 of its terms (FP32, BF16x6: 2e-6); the products that the
# two-piece split leaves out are 2^-16 of a term, and its sums run over K (BF16x3: 1e-4).
@pytest.mark.parametrize("prec,flags,bar", [
    (cc3.FP32, 0, 2e-6), (cc3.BF16X6, 0, 2e-6), (cc3.BF16X3, 0, 1e-4),
    (cc3.BF16X3, cc3.LOWP_CONTRACT, 1e-4)])
@pytest.mark.parametrize("no,nv", [(2, 15), (3, 63), (3, 65), (2, 81), (3, 97), (2, 112), (3, 113),
                                   (2, 117), (3, 118), (2, 129)])
def test_reduced_precision_w_at_tile_edges(no, nv, prec, flags, bar):
    d = make_inputs(no, nv, 2 * (no + nv), tag=23)
    ctx = cc3.Context(0)
    g = {k: torch.from_numpy(d[k]).cuda() for k in ("eps", "L", "t1", "t2")}
    o1, o2 = ctx.triples_residual(g["eps"], g["L"], g["t1"], g["t2"], prec=prec, flags=flags)
    r1, r2 = O.triples_residual(d["eps"], d["L"], d["t1"], d["t2"])
    assert rel(o1.cpu().numpy(), r1) < bar
    assert rel(o2.cpu().numpy(), r2) < bar


@pytest.mark.parametrize("prec,flags,bar", [
    (cc3.FP32, 0, 2e-6), (cc3.BF16X3, cc3.LOWP_CONTRACT, 1e-4)])
def test_reduced_precision_beyond_2_gib_of_rows(prec, flags, bar):
    """nv = 896: the rows of Gw that are one slab apart span 2.9 GB in FP32, more than a
    buffer load's offset reaches.  The FP64 form (bars as above) is the reference."""
    d = make_inputs(2, 896, 24, tag=25)
    ctx = cc3.Context(0)
    g = {k: torch.from_numpy(d[k]).cuda() for k in ("eps", "L", "t1", "t2")}
    r1, r2 = (x.cpu().numpy() for x in ctx.triples_residual(g["eps"], g["L"], g["t1"], g["t2"]))
    o1, o2 = ctx.triples_residual(g["eps"], g["L"], g["t1"], g["t2"], prec=prec, flags=flags)
    assert rel(o1.cpu().numpy(), r1) < bar
    assert rel(o2.cpu().numpy(), r2) < bar


@pytest.mark.parametrize("ijk", [(2, 1, 0), (0, 1, 2), (1, 2, 0), (2, 2, 1), (1, 2, 2), (2, 1, 2)])
def test_t3_block_orderings(ijk):
    """The planes of every kind of ordered triple (the export builds all six terms)."""
    no, nv = 3, 37
    d = make_inputs(no, nv, 80, tag=22)
    ctx = cc3.Context(0)
    g = {k: torch.from_numpy(d[k]).cuda() for k in ("eps", "L", "t1", "t2")}
    tau = ctx.t3_block(g["eps"], g["L"], g["t1"], g["t2"], *ijk).cpu().numpy()
    blk = O.IntegralBlocks(O.t1_transform(d["L"], d["t1"]), no)
    assert rel(tau, O.t3_amplitudes(*ijk, d["eps"], d["t2"], blk)) < TOL


@pytest.mark.parametrize("no,nv", [(2, 1), (3, 15), (2, 17), (3, 33), (2, 49), (17, 10), (2, 65),
                                   (33, 5), (2, 97), (49, 2), (2, 129)])
def test_jacobian_at_tile_edges(no, nv):
    """Zv (tiles of (a, d)) and Zo (tiles of a, 16 l per block and up to four blocks)."""
    d = make_inputs(no, nv, 2 * (no + nv), tag=24)
    ctx = cc3.Context(0)
    g = {k: torch.from_numpy(d[k]).cuda() for k in ("eps", "L", "t1", "t2")}
    zv, zo = ctx.jacobian_prep(g["eps"], g["L"], g["t1"], g["t2"])
    rv, ro = O.jacobian_prep(d["eps"], d["L"], d["t1"], d["t2"])
    assert rel(zv.cpu().numpy(), rv) < TOL
    assert rel(zo.cpu().numpy(), ro) < TOL
