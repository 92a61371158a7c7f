"""The allocation-free residual at the largest sizes that a workspace of two buffer sets and
five cubes per triple let into its 256 MiB array, against the workspace entry point.  Both
run the same kernels on other batches, so the FP64 bar of the parity tests applies, 1e-11; in
the mixed-all form the K chunks follow the batch, and partial sums of 32 terms are rounded to
FP32 (at most 32 x 6e-8 of their terms, 2e-6)."""
import pytest
import torch

from paper_2007_01088_amd import cc3
from paper_2007_01088_amd.synth import make_inputs

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("no,nv,prec,flags,bar", [
    (2, 104, cc3.FP64, 0, 1e-11), (4, 97, cc3.FP64, 0, 1e-11), (8, 84, cc3.FP64, 0, 1e-11),
    (10, 81, cc3.FP64, 0, 1e-11), (12, 76, cc3.FP64, 0, 1e-11), (31, 46, cc3.FP64, 0, 1e-11),
    (4, 95, cc3.FP32, 0, 1e-11), (8, 81, cc3.BF16X6, 0, 1e-11),
    (6, 79, cc3.BF16X6, cc3.LOWP_CONTRACT, 2e-6)])
def test_noalloc_at_its_limit(no, nv, prec, flags, bar):
    print(f"no-alloc call no={no} nv={nv} prec={prec} flags={flags}", flush=True)
    d = make_inputs(no, nv, 3 * (no + nv), tag=41)
    ctx = cc3.Context(0)
    g = {k: torch.from_numpy(d[k]).cuda() for k in ("eps", "L", "t1", "t2")}
    r1, r2 = ctx.triples_residual(g["eps"], g["L"], g["t1"], g["t2"], prec=prec, flags=flags)
    o1, o2 = torch.full_like(r1, float("nan")), torch.full_like(r2, float("nan"))
    ctx.triples_residual_noalloc(g["eps"], g["L"], g["t1"], g["t2"], o1, o2, prec=prec, flags=flags)
    torch.cuda.synchronize()
    assert float((o1 - r1).norm() / r1.norm()) <= bar
    assert float((o2 - r2).norm() / r2.norm()) <= bar
    ctx.close()
