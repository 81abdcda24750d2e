"""The kernels for small grids and their neighbours (GPU): grids just below and
above the limit at which a call moves to the large-grid kernels, and lengths
at the edges of their 32-row blocks and of the four waves' shares (1 to 9
blocks), every output against float64 at the dtype's bound."""
import numpy as np
import pytest

import oracle
import workloads
from helpers import OUTPUTS, TOL, compare, gpu_available, run_fwd_bwd, to_gpu, to_host64

pytestmark = [pytest.mark.gpu, pytest.mark.skipif(not gpu_available(), reason="needs a GPU")]


@pytest.mark.parametrize("dtype", ["f32", "bf16"])
@pytest.mark.parametrize("d", [32, 64, 128])
@pytest.mark.parametrize("causal", [False, True])
def test_block_and_wave_edges(dtype, d, causal):
    for n in (31, 32, 33, 96, 128, 160, 257, 288):
        w = workloads.Workload(f"split_n{n}", 1, 2, n, d, dtype, causal, 1.0, 1.0, 1.0, 100 + n + d)
        inp = workloads.generate(w)
        got = run_fwd_bwd(to_gpu(inp), -0.3 if n == 160 else w.scale, causal)
        ref = oracle.attention(inp.q, inp.k, inp.v, inp.do, -0.3 if n == 160 else w.scale, causal)
        errs = compare({k: to_host64(got[k]) for k in OUTPUTS}, ref)
        assert all(v <= TOL[dtype] for v in errs.values()), (n, errs)


@pytest.mark.parametrize("heads", [28, 29, 48, 64, 65, 96, 97])
def test_both_sides_of_the_limits(heads):
    """512 rows are four 128-row tiles a head: limits of 112 to 384 tiles."""
    for dtype, d, causal in (("bf16", 128, True), ("bf16", 64, False), ("f32", 64, True)):
        w = workloads.Workload("limit", 1, heads, 512, d, dtype, causal, 1.0, 1.0, 1.0, heads)
        inp = workloads.generate(w)
        got = run_fwd_bwd(to_gpu(inp), w.scale, causal)
        some = [(0, 0), (0, heads // 2), (0, heads - 1)]
        ref = oracle.attention(inp.q, inp.k, inp.v, inp.do, w.scale, causal, heads=some)
        host = {k: np.stack([to_host64(got[k])[b, h] for b, h in some]) for k in OUTPUTS}
        errs = compare(host, ref)
        assert all(v <= TOL[dtype] for v in errs.values()), (dtype, d, causal, errs)


@pytest.mark.parametrize("dtype,d,causal,heads", [("bf16", 128, False, 29), ("bf16", 128, True, 33), ("bf16", 64, False, 65),
                                                  ("f32", 64, False, 26), ("f32", 64, False, 27)])
def test_one_launch_equals_two(dtype, d, causal, heads):
    """Around the limits of the one-launch backward: attn_fwd_bwd and the timed
    form, which launches dK/dV and dQ apart, give the same bits, and both hold
    against float64."""
    import torch
    import paper_2609_33916_amd as lib
    from bench import HipEvents
    for h in (heads - 1, heads):
        w = workloads.Workload("one", 1, h, 512, d, dtype, causal, 1.0, 1.0, 1.0, h)
        inp = workloads.generate(w)
        dev = to_gpu(inp)
        got = run_fwd_bwd(dev, w.scale, causal)
        ev = HipEvents()
        marks = [ev.create() for _ in range(4)]
        two = lib.attn_fwd_bwd_timed(dev["q"], dev["k"], dev["v"], dev["do"], marks, scale=w.scale, causal=causal)
        torch.cuda.synchronize()
        assert all(torch.equal(got[k], x) for k, x in zip(OUTPUTS, two))
        some = [(0, 0), (0, h - 1)]
        ref = oracle.attention(inp.q, inp.k, inp.v, inp.do, w.scale, causal, heads=some)
        errs = compare({k: np.stack([to_host64(got[k])[b, x] for b, x in some]) for k in OUTPUTS}, ref)
        assert all(v <= TOL[dtype] for v in errs.values()), errs


@pytest.mark.parametrize("d", [32, 64, 128])
@pytest.mark.parametrize("causal", [False, True])
@pytest.mark.parametrize("n", [33, 40, 97, 127, 128])
def test_an_infinity_in_the_last_row_stays_one(d, causal, n):
    """float32 tiles read zeros past the end: an infinity in the last row of V, or
    of dO, makes its column of O, or of dV, infinite and no other value NaN."""
    import torch
    import paper_2609_33916_amd as lib
    torch.manual_seed(n + d)
    q, k, v, g = (torch.randn(1, 2, n, d, device="cuda") for _ in range(4))
    vi, gi = v.clone(), g.clone()
    vi[:, :, n - 1, 5] = float("inf")
    gi[:, :, n - 1, 7] = float("inf")
    # and the rows that follow a matrix in memory, those of the next head, are not read
    for x in (q, k, v, g, vi, gi):
        x[:, 1] = float("nan")
    o, lse = lib.attn_fwd(q, k, vi, causal=causal)
    _, _, _, _, dv = lib.attn_fwd_bwd(q, k, v, gi, causal=causal)
    torch.cuda.synchronize()
    o, lse, dv = o[:, 0], lse[:, 0], dv[:, 0]
    seen = o[:, n - 1:] if causal else o   # the queries that see the last key
    assert bool((seen[..., 5] == float("inf")).all()) and bool(torch.isfinite(lse).all())
    assert bool((dv[..., 7] == float("inf")).all())
    rest = torch.arange(d, device="cuda")
    assert bool(torch.isfinite(o[..., rest != 5]).all()) and bool(torch.isfinite(dv[..., rest != 7]).all())
    grads = lib.attn_fwd_bwd(q, k, v, g, causal=causal)
    torch.cuda.synchronize()
    assert all(bool(torch.isfinite(x[:, 0]).all()) for x in grads)
