"""The bf16 forward at d <= 64 with rows whose maximum moves late, often, or not
at all (GPU): scores that grow along the keys, that shrink, and single peaks in
the last tile, against float64."""
import numpy as np
import pytest

import oracle
from helpers import TOL, compare, gpu_available, to_host64

pytestmark = [pytest.mark.gpu, pytest.mark.skipif(not gpu_available(), reason="needs a GPU")]


@pytest.mark.parametrize("d", [32, 64])
@pytest.mark.parametrize("causal", [False, True])
@pytest.mark.parametrize("shape", ["grow", "shrink", "peak", "low"])
@pytest.mark.parametrize("n,heads", [(64, 600), (65, 400), (700, 100)])
def test_moving_maxima(d, causal, shape, n, heads):
    import torch
    import paper_2609_33916_amd as lib
    torch.manual_seed(d + n)
    q, k, v = (torch.randn(1, heads, n, d, device="cuda") for _ in range(3))
    q[..., 0] = 1.0
    along = torch.arange(n, device="cuda") / n
    k[..., 0] = {"grow": 400 * along, "shrink": -400 * along, "peak": torch.zeros_like(along),
                 "low": torch.full_like(along, -500.0)}[shape]
    if shape == "peak":
        k[..., n - 2:, 0] = 300.0
    q, k, v = (x.bfloat16() for x in (q, k, v))
    o, lse = lib.attn_fwd(q, k, v, scale=0.25, causal=causal)
    torch.cuda.synchronize()
    for h in (0, heads - 1):
        ref = oracle.attention_forward(*(to_host64(x[:, h:h + 1]) for x in (q, k, v)), 0.25, causal)
        errs = compare({"O": to_host64(o[:, h:h + 1]), "L": to_host64(lse[:, h:h + 1])}, ref, keys=("O", "L"))
        assert all(e <= TOL["bf16"] for e in errs.values()), (shape, errs)
