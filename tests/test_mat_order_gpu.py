"""Issue order of the materialising forward under the causal mask (GPU): in
groups of heads while the keys and values of a group's heads on one XCD fit
its 4 MB L2, else head by head. Two head counts on either side of that line
(27 and 28 heads of 150 KB on an XCD) against attention in float32: every row
of every head has to be written, in either order.
"""
import pytest

from helpers import TOL, gpu_available

pytestmark = [pytest.mark.gpu, pytest.mark.skipif(not gpu_available(), reason="needs a GPU")]


@pytest.mark.parametrize("heads", [216, 224])
def test_every_head_and_row_in_either_order(heads):
    import torch
    import paper_2609_33916_amd as lib
    n, d = 300, 128
    g = torch.Generator(device="cuda").manual_seed(heads)
    q, k, v = (torch.randn(1, heads, n, d, device="cuda", generator=g).to(torch.bfloat16) for _ in range(3))
    O = torch.full_like(q, float("nan"))
    L = torch.full((1, heads, n), float("nan"), device="cuda")
    lib.attn_mat_fwd(q, k, v, causal=True, out=(O, L))
    s = torch.matmul(q.float(), k.float().transpose(-1, -2).contiguous()) * d ** -0.5
    s = s.masked_fill(~torch.ones(n, n, dtype=torch.bool, device="cuda").tril(), float("-inf"))
    ref_O, ref_L = torch.matmul(torch.softmax(s, -1), v.float()), torch.logsumexp(s, -1)
    for got, ref in ((O.float(), ref_O), (L, ref_L)):
        err = ((got - ref).abs().amax() / ref.abs().amax()).item()
        print(heads, f"{err:.2e}", flush=True)
        assert err <= TOL["bf16"]
