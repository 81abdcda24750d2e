"""float32 on the bfloat16 matrix cores (GPU): four- and eight-wave workgroups
on both sides of their limit, lengths at the tile edges, values that do not
split (infinities, large ones and those below 2^-110, as operands, products,
probabilities and dS), keys masked by value, and the error against float64."""
import numpy as np
import pytest

import oracle
import workloads
from helpers import OUTPUTS, TOL, compare, gpu_available, max_rel, run_fwd_bwd, to_gpu, to_host64

pytestmark = [pytest.mark.gpu, pytest.mark.skipif(not gpu_available(), reason="needs a GPU")]


@pytest.mark.parametrize("d", [32, 64, 128])
@pytest.mark.parametrize("causal", [False, True])
@pytest.mark.parametrize("n,heads", [(129, 100), (192, 129), (255, 150), (511, 64), (520, 80), (40, 400)])
def test_tile_edges(d, causal, n, heads):
    w = workloads.Workload("x3", 1, heads, n, d, "f32", causal, 1.0, 1.0, 1.0, n + d)
    scale = -0.2 if heads == 100 else w.scale
    inp = workloads.generate(w)
    got = run_fwd_bwd(to_gpu(inp), scale, causal)
    some = [(0, 0), (0, heads - 1)]
    ref = oracle.attention(inp.q, inp.k, inp.v, inp.do, scale, causal, heads=some)
    errs = compare({k: np.stack([to_host64(got[k])[b, h] for b, h in some]) for k in OUTPUTS}, ref)
    # sums of at most 520 terms, each rounded to 2^-24 of the running sum, and
    # products to 2^-25: far below the workload bound
    assert all(v <= 1e-5 for v in errs.values()), errs


@pytest.mark.parametrize("d", [32, 64, 128])
@pytest.mark.parametrize("pad", [-np.inf, np.finfo(np.float32).min])
@pytest.mark.parametrize("n,heads", [(200, 200), (200, 100)])
def test_keys_masked_by_value(d, pad, n, heads):
    """A column of ones in Q and -inf (or the lowest value) in K masks a key;
    the scores, O, L and dV are those without the masked keys."""
    import torch
    import paper_2609_33916_amd as lib
    w = workloads.Workload("pad", 1, heads, n, d, "f32", False, 1.0, 1.0, 1.0, d)
    inp = workloads.generate(w)
    inp.q[..., 0], inp.k[..., 0] = 1.0, 0.0
    inp.k[..., 150:, 0] = pad
    dev = to_gpu(inp)
    o, lse, _, _, dv = lib.attn_fwd_bwd(dev["q"], dev["k"], dev["v"], dev["do"], scale=1.0)
    torch.cuda.synchronize()
    ref = oracle.attention(inp.q[:, :1], inp.k[:, :1], inp.v[:, :1], inp.do[:, :1], 1.0, False) \
        if pad != -np.inf else None
    q, k, v, g = (torch.from_numpy(x[0, 0].astype(np.float64)) for x in (inp.q, inp.k, inp.v, inp.do))
    s = q @ k[:150].T
    p = torch.softmax(s, 1)
    want = {"O": p @ v[:150], "L": torch.logsumexp(s, 1)}
    errs = compare({"O": to_host64(o)[0, 0], "L": to_host64(lse)[0, 0]},
                   {k2: x.numpy() for k2, x in want.items()}, keys=("O", "L"))
    assert all(e <= TOL["f32"] for e in errs.values()), errs
    got_dv = to_host64(dv)[0, 0]
    assert np.abs(got_dv[:150] - (p.T @ g).numpy()).max() <= 1e-4 * np.abs(got_dv).max()
    assert np.all(got_dv[150:] == 0.0)
    if ref is not None:
        assert np.abs(to_host64(o)[0, 0] - ref["O"][0, 0]).max() <= 1e-4


@pytest.mark.parametrize("d", [32, 64, 128])
@pytest.mark.parametrize("causal", [False, True])
@pytest.mark.parametrize("qcol,pad", [(1e4, -1.1e38), (100300.0, -1e38), (2.0 ** 25, -2.0 ** 109)])
def test_keys_masked_by_an_overflowing_product(d, causal, qcol, pad):
    """Finite operands whose product leaves the float32 range: the score is
    -inf, as the float32 product is, although a part product of the other sign
    overflows too; such a key is masked and nothing becomes NaN."""
    n, heads, tail = 200, 200, 150
    w = workloads.Workload("over", 1, heads, n, d, "f32", causal, 1.0, 1.0, 1.0, d)
    inp = workloads.generate(w)
    inp.q[..., 0], inp.k[..., 0] = qcol, 0.0
    inp.k[..., tail:, 0] = pad
    scale = 0.2
    got = run_fwd_bwd(to_gpu(inp), scale, causal)
    for head in (0, heads - 1):
        q, k, v, g = (x[0, head].astype(np.float64) for x in (inp.q, inp.k, inp.v, inp.do))
        s = scale * q[:, 1:] @ k[:, 1:].T
        s[:, tail:] = -np.inf
        if causal:
            s[np.triu_indices(n, 1)] = -np.inf
        lse = np.log(np.exp(s).sum(1))
        p = np.exp(s - lse[:, None])
        o = p @ v
        ds = p * (g @ v.T - (g * o).sum(1)[:, None]) * scale
        ref = {"O": o, "L": lse, "dQ": ds[:, :tail] @ k[:tail], "dK": ds.T @ q, "dV": p.T @ g}
        errs = compare({key: to_host64(got[key])[0, head] for key in OUTPUTS}, ref)
        # dK's first column sums 200 terms of about qcol that nearly cancel
        assert all(e <= TOL["f32"] for e in errs.values()), errs


@pytest.mark.parametrize("d", [32, 64, 128])
@pytest.mark.parametrize("causal", [False, True])
@pytest.mark.parametrize("which,shrink", [("do", 108), ("do", 116), ("do", 120), ("v", 116), ("q", 120), ("k", 120)])
def test_small_operands_keep_their_bits(d, causal, which, shrink):
    """One operand down by a power of two, to where its low part would fall under
    the smallest bfloat16: results as precise as those of float32 products."""
    n, heads = 200, 200
    w = workloads.Workload("small", 1, heads, n, d, "f32", causal, 1.0, 1.0, 1.0, d + shrink)
    inp = workloads.generate(w)
    setattr(inp, which, getattr(inp, which) * np.float32(2.0 ** -shrink))
    got = run_fwd_bwd(to_gpu(inp), w.scale, causal)
    some = [(0, 0), (0, heads - 1)]
    ref = oracle.attention(inp.q, inp.k, inp.v, inp.do, w.scale, causal, heads=some)
    errs = compare({k: np.stack([to_host64(got[k])[b, h] for b, h in some]) for k in OUTPUTS}, ref)
    # as test_tile_edges; dS of 2^-120 P is subnormal, to 2^-149: 2^-20 of the largest
    assert all(v <= 1e-5 for v in errs.values()), errs


@pytest.mark.parametrize("d", [32, 64, 128])
def test_small_probabilities_keep_their_bits(d):
    """Keys 80 below the others, P about 2^-123: their rows of dK and dV, and a
    column of O that only they reach, are as precise as the rest."""
    n, heads, tail = 200, 200, 150
    w = workloads.Workload("smallp", 1, heads, n, d, "f32", False, 0.1, 1.0, 1.0, d)
    inp = workloads.generate(w)
    inp.q[..., 0], inp.k[..., 0] = 1.0, 0.0
    inp.k[..., tail:, 0] = -80.0
    inp.v[..., :tail, 1] = 0.0
    inp.v[..., tail:, 1] = np.abs(inp.v[..., tail:, 1])
    got = run_fwd_bwd(to_gpu(inp), 1.0, False)
    ref = oracle.attention(inp.q, inp.k, inp.v, inp.do, 1.0, False, heads=[(0, heads - 1)])
    cut = {"O": np.s_[:, 1], "dK": np.s_[tail:], "dV": np.s_[tail:]}
    errs = {k: max_rel(to_host64(got[k])[0, heads - 1][x], np.asarray(ref[k])[0][x]) for k, x in cut.items()}
    # each of the up to 64 additions that form a score of -80 rounds it to 2^-18 =
    # 3.8e-6, which is as much of P: 3e-5 when they are independent
    assert all(v <= 1e-4 for v in errs.values()), errs


@pytest.mark.parametrize("d", [32, 64, 128])
@pytest.mark.parametrize("causal", [False, True])
@pytest.mark.parametrize("which", ["q", "k", "v", "do"])
@pytest.mark.parametrize("row,heads", [(5, 100), (200, 60), (330, 100), (519, 60)])
def test_from_one_large_value_on(d, causal, which, row, heads):
    """A value of 2^25 in one row: the tiles from there on take the float32
    instructions, those before stay as they are; every row against float64."""
    n = 520
    w = workloads.Workload("large", 1, heads, n, d, "f32", causal, 1.0, 1.0, 1.0, d + row)
    inp = workloads.generate(w)
    getattr(inp, which)[:, :, row, 3] = 2.0 ** 25
    other = {"q": "k", "k": "q", "v": "do", "do": "v"}[which]   # keeps S and dP of order 1
    getattr(inp, other)[..., 3] *= np.float32(2.0 ** -25)
    got = run_fwd_bwd(to_gpu(inp), w.scale, causal)
    some = [(0, 0), (0, heads - 1)]
    ref = oracle.attention(inp.q, inp.k, inp.v, inp.do, w.scale, causal, heads=some)
    host = {k: np.stack([to_host64(got[k])[b, h] for b, h in some]) for k in OUTPUTS}
    rest = np.arange(d) != 3
    for cols in (rest, ~rest):   # the large value's column apart from the others
        errs = {k: max_rel(host[k][..., cols], np.asarray(ref[k])[..., cols]) for k in OUTPUTS if k != "L"}
        assert all(v <= 1e-5 for v in errs.values()), errs
    assert max_rel(host["L"], np.asarray(ref["L"])) <= 1e-5


@pytest.mark.parametrize("d", [32, 64, 128])
@pytest.mark.parametrize("causal", [False, True])
@pytest.mark.parametrize("lse,do,v", [(0.0, 1.5e19, 3.4e38 / 1.5e19), (-60.0, 1.8e6, 3.4e38 / 1.8e6 / np.exp(60.0))])
def test_dS_up_to_the_largest_float(d, causal, lse, do, v):
    """dS = 3.4e38, which bfloat16 rounds to infinity, gives the dQ that float32
    gives (O = 0, so that D = 0; Q = 0 and the given L make P exp(-L))."""
    import torch
    import paper_2609_33916_amd as lib
    n, heads = 200, 200
    q, o = torch.zeros(1, heads, n, d, device="cuda"), torch.zeros(1, heads, n, d, device="cuda")
    k = torch.full_like(q, 2.0 ** -10)
    vt, g = torch.zeros_like(q), torch.zeros_like(q)
    vt[..., 0], g[..., 0] = v, do
    dq, dk, dv = lib.attn_bwd(q, k, vt, o, torch.full((1, heads, n), lse, device="cuda"), g, scale=1.0, causal=causal)
    torch.cuda.synchronize()
    keys = np.arange(1, n + 1) if causal else np.full(n, n)
    want = np.exp(-lse) * float(np.float32(do)) * float(np.float32(v)) * 2.0 ** -10 * keys[:, None] * np.ones(d)
    assert max_rel(to_host64(dq)[0, 0], want) <= TOL["f32"] and max_rel(to_host64(dq)[0, -1], want) <= TOL["f32"]
    want = np.exp(-lse) * float(np.float32(do)) * (n - np.arange(n) if causal else np.full(n, n))
    assert max_rel(to_host64(dv)[0, 0, :, 0], want) <= TOL["f32"]
    assert bool((dk == 0).all())


def test_infinite_values_stay_infinite():
    """An infinity in V makes that column of O infinite, as float32 sums do."""
    import torch
    import paper_2609_33916_amd as lib
    x = torch.randn(1, 300, 200, 64, device="cuda")
    v = x.clone()
    v[0, :, 17, 5] = float("inf")
    o, lse = lib.attn_fwd(x, x, v, scale=0.01)
    torch.cuda.synchronize()
    assert bool(torch.isinf(o[..., 5]).all()) and bool(torch.isfinite(o[..., 6:]).all()) and bool(torch.isfinite(lse).all())
