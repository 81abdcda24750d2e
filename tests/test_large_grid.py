"""The bf16 kernels for large grids at their edges: lengths that end inside a tile,
scales of either sign and zero, each entry point, in grids above every limit
of the small-grid kernels. Which side of the limits a case is on is asserted on
the CPU, from the rules in csrc/grid.hpp, so that a change of a limit cannot move it.

Without a mask the last key holds about half of every row's probability, and the last
query has a dO eight times the others', so that a row too many or too few at the end shows
(copies past the end repeat the last row)."""
import os
import shutil
import subprocess

import numpy as np
import pytest

import oracle
from helpers import OUTPUTS, TOL, compare, gpu_available, to_host64

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CSRC = os.path.join(ROOT, "paper_2609_33916_amd", "csrc")
gpu = [pytest.mark.gpu, pytest.mark.skipif(not gpu_available(), reason="needs a GPU")]


def on_gpu(f):
    for m in gpu:
        f = m(f)
    return f


# lengths and heads: more than 384 tiles of 128 rows
RAGGED = [(129, 200), (333, 130), (520, 80), (1000, 50)]
# ends of the last 32-key block of the unmasked dQ at d <= 64, in both lane halves
TAILS = [(32 * 4 + r, 200) for r in (1, 15, 16, 17, 31)]

MAIN = r"""
#include <cstdio>
#include "grid.hpp"
int main() {
  int n, heads, d, causal;
  while (std::scanf("%d %d %d %d", &n, &heads, &d, &causal) == 4)
    std::printf("%d%d%d%d%d\n", attn::use_split(attn::kFwd, true, d, causal, heads, n),
                attn::use_split(attn::kDkdv, true, d, causal, heads, n), attn::use_split(attn::kDq, true, d, causal, heads, n),
                attn::one_backward(true, d, causal, heads, n), attn::use_split_atomic(d, causal, heads, n));
}
"""


@pytest.mark.skipif(shutil.which("g++") is None, reason="needs g++")
def test_every_case_is_on_the_large_grid_side(tmp_path):
    src, exe = tmp_path / "route.cpp", tmp_path / "route"
    src.write_text(MAIN)
    subprocess.run(["g++", "-std=c++17", "-O1", "-I", CSRC, str(src), "-o", str(exe)], check=True)
    cases = [(n, heads, d, c) for n, heads in RAGGED + TAILS for d in (32, 64, 128) for c in (0, 1)]
    out = subprocess.run([str(exe)], input="".join(f"{n} {h} {d} {c}\n" for n, h, d, c in cases),
                         capture_output=True, text=True, check=True).stdout.split()
    assert out == ["00000"] * len(cases), [x for x in zip(cases, out) if x[1] != "00000"]


def _inputs(n, heads, d, scale, causal):
    """Under the causal mask the keys stay as drawn: only the last query sees the
    last key and none a later one, and that row's dQ would be dS, a difference of
    two numbers that bf16 rounds to 2^-9 of 8, times a key of 50, where it nearly
    cancels several 2^-9 of the tensor's largest value off."""
    import torch
    g = torch.Generator(device="cuda").manual_seed(1000 * d + n)
    q, k, v, do = (torch.randn(1, heads, n, d, generator=g, device="cuda") for _ in range(4))
    if scale and not causal:
        q[..., 0], k[..., 0] = 1.0, 0.0
        k[..., n - 1, 0] = np.log(n) / scale
    do[..., n - 1, :] *= 8.0
    return [x.bfloat16() for x in (q, k, v, do)]


def _check(got, ins, scale, causal, keys=OUTPUTS):
    heads = ins[0].shape[1]
    for h in (0, heads // 2, heads - 1):
        ref = oracle.attention(*(to_host64(x[:, h:h + 1]) for x in ins), scale, causal)
        errs = compare({k: to_host64(got[k][:, h:h + 1]) for k in keys}, ref, keys=keys)
        assert all(e <= TOL["bf16"] for e in errs.values()), (h, errs)


@on_gpu
@pytest.mark.parametrize("n,heads", RAGGED)
@pytest.mark.parametrize("causal", [False, True])
@pytest.mark.parametrize("d", [32, 64, 128])
def test_ragged_lengths(d, causal, n, heads):
    """attn_fwd_bwd, attn_fwd, attn_bwd from the forward's O and L, and the atomic form."""
    import torch
    import paper_2609_33916_amd as lib
    scale = d ** -0.5
    ins = _inputs(n, heads, d, scale, causal)
    q, k, v, do = ins
    got = dict(zip(OUTPUTS, lib.attn_fwd_bwd(q, k, v, do, causal=causal)))
    o, lse = lib.attn_fwd(q, k, v, causal=causal)
    bwd = dict(zip(OUTPUTS[2:], lib.attn_bwd(q, k, v, o, lse, do, causal=causal)))
    atomic = dict(zip(OUTPUTS, lib.attn_fwd_bwd_atomic(q, k, v, do, causal=causal)))
    torch.cuda.synchronize()
    _check(got, ins, scale, causal)
    assert torch.equal(got["O"], o) and torch.equal(got["L"], lse)
    _check(bwd, ins, scale, causal, keys=OUTPUTS[2:])
    _check(atomic, ins, scale, causal)
    for x in ("O", "L", "dK", "dV"):
        assert torch.equal(atomic[x], got[x]), x


@on_gpu
@pytest.mark.parametrize("scale", [-0.3, 0.0])
@pytest.mark.parametrize("causal", [False, True])
@pytest.mark.parametrize("d", [32, 64, 128])
def test_scales(d, causal, scale):
    """A negative scale (at d = 128 the dK/dV kernel takes it as the sign of
    s log2(e) instead of a sign flip of K) and zero, which gives uniform attention."""
    import torch
    import paper_2609_33916_amd as lib
    n, heads = 333, 130
    ins = _inputs(n, heads, d, scale, causal)
    got = dict(zip(OUTPUTS, lib.attn_fwd_bwd(*ins, scale=scale, causal=causal)))
    atomic = dict(zip(OUTPUTS, lib.attn_fwd_bwd_atomic(*ins, scale=scale, causal=causal)))
    torch.cuda.synchronize()
    _check(got, ins, scale, causal)
    _check(atomic, ins, scale, causal)


@on_gpu
@pytest.mark.parametrize("n,heads", TAILS)
@pytest.mark.parametrize("d", [32, 64])
def test_last_keys_of_the_unmasked_dq(d, n, heads):
    """dQ at d <= 64 masks the keys past the end by element index."""
    import torch
    import paper_2609_33916_amd as lib
    scale = d ** -0.5
    ins = _inputs(n, heads, d, scale, False)
    q, k, v, do = ins
    o, lse, dq, _, _ = lib.attn_fwd_bwd(q, k, v, do)
    dq2 = lib.attn_bwd(q, k, v, o, lse, do)[0]
    torch.cuda.synchronize()
    _check({"dQ": dq}, ins, scale, False, keys=("dQ",))
    _check({"dQ": dq2}, ins, scale, False, keys=("dQ",))
