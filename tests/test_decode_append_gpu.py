"""The appended row of a decode step (GPU): it is taken from k_new / v_new, never
from the cache row it replaces, which here holds NaN as all rows behind it do.
Lengths at the edges of the 32-key blocks, the 64-row copies and the 128-key
tiles, with unsplit and split caches."""
import numpy as np
import pytest

from helpers import TOL, gpu_available, max_rel, to_host64
from oracle import decode as dec

pytestmark = [pytest.mark.gpu, pytest.mark.skipif(not gpu_available(), reason="needs a GPU")]


@pytest.mark.parametrize("d", [32, 64, 128])
@pytest.mark.parametrize("Hq,Hkv,n", [(4, 2, 127), (4, 2, 255), (8, 1, 700), (64, 32, 1100), (40, 1, 300)])
def test_stale_rows_are_not_read(d, Hq, Hkv, n):
    import torch
    import paper_2609_33916_amd as lib
    lens = [x for x in (0, 1, 31, 32, 63, 64, 95, 127, 128, 191, 255, 256, 384, 511, 512, 640, 1023, 1024, n) if x <= n]
    B = len(lens)
    torch.manual_seed(n + d)
    q, kn, vn = (torch.randn(B, h, d, device="cuda").bfloat16() for h in (Hq, Hkv, Hkv))
    kc, vc = (torch.randn(B, Hkv, n + 1, d, device="cuda").bfloat16() for _ in range(2))
    for b, x in enumerate(lens):
        kc[b, :, x:] = float("nan")
        vc[b, :, x:] = float("nan")
    k0, v0 = kc.clone(), vc.clone()
    lt = torch.tensor(lens, dtype=torch.int32, device="cuda")
    O, L = lib.attn_decode(q, kc, vc, kn, vn, cache_lens=lt, n=n)
    torch.cuda.synchronize()
    ref = dec.decode_step(*(to_host64(x) for x in (q, k0, v0)), np.array(lens), 1.0 / np.sqrt(d), to_host64(kn), to_host64(vn))
    assert max_rel(to_host64(O), ref["O"]) <= TOL["bf16"] and max_rel(to_host64(L), ref["L"]) <= TOL["bf16"]
    for b, x in enumerate(lens):
        assert torch.equal(kc[b, :, x], kn[b]) and torch.equal(vc[b, :, x], vn[b])
        assert torch.equal(kc[b, :, :x], k0[b, :, :x]) and bool(torch.isnan(kc[b, :, x + 1:]).all())


@pytest.mark.parametrize("d", [64, 128])
@pytest.mark.parametrize("n", [5887, 5888, 6015])
def test_two_long_splits(d, n):
    """Around the line (48 tiles of 128 keys) from which two splits take a fixed
    number of tiles: sequences that end in the first split, at its end, in the
    second and at n, the cache rows behind them NaN."""
    import torch
    import paper_2609_33916_amd as lib
    B, Hq, Hkv = 64, 8, 4   # 256 workgroups: two splits
    cut = 128 * ((n + 128) // 128 // 2)
    lens = [1, 127, 128, cut - 129, cut - 1, cut, cut + 1, cut + 127, cut + 128, n - 128, n - 1] + [n] * (B - 11)
    g = torch.Generator(device="cuda").manual_seed(n + d)
    q, kn, vn = (torch.randn(B, h, d, generator=g, device="cuda").bfloat16() for h in (Hq, Hkv, Hkv))
    kc, vc = (torch.randn(B, Hkv, n + 1, d, generator=g, device="cuda").bfloat16() for _ in range(2))
    for b, x in enumerate(lens):
        kc[b, :, x:] = float("nan")
        vc[b, :, x:] = float("nan")
    some = list(range(12))
    k0, v0 = kc[some].clone(), vc[some].clone()
    O, L = lib.attn_decode(q, kc, vc, kn, vn, cache_lens=torch.tensor(lens, dtype=torch.int32, device="cuda"), n=n)
    torch.cuda.synchronize()
    ref = dec.decode_step(*(to_host64(x) for x in (q[some], k0, v0)), np.array([lens[b] for b in some]), 1.0 / np.sqrt(d),
                          to_host64(kn[some]), to_host64(vn[some]))
    assert max_rel(to_host64(O[some]), ref["O"]) <= TOL["bf16"] and max_rel(to_host64(L[some]), ref["L"]) <= TOL["bf16"]
    assert bool(torch.isfinite(O).all()) and bool(torch.isfinite(L).all())
