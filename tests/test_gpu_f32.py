"""fp32 attention against the CPU oracle at the edges of its 16-row blocks and 16-key units, with one and several units per
wave, key splits, both row tiles of d = 64, GQA groups that end inside a row block, and block rows spliced in."""
import pytest

import oracle
import paper_2604_05250_amd as dd
from paper_2604_05250_amd import workloads as wl
from _util import assert_attention_close, out_to_f64, to_dev

pytestmark = pytest.mark.gpu
F32 = wl.F32


# (32 x 17 heads x 17 rows: enough workgroups for the 32-row tile)
@pytest.mark.parametrize("B,H,Hkv,N,d", [(1, 1, 1, 1, 64), (1, 2, 1, 15, 128), (1, 2, 2, 16, 64), (2, 3, 1, 17, 128), (1, 2, 2, 129, 64),
                                         (1, 4, 2, 255, 128), (1, 5, 1, 257, 64), (32, 17, 17, 17, 64), (16, 32, 32, 33, 64)])
def test_bidir_f32(B, H, Hkv, N, d):
    import torch
    cfg = wl.custom_config(B=B, H=H, Hkv=Hkv, N=N, d=d, qk_dtype=F32, v_dtype=F32, prompt=0, G=N, bl=min(16, N))
    inp = wl.attention_inputs(cfg, seed=N)
    O = dd.dd_bidir_attention(to_dev(inp["Q"]), to_dev(inp["K"]), to_dev(inp["V"]))
    torch.cuda.synchronize()
    assert_attention_close(out_to_f64(O, F32), oracle.bidir_attention(inp["Q"], inp["K"], inp["V"], F32, F32), F32,
                           f"fp32 {B}x{H}/{Hkv}x{N}x{d}")


@pytest.mark.parametrize("B,H,Hkv,N,d,bl,bs", [(1, 4, 4, 128, 64, 16, 64), (1, 4, 1, 511, 128, 5, 506), (1, 2, 2, 512, 64, 17, 0),
                                               (1, 2, 1, 1037, 128, 16, 77), (2, 2, 2, 2050, 64, 1, 2049)])
def test_block_f32(B, H, Hkv, N, d, bl, bs):
    import torch
    cfg = wl.custom_config(B=B, H=H, Hkv=Hkv, N=N, d=d, qk_dtype=F32, v_dtype=F32, bl=bl, prompt=0, G=N)
    cache = wl.cache_inputs(cfg, seed=bs + N)
    blk = wl.block_inputs(cfg, bs, 0)
    for fresh in (True, False):
        Kb, Vb = (blk["Kblk"], blk["Vblk"]) if fresh else (None, None)
        O = dd.dd_block_attention_cached(to_dev(blk["Qblk"]), to_dev(cache["Kc"]), to_dev(cache["Vc"]), bs, Kblk=to_dev(Kb), Vblk=to_dev(Vb))
        torch.cuda.synchronize()
        ref = oracle.block_attention_cached(blk["Qblk"], cache["Kc"], cache["Vc"], bs, F32, F32, Kb, Vb)
        assert_attention_close(out_to_f64(O, F32), ref, F32, f"fp32 block {B}x{H}/{Hkv} N{N} d{d} bl{bl}@{bs} fresh={fresh}")


@pytest.mark.parametrize("N,d", [(1, 64), (15, 128), (100, 64), (333, 128), (515, 64)])
def test_infinite_value_f32(N, d):
    # one infinite value in any row, the last one of a ragged range included: infinite in its dimension for every query
    import torch
    cfg = wl.custom_config(B=1, H=2, Hkv=1, N=N, d=d, qk_dtype=F32, v_dtype=F32, prompt=0, G=N, bl=min(16, N))
    inp = wl.attention_inputs(cfg, seed=N)
    Q, K, V = (to_dev(inp[k]) for k in "QKV")
    want = dd.dd_bidir_attention(Q, K, V).clone()
    want[..., 5] = float("inf")
    for row in (0, N // 2, N - 1):
        V2 = V.clone()
        V2[:, :, row, 5] = float("inf")
        got = dd.dd_bidir_attention(Q, K, V2)
        torch.cuda.synchronize()
        assert torch.equal(got, want), f"{N} keys, d {d}, row {row}"


@pytest.mark.parametrize("N,d,first,last", [(100, 64, 0, 16), (128, 64, 16, 32), (133, 128, 66, 133), (333, 128, 0, 70), (515, 64, 257, 515),
                                            (1100, 128, 0, 600)])
def test_keys_that_score_minus_infinity_f32(N, d, first, last):
    # a run of keys out of reach (an infinite component against positive queries), a wave's whole 16-key units among them:
    # the result is that of the other keys alone
    import torch
    cfg = wl.custom_config(B=1, H=2, Hkv=2, N=N, d=d, qk_dtype=F32, v_dtype=F32, prompt=0, G=N, bl=min(16, N))
    inp = wl.attention_inputs(cfg, seed=N)
    Q, K, V = (inp[k].copy() for k in "QKV")
    Q[..., 5] = abs(Q[..., 5]) + 0.1
    K[:, :, first:last, :] = 0
    K[:, :, first:last, 5] = -float("inf")
    O = dd.dd_bidir_attention(to_dev(Q), to_dev(K), to_dev(V))
    torch.cuda.synchronize()
    keep = [j for j in range(N) if not first <= j < last]
    bl = min(N, 16)
    ref = oracle.block_attention_cached(Q[:, :, :bl].copy(), K[:, :, keep].copy(), V[:, :, keep].copy(), 0, F32, F32)
    assert_attention_close(out_to_f64(O, F32)[:, :, :bl], ref, F32, f"{N} keys, [{first}, {last}) at -inf")


# The error of a sharp softmax is that of its scores: an absolute error of one is a relative error of its weight.  Summing n
# products of rms sigma in a chain, rounding by u / sqrt(3) rms (u = 2^-24) of a partial sum that grows as sqrt(k), loses
# u sigma sqrt(n^2 / 6); scores of d = 128 in four chains of 32, added in pairs, lose 28 u sigma before the division by
# sqrt(d), 2.5 u sigma after it: 4.4e-7 of the result at sigma = 3.  (One chain of 128: 4.6 u sigma, 8.3e-7.)  The exponential
# and the weighted sum add about 2 u each.
@pytest.mark.parametrize("B,H,Hkv,N,d,bl", [(1, 4, 4, 128, 64, 0), (16, 32, 32, 128, 64, 0), (1, 4, 2, 333, 128, 16), (1, 8, 2, 700, 128, 64),
                                            (1, 4, 2, 333, 128, 0), (1, 2, 2, 2050, 128, 16)])
def test_error_of_sharp_scores_f32(B, H, Hkv, N, d, bl):
    import numpy as np
    import torch
    rng = np.random.default_rng(N + d)
    Q, K, V = (rng.standard_normal((B, h, n, d), dtype=np.float32) for h, n in ((H, bl or N), (Hkv, N), (Hkv, N)))
    Q *= 3
    t = [to_dev(x) for x in (Q, K, V)]
    O = out_to_f64(dd.dd_block_attention_cached(*t, 5) if bl else dd.dd_bidir_attention(*t), F32)
    torch.cuda.synchronize()
    if bl:
        ref = oracle.block_attention_cached(Q, K, V, 5, F32, F32)
    else:
        rows = np.stack([rng.integers(0, n, 512) for n in (B, H, N)], 1)
        O, ref = O[rows[:, 0], rows[:, 1], rows[:, 2]], oracle.bidir_attention(Q, K, V, F32, F32, rows=rows)
    assert np.linalg.norm(O - ref) <= 7e-7 * np.linalg.norm(ref)     # sqrt(4.4^2 + 1.2^2 + 1.2^2) = 4.7, half as much again for scatter
