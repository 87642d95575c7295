"""The drafter's kernel whose waves stream keys of their own against the CPU oracle: row counts at the edges of
its 32-row tiles, key ranges at the edges of its 32-key units and of a round of them (waves without a unit, with one, with a ragged
one), block rows that start and end inside a unit, key splits, positions outside the sequence, windows, refresh, and non-finite
values it must not spread."""
import numpy as np
import pytest

import oracle
import paper_2604_05250_amd as dd
from paper_2604_05250_amd import workloads as wl
from _util import assert_attention_close, out_to_f64, to_dev

pytestmark = pytest.mark.gpu
STORES = [(wl.BF16, 128), (wl.BF16, 64), (wl.FP8_E4M3, 128)]
# (B, H, Hkv, N, block_len, block_start, key splits)
BLOCKS = [(1, 1, 1, 1, 1, 0, 1), (1, 1, 1, 31, 1, 30, 1), (2, 2, 2, 32, 32, 0, 1), (1, 33, 1, 33, 1, 32, 1), (1, 4, 1, 127, 8, 60, 1),
          (1, 2, 1, 129, 31, 90, 1), (2, 3, 1, 255, 21, 100, 1), (1, 4, 2, 257, 16, 250 - 9, 1), (1, 8, 8, 512, 32, 200, 1), (1, 2, 1, 641, 32, 609, 1),
          (3, 8, 2, 700, 16, 333, 4), (1, 64, 1, 1000, 1, 999, 3), (1, 5, 1, 2049, 12, 1000, 16),
          (1, 5, 1, 700, 13, 687, 1), (2, 8, 2, 515, 32, 0, 2), (1, 7, 1, 300, 150, 150, 1)]


def _call(inputs, Kb, Vb, fn=dd.dd_block_attention_cached, K=None, V=None):
    blk, cache, bs, qk = inputs
    return fn(to_dev(blk["Qblk"]), to_dev(cache["Kc"]) if K is None else K, to_dev(cache["Vc"]) if V is None else V, bs,
              Kblk=to_dev(Kb), Vblk=to_dev(Vb), q_scale=to_dev(blk["q_scale"]), k_scale=to_dev(cache["k_scale"]), qk_dtype=qk, v_dtype=wl.BF16)


@pytest.mark.parametrize("solo", ["1", "0"])                 # (0: the same calls on the kernels before it)
@pytest.mark.parametrize("qk,d", STORES)
@pytest.mark.parametrize("B,H,Hkv,N,bl,bs,splits", BLOCKS)
def test_block(monkeypatch, solo, qk, d, B, H, Hkv, N, bl, bs, splits):
    import torch
    monkeypatch.setenv("DD_TUNE_SOLO", solo)
    monkeypatch.setenv("DD_TUNE_BLOCK_SPLITS", str(splits))
    cfg = wl.custom_config(B=B, H=H, Hkv=Hkv, N=N, d=d, qk_dtype=qk, v_dtype=wl.BF16, bl=bl, prompt=0, G=N)
    cache = wl.cache_inputs(cfg, seed=bs + N)
    blk = wl.block_inputs(cfg, bs, 0, k_scale=cache["k_scale"])
    for fresh in (True, False):
        Kb, Vb = (blk["Kblk"], blk["Vblk"]) if fresh else (None, None)
        O = _call((blk, cache, bs, qk), Kb, Vb)
        torch.cuda.synchronize()
        ref = oracle.block_attention_cached(blk["Qblk"], cache["Kc"], cache["Vc"], bs, qk, wl.BF16, Kb, Vb, blk["q_scale"], cache["k_scale"])
        assert_attention_close(out_to_f64(O, wl.BF16), ref, qk, f"solo {solo} {B}x{H}/{Hkv} N{N} d{d} bl{bl}@{bs} splits {splits} fresh={fresh}")


@pytest.mark.parametrize("solo", ["1", "0"])
@pytest.mark.parametrize("qk", [wl.BF16, wl.FP8_E4M3])
def test_positions_window_and_refresh(monkeypatch, solo, qk):
    # a position per batch entry, some over an end of the sequence or outside it; a window over part of the cache whose other
    # rows, and the rows under the block, hold NaN; the block's rows written back
    import torch
    monkeypatch.setenv("DD_TUNE_SOLO", solo)
    B, N, bl = 8, 391, 12
    cfg = wl.custom_config(B=B, H=8, Hkv=2, N=N, d=128, bl=bl, qk_dtype=qk, v_dtype=wl.BF16, prompt=0, G=N)
    cache = wl.cache_inputs(cfg, seed=N)
    blk = wl.block_inputs(cfg, N, 0, k_scale=cache["k_scale"])
    starts = np.array([0, N - bl, -10, N - 5, -bl, N, 100, -(2**31)], np.int32)
    scales = {"q_scale": to_dev(blk["q_scale"]), "k_scale": to_dev(cache["k_scale"]), "qk_dtype": qk, "v_dtype": wl.BF16}
    O = dd.dd_block_attention_batched(to_dev(blk["Qblk"]), to_dev(cache["Kc"]), to_dev(cache["Vc"]), torch.from_numpy(starts).to("cuda:0"),
                                      to_dev(blk["Kblk"]), to_dev(blk["Vblk"]), **scales)
    torch.cuda.synchronize()
    ref = oracle.block_attention_batched(blk["Qblk"], cache["Kc"], cache["Vc"], starts, qk, wl.BF16, blk["Kblk"], blk["Vblk"],
                                         blk["q_scale"], cache["k_scale"])
    assert_attention_close(out_to_f64(O, wl.BF16), ref, qk, f"positions {starts.tolist()}")
    first, length, bs = 37, 211, 130
    K, V = to_dev(cache["Kc"]), to_dev(cache["Vc"])
    for t in (K, V):
        nan = 0x7F if t.element_size() == 1 else 0x7FC0
        t[:, :, :first] = nan
        t[:, :, first + length:] = nan
        t[:, :, bs:bs + bl] = nan
    O = dd.dd_block_attention_window(to_dev(blk["Qblk"]), K, V, bs, first, length, Kblk=to_dev(blk["Kblk"]), Vblk=to_dev(blk["Vblk"]), **scales)
    torch.cuda.synchronize()
    ref = oracle.block_attention_cached(blk["Qblk"], cache["Kc"][:, :, first:first + length], cache["Vc"][:, :, first:first + length],
                                        bs - first, qk, wl.BF16, blk["Kblk"], blk["Vblk"], blk["q_scale"], cache["k_scale"])
    assert_attention_close(out_to_f64(O, wl.BF16), ref, qk, f"window")
    K, V = to_dev(cache["Kc"]), to_dev(cache["Vc"])
    O = _call((blk, cache, bs, qk), blk["Kblk"], blk["Vblk"], dd.dd_block_attention_refresh, K=K, V=V)
    torch.cuda.synchronize()
    ref = oracle.block_attention_cached(blk["Qblk"], cache["Kc"], cache["Vc"], bs, qk, wl.BF16, blk["Kblk"], blk["Vblk"], blk["q_scale"], cache["k_scale"])
    assert_attention_close(out_to_f64(O, wl.BF16), ref, qk, f"refresh")
    assert torch.equal(K[:, :, bs:bs + bl], to_dev(blk["Kblk"])) and torch.equal(V[:, :, bs:bs + bl], to_dev(blk["Vblk"]))


def test_values_that_are_not_finite(monkeypatch):
    # a NaN query row stays in its row; an infinite value in the last of a ragged number of rows stays infinite, in its dim
    import torch
    monkeypatch.setenv("DD_TUNE_SOLO", "1")
    cfg = wl.custom_config(B=1, H=3, Hkv=1, N=333, d=128, bl=16, qk_dtype=wl.BF16, v_dtype=wl.BF16, prompt=0, G=333)
    cache, blk = wl.cache_inputs(cfg, seed=5), wl.block_inputs(cfg, 5, 0)
    Q, K, V = to_dev(blk["Qblk"]), to_dev(cache["Kc"]), to_dev(cache["Vc"])
    want = dd.dd_block_attention_cached(Q, K, V, 100)
    q2 = Q.clone()
    q2[0, 1, 5] = 0x7FC0
    got = dd.dd_block_attention_cached(q2, K, V, 100)
    torch.cuda.synchronize()
    assert torch.isnan(got[0, 1, 5].view(torch.bfloat16)).all()
    got[0, 1, 5] = want[0, 1, 5]
    assert torch.equal(got, want)
    v2 = V.clone()
    v2[0, 0, 332, 7] = 0x7F80
    got = dd.dd_block_attention_cached(Q, K, v2, 100).view(torch.bfloat16)
    torch.cuda.synchronize()
    assert torch.isposinf(got[..., 7]).all() and torch.isfinite(got[..., :7]).all() and torch.isfinite(got[..., 8:]).all()


# (the last row of a ragged range in the cache or in the block; e4m3 has no infinity: there a NaN, which stays in its dim as well)
@pytest.mark.parametrize("fresh", [False, True])
@pytest.mark.parametrize("qk,v,d", [(wl.BF16, wl.BF16, 64), (wl.BF16, wl.BF16, 128), (wl.FP8_E4M3, wl.BF16, 128), (wl.FP8_E4M3, wl.FP8_E4M3, 128)])
def test_values_that_are_not_finite_in_every_storage(monkeypatch, qk, v, d, fresh):
    import torch
    monkeypatch.setenv("DD_TUNE_SOLO", "1")
    cfg = wl.custom_config(B=1, H=3, Hkv=1, N=333, d=d, bl=16, qk_dtype=qk, v_dtype=v, prompt=0, G=333)
    cache = wl.cache_inputs(cfg, seed=5)
    blk = wl.block_inputs(cfg, 5, 0, k_scale=cache["k_scale"], v_scale=cache.get("v_scale"))
    K, qs, ks, vs = (to_dev(x) for x in (cache["Kc"], blk["q_scale"], cache["k_scale"], cache.get("v_scale")))
    Kb, bs = (to_dev(blk["Kblk"]), 333 - 16) if fresh else (None, 100)

    def run(Q, V, Vb):
        if v == wl.FP8_E4M3:
            O = dd.dd_block_attention_cached_fp8v(Q, K, V, bs, qs, ks, vs, Kblk=Kb, Vblk=Vb)
        else:
            O = dd.dd_block_attention_cached(Q, K, V, bs, Kblk=Kb, Vblk=Vb, q_scale=qs, k_scale=ks, qk_dtype=qk, v_dtype=v)
        torch.cuda.synchronize()
        return O
    Q, V, Vb = to_dev(blk["Qblk"]), to_dev(cache["Vc"]), to_dev(blk["Vblk"]) if fresh else None
    want = run(Q, V, Vb)
    q2 = Q.clone()
    q2[0, 1, 5] = 0x7F if qk == wl.FP8_E4M3 else 0x7FC0
    got = run(q2, V, Vb)
    assert torch.isnan(got[0, 1, 5].view(torch.bfloat16)).all()
    got[0, 1, 5] = want[0, 1, 5]
    assert torch.equal(got, want)
    V2, Vb2 = V.clone(), Vb.clone() if fresh else None
    if fresh:                                                # (what the cache holds under the block is not looked at)
        V2[0, 0, bs:bs + 16] = 0x7F if v == wl.FP8_E4M3 else 0x7FC0
    (Vb2 if fresh else V2)[0, 0, -1, 7] = 0x7F if v == wl.FP8_E4M3 else 0x7F80
    got = run(Q, V2, Vb2).view(torch.bfloat16)
    bad = torch.isnan(got[..., 7]) if v == wl.FP8_E4M3 else torch.isposinf(got[..., 7])
    assert bad.all() and torch.isfinite(got[..., :7]).all() and torch.isfinite(got[..., 8:]).all()


@pytest.mark.parametrize("scale,order", [(1.0, 1), (30.0, 1), (30.0, -1), (1e-3, 1)])
def test_reference_of_the_weights(monkeypatch, scale, order):
    # scores that grow (the reference is raised again and again), that fall (it stays far above) and that hardly differ
    import torch
    monkeypatch.setenv("DD_TUNE_SOLO", "1")
    monkeypatch.setenv("DD_TUNE_BLOCK_SPLITS", "1")          # (a wave sees one unit only where the key range is split far enough)
    rng = np.random.default_rng(3)
    N = 1400
    Q = np.abs(rng.standard_normal((1, 2, 32, 128), dtype=np.float32))
    K = np.abs(rng.standard_normal((1, 1, N, 128), dtype=np.float32)) * (np.linspace(0.0, 1.0, N, dtype=np.float32)[::order, None] * scale / 10)
    V = rng.standard_normal((1, 1, N, 128), dtype=np.float32)
    Q, K, V = (wl.f32_to_bf16_bits(np.ascontiguousarray(x)) for x in (Q, K, V))
    O = dd.dd_block_attention_cached(to_dev(Q), to_dev(K), to_dev(V), 700)
    torch.cuda.synchronize()
    ref = oracle.block_attention_cached(Q, K, V, 700, wl.BF16, wl.BF16, None, None, None, None)
    assert_attention_close(out_to_f64(O, wl.BF16), ref, wl.BF16, f"scale {scale} order {order}")


@pytest.mark.parametrize("solo", ["1", "0"])                 # (0: the same calls on the kernels before it)
@pytest.mark.parametrize("B,H,Hkv,N,bl,bs,splits", BLOCKS)
def test_block_fp8v(monkeypatch, solo, B, H, Hkv, N, bl, bs, splits):
    import torch
    monkeypatch.setenv("DD_TUNE_SOLO", solo)
    monkeypatch.setenv("DD_TUNE_BLOCK_SPLITS", str(splits))
    fp8 = wl.FP8_E4M3
    cfg = wl.custom_config(B=B, H=H, Hkv=Hkv, N=N, d=128, qk_dtype=fp8, v_dtype=fp8, bl=bl, prompt=0, G=N)
    cache = wl.cache_inputs(cfg, seed=bs + N)
    blk = wl.block_inputs(cfg, bs, 0, k_scale=cache["k_scale"], v_scale=cache["v_scale"])
    for fresh in (True, False):
        Kb, Vb = (blk["Kblk"], blk["Vblk"]) if fresh else (None, None)
        O = dd.dd_block_attention_cached_fp8v(to_dev(blk["Qblk"]), to_dev(cache["Kc"]), to_dev(cache["Vc"]), bs, to_dev(blk["q_scale"]),
                                              to_dev(cache["k_scale"]), to_dev(cache["v_scale"]), Kblk=to_dev(Kb), Vblk=to_dev(Vb))
        torch.cuda.synchronize()
        ref = oracle.block_attention_cached(blk["Qblk"], cache["Kc"], cache["Vc"], bs, fp8, fp8, Kb, Vb, blk["q_scale"], cache["k_scale"],
                                            v_scale=cache["v_scale"])
        assert_attention_close(out_to_f64(O, wl.BF16), ref, fp8, f"fp8v, solo {solo} {B}x{H}/{Hkv} N{N} bl{bl}@{bs} splits {splits} fresh={fresh}")


# (one row; a tile's rows and one more; a wave's first, second and ragged unit; grouped heads that share tiles)
@pytest.mark.parametrize("solo", ["1", "0"])                 # (0: the same calls on the kernels before it)
@pytest.mark.parametrize("qk,v,d", [(wl.BF16, wl.BF16, 128), (wl.BF16, wl.BF16, 64), (wl.FP8_E4M3, wl.BF16, 128), (wl.FP8_E4M3, wl.FP8_E4M3, 128)])
@pytest.mark.parametrize("B,H,Hkv,N", [(1, 1, 1, 1), (1, 2, 1, 31), (2, 3, 1, 33), (1, 2, 2, 64), (1, 3, 3, 65), (1, 4, 1, 127), (2, 2, 2, 128),
                                       (1, 3, 1, 129), (1, 2, 1, 257), (1, 5, 1, 300), (1, 2, 2, 641)])
def test_bidir(monkeypatch, solo, qk, v, d, B, H, Hkv, N):
    import torch
    monkeypatch.setenv("DD_TUNE_SOLO", solo)
    cfg = wl.custom_config(B=B, H=H, Hkv=Hkv, N=N, d=d, qk_dtype=qk, v_dtype=v, prompt=0, G=N, bl=min(16, N))
    inp = wl.attention_inputs(cfg, seed=N + d)
    Q, K, V, qs, ks = (to_dev(inp[k]) for k in ("Q", "K", "V", "q_scale", "k_scale"))
    if v == wl.FP8_E4M3:
        O = dd.dd_bidir_attention_fp8v(Q, K, V, qs, ks, to_dev(inp["v_scale"]))
    else:
        O = dd.dd_bidir_attention(Q, K, V, q_scale=qs, k_scale=ks, qk_dtype=qk, v_dtype=v)
    torch.cuda.synchronize()
    ref = oracle.bidir_attention(inp["Q"], inp["K"], inp["V"], qk, v, inp["q_scale"], inp["k_scale"], v_scale=inp.get("v_scale"))
    assert_attention_close(out_to_f64(O, wl.BF16), ref, qk, f"solo {solo} {B}x{H}/{Hkv}x{N}x{d}")
