"""The two-waves-per-SIMD attention kernel (8 waves = row blocks x key phases) against the CPU oracle, on both of its row tiles:
row counts and key ranges at the edges of its tiles (64 / 128 rows, 128 / 64 keys; phases without a key), block rows that
start and end inside a tile, key splits, positions outside the sequence, windows, and non-finite values it must not spread."""
import numpy as np
import pytest

import oracle
import paper_2604_05250_amd as dd
from paper_2604_05250_amd import workloads as wl
from _util import assert_attention_close, out_to_f64, to_dev

pytestmark = pytest.mark.gpu
STORES = [(wl.BF16, 128), (wl.BF16, 64), (wl.FP8_E4M3, 128)]


@pytest.mark.parametrize("blocks", ["2", "4"])
@pytest.mark.parametrize("qk,d", STORES)
@pytest.mark.parametrize("B,H,Hkv,N", [(1, 1, 1, 1), (1, 2, 1, 31), (2, 3, 1, 33), (1, 2, 2, 64), (1, 3, 3, 65), (1, 4, 1, 127), (2, 2, 2, 128),
                                       (1, 3, 1, 129), (1, 2, 1, 257), (1, 5, 1, 300), (1, 2, 2, 641)])
def test_bidir(monkeypatch, blocks, qk, d, B, H, Hkv, N):
    import torch
    monkeypatch.setenv("DD_TUNE_DUO", blocks)
    cfg = wl.custom_config(B=B, H=H, Hkv=Hkv, N=N, d=d, qk_dtype=qk, v_dtype=wl.BF16, prompt=0, G=N, bl=min(16, N))
    inp = wl.attention_inputs(cfg, seed=N + d)
    O = dd.dd_bidir_attention(to_dev(inp["Q"]), to_dev(inp["K"]), to_dev(inp["V"]), q_scale=to_dev(inp["q_scale"]),
                              k_scale=to_dev(inp["k_scale"]), qk_dtype=qk, v_dtype=wl.BF16)
    torch.cuda.synchronize()
    ref = oracle.bidir_attention(inp["Q"], inp["K"], inp["V"], qk, wl.BF16, inp["q_scale"], inp["k_scale"])
    assert_attention_close(out_to_f64(O, wl.BF16), ref, qk, f"{blocks} blocks {B}x{H}/{Hkv}x{N}x{d}")


# (B, H, Hkv, N, block_len, block_start, key splits): rows per kv head 1, 63-65, 127-129 and several tiles; the block inside
# one tile, across tiles, at either end, the whole sequence
BLOCKS = [(1, 1, 1, 130, 1, 77, 1), (2, 3, 1, 333, 21, 100, 1), (1, 4, 1, 512, 16, 120, 2), (1, 5, 1, 700, 13, 687, 1), (1, 127, 1, 200, 1, 199, 1),
          (2, 8, 2, 515, 32, 0, 2), (1, 3, 1, 1000, 43, 500, 3), (1, 8, 2, 2049, 64, 1000, 8), (1, 7, 1, 300, 150, 150, 1), (1, 2, 1, 100, 100, 0, 1)]


@pytest.mark.parametrize("blocks", ["2", "4"])
@pytest.mark.parametrize("qk,d", STORES)
@pytest.mark.parametrize("B,H,Hkv,N,bl,bs,splits", BLOCKS)
def test_block(monkeypatch, blocks, qk, d, B, H, Hkv, N, bl, bs, splits):
    import torch
    monkeypatch.setenv("DD_TUNE_DUO", blocks)
    monkeypatch.setenv("DD_TUNE_BLOCK_SPLITS", str(splits))
    cfg = wl.custom_config(B=B, H=H, Hkv=Hkv, N=N, d=d, qk_dtype=qk, v_dtype=wl.BF16, bl=bl, prompt=0, G=N)
    cache = wl.cache_inputs(cfg, seed=bs + N)
    blk = wl.block_inputs(cfg, bs, 0, k_scale=cache["k_scale"])
    for fresh in (True, False):
        Kb, Vb = (blk["Kblk"], blk["Vblk"]) if fresh else (None, None)
        O = dd.dd_block_attention_cached(to_dev(blk["Qblk"]), to_dev(cache["Kc"]), to_dev(cache["Vc"]), bs, Kblk=to_dev(Kb), Vblk=to_dev(Vb),
                                         q_scale=to_dev(blk["q_scale"]), k_scale=to_dev(cache["k_scale"]), qk_dtype=qk, v_dtype=wl.BF16)
        torch.cuda.synchronize()
        ref = oracle.block_attention_cached(blk["Qblk"], cache["Kc"], cache["Vc"], bs, qk, wl.BF16, Kb, Vb, blk["q_scale"], cache["k_scale"])
        assert_attention_close(out_to_f64(O, wl.BF16), ref, qk, f"{blocks} blocks {B}x{H}/{Hkv} N{N} d{d} bl{bl}@{bs} splits {splits} fresh={fresh}")


@pytest.mark.parametrize("blocks", ["2", "4"])
@pytest.mark.parametrize("qk", [wl.BF16, wl.FP8_E4M3])
def test_positions_and_window(monkeypatch, blocks, qk):
    # a position per batch entry, some over an end of the sequence or outside it; a window over part of the cache whose other
    # rows, and the rows under the block, hold NaN
    import torch
    monkeypatch.setenv("DD_TUNE_DUO", blocks)
    B, N, bl = 8, 391, 24
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
    assert_attention_close(out_to_f64(O, wl.BF16), ref, qk, f"{blocks} blocks, positions {starts.tolist()}")
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
    assert_attention_close(out_to_f64(O, wl.BF16), ref, qk, f"{blocks} blocks, window")


@pytest.mark.parametrize("blocks", ["2", "4"])
def test_values_that_are_not_finite(monkeypatch, blocks):
    # a NaN query row stays in its row; an infinite value in the last of a ragged number of rows stays infinite, in its dim
    import torch
    monkeypatch.setenv("DD_TUNE_DUO", blocks)
    cfg = wl.custom_config(B=1, H=3, Hkv=1, N=333, d=128, qk_dtype=wl.BF16, v_dtype=wl.BF16, prompt=0, G=333)
    inp = wl.attention_inputs(cfg, seed=5)
    Q, K, V = (to_dev(inp[k]) for k in "QKV")
    want = dd.dd_bidir_attention(Q, K, V)
    q2 = Q.clone()
    q2[0, 1, 5] = 0x7FC0
    got = dd.dd_bidir_attention(q2, K, V)
    torch.cuda.synchronize()
    assert torch.isnan(got[0, 1, 5].view(torch.bfloat16)).all()
    got[0, 1, 5] = want[0, 1, 5]
    assert torch.equal(got, want)
    v2 = V.clone()
    v2[0, 0, 332, 7] = 0x7F80
    got = dd.dd_bidir_attention(Q, K, v2).view(torch.bfloat16)
    torch.cuda.synchronize()
    assert torch.isposinf(got[..., 7]).all() and torch.isfinite(got[..., :7]).all() and torch.isfinite(got[..., 8:]).all()


@pytest.mark.parametrize("blocks", ["2", "4"])
@pytest.mark.parametrize("scale,order", [(1.0, 1), (30.0, 1), (30.0, -1), (1e-3, 1)])
def test_reference_of_the_weights(monkeypatch, blocks, scale, order):
    # scores that grow (the reference is raised again and again), that fall (it stays far above) and that hardly differ
    import torch
    monkeypatch.setenv("DD_TUNE_DUO", blocks)
    rng = np.random.default_rng(3)
    N = 700
    Q = np.abs(rng.standard_normal((1, 2, N, 128), dtype=np.float32))
    K = np.abs(rng.standard_normal((1, 1, N, 128), dtype=np.float32)) * (np.linspace(0.0, 1.0, N, dtype=np.float32)[::order, None] * scale / 10)
    V = rng.standard_normal((1, 1, N, 128), dtype=np.float32)
    Q, K, V = (wl.f32_to_bf16_bits(np.ascontiguousarray(x)) for x in (Q, K, V))
    O = dd.dd_bidir_attention(to_dev(Q), to_dev(K), to_dev(V))
    torch.cuda.synchronize()
    ref = oracle.bidir_attention(Q, K, V, wl.BF16, wl.BF16)
    assert_attention_close(out_to_f64(O, wl.BF16), ref, wl.BF16, f"{blocks} blocks, scale {scale} order {order}")


@pytest.mark.parametrize("call", ["bidir", "block"])
def test_switching_this_kernel_off_moves_no_other_call(monkeypatch, call):
    # a call of the kernel whose waves stream keys of their own, by the rule: the same bits without this kernel, others when it is off
    import torch
    N, bl = 301, 301 if call == "bidir" else 16
    cfg = wl.custom_config(B=1, H=4, Hkv=2, N=N, d=128, qk_dtype=wl.BF16, v_dtype=wl.BF16, bl=bl, prompt=0, G=N)
    cache, blk = wl.cache_inputs(cfg, seed=N), wl.block_inputs(cfg, 0, 0)
    Q, K, V = to_dev(blk["Qblk"]), to_dev(cache["Kc"]), to_dev(cache["Vc"])

    def run(**env):
        for k in ("DD_TUNE_DUO", "DD_TUNE_SOLO"):
            monkeypatch.delenv(k, raising=False)
        for k, v in env.items():
            monkeypatch.setenv(k, v)
        O = dd.dd_bidir_attention(Q, K, V) if call == "bidir" else dd.dd_block_attention_cached(Q, K, V, 0)
        torch.cuda.synchronize()
        return O
    rule = run()
    assert torch.equal(rule, run(DD_TUNE_SOLO="1"))
    assert torch.equal(rule, run(DD_TUNE_DUO="0")) and not torch.equal(rule, run(DD_TUNE_SOLO="0"))
