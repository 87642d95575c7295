"""Drafter calls with fp8 Q/K and at most 64 query rows per kv head on the streaming kernel: against the CPU oracle at the
contract's fp8 tolerance, and against the MFMA kernel that served them before (same operands, same matrix instruction, both
round the weights to bf16: they differ by the order of the fp32 sums and the maxima in use, one bf16 step of an output)."""
import numpy as np
import pytest

import oracle
import paper_2604_05250_amd as dd
from paper_2604_05250_amd import workloads as wl
from _util import assert_attention_close, out_to_f64, to_dev

pytestmark = pytest.mark.gpu
FP8 = wl.FP8_E4M3

# (B, H, Hkv, N, bl, block_start, forced key splits): one key, less than a tile, the edges of one to four tiles (the ring's
# depth), more tiles than the ring, a block at both ends and across tiles, one query row, 33 rows (a second row block nearly
# empty), GQA up to 64 rows, splits of one tile and of unequal length
SHAPES = [(1, 2, 1, 1, 1, 0, None), (1, 2, 2, 17, 16, 1, None), (2, 4, 1, 64, 16, 48, None), (1, 4, 2, 65, 32, 20, None),
          (1, 8, 1, 128, 8, 60, None), (1, 3, 3, 193, 33, 100, None), (2, 4, 2, 256, 32, 0, None), (1, 4, 1, 257, 16, 241, None),
          (3, 8, 2, 700, 16, 333, None), (1, 2, 2, 1237, 64, 900, "3"), (1, 4, 4, 2048, 1, 2047, "16"), (2, 28, 4, 321, 8, 7, "2")]


@pytest.mark.parametrize("B,H,Hkv,N,bl,bs,splits", SHAPES)
def test_block_fp8(monkeypatch, B, H, Hkv, N, bl, bs, splits):
    import torch
    monkeypatch.setenv("DD_TUNE_BLOCK_STREAM", "1")        # (by the rule such small calls run on another kernel)
    if splits:
        monkeypatch.setenv("DD_TUNE_BLOCK_SPLITS", splits)
    cfg = wl.custom_config(B=B, H=H, Hkv=Hkv, N=N, d=128, qk_dtype=FP8, v_dtype=wl.BF16, bl=bl, prompt=0, G=N)
    cache = wl.cache_inputs(cfg, seed=bs + N)
    blk = wl.block_inputs(cfg, bs, 0, k_scale=cache["k_scale"])
    for fresh in (True, False):
        Kb, Vb = (blk["Kblk"], blk["Vblk"]) if fresh else (None, None)

        def call():
            O = dd.dd_block_attention_cached(to_dev(blk["Qblk"]), to_dev(cache["Kc"]), to_dev(cache["Vc"]), bs, Kblk=to_dev(Kb),
                                             Vblk=to_dev(Vb), q_scale=to_dev(blk["q_scale"]), k_scale=to_dev(cache["k_scale"]),
                                             qk_dtype=FP8, v_dtype=wl.BF16)
            torch.cuda.synchronize()
            return out_to_f64(O, wl.BF16)
        got = call()
        ref = oracle.block_attention_cached(blk["Qblk"], cache["Kc"], cache["Vc"], bs, FP8, wl.BF16, Kb, Vb, blk["q_scale"],
                                            cache["k_scale"])
        what = f"fp8 streaming {B}x{H}/{Hkv} N{N} bl{bl}@{bs} splits {splits} fresh={fresh}"
        assert_attention_close(got, ref, FP8, what)
        monkeypatch.setenv("DD_TUNE_BLOCK_STREAM", "0")
        old = call()
        monkeypatch.setenv("DD_TUNE_BLOCK_STREAM", "1")
        # no precision lost: both errors are roundings of the weights and of n >= 128 outputs, whose 2-norms scatter by about
        # 1 / sqrt(2 n) <= 6 %; 1.25 is four of those
        assert np.linalg.norm(got - ref) <= 1.25 * np.linalg.norm(old - ref) + 1e-6 * np.linalg.norm(ref), what


@pytest.mark.parametrize("stream", ["1", None])               # (None: the kernel of the library's own rule)
@pytest.mark.parametrize("N,win", [(333, 100), (1000, 64), (1237, 600)])
def test_window_batched_refresh_fp8(monkeypatch, N, win, stream):
    import torch
    if stream:
        monkeypatch.setenv("DD_TUNE_BLOCK_STREAM", stream)
    B, bl = 3, 16
    cfg = wl.custom_config(B=B, H=8, Hkv=2, N=N, d=128, qk_dtype=FP8, v_dtype=wl.BF16, bl=bl, prompt=0, G=N)
    cache = wl.cache_inputs(cfg, seed=N)
    blk = wl.block_inputs(cfg, 0, 0, k_scale=cache["k_scale"])
    scales = {"q_scale": to_dev(blk["q_scale"]), "k_scale": to_dev(cache["k_scale"]), "qk_dtype": FP8, "v_dtype": wl.BF16}
    Q, Kb, Vb = to_dev(blk["Qblk"]), to_dev(blk["Kblk"]), to_dev(blk["Vblk"])
    ws = N - win - 5
    O = dd.dd_block_attention_window(Q, to_dev(cache["Kc"]), to_dev(cache["Vc"]), ws + 3, ws, win, Kblk=Kb, Vblk=Vb, **scales)
    cut = {k: np.ascontiguousarray(cache[k][:, :, ws:ws + win]) for k in ("Kc", "Vc")}
    ref = oracle.block_attention_cached(blk["Qblk"], cut["Kc"], cut["Vc"], 3, FP8, wl.BF16, blk["Kblk"], blk["Vblk"],
                                        blk["q_scale"], cache["k_scale"])
    torch.cuda.synchronize()
    assert_attention_close(out_to_f64(O, wl.BF16), ref, FP8, f"fp8 window {win} of {N}")
    starts = np.array([0, N - bl, N // 3], np.int32)
    O = dd.dd_block_attention_batched(Q, to_dev(cache["Kc"]), to_dev(cache["Vc"]), torch.from_numpy(starts).to("cuda:0"), Kb, Vb, **scales)
    ref = oracle.block_attention_batched(blk["Qblk"], cache["Kc"], cache["Vc"], starts, FP8, wl.BF16, blk["Kblk"], blk["Vblk"],
                                         blk["q_scale"], cache["k_scale"])
    torch.cuda.synchronize()
    assert_attention_close(out_to_f64(O, wl.BF16), ref, FP8, f"fp8 batched {N}")
    Kc, Vc = to_dev(cache["Kc"]), to_dev(cache["Vc"])
    O = dd.dd_block_attention_refresh(Q, Kc, Vc, 7, Kb, Vb, **scales)
    ref = oracle.block_attention_cached(blk["Qblk"], cache["Kc"], cache["Vc"], 7, FP8, wl.BF16, blk["Kblk"], blk["Vblk"],
                                        blk["q_scale"], cache["k_scale"])
    torch.cuda.synchronize()
    assert_attention_close(out_to_f64(O, wl.BF16), ref, FP8, f"fp8 refresh {N}")
    for have, block, before in ((Kc, Kb, cache["Kc"]), (Vc, Vb, cache["Vc"])):
        want = to_dev(before).clone()
        want[:, :, 7:7 + bl] = block
        assert torch.equal(have, want)
