"""Every form of the kernel whose waves stream keys of their own (row blocks, parts of the head dims, waves) against the CPU oracle: rows
at the edges of one and two blocks of 32, key ranges that leave waves of four and of eight without a unit, with one and with a ragged
one, key splits, and the block's rows written back beside a call whose head dims are divided."""
import pytest

import oracle
import paper_2604_05250_amd as dd
from paper_2604_05250_amd import workloads as wl
from _util import assert_attention_close, out_to_f64, to_dev

pytestmark = pytest.mark.gpu
BF16, FP8 = wl.BF16, wl.FP8_E4M3
FORMS = [(qk, v, d, f) for qk, v, d, forms in ((BF16, BF16, 128, (114, 124, 128, 144, 148, 224)), (FP8, BF16, 128, (114, 124, 128, 144, 148, 228)),
                                               (FP8, FP8, 128, (114, 124, 128, 144, 148, 224, 228)), (BF16, BF16, 64, (114, 118, 124, 128))) for f in forms]
# (B, H, Hkv, N, block_len, block_start, key splits)
CALLS = [(1, 1, 1, 31, 1, 30, 1), (2, 4, 2, 129, 16, 100, 1), (1, 3, 1, 257, 11, 0, 1), (1, 2, 1, 300, 32, 250, 1), (1, 5, 1, 641, 13, 628, 3), (2, 2, 2, 1000, 31, 480, 4)]


@pytest.mark.parametrize("qk,v,d,form", FORMS)
@pytest.mark.parametrize("B,H,Hkv,N,bl,bs,splits", CALLS)
def test_block(monkeypatch, qk, v, d, form, B, H, Hkv, N, bl, bs, splits):
    import torch
    monkeypatch.setenv("DD_TUNE_SOLO", "1")
    monkeypatch.setenv("DD_TUNE_SOLO_FORM", str(form))
    monkeypatch.setenv("DD_TUNE_BLOCK_SPLITS", str(splits))
    cfg = wl.custom_config(B=B, H=H, Hkv=Hkv, N=N, d=d, qk_dtype=qk, v_dtype=v, bl=bl, prompt=0, G=N)
    cache = wl.cache_inputs(cfg, seed=bs + N)
    blk = wl.block_inputs(cfg, bs, 0, k_scale=cache["k_scale"], v_scale=cache.get("v_scale"))
    Q, K, V, Kb, Vb, qs, ks, vs = (to_dev(x) for x in (blk["Qblk"], cache["Kc"], cache["Vc"], blk["Kblk"], blk["Vblk"], blk["q_scale"],
                                                       cache["k_scale"], cache.get("v_scale")))
    ref = oracle.block_attention_cached(blk["Qblk"], cache["Kc"], cache["Vc"], bs, qk, v, blk["Kblk"], blk["Vblk"], blk["q_scale"], cache["k_scale"],
                                        v_scale=cache.get("v_scale"))
    what = f"form {form} {B}x{H}/{Hkv} N{N} d{d} bl{bl}@{bs} splits {splits}"
    if v == FP8:
        O = dd.dd_block_attention_cached_fp8v(Q, K, V, bs, qs, ks, vs, Kblk=Kb, Vblk=Vb)
    else:
        O = dd.dd_block_attention_refresh(Q, K, V, bs, Kblk=Kb, Vblk=Vb, q_scale=qs, k_scale=ks, qk_dtype=qk, v_dtype=v)
    torch.cuda.synchronize()
    assert_attention_close(out_to_f64(O, BF16), ref, qk, what)
    if v != FP8:
        assert torch.equal(K[:, :, bs:bs + bl], Kb) and torch.equal(V[:, :, bs:bs + bl], Vb)
    if splits == 1:                                          # the verifier's call on the same heads
        inp = wl.attention_inputs(cfg, seed=N + d)
        Q, K, V, qs, ks, vs = (to_dev(inp.get(k)) for k in ("Q", "K", "V", "q_scale", "k_scale", "v_scale"))
        O = dd.dd_bidir_attention_fp8v(Q, K, V, qs, ks, vs) if v == FP8 else dd.dd_bidir_attention(Q, K, V, q_scale=qs, k_scale=ks, qk_dtype=qk, v_dtype=v)
        torch.cuda.synchronize()
        ref = oracle.bidir_attention(inp["Q"], inp["K"], inp["V"], qk, v, inp["q_scale"], inp["k_scale"], v_scale=inp.get("v_scale"))
        assert_attention_close(out_to_f64(O, BF16), ref, qk, "verifier, " + what)
