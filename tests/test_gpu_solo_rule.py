"""Verifier calls on both sides of the line up to which the kernel whose waves stream keys of their own serves them (workgroups of 32
rows, keys, storage type), against the CPU oracle."""
import pytest

import oracle
import paper_2604_05250_amd as dd
from paper_2604_05250_amd import workloads as wl
from _util import assert_attention_close, out_to_f64, to_dev

pytestmark = pytest.mark.gpu
BF16, FP8 = wl.BF16, wl.FP8_E4M3


@pytest.mark.parametrize("qk,v,d,H,Hkv,N", [
    (BF16, BF16, 64, 48, 48, 512), (BF16, BF16, 64, 45, 45, 513), (BF16, BF16, 64, 46, 46, 513),      # 768, 765 and 782 workgroups
    (BF16, BF16, 64, 38, 38, 511), (BF16, BF16, 64, 38, 38, 512),                                     # 608, shorter and just long enough
    (BF16, BF16, 64, 12, 3, 1345),                                                                    # grouped heads, 507
    (FP8, FP8, 128, 16, 16, 1024), (FP8, FP8, 128, 14, 14, 1057), (FP8, BF16, 128, 14, 14, 1121),     # 512, 476 and 504
    (BF16, BF16, 128, 128, 128, 64), (BF16, BF16, 128, 129, 129, 33), (FP8, BF16, 128, 128, 32, 33), (FP8, BF16, 128, 129, 129, 64),      # 64 keys and
    (FP8, FP8, 128, 128, 128, 64), (FP8, FP8, 128, 129, 129, 33), (BF16, BF16, 64, 96, 96, 64), (BF16, BF16, 64, 97, 97, 33),             # fewer: 256, 192
    (BF16, BF16, 128, 86, 86, 65),                                                                                                       # ... 258 of more
    (BF16, BF16, 128, 11, 11, 1344), (BF16, BF16, 128, 11, 11, 1345), (BF16, BF16, 128, 13, 13, 1231)])      # 462, 473, 507 (not one round of 64 rows)
def test_verifier_calls_at_the_line(qk, v, d, H, Hkv, N):
    import torch
    cfg = wl.custom_config(B=1, H=H, Hkv=Hkv, N=N, d=d, qk_dtype=qk, v_dtype=v)
    inp = wl.attention_inputs(cfg, seed=N + H)
    Q, K, V, qs, ks, vs = (to_dev(inp.get(k)) if inp.get(k) is not None else None for k in ("Q", "K", "V", "q_scale", "k_scale", "v_scale"))
    O = dd.dd_bidir_attention_fp8v(Q, K, V, qs, ks, vs) if v == FP8 else dd.dd_bidir_attention(Q, K, V, q_scale=qs, k_scale=ks, qk_dtype=qk, v_dtype=v)
    torch.cuda.synchronize()
    got = out_to_f64(O, BF16 if v == FP8 else v)
    ref = oracle.bidir_attention(inp["Q"], inp["K"], inp["V"], qk, v, inp["q_scale"], inp["k_scale"], v_scale=inp.get("v_scale"))
    assert_attention_close(got, ref, qk, f"H={H}/{Hkv} N={N} d={d} qk={qk} v={v}")
