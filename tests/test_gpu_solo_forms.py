"""Every form of the kernel whose waves stream keys of their own (row blocks, parts of the head dims, waves) against the CPU oracle: rows
at the edges of one and two blocks of 32, key ranges that leave waves of four and of eight without a unit, with one and with a ragged
one, with three and more, key splits, and the block's rows written back beside a call whose head dims are divided; weights whose
reference is raised again and again, in one row block and not in the other; values that are not finite; positions per batch entry and windows."""
import numpy as np
import pytest

import oracle
import paper_2604_05250_amd as dd
from paper_2604_05250_amd import workloads as wl
from _kernels import SOLO_FORMS, solo_form
from _util import assert_attention_close, out_to_f64, to_dev

pytestmark = pytest.mark.gpu
BF16, FP8 = wl.BF16, wl.FP8_E4M3
FORMS = [(*store, f) for store, forms in SOLO_FORMS.items() for f in forms]
# (B, H, Hkv, N, block_len, block_start, key splits)
CALLS = [(1, 1, 1, 31, 1, 30, 1), (2, 4, 2, 129, 16, 100, 1), (1, 3, 1, 257, 11, 0, 1), (1, 2, 1, 300, 32, 250, 1), (1, 5, 1, 641, 13, 628, 3), (2, 2, 2, 1000, 31, 480, 4),
         (1, 4, 1, 801, 11, 500, 1)]


def set_env(monkeypatch, env):
    for k, x in env.items():
        monkeypatch.setenv(k, x)


@pytest.mark.parametrize("qk,v,d,form", FORMS)
@pytest.mark.parametrize("B,H,Hkv,N,bl,bs,splits", CALLS)
def test_block(monkeypatch, qk, v, d, form, B, H, Hkv, N, bl, bs, splits):
    import torch
    set_env(monkeypatch, solo_form(form, splits))
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


def run_block(qk, v, Q, K, V, bs, Kb, Vb, qs, ks, vs):
    import torch
    if v == FP8:
        O = dd.dd_block_attention_cached_fp8v(Q, K, V, bs, qs, ks, vs, Kblk=Kb, Vblk=Vb)
    else:
        O = dd.dd_block_attention_cached(Q, K, V, bs, Kblk=Kb, Vblk=Vb, q_scale=qs, k_scale=ks, qk_dtype=qk, v_dtype=v)
    torch.cuda.synchronize()
    return O


def stored(x, t):
    if t != FP8:
        return wl.f32_to_bf16_bits(x), None
    scale = np.abs(x).max(axis=(2, 3)) / np.float32(448.0)
    return wl.f32_to_e4m3_bits(x / scale[:, :, None, None]), scale


# One split, so that a wave of eight has six units (four: eleven).  Head 0's rows are the first row block, head 1's the second: their scores
# grow along the keys, so that the reference is raised again and again, or fall, so that it stays far above, in either block or both.
@pytest.mark.parametrize("signs", [(1, 1), (1, -1), (-1, 1)])
@pytest.mark.parametrize("scale", [30.0, 1e-3])
@pytest.mark.parametrize("qk,v,d,form", FORMS)
def test_reference_of_the_weights(monkeypatch, qk, v, d, form, scale, signs):
    set_env(monkeypatch, solo_form(form))
    rng = np.random.default_rng(3)
    N = 1400
    Q = np.abs(rng.standard_normal((1, 2, 32, d), dtype=np.float32)) * np.float32(signs)[None, :, None, None]
    K = np.abs(rng.standard_normal((1, 1, N, d), dtype=np.float32)) * (np.linspace(0.0, 1.0, N, dtype=np.float32)[:, None] * scale / 10)
    V = rng.standard_normal((1, 1, N, d), dtype=np.float32)
    (Qc, qs), (Kc, ks), (Vc, vs) = (stored(x, t) for x, t in ((Q, qk), (K, qk), (V, v)))
    O = run_block(qk, v, *(to_dev(x) for x in (Qc, Kc, Vc)), 700, None, None, *(to_dev(x) for x in (qs, ks, vs)))
    ref = oracle.block_attention_cached(Qc, Kc, Vc, 700, qk, v, None, None, qs, ks, v_scale=vs)
    assert_attention_close(out_to_f64(O, BF16), ref, qk, f"form {form} scale {scale} signs {signs}")


# (the last row of a ragged range in the cache or in the block; e4m3 has no infinity: there a NaN, which stays in its dim as well)
@pytest.mark.parametrize("fresh", [False, True])
@pytest.mark.parametrize("qk,v,d,form", FORMS)
def test_values_that_are_not_finite(monkeypatch, qk, v, d, form, fresh):
    import torch
    set_env(monkeypatch, solo_form(form))
    N = 333
    cfg = wl.custom_config(B=1, H=3, Hkv=1, N=N, d=d, bl=16, qk_dtype=qk, v_dtype=v, prompt=0, G=N)
    cache = wl.cache_inputs(cfg, seed=5)
    blk = wl.block_inputs(cfg, 5, 0, k_scale=cache["k_scale"], v_scale=cache.get("v_scale"))
    Q, K, V, qs, ks, vs = (to_dev(x) for x in (blk["Qblk"], cache["Kc"], cache["Vc"], blk["q_scale"], cache["k_scale"], cache.get("v_scale")))
    Kb, Vb, bs = (to_dev(blk["Kblk"]), to_dev(blk["Vblk"]), N - 16) if fresh else (None, None, 100)
    nan_q, nan_v, bad_v = 0x7F if qk == FP8 else 0x7FC0, 0x7F if v == FP8 else 0x7FC0, 0x7F if v == FP8 else 0x7F80
    want = run_block(qk, v, Q, K, V, bs, Kb, Vb, qs, ks, vs)
    for head in (0, 2):                                      # 48 rows: the first row block, the second
        q2 = Q.clone()
        q2[0, head, 5] = nan_q
        got = run_block(qk, v, q2, K, V, bs, Kb, Vb, qs, ks, vs)
        assert torch.isnan(got[0, head, 5].view(torch.bfloat16)).all()
        got[0, head, 5] = want[0, head, 5]
        assert torch.equal(got, want)
    V2, Vb2 = V.clone(), Vb.clone() if fresh else None
    if fresh:                                                # (what the cache holds under the block is not looked at)
        V2[0, 0, bs:bs + 16] = nan_v
    (Vb2 if fresh else V2)[0, 0, -1, 7] = bad_v
    got = run_block(qk, v, Q, K, V2, bs, Kb, Vb2, qs, ks, vs).view(torch.bfloat16)
    bad = torch.isnan(got[..., 7]) if v == FP8 else torch.isposinf(got[..., 7])
    assert bad.all() and torch.isfinite(got[..., :7]).all() and torch.isfinite(got[..., 8:]).all()


@pytest.mark.parametrize("qk,v,d,form", [f for f in FORMS if f[1] != FP8])
def test_positions_and_window(monkeypatch, qk, v, d, form):
    # a position per batch entry, some over an end of the sequence or outside it; a window over part of the cache whose other
    # rows, and the rows under the block, hold NaN
    import torch
    set_env(monkeypatch, solo_form(form))
    B, N, bl = 8, 391, 12
    cfg = wl.custom_config(B=B, H=8, Hkv=2, N=N, d=d, bl=bl, qk_dtype=qk, v_dtype=v, prompt=0, G=N)
    cache = wl.cache_inputs(cfg, seed=N)
    blk = wl.block_inputs(cfg, N, 0, k_scale=cache["k_scale"])
    Q, Kb, Vb = (to_dev(blk[k]) for k in ("Qblk", "Kblk", "Vblk"))
    scales = {"q_scale": to_dev(blk["q_scale"]), "k_scale": to_dev(cache["k_scale"]), "qk_dtype": qk, "v_dtype": v}
    starts = np.array([0, N - bl, -10, N - 5, -bl, N, 100, -(2**31)], np.int32)
    O = dd.dd_block_attention_batched(Q, to_dev(cache["Kc"]), to_dev(cache["Vc"]), torch.from_numpy(starts).to("cuda:0"), Kb, Vb, **scales)
    torch.cuda.synchronize()
    ref = oracle.block_attention_batched(blk["Qblk"], cache["Kc"], cache["Vc"], starts, qk, v, blk["Kblk"], blk["Vblk"], blk["q_scale"], cache["k_scale"])
    assert_attention_close(out_to_f64(O, BF16), ref, qk, f"form {form} positions {starts.tolist()}")
    first, length, bs = 37, 311, 130
    K, V = to_dev(cache["Kc"]), to_dev(cache["Vc"])
    for t in (K, V):
        nan = 0x7F if t.element_size() == 1 else 0x7FC0
        t[:, :, :first] = nan
        t[:, :, first + length:] = nan
        t[:, :, bs:bs + bl] = nan
    O = dd.dd_block_attention_window(Q, K, V, bs, first, length, Kblk=Kb, Vblk=Vb, **scales)
    torch.cuda.synchronize()
    ref = oracle.block_attention_cached(blk["Qblk"], cache["Kc"][:, :, first:first + length], cache["Vc"][:, :, first:first + length],
                                        bs - first, qk, v, blk["Kblk"], blk["Vblk"], blk["q_scale"], cache["k_scale"])
    assert_attention_close(out_to_f64(O, BF16), ref, qk, f"form {form} window")
