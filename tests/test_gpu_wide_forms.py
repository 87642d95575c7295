"""The wide kernel's forms beside the 256-row bf16 / fp8 one: V tiles decoded on their way to the matrix cores (e4m3, and
block-scaled e2m1), and verifier calls on 128-row tiles, against the CPU oracle at the contract's tolerances.  Shapes: one row
tile and several per workgroup, key ranges at the edges of the 64-key tiles, an even and an odd tile count, GQA groups that
end inside a row tile; the drafter's form on both row tiles, with and without key splits."""
import numpy as np
import pytest

import oracle
import paper_2604_05250_amd as dd
from paper_2604_05250_amd import workloads as wl
from _util import assert_attention_close, out_to_f64, to_dev

pytestmark = pytest.mark.gpu
FP8 = wl.FP8_E4M3

# (B, H, Hkv, N, cap on the persistent workgroups)
SHAPES = [(1, 2, 2, 64, None), (1, 2, 1, 65, None), (2, 3, 1, 127, None), (1, 4, 4, 128, "1"), (1, 4, 2, 129, "2"),
          (2, 4, 1, 255, "3"), (1, 5, 5, 320, "2"), (1, 3, 1, 641, "1"), (2, 7, 1, 1000, "5")]


@pytest.mark.parametrize("B,H,Hkv,N,grid", SHAPES)
@pytest.mark.parametrize("store", ["fp8v", "mx"])
@pytest.mark.parametrize("tile", ["256", "128"])
def test_bidir_decoded_v(monkeypatch, store, tile, B, H, Hkv, N, grid):
    import torch
    monkeypatch.setenv("DD_TUNE_ATTN_WIDE", "1" if tile == "256" else "2")
    if grid:
        monkeypatch.setenv("DD_TUNE_ATTN_WIDE_GRID", grid)
    cfg = wl.custom_config(B=B, H=H, Hkv=Hkv, N=N, d=128, qk_dtype=FP8, v_dtype=FP8, prompt=0, G=N, bl=min(16, N))
    if store == "mx":
        inp = wl.mx_attention_inputs(cfg, seed=N)
        # scales that differ from block to block: a misplaced one is a gross error
        inp["Vs"] = (inp["Vs"].astype(np.int32) + np.random.default_rng(N).integers(-3, 2, inp["Vs"].shape)).astype(np.uint8)
        O = dd.dd_bidir_attention_mx(*(to_dev(inp[k]) for k in ("Q", "Qs", "K", "Ks", "V", "Vs")))
        ref = oracle.bidir_attention_mx(inp["Q"], inp["Qs"], inp["K"], inp["Ks"], inp["V"], inp["Vs"])
    else:
        inp = wl.attention_inputs(cfg, seed=N)
        O = dd.dd_bidir_attention_fp8v(*(to_dev(inp[k]) for k in ("Q", "K", "V", "q_scale", "k_scale", "v_scale")))
        ref = oracle.bidir_attention(inp["Q"], inp["K"], inp["V"], FP8, FP8, inp["q_scale"], inp["k_scale"], v_scale=inp["v_scale"])
    torch.cuda.synchronize()
    assert_attention_close(out_to_f64(O, wl.BF16), ref, FP8, f"{store} bidir {B}x{H}/{Hkv}x{N} grid {grid}")


# (B, H, Hkv, N, block_len, block_start, rows per workgroup): key-stream parts that are empty, whole tiles, ragged
BLOCKS = [(1, 8, 2, 64, 64, 0, "128"), (2, 4, 2, 333, 64, 101, "128"), (1, 8, 2, 1000, 64, 936, "256"), (1, 6, 1, 517, 80, 0, "256"),
          (1, 4, 2, 4097, 64, 2000, "128"), (2, 12, 3, 2048, 96, 1536, "256")]


@pytest.mark.parametrize("B,H,Hkv,N,bl,bs,rows", BLOCKS)
def test_block_decoded_v(monkeypatch, B, H, Hkv, N, bl, bs, rows):
    import torch
    monkeypatch.setenv("DD_TUNE_BLOCK_WIDE_ROWS", rows)
    cfg = wl.custom_config(B=B, H=H, Hkv=Hkv, N=N, d=128, qk_dtype=FP8, v_dtype=FP8, bl=bl, prompt=0, G=N)
    cache = wl.cache_inputs(cfg, seed=bs + N)
    blk = wl.block_inputs(cfg, bs, 0, k_scale=cache["k_scale"], v_scale=cache["v_scale"])
    for fresh in (True, False):
        Kb, Vb = (blk["Kblk"], blk["Vblk"]) if fresh else (None, None)
        O = dd.dd_block_attention_cached_fp8v(to_dev(blk["Qblk"]), to_dev(cache["Kc"]), to_dev(cache["Vc"]), bs,
                                              to_dev(blk["q_scale"]), to_dev(cache["k_scale"]), to_dev(cache["v_scale"]),
                                              Kblk=to_dev(Kb), Vblk=to_dev(Vb))
        torch.cuda.synchronize()
        ref = oracle.block_attention_cached(blk["Qblk"], cache["Kc"], cache["Vc"], bs, FP8, FP8, Kb, Vb, blk["q_scale"],
                                            cache["k_scale"], v_scale=cache["v_scale"])
        assert_attention_close(out_to_f64(O, wl.BF16), ref, FP8, f"fp8-V block {B}x{H}/{Hkv} N{N} bl{bl}@{bs} fresh={fresh}")


# verifier calls on 128-row tiles (one per workgroup): (B, H, Hkv, N, d) - one key tile, overlapping last tiles, rows of
# a kv head that end inside a wave / inside a workgroup, and 1025 keys (17 tiles: a stand-in)
NARROW = [(1, 2, 2, 64, 128), (1, 2, 1, 65, 64), (2, 3, 1, 127, 128), (1, 4, 4, 129, 64), (1, 5, 1, 191, 128), (2, 2, 2, 320, 128),
          (1, 2, 1, 1025, 128), (1, 2, 1, 1025, 64)]


@pytest.mark.parametrize("B,H,Hkv,N,d", NARROW)
@pytest.mark.parametrize("qk", [wl.BF16, FP8])
def test_bidir_128_row_tiles(monkeypatch, qk, B, H, Hkv, N, d):
    import torch
    if qk == FP8 and d == 64:
        pytest.skip("fp8 with 64 head dims has no wide form")
    monkeypatch.setenv("DD_TUNE_ATTN_WIDE", "2")
    cfg = wl.custom_config(B=B, H=H, Hkv=Hkv, N=N, d=d, qk_dtype=qk, v_dtype=wl.BF16, prompt=0, G=N, bl=min(16, N))
    inp = wl.attention_inputs(cfg, seed=N + d)
    O = dd.dd_bidir_attention(to_dev(inp["Q"]), to_dev(inp["K"]), to_dev(inp["V"]), q_scale=to_dev(inp["q_scale"]),
                              k_scale=to_dev(inp["k_scale"]), qk_dtype=qk, v_dtype=wl.BF16)
    torch.cuda.synchronize()
    ref = oracle.bidir_attention(inp["Q"], inp["K"], inp["V"], qk, wl.BF16, inp["q_scale"], inp["k_scale"])
    assert_attention_close(out_to_f64(O, wl.BF16), ref, qk, f"128-row tiles {B}x{H}/{Hkv}x{N}x{d}")


# Verifier calls of 1024 keys or more on few row tiles: Q is multiplied as stored.  What a result then loses is two
# roundings to bf16, the weights' and its own.  One has a relative error uniform in +-2^-8 / m for a mantissa m in [1, 2),
# whose rms over log-uniform m is 2^-8 sqrt(1/3) sqrt(3 / (8 ln 2)) = 1.66e-3; two of them 2.35e-3.  (Q rounded once more
# with the softmax scale in it: 2.86e-3 already for N(0, 1) inputs, and growing with the scores.)
TWO_ROUNDINGS = 2.0 ** 0.5 * 2.0 ** -8 * (1 / 3) ** 0.5 * (3 / (8 * np.log(2))) ** 0.5


@pytest.mark.parametrize("B,H,Hkv,N,d", [(1, 4, 4, 1024, 128), (1, 16, 16, 2048, 64), (1, 28, 4, 1100, 128), (1, 32, 32, 1100, 128)])
@pytest.mark.parametrize("sharp", [1, 4])
def test_bidir_q_is_rounded_once(sharp, B, H, Hkv, N, d):
    import torch
    rng = np.random.default_rng(N + d + sharp)
    Q, K, V = (wl.f32_to_bf16_bits(s * rng.standard_normal((B, h, N, d), dtype=np.float32)) for s, h in ((sharp, H), (1, Hkv), (1, Hkv)))
    O = out_to_f64(dd.dd_bidir_attention(to_dev(Q), to_dev(K), to_dev(V)), wl.BF16)
    torch.cuda.synchronize()
    rows = np.stack([np.zeros(512, int), rng.integers(0, H, 512), rng.integers(0, N, 512)], 1)
    ref = oracle.bidir_attention(Q, K, V, wl.BF16, wl.BF16, rows=rows)
    got = O[rows[:, 0], rows[:, 1], rows[:, 2]]
    # (32768 sampled values or more: the 2-norm of their errors scatters by well under 2 %)
    assert np.linalg.norm(got - ref) <= 1.05 * TWO_ROUNDINGS * np.linalg.norm(ref)


def _poison(t, rows):
    """NaN in the given cache rows: the e4m3 code, or the bf16 bit pattern"""
    t = t.clone()
    t[:, :, rows] = 0x7F if t.element_size() == 1 else 0x7FC0
    return t


# (B, H, Hkv, N, block_len, block_start, rows per workgroup): the block at either end, inside the first tile, across tiles
@pytest.mark.parametrize("B,H,Hkv,N,bl,bs,rows", [(1, 8, 2, 515, 64, 5, "128"), (1, 8, 2, 515, 64, 451, "256"), (1, 4, 2, 333, 70, 0, "128"),
                                                  (2, 4, 1, 700, 80, 200, "256"), (1, 2, 2, 1237, 100, 1130, "128")])
@pytest.mark.parametrize("store", ["bf16", "fp8", "fp8v"])
def test_rows_under_the_block_are_not_looked_at(monkeypatch, store, B, H, Hkv, N, bl, bs, rows):
    # cache rows that fresh block rows stand in for - and, for a window, rows outside it - may hold anything, NaN included:
    # the tiles of 64 rows that are loaded reach into them, the result may not
    import torch
    monkeypatch.setenv("DD_TUNE_BLOCK_WIDE_ROWS", rows)
    qk, v = (wl.BF16, wl.BF16) if store == "bf16" else (FP8, FP8 if store == "fp8v" else wl.BF16)
    cfg = wl.custom_config(B=B, H=H, Hkv=Hkv, N=N, d=128, qk_dtype=qk, v_dtype=v, bl=bl, prompt=0, G=N)
    cache = wl.cache_inputs(cfg, seed=bs + N)
    blk = wl.block_inputs(cfg, bs, 0, k_scale=cache["k_scale"], v_scale=cache.get("v_scale"))
    Q, Kb, Vb, K, V = (to_dev(x) for x in (blk["Qblk"], blk["Kblk"], blk["Vblk"], cache["Kc"], cache["Vc"]))
    stale = slice(bs, bs + bl)
    K2, V2 = _poison(K, stale), _poison(V, stale)
    qs, ks = to_dev(blk["q_scale"]), to_dev(cache["k_scale"])
    if store == "fp8v":
        vs = to_dev(cache["v_scale"])
        calls = [(lambda k, v: dd.dd_block_attention_cached_fp8v(Q, k, v, bs, qs, ks, vs, Kblk=Kb, Vblk=Vb), K2, V2)]
    else:
        kw = {"q_scale": qs, "k_scale": ks, "qk_dtype": qk, "v_dtype": v}
        w0 = max(0, bs - 3)
        wn = min(N - w0, bl + 70)
        starts = torch.full((B,), bs, dtype=torch.int32, device="cuda:0")
        Kw, Vw = (_poison(_poison(t, slice(0, w0)), slice(w0 + wn, N)) for t in (K2, V2))
        calls = [(lambda k, v: dd.dd_block_attention_cached(Q, k, v, bs, Kblk=Kb, Vblk=Vb, **kw), K2, V2),
                 (lambda k, v: dd.dd_block_attention_batched(Q, k, v, starts, Kb, Vb, **kw), K2, V2),
                 (lambda k, v: dd.dd_block_attention_refresh(Q, k.clone(), v.clone(), bs, Kb, Vb, **kw), K2, V2),
                 (lambda k, v: dd.dd_block_attention_window(Q, k, v, bs, w0, wn, Kblk=Kb, Vblk=Vb, **kw), Kw, Vw)]
    for i, (call, k, v) in enumerate(calls):
        clean, poisoned = call(K, V), call(k, v)
        torch.cuda.synchronize()
        assert torch.equal(clean.view(torch.int16), poisoned.view(torch.int16)), f"{store} call {i}: {B}x{H}/{Hkv} N{N} bl{bl}@{bs}"


# (odd and even tile counts, a last tile that repeats rows, the folded-scale form)
@pytest.mark.parametrize("B,H,Hkv,N,d", [(1, 2, 2, 65, 128), (1, 2, 1, 128, 64), (1, 3, 1, 191, 128), (1, 2, 2, 515, 128), (1, 2, 1, 1100, 128)])
@pytest.mark.parametrize("qk", [wl.BF16, FP8])
@pytest.mark.parametrize("tile", ["1", "2"])
def test_bidir_infinite_value(monkeypatch, tile, qk, B, H, Hkv, N, d):
    # one infinite value: infinite in its dimension for every query (all weights are positive here), the same bits elsewhere
    import torch
    if qk == FP8 and d == 64:
        pytest.skip("fp8 with 64 head dims has no wide form")
    monkeypatch.setenv("DD_TUNE_ATTN_WIDE", tile)
    cfg = wl.custom_config(B=B, H=H, Hkv=Hkv, N=N, d=d, qk_dtype=qk, v_dtype=wl.BF16, prompt=0, G=N, bl=min(16, N))
    inp = wl.attention_inputs(cfg, seed=N + d)
    Q, K, V = (to_dev(inp[k]) for k in "QKV")
    kw = {"q_scale": to_dev(inp["q_scale"]), "k_scale": to_dev(inp["k_scale"]), "qk_dtype": qk, "v_dtype": wl.BF16}
    want = dd.dd_bidir_attention(Q, K, V, **kw).clone()
    want[..., 5] = 0x7F80
    for row in (0, 3, max(0, N - 70), N - 20, N - 1):
        V2 = V.clone()
        V2[:, :, row, 5] = 0x7F80
        got = dd.dd_bidir_attention(Q, K, V2, **kw)
        torch.cuda.synchronize()
        assert torch.equal(got, want), f"tile {tile}, {B}x{H}/{Hkv}x{N}x{d}, row {row}"


@pytest.mark.parametrize("call", ["cached", "window"])
def test_whole_sequence_block_without_fresh_rows(monkeypatch, call):
    # a block as long as its cache (or window) takes the verifier's path; with no block rows given, every row is the cache's
    import torch
    monkeypatch.setenv("DD_TUNE_ATTN_WIDE", "2")
    N = 64
    cfg = wl.custom_config(B=1, H=2, Hkv=2, N=N, d=128, qk_dtype=wl.BF16, v_dtype=wl.BF16, prompt=0, G=N, bl=N)
    inp = wl.attention_inputs(cfg, seed=N)
    Q, K, V = (to_dev(inp[k]) for k in "QKV")
    if call == "cached":
        O = dd.dd_block_attention_cached(Q, K, V, 0)
    else:
        pad = torch.zeros_like(K[:, :, :5])
        O = dd.dd_block_attention_window(Q, torch.cat([pad, K], 2), torch.cat([pad, V], 2), 5, 5, N)
    torch.cuda.synchronize()
    ref = oracle.bidir_attention(inp["Q"], inp["K"], inp["V"], wl.BF16, wl.BF16)
    assert_attention_close(out_to_f64(O, wl.BF16), ref, wl.BF16, call)


# (the verifier's form; the drafter's with one and with several key splits)
@pytest.mark.parametrize("B,H,Hkv,N,bl,rows", [(1, 2, 2, 191, 0, None), (1, 8, 2, 1025, 0, None), (1, 8, 2, 333, 32, "128"), (1, 4, 1, 1000, 64, "128")])
@pytest.mark.parametrize("store", ["bf16", "fp8", "fp8v"])
def test_nan_query_stays_in_its_row(monkeypatch, store, B, H, Hkv, N, bl, rows):
    # on 128-row tiles: a NaN in a query row makes that row of the output NaN and changes no other
    import torch
    monkeypatch.setenv("DD_TUNE_ATTN_WIDE", "2")
    if rows:
        monkeypatch.setenv("DD_TUNE_BLOCK_WIDE_ROWS", rows)
    qk, v = (wl.BF16, wl.BF16) if store == "bf16" else (FP8, FP8 if store == "fp8v" else wl.BF16)
    cfg = wl.custom_config(B=B, H=H, Hkv=Hkv, N=N, d=128, qk_dtype=qk, v_dtype=v, bl=bl or 16, prompt=0, G=N)
    inp = wl.attention_inputs(cfg, seed=N)
    Q, K, V = (to_dev(inp[k]) for k in "QKV")
    if bl:
        Q = Q[:, :, :bl].contiguous()
    qs, ks = to_dev(inp["q_scale"]), to_dev(inp["k_scale"])

    def call(q):
        if store == "fp8v":
            vs = to_dev(inp["v_scale"])
            return dd.dd_block_attention_cached_fp8v(q, K, V, 3, qs, ks, vs) if bl else dd.dd_bidir_attention_fp8v(q, K, V, qs, ks, vs)
        kw = {"q_scale": qs, "k_scale": ks, "qk_dtype": qk, "v_dtype": v}
        return dd.dd_block_attention_cached(q, K, V, 3, **kw) if bl else dd.dd_bidir_attention(q, K, V, **kw)
    want = call(Q)
    q2 = Q.clone()
    q2[0, 1, 5] = 0x7F if qk == FP8 else 0x7FC0
    got = call(q2)
    torch.cuda.synchronize()
    assert torch.isnan(got[0, 1, 5].view(torch.bfloat16)).all()
    got[0, 1, 5] = want[0, 1, 5]
    assert torch.equal(got, want), f"{store} {B}x{H}/{Hkv} N{N} bl{bl}"


def test_nan_query_stays_in_its_row_tile(monkeypatch):
    # folded-scale form, one workgroup for all row tiles (256 rows each): the softmax reference of a NaN row ends with its tile
    import torch
    monkeypatch.setenv("DD_TUNE_ATTN_WIDE", "1")
    monkeypatch.setenv("DD_TUNE_ATTN_WIDE_GRID", "1")
    cfg = wl.custom_config(B=2, H=2, Hkv=1, N=1100, d=128, qk_dtype=wl.BF16, v_dtype=wl.BF16, prompt=0, G=1100)
    inp = wl.attention_inputs(cfg, seed=3)
    Q, K, V = (to_dev(inp[k]) for k in "QKV")
    want = dd.dd_bidir_attention(Q, K, V)
    q2 = Q.clone()
    q2[0, 0, 5] = 0x7FC0
    got = dd.dd_bidir_attention(q2, K, V)
    torch.cuda.synchronize()
    assert torch.isnan(got[0, 0, 5].view(torch.bfloat16)).all()
    got[0, 0, :256] = want[0, 0, :256]
    got, want = got.view(torch.bfloat16).double(), want.view(torch.bfloat16).double()
    # (the others' references may be raised beside it, which rounds their weights elsewhere: a step or two of an output)
    assert ((got - want).abs() <= 2.0 ** -6 * want.abs() + 2.0 ** -8 * want.abs().max()).all()
