"""Which kernel, form and key splits the library's rules pick, told by the bits of the result: a call by rule gives those of the same call
forced there by hook, and not those of the route that its neighbours across a line of the rule take."""
import pytest

import paper_2604_05250_amd as dd
from paper_2604_05250_amd import workloads as wl
from _kernels import solo_form
from _util import to_dev

pytestmark = pytest.mark.gpu
BF16, FP8 = wl.BF16, wl.FP8_E4M3
ELSEWHERE = {"DD_TUNE_SOLO": "0"}
HOOKS = ("DD_TUNE_SOLO", "DD_TUNE_SOLO_FORM", "DD_TUNE_BLOCK_SPLITS")
# (q and k, v, head dims), (B, H, Hkv, N, block_len, fresh), the rule's route, another one
DRAFTS = [
    # long streams of few workgroups: in key splits, not eight waves with every one of them (from the cache alone that is faster)
    ((FP8, BF16, 128), (4, 32, 8, 3643, 16, True), solo_form(128, 2), solo_form(148)),
    ((BF16, BF16, 128), (4, 32, 8, 2250, 16, True), solo_form(114, 4), solo_form(148)),
    ((FP8, FP8, 128), (3, 16, 16, 3773, 32, True), solo_form(114, 5), solo_form(148)),
    ((FP8, FP8, 128), (6, 32, 32, 1598, 32, True), solo_form(114), solo_form(124)),
    ((FP8, BF16, 128), (1, 32, 32, 1024, 32, True), solo_form(148), solo_form(114, 4)),       # (a short one stays)
    # e4m3 V, more than 64 rows, 257 to 512 workgroups: at 64 keys and fewer too ...
    ((FP8, FP8, 128), (6, 32, 8, 64, 64, True), solo_form(114), ELSEWHERE),
    ((FP8, FP8, 128), (12, 28, 4, 40, 24, True), solo_form(114), ELSEWHERE),
    ((FP8, FP8, 128), (12, 32, 8, 25, 18, True), solo_form(114), ELSEWHERE),
    ((FP8, FP8, 128), (12, 32, 8, 24, 18, True), ELSEWHERE, solo_form(114)),
    # ... but not long streams that the wide kernel can serve
    ((FP8, FP8, 128), (10, 40, 8, 2600, 16, False), solo_form(114), ELSEWHERE),
    ((FP8, FP8, 128), (10, 40, 8, 2601, 16, False), ELSEWHERE, solo_form(114)),
    ((FP8, FP8, 128), (10, 40, 8, 2601, 16, True), solo_form(114), ELSEWHERE),                # its own rows: shorter than a tile there
    ((FP8, FP8, 128), (5, 32, 8, 2600, 64, True), solo_form(224), ELSEWHERE),
    ((FP8, FP8, 128), (5, 32, 8, 2601, 64, True), ELSEWHERE, solo_form(224)),
    ((FP8, FP8, 128), (11, 16, 4, 3328, 64, True), solo_form(224), ELSEWHERE),
    ((FP8, FP8, 128), (11, 16, 4, 3329, 64, True), ELSEWHERE, solo_form(224)),
    ((FP8, FP8, 128), (11, 32, 4, 3329, 32, True), solo_form(224), ELSEWHERE),
    ((FP8, FP8, 128), (4, 32, 8, 3500, 96, True), solo_form(224), ELSEWHERE),                 # 384 rows: a tile is half empty
    ((FP8, FP8, 128), (8, 32, 8, 3328, 64, True), solo_form(224), ELSEWHERE),
    ((FP8, FP8, 128), (8, 32, 8, 3329, 64, True), ELSEWHERE, solo_form(224)),
    ((FP8, FP8, 128), (9, 32, 8, 2200, 28, False), solo_form(224), ELSEWHERE),                # 128-row tiles nearly full
    ((FP8, FP8, 128), (9, 32, 8, 2201, 28, False), ELSEWHERE, solo_form(224)),
    # more than 64 rows: bf16 past 95 MB (two workgroups per compute unit), fp8 likewise (one, four waves)
    ((BF16, BF16, 128), (21, 32, 8, 1104, 24, True), solo_form(114), ELSEWHERE),
    ((BF16, BF16, 128), (21, 32, 8, 1105, 24, True), ELSEWHERE, solo_form(114)),
    ((FP8, BF16, 128), (10, 32, 8, 3092, 24, True), solo_form(114), ELSEWHERE),
    ((FP8, BF16, 128), (10, 32, 8, 3093, 24, True), ELSEWHERE, solo_form(114)),
    # 33 to 64 rows, 64 keys and fewer: here, but where keys of both kinds meet in a unit that is not full
    ((BF16, BF16, 128), (15, 32, 8, 48, 16, False), solo_form(124), ELSEWHERE),
    ((BF16, BF16, 128), (15, 32, 8, 48, 14, True), solo_form(124), ELSEWHERE),
    ((BF16, BF16, 128), (15, 32, 8, 48, 13, True), ELSEWHERE, solo_form(124)),
    ((BF16, BF16, 128), (15, 32, 8, 15, 15, True), ELSEWHERE, solo_form(124)),                # the block's keys alone
    ((FP8, BF16, 128), (15, 32, 8, 15, 15, True), solo_form(124), ELSEWHERE),
    ((BF16, BF16, 128), (15, 32, 8, 64, 13, True), solo_form(124), ELSEWHERE),
    ((FP8, BF16, 128), (15, 32, 8, 64, 16, True), solo_form(124), ELSEWHERE),
    ((FP8, BF16, 128), (15, 32, 8, 48, 16, True), ELSEWHERE, solo_form(124)),
    # fp8, one workgroup of rows per head, two to a compute unit: streamed past 100 MB
    ((FP8, BF16, 128), (9, 32, 32, 904, 32, True), solo_form(114), ELSEWHERE),
    ((FP8, BF16, 128), (9, 32, 32, 905, 32, True), ELSEWHERE, solo_form(114)),
    # a block that is the whole sequence
    ((BF16, BF16, 128), (5, 16, 16, 24, 24, True), ELSEWHERE, solo_form(124)),
    ((BF16, BF16, 128), (5, 16, 16, 24, 24, False), solo_form(124), ELSEWHERE),
    ((BF16, BF16, 128), (5, 16, 16, 25, 24, True), solo_form(124), ELSEWHERE),
]


def by(monkeypatch, env, call):
    import torch
    for k in HOOKS:
        monkeypatch.delenv(k, raising=False)
    for k, v in env.items():
        monkeypatch.setenv(k, v)
    O = call()
    torch.cuda.synchronize()
    return O


@pytest.mark.parametrize("store,shape,here,there", DRAFTS)
def test_drafter_routes(monkeypatch, store, shape, here, there):
    import torch
    (qk, v, d), (B, H, Hkv, N, bl, fresh) = store, shape
    g = torch.Generator(device="cuda:0").manual_seed(N)
    normal = lambda *s: torch.randn(s, generator=g, device="cuda:0")
    of = lambda x, t: (x * 90).clamp(-448, 448).to(torch.float8_e4m3fn) if t == FP8 else x.bfloat16()
    Q, K, V = of(normal(B, H, bl, d), qk), of(normal(B, Hkv, N, d), qk), of(normal(B, Hkv, N, d), v)
    Kb, Vb = (of(normal(B, Hkv, bl, d), qk), of(normal(B, Hkv, bl, d), v)) if fresh else (None, None)
    scale = lambda heads: torch.full((B, heads), 1 / 90, device="cuda:0")
    s = {"q_scale": scale(H), "k_scale": scale(Hkv)} if qk == FP8 else {}

    def call():
        if v == FP8:
            return dd.dd_block_attention_cached_fp8v(Q, K, V, 0, scale(H), scale(Hkv), scale(Hkv), Kblk=Kb, Vblk=Vb)
        return dd.dd_block_attention_cached(Q, K, V, 0, Kblk=Kb, Vblk=Vb, **s)
    got, want, other = by(monkeypatch, {}, call), by(monkeypatch, here, call), by(monkeypatch, there, call)
    assert not torch.equal(want, other), "the bits do not tell the two routes apart"
    assert torch.equal(got, want)


@pytest.mark.parametrize("qk,v,d,H,Hkv,N,here", [
    (FP8, BF16, 128, 128, 128, 12, True), (FP8, BF16, 128, 129, 129, 12, False), (FP8, BF16, 128, 129, 129, 31, False), (FP8, BF16, 128, 129, 129, 32, True),
    (FP8, FP8, 128, 129, 129, 31, False), (FP8, BF16, 128, 80, 80, 40, True),
    (BF16, BF16, 64, 129, 129, 31, False), (BF16, BF16, 64, 80, 80, 40, False), (BF16, BF16, 128, 129, 129, 12, True),
    (FP8, BF16, 128, 325, 65, 9, False), (FP8, BF16, 128, 390, 65, 8, True)])                 # 45 and 48 rows per kv head, 130 workgroups
def test_verifier_routes_of_few_keys(monkeypatch, qk, v, d, H, Hkv, N, here):
    import torch
    cfg = wl.custom_config(B=1, H=H, Hkv=Hkv, N=N, d=d, qk_dtype=qk, v_dtype=v, prompt=0, G=N, bl=N)
    inp = wl.attention_inputs(cfg, seed=N + d)
    Q, K, V, qs, ks, vs = (to_dev(inp.get(k)) if inp.get(k) is not None else None for k in ("Q", "K", "V", "q_scale", "k_scale", "v_scale"))
    call = lambda: dd.dd_bidir_attention_fp8v(Q, K, V, qs, ks, vs) if v == FP8 else dd.dd_bidir_attention(Q, K, V, q_scale=qs, k_scale=ks, qk_dtype=qk, v_dtype=v)
    got, solo, other = by(monkeypatch, {}, call), by(monkeypatch, {"DD_TUNE_SOLO": "1"}, call), by(monkeypatch, ELSEWHERE, call)
    assert not torch.equal(solo, other), "the bits do not tell the two routes apart"
    assert torch.equal(got, solo if here else other)
