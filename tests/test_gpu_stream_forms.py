"""The streaming attention kernel's forms (bf16 with 64 and 128 head dims, fp8 Q/K) against the CPU oracle."""
import pytest

import oracle
import paper_2604_05250_amd as dd
from paper_2604_05250_amd import workloads as wl
from _util import assert_attention_close, out_to_f64, to_dev

pytestmark = pytest.mark.gpu
FORMS = [(wl.BF16, 64), (wl.BF16, 128), (wl.FP8_E4M3, 128)]


def check_block(B, H, Hkv, N, d, qk, bl, bs, what):
    import torch
    cfg = wl.custom_config(B=B, H=H, Hkv=Hkv, N=N, d=d, qk_dtype=qk, v_dtype=wl.BF16, bl=bl, prompt=0, G=N)
    cache = wl.cache_inputs(cfg, seed=bs + N)
    blk = wl.block_inputs(cfg, bs, 0, k_scale=cache["k_scale"])
    O = dd.dd_block_attention_cached(to_dev(blk["Qblk"]), to_dev(cache["Kc"]), to_dev(cache["Vc"]), bs, Kblk=to_dev(blk["Kblk"]),
                                     Vblk=to_dev(blk["Vblk"]), q_scale=to_dev(blk["q_scale"]), k_scale=to_dev(cache["k_scale"]),
                                     qk_dtype=qk, v_dtype=wl.BF16)
    torch.cuda.synchronize()
    ref = oracle.block_attention_cached(blk["Qblk"], cache["Kc"], cache["Vc"], bs, qk, wl.BF16, blk["Kblk"], blk["Vblk"],
                                        blk["q_scale"], cache["k_scale"])
    assert_attention_close(out_to_f64(O, wl.BF16), ref, qk, f"{what}: {B}x{H}/{Hkv} N{N} d{d} bl{bl}@{bs}")


# one tile: the ring's other slots hold stand-ins that nobody reads, and then the key phases' states.  Many workgroups, one
# and two row blocks, one key phase without keys (32 keys)
@pytest.mark.parametrize("N,bl", [(64, 60), (33, 17), (32, 31), (63, 8)])
@pytest.mark.parametrize("qk,d", FORMS)
def test_one_tile(monkeypatch, qk, d, N, bl):
    monkeypatch.setenv("DD_TUNE_BLOCK_STREAM", "1")
    check_block(16, 32, 32, N, d, qk, bl, N - bl, "one tile")


# tiles loaded with and without the non-temporal hint: less than a tile, the ring's depth and more, key splits, GQA
@pytest.mark.parametrize("B,H,Hkv,N,bl,bs", [(2, 4, 2, 33, 16, 5), (1, 4, 4, 193, 33, 100), (1, 8, 2, 1237, 16, 900)])
@pytest.mark.parametrize("qk,d", FORMS)
@pytest.mark.parametrize("hint", ["0", "1"])
def test_non_temporal_loads(monkeypatch, hint, qk, d, B, H, Hkv, N, bl, bs):
    monkeypatch.setenv("DD_TUNE_STREAM_NT", hint)
    check_block(B, H, Hkv, N, d, qk, bl, bs, f"hint {hint}")
