"""What the Python binding refuses before a launch: tensors that hold fewer bytes than their shapes and dtype tags say would
be read or written.  The checks come before the one for GPU memory, so CPU tensors reach them."""
import pytest
import torch

import paper_2604_05250_amd as dd

B, H, Hkv, N, d, bl = 2, 4, 2, 64, 64, 16
bf, f32, u8 = torch.bfloat16, torch.float32, torch.uint8


def z(*shape, t=bf):
    return torch.zeros(shape, dtype=t)


def bidir(q=bf, k=bf, v=bf, O=None, qs=None, ks=None, **kw):
    return dd.dd_bidir_attention(z(B, H, N, d, t=q), z(B, Hkv, N, d, t=k), z(B, Hkv, N, d, t=v), O=O, q_scale=qs, k_scale=ks, **kw)


def block(q=bf, k=bf, v=bf, kb=bf, vb=bf, O=None, qs=None, ks=None, call="cached", **kw):
    Q, K, V, Kb, Vb = z(B, H, bl, d, t=q), z(B, Hkv, N, d, t=k), z(B, Hkv, N, d, t=v), z(B, Hkv, bl, d, t=kb), z(B, Hkv, bl, d, t=vb)
    kw.update(O=O, q_scale=qs, k_scale=ks)
    if call == "cached":
        return dd.dd_block_attention_cached(Q, K, V, 3, Kblk=Kb, Vblk=Vb, **kw)
    if call == "refresh":
        return dd.dd_block_attention_refresh(Q, K, V, 3, Kb, Vb, **kw)
    if call == "window":
        return dd.dd_block_attention_window(Q, K, V, 3, 0, 40, Kblk=Kb, Vblk=Vb, **kw)
    return dd.dd_block_attention_batched(Q, K, V, z(B, t=torch.int32), Kb, Vb, **kw)


def fp8v(kb=u8, vb=u8, O=None, qs=B * H, ks=B * Hkv, vs=B * Hkv, t=f32, block=True):
    sc = [z(n, t=t) for n in (qs, ks, vs)]
    K = z(B, Hkv, N, d, t=u8)
    if not block:
        return dd.dd_bidir_attention_fp8v(z(B, H, N, d, t=u8), K, K, *sc, O=O)
    return dd.dd_block_attention_cached_fp8v(z(B, H, bl, d, t=u8), K, K, 3, *sc, O=O, Kblk=z(B, Hkv, bl, d, t=kb), Vblk=z(B, Hkv, bl, d, t=vb))


def verify(d_=bf, v=bf, mode=dd.KL_THRESH, **kw):
    return dd.dd_verify_remask(z(16, 64, t=d_), z(16, 64, t=v), z(16, t=u8), mode, 0.5, 0, 2, 8, **kw)


MX = (z(B, H, N, d, t=u8), z(B, H, N, 2, t=u8), z(B, Hkv, N, d, t=u8), z(B, Hkv, N, 2, t=u8), z(B, Hkv, N, d // 2, t=u8), z(B, Hkv, N, 2, t=u8))

REFUSED = [
    # elements narrower (or wider) than the tag of the operand's group
    (TypeError, "K", lambda: bidir(k=u8)), (TypeError, "K", lambda: bidir(q=u8, k=bf)), (TypeError, "Q", lambda: bidir(qk_dtype=dd.F32)),
    (TypeError, "V", lambda: bidir(v=u8, v_dtype=dd.BF16)), (TypeError, "K", lambda: bidir(q=f32, k=bf, v=f32)),
    (TypeError, "Kc", lambda: block(k=u8)), (TypeError, "Kblk", lambda: block(kb=u8)), (TypeError, "Vblk", lambda: block(vb=u8, call="refresh")),
    (TypeError, "Kblk", lambda: block(kb=u8, call="batched")), (TypeError, "Vc", lambda: block(v=u8, v_dtype=dd.BF16, call="window")),
    (TypeError, "Kblk", lambda: fp8v(kb=bf)), (TypeError, "Vblk", lambda: fp8v(vb=bf)),
    (TypeError, "Krows", lambda: dd.dd_cache_insert_rows(z(B, Hkv, N, d), z(B, Hkv, N, d), z(B, Hkv, 1, d, t=u8), z(B, Hkv, 1, d), z(B, t=torch.int32))),
    (TypeError, "Vrows", lambda: dd.dd_cache_insert_rows(z(B, Hkv, N, d), z(B, Hkv, N, d), z(B, Hkv, 1, d), z(B, Hkv, 1, d, t=u8), z(B, t=torch.int32))),
    (TypeError, "logits_d", lambda: verify(v=f32)), (TypeError, "logits_v", lambda: verify(logit_dtype=dd.F32)),
    (TypeError, "logits_d", lambda: dd.dd_unmask(z(16, 64), z(16, t=u8), dd.UNMASK_THRESH, 0.5, 2, 8, logit_dtype=dd.F32)),
    (TypeError, "logits_d", lambda: dd.dd_verify_scores(z(16, 64), z(16, 64, t=f32), logit_dtype=dd.F32)),
    # outputs
    (ValueError, "O", lambda: bidir(O=z(B, H, N, d - 1))), (ValueError, "O", lambda: bidir(O=z(B, H, N, d, t=u8))),
    (ValueError, "O", lambda: bidir(q=f32, k=f32, v=f32, O=z(B, H, N, d))), (ValueError, "O", lambda: block(O=z(B, H, bl - 1, d))),
    (ValueError, "O", lambda: fp8v(O=z(B, H, bl, d, t=u8))), (ValueError, "O", lambda: fp8v(O=z(B, H, N, d, t=u8), block=False)),
    (ValueError, "O", lambda: dd.dd_bidir_attention_mx(*MX, O=z(B, H, N, d, t=u8))),
    # scales
    (TypeError, "q_scale", lambda: bidir(qs=z(B * H))), (ValueError, "q_scale", lambda: bidir(qs=z(B * H - 1, t=f32))),
    (ValueError, "k_scale", lambda: block(ks=z(B * Hkv - 1, t=f32))), (ValueError, "v_scale", lambda: fp8v(vs=1)),
    (TypeError, "q_scale", lambda: fp8v(t=bf)), (ValueError, "k_scale", lambda: fp8v(ks=1, block=False)),
]


@pytest.mark.parametrize("error,what,call", REFUSED, ids=[str(i) for i in range(len(REFUSED))])
def test_refused(error, what, call):
    with pytest.raises(error, match=f"^{what}: (elements|too small|float32|one byte)"):
        call()


@pytest.mark.parametrize("call", [lambda: bidir(O=z(B, H, N, d)), lambda: bidir(O=z(B * H * N * d + 8, t=torch.int16), qs=z(B * H + 1, t=f32)),
                                  lambda: block(qs=z(B, H, t=f32), ks=z(B, Hkv, t=f32)), lambda: fp8v(O=z(B, H, bl, d)),
                                  lambda: verify(d_=f32, mode=dd.CONF_THRESH), lambda: verify(),
                                  lambda: bidir(q=torch.int16, k=torch.uint16, v=bf), lambda: dd.dd_bidir_attention_mx(*MX)])
def test_not_refused_for_its_size(call):
    # (an output of another shape with room enough, logits that the rule does not read, another type of the same width)
    with pytest.raises(ValueError, match="must live in GPU memory"):
        call()
