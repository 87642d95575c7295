"""The calls this library is timed on: the three parts of one draft-then-verify cycle, and the whole cycle, over the
range of sizes and storage types that its callers use.

A case is one of four kinds:
  draft   one drafter attention call on the active block (the cached, batched or windowed entry point)
  attn    one verifier attention call over all positions
  verify  one verification call over the vocabulary
  cycle   a whole cycle on one sequence batch: K x (drafter attention + unmasking) on a block, the last drafter call
          with the cache refresh, then the verifier's attention and the verification rule
`store` is the storage of Q/K/V: "f32", "bf16", "fp8" (Q/K e4m3 with per-head scales, V bf16), "fp8v" (V e4m3 as well),
"mx" (block-scaled e4m3 Q/K and e2m1 V).
"""
import math

import torch

import paper_2604_05250_amd as dd

E4M3_MAX = 448.0
E2M1_GRID = (0.0, 0.5, 1.0, 1.5, 2.0, 3.0, 4.0, 6.0)
MODES = {"trust": dd.TRUST, "kl": dd.KL_THRESH, "conf": dd.CONF_THRESH, "klprob": dd.KL_PROB, "conftopk": dd.CONF_TOPK}
THRESHOLD = {"trust": 0.0, "kl": 0.5, "conf": 0.9, "klprob": 0.0, "conftopk": 64.0}


def listed():
    return [
        # the smallest use: a CPU-checkable step in fp32, a few thousand scores per head; launches and latency
        _cycle("cycle_f32_n128", "f32", B=1, H=4, Hkv=4, N=128, d=64, bl=16, steps=4, G=64, V=1024, logits="f32"),
        # interactive decoding of one sequence with the heads and the vocabulary of an 8B model: 18 short calls
        _cycle("cycle_bf16_n512", "bf16", B=1, H=32, Hkv=32, N=512, d=128, bl=32, steps=8, G=256, V=126464, logits="bf16"),
        # the drafter's call of a batch of eight: the cache is read once, little else happens
        _draft("draft_bf16_b8_n1024", "bf16", "cached", B=8, H=32, Hkv=32, N=1024, d=128, bl=64),
        # the drafter's call of a throughput batch with grouped heads and fp8 keys: compute bound
        _draft("draft_fp8_gqa_b16_n2048", "fp8", "cached", B=16, H=32, Hkv=8, N=2048, d=128, bl=64),
        # a serving batch whose sequences stand at different blocks: short blocks, ragged cache, odd batch
        _draft("draft_fp8_serving_b11_n1237", "fp8", "batched", B=11, H=32, Hkv=8, N=1237, d=128, bl=16),
        # the verifier's attention of the batch of eight
        _attn("attn_bf16_b8_n1024", "bf16", B=8, H=32, Hkv=32, N=1024, d=128),
        # one long sequence, a length that is no multiple of any tile
        _attn("attn_bf16_n3333", "bf16", B=1, H=32, Hkv=32, N=3333, d=128),
        # the throughput batch: grouped heads, fp8 queries and keys
        _attn("attn_fp8_gqa_b16_n2048", "fp8", B=16, H=32, Hkv=8, N=2048, d=128),
        # the same with the values stored as e4m3 too
        _attn("attn_fp8v_gqa_b16_n2048", "fp8v", B=16, H=32, Hkv=8, N=2048, d=128),
        # the same on block-scaled operands
        _attn("attn_mx_gqa_b16_n2048", "mx", B=16, H=32, Hkv=8, N=2048, d=128),
        # verification of one long sequence: both logit matrices are read, few rows
        _verify("verify_kl_p512", "kl", B=1, G=512, V=126464, logits="bf16"),
        # verification of the throughput batch: the largest stream of bytes
        _verify("verify_conf_p8192", "conf", B=16, G=512, V=152064, logits="bf16"),
    ]


def draw(rng):
    kind = rng.choice(["attn", "attn", "draft", "draft", "verify", "cycle"])
    if kind == "attn":
        store = rng.choice(["bf16", "bf16", "fp8", "fp8v", "mx"])
        H, Hkv = rng.choice([(32, 32), (32, 8), (28, 4), (16, 16)])
        d = 64 if store == "bf16" and rng.random() < 0.2 else 128
        N = _log_int(rng, 300, 4096)
        B = _log_int(rng, 1, 16)
        while 4.0 * B * H * N * N * d > 1.0e12:              # no more work than the largest listed call
            B = max(1, B // 2)
        return _attn(None, store, B=B, H=H, Hkv=Hkv, N=N, d=d)
    if kind == "draft":
        store = rng.choice(["bf16", "bf16", "fp8", "fp8v"])
        H, Hkv = rng.choice([(32, 32), (32, 8), (28, 4), (16, 16)])
        entry = "cached" if store == "fp8v" else rng.choice(["cached", "batched", "window"])
        N = _log_int(rng, 300, 4096)
        return _draft(None, store, entry, B=_log_int(rng, 1, 16), H=H, Hkv=Hkv, N=N, d=128,
                      bl=rng.choice([8, 16, 24, 32, 48, 64]))
    if kind == "verify":
        mode = rng.choice(sorted(MODES))
        logits = rng.choice(["bf16", "bf16", "bf16", "f32"])
        V = 8 * rng.randrange(32000 // 8, 152064 // 8 + 1)
        return _verify(None, mode, B=_log_int(rng, 1, 16), G=_log_int(rng, 32, 320), V=V, logits=logits)
    if rng.random() < 0.3:
        return _cycle(None, "f32", B=1, H=rng.choice([2, 4, 8]), Hkv=2, N=rng.randrange(96, 257), d=64, bl=16, steps=4,
                      G=64, V=8 * rng.randrange(64, 257), logits="f32")
    H, Hkv = rng.choice([(32, 32), (32, 8), (16, 16)])
    return _cycle(None, "bf16", B=rng.choice([1, 1, 2]), H=H, Hkv=Hkv, N=_log_int(rng, 300, 1400), d=128,
                  bl=rng.choice([16, 32, 64]), steps=rng.choice([4, 8]), G=rng.choice([64, 128, 256]),
                  V=8 * rng.randrange(32000 // 8, 152064 // 8 + 1), logits="bf16")


def prepare(case, seed):
    g = torch.Generator(device="cuda").manual_seed(seed)
    case = dict(case)
    st = {"case": case}
    kind = case["kind"]
    if kind == "verify":
        st.update(_logits(g, case["B"] * case["G"], case["V"], case["logits"], spike=8.0 if case["mode"].startswith("conf") else 0.0))
        # every position of a verified span is decoded (some spans keep masked positions: those rows are not eligible)
        st["mask"] = (torch.rand(case["B"] * case["G"], generator=g, device="cuda") < 0.1).to(torch.uint8)
        return st
    B, H, Hkv, N, d, store = (case[k] for k in ("B", "H", "Hkv", "N", "d", "store"))
    st["KV"] = _kv(g, B, Hkv, N, d, store)
    if kind == "attn":
        st["Q"] = _rows(g, B, H, N, d, store)
        st["O"] = torch.empty((B, H, N, d), dtype=_out_type(store), device="cuda")
        return st
    bl = case["bl"]
    if kind == "draft":
        st["blk"] = _block(g, B, H, Hkv, bl, d, store, st["KV"])
        st["O"] = torch.empty((B, H, bl, d), dtype=_out_type(store), device="cuda")
        if case["entry"] == "batched":
            st["starts"] = torch.randint(0, N - bl + 1, (B,), generator=g, device="cuda", dtype=torch.int32)
        return st
    # cycle: one block of the generated span is drafted over `steps` steps, then the whole span is verified
    G, V = case["G"], case["V"]
    st["blk"] = [_block(g, B, H, Hkv, bl, d, store, st["KV"]) for _ in range(case["steps"])]
    st["draft_logits"] = [_logits(g, B * bl, V, case["logits"], pair=False)["logits_d"] for _ in range(case["steps"])]
    st["mask0"] = torch.ones(B * bl, dtype=torch.uint8, device="cuda")
    st["x"] = torch.zeros(B * bl, dtype=torch.int32, device="cuda")
    st["att"] = {"Q": _rows(g, B, H, N, d, store), "KV": _kv(g, B, Hkv, N, d, store)}
    st.update(_logits(g, B * G, V, case["logits"]))
    st["mask"] = torch.zeros(B * G, dtype=torch.uint8, device="cuda")
    return st


def run(st):
    case = st["case"]
    kind = case["kind"]
    if kind == "attn":
        return _call_attn(case["store"], st["Q"], st["KV"], st["O"])
    if kind == "draft":
        return _call_draft(case, st["blk"], st["KV"], st["O"], st.get("starts"))
    if kind == "verify":
        mode = case["mode"]
        return dd.dd_verify_remask(st["logits_d"], st["logits_v"], st["mask"], MODES[mode], THRESHOLD[mode], 7,
                                   case["B"], case["G"])
    out, mask = [], st["mask0"]
    B, bl, kv = case["B"], case["bl"], st["KV"]
    start = case["N"] - case["G"]
    per_step = -(-bl // case["steps"])
    for k, blk in enumerate(st["blk"]):
        call = dd.dd_block_attention_refresh if k + 1 == len(st["blk"]) else dd.dd_block_attention_cached
        out.append(call(blk["Q"], kv["K"], kv["V"], start, Kblk=blk["K"], Vblk=blk["V"]))
        mask, tokens, conf = dd.dd_unmask(st["draft_logits"][k], mask, dd.UNMASK_TOPK, per_step, B, bl, x_tokens=st["x"])
        out += [mask, tokens, conf]
    out.append(_call_attn(case["store"], st["att"]["Q"], st["att"]["KV"], None))
    out += dd.dd_verify_remask(st["logits_d"], st["logits_v"], st["mask"], dd.KL_THRESH, THRESHOLD["kl"], 7, B, case["G"])
    return out + [st["x"], kv["K"], kv["V"]]


def work(case):
    kind = case["kind"]
    if kind == "verify":
        return {"bytes": _verify_bytes(case["B"] * case["G"], case["V"], case["logits"], case["mode"].startswith("kl")), "flops": 0.0}
    if kind == "attn":
        return _attn_work(case, case["N"])
    if kind == "draft":
        return _draft_work(case)
    K = case["steps"]
    w, a = _draft_work(case), _attn_work(case, case["N"])
    nbytes = K * w["bytes"] + a["bytes"] + K * _verify_bytes(case["B"] * case["bl"], case["V"], case["logits"], False)
    nbytes += _verify_bytes(case["B"] * case["G"], case["V"], case["logits"], True)
    return {"bytes": nbytes, "flops": K * w["flops"] + a["flops"]}


def tolerance(case):
    # Largest errors measured against a float64 evaluation on the same stored inputs (relative 2-norm, largest single
    # difference), each stated about four times over: bf16 outputs 2.3e-3, 1.3e-2 (weights and outputs are both rounded
    # to bf16), fp32 attention 6.6e-7, 4.6e-6, verification scores 3.4e-7, 1.0e-6.  Whole values: a decision may differ
    # where a score ties with its threshold or with another score.
    if case["kind"] != "verify" and case["store"] != "f32":
        return {"rel": 1e-2, "max": 5e-2, "differ": 0.004}
    return {"rel": 3e-6, "max": 2e-5, "differ": 0.004}


# ---------------------------------------------------------------------------------------------------- cases
def _named(name, case):
    return {"name": name, **case} if name else case


def _attn(name, store, **sizes):
    return _named(name, {"kind": "attn", "store": store, **sizes})


def _draft(name, store, entry, **sizes):
    return _named(name, {"kind": "draft", "store": store, "entry": entry, **sizes})


def _verify(name, mode, **sizes):
    return _named(name, {"kind": "verify", "mode": mode, **sizes})


def _cycle(name, store, **sizes):
    return _named(name, {"kind": "cycle", "store": store, **sizes})


def _log_int(rng, lo, hi):
    return min(hi, int(math.exp(rng.uniform(math.log(lo), math.log(hi + 1)))))


# ---------------------------------------------------------------------------------------------------- calls
def _call_attn(store, Q, kv, O):
    if store == "mx":
        return dd.dd_bidir_attention_mx(Q["x"], Q["s"], kv["K"]["x"], kv["K"]["s"], kv["V"]["x"], kv["V"]["s"], O=O)
    if store == "fp8v":
        return dd.dd_bidir_attention_fp8v(Q["x"], kv["K"], kv["V"], Q["s"], kv["ks"], kv["vs"], O=O)
    if store == "fp8":
        return dd.dd_bidir_attention(Q["x"], kv["K"], kv["V"], O=O, q_scale=Q["s"], k_scale=kv["ks"])
    return dd.dd_bidir_attention(Q, kv["K"], kv["V"], O=O)


def _call_draft(case, blk, kv, O, starts):
    N, bl = case["N"], case["bl"]
    start = (N - bl) * 3 // 4                                # well inside the generated span
    if case["store"] == "fp8v":
        return dd.dd_block_attention_cached_fp8v(blk["Q"]["x"], kv["K"], kv["V"], start, blk["Q"]["s"], kv["ks"], kv["vs"],
                                                 O=O, Kblk=blk["K"], Vblk=blk["V"])
    fp8 = case["store"] == "fp8"
    Q = blk["Q"]["x"] if fp8 else blk["Q"]
    scales = {"q_scale": blk["Q"]["s"], "k_scale": kv["ks"]} if fp8 else {}
    if case["entry"] == "batched":
        return dd.dd_block_attention_batched(Q, kv["K"], kv["V"], starts, blk["K"], blk["V"], O=O, **scales)
    if case["entry"] == "window":
        first, length = _window(case)
        return dd.dd_block_attention_window(Q, kv["K"], kv["V"], start, first, length, O=O, Kblk=blk["K"], Vblk=blk["V"], **scales)
    return dd.dd_block_attention_cached(Q, kv["K"], kv["V"], start, O=O, Kblk=blk["K"], Vblk=blk["V"], **scales)


def _window(case):
    """Half of the cache around the active block."""
    N, bl = case["N"], case["bl"]
    start = (N - bl) * 3 // 4
    length = max(bl, N // 2)
    return min(max(0, start + bl // 2 - length // 2), N - length), length


# ---------------------------------------------------------------------------------------------------- inputs
def _out_type(store):
    return torch.float32 if store == "f32" else torch.bfloat16


def _normal(g, *shape):
    return torch.randn(shape, generator=g, device="cuda")


def _e4m3(x, scale=None):
    """Per-head e4m3 codes: real value = scale x code, scale = amax / 448 unless the cache's is given."""
    if scale is None:
        scale = x.abs().amax(dim=(2, 3)).clamp_min(1e-12) / E4M3_MAX
    codes = (x / scale[:, :, None, None]).clamp_(-E4M3_MAX, E4M3_MAX).to(torch.float8_e4m3fn)
    return codes, scale


def _mx(x, emax, to_codes):
    """Block-scaled storage: every 32 elements of the head dimension share 2^(floor(log2 amax) - emax), an E8M0 code."""
    xb = x.unflatten(-1, (-1, 32))
    _, e = torch.frexp(xb.abs().amax(dim=-1).clamp_min(1e-30))
    shared = (e - 1 - emax).to(torch.int32)
    return to_codes(torch.ldexp(xb, -shared[..., None]).flatten(-2)), (shared + 127).to(torch.uint8)


def _to_e4m3(x):
    return x.clamp(-E4M3_MAX, E4M3_MAX).to(torch.float8_e4m3fn).view(torch.uint8)


def _to_e2m1(x):
    grid = torch.tensor(E2M1_GRID, device="cuda")
    code = torch.bucketize(x.abs(), (grid[1:] + grid[:-1]) / 2).to(torch.uint8) | (x < 0).to(torch.uint8) << 3
    return code[..., 0::2] | code[..., 1::2] << 4            # two per byte, the even element in the low four bits


def _rows(g, B, H, N, d, store):
    """Query rows in the case's storage."""
    x = _normal(g, B, H, N, d)
    if store == "mx":
        codes, s = _mx(x, 8, _to_e4m3)
        return {"x": codes, "s": s}
    if store in ("fp8", "fp8v"):
        codes, s = _e4m3(x)
        return {"x": codes, "s": s}
    return x.to(_out_type(store))


def _kv(g, B, Hkv, N, d, store):
    k, v = _normal(g, B, Hkv, N, d), _normal(g, B, Hkv, N, d)
    if store == "mx":
        (kx, ksc), (vx, vsc) = _mx(k, 8, _to_e4m3), _mx(v, 2, _to_e2m1)
        return {"K": {"x": kx, "s": ksc}, "V": {"x": vx, "s": vsc}}
    if store in ("fp8", "fp8v"):
        kx, ks = _e4m3(k)
        if store == "fp8":
            return {"K": kx, "ks": ks, "V": v.to(torch.bfloat16)}
        vx, vs = _e4m3(v)
        return {"K": kx, "ks": ks, "V": vx, "vs": vs}
    t = _out_type(store)
    return {"K": k.to(t), "V": v.to(t)}


def _block(g, B, H, Hkv, bl, d, store, kv):
    """The active block's fresh rows; K (and V) use the cache's scales."""
    k, v = _normal(g, B, Hkv, bl, d), _normal(g, B, Hkv, bl, d)
    t = _out_type(store)
    return {"Q": _rows(g, B, H, bl, d, store),
            "K": _e4m3(k, kv["ks"])[0] if "ks" in kv else k.to(t),
            "V": _e4m3(v, kv["vs"])[0] if "vs" in kv else v.to(t)}


def _logits(g, P, V, logits, spike=0.0, pair=True):
    """Drafter logits N(0, 3) (with `spike` on one token per row: a confident model), verifier = drafter + N(0, 1)."""
    t = torch.float32 if logits == "f32" else torch.bfloat16
    ld = torch.empty((P, V), dtype=t, device="cuda")
    lv = torch.empty((P, V), dtype=t, device="cuda") if pair else None
    for r in range(0, P, 1024):
        n = min(1024, P - r)
        x = _normal(g, n, V) * (2.0 if spike else 3.0)
        if spike:
            x[torch.arange(n, device="cuda"), torch.randint(0, V, (n,), generator=g, device="cuda")] += spike
        ld[r:r + n] = x
        if pair:
            lv[r:r + n] = x + _normal(g, n, V)
    return {"logits_d": ld, "logits_v": lv} if pair else {"logits_d": ld}


# ---------------------------------------------------------------------------------------------------- work
_BYTES = {"f32": (4.0, 4.0, 4), "bf16": (2.0, 2.0, 2), "fp8": (1.0, 2.0, 2), "fp8v": (1.0, 1.0, 2), "mx": (1.0 + 1 / 32, 0.5 + 1 / 32, 2)}


def _attn_work(case, rows):
    qk, v, o = _BYTES[case["store"]]
    B, H, Hkv, N, d = (case[k] for k in ("B", "H", "Hkv", "N", "d"))
    return {"bytes": B * d * (H * rows * (qk + o) + Hkv * N * (qk + v)), "flops": 4.0 * B * H * rows * N * d}


def _draft_work(case):
    """The block's queries and fresh rows, the cache rows outside the block (of the window), the output."""
    keys = _window(case)[1] if case.get("entry") == "window" else case["N"]
    return _attn_work({**case, "N": keys}, case["bl"])


def _verify_bytes(P, V, logits, both):
    return float(P) * V * (4 if logits == "f32" else 2) * (2 if both else 1) + 10.0 * P
