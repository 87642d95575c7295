"""Scratch memory of a verification with few rows: what holds the states of splits of whole load rounds serves the call, also where the
library would rather split its rows further, and nothing past it is written; a state less is refused."""
import numpy as np
import pytest

import paper_2604_05250_amd as dd
from paper_2604_05250_amd import workloads as wl
from test_gpu_verify import check_against_oracle, check_all_scores, check_unmask

pytestmark = pytest.mark.gpu
STATE, BAND = 32, 8192                               # bytes


@pytest.mark.parametrize("P,V,dtype", [(1, 8200, wl.BF16), (4, 32000, wl.BF16), (16, 16384, wl.BF16), (5, 32776, wl.BF16), (3, 4100, wl.F32)])
def test_states_of_whole_load_rounds_are_enough(P, V, dtype):
    import torch
    nvec = V * (2 if dtype == wl.BF16 else 4) // 16
    need = P * -(-nvec // 1024) * STATE              # (a load round is 1024 vectors; sixteen of them hold each of these rows)
    assert need < dd.dd_verify_remask_workspace_bytes(1, P, V, dtype)
    base = torch.full((need + BAND,), 0xA5, dtype=torch.uint8, device="cuda:0")
    cfg = wl.custom_config(B=1, G=P, V=V, logit_dtype=dtype, sigma_d=3.0, sigma_n=1.0, decoded_frac=0.5)
    inp = wl.verify_inputs(cfg, seed=P)
    mask = (np.arange(P) % 3 != 0).astype(np.uint8)

    def run(what):
        for mode, tau in ((wl.KL_THRESH, 0.4), (wl.KL_PROB, 0.0), (wl.CONF_THRESH, 0.01)):
            check_against_oracle(inp, mode, tau, 3, 1, P, dtype, f"{what} mode={mode}")
        check_unmask(inp, mask, wl.UNMASK_TOPK, 2.0, 1, P, dtype, f"unmask {what}")
        check_all_scores(inp["logits_d"], inp["logits_v"], dtype, f"scores {what}")
    with dd.fixed_workspace(base[:need]):
        run(f"P={P} V={V} {need} bytes")
    torch.cuda.synchronize()
    assert bool((base[need:] == 0xA5).all()), "written past the workspace"
    with dd.fixed_workspace(base[:need - 1]):
        with pytest.raises(RuntimeError):
            run("refused")
