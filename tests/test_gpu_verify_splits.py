"""Row splits of a verification with few rows: the shortest ones (a workgroup per compute unit at most) and those of whole load
rounds, at the edges of a split, of a load round and of the rule, against the CPU oracle (same tolerances as everywhere)."""
import numpy as np
import pytest

import paper_2604_05250_amd as dd
from paper_2604_05250_amd import workloads as wl
from test_gpu_verify import check_against_oracle, check_all_scores, check_unmask

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("fine", [None, 0])
@pytest.mark.parametrize("P,V,dtype", [(1, 8200, wl.BF16),          # one vector past a row that is not split
                                       (16, 32768, wl.BF16),        # 16 x 256 vectors: the last shape of 256 workgroups ...
                                       (17, 32768, wl.BF16),        # ... and the first past it
                                       (5, 32776, wl.BF16),         # a last split of one vector
                                       (8, 152064, wl.BF16),        # a full round and a remainder of one load in every split
                                       (3, 4100, wl.F32), (16, 16640, wl.F32)])
def test_row_splits_at_their_edges(monkeypatch, fine, P, V, dtype):
    if fine is not None:
        monkeypatch.setenv("DD_TUNE_VERIFY_FINE", str(fine))
    cfg = wl.custom_config(B=1, G=P, V=V, logit_dtype=dtype, sigma_d=3.0, sigma_n=1.0, decoded_frac=0.5)
    inp = wl.verify_inputs(cfg, seed=P)
    for mode, tau in ((wl.KL_THRESH, 0.4), (wl.KL_PROB, 0.0), (wl.CONF_THRESH, 0.01)):
        check_against_oracle(inp, mode, tau, 3, 1, P, dtype, f"P={P} V={V} mode={mode} fine={fine}")
    mask = (np.arange(P) % 3 != 0).astype(np.uint8)
    check_unmask(inp, mask, wl.UNMASK_TOPK, 2.0, 1, P, dtype, f"unmask P={P} V={V} fine={fine}")
    check_all_scores(inp["logits_d"], inp["logits_v"], dtype, f"scores P={P} V={V} fine={fine}")


@pytest.mark.parametrize("V", [8200, 32000, 152064])
def test_a_workspace_serves_fewer_rows(V):
    need = [dd.dd_verify_remask_workspace_bytes(1, P, V, wl.BF16) for P in range(1, 192)]
    split = [n for n in need if n > 0]
    fine = [n for n, P in zip(need, range(1, 192)) if 0 < P * 16 <= 256]
    assert len(fine) == 16 and all(n >= fine[-1] for n in split[16:])
