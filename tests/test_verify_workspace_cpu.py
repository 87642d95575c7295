"""The verification's workspace query: a size queried for some number of split rows (191 at most) serves every smaller number."""
import pytest

import paper_2604_05250_amd as dd


@pytest.mark.parametrize("dtype,V", [(dd.BF16, V) for V in (8, 8192, 8200, 32000, 32776, 50264, 90184, 126464, 128256, 152064, 1 << 20)] +
                                    [(dd.F32, V) for V in (1000, 4096, 4100, 45092, 63232, 152064)])
def test_a_workspace_serves_fewer_rows(dtype, V):
    need = [dd.dd_verify_remask_workspace_bytes(1, P, V, dtype) for P in range(1, 192)]
    assert all(a <= b for a, b in zip(need, need[1:])), [P for P in range(1, 191) if need[P] < need[P - 1]]
    assert need[0] > 0 and need[-1] <= 97792             # (what the static scratch's limit counts on)
    assert dd.dd_verify_remask_workspace_bytes(1, 192, V, dtype) == 0
    for call in (dd.dd_unmask_workspace_bytes, lambda B, G, V, t: dd.dd_verify_scores_workspace_bytes(B * G, V, t)):
        assert [call(1, P, V, dtype) for P in range(1, 192)] == need


@pytest.mark.parametrize("V", [8200, 32000, 90184, 126464, 152064])
def test_the_query_holds_what_a_call_splits_into(V):
    # splits of whole load rounds (1024 vectors), about 2048 workgroups in all; of 256 vectors where that is at most 256 workgroups
    nvec = V // 8
    for P in range(1, 192):
        shortest = -(-nvec // max(1, min(16, -(-2048 // P))))
        fine, rounds = (P * -(-nvec // (-(-shortest // m) * m)) for m in (256, 1024))
        assert dd.dd_verify_remask_workspace_bytes(1, P, V, dd.BF16) >= 32 * (fine if fine <= 256 else rounds), P
