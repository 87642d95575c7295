"""The drafter call's key splits, as the workspace query shows them: a bf16 call with 128 head dims and at most 64 query rows per
kv head never asks for a second round of the chip's 256 compute units while its row tiles alone fit one."""
import pytest

import paper_2604_05250_amd as dd


@pytest.mark.parametrize("N", [128, 1000, 4096])
@pytest.mark.parametrize("bl", [1, 16, 64])
def test_bf16_splits_fit_one_round(N, bl):
    for tiles in list(range(1, 258)) + [300, 512]:
        need = dd.dd_block_attention_cached_workspace_bytes(bl, tiles, 1, 1, N, 128, dd.BF16, dd.BF16)
        splits = max(1, need // (tiles * bl * (128 + 2) * 4))
        assert splits == max(1, min(256 // tiles, N // 128, 16)), (tiles, splits)
