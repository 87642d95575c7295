"""The Python binding on GPU tensors: what its errors are."""
import pytest

import paper_2604_05250_amd as dd

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("call", ["output", "scratch"])
def test_failed_allocations_are_out_of_memory_errors(call):
    # the process may hold what it holds and no more; nothing is launched
    import torch
    with torch.cuda.stream(torch.cuda.Stream()):             # (a stream of its own: no scratch tensor kept from another call)
        z = lambda *s: torch.zeros(s, dtype=torch.bfloat16, device="cuda:0")
        q, kv, o = z(1, 32, 4096, 128), z(1, 32, 4096, 128), z(1, 32, 64, 128)
        qb = z(1, 32, 64, 128)
        torch.cuda.synchronize()
        torch.cuda.empty_cache()
        try:
            torch.cuda.set_per_process_memory_fraction(torch.cuda.memory_reserved() / torch.cuda.get_device_properties(0).total_memory)
            with pytest.raises(torch.OutOfMemoryError):
                if call == "output":
                    dd.dd_bidir_attention(q, kv, kv)
                else:
                    dd.dd_block_attention_cached(qb, kv, kv, 0, O=o)
        finally:
            torch.cuda.set_per_process_memory_fraction(1.0)
    assert dd.dd_bidir_attention(q, kv, kv).shape == q.shape
    torch.cuda.synchronize()
