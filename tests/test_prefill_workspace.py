"""Size of the prefill workspace (host only): calls that fill the chip with short contexts need room
for the row-block list, and none for split partials."""
import pytest


@pytest.mark.parametrize("n_tokens,hq,h,d,max_len", [(1024, 64, 8, 128, 128), (1024, 64, 8, 64, 128), (1200, 32, 8, 128, 30),
                                                     (4096, 40, 40, 128, 256), (8192, 32, 8, 128, 300),
                                                     (3967, 32, 16, 128, 139), (30868, 4, 1, 128, 224)])
def test_short_contexts_need_no_partials(n_tokens, hq, h, d, max_len):
    from paper_2503_18599_amd import binding as B
    assert B.lib().oaken_prefill_attention_workspace_bytes(n_tokens, hq, h, d, max_len, 0) <= 16 * n_tokens + 1024
