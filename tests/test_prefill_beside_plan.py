"""Host-only checks of what a short prompt's MLP-down beside the attention takes of the scratch (no GPU: the profiling library reports it)."""
import pytest

import paper_2604_23553_amd as cf


def beside(h, d, f, tokens, pos0=0, part_bytes=0, rows=128):
    with cf.profile_build():
        return cf.cfpp_debug_prefill_beside(cf.Config(h, h // d, d, 16, f, 2, 8192, 1, 10000.0, 1e-5, 0), rows, tokens, pos0, part_bytes)


# Less scratch than it has (which no entry point offers today): MLP-down moves behind the attention where its parts do not fit beside it, and
# where the second product's don't fit either the tiled plan stays as it was made.
@pytest.mark.parametrize("h,d,f,tokens", [(512, 64, 2048, 16), (1280, 80, 5120, 8), (1024, 128, 4096, 37), (4096, 128, 16384, 12)])
def test_scratch_that_is_too_small_for_the_parts(h, d, f, tokens):
    downs, splits, attention, _ = beside(h, d, f, tokens)
    assert downs > 0
    need = -(-(downs + splits) * tokens * h * 4 // 256) * 256
    assert beside(h, d, f, tokens, part_bytes=need)[:2] == (downs, splits)
    fewer = beside(h, d, f, tokens, part_bytes=need - 256)
    assert fewer[0] == 0 and fewer[1] > 0
    # (the queries' place, ahead of that part of the scratch, is 128 rows: with 128 rows of tokens in one part that is enough)
    for part in range(256, need, max(256, need // 7 // 256 * 256)):
        got = beside(h, d, f, tokens, part_bytes=part)
        if got is not True:
            assert got and got[0] == 0 and got[1] * tokens * h * 4 <= part + 128 * h * 4
