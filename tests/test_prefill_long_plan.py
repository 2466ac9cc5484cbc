"""Host-only checks of the first product of long passes: which tiles it takes, where it is cut in two, and that no tile's loads
leave the weights (no GPU: the profiling library reports the plan)."""
import pytest

import synth
from tests.prefill_long import LONG, first_product
from tests.prefill_middle import MIDDLE
from tests.prefill_plans import PLANS


@pytest.mark.parametrize("shape,tokens,tile,second", LONG)
def test_what_a_size_selects(shape, tokens, tile, second):
    (got, cut, rest), past = first_product(shape, tokens)
    assert (got, rest) == (tile, second) and past == (0, 0)
    assert 0 < cut <= shape.ffn and cut % 128 == 0 and (cut < shape.ffn) == (second is not None)


def test_the_passes_run_on_the_gpu_take_every_tile_of_long_passes():
    run = set()
    for shape, tokens in [p[:2] for p in (*LONG, *PLANS, *MIDDLE)]:
        (tile, _, second), _ = first_product(shape, tokens)
        run |= {(tile, second is not None), ("second", second)}
    for h in range(128, 4097, 128):
        for f in sorted({h, 2 * h, 4 * h, 8 * h, h + 128, 4 * h + 128, 32768} & set(range(128, 32769, 128))):
            shape = synth.ModelShape(h, h // 64, 64, 16, f, n_layers=2)
            for t in range(513, 4097, 56):
                for rows in (-(-t // 128) * 128, 4096):
                    (tile, cut, second), past = first_product(shape, t, rows)
                    assert past == (0, 0) and 0 < cut <= f and cut % 128 == 0 and (cut < f) == (second is not None), (h, f, t)
                    assert (tile, second is not None) in run and ("second", second) in run, (h, f, t, tile, second)


def test_shorter_passes_keep_their_plan():
    from tests.prefill_plans import H2560, H4096, taken
    for shape in (H2560, H4096):
        for t in (65, 100, 300, 500, 512):
            (tile, cut, second), _ = first_product(shape, t)
            assert tile == taken(shape, t)[0][0][:2] and cut == shape.ffn and second is None
