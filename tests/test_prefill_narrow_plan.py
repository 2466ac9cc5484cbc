"""Host-only checks of how the narrow products of a short prompt are cut (no GPU): the profiling library reports the plan."""
import pytest

import paper_2604_23553_amd as cf
from tests.prefill_middle import MIDDLE
from tests.prefill_plans import PLANS, WIDE, kinds, taken


def narrow(h, d, f, tokens, n_cu=256, rows=128):
    with cf.profile_build():
        return cf.cfpp_debug_prefill_narrow(cf.Config(h, h // d, d, 16, f, 2, 16, 1, 10000.0, 1e-5, 0), rows, tokens, n_cu)


@pytest.mark.parametrize("h,d", [(128, 64), (384, 128), (512, 64), (640, 80), (1024, 128), (1280, 80), (1536, 64), (2048, 64),
                                 (2560, 80), (2688, 128), (3072, 128), (3968, 64), (4096, 128)])
def test_plans_stay_inside_their_limits(h, d):
    scratch = 384 * 128 * 128 * 4 - 128 * 1024 + 128 * h * 4           # the parts' memory of a pass with 128 rows: queries and parts
    for f in {128, h, 4 * h, 4 * h + 128, 32768} & set(range(128, 32769, 128)):
        for n_cu in (32, 64, 80, 256, 304):
            for t in range(1, 129):
                p = narrow(h, d, f, t, n_cu)
                if p is None:
                    continue
                rows_in, tiles_in, rows_out, tiles_out, parts, sets = p
                assert t <= 64 and 8 * sets >= t and (tiles_in * sets <= 48 and tiles_out * sets <= 48)
                assert rows_in % 2 == 0 and rows_in <= 16 * tiles_in and rows_out % 2 == 0 and rows_out <= 16 * tiles_out
                assert -(-3 * h // rows_in) + -(-f // rows_in) <= n_cu and -(-h // rows_out) * parts <= 2 * n_cu
                assert 1 <= parts <= min(16, (h + f) // 64) and parts * t * h * 4 <= scratch


def test_which_passes_take_them():
    for t in (1, 8, 33, 64):
        assert narrow(512, 64, 2048, t) and narrow(2560, 80, 10240, t)
    assert narrow(2560, 80, 10240, 65) is None                          # more than 64 tokens
    assert narrow(4096, 128, 16384, 48) and narrow(4096, 128, 16384, 49) is None       # 8 tiles x 8 sets
    assert narrow(512, 64, 32768, 20) is None                           # more than 128 rows to a CU
    assert narrow(2560, 80, 10240, 20, n_cu=128) is None


# ---- passes of 65 .. 1024 tokens: other tiles where they are better --------------------------------------------------
def tiles(h, d, f, tokens):
    cfg = cf.Config(h, h // d, d, 16, f, 2, 16, 1, 10000.0, 1e-5, 0)
    rows = -(-tokens // 128) * 128
    with cf.profile_build():
        return cf.cfpp_debug_prefill_plan(cfg, rows, tokens), cf.cfpp_debug_prefill_tiles(cfg, rows, tokens)


@pytest.mark.parametrize("shape,tokens,first,second", MIDDLE)
def test_what_a_middle_size_takes(shape, tokens, first, second):
    (base, _), (got, _) = tiles(shape.hidden, shape.head_dim, shape.ffn, tokens)
    assert got == (first or base[0], second or base[1])


def test_middle_sizes_take_tiles_that_the_gpu_runs_and_load_inside_their_operands():
    run = set().union(*(kinds(taken(p[0], p[1])[0]) for p in (*PLANS, *MIDDLE, *WIDE)))
    for h, d in ((128, 64), (512, 64), (640, 80), (1024, 128), (1280, 80), (1536, 64), (1920, 80), (2048, 64), (2560, 80), (2688, 128),
                 (3072, 128), (3200, 80), (4096, 128)):
        for f in (h, 4 * h, min(32768, 8 * h)):
            for t in (*range(1, 131, 9), *range(131, 1025, 29), 1025, 2048, 4096):
                (base, _), (got, past) = tiles(h, d, f, t)
                assert past == ((0, 0), (0, 0)), (h, f, t, past)
                if not 64 < t <= 1024:
                    assert got == base
                if t > 64:
                    assert kinds(got) <= run, (h, f, t, got)
