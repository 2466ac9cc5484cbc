"""Host-only checks of how the prompt-sized products are cut into tiles (no GPU): the
profiling library reports the plan that a pass of a given size gets and the rows that its
tiles' loads reach."""
import os
import re

import pytest

import paper_2604_23553_amd as cf
import synth
from tests.prefill_middle import MIDDLE
from tests.prefill_plans import PLANS, WIDE, kinds, taken

CSRC = os.path.join(os.path.dirname(os.path.abspath(cf.__file__)), "csrc")
TOKENS = (1, 20, 32, 33, 64, 65, 100, 128, 129, 256, 300, 384, 500, 640, 900, 1100, 1153, 1408, 1531, 2048, 2600, 2688,
          2700, 3100, 3200, 3400, 3840, 3968, 4096)


def plan(h, d, f, tokens, rows=None):
    cfg = cf.Config(h, h // d, d, 16, f, 2, 16, 1, 10000.0, 1e-5, 0)
    with cf.profile_build():
        return cf.cfpp_debug_prefill_plan(cfg, rows or -(-tokens // 128) * 128, tokens)


@pytest.mark.parametrize("h,d", [(128, 64), (256, 64), (512, 64), (640, 80), (1024, 128), (1280, 80), (1536, 64), (2048, 64),
                                 (2560, 80), (2688, 128), (3200, 80), (3968, 64), (4096, 128), (4096, 64)])
def test_no_tile_loads_outside_its_operands(h, d):
    """Tiles overhang the features (192, 256 and 320 columns) and the tokens (256 rows): their loads stay inside."""
    for f in {128, h, 4 * h, 4 * h + 128, 32768} & set(range(128, 32769, 128)):
        for t in TOKENS:
            _, past = plan(h, d, f, t)
            assert past == ((0, 0), (0, 0)), (h, f, t, past)


@pytest.mark.parametrize("shape,tokens,first,second", PLANS)
def test_what_a_size_selects(shape, tokens, first, second):
    got, past = taken(shape, tokens)
    assert got == (first, second) and past == ((0, 0), (0, 0))


def test_the_passes_run_on_the_gpu_take_every_tile_that_passes_take():
    run = set().union(*(kinds(taken(p[0], p[1])[0]) for p in (*PLANS, *MIDDLE, *WIDE)))
    for h in range(128, 4097, 128):
        for f in sorted({h, 2 * h, 4 * h, 8 * h, h // 256 * 128, 11 * h // 512 * 128, 32768} & set(range(128, 32769, 128))):
            shape = synth.ModelShape(h, h // 64, 64, 16, f, n_layers=2)
            for t in (*range(1, 260, 5), *range(260, 4097, 41)):
                for rows in (-(-t // 128) * 128, 4096):
                    p = taken(shape, t, rows)
                    new = kinds(p[0]) - run if p else set()
                    assert not new, (h, f, t, new)


def test_a_plan_is_refused_as_the_call_is():
    cfg = cf.Config(512, 8, 64, 16, 2048, 2, 16, 1, 10000.0, 1e-5, 2)          # the sequential form
    with cf.profile_build():
        for rows, n in ((128, 129), (100, 20), (4224, 20), (128, 0)):
            with pytest.raises(cf.CfppError):
                cf.cfpp_debug_prefill_plan(cfg, rows, n)
        with pytest.raises(cf.CfppError) as e:
            cf.cfpp_debug_prefill_plan(cfg, 128, 20)
        assert e.value.status == -2


def test_asm_that_sets_m0_says_so():
    """M0 carries the LDS address of a memory-to-LDS load: the compiler has to know of it."""
    found = 0
    for name in sorted(os.listdir(CSRC)):
        if name.endswith((".hip", ".h")):
            text = open(os.path.join(CSRC, name)).read()
            for stmt in re.findall(r"\basm\s+(?:volatile)?\s*\(.*?\)\s*;", text, flags=re.S):
                if "m0," in stmt:
                    found += 1
                    assert '"m0"' in stmt.rsplit(":", 1)[1], f"{name}: {stmt}"
    assert found >= 2
