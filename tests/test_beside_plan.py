"""Host-only checks of what runs beside the attention (no GPU: the profiling library reports it): what each case of the GPU tests selects, that
these cases take every branch, and limits over all shapes."""
import pytest

import paper_2604_23553_amd as cf
from tests.beside_plans import ALONE, GROUPS, SHORT, STEPS, _shape, groups, short, step


@pytest.mark.parametrize("shape,lens,downs,workgroups", STEPS)
def test_what_a_step_selects(shape, lens, downs, workgroups):
    together, pieces, attention, *down = step(shape, lens)
    assert not together and down == [downs, workgroups]


@pytest.mark.parametrize("shape,pos0,T,max_batch,b,plans", GROUPS + ALONE)
def test_what_a_group_selects(shape, pos0, T, max_batch, b, plans):
    assert [(g[0], g[1], g[3]) for g in groups(shape, pos0, T, max_batch)] == plans


@pytest.mark.parametrize("shape,pos0,T,downs,workgroups,attention", SHORT)
def test_what_a_short_prompt_selects(shape, pos0, T, downs, workgroups, attention):
    got = short(shape, pos0, T)
    assert (got[0], got[3], got[2]) == (downs, workgroups, attention)


def test_the_cases_take_every_branch():
    one, several = [c for c in STEPS if len(c[1]) == 1], [c for c in STEPS if len(c[1]) > 1]
    assert {c[2] for c in one} >= {1, 4, 7, 8}
    assert {c[2] for c in several} == {1, 2, 3, 4, 5, 7, 8} and any(c[3] > 256 for c in several)           # (two workgroups to a CU)
    plans = [(g, (c[0], c[1] + i * min(c[3], 8))) for c in GROUPS + ALONE for i, g in enumerate(groups(*c[:4]))]
    assert {s.head_dim for g, (s, _) in plans if g[0]} == {64, 80, 128} == {s.head_dim for g, (s, _) in plans if not g[0]}
    assert {g[1] for g, _ in plans if g[0]} >= {3, 7, 8} and {first for g, (_, first) in plans} >= {890, 895, 896}
    fewer = [g for c in GROUPS + ALONE for i, g in enumerate(groups(*c[:4])) if min(c[3], 8, c[2] - i * min(c[3], 8)) > 1
             and g[3] < step(c[0], [1] * min(c[3], 8, c[2] - i * min(c[3], 8)))[3]]
    assert fewer and any(g[0] for g in fewer) and any(not g[0] for g in fewer)                              # (fewer parts than a step's)
    assert {c[3] for c in SHORT} == set(range(9)) and any(c[4] > 256 for c in SHORT)
    assert {-(-c[2] // 8) for c in SHORT} == {1, 2, 3, 4, 5, 6} and any(c[5] == 1 for c in SHORT)
    assert {c[0].head_dim for c in SHORT if c[5] > 1} == {64, 80, 128}


# Which parts of MLP-down there may be, over all the shapes that the batched path takes: a head has room for eight behind the attention's pieces
# (18 slots and more at hidden <= 4096), a part has chunks of 64 columns, and the attention's workgroups are counted right for a grid below 2^31.
def test_parts_stay_inside_their_limits():
    for h in range(128, 4097, 128):
        for d in (64, 80, 128):
            if h % d:
                continue
            for f in {h, 2 * h, 4 * h, 8 * h}:
                if f > 32768:
                    continue
                cfg = cf.Config(h, h // d, d, 0, f, 1, 70000, 8, 10000.0, 1e-5, 0)
                with cf.profile_build():
                    for n in (1, 2, 4, 5, 8):
                        for first in (-1, 0, 20, 127, 128, 500, 895, 896, 1000, 3000, 60000):
                            together, pieces, attention, downs, workgroups = cf.cfpp_debug_attention_plan(cfg, n, first)
                            assert 1 <= downs <= 8 and downs <= max(1, f // 1024) and workgroups == downs * h // (16 if n == 1 else 32)
                            assert attention % (h // d) == 0 and 1 <= attention < 1 << 20 and pieces >= 1
                            if together:
                                assert n >= 2 and pieces <= 8 and attention == (pieces + 1) * (h // d)


def test_every_branch_has_its_shapes():
    assert groups(_shape(640, 80, 640, 20), 896, 8, 8)[0][0] is False and groups(_shape(512, 64, 512, 0), 896, 2, 8)[0][0] is True
    assert groups(_shape(512, 64, 512, 0), 4000, 1, 8)[0][0] is False                  # one token
    for h, d, line in ((1024, 64, 10000), (1280, 64, 8000), (1280, 80, 10000), (2560, 128, 8000), (1408, 64, 0), (2816, 128, 0), (1920, 80, 0), (4096, 64, 0)):
        for n in (2, 3, 5, 8):
            at = max(896, -(-line // n))               # the first position at which a group of n attends together
            assert [g[0] for p in (at - 1, at) for g in groups(_shape(h, d, h, 0), p, n, 8)] == [False, True], (h, d, n)
