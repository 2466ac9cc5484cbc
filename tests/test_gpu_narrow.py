"""GPU parity of the kernels for few tokens (csrc/narrow_gemm.hip, prefill_narrow.hip), of the split prompt attention and of the
tiles of middle-sized passes, where their cut can go wrong: wavefronts with
unequal shares of K or with none, tiles of 16 rows that are partly there, one row group or eight tiles to a workgroup."""
import numpy as np
import pytest
import torch                       # (ahead of the library: both take the HIP runtime that comes with it)

import synth
from tests.beside_plans import ALONE, GROUPS, SHORT, STEPS, groups, short, step
from tests.parity import MAX_ABS, assert_appended_rows, assert_block_close, ulp16
from tests.prefill_long import LONG, first_product
from tests.prefill_middle import MIDDLE
from tests.prefill_plans import WIDE
from tests.test_gpu_stack import _batched_case, check_appended_rows

pytestmark = pytest.mark.gpu


def _shape(h, d, f, r, layers=2):
    return synth.ModelShape(h, h // d, d, r, f, n_layers=layers, name=f"d{d}-h{h}-f{f}")


# hidden / 64 chunks over 8 wavefronts: 2 (six wavefronts without), 6, 10, 20, 22; rows of a workgroup by tiles of 16:
# 2 .. 14 (one tile), 18 (two, the second a quarter), 36, 48 (three), 72 (five), 84 (eight)
@pytest.mark.parametrize("shape,B", [
    (_shape(128, 64, 128, 16), 1 + 1), (_shape(384, 128, 384, 0), 8), (_shape(640, 80, 2560, 20), 3), (_shape(1280, 80, 5120, 80), 7),
    (_shape(1408, 128, 4224, 32), 9), (_shape(3072, 128, 3072, 32, 1), 4), (_shape(3072, 64, 12288, 16, 1), 2),
])
def test_shares_of_rows_and_columns(orc, shape, B):
    _batched_case(orc, shape, B, shape.n_layers, synth.seq_lens(5, B, 0, 40))


# MLP-down beside the attention: K in one to five, seven and eight parts (six there are none), one workgroup to a CU and two, parts and wavefronts
# with unequal shares of chunks; and 64 heads of so long a context that their pieces stop where the parts begin.
@pytest.mark.parametrize("shape,lens,downs,workgroups", STEPS)
def test_mlp_down_beside_the_attention(orc, shape, lens, downs, workgroups):
    from paper_2604_23553_amd.harness import DeviceStack
    assert step(shape, lens)[3:] == (downs, workgroups)
    if len(lens) > 1:
        return _batched_case(orc, shape, len(lens), shape.n_layers, np.array(lens, dtype=np.int32))
    print(f"[case] one sequence {shape.name} S={lens[0]}", flush=True)
    S, w = lens[0], synth.layer_weights(shape, 13, 0)
    K, V = synth.kv_cache(shape, 13, 0, S, S + 1)
    x = synth.x_input(shape, 13)
    ds = DeviceStack(shape, S + 1, 1, 1)
    try:
        ds.load_layer(0, w)
        ds.load_kv(0, K, V, S)
        ds.set_inputs(x, S)
        ds.block_decode(0)
        ds.check()
        assert_block_close(ds.result()[0], orc.block_decode_f16(shape, w, K[0].copy(), V[0].copy(), S, x[0]), shape.name)
    finally:
        ds.close()


# A group of prompt tokens behind a longer context attends together: the first such position and the one ahead of it, lengths on both
# sides of a row of 32 positions, groups of 2 to 8 tokens (the last one of a prompt smaller; one alone takes the other kernel), pieces that
# share rows unevenly, fewer than eight, another sequence's cache, at the three head sizes; 16 to 21 heads on both sides of their own line; eight heads of
# 128, which keep to the other kernel.
@pytest.mark.parametrize("shape,pos0,T,max_batch,b,plans", GROUPS)
def test_group_attention(orc, shape, pos0, T, max_batch, b, plans):
    from tests.test_gpu_prefill import _check_prompt
    assert [(g[0], g[1], g[3]) for g in groups(shape, pos0, T, max_batch)] == plans
    _check_prompt(orc, shape, 41, pos0, T, max_batch, b, then_decode=False, row_check_every=5)


# Ahead of that every query attends for itself, in a grid made for the group's positions: one piece a head and the first position with
# two, of 16 rows (up to 4 tokens) and of 32; heads of 128, whose rows are 16 positions; as many pieces as workgroups allow; one token; and fewer
# parts of MLP-down beside it (hidden 1280 and 1536) or not, on both sides of position 128 (hidden 2560).
@pytest.mark.parametrize("shape,pos0,T,max_batch,b,plans", ALONE)
def test_group_with_a_grid_for_its_positions(orc, shape, pos0, T, max_batch, b, plans):
    from tests.test_gpu_prefill import _check_prompt
    assert [(g[0], g[1], g[3]) for g in groups(shape, pos0, T, max_batch)] == plans
    _check_prompt(orc, shape, 47, pos0, T, max_batch, b, then_decode=False, row_check_every=5)


# Its error against 64 bits: the queries and the cache rows that the kernel read (taps, exported cache), attention in numpy's doubles.
# What bounds it: the tap's head and remainder, 2^-25 of an output of about 1 / sqrt(positions) (1e-6 of it at 1000 positions), a few 2^-24 of
# the weights (exponential, head and remainder) and of the sums; and the scores' own rounding, 2^-24 of the sum of a score's terms' sizes or
# so, which the weights take up as it stands.  Also where the queries are large or small as a whole.
@pytest.mark.parametrize("gain", [1.0, 300.0, 1e-4])
@pytest.mark.parametrize("shape,pos0", [(_shape(512, 64, 2048, 16, 1), 1001), (_shape(1280, 80, 2560, 20, 1), 1290), (_shape(2048, 128, 2048, 32, 1), 2100)])
def test_group_attention_against_64_bits(shape, pos0, gain):
    import paper_2604_23553_amd as cf
    from paper_2604_23553_amd.harness import DeviceStack
    T, h, H, d = 8, shape.hidden, shape.n_heads, shape.head_dim
    assert groups(shape, pos0, T, T)[0][0]
    print(f"[case] group attention error {shape.name} pos0={pos0} gain={gain}", flush=True)
    w = {n: a.copy() for n, a in synth.layer_weights(shape, 43, 0).items()}
    rows = np.arange(3 * h).reshape(H, 3, d)[:, 0].ravel()                 # the queries' rows
    w["w_qkv"][rows] = (w["w_qkv"][rows].astype(np.float32) * gain).astype(np.float16)
    w["b_qkv"][rows] = (w["b_qkv"][rows].astype(np.float32) * gain).astype(np.float16)
    with cf.profile_build():
        ds = DeviceStack(shape, pos0 + T, T, 1)
        try:
            ds.load_layer(0, w)
            K, V = synth.kv_cache(shape, 43, 0, pos0, pos0 + T, T)
            if gain > 1.0:
                K = (K.astype(np.float32) / gain).astype(np.float16)
            ds.load_kv(0, K, V, pos0)
            ds.prefill(synth.x_input(shape, 43, T), pos0)
            ds.check()
            q = ds.tap(0, T * h).reshape(T, H, d).astype(np.float64)
            o = ds.tap(3, T * h).reshape(T, H, d).astype(np.float64)
            k, v = (a.astype(np.float64) for a in ds.export_kv(0, 0, 0, pos0 + T))
        finally:
            ds.close()
    for t in range(T):
        s = np.einsum("hd,hpd->hp", q[t], k[:, :pos0 + t + 1]) / np.sqrt(d)
        p = np.exp(s - s.max(axis=1, keepdims=True))
        want = np.einsum("hp,hpd->hd", p / p.sum(axis=1, keepdims=True), v[:, :pos0 + t + 1])
        terms = np.einsum("hd,hpd->hp", np.abs(q[t]), np.abs(k[:, :pos0 + t + 1])) / np.sqrt(d)
        err = np.abs(o[t] - want)
        size = np.einsum("hp,hpd->hd", p / p.sum(axis=1, keepdims=True), np.abs(v[:, :pos0 + t + 1]))
        bound = 2.0 ** -25 + 2.0 ** -22 * np.abs(want) + 2.0 ** -24 * size * (4 + terms.max(axis=1, keepdims=True))
        print(f"  token {t}: relative 2-norm {np.linalg.norm(err) / np.linalg.norm(want):.2e}, most of the bound {(err / bound).max():.2f}")
        assert (err <= bound).all(), f"token {t}"


# Weights far below the largest and query elements far below theirs keep the precision of fp32.  "light": one key has 2^16 times the weight of
# every other, and its V is zero, so that the outputs are the light ones'.  "uneven": a query's first element is 3000 where every
# other is about 1, and meets zeros in K.  Bound: the tap's head and remainder, 2^-25 and 2^-22 of the output; of a key's weight, 2^-22 (its two halves, the
# exponential, the sums) and its score's error, 2^-23 of the sum of its terms' sizes, plus 2^-24 of its distance from the largest score, whose
# difference is rounded.  Two fp16 values that keep 2^-25 of the largest only are off by 12 to 30 of it.
@pytest.mark.parametrize("kind", ["light", "uneven"])
@pytest.mark.parametrize("shape,pos0", [(_shape(512, 64, 512, 0, 1), 1001), (_shape(1280, 80, 1280, 0, 1), 1700), (_shape(2048, 128, 2048, 0, 1), 1300)])
def test_group_attention_of_light_keys_and_uneven_queries(shape, pos0, kind):
    import paper_2604_23553_amd as cf
    from paper_2604_23553_amd.harness import DeviceStack
    T, h, H, d = 8, shape.hidden, shape.n_heads, shape.head_dim
    assert groups(shape, pos0, T, T)[0][0]
    print(f"[case] group attention {kind} {shape.name} pos0={pos0}", flush=True)
    w = {n: a.copy() for n, a in synth.layer_weights(shape, 67, 0).items()}
    rng, at = np.random.default_rng(67), np.arange(3 * h).reshape(H, 3, d)
    K, V = synth.kv_cache(shape, 67, 0, pos0, pos0 + T, T)
    if kind == "light":
        u = rng.choice([-1.0, 1.0], (H, d))
        w["w_qkv"][at[:, 0].ravel()] *= np.float16(0.05)                   # every query: nearly u
        w["b_qkv"][at[:, 0].ravel()] = u.ravel().astype(np.float16)
        K[0, :, :pos0] *= np.float16(0.3)
        V[0, :, :pos0] *= np.float16(100.0)
        K[0, :, pos0 // 2] = (u * 16 * np.log(2.0) / np.sqrt(d)).astype(np.float16)
        V[0, :, pos0 // 2] = 0
    else:
        w["b_qkv"][at[:, 0, 0]] = np.float16(3000.0)
        w["w_qkv"][at[:, 1, 0]] = 0
        w["b_qkv"][at[:, 1, 0]] = 0
        K[0, :, :, 0] = 0
    with cf.profile_build():
        ds = DeviceStack(shape, pos0 + T, T, 1)
        try:
            ds.load_layer(0, w)
            ds.load_kv(0, K, V, pos0)
            ds.prefill(synth.x_input(shape, 67, T), pos0)
            ds.check()
            q = ds.tap(0, T * h).reshape(T, H, d).astype(np.float64)
            o = ds.tap(3, T * h).reshape(T, H, d).astype(np.float64)
            k, v = (a.astype(np.float64) for a in ds.export_kv(0, 0, 0, pos0 + T))
        finally:
            ds.close()
    worst = 0.0
    for t in range(T):
        n = pos0 + t + 1
        s = np.einsum("hd,hpd->hp", q[t], k[:, :n]) / np.sqrt(d)
        far = s.max(axis=1, keepdims=True) - s
        p = np.exp(-far) / np.exp(-far).sum(axis=1, keepdims=True)
        want = np.einsum("hp,hpd->hd", p, v[:, :n])
        terms = np.einsum("hd,hpd->hp", np.abs(q[t]), np.abs(k[:, :n])) / np.sqrt(d)
        bound = 2.0 ** -25 + 2.0 ** -22 * np.abs(want) + np.einsum("hp,hpd->hd", p * (2.0 ** -22 + 2.0 ** -23 * terms + 2.0 ** -24 * far), np.abs(v[:, :n]))
        worst = max(worst, (np.abs(o[t] - want) / bound).max())
    print(f"  most of the bound {worst:.2f}")
    assert worst <= 1.0


# A token of the group that is not finite reaches no earlier one; a cached V element that is infinite makes that dimension of every
# token's output infinite and no other.
@pytest.mark.parametrize("shape,pos0,bad", [
    (_shape(512, 64, 2048, 16), 37, 3), (_shape(512, 64, 2048, 16), 911, 3), (_shape(1280, 80, 2560, 20), 1260, 7), (_shape(2048, 128, 2048, 32), 1280, 5),
])
def test_group_with_a_token_that_is_not_finite(shape, pos0, bad):
    from paper_2604_23553_amd.harness import DeviceStack
    print(f"[case] group ahead of a NaN {shape.name} bad={bad}", flush=True)
    T, X = 8, synth.x_input(shape, 47, 8)
    assert groups(shape, pos0, T, T)[0][0] == (pos0 > 800)
    outs = []
    for nan in (False, True):
        ds = DeviceStack(shape, pos0 + T, T, shape.n_layers)
        try:
            for l in range(shape.n_layers):
                ds.load_layer(l, synth.layer_weights(shape, 47, l))
                ds.load_kv(l, *synth.kv_cache(shape, 47, l, pos0, pos0 + T, T), pos0)
            if nan:
                X[bad] = np.nan
            outs.append(ds.prefill(X, pos0).copy())
        finally:
            ds.close()
    assert np.array_equal(outs[0][:bad].view(np.uint16), outs[1][:bad].view(np.uint16))
    assert not np.isfinite(outs[1][bad:].astype(np.float32)).all(axis=1).any()


@pytest.mark.parametrize("shape,pos0", [
    (_shape(512, 64, 2048, 16, 1), 300), (_shape(512, 64, 2048, 16, 1), 901), (_shape(1280, 80, 2560, 20, 1), 1333), (_shape(2048, 128, 2048, 32, 1), 1260),
])
def test_group_behind_an_infinite_v_element(shape, pos0):
    import paper_2604_23553_amd as cf
    from paper_2604_23553_amd.harness import DeviceStack
    T, h = 8, shape.hidden
    assert groups(shape, pos0, T, T)[0][0] == (pos0 > 800)
    print(f"[case] group behind an infinite V {shape.name}", flush=True)
    K, V = synth.kv_cache(shape, 49, 0, pos0, pos0 + T, T)
    V[0, 1, pos0 // 2, 3] = np.inf
    with cf.profile_build():
        ds = DeviceStack(shape, pos0 + T, T, 1)
        try:
            ds.load_layer(0, synth.layer_weights(shape, 49, 0))
            ds.load_kv(0, K, V, pos0)
            ds.prefill(synth.x_input(shape, 49, T), pos0)
            o = ds.tap(3, T * h).reshape(T, h)
        finally:
            ds.close()
    at = shape.head_dim + 3
    assert (o[:, at] == np.inf).all()
    assert np.isfinite(np.delete(o, at, axis=1)).all()


# The statistics come from 16 columns at a time: inputs far from zero mean and with single large values lose nothing
# (the appended rows are held to the bound of fp32 sums, in which the mean's size enters).
@pytest.mark.parametrize("shape", [_shape(640, 80, 2560, 20, 1), _shape(1024, 128, 4096, 32, 1)])
@pytest.mark.parametrize("offset,spike", [(0.0, 0.0), (25.0, 0.0), (-3.0, 900.0)])
def test_layer_inputs_far_from_zero_mean(orc, shape, offset, spike):
    from paper_2604_23553_amd.harness import DeviceStack
    B, S, cap = 5, 9, 10
    print(f"[case] {shape.name} offset {offset} spike {spike}", flush=True)
    lens = np.full(B, S, dtype=np.int32)
    w, (K, V) = synth.layer_weights(shape, 7, 0), synth.kv_cache(shape, 7, 0, lens, cap, B)
    x = (synth.x_input(shape, 7, B).astype(np.float32) + offset)
    x[:, 3::517] += spike
    x = x.astype(np.float16)
    ds = DeviceStack(shape, cap, B, 1)
    try:
        ds.set_options(mode=0)
        ds.load_layer(0, w)
        ds.load_kv(0, K, V, lens)
        ds.set_inputs(x, lens)
        ds.block_decode(0)
        ds.check()
        got = ds.result().copy()
        for b in range(B):
            _, taps = orc.block_decode(shape, w, K[b].copy(), V[b].copy(), S, orc.half_to_real(x[b]), taps=True)
            kg, vg = ds.export_kv(0, b, S, 1)
            assert_appended_rows(kg[:, 0], vg[:, 0], shape, w, orc.half_to_real(x[b]), taps, f"sequence {b}")
            ref = orc.block_decode_f16(shape, w, K[b].copy(), V[b].copy(), S, x[b]).astype(np.float64)
            # (a large input reaches the output as it is: there the step of its size counts, elsewhere the block tolerance)
            assert (np.abs(got[b].astype(np.float64) - ref) <= np.maximum(ulp16(ref), MAX_ABS)).all(), f"sequence {b}"
            if spike == 0.0:
                assert_block_close(got[b], ref, f"sequence {b}")
    finally:
        ds.close()


# A short prompt's products: sets of 1 .. 6 and 8 tokens' eights (7 runs as 8), the last one partly there, with 1, 2, 3, 5 and 8
# tiles; K of the second product in unequal parts; pairs of rows over the ends of items.  Over two layers, every token against the oracle.
@pytest.mark.parametrize("shape,T", [
    (_shape(128, 64, 128, 16), 9), (_shape(384, 128, 896, 0), 64), (_shape(512, 64, 2048, 16), 31), (_shape(512, 64, 2048, 64), 50),
    (_shape(512, 64, 2048, 18), 20), (_shape(640, 80, 2560, 20), 1), (_shape(640, 80, 2560, 20), 48), (_shape(1280, 80, 5120, 20), 17), (_shape(1280, 80, 5120, 20), 64),
    (_shape(1408, 128, 4224, 32), 40), (_shape(2560, 80, 10240, 20), 8), (_shape(2560, 80, 10240, 20), 37),
    (_shape(2560, 80, 10240, 20), 57), (_shape(3072, 64, 12288, 16), 3), (_shape(3072, 128, 12288, 32), 26), (_shape(3072, 128, 12288, 32), 45),
])
def test_short_prompts(orc, shape, T):
    import paper_2604_23553_amd as cf
    from tests.test_gpu_prefill import _check_prompt
    with cf.profile_build():
        assert cf.cfpp_debug_prefill_narrow(cf.Config.from_shape(shape, 16), 128, T)
    _check_prompt(orc, shape, 29, 5, T, 2, 1, then_decode=False, gemm_rows=128, row_check_every=7)


# MLP-down beside the attention of a short prompt: 1 .. 6 sets of tokens, the last one partly there, K in one to eight parts, wavefronts without
# chunks, one and two workgroups to a CU, behind a context that the attention cuts into parts of its own, at the three head sizes.
@pytest.mark.parametrize("shape,pos0,T,downs,workgroups,attention", SHORT)
def test_short_prompts_with_mlp_down_beside_the_attention(orc, shape, pos0, T, downs, workgroups, attention):
    from tests.test_gpu_prefill import _check_prompt
    got = short(shape, pos0, T)
    assert (got[0], got[3], got[2]) == (downs, workgroups, attention)
    _check_prompt(orc, shape, 53, pos0, T, 2, 1, then_decode=False, gemm_rows=128, row_check_every=13)


# The tiled products of few tokens, where the narrow ones do not go: an MLP of more than 128 rows to a CU.
@pytest.mark.parametrize("shape,T", WIDE)
def test_short_prompts_in_tiles(orc, shape, T):
    import paper_2604_23553_amd as cf
    from tests.test_gpu_prefill import _check_prompt
    with cf.profile_build():
        assert cf.cfpp_debug_prefill_narrow(cf.Config.from_shape(shape, 16), 128, T) is None
    _check_prompt(orc, shape, 31, 3, T, 1, 0, then_decode=False, gemm_rows=128, row_check_every=9)


# A sequence on its own (a block at any size, a stack below hidden 2048) takes products of its own, cut alike: rows of 2 .. 128 to a
# workgroup, one row group or eight tiles.  Output and appended rows against the oracle; beside a second sequence the same
# to a rounding of the output (the two paths' values are within fp32 errors of each other, and so are roundings of the same or of
# neighbouring fp16 values, plus what a neighbouring V row moves: see test_gpu_prefill.py).
@pytest.mark.parametrize("shape,S", [
    (_shape(128, 64, 128, 16), 0), (_shape(512, 64, 2048, 16), 128), (_shape(640, 80, 2560, 20), 33), (_shape(1536, 64, 6144, 16), 700),
    (_shape(1792, 128, 7168, 32), 64), (_shape(2560, 80, 10240, 20, 1), 1000), (_shape(4096, 128, 16384, 32, 1), 17),
    (_shape(3072, 64, 12288, 16, 1), 5), (_shape(2048, 64, 2048, 16, 1), 90), (_shape(1920, 80, 15360, 20), 12),
])
def test_a_single_sequence(orc, shape, S):
    from paper_2604_23553_amd.harness import DeviceStack
    print(f"[case] single sequence {shape.name} S={S}", flush=True)
    L, outs = shape.n_layers, []
    ws = [synth.layer_weights(shape, 9, l) for l in range(L)]
    x = synth.x_input(shape, 9, 2)
    for B in (1, 2):
        lens = np.full(B, S, dtype=np.int32)
        kvs = [synth.kv_cache(shape, 9, l, lens, S + 1, B) for l in range(L)]
        ds = DeviceStack(shape, S + 1, B, L)
        try:
            for l in range(L):
                ds.load_layer(l, ws[l])
                ds.load_kv(l, kvs[l][0], kvs[l][1], lens)
            ds.set_inputs(x[:B], lens)
            if L == 1:
                ds.block_decode(0)
            else:
                ds.stack_decode()
            ds.check()
            outs.append(ds.result().copy())
            if B == 1:
                Ks, Vs = [kv[0][0].copy() for kv in kvs], [kv[1][0].copy() for kv in kvs]
                want, _ = orc.stack_decode(shape, ws, Ks, Vs, S, x[0])
                assert_block_close(outs[0][0], want, shape.name)
                check_appended_rows(orc, ds, shape, ws, kvs, S, x[0])
        finally:
            ds.close()
    one, two = (o[0].astype(np.float64) for o in outs)
    step = np.ldexp(1.0, np.frexp(np.maximum(np.abs(one), np.abs(two)).clip(2.0 ** -14))[1] - 11)
    assert (np.abs(one - two) <= 1.001 * step + 2e-3 * L * np.sqrt((two ** 2).mean()) + 2e-5).all()


# Few queries behind a long context: the keys in 2 .. 8 parts, parts of unequal tiles, blocks of queries with unequal tiles, at the
# three head sizes, through narrow and tiled products.
@pytest.mark.parametrize("shape,pos0,T", [
    (_shape(512, 64, 2048, 16, 1), 1500, 1), (_shape(512, 64, 2048, 16, 1), 890, 70), (_shape(640, 80, 2560, 20, 1), 2100, 33),
    (_shape(640, 80, 2560, 20, 1), 1000, 100), (_shape(1024, 128, 4096, 32, 1), 700, 65), (_shape(2560, 80, 2560, 20, 1), 1400, 5),
])
def test_prompt_attention_in_parts(orc, shape, pos0, T):
    from tests.test_gpu_prefill import _check_prompt
    _check_prompt(orc, shape, 37, pos0, T, 1, 0, then_decode=False, gemm_rows=128, row_check_every=11)


# The weights of a query are relative to a score that follows its maximum only when that is 2^4 times it: scores that rise along the
# context in steps below and far above that, fall again, and start with keys that weigh nothing against the later ones; 32, 64 and 128 queries
# to a workgroup, keys whole and in parts, wavefronts that share the keys.  Against the batched path, which keeps the maximum.
@pytest.mark.parametrize("shape,pos0,T", [
    (_shape(512, 64, 2048, 0, 1), 700, 40), (_shape(640, 80, 2560, 0, 1), 900, 100), (_shape(2560, 80, 2560, 0, 1), 650, 800), (_shape(1024, 128, 4096, 0, 1), 500, 70),
    (_shape(2048, 64, 2048, 0, 1), 300, 2050),
])
def test_prompt_attention_with_scores_that_rise(shape, pos0, T):
    from paper_2604_23553_amd.harness import DeviceStack
    print(f"[case] rising scores {shape.name} pos0={pos0} T={T}", flush=True)
    H, d, h, cap = shape.n_heads, shape.head_dim, shape.hidden, pos0 + T
    w = {n: a.copy() for n, a in synth.layer_weights(shape, 59, 0).items()}
    rng = np.random.default_rng(59)
    u = rng.choice([-1.0, 1.0], (H, d))
    rows = np.arange(3 * h).reshape(H, 3, d)
    w["w_qkv"][rows[:, 0].ravel()] *= np.float16(0.05)                     # every query: nearly u
    w["b_qkv"][rows[:, 0].ravel()] = u.ravel().astype(np.float16)
    K, V = synth.kv_cache(shape, 59, 0, pos0, cap, 8)
    level = np.array([0.0, 2.0, 4.5, 9.0, 11.0, 25.0, 18.0, 26.0])[np.minimum(np.arange(pos0) * 8 // pos0, 7)]         # scores, in units of e
    K[0, :, :pos0] = (u[:, None] * (level / np.sqrt(d))[None, :, None] + 0.3 * K[0, :, :pos0].astype(np.float32)).astype(np.float16)
    X = synth.x_input(shape, 61, batch=T)
    outs = []
    for gemm in (False, True):
        ds = DeviceStack(shape, cap, 8, 1)
        try:
            ds.load_layer(0, w)
            ds.load_kv(0, K, V, pos0)
            outs.append((ds.prefill_gemm(X, pos0, rows=-(-T // 128) * 128) if gemm else ds.prefill(X, pos0)).astype(np.float64))
            ds.check()
        finally:
            ds.close()
    want, got = outs
    rms = np.sqrt((want ** 2).mean(axis=1, keepdims=True))
    step = np.ldexp(1.0, np.frexp(np.maximum(np.abs(got), np.abs(want)).clip(2.0 ** -14))[1] - 11)
    assert np.isfinite(got).all() and (np.abs(got - want) <= 1.001 * step + 2e-3 * rms + 2e-5).all()       # (as test_gpu_prefill.py's)
    assert np.linalg.norm(got - want) <= 2.5e-4 * np.linalg.norm(want)


# What such a rise leaves in the weights, against 64 bits: sixteen keys in one tile are `rise` (base 2) above all others, nearly 0, so that the
# outputs are these keys' and carry their scores' errors as they stand.  Queries and rows are their biases (no rotary, zero weights): known to the
# last bit.  Bound: the output's head and remainder, 2^-22 of it and 2^-25; of a key's weight, 2^-22 for its own head and remainder, the exponential and the
# sum, and its score's error, 2^-22 of the sum of its terms' sizes (the query's head and remainder, and the roundings of so small a sum).  A rounding of
# the size of the rise is 2^-24 of it, 7 times that at 30.
@pytest.mark.parametrize("rise", [6, 30, 500])
@pytest.mark.parametrize("shape,pos0,T", [
    (_shape(512, 64, 512, 0, 1), 900, 40), (_shape(640, 80, 640, 0, 1), 700, 100), (_shape(1024, 128, 1024, 0, 1), 500, 30), (_shape(2560, 80, 2560, 0, 1), 512, 800),
    (_shape(2048, 64, 2048, 0, 1), 512, 2050), (_shape(2048, 128, 2048, 0, 1), 512, 200),
])
def test_prompt_attention_after_a_rise_against_64_bits(shape, pos0, T, rise):
    import paper_2604_23553_amd as cf
    from paper_2604_23553_amd.harness import DeviceStack
    print(f"[case] error after a rise of {rise} {shape.name} pos0={pos0} T={T}", flush=True)
    H, d, h, cap, rows = shape.n_heads, shape.head_dim, shape.hidden, pos0 + T, -(-T // 128) * 128
    w = {n: a.copy() for n, a in synth.layer_weights(shape, 59, 0).items()}
    rng, at = np.random.default_rng(59), np.arange(3 * h).reshape(H, 3, d)
    u = rng.choice([-1.0, 1.0], (H, d)).astype(np.float16)
    low = (-u.astype(np.float32) * rise * np.log(2.0) / np.sqrt(d)).astype(np.float16)             # a key `rise` below 0
    for i, bias in ((0, u), (1, low)):
        w["w_qkv"][at[:, i].ravel()] = 0
        w["b_qkv"][at[:, i].ravel()] = bias.ravel()
    K, V = synth.kv_cache(shape, 59, 0, pos0, cap, 1)
    K[0, :, :pos0] = (low[:, None] + 0.3 * K[0, :, :pos0].astype(np.float32)).astype(np.float16)
    K[0, :, 300:316] = (0.3 * rng.standard_normal((H, 16, d))).astype(np.float16)
    with cf.profile_build():
        cfg = cf.Config.from_shape(shape, cap)
        narrow = cf.cfpp_debug_prefill_narrow(cfg, rows, T) is not None
        offsets, halves = cf.cfpp_debug_prefill_scratch(cfg, rows)
        ds = DeviceStack(shape, cap, 1, 1)
        try:
            ds.load_layer(0, w)
            ds.load_kv(0, K, V, pos0)
            x = torch.from_numpy(synth.x_input(shape, 61, batch=T)).to(ds.dev)
            out, nbytes = torch.zeros_like(x), cf.cfpp_prefill_scratch_bytes(ds.cfg, rows)
            scratch = torch.empty(nbytes, dtype=torch.uint8, device=ds.dev)
            torch.cuda.synchronize()
            cf.cfpp_stack_prefill_gemm(ds.ctx, ds.packed, ds.kv, x, pos0, T, 0, out, scratch, nbytes, rows, ds.s)
            ds.check()
            k, v = (a.astype(np.float64) for a in ds.export_kv(0, 0, 0, cap))
            planes = scratch[offsets[3]:].view(torch.float16)[:rows * halves[0]].cpu().numpy().astype(np.float64)
        finally:
            ds.close()
    if narrow:      # sets of 8 tokens, 32 columns at a time: four times 8 columns of heads [token][8], then of remainders
        o = planes[:-(-T // 8) * h * 16].reshape(-1, h // 32, 4, 2, 8, 8).sum(axis=3).transpose(0, 3, 1, 2, 4).reshape(-1, H, d)[:T]
    else:           # rows of 32 heads, then their 32 remainders
        o = planes.reshape(rows, -1)[:T, :2 * h].reshape(T, h // 32, 2, 32).sum(axis=2).reshape(T, H, d)
    q, worst = u.astype(np.float64), 0.0
    for n in range(0, H, max(1, H // 4)):
        s, terms = k[n] @ q[n] / np.sqrt(d), np.abs(k[n]) @ np.abs(q[n]) / np.sqrt(d)
        e = np.exp(s - s.max())
        for t in list(range(0, T, max(1, T // 40))) + [T - 1]:
            p = e[:pos0 + t + 1] / e[:pos0 + t + 1].sum()
            want = p @ v[n, :pos0 + t + 1]
            bound = 2.0 ** -25 + 2.0 ** -22 * np.abs(want) + 2.0 ** -22 * ((p * (1 + terms[:pos0 + t + 1])) @ np.abs(v[n, :pos0 + t + 1]))
            worst = max(worst, (np.abs(o[t, n] - want) / bound).max())
    print(f"  most of the bound {worst:.2f}")
    assert worst <= 1.0


@pytest.mark.parametrize("kind", ["overflow", "nan"])
@pytest.mark.parametrize("shape,pos0,T,bad", [
    (_shape(512, 64, 2048, 16), 1200, 64, 31), (_shape(640, 80, 2560, 20), 1210, 37, 36), (_shape(1024, 128, 4096, 32), 640, 100, 63),
])
def test_prompt_attention_in_parts_ahead_of_a_token_that_is_not_finite(shape, pos0, T, bad, kind):
    from tests.test_gpu_nonfinite import test_prompt_tokens_ahead_of_one_that_is_not_finite as check
    check(shape, pos0, T, bad, kind)


# The tiles of passes of 65 .. 1024 tokens, over two layers, against the batched projections (as the plans of all passes are).
@pytest.mark.parametrize("shape,T,first,second", MIDDLE)
def test_middle_tiles_over_two_layers(shape, T, first, second):
    import paper_2604_23553_amd as cf
    from tests.test_gpu_prefill import test_gemm_plans_over_two_layers as check
    cfg, rows = cf.Config.from_shape(shape, 3 + T), -(-T // 128) * 128
    with cf.profile_build():
        base, got = cf.cfpp_debug_prefill_plan(cfg, rows, T)[0], cf.cfpp_debug_prefill_tiles(cfg, rows, T)[0]
    assert got == (first or base[0], second or base[1])
    check(shape, T, *got)


# Long passes: the first product with 256 x 320 tiles and as two launches, over two layers (as above).
@pytest.mark.parametrize("shape,T,tile,second", LONG)
def test_long_passes_over_two_layers(shape, T, tile, second):
    from tests.prefill_plans import taken
    from tests.test_gpu_prefill import test_gemm_plans_over_two_layers as check
    got, _ = first_product(shape, T)
    assert (got[0], got[2]) == (tile, second)
    check(shape, T, *taken(shape, T)[0])


# The launch option names the workgroups of the first product: eight tiles of rows to each of the fewest, two rows to each of
# the most.  One workgroup fewer and there is no such cut: a prompt is refused, sequences run one after the other.
@pytest.mark.parametrize("grid", [34, 35, 100, 1024])
def test_explicit_grids(orc, grid):
    from paper_2604_23553_amd import CfppError
    from tests.test_gpu_stack import build_stack, oracle_stack
    shape, lens = _shape(640, 80, 2560, 20), np.array([5, 6, 7], dtype=np.int32)
    print(f"[case] batched path, grid {grid}", flush=True)
    ds, ws, kvs = build_stack(shape, 61, lens, 12, batch=3)
    try:
        ds.set_options(mode=0, grid=grid)
        x = synth.x_input(shape, 61, 3)
        ds.set_inputs(x, lens)
        ds.stack_decode()
        ds.check()
        for b in range(3):
            assert_block_close(ds.result()[b], oracle_stack(orc, shape, ws, kvs, lens[b], x[b], b)[0], f"sequence {b}")
        if grid < 35:
            with pytest.raises(CfppError) as e:
                ds.prefill(x, 0)
            assert e.value.status == -2
        else:
            assert_block_close(ds.prefill(x[:1], 5), oracle_stack(orc, shape, ws, kvs, 5, x[0])[0], "prompt")
    finally:
        ds.close()
