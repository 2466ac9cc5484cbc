"""Values that are not finite stay where they belong: a V element that overflows fp16, or a token that is NaN,
reaches the tokens that attend to it and no earlier one, whatever shares a tile with it."""
import numpy as np
import pytest

import synth
from tests.beside_plans import groups

pytestmark = pytest.mark.gpu

HEAD, DIM = 1, 3          # the V element that overflows


def _overflowing(shape, seed, layer, x):
    """A layer's weights with the V row of (HEAD, DIM) along LayerNorm1(x): 120000 for that token's V, which fp16 does
    not hold, and 120000 / sqrt(hidden) or so for another's."""
    w = {n: a.copy() for n, a in synth.layer_weights(shape, seed, layer).items()}
    x = x.astype(np.float64)
    y = (x - x.mean()) / np.sqrt(x.var() + shape.ln_eps) * w["ln1_g"].astype(np.float64) + w["ln1_b"].astype(np.float64)
    w["w_qkv"][(3 * HEAD + 2) * shape.head_dim + DIM] = (y * (120000.0 / (y @ y))).astype(np.float16)
    return w


# Every way the prompt attention splits a workgroup over queries and keys (32, 64 and 128 queries), at the three head
# sizes: the token in a block's middle, at its first and its last query, behind cached positions and from an empty cache.
@pytest.mark.parametrize("kind", ["overflow", "nan"])
@pytest.mark.parametrize("shape,pos0,T,bad", [
    (synth.ModelShape(512, 8, 64, 16, 2048, n_layers=2, name="neox-h512-x2"), 5, 95, 43),
    (synth.ModelShape(640, 8, 80, 20, 2560, n_layers=2, name="d80-h640-x2"), 0, 64, 63),
    (synth.ModelShape(640, 8, 80, 20, 2560, n_layers=2, name="d80-h640-x2"), 3, 70, 32),
    (synth.ModelShape(1024, 8, 128, 32, 4096, n_layers=2, name="d128-h1024-x2"), 100, 140, 101),
    (synth.ModelShape(2560, 32, 80, 20, 2560, n_layers=1, name="d80-h2560"), 0, 801, 700),
    (synth.ModelShape(2048, 32, 64, 16, 2048, n_layers=1, name="d64-h2048"), 9, 2050, 1300),
])
def test_prompt_tokens_ahead_of_one_that_is_not_finite(shape, pos0, T, bad, kind):
    from paper_2604_23553_amd.harness import DeviceStack
    print(f"[case] nonfinite prompt {shape.name} T={T} bad={bad} {kind}", flush=True)
    X = synth.x_input(shape, 71, batch=T)
    cap = pos0 + T + 1
    ds = DeviceStack(shape, cap, 8, shape.n_layers)
    try:
        for l in range(shape.n_layers):
            ds.load_layer(l, _overflowing(shape, 70, l, X[bad]) if kind == "overflow" and l == 0 else synth.layer_weights(shape, 70, l))
            ds.load_kv(l, *synth.kv_cache(shape, 70, l, pos0, cap, 8), pos0)
        want = ds.prefill(X[:bad], pos0).astype(np.float64)
        assert np.isfinite(want).all()
        if kind == "nan":
            X[bad] = np.nan
        got = ds.prefill_gemm(X, pos0, rows=-(-T // 128) * 128).astype(np.float64)
        ds.check()
        assert not np.isfinite(got[bad:]).all(axis=1).any()
        g = got[:bad]
        assert np.isfinite(g).all(), f"tokens {sorted(set(np.where(~np.isfinite(g))[0]))} are not finite"
        # the bound of the two paths' agreement: one fp16 step of the element, a step of the appended rows (2e-3 of the
        # row's root mean square covers it), which the second layer's attention and products take up once more
        rms = np.sqrt((want ** 2).mean(axis=1, keepdims=True))
        step = np.ldexp(1.0, np.frexp(np.maximum(np.abs(g), np.abs(want)).clip(2.0 ** -14))[1] - 11)
        assert (np.abs(g - want) <= step + 2e-3 * shape.n_layers * rms + 2e-5).all()
        assert np.linalg.norm(g - want) <= 2.5e-4 * shape.n_layers * np.linalg.norm(want)
    finally:
        ds.close()


# A new token whose V overflows in one dimension: that dimension of its own attention output is infinite, the others
# and the other sequences' are finite (contexts that do not fill the last row of positions).
@pytest.mark.parametrize("shape,lens", [
    (synth.ModelShape(512, 8, 64, 16, 2048, n_layers=1, name="neox-h512"), [37, 5, 63, 100]),
    (synth.ModelShape(640, 8, 80, 20, 2560, n_layers=1, name="d80-h640"), [1500, 5, 31]),
    (synth.ModelShape(1024, 8, 128, 32, 4096, n_layers=1, name="d128-h1024"), [20, 16]),
])
def test_batched_step_with_a_v_element_that_overflows(shape, lens):
    import paper_2604_23553_amd as cf
    from paper_2604_23553_amd.harness import DeviceStack
    print(f"[case] nonfinite batch {shape.name} lens={lens}", flush=True)
    B, cap = len(lens), max(lens) + 2
    X = synth.x_input(shape, 73, batch=B)
    with cf.profile_build():
        ds = DeviceStack(shape, cap, B, 1)
        try:
            ds.load_layer(0, _overflowing(shape, 72, 0, X[0]))
            ds.load_kv(0, *synth.kv_cache(shape, 72, 0, np.array(lens), cap, B), np.array(lens))
            ds.set_inputs(X, np.array(lens, dtype=np.int32))
            ds.block_decode(0)
            ds.check()
            o = ds.tap(3, B * shape.hidden).reshape(B, shape.hidden)
        finally:
            ds.close()
    at = HEAD * shape.head_dim + DIM
    assert o[0, at] == np.inf
    o[0, at] = 0.0
    assert np.isfinite(o).all()


def _check_minus_infinity(shape, taps, k, v, lens, what):
    """The attention outputs of one head against 64 bits where some scores are minus infinity: those keys weigh nothing."""
    q, o = taps
    d = shape.head_dim
    for t, n in enumerate(lens):
        with np.errstate(invalid="ignore"):
            s = np.where(np.isinf(k[t][:n]).any(axis=1), -np.inf, k[t][:n] @ q[t] / np.sqrt(d))
        p = np.exp(s - s.max())
        want = (p / p.sum()) @ v[t][:n]
        assert np.isfinite(o[t]).all(), f"{what}: query {t} is not finite"
        assert np.abs(o[t] - want).max() <= 2e-5 * np.abs(v[t][:n]).max(), f"{what}: query {t}"


# A K element that is infinite and meets a query's element of the other sign: that key weighs nothing, wherever it lies - the
# only key that a lane has, a token's own, the first of a group, cached ahead of a group that attends together or of one that does not.
@pytest.mark.parametrize("d,H,lens,bad", [(64, 8, [0, 3, 70], 0), (80, 8, [5], 2), (128, 8, [40, 7], 7), (64, 8, [2000], 1999)])
def test_step_behind_a_key_of_minus_infinity(d, H, lens, bad):
    import paper_2604_23553_amd as cf
    from paper_2604_23553_amd.harness import DeviceStack
    shape = synth.ModelShape(H * d, H, d, 0, H * d, n_layers=1, name=f"d{d}")
    print(f"[case] minus infinity, step {shape.name} {lens}", flush=True)
    B, cap, h = len(lens), max(lens) + 1, H * d
    w = {n: a.copy() for n, a in synth.layer_weights(shape, 75, 0).items()}
    w["w_qkv"][3 * HEAD * d + DIM] = 0
    w["b_qkv"][3 * HEAD * d + DIM] = -1.0                                  # the query's element
    K, V = synth.kv_cache(shape, 75, 0, np.array(lens), cap, B)
    for b, n in enumerate(lens):
        if bad < n:
            K[b, HEAD, bad, DIM] = np.inf
    with cf.profile_build():
        ds = DeviceStack(shape, cap, B, 1)
        try:
            ds.load_layer(0, w)
            ds.load_kv(0, K, V, np.array(lens))
            ds.set_inputs(synth.x_input(shape, 75, B), np.array(lens, dtype=np.int32))
            ds.block_decode(0)
            ds.check()
            q, o = (ds.tap(i, B * h).reshape(B, H, d)[:, HEAD].astype(np.float64) for i in (0, 3))
            kv = [ds.export_kv(0, b, 0, lens[b] + 1) for b in range(B)]
        finally:
            ds.close()
    k, v = ([a[i][HEAD].astype(np.float64) for a in kv] for i in (0, 1))
    _check_minus_infinity(shape, (q, o), k, v, [n + 1 for n in lens], shape.name)


@pytest.mark.parametrize("d,H,pos0,token,cached", [(64, 8, 930, 0, None), (80, 16, 1300, 3, None), (128, 16, 1260, 0, 37), (64, 8, 930, None, 929), (64, 8, 300, 0, 299), (80, 16, 40, 2, 33)])
def test_group_with_a_key_of_minus_infinity(d, H, pos0, token, cached):
    import paper_2604_23553_amd as cf
    from paper_2604_23553_amd.harness import DeviceStack
    T, h = 8, H * d
    shape = synth.ModelShape(h, H, d, 0, h, n_layers=1, name=f"d{d}")
    assert groups(shape, pos0, T, T)[0][0] == (pos0 > 800)
    print(f"[case] minus infinity, group {shape.name} pos0={pos0} token={token}", flush=True)
    x = synth.x_input(shape, 77, T)
    w = {n: a.copy() for n, a in synth.layer_weights(shape, 77, 0).items()}
    w["w_qkv"][3 * HEAD * d + DIM] = 0
    w["b_qkv"][3 * HEAD * d + DIM] = -1.0
    if token is not None:       # the K row of (HEAD, DIM) along LayerNorm1 of that token: 120000 for it, which fp16 does not hold
        row = _overflowing(shape, 77, 0, x[token])["w_qkv"][(3 * HEAD + 2) * d + DIM]
        w["w_qkv"][(3 * HEAD + 1) * d + DIM] = row
    K, V = synth.kv_cache(shape, 77, 0, pos0, pos0 + T, T)
    if cached is not None:
        K[0, HEAD, cached, DIM] = np.inf
    with cf.profile_build():
        ds = DeviceStack(shape, pos0 + T, T, 1)
        try:
            ds.load_layer(0, w)
            ds.load_kv(0, K, V, pos0)
            ds.prefill(x, pos0)
            ds.check()
            q, o = (ds.tap(i, T * h).reshape(T, H, d)[:, HEAD].astype(np.float64) for i in (0, 3))
            k, v = (a[HEAD].astype(np.float64) for a in ds.export_kv(0, 0, 0, pos0 + T))
        finally:
            ds.close()
    if token is not None:
        assert k[pos0 + token, DIM] == np.inf
    _check_minus_infinity(shape, (q, o), [k] * T, [v] * T, [pos0 + t + 1 for t in range(T)], shape.name)
