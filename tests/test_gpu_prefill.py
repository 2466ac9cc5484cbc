"""GPU parity of prompt processing (cfpp_stack_prefill) against the CPU oracle,
through the C ABI: every token's output, the rows appended to every layer's
cache, and a decode step that continues behind the prompt."""
import numpy as np
import pytest

import synth
from tests.parity import assert_appended_rows, assert_block_close, errors
from tests.prefill_plans import PLANS, taken

pytestmark = pytest.mark.gpu

TINY_STACK = synth.ModelShape(512, 8, 64, 16, 2048, n_layers=4, name="neox-h512-x4")


def _build(shape, seed, pos0, cap, max_batch):
    from paper_2604_23553_amd.harness import DeviceStack
    L = shape.n_layers
    ds = DeviceStack(shape, cap, max_batch, L)
    ws = [synth.layer_weights(shape, seed, l) for l in range(L)]
    kvs = [synth.kv_cache(shape, seed, l, pos0, cap, max_batch) for l in range(L)]
    for l in range(L):
        ds.load_layer(l, ws[l])
        ds.load_kv(l, kvs[l][0], kvs[l][1], pos0)
    return ds, ws, kvs


def _check_prompt(orc, shape, seed, pos0, T, max_batch, b=0, then_decode=True, gemm_rows=0, row_check_every=1):
    cap = pos0 + T + 2
    print(f"[case] prefill shape={shape.name} seed={seed} pos0={pos0} T={T} max_batch={max_batch} b={b} gemm_rows={gemm_rows}", flush=True)
    ds, ws, kvs = _build(shape, seed, pos0, cap, max_batch)
    try:
        ds.set_options(mode=0)
        X = synth.x_input(shape, seed + 1, batch=T)
        got = ds.prefill_gemm(X, pos0, b, gemm_rows) if gemm_rows else ds.prefill(X, pos0, b)
        ds.check()
        Ks = [kv[0][b].copy() for kv in kvs]
        Vs = [kv[1][b].copy() for kv in kvs]
        want16, _ = orc.prefill(shape, ws, Ks, Vs, pos0, X)
        for t in range(T):
            assert_block_close(got[t], want16[t], f"token {t}")
        # rows appended to every layer's cache of sequence b; nothing else of the cache touched
        for l in range(shape.n_layers):
            kg, vg = ds.export_kv(l, b, 0, cap)
            if l == 0:
                # the first layer reads each token's own input row, the same bits on both sides: its
                # rows must be correct roundings of the oracle's unrounded values
                for t in range(0, T, row_check_every):
                    _, taps = orc.block_decode(shape, ws[0], kvs[0][0][b].copy(), kvs[0][1][b].copy(), pos0 + t,
                                               orc.half_to_real(X[t]), taps=True)
                    assert_appended_rows(kg[:, pos0 + t], vg[:, pos0 + t], shape, ws[0], orc.half_to_real(X[t]), taps,
                                         f"token {t} layer 0")
            else:   # deeper layers see an input that already carries the earlier layers' rounding
                for g_, w_ in ((kg, Ks[l]), (vg, Vs[l])):
                    e = errors(g_[:, pos0:pos0 + T], w_[:, pos0:pos0 + T])
                    assert e[0] <= 2e-2 and e[1] <= 5e-3, f"appended rows, layer {l}: {e}"
            assert np.array_equal(np.ascontiguousarray(kg[:, :pos0]).view(np.uint16),
                                  np.ascontiguousarray(kvs[l][0][b][:, :pos0]).view(np.uint16))
            assert np.isnan(kg[:, pos0 + T:].astype(np.float32)).all() and np.isnan(vg[:, pos0 + T:].astype(np.float32)).all()
            for other in range(max_batch):
                if other != b:
                    ko, _ = ds.export_kv(l, other, 0, cap)
                    assert np.isnan(ko[:, pos0:].astype(np.float32)).all(), "another sequence's cache was written"
        if then_decode and b == 0:
            # one decode step behind the prompt reads what the prompt left in the caches
            x1 = synth.x_input(shape, seed + 2)
            ds.set_inputs(x1, pos0 + T)
            ds.stack_decode()
            ds.check()
            ref16, _ = orc.stack_decode(shape, ws, Ks, Vs, pos0 + T, x1[0])
            assert_block_close(ds.result()[0], ref16, "decode step behind the prompt")
    finally:
        ds.close()


@pytest.mark.parametrize("pos0,T,max_batch,b", [
    (5, 19, 8, 0),        # groups of 8, 8 and 3 behind five cached positions
    (0, 7, 3, 0),         # groups of 3, 3 and 1 from an empty cache
    (3, 9, 8, 2),         # into the cache of the third sequence
    (0, 1, 8, 0),         # a single token
])
def test_prompt_through_the_tiny_stack(orc, pos0, T, max_batch, b):
    _check_prompt(orc, TINY_STACK, 17, pos0, T, max_batch, b)


def test_prompt_at_the_2_8b_shape(orc):
    shape = synth.ModelShape(2560, 32, 80, 20, 10240, n_layers=2, name="pythia-2.8b-x2")
    _check_prompt(orc, shape, 23, 100, 11, 8)


# The same prompts through the prompt-sized kernels (cfpp_stack_prefill_gemm): two products on the
# matrix cores, one causal-attention launch and the LayerNorm's per layer and pass.
@pytest.mark.parametrize("pos0,T,max_batch,b,rows", [
    (5, 19, 8, 0, 128),       # one pass, most of its tile padding
    (0, 7, 3, 0, 128),        # from an empty cache
    (3, 9, 8, 2, 256),        # into the cache of the third sequence
    (0, 1, 8, 0, 128),        # a single token
    (2, 150, 2, 1, 128),      # two passes (128 + 22): the second attends over the first one's rows
    (0, 200, 1, 0, 256),      # several key tiles and query blocks, ragged at both ends
])
def test_prompt_through_the_tiny_stack_with_the_gemm_kernels(orc, pos0, T, max_batch, b, rows):
    _check_prompt(orc, TINY_STACK, 19, pos0, T, max_batch, b, gemm_rows=rows)


def test_prompt_at_the_2_8b_shape_with_the_gemm_kernels(orc):
    shape = synth.ModelShape(2560, 32, 80, 20, 10240, n_layers=2, name="pythia-2.8b-x2")
    _check_prompt(orc, shape, 29, 60, 70, 1, gemm_rows=128)


def test_gemm_prompt_with_head_dim_128_and_tanh_gelu(orc):
    # the third head size of the attention launch (two dimensions per lane), with the other GELU reading
    shape = synth.ModelShape(1024, 8, 128, 32, 4096, n_layers=2, flags=synth.FLAG_TANH_GELU, name="neox-h1024-d128-x2")
    _check_prompt(orc, shape, 31, 7, 90, 1, gemm_rows=128)


# The cases above are small enough that products split K (few tiles) and the parts meet in k_pf_reduce
# and k_pf_row.  These two are long enough for a first product that is not split (in tiles of 64 x 128 and of
# 128 x 320; the second one's parts are 5 and 4), at a head size that does not
# divide the tiles (heads cut by tile edges) and a rotated part that is not a multiple of 8 dimensions.
# Layer-0 rows are held to the rounding bound for every 7th token.


def test_gemm_prompt_long_enough_for_unsplit_products(orc):
    shape = synth.ModelShape(1280, 16, 80, 20, 5120, n_layers=1, name="neox-h1280-x1")
    _check_prompt(orc, shape, 37, 9, 600, 1, gemm_rows=640, row_check_every=7)


def test_gemm_prompt_long_enough_for_128_token_tiles(orc):
    shape = synth.ModelShape(1280, 16, 80, 20, 5120, n_layers=2, name="neox-h1280-x2")
    _check_prompt(orc, shape, 41, 0, 2200, 1, gemm_rows=2304, row_check_every=7)


# Long passes at head sizes 64 and 128 that end inside a query block and inside a key tile.
def test_gemm_prompt_wide_attention_head_dim_64(orc):
    shape = synth.ModelShape(512, 8, 64, 16, 2048, n_layers=2, name="neox-h512-x2")
    _check_prompt(orc, shape, 43, 3, 1100, 1, gemm_rows=1152, row_check_every=7)


def test_gemm_prompt_wide_attention_head_dim_128(orc):
    shape = synth.ModelShape(1024, 8, 128, 32, 4096, n_layers=1, flags=synth.FLAG_TANH_GELU, name="neox-h1024-d128-x1")
    _check_prompt(orc, shape, 47, 0, 1030, 1, gemm_rows=1152, row_check_every=7)


# Edges of the GEMM's tiles (token counts around multiples of 64, 128 and 256) and of the attention's: against the path
# through the batched projections, which the cases above hold to the oracle.  Both sides
# round the same fp32 values to fp16 once, so an element differs by one step of its size at most, plus the drift of
# the appended rows' own roundings (2e-3 of the row's root mean square covers it: a step of one V row in a mean of
# two rows or more).
@pytest.mark.parametrize("shape,pos0,T", [
    (synth.ModelShape(2560, 32, 80, 20, 10240, name="pythia-2.8b-block"), 3, T) for T in (1, 31, 32, 33, 64, 65, 129, 191, 257, 515, 701, 2049, 4095)
] + [
    (synth.ModelShape(640, 8, 80, 20, 2560, name="d80-h640"), 0, 333),          # features not a multiple of the wide tiles
    (synth.ModelShape(128, 2, 64, 64, 128, name="d64-h128"), 5, 20),
    (synth.ModelShape(4096, 32, 128, 32, 16384, name="pythia-6.9b-block"), 0, 24),
    (synth.ModelShape(128, 2, 64, 64, 128, name="d64-h128"), 1, 130),           # the smallest K: fewer steps than stages
    (synth.ModelShape(1536, 24, 64, 16, 6144, name="d64-h1536"), 2, 1000),
    (synth.ModelShape(4096, 32, 128, 32, 16384, name="pythia-6.9b-block"), 1, 1531),
    # the attention's three splits of a workgroup over queries and keys, at every head size, behind cached positions
    (synth.ModelShape(512, 8, 64, 16, 2048, name="neox-h512"), 259, 95),
    (synth.ModelShape(2048, 32, 64, 16, 2048, name="d64-h2048"), 31, 801),
    (synth.ModelShape(2048, 32, 64, 16, 2048, name="d64-h2048"), 0, 2050),
    (synth.ModelShape(1024, 8, 128, 32, 4096, name="d128-h1024"), 1000, 33),
    # a rotated part that ends between the two pairs of a lane's four features (not a multiple of four dimensions)
    (synth.ModelShape(512, 8, 64, 18, 2048, name="neox-h512-r18"), 5, 150),
    (synth.ModelShape(640, 8, 80, 22, 2560, name="d80-h640-r22"), 2, 1100),
    # a group of 8 whose heads are 16 pieces each in the batched attention
    (synth.ModelShape(1024, 8, 128, 32, 4096, name="d128-h1024"), 8000, 8),
])
def test_gemm_tiles_against_the_batched_projections(shape, pos0, T):
    import torch
    import synth.device as sdev
    from paper_2604_23553_amd.harness import DeviceStack
    print(f"[case] gemm tiles shape={shape.name} T={T}", flush=True)
    cap = pos0 + T + 3
    ds = DeviceStack(shape, cap, 8, 1)
    try:
        ds.load_layer_device(0, sdev.layer_tensors(shape, 5, 0, ds.dev))
        sdev.fill_kv(ds.kv[0], 5, 0)
        start = ds.kv[0].clone()
        X = synth.x_input(shape, 6, batch=T)
        want = ds.prefill(X, pos0).astype(np.float64)
        kw, vw = ds.export_kv(0, 0, pos0, T)
        ds.kv[0].copy_(start)
        torch.cuda.synchronize()
        got = ds.prefill_gemm(X, pos0, rows=(T + 127) // 128 * 128).astype(np.float64)
        kg, vg = ds.export_kv(0, 0, pos0, T)
        ds.check()
        rms = np.sqrt((want ** 2).mean(axis=1, keepdims=True))
        for g, w, scale in ((got, want, rms), (kg, kw, 0.0), (vg, vw, 0.0)):
            g, w = g.astype(np.float64), w.astype(np.float64)
            assert np.isfinite(g).all()
            step = np.ldexp(1.0, np.frexp(np.maximum(np.abs(g), np.abs(w)).clip(2.0 ** -14))[1] - 11)
            # K and V rows near zero: the fp32 sums behind them differ by their own rounding, 2e-6 of the terms
            assert (np.abs(g - w) <= 1.001 * step + 2e-3 * scale + 2e-5).all(), float((np.abs(g - w) / (step + 2e-3 * scale + 2e-5)).max())
            assert np.linalg.norm(g - w) <= 2.5e-4 * np.linalg.norm(w)
        kv, st = ds.kv[0].view(torch.float16), start.view(torch.float16)
        d, H = shape.head_dim, shape.n_heads
        v, s = (t.view(2, 8, H, d // 16, cap, 16) for t in (kv, st))
        assert torch.equal(v[:, :, :, :, :pos0], s[:, :, :, :, :pos0]) and torch.equal(v[:, :, :, :, pos0 + T:], s[:, :, :, :, pos0 + T:])
        assert torch.equal(v[:, 1:], s[:, 1:])
    finally:
        ds.close()


# Every kind of tile, with K split and whole, that a plan takes for either product, each over two layers, so that what a
# pass hands to the next layer (parts added on the way, or an unsplit result and a launch of its own) is used.  The bounds
# are those above, per layer: the second layer's input carries the first's differences, and so do its K and V rows.
@pytest.mark.parametrize("shape,T,first,second", PLANS)
def test_gemm_plans_over_two_layers(shape, T, first, second):
    import torch
    import synth.device as sdev
    from paper_2604_23553_amd.harness import DeviceStack
    rows, pos0 = (T + 127) // 128 * 128, 3
    assert taken(shape, T)[0] == (first, second)
    print(f"[case] gemm plan shape={shape.name} T={T}", flush=True)
    ds = DeviceStack(shape, pos0 + T, 8, 2)
    try:
        for l in range(2):
            ds.load_layer_device(l, sdev.layer_tensors(shape, 5, l, ds.dev))
            sdev.fill_kv(ds.kv[l], 5, l)
        X = synth.x_input(shape, 6, batch=T)
        want = [ds.prefill(X, pos0)] + [a for l in range(2) for a in ds.export_kv(l, 0, pos0, T)]
        for l in range(2):
            sdev.fill_kv(ds.kv[l], 5, l)
        torch.cuda.synchronize()
        got = [ds.prefill_gemm(X, pos0, rows=rows)] + [a for l in range(2) for a in ds.export_kv(l, 0, pos0, T)]
        ds.check()
        for g, w, layers in zip(got, want, (2, 0, 0, 1, 1)):       # layers in front of the values
            g, w = g.astype(np.float64), w.astype(np.float64)
            assert np.isfinite(g).all()
            rms = np.sqrt((w ** 2).mean(axis=-1, keepdims=True))
            step = np.ldexp(1.0, np.frexp(np.maximum(np.abs(g), np.abs(w)).clip(2.0 ** -14))[1] - 11)
            bound = 1.001 * step + 2e-3 * layers * rms + 2e-5
            assert (np.abs(g - w) <= bound).all(), float((np.abs(g - w) / bound).max())
            assert np.linalg.norm(g - w) <= 2.5e-4 * max(layers, 1) * np.linalg.norm(w)
    finally:
        ds.close()


# What passes between a layer's kernels as head + remainder, and the attention, against 64 bits: a value whose head and
# remainder come from two roundings is off by up to 2^-11, which the fp16 output hides.  Sizes whose second product keeps
# K whole (the queries stay in the scratch), with 32, 64 and 128 queries to a workgroup; the scores reach 10 and more.
@pytest.mark.parametrize("shape,T", [
    (synth.ModelShape(512, 8, 64, 16, 2048, n_layers=1, name="d64-h512"), 2700),
    (synth.ModelShape(768, 12, 64, 16, 3072, n_layers=1, name="d64-h768"), 2300),
    (synth.ModelShape(2560, 32, 80, 20, 10240, n_layers=1, name="d80-h2560"), 3100),
    (synth.ModelShape(4096, 32, 128, 32, 16384, n_layers=1, name="d128-h4096"), 2600),
])
def test_intermediates_of_a_pass_against_64_bits(shape, T):
    import math
    import torch
    import paper_2604_23553_amd as cf
    import synth.device as sdev
    from paper_2604_23553_amd.harness import DeviceStack
    print(f"[case] intermediates shape={shape.name} T={T}", flush=True)
    h, f, H, d = shape.hidden, shape.ffn, shape.n_heads, shape.head_dim
    rows = (T + 127) // 128 * 128
    with cf.profile_build():
        cfg = cf.Config.from_shape(shape, T)
        assert cf.cfpp_debug_prefill_plan(cfg, rows, T)[0][1][3] == 1
        at, halves = cf.cfpp_debug_prefill_scratch(cfg, rows)
    ds = DeviceStack(shape, T, 1, 1)
    try:
        w = sdev.layer_tensors(shape, 5, 0, ds.dev)
        w["w_qkv"] *= 2
        ds.load_layer_device(0, w)
        x = torch.from_numpy(synth.x_input(shape, 6, batch=T)).to(ds.dev)
        out = torch.zeros_like(x)
        nbytes = cf.cfpp_prefill_scratch_bytes(ds.cfg, rows)
        sc = torch.empty(nbytes, dtype=torch.uint8, device=ds.dev)
        torch.cuda.synchronize()
        cf.cfpp_stack_prefill_gemm(ds.ctx, ds.packed, ds.kv, x, 0, T, 0, out, sc, nbytes, rows, ds.s)
        ds.check()
        k, v = (torch.from_numpy(a).to(ds.dev).double() for a in ds.export_kv(0, 0, 0, T))

        def planes(i, width, stride):
            t = sc[at[i]:at[i] + rows * stride * 2].view(torch.float16).view(rows, stride)[:T, :2 * width]
            return t.reshape(T, width // 32, 2, 32).double().sum(2).reshape(T, width)

        xd = x.double()
        for i, g in ((0, "ln1_g"), (1, "ln2_g")):          # one rounding to 2^-22, or to a step of the smallest fp16
            want = xd * w[g].double()
            assert ((planes(i, h, halves[0]) - want).abs() <= want.abs() * 2.0 ** -21 + 2.0 ** -24).all(), g
        # GELU(up): an fp32 sum of h products (64 x its rounding), then as above
        mu = xd.mean(1, keepdim=True)
        y = (xd - mu) / torch.sqrt(((xd - mu) ** 2).mean(1, keepdim=True) + shape.ln_eps) * w["ln2_g"].double() + w["ln2_b"].double()
        m = planes(4, f, halves[1])
        for r in range(0, T, 512):
            z = y[r:r + 512] @ w["w_up"].double().t().contiguous() + w["b_up"].double()
            want = 0.5 * z * torch.special.erfc(-z / math.sqrt(2.0))
            assert ((m[r:r + 512] - want).abs() <= 64 * 2.0 ** -24 * (1.0 + z.abs())).all(), "GELU(up)"
        # attention from the queries and the cache as they stand: a score is an fp32 sum over d / 16 steps (4 x the rounding of
        # its terms' absolute sum, and of the two planes'), a weight the exponential of it, the sums over keys 32 x a rounding;
        # a weight's remainder is rounded to half a step of the smallest fp16 where the largest weight is 1
        q, o = sc[at[2]:at[2] + rows * h * 4].view(torch.float32).view(rows, h)[:T].double(), planes(3, h, halves[0])
        worst = 0.0
        for n in range(0, H, max(1, H // 8)):
            for r in range(0, T, 1024):
                s = (q[r:r + 1024, n * d:(n + 1) * d] @ k[n].t().contiguous()) / math.sqrt(d)
                s.masked_fill_(torch.arange(T, device=ds.dev)[None] > torch.arange(r, min(r + 1024, T), device=ds.dev)[:, None], -math.inf)
                p = torch.softmax(s, 1)
                A = (q[r:r + 1024, n * d:(n + 1) * d].abs() @ k[n].abs().t().contiguous()).masked_fill_(s == -math.inf, 0.0) / math.sqrt(d)
                e = (o[r:r + 1024, n * d:(n + 1) * d] - p @ v[n]).abs()
                bound = 2.0 ** -24 * (32.0 + 4.0 * A.max(1, keepdim=True).values) * (p @ v[n].abs())
                bound += 2.0 ** -25 * p.max(1, keepdim=True).values * v[n].abs().cumsum(0)[r:r + 1024]
                worst = max(worst, float((e / bound).max()))
                assert (e <= bound).all(), f"head {n} rows {r} ..: {int((e > bound).any(1).sum())} queries, up to {float((e / bound).max()):.1f} x"
        print(f"[result] attention {shape.name}: {worst:.2f} of the bound", flush=True)
    finally:
        ds.close()


# The epilogues' GELU loses nothing against the forms with the device library's functions: over what the MLP-up
# products of the supported sizes give (0.02 sqrt(hidden) or so: N(0, 0.2) .. N(0, 1.3)) and over the whole curve its distance
# from 64 bits is no larger, and infinities and NaN come out the same.
@pytest.mark.parametrize("flags", [0, synth.FLAG_TANH_GELU])
def test_gelu_of_the_epilogues(flags):
    import math
    import torch
    import paper_2604_23553_amd as cf
    n = 2_000_000
    g = torch.Generator(device="cuda")
    g.manual_seed(3)
    with cf.profile_build():
        for std in (0.1, 0.2, 0.3, 0.45, 0.6, 1.0, 1.3, 3.0, 0.0):
            z = torch.randn(n, generator=g, device="cuda") * std if std else torch.linspace(-9.0, 9.0, n, device="cuda")
            new, old = torch.empty_like(z), torch.empty_like(z)
            torch.cuda.synchronize()
            cf.cfpp_debug_gelu(z, new, old, n, flags)
            torch.cuda.synchronize()
            d = z.double()
            want = (d / (1.0 + torch.exp(-2.0 * math.sqrt(2.0 / math.pi) * (d + 0.044715 * d ** 3))) if flags
                    else 0.5 * d * torch.special.erfc(-d / math.sqrt(2.0)))
            en, eo = (new.double() - want), (old.double() - want)
            mn, mo = float(en.abs().max()), float(eo.abs().max())
            rn, ro = float(en.norm() / want.norm()), float(eo.norm() / want.norm())
            print(f"[result] gelu flags {flags} std {std}: largest {mo:.3e} -> {mn:.3e}, relative {ro:.3e} -> {rn:.3e}", flush=True)
            # (the largest of two million errors moves by a rounding step of its value from seed to seed, the norm does not)
            assert rn <= ro and mn <= 1.25 * mo
        z = torch.tensor([math.inf, -math.inf, math.nan, 0.0, -0.0, 1e30, -1e30, 1.0, -1.0], device="cuda")
        new, old = torch.empty_like(z), torch.empty_like(z)
        torch.cuda.synchronize()
        cf.cfpp_debug_gelu(z, new, old, z.numel(), flags)
        torch.cuda.synchronize()
        assert torch.allclose(new, old, rtol=3e-7, atol=0.0, equal_nan=True)


def test_gemm_prompt_refuses_the_sequential_form():
    import dataclasses
    from paper_2604_23553_amd import CfppError
    shape = dataclasses.replace(TINY_STACK, flags=synth.FLAG_SEQUENTIAL_RESIDUAL)
    ds, ws, kvs = _build(shape, 1, 0, 12, 1)
    try:
        with pytest.raises(CfppError) as e:
            ds.prefill_gemm(synth.x_input(shape, 2, batch=4), 0, rows=128)
        assert e.value.status == -2
    finally:
        ds.close()


def test_gemm_prompt_requests_that_are_refused():
    import torch
    from paper_2604_23553_amd import CfppError, binding as B
    ds, ws, kvs = _build(TINY_STACK, 1, 0, 12, 8)
    try:
        X = synth.x_input(TINY_STACK, 2, batch=4)
        assert B.cfpp_prefill_scratch_bytes(ds.cfg, 100) == 0 and B.cfpp_prefill_scratch_bytes(ds.cfg, 8192) == 0
        with pytest.raises(CfppError) as e:
            ds.prefill_gemm(X, 9, rows=128)               # positions 9..12 of a cache of 12
        assert e.value.status == -1
        need = B.cfpp_prefill_scratch_bytes(ds.cfg, 128)
        xd = torch.from_numpy(X).to(ds.dev)
        od = torch.zeros_like(xd)
        small = torch.empty(need - 256, dtype=torch.uint8, device=ds.dev)
        with pytest.raises(CfppError) as e:
            B.cfpp_stack_prefill_gemm(ds.ctx, ds.packed, ds.kv, xd, 0, 4, 0, od, small, need - 256, 128, ds.s)
        assert e.value.status == -3                       # scratch too small
        with pytest.raises(CfppError) as e:
            B.cfpp_stack_prefill_gemm(ds.ctx, ds.packed, ds.kv, xd, 0, 4, 0, od, small, need, 100, ds.s)
        assert e.value.status == -1                       # rows not a multiple of 128
        ds.prefill_gemm(X, 8, rows=128)                   # the last four rows fit
        ds.check()
    finally:
        ds.close()


def test_prompt_requests_that_are_refused():
    from paper_2604_23553_amd import CfppError
    ds, ws, kvs = _build(TINY_STACK, 1, 0, 12, 8)
    try:
        X = synth.x_input(TINY_STACK, 2, batch=4)
        ds.set_options(mode=2)
        with pytest.raises(CfppError) as e:
            ds.prefill(X, 0)
        assert e.value.status == -2                       # launch mode 0 only
        ds.set_options(mode=0)
        with pytest.raises(CfppError) as e:
            ds.prefill(X, 9)                              # positions 9..12 of a cache of 12
        assert e.value.status == -1
        with pytest.raises(CfppError) as e:
            ds.prefill(X, 0, b=8)                         # no such sequence
        assert e.value.status == -1
        ds.prefill(X, 8)                                  # the last four rows fit
        ds.check()
    finally:
        ds.close()
