"""Values that are not finite stay where they belong: a V element that overflows fp16 makes that dimension of what
attends to it infinite and nothing else."""
import numpy as np
import pytest

import synth

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
