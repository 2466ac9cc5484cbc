"""Passes of the prompt-sized tiled products and the plan that each runs in the end: (tokens, features, K step, parts of K) of
the first product (QKV, MLP-up) and of the second (output projection, MLP-down).  Together with WIDE and with
prefill_middle.py's they take every kind of tile of either product, with K split and whole, that any pass runs on 256 CUs (held
on the CPU); the GPU runs each over two layers."""
import synth


def _shape(h, d, f, r):
    return synth.ModelShape(h, h // d, d, r, f, n_layers=2, name=f"d{d}-h{h}-f{f}-x2")


H128, H512, H1024 = _shape(128, 64, 128, 16), _shape(512, 64, 2048, 16), _shape(1024, 128, 4096, 32)
H2560, H4096 = _shape(2560, 80, 10240, 20), _shape(4096, 128, 16384, 32)
H1280, H1536, H3072, H3200 = _shape(1280, 80, 5120, 20), _shape(1536, 64, 6144, 16), _shape(3072, 128, 3072, 32), _shape(3200, 80, 12800, 20)

PLANS = [
    (H512, 100, (64, 128, 32, 4), (64, 128, 32, 16)),
    (H4096, 50, (64, 128, 64, 1), (64, 128, 64, 8)),
    (H1280, 150, (64, 128, 64, 1), (64, 128, 64, 8)),
    (H1024, 100, (64, 128, 64, 2), (64, 128, 64, 16)),
    (H3200, 55, (64, 256, 64, 2), (64, 128, 64, 10)),
    (H1536, 88, (128, 128, 32, 3), (64, 128, 64, 10)),
    (H512, 2700, (64, 128, 32, 1), (64, 128, 64, 1)),
    (H128, 2600, (64, 128, 32, 1), (64, 128, 32, 1)),
    (H2560, 3100, (256, 256, 32, 1), (128, 128, 32, 1)),
    (H2560, 1100, (128, 320, 32, 1), (128, 320, 32, 3)),
    (H4096, 2600, (256, 256, 32, 1), (256, 192, 32, 1)),
    (H2560, 2100, (128, 320, 32, 1), (256, 192, 32, 2)),
    (H4096, 3400, (256, 256, 32, 1), (256, 256, 32, 1)),
    (H2560, 1200, (256, 192, 32, 1), (256, 256, 32, 4)),
    (H2560, 1600, (256, 256, 32, 1), (256, 320, 32, 4)),
    (H2560, 515, (128, 128, 32, 1), (128, 128, 32, 5)),
    (H2560, 100, (128, 96, 64, 1), (128, 128, 32, 12)),
    (H3072, 3073, (128, 320, 32, 1), (128, 320, 32, 1)),
]

# an MLP so wide that only the tiled products take it, and neither the batched path nor a decode step: against the oracle
WIDE = [(_shape(512, 64, 32768, 16), T) for T in (20, 40, 64)]


def taken(shape, tokens, rows=None, n_cu=256):
    """The plan that a pass runs in the end, and by how many rows its loads pass their operands; None: the narrow products."""
    import paper_2604_23553_amd as cf
    cfg, rows = cf.Config.from_shape(shape, 16), rows or -(-tokens // 128) * 128
    with cf.profile_build():
        return None if cf.cfpp_debug_prefill_narrow(cfg, rows, tokens, n_cu) else cf.cfpp_debug_prefill_tiles(cfg, rows, tokens)


def kinds(plan):
    """(product, tile, K split) of a plan's two products."""
    return {(k, plan[k][:3], plan[k][3] > 1) for k in (0, 1)}
