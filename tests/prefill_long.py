"""Passes of more than 512 tokens and what the first product of each is to run as: the tile, and, where MLP-up is finished by a launch of
its own, that one's tile.  Together with the passes of prefill_plans.py and prefill_middle.py they take every tile that such
a pass runs whole, in the first of two launches and in the second (held on the CPU)."""
from tests.prefill_plans import _shape

LONG = [
    (_shape(512, 64, 4096, 16), 3362, (256, 320), None),
    (_shape(1152, 64, 4608, 16), 1179, (128, 160), None),
    (_shape(1152, 64, 4608, 16), 513, (128, 192), None),
    (_shape(1280, 80, 10240, 20), 3621, (256, 256), (256, 320)),
    (_shape(1536, 128, 12288, 32), 1438, (256, 256), (128, 160)),
    (_shape(1664, 64, 6656, 16), 2067, (256, 320), (128, 192)),
    (_shape(1536, 64, 12288, 0), 2844, (256, 320), (256, 256)),
    (_shape(2688, 128, 10752, 32), 1290, (256, 320), (128, 256)),
    (_shape(2688, 64, 10752, 16), 1549, (128, 256), (256, 256)),
    (_shape(3328, 128, 6656, 32), 1808, (256, 192), (128, 256)),
    (_shape(3840, 80, 7680, 20), 1549, (128, 320), (256, 192)),
]


def first_product(shape, tokens, rows=None):
    """((tile, MLP-up rows of the first launch, tile of the second or None), reach past the weights) of a pass."""
    import paper_2604_23553_amd as cf
    with cf.profile_build():
        return cf.cfpp_debug_prefill_long(cf.Config.from_shape(shape, 16), rows or -(-tokens // 128) * 128, tokens)
