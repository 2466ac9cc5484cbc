"""What the tests of MLP-down beside the attention, of prompt groups and of short prompts run, and what each is to run as: the host's
decisions, which the profiling library reports (held on the CPU and ahead of each run on the GPU)."""
import synth


def _shape(h, d, f, r, layers=2):
    return synth.ModelShape(h, h // d, d, r, f, n_layers=layers, name=f"d{d}-h{h}-f{f}")


# A decode step: its sequences' positions; MLP-down's parts of K and its workgroups.
STEPS = [
    (_shape(512, 64, 512, 16), [9, 3], 1, 16), (_shape(640, 80, 3200, 20), [40, 0, 7], 3, 60), (_shape(1408, 128, 7040, 32), [33, 5], 5, 220),
    (_shape(1152, 64, 9216, 16), [12, 30], 7, 252), (_shape(3072, 128, 12288, 32, 1), [4, 90], 5, 480), (_shape(4096, 64, 4096, 16, 1), [11300], 4, 1024),
    (_shape(4096, 64, 4096, 16, 1), [11300, 0], 2, 256), (_shape(1920, 80, 7680, 20), [21], 7, 840), (_shape(640, 80, 1920, 20), [21], 1, 40),
    (_shape(1024, 128, 8192, 32), [12, 0, 40], 8, 256), (_shape(1024, 64, 8192, 16), [77], 8, 512), (_shape(640, 80, 2560, 20), [5, 60], 2, 40),
    (_shape(4096, 128, 16384, 32, 1), [3, 17], 4, 512),
]

# A prompt in groups: its first position, tokens, sequences of the context (the tokens of a group), the one it is appended to; of each
# group whether it attends together, pieces of a head at most, parts of MLP-down.
GROUPS = [
    (_shape(512, 64, 2048, 16), 890, 13, 8, 1, [(False, 4, 2), (True, 8, 2)]), (_shape(512, 64, 2048, 16), 896, 10, 8, 0, [(True, 7, 2), (True, 8, 2)]),
    (_shape(512, 64, 2048, 16), 895, 9, 8, 0, [(False, 4, 2), (False, 32, 2)]), (_shape(512, 64, 2048, 16), 888, 16, 8, 0, [(False, 4, 2), (True, 7, 2)]),
    (_shape(512, 64, 2048, 16, 1), 6000, 7, 8, 0, [(True, 8, 2)]),
    (_shape(1280, 80, 2560, 20), 927, 8, 8, 0, [(False, 2, 2)]), (_shape(1280, 80, 2560, 20), 928, 5, 5, 4, [(False, 3, 2)]),
    (_shape(1280, 80, 2560, 20), 929, 15, 6, 0, [(False, 2, 2)] * 2 + [(False, 5, 2)]), (_shape(1280, 80, 2560, 20), 1249, 16, 8, 0, [(False, 2, 2), (True, 8, 2)]),
    (_shape(1280, 80, 2560, 20), 1250, 8, 8, 0, [(True, 8, 2)]), (_shape(1280, 80, 5120, 20, 1), 2000, 5, 5, 4, [(True, 8, 5)]), (_shape(1280, 64, 1280, 16, 1), 1700, 15, 6, 0, [(True, 8, 1), (True, 8, 1), (False, 4, 1)]),
    (_shape(2560, 80, 2560, 20, 1), 2060, 8, 8, 0, [(True, 7, 2)]), (_shape(2560, 80, 2560, 20, 1), 1023, 3, 3, 0, [(True, 7, 2)]),
    (_shape(2048, 128, 2048, 32), 1025, 9, 8, 3, [(False, 2, 2), (False, 16, 2)]), (_shape(2048, 128, 2048, 32), 1281, 9, 8, 3, [(True, 8, 1), (False, 16, 2)]),
    (_shape(4096, 128, 4096, 32, 1), 1300, 4, 4, 0, [(True, 7, 2)]),
    (_shape(1024, 128, 4096, 32, 1), 2049, 6, 8, 0, [(False, 5, 4)]),
    (_shape(4096, 64, 4096, 16, 1), 1500, 8, 8, 0, [(True, 3, 2)]), (_shape(4096, 64, 4096, 16, 1), 900, 2, 2, 1, [(True, 3, 2)]),
]
# ... where every query attends for itself: in a grid for the positions they have.
ALONE = [
    (_shape(1280, 80, 5120, 20), 0, 11, 8, 0, [(False, 2, 3), (False, 5, 5)]), (_shape(1280, 80, 5120, 20, 1), 880, 8, 8, 0, [(False, 2, 3)]), (_shape(1536, 64, 6144, 16, 1), 510, 4, 2, 1, [(False, 5, 4), (False, 5, 3)]),
    (_shape(2560, 80, 10240, 20, 1), 126, 4, 2, 0, [(False, 4, 3), (False, 4, 2)]), (_shape(1024, 128, 4096, 32, 1), 2040, 9, 8, 0, [(False, 4, 4), (False, 32, 4)]), (_shape(1024, 128, 1024, 32, 1), 505, 10, 8, 2, [(False, 4, 1), (False, 16, 1)]),
    (_shape(4096, 128, 4096, 32, 1), 255, 3, 2, 0, [(False, 4, 2), (False, 8, 4)]), (_shape(640, 80, 640, 20, 1), 3000, 1, 8, 0, [(False, 32, 1)]), (_shape(512, 64, 512, 16, 1), 511, 3, 3, 0, [(False, 10, 1)]),
]

# A short prompt behind pos0 positions: parts of MLP-down beside the attention, its workgroups, parts of the attention's keys.
SHORT = [
    (_shape(128, 64, 128, 16), 3, 5, 1, 2, 1), (_shape(512, 64, 2048, 16), 0, 16, 3, 24, 1), (_shape(512, 64, 2048, 16), 7, 23, 3, 24, 1), (_shape(640, 80, 1920, 20), 40, 31, 3, 30, 1),
    (_shape(1280, 80, 2560, 20), 1, 40, 4, 80, 1), (_shape(1280, 80, 5120, 20), 5, 48, 6, 240, 1), (_shape(1024, 128, 4096, 32), 9, 33, 6, 96, 1), (_shape(1152, 64, 9216, 0), 2, 3, 8, 144, 1),
    (_shape(4096, 128, 8192, 32, 1), 4, 12, 4, 256, 1), (_shape(512, 64, 2048, 16, 1), 1500, 44, 3, 48, 6), (_shape(640, 80, 2560, 20, 1), 1300, 8, 4, 40, 5), (_shape(1024, 128, 4096, 32, 1), 900, 19, 6, 96, 7),
    (_shape(640, 80, 1280, 20), 6, 14, 2, 20, 1), (_shape(640, 64, 3200, 16), 2, 26, 5, 50, 1), (_shape(640, 128, 4480, 32), 3, 8, 7, 70, 1), (_shape(3072, 128, 12288, 32, 1), 4, 11, 8, 384, 1),
    (_shape(512, 64, 2048, 16), 5, 38, 0, 0, 1), (_shape(640, 80, 2560, 20, 1), 1300, 37, 4, 40, 5), (_shape(640, 64, 2560, 16), 9, 34, 4, 40, 1), (_shape(1280, 80, 5120, 20, 1), 2000, 33, 8, 160, 8),
    (_shape(4096, 64, 16384, 16, 1), 2000, 16, 8, 512, 4),
]


def step(shape, lens):
    import paper_2604_23553_amd as cf
    with cf.profile_build():
        return cf.cfpp_debug_attention_plan(cf.Config.from_shape(shape, max(lens) + 1, len(lens)), len(lens))


def groups(shape, pos0, T, max_batch):
    import paper_2604_23553_amd as cf
    cfg, n = cf.Config.from_shape(shape, pos0 + T, max_batch), min(max_batch, 8)
    with cf.profile_build():
        return [cf.cfpp_debug_attention_plan(cfg, min(n, T - t), pos0 + t) for t in range(0, T, n)]


def short(shape, pos0, T):
    import paper_2604_23553_amd as cf
    with cf.profile_build():
        return cf.cfpp_debug_prefill_beside(cf.Config.from_shape(shape, pos0 + T), 128, T, pos0)
