"""Passes of 65 .. 1024 tokens and the tiles that each is to take in the end: (tokens, features, K step, parts of K) of the
first product and of the second, None where it keeps the plan of prefill_plans.py's kind.  Together they take every
tile that only such passes take, with K split and whole where a plan does (held on the CPU)."""
from tests.prefill_plans import H1024, H2560, H4096, _shape

H1536, H1664 = _shape(1536, 64, 6144, 16), _shape(1664, 64, 6656, 16)
H3072, H3200 = _shape(3072, 64, 6144, 16), _shape(3200, 80, 12800, 20)

MIDDLE = [
    (H2560, 100, (128, 96, 64, 1), None),
    (H3200, 600, (128, 160, 32, 1), None),
    (H4096, 96, (128, 128, 64, 1), (128, 128, 64, 8)),
    (H3072, 70, (128, 128, 64, 2), None),
    (H1536, 512, (128, 192, 32, 1), None),
    (H1536, 205, (128, 96, 64, 1), None),
    (H1664, 130, (128, 96, 64, 1), None),
    (H1024, 900, (128, 256, 32, 1), None),
    (H1536, 900, None, (128, 192, 32, 4)),
]
