"""fp32 3x3 layers of up to 32 channels, at the sizes where the pixel blocks, staging passes and channel tiles of
their kernels end, against the oracle in float64 (the check and its bars are those of the flat-pixel kernels).  Every
compiled instance of the forward and of the gradient kernel is launched by a case; a host test sees to that."""
import random

import pytest

import test_gpu_conv_gemm as G

CASES = [
    # one pixel an image (not with one channel: the BN layer behind it removes its scale, and with it the gradient)
    dict(n=40, c=10, h=1, w=1),
    dict(n=3, c=6, h=5, w=3),          # a quad longer than the row
    dict(n=37, c=30, h=2, w=2),        # many images per block, the last block not full
    dict(n=4, c=16, h=8, w=8),         # one block, whole
    dict(n=5, c=32, h=8, w=8),         # a last block of one image; 16 channels
    dict(n=2, c=32, h=9, w=32),        # a last band of one row
    dict(n=3, c=26, h=7, w=65),        # 17 quads a row, ragged
    dict(n=2, c=18, h=6, w=64),        # 16 quads a row
    dict(n=2, c=32, h=4, w=160),       # widest rows with a backward plan
    dict(n=2, c=34, h=3, w=166),       # nearly the widest rows taken; forward only
    dict(n=1, c=34, h=2, w=172),       # too wide: row-band kernel; forward only
    dict(n=6, c=34, h=11, w=13),       # a second channel tile of one channel, a second chunk of one
    dict(n=3, c=64, h=16, w=16),       # two full channel tiles, whole blocks
    dict(n=130, c=34, h=32, w=15),     # the flat-pixel kernel's by its rounds; the gradients not
    dict(n=64, c=40, h=16, w=64),      # 256 blocks and more: both channel tiles in one workgroup; whole blocks, 8 staging passes
    dict(n=86, c=36, h=9, w=66),       # the same, ragged
    dict(n=128, c=64, h=16, w=32),     # the same, whole blocks
    # the other instances: forward
    dict(n=8, c=12, h=4, w=8),         # one tile, 8 passes, whole blocks
    dict(n=270, c=36, h=5, w=28),      # both tiles, blocks that are not whole
    dict(n=283, c=38, h=1, w=114),     # both tiles, 8 passes, ragged
    dict(n=18, c=34, h=16, w=136),     # both tiles, 8 passes, blocks that are not whole
    # and gradients: four wavefronts, 8 passes
    dict(n=11, c=20, h=1, w=11), dict(n=16, c=34, h=1, w=6), dict(n=4, c=36, h=1, w=32),
    # eight wavefronts
    dict(n=132, c=10, h=93, w=1), dict(n=134, c=10, h=4, w=68), dict(n=141, c=36, h=37, w=1),
    dict(n=382, c=10, h=1, w=85), dict(n=3, c=10, h=88, w=156), dict(n=310, c=34, h=1, w=62), dict(n=152, c=38, h=4, w=40),
]
# (channels, images, rows, columns, forward taken, gradients taken): ragged layers that were timed on both kernels
LINE = [
    (18, 58, 19, 21, 1, 1), (18, 72, 19, 21, 0, 1), (18, 85, 19, 21, 1, 1), (24, 142, 13, 13, 0, 1), (24, 210, 13, 13, 1, 1),
    (24, 285, 13, 13, 0, 0), (28, 20, 41, 41, 1, 1), (28, 57, 41, 41, 0, 1), (28, 1858, 9, 9, 1, 0), (28, 946, 13, 13, 1, 0),
    (31, 4, 26, 23, 0, 1), (32, 31, 19, 21, 0, 1), (32, 47, 19, 21, 1, 1), (32, 138, 33, 35, 0, 0), (32, 86, 31, 31, 1, 1), (32, 182, 31, 31, 0, 1),
    # rows whose gradients are refused
    (32, 40, 4, 150, 1, 0), (17, 4, 6, 101, 0, 0), (17, 20, 6, 101, 1, 0),
    # channels that the flat-pixel kernels do not take
    (16, 946, 13, 13, 1, 1),
]


def forward(c, n, h, w):
    """(channel tiles, staging passes, whole quads, whole blocks) of the forward launch; None: another kernel."""
    import paper_1707_04585_amd as rv
    v = rv.load_library().rvn_conv3x3_f32_form(c, c, n, h, w)
    return None if v < 0 else tuple(v >> 8 * k & 255 for k in (3, 2, 1, 0))


def gradients(c, n, h, w):
    """(wavefronts, staging passes, chunks of output channels, whole quads) of the gradient launch; None: other kernels."""
    import paper_1707_04585_amd as rv
    v = rv.load_library().rvn_conv3x3_f32_bwd_form(c, c, n, h, w)
    return None if v < 0 else tuple(v >> 8 * k & 255 for k in (3, 2, 1, 0))


def test_every_instance_has_a_case():
    """Every instance that a large sample of layers selects is launched by a case above."""
    layers = [(k["c"] // 2, k["n"], k["h"], k["w"]) for k in CASES]
    have, have_b = {forward(*l) for l in layers}, {gradients(*l) for l in layers}
    rng = random.Random(5)
    log = lambda lo, hi: int(round(lo * (hi / lo) ** rng.random()))
    seen, seen_b = set(), set()
    for _ in range(40000):
        layer = (rng.randint(1, 32), log(1, 512), log(1, 128), log(1, 180))
        for c, n, h, w in (layer, (layer[0], layer[1], 4 * (layer[2] // 4) or 1, 4 * (layer[3] // 4) or 4)):
            if n * h * w <= 1000000:
                seen.add(forward(c, n, h, w))
                seen_b.add(gradients(c, n, h, w))
    assert len(seen - {None}) == 12 and len(seen_b - {None}) == 16
    assert seen - {None} <= have, seen - have
    assert seen_b - {None} <= have_b, seen_b - have_b


@pytest.mark.parametrize("shape", LINE, ids=lambda k: "c%d n%d %dx%d" % k[:4])
def test_line(shape):
    """A layer that the flat-pixel kernels take as well goes to the faster ones."""
    *layer, fwd, bwd = shape
    assert (forward(*layer) is not None, gradients(*layer) is not None) == (bool(fwd), bool(bwd))


@pytest.mark.gpu
@pytest.mark.parametrize("case", CASES, ids=lambda k: "n%d c%d %dx%d" % (k["n"], k["c"], k["h"], k["w"]))
def test_block_against_oracle(case, monkeypatch):
    if case["c"] <= 32:  # (the filter gradient's limit on the row length is twice that of wider layers)
        monkeypatch.setattr(G, "WIDEST_BACKWARD", 160)
    G.test_block_against_oracle(dict(kind="basic", **case))
