"""bf16 3x3 layers of up to 64 channels, at the sizes where the pixel blocks, staging passes, channel octets and channel
classes of their kernels end, against the oracle with operands rounded to bf16; the check, its bars and the infinities
next to the tensors are those of the ragged-channel layers.  Every instance that a layer's shape selects is launched by a
case; a host test sees to that."""
import ctypes
import random

import numpy as np
import pytest

import synth_inputs as S
import test_gpu_ragged_channels as R
from oracle import revnet_oracle as O


def form(c, n, h, w, converted=-1):
    """(class, tiles per wavefront, passes, ragged, order, whole blocks, filter converted) of a layer of c channels; None:
    another kernel.  converted: -1 for what the driver does in a function of two such layers."""
    import paper_1707_04585_amd as rv
    query = rv.load_library().rvn_conv3x3_bf16_narrow_form
    query.restype = ctypes.c_int64
    v = query(c, c, n, h, w, converted)
    return None if v < 0 else tuple(v >> 8 * k & 255 for k in range(6, -1, -1))


# (channels, images, rows, columns, filter converted by the driver, taken): shapes that were timed on both kernels
LINE = [
    # one block per compute unit, and two
    (60, 64, 13, 13, 1, 1), (60, 100, 13, 13, 1, 0), (60, 30, 27, 23, 1, 0), (44, 100, 13, 13, 1, 1), (44, 42, 27, 23, 1, 0),
    (48, 14, 40, 40, 1, 0), (48, 48, 14, 14, 1, 1), (52, 50, 19, 21, 1, 1),
    # the register-tiled kernel splits, and does not
    (64, 9, 56, 56, 1, 1), (64, 10, 56, 56, 1, 0), (64, 32, 28, 28, 1, 1), (64, 33, 28, 28, 1, 0), (64, 128, 14, 14, 1, 1),
    (64, 140, 14, 14, 1, 0), (64, 32, 32, 32, 1, 1), (64, 40, 32, 32, 1, 0),
    # a filter converted in the kernel, a chunk of channels at a time and all at once
    (36, 100, 16, 16, 0, 1), (42, 42, 27, 23, 0, 0), (36, 33, 12, 50, 0, 1), (33, 33, 8, 70, 0, 1), (33, 50, 8, 70, 0, 0),
    (36, 64, 13, 13, 0, 1), (33, 80, 13, 13, 0, 0), (36, 32, 19, 21, 0, 0), (39, 64, 19, 21, 0, 0),
    # ragged rows of up to 32 channels
    (28, 64, 31, 31, 0, 1), (28, 100, 31, 31, 0, 0), (28, 45, 31, 33, 0, 1), (28, 50, 31, 33, 0, 0), (22, 63, 31, 33, 0, 1),
    (32, 100, 19, 21, 1, 1), (32, 128, 19, 21, 1, 0), (32, 200, 20, 20, 1, 1),
]


@pytest.mark.parametrize("shape", LINE, ids=lambda k: "c%d n%d %dx%d-%d" % k[:5])
def test_line(shape):
    """The kernel takes a layer where it was the faster one."""
    *layer, converted, taken = shape
    assert (form(*layer, converted) is not None) == bool(taken)


CASES = [
    # up to 16 channels
    dict(n=64, c=32, h=32, w=32),      # 256 blocks of 256 pixels, whole; statistics of four wavefronts
    dict(n=33, c=32, h=32, w=32),      # blocks of 128 pixels
    dict(n=4, c=32, h=8, w=8),         # two images a block
    dict(n=5, c=16, h=8, w=8),         # one octet; a last block that is not full
    dict(n=70, c=32, h=1, w=4),        # 32 images a block
    dict(n=70, c=30, h=1, w=3),        # the same, ragged
    dict(n=3, c=6, h=5, w=4),          # three channels, one quad a row
    dict(n=3, c=18, h=7, w=3),         # a quad longer than the row; an octet of one channel
    # up to 32
    dict(n=128, c=64, h=16, w=32),     # blocks of 256 pixels, two staging passes
    dict(n=64, c=48, h=16, w=16),      # blocks of 128 pixels, three octets
    dict(n=9, c=34, h=9, w=13),        # one channel into the second tile and the third octet
    dict(n=70, c=62, h=30, w=30),      # ragged rows up to 65536 pixels
    # up to 64
    dict(n=32, c=128, h=32, w=32),     # blocks of 128 pixels, two staging passes; the most that conv3x3_bf16 would split
    dict(n=64, c=112, h=8, w=8),       # seven octets, blocks of 64 pixels
    dict(n=3, c=66, h=9, w=9),         # one channel into the third tile and the fifth octet
    dict(n=11, c=126, h=32, w=32),     # a last octet of seven channels
    dict(n=2, c=128, h=3, w=80),       # one row a block, two staging passes
    # statistics by the pass in tiles: one workgroup a channel, and several
    dict(n=2, c=128, h=8, w=24), dict(n=1, c=112, h=8, w=40), dict(n=6, c=128, h=24, w=24),
]
# The remaining instances: (images, channels, rows, columns), by class, tiles per wavefront and staging passes.
INSTANCES = [
    (66, 2, 4, 68), (1, 8, 3, 132), (2, 2, 3, 149), (2, 2, 65, 130), (1, 8, 3, 172), (1, 8, 3, 256), (1, 2, 3, 172), (18, 2, 8, 196),
    # 17 to 32 channels
    (5, 24, 13, 4), (1, 32, 13, 20), (2, 32, 32, 4), (7, 17, 4, 11), (73, 17, 4, 67), (1, 32, 37, 7),
    (1, 24, 3, 100), (1, 24, 4, 128), (1, 32, 4, 88), (1, 32, 4, 128), (1, 17, 4, 88), (1, 24, 3, 93), (1, 17, 3, 87), (1, 32, 3, 89),
    (129, 24, 24, 12), (136, 32, 68, 4), (132, 18, 47, 1), (137, 17, 48, 5), (67, 17, 123, 1), (276, 32, 19, 5),
    (1, 24, 4, 132), (16, 24, 64, 64), (1, 32, 3, 132), (1, 17, 4, 148), (1, 17, 2, 129), (1, 32, 4, 129),
    # 33 to 64
    (5, 56, 13, 4), (13, 40, 5, 4), (8, 40, 8, 4), (1, 56, 7, 37), (16, 33, 4, 4), (2, 40, 13, 10), (6, 33, 5, 9), (1, 43, 86, 3),
    (2, 56, 4, 44), (1, 56, 4, 64), (1, 40, 5, 52), (1, 40, 4, 64), (2, 56, 3, 43), (2, 33, 4, 44), (2, 40, 3, 43), (1, 33, 4, 64),
    (2, 43, 3, 48), (348, 37, 1, 1), (288, 44, 1, 1),
    (128, 56, 12, 12), (143, 40, 34, 4), (141, 56, 18, 5), (133, 33, 40, 4), (345, 45, 17, 1), (149, 44, 17, 6),
    (1, 40, 4, 68), (128, 40, 4, 64), (1, 56, 4, 82), (1, 33, 13, 66), (1, 40, 4, 66), (1, 33, 4, 68), (1, 43, 4, 72), (64, 44, 16, 24), (279, 33, 20, 1),
]
WIDEST_BACKWARD = 168
CASES += [dict(n=n, c=2 * c, h=h, w=w) for n, c, h, w in INSTANCES]


def test_every_instance_has_a_case():
    """Every form that a large sample of layers takes is that of a case above."""
    have = {form(k["c"] // 2, k["n"], k["h"], k["w"]) for k in CASES}
    rng = random.Random(11)
    log = lambda lo, hi: int(round(lo * (hi / lo) ** rng.random()))
    seen = set()
    for _ in range(60000):
        c, n, h, w = rng.randint(1, 64), log(1, 512), log(1, 128), log(1, 260)
        for layer in ((c, n, h, w), (8 * (c // 8) or 8, n, h, w), (8 * (c // 8) or 8, n, 4 * (h // 4) or 4, 4 * (w // 4) or 4)):
            if layer[1] * layer[2] * layer[3] <= 300000:
                seen.add(form(*layer))
    assert seen - {None} <= have, sorted(seen - {None} - have)


@pytest.mark.gpu
@pytest.mark.parametrize("case", CASES, ids=lambda k: "n%d c%d %dx%d" % (k["n"], k["c"], k["h"], k["w"]))
def test_block(case):
    if case["w"] <= WIDEST_BACKWARD:
        R.test_block(dict(kind="basic", **case))
        return
    import torch
    import paper_1707_04585_amd as rv
    from paper_1707_04585_amd.torch_harness import StackRunner
    cfg = dict(kind="basic", width=None, depth=1, conv="bf16", affine="random", **case)
    x, params, _ = S.draw_stack(S.BASE_SEED + 1620, **cfg)
    c = cfg["c"] // 2
    r = StackRunner(**cfg)
    r.set_params(params)
    Y = r.new_pair(x)
    r.forward(Y, Y)
    torch.cuda.synchronize()
    with O.conv_operands("bf16"):
        y1, y2, *_ = O.stack_fwd(np.ascontiguousarray(x[:, :c]), np.ascontiguousarray(x[:, c:]), params, keep=True)
    assert O.rel_l2(r.to_host(Y[0]), np.concatenate([y1, y2], 1)) < 1e-2
    with pytest.raises(rv.RevnetError):   # refused by the filter gradient
        r.backward(Y, Y, Y, Y)


@pytest.mark.gpu
def test_statistics_in_tiles_of_an_unaligned_tensor():
    """The same pass where the stream's halves start one float off a 16-byte boundary."""
    import torch
    cfg = dict(kind="basic", n=3, c=128, h=8, w=24, width=None, depth=1, conv="bf16", affine="random")
    x, params, dy = S.draw_stack(S.BASE_SEED + 1621, **cfg)

    def halves(src, device):
        out = []
        for part in (src[:, :64], src[:, 64:]):
            t = torch.empty(part.size + 1, dtype=torch.float32, device=device)[1:].view(part.shape)
            out.append(t.copy_(torch.as_tensor(part.astype(np.float32))))
        return out

    R.check_block(cfg, x, params, dy, halves)


SAME_BITS = [
    # (images, channels, rows, columns); blocks that are whole, so that both kernels leave statistics
    (33, 16, 32, 32), (32, 16, 32, 32), (24, 16, 8, 8), (140, 16, 32, 32), (33, 32, 16, 16), (300, 32, 16, 16), (40, 48, 16, 16), (20, 40, 32, 32),
    (64, 56, 8, 8), (33, 64, 16, 16), (20, 64, 32, 32),
    # blocks that are not whole, in layers that the wider kernel splits and leaves statistics of
    (20, 64, 24, 24), (17, 56, 40, 40), (30, 64, 16, 12), (25, 56, 32, 6), (70, 56, 4, 48),
    # ragged, where the general kernel's chunks are 16, 32 and 64 channels: with a filter that the driver converts
    (20, 44, 13, 11), (20, 46, 14, 30), (17, 56, 7, 6), (17, 64, 5, 2), (30, 52, 20, 21), (60, 61, 12, 12),
    # and without
    (20, 33, 13, 13), (40, 36, 9, 9), (24, 28, 9, 9), (20, 18, 30, 30), (17, 24, 9, 3),
]


@pytest.mark.gpu
@pytest.mark.parametrize("shape", SAME_BITS, ids=lambda k: "n%d c%d %dx%d" % k)
def test_forward_bits_are_those_of_the_wider_kernels(shape):
    """Sums and statistics keep the order of the kernels that take the layer where this one does not: tensors that end just
    short of 4 GiB, which only those take, give the same bits as dense ones."""
    import torch
    import paper_1707_04585_amd as rv
    from paper_1707_04585_amd.torch_harness import StackRunner
    n, ch, h, w = shape
    cfg = dict(kind="basic", n=n, c=2 * ch, h=h, w=w, width=None, depth=2, conv="bf16", affine="random")
    x, params, _ = S.draw_stack(S.BASE_SEED + 1619, **cfg)
    r = StackRunner(**cfg)
    r.set_params(params)
    full = torch.as_tensor(x.astype(np.float32)).to(r.device)
    dense, far = 2 * ch * h * w, ((1 << 30) - 2 * ch * h * w) // n // 4 * 4 - 4
    assert (n - 1) * far * 4 > 0xf0000000 and (n * far + ch * h * w) * 4 < 1 << 32
    got = []
    for sn in (dense, far):
        both = torch.empty((n - 1) * sn + dense, dtype=torch.float32, device=r.device).as_strided((n, 2 * ch, h, w), (sn, h * w, w, 1))
        both.copy_(full)
        X = [both[:, :ch], both[:, ch:]]
        rv.revnet_stack_fwd(r.desc, 2, *X, r.params, *X, r.ws)
        torch.cuda.synchronize()
        got.append(both.cpu().numpy())
    np.testing.assert_array_equal(got[0], got[1])
