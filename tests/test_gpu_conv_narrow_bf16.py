"""bf16 3x3 layers of up to 64 channels, at the sizes where the pixel blocks, staging passes, channel octets and channel
classes of their kernels end, against the oracle with operands rounded to bf16; the check, its bars and the infinities
next to the tensors are those of the ragged-channel layers."""
import ctypes

import numpy as np
import pytest

import synth_inputs as S
import test_gpu_ragged_channels as R


def form(c, n, h, w, converted):
    """(class, tiles per wavefront, passes, ragged, order, whole blocks) of a layer of c channels; None: another kernel."""
    import paper_1707_04585_amd as rv
    query = rv.load_library().rvn_conv3x3_bf16_narrow_form
    query.restype = ctypes.c_int64
    v = query(c, c, n, h, w, int(converted))
    return None if v < 0 else tuple(v >> 8 * k & 255 for k in range(5, -1, -1))


# (channels, images, rows, columns, filter converted by the driver, taken): shapes that were timed on both kernels
LINE = [
    # one block per compute unit, and two
    (60, 64, 13, 13, 1, 1), (60, 100, 13, 13, 1, 0), (60, 30, 27, 23, 1, 0), (44, 100, 13, 13, 1, 1), (44, 42, 27, 23, 1, 0),
    (48, 14, 40, 40, 1, 0), (48, 48, 14, 14, 1, 1), (52, 50, 19, 21, 1, 1),
    # the register-tiled kernel splits, and does not
    (64, 9, 56, 56, 1, 1), (64, 10, 56, 56, 1, 0), (64, 32, 28, 28, 1, 1), (64, 33, 28, 28, 1, 0), (64, 128, 14, 14, 1, 1),
    (64, 140, 14, 14, 1, 0), (64, 32, 32, 32, 1, 1), (64, 40, 32, 32, 1, 0),
    # a filter converted in the kernel
    (36, 64, 13, 13, 0, 1), (33, 80, 13, 13, 0, 0), (42, 21, 12, 50, 0, 1), (36, 32, 19, 21, 0, 0), (33, 8, 8, 70, 0, 1), (33, 16, 8, 70, 0, 0),
    # ragged rows of up to 32 channels
    (28, 64, 31, 31, 0, 1), (28, 100, 31, 31, 0, 0), (32, 100, 19, 21, 1, 1), (32, 128, 19, 21, 1, 0), (32, 200, 20, 20, 1, 1),
]


@pytest.mark.parametrize("shape", LINE, ids=lambda k: "c%d n%d %dx%d-%d" % k[:5])
def test_line(shape):
    """The kernel takes a layer where it was the faster one."""
    *layer, converted, taken = shape
    assert (form(*layer, converted) is not None) == bool(taken)


CASES = [
    # up to 16 channels: two taps an instruction
    dict(n=64, c=32, h=32, w=32),      # 256 blocks of 256 pixels, whole; statistics of four wavefronts
    dict(n=33, c=32, h=32, w=32),      # blocks of 128 pixels
    dict(n=4, c=32, h=8, w=8),         # blocks of 64 pixels
    dict(n=5, c=16, h=8, w=8),         # one octet; a last block that is not full
    dict(n=70, c=32, h=1, w=4),        # 64 images a block: two staging passes
    dict(n=70, c=30, h=1, w=3),        # the same, ragged
    dict(n=3, c=6, h=5, w=4),          # three channels, one quad a row
    dict(n=3, c=18, h=7, w=3),         # a quad longer than the row; an octet of one channel
    # up to 32
    dict(n=128, c=64, h=16, w=32),     # blocks of 256 pixels, two staging passes
    dict(n=64, c=48, h=16, w=16),      # blocks of 64 pixels, three octets
    dict(n=9, c=34, h=9, w=13),        # one channel into the second tile and the third octet
    dict(n=70, c=62, h=30, w=30),      # ragged rows up to 65536 pixels
    # up to 64
    dict(n=32, c=128, h=32, w=32),     # blocks of 128 pixels, two staging passes; the most pixels taken
    dict(n=64, c=112, h=8, w=8),       # seven octets, blocks of 32 pixels
    dict(n=3, c=66, h=9, w=9),         # one channel into the third tile and the fifth octet
    dict(n=11, c=126, h=32, w=32),     # the most pixels taken with a filter that is converted in the kernel
    dict(n=2, c=128, h=3, w=80),       # one row a block, two staging passes
]


@pytest.mark.gpu
@pytest.mark.parametrize("case", CASES, ids=lambda k: "n%d c%d %dx%d" % (k["n"], k["c"], k["h"], k["w"]))
def test_block(case):
    R.test_block(dict(kind="basic", **case))


SAME_BITS = [
    # (images, channels, rows, columns); blocks that are whole, so that both kernels leave statistics
    (33, 16, 32, 32), (24, 16, 8, 8), (140, 16, 32, 32), (33, 32, 16, 16), (300, 32, 16, 16), (40, 48, 16, 16), (20, 40, 32, 32),
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
