"""bf16 3x3 layers of up to 64 channels, at the sizes where the pixel blocks, staging passes, channel octets and channel
classes of their kernels end, against the oracle with operands rounded to bf16; the check, its bars and the infinities
next to the tensors are those of the ragged-channel layers."""
import pytest

import test_gpu_ragged_channels as R

pytestmark = pytest.mark.gpu

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


@pytest.mark.parametrize("case", CASES, ids=lambda k: "n%d c%d %dx%d" % (k["n"], k["c"], k["h"], k["w"]))
def test_block(case):
    R.test_block(dict(kind="basic", **case))
