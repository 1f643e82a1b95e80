"""The fp32 convolution and filter gradient over flat pixels, at the sizes where their tiles, channel
chunks, pixel chunks and staged runs end: against the oracle in float64, one block.  Every compiled instance
of both kernels is launched by a case; a host test below sees to that.  The bars are those of
the fp32 parity cases (forward 1e-5, gradients 1e-4).  About one ReLU argument in a million lies within
rounding of zero, and a decision taken the other way changes a gradient tensor of N elements by about
1 / sqrt(N) of its norm, which is above the bar.  So the cases of more than 100000 decisions per layer add 8 to
every beta: their ReLUs are all open (a normalised input below -8 / 1.5 is one in 10^7), no decision is close, and the
activation next to a border differs from the zero beyond it by more, not less."""
import random

import numpy as np
import pytest

import synth_inputs as S
from oracle import revnet_oracle as O

# (most leave a remainder of pixels and of channels in every tile)
CASES = [
    dict(kind="basic", n=3, c=34, h=3, w=7),        # 17 channels, 63 pixels (conv3x3_f32, as some of the next)
    dict(kind="basic", n=1, c=66, h=5, w=13),       # 33 channels, 65 pixels
    dict(kind="basic", n=1, c=66, h=7, w=9),        # 63 pixels
    dict(kind="basic", n=1, c=70, h=2, w=63),       # widest rows of the 128-pixel pitch; 35 channels
    dict(kind="basic", n=2, c=80, h=3, w=76),       # widest rows that have a backward plan
    dict(kind="basic", n=2, c=80, h=3, w=95),       # widest rows of the 64-pixel tiles: forward only
    dict(kind="basic", n=1, c=80, h=2, w=111),      # widest rows of the 32-pixel tile; forward only
    dict(kind="basic", n=1, c=68, h=3, w=1),        # one column: every side tap leaves the image
    dict(kind="bottleneck", n=5, c=136, h=7, w=7, width=33),      # one channel past a 32-channel chunk
    dict(kind="bottleneck", n=16, c=384, h=14, w=14, width=40),   # several tiles of channels, chunks and slices
    dict(kind="bottleneck", n=40, c=256, h=28, w=28, width=72),
    dict(kind="bottleneck", n=2, c=1100, h=7, w=5, width=520),    # filters larger than the activations
    # fewer partial filter gradients fit the scratch than would fill the chip
    dict(kind="bottleneck", n=70, c=66, h=8, w=2, width=263),
    dict(kind="basic", n=48, c=96, h=2, w=69),
    # the remaining tile shapes (channels x pixels) of the 3x3 kernel, by 8- and 16-channel chunks
    dict(kind="basic", n=40, c=66, h=41, w=10),     # 64 x 128
    dict(kind="basic", n=5, c=66, h=53, w=31),      # 64 x 64
    dict(kind="basic", n=80, c=34, h=5, w=41),      # (conv3x3_f32)
    dict(kind="basic", n=95, c=34, h=30, w=23),     # (conv3x3_f32)
    dict(kind="basic", n=99, c=34, h=17, w=39),     # (conv3x3_f32)
    dict(kind="basic", n=19, c=66, h=36, w=12),     # 32 x 128, 16-channel chunks
    dict(kind="basic", n=20, c=34, h=10, w=41),     # (conv3x3_f32)
    dict(kind="basic", n=101, c=130, h=9, w=12),    # 32 x 32, one piece
    dict(kind="basic", n=1, c=34, h=2, w=34),       # 32 x 32, two pieces
    dict(kind="basic", n=1, c=34, h=2, w=49),       # 32 x 32, four pieces
    dict(kind="basic", n=22, c=130, h=12, w=32),    # 32 x 128, 8-channel chunks
    dict(kind="basic", n=6, c=130, h=19, w=72),     # 32 x 64, 8-channel chunks, the wider pitch
    dict(kind="basic", n=10, c=66, h=10, w=42),     # 32 x 64, 16-channel chunks, four pieces
    dict(kind="basic", n=1, c=66, h=1, w=35),       # 32 x 32, two pieces
    dict(kind="basic", n=1, c=66, h=1, w=48),       # 32 x 32, four pieces
    # and of the 1x1 kernel
    dict(kind="bottleneck", n=5, c=818, h=49, w=19, width=17),    # 64 x 64
    dict(kind="bottleneck", n=24, c=38, h=53, w=26, width=17),    # 32 x 128
    dict(kind="bottleneck", n=3, c=336, h=50, w=18, width=33),    # 32 x 32
    dict(kind="bottleneck", n=6, c=500, h=9, w=11, width=60),     # filter gradient: 64 x 128 and 128 x 64
]
WIDEST_BACKWARD = 76


def layers(cfg):
    """(c_in, c_out, filter side) of a function's layers; the data gradient's are the same with the counts exchanged."""
    c = cfg["c"] // 2
    return [(c, c, 3)] if cfg["kind"] == "basic" else [(c, cfg["width"], 1), (cfg["width"],) * 2 + (3,), (cfg["width"], c, 1)]


def test_every_instance_has_a_case():
    """Every instance that a large sample of layers selects is launched by a case above: forward, data and filter gradient."""
    import paper_1707_04585_amd as rv
    lib = rv.load_library()
    conv = lambda ci, co, ks, n, h, w: lib.rvn_conv_gemm_f32_instance(ci, co, ks, n, h, w)
    wgrad = lambda ci, co, ks, n, h, w: lib.rvn_conv_wgrad_gemm_f32_instance(ci, co, ks, n, h, w)
    have, have_w = set(), set()
    for cfg in CASES:
        geo = (cfg["n"], cfg["h"], cfg["w"])
        for ci, co, ks in layers(cfg):
            have |= {conv(ci, co, ks, *geo), conv(co, ci, ks, *geo)}
            if cfg["w"] <= WIDEST_BACKWARD:
                have_w.add(wgrad(ci, co, ks, *geo))
    rng = random.Random(7)
    log = lambda lo, hi: int(round(lo * (hi / lo) ** rng.random()))
    seen, seen_w = set(), set()
    for _ in range(60000):
        ks, ci, co = rng.choice([1, 3]), log(1, 2048), log(17, 2048)
        geo = (log(1, 256), log(1, 128), log(1, 128))
        seen.add(conv(ci, co, ks, *geo))
        seen_w.add(wgrad(ci, co, ks, *geo))
    assert len(seen - {-1}) == 18 and len(seen_w - {-1}) == 7
    assert seen <= have | {-1}, sorted(divmod(v, 4096) for v in seen - have)
    assert seen_w <= have_w | {-1}, sorted(divmod(v, 8) for v in seen_w - have_w)


@pytest.mark.gpu
@pytest.mark.parametrize("case", CASES, ids=lambda k: "%s n%d c%d %dx%d" % (k["kind"], k["n"], k["c"], k["h"], k["w"]))
def test_block_against_oracle(case):
    import torch
    import paper_1707_04585_amd as rv
    from paper_1707_04585_amd.torch_harness import StackRunner, download_grads
    cfg = dict(width=None, depth=1, conv="f32", affine="random")
    cfg.update(case)
    x, params, dy = S.draw_stack(S.BASE_SEED + 909, **cfg)
    c = cfg["c"] // 2
    if cfg["n"] * cfg["h"] * cfg["w"] * max(ci for ci, _, _ in layers(cfg)) > 100000:
        for fn in ("F", "G"):
            for layer in params[0][fn]:
                layer["beta"] += 8
    print(case, flush=True)
    r = StackRunner(**cfg)
    r.set_params(params)
    Y, DY = r.new_pair(x), r.new_pair(dy)
    r.forward(Y, Y)
    torch.cuda.synchronize()
    y = r.to_host(Y[0])
    sp = lambda t: (np.ascontiguousarray(t[:, :c]), np.ascontiguousarray(t[:, c:]))
    y1, y2, _, stored = O.stack_fwd(*sp(x), params, keep=True)
    assert O.rel_l2(y, np.concatenate([y1, y2], 1)) < 1e-5
    # the skip operand in a tensor of its own: the same bits
    X, Z = r.new_pair(x), r.new_pair()
    r.forward(X, Z)
    torch.cuda.synchronize()
    np.testing.assert_array_equal(r.to_host(Z[0]), y)
    if cfg["w"] > WIDEST_BACKWARD:
        with pytest.raises(rv.RevnetError):   # refused, as by the row-band filter gradient
            r.backward(Y, DY, Y, DY)
        return
    XR, DX = r.new_pair(), r.new_pair()
    r.backward(Z, DY, XR, DX)
    torch.cuda.synchronize()
    grads = download_grads(r.grads)
    r.backward(Y, DY, Y, DY, accumulate=True)   # in place, added to the gradients that are there: twice those, to rounding
    torch.cuda.synchronize()
    x_rec, dx = r.to_host(Y[0]), r.to_host(DY[0])
    np.testing.assert_array_equal(x_rec, r.to_host(XR[0]))
    np.testing.assert_array_equal(dx, r.to_host(DX[0]))
    twice = download_grads(r.grads)
    dx1, dx2, ref = O.stack_bwd_stored(stored, params, *sp(dy))
    want_dx = np.concatenate([dx1, dx2], 1)
    errs = dict(dx=O.rel_l2(dx, want_dx))
    for fn in ("F", "G"):
        for l, (got, want, both) in enumerate(zip(grads[0][fn], ref[0][fn], twice[0][fn])):
            # (of the larger of the two: a shift that reaches the next BN through open ReLUs and a 1x1 layer cancels
            # there, and its gradient is zero)
            scale = max(np.linalg.norm(want[k]) for k in ("gamma", "beta"))
            errs["%s%d.w" % (fn, l)] = O.rel_l2(got["w"], want["w"])
            for k in ("gamma", "beta"):
                errs["%s%d.%s" % (fn, l, k)] = np.linalg.norm(got[k] - want[k]) / scale
            for k in ("w", "gamma", "beta"):
                np.testing.assert_allclose(both[k], 2 * got[k], rtol=3e-7, atol=0)
    print({k: "%.1e" % v for k, v in errs.items()}, flush=True)
    assert O.rel_l2(x_rec, x) < 1e-5
    assert max(errs.values()) < 1e-4, errs
