"""Host-only checks of the C ABI: the library loads without a GPU, exports
every symbol the header declares, rejects bad arguments before touching the
device, and its driver enqueues the amount of work the paper states."""
import json
import os
import re

import pytest

import paper_1707_04585_amd as rv
from paper_1707_04585_amd.binding import rvn_tensor

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


def declared_functions():
    text = open(os.path.join(ROOT, "include", "revnet.h")).read()
    text = re.sub(r"/\*.*?\*/", "", text, flags=re.S)
    return sorted(set(re.findall(r"\b(revnet_\w+)\s*\(", text)))


def test_library_exports_every_declared_symbol():
    lib = rv.load_library()
    names = declared_functions()
    assert {"revnet_block_fwd", "revnet_block_bwd_reconstruct", "revnet_stack_fwd", "revnet_stack_bwd"} <= set(names)
    for name in names:
        assert hasattr(lib, name), name
    assert rv.revnet_version() >= 1000


def fake(ptr, n=2, c=4, h=4, w=4, sn=None, sc=None, sh=None, sw=1):
    sc = h * w if sc is None else sc
    sn = 2 * c * sc if sn is None else sn
    sh = w if sh is None else sh
    return rvn_tensor(ptr, n, c, h, w, sn, sc, sh, sw)


def fake_params(desc):
    layer = dict(w=0x10, gamma=0x20, beta=0x30)
    return dict(F=[layer] * desc.num_layers(), G=[layer] * desc.num_layers())


BASE = 0x10000000


def halves(base, c=4, h=4, w=4):
    """Two channel halves of one [2, 2c, h, w] buffer."""
    return fake(base, c=c, h=h, w=w), fake(base + 4 * c * h * w, c=c, h=h, w=w)


def status_of(fn, *a, **k):
    with pytest.raises(rv.RevnetError) as e:
        fn(*a, **k)
    return e.value.status, str(e.value)


def test_forward_argument_validation_happens_before_any_device_call():
    d = rv.BlockDesc("basic", 4)
    x1, x2 = halves(BASE)
    y1, y2 = halves(BASE + 0x100000)
    p = fake_params(d)
    fwd, _ = rv.revnet_workspace_bytes(d, 2, 4, 4)
    ws = (BASE + 0x800000, fwd)
    ERR = dict(null=-1, shape=-2, stride=-3, dtype=-4, ws=-5, alias=-6)

    assert status_of(rv.revnet_block_fwd, d, fake(0), x2, p, y1, y2, ws)[0] == ERR["null"]
    assert status_of(rv.revnet_block_fwd, d, fake(BASE, c=3), x2, p, y1, y2, ws)[0] == ERR["shape"]
    assert status_of(rv.revnet_block_fwd, d, fake(BASE, n=0), x2, p, y1, y2, ws)[0] == ERR["shape"]
    assert status_of(rv.revnet_block_fwd, d, x1, fake(BASE + 256, h=5), p, y1, y2, ws)[0] == ERR["shape"]
    assert status_of(rv.revnet_block_fwd, d, fake(BASE, sw=2), x2, p, y1, y2, ws)[0] == ERR["stride"]
    assert status_of(rv.revnet_block_fwd, d, fake(BASE, sh=8), x2, p, y1, y2, ws)[0] == ERR["stride"]
    assert status_of(rv.revnet_block_fwd, d, fake(BASE, sc=8), x2, p, y1, y2, ws)[0] == ERR["stride"]
    assert status_of(rv.revnet_block_fwd, d, fake(BASE, sn=32), x2, p, y1, y2, ws)[0] == ERR["stride"]
    # aliasing: x1 with x2 (overlapping planes) is refused, y1 == x1 is allowed (would proceed)
    assert status_of(rv.revnet_block_fwd, d, x1, fake(BASE + 64), p, y1, y2, ws)[0] == ERR["alias"]
    assert status_of(rv.revnet_block_fwd, d, x1, x2, p, x2, y2, ws)[0] == ERR["alias"]
    # workspace: missing, misaligned, too small, overlapping a tensor
    assert status_of(rv.revnet_block_fwd, d, x1, x2, p, y1, y2, None)[0] == ERR["ws"]
    assert status_of(rv.revnet_block_fwd, d, x1, x2, p, y1, y2, (ws[0] + 4, fwd))[0] == ERR["ws"]
    assert status_of(rv.revnet_block_fwd, d, x1, x2, p, y1, y2, (ws[0], fwd - 1))[0] == ERR["ws"]
    assert status_of(rv.revnet_block_fwd, d, x1, x2, p, y1, y2, (BASE, fwd))[0] == ERR["alias"]
    # parameters
    bad = dict(F=p["F"], G=[dict(w=0x10, gamma=None, beta=0x30)] * 2)
    assert status_of(rv.revnet_block_fwd, d, x1, x2, bad, y1, y2, ws)[0] == ERR["null"]
    # descriptor
    assert status_of(rv.revnet_block_fwd, rv.BlockDesc(7, 4), x1, x2, p, y1, y2, ws)[0] == ERR["dtype"]
    assert status_of(rv.revnet_block_fwd, rv.BlockDesc("basic", 4, conv_dtype=5), x1, x2, p, y1, y2, ws)[0] == ERR["dtype"]
    assert status_of(rv.revnet_block_fwd, rv.BlockDesc("basic", 4, bn_eps=0.0), x1, x2, p, y1, y2, ws)[0] == ERR["shape"]
    assert status_of(rv.revnet_block_fwd, rv.BlockDesc("bottleneck", 4, width=0), x1, x2, p, y1, y2, ws)[0] == ERR["shape"]
    assert status_of(rv.revnet_stack_fwd, d, 0, x1, x2, [p], y1, y2, ws)[0] == ERR["shape"]
    st, msg = status_of(rv.revnet_block_fwd, d, x1, x2, p, y1, y2, (ws[0], 8))
    assert "workspace" in msg and str(fwd) in msg


def test_backward_argument_validation():
    d = rv.BlockDesc("bottleneck", 4, width=2, conv_dtype="bf16")
    y1, y2 = halves(BASE)
    dy1, dy2 = halves(BASE + 0x100000)
    x1, x2 = halves(BASE + 0x200000)
    dx1, dx2 = halves(BASE + 0x300000)
    p = fake_params(d)
    _, bwd = rv.revnet_workspace_bytes(d, 2, 4, 4)
    ws = (BASE + 0x800000, bwd)
    call = rv.revnet_block_bwd_reconstruct
    assert status_of(call, d, y1, y2, dy1, dy2, p, x1, x2, dx1, dx2, p, 0, (ws[0], bwd - 1))[0] == -5
    assert status_of(call, d, y1, y2, dy1, dy2, p, x1, x2, dx1, fake(0), p, 0, ws)[0] == -1
    # dx may alias dy and x may alias y, but x must not alias dy
    assert status_of(call, d, y1, y2, dy1, dy2, p, dy1, x2, dx1, dx2, p, 0, ws)[0] == -6
    g_bad = dict(F=p["F"], G=[dict(w=None, gamma=0x20, beta=0x30)] * 3)
    assert status_of(call, d, y1, y2, dy1, dy2, p, x1, x2, dx1, dx2, g_bad, 0, ws)[0] == -1
    assert status_of(rv.revnet_stack_bwd, d, -1, y1, y2, dy1, dy2, [p], x1, x2, dx1, dx2, [p], 0, ws)[0] == -2


@pytest.mark.parametrize("kind,c,width,convs", [("basic", 16, 0, 4), ("bottleneck", 128, 64, 6)])
def test_driver_operation_count_matches_paper(kind, c, width, convs):
    """Section 3.2 'Computational overhead': forward N, reversible backward 3N
    (one recomputation + data gradient + filter gradient per convolution)."""
    gold = json.load(open(os.path.join(ROOT, "tests", "golden", "cost_model.json")))
    d = rv.BlockDesc(kind, c, width)
    for depth in (1, 5):
        fwd, bwd = rv.revnet_stack_cost(d, depth, 8, 16, 16)
        n_conv = convs * depth
        assert fwd["conv_fwd_calls"] == gold["reversible_forward"] * n_conv
        assert fwd["conv_dgrad_calls"] == fwd["conv_wgrad_calls"] == 0
        assert bwd["conv_fwd_calls"] + bwd["conv_dgrad_calls"] + bwd["conv_wgrad_calls"] == gold["reversible_backward"] * n_conv
        assert bwd["conv_fwd_calls"] == bwd["conv_dgrad_calls"] == bwd["conv_wgrad_calls"] == n_conv
        assert abs(bwd["conv_flops"] / fwd["conv_flops"] - 3.0) < 1e-12
        total = fwd["conv_flops"] + bwd["conv_flops"]
        assert abs(total / fwd["conv_flops"] - gold["reversible_total"]) < 1e-12


def test_workspace_does_not_depend_on_depth_and_scales_with_batch():
    """Section 3.2: activation storage independent of depth.  The workspace
    query has no depth argument at all; the cost query confirms the driver
    uses the same plan for depth 1 and depth 50."""
    d = rv.BlockDesc("basic", 16)
    f1, b1 = rv.revnet_workspace_bytes(d, 8, 32, 32)
    f2, b2 = rv.revnet_workspace_bytes(d, 16, 32, 32)
    assert b1 > f1 > 0
    assert 1.9 < b2 / b1 < 2.1
    c1 = rv.revnet_stack_cost(d, 1, 8, 32, 32)
    c50 = rv.revnet_stack_cost(d, 50, 8, 32, 32)
    # linear in depth: the top block pays for one statistics pass that every block below it gets
    # from the launch that merged its input's statistics ahead, so count from depth 1 and 2
    c2 = rv.revnet_stack_cost(d, 2, 8, 32, 32)
    per_block = c2[1]["kernel_launches"] - c1[1]["kernel_launches"]
    assert 0 < per_block <= c1[1]["kernel_launches"] - 1
    assert c50[1]["kernel_launches"] == c1[1]["kernel_launches"] + 49 * per_block
    per_block_bytes = c2[1]["algorithmic_bytes"] - c1[1]["algorithmic_bytes"]
    assert 0.9 * c1[1]["algorithmic_bytes"] < per_block_bytes <= c1[1]["algorithmic_bytes"]
    assert abs(c50[1]["algorithmic_bytes"] - (c1[1]["algorithmic_bytes"] + 49 * per_block_bytes)) < 1e-6 * c50[1]["algorithmic_bytes"]


@pytest.mark.parametrize("kind,conv,c_half,width,n,h,w,fwd,bwd", [
    ("basic", "bf16", 390, 0, 23, 15, 3, 8055552, 23019264),
    ("bottleneck", "bf16", 3, 413, 26, 7, 3, 5849856, 16976896),
    ("bottleneck", "f32", 33, 263, 70, 8, 2, 2413312, 13728000),
    ("basic", "f32", 48, 0, 48, 2, 69, 1290752, 10912256),
    ("bottleneck", "bf16", 132, 66, 64, 56, 56, 107887104, 356190464),   # small filters of ragged channel counts
    ("bottleneck", "bf16", 100, 44, 13, 27, 23, 3043840, 19125504),
    ("basic", "bf16", 26, 0, 64, 32, 32, 7097600, 30166272),
])
def test_workspace_sizes_are_kept(kind, conv, c_half, width, n, h, w, fwd, bwd):
    """Sizes that callers may have stored: a kernel added later lives in the room that was there."""
    assert rv.revnet_workspace_bytes(rv.BlockDesc(kind, c_half, width, conv_dtype=conv), n, h, w) == (fwd, bwd)


@pytest.mark.parametrize("kind,c,width", [("basic", 66, 0), ("bottleneck", 136, 34)])
def test_ragged_bf16_layers_take_their_statistics_from_a_pass_over_the_tensor(kind, c, width):
    """bf16 channel counts off the 8- and 16-channel steps: 32 rows cut into whole tiles and 31 do not, and the bytes
    per pixel are the same (statistics merged from tile moments would spare a read of the tensor)."""
    d = rv.BlockDesc(kind, c // 2, width, conv_dtype="bf16")
    per_pixel = [rv.revnet_stack_cost(d, 2, 40, h, 32)[0]["algorithmic_bytes"] / (40 * h * 32) for h in (32, 31)]
    assert abs(per_pixel[0] / per_pixel[1] - 1) < 0.01, per_pixel


def test_cost_query_takes_the_largest_descriptors():
    """65536 channels, the most a descriptor allows: counted as any other, although no filter gradient of that size
    (2^32 elements per partial result) fits the 32-bit indices of the flat-pixel kernel."""
    for c_half, width in ((65536, 65536), (46341, 46341), (65536, 64)):
        fwd, bwd = rv.revnet_stack_cost(rv.BlockDesc("bottleneck", c_half, width), 1, 2, 7, 7)
        assert (fwd["conv_fwd_calls"], bwd["conv_wgrad_calls"]) == (6, 6)
        assert bwd["kernel_launches"] == 31


def test_down_block_and_body_argument_validation():
    """The subsampling block and the body check shapes, channel chains, even
    sizes, overlaps and the workspace before anything is enqueued."""
    d = rv.DownDesc("bottleneck", 8, 16)
    assert d.width == 4
    layer = dict(w=0x10, gamma=0x20, beta=0x30)
    p = dict(R=[layer] * 3, S=dict(w=0x40))
    x = fake(BASE, n=2, c=8, h=4, w=4, sn=8 * 16)
    y = fake(BASE + 0x100000, n=2, c=16, h=2, w=2, sn=16 * 4)
    dy = fake(BASE + 0x200000, n=2, c=16, h=2, w=2, sn=16 * 4)
    dx = fake(BASE + 0x300000, n=2, c=8, h=4, w=4, sn=8 * 16)
    fwd, bwd = rv.revnet_down_workspace_bytes(d, 2, 4, 4)
    assert bwd > fwd > 0
    ws = (BASE + 0x800000, bwd)
    assert status_of(rv.revnet_down_workspace_bytes, d, 2, 5, 4)[0] == -2          # odd height
    assert status_of(rv.revnet_down_fwd, d, x, p, fake(BASE + 0x100000, n=2, c=16, h=4, w=4), ws)[0] == -2
    assert status_of(rv.revnet_down_fwd, d, x, p, y, (ws[0], fwd - 1))[0] == -5
    assert status_of(rv.revnet_down_fwd, d, x, dict(R=[layer] * 3, S=dict(w=None)), y, ws)[0] == -1
    assert status_of(rv.revnet_down_fwd, d, x, p, fake(BASE + 64, n=2, c=16, h=2, w=2, sn=16 * 4), ws)[0] == -6
    assert status_of(rv.revnet_down_bwd, d, x, dy, p, x, p, 0, ws)[0] == -6          # dx must not be x
    assert status_of(rv.revnet_down_bwd, d, x, dy, p, dx, dict(R=[layer] * 2 + [dict(w=None, gamma=1, beta=1)], S=dict(w=1)), 0, ws)[0] == -1
    assert status_of(rv.revnet_down_bwd, d, x, dy, p, dx, p, 0, (BASE, bwd))[0] == -6  # workspace over x

    stages = [rv.BlockDesc("basic", 4), rv.BlockDesc("basic", 8)]
    body = rv.BodyDesc(stages, [2, 3], [rv.DownDesc("basic", 8, 16)])
    f, b = rv.revnet_body_workspace_bytes(body, 2, 4, 4)
    assert b > f > 0
    # the workspace is the largest single need, not a sum over stages or depths
    deeper = rv.BodyDesc(stages, [20, 30], [rv.DownDesc("basic", 8, 16)])
    assert rv.revnet_body_workspace_bytes(deeper, 2, 4, 4) == (f, b)
    wrong_chain = rv.BodyDesc(stages, [2, 3], [rv.DownDesc("basic", 8, 12)])
    assert status_of(rv.revnet_body_workspace_bytes, wrong_chain, 2, 4, 4)[0] == -2
    assert status_of(rv.revnet_body_workspace_bytes, body, 2, 6, 5)[0] == -2        # odd width at the block
    bp = dict(F=[layer] * 2, G=[layer] * 2)
    dp = dict(R=[layer] * 2, S=dict(w=0x40))
    tops = [fake(BASE + 0x100000, n=2, c=8, h=4, w=4, sn=8 * 16), fake(BASE + 0x200000, n=2, c=16, h=2, w=2, sn=16 * 4)]
    wsb = (BASE + 0x800000, b)
    assert status_of(rv.revnet_body_fwd, body, x, [[bp] * 2, [bp] * 3], [dp], [tops[0], tops[0]], wsb)[0] == -2
    assert status_of(rv.revnet_body_fwd, body, x, [[bp] * 2, [bp] * 3], [dp], tops, (wsb[0], f - 1))[0] == -5
    overl = [tops[0], fake(BASE + 0x100000 + 64, n=2, c=16, h=2, w=2, sn=16 * 4)]
    assert status_of(rv.revnet_body_fwd, body, x, [[bp] * 2, [bp] * 3], [dp], overl, wsb)[0] == -6
    dtops = [fake(BASE + 0x300000, n=2, c=8, h=4, w=4, sn=8 * 16), fake(BASE + 0x400000, n=2, c=16, h=2, w=2, sn=16 * 4)]
    assert status_of(rv.revnet_body_bwd, body, tops, [dtops[0], tops[1]], [[bp] * 2, [bp] * 3], [dp],
                     [[bp] * 2, [bp] * 3], [dp], 0, wsb)[0] == -6
    assert status_of(rv.revnet_body_bwd, body, tops, dtops, [[bp] * 2, [bp] * 3], [dp],
                     [[bp] * 2, [bp] * 3], [dp], 0, (wsb[0], b - 1))[0] == -5


def test_fixed_point_entry_points_validate_arguments():
    d = rv.BlockDesc("basic", 4)
    x1, x2 = halves(BASE)
    y1, y2 = halves(BASE + 0x100000)
    p = fake_params(d)
    fwd, bwd = rv.revnet_fixed_workspace_bytes(d, 2, 4, 4)
    plain_fwd, plain_bwd = rv.revnet_workspace_bytes(d, 2, 4, 4)
    assert fwd > plain_fwd and bwd > plain_bwd
    ws = (BASE + 0x800000, fwd)
    assert status_of(rv.revnet_stack_fwd_fixed, d, 1, 0, x1, x2, [p], y1, y2, ws)[0] == -2     # frac_bits out of range
    assert status_of(rv.revnet_stack_fwd_fixed, d, 1, 31, x1, x2, [p], y1, y2, ws)[0] == -2
    assert status_of(rv.revnet_stack_fwd_fixed, d, 1, 16, x1, x2, [p], y1, y2, (ws[0], plain_fwd))[0] == -5
    assert status_of(rv.revnet_stack_fwd_fixed, d, 1, 16, x1, x2, [p], x2, y2, ws)[0] == -6
    full = fake(BASE, c=8, sn=8 * 16)
    strided = fake(BASE + 0x100000, c=8, sc=32, sn=8 * 32)
    assert status_of(rv.revnet_fixed_to_float, full, 16, strided)[0] == -3                     # destination must be dense
    assert status_of(rv.revnet_fixed_from_float, full, 40, full)[0] == -2
    assert status_of(rv.revnet_fixed_from_float, full, 16, fake(BASE + 64, c=8, sn=8 * 16))[0] == -6


def test_stem_argument_validation():
    d = rv.rvn_stem_desc(3, 8, 7, 2, 1)
    img = fake(BASE, n=2, c=3, h=16, w=12, sn=3 * 192)
    conv = fake(BASE + 0x100000, n=2, c=8, h=8, w=6, sn=8 * 48)
    y = fake(BASE + 0x200000, n=2, c=8, h=4, w=3, sn=8 * 12)
    bwd = rv.revnet_stem_workspace_bytes(d, 2, 16, 12)
    assert bwd >= 2 * 8 * 48 * 4
    assert status_of(rv.revnet_stem_workspace_bytes, rv.rvn_stem_desc(3, 8, 4, 2, 1), 2, 16, 12)[0] == -2    # even kernel
    assert status_of(rv.revnet_stem_workspace_bytes, rv.rvn_stem_desc(8, 8, 7, 2, 1), 2, 16, 12)[0] == -2    # reduction too long
    assert status_of(rv.revnet_stem_workspace_bytes, rv.rvn_stem_desc(3, 8, 7, 3, 1), 2, 16, 12)[0] == -2    # stride
    assert status_of(rv.revnet_stem_fwd, d, img, 0x10, None, y)[0] == -1                                    # conv_out needed
    assert status_of(rv.revnet_stem_fwd, d, img, 0x10, conv, fake(BASE + 0x200000, n=2, c=8, h=8, w=6, sn=8 * 48))[0] == -2
    assert status_of(rv.revnet_stem_fwd, d, img, None, conv, y)[0] == -1
    assert status_of(rv.revnet_stem_fwd, rv.rvn_stem_desc(3, 8, 7, 2, 0), img, 0x10, conv, conv)[0] == -2   # no pooling: no conv_out
    assert status_of(rv.revnet_stem_bwd, d, img, conv, y, 0x10, 0, (BASE + 0x800000, bwd - 1))[0] == -5
    assert status_of(rv.revnet_stem_bwd, d, img, conv, y, None, 0, (BASE + 0x800000, bwd))[0] == -1
    assert status_of(rv.revnet_stem_bwd, d, img, conv, y, 0x10, 0, (BASE, bwd))[0] == -6


def test_static_workspace_entry_point_validates_and_rejects_oversize_on_the_host():
    """revnet_stack_fwd_static: argument checks and the size limit of its
    built-in workspace come before the first device call."""
    d = rv.BlockDesc("bottleneck", 128, 64, conv_dtype="bf16")
    n, c, h, w = 64, 128, 56, 56
    fwd, _ = rv.revnet_workspace_bytes(d, n, h, w)
    assert fwd > rv.STATIC_WS_BYTES
    big = lambda base: fake(base, n=n, c=c, h=h, w=w, sn=c * h * w)
    step = 4 * n * c * h * w
    x1, x2 = big(BASE), big(BASE + step)
    st, msg = status_of(rv.revnet_stack_fwd_static, d, 1, x1, x2, [fake_params(d)], x1, x2)
    assert st == -5 and "built-in workspace" in msg and str(fwd) in msg
    assert status_of(rv.revnet_stack_fwd_static, d, 0, x1, x2, [fake_params(d)], x1, x2)[0] == -2
    assert status_of(rv.revnet_stack_fwd_static, d, 1, x1, x1, [fake_params(d)], x1, x2)[0] == -6
    assert status_of(rv.revnet_stack_fwd_static, d, 1, big(0), x2, [fake_params(d)], x1, x2)[0] == -1


def test_a_setting_made_on_one_device_is_still_wanted_on_the_next(tmp_path):
    """The limit on a kernel's dynamic LDS is asked for once per device of the process, whichever thread comes first."""
    import subprocess
    src = tmp_path / "once.cpp"
    src.write_text("""
#include <thread>
#include <vector>
#include "once_per_device.h"
int main() {
    static rvn::OncePerDevice once;
    auto make = [](int device) { if (once.wanted(device)) once.made(device); };
    std::vector<std::thread> threads;
    for (int t = 0; t < 8; ++t) threads.emplace_back([=] { for (int d = 0; d < 63; d += 2) make(d); });
    for (auto &t : threads) t.join();
    for (int d = 0; d < 64; ++d)
        if (once.wanted(d) != (d % 2 == 1)) return 1;
    make(64);
    return once.wanted(64) && once.wanted(1000) && once.wanted(-1) ? 0 : 2;
}
""")
    exe = tmp_path / "once"
    subprocess.run(["g++", "-std=c++17", "-pthread", "-I", os.path.join(ROOT, "paper_1707_04585_amd", "csrc"), str(src), "-o", str(exe)], check=True)
    subprocess.run([str(exe)], check=True)
