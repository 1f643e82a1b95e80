// fp32 3x3 convolution (forward and data gradient) of layers of up to 32 output channels, for the units
// c_3(x) = Conv_3x3(ReLU(BN(x))) of Section 2.2.
//
// What bounds it.  A workgroup's work is one chain -- set-up, one round trip to memory, staging, 36 matrix
// instructions per 4 channels, stores -- run by one or two wavefronts per SIMD, so every instruction outside the
// matrix loop costs its issue time, some 4 to 8 cycles.  Clock stamps in the row-band kernel (conv_mfma.hip) at 16 -> 16
// channels of 32x32: 3.0 us of index set-up, 2.7 us until the loads were out, 0.1 us of waiting for them, 2.7 us into LDS,
// 2.7 us of matrix instructions (1.9 without stalls), 0.8 us of epilogue.  So this kernel is laid out for few instructions:
//  * a thread stages one fixed 4-pixel group of the band for every cpp-th channel: its offsets are formed once, an
//    item adds a scalar, and what lies outside is loaded from past the buffer's end, which gives zero;
//  * the filter needs neither LDS nor index arithmetic: the nine taps of the (output, input) channel pair of a
//    lane's matrix operand are consecutive in memory and are loaded into registers as they are;
//  * a lane multiplies four consecutive pixels (four 16-pixel tiles, interleaved), so the twelve operands of a filter
//    row are one 16-byte and two 4-byte LDS reads, and results leave as 16-byte stores (16 of 4 bytes before);
//  * input channels past the last one are skipped four at a time.
// Measured, forward launch of 16 -> 16 channels with statistics: 128 images of 32x32 15.8 -> 12.0 us; 8 -> 8 at 4 of 8x8
// (one workgroup) 11.4 -> 4.7 us.  28 -> 28 at 19x21, 51 images (flat-pixel kernel before): 14.7 -> 11.8 us, data
// gradient 9.5 (beside the filter gradient it has a kernel of its own, conv3x3_f32_bwd.hip).
#include <algorithm>

#include "conv3x3_f32_body.h"
#include "kernels.h"

namespace rvn {

namespace {

using namespace c3f;

template <int MT, int PASSES, bool TR, bool VEC, bool EMIT>
__global__ __launch_bounds__(kThreads, 2) void conv3x3_f32_k(const C3fArgs p) {
    extern __shared__ __align__(16) float smem[];
    conv3x3_f32_body<MT, PASSES, TR, VEC, EMIT>(p, blockIdx.x, blockIdx.y, smem);
}

// Multiplier of fdiv_c3f: exact for e * d < 2^32 (e is a thread or block index here).
uint32_t mul_of(int d) { return d == 1 ? 0u : (uint32_t)((1ull << 32) / (uint64_t)d + 1ull); }

// Up to 32 output channels.  Against the row-band kernel 0.31 to 0.86 of the time (forward of two basic blocks).  From 33
// channels on the flat-pixel kernel's 32-row tiles win: 33 to 64 channels took 0.87 to 1.45.
// Where the flat-pixel kernel takes the layer too (17 to 32 channels, rows that are not whole quads) both run in rounds
// over the 256 compute units: this one by its blocks of 64 quads, which rows and images fill to 60 to 95 %, that one by
// pixels, so each is ahead just where the other has begun another round, by a fifth to a half.
//  * up to 128 blocks: 0.77 to 1.03.  In rows of up to 32 pixels that begins at 16384 pixels from 29 channels on (as many
//    fours as 32; 1.02 to 1.10 below), in longer rows at 4096 (1.00 to 1.18 below, with three rows staged for one).
//  * above, a round of 256 blocks takes as long as two of 32768 pixels.  This kernel multiplies channels in fours, that one in
//    eights: with 17 to 20 and 25 to 28 channels 0.66 to 1.01 where the even number of rounds is rounded up, with 21 to 24 and 29
//    to 32 0.85 to 1.00 where it is rounded down, up to four rounds (six where channels are not whole octets), and no gain
//    beyond.  One round more 1.02 to 1.50.
//  * its 64-pixel tiles with chunks of 16 channels take nearly twice as long per round: 0.79 to 0.96.
//  * rows of 64 pixels and more, where it stages twice its tile: 0.60 to 1.02.
// Measured over 1362 shapes of 2000 to 400000 pixels; none that this rule sends here takes more than 1.04.
bool takes(int ci, int co, const Geo &g, const C3fPlan &pl) {
    if (co > 32) return false;
    const ConvGemmTile flat = conv_gemm_f32_tile(ci, co, 3, g);
    if (flat.pixels == 0) return true;
    const int64_t px = g.pixels();
    if (g.w >= 64) return px >= 4096;
    const int fours = (ci + 3) / 4;
    if (pl.blocks <= 128) return g.w > 32 ? px >= 4096 : fours < 8 || px > 16384;
    const bool slow = flat.pixels == 64 && flat.chunk == 16, octets = fours % 2 == 0;
    const int64_t rounds = (pl.blocks + 255) / 256, single = (px + 32767) / 32768, theirs = slow ? 2 * single - 1 : single;
    return theirs > 1 && 2 * rounds <= theirs + (octets ? 0 : 1) && (!octets || slow || theirs <= (ci % 8 ? 6 : 4));
}

template <bool TR>
void launch_c3f(Ctx &cx, const C3fLaunch &L) {
    const C3fArgs &a = L.a;
#define RVN_CASE(MT_, P_, V_)                                                                                  \
    if (L.mt == MT_ && L.passes == P_ && L.vec == V_) {                                                        \
        if constexpr (!TR && V_) {                                                                             \
            if (a.emit) {                                                                                      \
                cx.run(conv3x3_f32_k<MT_, P_, false, true, true>, L.grid, dim3(kThreads), L.lds_bytes, a);     \
                return;                                                                                        \
            }                                                                                                  \
        }                                                                                                      \
        cx.run(conv3x3_f32_k<MT_, P_, TR, V_, false>, L.grid, dim3(kThreads), L.lds_bytes, a);                 \
        return;                                                                                                \
    }
    RVN_CASE(1, 6, true) RVN_CASE(1, 8, true) RVN_CASE(2, 6, true) RVN_CASE(2, 8, true)
    RVN_CASE(1, 6, false) RVN_CASE(1, 8, false) RVN_CASE(2, 6, false) RVN_CASE(2, 8, false)
#undef RVN_CASE
}

}  // namespace

// The pixel block of a workgroup: whole rows of one image, or whole images, of at most 16 quads per wavefront, such
// that a channel of the band (halo rows included) takes half of the threads at most.
C3fPlan plan_c3f(const Geo &g, int waves) {
    C3fPlan best{};
    double best_score = -1.0;
    const int wq = (g.w + 3) / 4, slots = 16 * waves, threads = 64 * waves;
    for (int imgs = 1; imgs <= slots && imgs <= g.n; ++imgs) {
        for (int th = imgs > 1 ? g.h : 1; th <= g.h; ++th) {
            const int quads = imgs * th * wq, items = imgs * (th + 2) * wq;
            if (quads > slots || items > threads / 2) break;
            const int64_t bands = (g.h + th - 1) / th, blocks = bands * ((g.n + imgs - 1) / imgs);
            const double score = (double)g.n * g.h * wq / ((double)blocks * slots) - (items > threads / 3 ? 0.02 : 0.0);
            const int cpp = items <= threads / 3 ? 3 : 2, pitch = 4 * wq + 4;
            // (an odd number of quads: eight lanes reading a quad each of eight channels take all 32 banks)
            const int plane = ((imgs * (th + 2) * pitch + 4) / 4 | 1) * 4;
            if (score <= best_score + 1e-9 || 18 * plane * 4 > 16 * 1024 * (1 + waves / 2)) continue;
            best_score = score;
            best.passes = cpp == 3 ? 6 : 8;
            best.blocks = blocks;
            C3fShape &s = best.s;
            s.N = g.n; s.H = g.h; s.W = g.w;
            s.TH = th; s.IMGS = imgs; s.bands = (int)bands; s.wq = wq; s.quads = quads; s.lrows = th + 2; s.items = items;
            s.cpp = cpp; s.pitch = pitch; s.plane = plane;
        }
    }
    if (best.passes == 0 || best.blocks * best.s.bands >= ((int64_t)1 << 32)) return C3fPlan{};
    C3fShape &s = best.s;
    s.m_bands = mul_of(s.bands); s.m_items = mul_of(s.items); s.m_rq = mul_of(s.lrows * s.wq);
    s.m_wq = mul_of(s.wq); s.m_q = mul_of(s.TH * s.wq);
    return best;
}

bool conv3x3_f32_plan(View in, const float *scale_shift, const float *w, bool transposed, int ci, int co, Geo g,
                      Epilogue ep, const View *r, View out, C3fLaunch &L) {
    if (co > 32) return false;
    const C3fPlan pl = plan_c3f(g, 4);
    if (pl.passes == 0 || !takes(ci, co, g, pl)) return false;
    // bytes from the base to the end of the last plane; every one must end below kNowhere
    const int64_t in_b = 4 * ((g.n - 1) * in.sn + (ci - 1) * in.sc + g.hw()), out_b = 4 * ((g.n - 1) * out.sn + (co - 1) * out.sc + g.hw());
    const int64_t r_b = r ? 4 * ((g.n - 1) * r->sn + (co - 1) * r->sc + g.hw()) : 0, w_b = (int64_t)ci * co * 36;
    if (std::max(std::max(in_b, out_b), std::max(r_b, w_b)) >= (int64_t)kNowhere) return false;
    auto aligned = [](const View &v) { return v.sn % 4 == 0 && v.sc % 4 == 0 && (reinterpret_cast<uintptr_t>(v.p) & 15) == 0; };
    C3fArgs a{};
    a.in = in.p; a.scale_shift = scale_shift; a.w = w; a.r = r ? r->p : nullptr; a.out = out.p;
    a.isn = (uint32_t)in.sn; a.isc = (uint32_t)in.sc;
    a.rsn = r ? (uint32_t)r->sn : 0; a.rsc = r ? (uint32_t)r->sc : 0;
    a.osn = (uint32_t)out.sn; a.osc = (uint32_t)out.sc;
    a.in_bytes = (uint32_t)in_b; a.out_bytes = (uint32_t)out_b; a.r_bytes = (uint32_t)r_b; a.w_bytes = (uint32_t)w_b;
    a.CI = ci; a.CO = co; a.ep = (int)ep;
    a.s = pl.s;
    L.a = a;
    L.vec = g.w % 4 == 0 && aligned(in) && aligned(out) && (!r || aligned(*r));
    L.whole = g.w % 4 == 0 && pl.s.quads == 64 && g.n % pl.s.IMGS == 0 && g.h % pl.s.TH == 0;
    // More than 16 channels: both tiles in one workgroup (the band is staged once), or one each where that leaves
    // compute units idle.  Step of two blocks of 32 channels: 128 blocks 652 us together, 571 apart;
    // 512 blocks 1225 and 1447.
    L.mt = co > 16 && pl.blocks >= 256 ? 2 : 1;
    L.passes = pl.passes;
    L.grid = dim3((unsigned)pl.blocks, (unsigned)((co + L.mt * 16 - 1) / (L.mt * 16)));
    L.lds_bytes = (size_t)pl.passes * pl.s.cpp * pl.s.plane * 4;
    return true;
}

// How a layer of dense, aligned tensors runs, for the tests: channel tiles of a workgroup, staging passes, whole quads a row, whole
// blocks (statistics are left of the output), in pairs of hexadecimal digits, or -1 (another kernel).
extern "C" int rvn_conv3x3_f32_form(int ci, int co, int n, int h, int w) {
    const Geo g{n, h, w};
    float *const at = reinterpret_cast<float *>(256);
    C3fLaunch L;
    if (!conv3x3_f32_plan(dense_view(at, ci, g), at, at, false, ci, co, g, EP_STORE, nullptr, dense_view(at, co, g), L)) return -1;
    return ((L.mt * 256 + L.passes) * 256 + (int)L.vec) * 256 + (int)(L.vec && L.whole);
}

bool conv3x3_f32(Ctx &cx, View in, const float *scale_shift, const float *w, bool transposed, int ci, int co, Geo g,
                 Epilogue ep, const View *r, View out) {
    C3fLaunch L;
    if (!conv3x3_f32_plan(in, scale_shift, w, transposed, ci, co, g, ep, r, out, L)) return false;
    const int tiles = (int)L.grid.x * 4;
    if (cx.want_emit && cx.emit_buf && !transposed && L.vec && L.whole && (size_t)co * tiles * 2 <= cx.emit_floats) {
        L.a.emit = cx.emit_buf;
        L.a.emit_tiles = tiles;
        cx.emitted = EmittedStats{out.p, out.sn, out.sc, co, g.n, g.h, g.w, tiles, 64};
    }
    if (transposed) launch_c3f<true>(cx, L);
    else launch_c3f<false>(cx, L);
    return true;
}

}  // namespace rvn
