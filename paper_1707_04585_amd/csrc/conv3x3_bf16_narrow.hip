// 3x3 convolution with bf16 operands of layers of up to 64 channels that are small enough to be bound by the chain of
// one workgroup, for the units c_3(x) = Conv_3x3(ReLU(BN(x))) of Section 2.2.
//
// What bounds such a launch: set-up, one round trip to memory, staging, operand reads, stores; the matrix
// instructions themselves are 0.1 to 0.4 us.  So the whole reduction is staged at once and multiplied without a second
// barrier, and every phase is kept short:
//  * all loads of a thread -- 8 channels of one 4-pixel group, scale and shift, filter, skip values -- are issued
//    before the first of them is used; what lies outside is loaded from past the buffer's end, which gives zero;
//  * the filter goes from memory to operand registers, without LDS; a filter that the driver has not converted is
//    converted there (the 72 taps of an octet of input channels are consecutive);
//  * pixels lie on M and channels on N of v_mfma_f32_32x32x16_bf16, so four consecutive results of a lane are
//    consecutive pixels of one channel: 16-byte stores, and statistics that need few shuffles;
//  * blocks shrink (256 to 64 pixels) until every compute unit has one, instead of a split of the channels with a second
//    launch that sums it.
// Sums and statistics keep the order of the kernel that would take the layer otherwise, conv3x3_bf16 or the general one
// (Order in conv3x3_bf16_narrow_body.h): its results are the same bits, and so are those of the layers behind it.  Where
// blocks are not whole tiles of 64 pixels and that kernel would have left statistics, the pass over the tensor forms them
// in its order (bn_stats_tiles_k).  Where that kernel leaves none and this one does, they come from tiles of 64 pixels
// merged in double instead of fp32 sums over whole images: other roundings.
// Measured, forward launch with statistics (register-tiled kernel before): 16 -> 16 channels, 8 images of 32x32 8.8 -> 4.7 us,
// 128 images 13.0 -> 8.4; 32 -> 32, 128 of 16x16 12.5 -> 6.6; 56 -> 56, 128 of 8x8 10.8 + 4.2 (sum of the split) -> 6.6.
// With v_mfma_f32_16x16x32_bf16 (two taps of 16 channels an instruction, blocks down to 64 pixels) the 16-channel launches took
// 7.0 and 3.8 us, the others as long; sums in that order turned roundings of later layers.
#include <algorithm>

#include "conv3x3_bf16_narrow_body.h"
#include "kernels.h"

namespace rvn {

namespace {

using namespace c3n;

template <int NT, int CH, int PASSES, bool GEN, bool EMIT, bool W32, int ORDER, bool MERGE>
__global__ __launch_bounds__(kThreads, 2) void conv3x3_bf16_narrow_k(const C3nArgs p) {
    extern __shared__ __align__(16) char smem_c[];
    conv3x3_bf16_narrow_body<NT, CH, PASSES, GEN, EMIT, W32, ORDER, MERGE>(p, blockIdx.x, smem_c);
}

// Multiplier of fdiv_c3f: exact for e * d < 2^32 (e is a thread or block index here).
uint32_t mul_of(int d) { return d == 1 ? 0u : (uint32_t)((1ull << 32) / (uint64_t)d + 1ull); }

struct C3nPlan {
    C3nShape s;
    int passes;  // 0: no block fits
    int64_t blocks;
    size_t lds_bytes;
};

// The pixel block of a workgroup: whole rows of one image, or whole images, of at most `slots` quads.
C3nPlan plan_c3n(const Geo &g, int slots, int ch) {
    C3nPlan best{};
    double best_score = -1.0;
    const int wq = (g.w + 3) / 4, octs = ch / 8, pitch = 4 * wq + 1;
    for (int imgs = 1; imgs <= slots && imgs <= g.n; ++imgs) {
        for (int th = imgs > 1 ? g.h : 1; th <= g.h; ++th) {
            const int quads = imgs * th * wq, bquads = imgs * (th + 2) * wq, items = bquads * octs;
            const size_t lds = ((size_t)imgs * (th + 2) * pitch + 1) * record_bytes(ch) + 2 * ch * 4;  // (and scale and shift)
            if (quads > slots || items > 2 * kThreads || lds > 64 * 1024) break;
            const int64_t bands = (g.h + th - 1) / th, blocks = bands * ((g.n + imgs - 1) / imgs);
            const double score = (double)g.n * g.h * wq / ((double)blocks * slots) - (items > kThreads ? 0.02 : 0.0);
            if (score <= best_score + 1e-9) continue;
            best_score = score;
            best.passes = items > kThreads ? 2 : 1;
            best.blocks = blocks;
            best.lds_bytes = std::max(lds, (size_t)2 * 64 * 64);  // (two wavefronts' results, for the statistics)
            C3nShape &s = best.s;
            s.N = g.n; s.H = g.h; s.W = g.w;
            s.TH = th; s.IMGS = imgs; s.bands = (int)bands; s.wq = wq; s.quads = quads; s.lrows = th + 2; s.pitch = pitch;
            s.bquads = bquads; s.items = items;
        }
    }
    if (best.passes == 0 || best.blocks * best.s.bands >= ((int64_t)1 << 32)) return C3nPlan{};
    C3nShape &s = best.s;
    s.m_bands = mul_of(s.bands); s.m_bq = mul_of(s.bquads); s.m_rq = mul_of(s.lrows * s.wq);
    s.m_wq = mul_of(s.wq); s.m_q = mul_of(s.TH * s.wq);
    return best;
}

int class_of(int ci, int co) {
    const int most = std::max(ci, co);
    return most <= 16 ? 16 : most <= 32 ? 32 : most <= 64 ? 64 : 0;
}

// What depends on the sizes of a layer alone.
struct C3nChoice {
    bool converted, taken, sum_emits;
    int cls, nt, order;  // class of channels (16, 32 or 64), 32-pixel tiles of a wavefront, Order
    C3nPlan pl;
};

// Where the line lies (forward pass of two basic blocks, time over that of the kernels before):
//  * 33 to 64 channels: a block reads the whole filter (73 KB from L2) for 64 or 128 pixels, so what counts is whether the
//    blocks run side by side, one on each of the 256 compute units: 0.41 to 0.95 over 106 shapes up to there.  A second
//    block per unit: 40 to 56 channels up to 512 blocks and 32768 pixels 0.65 to 1.02 over 50 shapes, 588 blocks of 44 channels
//    1.04; 60 to 64 channels 1.01 to 1.19.  Where conv3x3_bf16 splits the channels and needs a second launch for their sum
//    (49 to 64, whole octets, at most 128 of its blocks) 0.52 to 1.00 at up to 720 blocks.
//    A filter that is converted here (33 to 42 channels, not whole octets), a chunk of 16 or 32 channels at a time: up to 512
//    blocks of 64 pixels 0.48 to 0.97 over 190 shapes, 588 1.02 to 1.17; up to 336 blocks of 128 pixels 0.61 to 0.96.  In
//    chunks of 64, all of it in registers beforehand: up to 256 blocks of 64 pixels 0.40 to 0.93, beyond and with
//    blocks of 128 1.02 to 1.19.
//  * 17 to 32 channels in rows that are not whole quads: 0.42 to 1.04 over 130 shapes up to 65536 pixels, 0.99 to 1.11 from
//    79000 on; with 25 and more channels in rows of more than 32 pixels, and with 32, one chunk of the register-tiled kernel,
//    0.75 to 1.00 up to 49152 pixels and 0.98 to 1.09 above.  In rows of whole quads 0.75 to 1.02 up to 128 images of 56x56.
//  * up to 16 channels: 0.59 to 0.99 over 48 shapes from four images of 2x2 to 64 of 112x112.
bool takes(const C3nChoice &c, const Conv3x3Bf16Form &form, int ci, int co, const Geo &g) {
    if (c.cls == 64) {
        if (!c.converted) return c.order == kChunk64 ? c.nt == 1 && c.pl.blocks <= 256 : c.pl.blocks <= (c.nt == 1 ? 512 : 336);
        if (form.parts > 1) return true;
        return c.pl.blocks <= 256 || (std::max(ci, co) <= 56 && c.pl.blocks <= 512 && g.pixels() <= 32768);
    }
    if (c.cls == 32) return g.w % 4 == 0 || g.pixels() <= (ci == 32 || (g.w > 32 && std::max(ci, co) > 24) ? 49152 : 65536);
    return true;
}

C3nChoice choose(int ci, int co, const Geo &g, bool converted) {
    C3nChoice c{};
    c.converted = converted;
    c.cls = class_of(ci, co);
    if (c.cls == 0) return c;
    // The larger block if it still gives every compute unit one (up to 32 channels with a filter that is converted in the
    // kernel, every second one).
    for (int nt = 2; nt >= 1; --nt) {
        const C3nPlan next = plan_c3n(g, 8 * nt * (4 / chan_waves(c.cls)), c.cls);
        if (next.passes == 0) continue;
        c.pl = next;
        c.nt = nt;
        if (next.blocks >= (converted || c.cls == 64 ? 256 : 128)) break;
    }
    if (c.pl.passes == 0) return c;
    const Conv3x3Bf16Form form = c.cls > 16 ? conv3x3_bf16_form(ci, co, g) : Conv3x3Bf16Form{16, 1, false};
    if (c.cls == 16) c.order = kChunk16;
    else if (converted && form.chunk > 0) c.order = form.parts > 1 ? kHalves : form.chunk / 16;
    else c.order = std::max(16, conv_bf16_chunk(ci, co, 3, g)) / 16;
    c.sum_emits = form.sum_emits;
    c.taken = takes(c, form, ci, co, g);
    return c;
}

struct C3nLaunch {
    C3nArgs a;
    int cls, nt, passes, order;  // cls: 16, 32 or 64 channels
    bool gen, whole, owes;       // owes: leaves no statistics where conv3x3_bf16 would
    dim3 grid;
    size_t lds_bytes;
};

// What no plan leads to is not compiled: tiles of 32 pixels by twos mean at least 512 partial results, beyond what
// conv3x3_bf16_narrow_merges allows (a filter converted here allows them from half the blocks on); from 17 channels on a whole
// block of theirs is more than one staging pass.
template <int NT, int CH, int PASSES, int ORDER, bool W32 = false, bool GEN_ONLY = false>
void launch_order(Ctx &cx, const C3nLaunch &L) {
    constexpr bool kMerges = PASSES == 1 && (NT == 1 || W32), kEmits = !(NT == 2 && PASSES == 1 && CH > 16);
#define RVN_RUN(G_, E_, M_) cx.run(conv3x3_bf16_narrow_k<NT, CH, PASSES, G_, E_, W32, ORDER, M_>, L.grid, dim3(kThreads), L.lds_bytes, L.a)
    if constexpr (GEN_ONLY) {
        RVN_RUN(true, false, false);
    } else {
        if (L.a.merge.blocks > 0) {
            if constexpr (kMerges) {
                if (L.a.emit) RVN_RUN(false, true, true);
                else RVN_RUN(false, false, true);
            } else {
                cx.fail(hipErrorInvalidConfiguration);
            }
        } else if (L.gen) {
            RVN_RUN(true, false, false);
        } else if (L.a.emit) {
            if constexpr (kEmits) RVN_RUN(false, true, false);
            else cx.fail(hipErrorInvalidConfiguration);
        } else {
            RVN_RUN(false, false, false);
        }
    }
#undef RVN_RUN
}

// More than 16 channels: a filter that has not been converted, and the general kernel's chunk of 64, come with ragged
// channel counts or rows only, the chunk of 32 in the 64-channel class too (32 channels that become more are a
// subsampling block's, which has a strided kernel).
template <int NT, int CH, int PASSES>
void launch_c3n(Ctx &cx, const C3nLaunch &L) {
    if constexpr (CH == 16) {
        if (L.a.wq) launch_order<NT, CH, PASSES, kChunk16>(cx, L);
        else launch_order<NT, CH, PASSES, kChunk16, true>(cx, L);
    } else {
        if constexpr (CH == 64) {
            if (L.order == kHalves) return launch_order<NT, CH, PASSES, kHalves>(cx, L);
            if (L.order == kChunk64)
                return L.a.wq ? launch_order<NT, CH, PASSES, kChunk64, false, true>(cx, L) : launch_order<NT, CH, PASSES, kChunk64, true, true>(cx, L);
        }
        if (L.order == kChunk32)
            return L.a.wq ? launch_order<NT, CH, PASSES, kChunk32, false, CH == 64>(cx, L) : launch_order<NT, CH, PASSES, kChunk32, true, true>(cx, L);
        if (L.a.wq) launch_order<NT, CH, PASSES, kChunk16>(cx, L);
        else launch_order<NT, CH, PASSES, kChunk16, true, true>(cx, L);
    }
}

bool plan_launch(View in, const float *scale_shift, const float *w, const uint16_t *wq, int ci, int co, Geo g, Epilogue ep,
                 const View *r, View out, C3nLaunch &L) {
    const C3nChoice c = choose(ci, co, g, wq != nullptr);
    if (!c.taken) return false;
    const C3nPlan &pl = c.pl;
    L.cls = c.cls; L.nt = c.nt; L.order = c.order;
    // bytes from the base to the end of the last plane; every one must end below kNowhere
    const int64_t in_b = 4 * ((g.n - 1) * in.sn + (ci - 1) * in.sc + g.hw()), out_b = 4 * ((g.n - 1) * out.sn + (co - 1) * out.sc + g.hw());
    const int64_t r_b = r ? 4 * ((g.n - 1) * r->sn + (co - 1) * r->sc + g.hw()) : 0;
    if (std::max(std::max(in_b, out_b), r_b) >= (int64_t)kNowhere) return false;
    C3nArgs a{};
    a.in = in.p; a.scale_shift = scale_shift; a.wq = wq; a.w = w; a.r = r ? r->p : nullptr; a.out = out.p;
    a.isn = (uint32_t)in.sn; a.isc = (uint32_t)in.sc;
    a.rsn = r ? (uint32_t)r->sn : 0; a.rsc = r ? (uint32_t)r->sc : 0;
    a.osn = (uint32_t)out.sn; a.osc = (uint32_t)out.sc;
    a.CI = ci; a.CO = co; a.CIP = (ci + 7) / 8 * 8; a.ep = (int)ep;
    a.in_bytes = (uint32_t)in_b; a.out_bytes = (uint32_t)out_b; a.r_bytes = (uint32_t)r_b; a.w_bytes = (uint32_t)(wq ? co * 9 * a.CIP * 2 : co * ci * 36);
    a.s = pl.s;
    L.a = a;
    L.gen = g.w % 4 != 0 || ci % 8 != 0 || (!wq && L.cls != 16);
    L.whole = g.w % 4 == 0 && pl.s.quads == 8 * L.nt * (4 / chan_waves(L.cls)) && g.n % pl.s.IMGS == 0 && g.h % pl.s.TH == 0;
    L.passes = pl.passes;
    L.owes = wq && c.sum_emits && !(L.whole && !L.gen);
    // (64-channel class: no caller has these, see launch_c3n)
    if (L.cls > 16 && !L.gen && (L.order == kChunk64 || (L.cls == 64 && L.order == kChunk32))) return false;
    L.grid = dim3((unsigned)pl.blocks);
    L.lds_bytes = pl.lds_bytes;
    return true;
}

}  // namespace

// How a layer of dense tensors runs, for the tests: class (16, 32 or 64 channels), 32-pixel tiles a wavefront has, staging passes,
// whether the rows or channels are ragged, Order, whether every block is whole, whether the filter comes converted; in pairs of
// hexadecimal digits from the class down, or -1 (another kernel).  converted: -1 for what the driver does in a function of two
// such layers.
extern "C" int64_t rvn_conv3x3_bf16_narrow_form(int ci, int co, int n, int h, int w, int converted) {
    const Geo g{n, h, w};
    if (converted < 0) converted = (int64_t)ci * co * 9 >= 16384 || conv3x3_bf16_ok(ci, co, g);
    const uint16_t wq = 0;
    float f = 0.f;
    C3nLaunch L;
    if (!plan_launch(dense_view(&f, ci, g), &f, &f, converted ? &wq : nullptr, ci, co, g, EP_STORE, nullptr, dense_view(&f, co, g), L)) return -1;
    int64_t form = 0;
    for (int v : {L.cls, L.nt, L.passes, (int)L.gen, L.order, (int)(L.whole && !L.gen), converted}) form = form * 256 + v;
    return form;
}

// The merge in every workgroup costs reads of all partial results, against a launch of 3.8 to 4.7 us: 1.4 us for 16 KB (16
// channels, 8 images of 32x32, 64 workgroups), 3.4 for 57 KB (56, 128 of 8x8, 128 workgroups; 4.1 saved); so 64 KB at most.  The
// convolution's own partial results must find room beside them.
bool conv3x3_bf16_narrow_merges(const Ctx &cx, int ci, int co, Geo g, const EmittedStats &e) {
    const int cls = class_of(ci, co);
    if (cls == 0 || e.to_come || e.count != 64 || e.tiles % 2 != 0 || e.tiles * cls > 8192 || ci % 8 != 0 || g.w % 4 != 0) return false;
    return (size_t)(ci + co) * e.tiles * 2 <= cx.emit_floats;
}

// Where a forward pass does without converted filters: small layers of up to 16 channels whose statistics come from partial
// results, so that the launch which would merge them and convert the filters is not needed (3.8 us against 1.4 for the merge
// and some 0.6 in each of two convolutions).  Forward of nine blocks of 16 channels, 8 images of 32x32: 251 -> 240 us.
bool conv3x3_bf16_narrow_unconverted(const Ctx &cx, int ci, int co, Geo g, const EmittedStats &e) {
    return class_of(ci, co) == 16 && conv3x3_bf16_narrow_merges(cx, ci, co, g, e);
}

bool conv3x3_bf16_narrow_takes(View in, const float *scale_shift, const float *w, const uint16_t *wq, int ci, int co, Geo g,
                               Epilogue ep, const View *r, View out) {
    C3nLaunch L;
    return plan_launch(in, scale_shift, w, wq, ci, co, g, ep, r, out, L) && L.passes == 1 && !L.gen && (L.nt == 1 || !wq);
}

bool conv3x3_bf16_narrow(Ctx &cx, View in, const float *scale_shift, const float *w, const uint16_t *wq, int ci, int co, Geo g, Epilogue ep,
                         const View *r, View out) {
    C3nLaunch L;
    if (!plan_launch(in, scale_shift, w, wq, ci, co, g, ep, r, out, L)) return false;
    const int tiles = (int)((int64_t)g.pixels() / 64);
    float *emit = cx.emit_buf;
    if (cx.deferred.blocks > 0) {  // (conv_fwd has made sure that this launch can merge)
        L.a.merge = cx.deferred;
        cx.deferred = StatsMerge{};
        // partial results are read and written by one launch: not in the same place
        if (emit && (size_t)(L.a.merge.partials - emit) < (size_t)co * tiles * 2) emit = const_cast<float *>(L.a.merge.partials) + (size_t)ci * L.a.merge.tiles * 2;
    }
    // (not for ragged channel counts, as in conv1x1_bf16)
    if (cx.want_emit && emit && !L.gen && L.whole && (size_t)(emit - cx.emit_buf) + (size_t)co * tiles * 2 <= cx.emit_floats) {
        L.a.emit = emit;
        L.a.emit_tiles = tiles;
        cx.emitted = EmittedStats{out.p, out.sn, out.sc, co, g.n, g.h, g.w, tiles, 64, emit};
    } else if (cx.want_emit && cx.emit_buf && L.owes && (size_t)co * tiles * 2 <= cx.emit_floats) {
        // Blocks that are not whole tiles, in a layer whose tiles the split launch would have left: they come from the
        // statistics pass, so that the layers behind see the same bits.
        cx.emitted = EmittedStats{out.p, out.sn, out.sc, co, g.n, g.h, g.w, tiles, 64, nullptr, true};
    }
#define RVN_CASE(NT_, CH_, P_) \
    if (L.cls == CH_ && L.nt == NT_ && L.passes == P_) launch_c3n<NT_, CH_, P_>(cx, L);
    // (one tile of up to 16 channels is at most 192 staging items: one pass)
    RVN_CASE(1, 16, 1) RVN_CASE(2, 16, 1) RVN_CASE(2, 16, 2)
    RVN_CASE(1, 32, 1) RVN_CASE(1, 32, 2) RVN_CASE(2, 32, 1) RVN_CASE(2, 32, 2)
    RVN_CASE(1, 64, 1) RVN_CASE(1, 64, 2) RVN_CASE(2, 64, 1) RVN_CASE(2, 64, 2)
#undef RVN_CASE
    return true;
}

}  // namespace rvn
