// fp32 filter gradient as a tiled matrix product over the flat pixel index, for layers of more channels
// than the row-band kernel's 16x16 tiles serve well (the rule is in conv_wgrad_gemm_f32).
//
// GEMM view.  dW[ko][c][tap] = sum_p dh[ko][p] * a[c][p + d(tap)] with p = (n * H + row) * W + col over the
// whole batch and d(tap) = (r - 1) * W + (s - 1): the reduction runs over flat pixels in chunks of 64, so
// no image side, row length or alignment is padded, and a chunk's operands are runs of 64 (dh) and
// 64 + 2W + 2 (a) consecutive values per channel.  A tap that leaves the image is a zero of `a`: a nine-bit
// mask per pixel, made once per chunk, is spread to an all-ones / all-zeros word and ANDed to the operand.
//
// Pipeline.  One v_mfma_f32_32x32x2_f32 takes 64 cycles for two operand words; the next chunk is requested
// into registers before the matrix instructions of the present one.  A 3x3 wavefront holds one 32x32 tile for all nine taps (144
// accumulators) and the workgroup's four wavefronts share the tile and split the pixels, which costs no
// partial results in memory; a 1x1 wavefront holds 2x2 tiles, because with one tap the words staged per
// flop would otherwise exceed what the last-level cache delivers.  Slices of the pixels go to further
// workgroups until two are resident per compute unit, or as many as the caller's scratch has room for;
// their partial results are summed by wgrad_reduce_body in a fixed order (no floating-point atomics).
//
// What bounds it (four-stage network, 16 images, parts left out as a measurement): not the loads.  3x3, 448
// workgroups: 51 us, 50 without the loads, 47 without the LDS writes as well, for 24 of matrix work: the matrix loop (an
// operand read, a mask and a wait per tap) and the sums at the end.  1x1, 272 workgroups: 31, 31 and 27 us for 5.3 of
// matrix work: one LDS buffer and two barriers a chunk, 32 operands that each wait for LDS, and the partial results;
// its 64-bit channel bases do not fit the scalar registers either (97 to 279 spills).
//
// Measured (mean over the layers of the four-stage bottleneck network, 16 images; the row-band kernel
// before): 1x1 95 -> 32 us, 3x3 111 -> 61 us; 28 -> 28 3x3 at 19x21, 51 images: 21.7 -> 15.5 us.
#include <algorithm>

#include "flat_pixels.h"

namespace rvn {

namespace {

using namespace flat;

typedef float float16_t __attribute__((ext_vector_type(16)));

constexpr int kThreads = 256;
constexpr int kWaves = 4;
constexpr int kChunk = 64;  // pixels per chunk

struct WgemmArgs {
    const float *x;            // layer input
    const float *scale_shift;  // [2*CI]: a = max(x*scale + shift, 0)
    const float *dh;           // upstream gradient
    float *part;
    uint32_t xsn, xsc, dsn, dsc;
    int P, HW, W, H, CI, CO;
    int slices, groups, tiles_c;
    int chunks_per_slice, chunks;
    int part_stride;
    uint32_t m_hw, m_w;
};

constexpr int lds_floats(int ks, int rows_a, int rows_b, int seg, int tiles) {
    // odd pitches: the 32 rows an operand read touches fall into different banks
    const int stage = rows_a * (kChunk + 1) + rows_b * (seg * 64 + 1) + kChunk;
    const int sum = (ks == 3 ? 3 : tiles) * 1024 * kWaves;  // shares of three taps / of the tiles, added at the end
    return sum > stage ? sum : stage;
}

// MW x CW x KW wavefronts, each with MT x CT tiles of 32x32 (ko, c) for all taps.
template <int KS, int MT, int CT, int MW, int CW, int KW, int SEG>
__global__ __launch_bounds__(kThreads, 2) void conv_wgrad_gemm_f32_k(const WgemmArgs p) {
    static_assert(MW * CW * KW == kWaves && KW > 1, "four wavefronts, the pixels shared");
    constexpr int KS2 = KS * KS, NTILE = MT * CT;
    constexpr int RA = MT * MW * 32, RB = CT * CW * 32;  // channels of dh / of a in the workgroup's tile
    constexpr int PA = kChunk + 1, PB = SEG * 64 + 1;
    constexpr int AI = RA / kWaves, BI = RB / kWaves;    // channels a wavefront stages
    extern __shared__ __align__(16) float smem[];
    float *a_lds = smem, *b_lds = smem + RA * PA;
    uint32_t *masks = reinterpret_cast<uint32_t *>(smem + RA * PA + RB * PB);

    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    // the tiles of one slice are consecutive modulo the slices: they read the same pixels at about the same time
    const int slice = blockIdx.x % p.slices, grp = blockIdx.x / p.slices;
    const int gy = grp / p.tiles_c, gz = grp - gy * p.tiles_c;
    const int ko0 = gy * RA, c0 = gz * RB;
    const int ch_begin = slice * p.chunks_per_slice, ch_end = min(p.chunks, ch_begin + p.chunks_per_slice);
    const int halo = KS == 3 ? p.W + 1 : 0;

    const int kw = wave % KW, cw = (wave / KW) % CW, mw = wave / (KW * CW);
    const int l32 = lane & 31, kg = lane >> 5;

    float16_t acc[NTILE][KS2];
#pragma unroll
    for (int t = 0; t < NTILE; ++t)
#pragma unroll
        for (int k = 0; k < KS2; ++k)
#pragma unroll
            for (int i = 0; i < 16; ++i) acc[t][k][i] = 0.f;

    float av[AI], bv[BI][SEG];
    uint32_t mask = 0;
    bool live = false;            // this lane's pixel of the chunk lies in the batch
    bool live_b[SEG];
    // Every load is issued, from the channel's first element where the pixel lies outside the batch and
    // from the last channel where the tile reaches past it.
    auto request = [&](int chunk) {
        const int q0 = chunk * kChunk;
        {
            const int q = q0 + lane;
            live = q < p.P;
            const int qq = live ? q : 0;
            const int n = div_u(qq, p.HW, p.m_hw), rem = qq - n * p.HW;
            const uint32_t off = (uint32_t)n * p.dsn + (uint32_t)rem;
#pragma unroll
            for (int i = 0; i < AI; ++i) {
                const int ko = min(ko0 + wave + i * kWaves, p.CO - 1);
                const char *base = reinterpret_cast<const char *>(p.dh + (size_t)ko * p.dsc);  // uniform
                av[i] = *reinterpret_cast<const float *>(base + off * 4u);
            }
            if (KS == 3) {
                const int row = div_u(rem, p.W, p.m_w), col = rem - row * p.W;
                const uint32_t cols = (col > 0 ? 1u : 0u) | 2u | (col + 1 < p.W ? 4u : 0u);
                mask = live ? (row > 0 ? cols : 0u) | cols << 3 | (row + 1 < p.H ? cols << 6 : 0u) : 0u;
            }
        }
        uint32_t off[SEG];
#pragma unroll
        for (int s = 0; s < SEG; ++s) {
            const int q = q0 - halo + s * 64 + lane;
            live_b[s] = q >= 0 && q < p.P;
            const int qq = live_b[s] ? q : 0;
            const int n = div_u(qq, p.HW, p.m_hw);
            off[s] = (uint32_t)n * p.xsn + (uint32_t)(qq - n * p.HW);
        }
#pragma unroll
        for (int i = 0; i < BI; ++i) {
            const int ch = min(c0 + wave + i * kWaves, p.CI - 1);
            const char *base = reinterpret_cast<const char *>(p.x + (size_t)ch * p.xsc);  // uniform
#pragma unroll
            for (int s = 0; s < SEG; ++s) bv[i][s] = *reinterpret_cast<const float *>(base + off[s] * 4u);
        }
    };
    auto commit = [&]() {
#pragma unroll
        for (int i = 0; i < AI; ++i) a_lds[(wave + i * kWaves) * PA + lane] = live ? av[i] : 0.f;
#pragma unroll
        for (int i = 0; i < BI; ++i) {
            const int ch = min(c0 + wave + i * kWaves, p.CI - 1);
            const float sc = p.scale_shift[ch], sh = p.scale_shift[p.CI + ch];
#pragma unroll
            for (int s = 0; s < SEG; ++s)
                b_lds[(wave + i * kWaves) * PB + s * 64 + lane] = live_b[s] ? fmaxf(fmaf(bv[i][s], sc, sh), 0.f) : 0.f;
        }
        if (KS == 3 && wave == 0) masks[lane] = mask;
    };

    if (ch_begin < ch_end) request(ch_begin);
    for (int ch = ch_begin; ch < ch_end; ++ch) {
        __syncthreads();  // the previous chunk has been consumed
        commit();
        __syncthreads();
        if (ch + 1 < ch_end) request(ch + 1);
#pragma unroll 2
        for (int s = 0; s < kChunk / 2 / KW; ++s) {
            const int px = (kw * (kChunk / 2 / KW) + s) * 2 + kg;
            float a[MT];
#pragma unroll
            for (int m = 0; m < MT; ++m) a[m] = a_lds[((mw * MT + m) * 32 + l32) * PA + px];
            const uint32_t ok = KS == 3 ? masks[px] : 0u;
#pragma unroll
            for (int tap = 0; tap < KS2; ++tap) {
#pragma unroll
                for (int c = 0; c < CT; ++c) {
                    float b = b_lds[((cw * CT + c) * 32 + l32) * PB + px + (KS == 3 ? (tap / KS) * p.W + tap % KS : 0)];
                    if (KS == 3) b = __uint_as_float(__float_as_uint(b) & (uint32_t)((int32_t)(ok << (31 - tap)) >> 31));
#pragma unroll
                    for (int m = 0; m < MT; ++m)
                        acc[m * CT + c][tap] = __builtin_amdgcn_mfma_f32_32x32x2f32(a[m], b, acc[m * CT + c][tap], 0, 0, 0);
                }
            }
        }
    }

    // ---- the workgroup's partial result in register order [tile][tap][register][lane]; the shares of the
    //      wavefronts that split the pixels are added in order
    float *out = p.part + (int64_t)slice * p.part_stride + (int64_t)grp * (MW * CW * NTILE * KS2 * 1024);
    // rounds of RT results per wavefront: three taps of the one tile, or all tiles of the one tap
    constexpr int RT = KS == 3 ? 3 : NTILE;
    static_assert(KS == 1 || NTILE == 1, "one tile per wavefront for 3x3");
#pragma unroll
    for (int rnd = 0; rnd < NTILE * KS2 / RT; ++rnd) {
        __syncthreads();
#pragma unroll
        for (int j = 0; j < RT; ++j) {
            const int t = KS == 3 ? 0 : j, k = KS == 3 ? rnd * 3 + j : 0;
#pragma unroll
            for (int i = 0; i < 16; ++i) smem[((wave * RT + j) * 16 + i) * 64 + lane] = acc[t][k][i];
        }
        __syncthreads();
        for (int e = tid; e < MW * CW * RT * 1024; e += kThreads) {
            const int own = e / (RT * 1024), rest = e - own * (RT * 1024);  // own: (mw, cw) pair
            const float *src = smem + (own * KW) * RT * 1024 + rest;
            float v = src[0];
#pragma unroll
            for (int k = 1; k < KW; ++k) v += src[k * RT * 1024];
            const int j = rest >> 10, t = KS == 3 ? 0 : j, k = KS == 3 ? rnd * 3 + j : 0;
            const int tl = ((own / CW) * MT + t / CT) * (CW * CT) + (own % CW) * CT + t % CT;
            out[(tl * KS2 + k) * 1024 + (rest & 1023)] = v;
        }
    }
}

// Tiles (in 32s) of a workgroup for 1x1 filters: the shapes conv_wgrad_gemm_f32 launches.
struct Tile {
    int m, c;
};
constexpr Tile kTiles1[] = {{2, 4}, {4, 2}, {2, 2}, {1, 1}};

struct WgemmPlan {
    int shape, m, c, seg, groups, tiles_ko, tiles_c, slices, chunks, per_slice, part_stride;
    bool ok;
};

WgemmPlan plan(int cin, int cout, int ks, const Geo &g, size_t scratch_floats) {
    WgemmPlan w{};
    const int seg = ks == 3 ? (kChunk + 2 * g.w + 2 + 63) / 64 : 1;
    if (seg > 4) return w;  // rows too wide for the staged runs
    // 16 channels on either side leave half of a 32x32 tile idle, and up to 32 in rows of whole 4-pixel
    // groups a 3x3 layer's two gradients share a launch of the row-band kernels (1x1 layers: see conv_gemm_f32.hip).
    if (std::min(cin, cout) <= 16 || (std::max(cin, cout) <= 32 && (g.w & 3) == 0)) return w;
    w.seg = seg;
    w.m = w.c = 1;
    w.shape = 3;
    if (ks == 1) {  // least padding first, then the largest tile
        int64_t best = -1;
        for (int i = 0; i < 4; ++i) {
            const int bm = kTiles1[i].m * 32, bc = kTiles1[i].c * 32;
            const int64_t area = (int64_t)((cout + bm - 1) / bm * bm) * ((cin + bc - 1) / bc * bc);
            if (best < 0 || area < best) {
                best = area;
                w.shape = i;
                w.m = kTiles1[i].m;
                w.c = kTiles1[i].c;
            }
        }
    }
    w.tiles_ko = (cout + w.m * 32 - 1) / (w.m * 32);
    w.tiles_c = (cin + w.c * 32 - 1) / (w.c * 32);
    w.groups = w.tiles_ko * w.tiles_c;
    if ((int64_t)w.groups * w.m * w.c * ks * ks * 1024 > 0x7fffffff) return w;  // a partial result is indexed in 32 bits
    w.part_stride = w.groups * w.m * w.c * ks * ks * 1024;
    w.chunks = (int)((g.pixels() + kChunk - 1) / kChunk);
    int s = std::max(1, 512 / w.groups);  // two workgroups per compute unit
    s = std::min(s, std::max(1, w.chunks / 2));
    // The scratch is sized for the row-band and bf16 kernels.  One partial result of the row-band kernel is as
    // large as one of these (the tile chosen above pads no more than 32x32 does), so one always fits; fewer
    // than wished fit only for a few pixels or rows of up to three (33 -> 263 channels, 70 images of 8x2).
    s = (int)std::min<size_t>(s, scratch_floats / (size_t)w.part_stride);
    if (s < 1) return w;
    w.per_slice = (w.chunks + s - 1) / s;
    w.slices = (w.chunks + w.per_slice - 1) / w.per_slice;
    w.ok = true;
    return w;
}

template <int KS, int MT, int CT, int MW, int CW, int KW, int SEG>
void run_one(Ctx &cx, const WgemmArgs &a) {
    const size_t lds = (size_t)lds_floats(KS, MT * MW * 32, CT * CW * 32, SEG, MT * CT) * 4;
    cx.run(conv_wgrad_gemm_f32_k<KS, MT, CT, MW, CW, KW, SEG>, dim3((unsigned)(a.slices * a.groups)), dim3(kThreads), lds, a);
}

}  // namespace

extern "C" int rvn_conv3x3_f32_bwd_form(int cin, int cout, int n, int h, int w);

// Which instance a layer of dense tensors runs on given the scratch it is planned with, for the tests: ks * 8 + pieces (3x3) or
// tile shape (1x1), or -1 (another kernel, that of both gradients among them).
extern "C" int rvn_conv_wgrad_gemm_f32_instance(int cin, int cout, int ks, int n, int h, int w) {
    const Geo g{n, h, w};
    if (ks == 3 && rvn_conv3x3_f32_bwd_form(cin, cout, n, h, w) >= 0) return -1;
    const WgemmPlan p = plan(cin, cout, ks, g, wgrad_scratch_floats(cin, cout, ks, g));
    return p.ok ? ks * 8 + (ks == 3 ? p.seg : p.shape) : -1;
}

bool conv_wgrad_gemm_f32(Ctx &cx, View x, const float *scale_shift, View dh, int cin, int cout, int ks, Geo g,
                         float *scratch, size_t scratch_floats, float *dw, bool accumulate, double bytes, double flops,
                         WgradReduce *defer) {
    if (!fits(x, cin, g) || !fits(dh, cout, g)) return false;
    const WgemmPlan w = plan(cin, cout, ks, g, scratch_floats);
    if (!w.ok) return false;
    WgradReduce red{};
    red.part = scratch; red.dw = dw;
    red.part_stride = w.part_stride; red.S = w.slices; red.KS2 = ks * ks; red.MT = w.m; red.CT = w.c;
    red.tiles_c = w.tiles_c; red.CO = cout; red.CI = cin; red.accumulate = accumulate ? 1 : 0;
    red.tile = 32; red.wide = w.slices <= 16 ? 1 : 0;
    red.blocks = red.wide ? (w.part_stride + 255) / 256 : (w.part_stride + 31) / 32;
    if (cx.launch(K_CONV_WGRAD, bytes, flops)) {
        WgemmArgs a{};
        a.x = x.p; a.scale_shift = scale_shift; a.dh = dh.p; a.part = scratch;
        a.xsn = (uint32_t)x.sn; a.xsc = (uint32_t)x.sc; a.dsn = (uint32_t)dh.sn; a.dsc = (uint32_t)dh.sc;
        a.P = (int)g.pixels(); a.HW = g.hw(); a.W = g.w; a.H = g.h; a.CI = cin; a.CO = cout;
        a.slices = w.slices; a.groups = w.groups; a.tiles_c = w.tiles_c;
        a.chunks = w.chunks; a.chunks_per_slice = w.per_slice; a.part_stride = w.part_stride;
        a.m_hw = magic(a.HW); a.m_w = magic(a.W);
        if (ks == 3) {
            if (w.seg == 2) run_one<3, 1, 1, 1, 1, 4, 2>(cx, a);
            else if (w.seg == 3) run_one<3, 1, 1, 1, 1, 4, 3>(cx, a);
            else run_one<3, 1, 1, 1, 1, 4, 4>(cx, a);
        } else {
            if (w.shape == 0) run_one<1, 2, 2, 1, 2, 2, 1>(cx, a);
            else if (w.shape == 1) run_one<1, 2, 2, 2, 1, 2, 1>(cx, a);
            else if (w.shape == 2) run_one<1, 2, 2, 1, 1, 4, 1>(cx, a);
            else run_one<1, 1, 1, 1, 1, 4, 1>(cx, a);
        }
    }
    if (defer) *defer = red;
    else wgrad_reduce(cx, red);
    return true;
}

}  // namespace rvn
