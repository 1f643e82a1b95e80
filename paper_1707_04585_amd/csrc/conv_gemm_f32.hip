// fp32 convolution (forward and data gradient) as a tiled matrix product over the flat pixel index, for
// the layers whose output channels fill 32-row matrix tiles (the rule is in conv_gemm_f32).
//
// GEMM view.  D[ko][p] = sum_k Wt[ko][k] * A[k][p] with p = (n * H + row) * W + col running over all
// pixels of the batch: a tile is BN consecutive pixels, whatever the image sides are, so nothing is
// padded to rows, images or 4-pixel groups, and one form serves every width and alignment.  A tap of a
// 3x3 filter is the constant distance (r - 1) * W + (s - 1) along p, so a workgroup stages, per input
// channel, the BN + 2W + 2 consecutive values its tile can touch, in whole pieces of 64 (2.0 loads per pixel
// and channel for BN = 128, at 56 columns and at 14 alike: what lies past them is loaded and not used); the taps
// that leave the image read a zero kept at the end of each staged plane, by one address select per tap and tile.
//
// Pipeline.  v_mfma_f32_32x32x2_f32 takes 64 cycles for two operand words per lane.  The next chunk's
// activations and filters are requested into registers before the matrix instructions of the present one and
// written to the other LDS buffer after them (one barrier per chunk).  A lane's pixel offset is fixed for the
// whole kernel and the channel is wavefront-uniform, so a staged element costs one load with a scalar base, one
// fma, one max and one LDS write.  Where the output is small, a workgroup's wavefronts share one tile and split
// the channels (KW), summed through LDS in a fixed order, instead of leaving compute units idle.
//
// What bounds it, by leaving parts out (four-stage network, 16 images; 3x3, 3.7 GFLOP a layer, 64 x 128 tiles):
//                                    128 -> 128 at 28x28,    64 -> 64 at 56x56,
//                                    200 workgroups          392 workgroups
//   whole kernel                     57 us                   51 us
//   without the loads                55                      51
//   and without the LDS writes       49                      48
//   and without the tap selects      46                      45
//   matrix instructions alone        31                      31
// so most of it is the matrix loop itself (operand reads and their waits, barriers, prologue, epilogue), not the
// memory round trip.  The small tiles do wait for memory: without the loads the 512 -> 512 layer at 7x7 takes 67 us
// of 81, 1x1 layers with 64-channel chunks 20 to 23 of 28 to 50.
//
// Measured (mean over the layers of the four-stage 50176-pixel-to-784-pixel bottleneck network, 16 images;
// the row-band kernel before): 1x1 132 -> 28 us, 3x3 314 -> 73 us (the 512 -> 512 layer at 7x7 takes 113 us
// with 8-channel chunks, 81 with 16); 28 -> 28 3x3 at 19x21, 51 images: 25.7 -> 14.7 us.
#include <algorithm>
#include <cmath>

#include "flat_pixels.h"

namespace rvn {

namespace {

using namespace flat;

typedef float float16_t __attribute__((ext_vector_type(16)));

constexpr int kThreads = 256;
constexpr int kWaves = 4;
constexpr int kDies = 8;  // consecutive workgroup ids go to the dies (one L2 each) in turn

struct GemmArgs {
    const float *in;  // x (forward) or upstream gradient (data gradient)
    const float *scale_shift;  // [2*CI]: a = max(in*scale + shift, 0); null = use `in` as is
    const float *w;   // [CO][CI][KS][KS] forward; [CI][CO][KS][KS] read transposed and flipped otherwise
    const float *r;   // skip operand (may alias out)
    float *out;
    uint32_t isn, isc, rsn, rsc, osn, osc;
    int P, HW, W, H, CI, CO;
    int ep, transposed;
    int tiles_p, tiles_co, per_die;
    int co_major;     // a die gets a range of output channels (else a range of pixels)
    uint32_t m_hw, m_w;
};

// LDS of one buffer: the filter chunk [tap][channel][ko] with an odd pitch, then the staged planes.
constexpr int buffer_floats(int ks, int bm, int kc, int pb) { return kc * ks * ks * (bm + 1) + kc * pb; }

// MW x NW x KW wavefronts; a wavefront holds NT 32x32 tiles side by side along the pixels.
// KC: channels per chunk.  SEG: 64-position pieces of a staged plane; PB: its pitch (3x3: the last float is the zero).
template <int KS, int MW, int NW, int KW, int NT, int KC, int SEG, int PB>
__global__ __launch_bounds__(kThreads, 2) void conv_gemm_f32_k(const GemmArgs p) {
    static_assert(MW * NW * KW == kWaves, "four wavefronts");
    constexpr int KS2 = KS * KS, ZERO = PB - 1;
    constexpr int BM = MW * 32, BN = NW * NT * 32, PA = BM + 1;
    constexpr int A_ELEMS = BM * KC * KS2, AI = A_ELEMS / kThreads;
    static_assert(A_ELEMS % kThreads == 0, "whole filter items");
    constexpr int A_FLOATS = KC * KS2 * PA, BUF = buffer_floats(KS, BM, KC, PB);
    constexpr int CG = kWaves / SEG, BI = KC / CG;  // channel groups of the staging; channels a wavefront stages
    static_assert(kWaves % SEG == 0 && KC % CG == 0, "staging split");
    static_assert((KW - 1) * MW * NW * NT * 1024 <= 2 * BUF, "the sum over KW fits");
    extern __shared__ __align__(16) float smem[];

    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int work = (blockIdx.x % kDies) * p.per_die + blockIdx.x / kDies;
    if (work >= p.tiles_p * p.tiles_co) return;
    const int tile_co = p.co_major ? work / p.tiles_p : work % p.tiles_co;
    const int tile_p = p.co_major ? work - tile_co * p.tiles_p : work / p.tiles_co;
    const int co0 = tile_co * BM, p0 = tile_p * BN;
    const int halo = KS == 3 ? p.W + 1 : 0;

    // ---- staging of the activations: this lane's position, this wavefront's channels cg, cg + CG, ...
    const int seg = wave % SEG, cg = wave / SEG;
    const int pos = seg * 64 + lane;
    uint32_t b_off;  // element offset inside a channel, 0 outside the batch (never multiplied then)
    {
        const int q = p0 - halo + pos;
        const bool in = q >= 0 && q < p.P;
        const int n = in ? div_u(q, p.HW, p.m_hw) : 0;
        b_off = in ? (uint32_t)n * p.isn + (uint32_t)(q - n * p.HW) : 0u;
    }
    // ---- staging of the filter: element e = (output channel, input channel, tap), the input channel
    //      the slower one when transposed
    uint32_t a_off[AI];
    int a_dst[AI];
    const uint32_t s_ko = p.transposed ? (uint32_t)KS2 : (uint32_t)p.CI * KS2;
    const uint32_t s_ch = p.transposed ? (uint32_t)p.CO * KS2 : (uint32_t)KS2;
#pragma unroll
    for (int i = 0; i < AI; ++i) {
        const int e = tid + i * kThreads;
        const int o1 = e / (KC * KS2), r1 = e - o1 * (KC * KS2), i1 = r1 / KS2, t1 = r1 - i1 * KS2;
        const int o2 = e / (BM * KS2), r2 = e - o2 * (BM * KS2), i2 = r2 / KS2, t2 = r2 - i2 * KS2;
        const int kol = p.transposed ? i2 : o1, cl = p.transposed ? o2 : i1, t = p.transposed ? t2 : t1;
        const int tt = p.transposed ? KS2 - 1 - t : t;
        const int ko = min(co0 + kol, p.CO - 1);  // rows past the last channel are not stored
        a_off[i] = (uint32_t)ko * s_ko + (uint32_t)cl * s_ch + (uint32_t)t;
        a_dst[i] = (tt * KC + cl) * PA + kol;
    }
    // ---- operands of this wavefront
    const int kw = wave % KW, nw = (wave / KW) % NW, mw = wave / (KW * NW);
    const int l32 = lane & 31, kg = lane >> 5;
    uint32_t ok_taps[NT];  // bit tap: the tap lies inside the image
    int pix[NT];           // pixel index in the batch
#pragma unroll
    for (int t = 0; t < NT; ++t) {
        pix[t] = p0 + (nw * NT + t) * 32 + l32;
        ok_taps[t] = 0;
        if (KS == 3 && pix[t] < p.P) {
            const int n = div_u(pix[t], p.HW, p.m_hw), rem = pix[t] - n * p.HW;
            const int row = div_u(rem, p.W, p.m_w), col = rem - row * p.W;
            const uint32_t cols = (col > 0 ? 1u : 0u) | 2u | (col + 1 < p.W ? 4u : 0u);
            ok_taps[t] = (row > 0 ? cols : 0u) | cols << 3 | (row + 1 < p.H ? cols << 6 : 0u);
        }
    }
    float16_t acc[NT];
#pragma unroll
    for (int t = 0; t < NT; ++t)
#pragma unroll
        for (int i = 0; i < 16; ++i) acc[t][i] = 0.f;

    if (KS == 3)
        for (int e = tid; e < 2 * KC; e += kThreads) smem[(e / KC) * BUF + A_FLOATS + (e % KC) * PB + ZERO] = 0.f;

    float av[AI], bv[BI], sc[BI], sh[BI];  // sc, sh: wavefront-uniform
    const bool bn = p.scale_shift != nullptr;
    const char *const wb = reinterpret_cast<const char *>(p.w);
    auto request = [&](int c0) {
#pragma unroll
        for (int j = 0; j < BI; ++j) {
            const int ch = min(c0 + cg + j * CG, p.CI - 1);
            const char *base = reinterpret_cast<const char *>(p.in + (size_t)ch * p.isc);  // uniform
            bv[j] = *reinterpret_cast<const float *>(base + b_off * 4u);
        }
        if (bn) {
#pragma unroll
            for (int j = 0; j < BI; ++j) {
                const int ch = min(c0 + cg + j * CG, p.CI - 1);
                sc[j] = p.scale_shift[ch];
                sh[j] = p.scale_shift[p.CI + ch];
            }
        }
        const uint32_t step = (uint32_t)c0 * s_ch;
        if (c0 + KC <= p.CI) {
#pragma unroll
            for (int i = 0; i < AI; ++i) av[i] = *reinterpret_cast<const float *>(wb + (a_off[i] + step) * 4u);
        } else {  // the filter is zero past the last input channel
#pragma unroll
            for (int i = 0; i < AI; ++i) {
                const int cl = (a_dst[i] / PA) % KC;
                const float v = *reinterpret_cast<const float *>(wb + (c0 + cl < p.CI ? a_off[i] + step : 0u) * 4u);
                av[i] = c0 + cl < p.CI ? v : 0.f;
            }
        }
    };
    auto commit = [&](float *buf, int c0) {
#pragma unroll
        for (int i = 0; i < AI; ++i) buf[a_dst[i]] = av[i];
        if (bn) {
#pragma unroll
            for (int j = 0; j < BI; ++j) bv[j] = fmaxf(fmaf(bv[j], sc[j], sh[j]), 0.f);
        }
        if (SEG * 64 < PB || pos < (KS == 3 ? ZERO : PB)) {
#pragma unroll
            for (int j = 0; j < BI; ++j) {
                const int cl = cg + j * CG;
                buf[A_FLOATS + cl * PB + pos] = c0 + cl < p.CI ? bv[j] : 0.f;
            }
        }
    };

    request(0);
    commit(smem, 0);
    __syncthreads();
    int cur = 0;
    for (int c0 = 0; c0 < p.CI; c0 += KC) {
        const bool more = c0 + KC < p.CI;
        if (more) request(c0 + KC);
        const float *a_lds = smem + cur * BUF, *b_lds = a_lds + A_FLOATS;
        // Steps of two channels at one tap, G at a time: the operands of a group are read before the
        // matrix instructions of the group ahead of it are issued (left to itself the compiler reads them
        // right before their use, and a wavefront waits out the LDS latency every four instructions).
        constexpr int SPT = KC / 2 / KW, STEPS = KS2 * SPT, G = 4, GROUPS = (STEPS + G - 1) / G;
        float oa[2][G], ob[2][G][NT];
        auto operands = [&](int grp) {
#pragma unroll
            for (int u = 0; u < G; ++u) {
                const int step = grp * G + u, tap = step / SPT, c = (step % SPT * KW + kw) * 2;
                if (step >= STEPS) continue;
                oa[grp & 1][u] = a_lds[(tap * KC + c + kg) * PA + mw * 32 + l32];
#pragma unroll
                for (int t = 0; t < NT; ++t) {
                    const int own = (nw * NT + t) * 32 + l32;
                    const int at = KS == 1 ? own : (ok_taps[t] >> tap & 1u) ? own + (tap / KS) * p.W + tap % KS : ZERO;
                    ob[grp & 1][u][t] = b_lds[c * PB + at + kg * PB];
                }
            }
        };
        operands(0);
#pragma unroll
        for (int grp = 0; grp < GROUPS; ++grp) {
            if (grp + 1 < GROUPS) operands(grp + 1);
            __builtin_amdgcn_sched_barrier(0);
#pragma unroll
            for (int u = 0; u < G; ++u)
                if (grp * G + u < STEPS)
#pragma unroll
                    for (int t = 0; t < NT; ++t)
                        acc[t] = __builtin_amdgcn_mfma_f32_32x32x2f32(oa[grp & 1][u], ob[grp & 1][u][t], acc[t], 0, 0, 0);
            __builtin_amdgcn_sched_barrier(0);
        }
        if (more) commit(smem + (cur ^ 1) * BUF, c0 + KC);
        __syncthreads();
        cur ^= 1;
    }

    if (KW > 1) {  // shares 1 .. KW-1 through LDS, added in order by share 0
        const int mn = mw * NW + nw;
        if (kw > 0) {
            float *dst = smem + ((kw - 1) * MW * NW + mn) * NT * 1024 + lane;
#pragma unroll
            for (int t = 0; t < NT; ++t)
#pragma unroll
                for (int i = 0; i < 16; ++i) dst[(t * 16 + i) * 64] = acc[t][i];
        }
        __syncthreads();
        if (kw > 0) return;
#pragma unroll
        for (int k = 1; k < KW; ++k) {
            const float *src = smem + ((k - 1) * MW * NW + mn) * NT * 1024 + lane;
#pragma unroll
            for (int t = 0; t < NT; ++t)
#pragma unroll
                for (int i = 0; i < 16; ++i) acc[t][i] += src[(t * 16 + i) * 64];
        }
    }

    // ---- epilogue: register i of a lane is channel 8 * (i / 4) + 4 * kg + i % 4 of its pixel; every skip
    //      value is requested before the first store (r may alias out element for element)
    const int kb = co0 + mw * 32 + 4 * kg;
#pragma unroll
    for (int t = 0; t < NT; ++t) {
        const bool okp = pix[t] < p.P;
        const int n = okp ? div_u(pix[t], p.HW, p.m_hw) : 0;
        const uint32_t rem = okp ? (uint32_t)(pix[t] - n * p.HW) : 0u;
        const uint32_t o = (uint32_t)n * p.osn + rem, ro = (uint32_t)n * p.rsn + rem;
        if (p.ep != EP_STORE) {
            float rv[16];
#pragma unroll
            for (int i = 0; i < 16; ++i) {
                const int ko = min(kb + 8 * (i >> 2) + (i & 3), p.CO - 1);
                rv[i] = *reinterpret_cast<const float *>(reinterpret_cast<const char *>(p.r) + (ro + (uint32_t)ko * p.rsc) * 4u);
            }
#pragma unroll
            for (int i = 0; i < 16; ++i) acc[t][i] = p.ep == EP_ADD ? rv[i] + acc[t][i] : rv[i] - acc[t][i];
        }
#pragma unroll
        for (int i = 0; i < 16; ++i) {
            const int ko = kb + 8 * (i >> 2) + (i & 3);
            if (okp && ko < p.CO)
                *reinterpret_cast<float *>(reinterpret_cast<char *>(p.out) + (o + (uint32_t)ko * p.osc) * 4u) = acc[t][i];
        }
    }
}

// A tile shape: BM = 32 * mw channels by BN = 32 * nw * nt pixels, channels split over kw wavefronts, kc
// channels per chunk.  Chunks of twice the channels halve the number of memory round trips in the chain of
// a workgroup; they fit where the other tile side is small.
struct Shape {
    int ks, mw, nw, kw, nt, kc;
    int bm() const { return 32 * mw; }
    int bn() const { return 32 * nw * nt; }
};
constexpr Shape kShapes[] = {
    {3, 2, 2, 1, 2, 8}, {3, 2, 2, 1, 1, 8}, {3, 1, 4, 1, 1, 8}, {3, 1, 2, 2, 1, 8}, {3, 1, 1, 4, 1, 8},
    {3, 1, 4, 1, 1, 16}, {3, 1, 2, 2, 1, 16}, {3, 1, 1, 4, 1, 16},
    {1, 2, 2, 1, 2, 32}, {1, 2, 2, 1, 1, 32}, {1, 1, 4, 1, 1, 32}, {1, 1, 2, 2, 1, 64}, {1, 1, 1, 4, 1, 64},
};

// Pieces and pitch of a staged plane; seg = 0: rows too wide for this shape.  The pitch is 32 modulo 64, so
// that the two channels a matrix instruction reads lie in different halves of the banks (64-channel chunks
// of a 1x1 filter give that up for LDS).
struct Plane {
    int seg, pb;
};
Plane plane_of(const Shape &s, int w) {
    if (s.ks == 1) return {(s.bn() + 63) / 64, (s.bn() + 63) / 64 * 64 + (s.kc == 64 ? 0 : 32)};
    const int need = s.bn() + 2 * w + 2;
    if (need <= 64) return {1, 96};
    if (need <= 128) return {2, 160};
    if (need <= 159 && s.kc == 16) return {4, 160};
    if (need <= 256 && s.kc == 8) return {4, 288};
    return {0, 0};
}

// The tile shape with the smallest estimated time in cycles.  A compute unit holds two workgroups at a
// time; they take the larger of their matrix and staging work (256 flop and 16 bytes per cycle) and of one
// workgroup's chain of chunks, each a memory round trip (taken as 3500 cycles) or its matrix work.  It ranks the
// shapes and does not predict times: 35 and 42 us for the two layers above that take 57 and 51.
int choose_shape(const Geo &g, int ci, int co, int ks) {
    int best = -1;
    double best_cost = 0.0;
    for (int i = 0; i < (int)(sizeof kShapes / sizeof kShapes[0]); ++i) {
        const Shape &s = kShapes[i];
        const Plane pl = plane_of(s, g.w);
        if (s.ks != ks || pl.seg == 0) continue;
        const int64_t wgs = ((g.pixels() + s.bn() - 1) / s.bn()) * ((co + s.bm() - 1) / s.bm());
        const double chunks = (double)((ci + s.kc - 1) / s.kc), rounds = (double)((wgs + 255) / 256);
        const double matrix = (double)s.bm() * s.bn() * s.kc * ks * ks * 2.0 / 256.0;
        const double staged = s.kc * (s.bm() * ks * ks + pl.seg * 64.0) * 4.0 / 16.0;
        const double chain = chunks * (std::max(matrix, 3500.0) + 600.0), load = chunks * (matrix + staged);
        const double cost = std::ceil(rounds / 2.0) * std::max(std::min(rounds, 2.0) * load, chain);
        if (best < 0 || cost < best_cost) {
            best = i;
            best_cost = cost;
        }
    }
    return best;
}

template <int I, int SEG, int PB>
bool launch_if(Ctx &cx, const GemmArgs &a, Plane pl, dim3 grid) {
    constexpr Shape s = kShapes[I];
    if (pl.seg != SEG || pl.pb != PB) return false;
    constexpr size_t lds = (size_t)2 * buffer_floats(s.ks, 32 * s.mw, s.kc, PB) * 4;
    static_assert(lds <= 64 * 1024, "LDS of a launch");
    cx.run(conv_gemm_f32_k<s.ks, s.mw, s.nw, s.kw, s.nt, s.kc, SEG, PB>, grid, dim3(kThreads), lds, a);
    return true;
}

bool launch_shape(Ctx &cx, const GemmArgs &a, int shape, Plane pl, dim3 grid) {
    switch (shape) {
        case 0: return launch_if<0, 4, 288>(cx, a, pl, grid);
        case 1: return launch_if<1, 2, 160>(cx, a, pl, grid) || launch_if<1, 4, 288>(cx, a, pl, grid);
        case 2: return launch_if<2, 4, 288>(cx, a, pl, grid);
        case 3: return launch_if<3, 2, 160>(cx, a, pl, grid) || launch_if<3, 4, 288>(cx, a, pl, grid);
        case 4: return launch_if<4, 4, 288>(cx, a, pl, grid);  // (shorter rows: shape 3, 6 or 7)
        case 5: return launch_if<5, 4, 160>(cx, a, pl, grid);
        case 6: return launch_if<6, 2, 160>(cx, a, pl, grid) || launch_if<6, 4, 160>(cx, a, pl, grid);
        case 7: return launch_if<7, 1, 96>(cx, a, pl, grid) || launch_if<7, 2, 160>(cx, a, pl, grid) || launch_if<7, 4, 160>(cx, a, pl, grid);
        case 8: return launch_if<8, 2, 160>(cx, a, pl, grid);
        case 9: return launch_if<9, 1, 96>(cx, a, pl, grid);
        case 10: return launch_if<10, 2, 160>(cx, a, pl, grid);
        case 11: return launch_if<11, 1, 64>(cx, a, pl, grid);
        case 12: return launch_if<12, 1, 64>(cx, a, pl, grid);
    }
    return false;
}

// Fewer than 17 channels would leave half of a 32-row tile idle; above, this kernel took a quarter to a half of the
// row-band kernel's time.  3x3 layers of up to 32 channels go to conv3x3_f32 first; what comes here is
// what its own rule leaves, and rows too long for it.  1x1 layers of up to 32 channels have neither advantage and stay there only because the line was drawn for
// 3x3: with them and their filter gradients here, two bottleneck blocks of 64 channels reduced to 32 take 884 us
// instead of 1196 (8 images of 28x28), of 128 to 32 2136 instead of 2302 (32 of 56x56), and no shape tried took longer.
bool takes(int co, const Geo &g) { return co > 32 || (co > 16 && (g.w & 3) != 0); }

}  // namespace

ConvGemmTile conv_gemm_f32_tile(int ci, int co, int ks, const Geo &g) {
    const int shape = takes(co, g) ? choose_shape(g, ci, co, ks) : -1;
    return shape < 0 ? ConvGemmTile{0, 0} : ConvGemmTile{kShapes[shape].bn(), kShapes[shape].kc};
}

extern "C" int rvn_conv3x3_f32_form(int ci, int co, int n, int h, int w);

// Which instance a layer of dense tensors runs on, for the tests: shape * 4096 + pieces * 512 + pitch, or -1 (another
// kernel, conv3x3_f32 among them).
extern "C" int rvn_conv_gemm_f32_instance(int ci, int co, int ks, int n, int h, int w) {
    const Geo g{n, h, w};
    if (ks == 3 && rvn_conv3x3_f32_form(ci, co, n, h, w) >= 0) return -1;
    const int shape = takes(co, g) ? choose_shape(g, ci, co, ks) : -1;
    if (shape < 0) return -1;
    const Plane pl = plane_of(kShapes[shape], w);
    return shape * 4096 + pl.seg * 512 + pl.pb;
}

bool conv_gemm_f32(Ctx &cx, View in, const float *scale_shift, const float *w, bool transposed, int ci, int co, int ks,
                   Geo g, Epilogue ep, const View *r, View out) {
    if (!takes(co, g)) return false;
    if (!fits(in, ci, g) || !fits(out, co, g) || (r && !fits(*r, co, g)) || (int64_t)ci * co * ks * ks >= kMaxElems) return false;
    const int shape = choose_shape(g, ci, co, ks);
    if (shape < 0) return false;  // rows too wide for the staged planes
    const Shape &s = kShapes[shape];
    GemmArgs a{};
    a.in = in.p; a.scale_shift = scale_shift; a.w = w; a.r = r ? r->p : nullptr; a.out = out.p;
    a.isn = (uint32_t)in.sn; a.isc = (uint32_t)in.sc;
    a.rsn = r ? (uint32_t)r->sn : 0; a.rsc = r ? (uint32_t)r->sc : 0;
    a.osn = (uint32_t)out.sn; a.osc = (uint32_t)out.sc;
    a.P = (int)g.pixels(); a.HW = g.hw(); a.W = g.w; a.H = g.h; a.CI = ci; a.CO = co;
    a.ep = (int)ep; a.transposed = transposed ? 1 : 0;
    a.tiles_p = (a.P + s.bn() - 1) / s.bn();
    a.tiles_co = (co + s.bm() - 1) / s.bm();
    // What the eight L2s fetch together: the filter eight times when a die owns pixels, the activations
    // eight times when it owns channels.
    a.co_major = (int64_t)ci * co * ks * ks > g.pixels() * ci ? 1 : 0;
    a.m_hw = magic(a.HW); a.m_w = magic(a.W);
    const int total = a.tiles_p * a.tiles_co;
    a.per_die = (total + kDies - 1) / kDies;
    const dim3 grid((unsigned)(a.per_die * kDies));
    if (!launch_shape(cx, a, shape, plane_of(s, g.w), grid)) cx.fail(hipErrorInvalidConfiguration);
    return true;
}

}  // namespace rvn
