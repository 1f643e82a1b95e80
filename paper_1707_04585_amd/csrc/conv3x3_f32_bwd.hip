// Data gradient and filter gradient of an fp32 3x3 layer of up to 32 channels in one workgroup (Algorithm 1: the
// "ordinary backprop" steps).
//
// Both need the upstream gradient dh with its halo, both cut the pixels into the same blocks: the set-up, the index
// arithmetic and the staging of dh are done once, and the matrix instructions of the two (144 each per wavefront and 16 x 16
// channels) follow each other without a wait.  The data gradient is the forward kernel's (conv3x3_f32_body.h).  In
// the filter gradient a lane holds one channel of each operand; its share of the reduction is a quad of
// consecutive pixels, so the operands of 36 matrix instructions are 10 16-byte and 18 4-byte LDS reads.  A workgroup
// keeps its partial filter in registers over all its blocks; the partial results are summed in a fixed order by
// wgrad_reduce_body in a later launch.  What bounds it is the same as there, one chain per workgroup, with 7.7 us of
// matrix instructions per SIMD at the size below.
//
// Measured, with row-band kernels beside each other in one launch before: 16 -> 16 channels at 128 of 32x32 23.7 -> 17.8 us
// (22.5 with the data gradient alone replaced); 28 -> 28 at 51 of 19x21 (two launches before) 30.2 -> 18.3 us.
#include <algorithm>
#include <cstdlib>

#include "conv3x3_f32_body.h"
#include "kernels.h"

namespace rvn {

namespace {

using namespace c3f;

enum Parts { kDgrad = 1, kWgrad = 2 };

struct B3fArgs {
    const float *x;            // layer input
    const float *scale_shift;  // [2*CI]: a = max(x*scale + shift, 0)
    const float *dh;           // upstream gradient
    const float *w;            // [CO][CI][3][3]
    float *da;                 // dense [n][CI][h*w]
    float *part;               // partial filter gradients [gridDim.x][part_stride]
    uint32_t xsn, xsc, dsn, dsc;
    uint32_t x_bytes, dh_bytes, w_bytes, da_bytes;
    int CI, CO, parts;
    int units, upw;            // pixel blocks in all and per workgroup
    int part_stride, tiles_c;
    int d_lds;                 // floats ahead of the second staged band
    C3fShape s;
};

// Workgroup (x, y, z): the blocks x * upw ... and the input channels 16 y ... 16 y + 15; z: which of the two gradients,
// where they have a workgroup each.  KT: chunks of 16 output channels.
template <int NW, int PASSES, int KT, bool VEC>
__global__ __launch_bounds__(64 * NW, 2) void conv3x3_f32_bwd_k(const B3fArgs p) {
    extern __shared__ __align__(16) float smem[];
    constexpr int kThreads = 64 * NW;
    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int l16 = lane & 15, kq = lane >> 4;
    const C3fShape &s = p.s;
    const int c0 = (int)blockIdx.y * 16;
    const int parts = gridDim.z == 1 ? p.parts : blockIdx.z == 0 ? kWgrad : kDgrad;
    const bool dgrad = parts & kDgrad, wgrad = parts & kWgrad;
    float *const x_lds = smem, *const d_lds = smem + p.d_lds;
    const __amdgpu_buffer_rsrc_t x_rs = rsrc(p.x, p.x_bytes), d_rs = rsrc(p.dh, p.dh_bytes), w_rs = rsrc(p.w, p.w_bytes);
    const __amdgpu_buffer_rsrc_t ss_rs = rsrc(p.scale_shift, (uint32_t)p.CI * 8u);

    const Place at(s, tid);
    Band<PASSES, VEC, true> bx;
    Band<PASSES, VEC, false> bd;
    auto block_of = [&](int u, int &n0, int &row0) {
        const int grp = fdiv_c3f(u, s.m_bands);
        n0 = grp * s.IMGS;
        row0 = (u - grp * s.bands) * s.TH;
    };
    auto request_x = [&](int u) {
        int n0, row0;
        block_of(u, n0, row0);
        bx.request(s, at, x_rs, p.xsn, p.xsc, ss_rs, p.CI, c0, n0, row0, true);
    };
    auto request_d = [&](int u, int k) {
        int n0, row0;
        block_of(u, n0, row0);
        bd.request(s, at, d_rs, p.dsn, p.dsc, ss_rs, p.CO, 16 * k, n0, row0, false);
    };
    const int u0 = (int)blockIdx.x * p.upw, u1 = min(p.units, u0 + p.upw);
    request_d(u0, 0);
    if (wgrad) request_x(u0);
    // data gradient: lane (l16, kq) multiplies with the taps of input channel c0 + l16 and output channel 16 k + 4 c4 + kq
    float a[4][9];
    auto filter = [&](int k) {
#pragma unroll
        for (int c4 = 0; c4 < 4; ++c4) {
            const int ko = 16 * k + 4 * c4 + kq, c = c0 + l16;
            load_taps<true>(w_rs, ko < p.CO && c < p.CI ? (uint32_t)(ko * p.CI + c) * 36u : kNowhere, a[c4]);
        }
    };
    if (dgrad) filter(0);
    zero_columns(s, x_lds, tid, kThreads);
    zero_columns(s, d_lds, tid, kThreads);

    // data gradient: this lane's quad; filter gradient: quad 4 g + kq of the wavefront's sixteen is this lane's part of
    // step g's reduction (a quad that the block does not have reads the zeros ahead of a row for dh)
    const int quad = wave * 16 + l16;
    const QuadAt own(s, quad);
    const float *const win = d_lds + kq * s.plane + own.lds(s);
    int xq[4], dq[4];
#pragma unroll
    for (int g = 0; g < 4; ++g) {
        const int e = wave * 16 + 4 * g + kq;
        const QuadAt q(s, e);
        xq[g] = l16 * s.plane + q.lds(s);
        dq[g] = p.d_lds + l16 * s.plane + (e < s.quads ? q.lds(s) + s.pitch : 0);
    }
    f4_t wacc[KT][9];  // [chunk][tap]: output channels 4 * kq + 0 .. 3 of the chunk, input channel l16
#pragma unroll
    for (int k = 0; k < KT; ++k)
#pragma unroll
        for (int t = 0; t < 9; ++t) wacc[k][t] = f4_t{0.f, 0.f, 0.f, 0.f};

    for (int u = u0; u < u1; ++u) {
        f4_t acc[4];
#pragma unroll
        for (int t = 0; t < 4; ++t) acc[t] = f4_t{0.f, 0.f, 0.f, 0.f};
#pragma unroll
        for (int k = 0; k < KT; ++k) {
            if (16 * k >= p.CO) break;
            if (k == 0 && wgrad) bx.commit(s, at, x_lds, true);
            bd.commit(s, at, d_lds, false);
            __syncthreads();
            if (k + 1 < KT && 16 * (k + 1) < p.CO) {
                request_d(u, k + 1);
            } else if (KT == 1 && u + 1 < u1) {
                request_d(u + 1, 0);
                if (wgrad) request_x(u + 1);
            }
            if (dgrad) {
#pragma unroll
                for (int c4 = 0; c4 < 4; ++c4) {
                    if (16 * k + 4 * c4 >= p.CO) continue;
#pragma unroll
                    for (int rr = 0; rr < 3; ++rr) {
                        const Window v(win + c4 * 4 * s.plane + rr * s.pitch);
#pragma unroll
                        for (int ss = 0; ss < 3; ++ss)
#pragma unroll
                            for (int t = 0; t < 4; ++t)
                                acc[t] = __builtin_amdgcn_mfma_f32_16x16x4f32(a[c4][rr * 3 + ss], v.b[t + ss], acc[t], 0, 0, 0);
                    }
                }
                if (KT > 1) filter(k + 1 < KT && 16 * (k + 1) < p.CO ? k + 1 : 0);
            }
            if (wgrad) {
#pragma unroll
                for (int g = 0; g < 4; ++g) {
                    const f4_t d = *reinterpret_cast<const f4_t *>(smem + dq[g]);
#pragma unroll
                    for (int rr = 0; rr < 3; ++rr) {
                        const Window v(x_lds + xq[g] + rr * s.pitch);
#pragma unroll
                        for (int t = 0; t < 4; ++t)
#pragma unroll
                            for (int ss = 0; ss < 3; ++ss)
                                wacc[k][rr * 3 + ss] = __builtin_amdgcn_mfma_f32_16x16x4f32(d[t], v.b[t + ss], wacc[k][rr * 3 + ss], 0, 0, 0);
                    }
                }
            }
            __syncthreads();  // every wavefront has read the chunk
        }
        if (KT > 1 && u + 1 < u1) {  // (not ahead of the matrix instructions: the registers are not there)
            request_d(u + 1, 0);
            if (wgrad) request_x(u + 1);
        }
        if (dgrad) {  // channels c0 + 4 * kq + j of this lane's quad
            int n0, row0;
            block_of(u, n0, row0);
            const int n = n0 + own.img, row = row0 + own.row;
            const bool ok = quad < s.quads && n < s.N && row < s.H;
            const uint32_t hw = (uint32_t)(s.H * s.W);
            const uint32_t o_off = (((uint32_t)n * p.CI + (uint32_t)(c0 + 4 * kq)) * hw + (uint32_t)(row * s.W + 4 * own.q)) * 4u;
            const __amdgpu_buffer_rsrc_t o_rs = rsrc(p.da, p.da_bytes);
#pragma unroll
            for (int j = 0; j < 4; ++j) {
                const f4_t v = {acc[0][j], acc[1][j], acc[2][j], acc[3][j]};
                const bool has = ok && c0 + 4 * kq + j < p.CI;
                const uint32_t o = o_off + (uint32_t)j * hw * 4u;
                if (VEC) {
                    store4(o_rs, has ? o : kNowhere, v);
                } else {
                    const int left = has ? s.W - 4 * own.q : 0;  // pixels of the row from here on
                    store4(o_rs, left >= 4 ? o : kNowhere, v);
#pragma unroll
                    for (int t = 0; t < 3; ++t)
                        __builtin_amdgcn_raw_buffer_store_b32(__float_as_uint(v[t]), o_rs, left < 4 && t < left ? o + 4u * t : kNowhere, 0, 0);
                }
            }
        }
    }
    if (!wgrad) return;
    // ---- the wavefronts' shares of the filter gradient, added in order; a partial result keeps the register order
    //      [chunk][tap][j][lane]
#pragma unroll
    for (int k = 0; k < KT; ++k) {
        if (16 * k >= p.CO) break;
        if (k > 0) __syncthreads();
#pragma unroll
        for (int t = 0; t < 9; ++t)
#pragma unroll
            for (int j = 0; j < 4; ++j) smem[((wave * 9 + t) * 4 + j) * 64 + lane] = wacc[k][t][j];
        __syncthreads();
        float *const out = p.part + (int64_t)blockIdx.x * p.part_stride + (k * p.tiles_c + (int)blockIdx.y) * 2304;
        for (int i = tid; i < 2304; i += kThreads) {
            float v = smem[i];
#pragma unroll
            for (int wv = 1; wv < NW; ++wv) v += smem[wv * 2304 + i];
            out[i] = v;
        }
    }
}

// Where the flat-pixel kernels take both gradients too (17 to 32 channels, rows that are not whole quads; two launches): as
// long as a workgroup has one block this kernel is ahead, 0.77 to 0.97 of the time of a training step of two basic blocks; from
// there on both run in rounds, this one of `upw` blocks a workgroup, those of 32768 pixels.  Two rounds against three, three
// against five, four against six, five against eight 0.85 to 0.99; with fewer in hand 0.93 to 1.11, most above 1 (426 shapes
// of 3000 to 255000 pixels).
bool takes(int cin, int cout, const Geo &g, int upw) {
    if (upw == 1 || conv_gemm_f32_tile(cout, cin, 3, g).pixels == 0) return true;
    return 3 * upw <= 2 * ((g.pixels() + 32767) / 32768);
}

struct B3fLaunch {
    B3fArgs a;
    WgradReduce red;
    int waves, passes;
    bool vec;
    dim3 grid;
    size_t lds_bytes;
};

// Tiling and arguments; scratch_floats: what there is of scratch.
bool plan_b3f(View x, const float *scale_shift, View dh, const float *w, int cin, int cout, Geo g, float *scratch,
              size_t scratch_floats, float *dw, bool accumulate, float *da, B3fLaunch &L) {
    if (cin > 32 || cout > 32) return false;
    const int tiles_c = (cin + 15) / 16, tiles_k = (cout + 15) / 16;
    // Blocks of twice the size where four wavefronts a workgroup would make more workgroups than there may be partial
    // results (256 of 16 x 16 channels: what the scratch is sized for).
    C3fPlan pl = plan_c3f(g, 4);
    int waves = 4;
    if (pl.passes && pl.blocks * tiles_c > 256) {
        const C3fPlan wide = plan_c3f(g, 8);
        if (wide.passes) pl = wide, waves = 8;
    }
    if (pl.passes == 0) return false;
    const int64_t x_b = 4 * ((g.n - 1) * x.sn + (cin - 1) * x.sc + g.hw()), d_b = 4 * ((g.n - 1) * dh.sn + (cout - 1) * dh.sc + g.hw());
    const int64_t a_b = 4 * g.pixels() * cin;
    if (std::max(std::max(x_b, d_b), a_b) >= (int64_t)kNowhere) return false;
    auto aligned = [](const View &v) { return v.sn % 4 == 0 && v.sc % 4 == 0 && (reinterpret_cast<uintptr_t>(v.p) & 15) == 0; };
    B3fArgs a{};
    a.x = x.p; a.scale_shift = scale_shift; a.dh = dh.p; a.w = w; a.da = da; a.part = scratch;
    a.xsn = (uint32_t)x.sn; a.xsc = (uint32_t)x.sc; a.dsn = (uint32_t)dh.sn; a.dsc = (uint32_t)dh.sc;
    a.x_bytes = (uint32_t)x_b; a.dh_bytes = (uint32_t)d_b; a.da_bytes = (uint32_t)a_b; a.w_bytes = (uint32_t)cin * cout * 36;
    a.CI = cin; a.CO = cout;
    a.s = pl.s;
    a.part_stride = tiles_k * tiles_c * 2304; a.tiles_c = tiles_c;
    int64_t slices = std::min<int64_t>(pl.blocks, std::max(1, 256 / tiles_c));
    slices = std::min<int64_t>(slices, (int64_t)(scratch_floats / (size_t)a.part_stride));
    if (slices < 1) return false;
    a.units = (int)pl.blocks;
    a.upw = (int)((pl.blocks + slices - 1) / slices);
    if (!takes(cin, cout, g, a.upw)) return false;
    slices = (pl.blocks + a.upw - 1) / a.upw;
    a.d_lds = pl.passes * pl.s.cpp * pl.s.plane;
    L.a = a;
    L.waves = waves; L.passes = pl.passes;
    L.vec = g.w % 4 == 0 && aligned(x) && aligned(dh) && (reinterpret_cast<uintptr_t>(da) & 15) == 0;
    L.grid = dim3((unsigned)slices, (unsigned)tiles_c);
    L.lds_bytes = std::max((size_t)2 * a.d_lds, (size_t)waves * 2304) * 4;
    WgradReduce red{};
    red.part = scratch; red.dw = dw;
    red.part_stride = a.part_stride; red.S = (int)slices; red.KS2 = 9; red.MT = 1; red.CT = 1;
    red.tiles_c = tiles_c; red.CO = cout; red.CI = cin; red.accumulate = accumulate ? 1 : 0;
    red.tile = 16; red.wide = red.S <= 16 ? 1 : 0;
    red.blocks = red.wide ? (a.part_stride + 255) / 256 : (a.part_stride + 31) / 32;
    L.red = red;
    return true;
}

template <int NW, int PASSES, int KT, bool VEC>
void run_one(Ctx &cx, const B3fLaunch &L, const B3fArgs &a) {
    static OncePerDevice raised;
    if (!raise_lds_limit(cx, conv3x3_f32_bwd_k<NW, PASSES, KT, VEC>, L.lds_bytes, 160 * 1024, raised)) return;
    // While the chip has room the two gradients get workgroups of their own: half the chain of one that does both.
    dim3 grid = L.grid;
    if (a.parts == (kDgrad | kWgrad) && grid.x * grid.y <= 128) grid.z = 2;
    cx.run(conv3x3_f32_bwd_k<NW, PASSES, KT, VEC>, grid, dim3(64 * NW), L.lds_bytes, a);
}

void launch_b3f(Ctx &cx, const B3fLaunch &L, int parts) {
    B3fArgs a = L.a;
    a.parts = parts;
    const int kt = a.CO > 16 ? 2 : 1;
#define RVN_CASE(W_, P_, K_)                                               \
    if (L.waves == W_ && L.passes == P_ && kt == K_) {                     \
        if (L.vec) run_one<W_, P_, K_, true>(cx, L, a);                    \
        else run_one<W_, P_, K_, false>(cx, L, a);                         \
    }
    RVN_CASE(4, 6, 1) RVN_CASE(4, 6, 2) RVN_CASE(4, 8, 1) RVN_CASE(4, 8, 2)
    RVN_CASE(8, 6, 1) RVN_CASE(8, 6, 2) RVN_CASE(8, 8, 1) RVN_CASE(8, 8, 2)
#undef RVN_CASE
}

}  // namespace

// How the gradients of a layer of dense, aligned tensors run, for the tests: wavefronts, staging passes, chunks of output
// channels, whole quads a row, in pairs of hexadecimal digits, or -1 (kernels of their own).
extern "C" int rvn_conv3x3_f32_bwd_form(int cin, int cout, int n, int h, int w) {
    const Geo g{n, h, w};
    float *const at = reinterpret_cast<float *>(256);
    B3fLaunch L;
    if (!wgrad_rows_fit(cin, cout, 3, g) ||
        !plan_b3f(dense_view(at, cin, g), at, dense_view(at, cout, g), at, cin, cout, g, at, wgrad_scratch_floats(cin, cout, 3, g), at, false, at, L))
        return -1;
    return ((L.waves * 256 + L.passes) * 256 + (cout > 16 ? 2 : 1)) * 256 + (int)L.vec;
}

bool separate_launches() {
    const char *e = std::getenv("RVN_SEPARATE_LAUNCHES");
    return e && e[0] == '1' && e[1] == 0;
}

bool conv_dgrad_wgrad_f32(Ctx &cx, View x, const float *scale_shift, View dh, const float *w, int cin, int cout, int ks,
                          Geo g, float *scratch, float *dw, bool accumulate, float *da, WgradReduce *defer) {
    if (ks != 3 || !defer || !wgrad_rows_fit(cin, cout, ks, g)) return false;
    B3fLaunch L;
    if (!plan_b3f(x, scale_shift, dh, w, cin, cout, g, scratch, wgrad_scratch_floats(cin, cout, ks, g), dw, accumulate, da, L))
        return false;
    const double P = (double)g.pixels();
    const double flops = 2.0 * P * cin * cout * 9, bytes = P * cin * 4.0 + P * cout * 4.0;
    cx.cost.conv_dgrad_calls += 1;
    cx.cost.conv_wgrad_calls += 1;
    cx.cost.conv_flops += 2.0 * flops;
    *defer = L.red;
    if (separate_launches()) {
        if (cx.launch(K_CONV_WGRAD, bytes, flops)) launch_b3f(cx, L, kWgrad);
        if (cx.launch(K_CONV_DGRAD, bytes, flops)) launch_b3f(cx, L, kDgrad);
    } else if (cx.launch(K_CONV_DGRAD_WGRAD, 2.0 * bytes, 2.0 * flops)) {
        launch_b3f(cx, L, kDgrad | kWgrad);
    }
    return true;
}

}  // namespace rvn
