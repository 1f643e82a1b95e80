// Kernel body and argument block of the fp32 3x3 convolution of narrow layers (see conv3x3_f32.hip for the
// design); its staging, filter and operand helpers also serve the kernel of both gradients (conv3x3_f32_bwd.hip) and, the
// buffer accesses, the bf16 form.  Device code only, but for the plans.
#pragma once

#include "kernels.h"

namespace rvn {

// The pixel block of a workgroup and how its band lies in LDS.
struct C3fShape {
    int N, H, W;
    int TH, IMGS, bands;       // rows per block, images per block (bands == 1 then), blocks per image column
    int wq, quads;             // 4-pixel groups per row and per block
    int lrows, pitch, plane;   // LDS rows per image (TH + 2); floats from row to row and from channel to channel
    int items, cpp;            // quads a channel of the band has, halo rows included; channels staged per pass
    uint32_t m_bands, m_items, m_rq, m_wq, m_q;  // multipliers of fdiv_c3f for bands, items, lrows * wq, wq, TH * wq
};

struct C3fArgs {
    const float *in;           // x (forward) or upstream gradient (data gradient)
    const float *scale_shift;  // [2*CI]: a = max(in*scale + shift, 0); null = use `in` as is
    const float *w;            // [CO][CI][3][3] forward; [CI][CO][3][3] read transposed and flipped otherwise
    const float *r;            // skip operand of the epilogue (may alias out)
    float *out;
    uint32_t isn, isc, rsn, rsc, osn, osc;             // element strides
    uint32_t in_bytes, r_bytes, out_bytes, w_bytes;    // extents, from each base
    int CI, CO, ep;
    C3fShape s;
    // EMIT instances (every quad of every block a whole, valid one): per channel and wavefront the mean and
    // centred sum of squares of the 64 pixels it stores, at emit[(channel * emit_tiles + block * 4 + wavefront) * 2]
    float *emit;
    int emit_tiles;
};

struct C3fLaunch {
    C3fArgs a;
    int mt, passes;
    bool vec, whole;
    dim3 grid;
    size_t lds_bytes;
};

// The block for `waves` wavefronts (16 quads each), its staging passes (6 or 8; 0: no block fits) and the blocks in
// all.  Defined in conv3x3_f32.hip, as is the next.
struct C3fPlan {
    C3fShape s;
    int passes;
    int64_t blocks;
};
C3fPlan plan_c3f(const Geo &g, int waves);

// Tiling and arguments; false if the kernel does not take the layer.  Defined in conv3x3_f32.hip.
bool conv3x3_f32_plan(View in, const float *scale_shift, const float *w, bool transposed, int ci, int co, Geo g,
                      Epilogue ep, const View *r, View out, C3fLaunch &L);

namespace {

namespace c3f {

typedef float f4_t __attribute__((ext_vector_type(4)));
typedef uint32_t u4_t __attribute__((ext_vector_type(4)));

constexpr int kThreads = 256;
constexpr int kChunk = 16;              // channels staged at a time
constexpr uint32_t kNowhere = 0xf0000000u;  // a byte offset past every extent (host: extents end below it)

__device__ __forceinline__ int fdiv_c3f(int e, uint32_t m) { return m ? (int)__umulhi((uint32_t)e, m) : e; }

__device__ __forceinline__ __amdgpu_buffer_rsrc_t rsrc(const void *p, uint32_t bytes) {
    return __builtin_amdgcn_make_buffer_rsrc(const_cast<void *>(p), 0, (int)bytes, 0x00020000);
}
__device__ __forceinline__ float load1(__amdgpu_buffer_rsrc_t b, uint32_t lane, uint32_t uniform) {
    return __uint_as_float(__builtin_amdgcn_raw_buffer_load_b32(b, lane, uniform, 0));
}
__device__ __forceinline__ f4_t load4(__amdgpu_buffer_rsrc_t b, uint32_t lane, uint32_t uniform) {
    const u4_t v = __builtin_amdgcn_raw_buffer_load_b128(b, lane, uniform, 0);
    return *reinterpret_cast<const f4_t *>(&v);
}
// The whole offset in the lane part.  With a register as the scalar offset the compiler takes a store of more
// than 8 bytes to need no wait state before its data registers are written again; on this chip it does: in a kernel
// where other instructions followed at once (a launch of this body and a filter gradient's, since given up) such
// stores wrote what came into the registers next.
__device__ __forceinline__ void store4(__amdgpu_buffer_rsrc_t b, uint32_t lane, f4_t v) {
    __builtin_amdgcn_raw_buffer_store_b128(*reinterpret_cast<const u4_t *>(&v), b, lane, 0, 0);
}

// A thread's part in staging the band of a pixel block: one fixed quad of it (halo rows included) and the channels
// cs, cs + cpp, ... of a chunk, so a further item costs a scalar offset and no index arithmetic.  What lies
// outside the tensor is loaded from kNowhere, which gives zero, with scale and shift zero as well.
struct Place {
    int cs, img, lr, q, dst;
    bool staging;
    __device__ __forceinline__ Place(const C3fShape &s, int tid) {
        cs = fdiv_c3f(tid, s.m_items);
        const int e = tid - cs * s.items;
        img = fdiv_c3f(e, s.m_rq);
        const int e2 = e - img * (s.lrows * s.wq);
        lr = fdiv_c3f(e2, s.m_wq);
        q = e2 - lr * s.wq;
        staging = cs < s.cpp;
        dst = cs * s.plane + (img * s.lrows + lr) * s.pitch + 4 + 4 * q;
    }
};

template <int PASSES, bool VEC, bool BN>
struct Band {
    f4_t g[PASSES];
    float sc[BN ? PASSES : 1], sh[BN ? PASSES : 1];

    // the chunk of channels c0 .. c0 + 15 of the block whose first image and row are n0, row0
    __device__ __forceinline__ void request(const C3fShape &s, const Place &at, __amdgpu_buffer_rsrc_t in, uint32_t sn, uint32_t sch,
                                            __amdgpu_buffer_rsrc_t ss, int C, int c0, int n0, int row0, bool bn) {
        const int n = n0 + at.img, row = row0 - 1 + at.lr;
        const bool live = at.staging && n < s.N && row >= 0 && row < s.H;
        const uint32_t off = ((uint32_t)n * sn + (uint32_t)(row * s.W + 4 * at.q) + (uint32_t)at.cs * sch) * 4u;
        const int left = min(kChunk, C - c0) - at.cs;
        // (the scalar part of an offset stays inside the extent: the hardware takes it off before it compares)
#pragma unroll
        for (int i = 0; i < PASSES; ++i)
            g[i] = load4(in, live && i * s.cpp < left ? off : kNowhere, (uint32_t)min(c0 + i * s.cpp, C - 1) * sch * 4u);
        if (BN && bn) {
#pragma unroll
            for (int i = 0; i < PASSES; ++i) {
                const uint32_t lane = live && i * s.cpp < left ? (uint32_t)at.cs * 4u : kNowhere;
                const int c = min(c0 + i * s.cpp, C - 1);
                sc[i] = load1(ss, lane, (uint32_t)c * 4u);
                sh[i] = load1(ss, lane, (uint32_t)(C + c) * 4u);
            }
        }
    }
    // a(x) = max(x*scale + shift, 0), or the values as they are, into LDS
    __device__ __forceinline__ void commit(const C3fShape &s, const Place &at, float *lds, bool bn) const {
        if (!at.staging) return;
#pragma unroll
        for (int i = 0; i < PASSES; ++i) {
            f4_t v = g[i];
            if (BN && bn) {
#pragma unroll
                for (int j = 0; j < 4; ++j) v[j] = fmaxf(fmaf(v[j], sc[i], sh[i]), 0.f);
            }
            if (!VEC) {  // past the row's end a(x) is zero
#pragma unroll
                for (int j = 1; j < 4; ++j) v[j] = 4 * at.q + j < s.W ? v[j] : 0.f;
            }
            *reinterpret_cast<f4_t *>(lds + at.dst + i * s.cpp * s.plane) = v;
        }
    }
};

// The zero columns of 16 staged channels: four floats ahead of every row and behind the last one.
__device__ __forceinline__ void zero_columns(const C3fShape &s, float *lds, int tid, int threads) {
    const int rows = s.IMGS * s.lrows + 1;
    for (int z = tid; z < kChunk * rows; z += threads) {
        const int c = z & (kChunk - 1), rr = z / kChunk;
        *reinterpret_cast<f4_t *>(lds + c * s.plane + rr * s.pitch) = f4_t{0.f, 0.f, 0.f, 0.f};
    }
}

// Quad `quad` of a block (the last one where there are fewer): image, row and quad of the row.
struct QuadAt {
    int img, row, q;
    __device__ __forceinline__ QuadAt(const C3fShape &s, int quad) {
        const int e = min(quad, s.quads - 1);
        img = fdiv_c3f(e, s.m_q);
        const int e2 = e - img * (s.TH * s.wq);
        row = fdiv_c3f(e2, s.m_wq);
        q = e2 - row * s.wq;
    }
    // float offset in a staged plane of the quad's pixels in the row above it
    __device__ __forceinline__ int lds(const C3fShape &s) const { return (img * s.lrows + row) * s.pitch + 4 + 4 * q; }
};

// The nine taps of output channel (row of the operand) and input channel `c`, where both exist, `at` bytes into the filter.
template <bool TR>
__device__ __forceinline__ void load_taps(__amdgpu_buffer_rsrc_t w, uint32_t at, float (&a)[9]) {
    const f4_t lo = load4(w, at, 0), hi = load4(w, at + 16u, 0);
    const float last = load1(w, at + 32u, 0);
#pragma unroll
    for (int t = 0; t < 4; ++t) {
        a[TR ? 8 - t : t] = lo[t];
        a[TR ? 4 - t : 4 + t] = hi[t];
    }
    a[TR ? 0 : 8] = last;
}

// Four matrix columns (pixels) at the three taps of one filter row: the staged quad and its two neighbours.
struct Window {
    float b[6];
    __device__ __forceinline__ explicit Window(const float *at) {
        const f4_t mid = *reinterpret_cast<const f4_t *>(at);
        b[0] = at[-1];
        b[1] = mid[0]; b[2] = mid[1]; b[3] = mid[2]; b[4] = mid[3];
        b[5] = at[4];
    }
};

// Workgroup (bx, by); `smem` is the workgroup's dynamic LDS.  MT: 16-channel output tiles.  PASSES: staging
// passes per chunk.  TR: the filter is read transposed and flipped (data gradient).  VEC: rows are whole
// 4-pixel groups.
template <int MT, int PASSES, bool TR, bool VEC, bool EMIT>
__device__ __forceinline__ void conv3x3_f32_body(const C3fArgs &p, int bx, int by, float *smem) {
    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int l16 = lane & 15, kq = lane >> 4;
    const int img_grp = fdiv_c3f(bx, p.s.m_bands), band = bx - img_grp * p.s.bands;
    const int n0 = img_grp * p.s.IMGS, row0 = band * p.s.TH, co0 = by * (MT * 16);
    const bool bn = p.scale_shift != nullptr;
    const __amdgpu_buffer_rsrc_t in_rs = rsrc(p.in, p.in_bytes), w_rs = rsrc(p.w, p.w_bytes);
    const __amdgpu_buffer_rsrc_t ss_rs = rsrc(bn ? p.scale_shift : p.in, bn ? (uint32_t)p.CI * 8u : 0u);

    const Place at(p.s, tid);
    Band<PASSES, VEC, !TR> band_g;
    auto request = [&](int c0) { band_g.request(p.s, at, in_rs, p.isn, p.isc, ss_rs, p.CI, c0, n0, row0, bn); };
    // ---- filter operands, straight from memory: lane (l16, kq) multiplies with the nine taps of output channel
    //      l16 and input channel 4 * c4 + kq, which lie next to each other
    float a[MT][kChunk / 4][9];
    auto filter = [&](int c4, int c0) {
        const int c = c0 + 4 * c4 + kq;
#pragma unroll
        for (int m = 0; m < MT; ++m) {
            const int ko = co0 + m * 16 + l16;
            load_taps<TR>(w_rs, c < p.CI && ko < p.CO ? (TR ? (uint32_t)(c * p.CO + ko) : (uint32_t)(ko * p.CI + c)) * 36u : kNowhere, a[m][c4]);
        }
    };
    request(0);
#pragma unroll
    for (int c4 = 0; c4 < kChunk / 4; ++c4) filter(c4, 0);

    // ---- this lane's four pixels and where its results go: channels co0 + m * 16 + 4 * kq + j
    const int quad = wave * 16 + l16;
    const QuadAt own(p.s, quad);
    const int n = n0 + own.img, row = row0 + own.row;
    const bool ok = quad < p.s.quads && n < p.s.N && row < p.s.H;
    const uint32_t pix = (uint32_t)(row * p.s.W + 4 * own.q);
    const uint32_t o_off = ((uint32_t)n * p.osn + pix + (uint32_t)(4 * kq) * p.osc) * 4u;
    const uint32_t r_off = ((uint32_t)n * p.rsn + pix + (uint32_t)(4 * kq) * p.rsc) * 4u;
    const float *const win = smem + kq * p.s.plane + own.lds(p.s);
    const int ko_lane = co0 + 4 * kq;
    f4_t rv[MT][4];  // (every skip value is requested before the first store: r may alias out element for element)
    if (!TR && p.ep != EP_STORE) {
        const __amdgpu_buffer_rsrc_t r_rs = rsrc(p.r, p.r_bytes);
#pragma unroll
        for (int m = 0; m < MT; ++m)
#pragma unroll
            for (int j = 0; j < 4; ++j)
                rv[m][j] = load4(r_rs, ok && ko_lane + m * 16 + j < p.CO ? r_off : kNowhere, (uint32_t)min(co0 + m * 16 + j, p.CO - 1) * p.rsc * 4u);
    }
    zero_columns(p.s, smem, tid, kThreads);
    f4_t acc[MT][4];  // [.][pixel]: channels 4 * kq + 0 .. 3
#pragma unroll
    for (int m = 0; m < MT; ++m)
#pragma unroll
        for (int t = 0; t < 4; ++t) acc[m][t] = f4_t{0.f, 0.f, 0.f, 0.f};

    band_g.commit(p.s, at, smem, bn);
    __syncthreads();
    for (int c0 = 0;; c0 += kChunk) {
        const bool more = c0 + kChunk < p.CI;
        if (more) request(c0 + kChunk);
#pragma unroll
        for (int c4 = 0; c4 < kChunk / 4; ++c4) {
            if (c0 + 4 * c4 < p.CI) {
#pragma unroll
                for (int rr = 0; rr < 3; ++rr) {
                    const Window v(win + c4 * 4 * p.s.plane + rr * p.s.pitch);
#pragma unroll
                    for (int ss = 0; ss < 3; ++ss)
#pragma unroll
                        for (int m = 0; m < MT; ++m)
#pragma unroll
                            for (int t = 0; t < 4; ++t)
                                acc[m][t] = __builtin_amdgcn_mfma_f32_16x16x4f32(a[m][c4][rr * 3 + ss], v.b[t + ss], acc[m][t], 0, 0, 0);
                }
            }
            if (more) filter(c4, c0 + kChunk);
        }
        if (!more) break;
        __syncthreads();  // every wavefront has read the chunk
        band_g.commit(p.s, at, smem, bn);
        __syncthreads();
    }

    // ---- epilogue
    const __amdgpu_buffer_rsrc_t o_rs = rsrc(p.out, p.out_bytes);
#pragma unroll
    for (int m = 0; m < MT; ++m)
#pragma unroll
        for (int j = 0; j < 4; ++j) {
            f4_t v = {acc[m][0][j], acc[m][1][j], acc[m][2][j], acc[m][3][j]};
            if (!TR && p.ep == EP_ADD) v = rv[m][j] + v;
            if (!TR && p.ep == EP_SUB) v = rv[m][j] - v;
#pragma unroll
            for (int t = 0; t < 4; ++t) acc[m][t][j] = v[t];
            const bool has = ok && ko_lane + m * 16 + j < p.CO;
            const uint32_t at = (uint32_t)min(co0 + m * 16 + j, p.CO - 1) * p.osc * 4u;
            if (VEC) {
                store4(o_rs, has ? o_off + at : kNowhere, v);
            } else {
                const int left = has ? p.s.W - 4 * own.q : 0;  // pixels of the row from here on
                store4(o_rs, left >= 4 ? o_off + at : kNowhere, v);
#pragma unroll
                for (int t = 0; t < 3; ++t)
                    __builtin_amdgcn_raw_buffer_store_b32(__float_as_uint(v[t]), o_rs, left < 4 && t < left ? o_off + 4u * t : kNowhere, at, 0);
            }
        }
    // Statistics of what was stored, for the BN layer that reads it next: a channel's 64 pixels of this wavefront
    // are four registers in each of the 16 lanes of one quarter.  Sums of (v - pivot) and (v - pivot)^2, pivot =
    // the quarter's first value, are folded over the lanes four channels at a time (two steps halve the
    // channels a lane holds and add its partner's, two plain steps follow).
    if constexpr (EMIT) {
#pragma unroll
        for (int m = 0; m < MT; ++m) {
            float ea[4], eb[4], piv[4];  // the pivots are uniform over the quarter
#pragma unroll
            for (int j = 0; j < 4; ++j) {
                piv[j] = __shfl(acc[m][0][j], kq * 16, 64);
                float s1 = 0.f, s2 = 0.f;
#pragma unroll
                for (int t = 0; t < 4; ++t) {
                    const float d = acc[m][t][j] - piv[j];
                    s1 += d;
                    s2 += d * d;
                }
                ea[j] = s1;
                eb[j] = s2;
            }
            const bool up8 = (l16 & 8) != 0, up4 = (l16 & 4) != 0;
#pragma unroll
            for (int k = 0; k < 2; ++k) {
                const float keep_a = up8 ? ea[k + 2] : ea[k], send_a = up8 ? ea[k] : ea[k + 2];
                const float keep_b = up8 ? eb[k + 2] : eb[k], send_b = up8 ? eb[k] : eb[k + 2];
                ea[k] = keep_a + __shfl_xor(send_a, 8, 64);
                eb[k] = keep_b + __shfl_xor(send_b, 8, 64);
            }
            {
                const float keep_a = up4 ? ea[1] : ea[0], send_a = up4 ? ea[0] : ea[1];
                const float keep_b = up4 ? eb[1] : eb[0], send_b = up4 ? eb[0] : eb[1];
                ea[0] = keep_a + __shfl_xor(send_a, 4, 64);
                eb[0] = keep_b + __shfl_xor(send_b, 4, 64);
            }
#pragma unroll
            for (int off = 2; off > 0; off >>= 1) {
                ea[0] += __shfl_xor(ea[0], off, 64);
                eb[0] += __shfl_xor(eb[0], off, 64);
            }
            const int j = l16 >> 2;  // the channel of its quarter that the lane now holds
            const float pivot = j == 0 ? piv[0] : j == 1 ? piv[1] : j == 2 ? piv[2] : piv[3];
            const int ko = ko_lane + m * 16 + j;
            if ((l16 & 3) == 0 && ko < p.CO) {
                constexpr float inv = 1.f / 64;
                const float mean = pivot + ea[0] * inv;
                const float m2 = fmaxf(eb[0] - ea[0] * ea[0] * inv, 0.f);
                reinterpret_cast<float2 *>(p.emit)[(int64_t)ko * p.emit_tiles + bx * 4 + wave] = make_float2(mean, m2);
            }
        }
    }
}

}  // namespace c3f

}  // namespace

}  // namespace rvn
