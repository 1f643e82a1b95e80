// Kernel body and argument block of the bf16 3x3 convolution of narrow layers (see conv3x3_bf16_narrow.hip for the
// design), as a device function.  Device code only.
#pragma once

#include "conv3x3_f32_body.h"
#include "kernels.h"

namespace rvn {

struct C3nShape {
    int N, H, W;
    int TH, IMGS, bands;       // rows per block, images per block (bands == 1 then), blocks per image column
    int wq, quads;             // 4-pixel groups per row and per block
    int lrows, pitch;          // LDS rows per image (TH + 2); records from row to row
    int bquads, items;         // quads of the band (halo rows included), and times the channel octets
    uint32_t m_bands, m_bq, m_rq, m_wq, m_q;  // multipliers of fdiv_c3f for bands, bquads, lrows * wq, wq, TH * wq
};

struct C3nArgs {
    const float *in;           // x (forward) or upstream gradient (data gradient), fp32 NCHW planes
    const float *scale_shift;  // [2*CI]: a = max(in*scale + shift, 0); null = use `in` as is
    const uint16_t *wq;        // filter in bf16, [CO][9][CIP]
    const float *w;            // W32 instances: the filter as it is, [CO][CI][9]
    const float *r;            // skip operand of the epilogue (may alias out)
    float *out;
    uint32_t isn, isc, rsn, rsc, osn, osc;           // element strides
    uint32_t in_bytes, r_bytes, out_bytes, w_bytes;  // extents, from each base
    int CI, CO, CIP, ep;
    C3nShape s;
    // EMIT instances (every quad of every block a whole, valid one): per channel and 64 consecutive pixels the mean and
    // centred sum of squares of what is stored, at emit[(channel * emit_tiles + tile) * 2]
    float *emit;
    int emit_tiles;
    // MERGE instances: the BN layer's statistics still lie in such partial results (of `in`); every workgroup merges them
    // for itself, the first one also into stats [4][CI]
    StatsMerge merge;
};

namespace {

namespace c3n {

using c3f::f4_t;
using c3f::fdiv_c3f;
using c3f::kNowhere;
using c3f::load4;
using c3f::rsrc;
using c3f::store4;
using c3f::u4_t;

typedef float float16_t __attribute__((ext_vector_type(16)));
typedef __bf16 bf16x8_t __attribute__((ext_vector_type(8)));
typedef __bf16 bf16x2_t __attribute__((ext_vector_type(2)));
typedef float float2_t __attribute__((ext_vector_type(2)));

constexpr int kThreads = 256;

// LDS record of one pixel: its CH channels and 16 bytes, an odd number of 16-byte units (lanes that read
// consecutive records touch every bank once).
constexpr int record_bytes(int ch) { return ch * 2 + 16; }
constexpr int chan_waves(int ch) { return ch == 64 ? 2 : 1; }  // wavefronts side by side along the output channels

// Order of a result's sum, that of the kernels that take the layer at other sizes: chunks of 16, 32 or 64 channels, in each
// the taps, and for every tap the chunk's channels; or two chains of half the channels in chunks of 16.
enum Order { kChunk16 = 1, kChunk32 = 2, kChunk64 = 4, kHalves = 0 };

__device__ __forceinline__ uint32_t pack2(float lo, float hi) {
    const float2_t v = {lo, hi};
    const bf16x2_t b = __builtin_convertvector(v, bf16x2_t);
    return *reinterpret_cast<const uint32_t *>(&b);
}

// Quad `quad` of a block (the last one where there are fewer): image, row and quad of the row.
struct QuadAt {
    int img, row, q;
    __device__ __forceinline__ QuadAt(const C3nShape &s, int quad) {
        const int e = min(quad, s.quads - 1);
        img = fdiv_c3f(e, s.m_q);
        const int e2 = e - img * (s.TH * s.wq);
        row = fdiv_c3f(e2, s.m_wq);
        q = e2 - row * s.wq;
    }
    // record of the quad's first pixel at the filter's first tap
    __device__ __forceinline__ int rec(const C3nShape &s) const { return (img * s.lrows + row) * s.pitch + 4 * q; }
};

// Staging of a band: item e of a thread is one quad and one octet of channels, eight 16-byte loads.  What lies outside
// the tensor is loaded from kNowhere, which gives zero, with scale and shift zero as well (the scalar part of an offset stays
// inside the extent, which the hardware takes it off).  GEN: rows that are not
// whole quads, or a last octet of fewer channels.
template <int CH, int PASSES, bool GEN, bool MERGE>
struct Stage {
    f4_t g[PASSES][8], sc[PASSES][2], sh[PASSES][2];
    int dst[PASSES], col[PASSES], left[PASSES], oct[PASSES];  // LDS bytes of the first pixel (-1: nothing); its column; channels from the octet on; the octet, -1 outside

    __device__ __forceinline__ void request(const C3nShape &s, int tid, __amdgpu_buffer_rsrc_t in, uint32_t sn, uint32_t sch,
                                            __amdgpu_buffer_rsrc_t ss, int C, int n0, int row0, bool bn) {
#pragma unroll
        for (int i = 0; i < PASSES; ++i) {
            const int e = tid + i * kThreads;
            const int oc = fdiv_c3f(e, s.m_bq), b = e - oc * s.bquads;
            const int img = fdiv_c3f(b, s.m_rq), b2 = b - img * (s.lrows * s.wq);
            const int lr = fdiv_c3f(b2, s.m_wq), q = b2 - lr * s.wq;
            const int n = n0 + img, row = row0 - 1 + lr;
            dst[i] = e < s.items ? ((img * s.lrows + lr) * s.pitch + 1 + 4 * q) * record_bytes(CH) + oc * 16 : -1;
            col[i] = 4 * q;
            left[i] = C - 8 * oc;
            const bool live = e < s.items && n < s.N && row >= 0 && row < s.H && left[i] > 0;
            const uint32_t off = live ? ((uint32_t)n * sn + (uint32_t)(row * s.W + 4 * q) + (uint32_t)(8 * oc) * sch) * 4u : kNowhere;
#pragma unroll
            for (int k = 0; k < 8; ++k) g[i][k] = load4(in, off, (uint32_t)min(k, C - 1) * sch * 4u);
            oct[i] = live ? oc : -1;
            if (!MERGE && bn) {
                const uint32_t at = live ? (uint32_t)oc * 32u : kNowhere;
                const uint32_t at2 = live ? (uint32_t)(C + 8 * oc) * 4u : kNowhere;
#pragma unroll
                for (int k = 0; k < 2; ++k) {
                    sc[i][k] = load4(ss, at + 16u * k, 0);
                    sh[i][k] = load4(ss, at2 + 16u * k, 0);
                }
            }
        }
    }
    // a(x) = max(x*scale + shift, 0), or the values as they are, rounded into the pixels' records
    // (MERGE: scale and shift from `ss`, [2][CH] in LDS)
    __device__ __forceinline__ void commit(const C3nShape &s, char *lds, const float *ss, bool bn) {
#pragma unroll
        for (int i = 0; i < PASSES; ++i) {
            if (dst[i] < 0) continue;
            if (MERGE) {
#pragma unroll
                for (int k = 0; k < 2; ++k) {
                    const f4_t zero = {0.f, 0.f, 0.f, 0.f};
                    const int oc = max(oct[i], 0);
                    sc[i][k] = *reinterpret_cast<const f4_t *>(ss + 8 * oc + 4 * k);
                    sh[i][k] = *reinterpret_cast<const f4_t *>(ss + CH + 8 * oc + 4 * k);
                    if (oct[i] < 0) sc[i][k] = sh[i][k] = zero;
                }
            }
            if (bn) {
#pragma unroll
                for (int k = 0; k < 8; ++k)
#pragma unroll
                    for (int j = 0; j < 4; ++j) g[i][k][j] = fmaxf(fmaf(g[i][k][j], sc[i][k >> 2][k & 3], sh[i][k >> 2][k & 3]), 0.f);
            }
#pragma unroll
            for (int j = 0; j < 4; ++j) {
                if (GEN) {
#pragma unroll
                    for (int k = 0; k < 8; ++k) g[i][k][j] = k < left[i] && col[i] + j < s.W ? g[i][k][j] : 0.f;
                }
                const u4_t v = {pack2(g[i][0][j], g[i][1][j]), pack2(g[i][2][j], g[i][3][j]), pack2(g[i][4][j], g[i][5][j]),
                                pack2(g[i][6][j], g[i][7][j])};
                *reinterpret_cast<u4_t *>(lds + dst[i] + j * record_bytes(CH)) = v;
            }
        }
    }
};

// The zero records ahead of every row and behind the last one.
template <int CH>
__device__ __forceinline__ void zero_records(const C3nShape &s, char *lds, int tid) {
    constexpr int U = CH / 8;
    const int units = (s.IMGS * s.lrows + 1) * U;
    for (int z = tid; z < units; z += kThreads)
        *reinterpret_cast<u4_t *>(lds + z / U * s.pitch * record_bytes(CH) + z % U * 16) = u4_t{0u, 0u, 0u, 0u};
}

// The operands of output channel ko and the channels 16 ks ... 16 ks + 15, straight from memory: nine taps of the octet of
// input channels that kg stands for.  In a filter that has not been converted the taps of an octet are consecutive.
template <bool W32>
__device__ __forceinline__ void load_filter(__amdgpu_buffer_rsrc_t rs, const C3nArgs &p, int ko, int ks, int kg, bf16x8_t (&w)[9]) {
    const int oc = 2 * ks + kg;
    if constexpr (W32) {
        const uint32_t at = ko < p.CO && 8 * oc < p.CI ? (uint32_t)(ko * p.CI + 8 * oc) * 36u : kNowhere;
        float v[72];
#pragma unroll
        for (int i = 0; i < 18; ++i) {
            const f4_t q = load4(rs, at + 16u * i, 0);
#pragma unroll
            for (int j = 0; j < 4; ++j) v[4 * i + j] = q[j];
        }
        const int left = p.CI - 8 * oc;
#pragma unroll
        for (int k = 0; k < 8; ++k)
#pragma unroll
            for (int t = 0; t < 9; ++t) v[9 * k + t] = k < left ? v[9 * k + t] : 0.f;
#pragma unroll
        for (int t = 0; t < 9; ++t) {
            const u4_t q = {pack2(v[t], v[9 + t]), pack2(v[18 + t], v[27 + t]), pack2(v[36 + t], v[45 + t]), pack2(v[54 + t], v[63 + t])};
            w[t] = *reinterpret_cast<const bf16x8_t *>(&q);
        }
    } else {
        const uint32_t at = ko < p.CO && 8 * oc < p.CIP ? (uint32_t)(ko * 9 * p.CIP + 8 * oc) * 2u : kNowhere;
#pragma unroll
        for (int t = 0; t < 9; ++t) {
            const f4_t q = load4(rs, at, (uint32_t)(t * p.CIP) * 2u);
            w[t] = *reinterpret_cast<const bf16x8_t *>(&q);
        }
    }
}

__device__ __forceinline__ double shfl_xor_f64(double v, int mask) {
    const int64_t b = __double_as_longlong(v);
    const int lo = __shfl_xor((int)(b & 0xffffffff), mask, 64), hi = __shfl_xor((int)(b >> 32), mask, 64);
    return __longlong_as_double(((int64_t)hi << 32) | (uint32_t)lo);
}

// The merge of bn_stats_merge_k by one workgroup for all of its channels: 256 / CH neighbouring lanes share a channel.  Equal
// counts, so means are averaged (about the first one) instead of merged pair by pair; all in double, so the floats that
// come of it are those of the other form unless they lie within some 1e-15 of a rounding boundary.  Scale and shift
// go to `ss` [2][CH].
template <int CH>
__device__ __forceinline__ void merge_statistics(const StatsMerge &m, float *ss, int tid, bool store) {
    constexpr int T = kThreads / CH;
    const int ch = tid / T, j = tid % T;
    const bool has = ch < m.C;
    const int c = has ? ch : 0;
    const f4_t *const q = reinterpret_cast<const f4_t *>(m.partials) + (int64_t)c * (m.tiles / 2);
    const float gamma = m.gamma[c], beta = m.beta[c];
    const double pivot = (double)m.partials[(int64_t)c * m.tiles * 2];
    double sum = 0.0, sq = 0.0, m2 = 0.0;
    const int pairs = m.tiles / 2;
    for (int t0 = j; t0 < pairs; t0 += 4 * T) {
        f4_t v[4];
#pragma unroll
        for (int u = 0; u < 4; ++u) v[u] = q[min(t0 + u * T, pairs - 1)];
#pragma unroll
        for (int u = 0; u < 4; ++u) {
            const bool in = t0 + u * T < pairs;
            const double d0 = in ? (double)v[u][0] - pivot : 0.0, d1 = in ? (double)v[u][2] - pivot : 0.0;
            sum += d0 + d1;
            sq += d0 * d0 + d1 * d1;
            m2 += in ? (double)v[u][1] + (double)v[u][3] : 0.0;
        }
    }
#pragma unroll
    for (int off = T / 2; off > 0; off >>= 1) {
        sum += shfl_xor_f64(sum, off);
        sq += shfl_xor_f64(sq, off);
        m2 += shfl_xor_f64(m2, off);
    }
    const double inv = 1.0 / m.tiles, mean = pivot + sum * inv;
    const double var = (m2 / m.count + (sq - sum * sum * inv)) * inv;
    const float mean_f = (float)mean, rstd_f = (float)(1.0 / sqrt(var + (double)m.eps));
    const float scale = gamma * rstd_f, shift = fmaf(-mean_f, scale, beta);
    if (j == 0) {
        ss[ch] = has ? scale : 0.f;
        ss[CH + ch] = has ? shift : 0.f;
        if (store && has) {
            m.stats[ch] = mean_f;
            m.stats[m.C + ch] = rstd_f;
            m.stats[2 * m.C + ch] = scale;
            m.stats[3 * m.C + ch] = shift;
        }
    }
}

// Workgroup bx; `lds` is its dynamic LDS.  CH: channels of a record, and output channels at most.  A wavefront has one
// tile of 32 output channels and NT of 32 pixels.
template <int NT, int CH, int PASSES, bool GEN, bool EMIT, bool W32, int ORDER, bool MERGE>
__device__ __forceinline__ void conv3x3_bf16_narrow_body(const C3nArgs &p, int bx, char *lds) {
    constexpr int WM = chan_waves(CH), WP = 4 / WM, KS = CH / 16, REC = record_bytes(CH);
    constexpr int KS1 = W32 || PASSES == 2 ? 1 : KS > 2 ? 2 : KS;  // filter chunks requested up front; the rest when the staging registers are free
    const C3nShape &s = p.s;
    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int wm = wave % WM, wp = wave / WM;
    const int l32 = lane & 31, kg = lane >> 5;
    const int img_grp = fdiv_c3f(bx, s.m_bands), band = bx - img_grp * s.bands;
    const int n0 = img_grp * s.IMGS, row0 = band * s.TH;
    const bool bn = p.scale_shift != nullptr;

    Stage<CH, PASSES, GEN, MERGE> st;
    st.request(s, tid, rsrc(p.in, p.in_bytes), p.isn, p.isc, rsrc(bn ? p.scale_shift : p.in, bn ? (uint32_t)p.CI * 8u : 0u), p.CI, n0, row0, bn);
    const __amdgpu_buffer_rsrc_t w_rs = rsrc(W32 ? (const void *)p.w : (const void *)p.wq, p.w_bytes);
    bf16x8_t w[KS][9];
    const int ko = wm * 32 + l32;
    const bool ko_ok = ko < p.CO;
#pragma unroll
    for (int ks = 0; ks < KS1; ++ks) load_filter<W32>(w_rs, p, ko, ks, kg, w[ks]);
    zero_records<CH>(s, lds, tid);
    float *const ss_lds = reinterpret_cast<float *>(lds + (s.IMGS * s.lrows * s.pitch + 1) * REC);
    if constexpr (MERGE) merge_statistics<CH>(p.merge, ss_lds, tid, bx == 0);

    // ---- where this lane's results go (channel ko; four consecutive pixels per register quad) and its skip values, all
    //      requested before the first store: r may alias out element for element
    uint32_t o_off[NT][4];
    int o_left[NT][4];  // pixels of the row from the quad's first on, 0 where there is no quad or no channel
    f4_t rv[NT][4];
    const __amdgpu_buffer_rsrc_t r_rs = rsrc(p.ep != EP_STORE ? p.r : p.out, p.ep != EP_STORE ? p.r_bytes : 0u);
#pragma unroll
    for (int t = 0; t < NT; ++t)
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            const int quad = (wp * NT + t) * 8 + 2 * i + kg;
            const QuadAt at(s, quad);
            const int n = n0 + at.img, row = row0 + at.row;
            o_left[t][i] = ko_ok && quad < s.quads && n < s.N && row < s.H ? s.W - 4 * at.q : 0;
            const uint32_t pix = (uint32_t)(row * s.W + 4 * at.q);
            o_off[t][i] = ((uint32_t)n * p.osn + pix + (uint32_t)ko * p.osc) * 4u;
            if (p.ep != EP_STORE)
                rv[t][i] = load4(r_rs, o_left[t][i] > 0 ? ((uint32_t)n * p.rsn + pix + (uint32_t)ko * p.rsc) * 4u : kNowhere, 0);
        }
    // ---- activation operands: pixel l32 of each tile
    const char *win[NT];
#pragma unroll
    for (int t = 0; t < NT; ++t) {
        const QuadAt at(s, (wp * NT + t) * 8 + (l32 >> 2));
        win[t] = lds + (at.rec(s) + (l32 & 3)) * REC + kg * 16;
    }
    constexpr int CHAINS = ORDER == kHalves ? 2 : 1;
    float16_t acc[CHAINS][NT];
#pragma unroll
    for (int h = 0; h < CHAINS; ++h)
#pragma unroll
        for (int t = 0; t < NT; ++t)
#pragma unroll
            for (int i = 0; i < 16; ++i) acc[h][t][i] = 0.f;

    if (MERGE) __syncthreads();  // scale and shift are there
    st.commit(s, lds, ss_lds, bn);
    constexpr int CS = ORDER == kHalves ? 1 : ORDER;  // 16-channel steps of a chunk
    // Steps of the filter that are there before the first is used: all, or a chunk where 64 channels have to be converted
    // (the next step's 72 fp32 taps beside the operands of all four spilled 84 to 116 registers: forward of three blocks
    // of 34 channels, 12 images of 28x28, 200 us, now 158).
    constexpr int AHEAD = W32 && CH == 64 ? CS : KS;
#pragma unroll
    for (int ks = KS1; ks < AHEAD; ++ks) load_filter<W32>(w_rs, p, ko, ks, kg, w[ks]);
    __syncthreads();
    const int row_bytes = s.pitch * REC;
#pragma unroll
    for (int c0 = 0; c0 < KS; c0 += CS) {
        if (AHEAD < KS && c0 > 0) {
#pragma unroll
            for (int ks = c0; ks < c0 + CS; ++ks) load_filter<W32>(w_rs, p, ko, ks, kg, w[ks]);
        }
        const int h = ORDER == kHalves && c0 >= 2 ? 1 : 0;
#pragma unroll
        for (int tap = 0; tap < 9; ++tap)
#pragma unroll
            for (int ks = c0; ks < c0 + CS; ++ks) {
                bf16x8_t a[NT];
#pragma unroll
                for (int t = 0; t < NT; ++t) a[t] = *reinterpret_cast<const bf16x8_t *>(win[t] + tap / 3 * row_bytes + (tap % 3 * REC + ks * 32));
#pragma unroll
                for (int t = 0; t < NT; ++t) acc[h][t] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a[t], w[ks][tap], acc[h][t], 0, 0, 0);
            }
    }
    if constexpr (ORDER == kHalves) {
#pragma unroll
        for (int t = 0; t < NT; ++t)
#pragma unroll
            for (int i = 0; i < 16; ++i) acc[0][t][i] += acc[1][t][i];
    }

    // ---- epilogue
    const __amdgpu_buffer_rsrc_t o_rs = rsrc(p.out, p.out_bytes);
#pragma unroll
    for (int t = 0; t < NT; ++t)
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            f4_t v = {acc[0][t][4 * i], acc[0][t][4 * i + 1], acc[0][t][4 * i + 2], acc[0][t][4 * i + 3]};
            if (p.ep == EP_ADD) v = rv[t][i] + v;
            if (p.ep == EP_SUB) v = rv[t][i] - v;
#pragma unroll
            for (int j = 0; j < 4; ++j) acc[0][t][4 * i + j] = v[j];
            const int left = o_left[t][i];
            store4(o_rs, left >= 4 ? o_off[t][i] : kNowhere, v);
            if (GEN) {
#pragma unroll
                for (int j = 0; j < 3; ++j)
                    __builtin_amdgcn_raw_buffer_store_b32(__float_as_uint(v[j]), o_rs, left < 4 && j < left ? o_off[t][i] + 4u * j : kNowhere, 0, 0);
            }
        }
    // Statistics of what was stored, for the BN layer that reads it next: per channel and 64 consecutive pixels, sums of
    // (v - pivot) and (v - pivot)^2, pivot = the first value.  The order is that of the kernels that take the layer at
    // other sizes (pixel p and p + 32, then halves down to neighbours; the compiler contracts their first sum of squares,
    // also the one across lanes in the kernel that sums a split layer, to the fma below), so a tensor's statistics
    // are the same bits.
    if constexpr (EMIT) {
        float hi[16];  // the later 32 pixels of the 64 that this lane sums
        if constexpr (NT == 2) {
#pragma unroll
            for (int i = 0; i < 16; ++i) hi[i] = acc[0][1][i];
        } else {  // they are the next wavefront's along the pixels
            f4_t *const swap = reinterpret_cast<f4_t *>(lds) + (wave / (2 * WM) * WM + wm) * 4 * 64 + lane;
            __syncthreads();  // the operands have been read
            if (wp & 1) {
#pragma unroll
                for (int i = 0; i < 4; ++i)
                    swap[i * 64] = f4_t{acc[0][0][4 * i], acc[0][0][4 * i + 1], acc[0][0][4 * i + 2], acc[0][0][4 * i + 3]};
            }
            __syncthreads();
            if (wp & 1) return;
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                const f4_t v = swap[i * 64];
#pragma unroll
                for (int j = 0; j < 4; ++j) hi[4 * i + j] = v[j];
            }
        }
        const float pivot = __shfl(acc[0][0][0], l32, 64);
        float ea[16], eb[16];
#pragma unroll
        for (int i = 0; i < 16; ++i) {
            const float d0 = acc[0][0][i] - pivot, d1 = hi[i] - pivot;
            ea[i] = d0 + d1;
            eb[i] = fmaf(d0, d0, d1 * d1);
        }
        // register i of a lane is pixel 8 * (i / 4) + 4 * kg + i % 4
#pragma unroll
        for (int h = 8; h >= 4; h >>= 1)
#pragma unroll
            for (int i = 0; i < h; ++i) {
                ea[i] += ea[i + h];
                eb[i] += eb[i + h];
            }
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            ea[i] += __shfl_xor(ea[i], 32, 64);
            eb[i] += __shfl_xor(eb[i], 32, 64);
        }
        const float s1 = (ea[0] + ea[2]) + (ea[1] + ea[3]), s2 = (eb[0] + eb[2]) + (eb[1] + eb[3]);
        if (kg == 0 && ko_ok) {
            constexpr float inv = 1.f / 64;
            const int tile = NT == 2 ? bx * WP + wp : bx * (WP / 2) + wp / 2;
            reinterpret_cast<float2 *>(p.emit)[(int64_t)ko * p.emit_tiles + tile] =
                make_float2(pivot + s1 * inv, fmaxf(s2 - s1 * s1 * inv, 0.f));
        }
    }
}

}  // namespace c3n

}  // namespace

}  // namespace rvn
