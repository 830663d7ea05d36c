// FP32 decode on the FP16 matrix cores, every FP32 factor split into two FP16 halves.
//
// A weight or activation x (scaled by a power of two) is h + l with h = fp16(x) and
// l = fp16(x - h): 22 bits and the sign of l, so |x - h - l| <= 2^-23 of its binade.  A product
// is h h' + h l' + l h' (l l' lies below 2^-24 of it), three v_mfma_f32_16x16x32_f16 with FP32
// accumulation in the place of eight v_mfma_f32_16x16x4_f32: 48 matrix-core cycles per 16 x 16
// x 32 product instead of 256.  The matrix cores sum 32 products with fewer roundings than an FP32
// chain, which pays for the bits the halves leave (split_parts).
//
// Ranges.  FP16 holds 2^-24 .. 2^16, FP32 far more, so every layer has its own powers of two,
// chosen when the material is loaded (prepare_decode_split) from the largest texel and the
// absolute row sums of the weights: with S_k x_k below 2^15 for every query whose direction
// components are at most kSplitMaxDir no half can overflow, and the subnormal step of the low
// half, propagated to the output, stays below the FP32 rounding there.  A material that has no
// such scales (non-finite or extreme values) keeps the FP32 kernels.
//
// A query with larger directions (not normalised) is decoded again with its input and all biases times
// the power of two that brings them into range, which the ReLUs pass on to the output: exact, and with
// components up to 2^15 the codes' low halves still reach 2^-25 of the largest code.  A query with
// directions beyond or not finite, or with a learned frame so short before its normalisation that the
// halves' step shows in its direction, is decoded in FP32 on the vector ALU by the wave that finds it.
//
// Work decomposition and operand layouts are those of the FP16 decode (decode_mfma.h): a wave
// fetches and decodes chunks of 64 queries on its own, weights in LDS as the A operand, one query
// per column, each A operand read once for the chunk's 4 tiles, accumulators becoming the next
// layer's B operand in place.  FP32 texels: C / 4 lanes share a texel, 16 bytes each, so a load
// instruction covers the whole texels of 256 / C queries.
#pragma once

#include "decode_mfma.h"
#include "decode_vec.h"

#include <type_traits>

namespace nam {

constexpr float kSplitMaxDir = 2.0f;      // direction components up to here stay on the split path as they are,
constexpr float kSplitFarDir = 32768.0f;  // up to here by a power of two

struct SplitArgs {
    PyrArgs pyr;
    const float* tex;          // FP32 texels (below 4 GiB)
    const uint4* w;            // A blocks in the order of mfma_pack.h, 64 x 16 bytes per part (layer 0: 3 parts)
    const floatx4* bias;       // per (layer, row tile): 4 lane groups x 4 biases, in accumulator scale
    const half4* wf;           // frame layer: A operand of v_mfma_f32_16x16x16_f16, 64 x 3 parts
    const floatx4* fbias;      // its biases per lane group, in accumulator scale
    float one;                 // 1.0f (split_pair)
    float sz, sd;              // scales of the latent code and of the directions in the network input
    float finv[4];             // frame layer accumulator to its vectors
    float shortest2;           // square of the shortest frame vector that stays on the split path
    float c[kMaxLayers];       // half of: accumulator of layer k to the input of layer k + 1
    float oinv[6];             // output accumulator row to q
    int n;
    int nchunks;
    int groups;                // XCD groups: min(8, grid); the grid is a multiple of it
    int wpb;                   // waves of a workgroup that take chunks
    int nf;                    // learned shading frames
    const float2* uv;
    const float* lod;
    const float* xi;
    const float* wi;
    const float* wo;
    float* rgb;
    const float* wt32;         // FP32 decoder, transposed per layer, and frame layer (queries handed back)
    const float* frames32;
};

// Two values split into halves, h = fp16(y) and l = fp16(y - h) (y - h is exact).  Written for the
// rates measured on gfx950 (cycles per wave and SIMD: FP32 add, multiply, multiply-add 2.7; max,
// mixed multiply-add, packed conversion 4.7; the mixed multiply-adds that write a half, exp2 and rcp
// 8.5): one packed conversion per half pair and a mixed multiply-add per value.  The empty
// statements keep the compiler from converting y once more to read one half of h, and from fusing
// y - h with its conversion into the slower form; `one` is 1.0f in a register it cannot see
// through, which keeps y - h a mixed multiply-add.
__device__ __forceinline__ void split_pair(float y0, float y1, float one, half2_t& h, half2_t& l, half2_t* rest = nullptr) {
    h = half2_t{(_Float16)y0, (_Float16)y1};
    asm("" : "+v"(h));
    float r0 = fmaf(y0, one, -(float)h[0]), r1 = fmaf(y1, one, -(float)h[1]);
    asm("" : "+v"(r0), "+v"(r1));
    l = half2_t{(_Float16)r0, (_Float16)r1};
    if (rest) {                               // what both halves leave (the last bit), where a caller has room for it
        asm("" : "+v"(l));
        float q0 = fmaf(r0, one, -(float)l[0]), q1 = fmaf(r1, one, -(float)l[1]);
        asm("" : "+v"(q0), "+v"(q1));
        *rest = half2_t{(_Float16)q0, (_Float16)q1};
    }
}

// 2 max(x, 0), exact, by an addition (2.7 cycles where a max takes 4.7); a NaN stays.
__device__ __forceinline__ float relu_twice(float x) { return x + fabsf(x); }

// softplus(q) = max(q, 0) + log1p(e), e = exp(-|q|), to about one rounding.  e = 2^f 2^i from the
// argument split at its nearest integer, f in two steps (the second adds the low part of log2 e);
// log1p(e) = 2 atanh(s / 2), s = e / (1 + e / 2) <= 2/3, by the series in s^2 (the first term left out is
// below 2^-27 of the sum), with the quotient's remainder, that of the rounded 1 + e / 2 included, added
// to the small terms.  The smallest e (subnormal) pass through unchanged.  Past |q| = 128, where e is
// below every FP32 number, x stays -128: the split of a larger argument would leave more in f than exp2
// takes.  A NaN stays.
// (Contracting s into the last sum would count its rounding twice.)
__device__ __forceinline__ float softplus_split(float q) {
    #pragma clang fp contract(off)
    const float x = fabsf(q) > 128.0f ? -128.0f : -fabsf(q);
    const float i = __builtin_rintf(x * 1.44269502162933349609375f);
    float f = fmaf(x, 1.44269502162933349609375f, -i);
    f = fmaf(x, 1.92596299e-8f, f);
    const float e = ldexpf(__builtin_amdgcn_exp2f(f), (int)i);
    const float u = fmaf(0.5f, e, 1.0f), ul = fmaf(0.5f, e, -(u - 1.0f)), r = __builtin_amdgcn_rcpf(u);
    const float s = e * r;
    const float sl = fmaf(-s, ul, fmaf(-s, u, e)) * r;
    const float t = s * s;
    float p = 1.0f / (15 << 14);
    p = fmaf(p, t, 1.0f / (13 << 12));
    p = fmaf(p, t, 1.0f / (11 << 10));
    p = fmaf(p, t, 1.0f / (9 << 8));
    p = fmaf(p, t, 1.0f / (7 << 6));
    p = fmaf(p, t, 1.0f / (5 << 4));
    p = fmaf(p, t, 1.0f / (3 << 2));
    return fmaxf(q, 0.0f) + (s + fmaf(s * t, p, sl));
}

// Parts of a weight: high and low half, and where a third is kept what those two leave (a weight's
// last bit).  With it the sums also take the product of the low halves: five products in the place of
// three, for the layers of few inputs, whose FP32 sums have few roundings to beat.  Measured error of
// one layer against 64 bits (2-norm, weights uniform, inputs ReLU of normal; FP32 chain / three / five
// products): 16 inputs 5.5e-8 / 8.6e-8 / 5.7e-8, 24 6.6 / 8.7 / 6.0, 32 7.5 / 8.9 / 6.2, 64 10.3 / 9.6 / 7.2.
__host__ __device__ constexpr int split_parts(int inputs) { return inputs <= 32 ? 3 : 2; }

// The chunk's 4 tiles through one row tile: acc[t] = b[t] + W x[t] over KS K steps (the tiles are
// independent chains).  Small products first, before the roundings of the large ones.
template <int KS, int P>
__device__ __forceinline__ void split_tiles(const half8 (&a)[KS][P], const half8 (&bh)[4][KS], const half8 (&bl)[4][KS],
                                            const floatx4 (&b)[4], floatx4* acc, int stride) {
    #pragma unroll
    for (int s = 0; s < KS; ++s) {
        if constexpr (P == 3) {
            #pragma unroll
            for (int t = 0; t < 4; ++t) acc[t * stride] = mfma_f16(a[s][2], bh[t][s], s == 0 ? b[t] : acc[t * stride]);
            #pragma unroll
            for (int t = 0; t < 4; ++t) acc[t * stride] = mfma_f16(a[s][1], bl[t][s], acc[t * stride]);
        }
        #pragma unroll
        for (int t = 0; t < 4; ++t) acc[t * stride] = mfma_f16(a[s][1], bh[t][s], P < 3 && s == 0 ? b[t] : acc[t * stride]);
        #pragma unroll
        for (int t = 0; t < 4; ++t) acc[t * stride] = mfma_f16(a[s][0], bl[t][s], acc[t * stride]);
    }
    #pragma unroll
    for (int s = 0; s < KS; ++s)
        #pragma unroll
        for (int t = 0; t < 4; ++t) acc[t * stride] = mfma_f16(a[s][0], bh[t][s], acc[t * stride]);
}

template <int H, int NH, bool AL>
struct SplitSizes {
    static constexpr int RT = H / 16, KS = (H + 31) / 32;
    static constexpr int kOutCopies = AL ? 2 : 4;
    static constexpr int P = split_parts(H);       // parts of a block after layer 0
    static constexpr int NHB = (NH - 1) * RT * KS; // hidden blocks after layer 0
    static constexpr int kW = 8;               // waves: two per SIMD, 8 KiB of LDS each
};

// The queries of `mask` of one chunk in full FP32, as decode_f32_kernel does them: 32 lanes at a
// time, activations in the wave's 8 KiB of LDS.
template <int C, int H, int NH, int NW, int NO>
__device__ __forceinline__ void decode_lanes_f32(const SplitArgs& a, float* table, int first, int lane, bool mine) {
    #pragma unroll 1
    for (int half = 0; half < 2; ++half) {
        if (!mine || (lane >> 5) != half) continue;
        const int i = first + lane;
        float* col = table + (lane & 31);
        const float2 q = a.uv[i];
        const float l = a.lod[i];
        Taps t;
        float z[C], dwi[3], dwo[3], dirs[6 * NW];
        if (a.xi) {
            query_taps_rr(a.pyr, q.x, q.y, l, a.xi[i], t);
            gather_f32<C, 4>(a.tex, t, z);
        } else {
            query_taps(a.pyr, q.x, q.y, l, t);
            gather_f32<C>(a.tex, t, z);
        }
        #pragma unroll
        for (int d = 0; d < 3; ++d) {
            dwi[d] = a.wi[3 * (int64_t)i + d];
            dwo[d] = a.wo[3 * (int64_t)i + d];
        }
        if constexpr (NW == 2) {
            frame_inputs<C, 2>(as_constant(a.frames32), z, dwi, dwo, dirs);
        } else if (a.nf == 1) {
            frame_inputs<C, 1>(as_constant(a.frames32), z, dwi, dwo, dirs);
        } else {
            #pragma unroll
            for (int d = 0; d < 3; ++d) {
                dirs[d] = dwi[d];
                dirs[3 + d] = dwo[d];
            }
        }
        #pragma unroll
        for (int c = 0; c < C; ++c) col[c * 32] = z[c];
        #pragma unroll
        for (int c = 0; c < 6 * NW; ++c) col[(C + c) * 32] = dirs[c];
        const float* W = a.wt32;
        float h[H];
        dense_from_lds<C + 6 * NW, H, 32>(W, col, h);
        W += (C + 6 * NW) * H + H;
        #pragma unroll 1
        for (int k = 1; k < NH; ++k) {
            #pragma unroll
            for (int o = 0; o < H; ++o) col[o * 32] = fmaxf(h[o], 0.0f);
            dense_from_lds<H, H, 32>(W, col, h);
            W += H * H + H;
        }
        #pragma unroll
        for (int o = 0; o < H; ++o) col[o * 32] = fmaxf(h[o], 0.0f);
        float qv[NO];
        dense_from_lds<H, NO, 32>(W, col, qv);
        #pragma unroll
        for (int c = 0; c < NO; ++c) a.rgb[NO * (int64_t)i + c] = softplus_f32(qv[c]);
    }
}

// One workgroup of 8 waves per CU, 254 registers (three waves per SIMD spilled at 168 and were no
// faster).  Measured, 22-64-64-64-3 on the 1080p frame of a 2048^2 x 16 texture: 155 us (592 us on the
// FP32 matrix cores), error against 64 bits 4.3e-8 (7.8e-8); 20-32-32-3 with two frames and the
// stochastic filter, 500,009 queries: 23.8 us (57.5 us on the vector ALU), 4.2e-8 (4.3e-8).  Without its
// texel loads the frame took 110 us: per 64 queries a SIMD issues 296 matrix-core instructions (4,736
// cycles of the matrix pipe) and 1,244 vector ones (about 5,000 cycles) through one port, and twice the
// FP16 decode's texel bytes come from beyond the L2.
template <int C, int H, int NH, bool RR, bool FR, bool AL>
__global__ void __launch_bounds__((SplitSizes<H, NH, AL>::kW * 64), 1) decode_split_kernel(const SplitArgs a) {
    using Z = SplitSizes<H, NH, AL>;
    constexpr int RT = Z::RT, KS = Z::KS, kOutCopies = Z::kOutCopies, kW = Z::kW, kThreads = kW * 64;
    constexpr int NT = RR ? 4 : 8;             // taps per query
    constexpr int P = Z::P, NHB = Z::NHB;
    constexpr int kParts = C / 4;              // lanes that share a texel
    constexpr int kQ = 64 / kParts;            // queries per load round
    struct alignas(16) Smem {
        uint8_t A0[RT][3][1024];
        uint8_t A[NHB + kOutCopies * KS][P][1024];
        floatx4 bias[NH * RT + 1][4];
        LevelRowL rows[kMaxLevels];
        uint8_t wreg[kW][8192];
    };
    __shared__ Smem sm;
    const int lane = threadIdx.x & 63;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int g = lane >> 4, q16 = lane & 15;
    const MfmaLayout lay = mfma_layout(C, H, NH, true, false);
    {
        for (int i = threadIdx.x; i < RT * 192; i += kThreads) reinterpret_cast<uint4*>(sm.A0)[i] = a.w[i];
        const uint4* w = a.w + RT * 192;
        for (int i = threadIdx.x; i < NHB * P * 64; i += kThreads) reinterpret_cast<uint4*>(sm.A)[i] = w[i];
        // output copies, moved to rows 4t.. (albedo head: 8t..) as in decode_mfma_kernel
        constexpr int kRows = AL ? 6 : 3, kStride = AL ? 8 : 4;
        for (int i = threadIdx.x; i < kOutCopies * KS * P * 64; i += kThreads) {
            const int ln = i & 63, part = (i >> 6) % P, s = (i >> 6) / P % KS, t = (i >> 6) / (P * KS);
            const int d = (ln & 15) - kStride * t;
            reinterpret_cast<uint4*>(sm.A[NHB + t * KS + s][part])[ln] =
                (d >= 0 && d < kRows) ? w[((NHB + s) * P + part) * 64 + ln - kStride * t] : make_uint4(0, 0, 0, 0);
        }
        for (int i = threadIdx.x; i < (NH * RT + 1) * 4; i += kThreads) sm.bias[i >> 2][i & 3] = a.bias[i];
        if (threadIdx.x < a.pyr.M) {
            const LevelRow r = a.pyr.rows[threadIdx.x];
            sm.rows[threadIdx.x] = LevelRowL{(float)r.w, (float)r.h, r.w - 1, r.h - 1, (uint32_t)(r.off * C * 4),
                                             (uint32_t)(r.w * C * 4), 0, 0};
        }
    }
    __syncthreads();

    const int X = a.groups;
    const int grp = blockIdx.x % X;
    const int stride = (gridDim.x / X) * a.wpb;
    int c = (int)((int64_t)a.nchunks * grp / X) + (blockIdx.x / X) * a.wpb + wave;
    const int c_end = (int)((int64_t)a.nchunks * (grp + 1) / X);
    if (wave >= a.wpb || c >= c_end) return;
    const int n = a.n;
    // The wave's 8 KiB: the input's K slots 0..15 ([half][tile][g & 1][query] of 16 bytes), then
    // slots 16..31 alike, which first hold the tap table (and the frame layer's outputs)
    uint8_t* const xb = sm.wreg[wave];
    uint8_t* const tb = xb + 4096;
    uint8_t* const xr = xb + (g >> 1) * 4096 + (g & 1) * 256 + q16 * 16;   // this lane's B operand of tile 0, high halves
    const int t_own = lane >> 4;

    half4 fah = {}, fal = {}, fa_rest = {};
    floatx4 fb = {0.0f, 0.0f, 0.0f, 0.0f};
    if constexpr (FR) {
        fah = a.wf[lane];
        fal = a.wf[64 + lane];
        fa_rest = a.wf[128 + lane];
        fb = a.fbias[g];
    }
    // The decoder on the chunk's input in LDS, to the output accumulators of tiles 0-1 and 2-3 (rows as in
    // decode_mfma_kernel).  scaled: tile t's input comes times f[t], its biases are to follow; fo, fo2: those
    // of the lane's queries in out and out2.
    const auto decode = [&](auto scaled, const float (&f)[4], float fo, float fo2, floatx4& out, floatx4& out2) {
        struct Bias {
            floatx4 b[4];
        };
        const auto bias = [&](int row_tile) {
            const floatx4 b = sm.bias[row_tile][g];
            Bias r;
            #pragma unroll
            for (int t = 0; t < 4; ++t) r.b[t] = scaled ? b * f[t] : b;
            return r;
        };
        floatx4 acc[4][RT];
        {
            half8 bh[4][1], bl[4][1];
            #pragma unroll
            for (int t = 0; t < 4; ++t) {
                bh[t][0] = *reinterpret_cast<const half8*>(xr + t * 512);
                bl[t][0] = *reinterpret_cast<const half8*>(xr + t * 512 + 2048);
            }
            #pragma unroll
            for (int j = 0; j < RT; ++j) {
                half8 wa[1][3];
                #pragma unroll
                for (int part = 0; part < 3; ++part) wa[0][part] = *reinterpret_cast<const half8*>(&sm.A0[j][part][lane * 16]);
                split_tiles<1, 3>(wa, bh, bl, bias(j).b, &acc[0][j], RT);
            }
        }
        // output accumulators: tiles 0-1 and 2-3, rows as in decode_mfma_kernel
        const floatx4 bout = AL ? sm.bias[NH * RT][g & 1] : sm.bias[NH * RT][0];
        out = scaled ? bout * fo : bout;
        out2 = scaled ? bout * fo2 : bout;
        #pragma unroll
        for (int kk = 0; kk < NH; ++kk) {
            const float cs = a.c[kk];
            half8 bh[4][KS], bl[4][KS];
            #pragma unroll
            for (int t = 0; t < 4; ++t)
                #pragma unroll
                for (int s = 0; s < KS; ++s)
                    #pragma unroll
                    for (int e = 0; e < 8; e += 2) {
                        const int j = 2 * s + e / 4;
                        half2_t h = {}, l = {}, rest = {};
                        if (H == 16 && e >= 4) continue;
                        split_pair(relu_twice(acc[t][j][e % 4]) * cs, relu_twice(acc[t][j][e % 4 + 1]) * cs, a.one, h, l,
                                   H == 16 ? &rest : nullptr);
                        if (H == 16) {             // 16 inputs: the other 16 K slots take their last bits
                            bh[t][s][e + 4] = rest[0]; bh[t][s][e + 5] = rest[1];
                            bl[t][s][e + 4] = bl[t][s][e + 5] = (_Float16)0.0f;
                        }
                        bh[t][s][e] = h[0]; bh[t][s][e + 1] = h[1];
                        bl[t][s][e] = l[0]; bl[t][s][e + 1] = l[1];
                    }
            if (kk < NH - 1) {
                #pragma unroll
                for (int j = 0; j < RT; ++j) {
                    half8 wa[KS][P];
                    #pragma unroll
                    for (int s = 0; s < KS; ++s)
                        #pragma unroll
                        for (int part = 0; part < P; ++part)
                            wa[s][part] = *reinterpret_cast<const half8*>(&sm.A[kk * RT * KS + j * KS + s][part][lane * 16]);
                    split_tiles<KS, P>(wa, bh, bl, bias((kk + 1) * RT + j).b, &acc[0][j], RT);
                }
            } else {
                #pragma unroll
                for (int low = 1; low >= 0; --low)
                    #pragma unroll
                    for (int t = 0; t < 4; ++t)
                        #pragma unroll
                        for (int s = 0; s < KS; ++s) {
                            const uint8_t(*wt)[1024] = sm.A[NHB + (AL ? (t & 1) : t) * KS + s];
                            const half8 ah = *reinterpret_cast<const half8*>(&wt[0][lane * 16]);
                            floatx4& o = t < 2 ? out : out2;
                            if (low) {
                                const half8 al = *reinterpret_cast<const half8*>(&wt[1][lane * 16]);
                                if constexpr (P == 3) {
                                    o = mfma_f16(*reinterpret_cast<const half8*>(&wt[2][lane * 16]), bh[t][s], o);
                                    o = mfma_f16(al, bl[t][s], o);
                                }
                                o = mfma_f16(al, bh[t][s], o);
                                o = mfma_f16(ah, bl[t][s], o);
                            } else {
                                o = mfma_f16(ah, bh[t][s], o);
                            }
                        }
            }
        }
    };
    // Largest direction component of the lane's query.
    const auto largest = [](const float* dir, bool& finite) {
        float m = 0.0f;
        finite = true;
        #pragma unroll
        for (int d = 0; d < 6; ++d) {
            m = fmaxf(m, fabsf(dir[d]));
            finite = finite && dir[d] == dir[d];
        }
        return m;
    };
    float2 uv = *chunk_elem<1>(a.uv, n, c * kChunk, lane);
    float lod = *chunk_elem<1>(a.lod, n, c * kChunk, lane);
    float xi = RR ? *chunk_elem<1>(a.xi, n, c * kChunk, lane) : 0.0f;
    for (; c < c_end; c += stride) {
        const int first = c * kChunk;
        const bool use = query_ok(uv.x, uv.y, lod);
        const bool okc = (first + lane < n) && use;
        // ---- taps of the lane's query into the table (offsets, then weights times the input scale)
        {
            uint32_t off[NT];
            float w[NT];
            if (a.pyr.address == NAM_WRAP)
                tap_stencil<C == 16 ? 6 : 5, NAM_WRAP, RR>(a.pyr.M, sm.rows, use, uv.x, uv.y, lod, xi, off, w);
            else
                tap_stencil<C == 16 ? 6 : 5, NAM_CLAMP, RR>(a.pyr.M, sm.rows, use, uv.x, uv.y, lod, xi, off, w);
            #pragma unroll
            for (int k = 0; k < NT; k += 4) {
                *reinterpret_cast<uint4*>(tb + ((k / 4) * 64 + lane) * 16) = make_uint4(off[k], off[k + 1], off[k + 2], off[k + 3]);
                *reinterpret_cast<floatx4*>(tb + ((NT / 4 + k / 4) * 64 + lane) * 16) =
                    floatx4{w[k] * a.sz, w[k + 1] * a.sz, w[k + 2] * a.sz, w[k + 3] * a.sz};
            }
        }
        float dir[6];
        {
            const float* wi = chunk_elem<3>(a.wi, n, first, lane);
            const float* wo = chunk_elem<3>(a.wo, n, first, lane);
            #pragma unroll
            for (int d = 0; d < 3; ++d) {
                dir[d] = wi[d];
                dir[3 + d] = wo[d];
            }
        }
        lds_wave_sync();
        // ---- texels: lane (q, p) takes channels 4p..4p+3 of queries q + kQ r, two rounds in flight
        {
            const int q = lane % kQ, p = lane / kQ;
            const uint8_t* tex = reinterpret_cast<const uint8_t*>(a.tex);
            #pragma unroll
            for (int rr = 0; rr < kParts; rr += 2) {
                floatx4 tl[2][NT];
                #pragma unroll
                for (int r = 0; r < 2; ++r) {
                    const int Q = (rr + r) * kQ + q;
                    #pragma unroll
                    for (int k = 0; k < NT; k += 4) {
                        const uint4 o = *reinterpret_cast<const uint4*>(tb + ((k / 4) * 64 + Q) * 16);
                        tl[r][k] = *reinterpret_cast<const floatx4*>(tex + (o.x + 16u * (uint32_t)p));
                        tl[r][k + 1] = *reinterpret_cast<const floatx4*>(tex + (o.y + 16u * (uint32_t)p));
                        tl[r][k + 2] = *reinterpret_cast<const floatx4*>(tex + (o.z + 16u * (uint32_t)p));
                        tl[r][k + 3] = *reinterpret_cast<const floatx4*>(tex + (o.w + 16u * (uint32_t)p));
                    }
                }
                if (rr == 0) {                                        // the next chunk's queries
                    const int nf = (c + stride) * kChunk;
                    uv = *chunk_elem<1>(a.uv, n, nf, lane);
                    lod = *chunk_elem<1>(a.lod, n, nf, lane);
                    if constexpr (RR) xi = *chunk_elem<1>(a.xi, n, nf, lane);
                }
                __builtin_amdgcn_sched_barrier(0);                    // two rounds' texels in registers, not four
                #pragma unroll
                for (int r = 0; r < 2; ++r) {
                    const int Q = (rr + r) * kQ + q;
                    floatx4 z = {0.0f, 0.0f, 0.0f, 0.0f};
                    #pragma unroll
                    for (int k = 0; k < NT; k += 4) {
                        const floatx4 ww = *reinterpret_cast<const floatx4*>(tb + ((NT / 4 + k / 4) * 64 + Q) * 16);
                        #pragma unroll
                        for (int e = 0; e < 4; ++e)
                            #pragma unroll
                            for (int d = 0; d < 4; ++d) z[d] = fmaf(ww[e], tl[r][k + e][d], z[d]);
                    }
                    half4 zh, zl;
                    #pragma unroll
                    for (int d = 0; d < 4; d += 2) {
                        half2_t h, l;
                        split_pair(z[d], z[d + 1], a.one, h, l);
                        zh[d] = h[0]; zh[d + 1] = h[1];
                        zl[d] = l[0]; zl[d + 1] = l[1];
                    }
                    uint8_t* dst = xb + (Q >> 4) * 512 + (p >> 1) * 256 + (Q & 15) * 16 + (p & 1) * 8;
                    *reinterpret_cast<half4*>(dst) = zh;
                    *reinterpret_cast<half4*>(dst + 2048) = zl;
                }
                __builtin_amdgcn_sched_barrier(0);
            }
        }
        lds_wave_sync();                                              // the table is spent, z is written
        // ---- directions (or their frame transforms) after z, zeros up to slot 32
        bool bad, far;
        {
            bool fin;
            const float m = largest(dir, fin);
            bad = okc && !(fin && m <= kSplitFarDir);
            far = okc && !bad && m > kSplitMaxDir;
            if (__builtin_expect(__ballot(far) != 0, 0)) {
                #pragma unroll
                for (int d = 0; d < 6; ++d) dir[d] = far ? ldexpf(dir[d], 1 - __builtin_amdgcn_frexp_expf(m)) : dir[d];
            }
            // the output layer sums the tiles' products with zero rows for the other tiles: no lane may bring an
            // infinity there, also none without a result (past the batch, non-finite uv or lod)
            #pragma unroll
            for (int d = 0; d < 6; ++d) dir[d] = bad || !okc ? 0.0f : dir[d];
            float x[24];
            #pragma unroll
            for (int k = 0; k < 24; ++k) x[k] = 0.0f;
            if constexpr (FR) {
                // the frame layer on the matrix cores: K = 16 channels (lane (g, q): 4g..4g+3)
                #pragma unroll
                for (int t = 0; t < 4; ++t) {
                    half4 zh = {}, zl = {};
                    if (C == 16 || g < 2) {
                        const uint8_t* src = xb + t * 512 + (g >> 1) * 256 + q16 * 16 + (g & 1) * 8;
                        zh = *reinterpret_cast<const half4*>(src);
                        zl = *reinterpret_cast<const half4*>(src + 2048);
                    }
                    floatx4 o = __builtin_amdgcn_mfma_f32_16x16x16f16(fa_rest, zh, fb, 0, 0, 0);
                    o = __builtin_amdgcn_mfma_f32_16x16x16f16(fal, zl, o, 0, 0, 0);
                    o = __builtin_amdgcn_mfma_f32_16x16x16f16(fal, zh, o, 0, 0, 0);
                    o = __builtin_amdgcn_mfma_f32_16x16x16f16(fah, zl, o, 0, 0, 0);
                    o = __builtin_amdgcn_mfma_f32_16x16x16f16(fah, zh, o, 0, 0, 0);
                    if (g < 3) *reinterpret_cast<floatx4*>(tb + ((t * 3 + g) * 16 + q16) * 16) = o;
                }
                lds_wave_sync();
                float v[12];
                #pragma unroll
                for (int gg = 0; gg < 3; ++gg) {
                    const floatx4 o = *reinterpret_cast<const floatx4*>(tb + ((t_own * 3 + gg) * 16 + q16) * 16);
                    #pragma unroll
                    for (int e = 0; e < 4; ++e) v[4 * gg + e] = o[e] * a.finv[(4 * gg + e) / 3];
                }
                #pragma unroll
                for (int k = 0; k < 4; ++k) {
                    if (k >= 2 && a.nf < 2) continue;
                    const float ss = fmaf(v[3 * k], v[3 * k], fmaf(v[3 * k + 1], v[3 * k + 1], v[3 * k + 2] * v[3 * k + 2]));
                    bad = bad || (okc && fmaxf(ss, 1e-12f) < a.shortest2);
                }
                lds_wave_sync();                                      // tb takes the directions
                if (a.nf == 2) {
                    frame_apply<2>(0, v, dir, dir + 3, x);
                    frame_apply<2>(1, v + 6, dir, dir + 3, x);
                } else {
                    frame_apply<1>(0, v, dir, dir + 3, x);
                }
            } else {
                #pragma unroll
                for (int d = 0; d < 6; ++d) x[d] = dir[d];
            }
            #pragma unroll
            for (int gg = C / 8; gg < 4; ++gg) {
                half8 h, l;
                #pragma unroll
                for (int e = 0; e < 8; e += 2) {
                    const int k = 8 * (gg - C / 8) + e;
                    half2_t hh, ll;
                    split_pair(x[k] * a.sd, x[k + 1] * a.sd, a.one, hh, ll);
                    h[e] = hh[0]; h[e + 1] = hh[1];
                    l[e] = ll[0]; l[e + 1] = ll[1];
                }
                uint8_t* dst = xb + (gg >> 1) * 4096 + t_own * 512 + (gg & 1) * 256 + q16 * 16;
                *reinterpret_cast<half8*>(dst) = h;
                *reinterpret_cast<half8*>(dst + 2048) = l;
            }
        }
        lds_wave_sync();

        // ---- the decoder
        floatx4 out, out2;
        const float unscaled[4] = {1.0f, 1.0f, 1.0f, 1.0f};
        __builtin_amdgcn_s_setprio(1);
        decode(std::false_type{}, unscaled, 1.0f, 1.0f, out, out2);
        __builtin_amdgcn_s_setprio(0);
        const uint64_t badm = __ballot(bad), farm = __ballot(far && !bad);
        // the results of the queries in `of`, times 2^k of the lane's query
        const uint64_t okm = __ballot(okc);
        const auto store = [&](auto scaled, uint64_t of, int k) {
            if constexpr (AL) {
                const int half_sel = g & 1;
                float* dst = a.rgb + 6 * (int64_t)first;
                #pragma unroll
                for (int h = 0; h < 2; ++h) {
                    const floatx4 o = h == 0 ? out : out2;
                    const int qi = (2 * h + (g >> 1)) * 16 + q16;
                    const bool okq = (okm >> qi) & 1;
                    const int kq = scaled ? __shfl(k, qi, 64) : 0;
                    if (first + qi < n && ((of >> qi) & 1)) {
                        #pragma unroll
                        for (int i = 0; i < 4; ++i)
                            if (i < 2 || !half_sel) {
                                const float q = o[i] * (half_sel ? a.oinv[i < 2 ? 4 + i : 0] : a.oinv[i]);
                                dst[6 * qi + 4 * half_sel + i] = okq ? softplus_split(scaled ? ldexpf(q, kq) : q) : __builtin_nanf("");
                            }
                    }
                }
            } else {
                Rgb v;
                float* vp = &v.r;
                #pragma unroll
                for (int i = 0; i < 3; ++i) {
                    const float q = (g < 2 ? out[i] : out2[i]) * a.oinv[i];
                    const float sp = softplus_split(scaled ? ldexpf(q, k) : q);
                    vp[i] = okc ? sp : __builtin_nanf("");
                }
                if (first + lane < n && ((of >> lane) & 1)) reinterpret_cast<Rgb*>(a.rgb + 3 * (int64_t)first)[lane] = v;
            }
        };
        store(std::false_type{}, ~(badm | farm), 0);
        if (__builtin_expect(farm != 0, 0)) {                         // uniform, rare
            int k = 0;
            if (far) {
                const float* wi = chunk_elem<3>(a.wi, n, first, lane);
                const float* wo = chunk_elem<3>(a.wo, n, first, lane);
                float d6[6] = {wi[0], wi[1], wi[2], wo[0], wo[1], wo[2]};
                bool fin;
                k = __builtin_amdgcn_frexp_expf(largest(d6, fin)) - 1;
            }
            const float f = ldexpf(1.0f, -k);
            const _Float16 fh = (_Float16)f;
            lds_wave_sync();                                          // the input has been read
            #pragma unroll
            for (int gg = 0; gg < C / 8; ++gg)
                #pragma unroll
                for (int part = 0; part < 2; ++part) {
                    half8* z = reinterpret_cast<half8*>(xb + t_own * 512 + gg * 256 + q16 * 16 + part * 2048);
                    *z = *z * fh;
                }
            lds_wave_sync();
            float ft[4];
            #pragma unroll
            for (int t = 0; t < 4; ++t) ft[t] = __shfl(f, t * 16 + q16, 64);
            const float fo = AL ? ((g >> 1) ? ft[1] : ft[0]) : f, fo2 = AL ? ((g >> 1) ? ft[3] : ft[2]) : f;
            decode(std::true_type{}, ft, fo, fo2, out, out2);
            store(std::true_type{}, farm, k);
        }
        if (badm) {                                                   // uniform, rare
            lds_wave_sync();
            float* table = reinterpret_cast<float*>(xb);
            if (FR && a.nf == 2) decode_lanes_f32<C, H, NH, 2, AL ? 6 : 3>(a, table, first, lane, bad);
            else decode_lanes_f32<C, H, NH, 1, AL ? 6 : 3>(a, table, first, lane, bad);
            lds_wave_sync();
        }
    }
}

template <int C, int H, int NH, bool RR, bool FR, bool AL>
static hipError_t launch_split_shape(SplitArgs& a, int cu_count, hipStream_t s) {
    constexpr int kW = SplitSizes<H, NH, AL>::kW;
    // One workgroup per CU (its LDS holds the decoder).  A small batch is spread over the CUs, a
    // few waves on each, instead of filling some: a chunk's time is its own latency there.
    int grid = std::min(cu_count, a.nchunks);
    if (grid >= 8) grid -= grid % 8;
    a.groups = std::min(grid, 8);
    a.wpb = std::min(kW, (a.nchunks + grid - 1) / grid);
    clear_stale_hip_error();
    decode_split_kernel<C, H, NH, RR, FR, AL><<<grid, kW * 64, 0, s>>>(a);
    return hipGetLastError();
}

template <bool RR, bool FR, bool AL>
static hipError_t dispatch_split_shape(const MlpShape& sh, SplitArgs& a, int cu, hipStream_t s) {
#define NAM_S_CASE(C_, H_, NH_) \
    if (sh.C == C_ && sh.H == H_ && sh.NH == NH_) return launch_split_shape<C_, H_, NH_, RR, FR, AL>(a, cu, s);
#define NAM_S_H(C_, H_) NAM_S_CASE(C_, H_, 1) NAM_S_CASE(C_, H_, 2) NAM_S_CASE(C_, H_, 3) NAM_S_CASE(C_, H_, 4)
    NAM_S_H(8, 16) NAM_S_H(8, 32) NAM_S_H(8, 64)
    NAM_S_H(16, 16) NAM_S_H(16, 32) NAM_S_H(16, 64)
#undef NAM_S_H
#undef NAM_S_CASE
    return hipErrorInvalidValue;
}

template <bool FR, bool AL>
static hipError_t dispatch_split_filter(const MlpShape& sh, SplitArgs& a, int cu, hipStream_t s) {
    return a.xi ? dispatch_split_shape<true, FR, AL>(sh, a, cu, s) : dispatch_split_shape<false, FR, AL>(sh, a, cu, s);
}

// The four kernel families, each instantiated in a translation unit of its own.
hipError_t dispatch_split(const MlpShape& sh, SplitArgs& a, int cu, hipStream_t s);
hipError_t dispatch_split_frames(const MlpShape& sh, SplitArgs& a, int cu, hipStream_t s);
hipError_t dispatch_split_albedo(const MlpShape& sh, SplitArgs& a, int cu, hipStream_t s);
hipError_t dispatch_split_frames_albedo(const MlpShape& sh, SplitArgs& a, int cu, hipStream_t s);

}  // namespace nam
