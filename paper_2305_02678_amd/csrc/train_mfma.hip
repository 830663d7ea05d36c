// Matrix-core training kernels (layouts and the scheme are described in train_mfma.h).
#include "train_mfma.h"

namespace nam {

constexpr int kTMPairs = 4;                     // pairs of a front and a back wave per workgroup
constexpr int kTMThreads = 2 * 64 * kTMPairs;
constexpr int kTMFwdWaves = 8;                  // forward kernel: waves per workgroup

// softplus and its derivative, the logistic function, in FP32 on the hardware exp2, log2 and
// reciprocal (a few ulp).  Both start from e = exp(-|q|), which the compiler shares between them;
// log1p(e) = log(1 + e) e / ((1 + e) - 1) is Kahan's correction of the rounding of 1 + e (e itself
// where 1 + e rounds to 1), and logistic(q) = 1 / (1 + e) for q >= 0 and e / (1 + e) below.  The
// shapes in natural order keep the library's functions, as their vector kernel had them.
template <bool EXACT>
__device__ __forceinline__ float tm_softplus(float q) {
    if constexpr (EXACT) return fmaxf(q, 0.0f) + log1pf(expf(-fabsf(q)));
    const float e = __builtin_amdgcn_exp2f(-fabsf(q) * 1.44269504088896341f);
    const float u = 1.0f + e, d = u - 1.0f;
    const float l = d == 0.0f ? e : (__builtin_amdgcn_logf(u) * 0.693147180559945309f) * (e * __builtin_amdgcn_rcpf(d));
    return fmaxf(q, 0.0f) + l;
}
template <bool EXACT>
__device__ __forceinline__ float tm_logistic(float q) {
    if constexpr (EXACT) return 1.0f / (1.0f + expf(-q));
    const float e = __builtin_amdgcn_exp2f(-fabsf(q) * 1.44269504088896341f);
    const float r = __builtin_amdgcn_rcpf(1.0f + e);
    return q >= 0.0f ? r : e * r;
}

__device__ __forceinline__ f32x4 ld4(const float* p) { return *reinterpret_cast<const f32x4*>(p); }
__device__ __forceinline__ void st4(float* p, f32x4 v) { *reinterpret_cast<f32x4*>(p) = v; }

__device__ __forceinline__ bool no_weights(const float* __restrict__ w, int count) {
    bool none = true;
    for (int j = 0; j < count && none; j += 16) {             // 16 loads under way
        float v[16];
        #pragma unroll
        for (int c = 0; c < 16; ++c) v[c] = w[min(j + c, count - 1)];
        #pragma unroll
        for (int c = 0; c < 16; ++c) none = none && v[c] == 0.0f;
    }
    return none;
}

// FP32 blocks of TrainLayout (everything ahead of AW) from packed parameters, one thread per float.  p:
// the decoder; fp: the frame layer (NF > 0).
template <int C, int H, int NH, int NF>
__device__ __forceinline__ float packed_float(const float* __restrict__ p, const float* __restrict__ fp, int NO, int e) {
    using L = TrainLayout<C, H, NH, NF>;
    constexpr int IN = L::IN, HT = L::HT;
    const auto nat = [](int i) { return slot_neuron<L::NAT>(i); };
    const int oo = param_off<IN, H>(NH + 1);
    if (e < L::FWH) {
        const int x = e - L::FW1, qq = x & 3, lane = (x >> 2) & 63, blk = x >> 8;
        const int grp = blk % L::G1, tp = blk / L::G1, g = lane >> 4, o = 16 * tp + nat(lane & 15);
        const int q = 4 * grp + qq;
        if (q < L::Q1) {
            const int in = L::NAT ? 4 * q + g : slot_input<C>(q, g);
            if (in >= 0 && in < IN) return p[o * IN + in];
            if (!L::NAT && in == C + 6) return p[IN * H + o];
        }
    } else if (e < L::FWO) {
        const int k = 2 + (e - L::FWH) / L::WH_SZ, x = (e - L::FWH) % L::WH_SZ;
        const int r = x & 3, lane = (x >> 2) & 63, blk = x >> 8, t = blk % HT, tp = blk / HT;
        return p[param_off<IN, H>(k) + (16 * tp + nat(lane & 15)) * H + 16 * t + nat(4 * (lane >> 4) + r)];
    } else if (e < L::BIAS) {
        const int x = e - L::FWO, r = x & 3, lane = (x >> 2) & 63, t = x >> 8, i = lane & 15;
        if (i < NO) return p[oo + i * H + 16 * t + nat(4 * (lane >> 4) + r)];
    } else if (e < L::FF) {
        const int x = e - L::BIAS, k = 1 + x / (HT * 16), y = x % (HT * 16);   // y = slot 16t + 4g + r
        if (k <= NH) return p[param_off<IN, H>(k) + (k == 1 ? IN : H) * H + (y & ~15) + nat(y & 15)];
        if (y < NO) return p[oo + NO * H + y];
    } else if (e < L::FWD) {
        if (e < L::FFB) {
            const int x = e - L::FF, lane = x & 63, i = lane & 15;
            if (i < 6 * NF) return fp[i * C + 4 * (x >> 6) + (lane >> 4)];
        } else if (e - L::FFB < 6 * NF) {
            return fp[6 * NF * C + e - L::FFB];
        }
    } else {
        const int x = e - L::BF, lane = x & 63, i = lane & 15, o = 4 * (x >> 6) + (lane >> 4);
        if (i < C && o < 6 * NF) return fp[o * C + i];
    }
    return 0.0f;
}

// Input of layer-1 K slot (g, e) of the split forward (-1: none).
template <int C, int NF>
__host__ __device__ constexpr int split_input(int g, int e) {
    if (e < 4) return 4 * g + e < C ? 4 * g + e : -1;
    const int d = 4 * (e - 4) + g;
    return d < 6 * (NF > 1 ? NF : 1) ? C + d : -1;
}

// Exponent that puts a layer's largest weight in [2^14, 2^15) (0 for a layer of zeros); one wave.  With an
// infinite weight there is none: every tile's forward pass runs in FP32.
constexpr int kNoExponent = 1000;
__device__ __forceinline__ int weight_exponent(const float* __restrict__ w, int count, int lane) {
    float m = 0.0f;
    for (int i = lane; i < count; i += 16 * 64) {             // 16 loads under way
        float v[16];
        #pragma unroll
        for (int j = 0; j < 16; ++j) v[j] = w[min(i + 64 * j, count - 1)];
        #pragma unroll
        for (int j = 0; j < 16; ++j) m = fmaxf(m, fabsf(v[j]));
    }
    for (int o = 32; o > 0; o >>= 1) m = fmaxf(m, __shfl_xor(m, o, 64));
    if (!__builtin_isfinite(m)) return kNoExponent;
    return m > 0.0f ? 15 - __builtin_amdgcn_frexp_expf(m) : 0;
}

// Packs a decoder: workgroups [0, nf) write the FP32 blocks, a wave of the later ones one block of
// halves (all its parts) or one layer's exponent.
template <int C, int H, int NH, int NF>
__global__ void __launch_bounds__(256) pack_train_kernel(const float* __restrict__ p, const float* __restrict__ fp,
                                                         int NO, float* __restrict__ blob) {
    using L = TrainLayout<C, H, NH, NF>;
    constexpr int IN = L::IN, HT = L::HT, KS = L::KS, P = L::P, nf = (L::AW + 255) / 256;
    const auto nat = [](int i) { return slot_neuron<L::NAT>(i); };
    const int block = (int)blockIdx.x;
    if (block < nf) {
        const int e = block * 256 + threadIdx.x;
        if (e < L::AW) blob[e] = packed_float<C, H, NH, NF>(p, fp, NO, e);
        return;
    }
    const int lane = threadIdx.x & 63, g = lane >> 4, i = lane & 15;
    int b = (block - nf) * 4 + (threadIdx.x >> 6);
    const auto fan_in = [](int k) { return k == 1 ? IN : H; };
    const auto exponent = [&](int k) {                        // k = 1 .. NH + 1
        return weight_exponent(p + param_off<IN, H>(k), fan_in(k) * (k > NH ? NO : H), lane);
    };
    // the parts of value v(e) for the lane's `halves` K slots, at dst + part * stride bytes
    const auto put = [&](float* dst, int parts, int stride, int halves, int aw, auto v) {
        uint8_t* d = reinterpret_cast<uint8_t*>(dst);
        float w[8];
        #pragma unroll
        for (int e = 0; e < 8; ++e) w[e] = e < halves ? v(e) : 0.0f;
        if (aw == kNoExponent) aw = 0;
        #pragma unroll
        for (int e = 0; e < 8; ++e) {
            if (e >= halves) break;
            float rest = ldexpf(w[e], aw);
            for (int part = 0; part < parts; ++part) {
                const _Float16 h = (_Float16)rest;
                *reinterpret_cast<_Float16*>(d + part * stride + 2 * e) = h;
                const float left = rest - (float)h;
                if (L::ALT) {
                    const _Float16 other = (_Float16)(rest + left);         // exact where h rounded a tie
                    const bool tie = part == parts - 1 && (float)other - rest == left;
                    *reinterpret_cast<_Float16*>(d + L::ALT * 4 + part * stride + 2 * e) = tie ? other : h;
                }
                rest = left;
            }
        }
    };
    const auto hidden_slot = [&](int s, int e) { return 16 * (2 * s + e / 4) + nat(4 * g + e % 4); };
    constexpr int KB = HT * KS;                               // blocks of a hidden layer
    if (b < NH + 1) {                                         // exponents, and the biases times 2^exponent
        const int k = b + 1, aw = exponent(k), fi = fan_in(k), o = 16 * (lane >> 4) + nat(i);
        const float* w = p + param_off<IN, H>(k);
        if (lane == 0) reinterpret_cast<int*>(blob)[L::AW + k] = aw;
        float v = 0.0f;
        if (k > NH) v = lane < NO ? w[NO * H + lane] : 0.0f;
        else if (lane < H) v = w[fi * H + o];
        const bool none = k <= NH && lane < H && v == 0.0f && no_weights(w + o * fi, fi);
        v = none ? __builtin_nanf("") : ldexpf(v, aw == kNoExponent ? 0 : aw);
        if (lane < (k > NH ? 16 : H)) blob[L::BA + b * H + lane] = v;
        return;
    }
    b -= NH + 1;
    if (b < HT) {                                             // layer 1
        const int o = 16 * b + nat(i);
        put(blob + L::A1 + b * 768 + lane * 4, 3, 1024, 8, exponent(1), [&](int e) {
            const int in = split_input<C, NF>(g, e);
            return in >= 0 ? p[o * IN + in] : 0.0f;
        });
        return;
    }
    b -= HT;
    if (b < (NH - 1) * KB) {                                  // layers 2..NH
        const int k = 2 + b / KB, s = b % KS, o = 16 * (b % KB / KS) + nat(i);
        put(blob + L::AH + b * P * 256 + lane * 4, P, 1024, 8, exponent(k), [&](int e) {
            const int in = hidden_slot(s, e);
            return in < H ? p[param_off<IN, H>(k) + o * H + in] : 0.0f;
        });
        return;
    }
    b -= (NH - 1) * KB;
    if (b < KS) {                                             // output layer, rows 0..7
        const int aw = exponent(NH + 1);
        if (i < 8)
            put(blob + L::AO + b * P * 128 + (g * 8 + i) * 4, P, 512, 8, aw, [&](int e) {
                const int in = hidden_slot(b, e);
                return i < NO && in < H ? p[param_off<IN, H>(NH + 1) + i * H + in] : 0.0f;
            });
        return;
    }
    b -= KS;
    if (b < HT) {                                             // W_out^T, outputs 0..7
        const int aw = exponent(NH + 1);
        if (g < 2)
            put(blob + L::BO + b * P * 64 + lane * 2, P, 256, 4, aw, [&](int e) {
                const int o = 4 * g + e;
                return o < NO ? p[param_off<IN, H>(NH + 1) + o * H + 16 * b + nat(i)] : 0.0f;
            });
        return;
    }
    b -= HT;
    if (b < L::NR1 * KS) {                                    // W_1^T
        const int in = 16 * (b / KS) + i;
        put(blob + L::B1 + b * P * 256 + lane * 4, P, 1024, 8, exponent(1), [&](int e) {
            const int o = hidden_slot(b % KS, e);
            return in < (NF > 0 ? IN : C) && o < H ? p[o * IN + in] : 0.0f;
        });
    }
}

template <int C, int H, int NH, int NF>
constexpr int pack_train_grid() {
    using L = TrainLayout<C, H, NH, NF>;
    constexpr int waves = NH + 1 + 2 * L::HT + (NH - 1) * L::HT * L::KS + L::KS + L::NR1 * L::KS;
    return (L::AW + 255) / 256 + (waves + 3) / 4;
}

// A tile's query, loaded a tile before its texels.
struct TmQuery {
    float2 uv;
    float lod;
};

// One lane's share of a sample: the texel offsets and weights of its 8 taps (its 4 channels),
// the loaded texel words, the directions it needs and its targets or output gradients (of outputs g
// and 4 + g).
struct TmFetch {
    int off[8];
    float w[8];
    f32x4 v[8];
    float dir[6];
    float t[2];
    bool finite;
};

__device__ __forceinline__ int tm_sample(const TrainArgs& a, int tile, int s) {
    const int64_t i = (int64_t)tile * 16 + s;              // a prefetched tile may lie past the batch
    return i < a.n ? (int)i : a.n - 1;
}

__device__ __forceinline__ void tm_query(const TrainArgs& a, int tile, int s, TmQuery& q) {
    if (a.z_in) return;
    const int ic = tm_sample(a, tile, s);
    q.uv = reinterpret_cast<const float2*>(a.uv)[ic];
    q.lod = a.lod[ic];
}

// dir: with frames all six of the sample; else direction inputs g and 4 + g (0 past the sixth).
template <int C, int NF, bool TRAIN>
__device__ __forceinline__ void tm_issue(const TrainArgs& a, const LevelRow* lrows, int tile, const TmQuery& q, int g,
                                         int s, TmFetch& f) {
    const int ic = tm_sample(a, tile, s);
    const bool fetching = C == 16 || g < 2;
    const int cg = fetching ? 4 * g : 0;
    if (a.z_in) {
        // the sample's given code: channels 4g..4g+3 as a single tap of weight 1; the code is
        // finite only if all C channels are (the other lanes of the sample hold the rest)
        f.v[0] = ld4(a.z_in + (int64_t)ic * C + cg);
        f.w[0] = 1.0f;
        #pragma unroll
        for (int k = 1; k < 8; ++k) {
            f.v[k] = f32x4{0, 0, 0, 0};
            f.w[k] = 0.0f;
            f.off[k] = 0;
        }
        f.off[0] = 0;
    } else {
        f.finite = query_ok(q.uv.x, q.uv.y, q.lod);
        Taps t;
        query_taps_rows(lrows, a.M, a.address, q.uv.x, q.uv.y, q.lod, t);
        #pragma unroll
        for (int k = 0; k < 8; ++k) {
            f.off[k] = (int)t.idx[k] * C + cg;
            f.w[k] = t.w[k];
        }
        if (fetching) {
            #pragma unroll
            for (int k = 0; k < 8; ++k) f.v[k] = ld4(a.tex + f.off[k]);
        }
    }
    if (TRAIN) {
        const float* src = a.target ? a.target : a.d_rgb;
        #pragma unroll
        for (int j = 0; j < 2; ++j) f.t[j] = 4 * j + g < a.NO ? src[(int64_t)a.NO * ic + 4 * j + g] : 0.0f;
    }
    auto dir = [&](int d) { return d < 3 ? a.wi[3 * (int64_t)ic + d] : a.wo[3 * (int64_t)ic + d - 3]; };
    if (NF > 0) {
        #pragma unroll
        for (int d = 0; d < 6; ++d) f.dir[d] = dir(d);
    } else {
        f.dir[0] = dir(g);
        f.dir[1] = g < 2 ? dir(4 + g) : 0.0f;
    }
}

// Registers r of lane group g <-> registers g of lane group r: channels 4g + r become 4r + g.
__device__ __forceinline__ void transpose_groups(float* v) {
    auto swap16 = [&](int i, int j) {
        const auto o = __builtin_amdgcn_permlane16_swap(__float_as_uint(v[i]), __float_as_uint(v[j]), false, false);
        v[i] = __uint_as_float(o[0]);
        v[j] = __uint_as_float(o[1]);
    };
    auto swap32 = [&](int i, int j) {
        const auto o = __builtin_amdgcn_permlane32_swap(__float_as_uint(v[i]), __float_as_uint(v[j]), false, false);
        v[i] = __uint_as_float(o[0]);
        v[j] = __uint_as_float(o[1]);
    };
    swap16(0, 1);
    swap16(2, 3);
    swap32(0, 2);
    swap32(1, 3);
}

// v[4 q + g] for the lane's group g.
__device__ __forceinline__ float pick4(const float* v, int g) {
    const float lo = (g & 1) ? v[1] : v[0], hi = (g & 1) ? v[3] : v[2];
    return (g & 2) ? hi : lo;
}

// The filtered code of a tile (channels 4g..4g+3 of sample s) and its direction inputs: dirs[j] =
// direction input 4j + g, zero past the last; with frames also the frame layer's raw outputs v of
// the lane group's frame.  ff: the FP32 blocks FF and FFB; xch: the wave's exchange space.
template <int C, int H, int NH, int NF>
struct TmInput {
    using L = TrainLayout<C, H, NH, NF>;
    static constexpr int ND = NF > 0 ? (6 * NF + 3) / 4 : 2;
    f32x4 z;
    float dirs[ND];
    float v[NF > 0 ? 6 : 1];

    __device__ __forceinline__ void run(const float* ff, const TmFetch& f, bool live, float* xch, int lane) {
        const int g = lane >> 4, s = lane & 15;
        z = f32x4{0, 0, 0, 0};
        if (C == 16 || g < 2) {
            #pragma unroll
            for (int k = 0; k < 8; ++k)
                #pragma unroll
                for (int c = 0; c < 4; ++c) z[c] = fmaf(f.w[k], f.v[k][c], z[c]);
        }
        #pragma unroll
        for (int c = 0; c < 4; ++c) z[c] = live ? z[c] : 0.0f;
        if constexpr (NF > 0) {
            // the frame layer: bias, then the channels in ascending order, as frame_inputs sums them
            float zt[4] = {z[0], z[1], z[2], z[3]};
            transpose_groups(zt);
            f32x4 o = ld4(ff + (L::FFB - L::FF) + 4 * g);
            #pragma unroll
            for (int q = 0; q < C / 4; ++q) o = mfma_f32(ff[q * 64 + lane], zt[q], o);
            if (g < 3) st4(xch + s * 12 + 4 * g, o);
            lds_sync_wave();
            // lane groups share the frames: group g takes frame g % NF
            const int fr = NF > 1 ? g & 1 : 0;
            #pragma unroll
            for (int j = 0; j < 6; ++j) v[j] = xch[s * 12 + 6 * fr + j];
            lds_sync_wave();
            float x[6];
            frame_apply<1>(0, v, f.dir, f.dir + 3, x);
            if (g < NF) {
                #pragma unroll
                for (int j = 0; j < 3; ++j) {
                    xch[s * 12 + 3 * fr + j] = x[j];
                    xch[s * 12 + 3 * NF + 3 * fr + j] = x[3 + j];
                }
            }
            lds_sync_wave();
            #pragma unroll
            for (int j = 0; j < ND; ++j) {
                const float y = xch[s * 12 + 4 * j + g];
                dirs[j] = 4 * j + g < 6 * NF ? y : 0.0f;
            }
            lds_sync_wave();
        } else {
            dirs[0] = f.dir[0];
            dirs[1] = f.dir[1];
        }
        #pragma unroll
        for (int j = 0; j < ND; ++j) dirs[j] = live ? dirs[j] : 0.0f;
    }
};

// The layers in FP32 from the FP32 blocks (LDS or memory) to the output accumulator; hidden(k, act)
// receives the activations of layer k.
template <int C, int H, int NH, int NF, typename Hidden>
__device__ __forceinline__ f32x4 forward_f32(const float* blob, const TmInput<C, H, NH, NF>& in, bool live, int lane,
                                             Hidden&& hidden) {
    using L = TrainLayout<C, H, NH, NF>;
    constexpr int HT = L::HT, Q1 = L::Q1, G1 = L::G1;
    const int g = lane >> 4, s = lane & 15;
    float x0[Q1];
    if constexpr (L::NAT) {
        float zt[4] = {in.z[0], in.z[1], in.z[2], in.z[3]};
        transpose_groups(zt);
        #pragma unroll
        for (int q = 0; q < C / 4; ++q) x0[q] = zt[q];
        #pragma unroll
        for (int q = C / 4; q < Q1; ++q) x0[q] = in.dirs[q - C / 4];
    } else if constexpr (C == 16) {
        #pragma unroll
        for (int q = 0; q < 4; ++q) x0[q] = in.z[q];
        x0[4] = in.dirs[0];
        x0[5] = g == 2 && live ? 1.0f : in.dirs[1];
    } else {
        // lane group 2 takes direction inputs 0..3, group 3 inputs 4, 5 and the constant
        #pragma unroll
        for (int q = 0; q < 4; ++q) {
            const float lo = __shfl(in.dirs[0], 16 * q + s, 64), hi = __shfl(in.dirs[1], 16 * q + s, 64);
            x0[q] = g < 2 ? in.z[q] : (g == 2 ? lo : (q < 2 ? hi : (q == 2 && live ? 1.0f : 0.0f)));
        }
    }
    f32x4 act[HT], acc[HT];
    #pragma unroll
    for (int t = 0; t < HT; ++t) acc[t] = L::NAT ? ld4(blob + L::BIAS + t * 16 + 4 * g) : f32x4{0, 0, 0, 0};
    #pragma unroll
    for (int grp = 0; grp < G1; ++grp) {
        f32x4 A[HT];
        #pragma unroll
        for (int t = 0; t < HT; ++t) A[t] = ld4(blob + L::FW1 + ((t * G1 + grp) * 64 + lane) * 4);
        #pragma unroll
        for (int qq = 0; qq < 4; ++qq)
            #pragma unroll
            for (int t = 0; t < HT; ++t)
                if (4 * grp + qq < Q1) acc[t] = mfma_f32(A[t][qq], x0[4 * grp + qq], acc[t]);
    }
    #pragma unroll
    for (int t = 0; t < HT; ++t)
        #pragma unroll
        for (int r = 0; r < 4; ++r) act[t][r] = fmaxf(acc[t][r], 0.0f);
    hidden(1, act);
    #pragma unroll
    for (int k = 2; k <= NH; ++k) {
        #pragma unroll
        for (int t = 0; t < HT; ++t) acc[t] = ld4(blob + L::BIAS + ((k - 1) * HT + t) * 16 + 4 * g);
        #pragma unroll
        for (int t = 0; t < HT; ++t) {
            f32x4 A[HT];
            #pragma unroll
            for (int tp = 0; tp < HT; ++tp) A[tp] = ld4(blob + L::FWH + (k - 2) * L::WH_SZ + ((tp * HT + t) * 64 + lane) * 4);
            #pragma unroll
            for (int r = 0; r < 4; ++r)
                #pragma unroll
                for (int tp = 0; tp < HT; ++tp) acc[tp] = mfma_f32(A[tp][r], act[t][r], acc[tp]);
        }
        #pragma unroll
        for (int t = 0; t < HT; ++t)
            #pragma unroll
            for (int r = 0; r < 4; ++r) act[t][r] = fmaxf(acc[t][r], 0.0f);
        hidden(k, act);
    }
    f32x4 qo = ld4(blob + L::BIAS + NH * HT * 16 + 4 * g);
    #pragma unroll
    for (int t = 0; t < HT; ++t) {
        const f32x4 A = ld4(blob + L::FWO + (t * 64 + lane) * 4);
        #pragma unroll
        for (int r = 0; r < 4; ++r) qo = mfma_f32(A[r], act[t][r], qo);
    }
    return qo;
}

// ---- forward only: every wave of a workgroup walks its own tiles
template <int C, int H, int NH, int NF>
__global__ void __launch_bounds__(64 * kTMFwdWaves, 1) train_forward_kernel(const TrainArgs a) {
    using L = TrainLayout<C, H, NH, NF>;
    __shared__ __attribute__((aligned(16))) float smem[L::FWD + kTMFwdWaves * L::XCH];
    __shared__ LevelRow lrows[kMaxLevels];
    const int tid = threadIdx.x;
    const int wave = tid >> 6, lane = tid & 63, g = lane >> 4, s = lane & 15;
    for (int e = tid; e < L::FWD / 4; e += 64 * kTMFwdWaves) st4(smem + 4 * e, ld4(a.blob + 4 * e));
    if (tid < a.M) lrows[tid] = a.rows[tid];
    __syncthreads();
    float* xch = smem + L::FWD + wave * L::XCH;
    const int tiles = (a.n + 15) / 16;
    const int waves = gridDim.x * kTMFwdWaves;
    // consecutive tiles on different workgroups: a small batch spreads over the CUs
    const int wid = wave * gridDim.x + blockIdx.x;
    TmQuery q;
    TmFetch cur, nxt;
    if (wid < tiles) {
        tm_query(a, wid, s, q);
        tm_issue<C, NF, false>(a, lrows, wid, q, g, s, cur);
        tm_query(a, wid + waves, s, q);
    }
    for (int tile = wid; tile < tiles; tile += waves) {
        if (tile + waves < tiles) {
            tm_issue<C, NF, false>(a, lrows, tile + waves, q, g, s, nxt);
            tm_query(a, tile + 2 * waves, s, q);
        }
        const int i = tile * 16 + s;
        const bool in_range = i < a.n;
        asm volatile("" ::: "memory");          // the weights are read per tile, not kept in registers
        const bool live = in_range && cur.finite;
        TmInput<C, H, NH, NF> in;
        in.run(smem + L::FF, cur, live, xch, lane);
        const f32x4 qo = forward_f32(smem, in, live, lane, [](int, const f32x4*) {});
        if (in_range) {
            #pragma unroll
            for (int r = 0; r < 4; ++r) {
                const int row = 4 * g + r;
                if (row < a.NO) a.rgb[(int64_t)a.NO * i + row] = cur.finite ? tm_softplus<L::NAT>(qo[r]) : __builtin_nanf("");
            }
        }
        cur = nxt;
    }
}

// ---- forward and backward

// The lane, counted anew: in the back wave's loop, where the gradients fill the registers, nothing that
// follows from it is kept (or spilled, whose reloads would wait for the atomics under way).
__device__ __forceinline__ int fresh_lane() {
    int lane = __builtin_amdgcn_mbcnt_hi(~0u, __builtin_amdgcn_mbcnt_lo(~0u, 0));
    asm volatile("" : "+v"(lane));
    return lane;
}

// A tile's scatter: each pair has two, for even and odd tiles.  taps: offsets of taps 0..3, 4..7 (of channel 0), weights 0..3, 4..7.
struct alignas(16) TmScatter {
    int taps[16][4][4];
    float dz[16][20];
    int live[16];
};

// The slots of one pair: handoff n lies in slot n & 1.  `filled` counts the handoffs written by the
// front wave, `emptied` those the back wave has read; each is written by one wave only.  The front
// wave waits until handoff n - 2 is read, the back wave until handoff n is written.  Both waves of a
// pair walk the same tiles with the same number of handoffs each (`more` tells of a repeated one), so
// every wait ends.
typedef __attribute__((address_space(3))) volatile int lds_count;

struct TmRing {
    TmSlot* slots;
    TmSlotScale* scales;
    TmScatter* scatter;
    lds_count* filled;
    lds_count* emptied;
    int n;

    __device__ __forceinline__ TmSlot* slot() const { return slots + (n & 1); }
    __device__ __forceinline__ TmSlotScale* scale() const { return scales + (n & 1); }
    __device__ __forceinline__ static void wait(lds_count* count, int need) {
        while (__builtin_amdgcn_readfirstlane(*count) < need) __builtin_amdgcn_s_sleep(1);
        __builtin_amdgcn_wave_barrier();
    }
    // A count read ahead of its use (the read's latency passes meanwhile).
    __device__ __forceinline__ int peek_emptied() const { return *emptied; }
    __device__ __forceinline__ void begin_fill(int peeked) const {
        if (__builtin_amdgcn_readfirstlane(peeked) < n - 1) wait(emptied, n - 1);
        __builtin_amdgcn_wave_barrier();
    }
    __device__ __forceinline__ void end_fill() {
        __builtin_amdgcn_sched_barrier(0);
        lds_sync_wave();                        // the slot's writes are done
        *filled = ++n;
    }
    __device__ __forceinline__ void begin_read() const { wait(filled, n + 1); }
    __device__ __forceinline__ void end_read() {
        lds_sync_wave();                        // the reads are done
        *emptied = ++n;
    }
};

// Largest of a value over the four lane groups (the lanes of a sample).
__device__ __forceinline__ float sample_max(float m) {
    const auto a = __builtin_amdgcn_permlane16_swap(__float_as_uint(m), __float_as_uint(m), false, false);
    m = fmaxf(__uint_as_float(a[0]), __uint_as_float(a[1]));
    const auto b = __builtin_amdgcn_permlane32_swap(__float_as_uint(m), __float_as_uint(m), false, false);
    return fmaxf(__uint_as_float(b[0]), __uint_as_float(b[1]));
}

// Exponent e with 2^e times a sample's largest magnitude m in [2^14, 2^15), at most `most` (so that a power
// of two taken of it is a float).
__device__ __forceinline__ int half_exponent(float m, int most = 126) { return min(15 - __builtin_amdgcn_frexp_expf(m), most); }

__device__ __forceinline__ float pow2(int e) { return ldexpf(1.0f, e); }

// max(x, 0), 0 for NaN, in one instruction (a max takes two: one quiets NaNs).
__device__ __forceinline__ float relu(float x) { return __builtin_amdgcn_fmed3f(x, 0.0f, __builtin_inff()); }

// Sum exponents of a sample that adds nothing: above any other.
constexpr int kNoSample = 1 << 20;

// The halves of one layer's values of a tile, as B operands: word w of step s holds slots (s, g, 2w),
// (s, g, 2w + 1).
template <int KS>
struct TmHalves {
    half8 h[KS], l[KS];
};

__device__ __forceinline__ void put_pair(half8& v, int e, half2_t p) {
    v[e] = p[0];
    v[e + 1] = p[1];
}

// 0xffff for the halves above zero (they are zero or more, so no sum carries into the upper half).
__device__ __forceinline__ uint32_t half_mask(half2_t of) {
    return (((half2_bits(of) + 0x7fff7fffu) >> 15) & 0x00010001u) * 0xffffu;
}
__device__ __forceinline__ half2_t mask_half(half2_t v, uint32_t m) { return __builtin_bit_cast(half2_t, half2_bits(v) & m); }

// The operands of two row tiles (P parts of KS K steps each), read ahead of the products.
template <int KS, int P>
struct TmWeights {
    half8 a[2][KS][P];

    // row tiles 2q, 2q + 1 of W: this lane's part of its blocks at w
    __device__ __forceinline__ void load(const float* w, int q) {
        #pragma unroll
        for (int t = 0; t < 2; ++t)
            #pragma unroll
            for (int s = 0; s < KS; ++s)
                #pragma unroll
                for (int p = 0; p < P; ++p)
                    a[t][s][p] = *reinterpret_cast<const half8*>(w + (((2 * q + t) * KS + s) * P + p) * 256);
    }
    // row tiles 2q, 2q + 1 of W^T, out of W's blocks at w: their K step q holds those columns, and a
    // transposing read takes 16 rows of 16 columns (HT row tiles of W; w is moved by tr_lane).
    template <int HT>
    __device__ __forceinline__ void load_transposed(const float* w, int q) {
        typedef __fp16 fp16x4 __attribute__((ext_vector_type(4)));
        typedef __attribute__((address_space(3))) fp16x4 lds_fp16x4;
        #pragma unroll
        for (int t = 0; t < 2; ++t)
            #pragma unroll
            for (int s = 0; s < KS; ++s)
                #pragma unroll
                for (int p = 0; p < P; ++p) {
                    half4 part[2] = {};
                    #pragma unroll
                    for (int h = 0; h < 2; ++h)
                        if (2 * s + h < HT)
                            part[h] = __builtin_bit_cast(half4, __builtin_amdgcn_ds_read_tr16_b64_v4f16(
                                (lds_fp16x4*)(w + (((2 * s + h) * KS + q) * P + p) * 256 + 2 * t)));
                    a[t][s][p] = __builtin_shufflevector(part[0], part[1], 0, 1, 2, 3, 4, 5, 6, 7);
                }
    }
    // acc[t] += W x, small products first, the tiles in turn (each chain's latency covers the other's)
    template <int RT>
    __device__ __forceinline__ void multiply(const TmHalves<KS>& x, floatx4* acc) const {
        const auto add = [&](int s, int p, const half8& v) {
            #pragma unroll
            for (int t = 0; t < RT; ++t) acc[t] = mfma_f16(a[t][s][p], v, acc[t]);
        };
        #pragma unroll
        for (int s = 0; s < KS; ++s) {
            if constexpr (P == 3) {
                add(s, 2, x.h[s]);
                add(s, 1, x.l[s]);
            }
            add(s, 1, x.h[s]);
            add(s, 0, x.l[s]);
        }
        #pragma unroll
        for (int s = 0; s < KS; ++s) add(s, 0, x.h[s]);
    }
};

// Float offset of a lane's addresses in a transposing read: columns 4 (lane % 4) .. + 3 of row lane / 4.
__device__ __forceinline__ int tr_lane(int lane) { return ((lane & 3) * 16 + (lane >> 2)) * 4; }

// acc[t] += W_t x for the HT row tiles of a layer (W^T: TR); the first two tiles' operands are read at
// the start, those of the others ahead of the first ones' products (AHEAD) or after them.
template <int HT, int KS, int P, bool TR, bool AHEAD>
struct TmLayer {
    static_assert(HT == 1 || HT == 2 || HT == 4, "pairs of row tiles");
    const float* w;
    TmWeights<KS, P> first;

    __device__ __forceinline__ static void load(TmWeights<KS, P>& to, const float* w, int q) {
        if constexpr (TR) {
            to.template load_transposed<HT>(w, q);
        } else if constexpr (HT == 1) {
            #pragma unroll
            for (int s = 0; s < KS; ++s)
                #pragma unroll
                for (int p = 0; p < P; ++p) to.a[0][s][p] = *reinterpret_cast<const half8*>(w + (s * P + p) * 256);
        } else {
            to.load(w, q);
        }
    }
    __device__ __forceinline__ TmLayer() {}
    __device__ __forceinline__ TmLayer(const float* blocks, int lane) { start(blocks, lane); }
    __device__ __forceinline__ void start(const float* blocks, int lane) {
        w = blocks + (TR ? tr_lane(lane) : lane * 4);
        load(first, w, 0);
        __builtin_amdgcn_sched_barrier(0);
    }
    __device__ __forceinline__ void multiply(const TmHalves<KS>& x, floatx4* acc) const {
        if constexpr (HT == 4) {
            TmWeights<KS, P> second;
            if (AHEAD) {
                load(second, w, 1);
                __builtin_amdgcn_sched_barrier(0);
            }
            first.template multiply<2>(x, acc);
            if (!AHEAD) {
                __builtin_amdgcn_sched_barrier(0);
                load(second, w, 1);
            }
            second.template multiply<2>(x, acc + 2);
        } else {
            first.template multiply<HT>(x, acc);
        }
    }
};

// One row tile.
template <int KS, int P>
__device__ __forceinline__ void tm_products_one(const float* w, const TmHalves<KS>& x, floatx4& acc) {
    #pragma unroll
    for (int s = 0; s < KS; ++s) {
        const half8 ah = *reinterpret_cast<const half8*>(w + s * P * 256);
        const half8 al = *reinterpret_cast<const half8*>(w + s * P * 256 + 256);
        if constexpr (P == 3) {
            acc = mfma_f16(*reinterpret_cast<const half8*>(w + s * P * 256 + 512), x.h[s], acc);
            acc = mfma_f16(al, x.l[s], acc);
        }
        acc = mfma_f16(al, x.h[s], acc);
        acc = mfma_f16(ah, x.l[s], acc);
    }
    #pragma unroll
    for (int s = 0; s < KS; ++s) acc = mfma_f16(*reinterpret_cast<const half8*>(w + s * P * 256), x.h[s], acc);
}

// Magnitude and smallest magnitude of a lane's accumulators.
template <int HT>
__device__ __forceinline__ void tm_range(const floatx4* acc, float& most, float& least) {
    most = 0.0f;
    least = __builtin_inff();
    #pragma unroll
    for (int t = 0; t < HT; ++t)
        #pragma unroll
        for (int r = 0; r < 4; ++r) {
            most = fmaxf(most, fabsf(acc[t][r]));
            least = fminf(least, fabsf(acc[t][r]));
        }
}

// The exponent x that a layer's sums have in the back wave (times 2^x), and the least it has had: sums
// that were taken there, of up to 2^50, are still floats 2^(kFarStep kFarSteps) above.
struct TmScale {
    int x = kNoSample, least = kNoSample;

    __device__ __forceinline__ int room() const { return (least - x) / kFarStep + kFarSteps; }   // steps above x
    // Step of a sample of exponent e: its factor 2^(x + step kFarStep - e) is at most 1 and at least
    // 2^-kFarStep, where the room suffices.
    __device__ __forceinline__ int step(int e) const { return min(max(e - x - 1, 0) / kFarStep, room()); }
    // Fits x to exponents from lo to hi: unchanged if step 0 does for all of them.
    __device__ __forceinline__ void fit(int lo, int hi) {
        if (lo < x || hi > x + kFarStep) x = min(lo, least + kFarStep * kFarSteps);
        least = min(least, x);
    }
};

// Hands one layer over: deltas (NT row tiles, halves, scale exponent ed per sample), inputs (NA column
// tiles, halves, scale exponent ea).  xw, xb: scales of the sums of this layer's weight and bias
// gradients.  They follow the tile; one whose samples span more than kFarStep goes in several handoffs,
// with the factors of all but a step's samples zero.  The caller ends the last fill, with other work
// between the writes and that wait.
template <int NT, int NA>
__device__ __forceinline__ void tm_handoff(TmRing& ring, const half2_t (*dh)[2], const half2_t (*dl)[2], int ed,
                                           const half2_t (*ah)[2], const half2_t (*al)[2], int ea, TmScale& xw, TmScale& xb,
                                           float sign, int lane) {
    const int g = lane >> 4, s = lane & 15;
    int emptied = ring.peek_emptied();
    const bool sample = ed < kNoSample / 2;
    const int e = ed + ea;
    int last = 0;
    const bool fits = !sample || max((unsigned)(e - xw.x), (unsigned)(ed - xb.x)) <= (unsigned)kFarStep;
    if (__builtin_expect(__builtin_amdgcn_ballot_w64(!fits) != 0, 0)) {
        const auto over_samples = [&](int m, auto pick) {                 // uniform, rare
            #pragma unroll
            for (int o = 8; o > 0; o >>= 1) m = pick(m, __shfl_xor(m, o, 64));
            return __builtin_amdgcn_readfirstlane(m);
        };
        const auto fit = [&](TmScale& to, int of) {
            const int lo = over_samples(sample ? of : kNoSample, [](int a, int b) { return a < b ? a : b; });
            const int hi = over_samples(sample ? of : -kNoSample, [](int a, int b) { return a < b ? b : a; });
            to.fit(lo, hi);
            return to.step(hi);
        };
        last = fit(xw, e);
        last = max(last, fit(xb, ed));
    }
    for (int k = 0;; ++k) {
        // at most 1; 0 for no sample
        float fw = sample ? pow2(xw.x - e) : 0.0f, fb = sample ? pow2(xb.x - ed) : 0.0f;
        int x = xw.x, b = xb.x;
        if (__builtin_expect(last > 0, 0)) {                              // uniform, rarer
            TmScale w = xw, v = xb;
            asm volatile("" : "+s"(w.x), "+s"(v.x));                      // nothing of this ahead of the branch
            x = w.x + min(k, w.room()) * kFarStep;
            b = v.x + min(k, v.room()) * kFarStep;
            fw = sample && w.step(e) == k ? pow2(x - e) : 0.0f;
            fb = sample && v.step(ed) == k ? pow2(b - ed) : 0.0f;
        }
        const _Float16 f = (_Float16)(sign * fw);
        const half2_t f2 = {f, f};
        ring.begin_fill(emptied);
        TmSlot* m = ring.slot();
        TmSlotScale* sc = ring.scale();
        if (g == 0) sc->bias_weight[s] = (_Float16)(sign * fb);
        if (lane == 0) {
            sc->x = x;
            sc->xb = b;
            sc->more = last - k;
        }
        const auto store = [](uint8_t* p, half2_t a, half2_t b) { *reinterpret_cast<uint2*>(p) = make_uint2(half2_bits(a), half2_bits(b)); };
        #pragma unroll
        for (int t = 0; t < (NT > NA ? NT : NA); ++t) {
            const int at = slot_group(s, 4 * t + g);
            if (t < NT) {
                store(m->delta + at, dh[t][0], dh[t][1]);
                store(m->delta + kPlane + at, dl[t][0], dl[t][1]);
            }
            if (t < NA) {
                store(m->input + at, ah[t][0] * f2, ah[t][1] * f2);
                store(m->input + kPlane + at, al[t][0] * f2, al[t][1] * f2);
            }
        }
        if (__builtin_expect(k == last, 1)) break;
        ring.end_fill();
        emptied = ring.peek_emptied();
    }
}

// The packed pairs of a layer's halves by row tile (t: slots 16t + 4g .. + 3).
template <int HT, int KS>
__device__ __forceinline__ void tm_tiles(const half8 (&v)[KS], half2_t (*out)[2]) {
    #pragma unroll
    for (int t = 0; t < HT; ++t)
        #pragma unroll
        for (int j = 0; j < 2; ++j) out[t][j] = half2_t{v[t / 2][4 * (t % 2) + 2 * j], v[t / 2][4 * (t % 2) + 2 * j + 1]};
}

template <int C, int H, int NH, int NF>
__device__ __forceinline__ void train_front(const TrainArgs& a, const float* lds, const LevelRow* lrows, float* xch,
                                            TmRing ring, int wid, int waves, int tiles, int lane) {
    using L = TrainLayout<C, H, NH, NF>;
    using In = TmInput<C, H, NH, NF>;
    constexpr int HT = L::HT, KS = L::KS, P = L::P;
    constexpr bool AHEAD = NF == 0;               // with frames the registers do not suffice
    const auto block = [&](int at) { return lds + (at - L::BIAS); };
    const int g = lane >> 4, s = lane & 15;
    const int NO = a.NO;
    const bool fetching = C == 16 || g < 2;
    const float one = a.one;
    float loss_acc = 0.0f, absmax = 0.0f;
    int odd_tile = 0;
    int aw[NH + 2];
    #pragma unroll
    for (int k = 1; k <= NH + 1; ++k) aw[k] = __builtin_amdgcn_readfirstlane(reinterpret_cast<const int*>(block(L::AW))[k]);
    bool no_exponent = false;
    #pragma unroll
    for (int k = 1; k <= NH + 1; ++k) {
        no_exponent = no_exponent || aw[k] == kNoExponent;
        aw[k] = aw[k] == kNoExponent ? 0 : aw[k];
    }
    // The matrix cores round the sums inside a product down, by a part of the last bit: a bias that a sum
    // over many samples would keep.  Odd samples' deltas therefore run through the backward pass with
    // the other sign, and odd waves sum their gradients with the other sign (TmGradient::weight).
    const float sign = (s & 1) ? -1.0f : 1.0f, back_sign = (wid & 1) ? -sign : sign;
    // scales of the gradients of layers 1..NH, the output layer and the frame layer
    TmScale x[NH + 3], xb[NH + 3];
    TmQuery q;
    TmFetch cur, nxt;
    if (wid < tiles) {
        tm_query(a, wid, s, q);
        tm_issue<C, NF, true>(a, lrows, wid, q, g, s, cur);
        tm_query(a, wid + waves, s, q);
    }
    for (int tile = wid; tile < tiles; tile += waves) {
        asm volatile("" ::: "memory");          // the weights are read per tile, not kept in registers
        const int i = tile * 16 + s;
        const bool in_range = i < a.n;
        bool finite = cur.finite;
        if (a.z_in) {
            int ok = !fetching || (__builtin_isfinite(cur.v[0][0]) && __builtin_isfinite(cur.v[0][1]) &&
                                   __builtin_isfinite(cur.v[0][2]) && __builtin_isfinite(cur.v[0][3]));
            ok &= __shfl_xor(ok, 16, 64);
            ok &= __shfl_xor(ok, 32, 64);
            finite = ok != 0;
        }
        const bool live = in_range && finite;
        In in;
        in.run(block(L::FF), cur, live, xch, lane);

        // ---- layer 1's input in halves: channels, directions, the constant 1 (slot 7 of group 0)
        TmHalves<1> x0;
        int e0;
        {
            float v[8] = {in.z[0], in.z[1], in.z[2], in.z[3], 0.0f, 0.0f, 0.0f, g == 0 ? 1.0f : 0.0f};
            #pragma unroll
            for (int j = 0; j < In::ND; ++j) v[4 + j] = in.dirs[j];
            float m = 1.0f;
            #pragma unroll
            for (int j = 0; j < 7; ++j) m = fmaxf(m, fabsf(v[j]));
            e0 = half_exponent(sample_max(m));
            const float c = pow2(e0);
            #pragma unroll
            for (int j = 0; j < 8; j += 2) {
                half2_t h, l;
                split_pair(v[j] * c, v[j + 1] * c, one, h, l);
                put_pair(x0.h[0], j, h);
                put_pair(x0.l[0], j, l);
            }
        }
        // ---- forward in halves
        TmHalves<KS> act[NH];
        int ea[NH];                              // 2^ea times an activation is in the halves
        bool near = no_exponent;                 // a unit near its kink
        f32x4 qo;
        {
            floatx4 acc[HT];
            const TmLayer<HT, 1, 3, false, AHEAD> layer1(block(L::A1), lane);
            TmLayer<HT, KS, P, false, AHEAD> layer;
            #pragma unroll
            for (int k = 1; k <= NH; ++k) {
                if (!AHEAD && k > 1) layer.start(block(L::AH) + (k - 2) * L::AH_SZ, lane);
                const int ei = k == 1 ? e0 : ea[k > 1 ? k - 2 : 0], t0 = aw[k] + ei;   // accumulator exponent
                const float bs = pow2(ei);
                #pragma unroll
                for (int t = 0; t < HT; ++t) acc[t] = ld4(block(L::BA) + ((k - 1) * HT + t) * 16 + 4 * g) * bs;
                if (k == 1) layer1.multiply(x0, acc);
                else layer.multiply(act[k > 1 ? k - 2 : 0], acc);
                // the next layer's first operands, ahead of the conversions that it waits for
                if (AHEAD && k < NH) layer.start(block(L::AH) + (k - 1) * L::AH_SZ, lane);
                float most, least;
                tm_range<HT>(acc, most, least);
                const float m = sample_max(most);
                near = near || least < m * 0x1p-19f;
                const int ec = half_exponent(m, 126 - t0);
                ea[k - 1] = ec + t0;
                const float c = pow2(ec);
                #pragma unroll
                for (int t = 0; t < 2 * KS; ++t)
                    #pragma unroll
                    for (int j = 0; j < 4; j += 2) {
                        half2_t h = {}, l = {};
                        if (t < HT) split_pair(relu(acc[t < HT ? t : 0][j]) * c, relu(acc[t < HT ? t : 0][j + 1]) * c, one, h, l);
                        put_pair(act[k - 1].h[t / 2], 4 * (t % 2) + j, h);
                        put_pair(act[k - 1].l[t / 2], 4 * (t % 2) + j, l);
                    }
            }
            const int t0 = aw[NH + 1] + ea[NH - 1];
            floatx4 o = ld4(block(L::BA) + NH * HT * 16 + 4 * g) * pow2(ea[NH - 1]);
            // rows 0..7 of the output blocks: 8 x 16 bytes per lane group
            const float* w = block(L::AO) + (g * 8 + (s & 7)) * 4;
            const auto rows = [&](int at) {
                const half8 v = *reinterpret_cast<const half8*>(w + at);
                return s < 8 ? v : half8{};
            };
            #pragma unroll
            for (int st = 0; st < KS; ++st) {
                const half8 wh = rows(st * P * 128), wl = rows(st * P * 128 + 128);
                if constexpr (P == 3) {
                    o = mfma_f16(rows(st * P * 128 + 256), act[NH - 1].h[st], o);
                    o = mfma_f16(wl, act[NH - 1].l[st], o);
                }
                o = mfma_f16(wl, act[NH - 1].h[st], o);
                o = mfma_f16(wh, act[NH - 1].l[st], o);
            }
            #pragma unroll
            for (int st = 0; st < KS; ++st) o = mfma_f16(rows(st * P * 128), act[NH - 1].h[st], o);
            #pragma unroll
            for (int r = 0; r < 4; ++r) qo[r] = ldexpf(o[r], -t0);
        }
        // ---- the forward again in FP32 where a unit is near its kink or a value is out of range
        {
            bool odd = near && live;
            #pragma unroll
            for (int r = 0; r < 4; ++r) odd = odd || (4 * g + r < NO && !__builtin_isfinite(qo[r]));
            if (__builtin_amdgcn_ballot_w64(odd)) {
                int ln = lane;                   // opaque: no addresses of the rare path are kept over the tiles
                asm volatile("" : "+v"(ln));
                qo = forward_f32(a.blob, in, live, ln, [&](int k, const f32x4* v) {
                    float most, least;
                    tm_range<HT>(v, most, least);
                    const int e = half_exponent(sample_max(most));
                    const float c = pow2(e);
                    #pragma unroll
                    for (int kk = 0; kk < NH; ++kk) {
                        if (kk != k - 1) continue;
                        ea[kk] = e;
                        #pragma unroll
                        for (int t = 0; t < HT; ++t)
                            #pragma unroll
                            for (int j = 0; j < 4; j += 2) {
                                half2_t h, l;
                                split_pair(v[t][j] * c, v[t][j + 1] * c, one, h, l);
                                // an activation that the halves lose stays above zero for the ReLU's mask
                                #pragma unroll
                                for (int d = 0; d < 2; ++d)
                                    if (v[t][j + d] > 0.0f && h[d] == (_Float16)0.0f) h[d] = (_Float16)5.9604644775390625e-8f;
                                put_pair(act[kk].h[t / 2], 4 * (t % 2) + j, h);
                                put_pair(act[kk].l[t / 2], 4 * (t % 2) + j, l);
                            }
                    }
                });
            }
        }

        // ---- output deltas: dL/dq = dL/dy * logistic(q)
        // (lane group g takes outputs g and 4 + g, so that one or two evaluations serve all)
        float dq[4] = {qo[0], qo[1], qo[2], qo[3]};
        transpose_groups(dq);
        #pragma unroll
        for (int j = 0; j < 2; ++j) {
            float v = 0.0f;
            if (j == 0 || NO > 4) {
                const bool mine = 4 * j + g < NO && live;
                float gy = cur.t[j];
                if (a.target) {
                    const float e = mine ? tm_softplus<L::NAT>(dq[j]) - cur.t[j] : 0.0f;
                    loss_acc = fmaf(e, e, loss_acc);
                    gy = 2.0f * e * a.inv_count;
                }
                v = mine ? gy * tm_logistic<L::NAT>(dq[j]) : 0.0f;
            }
            dq[j] = v;
        }
        dq[2] = dq[3] = 0.0f;
        const float dq_most = fmaxf(fabsf(dq[0]), fabsf(dq[1]));
        transpose_groups(dq);
        half2_t th[4][2], tl[4][2], uh[4][2], ul[4][2];          // handoff operands by tile
        half2_t dr[2];                                            // what the output deltas' halves leave
        TmHalves<KS> d;                                           // the layer's deltas as B operands
        int ed, eds;                                              // their exponent; kNoSample where they are zero
        {
            const float m = sample_max(dq_most);
            ed = half_exponent(m);
            eds = m > 0.0f ? ed : kNoSample;
            #pragma unroll
            for (int j = 0; j < 2; ++j)
                split_pair(ldexpf(sign * dq[2 * j], ed), ldexpf(sign * dq[2 * j + 1], ed), one, th[0][j], tl[0][j], &dr[j]);
            tm_tiles<HT, KS>(act[NH - 1].h, uh);
            tm_tiles<HT, KS>(act[NH - 1].l, ul);
        }
        // delta_k = W_{k+1}^T delta_{k+1}, masked by a_k > 0, from the accumulators in exponent t0
        const auto take_deltas = [&](const floatx4* acc, int t0, const TmHalves<KS>& ak) {
            float most, least;
            tm_range<HT>(acc, most, least);
            const float m = sample_max(most);
            const int ec = half_exponent(m);
            ed = ec + t0;
            eds = m > 0.0f ? ed : kNoSample;
            const float c = pow2(ec);
            #pragma unroll
            for (int t = 0; t < 2 * KS; ++t)
                #pragma unroll
                for (int j = 0; j < 4; j += 2) {
                    half2_t h = {}, l = {};
                    if (t < HT) {
                        split_pair(acc[t < HT ? t : 0][j] * c, acc[t < HT ? t : 0][j + 1] * c, one, h, l);
                        const uint32_t on = half_mask(half2_t{ak.h[t / 2][4 * (t % 2) + j], ak.h[t / 2][4 * (t % 2) + j + 1]});
                        h = mask_half(h, on);
                        l = mask_half(l, on);
                    }
                    put_pair(d.h[t / 2], 4 * (t % 2) + j, h);
                    put_pair(d.l[t / 2], 4 * (t % 2) + j, l);
                }
        };
        {
            half4 wo[HT][P];                     // W_out^T: outputs 4g..4g+3 for lane groups 0 and 1
            #pragma unroll
            for (int t = 0; t < HT; ++t) {
                #pragma unroll
                for (int p = 0; p < P; ++p) {
                    wo[t][p] = *reinterpret_cast<const half4*>(block(L::BO) + (t * P + p) * 64 + (lane & 31) * 2);
                    wo[t][p] = g < 2 ? wo[t][p] : half4{};
                }
            }
            tm_handoff<1, HT>(ring, th, tl, eds, uh, ul, ea[NH - 1], x[NH + 1], xb[NH + 1], back_sign, lane);
            const half4 dh = {th[0][0][0], th[0][0][1], th[0][1][0], th[0][1][1]};
            const half4 dl = {tl[0][0][0], tl[0][0][1], tl[0][1][0], tl[0][1][1]};
            floatx4 acc[HT];
            #pragma unroll
            for (int t = 0; t < HT; ++t) acc[t] = floatx4{0, 0, 0, 0};
            const auto add = [&](int p, const half4& v) {
                #pragma unroll
                for (int t = 0; t < HT; ++t) acc[t] = __builtin_amdgcn_mfma_f32_16x16x16f16(wo[t][p], v, acc[t], 0, 0, 0);
            };
            // few terms, so that an FP32 chain would have few roundings: all that the halves leave counts
            add(0, half4{dr[0][0], dr[0][1], dr[1][0], dr[1][1]});
            if (P == 3) add(P - 1, dh);
            add(1, dl);
            add(1, dh);
            add(0, dl);
            add(0, dh);
            ring.end_fill();
            take_deltas(acc, aw[NH + 1] + ed, act[NH - 1]);
        }
        // hidden layers k = NH .. 2: hand (delta_k, a_{k-1}) over, then delta_{k-1}
        #pragma unroll
        for (int k = NH; k >= 2; --k) {
            tm_tiles<HT, KS>(d.h, th);
            tm_tiles<HT, KS>(d.l, tl);
            tm_tiles<HT, KS>(act[k - 2].h, uh);
            tm_tiles<HT, KS>(act[k - 2].l, ul);
            const TmLayer<HT, KS, P, true, AHEAD> layer(block(L::AH) + (k - 2) * L::AH_SZ, lane);
            tm_handoff<HT, HT>(ring, th, tl, eds, uh, ul, ea[k - 2], x[k], xb[k], back_sign, lane);
            floatx4 acc[HT];
            #pragma unroll
            for (int t = 0; t < HT; ++t) acc[t] = floatx4{0, 0, 0, 0};
            layer.multiply(d, acc);
            ring.end_fill();
            take_deltas(acc, aw[k] + ed, act[k - 2]);
        }
        // the next tile's texels, now that the activations' registers are free
        if (tile + waves < tiles) {
            tm_issue<C, NF, true>(a, lrows, tile + waves, q, g, s, nxt);
            tm_query(a, tile + 2 * waves, s, q);
        }
        // (delta_1, the input with its constant-1 column)
        tm_tiles<HT, KS>(d.h, th);
        tm_tiles<HT, KS>(d.l, tl);
        tm_tiles<2, 1>(x0.h, uh);
        tm_tiles<2, 1>(x0.l, ul);
        tm_handoff<HT, 2>(ring, th, tl, eds, uh, ul, e0, x[1], xb[1], back_sign, lane);
        // the gradient of the latent code (with frames of the whole input: row tile u, inputs 16u ..)
        f32x4 dx[L::NR1];
        #pragma unroll
        for (int u = 0; u < L::NR1; ++u) {
            floatx4 acc = {0, 0, 0, 0};
            tm_products_one<KS, P>(block(L::B1) + u * KS * P * 256 + lane * 4, d, acc);
            if (u == 0) ring.end_fill();
            #pragma unroll
            for (int r = 0; r < 4; ++r) dx[u][r] = sign * ldexpf(acc[r], -(aw[1] + ed));
        }
        f32x4 dz = dx[0];
        if constexpr (NF > 0) {
            // through the frame transform into the frame layer and the latent code, a frame per lane
            // group; the layer's back product is one more MFMA chain
            #pragma unroll
            for (int u = C / 16; u < L::NR1; ++u) {
                const int col = 16 * u + 4 * g - C;
                if (col >= 0 && col < 12) st4(xch + s * 12 + col, dx[u]);
            }
            lds_sync_wave();
            const int fr = NF > 1 ? g & 1 : 0;
            float G[6], draw[6];
            #pragma unroll
            for (int j = 0; j < 3; ++j) {
                G[j] = xch[s * 12 + 3 * fr + j];
                G[3 + j] = xch[s * 12 + 3 * NF + 3 * fr + j];
            }
            lds_sync_wave();
            frame_backward_raw<1>(0, in.v, cur.dir, cur.dir + 3, G, draw);
            float m = 0.0f;
            #pragma unroll
            for (int j = 0; j < 6; ++j) {
                draw[j] = live ? draw[j] : 0.0f;
                m = fmaxf(m, fabsf(draw[j]));
                if (g < NF) xch[s * 12 + 6 * fr + j] = draw[j];
            }
            m = sample_max(m);
            lds_sync_wave();
            #pragma unroll
            for (int j = 0; j < (6 * NF + 3) / 4; ++j) {
                const float y = xch[s * 12 + 4 * j + g];
                dz = mfma_f32(block(L::BF)[j * 64 + lane], 4 * j + g < 6 * NF ? y : 0.0f, dz);
            }
            const int e = half_exponent(m);
            float w[4];                           // outputs 4g .. 4g + 3
            #pragma unroll
            for (int r = 0; r < 4; ++r) {
                const float y = xch[s * 12 + (4 * g + r < 12 ? 4 * g + r : 0)];
                w[r] = 4 * g + r < 6 * NF ? y : 0.0f;
            }
            lds_sync_wave();
            #pragma unroll
            for (int j = 0; j < 2; ++j) split_pair(ldexpf(sign * w[2 * j], e), ldexpf(sign * w[2 * j + 1], e), one, th[0][j], tl[0][j]);
            tm_tiles<1, 1>(x0.h, uh);
            tm_tiles<1, 1>(x0.l, ul);
            tm_handoff<1, 1>(ring, th, tl, m > 0.0f ? e : kNoSample, uh, ul, e0, x[0], xb[0], back_sign, lane);
            ring.end_fill();
        }
        // lane (g, s) holds channels 4g..4g+3 of sample s (C = 8: lanes g < 2)
        if (a.dz) {
            if (in_range && fetching) {
                const f32x4 v = live ? dz : f32x4{0, 0, 0, 0};
                st4(a.dz + (int64_t)i * C + 4 * g, v);
                #pragma unroll
                for (int r = 0; r < 4; ++r) absmax = fmaxf(absmax, __builtin_isfinite(v[r]) ? fabsf(v[r]) : __builtin_inff());
            }
        } else {
            // the taps and the code's gradient, for the back wave to scatter (zero where not live)
            const int emptied = ring.peek_emptied();
            const f32x4 v = live ? dz : f32x4{0, 0, 0, 0};
            f32x4 tap;                            // group 0, 1: offsets 0.., 4.. (its own
                                                  // point at channel 4g), else weights
            #pragma unroll
            for (int r = 0; r < 4; ++r) {
                const float v0 = __int_as_float(cur.off[r]), v1 = __int_as_float(cur.off[4 + r] - 4);
                const float v2 = cur.w[r], v3 = cur.w[4 + r];
                const float o = (g & 1) ? v1 : v0, w = (g & 1) ? v3 : v2;
                tap[r] = g < 2 ? o : w;
            }
            ring.begin_fill(emptied);
            // the back wave has added the tile before last: it does so ahead of handoffs that are read
            TmScatter* m = ring.scatter + odd_tile;
            odd_tile ^= 1;
            st4(reinterpret_cast<float*>(m->taps[s][g]), tap);
            if (fetching) st4(&m->dz[s][4 * g], v);
            if (g == 0) m->live[s] = live;
            ring.end_fill();
        }
        cur = nxt;
    }
    #pragma unroll
    for (int o = 32; o > 0; o >>= 1) {
        loss_acc += __shfl_xor(loss_acc, o, 64);
        absmax = fmaxf(absmax, __shfl_xor(absmax, o, 64));
    }
    if (lane == 0) {
        a.loss_partial[wid] = loss_acc;
        if (a.dz && a.dz_absmax && absmax > 0.0f) atomicMax(a.dz_absmax, __float_as_uint(absmax));
    }
}

// Gradients of one layer in the back wave's registers: RT row tiles (outputs) x CT column tiles
// (inputs), times 2^x; the bias sums of row 16t + lane % 16 (partial: over the lane group's samples),
// times 2^xb.
template <int RT, int CT>
struct TmGradient {
    floatx4 w[RT][CT];
    float b[RT];
    int x, xb;

    __device__ __forceinline__ void clear() {
        #pragma unroll
        for (int t = 0; t < RT; ++t) {
            #pragma unroll
            for (int c = 0; c < CT; ++c) w[t][c] = floatx4{0, 0, 0, 0};
            b[t] = 0.0f;
        }
        x = xb = 0;
    }

    // Adds the layer's handoffs of a tile.
    __device__ __forceinline__ void add(TmRing& ring) {
        while (add_one(ring)) {}
    }
    __device__ __forceinline__ bool add_one(TmRing& ring) {
        typedef __fp16 fp16x4 __attribute__((ext_vector_type(4)));
        typedef __attribute__((address_space(3))) fp16x4 lds_fp16x4;
        const int lane = fresh_lane(), g = lane >> 4, j = lane & 15;
        ring.begin_read();
        const TmSlot* m = ring.slot();
        const TmSlotScale* sc = ring.scale();
        // lane j of a group points at 4 columns of sample 4g + j / 4 and receives column j of the four
        const int row = 4 * g + (j >> 2);
        const auto read = [&](const uint8_t* p, int c) {
            const auto v = __builtin_amdgcn_ds_read_tr16_b64_v4f16((lds_fp16x4*)(p + slot_group(row, 4 * c + (j & 3))));
            return __builtin_bit_cast(half4, v);
        };
        // the gradients fill most registers: the inputs of all column tiles, the deltas of two row tiles
        half4 ah[CT], al[CT], dh[2], dl[2];
        #pragma unroll
        for (int c = 0; c < CT; ++c) {
            ah[c] = read(m->input, c);
            al[c] = read(m->input + kPlane, c);
        }
        dh[0] = read(m->delta, 0);
        dl[0] = read(m->delta + kPlane, 0);
        const half4 bw = *reinterpret_cast<const half4*>(&sc->bias_weight[4 * g]);
        const int nx = __builtin_amdgcn_readfirstlane(sc->x), nb = __builtin_amdgcn_readfirstlane(sc->xb);
        const bool more = __builtin_amdgcn_readfirstlane(sc->more) != 0;
        if (nx != x || nb != xb) {               // uniform, rare: the exponents changed
            #pragma unroll
            for (int t = 0; t < RT; ++t) {
                #pragma unroll
                for (int c = 0; c < CT; ++c)
                    #pragma unroll
                    for (int r = 0; r < 4; ++r) w[t][c][r] = ldexpf(w[t][c][r], nx - x);
                b[t] = ldexpf(b[t], nb - xb);
            }
            x = nx;
            xb = nb;
        }
        #pragma unroll
        for (int t = 0; t < RT; ++t) {
            const half4 h = dh[t & 1], l = dl[t & 1];
            if (t + 1 < RT) {
                dh[(t + 1) & 1] = read(m->delta, t + 1);
                dl[(t + 1) & 1] = read(m->delta + kPlane, t + 1);
            }
            __builtin_amdgcn_sched_barrier(0);
            #pragma unroll
            for (int c = 0; c < CT; ++c) w[t][c] = __builtin_amdgcn_mfma_f32_16x16x16f16(l, ah[c], w[t][c], 0, 0, 0);
            #pragma unroll
            for (int c = 0; c < CT; ++c) w[t][c] = __builtin_amdgcn_mfma_f32_16x16x16f16(h, al[c], w[t][c], 0, 0, 0);
            #pragma unroll
            for (int c = 0; c < CT; ++c) w[t][c] = __builtin_amdgcn_mfma_f32_16x16x16f16(h, ah[c], w[t][c], 0, 0, 0);
            const half2_t b0 = {bw[0], bw[1]}, b1 = {bw[2], bw[3]};
            b[t] = __builtin_amdgcn_fdot2(half2_t{l[0], l[1]}, b0, b[t], false);
            b[t] = __builtin_amdgcn_fdot2(half2_t{l[2], l[3]}, b1, b[t], false);
            b[t] = __builtin_amdgcn_fdot2(half2_t{h[0], h[1]}, b0, b[t], false);
            b[t] = __builtin_amdgcn_fdot2(half2_t{h[2], h[3]}, b1, b[t], false);
        }
        ring.end_read();
        return more;
    }

    // sign: the wave's
    __device__ __forceinline__ float weight(int t, int c, int r, float sign) const { return sign * ldexpf(w[t][c][r], -x); }
    // the bias of row 16t + lane % 16, over the four lane groups
    __device__ __forceinline__ float bias(int t, float sign) const {
        float v = b[t];
        v += __shfl_xor(v, 16, 64);
        v += __shfl_xor(v, 32, 64);
        return sign * ldexpf(v, -xb);
    }
};

// Adds part of a tile's code gradients to the texels, C lanes per sample: in round r, lane (u, c) =
// (lane / C, lane % C) adds channel c of sample r (64 / C) + u, so one atomic instruction covers 64 / C
// whole texels and the memory side takes each texel as one request (with the lanes of the accumulator
// layout it took a quarter of a texel per request).  Unit i is half the taps of round i / 2.
template <int C>
__device__ __forceinline__ void tm_scatter(float* d_tex, const TmScatter* m, int unit) {
    const int lane = fresh_lane();
    const int s = (unit >> 1) * (64 / C) + lane / C, c = lane % C, half = unit & 1;
    const float dv = m->dz[s][c];
    if (m->live[s]) {
        #pragma unroll
        for (int k = 0; k < 4; ++k)
            unsafeAtomicAdd(d_tex + m->taps[s][half][k] + c, __int_as_float(m->taps[s][2 + half][k]) * dv);
    }
}

template <int C, int H, int NH, int NF>
__device__ __forceinline__ void train_back(const TrainArgs& a, TmRing ring, int wid, int waves, int tiles, int lane) {
    using L = TrainLayout<C, H, NH, NF>;
    constexpr int HT = L::HT, IN = L::IN, HH = NH > 1 ? NH - 1 : 1;
    const int g = lane >> 4, s = lane & 15;
    const int NO = a.NO;
    TmGradient<HT, 2> g1;
    TmGradient<HT, HT> gh[HH];
    TmGradient<1, HT> go;
    TmGradient<1, 1> gf;
    g1.clear();
    go.clear();
    gf.clear();
    #pragma unroll
    for (int k = 0; k < HH; ++k) gh[k].clear();
    // the scatter of the tile before goes between the sums of a tile, ahead of each handoff's read: the
    // atomics drain meanwhile
    constexpr int UNITS = 2 * 16 / (64 / C), EVENTS = NH + 1;
    const bool scatters = a.dz == nullptr;
    const TmScatter* last = nullptr;
    int odd_tile = 0;
    const auto scatter = [&](int event) {
        if (!last) return;
        #pragma unroll
        for (int i = event * UNITS / EVENTS; i < (event + 1) * UNITS / EVENTS; ++i) tm_scatter<C>(a.d_tex, last, i);
    };
    for (int tile = wid; tile < tiles; tile += waves) {
        scatter(0);
        go.add(ring);
        #pragma unroll
        for (int k = NH; k >= 2; --k) {
            scatter(NH + 1 - k);
            gh[k - 2].add(ring);
        }
        scatter(NH);
        g1.add(ring);
        if constexpr (NF > 0) gf.add(ring);
        if (scatters) {
            ring.begin_read();
            last = ring.scatter + odd_tile;
            odd_tile ^= 1;
            ring.end_read();
        }
    }
    #pragma unroll
    for (int e = 0; e < EVENTS; ++e) scatter(e);

    // ---- this wave's gradients into its own partial slice (every parameter written once)
    const float sign = (wid & 1) ? -1.0f : 1.0f;
    float* part = a.partial + (size_t)wid * a.np;
    const auto nat = [](int i) { return slot_neuron<L::NAT>(i); };
    if constexpr (NF > 0) {
        #pragma unroll
        for (int r = 0; r < 4; ++r)
            if (4 * g + r < 6 * NF && s < C) part[(4 * g + r) * C + s] = gf.weight(0, 0, r, sign);
        const float b = gf.bias(0, sign);
        if (g == 0 && s < 6 * NF) part[6 * NF * C + s] = b;
        part += L::NP1;
    }
    // layer 1: column 4g' + e of tile 0 is channel 4g' + e, of tile 1 direction input 4e + g'; its column 3
    // (e = 3, g' = 0) the constant 1
    #pragma unroll
    for (int co = 0; co < HT; ++co)
        #pragma unroll
        for (int r = 0; r < 4; ++r) {
            const int o = 16 * co + nat(4 * g + r);
            if (s < C) part[o * IN + s] = g1.weight(co, 0, r, sign);
            const int d = 4 * (s & 3) + (s >> 2);
            const float w = g1.weight(co, 1, r, sign);
            if (d < IN - C) part[o * IN + C + d] = w;
            else if (s == 3) part[IN * H + o] = w;
        }
    #pragma unroll
    for (int k = 2; k <= NH; ++k) {
        const int off = param_off<IN, H>(k);
        #pragma unroll
        for (int co = 0; co < HT; ++co) {
            #pragma unroll
            for (int cj = 0; cj < HT; ++cj)
                #pragma unroll
                for (int r = 0; r < 4; ++r)
                    part[off + (16 * co + nat(4 * g + r)) * H + 16 * cj + nat(s)] = gh[k - 2].weight(co, cj, r, sign);
            const float b = gh[k - 2].bias(co, sign);
            if (g == 0) part[off + H * H + 16 * co + nat(s)] = b;
        }
    }
    const int off = param_off<IN, H>(NH + 1);
    #pragma unroll
    for (int c = 0; c < HT; ++c)
        #pragma unroll
        for (int r = 0; r < 4; ++r)
            if (4 * g + r < NO) part[off + (4 * g + r) * H + 16 * c + nat(s)] = go.weight(0, c, r, sign);
    const float b = go.bias(0, sign);
    if (g == 0 && s < NO) part[off + NO * H + s] = b;
}

template <int C, int H, int NH, int NF>
struct alignas(16) TmSmem {
    using L = TrainLayout<C, H, NH, NF>;
    float blocks[L::LDS_FLOATS];
    TmSlot slots[kTMPairs][2];
    float xch[kTMPairs][L::XCH > 0 ? L::XCH : 4];
    TmSlotScale scales[kTMPairs][2];
    TmScatter scatter[kTMPairs][2];
    LevelRow rows[kMaxLevels];
    int counts[2][kTMPairs];
};

// What bounds it: the front wave's serial chain (at 16 channels and three layers of 64, 2^20 samples of
// given codes: 14,300 cycles per tile, of which the matrix cores are busy for 4,500; the LDS moves 50% of
// what it could), and with a texture the atomics, 412 us of lines by themselves.  More waves do not fit:
// the gradients of a back wave take 176 registers, the activations of a front wave 96, two waves per SIMD
// have 256 each.  Measured on 2^20 samples against FP32 matrix products in the same pairs: given codes
// 611 -> 382 us, with fetch and scatter 770 -> 476 us (scattered by the front wave 664 us); 250,007
// samples with two frames 250 -> 162 us.
template <int C, int H, int NH, int NF>
__global__ void __launch_bounds__(kTMThreads, 1) train_mfma_kernel(const TrainArgs a) {
    using L = TrainLayout<C, H, NH, NF>;
    static_assert(sizeof(TmSmem<C, H, NH, NF>) <= 160 * 1024, "the decoder's blocks and the slots exceed the LDS");
    __shared__ TmSmem<C, H, NH, NF> sm;
    const int tid = threadIdx.x;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6), lane = tid & 63;
    const int alt = (blockIdx.x & 1) * L::ALT;
    for (int e = tid; e < L::LDS_FLOATS / 4; e += kTMThreads)
        st4(sm.blocks + 4 * e, ld4(a.blob + L::BIAS + 4 * e + (4 * e >= L::BLOCKS - L::BIAS ? alt : 0)));
    if (tid < a.M) sm.rows[tid] = a.rows[tid];
    if (tid < 2 * kTMPairs) sm.counts[tid / kTMPairs][tid % kTMPairs] = 0;
    __syncthreads();
    const int pair = wave % kTMPairs;
    if (pair >= a.pairs) return;
    const int tiles = (a.n + 15) / 16;
    const int waves = gridDim.x * a.pairs;
    const int wid = blockIdx.x * a.pairs + pair;
    const TmRing ring{sm.slots[pair], sm.scales[pair], sm.scatter[pair], (lds_count*)&sm.counts[0][pair], (lds_count*)&sm.counts[1][pair], 0};
    if (wave < kTMPairs) {
        __builtin_amdgcn_s_setprio(1);          // the chain that the back wave waits for goes first
        train_front<C, H, NH, NF>(a, sm.blocks, sm.rows, sm.xch[pair], ring, wid, waves, tiles, lane);
    } else {
        train_back<C, H, NH, NF>(a, ring, wid, waves, tiles, lane);
    }
}

// pack: pack the decoder from params (and the frame layer) into blob; run: launch the kernel on it
template <int C, int H, int NH, int NF>
static hipError_t launch_tm_shape(bool pack, bool run, bool train, const float* params, const float* fparams, int NO,
                                  float* blob, const TrainArgs& a, int grid, hipStream_t st) {
    clear_stale_hip_error();
    if (pack) {
        pack_train_kernel<C, H, NH, NF><<<pack_train_grid<C, H, NH, NF>(), 256, 0, st>>>(params, fparams, NO, blob);
        const hipError_t e = hipGetLastError();
        if (e != hipSuccess || !run) return e;
    }
    if (train) train_mfma_kernel<C, H, NH, NF><<<grid, kTMThreads, 0, st>>>(a);
    else train_forward_kernel<C, H, NH, NF><<<grid, 64 * kTMFwdWaves, 0, st>>>(a);
    return hipGetLastError();
}

// Every shape of the kernels: X(C, H, NH, NF).  64-wide decoders of four hidden layers exceed the LDS.
#define NAM_TM_C(X, H_, NH_, NF_) X(8, H_, NH_, NF_) X(16, H_, NH_, NF_)
#define NAM_TM_SHAPES(X)                                                                              \
    NAM_TM_C(X, 16, 1, 0) NAM_TM_C(X, 16, 2, 0) NAM_TM_C(X, 16, 3, 0) NAM_TM_C(X, 16, 4, 0)           \
    NAM_TM_C(X, 32, 1, 0) NAM_TM_C(X, 32, 2, 0) NAM_TM_C(X, 32, 3, 0) NAM_TM_C(X, 32, 4, 0)           \
    NAM_TM_C(X, 64, 1, 0) NAM_TM_C(X, 64, 2, 0) NAM_TM_C(X, 64, 3, 0)                                 \
    NAM_TM_C(X, 32, 2, 1) NAM_TM_C(X, 32, 3, 1) NAM_TM_C(X, 64, 2, 1) NAM_TM_C(X, 64, 3, 1)           \
    NAM_TM_C(X, 32, 2, 2) NAM_TM_C(X, 32, 3, 2) NAM_TM_C(X, 64, 2, 2) NAM_TM_C(X, 64, 3, 2)

int train_mfma_blob_floats(const MlpShape& sh) {
#define NAM_TM_SZ(C_, H_, NH_, NF_) \
    if (sh.C == C_ && sh.H == H_ && sh.NH == NH_ && sh.NF == NF_) return TrainLayout<C_, H_, NH_, NF_>::BLOB;
    NAM_TM_SHAPES(NAM_TM_SZ)
#undef NAM_TM_SZ
    return 0;
}

bool train_mfma_supported(const MlpShape& sh) {
    return train_mfma_blob_floats(sh) > 0 && (sh.NO == 3 || (sh.NO == 6 && sh.NF == 0));
}

static hipError_t dispatch_tm(const MlpShape& sh, bool pack, bool run, bool train, const float* params,
                              const float* fparams, float* blob, const TrainArgs& a, int grid, hipStream_t st) {
#define NAM_TM_CASE(C_, H_, NH_, NF_)                                     \
    if (sh.C == C_ && sh.H == H_ && sh.NH == NH_ && sh.NF == NF_)         \
        return launch_tm_shape<C_, H_, NH_, NF_>(pack, run, train, params, fparams, sh.NO, blob, a, grid, st);
    NAM_TM_SHAPES(NAM_TM_CASE)
#undef NAM_TM_CASE
    return hipErrorInvalidValue;
}

void train_mfma_grid(int64_t n, int cu_count, bool train, int* grid, int* pairs) {
    const int64_t tiles = (n + 15) / 16;
    *grid = (int)(tiles < 1 ? 1 : tiles < cu_count ? tiles : cu_count);
    const int64_t per = (tiles + *grid - 1) / *grid;
    *pairs = train ? (int)(per < 1 ? 1 : per < kTMPairs ? per : kTMPairs) : 0;
}

hipError_t launch_train_mfma(const MlpShape& sh, bool train, const float* params, float* blob, const TrainArgs& a,
                             int grid, hipStream_t st) {
    return dispatch_tm(sh, true, true, train, params, a.fparams, blob, a, grid, st);
}

// ---- plain FP32 decodes on the FP32 matrix cores: the forward kernel on a blob packed once
// per material
static bool decode_f32_mfma_supported(const nam_material* m) {
    return train_mfma_supported(m->shape) && m->shape.NF == 0 && m->texel_count * m->desc.channels < (int64_t(1) << 31);
}

hipError_t prepare_decode_f32_mfma(nam_material* m) {
    if (!decode_f32_mfma_supported(m)) return hipSuccess;
    const size_t floats = (size_t)train_mfma_blob_floats(m->shape);
    float* blob = nullptr;
    hipError_t e = hipMalloc(&blob, floats * sizeof(float));
    if (e != hipSuccess) return e;
    e = dispatch_tm(m->shape, true, false, false, m->params32, nullptr, blob, TrainArgs{}, 0, nullptr);
    if (e == hipSuccess) e = hipDeviceSynchronize();
    if (e != hipSuccess) {
        (void)hipFree(blob);
        return e;
    }
    m->fblob = blob;
    m->fblob_bytes = floats * sizeof(float);
    return hipSuccess;
}

hipError_t launch_decode_f32_mfma(const nam_material* m, int64_t n, const float* uv, const float* lod, const float* wi,
                                  const float* wo, float* rgb, hipStream_t st) {
    if (n <= 0) return hipSuccess;
    if (!m->fblob || n > INT32_MAX) return hipErrorInvalidValue;
    TrainArgs a{};
    a.rows = m->rows;
    a.M = m->desc.levels;
    a.address = (int)m->desc.address;
    a.tex = m->texels32;
    a.params = m->params32;
    a.wt = m->fblob;
    a.blob = m->fblob;
    a.n = (int)n;
    a.uv = uv;
    a.lod = lod;
    a.wi = wi;
    a.wo = wo;
    a.rgb = rgb;
    a.NO = m->shape.NO;
    int grid, pairs;
    train_mfma_grid(n, m->ctx->cu_count, false, &grid, &pairs);
    return dispatch_tm(m->shape, false, true, false, nullptr, nullptr, m->fblob, a, grid, st);
}

}  // namespace nam
