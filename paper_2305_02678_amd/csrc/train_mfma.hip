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

// Builds the operand blocks of TrainLayout from packed parameters, one thread per float.  p: the
// decoder; fp: the frame layer (NF > 0).
template <int C, int H, int NH, int NF>
__global__ void __launch_bounds__(256) pack_train_kernel(const float* __restrict__ p, const float* __restrict__ fp,
                                                         int NO, float* __restrict__ blob) {
    using L = TrainLayout<C, H, NH, NF>;
    constexpr int IN = L::IN, HT = L::HT;
    const auto nat = [](int i) { return slot_neuron<L::NAT>(i); };
    const int e = blockIdx.x * blockDim.x + threadIdx.x;
    if (e >= L::BLOB) return;
    const int oo = param_off<IN, H>(NH + 1);
    float v = 0.0f;
    if (e < L::FWH) {
        const int x = e - L::FW1, qq = x & 3, lane = (x >> 2) & 63, blk = x >> 8;
        const int grp = blk % L::G1, tp = blk / L::G1, g = lane >> 4, o = 16 * tp + nat(lane & 15);
        const int q = 4 * grp + qq;
        if (q < L::Q1) {
            const int in = L::NAT ? 4 * q + g : slot_input<C>(q, g);
            if (in >= 0 && in < IN) v = p[o * IN + in];
            else if (!L::NAT && in == C + 6) v = p[IN * H + o];
        }
    } else if (e < L::FWO) {
        const int k = 2 + (e - L::FWH) / L::WH_SZ, x = (e - L::FWH) % L::WH_SZ;
        const int r = x & 3, lane = (x >> 2) & 63, blk = x >> 8, t = blk % HT, tp = blk / HT;
        v = p[param_off<IN, H>(k) + (16 * tp + nat(lane & 15)) * H + 16 * t + nat(4 * (lane >> 4) + r)];
    } else if (e < L::BIAS) {
        const int x = e - L::FWO, r = x & 3, lane = (x >> 2) & 63, t = x >> 8, i = lane & 15;
        if (i < NO) v = p[oo + i * H + 16 * t + nat(4 * (lane >> 4) + r)];
    } else if (e < L::FF) {
        const int x = e - L::BIAS, k = 1 + x / (HT * 16), y = x % (HT * 16);   // y = slot 16t + 4g + r
        if (k <= NH) v = p[param_off<IN, H>(k) + (k == 1 ? IN : H) * H + (y & ~15) + nat(y & 15)];
        else if (y < NO) v = p[oo + NO * H + y];
    } else if (e < L::FWD) {
        if (e < L::FFB) {
            const int x = e - L::FF, lane = x & 63, i = lane & 15;
            if (i < 6 * NF) v = fp[i * C + 4 * (x >> 6) + (lane >> 4)];
        } else if (e - L::FFB < 6 * NF) {
            v = fp[6 * NF * C + e - L::FFB];
        }
    } else if (e < L::BWH) {
        const int x = e - L::BWO, lane = x & 63, blk = x >> 6, r = blk % L::NKO, tp = blk / L::NKO;
        const int o = 4 * (lane >> 4) + r;
        if (o < NO) v = p[oo + o * H + 16 * tp + nat(lane & 15)];
    } else if (e < L::BW1) {
        const int k = 2 + (e - L::BWH) / L::WH_SZ, x = (e - L::BWH) % L::WH_SZ;
        const int r = x & 3, lane = (x >> 2) & 63, blk = x >> 8, t = blk % HT, tp = blk / HT;
        v = p[param_off<IN, H>(k) + (16 * t + nat(4 * (lane >> 4) + r)) * H + 16 * tp + nat(lane & 15)];
    } else if (e < L::BF) {
        const int x = e - L::BW1, r = x & 3, lane = (x >> 2) & 63, blk = x >> 8, t = blk % HT, u = blk / HT;
        const int i = 16 * u + (lane & 15);
        if (i < (NF > 0 ? IN : C)) v = p[(16 * t + nat(4 * (lane >> 4) + r)) * IN + i];
    } else {
        const int x = e - L::BF, lane = x & 63, i = lane & 15, o = 4 * (x >> 6) + (lane >> 4);
        if (i < C && o < 6 * NF) v = fp[o * C + i];
    }
    blob[e] = v;
}

// A tile's query, loaded a tile before its texels.
struct TmQuery {
    float2 uv;
    float lod;
};

// One lane's share of a sample: the texel offsets and weights of its 8 taps (its 4 channels),
// the loaded texel words, the directions it needs and its targets or output gradients.
struct TmFetch {
    int off[8];
    float w[8];
    f32x4 v[8];
    float dir[6];
    f32x4 t;
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

// dir: without natural order the values of the lane's layer-1 slots (C = 16: [0..1], C = 8: lanes
// g >= 2 [0..3]); in natural order without frames inputs C + g and C + 4 + g; with frames all six.
template <int C, int NF, bool NAT, bool TRAIN>
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
        for (int r = 0; r < 4; ++r) f.t[r] = 4 * g + r < a.NO ? src[(int64_t)a.NO * ic + 4 * g + r] : 0.0f;
    }
    auto dir = [&](int d) { return d < 3 ? a.wi[3 * (int64_t)ic + d] : a.wo[3 * (int64_t)ic + d - 3]; };
    if (NF > 0) {
        #pragma unroll
        for (int d = 0; d < 6; ++d) f.dir[d] = dir(d);
    } else if (NAT || C == 16) {
        f.dir[0] = dir(g);
        f.dir[1] = g < 2 ? dir(4 + g) : (!NAT && g == 2 ? 1.0f : 0.0f);
    } else if (g == 2) {
        #pragma unroll
        for (int d = 0; d < 4; ++d) f.dir[d] = dir(d);
    } else if (g == 3) {
        f.dir[0] = dir(4);
        f.dir[1] = dir(5);
        f.dir[2] = 1.0f;
        f.dir[3] = 0.0f;
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

// The forward pass of a tile up to the output accumulator: what the backward pass needs is kept in
// x0 (layer-1 K slots), act (hidden activations) and, with frames, v (the frame layer's raw outputs,
// all of the sample's in every lane).  xch: the wave's exchange space (NF > 0).
template <int C, int H, int NH, int NF>
struct TmForward {
    using L = TrainLayout<C, H, NH, NF>;
    f32x4 z;                      // channels 4g..4g+3
    float x0[L::Q1];
    f32x4 act[NH][L::HT];
    float v[12];
    f32x4 qo;

    __device__ __forceinline__ void run(const float* blob, const TmFetch& f, bool live, float* xch, int lane) {
        constexpr int HT = L::HT, Q1 = L::Q1, G1 = L::G1;
        const int g = lane >> 4, s = lane & 15;
        const bool fetching = C == 16 || g < 2;
        z = f32x4{0, 0, 0, 0};
        if (fetching) {
            #pragma unroll
            for (int k = 0; k < 8; ++k)
                #pragma unroll
                for (int c = 0; c < 4; ++c) z[c] = fmaf(f.w[k], f.v[k][c], z[c]);
        }
        #pragma unroll
        for (int c = 0; c < 4; ++c) z[c] = live ? z[c] : 0.0f;
        if constexpr (L::NAT) {
            float zt[4] = {z[0], z[1], z[2], z[3]};
            transpose_groups(zt);
            #pragma unroll
            for (int q = 0; q < C / 4; ++q) x0[q] = zt[q];
            if constexpr (NF > 0) {
                // the frame layer: bias, then the channels in ascending order, as frame_inputs sums them
                f32x4 o = ld4(blob + L::FFB + 4 * g);
                #pragma unroll
                for (int q = 0; q < C / 4; ++q) o = mfma_f32(blob[L::FF + q * 64 + lane], zt[q], o);
                if (g < 3) st4(xch + s * 12 + 4 * g, o);
                lds_sync_wave();
                #pragma unroll
                for (int j = 0; j < 3; ++j) {
                    const f32x4 w = ld4(xch + s * 12 + 4 * j);
                    #pragma unroll
                    for (int r = 0; r < 4; ++r) v[4 * j + r] = w[r];
                }
                lds_sync_wave();
                float x[12];
                #pragma unroll
                for (int j = 6 * NF; j < 12; ++j) x[j] = 0.0f;
                #pragma unroll
                for (int i = 0; i < NF; ++i) frame_apply<NF>(i, v + 6 * i, f.dir, f.dir + 3, x);
                #pragma unroll
                for (int q = C / 4; q < Q1; ++q) x0[q] = pick4(x + 4 * (q - C / 4), g);
            } else {
                x0[C / 4] = f.dir[0];
                x0[C / 4 + 1] = f.dir[1];
            }
            #pragma unroll
            for (int q = C / 4; q < Q1; ++q) x0[q] = live ? x0[q] : 0.0f;
        } else if constexpr (C == 16) {
            #pragma unroll
            for (int q = 0; q < 4; ++q) x0[q] = z[q];
            x0[4] = live ? f.dir[0] : 0.0f;
            x0[5] = live ? f.dir[1] : 0.0f;
        } else {
            #pragma unroll
            for (int q = 0; q < 4; ++q) x0[q] = fetching ? z[q] : (live ? f.dir[q] : 0.0f);
        }

        f32x4 acc[HT];
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
            for (int r = 0; r < 4; ++r) act[0][t][r] = fmaxf(acc[t][r], 0.0f);
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
                    for (int tp = 0; tp < HT; ++tp) acc[tp] = mfma_f32(A[tp][r], act[k - 2][t][r], acc[tp]);
            }
            #pragma unroll
            for (int t = 0; t < HT; ++t)
                #pragma unroll
                for (int r = 0; r < 4; ++r) act[k - 1][t][r] = fmaxf(acc[t][r], 0.0f);
        }
        qo = ld4(blob + L::BIAS + NH * HT * 16 + 4 * g);
        #pragma unroll
        for (int t = 0; t < HT; ++t) {
            const f32x4 A = ld4(blob + L::FWO + (t * 64 + lane) * 4);
            #pragma unroll
            for (int r = 0; r < 4; ++r) qo = mfma_f32(A[r], act[NH - 1][t][r], qo);
        }
    }
};

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
        tm_issue<C, NF, L::NAT, false>(a, lrows, wid, q, g, s, cur);
        tm_query(a, wid + waves, s, q);
    }
    for (int tile = wid; tile < tiles; tile += waves) {
        if (tile + waves < tiles) {
            tm_issue<C, NF, L::NAT, false>(a, lrows, tile + waves, q, g, s, nxt);
            tm_query(a, tile + 2 * waves, s, q);
        }
        const int i = tile * 16 + s;
        const bool in_range = i < a.n;
        asm volatile("" ::: "memory");          // the weights are read per tile, not kept in registers
        TmForward<C, H, NH, NF> fw;
        fw.run(smem, cur, in_range && cur.finite, xch, lane);
        if (in_range) {
            #pragma unroll
            for (int r = 0; r < 4; ++r) {
                const int row = 4 * g + r;
                if (row < a.NO) a.rgb[(int64_t)a.NO * i + row] = cur.finite ? tm_softplus<L::NAT>(fw.qo[r]) : __builtin_nanf("");
            }
        }
        cur = nxt;
    }
}

// ---- forward and backward

// The slots of one pair: handoff n lies in slot n & 1.  `filled` counts the handoffs written by the
// front wave, `emptied` those the back wave has read; each is written by one wave only.  The front
// wave waits until handoff n - 2 is read, the back wave until handoff n is written.  Both waves of a
// pair walk the same tiles with the same number of handoffs each, so every wait ends.
typedef __attribute__((address_space(3))) volatile int lds_count;

struct TmRing {
    float* slots;
    lds_count* filled;
    lds_count* emptied;
    int n;

    __device__ __forceinline__ float* slot() const { return slots + (n & 1) * (2 * kSlotMatrix); }
    __device__ __forceinline__ static void wait(lds_count* count, int need) {
        while (__builtin_amdgcn_readfirstlane(*count) < need) __builtin_amdgcn_s_sleep(1);
        __builtin_amdgcn_wave_barrier();
    }
    __device__ __forceinline__ float* begin_fill() const {
        wait(emptied, n - 1);
        return slot();
    }
    __device__ __forceinline__ void end_fill() {
        lds_sync_wave();                        // the slot's writes are done
        *filled = ++n;
    }
    __device__ __forceinline__ const float* begin_read() const {
        wait(filled, n + 1);
        return slot();
    }
    __device__ __forceinline__ void end_read() {
        lds_sync_wave();                        // the reads are done
        *emptied = ++n;
    }
};

// Operand of a contraction over the tile's samples: column tile c of a slot matrix, sample 4g + r in
// register r.
__device__ __forceinline__ f32x4 slot_column(const float* m, int c, int lane) {
    const int g = lane >> 4, i = lane & 15;
    f32x4 v;
    #pragma unroll
    for (int r = 0; r < 4; ++r) v[r] = m[slot_at(4 * g + r, 16 * c + i)];
    return v;
}

__device__ __forceinline__ float sum4(const f32x4 v) { return (v[0] + v[1]) + (v[2] + v[3]); }

template <int C, int H, int NH, int NF>
__device__ __forceinline__ void train_front(const TrainArgs& a, const float* blob, const LevelRow* lrows, float* xch,
                                            TmRing ring, int wid, int waves, int tiles, int lane) {
    using L = TrainLayout<C, H, NH, NF>;
    constexpr int HT = L::HT;
    const int g = lane >> 4, s = lane & 15;
    const int NO = a.NO;
    const bool fetching = C == 16 || g < 2;
    float loss_acc = 0.0f, absmax = 0.0f;
    TmQuery q;
    TmFetch cur, nxt;
    if (wid < tiles) {
        tm_query(a, wid, s, q);
        tm_issue<C, NF, L::NAT, true>(a, lrows, wid, q, g, s, cur);
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
        TmForward<C, H, NH, NF> fw;
        fw.run(blob, cur, live, xch, lane);

        // ---- output deltas: dL/dq = dL/dy * logistic(q)
        f32x4 dq = f32x4{0, 0, 0, 0};
        #pragma unroll
        for (int r = 0; r < 4; ++r) {
            if (4 * g + r < NO && live) {
                float gy = cur.t[r];
                if (a.target) {
                    const float e = tm_softplus<L::NAT>(fw.qo[r]) - cur.t[r];
                    loss_acc = fmaf(e, e, loss_acc);
                    gy = 2.0f * e * a.inv_count;
                }
                dq[r] = gy * tm_logistic<L::NAT>(fw.qo[r]);
            }
        }
        {
            float* m = ring.begin_fill();
            st4(m + slot_at(s, 4 * g), dq);
            #pragma unroll
            for (int t = 0; t < HT; ++t) st4(m + kSlotMatrix + slot_at(s, 16 * t + 4 * g), fw.act[NH - 1][t]);
            ring.end_fill();
        }
        // delta_NH = W_out^T delta_out, masked by a_NH > 0 (K step r: outputs 4g + r)
        f32x4 dl[HT];
        #pragma unroll
        for (int tp = 0; tp < HT; ++tp) {
            f32x4 acc = f32x4{0, 0, 0, 0};
            #pragma unroll
            for (int r = 0; r < L::NKO; ++r)
                if (r < 3 || NO > 3) acc = mfma_f32(blob[L::BWO + (tp * L::NKO + r) * 64 + lane], dq[r], acc);
            #pragma unroll
            for (int r = 0; r < 4; ++r) dl[tp][r] = fw.act[NH - 1][tp][r] > 0.0f ? acc[r] : 0.0f;
        }
        // hidden layers k = NH .. 2: hand (delta_k, a_{k-1}) over, then delta_{k-1}
        #pragma unroll
        for (int k = NH; k >= 2; --k) {
            float* m = ring.begin_fill();
            #pragma unroll
            for (int t = 0; t < HT; ++t) {
                st4(m + slot_at(s, 16 * t + 4 * g), dl[t]);
                st4(m + kSlotMatrix + slot_at(s, 16 * t + 4 * g), fw.act[k - 2][t]);
            }
            ring.end_fill();
            f32x4 acc[HT];
            #pragma unroll
            for (int tp = 0; tp < HT; ++tp) acc[tp] = f32x4{0, 0, 0, 0};
            #pragma unroll
            for (int t = 0; t < HT; ++t) {
                f32x4 A[HT];
                #pragma unroll
                for (int tp = 0; tp < HT; ++tp) A[tp] = ld4(blob + L::BWH + (k - 2) * L::WH_SZ + ((tp * HT + t) * 64 + lane) * 4);
                #pragma unroll
                for (int r = 0; r < 4; ++r)
                    #pragma unroll
                    for (int tp = 0; tp < HT; ++tp) acc[tp] = mfma_f32(A[tp][r], dl[t][r], acc[tp]);
            }
            #pragma unroll
            for (int tp = 0; tp < HT; ++tp)
                #pragma unroll
                for (int r = 0; r < 4; ++r) dl[tp][r] = fw.act[k - 2][tp][r] > 0.0f ? acc[tp][r] : 0.0f;
        }
        // the next tile's texels, now that the activations' registers are free
        if (tile + waves < tiles) {
            tm_issue<C, NF, L::NAT, true>(a, lrows, tile + waves, q, g, s, nxt);
            tm_query(a, tile + 2 * waves, s, q);
        }
        // (delta_1, the input with its constant-1 column)
        {
            float* m = ring.begin_fill();
            #pragma unroll
            for (int t = 0; t < HT; ++t) st4(m + slot_at(s, 16 * t + 4 * g), dl[t]);
            float* x = m + kSlotMatrix;
            if constexpr (!L::NAT && C == 8) {
                st4(x + slot_at(s, 4 * g), f32x4{fw.x0[0], fw.x0[1], fw.x0[2], fw.x0[3]});
            } else {
                if (fetching) st4(x + slot_at(s, 4 * g), fw.z);
                #pragma unroll
                for (int qq = C / 4; qq < 4 * L::NCT1; ++qq) {
                    const int col = 4 * qq + g;
                    x[slot_at(s, col)] = qq < L::Q1 && col < L::IN ? fw.x0[qq < L::Q1 ? qq : 0] : (col == L::IN ? 1.0f : 0.0f);
                }
            }
            ring.end_fill();
        }
        // the gradient of the latent code (with frames of the whole input: row tile u, inputs 16u ..)
        f32x4 dx[L::NR1];
        #pragma unroll
        for (int u = 0; u < L::NR1; ++u) dx[u] = f32x4{0, 0, 0, 0};
        #pragma unroll
        for (int t = 0; t < HT; ++t) {
            f32x4 A[L::NR1];
            #pragma unroll
            for (int u = 0; u < L::NR1; ++u) A[u] = ld4(blob + L::BW1 + ((u * HT + t) * 64 + lane) * 4);
            #pragma unroll
            for (int r = 0; r < 4; ++r)
                #pragma unroll
                for (int u = 0; u < L::NR1; ++u) dx[u] = mfma_f32(A[u][r], dl[t][r], dx[u]);
        }
        f32x4 dz = dx[0];
        if constexpr (NF > 0) {
            // through the frame transform into the frame layer and the latent code: every lane takes
            // the sample's 6 NF direction gradients, the layer's back product is one more MFMA chain
            #pragma unroll
            for (int u = C / 16; u < L::NR1; ++u) {
                const int col = 16 * u + 4 * g - C;
                if (col >= 0 && col < 12) st4(xch + s * 12 + col, dx[u]);
            }
            lds_sync_wave();
            float G[12], draw[12];
            #pragma unroll
            for (int j = 0; j < (6 * NF + 3) / 4; ++j) {
                const f32x4 w = ld4(xch + s * 12 + 4 * j);
                #pragma unroll
                for (int r = 0; r < 4; ++r) G[4 * j + r] = w[r];
            }
            lds_sync_wave();
            #pragma unroll
            for (int j = 6 * NF; j < 12; ++j) draw[j] = 0.0f;
            #pragma unroll
            for (int f = 0; f < NF; ++f) frame_backward_raw<NF>(f, fw.v + 6 * f, cur.dir, cur.dir + 3, G, draw + 6 * f);
            #pragma unroll
            for (int j = 0; j < 6 * NF; ++j) draw[j] = live ? draw[j] : 0.0f;
            #pragma unroll
            for (int qq = 0; qq < (6 * NF + 3) / 4; ++qq) dz = mfma_f32(blob[L::BF + qq * 64 + lane], pick4(draw + 4 * qq, g), dz);
            float* m = ring.begin_fill();
            f32x4 w = f32x4{0, 0, 0, 0};
            #pragma unroll
            for (int r = 0; r < 4; ++r) w[r] = g == 0 ? draw[r] : (g == 1 ? draw[4 + r] : (g == 2 ? draw[8 + r] : 0.0f));
            st4(m + slot_at(s, 4 * g), w);
            st4(m + kSlotMatrix + slot_at(s, 4 * g), fetching ? fw.z : f32x4{0, 0, 0, 0});
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
            // scatter into the texels, C lanes per sample: in round r, lane (u, c) =
            // (lane / C, lane % C) adds channel c of sample r (64 / C) + u, so one atomic
            // instruction covers 64 / C whole texels and the memory side takes each texel as
            // one request (with the lanes of the accumulator layout it took a quarter of a
            // texel per request).  Channel c of sample q is component c % 4 of lane
            // 16 (c / 4) + q; the taps of sample q are in lane q, whose offsets point at
            // channel 0.  Every lane runs the exchanges; only live samples add.
            constexpr int SPR = 64 / C;
            const int u = lane / C, c = lane % C;
            #pragma unroll
            for (int r = 0; r < 16 / SPR; ++r) {
                const int qs = r * SPR + u;
                const int src = 16 * (c >> 2) + qs;
                const float d0 = __shfl(dz[0], src), d1 = __shfl(dz[1], src);
                const float d2 = __shfl(dz[2], src), d3 = __shfl(dz[3], src);
                const int cc = c & 3;
                const float d = cc == 0 ? d0 : (cc == 1 ? d1 : (cc == 2 ? d2 : d3));
                const bool lq = __shfl((int)live, qs) != 0;
                #pragma unroll
                for (int k = 0; k < 8; ++k) {
                    const int o = __shfl(cur.off[k], qs);
                    const float w = __shfl(cur.w[k], qs);
                    if (lq) unsafeAtomicAdd(a.d_tex + o + c, w * d);
                }
            }
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

template <int C, int H, int NH, int NF>
__device__ __forceinline__ void train_back(const TrainArgs& a, TmRing ring, int wid, int waves, int tiles, int lane) {
    using L = TrainLayout<C, H, NH, NF>;
    constexpr int HT = L::HT, NCT1 = L::NCT1, IN = L::IN, HH = NH > 1 ? NH - 1 : 1;
    const int g = lane >> 4, s = lane & 15;
    const int NO = a.NO;
    f32x4 dW1[HT][NCT1], dWh[HH][HT][HT], dWo[HT], dF = f32x4{0, 0, 0, 0};
    float dbh[HH][HT], dbo = 0.0f, dbf = 0.0f;
    #pragma unroll
    for (int t = 0; t < HT; ++t) {
        #pragma unroll
        for (int c = 0; c < NCT1; ++c) dW1[t][c] = f32x4{0, 0, 0, 0};
        dWo[t] = f32x4{0, 0, 0, 0};
        #pragma unroll
        for (int k = 0; k < HH; ++k) {
            #pragma unroll
            for (int c = 0; c < HT; ++c) dWh[k][t][c] = f32x4{0, 0, 0, 0};
            dbh[k][t] = 0.0f;
        }
    }
    for (int tile = wid; tile < tiles; tile += waves) {
        {   // dW_out += delta_out a_NH^T (samples on K)
            const float* m = ring.begin_read();
            const f32x4 Ad = slot_column(m, 0, lane);
            f32x4 B[HT];
            #pragma unroll
            for (int c = 0; c < HT; ++c) B[c] = slot_column(m + kSlotMatrix, c, lane);
            ring.end_read();
            #pragma unroll
            for (int r = 0; r < 4; ++r)
                #pragma unroll
                for (int c = 0; c < HT; ++c) dWo[c] = mfma_f32(Ad[r], B[c][r], dWo[c]);
            dbo += sum4(Ad);
        }
        #pragma unroll
        for (int k = NH; k >= 2; --k) {
            const float* m = ring.begin_read();
            f32x4 Ad[HT], B[HT];
            #pragma unroll
            for (int c = 0; c < HT; ++c) {
                Ad[c] = slot_column(m, c, lane);
                B[c] = slot_column(m + kSlotMatrix, c, lane);
            }
            ring.end_read();
            #pragma unroll
            for (int co = 0; co < HT; ++co) {
                #pragma unroll
                for (int r = 0; r < 4; ++r)
                    #pragma unroll
                    for (int cj = 0; cj < HT; ++cj) dWh[k - 2][co][cj] = mfma_f32(Ad[co][r], B[cj][r], dWh[k - 2][co][cj]);
                dbh[k - 2][co] += sum4(Ad[co]);
            }
        }
        {   // dW_1, the bias as one more column
            const float* m = ring.begin_read();
            f32x4 Ad[HT], B[NCT1];
            #pragma unroll
            for (int c = 0; c < HT; ++c) Ad[c] = slot_column(m, c, lane);
            #pragma unroll
            for (int c = 0; c < NCT1; ++c) B[c] = slot_column(m + kSlotMatrix, c, lane);
            ring.end_read();
            #pragma unroll
            for (int r = 0; r < 4; ++r)
                #pragma unroll
                for (int co = 0; co < HT; ++co)
                    #pragma unroll
                    for (int cj = 0; cj < NCT1; ++cj) dW1[co][cj] = mfma_f32(Ad[co][r], B[cj][r], dW1[co][cj]);
        }
        if constexpr (NF > 0) {   // the frame layer: its raw outputs' gradients with the latent code
            const float* m = ring.begin_read();
            const f32x4 Ad = slot_column(m, 0, lane), B = slot_column(m + kSlotMatrix, 0, lane);
            ring.end_read();
            #pragma unroll
            for (int r = 0; r < 4; ++r) dF = mfma_f32(Ad[r], B[r], dF);
            dbf += sum4(Ad);
        }
    }

    // ---- this wave's gradients into its own partial slice (every parameter written once)
    float* part = a.partial + (size_t)wid * a.np;
    const auto nat = [](int i) { return slot_neuron<L::NAT>(i); };
    // a bias sum over the samples lies in the four lane groups
    const auto over_groups = [](float v) {
        v += __shfl_xor(v, 16, 64);
        return v + __shfl_xor(v, 32, 64);
    };
    if constexpr (NF > 0) {
        #pragma unroll
        for (int r = 0; r < 4; ++r)
            if (4 * g + r < 6 * NF && s < C) part[(4 * g + r) * C + s] = dF[r];
        const float b = over_groups(dbf);
        if (g == 0 && s < 6 * NF) part[6 * NF * C + s] = b;
        part += L::NP1;
    }
    #pragma unroll
    for (int co = 0; co < HT; ++co)
        #pragma unroll
        for (int cj = 0; cj < NCT1; ++cj)
            #pragma unroll
            for (int r = 0; r < 4; ++r) {
                const int o = 16 * co + nat(4 * g + r), j = 16 * cj + s;
                if (j < IN) part[o * IN + j] = dW1[co][cj][r];
                else if (j == IN) part[IN * H + o] = dW1[co][cj][r];
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
                    part[off + (16 * co + nat(4 * g + r)) * H + 16 * cj + nat(s)] = dWh[k - 2][co][cj][r];
            const float b = over_groups(dbh[k - 2][co]);
            if (g == 0) part[off + H * H + 16 * co + nat(s)] = b;
        }
    }
    const int off = param_off<IN, H>(NH + 1);
    #pragma unroll
    for (int c = 0; c < HT; ++c)
        #pragma unroll
        for (int r = 0; r < 4; ++r)
            if (4 * g + r < NO) part[off + (4 * g + r) * H + 16 * c + nat(s)] = dWo[c][r];
    const float b = over_groups(dbo);
    if (g == 0 && s < NO) part[off + NO * H + s] = b;
}

// Measured on 2^20 samples of 22-64-64-64-3 (one wave doing both jobs before): 770 us with fetch and
// scatter (903), 611 us on given codes (707).  What bounds it: FP32 matrix instructions and vector
// instructions take turns on a SIMD (the forward kernel takes the sum of both, 224 us at four waves
// per SIMD), here 496 x 32 cycles and about 1,300 vector instructions per 16 samples.  The scatter's
// atomics alone take 412 us (random 128-byte lines beyond the L2) and overlap it.  With two learned
// frames (28-64-64-64-3, 250,007 samples) the call takes 321 us; the vector kernel took 2,570 us.
template <int C, int H, int NH, int NF>
__global__ void __launch_bounds__(kTMThreads, 1) train_mfma_kernel(const TrainArgs a) {
    using L = TrainLayout<C, H, NH, NF>;
    __shared__ __attribute__((aligned(16))) float smem[L::LDS_FLOATS];
    __shared__ LevelRow lrows[kMaxLevels];
    __shared__ int counts[2][kTMPairs];
    const int tid = threadIdx.x;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6), lane = tid & 63;
    for (int e = tid; e < L::BLOB / 4; e += kTMThreads) st4(smem + 4 * e, ld4(a.blob + 4 * e));
    if (tid < a.M) lrows[tid] = a.rows[tid];
    if (tid < 2 * kTMPairs) counts[tid / kTMPairs][tid % kTMPairs] = 0;
    __syncthreads();
    const int pair = wave % kTMPairs;
    if (pair >= a.pairs) return;
    const int tiles = (a.n + 15) / 16;
    const int waves = gridDim.x * a.pairs;
    const int wid = blockIdx.x * a.pairs + pair;
    const TmRing ring{smem + L::BLOB + pair * 2 * L::SLOT, (lds_count*)&counts[0][pair], (lds_count*)&counts[1][pair], 0};
    if (wave < kTMPairs) {
        __builtin_amdgcn_s_setprio(1);          // the chain that the back wave waits for goes first
        train_front<C, H, NH, NF>(a, smem, lrows, smem + L::BLOB + kTMPairs * 2 * L::SLOT + pair * L::XCH, ring, wid, waves,
                                  tiles, lane);
    } else {
        train_back<C, H, NH, NF>(a, ring, wid, waves, tiles, lane);
    }
}

// pack: pack the decoder from params (and the frame layer) into blob; run: launch the kernel on it
template <int C, int H, int NH, int NF>
static hipError_t launch_tm_shape(bool pack, bool run, bool train, const float* params, const float* fparams, int NO,
                                  float* blob, const TrainArgs& a, int grid, hipStream_t st) {
    using L = TrainLayout<C, H, NH, NF>;
    static_assert(L::FITS, "the decoder's blocks and the slots exceed the LDS");
    clear_stale_hip_error();
    if (pack) {
        pack_train_kernel<C, H, NH, NF><<<(L::BLOB + 255) / 256, 256, 0, st>>>(params, fparams, NO, blob);
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
