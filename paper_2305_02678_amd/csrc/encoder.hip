// The encoder of Sec. 5.1 on the FP32 matrix cores: an MLP from the parameters of the original
// material at a location (A attributes: albedo, roughness, ...) to the latent code (C
// channels), ReLU hidden layers and a linear output layer.  Its weights are packed as the
// decoder's (W_1[HE][A], b_1, ..., W_out[C][HE], b_out).
//
// Each wave of a workgroup walks its own tiles of 16 items; lane (g, s) = (lane / 16, lane % 16) works
// on item s.  A layer is Y = W X on v_mfma_f32_16x16x4_f32, a chain of FMAs in ascending k, with the
// weights as the A operand: row slot i of a row tile is neuron 4 (i % 4) + i / 4, so that the accumulator
// of lane (g, s) holds neurons 4 r + g, the B operand of K step r of the next layer, and the sums run over
// the neurons in ascending order.  The weights lie in LDS as operands, shared by the workgroup.
//
// encoder_forward_kernel: for queries the parameters are first filtered at (uv, lod) with the latent
// fetch's trilinear taps over a pyramid of the parameters (levels concatenated, [texel][A]); the bake
// instead takes parameter rows as given (every texel of every level: the latent texture's
// initialisation).
//
// encoder_backward_kernel: the encoder's share of the first training phase, the gradient of
// sum_i dz_i . E(filtered parameters at query i).
#include "train_vec.h"

namespace nam {

typedef float f32x4e __attribute__((ext_vector_type(4)));

__device__ __forceinline__ int enc_neuron(int i) { return 4 * (i & 3) + (i >> 2); }

// acc[t] += W b over K steps, blocks at w
template <int HT, int K>
__device__ __forceinline__ void enc_layer(const float* w, const float* b, f32x4e* acc, int lane) {
    #pragma unroll
    for (int q = 0; q < K; ++q)
        #pragma unroll
        for (int t = 0; t < HT; ++t)
            acc[t] = __builtin_amdgcn_mfma_f32_16x16x4f32(w[(t * K + q) * 64 + lane], b[q], acc[t], 0, 0, 0);
}

// Attributes 4q + g of an item: of a parameter row, or the trilinear filter of the pyramid at the query;
// false for a query with a non-finite uv or lod.
template <int A, bool QUERIES>
__device__ __forceinline__ bool enc_input(const EncoderArgs& a, const LevelRow* rows, int i, int g, float* x) {
    if (!QUERIES) {
        #pragma unroll
        for (int q = 0; q < A / 4; ++q) x[q] = a.attrs[(int64_t)i * A + 4 * q + g];
        return true;
    }
    const float2 uv = reinterpret_cast<const float2*>(a.uv)[i];
    const float l = a.lod[i];
    Taps t;
    query_taps_rows(rows, a.M, a.address, uv.x, uv.y, l, t);
    #pragma unroll
    for (int q = 0; q < A / 4; ++q) x[q] = 0.0f;
    #pragma unroll
    for (int k = 0; k < 8; ++k) {
        const float* T = a.attrs + t.idx[k] * A + g;
        #pragma unroll
        for (int q = 0; q < A / 4; ++q) x[q] = fmaf(t.w[k], T[4 * q], x[q]);
    }
    return query_ok(uv.x, uv.y, l);
}

// ---- forward
//
// What bounds it: the random texels, 8 per item at uniform queries: 2^20 items at 4-32-32-16 over a
// 1024 x 1024 pyramid of 22 MB take 81 us (one item per lane with the layers on the vector ALU and a
// code written 64 bytes apart per lane 89 us), the 100,003 of an encoder of width 16 10 us less.
constexpr int kEncFwdWaves = 4;

template <int A, int C, int HE, int NHE>
struct EncForward {
    static constexpr int HT = HE / 16, KA = A / 4, KH = HE / 4;
    // operand blocks [row tile][K step][lane]; W_out's rows are channels in order; the biases
    static constexpr int W1 = 0;
    static constexpr int W2 = W1 + HT * KA * 64;
    static constexpr int WO = W2 + (NHE - 1) * HT * KH * 64;
    static constexpr int BIAS = WO + KH * 64;
    static constexpr int BO = BIAS + NHE * HE;
    static constexpr int FLOATS = BO + 16;
};

template <int A, int C, int HE, int NHE, bool QUERIES>
__global__ void __launch_bounds__(64 * kEncFwdWaves) encoder_forward_kernel(const EncoderArgs a) {
    using L = EncForward<A, C, HE, NHE>;
    constexpr int HT = L::HT;
    __shared__ __attribute__((aligned(16))) float lds[L::FLOATS];
    __shared__ LevelRow rows[kMaxLevels];
    const int tid = threadIdx.x, lane = tid & 63, g = lane >> 4, s = lane & 15;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    if (QUERIES && tid < a.M) rows[tid] = a.rows[tid];
    const float* P2 = a.params + A * HE + HE;
    const float* PO = P2 + (NHE - 1) * (HE * HE + HE);
    for (int e = tid; e < L::FLOATS; e += 64 * kEncFwdWaves) {
        const int eg = (e >> 4) & 3, ei = enc_neuron(e & 15);
        float v;
        if (e < L::W2) {
            const int b = e >> 6, q = b % L::KA, t = b / L::KA;
            v = a.params[(16 * t + ei) * A + 4 * q + eg];
        } else if (e < L::WO) {
            const int b = (e - L::W2) >> 6, q = b % L::KH, t = b / L::KH;
            v = P2[(16 * t + ei) * HE + 4 * q + eg];
        } else if (e < L::BIAS) {
            const int q = (e - L::WO) >> 6, o = e & 15;
            v = o < C ? PO[o * HE + 4 * q + eg] : 0.0f;
        } else if (e < L::BO) {
            const int k = (e - L::BIAS) / HE, y = (e - L::BIAS) % HE, o = (y & ~15) + 4 * (y & 3) + ((y >> 2) & 3);
            v = k == 0 ? a.params[A * HE + o] : P2[HE * HE + o];
        } else {
            const int o = e - L::BO;
            v = o < C ? PO[C * HE + o] : 0.0f;
        }
        lds[e] = v;
    }
    __syncthreads();
    const bool wide = (reinterpret_cast<uintptr_t>(a.z) & 15) == 0;
    const int tiles = (a.n - 1) / 16 + 1, waves = gridDim.x * kEncFwdWaves;
    // consecutive tiles on different workgroups: a small batch spreads over the CUs
    for (int tile = wave * gridDim.x + blockIdx.x; tile < tiles; tile += waves) {
        asm volatile("" ::: "memory");         // the weights are read per tile, not kept in registers
        const int64_t i = (int64_t)tile * 16 + s;
        const int ic = i < a.n ? (int)i : a.n - 1;
        float x[HE / 4 > L::KA ? HE / 4 : L::KA];
        const bool ok = enc_input<A, QUERIES>(a, rows, ic, g, x);
        f32x4e acc[HT];
        #pragma unroll
        for (int k = 0; k < NHE; ++k) {
            #pragma unroll
            for (int u = 0; u < HT; ++u) acc[u] = *reinterpret_cast<const f32x4e*>(lds + L::BIAS + (k * HT + u) * 16 + 4 * g);
            if (k == 0) enc_layer<HT, L::KA>(lds + L::W1, x, acc, lane);
            else enc_layer<HT, L::KH>(lds + L::W2, x, acc, lane);
            #pragma unroll
            for (int j = 0; j < HE / 4; ++j) x[j] = fmaxf(acc[j / 4][j % 4], 0.0f);
        }
        f32x4e z[1] = {*reinterpret_cast<const f32x4e*>(lds + L::BO + 4 * g)};
        enc_layer<1, L::KH>(lds + L::WO, x, z, lane);
        if (i < a.n && 4 * g < C) {
            float* to = a.z + i * C + 4 * g;
            #pragma unroll
            for (int r = 0; r < 4; ++r) z[0][r] = ok ? z[0][r] : __builtin_nanf("");
            if (wide) {
                *reinterpret_cast<f32x4e*>(to) = z[0];
            } else {
                #pragma unroll
                for (int r = 0; r < 4; ++r) to[r] = z[0][r];
            }
        }
    }
}

// ---- backward
//
// A layer's weight gradient is a contraction over the samples (the activations are bit for bit the forward
// kernel's): activations and deltas pass through the wave's LDS rows, which give them back with the
// samples on the K index, and the sums stay in registers over all of the wave's tiles.  At the end the
// workgroup sums its waves in ascending order into its slice of the partial buffer; the slices are
// reduced in a fixed order afterwards.
//
// What bounds it: FP32 matrix and vector instructions, which take turns on a SIMD: at 4-32-32-16 86 of
// the former at 32 cycles per tile, 73 us of 2^20 samples.  One sample per lane with the layers on the
// vector ALU and one wave per SIMD took 371 us; this takes 130 us, 81 us of it the forward kernel's
// fetch.
constexpr int kEncWaves = 8;
constexpr int kES = 17;                        // LDS row stride: the 16 samples of a tile, one bank apart

template <int A, int C, int HE, int NHE>
struct EncTile {
    static constexpr int HT = HE / 16, KA = A / 4, KH = HE / 4, KC = C / 4;   // row tiles, K steps
    // operand blocks [row tile][K step][lane], then the biases [layer][row tile][g][r]
    static constexpr int W1 = 0;
    static constexpr int W2 = W1 + HT * KA * 64;
    static constexpr int WOT = W2 + (NHE - 1) * HT * KH * 64;                 // W_out^T
    static constexpr int W2T = WOT + HT * KC * 64;
    static constexpr int BIAS = W2T + (NHE - 1) * HT * KH * 64;
    static constexpr int WEIGHTS = BIAS + NHE * HE;
    // a wave's rows: input, hidden layers (activations, then their deltas), output deltas
    static constexpr int X = 0;
    static constexpr int hid(int k) { return A + k * HE; }
    static constexpr int D = A + NHE * HE;
    static constexpr int ROWS = D + C;
    static constexpr int SUM = kEncWaves * 4 * 256;                           // 4 tiles of every wave
    static constexpr int WORK = WEIGHTS + kEncWaves * ROWS * kES;
    static constexpr int LDS = WORK > SUM ? WORK : SUM;
    // packed offsets of the layers
    static constexpr int off(int k) {
        return k == 0 ? 0 : (k == NHE ? A * HE + HE + (NHE - 1) * (HE * HE + HE) : A * HE + HE);
    }
};

// Weight gradient of one layer: G[o][j] += sum_s delta[o][s] x[j][s] for o < FO, j <= FI, with
// x[FI][s] = 1 so that column FI is the bias gradient.
template <int FI, int FO>
struct GradTiles {
    static constexpr int RO = (FO + 15) / 16;
    static constexpr int CJ = (FI + 1 + 15) / 16;
    f32x4e acc[RO][CJ];

    __device__ __forceinline__ void zero() {
        #pragma unroll
        for (int r = 0; r < RO; ++r)
            #pragma unroll
            for (int c = 0; c < CJ; ++c) acc[r][c] = f32x4e{0.0f, 0.0f, 0.0f, 0.0f};
    }

    // delta, x: the wave's rows of the layer
    __device__ __forceinline__ void add(const float* delta, const float* x, int lane) {
        const int i = lane & 15, g = lane >> 4;
        #pragma unroll
        for (int k = 0; k < 4; ++k) {
            const int smp = 4 * k + g;
            float av[RO], bv[CJ];
            #pragma unroll
            for (int r = 0; r < RO; ++r) {
                const int o = 16 * r + i;
                av[r] = o < FO ? delta[o * kES + smp] : 0.0f;
            }
            #pragma unroll
            for (int c = 0; c < CJ; ++c) {
                const int j = 16 * c + i;
                bv[c] = j < FI ? x[j * kES + smp] : (j == FI ? 1.0f : 0.0f);
            }
            #pragma unroll
            for (int r = 0; r < RO; ++r)
                #pragma unroll
                for (int c = 0; c < CJ; ++c)
                    acc[r][c] = __builtin_amdgcn_mfma_f32_16x16x4f32(av[r], bv[c], acc[r][c], 0, 0, 0);
        }
    }

    // The workgroup's sum into the packed slice (W[FO][FI], then b[FO]), four tiles at a time.
    __device__ __forceinline__ void store(float* sum, float* part, int wave, int lane) const {
        #pragma unroll
        for (int first = 0; first < RO * CJ; first += 4) {
            __syncthreads();
            #pragma unroll
            for (int u = 0; u < 4; ++u)
                if (first + u < RO * CJ)
                    *reinterpret_cast<f32x4e*>(sum + ((wave * 4 + u) * 64 + lane) * 4) = acc[(first + u) / CJ][(first + u) % CJ];
            __syncthreads();
            const int tile = first + wave, r = tile / CJ, c = tile % CJ;
            if (wave < 4 && tile < RO * CJ) {
                f32x4e v = {0.0f, 0.0f, 0.0f, 0.0f};
                #pragma unroll
                for (int w = 0; w < kEncWaves; ++w)
                    v += *reinterpret_cast<const f32x4e*>(sum + ((w * 4 + wave) * 64 + lane) * 4);
                #pragma unroll
                for (int e = 0; e < 4; ++e) {
                    const int o = 16 * r + 4 * (lane >> 4) + e, j = 16 * c + (lane & 15);
                    if (o < FO && j < FI) part[o * FI + j] = v[e];
                    else if (o < FO && j == FI) part[FI * FO + o] = v[e];
                }
            }
        }
    }
};

// Waves per SIMD: at width 64 the gradients' registers leave room for two.
template <int A, int C, int HE, int NHE>
__global__ void __launch_bounds__(64 * kEncWaves, HE == 64 ? 2 : 4) encoder_backward_kernel(const EncoderArgs a) {
    using L = EncTile<A, C, HE, NHE>;
    constexpr int HT = L::HT;
    __shared__ __attribute__((aligned(16))) float lds[L::LDS];
    __shared__ LevelRow rows[kMaxLevels];
    const int tid = threadIdx.x, lane = tid & 63, g = lane >> 4, s = lane & 15;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    if (tid < a.M) rows[tid] = a.rows[tid];
    const float* P2 = a.params + L::off(1);
    const float* PO = a.params + L::off(NHE);
    for (int e = tid; e < L::WEIGHTS; e += 64 * kEncWaves) {
        const int eg = (e >> 4) & 3, ei = enc_neuron(e & 15);
        float v;
        if (e < L::W2) {
            const int b = e >> 6, q = b % L::KA, t = b / L::KA;
            v = a.params[(16 * t + ei) * A + 4 * q + eg];
        } else if (e < L::WOT) {
            const int b = (e - L::W2) >> 6, q = b % L::KH, t = b / L::KH;
            v = P2[(16 * t + ei) * HE + 4 * q + eg];
        } else if (e < L::W2T) {
            const int b = (e - L::WOT) >> 6, q = b % L::KC, t = b / L::KC;
            v = PO[(4 * q + eg) * HE + 16 * t + ei];
        } else if (e < L::BIAS) {
            const int b = (e - L::W2T) >> 6, q = b % L::KH, t = b / L::KH;
            v = P2[(4 * q + eg) * HE + 16 * t + ei];
        } else {
            const int k = (e - L::BIAS) / HE, y = (e - L::BIAS) % HE, o = (y & ~15) + 4 * (y & 3) + ((y >> 2) & 3);
            v = k == 0 ? a.params[A * HE + o] : P2[HE * HE + o];
        }
        lds[e] = v;
    }
    __syncthreads();
    float* table = lds + L::WEIGHTS + wave * L::ROWS * kES;
    GradTiles<A, HE> g0;
    GradTiles<HE, HE> gh;                      // the hidden-to-hidden layer (NHE = 2)
    GradTiles<HE, C> go;
    g0.zero();
    gh.zero();
    go.zero();
    const int tiles = (a.n - 1) / 16 + 1, waves = gridDim.x * kEncWaves;
    // consecutive tiles on different workgroups: a small batch spreads over the CUs
    for (int tile = wave * gridDim.x + blockIdx.x; tile < tiles; tile += waves) {
        asm volatile("" ::: "memory");         // the weights are read per tile, not kept in registers
        const int64_t i = (int64_t)tile * 16 + s;
        const int ic = i < a.n ? (int)i : a.n - 1;
        // ---- input (attributes 4q + g): a sample that contributes nothing has zero input and delta
        float x[L::KA], d[L::KC];
        const bool live = enc_input<A, true>(a, rows, ic, g, x) && i < a.n;
        #pragma unroll
        for (int q = 0; q < L::KC; ++q) d[q] = a.dz[(int64_t)ic * C + 4 * q + g];
        #pragma unroll
        for (int q = 0; q < L::KA; ++q) {
            x[q] = live ? x[q] : 0.0f;
            table[(L::X + 4 * q + g) * kES + s] = x[q];
        }
        #pragma unroll
        for (int q = 0; q < L::KC; ++q) {
            d[q] = live ? d[q] : 0.0f;
            table[(L::D + 4 * q + g) * kES + s] = d[q];
        }
        // ---- forward
        float act[NHE][HE / 4];                // K step 4t + r: neuron 16t + 4r + g
        f32x4e acc[HT];
        #pragma unroll
        for (int k = 0; k < NHE; ++k) {
            #pragma unroll
            for (int u = 0; u < HT; ++u) acc[u] = *reinterpret_cast<const f32x4e*>(lds + L::BIAS + (k * HT + u) * 16 + 4 * g);
            if (k == 0) enc_layer<HT, L::KA>(lds + L::W1, x, acc, lane);
            else enc_layer<HT, L::KH>(lds + L::W2, act[0], acc, lane);
            #pragma unroll
            for (int j = 0; j < HE / 4; ++j) {
                act[k][j] = fmaxf(acc[j / 4][j % 4], 0.0f);
                table[(L::hid(k) + 4 * j + g) * kES + s] = act[k][j];
            }
        }
        lds_sync_wave();
        // ---- layers from the output down: weight gradient, then the deltas of the layer below
        go.add(table + L::D * kES, table + L::hid(NHE - 1) * kES, lane);
        float dh[HE / 4];
        #pragma unroll
        for (int k = NHE - 1; k >= 0; --k) {
            #pragma unroll
            for (int u = 0; u < HT; ++u) acc[u] = f32x4e{0.0f, 0.0f, 0.0f, 0.0f};
            if (k == NHE - 1) enc_layer<HT, L::KC>(lds + L::WOT, d, acc, lane);
            else enc_layer<HT, L::KH>(lds + L::W2T, dh, acc, lane);
            lds_sync_wave();                   // the gradient has read the activations
            #pragma unroll
            for (int j = 0; j < HE / 4; ++j) {
                dh[j] = act[k][j] > 0.0f ? acc[j / 4][j % 4] : 0.0f;
                table[(L::hid(k) + 4 * j + g) * kES + s] = dh[j];
            }
            lds_sync_wave();
            if (k == 0) g0.add(table + L::hid(0) * kES, table + L::X * kES, lane);
            else gh.add(table + L::hid(k) * kES, table + L::hid(0) * kES, lane);
        }
        lds_sync_wave();                       // the rows are free for the next tile
    }
    float* part = a.partial + (size_t)blockIdx.x * a.np;
    g0.store(lds, part + L::off(0), wave, lane);
    if (NHE == 2) gh.store(lds, part + L::off(1), wave, lane);
    go.store(lds, part + L::off(NHE), wave, lane);
}

// Four tiles per workgroup at least (backward: fewer slices); a small batch has a wave per SIMD on each CU.
int encoder_forward_grid(int64_t n, int cu_count) {
    const int64_t quads = (n + 63) / 64, most = (int64_t)cu_count * 5;
    return (int)(quads < most ? quads : most);
}

int encoder_backward_grid(int64_t n, int HE, int cu_count) {
    const int64_t quads = (n + 63) / 64, most = (int64_t)cu_count * (HE == 64 ? 1 : 2);
    return (int)(quads < most ? quads : most);
}

template <int A, int C, int HE, int NHE>
static hipError_t launch_encoder_shape(int mode, const EncoderArgs& a, int grid, hipStream_t s) {
    clear_stale_hip_error();
    if (mode == 0) encoder_forward_kernel<A, C, HE, NHE, false><<<grid, 64 * kEncFwdWaves, 0, s>>>(a);
    else if (mode == 1) encoder_forward_kernel<A, C, HE, NHE, true><<<grid, 64 * kEncFwdWaves, 0, s>>>(a);
    else encoder_backward_kernel<A, C, HE, NHE><<<grid, 64 * kEncWaves, 0, s>>>(a);
    return hipGetLastError();
}

bool encoder_shape_supported(int A, int C, int HE, int NHE) {
    return (A == 4 || A == 8 || A == 16) && (C == 8 || C == 16) && (HE == 16 || HE == 32 || HE == 64) &&
           (NHE == 1 || NHE == 2);
}

// mode 0: bake (rows), 1: query codes, 2: backward into a.partial (grid workgroups)
hipError_t launch_encoder(int A, int C, int HE, int NHE, int mode, const EncoderArgs& a, int grid, hipStream_t s) {
#define NAM_E_CASE(A_, C_, HE_, NHE_) \
    if (A == A_ && C == C_ && HE == HE_ && NHE == NHE_) return launch_encoder_shape<A_, C_, HE_, NHE_>(mode, a, grid, s);
#define NAM_E_H(A_, C_) NAM_E_CASE(A_, C_, 16, 1) NAM_E_CASE(A_, C_, 16, 2) NAM_E_CASE(A_, C_, 32, 1) \
    NAM_E_CASE(A_, C_, 32, 2) NAM_E_CASE(A_, C_, 64, 1) NAM_E_CASE(A_, C_, 64, 2)
    NAM_E_H(4, 8) NAM_E_H(4, 16) NAM_E_H(8, 8) NAM_E_H(8, 16) NAM_E_H(16, 8) NAM_E_H(16, 16)
#undef NAM_E_H
#undef NAM_E_CASE
    return hipErrorInvalidValue;
}

}  // namespace nam
