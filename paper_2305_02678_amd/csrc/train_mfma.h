// Differentiation of the decode on the gfx950 matrix cores:
// training by backpropagation into the decoder, the learned shading frames and directly into the
// latent texels (Sec. 5 and the direct optimisation of Sec. 2 "Obtaining latent textures").
//
// Work decomposition.  One workgroup of 8 waves per CU, two per SIMD: waves p and p + 4 (on the
// same SIMD) form a pair that walks its own 16-sample tiles.  The front wave fetches a tile, runs
// the forward pass and takes the deltas down through the layers, all in registers; the back wave
// contracts the weight gradients and, between the layers of the next tile, scatters the code's gradient
// into the texels.  Each layer's (deltas, inputs) pass from front to back through two 8 KiB slots of
// LDS per pair, so the back wave's matrix-core chains and atomics fill the front wave's latencies
// (taps, texels, softplus), and neither wave holds the other's registers.  The decoder's operand blocks sit in LDS, shared by the
// workgroup.
//
// Arithmetic.  FP32 matrix instructions and vector instructions take turns on a SIMD, so products of
// FP32 factors run on the FP16 matrix cores, each factor split into two FP16 halves as in the split
// decode (decode_split.h).  Weights have a power of two per layer (AW), the values of a sample one per
// layer, each of which puts their largest magnitude in [2^14, 2^15): nothing overflows, samples of any
// scale keep their 22 bits beside each other, and so do weights down to 2^-17 of a layer's largest.  Two
// halves lose the last bit of a quarter of the weights, a tie of the low half's rounding.  The loss would
// be the same for every sample and add up over them, so the odd workgroups hold the tie's other neighbour:
// the two errors are opposite (ALT).
//
// In a weight gradient, a sum over samples, every sample's inputs are multiplied by the power of two that brings its product to the
// scale 2^x of the accumulators; x follows the samples, and the back wave rescales its accumulators when
// it changes.  The factor is applied in FP16 and so not below 2^-12 (kFarStep): an input's low half
// keeps its bits down to 2^-5 of the sample's largest there, and loses 2^-28 of the largest below.  A
// sample further down would lose bits, or all of itself, also in the rows that no large sample touches
// (its inactive neurons'), so a tile whose samples span more than that hands the layer over once more
// for each 12 powers of two, with those samples alone and an x that is larger by as many.
//
// ReLUs.  A unit within rounding of its kink would fall on a side that depends on the arithmetic, and
// with it a sample's whole gradient.  A tile with such a unit (a pre-activation below 2^-19 of its
// sample's largest one in the layer; about 1% of tiles), or whose output is not finite, runs its forward
// pass again in FP32 (v_mfma_f32_16x16x4_f32) and takes activations and outputs from there.  The margin
// is a measured one: over 7 million units of random decoders the two arithmetics differ by 2^-20.4 of
// that largest one at most, mostly by 2^-23, and a ReLU changes side only where a rare difference meets a
// pre-activation smaller than itself; inputs that cancel to pre-activations far below their products may
// exceed it.  A unit without weights and bias (pruned, or not yet trained) is 0 in either arithmetic: its
// packed bias is NaN, which the comparisons pass over and the ReLU turns into its 0, so such units send
// no tile the long way.  An infinite weight sends all of them there.
//
// The FP32 sums have a fixed order.  Slot 4g + r of an accumulator's row tile holds neuron 4g + r or, in
// natural order, neuron 4r + g: then the K steps run over the neurons in ascending order, and as the
// instruction is a chain of four FMAs in ascending k, the sums are bit for bit those of the vector kernel
// (train_vec.h), whose shapes (learned frames, width 16, 1 or 4 hidden layers) keep that order.
//
// Layouts.  Lane (g, s) = (lane / 16, lane % 16) works on sample s of the tile.  A layer is Y = W X with
// the weights as the A operand (16 output rows per row tile) and one sample per column; its
// accumulator leaves lane (g, s) holding row slots 4g..4g+3 of each row tile, which are the next
// layer's B operand in place (the weights' K order is permuted when they are packed).  The backward
// products W^T delta read the same blocks transposed (W_1^T and W_out^T are packed).  The weight gradients
// dW = delta a^T take both operands from the slots, transposed by the LDS read (samples on the K
// index), and accumulate in registers over all tiles of the wave.  At the end each back wave writes
// its gradients to its own slice of a partial buffer, reduced in a fixed order afterwards, so
// parameter gradients do not depend on scheduling.
//
// Layer 1 input.  For the fetch, lane (g, s) loads channels 4g..4g+3 of the 8 trilinear taps of
// sample s (C = 16; for C = 8 lanes g < 2 load): K slots e = 0..3 of its lane group.  Slot 4 + j of
// group g holds direction input 4j + g; slot 7 of group 0 a constant 1 with no weight, which makes the
// bias gradient one more column of dW_1.  The FP32 forward's K slots (q, g) are slot_input's, where a
// constant-1 slot makes the bias part of the weights, or in natural order inputs 4q + g with the
// bias as the initial accumulator.
#pragma once

#include "decode_split.h"
#include "frames.h"
#include "latent_fetch.h"
#include "train_internal.h"

namespace nam {

typedef float f32x4 __attribute__((ext_vector_type(4)));

__device__ __forceinline__ f32x4 mfma_f32(float a, float b, f32x4 c) {
    return __builtin_amdgcn_mfma_f32_16x16x4f32(a, b, c, 0, 0, 0);
}

// Input index of layer-1 K slot (q, g) without natural order: 0..C-1 latent channels, C..C+5 the
// directions (wi x, y, z, wo x, y, z), C+6 the constant 1 (bias), -1 a zero slot.
template <int C>
__host__ __device__ constexpr int slot_input(int q, int g) {
    if (C == 16) {
        if (q < 4) return 4 * g + q;
        if (q == 4) return C + g;
        return g < 2 ? C + 4 + g : (g == 2 ? C + 6 : -1);
    }
    if (g < 2) return 4 * g + q;
    if (g == 2) return C + q;
    return q < 2 ? C + 4 + q : (q == 2 ? C + 6 : -1);
}

// A matrix of a slot: 16 samples x 64 columns of FP16 high halves, then of low ones.  The 8-byte groups
// (4 columns) of a sample are exchanged by the sample, so that the front wave's 8-byte writes (a
// sample's neurons) and the back wave's transposing 8-byte reads (ds_read_b64_tr_b16: 4 samples of 16
// neurons per lane group) both take two turns of all banks.  Byte offset of group c4 of sample s:
constexpr int kPlane = 16 * 64 * 2;
constexpr int kSlotMatrix = 2 * kPlane;
__device__ __forceinline__ int slot_group(int s, int c4) { return s * 128 + ((c4 ^ s) & 15) * 8; }

// A handoff: deltas, inputs, and per sample the weight of its deltas in the bias sums.
struct TmSlot {
    uint8_t delta[kSlotMatrix];
    uint8_t input[kSlotMatrix];
};
struct alignas(16) TmSlotScale {
    _Float16 bias_weight[16];
    int x, xb;                    // weight gradients are summed times 2^x, bias gradients times 2^xb
    int more;                     // the same layer of the same tile follows, with smaller samples
};
constexpr int kFarStep = 12, kFarSteps = 5;

// The decoder's operand blocks: FP32 blocks of the exact forward (read from memory by the forward
// kernel and by tiles that need it), then the part that the training kernel keeps in LDS.  Offsets in
// floats.  An FP32 block of 4 consecutive K steps is 64 lanes x 4 floats.  A block of halves is, per
// part (high, low, and split_parts' third), the A operand of one v_mfma_f32_16x16x32_f16: 64 lanes x 8
// halves, K slot (s, g, e) being slot 16 (2s + e / 4) + 4g + e % 4 of the previous layer's accumulator
// (decode_mfma.h); the operands of W_k^T are read out of the same blocks by transposing LDS reads.  W_out's blocks hold their first 8 rows only (32 x 16 bytes), W_out^T's are operands
// of v_mfma_f32_16x16x16_f16 (K slot 4g + e = output) of their first two lane groups (32 x 8 bytes).
template <int C, int H, int NH, int NF>
struct TrainLayout {
    static constexpr bool NAT = NF > 0 || H == 16 || NH == 1 || NH == 4;   // natural neuron order
    static constexpr int IN = C + 6 * (NF > 1 ? NF : 1);
    static constexpr int NP1 = 6 * NF * (C + 1);   // frame-layer parameters ahead of the decoder's
    static constexpr int HT = H / 16;              // row tiles of a hidden layer
    static constexpr int KS = (H + 31) / 32;       // K steps of 32 over a hidden layer
    static constexpr int P = split_parts(H);       // parts of a block after layer 1
    static constexpr int Q1 = NAT ? (IN + 3) / 4 : (C + 8) / 4;   // FP32 K steps of layer 1
    static constexpr int G1 = (Q1 + 3) / 4;        // groups of 4 K steps of layer 1
    static constexpr int NR1 = NF > 0 ? (IN + 15) / 16 : 1;       // row tiles of W_1^T delta_1
    static constexpr int FW1 = 0;                                  // [t'][grp][lane][4]
    static constexpr int FWH = FW1 + HT * G1 * 256;                // layers 2..NH: [t'][t][lane][4]
    static constexpr int WH_SZ = HT * HT * 256;
    static constexpr int FWO = FWH + (NH - 1) * WH_SZ;             // [t][lane][4], rows < NO
    static constexpr int BIAS = FWO + HT * 256;                    // layers 1..NH, output: [t][g][4]
    static constexpr int FF = BIAS + NH * HT * 16 + 16;            // frame layer: [channel / 4][lane]
    static constexpr int FFB = FF + (NF > 0 ? C / 4 * 64 : 0);     // its biases
    static constexpr int FWD = FFB + (NF > 0 ? 16 : 0);            // end of the forward kernel's part
    static constexpr int BF = FWD;                                 // frame layer transposed: [q][lane]
    static constexpr int AW = BF + (NF > 0 ? 3 * 64 : 0);          // exponents of the layers' weight scales (kNoExponent)
    static constexpr int BA = AW + 8;                              // BIAS times 2^AW, NaN for units without weights
    static constexpr int BLOCKS = BA + FF - BIAS;                  // blocks of halves
    static constexpr int A1 = BLOCKS;                              // [j][3 parts][256]
    static constexpr int AH = A1 + HT * 3 * 256;                   // [k][j][s][P][256]
    static constexpr int AH_SZ = HT * KS * P * 256;
    static constexpr int AO = AH + (NH - 1) * AH_SZ;               // [s][P][128]
    static constexpr int BO = AO + KS * P * 128;                   // W_out^T: [j][P][64]
    static constexpr int B1 = BO + HT * P * 64;                    // W_1^T: [u][s][P][256]
    static constexpr int END = B1 + NR1 * KS * P * 256;
    static constexpr int LDS_FLOATS = END - BIAS;                  // the training kernel's part
    static constexpr int ALT = P == 2 ? END - BLOCKS : 0;          // the odd workgroups' blocks lie this far on
    static constexpr int BLOB = END + ALT;
    static constexpr int XCH = NF > 0 ? 16 * 12 : 0;   // per front wave: values handed across lanes
    static_assert(BIAS % 4 == 0 && FWD % 4 == 0 && BLOCKS % 4 == 0 && BLOB % 4 == 0, "16-byte alignment of blocks");
};

// Neuron of row slot i of a row tile (an involution).
template <bool NAT>
__host__ __device__ constexpr int slot_neuron(int i) { return NAT ? 4 * (i & 3) + (i >> 2) : i; }

// Packed parameter offsets of the decoder (W_1[H][IN], b_1, W_k[H][H], b_k, ..., W_out[NO][H], b_out).
template <int IN, int H>
__host__ __device__ constexpr int param_off(int k) {   // k = 1 .. NH (hidden), NH + 1 output
    return k == 1 ? 0 : IN * H + H + (k - 2) * (H * H + H);
}

}  // namespace nam
