// Differentiation of the decode on the gfx950 matrix cores (FP32 v_mfma_f32_16x16x4_f32):
// training by backpropagation into the decoder, the learned shading frames and directly into the
// latent texels (Sec. 5 and the direct optimisation of Sec. 2 "Obtaining latent textures").
//
// Work decomposition.  One workgroup of 8 waves per CU, two per SIMD: waves p and p + 4 (on the
// same SIMD) form a pair that walks its own 16-sample tiles.  The front wave fetches a tile, runs
// the forward pass and takes the deltas down through the layers, all in registers, and scatters the
// code's gradient into the texels; the back wave contracts the weight gradients.  Each layer's
// (deltas, inputs) pass from front to back through two 8 KiB slots of LDS per pair, so the back
// wave's matrix-core chains fill the front wave's latencies (taps, texels, atomics, softplus), and
// neither wave holds the other's registers (one wave doing both needs 428 + 72, a single wave per
// SIMD).  The decoder's operand blocks (below) sit in LDS, shared by the workgroup.
//
// Lane (g, s) = (lane / 16, lane % 16) works on sample s of the tile.  A layer is Y = W X with the
// weights as the A operand (16 output rows per row tile) and one sample per column; its accumulator
// leaves lane (g, s) holding row slots 4g..4g+3 of each row tile.  The next layer takes K steps (t, r)
// = {slots 16t + 4g + r : g = 0..3}, so the accumulator registers [t][r] are exactly its B operands:
// the weights' K order is permuted when they are packed, and no activation moves between lanes.
// Slot 4g + r of a row tile holds neuron 4g + r or, in natural order, neuron 4r + g: then the K steps
// run over the neurons in ascending order, and as the instruction is a chain of four FMAs in
// ascending k, a layer's sums are bit for bit those of the vector kernel (train_vec.h), whose shapes
// (learned frames, width 16, 1 or 4 hidden layers) it took over: no ReLU changes side.
// The backward products W^T delta use the same trick with the packed transposes.  The weight
// gradients dW = delta a^T contract over the samples: both operands are read from the slots with
// samples on the K index and accumulate in registers over all tiles of the wave.  At the end each
// back wave writes its gradients to its own slice of a partial buffer, reduced in a fixed order
// afterwards, so parameter gradients do not depend on scheduling.
//
// Layer 1 input.  For the fetch, lane (g, s) loads channels 4g..4g+3 of the 8 trilinear taps of
// sample s (C = 16; for C = 8 lanes g < 2 load).  Without natural order those registers become the
// K slots (q, g) of layer 1 directly (slot_input; for C = 8 lanes g >= 2 carry the directions), and
// a constant-1 slot makes the bias part of the weights; in natural order they are transposed across
// the four lane groups and the bias is the initial accumulator.  Either way a constant-1 column of
// the input makes the bias gradient one more column of dW_1.
#pragma once

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

// A slot matrix holds 16 samples x 64 columns, 16 floats of padding every 4 samples and the 16-byte
// groups of a 16-column tile exchanged by the sample: the 16-byte writes (a sample's neurons) and the
// 4-byte reads (a neuron's samples) touch every bank once, and the column tile is an immediate offset.
constexpr int kSlotMatrix = 16 * 64 + 3 * 16;
__device__ __forceinline__ int slot_at(int s, int n) {
    return s * 64 + (s >> 2) * 16 + (n & ~15) + ((((n >> 2) ^ s) & 3) << 2) + (n & 3);
}

// Operand blocks of the decoder in LDS (floats).  A block of 4 consecutive K steps is 64 lanes x 4
// floats, one 16-byte read per lane.
template <int C, int H, int NH, int NF>
struct TrainLayout {
    static constexpr bool NAT = NF > 0 || H == 16 || NH == 1 || NH == 4;   // natural neuron order
    static constexpr int IN = C + 6 * (NF > 1 ? NF : 1);
    static constexpr int NP1 = 6 * NF * (C + 1);   // frame-layer parameters ahead of the decoder's
    static constexpr int HT = H / 16;              // row tiles of a hidden layer
    static constexpr int Q1 = NAT ? (IN + 3) / 4 : (C + 8) / 4;   // K steps of layer 1
    static constexpr int G1 = (Q1 + 3) / 4;        // groups of 4 K steps of layer 1
    static constexpr int NCT1 = (IN + 16) / 16;    // column tiles of dW_1 (inputs, 1, padding)
    static constexpr int NR1 = NF > 0 ? (IN + 15) / 16 : 1;       // row tiles of W_1^T delta_1
    static constexpr int FW1 = 0;                                  // [t'][grp][lane][4]
    static constexpr int FWH = FW1 + HT * G1 * 256;                // layers 2..NH: [t'][t][lane][4]
    static constexpr int WH_SZ = HT * HT * 256;
    static constexpr int FWO = FWH + (NH - 1) * WH_SZ;             // [t][lane][4], rows < NO
    static constexpr int BIAS = FWO + HT * 256;                    // layers 1..NH, output: [t][g][4]
    static constexpr int FF = BIAS + NH * HT * 16 + 16;            // frame layer: [channel / 4][lane]
    static constexpr int FFB = FF + (NF > 0 ? C / 4 * 64 : 0);     // its biases
    static constexpr int FWD = FFB + (NF > 0 ? 16 : 0);            // end of the forward part
    static constexpr int NKO = NF > 0 ? 3 : 4;                     // K steps of W_out^T (outputs 4g + r)
    static constexpr int BWO = FWD;                                // W_out^T: [t'][r][lane]
    static constexpr int BWH = BWO + HT * NKO * 64;                 // W_k^T, k = 2..NH: [t'][t][lane][4]
    static constexpr int BW1 = BWH + (NH - 1) * WH_SZ;             // W_1^T: [u][t][lane][4]
    static constexpr int BF = BW1 + NR1 * HT * 256;                // frame layer transposed: [q][lane]
    static constexpr int BLOB = BF + (NF > 0 ? 3 * 64 : 0);
    static constexpr int SLOT = 2 * kSlotMatrix;   // deltas, inputs
    static constexpr int XCH = NF > 0 ? 16 * 12 : 0;   // per front wave: values handed across lanes
    static constexpr int LDS_FLOATS = BLOB + 4 * (2 * SLOT + XCH);
    static constexpr bool FITS = LDS_FLOATS * 4 + 16 * 16 + 64 <= 160 * 1024;
    static_assert(FWD % 4 == 0 && BLOB % 4 == 0, "16-byte alignment of blocks");
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
