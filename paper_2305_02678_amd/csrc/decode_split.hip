// Host side of the split FP32 decode (decode_split.h): the scales and operand blocks of a
// material, prepared once when it is loaded, and the launch; the kernels of decoders without
// learned frames and albedo head are instantiated here.
#include "decode_split.h"

#include <cmath>
#include <cstring>
#include <vector>

namespace nam {

hipError_t dispatch_split(const MlpShape& sh, SplitArgs& a, int cu, hipStream_t s) {
    return dispatch_split_filter<false, false>(sh, a, cu, s);
}

// Largest |x| as float bits (NaN counts as the largest).
__global__ void __launch_bounds__(256) absmax_kernel(const uint4* __restrict__ p, int64_t count, unsigned int* __restrict__ out) {
    unsigned int m = 0;
    for (int64_t i = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; i < count; i += (int64_t)gridDim.x * blockDim.x) {
        const uint4 v = p[i];
        m = max(max(max(v.x & 0x7fffffffu, v.y & 0x7fffffffu), max(v.z & 0x7fffffffu, v.w & 0x7fffffffu)), m);
    }
    for (int o = 32; o > 0; o >>= 1) m = max(m, (unsigned int)__shfl_xor((int)m, o, 64));
    if ((threadIdx.x & 63) == 0) atomicMax(out, m);
}

// The largest power of two s with s x <= top (1 for x = 0).
static double scale_to(double top, double x) {
    int e = 0;
    if (!(x > 0.0)) return 1.0;
    (void)std::frexp(top / x, &e);
    return std::ldexp(1.0, e - 1);
}

static bool usable_scale(double s) { return s >= std::ldexp(1.0, -100) && s <= std::ldexp(1.0, 100); }

// Accumulators of this magnitude stay floats (weights far below their bias have a scale of their own).
static bool usable_sum(double s) { return s <= std::ldexp(1.0, 120); }

// FP16 of |x| < 32768, round to nearest even, and back.  (The host's _Float16 conversions are library
// calls, most of the time of packing a decoder of three layers of 64.)
static uint16_t half_bits(float x) {
    uint32_t u;
    std::memcpy(&u, &x, 4);
    const uint16_t sign = (uint16_t)((u >> 16) & 0x8000);
    const uint32_t a = u & 0x7fffffffu;
    if (a >= 0x38800000u)                       // normal, from 2^-14
        return sign | (uint16_t)((a + 0xfffu + ((a >> 13) & 1u) - 0x38000000u) >> 13);
    const float s = std::fabs(x) + 0.5f;        // its last place is 2^-24
    std::memcpy(&u, &s, 4);
    return sign | (uint16_t)(u - 0x3f000000u);
}

static float half_value(uint16_t h) {
    const uint32_t m = h & 0x7fff, u = (m << 13) + 0x38000000u;
    float v = (float)m * 0x1p-24f;
    if (m >= 0x400) std::memcpy(&v, &u, 4);
    return h & 0x8000 ? -v : v;
}

// The parts of v (a weight times a power of two), `stride` bytes apart.
static void put_parts(uint8_t* dst, size_t stride, int parts, float v) {
    for (int i = 0; i < parts; ++i) {
        const uint16_t h = half_bits(v);
        std::memcpy(dst + i * stride, &h, 2);
        v -= half_value(h);                     // exact
    }
}

// Bytes of the A blocks: layer 0 in three parts, the rest as split_parts has it.
static size_t split_block_offset(const MfmaLayout& lay, int H, int block) {
    const size_t b0 = std::min(block, lay.RT);
    return b0 * 3072 + (block - b0) * 1024 * split_parts(H);
}

// Largest |texel| of the material as float bits; `word`: four bytes of device memory.
static hipError_t texel_absmax(const nam_material* m, unsigned int* word, unsigned int* bits) {
    hipError_t e = hipMemset(word, 0, sizeof(unsigned int));
    if (e != hipSuccess) return e;
    clear_stale_hip_error();
    const int64_t count = m->texel_count * m->desc.channels / 4;
    const int blocks = (int)std::min<int64_t>(m->ctx->cu_count * 8, (count + 255) / 256);
    absmax_kernel<<<blocks, 256, 0, nullptr>>>(reinterpret_cast<const uint4*>(m->texels32), count, word);
    if ((e = hipGetLastError()) != hipSuccess) return e;
    return hipMemcpy(bits, word, sizeof(unsigned int), hipMemcpyDeviceToHost);
}

// Packs the decoder behind `dev`, which holds `host.size()` bytes; *packed tells whether it has scales.
static hipError_t pack_decode_split(nam_material* m, void* dev, std::vector<uint8_t>& host, bool* packed);

hipError_t prepare_decode_split(nam_material* m) {
    const MlpShape& sh = m->shape;
    // 32-bit byte offsets into the FP32 texels
    if (m->texel_count * sh.C * 4 >= (int64_t(1) << 32)) return hipSuccess;
    for (float p : m->host_params)
        if (!std::isfinite(p)) return hipSuccess;
    for (float p : m->host_frames)
        if (!std::isfinite(p)) return hipSuccess;
    const MfmaLayout lay = mfma_layout(sh.C, sh.H, sh.NH, true, false);
    std::vector<uint8_t> host(split_block_offset(lay, sh.H, lay.a_blocks()) + (size_t)lay.b_blocks() * 64 + (sh.NF ? 3 * 512 + 64 : 0), 0);
    // one allocation for the search of the largest texel and for the blocks: a load's allocations are most
    // of what it costs (a material of 64 x 64 x 8)
    void* dev = nullptr;
    hipError_t e = hipMalloc(&dev, host.size());
    if (e != hipSuccess) return e;
    bool packed = false;
    e = pack_decode_split(m, dev, host, &packed);
    if (e != hipSuccess || !packed) {
        (void)hipFree(dev);
        return e;
    }
    m->split = dev;
    m->split_bytes = host.size();
    return hipSuccess;
}

static hipError_t pack_decode_split(nam_material* m, void* dev, std::vector<uint8_t>& host, bool* packed) {
    const MlpShape& sh = m->shape;
    const int C = sh.C, NH = sh.NH, NO = sh.NO, rows_f = 6 * sh.NF;
    unsigned int bits = 0;
    hipError_t e = texel_absmax(m, static_cast<unsigned int*>(dev), &bits);
    if (e != hipSuccess) return e;
    float zmax;
    std::memcpy(&zmax, &bits, 4);
    if (!std::isfinite(zmax)) return hipSuccess;

    // Scales.  T: a layer's accumulator holds T times its pre-activation; S: its output's halves
    // hold S times its activation, S bound <= 2^15.  `err` follows the subnormal step of the low
    // halves (at most 2^-25 / S per value, independent over a row) to the output.
    // Directions: |T w| <= sqrt(3) max |w_i|; the same bound without frames, so that an identity
    // frame changes no bit.
    const double dirs = 1.75 * kSplitMaxDir;
    const MfmaLayout lay = mfma_layout(C, sh.H, NH, true, false);
    const int nB = lay.b_blocks();
    const size_t a_bytes = split_block_offset(lay, sh.H, lay.a_blocks());
    float* bias = reinterpret_cast<float*>(host.data() + a_bytes);
    // Codes and directions have scales of their own: codes far below the directions keep their bits (learned
    // frames normalise what they give).
    const double sz = std::min(scale_to(32768.0, (double)zmax), std::ldexp(1.0, 40)), sd = scale_to(32768.0, dirs);
    if (!usable_scale(sz)) return hipSuccess;
    double bound = 0.0, S = 1.0, err = 0.0;
    SplitScales sc{};
    sc.sz = (float)sz;
    sc.sd = (float)sd;
    size_t off = 0;
    for (int L = 0; L <= NH; ++L) {
        const int fi = m->dims[L], fo = m->dims[L + 1];
        const float* W = m->host_params.data() + off;
        const float* b = W + (size_t)fi * fo;
        off += (size_t)fi * fo + fo;
        const auto scale_in = [&](int j) { return L > 0 ? S : j < C ? sz : sd; };
        double wmax = 0.0, next = 0.0, step = 0.0, top_row[64] = {}, row_sum[64];
        double in_scale[64], in_bound[64], in_err[64];             // per input: 1 / scale, bound, error
        for (int j = 0; j < fi; ++j) {
            in_scale[j] = 1.0 / scale_in(j);
            in_bound[j] = L > 0 ? bound : j < C ? (double)zmax : dirs;
            in_err[j] = err + 0x1p-25 * in_scale[j];
        }
        for (int r = 0; r < fo; ++r) {
            double sum = std::fabs((double)b[r]), sq = 0.0;
            for (int j = 0; j < fi; ++j) {
                const double w = std::fabs((double)W[(size_t)r * fi + j]), e = w * in_err[j];
                top_row[r] = std::max(top_row[r], w * in_scale[j]);
                sum += w * in_bound[j];
                sq += e * e;
            }
            wmax = std::max(wmax, top_row[r]);
            next = std::max(next, sum);
            row_sum[r] = sum;
            step = std::max(step, std::sqrt(sq));
        }
        err = step;
        // every row of the output layer has a scale of its own (RGB does not depend on an albedo head)
        double T[64];
        for (int r = 0; r < fo; ++r) {
            T[r] = scale_to(1023.0, L == NH ? top_row[r] : wmax);
            if (!usable_scale(T[r]) || !usable_sum(T[r] * row_sum[r])) return hipSuccess;
        }
        const int rts = L < NH ? lay.RT : 1, kss = L == 0 ? 1 : lay.KS;
        for (int j = 0; j < rts; ++j) {
            for (int s = 0; s < kss; ++s) {
                uint8_t* blk = host.data() + split_block_offset(lay, sh.H, lay.a_index(L, j, s));
                for (int lane = 0; lane < 64; ++lane) {
                    const int row = 16 * j + lane % 16;
                    if (row >= fo) continue;
                    const double up = T[row] / scale_in(0), up_dirs = T[row] / scale_in(C);   // (the same past layer 0)
                    for (int x = 0; x < 8; ++x) {
                        int in = MfmaLayout::k_source(L, s, lane / 16, x);
                        int parts = L == 0 ? 3 : split_parts(sh.H);
                        if (L > 0 && sh.H == 16 && x >= 4) {
                            // slots past 16 inputs: the inputs' last bits, weighed by the high halves
                            in = MfmaLayout::k_source(L, s, lane / 16, x - 4);
                            parts = 1;
                        }
                        if (in < fi)
                            put_parts(blk + lane * 16 + 2 * x, 1024, parts,
                                      (float)((double)W[(size_t)row * fi + in] * (in < C ? up : up_dirs)));
                    }
                }
            }
            float* bb = bias + (size_t)lay.b_index(L, j) * 16;
            for (int i = 0; i < 16; ++i)
                if (16 * j + i < fo) bb[i] = (float)((double)b[16 * j + i] * T[16 * j + i]);
        }
        if (L < NH) {
            const double Sn = scale_to(32768.0, next);
            if (!usable_scale(Sn) || !usable_scale(Sn / T[0])) return hipSuccess;
            sc.c[L] = (float)(Sn / T[0]);
            S = Sn;
            bound = next;
        } else {
            for (int r = 0; r < NO; ++r) sc.oinv[r] = (float)(1.0 / T[r]);
        }
    }
    // a quarter of the rounding of an FP32 output near 1
    if (!(err <= std::ldexp(1.0, -26))) return hipSuccess;
    if (rows_f) {
        // a scale per vector (three rows), which its normalisation takes out again
        const float* W = m->host_frames.data();
        uint8_t* wf = host.data() + a_bytes + (size_t)nB * 64;
        float* fb = reinterpret_cast<float*>(wf + 3 * 512);
        double up[4], norm = 0.0;
        for (int v = 0; v < rows_f / 3; ++v) {
            double top = 0.0;
            for (int i = 3 * v * C; i < 3 * (v + 1) * C; ++i) top = std::max(top, std::fabs((double)W[i]));
            up[v] = scale_to(1023.0, top);
            if (!usable_scale(up[v]) || !usable_scale(up[v] * sz)) return hipSuccess;
            sc.finv[v] = (float)(1.0 / (up[v] * sz));
        }
        for (int r = 0; r < rows_f; ++r) {
            double sq = 0.0;
            for (int c = 0; c < C; ++c) sq += (double)W[r * C + c] * W[r * C + c];
            norm = std::max(norm, std::sqrt(sq));
            // (no row of weights sums to more than C times its norm)
            if (!usable_sum(up[r / 3] * sz * (std::fabs((double)W[rows_f * C + r]) + C * std::sqrt(sq) * zmax))) return hipSuccess;
            fb[r] = (float)((double)W[rows_f * C + r] * (up[r / 3] * sz));
        }
        for (int lane = 0; lane < 64; ++lane)
            for (int x = 0; x < 4; ++x) {
                const int r = lane % 16, ch = 4 * (lane / 16) + x;
                if (r < rows_f && ch < C) put_parts(wf + lane * 8 + 2 * x, 512, 3, (float)((double)W[r * C + ch] * up[r / 3]));
            }
        // The subnormal step of a code's low halves, 2^-25 / sz per channel, moves a vector by about
        // 2^-25 norm / sz, as much again for the weights': at this length by an FP32 rounding.
        const double shortest = 2.0 * norm / sz;
        sc.shortest2 = (float)std::min(shortest * shortest, 1e38);
    }
    if ((e = hipMemcpy(dev, host.data(), host.size(), hipMemcpyHostToDevice)) != hipSuccess) return e;
    m->split_scales = sc;
    *packed = true;
    return hipSuccess;
}

hipError_t launch_decode_split(const nam_material* m, int64_t n, const float* uv, const float* lod, const float* xi,
                               const float* wi, const float* wo, float* rgb, hipStream_t st) {
    if (n <= 0) return hipSuccess;
    if (!m->split || n > (int64_t(1) << 30)) return hipErrorInvalidValue;
    const MfmaLayout lay = mfma_layout(m->shape.C, m->shape.H, m->shape.NH, true, false);
    const char* base = static_cast<const char*>(m->split);
    SplitArgs a{};
    a.pyr = m->pyr();
    a.tex = m->texels32;
    a.w = reinterpret_cast<const uint4*>(base);
    base += split_block_offset(lay, m->shape.H, lay.a_blocks());
    a.bias = reinterpret_cast<const floatx4*>(base);
    base += (size_t)lay.b_blocks() * 64;
    a.wf = reinterpret_cast<const half4*>(base);
    a.fbias = reinterpret_cast<const floatx4*>(base + 3 * 512);
    const SplitScales& sc = m->split_scales;
    a.one = 1.0f;
    a.sz = sc.sz;
    a.sd = sc.sd;
    std::copy(sc.finv, sc.finv + 4, a.finv);
    a.shortest2 = sc.shortest2;
    for (int k = 0; k < kMaxLayers; ++k) a.c[k] = 0.5f * sc.c[k];
    std::copy(sc.oinv, sc.oinv + 6, a.oinv);
    a.n = (int)n;
    a.nchunks = (int)((n + kChunk - 1) / kChunk);
    a.nf = m->shape.NF;
    a.uv = reinterpret_cast<const float2*>(uv);
    a.lod = lod;
    a.xi = xi;
    a.wi = wi;
    a.wo = wo;
    a.rgb = rgb;
    a.wt32 = m->wt32;
    a.frames32 = m->frames32;
    const int cu = m->ctx->cu_count;
    if (m->shape.NF) return m->shape.NO == 6 ? dispatch_split_frames_albedo(m->shape, a, cu, st) : dispatch_split_frames(m->shape, a, cu, st);
    return m->shape.NO == 6 ? dispatch_split_albedo(m->shape, a, cu, st) : dispatch_split(m->shape, a, cu, st);
}

}  // namespace nam
