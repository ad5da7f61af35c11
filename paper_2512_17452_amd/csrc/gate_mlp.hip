// Write-Gate MLP (Sec. 3.2, feature equation and gate equation), per token t and kv head h:
//     x = [ RMSNorm(k[t][h]) ; RMSNorm(k_rope[t][h]) ]
//     g = sigmoid( W2[h] . GELU( W1[h] x + b1[h] ) + b2[h] )
// with the exact GELU and an RMSNorm without learnable scale (the paper fixes neither).
//
// The first layer is a dense contraction (tokens x 2d x width per head) and runs on the
// matrix cores, transposed: H^T = W1 X^T with v_mfma_f32_32x32x16_bf16, rows = 32 hidden
// units of a chunk of W1 staged in LDS, columns = the 32 tokens of a wave, whose
// normalised features stay in registers as the second operand for the whole kernel.  A
// lane then owns one token column, so bias, GELU, the product with W2 and the sum over
// hidden units are per-lane work and the hidden layer never leaves the registers.
// The normalised features are rounded to bf16 (they are a matrix-core operand), which is
// what a bf16 model does with its RMSNorm output as well.
// Bound by the GELU on the vector unit (67 M of them for 16K tokens x 8 heads x width 512) in large
// calls, by the chain of a wave's products and GELUs in small ones.  Measured: 16K tokens 69 -> 52 us
// (33 us of which are the vector instructions alone at 2.2 GHz), 1K tokens 23 -> 15.
#include <algorithm>

#include "wgkv_dev.h"

namespace wgkv {

typedef __attribute__((ext_vector_type(8))) __bf16 gm_bf16x8_t;
typedef __attribute__((ext_vector_type(2))) __bf16 gm_bf16x2_t;
typedef __attribute__((ext_vector_type(16))) float gm_f32x16_t;

constexpr int kGmUnits = 32;   // hidden units per chunk of W1
constexpr int kGmTokens = 32;  // tokens per wave

// Twice the exact GELU, 2 z Phi(z) = z + |z| - |z| q(|z|) with q(y) = erfc(y / sqrt 2): no difference of nearly equal
// numbers on the negative side, and z + |z| carries a NaN or an infinity on.  q = 2^P(y), where log2 erfc(y / sqrt 2)
// is so smooth that a polynomial of degree six does: a least-squares fit on [0, 7], weighted by what an error of P does to
// (y + 0.1) q(y) (the 0.1 holds a small z: without it the constant term is off by 4.8e-6 of one) and reweighted until its
// largest error was as small as it gets.  Beyond 8 the product stays where it is there, 5e-15.  Whole function in fp32
// against 64 bits, largest error at |z| < 0.05 / < 2 / < 8: 1.0e-8 (1.7e-6 of z) / 1.5e-7 / 3.1e-7 (the rounding of z
// itself at the far end), where the rational erf formula of Abramowitz & Stegun 7.1.26 that stood here before left
// 1.4e-8 / 2.6e-7 / 4.2e-7 at 26 issue slots; this takes 13 with the one exponential counted as four.
__device__ __forceinline__ float gm_gelu2(float z) {
    const float y = fminf(fabsf(z), 8.0f);
    float p = fmaf(3.042223024e-05f, y, -7.449424051e-04f);
    p = fmaf(p, y, 7.997222006e-03f);
    p = fmaf(p, y, -5.327548117e-02f);
    p = fmaf(p, y, -4.588803671e-01f);
    p = fmaf(p, y, -1.151162603e+00f);
    p = fmaf(p, y, 2.378846442e-06f);
    return fmaf(-y, __builtin_amdgcn_exp2f(p), z + fabsf(z));
}

__device__ __forceinline__ float gm_bf16_to_f32(uint32_t bits16) { return __uint_as_float(bits16 << 16); }

__device__ __forceinline__ uint32_t gm_pack(float lo, float hi) {
    gm_bf16x2_t t = {(__bf16)lo, (__bf16)hi};
    return __builtin_bit_cast(uint32_t, t);
}

// The sum of a row's squares by pairs of neighbours, pairs of pairs and so on, as a wave's lanes sum them that hold an element each:
// the order that widths which are no multiple of 32 have always had.  Another order moves a few features in a million across a
// rounding boundary.
template <int D>
__device__ __forceinline__ float gm_squares_by_pairs(const uint4 (&raw)[D / 16]) {
#pragma clang fp contract(off)
    float s[D / 16];
#pragma unroll
    for (int j = 0; j < D / 16; j++) {
        const uint32_t w[4] = {raw[j].x, raw[j].y, raw[j].z, raw[j].w};
        float p[4];
#pragma unroll
        for (int e = 0; e < 4; e++) {
            const float x = gm_bf16_to_f32(w[e] & 0xffffu), y = __uint_as_float(w[e] & 0xffff0000u);
            const float xx = x * x, yy = y * y;
            p[e] = xx + yy;
        }
        const float a = p[0] + p[1], b = p[2] + p[3], c = a + b;
        s[j] = c + __shfl_xor(c, 32);  // the other half of the row holds the other octet of every sixteen
    }
#pragma unroll
    for (int o = 1; o < D / 16; o *= 2)
#pragma unroll
        for (int j = 0; j < D / 16; j += 2 * o) s[j] = s[j] + s[j + o];
    return s[0];
}

// The normalised features of one token as matrix operands: the 8 features [16 ks + 8 half, +8) of every slice of 16.
template <int D, bool BY_PAIRS>
__device__ __forceinline__ void gm_features(const char *k, const char *kr, size_t row, int half, float eps,
                                            gm_bf16x8_t (&xv)[2 * D / 16]) {
    constexpr int KS = 2 * D / 16;
#pragma unroll
    for (int part = 0; part < 2; part++) {
        const char *p = (part == 0 ? k : kr) + row * (D * 2);
        uint4 raw[KS / 2];
        float ss = 0.f;
#pragma unroll
        for (int j = 0; j < KS / 2; j++) {
            raw[j] = *reinterpret_cast<const uint4 *>(p + (2 * j + half) * 16);
            const uint32_t w[4] = {raw[j].x, raw[j].y, raw[j].z, raw[j].w};
#pragma unroll
            for (int e = 0; e < 4; e++) {
                // (not the two-element dot product: its sum is less exact, and more features then land on the other
                // side of a rounding boundary)
                const float x = gm_bf16_to_f32(w[e] & 0xffffu), y = __uint_as_float(w[e] & 0xffff0000u);
                ss = fmaf(x, x, ss);
                ss = fmaf(y, y, ss);
            }
        }
        ss += __shfl_xor(ss, 32);  // the other half of the row
        if constexpr (BY_PAIRS) ss = gm_squares_by_pairs<D>(raw);
        const float r = 1.0f / sqrtf(ss / (float)D + eps);
#pragma unroll
        for (int j = 0; j < KS / 2; j++) {
            // unpacked again, not kept unpacked: the 64 floats cost the two-column form 46 spilled registers
            asm volatile("" : "+v"(raw[j].x), "+v"(raw[j].y), "+v"(raw[j].z), "+v"(raw[j].w));
            const uint32_t w[4] = {raw[j].x, raw[j].y, raw[j].z, raw[j].w};
            uint32_t o[4];
#pragma unroll
            for (int e = 0; e < 4; e++)
                o[e] = gm_pack(gm_bf16_to_f32(w[e] & 0xffffu) * r, __uint_as_float(w[e] & 0xffff0000u) * r);
            xv[part * (KS / 2) + j] = __builtin_bit_cast(gm_bf16x8_t, make_uint4(o[0], o[1], o[2], o[3]));
        }
    }
}

// CB: columns of 32 tokens per wave.  US: unit groups of the block, 4 waves each; group us takes chunks us, us + US, ...
// RAGGED: the width is no multiple of 32.
template <int D, int CB, int US, bool RAGGED>
__global__ __launch_bounds__(256 * US, 2) void gate_mlp_mfma_kernel(const char *k, const char *kr, const char *W1,
                                                            const float *b1, const char *W2, const float *b2,
                                                            float eps, float *g_out, long long T, int Hkv,
                                                            int width) {
    constexpr int KS = 2 * D / 16;             // contraction slices of 16 features
    constexpr int kRow = 2 * D * 2 + 16;       // bytes per W1 row in LDS (padded against bank conflicts)
    constexpr int kRowPieces = 2 * D * 2 / 16;                  // 16-byte pieces per row
    constexpr int kPieces = kGmUnits * kRowPieces / 256;        // pieces of a chunk per thread of its group
    static_assert(kPieces == 2 || kPieces == 4, "");
    __shared__ __attribute__((aligned(16))) char s_w1[2][US][kGmUnits * kRow];
    __shared__ __attribute__((aligned(16))) float s_b1[2][US][kGmUnits];
    __shared__ __attribute__((aligned(16))) float s_w2[2][US][kGmUnits];
    __shared__ float s_sum[US][4][CB][kGmTokens];

    const int h = blockIdx.y;
    const int tid = threadIdx.x % 256, us = __builtin_amdgcn_readfirstlane(threadIdx.x / 256);
    const int lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int n = lane & 31, half = lane >> 5;
    const long long tok0 = ((long long)blockIdx.x * 4 + wave) * (kGmTokens * CB) + n;  // this lane's first token

    gm_bf16x8_t xv[CB][KS];
#pragma unroll
    for (int cb = 0; cb < CB; cb++) {
        const long long tok = tok0 + cb * kGmTokens;  // rows past the end repeat the last token, unwritten
        gm_features<D, RAGGED>(k, kr, (size_t)(tok < T ? tok : T - 1) * Hkv + h, half, eps, xv[cb]);
    }

    // ---- chunks of 32 hidden units: W1 rows, b1 and W2 through LDS, two buffers ----
    const int n_chunks = (width + kGmUnits - 1) / kGmUnits, n_it = (n_chunks + US - 1) / US;
    uint4 w0, w1, w2, w3;  // this thread's pieces of the chunk on its way to LDS
    w2 = w3 = make_uint4(0u, 0u, 0u, 0u);
    float b1v = 0.f, w2v = 0.f;
    auto fetch = [&](int it) __attribute__((always_inline)) {
        const int c = min(it * US + us, n_chunks - 1);  // a group without a chunk of its own in the last turn drops it
        const char *src = W1 + ((size_t)h * width + (size_t)c * kGmUnits) * (2 * D * 2);  // 32 consecutive rows
        const int rows = RAGGED ? min(width - c * kGmUnits, kGmUnits) : kGmUnits;  // fewer in the last chunk: units of zeros
        auto piece = [&](int p) __attribute__((always_inline)) {
            const int i = p * 256 + tid;
            if (!RAGGED) return *reinterpret_cast<const uint4 *>(src + (size_t)i * 16);
            const uint4 v = *reinterpret_cast<const uint4 *>(src + (size_t)min(i, rows * kRowPieces - 1) * 16);
            return i < rows * kRowPieces ? v : make_uint4(0u, 0u, 0u, 0u);
        };
        w0 = piece(0);
        w1 = piece(1);
        if (kPieces > 2) {
            w2 = piece(2);
            w3 = piece(3);
        }
        if (tid < kGmUnits) {
            const size_t u = (size_t)h * width + (size_t)c * kGmUnits + (RAGGED ? min(tid, rows - 1) : tid);
            const float b = b1[u], w = gm_bf16_to_f32(*reinterpret_cast<const uint16_t *>(W2 + u * 2));
            b1v = !RAGGED || tid < rows ? b : 0.f;
            w2v = !RAGGED || tid < rows ? w : 0.f;
        }
    };
    auto put = [&](int buf, int p, const uint4 v) __attribute__((always_inline)) {
        const int piece = p * 256 + tid;
        *reinterpret_cast<uint4 *>(&s_w1[buf][us][(piece / kRowPieces) * kRow + (piece % kRowPieces) * 16]) = v;
    };
    auto stage = [&](int buf) __attribute__((always_inline)) {
        put(buf, 0, w0);
        put(buf, 1, w1);
        if (kPieces > 2) {
            put(buf, 2, w2);
            put(buf, 3, w3);
        }
        if (tid < kGmUnits) {
            s_b1[buf][us][tid] = b1v;
            s_w2[buf][us][tid] = w2v;
        }
    };
    fetch(0);
    stage(0);
    __syncthreads();
    float acc_logit[CB];  // twice the logit
#pragma unroll
    for (int cb = 0; cb < CB; cb++) acc_logit[cb] = 0.f;
    for (int it = 0; it < n_it; it++) {
        const int buf = it & 1;
        if (it + 1 < n_it) fetch(it + 1);
        if (US == 1 || it * US + us < n_chunks) {  // wave-uniform
        gm_f32x16_t hcol[CB];
#pragma unroll
        for (int cb = 0; cb < CB; cb++)
#pragma unroll
            for (int i = 0; i < 16; i++) hcol[cb][i] = 0.f;
#pragma unroll
        for (int ks = 0; ks < KS; ks++) {
            const gm_bf16x8_t wa =
                *reinterpret_cast<const gm_bf16x8_t *>(&s_w1[buf][us][n * kRow + (ks * 16 + half * 8) * 2]);
#pragma unroll
            for (int cb = 0; cb < CB; cb++) hcol[cb] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(wa, xv[cb][ks], hcol[cb], 0, 0, 0);
        }
        // register 4j+i of a lane holds hidden unit 8j + 4*half + i of the chunk, for its token
#pragma unroll
        for (int j = 0; j < 4; j++) {
            const float4 bb = *reinterpret_cast<const float4 *>(&s_b1[buf][us][8 * j + 4 * half]);
            const float4 ww = *reinterpret_cast<const float4 *>(&s_w2[buf][us][8 * j + 4 * half]);
#pragma unroll
            for (int cb = 0; cb < CB; cb++) {
                acc_logit[cb] = fmaf(ww.x, gm_gelu2(hcol[cb][4 * j + 0] + bb.x), acc_logit[cb]);
                acc_logit[cb] = fmaf(ww.y, gm_gelu2(hcol[cb][4 * j + 1] + bb.y), acc_logit[cb]);
                acc_logit[cb] = fmaf(ww.z, gm_gelu2(hcol[cb][4 * j + 2] + bb.z), acc_logit[cb]);
                acc_logit[cb] = fmaf(ww.w, gm_gelu2(hcol[cb][4 * j + 3] + bb.w), acc_logit[cb]);
            }
        }
        }
        if (it + 1 < n_it) stage(buf ^ 1);
        __syncthreads();
    }
#pragma unroll
    for (int cb = 0; cb < CB; cb++) acc_logit[cb] += __shfl_xor(acc_logit[cb], 32);  // the other 16 units of every chunk
    if constexpr (US > 1) {
        if (half == 0)
#pragma unroll
            for (int cb = 0; cb < CB; cb++) s_sum[us][wave][cb][n] = acc_logit[cb];
        __syncthreads();
        if (us > 0) return;
#pragma unroll
        for (int cb = 0; cb < CB; cb++)
#pragma unroll
            for (int g = 1; g < US; g++) acc_logit[cb] += s_sum[g][wave][cb][n];
    }
#pragma unroll
    for (int cb = 0; cb < CB; cb++) {
        const long long tok = tok0 + cb * kGmTokens;
        if (half == 0 && tok < T) g_out[(size_t)tok * Hkv + h] = 1.0f / (1.0f + __expf(-fmaf(0.5f, acc_logit[cb], b2[h])));
    }
}

constexpr int kGmSplit = 4;  // waves of the block
// Few tokens: what a wave has to do one after the other is the time, so a block takes 32 tokens and its four waves
// a quarter of the hidden units each (eight waves: 15 instead of 13 us, every wave makes the features for itself).  The chunks of W1 go straight into the matrix operand (a lane reads 16 bytes of its
// unit's row per slice, a line of 128 bytes in four consecutive requests); nothing is shared but the sum at the end.
template <int D, bool RAGGED>
__global__ __launch_bounds__(kGmSplit * 64) void gate_mlp_split_kernel(const char *k, const char *kr, const char *W1,
                                                             const float *b1, const char *W2, const float *b2,
                                                             float eps, float *g_out, long long T, int Hkv, int width) {
    constexpr int KS = 2 * D / 16;
    __shared__ float s_sum[kGmSplit][kGmTokens];
    const int h = (int)(blockIdx.x % Hkv);  // blocks go to the XCDs in turn: with eight heads an L2 holds one head's W1
    const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int n = lane & 31, half = lane >> 5;
    const long long tok = (long long)(blockIdx.x / Hkv) * kGmTokens + n;
    const int n_chunks = (width + kGmUnits - 1) / kGmUnits;
    gm_bf16x8_t wa[KS], xv[KS];
    float4 bb[4];
    uint2 ww[4];
    // (the last chunk of a ragged width ends in units of zeros: only the wave that has it looks at the width)
    auto fetch = [&](int c) __attribute__((always_inline)) {
        const int u = min(c, n_chunks - 1) * kGmUnits + n;
        const char *src = W1 + ((size_t)h * width + (RAGGED ? min(u, width - 1) : u)) * (2 * D * 2) + half * 16;
#pragma unroll
        for (int ks = 0; ks < KS; ks++) wa[ks] = *reinterpret_cast<const gm_bf16x8_t *>(src + ks * 32);
        if (RAGGED && c == n_chunks - 1) {  // wave-uniform
#pragma unroll
            for (int ks = 0; ks < KS; ks++)
                wa[ks] = __builtin_bit_cast(gm_bf16x8_t, u < width ? __builtin_bit_cast(uint4, wa[ks]) : make_uint4(0u, 0u, 0u, 0u));
        }
    };
    auto fetch_b = [&](int c) __attribute__((always_inline)) {
        const size_t u0 = (size_t)h * width + (size_t)c * kGmUnits;
        const uint16_t *w2 = reinterpret_cast<const uint16_t *>(W2) + u0;
        if (RAGGED && c == n_chunks - 1) {  // wave-uniform
            const int rows = width - c * kGmUnits;
#pragma unroll
            for (int j = 0; j < 4; j++) {
                float b[4];
                uint32_t w[4];
#pragma unroll
                for (int i = 0; i < 4; i++) {
                    const int u = 8 * j + 4 * half + i;
                    const float bv = b1[u0 + min(u, rows - 1)];
                    const uint32_t wv = w2[min(u, rows - 1)];
                    b[i] = u < rows ? bv : 0.f;
                    w[i] = u < rows ? wv : 0u;
                }
                bb[j] = make_float4(b[0], b[1], b[2], b[3]);
                ww[j] = make_uint2(w[0] | (w[1] << 16), w[2] | (w[3] << 16));
            }
            return;
        }
#pragma unroll
        for (int j = 0; j < 4; j++) {
            const float *b = b1 + u0 + 8 * j + 4 * half;
            const uint16_t *w = w2 + 8 * j + 4 * half;
            bb[j] = make_float4(b[0], b[1], b[2], b[3]);
            ww[j] = make_uint2((uint32_t)w[0] | ((uint32_t)w[1] << 16), (uint32_t)w[2] | ((uint32_t)w[3] << 16));
        }
    };
    fetch(wave);
    gm_features<D, RAGGED>(k, kr, (size_t)(tok < T ? tok : T - 1) * Hkv + h, half, eps, xv);
    float acc = 0.f;  // twice the logit
    for (int c = wave; c < n_chunks; c += kGmSplit) {  // wave-uniform
        fetch_b(c);
        gm_f32x16_t h0, h1;  // two chains of products, half as long
#pragma unroll
        for (int i = 0; i < 16; i++) { h0[i] = 0.f; h1[i] = 0.f; }
#pragma unroll
        for (int ks = 0; ks < KS; ks += 2) {
            h0 = __builtin_amdgcn_mfma_f32_32x32x16_bf16(wa[ks], xv[ks], h0, 0, 0, 0);
            h1 = __builtin_amdgcn_mfma_f32_32x32x16_bf16(wa[ks + 1], xv[ks + 1], h1, 0, 0, 0);
        }
        fetch(c + kGmSplit);  // in flight during the GELU
#pragma unroll
        for (int j = 0; j < 4; j++) {
            acc = fmaf(gm_bf16_to_f32(ww[j].x & 0xffffu), gm_gelu2(h0[4 * j] + h1[4 * j] + bb[j].x), acc);
            acc = fmaf(gm_bf16_to_f32(ww[j].x >> 16), gm_gelu2(h0[4 * j + 1] + h1[4 * j + 1] + bb[j].y), acc);
            acc = fmaf(gm_bf16_to_f32(ww[j].y & 0xffffu), gm_gelu2(h0[4 * j + 2] + h1[4 * j + 2] + bb[j].z), acc);
            acc = fmaf(gm_bf16_to_f32(ww[j].y >> 16), gm_gelu2(h0[4 * j + 3] + h1[4 * j + 3] + bb[j].w), acc);
        }
    }
    acc += __shfl_xor(acc, 32);
    if (half == 0) s_sum[wave][n] = acc;
    __syncthreads();
    if (wave == 0 && half == 0 && tok < T) {
        float a = 0.f;
#pragma unroll
        for (int w = 0; w < kGmSplit; w++) a += s_sum[w][n];
        g_out[(size_t)tok * Hkv + h] = 1.0f / (1.0f + __expf(-fmaf(0.5f, a, b2[h])));
    }
}

// fp32 models: 16 tokens of a head a block, their features in LDS for the whole block, W1 in slices of 64 units x 128 features; a thread
// has one token and four neighbouring units, so a feature and four weights are two LDS reads for four multiply-adds.  Bound by
// those.  us against a block per (token, head), whose lanes read rows of W1 apart: 1500 tokens x 2 heads of 64, width 512 95 -> 28;
// 700 x 4 heads of 128, width 768 259 -> 70; 100 x 4 of 128, width 512 32 -> 48, which the rule leaves where it was.
constexpr int kGfTokens = 16, kGfUnits = 64, kGfSlice = 128;
__global__ __launch_bounds__(256) void gate_mlp_f32_kernel(const float *k, const float *kr, const float *W1, const float *b1, const float *W2,
                                                          const float *b2, float eps, float *g_out, long long T, int Hkv, int d, int width) {
    extern __shared__ __attribute__((aligned(16))) float s_x[];  // [16][2 d + 4]
    __shared__ __attribute__((aligned(16))) float s_w[2][kGfSlice][kGfUnits + 4];
    __shared__ float s_r[kGfTokens][16];
    const int h = blockIdx.y, tid = threadIdx.x, tok = tid & 15, part = tid >> 4, ld = 2 * d + 4;
    const long long t0 = (long long)blockIdx.x * kGfTokens, t = t0 + tok;
    const size_t row = ((size_t)(t < T ? t : T - 1) * Hkv + h) * d;  // rows past the end repeat the last token, unwritten
    for (int half = 0; half < 2; half++) {
        const float *src = half == 0 ? k : kr;
        float ss = 0.f;
        for (int e = part; e < d; e += 16) {
            const float v = src[row + e];
            s_x[tok * ld + half * d + e] = v;
            ss = fmaf(v, v, ss);
        }
        __syncthreads();  // the sums of the half before are read
        s_r[tok][part] = ss;
        __syncthreads();
        ss = 0.f;
#pragma unroll
        for (int i = 0; i < 16; i++) ss += s_r[tok][i];
        const float r = 1.0f / sqrtf(ss / (float)d + eps);
        for (int e = part; e < d; e += 16) s_x[tok * ld + half * d + e] *= r;
    }
    const int n_sl = (2 * d + kGfSlice - 1) / kGfSlice, n_ut = (width + kGfUnits - 1) / kGfUnits, total = n_sl * n_ut;
    float4 w[8];  // this thread's part of the slice on its way to LDS: unit tid / 4 of 64, features 16 * i + 4 * (tid % 4) ..
    auto fetch = [&](int it) __attribute__((always_inline)) {
        const int u = it / n_sl * kGfUnits + (tid >> 2), e0 = it % n_sl * kGfSlice + (tid & 3) * 4;
        const float *src = W1 + ((size_t)h * width + min(u, width - 1)) * (2 * d);  // a unit past the last one repeats it, unused
#pragma unroll
        for (int i = 0; i < 8; i++) w[i] = *reinterpret_cast<const float4 *>(src + min(e0 + 16 * i, 2 * d - 4));
    };
    auto stage = [&](int buf) __attribute__((always_inline)) {
#pragma unroll
        for (int i = 0; i < 8; i++) {
            float *dst = &s_w[buf][16 * i + (tid & 3) * 4][tid >> 2];
            dst[0] = w[i].x; dst[kGfUnits + 4] = w[i].y; dst[2 * (kGfUnits + 4)] = w[i].z; dst[3 * (kGfUnits + 4)] = w[i].w;
        }
    };
    fetch(0);
    stage(0);
    __syncthreads();
    float acc = 0.f, z[4] = {0.f, 0.f, 0.f, 0.f};  // acc: twice the logit
    for (int i = 0; i < total; i++) {
        if (i + 1 < total) fetch(i + 1);
        const int e0 = i % n_sl * kGfSlice, ne = min(kGfSlice, 2 * d - e0);
        const float *x = &s_x[tok * ld + e0];
#pragma unroll 4
        for (int e = 0; e < ne; e += 4) {
            const float4 xv = *reinterpret_cast<const float4 *>(x + e);
#pragma unroll
            for (int c = 0; c < 4; c++) {
                const float4 wv = *reinterpret_cast<const float4 *>(&s_w[i & 1][e + c][part * 4]);
                const float xc = c == 0 ? xv.x : c == 1 ? xv.y : c == 2 ? xv.z : xv.w;
                z[0] = fmaf(wv.x, xc, z[0]); z[1] = fmaf(wv.y, xc, z[1]); z[2] = fmaf(wv.z, xc, z[2]); z[3] = fmaf(wv.w, xc, z[3]);
            }
        }
        if (i % n_sl == n_sl - 1) {
#pragma unroll
            for (int c = 0; c < 4; c++) {
                const int u = i / n_sl * kGfUnits + part * 4 + c;
                if (u < width) acc = fmaf(W2[(size_t)h * width + u], gm_gelu2(z[c] + b1[(size_t)h * width + u]), acc);
                z[c] = 0.f;
            }
        }
        if (i + 1 < total) stage((i + 1) & 1);
        __syncthreads();
    }
    s_r[tok][part] = acc;
    __syncthreads();
    if (tid < kGfTokens && t < T) {
        float a = 0.f;
#pragma unroll
        for (int i = 0; i < 16; i++) a += s_r[tok][i];
        g_out[(size_t)t * Hkv + h] = 1.0f / (1.0f + __expf(-fmaf(0.5f, a, b2[h])));
    }
}

// Any other shape, and few tokens of an fp32 model: one block per (token, head), one hidden unit per
// thread and turn, fp32 arithmetic.  With bf16 inputs the features are rounded to bf16 like
// in the matrix-core kernel, so both compute the same function.
template <int DT>
__global__ __launch_bounds__(256) void gate_mlp_generic_kernel(const char *k, const char *kr, const char *W1,
                                                               const float *b1, const char *W2, const float *b2,
                                                               float eps, float *g_out, int Hkv, int d, int width) {
    extern __shared__ float s_x[];  // 2d features, then 8 partial sums
    float *s_red = s_x + 2 * d;
    const long long t = blockIdx.x;
    const int h = blockIdx.y, lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    auto ld = [&](const char *p, size_t i) -> float {
        return DT == WGKV_F32 ? reinterpret_cast<const float *>(p)[i]
                              : gm_bf16_to_f32(reinterpret_cast<const uint16_t *>(p)[i]);
    };
    for (int part = 0; part < 2; part++) {
        const char *src = part == 0 ? k : kr;
        const size_t row = ((size_t)t * Hkv + h) * d;
        float ss = 0.f;
        for (int e = threadIdx.x; e < d; e += 256) {
            const float v = ld(src, row + e);
            ss = fmaf(v, v, ss);
        }
        ss = group_sum<64>(ss);
        __syncthreads();
        if (lane == 0) s_red[wave] = ss;
        __syncthreads();
        ss = s_red[0] + s_red[1] + s_red[2] + s_red[3];
        const float r = 1.0f / sqrtf(ss / (float)d + eps);
        for (int e = threadIdx.x; e < d; e += 256) {
            float xn = ld(src, row + e) * r;
            if (DT == WGKV_BF16) xn = (float)(__bf16)xn;
            s_x[part * d + e] = xn;
        }
    }
    __syncthreads();
    float acc = 0.f;  // twice the logit
    for (int u = threadIdx.x; u < width; u += 256) {
        const size_t wrow = ((size_t)h * width + u) * 2 * d;
        float z = b1[(size_t)h * width + u];
        for (int e = 0; e < 2 * d; e++) z = fmaf(ld(W1, wrow + e), s_x[e], z);
        acc = fmaf(ld(W2, (size_t)h * width + u), gm_gelu2(z), acc);
    }
    acc = group_sum<64>(acc);
    __syncthreads();
    if (lane == 0) s_red[4 + wave] = acc;
    __syncthreads();
    if (threadIdx.x == 0) {
        const float logit = 0.5f * (s_red[4] + s_red[5] + s_red[6] + s_red[7]) + b2[h];
        g_out[(size_t)t * Hkv + h] = 1.0f / (1.0f + __expf(-logit));
    }
}

hipError_t launch_gate_mlp(int dtype, int64_t n_tokens, int n_kv_heads, int head_dim, int width,
                           const void *k, const void *k_rope, const void *w1, const float *b1,
                           const void *w2, const float *b2, float eps, float *g_out, hipStream_t st) {
    if (n_tokens == 0) return hipSuccess;
    const char *kp = (const char *)k, *krp = (const char *)k_rope, *w1p = (const char *)w1, *w2p = (const char *)w2;
    const int64_t pairs = n_tokens * n_kv_heads;
    // A few tokens at a ragged width of some hundred units are the plain kernel's: one turn of its threads over the units, where a chunk that
    // ends in zeros, the two halves of a row's sum and the matrix operands cost a microsecond (us there / in chunks: 64 pairs, width 130
    // 6.7 / 7.5 and 8.6 / 9.5, width 500 9.2 / 10.0 and 13.1 / 14.7, 64- and 128-wide; 400 pairs of width 500 16.8 / 10.4 and 26.9 / 15.6; 8
    // pairs of width 33 6.3 / 5.9 and 8.1 / 7.1, of 2000 25.9 / 22.7 and 39.4 / 37.2).
    const bool few_ragged = pairs <= 256 && width % kGmUnits != 0 && width > 96 && width < 1024;
    if (dtype == WGKV_BF16 && (head_dim == 128 || head_dim == 64) && !few_ragged) {
        // Which form, by the number of (token, head) pairs: each up to one round of its resident blocks, where its time
        // is nearly flat.  us at head_dim 128, width 512, for 8K / 32K / 64K / 96K / 128K pairs (the lines lie where
        // two columns cross; 64-wide heads cross at the same places):
        //   32 tokens a block, the units split over its waves        15   45    87   129
        //   128 tokens, two groups of waves with half the units each  20   23    44    65    86
        //   128 tokens, three blocks per compute unit                 23   26    35    46    63
        //   256 tokens (a product's W1 operand used twice)            34   37    42    53    56
        // The rounds are those of 256 compute units, and other widths than 512 (and 32, below) were not timed for the lines:
        // a pair's work grows with the width in every form alike, what a form leaves idle does not depend on it.
        // A width that is no multiple of 32 ends in a chunk with units of zeros (2048 tokens x 8 heads, width 200: 301 us with a
        // block per (token, head), 13 here).
        // One or two chunks of hidden units leave nothing to split over waves, one chunk nothing to use twice either: those calls
        // count as of the size that takes the third form.  Width 32, 33 / 4096 / 16384 tokens x 8 heads: 6.3 / 7.5 / 19.3 us, by
        // their own size 8.5 / 9.6 / 20.5.
        const int64_t cols = width <= kGmUnits ? 98304 : width <= 2 * kGmUnits ? std::max<int64_t>(pairs, 98304) : pairs;
#define WGKV_GM(D_, CB_, US_, R_)                                                                                       \
    hipLaunchKernelGGL((gate_mlp_mfma_kernel<D_, CB_, US_, R_>),                                                        \
                       dim3((unsigned)((n_tokens + 4 * kGmTokens * CB_ - 1) / (4 * kGmTokens * CB_)), n_kv_heads),       \
                       dim3(256 * US_), 0, st, kp, krp, w1p, b1, w2p, b2, eps, g_out, (long long)n_tokens, n_kv_heads, width)
#define WGKV_GM_D(D_, R_)                                                                                               \
    if (cols <= 8192)                                                                                              \
        hipLaunchKernelGGL((gate_mlp_split_kernel<D_, R_>), dim3((unsigned)((n_tokens + kGmTokens - 1) / kGmTokens * n_kv_heads)), \
                           dim3(kGmSplit * 64), 0, st, kp, krp, w1p, b1, w2p, b2, eps, g_out, (long long)n_tokens, n_kv_heads, width); \
    else if (cols <= 32768) WGKV_GM(D_, 1, 2, R_);                                                                     \
    else if (cols <= 98304) WGKV_GM(D_, 1, 1, R_);                                                                    \
    else WGKV_GM(D_, 2, 1, R_)
        const bool ragged = width % kGmUnits != 0;
        if (head_dim == 128) {
            if (ragged) { WGKV_GM_D(128, true); } else { WGKV_GM_D(128, false); }
        } else {
            if (ragged) { WGKV_GM_D(64, true); } else { WGKV_GM_D(64, false); }
        }
#undef WGKV_GM_D
#undef WGKV_GM
        return hipGetLastError();
    }
    // A block of 16 tokens stages W1 slice by slice (rows of whole 16-byte pieces), 64 units by 128 features, and its time is that chain up to
    // some 300 blocks; the plain kernel's grows with the pairs from 200 on.  They cross at the fewer pairs the more of a slice is used
    // and the more turns the plain kernel takes.  Timed over 1 to 16000 pairs, widths of 1 to 2000, head dimensions of 16 to 256; us there /
    // here for 128-wide heads: width 512, 400 pairs 32.7 / 49.8, 800 60.6 / 49.6; width 100, 800 16.5 / 18.3, 1200 19.6 / 17.9; width 33, 1200 10.5 /
    // 12.6, 2400 18.1 / 12.6; width 1, 1600 8.9 / 12.2, 4000 14.6 / 12.7; 16-wide heads, width 512, 1200 13.8 / 17.7, 2400 22.9 / 17.9.
    const int64_t line = std::max<int64_t>(width >= 256 ? 640 : width >= 64 ? 1088 : width >= 32 ? 1600 : 2304,
                                           head_dim <= 16 ? 1600 : head_dim > 32 ? 0 : width >= 256 ? 1024 : 1408);
    const size_t smem_f32 = (size_t)kGfTokens * (2 * head_dim + 4) * sizeof(float);
    if (dtype == WGKV_F32 && pairs > line && head_dim % 2 == 0 && n_tokens < ((int64_t)1 << 34) && smem_f32 <= 40 * 1024) {
        hipLaunchKernelGGL(gate_mlp_f32_kernel, dim3((unsigned)((n_tokens + kGfTokens - 1) / kGfTokens), n_kv_heads), dim3(256), smem_f32, st, (const float *)k,
                           (const float *)k_rope, (const float *)w1, b1, (const float *)w2, b2, eps, g_out, (long long)n_tokens, n_kv_heads, head_dim, width);
        return hipGetLastError();
    }
    // grid.x carries the tokens: split very long inputs over several launches
    const size_t smem = (size_t)(2 * head_dim + 8) * sizeof(float);
    const int es = dtype == WGKV_F32 ? 4 : 2;
    for (int64_t t0 = 0; t0 < n_tokens; t0 += (1 << 30)) {
        const int64_t nt = n_tokens - t0 < (1 << 30) ? n_tokens - t0 : (1 << 30);
        const dim3 grid((unsigned)nt, n_kv_heads);
        const size_t off = (size_t)t0 * n_kv_heads * head_dim * es;
        if (dtype == WGKV_F32)
            hipLaunchKernelGGL(gate_mlp_generic_kernel<WGKV_F32>, grid, dim3(256), smem, st, kp + off, krp + off, w1p,
                               b1, w2p, b2, eps, g_out + (size_t)t0 * n_kv_heads, n_kv_heads, head_dim, width);
        else
            hipLaunchKernelGGL(gate_mlp_generic_kernel<WGKV_BF16>, grid, dim3(256), smem, st, kp + off, krp + off,
                               w1p, b1, w2p, b2, eps, g_out + (size_t)t0 * n_kv_heads, n_kv_heads, head_dim, width);
        const hipError_t e = hipGetLastError();
        if (e != hipSuccess) return e;
    }
    return hipSuccess;
}

}  // namespace wgkv
