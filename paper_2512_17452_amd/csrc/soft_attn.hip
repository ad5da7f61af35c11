// Training-time Write-Gated Attention (Sec. 3.2, "Write-Gated Attention" and "Log-space
// transformation for efficient training") on the gfx950 matrix cores: causal attention of a
// whole sequence with the additive bias
//     B_ij = log(m_ij + eps),   m_ij = max(1(i - j < W_local), g_j),
// forward with the row log-sum-exp, and the gradients with respect to q, k, v and g.
//
//   soft_attn_fwd_kernel       block = 32 or 64 query positions x the 4 query heads of a kv head,
//                              key tiles of 64 in LDS; S^T = K Q^T, O^T = V^T P^T
//   soft_attn_rowdot_kernel    D_i = dO_i . O_i per (position, query head)
//   soft_attn_bwd_dq_kernel    same blocking as the forward: S^T and dP^T = V dO^T per key tile,
//                              dS^T = P^T (dP^T - D), dQ^T += K^T dS^T
//   soft_attn_bwd_dkv_kernel   a wave owns 32 keys of a kv head and streams (32 queries, head) tiles: S = Q K^T,
//                              dP = dO V^T, dV^T += dO^T P, dK^T += Q^T dS and the sum that becomes dg
//
// All products are v_mfma_f32_32x32x16_bf16 with fp32 accumulation; every operand that is
// reused over the whole loop (the wave's own rows) sits in registers.  The streamed tiles come from memory straight
// into LDS, once, in an order of their 16-byte pieces that serves products over d (whole rows) and products that contract
// over positions (columns, with the transposing LDS load) alike; they used to pass through registers into two
// padded copies.  A lane of an accumulator tile owns one column, so per-column quantities are plain scalars.
//
// What bounds them on one 16384-token sequence (8 kv heads, window 256): power.  The chip runs the three kernels at 1.9 /
// 1.9 / 1.76 GHz of 2.4 with the matrix cores busy 41 / 50 / 48 % of those cycles, no bank conflict, waves waiting for
// an instruction's result a quarter of their time.  Forward 2.71 -> 2.64 ms, dQ 3.46 -> 3.25, dK/dV 6.32 -> 4.75 (two
// waves used to share 32 keys, one forming P and dV, one dP and dK, with P in 32 bits through LDS: one and a half
// times the LDS traffic that the matrix cores hide).
#include <algorithm>
#include <climits>
#include <type_traits>

#include "lds_tiles.h"
#include "wgkv_dev.h"

namespace wgkv {

typedef __attribute__((ext_vector_type(2))) __bf16 sa_bf16x2_t;
typedef __attribute__((ext_vector_type(16))) float sa_f32x16_t;

constexpr int kSaG = 4;         // query heads per kv head

struct SoftSeqs {
    int32_t n;
    int32_t ntok[kMaxCallSeqs];
    int32_t base[kMaxCallSeqs];  // first packed row of the sequence
};

struct SoftArgs {
    int nx;                 // blocks per (sequence, kv head) of the launch
    int Hq, Hkv, W;
    float scale_log2e;      // scale * log2(e): scores are kept in base-2 units
    float scale;
    float eps;
    const char *q, *k, *v;  // bf16 [rows][heads][128]
    const float *g;         // [rows][Hkv]
    float *out;             // [rows][Hq][128]
    float *lse;             // [rows][Hq], natural logarithm
    // backward only
    const char *dout;       // bf16 [rows][Hq][128]
    float *rowdot;          // [rows][Hq]
    float *dq, *dk, *dv, *dg;
};

__device__ __forceinline__ uint32_t sa_pack(float lo, float hi) {
    sa_bf16x2_t t = {(__bf16)lo, (__bf16)hi};
    return __builtin_bit_cast(uint32_t, t);
}

// The two bias values of a key in base-2 units: inside the window m = max(1, g), outside m = max(0, g).
__device__ __forceinline__ void sa_bias(float gj, float eps, float &b_in, float &b_out) {
    b_in = __log2f(fmaxf(1.0f, gj) + eps);
    b_out = __log2f(fmaxf(0.0f, gj) + eps);
}

// Key tiles of the forward and the dQ kernel: 64 rows of K and of V in two LDS buffers, requested one tile ahead.  The
// scores g of a tile are requested two tiles ahead into a copy per wave, and a wave turns them into the two biases
// of a key (both halves of the wave take part) one tile ahead.
constexpr int kSaT2 = 64;                       // keys per tile
constexpr int kSaTile2B = kSaT2 * kSaD * 2;

template <int NW>
struct SoftKeyTiles {
    __attribute__((aligned(1024))) char t[2][2][kSaTile2B];     // K and V
    __attribute__((aligned(16))) float b_in[2][NW][kSaT2], b_out[2][NW][kSaT2];
    __attribute__((aligned(16))) float g[2][NW][kSaT2];
};

template <int NW>
__device__ __forceinline__ void sa_fetch_keys(SoftKeyTiles<NW> &l, const SoftArgs &a, int base, int T, int h, int t, int wave, int lane) {
    asm volatile("" : "+v"(lane));  // the lane's offsets are formed per tile: no registers to keep them
    {
        const int last = T - 1 - t * kSaT2;  // >= 0
        const size_t row = (size_t)(base + t * kSaT2) * a.Hkv + h;
        const char *kp = a.k + row * (kSaD * 2), *vp = a.v + row * (kSaD * 2);
        constexpr int kRows = kSaT2 / NW;
#pragma unroll
        for (int i = 0; i < kRows / 4; i++) {
            const int r = wave * kRows + 4 * i + (lane >> 4);
            const uint32_t o = (uint32_t)(min(r, last) * a.Hkv * (kSaD * 2) + ((lane & 15) ^ sa_sw_f(r)) * 16);
            sa_dma16(kp, o, &l.t[t & 1][0][(wave * kRows + 4 * i) * (kSaD * 2)]);
            sa_dma16(vp, o, &l.t[t & 1][1][(wave * kRows + 4 * i) * (kSaD * 2)]);
        }
    }
}
template <int NW>
__device__ __forceinline__ void sa_fetch_g(SoftKeyTiles<NW> &l, const SoftArgs &a, int base, int T, int h, int t, int wave, int lane) {
    const int r0 = min(t * kSaT2, T - 1);  // a tile past the end reads the last row
    const int off = min(lane, T - 1 - r0) * a.Hkv * 4;
    sa_dma4(a.g + (size_t)(base + r0) * a.Hkv + h, (uint32_t)off, l.g[t & 1][wave]);
}
template <int NW>
__device__ __forceinline__ void sa_put_bias(SoftKeyTiles<NW> &l, float eps, int t, int wave, int lane) {
    float b_in, b_out;
    sa_bias(l.g[t & 1][wave][lane], eps, b_in, b_out);
    l.b_in[t & 1][wave][lane] = b_in;
    l.b_out[t & 1][wave][lane] = b_out;
}

// ---------------------------------------------------------------------------------------------
// forward
// ---------------------------------------------------------------------------------------------
template <int NRB>
__global__ __launch_bounds__(256 * NRB, 2) void soft_attn_fwd_kernel(SoftSeqs cs, SoftArgs a) {
    constexpr int NW = 4 * NRB, kQ = 32 * NRB;
    __shared__ SoftKeyTiles<NW> l_t;

    int bx, h, b;
    xcd_item(a.nx, a.Hkv, cs.n, bx, h, b);
    const int qt = a.nx - 1 - bx;  // longest rows first
    const int T = cs.ntok[b], base = cs.base[b];
    if (qt * kQ >= T) return;  // block-uniform
    const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int head = wave & 3, rb = wave >> 2;
    const int qn = lane & 31, half = lane >> 5;
    const int q0 = qt * kQ;
    const int i_end = min(T, q0 + kQ);
    const int n_tiles = (i_end + kSaT2 - 1) / kSaT2;
    const int n_far = q0 - a.W >= kSaT2 - 1 ? (q0 - a.W + 1) / kSaT2 : 0;  // tiles wholly outside every window of the block

    sa_bf16x8_t qv[8];
    const int qi = min(q0 + rb * 32 + qn, T - 1);
    {
        const char *qp = a.q + ((size_t)(base + qi) * a.Hq + (size_t)h * kSaG + head) * kSaD * 2;
#pragma unroll
        for (int ks = 0; ks < 8; ks++) qv[ks] = *reinterpret_cast<const sa_bf16x8_t *>(qp + (ks * 16 + half * 8) * 2);
    }
    sa_f32x16_t o[4];
    // l sums the weights as the second product sees them (rounded to bf16) and normalises the
    // output; lx sums them unrounded and gives the log-sum-exp the backward pass starts from
    float m = -INFINITY, l = 0.f, lx = 0.f;
#pragma unroll
    for (int db = 0; db < 4; db++)
#pragma unroll
        for (int c = 0; c < 16; c++) o[db][c] = 0.f;
    const int o_row = sa_sw_row(qn, half), o_col = sa_sw_col(lane);

    auto body = [&](int t, auto far_t) __attribute__((always_inline)) {
        constexpr bool kFar = decltype(far_t)::value;
        if (t + 1 < n_tiles) sa_fetch_keys(l_t, a, base, T, h, t + 1, wave, lane);
        sa_fetch_g(l_t, a, base, T, h, t + 2, wave, lane);
        const char *tk = l_t.t[t & 1][0], *tv = l_t.t[t & 1][1];
        // ---- S^T for the two halves of 32 keys ----
        sa_f32x16_t s[2];
#pragma unroll
        for (int hf = 0; hf < 2; hf++) {
#pragma unroll
            for (int c = 0; c < 16; c++) s[hf][c] = 0.f;
#pragma unroll
            for (int ks = 0; ks < 8; ks++)
                s[hf] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(sa_sw_get_row(tk + hf * kSaTileB, o_row, ks), qv[ks], s[hf], 0, 0, 0);
        }
        // register c = 4j+i of s[hf] holds key 32*hf + 8j + 4*half + i of the tile
        float mt = -INFINITY;
#pragma unroll
        for (int hf = 0; hf < 2; hf++)
#pragma unroll
            for (int j = 0; j < 4; j++) {
                const float4 bo4 = *reinterpret_cast<const float4 *>(&l_t.b_out[t & 1][wave][32 * hf + 8 * j + 4 * half]);
                const float bo[4] = {bo4.x, bo4.y, bo4.z, bo4.w};
                if (kFar) {
#pragma unroll
                    for (int i = 0; i < 4; i++) {
                        s[hf][4 * j + i] = fmaf(s[hf][4 * j + i], a.scale_log2e, bo[i]);
                        mt = fmaxf(mt, s[hf][4 * j + i]);
                    }
                } else {
                    const float4 bi4 = *reinterpret_cast<const float4 *>(&l_t.b_in[t & 1][wave][32 * hf + 8 * j + 4 * half]);
                    const float bi[4] = {bi4.x, bi4.y, bi4.z, bi4.w};
#pragma unroll
                    for (int i = 0; i < 4; i++) {
                        const int jg = t * kSaT2 + 32 * hf + 8 * j + 4 * half + i;
                        const float bias = (qi - jg < a.W) ? bi[i] : bo[i];
                        s[hf][4 * j + i] = (jg <= qi) ? fmaf(s[hf][4 * j + i], a.scale_log2e, bias) : -INFINITY;
                        mt = fmaxf(mt, s[hf][4 * j + i]);
                    }
                }
            }
        mt = fmaxf(mt, __shfl_xor(mt, 32));
        const float mnew = fmaxf(m, mt);
        const float msafe = mnew == -INFINITY ? 0.f : mnew;
        const float corr = __builtin_amdgcn_exp2f(m - msafe);
        uint32_t pb[16];
        float ps = 0.f, px = 0.f;
        const sa_bf16x2_t ones = {(__bf16)1.0f, (__bf16)1.0f};
#pragma unroll
        for (int c = 0; c < 16; c++) {
            const float p0 = __builtin_amdgcn_exp2f(s[c >> 3][(2 * c) & 15] - msafe);
            const float p1 = __builtin_amdgcn_exp2f(s[c >> 3][(2 * c + 1) & 15] - msafe);
            px += p0 + p1;
            pb[c] = sa_pack(p0, p1);
            ps = __builtin_amdgcn_fdot2_f32_bf16(__builtin_bit_cast(sa_bf16x2_t, pb[c]), ones, ps, false);
        }
        l = l * corr + ps;
        lx = lx * corr + px;
        if (__builtin_amdgcn_ballot_w64(mnew > m) != 0) {
#pragma unroll
            for (int db = 0; db < 4; db++)
#pragma unroll
                for (int c = 0; c < 16; c++) o[db][c] *= corr;
        }
        m = mnew;
        // ---- O^T += V^T P^T, four steps of 16 keys ----
#pragma unroll
        for (int t2 = 0; t2 < 4; t2++) {
            const uint4 p4 = make_uint4(pb[4 * t2], pb[4 * t2 + 1], pb[4 * t2 + 2], pb[4 * t2 + 3]);
            const sa_bf16x8_t pbv = __builtin_bit_cast(sa_bf16x8_t, p4);
#pragma unroll
            for (int db = 0; db < 4; db++)
                o[db] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(sa_sw_get_cols(tv, o_col, db, t2), pbv, o[db], 0, 0, 0);
        }
        sa_put_bias(l_t, a.eps, t + 1, wave, lane);
        sa_dma_wait_barrier<0>();  // tile t + 1 is there, and nobody reads tile t any more
    };
#pragma unroll
    for (int ks = 0; ks < 8; ks++) asm volatile("" : "+v"(qv[ks]));  // waited for here, not in the loop
    sa_fetch_keys(l_t, a, base, T, h, 0, wave, lane);
    sa_fetch_g(l_t, a, base, T, h, 0, wave, lane);
    sa_fetch_g(l_t, a, base, T, h, 1, wave, lane);
    sa_dma_wait_barrier<0>();
    sa_put_bias(l_t, a.eps, 0, wave, lane);
    int t = 0;
    for (; t < n_far; t++) body(t, std::true_type());
    for (; t < n_tiles; t++) body(t, std::false_type());
    // register c = 4j+i of o[db] is d = 32*db + 8j + 4*half + i
    const int i = q0 + rb * 32 + qn;
    const float lt = l + __shfl_xor(l, 32), lxt = lx + __shfl_xor(lx, 32);
    if (i < T) {
        const float inv = 1.0f / lt;
        const size_t orow = (size_t)(base + i) * a.Hq + (size_t)h * kSaG + head;
        float *op = a.out + orow * kSaD;
#pragma unroll
        for (int db = 0; db < 4; db++)
#pragma unroll
            for (int j = 0; j < 4; j++) {
                const float4 w4 = make_float4(o[db][4 * j] * inv, o[db][4 * j + 1] * inv, o[db][4 * j + 2] * inv,
                                              o[db][4 * j + 3] * inv);
                *reinterpret_cast<float4 *>(op + 32 * db + 8 * j + 4 * half) = w4;
            }
        if (half == 0) a.lse[orow] = (m + __log2f(lxt)) * 0.6931471805599453f;
    }
}

// ---------------------------------------------------------------------------------------------
// backward, step 0: D_i = dO_i . O_i   (32 lanes per row)
// ---------------------------------------------------------------------------------------------
__global__ __launch_bounds__(256) void soft_attn_rowdot_kernel(int64_t n_rows, const char *dout, const float *out,
                                                               float *rowdot) {
    const int64_t r = (int64_t)blockIdx.x * 8 + (threadIdx.x >> 5);
    const int sub = threadIdx.x & 31;
    float acc = 0.f;
    if (r < n_rows) {
        const uint2 d2 = *reinterpret_cast<const uint2 *>(dout + (size_t)r * kSaD * 2 + sub * 8);
        const float4 o4 = *reinterpret_cast<const float4 *>(out + (size_t)r * kSaD + sub * 4);
        acc = __uint_as_float(d2.x << 16) * o4.x + __uint_as_float(d2.x & 0xffff0000u) * o4.y +
              __uint_as_float(d2.y << 16) * o4.z + __uint_as_float(d2.y & 0xffff0000u) * o4.w;
    }
    acc = group_sum<32>(acc);
    if (r < n_rows && sub == 0) rowdot[r] = acc;
}

// ---------------------------------------------------------------------------------------------
// backward, dQ: columns of every tile are this wave's 32 queries
//
// Slices of the two products of a half tile go in turn (two chains, not one behind the other), and the sums of 16 keys beside the dS of
// the next 16.  Backward and forward, us before / now: 16384 tokens 10790 / 10660, 9000 3670 / 3620, four of 1000-3000 1136 / 1116, 1000
// 173 / 164.  (The second half's products beside the first one's dS too: three spilled registers, 0.5 % slower.  The same
// in the other two kernels: forward 2.60 -> 2.74 ms, dK/dV, which has no registers to spare, 4.83 -> 5.09.)
// ---------------------------------------------------------------------------------------------
template <int NRB>
__global__ __launch_bounds__(256 * NRB, 2) void soft_attn_bwd_dq_kernel(SoftSeqs cs, SoftArgs a) {
    constexpr int NW = 4 * NRB, kQ = 32 * NRB;
    __shared__ SoftKeyTiles<NW> l_t;

    int bx, h, b;
    xcd_item(a.nx, a.Hkv, cs.n, bx, h, b);
    const int qt = a.nx - 1 - bx;
    const int T = cs.ntok[b], base = cs.base[b];
    if (qt * kQ >= T) return;
    const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int head = wave & 3, rb = wave >> 2;
    const int qn = lane & 31, half = lane >> 5;
    const int q0 = qt * kQ;
    const int i_end = min(T, q0 + kQ);
    const int n_tiles = (i_end + kSaT2 - 1) / kSaT2;
    const int n_far = q0 - a.W >= kSaT2 - 1 ? (q0 - a.W + 1) / kSaT2 : 0;

    const int qi = min(q0 + rb * 32 + qn, T - 1);
    const size_t qrow = (size_t)(base + qi) * a.Hq + (size_t)h * kSaG + head;
    sa_bf16x8_t qv[8], dov[8];
    {
        const char *qp = a.q + qrow * kSaD * 2, *dp = a.dout + qrow * kSaD * 2;
#pragma unroll
        for (int ks = 0; ks < 8; ks++) {
            qv[ks] = *reinterpret_cast<const sa_bf16x8_t *>(qp + (ks * 16 + half * 8) * 2);
            dov[ks] = *reinterpret_cast<const sa_bf16x8_t *>(dp + (ks * 16 + half * 8) * 2);
        }
    }
    float lse2 = a.lse[qrow] * 1.4426950408889634f;
    float Di = a.rowdot[qrow];
    sa_f32x16_t dq[4];
#pragma unroll
    for (int db = 0; db < 4; db++)
#pragma unroll
        for (int c = 0; c < 16; c++) dq[db][c] = 0.f;
    const int o_row = sa_sw_row(qn, half), o_col = sa_sw_col(lane);

    auto body = [&](int t, auto far_t) __attribute__((always_inline)) {
        constexpr bool kFar = decltype(far_t)::value;
        if (t + 1 < n_tiles) sa_fetch_keys(l_t, a, base, T, h, t + 1, wave, lane);
        sa_fetch_g(l_t, a, base, T, h, t + 2, wave, lane);
        sa_f32x16_t s[2], dp[2];
        // scores and dP of 32 keys, slices of both in turn
        auto products = [&](int hf, int ks) __attribute__((always_inline)) {
            s[hf] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(sa_sw_get_row(l_t.t[t & 1][0] + hf * kSaTileB, o_row, ks), qv[ks], s[hf], 0, 0, 0);
            dp[hf] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(sa_sw_get_row(l_t.t[t & 1][1] + hf * kSaTileB, o_row, ks), dov[ks], dp[hf], 0, 0, 0);
        };
        // dS^T = P^T (dP^T - D_i) of registers 4j .. 4j+3, rounded to bf16 for the last product
        uint32_t db_[2][8];
        auto dscores = [&](int hf, int j) __attribute__((always_inline)) {
            const float4 bo4 = *reinterpret_cast<const float4 *>(&l_t.b_out[t & 1][wave][32 * hf + 8 * j + 4 * half]);
            const float bo[4] = {bo4.x, bo4.y, bo4.z, bo4.w};
            float ds[4];
            if (kFar) {
#pragma unroll
                for (int i = 0; i < 4; i++)
                    ds[i] = __builtin_amdgcn_exp2f(fmaf(s[hf][4 * j + i], a.scale_log2e, bo[i] - lse2)) * (dp[hf][4 * j + i] - Di);
            } else {
                const float4 bi4 = *reinterpret_cast<const float4 *>(&l_t.b_in[t & 1][wave][32 * hf + 8 * j + 4 * half]);
                const float bi[4] = {bi4.x, bi4.y, bi4.z, bi4.w};
#pragma unroll
                for (int i = 0; i < 4; i++) {
                    const int jg = t * kSaT2 + 32 * hf + 8 * j + 4 * half + i;
                    const float bias = (qi - jg < a.W) ? bi[i] : bo[i];
                    const float x = (jg <= qi) ? fmaf(s[hf][4 * j + i], a.scale_log2e, bias) - lse2 : -INFINITY;
                    ds[i] = __builtin_amdgcn_exp2f(x) * (dp[hf][4 * j + i] - Di);
                }
            }
            db_[hf][2 * j] = sa_pack(ds[0], ds[1]);
            db_[hf][2 * j + 1] = sa_pack(ds[2], ds[3]);
        };
        auto sums = [&](int hf, int t2, int db) __attribute__((always_inline)) {
            const uint32_t *w = &db_[hf][4 * t2];
            dq[db] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(sa_sw_get_cols(l_t.t[t & 1][0] + hf * kSaTileB, o_col, db, t2),
                                                             __builtin_bit_cast(sa_bf16x8_t, make_uint4(w[0], w[1], w[2], w[3])), dq[db], 0, 0, 0);
        };
#pragma unroll
        for (int hf = 0; hf < 2; hf++)
#pragma unroll
            for (int c = 0; c < 16; c++) { s[hf][c] = 0.f; dp[hf][c] = 0.f; }
#pragma unroll
        for (int hf = 0; hf < 2; hf++) {
#pragma unroll
            for (int ks = 0; ks < 8; ks++) products(hf, ks);
            dscores(hf, 0);
            dscores(hf, 1);
            // the first 16 keys' sums beside the dS of the others
#pragma unroll
            for (int j = 0; j < 2; j++) {
                __builtin_amdgcn_sched_barrier(0);
                sums(hf, 0, 2 * j);
                sums(hf, 0, 2 * j + 1);
                dscores(hf, 2 + j);
                if (kFar) {
                    __builtin_amdgcn_sched_group_barrier(0x100, 5, 0);
#pragma unroll
                    for (int i = 0; i < 2; i++) {
                        __builtin_amdgcn_sched_group_barrier(0x008, 1, 0);
                        __builtin_amdgcn_sched_group_barrier(0x402, 11, 0);
                    }
                }
            }
            __builtin_amdgcn_sched_barrier(0);
#pragma unroll
            for (int db = 0; db < 4; db++) sums(hf, 1, db);
        }
        sa_put_bias(l_t, a.eps, t + 1, wave, lane);
        sa_dma_wait_barrier<0>();  // tile t + 1 is there, and nobody reads tile t any more
    };
#pragma unroll
    for (int ks = 0; ks < 8; ks++) asm volatile("" : "+v"(qv[ks]), "+v"(dov[ks]));  // waited for here, not in the loop
    asm volatile("" : "+v"(lse2), "+v"(Di));
    sa_fetch_keys(l_t, a, base, T, h, 0, wave, lane);
    sa_fetch_g(l_t, a, base, T, h, 0, wave, lane);
    sa_fetch_g(l_t, a, base, T, h, 1, wave, lane);
    sa_dma_wait_barrier<0>();
    sa_put_bias(l_t, a.eps, 0, wave, lane);
    int t = 0;
    for (; t < n_far; t++) body(t, std::true_type());
    for (; t < n_tiles; t++) body(t, std::false_type());
    const int i = q0 + rb * 32 + qn;
    if (i < T) {
        float *op = a.dq + qrow * kSaD;
#pragma unroll
        for (int db = 0; db < 4; db++)
#pragma unroll
            for (int j = 0; j < 4; j++) {
                const float4 w4 = make_float4(dq[db][4 * j] * a.scale, dq[db][4 * j + 1] * a.scale,
                                              dq[db][4 * j + 2] * a.scale, dq[db][4 * j + 3] * a.scale);
                *reinterpret_cast<float4 *>(op + 32 * db + 8 * j + 4 * half) = w4;
            }
    }
}

// ---------------------------------------------------------------------------------------------
// backward, dK / dV / dg: columns of every tile are this wave's keys
//
// A wave owns 32 keys and forms all four products of them: S = Q K^T and dP = dO V^T with its K and V rows in
// registers as the column operand, dV^T += dO^T P and dK^T += Q^T dS with P and dS straight from the accumulators.
// Streamed tiles (32 queries of one query head, Q and dO) come through LDS once and are read in both layouts.
// HS waves of a block share 32 keys and take one query head each (at the end their sums meet in LDS in a fixed
// order), the other factor of the four waves is keys: HS = 1 reads a streamed tile for 128 keys and runs two blocks
// per compute unit; HS = 4 makes blocks of a quarter of the length and four times their number.
// ---------------------------------------------------------------------------------------------
template <int HS>
__global__ __launch_bounds__(256, HS == 1 ? 2 : 1) void soft_attn_bwd_dkv_kernel(SoftSeqs cs, SoftArgs a) {
    constexpr int kBufs = HS == 4 ? 2 : 3;  // one tile in use, the others arriving
    constexpr int kReq = 4 * HS + 2;        // requests of a wave per tile
    constexpr int kTurns = kSaG / HS;       // turns per query tile
    __shared__ __attribute__((aligned(1024))) char s_t[kBufs][HS][2][kSaTileB];  // Q and dO
    __shared__ __attribute__((aligned(16))) float s_ld[kBufs][4][128];           // lse and D of the wave's tile

    int kbk, h, b;  // early key blocks have the most queries: first
    xcd_item(a.nx, a.Hkv, cs.n, kbk, h, b);
    const int T = cs.ntok[b], base = cs.base[b];
    const int j0 = kbk * (128 / HS);
    if (j0 >= T) return;  // block-uniform
    const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int qn = lane & 31, half = lane >> 5;
    const int hs = wave % HS;
    const int jw = j0 + wave / HS * 32;  // first key of this wave
    const int jg = jw + qn;              // this lane's key

    sa_bf16x8_t ok[8], ov[8];
    float gk, b_far, dg_acc = 0.f;
    {
        const size_t krow = (size_t)(base + min(jg, T - 1)) * a.Hkv + h;
        const char *kp = a.k + krow * kSaD * 2, *vp = a.v + krow * kSaD * 2;
#pragma unroll
        for (int ks = 0; ks < 8; ks++) {
            ok[ks] = *reinterpret_cast<const sa_bf16x8_t *>(kp + (ks * 16 + half * 8) * 2);
            ov[ks] = *reinterpret_cast<const sa_bf16x8_t *>(vp + (ks * 16 + half * 8) * 2);
        }
        gk = a.g[krow];
        b_far = __log2f(fmaxf(0.0f, gk) + a.eps);
    }
    sa_f32x16_t av[4], ak[4];  // dV^T and dK^T: rows d, columns keys
#pragma unroll
    for (int db = 0; db < 4; db++)
#pragma unroll
        for (int c = 0; c < 16; c++) { av[db][c] = 0.f; ak[db][c] = 0.f; }

    // streamed tiles: iteration it = (query tile, HS query heads)
    const int qt_first = j0 / kSaT, n_qt = (T + kSaT - 1) / kSaT;
    const int n_it = (n_qt - qt_first) * kTurns;
    // a wave brings 8 * HS rows of Q and of dO, four rows per request, and its own copy of its tile's lse and D
    auto fetch = [&](int it_, int buf) __attribute__((always_inline)) {
        const int it = min(it_, n_it - 1);  // past the end: the last tile again, so that the count of requests stays
        const int i0 = (qt_first + it / kTurns) * kSaT;
        const size_t row0 = (size_t)(base + i0) * a.Hq + (size_t)h * kSaG + it % kTurns * HS;  // uniform; lanes add 32 bits
        const int last = T - 1 - i0;
        int ln = lane;
        asm volatile("" : "+v"(ln));  // the lane's offsets are formed per tile: no registers to keep them
#pragma unroll
        for (int i = 0; i < 2 * HS; i++) {
            const int R = wave * 8 * HS + 4 * i, hd = R / kSaT, r = R % kSaT + (ln >> 4);
            const uint32_t o = (uint32_t)(min(r, last) * a.Hq * (kSaD * 2) + ((ln & 15) ^ sa_sw_f(r)) * 16);
            sa_dma16(a.q + (row0 + hd) * (kSaD * 2), o, &s_t[buf][hd][0][R % kSaT * (kSaD * 2)]);
            sa_dma16(a.dout + (row0 + hd) * (kSaD * 2), o, &s_t[buf][hd][1][R % kSaT * (kSaD * 2)]);
        }
        const uint32_t ol = (uint32_t)(min(ln & 31, last) * a.Hq * 4);
        sa_dma4(a.lse + row0 + hs, ol, s_ld[buf][wave]);
        sa_dma4(a.rowdot + row0 + hs, ol, s_ld[buf][wave] + 64);
    };

    // one tile; far: every query of it follows every key of this wave by at least the window, and none is past the
    // end, so no pair is masked and every bias is the one outside the window (nearly all tiles of a long sequence)
    auto body = [&](int it, int buf, auto far_t) __attribute__((always_inline)) {
        constexpr bool kFar = decltype(far_t)::value;
        constexpr bool kTight = HS == 1;  // 256 registers: more than four operands in flight would spill
        const int i0 = (qt_first + it / kTurns) * kSaT;
        const char *tq = s_t[buf][hs][0], *td = s_t[buf][hs][1];
        int ln = lane;
        if (kTight) asm volatile("" : "+v"(ln));  // as above
        const int qn = ln & 31, half = ln >> 5, o_row = sa_sw_row(qn, half), o_col = sa_sw_col(ln);
        float b_in = 0.f, b_out = b_far;
        if (!kFar) {
            float gg = gk;
            asm volatile("" : "+v"(gg));
            sa_bias(gg, a.eps, b_in, b_out);
        }
        sa_f32x16_t s, dp;
#pragma unroll
        for (int c = 0; c < 16; c++) { s[c] = 0.f; dp[c] = 0.f; }
#pragma unroll
        for (int ks = 0; ks < 8; ks++) {
            const sa_bf16x8_t f = sa_sw_get_row(tq, o_row, ks);
            if (kTight && (ks & 3) == 3) __builtin_amdgcn_sched_barrier(0);
            s = __builtin_amdgcn_mfma_f32_32x32x16_bf16(f, ok[ks], s, 0, 0, 0);
        }
        if (kTight) __builtin_amdgcn_sched_barrier(0);
#pragma unroll
        for (int ks = 0; ks < 8; ks++) {
            const sa_bf16x8_t f = sa_sw_get_row(td, o_row, ks);
            if (kTight && (ks & 3) == 3) __builtin_amdgcn_sched_barrier(0);
            dp = __builtin_amdgcn_mfma_f32_32x32x16_bf16(f, ov[ks], dp, 0, 0, 0);
        }
        // register c = 4j+i of a lane holds query i0 + 8j + 4*half + i
        uint32_t pk[8];
#pragma unroll
        for (int j = 0; j < 4; j++) {
            const float4 l4 = *reinterpret_cast<const float4 *>(&s_ld[buf][wave][8 * j + 4 * half]);
            const float ls[4] = {l4.x * 1.4426950408889634f, l4.y * 1.4426950408889634f, l4.z * 1.4426950408889634f,
                                 l4.w * 1.4426950408889634f};
#pragma unroll
            for (int i = 0; i < 4; i++) {
                if (kFar) {
                    s[4 * j + i] = __builtin_amdgcn_exp2f(fmaf(s[4 * j + i], a.scale_log2e, b_out - ls[i]));
                } else {
                    const int ig = i0 + 8 * j + 4 * half + i, jl = jw + qn;
                    const float bias = (ig - jl < a.W) ? b_in : b_out;
                    const float x = (jl <= ig && ig < T) ? fmaf(s[4 * j + i], a.scale_log2e, bias) - ls[i] : -INFINITY;
                    s[4 * j + i] = __builtin_amdgcn_exp2f(x);
                }
            }
            pk[2 * j] = sa_pack(s[4 * j], s[4 * j + 1]);
            pk[2 * j + 1] = sa_pack(s[4 * j + 2], s[4 * j + 3]);
        }
        if (kTight) __builtin_amdgcn_sched_barrier(0);
        // rows = d, columns = keys, contraction over the 32 queries
#pragma unroll
        for (int t2 = 0; t2 < 2; t2++) {
            const uint4 p4 = make_uint4(pk[4 * t2], pk[4 * t2 + 1], pk[4 * t2 + 2], pk[4 * t2 + 3]);
#pragma unroll
            for (int db = 0; db < 4; db++) {
                const sa_bf16x8_t f = sa_sw_get_cols(td, o_col, db, t2);
                if (kTight && db == 3) __builtin_amdgcn_sched_barrier(0);
                av[db] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(f, __builtin_bit_cast(sa_bf16x8_t, p4), av[db], 0, 0, 0);
            }
        }
        if (kTight) __builtin_amdgcn_sched_barrier(0);
        // dS = P (dP - D_i); the part of it where m_ij follows g_j adds up to dg_j (g_j + eps)
        float dsum = 0.f;
#pragma unroll
        for (int j = 0; j < 4; j++) {
            const float4 d4 = *reinterpret_cast<const float4 *>(&s_ld[buf][wave][64 + 8 * j + 4 * half]);
            const float dd[4] = {d4.x, d4.y, d4.z, d4.w};
            float ds[4];
#pragma unroll
            for (int i = 0; i < 4; i++) {
                ds[i] = s[4 * j + i] * (dp[4 * j + i] - dd[i]);
                if (kFar) {
                    dsum += ds[i];
                } else {
                    const int ig = i0 + 8 * j + 4 * half + i, jl = jw + qn;
                    const bool follows = (ig - jl < a.W) ? gk > 1.0f : gk > 0.0f;
                    dsum += follows ? ds[i] : 0.f;
                }
            }
            pk[2 * j] = sa_pack(ds[0], ds[1]);
            pk[2 * j + 1] = sa_pack(ds[2], ds[3]);
        }
        dg_acc += dsum;  // of no use where g <= 0, and dropped there at the end
        if (kTight) __builtin_amdgcn_sched_barrier(0);
#pragma unroll
        for (int t2 = 0; t2 < 2; t2++) {
            const uint4 p4 = make_uint4(pk[4 * t2], pk[4 * t2 + 1], pk[4 * t2 + 2], pk[4 * t2 + 3]);
#pragma unroll
            for (int db = 0; db < 4; db++) {
                const sa_bf16x8_t f = sa_sw_get_cols(tq, o_col, db, t2);
                if (kTight && db == 3) __builtin_amdgcn_sched_barrier(0);
                ak[db] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(f, __builtin_bit_cast(sa_bf16x8_t, p4), ak[db], 0, 0, 0);
            }
        }
    };

    // the wave's own rows are here before the first request: the compiler's wait for them would otherwise sit in the
    // loop and wait for the requests too
#pragma unroll
    for (int ks = 0; ks < 8; ks++) asm volatile("" : "+v"(ok[ks]), "+v"(ov[ks]));
    for (int t = 0; t < kBufs - 1; t++) fetch(t, t);
    sa_dma_wait_barrier<(kBufs - 2) * kReq>();
    int buf = 0, it = 0;
    // runs body(it) while the tile kBufs - 1 turns ahead is requested
    auto turns = [&](int end, auto &&work) __attribute__((always_inline)) {
        while (it < end) {
            fetch(it + kBufs - 1, buf == 0 ? kBufs - 1 : buf - 1);
            work();
            sa_dma_wait_barrier<(kBufs - 2) * kReq>();  // tile it + 1 is there, and nobody reads tile it any more
            buf = buf == kBufs - 1 ? 0 : buf + 1;
            it++;
        }
    };
    // four stretches of tiles: every query before every key of the wave, some inside a window, far, the ragged end
    const int it_near = min(n_it, (jw / kSaT - qt_first) * kTurns);
    const int it_end = min(n_it, max(it_near, (T / kSaT - qt_first) * kTurns));
    const int it_far = min(it_end, max(it_near, ((jw + 31 + a.W + kSaT - 1) / kSaT - qt_first) * kTurns));
    turns(it_near, [&]() __attribute__((always_inline)) {});
    turns(it_far, [&]() __attribute__((always_inline)) { body(it, buf, std::false_type()); });
    turns(it_end, [&]() __attribute__((always_inline)) { body(it, buf, std::true_type()); });
    turns(n_it, [&]() __attribute__((always_inline)) { body(it, buf, std::false_type()); });
    sa_dma_wait_barrier<0>();

    if constexpr (HS > 1) {
        // the waves that share keys add up, head HS - 1 first, one product's sums at a time
        float *red = reinterpret_cast<float *>(&s_t[0][0][0][0]);
        static_assert(kBufs * HS * 2 * kSaTileB >= 4 * 64 * 64 * 4, "the sums of four waves");
        float *mine = red + wave * 4096, *next = mine + 4096;
        for (int pass = 0; pass < 2; pass++) {
            for (int w = HS - 1; w >= 1; w--) {
                if (hs == w)
#pragma unroll
                    for (int db = 0; db < 4; db++)
#pragma unroll
                        for (int c = 0; c < 16; c++) mine[(db * 16 + c) * 64 + lane] = pass == 0 ? av[db][c] : ak[db][c];
                __syncthreads();
                if (hs == w - 1)
#pragma unroll
                    for (int db = 0; db < 4; db++)
#pragma unroll
                        for (int c = 0; c < 16; c++) {
                            if (pass == 0) av[db][c] += next[(db * 16 + c) * 64 + lane];
                            else ak[db][c] += next[(db * 16 + c) * 64 + lane];
                        }
                __syncthreads();
            }
        }
        float *rg = &s_ld[0][0][0];
        __syncthreads();
        rg[wave * 64 + lane] = dg_acc;
        __syncthreads();
        if (hs != 0) return;
#pragma unroll
        for (int w = 1; w < HS; w++) dg_acc += rg[(wave + w) * 64 + lane];
    }
    const float tot = dg_acc + __shfl_xor(dg_acc, 32);
    if (jg < T) {
        const size_t krow = (size_t)(base + jg) * a.Hkv + h;
        float *opv = a.dv + krow * kSaD, *opk = a.dk + krow * kSaD;
#pragma unroll
        for (int db = 0; db < 4; db++)
#pragma unroll
            for (int j = 0; j < 4; j++) {
                *reinterpret_cast<float4 *>(opv + 32 * db + 8 * j + 4 * half) =
                    make_float4(av[db][4 * j], av[db][4 * j + 1], av[db][4 * j + 2], av[db][4 * j + 3]);
                *reinterpret_cast<float4 *>(opk + 32 * db + 8 * j + 4 * half) =
                    make_float4(ak[db][4 * j] * a.scale, ak[db][4 * j + 1] * a.scale, ak[db][4 * j + 2] * a.scale,
                                ak[db][4 * j + 3] * a.scale);
            }
        if (half == 0) a.dg[krow] = gk > 0.0f ? tot / (gk + a.eps) : 0.f;
    }
}

// ---------------------------------------------------------------------------------------------
static bool soft_fill(SoftSeqs &cs, int n_seqs, const int32_t *n_tokens, int *max_t, int64_t *total) {
    if (n_seqs < 0 || n_seqs > kMaxCallSeqs) return false;
    cs.n = n_seqs;
    int64_t tot = 0;
    int mx = 0;
    for (int b = 0; b < n_seqs; b++) {
        if (n_tokens[b] < 0) return false;
        cs.ntok[b] = n_tokens[b];
        cs.base[b] = (int32_t)tot;
        tot += n_tokens[b];
        if (tot >= ((int64_t)1 << 24)) return false;  // keeps every packed row index far inside 32 bits
        mx = max(mx, n_tokens[b]);
    }
    *max_t = mx;
    *total = tot;
    return true;
}

size_t soft_attn_ws_bytes(int64_t total_tokens, int n_q_heads) {
    return (size_t)((total_tokens * n_q_heads * 4 + 255) / 256) * 256;
}

// Blocks of 32 positions that share a key tile in the forward and the dQ kernel.  One (four waves, two blocks per compute
// unit) ends more evenly and meets at its barrier with fewer waves: forward, one / two, in us, 8 kv heads: 1 x 1000
// tokens 36 / 46, 1 x 3000 107 / 114, 4 x 2000 195 / 214, 7 x 1500 210 / 237.  Two halve the traffic into LDS, which
// is worth more once the launch runs long: 1 x 12000 1340 / 1317, 1 x 16384 2669 / 2637 (dQ 3354 / 3253).  (256 compute units.)
static int soft_row_blocks(int max_t) { return max_t >= 8192 ? 2 : 1; }

hipError_t launch_soft_attn_fwd(int n_seqs, const int32_t *n_tokens, int Hq, int Hkv, int d, int W,
                                const void *q, const void *k, const void *v, const float *g, float scale,
                                float eps, float *out, float *lse, hipStream_t st) {
    if (d != kSaD || Hq != Hkv * kSaG) return hipErrorNotSupported;
    SoftSeqs cs;
    int max_t;
    int64_t total;
    if (!soft_fill(cs, n_seqs, n_tokens, &max_t, &total)) return hipErrorInvalidValue;
    if (max_t == 0) return hipSuccess;
    SoftArgs a = {};
    a.Hq = Hq; a.Hkv = Hkv; a.W = min(W, 1 << 24);
    a.scale = scale; a.scale_log2e = scale * 1.4426950408889634f; a.eps = eps;
    a.q = (const char *)q; a.k = (const char *)k; a.v = (const char *)v; a.g = g;
    a.out = out; a.lse = lse;
    a.nx = (max_t + 32 * soft_row_blocks(max_t) - 1) / (32 * soft_row_blocks(max_t));
    if (soft_row_blocks(max_t) == 2)
        hipLaunchKernelGGL(soft_attn_fwd_kernel<2>, dim3(a.nx * Hkv * n_seqs), dim3(512), 0, st, cs, a);
    else
        hipLaunchKernelGGL(soft_attn_fwd_kernel<1>, dim3(a.nx * Hkv * n_seqs), dim3(256), 0, st, cs, a);
    return hipGetLastError();
}

hipError_t launch_soft_attn_bwd(int n_seqs, const int32_t *n_tokens, int Hq, int Hkv, int d, int W,
                                const void *q, const void *k, const void *v, const float *g, float scale,
                                float eps, const float *out, const float *lse, const void *dout, float *dq,
                                float *dk, float *dv, float *dg, void *ws, hipStream_t st) {
    if (d != kSaD || Hq != Hkv * kSaG) return hipErrorNotSupported;
    SoftSeqs cs;
    int max_t;
    int64_t total;
    if (!soft_fill(cs, n_seqs, n_tokens, &max_t, &total)) return hipErrorInvalidValue;
    if (max_t == 0) return hipSuccess;
    SoftArgs a = {};
    a.Hq = Hq; a.Hkv = Hkv; a.W = min(W, 1 << 24);
    a.scale = scale; a.scale_log2e = scale * 1.4426950408889634f; a.eps = eps;
    a.q = (const char *)q; a.k = (const char *)k; a.v = (const char *)v; a.g = g;
    a.out = const_cast<float *>(out); a.lse = const_cast<float *>(lse);
    a.dout = (const char *)dout;
    a.rowdot = (float *)ws;
    a.dq = dq; a.dk = dk; a.dv = dv; a.dg = dg;
    const int64_t n_rows = total * Hq;
    hipLaunchKernelGGL(soft_attn_rowdot_kernel, dim3((unsigned)((n_rows + 7) / 8)), dim3(256), 0, st, n_rows,
                       a.dout, out, a.rowdot);
    hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
    a.nx = (max_t + 32 * soft_row_blocks(max_t) - 1) / (32 * soft_row_blocks(max_t));
    if (soft_row_blocks(max_t) == 2)
        hipLaunchKernelGGL(soft_attn_bwd_dq_kernel<2>, dim3(a.nx * Hkv * n_seqs), dim3(512), 0, st, cs, a);
    else
        hipLaunchKernelGGL(soft_attn_bwd_dq_kernel<1>, dim3(a.nx * Hkv * n_seqs), dim3(256), 0, st, cs, a);
    e = hipGetLastError();
    if (e != hipSuccess) return e;
    // Waves that share keys (HS): the time of a short call is that of its longest block, the one of the first keys, so
    // blocks of a fraction of the length pay as long as compute units are idle or HS = 1 would run in one go (two
    // blocks per compute unit, 256 of these); past that the single read of a tile for 128 keys is worth more.  Adding up what
    // four waves have takes some 25 us more than a long block saves below 400 tokens.  Backward, HS = 1 / 2 / 4, in us, 8 kv heads:
    // 1 x 64 tokens 34 / 29 / 46, 16 x 64 45 / 39 / 57, 32 x 128 111 / 121 / 217, 1 x 300 110 / 71 / 72, 16 x 300 196 / 194 / 304,
    // 1 x 500 158 / 96 / 89, 4 x 500 184 / 124 / 163, 1 x 1000 267 / 158 / 136, 2 x 1000 290 / 182 / 193, 4 x 1000 329 / 301 / 345,
    // 8 x 1000 457 / 520 / 667, 1 x 2000 478 / 284 / 261, 1 x 3000 691 / 419 / 476, 1 x 8000 2306 / 2203 / 2688,
    // 1 x 9000 2759 / 2773 / 3446, 1 x 12000 4374 / 4831 / 5869.
    const int64_t n_wide = (int64_t)((max_t + 127) / 128) * Hkv * n_seqs;  // blocks of HS = 1
    if (n_wide <= (max_t >= 2000 ? 128 : max_t >= 400 ? 64 : 0)) {
        a.nx = (max_t + 31) / 32;
        hipLaunchKernelGGL(soft_attn_bwd_dkv_kernel<4>, dim3(a.nx * Hkv * n_seqs), dim3(256), 0, st, cs, a);
    } else if (n_wide <= (max_t >= 2000 ? 512 : max_t > 128 ? 384 : 192)) {
        a.nx = (max_t + 63) / 64;
        hipLaunchKernelGGL(soft_attn_bwd_dkv_kernel<2>, dim3(a.nx * Hkv * n_seqs), dim3(256), 0, st, cs, a);
    } else {
        a.nx = (max_t + 127) / 128;
        hipLaunchKernelGGL(soft_attn_bwd_dkv_kernel<1>, dim3(a.nx * Hkv * n_seqs), dim3(256), 0, st, cs, a);
    }
    return hipGetLastError();
}

// ---------------------------------------------------------------------------------------------
// Sparsity term of the training objective (Sec. 3.3): sum over the given scores of
// (g + g (1 - g)) / n_total and its derivative (2 - 2 g) / n_total.  Two launches with a fixed
// order of additions (per-thread strided sums, block tree, then one wave over the blocks in
// double), so the value repeats bit for bit.
// ---------------------------------------------------------------------------------------------
constexpr int kSpBlocks = 1024;

__global__ __launch_bounds__(256) void sparsity_partial_kernel(const float *g, int64_t n, float inv_n, float *dg,
                                                               float *partial) {
    __shared__ float s_red[256];
    float acc = 0.f;
    for (int64_t x = (int64_t)blockIdx.x * 256 + threadIdx.x; x < n; x += (int64_t)gridDim.x * 256) {
        const float v = g[x];
        acc += v + v * (1.0f - v);
        if (dg) dg[x] = (2.0f - 2.0f * v) * inv_n;
    }
    s_red[threadIdx.x] = acc;
    __syncthreads();
    for (int o = 128; o > 0; o >>= 1) {
        if ((int)threadIdx.x < o) s_red[threadIdx.x] += s_red[threadIdx.x + o];
        __syncthreads();
    }
    if (threadIdx.x == 0) partial[blockIdx.x] = s_red[0];
}

// One wave: a lane adds up every 64th partial, then the lanes in pairs, all in double.  (One thread over all of them waited for a
// load and an addition 1024 times: 24 us of 16K tokens, now 5.)
__global__ __launch_bounds__(64) void sparsity_final_kernel(const float *partial, int nb, double inv_n, float *loss) {
    double t = 0.0;
#pragma unroll
    for (int i = 0; i < kSpBlocks / 64; i++) {
        const int at = i * 64 + (int)threadIdx.x;
        t += at < nb ? (double)partial[at] : 0.0;
    }
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) t += __shfl_xor(t, o);
    if (threadIdx.x == 0) *loss = (float)(t * inv_n);
}

size_t sparsity_ws_bytes() { return kSpBlocks * sizeof(float); }

hipError_t launch_sparsity_loss(const float *g, int64_t n, int64_t n_total, float *loss, float *dg, void *ws,
                                hipStream_t st) {
    const int nb = (int)std::min<int64_t>(kSpBlocks, std::max<int64_t>(1, (n + 255) / 256));
    const double inv = 1.0 / (double)n_total;
    hipLaunchKernelGGL(sparsity_partial_kernel, dim3(nb), dim3(256), 0, st, g, n, (float)inv, dg, (float *)ws);
    hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
    hipLaunchKernelGGL(sparsity_final_kernel, dim3(1), dim3(64), 0, st, (const float *)ws, nb, inv, loss);
    return hipGetLastError();
}

}  // namespace wgkv
