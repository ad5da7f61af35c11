// Chunk attention under the vertical-slash mask (Sec. 4.2 "Vertical-slash sparse attention"; mask equation of
// Sec. 4.2 on the attention of Sec. 2.1) for fp32 pools, on the fp32 matrix instruction
// v_mfma_f32_32x32x2_f32: products and sums are fp32, nothing is rounded to a shorter type.
//
// One block = 32 chunk positions of one query head.  Its keys are, in this order, the head's global cache (all
// visible: admitted and older than every window of the chunk), the ring (oldest position first), the admitted chunk
// keys that no window of the block reaches (picked out beforehand, as for bf16 pools) and the rest of the chunk up to
// the block's last query; a ring or chunk key at position p is visible to the query at position i iff i - p < W or its
// score >= tau.  The waves of the block take the tiles of 32 keys in turn and are folded once at the end: the
// matrix instruction is so slow (64 clocks for 4096 multiply-adds) that a tile of 64-element heads occupies a SIMD for
// 4096 clocks, so a short call needs its keys spread over the SIMDs, and sharing a tile between waves would gain
// nothing: the 16 KiB of a tile's rows per 4096 clocks and wave come out of the L2.  Measured on 512 tokens of 8 / 2
// heads of 64, window 64 / 1024, lists included: 67 / 112 us with one wave of plain arithmetic per (query, head), 15 / 19 here.
//
// The block's queries sit in LDS (in the space that the fold uses at the end): the accumulators of 128 elements, a key
// row's half and the weights leave no registers for them.
//
// S^T = K Q^T and O^T = V^T P^T.  The instruction contracts two elements, one from each half of the wave.  The first
// product takes element ks from half 0 and D/2 + ks from half 1, so that a lane reads D/2 consecutive floats of its
// key's row (and of its query's); the second takes the keys 8j + i and 8j + 4 + i, whose weights are exactly where the
// first product left them, so P needs no exchange at all.
#include <climits>

#include "wgkv_dev.h"

namespace wgkv {

typedef __attribute__((ext_vector_type(16))) float pw_f32x16_t;

hipError_t launch_prefill_look(const View &pv, const CallSeqs &cs, int layer, float tau, const float *g, void *ws,
                               size_t ws_bytes, bool need_order, const int32_t **order, const int32_t **pick, const int32_t **picked,
                               hipStream_t st);

struct PrefillF32Args {
    int32_t first[kMaxCallSeqs + 1];  // position tiles of the sequences before sequence b
    int layer;
    float tau, scale_log2e;
    const char *q, *k, *v;  // chunk tensors, fp32
    const float *g;         // chunk scores
    const int32_t *pick, *picked;  // admitted chunk positions of every unit and their counts, or NULL
    float *out;
};

template <int D, int NW>
__global__ __launch_bounds__(NW * 64, 2) void attend_prefill_f32_kernel(View pv, CallSeqs cs, PrefillF32Args a) {
    constexpr int H2 = D / 2, DB = D / 32, OS = D + 4;  // OS: floats per output row in LDS (padded against bank conflicts)
    constexpr int ROWB = D * 4;
    __shared__ __attribute__((aligned(16))) uint64_t s_vp[NW][2][32];  // V row of every key of a wave's tile (two tiles)
    __shared__ __attribute__((aligned(16))) int s_lo[NW][2][32], s_hi[NW][2][32];  // first and last position that sees it
    __shared__ float s_m[NW][32], s_l[NW][32];
    __shared__ __attribute__((aligned(16))) float s_o[NW][32 * OS];
    // all query heads of a position tile next to each other (they share K and V), a sequence's latest positions first
    const int x = (int)blockIdx.x / pv.Hq, qh = (int)blockIdx.x % pv.Hq, h = qh / pv.G;
    int b = 0;
    for (int hi = cs.n - 1; b < hi;) {  // the last sequence whose tiles begin at or before tile x (not one without tokens)
        const int mid = (b + hi + 1) >> 1;
        if (a.first[mid] <= x) b = mid; else hi = mid - 1;
    }
    const int qt = a.first[b + 1] - 1 - x;
    const int T = cs.ntok[b], t0 = cs.t0[b], base = cs.base[b];
    const int um = unit_meta(pv, cs.sid[b], a.layer, h);
    const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int n = lane & 31, half = lane >> 5;
    const int gl = pv.global_len[um];
    const int w_eff = min(pv.W, t0);              // ring entries that exist
    const int slot0 = t0 > pv.W ? t0 % pv.W : 0;  // ring slot of the oldest position
    const int i_end = min(T, qt * 32 + 32);       // chunk keys this block can see
    const int near = a.pick ? max(0, qt * 32 - pv.W + 1) / 32 * 32 : 0;  // no window of the block reaches below
    const int32_t *pick = a.pick + (a.pick ? pick_of(pv.Hkv, b, h, base, T) : 0);
    const int n_far = near > 0 ? a.picked[picked_of(pv.Hkv, b, h, base, T) + near / 32] : 0;
    const int n_g = (gl + 31) / 32, n_r = (w_eff + 31) / 32;
    const int t_far = n_g + n_r, t_near = t_far + (n_far + 31) / 32, n_tiles = t_near + (i_end - near + 31) / 32;
    const int n_plain = gl / 32;                  // full tiles of the global cache: no mask, nor for full picked ones
    const int t_plain = t_far + n_far / 32;
    const int qpos = t0 + min(qt * 32 + n, T - 1);

    float *s_q = &s_o[0][0];  // [32][OS] until the fold
    for (int e = threadIdx.x; e < 32 * (D / 4); e += NW * 64) {
        const int row = e / (D / 4), c = e % (D / 4);
        const float4 x = *reinterpret_cast<const float4 *>(
            a.q + ((size_t)(base + min(qt * 32 + row, T - 1)) * pv.Hq + qh) * ROWB + 16 * c);
        *reinterpret_cast<float4 *>(&s_q[row * OS + 4 * c]) = x;
    }
    __syncthreads();
    const float *q_half = s_q + n * OS + half * H2;
    // Lane n looks after key n of a tile.  page_of: the page its row sits in (a picked key: its position), one load; locate: the row's
    // address and who sees it.  A key past the end of its region repeats the region's last one, invisibly.
    auto page_of = [&](int t) __attribute__((always_inline)) {
        if (t < n_g) return pv.global_pt[(size_t)um * pv.maxgp + (min(t * 32 + n, gl - 1) >> pv.logP)];
        if (t < t_far) {
            int slot = slot0 + min((t - n_g) * 32 + n, w_eff - 1);
            slot = slot >= pv.W ? slot - pv.W : slot;
            return pv.local_pt[(size_t)um * pv.nlp + (slot >> pv.logP)];
        }
        return t < t_near ? pick[min((t - t_far) * 32 + n, n_far - 1)] : -1;
    };
    auto locate = [&](int t, int pg, int buf) __attribute__((always_inline)) {
        const char *kp, *vp;
        int lo = INT_MAX, hi = INT_MAX;  // invisible unless shown otherwise
        if (t < n_g) {
            const int idx = t * 32 + n, idc = min(idx, gl - 1);
            kp = page_ptr(pv, pg) + (size_t)(idc & (pv.P - 1)) * ROWB;
            vp = kp + pv.v_off;
            if (idx < gl) lo = INT_MIN;
        } else if (t < t_far) {
            const int idx = (t - n_g) * 32 + n, idc = min(idx, w_eff - 1);
            int slot = slot0 + idc;
            slot = slot >= pv.W ? slot - pv.W : slot;
            kp = page_ptr(pv, pg) + (size_t)(slot & (pv.P - 1)) * ROWB;
            vp = kp + pv.v_off;
            if (idx < w_eff) {
                lo = t0 - w_eff + idx;
                hi = (pv.ring_g[(size_t)um * pv.W + slot] >= a.tau) ? INT_MAX : lo + pv.W - 1;
            }
        } else if (t < t_near) {
            const size_t row = (size_t)(base + pg) * pv.Hkv + h;
            kp = a.k + row * ROWB;
            vp = a.v + row * ROWB;
            if ((t - t_far) * 32 + n < n_far) lo = INT_MIN;
        } else {
            const int idx = near + (t - t_near) * 32 + n, idc = min(idx, T - 1);
            const size_t row = (size_t)(base + idc) * pv.Hkv + h;
            kp = a.k + row * ROWB;
            vp = a.v + row * ROWB;
            if (idx < T) {
                lo = t0 + idx;
                hi = (a.g[row] >= a.tau) ? INT_MAX : lo + pv.W - 1;
            }
        }
        if (half == 0) {
            s_vp[wave][buf][n] = (uint64_t)(uintptr_t)vp;
            s_lo[wave][buf][n] = lo;
            s_hi[wave][buf][n] = hi;
        }
        return kp + half * (H2 * 4);
    };
    float4 kv[H2 / 4];
    auto load_k = [&](const char *kp) __attribute__((always_inline)) {
#pragma unroll
        for (int c = 0; c < H2 / 4; c++) kv[c] = *reinterpret_cast<const float4 *>(kp + 16 * c);
    };

    pw_f32x16_t o[DB];
    float m = -INFINITY, l = 0.f;
#pragma unroll
    for (int db = 0; db < DB; db++)
#pragma unroll
        for (int c = 0; c < 16; c++) o[db][c] = 0.f;
    int buf = 0;
    if (wave < n_tiles) load_k(locate(wave, page_of(wave), 0));
    for (int t = wave; t < n_tiles; t += NW, buf ^= 1) {  // wave-uniform; no barrier inside
        const bool masked = t >= n_plain && (t < t_far || t >= t_plain);
        const int tn = min(t + NW, n_tiles - 1);          // the tile asked for next (the last one again at the end)
        const int pgn = page_of(tn);
        pw_f32x16_t s;
#pragma unroll
        for (int c = 0; c < 16; c++) s[c] = 0.f;
#pragma unroll
        for (int c = 0; c < H2 / 4; c++) {
            const float4 qv = *reinterpret_cast<const float4 *>(q_half + 4 * c);
            s = __builtin_amdgcn_mfma_f32_32x32x2f32(kv[c].x, qv.x, s, 0, 0, 0);
            s = __builtin_amdgcn_mfma_f32_32x32x2f32(kv[c].y, qv.y, s, 0, 0, 0);
            s = __builtin_amdgcn_mfma_f32_32x32x2f32(kv[c].z, qv.z, s, 0, 0, 0);
            s = __builtin_amdgcn_mfma_f32_32x32x2f32(kv[c].w, qv.w, s, 0, 0, 0);
        }
        load_k(locate(tn, pgn, buf ^ 1));  // in flight during the softmax and the second product
        __builtin_amdgcn_wave_barrier();
        // register 4j+i holds key 8j + 4*half + i of the tile
        float sc[16], mt = -INFINITY;
        uint32_t seen = 0xffffu;  // bit c: the query sees the key of register c
#pragma unroll
        for (int c = 0; c < 16; c++) sc[c] = s[c] * a.scale_log2e;
        if (masked) {
#pragma unroll
            for (int j = 0; j < 4; j++) {
                const int4 lo4 = *reinterpret_cast<const int4 *>(&s_lo[wave][buf][8 * j + 4 * half]);
                const int4 hi4 = *reinterpret_cast<const int4 *>(&s_hi[wave][buf][8 * j + 4 * half]);
                const int lo_[4] = {lo4.x, lo4.y, lo4.z, lo4.w}, hi_[4] = {hi4.x, hi4.y, hi4.z, hi4.w};
#pragma unroll
                for (int i = 0; i < 4; i++) {
                    const bool vis = qpos >= lo_[i] && qpos <= hi_[i];
                    sc[4 * j + i] = vis ? sc[4 * j + i] : -INFINITY;
                    seen &= ~((vis ? 0u : 1u) << (4 * j + i));
                }
            }
        }
#pragma unroll
        for (int c = 0; c < 16; c++) mt = fmaxf(mt, sc[c]);
        mt = fmaxf(mt, __shfl_xor(mt, 32));
        const float mnew = fmaxf(m, mt), msafe = mnew == -INFINITY ? 0.f : mnew;
        const float corr = __builtin_amdgcn_exp2f(m - msafe);
        float ps = 0.f;
#pragma unroll
        for (int c = 0; c < 16; c++) {
            sc[c] = __builtin_amdgcn_exp2f(sc[c] - msafe);
            ps += sc[c];
        }
        l = l * corr + ps;
        if (__builtin_amdgcn_ballot_w64(mnew > m) != 0) {
#pragma unroll
            for (int db = 0; db < DB; db++)
#pragma unroll
                for (int c = 0; c < 16; c++) o[db][c] *= corr;
        }
        m = mnew;
        // VB keys of the lane's half at a time, their rows requested together
        constexpr int VB = D == 64 ? 4 : 2;
        bool bad = false;  // a masked tile holds a value that is not finite: a weight of zero does not keep it out
#pragma unroll
        for (int c0 = 0; c0 < 16; c0 += VB) {
            float vv[VB][DB];
#pragma unroll
            for (int i = 0; i < VB; i++) {
                const int c = c0 + i, key = 8 * (c / 4) + 4 * half + c % 4;
                const float *vp = reinterpret_cast<const float *>((uintptr_t)s_vp[wave][buf][key]) + n;
#pragma unroll
                for (int db = 0; db < DB; db++) vv[i][db] = vp[32 * db];
            }
            if (masked) {
#pragma unroll
                for (int i = 0; i < VB; i++)
#pragma unroll
                    for (int db = 0; db < DB; db++) {
                        const bool fin = fabsf(vv[i][db]) < INFINITY;
                        bad = bad || !fin;
                        vv[i][db] = fin ? vv[i][db] : 0.f;
                    }
            }
#pragma unroll
            for (int i = 0; i < VB; i++)
#pragma unroll
                for (int db = 0; db < DB; db++)
                    o[db] = __builtin_amdgcn_mfma_f32_32x32x2f32(vv[i][db], sc[c0 + i], o[db], 0, 0, 0);
        }
        if (__builtin_amdgcn_ballot_w64(bad) != 0) {
            // what the queries that do see them get: counts of +inf, -inf and NaN in one product (at most 32 of
            // each: 1, 64 and 4096 apiece), then the value that the sum would have had
#pragma unroll 1
            for (int db = 0; db < DB; db++) {
                pw_f32x16_t cnt;
#pragma unroll
                for (int c = 0; c < 16; c++) cnt[c] = 0.f;
#pragma unroll
                for (int c = 0; c < 16; c++) {
                    const float x = reinterpret_cast<const float *>(
                        (uintptr_t)s_vp[wave][buf][8 * (c / 4) + 4 * half + c % 4])[32 * db + n];
                    const float code = x == INFINITY ? 1.f : x == -INFINITY ? 64.f : x != x ? 4096.f : 0.f;
                    cnt = __builtin_amdgcn_mfma_f32_32x32x2f32(code, (float)((seen >> c) & 1u), cnt, 0, 0, 0);
                }
#pragma unroll
                for (int d2 = 0; d2 < DB; d2++)
#pragma unroll
                    for (int c = 0; c < 16; c++)
                        if (d2 == db && cnt[c] > 0.f)
                            o[d2][c] += cnt[c] < 64.f ? INFINITY : (cnt[c] < 4096.f && fmodf(cnt[c], 64.f) == 0.f) ? -INFINITY : NAN;
            }
        }
        __builtin_amdgcn_wave_barrier();
    }
    // ---- fold the waves: register 4j+i of o[db] is d = 32*db + 8j + 4*half + i of query n ----
    l += __shfl_xor(l, 32);
    __syncthreads();  // every wave is done with the queries
    if (half == 0) {
        s_m[wave][n] = m;
        s_l[wave][n] = l;
    }
#pragma unroll
    for (int db = 0; db < DB; db++)
#pragma unroll
        for (int j = 0; j < 4; j++)
            *reinterpret_cast<float4 *>(&s_o[wave][n * OS + 32 * db + 8 * j + 4 * half]) =
                make_float4(o[db][4 * j], o[db][4 * j + 1], o[db][4 * j + 2], o[db][4 * j + 3]);
    __syncthreads();
    for (int e = threadIdx.x; e < 32 * (D / 4); e += NW * 64) {
        const int col = e / (D / 4), d4 = e % (D / 4), i = qt * 32 + col;
        if (i >= T) continue;
        float M = s_m[0][col], L = 0.f;
#pragma unroll
        for (int w = 1; w < NW; w++) M = fmaxf(M, s_m[w][col]);  // finite: a query sees itself
        float4 acc = make_float4(0.f, 0.f, 0.f, 0.f);
#pragma unroll
        for (int w = 0; w < NW; w++) {
            const float f = __builtin_amdgcn_exp2f(s_m[w][col] - M);  // 0 for a wave that saw nothing
            const float4 x = *reinterpret_cast<const float4 *>(&s_o[w][col * OS + 4 * d4]);
            L = fmaf(s_l[w][col], f, L);
            acc.x = fmaf(x.x, f, acc.x); acc.y = fmaf(x.y, f, acc.y);
            acc.z = fmaf(x.z, f, acc.z); acc.w = fmaf(x.w, f, acc.w);
        }
        const float inv = 1.0f / L;
        *reinterpret_cast<float4 *>(a.out + ((size_t)(base + i) * pv.Hq + qh) * D + 4 * d4) =
            make_float4(acc.x * inv, acc.y * inv, acc.z * inv, acc.w * inv);
    }
}

hipError_t launch_attend_prefill_f32(const View &pv, const CallSeqs &cs, int layer, const void *q, const void *k,
                                     const void *v, const float *g, float tau, float scale, float *out, void *ws,
                                     size_t ws_bytes, hipStream_t st) {
    if (pv.dtype != WGKV_F32) return hipErrorNotSupported;
    PrefillF32Args a;
    a.layer = layer;
    a.tau = tau;
    a.scale_log2e = scale * 1.4426950408889634f;
    a.q = (const char *)q;
    a.k = (const char *)k;
    a.v = (const char *)v;
    a.g = g;
    a.out = out;
    int max_t = 0;
    a.first[0] = 0;
    for (int b = 0; b < cs.n; b++) {
        max_t = max(max_t, cs.ntok[b]);
        a.first[b + 1] = a.first[b] + (cs.ntok[b] + 31) / 32;
    }
    if (max_t == 0) return hipSuccess;
    a.pick = a.picked = nullptr;
    if (max_t > pv.W) {
        const int32_t *order;
        const hipError_t e = launch_prefill_look(pv, cs, layer, tau, g, ws, ws_bytes, false, &order, &a.pick, &a.picked, st);
        if (e != hipSuccess) return e;
    }
    // Blocks for the tiles that there are: a launch holds fewer than 2^32 threads, and one long chunk beside many short ones
    // would be over that if every sequence had the blocks of the longest.
    const int64_t blocks = (int64_t)a.first[cs.n] * pv.Hq;
    if (blocks * (pv.d == 64 ? 512 : 256) >= ((int64_t)1 << 32)) return hipErrorInvalidValue;
    // eight waves of 64-element heads fill the block's 64 KiB of folded outputs, four of 128-element heads do
    if (pv.d == 64)
        hipLaunchKernelGGL((attend_prefill_f32_kernel<64, 8>), dim3((unsigned)blocks), dim3(512), 0, st, pv, cs, a);
    else if (pv.d == 128)
        hipLaunchKernelGGL((attend_prefill_f32_kernel<128, 4>), dim3((unsigned)blocks), dim3(256), 0, st, pv, cs, a);
    else
        return hipErrorNotSupported;
    return hipGetLastError();
}

}  // namespace wgkv
