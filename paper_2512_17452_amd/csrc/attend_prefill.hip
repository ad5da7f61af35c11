// Chunked-prefill attention under the vertical-slash mask (Sec. 4.2 mask equation)
// on the gfx950 matrix cores.
//
// Query i of the chunk (position t0+i) of a kv head's group sees
//   - every entry of the head's global cache (admitted tokens older than the window),
//   - ring positions j in [t0-W, t0) with  pos_i - j < W  or stored g_j >= tau,
//   - chunk keys j <= i with  i - j < W  or g_j >= tau,
// which is exactly M_ij restricted to what is still known about the past: tokens
// that were neither admitted nor inside the window are gone (Sec. 4.2, "Initial
// cache population") and are invisible under M_ij anyway.
//
// What a block reads: the global cache, the ring, and of the chunk the keys that some window of the
// block reaches, plus those older ones that are admitted.  The latter are picked out by a small kernel
// in front (one list of admitted chunk positions per unit), so that tiles are full of keys that every
// query of the block sees, instead of running over the whole chunk with a mask (4096-token chunks at an
// admission rate of a half, 0-12K tokens before them: 1095 -> 803 us per chunk of two prompts, lists included).
//
// attend_prefill_kernel (every shape but the one of the paper's models): one block owns 256 / G chunk
// positions of one (sequence, kv head) with a group of G query heads;
// its eight waves are (query head of the group) x (row block of 32 positions), so a K/V tile staged
// in LDS feeds all of them and two waves share each SIMD.  A tile is 8 KiB of K and of V (16 bytes of
// each per thread): 32 keys of 128 elements, 64 keys of 64.
// K and V tiles are staged row-major; the V^T operand is read from the V tile with the
// transposing LDS load.  Everything is computed transposed, S^T = K Q^T and O^T = V^T P^T with
// v_mfma_f32_32x32x16_bf16: a lane then owns one query column, so the running max,
// the denominator and the rescale factor are plain per-lane scalars, and the
// probabilities leave the first product already in the operand layout of the second.
//
// Two forms of the weights P.  For the shape of the paper's models (128 wide, four heads a group;
// attend_prefill_tiles_kernel) they are rounded to bf16 once, and the denominator sums the rounded ones.  For
// every other shape they keep 24 bits: p = hi + mid + lo, each part the upper half of an fp32 word and hi, mid
// exact remainders, three products with the same V^T operand; V is bf16, so the products are exact and
// the sums are fp32 as they are in plain fp32 arithmetic.  The matrix cores have the room: at 64 elements
// the vector work per score is twice the four extra products.  Measured: a 6001-token prompt of 32 / 8 heads
// of 64 in chunks of 2048, gate and admission included, 17.3 ms -> 0.40 ms against one wave of plain fp32
// arithmetic per (query, head), the error against 64 bits 9.3e-7 -> 6.4e-7.
#include <algorithm>
#include <climits>
#include <type_traits>

#include "lds_tiles.h"
#include "wgkv_dev.h"

namespace wgkv {

typedef __attribute__((ext_vector_type(8))) __bf16 pf_bf16x8_t;
typedef __attribute__((ext_vector_type(2))) __bf16 pf_bf16x2_t;
typedef __attribute__((ext_vector_type(16))) float pf_f32x16_t;

// The shape of one instantiation: head_dim D, group size G.
template <int D_, int G_>
struct PfShape {
    static constexpr int D = D_, G = G_;
    static constexpr int Q = 256 / G;       // chunk positions per block (8 / G row blocks of 32)
    static constexpr int CPR = D / 8;       // 16-byte chunks per row
    static constexpr int KT = 512 / CPR;    // keys per tile: a chunk of K and of V per thread
    static constexpr int NS = KT / 32;      // score tiles of 32 keys
    static constexpr int KS = D / 16;       // contraction slices of the first product
    static constexpr int DB = D / 32;       // output blocks of 32 elements
    static constexpr int KPW = 64 / CPR;    // keys a wave stages
    static constexpr int KStride = D * 2 + 16;  // bytes per key row of the K tile in LDS: rows are read whole
    static constexpr int VStride = D * 2 + 64;  // bytes per key row of the V tile: columns are read, four rows and
                                                // 64 bytes of each at a time per half wave, which this stride
                                                // (320 or 192 bytes) spreads over all banks
};

struct PrefillAttnArgs {
    int nx;                 // blocks per (sequence, kv head) of the launch
    int rank0;              // place in the order of the launch's first unit
    int ordered;            // else the units in their own order, and `order` is only somewhere to read from
    const int32_t *order;   // [n_units] (sequence, kv head) units, the one with the longest global cache first
    const int32_t *pick;    // admitted chunk positions of every unit, ascending (pick_of), or NULL
    const int32_t *picked;  // how many of them lie below position 32 i, for every i (picked_of)
    int layer;
    float tau;
    float scale_log2e;
    const char *q, *k, *v;  // chunk tensors, bf16
    const float *g;         // chunk scores
    float *out;
};

// A operand of O^T += V^T P^T from the row-major V tile: the output row of this lane is
// d = db*32 + qn, its 8 contraction slots are keys r0 + 4*half + {0..3} and r0 + 8 + 4*half + {0..3}
// of the tile.  ds_read_b64_tr_b16 transposes inside groups of 16 lanes: lane i of a group receives
// element i%4 of the 8 bytes addressed by lanes i/4, 4 + i/4, 8 + i/4 and 12 + i/4, so lane s of a
// group addresses (key s/4 of the four, columns 4*(s%4)..+3 of the group's 16).
typedef short pf_s16x4_t __attribute__((ext_vector_type(4)));
template <int STRIDE>
__device__ __forceinline__ pf_bf16x8_t pf_get_cols(const char *tile, int lane, int db, int r0) {
    const int half = lane >> 5;
    const char *p = tile + (r0 + 4 * half + ((lane & 15) >> 2)) * STRIDE +
                    (db * 32 + 16 * ((lane >> 4) & 1) + 4 * (lane & 3)) * 2;
    typedef pf_s16x4_t __attribute__((address_space(3))) *lds_ptr_t;
    const pf_s16x4_t lo = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_ptr_t)p);
    const pf_s16x4_t hi = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_ptr_t)(p + 8 * STRIDE));
    const uint2 l2 = __builtin_bit_cast(uint2, lo), h2 = __builtin_bit_cast(uint2, hi);
    const uint4 u4 = make_uint4(l2.x, l2.y, h2.x, h2.y);
    return __builtin_bit_cast(pf_bf16x8_t, u4);
}

__device__ __forceinline__ uint32_t pf_pack(float lo, float hi) {
    pf_bf16x2_t t = {(__bf16)lo, (__bf16)hi};
    return __builtin_bit_cast(uint32_t, t);
}

// The upper halves of two fp32 words as one pair of bf16 (the low word first).
__device__ __forceinline__ uint32_t pf_top(float lo, float hi) {
    return __builtin_amdgcn_perm(__float_as_uint(hi), __float_as_uint(lo), 0x07060302u);
}
__device__ __forceinline__ float pf_rest(float x) { return x - __uint_as_float(__float_as_uint(x) & 0xffff0000u); }

// Eight bf16 hold an inf or a NaN: an exponent of ones carries into the bit above it.
__device__ __forceinline__ bool pf_nonfinite(const uint4 &x) {
    constexpr uint32_t kExp = 0x7f807f80u, kOne = 0x00800080u;
    return ((((x.x & kExp) + kOne) | ((x.y & kExp) + kOne) | ((x.z & kExp) + kOne) | ((x.w & kExp) + kOne)) & 0x80008000u) != 0u;
}
// Takes the infinities and NaNs out of an operand of V^T and gives them to the columns of o that see their keys (seen:
// bf16 ones and zeros in the operand layout of P^T): one product of codes counts +inf, -inf and NaN (at most 16 of
// each: 1, 32 and 1024 apiece), then o gets what the sum would have had.
__device__ __forceinline__ void pf_take_nonfinite(pf_bf16x8_t &v, const uint32_t (&seen)[4], pf_f32x16_t &o) {
    uint4 w = __builtin_bit_cast(uint4, v);
    uint32_t x[4] = {w.x, w.y, w.z, w.w}, code[4];
#pragma unroll
    for (int i = 0; i < 4; i++) {
        code[i] = 0u;
#pragma unroll
        for (int e = 0; e < 2; e++) {
            const uint32_t h = (x[i] >> (16 * e)) & 0xffffu;
            // 1, 32 and 1024 in bf16
            const uint32_t cd = (h & 0x7f80u) != 0x7f80u ? 0u : h == 0x7f80u ? 0x3f80u : h == 0xff80u ? 0x4200u : 0x4480u;
            code[i] |= cd << (16 * e);
            if (cd) x[i] &= ~(0xffffu << (16 * e));
        }
    }
    v = __builtin_bit_cast(pf_bf16x8_t, make_uint4(x[0], x[1], x[2], x[3]));
    pf_f32x16_t cnt;
#pragma unroll
    for (int c = 0; c < 16; c++) cnt[c] = 0.f;
    cnt = __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(pf_bf16x8_t, make_uint4(code[0], code[1], code[2], code[3])),
                                                  __builtin_bit_cast(pf_bf16x8_t, make_uint4(seen[0], seen[1], seen[2], seen[3])),
                                                  cnt, 0, 0, 0);
#pragma unroll
    for (int c = 0; c < 16; c++)
        if (cnt[c] > 0.f) {
            const int n = (int)cnt[c];
            o[c] += n < 32 ? INFINITY : (n < 1024 && n % 32 == 0) ? -INFINITY : NAN;
        }
}

// Whether every query of the block (chunk positions q_first to q_last) sees every key of tile t: full tiles of the global
// cache and of the picked keys, and those of the ring and the chunk that lie inside all its windows.
__device__ __forceinline__ bool pf_no_mask(int t, int KT, int n_g, int n_plain, int t_far, int t_near, int n_far, int near,
                                           int w_eff, int W, int q_first, int q_last) {
    if (t < n_g) return t < n_plain;
    if (t < t_far) {
        const int i0 = (t - n_g) * KT;  // the oldest ring entry is w_eff positions before the chunk
        return i0 + KT <= w_eff && q_last + w_eff - i0 < W;
    }
    if (t < t_near) return t - t_far < n_far / KT;
    const int i0 = near + (t - t_near) * KT;
    return i0 + KT - 1 <= q_first && q_last - i0 < W;
}

template <int D_, int G_>
__global__ __launch_bounds__(512) void attend_prefill_kernel(View pv, CallSeqs cs, PrefillAttnArgs a) {
    using S = PfShape<D_, G_>;
    constexpr int D = S::D, G = S::G, KT = S::KT, NS = S::NS, KS = S::KS, DB = S::DB;
    __shared__ __attribute__((aligned(16))) char s_k[2][KT * S::KStride];
    __shared__ __attribute__((aligned(16))) char s_v[2][KT * S::VStride];
    __shared__ __attribute__((aligned(16))) int s_lo[2][KT];
    __shared__ __attribute__((aligned(16))) int s_hi[2][KT];
    __shared__ int s_bad[2];  // the tile in that buffer if it holds a V that is not finite

    // Blocks are handed out in the order of their index and go to the 8 XCDs round-robin: all
    // blocks of the unit with the longest global cache come first, its latest positions (which see
    // the most chunk keys) at the front, then the next unit.  Admission is head-specific, so units
    // differ several-fold in work: with the long ones at the front the launch does not end on a
    // late-started long one, and every unit is spread evenly over the XCDs (giving each XCD whole
    // heads, for the sake of its L2, leaves the XCDs as unbalanced as the heads are).
    const int rank = a.rank0 + (int)(blockIdx.x / a.nx), unit = a.ordered ? a.order[rank] : rank;
    const int b = unit / pv.Hkv, h = unit % pv.Hkv;
    const int qt = a.nx - 1 - (int)(blockIdx.x % a.nx);
    const int T = cs.ntok[b], t0 = cs.t0[b], base = cs.base[b];
    if (qt * S::Q >= T) return;  // block-uniform
    const int sid = cs.sid[b];
    const int um = unit_meta(pv, sid, a.layer, h);
    // eight waves: wave -> (query head of the group, row block of 32 positions); two waves
    // share a SIMD, so one can run its softmax while the other keeps the matrix core busy
    const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int head = wave % G, rb = wave / G;
    const int qn = lane & 31, half = lane >> 5;
    const int gl = pv.global_len[um];
    const int w_eff = min(pv.W, t0);              // ring entries that exist
    const int i_end = min(T, qt * S::Q + S::Q);   // chunk keys this block can see: [0, i_end)
    // tiles: global cache, ring, picked chunk keys below `near`, all chunk keys from there on
    const int near = a.pick ? max(0, qt * S::Q - pv.W + 1) / KT * KT : 0;  // no window of the block reaches below
    const int32_t *pick = a.pick ? a.pick + pick_of(pv.Hkv, b, h, base, T) : a.order;
    const int n_far = near > 0 ? a.picked[picked_of(pv.Hkv, b, h, base, T) + near / 32] : 0;
    const int n_g = (gl + KT - 1) / KT, n_r = (w_eff + KT - 1) / KT;
    const int t_far = n_g + n_r, t_near = t_far + (n_far + KT - 1) / KT;  // first tile of each kind
    const int n_tiles = t_near + (i_end - near + KT - 1) / KT;

    // ---- Q^T operand: this lane's query, all d-slices of 16 ----
    pf_bf16x8_t qv[KS];
    const int q_first = qt * S::Q + rb * 32;      // first position of this wave's rows
    const int qi = min(q_first + qn, T - 1);
    const int qpos = t0 + qi;
    {
        const char *qp = a.q + ((size_t)(base + qi) * pv.Hq + (size_t)h * G + head) * D * 2;
#pragma unroll
        for (int ks = 0; ks < KS; ks++)
            qv[ks] = *reinterpret_cast<const pf_bf16x8_t *>(qp + (ks * 16 + half * 8) * 2);
    }
    pf_f32x16_t o[DB];
    float m = -INFINITY, l = 0.f;
#pragma unroll
    for (int db = 0; db < DB; db++)
#pragma unroll
        for (int c = 0; c < 16; c++) o[db][c] = 0.f;

    // ---- staging of a key tile: thread -> (key of the tile, 16-byte d chunk), K and V row-major ----
    const int ld_key = threadIdx.x / S::CPR, ld_dc = threadIdx.x % S::CPR;
    // two sets of staging registers: a tile is requested two iterations before it is multiplied
    // (plain variables passed one by one: a struct of them ends up in scratch memory)
    uint4 k0r, v0r, k1r, v1r;
    int lo0r, hi0r, lo1r, hi1r;
    // Page ids live in registers, one per lane, so that the address of a key row never
    // waits for a page-table load: 64 consecutive entries of the global table (reloaded
    // every 64 pages) and the whole local table when it has at most 64 entries.
    int pt_base = 0;
    int ptreg = (lane < pv.maxgp) ? pv.global_pt[(size_t)um * pv.maxgp + lane] : 0;
    const bool lp_in_reg = pv.nlp <= 64;
    const int lpreg = (lp_in_reg && lane < pv.nlp) ? pv.local_pt[(size_t)um * pv.nlp + lane] : 0;
    const int slot0 = t0 > pv.W ? t0 % pv.W : 0;  // ring slot of the oldest position
    const int64_t v_delta_chunk = a.v - a.k;
    // position of this thread's key of a picked tile (anything for another tile): asked for an iteration before its
    // row is
    auto ask_far = [&](int t) __attribute__((always_inline)) {
        return pick[max(0, min((t - t_far) * KT + ld_key, n_far - 1))];
    };
    auto fetch = [&](int t, int far, uint4 &r_k, uint4 &r_v, int &r_lo, int &r_hi) __attribute__((always_inline)) {
        const char *kp;
        int64_t v_delta;
        int lo = INT_MAX, hi = INT_MAX;  // invisible unless shown otherwise
        if (t < n_g) {  // global cache: visible to every query
            if (((t * KT + KT - 1) >> pv.logP) >= pt_base + 64) {
                pt_base = (t * KT) >> pv.logP;
                ptreg = (pt_base + lane < pv.maxgp) ? pv.global_pt[(size_t)um * pv.maxgp + pt_base + lane] : 0;
            }
            const int idx = t * KT + ld_key, idc = min(idx, gl - 1);
            const int pg = __shfl(ptreg, (idc >> pv.logP) - pt_base);
            kp = page_ptr(pv, pg) + (size_t)(idc & (pv.P - 1)) * (D * 2);
            if (idx < gl) lo = INT_MIN;
            v_delta = pv.v_off;
        } else if (t < t_far) {  // ring, oldest position first
            const int idx = (t - n_g) * KT + ld_key, idc = min(idx, w_eff - 1);
            int slot = slot0 + idc;
            slot = slot >= pv.W ? slot - pv.W : slot;
            const int pos = t0 - w_eff + idc;
            const int pg = lp_in_reg ? __shfl(lpreg, slot >> pv.logP)
                                     : pv.local_pt[(size_t)um * pv.nlp + (slot >> pv.logP)];
            kp = page_ptr(pv, pg) + (size_t)(slot & (pv.P - 1)) * (D * 2);
            if (idx < w_eff) {
                lo = pos;
                hi = (pv.ring_g[(size_t)um * pv.W + slot] >= a.tau) ? INT_MAX : pos + pv.W - 1;
            }
            v_delta = pv.v_off;
        } else if (t < t_near) {  // picked keys of this chunk: visible to every query
            kp = a.k + ((size_t)(base + far) * pv.Hkv + h) * (D * 2);
            if ((t - t_far) * KT + ld_key < n_far) lo = INT_MIN;
            v_delta = v_delta_chunk;
        } else {  // this chunk
            const int idx = near + (t - t_near) * KT + ld_key, idc = min(idx, T - 1);
            const size_t row = (size_t)(base + idc) * pv.Hkv + h;
            kp = a.k + row * (D * 2);
            if (idx < T) {
                lo = t0 + idx;
                hi = (a.g[row] >= a.tau) ? INT_MAX : t0 + idx + pv.W - 1;
            }
            v_delta = v_delta_chunk;
        }
        r_k = *reinterpret_cast<const uint4 *>(kp + ld_dc * 16);
        r_v = *reinterpret_cast<const uint4 *>(kp + v_delta + ld_dc * 16);
        r_lo = lo;
        r_hi = hi;
    };
    // Full tiles of the global cache, pages of at least as many tokens as a wave stages: its keys
    // share a page, so the page base is scalar and a lane only adds a fixed offset.
    const bool lean_ok = pv.P >= S::KPW;
    const uint32_t lean_k_off = (uint32_t)(ld_key & (pv.P - 1)) * (D * 2) + ld_dc * 16;
    auto fetch_lean = [&](int t, uint4 &r_k, uint4 &r_v, int &r_lo, int &r_hi) __attribute__((always_inline)) {
        if (((t * KT + KT - 1) >> pv.logP) >= pt_base + 64) {
            pt_base = (t * KT) >> pv.logP;
            ptreg = (pt_base + lane < pv.maxgp) ? pv.global_pt[(size_t)um * pv.maxgp + pt_base + lane] : 0;
        }
        const int pg = __builtin_amdgcn_readlane(ptreg, ((t * KT + S::KPW * wave) >> pv.logP) - pt_base);
        // inside its page the tile begins at row (KT t) mod P (0 unless a page holds several tiles)
        const char *sb = page_ptr(pv, pg) + (size_t)((t * KT) & (pv.P - 1)) * (D * 2);
        r_k = *reinterpret_cast<const uint4 *>(sb + lean_k_off);
        r_v = *reinterpret_cast<const uint4 *>(sb + lean_k_off + pv.v_off);
        r_lo = INT_MIN;
        r_hi = INT_MAX;
    };
    auto stage = [&](int buf, const uint4 &r_k, const uint4 &r_v, int r_lo, int r_hi) __attribute__((always_inline)) {
        *reinterpret_cast<uint4 *>(&s_k[buf][ld_key * S::KStride + ld_dc * 16]) = r_k;
        *reinterpret_cast<uint4 *>(&s_v[buf][ld_key * S::VStride + ld_dc * 16]) = r_v;
        if (ld_dc == 0) { s_lo[buf][ld_key] = r_lo; s_hi[buf][ld_key] = r_hi; }
    };
    const int n_plain = gl / KT;  // full tiles of the global cache
    auto no_mask = [&](int t) __attribute__((always_inline)) {
        return pf_no_mask(t, KT, n_g, n_plain, t_far, t_near, n_far, near, w_eff, pv.W, qt * S::Q, qt * S::Q + S::Q - 1);
    };
    // A weight of zero does not keep an inf or NaN of V out of a product, and the middle and low parts of a weight are often zero,
    // of a visible key too: every tile is looked through (t: the one that goes to the buffer).
    auto look = [&](int buf, const uint4 &r_v, int t) __attribute__((always_inline)) {
        if (pf_nonfinite(r_v)) s_bad[buf] = t;  // all writers of a tile write the same
    };
    if (threadIdx.x < 2) s_bad[threadIdx.x] = -1;

    auto fetch_any = [&](int t, int far, uint4 &r_k, uint4 &r_v, int &r_lo, int &r_hi) __attribute__((always_inline)) {
        if (lean_ok && t < n_plain) fetch_lean(t, r_k, r_v, r_lo, r_hi);
        else fetch(t, far, r_k, r_v, r_lo, r_hi);
    };
    const int far0 = ask_far(0), far1 = ask_far(1);
    int far_next = ask_far(2);
    fetch_any(0, far0, k0r, v0r, lo0r, hi0r);
    stage(0, k0r, v0r, lo0r, hi0r);
    __syncthreads();  // s_bad is set
    look(0, v0r, 0);
    if (n_tiles > 1) fetch_any(1, far1, k1r, v1r, lo1r, hi1r);
    __syncthreads();

    // one iteration: tile t is multiplied, tile t+2 is requested into rf, tile t+1 goes from rs to LDS
    auto body = [&](int t, uint4 &f_k, uint4 &f_v, int &f_lo, int &f_hi, const uint4 &s_kk, const uint4 &s_vv,
                    const int &s_lo_, const int &s_hi_) __attribute__((always_inline)) {
        const int buf = t & 1;
        // A block of more than 64 positions has waves whose rows end before a chunk tile begins, and a short
        // sequence leaves waves without rows: they only stage.  (At 64 positions it is one tile in a block.)
        const bool act = S::Q <= 64 || (q_first < T && near + (t - t_near) * KT <= q_first + 31);  // wave-uniform
        // LDS latency is the scarce thing here: the K fragments are requested at once,
        // the address arithmetic and global loads of the next tile run while they arrive,
        // and the V fragments are requested before the softmax that hides their latency.
        pf_bf16x8_t ka[NS][KS];
        if (act) {
#pragma unroll
            for (int n = 0; n < NS; n++)
#pragma unroll
                for (int ks = 0; ks < KS; ks++)
                    ka[n][ks] = *reinterpret_cast<const pf_bf16x8_t *>(
                        &s_k[buf][(32 * n + qn) * S::KStride + (ks * 16 + half * 8) * 2]);
        }
        __builtin_amdgcn_sched_barrier(0);
        const int far = far_next;
        far_next = ask_far(t + 3);
        if (t + 2 < n_tiles) fetch_any(t + 2, far, f_k, f_v, f_lo, f_hi);  // in flight while this tile and the next are multiplied
        __builtin_amdgcn_sched_barrier(0);
        if (act) {
            // ---- S^T = K Q^T : rows = keys of the tile, columns = this wave's queries ----
            pf_f32x16_t s[NS];
#pragma unroll
            for (int n = 0; n < NS; n++) {
#pragma unroll
                for (int c = 0; c < 16; c++) s[n][c] = 0.f;
#pragma unroll
                for (int ks = 0; ks < KS; ks++)
                    s[n] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(ka[n][ks], qv[ks], s[n], 0, 0, 0);
            }
            // V^T fragments read column-wise from the row-major V tile
            // (there are no registers for all of them during the softmax: read at their products)
            pf_bf16x8_t va[DB];
            auto read_v = [&](int t2) __attribute__((always_inline)) {
#pragma unroll
                for (int db = 0; db < DB; db++) va[db] = pf_get_cols<S::VStride>(s_v[buf], lane, db, 16 * t2);
            };
            __builtin_amdgcn_sched_barrier(0);
            // register c = 4j+i of a lane holds key 8j + 4*half + i of a score tile
            const bool plain = no_mask(t);
            float sc[16 * NS];
            float mt = -INFINITY;
            if (plain) {
#pragma unroll
                for (int c = 0; c < 16 * NS; c++) {
                    sc[c] = s[c / 16][c % 16] * a.scale_log2e;
                    mt = fmaxf(mt, sc[c]);
                }
            } else {
#pragma unroll
                for (int j = 0; j < 4 * NS; j++) {
                    const int4 lo4 = *reinterpret_cast<const int4 *>(&s_lo[buf][8 * j + 4 * half]);
                    const int4 hi4 = *reinterpret_cast<const int4 *>(&s_hi[buf][8 * j + 4 * half]);
                    const int lo_[4] = {lo4.x, lo4.y, lo4.z, lo4.w}, hi_[4] = {hi4.x, hi4.y, hi4.z, hi4.w};
#pragma unroll
                    for (int i = 0; i < 4; i++) {
                        const bool vis = (qpos >= lo_[i]) && (qpos <= hi_[i]);
                        const float x = vis ? s[j / 4][4 * (j % 4) + i] * a.scale_log2e : -INFINITY;
                        sc[4 * j + i] = x;
                        mt = fmaxf(mt, x);
                    }
                }
            }
            mt = fmaxf(mt, __shfl_xor(mt, 32));  // the other half of the keys of this query
            const float mnew = fmaxf(m, mt);
            const float msafe = mnew == -INFINITY ? 0.f : mnew;
            const float corr = __builtin_amdgcn_exp2f(m - msafe);
            uint32_t pb[3][8 * NS];
            float ps = 0.f;
#pragma unroll
            for (int c = 0; c < 8 * NS; c++) {
                const float p0 = __builtin_amdgcn_exp2f(sc[2 * c] - msafe), p1 = __builtin_amdgcn_exp2f(sc[2 * c + 1] - msafe);
                ps += p0 + p1;
                const float r0 = pf_rest(p0), r1 = pf_rest(p1);
                pb[0][c] = pf_top(p0, p1);
                pb[1][c] = pf_top(r0, r1);
                pb[2][c] = pf_top(pf_rest(r0), pf_rest(r1));
            }
            l = l * corr + ps;
            if (__builtin_amdgcn_ballot_w64(mnew > m) != 0) {
#pragma unroll
                for (int db = 0; db < DB; db++)
#pragma unroll
                    for (int c = 0; c < 16; c++) o[db][c] *= corr;
            }
            m = mnew;
            // ---- O^T += V^T P^T : rows = d, columns = queries, contraction over the keys, small parts first ----
            __builtin_amdgcn_sched_barrier(0);
#pragma unroll
            for (int t2 = 0; t2 < 2 * NS; t2++) {
                read_v(t2);
                if (s_bad[buf] == t) {  // block-uniform
                    // the finite values go on to the product; the queries that see the others get them here
                    uint32_t seen[4];
#pragma unroll
                    for (int c = 0; c < 4; c++) {  // pair c of the eight keys of this lane's half
                        const int key = 16 * t2 + 8 * (c / 2) + 4 * half + 2 * (c % 2);
                        seen[c] = (qpos >= s_lo[buf][key] && qpos <= s_hi[buf][key] ? 0x3f80u : 0u) |
                                  (qpos >= s_lo[buf][key + 1] && qpos <= s_hi[buf][key + 1] ? 0x3f800000u : 0u);
                    }
#pragma unroll
                    for (int db = 0; db < DB; db++) pf_take_nonfinite(va[db], seen, o[db]);
                }
#pragma unroll
                for (int part = 2; part >= 0; part--) {
                    const uint4 p4 = make_uint4(pb[part][4 * t2], pb[part][4 * t2 + 1], pb[part][4 * t2 + 2], pb[part][4 * t2 + 3]);
                    const pf_bf16x8_t pbv = __builtin_bit_cast(pf_bf16x8_t, p4);
#pragma unroll
                    for (int db = 0; db < DB; db++)
                        o[db] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(va[db], pbv, o[db], 0, 0, 0);
                }
            }
        }
        if (t + 1 < n_tiles) {
            stage(buf ^ 1, s_kk, s_vv, s_lo_, s_hi_);
            look(buf ^ 1, s_vv, t + 1);
        }
        __syncthreads();
    };
    {
        int t = 0;
        for (; t + 1 < n_tiles; t += 2) {
            body(t, k0r, v0r, lo0r, hi0r, k1r, v1r, lo1r, hi1r);
            body(t + 1, k1r, v1r, lo1r, hi1r, k0r, v0r, lo0r, hi0r);
        }
        if (t < n_tiles) body(t, k0r, v0r, lo0r, hi0r, k1r, v1r, lo1r, hi1r);
    }

    // ---- normalise and write: register c = 4j+i of o[db] is d = 32*db + 8j + 4*half + i ----
    {
        const int i = q_first + qn;
        const float lt = l + __shfl_xor(l, 32);
        if (i < T) {
            const float inv = 1.0f / lt;
            float *op = a.out + ((size_t)(base + i) * pv.Hq + (size_t)h * G + head) * D;
#pragma unroll
            for (int db = 0; db < DB; db++)
#pragma unroll
                for (int j = 0; j < 4; j++) {
                    const float4 w4 = make_float4(o[db][4 * j] * inv, o[db][4 * j + 1] * inv,
                                                  o[db][4 * j + 2] * inv, o[db][4 * j + 3] * inv);
                    *reinterpret_cast<float4 *>(op + 32 * db + 8 * j + 4 * half) = w4;
                }
        }
    }
}

// ---------------------------------------------------------------------------------------------
// The shape of the paper's models: 128 wide, four heads a group, weights rounded to bf16
//
// A block is 32 chunk positions x the four heads of a group, one wave each, two blocks to a compute unit; key tiles are
// 64 rows of K and of V, requested straight into one of two LDS buffers a tile ahead (no staging registers, one unpadded
// copy each).  Against blocks of 64 positions with tiles of 32 keys staged through registers, which this shape had:
// two 16K prompts in 4096-token chunks 797 -> 708 us per launch, eight of 131-1501 tokens 81 -> 71, four 128K prompts,
// all 32 chunks, 350 -> 312 ms (808 -> 906 TFLOP/s).  Two row blocks of 32 that share a tile: 732 us, 81 us, 316 ms.
// Bound by the matrix cores and the softmax beside them: the last chunks run at 950 TFLOP/s, where a library product of
// 8192 cubed reaches 1260 on the same card.
// ---------------------------------------------------------------------------------------------
constexpr int kPfTilesQ = 32;
// What stands in V past the last row of a region: a weight of zero does not keep an infinity out of a product, so these
// rows do not repeat the last one.
static __device__ const uint4 pf_zero_row[kSaD * 2 / 16] = {};
__global__ __launch_bounds__(256, 2) void attend_prefill_tiles_kernel(View pv, CallSeqs cs, PrefillAttnArgs a) {
    constexpr int NW = 4, Q = kPfTilesQ, KT = 64, kRows = KT / NW, G = 4, D = kSaD;
    __shared__ __attribute__((aligned(1024))) char s_t[2][2][KT * D * 2];  // K and V
    __shared__ __attribute__((aligned(16))) int s_lo[2][KT];
    __shared__ __attribute__((aligned(16))) int s_hi[2][KT];

    // order of the blocks: as in attend_prefill_kernel
    const int rank = a.rank0 + (int)(blockIdx.x / a.nx), unit = a.ordered ? a.order[rank] : rank;
    const int b = unit / pv.Hkv, h = unit % pv.Hkv;
    const int qt = a.nx - 1 - (int)(blockIdx.x % a.nx);
    const int T = cs.ntok[b], t0 = cs.t0[b], base = cs.base[b];
    if (qt * Q >= T) return;  // block-uniform
    const int um = unit_meta(pv, cs.sid[b], a.layer, h);
    const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int head = wave;
    const int qn = lane & 31, half = lane >> 5;
    const int gl = pv.global_len[um];
    const int w_eff = min(pv.W, t0);              // ring entries that exist
    const int i_end = min(T, qt * Q + Q);         // chunk keys this block can see: [0, i_end)
    // tiles: global cache, ring, picked chunk keys below `near`, all chunk keys from there on
    const int near = a.pick ? max(0, qt * Q - pv.W + 1) / KT * KT : 0;  // no window of the block reaches below
    const int32_t *pick = a.pick ? a.pick + pick_of(pv.Hkv, b, h, base, T) : a.order;
    const int n_far = near > 0 ? a.picked[picked_of(pv.Hkv, b, h, base, T) + near / 32] : 0;
    const int n_g = (gl + KT - 1) / KT, n_r = (w_eff + KT - 1) / KT;
    const int t_far = n_g + n_r, t_near = t_far + (n_far + KT - 1) / KT;  // first tile of each kind
    const int n_tiles = t_near + (i_end - near + KT - 1) / KT;

    sa_bf16x8_t qv[8];
    const int q_first = qt * Q;
    const int qi = min(q_first + qn, T - 1);
    const int qpos = t0 + qi;
    {
        const char *qp = a.q + ((size_t)(base + qi) * pv.Hq + (size_t)h * G + head) * D * 2;
#pragma unroll
        for (int ks = 0; ks < 8; ks++) qv[ks] = *reinterpret_cast<const sa_bf16x8_t *>(qp + (ks * 16 + half * 8) * 2);
    }
    pf_f32x16_t o[4];
    float m = -INFINITY, l = 0.f;
#pragma unroll
    for (int db = 0; db < 4; db++)
#pragma unroll
        for (int c = 0; c < 16; c++) o[db][c] = 0.f;

    // Page ids live in registers, one per lane, so that the address of a key row never waits for a page-table load: 64
    // consecutive entries of the global table (reloaded every 64 pages) and the whole local table of at most 64 entries.
    int pt_base = 0;
    int ptreg = (lane < pv.maxgp) ? pv.global_pt[(size_t)um * pv.maxgp + lane] : 0;
    const bool lp_in_reg = pv.nlp <= 64;
    int lpreg = (lp_in_reg && lane < pv.nlp) ? pv.local_pt[(size_t)um * pv.nlp + lane] : 0;
    const int slot0 = t0 > pv.W ? t0 % pv.W : 0;  // ring slot of the oldest position
    auto ring_slot = [&](int idx) __attribute__((always_inline)) {
        const int s = slot0 + min(idx, w_eff - 1);
        return s >= pv.W ? s - pv.W : s;
    };
    // chunk positions of the wave's rows of a picked tile, one per lane (anything for another tile): asked for a tile
    // before its rows are
    auto ask_far = [&](int t) __attribute__((always_inline)) {
        return pick[max(0, min((t - t_far) * KT + wave * kRows + (lane & (kRows - 1)), n_far - 1))];
    };
    const bool lean_ok = pv.P >= kRows;  // the wave's rows of a full tile of the global cache share a page
    const int n_plain = gl / KT;         // full tiles of the global cache
    auto fetch = [&](int t, int far) __attribute__((always_inline)) {
        char *lk = &s_t[t & 1][0][wave * kRows * (D * 2)], *lv = &s_t[t & 1][1][wave * kRows * (D * 2)];
        int ln = lane;
        asm volatile("" : "+v"(ln));  // the lane's offsets are formed per tile: no registers to keep them
        const int sub = ln >> 4;
        if (t < n_g && ((t * KT + KT - 1) >> pv.logP) >= pt_base + 64) {
            pt_base = (t * KT) >> pv.logP;
            ptreg = (pt_base + ln < pv.maxgp) ? pv.global_pt[(size_t)um * pv.maxgp + pt_base + ln] : 0;
        }
        if (lean_ok && t < n_plain) {
            const int idx = t * KT + kRows * wave;
            const int pg = __builtin_amdgcn_readlane(ptreg, (idx >> pv.logP) - pt_base);
            const char *sb = page_ptr(pv, pg) + (size_t)(idx & (pv.P - 1)) * (D * 2);
#pragma unroll
            for (int i = 0; i < kRows / 4; i++) {
                const uint32_t off = (uint32_t)((4 * i + sub) * (D * 2) + ((ln & 15) ^ sa_sw_f(wave * kRows + 4 * i + sub)) * 16);
                sa_dma16(sb, off, lk + i * 1024);
                sa_dma16(sb + pv.v_off, off, lv + i * 1024);
            }
            return;
        }
        // rows of the region from this tile on: the tile's others are past its end
        const int rows = t < n_g ? gl - t * KT : t < t_far ? w_eff - (t - n_g) * KT : t < t_near ? n_far - (t - t_far) * KT
                                                                                              : T - near - (t - t_near) * KT;
        auto pieces = [&](auto last_t) __attribute__((always_inline)) {
            constexpr bool kLast = decltype(last_t)::value;
#pragma unroll
            for (int i = 0; i < kRows / 4; i++) {
                const int r = wave * kRows + 4 * i + sub;
                const char *kp;
                int64_t v_delta = pv.v_off;
                if (t < n_g) {  // global cache
                    const int idc = min(t * KT + r, gl - 1);
                    const int pg = __shfl(ptreg, (idc >> pv.logP) - pt_base);
                    kp = page_ptr(pv, pg) + (size_t)(idc & (pv.P - 1)) * (D * 2);
                } else if (t < t_far) {  // ring, oldest position first
                    const int slot = ring_slot((t - n_g) * KT + r);
                    const int pg = lp_in_reg ? __shfl(lpreg, slot >> pv.logP)
                                             : pv.local_pt[(size_t)um * pv.nlp + (slot >> pv.logP)];
                    kp = page_ptr(pv, pg) + (size_t)(slot & (pv.P - 1)) * (D * 2);
                } else {  // this chunk
                    const int idc = t < t_near ? __shfl(far, 4 * i + sub) : min(near + (t - t_near) * KT + r, T - 1);
                    kp = a.k + ((size_t)(base + idc) * pv.Hkv + h) * (D * 2);
                    v_delta = a.v - a.k;
                }
                const int at = ((ln & 15) ^ sa_sw_f(r)) * 16;
                kp += at;
                sa_dma16_at(kp, lk + i * 1024);
                sa_dma16_at(kLast && r >= rows ? reinterpret_cast<const char *>(pf_zero_row) + at : kp + v_delta, lv + i * 1024);
            }
        };
        if (rows >= KT) pieces(std::false_type());
        else pieces(std::true_type());
    };
    auto no_mask = [&](int t) __attribute__((always_inline)) {
        return pf_no_mask(t, KT, n_g, n_plain, t_far, t_near, n_far, near, w_eff, pv.W, q_first, q_first + Q - 1);
    };
    // Who sees key `lane` of a tile with a mask: positions lo to hi.  A wave of the block in turn asks for its score and,
    // at the end of the turn, writes the two bounds.
    auto ask_score = [&](int t) __attribute__((always_inline)) {
        const int idx = t < t_far ? (t - n_g) * KT + lane : near + (t - t_near) * KT + lane;
        if (t >= n_g && t < t_far) return pv.ring_g[(size_t)um * pv.W + ring_slot(idx)];
        if (t >= t_near) return a.g[(size_t)(base + min(idx, T - 1)) * pv.Hkv + h];
        return 0.f;
    };
    auto put_bounds = [&](int t, float g) __attribute__((always_inline)) {
        int lo = INT_MAX, hi = INT_MAX;  // invisible unless shown otherwise
        if (t < n_g) {
            if (t * KT + lane < gl) lo = INT_MIN;
        } else if (t < t_far) {
            const int idx = (t - n_g) * KT + lane;
            if (idx < w_eff) {
                lo = t0 - w_eff + idx;
                hi = g >= a.tau ? INT_MAX : lo + pv.W - 1;
            }
        } else if (t < t_near) {
            if ((t - t_far) * KT + lane < n_far) lo = INT_MIN;
        } else {
            const int idx = near + (t - t_near) * KT + lane;
            if (idx < T) {
                lo = t0 + idx;
                hi = g >= a.tau ? INT_MAX : lo + pv.W - 1;
            }
        }
        s_lo[t & 1][lane] = lo;
        s_hi[t & 1][lane] = hi;
    };

    asm volatile("" : "+v"(ptreg), "+v"(lpreg));  // waited for here, not behind the requests; so is the query
#pragma unroll
    for (int ks = 0; ks < 8; ks++) asm volatile("" : "+v"(qv[ks]));
    const int o_row = sa_sw_row(qn, half), o_col = sa_sw_col(lane);
    int far_next = ask_far(1);
    fetch(0, ask_far(0));
    if (wave == 0) put_bounds(0, ask_score(0));
    sa_dma_wait_barrier<0>();
    bool plain_next = no_mask(0);
    for (int t = 0; t < n_tiles; t++) {
        const int buf = t & 1;
        const char *tk = s_t[buf][0], *tv = s_t[buf][1];
        const int far = far_next;
        far_next = ask_far(t + 2);
        const bool plain = plain_next;
        plain_next = no_mask(t + 1);
        const bool mine = t + 1 < n_tiles && wave == (t + 1) % NW && !plain_next;
        float g_next = 0.f;
        if (mine) g_next = ask_score(t + 1);
        if (t + 1 < n_tiles) fetch(t + 1, far);
        // ---- S^T = K Q^T : rows = keys of the tile, columns = this wave's queries ----
        pf_f32x16_t s[2];
#pragma unroll
        for (int n = 0; n < 2; n++) {
#pragma unroll
            for (int c = 0; c < 16; c++) s[n][c] = 0.f;
#pragma unroll
            for (int ks = 0; ks < 8; ks++)
                s[n] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(sa_sw_get_row(tk + n * kSaTileB, o_row, ks), qv[ks], s[n], 0, 0, 0);
        }
        // register c = 4j+i of s[n] holds key 32*n + 8j + 4*half + i
        float mt = -INFINITY;
        if (plain) {
#pragma unroll
            for (int c = 0; c < 32; c++) {
                s[c / 16][c % 16] *= a.scale_log2e;
                mt = fmaxf(mt, s[c / 16][c % 16]);
            }
        } else {
#pragma unroll
            for (int j = 0; j < 8; j++) {
                const int4 lo4 = *reinterpret_cast<const int4 *>(&s_lo[buf][8 * j + 4 * half]);
                const int4 hi4 = *reinterpret_cast<const int4 *>(&s_hi[buf][8 * j + 4 * half]);
                const int lo_[4] = {lo4.x, lo4.y, lo4.z, lo4.w}, hi_[4] = {hi4.x, hi4.y, hi4.z, hi4.w};
#pragma unroll
                for (int i = 0; i < 4; i++) {
                    const bool vis = (qpos >= lo_[i]) && (qpos <= hi_[i]);
                    const float x = vis ? s[j / 4][4 * (j % 4) + i] * a.scale_log2e : -INFINITY;
                    s[j / 4][4 * (j % 4) + i] = x;
                    mt = fmaxf(mt, x);
                }
            }
        }
        mt = fmaxf(mt, __shfl_xor(mt, 32));  // the other half of the keys of this query
        const float mnew = fmaxf(m, mt);
        const float msafe = mnew == -INFINITY ? 0.f : mnew;
        const float corr = __builtin_amdgcn_exp2f(m - msafe);
        uint32_t pb[16];
        float ps = 0.f;
        const pf_bf16x2_t ones = {(__bf16)1.0f, (__bf16)1.0f};
#pragma unroll
        for (int c = 0; c < 16; c++) {
            pb[c] = pf_pack(__builtin_amdgcn_exp2f(s[c / 8][2 * c % 16] - msafe), __builtin_amdgcn_exp2f(s[c / 8][2 * c % 16 + 1] - msafe));
            // the denominator sums the rounded weights, the ones the second product uses
            ps = __builtin_amdgcn_fdot2_f32_bf16(__builtin_bit_cast(pf_bf16x2_t, pb[c]), ones, ps, false);
        }
        l = l * corr + ps;
        if (__builtin_amdgcn_ballot_w64(mnew > m) != 0) {
#pragma unroll
            for (int db = 0; db < 4; db++)
#pragma unroll
                for (int c = 0; c < 16; c++) o[db][c] *= corr;
        }
        m = mnew;
        // ---- O^T += V^T P^T : rows = d, columns = queries, contraction over the keys ----
#pragma unroll
        for (int t2 = 0; t2 < 4; t2++) {
            const uint4 p4 = make_uint4(pb[4 * t2], pb[4 * t2 + 1], pb[4 * t2 + 2], pb[4 * t2 + 3]);
#pragma unroll
            for (int db = 0; db < 4; db++)
                o[db] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(sa_sw_get_cols(tv, o_col, db, t2), __builtin_bit_cast(sa_bf16x8_t, p4), o[db], 0, 0, 0);
        }
        if (mine) put_bounds(t + 1, g_next);
        sa_dma_wait_barrier<0>();  // tile t + 1 is there, and nobody reads tile t any more
    }

    // ---- normalise and write: register c = 4j+i of o[db] is d = 32*db + 8j + 4*half + i ----
    const int i = q_first + qn;
    const float lt = l + __shfl_xor(l, 32);
    if (i < T) {
        const float inv = 1.0f / lt;
        float *op = a.out + ((size_t)(base + i) * pv.Hq + (size_t)h * G + head) * D;
#pragma unroll
        for (int db = 0; db < 4; db++)
#pragma unroll
            for (int j = 0; j < 4; j++) {
                const float4 w4 = make_float4(o[db][4 * j] * inv, o[db][4 * j + 1] * inv,
                                              o[db][4 * j + 2] * inv, o[db][4 * j + 3] * inv);
                *reinterpret_cast<float4 *>(op + 32 * db + 8 * j + 4 * half) = w4;
            }
    }
}

// What the attention kernel wants to know about the call first.  Block u < n_units: the admitted positions of unit u's
// chunk in ascending order, and how many of them lie below every multiple of 32 (a thread takes 8 consecutive positions
// of every stretch of 2048).  The last block: the units by descending length of their global cache (equal lengths:
// lower unit first).  Without room for the lists only the last block is launched.
constexpr int kPickOwn = 8;
__global__ __launch_bounds__(256) void prefill_look_kernel(View pv, CallSeqs cs, int layer, float tau, const float *g,
                                                           int32_t *order, int32_t *pick, int32_t *picked) {
    __shared__ int s_len[kMaxCallUnits];
    __shared__ int s_tmp[20];
    const int n_units = cs.n * pv.Hkv;
    if (blockIdx.x == gridDim.x - 1) {
        for (int u = threadIdx.x; u < n_units; u += 256)
            s_len[u] = pv.global_len[unit_meta(pv, cs.sid[u / pv.Hkv], layer, u % pv.Hkv)];
        __syncthreads();
        for (int u = threadIdx.x; u < n_units; u += 256) {
            const int mine = s_len[u];
            int rank = 0;
            for (int v = 0; v < n_units; v++) rank += (s_len[v] > mine || (s_len[v] == mine && v < u)) ? 1 : 0;
            order[rank] = u;
        }
        return;
    }
    const int b = (int)blockIdx.x / pv.Hkv, h = (int)blockIdx.x % pv.Hkv;
    const int T = cs.ntok[b], base = cs.base[b];
    int32_t *list = pick + pick_of(pv.Hkv, b, h, base, T), *below = picked + picked_of(pv.Hkv, b, h, base, T);
    const float *gu = g + (size_t)base * pv.Hkv + h;
    int carry = 0;
    for (int i0 = 0; i0 <= T; i0 += 256 * kPickOwn) {  // T itself included: the count below T if 32 divides it
        const int i = i0 + (int)threadIdx.x * kPickOwn;
        float x[kPickOwn];
#pragma unroll
        for (int e = 0; e < kPickOwn; e++) x[e] = T > 0 ? gu[(size_t)min(i + e, T - 1) * pv.Hkv] : 0.f;
        int n = 0;
#pragma unroll
        for (int e = 0; e < kPickOwn; e++) n += (i + e < T && x[e] >= tau) ? 1 : 0;
        int total;
        int at = carry + block_excl_scan(n, s_tmp, &total);
        if (i % 32 == 0 && i <= T) below[i / 32] = at;
#pragma unroll
        for (int e = 0; e < kPickOwn; e++)
            if (i + e < T && x[e] >= tau) list[at++] = i + e;
        carry += total;
    }
}

// The order of the units, then the lists of picked chunk keys (one entry per token and kv head at most) and their counts.
constexpr size_t kPfOrderBytes = 256 + sizeof(int32_t) * kMaxCallUnits;
size_t attend_prefill_ws_min_bytes() { return kPfOrderBytes; }
size_t attend_prefill_ws_bytes(const View &pv, int n_seqs, int64_t total_q) {
    return kPfOrderBytes + sizeof(int32_t) * (size_t)pv.Hkv * (size_t)(total_q + total_q / 32 + n_seqs);
}

// Blocks of q positions for every unit of the call.  A launch holds fewer than 2^32 threads: where one long chunk beside many
// short ones would be over that (every unit has the blocks of the longest), the units go to several launches.
template <class Kernel>
static hipError_t launch_units(Kernel kernel, int q, int threads, const View &pv, const CallSeqs &cs, PrefillAttnArgs &a, int max_t,
                               hipStream_t st) {
    a.nx = (max_t + q - 1) / q;
    const int n_units = cs.n * pv.Hkv;
    const int per = (int)std::min<int64_t>(n_units, (((int64_t)1 << 32) - 1) / ((int64_t)a.nx * threads));
    for (a.rank0 = 0; a.rank0 < n_units; a.rank0 += per) {
        hipLaunchKernelGGL(kernel, dim3((unsigned)a.nx * std::min(per, n_units - a.rank0)), dim3(threads), 0, st, pv, cs, a);
        const hipError_t e = hipGetLastError();
        if (e != hipSuccess) return e;
    }
    return hipSuccess;
}
template <int D, int G>
static hipError_t launch_shape(const View &pv, const CallSeqs &cs, PrefillAttnArgs &a, int max_t, hipStream_t st) {
    return launch_units(attend_prefill_kernel<D, G>, PfShape<D, G>::Q, 512, pv, cs, a, max_t, st);
}

// Lists of picked chunk keys pay as soon as some block of the call has keys behind all its windows, and need room; without them
// and without a need of the order there is nothing to look at.
hipError_t launch_prefill_look(const View &pv, const CallSeqs &cs, int layer, float tau, const float *g, void *ws,
                               size_t ws_bytes, bool need_order, const int32_t **order, const int32_t **pick, const int32_t **picked,
                               hipStream_t st) {
    int64_t total = 0;
    int max_t = 0;
    for (int b = 0; b < cs.n; b++) {
        total += cs.ntok[b];
        max_t = max(max_t, cs.ntok[b]);
    }
    const int n_units = cs.n * pv.Hkv;
    const bool lists = max_t > pv.W && ws_bytes >= attend_prefill_ws_bytes(pv, cs.n, total);
    int32_t *o = (int32_t *)ws, *p = lists ? o + kPfOrderBytes / sizeof(int32_t) : nullptr;
    int32_t *c = lists ? p + (size_t)pv.Hkv * total : nullptr;
    if (lists || need_order)
        hipLaunchKernelGGL(prefill_look_kernel, dim3((lists ? n_units : 0) + 1), dim3(256), 0, st, pv, cs, layer, tau, g, o, p, c);
    *order = o;
    *pick = p;
    *picked = c;
    return hipGetLastError();
}

// bf16 pools of every head_dim and group size (fp32 pools: launch_attend_prefill_f32)
hipError_t launch_attend_prefill(const View &pv, const CallSeqs &cs, int layer, const void *q,
                                 const void *k, const void *v, const float *g, float tau,
                                 float scale, float *out, void *ws, size_t ws_bytes, int n_cu, hipStream_t st) {
    if (pv.dtype != WGKV_BF16) return hipErrorNotSupported;
    PrefillAttnArgs a;
    a.layer = layer;
    a.tau = tau;
    a.scale_log2e = scale * 1.4426950408889634f;
    a.q = (const char *)q;
    a.k = (const char *)k;
    a.v = (const char *)v;
    a.g = g;
    a.out = out;
    int max_t = 0;
    for (int b = 0; b < cs.n; b++) max_t = max(max_t, cs.ntok[b]);
    if (max_t == 0) return hipSuccess;
    if (max_t >= 1 << 28) return hipErrorInvalidValue;  // the blocks of one unit have to fit a launch
    // The order is for launches of more than one round of blocks (a block per compute unit, two of the tiles kernel): below, its
    // own launch is all it adds.  us with / without: 33 tokens of 16 / 8 heads of 128 12.5 / 9.8, 16 x 100 of 32 / 8 24.2 / 19.4.
    const bool tiles = pv.d == 128 && pv.G == 4;
    const int per_block = tiles ? kPfTilesQ : 256 / pv.G;
    a.ordered = (int64_t)((max_t + per_block - 1) / per_block) * pv.Hkv * cs.n > (int64_t)n_cu * (tiles ? 2 : 1);
    hipError_t e = launch_prefill_look(pv, cs, layer, tau, g, ws, ws_bytes, a.ordered, &a.order, &a.pick, &a.picked, st);
    if (e != hipSuccess) return e;
    if (pv.d == 128) {
        switch (pv.G) {
            case 1: return launch_shape<128, 1>(pv, cs, a, max_t, st);
            case 2: return launch_shape<128, 2>(pv, cs, a, max_t, st);
            case 4: return launch_units(attend_prefill_tiles_kernel, kPfTilesQ, 256, pv, cs, a, max_t, st);
            case 8: return launch_shape<128, 8>(pv, cs, a, max_t, st);
            default: break;
        }
    } else if (pv.d == 64) {
        switch (pv.G) {
            case 1: return launch_shape<64, 1>(pv, cs, a, max_t, st);
            case 2: return launch_shape<64, 2>(pv, cs, a, max_t, st);
            case 4: return launch_shape<64, 4>(pv, cs, a, max_t, st);
            case 8: return launch_shape<64, 8>(pv, cs, a, max_t, st);
            default: break;
        }
    }
    return hipErrorNotSupported;
}

}  // namespace wgkv
