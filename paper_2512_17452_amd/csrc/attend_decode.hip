// Ragged, per-head paged GQA decode attention for gfx950 (wave64), bandwidth-bound.
//
// One query token per sequence.  A unit is one (sequence, kv head): its keys are
// the global cache [0, G_h) followed by the valid ring slots [0, min(t, W)); the
// G query heads of the group all read the same K/V rows (Sec. 4.3 last sentence,
// Sec. 2.1 equation; head-to-batch folding of App. A).  The cached tokens of all
// units are cut into 16-token tiles, and the tiles are split over the blocks of the launch,
// one block per compute unit (the split-then-reduce balancing of App. E "Decode phase",
// without a second launch and without any block waiting for another).  For calls of at most
// one unit per block there are two ways of cutting (attend_decode_kernel), and every block works
// out by itself which one has the shorter longest block:
//   pieces  every unit in equal pieces of 8 to 24 tiles at least, one piece per block: what a
//           small call wants, whose time is the chain in front of and behind its loops
//           (launch, lengths, page ids, first rows, publish, count, fold), and a unit of
//           one piece has no exchange through memory at all;
//   shares  one long list split evenly over the blocks, a share may start in the middle
//           of one unit and end in the middle of another: what a large call wants, where
//           pieces of unequal units would leave blocks idle.
// The four waves of a block take a quarter each of what the block has of a unit and meet
// in LDS; a unit that several blocks share is put together from one partial (m, l, acc)
// per block, by all threads of the block that arrives last, in a fixed order.
// Calls of more units than blocks go to attend_decode_many_kernel, which can also give whole units or
// even shares to single waves; its three ways stand above it.
//
// Data path of bf16 pools: rows go straight into LDS, 32 KiB ahead of their use in every wave, and both products run on
// the matrix cores (stream_pairs).  Of fp32 pools, of bf16 pages smaller than a tile and of many units of one or two narrow heads
// (launch_one): registers and the vector unit (stream_tiles).  Either way few waves per SIMD
// cover the HBM latency and no wave depends on the issue priority of another.
// What bounds a call: a long one the memory's rate; a short one chains of round trips and of instructions.  A wave issues one
// instruction in four clocks at best, and the first time through, out of a cold instruction cache, 64 bytes of code take
// about 70 ns, so what runs once is kept small.  Measured, us per launch, registers and dot products on the vector unit
// throughout / now (rows of memory in both): batch 1 at 32K 15.8 / 13.9; at 8K 12.9 / 10.4; at 2K 12.1 / 10.1; batch 8 at 1K 12.1 /
// 10.9; batch 2 at 60K 25.1 / 23.3; batch 8 at 100K (442 MB) 77 / 76.5; 32 x 4000 tokens 31.5 / 30.2; 64-wide heads, 2 x 30K 15.7 / 13.5;
// groups of eight 21.6 / 18.9; of one, batch 1 at 32K 14.4 / 12.9; fp32 128-wide, 2 x 30K 18.0 / 16.5; fp32 2 heads of 20K 13.1 / 10.8.
#include <type_traits>

#include <hip/hip_ext.h>

#include "wgkv_dev.h"

namespace wgkv {

constexpr int kTile = 16;        // tokens per tile
constexpr int kAttnThreads = 256;
constexpr int kAttnWaves = 4;
// A block that begins a unit in the middle of its share drains its loads, folds and publishes a partial
// and waits for the new unit's lengths, query rows and page ids.  The split charges that to the unit, as
// tiles in front of the first real one that nobody reads: 12 / 24 / 48 tiles of a block give 75.7 / 75.9 / 76.5 us on batch 8 at
// 100K, 25.9 / 25.5 / 25.3 on 64 ragged heads of 32K, 40.8 / 41.0 / 42.7 on batch 16 at 16K.
constexpr int kUnitStartTiles = 24;
// Blocks go to the XCDs round-robin, and in every launch measured the odd XCD of a pair streams
// slower than the even one, by 4-5 % on some machines and by about twice that on others: with even
// shares an odd block gets a number of thousandths fewer tiles, the even block before it as many
// more (AttendArgs::skew_permille; 50 unless the pool was tuned on its machine, see
// wgkv_tune_decode_attention).
// Smaller pieces mean fewer tiles per wave and more partials to publish, count and fold.  Where the blocks do not ask for more than
// the memory gives, pieces are as small as 8 tiles (of at least 4 / 8 / 12 / 24 tiles, us: batch 1 at 8K 11.7 / 10.6 / 11.0 / 12.9, batch 1
// at 2K 9.4 / 9.9 / 10.1 / 11.9, fp32 2 heads of 20K 12.5 / 11.2 / 11.9 / 13.1); where 140 blocks already do, smaller ones only cost
// (batch 1 at 32K, 8 / 16 / 24 tiles: 17.5 / 16.1 / 15.1; 100 and 200 instead of 140 blocks: 14.1 / 15.3 against 14.5 there, but 11.5 /
// 11.2 against 10.9 on batch 8 at 1K).  Units of up to 16 tiles stay whole: 180 tokens x 2 heads 8.4 / 7.1 us with pieces of 8 / 16.
constexpr int kMinBlockTiles = 24, kMinPieceTiles = 8, kWholeTiles = 16, kStreamBlocks = 140;
struct AttendArgs {
    int layer;
    int n_seqs;
    int skew_permille;        // share of the odd blocks' tiles that goes to the even blocks instead
    float scale_log2e;        // scale * log2(e)
    const char *q;            // [n_seqs][Hq][d]
    float *out;               // [n_seqs][Hq][d]
    float *part_ml;           // [(waves of the launch + n_units)][G][2]: a worker's partial of unit u is in slot worker + u
    float *part_acc;          // [(waves of the launch + n_units)][G][d]
    uint32_t part_ml_bytes, part_acc_bytes;
    int32_t *counters;        // [n_units] zero between calls: workers (blocks, or waves in calls of many units) done per unit
    // optional page selection: only these pages of each head's global cache are read
    const int32_t *sel_pages; // [n_units][sel_stride] ascending indices into the head's global table, or NULL
    const int32_t *sel_count; // [n_units]
    int sel_stride;
    int32_t sid[kMaxCallSeqs];
};

// Tokens a unit reads from its global cache: all gl of them, or those of the selected pages (every
// page is full except possibly the last one of the cache, which then is the last one selected).
__device__ __forceinline__ int global_tokens(const View &pv, const AttendArgs &a, int u, int gl) {
    if (!a.sel_pages) return gl;
    const int n_pages = (gl + pv.P - 1) >> pv.logP;
    const int cnt = min(min(max(a.sel_count[u], 0), a.sel_stride), n_pages);
    if (cnt == 0) return 0;
    const int last = a.sel_pages[(size_t)u * a.sel_stride + cnt - 1];
    return (cnt - 1) * pv.P + (last >= n_pages - 1 ? gl - (n_pages - 1) * pv.P : pv.P);
}

__device__ __forceinline__ int ceil_tiles(int n) { return (n + kTile - 1) / kTile; }

// How rows are worked with: fp32, bf16 on the matrix cores, or (a third value beside the two types) bf16 on the vector unit.
constexpr int kBf16Vec = 2;
static_assert(kBf16Vec != WGKV_F32 && kBf16Vec != WGKV_BF16, "");
template <int DT> struct Elem;
template <> struct Elem<WGKV_F32> { static constexpr int es = 4; };
template <> struct Elem<WGKV_BF16> { static constexpr int es = 2; };
template <> struct Elem<kBf16Vec> { static constexpr int es = 2; };

typedef __attribute__((ext_vector_type(2))) __bf16 dec_bf16x2_t;
__device__ __forceinline__ float dec_dot2(uint32_t a, uint32_t b, float c) {
    return __builtin_amdgcn_fdot2_f32_bf16(__builtin_bit_cast(dec_bf16x2_t, a), __builtin_bit_cast(dec_bf16x2_t, b), c, false);
}
// A row's dot product with the query, 16 bytes of each.
template <int DT>
__device__ __forceinline__ float dec_dot(const uint32_t (&k)[4], const uint32_t (&q)[4]) {
    float d = 0.f;
#pragma unroll
    for (int e = 0; e < 4; e++) d = DT == WGKV_F32 ? fmaf(__uint_as_float(k[e]), __uint_as_float(q[e]), d) : dec_dot2(k[e], q[e], d);
    return d;
}

// Partials cross compute units (and their L2 slices) inside one launch: they are
// written and read with device-coherent accesses, so no cache-wide flush is needed.
// Buffer accesses carry the same cache policy as a device-scope atomic access (sc1) at up to
// 16 bytes per lane, and an access outside the buffer reads zero or is dropped.
typedef unsigned u32x4 __attribute__((ext_vector_type(4)));
typedef unsigned u32x2 __attribute__((ext_vector_type(2)));
constexpr int kCoherent = 16;  // cache-policy operand of the buffer builtins: sc1
__device__ __forceinline__ __amdgpu_buffer_rsrc_t part_rsrc(float *p, uint32_t bytes) {
    return __builtin_amdgcn_make_buffer_rsrc(p, 0, (int)bytes, 0x00020000);  // raw buffer, 32-bit data format
}

// What one instantiation of the decode kernels works with.
template <int DT, int D_, int G_>
struct DecShape {
    static constexpr int D = D_, G = G_;
    static constexpr int ES = Elem<DT>::es;
    static constexpr int EPL = 16 / ES;      // elements per lane per row
    static constexpr int LPT = D / EPL;      // lanes per token row
    static constexpr int TPW = 64 / LPT;     // token rows per wave load
    static constexpr int RPT = kTile / TPW;  // wave loads per tile (K and V each)
    static constexpr int ROWB = D * ES;      // bytes of a K or V row
    static constexpr bool MX = DT == WGKV_BF16;  // on the matrix cores
    static_assert(LPT == 8 || LPT == 16 || LPT == 32, "row must be 128, 256 or 512 bytes");
    // Vector unit, groups of four or eight query heads: four heads' scores of a tile are as many as a row group has lanes
    // (16 / TPW rows x 4 = LPT), so they are spread one per lane, and max, exp and sum run once instead of LPT
    // times.  m[hh] and l[hh] then belong to head 4 * hh + sub % 4; the other entries are unused.
    static constexpr bool SPREAD = !MX && G % 4 == 0;
    static constexpr int HH = SPREAD ? G / 4 : 1;
    // Matrix cores: weights enter their product in parts of 8 bits: two for the shape of the paper's two models (error against 64 bits 2.3e-6; rounded
    // to one part 1.5e-3, and 9.4e-4 where each of 16 streams a wave has its largest weight exact), three for the others
    static constexpr int PARTS = D == 128 && G == 4 ? 2 : 3;
    // Vector unit: register sets = tiles in flight per wave.  With one wave per SIMD the loads of a wave's own next tiles are all
    // there is to cover the latency; 512-byte rows take 64 registers a tile, and with eight heads to a group four sets
    // leave too few registers.
    static constexpr int S = RPT <= 4 && G <= 4 ? 4 : 2;
    // Matrix cores: pairs of tiles that a wave has in LDS, 32 KiB
    static constexpr int NP = 512 / ROWB;
    static constexpr int EP = D / 16;        // output elements per lane, head and pair
    static constexpr int NSW = MX ? 1 : TPW; // softmax states of a wave: one, or one per row group
};

// Weights and rows of 64 keys (see sum_again).
template <int G>
struct DecStrip {
    float w[64][G];
    const char *v[64];
};
// What a wave works with in LDS.  Vector unit: strips through which the weights of a tile go back to the row layout; matrix cores: its tiles.
template <int DT, int D, int G>
struct DecWaveLds {
    float p[2][64];         // fp32 weights of a tile, four heads in each half
};
template <int D, int G>
struct DecWaveLds<kBf16Vec, D, G> {
    union {
        float p[2][64];
        DecStrip<G> again;
    };
};
template <int D, int G>
struct DecWaveLds<WGKV_BF16, D, G> {
    __attribute__((aligned(1024))) char t[DecShape<WGKV_BF16, D, G>::NP][2][2][kTile * D * 2];  // [pair][K, V][tile of the pair]
};

// A wave's running softmax.  Vector unit: per row group.
template <int DT, int D, int G>
struct DecSoftmax {
    float m[G], l[G], acc[G][DecShape<DT, D, G>::EPL];
    __device__ __forceinline__ void init() {
#pragma unroll
        for (int g = 0; g < G; g++) {
            m[g] = -INFINITY;
            l[g] = 0.f;
#pragma unroll
            for (int e = 0; e < DecShape<DT, D, G>::EPL; e++) acc[g][e] = 0.f;
        }
    }
};
// Matrix cores: m is that of head lane % G; register i of l and of acc[c] belongs to head (4 * (lane / 16) + i) % G, acc[c] to output
// element 16 * c + lane % 16.
typedef float dec_f32x4_t __attribute__((ext_vector_type(4)));
typedef __bf16 dec_bf16x8_t __attribute__((ext_vector_type(8)));
typedef unsigned dec_u32x4_t __attribute__((ext_vector_type(4)));
template <int D, int G>
struct DecSoftmax<WGKV_BF16, D, G> {
    static constexpr int EP = DecShape<WGKV_BF16, D, G>::EP;
    float m;
    dec_f32x4_t l, acc[EP];
    __device__ __forceinline__ void init() {
        m = -INFINITY;
#pragma unroll
        for (int i = 0; i < 4; i++) {
            l[i] = 0.f;
#pragma unroll
            for (int c = 0; c < EP; c++) acc[c][i] = 0.f;
        }
    }
};

// 16 bytes per lane from memory to LDS at dst + 16 * lane, with the non-temporal hint: rows are read once.  In assembly, as the
// compiler would put a wait for every outstanding request in front of the next LDS read; readers wait by count.  No result
// register, and M0 is free for it.  The instruction's offset counts on both sides.
// The base comes out of a lane (v_readlane), and a vector-memory instruction may not read a scalar register within five wait states of the
// vector unit's writing it; the compiler, which sees to that elsewhere, does not look into an assembly block.  So the base is copied by the
// scalar unit, whose reads of such a register the hardware holds back, and whose writes need no wait.  The copy is also
// the wait state that a request needs behind M0.
#pragma clang diagnostic push
#pragma clang diagnostic ignored "-Winline-asm"
__device__ __forceinline__ uint32_t dec_lds(const void *p) { return (uint32_t)(uintptr_t)(__attribute__((address_space(3))) const char *)p; }
__device__ __forceinline__ void dec_dma(const void *base, uint32_t off, const void *dst) {
    const void *b;
    asm volatile("s_mov_b32 m0, %1\n\ts_mov_b64 %0, %3\n\tglobal_load_lds_dwordx4 %2, %0 nt" : "=&s"(b) : "s"(dec_lds(dst)), "v"(off), "s"(base) : "memory", "m0");
}
// a tile of N * 1024 bytes, each request with its own lane offsets
__device__ __forceinline__ void dec_dma_tile(const void *base, const uint32_t (&off)[4], const void *dst) {
    const void *b;
    asm volatile("s_mov_b32 m0, %1\n\ts_mov_b64 %0, %6\n\tglobal_load_lds_dwordx4 %2, %0 nt\n\tglobal_load_lds_dwordx4 %3, %0 offset:1024 nt\n\t"
                 "global_load_lds_dwordx4 %4, %0 offset:2048 nt\n\tglobal_load_lds_dwordx4 %5, %0 offset:3072 nt"
                 : "=&s"(b) : "s"(dec_lds(dst)), "v"(off[0]), "v"(off[1]), "v"(off[2]), "v"(off[3]), "s"(base) : "memory", "m0");
}
__device__ __forceinline__ void dec_dma_tile(const void *base, const uint32_t (&off)[2], const void *dst) {
    const void *b;
    asm volatile("s_mov_b32 m0, %1\n\ts_mov_b64 %0, %4\n\tglobal_load_lds_dwordx4 %2, %0 nt\n\tglobal_load_lds_dwordx4 %3, %0 offset:1024 nt"
                 : "=&s"(b) : "s"(dec_lds(dst)), "v"(off[0]), "v"(off[1]), "s"(base) : "memory", "m0");
}
#pragma clang diagnostic pop
template <int N>
__device__ __forceinline__ void dec_wait_vm() { asm volatile("s_waitcnt vmcnt(%0)" ::"n"(N) : "memory"); }
__device__ __forceinline__ uint32_t dec_pack_bf16(float lo, float hi) {  // round to nearest even
    typedef __attribute__((ext_vector_type(2))) __bf16 bf16x2_t;
    const bf16x2_t t = {(__bf16)lo, (__bf16)hi};
    return __builtin_bit_cast(uint32_t, t);
}

// bf16: tiles [cur, u_end) of a unit into the wave's running softmax, on the matrix cores; the unit's tiles are those of its global
// cache followed by those of its ring.
// Two tiles (32 keys) at a time.  Rows come from memory straight into LDS (no registers, no copies of the loop's code per register
// set: the instructions of a launch's first pass come out of a cold cache too), 32 KiB ahead of their use; the K half of a pair is
// asked for again as soon as its operands are read, then the V half.
// S = K Q^T with the G heads repeated over the 16 columns: a lane ends up with the scores of one head and keys 4 * (lane / 16) + {0..3}
// of both tiles, which is the row operand of P V as it stands; the second operand is read transposed.  Sums over keys, those of the denominator too,
// are the matrix core's.  About 0.65 us a pair where a tile took 0.65 us with dot products and reductions on the vector unit.
// The maximum is brought up to date when a score exceeds it by 8 (weights of up to 256), so it costs no exchange between lanes in
// the rule; sums are fp32 either way.  What is folded is scaled back (kBack), and a value so large that a sum overflows on the
// way is one of those that are taken once more (sum_again).  Exponents relative to 8 above the maximum instead, which
// keep weights at one, are rounded at 8 and cost bits of the largest weights: error against 64 bits 2.6e-7 for 2.2e-7 with three parts.
template <int D, int G>
__device__ __forceinline__ void stream_pairs(const View &pv, const AttendArgs &a, int u, int um, int gl_all, int gl, int nloc, int cur, int u_end,
                                             dec_u32x4_t (&q)[D / 32], float c_exp, DecSoftmax<WGKV_BF16, D, G> &st,
                                             DecWaveLds<WGKV_BF16, D, G> &lds, int lane) {
    using SH = DecShape<WGKV_BF16, D, G>;
    constexpr int ROWB = SH::ROWB, LPT = SH::LPT, NI = SH::RPT, NP = SH::NP, EP = SH::EP, KS = D / 32, TILEB = kTile * ROWB;
    constexpr int H = 2 * NI, PI = 2 * H;  // requests of half a pair (K or V) and of a pair
    static_assert(NI * 1024 == TILEB, "");
    const int n_gt = ceil_tiles(gl);
    bool first = true;
    while (cur < u_end) {
        // one piece: at most 64 tiles [k0, k0+n) of one region (global or local) of unit u
        const bool is_glob = cur < n_gt;
        const int k0 = is_glob ? cur : cur - n_gt;
        const int region_tiles = is_glob ? n_gt : ceil_tiles(nloc);
        const int count = is_glob ? gl : nloc;
        const int n = min(min(region_tiles - k0, 64), u_end - cur);
        const int32_t *pt = is_glob ? pv.global_pt + (size_t)um * pv.maxgp : pv.local_pt + (size_t)um * pv.nlp;
        // page id of the vp-th page of the region as this call reads it (with a selection: the vp-th selected page; an
        // index outside the table is clamped, never followed)
        const int32_t *sel = (is_glob && a.sel_pages) ? a.sel_pages + (size_t)u * a.sel_stride : nullptr;
        const int last_page = max(((gl_all + pv.P - 1) >> pv.logP) - 1, 0);
        auto page_at = [&](int vp) __attribute__((always_inline)) { return pt[sel ? min(max(sel[vp], 0), last_page) : vp]; };
        // A tile lies inside one page (P >= 16) and has one address for the whole wave: lane i keeps that of tile k0 + i.
        const int k_lane = (k0 + min(lane, n - 1)) * kTile;
        int page = page_at(k_lane >> pv.logP);
        // (what follows from the lane alone is worked out while the page ids come: not hoisted in front of the request for them)
        int ln = lane;
        asm volatile("" : "+v"(ln));
        const int col = ln & 15, grp = ln >> 4;
        // Request i of a tile brings rows i * (64 / LPT) .., 16-byte piece x of row r at place x ^ f(r) of its row: K rows r % LPT, so
        // that one column of sixteen rows is on different banks; V rows by their low two bits, so that 32 bytes of four
        // consecutive rows are.
        const int r0 = ln / LPT, x0 = ln % LPT;
        auto v_sw = [](int r) __attribute__((always_inline)) { return D == 128 ? (r & 3) << 2 : r & 2; };
        uint32_t off_k[NI], off_v[NI];
#pragma unroll
        for (int i = 0; i < NI; i++) {
            off_k[i] = (uint32_t)(r0 * ROWB + (x0 ^ ((i * (64 / LPT) + r0) % LPT)) * 16);
            off_v[i] = (uint32_t)(r0 * ROWB + (x0 ^ v_sw(r0)) * 16);
        }
        const int o_k = col * ROWB + ((grp ^ (col % LPT)) * 16);  // ^ 64 * ks
        // ds_read_b64_tr_b16 transposes inside groups of 16 lanes: lane i of a group receives element i % 4 of the 8 bytes addressed by
        // lanes i / 4, 4 + i / 4, 8 + i / 4 and 12 + i / 4: lane s addresses (row s / 4 of the group's four, columns 4 * (s % 4)..+3 of
        // 16) and ends up with the four rows at its own column
        const int vr = 4 * grp + (col >> 2), o_v = vr * ROWB + (((col & 3) >> 1) ^ v_sw(vr)) * 16 + (col & 1) * 8;  // ^ 32 * c
        // the page ids and the query are waited for here: a wait that the compiler puts in later would be for the rows too
        asm volatile("" : "+v"(page));
#pragma unroll
        for (int ks = 0; ks < KS; ks++) asm volatile("" : "+v"(q[ks]));
        if (first && a.scale_log2e < 0.f) {  // a maximum of the products themselves: a negative scale turns the query's sign instead
#pragma unroll
            for (int ks = 0; ks < KS; ks++) {
                q[ks].x ^= 0x80008000u; q[ks].y ^= 0x80008000u; q[ks].z ^= 0x80008000u; q[ks].w ^= 0x80008000u;
            }
        }
        first = false;
        const uint64_t at = (uint64_t)page_ptr(pv, page) + (uint64_t)(k_lane & (pv.P - 1)) * ROWB;
        const uint32_t at_lo = (uint32_t)at, at_hi = (uint32_t)(at >> 32);
        const int pairs = (n + 1) / 2;
        auto valid_of = [&](int p) __attribute__((always_inline)) { return min(count - (k0 + 2 * p) * kTile, (n - 2 * p) * kTile); };  // keys of a pair that count
        // Half a pair into its place.  Rows past the last token of the piece read a valid row again (the last one of their tile,
        // or the first of a tile that is missing) and count for nothing: nothing that is not a cached row of this head is
        // ever read (a recycled page keeps whatever its last owner left in it, which need not be finite).
        auto request = [&](int p, bool v_half) __attribute__((always_inline)) {
            char *dst = lds.t[p % NP][v_half ? 1 : 0][0];
            auto base_of = [&](int j) __attribute__((always_inline)) {
                const uint64_t at = ((uint64_t)(uint32_t)__builtin_amdgcn_readlane(at_hi, j) << 32) | (uint32_t)__builtin_amdgcn_readlane(at_lo, j);
                return (const char *)(at + (v_half ? pv.v_off : 0u));
            };
            if (valid_of(p) >= 2 * kTile) {
                if (v_half) {
                    dec_dma_tile(base_of(2 * p), off_v, dst);
                    dec_dma_tile(base_of(2 * p + 1), off_v, dst + TILEB);
                } else {
                    dec_dma_tile(base_of(2 * p), off_k, dst);
                    dec_dma_tile(base_of(2 * p + 1), off_k, dst + TILEB);
                }
                return;
            }
#pragma unroll 1
            for (int t = 0; t < 2; t++) {
                const bool is = 2 * p + t < n;
                const int j = 2 * p + (is ? t : 0), k = k0 + j;
                const int last_row = is ? min(count - 1 - k * kTile, kTile - 1) : 0;
#pragma unroll
                for (int i = 0; i < NI; i++) {
                    const int r = i * (64 / LPT) + r0, row = min(r, last_row);
                    const uint32_t x = (v_half ? off_v[i] : off_k[i]) - (uint32_t)(r0 * ROWB);
                    dec_dma(base_of(j), (uint32_t)(row * ROWB) + x, dst + t * TILEB + i * 1024);
                }
            }
        };
#pragma unroll 1
        for (int p = 0; p < min(NP, pairs); p++) {
            request(p, false);
            request(p, true);
        }
        for (int p = 0; p < pairs; p++) {
            const int left = pairs - p;  // with this one; min(left, NP) of them are asked for
            if (left >= NP) dec_wait_vm<NP * PI - H>();
            else if (NP > 2 && left == 3) dec_wait_vm<3 * PI - H>();
            else if (NP > 2 && left == 2) dec_wait_vm<2 * PI - H>();
            else dec_wait_vm<PI - H>();
            const char *tk = lds.t[p % NP][0][0], *tv = lds.t[p % NP][1][0];
            dec_bf16x8_t kf[2][KS];
#pragma unroll
            for (int ks = 0; ks < KS; ks++)
#pragma unroll
                for (int t = 0; t < 2; t++) kf[t][ks] = *reinterpret_cast<const dec_bf16x8_t *>(tk + t * TILEB + (o_k ^ (64 * ks)));
            asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
            const bool more = left > NP;
            if (more) request(p + NP, false);
            dec_f32x4_t s[2];
#pragma unroll
            for (int t = 0; t < 2; t++) {
#pragma unroll
                for (int i = 0; i < 4; i++) s[t][i] = 0.f;
#pragma unroll
                for (int ks = 0; ks < KS; ks++) s[t] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(kf[t][ks], __builtin_bit_cast(dec_bf16x8_t, q[ks]), s[t], 0, 0, 0);
            }
            const int valid = valid_of(p);  // all 32, but in the last pair of a piece
            if (valid < 2 * kTile) {
#pragma unroll
                for (int t = 0; t < 2; t++)
#pragma unroll
                    for (int i = 0; i < 4; i++) s[t][i] = t * kTile + 4 * grp + i < valid ? s[t][i] : -INFINITY;
            }
            float mt = fmaxf(fmaxf(fmaxf(s[0][0], s[0][1]), fmaxf(s[0][2], s[0][3])), fmaxf(fmaxf(s[1][0], s[1][1]), fmaxf(s[1][2], s[1][3]))) * c_exp;
            if (__builtin_amdgcn_ballot_w64(mt > st.m + 8.f) != 0) {  // rare once the maxima settle
                const LanePair x = swap16(mt, mt);
                const float mnew = fmaxf(st.m, max_xor32(fmaxf(x.a, x.b)));
                const float corr = __builtin_amdgcn_exp2f(st.m - (mnew == -INFINITY ? 0.f : mnew));
                st.m = mnew;
                float ch[G];
#pragma unroll
                for (int g = 0; g < G; g++) ch[g] = __uint_as_float(__builtin_amdgcn_readlane(__float_as_uint(corr), g));
#pragma unroll
                for (int i = 0; i < 4; i++) {
                    const float f = G == 8 ? ((grp & 1) ? ch[(4 + i) % G] : ch[i % G]) : ch[i % G];
                    st.l[i] *= f;
#pragma unroll
                    for (int c = 0; c < EP; c++) st.acc[c][i] *= f;
                }
            }
            const float off = st.m == -INFINITY ? 0.f : -st.m;
            float w[2][4];
#pragma unroll
            for (int t = 0; t < 2; t++)
#pragma unroll
                for (int i = 0; i < 4; i++) w[t][i] = __builtin_amdgcn_exp2f(fmaf(s[t][i], c_exp, off));
            dec_bf16x8_t pw[SH::PARTS];
#pragma unroll
            for (int part = 0; part < SH::PARTS; part++) {
                uint32_t wd[4];
#pragma unroll
                for (int t = 0; t < 2; t++)
#pragma unroll
                    for (int i = 0; i < 4; i += 2) {
                        uint32_t pk = dec_pack_bf16(w[t][i], w[t][i + 1]);
                        asm("" : "+v"(pk));  // (or the two are rounded once more, one by one)
                        wd[2 * t + i / 2] = pk;
                        if (part + 1 < SH::PARTS) {  // what is left over, exactly
                            w[t][i] -= __uint_as_float(pk << 16);
                            w[t][i + 1] -= __uint_as_float(pk & 0xffff0000u);
                        }
                    }
                pw[part] = __builtin_bit_cast(dec_bf16x8_t, make_uint4(wd[0], wd[1], wd[2], wd[3]));
            }
            if (more) dec_wait_vm<NP * PI - H>();
            else if (NP > 2 && left == 4) dec_wait_vm<3 * PI>();
            else if (NP > 2 && left == 3) dec_wait_vm<2 * PI>();
            else if (left == 2) dec_wait_vm<PI>();
            else dec_wait_vm<0>();
            typedef short dec_s16x4_t __attribute__((ext_vector_type(4)));
            typedef __attribute__((address_space(3))) dec_s16x4_t *lds_ptr_t;
            uint2 vw[2][EP];  // rows 4 * grp + {0..3} of both tiles at column 16 * c + col
#pragma unroll
            for (int c = 0; c < EP; c++)
#pragma unroll
                for (int t = 0; t < 2; t++)
                    vw[t][c] = __builtin_bit_cast(uint2, __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_ptr_t)(tv + t * TILEB + (o_v ^ (32 * c)))));
            asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
            if (more) request(p + NP, true);
            if (valid < 2 * kTile) {  // a weight of zero times what is not finite
#pragma unroll
                for (int t = 0; t < 2; t++) {
                    const int nv = valid - t * kTile - 4 * grp;
                    const uint32_t m0 = nv >= 2 ? 0xffffffffu : nv == 1 ? 0xffffu : 0u, m1 = nv >= 4 ? 0xffffffffu : nv == 3 ? 0xffffu : 0u;
#pragma unroll
                    for (int c = 0; c < EP; c++) {
                        vw[t][c].x &= m0;
                        vw[t][c].y &= m1;
                    }
                }
            }
            constexpr uint32_t kOnes = 0x3f803f80u;
            const dec_bf16x8_t ones = __builtin_bit_cast(dec_bf16x8_t, make_uint4(kOnes, kOnes, kOnes, kOnes));
#pragma unroll
            for (int part = 0; part < SH::PARTS; part++) {
                st.l = __builtin_amdgcn_mfma_f32_16x16x32_bf16(pw[part], ones, st.l, 0, 0, 0);
#pragma unroll
                for (int c = 0; c < EP; c++) {
                    const dec_bf16x8_t vf = __builtin_bit_cast(dec_bf16x8_t, make_uint4(vw[0][c].x, vw[0][c].y, vw[1][c].x, vw[1][c].y));
                    st.acc[c] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(pw[part], vf, st.acc[c], 0, 0, 0);
                }
            }
        }
        cur += n;
    }
}

// The same on the vector unit (fp32, and bf16 where the rule of launch_one says so).  Each lane loads 16 bytes of a K row and of a V row straight into registers, 1 KiB per
// instruction; a wave keeps S tiles in flight in register sets that are refilled in place as soon as they have been consumed.
// A group of lanes (LPT of them) owns one token per row, so a wave holds several independent softmax streams.
template <int DT, int D, int G>
__device__ __forceinline__ void stream_tiles(const View &pv, const AttendArgs &a, int u, int um, int gl_all, int gl,
                                             int nloc, int cur, int u_end,
                                             const uint32_t (&qreg)[G][4], float scale_log2e, DecSoftmax<DT, D, G> &st,
                                             DecWaveLds<DT, D, G> &strips, int lane) {
    using SH = DecShape<DT, D, G>;
    auto &m = st.m;
    auto &l = st.l;
    auto &acc = st.acc;
    constexpr int EPL = SH::EPL, LPT = SH::LPT, TPW = SH::TPW, RPT = SH::RPT, ROWB = SH::ROWB, S = SH::S;
    constexpr bool SPREAD = SH::SPREAD;
    constexpr int HH = SH::HH;
    const int grp = lane / LPT, sub = lane % LPT;
    const int n_gt = ceil_tiles(gl);
    while (cur < u_end) {
        // one piece: at most 64 tiles [k0, k0+n) of one region (global or local) of unit u
        const int kk = cur;
        const bool is_glob = kk < n_gt;
        const int k0 = is_glob ? kk : kk - n_gt;
        const int region_tiles = is_glob ? n_gt : ceil_tiles(nloc);
        const int count = is_glob ? gl : nloc;
        const int n = min(min(region_tiles - k0, 64), u_end - cur);
        const int32_t *pt = is_glob ? pv.global_pt + (size_t)um * pv.maxgp
                                    : pv.local_pt + (size_t)um * pv.nlp;
        // A tile inside one page (P >= 16) needs one page id for the whole wave:
        // lane i keeps the page id of tile k0+i and the base address goes through
        // scalar registers.  In a partly filled last tile the rows beyond the last token
        // read the last valid row again and get weight zero: nothing that is not a cached
        // row of this head is ever read (a recycled page keeps whatever its last owner
        // left in it, which need not be finite).  With pages smaller than a tile every
        // tile is handled one at a time with a page lookup per row.
        // page id of the vp-th page of the region as this call reads it (with a selection: the
        // vp-th selected page; an index outside the table is clamped, never followed)
        const int32_t *sel = (is_glob && a.sel_pages) ? a.sel_pages + (size_t)u * a.sel_stride : nullptr;
        const int last_page = max(((gl_all + pv.P - 1) >> pv.logP) - 1, 0);
        auto page_at = [&](int vp) { return pt[sel ? min(max(sel[vp], 0), last_page) : vp]; };
        const bool page_per_tile = pv.logP >= 4;
        const int n_fast = page_per_tile ? n : 0;
        int ptreg = 0;

        // Row addresses of tile j (clamped to the last tile of the piece: a tile asked
        // for beyond the end is re-read and never used).  No memory access.
        auto tile_rows = [&](int j, const char *(&rowp)[RPT]) {
            j = min(j, n_fast - 1);
            const int k = k0 + j;
            const int page = __builtin_amdgcn_readlane(ptreg, j);
            const char *base = page_ptr(pv, page) + (size_t)((k * kTile) & (pv.P - 1)) * ROWB;
            const int last_row = count - 1 - k * kTile;  // wave-uniform; >= kTile - 1 except in the last tile
#pragma unroll
            for (int r = 0; r < RPT; r++)
                rowp[r] = base + ((uint32_t)min(grp + r * TPW, last_row) * ROWB + (uint32_t)(sub * 16));
        };
        // Row addresses of any tile, one page lookup per row.
        auto tile_rows_any = [&](int j, const char *(&rowp)[RPT]) {
            const int k = k0 + j;
#pragma unroll
            for (int r = 0; r < RPT; r++) {
                int tok = k * kTile + r * TPW + grp;
                tok = min(tok, count - 1);  // rows past the end re-read a valid row and get weight 0
                const int page = page_at(tok >> pv.logP);
                rowp[r] = page_ptr(pv, page) + (size_t)(tok & (pv.P - 1)) * ROWB + sub * 16;
            }
        };

        // a head's weight times word e of a V row
        auto weigh = [](float w, uint32_t v, float (&acc)[EPL], int e) __attribute__((always_inline)) {
            if constexpr (DT == WGKV_F32) {
                acc[e] = fmaf(w, __uint_as_float(v), acc[e]);
            } else {
                acc[2 * e] = fmaf(w, __uint_as_float(v << 16), acc[2 * e]);
                acc[2 * e + 1] = fmaf(w, __uint_as_float(v & 0xffff0000u), acc[2 * e + 1]);
            }
        };
        uint4 kb[S][RPT], vb[S][RPT];

        // One tile out of register set ST; the set is refilled with tile j+S.
        auto process = [&](auto st_tag, auto refill_tag, int j) {
            constexpr int ST = decltype(st_tag)::value;
            constexpr bool REFILL = decltype(refill_tag)::value;
            const int k = k0 + j;
            const char *rowp[RPT];
            if constexpr (REFILL) tile_rows(j + S, rowp);
            if constexpr (SPREAD) {
#pragma unroll
                for (int hh = 0; hh < HH; hh++) {
                    // ---- LPT partial dot products for four heads: x[r*4+g]; a K row register is
                    //      refilled as soon as it has been used ----
                    float x[LPT];
#pragma unroll
                    for (int r = 0; r < RPT; r++) {
                        const uint32_t kw[4] = {kb[ST][r].x, kb[ST][r].y, kb[ST][r].z, kb[ST][r].w};
#pragma unroll
                        for (int g = 0; g < 4; g++) x[r * 4 + g] = dec_dot<DT>(kw, qreg[4 * hh + g]);
                        __builtin_amdgcn_sched_barrier(0);
                        if constexpr (REFILL)
                            if (hh == HH - 1) kb[ST][r] = load_once16(rowp[r]);
                        __builtin_amdgcn_sched_barrier(0);
                    }
                    // ---- reduce-scatter over the lanes of the row group: lane `sub` ends up with the
                    //      full dot product x[sub], i.e. row sub/4, head 4*hh + sub%4 ----
                    float y16[16], y8[8], y4[4], y2[2];
                    if constexpr (LPT == 32) {
#pragma unroll
                        for (int i = 0; i < 16; i++) {
                            const LanePair t = swap16(x[i], x[i + 16]);
                            y16[i] = t.a + t.b;
                        }
                    } else if constexpr (LPT == 16) {
#pragma unroll
                        for (int i = 0; i < 16; i++) y16[i] = x[i];
                    }
                    if constexpr (LPT >= 16) {
#pragma unroll
                        for (int i = 0; i < 8; i++) {
                            const float lo_ = y16[i] + dpp_f<kDppRor8>(y16[i]);
                            const float hi_ = y16[i + 8] + dpp_f<kDppRor8>(y16[i + 8]);
                            y8[i] = (sub & 8) ? hi_ : lo_;
                        }
                    } else {
#pragma unroll
                        for (int i = 0; i < 8; i++) y8[i] = x[i];
                    }
#pragma unroll
                    for (int i = 0; i < 4; i++) {
                        const float lo_ = y8[i] + dpp_f<kDppShl4>(y8[i]);
                        const float hi_ = y8[i + 4] + dpp_f<kDppShr4>(y8[i + 4]);
                        y4[i] = (sub & 4) ? hi_ : lo_;
                    }
#pragma unroll
                    for (int i = 0; i < 2; i++) {
                        const float lo_ = y4[i] + dpp_f<kDppXor2>(y4[i]);
                        const float hi_ = y4[i + 2] + dpp_f<kDppXor2>(y4[i + 2]);
                        y2[i] = (sub & 2) ? hi_ : lo_;
                    }
                    float sc;
                    {
                        const float lo_ = y2[0] + dpp_f<kDppXor1>(y2[0]);
                        const float hi_ = y2[1] + dpp_f<kDppXor1>(y2[1]);
                        sc = (sub & 1) ? hi_ : lo_;
                    }
                    const int tok_l = k * kTile + (sub >> 2) * TPW + grp;
                    sc = tok_l < count ? sc * scale_log2e : -INFINITY;
                    // ---- online softmax on one (row, head) per lane; the lanes of the row group with
                    //      the same sub%4 hold the rows of the same head ----
                    auto over_rows = [&](float v, auto op) __attribute__((always_inline)) {
                        if constexpr (LPT == 32) {
                            const LanePair t = swap16(v, v);
                            v = op(t.a, t.b);
                        }
                        if constexpr (LPT >= 16) {
                            v = op(v, dpp_f<kDppRor8>(v));
                            return op(v, dpp_f<kDppRor4>(v));
                        } else {
                            const float up = dpp_f<kDppShl4>(v), dn = dpp_f<kDppShr4>(v);
                            return op(v, (sub & 4) ? dn : up);
                        }
                    };
                    const float mt = over_rows(sc, [](float p, float q) { return fmaxf(p, q); });
                    const float mnew = fmaxf(m[hh], mt);
                    const float msafe = mnew == -INFINITY ? 0.f : mnew;
                    const float corr = __builtin_amdgcn_exp2f(m[hh] - msafe);
                    const float pl = __builtin_amdgcn_exp2f(sc - msafe);
                    l[hh] = l[hh] * corr + over_rows(pl, [](float p, float q) { return p + q; });
                    if (__builtin_amdgcn_ballot_w64(mnew > m[hh]) != 0) {  // rare once the maxima settle
                        const float c0 = dpp_f<0x00>(corr), c1 = dpp_f<0x55>(corr);
                        const float c2 = dpp_f<0xAA>(corr), c3 = dpp_f<0xFF>(corr);
#pragma unroll
                        for (int e = 0; e < EPL; e++) {
                            acc[4 * hh][e] *= c0; acc[4 * hh + 1][e] *= c1; acc[4 * hh + 2][e] *= c2; acc[4 * hh + 3][e] *= c3;
                        }
                    }
                    m[hh] = mnew;
                    strips.p[hh][lane] = pl;
                }
                // ---- weights back to the row layout through the wave's LDS strip ----
                __builtin_amdgcn_wave_barrier();
#pragma unroll
                for (int r = 0; r < RPT; r++) {
                    float pg[G];
#pragma unroll
                    for (int hh = 0; hh < HH; hh++) {
                        const float4 pr = *reinterpret_cast<const float4 *>(&strips.p[hh][grp * LPT + r * 4]);
                        pg[4 * hh] = pr.x; pg[4 * hh + 1] = pr.y; pg[4 * hh + 2] = pr.z; pg[4 * hh + 3] = pr.w;
                    }
                    const uint32_t vw[4] = {vb[ST][r].x, vb[ST][r].y, vb[ST][r].z, vb[ST][r].w};
#pragma unroll
                    for (int e = 0; e < 4; e++) {
#pragma unroll
                        for (int g = 0; g < G; g++) weigh(pg[g], vw[e], acc[g], e);
                    }
                    __builtin_amdgcn_sched_barrier(0);
                    if constexpr (REFILL) vb[ST][r] = load_once16(rowp[r] + pv.v_off);
                    __builtin_amdgcn_sched_barrier(0);
                }
                __builtin_amdgcn_wave_barrier();
            } else {
                // ---- scores of the tile, every lane of a row group gets all of them ----
                float s[RPT][G];
#pragma unroll
                for (int r = 0; r < RPT; r++) {
                    const uint32_t kw[4] = {kb[ST][r].x, kb[ST][r].y, kb[ST][r].z, kb[ST][r].w};
                    const int tok = k * kTile + r * TPW + grp;
#pragma unroll
                    for (int g = 0; g < G; g++) {
                        const float d = group_sum<LPT>(dec_dot<DT>(kw, qreg[g]));
                        s[r][g] = tok < count ? d * scale_log2e : -INFINITY;
                    }
                }
                __builtin_amdgcn_sched_barrier(0);  // the K registers are free from here on
                if constexpr (REFILL) {
#pragma unroll
                    for (int r = 0; r < RPT; r++) kb[ST][r] = load_once16(rowp[r]);
                }
                __builtin_amdgcn_sched_barrier(0);
                // ---- online softmax per query head, one rescale per tile ----
                float p[RPT][G];
#pragma unroll
                for (int g = 0; g < G; g++) {
                    float mt = s[0][g];
#pragma unroll
                    for (int r = 1; r < RPT; r++) mt = fmaxf(mt, s[r][g]);
                    const float mnew = fmaxf(m[g], mt);
                    const float msafe = mnew == -INFINITY ? 0.f : mnew;
                    const float corr = __builtin_amdgcn_exp2f(m[g] - msafe);
                    m[g] = mnew;
                    float ps = 0.f;
#pragma unroll
                    for (int r = 0; r < RPT; r++) {
                        p[r][g] = __builtin_amdgcn_exp2f(s[r][g] - msafe);
                        ps += p[r][g];
                    }
                    l[g] = l[g] * corr + ps;
#pragma unroll
                    for (int e = 0; e < EPL; e++) acc[g][e] *= corr;
                }
#pragma unroll
                for (int r = 0; r < RPT; r++) {
                    const uint32_t vw[4] = {vb[ST][r].x, vb[ST][r].y, vb[ST][r].z, vb[ST][r].w};
#pragma unroll
                    for (int e = 0; e < 4; e++)
#pragma unroll
                        for (int g = 0; g < G; g++) weigh(p[r][g], vw[e], acc[g], e);
                }
                __builtin_amdgcn_sched_barrier(0);  // the V registers are free from here on
                if constexpr (REFILL) {
#pragma unroll
                    for (int r = 0; r < RPT; r++) vb[ST][r] = load_once16(rowp[r] + pv.v_off);
                }
                __builtin_amdgcn_sched_barrier(0);
            }
        };

        if (n_fast > 0) {
            ptreg = page_at(((k0 + min(lane, n_fast - 1)) * kTile) >> pv.logP);
            // prologue: fill every register set
#pragma unroll
            for (int st = 0; st < S; st++) {
                const char *rowp[RPT];
                tile_rows(st, rowp);
#pragma unroll
                for (int r = 0; r < RPT; r++) kb[st][r] = load_once16(rowp[r]);
#pragma unroll
                for (int r = 0; r < RPT; r++) vb[st][r] = load_once16(rowp[r] + pv.v_off);
            }
            // Main loop: S tiles per trip, straight-line, so that every wait is for exactly
            // the load that is needed and the younger ones stay in flight.  It runs while every
            // refill is a real tile of the piece.
            using std::integral_constant;
            constexpr std::true_type kRefill{};
            constexpr std::false_type kNoRefill{};
            static_assert(S == 2 || S == 4, "the loops below are written out for 2 or 4 register sets");
            int j = 0;
            for (; j + 2 * S <= n_fast; j += S) {
                process(integral_constant<int, 0>{}, kRefill, j);
                process(integral_constant<int, 1>{}, kRefill, j + 1);
                if constexpr (S == 4) {
                    process(integral_constant<int, 2>{}, kRefill, j + 2);
                    process(integral_constant<int, 3>{}, kRefill, j + 3);
                }
            }
            // the last full trip: only the first n_fast - j - S sets still have a tile to fetch
            // (a set without one is left alone: asking again for the last tile would be traffic
            // for nothing)
            if (j + S <= n_fast) {
                const int more = n_fast - j - S;
                if (more > 0) process(integral_constant<int, 0>{}, kRefill, j);
                else process(integral_constant<int, 0>{}, kNoRefill, j);
                if constexpr (S == 4) {
                    if (more > 1) process(integral_constant<int, 1>{}, kRefill, j + 1);
                    else process(integral_constant<int, 1>{}, kNoRefill, j + 1);
                    if (more > 2) process(integral_constant<int, 2>{}, kRefill, j + 2);
                    else process(integral_constant<int, 2>{}, kNoRefill, j + 2);
                    process(integral_constant<int, 3>{}, kNoRefill, j + 3);
                } else {
                    process(integral_constant<int, 1>{}, kNoRefill, j + 1);
                }
                j += S;
            }
            // the last n_fast % S tiles are already in their register sets
            if (j < n_fast) process(integral_constant<int, 0>{}, kNoRefill, j);
            if constexpr (S == 4) {
                if (j + 1 < n_fast) process(integral_constant<int, 1>{}, kNoRefill, j + 1);
                if (j + 2 < n_fast) process(integral_constant<int, 2>{}, kNoRefill, j + 2);
            }
        }
        // whatever is left of the piece, one tile at a time through register set 0
        for (int j = n_fast; j < n; j++) {
            const char *rowp[RPT];
            tile_rows_any(j, rowp);
#pragma unroll
            for (int r = 0; r < RPT; r++) kb[0][r] = load_once16(rowp[r]);
#pragma unroll
            for (int r = 0; r < RPT; r++) vb[0][r] = load_once16(rowp[r] + pv.v_off);
            process(std::integral_constant<int, 0>{}, std::false_type{}, j);
        }
        cur += n;
    }
}

// A wave's part of a unit: its query, and tiles [w0, w1) into a fresh softmax.
template <int DT, int D, int G>
__device__ __forceinline__ void run_part(const View &pv, const AttendArgs &a, int u, int um, int gl_all, int gl, int nloc, int w0, int w1,
                                         DecSoftmax<DT, D, G> &st, DecWaveLds<DT, D, G> &lds, int lane) {
    using SH = DecShape<DT, D, G>;
    st.init();
    if (w0 >= w1) return;
    // wave-uniform, which the compiler does not always see: the requests' bases are scalar operands (the vector unit's loads have no use
    // for it: 166 calls of many units there 1.4 % slower with it)
    if constexpr (DT == WGKV_BF16) {
        u = __builtin_amdgcn_readfirstlane(u);
        um = __builtin_amdgcn_readfirstlane(um);
        gl_all = __builtin_amdgcn_readfirstlane(gl_all);
        gl = __builtin_amdgcn_readfirstlane(gl);
        nloc = __builtin_amdgcn_readfirstlane(nloc);
        w0 = __builtin_amdgcn_readfirstlane(w0);
        w1 = __builtin_amdgcn_readfirstlane(w1);
    }
    const char *qu = a.q + (size_t)u * G * D * SH::ES;
    if constexpr (DT == WGKV_BF16) {
        dec_u32x4_t q[D / 32];
#pragma unroll
        for (int ks = 0; ks < D / 32; ks++)
            q[ks] = *reinterpret_cast<const dec_u32x4_t *>(qu + ((lane & 15) % G) * (D * 2) + (4 * ks + (lane >> 4)) * 16);
        // (a scale of zero stays a hair above it: -inf times it stays -inf)
        stream_pairs<D, G>(pv, a, u, um, gl_all, gl, nloc, w0, w1, q, fmaxf(fabsf(a.scale_log2e), 1e-37f), st, lds, lane);
    } else {
        uint32_t qreg[G][4];
#pragma unroll
        for (int g = 0; g < G; g++) {
            const uint4 t4 = *reinterpret_cast<const uint4 *>(qu + lane % SH::LPT * 16 + (size_t)g * D * SH::ES);
            qreg[g][0] = t4.x; qreg[g][1] = t4.y; qreg[g][2] = t4.z; qreg[g][3] = t4.w;
        }
        stream_tiles<DT, D, G>(pv, a, u, um, gl_all, gl, nloc, w0, w1, qreg, a.scale_log2e, st, lds, lane);
    }
}

// What the decode kernels have in LDS for the states of a block, and how a unit's output is dealt over threads.
template <int DT, int D, int G>
struct DecOut {
    static constexpr int NSW = DecShape<DT, D, G>::NSW;
    static constexpr int NST = kAttnWaves * NSW;  // softmax states of a block
    static constexpr int PAR = 4 * kAttnThreads / (G * D);  // partials that a block reads side by side, 16 bytes a thread
    static constexpr int VPT = G * D >= 2 * kAttnThreads ? G * D / kAttnThreads : 2;  // output elements per thread
    static constexpr int NT = G * D / VPT;        // threads that hold some
    static_assert(NT <= kAttnThreads && D % VPT == 0 && (VPT == 2 || VPT == 4), "");
};
template <int DT, int D, int G>
struct DecStates {
    static constexpr int N = DecOut<DT, D, G>::NST > DecOut<DT, D, G>::PAR ? DecOut<DT, D, G>::NST : DecOut<DT, D, G>::PAR;
    float m[N][G], l[N][G];
    __attribute__((aligned(16))) float acc[N][G * D];
};

// A wave's states into their places.
template <int DT, int D, int G>
__device__ __forceinline__ void put_states(DecStates<DT, D, G> &s, int wave, int lane, const DecSoftmax<DT, D, G> &w) {
    using SH = DecShape<DT, D, G>;
    if constexpr (DT == WGKV_BF16) {
        const int grp = lane >> 4, col = lane & 15;
        if (grp < (G + 3) / 4) {  // the other lanes hold the same
#pragma unroll
            for (int i = 0; i < 4; i++)
                if (4 * grp + i < G) {
#pragma unroll
                    for (int c = 0; c < SH::EP; c += 4)
                        *reinterpret_cast<float4 *>(&s.acc[wave][(4 * grp + i) * D + col * SH::EP + c]) =
                            make_float4(w.acc[c][i], w.acc[c + 1][i], w.acc[c + 2][i], w.acc[c + 3][i]);
                    if (col == 0) s.l[wave][4 * grp + i] = w.l[i];
                }
            if (lane < G) s.m[wave][lane] = w.m;
        }
    } else {
        const int grp = lane / SH::LPT, sub = lane % SH::LPT, st = wave * SH::TPW + grp;
#pragma unroll
        for (int g = 0; g < G; g++)
#pragma unroll
            for (int e = 0; e < SH::EPL; e += 4)
                *reinterpret_cast<float4 *>(&s.acc[st][g * D + sub * SH::EPL + e]) =
                    make_float4(w.acc[g][e], w.acc[g][e + 1], w.acc[g][e + 2], w.acc[g][e + 3]);
        if constexpr (SH::SPREAD) {
            if (sub < 4) {  // m[hh] and l[hh] belong to head 4 * hh + sub % 4
#pragma unroll
                for (int hh = 0; hh < SH::HH; hh++) {
                    s.m[st][4 * hh + sub] = w.m[hh];
                    s.l[st][4 * hh + sub] = w.l[hh];
                }
            }
        } else if (sub == 0) {
#pragma unroll
            for (int g = 0; g < G; g++) {
                s.m[st][g] = w.m[g];
                s.l[st][g] = w.l[g];
            }
        }
    }
}

// Place x of a state's accumulators is output element ...
constexpr float kTiny = 1.401298464e-45f;  // the smallest above zero
template <int DT, int D>
__device__ __forceinline__ int out_of(int x) {
    constexpr int EP = D / 16;
    return DT == WGKV_BF16 ? x / D * D + x % EP * 16 + x % D / EP : x;
}

// On the matrix cores a weight may be 256: what leaves a block or a wave, sums of weights and of weighted values, is scaled back by that much (its
// maximum stays what it is, all partials are scaled alike), so that partials of values at the end of the range can be added up.
template <int DT>
constexpr float kBack = DT == WGKV_BF16 ? 1.f / 256.f : 1.f;
// N states from s0 on into one, for places x0 .. of head xg.  BACK: scaled back.
template <int N, bool BACK, int DT, int D, int G>
__device__ __forceinline__ void fold_states(const DecStates<DT, D, G> &s, int s0, int x0, int xg, float &M, float &L,
                                            float (&o)[DecOut<DT, D, G>::VPT]) {
    constexpr int VPT = DecOut<DT, D, G>::VPT;
    M = s.m[s0][xg];
    L = 0.f;
#pragma unroll
    for (int i = 1; i < N; i++) M = fmaxf(M, s.m[s0 + i][xg]);
    const float Ms = M == -INFINITY ? 0.f : M;
#pragma unroll
    for (int e = 0; e < VPT; e++) o[e] = 0.f;
#pragma unroll
    for (int i = 0; i < N; i++) {
        const float f = __builtin_amdgcn_exp2f(s.m[s0 + i][xg] - Ms);  // 0 for a state that saw nothing
        L = fmaf(s.l[s0 + i][xg], f, L);
#pragma unroll
        for (int e = 0; e < VPT; e++) o[e] = fmaf(s.acc[s0 + i][x0 + e], f, o[e]);
    }
    if constexpr (BACK && kBack<DT> != 1.f) {
        L *= kBack<DT>;
#pragma unroll
        for (int e = 0; e < VPT; e++) o[e] *= kBack<DT>;
    }
}

// bf16: the weighted sums of tiles [p0, p1) of a unit once more, for a wave one of whose sums is not finite, with each key's whole weight
// times its value.  The parts that a weight is split into do not carry an infinity of V: later ones are zero or of either sign, and zero times
// an infinity, or the sum of two that differ in sign, is NaN; and so is an infinity times a factor too small
// for its type.  A finite value gets here only if it is above some 1e36 (weights of up to 256 in the sums), so this is short and not
// fast: a lane works out the scores of a key (64 keys at a time), then the lanes go through the keys.  Relative to the same maximum as
// the sums that it replaces (states s0 .. s0 + N - 1), and scaled back like them; a weight too small for its type stays above zero as a number does.
template <int N, int DT, int D, int G>
__device__ __forceinline__ void sum_again(int u, int um, int gl_all, int gl, int nloc, int p0, int p1,
                                          const DecStates<DT, D, G> &s, int s0, int x0, int xg, DecWaveLds<DT, D, G> &lds, int lane,
                                          float (&o)[DecOut<DT, D, G>::VPT]) {
    constexpr int VPT = DecOut<DT, D, G>::VPT;
    // the kernel's arguments, read again: kept in registers past the loops for this they cost every call some spilled ones (batch 1 at 32K
    // 13.97 us; 13.92 with this and the branch to here marked as rare; 13.90 without the check)
    auto karg = (const char *)__builtin_amdgcn_kernarg_segment_ptr();
    asm volatile("" : "+s"(karg));
    const View &pv = *(const View *)karg;
    const AttendArgs &a = *(const AttendArgs *)(karg + (sizeof(View) + alignof(AttendArgs) - 1) / alignof(AttendArgs) * alignof(AttendArgs));
    static_assert(sizeof(DecStrip<G>) <= sizeof(lds), "");
    DecStrip<G> &strip = *reinterpret_cast<DecStrip<G> *>(&lds);  // the wave has no requests under way
    const char *qu = a.q + (size_t)u * G * D * 2;
    const int n_gt = ceil_tiles(gl), last_page = max(((gl_all + pv.P - 1) >> pv.logP) - 1, 0);
    const int32_t *sel = a.sel_pages ? a.sel_pages + (size_t)u * a.sel_stride : nullptr;
#pragma unroll
    for (int e = 0; e < VPT; e++) o[e] = 0.f;
#pragma unroll 1
    for (int t0 = p0; t0 < p1; t0 += 4) {
        const int t = t0 + (lane >> 4);
        const bool is_glob = t < n_gt;
        const int tok = (is_glob ? t : t - n_gt) * kTile + (lane & 15);
        const bool is = t < p1 && tok < (is_glob ? gl : nloc);
        if (is) {
            const int vp = tok >> pv.logP;
            const int page = is_glob ? pv.global_pt[(size_t)um * pv.maxgp + (sel ? min(max(sel[vp], 0), last_page) : vp)]
                                     : pv.local_pt[(size_t)um * pv.nlp + vp];
            const char *row = page_ptr(pv, page) + (size_t)(tok & (pv.P - 1)) * (D * 2);
            float sc[G];
#pragma unroll
            for (int g = 0; g < G; g++) sc[g] = 0.f;
#pragma unroll 1
            for (int x = 0; x < D / 8; x++) {
                const uint4 kx = *reinterpret_cast<const uint4 *>(row + x * 16);
                const uint32_t kw[4] = {kx.x, kx.y, kx.z, kx.w};
#pragma unroll
                for (int g = 0; g < G; g++) {
                    const uint4 qx = *reinterpret_cast<const uint4 *>(qu + g * (D * 2) + x * 16);
                    const uint32_t qw[4] = {qx.x, qx.y, qx.z, qx.w};
#pragma unroll
                    for (int e = 0; e < 4; e++) {
                        sc[g] = fmaf(__uint_as_float(kw[e] << 16), __uint_as_float(qw[e] << 16), sc[g]);
                        sc[g] = fmaf(__uint_as_float(kw[e] & 0xffff0000u), __uint_as_float(qw[e] & 0xffff0000u), sc[g]);
                    }
                }
            }
#pragma unroll
            for (int g = 0; g < G; g++) {
                float m = s.m[s0][g];
#pragma unroll
                for (int i = 1; i < N; i++) m = fmaxf(m, s.m[s0 + i][g]);
                const float x = sc[g] * a.scale_log2e, w = __builtin_amdgcn_exp2f(x - (m == -INFINITY ? 0.f : m)) * kBack<DT>;
                strip.w[lane][g] = x > -INFINITY ? fmaxf(w, kTiny) : w;
            }
            strip.v[lane] = row + pv.v_off;
        }
        __builtin_amdgcn_wave_barrier();
#pragma unroll 1
        for (uint64_t left = __builtin_amdgcn_ballot_w64(is); left != 0; left &= left - 1) {
            const int j = __builtin_ctzll(left);
            const float w = strip.w[j][xg];
            const char *row = strip.v[j];
#pragma unroll
            for (int e = 0; e < VPT; e++)
                o[e] = fmaf(w, __uint_as_float((uint32_t)*reinterpret_cast<const uint16_t *>(row + out_of<DT, D>(x0 + e) % D * 2) << 16), o[e]);
        }
        __builtin_amdgcn_wave_barrier();
    }
}

// Whether a thread of the wave has a sum that is not finite.
template <int VPT>
__device__ __forceinline__ bool any_not_finite(const float (&o)[VPT]) {
    float t = fabsf(o[0]) + fabsf(o[1]);
    if constexpr (VPT == 4) t += fabsf(o[2]) + fabsf(o[3]);
    return __builtin_amdgcn_ballot_w64(!(t < INFINITY)) != 0;
}

// The maximum of a partial is kept so that what a buffer load returns past the buffer's end, zero, stands for "nothing seen".
constexpr uint32_t kNoM = 0xff800000u;  // -inf
__device__ __forceinline__ float partial_m(uint32_t x) { return __uint_as_float(x ^ kNoM); }
// The partial of a slot goes out with device-scope stores ...
template <int D, int G, int VPT>
__device__ __forceinline__ void put_partial(__amdgpu_buffer_rsrc_t r_ml, __amdgpu_buffer_rsrc_t r_acc, int slot, int x0, int xg,
                                            float M, float L, const float (&o)[VPT]) {
    const uint32_t rec0 = (uint32_t)slot * G, off = rec0 * (D * 4) + x0 * 4;
    if constexpr (VPT == 4) {
        const u32x4 pk = {__float_as_uint(o[0]), __float_as_uint(o[1]), __float_as_uint(o[2]), __float_as_uint(o[3])};
        __builtin_amdgcn_raw_buffer_store_b128(pk, r_acc, off, 0, kCoherent);
    } else {
        const u32x2 pk = {__float_as_uint(o[0]), __float_as_uint(o[1])};
        __builtin_amdgcn_raw_buffer_store_b64(pk, r_acc, off, 0, kCoherent);
    }
    if (x0 % D == 0) {
        const u32x2 pk = {__float_as_uint(M) ^ kNoM, __float_as_uint(L)};
        __builtin_amdgcn_raw_buffer_store_b64(pk, r_ml, (rec0 + xg) * 8, 0, kCoherent);
    }
}
// ... and np of them from slot0 on, asked for eight together (four where a thread has more than two parts), become one; a thread has NP parts of the output, 64 threads
// apart, whose loads go out together too.
template <int D, int G, int NP, int VPT>
__device__ __forceinline__ void fold_partials(__amdgpu_buffer_rsrc_t r_ml, __amdgpu_buffer_rsrc_t r_acc, int slot0, int np, const int (&x0)[NP],
                                              float (&L)[NP], float (&o)[NP][VPT]) {
    float M[NP];
#pragma unroll
    for (int k = 0; k < NP; k++) {
        M[k] = -INFINITY;
        L[k] = 0.f;
#pragma unroll
        for (int e = 0; e < VPT; e++) o[k][e] = 0.f;
    }
    constexpr int MB = NP > 2 ? 4 : 8;
    for (int q0 = 0; q0 < np; q0 += MB) {
        u32x2 ml[NP][MB];
        uint32_t av[NP][MB][VPT];
#pragma unroll
        for (int i = 0; i < MB; i++) {
            const uint32_t rec = (uint32_t)(slot0 + min(q0 + i, np - 1)) * G;
#pragma unroll
            for (int k = 0; k < NP; k++) {
                ml[k][i] = __builtin_amdgcn_raw_buffer_load_b64(r_ml, (rec + x0[k] / D) * 8, 0, kCoherent);
                const uint32_t off = rec * (D * 4) + x0[k] * 4;
                if constexpr (VPT == 4) {
                    const u32x4 v = __builtin_amdgcn_raw_buffer_load_b128(r_acc, off, 0, kCoherent);
                    av[k][i][0] = v.x; av[k][i][1] = v.y; av[k][i][2] = v.z; av[k][i][3] = v.w;
                } else {
                    const u32x2 v = __builtin_amdgcn_raw_buffer_load_b64(r_acc, off, 0, kCoherent);
                    av[k][i][0] = v.x; av[k][i][1] = v.y;
                }
            }
        }
#pragma unroll
        for (int k = 0; k < NP; k++) {
            float mb = M[k];
#pragma unroll
            for (int i = 0; i < MB; i++) mb = fmaxf(mb, partial_m(ml[k][i].x));  // a repeated last one changes nothing
            const float ms = mb == -INFINITY ? 0.f : mb;
            const float c = fmaxf(__builtin_amdgcn_exp2f(M[k] - ms), kTiny);
            L[k] *= c;
#pragma unroll
            for (int e = 0; e < VPT; e++) o[k][e] *= c;
#pragma unroll
            for (int i = 0; i < MB; i++)
                if (q0 + i < np) {
                    const float f = fmaxf(__builtin_amdgcn_exp2f(partial_m(ml[k][i].x) - ms), kTiny);  // (an infinity times zero is none)
                    L[k] = fmaf(__uint_as_float(ml[k][i].y), f, L[k]);
#pragma unroll
                    for (int e = 0; e < VPT; e++) o[k][e] = fmaf(__uint_as_float(av[k][i][e]), f, o[k][e]);
                }
            M[k] = mb;
        }
    }
}

// The same by all threads of a block: a partial is read by G * D / 4 of them, 16 bytes each, so several partials are read side by
// side and up to 16 one behind the other in one round trip; the sums of those side by side meet in LDS.
template <int DT, int D, int G>
__device__ __forceinline__ void fold_partials_block(const AttendArgs &a, int slot0, int np, DecStates<DT, D, G> &s, int tid,
                                                    int x0, int xg, float &L, float (&o)[DecOut<DT, D, G>::VPT]) {
    constexpr int TP = G * D / 4, PAR = DecOut<DT, D, G>::PAR;
    static_assert(TP * PAR == kAttnThreads, "");
    // (a buffer that ends behind the last partial: an access past it moves no bytes)
    const uint32_t slots = (uint32_t)__builtin_amdgcn_readfirstlane(slot0 + np);
    const __amdgpu_buffer_rsrc_t r_acc = part_rsrc(a.part_acc, slots * (G * D * 4));
    const __amdgpu_buffer_rsrc_t r_ml = part_rsrc(a.part_ml, slots * (G * 8));
    const int pi = tid / TP, x = (tid % TP) * 4, g = x / D;
    float M = -INFINITY, l = 0.f, v[4] = {0.f, 0.f, 0.f, 0.f};
    auto batch = [&](auto mb_tag, int q0) __attribute__((always_inline)) {
        constexpr int MB = decltype(mb_tag)::value;
        u32x2 ml[MB];
        u32x4 av[MB];
#pragma unroll
        for (int i = 0; i < MB; i++) {
            const uint32_t rec = (uint32_t)(slot0 + q0 + i * PAR) * G;
            ml[i] = __builtin_amdgcn_raw_buffer_load_b64(r_ml, (rec + g) * 8, 0, kCoherent);
            av[i] = __builtin_amdgcn_raw_buffer_load_b128(r_acc, rec * (D * 4) + x * 4, 0, kCoherent);
        }
        float mb = M;
#pragma unroll
        for (int i = 0; i < MB; i++) mb = fmaxf(mb, partial_m(ml[i].x));
        const float ms = mb == -INFINITY ? 0.f : mb, c = fmaxf(__builtin_amdgcn_exp2f(M - ms), kTiny);
        l *= c;
#pragma unroll
        for (int e = 0; e < 4; e++) v[e] *= c;
#pragma unroll
        for (int i = 0; i < MB; i++) {
            const float f = fmaxf(__builtin_amdgcn_exp2f(partial_m(ml[i].x) - ms), kTiny);  // (an infinity times zero is none)
            l = fmaf(__uint_as_float(ml[i].y), f, l);
#pragma unroll
            for (int e = 0; e < 4; e++) v[e] = fmaf(__uint_as_float(av[i][e]), f, v[e]);
        }
        M = mb;
    };
    for (int q0 = 0; q0 < np; q0 += 16 * PAR) {
        // (code that runs once comes out of a cold instruction cache: about 70 ns for 64 bytes, so no more of it than it takes)
        if (np - q0 > 12 * PAR) batch(std::integral_constant<int, 16>{}, q0 + pi);
        else if (np - q0 > 8 * PAR) batch(std::integral_constant<int, 12>{}, q0 + pi);
        else batch(std::integral_constant<int, 8>{}, q0 + pi);
    }
    if constexpr (PAR == 1) {
        static_assert(PAR > 1 || DecOut<DT, D, G>::VPT == 4, "");
        L = l;
#pragma unroll
        for (int e = 0; e < DecOut<DT, D, G>::VPT; e++) o[e] = v[e];
    } else {
        *reinterpret_cast<float4 *>(&s.acc[pi][x]) = make_float4(v[0], v[1], v[2], v[3]);
        if (x % D == 0) {
            s.m[pi][g] = M;
            s.l[pi][g] = l;
        }
        __syncthreads();
        float m;
        fold_states<PAR, false>(s, 0, x0, xg, m, L, o);
    }
}

constexpr int kMaxUnits = 512;  // and no more than there are blocks
template <int DT, int D, int G>
struct DecBlocksLds {
    DecWaveLds<DT, D, G> wave[kAttnWaves];
    DecStates<DT, D, G> states;
    int ts[kMaxUnits + 1];  // pieces (or, with even shares, tiles) before unit u
    int gl[kMaxUnits];      // entries in the unit's global cache
    int gt[kMaxUnits];      // those of them that are read
    int nl[kMaxUnits];      // tokens in its ring
    int um[kMaxUnits];      // its index into the per-unit metadata
    int tmp[3 * kAttnWaves];
    int arrived;
};
template <int DT, int D, int G, bool FEW>  // FEW: at most 64 units
__device__ __forceinline__ void decode_blocks(const View &pv, const AttendArgs &a) {
    using OUT = DecOut<DT, D, G>;
    constexpr int VPT = OUT::VPT, NT = OUT::NT;
    extern __shared__ __attribute__((aligned(1024))) char s_mem[];
    auto &lds = *reinterpret_cast<DecBlocksLds<DT, D, G> *>(s_mem);
    auto &s_wave_lds = lds.wave;
    auto &s_st = lds.states;
    auto &s_ts = lds.ts;
    auto &s_gl = lds.gl;
    auto &s_gt = lds.gt;
    auto &s_nl = lds.nl;
    auto &s_um = lds.um;
    auto &s_tmp = lds.tmp;
    auto &s_arrived = lds.arrived;

    const int n_units = a.n_seqs * pv.Hkv, n_blocks = (int)gridDim.x;
    const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    // What stands in front of the first row is a chain of round trips and of instructions that a block's one wave per SIMD issues
    // one after the other, and every call pays it: all that is known early is asked for together, what every block needs is found
    // by every wave for itself (no barrier) and, for up to 64 units, kept in a register of the unit's lane (no LDS), and
    // quotients of small numbers come from a reciprocal.
    asm volatile("" ::"s"(a.out), "s"(a.part_acc_bytes), "s"(a.sel_stride), "s"(pv.v_off), "s"(pv.ahead));  // the arguments' lines
    auto unit_of = [&](int u, int &um, int &gl, int &gt, int &nl) __attribute__((always_inline)) {
        const int b = (int)(((float)u + 0.5f) * __builtin_amdgcn_rcpf((float)pv.Hkv)), h = u - b * pv.Hkv;  // exact: u < 1024
        const int sid = a.sid[b];
        um = unit_meta(pv, sid, a.layer, h);
        const int t = pv.seq_len[sid * pv.L + a.layer];
        gl = pv.global_len[um];
        gt = global_tokens(pv, a, u, gl);
        nl = min(t, pv.W);
    };
    // pieces of a unit of `tiles` tiles at about `most` tiles a piece; every unit has one at least (a unit with nothing
    // cached writes its zeros).  Any number is correct: a quotient that rounds the other way moves a boundary.
    auto pieces_of = [](int tiles, int most) __attribute__((always_inline)) {
        return tiles <= kWholeTiles ? 1 : max(1, (int)((float)(tiles + most - 1) * __builtin_amdgcn_rcpf((float)most)));
    };
    auto least_piece = [&](int total) __attribute__((always_inline)) {
        return min(max(total / kStreamBlocks, kMinPieceTiles), kMinBlockTiles);
    };
    auto even_share = [&](int total, int used) __attribute__((always_inline)) {
        return max(kMinBlockTiles, (total + used * kUnitStartTiles + n_blocks - 1) / n_blocks);
    };
    const int mine_at = FEW ? wave * (kMaxUnits / kAttnWaves) : 0;  // a wave's own part of the lists, or the block's
    int listed, share = 0, u = 0;  // share: tiles of a block's even share, 0: pieces
    if constexpr (FEW) {
        int l_um, l_gl, l_gt, l_nl;  // of unit `lane`
        unit_of(min(lane, n_units - 1), l_um, l_gl, l_gt, l_nl);
        const bool is = lane < n_units;
        const int tiles = is ? ceil_tiles(l_gt) + ceil_tiles(l_nl) : 0;
        const int total = __builtin_amdgcn_readlane(wave_incl_scan(tiles, lane), 63);
        const int used = __builtin_popcountll(__builtin_amdgcn_ballot_w64(tiles > 0));
        // the smallest piece with which all pieces fit the grid, between what an even split would need and what
        // always fits; a few units leave nothing to look for between the two
        const float per = (float)total;
        int lo = max(least_piece(total), (int)(per * __builtin_amdgcn_rcpf((float)n_blocks)));
        int hi = max(lo, (int)(per * __builtin_amdgcn_rcpf((float)max(1, n_blocks - n_units))) + 1);
        for (int i = 0; i < 5 && (hi - lo) * 16 > hi; i++) {
            const int mid = (lo + hi) >> 1;
            const int np = is ? pieces_of(tiles, mid) : 0;
            if (__builtin_amdgcn_readlane(wave_incl_scan(np, lane), 63) <= n_blocks) hi = mid; else lo = mid;
        }
        // (the rounding of the quotients decides whether they do fit: counted, not assumed)
        int mine = is ? pieces_of(tiles, hi) : 0;
        int l_te = wave_incl_scan(mine, lane);
        if (__builtin_amdgcn_readlane(l_te, 63) > n_blocks ||
            hi > max(kMinBlockTiles, (int)((float)(total + used * kUnitStartTiles) * __builtin_amdgcn_rcpf((float)n_blocks)) + 1)) {
            share = even_share(total, used);
            mine = tiles + (tiles > 0 ? kUnitStartTiles : 0);
            l_te = wave_incl_scan(mine, lane);
        }
        listed = __builtin_amdgcn_readlane(l_te, 63);
        if (is) {
            s_ts[mine_at + lane] = l_te - mine;
            s_ts[mine_at + lane + 1] = l_te;
            s_um[mine_at + lane] = l_um;
            s_gl[mine_at + lane] = l_gl;
            s_gt[mine_at + lane] = l_gt;
            s_nl[mine_at + lane] = l_nl;
        }
        __builtin_amdgcn_wave_barrier();
    } else {
        constexpr int NU = kMaxUnits / kAttnThreads;  // consecutive units a thread looks after, asked for together
        int um[NU], gl[NU], gt[NU], nl[NU], tl[NU], sum = 0, some = 0;
#pragma unroll
        for (int i = 0; i < NU; i++) unit_of(min((int)threadIdx.x * NU + i, n_units - 1), um[i], gl[i], gt[i], nl[i]);
#pragma unroll
        for (int i = 0; i < NU; i++) {
            const int v = (int)threadIdx.x * NU + i;
            tl[i] = 0;
            if (v < n_units) {
                s_um[v] = um[i];
                s_gl[v] = gl[i];
                s_gt[v] = gt[i];
                s_nl[v] = nl[i];
                tl[i] = ceil_tiles(gt[i]) + ceil_tiles(nl[i]);
            }
            sum += tl[i];
            some += tl[i] > 0 ? 1 : 0;
        }
        const int inc_tiles = wave_incl_scan(sum, lane), inc_units = wave_incl_scan(some, lane);
        if (lane == 63) {
            s_tmp[wave] = inc_tiles;
            s_tmp[kAttnWaves + wave] = inc_units;
        }
        __syncthreads();
        int total = 0, used = 0, at = inc_tiles - sum + (inc_units - some) * kUnitStartTiles;  // at: what stands before the thread's units
#pragma unroll
        for (int w = 0; w < kAttnWaves; w++) {
            total += s_tmp[w];
            used += s_tmp[kAttnWaves + w];
            at += w < wave ? s_tmp[w] + s_tmp[kAttnWaves + w] * kUnitStartTiles : 0;
        }
        const int even = even_share(total, used);
        const int most = max(least_piece(total), total / max(1, n_blocks - n_units) + 1);
        const bool pieces = most <= even;  // T / most + n_units pieces at most: they fit
        int mine[NU];
#pragma unroll
        for (int i = 0; i < NU; i++) mine[i] = tl[i] + (tl[i] > 0 ? kUnitStartTiles : 0);
        listed = total + used * kUnitStartTiles;
        if (pieces) {  // block-uniform
            int n = 0;
#pragma unroll
            for (int i = 0; i < NU; i++) {
                const int v = (int)threadIdx.x * NU + i;
                mine[i] = v < n_units ? (tl[i] <= kWholeTiles ? 1 : (tl[i] + most - 1) / most) : 0;
                n += mine[i];
            }
            const int inc = wave_incl_scan(n, lane);
            if (lane == 63) s_tmp[2 * kAttnWaves + wave] = inc;
            __syncthreads();
            listed = 0;
            at = inc - n;
#pragma unroll
            for (int w = 0; w < kAttnWaves; w++) {
                listed += s_tmp[2 * kAttnWaves + w];
                at += w < wave ? s_tmp[2 * kAttnWaves + w] : 0;
            }
        }
#pragma unroll
        for (int i = 0; i < NU; i++) {
            const int v = (int)threadIdx.x * NU + i;
            if (v < n_units) s_ts[v] = at;
            at += mine[i];
        }
        if (threadIdx.x == 0) s_ts[n_units] = listed;
        share = __builtin_amdgcn_readfirstlane(pieces ? 0 : even);
        listed = __builtin_amdgcn_readfirstlane(listed);
        __syncthreads();
    }
    auto of_unit = [&](const int *list, int u) __attribute__((always_inline)) { return __builtin_amdgcn_readfirstlane(list[mine_at + u]); };
    auto begin_of = [&](int u) __attribute__((always_inline)) { return of_unit(s_ts, u); };
    auto end_of = [&](int u) __attribute__((always_inline)) { return of_unit(s_ts, u + 1); };
    // even shares: a pair of blocks (even, odd) covers 2 * share tiles, te of them the even block and to the odd one
    const int skew = n_blocks % 2 == 0 ? share * a.skew_permille / 1000 : 0;
    const int te = share + skew, to = share - skew;
    auto block_of = [&](int x) {  // the block whose share holds tile x
        const int pr = x / (2 * share);
        return 2 * pr + (x - pr * 2 * share >= te ? 1 : 0);
    };
    int cur = 0, end = 0;
    if (share > 0) {
        cur = (int)(blockIdx.x / 2) * 2 * share + ((blockIdx.x & 1) ? te : 0);
        end = min(listed, cur + ((blockIdx.x & 1) ? to : te));
        for (int uu = blockIdx.x; uu < n_units; uu += n_blocks)  // units with nothing cached: the output is zero
            if (begin_of(uu) == end_of(uu))
                for (int e = threadIdx.x; e < G * D; e += kAttnThreads) a.out[(size_t)uu * G * D + e] = 0.f;
    }
    // the unit u with s_ts[u] <= first < s_ts[u+1]
    {
        const int first = share > 0 ? cur : (int)blockIdx.x;
        if constexpr (FEW) {  // one comparison per lane; true for lane 0
            u = __builtin_popcountll(__builtin_amdgcn_ballot_w64(lane < n_units && s_ts[mine_at + lane] <= first)) - 1;
        } else {
            int lo = 0, hi = n_units - 1;
            while (lo < hi) {
                const int mid = (lo + hi + 1) >> 1;
                if (begin_of(mid) <= first) lo = mid; else hi = mid - 1;
            }
            u = lo;
        }
    }
    for (bool again = false;; again = true) {  // all conditions are block-uniform
        int np, slot0, slot, p0, p1;  // parts of the unit, the partials' slots, this part's tiles of the unit
        if (share == 0) {
            if (again || (int)blockIdx.x >= listed) break;
            slot0 = begin_of(u);
            slot = blockIdx.x;
            np = end_of(u) - slot0;
        } else {
            if (cur >= end) break;
            while (end_of(u) <= cur) u++;  // also skips units without tiles
            const int first = begin_of(u) + kUnitStartTiles;  // the unit's first real tile
            if (cur < first) {
                cur = first;
                if (cur >= end) break;  // the share ends inside the allowance: the next block begins the unit
            }
            slot0 = block_of(first);
            np = block_of(end_of(u) - 1) - slot0 + 1;
            slot0 += u;
            slot = (int)blockIdx.x + u;
            p0 = cur - first;
            cur = min(end_of(u), end);
            p1 = cur - first;
        }
        const int um = of_unit(s_um, u), gl_all = of_unit(s_gl, u), gl = of_unit(s_gt, u), nloc = of_unit(s_nl, u);
        const int tiles = ceil_tiles(gl) + ceil_tiles(nloc);
        if (share == 0) {  // ascending in the part, and the same for all blocks of the unit
            const float each = (float)tiles * __builtin_amdgcn_rcpf((float)np);
            auto cut = [&](int i) __attribute__((always_inline)) {
                return i == np ? tiles : min(__builtin_amdgcn_readfirstlane((int)((float)i * each)), tiles);
            };
            p0 = cut(slot - slot0);
            p1 = cut(slot - slot0 + 1);
        }
        const int w0 = p0 + (p1 - p0) * wave / kAttnWaves, w1 = p0 + (p1 - p0) * (wave + 1) / kAttnWaves;
        if (again) __syncthreads();  // the states in LDS are rewritten
        DecSoftmax<DT, D, G> st;
        run_part<DT, D, G>(pv, a, u, um, gl_all, gl, nloc, w0, w1, st, s_wave_lds[wave], lane);
        // the waves of the block meet in LDS
        int tid = threadIdx.x;
        asm volatile("" : "+v"(tid));  // (what follows from it is worked out here and not in front of the first row)
        const int x0 = min(tid, NT - 1) * VPT, xg = x0 / D;  // this thread's part of the unit's output
        const bool mine = tid < NT;
        put_states<DT, D, G>(s_st, wave, tid & 63, st);
        __syncthreads();
        float M, L, o[VPT];
        fold_states<OUT::NST, true>(s_st, 0, x0, xg, M, L, o);
        if constexpr (DT != WGKV_F32)
            if (__builtin_expect(any_not_finite(o), 0))
                sum_again<OUT::NST>(u, of_unit(s_um, u), of_unit(s_gl, u), of_unit(s_gt, u), of_unit(s_nl, u), p0, p1, s_st, 0, x0, xg, s_wave_lds[wave],
                                    threadIdx.x & 63, o);
        float *out = a.out + (size_t)u * G * D;
        if (np > 1) {  // block-uniform
            // The stores carry the policy of a device-scope access (written through) and vmcnt counts them until they are
            // acknowledged there: every wave waits for its own, then one thread counts the block; the folding block's loads
            // come after the count.
            const __amdgpu_buffer_rsrc_t r_acc = part_rsrc(a.part_acc, a.part_acc_bytes);
            const __amdgpu_buffer_rsrc_t r_ml = part_rsrc(a.part_ml, a.part_ml_bytes);
            if (mine) put_partial<D, G>(r_ml, r_acc, slot, x0, xg, M, L, o);
            asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
            __syncthreads();
            if (threadIdx.x == 0)
                s_arrived = __hip_atomic_fetch_add(&a.counters[u], 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            __syncthreads();
            if (__builtin_amdgcn_readfirstlane(s_arrived) != np - 1) continue;
            asm volatile("" ::: "memory");
            if (np <= 8) {
                const int xs[1] = {x0};
                float Ls[1], os[1][VPT];
                fold_partials<D, G>(r_ml, r_acc, slot0, np, xs, Ls, os);
                L = Ls[0];
#pragma unroll
                for (int e = 0; e < VPT; e++) o[e] = os[0][e];
            } else {
                fold_partials_block<DT, D, G>(a, slot0, np, s_st, tid, x0, xg, L, o);
            }
            if (threadIdx.x == 0) __hip_atomic_store(&a.counters[u], 0, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        }
        if (mine) {
            const float inv = tiles > 0 ? 1.0f / L : 0.f;
#pragma unroll
            for (int e = 0; e < VPT; e++) out[out_of<DT, D>(x0 + e)] = tiles > 0 ? o[e] * inv : 0.f;
        }
    }
}

// Calls of more units than blocks (batches of 33 and more sequences on eight kv heads): a block has several units one after
// the other, and a chain of round trips (page ids, first rows, fold) for each of them.  Three ways of cutting:
//   solo    a wave takes whole units, and there is no exchange at all: for units of about one length;
//   waves   one list split evenly over the waves, a share may start and end inside a unit (16 tiles at least, and 12 tiles'
//           worth for a unit that begins); a unit's partials, one per wave, are put together by the wave that arrives last:
//           for short units of very different lengths, and for rows of 128 bytes;
//   blocks  the same over blocks, as in the kernel above: for long ones.
// Every block estimates the three in us from the lengths and takes the cheapest.  The model was fitted to the kernel that had all types on the
// vector unit; what it picks was timed against every way of the kernels as they are (558 calls: 33 to 128 sequences of 100 to 8000
// tokens, even and ragged heads, ten head shapes).  Behind the best way, in the mean / at most: main head shape 1.0 / 15 %, the other
// shapes on the matrix cores 0.5 to 1.0 / 15 % (with the factor that eight heads take on the vector unit, 3.1 and 4.6 / 36 %; a fit of all
// constants to these calls 0.5 / 14 %), on the vector unit fp32 0.8 and 1.0 / 26 %, bf16 0.3 to 1.7 / 22 %.  us of blocks / waves / solo, main
// head shape, a third of the tokens admitted: 33 x 100 tokens 15.8 / 17.5 / 10.2, 64 x 300 23.3 / 18.8 / 12.5, 128 x 1000 49.1 / 38.3 /
// 32.7, 33 x 4000 34.4 / 37.0 / 40.5; heads from 1 to 90 %: 64 x 1000 25.1 / 22.7 / 30.8, 128 x 1000 38.6 / 31.3 / 52.4, 33 x 4000
// 26.0 / 29.7 / 95.2 (where it picks waves).
constexpr int kMinWaveTiles = 16, kWaveStartTiles = 12;
template <int DT, int D, int G>
struct DecManyLds {
    DecWaveLds<DT, D, G> wave[kAttnWaves];
    DecStates<DT, D, G> states;
    int ts[kMaxCallUnits + 1];  // tiles before unit u, those charged to the begin of a unit included
    int gl[kMaxCallUnits];      // entries in the unit's global cache
    int um[kMaxCallUnits];      // its index into the per-unit metadata
    int nl[kMaxCallSeqs];       // tokens in the rings of sequence b
    int totals[3][kAttnWaves];  // a wave's tiles, units with any, and tiles of its longest unit
    int arrived;
};
template <int DT, int D, int G>
__device__ __forceinline__ void decode_many(const View &pv, const AttendArgs &a) {
    using SH = DecShape<DT, D, G>;
    using OUT = DecOut<DT, D, G>;
    constexpr int VPT = OUT::VPT, NT = OUT::NT;
    extern __shared__ __attribute__((aligned(1024))) char s_mem[];
    auto &lds = *reinterpret_cast<DecManyLds<DT, D, G> *>(s_mem);
    auto &s_wave_lds = lds.wave;
    auto &s_st = lds.states;
    auto &s_ts = lds.ts;
    auto &s_gl = lds.gl;
    auto &s_um = lds.um;
    auto &s_nl = lds.nl;
    auto &s_wave = lds.totals;
    auto &s_arrived = lds.arrived;

    const int n_units = a.n_seqs * pv.Hkv, n_blocks = (int)gridDim.x, n_waves = n_blocks * kAttnWaves;
    const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    constexpr int NU = kMaxCallUnits / kAttnThreads;  // consecutive units a thread looks after
    int tl[NU], um[NU], len[NU], gl_all[NU], sum = 0, some = 0, longest = 0;
    const float per_seq = __builtin_amdgcn_rcpf((float)pv.Hkv);
    auto seq_of = [&](int u) __attribute__((always_inline)) { return (int)(((float)u + 0.5f) * per_seq); };  // exact: u < 1024
    // What stands in front of the first row is paid by every call: all of a thread's lengths are asked for together, the last unit's
    // again past the end (a branch around each would wait for every one in turn), three sums share one barrier, and what is cut by a
    // few comparisons is not divided.  33 x 100 tokens 11.1 -> 10.2 us, 33 x 1000 22.8 -> 21.5, 64 x 1000 24.2 -> 22.7.
    {
        int u = min((int)threadIdx.x * NU, n_units - 1), b = u / pv.Hkv, h = u - b * pv.Hkv;
#pragma unroll
        for (int i = 0; i < NU; i++) {
            const int sid = a.sid[b];
            um[i] = unit_meta(pv, sid, a.layer, h);
            len[i] = pv.seq_len[sid * pv.L + a.layer];
            gl_all[i] = pv.global_len[um[i]];
            if (++u < n_units && ++h == pv.Hkv) {
                h = 0;
                b++;
            }
        }
    }
#pragma unroll
    for (int i = 0; i < NU; i++) {
        const int u = (int)threadIdx.x * NU + i, nl = min(len[i], pv.W);
        tl[i] = 0;
        if (u < n_units) {
            s_gl[u] = gl_all[i];
            s_um[u] = um[i];
            s_nl[seq_of(u)] = nl;
            tl[i] = ceil_tiles(global_tokens(pv, a, u, gl_all[i])) + ceil_tiles(nl);
        }
        sum += tl[i];
        some += tl[i] > 0 ? 1 : 0;
        longest = max(longest, tl[i]);
    }
    const int inc_tiles = wave_incl_scan(sum, lane), inc_units = wave_incl_scan(some, lane);
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) longest = max(longest, __shfl_xor(longest, o));
    if (lane == 63) {
        s_wave[0][wave] = inc_tiles;
        s_wave[1][wave] = inc_units;
        s_wave[2][wave] = longest;
    }
    __syncthreads();
    int total = 0, used = 0, before_tiles = inc_tiles - sum, before_units = inc_units - some;
#pragma unroll
    for (int w = 0; w < kAttnWaves; w++) {
        before_tiles += w < wave ? s_wave[0][w] : 0;
        before_units += w < wave ? s_wave[1][w] : 0;
        total += s_wave[0][w];
        used += s_wave[1][w];
        longest = max(longest, s_wave[2][w]);
    }
    const int share_b = max(kMinBlockTiles, (total + used * kUnitStartTiles + n_blocks - 1) / n_blocks);
    const int share_w = max(kMinWaveTiles, (total + used * kWaveStartTiles + n_waves - 1) / n_waves);
    constexpr bool kMany8 = G == 8 && !SH::MX;  // the products of eight heads, on the vector unit
    constexpr float kC = (float)SH::ROWB / 256.f * (kMany8 ? 1.6f : 1.f);  // a tile: its bytes, or those products
    const float t_blocks = 8.2f + kC * 0.25f * (float)share_b, t_waves = 3.5f + (SH::ROWB >= 256 ? 1.35f : 1.18f) * kC * (float)share_w;
    // alone a wave streams faster than its share of the memory's rate, until all of them do
    const float full = (float)n_units / (float)n_waves, alone = (kMany8 ? 1.f : 0.68f) * kC * (float)longest;
    const float t_solo = 4.6f + fmaxf(alone * fmaxf(1.f, full), 1.1f + 0.85f * kC * (float)total / (float)n_waves) + 0.3f * alone * full * full;
    const bool solo = t_solo <= fminf(t_blocks, t_waves), by_wave = solo || t_waves <= t_blocks;
    const int begin = solo ? 0 : by_wave ? kWaveStartTiles : kUnitStartTiles, share = by_wave ? share_w : share_b;
    if (!solo) {
        int at = before_tiles + before_units * begin;
#pragma unroll
        for (int i = 0; i < NU; i++) {
            const int u = (int)threadIdx.x * NU + i;
            if (u <= n_units) s_ts[u] = at;  // thread n_units / NU writes the end of the list behind its own units
            at += tl[i] + (tl[i] > 0 ? begin : 0);
        }
        if ((int)threadIdx.x == kAttnThreads - 1 && n_units == kMaxCallUnits) s_ts[kMaxCallUnits] = at;
    }
    __syncthreads();
    // Even shares: the KW workers of an even block and those of the odd one behind it cover 2 * KW * share tiles, te each
    // on the even block and to on the odd one.
    const int KW = by_wave ? kAttnWaves : 1, log2KW = by_wave ? 2 : 0, wid = by_wave ? (int)blockIdx.x * kAttnWaves + wave : (int)blockIdx.x;
    static_assert(kAttnWaves == 4, "a pair of blocks is cut by comparisons");
    const int skew = n_blocks % 2 == 0 ? share * a.skew_permille / 1000 : 0, te = share + skew, to = share - skew, pair = 2 * KW * share;
    auto worker_of = [&](int x) __attribute__((always_inline)) {  // whose share holds tile x
        const int pr = x / pair, r = x - pr * pair, rest = r - KW * te, in = rest < 0 ? r : rest, n = rest < 0 ? te : to;
        return pr * 2 * KW + (rest < 0 ? 0 : KW) + (in >= n) + (in >= 2 * n) + (in >= 3 * n);
    };
    int cur = 0, end = 0, u = 0;
    if (solo) {
        u = wave * n_blocks + (int)blockIdx.x;
    } else {
        const int i = wid & (2 * KW - 1);
        cur = (wid >> (log2KW + 1)) * pair + (i < KW ? i * te : KW * te + (i - KW) * to);
        end = min(s_ts[n_units], cur + (i < KW ? te : to));
        for (int uu = blockIdx.x; uu < n_units; uu += n_blocks)  // units with nothing cached: the output is zero
            if (s_ts[uu + 1] == s_ts[uu])
                for (int e = threadIdx.x; e < G * D; e += kAttnThreads) a.out[(size_t)uu * G * D + e] = 0.f;
        int lo = 0, hi = n_units - 1;  // the unit with s_ts[u] <= cur < s_ts[u + 1]
        while (lo < hi) {
            const int mid = (lo + hi + 1) >> 1;
            if (s_ts[mid] <= cur) lo = mid; else hi = mid - 1;
        }
        u = __builtin_amdgcn_readfirstlane(lo);
    }
    // what a worker has of the unit's output: a thread of a block one part, a wave's lane all of them
    const int part0 = by_wave ? 0 : wave, part1 = by_wave ? (NT + 63) / 64 : wave + 1;
    for (bool again = false;; again = true) {  // all conditions are block-uniform, or wave-uniform where a wave works alone
        int np = 1, slot0 = 0, slot = 0, p0 = 0, p1 = 0;  // parts of the unit, the partials' slots, this part's tiles of the unit
        if (solo) {
            if (again) u += n_waves;
            if (u >= n_units) break;
        } else {
            if (cur >= end) break;
            while (s_ts[u + 1] <= cur) u++;  // also skips units without tiles
            const int first = s_ts[u] + begin;  // the unit's first real tile
            if (cur < first) {
                cur = first;
                if (cur >= end) break;  // the share ends inside the allowance: the next worker begins the unit
            }
            slot0 = worker_of(first);
            np = worker_of(s_ts[u + 1] - 1) - slot0 + 1;
            slot0 += u;
            slot = wid + u;
            p0 = cur - first;
            cur = min(s_ts[u + 1], end);
            p1 = cur - first;
        }
        const int um = s_um[u], gl_all = s_gl[u], nloc = s_nl[seq_of(u)];
        const int gl = global_tokens(pv, a, u, gl_all);
        if (solo) p1 = ceil_tiles(gl) + ceil_tiles(nloc);
        const int w0 = by_wave ? p0 : p0 + (p1 - p0) * wave / kAttnWaves, w1 = by_wave ? p1 : p0 + (p1 - p0) * (wave + 1) / kAttnWaves;
        if (again && !by_wave) __syncthreads();  // the states in LDS are rewritten
        DecSoftmax<DT, D, G> st;
        run_part<DT, D, G>(pv, a, u, um, gl_all, gl, nloc, w0, w1, st, s_wave_lds[wave], lane);
        // the row groups of the block meet in LDS, or those of the wave (whose LDS accesses stay in order)
        __builtin_amdgcn_wave_barrier();
        put_states<DT, D, G>(s_st, wave, lane, st);
        if (by_wave) __builtin_amdgcn_wave_barrier(); else __syncthreads();
        const __amdgpu_buffer_rsrc_t r_acc = part_rsrc(a.part_acc, a.part_acc_bytes);
        const __amdgpu_buffer_rsrc_t r_ml = part_rsrc(a.part_ml, a.part_ml_bytes);
        float *out = a.out + (size_t)u * G * D;
        for (int part = part0; part < part1; part++) {
            const int x = part * 64 + lane, x0 = min(x, NT - 1) * VPT, xg = x0 / D;
            float M, L, o[VPT];
            if (by_wave) fold_states<OUT::NSW, true>(s_st, wave * OUT::NSW, x0, xg, M, L, o);
            else fold_states<OUT::NST, true>(s_st, 0, x0, xg, M, L, o);
            if constexpr (DT != WGKV_F32)
                if (__builtin_expect(any_not_finite(o), 0)) {
                    if (by_wave) sum_again<OUT::NSW>(u, um, gl_all, gl, nloc, p0, p1, s_st, wave * OUT::NSW, x0, xg, s_wave_lds[wave], lane, o);
                    else sum_again<OUT::NST>(u, um, gl_all, gl, nloc, p0, p1, s_st, 0, x0, xg, s_wave_lds[wave], lane, o);
                }
            if (x >= NT) continue;
            if (np > 1) {
                put_partial<D, G>(r_ml, r_acc, slot, x0, xg, M, L, o);
            } else {
                const float inv = p1 > p0 ? 1.0f / L : 0.f;  // nothing cached: zero
#pragma unroll
                for (int e = 0; e < VPT; e++) out[out_of<DT, D>(x0 + e)] = p1 > p0 ? o[e] * inv : 0.f;
            }
        }
        if (np == 1) continue;
        // the hand-over, as above
        asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
        int before = 0;
        if (by_wave) {
            if (lane == 0) before = __hip_atomic_fetch_add(&a.counters[u], 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            before = __builtin_amdgcn_readfirstlane(before);
        } else {
            __syncthreads();
            if (threadIdx.x == 0)
                s_arrived = __hip_atomic_fetch_add(&a.counters[u], 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            __syncthreads();
            before = s_arrived;
        }
        if (before != np - 1) continue;
        asm volatile("" ::: "memory");
        auto fold = [&](auto parts) __attribute__((always_inline)) {
            constexpr int NP = decltype(parts)::value;
            int x0[NP];
            float L[NP], o[NP][VPT];
#pragma unroll
            for (int k = 0; k < NP; k++) x0[k] = min((part0 + k) * 64 + lane, NT - 1) * VPT;
            fold_partials<D, G>(r_ml, r_acc, slot0, np, x0, L, o);
#pragma unroll
            for (int k = 0; k < NP; k++) {
                if ((part0 + k) * 64 + lane >= NT) continue;
                const float inv = 1.0f / L[k];
#pragma unroll
                for (int e = 0; e < VPT; e++) out[out_of<DT, D>(x0[k] + e)] = o[k][e] * inv;
            }
        };
        if (by_wave) fold(std::integral_constant<int, (NT + 63) / 64>{}); else fold(std::integral_constant<int, 1>{});
        if (by_wave ? lane == 0 : threadIdx.x == 0) __hip_atomic_store(&a.counters[u], 0, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    }
}

// The kernels.  On the matrix cores they keep to 256 registers (bounds of two waves per SIMD, though its LDS leaves room for one: that is why it is
// allocated at the launch), where the compiler puts a product's accumulators into vector registers and not into the other half of
// the file, from which it copies them all back in every turn; on the vector unit they need more.
template <int D, int G, bool FEW>
__global__ __launch_bounds__(kAttnThreads, 2) void attend_decode_kernel(View pv, AttendArgs a) { decode_blocks<WGKV_BF16, D, G, FEW>(pv, a); }
template <int D, int G>
__global__ __launch_bounds__(kAttnThreads, 2) void attend_decode_many_kernel(View pv, AttendArgs a) { decode_many<WGKV_BF16, D, G>(pv, a); }
template <int D, int G, bool FEW>
__global__ __launch_bounds__(kAttnThreads) void attend_decode_vec_kernel(View pv, AttendArgs a) { decode_blocks<kBf16Vec, D, G, FEW>(pv, a); }
template <int D, int G>
__global__ __launch_bounds__(kAttnThreads) void attend_decode_many_vec_kernel(View pv, AttendArgs a) { decode_many<kBf16Vec, D, G>(pv, a); }
template <int D, int G, bool FEW>
__global__ __launch_bounds__(kAttnThreads) void attend_decode_f32_kernel(View pv, AttendArgs a) { decode_blocks<WGKV_F32, D, G, FEW>(pv, a); }
template <int D, int G>
__global__ __launch_bounds__(kAttnThreads) void attend_decode_many_f32_kernel(View pv, AttendArgs a) { decode_many<WGKV_F32, D, G>(pv, a); }

// One block per compute unit: an even split is one round of blocks, and more waves on a compute unit stream slower.
template <int DT, int D, int G>
static void launch_one(const View &pv, const AttendArgs &a, int grid, hipStream_t st, hipEvent_t ev0, hipEvent_t ev1) {
    const int n_units = a.n_seqs * pv.Hkv;
    const bool many = n_units > min(grid, kMaxUnits), few = n_units <= 64;
    void (*kernel)(View, AttendArgs);
    unsigned lds;
    auto take = [&](auto dt, void (*k_many)(View, AttendArgs), void (*k_few)(View, AttendArgs), void (*k)(View, AttendArgs)) {
        using Many = DecManyLds<decltype(dt)::value, D, G>;
        using Blocks = DecBlocksLds<decltype(dt)::value, D, G>;
        static_assert(sizeof(Many) <= 160 * 1024 && sizeof(Blocks) <= 160 * 1024, "");
        kernel = many ? k_many : few ? k_few : k;
        lds = many ? sizeof(Many) : sizeof(Blocks);
    };
    // bf16 rows go to the vector unit
    //  - in calls of many units where a key's products with its group fill little of a matrix instruction (of its 16 columns one head's, or two
    //    heads' of 64): us there / on the matrix cores, 33 sequences of 600 tokens with 8 heads of 64 9.7 / 12.5, 64 of 300 with 8 heads of 128
    //    12.7 / 13.9, 40 of 2000 with groups of two of 64 14.6 / 16.8; the next larger, groups of four of 64 or of two of 128, lose 3 to 8 %.
    //    Few units wait for their chains, which are shorter on the matrix cores: 8 of 4096 tokens 9.4 / 8.9 (one of 64) and 9.4 / 8.8 (two),
    //    32 of 20000 18.1 / 18.7 and 19.2 / 18.2;
    //  - where pages are smaller than a tile: their rows are looked up one by one, and a lookup waits for every request of
    //    the wave before it (batch 4 at 20K in pages of 8: 42 / 97).
    if constexpr (DT == WGKV_F32)
        take(std::integral_constant<int, WGKV_F32>{}, attend_decode_many_f32_kernel<D, G>, attend_decode_f32_kernel<D, G, true>, attend_decode_f32_kernel<D, G, false>);
    else if (pv.logP < 4 || (G * D <= 128 && (many || n_units > 16 * G)))
        take(std::integral_constant<int, kBf16Vec>{}, attend_decode_many_vec_kernel<D, G>, attend_decode_vec_kernel<D, G, true>, attend_decode_vec_kernel<D, G, false>);
    else if constexpr (G * D <= 128)
        take(std::integral_constant<int, WGKV_BF16>{}, nullptr, attend_decode_kernel<D, G, true>, nullptr);
    else
        take(std::integral_constant<int, WGKV_BF16>{}, attend_decode_many_kernel<D, G>, attend_decode_kernel<D, G, true>, attend_decode_kernel<D, G, false>);
    if (ev0 && ev1)  // the events take the begin and end time stamps of this dispatch itself
        hipExtLaunchKernelGGL(kernel, dim3(grid), dim3(kAttnThreads), lds, st, ev0, ev1, 0, pv, a);
    else
        hipLaunchKernelGGL(kernel, dim3(grid), dim3(kAttnThreads), lds, st, pv, a);
}
template <int DT, int D>
static hipError_t launch_g(const View &pv, const AttendArgs &a, int grid, hipStream_t st, hipEvent_t ev0, hipEvent_t ev1) {
    switch (pv.G) {
#define WGKV_CASE(GG)                                                                                          \
    case GG: launch_one<DT, D, GG>(pv, a, grid, st, ev0, ev1); break;
        WGKV_CASE(1)
        WGKV_CASE(2)
        WGKV_CASE(4)
        WGKV_CASE(8)
#undef WGKV_CASE
        default: return hipErrorInvalidValue;
    }
    return hipGetLastError();
}

// workspace bytes for a decode attend launched with at most grid_max blocks: a partial per wave (calls of many units) and one
// more per unit, as the slots of two workers on one unit are a unit's number apart
size_t attend_decode_ws_bytes(const View &pv, int n_seqs, int grid_max) {
    const size_t n_units = (size_t)n_seqs * pv.Hkv, slots = (size_t)grid_max * kAttnWaves + n_units;
    size_t b = slots * pv.G * 2 * sizeof(float);
    b = (b + 255) & ~(size_t)255;
    b += slots * pv.G * pv.d * sizeof(float);
    return b;
}

// ---- scratch for callers that bring no workspace ----
// One array per GPU, part of the loaded code object: it exists from the moment the library is
// loaded on a device until the process ends.  In host code the array's name is only a handle
// for hipGetSymbolAddress; the address that kernels and copies use is the one that call returns,
// looked up once per device while that device is current.
static __device__ __align__(256) unsigned char scratch[WGKV_STATIC_SCRATCH_BYTES];
constexpr int kMaxDevices = 64;
static void *g_scratch_ptr[kMaxDevices];  // device address of `scratch` on each device, NULL = not looked up yet

hipError_t static_scratch_init() {
    int dev = -1;
    hipError_t e = hipGetDevice(&dev);
    if (e != hipSuccess) return e;
    if (dev < 0 || dev >= kMaxDevices) return hipErrorInvalidDevice;
    if (g_scratch_ptr[dev]) return hipSuccess;
    void *ptr = nullptr;
    e = hipGetSymbolAddress(&ptr, HIP_SYMBOL(scratch));
    if (e != hipSuccess) return e;
    if (!ptr) return hipErrorInvalidSymbol;
    g_scratch_ptr[dev] = ptr;
    return hipSuccess;
}

// The current device's scratch array, or NULL when static_scratch_init has not run on it.
void *static_scratch() {
    int dev = -1;
    if (hipGetDevice(&dev) != hipSuccess || dev < 0 || dev >= kMaxDevices) return nullptr;
    return g_scratch_ptr[dev];
}

hipError_t launch_attend_decode(const View &pv, int layer, int n_seqs, const int32_t *sids,
                                const void *q, float scale, float *out, void *ws, int32_t *counters,
                                int n_cu, int grid_max, hipStream_t st, hipEvent_t ev0, hipEvent_t ev1,
                                const int32_t *sel_pages, const int32_t *sel_count,
                                int sel_stride, int skew_permille) {
    AttendArgs a;
    a.skew_permille = skew_permille;
    a.sel_pages = sel_pages;
    a.sel_count = sel_count;
    a.sel_stride = sel_stride;
    a.layer = layer;
    a.n_seqs = n_seqs;
    a.scale_log2e = scale * 1.4426950408889634f;
    a.q = (const char *)q;
    a.out = out;
    a.counters = counters;
    // the partial slots are laid out for the largest grid any instantiation may use
    const size_t n_units = (size_t)n_seqs * pv.Hkv, slots = (size_t)grid_max * kAttnWaves + n_units;
    char *w = (char *)ws;
    a.part_ml = (float *)w;
    size_t off = (slots * pv.G * 2 * sizeof(float) + 255) & ~(size_t)255;
    a.part_acc = (float *)(w + off);
    const size_t acc_bytes = slots * pv.G * pv.d * sizeof(float);
    if (acc_bytes > 0x7fffffffu) return hipErrorInvalidValue;  // 32-bit offsets into the partials
    a.part_ml_bytes = (uint32_t)(slots * pv.G * 2 * sizeof(float));
    a.part_acc_bytes = (uint32_t)acc_bytes;
    for (int i = 0; i < n_seqs; i++) a.sid[i] = sids[i];
    const int grid = n_cu < grid_max ? n_cu : grid_max;
    if (pv.dtype == WGKV_BF16 && pv.d == 128) return launch_g<WGKV_BF16, 128>(pv, a, grid, st, ev0, ev1);
    if (pv.dtype == WGKV_BF16 && pv.d == 64) return launch_g<WGKV_BF16, 64>(pv, a, grid, st, ev0, ev1);
    if (pv.dtype == WGKV_F32 && pv.d == 128) return launch_g<WGKV_F32, 128>(pv, a, grid, st, ev0, ev1);
    if (pv.dtype == WGKV_F32 && pv.d == 64) return launch_g<WGKV_F32, 64>(pv, a, grid, st, ev0, ev1);
    return hipErrorInvalidValue;
}

}  // namespace wgkv
