// Budgeted eviction on the global cache (appendix "Eviction policy implementation"):
// remove from every head its floor(frac * N) lowest-scored entries, pack the survivors
// to the front in place, give the emptied pages back.
//
//  evict_compact_kernel   several blocks per (sequence, kv head): radix select of the cut in
//                         the total order of the fp32 bit patterns (equal scores: the
//                         older entry goes first), then in-place compaction of the block's
//                         columns of the K/V rows
//  evict_release_kernel   one block: new lengths, and the emptied pages back on the free stack,
//                         units in (position in the call, kv head) order, a unit's pages in
//                         ascending table index
#include "wgkv_dev.h"

namespace wgkv {

constexpr int kEvictThreads = 1024;
constexpr int kEvictKeep = 8;  // tiles of 1024 entries whose keys stay in registers

struct EvictArgs {
    int layer;
    float frac;
    const float *scores;   // [n_units][stride]
    long long stride;
    int32_t *n_evicted;    // optional [n_units]
    int slices;            // blocks per unit: 1, 2 or 4
};

// Entries a unit loses.  A cache longer than the caller's score row (the host's bound was stale) is left alone.
__device__ __forceinline__ int evict_count(const EvictArgs &a, int N) {
    return N <= a.stride ? (int)floor((double)a.frac * (double)N) : 0;
}

__device__ __forceinline__ uint32_t evict_key(float x) {
    const uint32_t u = __float_as_uint(x);
    return (u & 0x80000000u) ? ~u : (u | 0x80000000u);
}

// The rows of a head are packed in place, so one block has to walk them in order; but the columns of the rows are
// independent, so `slices` blocks walk the same head, each with its own 16-byte columns of K or of V, and each finds
// the cut for itself (18 KB of scores, out of the L2).  A block reads a whole tile of 1024 rows of its columns before it
// writes any of them: eight requests in flight per thread.  (One block per head with one row in flight per thread,
// a barrier and a round trip for every 64 rows, took 103 us for 64 heads of 4.4K entries, 270 MB read and written; this
// form 57, the rate of a plain copy.)
// Nobody changes a length here, which the other blocks of the head may not have read yet: evict_release_kernel does.
__global__ __launch_bounds__(kEvictThreads) void evict_compact_kernel(View pv, CallSeqs cs, EvictArgs a) {
    __shared__ unsigned s_hist[256];
    __shared__ unsigned s_sel[4];      // prefix, mask, remaining rank
    __shared__ int s_tmp[20];
    __shared__ int s_src[kEvictThreads], s_dst[kEvictThreads];
    const int u = (int)blockIdx.x / a.slices, slice = (int)blockIdx.x % a.slices;
    const int b = u / pv.Hkv, h = u % pv.Hkv;
    const int um = unit_meta(pv, cs.sid[b], a.layer, h);
    const int N = pv.global_len[um];
    const int n_e = evict_count(a, N);
    if (threadIdx.x == 0 && slice == 0 && a.n_evicted) a.n_evicted[u] = n_e;
    if (n_e == 0) return;  // block-uniform
    const float *sc = a.scores + (size_t)u * a.stride;
    // the first entries' keys stay in registers, one per thread and tile; longer caches read the rest again
    uint32_t kreg[kEvictKeep];
#pragma unroll
    for (int i = 0; i < kEvictKeep; i++) kreg[i] = evict_key(sc[min(i * kEvictThreads + (int)threadIdx.x, N - 1)]);

    // ---- the n_e-th smallest key: four passes over one byte each, most significant first ----
    if (threadIdx.x == 0) { s_sel[0] = 0u; s_sel[1] = 0u; s_sel[2] = (unsigned)n_e; }
    for (int pass = 3; pass >= 0; pass--) {
        if (threadIdx.x < 256) s_hist[threadIdx.x] = 0u;
        __syncthreads();
        const unsigned prefix = s_sel[0], mask = s_sel[1];
#pragma unroll
        for (int i = 0; i < kEvictKeep; i++)
            if (i * kEvictThreads + (int)threadIdx.x < N && (kreg[i] & mask) == prefix)
                atomicAdd(&s_hist[(kreg[i] >> (8 * pass)) & 255u], 1u);
        for (int j = kEvictKeep * kEvictThreads + threadIdx.x; j < N; j += kEvictThreads) {
            const uint32_t key = evict_key(sc[j]);
            if ((key & mask) == prefix) atomicAdd(&s_hist[(key >> (8 * pass)) & 255u], 1u);
        }
        __syncthreads();
        // the bin in which the running count reaches the rank: a block-wide prefix over the 256 bins
        {
            const unsigned want = s_sel[2];
            const int cnt = threadIdx.x < 256 ? (int)s_hist[threadIdx.x] : 0;
            int total;
            const int ex = block_excl_scan(cnt, s_tmp, &total);
            __syncthreads();  // everybody has read s_sel
            if (threadIdx.x < 256 && (unsigned)ex < want && want <= (unsigned)(ex + cnt)) {
                s_sel[0] = prefix | ((unsigned)threadIdx.x << (8 * pass));
                s_sel[1] = mask | (255u << (8 * pass));
                s_sel[2] = want - (unsigned)ex;  // rank among the keys that share the longer prefix
            }
        }
        __syncthreads();
    }
    const uint32_t cut = s_sel[0];          // key of the last entry to go
    const int ties_to_go = (int)s_sel[2];   // entries with exactly that key that go (the oldest ones)

    // ---- in-place compaction, tiles of 1024 entries in ascending order ----
    // A survivor moves to an index not above its own, and rows are taken in ascending order with all
    // reads of a tile finished before its writes start, so no unread row is overwritten.
    const int cps = (int)(pv.row_bytes / 8) / a.slices;      // 16-byte chunks of this block per row (K and V: 2 rows)
    const int rows_per_turn = kEvictThreads / cps;
    const int my_row = threadIdx.x / cps, col = slice * cps + threadIdx.x % cps, cpr = (int)(pv.row_bytes / 16);
    const size_t col_off = col < cpr ? (size_t)col * 16 : pv.v_off + (size_t)(col - cpr) * 16;
    const int32_t *gpt = pv.global_pt + (size_t)um * pv.maxgp;
    int ties_seen = 0, kept = 0;
    auto compact_tile = [&](int j0, uint32_t key) __attribute__((always_inline)) {
        const int j = j0 + threadIdx.x;
        const int is_tie = (j < N && key == cut) ? 1 : 0;
        int n_ties;
        const int tie_rank = ties_seen + block_excl_scan(is_tie, s_tmp, &n_ties);
        const int stays = (j < N && !(key < cut || (is_tie && tie_rank < ties_to_go))) ? 1 : 0;
        int n_stay;
        const int idx = block_excl_scan(stays, s_tmp, &n_stay);
        __syncthreads();  // the previous tile's copy loop is done with s_src / s_dst
        if (stays) { s_src[idx] = j; s_dst[idx] = kept + idx; }
        __syncthreads();
        // the tile's rows in turns of eight per thread (one turn at 128 bytes a row)
        for (int r0 = 0; r0 < n_stay; r0 += rows_per_turn * 8) {
            const int last = min(r0 + rows_per_turn * 8, n_stay) - 1;
            if (s_src[last] == s_dst[last]) continue;  // nothing before it went: the turn's rows stay where they are (block-uniform)
            uint4 x[8];
            int pg[8];
#pragma unroll
            for (int i = 0; i < 8; i++) pg[i] = gpt[s_src[min(r0 + i * rows_per_turn + my_row, n_stay - 1)] >> pv.logP];
#pragma unroll
            for (int i = 0; i < 8; i++) {
                const int src = s_src[min(r0 + i * rows_per_turn + my_row, n_stay - 1)];
                x[i] = *reinterpret_cast<const uint4 *>(page_ptr(pv, pg[i]) + (size_t)(src & (pv.P - 1)) * pv.row_bytes + col_off);
            }
            // the rows are in registers before anybody writes: naming them here makes the wave wait for them
#pragma unroll
            for (int i = 0; i < 8; i++) asm volatile("" : "+v"(x[i].x), "+v"(x[i].y), "+v"(x[i].z), "+v"(x[i].w));
            __syncthreads();
#pragma unroll
            for (int i = 0; i < 8; i++) {
                const int r = r0 + i * rows_per_turn + my_row;
                if (my_row < rows_per_turn && r < n_stay && s_src[r] != s_dst[r]) {
                    const int dst = s_dst[r];
                    *reinterpret_cast<uint4 *>(page_ptr(pv, gpt[dst >> pv.logP]) + (size_t)(dst & (pv.P - 1)) * pv.row_bytes + col_off) = x[i];
                }
            }
        }
        ties_seen += n_ties;
        kept += n_stay;
    };
#pragma unroll
    for (int i = 0; i < kEvictKeep; i++)
        if (i * kEvictThreads < N) compact_tile(i * kEvictThreads, kreg[i]);  // block-uniform
    for (int j0 = kEvictKeep * kEvictThreads; j0 < N; j0 += kEvictThreads)
        compact_tile(j0, evict_key(sc[min(j0 + (int)threadIdx.x, N - 1)]));
}

// The new lengths, and the table entries behind the last one in use back on the stack: the pages of all units are one
// flat list behind a prefix over the units (one thread per unit walking its pages took 12 us for 64 heads).
__global__ __launch_bounds__(kEvictThreads) void evict_release_kernel(View pv, CallSeqs cs, EvictArgs a, int n_units) {
    __shared__ int s_tmp[20];
    __shared__ int s_base[kMaxCallUnits], s_first[kMaxCallUnits], s_um[kMaxCallUnits];
    const int u = threadIdx.x;
    int n = 0;
    if (u < n_units) {
        const int um = unit_meta(pv, cs.sid[u / pv.Hkv], a.layer, u % pv.Hkv);
        const int N = pv.global_len[um], kept = N - evict_count(a, N);
        const int first = (kept + pv.P - 1) >> pv.logP;
        n = ((N + pv.P - 1) >> pv.logP) - first;
        pv.global_len[um] = kept;
        s_first[u] = first;
        s_um[u] = um;
    }
    int total;
    const int ex = block_excl_scan(n, s_tmp, &total);
    if (u < n_units) s_base[u] = ex;
    __syncthreads();
    const int top = *pv.free_top;
    for (int f = threadIdx.x; f < total; f += kEvictThreads) {
        int lo_u = 0, hi_u = n_units - 1;  // the last unit whose base is <= f (units that give nothing back are never picked)
        while (lo_u < hi_u) {
            const int mid = (lo_u + hi_u + 1) >> 1;
            if (s_base[mid] <= f) lo_u = mid; else hi_u = mid - 1;
        }
        int32_t *e = pv.global_pt + (size_t)s_um[lo_u] * pv.maxgp + s_first[lo_u] + (f - s_base[lo_u]);
        pv.free_stack[top + f] = *e;
        *e = -1;
    }
    __syncthreads();
    if (threadIdx.x == 0) *pv.free_top = top + total;
}

// What the removal asks of the caller's workspace.  Its kernels keep nothing there (the release works out by itself what every
// unit gives back); the bound is part of the entry point and stays, so that what was refused is refused.
size_t evict_ws_bytes(int n_units) { return (size_t)((n_units * 4 + 255) / 256) * 256; }

hipError_t launch_evict_apply(const View &pv, const CallSeqs &cs, int layer, const float *scores,
                              int64_t stride, float frac, int32_t *n_evicted, int64_t max_len, hipStream_t st) {
    const int n_units = cs.n * pv.Hkv;
    if (pv.row_bytes % 128 != 0 || pv.row_bytes / 8 > kEvictThreads) return hipErrorNotSupported;
    EvictArgs a;
    a.layer = layer;
    a.frac = frac;
    a.scores = scores;
    a.stride = stride;
    a.n_evicted = n_evicted;
    // Blocks per head as long as they are one round (a block of 1024 threads fills a compute unit), then one, as every block
    // finds the cut for itself, or two where the rows are what takes the time (max_len: the host's bound of the longest head);
    // 128 bytes a block and row at the least are kept for four.  us for 1 / 2 / 4, 8 heads of 256-byte rows: 8 sequences of 2250
    // entries 54 / 40 / 36, 16 of 300 20 / 18 / 27 and of 2250 58 / 49 / 63, 32 of 300 23 / 31 / 51, 64 of 300 43 / 58 / 95,
    // 40 of 1000 64 / 70 / 83, of 4500 287 / 249 / 258.
    a.slices = n_units <= 64 && pv.row_bytes >= 256 ? 4 : n_units <= 128 || (n_units > 256 && max_len >= 2048) ? 2 : 1;
    hipLaunchKernelGGL(evict_compact_kernel, dim3(n_units * a.slices), dim3(kEvictThreads), 0, st, pv, cs, a);
    hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
    hipLaunchKernelGGL(evict_release_kernel, dim3(1), dim3(kEvictThreads), 0, st, pv, cs, a, n_units);
    return hipGetLastError();
}

}  // namespace wgkv
