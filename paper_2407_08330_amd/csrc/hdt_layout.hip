// hdt_build_layout: per-position level/parent ids -> block-sparse tile schedule, on the device.
//
// What is computed is fixed by the paper (Sec. 3.2: a position attends to parent, siblings and
// children; App. A.1, Alg. 1: sort keys by hierarchy level, partition into blocks, process a block
// only if its mask has a non-zero entry).  How it is computed is ours.  Two kinds of schedule:
//
//  key lists (the default): ONE kernel, key_lists, a workgroup per query tile.  It finds the keys the
//   tile's rows may attend to by scanning level[] / parent[] of the sample once, packs them in key order
//   (by level, ties in document order) into entries of tile_n keys, reserves the tile's slice of the
//   per-entry arrays with one atomic, and evaluates its entries exactly, by key columns (lane masks for
//   the MFMA kernels, pair count, 32x32 sub-block summary).  See the comment at the kernel.
//
//  windowed (Alg. 1 as printed: the key tiles are windows of the globally sorted key order; also the
//  dense baseline): four kernels.
//   sort_count / sort_scatter (one workgroup per 1024 positions)
//    1. key order: stable counting sort by level with wave ballots; the first kernel counts the levels
//       of every chunk, the second turns the counts into each chunk's first slot per level and hands
//       out the slots in document order;
//    2. per anchor, the range of sorted slots its children occupy (integer atomic min/max, one
//       pair of atomics per run of consecutive children);
//   candidates (one wave per query tile)
//    3. every allowed key of a row lies in one of <= 2 slot ranges (its siblings = the children of its
//       parent, and its own children) or is one of 2 single slots (itself, its parent), so a row marks
//       O(1) ranges in a bitmap over the key windows: the candidate windows of the query tile (exact for
//       documents laid out in pre-order, a superset for other forests); the workgroup reserves a slice
//       of the per-entry arrays with one atomic add and writes its candidates there;
//   tile_bitmaps (grid-stride over candidates)
//    4. every candidate is evaluated exactly, pair by pair (lane masks, pair count, sub-block summary,
//       the positions behind its key slots), so the result never depends on step 3 being tight.  A
//       candidate without any allowed pair keeps its list entry with an all-zero summary, which every
//       kernel skips; it is not counted as a tile and hdt_layout_export leaves it out.
//  The same two sort kernels produce the global key order of a key-list layout when hdt_layout_export
//  asks for it.
//
// The per-entry arrays are sized before the number of entries is known (a heuristic, raised by what
// earlier builds needed); the kernels check the capacity.  The kernel that reserves the entries reports
// the count (and whether the hierarchy was valid) through one word of pinned host memory as soon as it
// is known; the host waits for that word only, not for the stream, and repeats the build with the exact
// size in the rare case the guess was too small.
// Device memory comes from a small cache of earlier layouts' buffers.
#include <limits.h>
#include <stdio.h>
#include <string.h>
#include <unistd.h>

#include <algorithm>
#include <chrono>
#include <mutex>
#include <new>
#include <vector>

#include "hdt_internal.h"

namespace {

constexpr int kThreads = 1024;
constexpr int kWaves = kThreads / 64;
constexpr int kBuckets = HDT_MAX_LEVELS + 1;  // levels 0..31, pads in the last bucket
constexpr int kChunk = kThreads;              // positions per workgroup of the two sort kernels

// counters[CNT_ERR]: hierarchy error flag.  counters[CNT_CAND], counters[CNT_CAND + 1]: ONE 64-bit word,
// [39:0] list entries reserved so far, [63:40] workgroups that have reserved theirs: a single returning
// atomic gives a workgroup its slice and tells the last one that it is the last.
enum { CNT_ERR = 0, CNT_CAND = 2 };

// reserves `count` entries; what comes back is looked at with reserved_first and is_last (apart, so that a caller can do
// other work while the atomic is in flight)
__device__ __forceinline__ unsigned long long reserve_entries(int32_t *counters, int count)
{
    // (a lane's own address, as far as the compiler can tell: for a uniform one it adds the lanes up first and hands the
    // result round with readfirstlane, which waits for it on the spot)
    int word = CNT_CAND;
    asm volatile("" : "+v"(word));
    return atomicAdd(reinterpret_cast<unsigned long long *>(counters + word), (1ull << 40) + (unsigned long long)count);
}
__device__ __forceinline__ int reserved_first(unsigned long long old) { return (int)(old & 0xffffffffffull); }
__device__ __forceinline__ bool is_last(unsigned long long old) { return (int)(old >> 40) == (int)gridDim.x - 1; }

// What the candidate kernel reports to the host through pinned host memory: one 64-bit word
// [63:40] ticket of the build, [39] hierarchy error, [31:0] list entries needed.
__host__ __device__ inline unsigned long long report_word(uint32_t ticket, int err, uint32_t need)
{
    return ((unsigned long long)(ticket & 0xffffffu) << 40) | ((unsigned long long)(err != 0) << 39) | need;
}

__device__ __forceinline__ unsigned long long lanemask_lt() { return (1ull << (threadIdx.x & 63)) - 1ull; }

__device__ __forceinline__ int wave_sum(int x)
{
#pragma unroll
    for (int d = 32; d > 0; d >>= 1) x += __shfl_xor(x, d);
    return x;
}

// inclusive sum over the lanes of a wave
__device__ __forceinline__ int wave_scan(int x)
{
#define SCAN_STEP(ctrl, rows) x += __builtin_amdgcn_update_dpp(0, x, ctrl, rows, 0xf, false)
    SCAN_STEP(0x111, 0xf);  // row_shr:1, 2, 4, 8: inside the rows of 16 lanes
    SCAN_STEP(0x112, 0xf);
    SCAN_STEP(0x114, 0xf);
    SCAN_STEP(0x118, 0xf);
    SCAN_STEP(0x142, 0xa);  // row_bcast:15 into rows 1 and 3, row_bcast:31 into rows 2 and 3
    SCAN_STEP(0x143, 0xc);
#undef SCAN_STEP
    return x;
}

__device__ __forceinline__ int bucket_of(int level) { return (level >= 0 && level < HDT_MAX_LEVELS) ? level : kBuckets - 1; }

// histogram of `bucket` over the lanes with `in`: lane k gets the number of lanes that hold bucket k
__device__ __forceinline__ int wave_bucket_count(bool in, int bucket)
{
    const int lane = threadIdx.x & 63;
    int mine = 0;
    unsigned long long remaining = __ballot(in);
    while (remaining) {
        const int leader = __ffsll((long long)remaining) - 1;
        const int bk = __builtin_amdgcn_readlane(bucket, leader);
        const unsigned long long m = __ballot(in && bucket == bk);
        if (lane == bk) mine = __popcll(m);
        remaining &= ~m;
    }
    return mine;
}

// the lanes with `in` that hold this lane's bucket (below 64), from the bits of the buckets: time does not depend on how
// many different ones there are, and bits that all lanes agree on (all but two in a document) cost a ballot
__device__ __forceinline__ unsigned long long wave_bucket_match(bool in, int bucket)
{
    const unsigned long long all = __ballot(in);
    unsigned long long m = all;
#pragma unroll
    for (int bit = 0; bit < 6; bit++) {
        const bool set = (bucket >> bit) & 1;
        const unsigned long long b = __ballot(in && set);
        if (b != 0ull && b != all) m &= set ? b : ~b;
    }
    return m;
}

__device__ __forceinline__ void mark_tiles(uint32_t *bits, int tlo, int thi)
{
    for (int w = tlo >> 5; w <= (thi >> 5); w++) {
        const int lo = max(tlo, w << 5) & 31, hi = min(thi, (w << 5) + 31) & 31;
        const uint32_t m = (hi == 31 ? 0xffffffffu : ((1u << (hi + 1)) - 1u)) & ~((1u << lo) - 1u);
        atomicOr(&bits[w], m);
    }
}

struct SortArgs {
    const int32_t *level, *parent;
    int n, n_slots, nchunks, no_sort;
    int32_t *hist;  // [B][nchunks][kBuckets] positions of every level in every chunk of kChunk positions
    int32_t *kperm, *slot, *cmin, *cmax;
    int32_t *counters;
    int ranges;  // also compute the slot range of every node's children (windowed layouts)
    int32_t *level_copy;  // [B][n] or NULL: the layout's own copy of the level ids
};

// ---- sort, first half: validate, count the levels of each chunk ---------------------------------
__global__ __launch_bounds__(kThreads) void k_sort_count(SortArgs a)
{
    __shared__ int s_cnt[kWaves][kBuckets];
    const int b = blockIdx.x / a.nchunks, chunk = blockIdx.x - b * a.nchunks, n = a.n;
    const int tid = threadIdx.x, wave = tid >> 6, lane = tid & 63;
    const int i = chunk * kChunk + tid;
    const bool in = i < n;
    const size_t o = (size_t)b * n;
    int l = -1, p = -1;
    if (in) {
        l = a.level[o + i];
        p = a.parent[o + i];
        if (a.ranges) {
            a.cmin[o + i] = INT_MAX;
            a.cmax[o + i] = -1;
        }
        if (a.level_copy) a.level_copy[o + i] = l;
    }
    const bool bad = in && (l < -1 || l >= HDT_MAX_LEVELS || p < -1 || p >= n || p == i || (l < 0 && p != -1));
    if (__ballot(bad) && lane == 0) atomicOr(&a.counters[CNT_ERR], 1);
    if (chunk == a.nchunks - 1)
        for (int s = n + tid; s < a.n_slots; s += kThreads) a.kperm[(size_t)b * a.n_slots + s] = -1;
    const int mine = wave_bucket_count(in, bucket_of(l));
    if (lane < kBuckets) s_cnt[wave][lane] = mine;
    __syncthreads();
    if (tid < kBuckets) {
        int t = 0;
#pragma unroll
        for (int w = 0; w < kWaves; w++) t += s_cnt[w][tid];
        a.hist[((size_t)b * a.nchunks + chunk) * kBuckets + tid] = t;
    }
}

// ---- sort, second half: slots in document order; slot range of every node's children ------------
__global__ __launch_bounds__(kThreads) void k_sort_scatter(SortArgs a)
{
    __shared__ int s_cnt[kWaves][kBuckets], s_tot[kWaves][kBuckets], s_pre[kWaves][kBuckets];
    const int b = blockIdx.x / a.nchunks, chunk = blockIdx.x - b * a.nchunks, n = a.n;
    const int tid = threadIdx.x, wave = tid >> 6, lane = tid & 63;
    const int i = chunk * kChunk + tid;
    const bool in = i < n;
    const size_t o = (size_t)b * n;
    int l = -1, p = -1;
    if (in) {
        l = a.level[o + i];
        p = a.parent[o + i];
    }
    // what the parent check below needs, requested before the counting so that its latency hides there
    bool valid = in && l >= 0 && p >= 0 && p < n;
    const int lp = valid ? a.level[o + p] : 0;
    const int bucket = bucket_of(l);
    const int mine = wave_bucket_count(in, bucket);
    // lane k sums level k over the chunks this wave looks at: all of them, and those before this chunk
    int tot = 0, pre = 0;
    if (lane < kBuckets)
        for (int c = wave; c < a.nchunks; c += kWaves) {
            const int v = a.hist[((size_t)b * a.nchunks + c) * kBuckets + lane];
            tot += v;
            if (c < chunk) pre += v;
        }
    if (lane < kBuckets) {
        s_cnt[wave][lane] = mine;
        s_tot[wave][lane] = tot;
        s_pre[wave][lane] = pre;
    }
    __syncthreads();
    if (wave == 0) {  // first slot of every (level, wave of this chunk): level major, then chunk, then wave
        int t = 0, pr = 0;
        if (lane < kBuckets) {
#pragma unroll
            for (int w = 0; w < kWaves; w++) {
                t += s_tot[w][lane];
                pr += s_pre[w][lane];
            }
        }
        int incl = t;  // inclusive scan of the level totals over lanes
#pragma unroll
        for (int d = 1; d < 64; d <<= 1) {
            const int y = __shfl_up(incl, d);
            if (lane >= d) incl += y;
        }
        int run = incl - t + pr;
        if (lane < kBuckets) {
#pragma unroll
            for (int w = 0; w < kWaves; w++) {
                const int c = s_cnt[w][lane];
                s_cnt[w][lane] = run;
                run += c;
            }
        }
    }
    __syncthreads();
    const int mybase = lane < kBuckets ? s_cnt[wave][lane] : 0;
    int my_slot = i;
    {
        unsigned long long remaining = __ballot(in);
        while (remaining) {
            const int leader = __ffsll((long long)remaining) - 1;
            const int bk = __builtin_amdgcn_readlane(bucket, leader);
            const bool is_bk = in && bucket == bk;
            const unsigned long long m = __ballot(is_bk);
            const int first = __builtin_amdgcn_readlane(mybase, bk);
            if (is_bk) my_slot = first + __popcll(m & lanemask_lt());
            remaining &= ~m;
        }
    }
    if (a.no_sort) my_slot = i;
    if (in) {
        a.kperm[(size_t)b * a.n_slots + my_slot] = i;
    }
    if (!a.ranges) {
        if (valid && lp < 0) atomicOr(&a.counters[CNT_ERR], 1);  // a parent must be a real position
        return;
    }
    if (in) a.slot[o + i] = my_slot;
    // Slot range of every node's children.  Consecutive positions with the same parent and consecutive
    // slots (the tokens of a sentence, for one) form a run whose minimum and maximum are its first and
    // last slot: one atomic each per run.
    if (valid && lp < 0) {  // a parent must be a real position
        atomicOr(&a.counters[CNT_ERR], 1);
        valid = false;
    }
    const int sl = valid ? my_slot : -1;
    const int p_prev = __shfl_up(p, 1), s_prev = __shfl_up(sl, 1);
    const bool v_prev = __shfl_up((int)valid, 1) != 0;
    const bool head = lane == 0 || !v_prev || p_prev != p || s_prev + 1 != sl;
    const bool next_head = __shfl_down((int)(head || !valid), 1) != 0;  // lane+1 starts a new run (or is invalid)
    const bool tail = lane == 63 || next_head;
    if (valid && head) atomicMin(&a.cmin[o + p], sl);
    if (valid && tail) atomicMax(&a.cmax[o + p], sl);
}

struct CandArgs {
    const int32_t *level, *parent, *slot, *cmin, *cmax;
    int n, bm, bn, tr, tc, wc, force_dense, edges;
    int64_t capacity;
    int32_t *q_range;  // [B][tr][2]: first and one-past-last list entry of every query tile
    int32_t *c_row, *q_cols;
    int32_t *counters;
    unsigned long long *report;  // pinned host memory, written once by the last workgroup to get there
    uint32_t ticket;
};

// ---- candidate key tiles of every query tile: one wave per query tile, a bitmap per wave in LDS ----
__global__ __launch_bounds__(kThreads) void k_candidates(CandArgs a)
{
    extern __shared__ uint32_t s_bitmaps[];  // [kWaves][wc]
    __shared__ int s_n[kWaves];
    __shared__ int s_base;
    const int groups = (a.tr + kWaves - 1) / kWaves;
    const int b = blockIdx.x / groups, g = blockIdx.x - b * groups, n = a.n;
    const int tid = threadIdx.x, wave = tid >> 6, lane = tid & 63;
    const int bm = a.bm, bn = a.bn, tr = a.tr, tc = a.tc, wc = a.wc;
    const int I = g * kWaves + wave;
    const bool active = I < tr;
    const int32_t *level = a.level + (size_t)b * n, *parent = a.parent + (size_t)b * n;
    const int32_t *slot = a.slot + (size_t)b * n, *cmin = a.cmin + (size_t)b * n, *cmax = a.cmax + (size_t)b * n;
    uint32_t *wbits = s_bitmaps + (size_t)wave * wc;
    for (int w = lane; w < wc; w += 64) wbits[w] = 0;
    __builtin_amdgcn_wave_barrier();
    if (active && a.force_dense) {
        if (lane == 0) mark_tiles(wbits, 0, tc - 1);
    } else if (active) {
        // rows lane and lane + 64 of the tile; all loads of one dependency level are issued together
        int i2[2], sl2[2], p2[2], lo_c[2], hi_c[2];
        bool ok[2];
#pragma unroll
        for (int u = 0; u < 2; u++) {
            const int rr = lane + 64 * u;
            i2[u] = I * bm + rr;
            ok[u] = rr < bm && i2[u] < n;
            const int ii = ok[u] ? i2[u] : 0;
            ok[u] = ok[u] && level[ii] >= 0;
            sl2[u] = slot[ii];
            p2[u] = parent[ii];
            lo_c[u] = cmin[ii];
            hi_c[u] = cmax[ii];
        }
        int sp2[2], lo_s[2], hi_s[2];
        bool okp[2];
#pragma unroll
        for (int u = 0; u < 2; u++) {
            okp[u] = ok[u] && p2[u] >= 0 && p2[u] < n;
            const int pp = okp[u] ? p2[u] : 0;
            okp[u] = okp[u] && level[pp] >= 0;
            sp2[u] = slot[pp];
            lo_s[u] = cmin[pp];
            hi_s[u] = cmax[pp];
        }
#pragma unroll
        for (int u = 0; u < 2; u++) {
            if (!ok[u]) continue;
            mark_tiles(wbits, sl2[u] / bn, sl2[u] / bn);  // itself
            if (okp[u]) {
                if (a.edges & HDT_EDGE_UP) mark_tiles(wbits, sp2[u] / bn, sp2[u] / bn);  // its parent
                if ((a.edges & HDT_EDGE_SIBLING) && lo_s[u] <= hi_s[u] && lo_s[u] >= 0 && hi_s[u] < n)
                    mark_tiles(wbits, lo_s[u] / bn, hi_s[u] / bn);  // its siblings: the children of its parent
            }
            if ((a.edges & HDT_EDGE_DOWN) && lo_c[u] <= hi_c[u] && lo_c[u] >= 0 && hi_c[u] < n)
                mark_tiles(wbits, lo_c[u] / bn, hi_c[u] / bn);  // its children
        }
    }
    __builtin_amdgcn_wave_barrier();
    int cnt = 0;
    for (int w = lane; w < wc; w += 64) cnt += __popc(wbits[w]);
    cnt = wave_sum(cnt);
    if (lane == 0) s_n[wave] = cnt;
    __syncthreads();
    if (tid == 0) {
        int total = 0;
#pragma unroll
        for (int w = 0; w < kWaves; w++) total += s_n[w];
        // this workgroup's slice of the list arrays
        // this workgroup's slice of the list arrays; the last workgroup to get here knows the final count
        // and tells the host, which is waiting for exactly this word, while the lists and the bitmaps are
        // still being written (no device-scope fence: it would write back the whole L2 of this XCD)
        const unsigned long long old = reserve_entries(a.counters, total);
        s_base = reserved_first(old);
        if (is_last(old)) {
            const int err = __hip_atomic_load(&a.counters[CNT_ERR], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            __hip_atomic_store(a.report, report_word(a.ticket, err, (uint32_t)(reserved_first(old) + total)), __ATOMIC_RELEASE,
                               __HIP_MEMORY_SCOPE_SYSTEM);
        }
    }
    __syncthreads();
    if (!active) return;
    int cbase = s_base;
    for (int w = 0; w < wave; w++) cbase += s_n[w];
    const size_t row = (size_t)b * tr + I;
    if (lane == 0) {
        a.q_range[2 * row] = cbase;
        a.q_range[2 * row + 1] = cbase + cnt;
    }
    int n_cand = 0;
    for (int w0 = 0; w0 < wc; w0 += 2) {
        const int w = w0 + (lane >> 5), bit = lane & 31;
        const uint32_t word = w < wc ? wbits[w] : 0u;
        const bool is_cand = (word >> bit) & 1u;
        const unsigned long long cm = __ballot(is_cand);
        const int64_t c = (int64_t)cbase + n_cand + __popcll(cm & lanemask_lt());
        if (is_cand && c < a.capacity) {
            a.c_row[c] = (int32_t)row;
            a.q_cols[c] = (w << 5) + bit;
        }
        n_cand += __popcll(cm);
    }
}

// ---- exact evaluation of one list entry pair by pair, by two waves (windowed layouts) ---------------
// Wave `wsub` (0 or 1) holds rows 64*wsub + lane of the query tile (position i, parent pi, rowok = a
// real position) and evaluates them against all keys (khalf < 0) or against one half of the entry's
// 32-key words (khalf = 0, 1); every wave holds the entry's keys, lane l the slots l and 64 + l (position
// and parent, -1 where the slot holds no key), which are broadcast by lane index while each lane tests
// its row against every key.  Outputs of entry c: per 32x32 sub-block the 16 x 64-bit lane masks the
// MFMA kernels apply to their accumulator registers (wave ballots), and through `part` (this wave's slot
// of a pair's scratch in LDS) the pair count and the sub-block summary, which the caller adds up after
// a barrier.
struct EntryPart {
    int cnt;
    uint32_t any, all;
    uint32_t col[4];  // entry_bitmaps only: key slots (32 per word) that some row of this wave may attend to
};

__device__ __forceinline__ uint32_t wave_or(uint32_t x)
{
#pragma unroll
    for (int d = 32; d > 0; d >>= 1) x |= (uint32_t)__shfl_xor((int)x, d);
    return x;
}

__device__ __forceinline__ EntryPart entry_bitmaps(bool active, int64_t c, int wsub, int khalf, int lane, int i, int pi,
                                                   bool rowok,
                                                   const int (&kpos)[2], const int (&kpar)[2], int bm, int bn, int edges,
                                                   unsigned long long *bits_rm)
{
    const int wpr = bn >> 5, nrb = bm >> 5, nsub = nrb * wpr;
    // a disabled edge kind is a comparison against a value no key carries
    const int pi_sib = (edges & HDT_EDGE_SIBLING) && pi >= 0 ? pi : -3;  // my parent, for "same parent"
    const int pi_up = (edges & HDT_EDGE_UP) ? pi : -3;                   // my parent, for "is my parent"
    const int i_down = (edges & HDT_EDGE_DOWN) ? i : -3;                 // me, for "is my child"
    uint32_t w[4] = {0u, 0u, 0u, 0u};
    int cnt = 0;
#pragma unroll
    for (int wd = 0; wd < 4; wd++) {
        if (wd < wpr && (khalf < 0 || (wd * 2) / wpr == khalf)) {
            const int kp = kpos[wd >> 1], kq = kpar[wd >> 1];
            uint32_t out = 0;
#pragma unroll 8
            for (int cc = 0; cc < 32; cc++) {
                const int kj = __builtin_amdgcn_readlane(kp, (wd & 1) * 32 + cc);
                const int kr = __builtin_amdgcn_readlane(kq, (wd & 1) * 32 + cc);
                const bool ok = kj >= 0 && (kj == i || pi_sib == kr || pi_up == kj || kr == i_down);
                out |= (uint32_t)ok << cc;
            }
            w[wd] = rowok ? out : 0u;
            cnt += __popc(w[wd]);
        }
    }
    EntryPart part;
    part.cnt = wave_sum(cnt);
    part.any = part.all = 0;
#pragma unroll
    for (int wd = 0; wd < 4; wd++) part.col[wd] = wave_or(w[wd]);
    // register-major masks of sub-block (rblk, cblk), accumulator register e: bit l <=> row
    // rblk*32 + l%32, column cblk*32 + (l/32)*4 + 8*(e/4) + e%4
#pragma unroll
    for (int rr = 0; rr < 2; rr++) {
        const int rblk = 2 * wsub + rr;
        if (rblk < nrb) {
#pragma unroll
            for (int cblk = 0; cblk < 4; cblk++) {
                if (cblk < wpr && (khalf < 0 || (cblk * 2) / wpr == khalf)) {
                    const uint32_t x = (uint32_t)__shfl((int)w[cblk], rr * 32 + (lane & 31));
                    unsigned long long mine = 0;
#pragma unroll
                    for (int e = 0; e < 16; e++) {
                        const int bit = (lane >> 5) * 4 + 8 * (e >> 2) + (e & 3);
                        const unsigned long long m = __ballot((x >> bit) & 1u);
                        if (lane == e) mine = m;
                    }
                    const int sb = rblk * wpr + cblk;
                    if (active && lane < 16) bits_rm[((size_t)c * nsub + sb) * 16 + lane] = mine;
                    if (__ballot(x != 0u) != 0ull) part.any |= 1u << sb;
                    if (__ballot(x == 0xffffffffu) == ~0ull) part.all |= 1u << sb;
                }
            }
        }
    }
    return part;
}

// ---- bitmaps of a list entry by columns, one wave per 64 key slots ----------------------------------
// Lane c stands for key slot k0 + c and builds that key's COLUMN of the tile: bit r%32 of col[r/32] <=> row r
// may attend to it.  Rows see a key through their own parent in two ways - the key is that parent, or the
// key has the same parent - so for both the rows are R(v) = {rows whose parent is v}, with v the key's
// position or the key's parent; R is tabulated once per tile, in a hash table over the distinct parents of its
// rows.  (A handful in a document, since the tokens of a sentence share theirs, dozens in a tree or among shuffled
// positions: a list of them that one wave makes, one by one, and every key is compared with was the longest phase of
// such builds.  Event-bracketed us, with such a list and a sort that takes the levels one by one - as it is: 16
// ListOps-shaped trees of 1536 positions, 64 x 32 tiles, 16.2 - 10.7, 128 x 64 19.4 - 10.4, both schedules of a directed mask
// 17.2 - 11.8 and 20.5 - 11.2; documents of 1000 positions 10.2 - 9.7, of 8192 the same; lists of 500 keys of two or three
// parents, 64 x 32 tiles, 4 samples of 4500 11.1 - 11.5, of 16384 28.0 - 28.7.)  The key itself and the key's own parent
// are single rows.  The lane masks of the MFMA kernels need no transposition from there: mask e of sub-block
// (rblk, cblk) is the column word of key 32*cblk + 8*(e/4) + e%4 (lanes 0..31) next to that of key
// 32*cblk + 4 + 8*(e/4) + e%4 (lanes 32..63), so every lane stores its own words.
struct ParentTable {
    static constexpr int kSlots = 256;  // of a workgroup's tiles together, twice the rows they can have
    int slots;                          // of this tile, a power of two
    int *v;                             // [slots] a parent, or -1
    uint4 *rows;                        // [slots] the rows with that parent, 32 per word
    __device__ __forceinline__ int home(int p) const { return (int)(((uint32_t)p * 0x9e3779b1u) >> 16) & (slots - 1); }
    // row r has parent p.  (At most half of the slots are ever taken, so a search ends.)
    __device__ __forceinline__ void add(int p, int r) const
    {
        int at = home(p);
        for (;;) {
            const int old = atomicCAS(&v[at], -1, p);
            if (old == -1 || old == p) break;
            at = (at + 1) & (slots - 1);
        }
        atomicOr(reinterpret_cast<uint32_t *>(&rows[at]) + (r >> 5), 1u << (r & 31));
    }
    // the slot of p, -1 if there is none (p < 0: none)
    __device__ __forceinline__ int find(int p) const
    {
        int at = home(p), x = p < 0 ? -1 : v[at];
        while (x != p && x != -1) {
            at = (at + 1) & (slots - 1);
            x = v[at];
        }
        return x == -1 ? -1 : at;
    }
};

__device__ __forceinline__ EntryPart entry_columns(int64_t c, int k0, int lane, const ParentTable &tab, const int *ek,
                                                   const int *ep, int row0, int bm, int bn, int edges,
                                                   unsigned long long *bits_rm)
{
    const int wpr = bn >> 5, nrb = bm >> 5, nsub = nrb * wpr;
    const int k = k0 + lane;
    const bool slot = k < bn;
    const int kj = slot ? ek[k] : -1, kr = slot ? ep[k] : -1;  // -1: no key
    const int v_up = (edges & HDT_EDGE_UP) ? kj : -1, v_sib = (edges & HDT_EDGE_SIBLING) ? kr : -1;
    uint32_t col[4] = {0u, 0u, 0u, 0u};
    const int at_up = tab.find(v_up), at_sib = tab.find(v_sib);
    if (at_up >= 0) {
        const uint4 r = tab.rows[at_up];
        col[0] = r.x, col[1] = r.y, col[2] = r.z, col[3] = r.w;
    }
    if (at_sib >= 0) {
        const uint4 r = tab.rows[at_sib];
        col[0] |= r.x, col[1] |= r.y, col[2] |= r.z, col[3] |= r.w;
    }
    // the key itself; the key's parent (the key is that row's child).  A key or a key's parent inside the
    // tile's range is a real position, hence a valid row.
    const int r_self = kj - row0, r_down = (edges & HDT_EDGE_DOWN) ? kr - row0 : -1;
    const bool has_self = kj >= 0 && r_self >= 0 && r_self < bm, has_down = kr >= 0 && r_down >= 0 && r_down < bm;
#pragma unroll
    for (int w = 0; w < 4; w++) {
        if (has_self && (r_self >> 5) == w) col[w] |= 1u << (r_self & 31);
        if (has_down && (r_down >> 5) == w) col[w] |= 1u << (r_down & 31);
    }
    EntryPart part;
    part.cnt = __builtin_amdgcn_readlane(wave_scan(__popc(col[0]) + __popc(col[1]) + __popc(col[2]) + __popc(col[3])), 63);
    part.any = part.all = 0;
    const int cblk = k >> 5, cc = k & 31, e = ((cc >> 3) << 2) | (cc & 3), hf = (cc >> 2) & 1;
    uint32_t *rm32 = reinterpret_cast<uint32_t *>(bits_rm + (size_t)c * nsub * 16);
#pragma unroll
    for (int rblk = 0; rblk < 4; rblk++) {
        if (rblk >= nrb) break;
        if (slot) rm32[((size_t)(rblk * wpr + cblk) * 16 + e) * 2 + hf] = col[rblk];
        const unsigned long long any = __ballot(col[rblk] != 0u), all = __ballot(col[rblk] == 0xffffffffu);
        const int sb = rblk * wpr + (k0 >> 5);  // lanes 0..31: sub-block sb, lanes 32..63: sb + 1
        if ((uint32_t)any) part.any |= 1u << sb;
        if ((uint32_t)(any >> 32)) part.any |= 2u << sb;
        if ((uint32_t)all == 0xffffffffu) part.all |= 1u << sb;
        if ((uint32_t)(all >> 32) == 0xffffffffu) part.all |= 2u << sb;
    }
    return part;
}

struct KeyListArgs {
    const int32_t *level, *parent;
    int n, bm, bn, tr, no_sort, edges;
    int64_t capacity;
    int32_t *q_range;  // [B][tr][2]
    int32_t *c_row, *q_keys, *q_kpar, *c_cnt;
    int32_t *level_copy, *parent_copy;  // the layout's own copy of the ids (the key order is sorted from it on demand)
    uint32_t *q_sub;
    unsigned long long *bits_rm;
    int32_t *counters;
    unsigned long long *report;      // pinned host memory
    unsigned long long *report_dev;  // the layout's own copy of the report
    uint32_t ticket;
    int self_reset;  // the counters are a slot that must be zero again when the build has reported
    int host_waits;  // the host is waiting for the report
};

struct KeyListLaunch {
    KeyListArgs args[2];
};

// Workgroup barrier for data exchanged through LDS only: unlike __syncthreads() it does not wait for this
// wave's global loads and stores (a store to HBM takes 2-3 us to be acknowledged).
__device__ __forceinline__ void lds_barrier() { asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory"); }

// Sets the hierarchy error flag and waits for it to be set (a returning atomic): what this thread does next,
// a barrier in front of the workgroup's reservation, is then ordered behind it for the workgroup that reads
// the flag after the last reservation.
__device__ __forceinline__ void raise_error(int32_t *counters)
{
    const int old = atomicOr(&counters[CNT_ERR], 1);
    asm volatile("" ::"v"(old));
}

constexpr int kBatch = 8;
constexpr int kLdsKeys = 2048;  // key lists up to this length stay in LDS between the packing and the bitmaps

// ---- key lists: ONE kernel from level/parent to the finished entries -------------------------------------
// A workgroup makes the lists of T neighbouring query tiles (T = 2: tiles of up to 64 rows, which share one scan of
// the sample's ids; T = 1: tiles of up to 128 rows, and documents whose bitmaps do not fit the LDS twice).
// Key j is needed by a tile iff it is one of the tile's rows, the parent of one, a child of one (its parent is a row of the
// tile) or a sibling of one (its parent is the parent of a row) - each kind only if its edges are enabled.  Two
// bitmaps over the positions, in LDS, say so exactly for any forest: `keys`, the positions that are needed by themselves
// (rows, and parents of rows), and `pars`, those whose children are (the same two kinds).  The workgroup scans level[] and
// parent[] of the whole sample once (two coalesced streams, nothing waits on a chain of dependent loads): for 64
// positions the first kind is a word of `keys` as it stands, the second one look-up per lane; the result replaces that
// word.  The needed keys are then packed in KEY ORDER - by level, ties in document order, i.e. the order of kperm
// restricted to the needed keys - in two steps: into LDS in document order (a prefix sum over the bitmap), and from there
// by a counting sort over the levels of the needed keys alone, 64 of them per wave.  The global key order is therefore
// not an input of this kernel.
// What bounds it is the chain of these phases in one workgroup (a compute unit has one or two) and, in the scan, the
// instructions per position.  The groups of 64 positions go round the waves: the keys a tile needs lie close together, and
// with a contiguous share of the document per wave one or two waves had all of the packing to do.  Event-bracketed, with
// level counts taken in the scan, bitmap tests of every kind per position and contiguous shares before: 8192 positions x 4
// samples, 64 x 32 tiles: 19.6 -> 13.5 us; 128 x 64: 17.6 -> 12.5; 32768 positions, 64 x 32: 43.2 -> 21.0.
// Then the workgroup evaluates its own entries by key columns (entry_columns: lane masks, pair counts, summaries), one
// wave per 64 key slots, the entries of both tiles in one sequence.  It also validates its own rows.
// The lists are in LDS by the time the reservation of their entries (a returning device-scope atomic, about 2 us) is
// back, unless the host waits for the build: then it is waited for first (see there).  Lists beyond kLdsKeys keys in all are packed straight into global memory instead, with a contiguous share of
// the document per wave, and read again from there.
// 512 threads for documents whose scan is a single batch of their 8 waves, 4096 positions: a barrier is shorter, and two or
// three workgroups share a compute unit where one of 1024 fills it.  Event-bracketed us, 1024 - 512 threads: sections,
// 64 x 32 tiles, 1 sample of 1000 positions 11.8 - 11.0, 16 of 1536 12.3 - 11.6, 8 of 4096 13.0 - 12.4, 32 of 2048 20.7 - 15.8;
// 128 x 64 the same or a little more; two schedules of ListOps-shaped trees, 16 of 1536, 21.5 - 17.2 (before the parents were
// hashed, all of them); but 4 of 8192 13.1 - 15.5, 1 of 32768 20.8 - 23.8.  (256: 12.5, 13.1, 17.1 and 16.6 in the first
// four.)  Longer documents get 1024, with T = 1 and tiles of up to 64 rows, which make twice the workgroups, 512.
__host__ __device__ inline int list_words(int n) { return (((n + 31) >> 5) + 4) & ~3; }  // of `pars`, per tile: a zero word behind
__host__ inline size_t list_lds(int n, int tiles)
{
    return (size_t)tiles * ((size_t)list_words(n) + 2 * (size_t)((n + 63) >> 6)) * sizeof(uint32_t);
}

template <int kListThreads, int T>
__device__ __forceinline__ void key_lists(const KeyListArgs &a)
{
    constexpr int W = kListThreads / 64, RT = 128 / T;
    constexpr int kItemGroups = kLdsKeys / 64 + T, kRounds = (kItemGroups + W - 1) / W;  // groups of 64 packed keys
    static_assert(W <= kItemGroups, "the level counts of the waves share the array of the item groups");
    // pars: word w of tile h at [w * T + h]; after the scan its place holds the number of needed keys in front of every
    // group of 64 positions (16 bits, group g of tile h at [g * T + h]).  keys: the same order, so that the words of all
    // tiles for 64 positions are 8 T consecutive bytes.
    extern __shared__ __attribute__((aligned(16))) uint32_t s_dyn[];
    __shared__ int s_lcnt[kItemGroups][kBuckets];  // keys per (group of 64 packed keys, level)
    __shared__ int s_cnt[2][W];          // partial results of an entry's two waves (tile_n > 64), by parity of the round
    __shared__ uint32_t s_any[2][W], s_all[2][W];
    __shared__ int s_base, s_wtotal[T][W], s_total[T];
    __shared__ __attribute__((aligned(16))) int s_keys[kLdsKeys], s_kpar[kLdsKeys];
    __shared__ int s_tab_v[ParentTable::kSlots];  // the tiles' parent tables
    __shared__ uint4 s_tab_rows[ParentTable::kSlots];
    __shared__ int s_first[T];               // first real row of a tile (a position), INT_MAX if it has none
    const int per_sample = (a.tr + T - 1) / T;
    const int b = blockIdx.x / per_sample, I0 = (blockIdx.x - b * per_sample) * T, n = a.n;
    const int tid = threadIdx.x, wave = __builtin_amdgcn_readfirstlane(tid >> 6), lane = tid & 63;
    const int bm = a.bm, bn = a.bn;
    const int32_t *level = a.level + (size_t)b * n, *parent = a.parent + (size_t)b * n;
    const int pw = list_words(n), ng = (n + 63) >> 6;
    uint32_t *s_pars = s_dyn, *s_need = s_dyn + T * pw;
    uint16_t *s_before = reinterpret_cast<uint16_t *>(s_dyn);
    struct Words { uint32_t w[2 * T]; };  // of 64 positions: [half * T + h]
    auto words = [&](int g) { return reinterpret_cast<Words *>(s_need) + g; };
    int row0[T];
#pragma unroll
    for (int h = 0; h < T; h++) row0[h] = (I0 + h) * bm;
    const bool e_up = a.edges & HDT_EDGE_UP, e_sib = a.edges & HDT_EDGE_SIBLING, e_down = a.edges & HDT_EDGE_DOWN;
    // kBatch groups of 64 positions per wave at a time: all their loads are issued before the first is used, and those
    // of the next batch before this one is looked at
    const int rounds = (ng + W - 1) / W;  // group u * W + wave is this wave's u-th
    int klv[kBatch], kp[kBatch];
    auto load_batch = [&](int u0, int (&l)[kBatch], int (&p)[kBatch]) {
#pragma unroll
        for (int u = 0; u < kBatch; u++) {
            const int j = ((u0 + u) * W + wave) * 64 + lane;
            const bool ok = j < n;
            l[u] = ok ? level[j] : -1;
            p[u] = ok ? parent[j] : -1;
        }
    };
    // the rows' ids first: they are looked at first
    int my_level = -1, my_parent = -1;
    const int my_tile = tid / RT, my_row = (I0 + my_tile) * bm + tid % RT;  // of the first 128 threads
    const bool have_row = tid < 128 && tid % RT < bm && I0 + my_tile < a.tr && my_row < n;
    if (have_row) {
        my_level = level[my_row];
        my_parent = parent[my_row];
    }
    load_batch(0, klv, kp);
    for (int w = tid; w < T * (pw + 2 * ng); w += kListThreads) s_dyn[w] = 0u;
    if (tid < ParentTable::kSlots) {
        s_tab_v[tid] = -1;
        s_tab_rows[tid] = make_uint4(0u, 0u, 0u, 0u);
    }
    ParentTable tab[T];
#pragma unroll
    for (int h = 0; h < T; h++) {
        tab[h].slots = ParentTable::kSlots / T;
        tab[h].v = s_tab_v + h * (ParentTable::kSlots / T);
        tab[h].rows = s_tab_rows + h * (ParentTable::kSlots / T);
    }
    if (tid < T) s_first[tid] = INT_MAX;
    lds_barrier();
    bool check_parent = false;
    if (tid < 128) {
        const int p = my_parent;
        if (have_row && (my_level < -1 || my_level >= HDT_MAX_LEVELS || p < -1 || p >= n || p == my_row || (my_level < 0 && p != -1))) {
            raise_error(a.counters);
            my_level = -1;
        }
        const bool real = have_row && my_level >= 0;
        // this wave's rows: two words of the bitmaps
        const unsigned long long rows = __ballot(real);
        if (lane < 2 && rows) {
            const uint32_t word = (uint32_t)(rows >> (32 * lane));
            const int at = (((my_row - lane) >> 5) + lane) * T + my_tile;
            if (word) atomicOr(&s_need[at], word);
            if (word && e_down) atomicOr(&s_pars[at], word);
            if (lane == 0) atomicMin(&s_first[my_tile], my_row + __ffsll((long long)rows) - 1);
        }
        if (real && p >= 0) {
            (my_tile ? tab[T - 1] : tab[0]).add(p, tid % RT);
            if (e_sib) atomicOr(&s_pars[(p >> 5) * T + my_tile], 1u << (p & 31));
            if (e_up) atomicOr(&s_need[(p >> 5) * T + my_tile], 1u << (p & 31));
            check_parent = true;
        }
    }
    const int parent_level = check_parent ? level[my_parent] : 0;  // looked at once the scan is under way
    lds_barrier();
    const bool one_batch = rounds <= kBatch;
    Words need{};  // lane u: the needed positions of the last batch's group u
    int wtotal[T];  // needed keys in this lane's groups
#pragma unroll
    for (int h = 0; h < T; h++) wtotal[h] = 0;
    for (int u0 = 0; u0 < rounds; u0 += kBatch) {
        int nlv[kBatch], np[kBatch];
        const bool more = u0 + kBatch < rounds;
        if (more) load_batch(u0 + kBatch, nlv, np);
        const int mine = (u0 + lane) * W + wave;  // the group lane u < kBatch puts together
        const bool have = lane < kBatch && mine < ng;
        Words par_words[kBatch];  // of the position's parent (T words); no parent, or one that is none: the zero word
#pragma unroll
        for (int u = 0; u < kBatch; u++) {
            const unsigned pc = min((unsigned)kp[u], (unsigned)pw * 32u - 1u);
#pragma unroll
            for (int h = 0; h < T; h++) par_words[u].w[h] = s_pars[(pc >> 5) * T + h];
        }
        if (have) need = *words(mine);
#pragma unroll
        for (int u = 0; u < kBatch; u++) {
#pragma unroll
            for (int h = 0; h < T; h++) {
                const unsigned long long by_parent = __ballot((par_words[u].w[h] >> (kp[u] & 31)) & 1u);
                if (lane == u) {
                    need.w[h] |= (uint32_t)by_parent;
                    need.w[T + h] |= (uint32_t)(by_parent >> 32);
                }
            }
        }
        if (have) {
            *words(mine) = need;
#pragma unroll
            for (int h = 0; h < T; h++) wtotal[h] += __popc(need.w[h]) + __popc(need.w[T + h]);
        }
        if (more) {
#pragma unroll
            for (int u = 0; u < kBatch; u++) klv[u] = nlv[u], kp[u] = np[u];
        }
    }
#pragma unroll
    for (int h = 0; h < T; h++) {
        const int t = __builtin_amdgcn_readlane(wave_scan(wtotal[h]), 63);
        if (lane == 0) s_wtotal[h][wave] = t;
    }
    if (check_parent && parent_level < 0) raise_error(a.counters);  // a parent must be a real position
    // (all loads have landed by now; said here, or the compiler waits for them, and with them for the reservation, where
    // the registers are used)
#pragma unroll
    for (int u = 0; u < kBatch; u++) asm volatile("" : "+v"(klv[u]), "+v"(kp[u]));
    lds_barrier();
    // These tiles' slice of the per-entry arrays: reserved by wave 1 as soon as the length of the lists is known,
    // used once the lists have been packed.  The last workgroup to reserve knows the final count and reports it
    // (no device-scope fence: it would write back the whole L2 of this XCD).  Where the host is waiting for exactly this
    // word, wave 1 looks at its reservation on the spot, and the lists and the bitmaps are made while the host goes on:
    // the others wait for it at the next barrier, 0.4 us of the kernel, and the host has its word some 2 us earlier.  Otherwise
    // it is looked at once the lists are sorted.  Us for a build that is waited for and a forward, later - on the spot: 1000
    // positions x 12 heads 27.2 - 25.9, 4 samples of them 27.7 - 26.4, 8192 x 12 32.7 - 31.7, 32768 x 4 43.1 - 42.1, with 256
    // workgroups, whose reservations queue, 8192 x 4 x 12 60.2 - 60.0; a build that is not waited for and a forward,
    // 8192 x 4 x 12, 50.3 - 51.5.
    auto look_at_reservation = [&](unsigned long long reserved, int n_all) {
        s_base = reserved_first(reserved);
        if (is_last(reserved)) {
            const int err = __hip_atomic_load(&a.counters[CNT_ERR], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            if (a.self_reset) {  // nobody touches the counters after the last reservation: clear them for the next build
                __hip_atomic_store(&a.counters[CNT_ERR], 0, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
                __hip_atomic_store(reinterpret_cast<unsigned long long *>(a.counters + CNT_CAND), 0ull, __ATOMIC_RELAXED,
                                   __HIP_MEMORY_SCOPE_AGENT);
            }
            const unsigned long long word = report_word(a.ticket, err, (uint32_t)(s_base + n_all));
            *a.report_dev = word;
            __hip_atomic_store(a.report, word, __ATOMIC_RELEASE, __HIP_MEMORY_SCOPE_SYSTEM);
        }
    };
    const bool early = a.host_waits != 0;
    unsigned long long reserved;  // (of thread 64; no value elsewhere, so that nothing waits for it before it is looked at)
    if (wave == 1) {
        int entries = 0;
#pragma unroll
        for (int h = 0; h < T; h++) {
            const int t = __builtin_amdgcn_readlane(wave_scan(lane < W ? s_wtotal[h][lane] : 0), 63);
            entries += (t + bn - 1) / bn;
            if (lane == 0) s_total[h] = t;
        }
        if (lane == 0) {
            const unsigned long long mine = reserve_entries(a.counters, entries);
            if (early)
                look_at_reservation(mine, entries);
            else
                reserved = mine;
        }
    }
    if (wave >= 4 && wave < 4 + T) {  // the needed keys of a tile in front of every group of 64 positions
        const int h = wave - 4;
        int first = 0;
        for (int g0 = 0; g0 < ng; g0 += 64) {
            const int g = g0 + lane;
            const int c = g < ng ? __popc(words(g)->w[h]) + __popc(words(g)->w[T + h]) : 0, incl = wave_scan(c);
            // (lists of more than kLdsKeys keys do not use these: that the counts wrap does not matter)
            if (g < ng) s_before[g * T + h] = (uint16_t)(first + incl - c);
            first += __builtin_amdgcn_readlane(incl, 63);
        }
    }
    lds_barrier();
    int total[T], n_ent[T], koff[T], n_all = 0;  // lengths of the lists, and where they begin in s_keys
#pragma unroll
    for (int h = 0; h < T; h++) {
        total[h] = __builtin_amdgcn_readfirstlane(s_total[h]);
        n_ent[h] = (total[h] + bn - 1) / bn;
        koff[h] = n_all * bn;
        n_all += n_ent[h];
    }
    const bool in_lds = n_all * bn <= kLdsKeys;
    auto bucket = [&](int l) { return a.no_sort ? 0 : bucket_of(l); };
    if (in_lds) {  // (while the reservation is in flight, unless the host waits)
        // document order: key and level in one word (positions take 19 bits), the parents beside it
        auto put = [&](uint32_t lo, uint32_t hi, int first, int g, int l, int p) {
            const unsigned long long m = (unsigned long long)lo | ((unsigned long long)hi << 32);
            if ((m >> lane) & 1ull) {
                const int t = first + __popcll(m & lanemask_lt());
                s_keys[t] = (bucket(l) << 24) | (g * 64 + lane);
                s_kpar[t] = p;
            }
        };
        if (one_batch) {
            const int mine = min(lane * W + wave, ng - 1);
#pragma unroll
            for (int h = 0; h < T; h++) {
                const int first = (h ? total[0] : 0) + s_before[mine * T + h];
                const unsigned long long some = __ballot(lane < kBatch && (need.w[h] | need.w[T + h]) != 0u);
#pragma unroll
                for (int u = 0; u < kBatch; u++)
                    if ((some >> u) & 1ull)
                        put(__builtin_amdgcn_readlane(need.w[h], u), __builtin_amdgcn_readlane(need.w[T + h], u),
                            __builtin_amdgcn_readlane(first, u), u * W + wave, klv[u], kp[u]);
            }
        } else {
            for (int u0 = 0; u0 < rounds; u0 += 64) {  // lane l looks at this wave's group u0 + l
                const int mine = (u0 + lane) * W + wave;
#pragma unroll
                for (int h = 0; h < T; h++) {
                    const bool have = mine < ng;
                    const uint32_t lo = have ? words(mine)->w[h] : 0u, hi = have ? words(mine)->w[T + h] : 0u;
                    const int first = (h ? total[0] : 0) + (have ? s_before[mine * T + h] : 0);
                    unsigned long long todo = __ballot((lo | hi) != 0u);
                    while (todo) {
                        const int x = __ffsll((long long)todo) - 1, g = (u0 + x) * W + wave, j = min(g * 64 + lane, n - 1);
                        todo &= todo - 1ull;
                        put(__builtin_amdgcn_readlane(lo, x), __builtin_amdgcn_readlane(hi, x), __builtin_amdgcn_readlane(first, x), g,
                            level[j], parent[j]);
                    }
                }
            }
        }
        lds_barrier();
        // key order: a wave takes groups of 64 of them (of one tile each) into registers and counts their levels; from
        // the counts of all groups it knows the first index of every level in its own
        int igroups[T], i0[T];
#pragma unroll
        for (int h = 0; h < T; h++) {
            igroups[h] = (total[h] + 63) >> 6;
            i0[h] = h ? igroups[0] : 0;
        }
        const int n_groups = igroups[0] + (T > 1 ? igroups[T - 1] : 0);
        int key[kRounds], par[kRounds], rank[kRounds];  // rank: keys of this one's level in front of it in its group
        auto tile_of = [&](int k) { return T > 1 && k >= igroups[0] ? T - 1 : 0; };
#pragma unroll
        for (int x = 0; x < kRounds; x++) {
            const int k = x * W + wave;
            if (k >= n_groups) break;
            const int h = tile_of(k), t = (k - i0[h]) * 64 + lane, at = (h ? total[0] : 0) + t;
            key[x] = t < total[h] ? s_keys[at] : -1;
            par[x] = t < total[h] ? s_kpar[at] : -1;
            const unsigned long long same = wave_bucket_match(key[x] >= 0, key[x] >> 24);
            rank[x] = __popcll(same & lanemask_lt());
            if (lane < kBuckets) s_lcnt[k][lane] = 0;
            if (key[x] >= 0 && rank[x] == 0) s_lcnt[k][key[x] >> 24] = __popcll(same);
        }
        lds_barrier();
        // Slots behind the last key name no key: they hold ~f, f = the tile's first real row (a list with a key has
        // one), which is the row the attention kernels gather for such a slot.
#pragma unroll
        for (int h = 0; h < T; h++)
            for (int t = total[h] + tid; t < n_ent[h] * bn; t += kListThreads) {
                s_keys[koff[h] + t] = ~s_first[h];
                s_kpar[koff[h] + t] = -1;
            }
#pragma unroll
        for (int x = 0; x < kRounds; x++) {
            const int k = x * W + wave;
            if (k >= n_groups) break;
            const int h = tile_of(k);
            int all = 0, before = 0;  // lane l: keys of level l, and those in front of this group
            if (lane < kBuckets)
                for (int e = i0[h]; e < i0[h] + igroups[h]; e++) {
                    const int c = s_lcnt[e][lane];
                    all += c;
                    before += e < k ? c : 0;
                }
            const int first_of_level = koff[h] + wave_scan(all) - all + before;
            const bool in = key[x] >= 0;
            const int t = __shfl(first_of_level, in ? key[x] >> 24 : 0) + rank[x];
            if (in) {
                s_keys[t] = key[x] & 0xffffff;
                s_kpar[t] = par[x];
            }
        }
    }
    if (tid == 64 && !early) look_at_reservation(reserved, n_all);
    lds_barrier();
    if (have_row) {  // (not earlier: a store takes 2-3 us to be acknowledged, and a wait for a later load waits for it)
        a.level_copy[(size_t)b * n + my_row] = my_level;
        a.parent_copy[(size_t)b * n + my_row] = my_parent;
    }
    // Entries past the capacity are not written, and a tile's range ends where they would begin: whoever walks
    // the lists stays inside the arrays (the host learns of the shortfall from the report and repeats the build
    // with larger arrays, or tells the caller of a deferred build to)
    int64_t base[T];
    int n_fit[T], key_fit[T];
    int32_t *keys[T], *kpars[T];
#pragma unroll
    for (int h = 0; h < T; h++) {
        base[h] = (int64_t)s_base + (h ? n_ent[0] : 0);
        const int64_t room = a.capacity - base[h];
        n_fit[h] = room <= 0 ? 0 : (room < n_ent[h] ? (int)room : n_ent[h]);
        key_fit[h] = n_fit[h] * bn;
        keys[h] = a.q_keys + (size_t)(room <= 0 ? 0 : base[h]) * bn;
        kpars[h] = a.q_kpar + (size_t)(room <= 0 ? 0 : base[h]) * bn;
        if (I0 + h < a.tr && tid == 0) {
            const size_t row = (size_t)b * a.tr + I0 + h;
            const int32_t first = (int32_t)(room <= 0 ? a.capacity : base[h]);
            a.q_range[2 * row] = first;
            a.q_range[2 * row + 1] = first + n_fit[h];
        }
        for (int e = tid; e < n_fit[h]; e += kListThreads) a.c_row[base[h] + e] = (int32_t)((size_t)b * a.tr + I0 + h);
        if (in_lds)
            for (int t = tid; t < key_fit[h]; t += kListThreads) keys[h][t] = s_keys[koff[h] + t];
    }
    if (!in_lds) {
        const int gpw = (ng + W - 1) / W, g0 = min(wave * gpw, ng), g1 = min(g0 + gpw, ng);  // this wave's share
#pragma unroll
        for (int h = 0; h < T; h++) {
            for (int t = total[h] + tid; t < key_fit[h]; t += kListThreads) keys[h][t] = ~s_first[h];
            // levels of the needed keys of the share, kBatch groups in flight
            auto each = [&](auto work) {
                for (int gb = g0; gb < g1; gb += kBatch) {
                    int l[kBatch], p[kBatch];
#pragma unroll
                    for (int u = 0; u < kBatch; u++) {
                        const int j = (gb + u) * 64 + lane;
                        const bool ok = gb + u < g1 && j < n;
                        l[u] = ok ? level[j] : -1;
                        p[u] = ok ? parent[j] : -1;
                    }
#pragma unroll
                    for (int u = 0; u < kBatch; u++) {
                        const int g = gb + u;
                        if (g >= g1) break;
                        const unsigned long long need = (unsigned long long)words(g)->w[h] | ((unsigned long long)words(g)->w[T + h] << 32);
                        if (need != 0ull) work(g, need, bucket(l[u]), p[u]);
                    }
                }
            };
            int mine = 0;  // lane k: needed keys of level k in the share
            each([&](int, unsigned long long m, int bk, int) { mine += wave_bucket_count((m >> lane) & 1ull, bk); });
            if (lane < kBuckets) s_lcnt[wave][lane] = mine;
            lds_barrier();
            int all = 0, before = 0;
            if (lane < kBuckets) {
#pragma unroll
                for (int w = 0; w < W; w++) {
                    all += s_lcnt[w][lane];
                    before += w < wave ? s_lcnt[w][lane] : 0;
                }
            }
            int next = wave_scan(all) - all + before;  // lane k: next index of level k in this wave
            each([&](int g, unsigned long long m, int bk_mine, int p) {
                const bool need = (m >> lane) & 1ull;
                int t = 0;
                unsigned long long remaining = m;
                while (remaining) {
                    const int bk = __builtin_amdgcn_readlane(bk_mine, __ffsll((long long)remaining) - 1);
                    const bool is_bk = need && bk_mine == bk;
                    const unsigned long long mm = __ballot(is_bk);
                    const int first = __builtin_amdgcn_readlane(next, bk);
                    if (is_bk) t = first + __popcll(mm & lanemask_lt());
                    if (lane == bk) next += __popcll(mm);
                    remaining &= ~mm;
                }
                if (need && t < key_fit[h]) {
                    keys[h][t] = g * 64 + lane;
                    kpars[h][t] = p;
                }
            });
            // The keys were written to global memory by other waves of this workgroup; the barrier orders those
            // stores before the loads below at workgroup scope, which is all that is needed on one compute unit
            // (the loads also bypass the vector cache).
            __syncthreads();
        }
    }
    // The entries, one wave per 64 key slots.  Lists kept in LDS: the waves take the entries of all tiles in one
    // sequence; lists that did not fit are brought back tile by tile, as many entries at a time as fit.
    const int wpe = (bn + 63) >> 6, per_round = W / wpe;  // waves per entry, entries per round
    const int quad = wave / wpe, k0 = (wave - quad * wpe) * 64;
    int parity = 0;
    auto finish = [&](bool active, int64_t c, const EntryPart &part) {  // pair count and summary of entry c
        if (wpe == 1) {
            if (active && lane == 0) {
                a.c_cnt[c] = part.cnt;
                a.q_sub[c] = part.any | (part.all << 16);
            }
            return;
        }
        // two waves per entry: the slots of this parity were last read two rounds ago, in front of the previous
        // round's barrier
        if (lane == 0) {
            s_cnt[parity][wave] = part.cnt;
            s_any[parity][wave] = part.any;
            s_all[parity][wave] = part.all;
        }
        lds_barrier();
        if (active && k0 == 0 && lane == 0) {
            a.c_cnt[c] = s_cnt[parity][wave] + s_cnt[parity][wave + 1];
            a.q_sub[c] = (s_any[parity][wave] | s_any[parity][wave + 1]) | ((s_all[parity][wave] | s_all[parity][wave + 1]) << 16);
        }
        parity ^= 1;
    };
    if (in_lds) {
        const int fit0 = n_fit[0], fits = fit0 + (T > 1 ? n_fit[T - 1] : 0);
        for (int x0 = 0; x0 < fits; x0 += per_round) {
            const int x = x0 + quad;
            const bool active = x < fits;
            const int h = T > 1 && active && x >= fit0 ? T - 1 : 0, e = x - (h ? fit0 : 0);
            EntryPart part;
            part.cnt = 0;
            part.any = part.all = 0;
            if (active)
                part = entry_columns(base[h] + e, k0, lane, tab[h], s_keys + koff[h] + e * bn, s_kpar + koff[h] + e * bn, row0[h],
                                     bm, bn, a.edges, a.bits_rm);
            finish(active, base[h] + e, part);
        }
        return;
    }
#pragma unroll
    for (int h = 0; h < T; h++) {
        const int at_once = kLdsKeys / bn;
        for (int e0 = 0; e0 < n_fit[h]; e0 += at_once) {
            const int entries = min(at_once, n_fit[h] - e0);
            lds_barrier();  // the previous entries' keys have been read
            for (int t = tid; t < entries * bn; t += kListThreads) {
                const int gi = e0 * bn + t;
                const int kk = __hip_atomic_load(&keys[h][gi], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
                int kq = -1;
                if (kk >= 0 && kk < n) kq = __hip_atomic_load(&kpars[h][gi], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
                s_keys[t] = (kk >= 0 && kk < n) ? kk : -1;
                s_kpar[t] = kq;
            }
            lds_barrier();
            for (int x0 = 0; x0 < entries; x0 += per_round) {
                const int x = x0 + quad;
                const bool active = x < entries;
                EntryPart part;
                part.cnt = 0;
                part.any = part.all = 0;
                if (active)
                    part = entry_columns(base[h] + e0 + x, k0, lane, tab[h], s_keys + x * bn, s_kpar + x * bn, row0[h], bm, bn,
                                         a.edges, a.bits_rm);
                finish(active, base[h] + e0 + x, part);
            }
        }
    }
}

template <int kListThreads, int T>
__global__ __launch_bounds__(kListThreads) void k_key_lists(KeyListArgs a)
{
    key_lists<kListThreads, T>(a);
}

// Two builds in one launch (the two schedules of a directed mask), blockIdx.y says which: twice the workgroups, so two of
// them share a compute unit, which with 1024 threads takes registers for 8 waves per SIMD (48 tiles of 64 rows per sample, 16
// samples: two launches 35 us, one with the registers of the kernel above 25.8, this one 22.5, and 17.2 with 512 threads; a
// kernel of its own, because the arguments read by index cost the single build 0.5 us).  With 1024 threads and T = 2 the
// bound spills 5 registers (24 bytes of scratch per lane) and keeps 32 scalars in vector lanes, which the figure includes.
template <int kListThreads, int T>
__global__ __launch_bounds__(kListThreads, kListThreads == 1024 ? 8 : 4) void k_key_lists_both(KeyListLaunch builds)
{
    key_lists<kListThreads, T>(builds.args[blockIdx.y]);
}

// ---- bitmaps of a windowed layout: exact evaluation of every candidate tile -----------------------
// One candidate per workgroup iteration, a pair of waves (entry_bitmaps).  The keys of the tile are a
// window of the key order; the positions behind its slots are also written to q_keys, which is what the
// attention kernels read.
__global__ __launch_bounds__(128) void k_tile_bitmaps(const int32_t *__restrict__ level,
                                                      const int32_t *__restrict__ parent,
                                                      const int32_t *__restrict__ kperm,
                                                      const int32_t *__restrict__ c_row,
                                                      const int32_t *__restrict__ c_col, int32_t *q_keys,
                                                      const int32_t *__restrict__ counters, int64_t capacity,
                                                      int n, int n_slots, int bm, int bn, int tr, int edges,
                                                      int force_dense, unsigned long long *bits_rm, int32_t *c_cnt,
                                                      uint32_t *c_sub)
{
    __shared__ int s_cnt[2], s_first[2];
    __shared__ uint32_t s_any[2], s_all[2], s_col[2][4];
    const int tid = threadIdx.x, wave = tid >> 6, lane = tid & 63;
    const int64_t total = min((int64_t)(uint32_t)counters[CNT_CAND], capacity);  // low word of the combined counter
    for (int64_t c = blockIdx.x; c < total; c += gridDim.x) {
        const int row = c_row[c], J = c_col[c];
        const int b = row / tr, I = row - b * tr;
        const size_t o = (size_t)b * n;
        // keys: lane l holds slots l and 64 + l of the tile
        int kpos[2], kpar[2];
#pragma unroll
        for (int u = 0; u < 2; u++) {
            const int si = 64 * u + lane, s = J * bn + si;
            kpos[u] = (si < bn && s < n_slots) ? kperm[(size_t)b * n_slots + s] : -1;
        }
        // this lane's row
        const int r = wave * 64 + lane, i = I * bm + r;
        bool rowok = r < bm && i < n;
        const int ii = rowok ? i : 0;
        const int li = level[o + ii], pi = parent[o + ii];
        rowok = rowok && li >= 0;
#pragma unroll
        for (int u = 0; u < 2; u++) {
            const bool okp = kpos[u] >= 0 && kpos[u] < n;
            const int pp = okp ? kpos[u] : 0;
            const int lv = level[o + pp], pr = parent[o + pp];
            kpos[u] = (okp && lv >= 0) ? kpos[u] : -1;
            kpar[u] = (okp && lv >= 0) ? pr : -1;
        }
        const EntryPart part = entry_bitmaps(true, c, wave, -1, lane, i, pi, rowok, kpos, kpar, bm, bn, edges, bits_rm);
        const unsigned long long real_rows = __ballot(rowok);
        __syncthreads();  // the previous candidate's partial results have been read
        if (lane == 0) {
            s_cnt[wave] = part.cnt;
            s_any[wave] = part.any;
            s_all[wave] = part.all;
            s_first[wave] = real_rows ? I * bm + wave * 64 + __ffsll((long long)real_rows) - 1 : INT_MAX;
#pragma unroll
            for (int wd = 0; wd < 4; wd++) s_col[wave][wd] = part.col[wd];
        }
        __syncthreads();
        if (wave == 0) {
            // A slot keeps its key only if some row of the tile may attend to it; the others (pads, slots past the
            // key order, keys of no concern to this tile) hold ~f, f = the tile's first real row (0 if it has
            // none): the row the attention kernels gather in their place.
            const int f = s_first[0] != INT_MAX ? s_first[0] : (s_first[1] != INT_MAX ? s_first[1] : 0);
#pragma unroll
            for (int u = 0; u < 2; u++) {
                const int si = 64 * u + lane;
                const bool seen = ((s_col[0][si >> 5] | s_col[1][si >> 5]) >> (si & 31)) & 1u;
                if (si < bn) q_keys[(size_t)c * bn + si] = seen ? kpos[u] : ~f;
            }
        }
        if (tid == 0) {
            c_cnt[c] = s_cnt[0] + s_cnt[1];
            // the dense baseline computes every sub-block, allowed pairs or not
            const uint32_t any = force_dense ? (1u << ((bm >> 5) * (bn >> 5))) - 1u : (s_any[0] | s_any[1]);
            c_sub[c] = any | ((s_all[0] | s_all[1]) << 16);
        }
    }
}

// ---- device memory: a small cache of buffers of destroyed layouts ------------------------------
struct CachedBlock {
    void *ptr;
    size_t bytes;
    int device;
    HdtUsers users;  // work that may still read or write the block
};
std::mutex g_pool_mutex;
std::vector<CachedBlock> g_pool;
constexpr size_t kPoolMaxBlocks = 16;
constexpr size_t kPoolMaxBytes = (size_t)1 << 30;
int64_t g_capacity_hint = 0;  // candidates the last build needed

// Events for the fences: a free list, the events carry no timing.  The list and its mutex are never destroyed:
// fences held by the cache return their events when the process ends, in an order nobody controls.
std::mutex &g_event_mutex = *new std::mutex();
std::vector<hipEvent_t> &g_free_events = *new std::vector<hipEvent_t>();
hipStream_t g_last_build_stream = nullptr;  // where the most recent layout build was enqueued (under g_event_mutex)

hipError_t take_fence_event(hipEvent_t *ev)
{
    {
        std::lock_guard<std::mutex> lk(g_event_mutex);
        if (!g_free_events.empty()) {
            *ev = g_free_events.back();
            g_free_events.pop_back();
            return hipSuccess;
        }
    }
    return hipEventCreateWithFlags(ev, hipEventDisableTiming);
}

// Whatever is enqueued on `next` from here on runs after the work the users of a block had enqueued: the fences
// recorded at the release, and for the remembered streams an event recorded now (that covers more work than
// needed, never less); nothing at all for `next` itself (stream order), and no host wait.
hipError_t order_after(const HdtUsers &users, hipStream_t next)
{
    if (users.whole_device) return hipDeviceSynchronize();
    for (auto &f : users.fences) {
        if (f->stream == next) continue;
        const hipError_t e = hipStreamWaitEvent(next, f->ev, 0);
        if (e != hipSuccess) return e;
    }
    for (int i = 0; i < users.lazy.n; i++) {
        if (users.lazy.s[i] == next) continue;
        hipEvent_t ev;
        hipError_t e = take_fence_event(&ev);
        if (e != hipSuccess) return e;
        e = hipEventRecord(ev, users.lazy.s[i]);
        if (e == hipSuccess) e = hipStreamWaitEvent(next, ev, 0);
        {
            std::lock_guard<std::mutex> lk(g_event_mutex);
            g_free_events.push_back(ev);  // a later record on it does not disturb the wait already enqueued
        }
        if (e != hipSuccess) {  // e.g. the caller has destroyed that stream since: wait for everything instead
            (void)hipGetLastError();
            e = hipDeviceSynchronize();
            if (e != hipSuccess) return e;
        }
    }
    return hipSuccess;
}

hipError_t pool_alloc(void **out, size_t bytes, size_t *got, hipStream_t next_user)
{
    int dev = 0;
    (void)hipGetDevice(&dev);
    HdtUsers users;
    bool found = false;
    {
        std::lock_guard<std::mutex> lk(g_pool_mutex);
        int best = -1;
        for (size_t i = 0; i < g_pool.size(); i++)
            if (g_pool[i].device == dev && g_pool[i].bytes >= bytes && g_pool[i].bytes <= 2 * bytes + (1 << 20) &&
                (best < 0 || g_pool[i].bytes < g_pool[best].bytes))
                best = (int)i;
        if (best >= 0) {
            *out = g_pool[best].ptr;
            *got = g_pool[best].bytes;
            users = std::move(g_pool[best].users);
            g_pool.erase(g_pool.begin() + best);
            found = true;
        }
    }
    if (found) {
        const hipError_t e = order_after(users, next_user);
        if (e != hipSuccess) {  // the block goes back as it was
            std::lock_guard<std::mutex> lk(g_pool_mutex);
            g_pool.push_back({*out, *got, dev, std::move(users)});
            *out = nullptr;
        }
        return e;
    }
    *got = bytes;
    return hipMalloc(out, bytes);
}

// The block goes to the cache; where it has no room, the blocks that have been there longest make some (the sizes a
// program has stopped using: kept, they would send every later build to hipMalloc and hipFree, which waits for the device).
void pool_free(void *ptr, size_t bytes, int device, const HdtUsers &users)
{
    if (!ptr) return;
    std::vector<CachedBlock> out;
    if (bytes <= kPoolMaxBytes) {
        std::lock_guard<std::mutex> lk(g_pool_mutex);
        size_t held = bytes, drop = 0;
        for (auto &b : g_pool) held += b.bytes;
        while (drop < g_pool.size() && (held > kPoolMaxBytes || g_pool.size() - drop >= kPoolMaxBlocks)) held -= g_pool[drop++].bytes;
        for (size_t i = 0; i < drop; i++) out.push_back(std::move(g_pool[i]));
        g_pool.erase(g_pool.begin(), g_pool.begin() + (ptrdiff_t)drop);
        g_pool.push_back({ptr, bytes, device, users});
        ptr = nullptr;
    }
    for (auto &b : out) (void)hipFree(b.ptr);  // waits for the device
    if (ptr) (void)hipFree(ptr);
}

// carve buffers (each rounded up to 256 bytes) out of an arena
struct Carver {
    char *base;
    size_t off = 0;
    template <typename T>
    T *take(size_t count)
    {
        T *p = base ? reinterpret_cast<T *>(base + off) : nullptr;
        off += (count * sizeof(T) + 255) & ~(size_t)255;
        return p;
    }
};

struct Phase1 {
    int32_t *kperm, *slot, *cmin, *cmax, *hist, *q_range, *counters, *level_copy, *parent_copy;
    unsigned long long *report_copy;
    size_t zero_begin, zero_end;  // byte range that must start at zero
    size_t bytes;
};

Phase1 carve_phase1(char *base, int B, int n, int n_slots, int tr, int nchunks)
{
    Carver c{base};
    Phase1 p;
    p.kperm = c.take<int32_t>((size_t)B * n_slots);
    p.slot = c.take<int32_t>((size_t)B * n);
    p.cmin = c.take<int32_t>((size_t)B * n);
    p.cmax = c.take<int32_t>((size_t)B * n);
    p.hist = c.take<int32_t>((size_t)B * nchunks * kBuckets);
    p.q_range = c.take<int32_t>((size_t)B * tr * 2);
    p.level_copy = c.take<int32_t>((size_t)B * n);
    p.parent_copy = c.take<int32_t>((size_t)B * n);
    p.report_copy = c.take<unsigned long long>(1);
    p.zero_begin = c.off;
    p.counters = c.take<int32_t>(64);
    p.zero_end = c.off;
    p.bytes = c.off;
    return p;
}

struct Phase2 {
    int32_t *q_cols, *c_row, *c_cnt, *q_keys, *q_kpar;
    uint32_t *q_sub;
    unsigned long long *bits_rm;
    size_t bytes;
};

Phase2 carve_phase2(char *base, int64_t cap, int bm, int bn)
{
    Carver c{base};
    Phase2 p;
    const size_t n = (size_t)cap, nsub = (size_t)(bm / 32) * (bn / 32);
    p.q_cols = c.take<int32_t>(n);
    p.q_sub = c.take<uint32_t>(n);
    p.c_row = c.take<int32_t>(n);
    p.c_cnt = c.take<int32_t>(n);
    p.q_keys = c.take<int32_t>(n * (size_t)bn);
    p.q_kpar = c.take<int32_t>(n * (size_t)bn);
    p.bits_rm = c.take<unsigned long long>(n * nsub * 16);
    p.bytes = c.off;
    return p;
}

// ---- the build's report from the device: words of pinned host memory, one per build in flight ----
constexpr int kReportSlots = 1024;
unsigned long long *g_reports = nullptr;  // never freed: a kernel may still write to it at exit
uint32_t g_ticket = 0;

unsigned long long *report_slot(uint32_t *ticket, uint32_t *ticket_before)
{
    std::lock_guard<std::mutex> lk(g_pool_mutex);
    if (!g_reports) {
        void *ptr = nullptr;
        if (hipHostMalloc(&ptr, kReportSlots * 64, hipHostMallocPortable | hipHostMallocMapped) != hipSuccess) {
            (void)hipGetLastError();
            return nullptr;
        }
        memset(ptr, 0, kReportSlots * 64);
        g_reports = static_cast<unsigned long long *>(ptr);
    }
    g_ticket = (g_ticket + 1) & 0xffffffu;
    if (g_ticket == 0) g_ticket = 1;
    *ticket = g_ticket;
    unsigned long long *slot = g_reports + (size_t)(g_ticket % kReportSlots) * 8;  // one 64-byte line per slot
    *ticket_before = (uint32_t)(__atomic_load_n(slot, __ATOMIC_ACQUIRE) >> 40);
    if (*ticket_before == *ticket) {  // the ticket counter has wrapped around: a report of 2^24 builds ago
        __atomic_store_n(slot, 0ull, __ATOMIC_RELEASE);
        *ticket_before = 0;
    }
    return slot;
}

// How many list entries builds of a shape need: a build whose report nobody waits for has lists about as long as the last one
// of its shape that has reported (documents of one kind, step after step, while the host runs ahead).  The reports are
// read in the order of the builds, as far as they are in, whenever a build is noted; the last kShapes shapes are kept.
struct BuildShape {
    int32_t batch, n, bm, bn, edges;
    bool operator==(const BuildShape &o) const
    {
        return batch == o.batch && n == o.n && bm == o.bm && bn == o.bn && edges == o.edges;
    }
};
struct SlotBuild {
    BuildShape shape;
    uint32_t ticket;
} g_slot_builds[kReportSlots] = {};  // who owns or owned a report slot
struct ShapeEntries {
    BuildShape shape;
    int64_t entries;
};
constexpr int kShapes = 32;
std::vector<ShapeEntries> &g_shapes = *new std::vector<ShapeEntries>();  // oldest first
uint32_t g_unread = 1;                                                   // the first ticket whose report has not been read

// Notes the build of `ticket`; list entries of the last build before it that had its shape, -1: none is known.
int64_t entries_of_one_like(uint32_t ticket, const BuildShape &shape)
{
    std::lock_guard<std::mutex> lk(g_pool_mutex);
    auto find = [](const BuildShape &what) {
        size_t i = 0;
        while (i < g_shapes.size() && !(g_shapes[i].shape == what)) i++;
        return i;
    };
    // (a build of another thread with a later ticket may have been here before: then there is nothing to read)
    const uint32_t ahead = (ticket - g_unread) & 0xffffffu, until = ahead < 0x800000u ? ticket : g_unread;
    if (until == ticket && ahead >= (uint32_t)kReportSlots) g_unread = (ticket - kReportSlots + 1) & 0xffffffu;
    for (; g_unread != until; g_unread = (g_unread + 1) & 0xffffffu) {
        const SlotBuild &x = g_slot_builds[g_unread % kReportSlots];
        if (g_unread == 0 || x.ticket != g_unread) continue;  // a build of another kind
        const unsigned long long word = __atomic_load_n(g_reports + (size_t)(g_unread % kReportSlots) * 8, __ATOMIC_ACQUIRE);
        if ((uint32_t)(word >> 40) != g_unread) break;
        if ((word >> 39) & 1u) continue;
        const size_t at = find(x.shape);
        if (at < g_shapes.size()) {
            g_shapes[at].entries = (int64_t)(word & 0xffffffffu);
            continue;
        }
        if (g_shapes.size() == kShapes) g_shapes.erase(g_shapes.begin());
        g_shapes.push_back({x.shape, (int64_t)(word & 0xffffffffu)});
    }
    g_slot_builds[ticket % kReportSlots] = {shape, ticket};
    const size_t at = find(shape);
    return at < g_shapes.size() ? g_shapes[at].entries : -1;
}

// The counters of a key-list build: device memory, one 256-byte slot per build in flight (chosen by the
// ticket, like the report word), zero whenever no build owns it: the kernel's last workgroup clears the slot
// before it reports, so a build needs no clearing launch of its own.  Never freed.
constexpr int kCounterDevices = 64;
int32_t *g_counter_slots[kCounterDevices] = {};

int32_t *counter_slot(int device, uint32_t ticket)
{
    if (device < 0 || device >= kCounterDevices) return nullptr;
    std::lock_guard<std::mutex> lk(g_pool_mutex);
    if (!g_counter_slots[device]) {
        void *ptr = nullptr;
        const size_t bytes = (size_t)kReportSlots * 64 * sizeof(int32_t);
        if (hipMalloc(&ptr, bytes) != hipSuccess || hipMemset(ptr, 0, bytes) != hipSuccess) {
            (void)hipGetLastError();
            if (ptr) (void)hipFree(ptr);
            return nullptr;
        }
        g_counter_slots[device] = static_cast<int32_t *>(ptr);
    }
    return g_counter_slots[device] + (size_t)(ticket % kReportSlots) * 64;
}

// polls the word until it carries this build's ticket; false after 10 s without it, or at once when the slot
// has been taken over by a later build (it then holds neither this ticket nor the one it held before)
bool wait_for_report(const unsigned long long *slot, uint32_t ticket, uint32_t ticket_before, unsigned long long *word)
{
    const auto t0 = std::chrono::steady_clock::now();
    for (uint64_t spins = 0;; spins++) {
        const unsigned long long w = __atomic_load_n(slot, __ATOMIC_ACQUIRE);
        if ((uint32_t)(w >> 40) == ticket) {
            *word = w;
            return true;
        }
        if ((uint32_t)(w >> 40) != ticket_before) return false;
        if ((spins & 0x3ff) == 0x3ff && std::chrono::steady_clock::now() - t0 > std::chrono::seconds(10)) return false;
        __builtin_ia32_pause();
    }
}

// The same for a cross-attention build, whose word no other build writes before its report is in: until it is, however long
// the stream takes, and without a call that a stream being captured would refuse.  False: another thread has recorded the
// report meanwhile (the word may be another build's by now).
bool wait_for_own_report(const hdt_layout_t *L, unsigned long long *word)
{
    const auto t0 = std::chrono::steady_clock::now();
    for (uint64_t spins = 1;; spins++) {
        const unsigned long long w = __atomic_load_n(L->report, __ATOMIC_ACQUIRE);
        if ((uint32_t)(w >> 40) == L->ticket) {
            *word = w;
            return true;
        }
        if (!L->pending.load(std::memory_order_acquire)) return false;
        if ((spins & 0x3ff) == 0 && std::chrono::steady_clock::now() - t0 > std::chrono::seconds(1)) usleep(100);
        __builtin_ia32_pause();
    }
}

// Words and counters of cross-attention builds, per device: the ones without a layout that reads them, longest there first.
// One whose layout was destroyed early may still be waiting for its report.  Never freed: a kernel may still write at exit,
// and a layout may be destroyed then.
constexpr int kReportPage = 256;
std::mutex &g_reports_mutex = *new std::mutex();
std::vector<HdtReport> *const g_free_reports = new std::vector<HdtReport>[kCounterDevices];

const char kHierarchyText[] =
    "level/parent arrays are not a valid hierarchy (level outside [-1, 32), parent outside [-1, n_pos), self-parent, "
    "pad with a parent, or pad parent)";

// One launch for one key-list build, or for two that differ in their edges and arrays only.
hipError_t launch_key_lists(const KeyListArgs *args, int builds, int batch, hipStream_t st)
{
    const KeyListArgs &a = args[0];
    const bool small_wg = a.bm <= 64;
    // tiles of up to 64 rows: two per workgroup, as long as the two sets of bitmaps fit the LDS beside the
    // kernel's static arrays (documents of up to 67 K positions)
    const bool pair = small_wg && list_lds(a.n, 2) <= 33 * 1024;
    const size_t lds = list_lds(a.n, pair ? 2 : 1);
    const dim3 grid((unsigned)batch * (pair ? (a.tr + 1) / 2 : a.tr), (unsigned)builds);
#define LIST_LAUNCH(THREADS, TILES)                                                                                         \
    do {                                                                                                                    \
        if (lds > 33 * 1024) { /* with the kernel's static arrays: beyond the 64 KB a launch gets by default */             \
            const void *f = builds == 2 ? (const void *)k_key_lists_both<THREADS, TILES> : (const void *)k_key_lists<THREADS, TILES>; \
            const hipError_t e = hipFuncSetAttribute(f, hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds);              \
            if (e != hipSuccess) return e;                                                                                  \
        }                                                                                                                   \
        HdtTimer t("hdt_layout_key_lists", st);                                                                             \
        if (builds == 2) {                                                                                                  \
            const KeyListLaunch two = {{args[0], args[1]}};                                                                 \
            hipLaunchKernelGGL((k_key_lists_both<THREADS, TILES>), grid, dim3(THREADS), lds, st, two);                      \
        } else {                                                                                                            \
            hipLaunchKernelGGL((k_key_lists<THREADS, TILES>), grid, dim3(THREADS), lds, st, a);                             \
        }                                                                                                                   \
    } while (0)
    // 512 threads where the scan then still is a single batch (see key_lists)
    const bool short_doc = a.n <= 512 * kBatch;
    if (pair && short_doc)
        LIST_LAUNCH(512, 2);
    else if (pair)
        LIST_LAUNCH(1024, 2);
    else if (small_wg || short_doc)
        LIST_LAUNCH(512, 1);
    else
        LIST_LAUNCH(1024, 1);
#undef LIST_LAUNCH
    return hipGetLastError();
}

// Two key-list builds that share a launch: the second one makes it.
struct BothBuilds {
    KeyListArgs args[2];
    int n = 0;
};

}  // namespace

// What the report of a build says that went out with it unread; recorded at most once per layout.
static hdt_status_t resolve_one(const hdt_layout_t *L, bool wait, const hipStream_t *built_on)
{
    if (L->pending.load(std::memory_order_acquire)) {
        unsigned long long word = __atomic_load_n(L->report, __ATOMIC_ACQUIRE);
        bool have = (uint32_t)(word >> 40) == L->ticket;
        if (!have && !wait) return HDT_OK;
        // No lock is held here: a build behind a busy stream keeps its caller waiting and nobody else.
        if (!have) have = L->cross ? wait_for_own_report(L, &word) : wait_for_report(L->report, L->ticket, L->ticket_before, &word);
        if (!have && !L->cross) {
            // the slot has gone to a later build (or nothing came for 10 s): the copy in the layout's own memory
            int dev = 0;
            HDT_HIP_TRY(hipGetDevice(&dev));
            if (dev != L->device) HDT_HIP_TRY(hipSetDevice(L->device));
            hipError_t e = built_on ? hipStreamSynchronize(*built_on) : hipDeviceSynchronize();
            if (e == hipSuccess) e = hipMemcpy(&word, L->report_dev, sizeof(word), hipMemcpyDeviceToHost);
            if (dev != L->device) (void)hipSetDevice(dev);
            if (e != hipSuccess) return hdt_fail(HDT_ERR_HIP, "hdt_layout_resolve: %s", hipGetErrorString(e));
            if ((uint32_t)(word >> 40) != L->ticket)
                return hdt_fail(HDT_ERR_HIP, "hdt_layout_resolve: the build kernel finished without its report");
        }
        static std::mutex record_mutex;
        std::lock_guard<std::mutex> lk(record_mutex);
        if (L->pending.load(std::memory_order_relaxed) && L->cross) {
            hdt_cross_record(L, (int)(uint32_t)(word & 0xffffffffu));
            L->pending.store(false, std::memory_order_release);
            hdt_report_close(L->device, L->own_report);
        } else if (L->pending.load(std::memory_order_relaxed)) {
            const int64_t need = (int64_t)(word & 0xffffffffu);
            L->entries_needed = need;
            if ((word >> 39) & 1u) {
                L->build_status = HDT_ERR_HIERARCHY;
                snprintf(L->build_error, sizeof(L->build_error), "deferred hdt_build_layout: %s", kHierarchyText);
            } else if (need > L->capacity) {
                L->build_status = HDT_ERR_SHAPE;
                snprintf(L->build_error, sizeof(L->build_error),
                         "deferred hdt_build_layout: the schedule needs %lld list entries, the layout holds %lld "
                         "(build again with opts->capacity)", (long long)need, (long long)L->capacity);
            } else {
                L->n_entries = need;
            }
            if (!((word >> 39) & 1u)) {
                std::lock_guard<std::mutex> lk2(g_pool_mutex);
                g_capacity_hint = need;
            }
            L->pending.store(false, std::memory_order_release);
        }
    }
    if (L->build_status != HDT_OK) return hdt_fail(L->build_status, "%s", L->build_error);
    return HDT_OK;
}

hdt_status_t hdt_layout_resolve(const hdt_layout_t *L, bool wait, const hipStream_t *built_on)
{
    if (hdt_status_t st = resolve_one(L, wait, built_on)) return st;
    if (L->transposed) return resolve_one(L->transposed, wait, built_on);
    return HDT_OK;
}

hipError_t hdt_pool_alloc(void **out, size_t bytes, size_t *got, hipStream_t next_user)
{
    return pool_alloc(out, bytes, got, next_user);
}

bool hdt_report_open(int device, HdtReport *r)
{
    if (device < 0 || device >= kCounterDevices) return false;
    std::lock_guard<std::mutex> lk(g_reports_mutex);
    std::vector<HdtReport> &free = g_free_reports[device];
    for (size_t i = 0; i < free.size(); i++) {
        if ((uint32_t)(__atomic_load_n(free[i].word, __ATOMIC_ACQUIRE) >> 40) != free[i].ticket) continue;  // not in yet
        *r = free[i];
        r->ticket = (r->ticket + 1) & 0xffffffu;
        free.erase(free.begin() + (ptrdiff_t)i);
        return true;
    }
    // none: kReportPage more (a line per word, 256 bytes per build's counters), cleared on a stream that waits for no other
    void *words = nullptr, *counters = nullptr;
    hipStream_t st = nullptr;
    const size_t counter_bytes = (size_t)kReportPage * 64 * sizeof(int32_t);
    bool ok = hipHostMalloc(&words, kReportPage * 64, hipHostMallocPortable | hipHostMallocMapped) == hipSuccess &&
              hipMalloc(&counters, counter_bytes) == hipSuccess &&
              hipStreamCreateWithFlags(&st, hipStreamNonBlocking) == hipSuccess;
    if (ok) {
        ok = hipMemsetAsync(counters, 0, counter_bytes, st) == hipSuccess && hipStreamSynchronize(st) == hipSuccess;
        (void)hipStreamDestroy(st);
    }
    if (!ok) {
        (void)hipGetLastError();
        if (words) (void)hipHostFree(words);
        if (counters) (void)hipFree(counters);
        return false;
    }
    memset(words, 0, kReportPage * 64);
    for (size_t i = 0; i < kReportPage; i++)
        free.push_back({static_cast<unsigned long long *>(words) + i * 8, static_cast<int32_t *>(counters) + i * 64, 0});
    *r = free[free.size() - kReportPage];
    r->ticket = 1;
    free.erase(free.end() - kReportPage);
    return true;
}

void hdt_report_close(int device, const HdtReport &r)
{
    std::lock_guard<std::mutex> lk(g_reports_mutex);
    g_free_reports[device].push_back(r);
}

void hdt_layout_release(hdt_layout_t *L, const HdtUsers &users)
{
    pool_free(L->arena, L->arena_bytes, L->device, users);
    pool_free(L->arena2, L->arena2_bytes, L->device, users);
    L->arena = L->arena2 = nullptr;
}

HdtFence::~HdtFence()
{
    std::lock_guard<std::mutex> lk(g_event_mutex);
    g_free_events.push_back(ev);
}

HdtUsers hdt_users_at_release(const HdtStreams &streams)
{
    HdtUsers u;
    if (streams.more) {
        u.whole_device = true;
        return u;
    }
    hipStream_t builds;
    {
        std::lock_guard<std::mutex> lk(g_event_mutex);
        builds = g_last_build_stream;
    }
    for (int i = 0; i < streams.n; i++) {
        if (streams.s[i] == builds) {
            u.lazy.add(streams.s[i]);
            continue;
        }
        hipEvent_t ev;
        if (take_fence_event(&ev) != hipSuccess || hipEventRecord(ev, streams.s[i]) != hipSuccess) {
            (void)hipGetLastError();
            u.whole_device = true;  // the next owner waits for the device instead
            return u;
        }
        u.fences.push_back(std::shared_ptr<HdtFence>(new HdtFence{ev, streams.s[i]}));
    }
    return u;
}

// a buffer that only a build on `st` has touched
static HdtUsers only_stream(hipStream_t st)
{
    HdtUsers u;
    u.lazy.add(st);
    return u;
}

void hdt_note_build_stream(hipStream_t st)
{
    std::lock_guard<std::mutex> lk(g_event_mutex);
    g_last_build_stream = st;
}

static std::mutex g_streams_mutex;  // attention calls on one layout may come from several host threads

void hdt_layout_note_stream(const hdt_layout_t *L, hipStream_t st)
{
    std::lock_guard<std::mutex> lk(g_streams_mutex);
    L->streams.add(st);
}

HdtStreams hdt_layout_streams(const hdt_layout_t *L)
{
    std::lock_guard<std::mutex> lk(g_streams_mutex);
    return L->streams;
}

// Surviving tiles and allowed pairs per sample, summed on the host from the query tile and the pair
// count of every list entry (two adjacent device arrays): cheaper than thousands of device atomics on
// a handful of addresses, and only paid by callers that ask.
hdt_status_t hdt_layout_stats(const hdt_layout_t *L)
{
    static std::mutex stats_mutex;
    std::lock_guard<std::mutex> lk(stats_mutex);
    if (L->stats_ready) return HDT_OK;
    if (hdt_status_t st = hdt_layout_resolve(L, true)) return st;
    const int64_t E = L->n_entries;
    std::vector<int32_t> row((size_t)E), cnt((size_t)E);
    int dev = 0;
    HDT_HIP_TRY(hipGetDevice(&dev));
    if (dev != L->device) HDT_HIP_TRY(hipSetDevice(L->device));
    hipError_t e = hipDeviceSynchronize();
    if (e == hipSuccess && E > 0) e = hipMemcpy(row.data(), L->d_row, sizeof(int32_t) * E, hipMemcpyDeviceToHost);
    if (e == hipSuccess && E > 0) e = hipMemcpy(cnt.data(), L->d_cnt, sizeof(int32_t) * E, hipMemcpyDeviceToHost);
    if (dev != L->device) (void)hipSetDevice(dev);
    if (e != hipSuccess) return hdt_fail(HDT_ERR_HIP, "hdt_layout_stats: %s", hipGetErrorString(e));
    std::fill(L->h_stats.begin(), L->h_stats.end(), 0);
    const int B = L->s.batch, tr = L->s.tr;
    for (int64_t c = 0; c < E; c++) {
        const int b = row[c] / tr;
        if (b < 0 || b >= B) continue;
        if (cnt[c] > 0 || L->force_dense) {
            L->h_stats[2 * b] += 1;
            L->h_stats[2 * b + 1] += cnt[c];
        }
    }
    L->stats_ready = true;
    return HDT_OK;
}

// The key order of a layout built from key lists: sorted from the layout's own copy of the ids by the
// first caller that asks for it (the build itself never needs it).  Waits for the device.
hdt_status_t hdt_layout_ensure_kperm(const hdt_layout_t *L)
{
    static std::mutex kperm_mutex;
    std::lock_guard<std::mutex> lk(kperm_mutex);
    if (L->kperm_ready || L->s.batch == 0 || L->s.n_pos == 0) return HDT_OK;
    int dev = 0;
    HDT_HIP_TRY(hipGetDevice(&dev));
    if (dev != L->device) HDT_HIP_TRY(hipSetDevice(L->device));
    hipError_t e = hipDeviceSynchronize();
    if (e == hipSuccess) {
        const int B = L->s.batch, n = L->s.n_pos, nchunks = (n + kChunk - 1) / kChunk;
        SortArgs sa{L->level_copy, L->parent_copy, n, L->s.n_slots, nchunks, L->no_sort, L->sort_hist,
                    const_cast<int32_t *>(L->s.kperm), nullptr, nullptr, nullptr, L->sort_counters, 0, nullptr};
        hipLaunchKernelGGL(k_sort_count, dim3((unsigned)B * nchunks), dim3(kThreads), 0, nullptr, sa);
        hipLaunchKernelGGL(k_sort_scatter, dim3((unsigned)B * nchunks), dim3(kThreads), 0, nullptr, sa);
        e = hipGetLastError();
        if (e == hipSuccess) e = hipDeviceSynchronize();
    }
    if (dev != L->device) (void)hipSetDevice(dev);
    if (e != hipSuccess) return hdt_fail(HDT_ERR_HIP, "hdt_layout_ensure_kperm: %s", hipGetErrorString(e));
    L->kperm_ready = true;
    return HDT_OK;
}

extern "C" __attribute__((visibility("default"))) hdt_status_t hdt_release_cached_memory(void)
{
    std::vector<CachedBlock> blocks;
    {
        std::lock_guard<std::mutex> lk(g_pool_mutex);
        blocks.swap(g_pool);
    }
    hipError_t e = hipSuccess;
    for (auto &b : blocks) {
        hipError_t e2 = hipFree(b.ptr);
        if (e == hipSuccess) e = e2;
    }
    if (e != hipSuccess) return hdt_fail(HDT_ERR_HIP, "hipFree: %s", hipGetErrorString(e));
    return HDT_OK;
}

static hdt_status_t build_one(const int32_t *d_level, const int32_t *d_parent, int32_t batch, int32_t n_pos,
                              const hdt_layout_opts_t *opts, int edges, void *stream, BothBuilds *both, hdt_layout_t **out);

static int swap_up_down(int edges)
{
    return (edges & HDT_EDGE_SIBLING) | ((edges & HDT_EDGE_UP) ? HDT_EDGE_DOWN : 0) | ((edges & HDT_EDGE_DOWN) ? HDT_EDGE_UP : 0);
}

extern "C" __attribute__((visibility("default"))) hdt_status_t hdt_build_layout(const int32_t *d_level,
                                                                                 const int32_t *d_parent,
                                                                                 int32_t batch, int32_t n_pos,
                                                                                 const hdt_layout_opts_t *opts,
                                                                                 void *stream, hdt_layout_t **out)
{
    if (!out) return hdt_fail(HDT_ERR_INVALID_ARG, "hdt_build_layout: out is NULL");
    *out = nullptr;
    int edges = opts && opts->edges ? opts->edges : HDT_EDGE_ALL;
    if (edges & ~HDT_EDGE_ALL) return hdt_fail(HDT_ERR_INVALID_ARG, "hdt_build_layout: edges = %d", edges);
    hdt_layout_t *L = nullptr;
    hdt_status_t st;
    if (swap_up_down(edges) == edges) {
        st = build_one(d_level, d_parent, batch, n_pos, opts, edges, stream, nullptr, &L);
        if (st == HDT_OK) *out = L;
        return st;
    }
    // A directed mask: the backward pass also needs the schedule of its transpose, which is the same
    // construction with the parent and child kinds exchanged.  Key lists: both in one launch, neither waited for before
    // both are enqueued.
    const bool lists = batch > 0 && n_pos > 0 && !(opts && (opts->windowed || opts->force_dense));
    const bool deferred = opts && opts->deferred;
    for (int attempt = 0; attempt < 2; attempt++) {
        BothBuilds builds, *both = lists && attempt == 0 ? &builds : nullptr;
        st = build_one(d_level, d_parent, batch, n_pos, opts, edges, stream, both, &L);
        if (st != HDT_OK) return st;
        st = build_one(d_level, d_parent, batch, n_pos, opts, swap_up_down(edges), stream, both, &L->transposed);
        if (st == HDT_OK && both && !deferred) {
            const hipStream_t built_on = (hipStream_t)stream;
            st = hdt_layout_resolve(L, true, &built_on);
            if (st == HDT_ERR_HIERARCHY) st = hdt_fail(st, "hdt_build_layout: %s", kHierarchyText);
            if (st == HDT_ERR_SHAPE && !(opts && opts->capacity > 0)) {
                // the guess of the arrays' sizes was too small (the exact number is known now): one after the other
                (void)hdt_layout_destroy(L);
                continue;
            }
            if (st == HDT_ERR_SHAPE)
                st = hdt_fail(st, "hdt_build_layout: the schedule needs %lld list entries, opts->capacity is %lld",
                              (long long)std::max(L->entries_needed, L->transposed->entries_needed), (long long)opts->capacity);
        }
        break;
    }
    if (st != HDT_OK) {
        (void)hdt_layout_destroy(L);
        return st;
    }
    L->device_bytes += L->transposed->device_bytes;
    *out = L;
    return HDT_OK;
}

// `both`: the kernel is launched with that of the other build, by the second of the two calls; the layout then comes back
// with its report not yet looked at, as from a deferred build.
static hdt_status_t build_one(const int32_t *d_level, const int32_t *d_parent, int32_t batch, int32_t n_pos,
                              const hdt_layout_opts_t *opts, int edges, void *stream, BothBuilds *both, hdt_layout_t **out)
{
    *out = nullptr;
    if (batch < 0 || n_pos < 0) return hdt_fail(HDT_ERR_INVALID_ARG, "hdt_build_layout: negative size");
    if (n_pos > (1 << 19)) return hdt_fail(HDT_ERR_SHAPE, "hdt_build_layout: n_pos %d > 2^19", n_pos);
    int bm = 128, bn = 64, force_dense = 0, no_sort = 0, windowed = 0;
    bool deferred = false;
    int64_t capacity_opt = 0;
    if (opts) {
        if (opts->tile_m) bm = opts->tile_m;
        if (opts->tile_n) bn = opts->tile_n;
        force_dense = opts->force_dense != 0;
        no_sort = opts->no_sort != 0;
        windowed = opts->windowed != 0 || force_dense;
        if (opts->capacity < 0) return hdt_fail(HDT_ERR_INVALID_ARG, "hdt_build_layout: capacity = %lld", (long long)opts->capacity);
        capacity_opt = opts->capacity;
        deferred = opts->deferred != 0 && !windowed;  // the windowed kernels are launched from what the first reports
    }
    if (bm < 32 || bm > 128 || bm % 32 || bn < 32 || bn > 128 || bn % 32)
        return hdt_fail(HDT_ERR_UNSUPPORTED, "hdt_build_layout: tile %dx%d (each side: 32, 64, 96 or 128)", bm, bn);
    const bool empty = batch == 0 || n_pos == 0;
    if (!empty && (!d_level || !d_parent)) return hdt_fail(HDT_ERR_INVALID_ARG, "hdt_build_layout: NULL id array");

    hdt_layout_t *L = new (std::nothrow) hdt_layout_t();
    if (!L) return hdt_fail(HDT_ERR_OOM, "hdt_build_layout: host allocation failed");
    L->magic = HDT_LAYOUT_MAGIC;
    L->arena = L->arena2 = nullptr;
    L->arena_bytes = L->arena2_bytes = 0;
    L->capacity = 0;
    L->d_cnt = nullptr;
    L->d_row = nullptr;
    L->n_entries = 0;
    L->stats_ready = false;
    L->kperm_ready = true;
    L->no_sort = 0;
    L->sort_hist = L->sort_counters = nullptr;
    L->level_copy = L->parent_copy = nullptr;
    L->force_dense = force_dense;
    L->windowed = windowed;
    L->edges = edges;
    L->cross = 0;
    L->cross_level_mask = 0;
    L->transposed = nullptr;
    L->compact = L->compact_built = nullptr;
    L->n_compact = 0;
    L->device_bytes = 0;
    L->device = 0;
    L->pending = false;
    L->build_status = HDT_OK;
    L->entries_needed = 0;
    L->entries_like = -1;
    L->build_error[0] = 0;
    L->report = L->report_dev = nullptr;
    L->ticket = L->ticket_before = 0;
    HdtSchedule &s = L->s;
    memset(&s, 0, sizeof(s));
    s.batch = batch;
    s.n_pos = n_pos;
    s.n_kv = n_pos;
    s.bm = bm;
    s.bn = bn;
    s.wpr = bn / 32;
    s.tr = empty ? 0 : (n_pos + bm - 1) / bm;
    s.tc = empty ? 0 : (n_pos + bn - 1) / bn;
    s.n_slots = s.tc * bn;
    s.n_own = n_pos;
    s.tr_own = s.tr;
    L->h_stats.assign((size_t)batch * 2, 0);
    if (empty) {
        L->stats_ready = true;
        *out = L;
        return HDT_OK;
    }
    if ((int64_t)batch * n_pos > (1LL << 30) || (int64_t)batch * s.tr * s.tc >= (1LL << 31)) {
        delete L;
        return hdt_fail(HDT_ERR_SHAPE, "hdt_build_layout: batch * n_pos too large");
    }

    hipStream_t st = (hipStream_t)stream;
    L->streams.add(st);
    hdt_note_build_stream(st);
    const int B = batch, n = n_pos, tr = s.tr, tc = s.tc, wc = (tc + 31) / 32;
    hdt_status_t status = HDT_OK;
    (void)hipGetDevice(&L->device);
#define BUILD_TRY(expr)                                                                                 \
    do {                                                                                                \
        hipError_t _e = (expr);                                                                         \
        if (_e != hipSuccess) {                                                                         \
            status = hdt_fail(_e == hipErrorOutOfMemory ? HDT_ERR_OOM : HDT_ERR_HIP, "%s: %s", #expr, \
                              hipGetErrorString(_e));                                                   \
            goto fail;                                                                                  \
        }                                                                                               \
    } while (0)

    {
        const int nchunks = (n + kChunk - 1) / kChunk, groups = (tr + kWaves - 1) / kWaves;
        Phase1 p = carve_phase1(nullptr, B, n, s.n_slots, tr, nchunks);
        BUILD_TRY(pool_alloc(&L->arena, p.bytes, &L->arena_bytes, st));
        p = carve_phase1((char *)L->arena, B, n, s.n_slots, tr, nchunks);

        // The schedule as far as the host knows it before the device has reported.
        auto adopt = [&](const Phase2 &q, int64_t cap) {
            L->capacity = cap;
            s.kperm = p.kperm;
            L->kperm_ready = windowed != 0;
            L->no_sort = no_sort;
            L->sort_hist = p.hist;
            L->sort_counters = p.counters;
            L->level_copy = p.level_copy;
            L->parent_copy = p.parent_copy;
            s.q_range = p.q_range;
            s.q_cols = q.q_cols;
            s.q_keys = q.q_keys;
            s.q_sub = q.q_sub;
            s.bits_rm = q.bits_rm;
            s.row_flag = p.level_copy;
            L->d_cnt = q.c_cnt;
            L->d_row = q.c_row;
            L->force_dense = force_dense;
            L->device_bytes = (int64_t)(L->arena_bytes + L->arena2_bytes);
        };
        // capacity of the per-tile arrays: exact for the dense baseline, the caller's if given, else a guess raised
        // by what earlier builds needed.  A deferred build cannot be repeated by this call, so it takes what no
        // document can exceed (every query tile listing every key) as far as that stays below 256 MiB.
        const int64_t cap_bound = (int64_t)B * tr * tc;
        int64_t cap = force_dense ? cap_bound : (int64_t)B * ((int64_t)tr * 8 + 64);
        if (!force_dense) {
            std::lock_guard<std::mutex> lk(g_pool_mutex);
            if (g_capacity_hint + g_capacity_hint / 8 > cap) cap = g_capacity_hint + g_capacity_hint / 8;
        }
        if (deferred) {
            const int64_t per_entry = (int64_t)carve_phase2(nullptr, 1024, bm, bn).bytes / 1024 + 1;
            cap = std::max(cap, ((int64_t)256 << 20) / per_entry);
        }
        if (!force_dense && capacity_opt > 0) cap = capacity_opt;
        cap = cap > cap_bound ? cap_bound : cap;
        for (int attempt = 0; attempt < 2; attempt++) {
            if (cap >= (1LL << 31)) {
                status = hdt_fail(HDT_ERR_SHAPE, "hdt_build_layout: %lld candidate tiles", (long long)cap);
                goto fail;
            }
            Phase2 q = carve_phase2(nullptr, cap, bm, bn);
            BUILD_TRY(pool_alloc(&L->arena2, q.bytes, &L->arena2_bytes, st));
            q = carve_phase2((char *)L->arena2, cap, bm, bn);
            uint32_t ticket = 0, ticket_before = 0;
            unsigned long long *report = report_slot(&ticket, &ticket_before);
            if (!report) {
                status = hdt_fail(HDT_ERR_OOM, "hdt_build_layout: no pinned host memory for the build report");
                goto fail;
            }
            // the windowed kernels count in the arena, cleared here; a key-list build counts in a slot that is
            // already clear (if there is none, in the arena as well)
            int32_t *slot_counters = windowed ? nullptr : counter_slot(L->device, ticket);
            if (!slot_counters)
                BUILD_TRY(hipMemsetAsync((char *)L->arena + p.zero_begin, 0, p.zero_end - p.zero_begin, st));
            if (windowed) {
                SortArgs sa{d_level, d_parent, n, s.n_slots, nchunks, no_sort, p.hist, p.kperm, p.slot, p.cmin,
                            p.cmax, p.counters, 1, p.level_copy};
                {
                    HdtTimer t("hdt_layout_sort_count", st);
                    hipLaunchKernelGGL(k_sort_count, dim3((unsigned)B * nchunks), dim3(kThreads), 0, st, sa);
                }
                {
                    HdtTimer t("hdt_layout_sort_scatter", st);
                    hipLaunchKernelGGL(k_sort_scatter, dim3((unsigned)B * nchunks), dim3(kThreads), 0, st, sa);
                }
                CandArgs ca{d_level, d_parent, p.slot, p.cmin, p.cmax, n, bm, bn, tr, tc, wc, force_dense, edges, cap,
                            p.q_range, q.c_row, q.q_cols, p.counters, report, ticket};
                HdtTimer t("hdt_layout_candidates", st);
                hipLaunchKernelGGL(k_candidates, dim3((unsigned)B * groups), dim3(kThreads),
                                   (size_t)kWaves * wc * sizeof(uint32_t), st, ca);
            } else {
                // one kernel from the ids to the finished entries; the global key order is not needed for it
                // and is sorted from the layout's copy of the ids only when someone asks (hdt_layout_export)
                KeyListArgs ka{d_level, d_parent, n, bm, bn, tr, no_sort, edges, cap, p.q_range, q.c_row, q.q_keys, q.q_kpar,
                               q.c_cnt, p.level_copy, p.parent_copy, q.q_sub, q.bits_rm,
                               slot_counters ? slot_counters : p.counters, report, p.report_copy, ticket,
                               slot_counters != nullptr, !deferred};
                L->entries_like = entries_of_one_like(ticket, {batch, n, bm, bn, edges});
                if (both) {
                    both->args[both->n++] = ka;
                    if (both->n == 2) BUILD_TRY(launch_key_lists(both->args, 2, B, st));
                } else {
                    BUILD_TRY(launch_key_lists(&ka, 1, B, st));
                }
            }
            if (windowed) {
                const unsigned grid = (unsigned)(cap < 2048 ? (cap > 0 ? cap : 1) : 2048);
                HdtTimer t("hdt_layout_tile_bitmaps", st);
                hipLaunchKernelGGL(k_tile_bitmaps, dim3(grid), dim3(128), 0, st, d_level, d_parent, p.kperm, q.c_row,
                                   q.q_cols, q.q_keys, p.counters, cap, n, s.n_slots, bm, bn, tr, edges, force_dense,
                                   q.bits_rm, q.c_cnt, q.q_sub);
            }
            BUILD_TRY(hipGetLastError());
            if (deferred || both) {
                // The layout goes out as it is.  What the device reports (through the same word of pinned host
                // memory, and a copy in the layout's own memory) is read by hdt_layout_resolve, when someone asks.
                adopt(q, cap);
                L->n_entries = 0;
                L->entries_needed = -1;
                L->pending = true;
                L->report = report;
                L->report_dev = p.report_copy;
                L->ticket = ticket;
                L->ticket_before = ticket_before;
                *out = L;
                return HDT_OK;
            }
            // The host needs two facts before it can hand the layout out: whether the hierarchy was valid and
            // whether the per-tile arrays were large enough.  The candidate kernel knows both before it writes
            // the lists; it stores them into pinned host memory and the host polls that word instead of
            // draining the stream, so the bitmap kernel and whatever the caller enqueues next keep the GPU busy.
            unsigned long long word = 0;
            if (!wait_for_report(report, ticket, ticket_before, &word)) {
                // no word within the time limit: drain the stream and look again, then read the counters the slow way
                BUILD_TRY(hipStreamSynchronize(st));
                word = __atomic_load_n(report, __ATOMIC_ACQUIRE);
                if ((uint32_t)(word >> 40) != ticket) {
                    if (slot_counters) {
                        BUILD_TRY(hipMemcpy(&word, p.report_copy, sizeof(word), hipMemcpyDeviceToHost));
                        if ((uint32_t)(word >> 40) != ticket) {
                            status = hdt_fail(HDT_ERR_HIP, "hdt_build_layout: the build kernel finished without its report");
                            goto fail;
                        }
                    } else {
                        int32_t cnt[4] = {0, 0, 0, 0};
                        BUILD_TRY(hipMemcpy(cnt, p.counters, sizeof(cnt), hipMemcpyDeviceToHost));
                        word = report_word(ticket, cnt[CNT_ERR], (uint32_t)cnt[CNT_CAND]);  // low word of the combined counter
                    }
                }
            }
            if ((word >> 39) & 1u) {
                BUILD_TRY(hipStreamSynchronize(st));  // the bitmap kernel still reads the arenas
                status = hdt_fail(HDT_ERR_HIERARCHY, "hdt_build_layout: %s", kHierarchyText);
                goto fail;
            }
            const int64_t need = (int64_t)(word & 0xffffffffu);
            {
                std::lock_guard<std::mutex> lk(g_pool_mutex);
                if (!force_dense) g_capacity_hint = need;
            }
            if (need <= cap) {
                adopt(q, cap);
                L->n_entries = need;
                L->entries_needed = need;
                *out = L;
                return HDT_OK;
            }
            BUILD_TRY(hipStreamSynchronize(st));  // the bitmap kernel still writes the arrays about to be replaced
            if (capacity_opt > 0) {
                status = hdt_fail(HDT_ERR_SHAPE, "hdt_build_layout: the schedule needs %lld list entries, opts->capacity is %lld",
                                  (long long)need, (long long)capacity_opt);
                goto fail;
            }
            // the guess was too small: once more with the exact size
            pool_free(L->arena2, L->arena2_bytes, L->device, only_stream(st));
            L->arena2 = nullptr;
            cap = need;
        }
        status = hdt_fail(HDT_ERR_HIP, "hdt_build_layout: candidate count changed between two passes");
    }
fail:
    hdt_layout_release(L, only_stream((hipStream_t)stream));
    L->magic = 0;
    delete L;
    return status;
#undef BUILD_TRY
}
