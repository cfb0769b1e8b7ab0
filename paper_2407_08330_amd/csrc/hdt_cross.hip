// hdt_build_cross_layout: the schedule of decoder cross-attention over a level subset of the encoder's
// positions (Sec. 4.2, FacetSum study: the decoder attends only to the [SEC] anchors, or additionally to
// the [SENT] anchors, or additionally to the regular tokens).
//
// The mask is a rectangle: every decoder row may attend to every visible encoder position (non-pad, level
// in the given set).  In the terms of the attention kernels that is a key list per row tile, the same for
// all row tiles of a sample: the visible positions in document order, tile_n per list entry.  So the
// "gather of the anchor rows" is the gather the attention kernels do anyway, straight into LDS; no compacted
// copy of K and V is made.  The backward pass needs the transposed schedule as well: rows are the encoder
// positions (allowed iff visible), a row tile that holds a visible position lists all decoder rows.
//
// The list entries of a row tile sit at a fixed stride (room for the longest possible list), the unused ones
// are marked empty, and a tile's range covers the ones in use.
//
// The dK/dV pass of the backward tiles the ENCODER rows, and with a few anchors visible nearly every 32-row
// block of them holds one allowed row among 31 idle ones.  When the visible positions are at most a quarter of the
// encoder's, the build therefore makes a second transposed schedule in the index space of the visible positions (row =
// rank among them).  Whether they are, the device finds out: the build makes that schedule or leaves it, in arrays
// that hold a quarter of the encoder's positions, and the host reads the count when a call depends on it, so the build
// waits for nothing (512 x 8192, anchors visible, build, forward and backward: 56.3 -> 43.4 us; a wait for the count and a
// launch for that schedule before).  The dK/dV role of hdt_attn_bwd then reads its K and V rows and writes its dK and dV
// rows through the list of visible positions, and further workgroups of the same launch write the zeros of the rows that
// are not visible (512 x 8192, [SEC] and [SENT] visible: one launch of 24 us where gathering compact copies, the roles and
// scattering the results took 5 + 21 + 24).
//
// With the regular tokens visible the opposite happens: a handful of decoder row tiles each walk a key list of
// more than a hundred entries one after the other, on a few workgroups.  The list of a row tile is the same for
// every row tile of a sample, so cutting it costs nothing but a second table of entry ranges: with the lists cut
// into P pieces the forward (and the dQ role of the backward) see P times the row tiles, piece p of tile I
// covering entries [p * chunk, (p + 1) * chunk) of the tile's list and producing a partial result for the tile's
// rows (O and LSE over its keys; its part of dQ), and a small kernel puts the pieces together in a fixed order
// (O = sum_p w_p O_p with w_p = exp(LSE_p - LSE), LSE = log sum_p exp(LSE_p); dQ = sum_p dQ_p).  The partial
// results live in the caller's workspace (hdt_attn_fwd_ws, hdt_attn_bwd).
#include <string.h>

#include <algorithm>
#include <new>
#include <vector>

#include "hdt_internal.h"
#include "hdt_share.h"

namespace {

constexpr int kSplitEntries = 16;  // lists of this many entries are worth cutting
typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));

__device__ __forceinline__ bool visible(int level, uint32_t level_mask)
{
    return level >= 0 && level < 32 && ((level_mask >> level) & 1u);
}

// One of the schedules of a layout: 0 rows = decoder positions, keys = visible encoder positions; 1 rows = encoder positions
// (allowed iff visible), keys = decoder positions; 2 the same with rows = visible positions by rank.
struct CrossSide {
    int tr, e_max;  // row tiles per sample (2: room for as many), list entries reserved per row tile
    int32_t *q_range, *c_row, *c_cnt, *q_keys;
    uint32_t *q_sub;
    unsigned long long *bits_rm;
};
struct CrossArgs {
    const int32_t *level;  // [B][n_enc]
    uint32_t level_mask;
    int batch, n_enc, n_dec, bm, bn;
    int shares;            // workgroups per sample
    int32_t *sel;          // [B][n_enc] visible positions in document order
    int32_t *rank;         // [B][n_enc] every position's rank among them, or -1
    int32_t *count;        // [B]
    CrossSide side[3];
    int32_t *split_range[3];  // forward schedule: entry ranges with the lists cut, see below; NULL: no list can be long
    HdtReport report;
};

// rows per sample of the compact schedule for c_max visible positions, 0: there is none
__host__ __device__ __forceinline__ int compact_rows(int c_max, int n_enc)
{
    return c_max > 0 && (long long)c_max * 4 <= n_enc ? (c_max + 31) / 32 * 32 : 0;
}

// the lowest n bits (none for n <= 0, all for n >= 32)
__device__ __forceinline__ uint32_t low_bits(int n) { return n >= 32 ? 0xffffffffu : (n <= 0 ? 0u : (1u << n) - 1u); }

// position of the k-th set bit (k counts from 0; there is one)
__device__ __forceinline__ int select_bit(unsigned long long m, int k)
{
    int at = 0;
#pragma unroll
    for (int half = 32; half > 0; half >>= 1) {
        const int low = __popcll((m >> at) & ((1ull << half) - 1ull));
        if (k >= low) {
            k -= low;
            at += half;
        }
    }
    return at;
}

// The list entries of a sample, written a wave each.
struct CrossEntries {
    const unsigned long long *seen;  // [groups] the sample's visible positions, in LDS
    const int *before;               // [groups] visible positions in front of every group of 64, in LDS
    int groups, count;               // count: visible positions of the sample
    int b, lane;

    // the entries x, x + step, ... of side K, whose first one is number `first`; returns where that ended
    template <int K>
    __device__ __forceinline__ int write(const CrossArgs &a, int x, int step, int first) const
    {
        const CrossSide s = a.side[K];
        const int bm = a.bm, bn = a.bn, wpr = bn >> 5, nrb = bm >> 5, nsub = nrb * wpr, div_wpr = 65536 / wpr + 1;  // (of numbers below 16)
        const int n_keys = K == 0 ? count : a.n_dec, last = first + s.tr * s.e_max;
        for (; x < last; x += step) {
            const int I = (x - first) / s.e_max, e = x - first - I * s.e_max;
            const int64_t tile = (int64_t)b * s.tr + I, entry = tile * s.e_max + e;
            // allowed rows of the tile, 32 at a time
            uint32_t rows[4], any_row = 0u;
#pragma unroll
            for (int h = 0; h < 4; h++) {
                const int r0 = I * bm + h * 32;
                const uint32_t m = K == 1 ? reinterpret_cast<const uint32_t *>(seen)[min(r0 >> 5, 2 * groups - 1)]
                                          : low_bits((K == 0 ? a.n_dec : count) - r0);
                rows[h] = (uint32_t)__builtin_amdgcn_readfirstlane((int)(h < nrb && (K != 1 || r0 < 64 * groups) ? m : 0u));
                any_row |= rows[h];
            }
            const int n_ent = K > 0 && any_row == 0u ? 0 : (n_keys + bn - 1) / bn;
            if (e == 0) {
                if (lane < 2) s.q_range[2 * tile + lane] = (int32_t)entry + (lane ? n_ent : 0);
                if (K == 0 && a.split_range[0]) {
#pragma unroll
                    for (int c = 0; c < 3; c++) {
                        const int pieces = 2 << c, chunk = (n_ent + pieces - 1) / pieces;
                        if (lane < pieces) {
                            const int from = min(lane * chunk, n_ent), to = min(from + chunk, n_ent);
                            int32_t *out = a.split_range[c] + 2 * ((size_t)(b * pieces + lane) * s.tr + I);
                            out[0] = (int32_t)entry + from;
                            out[1] = (int32_t)entry + to;
                        }
                    }
                }
            }
            const int n_cols = e < n_ent ? min(n_keys - e * bn, bn) : 0;  // 0: reserved, not in use
            uint32_t any = 0u, all = 0u;
            int n_rows = 0;
#pragma unroll
            for (int rblk = 0; rblk < 4; rblk++) {
                n_rows += __popc(rows[rblk]);
                if (rows[rblk] != 0u) any |= low_bits((n_cols + 31) >> 5) << (rblk * wpr);
                if (rows[rblk] == 0xffffffffu) all |= low_bits(n_cols >> 5) << (rblk * wpr);
            }
            if (lane == 0) {
                s.c_row[entry] = (int32_t)tile;
                s.c_cnt[entry] = n_rows * n_cols;
                s.q_sub[entry] = any | (all << 16);
            }
            if (n_cols == 0) continue;
            // The group of the entry's first key (K = 0): the last one with no more than its rank in front of it, found 64
            // groups at a time; and how many groups from there on hold keys of the entry.
            int g0 = 0, span = 0;
            if (K == 0) {
                for (int n = groups; n > 1;) {
                    const int stride = (n + 63) >> 6, off = lane * stride;
                    const int c = __popcll(__ballot(off < n && before[min(g0 + off, groups - 1)] <= e * bn));
                    g0 += (c - 1) * stride;
                    n = min(stride, n - (c - 1) * stride);
                }
                span = __popcll(__ballot(g0 + lane < groups && before[min(g0 + lane, groups - 1)] < e * bn + n_cols));
            }
            // key slots; one past the last key holds ~f, f = the entry's first key: the row gathered in its place
            for (int c = lane; c < bn; c += 64) {
                const bool ok = c < n_cols;
                int key = ok ? e * bn + c : e * bn;
                if (K == 0) {  // the position of that rank
                    int g = g0;
                    if (span <= 4) {
                        for (int u = 1; u < span; u++) g += before[g0 + u] <= key ? 1 : 0;
                    } else {
                        for (int hi = groups - 1; g < hi;) {
                            const int mid = (g + hi + 1) >> 1;
                            if (before[mid] <= key)
                                g = mid;
                            else
                                hi = mid - 1;
                        }
                    }
                    key = g * 64 + select_bit(seen[g], key - before[g]);
                }
                s.q_keys[entry * bn + c] = ok ? key : ~key;
            }
            // lane masks of the MFMA accumulator registers: sub-block (rblk, cblk), register r: bit l <=> row
            // rblk*32 + l%32, column cblk*32 + (l/32)*4 + 8*(r/4) + r%4
            for (int m = lane; m < nsub * 16; m += 64) {
                const int sb = m >> 4, r = m & 15, rblk = (sb * div_wpr) >> 16, cblk = sb - rblk * wpr;
                const uint32_t row = rblk == 0 ? rows[0] : (rblk == 1 ? rows[1] : (rblk == 2 ? rows[2] : rows[3]));
                const int left = n_cols - cblk * 32 - 8 * (r >> 2) - (r & 3);  // columns from this one on
                s.bits_rm[((size_t)entry * nsub + sb) * 16 + r] = (unsigned long long)(left > 4 ? row : 0u) << 32 | (left > 0 ? row : 0u);
            }
        }
        return x;
    }
};

// The whole build in one launch.  Every workgroup goes over its sample's levels by itself (kBuildBatch groups of 64 positions
// per wave in flight) and keeps a bit per position and the visible positions in front of every group in LDS; from there its
// waves write its share of sel and rank and take the sample's reserved list entries in turn, one each: keys, bitmaps and
// summary, or the "empty" marks.  An entry's rows and columns follow from the counts, its keys are found by rank (a binary
// search over the groups and one inside a group, per key slot).  The first entry of a forward row tile also writes the
// tile's entry ranges with every key list cut into 2, 4 and 8 pieces: row tile p * tr + I of sample b gets entries
// [p * chunk, (p + 1) * chunk) of the list of tile (b, I), chunk = ceil(entries / pieces).  A workgroup knows the number of
// visible positions of its own sample only: the compact schedule's tiles sit at a fixed stride, and are left out where the
// sample alone has too many.  The last of the samples' first workgroups tells the host the largest count.
//
// Bound by latencies: a chain of a load, three barriers and an entry's stores, with a launch around it.  A kernel that
// selected the positions, a workgroup per sample, and one that wrote the entries behind it took longer at all sizes
// (us from start to end, both kernels - this one; [SEC] / all tokens visible): 512 x 64 decoder rows, 1 sample 14.2 / 14.8 - 7.2 / 7.0;
// 8192 x 512, 4 samples 16.2 / 17.4 - 8.5 / 9.1, 16 samples 20.9 / 26.7 - 14.9 / 17.3; 524288 x 512 226 / 255 - 101 / 113; 512 x 512,
// 1024 samples 71 / 76 - 43 / 46; 8192 x 64, 256 samples 44 / 48 - 28 / 39.  512 x 8192 x 4 x 12 heads, anchors visible, build, forward
// and backward: 42.9 -> 39.2 us.  Workgroups for half of the compute units' LDS instead of one each (512): 8.5 -> 12.3 at 8192 x
// 4 samples.  One loop over all sides instead of one per side: 9.1 at 8192 x 4, 60.8 at 8192 x 256, tokens visible.
constexpr int kBuildThreads = kCrossBuildThreads, kBuildBatch = kCrossBuildBatch;
__global__ __launch_bounds__(kBuildThreads) void k_cross_build(CrossArgs a)
{
    constexpr int W = kBuildThreads / 64;
    extern __shared__ unsigned long long s_seen[];  // [groups] visible positions of every group of 64, and behind them
    __shared__ int s_wave[W];
    const int n_enc = a.n_enc, groups = (n_enc + 63) >> 6;
    int *s_before = reinterpret_cast<int *>(s_seen + groups);  // [groups] visible positions in front of the group
    const int b = blockIdx.x / a.shares, w = blockIdx.x % a.shares;
    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int32_t *lv = a.level + (size_t)b * n_enc;
    for (int g0 = wave; g0 < groups; g0 += W * kBuildBatch) {
        int l[kBuildBatch];
#pragma unroll
        for (int u = 0; u < kBuildBatch; u++) {
            const int i = (g0 + u * W) * 64 + lane;
            l[u] = i < n_enc ? lv[i] : -1;
        }
#pragma unroll
        for (int u = 0; u < kBuildBatch; u++) {
            const unsigned long long m = __ballot(visible(l[u], a.level_mask));
            if (lane == 0 && g0 + u * W < groups) s_seen[g0 + u * W] = m;
        }
    }
    __syncthreads();
    // visible positions in front of every group: a thread takes `per` consecutive ones
    const int per = (groups + kBuildThreads - 1) / kBuildThreads, first = min(tid * per, groups), last = min(first + per, groups);
    int mine = 0;
    for (int g = first; g < last; g++) mine += __popcll(s_seen[g]);
    int incl = mine;
#pragma unroll
    for (int d = 1; d < 64; d <<= 1) {
        const int y = __shfl_up(incl, d);
        if (lane >= d) incl += y;
    }
    if (lane == 63) s_wave[wave] = incl;
    __syncthreads();
    int at = incl - mine, count = 0;
#pragma unroll
    for (int k = 0; k < W; k++) {
        at += k < wave ? s_wave[k] : 0;
        count += s_wave[k];
    }
    for (int g = first; g < last; g++) {
        s_before[g] = at;
        at += __popcll(s_seen[g]);
    }
    count = __builtin_amdgcn_readfirstlane(count);
    __syncthreads();

    if (w == 0 && tid == kBuildThreads - 64) {  // (a wave that gets the fewest entries)
        a.count[b] = count;
        if (a.report.word) {
            // the maximum first, and only when it is in place the arrival (returning atomics: each waits for the one before)
            const int before = atomicMax(&a.report.counters[0], count);
            asm volatile("" ::"v"(before));
            if (atomicAdd(&a.report.counters[1], 1) == a.batch - 1) {
                const int most = __hip_atomic_load(&a.report.counters[0], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
                __hip_atomic_store(&a.report.counters[0], 0, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
                __hip_atomic_store(&a.report.counters[1], 0, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
                const unsigned long long word = ((unsigned long long)(a.report.ticket & 0xffffffu) << 40) | (uint32_t)most;
                __hip_atomic_store(a.report.word, word, __ATOMIC_RELEASE, __HIP_MEMORY_SCOPE_SYSTEM);
            }
        }
    }

    {  // sel and rank of this workgroup's share of the groups
        const int share = (groups + a.shares - 1) / a.shares, g1 = min((w + 1) * share, groups);
        int32_t *out = a.sel + (size_t)b * n_enc, *rk = a.rank + (size_t)b * n_enc;
        for (int g = w * share + wave; g < g1; g += W) {
            const unsigned long long seen = s_seen[g];
            const int i = g * 64 + lane, r = s_before[g] + __popcll(seen & ((1ull << lane) - 1ull));
            const bool vis = (seen >> lane) & 1ull;
            if (vis) out[r] = i;
            if (i < n_enc) rk[i] = vis ? r : -1;
        }
    }

    // the list entries, side by side
    int x = wave * a.shares + w;
    const int step = W * a.shares;
    const CrossEntries en{s_seen, s_before, groups, count, b, lane};
    x = en.write<0>(a, x, step, 0);
    x = en.write<1>(a, x, step, a.side[0].tr * a.side[0].e_max);
    if (4ll * count <= n_enc) en.write<2>(a, x, step, a.side[0].tr * a.side[0].e_max + a.side[1].tr * a.side[1].e_max);
}

// O, LSE of row (bh, r) from the partial results of the pieces: o_part [bh][PIECES * rows_pad][D] bf16 (piece p of
// row r at p * rows_pad + r), lse_part [bh][PIECES * rows_pad].  One thread per 8 columns; all loads of a thread are
// issued before the first is used.
template <int D, int PIECES>
__global__ __launch_bounds__(256) void k_cross_combine_fwd(const u32x4 *__restrict__ o_part, const float *__restrict__ lse_part,
                                                            u32x4 *__restrict__ o, float *__restrict__ lse, int n_rows,
                                                            int rows_pad, long long total)
{
    constexpr int CPR = D / 8;
    const long long t = (long long)blockIdx.x * 256 + threadIdx.x;
    if (t >= total) return;
    const int c = (int)(t % CPR);
    const long long row = t / CPR;  // bh * n_rows + r
    const int r = (int)(row % n_rows);
    const long long bh = row / n_rows;
    const size_t prow = (size_t)bh * PIECES * rows_pad + r;
    float l[PIECES];
    u32x4 x[PIECES];
#pragma unroll
    for (int p = 0; p < PIECES; p++) {
        l[p] = lse_part[prow + (size_t)p * rows_pad];
        x[p] = o_part[(prow + (size_t)p * rows_pad) * CPR + c];
    }
    float m = -INFINITY;
#pragma unroll
    for (int p = 0; p < PIECES; p++) m = fmaxf(m, l[p]);
    float acc[8] = {0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f}, z = 0.f;
#pragma unroll
    for (int p = 0; p < PIECES; p++) {
        // a piece without keys has LSE = -inf and rows of zeros: weight 0
        const float w = (m == -INFINITY || l[p] == -INFINITY) ? 0.f : __expf(l[p] - m);
        z += w;
#pragma unroll
        for (int e = 0; e < 4; e++) {
            acc[2 * e] += w * __uint_as_float(x[p][e] << 16);
            acc[2 * e + 1] += w * __uint_as_float(x[p][e] & 0xffff0000u);
        }
    }
    const float inv = z > 0.f ? 1.f / z : 0.f;
    u32x4 y;
#pragma unroll
    for (int e = 0; e < 4; e++) {
        const __bf16 lo = (__bf16)(acc[2 * e] * inv), hi = (__bf16)(acc[2 * e + 1] * inv);
        y[e] = (uint32_t)__builtin_bit_cast(unsigned short, lo) | ((uint32_t)__builtin_bit_cast(unsigned short, hi) << 16);
    }
    o[row * CPR + c] = y;
    if (c == 0) lse[row] = z > 0.f ? m + __logf(z) : -INFINITY;
}

// dQ of row (bh, r) = the sum of the pieces' parts, in piece order
template <int D, int PIECES>
__global__ __launch_bounds__(256) void k_cross_sum_dq(const u32x4 *__restrict__ dq_part, u32x4 *__restrict__ dq, int n_rows,
                                                       int rows_pad, long long total)
{
    constexpr int CPR = D / 8;
    const long long t = (long long)blockIdx.x * 256 + threadIdx.x;
    if (t >= total) return;
    const int c = (int)(t % CPR);
    const long long row = t / CPR;
    const int r = (int)(row % n_rows);
    const long long bh = row / n_rows;
    const size_t prow = (size_t)bh * PIECES * rows_pad + r;
    u32x4 x[PIECES];
#pragma unroll
    for (int p = 0; p < PIECES; p++) x[p] = dq_part[(prow + (size_t)p * rows_pad) * CPR + c];
    float acc[8] = {0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int p = 0; p < PIECES; p++) {
#pragma unroll
        for (int e = 0; e < 4; e++) {
            acc[2 * e] += __uint_as_float(x[p][e] << 16);
            acc[2 * e + 1] += __uint_as_float(x[p][e] & 0xffff0000u);
        }
    }
    u32x4 y;
#pragma unroll
    for (int e = 0; e < 4; e++) {
        const __bf16 lo = (__bf16)acc[2 * e], hi = (__bf16)acc[2 * e + 1];
        y[e] = (uint32_t)__builtin_bit_cast(unsigned short, lo) | ((uint32_t)__builtin_bit_cast(unsigned short, hi) << 16);
    }
    dq[row * CPR + c] = y;
}

struct CrossBuffers {
    int32_t *split_range[3];                // first arena, forward schedule only: entry ranges with the lists cut in 2, 4, 8
    int32_t *sel, *rank, *count, *q_range;  // first arena
    int32_t *c_row, *c_cnt, *q_keys;  // second arena
    uint32_t *q_sub;
    unsigned long long *bits_rm;
    size_t bytes1, bytes2;
};

template <typename T>
T *carve(char *base, size_t &off, size_t count)
{
    T *p = base ? reinterpret_cast<T *>(base + off) : nullptr;
    off += (count * sizeof(T) + 255) & ~(size_t)255;
    return p;
}

CrossBuffers carve_cross(char *a1, char *a2, int B, int n_enc, int tr, int64_t entries, int bm, int bn, bool with_sel)
{
    CrossBuffers c{};
    size_t o1 = 0, o2 = 0;
    if (with_sel) {
        c.sel = carve<int32_t>(a1, o1, (size_t)B * n_enc);
        c.rank = carve<int32_t>(a1, o1, (size_t)B * n_enc);
        c.count = carve<int32_t>(a1, o1, (size_t)B);
        for (int k = 0; k < 3; k++) c.split_range[k] = carve<int32_t>(a1, o1, (size_t)B * tr * (2 << k) * 2);
    }
    c.q_range = carve<int32_t>(a1, o1, (size_t)B * tr * 2);
    const size_t n = (size_t)entries;
    c.c_row = carve<int32_t>(a2, o2, n);
    c.c_cnt = carve<int32_t>(a2, o2, n);
    c.q_sub = carve<uint32_t>(a2, o2, n);
    c.q_keys = carve<int32_t>(a2, o2, n * (size_t)bn);
    c.bits_rm = carve<unsigned long long>(a2, o2, n * (size_t)(bm / 32) * (bn / 32) * 16);
    c.bytes1 = o1;
    c.bytes2 = o2;
    return c;
}

hdt_layout_t *new_layout(int batch, int n_rows, int n_kv, int bm, int bn)
{
    hdt_layout_t *L = new (std::nothrow) hdt_layout_t();
    if (!L) return nullptr;
    L->magic = HDT_LAYOUT_MAGIC;
    L->arena = L->arena2 = nullptr;
    L->arena_bytes = L->arena2_bytes = 0;
    L->capacity = 0;
    L->d_cnt = L->d_row = nullptr;
    L->n_entries = 0;
    L->stats_ready = false;
    L->kperm_ready = true;
    L->no_sort = 0;
    L->sort_hist = L->sort_counters = nullptr;
    L->level_copy = L->parent_copy = nullptr;
    L->force_dense = 0;
    L->windowed = 0;
    L->edges = 0;
    L->cross = 1;
    L->transposed = nullptr;
    L->compact = L->compact_built = nullptr;
    L->n_compact = 0;
    L->pending = false;
    L->build_status = HDT_OK;
    for (auto &r : L->cross_split_range) r = nullptr;
    L->cross_entries_max = 0;
    L->device_bytes = 0;
    L->device = 0;
    (void)hipGetDevice(&L->device);
    HdtSchedule &s = L->s;
    memset(&s, 0, sizeof(s));
    s.batch = batch;
    s.n_pos = n_rows;
    s.n_kv = n_kv;
    s.bm = bm;
    s.bn = bn;
    s.wpr = bn / 32;
    s.tr = (n_rows + bm - 1) / bm;
    s.tc = (n_kv + bn - 1) / bn;
    s.n_slots = s.tc * bn;
    s.n_own = n_rows;
    s.tr_own = s.tr;
    L->h_stats.assign((size_t)batch * 2, 0);
    return L;
}

// the finished arrays become the layout's schedule
void adopt(hdt_layout_t *l, const CrossBuffers &c, int64_t n)
{
    HdtSchedule &s = l->s;
    s.q_range = c.q_range;
    s.q_keys = c.q_keys;
    s.q_sub = c.q_sub;
    s.bits_rm = c.bits_rm;
    s.q_cols = nullptr;
    s.kperm = nullptr;
    l->d_cnt = c.c_cnt;
    l->d_row = c.c_row;
    l->n_entries = n;
    l->capacity = n;
    l->device_bytes = (int64_t)(c.bytes1 + c.bytes2);
    if (n == 0) l->stats_ready = true;
}

}  // namespace

extern "C" __attribute__((visibility("default"))) hdt_status_t hdt_build_cross_layout(
    const int32_t *d_level_enc, int32_t batch, int32_t n_enc, int32_t n_dec, uint32_t level_mask,
    const hdt_layout_opts_t *opts, void *stream, hdt_layout_t **out)
{
    if (!out) return hdt_fail(HDT_ERR_INVALID_ARG, "hdt_build_cross_layout: out is NULL");
    *out = nullptr;
    if (batch < 0 || n_enc < 0 || n_dec < 0) return hdt_fail(HDT_ERR_INVALID_ARG, "hdt_build_cross_layout: negative size");
    if (n_enc > (1 << 19) || n_dec > (1 << 19))
        return hdt_fail(HDT_ERR_SHAPE, "hdt_build_cross_layout: n_enc %d or n_dec %d > 2^19", n_enc, n_dec);
    int bm = 128, bn = 64;
    if (opts) {
        if (opts->tile_m) bm = opts->tile_m;
        if (opts->tile_n) bn = opts->tile_n;
        if (opts->force_dense || opts->no_sort || opts->windowed || opts->edges || opts->deferred || opts->capacity)
            return hdt_fail(HDT_ERR_UNSUPPORTED, "hdt_build_cross_layout: only the tile shape can be chosen");
    }
    if (bm < 32 || bm > 128 || bm % 32 || bn < 32 || bn > 128 || bn % 32)
        return hdt_fail(HDT_ERR_UNSUPPORTED, "hdt_build_cross_layout: tile %dx%d (each side: 32, 64, 96 or 128)", bm, bn);
    if (batch > 0 && (n_enc == 0 || n_dec == 0))
        return hdt_fail(HDT_ERR_SHAPE, "hdt_build_cross_layout: n_enc = %d, n_dec = %d (both sides need rows)", n_enc, n_dec);
    const bool empty = batch == 0;
    if (!empty && !d_level_enc) return hdt_fail(HDT_ERR_INVALID_ARG, "hdt_build_cross_layout: NULL level array");

    hdt_layout_t *L = new_layout(batch, n_dec, n_enc, bm, bn);
    hdt_layout_t *T = L ? new_layout(batch, n_enc, n_dec, bm, bn) : nullptr;
    if (!L || !T) {
        delete L;
        return hdt_fail(HDT_ERR_OOM, "hdt_build_cross_layout: host allocation failed");
    }
    L->transposed = T;
    L->cross_level_mask = T->cross_level_mask = level_mask;
    hdt_layout_t *Tc = nullptr;  // the compact schedule, for as many rows as it can have
    HdtReport report{};
    bool reported = false;
    hdt_status_t status = HDT_OK;
    hipStream_t st = (hipStream_t)stream;
    L->streams.add(st);
    hdt_note_build_stream(st);
    HdtUsers build_only;  // what the buffers of a failed build have been touched by
    build_only.lazy.add(st);
    const int e_fwd = (n_enc + bn - 1) / bn, e_tr = (n_dec + bn - 1) / bn, n_c = compact_rows(n_enc / 4, n_enc);
    const int64_t ent_fwd = (int64_t)batch * L->s.tr * e_fwd, ent_tr = (int64_t)batch * T->s.tr * e_tr;
    const int64_t ent_c = (int64_t)batch * ((n_c + bm - 1) / bm) * e_tr;
    if (ent_fwd >= (1LL << 31) || ent_tr >= (1LL << 31)) {
        status = hdt_fail(HDT_ERR_SHAPE, "hdt_build_cross_layout: %lld list entries", (long long)(ent_fwd > ent_tr ? ent_fwd : ent_tr));
        goto fail;
    }
#define CROSS_TRY(expr)                                                                                \
    do {                                                                                               \
        hipError_t _e = (expr);                                                                        \
        if (_e != hipSuccess) {                                                                        \
            status = hdt_fail(_e == hipErrorOutOfMemory ? HDT_ERR_OOM : HDT_ERR_HIP, "%s: %s", #expr, \
                              hipGetErrorString(_e));                                                  \
            goto fail;                                                                                 \
        }                                                                                              \
    } while (0)
    if (n_c > 0 && !empty) {
        Tc = new_layout(batch, n_c, n_dec, bm, bn);
        if (!Tc) {
            status = hdt_fail(HDT_ERR_OOM, "hdt_build_cross_layout: host allocation failed");
            goto fail;
        }
        Tc->cross_level_mask = level_mask;
    }
    {
        struct {
            hdt_layout_t *l;
            int64_t n;
            CrossBuffers c;
        } all[3] = {{L, empty ? 0 : ent_fwd, {}}, {T, empty ? 0 : ent_tr, {}}, {Tc, empty ? 0 : ent_c, {}}};
        // The schedules share the two buffers of L, which goes through the cache of buffers with two of them: with two per
        // schedule, the cache's 16 held two layouts at a time, and a third one destroyed gave buffers back to the system.
        size_t bytes1 = 0, bytes2 = 0;
        for (auto &x : all) {
            if (!x.l) continue;
            x.c = carve_cross(nullptr, nullptr, batch, n_enc, x.l->s.tr, x.n, bm, bn, x.l == L);
            bytes1 += x.c.bytes1;
            bytes2 += x.c.bytes2;
        }
        CROSS_TRY(hdt_pool_alloc(&L->arena, bytes1 + 256, &L->arena_bytes, st));
        CROSS_TRY(hdt_pool_alloc(&L->arena2, bytes2 + 256, &L->arena2_bytes, st));
        char *at1 = (char *)L->arena, *at2 = (char *)L->arena2;
        for (auto &x : all) {
            if (!x.l) continue;
            x.c = carve_cross(at1, at2, batch, n_enc, x.l->s.tr, x.n, bm, bn, x.l == L);
            at1 += x.c.bytes1;
            at2 += x.c.bytes2;
            adopt(x.l, x.c, x.n);
        }
        L->device_bytes = (int64_t)(L->arena_bytes + L->arena2_bytes);
        const CrossBuffers &f = all[0].c;
        T->s.row_flag = f.rank;  // encoder rows that are not visible (pads among them) may hold anything
        if (Tc) {
            Tc->s.own_index = f.sel;
            Tc->s.own_count = f.count;
            Tc->s.own_rank = f.rank;
            Tc->s.own_stride = n_enc;
            Tc->s.own_tiles = Tc->s.tr;
        }
        if (!empty) {
            // (a stream that is being captured runs nothing now: no report would come)
            hipStreamCaptureStatus capture = hipStreamCaptureStatusNone;
            reported = hipStreamIsCapturing(st, &capture) == hipSuccess && capture == hipStreamCaptureStatusNone &&
                       hdt_report_open(L->device, &report);
            if (!reported) report = HdtReport{};
            CrossArgs args{d_level_enc, level_mask, batch, n_enc, n_dec, bm, bn, 1, f.sel, f.rank, f.count, {}, {}, report};
            int64_t per_sample = 0;  // list entries
            for (int k = 0; k < 3; k++) {
                const CrossBuffers &c = all[k].c;
                if (!all[k].l) continue;
                args.side[k] = CrossSide{all[k].l->s.tr, k == 0 ? e_fwd : e_tr, c.q_range, c.c_row, c.c_cnt, c.q_keys, c.q_sub, c.bits_rm};
                per_sample += all[k].n / batch;
            }
            if (e_fwd >= kSplitEntries)
                for (int k = 0; k < 3; k++) L->cross_split_range[k] = args.split_range[k] = f.split_range[k];
            args.shares = cross_build_shares(batch, n_enc, per_sample);
            const size_t lds = (size_t)((n_enc + 63) / 64) * (sizeof(unsigned long long) + sizeof(int));
            if (lds > 60 * 1024)  // with the static array: beyond the 64 KB a launch gets by default
                CROSS_TRY(hipFuncSetAttribute((const void *)k_cross_build, hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds));
            {
                HdtTimer tm("hdt_cross_build", st);
                hipLaunchKernelGGL(k_cross_build, dim3((unsigned)batch * args.shares), dim3(kBuildThreads), lds, st, args);
            }
            CROSS_TRY(hipGetLastError());
            L->compact_built = Tc;  // owned by L from here on
            if (reported) {
                L->own_report = report;
                L->report = report.word;
                L->ticket = report.ticket;
                L->pending.store(true, std::memory_order_release);
            } else {  // no report: the counts are read back
                std::vector<int32_t> h_count((size_t)batch, 0);
                L->compact_built = nullptr;
                CROSS_TRY(hipMemcpyAsync(h_count.data(), f.count, sizeof(int32_t) * batch, hipMemcpyDeviceToHost, st));
                CROSS_TRY(hipStreamSynchronize(st));
                L->compact_built = Tc;
                hdt_cross_record(L, *std::max_element(h_count.begin(), h_count.end()));
            }
        }
        *out = L;
        return HDT_OK;
    }
fail:
    if (reported) hdt_report_close(L->device, report);
    if (Tc) {
        Tc->magic = 0;
        delete Tc;
    }
    T->magic = 0;
    delete T;
    L->transposed = nullptr;
    hdt_layout_release(L, build_only);
    L->magic = 0;
    delete L;
    return status;
#undef CROSS_TRY
}

void hdt_cross_record(const hdt_layout_t *l, int c_max)
{
    l->cross_entries_max = (c_max + l->s.bn - 1) / l->s.bn;
    const int n_c = compact_rows(c_max, l->s.n_kv);
    hdt_layout_t *c = l->compact_built;
    if (n_c == 0 || !c) return;
    // The rows there are, not those there was room for.  The tiles keep their places: q_range and c_row go by own_tiles per sample, not
    // by tr, and the list entries stay the reserved ones, spread over all of them.
    HdtSchedule &s = c->s;
    s.n_pos = s.n_own = n_c;
    s.tr = s.tr_own = (n_c + s.bm - 1) / s.bm;
    l->n_compact = n_c;
    l->compact = c;
}

static size_t compact_tensor_bytes(const hdt_layout_t *l, int heads, int head_dim, int elem_bytes)
{
    const size_t n = (size_t)l->s.batch * (size_t)heads * (size_t)l->n_compact * (size_t)head_dim * (size_t)elem_bytes;
    return (n + 255) & ~(size_t)255;
}

// Room for copies of the visible rows of K, V, dK and dV: what hdt_attn_bwd_workspace_bytes has always asked for a layout
// with a compact schedule, and the size the limit of hdt_attn_bwd_no_alloc is counted in.
size_t hdt_cross_compact_workspace_bytes(const hdt_layout_t *l, int heads, int head_dim, int elem_bytes)
{
    return l->compact ? 4 * compact_tensor_bytes(l, heads, head_dim, elem_bytes) : 0;
}

// ---- key lists cut into pieces ---------------------------------------------------------------------------
// How many pieces for this many heads: enough row tiles for a thousand workgroups (measured on 512 decoder rows x
// 8192 keys x 48 heads: forward kernel 201 us uncut, 91 in 4 pieces, 85 in 8, 82 in 16 where combining the pieces
// costs more than that gains), pieces of at least 8 entries, and none at all where the transposed schedule tiles the
// visible positions only (few keys, short lists).
int hdt_cross_pieces(const hdt_layout_t *l, int heads)
{
    if (!l->cross || l->compact || l->cross_entries_max < kSplitEntries || heads <= 0) return 1;
    const long long tiles = (long long)l->s.batch * l->s.tr * heads;
    int pieces = 1;
    while (pieces < 8 && tiles * pieces < 1024 && l->cross_entries_max / (2 * pieces) >= 8) pieces *= 2;
    return pieces;
}

static size_t align256(size_t n) { return (n + 255) & ~(size_t)255; }

// the schedule with the lists cut: every row tile once per piece, partial results of rows_pad rows per piece
static HdtSchedule split_schedule(const hdt_layout_t *l, int pieces)
{
    HdtSchedule s = l->s;
    const int k = pieces == 2 ? 0 : (pieces == 4 ? 1 : 2);
    s.q_range = l->cross_split_range[k];
    s.tr = pieces * l->s.tr;
    s.n_pos = pieces * l->s.tr * l->s.bm;
    return s;  // n_own, tr_own keep the real rows
}

size_t hdt_cross_fwd_workspace_bytes(const hdt_layout_t *l, int heads, int head_dim)
{
    const int pieces = hdt_cross_pieces(l, heads);
    if (pieces == 1) return 0;
    const size_t rows = (size_t)l->s.batch * heads * pieces * l->s.tr * l->s.bm;
    return align256(rows * head_dim * 2) + align256(rows * sizeof(float));
}

size_t hdt_cross_dq_workspace_bytes(const hdt_layout_t *l, int heads, int head_dim)
{
    const int pieces = hdt_cross_pieces(l, heads);
    if (pieces == 1) return 0;
    return align256((size_t)l->s.batch * heads * pieces * l->s.tr * l->s.bm * head_dim * 2);
}

hdt_status_t hdt_cross_fwd_split(const hdt_layout_t *l, const void *q, const void *k, const void *v, void *o, float *lse,
                                 int heads, int head_dim, float scale, void *workspace, hipStream_t st)
{
    const int pieces = hdt_cross_pieces(l, heads);
    const HdtSchedule s = split_schedule(l, pieces);
    const size_t rows = (size_t)s.batch * heads * s.n_pos;
    char *w = static_cast<char *>(workspace);
    void *o_part = w;
    float *lse_part = reinterpret_cast<float *>(w + align256(rows * head_dim * 2));
    if (hdt_status_t status = hdt_launch_fwd_bf16(s, q, k, v, o_part, lse_part, heads, head_dim, scale, st)) return status;
    const int rows_pad = l->s.tr * l->s.bm;
    const long long total = (long long)l->s.batch * heads * l->s.n_pos * (head_dim / 8);
    HdtTimer tm("hdt_cross_combine_fwd", st);
    const dim3 grid((unsigned)((total + 255) / 256)), block(256);
#define COMBINE(DD, PP)                                                                                                  \
    hipLaunchKernelGGL((k_cross_combine_fwd<DD, PP>), grid, block, 0, st, (const u32x4 *)o_part, lse_part, (u32x4 *)o, lse, \
                       l->s.n_pos, rows_pad, total)
    if (head_dim == 64) {
        if (pieces == 2) COMBINE(64, 2); else if (pieces == 4) COMBINE(64, 4); else COMBINE(64, 8);
    } else {
        if (pieces == 2) COMBINE(128, 2); else if (pieces == 4) COMBINE(128, 4); else COMBINE(128, 8);
    }
#undef COMBINE
    HDT_HIP_TRY(hipGetLastError());
    return HDT_OK;
}

// Workspace: D of the decoder rows, then the pieces' parts of dQ.
hdt_status_t hdt_cross_bwd_split(const hdt_layout_t *l, const void *q, const void *k, const void *v, const void *o,
                                 const float *lse, const void *d_o, void *dq, void *dk, void *dv, int heads,
                                 int head_dim, float scale, void *workspace, hipStream_t st)
{
    const int pieces = hdt_cross_pieces(l, heads);
    const HdtSchedule s = split_schedule(l, pieces);
    const size_t d_bytes = hdt_bwd_row_scalars_bytes((size_t)l->s.batch * heads * (size_t)l->s.n_pos);
    char *w = static_cast<char *>(workspace);
    float *delta = reinterpret_cast<float *>(w);
    void *dq_part = w + d_bytes;
    // D is computed over the real rows (the D pass takes its row count from the first schedule's n_own)
    if (hdt_status_t status = hdt_launch_bwd_bf16(s, l->transposed->s, q, k, v, o, lse, d_o, dq_part, dk, dv, heads, head_dim,
                                                  scale, delta, HdtLists{true, -1}, st))
        return status;
    const int rows_pad = l->s.tr * l->s.bm;
    const long long total = (long long)l->s.batch * heads * l->s.n_pos * (head_dim / 8);
    HdtTimer tm("hdt_cross_sum_dq", st);
    const dim3 grid((unsigned)((total + 255) / 256)), block(256);
#define SUM_DQ(DD, PP) \
    hipLaunchKernelGGL((k_cross_sum_dq<DD, PP>), grid, block, 0, st, (const u32x4 *)dq_part, (u32x4 *)dq, l->s.n_pos, rows_pad, total)
    if (head_dim == 64) {
        if (pieces == 2) SUM_DQ(64, 2); else if (pieces == 4) SUM_DQ(64, 4); else SUM_DQ(64, 8);
    } else {
        if (pieces == 2) SUM_DQ(128, 2); else if (pieces == 4) SUM_DQ(128, 4); else SUM_DQ(128, 8);
    }
#undef SUM_DQ
    HDT_HIP_TRY(hipGetLastError());
    return HDT_OK;
}
