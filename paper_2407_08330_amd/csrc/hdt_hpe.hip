// Hierarchical positional encoding (paper Sec. 3.2 "Hierarchical Positional Encoding", Eq. pos_enc,
// Fig. 3 caption): every position carries one index per hierarchy level, each index goes through the
// standard sinusoidal functions, and the encodings of the levels are summed and added to the embeddings.
//
//   hdt_parents_from_levels  levels of a document in the paper's layout (anchors in front) -> parent ids
//   hdt_index_vectors   level/parent ids -> index vectors p[B][N][L] (1-based ordinal among the siblings
//                       of the position's ancestor-or-self at each level, 0 where there is none)
//   hdt_hpe_table       the sinusoidal table T[v][c] = sin / cos (w_k v), w_k = 10000^(-2k/d_model)
//   hdt_hpe_add         x[b][n][c] += sum_l T[p^l][c]
//
// The indices of a document are small integers (ordinal of a section, of a sentence in its section, of a
// token in its sentence), so the encoding of a position is the sum of L rows of a small table that stays in
// L2: the add is then bound by reading and writing x once, not by 2*L*d_model sine evaluations per position.
// Indices beyond the table are evaluated directly.
#include <math.h>

#include <algorithm>

#include "hdt_internal.h"
#include "hdt_share.h"

namespace {

constexpr int kOrdWaves = kOrdThreads / 64;

// Both kernels below give a workgroup a contiguous share of a sample's positions, which it takes 1024 at a time; what it
// has to know about the positions in front of its share it finds by reading them, all waves together.  That reads up
// to `shares` / 2 times the sample's ids (a few hundred KB, out of L2), and takes less time than carrying the state from
// chunk to chunk in one workgroup per sample, whose chunks follow one another (8192 positions x 4 samples: parents
// 31 -> 6.7 us, ordinals 20.8 -> 8.2, now 6.3; 32768 positions, 1 sample: 126 -> 11 and 78 -> 18), as long as the workgroups of all
// samples are on the chip at the same time, one per compute unit: further ones only wait, and read more.  8192 positions,
// us for parents / index vectors, one workgroup per sample - a share per 1024 positions - at most 256 workgroups:
// 64 samples 31 / 29 - 12 / 22 - 8.6 / 16; 256 samples 32 / 47 - 46 / 80 - 20 / 41; 512 samples 61 / 89 - 91 / 152 - 37 / 63.
// (hdt_share.h)

// ---- parents of a document laid out with its anchors in front (pre-order) ---------------------------
// parent[i] = the nearest earlier position whose level is level[i] - 1 (none: -1).  Inside a wave by ballots, across
// the waves of a chunk and in front of it through LDS (the last position of every level).  The positions in front of a
// share are read backwards until every level that somebody still misses has been seen; the first 8192 of them are requested
// with the share itself (event-bracketed us, where an empty kernel takes 6.1: 8192 positions x 4 samples 8.6 -> 8.1, 32768 x 1
// 13.2 -> 11.2; batches with one share per sample, without the search, 8192 x 512 40.0 -> 38.3, 512 x 1024 13.7 -> 13.0).
// With one share `parent` may be `level`: a position's level is read by its own thread alone, before its parent is written.
// SPREAD: several shares per sample; otherwise nothing stands in front of a share, and nothing is looked for there.
template <bool SPREAD>
__global__ __launch_bounds__(kOrdThreads) void k_parents_from_levels(const int32_t *level, int n, int shares, int32_t *parent)
{
    __shared__ int s_last[kOrdWaves][32];  // last position of each level in each wave of the chunk (-1: none)
    __shared__ int s_carry[32];            // last position of each level in front of the chunk
    __shared__ unsigned s_missing;         // levels that positions of the chunk look for and the share has not seen
    const int tid = threadIdx.x, wave = tid >> 6, lane = tid & 63;
    const size_t o = (size_t)(blockIdx.x / shares) * n;
    const HpeShare share = hpe_share(blockIdx.x % shares, n, shares);
    if (share.empty()) return;
    unsigned searched = 0u;  // levels looked for in front of the share
    // the kBack * 1024 positions that end at `end`
    auto load_back = [&](int end, int (&l)[kBack]) {
#pragma unroll
        for (int u = 0; u < kBack; u++) {
            const int j = hpe_position_in_front(share, end, u, tid);
            l[u] = j >= 0 ? level[o + j] : -1;
        }
    };
    // the first chunk and the positions in front of the share are requested together, whoever turns out to need the latter
    const int first_level = share.first + tid < share.last ? level[o + share.first + tid] : -1;
    int back[kBack];
    if (SPREAD && share.first > 0) load_back(share.first, back);
    if (tid < 32) s_carry[tid] = -1;
    if (tid == 0) s_missing = 0u;
    __syncthreads();
    for (int c0 = share.first; c0 < share.last; c0 += kOrdThreads) {
        const int i = c0 + tid;
        int lv = c0 == share.first ? first_level : (i < share.last ? level[o + i] : -1);
        if (lv < 0 || lv >= 32) lv = -1;
        // level by level of those in this wave: its last position (kept by lane = level), and for the positions one
        // level down the nearest earlier one
        int mine = -1, par = -1;
        unsigned long long todo = __ballot(lv >= 0);
        while (todo) {
            const int t = __builtin_amdgcn_readlane(lv, __ffsll((long long)todo) - 1);
            const unsigned long long m = __ballot(lv == t), before = m & ((1ull << lane) - 1ull);
            if (lane == t) mine = c0 + wave * 64 + 63 - __builtin_clzll(m);
            if (lv == t + 1 && before) par = c0 + wave * 64 + 63 - __builtin_clzll(before);
            todo &= ~m;
        }
        if (lane < 32) s_last[wave][lane] = mine;
        __syncthreads();
        if (lv > 0)  // not in this wave: earlier waves of the chunk, then earlier chunks of the share
            for (int w = wave - 1; w >= 0 && par < 0; w--) par = s_last[w][lv - 1];
        const bool miss = lv > 0 && par < 0;
        if (SPREAD) {
            if (miss && s_carry[lv - 1] < 0) atomicOr(&s_missing, 1u << (lv - 1));
            __syncthreads();
            unsigned missing = s_missing & ~searched;
            searched |= missing;
            for (int end = share.first; missing && end > 0; end -= kBack * kOrdThreads) {
                if (end < share.first || c0 > share.first) load_back(end, back);
#pragma unroll
                for (int u = 0; u < kBack; u++) {
                    const int j = hpe_position_in_front(share, end, u, tid);
                    if (back[u] >= 0 && back[u] < 32 && ((missing >> back[u]) & 1u) && s_carry[back[u]] < j) atomicMax(&s_carry[back[u]], j);
                }
                __syncthreads();
                missing &= ~(unsigned)__ballot(lane < 32 && s_carry[lane & 31] >= 0);
                __syncthreads();  // everybody has looked before the next round writes
            }
        }
        if (miss) par = s_carry[lv - 1];
        if (i < share.last) parent[o + i] = par;
        __syncthreads();
        if (tid < 32) {
            for (int w = kOrdWaves - 1; w >= 0; w--)
                if (s_last[w][tid] >= 0) {
                    s_carry[tid] = s_last[w][tid];
                    break;
                }
        }
        if (SPREAD && tid == 0) s_missing = 0u;
        __syncthreads();
    }
}

// ---- ordinal of every position among its siblings (same parent), in document order ---------------
// Consecutive positions with the same parent form a run (the tokens of a sentence, for one); a run ends at the latest
// with the 64 positions a wave holds.  A position's ordinal is
//   1 + (siblings in front of the chunk: a counter per parent in LDS, filled from the positions in front of the share
//        and then chunk by chunk)
//     + (siblings in earlier runs of the chunk: a sum over the earlier runs, shared by kOrdSplit lanes)
//     + (its offset inside its run).
// Roots (parent -1) count as children of one virtual parent, n.  Pads and positions past the share are a group of their
// own (-1), which only serves to end the runs before them.  The counters cover a window of the parents at a time: one
// window up to kOrdWindow positions, as many LDS words as that takes; beyond, the windows in which parents of the share
// lie, each of which reads the positions in front of the share again.  In a document these are the share's own window and
// the first one; parents anywhere are in all of them, and the time would grow with the square of the length.  So with
// several windows the kernel is used up to kMaxWindowed positions and with at least kMinShares shares (16 samples), and
// k_sibling_ordinals_chain, whose time is linear whatever the parents are, otherwise.  us for the index vectors of
// documents / of runs of 64 siblings with parents anywhere, chain - windows: 70001 x 1 sample 176 / 135 - 74 / 95,
// 131072 x 1 304 / 217 - 96 / 177, 131072 x 16 331 / 396 - 196 / 461; beyond the lines 131072 x 32 346 / 591 - 257 / 693,
// 524288 x 1 1203 / 809 - 520 / 2389.
constexpr int kOrdSplit = 16, kOrdWindow = 33 * 1024;
constexpr int kMinShares = 16, kMaxWindowed = 1 << 17;

__device__ __forceinline__ int ord_group(int level, int parent, int n)
{
    return level < 0 ? -1 : ((parent >= 0 && parent < n) ? parent : n);
}
// whether this lane's position starts a run, and the run's length (1 .. 64)
__device__ __forceinline__ bool run_head(int grp, int lane, int *len)
{
    const int before = __shfl_up(grp, 1);
    const bool head = lane == 0 || before != grp;
    const unsigned long long heads = __ballot(head), rest = lane == 63 ? 0ull : heads >> (lane + 1);
    *len = rest ? __ffsll((long long)rest) : 64 - lane;
    return head;
}

// SPREAD: several shares per sample; otherwise nothing stands in front of a share.
template <bool SPREAD>
__global__ __launch_bounds__(kOrdThreads, SPREAD ? 4 : 8) void k_sibling_ordinals(const int32_t *__restrict__ level,
                                                                   const int32_t *__restrict__ parent, int n, int shares,
                                                                   int32_t *__restrict__ ord)  // [B][n]
{
    extern __shared__ int s_count[];  // children seen so far of the parents w0 .. w0 + window - 1
    __shared__ int s_run_grp[kOrdThreads], s_run_len[kOrdThreads], s_run_base[kOrdThreads];
    __shared__ int s_wave_runs[kOrdWaves];
    __shared__ unsigned s_windows;  // the windows in which groups of the share lie
    const int tid = threadIdx.x, wave = tid >> 6, lane = tid & 63;
    const size_t o = (size_t)(blockIdx.x / shares) * n;
    const HpeShare share = hpe_share(blockIdx.x % shares, n, shares);
    if (share.empty()) return;
    const int window = min(n + 1, kOrdWindow);
    // The first positions in front of the share, and its own first chunk, are on their way while the counters are cleared, and a
    // chunk's while the one before it is worked on.  The kernel is bound by such round trips.  What they used to be were loads
    // under a branch with the use beside them, each waited for before the next went out.  (Us for this kernel, documents: 32768 x 1
    // 16.4 -> 14.5, 70001 x 1 72 -> 58, 131072 x 16 178 -> 99, 8192 x 512 25.6 -> 23.3, 2000 x 4 7.8 -> 7.3; 8192 x 4 in a front end
    // 8.4 -> 6.3.)
    auto load = [&](int i, int &l, int &p) {
        const int j = min(i, n - 1);
        l = level[o + j];
        p = parent[o + j];
    };
    auto group_of = [&](int i, int end, int l, int p) { return i < end ? ord_group(l, p, n) : -1; };
    int front_l[kBack], front_p[kBack], first_l, first_p;
    if (SPREAD && share.first > 0) {
#pragma unroll
        for (int u = 0; u < kBack; u++) load(u * kOrdThreads + tid, front_l[u], front_p[u]);
    }
    load(share.first + tid, first_l, first_p);
    if (tid == 0) s_windows = n + 1 > kOrdWindow ? 0u : 1u;
    for (int t = tid; t < window; t += kOrdThreads) s_count[t] = 0;
    __syncthreads();
    if (n + 1 > kOrdWindow) {
        unsigned mine = 0u;
        for (int i = share.first + tid; i < share.last; i += kOrdThreads) {
            const int g = ord_group(level[o + i], parent[o + i], n);
            if (g >= 0) mine |= 1u << (g / kOrdWindow);
        }
        if (mine) atomicOr(&s_windows, mine);
        __syncthreads();
    }
    const unsigned windows = s_windows;
    for (unsigned todo = windows; todo; todo &= todo - 1u) {
        const int w0 = (__ffs(todo) - 1) * window;
        if (todo != windows) {
            for (int t = tid; t < window; t += kOrdThreads) s_count[t] = 0;
            __syncthreads();
        }
        for (int j0 = 0; SPREAD && j0 < share.first; j0 += kBack * kOrdThreads) {
            int l[kBack], p[kBack];
#pragma unroll
            for (int u = 0; u < kBack; u++) {
                l[u] = front_l[u], p[u] = front_p[u];
                asm volatile("" : "+v"(l[u]), "+v"(p[u]));  // (what is made of them is made here, not in front of the loops)
            }
            if (j0 > 0) {
#pragma unroll
                for (int u = 0; u < kBack; u++) load(j0 + u * kOrdThreads + tid, l[u], p[u]);
            }
#pragma unroll
            for (int u = 0; u < kBack; u++) {
                const int g = group_of(j0 + u * kOrdThreads + tid, share.first, l[u], p[u]);
                int len;
                const bool head = run_head(g, lane, &len);
                if (head && g >= w0 && g < w0 + window) atomicAdd(&s_count[g - w0], len);
            }
        }
        int next_l = first_l, next_p = first_p;
        for (int c0 = share.first; c0 < share.last; c0 += kOrdThreads) {
            const int i = c0 + tid;
            const int grp = group_of(i, share.last, next_l, next_p);
            if (c0 + kOrdThreads < share.last) load(i + kOrdThreads, next_l, next_p);
            int len;
            const bool head = run_head(grp, lane, &len);
            const unsigned long long heads = __ballot(head);
            if (lane == 0) s_wave_runs[wave] = __popcll(heads);
            __syncthreads();
            int first = 0, runs = 0;  // runs in front of this wave's, runs of the chunk
#pragma unroll
            for (int w = 0; w < kOrdWaves; w++) {
                first += w < wave ? s_wave_runs[w] : 0;
                runs += s_wave_runs[w];
            }
            const int run = first + __popcll(heads & ((2ull << lane) - 1ull)) - 1;  // this lane's
            if (head) {
                s_run_grp[run] = grp;
                s_run_len[run] = len;
            }
            __syncthreads();
            for (int r = tid / kOrdSplit; r < runs; r += kOrdThreads / kOrdSplit) {
                const int g = s_run_grp[r];
                if (g < w0 || g >= w0 + window) continue;  // a pad's, or of another window
                int k = 0;
                // (No branch on the group: with one, and a wait for each look, the loop's place in the program decided 5 % of the
                // kernel.  ListOps-shaped trees, us for this kernel: 130 x 8192 110 to 116 - 83, 4 x 1000 17.1 to 18.0 - 14.2.  Unrolled
                // four times it takes more than 64 registers where a sample has several shares: 16 x 131072 99 -> 109.)
#pragma unroll 1
                for (int e = tid % kOrdSplit; e < r; e += kOrdSplit) {
                    const int length = s_run_len[e];
                    k += s_run_grp[e] == g ? length : 0;
                }
#pragma unroll
                for (int d = 1; d < kOrdSplit; d <<= 1) k += __shfl_xor(k, d);
                if (tid % kOrdSplit == 0) s_run_base[r] = s_count[g - w0] + k;
            }
            __syncthreads();
            if (grp >= w0 && grp < w0 + window) {
                const int start = 63 - __builtin_clzll(heads & ((2ull << lane) - 1ull));
                ord[o + i] = 1 + s_run_base[run] + (lane - start);
                if (head && c0 + kOrdThreads < share.last) atomicAdd(&s_count[grp - w0], len);
            }
            __syncthreads();
        }
    }
}

// The same by one workgroup per sample, chunk of 1024 * kChainV positions after chunk (a thread takes kChainV consecutive
// ones), the siblings in earlier chunks counted per parent in global memory (2.4 us per 1024 positions of a document).  A
// run may be as long as the chunk here.
constexpr int kChainV = 4, kChainChunk = kOrdThreads * kChainV;

__global__ __launch_bounds__(kOrdThreads) void k_sibling_ordinals_chain(const int32_t *__restrict__ level,
                                                                         const int32_t *__restrict__ parent, int n,
                                                                         int32_t *cnt,  // [B][n + 1] scratch
                                                                         int32_t *ord)  // [B][n]
{
    // per run head of the chunk: its group, its first position in the chunk; per position of the chunk that
    // starts a run: siblings before that run (s_run_base)
    __shared__ int s_head_parent[kChainChunk], s_head_start[kChainChunk], s_run_base[kChainChunk];
    __shared__ int s_last_grp[kOrdThreads];
    __shared__ int s_wave_max[kOrdWaves], s_wave_heads[kOrdWaves];
    const int b = blockIdx.x, tid = threadIdx.x, wave = tid >> 6, lane = tid & 63;
    const size_t o = (size_t)b * n;
    int32_t *my_cnt = cnt + (size_t)b * (n + 1);
    for (int i = tid; i <= n; i += kOrdThreads) my_cnt[i] = 0;
    __syncthreads();
    for (int c0 = 0; c0 < n; c0 += kChainChunk) {
        const int idx0 = tid * kChainV;  // this thread's first position inside the chunk
        int grp[kChainV];                // the parent (n for roots), -1 for pads and positions past n
#pragma unroll
        for (int u = 0; u < kChainV; u++) {
            const int i = c0 + idx0 + u;
            grp[u] = -1;
            if (i < n && level[o + i] >= 0) {
                const int p = parent[o + i];
                grp[u] = (p >= 0 && p < n) ? p : n;
            }
        }
        s_last_grp[tid] = grp[kChainV - 1];
        __syncthreads();
        // run heads; the last head at or before every position: a running maximum over the threads
        int before = tid == 0 ? -2 : s_last_grp[tid - 1];
        bool head[kChainV];
        int n_mine = 0, last_head = -1;
#pragma unroll
        for (int u = 0; u < kChainV; u++) {
            head[u] = grp[u] != before;
            before = grp[u];
            if (head[u]) {
                n_mine++;
                last_head = idx0 + u;
            }
        }
        int run_max = last_head, heads_incl = n_mine;
#pragma unroll
        for (int d = 1; d < 64; d <<= 1) {
            const int y = __shfl_up(run_max, d), z = __shfl_up(heads_incl, d);
            if (lane >= d) {
                run_max = max(run_max, y);
                heads_incl += z;
            }
        }
        if (lane == 63) {
            s_wave_max[wave] = run_max;
            s_wave_heads[wave] = heads_incl;
        }
        __syncthreads();
        int start_in = __shfl_up(run_max, 1);  // last head before this thread's positions
        if (lane == 0) start_in = -1;
        int my_head = heads_incl - n_mine, n_heads = 0;
        for (int w = 0; w < kOrdWaves; w++) {
            if (w < wave) {
                start_in = max(start_in, s_wave_max[w]);
                my_head += s_wave_heads[w];
            }
            n_heads += s_wave_heads[w];
        }
        int start[kChainV];
        {
            int cur = start_in, h = my_head;
#pragma unroll
            for (int u = 0; u < kChainV; u++) {
                if (head[u]) {
                    cur = idx0 + u;
                    s_head_parent[h] = grp[u];
                    s_head_start[h] = cur;
                    h++;
                }
                start[u] = cur;
            }
        }
        __syncthreads();
        // siblings in earlier runs of this chunk: kOrdSplit lanes share the scan over the earlier heads of one head
        for (int h = tid / kOrdSplit; h < n_heads; h += kOrdThreads / kOrdSplit) {
            const int g = s_head_parent[h];
            if (g < 0) continue;
            int k = 0;
            for (int e = tid % kOrdSplit; e < h; e += kOrdSplit)
                if (s_head_parent[e] == g) k += s_head_start[e + 1] - s_head_start[e];
#pragma unroll
            for (int d = 1; d < kOrdSplit; d <<= 1) k += __shfl_xor(k, d);
            if (tid % kOrdSplit == 0) {
                // siblings in earlier chunks (the counter last changed before the barrier that ended the previous chunk)
                const int base = __hip_atomic_load(&my_cnt[g], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
                s_run_base[s_head_start[h]] = base + k;
            }
        }
        __syncthreads();
#pragma unroll
        for (int u = 0; u < kChainV; u++)
            if (grp[u] >= 0) ord[o + c0 + idx0 + u] = 1 + s_run_base[start[u]] + (idx0 + u - start[u]);
        // add this chunk's runs to the counters; the returned value makes the thread wait for the atomic
        {
            int h = my_head;
#pragma unroll
            for (int u = 0; u < kChainV; u++) {
                if (!head[u]) continue;
                if (grp[u] >= 0) {
                    const int end = h + 1 < n_heads ? s_head_start[h + 1] : kChainChunk;
                    const int old = atomicAdd(&my_cnt[grp[u]], end - (idx0 + u));
                    asm volatile("" ::"v"(old));
                }
                h++;
            }
        }
        __syncthreads();
    }
}

// ---- index vectors: walk up the ancestors ------------------------------------------------------------
// A chain of round trips, one per ancestor: level, parent and ordinal of a position are requested together.  With
// few levels, a template argument (0: any), the vector stays in registers until it is whole.  (It was written twice, each
// ancestor took two round trips, and the sample of a position was found by a 64-bit division.  us for the ordinals and the
// vectors, before - now: 8192 x 4 10.3 - 9.9, 8192 x 16 11.2 - 10.4, 2048 x 256 14.4 - 12.9.)
template <int LEVELS>
__global__ __launch_bounds__(256) void k_index_vectors(const int32_t *__restrict__ level,
                                                       const int32_t *__restrict__ parent,
                                                       const int32_t *__restrict__ ord, int n, int n_levels, unsigned total,
                                                       int32_t *__restrict__ p)
{
    const unsigned g = blockIdx.x * 256u + threadIdx.x;  // (positions, at most 2^30)
    if (g >= total) return;
    const int i = (int)(g % (unsigned)n), L = LEVELS ? LEVELS : n_levels;
    const size_t o = (size_t)(g - (unsigned)i);
    int32_t *mine = p + (size_t)g * L;
    int held[LEVELS > 0 ? LEVELS : 1];
    if (LEVELS > 0) {
#pragma unroll
        for (int l = 0; l < LEVELS; l++) held[l] = 0;
    } else {
        for (int l = 0; l < L; l++) mine[l] = 0;
    }
    int a = i;
    for (int steps = 0; a >= 0 && a < n && steps < 2 * HDT_MAX_LEVELS; steps++) {
        const int l = level[o + a], up = parent[o + a], r = ord[o + a];
        if (l < 0) break;
        if (LEVELS > 0) {
#pragma unroll
            for (int t = 0; t < LEVELS; t++) held[t] = l == t + 1 ? r : held[t];
        } else if (l >= 1 && l <= L) {
            mine[l - 1] = r;
        }
        a = up;
    }
#pragma unroll
    for (int l = 0; l < LEVELS; l++) mine[l] = held[l];
}

static auto index_vectors_kernel(int n_levels)
{
    switch (n_levels) {
    case 1: return k_index_vectors<1>;
    case 2: return k_index_vectors<2>;
    case 3: return k_index_vectors<3>;
    case 4: return k_index_vectors<4>;
    default: return k_index_vectors<0>;
    }
}

// ---- the sinusoidal table ------------------------------------------------------------------------------
__global__ __launch_bounds__(256) void k_hpe_table(float *__restrict__ table, int rows, int d_model)
{
    const int64_t g = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (g >= (int64_t)rows * d_model) return;
    const int v = (int)(g / d_model), c = (int)(g - (int64_t)v * d_model);
    const double w = pow(10000.0, -2.0 * (double)(c / 2) / (double)d_model);
    const double x = w * (double)v;
    table[g] = (float)((c & 1) ? cos(x) : sin(x));
}

// ---- x += sum over the levels of the table rows -------------------------------------------------------
// A thread owns 8 consecutive channels (16 bytes of bf16) of kPerThread consecutive positions: the kernel is a stream
// over x, and what it must keep away from that stream is the table, whose rows (fp32, out of L2) are three times
// the bytes of x.  Consecutive positions mostly share their upper-level indices, so a position's row of a level is read only
// where the index differs from that of the position before it.
// What bounds a thread is its chain of round trips: x, then the indices, then all rows it needs, requested together.  (With
// a branch per row for indices beyond the table, every row was waited for before the next was asked for, six in turn.)  So
// one question for the whole wave, are all indices inside the table, and no branch behind it but the masks of rows that
// repeat.  us, before - now, over six batches in turn: bf16 4 x 8192 x 768 26.2 - 25.9, 32768 x 512 17.6 - 14.9, 2 x 8192 x
// 1024 17.3 - 14.6, 1024 x 768 4.15 - 3.6; fp32 4 x 8192 x 768 47.7 - 44.3, 8 x 2048 x 512 15.8 - 15.1; the first behind the
// kernels that make its indices 23 - 19.5.  With repeated rows read again 27.3, 16.0 and 15.7 for the first three; one
// position per thread 27.5, 15.3, 15.2, four 27.7, 17.2, 16.8; the indices in front of x 25.7, 15.9, 15.1 and, the first behind
// its index kernels, a microsecond more; x behind the rows 26.7, 14.7, 14.6.  The first 128 rows in the LDS of workgroups
// that take 64 channels each: 27.8, 16.5, 16.1.
constexpr int kPerThread = 2, kMoreLevels = 2;

__device__ __noinline__ double hpe_frequency(int c, int d_model) { return pow(10000.0, -2.0 * (double)(c / 2) / (double)d_model); }
__device__ __noinline__ float hpe_value(double x, int c) { return (float)((c & 1) ? cos(x) : sin(x)); }
// (both in one call)
__device__ __noinline__ float hpe_direct(int v, int c, int d_model)
{
    const double w = pow(10000.0, -2.0 * (double)(c / 2) / (double)d_model);
    const double x = w * (double)v;
    return (float)((c & 1) ? cos(x) : sin(x));
}

// The whole add of one thread of a wave in which an index has no row, for more than four levels: around calls the form below would
// hold what it keeps from group to group in registers of two waves per SIMD, so this starts again and nothing is kept.  Two channels at
// a time, which have their frequency in common (4 x 8192 x 768, five levels, no table, us: 865, 563 with what repeats evaluated once,
// 196 with the frequency found once).
template <bool BF16>
__device__ __forceinline__ void hpe_add_beyond(const int32_t *p, unsigned pos0, unsigned pos1, int n_levels, const float *table, int rows,
                                               void *x, int d_model, int c0)
{
#pragma unroll 1
    for (int c = c0; c < c0 + 8; c += 2) {
        const double w = hpe_frequency(c, d_model);
        float acc[2][2] = {};
#pragma unroll 1
        for (int l = 0; l < n_levels; l++) {
            const int first = p[(size_t)pos0 * n_levels + l], second = p[(size_t)pos1 * n_levels + l];
#pragma unroll
            for (int u = 0; u < 2; u++) {
                const int v = u ? second : first;
                if (u > 0 && second == first) continue;
                const bool both = u == 0 && second == first;
                if (v >= 0 && v < rows) {
                    const float *row = table + (size_t)v * d_model + c;
#pragma unroll
                    for (int e = 0; e < 2; e++) {
                        acc[u][e] += row[e];
                        if (both) acc[1][e] += row[e];
                    }
                } else {
#pragma unroll
                    for (int e = 0; e < 2; e++) {
                        const float value = hpe_value(w * (double)v, c + e);
                        acc[u][e] += value;
                        if (both) acc[1][e] += value;
                    }
                }
            }
        }
#pragma unroll
        for (unsigned u = 0; u < 2; u++) {
            if (u && pos1 == pos0) break;
            const size_t at = (size_t)(u ? pos1 : pos0) * d_model + c;
#pragma unroll
            for (int e = 0; e < 2; e++) {
                if (BF16) {
                    __bf16 *to = reinterpret_cast<__bf16 *>(x) + at;
                    to[e] = (__bf16)((float)to[e] + acc[u][e]);
                } else {
                    reinterpret_cast<float *>(x)[at + e] += acc[u][e];
                }
            }
        }
    }
}

// L levels at a time: all of them, or with MORE (five levels and more) group after group, the next group's indices requested in
// front of this one's rows.  Groups of two, and fp32 asks for x last: five waves per SIMD.  us, bf16 and fp32, of 4 x 8192 x 768 with
// five levels / nine / 25: groups of four 35.1, 42.3 / 48.3, 55.3 / 95.6, 102 (133 and 141 registers); of two 24.1, 33.5 / 34.2, 42.8 / 81.7,
// 90.5; of three, without the next indices, 24.2, 34.2 / 35.6, 43.7 / 84.7, 93.6; one level after the other, each row waited for, 25.7,
// 35.7 / 37.3, 47.3 / 86, 96.  At 1001 x 512 the groups of four are ahead, by a tenth from 12 levels on (25: 8.4, of two 9.5).
template <bool BF16, int L, bool MORE>
__global__ __launch_bounds__(256) void k_hpe_add(const int32_t *__restrict__ p, unsigned positions, int n_levels,
                                                 const float *__restrict__ table, int rows, void *__restrict__ x,
                                                 int d_model, unsigned groups)
{
    typedef __attribute__((ext_vector_type(8))) __bf16 bf16x8;
    constexpr bool X_LAST = MORE && !BF16;
    constexpr int XV = BF16 ? 1 : 2;  // 16-byte pieces of x per thread and position
    const unsigned per_pos = (unsigned)d_model / 8u;
    const unsigned g = blockIdx.x * blockDim.x + threadIdx.x;  // (group of kPerThread positions, channel group)
    const unsigned pos0 = g / per_pos, c0 = (g - pos0 * per_pos) * 8u;
    if (pos0 >= groups) return;
    unsigned pos[kPerThread];  // a position behind the last one stands for the last
    float4 xv[kPerThread][XV];
    float acc[kPerThread][8];
    float4 *xs = reinterpret_cast<float4 *>(x);
#pragma unroll
    for (int u = 0; u < kPerThread; u++) {
        pos[u] = min(pos0 * kPerThread + u, positions - 1u);
#pragma unroll
        for (int w = 0; w < (X_LAST ? 0 : XV); w++) xv[u][w] = xs[((size_t)pos[u] * per_pos + c0 / 8u) * XV + w];
#pragma unroll
        for (int e = 0; e < 8; e++) acc[u][e] = 0.f;
    }
    asm volatile("" ::: "memory");  // (x is asked for first)
    auto add = [&](int u, const float4 &a, const float4 &b) {
        acc[u][0] += a.x, acc[u][1] += a.y, acc[u][2] += a.z, acc[u][3] += a.w;
        acc[u][4] += b.x, acc[u][5] += b.y, acc[u][6] += b.z, acc[u][7] += b.w;
    };
    auto row_of = [&](int v) { return reinterpret_cast<const float4 *>(table + (size_t)v * d_model + c0); };
    const int stride = MORE ? n_levels : L;
    int v[kPerThread][L], next[kPerThread][L];
    auto indices = [&](int l0, int (&to)[kPerThread][L]) {
#pragma unroll
        for (int u = 0; u < kPerThread; u++)
#pragma unroll
            for (int l = 0; l < L; l++) to[u][l] = p[(size_t)pos[u] * stride + (MORE ? min(l0 + l, n_levels - 1) : l)];
    };
    indices(0, v);
    for (int l0 = 0; l0 < (MORE ? n_levels : 1); l0 += L) {
        bool inside = true;
        if (MORE && l0 > 0) {
#pragma unroll
            for (int u = 0; u < kPerThread; u++)
#pragma unroll
                for (int l = 0; l < L; l++) v[u][l] = next[u][l];
        }
        if (MORE) indices(l0 + L, next);
#pragma unroll
        for (int u = 0; u < kPerThread; u++)
#pragma unroll
            for (int l = 0; l < L; l++) inside = inside && v[u][l] >= 0 && v[u][l] < rows;
        const bool beyond = __any(!inside);
        if (MORE && beyond) {
            hpe_add_beyond<BF16>(p, pos[0], pos[1], n_levels, table, rows, x, d_model, (int)c0);
            return;
        }
        if (!beyond) {
            float4 t[kPerThread][L][2];
#pragma unroll
            for (int l = 0; l < L; l++)
#pragma unroll
                for (int u = 0; u < kPerThread; u++) {
                    const float4 *row = row_of(v[u][l]);
                    if (u > 0 || (MORE && l > 0)) t[u][l][0] = t[u][l][1] = make_float4(0.f, 0.f, 0.f, 0.f);
                    if (MORE && l > 0 && l0 + l >= n_levels) continue;
                    if (u == 0 || v[u][l] != v[u > 0 ? u - 1 : 0][l]) {
                        t[u][l][0] = row[0];
                        t[u][l][1] = row[1];
                    }
                }
#pragma unroll
            for (int u = 0; u < kPerThread; u++)
#pragma unroll
                for (int l = 0; l < L; l++) {
                    if (u > 0 && v[u][l] == v[u > 0 ? u - 1 : 0][l]) {
                        t[u][l][0] = t[u > 0 ? u - 1 : 0][l][0];
                        t[u][l][1] = t[u > 0 ? u - 1 : 0][l][1];
                    }
                    if (!MORE || l0 + l < n_levels) add(u, t[u][l][0], t[u][l][1]);
                }
        } else {
            // Some index has no row.  What an index adds goes to both positions at once where it repeats: its values take longer
            // than everything else here.  (us, every position its own - one evaluation: 4 x 8192 x 768, three levels, no table
            // 507 - 341, the top level alone beyond the table 178 - 94.)
            static_assert(kPerThread == 2, "one repeat to look for");
#pragma unroll 1
            for (int l = 0; l < L; l++) {
                const int first = p[(size_t)pos[0] * stride + l], second = p[(size_t)pos[1] * stride + l];
#pragma unroll
                for (int u = 0; u < kPerThread; u++) {
                    const int vv = u ? second : first;
                    if (u > 0 && second == first) continue;
                    const bool both = u == 0 && second == first;
                    if (vv >= 0 && vv < rows) {
                        const float4 *row = row_of(vv);
                        const float4 r0 = row[0], r1 = row[1];
                        add(u, r0, r1);
                        if (both) add(1, r0, r1);
                    } else {
#pragma unroll
                        for (int e = 0; e < 8; e++) {
                            const float value = hpe_direct(vv, (int)c0 + e, d_model);
                            acc[u][e] += value;
                            if (both) acc[1][e] += value;
                        }
                    }
                }
            }
        }
    }
    if (X_LAST) {
#pragma unroll
        for (int u = 0; u < kPerThread; u++)
#pragma unroll
            for (int w = 0; w < XV; w++) xv[u][w] = xs[((size_t)pos[u] * per_pos + c0 / 8u) * XV + w];
    }
#pragma unroll
    for (int u = 0; u < kPerThread; u++) {
        if (pos0 * kPerThread + u >= positions) continue;
        const size_t at = ((size_t)pos[u] * per_pos + c0 / 8u) * XV;
        if (BF16) {
            bf16x8 xb = __builtin_bit_cast(bf16x8, xv[u][0]);
#pragma unroll
            for (int e = 0; e < 8; e++) xb[e] = (__bf16)((float)xb[e] + acc[u][e]);
            xs[at] = __builtin_bit_cast(float4, xb);
        } else {
            float4 a = xv[u][0], b = xv[u][XV - 1];
            a.x += acc[u][0], a.y += acc[u][1], a.z += acc[u][2], a.w += acc[u][3];
            b.x += acc[u][4], b.y += acc[u][5], b.z += acc[u][6], b.w += acc[u][7];
            xs[at] = a;
            xs[at + 1] = b;
        }
    }
}

template <bool BF16>
auto hpe_add_kernel(int n_levels)
{
    switch (n_levels) {
    case 1: return k_hpe_add<BF16, 1, false>;
    case 2: return k_hpe_add<BF16, 2, false>;
    case 3: return k_hpe_add<BF16, 3, false>;
    case 4: return k_hpe_add<BF16, 4, false>;
    default: return k_hpe_add<BF16, kMoreLevels, true>;
    }
}

}  // namespace

extern "C" __attribute__((visibility("default"))) hdt_status_t hdt_parents_from_levels(const int32_t *d_level,
                                                                                        int32_t batch, int32_t n_pos,
                                                                                        int32_t *d_parent, void *stream)
{
    if (batch < 0 || n_pos < 0) return hdt_fail(HDT_ERR_INVALID_ARG, "hdt_parents_from_levels: negative size");
    if (batch == 0 || n_pos == 0) return HDT_OK;
    if (!d_level || !d_parent) return hdt_fail(HDT_ERR_INVALID_ARG, "hdt_parents_from_levels: NULL pointer");
    if ((int64_t)batch * n_pos > (1LL << 30)) return hdt_fail(HDT_ERR_SHAPE, "hdt_parents_from_levels: batch * n_pos too large");
    hipStream_t st = (hipStream_t)stream;
    HdtTimer t("hdt_hpe_parents_from_levels", st);
    // in place: the levels in front of a share would be gone by the time it reads them, so one workgroup has the whole sample
    const int shares = d_parent == d_level ? 1 : hpe_shares(batch, n_pos);
    const dim3 grid((unsigned)batch * shares), block(kOrdThreads);
    if (shares > 1)
        hipLaunchKernelGGL(k_parents_from_levels<true>, grid, block, 0, st, d_level, n_pos, shares, d_parent);
    else
        hipLaunchKernelGGL(k_parents_from_levels<false>, grid, block, 0, st, d_level, n_pos, shares, d_parent);
    HDT_HIP_TRY(hipGetLastError());
    return HDT_OK;
}

extern "C" __attribute__((visibility("default"))) size_t hdt_index_vectors_workspace_bytes(int32_t batch, int32_t n_pos)
{
    if (batch <= 0 || n_pos <= 0) return 0;
    // per-parent counters [B][N+1] (of k_sibling_ordinals_chain) and sibling ordinals [B][N]
    const size_t ints = (size_t)batch * ((size_t)n_pos + 1) + (size_t)batch * (size_t)n_pos;
    return (ints * sizeof(int32_t) + 255) & ~(size_t)255;
}

extern "C" __attribute__((visibility("default"))) hdt_status_t hdt_index_vectors(
    const int32_t *d_level, const int32_t *d_parent, int32_t batch, int32_t n_pos, int32_t n_levels, int32_t *d_p,
    void *workspace, size_t workspace_bytes, void *stream)
{
    if (batch < 0 || n_pos < 0) return hdt_fail(HDT_ERR_INVALID_ARG, "hdt_index_vectors: negative size");
    if (n_levels < 1 || n_levels >= HDT_MAX_LEVELS)
        return hdt_fail(HDT_ERR_INVALID_ARG, "hdt_index_vectors: n_levels = %d (1 .. %d)", n_levels, HDT_MAX_LEVELS - 1);
    if (batch == 0 || n_pos == 0) return HDT_OK;
    if (!d_level || !d_parent || !d_p) return hdt_fail(HDT_ERR_INVALID_ARG, "hdt_index_vectors: NULL pointer");
    const size_t need = hdt_index_vectors_workspace_bytes(batch, n_pos);
    if (!workspace || workspace_bytes < need || ((uintptr_t)workspace & 15u))
        return hdt_fail(HDT_ERR_INVALID_ARG, "hdt_index_vectors: workspace of %zu bytes (16-byte aligned) needed", need);
    if ((int64_t)batch * n_pos > (1LL << 30)) return hdt_fail(HDT_ERR_SHAPE, "hdt_index_vectors: batch * n_pos too large");
    hipStream_t st = (hipStream_t)stream;
    int32_t *cnt = static_cast<int32_t *>(workspace);
    int32_t *ord = cnt + (size_t)batch * ((size_t)n_pos + 1);
    {
        const int shares = hpe_shares(batch, n_pos);
        const size_t lds = (size_t)std::min(n_pos + 1, kOrdWindow) * sizeof(int);
        HdtTimer t("hdt_hpe_sibling_ordinals", st);
        if (n_pos >= kOrdWindow && (shares < kMinShares || n_pos > kMaxWindowed)) {
            hipLaunchKernelGGL(k_sibling_ordinals_chain, dim3((unsigned)batch), dim3(kOrdThreads), 0, st, d_level, d_parent, n_pos,
                               cnt, ord);
        } else {
            const auto kernel = shares > 1 ? k_sibling_ordinals<true> : k_sibling_ordinals<false>;
            if (lds > 48 * 1024)  // with the static arrays: beyond the 64 KB a launch gets by default
                HDT_HIP_TRY(hipFuncSetAttribute((const void *)kernel, hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds));
            hipLaunchKernelGGL(kernel, dim3((unsigned)batch * shares), dim3(kOrdThreads), lds, st, d_level, d_parent, n_pos, shares,
                               ord);
        }
    }
    {
        const int64_t total = (int64_t)batch * n_pos;
        HdtTimer t("hdt_hpe_index_vectors", st);
        hipLaunchKernelGGL(index_vectors_kernel(n_levels), dim3((unsigned)((total + 255) / 256)), dim3(256), 0, st, d_level, d_parent,
                           ord, n_pos, n_levels, (unsigned)total, d_p);
    }
    HDT_HIP_TRY(hipGetLastError());
    return HDT_OK;
}

extern "C" __attribute__((visibility("default"))) hdt_status_t hdt_hpe_table(float *d_table, int32_t rows,
                                                                              int32_t d_model, void *stream)
{
    if (rows < 0 || d_model <= 0 || d_model % 8) return hdt_fail(HDT_ERR_INVALID_ARG, "hdt_hpe_table: rows >= 0, d_model a positive multiple of 8");
    if (rows == 0) return HDT_OK;
    if (!d_table || ((uintptr_t)d_table & 15u)) return hdt_fail(HDT_ERR_INVALID_ARG, "hdt_hpe_table: NULL or misaligned table");
    const int64_t total = (int64_t)rows * d_model;
    if (total > (1LL << 31)) return hdt_fail(HDT_ERR_SHAPE, "hdt_hpe_table: table too large");
    HdtTimer t("hdt_hpe_table", (hipStream_t)stream);
    hipLaunchKernelGGL(k_hpe_table, dim3((unsigned)((total + 255) / 256)), dim3(256), 0, (hipStream_t)stream, d_table,
                       rows, d_model);
    HDT_HIP_TRY(hipGetLastError());
    return HDT_OK;
}

extern "C" __attribute__((visibility("default"))) hdt_status_t hdt_hpe_add(const int32_t *d_p, int32_t batch,
                                                                            int32_t n_pos, int32_t n_levels,
                                                                            const float *d_table, int32_t table_rows,
                                                                            void *x, int32_t d_model, hdt_dtype_t dt,
                                                                            void *stream)
{
    if (batch < 0 || n_pos < 0 || table_rows < 0) return hdt_fail(HDT_ERR_INVALID_ARG, "hdt_hpe_add: negative size");
    if (n_levels < 1 || n_levels >= HDT_MAX_LEVELS) return hdt_fail(HDT_ERR_INVALID_ARG, "hdt_hpe_add: n_levels = %d", n_levels);
    if (d_model <= 0 || d_model % 8) return hdt_fail(HDT_ERR_INVALID_ARG, "hdt_hpe_add: d_model must be a positive multiple of 8");
    if (dt != HDT_BF16 && dt != HDT_F32) return hdt_fail(HDT_ERR_UNSUPPORTED, "hdt_hpe_add: unknown dtype %d", (int)dt);
    if (batch == 0 || n_pos == 0) return HDT_OK;
    if (!d_p || !x || (table_rows > 0 && !d_table)) return hdt_fail(HDT_ERR_INVALID_ARG, "hdt_hpe_add: NULL pointer");
    if (((uintptr_t)x & 15u) || ((uintptr_t)d_table & 15u)) return hdt_fail(HDT_ERR_INVALID_ARG, "hdt_hpe_add: pointers must be 16-byte aligned");
    const int64_t positions = (int64_t)batch * n_pos;
    const int64_t pos_stride = (positions + kPerThread - 1) / kPerThread, threads = pos_stride * (d_model / 8);
    if (positions > 0x7fffffffLL || threads > 0x7fffffffLL) return hdt_fail(HDT_ERR_SHAPE, "hdt_hpe_add: too many elements");
    hipStream_t st = (hipStream_t)stream;
    HdtTimer t(dt == HDT_BF16 ? "hdt_hpe_add_bf16" : "hdt_hpe_add_f32", st);
    const auto kernel = dt == HDT_BF16 ? hpe_add_kernel<true>(n_levels) : hpe_add_kernel<false>(n_levels);
    hipLaunchKernelGGL(kernel, dim3((unsigned)((threads + 255) / 256)), dim3(256), 0, st, d_p, (unsigned)positions, n_levels,
                       d_table, table_rows, x, d_model, (unsigned)pos_stride);
    HDT_HIP_TRY(hipGetLastError());
    return HDT_OK;
}
