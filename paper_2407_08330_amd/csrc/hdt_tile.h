// Pieces shared by the three bf16 kernels (forward, dQ pass, dK/dV pass).  All of them have the same
// skeleton: a workgroup of BM/32 waves owns BM consecutive rows of the schedule (wave w the rows
// 32w..32w+31, whose operands stay in registers as MFMA B fragments), walks the row tile's list
// entries, and for each entry gathers the BN rows of two [n_pos][D] tensors that the entry's key
// positions name into LDS.  Two tile shapes are built: 128 x 64 (four waves; the layout's default) and
// 64 x 32 (two waves).  The waves of a workgroup meet at a barrier once per entry and the mask is close to
// block diagonal, so with four waves a wave often waits through entries that hold nothing for its rows;
// the finer shape loses fewer such slots and skips more of the mask, but walks more entries and needs
// twice the workgroups.  Measured, the two are within a few percent of each other at head size 64 and the
// finer one is ~5-10 % ahead at head size 128; its layout takes 1-4 us longer to build.
//
// The gather uses the CDNA direct-to-LDS loads (global_load_lds_*: every lane supplies a global
// address, the 64 results land in LDS at M0 + lane*size) into a ring of two stages, so that a
// tile is in flight per workgroup without being held in registers:
//   iteration t:  wait until tile t has landed -> barrier -> start tile t+1 -> compute tile t.
// The key positions of an entry are read the same way, one tile further ahead than the rows they
// address, and the entries' summaries with scalar loads, so no iteration waits on a chain of dependent
// loads.
// The vector-memory instructions inside the loop are those issued here with inline asm, which the compiler does not
// count: the waits for them stand here too.  With two stages an iteration waits for all of them; in front of the loop the
// first entry's positions are waited for with the second entry's in flight (a load more would make that wait longer, not wrong).
//
// A wave of the backward on 64 x 32 tiles works on 4 to 5 entries, so what stands around its loop counts as much as the
// loop: counters put 540 of 980 vector instructions and 500 of 600 scalar ones there, with a vector instruction in
// flight 53 % of the time.  Hence the divisions by numbers the host knows (FastDiv), blocks of zeros from the matrix pipe
// (zero_block), results leaving at constant offsets (store_rows_via_lds), and an entry's positions read together and in
// front of the barrier (Ring::top).  Together, us per launch: backward 86.8 -> 82.9 (8192 positions x 4 x 12, 64 x 32), 98 ->
// 94 (128 x 64), 231 -> 222 (32768 x 16, head size 128), 25.5 -> 24.2 (2047 x 3 x 12); forward 46.3 -> 45.5, 104.3 -> 102.2.
//
// A wave-level load writes 1024 contiguous bytes, so LDS rows cannot be padded; bank conflicts are
// avoided with an XOR swizzle of the 16-byte chunks of a row instead (applied to the global address
// of each lane on the way in, and to the LDS address on the way out).
#pragma once

#include "hdt_internal.h"
#include "hdt_mfma.h"

namespace hdt_tile {

// tile geometry: BM query rows x BN key slots, one wave per 32 rows; a ring stage (two tiles of BN rows)
// also has to hold the workgroup's own BM rows, hence BM = 2 BN, and every wave loads 16 rows of a tile
template <int BM_, int BN_>
struct Geo {
    static constexpr int BM = BM_, BN = BN_;
    static constexpr int NW = BM_ / 32;               // waves per workgroup
    static constexpr int THREADS = NW * 64;
    static constexpr int KB = BN_ / 32;               // 32-key sub-blocks per tile
    static constexpr int NSUB = (BM_ / 32) * KB;      // 32x32 sub-blocks per tile
    static constexpr unsigned XCD_CHUNK = 4096 / BM_; // consecutive row tiles handed to one XCD (see logical_block)
    static_assert(BM_ == 2 * BN_ && BN_ / NW == 16, "unsupported tile shape");
};
constexpr float LOG2E = 1.4426950408889634f;
constexpr float LN2 = 0.6931471805599453f;

// Read-only schedule arrays are read through the constant address space: with a wave-uniform index
// the compiler then uses scalar loads (lgkmcnt), which keeps them out of the vector-memory queue
// whose in-order counter the hand-scheduled loads rely on.
#define HDT_CONST __attribute__((address_space(4)))
typedef const int32_t HDT_CONST *cptr_i32;
typedef const uint32_t HDT_CONST *cptr_u32;
__device__ __forceinline__ cptr_i32 as_const(const int32_t *p) { return (cptr_i32)(uintptr_t)p; }
__device__ __forceinline__ cptr_u32 as_const(const uint32_t *p) { return (cptr_u32)(uintptr_t)p; }

// Workgroups are handed to the 8 XCDs round-robin (workgroup id mod 8).  Logical work items are dealt to
// the XCDs in chunks of consecutive items (at most Geo::XCD_CHUNK row tiles: 4096 rows), so that neighbouring row tiles
// (which gather largely the same rows) share an L2, while every XCD still gets an even mix of the samples: with
// whole (sample, head) ranges per XCD, one long document made two XCDs finish well after the others.  The chunk
// is counted in rows: with 32 tiles of 64 rows the forward took 48.8 us at 8192 positions x 4 samples x 12
// heads, with 64 of them 46.4, as with 32 tiles of 128 rows.  Every round of 8 chunks starts one XCD further: a
// sample of 8192 positions is two chunks, and the first halves of documents that end in pads are the heavier
// ones, which would otherwise all go to the even XCDs (7 % more work there).
// The items are spread over as few rounds as that chunk allows, and evenly: a grid that a whole number of full rounds
// does not make gets a smaller chunk, so that no XCD has a chunk more than another, and a small grid is
// spread over all of them (288 workgroups of a cross-attention backward: 33.6 -> 24.1 us; forward of 576 row tiles:
// 14.6 -> 13.7; full rounds as before).
// The grid is padded to whole rounds; padding workgroups get an index >= n_items and leave at once.  `unit`: items
// that must stay together (the roles of a tile).
__host__ __device__ __forceinline__ unsigned xcd_chunk(unsigned n_items, unsigned most, unsigned unit)
{
    const unsigned rounds = (n_items + 8u * most - 1u) / (8u * most);
    return n_items ? (n_items + 8u * rounds * unit - 1u) / (8u * rounds * unit) * unit : unit;
}
__host__ __device__ __forceinline__ unsigned padded_grid(unsigned n_items, unsigned chunk)
{
    return (n_items + 8u * chunk - 1u) / (8u * chunk) * (8u * chunk);
}
// Division by a divisor the host knows, by the multiplication of Granlund and Montgomery (PLDI 1994), of numbers below 2^31: three scalar instructions where the compiler's own takes
// about 25, vector ones and a reciprocal among them.  With l = ceil(log2 d) and mul = ceil(2^(31 + l) / d) (at most 2^32 - 1),
// n * mul = (2^(31 + l) n + e n) / d with e < d <= 2^l, so the error e n / d stays below 2^(31 + l) / d and the quotient is exact.
struct FastDiv {
    uint32_t d, mul, shift;
    FastDiv() = default;
    explicit FastDiv(uint32_t divisor) : d(divisor ? divisor : 1)
    {
        uint32_t l = 0;
        while ((1ull << l) < d) l++;
        shift = 31 + l;
        mul = (uint32_t)(((1ull << shift) + d - 1) / d);
    }
    __device__ __forceinline__ uint32_t div(uint32_t n) const { return (uint32_t)(((uint64_t)n * mul) >> shift); }
};
__device__ __forceinline__ unsigned logical_block(unsigned bid, const FastDiv &chunk)
{
    const unsigned x = bid & 7u, k = bid >> 3, round = chunk.div(k);
    return (round * 8u + ((x + round) & 7u)) * chunk.d + (k - round * chunk.d);
}

// Chunk swizzle of row r of a tile whose rows hold CPR chunks of 16 bytes.  The LDS has 64 banks of 4 bytes
// (256 bytes per clock): a 16-byte read is served 16 lanes at a time, a transposing 8-byte read 32 lanes at
// a time, and a group is conflict-free when its lanes fall into different 16-byte columns of the 256.
//   row reads (one logical chunk down 16 consecutive rows): 16 different columns.  With 128-byte rows the
//     row's parity picks the half of the 256 bytes, so the 8 even rows need 8 different values and so do the
//     8 odd ones; with 256-byte rows all 16 values differ.
//   transposing reads (4 consecutive aligned rows x 4 chunks 4i ^ {0..3}): the rows that share a half must
//     differ in the chunk bits above the low two.
// Rows r and r + 8 differ by 2 in both cases (what the second of a pair of transposing reads relies on).
// Measured on the chip: 4.0 clocks per 16-byte wave read against 6.4 with a swizzle of period 8.
template <int CPR>
__device__ __forceinline__ int swz(int r)
{
    if (CPR == 8) return (((r & 3) << 1) | ((r >> 2) & 1)) ^ ((r >> 2) & 2);
    return ((r & 3) << 2) | ((r >> 2) & 3);
}

__device__ __forceinline__ uint32_t lds_addr(const void *p)
{
    return (uint32_t)(uintptr_t)(HDT_LDS const char *)p;
}

// direct-to-LDS loads: lane l's 16 (4) bytes at base + off (a wave-uniform base pointer in scalar registers,
// a per-lane byte offset below 2^31) land at lds_base + 16*l (4*l)
__device__ __forceinline__ void dma16(const void *base, uint32_t off, uint32_t lds_base)
{
    asm volatile("s_mov_b32 m0, %2\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %0, %1" ::"v"(off), "s"(base), "s"(lds_base)
                 : "memory", "m0");
}
__device__ __forceinline__ void dma4(const void *base, uint32_t off, uint32_t lds_base)
{
    asm volatile("s_mov_b32 m0, %2\n\ts_nop 0\n\tglobal_load_lds_dword %0, %1" ::"v"(off), "s"(base), "s"(lds_base)
                 : "memory", "m0");
}
template <int N>
__device__ __forceinline__ void wait_vmcnt()
{
    asm volatile("s_waitcnt vmcnt(%0)" ::"n"(N) : "memory");
}
// workgroup barrier without the fence __syncthreads() carries: LDS traffic of this wave is drained
// by the lgkmcnt wait, the direct-to-LDS loads by the explicit vmcnt waits of the callers
__device__ __forceinline__ void wg_barrier()
{
    asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory");
}

// A value the compiler cannot see through: what is derived from it is computed after this point.  Used on
// the lane index in front of an epilogue, whose per-lane addresses would otherwise be hoisted above the
// tile loop and held in registers throughout it.
__device__ __forceinline__ int opaque(int x)
{
    asm volatile("" : "+v"(x));
    return x;
}

// The row to gather for a key slot.  A slot without a key holds ~f, f being a position of the same sample that
// some row of the tile may attend to: its rows are finite whenever the tile's real rows are, so the zero weights
// the bitmap gives the slot never meet a non-finite operand (pad rows may hold anything).
__device__ __forceinline__ int gather_row(int slot_value) { return slot_value ^ (slot_value >> 31); }

// What is gathered of an entry's positions besides the rows of two tensors: nothing, the two components of an array of float
// pairs, or the rows of a third tensor and one float each.
enum class Aux { NONE, PAIRS, THIRD };

// LEAN: the gather's per-lane offsets are computed anew for every tile instead of being held in registers throughout
template <int D, Aux AUX, typename G, bool LEAN = false>
struct Pipe {
    static constexpr int BM = G::BM, BN = G::BN, NW = G::NW;
    static constexpr int S = 2;                       // data stages in the ring
    static constexpr int PS = 2;                      // position stages: one being read, one on its way
    static constexpr int KSTEPS = D / 16;             // MFMA steps over the head dimension
    static constexpr int DBLK = D / 32;               // 32-wide blocks of the head dimension
    static constexpr int ROWB = D * 2;                // bytes per LDS row (unpadded)
    static constexpr int CPR = D / 8;                 // 16-byte chunks per row
    static constexpr int TILE = BN * ROWB;            // bytes of one gathered tile of one tensor
    static constexpr int RPI = 1024 / ROWB;           // rows per wave-level load
    static constexpr int LPW = BN / NW;               // rows of a tile each wave loads (16)
    static constexpr int NI = LPW / RPI;              // wave-level loads per tensor per tile per wave
    static constexpr int POSW = 64;                   // ints per position buffer (one wave-level load; BN are used)
    static constexpr int DATA_BYTES = S * 2 * TILE;
    static constexpr int POS_BYTES = PS * NW * POSW * 4;
    static constexpr int AUX_BYTES = AUX != Aux::NONE ? S * NW * POSW * 4 : 0;
    static constexpr int THIRD_AT = DATA_BYTES + POS_BYTES + AUX_BYTES;  // tiles of the third tensor, by stage
    static constexpr int SMEM_BYTES = THIRD_AT + (AUX == Aux::THIRD ? S * TILE : 0);

    char *smem;
    uint32_t smem_addr;
    int wave, lane;
    const int32_t *keys;       // key positions of this row tile's entries: [n][BN]
    const __bf16 *a, *b;       // the two gathered tensors, already offset to this (sample, head)
    const float *aux0, *aux1;  // per-position floats gathered with the rows: the two halves of an array of float pairs, hence
                               // 8 bytes from one position to the next; or an array of floats (aux0)
    const __bf16 *c;           // the third tensor

    __device__ __forceinline__ const char *tile_a(int stage) const { return smem + (stage * 2 + 0) * TILE; }
    __device__ __forceinline__ const char *tile_b(int stage) const { return smem + (stage * 2 + 1) * TILE; }
    __device__ __forceinline__ const int *pos_buf(int ps) const
    {
        return reinterpret_cast<const int *>(smem + DATA_BYTES) + (ps * NW + wave) * POSW;
    }
    __device__ __forceinline__ const char *tile_c(int stage) const { return smem + THIRD_AT + stage * TILE; }
    // aux values of the 64 slots: of pairs, array 0 is written by wave 0, array 1 by wave 1; of floats, every wave has a copy
    __device__ __forceinline__ const float *aux_buf(int stage, int which) const
    {
        return reinterpret_cast<const float *>(smem + DATA_BYTES + POS_BYTES) + (stage * NW + which) * POSW;
    }

    // start loading the key positions of the row tile's j-th entry (every wave keeps its own copy)
    __device__ __forceinline__ void issue_pos(int j, int ps) const
    {
        // (64 lanes load; with BN = 32 the upper half repeats the lower one)
        dma4(keys + j * BN, (uint32_t)(lane & (BN - 1)) * 4u, smem_addr + DATA_BYTES + ((ps * NW + wave) * POSW) * 4);
    }

    // where the rows of an entry whose positions sit in position stage ps are, relative to a and b (and aux0, aux1): all
    // positions are read before anything is made of them, so that one wait covers the reads
    struct Offsets {
        uint32_t row[NI], aux;
    };
    __device__ __forceinline__ Offsets offsets(int ps) const
    {
        const int *pb = pos_buf(ps);
        const int ol = LEAN ? opaque(lane) : lane, lr = ol / CPR, c = ol % CPR;  // row inside the wave-level load, chunk slot
        int pos[NI], pos_aux = 0;
#pragma unroll
        for (int i = 0; i < NI; i++) pos[i] = pb[wave * LPW + i * RPI + lr];
        if (AUX != Aux::NONE) pos_aux = pb[ol & (BN - 1)];
        Offsets o;
#pragma unroll
        for (int i = 0; i < NI; i++) {
            const int r = wave * LPW + i * RPI + lr;
            o.row[i] = (uint32_t)gather_row(pos[i]) * ROWB + (uint32_t)((c ^ swz<CPR>(r)) * 16);  // bytes
        }
        o.aux = AUX != Aux::NONE ? (uint32_t)gather_row(pos_aux) * (AUX == Aux::PAIRS ? 8u : 4u) : 0u;
        return o;
    }
    // start gathering them into ring stage `stage`
    __device__ __forceinline__ void issue_data(int stage, const Offsets &o) const
    {
#pragma unroll
        for (int i = 0; i < NI; i++) {
            const uint32_t dst = (uint32_t)((wave * LPW + i * RPI) * ROWB);
            dma16(a, o.row[i], smem_addr + (stage * 2 + 0) * TILE + dst);
            dma16(b, o.row[i], smem_addr + (stage * 2 + 1) * TILE + dst);
            if (AUX == Aux::THIRD) dma16(c, o.row[i], smem_addr + THIRD_AT + stage * TILE + dst);
        }
        if (AUX != Aux::NONE) {
            const float *src = AUX == Aux::PAIRS && (wave & 1) ? aux1 : aux0;
            dma4(src, o.aux, smem_addr + DATA_BYTES + POS_BYTES + ((stage * NW + wave) * POSW) * 4);
        }
    }
};

// Ring schedule (two stages; positions run one tile ahead of their rows).  Per wave the vector-memory
// instructions are issued in the order  pos(0), pos(1), data(0), pos(2), data(1), ..., pos(j+1), data(j), ...
//   start(n), prologue(n): start pos(0), pos(1); and data(0)
//   top(i):            call at the top of iteration i: waits until data(i) and pos(i+1) have landed in LDS for this
//                      wave and returns where the rows of data(i+1) are (every wave reads its own copy of the
//                      positions, so this needs no barrier); the caller then executes a workgroup barrier
//   advance(i, n, o):  after the barrier: starts pos(i+2) and data(i+1), whose rows are at o
// A third stage does not pay: in the backward at head size 64 the dQ role had one and is as fast or faster without (dense
// cross-attention 190 -> 183 us, 8192 positions on 64 x 32 tiles 80.9 -> 80.4, on 128 x 64 91.4 -> 90.5; nowhere slower by
// more than 0.3 %), and in the dK/dV role it takes registers that cost a wave per SIMD (81 -> 101).
template <typename P>
struct Ring {
    static constexpr int S = P::S, PS = P::PS;
    static_assert(S == 2, "the waits are those of two stages");

    // first half of the prologue.  The caller may issue its own (compiler-scheduled)
    // loads after this and before prologue(); the compiler's wait for those also covers these two.
    static __device__ __forceinline__ void start(const P &p, int n)
    {
        if (n > 0) p.issue_pos(0, 0);
        if (n > 1) p.issue_pos(1, 1);
    }

    // second half
    static __device__ __forceinline__ void prologue(const P &p, int n)
    {
        if (n > 0) {
            if (n > 1) wait_vmcnt<1>(); else wait_vmcnt<0>();  // pos(0) must have landed; issued after it: [pos(1)]
            p.issue_data(0, p.offsets(0));
        }
    }

    static __device__ __forceinline__ typename P::Offsets top(const P &p, int i)
    {
        wait_vmcnt<0>();
        return p.offsets((i + 1) % PS);  // (read, and not used, also where there is no such entry)
    }

    static __device__ __forceinline__ void advance(const P &p, int i, int n, const typename P::Offsets &o)
    {
        if (i + 2 < n) p.issue_pos(i + 2, (i + 2) % PS);
        if (i + 1 < n) p.issue_data((i + 1) % S, o);
    }
};

// A wave's own 32 rows of a [n_pos][D] tensor (rows row0 + 32*wave .. +31, clamped to n_pos-1; with an index, the rows
// it names), loaded straight into LDS as rows 32*wave .. of a swizzled tile at byte offset lds_off: full rows per
// 8 or 16 lanes, so every 128-byte line is fetched once.  The MFMA B fragments of those rows are
// then read back with read_row().  Issues 32/RPI vector-memory instructions.
template <typename P>
struct OwnRows {
    int g[32 / P::RPI];  // the row this lane loads 16 bytes of, per instruction
};
template <typename P>
__device__ __forceinline__ OwnRows<P> own_rows(const P &p, int row0, int n_pos, const int32_t *index = nullptr)
{
    OwnRows<P> o;
    const int lr = p.lane / P::CPR;
#pragma unroll
    for (int i = 0; i < 32 / P::RPI; i++) {
        const int g = min(row0 + p.wave * 32 + i * P::RPI + lr, n_pos - 1);
        o.g[i] = index ? index[g] : g;
    }
    return o;
}
template <typename P>
__device__ __forceinline__ void stage_own_rows(const P &p, const __bf16 *t, const OwnRows<P> &rows, uint32_t lds_off)
{
    const int lr = p.lane / P::CPR, c = p.lane % P::CPR;
#pragma unroll
    for (int i = 0; i < 32 / P::RPI; i++) {
        const int r = p.wave * 32 + i * P::RPI + lr;
        dma16(t, (uint32_t)rows.g[i] * P::ROWB + (uint32_t)((c ^ swz<P::CPR>(r)) * 16),
              p.smem_addr + lds_off + (uint32_t)((p.wave * 32 + i * P::RPI) * P::ROWB));
    }
}

// An accumulator block of zeros by a contraction of zeros: the matrix pipe, which has time to spare, writes the 16 registers
// where 16 moves would take the vector pipe's.
__device__ __forceinline__ f32x16 zero_block()
{
    s16x8 z = {0, 0, 0, 0, 0, 0, 0, 0};
    asm volatile("" : "+v"(z));  // (a value of its own per block: equal blocks would be made once and copied)
    const bf16x8 zb = __builtin_bit_cast(bf16x8, z);
    f32x16 c;
#pragma unroll
    for (int e = 0; e < 16; e++) c[e] = 0.f;
    return mfma_32x32x16(zb, zb, c);
}

// Epilogue: a wave's 32 x D accumulator block, held transposed in C fragments (lane (row l%32, hf)
// holds columns 32j + 4hf + 8g + 0..3), is scaled, rounded to bf16, transposed through a wave-private
// LDS area of 32*ROWB bytes and written to global memory as full rows (16 bytes per lane): row r of the block to row r
// of dst, or with an index (in LDS) to row index[r].  Row r keeps chunk c at c ^ (r & 7): with the area aligned to a row, that
// is one exclusive-or per write, and a wave-level store covers 1024 consecutive bytes of dst, an offset of the one before.
template <typename P, int D>
__device__ __forceinline__ void store_rows_via_lds(char *wave_lds, int lane, const f32x16 (&acc)[D / 32], float mult,
                                                   __bf16 *dst, int rows_valid, const int *index = nullptr)
{
    const int r = lane & 31, hf = lane >> 5;
    const uint32_t at0 = lds_addr(wave_lds) + (uint32_t)(r * P::ROWB + ((r & 7) << 4) + hf * 8);
#pragma unroll
    for (int j = 0; j < D / 32; j++)
#pragma unroll
        for (int gq = 0; gq < 4; gq++) {
            bf16x4 w;
#pragma unroll
            for (int e = 0; e < 4; e++) w[e] = (__bf16)(acc[j][gq * 4 + e] * mult);
            const int cl = j * 4 + gq;  // 16-byte chunk holding columns 32j + 8gq .. +7
            *(HDT_LDS bf16x4 *)(uintptr_t)((at0 ^ ((cl & 7) << 4)) + (cl >> 3) * 128) = w;
        }
    const int lr = lane / P::CPR, c = lane % P::CPR;
    auto chunk = [&](int i) {
        const int row = i * P::RPI + lr;
        return *reinterpret_cast<const u32x4 *>(wave_lds + i * 1024 + lr * P::ROWB + ((c ^ (row & 7)) << 4));
    };
    // streaming stores: results are not read again by this launch and should not displace its inputs in L2
    if (index == nullptr && rows_valid >= 32) {
        char *to = reinterpret_cast<char *>(dst);
        const uint32_t off = (uint32_t)lane * 16u;
#pragma unroll
        for (int i = 0; i < 32 / P::RPI; i++) __builtin_nontemporal_store(chunk(i), reinterpret_cast<u32x4 *>(to + i * 1024 + off));
        return;
    }
#pragma unroll
    for (int i = 0; i < 32 / P::RPI; i++) {
        const int row = i * P::RPI + lr;
        if (row < rows_valid) {
            const int at = index ? index[row] : row;
            __builtin_nontemporal_store(chunk(i), reinterpret_cast<u32x4 *>(dst + (size_t)at * D + c * 8));
        }
    }
}

// Per-lane constants for reading MFMA A operands by rows out of a swizzled tile: the lane's row
// inside a 32-row block and its swizzle term; 16-byte chunk 2*st + hf of that row sits at
// ((2*st) ^ x) * 16.
struct RowLane {
    int row;  // l % 32
    int x;    // hf ^ swz(row)
};
template <int CPR>
__device__ __forceinline__ RowLane row_lane(int lane)
{
    RowLane r;
    r.row = lane & 31;
    r.x = (lane >> 5) ^ swz<CPR>(r.row);
    return r;
}
template <int ROWB>
__device__ __forceinline__ bf16x8 read_row(const char *tile, const RowLane &r, int r0, int st)
{
    return lds_read_8(tile + (r0 + r.row) * ROWB + ((((st << 1) ^ r.x)) << 4));
}

// Per-lane constants of the transposing reads of a 32(k) x 32(n) operand block out of a swizzled
// row-major tile: row of the first read and the swizzle term; the chunk of n-block i is (4i) ^ y.
struct TrLane {
    int row;   // (g>>1)*4 + (tl>>2)
    int y;     // ((g&1)*2 + ((tl&3)>>1)) ^ swz(row)
    int half;  // (tl & 1) * 8 bytes inside the chunk
};
template <int CPR>
__device__ __forceinline__ TrLane tr_lane(int lane)
{
    const int g = lane >> 4, tl = lane & 15;
    TrLane t;
    t.row = (g >> 1) * 4 + (tl >> 2);
    t.y = (((g & 1) << 1) | ((tl & 3) >> 1)) ^ swz<CPR>(t.row);
    t.half = (tl & 1) * 8;
    return t;
}
// the 8 contraction values {k0 + hf*4 + 0..3} and {k0 + 8 + hf*4 + 0..3} at n = 32*i + l%32 (k0 a multiple of 16:
// the rows of the second read sit 8 further down, where the swizzle differs by 2)
template <int ROWB>
__device__ __forceinline__ bf16x8 read_tr(const char *tile, const TrLane &t, int k0, int i)
{
    const char *p0 = tile + (k0 + t.row) * ROWB + ((((i << 2) ^ t.y)) << 4) + t.half;
    const char *p1 = tile + (k0 + 8 + t.row) * ROWB + ((((i << 2) ^ t.y ^ 2)) << 4) + t.half;
    return lds_read_tr_8(p0, p1);
}

// Apply a 32x32 sub-block's bitmap to a C fragment: element e of lane l is kept iff bit l of
// mask[e] is set (the "register-major" bitmap the layout stores per sub-block), else replaced.
// The 16 masks are fetched with scalar loads (the address is the same for the whole wave; the
// layout is read-only while attention kernels run) and used directly as the lane masks of
// v_cndmask (a wave-uniform 64-bit value turned into a per-lane condition).
typedef const unsigned long long __attribute__((address_space(4))) hdt_cmask_t;

__device__ __forceinline__ void apply_mask(f32x16 &x, const unsigned long long *mask, float fill)
{
    hdt_cmask_t *cm = (hdt_cmask_t *)(uintptr_t)mask;
#pragma unroll
    for (int e = 0; e < 16; e++) x[e] = __builtin_amdgcn_inverse_ballot_w64(cm[e]) ? x[e] : fill;
}

// Asking for an entry's masks ahead of their use: one word of each 64-byte line of a wave's masks (WORDS 64-bit masks),
// requested in front of the wait for the entry's rows and looked at behind the barrier.  apply_mask's own loads then find
// the lines in the scalar cache; without this they are requested between two contractions and waited for on the spot, and
// they mostly come from beyond the L2 (a line is read by the few heads of a sample that share an XCD).
template <int WORDS>
struct MaskTouch {
    uint32_t w[WORDS / 8];
    __device__ __forceinline__ void request(const unsigned long long *mask)
    {
#pragma unroll
        for (int i = 0; i < WORDS / 8; i++) w[i] = as_const(reinterpret_cast<const uint32_t *>(mask))[i * 16];
    }
    __device__ __forceinline__ void arrived()
    {
#pragma unroll
        for (int i = 0; i < WORDS / 8; i++) asm volatile("" ::"s"(w[i]));
    }
};

}  // namespace hdt_tile
