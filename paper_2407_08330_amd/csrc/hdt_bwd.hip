// hdt_attn_bwd, bf16 MFMA kernels for gfx950.
//
// The paper gives no backward pass; these kernels evaluate the gradient of the definition in
// Sec. 3.2 (S = softmax(mask(Q K^T * scale)), O = S V) over the same surviving tiles the forward
// walks:  D_i = sum_c dO_ic O_ic,  P = exp(S - LSE),  dV = P^T dO,  dP = dO V^T,
//         dS = P o (dP - D),  dQ = scale dS K,  dK = scale dS^T Q.
//
// Deterministic, no atomics.  Two launches, or the second alone, whose roles then compute D themselves (roles_compute_d):
//   k_bwd_delta  D for every row (a streaming pass over O and dO).
//   k_bwd_bf16   two workgroups per row tile I (rows in document order), one per role, both with the
//                forward kernel's skeleton (hdt_tile.h):
//     dQ role      the tile's rows as QUERIES: walks their key tiles (the key positions of each list
//                  entry, gathered row by row), recomputes S^T and dP^T with queries along the MFMA
//                  columns (LSE_i and D_i are per-lane scalars) and accumulates dQ^T = K^T dS^T.
//     dK/dV role   the tile's rows as KEYS: walks the schedule of the TRANSPOSED mask.  The paper's mask
//                  is symmetric (i may attend to j iff j may attend to i: parent/child and sibling
//                  relations are mutual), so the entries of "query rows I x the keys they attend to" are
//                  also the entries of "key rows I x the queries attending to them", bitmaps included.
//                  K, V rows of the tile sit in registers; the Q and dO rows (and LSE, D) of an entry's
//                  QUERY positions are gathered into LDS and dV^T = dO^T P, dK^T = Q^T dS accumulate
//                  with keys along the MFMA columns.  Same load balance as the forward, no cross-wave
//                  reduction, contiguous stores.  For the directed variants (edge kinds without up/down
//                  symmetry) the layout holds a second schedule, built from the same ids with the
//                  parent and child kinds exchanged.
// Both roles recompute the scores, which costs two extra contractions but keeps dQ out of HBM as fp32
// partial sums.  Where a call of head size 128 does not fill the chip, the dK/dV role is split once more, into a dV role
// and a dK role (three workgroups per tile, see launch_bwd).  The workgroups of a tile are neighbours in the launch
// order and run on the same XCD at the same time.  That is what the pairing is for: the dQ role reads the tile's Q, dO
// rows and gathers K, V rows of the neighbourhood, the dK/dV role reads the tile's K, V rows and gathers Q, dO rows of the
// same neighbourhood, so each role finds in the XCD's L2 what the other (or a neighbouring pair) has just
// fetched, and Q, K, V, dO come from HBM once per backward pass instead of once per role (measured: the
// L2 fetch volume of this kernel is that of four tensors; as two separate passes it was that of eight).
#include "hdt_tile.h"

namespace {

using namespace hdt_tile;

template <int D>
struct BwdCfg {
    // waves per SIMD (register budget) of the kernel.  Three waves at head size
    // 64 pay on 128 x 64 tiles only (measured, config 4: 107 us against 122 with two; on 64 x 32 tiles 101
    // against 99 with two, whose allocation the compiler then leaves unconstrained).
    // The INDEXED form on 128 x 64 tiles is compiled for one wave less.  Bounded to the third, it spills 8 registers at head
    // size 64 where D comes from a pass, and takes longer (three waves - two, 1024 x 4096 x 16 heads 35.9 - 31.3 us, 2048 x
    // 8192 x 48 79.8 - 71.3); where the roles compute D it makes no difference (512 x 8192 x 48 24.1 - 24.0).  It gets two per
    // SIMD (175 registers at head size 64, 247 at 128); at head size 128 with the split roles only, see launch_bwd.
    template <typename G, bool INDEXED>
    static constexpr int WAVES = G::BM == 128 ? (D == 64 ? 3 : 2) - (INDEXED ? 1 : 0) : 2;
};

// ---------------------------------------------------------------------------------------- D
// For all rows of [rows][D] tensors: D_i = sum_c dO_ic O_ic (every lane multiplies 8 values, 16 bytes of each
// tensor; the lanes of a row are added up; kDeltaRows rows per lane in flight).  Bound by reading the two: O, which
// nothing behind this pass wants, by streaming (non-temporal) loads, so that dO, which the main kernel reads next, is still
// in the caches then.  32768 positions x 16 heads of 128, pass + main kernel: plain loads, 4 rows 49.2 + 220.7 us;
// streaming O 45.0 + 218.3 (2 rows 44.4, 8 rows 46.1: 6.0 TB/s), dO too 44.4 + 220.4.  What the main kernel wants of a row
// are the two values its contractions start from, so those are what is written, side by side:
//   .x = -D_i            dP - D        = -D + dO V^T          (accumulator of dP preset to it)
//   .y = -LSE_i / scale  scale S - LSE = scale (-LSE / scale + Q K^T)   (accumulator of S preset to it)
// which takes a subtraction and a multiplication per score out of both roles.  Rows without a key (LSE = -inf:
// pads) get 0 for both: they are masked, and their dO may hold anything.
// The sum is taken the same way wherever it is taken, here or in the roles (WITH_D): 8 columns by dot_8, then neighbours
// in pairs, pairs of pairs, and so on, so that the results of a backward do not depend on which of the two computes D.
constexpr int kDeltaRows = 2;
template <int D>
__global__ __launch_bounds__(256) void k_bwd_delta(const __bf16 *__restrict__ o, const __bf16 *__restrict__ d_o,
                                                   const float *__restrict__ lse, float inv_scale,
                                                   float2 *__restrict__ row_scalars, long long rows)
{
    constexpr int CPR = D / 8, RPB = 256 / CPR, kRows = kDeltaRows;
    const int lr = threadIdx.x / CPR, c = threadIdx.x % CPR;
    const long long r0 = (long long)blockIdx.x * (RPB * kRows) + lr;
    bf16x8 a[kRows], b[kRows];
    float l[kRows];
#pragma unroll
    for (int u = 0; u < kRows; u++) {
        const long long r = min(r0 + (long long)u * RPB, rows - 1);
        a[u] = __builtin_nontemporal_load(reinterpret_cast<const bf16x8 *>(o + (size_t)r * D + c * 8));
        b[u] = *reinterpret_cast<const bf16x8 *>(d_o + (size_t)r * D + c * 8);
        l[u] = c == 0 ? lse[r] : 0.f;
    }
#pragma unroll
    for (int u = 0; u < kRows; u++) {
        float part = dot_8(a[u], b[u], 0.f);
#pragma unroll
        for (int m = 1; m < CPR; m <<= 1) part += __shfl_xor(part, m);
        const long long r = r0 + (long long)u * RPB;
        if (c == 0 && r < rows) {
            const bool dead = l[u] == -INFINITY;
            row_scalars[r] = dead ? make_float2(0.f, 0.f) : make_float2(-part, -l[u] * inv_scale);
        }
    }
}

// ------------------------------------------------------------------------------------------- dQ
// WITH_D: the rows' D is computed here, see k_bwd_bf16.  Own rows of O have a place of their own behind the ring.
template <int D, typename G, bool WITH_D>
struct DqLds {
    using P = Pipe<D, Aux::NONE, G>;
    static constexpr int O_AT = (P::SMEM_BYTES + 255) / 256 * 256;
    static constexpr int BYTES = WITH_D ? O_AT + G::BM * P::ROWB : P::SMEM_BYTES;
};

template <int D, typename G, bool WITH_D>
__device__ __forceinline__ void dq_role(char *smem, const HdtSchedule &s, const __bf16 *__restrict__ q,
                                         const __bf16 *__restrict__ k, const __bf16 *__restrict__ v,
                                         const __bf16 *__restrict__ o, const float *__restrict__ lse,
                                         const __bf16 *__restrict__ d_o, const float2 *__restrict__ row_scalars,
                                         __bf16 *__restrict__ dq, int wave, int I, int bh, int b, float scale,
                                         float inv_scale)
{
    using P = Pipe<D, Aux::NONE, G>;
    using R = Ring<P>;
    constexpr int BM = G::BM, BN = G::BN, KB = G::KB;
    constexpr int ROWB = P::ROWB, KSTEPS = P::KSTEPS, DBLK = P::DBLK, S = P::S;

    const int lane = threadIdx.x & 63;
    const int qn = lane & 31;
    const int I_own = I % s.tr_own;  // the rows this tile works on (several tiles share them when key lists are cut)
    const size_t base = (size_t)bh * s.n_pos * D, own_base = (size_t)bh * s.n_own * D, kv_base = (size_t)bh * s.n_kv * D;
    const float scale_log2 = scale * LOG2E;

    const size_t row = (size_t)b * s.tr + I;
    const cptr_i32 range = as_const(s.q_range);
    const int t0 = range[2 * row], n = range[2 * row + 1] - t0;
    const cptr_u32 subs = as_const(s.q_sub) + t0;

    P pipe;
    pipe.smem = smem;
    pipe.smem_addr = lds_addr(smem);
    pipe.wave = wave;
    pipe.lane = lane;
    pipe.keys = s.q_keys + (size_t)t0 * BN;
    pipe.a = k + kv_base;
    pipe.b = v + kv_base;
    pipe.aux0 = pipe.aux1 = nullptr;
    const int qrow = I_own * BM + wave * 32 + qn;
    const RowLane rl = row_lane<P::CPR>(lane);
    const TrLane tl = tr_lane<P::CPR>(lane);

    // Q and dO rows of this wave go through the two ring stages (full-row loads into LDS); the B fragments are read back
    // from there.  The ring may only take the stages over after a barrier.
    constexpr uint32_t STG_Q = 2 * P::TILE, STG_DO = 0;
    const OwnRows<P> own = own_rows(pipe, I_own * BM, s.n_own);
    stage_own_rows(pipe, q + own_base, own, STG_Q);
    stage_own_rows(pipe, d_o + own_base, own, STG_DO);
    constexpr uint32_t STG_O = DqLds<D, G, WITH_D>::O_AT;
    if (WITH_D) stage_own_rows(pipe, o + own_base, own, STG_O);
    R::start(pipe, n);
    wait_vmcnt<0>();
    bf16x8 qf[KSTEPS], dof[KSTEPS];
#pragma unroll
    for (int st = 0; st < KSTEPS; st++) {
        qf[st] = read_row<ROWB>(smem + STG_Q, rl, wave * 32, st);
        dof[st] = read_row<ROWB>(smem + STG_DO, rl, wave * 32, st);
    }
    const int qrow_ld = min(qrow, s.n_own - 1);
    const float lse_i = lse[(size_t)bh * s.n_own + qrow_ld];
    float dp_init, s_init;  // -D_i, -LSE_i / scale; 0, 0 for a row without a key
    if (WITH_D) {
        float part[KSTEPS];  // 8 columns from this half-wave, the next 8 from the other
#pragma unroll
        for (int st = 0; st < KSTEPS; st++) {
            part[st] = dot_8(dof[st], read_row<ROWB>(smem + STG_O, rl, wave * 32, st), 0.f);
            part[st] += __shfl_xor(part[st], 32);
        }
#pragma unroll
        for (int m = 1; m < KSTEPS; m <<= 1)
#pragma unroll
            for (int st = 0; st < KSTEPS; st += 2 * m) part[st] += part[st + m];
        dp_init = lse_i == -INFINITY ? 0.f : -part[0];
        s_init = lse_i == -INFINITY ? 0.f : -lse_i * inv_scale;
    } else {
        const float2 init = row_scalars[(size_t)bh * s.n_own + qrow_ld];
        dp_init = init.x;
        s_init = init.y;
    }
    // A row without any key (a pad: LSE = -inf) is masked by the bitmap, but its Q and dO may hold anything,
    // NaN included, which a zero weight would not remove: it takes part as a row of zeros.
    const bool dead_row = lse_i == -INFINITY;
    if (dead_row) {
#pragma unroll
        for (int st = 0; st < KSTEPS; st++) qf[st] = dof[st] = zero_bf16x8();
    }
    // the compiler must finish its own loads before the hand-scheduled ones continue
    asm volatile("" ::"v"(dp_init), "v"(s_init), "v"(lse_i));
    wg_barrier();  // every wave has read its fragments: the ring may use all stages
    R::prologue(pipe, n);

    f32x16 dqacc[DBLK];
#pragma unroll
    for (int i = 0; i < DBLK; i++) dqacc[i] = zero_block();

    uint32_t sub_next = n > 0 ? subs[0] : 0u;
    for (int i = 0; i < n; i++) {
        const uint32_t sub = sub_next;
        const int bidx = t0 + i;  // bitmaps are stored in list order
        if (i + 1 < n) {
            sub_next = subs[i + 1];
        }
        const typename P::Offsets next = R::top(pipe, i);
        wg_barrier();
        R::advance(pipe, i, n, next);
        const char *sK = pipe.tile_a(i % S), *sV = pipe.tile_b(i % S);

#pragma unroll
        for (int kb = 0; kb < KB; kb++) {
            const int sb = wave * KB + kb;
            if (!((sub >> sb) & 1u)) continue;
            f32x16 sacc, dpacc;  // every element of a lane belongs to the lane's query
#pragma unroll
            for (int e = 0; e < 16; e++) {
                sacc[e] = s_init;
                dpacc[e] = dp_init;
            }
            // (a wave at its contractions goes before the waves of this SIMD that are at their exponentials: the
            // kernel is 3 % faster with the priorities than with the round-robin order)
            __builtin_amdgcn_s_setprio(1);
#pragma unroll
            for (int st = 0; st < KSTEPS; st++) {
                sacc = mfma_32x32x16(read_row<ROWB>(sK, rl, kb * 32, st), qf[st], sacc);     // K Q^T - LSE / scale
                dpacc = mfma_32x32x16(read_row<ROWB>(sV, rl, kb * 32, st), dof[st], dpacc);  // dP^T - D = V dO^T - D
            }
            __builtin_amdgcn_s_setprio(0);
#pragma unroll
            for (int e = 0; e < 16; e++) sacc[e] = fast_exp2(sacc[e] * scale_log2);  // P^T
            if (!((sub >> (16 + sb)) & 1u)) apply_mask(sacc, s.bits_rm + ((size_t)bidx * G::NSUB + sb) * 16, 0.f);
#pragma unroll
            for (int e = 0; e < 16; e++) sacc[e] *= dpacc[e];  // dS^T
            // dQ^T += K^T dS^T
            const bf16x8 b0 = pack_bf16x8(sacc, 0), b1 = pack_bf16x8(sacc, 8);
            __builtin_amdgcn_s_setprio(1);
#pragma unroll
            for (int j = 0; j < DBLK; j++) {
                dqacc[j] = mfma_32x32x16(read_tr<ROWB>(sK, tl, kb * 32, j), b0, dqacc[j]);
                dqacc[j] = mfma_32x32x16(read_tr<ROWB>(sK, tl, kb * 32 + 16, j), b1, dqacc[j]);
            }
            __builtin_amdgcn_s_setprio(0);
        }
    }

    {
        // through this wave's slice of the stage tile n would have used: free since the last barrier (see
        // the forward kernel), so waves leave independently
        const int wrow0 = I * BM + wave * 32;
        store_rows_via_lds<P, D>(smem + (n % S) * 2 * P::TILE + wave * 32 * ROWB, opaque(lane), dqacc, scale,
                                 dq + base + (size_t)wrow0 * D, s.n_pos - wrow0);
    }
}

// ---------------------------------------------------------------------------------------- dK, dV
// WHICH: 0 = dK and dV, 1 = dV only, 2 = dK only.  INDEXED: the rows are those own_index names (see HdtSchedule).
// WITH_D: O and LSE of an entry's queries are gathered with Q and dO, and the workgroup computes D when they have landed.
template <int D, typename G, int WHICH, bool INDEXED, bool WITH_D>
struct DkvLds {
    static constexpr bool LEAN = D == 128 && WHICH == 0;
    using P = Pipe<D, WITH_D ? Aux::THIRD : Aux::PAIRS, G, LEAN>;
    static constexpr int ROW_AT = P::SMEM_BYTES, INIT_AT = ROW_AT + (INDEXED ? G::BM * 4 : 0);
    static constexpr int BYTES = INIT_AT + (WITH_D ? 2 * G::BN * 4 : 0);
};
template <int D, typename G, int WHICH, bool INDEXED, bool WITH_D>
__device__ __forceinline__ void dkv_role(char *smem, const HdtSchedule &s, const __bf16 *__restrict__ q,
                                          const __bf16 *__restrict__ k, const __bf16 *__restrict__ v,
                                          const __bf16 *__restrict__ o, const float *__restrict__ lse,
                                          const __bf16 *__restrict__ d_o, const float2 *__restrict__ row_scalars,
                                          __bf16 *__restrict__ dk, __bf16 *__restrict__ dv, int wave, int I, int bh,
                                          int b, float scale, float inv_scale)
{
    // Head size 128 and both results: 128 accumulator and 64 operand registers leave 64 of the 256 a wave gets at two per
    // SIMD.  What can be computed anew per entry or sub-block from the lane number is (LEAN): held in registers throughout
    // the loop, as the compiler would have it, 30 to 56 registers did not fit.
    using Lds = DkvLds<D, G, WHICH, INDEXED, WITH_D>;
    constexpr bool LEAN = Lds::LEAN;
    using P = typename Lds::P;
    using R = Ring<P>;
    constexpr int BM = G::BM, BN = G::BN, KB = G::KB;
    constexpr int ROWB = P::ROWB, KSTEPS = P::KSTEPS, DBLK = P::DBLK, S = P::S;
    constexpr bool DO_DV = WHICH != 2, DO_DK = WHICH != 1;

    const int lane = threadIdx.x & 63;
    const int hf = lane >> 5;
    const size_t q_base = (size_t)bh * s.n_kv * D;  // rows are keys here
    const size_t base = (size_t)bh * (INDEXED ? s.own_stride : s.n_pos) * D;
    const int n_rows = INDEXED ? as_const(s.own_count)[b] : s.n_pos;
    const int32_t *index = INDEXED ? s.own_index + (size_t)b * s.own_stride : nullptr;
    if (INDEXED && I * BM >= n_rows) return;  // the whole workgroup: no visible position in this tile
    const float scale_log2 = scale * LOG2E;

    const size_t row = (size_t)b * (INDEXED ? s.own_tiles : s.tr) + I;
    const cptr_i32 range = as_const(s.q_range);
    const int t0 = range[2 * row], n = range[2 * row + 1] - t0;
    const cptr_u32 subs = as_const(s.q_sub) + t0;

    P pipe;
    pipe.smem = smem;
    pipe.smem_addr = lds_addr(smem);
    pipe.wave = wave;
    pipe.lane = lane;
    pipe.keys = s.q_keys + (size_t)t0 * BN;
    pipe.a = q + q_base;
    pipe.b = d_o + q_base;
    if (WITH_D) {
        pipe.aux0 = pipe.aux1 = lse + (size_t)bh * s.n_kv;
        pipe.c = o + q_base;
    } else {
        pipe.aux0 = reinterpret_cast<const float *>(row_scalars + (size_t)bh * s.n_kv) + 1;  // -LSE / scale of a position
        pipe.aux1 = reinterpret_cast<const float *>(row_scalars + (size_t)bh * s.n_kv);      // -D
    }
    const RowLane own_rl = row_lane<P::CPR>(lane);
    // is this lane's own row a real position?  (Requested first, looked at once the rows are in registers.)
    // (An unconditional load: inside a branch the compiler would wait for it on the spot.  Without flags any
    // readable word will do, its value is not used.)
    const int own_row = min(I * BM + wave * 32 + (lane & 31), s.n_pos - 1);
    const int32_t *flag_at = s.row_flag ? s.row_flag + ((size_t)b * s.n_pos + own_row) : s.q_range;
    int own_flag = *flag_at;

    // K and V rows of this wave: through the two ring stages, as Q and dO in the dQ pass
    constexpr uint32_t STG_K = 2 * P::TILE, STG_V = 0;
    const OwnRows<P> own = own_rows(pipe, I * BM, n_rows, index);
    // where this wave's rows go: kept in LDS until the epilogue (registers are short, scalar ones included)
    int *row_at = reinterpret_cast<int *>(smem + Lds::ROW_AT) + wave * 32;
    if (INDEXED && lane % P::CPR == 0) {
#pragma unroll
        for (int i = 0; i < 32 / P::RPI; i++) row_at[i * P::RPI + lane / P::CPR] = own.g[i];
    }
    stage_own_rows(pipe, k + base, own, STG_K);
    if (DO_DK) stage_own_rows(pipe, v + base, own, STG_V);  // V only enters dP
    R::start(pipe, n);
    wait_vmcnt<0>();
    bf16x8 kf[KSTEPS], vf[KSTEPS];
#pragma unroll
    for (int st = 0; st < KSTEPS; st++) {
        kf[st] = read_row<ROWB>(smem + STG_K, own_rl, wave * 32, st);
        if (DO_DK) vf[st] = read_row<ROWB>(smem + STG_V, own_rl, wave * 32, st);
    }
    // A row that is no real position (a pad, an encoder position the decoder does not see) is masked by the
    // bitmap, but its K and V may hold anything, NaN included, which a zero weight would not remove: it takes
    // part as a row of zeros.
    if (s.row_flag != nullptr && own_flag < 0) {
#pragma unroll
        for (int st = 0; st < KSTEPS; st++) {
            kf[st] = zero_bf16x8();
            if (DO_DK) vf[st] = zero_bf16x8();
        }
    }
    wg_barrier();
    R::prologue(pipe, n);

    f32x16 dkacc[DBLK], dvacc[DBLK];
#pragma unroll
    for (int i = 0; i < DBLK; i++) {
        if (DO_DK) dkacc[i] = zero_block();
        if (DO_DV) dvacc[i] = zero_block();
    }

    uint32_t sub_next = n > 0 ? subs[0] : 0u;
    for (int i = 0; i < n; i++) {
        const uint32_t sub = sub_next;
        const int bidx = t0 + i;  // bitmaps are stored in list order
        if (i + 1 < n) {
            sub_next = subs[i + 1];
        }
        const typename P::Offsets next = R::top(pipe, i);
        wg_barrier();
        R::advance(pipe, i, n, next);
        const char *sQ = pipe.tile_a(i % S), *sDO = pipe.tile_b(i % S);
        // -LSE / scale, -D of the entry's queries
        float *init = reinterpret_cast<float *>(smem + Lds::INIT_AT);
        const float *sInitS = WITH_D ? init : pipe.aux_buf(i % S, 0), *sInitDP = WITH_D ? init + BN : pipe.aux_buf(i % S, 1);
        if (WITH_D) {
            static_assert(!WITH_D || WHICH == 0, "D is computed where both results are");
            // four lanes per query, a quarter of the columns each
            const int t = wave * 64 + opaque(lane), r = t >> 2, quarter = t & 3;
            const float lse_r = pipe.aux_buf(i % S, wave)[r];
            float part[P::CPR / 4];
#pragma unroll
            for (int u = 0; u < P::CPR / 4; u++) {
                const int at = r * ROWB + (((quarter * (P::CPR / 4) + u) ^ swz<P::CPR>(r)) << 4);
                part[u] = dot_8(lds_read_8(sDO + at), lds_read_8(pipe.tile_c(i % S) + at), 0.f);
            }
#pragma unroll
            for (int m = 1; m < P::CPR / 4; m <<= 1)
#pragma unroll
                for (int u = 0; u < P::CPR / 4; u += 2 * m) part[u] += part[u + m];
            float d = part[0];
            d += __builtin_bit_cast(float, __builtin_amdgcn_mov_dpp(__builtin_bit_cast(int, d), 0xb1, 0xf, 0xf, true));  // lane ^ 1
            d += __builtin_bit_cast(float, __builtin_amdgcn_mov_dpp(__builtin_bit_cast(int, d), 0x4e, 0xf, 0xf, true));  // lane ^ 2
            if (quarter == 0) {
                init[r] = lse_r == -INFINITY ? 0.f : -lse_r * inv_scale;
                init[BN + r] = lse_r == -INFINITY ? 0.f : -d;
            }
            wg_barrier();  // (the next entry's values come behind its own first barrier)
        }

#pragma unroll
        for (int kb = 0; kb < KB; kb++) {  // 32 query slots
            const int sb = wave * KB + kb;
            if (!((sub >> sb) & 1u)) continue;
            const int ol = LEAN ? opaque(lane) : lane;
            const RowLane rl = row_lane<P::CPR>(ol);
            const TrLane tl = tr_lane<P::CPR>(ol);
            // element gq * 4 + e of a lane belongs to the query in slot kb * 32 + hf * 4 + gq * 8 + e
            f32x16 sacc, dpacc;
#pragma unroll
            for (int gq = 0; gq < 4; gq++) {
                const float4 l4 = *reinterpret_cast<const float4 *>(&sInitS[kb * 32 + hf * 4 + gq * 8]);
                sacc[gq * 4 + 0] = l4.x;
                sacc[gq * 4 + 1] = l4.y;
                sacc[gq * 4 + 2] = l4.z;
                sacc[gq * 4 + 3] = l4.w;
                if (DO_DK) {
                    const float4 d4 = *reinterpret_cast<const float4 *>(&sInitDP[kb * 32 + hf * 4 + gq * 8]);
                    dpacc[gq * 4 + 0] = d4.x;
                    dpacc[gq * 4 + 1] = d4.y;
                    dpacc[gq * 4 + 2] = d4.z;
                    dpacc[gq * 4 + 3] = d4.w;
                }
            }
            __builtin_amdgcn_s_setprio(1);  // as in the dQ role
#pragma unroll
            for (int st = 0; st < KSTEPS; st++) {
                sacc = mfma_32x32x16(read_row<ROWB>(sQ, rl, kb * 32, st), kf[st], sacc);     // Q K^T - LSE / scale
                if (DO_DK) dpacc = mfma_32x32x16(read_row<ROWB>(sDO, rl, kb * 32, st), vf[st], dpacc);  // dO V^T - D
            }
            __builtin_amdgcn_s_setprio(0);
            f32x16 pacc;
#pragma unroll
            for (int e = 0; e < 16; e++) pacc[e] = fast_exp2(sacc[e] * scale_log2);  // P
            if (!((sub >> (16 + sb)) & 1u)) apply_mask(pacc, s.bits_rm + ((size_t)bidx * G::NSUB + sb) * 16, 0.f);
            if (DO_DK) {
#pragma unroll
                for (int e = 0; e < 16; e++) sacc[e] = pacc[e] * dpacc[e];  // dS
                const bf16x8 s0 = pack_bf16x8(sacc, 0), s1 = pack_bf16x8(sacc, 8);
                __builtin_amdgcn_s_setprio(1);
#pragma unroll
                for (int j = 0; j < DBLK; j++) {
                    dkacc[j] = mfma_32x32x16(read_tr<ROWB>(sQ, tl, kb * 32, j), s0, dkacc[j]);  // dK^T += Q^T dS
                    dkacc[j] = mfma_32x32x16(read_tr<ROWB>(sQ, tl, kb * 32 + 16, j), s1, dkacc[j]);
                }
            }
            if (DO_DV) {
                const bf16x8 p0 = pack_bf16x8(pacc, 0), p1 = pack_bf16x8(pacc, 8);
                __builtin_amdgcn_s_setprio(1);
#pragma unroll
                for (int j = 0; j < DBLK; j++) {
                    dvacc[j] = mfma_32x32x16(read_tr<ROWB>(sDO, tl, kb * 32, j), p0, dvacc[j]);  // dV^T += dO^T P
                    dvacc[j] = mfma_32x32x16(read_tr<ROWB>(sDO, tl, kb * 32 + 16, j), p1, dvacc[j]);
                }
            }
            __builtin_amdgcn_s_setprio(0);
        }
    }

    {
        // through this wave's slice of the stage tile n would have used: free since the last barrier
        const int wrow0 = I * BM + wave * 32;
        char *wl = smem + (n % S) * 2 * P::TILE + wave * 32 * ROWB;
        const int le = opaque(lane);
        const size_t at = base + (INDEXED ? 0 : (size_t)wrow0 * D);
        const int *to = INDEXED ? row_at : nullptr;
        if (DO_DK) store_rows_via_lds<P, D>(wl, le, dkacc, scale, dk + at, n_rows - wrow0, to);
        if (DO_DV) store_rows_via_lds<P, D>(wl, le, dvacc, 1.f, dv + at, n_rows - wrow0, to);
    }
}

// ---------------------------------------------------------------------------------------- zeros
// dK, dV rows of the positions an INDEXED schedule does not cover: workgroup z writes kZeroChunks 16-byte chunks per
// thread and tensor.  They ride in the same launch: with few positions visible the other workgroups leave most of the
// chip idle and last about as long as writing the zeros takes.
constexpr int kZeroChunks = 8;
template <int D, typename G>
struct ZeroRows {
    static constexpr int ROWS = kZeroChunks * G::THREADS / (D / 8);  // rows of a tensor per workgroup
};
template <int D, typename G>
__device__ __forceinline__ void zero_role(const HdtSchedule &s, __bf16 *__restrict__ dk, __bf16 *__restrict__ dv, unsigned z,
                                          int heads)
{
    constexpr int CPR = D / 8, ROWS = ZeroRows<D, G>::ROWS;
    const unsigned per = ((unsigned)s.own_stride + ROWS - 1u) / ROWS;
    const int bh = z / per, b = bh / heads, p0 = (z % per) * ROWS;
    const int32_t *rank = s.own_rank + (size_t)b * s.own_stride;
    int r[kZeroChunks];
#pragma unroll
    for (int u = 0; u < kZeroChunks; u++) {
        const int p = p0 + (u * G::THREADS + (int)threadIdx.x) / CPR;
        r[u] = p < s.own_stride ? rank[p] : 0;
    }
    const u32x4 zero = {0u, 0u, 0u, 0u};
#pragma unroll
    for (int u = 0; u < kZeroChunks; u++) {
        const size_t at = ((size_t)bh * s.own_stride + p0) * CPR + u * G::THREADS + threadIdx.x;
        if (r[u] < 0) {
            __builtin_nontemporal_store(zero, reinterpret_cast<u32x4 *>(dk) + at);
            __builtin_nontemporal_store(zero, reinterpret_cast<u32x4 *>(dv) + at);
        }
    }
}

// The grid of the roles: workgroups of the tiles both sides have, then those of the longer side's rest (padding included), and
// what logical_block deals out at a time in each.  In dense cross-attention the two kinds of workgroup last differently
// long: spread evenly as one row of items, some XCDs get a chunk more of the longer ones.  Whole backward of full chunks
// of both - one row spread evenly - each part by itself: 2048 x 2048 x 48 heads, 128 x 64 tiles, 225 - 246 - 216 us;
// 512 x 8192 x 48, 64 x 32 tiles, 224 - 236 - 217; 512 x 8192 x 8, 128 x 64, 54.7 - 45.2 - 41.3.
struct RoleGrid {
    unsigned tiles, rest;
    FastDiv chunk, rest_chunk;
    unsigned nq, nk;          // row tiles of the two sides, all samples and heads
    FastDiv tr_q, tr_k, heads;
};
template <typename G>
static RoleGrid role_grid(const HdtSchedule &s, const HdtSchedule &s_tr, int heads, unsigned roles)
{
    RoleGrid g;
    g.nq = (unsigned)s.batch * heads * s.tr;
    g.nk = (unsigned)s_tr.batch * heads * s_tr.tr;
    const unsigned nq = g.nq, nk = g.nk, common = nq < nk ? nq : nk, unit = nq > nk ? 1u : roles - 1u;
    const unsigned rest = nq + (roles - 1u) * nk - roles * common;
    g.chunk = FastDiv(xcd_chunk(roles * common, roles * G::XCD_CHUNK, roles));
    g.tiles = padded_grid(roles * common, g.chunk.d);
    g.rest_chunk = FastDiv(xcd_chunk(rest, unit * G::XCD_CHUNK, unit));
    g.rest = padded_grid(rest, g.rest_chunk.d);
    g.tr_q = FastDiv(s.tr);
    g.tr_k = FastDiv(s_tr.tr);
    g.heads = FastDiv(heads);
    return g;
}

// SPLIT: a dV and a dK role instead of one for both.  INDEXED: s_tr covers visible positions only
// (HdtSchedule::own_index); the workgroups behind the grid of the roles write the zeros of the rows it leaves out.
template <int D, typename G, bool INDEXED, bool SPLIT, bool WITH_D>
__global__ __launch_bounds__(G::THREADS, (BwdCfg<D>::template WAVES<G, INDEXED>)) void k_bwd_bf16(
    HdtSchedule s, HdtSchedule s_tr, const __bf16 *__restrict__ q, const __bf16 *__restrict__ k,
    const __bf16 *__restrict__ v, const __bf16 *__restrict__ o, const float *__restrict__ lse,
    const __bf16 *__restrict__ d_o, const float2 *__restrict__ row_scalars, __bf16 *__restrict__ dq,
    __bf16 *__restrict__ dk, __bf16 *__restrict__ dv, float scale, float inv_scale, RoleGrid grid)
{
    constexpr int SMEM_Q = DqLds<D, G, WITH_D>::BYTES, SMEM_K = DkvLds<D, G, SPLIT ? 2 : 0, INDEXED, WITH_D>::BYTES;
    constexpr int SMEM = SMEM_Q > SMEM_K ? SMEM_Q : SMEM_K;
    __shared__ __attribute__((aligned(1024))) char smem[SMEM];
    const int wave = __builtin_amdgcn_readfirstlane((int)threadIdx.x >> 6);
    // The roles tile different tensors (the same ones for self-attention): the workgroups of one tile follow each
    // other as far as both sides have that tile, the rest of the longer side comes behind them, each of the two spread
    // evenly over the XCDs by itself (see role_grid).
    constexpr unsigned R = SPLIT ? 3u : 2u;  // roles per tile: dQ, then dK/dV or dV, dK
    const unsigned nq = grid.nq, nk = grid.nk;
    const unsigned common = nq < nk ? nq : nk, items = nq + (R - 1u) * nk;
    unsigned w;
    if (blockIdx.x < grid.tiles) {
        w = logical_block(blockIdx.x, grid.chunk);
        if (w >= R * common) return;  // padding of the grid
    } else {
        const unsigned at = blockIdx.x - grid.tiles;
        if (INDEXED && at >= grid.rest) {
            zero_role<D, G>(s_tr, dk, dv, at - grid.rest, grid.heads.d);
            return;
        }
        w = R * common + logical_block(at, grid.rest_chunk);
        if (w >= items) return;
    }
    unsigned role, lb;
    if (w < R * common) {
        role = w % R;
        lb = w / R;
    } else if (nq > nk) {
        role = 0u;
        lb = w - (R - 1u) * common;
    } else {
        const unsigned rest = w - R * common;
        role = 1u + rest % (R - 1u);
        lb = common + rest / (R - 1u);
    }
    if (role == 0u) {
        const int bh = grid.tr_q.div(lb), I = lb - bh * grid.tr_q.d, b = grid.heads.div(bh);
        dq_role<D, G, WITH_D>(smem, s, q, k, v, o, lse, d_o, row_scalars, dq, wave, I, bh, b, scale, inv_scale);
    } else {
        const int bh = grid.tr_k.div(lb), I = lb - bh * grid.tr_k.d, b = grid.heads.div(bh);
        if constexpr (!SPLIT)
            dkv_role<D, G, 0, INDEXED, WITH_D>(smem, s_tr, q, k, v, o, lse, d_o, row_scalars, dk, dv, wave, I, bh, b, scale, inv_scale);
        else if (role == 1u)
            dkv_role<D, G, 1, INDEXED, WITH_D>(smem, s_tr, q, k, v, o, lse, d_o, row_scalars, dk, dv, wave, I, bh, b, scale, inv_scale);
        else
            dkv_role<D, G, 2, INDEXED, WITH_D>(smem, s_tr, q, k, v, o, lse, d_o, row_scalars, dk, dv, wave, I, bh, b, scale, inv_scale);
    }
}

}  // namespace

template <int D, typename G, bool INDEXED, bool SPLIT, bool WITH_D>
static void launch_kernel(const HdtSchedule &s, const HdtSchedule &s_tr, const __bf16 *Q, const __bf16 *K, const __bf16 *V,
                          const __bf16 *O, const float *lse, const __bf16 *DO, const float2 *row_scalars, void *dq, void *dk, void *dv,
                          int heads, float scale, hipStream_t st)
{
    constexpr unsigned roles = SPLIT ? 3u : 2u, zr = ZeroRows<D, G>::ROWS;
    const unsigned zeros = INDEXED ? (unsigned)s_tr.batch * heads * (((unsigned)s_tr.own_stride + zr - 1u) / zr) : 0u;
    const RoleGrid g = role_grid<G>(s, s_tr, heads, roles);
    dim3 grid(g.tiles + g.rest + zeros), block(G::THREADS);
    hipLaunchKernelGGL((k_bwd_bf16<D, G, INDEXED, SPLIT, WITH_D>), grid, block, 0, st, s, s_tr, Q, K, V, O, lse, DO, row_scalars,
                       (__bf16 *)dq, (__bf16 *)dk, (__bf16 *)dv, scale, 1.f / scale, g);
}

// Whether the roles compute D themselves (head size 64), from what the host knows.  What that saves is a launch (about 2 us in
// a graph, 4 outside) and a pass over O and dO; what it costs is D of a query once per list entry that names it, and a barrier
// and a third more rows per entry.  So it pays for short lists.  Either way D is the same to the last bit, so the choice shows
// in nothing but the time.  hipGraphs, time with the roles over time with the pass:
//   Self-attention, forward and backward on several sets of tensors in turn (what a layer finds is not in the caches), documents
//   with other sentences, 6 K to 524 K rows (batch x heads x positions).  64 x 32 tiles, keys a list on average: 120-155
//   0.90-0.99 (8192 x 4 x 12 140.4 - 138.1 us), 158-169 0.96-0.99, 174 1.02, 187-200 0.98-1.03, 209-220 1.00-1.04 (1 x 32768 x 16
//   227.6 - 236.2); 128 x 64: 192-248 0.91-0.99, 252-292 0.96-1.00, 300-310 0.97-1.01.  Again on one set, part of which the caches
//   hold, the lines lie at about 180 and 320 keys below 200 K rows, 155 and 270 beyond (8192 x 4 x 12, 64 x 32, 163 keys 140.3 -
//   142.2).  ListOps-shaped trees (30-190 keys) 0.72-0.97 of the backward, hundreds of siblings up to 1.22.  (A
//   deferred build whose report is not in counts as the last one of its shape that has reported.)
//   Cross-attention: every row tile with a visible row lists all decoder rows, and while there are few tiles the time is that of
//   one walk along a list.  Lists of 2, 4, 6, 8, 10 and 12 entries 0.83, 0.91, 0.96, 0.97-1.01, 1.02 and 1.04 (128 x 64: 128 to 768
//   decoder rows; 512 x 8192 x 48, 750 visible, 26 - 24 us), on 64 x 32 tiles 0.81, 0.85, 0.91, 0.93-0.98, 1.00 and 1.04 (64 to
//   384).  Full grids stop paying earlier, after about so many (list entry, head) pairs as stand below for lists of 8
//   entries: 128 x 64, 6 entries 1.03 at 4608 pairs (50 - 51 us), 4 entries 0.98 at 4096; 64 x 32, 8 entries 0.96-0.98 at 3072
//   and 1.01 at 4096, 4 entries 0.99 at 6144.
// At head size 128 the third tensor's tiles cost a workgroup per compute unit (16384 positions x 16 heads 136 - 157).
template <typename G>
static bool roles_compute_d(const HdtSchedule &s_tr, int heads, HdtLists lists)
{
    constexpr bool SMALL = G::BM == 64;
    const long long tiles = (long long)s_tr.batch * s_tr.tr;
    if (!lists.cross) {
        const long long entries = lists.entries >= 0 ? lists.entries : tiles * s_tr.tc;  // (not known: as long as they can be)
        return entries * G::BN <= tiles * (SMALL ? 170 : 290);
    }
    const long long list = (s_tr.n_kv + G::BN - 1) / G::BN, pairs = tiles * list * heads;
    return list <= 8 && pairs <= (SMALL ? 8000 : 5000) && pairs * list <= 8 * (SMALL ? 3100 : 2100);
}

// At head size 128 one role for dK and dV is less work than two (the scores are computed twice instead of three times,
// and the rows gathered), two are the shorter chain.  Two as long as their workgroups, two waves per SIMD, are all on the
// chip at the same time; measured, one role / two: 32768 positions x 16 heads 230 / 261 us (64 x 32 tiles) and 264 / 307
// (128 x 64); 3000 x 16 (2 samples x 8 heads) 33.4 / 33.2 and 37.1 / 37.0; 1000 x 4 heads 16.9 / 14.3.
// Always two where the rows are indexed and the tiles 128 x 64: one role takes 307 registers there, a single wave per SIMD
// (whole backward, one role / two: 512 x 8192 x 48 heads, 500 positions visible, 68.9 / 61.3 us, 750 81.3 / 68.6, 2000
// 185 / 130; 2048 x 8192 x 64 heads, 2000 visible, 716 / 540).  On 64 x 32 tiles it keeps two.
template <int D, typename G, bool INDEXED>
static void launch_bwd(const HdtSchedule &s, const HdtSchedule &s_tr, const __bf16 *Q, const __bf16 *K, const __bf16 *V,
                       const __bf16 *O, const float *lse, const __bf16 *DO, void *dq, void *dk, void *dv, int heads,
                       float scale, float *delta, HdtLists lists, hipStream_t st)
{
    // the rows' two scalars (-D, -LSE / scale), see hdt_bwd_row_scalars_bytes for the room they take
    float2 *row_scalars = reinterpret_cast<float2 *>(delta);
    if constexpr (D == 64) {
        if (roles_compute_d<G>(s_tr, heads, lists)) {
            HdtTimer t("hdt_bwd_bf16_d64", st);
            launch_kernel<D, G, INDEXED, false, true>(s, s_tr, Q, K, V, O, lse, DO, nullptr, dq, dk, dv, heads, scale, st);
            return;
        }
    }
    {
        const long long rows = (long long)s.batch * heads * s.n_own;  // the real rows, also when key lists are cut
        HdtTimer t(D == 64 ? "hdt_bwd_delta_d64" : "hdt_bwd_delta_d128", st);
        const int rpb = (256 / (D / 8)) * kDeltaRows;
        hipLaunchKernelGGL(k_bwd_delta<D>, dim3((unsigned)((rows + rpb - 1) / rpb)), dim3(256), 0, st, O, DO, lse, 1.f / scale,
                           row_scalars, rows);
    }
    HdtTimer t(D == 64 ? "hdt_bwd_bf16_d64" : "hdt_bwd_bf16_d128", st);
    constexpr unsigned kResident = 256u * 8u / G::NW;  // workgroups on the chip at two waves per SIMD
    const size_t nq = (size_t)s.batch * heads * s.tr, nk = (size_t)s_tr.batch * heads * s_tr.tr;
    constexpr bool ALWAYS = D == 128 && INDEXED && G::BM == 128;
    if (ALWAYS || (D == 128 && nq + 2 * nk <= kResident))
        launch_kernel<D, G, INDEXED, D == 128, false>(s, s_tr, Q, K, V, O, lse, DO, row_scalars, dq, dk, dv, heads, scale, st);
    else
        launch_kernel<D, G, INDEXED, ALWAYS, false>(s, s_tr, Q, K, V, O, lse, DO, row_scalars, dq, dk, dv, heads, scale, st);
}

template <typename G>
static void launch_shape(const HdtSchedule &s, const HdtSchedule &s_tr, const __bf16 *Q, const __bf16 *K, const __bf16 *V,
                         const __bf16 *O, const float *lse, const __bf16 *DO, void *dq, void *dk, void *dv, int heads,
                         int head_dim, float scale, float *delta, HdtLists lists, hipStream_t st)
{
    if (head_dim == 64)
        s_tr.own_index ? launch_bwd<64, G, true>(s, s_tr, Q, K, V, O, lse, DO, dq, dk, dv, heads, scale, delta, lists, st)
                       : launch_bwd<64, G, false>(s, s_tr, Q, K, V, O, lse, DO, dq, dk, dv, heads, scale, delta, lists, st);
    else
        s_tr.own_index ? launch_bwd<128, G, true>(s, s_tr, Q, K, V, O, lse, DO, dq, dk, dv, heads, scale, delta, lists, st)
                       : launch_bwd<128, G, false>(s, s_tr, Q, K, V, O, lse, DO, dq, dk, dv, heads, scale, delta, lists, st);
}

hdt_status_t hdt_launch_bwd_bf16(const HdtSchedule &s, const HdtSchedule &st_, const void *q, const void *k,
                                 const void *v, const void *o, const float *lse, const void *d_o, void *dq, void *dk,
                                 void *dv, int heads, int head_dim, float scale, float *delta, HdtLists lists,
                                 hipStream_t st)
{
    const __bf16 *Q = (const __bf16 *)q, *K = (const __bf16 *)k, *V = (const __bf16 *)v;
    const __bf16 *O = (const __bf16 *)o, *DO = (const __bf16 *)d_o;
    if (s.bm == 64)
        launch_shape<Geo<64, 32>>(s, st_, Q, K, V, O, lse, DO, dq, dk, dv, heads, head_dim, scale, delta, lists, st);
    else
        launch_shape<Geo<128, 64>>(s, st_, Q, K, V, O, lse, DO, dq, dk, dv, heads, head_dim, scale, delta, lists, st);
    HDT_HIP_TRY(hipGetLastError());
    return HDT_OK;
}
