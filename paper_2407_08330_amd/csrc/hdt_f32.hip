// fp32 debugging path: the same tile schedule walked with plain fp32 arithmetic, pair by pair.  It exists to check the
// schedule, the mask bitmaps and the online softmax separately from the MFMA kernels: a pair the mask does not allow
// never enters any arithmetic.
// Forward: App. A.1, Alg. 1 (online softmax over the surviving tiles).  Backward: gradient of
// the definition in Sec. 3.2.
//
// What bounds these kernels on the tiny documents they are meant for is the length of a row's dependent chain, so a
// whole wave works on one row: it packs the positions the row may attend to out of the bitmaps, 256 slots at a time,
// and takes 16 of them per step (four groups of 16 lanes, four keys per group in flight; a lane holds 4 columns of
// each 64, so a gathered row is read once, coalesced, and serves the dot product as well as the accumulation).
// Measured on one document of 512 positions, one head, head size 64 (one thread per row before): forward 205 ->
// 7.7 us, dQ, dK and dV 230 + 252 -> 8.6 us in one launch.
#include "hdt_internal.h"

namespace {

constexpr int kRows = 4;     // rows (waves) per workgroup
constexpr int kSlots = 256;  // key slots looked at per round
constexpr int kUnroll = 4;   // keys per group of 16 lanes and step

__device__ __forceinline__ float add_ror(float x, int y) { return x + __builtin_bit_cast(float, y); }
// sum over the 16 lanes of a group, in every lane of it
__device__ __forceinline__ float group_sum(float x)
{
#define ROR(n) __builtin_amdgcn_update_dpp(0, __builtin_bit_cast(int, x), 0x120 + (n), 0xf, 0xf, true)
    x = add_ror(x, ROR(8));
    x = add_ror(x, ROR(4));
    x = add_ror(x, ROR(2));
    x = add_ror(x, ROR(1));
#undef ROR
    return x;
}
__device__ __forceinline__ float across_groups(float x)  // sum over the four groups
{
    x += __shfl_xor(x, 16);
    return x + __shfl_xor(x, 32);
}

// a lane's share of one row: columns 64 f + 4 c .. + 3
template <int D>
struct Part {
    static constexpr int F = D / 64;
    float4 x[F];
    __device__ __forceinline__ void load(const float *row, int c)
    {
#pragma unroll
        for (int f = 0; f < F; f++) x[f] = *reinterpret_cast<const float4 *>(row + 64 * f + 4 * c);
    }
    __device__ __forceinline__ void fill(float v)
    {
#pragma unroll
        for (int f = 0; f < F; f++) x[f] = make_float4(v, v, v, v);
    }
    __device__ __forceinline__ float dot(const Part &o) const  // over the whole row
    {
        float s = 0.f;
#pragma unroll
        for (int f = 0; f < F; f++)
            s = fmaf(x[f].w, o.x[f].w, fmaf(x[f].z, o.x[f].z, fmaf(x[f].y, o.x[f].y, fmaf(x[f].x, o.x[f].x, s))));
        return group_sum(s);
    }
    __device__ __forceinline__ void scale(float w)
    {
#pragma unroll
        for (int f = 0; f < F; f++) x[f].x *= w, x[f].y *= w, x[f].z *= w, x[f].w *= w;
    }
    __device__ __forceinline__ void add(float w, const Part &o)
    {
#pragma unroll
        for (int f = 0; f < F; f++) {
            x[f].x = fmaf(w, o.x[f].x, x[f].x);
            x[f].y = fmaf(w, o.x[f].y, x[f].y);
            x[f].z = fmaf(w, o.x[f].z, x[f].z);
            x[f].w = fmaf(w, o.x[f].w, x[f].w);
        }
    }
    // the groups' partial sums added up and written by the first group
    __device__ __forceinline__ void store_sum(float *row, int c, int g, float w)
    {
#pragma unroll
        for (int f = 0; f < F; f++) {
            const float4 t = make_float4(across_groups(x[f].x) * w, across_groups(x[f].y) * w, across_groups(x[f].z) * w,
                                         across_groups(x[f].w) * w);
            if (g == 0) *reinterpret_cast<float4 *>(row + 64 * f + 4 * c) = t;
        }
    }
};

// Calls step(position[kUnroll], ok[kUnroll]) for the keys of row i of sample b, kUnroll of them per group of lanes at a
// time; a position without ok repeats another key of the row.  `list`: this wave's kSlots ints of LDS.
template <typename Step>
__device__ __forceinline__ void for_keys(const HdtSchedule &s, int b, int i, int *list, Step step)
{
    const int lane = threadIdx.x & 63, g = lane >> 4;
    const int I = i / s.bm, r = i - I * s.bm;
    const size_t row = (size_t)b * s.tr + I, nsub = (size_t)(s.bm >> 5) * s.wpr;
    const int t0 = s.q_range[2 * row], total = (s.q_range[2 * row + 1] - t0) * s.bn;
    for (int s0 = 0; s0 < total; s0 += kSlots) {
        unsigned long long word[kSlots / 64];
        int pos[kSlots / 64], bit[kSlots / 64];
#pragma unroll
        for (int u = 0; u < kSlots / 64; u++) {
            const int at = s0 + u * 64 + lane, slot = at < total ? at : 0;
            const int e = slot / s.bn, c = slot - e * s.bn;
            const size_t t = (size_t)(t0 + e);
            // the indexing of hdt_pair_allowed, with the load apart from the test
            word[u] = s.bits_rm[(t * nsub + (size_t)(r >> 5) * s.wpr + (c >> 5)) * 16 + (((c & 31) >> 3) * 4 + (c & 3))];
            bit[u] = (r & 31) + 32 * ((c >> 2) & 1);
            pos[u] = at < total ? s.q_keys[t * s.bn + c] : -1;
        }
        int n = 0;
#pragma unroll
        for (int u = 0; u < kSlots / 64; u++) {
            const bool ok = pos[u] >= 0 && ((word[u] >> bit[u]) & 1ull);
            const unsigned long long m = __ballot(ok);
            if (ok) list[n + __popcll(m & ((1ull << lane) - 1ull))] = pos[u];
            n += __popcll(m);
        }
        asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");  // the wave's own list: no barrier
        for (int k0 = 0; k0 < n; k0 += 4 * kUnroll) {
            int p[kUnroll];
            bool ok[kUnroll];
#pragma unroll
            for (int u = 0; u < kUnroll; u++) {
                const int k = k0 + 4 * u + g;
                ok[u] = k < n;
                p[u] = list[ok[u] ? k : n - 1];
            }
            step(p, ok);
        }
        asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
    }
}

template <int D>
__global__ __launch_bounds__(64 * kRows) void k_fwd_f32(HdtSchedule s, const float *__restrict__ q,
                                                        const float *__restrict__ k, const float *__restrict__ v,
                                                        float *__restrict__ o, float *__restrict__ lse, int heads,
                                                        float scale)
{
    __shared__ int s_list[kRows][kSlots];
    const int wave = threadIdx.x >> 6, lane = threadIdx.x & 63, g = lane >> 4, c = lane & 15;
    const int i = blockIdx.x * kRows + wave, bh = blockIdx.y, b = bh / heads;
    if (i >= s.n_pos) return;
    const size_t base = (size_t)bh * s.n_pos * D, kv_base = (size_t)bh * s.n_kv * D;
    Part<D> qi, acc;
    qi.load(q + base + (size_t)i * D, c);
    acc.fill(0.f);
    float m = -INFINITY, l = 0.f;  // of this group's keys
    for_keys(s, b, i, s_list[wave], [&](const int (&p)[kUnroll], const bool (&ok)[kUnroll]) {
        Part<D> kj[kUnroll], vj[kUnroll];
#pragma unroll
        for (int u = 0; u < kUnroll; u++) {
            kj[u].load(k + kv_base + (size_t)p[u] * D, c);
            vj[u].load(v + kv_base + (size_t)p[u] * D, c);
        }
        float sc[kUnroll], m_new = m;
#pragma unroll
        for (int u = 0; u < kUnroll; u++) {
            sc[u] = ok[u] ? qi.dot(kj[u]) * scale : -INFINITY;
            m_new = fmaxf(m_new, sc[u]);
        }
        const float m_sub = m_new == -INFINITY ? 0.f : m_new;  // no key in this group so far
        const float alpha = expf(m - m_sub);                   // m = -inf -> 0
        acc.scale(alpha);
        l *= alpha;
        m = m_new;
#pragma unroll
        for (int u = 0; u < kUnroll; u++) {
            const float w = expf(sc[u] - m_sub);
            l += w;
            if (ok[u]) acc.add(w, vj[u]);
        }
    });
    const float m_all = fmaxf(fmaxf(m, __shfl_xor(m, 16)), fmaxf(__shfl_xor(m, 32), __shfl_xor(m, 48)));
    const float w = m_all == -INFINITY ? 0.f : expf(m - m_all);
    acc.scale(w);
    const float l_all = across_groups(l * w);
    acc.store_sum(o + base + (size_t)i * D, c, g, l_all > 0.f ? 1.f / l_all : 0.f);
    if (lane == 0) lse[(size_t)bh * s.n_pos + i] = l_all > 0.f ? m_all + logf(l_all) : -INFINITY;
}

// blockIdx.z = 0: dQ, a wave per query row.  blockIdx.z = 1: dK and dV, a wave per key row, which walks the schedule of
// the transposed mask (for the paper's symmetric mask the forward's own: the list of query tile I x key slots J is also
// the list of key rows I x query slots J with the same bitmaps; directed variants bring a second schedule) and gathers
// the query rows its entries name.  It computes their D = dO . O itself, a third dot product per pair: both roles then
// fit one launch (two launches of the sizes this path is for take longer than the arithmetic).
template <int D>
__global__ __launch_bounds__(64 * kRows) void k_bwd_f32(HdtSchedule sq, HdtSchedule sk, const float *__restrict__ q,
                                                        const float *__restrict__ k, const float *__restrict__ v,
                                                        const float *__restrict__ o, const float *__restrict__ lse,
                                                        const float *__restrict__ d_o, float *__restrict__ dq,
                                                        float *__restrict__ dk, float *__restrict__ dv, int heads,
                                                        float scale)
{
    __shared__ int s_list[kRows][kSlots];
    const int wave = threadIdx.x >> 6, lane = threadIdx.x & 63, g = lane >> 4, c = lane & 15;
    const int i = blockIdx.x * kRows + wave, bh = blockIdx.y, b = bh / heads;
    const HdtSchedule &s = blockIdx.z == 0 ? sq : sk;
    if (i >= s.n_pos) return;
    const size_t base = (size_t)bh * s.n_pos, far = (size_t)bh * s.n_kv;  // rows of this role, rows it gathers
    const size_t own = (base + i) * D;
    if (blockIdx.z == 0) {
        Part<D> qi, doi, oi, acc;
        qi.load(q + own, c);
        doi.load(d_o + own, c);
        oi.load(o + own, c);
        acc.fill(0.f);
        const float Di = doi.dot(oi), li = lse[base + i];
        for_keys(s, b, i, s_list[wave], [&](const int (&p)[kUnroll], const bool (&ok)[kUnroll]) {
            Part<D> kj[kUnroll], vj[kUnroll];
#pragma unroll
            for (int u = 0; u < kUnroll; u++) {
                kj[u].load(k + (far + p[u]) * D, c);
                vj[u].load(v + (far + p[u]) * D, c);
            }
#pragma unroll
            for (int u = 0; u < kUnroll; u++) {
                const float w = expf(qi.dot(kj[u]) * scale - li), dp = doi.dot(vj[u]);
                if (ok[u]) acc.add(w * (dp - Di) * scale, kj[u]);
            }
        });
        acc.store_sum(dq + own, c, g, 1.f);
    } else {
        Part<D> kj, vj, ak, av;
        kj.load(k + own, c);
        vj.load(v + own, c);
        ak.fill(0.f);
        av.fill(0.f);
        for_keys(s, b, i, s_list[wave], [&](const int (&p)[kUnroll], const bool (&ok)[kUnroll]) {
            Part<D> qi[kUnroll], doi[kUnroll], oi[kUnroll];
            float li[kUnroll];
#pragma unroll
            for (int u = 0; u < kUnroll; u++) {
                qi[u].load(q + (far + p[u]) * D, c);
                doi[u].load(d_o + (far + p[u]) * D, c);
                oi[u].load(o + (far + p[u]) * D, c);
                li[u] = lse[far + p[u]];
            }
#pragma unroll
            for (int u = 0; u < kUnroll; u++) {
                const float w = expf(kj.dot(qi[u]) * scale - li[u]), dp = vj.dot(doi[u]), Di = doi[u].dot(oi[u]);
                if (ok[u]) {
                    av.add(w, doi[u]);
                    ak.add(w * (dp - Di) * scale, qi[u]);
                }
            }
        });
        ak.store_sum(dk + own, c, g, 1.f);
        av.store_sum(dv + own, c, g, 1.f);
    }
}

}  // namespace

hdt_status_t hdt_launch_fwd_f32(const HdtSchedule &s, const float *q, const float *k, const float *v, float *o,
                                float *lse, int heads, int head_dim, float scale, hipStream_t st)
{
    if ((int64_t)s.batch * heads > 65535) return hdt_fail(HDT_ERR_SHAPE, "fp32 path: batch*heads > 65535");
    dim3 grid((s.n_pos + kRows - 1) / kRows, s.batch * heads), block(64 * kRows);
    HdtTimer t("hdt_fwd_f32", st);
    if (head_dim == 64)
        hipLaunchKernelGGL(k_fwd_f32<64>, grid, block, 0, st, s, q, k, v, o, lse, heads, scale);
    else
        hipLaunchKernelGGL(k_fwd_f32<128>, grid, block, 0, st, s, q, k, v, o, lse, heads, scale);
    HDT_HIP_TRY(hipGetLastError());
    return HDT_OK;
}

hdt_status_t hdt_launch_bwd_f32(const HdtSchedule &s, const HdtSchedule &st_, const float *q, const float *k, const float *v,
                                const float *o, const float *lse, const float *d_o, float *dq, float *dk,
                                float *dv, int heads, int head_dim, float scale, hipStream_t st)
{
    if ((int64_t)s.batch * heads > 65535) return hdt_fail(HDT_ERR_SHAPE, "fp32 path: batch*heads > 65535");
    const int rows = s.n_pos > st_.n_pos ? s.n_pos : st_.n_pos;
    dim3 grid((rows + kRows - 1) / kRows, s.batch * heads, 2), block(64 * kRows);
    HdtTimer t("hdt_bwd_f32", st);
    if (head_dim == 64)
        hipLaunchKernelGGL(k_bwd_f32<64>, grid, block, 0, st, s, st_, q, k, v, o, lse, d_o, dq, dk, dv, heads, scale);
    else
        hipLaunchKernelGGL(k_bwd_f32<128>, grid, block, 0, st, s, st_, q, k, v, o, lse, d_o, dq, dk, dv, heads, scale);
    HDT_HIP_TRY(hipGetLastError());
    return HDT_OK;
}
