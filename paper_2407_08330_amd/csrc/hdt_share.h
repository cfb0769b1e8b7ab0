// How the positional encoding's kernels divide the positions of a sample among workgroups, and which positions they read.
// Index arithmetic alone, without any HIP header, so that a host program can walk through it.
#pragma once

constexpr int kOrdThreads = 1024;
constexpr int kMaxShares = 64;  // workgroups per sample
constexpr int kBack = 8;        // groups of 64 positions a wave has in flight while it looks at earlier positions

// Workgroups that are on the chip at the same time, one per compute unit (further ones only wait, see hdt_hpe.hip).
constexpr int kOnChip = 256;
__host__ inline int hpe_shares(int batch, int n)
{
    const int chunks = (n + kOrdThreads - 1) / kOrdThreads, fit = kOnChip / batch > 1 ? kOnChip / batch : 1;
    const int most = fit < kMaxShares ? fit : kMaxShares;
    return chunks < most ? chunks : most;
}

struct HpeShare {
    int first, last;  // positions [first, last) of the sample
    // Whole chunks go to the shares in turn, equally many to each, so the last shares may find none left (65 chunks in 64
    // shares of two): `first` then lies behind the sample's end, and nothing may be read relative to it.
    __host__ __device__ __forceinline__ bool empty() const { return first >= last; }
};
__host__ __device__ __forceinline__ HpeShare hpe_share(int k, int n, int shares)  // of the sample's k-th workgroup
{
    const int chunks = (n + kOrdThreads - 1) / kOrdThreads, per = (chunks + shares - 1) / shares;
    const int c0 = k * per < chunks ? k * per : chunks, c1 = c0 + per < chunks ? c0 + per : chunks;
    const int last = c1 * kOrdThreads < n ? c1 * kOrdThreads : n;
    return {c0 * kOrdThreads, last};
}
// Of the kBack * 1024 positions that end at `end`, which is the share's first or one in front of it: the u-th of thread `tid`
// (negative: none, as for every thread of an empty share).
__host__ __device__ __forceinline__ int hpe_position_in_front(const HpeShare &share, int end, int u, int tid)
{
    return share.empty() ? -1 : end - (u + 1) * kOrdThreads + tid;
}
