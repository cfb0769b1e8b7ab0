// How the positional encoding's kernels divide the positions of a sample among workgroups, and which positions they read; how
// many workgroups per sample the cross-attention build takes.
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

// Workgroups per sample of the cross-attention build (hdt_cross.hip), whose waves take the sample's `entries` list entries in turn
// behind a scan of its levels, which takes as long as 1.5 entries of a wave and one more per batch of groups (80 us for 524288
// positions, 3 for 8192).  They run in rounds of one per compute unit: as many as
// a number of rounds has room for, and the number of rounds that makes the whole shortest.  One round wherever it can be one gave 129
// samples a workgroup each and left half of the chip idle, and 300 a second round that was nearly empty.  us, [SEC] / all tokens
// visible, one round - this rule - a kernel for the positions and one for the entries, in any number of workgroups: encoder of 8192,
// 512 decoder rows, 96 samples 58.6 / 69.5 - 51.1 / 57.8 - 56.1 / 69.8, 129 samples 106 / 130 - 70.9 / 81.0 - 72.3 / 91.0; 8192 and 64 rows, 129
// samples 26.6 / 35.1 - 23.9 / 28.4 - 23.5 / 28.9, 300 samples 46.1 / 60.3 - 41.1 / 50.1 - 42.4 / 52.9; 2048 and 512 rows, 129 samples
// 32.9 / 38.0 - 28.0 / 30.4 - 31.8 / 32.8, 300 samples 57.5 / 65.0 - 50.3 / 54.0 - 62.6 / 63.4; 32768 and 64 rows, 129 samples
// 83.3 / 114 - 64.4 / 81.7 - 60.1 / 82.2; 131072 and 64, 96 samples 166 / 240 - 154 / 212 - 164 / 257.
constexpr int kCrossBuildThreads = 1024, kCrossBuildBatch = 8;  // a wave's groups of 64 positions in flight
__host__ inline int cross_build_shares(int batch, int n_enc, long long entries)
{
    constexpr int kWaves = kCrossBuildThreads / 64, kScanned = kCrossBuildThreads * kCrossBuildBatch;
    const double scan = kWaves * (1.5 + (double)((n_enc + (kScanned - 1ll)) / kScanned));
    const long long most = entries > kWaves ? (entries + kWaves - 1) / kWaves : 1;  // a wave per entry
    const long long least = (batch + (kOnChip - 1ll)) / kOnChip;
    long long best = 1;
    double best_time = 0.;
    for (long long room = least; room < least + 6; room++) {
        const long long fit = room * kOnChip / batch, shares = fit < most ? fit : most;
        const long long rounds = (batch * shares + kOnChip - 1) / kOnChip;
        const double time = (double)rounds * (scan + (double)entries / (double)shares);
        if (room == least || time < best_time) {
            best = shares;
            best_time = time;
        }
        if (shares == most) break;
    }
    return (int)best;
}
