// The chunk schedule of a ragged batch on the device: prefix sums over the clips and the entry
// of a given chunk.  Used by the schedule kernels (melt_fwd.hip) and, for up to 64 clips, by the
// forward kernels and the comparator themselves: every workgroup needs a few entries only, and
// a wave finds them with the clips in its lanes in about the time it takes to read them from a
// table, so that no schedule kernel (3.5-8.6 us and its launch gap) runs before them.
#pragma once
#include "melt_internal.h"

namespace melt {

// The batch of a kernel that schedules itself (off = nullptr: it reads a chunk table).
struct ClipTable {
    const int64_t *off;    // device, n_clips + 1
    int n_clips, N, bf;    // clips (<= 64), frame length, frames per chunk
    int cap;               // chunks at most: those beyond it start past the output's last row
    Chunk *tab;            // where the entries and their count are left for the prepared calls, as a
    int *n_tab;            // table's kernel leaves them (nullptr: nowhere)
};

// a value that is the same on every lane, as a scalar
__device__ __forceinline__ int64_t uniform64(int64_t v) {
    const int lo = __builtin_amdgcn_readfirstlane((int)(v & 0xffffffff));
    const int hi = __builtin_amdgcn_readfirstlane((int)(v >> 32));
    return (int64_t)(((uint64_t)(unsigned)hi << 32) | (unsigned)lo);
}

// inclusive prefix sum over the 64 lanes of a wave (shuffles, no barrier)
__device__ __forceinline__ int64_t wave_scan(int64_t v, int lane) {
#pragma unroll
    for (int d = 1; d < 64; d <<= 1) {
        const int64_t u = __shfl_up(v, d, 64);
        if (lane >= d) v += u;
    }
    return v;
}

// a / b for 0 <= a, 0 < b < 2^31: 32-bit division when a fits (the 64-bit one is a long
// software sequence)
__device__ __forceinline__ int64_t udiv_nonneg(int64_t a, int b) {
    return a <= 0x7fffffff ? (int64_t)((uint32_t)a / (uint32_t)b) : a / b;
}

// At most 64 clips in the lanes of a wave (lane = clip): first sample, length, and the inclusive
// prefix sums of the frame and chunk counts.
struct ClipScan {
    int64_t st, L, pf, pc, total;      // total: chunks of the batch (every lane)
};
__device__ __forceinline__ ClipScan clip_scan(const int64_t *__restrict__ off, int n_clips, int N, int H, int bf) {
    const int lane = threadIdx.x & 63;
    ClipScan s{};
    if (lane < n_clips) {
        s.st = off[lane];
        s.L = off[lane + 1] - s.st;
    }
    const int64_t T = (s.L >= N) ? 1 + udiv_nonneg(s.L - N, H) : 0;
    s.pf = wave_scan(T, lane);
    s.pc = wave_scan(udiv_nonneg(T + bf - 1, bf), lane);
    s.total = __shfl(s.pc, 63, 64);
    return s;
}
// Entry q (its own in every lane; meaningless for q >= total) by a binary search over the
// lanes' chunk prefix sums.  Every lane must be active: a lane left out of a shuffle (by a
// condition) would read as zero to the lanes that source from it.
__device__ __forceinline__ Chunk clip_chunk(const ClipScan &s, int H, int bf, int64_t q) {
    int t = 0;                                              // clips whose chunks all precede q
#pragma unroll
    for (int d = 32; d >= 1; d >>= 1)
        if (__shfl(s.pc, t + d - 1, 64) <= q) t += d;
    const int tp = t > 0 ? t - 1 : 0;
    const int64_t pc_p = __shfl(s.pc, tp, 64), pf_p = __shfl(s.pf, tp, 64);
    const int64_t pf_t = __shfl(s.pf, t & 63, 64);
    const int64_t st_t = __shfl(s.st, t & 63, 64), L_t = __shfl(s.L, t & 63, 64);
    const int64_t fb = t > 0 ? pf_p : 0, k = q - (t > 0 ? pc_p : 0), Tt = pf_t - fb;
    Chunk e;
    e.sample_start = st_t + k * bf * (int64_t)H;
    e.sample_end = st_t + L_t;
    e.out_row = fb + k * bf;
    e.n_frames = (int)((Tt - k * bf) < bf ? (Tt - k * bf) : bf);
    e.clip = t;
    return e;
}

// A whole wave: the chunk count of the batch, and (store) entry c, each lane its own, into
// list[lane] for the first `count` lanes whose chunk exists.
__device__ __forceinline__ int chunk_list(const ClipTable &b, int H, int64_t c, int count, Chunk *list, bool store) {
    const int lane = threadIdx.x & 63;
    const ClipScan s = clip_scan(b.off, b.n_clips, b.N, H, b.bf);
    const Chunk e = clip_chunk(s, H, b.bf, c);
    const int n = (int)(s.total < b.cap ? s.total : b.cap);
    if (store && lane < count && c < n) list[lane] = e;
    return __builtin_amdgcn_readfirstlane(n);
}
// The same wave's entries into the batch's table, and the count (n) from workgroup 0.
__device__ __forceinline__ void leave_chunks(const ClipTable &b, int64_t c, int count, const Chunk *list, int n) {
    if (!b.tab) return;
    const int lane = threadIdx.x & 63;
    if (lane < count && c < n) b.tab[c] = list[lane];
    if (lane == 0 && (blockIdx.x | blockIdx.y | blockIdx.z) == 0) *b.n_tab = n;
}

constexpr int kListEntries = 64;       // a workgroup's own entries, one per lane of the wave that finds them

}  // namespace melt
