// The two products of the gradient on three bfloat16 planes per operand (melt_split.h explains
// the split; every FP32 operand is the exact sum of its planes, six of nine plane products, FP32
// accumulation).
//
//   dx  hop-block row b = sum_j G[b - j] W_j is the forward's product with G as the waveform
//       (hop 2M, J whole segments, read J - 1 rows back) and the basis columns as its rows, so it
//       runs on k_melt_split with a job of its own
//   dW  G^T X over frames: k_bwd_dw_split below
//
// Measured on 32 x 10 s at 22.05 kHz, N 1024, M 128 (27 456 frames, 14.4 GFLOP each; FP32 MFMA
// kernels before): dx 202 -> 80 us, dW 224 -> 104 us, a training step with its forward 617 ->
// 296 us.  Relative error against 64 bits: dx 7.9e-7 -> 6.5e-7,
// dW 7.8e-7 -> 5.2e-7.
#include "bwd.h"
#include "melt_split.h"

namespace melt {

// ------------------------------------------------------------------ dx

// Row chunks of G in, waveform gradient out.  a.wave = G, a.H = 2M; the row tiles are 16
// consecutive samples of a hop.
struct SplitDx {
    FwdArgs a;             // wave = G, out = dx, chunks = the RowChunk table
    SplitGeo g;            // basis: stacked [2M][N]
    int hop;
    __device__ __forceinline__ bool lists() const { return false; }
    __device__ __forceinline__ int start(Chunk *) const { return 0; }
    __device__ __forceinline__ SplitItem item(int w, int, const Chunk *, int SF) const {
        const int ci = w / (g.nsub * g.parts);
        const int f0 = ((w - ci * g.nsub * g.parts) / g.parts) * SF;
        static_assert(sizeof(RowChunk) == 40, "five int64 per entry");
        const int64_t g_row0 = split_scalar(a.chunks, 5 * (int64_t)ci + 2), nr_lo = split_scalar(a.chunks, 5 * (int64_t)ci + 3);
        const int t_hi = (int)split_scalar(a.chunks, 5 * (int64_t)ci + 4);
        const int n_rows = (int)nr_lo, t_lo = (int)(nr_lo >> 32);
        const int nf = max(min(SF, n_rows - f0), 0);
        // LDS row r holds G of the chunk's frame f0 + r - (J - 1); frames outside [t_lo, t_hi) of
        // the clip, or past n_frames, are zero
        const int64_t left = a.n_frames - g_row0;
        const int hi = left < t_hi ? (int)left : t_hi, back = a.J - 1 - f0;
        const int rows = nf + a.J - 1;
        const int r_lo = min(max(t_lo + back, 0), rows), r_hi = min(max(hi + back, 0), rows);
        const int64_t start = (g_row0 - back) * a.H;
        return {start, start + (int64_t)max(r_hi, r_lo) * a.H, (int64_t)ci * kSplitChunk + f0, nf, r_lo * a.H};
    }
    template <class Op, int FT, int RT>
    __device__ __forceinline__ void store(const SplitItem &it, int fbase, int lane, const int (&tile)[RT], f32x4 (&acc)[FT][RT]) const;
};

// four floats at any 4-byte address (the hop and the clips' starts may be odd)
typedef float f32x4_any __attribute__((ext_vector_type(4), aligned(4)));

// One sample of dx in plain FP32: hop-block row b of the chunk (item-local row i), column c.
__device__ __forceinline__ float dx_redo(const SplitDx &d, const SplitItem &it, int i, int c) {
    const int Q = d.a.H, J = d.a.J, M = Q / 2;
    float s = 0.0f;
#pragma unroll 1
    for (int j = 0; j < J; ++j) {
        const int64_t at = it.start + (int64_t)(i + J - 1 - j) * Q;
        if (at < it.start + it.lo || at >= it.end || j * d.hop + c >= d.g.N) continue;
#pragma unroll 1
        for (int q = 0; q < Q; ++q)
            s = fmaf(d.a.wave[at + q], d.g.basis[(size_t)((q & 1) * M + (q >> 1)) * d.g.N + j * d.hop + c], s);
    }
    return s;
}

template <class Op, int FT, int RT>
__device__ __forceinline__ void SplitDx::store(const SplitItem &it, int fbase, int lane, const int (&tile)[RT],
                                               f32x4 (&acc)[FT][RT]) const {
    asm volatile("" : "+v"(lane));
    const int q = lane >> 4, i0 = fbase + (lane & 15);
    const int64_t ci = it.out_row / kSplitChunk, f0 = it.out_row - ci * kSplitChunk;
    const int64_t s0 = split_scalar(a.chunks, 5 * ci) + f0 * hop, s_end = split_scalar(a.chunks, 5 * ci + 1);
    float probe = 0.0f;
#pragma unroll
    for (int f = 0; f < FT; ++f) {
        const int i = i0 + 16 * f;
        if (i >= it.nf) continue;
        const int64_t s = s0 + (int64_t)i * hop;
        float *o = a.out + s;
#pragma unroll
        for (int r = 0; r < RT; ++r) {
            const int c = 16 * tile[r] + 4 * q;
            const f32x4 y = acc[f][r];
            probe = fmaf(y[0] + y[1] + y[2] + y[3], 0.0f, probe);
            if (tile[r] >= g.T16) continue;
            if (c + 4 <= hop && s + c + 4 <= s_end) {
                *(f32x4_any *)(o + c) = y;
            } else {
#pragma unroll
                for (int e = 0; e < 4; ++e)
                    if (c + e < hop && s + c + e < s_end) o[c + e] = y[e];
            }
        }
    }
    if (__any(!(probe == 0.0f))) {
#pragma unroll 1
        for (int n = 0; n < FT * RT * 4; ++n) {
            const int e = n & 3, f = (n >> 2) / RT, r = (n >> 2) - f * RT;
            float y = 0.0f;
            int t = 0;
#pragma unroll
            for (int ff = 0; ff < FT; ++ff)
#pragma unroll
                for (int rr = 0; rr < RT; ++rr)
                    if (ff == f && rr == r) {
                        t = tile[rr];
                        y = e == 0 ? acc[ff][rr][0] : e == 1 ? acc[ff][rr][1] : e == 2 ? acc[ff][rr][2] : acc[ff][rr][3];
                    }
            const int i = i0 + 16 * f, c = 16 * t + 4 * q + e;
            const int64_t s = s0 + (int64_t)i * hop + c;
            if (!(y * 0.0f == 0.0f) && i < it.nf && t < g.T16 && c < hop && s < s_end) a.out[s] = dx_redo(*this, it, i, c);
        }
    }
}

// k-groups of G rows: J segments of 2M columns
static Geometry dx_geometry(const Plan &p) { return make_geometry(2 * p.M * p.geo32.J, 2 * p.M, 32); }

// Six products on the bfloat16 matrix cores take 1 / 2.6 of the time of one on the FP32 ones, so
// the plane kernel is the faster one while its columns of 32 pad a G row by no more than that
// (5 Mel bins and up), where a shape fits (frames of very many hops do not).
bool dx_split_fits(const Plan &p) {
    const Geometry g = dx_geometry(p);
    return p.H <= 256 && 2 * g.Hp <= 5 * ((2 * p.M + 7) / 8 * 8) &&
           split_shape(g, 3, (p.H + 15) / 16, p.cu_count, 1 << 20, (int64_t)kSplitChunk << 20).parts > 0;
}

size_t dx_split_pack_bytes(const Plan &p) { return (size_t)((p.H + 15) / 16) * dx_geometry(p).n_groups * 3 * 1024; }

PackJob dx_split_job(const Plan &p, void *out) {
    return {PACK_DX_PLANES, out, nullptr, nullptr, dx_geometry(p).Hp / 32, (p.H + 15) / 16, 3};
}

melt_status launch_dx_split(const Plan &p, const float *G, const RowChunk *rows, const int *n_rows, int64_t est_chunks,
                            int64_t n_frames, float *dx, hipStream_t s) {
    const Geometry g = dx_geometry(p);
    SplitDx job{};
    job.a.wave = G;
    job.a.chunks = (const Chunk *)rows;
    job.a.n_chunks = n_rows;
    job.a.out = dx;
    job.a.n_frames = n_frames;
    job.a.J = g.J;
    job.a.H = 2 * p.M;
    job.a.Hp = g.Hp;
    job.a.S = 3 * g.Hp + 8;
    job.g = {g.n_groups, g.Hp / 32, (p.H + 15) / 16, 0, 0, p.d_basis32, p.N, 0};
    job.hop = p.H;
    const SplitShape h = split_shape(g, 3, job.g.T16, p.cu_count, est_chunks, n_frames);
    return launch_split<Split3BF16>(p, job, g, h, p.d_pack_dx, est_chunks, s);
}

// ------------------------------------------------------------------ dW

// dW = G^T X.  A workgroup of 8 waves owns a 128 (q) x 256 (n) block over the frames of its
// split; a wave a 64 x 64 quarter-by-half of it (4 x 4 tiles of 16 x 16).  A step is 32 frames:
// each thread loads 8 consecutive frames of one q and of two n (coalesced over q and n), splits
// them and writes each plane's 8 values as one 16-byte piece of an MFMA fragment, so the
// transposition costs nothing and neither write nor read conflicts.  Two LDS buffers, one
// barrier per step: step s + 1 is in flight to registers while step s multiplies.
// What bounds it: the matrix cores (96 MFMAs of 16 cycles per wave and step, two waves per SIMD),
// with the split's VALU work (144 instructions per wave and step) issued between them.
constexpr int kDwQ = 128, kDwN = 256, kDwT = 32;
constexpr int kDwBuf = (kDwQ + kDwN) / 16 * 3 * 1024;      // bytes of one step's fragments
__global__ __attribute__((amdgpu_flat_work_group_size(512, 512), amdgpu_waves_per_eu(2, 2)))
void k_bwd_dw_split(const float *__restrict__ G, const int64_t *__restrict__ fstart, const float *__restrict__ wave,
                    int64_t T, int M, int N, int splits, float *part) {
    extern __shared__ __attribute__((aligned(16))) unsigned char lds[];
    const int tid = threadIdx.x, lane = tid & 63;
    const int wid = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int Q = 2 * M, NB = (N + kDwN - 1) / kDwN, blocks = (Q + kDwQ - 1) / kDwQ * NB;
    const int split = blockIdx.x / blocks, bb = blockIdx.x - split * blocks;
    const int q0 = bb / NB * kDwQ, n0 = bb % NB * kDwN;
    const int64_t per = ((T + splits - 1) / splits + kDwT - 1) / kDwT * kDwT;
    const int64_t t0 = (int64_t)split * per, t1 = t0 + per < T ? t0 + per : T;
    // staging: unit 0 is column sq of G, frames 8 tg .. 8 tg + 7 (tg = wid / 2); units 1 and 2 are
    // columns sn and sn + 128 of X, the same frames
    const int tg = wid >> 1, sc = tid & 127;
    const int qc = q0 + sc < Q ? q0 + sc : 0, na = n0 + sc < N ? n0 + sc : 0, nb = n0 + 128 + sc < N ? n0 + 128 + sc : 0;
    const bool vq = q0 + sc < Q, va = n0 + sc < N, vb = n0 + 128 + sc < N;
    float rg[8], ra[8], rb[8];
    unsigned ok = 0;                                   // frames of the step that exist (wave-uniform)
    // Unconditional loads, all in flight together; what does not exist is cleared when it is
    // staged.  A row without a frame has no samples: it reads N floats of the partial sums instead.
    auto load = [&](int64_t tb) {
        int64_t st[8];
#pragma unroll
        for (int e = 0; e < 8; ++e) {
            const int64_t t = tb + 8 * tg + e;
            st[e] = split_scalar(fstart, t < t1 ? t : t1 - 1);      // -1: a row without a frame
        }
        ok = 0;
#pragma unroll
        for (int e = 0; e < 8; ++e) {
            const int64_t t = tb + 8 * tg + e;
            ok |= (t < t1 && st[e] >= 0 ? 1u : 0u) << e;
            const float *x = st[e] >= 0 ? wave + st[e] : part;
            rg[e] = G[(t < t1 ? t : t1 - 1) * Q + qc];
            ra[e] = x[na];
            rb[e] = x[nb];
        }
        __builtin_amdgcn_sched_barrier(0);
    };
    auto put = [&](const float (&r)[8], bool exists, int tile, unsigned char *buf) {
        float v[8];
#pragma unroll
        for (int e = 0; e < 8; ++e) v[e] = exists && (ok >> e & 1) ? r[e] : 0.0f;
        unsigned w0[6], w1[6];
        Split3BF16::split(f32x4{v[0], v[1], v[2], v[3]}, w0);
        Split3BF16::split(f32x4{v[4], v[5], v[6], v[7]}, w1);
        unsigned char *d = buf + tile * 3072 + (16 * tg + (sc & 15)) * 16;
#pragma unroll
        for (int p = 0; p < 3; ++p) *(split_u32x4 *)(d + p * 1024) = split_u32x4{w0[2 * p], w0[2 * p + 1], w1[2 * p], w1[2 * p + 1]};
    };
    auto stage = [&](unsigned char *buf) {
        put(rg, vq, sc >> 4, buf);
        put(ra, va, 8 + (sc >> 4), buf);
        put(rb, vb, 16 + (sc >> 4), buf);
    };
    const int wq = wid & 1, wn = wid >> 1;             // the wave's 64-wide quarters
    f32x4 acc[4][4];
#pragma unroll
    for (int i = 0; i < 4; ++i)
#pragma unroll
        for (int j = 0; j < 4; ++j) acc[i][j] = f32x4{};
    if (t0 < t1) {
        load(t0);
        stage(lds);
    }
    int cur = 0;
    for (int64_t tb = t0; tb < t1; tb += kDwT, cur ^= 1) {
        __syncthreads();                               // this step's fragments are written, the other buffer is free
        const bool more = tb + kDwT < t1;
        if (more) load(tb + kDwT);
        const unsigned char *fr = lds + cur * kDwBuf + lane * 16;
        split_u32x4 A[4][3], B[3];
#pragma unroll
        for (int i = 0; i < 4; ++i)
#pragma unroll
            for (int p = 0; p < 3; ++p) A[i][p] = *(const split_u32x4 *)(fr + (4 * wq + i) * 3072 + p * 1024);
#pragma unroll
        for (int j = 0; j < 4; ++j) {
#pragma unroll
            for (int p = 0; p < 3; ++p) B[p] = *(const split_u32x4 *)(fr + (8 + 4 * wn + j) * 3072 + p * 1024);
            // a step's six products are summed on their own and added once: a sixth of the roundings at
            // the magnitude of a sum over all the frames
            f32x4 sum[4];
#pragma unroll
            for (int k = 0; k < 6; ++k)
#pragma unroll
                for (int i = 0; i < 4; ++i)
                    sum[i] = Split3BF16::mma(A[i][Split3BF16::pa[k]], B[Split3BF16::pb[k]], k ? sum[i] : f32x4{});
#pragma unroll
            for (int i = 0; i < 4; ++i) acc[i][j] += sum[i];
        }
        if (more) stage(lds + (cur ^ 1) * kDwBuf);
    }
    // lane holds column n, rows q = tile base + 4 (lane / 16) + r (interleaved q)
    float *o = part + (size_t)split * Q * N;
#pragma unroll
    for (int j = 0; j < 4; ++j) {
        const int n = n0 + 64 * wn + 16 * j + (lane & 15);
        if (n >= N) continue;
#pragma unroll
        for (int i = 0; i < 4; ++i)
#pragma unroll
            for (int r = 0; r < 4; ++r) {
                const int q = q0 + 64 * wq + 16 * i + 4 * (lane >> 4) + r;
                if (q < Q) o[(size_t)q * N + n] = acc[i][j][r];
            }
    }
}

int dw_split_blocks(const Plan &p) { return (2 * p.M + kDwQ - 1) / kDwQ * ((p.N + kDwN - 1) / kDwN); }

melt_status launch_dw_split(const Plan &p, const float *G, const int64_t *fstart, const float *wave, int64_t n_frames,
                            int splits, float *part, hipStream_t s) {
    allow_lds(k_bwd_dw_split);
    k_bwd_dw_split<<<dw_split_blocks(p) * splits, 512, 2 * kDwBuf, s>>>(G, fstart, wave, n_frames, p.M, p.N, splits, part);
    return hip_check(hipGetLastError(), "bwd dW");
}

}  // namespace melt
