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
// kernels before): dx 202 -> 76-80 us, dW 224 -> 80-88 us, a training step with its forward 617 ->
// 258-274 us, card to card.  Relative error against 64 bits: dx 7.9e-7 -> 6.5e-7, dW 7.8e-7 -> 5.2e-7.
// Scaling the operands (exact for small gradients) takes 2.4 of dW's microseconds.
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
    __device__ __forceinline__ bool store(const SplitItem &it, int fbase, int lane, const int (&tile)[RT], f32x4 (&acc)[FT][RT]) const;
    template <int FS, int RT>
    __device__ __forceinline__ void again(const SplitItem &it, int f0, int lane, const int (&tile)[RT]) const;
    // split_plain: segment s holds G of the frame that began j = J - 1 - s hops before the row.  The one
    // of the most hops comes first: its sums are dropped for the samples that its frame has not (a
    // weight of zero is not the absence of a term, if G is not finite).
    __device__ __forceinline__ int plain_segments() const { return a.J; }
    __device__ __forceinline__ int plain_columns() const { return a.H; }
    __device__ __forceinline__ f32x4 plain_samples(const SplitItem &it, int row, int s, int c) const {
        const int64_t at = it.start + (int64_t)(row + s) * a.H;
        f32x4 v{};
        if (at < it.start + it.lo || at >= it.end) return v;
#pragma unroll
        for (int e = 0; e < 4; ++e)
            if (c + e < a.H) v[e] = a.wave[at + c + e];
        return v;
    }
    __device__ __forceinline__ f32x4 plain_weights(int t, int row, int s, int c) const {
        const int n = (a.J - 1 - s) * hop + 16 * t + row;
        f32x4 v{};
        if (16 * t + row >= hop || n >= g.N) return v;
#pragma unroll
        for (int e = 0; e < 4; ++e)
            if (c + e < a.H) v[e] = g.basis[(size_t)(((c + e) & 1) * (a.H / 2) + ((c + e) >> 1)) * g.N + n];
        return v;
    }
    __device__ __forceinline__ void plain_first_segment(int t, int q, f32x4 &acc) const {
#pragma unroll
        for (int e = 0; e < 4; ++e)
            if ((a.J - 1) * hop + 16 * t + 4 * q + e >= g.N) acc[e] = 0.0f;
    }
};

template <class Op, int FT, int RT>
__device__ __forceinline__ bool SplitDx::store(const SplitItem &it, int fbase, int lane, const int (&tile)[RT],
                                               f32x4 (&acc)[FT][RT]) const {
    asm volatile("" : "+v"(lane));
    const int q = lane >> 4, i0 = fbase + (lane & 15);
    const int64_t ci = it.out_row / kSplitChunk, f0 = it.out_row - ci * kSplitChunk;
    const int64_t s0 = split_scalar(a.chunks, 5 * ci) + f0 * hop, s_end = split_scalar(a.chunks, 5 * ci + 1);
    const float unscale = split_unscale(kPlaneUnscale);
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
            const f32x4 y = acc[f][r] *= unscale;
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
    return __any(!(probe == 0.0f));
}

template <int FS, int RT>
__device__ __forceinline__ void SplitDx::again(const SplitItem &it, int f0, int lane, const int (&tile)[RT]) const {
    const int64_t ci = it.out_row / kSplitChunk;
    const int64_t s0 = split_scalar(a.chunks, 5 * ci) + (it.out_row - ci * kSplitChunk) * hop, s_end = split_scalar(a.chunks, 5 * ci + 1);
    unsigned bad[FS], any = 0;                          // of a row tile's four samples
    // calls each(address, element, bit) for the samples of tile r of frame tile f
    auto samples = [&](int f, auto &&each) {
        int l = lane;
        asm volatile("" : "+v"(l));                     // addresses and conditions formed here, not kept
        const int i = f0 + 16 * f + (l & 15);
        const int64_t s = s0 + (int64_t)i * hop;
        if (i >= it.nf) return;
#pragma unroll
        for (int r = 0; r < RT; ++r)
#pragma unroll
            for (int e = 0; e < 4; ++e) {
                const int c = 16 * tile[r] + 4 * (l >> 4) + e;
                if (c < hop && s + c < s_end) each(a.out + s + c, r, e);
            }
    };
#pragma unroll
    for (int f = 0; f < FS; ++f) {
        bad[f] = 0;
        samples(f, [&](const float *o, int r, int e) { bad[f] |= (*o * 0.0f == 0.0f ? 0u : 1u) << (4 * r + e); });
        any |= bad[f];
    }
    if (!__any(any != 0)) return;
    f32x4 acc[FS][RT];
    split_plain(*this, it, f0, lane, tile, acc);
#pragma unroll
    for (int f = 0; f < FS; ++f)
        samples(f, [&](float *o, int r, int e) {
            if (bad[f] >> (4 * r + e) & 1) *o = acc[f][r][e];
        });
}

// k-groups of G rows: J segments of 2M columns
static Geometry dx_geometry(const Plan &p) { return make_geometry(2 * p.M * p.geo32.J, 2 * p.M, 32); }

// Six products on the bfloat16 matrix cores take 1 / 2.6 of the time of one on the FP32 ones, so
// the plane kernel is the faster one while its columns of 32 pad a G row by no more than that
// (5 Mel bins and up), where a shape fits (frames of very many hops do not).  d/dwave calls at that
// line, 5 Mel bins, us, planes against FP32 MFMA: 64 x 30 s N 400 68 : 84, N 1024 66 : 85, N 128 218 : 223;
// 32 x 10 s 24 : 24, 28 : 30, 48 : 48, N 480, hop 161 29 : 25; one 1 s clip N 400 13.9 : 17.4.  16 x 4 s at
// N 128, hop 32, one item a workgroup, is the other way round up to 16 Mel bins (24.4 : 17.2 at 5,
// 24.7 : 22.5 at 16).
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
// split, 32 frames a step.  Four waves, one per SIMD, multiply: 64 q x 128 n each (4 x 8 tiles
// of 16 x 16).  Four stage, each eight consecutive frames of the step: a lane loads two columns
// of G and four of X of every frame (8- and 16-byte loads), splits them and writes each plane's
// 8 values of a column as one 16-byte piece of an MFMA fragment, so the transposition costs
// nothing; 16 bytes between tiles keep the writes off one another's banks.  Two LDS buffers, one
// barrier per step; two steps of samples are in registers, landed and in flight.
// What bounds it: the matrix cores (192 MFMAs of 16 cycles per multiply wave and step).  With
// every wave staging its share behind its multiplies (24 4-byte loads each, the VALU work of
// the split after the last MFMA) a step took 7300 cycles for those 3072; the whole backward of
// 27 456 frames, N = 1024, M = 128, was 182 us where it became 164 (168 with scaled operands).
// A wave's 64 q x 128 n of dW over frames [t0, t1) in plain FP32, on the FP32 matrix cores (4 frames
// and 1024 cycles a step, the next one's loads in flight): where a sum on planes is not finite.
// A NaN or infinity costs the waves that meet it about twice the time that their planes took, however
// many there are: 27 456 frames, N = 1024, M = 128, 0.11 ms a d/dbasis, 0.27 with one NaN gradient,
// 0.28 with nothing else (36 ms where each sum was one thread's, over all frames).
__device__ __forceinline__ void dw_plain(const float *__restrict__ G, const int64_t *__restrict__ fstart,
                                         const float *__restrict__ wave, const float *some, int64_t t0, int64_t t1, int Q,
                                         int N, int qw, int nw, f32x4 (&acc)[4][8]) {
    const int lane = threadIdx.x & 63, k = lane >> 4;
    auto start = [&](int64_t t) { return t + k < t1 ? fstart[t + k] : -1; };
    auto load = [&](int64_t t, int64_t st, float (&a)[4], float (&b)[8]) {
        const bool ok = st >= 0;                       // else from where there are N floats (`some`) and a row of G
        const float *g = G + (ok ? t + k : t0) * Q, *x = ok ? wave + st : some;
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            const float v = g[min(qw + 16 * i + (lane & 15), Q - 1)];
            a[i] = ok ? v : 0.0f;
        }
#pragma unroll
        for (int j = 0; j < 8; ++j) {
            const float v = x[min(nw + 16 * j + (lane & 15), N - 1)];
            b[j] = ok ? v : 0.0f;
        }
    };
#pragma unroll
    for (int i = 0; i < 4; ++i)
#pragma unroll
        for (int j = 0; j < 8; ++j) acc[i][j] = f32x4{};
    float a[4], b[8], an[4], bn[8];
    load(t0, start(t0), a, b);
    int64_t st = start(t0 + 4);
#pragma unroll 1
    for (int64_t t = t0; t < t1; t += 4) {
        load(t + 4, st, an, bn);
        st = start(t + 8);
#pragma unroll
        for (int i = 0; i < 4; ++i)
#pragma unroll
            for (int j = 0; j < 8; ++j) acc[i][j] = __builtin_amdgcn_mfma_f32_16x16x4f32(a[i], b[j], acc[i][j], 0, 0, 0);
#pragma unroll
        for (int i = 0; i < 4; ++i) a[i] = an[i];
#pragma unroll
        for (int j = 0; j < 8; ++j) b[j] = bn[j];
    }
}

typedef float dw_f32x4 __attribute__((ext_vector_type(4), aligned(4)));
constexpr int kDwQ = 128, kDwN = 256, kDwT = 32;
constexpr int kDwTile = 3 * 1024 + 16;                     // bytes from one tile's planes to the next's
constexpr int kDwBuf = (kDwQ + kDwN) / 16 * kDwTile;       // bytes of one step's fragments
// How a lane loads its four columns of X: DW_QUADS where N is a multiple of 4, so that they exist
// together or not at all; DW_TAIL otherwise, the last lane with a column loading the frame's last
// four and moving its own to the front; DW_SINGLE, one by one, in frames of fewer than four samples.
enum DwLoad { DW_QUADS, DW_TAIL, DW_SINGLE };
template <DwLoad LX>
__global__ __attribute__((amdgpu_flat_work_group_size(512, 512), amdgpu_waves_per_eu(2, 2)))
void k_bwd_dw_split(const float *__restrict__ G, const int64_t *__restrict__ fstart, const float *__restrict__ wave,
                    int64_t T, int M, int N, int splits, float *part) {
    extern __shared__ __attribute__((aligned(16))) unsigned char lds[];
    const int lane = threadIdx.x & 63;
    const int wid = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int Q = 2 * M, NB = (N + kDwN - 1) / kDwN, blocks = (Q + kDwQ - 1) / kDwQ * NB;
    // Workgroups go round the eight XCDs: where the splits are a multiple of 8, the blocks of one
    // are put eight apart, so that its samples and gradients are read into one L2.
    const bool even = splits % 8 == 0;
    const int split = even ? blockIdx.x / (8 * blocks) * 8 + blockIdx.x % 8 : blockIdx.x / blocks;
    const int bb = even ? blockIdx.x / 8 % blocks : blockIdx.x - split * blocks;
    const int q0 = bb / NB * kDwQ, n0 = bb % NB * kDwN;
    const int64_t per = ((T + splits - 1) / splits + kDwT - 1) / kDwT * kDwT;
    const int64_t t0 = (int64_t)split * per, t1 = t0 + per < T ? t0 + per : T;
    if (wid >= 4) {
        if (t0 >= t1) return;
        const int tg = wid - 4;
        const int q = q0 + 2 * lane, n = n0 + 4 * lane;
        // byte offsets of the lane's columns; where there is none, of column 0
        const bool tail = LX == DW_TAIL && n < N && n + 4 > N;
        const unsigned qo = q < Q ? 4 * q : 0, no = tail ? 4 * (N - 4) : n < N ? 4 * n : 0;
        struct Raw {
            float2 g[8];
            f32x4 x[8];
            unsigned ok;                               // frames of the step that exist (wave-uniform)
        };
        int64_t st[8], s0[8], s1[8];                   // first samples of a load's frames, read ahead; -1: a row without one
        auto starts = [&](int64_t tb, int64_t (&st)[8]) {
            const int64_t t = tb + 8 * tg;
            if (t + 8 <= t1) {
                typedef long long cs64x8 __attribute__((ext_vector_type(8), aligned(8)));
                typedef const __attribute__((address_space(4))) cs64x8 *cptr;
                const cs64x8 v = *(cptr)(fstart + t);
#pragma unroll
                for (int e = 0; e < 8; ++e) st[e] = v[e];
            } else {
#pragma unroll
                for (int e = 0; e < 8; ++e) st[e] = split_scalar(fstart, t + e < t1 ? t + e : t1 - 1);
            }
        };
        // Unconditional loads, all in flight together; frames past the split read its last one, and
        // what does not exist is cleared when it is staged.  A row without a frame has no samples:
        // it reads N floats of the partial sums instead.
        auto load = [&](int64_t tb, Raw &r, const int64_t (&st)[8]) {
            const int64_t t = tb + 8 * tg;
            const char *g[8], *x[8];
            int64_t any = 0;
#pragma unroll
            for (int e = 0; e < 8; ++e) any |= st[e];
            if (t + 8 <= t1 && any >= 0) {
                r.ok = 255;
#pragma unroll
                for (int e = 0; e < 8; ++e) {
                    g[e] = (const char *)(G + (t + e) * Q);
                    x[e] = (const char *)(wave + st[e]);
                }
            } else {
                r.ok = 0;
#pragma unroll
                for (int e = 0; e < 8; ++e) {
                    r.ok |= (t + e < t1 && st[e] >= 0 ? 1u : 0u) << e;
                    g[e] = (const char *)(G + (t + e < t1 ? t + e : t1 - 1) * Q);
                    x[e] = (const char *)(st[e] >= 0 ? wave + st[e] : part);
                }
            }
#pragma unroll
            for (int e = 0; e < 8; ++e) {
                r.g[e] = *(const float2 *)(g[e] + qo);
                if constexpr (LX == DW_SINGLE) {
#pragma unroll
                    for (int c = 0; c < 4; ++c) r.x[e][c] = *(const float *)(x[e] + (n + c < N ? 4 * (n + c) : 0));
                } else {
                    r.x[e] = *(const dw_f32x4 *)(x[e] + no);
                }
            }
            __builtin_amdgcn_sched_barrier(0);
        };
        auto put = [&](const float (&v)[8], unsigned char *d) {
            unsigned w0[6], w1[6];
            Split3BF16::split(f32x4{v[0], v[1], v[2], v[3]}, w0);
            Split3BF16::split(f32x4{v[4], v[5], v[6], v[7]}, w1);
#pragma unroll
            for (int p = 0; p < 3; ++p) *(split_u32x4 *)(d + p * 1024) = split_u32x4{w0[2 * p], w0[2 * p + 1], w1[2 * p], w1[2 * p + 1]};
        };
        // (columns past Q or N hold column 0's values: their sums are not stored)
        auto stage = [&](Raw &r, unsigned char *buf) {
            unsigned char *dg = buf + (lane >> 3) * kDwTile + (16 * tg + (2 * lane & 15)) * 16;
            unsigned char *dx = buf + (8 + (lane >> 2)) * kDwTile + (16 * tg + (4 * lane & 15)) * 16;
            if (r.ok != 255) {
#pragma unroll
                for (int e = 0; e < 8; ++e)
                    if (!(r.ok >> e & 1)) {
                        r.g[e] = float2{0.0f, 0.0f};
                        r.x[e] = f32x4{};
                    }
            }
            if constexpr (LX == DW_TAIL) {
                const int have = N & 3;                // columns of the lane that has some, not all
#pragma unroll
                for (int e = 0; e < 8; ++e) {
                    const f32x4 y = r.x[e];
                    r.x[e][0] = tail ? have == 3 ? y[1] : have == 2 ? y[2] : y[3] : y[0];
                    r.x[e][1] = tail ? have == 3 ? y[2] : y[3] : y[1];
                    r.x[e][2] = tail ? y[3] : y[2];
                }
            }
#pragma unroll
            for (int c = 0; c < 2; ++c) {
                float v[8];
#pragma unroll
                for (int e = 0; e < 8; ++e) v[e] = c ? r.g[e].y : r.g[e].x;
                put(v, dg + 16 * c);
            }
#pragma unroll
            for (int c = 0; c < 4; ++c) {
                float v[8];
#pragma unroll
                for (int e = 0; e < 8; ++e) v[e] = r.x[e][c];
                put(v, dx + 16 * c);
            }
        };
        // One step: `r` holds step s and then takes step s + 2, while s + 1 flies in the other set.
        // Steps past the split are loaded (its last frame) and staged (as zeros) too, in pairs
        // without a branch: every wait is then for a known number of younger loads, and no
        // register set is copied.
        auto step = [&](int64_t tb, Raw &r, unsigned char *buf) {
            stage(r, buf);
            load(tb + 2 * kDwT, r, st);
            starts(tb + 3 * kDwT, st);
            __syncthreads();                           // step s is staged, step s - 1 multiplied
        };
        Raw r0, r1;
        starts(t0, s0);
        starts(t0 + kDwT, s1);
        starts(t0 + 2 * kDwT, st);
        load(t0, r0, s0);
        load(t0 + kDwT, r1, s1);
        for (int64_t tb = t0; tb < t1; tb += 2 * kDwT) {
            step(tb, r0, lds);
            step(tb + kDwT, r1, lds + kDwBuf);
        }
        return;
    }
    const int wq = wid & 1, wn = wid >> 1;             // the wave's quarter of the block
    f32x4 acc[4][8];
#pragma unroll
    for (int i = 0; i < 4; ++i)
#pragma unroll
        for (int j = 0; j < 8; ++j) acc[i][j] = f32x4{};
    int cur = 0;
    for (int64_t tb = t0; tb < t1; tb += kDwT, cur ^= 1) {
        __syncthreads();                               // this step is staged
        const unsigned char *fr = lds + cur * kDwBuf + lane * 16;
        split_u32x4 A[4][3], B[2][3];
        // a step's six products are summed on their own and added once, behind the next tile's first
        // MFMAs: a sixth of the roundings at the magnitude of a sum over all the frames
        f32x4 sum[2][4];
        auto load_b = [&](int j) {
#pragma unroll
            for (int p = 0; p < 3; ++p) B[j & 1][p] = *(const split_u32x4 *)(fr + (8 + 8 * wn + j) * kDwTile + p * 1024);
        };
        load_b(0);
#pragma unroll
        for (int p = 0; p < 3; ++p)
#pragma unroll
            for (int i = 0; i < 4; ++i) A[i][p] = *(const split_u32x4 *)(fr + (4 * wq + i) * kDwTile + p * 1024);
#pragma unroll
        for (int j = 0; j < 8; ++j) {
            if (j < 7) load_b(j + 1);
#pragma unroll
            for (int k = 0; k < 6; ++k) {
#pragma unroll
                for (int i = 0; i < 4; ++i)
                    sum[j & 1][i] = Split3BF16::mma(A[i][Split3BF16::pa[k]], B[j & 1][Split3BF16::pb[k]], k ? sum[j & 1][i] : f32x4{});
                if (k == 0 && j > 0) {
#pragma unroll
                    for (int i = 0; i < 4; ++i) acc[i][j - 1] += sum[(j - 1) & 1][i];
                }
            }
        }
#pragma unroll
        for (int i = 0; i < 4; ++i) acc[i][7] += sum[1][i];
    }
    // lane holds column n, rows q = tile base + 4 (lane / 16) + r (interleaved q)
    const int qw = q0 + 64 * wq, nw = n0 + 128 * wn;
    const float unscale = split_unscale(kPlaneUnscale);
    float *o = part + (size_t)split * Q * N, probe = 0.0f;      // probe stays 0 while every sum is finite
    auto each = [&](auto &&put) {
#pragma unroll
        for (int j = 0; j < 8; ++j) {
            const int n = nw + 16 * j + (lane & 15);
            if (n >= N) continue;
#pragma unroll
            for (int i = 0; i < 4; ++i)
#pragma unroll
                for (int r = 0; r < 4; ++r) {
                    const int q = qw + 16 * i + 4 * (lane >> 4) + r;
                    if (q < Q) put(o + (size_t)q * N + n, acc[i][j][r]);
                }
        }
    };
    each([&](float *at, float v) {
        v *= unscale;
        probe = fmaf(v, 0.0f, probe);
        *at = v;
    });
    if (cur) __syncthreads();                          // the staging waves take steps in pairs
    if (__any(!(probe == 0.0f))) {
        // the planes of an infinity are not a product with it
        dw_plain(G, fstart, wave, part, t0, t1, Q, N, qw, nw, acc);
        each([&](float *at, float v) {
            if (!(*at * 0.0f == 0.0f)) *at = v;
        });
    }
}

int dw_split_blocks(const Plan &p) { return (2 * p.M + kDwQ - 1) / kDwQ * ((p.N + kDwN - 1) / kDwN); }

melt_status launch_dw_split(const Plan &p, const float *G, const int64_t *fstart, const float *wave, int64_t n_frames,
                            int splits, float *part, hipStream_t s) {
    const auto kernel = p.N % 4 == 0 ? k_bwd_dw_split<DW_QUADS> : p.N > 4 ? k_bwd_dw_split<DW_TAIL> : k_bwd_dw_split<DW_SINGLE>;
    allow_lds(kernel);
    kernel<<<dw_split_blocks(p) * splits, 512, 2 * kDwBuf, s>>>(G, fstart, wave, n_frames, p.M, p.N, splits, part);
    return hip_check(hipGetLastError(), "bwd dW");
}

}  // namespace melt
