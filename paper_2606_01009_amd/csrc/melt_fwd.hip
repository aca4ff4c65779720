// MelT forward: chunk schedule of a ragged batch, basis packing for every operand format,
// the table of kernel variants and the dispatch to them.
#include <cstdio>
#include <mutex>
#include "fwd_common.h"
#include "melt_split.h"
#include "pack.h"

namespace melt {

// ------------------------------------------------------------------ schedule

// Chunk table for at most 64 clips, with no barrier: every wave scans the clips in its lanes and
// writes every (16 blocks)-th group of 64 entries (`blocks`, the grid: read from the dispatch packet it
// costs 0.2 us).  n_chunks receives min(total, cap).
__global__ __launch_bounds__(1024) void k_schedule64(const int64_t *__restrict__ off, int n_clips, int N, int H,
                                                     int bf, Chunk *__restrict__ tab, int64_t cap,
                                                     int *__restrict__ n_out, int blocks) {
    const int lane = threadIdx.x & 63, w = blockIdx.x * 16 + __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const ClipScan s = clip_scan(off, n_clips, N, H, bf);
    // the same on every lane; made scalar so the loop below keeps every lane active
    const int64_t n = uniform64(s.total < cap ? s.total : cap);
    for (int64_t q0 = 64 * w; q0 < n; q0 += 1024 * blocks) {      // wave-uniform trip count
        const Chunk e = clip_chunk(s, H, bf, q0 + lane);
        if (q0 + lane < n) tab[q0 + lane] = e;
    }
    if (blockIdx.x == 0 && threadIdx.x == 0) *n_out = (int)n;
}

// Any number of clips: every workgroup forms the prefix sums of frame and chunk counts over the
// clips, 1024 at a time, and writes its share of the chunk table.  n_chunks receives min(total, cap).
__global__ __launch_bounds__(1024) void k_schedule(const int64_t *__restrict__ off, int n_clips, int N,
                                                   int H, int bf, Chunk *__restrict__ tab, int64_t cap,
                                                   int *__restrict__ n_out, int blocks) {
    __shared__ int64_t sf[1024], sc[1024], s_start[1024], s_len[1024];
    __shared__ int64_t wf[16], wc[16];
    __shared__ int64_t carry_f, carry_c;
    const int tid = threadIdx.x, lane = tid & 63, w = tid >> 6;
    if (tid == 0) carry_f = carry_c = 0;
    for (int base = 0; base < n_clips; base += 1024) {
        const int c = base + tid;
        int64_t st = 0, L = 0;
        if (c < n_clips) {
            st = off[c];
            L = off[c + 1] - st;
        }
        const int64_t T = (L >= N) ? 1 + udiv_nonneg(L - N, H) : 0;
        const int64_t K = udiv_nonneg(T + bf - 1, bf);
        // inclusive prefix sums of T and K over the block: within each wave, then across the
        // 16 wave totals
        const int64_t pf = wave_scan(T, lane), pc = wave_scan(K, lane);
        if (lane == 63) {
            wf[w] = pf;
            wc[w] = pc;
        }
        __syncthreads();
        int64_t of = 0, oc = 0;
        for (int k = 0; k < w; ++k) {
            of += wf[k];
            oc += wc[k];
        }
        sf[tid] = pf + of;
        sc[tid] = pc + oc;
        s_start[tid] = st;
        s_len[tid] = L;
        __syncthreads();
        // entries of this block of clips, written by all threads: entry q belongs to the
        // first clip t whose inclusive chunk prefix exceeds q (binary search)
        const int64_t total = sc[1023];
        for (int64_t q = tid + 1024 * (int64_t)blockIdx.x; q < total; q += 1024 * blocks) {
            int lo = 0, hi = 1023;
            while (lo < hi) {
                const int mid = (lo + hi) >> 1;
                if (sc[mid] > q) hi = mid;
                else lo = mid + 1;
            }
            const int t = lo;
            const int64_t kc0 = t > 0 ? sc[t - 1] : 0;         // clip t's first entry in the block
            const int64_t k = q - kc0;                          // chunk index within the clip
            const int64_t Tt = sf[t] - (t > 0 ? sf[t - 1] : 0);
            const int64_t fb = carry_f + (t > 0 ? sf[t - 1] : 0);
            const int64_t idx = carry_c + q;
            if (idx >= cap) break;
            Chunk e;
            e.sample_start = s_start[t] + k * bf * (int64_t)H;
            e.sample_end = s_start[t] + s_len[t];
            e.out_row = fb + k * bf;
            e.n_frames = (int)((Tt - k * bf) < bf ? (Tt - k * bf) : bf);
            e.clip = base + t;
            tab[idx] = e;
        }
        __syncthreads();
        if (tid == 1023) {
            carry_f += sf[1023];
            carry_c += sc[1023];
        }
        __syncthreads();
    }
    if (blockIdx.x == 0 && tid == 0) *n_out = (int)(carry_c < cap ? carry_c : cap);
}

__global__ __launch_bounds__(1024) void k_frame_offsets(const int64_t *__restrict__ off, int n_clips, int N,
                                                        int H, int64_t *__restrict__ fo) {
    __shared__ int64_t sf[1024];
    __shared__ int64_t carry;
    const int tid = threadIdx.x;
    if (tid == 0) carry = 0;
    __syncthreads();
    for (int base = 0; base < n_clips; base += 1024) {
        const int c = base + tid;
        int64_t L = 0;
        if (c < n_clips) L = off[c + 1] - off[c];
        const int64_t T = (L >= N) ? 1 + (L - N) / H : 0;
        sf[tid] = T;
        __syncthreads();
        for (int d = 1; d < 1024; d <<= 1) {
            const int64_t v = tid >= d ? sf[tid - d] : 0;
            __syncthreads();
            sf[tid] += v;
            __syncthreads();
        }
        if (c < n_clips) fo[c] = carry + sf[tid] - T;
        __syncthreads();
        if (tid == 1023) carry += sf[1023];
        __syncthreads();
    }
    if (tid == 0) fo[n_clips] = carry;
}

// FP32: [rt][group][lane][4]
__device__ __forceinline__ void pack_f32(const PackJob &j, const float *b32, int M, int N, int H, int64_t i) {
    const int lane = (i >> 2) & 63;
    const int64_t tg = i >> 8;
    const int g = (int)(tg % j.NG), rt = (int)(tg / j.NG);
    ((float *)j.out)[i] = packed_value(b32, M, N, H, rt, j.seg[g], j.col[g], 4, lane, i & 3);
}

// 16-bit: [rt][group][lane][8]
__device__ __forceinline__ void pack_h16(const PackJob &j, const float *b32, int M, int N, int H, int64_t i) {
    const int lane = (i >> 3) & 63;
    const int64_t tg = i >> 9;
    const int g = (int)(tg % j.NG), rt = (int)(tg / j.NG);
    const float v = packed_value(b32, M, N, H, rt, j.seg[g], j.col[g], 8, lane, i & 7);
    ((unsigned short *)j.out)[i] = j.form == 0   ? f32_to_bf16_bits(v)
                                   : j.form == 1 ? f32_to_f16_bits(v)
                                   : j.form == 2 ? f32_to_bf16_bits(v - bf16_bits_to_f32(f32_to_bf16_bits(v)))
                                                 : f32_to_f16_bits(v - f16_bits_to_f32(f32_to_f16_bits(v)));
}

// P planes of a value, 512 elements apart (three: of the scaled value)
__device__ __forceinline__ void put_planes(unsigned short *out, float v, int form) {
    const int P = form & 7;
    if (P == 3) v *= kPlaneScale;
    for (int p = 0; p < P; ++p) {
        const unsigned short b = form & 8 ? f32_to_f16_bits(v) : f32_to_bf16_bits(v);
        out[p * 512] = b;
        v -= form & 8 ? f16_bits_to_f32(b) : bf16_bits_to_f32(b);
    }
}

// Planes of the split-plane kernel: [tile][group of 32][plane][lane][8], lane = row lane % 16 of
// the 16-row tile, columns 8 (lane / 16) ..; rows 4q .. 4q + 3 are (cos, sin) of two Mel bins.
__device__ __forceinline__ void pack_planes(const PackJob &j, const float *b32, int M, int N, int H, int64_t i) {
    const int e = i & 511, lane = e >> 3;
    const int64_t tg = i >> 9;
    const int g = (int)(tg % j.NG), t = (int)(tg / j.NG);
    const int row = lane & 15, sg = j.seg[g], c = j.col[g] + 8 * (lane >> 4) + (e & 7);
    const int mel = split_tile_mel(t, row >> 2, j.tiles) + ((row >> 1) & 1);
    float v = 0.0f;
    if (mel < M && c < min(H, N - sg * H)) v = b32[(size_t)((row & 1) * M + mel) * N + sg * H + c];
    put_planes((unsigned short *)j.out + (size_t)tg * (j.form & 7) * 512 + e, v, j.form);
}

// The backward's dx, FP32: fragments [ct][segment j][q-group of 8][lane][4], B[k = q][col = c] =
// W_q[jH + 32 ct + c] with q the interleaved row (2m cosine, 2m+1 sine) and lane half h holding
// q = 8 qg + 4 h + i for MFMA step i.  NG = segments.
__device__ __forceinline__ void pack_dx(const PackJob &j, const float *b32, int M, int N, int H, int64_t i) {
    const int QG = (2 * M + 7) / 8, lane = (i >> 2) & 63;
    int64_t r = i >> 8;
    const int qg = (int)(r % QG);
    r /= QG;
    const int sg = (int)(r % j.NG), ct = (int)(r / j.NG);
    const int q = qg * 8 + 4 * (lane >> 5) + (int)(i & 3), c = ct * 32 + (lane & 31), n = sg * H + c;
    ((float *)j.out)[i] = q < 2 * M && c < H && n < N ? b32[(size_t)((q & 1) * M + (q >> 1)) * N + n] : 0.0f;
}

// The backward's dx on planes: [tile][group][plane][lane][8], row 16 t + lane % 16 = sample c of a
// hop, columns segment s = group / GH (j = J - 1 - s) and interleaved q = 32 (group % GH) +
// 8 (lane / 16) + e.  NG = GH, the groups of one segment.
__device__ __forceinline__ void pack_dx_planes(const PackJob &j, const float *b32, int M, int N, int H, int64_t i) {
    const int J = (N + H - 1) / H, NG = J * j.NG, e = i & 511, lane = e >> 3;
    const int64_t tg = i >> 9;
    const int gr = (int)(tg % NG), t = (int)(tg / NG);
    const int s = gr / j.NG, sg = J - 1 - s, q = 32 * (gr - s * j.NG) + 8 * (lane >> 4) + (e & 7);
    const int c = 16 * t + (lane & 15), n = sg * H + c;
    float v = 0.0f;
    if (q < 2 * M && c < H && n < N) v = b32[(size_t)((q & 1) * M + (q >> 1)) * N + n];
    put_planes((unsigned short *)j.out + (size_t)tg * (j.form & 7) * 512 + e, v, j.form);
}

// elements of a job
__host__ __device__ __forceinline__ int64_t pack_total(const PackJob &j, int M, int N, int H) {
    return j.kind == PACK_COPY        ? (int64_t)2 * M * N
           : j.kind == PACK_F32       ? (int64_t)j.tiles * j.NG * 256
           : j.kind == PACK_DX        ? (int64_t)j.tiles * j.NG * ((2 * M + 7) / 8) * 256
           : j.kind == PACK_DX_PLANES ? (int64_t)j.tiles * j.NG * ((N + H - 1) / H) * 512
                                      : (int64_t)j.tiles * j.NG * 512;
}
__global__ __launch_bounds__(256) void k_pack(PackJobs jobs, const float *__restrict__ b32, int M, int N, int H) {
    const PackJob &j = jobs.job[blockIdx.x % jobs.n];
    const int64_t first = (blockIdx.x / jobs.n) * (int64_t)blockDim.x + threadIdx.x, step = (int64_t)(gridDim.x / jobs.n) * blockDim.x;
    const int64_t total = pack_total(j, M, N, H);
    for (int64_t i = first; i < total; i += step) {
        switch (j.kind) {
        case PACK_COPY: ((float *)j.out)[i] = b32[i]; break;
        case PACK_F32: pack_f32(j, b32, M, N, H, i); break;
        case PACK_H16: pack_h16(j, b32, M, N, H, i); break;
        case PACK_PLANES: pack_planes(j, b32, M, N, H, i); break;
        case PACK_DX: pack_dx(j, b32, M, N, H, i); break;
        case PACK_DX_PLANES: pack_dx_planes(j, b32, M, N, H, i); break;
        }
    }
}

// E4M3 pack of the basis: [rt][group of 64][lane][32 bytes].  blocks = 0: lane half h holds
// k = 64 g + 32 h + byte (any k order serves a product with unit block scales, as long as the
// frames use the same).  blocks = 1: the order in which the 32x32x64 MFMA's two 32-k scale
// blocks are whole: bytes 0-15 of half h are k = 64 g + 16 h + byte (block 0), bytes 16-31
// are k = 64 g + 32 + 16 h + byte - 16 (block 1).  Row scales r_j = 448 / max_n |W_j| (FP32);
// rinv[rt][i] = 1 / r_j of tile row i.  One workgroup of 256 threads per row tile: eight
// threads per tile row share its maximum, then every thread packs whole 4-byte words.
__global__ __launch_bounds__(256) void k_pack_f8(const float *__restrict__ b32, int M, int N, int NG, int blocks,
                                                 unsigned *__restrict__ out, float *__restrict__ rinv) {
    __shared__ float rmax[32];
    const int rt = blockIdx.x, t = threadIdx.x;
    {
        const int i = t >> 3, sub = t & 7;
        int ml, part;
        tile_row_to_mel(i, ml, part);
        const int mel = rt * 16 + ml;
        float mx = 0.0f;
        if (mel < M)
            for (int n = sub; n < N; n += 8) mx = fmaxf(mx, fabsf(b32[(size_t)(part * M + mel) * N + n]));
        // the eight threads of a row are consecutive lanes of one wave
        mx = fmaxf(mx, __shfl_xor(mx, 1, 64));
        mx = fmaxf(mx, __shfl_xor(mx, 2, 64));
        mx = fmaxf(mx, __shfl_xor(mx, 4, 64));
        if (sub == 0) {
            rmax[i] = mx;
            rinv[rt * 32 + i] = mx > 0.0f ? 1.0f / __fdiv_rn(448.0f, mx) : 1.0f;
        }
    }
    __syncthreads();
    for (int idx = t; idx < NG * 512; idx += 256) {
        const int w = idx & 7, lane = (idx >> 3) & 63, g = idx >> 9;
        int ml, part;
        tile_row_to_mel(lane & 31, ml, part);
        const int mel = rt * 16 + ml;
        const float mx = rmax[lane & 31];
        const float sc = mx > 0.0f ? __fdiv_rn(448.0f, mx) : 1.0f;
        float v[4];
        for (int e = 0; e < 4; ++e) {
            const int bb = 4 * w + e, h = lane >> 5;
            const int k = blocks ? g * 64 + 32 * (bb >> 4) + 16 * h + (bb & 15) : g * 64 + 32 * h + bb;
            v[e] = (mel < M && k < N) ? __fmul_rn(b32[(size_t)(part * M + mel) * N + k], sc) : 0.0f;
        }
        out[(((size_t)rt * NG + g) * 64 + lane) * 8 + w] = fp8x4(v[0], v[1], v[2], v[3]);
    }
}

// ------------------------------------------------------------------ host side

namespace {

melt_status upload_ints(const std::vector<int> &v, int **d) {
    if (hipMalloc(d, sizeof(int) * (v.size() + 1)) != hipSuccess) return set_error(MELT_E_NO_MEMORY, "hipMalloc");
    return hip_check(hipMemcpy(*d, v.data(), sizeof(int) * v.size(), hipMemcpyHostToDevice), "hipMemcpy");
}

}  // namespace

melt_status pack_tables_upload(Plan &p) {
    melt_status st = upload_ints(p.geo32.seg_of_group, &p.d_seg32);
    if (st == MELT_OK) st = upload_ints(p.geo32.col_of_group, &p.d_col32);
    if (st == MELT_OK) st = upload_ints(p.geo16.seg_of_group, &p.d_seg16);
    if (st == MELT_OK) st = upload_ints(p.geo16.col_of_group, &p.d_col16);
    if (st == MELT_OK) st = upload_ints(p.geoS.seg_of_group, &p.d_segS);
    if (st == MELT_OK) st = upload_ints(p.geoS.col_of_group, &p.d_colS);
    return st;
}

// Packs the basis `src` (device, stacked [2M][N]) into the layouts of the plan's precision and the
// backward's dx, and into d_basis32 unless that is where it is: enqueued on `s`, no allocation
// after plan creation and no host synchronisation (the k-group tables were uploaded then).
melt_status pack_basis(Plan &p, const float *src, hipStream_t s) {
    const int RT = p.row_tiles;
    PackJobs jobs;
    if (src != p.d_basis32) jobs.add({PACK_COPY, p.d_basis32, nullptr, nullptr, 0, 0, 0});
    if (split_used(p))
        jobs.add({PACK_PLANES, p.d_pack_split, p.d_segS, p.d_colS, p.geoS.n_groups, (p.M + 7) / 8,
                  split_planes(p) + (prec_f16(p) ? 8 : 0)});
    switch (p.cfg.precision) {
    case MELT_PREC_FP32: jobs.add({PACK_F32, p.d_pack_f32, p.d_seg32, p.d_col32, p.geo32.n_groups, RT, 0}); break;
    case MELT_PREC_FP8_E4M3:
    case MELT_PREC_FP8_E4M3_BLOCK32:
        k_pack_f8<<<RT, 256, 0, s>>>(src, p.M, p.N, (p.N + 63) / 64,
                                     p.cfg.precision == MELT_PREC_FP8_E4M3_BLOCK32 ? 1 : 0, (unsigned *)p.d_pack_f8,
                                     p.d_rowscale);
        break;
    default:
        jobs.add({PACK_H16, p.d_pack_h16, p.d_seg16, p.d_col16, p.geo16.n_groups, RT, prec_f16(p) ? 1 : 0});
        if (prec_split(p)) jobs.add({PACK_H16, p.d_pack_lo, p.d_seg16, p.d_col16, p.geo16.n_groups, RT, prec_f16(p) ? 3 : 2});
    }
    const melt_status st = pack_dx_job(p, jobs);
    if (st != MELT_OK) return st;
    // 256 workgroups a job (a CU each), up to 2048 where its elements are many: hops of a few samples pad
    // every layout (hop 1, N 1024, 512 Mel bins, FP32: 482 us with 256, 108 now)
    int64_t most = 0;
    for (int i = 0; i < jobs.n; ++i) most = std::max(most, pack_total(jobs.job[i], p.M, p.N, p.H));
    const int each = (int)std::min<int64_t>(2048, std::max<int64_t>(256, most / 4096));
    if (jobs.n > 0) k_pack<<<each * jobs.n, 256, 0, s>>>(jobs, src, p.M, p.N, p.H);
    return hip_check(hipGetLastError(), "pack basis");
}

melt_status ensure_chunks(Plan &p, int which, int64_t needed) {
    if (needed <= p.chunk_cap[which]) return MELT_OK;
    int64_t cap = std::max<int64_t>(needed, 2 * p.chunk_cap[which]);
    Chunk *d = nullptr;
    if (hipMalloc(&d, sizeof(Chunk) * cap) != hipSuccess) return set_error(MELT_E_NO_MEMORY, "chunk table");
    if (p.d_chunks[which]) {
        (void)hipDeviceSynchronize();
        (void)hipFree(p.d_chunks[which]);
    }
    p.d_chunks[which] = d;
    p.chunk_cap[which] = cap;
    return MELT_OK;
}

// One workgroup writes about 1024 entries in the time it takes to find them, so longer tables are
// shared by several (the comparator's table of 64 x 30 s, 8000 entries: 8.6 us with one).
static melt_status enqueue_schedule(const Plan &p, const int64_t *d_off, int n_clips, int bf, int64_t need, Chunk *tab,
                                    int64_t cap, int *n_tab, hipStream_t s) {
    const int grid = (int)std::min<int64_t>(16, (need + 1023) / 1024);
    if (n_clips <= 64) k_schedule64<<<grid, 1024, 0, s>>>(d_off, n_clips, p.N, p.H, bf, tab, cap, n_tab, grid);
    else k_schedule<<<grid, 1024, 0, s>>>(d_off, n_clips, p.N, p.H, bf, tab, cap, n_tab, grid);
    return hip_check(hipGetLastError(), "schedule launch");
}

static void set_prepared(Plan &p, int which, int n_clips, int64_t n_frames, int bf, int variant) {
    p.prepared_frames[which] = n_frames;
    p.prepared_bf[which] = bf;
    p.prepared_clips[which] = n_clips;
    if (which == 0) p.prepared_variant = variant;
}

melt_status launch_schedule(Plan &p, int which, const int64_t *d_off, int n_clips, int bf_max, int64_t n_frames,
                            hipStream_t s, int variant) {
    // Chunks of at most bf_max frames (the kernel's LDS image).  The comparator sizes its
    // chunks to the batch (whole sub-tasks, a few chunks per resident wave); measured, the
    // same for the MelT kernels costs more in per-chunk overhead than it gains, so their
    // chunks keep the full size.
    int bf = bf_max;
    if (which == 1 && n_frames > 0) bf = std::min(bf_max, stft_batch_chunk_frames(p, n_frames));
    const int64_t need = n_frames / bf + n_clips + 1;
    melt_status st = ensure_chunks(p, which, need);
    if (st != MELT_OK) return st;
    st = enqueue_schedule(p, d_off, n_clips, bf, need, p.d_chunks[which], p.chunk_cap[which], p.d_nchunks + which, s);
    if (st == MELT_OK) set_prepared(p, which, n_clips, n_frames, bf, variant < 0 ? p.tune_variant : variant);
    return st;
}

// The batch of a kernel that finds its own chunks and leaves them in table `which` (chunks of bf
// frames): the batch is the plan's prepared one afterwards, as when a table is built for the call.
// Where the table would have to grow inside a stream capture, which cannot be, none is left.
melt_status prepare_clips(Plan &p, int which, const int64_t *d_off, int n_clips, int64_t n_frames, int bf, int variant,
                          ClipTable &t, hipStream_t s) {
    const int64_t est = n_frames / bf + n_clips;
    if (est + 1 > p.chunk_cap[which]) {
        hipStreamCaptureStatus capture = hipStreamCaptureStatusNone;
        if (hipStreamIsCapturing(s, &capture) != hipSuccess || capture != hipStreamCaptureStatusNone) {
            t = {d_off, n_clips, p.N, bf, (int)est, nullptr, nullptr};
            p.prepared_frames[which] = -1;
            return MELT_OK;
        }
        const melt_status st = ensure_chunks(p, which, est + 1);
        if (st != MELT_OK) return st;
    }
    t = {d_off, n_clips, p.N, bf, (int)est, p.d_chunks[which], p.d_nchunks + which};
    set_prepared(p, which, n_clips, n_frames, bf, variant);
    return MELT_OK;
}

melt_status launch_frame_offsets(const int64_t *d_off, int n_clips, int N, int H, int64_t *d_fo, hipStream_t s) {
    k_frame_offsets<<<1, 1024, 0, s>>>(d_off, n_clips, N, H, d_fo);
    return hip_check(hipGetLastError(), "frame offsets launch");
}

// Kernel variants of a plan, in the order the autotuner times them (p.tune_variant selects;
// the first one is the default):
//   FP32       operand planes (melt_split.h; last for frames of few samples), frame-split on FP32 MFMA
//              with staging waves, the same with register prefetch
//   BF16/FP16  the 12-wave producer/consumer kernel (96- or 64-frame chunks) where its
//              register tiles and LDS fit; row pairs (two basis tiles per wave) where they fit;
//              row-split with direct-to-LDS staging (one span buffer: 128- then 64-frame
//              chunks; then two span buffers), producer/consumer row-split (one span, then
//              two; only with producer waves), row-split with register staging, K-split (frames
//              too long for one wave's tile), frame-split (the fallback; for the split
//              precisions only where no register-tile kernel applies)
//   BF16X3 / FP16X3  the 8-wave producer/consumer kernel (hi and lo tiles, 64-frame chunks)
//              where it fits, then as above without row pairs and K-split, with one-span
//              chunks of 96 then 64 frames
//   FP8        frame-split (hops that are multiples of 32, up to 8 row tiles), row-split with
//              direct-to-LDS staging (the largest chunk that fits LDS; 64-frame
//              chunks at two workgroups per CU), row-split with register staging, then the
//              producer/consumer kernel (first beyond 8 row tiles, which the others do not take)
//   FP8 with 32-sample block scales  producer/consumer block-scaled kernel, then the
//              one-buffer block-scaled kernel with 160- and 128-frame chunks
enum VariantKind { V_F32_WS, V_F32_FS, V_H16_PP, V_H16_AS, V_H16_AP, V_H16_RS, V_H16_KS, V_H16_FS, V_F8_AS, V_F8_RS,
                   V_F8B_AS, V_F8B_PC, V_H16_PC, V_F8_PC, V_SPLIT, V_F8_FS };
struct Variant {
    VariantKind kind;
    int bf;          // frames per chunk
    int nbuf = 1;    // FP32 span buffers of the direct-to-LDS 16-bit kernel
};

// Shape of the split-plane kernel for a batch: the one with the fewest cycles in the model
//   rounds over the CUs x max(k-groups x RT x max(MFMA, L1) + fixed, staging)
// where a k-group of a tile costs FT NP MFMAs of 16 cycles on its SIMD or, if that is more, P KB for
// each of the four multiply waves through the CU's 64-byte L1 port.  Clips are taken to be of one length
// where their number divides the frames, else to end half an item short.
// 128-frame items are the cheapest per frame; 64-frame ones (four row groups) serve rows too long for
// LDS at 128 and fill a last round better, and 32-frame ones spread a call of few frames over the chip.
// The other terms are fitted to whole calls of 28 front ends (N 48 to 1200, 8 to 512 Mel bins, FP32 and
// BF16X3) in 1 to 64 clips of 1 to 30 s, and of 11 in 16 to 300 clips of mixed lengths, every shape
// timed: fixed, an item's barriers, hand-over and first fragment reads, 300 a tile of accumulators, and
// 900 where the fragment ring has to be filled again (ring slots that are no divisor of the k-groups);
// staging, 20400 and a quarter a vector.  The choice is then within 0.4 % of the fastest shape on
// average (0.7 % for mixed lengths), 24 % at worst (BF16X3, N 800, 80 Mel bins, 16 x 4 s: 25.1 us in
// 64-frame items of three row parts, 20.3 of two); with one fixed term of 4500 and a chunk too many
// assumed for each clip it was 6 % and up to twice as long (FP32, N 400, 80 Mel bins, 32 x 10 s: 54.8 us
// with five row parts, 27.3 with one).  Fitted to clips of one length alone, 61 clips of 0.5 to 12 s
// (FP32, N 480, hop 161, 64 Mel bins) took 44.3 us in 128-frame items where 64-frame ones take 38.4.
SplitShape split_shape(const Geometry &g, int P, int T16, int cu_count, int64_t est_chunks, int64_t n_frames) {
    const int NP = P == 3 ? 6 : 3;
    static const struct {
        int wf, ft, rt_max, pv[2];
        double fixed;
    } families[3] = {{2, 4, 8, {18, 0}, 17900}, {1, 4, 4, {18, 18}, 14000}, {2, 1, 2, {10, 10}, 2900}};
    const int64_t clips = std::max<int64_t>(1, est_chunks - n_frames / kSplitChunk);
    SplitShape best{0, 0, 0, 0, 0};
    double best_cost = 1e300;
    for (int i = 0; i < 3; ++i) {
        const auto &f = families[i];
        SplitShape h{f.wf, f.ft, 0, 0, 0};
        const int sf = split_sf(h), wr = 4 / f.wf;
        const int vectors = (sf + g.J - 1) * (g.Hp / 4);
        const int wide = i == 0 ? (P == 3 ? 26 : 34) : f.pv[1];
        h.pv = vectors <= f.pv[0] * 256 ? f.pv[0] : wide;
        if (vectors > h.pv * 256 || split_lds(P, g, h) > (size_t)kMaxLds) continue;
        for (int parts = (T16 + wr * f.rt_max - 1) / (wr * f.rt_max); parts <= (T16 + wr - 1) / wr; ++parts) {
            h.parts = parts;
            h.rt = (T16 + wr * parts - 1) / (wr * parts);
            if (h.rt == 7) h.rt = 8;
            const int64_t whole = n_frames % clips == 0 ? clips * ((n_frames / clips + sf - 1) / sf)
                                                        : (n_frames + clips * sf / 2 + sf - 1) / sf;
            const int64_t items = std::max<int64_t>(whole, 1) * parts;
            const int64_t rounds = (items + cu_count - 1) / cu_count;
            const int ring = split_ring(f.ft, h.rt), U = ring > h.rt ? ring / h.rt : 1;
            const double multiply = std::max(f.ft * NP * 16, P * 64) * (double)g.n_groups * h.rt + f.fixed +
                                    300.0 * h.rt * f.ft + (U > 1 && g.n_groups % U ? 900.0 : 0.0);
            const double cost = (double)rounds * std::max(multiply, 20400.0 + 0.25 * vectors);
            if (cost < best_cost) {
                best_cost = cost;
                best = h;
            }
        }
    }
    return best;
}

// The split-plane kernel takes a plan if a shape fits LDS and its k-groups of 32 do not pad the
// frame by more than half (short hops do: at hop 8 three of four columns would be padding).
// 32 x 10 s, us, planes against the kernels on k-groups of 8 and 16.  Inside the line: FP32 N 400, hop 22,
// 80 Mel bins 209 : 339, 16 Mel bins 75 : 109; N 128, hop 20, 16 Mel bins 53 : 49.  Beyond it BF16X3
// loses where Mel bins are few or hops shorter still: N 400, hop 20, 16 Mel bins 63 : 52, 80 Mel bins
// 144 : 218; hop 12 140 : 66 and 332 : 273; N 128, hop 16, 16 Mel bins 50 : 30.  FP32 gains there down to
// hop 16 or so (hop 20 222 : 354, hop 12 540 : 593; 16 Mel bins 77 : 103, 176 : 174, N 128, hop 16
// 61 : 51): one line for both is drawn on the safe side.
static bool split_fits(const Plan &p) {
    return split_planes(p) && p.geoS.n_groups * 32 <= p.N + p.N / 2 + 32 && p.geoS.n_groups <= 512 &&
           split_shape(p.geoS, split_planes(p), (p.M + 7) / 8, p.cu_count, 1 << 20, (int64_t)kSplitChunk << 20).parts > 0;
}

// Frames of few samples and few Mel bins: the staging and hand-over of an item outweigh its products, and
// batches are the faster on the kernels that were there before (FP32 MFMA with staging waves, 16-bit
// frame-split).  64 clips of 30 s, us, planes against those: FP32 N 64, hop 32, 8 Mel bins 125 : 108,
// 24 Mel bins 119 : 153; N 128, hop 64, 8 Mel bins 68 : 72.  BF16X3, 16 Mel bins, N 40, hop 20
// 183 : 102, N 64 in one hop 57 : 57.  FP16X3, whose conversion costs the others more, only where the
// k-groups pad a frame by more than half (N 40, hop 20, 16 Mel bins 196 : 157).  One 1 s clip takes
// 9.1 us there where planes take 7.3.
static bool split_tiny(const Plan &p) {
    if (p.cfg.precision == MELT_PREC_FP16X3) return p.M <= 16 && 2 * p.geoS.n_groups * 32 > 3 * p.N;
    if (p.cfg.precision == MELT_PREC_BF16X3)
        return (p.M <= 16 && p.N < 128 && (p.N < 64 || p.H < p.N)) || (p.M <= 40 && p.N < 64);
    return p.M <= 16 && p.N < 128;
}

bool split_self_scheduled(const Plan &p, int64_t est_chunks, int64_t n_frames) {
    const int P = split_planes(p);
    const SplitShape h = split_shape(p.geoS, P, (p.M + 7) / 8, p.cu_count, est_chunks, n_frames);
    if (h.parts == 0 || split_lds(P, p.geoS, h) + kListBytes > (size_t)kMaxLds) return false;
    const int64_t items = est_chunks * (kSplitChunk / split_sf(h)) * h.parts;
    return items <= (int64_t)(kListEntries - 1) * split_grid(p, h, items);
}

static std::vector<Variant> variant_list(const Plan &p) {
    std::vector<Variant> v;
    switch (p.cfg.precision) {
    case MELT_PREC_FP32:
        // (the geometries the FP32-MFMA kernels refuse stay refused)
        if (f32_fits(p) && split_fits(p) && !split_tiny(p)) v.push_back({V_SPLIT, kSplitChunk});
        v.push_back({V_F32_WS, kBF32});
        v.push_back({V_F32_FS, kBF32});
        if (f32_fits(p) && split_fits(p) && split_tiny(p)) v.push_back({V_SPLIT, kSplitChunk});
        break;
    case MELT_PREC_FP8_E4M3: {
        // up to 8 row tiles: the largest all-wave chunk that fits LDS (one workgroup per CU),
        // then 64-frame chunks with two workgroups per CU; the producer/consumer kernel (two
        // images and two spans of 64-frame chunks) first beyond 8 row tiles, last otherwise
        const int ng8 = (p.N + 63) / 64;
        const bool pc = (ng8 == 4 || ng8 == 7 || ng8 == 8) && p.H % 4 == 0 && p.N % 4 == 0 &&
                        f8_pc_lds_bytes(p, 64) + 4 * sizeof(Chunk) + 8 * 32 * 4 <= (size_t)kMaxLds;
        if (f8fs_fits(p)) v.push_back({V_F8_FS, 128});
        if (pc && p.row_tiles > 8) v.push_back({V_F8_PC, 64});
        for (int bf : {128, 96, 64, 32})
            if (f8_as_lds_bytes(p, bf) + kRingBytes <= (size_t)kMaxLds) {
                v.push_back({V_F8_AS, bf});
                break;
            }
        if (!v.empty() && v.back().bf > 64 && 2 * (f8_as_lds_bytes(p, 64) + kRingBytes) <= (size_t)kMaxLds)
            v.push_back({V_F8_AS, 64});
        v.push_back({V_F8_RS, kBF32});
        if (pc && p.row_tiles <= 8) v.push_back({V_F8_PC, 64});
        break;
    }
    case MELT_PREC_FP8_E4M3_BLOCK32:
        // producer/consumer (the largest chunk whose two row buffers fit; three waves per SIMD,
        // so a basis tile of at most 8 k-groups of 64), then the one-buffer kernel at 160- and
        // 128-frame chunks
        for (int bf : {128, 96, 64})
            if ((p.N + 63) / 64 <= 8 && f8b_pc_lds_bytes(p, bf) + f8b_pc_static_bytes() <= (size_t)kMaxLds) {
                v.push_back({V_F8B_PC, bf});
                break;
            }
        for (int bf : {160, 128})
            if (f8b_lds_bytes(p, bf) + kRingBytes <= (size_t)kMaxLds) v.push_back({V_F8B_AS, bf});
        if (v.empty()) v.push_back({V_F8B_AS, 32});    // unsupported geometry: the launch reports it
        break;
    default: {
        const bool x3 = prec_split(p);
        // 12-wave producer/consumer first where it fits (96 then 64 frames per chunk), then row
        // pairs (two basis tiles per wave, 128 frames per chunk)
        if (!x3 && pc_fits(p))
            for (int bf : {96, 64})
                if (pc_lds_bytes(p, bf) + 4 * sizeof(Chunk) <= (size_t)kMaxLds) {
                    v.push_back({V_H16_PC, bf});
                    break;
                }
        // the split precisions' producer/consumer form (8 waves, hi and lo rows; 64-frame
        // chunks, row groups of at most 5 tiles): their default where it fits with at most 4
        // row groups (each group converts every chunk again: at 32 row tiles, 7 groups, the
        // row-split kernel is faster), the last variant otherwise
        const bool pc_x3 = x3 && pc_fits(p) && pc_x3_lds_bytes(p, 64) + 4 * sizeof(Chunk) <= (size_t)kMaxLds;
        const bool pc_x3_first = pc_x3 && (p.row_tiles + 4) / 5 <= 4;
        if (pc_x3_first) v.push_back({V_H16_PC, 64});
        // frame lengths without a register tile for it (N = 512, 480, ...): operand planes first
        // (512 ragged clips, N 512, M 128: 942 -> 676 us BF16X3; one 1 s clip: 23.2 -> 10.1 us)
        const bool split = x3 && !pc_fits(p) && h16_fs_fits(p) && split_fits(p);
        if (split && !split_tiny(p)) v.push_back({V_SPLIT, kSplitChunk});
        if (!x3 && ap_fits(p) && as_lds_bytes(p, 128) + kRingBytes <= (size_t)kMaxLds) v.push_back({V_H16_AP, 128});
        if (as_fits(p)) {
            // one span buffer (128 then 64 frames per chunk; 96 then 64 for BF16X3), then two
            for (int bf : {128, 96, 64}) {
                if (bf == (x3 ? 128 : 96)) continue;
                if (as_lds_bytes(p, bf) + kRingBytes <= (size_t)kMaxLds) v.push_back({V_H16_AS, bf, 1});
            }
            for (int bf : {96, 64})
                if (as_lds_bytes(p, bf, 2) + kRingBytes <= (size_t)kMaxLds) {
                    v.push_back({V_H16_AS, bf, 2});
                    break;
                }
        }
        // row pairs (two basis tiles per wave, 128 frames per chunk)
        if (pp_fits(p)) {
            // producer/consumer: one span (96 or 64 frames per chunk), then two spans
            for (int bf : {96, 64})
                if (pp_lds_bytes(p, bf, 1) + kRingBytes <= (size_t)kMaxLds) {
                    v.push_back({V_H16_PP, bf, 1});
                    break;
                }
            for (int bf : {96, 64})
                if (pp_lds_bytes(p, bf, 2) + kRingBytes <= (size_t)kMaxLds) {
                    v.push_back({V_H16_PP, bf, 2});
                    break;
                }
        }
        if (rs_fits(p)) v.push_back({V_H16_RS, 128});
        if (!x3 && !as_fits(p) && ks_fits(p))
            for (int bf : {64, 32})
                if (ks_lds_bytes(p, bf) + kRingBytes <= (size_t)kMaxLds) {
                    v.push_back({V_H16_KS, bf});
                    break;
                }
        if (pc_x3 && !pc_x3_first) v.push_back({V_H16_PC, 64});
        // frame-split: the fallback for every 16-bit precision (the split ones only where no
        // register-tile kernel applies)
        if (!x3 || v.empty()) v.push_back({V_H16_FS, kBF32});
        if (split && split_tiny(p)) v.push_back({V_SPLIT, kSplitChunk});
    }
    }
    return v;
}

void init_variants(Plan &p) {
    const std::vector<Variant> v = variant_list(p);
    p.n_variants = (int)std::min<size_t>(v.size(), Plan::kMaxVariants);
    for (int i = 0; i < p.n_variants; ++i) {
        p.var_kind[i] = v[i].kind;
        p.var_bf[i] = v[i].bf;
        p.var_nbuf[i] = v[i].nbuf;
    }
}

bool split_used(const Plan &p) {
    return std::count(p.var_kind, p.var_kind + p.n_variants, (int)V_SPLIT) > 0;
}

static Variant variant_at(const Plan &p, int i) {
    if (p.n_variants == 0) return {V_H16_FS, kBF32};    // unsupported geometry: the launch reports it
    const int k = i >= 0 && i < p.n_variants ? i : 0;
    return {(VariantKind)p.var_kind[k], p.var_bf[k], p.var_nbuf[k]};
}

int forward_variants(const Plan &p) { return p.n_variants; }

const char *forward_variant_name(const Plan &p, int i) {
    static thread_local char buf[64];
    if (i < 0 || i >= p.n_variants) return "none";
    const Variant v = variant_at(p, i);
    const char *k = v.kind == V_H16_PP   ? (v.nbuf == 2 ? "h16-producer-consumer-2span" : "h16-producer-consumer")
                    : v.kind == V_SPLIT  ? (p.cfg.precision == MELT_PREC_FP32 ? "f32-split-planes-frame-split"
                                                                              : "h16-split-planes-frame-split")
                    : v.kind == V_F32_WS ? "f32-frame-split-warp-specialised"
                    : v.kind == V_F32_FS ? "f32-frame-split"
                    : v.kind == V_H16_AS ? (v.nbuf == 2 ? "h16-row-split-lds-dma2" : "h16-row-split-lds-dma")
                    : v.kind == V_H16_AP ? "h16-row-pair-lds-dma"
                    : v.kind == V_H16_PC ? (p.cfg.precision == MELT_PREC_BF16X3 || p.cfg.precision == MELT_PREC_FP16X3
                                                ? "h16-producer-consumer-8w-lds-dma"
                                                : "h16-producer-consumer-12w-lds-dma")
                    : v.kind == V_H16_RS ? "h16-row-split"
                    : v.kind == V_H16_KS ? "h16-k-split-lds-dma"
                    : v.kind == V_H16_FS ? "h16-frame-split"
                    : v.kind == V_F8_AS  ? "f8-row-split-lds-dma"
                    : v.kind == V_F8_FS  ? "f8-frame-split"
                    : v.kind == V_F8_PC  ? "f8-producer-consumer-lds-dma"
                    : v.kind == V_F8B_AS ? "f8-block-scaled-lds-dma"
                    : v.kind == V_F8B_PC ? "f8-block-scaled-producer-consumer-lds-dma"
                                            : "f8-row-split";
    std::snprintf(buf, sizeof(buf), "%s-bf%d", k, v.bf);
    return buf;
}

int melt_chunk_frames(const Plan &p, int variant) { return variant_at(p, variant).bf; }
int melt_chunk_frames(const Plan &p) { return melt_chunk_frames(p, p.tune_variant); }

melt_status launch_melt_main(Plan &p, const float *d_wave, float *d_out, float *d_proj, hipStream_t s) {
    const int64_t n_frames = p.prepared_frames[0];
    if (n_frames < 0) return set_error(MELT_E_INVALID_ARG, "no batch prepared");
    if (n_frames == 0) return MELT_OK;
    const int v = p.prepared_variant;
    // chunk count bound: every clip ends in at most one partial chunk
    const int64_t est = n_frames / p.prepared_bf[0] + p.prepared_clips[0];
    if (p.K == 0)
        return launch_melt_table(p, v, p.d_chunks[0], p.d_nchunks, est, n_frames, d_wave, d_out, d_proj, s);
    // MFCCT (Eq. mfcct_matrix): log-Mel rows into the plan workspace, then C = L D^T
    melt_status st = ensure_lmel(p, n_frames);
    if (st == MELT_OK)
        st = launch_melt_table(p, v, p.d_chunks[0], p.d_nchunks, est, n_frames, d_wave, p.d_lmel, d_proj, s);
    if (st != MELT_OK) return st;
    return launch_cepstrum(p, p.d_lmel, n_frames, d_out, s);
}

static melt_status launch_variant(Plan &p, int variant, const FwdTask &t);

melt_status launch_melt_table(Plan &p, int variant, const Chunk *tab, const int *n_tab, int64_t est_chunks,
                              int64_t n_frames, const float *d_wave, float *d_out, float *d_proj, hipStream_t s) {
    return launch_variant(p, variant, FwdTask{tab, n_tab, est_chunks, n_frames, d_wave, d_out, d_proj, s});
}

// Whether a call's kernel finds its own chunks (schedule.h): one of the kernels that can, at most
// 64 clips (a wave's lanes), and few enough chunks that each workgroup's share fits its list of
// kListEntries or ring of kRing.  The shares: est_chunks over the workgroups of a row group (each
// kernel runs at least cu_count / row groups of them, and a row group is at least 4 tiles), or
// over the split kernel's items.  Measured at 64 x 30 s (5.3 us of schedule kernel, and the gap
// after it, saved): see the kernels; one 1 s clip, FP32: 13.1 -> 9.7 us a call.
static bool self_scheduled(const Plan &p, int variant, int n_clips, int64_t n_frames) {
    const Variant v = variant_at(p, variant);
    if (n_clips > 64) return false;
    const int64_t est = n_frames / v.bf + n_clips, groups = (p.row_tiles + 3) / 4;
    switch (v.kind) {
    case V_SPLIT: return split_self_scheduled(p, est, n_frames);
    case V_H16_PC:
    case V_F8B_PC: return pc_list_fits(p, v.kind == V_F8B_PC, v.bf) && est * groups <= (int64_t)kListEntries * p.cu_count;
    case V_F8_FS: return est <= (int64_t)kListEntries * p.cu_count;
    case V_H16_AS:
    case V_H16_KS:
    case V_F8_AS: return est * groups <= (int64_t)kRing * p.cu_count;
    default: return false;
    }
}

static melt_status launch_melt_clips(Plan &p, int variant, const ClipTable &clips, int64_t n_frames, const float *d_wave,
                                     float *d_out, float *d_proj, hipStream_t s) {
    FwdTask t{nullptr, nullptr, clips.cap, n_frames, d_wave, d_out, d_proj, s};
    t.clips = clips;
    return launch_variant(p, variant, t);
}

// The variant of one call, prepared batch or streaming state.  The FP8 kernels with per-frame scales
// give the same bits, so unless a variant is pinned a call may take either.  The frame-split one is the
// faster per frame, the row-split one per chunk (a chunk costs the first about the same however few
// its frames) and to start.  With clips of one length assumed, n_frames / n_clips frames each
// (N 400 and 80 Mel bins unless stated, us, frame-split against row-split):
//   from 4 row tiles, 64-frame chunks of at most one round of the CUs: row-split on those (16 x 4 s
//     14.1 : 11.9, one 1 s clip 11.8 : 9.7; below 4 row tiles frame-split, 24 Mel bins: 10.5 : 11.9)
//   chunks of 128 less than half full: row-split (512 x 0.3 s 22.3 : 17.5, 128 Mel bins 26.1 : 18.6;
//     three quarters full, 512 x 1 s, 28.4 : 28.8); below 4 row tiles less than a tenth, 3 row tiles
//     three tenths (512 x 0.1 s, 16 Mel bins, 15.9 : 12.5)
//   more than 64 clips and at most one round of 128-frame chunks, each a clip or (more than 6 row tiles,
//     the basis streamed) not: row-split (256 x 1 s 19.7 : 19.0, 128 Mel bins 22.3 : 20.5)
int call_variant(const Plan &p, int n_clips, int64_t n_frames) {
    const int v = p.tune_variant;
    if (p.tune_pinned || variant_at(p, v).kind != V_F8_FS || n_clips < 1 || n_frames < 1) return v;
    const int64_t each = (n_frames + n_clips - 1) / n_clips, c64 = n_clips * ((each + 63) / 64), c128 = n_clips * ((each + 127) / 128);
    bool small, large = false;                     // row-split on 64-frame chunks, on its largest
    if (p.row_tiles >= 4) {
        small = c64 <= p.cu_count;
        large = 2 * n_frames < 128 * c128 ||
                (n_clips > 64 && c128 <= p.cu_count && (each <= 128 || p.row_tiles > 6));
    } else {
        small = 10 * n_frames < (p.row_tiles == 3 ? 3 : 1) * 128 * c128;
    }
    int best = v;
    for (int i = 0; i < p.n_variants; ++i)
        if (p.var_kind[i] == V_F8_AS && (small ? p.var_bf[i] == 64 : large && best == v)) best = i;
    return best;
}

// The forward over a batch, which is the plan's prepared one afterwards: table 0 is written by the
// kernel where it schedules itself, and read by it otherwise.
melt_status launch_melt_forward(Plan &p, const int64_t *d_off, int n_clips, int64_t n_frames, const float *d_wave,
                                float *d_out, float *d_proj, hipStream_t s) {
    const int v = call_variant(p, n_clips, n_frames);
    if (!self_scheduled(p, v, n_clips, n_frames)) {
        const melt_status st = launch_schedule(p, 0, d_off, n_clips, melt_chunk_frames(p, v), n_frames, s, v);
        return st == MELT_OK ? launch_melt_main(p, d_wave, d_out, d_proj, s) : st;
    }
    ClipTable clips;
    melt_status st = prepare_clips(p, 0, d_off, n_clips, n_frames, melt_chunk_frames(p, v), v, clips, s);
    if (st != MELT_OK) return st;
    if (p.K == 0) return launch_melt_clips(p, v, clips, n_frames, d_wave, d_out, d_proj, s);
    st = ensure_lmel(p, n_frames);
    if (st == MELT_OK) st = launch_melt_clips(p, v, clips, n_frames, d_wave, p.d_lmel, d_proj, s);
    return st == MELT_OK ? launch_cepstrum(p, p.d_lmel, n_frames, d_out, s) : st;
}

static melt_status launch_variant(Plan &p, int variant, const FwdTask &t) {
    const Variant v = variant_at(p, variant);
    switch (v.kind) {
    case V_SPLIT: return p.cfg.precision == MELT_PREC_FP32 ? launch_melt_split_f32(p, t) : launch_melt_split_x3(p, t);
    case V_F32_WS: return launch_melt_f32(p, t, true);
    case V_F32_FS: return launch_melt_f32(p, t, false);
    case V_H16_PP: return launch_melt_h16(p, t, H16_PIPELINED, v.bf, v.nbuf);
    case V_H16_AS: return launch_melt_h16(p, t, H16_LDS_DMA, v.bf, v.nbuf);
    case V_H16_AP: return launch_melt_h16(p, t, H16_ROW_PAIR, v.bf);
    case V_H16_PC: return launch_melt_h16(p, t, H16_PC12, v.bf);
    case V_H16_RS: return launch_melt_h16(p, t, H16_REGISTER_STAGED, v.bf);
    case V_H16_KS: return launch_melt_h16(p, t, H16_K_SPLIT, v.bf);
    case V_H16_FS: return launch_melt_h16(p, t, H16_FRAME_SPLIT, v.bf);
    case V_F8_AS: return launch_melt_f8(p, t, true, v.bf);
    case V_F8_FS: return launch_melt_f8_fs(p, t);
    case V_F8_PC: return launch_melt_f8_pc(p, t, v.bf);
    case V_F8_RS: return launch_melt_f8(p, t, false, v.bf);
    case V_F8B_AS: return launch_melt_f8b(p, t, v.bf, false);
    case V_F8B_PC: return launch_melt_f8b(p, t, v.bf, true);
    }
    return set_error(MELT_E_UNSUPPORTED, "precision not implemented");
}

// ------------------------------------------------------------------ allocation-free forward
// melt_forward_noalloc keeps its chunk count and chunk table in a fixed device array instead
// of the plan's (growable) workspace, for callers that cannot allocate.  Every GPU the
// library runs on holds its own copy until the process ends; the host side reaches it only
// through the address hipGetSymbolAddress returns for that device (the array's name in host
// code is not a device address).  All calls on one GPU share it: calls that overlap in time
// on one GPU race.
constexpr size_t kScratchBytes = size_t(1) << 20;    // 1 MiB per device
constexpr size_t kScratchTable = 256;                // byte offset of the table (count at 0)
constexpr int64_t kScratchChunks = int64_t((kScratchBytes - kScratchTable) / sizeof(Chunk));
constexpr int kScratchDevices = 64;
static_assert(kScratchChunks == 32760, "chunk capacity stated in melt.h");

static __device__ __align__(256) unsigned char scratch[kScratchBytes];

static std::mutex g_scratch_mu;
static void *g_scratch_ptr[kScratchDevices] = {};

// Called once per device at plan creation, with `device` current.
melt_status scratch_init(int device) {
    if (device < 0 || device >= kScratchDevices) return set_error(MELT_E_UNSUPPORTED, "device index beyond 63");
    std::lock_guard<std::mutex> lock(g_scratch_mu);
    if (g_scratch_ptr[device]) return MELT_OK;
    void *ptr = nullptr;
    const melt_status st = hip_check(hipGetSymbolAddress(&ptr, HIP_SYMBOL(scratch)), "hipGetSymbolAddress(scratch)");
    if (st != MELT_OK) return st;
    g_scratch_ptr[device] = ptr;
    return MELT_OK;
}

melt_status forward_noalloc(Plan &p, const float *d_wave, const int64_t *d_off, int n_clips, int64_t n_frames,
                            float *d_out, hipStream_t s) {
    if (p.K > 0) return set_error(MELT_E_UNSUPPORTED, "melt_forward_noalloc: MELT_OUT_MFCC needs a log-Mel workspace");
    void *base = nullptr;
    {
        std::lock_guard<std::mutex> lock(g_scratch_mu);
        base = g_scratch_ptr[p.device];
    }
    if (!base) return set_error(MELT_E_HIP, "melt_forward_noalloc: no scratch address for this device");
    // (the limit is the plan's variant's, which the call falls back to where another needs more)
    const int bf = melt_chunk_frames(p, p.tune_variant);
    // every clip ends in at most one partial chunk
    int64_t need = n_frames / bf + n_clips + 1;
    if (need > kScratchChunks)
        return set_error(MELT_E_SHAPE, "melt_forward_noalloc: n_frames / " + std::to_string(bf) + " + n_clips + 1 = " +
                                           std::to_string(need) + " chunk entries exceed the 32760 of the scratch");
    int *n_tab = static_cast<int *>(base);
    Chunk *tab = reinterpret_cast<Chunk *>(static_cast<unsigned char *>(base) + kScratchTable);
    // the schedule kernels write the count unconditionally, so nothing in the scratch needs clearing
    int v = call_variant(p, n_clips, n_frames);
    if (n_frames / melt_chunk_frames(p, v) + n_clips + 1 > kScratchChunks) v = p.tune_variant;
    const int bc = melt_chunk_frames(p, v);
    need = n_frames / bc + n_clips + 1;
    if (self_scheduled(p, v, n_clips, n_frames)) {
        const ClipTable clips{d_off, n_clips, p.N, bc, (int)(need - 1), nullptr, nullptr};
        return launch_melt_clips(p, v, clips, n_frames, d_wave, d_out, nullptr, s);
    }
    const melt_status st = enqueue_schedule(p, d_off, n_clips, bc, need, tab, kScratchChunks, n_tab, s);
    if (st != MELT_OK) return st;
    return launch_melt_table(p, v, tab, n_tab, need - 1, n_frames, d_wave, d_out, nullptr, s);
}

}  // namespace melt
