// Gradient of the MelT forward on gfx950 (chain rule through Eqs. meltf, dmp_matrix_energy
// and dmp_projection; the paper has no backward pass).  For out = map(S), S = R^2 + I^2,
// R = X Wr^T, I = X Wi^T and upstream g:
//   G[t, 2m] = 2 R[t,m] g[t,m] map'(S),  G[t, 2m+1] = 2 I[t,m] g[t,m] map'(S)
//   dx[s]    = sum over (t, n) with start_t + n = s of (G W)[t, n]       (overlap-add)
//   dW       = G^T X                                                    (learnable basis)
// Everything is FP32, deterministic (no floating-point atomics); the two products run on three
// bfloat16 planes per operand (bwd_split.hip):
//   k_bwd_grad   G over every frame (a flat pass over the [T, M] gradient)
//   k_bwd_fstart the start sample of every frame
//   dx           owner-computes overlap-add: hop-block row b of dx is sum_j G[b - j] W_j,
//                W_j = basis columns [jH, jH + H); each sample is written once (k_bwd_dx, FP32
//                MFMA, where dx_split_fits says no: fewer than 5 Mel bins, or too many hops)
//   dW           split-K GEMM G^T X over frames into per-split partials
//   k_bwd_reduce fixed-order sum of the partials into the stacked [2M, N] gradient
#include <algorithm>

#include "bwd.h"

namespace melt {

typedef float f32x4 __attribute__((ext_vector_type(4)));
typedef float f32x16 __attribute__((ext_vector_type(16)));

constexpr int kMaxCT = 8;          // column tiles of 32 samples per hop-block row (H <= 256)

// ------------------------------------------------------------------ schedule of row chunks

__global__ __launch_bounds__(1024) void k_schedule_rows(const int64_t *__restrict__ off, int n_clips, int N, int H,
                                                        RowChunk *__restrict__ tab, int64_t cap, int *__restrict__ n_out) {
    __shared__ int64_t sf[1024], sc[1024];
    __shared__ int64_t carry_f, carry_c;
    const int tid = threadIdx.x;
    if (tid == 0) carry_f = carry_c = 0;
    __syncthreads();
    for (int base = 0; base < n_clips; base += 1024) {
        const int c = base + tid;
        int64_t st = 0, L = 0;
        if (c < n_clips) {
            st = off[c];
            L = off[c + 1] - st;
        }
        if (L < 0) L = 0;
        const int64_t T = (L >= N) ? 1 + (L - N) / H : 0;
        const int64_t R = (L + H - 1) / H;                      // rows covering the whole clip
        const int64_t K = (R + kRowsDx - 1) / kRowsDx;
        sf[tid] = T;
        sc[tid] = K;
        __syncthreads();
        for (int d = 1; d < 1024; d <<= 1) {
            const int64_t vf = tid >= d ? sf[tid - d] : 0;
            const int64_t vc = tid >= d ? sc[tid - d] : 0;
            __syncthreads();
            sf[tid] += vf;
            sc[tid] += vc;
            __syncthreads();
        }
        const int64_t fb = carry_f + sf[tid] - T;
        const int64_t cb = carry_c + sc[tid] - K;
        for (int64_t k = 0; k < K; ++k) {
            const int64_t idx = cb + k;
            if (idx >= cap) break;
            const int64_t b0 = k * kRowsDx;
            RowChunk e;
            e.sample_start = st + b0 * H;
            e.sample_end = st + L;
            e.g_row0 = fb + b0;
            e.n_rows = (int)((R - b0) < kRowsDx ? (R - b0) : kRowsDx);
            e.t_lo = (int)(-b0);
            e.t_hi = (int)(T - b0);
            e.pad = 0;
            tab[idx] = e;
        }
        __syncthreads();
        if (tid == 1023) {
            carry_f += sf[1023];
            carry_c += sc[1023];
        }
        __syncthreads();
    }
    if (tid == 0) *n_out = (int)(carry_c < cap ? carry_c : cap);
}

// ------------------------------------------------------------------ G and frame starts

__device__ __forceinline__ float map_dS(float S, int kind, float eps) {
    switch (kind) {
    case MELT_OUT_LOG_POWER: return 1.0f / (S + eps);
    case MELT_OUT_LOG_MAGNITUDE: {
        const float r = sqrtf(S);
        return S > 0.0f ? 1.0f / (2.0f * r * (r + eps)) : 0.0f;
    }
    case MELT_OUT_POWER: return 1.0f;
    default: return S > 0.0f ? 0.5f / sqrtf(S) : 0.0f;
    }
}

__global__ void k_fill_i64(int64_t *__restrict__ p, int64_t n, int64_t v) {
    for (int64_t i = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; i < n; i += (int64_t)gridDim.x * blockDim.x) p[i] = v;
}
__global__ void k_fill_f32(float *__restrict__ p, int64_t n, float v) {
    for (int64_t i = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; i < n; i += (int64_t)gridDim.x * blockDim.x) p[i] = v;
}

// G over every frame.  Element e = t M + m of the [T, M] upstream gradient pairs with
// projections proj[2e], proj[2e + 1] (R, I of Mel bin m) and G entries G[2e], G[2e + 1], so
// the pass is flat: two elements per thread step with 16-byte projection and G accesses and
// an 8-byte gradient load when vec (pointers aligned for them), one element otherwise.
__global__ __launch_bounds__(256) void k_bwd_grad(const float *__restrict__ gout, const float *__restrict__ proj,
                                                  int64_t n_elems, int kind, float eps, float *__restrict__ G,
                                                  int vec) {
    const int64_t stride = (int64_t)gridDim.x * blockDim.x;
    int64_t e0 = 0;
    if (vec) {
        const int64_t npairs = n_elems / 2;
        for (int64_t i = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; i < npairs; i += stride) {
            const f32x4 y = ((const f32x4 *)proj)[i];
            const float2 g = ((const float2 *)gout)[i];
            const float k0 = g.x * map_dS(y[0] * y[0] + y[1] * y[1], kind, eps);
            const float k1 = g.y * map_dS(y[2] * y[2] + y[3] * y[3], kind, eps);
            ((f32x4 *)G)[i] = f32x4{2.0f * y[0] * k0, 2.0f * y[1] * k0, 2.0f * y[2] * k1, 2.0f * y[3] * k1};
        }
        e0 = 2 * npairs;
    }
    for (int64_t e = e0 + blockIdx.x * (int64_t)blockDim.x + threadIdx.x; e < n_elems; e += stride) {
        const float r = proj[2 * e], im = proj[2 * e + 1];
        const float k = gout[e] * map_dS(r * r + im * im, kind, eps);
        G[2 * e] = 2.0f * r * k;
        G[2 * e + 1] = 2.0f * im * k;
    }
}

// Up to 64 clips: the start sample of every frame (-1 past the last one), the forward's chunk table
// (of which the backward itself reads nothing: its batch is the plan's prepared one afterwards) and
// the row chunks, from the clips in the lanes of each wave (schedule.h; a frame is a chunk of one).
// One launch where the chunk table, the fill, the frame starts and the row schedule were four.
__global__ __launch_bounds__(256) void k_bwd_tables(ClipTable b, int H, int64_t n_frames, int64_t *__restrict__ fstart,
                                                    RowChunk *__restrict__ rc, int64_t rc_cap, int *__restrict__ n_rc) {
    const int64_t *__restrict__ off = b.off;
    const int n_clips = b.n_clips, N = b.N;
    const int lane = threadIdx.x & 63, w = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    if (blockIdx.x + 1 == gridDim.x) {                   // the last workgroup: the chunk table
        if (!b.tab) return;
        const ClipScan s = clip_scan(off, n_clips, N, H, b.bf);
        const int64_t n = uniform64(s.total < b.cap ? s.total : b.cap);
        for (int64_t q0 = 64 * w; q0 < n; q0 += 256) {
            const Chunk e = clip_chunk(s, H, b.bf, q0 + lane);
            if (q0 + lane < n) b.tab[q0 + lane] = e;
        }
        if (threadIdx.x == 0) *b.n_tab = (int)n;
        return;
    }
    const int64_t wave = blockIdx.x * 4 + w, waves = (gridDim.x - 1) * 4;
    const ClipScan s = clip_scan(off, n_clips, N, H, 1);
    const int64_t total = uniform64(s.total);
    for (int64_t q0 = 64 * wave; q0 < n_frames; q0 += 64 * waves) {       // wave-uniform trip count
        const int64_t q = q0 + lane;
        const Chunk e = clip_chunk(s, H, 1, q);
        if (q < n_frames) fstart[q] = q < total ? e.sample_start : -1;
    }
    if (!rc) return;
    // rows covering the whole clip (samples in no frame get zero gradient)
    const int64_t L = s.L > 0 ? s.L : 0, R = (L + H - 1) / H, K = (R + kRowsDx - 1) / kRowsDx;
    const int64_t before = __shfl_up(s.pf, 1, 64), T = s.pf - (lane ? before : 0);
    const int64_t pk = wave_scan(K, lane), nk = uniform64(__shfl(pk, 63, 64)), n = nk < rc_cap ? nk : rc_cap;
    if (wave == 0 && lane == 0) *n_rc = (int)n;
    for (int64_t q0 = 64 * wave; q0 < n; q0 += 64 * waves) {
        const int64_t q = q0 + lane;
        int t = 0;                                                       // clips whose chunks all precede q
#pragma unroll
        for (int d = 32; d >= 1; d >>= 1)
            if (__shfl(pk, t + d - 1, 64) <= q) t += d;
        const int tp = t > 0 ? t - 1 : 0;
        const int64_t pk_p = __shfl(pk, tp, 64), pf_p = __shfl(s.pf, tp, 64);
        const int64_t st = __shfl(s.st, t & 63, 64), Lt = __shfl(L, t & 63, 64), Tt = __shfl(T, t & 63, 64);
        const int64_t b0 = (q - (t > 0 ? pk_p : 0)) * kRowsDx, Rt = (Lt + H - 1) / H;
        if (q < n)
            rc[q] = RowChunk{st + b0 * H, st + Lt, (t > 0 ? pf_p : 0) + b0, (int32_t)((Rt - b0) < kRowsDx ? (Rt - b0) : kRowsDx),
                             (int32_t)-b0, (int32_t)(Tt - b0), 0};
    }
}

// one workgroup per forward chunk: the start sample of each of its frames
__global__ __launch_bounds__(256) void k_bwd_fstart(const Chunk *__restrict__ chunks, const int *__restrict__ n_chunks,
                                                    int64_t n_frames, int H, int64_t *__restrict__ fstart) {
    const int nch = *n_chunks;
    for (int c = blockIdx.x; c < nch; c += gridDim.x) {
        const Chunk ch = chunks[c];
        for (int f = threadIdx.x; f < ch.n_frames; f += blockDim.x)
            if (ch.out_row + f < n_frames) fstart[ch.out_row + f] = ch.sample_start + (int64_t)f * H;
    }
}

// ------------------------------------------------------------------ dx: owner-computes overlap-add

// 4 waves x 32 hop-block rows; each wave computes its rows x all CT column tiles.  G rows
// [b0 - J + 1, b0 + 128) of the clip are staged in LDS (zero outside the clip's frames).
template <int CT>
__global__ __launch_bounds__(256) void k_bwd_dx(const RowChunk *__restrict__ rc, const int *__restrict__ n_rc,
                                                const float *__restrict__ G, const f32x4 *__restrict__ bpack,
                                                int M, int H, int J, int S, int64_t n_frames, float *__restrict__ dx) {
    extern __shared__ float lds[];
    const int tid = threadIdx.x, lane = tid & 63, wid = tid >> 6;
    const int Q = 2 * M, QG = (Q + 7) / 8;
    const int nch = *n_rc;
    for (int c = blockIdx.x; c < nch; c += gridDim.x) {
        const RowChunk ch = rc[c];
        __syncthreads();
        // LDS row r holds G of chunk-local frame r - (J - 1)
        const int rows = ch.n_rows + J - 1;
        for (int i = tid; i < rows * QG * 8; i += 256) {
            const int r = i / (QG * 8), q = i - r * (QG * 8);
            const int tl = r - (J - 1);
            float v = 0.0f;
            if (q < Q && tl >= ch.t_lo && tl < ch.t_hi && ch.g_row0 + tl < n_frames) v = G[(ch.g_row0 + tl) * Q + q];
            lds[r * S + q] = v;
        }
        __syncthreads();
        const int rbase = wid * 32;
        if (rbase >= ch.n_rows) continue;
        f32x16 acc[CT];
#pragma unroll
        for (int t = 0; t < CT; ++t) acc[t] = f32x16{};
        for (int j = 0; j < J; ++j) {
            // output row i uses G of frame (i - j): LDS row i - j + J - 1
            const float *lp = lds + (rbase + (lane & 31) + J - 1 - j) * S + 4 * (lane >> 5);
            const f32x4 *bp = bpack + ((size_t)j * QG) * 64 + lane;
            for (int qg = 0; qg < QG; ++qg) {
                const f32x4 a = *(const f32x4 *)(lp + qg * 8);
                f32x4 b[CT];
#pragma unroll
                for (int t = 0; t < CT; ++t) b[t] = bp[((size_t)t * J * QG + qg) * 64];
#pragma unroll
                for (int i = 0; i < 4; ++i)
#pragma unroll
                    for (int t = 0; t < CT; ++t)
                        acc[t] = __builtin_amdgcn_mfma_f32_32x32x2f32(a[i], b[t][i], acc[t], 0, 0, 0);
            }
        }
        // acc[t]: lane holds sample column 32 t + lane % 32 of rows 8(r/4) + 4h + r%4
        const int h = lane >> 5, col = lane & 31;
#pragma unroll
        for (int t = 0; t < CT; ++t) {
            const int cc = t * 32 + col;
            if (cc >= H) continue;
#pragma unroll
            for (int r = 0; r < 16; ++r) {
                const int row = rbase + 8 * (r >> 2) + 4 * h + (r & 3);
                if (row >= ch.n_rows) continue;
                const int64_t s = ch.sample_start + (int64_t)row * H + cc;
                if (s < ch.sample_end) dx[s] = acc[t][r];
            }
        }
    }
}

// ------------------------------------------------------------------ dW

// Sums the splits' partials in split order (so the result does not depend on the launch),
// four consecutive n per thread with 16-byte loads when N is a multiple of 4, eight splits'
// loads in flight at a time.
__global__ void k_bwd_reduce(const float *__restrict__ part, int splits, int M, int N, float *__restrict__ dW) {
    const int64_t total = (int64_t)2 * M * N;
    if ((N & 3) == 0) {
        const int64_t total4 = total / 4;
        for (int64_t i = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; i < total4;
             i += (int64_t)gridDim.x * blockDim.x) {
            f32x4 s = f32x4{0.0f, 0.0f, 0.0f, 0.0f};
            int k = 0;
            for (; k + 8 <= splits; k += 8) {
                f32x4 v[8];
#pragma unroll
                for (int u = 0; u < 8; ++u) v[u] = *(const f32x4 *)(part + (size_t)(k + u) * total + 4 * i);
#pragma unroll
                for (int u = 0; u < 8; ++u) s += v[u];
            }
            for (; k < splits; ++k) s += *(const f32x4 *)(part + (size_t)k * total + 4 * i);
            const int q = (int)((4 * i) / N), n = (int)(4 * i - (int64_t)q * N);
            *(f32x4 *)(dW + (size_t)((q & 1) * M + (q >> 1)) * N + n) = s;   // interleaved q -> stacked rows
        }
        return;
    }
    for (int64_t i = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; i < total; i += (int64_t)gridDim.x * blockDim.x) {
        float s = 0.0f;
        for (int k = 0; k < splits; ++k) s += part[(size_t)k * total + i];
        const int q = (int)(i / N), n = (int)(i - (int64_t)q * N);
        dW[(size_t)((q & 1) * M + (q >> 1)) * N + n] = s;    // interleaved q -> stacked rows
    }
}

// ------------------------------------------------------------------ host side

namespace {

melt_status grow(void **p, size_t *cap, size_t need) {
    if (need <= *cap) return MELT_OK;
    void *d = nullptr;
    if (hipMalloc(&d, need) != hipSuccess) return set_error(MELT_E_NO_MEMORY, "backward workspace");
    if (*p) {
        (void)hipDeviceSynchronize();
        (void)hipFree(*p);
    }
    *p = d;
    *cap = need;
    return MELT_OK;
}

template <int CT>
melt_status launch_dx(Plan &p, const float *G, int64_t n_frames, float *dx, int S, size_t lds, int grid, hipStream_t s) {
    (void)hipFuncSetAttribute((const void *)k_bwd_dx<CT>, hipFuncAttributeMaxDynamicSharedMemorySize, 160 * 1024);
    k_bwd_dx<CT><<<grid, 256, lds, s>>>((const RowChunk *)p.d_bwd_rows, p.d_nchunks + 1, G, (const f32x4 *)p.d_pack_dx,
                                        p.M, p.H, p.geo32.J, S, n_frames, dx);
    return hip_check(hipGetLastError(), "bwd dx launch");
}

}  // namespace

melt_status pack_dx_job(Plan &p, PackJobs &jobs) {
    const int CT = (p.H + 31) / 32;
    if (CT > kMaxCT) return MELT_OK;     // dx unsupported for this hop; reported at call time
    const int J = p.geo32.J, QG = (2 * p.M + 7) / 8;
    const bool split = dx_split_fits(p);
    const size_t need = split ? dx_split_pack_bytes(p) : (size_t)CT * J * QG * 64 * 4 * sizeof(float);
    const melt_status st = grow(&p.d_pack_dx, &p.pack_dx_cap, need);
    if (st == MELT_OK) jobs.add(split ? dx_split_job(p, p.d_pack_dx) : PackJob{PACK_DX, p.d_pack_dx, nullptr, nullptr, J, CT, 0});
    return st;
}

melt_status launch_melt_backward(Plan &p, const float *d_wave, const int64_t *d_off, int n_clips, int64_t n_frames,
                                 const float *d_gout, const float *d_proj, float *d_gwave, float *d_gbasis,
                                 hipStream_t s) {
    if (n_clips == 0 || n_frames == 0) {
        // a fill kernel rather than a memset, so that the call can be captured in a HIP graph
        if (d_gbasis) {
            k_fill_f32<<<64, 256, 0, s>>>(d_gbasis, (int64_t)2 * p.M * p.N, 0.0f);
            return hip_check(hipGetLastError(), "bwd fill");
        }
        return MELT_OK;
    }
    const int M = p.M, N = p.N, H = p.H, J = p.geo32.J, Q = 2 * M;
    const int CT = (H + 31) / 32;
    if (d_gwave && CT > kMaxCT) return set_error(MELT_E_UNSUPPORTED, "backward d/dwave supports hop <= 256");
    // workspace: proj (if recomputed) | G | frame starts | dW partials
    // dW: blocks of the basis, split over frames so that about one workgroup per CU runs, down
    // to two steps of 32 frames each (one: 43.2 us a backward of 1584 frames, N = 400, where
    // this takes 41.6: the sum over the splits grows)
    const int dw_blocks = dw_split_blocks(p);
    const int splits = (int)std::max<int64_t>(
        1, std::min<int64_t>({64, ((int64_t)p.cu_count + dw_blocks - 1) / dw_blocks, (n_frames + 63) / 64}));
    const size_t proj_b = d_proj ? 0 : sizeof(float) * n_frames * Q;
    const size_t g_b = sizeof(float) * n_frames * Q;
    const size_t fs_b = sizeof(int64_t) * n_frames;
    const size_t part_b = d_gbasis ? sizeof(float) * splits * Q * N : 0;
    const size_t gl_b = p.K > 0 ? sizeof(float) * n_frames * M : 0;   // dL = dC D under MFCC
    auto al = [](size_t x) { return (x + 255) & ~size_t(255); };
    melt_status st = grow(&p.d_bwd_ws, &p.bwd_ws_cap, al(proj_b) + al(g_b) + al(fs_b) + al(part_b) + al(gl_b) + 256);
    if (st != MELT_OK) return st;
    char *w = (char *)p.d_bwd_ws;
    float *proj_ws = (float *)w;
    float *G = (float *)(w + al(proj_b));
    int64_t *fstart = (int64_t *)(w + al(proj_b) + al(g_b));
    float *part = (float *)(w + al(proj_b) + al(g_b) + al(fs_b));
    if (p.K > 0) {
        // the cepstrum is linear: upstream over the log-Mel rows is dC D
        float *gl = (float *)(w + al(proj_b) + al(g_b) + al(fs_b) + al(part_b));
        st = launch_row_matmul(d_gout, n_frames, p.K, M, p.d_dct, 1, M, gl, s);
        if (st != MELT_OK) return st;
        d_gout = gl;
    }
    const float *proj = d_proj;
    if (!proj) {
        // recomputed; G's space holds the (unused) output of the recomputation first
        st = launch_melt_forward(p, d_off, n_clips, n_frames, d_wave, G, proj_ws, s);
        if (st != MELT_OK) return st;
        proj = proj_ws;
    }
    // frame starts and, for dx, row chunks: rows cover every sample of every clip (samples no
    // frame covers get 0: their G rows are zero)
    const int64_t rows_cap = n_frames / kRowsDx + 2 * (int64_t)n_clips + 2 + (int64_t)n_clips * (J + 1);
    if (d_gwave) {
        st = grow(&p.d_bwd_rows, &p.bwd_rows_cap, sizeof(RowChunk) * rows_cap);
        if (st != MELT_OK) return st;
    }
    const int64_t rc_cap = (int64_t)(p.bwd_rows_cap / sizeof(RowChunk));
    if (n_clips <= 64) {
        const int grid = (int)std::max<int64_t>(1, std::min<int64_t>((n_frames + 255) / 256, p.cu_count));
        const int v = call_variant(p, n_clips, n_frames);
        ClipTable clips;
        st = prepare_clips(p, 0, d_off, n_clips, n_frames, melt_chunk_frames(p, v), v, clips, s);
        if (st != MELT_OK) return st;
        k_bwd_tables<<<grid + 1, 256, 0, s>>>(clips, H, n_frames, fstart, d_gwave ? (RowChunk *)p.d_bwd_rows : nullptr, rc_cap,
                                          p.d_nchunks + 1);
        st = hip_check(hipGetLastError(), "bwd tables");
        if (st != MELT_OK) return st;
    } else {
        // (the forward over more than 64 clips has built the chunk table)
        const int v = call_variant(p, n_clips, n_frames);
        if (d_proj) st = launch_schedule(p, 0, d_off, n_clips, melt_chunk_frames(p, v), n_frames, s, v);
        if (st != MELT_OK) return st;
        k_fill_i64<<<256, 256, 0, s>>>(fstart, n_frames, -1);
        const int64_t nchunk_est = n_frames / p.prepared_bf[0] + n_clips + 1;
        const int grid_prep = (int)std::min<int64_t>(nchunk_est, (int64_t)p.cu_count * 4);
        k_bwd_fstart<<<grid_prep, 256, 0, s>>>(p.d_chunks[0], p.d_nchunks, n_frames, H, fstart);
        if (d_gwave)
            k_schedule_rows<<<1, 1024, 0, s>>>(d_off, n_clips, N, H, (RowChunk *)p.d_bwd_rows, rc_cap, p.d_nchunks + 1);
        st = hip_check(hipGetLastError(), "bwd tables");
        if (st != MELT_OK) return st;
    }
    if (d_gwave) p.prepared_frames[1] = -1;      // table 1's count now describes row chunks
    {
        const int64_t n_elems = n_frames * M;
        const int vec = ((uintptr_t)proj % 16 == 0) && ((uintptr_t)d_gout % 8 == 0) && ((uintptr_t)G % 16 == 0);
        const int grid_g = (int)std::max<int64_t>(1, std::min<int64_t>((n_elems / 2 + 255) / 256, (int64_t)p.cu_count * 8));
        k_bwd_grad<<<grid_g, 256, 0, s>>>(d_gout, proj, n_elems, p.kern_out, (float)p.cfg.log_eps, G, vec);
    }
    st = hip_check(hipGetLastError(), "bwd gradient of the projections");
    if (st != MELT_OK) return st;
    if (d_gwave) {
        const int S = ((Q + 7) / 8) * 8 + 4;
        const size_t lds = (size_t)(kRowsDx + J - 1) * S * sizeof(float);
        if (lds > 160 * 1024) return set_error(MELT_E_UNSUPPORTED, "backward LDS too large (n_mels * hop)");
        const int64_t n_rc = n_frames / kRowsDx + n_clips + 1;
        const int grid = (int)std::min<int64_t>(n_rc, p.cu_count);
        if (dx_split_fits(p))
            st = launch_dx_split(p, G, (const RowChunk *)p.d_bwd_rows, p.d_nchunks + 1, n_rc, n_frames, d_gwave, s);
        else switch (CT) {
        case 1: st = launch_dx<1>(p, G, n_frames, d_gwave, S, lds, grid, s); break;
        case 2: st = launch_dx<2>(p, G, n_frames, d_gwave, S, lds, grid, s); break;
        case 3: st = launch_dx<3>(p, G, n_frames, d_gwave, S, lds, grid, s); break;
        case 4: st = launch_dx<4>(p, G, n_frames, d_gwave, S, lds, grid, s); break;
        case 5: st = launch_dx<5>(p, G, n_frames, d_gwave, S, lds, grid, s); break;
        case 6: st = launch_dx<6>(p, G, n_frames, d_gwave, S, lds, grid, s); break;
        case 7: st = launch_dx<7>(p, G, n_frames, d_gwave, S, lds, grid, s); break;
        default: st = launch_dx<8>(p, G, n_frames, d_gwave, S, lds, grid, s); break;
        }
        if (st != MELT_OK) return st;
    }
    if (d_gbasis) {
        st = launch_dw_split(p, G, fstart, d_wave, n_frames, splits, part, s);
        if (st != MELT_OK) return st;
        k_bwd_reduce<<<512, 256, 0, s>>>(part, splits, M, N, d_gbasis);
        st = hip_check(hipGetLastError(), "bwd reduce");
    }
    return st;
}

}  // namespace melt
