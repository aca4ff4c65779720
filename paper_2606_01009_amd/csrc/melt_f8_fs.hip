// MelT forward, FP8 with per-frame scales, frame-split: the frames are quantised on their way
// into the matrix cores.
//
// The row-split kernel (melt_f8.hip) runs maxima, scales, an E4M3 image of every frame and the
// multiplies as phases between barriers, each waiting on memory or LDS with all its waves.
// Here a multiply wave owns 32 frames of a 128-frame chunk and all row tiles: it takes its
// frames' maxima from the FP32 hop-block rows in LDS (one pass), then walks the k-groups of 64,
// reading a lane's 32 samples, scaling and rounding them in registers (48 VALU instructions)
// into the B operand of RT MFMAs.  No image.  The basis (2 KB per tile and k-group, 70 KB for 80
// Mel bins at N = 400) sits in LDS where it fits beside the rows, else its fragments stream from
// L2 through a ring of registers (a fragment feeds one MFMA of 64 cycles on each of four waves,
// and L1 delivers 64 bytes a cycle: 56.9 us that way, 50.5 us from LDS, side by side).  Four more
// waves stage: they hold the samples of the next two chunks in registers, one landed and one in
// flight, and write the landed one to LDS between the two barriers of a chunk, while the multiply
// waves store.  Hop a multiple of 32 (a lane's 32 samples then lie in one row) and small enough that two
// chunks fit the stagers' registers.
//
// What bounds it: HBM (184.5 MB on 64 x 30 s, 26 us at the rate of a copy of this size and 36 at that
// of one beyond the caches) up to 2 or 3 row tiles (24 Mel bins: 38.6 us a call), then the multiply
// waves' LDS reads and conversions.  Measured against the row-split kernel, whole calls of 64 x 30 s:
// 80 Mel bins 73.2 -> 50.5 us (up to 55 on other cards, where the row-split one takes 77-80), 24 Mel
// bins 92.6 -> 38.6 us, 128 Mel bins 81.5 -> 76.1 us (eight row tiles spill four registers), N 256
// 71.6 -> 49.0 us, N 512 with 128 Mel bins 97.2 -> 93.2 us.  Where calls are small or clips short
// the row-split kernel is the faster: call_variant (melt_fwd.hip).
#include "fwd_common.h"

namespace melt {

constexpr int kF8fsFrames = 128;

// Issues a chunk's loads: vector v of thread lt is span samples 4 (lt + 256 v) .. + 3, zero past
// the clip end.
template <int PV>
__device__ __forceinline__ void f8fs_issue(const FwdArgs &a, const Chunk &ch, int lt, f32x4 (&x)[PV]) {
    const int span = (ch.n_frames + a.J - 1) * a.H;
    const int64_t left = ch.sample_end - ch.sample_start;
    const bool inside = left >= span;
    const int records = (int)(inside ? span : left > 0 ? left : 0);
    const __amdgpu_buffer_rsrc_t rs =
        __builtin_amdgcn_make_buffer_rsrc((void *)(a.wave + ch.sample_start), (short)0, records * 4, 0x00020000);
    asm volatile("" : "+v"(lt));        // addresses formed here, not kept from chunk to chunk
    if (inside) {
#pragma unroll
        for (int v = 0; v < PV; ++v) {
            const int o = 4 * (lt + v * 256);
            x[v] = __builtin_bit_cast(f32x4, __builtin_amdgcn_raw_buffer_load_b128(rs, o < span ? o * 4 : 0, 0, 0));
        }
    } else {
        // 4-byte loads, every one issued: an offset past the descriptor reads as zero
#pragma unroll
        for (int v = 0; v < PV; ++v)
#pragma unroll
            for (int e = 0; e < 4; ++e) {
                const int o = 4 * (lt + v * 256) + e;
                x[v][e] = __builtin_bit_cast(
                    float, __builtin_amdgcn_raw_buffer_load_b32(rs, o < records ? o * 4 : 0x7ffffff0, 0, 0));
            }
    }
}

template <int PV>
__device__ __forceinline__ void f8fs_write(const FwdArgs &a, const Chunk &ch, int lt, const f32x4 (&x)[PV], float *rows) {
    const int span = (ch.n_frames + a.J - 1) * a.H;
    asm volatile("" : "+v"(lt));
#pragma unroll
    for (int v = 0; v < PV; ++v) {
        const int o = 4 * (lt + v * 256);
        if (o < span) {
            const int r = span_row(a, o);
            *(f32x4 *)(rows + r * a.S + (o - r * a.H)) = x[v];
        }
    }
}

template <int NG, int RT, int PV, bool BL>
__global__ __attribute__((amdgpu_flat_work_group_size(512, 512), amdgpu_waves_per_eu(2, 2)))
void k_melt_f8_fs(FwdArgs a, const i32x8 *__restrict__ bq, const float *__restrict__ rinv_g, int N,
                  int basis_off) {
    extern __shared__ __attribute__((aligned(16))) float rows[];
    __shared__ __align__(16) float rinv_s[RT * 32];
    const int lane = threadIdx.x & 63;
    const int wid = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int G = gridDim.x;
    int c = blockIdx.x, k = 0;
    for (int i = threadIdx.x; i < 32 * min(RT, a.row_tiles); i += 512) rinv_s[i] = rinv_g[i];
    // BL: the basis in LDS, the two 16-byte halves of a fragment's lanes 1 KB apart
    unsigned char *bl = reinterpret_cast<unsigned char *>(rows) + basis_off;
    if constexpr (BL) {
        for (int i = threadIdx.x; i < RT * NG * 128; i += 512)
            *(uint4 *)(bl + (i >> 7) * 2048 + (i & 1) * 1024 + (i >> 1 & 63) * 16) = reinterpret_cast<const uint4 *>(bq)[i];
    }
    const bool own = a.clips.off != nullptr;
    Chunk *list = reinterpret_cast<Chunk *>(reinterpret_cast<char *>(rows) + a.list_off);
    const int nch = own ? list_start(a, list, c + (int64_t)lane * G) : *a.n_chunks;
    // chunk k of the workgroup (index ci), wave-uniform
    auto chunk_at = [&](int ci, int kk) {
        Chunk e;
        if (own) {
            e = list[kk];
            e.sample_start = uniform64(e.sample_start);
            e.sample_end = uniform64(e.sample_end);
            e.out_row = uniform64(e.out_row);
            e.n_frames = __builtin_amdgcn_readfirstlane(e.n_frames);
            return e;
        }
        uint4 lo, hi;
        load_chunk_scalar(a.chunks, ci, lo, hi);
        e.sample_start = (int64_t)(((uint64_t)lo.y << 32) | lo.x);
        e.sample_end = (int64_t)(((uint64_t)lo.w << 32) | lo.z);
        e.out_row = (int64_t)(((uint64_t)hi.y << 32) | hi.x);
        e.n_frames = (int)hi.z;
        e.clip = 0;
        return e;
    };
    if (wid >= 4) {
        const int lt = (int)threadIdx.x - 256;
        f32x4 x0[PV], x1[PV];
        if (c < nch) {
            const Chunk ch = chunk_at(c, 0);
            f8fs_issue<PV>(a, ch, lt, x0);
            f8fs_write<PV>(a, ch, lt, x0, rows);
        }
        __syncthreads();                           // rows of the first chunk ready
        if (c + G < nch) f8fs_issue<PV>(a, chunk_at(c + G, 1), lt, x0);
        for (; c < nch; c += 2 * G, k += 2) {
            // two chunks per turn, so that each register set has a name of its own
            if (c + 2 * G < nch) f8fs_issue<PV>(a, chunk_at(c + 2 * G, k + 2), lt, x1);
            __syncthreads();                       // A: the multiply waves are done with the rows
            if (c + G < nch) f8fs_write<PV>(a, chunk_at(c + G, k + 1), lt, x0, rows);
            __syncthreads();                       // B: rows of chunk k + 1 ready
            if (c + G >= nch) break;
            if (c + 3 * G < nch) f8fs_issue<PV>(a, chunk_at(c + 3 * G, k + 3), lt, x0);
            __syncthreads();                       // A
            if (c + 2 * G < nch) f8fs_write<PV>(a, chunk_at(c + 2 * G, k + 2), lt, x1, rows);
            __syncthreads();                       // B
        }
        return;
    }
    constexpr int D = RT >= 8 ? 4 : RT == 6 ? 3 : RT >= 3 ? RT : 4, U = D > RT ? D / RT : 1;
    static_assert((U * RT) % D == 0, "the ring's slots repeat every U k-groups");
    const __amdgpu_buffer_rsrc_t brs =
        __builtin_amdgcn_make_buffer_rsrc((void *)bq, (short)0, a.row_tiles * NG * 2048, 0x00020000);
    const int voff = lane * 32;
    uint4 A[D][2];
    auto load_a = [&](int slot, int r, int g) {
        if constexpr (BL) {
            const unsigned char *f = bl + (r * NG + g) * 2048 + lane * 16;
            A[slot][0] = *(const uint4 *)f;
            A[slot][1] = *(const uint4 *)(f + 1024);
            return;
        }
        const int so = (min(r, a.row_tiles - 1) * NG + g) * 2048;
        A[slot][0] = __builtin_bit_cast(uint4, __builtin_amdgcn_raw_buffer_load_b128(brs, voff, so, 0));
        A[slot][1] = __builtin_bit_cast(uint4, __builtin_amdgcn_raw_buffer_load_b128(brs, voff + 16, so, 0));
    };
    if constexpr (!BL) {
#pragma unroll
        for (int s = 0; s < D; ++s) load_a(s, s % RT, s / RT);
    }
    // LDS offset of the lane's 32 samples of each k-group, n = 64 g + 32 h: hop-block row n / H
    // (blocks past the frame read its first; they are cleared below)
    int goff[NG];
#pragma unroll
    for (int g = 0; g < NG; ++g) {
        const int n = 64 * g + 32 * (lane >> 5), nn = n < N ? n : 0, r = nn / a.H;
        goff[g] = r * a.S + nn - r * a.H;
    }
    __syncthreads();                               // rows of the first chunk (and the basis) ready
    if constexpr (BL) {
#pragma unroll
        for (int s = 0; s < D; ++s) load_a(s, s % RT, s / RT);
    }
    const int fbase = wid * 32, f_local = fbase + (lane & 31);
    const float *lp = rows + f_local * a.S;
    for (; c < nch; c += G, ++k) {
        const Chunk ch = chunk_at(c, k);
        const bool active = fbase < ch.n_frames;
        f32x16 acc[RT];
#pragma unroll
        for (int r = 0; r < RT; ++r) acc[r] = f32x16{};
        float is = 0.0f;
        if (active) {
            auto vec = [&](int g, int i) {
                f32x4 v = *(const f32x4 *)(lp + goff[g] + 4 * i);
                if (g == NG - 1) {                 // samples at or past N are zero
                    const int n = 64 * g + 32 * (lane >> 5) + 4 * i;
#pragma unroll
                    for (int e = 0; e < 4; ++e) v[e] = n + e < N ? v[e] : 0.0f;
                }
                return v;
            };
            float mx = 0.0f;
#pragma unroll
            for (int g = 0; g < NG; ++g)
#pragma unroll
                for (int i = 0; i < 8; ++i) {
                    const f32x4 v = vec(g, i);
                    mx = fmaxf(mx, fmaxf(fmaxf(fabsf(v[0]), fabsf(v[1])), fmaxf(fabsf(v[2]), fabsf(v[3]))));
                }
            mx = fmaxf(mx, __shfl_xor(mx, 32, 64));
            const float sc = mx > 0.0f ? __fdiv_rn(448.0f, mx) : 1.0f;
            is = 1.0f / sc;
            f32x4 X[8];
#pragma unroll
            for (int i = 0; i < 8; ++i) X[i] = vec(0, i);
#pragma unroll
            for (int g = 0; g < NG; ++g) {
                i32x8 B;
#pragma unroll
                for (int i = 0; i < 8; ++i)
                    B[i] = (int)fp8x4(__fmul_rn(X[i][0], sc), __fmul_rn(X[i][1], sc), __fmul_rn(X[i][2], sc),
                                      __fmul_rn(X[i][3], sc));
                // the next group's samples are read while this group multiplies
                if (g + 1 < NG) {
#pragma unroll
                    for (int i = 0; i < 8; ++i) X[i] = vec(g + 1, i);
                }
                __builtin_amdgcn_sched_barrier(0);
#pragma unroll
                for (int r = 0; r < RT; ++r) {
                    const int slot = (g % U * RT + r) % D;
                    const uint4 lo = A[slot][0], hi = A[slot][1];
                    const i32x8 Af = {(int)lo.x, (int)lo.y, (int)lo.z, (int)lo.w, (int)hi.x, (int)hi.y, (int)hi.z, (int)hi.w};
                    acc[r] = __builtin_amdgcn_mfma_scale_f32_32x32x64_f8f6f4(Af, B, acc[r], 0, 0, 0, 127, 0, 127);
                    __builtin_amdgcn_sched_barrier(0);
                    // the slot's next tile, D steps on (past the last group: the next chunk's first)
                    const int step = g * RT + r + D;
                    load_a(slot, step % RT, step / RT % NG);
                    __builtin_amdgcn_sched_barrier(0);
                }
            }
            // where NG is no multiple of U the tiles sit in rotated slots: refill
            if (U > 1 && NG % U != 0) {
#pragma unroll
                for (int s = 0; s < D; ++s) load_a(s, s % RT, s / RT);
            }
        }
        __syncthreads();                           // A: every row read
        if (active) {
            const float *ri = rinv_s + 4 * (lane >> 5);
            const float isf = f_local < ch.n_frames ? is : 0.0f;
#pragma unroll
            for (int r = 0; r < RT; ++r) {
                if (r >= a.row_tiles) continue;
#pragma unroll
                for (int q = 0; q < 4; ++q) {
                    const f32x4 r4 = *(const f32x4 *)(ri + 32 * r + 8 * q);
#pragma unroll
                    for (int e = 0; e < 4; ++e) acc[r][4 * q + e] = acc[r][4 * q + e] * (isf * r4[e]);
                }
                store_tile(a, ch, r, f_local, lane, acc[r]);
            }
        }
        __syncthreads();                           // B: rows of the next chunk ready
    }
}

// ------------------------------------------------------------------ launch

static size_t f8fs_rows_bytes(const Plan &p) { return (size_t)(kF8fsFrames + p.geo32.J - 1) * lds_stride(p.geo32.Hp, 4) * 4; }

bool f8fs_fits(const Plan &p) {
    const int ng = (p.N + 63) / 64;
    return (ng == 4 || ng == 7 || ng == 8) && p.H % 32 == 0 && p.row_tiles <= 8 &&
           (kF8fsFrames + p.geo32.J - 1) * p.H <= 22 * 1024 && f8fs_rows_bytes(p) + kListBytes + 8 * 32 * 4 <= (size_t)kMaxLds;
}

template <int NG, int RT>
static melt_status launch_f8fs_rt(const Plan &p, const FwdArgs &a, size_t lds, int grid, hipStream_t s) {
    const size_t basis = (size_t)RT * NG * 2048;
    if (RT <= 5 && RT == p.row_tiles && lds + basis + RT * 32 * 4 <= (size_t)kMaxLds) {
        const int off = (int)lds;
        lds += basis;
        constexpr int R = RT <= 5 ? RT : 5;
        if ((kF8fsFrames + a.J - 1) * a.H <= 17 * 1024) {
            allow_lds(k_melt_f8_fs<NG, R, 17, true>, R * 32 * 4);
            k_melt_f8_fs<NG, R, 17, true><<<grid, 512, lds, s>>>(a, (const i32x8 *)p.d_pack_f8, p.d_rowscale, p.N, off);
        } else {
            allow_lds(k_melt_f8_fs<NG, R, 22, true>, R * 32 * 4);
            k_melt_f8_fs<NG, R, 22, true><<<grid, 512, lds, s>>>(a, (const i32x8 *)p.d_pack_f8, p.d_rowscale, p.N, off);
        }
        return hip_check(hipGetLastError(), "melt f8 frame-split launch");
    }
    if ((kF8fsFrames + a.J - 1) * a.H <= 17 * 1024) {
        allow_lds(k_melt_f8_fs<NG, RT, 17, false>, RT * 32 * 4);
        k_melt_f8_fs<NG, RT, 17, false><<<grid, 512, lds, s>>>(a, (const i32x8 *)p.d_pack_f8, p.d_rowscale, p.N, 0);
    } else {
        allow_lds(k_melt_f8_fs<NG, RT, 22, false>, RT * 32 * 4);
        k_melt_f8_fs<NG, RT, 22, false><<<grid, 512, lds, s>>>(a, (const i32x8 *)p.d_pack_f8, p.d_rowscale, p.N, 0);
    }
    return hip_check(hipGetLastError(), "melt f8 frame-split launch");
}

template <int NG>
static melt_status launch_f8fs(const Plan &p, const FwdArgs &a, size_t lds, int grid, hipStream_t s) {
    switch (p.row_tiles) {
    case 1: return launch_f8fs_rt<NG, 1>(p, a, lds, grid, s);
    case 2: return launch_f8fs_rt<NG, 2>(p, a, lds, grid, s);
    case 3: return launch_f8fs_rt<NG, 3>(p, a, lds, grid, s);
    case 4: return launch_f8fs_rt<NG, 4>(p, a, lds, grid, s);
    case 5: return launch_f8fs_rt<NG, 5>(p, a, lds, grid, s);
    case 6: return launch_f8fs_rt<NG, 6>(p, a, lds, grid, s);
    default: return launch_f8fs_rt<NG, 8>(p, a, lds, grid, s);
    }
}

melt_status launch_melt_f8_fs(Plan &p, const FwdTask &t) {
    if (!f8fs_fits(p)) return set_error(MELT_E_UNSUPPORTED, "frame-split FP8 kernel: unsupported geometry");
    const Geometry &g = p.geo32;
    FwdArgs a = make_args(p, g, lds_stride(g.Hp, 4), t);
    size_t lds = f8fs_rows_bytes(p);
    if (t.clips.off) {
        a.list_off = (int)lds;
        lds += kListBytes;
    }
    const int grid = persistent_grid(p, t.est_chunks, 1);
    switch ((p.N + 63) / 64) {
    case 4: return launch_f8fs<4>(p, a, lds, grid, t.stream);
    case 7: return launch_f8fs<7>(p, a, lds, grid, t.stream);
    default: return launch_f8fs<8>(p, a, lds, grid, t.stream);
    }
}

}  // namespace melt
