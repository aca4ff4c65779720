// MelT forward on split operands: every FP32 value is the sum of P 16-bit planes and the
// projection runs as the plane products that matter, on the 16-bit matrix cores with FP32
// accumulation (Eq. dmp_projection, Eq. dmp_matrix_energy, Eq. meltf).
//
//   Split3BF16 (FP32)  three bfloat16 planes of 2^24 x hold all 24 significand bits of an FP32
//                      value (each residual is exact): bfloat16 has FP32's exponent range, and the
//                      factor, undone on the accumulators, keeps the third plane of the smallest
//                      values, subnormal ones too, out of bfloat16's own subnormals.  Values of
//                      2^103 and more become infinities (split_again).  Of the nine products the
//                      six down to 2^-16 relative are kept, so a term is off by about 2^-26,
//                      below the FP32 rounding of the basis itself
//   Split2BF16, Split2F16 (BF16X3, FP16X3)  hi and lo planes, three products
//
// What bounds it: the matrix cores (P = 3: six products, 147 GFLOP on 64 x 30 s at N = 400,
// M = 80), then the L1 path the basis fragments stream through.  The layout follows from
// that: a multiply wave owns FT tiles of 16 frames x RT tiles of 16 basis rows, so a basis
// fragment of P KB read through L1 feeds FT NP MFMAs (4 x 6 x 16 cycles against 48 of the
// shared L1 port) and a frame fragment read from LDS feeds RT NP.  16x16x32 tiles rather than
// 32x32x16: 80 Mel bins are ten of them, five for each of the two row halves, where 32-row
// tiles split 3 + 2.
//
// One workgroup per CU, 8 waves: 4 multiply (WF frame groups x 4 / WF row groups, one per
// SIMD) and 4 stage.  The stagers load the next item's samples and split them in registers
// while the multiply waves run; between the two barriers of an item they write the planes to
// LDS while the multiply waves empty their accumulators.
//
// Measured (whole calls, side by side): FP32 64 x 30 s, N 400, M 80: 213.5 us on FP32 MFMA, 123.4 us
// here (200 TFLOP/s of the method, 1.2 PFLOP/s of products); FP32 ragged 512 clips, N 512,
// M 128: 2.11 ms -> 1.00 ms (1.49 PFLOP/s of products); FP16X3 ragged, N 1024, M 128: 4.0 ms on
// the frame-split kernel with 128-frame chunks -> 0.84-0.92 ms.  Relative error of the log-Mel
// rows against 64 bits on the same calls: 4.5e-7 -> 3.5e-7, 5.6e-7 -> 4.1e-7, 7.2e-7 -> 5.4e-7.
#pragma once
#include <type_traits>
#include "fwd_common.h"

namespace melt {

typedef unsigned split_u32x4 __attribute__((ext_vector_type(4)));

// Four FP32 values -> P planes of four 16-bit values (two dwords each).  (kPlaneScale: fwd_common.h)
struct Split3BF16 {
    static constexpr int P = 3, NP = 6;
    // plane products (basis plane, frame plane), frame plane 2 first: the k-loop refills the
    // frame fragments plane by plane behind their last use, in this order
    static constexpr int pa[6] = {0, 1, 0, 2, 1, 0}, pb[6] = {2, 1, 1, 0, 0, 0};
    static constexpr int last_of_plane[3] = {5, 2, 0};      // index of the last product of frame plane p
    __device__ static void split(f32x4 v, unsigned (&w)[6]) {
#pragma unroll
        for (int h = 0; h < 2; ++h) {
            const float x = v[2 * h] * kPlaneScale, y = v[2 * h + 1] * kPlaneScale;
            const unsigned b0 = pk_bf16(x, y);
            const float x1 = x - __builtin_bit_cast(float, b0 << 16), y1 = y - __builtin_bit_cast(float, b0 & 0xffff0000u);
            const unsigned b1 = pk_bf16(x1, y1);
            const float x2 = x1 - __builtin_bit_cast(float, b1 << 16), y2 = y1 - __builtin_bit_cast(float, b1 & 0xffff0000u);
            w[h] = b0;
            w[2 + h] = b1;
            w[4 + h] = pk_bf16(x2, y2);
        }
    }
    __device__ static f32x4 mma(split_u32x4 a, split_u32x4 b, f32x4 c) {
        return __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8, a), __builtin_bit_cast(bf16x8, b), c, 0, 0, 0);
    }
};
struct Split2BF16 {
    static constexpr int P = 2, NP = 3;
    static constexpr int pa[3] = {0, 1, 0}, pb[3] = {1, 0, 0};
    static constexpr int last_of_plane[2] = {2, 0};
    __device__ static void split(f32x4 v, unsigned (&w)[4]) {
#pragma unroll
        for (int h = 0; h < 2; ++h) {
            const float x = v[2 * h], y = v[2 * h + 1];
            const unsigned b0 = pk_bf16(x, y);
            w[h] = b0;
            w[2 + h] = pk_bf16(x - __builtin_bit_cast(float, b0 << 16), y - __builtin_bit_cast(float, b0 & 0xffff0000u));
        }
    }
    __device__ static f32x4 mma(split_u32x4 a, split_u32x4 b, f32x4 c) { return Split3BF16::mma(a, b, c); }
};
struct Split2F16 {
    static constexpr int P = 2, NP = 3;
    static constexpr int pa[3] = {0, 1, 0}, pb[3] = {1, 0, 0};
    static constexpr int last_of_plane[2] = {2, 0};
    __device__ static void split(f32x4 v, unsigned (&w)[4]) {
#pragma unroll
        for (int h = 0; h < 2; ++h) {
            const float x = v[2 * h] * kF16x3Scale, y = v[2 * h + 1] * kF16x3Scale;
            const unsigned b0 = pk_f16(x, y);
            const cv_f32x2 r = __builtin_convertvector(__builtin_bit_cast(cv_f16x2, b0), cv_f32x2);
            w[h] = b0;
            w[2 + h] = pk_f16(x - r[0], y - r[1]);
        }
    }
    __device__ static f32x4 mma(split_u32x4 a, split_u32x4 b, f32x4 c) {
        return __builtin_amdgcn_mfma_f32_16x16x32_f16(__builtin_bit_cast(f16x8, a), __builtin_bit_cast(f16x8, b), c, 0, 0, 0);
    }
};

// Geometry of one launch, beside FwdArgs (whose S is the LDS row stride in 16-bit elements:
// the P planes of a hop-block row side by side, then 16 bytes so that the stride is an odd
// multiple of 16 bytes and the 16-byte reads of 16 consecutive rows hit distinct banks).
struct SplitGeo {
    int NG, GH;            // k-groups of 32: in all, and per full hop segment
    int T16;               // tiles of 16 basis rows (8 Mel bins)
    int nsub, parts;       // items per chunk: frame parts x row parts
    const float *basis;    // the FP32 basis [2M][N]
    int N;
    int half_tail;         // the last k-group holds at most 16 columns of the frame
};

// First Mel bin of lane quarter q of 16-row tile t.  The accumulator of a 16x16 tile holds in
// quarter q rows 4q .. 4q + 3, (cos, sin) of two bins.  Two neighbouring tiles share 16 bins,
// four consecutive ones per quarter (two from each tile), so that a quarter stores 16 bytes;
// the last tile of an odd count has its 8 bins to itself.
__host__ __device__ __forceinline__ int split_tile_mel(int t, int q, int T16) {
    return (T16 & 1) && t == T16 - 1 ? 8 * t + 2 * q : 16 * (t >> 1) + 4 * q + 2 * (t & 1);
}

// The stagers' share of one item: PV vectors of four columns per thread of 256, vector u of a
// hop-block row-major walk (row u / VR, columns 4 (u % VR) ..), split into planes in registers.
// Columns at or past the hop, and samples outside [start + lo, end), are zero.
template <class Op, int PV>
__device__ __forceinline__ void split_load(const FwdArgs &a, int64_t start, int lo, int64_t end, int nrows, int lt,
                                           float inv_vr, unsigned (&w)[PV][2 * Op::P]) {
    // Every load is unconditional, so that all of a batch are in flight together.  Where the whole
    // span (and the 3 samples a row's last vector may reach past it) lies in the clip: 16-byte
    // loads, columns past the hop cleared afterwards.  At a clip's end: 4-byte loads, with an
    // offset past the descriptor, which reads as zero, for columns and samples that do not exist.
    const int span = nrows * a.H, VR = a.Hp >> 2;
    const int64_t left = end - start - lo;
    const bool padded = a.Hp != a.H;
    const bool inside = nrows > 0 && lo == 0 && left >= span + (padded ? 3 : 0);
    const int64_t some = left < span - lo ? left : span - lo;
    const int records = (int)(inside ? span + (padded ? 3 : 0) : some > 0 ? some : 0);
    const __amdgpu_buffer_rsrc_t rs =
        __builtin_amdgcn_make_buffer_rsrc((void *)(a.wave + (start + lo)), (short)0, records * 4, 0x00020000);
    asm volatile("" : "+v"(lt));        // addresses formed here, not kept from item to item
    // at most 14 vectors in flight, so that the raw and the split values of all PV fit the registers
    constexpr int NB = PV > 14 ? 2 : 1, PB = (PV + NB - 1) / NB;
#pragma unroll
    for (int b = 0; b < NB; ++b) {
        f32x4 raw[PB];
        auto at = [&](int v, int &r) {       // column of vector b PB + v; r: its row
            const int u = lt + (b * PB + v) * 256;
            r = (int)(((float)u + 0.5f) * inv_vr);
            const int cv = u - r * VR;
            r += (cv >= VR) - (cv < 0);
            return 4 * (u - r * VR);
        };
        if (inside) {
#pragma unroll
            for (int v = 0; v < PB; ++v) {
                int r;
                const int col = at(v, r);
                const int o = r < nrows && col < a.H ? r * a.H + col : 0;
                raw[v] = __builtin_bit_cast(f32x4, __builtin_amdgcn_raw_buffer_load_b128(rs, o * 4, 0, 0));
            }
            if (padded) {
#pragma unroll
                for (int v = 0; v < PB; ++v) {
                    int r;
                    const int col = at(v, r);
#pragma unroll
                    for (int e = 0; e < 4; ++e) raw[v][e] = col + e < a.H ? raw[v][e] : 0.0f;
                }
            }
        } else {
#pragma unroll
            for (int v = 0; v < PB; ++v) {
                int r;
                const int col = at(v, r);
#pragma unroll
                for (int e = 0; e < 4; ++e) {
                    const int o = r * a.H + col + e - lo;
                    const int off = r < nrows && col + e < a.H && o >= 0 && o < records ? o * 4 : 0x7ffffff0;
                    raw[v][e] = __builtin_bit_cast(float, __builtin_amdgcn_raw_buffer_load_b32(rs, off, 0, 0));
                }
            }
        }
#pragma unroll
        for (int v = 0; v < PB; ++v)
            if (b * PB + v < PV) Op::split(raw[v], w[b * PB + v < PV ? b * PB + v : 0]);
        __builtin_amdgcn_sched_barrier(0);
    }
}

template <class Op, int PV>
__device__ __forceinline__ void split_write(const FwdArgs &a, int nrows, int lt, float inv_vr,
                                            const unsigned (&w)[PV][2 * Op::P], unsigned short *rows) {
    const int VR = a.Hp >> 2;
    // addresses formed here, not carried across the multiply phase
    asm volatile("" : "+v"(lt));
#pragma unroll
    for (int v = 0; v < PV; ++v) {
        const int u = lt + v * 256;
        int r = (int)(((float)u + 0.5f) * inv_vr);
        int cv = u - r * VR;
        r += (cv >= VR) - (cv < 0);
        if (r < nrows) {
            unsigned short *d = rows + r * a.S + 4 * (u - r * VR);
#pragma unroll
            for (int p = 0; p < Op::P; ++p) *(uint2 *)(d + p * a.Hp) = uint2{w[v][2 * p], w[v][2 * p + 1]};
        }
    }
}

// One item of a workgroup: frames [f0, f0 + nf) of a chunk.  Its hop-block rows start at sample
// `start`; samples before start + lo and from `end` on are zero.
struct SplitItem {
    int64_t start, end, out_row;
    int nf, lo;
};
// four floats at any 4-byte address
typedef float f32x4_any __attribute__((ext_vector_type(4), aligned(4)));

// FS frame tiles (from the item's frame f0 on) of a wave's RT row tiles in plain FP32, on the FP32
// matrix cores.  Sixteen columns a step, four of them consecutive per lane, of one segment after the
// other; frames and rows that do not exist repeat others.
template <class Job, int FS, int RT>
__device__ __forceinline__ void split_plain(const Job &job, const SplitItem &it, int f0, int lane, const int (&tile)[RT],
                                            f32x4 (&acc)[FS][RT]) {
    const int cols = job.plain_columns();
#pragma unroll
    for (int f = 0; f < FS; ++f)
#pragma unroll
        for (int r = 0; r < RT; ++r) acc[f][r] = f32x4{};
#pragma unroll 1
    for (int s = 0; s < job.plain_segments(); ++s) {
#pragma unroll 1
        for (int c0 = 0; c0 < cols; c0 += 16) {
            int l = lane;
            asm volatile("" : "+v"(l));                 // addresses and conditions formed here, not kept
            const int c = c0 + 4 * (l >> 4);
            f32x4 x[FS], w[RT];
#pragma unroll
            for (int f = 0; f < FS; ++f) x[f] = job.plain_samples(it, min(f0 + 16 * f + (l & 15), it.nf - 1), s, c);
#pragma unroll
            for (int r = 0; r < RT; ++r) w[r] = job.plain_weights(tile[r], l & 15, s, c);
#pragma unroll
            for (int r = 0; r < RT; ++r)
#pragma unroll
                for (int e = 0; e < 4; ++e)
#pragma unroll
                    for (int f = 0; f < FS; ++f)
                        acc[f][r] = __builtin_amdgcn_mfma_f32_16x16x4f32(w[r][e], x[f][e], acc[f][r], 0, 0, 0);
        }
        if (s == 0) {
#pragma unroll
            for (int f = 0; f < FS; ++f)
#pragma unroll
                for (int r = 0; r < RT; ++r) job.plain_first_segment(tile[r], lane >> 4, acc[f][r]);
        }
    }
}

// The kernel's first argument, read again: what a rare path alone uses of it takes no scalar registers
// on the way there.
template <class Job>
__device__ __forceinline__ Job split_job_again() {
    struct Words {
        unsigned w[sizeof(Job) / 4];
    } words;
    auto p = (const __attribute__((address_space(4))) unsigned *)__builtin_amdgcn_kernarg_segment_ptr();
    asm volatile("" : "+s"(p));
#pragma unroll
    for (unsigned i = 0; i < sizeof(Job) / 4; ++i) words.w[i] = p[i];
    return __builtin_bit_cast(Job, words);
}

// The factor that undoes the scaling of the operands, hidden from the compiler, which would move its
// multiplications up into the last block of the k-loop, for every k-group.
__device__ __forceinline__ float split_unscale(float v) {
    asm volatile("" : "+s"(v));
    return v;
}
// Chunk-table entries through the scalar cache: a vector load's wait would also drain the wave's
// output stores.
__device__ __forceinline__ int64_t split_scalar(const void *base, int64_t i) {
    typedef const __attribute__((address_space(4))) int64_t *cptr;
    return ((cptr)base)[i];
}

// What an item reads and what becomes of its accumulators.
struct SplitForward {
    FwdArgs a;
    SplitGeo g;
    // Whether the kernel finds its own chunks: then list[k] is the chunk of the workgroup's item k.
    __device__ __forceinline__ bool lists() const { return a.clips.off != nullptr; }
    __device__ __forceinline__ int start(Chunk *list) const {
        const int w = blockIdx.x + (threadIdx.x & 63) * gridDim.x;
        return list_start(a, list, w / (g.nsub * g.parts));
    }
    __device__ __forceinline__ SplitItem item(int w, int k, const Chunk *list, int SF) const {
        const int ci = w / (g.nsub * g.parts);
        const int f0 = ((w - ci * g.nsub * g.parts) / g.parts) * SF;
        static_assert(sizeof(Chunk) == 32, "four int64 per entry");
        if (lists()) {
            const Chunk e = list[k];
            const int nf = min(SF, __builtin_amdgcn_readfirstlane(e.n_frames) - f0);
            return {uniform64(e.sample_start) + (int64_t)f0 * a.H, uniform64(e.sample_end), uniform64(e.out_row) + f0,
                    nf > 0 ? nf : 0, 0};
        }
        const int64_t st = split_scalar(a.chunks, 4 * (int64_t)ci), en = split_scalar(a.chunks, 4 * (int64_t)ci + 1);
        const int64_t row = split_scalar(a.chunks, 4 * (int64_t)ci + 2);
        const int nf = min(SF, (int)split_scalar(a.chunks, 4 * (int64_t)ci + 3) - f0);      // low half: n_frames
        return {st + (int64_t)f0 * a.H, en, row + f0, nf > 0 ? nf : 0, 0};
    }
    // (whether an output is not finite, where Op has three planes)
    template <class Op, int FT, int RT>
    __device__ __forceinline__ bool store(const SplitItem &it, int fbase, int lane, const int (&tile)[RT], f32x4 (&acc)[FT][RT]) const;
    template <int FS, int RT>
    __device__ __forceinline__ void again(const SplitItem &it, int f0, int lane, const int (&tile)[RT]) const;
    // split_plain: one segment, the frame
    __device__ __forceinline__ int plain_segments() const { return 1; }
    __device__ __forceinline__ int plain_columns() const { return g.N; }
    __device__ __forceinline__ f32x4 columns4(const float *p, int c) const {
        if (c + 4 <= g.N) return *(const f32x4_any *)(p + c);
        f32x4 v{};
#pragma unroll
        for (int e = 0; e < 3; ++e)
            if (c + e < g.N) v[e] = p[c + e];
        return v;
    }
    __device__ __forceinline__ f32x4 plain_samples(const SplitItem &it, int frame, int, int c) const {
        return columns4(a.wave + it.start + (int64_t)frame * a.H, c);
    }
    __device__ __forceinline__ f32x4 plain_weights(int t, int row, int, int c) const {
        const int mel = min(split_tile_mel(min(t, g.T16 - 1), row >> 2, g.T16) + (row >> 1 & 1), a.M - 1);
        return columns4(g.basis + (size_t)((row & 1) * a.M + mel) * g.N, c);
    }
    __device__ __forceinline__ void plain_first_segment(int, int, f32x4 &) const {}
};

// Output values of the two bins of each tile of one frame.
template <int KIND, int RT>
__device__ __forceinline__ void split_map(float eps, const f32x4 (&acc)[RT], float (&v)[2 * RT]) {
#pragma unroll
    for (int r = 0; r < RT; ++r) {
        const f32x4 y = acc[r];
        v[2 * r] = out_map_k<KIND>(y[0] * y[0] + y[1] * y[1], eps);
        v[2 * r + 1] = out_map_k<KIND>(y[2] * y[2] + y[3] * y[3], eps);
    }
}

// Accumulators -> output rows.  tile[]: pairs (r, r + 1) start at even tiles.
template <class Op, int FT, int RT>
__device__ __forceinline__ bool SplitForward::store(const SplitItem &it, int fbase, int lane, const int (&tile)[RT],
                                                    f32x4 (&acc)[FT][RT]) const {
    asm volatile("" : "+v"(lane));      // addresses formed per item, not kept across the multiply phase
    const int q = lane >> 4, f0 = fbase + (lane & 15);
    if constexpr (!std::is_same<Op, Split2BF16>::value) {
        const float unscale = split_unscale(Op::P == 3 ? kPlaneUnscale : 1.0f / kF16x3Scale);     // exact
#pragma unroll
        for (int f = 0; f < FT; ++f)
#pragma unroll
            for (int r = 0; r < RT; ++r) acc[f][r] *= unscale;
    }
    if (a.proj) {
#pragma unroll
        for (int r = 0; r < RT; ++r) {
            const int m0 = split_tile_mel(tile[r], q, g.T16);
#pragma unroll
            for (int f = 0; f < FT; ++f) {
                const int64_t row = it.out_row + f0 + 16 * f;
                if (f0 + 16 * f >= it.nf || row >= a.n_frames || tile[r] >= g.T16) continue;
                float *p = a.proj + row * (2 * a.M) + 2 * m0;
                if (m0 + 1 < a.M) {
                    *(float2 *)p = float2{acc[f][r][0], acc[f][r][1]};
                    *(float2 *)(p + 2) = float2{acc[f][r][2], acc[f][r][3]};
                } else if (m0 < a.M) {
                    *(float2 *)p = float2{acc[f][r][0], acc[f][r][1]};
                }
            }
        }
    }
    float probe = 0.0f;                 // stays 0 while every output is finite
    // every bin of the wave's tiles exists and rows are whole 16-byte vectors: no edge tests
    const bool whole = (a.M & 7) == 0 && max(tile[0], tile[RT - 1]) < g.T16 && tile[RT > 1 ? RT - 2 : 0] < g.T16;
#pragma unroll
    for (int f = 0; f < FT; ++f) {
        const int64_t row = it.out_row + f0 + 16 * f;
        if (f0 + 16 * f >= it.nf || row >= a.n_frames) continue;
        float *o = a.out + row * a.M;
        float v[2 * RT];
        switch (a.out_kind) {
        case MELT_OUT_LOG_POWER: split_map<MELT_OUT_LOG_POWER, RT>(a.eps, acc[f], v); break;
        case MELT_OUT_LOG_MAGNITUDE: split_map<MELT_OUT_LOG_MAGNITUDE, RT>(a.eps, acc[f], v); break;
        case MELT_OUT_POWER: split_map<MELT_OUT_POWER, RT>(a.eps, acc[f], v); break;
        default: split_map<MELT_OUT_MAGNITUDE, RT>(a.eps, acc[f], v); break;
        }
#pragma unroll
        for (int r = 0; r < RT; r += 2) {
            const bool pair = r + 1 < RT;                       // known when unrolled
            const int r1 = pair ? r + 1 : r;
            const int m0 = split_tile_mel(tile[r], q, g.T16);
            const float v0 = v[2 * r], v1 = v[2 * r + 1], v2 = v[2 * r1], v3 = v[2 * r1 + 1];
            if constexpr (Op::P == 3) probe = fmaf(v0 + v1 + v2 + v3, 0.0f, probe);
            if (whole) {
                if (pair) *(f32x4 *)(o + m0) = f32x4{v0, v1, v2, v3};
                else *(float2 *)(o + m0) = float2{v0, v1};
            } else if (tile[r] < g.T16) {
                if (m0 < a.M) o[m0] = v0;
                if (m0 + 1 < a.M) o[m0 + 1] = v1;
                if (pair && tile[r1] < g.T16) {
                    if (m0 + 2 < a.M) o[m0 + 2] = v2;
                    if (m0 + 3 < a.M) o[m0 + 3] = v3;
                }
            }
        }
    }
    return Op::P == 3 && __any(!(probe == 0.0f));
}

// The outputs and projections of FS frame tiles that are not finite, once more in plain FP32.
template <int FS, int RT>
__device__ __forceinline__ void SplitForward::again(const SplitItem &it, int f0, int lane, const int (&tile)[RT]) const {
    const int q = lane >> 4;
    unsigned bad[FS], any = 0;                          // of a row tile's two bins: output, projection
#pragma unroll
    for (int f = 0; f < FS; ++f) {
        const int fl = f0 + 16 * f + (lane & 15);
        const int64_t row = it.out_row + fl;
        bad[f] = 0;
        if (fl < it.nf && row < a.n_frames) {
#pragma unroll
            for (int r = 0; r < RT; ++r)
#pragma unroll
                for (int k = 0; k < 2; ++k) {
                    const int mel = split_tile_mel(tile[r], q, g.T16) + k;
                    if (tile[r] >= g.T16 || mel >= a.M) continue;
                    if (!(a.out[row * a.M + mel] * 0.0f == 0.0f)) bad[f] |= 1u << (4 * r + 2 * k);
                    if (!a.proj) continue;
                    const float2 p = *(const float2 *)(a.proj + row * (2 * a.M) + 2 * mel);
                    if (!(fmaf(p.x, 0.0f, p.y * 0.0f) == 0.0f)) bad[f] |= 2u << (4 * r + 2 * k);
                }
        }
        any |= bad[f];
    }
    if (!__any(any != 0)) return;
    f32x4 acc[FS][RT];
    split_plain(*this, it, f0, lane, tile, acc);
#pragma unroll
    for (int f = 0; f < FS; ++f) {
        const int64_t row = it.out_row + f0 + 16 * f + (lane & 15);
#pragma unroll
        for (int r = 0; r < RT; ++r)
#pragma unroll
            for (int k = 0; k < 2; ++k) {
                const int mel = split_tile_mel(tile[r], q, g.T16) + k;
                const float R = acc[f][r][2 * k], I = acc[f][r][2 * k + 1], S = R * R + I * I;
                if (bad[f] >> (4 * r + 2 * k) & 1)
                    a.out[row * a.M + mel] = a.out_kind == MELT_OUT_LOG_POWER       ? out_map_k<MELT_OUT_LOG_POWER>(S, a.eps)
                                             : a.out_kind == MELT_OUT_LOG_MAGNITUDE ? out_map_k<MELT_OUT_LOG_MAGNITUDE>(S, a.eps)
                                             : a.out_kind == MELT_OUT_POWER         ? S
                                                                                    : sqrtf(S);
                if (bad[f] >> (4 * r + 2 * k) & 2) *(float2 *)(a.proj + row * (2 * a.M) + 2 * mel) = float2{R, I};
            }
    }
}

// The row tiles of a multiply wave (the row part is the workgroup's).
template <int RT, int WF>
__device__ __forceinline__ void split_wave_tiles(int wid, int parts, int (&tile)[RT]) {
    const int t0 = ((int)(blockIdx.x % parts) * (4 / WF) + wid / WF) * RT;
#pragma unroll
    for (int r = 0; r < RT; ++r) {
        // an odd tile count that starts at an odd tile keeps its unpaired tile for last
        tile[r] = (RT & 1) && (t0 & 1) ? (r == RT - 1 ? t0 : t0 + 1 + r) : t0 + r;
    }
}

// A wave's items k0 .. k1 once more, where an output is not finite.  The planes of an infinity (or of a
// value that becomes one, 2^24 times it in bfloat16) are inf and -inf or NaN, so what comes out is not
// what FP32 arithmetic gives.  After the wave's last item rather than where it is found: there it cost
// every call 1 to 2 % (scalar registers).  64 x 30 s, N 400, M 80: 0.130 ms, 0.161 with one NaN sample,
// 0.525 with nothing else (0.63 and 17.2 where one lane took an output's terms one by one).
template <class Job, int FT, int RT, int WF>
__device__ __forceinline__ void split_again(int k0, int k1, int wid, const unsigned short *rows) {
    const Job job = split_job_again<Job>();
    const Chunk *list = reinterpret_cast<const Chunk *>(reinterpret_cast<const char *>(rows) + job.a.list_off);
    const int lane = threadIdx.x & 63, fbase = wid % WF * FT * 16;
    int tile[RT];
    split_wave_tiles<RT, WF>(wid, job.g.parts, tile);
    for (int k = k0; k <= k1; ++k) {
        const SplitItem it = job.item(blockIdx.x + k * gridDim.x, k, list, WF * FT * 16);
        constexpr int FS = FT > 1 && RT < 8 ? 2 : 1;       // (two of eight row tiles would spill)
#pragma unroll 1
        for (int f = fbase; f < fbase + 16 * FT && f < it.nf; f += 16 * FS) job.template again<FS, RT>(it, f, lane, tile);
    }
}

// Depth of the basis ring in tiles: the fragments of the tile D steps ahead are loaded as soon
// as a tile's MFMAs have read theirs.  RT for 3 to 6 tiles (one k-group ahead: 384 cycles per
// tile and more cover an L2 access), half of 6 and 8 (registers), and several k-groups for the
// short steps of one or two tiles.
constexpr int split_ring(int FT, int RT) { return RT >= 8 ? 4 : RT == 6 ? 3 : RT >= 3 ? RT : FT >= 4 ? 4 : 8; }

template <class Job, class Op, int FT, int RT, int WF, int PV>
__global__ __attribute__((amdgpu_flat_work_group_size(512, 512), amdgpu_waves_per_eu(2, 2)))
void k_melt_split(Job job, const split_u32x4 *__restrict__ bpack) {
    const FwdArgs &a = job.a;
    const SplitGeo &g = job.g;
    extern __shared__ __attribute__((aligned(16))) unsigned short rows[];
    constexpr int P = Op::P, NP = Op::NP, SF = WF * FT * 16;
    const int lane = threadIdx.x & 63;
    const int wid = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    Chunk *list = reinterpret_cast<Chunk *>(reinterpret_cast<char *>(rows) + a.list_off);
    const int nitems = (job.lists() ? job.start(list) : *a.n_chunks) * g.nsub * g.parts;
    const int G = gridDim.x;                       // a multiple of parts: the row part is the workgroup's
    int w = blockIdx.x, k = 0;                     // item, and how many the workgroup had before it
    if (wid >= 4) {
        const int lt = (int)threadIdx.x - 256;
        const float inv_vr = 4.0f / (float)a.Hp;
        unsigned pl[PV][2 * P];
        SplitItem it{};
        if (w < nitems) {
            it = job.item(w, 0, list, SF);
            split_load<Op, PV>(a, it.start, it.lo, it.end, it.nf ? it.nf + a.J - 1 : 0, lt, inv_vr, pl);
            split_write<Op, PV>(a, it.nf ? it.nf + a.J - 1 : 0, lt, inv_vr, pl, rows);
        }
        __syncthreads();                           // rows of the first item ready
        for (; w < nitems; w += G, ++k) {
            const bool more = w + G < nitems;
            if (more) {
                it = job.item(w + G, k + 1, list, SF);
                split_load<Op, PV>(a, it.start, it.lo, it.end, it.nf ? it.nf + a.J - 1 : 0, lt, inv_vr, pl);
            }
            // split before the barrier, not between the two
#pragma unroll
            for (int v = 0; v < PV; ++v)
#pragma unroll
                for (int e = 0; e < 2 * P; ++e) asm volatile("" : "+v"(pl[v][e]));
            __syncthreads();                       // A: the multiply waves are done with the rows
            if (more) split_write<Op, PV>(a, it.nf ? it.nf + a.J - 1 : 0, lt, inv_vr, pl, rows);
            __syncthreads();                       // B: rows of the next item ready
        }
        return;
    }
    const int wf = wid % WF;
    constexpr int D = split_ring(FT, RT), U = D > RT ? D / RT : 1;
    static_assert((U * RT) % D == 0, "the ring's slots repeat every U k-groups");
    int tile[RT];
    split_wave_tiles<RT, WF>(wid, g.parts, tile);
    const __amdgpu_buffer_rsrc_t brs = __builtin_amdgcn_make_buffer_rsrc(
        (void *)bpack, (short)0, g.T16 * g.NG * P * 1024, 0x00020000);
    const int voff = lane * 16;
    int toff[RT];
#pragma unroll
    for (int r = 0; r < RT; ++r) toff[r] = min(tile[r], g.T16 - 1) * g.NG * (P * 1024);
    split_u32x4 A[D][P], B[FT][P];
    auto load_a = [&](int slot, int r, int grp) {
#pragma unroll
        for (int p = 0; p < P; ++p)
            A[slot][p] = __builtin_bit_cast(
                split_u32x4, __builtin_amdgcn_raw_buffer_load_b128(brs, voff + p * 1024, toff[r] + grp * (P * 1024), 0));
    };
#pragma unroll
    for (int s = 0; s < D; ++s) load_a(s, s % RT, min(s / RT, g.NG - 1));
    __syncthreads();                               // rows of the first item ready
    const int fbase = wf * FT * 16;
    const int la0 = (fbase + (lane & 15)) * a.S + 8 * (lane >> 4);
    int again0 = 0, again1 = -1;                   // items with an output that is not finite lie between
    for (; w < nitems; w += G, ++k) {
        const SplitItem it = job.item(w, k, list, SF);
        // two planes: a k-group's three products are summed on their own and added once, behind the
        // next tile's first MFMAs (a third of the roundings at the running sum's magnitude)
        f32x4 acc[FT][RT], sum[2][FT];
#pragma unroll
        for (int f = 0; f < FT; ++f)
#pragma unroll
            for (int r = 0; r < RT; ++r) acc[f][r] = f32x4{};
        auto load_b = [&](int p, int at) {
#pragma unroll
            for (int f = 0; f < FT; ++f) B[f][p] = *(const split_u32x4 *)(rows + at + f * 16 * a.S + p * a.Hp);
        };
        if (fbase < it.nf) {
#pragma unroll
            for (int p = P - 1; p >= 0; --p) load_b(p, la0);
            int col = 0, at = la0;                 // k-group within its segment, its LDS offset
            for (int g0 = 0; g0 < g.NG; g0 += U) {
#pragma unroll
                for (int u = 0; u < U; ++u) {
                    const int grp = g0 + u;
                    if (grp >= g.NG) break;
                    // offset of the next k-group's columns (past the last: any valid ones)
                    int nat = at + 32;
                    if (++col == g.GH) {
                        col = 0;
                        nat = at + a.S - (g.GH - 1) * 32;
                    }
                    if (grp + 1 >= g.NG) nat = la0;
                    at = nat;
                    if (P == 2 && g.half_tail && grp + 1 == g.NG && lane >= 32) {
                        // columns 16 .. 31 are samples after the frame (their weights are zero):
                        // one that overflows binary16 must not reach it
#pragma unroll
                        for (int f = 0; f < FT; ++f)
#pragma unroll
                            for (int p = 0; p < P; ++p) B[f][p] = split_u32x4{};
                    }
#pragma unroll
                    for (int r = 0; r < RT; ++r) {
                        const int slot = (u * RT + r) % D;
#pragma unroll
                        for (int m = 0; m < NP; ++m) {
#pragma unroll
                            for (int f = 0; f < FT; ++f) {
                                if constexpr (P == 3)
                                    acc[f][r] = Op::mma(A[slot][Op::pa[m]], B[f][Op::pb[m]], acc[f][r]);
                                else
                                    sum[r & 1][f] = Op::mma(A[slot][Op::pa[m]], B[f][Op::pb[m]], m ? sum[r & 1][f] : f32x4{});
                            }
                            if (P == 2 && m == 0 && r > 0) {
#pragma unroll
                                for (int f = 0; f < FT; ++f) acc[f][r - 1] += sum[(r - 1) & 1][f];
                            }
                            if (r == RT - 1) {
#pragma unroll
                                for (int p = 0; p < P; ++p)
                                    if (Op::last_of_plane[p] == m) {
                                        __builtin_amdgcn_sched_barrier(0);
                                        load_b(p, nat);
                                        __builtin_amdgcn_sched_barrier(0);
                                    }
                            }
                        }
                        // the slot's next tile: D steps on, wrapping to the next item's first
                        const int ahead = r + D, dg = ahead / RT, rr = ahead - dg * RT;
                        int ng = grp + dg;
                        if (ng >= g.NG) ng -= g.NG;
                        if (ng >= g.NG) ng = 0;
                        __builtin_amdgcn_sched_barrier(0);
                        load_a(slot, rr, ng);
                        __builtin_amdgcn_sched_barrier(0);
                    }
                    if constexpr (P == 2) {
#pragma unroll
                        for (int f = 0; f < FT; ++f) acc[f][RT - 1] += sum[(RT - 1) & 1][f];
                    }
                }
            }
            // the ring holds the tiles of steps NG RT .. NG RT + D - 1; where NG is no multiple of U
            // they sit in rotated slots: refill from the first step
            if (U > 1 && g.NG % U != 0) {
#pragma unroll
                for (int s = 0; s < D; ++s) load_a(s, s % RT, min(s / RT, g.NG - 1));
            }
        }
        __syncthreads();                           // A: every row read; the stagers may overwrite
        if (fbase < it.nf && job.template store<Op, FT, RT>(it, fbase, lane, tile, acc)) {
            if (again1 < 0) again0 = k;
            again1 = k;
        }
        __syncthreads();                           // B: rows of the next item ready
    }
    if constexpr (P == 3)
        if (again1 >= 0) split_again<Job, FT, RT, WF>(again0, again1, wid, rows);
}

// ------------------------------------------------------------------ launch

// A compiled shape: WF waves along the frames, FT frame tiles and RT row tiles per wave, PV
// staging vectors per thread; `parts` row parts of 4 / WF RT tiles each (0: nothing fits).
struct SplitShape {
    int wf, ft, rt, pv, parts;
};
inline int split_sf(const SplitShape &h) { return h.wf * h.ft * 16; }
inline size_t split_lds(int P, const Geometry &g, const SplitShape &h) {
    return (size_t)(split_sf(h) + g.J - 1) * (P * g.Hp + 8) * 2;
}
// The shape for n_frames frames in est_chunks chunks of kSplitChunk (melt_fwd.hip).
SplitShape split_shape(const Geometry &g, int P, int T16, int cu_count, int64_t est_chunks, int64_t n_frames);

// workgroups: a multiple of the row parts
inline int split_grid(const Plan &p, const SplitShape &h, int64_t items) {
    return std::max(persistent_grid(p, items, 1) / h.parts, 1) * h.parts;
}

template <class Job, class Op, int FT, int RT, int WF, int PV>
melt_status launch_split_k(const Job &job, const void *pack, size_t lds, int grid, hipStream_t s) {
    allow_lds(k_melt_split<Job, Op, FT, RT, WF, PV>);
    k_melt_split<Job, Op, FT, RT, WF, PV><<<grid, 512, lds, s>>>(job, (const split_u32x4 *)pack);
    return hip_check(hipGetLastError(), "melt split launch");
}

template <class Op, class Job>
melt_status launch_split(const Plan &p, Job job, const Geometry &geo, const SplitShape &h, const void *pk, int64_t est_chunks,
                         hipStream_t s) {
    if (h.parts == 0) return set_error(MELT_E_UNSUPPORTED, "split kernel: unsupported geometry");
    job.g.nsub = kSplitChunk / split_sf(h);
    job.g.parts = h.parts;
    const int grid = split_grid(p, h, est_chunks * job.g.nsub * h.parts);
    size_t lds = split_lds(Op::P, geo, h);
    if (job.a.clips.off) {
        job.a.list_off = (int)lds;                 // a multiple of 16
        lds += kListBytes;
    }
    constexpr int PW = Op::P == 3 ? 26 : 34;       // the wide staging of 128-frame items
#define SPLIT_CASE(FT, RT, WF, PV) \
    if (h.ft == FT && h.rt == RT && h.wf == WF && h.pv == PV) return launch_split_k<Job, Op, FT, RT, WF, PV>(job, pk, lds, grid, s);
    SPLIT_CASE(4, 1, 2, 18) SPLIT_CASE(4, 2, 2, 18) SPLIT_CASE(4, 3, 2, 18) SPLIT_CASE(4, 4, 2, 18)
    SPLIT_CASE(4, 5, 2, 18) SPLIT_CASE(4, 6, 2, 18) SPLIT_CASE(4, 8, 2, 18)
    SPLIT_CASE(4, 1, 2, PW) SPLIT_CASE(4, 2, 2, PW) SPLIT_CASE(4, 3, 2, PW) SPLIT_CASE(4, 4, 2, PW)
    SPLIT_CASE(4, 5, 2, PW) SPLIT_CASE(4, 6, 2, PW) SPLIT_CASE(4, 8, 2, PW)
    SPLIT_CASE(4, 1, 1, 18) SPLIT_CASE(4, 2, 1, 18) SPLIT_CASE(4, 3, 1, 18) SPLIT_CASE(4, 4, 1, 18)
    SPLIT_CASE(1, 1, 2, 10) SPLIT_CASE(1, 2, 2, 10)
#undef SPLIT_CASE
    return set_error(MELT_E_UNSUPPORTED, "split kernel: no such shape");
}

// The forward over a chunk table.
template <class Op>
melt_status launch_split_forward(const Plan &p, const FwdTask &t) {
    const Geometry &geo = p.geoS;
    const int T16 = (p.M + 7) / 8, tail = p.N - (geo.J - 1) * p.H;
    const SplitShape h = split_shape(geo, Op::P, T16, p.cu_count, t.est_chunks, t.n_frames);
    const SplitForward job{make_args(p, geo, Op::P * geo.Hp + 8, t),
                           {geo.n_groups, geo.Hp / 32, T16, 0, 0, p.d_basis32, p.N,
                            tail < p.H && tail % 32 > 0 && tail % 32 <= 16}};
    return launch_split<Op>(p, job, geo, h, p.d_pack_split, t.est_chunks, t.stream);
}

}  // namespace melt
