// The dense FP32 signal stage on fp16 pairs (gfx950 v_mfma_f32_32x32x16_f16):
// for scans whose band DFT does not factor over drive cycles (T no multiple of
// 32, or more bins a residue than the factored stage takes), or whose phase sums
// would have to be cut into ranges of line tiles that are slower.
//
// Per 32-time chunk c and line tile, forward: the PSF contraction
// S[time][line] = sum_p K[time][p] rho[p][line], then the band DFT
// b[column][line] += sum_time F[column][time] S[time][line]; adjoint the
// transpose of both.  Every operand is held as two fp16 values (split8: three
// products in place of one fp32 product at 1/16 of the rate); lines are scaled
// by a power of two each, the PSF tables by one for all, the band tables by one
// a column.  The time tile's result
// registers are the second contraction's operand as they stand, so nothing
// crosses lanes.  A wave holds 32 lines and GT column tiles (accumulators
// forward, data operands adjoint: GT 16 registers, the samples taking
// NUP / 2); column groups of their own blocks repeat the PSF contraction,
// (NUP / 16) 3 products of a chunk against the group's 6 GT.  Splits over T
// fill the chip; their partial sums are added in a fixed order afterwards.
//
// The long sums keep the small products (hi lo, lo hi) in accumulators of their own
// where the registers allow (blocks of 4 waves), and forward ranges of at most 24
// chunks are preferred: against products of fp32 numbers on the fp32 matrix unit the
// errors of 26 drawn scans are 0.4 to 1.0 times as large.
//
// Against the same stages on fp32 MFMA (forward, adjoint, with reductions): a
// raster of 131 x 117 x 37, 23 angles, T = 6001, 434 columns: 96 -> 58 us,
// 93 -> 49 (a normal product 246 -> 131); 192 x 192 x 96, 36 angles, T = 8101:
// 365 -> 165, 326 -> 164; 256 x 256 x 128, 60 angles, T = 10001, 658 columns:
// 1149 -> 826, 1135 -> 865 (a chunk's products 60 to 80% of the matrix rate; what
// keeps small scans off
// it is some 12 us a block for its lines, first chunks and results).

#include "device.h"

namespace mpi3d {

typedef float f32x4 __attribute__((ext_vector_type(4)));

namespace {

// A chunk's tables in LDS, 1 KB fragments: the PSF table's NUP / 8 (hi, lo),
// then the column group's 4 GT.  Three buffers, moved by buffer loads (the
// chunk after next while one is used), one barrier a chunk without a fence:
// each wave waits for its own part of the next chunk first.  Where the waves
// do not divide the fragments the last ones are moved twice (the same bytes).
template <int NUP, int GT, int WAVES>
struct ChunkStage {
    static constexpr int kPsf = NUP / 8;
    static constexpr int kFrags = kPsf + 4 * GT;
    static constexpr int kOps = (kFrags + WAVES - 1) / WAVES;   // fragments a wave moves per chunk
    static constexpr int kBytes = 3 * kFrags * 1024;
    __amdgpu_buffer_rsrc_t psf, band;
    int nct, tile0, last;

    // chunks [c0, c0 + n) of the tables; column tiles from ct on (past the
    // group's last tile: the next chunk's, or zeros past the table, unused)
    __device__ __forceinline__ ChunkStage(const __half *k, const __half *f, int c0, int n, int nct_, int ct)
        : psf(buffer_table((const char *)k + (size_t)c0 * kPsf * 1024, n * (kPsf * 1024))),
          band(buffer_table((const char *)f + (size_t)c0 * nct_ * 4096, n * nct_ * 4096)), nct(nct_), tile0(ct),
          last(n - 1)
    {
    }
    // chunk c (counted from c0; the last one again past it, unused)
    __device__ __forceinline__ void load(int c, f16x8 *lds, int buf, int wave, int lane) const
    {
        const int cc = min(c, last);
#pragma unroll
        for (int k = 0; k < kOps; ++k) {
            const int f = min(k * WAVES + wave, kFrags - 1);
            f16x8 *dst = lds + (buf * kFrags + f) * 64;
            if (f < kPsf)
                buffer_dma16(psf, dst, lane * 16, (cc * kPsf + f) * 1024);
            else
                buffer_dma16(band, dst, lane * 16, ((cc * nct + tile0) * 4 + f - kPsf) * 1024);
        }
    }
};

// Position of a wave: blocks are ordered split, column group, line tiles, so
// that neighbours (one XCD's) share a chunk range and with it the tables in L2.
struct SplitPos {
    int job, lines, tile, group, split, c0, c1;
};

template <int WAVES>
__device__ __forceinline__ SplitPos split_pos(const SplitArgs &a)
{
    SplitPos p;
    p.job = 0;
    for (int j = 1; j < a.njobs; ++j)
        if ((int)blockIdx.x >= a.jobs[j].blk0) p.job = j;
    const SplitJob &job = a.jobs[p.job];
    const int lb = xcd_logical((int)blockIdx.x - job.blk0, job.tgroups * a.ngroups * job.nsplit);
    const int sg = lb / job.tgroups, tg = lb - sg * job.tgroups;
    p.split = sg / a.ngroups;
    p.group = sg - p.split * a.ngroups;
    p.lines = a.nlines > 1 && tg >= job.lines[1].tile0 ? 1 : 0;
    p.tile = (tg - job.lines[p.lines].tile0) * WAVES + __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    p.c0 = (int)((unsigned)(p.split * a.nchunks) / (unsigned)job.nsplit);   // (at most 2^17 chunks, 128 splits)
    p.c1 = (int)((unsigned)((p.split + 1) * a.nchunks) / (unsigned)job.nsplit);
    return p;
}

// A line's scaled pairs in the 16-value steps of the MFMA operands (value
// 16 ks + 8 h + e in element e): the n values from column col0 of line il of
// `base` (il < 0: zeros), lines `stride` floats apart, by VEC-float loads where
// they are aligned.  Past the values the last word of the line is read and
// masked off: every load is unconditional, so all are in flight at once.
// EXP: cexp holds the exponents of the powers of two the values are taken by,
// from col0 on (16-byte aligned, padded); the line's largest exponent counts
// them, so nothing underflows on the way.  Returns the line's exponent.
template <int NKS, int VEC, bool EXP>
__device__ __forceinline__ int split_line(const float *base, long il, int stride, int col0, int n, int h,
                                          const int *cexp, f16x8 (&hi)[NKS], f16x8 (&lo)[NKS])
{
    typedef float vec __attribute__((ext_vector_type(VEC)));
    const float *src = base + (size_t)(il >= 0 ? il : 0) * stride;
    float v[NKS][8];
    if (stride % VEC == 0 && col0 % VEC == 0 && (uintptr_t)base % (4 * VEC) == 0) {
#pragma unroll
        for (int ks = 0; ks < NKS; ++ks)
#pragma unroll
            for (int e = 0; e < 8; e += VEC) {
                const int p = 16 * ks + 8 * h + e;
                const vec w = *reinterpret_cast<const vec *>(src + min(col0 + p, stride - VEC));
#pragma unroll
                for (int i = 0; i < VEC; ++i) v[ks][e + i] = (il >= 0) & (p + i < n) ? w[i] : 0.f;
            }
    } else {
#pragma unroll
        for (int ks = 0; ks < NKS; ++ks)
#pragma unroll
            for (int e = 0; e < 8; ++e) {
                const int p = 16 * ks + 8 * h + e;
                const float w = src[col0 + min(p, n - 1)];
                v[ks][e] = (il >= 0) & (p < n) ? w : 0.f;
            }
    }
    if constexpr (EXP) {
        // (a step's exponents at a time, read twice: the registers hold no more)
        typedef int i32x4 __attribute__((ext_vector_type(4)));
        auto exps = [&](int ks, int (&x)[8]) {
#pragma unroll
            for (int q = 0; q < 2; ++q) {
                const i32x4 w = *reinterpret_cast<const i32x4 *>(cexp + 16 * ks + 8 * h + 4 * q);
#pragma unroll
                for (int e = 0; e < 4; ++e) x[4 * q + e] = w[e];
            }
        };
        constexpr int kZero = -10000;             // below every exponent
        int m = kZero;
#pragma unroll
        for (int ks = 0; ks < NKS; ++ks) {
            int x[8];
            exps(ks, x);
#pragma unroll
            for (int e = 0; e < 8; ++e)
                m = max(m, v[ks][e] != 0.f ? __builtin_amdgcn_frexp_expf(v[ks][e]) + x[e] : kZero);
            __builtin_amdgcn_sched_barrier(0);
        }
        m = max(m, __shfl_xor(m, 32));
        const int le = m > kZero ? 15 - m : 0;
#pragma unroll
        for (int ks = 0; ks < NKS; ++ks) {
            int x[8];
            exps(ks, x);
            float w[8];
#pragma unroll
            for (int e = 0; e < 8; ++e) w[e] = __builtin_ldexpf(v[ks][e], le + x[e]);
            split8(w, hi[ks], lo[ks]);
            __builtin_amdgcn_sched_barrier(0);
        }
        return le;
    }
    float m = 0.f;
#pragma unroll
    for (int ks = 0; ks < NKS; ++ks)
#pragma unroll
        for (int e = 0; e < 8; ++e) m = fmaxf(m, fabsf(v[ks][e]));
    m = fmaxf(m, __shfl_xor(m, 32));
    const int le = line_exponent(m);
#pragma unroll
    for (int ks = 0; ks < NKS; ++ks) {
        float w[8];
#pragma unroll
        for (int e = 0; e < 8; ++e) w[e] = __builtin_ldexpf(v[ks][e], le);
        split8(w, hi[ks], lo[ks]);
    }
    return le;
}

// Result rows of a 32 x 32 tile (8 (s / 4) + 4 h + s % 4) of this lane's line, by
// the chain's sign and scaled back (rexp: by an exponent a row as well, from row 4 h on; null: none),
// as 16-byte words.
__device__ __forceinline__ void store_tile(float *dst, const f32x16 &v, float sign, int exp, const int *rexp)
{
#pragma unroll
    for (int q = 0; q < 4; ++q) {
        f32x4 w;
#pragma unroll
        for (int e = 0; e < 4; ++e) w[e] = __builtin_ldexpf(v[4 * q + e] * sign, exp - (rexp ? rexp[8 * q + e] : 0));
        *reinterpret_cast<f32x4 *>(dst + 8 * q) = w;
    }
}

// A chunk's time tile from NS fragment pairs (hi, lo) at kb and the operand's
// pairs.  LOW: the small products (hi lo, lo hi) first, so that only the large ones
// round a full sum (the hi fragments are read twice).
template <int NS, bool LOW>
__device__ __forceinline__ f32x16 chunk_tile(const f16x8 *kb, const f16x8 (&hi)[NS], const f16x8 (&lo)[NS])
{
    f32x16 t = 0.f;
    if constexpr (LOW) {
        lds_pipelined<3 * NS, 6>([&](int i) { return kb[(i < 2 * NS ? i : 2 * (i - 2 * NS)) * 64]; },
                                 [&](int i, const f16x8 &f) {
                                     t = MFMA16(f, i < 2 * NS && i % 2 == 0 ? lo[i / 2] : hi[i < 2 * NS ? i / 2 : i - 2 * NS], t);
                                 });
    } else {
        lds_pipelined<2 * NS, 6>([&](int i) { return kb[i * 64]; },
                                 [&](int i, const f16x8 &f) {
                                     t = MFMA16(f, hi[i / 2], t);
                                     if (i % 2 == 0) t = MFMA16(f, lo[i / 2], t);
                                 });
    }
    return t;
}
// One wave a SIMD: that order, and accumulators of their own for the small
// products of the second contraction, for which it has the registers.
constexpr bool own_low(int waves) { return waves == 4; }

template <int NUP, int GT, int WAVES>
__global__ __launch_bounds__(64 * WAVES, WAVES / 4) void split_fwd_kernel(SplitArgs a)
{
    using Stage = ChunkStage<NUP, GT, WAVES>;
    constexpr int NKS = NUP / 16;
    extern __shared__ __align__(16) f16x8 lk[];
    const SplitPos sp = split_pos<WAVES>(a);
    const SplitJob &job = a.jobs[sp.job];
    const SplitLines &lines = job.lines[sp.lines];
    const int lane = threadIdx.x & 63, h = lane >> 5;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int r = sp.tile * 32 + (lane & 31);
    // a wave past the last tile still stages (and with one wave a SIMD computes,
    // too: a branch around the products costs copies of their accumulators)
    const bool active = WAVES == 4 || sp.tile * 32 < lines.rows;
    const long il = r < lines.rows ? job_line(lines, r) : -1;
    const Stage stage(a.k[sp.lines], a.f, sp.c0, sp.c1 - sp.c0, a.nct, sp.group * GT);
    stage.load(0, lk, 0, wave, lane);
    stage.load(1, lk, 1, wave, lane);

    f16x8 rh[NKS], rl[NKS];
    const int le = split_line<NKS, 4, false>(job.in, il, job.in_stride, 0, a.nu, h, nullptr, rh, rl);
    constexpr bool LOW = own_low(WAVES);
    f32x16 acc[GT], low[LOW ? GT : 1];
#pragma unroll
    for (int g = 0; g < GT; ++g) acc[g] = low[LOW ? g : 0] = 0.f;
    const float sign = chain_sign(sp.split, sp.tile), sscale = a.s_scale * sign;
    wait_vm_lgkm<Stage::kOps>();
    block_barrier_nofence();

    int buf = 0, nbuf = 2;
    for (int c = sp.c0; c < sp.c1; ++c) {
        stage.load(c - sp.c0 + 2, lk, nbuf, wave, lane);
        if (active) {
            const f16x8 *kb = lk + buf * Stage::kFrags * 64 + lane;
            const f32x16 S = chunk_tile<NKS, LOW>(kb, rh, rl);
            f16x8 sh[2], sl[2];
#pragma unroll
            for (int q = 0; q < 2; ++q) {
                float w[8];
#pragma unroll
                for (int e = 0; e < 8; ++e) w[e] = S[8 * q + e] * sscale;
                split8(w, sh[q], sl[q]);
            }
            // fragments [tile][time step][hi, lo], taken time step by time step
            // so that consecutive products go to different accumulators
            const f16x8 *fb = kb + Stage::kPsf * 64;
            lds_pipelined<4 * GT, 6>([&](int i) { return fb[((i / 2 % GT) * 4 + i / (2 * GT) * 2 + i % 2) * 64]; },
                                     [&](int i, const f16x8 &f) {
                                         const int q = i / (2 * GT), g = i / 2 % GT;
                                         f32x16 &l = LOW ? low[LOW ? g : 0] : acc[g];
                                         if (i % 2 == 0) {
                                             acc[g] = MFMA16(f, sh[q], acc[g]);
                                             l = MFMA16(f, sl[q], l);
                                         } else {
                                             l = MFMA16(f, sh[q], l);
                                         }
                                     });
        }
        wait_vm_lgkm<Stage::kOps>();      // the next chunk is in, this wave's reads are done
        block_barrier_nofence();
        buf = buf == 2 ? 0 : buf + 1;
        nbuf = nbuf == 2 ? 0 : nbuf + 1;
    }
    wait_vm_lgkm<0>();   // the repeated loads still in flight land before the LDS is handed on
    if (il < 0) return;
    float *out = job.part + (size_t)sp.split * job.part_stride + (size_t)il * a.pitch + 4 * h;
#pragma unroll
    for (int g = 0; g < GT; ++g) {
        const int ct = sp.group * GT + g;
        if constexpr (LOW) acc[g] += low[g];
        if (ct < a.nct) store_tile(out + 32 * ct, acc[g], sign, -(le + a.out_exp), a.cexp + 32 * ct + 4 * h);
    }
}

// EXP: bins of unequal gain (a.cexp)
template <int NUP, int GT, int WAVES, bool EXP>
__global__ __launch_bounds__(64 * WAVES, WAVES / 4) void split_adj_kernel(SplitArgs a)
{
    using Stage = ChunkStage<NUP, GT, WAVES>;
    constexpr int PT = NUP / 32, NZS = 2 * GT;
    extern __shared__ __align__(16) f16x8 lk[];
    const SplitPos sp = split_pos<WAVES>(a);
    const SplitJob &job = a.jobs[sp.job];
    const SplitLines &lines = job.lines[sp.lines];
    const int lane = threadIdx.x & 63, h = lane >> 5;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int r = sp.tile * 32 + (lane & 31);
    const bool active = WAVES == 4 || sp.tile * 32 < lines.rows;
    const long il = r < lines.rows ? job_line(lines, r) : -1;
    const Stage stage(a.k[sp.lines], a.f, sp.c0, sp.c1 - sp.c0, a.nct, sp.group * GT);
    stage.load(0, lk, 0, wave, lane);
    stage.load(1, lk, 1, wave, lane);

    f16x8 zh[NZS], zl[NZS];
    const int col0 = sp.group * GT * 32;
    const int le = split_line<NZS, 2, EXP>(job.in, il, job.in_stride, col0, a.nb2 - col0, h,
                                              a.cexp + col0, zh, zl);
    constexpr bool LOW = own_low(WAVES);
    f32x16 acc[PT], low[LOW ? PT : 1];
#pragma unroll
    for (int pt = 0; pt < PT; ++pt) acc[pt] = low[LOW ? pt : 0] = 0.f;
    const float sign = chain_sign(sp.split, sp.tile), gscale = a.s_scale * sign;
    wait_vm_lgkm<Stage::kOps>();
    block_barrier_nofence();

    int buf = 0, nbuf = 2;
    for (int c = sp.c0; c < sp.c1; ++c) {
        stage.load(c - sp.c0 + 2, lk, nbuf, wave, lane);
        if (active) {
            const f16x8 *kb = lk + buf * Stage::kFrags * 64 + lane;
            const f32x16 G = chunk_tile<NZS, LOW>(kb + Stage::kPsf * 64, zh, zl);   // fragments [16-column step][hi, lo]
            f16x8 gh[2], gl[2];
#pragma unroll
            for (int q = 0; q < 2; ++q) {
                float w[8];
#pragma unroll
                for (int e = 0; e < 8; ++e) w[e] = G[8 * q + e] * gscale;
                split8(w, gh[q], gl[q]);
            }
            // fragments [time step][detector tile][hi, lo]
            lds_pipelined<4 * PT, 6>([&](int i) { return kb[i * 64]; },
                                     [&](int i, const f16x8 &f) {
                                         const int q = i / (2 * PT), pt = i / 2 % PT;
                                         f32x16 &l = LOW ? low[LOW ? pt : 0] : acc[pt];
                                         if (i % 2 == 0) {
                                             acc[pt] = MFMA16(f, gh[q], acc[pt]);
                                             l = MFMA16(f, gl[q], l);
                                         } else {
                                             l = MFMA16(f, gh[q], l);
                                         }
                                     });
        }
        wait_vm_lgkm<Stage::kOps>();
        block_barrier_nofence();
        buf = buf == 2 ? 0 : buf + 1;
        nbuf = nbuf == 2 ? 0 : nbuf + 1;
    }
    wait_vm_lgkm<0>();
    if (il < 0) return;
    float *out = job.part + (size_t)(sp.split * a.ngroups + sp.group) * job.part_stride + (size_t)il * a.pitch + 4 * h;
#pragma unroll
    for (int pt = 0; pt < PT; ++pt) {
        if constexpr (LOW) acc[pt] += low[pt];
        store_tile(out + 32 * pt, acc[pt], sign, -(le + a.out_exp), nullptr);
    }
}

typedef void (*SplitKernel)(SplitArgs);
struct SplitEntry {
    int nup, gt, waves;
    SplitKernel fwd, adj, adj_exp;
    int lds;
};
#define ENTRY(N, G, W) {N, G, W, split_fwd_kernel<N, G, W>, split_adj_kernel<N, G, W, false>, split_adj_kernel<N, G, W, true>, ChunkStage<N, G, W>::kBytes}
// (two waves a SIMD, or one with as many columns as three chunks in LDS hold)
const SplitEntry kSplit[] = {
    ENTRY(64, 4, 8), ENTRY(64, 6, 8), ENTRY(64, 8, 8), ENTRY(64, 4, 4), ENTRY(64, 6, 4), ENTRY(64, 8, 4),
    ENTRY(128, 4, 8), ENTRY(128, 6, 8), ENTRY(128, 7, 8), ENTRY(128, 8, 8), ENTRY(128, 4, 4), ENTRY(128, 6, 4), ENTRY(128, 7, 4), ENTRY(128, 8, 4),
    ENTRY(192, 4, 8), ENTRY(192, 5, 8), ENTRY(192, 6, 8), ENTRY(192, 4, 4), ENTRY(192, 5, 4), ENTRY(192, 7, 4),
    ENTRY(256, 3, 8), ENTRY(256, 4, 8), ENTRY(256, 3, 4), ENTRY(256, 5, 4)};
#undef ENTRY
constexpr int kEntries = sizeof(kSplit) / sizeof(kSplit[0]);

}  // namespace

int split_config(int i, int nup, int *gt, int *waves)
{
    if (i < 0 || i >= kEntries) return -1;
    *gt = kSplit[i].gt;
    *waves = kSplit[i].waves;
    return kSplit[i].nup == nup ? 1 : 0;
}

hipError_t launch_split(SplitArgs &a, bool fwd, hipStream_t st)
{
    if (a.config < 0 || a.config >= kEntries || a.njobs < 1 || a.njobs > kMaxSplitJobs || a.nlines < 1 || a.nlines > 2)
        return hipErrorInvalidValue;
    const SplitEntry &e = kSplit[a.config];
    if (e.nup != a.nup || a.nchunks > (1 << 17) || a.ngroups != (a.nct + e.gt - 1) / e.gt || a.nct != (a.nb2 + 31) / 32 ||
        a.pitch % 4 || a.pitch < (fwd ? 32 * a.nct : a.nup) || (double)a.nchunks * a.nct * 4096 >= 2147483647.0 ||
        (double)a.nchunks * a.nup * 128 >= 2147483647.0 || (fwd && !a.cexp))
        return hipErrorInvalidValue;
    int blocks = 0;
    for (int i = 0; i < a.njobs; ++i) {
        SplitJob &j = a.jobs[i];
        int tg = 0;
        for (int l = 0; l < a.nlines; ++l) {
            if (j.lines[l].tile0 != tg || j.lines[l].rows < 1) return hipErrorInvalidValue;
            tg += (j.lines[l].rows + 32 * e.waves - 1) / (32 * e.waves);
        }
        if (tg != j.tgroups || j.nsplit < 1 || j.nsplit > a.nchunks || j.nsplit > 128) return hipErrorInvalidValue;
        j.blk0 = blocks;
        blocks += j.tgroups * a.ngroups * j.nsplit;
    }
    const SplitKernel k = fwd ? e.fwd : a.cexp ? e.adj_exp : e.adj;
    const hipError_t err = hipFuncSetAttribute((const void *)k, hipFuncAttributeMaxDynamicSharedMemorySize, e.lds);
    if (err != hipSuccess) return err;
    hipLaunchKernelGGL(k, dim3(blocks), dim3(64 * e.waves), e.lds, st, a);
    return hipGetLastError();
}

}  // namespace mpi3d
