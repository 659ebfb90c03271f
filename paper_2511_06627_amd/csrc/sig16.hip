// Mixed-precision signal model: the same two chained contractions as sig.hip
// (time signal, then band DFT; and the transpose), on fp16 MFMA
// (gfx950 v_mfma_f32_32x32x16_f16) with fp32 accumulation.
//
// Scaling keeps every fp16 operand near unit magnitude:
//  * tables: K and F carry power-of-two scales ks, fs (max entry in [0.5, 1));
//  * per line: the projection row (forward) or the data row (adjoint) is
//    scaled by a power of two so its largest entry is in [0.5, 1) (computed
//    beforehand by the row_scale kernel) and the split reduction undoes it
//    in fp32;
//  * per harmonic band (adjoint): data columns of band b are multiplied by a
//    plan-fixed power of two bs_b that lifts weak high harmonics toward unit
//    size, and the matching F columns by 1/bs_b, so the band's products keep
//    fp16's relative precision instead of sinking into subnormals.
// The first contraction's fp32 result (the time tile, |.| <= n_u or 2 n_b)
// is rounded to fp16 once to feed the second.
//
// Layout and wave pairs follow sig.hip: a 32x32x16 MFMA result register j of
// lane l holds time 8(j/4) + 4(l/32) + j%4, so eight result registers form one
// fp16 A operand whose k index maps to time 16 h + 8(e/4) + 4(l/32) + e%4, and
// the second contraction's tables are stored with that permutation.  The two
// waves of a pair form half of a chunk's time tile each and swap the partial
// tiles through LDS.
//
// The swap is spread over a chunk so that no wave waits for it: the partial
// tile of chunk c + 1 is formed and written during chunk c, one barrier ends
// the chunk, and the partner's half is read at the start of chunk c + 1 behind
// the next first contraction.  Table slices reach LDS by buffer loads, one or
// two chunks ahead, with fence-free barriers (every wave waits for its own
// loads); fragments are read several products ahead of their use.  (Before,
// every chunk had its barrier between its two contractions, with both waves of
// a SIMD waiting at it, and slices went through registers: matrix units 40%
// busy.  One wave per SIMD with all columns was tried: no faster, its time
// tiles and accumulators share the accumulation registers and are copied.)
// Sums keep their order, so results keep their bits.  Measured at 256 x 256 x
// 128 (T = 16384, two groups of 12 tiles): forward 340 -> 315 us, adjoint 341 ->
// 311; 192 x 192 x 96 (T = 8192, 14 tiles): 59 -> 62, 56 -> 52 (there 9 time splits'
// partial sums are a third of it).  What bounds it now is LDS: fragments read
// by the four pairs, partial tiles and the slices' arrival take about as many
// cycles as the products.

#include "device.h"

namespace mpi3d {

namespace {

constexpr int kWaves8 = 2 * kWaves;
constexpr int kXsBytes = 2 * kWaves * 2 * 16 * 64 * (int)sizeof(float);   // two parities of partial tiles

// LDS of a kernel whose first contraction takes NA fragments (1 KB) a chunk
// and whose second takes NB: partial tiles, and two or three buffers of A and
// of B slices -- three, so that a slice has two chunks to arrive, where they
// fit, the larger slice's buffers first to give way.
template <int NA, int NB>
struct Lds16 {
    static constexpr int kFree = 160 - kXsBytes / 1024;
    static constexpr int AB = 3 * (NA + NB) <= kFree || (NA <= NB && 3 * NA + 2 * NB <= kFree) ? 3 : 2;
    static constexpr int BB = AB * NA + 3 * NB <= kFree ? 3 : 2;
    static constexpr int kBytes = kXsBytes + (AB * NA + BB * NB) * 1024;
    // loads of the A and B slices a wave issues each (the last repeated)
    static constexpr int kOpsA = (NA + kWaves8 - 1) / kWaves8, kOpsB = (NB + kWaves8 - 1) / kWaves8;
    static_assert(kBytes <= 160 * 1024, "LDS");
};

template <int N>
__device__ __forceinline__ void slice_load(const f16x8 *src, f16x8 *dst, int wave, int lane)
{
    const __amdgpu_buffer_rsrc_t rs = buffer_table(src, N * 1024);
#pragma unroll
    for (int k = 0; k < (N + kWaves8 - 1) / kWaves8; ++k) {
        const int f = min(k * kWaves8 + wave, N - 1);
        buffer_dma16(rs, dst + f * 64, lane * 16, f * 1024);
    }
}

// The time loop both directions share.  Per chunk c (from c0 to c1 - 1), with
// NA fragments of the first contraction's table slice (half of them this
// wave's, from a0) and NB of the second's: first(frag, partial) forms the
// wave's partial time tile, second(c's tile as fp16, frags) its products.
template <int NA, int NB, class First, class Second>
__device__ __forceinline__ void chunk_loop(float *xs, f16x8 *lds, const f16x8 *ag, size_t astride, const f16x8 *bg,
                                           size_t bstride, int c0, int c1, int pair, int half, int wave, int lane,
                                           First first, Second second)
{
    using L = Lds16<NA, NB>;
    typedef float f32x4v __attribute__((ext_vector_type(4)));
    f16x8 *la = lds, *lb = lds + L::AB * NA * 64;
    // partial tiles as 16-byte words, word q of lane l at q * 64 + l
    auto slot = [&](int parity, int hf) {
        return reinterpret_cast<f32x4v *>(xs) + (((parity * kWaves + pair) * 2 + hf) * 4) * 64 + lane;
    };
    auto aload = [&](int c, int buf) { slice_load<NA>(ag + (size_t)min(c, c1 - 1) * astride, la + buf * NA * 64, wave, lane); };
    auto bload = [&](int c, int buf) { slice_load<NB>(bg + (size_t)min(c, c1 - 1) * bstride, lb + buf * NB * 64, wave, lane); };
    auto put = [&](int parity, const f32x16 &t) {
        f32x4v *own = slot(parity, half);
#pragma unroll
        for (int q = 0; q < 4; ++q) own[q * 64] = f32x4v{t[4 * q], t[4 * q + 1], t[4 * q + 2], t[4 * q + 3]};
    };
    // (the first tile needs its own slice alone; the loop, A of chunk c0 + 1 and B of c0)
    constexpr int kSpare = (L::AB == 3 ? L::kOpsA : 0) + (L::BB == 3 ? L::kOpsB : 0);
    aload(c0, 0);
    bload(c0, 0);
    aload(c0 + 1, 1);
    if (L::AB == 3) aload(c0 + 2, 2);
    if (L::BB == 3) bload(c0 + 1, 1);
    wait_vm_lgkm<L::kOpsA + L::kOpsB + kSpare>();
    block_barrier_nofence();
    f32x16 own = first(la + lane);
    put(0, own);
    wait_vm_lgkm<kSpare>();
    block_barrier_nofence();
    int an = 1, af = 0, b = 0;                      // buffers: A of chunk c + 1, A free, B of chunk c
    for (int c = c0; c < c1; ++c) {
        const int parity = (c - c0) & 1;
        // into the buffers left by chunk c's A slice and chunk c - 1's B; those
        // the next chunk needs first
        auto aissue = [&] { aload(L::AB == 3 ? c + 3 : c + 2, af); };
        auto bissue = [&] { bload(L::BB == 3 ? c + 2 : c + 1, L::BB == 3 ? (b == 0 ? 2 : b - 1) : b ^ 1); };
        if (L::AB == 2) {
            aissue();
            bissue();
        } else {
            bissue();
            aissue();
        }
        f32x4v o[4];
        const f32x4v *other = slot(parity, 1 - half);
#pragma unroll
        for (int q = 0; q < 4; ++q) o[q] = other[q * 64];
        __builtin_amdgcn_sched_barrier(0);
        const f32x16 next = first(la + an * NA * 64 + lane);      // (past the range: unused)
        // the time tile: lower half + upper half, the same order on both waves
        f16x8 t16[2];
#pragma unroll
        for (int e = 0; e < 16; ++e) {
            const float p = o[e / 4][e % 4];
            t16[e / 8][e % 8] = (_Float16)(half == 0 ? own[e] + p : p + own[e]);
        }
        put(parity ^ 1, next);
        own = next;
        second(t16, lb + b * NB * 64 + lane);
        // the next chunk's slices are in (of this chunk's requests only those with
        // a chunk to spare may be outstanding), this wave's LDS accesses are done
        wait_vm_lgkm<kSpare>();
        block_barrier_nofence();
        af = an;
        an = an + 1 == L::AB ? 0 : an + 1;
        b = b + 1 == L::BB ? 0 : b + 1;
    }
    wait_vm_lgkm<0>();   // the repeated loads still in flight land before the LDS is handed on
}

template <int NUP, int GH>
__global__ __launch_bounds__(kSigThreads, 2) void sig_fwd_f16(SigArgs a)
{
    extern __shared__ __align__(16) unsigned char smem[];
    constexpr int NA = NUP / 16, NB = 4 * GH;     // PSF and band table fragments a chunk
    constexpr int NKS = NA / 2;                   // PSF steps of a half (16 samples each)
    const BlockPos bp = locate(a);
    const SigJob job = a.jobs[bp.job];
    const int lane = threadIdx.x & 63, h = lane >> 5;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), half = wave & 1;
    const int r = bp.row0 + (lane & 31);
    // input line of this lane's row (-1: past the job's rows, zero input)
    const long il = r < job.rows ? job_line(job, r) : -1;
    const int c0 = bp.split * a.cps, c1 = min(c0 + a.cps, a.nchunks);
    if (c0 >= c1) return;                         // the whole block

    // this wave's half of the line as fp16 B operands: the line scaled by its
    // power-of-two scale and rounded by the row_scale kernel (zero past n_u)
    f16x8 R[NKS];
    {
        const f16x8 *rin = (const f16x8 *)(job.in16 + (size_t)(il >= 0 ? il : 0) * job.in16_stride +
                                           half * (NUP / 2) + 8 * h);
#pragma unroll
        for (int st = 0; st < NKS; ++st) R[st] = rin[2 * st];     // (unconditional: all in flight)
#pragma unroll
        for (int st = 0; st < NKS; ++st) R[st] = il >= 0 ? R[st] : f16x8(0);
    }
    f32x16 acc[GH];
#pragma unroll
    for (int g = 0; g < GH; ++g) acc[g] = 0.f;

    const size_t fstride = (size_t)a.nct * 128;
    chunk_loop<NA, NB>(
        reinterpret_cast<float *>(smem), reinterpret_cast<f16x8 *>(smem + kXsBytes), (const f16x8 *)job.kf16,
        NA * 64, (const f16x8 *)a.ff16 + (size_t)bp.group * NB * 64, fstride, c0, c1, wave >> 1, half, wave, lane,
        [&](const f16x8 *kb) {
            f32x16 S = 0.f;
            lds_pipelined<NKS, 6>([&](int i) { return kb[(half * NKS + i) * 64]; },
                                  [&](int i, const f16x8 &f) { S = MFMA16(f, R[i], S); });
            return S;
        },
        [&](const f16x8 (&s16)[2], const f16x8 *fb) {
            lds_pipelined<2 * GH, 4>([&](int j) { return fb[(half * 2 * GH + (j % GH) * 2 + j / GH) * 64]; },
                                     [&](int j, const f16x8 &f) { acc[j % GH] = MFMA16(s16[j / GH], f, acc[j % GH]); });
        });
    if (bp.row0 >= job.rows) return;
    float *out = job.part + (size_t)bp.split * job.part_stride + (bp.group * 2 * GH + half * GH) * 32 + (lane & 31);
    store_rows<GH>(job, bp.row0 + 4 * h, a.nbp2, out, acc);
}

template <int NUP, int GH>
__global__ __launch_bounds__(kSigThreads, 2) void sig_adj_f16(SigArgs a)
{
    extern __shared__ __align__(16) unsigned char smem[];
    constexpr int NA = 4 * GH, NB = NUP / 16;     // band and PSF table fragments a chunk
    constexpr int NF = 2 * GH;                    // band steps of a half (16 columns each)
    constexpr int PTH = NUP / 64;                 // detector tiles of a half
    const BlockPos bp = locate(a);
    const SigJob job = a.jobs[bp.job];
    const int lane = threadIdx.x & 63, h = lane >> 5;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), half = wave & 1;
    const int r = bp.row0 + (lane & 31);
    const long il = r < job.rows ? job_line(job, r) : -1;
    const int c0 = bp.split * a.cps, c1 = min(c0 + a.cps, a.nchunks);
    if (c0 >= c1) return;                         // the whole block
    const int colbase = (bp.group * 2 * GH + half * GH) * 32;

    // this wave's bins of the line as fp16 B operands: the band-scaled row
    // times the line's power-of-two scale, rounded by the row_scale kernel
    // (zero past 2 nb)
    f16x8 Y[NF];
    {
        const f16x8 *yin = (const f16x8 *)(job.in16 + (size_t)(il >= 0 ? il : 0) * job.in16_stride + colbase + 8 * h);
#pragma unroll
        for (int st = 0; st < NF; ++st) Y[st] = yin[2 * st];
#pragma unroll
        for (int st = 0; st < NF; ++st) Y[st] = il >= 0 ? Y[st] : f16x8(0);
    }
    f32x16 racc[PTH];
#pragma unroll
    for (int pt = 0; pt < PTH; ++pt) racc[pt] = 0.f;

    const size_t fstride = (size_t)a.nct * 128;
    chunk_loop<NA, NB>(
        reinterpret_cast<float *>(smem), reinterpret_cast<f16x8 *>(smem + kXsBytes),
        (const f16x8 *)a.fa16 + (size_t)bp.group * NA * 64, fstride, (const f16x8 *)job.ka16, NB * 64, c0, c1,
        wave >> 1, half, wave, lane,
        [&](const f16x8 *fb) {
            f32x16 G = 0.f;
            lds_pipelined<NF, 6>([&](int i) { return fb[(half * NF + i) * 64]; },
                                 [&](int i, const f16x8 &f) { G = MFMA16(f, Y[i], G); });
            return G;
        },
        [&](const f16x8 (&g16)[2], const f16x8 *kb) {
            lds_pipelined<2 * PTH, 4>([&](int j) { return kb[((half * PTH + j % PTH) * 2 + j / PTH) * 64]; },
                                      [&](int j, const f16x8 &f) {
                                          racc[j % PTH] = MFMA16(g16[j / PTH], f, racc[j % PTH]);
                                      });
        });
    if (bp.row0 >= job.rows) return;
    float *out = job.part + (size_t)(bp.split * a.ngroups + bp.group) * job.part_stride + half * PTH * 32 + (lane & 31);
    store_rows<PTH>(job, bp.row0 + 4 * h, NUP, out, racc);
}

typedef void (*SigKernel)(SigArgs);

constexpr int kNups[] = {64, 128, 192, 256};
constexpr int kGHs[] = {3, 4, 6, 7};

int gh_slot(int gct)
{
    for (int i = 0; i < 4; ++i)
        if (gct == 2 * kGHs[i]) return i;
    return -1;
}
int nup_slot(int nup)
{
    for (int i = 0; i < 4; ++i)
        if (nup == kNups[i]) return i;
    return -1;
}

#define LDS2(NUP, GH) {Lds16<NUP / 16, 4 * GH>::kBytes, Lds16<4 * GH, NUP / 16>::kBytes}
#define LROW(NUP) {LDS2(NUP, 3), LDS2(NUP, 4), LDS2(NUP, 6), LDS2(NUP, 7)}
const int kLds[4][4][2] = {LROW(64), LROW(128), LROW(192), LROW(256)};   // forward, adjoint
#undef LROW
#undef LDS2

#define ROW(NUP, F) {F<NUP, 3>, F<NUP, 4>, F<NUP, 6>, F<NUP, 7>}
const SigKernel kFwd[4][4] = {ROW(64, sig_fwd_f16), ROW(128, sig_fwd_f16), ROW(192, sig_fwd_f16),
                              ROW(256, sig_fwd_f16)};
const SigKernel kAdj[4][4] = {ROW(64, sig_adj_f16), ROW(128, sig_adj_f16), ROW(192, sig_adj_f16),
                              ROW(256, sig_adj_f16)};
#undef ROW

}  // namespace

int sig16_supported(int nup, int gct, int pairs)
{
    return pairs == kWaves && nup_slot(nup) >= 0 && gh_slot(gct) >= 0;
}

// Dynamic LDS above 64 KB has to be allowed per kernel.
static hipError_t allow_lds(const void *kernel, int bytes)
{
    if (bytes <= 64 * 1024) return hipSuccess;
    return hipFuncSetAttribute(kernel, hipFuncAttributeMaxDynamicSharedMemorySize, bytes);
}

hipError_t launch_sig_fwd16(const mpi3d_plan *pl, SigArgs &a, hipStream_t st)
{
    const int ns = nup_slot(pl->nup), gs = gh_slot(a.gct);
    if (ns < 0 || gs < 0 || a.pairs != kWaves || !pl->kf16) return hipErrorInvalidValue;
    hipError_t e = allow_lds((const void *)kFwd[ns][gs], kLds[ns][gs][0]);
    if (e != hipSuccess) return e;
    const int blocks = a.total_tiles * a.nsplit * a.ngroups;
    hipLaunchKernelGGL(kFwd[ns][gs], dim3(blocks), dim3(kSigThreads), kLds[ns][gs][0], st, a);
    return hipGetLastError();
}

hipError_t launch_sig_adj16(const mpi3d_plan *pl, SigArgs &a, hipStream_t st)
{
    const int ns = nup_slot(pl->nup), gs = gh_slot(a.gct);
    if (ns < 0 || gs < 0 || a.pairs != kWaves || !pl->ka16) return hipErrorInvalidValue;
    hipError_t e = allow_lds((const void *)kAdj[ns][gs], kLds[ns][gs][1]);
    if (e != hipSuccess) return e;
    const int blocks = a.total_tiles * a.nsplit * a.ngroups;
    hipLaunchKernelGGL(kAdj[ns][gs], dim3(blocks), dim3(kSigThreads), kLds[ns][gs][1], st, a);
    return hipGetLastError();
}

}  // namespace mpi3d
