// The band DFT factored over drive cycles (FP32 results, gfx950
// v_mfma_f32_32x32x16_f16 on fp16 pairs).
//
// The kept bins omega_j (eq. bcompress) are integers, so with time t = n1 + P n2
// (n1 < P, n2 < C, T = C P) the DFT phase splits exactly:
//   omega_j t = omega_j n1 + (omega_j mod C) T n2 / C   (mod T),
// and the band DFT of a line's time signal s (Appendix A, eq. DCmodel)
//   b[j] = sum_t s[t] D_j e^{+2 pi i omega_j t / T} / sqrt(T)
// becomes two short sums: a C-point DFT over the drive cycles at the residues
// r of the kept bins mod C,
//   Y_r[n1] = sum_n2 s[n1 + P n2] e^{+2 pi i r n2 / C},
// then, per bin, a P-point sum over the phase within a cycle,
//   b[j] = sum_n1 G_j[n1] Y_r(j)[n1],   G_j[n1] = D_j e^{+2 pi i omega_j n1 / T} / sqrt(T).
// s is real, so Y_{C-r} is the conjugate of Y_r: the two share one slot of two
// columns (cos, sin), and C = 32 needs 16 slots whatever the bins are (several
// slots of equal columns where a pair has more bins than one takes).  The
// adjoint is the exact transpose of both steps.
//
// Forward: fac_fwd_kernel runs the PSF contraction of a line tile chunk by
// chunk (a chunk: 32 cycles n2 of one phase n1, PSF tables with their time
// rows in that order) and feeds each 32 x 32 (time x line) result straight
// into the residue DFT (table E), storing the phase sums Y once the C cycles
// of a phase are in; fac_fwd_out_kernel then forms b, one 32-column MFMA tile
// per unit of at most 16 bins of one slot.  Adjoint: fac_adj_in_kernel forms
// the phase sums Z from the data, fac_adj_kernel runs the residue DFT's
// transpose and the PSF contraction's transpose, accumulating the lines over
// its phases (split partial sums added in a fixed order afterwards).  Y and Z
// are laid out per 32-line tile as [phase][column][line] (column 2 slot +
// cos/sin): lanes are lines in the kernels that write them, so every store and
// load is whole 128-byte rows.
//
// Every product is of numbers held as two fp16 values (see split8): tables
// formed in float64, lines scaled by a power of two each.  At 256 x 256 x 128
// (7680 lines, T = 16384, C = 64, 20 slots) against the same contractions on
// fp32 MFMA: fac_fwd 715 -> 202 us, fac_adj 654 -> 210, fac_fwd_out 131 -> 74,
// fac_adj_in 142 -> 104 (1.1 PFLOP/s of fp16 products in the line-tile
// kernels, as a large fp16 matrix product reaches on this card; the outer sums
// write and read 315 MB of Y or Z at 3 to 4 TB/s, as 113 MB that stay in the last
// cache: what bounds them is the requests in flight, not the HBM); error of A
// against float64 4.5e-7 -> 2.4e-7.
//
// MFMA operand conventions: lane l supplies A[l % 32][8 (l / 32) + e] and
// B[8 (l / 32) + e][l % 32], e < 8; result register s of lane l holds row
// 8(s/4) + 4(l/32) + s%4, column l%32.  Every table is pre-swizzled so a
// lane's operand is one 16-byte word and a wave's 1 KB fragment is contiguous.

#include <type_traits>

#include "device.h"

namespace mpi3d {

typedef float f32x4 __attribute__((ext_vector_type(4)));

namespace {


// Wave position of the two line-tile kernels: a block of WAVES waves covers
// WAVES consecutive 32-line tiles for one of nsplit ranges of phases n1;
// consecutive logical blocks share a range, so they share the PSF table chunks
// in their XCD's L2.
struct FacPos {
    int tile, n1a, n1b, split;
};

// Kernel arguments of a launch of one job or of several.
template <bool BATCH>
using Args = std::conditional_t<BATCH, FacBatch, FacArgs>;
__device__ __forceinline__ const FacArgs &common(const FacArgs &a) { return a; }
__device__ __forceinline__ const FacArgs &common(const FacBatch &b) { return b.a; }

// The job of this block; block: its number in it (several jobs: blocks are laid
// one job after the other, else `one`).
__device__ __forceinline__ const FacJob &fac_job(const FacArgs &a, int &block, int one)
{
    block = one;
    return a.job;
}
__device__ __forceinline__ const FacJob &fac_job(const FacBatch &b, int &block, int)
{
    int jb = 0;
    for (int j = 1; j < b.njobs; ++j)
        if ((int)blockIdx.x >= b.jobs[j].blk0) jb = j;
    block = (int)blockIdx.x - b.jobs[jb].blk0;
    return b.jobs[jb];
}

template <int WAVES>
__device__ __forceinline__ FacPos fac_pos(const FacArgs &a, const FacJob &job, int block, int nsplit)
{
    const int tgroups = (job.tiles + WAVES - 1) / WAVES;
    const int lb = xcd_logical(block, tgroups * nsplit);
    FacPos p;
    p.split = lb / tgroups;
    p.tile = (lb - p.split * tgroups) * WAVES + __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    p.n1a = (int)((long)p.split * a.P / nsplit);
    p.n1b = (int)((long)(p.split + 1) * a.P / nsplit);
    return p;
}

// The same pair in one 32-bit word (hi in the low half), and eight of them as
// MFMA operands.
__device__ __forceinline__ uint32_t pack_split(float v)
{
    const _Float16 hi = (_Float16)v, lo = (_Float16)(v - (float)hi);
    return (uint32_t)__builtin_bit_cast(uint16_t, hi) | ((uint32_t)__builtin_bit_cast(uint16_t, lo) << 16);
}
__device__ __forceinline__ void unpack8(const uint32_t (&w)[8], f16x8 &hi, f16x8 &lo)
{
    uint32_t a[4], b[4];
#pragma unroll
    for (int e = 0; e < 4; ++e) {
        a[e] = __builtin_amdgcn_perm(w[2 * e + 1], w[2 * e], 0x05040100);
        b[e] = __builtin_amdgcn_perm(w[2 * e + 1], w[2 * e], 0x07060302);
    }
    typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));
    hi = __builtin_bit_cast(f16x8, u32x4{a[0], a[1], a[2], a[3]});
    lo = __builtin_bit_cast(f16x8, u32x4{b[0], b[1], b[2], b[3]});
}

// The PSF table of the line-tile kernels in LDS.  A chunk (32 times x NUP
// samples, hi and lo fragments, 128 NUP bytes) is used by all waves of a
// block; NS chunks make a stage, moved by buffer loads into three buffers so
// the stage after next is in flight while one is used, with one barrier a
// stage.  The barrier carries no fence: each wave waits for its own part of
// the next stage (every load but the youngest stage's) first.  (Buffer loads,
// because the compiler orders its LDS waits behind global_load_lds as behind
// flat accesses and then waits for every LDS read in flight at each use.)
template <int NUP, int NS, int WAVES>
struct PsfStage {
    static constexpr int kFragChunk = NUP / 8;                 // 1 KB fragments a chunk (hi, lo)
    static constexpr int kFrags = NS * kFragChunk;
    static constexpr int kOps = kFrags / WAVES;                // fragments a wave moves per stage
    static constexpr int kBytes = kFrags * 1024;
    static_assert(kFrags % WAVES == 0, "whole fragments a wave");
    // the stage from chunk c on (counted from the table at rs); chunks from
    // nchunks on repeat the last one (unused)
    static __device__ __forceinline__ void load(__amdgpu_buffer_rsrc_t rs, int c, int nchunks, f16x8 *lds, int buf,
                                                int wave, int lane)
    {
#pragma unroll
        for (int k = 0; k < kOps; ++k) {
            const int f = k * WAVES + wave;
            const int cc = min(c + f / kFragChunk, nchunks - 1);
            buffer_dma16(rs, lds + (buf * kFrags + f) * 64, lane * 16, (cc * kFragChunk + f % kFragChunk) * 1024);
        }
    }
    static __device__ __forceinline__ __amdgpu_buffer_rsrc_t table(const __half *tab, int c0, int chunks)
    {
        return buffer_table((const char *)tab + (size_t)c0 * kFragChunk * 1024, chunks * (kFragChunk * 1024));
    }
};

// Chunks a stage: about 32 KB for plain lines; a tensor line's NP tables are
// staged one by one (or all of a chunk's where they are small).
constexpr int stage_chunks(int nup, int np)
{
    if (np > 1) return nup == 64 && np % 2 == 0 ? np : 1;
    return nup == 64 ? 4 : nup == 128 ? 2 : 1;
}
// Waves of the forward line-tile kernel: two a SIMD while a line's operands
// (NP NUP / 2 registers) leave room, else one.
constexpr int fwd_waves(int nup, int np) { return np * nup <= 256 ? kFacWaves : 4; }

// Forward, per wave: 32 lines, phases [n1a, n1b).  Chunk c = n1 CJ + j holds
// the times n1 + P (32 j + i), i < 32.  Both contractions run on fp16 MFMA in
// split form (see split8): the lines scaled by a power of two each, the
// tables by one for all, three products a fragment.  The fp32 matrix unit has
// 1/16 of the fp16 rate, so three products cost 3/16 of one fp32 product; the
// errors against float64 are those of the fp32 form or less, because a step
// adds 16 products to the accumulator instead of 2.  The (time x line) result
// of the PSF contraction is split again and is the residue DFT's operand as
// it stands; that one's result rows are the phase's columns, its lanes lines,
// so a line's scale is undone by one exponent per lane and Y ([phase][column]
// [32 lines] per tile) is written in whole 128-byte rows.
//
// NP > 1, the tensor PSF: a line is the R + 1 = NP symmetric line sums laid
// end to end (NP NUP samples), its chunk the NP tables of a chunk one after
// the other, and their products go to one time tile.  The lines stay in
// registers (2 NP NUP / 64 words a lane, hi and lo), so above 256 samples a
// block is 4 waves of up to 512 registers.  At 192 x 192 x 96, 36 angles,
// T = 8192, four tables: 169 us against 628 for the dense pass on fp32 MFMA
// (0.8 PFLOP/s of fp16 products; with one wave a SIMD the splits of a time
// tile are not hidden), the adjoint 167 against 598.
template <int NUP, int ZST, int CJ, int NP, bool BATCH>
__global__ __launch_bounds__(64 * fwd_waves(NUP, NP), fwd_waves(NUP, NP) / 4) void fac_fwd_kernel(Args<BATCH> args)
{
    const FacArgs &a = common(args);
    constexpr int WAVES = fwd_waves(NUP, NP), NS = stage_chunks(NUP, NP);
    using Stage = PsfStage<NUP, NS, WAVES>;
    constexpr int NKS = NUP / 16;                     // PSF contraction steps a table
    constexpr int YC = 2 * ZST, RCT = (YC + 31) / 32; // columns of a phase, 32-column tiles
    constexpr int NE = RCT * 4;                       // residue table fragments a chunk
    constexpr int GRP = NP == 1 && NS > CJ ? NS : CJ;            // chunks of one loop body
    extern __shared__ __align__(16) f16x8 lk[];
    f16x8 *ebuf = lk + 3 * Stage::kFrags * 64;
    int block;
    const FacJob &job = fac_job(args, block, blockIdx.x);
    const FacPos fp = fac_pos<WAVES>(a, job, block, job.nsplit);
    if (fp.n1a >= fp.n1b) return;                 // the whole block
    const bool active = fp.tile < job.tiles;      // a wave past the last tile still stages
    const int tid = threadIdx.x, lane = tid & 63, h = lane >> 5;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int r = fp.tile * 32 + (lane & 31);
    const long il = active && job.row0 + r < job.rows ? job_line(job, job.row0 + r) : -1;
    const int c0 = fp.n1a * CJ, c1 = fp.n1b * CJ;

    const __amdgpu_buffer_rsrc_t kf = Stage::table(job.kf, c0 * NP, (c1 - c0) * NP);
    Stage::load(kf, 0, (c1 - c0) * NP, lk, 0, wave, lane);
    Stage::load(kf, NS, (c1 - c0) * NP, lk, 1, wave, lane);
    const f16x8 *ef = (const f16x8 *)a.ef;
    for (int idx = tid; idx < CJ * NE * 64; idx += 64 * WAVES) ebuf[idx] = ef[idx];

    // the line: samples 16 ks + 8 h + 0..7, scaled and split
    f16x8 rh[NP * NKS], rl[NP * NKS];
    {
        const float *rin = job.in + (size_t)(il >= 0 ? il : 0) * job.in_stride;
        const bool vec = job.in_stride % 4 == 0 && (uintptr_t)job.in % 16 == 0 && job.in_stride >= NP * NUP;
        auto get4 = [&](int ks, float (&v)[8]) {     // 16-byte loads
#pragma unroll
            for (int q = 0; q < 2; ++q) {
                const int p = 16 * ks + 8 * h + 4 * q;
                const f32x4 w = *reinterpret_cast<const f32x4 *>(rin + p);
#pragma unroll
                for (int e = 0; e < 4; ++e) v[4 * q + e] = (il >= 0) & (NP > 1 | p + e < a.nu) ? w[e] : 0.f;
            }
        };
        auto get1 = [&](int ks, float (&v)[8]) {
#pragma unroll
            for (int e = 0; e < 8; ++e) {
                const int p = 16 * ks + 8 * h + e;
                v[e] = il >= 0 && p < a.nu ? rin[p] : 0.f;
            }
        };
        float m = 0.f;
        auto scan = [&](const float (&v)[8]) {
#pragma unroll
            for (int e = 0; e < 8; ++e) m = fmaxf(m, fabsf(v[e]));
        };
        auto split = [&](int ks, int le, const float (&v)[8]) {
            float w[8];
#pragma unroll
            for (int e = 0; e < 8; ++e) w[e] = __builtin_ldexpf(v[e], le);
            split8(w, rh[ks], rl[ks]);
        };
        int le;
        if constexpr (NP == 1) {
            float v[NKS][8];
            if (vec) {               // (one branch: the loads of either form overlap)
#pragma unroll
                for (int ks = 0; ks < NKS; ++ks) get4(ks, v[ks]);
            } else {
#pragma unroll
                for (int ks = 0; ks < NKS; ++ks) get1(ks, v[ks]);
            }
#pragma unroll
            for (int ks = 0; ks < NKS; ++ks) scan(v[ks]);
            m = fmaxf(m, __shfl_xor(m, 32));
            le = line_exponent(m);
#pragma unroll
            for (int ks = 0; ks < NKS; ++ks) split(ks, le, v[ks]);
        } else {   // in two passes: the registers hold no whole line (the workspace's, 16-byte aligned)
#pragma unroll 4
            for (int ks = 0; ks < NP * NKS; ++ks) {
                float v[8];
                get4(ks, v);
                scan(v);
            }
            m = fmaxf(m, __shfl_xor(m, 32));
            le = line_exponent(m);
#pragma unroll
            for (int ks = 0; ks < NP * NKS; ++ks) {
                float v[8];
                get4(ks, v);
                split(ks, le, v);
            }
        }
        // (every phase range writes the same exponent)
        if (active && h == 0) job.lexp[r] = le + a.y_exp;
    }
    const float sscale = a.s_scale, yscale = a.y_scale;
    // this lane's line in the wave's Y tile (column 4 h of each group of 8)
    uint32_t *yrow = job.y + ((size_t)(active ? fp.tile : 0) * a.P * YC + 4 * h) * 32 + (lane & 31);

    f32x16 acc[RCT];
#pragma unroll
    for (int g = 0; g < RCT; ++g) acc[g] = 0.f;
    wait_vm_lgkm<Stage::kOps>();     // the first stage (and the table stores) are in
    block_barrier_nofence();

    int buf = 0, nbuf = 2;
    for (int cg = c0; cg < c1; cg += GRP) {
#pragma unroll
        for (int k = 0; k < GRP; ++k) {
            const int c = cg + k;
            // (with one wave a SIMD the waves past the last tile compute, too:
            // a branch around the time tile costs copies of it)
            const bool work = (NP > 1 || active) && (GRP == CJ || c < c1);
            f32x16 S;
#pragma unroll
            for (int e = 0; e < NP; ++e) {
                const int t = k * NP + e;
                if (t % NS == NS - 1) Stage::load(kf, (c - c0) * NP + e + NS + 1, (c1 - c0) * NP, lk, nbuf, wave, lane);
                if (work) {
                    const f16x8 *kb = lk + (buf * Stage::kFrags + (t % NS) * Stage::kFragChunk) * 64 + lane;
                    if (e == 0) S = 0.f;
                    lds_pipelined<2 * NKS, 6>([&](int i) { return kb[i * 64]; },
                                              [&](int i, const f16x8 &f) {
                                                  S = MFMA16(f, rh[e * NKS + i / 2], S);
                                                  if (i % 2 == 0) S = MFMA16(f, rl[e * NKS + i / 2], S);
                                              });
                    if (e == NP - 1) {
                        f16x8 sh[2], sl[2];
#pragma unroll
                        for (int q = 0; q < 2; ++q) {
                            float w[8];
#pragma unroll
                            for (int x = 0; x < 8; ++x) w[x] = S[8 * q + x] * sscale;
                            split8(w, sh[q], sl[q]);
                        }
                        const f16x8 *eb = ebuf + (k % CJ) * NE * 64 + lane;
#pragma unroll
                        for (int g = 0; g < RCT; ++g)
#pragma unroll
                            for (int q = 0; q < 2; ++q) {
                                const f16x8 eh = eb[(g * 4 + q * 2) * 64], el = eb[(g * 4 + q * 2 + 1) * 64];
                                acc[g] = MFMA16(eh, sh[q], acc[g]);
                                acc[g] = MFMA16(eh, sl[q], acc[g]);
                                acc[g] = MFMA16(el, sh[q], acc[g]);
                            }
                    }
                }
                if (t % NS == NS - 1) {
                    wait_vm_lgkm<Stage::kOps>();      // the next stage is in, this wave's reads are done
                    block_barrier_nofence();
                    buf = buf == 2 ? 0 : buf + 1;
                    nbuf = nbuf == 2 ? 0 : nbuf + 1;
                }
            }
            if (k % CJ == CJ - 1) {
                if (active && (GRP == CJ || c < c1)) {
                    uint32_t *d = yrow + (size_t)(c / CJ) * YC * 32;
#pragma unroll
                    for (int g = 0; g < RCT; ++g)
#pragma unroll
                        for (int s = 0; s < 16; ++s)
                            if (32 * g + 8 * (s / 4) < YC)
                                d[(32 * g + 8 * (s / 4) + s % 4) * 32] = pack_split(acc[g][s] * yscale);
                }
#pragma unroll
                for (int g = 0; g < RCT; ++g) acc[g] = 0.f;
            }
        }
    }
    wait_vm_lgkm<0>();   // the repeated loads still in flight land before the LDS is handed on
}

// Forward outer sum.  One wave: one slot, kOutTiles line tiles, a range of
// 8-phase stages (partial sums ps); no LDS and no barriers, since every value
// of Y is read by one wave only.  A step's K = 16 is 8 phases x 2 columns: a
// lane's operand is 8 packed words of its line, one per phase (two adjacent
// 128-byte rows a load), and the slot's bins are one or two units of 16 (32
// result columns, re/im).  The next stage's words and table fragments are
// requested before a stage's products.  What bounds it: the loads in flight (one
// stage ahead; Y at 4.0 TB/s, from HBM as from the last cache), and the
// tables from L2 (about as many bytes again for one tile a wave, so a wave
// takes two and the four waves of a block share the slot, hence its table
// lines in L1).
constexpr int kOutTiles = 2;
constexpr int kOutWaves = 4;
__host__ __device__ constexpr int out_groups(int tiles) { return (tiles + kOutTiles * kOutWaves - 1) / (kOutTiles * kOutWaves); }

template <int NU>
struct OutStage {
    uint32_t y[kOutTiles][8];
    f16x8 w[NU][2];
};

template <int NU>
__device__ __forceinline__ void fwd_out(const FacArgs &a, const FacJob &job, int q, int t0, int ps)
{
    const int lane = threadIdx.x & 63, h = lane >> 5;
    const int u0 = a.unit0[q];
    const int nst = (a.P + 7) / 8;
    const int s0 = (int)((long)ps * nst / job.psplit), s1 = (int)((long)(ps + 1) * nst / job.psplit);
    const uint32_t *y0 = job.y + ((size_t)t0 * a.P * a.yc + 2 * q) * 32 + lane;   // column 2 q + h, line l % 32
    const size_t tstep = t0 + 1 < job.tiles ? (size_t)a.P * a.yc * 32 : 0;        // (a missing second tile: the first)
    const f16x8 *w0 = (const f16x8 *)a.wf + (size_t)u0 * nst * 128 + lane;
    f32x16 acc[kOutTiles][NU];
#pragma unroll
    for (int t = 0; t < kOutTiles; ++t)
#pragma unroll
        for (int u = 0; u < NU; ++u) acc[t][u] = 0.f;
    // phases past P repeat the last one (their table entries are zero)
    auto load = [&](int stg, OutStage<NU> &g) {
#pragma unroll
        for (int j = 0; j < 8; ++j) {
            const uint32_t *yp = y0 + (size_t)min(8 * stg + j, a.P - 1) * a.yc * 32;
#pragma unroll
            for (int t = 0; t < kOutTiles; ++t) g.y[t][j] = yp[t * tstep];
        }
#pragma unroll
        for (int u = 0; u < NU; ++u)
#pragma unroll
            for (int p = 0; p < 2; ++p) g.w[u][p] = w0[((size_t)u * nst + stg) * 128 + p * 64];
    };
    auto products = [&](const OutStage<NU> &g) {
#pragma unroll
        for (int t = 0; t < kOutTiles; ++t) {
            f16x8 yh, yl;
            unpack8(g.y[t], yh, yl);
#pragma unroll
            for (int u = 0; u < NU; ++u) {
                acc[t][u] = MFMA16(yh, g.w[u][0], acc[t][u]);
                acc[t][u] = MFMA16(yl, g.w[u][0], acc[t][u]);
                acc[t][u] = MFMA16(yh, g.w[u][1], acc[t][u]);
            }
        }
    };
    int e[kOutTiles][16];
#pragma unroll
    for (int t = 0; t < kOutTiles; ++t)
#pragma unroll
        for (int j = 0; j < 16; ++j)
            e[t][j] = job.lexp[min(t0 + t, job.tiles - 1) * 32 + 4 * h + 8 * (j / 4) + j % 4];
    int we[NU];
#pragma unroll
    for (int u = 0; u < NU; ++u) we[u] = a.wexp[(u0 + u) * 32 + (lane & 31)];
    OutStage<NU> g0, g1;
    load(s0, g0);
    int stg = s0;
    for (; stg + 1 < s1; stg += 2) {
        load(stg + 1, g1);
        __builtin_amdgcn_sched_barrier(0);
        products(g0);
        load(min(stg + 2, s1 - 1), g0);
        __builtin_amdgcn_sched_barrier(0);
        products(g1);
    }
    if (stg < s1) products(g0);
    // rows: lines 8 (j / 4) + 4 h + j % 4; columns: the unit's 32
#pragma unroll
    for (int t = 0; t < kOutTiles; ++t) {
        const int row0 = (t0 + t) * 32 + 4 * h;
        if (t0 + t >= job.tiles) break;
#pragma unroll
        for (int j = 0; j < 16; ++j) {
            const int row = job.row0 + row0 + 8 * (j / 4) + j % 4;
            if (row >= job.rows) continue;
            float *o = job.part + ps * job.fwd_part_stride + (size_t)job_line(job, row) * a.ucols + u0 * 32 + (lane & 31);
#pragma unroll
            for (int u = 0; u < NU; ++u) o[32 * u] = __builtin_ldexpf(acc[t][u][j], -(e[t][j] + we[u]));
        }
    }
}

// (blocks of a job: tile groups, slots, stage ranges)
template <bool BATCH>
__global__ __launch_bounds__(64 * kOutWaves) void fac_fwd_out_kernel(Args<BATCH> args)
{
    const FacArgs &a = common(args);
    int group, q = blockIdx.y, ps = blockIdx.z;
    const FacJob &job = fac_job(args, group, blockIdx.x);
    if constexpr (BATCH) {
        const int tg = out_groups(job.tiles), sq = group / tg;
        group -= sq * tg;
        ps = sq / a.R;
        q = sq - ps * a.R;
    }
    const int t0 = kOutTiles * (group * kOutWaves + __builtin_amdgcn_readfirstlane(threadIdx.x >> 6));
    if (t0 >= job.tiles) return;
    if (a.unit0[q + 1] - a.unit0[q] == 1)
        fwd_out<1>(a, job, q, t0, ps);
    else
        fwd_out<2>(a, job, q, t0, ps);
}

// Adjoint outer sum: Z from the data, one block of kInWaves waves per 32-line
// tile and range of 16-phase stages.  Wave w takes slots w + kInWaves i (the
// plan numbers the slots so the waves' bin counts balance) and holds their
// bins of the tile's lines as split B operands (KST steps of 8 bins, re/im);
// per stage and slot the table's 32 rows (16 phases x 2 columns) times these
// give the slot's Z, whose lanes are lines: packed words stored in whole
// 128-byte rows.  No LDS in the loop and no barriers; the next stage's table
// fragments are requested before a stage's products, and slots in [R, zst)
// are written as zeros (the spare row takes the stores of slots past zst, so
// every stage issues the same stores).  What bounds it: the table loads from L2
// in flight beside Z's stores (Z at 3.1 TB/s, to HBM as to the last cache).  RPW slots a wave of KST steps: 16 slots of up to 32 bins
// or 24 of up to 24 -- what the registers of two waves a SIMD hold.
constexpr int kInWaves = kFacInWaves;

template <int RPW, int KST, bool BATCH>
__global__ __launch_bounds__(64 * kInWaves, 2) void fac_adj_in_kernel(Args<BATCH> args)
{
    const FacArgs &a = common(args);
    __shared__ int lmax[kInWaves][32];
    const int lane = threadIdx.x & 63, h = lane >> 5;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    int tile, zsp = blockIdx.y;
    const FacJob &job = fac_job(args, tile, blockIdx.x);
    if constexpr (BATCH) {
        zsp = tile / job.tiles;
        tile -= zsp * job.tiles;
    }
    const int row0 = tile * 32;
    const int r = row0 + (lane & 31);
    const long il = job.row0 + r < job.rows ? job_line(job, job.row0 + r) : -1;
    constexpr int QM = 8 * KST;
    // this block's stages [s0, s1): range zsp of zsplit
    const int nst = a.nzstage;
    const int s0 = (int)((long)zsp * nst / job.zsplit), s1 = (int)((long)(zsp + 1) * nst / job.zsplit);
    const int sfull = min(s1, a.P / 16);          // stages of 16 phases
    const float zscale = a.z_scale;
    auto table_load = [&](int stg, f16x8 (&t)[RPW][KST][2]) {
#pragma unroll
        for (int i = 0; i < RPW; ++i) {
            const int q = wave + kInWaves * i;
            const f16x8 *w = (const f16x8 *)a.wa + ((size_t)((q < a.R ? q : 0) * nst + stg) * KST) * 128 + lane;
#pragma unroll
            for (int ks = 0; ks < KST; ++ks)
#pragma unroll
                for (int p = 0; p < 2; ++p) t[i][ks][p] = w[(2 * ks + p) * 64];
        }
    };
    f16x8 ta[RPW][KST][2], tb[RPW][KST][2];
    table_load(s0, ta);
    // B operands: bins 8 ks + 4 h + 0..3 of the wave's slots, re/im.  The bin
    // numbers are requested together, then the data (clamped addresses,
    // masked values), so the loads overlap.  A bin's data takes the power of two
    // that its weights were raised by; the line's largest exponent counts it, so
    // nothing underflows on the way.
    f16x8 bh[RPW][KST], bl[RPW][KST];
    {
        float v[RPW][KST][8];
        int ex[RPW][KST][4];
        const float *yin = job.in + (size_t)(il >= 0 ? il : 0) * job.in_stride;
#pragma unroll
        for (int i = 0; i < RPW; ++i) {
            const int q = wave + kInWaves * i;
            const int *qb = a.qbin + (q < a.R ? q : 0) * QM + 4 * h;
            int jb[KST][4];
#pragma unroll
            for (int ks = 0; ks < KST; ++ks)
#pragma unroll
                for (int e = 0; e < 4; ++e) {
                    const int w = qb[8 * ks + e];
                    jb[ks][e] = (int16_t)w;
                    ex[i][ks][e] = w >> 16;
                }
#pragma unroll
            for (int ks = 0; ks < KST; ++ks)
#pragma unroll
                for (int e = 0; e < 8; ++e) {
                    const int j = jb[ks][e / 2];
                    const bool ok = q < a.R && il >= 0 && j >= 0;
                    const float w = yin[2 * max(j, 0) + e % 2];
                    v[i][ks][e] = ok ? w : 0.f;
                }
        }
        constexpr int kZero = -10000;         // below every exponent
        int m = kZero;
#pragma unroll
        for (int i = 0; i < RPW; ++i)
#pragma unroll
            for (int ks = 0; ks < KST; ++ks)
#pragma unroll
                for (int e = 0; e < 8; ++e) {
                    const float w = v[i][ks][e];
                    m = max(m, w != 0.f ? __builtin_amdgcn_frexp_expf(w) + ex[i][ks][e / 2] : kZero);
                }
        m = max(m, __shfl_xor(m, 32));
        if (lane < 32) lmax[wave][lane] = m;
        __syncthreads();
        m = kZero;
#pragma unroll
        for (int w = 0; w < kInWaves; ++w) m = max(m, lmax[w][lane & 31]);
        const int le = m > kZero ? 15 - m : 0;
        if (wave == 0 && lane < 32) job.lexp[r] = le + a.z_exp;   // (every stage range writes the same)
#pragma unroll
        for (int i = 0; i < RPW; ++i)
#pragma unroll
            for (int ks = 0; ks < KST; ++ks) {
                float w[8];
#pragma unroll
                for (int e = 0; e < 8; ++e) w[e] = __builtin_ldexpf(v[i][ks][e], le + ex[i][ks][e / 2]);
                split8(w, bh[i][ks], bl[i][ks]);
            }
    }
    uint32_t *const zt = job.y + (size_t)tile * 32 * a.P * a.yc;
    uint32_t *const spare = job.y + (size_t)job.ylines * a.P * a.yc;
    // result row 8 (s / 4) + 4 h + s % 4: phase row / 2, column row % 2
    auto stage = [&](int stg, const f16x8 (&t)[RPW][KST][2], bool full) {
#pragma unroll
        for (int i = 0; i < RPW; ++i) {
            const int q = wave + kInWaves * i;
            f32x16 acc = 0.f;
#pragma unroll
            for (int ks = 0; ks < KST; ++ks) {
                acc = MFMA16(t[i][ks][0], bh[i][ks], acc);
                acc = MFMA16(t[i][ks][0], bl[i][ks], acc);
                acc = MFMA16(t[i][ks][1], bh[i][ks], acc);
            }
            if (full) {
                uint32_t *d = (q < a.zst ? zt + ((size_t)16 * stg * a.yc + 2 * q) * 32 : spare);
                const int ph = q < a.zst ? a.yc * 32 : 0;   // words per phase
                d += (size_t)2 * h * ph + (lane & 31);
#pragma unroll
                for (int s = 0; s < 16; ++s)
                    d[(4 * (s / 4) + (s % 4) / 2) * ph + (s % 2) * 32] = q < a.R ? pack_split(acc[s] * zscale) : 0u;
            } else if (q < a.zst) {
#pragma unroll
                for (int s = 0; s < 16; ++s) {
                    const int n1 = 16 * stg + 4 * (s / 4) + 2 * h + (s % 4) / 2;
                    if (n1 < a.P)
                        zt[((size_t)n1 * a.yc + 2 * q + s % 2) * 32 + (lane & 31)] =
                            q < a.R ? pack_split(acc[s] * zscale) : 0u;
                }
            }
        }
    };
    int stg = s0;
    for (; stg + 1 < sfull; stg += 2) {
        table_load(stg + 1, tb);
        __builtin_amdgcn_sched_barrier(0);
        stage(stg, ta, true);
        table_load(min(stg + 2, s1 - 1), ta);
        __builtin_amdgcn_sched_barrier(0);
        stage(stg + 1, tb, true);
    }
    if (stg < sfull) {
        table_load(min(stg + 1, s1 - 1), tb);
        stage(stg, ta, true);
        if (stg + 1 < s1) stage(stg + 1, tb, false);
    } else if (stg < s1) {
        stage(stg, ta, false);
    }
}

// Adjoint, per wave: 32 lines, phases [n1a, n1b): for each chunk the residue
// DFT's transpose (A = E[time n2][column], B = Z[column][line]) then the PSF
// contraction's transpose into the lines; split partial sums per phase range.
// Split fp16 products and PSF-table stages as in the forward; Z comes in split
// pairs scaled by a power of two per line (lexp, undone in the partial sums),
// the next phase's words being requested before a phase's chunks.  The tensor
// PSF's tables are taken by blocks of their own (offset e's, whose lines are
// columns e NUP .. of the partial sums).
template <int NUP, int ZST, int CJ, bool BATCH>
__global__ __launch_bounds__(64 * kFacWaves, 2) void fac_adj_kernel(Args<BATCH> args)
{
    const FacArgs &a = common(args);
    constexpr int NS = stage_chunks(NUP, 1);
    using Stage = PsfStage<NUP, NS, kFacWaves>;
    constexpr int PT = NUP / 32;          // detector tiles
    constexpr int ZC = 2 * ZST, NZS = (ZC + 15) / 16;   // columns of a phase, steps of the residue DFT
    constexpr int NE = 2 * NZS;           // residue table fragments a chunk
    constexpr int GRP = NS > CJ ? NS : CJ;
    extern __shared__ __align__(16) f16x8 lk[];
    f16x8 *ebuf = lk + 3 * Stage::kFrags * 64;
    int block, pass = blockIdx.y;
    const FacJob &job = fac_job(args, block, blockIdx.x);
    if constexpr (BATCH) {
        const int per_pass = (job.tiles + kFacWaves - 1) / kFacWaves * job.nsplit_adj;
        pass = block / per_pass;
        block -= pass * per_pass;
    }
    const FacPos fp = fac_pos<kFacWaves>(a, job, block, job.nsplit_adj);
    if (fp.n1a >= fp.n1b) return;                 // the whole block
    const bool active = fp.tile < job.tiles;      // a wave past the last tile still stages
    const int tid = threadIdx.x, lane = tid & 63, h = lane >> 5;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int c0 = fp.n1a * CJ, c1 = fp.n1b * CJ;

    f32x16 racc[PT];
#pragma unroll
    for (int pt = 0; pt < PT; ++pt) racc[pt] = 0.f;
    const __amdgpu_buffer_rsrc_t ka = Stage::table(job.ka + pass * a.ka_stride, c0, c1 - c0);
    const f16x8 *ea = (const f16x8 *)a.ea;
    for (int idx = tid; idx < CJ * NE * 64; idx += 64 * kFacWaves) ebuf[idx] = ea[idx];
    // Z of this line tile, [phase][2 slot + part][32 lines]: this lane's line,
    // columns 16 ks + 8 h + 0..7 (past the last: a repeated column times zero
    // table entries)
    const uint32_t *zrow = job.y + (size_t)(active ? fp.tile : 0) * 32 * a.P * ZC + (lane & 31);
    auto zload = [&](int n1, uint32_t (&z)[NZS][8]) {
        const uint32_t *zp = zrow + (size_t)n1 * ZC * 32;
#pragma unroll
        for (int ks = 0; ks < NZS; ++ks)
#pragma unroll
            for (int e = 0; e < 8; ++e) {
                const int col = 16 * ks + 8 * h + e;
                z[ks][e] = zp[(16 * ks + 15 < ZC ? col : min(col, ZC - 1)) * 32];
            }
    };
    uint32_t zn[NZS][8];
    zload(fp.n1a, zn);
    __builtin_amdgcn_sched_barrier(0);
    Stage::load(ka, 0, c1 - c0, lk, 0, wave, lane);
    Stage::load(ka, NS, c1 - c0, lk, 1, wave, lane);
    const float sign = chain_sign(fp.split, fp.tile), gscale = a.g_scale * sign;
    wait_vm_lgkm<Stage::kOps>();
    block_barrier_nofence();

    int buf = 0, nbuf = 2;
    f16x8 zh[NZS], zl[NZS];
    for (int cg = c0; cg < c1; cg += GRP) {
#pragma unroll
        for (int k = 0; k < GRP; ++k) {
            const int c = cg + k;
            if (k % CJ == 0) {
#pragma unroll
                for (int ks = 0; ks < NZS; ++ks) unpack8(zn[ks], zh[ks], zl[ks]);
                zload(min(c / CJ + 1, fp.n1b - 1), zn);   // the next phase's operands
                __builtin_amdgcn_sched_barrier(0);
            }
            if (k % NS == NS - 1) Stage::load(ka, c - c0 + NS + 1, c1 - c0, lk, nbuf, wave, lane);
            if (active && (GRP == CJ || c < c1)) {
                const f16x8 *eb = ebuf + (k % CJ) * NE * 64 + lane;
                f32x16 G = 0.f;
#pragma unroll
                for (int ks = 0; ks < NZS; ++ks) {
                    const f16x8 eh = eb[2 * ks * 64], el = eb[(2 * ks + 1) * 64];
                    G = MFMA16(eh, zh[ks], G);
                    G = MFMA16(eh, zl[ks], G);
                    G = MFMA16(el, zh[ks], G);
                }
                f16x8 gh[2], gl[2];
#pragma unroll
                for (int q = 0; q < 2; ++q) {
                    float w[8];
#pragma unroll
                    for (int e = 0; e < 8; ++e) w[e] = G[8 * q + e] * gscale;
                    split8(w, gh[q], gl[q]);
                }
                // fragments in the order [step][tile][hi, lo]: consecutive
                // products go to different accumulators
                const f16x8 *kb = lk + (buf * Stage::kFrags + (k % NS) * Stage::kFragChunk) * 64 + lane;
                lds_pipelined<4 * PT, 4>([&](int i) { return kb[i * 64]; },
                                         [&](int i, const f16x8 &f) {
                                             const int q = i / (2 * PT), pt = i / 2 % PT;
                                             racc[pt] = MFMA16(gh[q], f, racc[pt]);
                                             if (i % 2 == 0) racc[pt] = MFMA16(gl[q], f, racc[pt]);
                                         });
            }
            if (k % NS == NS - 1) {
                wait_vm_lgkm<Stage::kOps>();      // the next stage is in, this wave's reads are done
                block_barrier_nofence();
                buf = buf == 2 ? 0 : buf + 1;
                nbuf = nbuf == 2 ? 0 : nbuf + 1;
            }
        }
    }
    wait_vm_lgkm<0>();   // the repeated loads still in flight land before the LDS is handed on
    if (!active) return;
    float *out = job.part + (size_t)fp.split * job.part_stride;
    const int row0 = fp.tile * 32 + 4 * h;
    int e[16];
#pragma unroll
    for (int j = 0; j < 16; ++j) e[j] = job.lexp[row0 + 8 * (j / 4) + j % 4];
#pragma unroll
    for (int j = 0; j < 16; ++j) {
        const int row = job.row0 + row0 + 8 * (j / 4) + j % 4;
        if (row >= job.rows) continue;
        float *o = out + (size_t)job_line(job, row) * a.adj_pitch + pass * NUP + (lane & 31);
#pragma unroll
        for (int pt = 0; pt < PT; ++pt) o[pt * 32] = __builtin_ldexpf(racc[pt][j] * sign, -(e[j] + a.r_exp));
    }
}

constexpr int kFacNups[] = {64, 128, 192, 256};
template <bool BATCH>
struct Kernels {
    typedef void (*Kernel)(Args<BATCH>);
    // C = 32 (CJ = 1): 16 slots hold every residue; C = 64 (CJ = 2): 16 to 24
#define FWD_ROW(NUP) \
    {fac_fwd_kernel<NUP, 16, 1, 1, BATCH>, fac_fwd_kernel<NUP, 16, 2, 1, BATCH>, fac_fwd_kernel<NUP, 20, 2, 1, BATCH>, fac_fwd_kernel<NUP, 24, 2, 1, BATCH>}
#define ADJ_ROW(NUP) \
    {fac_adj_kernel<NUP, 16, 1, BATCH>, fac_adj_kernel<NUP, 16, 2, BATCH>, fac_adj_kernel<NUP, 20, 2, BATCH>, fac_adj_kernel<NUP, 24, 2, BATCH>}
    static constexpr Kernel fwd[4][4] = {FWD_ROW(64), FWD_ROW(128), FWD_ROW(192), FWD_ROW(256)};
    static constexpr Kernel adj[4][4] = {ADJ_ROW(64), ADJ_ROW(128), ADJ_ROW(192), ADJ_ROW(256)};
#undef FWD_ROW
#undef ADJ_ROW
    // tensor lines of 2 to 4 sums, at most 768 samples (what the registers hold), C = 32
#define NP_ROW(NUP) {fac_fwd_kernel<NUP, 16, 1, 2, BATCH>, fac_fwd_kernel<NUP, 16, 1, 3, BATCH>, fac_fwd_kernel<NUP, 16, 1, 4, BATCH>}
    static constexpr Kernel fwd_np[4][3] = {
        NP_ROW(64), NP_ROW(128), NP_ROW(192), {fac_fwd_kernel<256, 16, 1, 2, BATCH>, fac_fwd_kernel<256, 16, 1, 3, BATCH>, nullptr}};
#undef NP_ROW
    static constexpr Kernel adj_in[2] = {fac_adj_in_kernel<2, 4, BATCH>, fac_adj_in_kernel<3, 3, BATCH>};
    static constexpr Kernel fwd_out = fac_fwd_out_kernel<BATCH>;
};

int fac_zst_slot(int zst, int cj)
{
    if (cj == 1) return zst == 16 ? 0 : -1;
    return zst >= 16 && zst <= 24 && zst % 4 == 0 ? 1 + (zst - 16) / 4 : -1;
}

int fac_nup_slot(int nup)
{
    for (int i = 0; i < 4; ++i)
        if (kFacNups[i] == nup) return i;
    return -1;
}

}  // namespace

int fac_supported(int nup, int zst, int cj, int np)
{
    if (np > 1 && (np > 4 || cj != 1 || np * nup > 768)) return 0;
    return fac_nup_slot(nup) >= 0 && cj >= 1 && cj <= 2 && fac_zst_slot(zst, cj) >= 0;
}

static bool fac_args_ok(const FacBatch &b, int part)
{
    const FacArgs &a = b.a;
    if (b.njobs < 1 || b.njobs > kMaxFacJobs || a.P < 1 || a.cj < 1 || a.np < 1 || a.yc != 2 * a.zst || a.R > a.zst ||
        !(a.qmax == 32 ? a.R <= 2 * kInWaves : a.qmax == 24 && a.R <= 3 * kInWaves) || a.U < a.R || a.U > 2 * a.R ||
        a.ucols != 32 * a.U || a.nzstage != (a.P + 15) / 16 || !fac_supported(a.nup, a.zst, a.cj, a.np) ||
        a.adj_pitch != a.np * a.nup)
        return false;
    for (int i = 0; i < b.njobs; ++i) {
        const FacJob &j = b.jobs[i];
        if (j.row0 < 0 || j.row0 % 32 || j.row0 >= j.rows || j.rows - j.row0 > j.tiles * 32 || j.ylines < j.tiles * 32 || (long)(j.ylines + 1) * a.P * a.yc >= 0x7fffffffL ||
            j.nsplit < 1 || j.nsplit > a.P || j.nsplit_adj < 1 || j.nsplit_adj > a.P || j.psplit < 1 ||
            j.psplit > (a.P + 7) / 8 || j.zsplit < 1 || j.zsplit > a.nzstage)
            return false;
        if (a.np > 1 && part == kFacFwdInner && (j.in_stride != a.np * a.nup || (uintptr_t)j.in % 16)) return false;
    }
    return true;
}

// Grid of kernel `part` of one job.
static dim3 fac_grid(const FacArgs &a, const FacJob &j, int part)
{
    const int waves = fwd_waves(a.nup, a.np);
    switch (part) {
    case kFacFwdInner: return dim3((j.tiles + waves - 1) / waves * j.nsplit);
    case kFacFwdOuter: return dim3(out_groups(j.tiles), a.R, j.psplit);
    case kFacAdjOuter: return dim3(j.tiles, j.zsplit);
    default: return dim3((j.tiles + kFacWaves - 1) / kFacWaves * j.nsplit_adj, a.np);
    }
}

// LDS bytes of a line-tile kernel: three PSF-table stages and its residue
// table (nfrag fragments of 1 KB).
static size_t fac_lds(int nup, int np, int nfrag)
{
    return 1024 * (size_t)(3 * stage_chunks(nup, np) * (nup / 8) + nfrag);
}

template <bool BATCH>
static hipError_t launch_part(const Args<BATCH> &args, const FacArgs &a, int part, dim3 grid, hipStream_t st)
{
    using K = Kernels<BATCH>;
    typename K::Kernel k;
    int threads = 64 * kFacWaves;
    size_t lds = 0;
    switch (part) {
    case kFacFwdInner:
        k = a.np > 1 ? K::fwd_np[fac_nup_slot(a.nup)][a.np - 2] : K::fwd[fac_nup_slot(a.nup)][fac_zst_slot(a.zst, a.cj)];
        threads = 64 * fwd_waves(a.nup, a.np);
        lds = fac_lds(a.nup, a.np, a.cj * 4 * ((a.yc + 31) / 32));
        break;
    case kFacFwdOuter:
        k = K::fwd_out;
        threads = 64 * kOutWaves;
        break;
    case kFacAdjOuter:
        k = K::adj_in[a.qmax == 32 ? 0 : 1];
        threads = 64 * kInWaves;
        break;
    default:
        k = K::adj[fac_nup_slot(a.nup)][fac_zst_slot(a.zst, a.cj)];
        lds = fac_lds(a.nup, 1, a.cj * 2 * ((a.yc + 15) / 16));
        break;
    }
    if (lds > 64 * 1024) {
        const hipError_t e = hipFuncSetAttribute((const void *)k, hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds);
        if (e != hipSuccess) return e;
    }
    hipLaunchKernelGGL(k, grid, dim3(threads), lds, st, args);
    return hipGetLastError();
}

hipError_t launch_fac_part(FacBatch &b, int part, hipStream_t st)
{
    if (part < 0 || part > 3 || !fac_args_ok(b, part)) return hipErrorInvalidValue;
    if (b.njobs == 1) {
        b.a.job = b.jobs[0];
        return launch_part<false>(b.a, b.a, part, fac_grid(b.a, b.a.job, part), st);
    }
    int blocks = 0;
    for (int i = 0; i < b.njobs; ++i) {
        const dim3 g = fac_grid(b.a, b.jobs[i], part);
        b.jobs[i].blk0 = blocks;
        blocks += (int)(g.x * g.y * g.z);
    }
    return launch_part<true>(b, b.a, part, dim3(blocks), st);
}

hipError_t launch_fac_fwd(FacBatch &b, hipStream_t st)
{
    const hipError_t e = launch_fac_part(b, kFacFwdInner, st);
    return e == hipSuccess ? launch_fac_part(b, kFacFwdOuter, st) : e;
}

hipError_t launch_fac_adj(FacBatch &b, hipStream_t st)
{
    const hipError_t e = launch_fac_part(b, kFacAdjOuter, st);
    return e == hipSuccess ? launch_fac_part(b, kFacAdjInner, st) : e;
}

}  // namespace mpi3d
