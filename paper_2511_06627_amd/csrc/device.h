// Device helpers shared by the kernel sources (proj.hip, sig.hip, sig16.hip).
#pragma once

#include "internal.h"

namespace mpi3d {

typedef float f32x16 __attribute__((ext_vector_type(16)));
typedef _Float16 f16x8 __attribute__((ext_vector_type(8)));

#define MFMA16(a, b, c) __builtin_amdgcn_mfma_f32_32x32x16_f16((a), (b), (c), 0, 0, 0)

namespace {

// blockIdx -> logical block so that consecutive logical blocks share an XCD
// (blocks are dealt to the 8 XCDs round-robin; XCD x receives
// nblocks / 8 + (x < nblocks % 8) of them).
__device__ __forceinline__ int xcd_logical(int bid, int nblocks)
{
    const int nx = 8;
    int xcd = bid % nx, slot = bid / nx;
    int per = nblocks / nx, rem = nblocks % nx;
    return xcd * per + min(xcd, rem) + slot;
}

// Where a signal-kernel block and wave sit: the block covers a.pairs *
// kRowsPerWave lines (a tile) of one job, for one time split and one column
// group; wave w is half w & 1 of pair w >> 1, which owns kRowsPerWave lines
// from row0.
struct BlockPos {
    int job, row0, split, group, half, pair;
};

__device__ __forceinline__ BlockPos locate(const SigArgs &a)
{
    BlockPos bp;
    const int lb = xcd_logical(blockIdx.x, gridDim.x);
    const int tile = lb % a.total_tiles;
    const int sg = lb / a.total_tiles;
    bp.group = sg % a.ngroups;
    bp.split = sg / a.ngroups;
    int jb = 0;
    for (int j = 1; j < a.njobs; ++j)
        if (tile >= a.jobs[j].tile0) jb = j;
    bp.job = jb;
    const int w = threadIdx.x >> 6;
    bp.pair = w >> 1;
    bp.half = w & 1;
    bp.row0 = (tile - a.jobs[jb].tile0) * (a.pairs * kRowsPerWave) + bp.pair * kRowsPerWave;
    return bp;
}

// The work of an FP32 signal-kernel block: tiles tile0 .. tile0 + ntiles - 1
// of column group `group` over time chunks [c0, c1), written to partial-sum
// slot `slot`.  The first total_tiles x main splits x ngroups logical blocks
// take one tile and one split of cps chunks each; with a tail (tail_c0 > 0,
// the main splits covering [0, tail_c0)), the remaining blocks take tail_tpb
// tiles each over [tail_c0, nchunks) into the last slot, so every block does
// about the same number of chunks on 256 CUs.
struct BlockWork {
    int tile0, ntiles, group, slot, c0, c1;
};

__device__ __forceinline__ BlockWork block_work(const SigArgs &a)
{
    BlockWork w;
    const int lb = xcd_logical(blockIdx.x, gridDim.x);
    const int msplit = a.tail_c0 > 0 ? a.nsplit - 1 : a.nsplit;
    const int nmain = a.total_tiles * msplit * a.ngroups;
    if (lb < nmain) {
        w.tile0 = lb % a.total_tiles;
        w.ntiles = 1;
        const int sg = lb / a.total_tiles;
        w.group = sg % a.ngroups;
        w.slot = sg / a.ngroups;
        w.c0 = w.slot * a.cps;
        w.c1 = min(w.c0 + a.cps, a.tail_c0 > 0 ? a.tail_c0 : a.nchunks);
    } else {
        const int tb = lb - nmain;
        w.group = tb % a.ngroups;
        w.tile0 = (tb / a.ngroups) * a.tail_tpb;
        w.ntiles = min(a.tail_tpb, a.total_tiles - w.tile0);
        w.slot = msplit;
        w.c0 = a.tail_c0;
        w.c1 = a.nchunks;
    }
    return w;
}

// The position of this wave in tile `tile` (see locate).
__device__ __forceinline__ BlockPos tile_pos(const SigArgs &a, int tile, int slot, int group)
{
    BlockPos bp;
    bp.group = group;
    bp.split = slot;
    int jb = 0;
    for (int j = 1; j < a.njobs; ++j)
        if (tile >= a.jobs[j].tile0) jb = j;
    bp.job = jb;
    const int w = threadIdx.x >> 6;
    bp.pair = w >> 1;
    bp.half = w & 1;
    bp.row0 = (tile - a.jobs[jb].tile0) * (a.pairs * kRowsPerWave) + bp.pair * kRowsPerWave;
    return bp;
}

// Swap partial time tiles within a pair: write mine, barrier, read the
// partner's, and return lo + hi (the same operand order on both waves).  xs
// holds two parities x PAIRS pairs x 2 halves x 16 x 64 floats.
template <int PAIRS>
__device__ __forceinline__ f32x16 pair_sum(float *xs, int parity, int pair, int half, int lane, const f32x16 &mine)
{
    // 16-byte words, word q of lane l at q * 64 + l: four 128-bit LDS
    // accesses each way, consecutive lanes on consecutive words
    typedef float f32x4v __attribute__((ext_vector_type(4)));
    f32x4v *slot = reinterpret_cast<f32x4v *>(xs) + ((parity * PAIRS + pair) * 2) * 4 * 64;
    f32x4v *own = slot + half * 4 * 64;
    const f32x4v *other = slot + (1 - half) * 4 * 64;
#pragma unroll
    for (int q = 0; q < 4; ++q) own[q * 64 + lane] = f32x4v{mine[4 * q], mine[4 * q + 1], mine[4 * q + 2], mine[4 * q + 3]};
    __syncthreads();
    f32x16 r;
#pragma unroll
    for (int q = 0; q < 4; ++q) {
        const f32x4v o = other[q * 64 + lane];
#pragma unroll
        for (int e = 0; e < 4; ++e) r[4 * q + e] = half == 0 ? mine[4 * q + e] + o[e] : o[e] + mine[4 * q + e];
    }
    return r;
}

// N result tiles' rows row0 + 8 (j / 4) + j % 4 to lines of `pitch` floats, a row
// at a time: one branch a row, not one a value (with the line loads left
// unguarded and the first tile waiting for its own slice alone: fp16 forward at
// 128 x 128 x 64, 24 angles 23.9 -> 21.7 us, at 192 x 192 x 96, 36 62 -> 60).
template <int N>
__device__ __forceinline__ void store_rows(const SigJob &job, int row0, int pitch, float *out, const f32x16 (&v)[N])
{
#pragma unroll
    for (int j = 0; j < 16; ++j) {
        const int row = row0 + 8 * (j / 4) + j % 4;
        if (row < job.rows) {
            float *o = out + (size_t)job_line(job, row) * pitch;
#pragma unroll
            for (int g = 0; g < N; ++g) o[g * 32] = v[g][j];
        }
    }
}

// bf16 bits of v, rounded to nearest even
__device__ __forceinline__ uint16_t bf16_bits(float v)
{
    uint32_t u = __float_as_uint(v);
    u += 0x7fffu + ((u >> 16) & 1u);
    return (uint16_t)(u >> 16);
}

// N products whose table operands come from LDS: fragment j is read WIN
// products ahead of its use, and a scheduling barrier after every product
// keeps that distance.
template <int N, int WIN, class Frag, class Prod>
__device__ __forceinline__ void lds_pipelined(Frag frag, Prod prod)
{
    constexpr int W = WIN < N ? WIN : N;
    f16x8 w[W];
#pragma unroll
    for (int j = 0; j < W; ++j) w[j] = frag(j);
#pragma unroll
    for (int j = 0; j < N; ++j) {
        const f16x8 f = w[j % W];
        if (j + W < N) w[j % W] = frag(j + W);
        prod(j, f);
        __builtin_amdgcn_sched_barrier(0);
    }
}

// A float as the sum of two fp16 values: hi = rn16(v), lo = rn16(v - hi).
// With |v| <= 2^15 the pair holds v to 2^-23 relative down to |v| = 2^-3 and
// to an absolute 2^-25 below (2^-40 of the largest value), so a product taken
// as hi hi + hi lo + lo hi drops only lo lo, 2^-22 of it at most.
__device__ __forceinline__ void split8(const float (&v)[8], f16x8 &hi, f16x8 &lo)
{
#pragma unroll
    for (int e = 0; e < 8; ++e) hi[e] = (_Float16)v[e];
#pragma unroll
    for (int e = 0; e < 8; ++e) lo[e] = (_Float16)(v[e] - (float)hi[e]);
}

// The exponent e that brings a line of largest magnitude m into [2^14, 2^15)
// (0 for a line of zeros or with a non-finite entry).
__device__ __forceinline__ int line_exponent(float m)
{
    return m > 0.f && m < __builtin_inff() ? 15 - __builtin_amdgcn_frexp_expf(m) : 0;
}

// The fp16 matrix instructions round their fp32 sums down, towards minus
// infinity, so a long chain leaves every sum a little low, alike in all lines: at
// 256 x 256 x 128 the adjoint's lines by 9e-8 of their size, which the
// backprojection adds up over the angles (8.1e-7 of its result, where the chains'
// other roundings leave 3.3e-7).  So half of the chains run on negated operands
// and their sums are negated back: this sign, by time range and line tile.
__device__ __forceinline__ float chain_sign(int split, int tile)
{
    return (split + __builtin_popcount(tile)) & 1 ? -1.f : 1.f;
}

// s_waitcnt vmcnt(n) lgkmcnt(0) (expcnt not waited for), n < 64
template <int N>
__device__ __forceinline__ void wait_vm_lgkm()
{
    static_assert(N >= 0 && N < 64, "vmcnt range");
    __builtin_amdgcn_s_waitcnt((N & 15) | (7 << 4) | ((N >> 4) << 14));
}

__device__ __forceinline__ void block_barrier_nofence() { asm volatile("s_barrier" ::: "memory"); }

// 16 bytes a lane from byte voff + soff of the buffer rs to LDS at dst + 16 lane
// (soff and dst wave-uniform).
__device__ __forceinline__ void buffer_dma16(__amdgpu_buffer_rsrc_t rs, void *dst, int voff, int soff)
{
    __builtin_amdgcn_raw_ptr_buffer_load_lds(rs, (__attribute__((address_space(3))) void *)dst, 16, voff, soff, 0, 0);
}

// A raw buffer of `bytes` bytes at p (reads past it return 0).
__device__ __forceinline__ __amdgpu_buffer_rsrc_t buffer_table(const void *p, int bytes)
{
    return __builtin_amdgcn_make_buffer_rsrc(const_cast<void *>(p), 0, bytes, 0x00020000);
}

}  // namespace

}  // namespace mpi3d
