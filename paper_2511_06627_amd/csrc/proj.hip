// Parallel-beam projection P_theta and its transpose on gfx950.
//
// Forward (Sec. 2.2, eq. ptheta2 / eq. ptheta1): for FFL angle m, z-slice k
// and detector sample p,
//   rho_theta[m][k][p] = sum_q bilerp(x[k]; u_p cos t + y_q sin t, -u_p sin t + y_q cos t)
// with unit-step ray samples y_q and zero outside the grid.
//
//   One block = one z-slice and a group of angles.  The slice is staged in
//   LDS with a one-voxel zero border (a band of rows at a time when a whole
//   slice does not fit in 160 KB), read once from HBM with coalesced row
//   loads and reused by every ray of every angle in the group.  Each thread
//   owns a few rays and walks the exact range of samples that fall in the
//   staged band, so no sample is read outside the tile and no ray sum needs
//   a cross-thread reduction.
//
// Adjoint (exact transpose, gather form, no atomics): every voxel collects,
// for each angle, the bilinear weights of the <= 3 x 3 ray samples whose
// 2x2 footprint covers it -- the same weights the forward pass uses --
// summed per ray into <= 3 ray weights.  Those weights do not depend on z,
// so one block covers a 16x16 voxel tile for a group of kz slices and reuses
// the weights kz times; the projections it needs for one angle (kz lines x
// <= 32 rays) are staged in LDS.  The epilogue optionally forms
// out = acc + x_add - lambda * x_sub and a float64 partial sum of out^2 (CGLS).

#include <algorithm>
#include <type_traits>

#include "device.h"

namespace mpi3d {

namespace {

// A ray sample's 2x2 footprint is the same in every z-slice, so a unit of
// work may cover NS consecutive slices k0 .. k0 + NS - 1 whose values share
// one staged texel (LDS column col = grid column col - 1): every address and
// bilinear weight is then formed once for all of them.  Texel types:
//  float    fp32, one slice;
//  float2   fp32, two slices {x[k0], x[k0 + 1]} (when a slice pair fits in LDS
//           in one band: row bands split the rays of a wave unevenly);
//  uint32_t bf16 (the mixed operator's gathers), two slices: low half the
//           bf16 voxel of k0, high half that of k0 + 1.
// A missing last slice (odd nz) is staged as zeros and never stored.
template <typename T>
struct Texel;
template <>
struct Texel<float> {
    static constexpr int NS = 1;
    using V = float;
};
template <>
struct Texel<float2> {
    static constexpr int NS = 2;
    using V = float;
};
template <>
struct Texel<uint32_t> {
    static constexpr int NS = 2;
    using V = uint16_t;
};

__device__ __forceinline__ void load(const float *p, float (&v)[1]) { v[0] = *p; }

__device__ __forceinline__ void load(const float2 *p, float (&v)[2])
{
    const float2 q = *p;
    v[0] = q.x;
    v[1] = q.y;
}

__device__ __forceinline__ void load(const uint32_t *p, float (&v)[2])
{
    const uint32_t w = *p;
    v[0] = __uint_as_float(w << 16);
    v[1] = __uint_as_float(w & 0xffff0000u);
}

// The 2x2 footprint whose corner (0,0) is the texel at p: t[0] = (0,0),
// t[1] = (1,0), t[2] = (0,1), t[3] = (1,1).
template <typename T, int NS>
__device__ __forceinline__ void fetch(const T *p, int W, float (&t)[4][NS])
{
    load(p, t[0]);
    load(p + 1, t[1]);
    load(p + W, t[2]);
    load(p + W + 1, t[3]);
}

// Staging.  LDS row r of a band holds grid row jb0 + r and LDS column col
// holds grid column col - 1; columns 0 and nx + 1 .. W - 1 are zero borders,
// written once per block.  A thread stages runs of VW consecutive voxels of
// one row (VW = 4 where every row start is aligned to a VW-voxel vector load,
// else 1), U runs at a time with all their global loads issued before the
// first LDS store: a band then costs a few memory latencies, not one per
// texel.
template <typename V, int VW>
struct Run {
    V v[VW];
};

template <typename V, int VW>
__device__ __forceinline__ Run<V, VW> load_run(const V *p)
{
    Run<V, VW> r;
    if constexpr (VW == 1) {
        r.v[0] = *p;
    } else {
        typedef V vec __attribute__((ext_vector_type(VW)));
        const vec q = *reinterpret_cast<const vec *>(p);
#pragma unroll
        for (int j = 0; j < VW; ++j) r.v[j] = q[j];
    }
    return r;
}

// The texel of voxel j of the runs a (slice k0) and b (slice k0 + 1); a
// run not in the grid (ia / ib false) contributes zeros.
template <typename T, typename V, int VW>
__device__ __forceinline__ T make_texel(const Run<V, VW> &ra, const Run<V, VW> &rb, bool ia, bool ib, int j)
{
    if constexpr (std::is_same_v<T, float>) {
        return ia ? ra.v[j] : 0.f;
    } else if constexpr (std::is_same_v<T, float2>) {
        return make_float2(ia ? ra.v[j] : 0.f, ib ? rb.v[j] : 0.f);
    } else {
        return (ia ? (uint32_t)ra.v[j] : 0u) | ((ib ? (uint32_t)rb.v[j] : 0u) << 16);
    }
}

// Stages LDS rows 0 .. rows - 1 (grid rows jb0 ..) of the slice group (s0,
// s1; s1 is read only where has1), LDS columns 1 .. nx.  Thread tid starts
// at run (r0, c0) of the row-major run order and steps by kFwdThreads runs,
// (dr, dc) rows and runs at a time.
template <typename T, int VW, int U>
__device__ __forceinline__ void stage_band(T *lds, const typename Texel<T>::V *s0, const typename Texel<T>::V *s1,
                                           bool has1, int nx, int ny, int W, int jb0, int rows, int r0, int c0,
                                           int dr, int dc, int tid)
{
    using V = typename Texel<T>::V;
    constexpr int NS = Texel<T>::NS;
    const int runs = nx / VW;
    const int total = rows * runs;
    int r = r0, c = c0;
    for (int e0 = tid; e0 < total; e0 += U * kFwdThreads) {
        Run<V, VW> ra[U], rb[U];
        int dst[U];
        bool in[U];
#pragma unroll
        for (int u = 0; u < U; ++u) {
            const int gj = jb0 + r;
            const bool live = e0 + u * kFwdThreads < total;
            in[u] = live && (unsigned)gj < (unsigned)ny;
            // out-of-grid runs load row 0 of the slice (in bounds) and are dropped
            const size_t off = (size_t)(in[u] ? gj : 0) * nx + (size_t)c * VW;
            ra[u] = load_run<V, VW>(s0 + off);
            if constexpr (NS == 2) rb[u] = load_run<V, VW>((has1 ? s1 : s0) + off);
            dst[u] = live ? r * W + 1 + c * VW : -1;
            c += dc;
            r += dr;
            if (c >= runs) {
                c -= runs;
                ++r;
            }
        }
#pragma unroll
        for (int u = 0; u < U; ++u) {
            if (dst[u] < 0) continue;
#pragma unroll
            for (int j = 0; j < VW; ++j) lds[dst[u] + j] = make_texel<T, V, VW>(ra[u], rb[u], in[u], in[u] && has1, j);
        }
    }
}

// Adds the bilinear interpolant of the footprint t at fractional offsets
// (wx, wy) to acc.  One slice: the three-lerp form.  Two slices: the corner
// weights (1-wx)(1-wy), wx(1-wy), (1-wx)wy, wx wy, formed once in five
// operations and shared.
template <int NS>
__device__ __forceinline__ void accum(float (&acc)[NS], const float (&t)[4][NS], float wx, float wy)
{
    if constexpr (NS == 1) {
        const float top = fmaf(wx, t[1][0] - t[0][0], t[0][0]);
        const float bot = fmaf(wx, t[3][0] - t[2][0], t[2][0]);
        acc[0] += fmaf(wy, bot - top, top);
    } else {
        const float w11 = wx * wy, w10 = wx - w11, w01 = wy - w11, w00 = (1.f - wx) - w01;
#pragma unroll
        for (int k = 0; k < NS; ++k) {
            acc[k] = fmaf(t[0][k], w00, acc[k]);
            acc[k] = fmaf(t[1][k], w10, acc[k]);
            acc[k] = fmaf(t[2][k], w01, acc[k]);
            acc[k] = fmaf(t[3][k], w11, acc[k]);
        }
    }
}

// One bilinear sample of the staged band, tested.  Branch-free: a sample whose
// 2x2 footprint lies outside the band reads a safe LDS address with zero
// weights.
template <typename T, int NS>
__device__ __forceinline__ void sample(const T *lds, int W, int nx, int nbase, int jb0, float bx, float by, float s,
                                       float c, float y, float (&acc)[NS])
{
    const float fx = fmaf(y, s, bx), fy = fmaf(y, c, by);
    const float ix = floorf(fx), iy = floorf(fy);
    int i0 = (int)ix, j0 = (int)iy - jb0;
    const bool ok = (unsigned)i0 <= (unsigned)nx && (unsigned)j0 < (unsigned)nbase;
    i0 = ok ? i0 : 0;
    j0 = ok ? j0 : 0;
    float t[4][NS];
    fetch(lds + j0 * W + i0, W, t);
    float v[NS];
#pragma unroll
    for (int k = 0; k < NS; ++k) v[k] = 0.f;
    accum(v, t, fx - ix, fy - iy);
#pragma unroll
    for (int k = 0; k < NS; ++k) acc[k] += ok ? v[k] : 0.f;
}

// Samples known to lie kEdge inside the staged band need no test: there fx
// (in LDS columns) and fyb (in band rows) are positive, so floor is the
// truncating conversion of the value and the fraction is fract().
constexpr float kEdge = 1.0f / 64.0f;
constexpr float kRange = 1.0f / 1024.0f;

// The texel at (column fx, band row fyb), both positive.  Wb = W * sizeof(T).
template <typename T>
__device__ __forceinline__ const T *texel_at(const T *lds, unsigned Wb, float fx, float fyb)
{
    const unsigned off = __umul24((unsigned)fyb, Wb) + (unsigned)fx * (unsigned)sizeof(T);
    return reinterpret_cast<const T *>(reinterpret_cast<const unsigned char *>(lds) + off);
}

// Four consecutive interior samples y, y+1, y+2, y+3: all LDS reads are
// issued before any is used.
template <typename T, int NS>
__device__ __forceinline__ void sample_in4(const T *lds, int W, unsigned Wb, float bx, float byb, float s, float c,
                                           float y, float (&acc)[NS])
{
    float wx[4], wy[4];
    const T *p[4];
#pragma unroll
    for (int j = 0; j < 4; ++j) {
        const float fx = fmaf(y + (float)j, s, bx), fy = fmaf(y + (float)j, c, byb);
        wx[j] = __builtin_amdgcn_fractf(fx);
        wy[j] = __builtin_amdgcn_fractf(fy);
        p[j] = texel_at(lds, Wb, fx, fy);
    }
    float t[4][4][NS];
#pragma unroll
    for (int j = 0; j < 4; ++j) fetch(p[j], W, t[j]);
#pragma unroll
    for (int j = 0; j < 4; ++j) accum(acc, t[j], wx[j], wy[j]);
}

template <typename T, int NS>
__device__ __forceinline__ void sample_in(const T *lds, int W, unsigned Wb, float bx, float byb, float s, float c,
                                          float y, float (&acc)[NS])
{
    const float fx = fmaf(y, s, bx), fy = fmaf(y, c, byb);
    float t[4][NS];
    fetch(texel_at(lds, Wb, fx, fy), W, t);
    accum(acc, t, __builtin_amdgcn_fractf(fx), __builtin_amdgcn_fractf(fy));
}

// T: the texel type above; weights and sums are fp32.
template <typename T>
__global__ __launch_bounds__(kFwdThreads) void proj_fwd_kernel(ProjArgs a, const typename Texel<T>::V *vol,
                                                               int out_stride)
{
    using V = typename Texel<T>::V;
    constexpr int NS = Texel<T>::NS;
    constexpr int kMaxRaysPerThread = fwd_rays_per_thread(NS);
    extern __shared__ __align__(16) unsigned char lds_raw[];
    T *lds = reinterpret_cast<T *>(lds_raw);
    const int nb = gridDim.x;
    const int lb = xcd_logical(blockIdx.x, nb);
    // The (slice group, angle) units g * M + m are dealt to the blocks in equal
    // contiguous ranges: a block stages each slice group its range touches
    // once and projects that group for its angles there.
    const int ng = (a.nz + NS - 1) / NS;
    const long U = (long)ng * a.M;
    const long u0 = (long)lb * U / nb, u1 = (long)(lb + 1) * U / nb;
    const int W = proj_pitch(a.nx);
    const unsigned Wb = (unsigned)(W * sizeof(T));
    const int tid = threadIdx.x;
    // zero borders of every LDS row a band uses
    const int border = W - a.nx;
    for (int idx = tid; idx < (a.band_rows + 1) * border; idx += kFwdThreads) {
        const int r = idx / border, b = idx - r * border;
        lds[r * W + (b == 0 ? 0 : a.nx + b)] = T{};
    }
    // run positions of this thread for the vector (4 voxels) and scalar stagings
    const bool vec = a.nx % 4 == 0 && reinterpret_cast<uintptr_t>(vol) % (4 * sizeof(V)) == 0;
    const int v_runs = max(1, a.nx / 4), s_runs = a.nx;
    const int v_r0 = tid / v_runs, v_c0 = tid - v_r0 * v_runs, v_dr = kFwdThreads / v_runs,
              v_dc = kFwdThreads - v_dr * v_runs;
    const int s_r0 = tid / s_runs, s_c0 = tid - s_r0 * s_runs, s_dr = kFwdThreads / s_runs,
              s_dc = kFwdThreads - s_dr * s_runs;
    for (long ku = u0; ku < u1;) {
        const int g = (int)(ku / a.M);
        const int m0 = (int)(ku - (long)g * a.M);
        const int m1 = (int)min((long)a.M, u1 - (long)g * a.M);
        ku = (long)g * a.M + m1;
        const int k0 = NS * g;
        const int ns = min(NS, a.nz - k0);     // slices present in the group
        const int nrays = (m1 - m0) * a.nu;
        float acc[kMaxRaysPerThread][NS];
#pragma unroll
        for (int r = 0; r < kMaxRaysPerThread; ++r)
#pragma unroll
            for (int k = 0; k < NS; ++k) acc[r][k] = 0.f;
        const V *s0 = vol + (size_t)k0 * a.nx * a.ny;
        const V *s1 = s0 + (size_t)(ns > 1 ? a.nx * a.ny : 0);
        for (int band = 0; band < a.n_bands; ++band) {
            const int jb0 = -1 + band * a.band_rows;               // first base row
            const int jb1 = min(jb0 + a.band_rows, a.ny);          // one past last base row
            const int nbase = jb1 - jb0;
            const int rows = nbase + 1;                            // LDS rows: grid rows jb0..jb1
            __syncthreads();
            if (vec)
                stage_band<T, 4, (NS == 2 && sizeof(V) == 4 ? 4 : 8)>(lds, s0, s1, ns > 1, a.nx, a.ny, W, jb0, rows,
                                                                       v_r0, v_c0, v_dr, v_dc, tid);
            else
                stage_band<T, 1, 8>(lds, s0, s1, ns > 1, a.nx, a.ny, W, jb0, rows, s_r0, s_c0, s_dr, s_dc, tid);
            __syncthreads();
#pragma unroll
            for (int i = 0; i < kMaxRaysPerThread; ++i) {
                const int ray = tid + kFwdThreads * i;
                if (ray >= nrays) continue;
                const int m = m0 + ray / a.nu, p = ray % a.nu;
                const float2 csv = a.cs[m];
                // samples lie symmetrically on a ray, so it is walked with sin >= 0
                // (both signs in the bounds below cost 3% at 490 x 793 x 15, 6 angles)
                const float c = csv.y < 0.f ? -csv.x : csv.x, s = fabsf(csv.y);
                const float bx = a.ax[(size_t)m * a.nu + p];
                const float by = a.ay[(size_t)m * a.nu + p];
                // sample coordinates: fx = bx + y s in LDS columns (column 0 is grid
                // column -1), fy = by + y c in grid rows, y = q - (nr-1)/2.  A sample
                // belongs to this band when its base row floor(fy) is in [jb0, jb1);
                // fy does not depend on the band, so every sample lands in exactly
                // one band.  Samples with floor(fx) outside [0, nx] touch no voxel.
                // [q0, q1] is a widened superset of the samples in the band (each
                // checked exactly): the edges are moved out by kRange in fx and fy,
                // beyond the rounding of fx and fy themselves, so a ray that runs
                // along a band edge (|c| tiny, fy rounding onto the edge row) keeps
                // all its samples; inside it, [qa, qb] holds samples at least kEdge
                // away from every edge in both coordinates, which need no test:
                // there the band-relative row fy - jb0 lies in [kEdge, nbase - kEdge]
                // and fx in [kEdge, nx + 1 - kEdge].  The bounds are solved with one
                // reciprocal per direction; its relative error (a few ulp, so below
                // 1e-4 samples over any ray) is far inside both margins.
                const float byb = by - (float)jb0;
                float ylo = -a.half_nr, yhi = a.half_nr;
                float ilo = -a.half_nr, ihi = a.half_nr;
                if (s > 0.f) {
                    const float rs = 1.f / s;
                    ylo = fmaxf(ylo, (-kRange - bx) * rs);
                    yhi = fminf(yhi, ((float)(a.nx + 1) + kRange - bx) * rs);
                    ilo = fmaxf(ilo, (kEdge - bx) * rs);
                    ihi = fminf(ihi, ((float)(a.nx + 1) - kEdge - bx) * rs);
                } else if (bx < kEdge || bx > (float)(a.nx + 1) - kEdge) {
                    ihi = ilo - 2.f;
                }
                if (c != 0.f) {
                    const float rc = 1.f / c;
                    const float e0 = ((float)jb0 - kRange - by) * rc, e1 = ((float)jb1 + kRange - by) * rc;
                    const float i0 = (kEdge - byb) * rc, i1 = ((float)nbase - kEdge - byb) * rc;
                    ylo = fmaxf(ylo, fminf(e0, e1));
                    yhi = fminf(yhi, fmaxf(e0, e1));
                    ilo = fmaxf(ilo, fminf(i0, i1));
                    ihi = fminf(ihi, fmaxf(i0, i1));
                } else if (byb < kEdge || byb > (float)nbase - kEdge) {
                    ihi = ilo - 2.f;
                }
                const int q0 = max(0, (int)floorf(ylo + a.half_nr) - 1);
                const int q1 = min(a.nr - 1, (int)ceilf(yhi + a.half_nr) + 1);
                int qa = max(q0, (int)ceilf(ilo + a.half_nr));
                int qb = min(q1, (int)floorf(ihi + a.half_nr));
                if (qa > qb) {   // no interior: every sample checked
                    qa = q1 + 1;
                    qb = q1;
                }
                float sa[NS], sb[NS];
#pragma unroll
                for (int k = 0; k < NS; ++k) sa[k] = sb[k] = 0.f;
                for (int q = q0; q < qa; ++q) sample(lds, W, a.nx, nbase, jb0, bx, by, s, c, (float)q - a.half_nr, sa);
                // interior, four samples at a time with their LDS reads in flight together
                int q = qa;
                for (; q + 3 <= qb; q += 4) sample_in4(lds, W, Wb, bx, byb, s, c, (float)q - a.half_nr, sb);
                for (; q <= qb; ++q) sample_in(lds, W, Wb, bx, byb, s, c, (float)q - a.half_nr, sb);
                for (q = max(qb + 1, qa); q <= q1; ++q)
                    sample(lds, W, a.nx, nbase, jb0, bx, by, s, c, (float)q - a.half_nr, sa);
#pragma unroll
                for (int k = 0; k < NS; ++k) acc[i][k] += sa[k] + sb[k];
            }
        }
#pragma unroll
        for (int i = 0; i < kMaxRaysPerThread; ++i) {
            const int ray = tid + kFwdThreads * i;
            if (ray >= nrays) continue;
            const int m = m0 + ray / a.nu, p = ray % a.nu;
            float *o = a.rt + ((size_t)m * a.nz + k0) * out_stride + p;
#pragma unroll
            for (int k = 0; k < NS; ++k)
                if (k < ns) o[(size_t)k * out_stride] = acc[i][k];
        }
        // zero the padding columns of the lines this block owns
        if (out_stride > a.nu) {
            const int pad = out_stride - a.nu;
            const int nl = (m1 - m0) * ns;
            for (int idx = tid; idx < nl * pad; idx += kFwdThreads) {
                const int l = idx / pad;
                const int m = m0 + l / ns, k = k0 + l % ns, p = a.nu + idx % pad;
                a.rt[((size_t)m * a.nz + k) * out_stride + p] = 0.f;
            }
        }
    }
}

// ---------------------------------------------------------------------------
// Forward projection, four slices a texel.  The kernel above spends most of
// its time forming each sample's address and weights (about 16 vector
// operations a sample and slice); a texel of four consecutive slices shares
// them four ways and one 16-byte LDS read serves a corner of all four, which
// leaves about 8.  160 KB then hold a band of the slice group only, so
//  - angles are taken in two classes, dealt apart: steep ones (|c| >= |s|)
//    with bands of rows, the others with bands of columns.  Every ray then
//    crosses every band at 45 degrees or more, in about the same number of
//    samples, and no wave idles while others work;
//  - a ray's samples in a band, and those inside the grid, are found exactly:
//    sample coordinates are monotone in the sample number, so the first sample
//    past a threshold is its estimate or a neighbour, decided by the sample's
//    own coordinate.  The samples of a range then need no test: their base
//    texel and its right and lower neighbours lie in the staged band.
// Coordinates are shifted by one (index 0 is the zero border), so truncation
// is floor.  What bounds it: vector work (about 80% busy; 17 of 34 operations a
// sample are address and weights) and the LDS reads, half of whose cycles are
// bank conflicts (16 lanes read over up to 23 texels, so two share a bank
// whatever the pitch).  Measured 432 -> 240 us at 256 x 256 x 128, 60 angles;
// 285 -> 127 us at 224 x 224 x 112, 48; 82 -> 71 us at 192 x 192 x 96, 36.
// The mixed operator's gathers (bf16 values, widened as they are staged; no
// bf16 copy where the caller has none) against row bands of its slice pairs:
// 385 -> 209 us, 242 -> 130, 97 -> 78 at 256 x 256 x 64, 24.
// ---------------------------------------------------------------------------
constexpr int kBandRays = 2;                     // rays a thread owns
constexpr int kBandSlices = 4;
constexpr int kBandTexels = 160 * 1024 / 16;     // LDS texels

// Sample q's coordinate on an axis: b + y_q k, as the sampling loop forms it.
__device__ __forceinline__ float coord(int q, float half_nr, float k, float b) { return fmaf((float)q - half_nr, k, b); }

// The first sample q of [0, nr] from which the coordinate is at least t (k > 0)
// or below t (k < 0).  |k| >= 1e-3: the estimate is within 0.1 of the real
// crossing, so the sample is the estimate or a neighbour; below that (rays
// along a grid axis) by bisection.
__device__ __forceinline__ int first_past(float t, int nr, float half_nr, float k, float rk, float b)
{
    const bool up = k > 0.f;
    auto past = [&](int q) {
        const float f = coord(q, half_nr, k, b);
        return up ? f >= t : f < t;
    };
    if (fabsf(k) >= 1e-3f) {
        const float e = fminf(fmaxf(ceilf((t - b) * rk + half_nr), 0.f), (float)nr);
        int q = (int)e;
        if (q > 0 && past(q - 1))
            --q;
        else if (q < nr && !past(q))
            ++q;
        return q;
    }
    int lo = 0, hi = nr;                         // past(hi - 1) or hi = nr; not past(lo - 1)
    while (lo < hi) {
        const int mid = (lo + hi) >> 1;
        if (past(mid))
            hi = mid;
        else
            lo = mid + 1;
    }
    return lo;
}

// The samples [q0, q1) whose coordinate is in [lo, hi).
__device__ __forceinline__ void samples_in(float lo, float hi, int nr, float half_nr, float k, float rk, float b,
                                           int &q0, int &q1)
{
    if (k == 0.f) {
        q0 = 0;
        q1 = b >= lo && b < hi ? nr : 0;
    } else {
        q0 = first_past(k > 0.f ? lo : hi, nr, half_nr, k, rk, b);
        q1 = first_past(k > 0.f ? hi : lo, nr, half_nr, k, rk, b);
    }
}

// Two consecutive samples: their corners' texels, read one pair ahead of
// their use, and weights.
struct SamplePair {
    float4 t[2][4];
    float wx[2], wy[2];
};

// Samples at coordinate numbers y and y + 1, no further than ylast.
__device__ __forceinline__ void pair_load(SamplePair &g, const unsigned char *lds, unsigned base, unsigned Wb, float bx,
                                          float by, float s, float c, float y, float ylast)
{
#pragma unroll
    for (int j = 0; j < 2; ++j) {
        const float yj = fminf(y + (float)j, ylast);
        const float fx = fmaf(yj, s, bx), fy = fmaf(yj, c, by);
        g.wx[j] = __builtin_amdgcn_fractf(fx);
        g.wy[j] = __builtin_amdgcn_fractf(fy);
        const unsigned o = __umul24((unsigned)fy, Wb) + base + (unsigned)fx * 16u;
        g.t[j][0] = *reinterpret_cast<const float4 *>(lds + o);
        g.t[j][1] = *reinterpret_cast<const float4 *>(lds + o + 16);
        g.t[j][2] = *reinterpret_cast<const float4 *>(lds + o + Wb);
        g.t[j][3] = *reinterpret_cast<const float4 *>(lds + o + Wb + 16);
    }
    __builtin_amdgcn_sched_barrier(0);
}

// Their interpolants, summed before they join the ray's sum: the long sum is
// then rounded once a pair, not once a corner.
template <int N>
__device__ __forceinline__ void pair_sum(const SamplePair &g, float (&acc)[kBandSlices])
{
    float v[kBandSlices];
#pragma unroll
    for (int j = 0; j < N; ++j) {
        const float w11 = g.wx[j] * g.wy[j], w10 = g.wx[j] - w11, w01 = g.wy[j] - w11, w00 = (1.f - g.wx[j]) - w01;
        const float w[4] = {w00, w10, w01, w11};
#pragma unroll
        for (int k = 0; k < 4; ++k) {
            const float4 t = g.t[j][k];
            const bool first = j == 0 && k == 0;
            v[0] = first ? t.x * w[k] : fmaf(t.x, w[k], v[0]);
            v[1] = first ? t.y * w[k] : fmaf(t.y, w[k], v[1]);
            v[2] = first ? t.z * w[k] : fmaf(t.z, w[k], v[2]);
            v[3] = first ? t.w * w[k] : fmaf(t.w, w[k], v[3]);
        }
    }
#pragma unroll
    for (int k = 0; k < kBandSlices; ++k) acc[k] += v[k];
    __builtin_amdgcn_sched_barrier(0);
}

// A staged value: the volume's, its bf16 copy's, or (Round16) the volume's
// rounded to bf16 as that copy would be.
struct Round16 {
    float v;
};
__device__ __forceinline__ float staged(float v) { return v; }
__device__ __forceinline__ float staged(uint16_t v) { return __uint_as_float((uint32_t)v << 16); }
__device__ __forceinline__ float staged(Round16 v) { return staged(bf16_bits(v.v)); }

// Stages LDS rows 0 .. rows - 1 of cols texels (grid rows j0 + r - 1, grid
// columns i0 + c - 1; zeros outside the grid and past the last slice).
template <class V>
__device__ __forceinline__ void stage_band4(float4 *lds, const V *vol, int k0, const ProjArgs &a, int j0, int i0,
                                            int rows, int cols, int W, int tid)
{
    constexpr int U = 10;      // a full band (10240 texels) in one round of loads
    const int total = rows * cols;
    const size_t slice = (size_t)a.nx * a.ny;
    const int ns = min(kBandSlices, a.nz - k0);
    const V *v0 = vol + (size_t)k0 * slice;
    const int dr = kFwdThreads / cols, dc = kFwdThreads - dr * cols;
    int r = tid / cols, c = tid - r * cols;
    for (int e0 = tid; e0 < total; e0 += U * kFwdThreads) {
        V v[U][kBandSlices];
        int dst[U];
        unsigned inside = 0;
#pragma unroll
        for (int u = 0; u < U; ++u) {
            const bool live = e0 + u * kFwdThreads < total;
            const int gj = j0 + r - 1, gi = i0 + c - 1;
            const bool in = live && (unsigned)gj < (unsigned)a.ny && (unsigned)gi < (unsigned)a.nx;
            const unsigned off = in ? (unsigned)(gj * a.nx + gi) : 0u;
            inside |= in ? 1u << u : 0u;
#pragma unroll
            for (int k = 0; k < kBandSlices; ++k) v[u][k] = (v0 + (k < ns ? k * slice : 0))[off];
            dst[u] = live ? r * W + c : -1;
            r += dr;
            c += dc;
            if (c >= cols) {
                c -= cols;
                ++r;
            }
        }
#pragma unroll
        for (int u = 0; u < U; ++u)
            if (dst[u] >= 0) {
                const bool in = inside & (1u << u);
                lds[dst[u]] = make_float4(in ? staged(v[u][0]) : 0.f, in && ns > 1 ? staged(v[u][1]) : 0.f,
                                          in && ns > 2 ? staged(v[u][2]) : 0.f, in && ns > 3 ? staged(v[u][3]) : 0.f);
            }
    }
}

template <class V>
__global__ __launch_bounds__(kFwdThreads) void proj_fwd_band_kernel(ProjArgs a, const V *vol, int out_stride)
{
    extern __shared__ __align__(16) unsigned char lds_raw[];
    const int nb = gridDim.x;
    const int lb = xcd_logical(blockIdx.x, nb);
    const int tid = threadIdx.x;
    // a.parts[0] blocks share the steep angles of a slice group, a.parts[1] the
    // others (a.order: a.n_steep steep ones first)
    const int per = a.parts[0] + a.parts[1];
    {
        const int g = lb / per;
        const int pp = lb - g * per;
        const bool steep = pp < a.parts[0];
        const int part = steep ? pp : pp - a.parts[0], np = steep ? a.parts[0] : a.parts[1];
        const int n0 = steep ? 0 : a.n_steep, nm = steep ? a.n_steep : a.M - a.n_steep;
        const int i0 = n0 + part * nm / np, i1 = n0 + (part + 1) * nm / np;
        const int k0 = kBandSlices * g, ns = min(kBandSlices, a.nz - k0);
        const int nrays = (i1 - i0) * a.nu;
        // band geometry: base indices [0, n_base) of the banded axis, nband a band
        const int n_base = (steep ? a.ny : a.nx) + 1, nband = steep ? a.band_rows : a.band_cols;
        const int W = steep ? proj_pitch(a.nx) : (a.band_cols + 1) | 1;
        const unsigned Wb = 16u * (unsigned)W;

        float bx[kBandRays], by[kBandRays], c[kBandRays], s[kBandRays], acc[kBandRays][kBandSlices];
        int glo[kBandRays], ghi[kBandRays];
        float *dst[kBandRays];
#pragma unroll
        for (int i = 0; i < kBandRays; ++i) {
            const int ray = tid + kFwdThreads * i;
            const bool ok = ray < nrays;
            glo[i] = ghi[i] = 0;
            if (ray - (tid & 63) >= nrays) continue;     // a wave without rays
            const int m = a.order[i0 + (ok ? ray / a.nu : 0)], p = ok ? ray % a.nu : 0;
            const float2 csv = a.cs[m];
            c[i] = csv.x;
            s[i] = csv.y;
            bx[i] = a.ax[(size_t)m * a.nu + p];
            by[i] = a.ay1[(size_t)m * a.nu + p];
            dst[i] = a.rt + ((size_t)m * a.nz + k0) * out_stride + p;
#pragma unroll
            for (int k = 0; k < kBandSlices; ++k) acc[i][k] = 0.f;
            // samples inside the bordered grid
            int x0, x1, y0, y1;
            samples_in(0.f, (float)(a.nx + 1), a.nr, a.half_nr, s[i], 1.f / s[i], bx[i], x0, x1);
            samples_in(0.f, (float)(a.ny + 1), a.nr, a.half_nr, c[i], 1.f / c[i], by[i], y0, y1);
            glo[i] = max(x0, y0);
            ghi[i] = ok ? min(x1, y1) : 0;
        }
        for (int b0 = 0; b0 < n_base; b0 += nband) {
            const int b1 = min(b0 + nband, n_base);
            __syncthreads();                     // the previous band is consumed
            if (steep)
                stage_band4(reinterpret_cast<float4 *>(lds_raw), vol, k0, a, b0, 0, b1 - b0 + 1, a.nx + 2, W, tid);
            else
                stage_band4(reinterpret_cast<float4 *>(lds_raw), vol, k0, a, 0, b0, a.ny + 2, b1 - b0 + 1, W, tid);
            __syncthreads();
            const unsigned base = 0u - (steep ? (unsigned)b0 * Wb : (unsigned)b0 * 16u);
#pragma unroll
            for (int i = 0; i < kBandRays; ++i) {
                if (kFwdThreads * i + (tid & ~63) >= nrays) continue;
                const float k = steep ? c[i] : s[i], b = steep ? by[i] : bx[i];
                int q0, q1;
                samples_in((float)b0, (float)b1, a.nr, a.half_nr, k, 1.f / k, b, q0, q1);
                q0 = max(q0, glo[i]);
                q1 = min(q1, ghi[i]);
                if (q0 >= q1) continue;
                auto get = [&](SamplePair &g, int q) {
                    pair_load(g, lds_raw, base, Wb, bx[i], by[i], s[i], c[i], (float)q - a.half_nr,
                              (float)(q1 - 1) - a.half_nr);
                };
                SamplePair ga, gb;
                int q = q0;
                get(ga, q);
                for (; q + 4 <= q1; q += 4) {
                    get(gb, q + 2);
                    pair_sum<2>(ga, acc[i]);
                    get(ga, q + 4);              // (past the end: the last sample again)
                    pair_sum<2>(gb, acc[i]);
                }
                const int left = q1 - q;
                if (left >= 2) {
                    get(gb, q + 2);
                    pair_sum<2>(ga, acc[i]);
                    if (left == 3) pair_sum<1>(gb, acc[i]);
                } else if (left == 1) {
                    pair_sum<1>(ga, acc[i]);
                }
            }
        }
#pragma unroll
        for (int i = 0; i < kBandRays; ++i) {
            if (tid + kFwdThreads * i >= nrays) continue;
#pragma unroll
            for (int k = 0; k < kBandSlices; ++k)
                if (k < ns) dst[i][(size_t)k * out_stride] = acc[i][k];
        }
        // zero the padding columns of the lines this block owns
        if (out_stride > a.nu) {
            const int pad = out_stride - a.nu;
            for (int idx = tid; idx < (i1 - i0) * ns * pad; idx += kFwdThreads) {
                const int l = idx / pad, m = a.order[i0 + l / ns];
                a.rt[((size_t)m * a.nz + k0 + l % ns) * out_stride + a.nu + idx % pad] = 0.f;
            }
        }
    }
}

constexpr int kTile = 16;
constexpr int kPW = 32;     // staged rays per angle per tile

// max(0, 1 - |t|), one clamped subtraction
__device__ __forceinline__ float hat(float t) { return __builtin_amdgcn_fmed3f(1.f - fabsf(t), 0.f, 1.f); }

// First staged detector index of angle (c, s) for the tile whose voxel-centre
// corners are (X0, Y0) .. (X0 + 15, Y0 + 15): u is linear in X and Y, so its
// minimum over the tile is at a corner; 2 rays of margin absorb the rounding
// between that minimum and any voxel's own u.
__device__ __forceinline__ int tile_p_lo(float c, float s, float X0, float Y0, float half_nu)
{
    const float X1 = X0 + (float)(kTile - 1), Y1 = Y0 + (float)(kTile - 1);
    const float u00 = X0 * c - Y0 * s, u10 = X1 * c - Y0 * s, u01 = X0 * c - Y1 * s, u11 = X1 * c - Y1 * s;
    return (int)floorf(fminf(fminf(u00, u10), fminf(u01, u11)) + half_nu) - 2;
}

// One block: a 16 x 16 voxel tile times KZ slices.  Angles are taken in
// chunks of a.adj_chunk: all lines a chunk needs (per angle KZ lines x 32
// rays) are staged in LDS in one pass, then every voxel accumulates the
// chunk's angles without further barriers.  H: the lines are fp16 with a
// power-of-two scale per line (the mixed operator's gathers), and each line's
// inverse scale multiplies its three-sample sum.  Weights and sums are fp32.
//
// What bounds it: vector work, the weights' (about 68 operations a voxel and
// angle) over the KZ slices that share them plus three products a slice.  So
// a ray's KZ values lie together in LDS: a 16-byte read serves 4 slices (8 in
// fp16) at the full LDS rate, the rays an odd number of 16-byte units apart so
// that the 16 rays of a voxel row fall in different banks; a staged unit is
// gathered from its lines by one thread, rays across lanes; the range tests of
// the weights are left to the waves whose rays end inside the tile (a detector
// index outside the lines meets staged zeros).  The sums are those of the
// untransposed form, bit for bit.  Measured at
// 256 x 256 x 128, 60 angles 228 -> 84 us (fp16 lines 149 -> 104), 192 x 192 x 96, 36
// 58 -> 37 (59 -> 43), 64^3, 24 16.3 -> 10.6 (15.7 -> 11.5).
template <int KZ, bool H>
struct AdjStage {
    static constexpr int E = H ? 8 : 4;            // slices a 16-byte unit
    static constexpr int QU = KZ / E;              // units a ray
    static constexpr int kPitch = QU | 1;          // units from a ray to the next
    static constexpr int kAngle = kPW * kPitch;    // units an angle
    static_assert(KZ % E == 0, "whole units");
};

// LDS bytes of a chunk: the lines, the inverse line scales (H), p_lo
template <int KZ, bool H>
constexpr size_t adj_lds(int chunk)
{
    return (size_t)chunk * (16 * AdjStage<KZ, H>::kAngle + (H ? 4 * KZ : 0) + 4);
}

template <int KZ, bool H>
__device__ __forceinline__ void adj_body(const ProjArgs &a, const uint16_t *__restrict__ rtb,
                                         const float *__restrict__ rtsc, int in_stride)
{
    using S = AdjStage<KZ, H>;
    typedef float f32x4 __attribute__((ext_vector_type(4)));
    typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));
    extern __shared__ __align__(16) float gs[];
    __shared__ double red[256 / 64];
    f32x4 *g4 = reinterpret_cast<f32x4 *>(gs);
    float *isc = gs + (size_t)4 * a.adj_chunk * S::kAngle;
    int *plo = reinterpret_cast<int *>(isc + (H ? (size_t)a.adj_chunk * KZ : 0));
    const int nb = gridDim.x;
    const int lb = xcd_logical(blockIdx.x, nb);
    const int zg = lb / (a.tiles_x * a.tiles_y);
    const int tile = lb % (a.tiles_x * a.tiles_y);
    const int tx0 = (tile % a.tiles_x) * kTile, ty0 = (tile / a.tiles_x) * kTile;
    const int k0 = zg * KZ;
    const int kn = min(KZ, a.nz - k0);
    const int tid = threadIdx.x;
    const int i = tx0 + (tid % kTile), j = ty0 + (tid / kTile);
    const bool valid = i < a.nx && j < a.ny;
    const float X = (float)i - a.cx, Y = (float)j - a.cy;
    const float X0 = (float)tx0 - a.cx, Y0 = (float)ty0 - a.cy;
    const int pp = tid % kPW, row0 = tid / kPW;   // staging: this thread's ray and first unit row

    float acc[KZ];
#pragma unroll
    for (int kk = 0; kk < KZ; ++kk) acc[kk] = 0.f;

    for (int mb = 0; mb < a.M; mb += a.adj_chunk) {
        const int mc = min(a.adj_chunk, a.M - mb);
        __syncthreads();                       // the previous chunk is consumed
        for (int mm = tid; mm < mc; mm += 256) {
            const float2 csv = a.cs[mb + mm];
            plo[mm] = tile_p_lo(csv.x, csv.y, X0, Y0, a.half_nu);
        }
        if constexpr (H) {
            for (int idx = tid; idx < mc * KZ; idx += 256) {
                const int mm = idx / KZ, kk = idx - mm * KZ;
                isc[idx] = kk < kn ? rtsc[(size_t)(mb + mm) * a.nz + k0 + kk] : 0.f;
            }
        }
        __syncthreads();
        // unit rows (angle mm, unit q) of 32 rays, 8 rows a pass, NS passes of
        // loads before their stores (a row past the end repeats the last)
        constexpr int NS = H ? 2 : 4;
        const int rows = mc * S::QU;
        for (int r0 = row0; r0 < rows; r0 += 8 * NS) {
            u32x4 v[NS];
            int dst[NS];
#pragma unroll
            for (int u = 0; u < NS; ++u) {
                const int r = min(r0 + 8 * u, rows - 1);
                const int mm = r / S::QU, q = r - mm * S::QU;
                const int p = plo[mm] + pp;
                const bool pin = p >= 0 && p < a.nu;
                dst[u] = mm * S::kAngle + pp * S::kPitch + q;
                // slices past the last repeat it (their sums are not stored)
                const size_t line = (size_t)(mb + mm) * a.nz + k0;
                const int e0 = S::E * q;
                if constexpr (H) {
                    const uint16_t *src = rtb + line * in_stride + (pin ? p : 0);
                    uint32_t w[8];
                    if (kn == KZ) {
                        src += (size_t)e0 * in_stride;
#pragma unroll
                        for (int e = 0; e < 8; ++e, src += in_stride) w[e] = *src;
                    } else {
#pragma unroll
                        for (int e = 0; e < 8; ++e) w[e] = src[(size_t)min(e0 + e, kn - 1) * in_stride];
                    }
#pragma unroll
                    for (int e = 0; e < 4; ++e) v[u][e] = pin ? w[2 * e] | (w[2 * e + 1] << 16) : 0u;
                } else {
                    const float *src = a.rt_in + line * in_stride + (pin ? p : 0);
                    float w[4];
                    if (kn == KZ) {
                        src += (size_t)e0 * in_stride;
#pragma unroll
                        for (int e = 0; e < 4; ++e, src += in_stride) w[e] = *src;
                    } else {
#pragma unroll
                        for (int e = 0; e < 4; ++e) w[e] = src[(size_t)min(e0 + e, kn - 1) * in_stride];
                    }
#pragma unroll
                    for (int e = 0; e < 4; ++e) v[u][e] = pin ? __float_as_uint(w[e]) : 0u;
                }
            }
#pragma unroll
            for (int u = 0; u < NS; ++u) g4[dst[u]] = __builtin_bit_cast(f32x4, v[u]);
        }
        __syncthreads();
        if (!valid) continue;
        for (int mm = 0; mm < mc; ++mm) {
            const float2 csv = a.cs[mb + mm];
            const float c = csv.x, s = csv.y;
            // voxel position in (detector, ray-sample) index coordinates
            const float u = fmaf(X, c, -Y * s) + a.half_nu;
            const float yv = fmaf(X, s, Y * c) + a.half_nr;
            const float pc = rintf(u), qc = rintf(yv);
            // displacement from the voxel to sample (pc + dp, qc + dq) in grid
            // coordinates: (dX0 + dp c + dq s, dY0 + dq c - dp s)
            const float du = pc - u, dy = qc - yv;
            const float dX0 = fmaf(du, c, dy * s), dY0 = fmaf(dy, c, -du * s);
            float w[3];
            {
#pragma clang fp contract(off)
                float h[3][3];    // [dp][dq]
#pragma unroll
                for (int dp = 0; dp < 3; ++dp) {
                    const float xp = dp == 0 ? dX0 - c : dp == 1 ? dX0 : dX0 + c;
                    const float yp = dp == 0 ? dY0 + s : dp == 1 ? dY0 : dY0 - s;
#pragma unroll
                    for (int dq = 0; dq < 3; ++dq) {
                        const float dX = dq == 0 ? xp - s : dq == 1 ? xp : xp + s;
                        const float dY = dq == 0 ? yp - c : dq == 1 ? yp : yp + c;
                        h[dp][dq] = hat(dX) * hat(dY);
                    }
                }
                if (__any(qc < 1.f || qc > (float)(a.nr - 2))) {   // a ray's end: samples that do not exist
#pragma unroll
                    for (int dp = 0; dp < 3; ++dp) {
                        h[dp][0] = qc >= 1.f ? h[dp][0] : 0.f;
                        h[dp][2] = qc <= (float)(a.nr - 2) ? h[dp][2] : 0.f;
                    }
                }
#pragma unroll
                for (int dp = 0; dp < 3; ++dp) w[dp] = (h[dp][0] + h[dp][1]) + h[dp][2];
            }
            const int off = min(max((int)pc - 1 - plo[mm], 0), kPW - 3);  // in range by construction
            const f32x4 *gp = g4 + mm * S::kAngle + off * S::kPitch;
            if constexpr (H) {
                typedef _Float16 f16x8 __attribute__((ext_vector_type(8)));
                const float *sc = isc + (size_t)mm * KZ;
#pragma unroll
                for (int q = 0; q < S::QU; ++q) {
                    const f16x8 v0 = __builtin_bit_cast(f16x8, gp[q]);
                    const f16x8 v1 = __builtin_bit_cast(f16x8, gp[S::kPitch + q]);
                    const f16x8 v2 = __builtin_bit_cast(f16x8, gp[2 * S::kPitch + q]);
#pragma unroll
                    for (int e = 0; e < 8; ++e) {
                        const float t = fmaf(w[0], (float)v0[e], fmaf(w[1], (float)v1[e], fmaf(w[2], (float)v2[e], 0.f)));
                        acc[8 * q + e] = fmaf(t, sc[8 * q + e], acc[8 * q + e]);
                    }
                }
            } else {
#pragma unroll
                for (int q = 0; q < S::QU; ++q) {
                    const f32x4 v0 = gp[q], v1 = gp[S::kPitch + q], v2 = gp[2 * S::kPitch + q];
#pragma unroll
                    for (int e = 0; e < 4; ++e)
                        acc[4 * q + e] = fmaf(w[0], v0[e], fmaf(w[1], v1[e], fmaf(w[2], v2[e], acc[4 * q + e])));
                }
            }
        }
    }

    double sq = 0.0;
    if (valid) {
#pragma unroll
        for (int kk = 0; kk < KZ; ++kk) {
            if (kk < kn) {
                const size_t idx = ((size_t)(k0 + kk) * a.ny + j) * a.nx + i;
                float v = acc[kk];
                if (a.x_sub || a.x_add) {
                    double t = (double)v;
                    if (a.x_add) t += (double)a.x_add[idx];
                    if (a.x_sub) t -= a.lambda * (double)a.x_sub[idx];
                    v = (float)t;
                }
                a.xo[idx] = v;
                sq += (double)v * (double)v;
            }
        }
    }
    if (a.norm_parts) {
        // block sum in float64, fixed order
        for (int o = 32; o > 0; o >>= 1) sq += __shfl_xor(sq, o);
        if ((tid & 63) == 0) red[tid >> 6] = sq;
        __syncthreads();
        if (tid == 0) a.norm_parts[blockIdx.x] = red[0] + red[1] + red[2] + red[3];
    }
}

template <int KZ>
__global__ __launch_bounds__(256) void proj_adj_kernel(ProjArgs a, int in_stride)
{
    adj_body<KZ, false>(a, nullptr, nullptr, in_stride);
}

template <int KZ>
__global__ __launch_bounds__(256) void proj_adj_f16(ProjArgs a, const uint16_t *rtb, const float *rtsc, int in_stride)
{
    adj_body<KZ, true>(a, rtb, rtsc, in_stride);
}

// Dual drive: z-drive line (m, p) of the workspace (line Lx + m*nu + p) holds
// column p of the projections of angle m across the z-rows, zero beyond nz.
// One block moves a 32 x 32 tile (rows k, columns p) of one angle through LDS
// so both the read and the write are row-contiguous.
constexpr int kTr = 32;

__global__ __launch_bounds__(256) void zlines_kernel(float *rt, int nz, int nu, int nup, long Lx)
{
    __shared__ float tile[kTr][kTr + 1];
    const int m = blockIdx.z, k0 = blockIdx.y * kTr, p0 = blockIdx.x * kTr;
    const int tx = threadIdx.x & 31, ty = threadIdx.x >> 5;   // 32 x 8 threads
    for (int j = ty; j < kTr; j += 8) {
        const int k = k0 + j, p = p0 + tx;
        tile[j][tx] = (k < nz && p < nu) ? rt[((size_t)m * nz + k) * nup + p] : 0.f;
    }
    __syncthreads();
    for (int j = ty; j < kTr; j += 8) {
        const int p = p0 + j, k = k0 + tx;
        if (p < nu && k < nup) rt[(size_t)(Lx + (long)m * nu + p) * nup + k] = tile[tx][j];
    }
}

// Transpose of zlines_kernel, added: x-drive line (m, k), column p gains
// element k of z-drive line (m, p).
__global__ __launch_bounds__(256) void fold_zlines_kernel(float *rt, int nz, int nu, int nup, long Lx)
{
    __shared__ float tile[kTr][kTr + 1];
    const int m = blockIdx.z, k0 = blockIdx.y * kTr, p0 = blockIdx.x * kTr;
    const int tx = threadIdx.x & 31, ty = threadIdx.x >> 5;
    for (int j = ty; j < kTr; j += 8) {
        const int p = p0 + j, k = k0 + tx;
        tile[j][tx] = (p < nu && k < nz) ? rt[(size_t)(Lx + (long)m * nu + p) * nup + k] : 0.f;
    }
    __syncthreads();
    for (int j = ty; j < kTr; j += 8) {
        const int k = k0 + j, p = p0 + tx;
        if (k < nz && p < nu) rt[((size_t)m * nz + k) * nup + p] += tile[tx][j];
    }
}

}  // namespace

static hipError_t launch_zlines(const mpi3d_plan *pl, float *rt, bool fold, hipStream_t st)
{
    // z-drive lines have nup entries (nz used), so the tiles cover nup rows k
    // when writing them and nz when folding back
    const int krows = fold ? pl->nz : pl->nup;
    const dim3 grid((pl->nu + kTr - 1) / kTr, (krows + kTr - 1) / kTr, pl->M);
    if (fold)
        hipLaunchKernelGGL(fold_zlines_kernel, grid, dim3(256), 0, st, rt, pl->nz, pl->nu, pl->nup, pl->Lx);
    else
        hipLaunchKernelGGL(zlines_kernel, grid, dim3(256), 0, st, rt, pl->nz, pl->nu, pl->nup, pl->Lx);
    return hipGetLastError();
}

static ProjArgs base_args(const mpi3d_plan *pl)
{
    ProjArgs a{};
    a.cs = pl->cs;
    a.ax = pl->ax;
    a.ay = pl->ay;
    a.ay1 = pl->ay1;
    a.order = pl->order;
    a.n_steep = pl->n_steep;
    a.nx = pl->nx; a.ny = pl->ny; a.nz = pl->nz; a.M = pl->M; a.nu = pl->nu; a.nup = pl->nup; a.nr = pl->nr;
    a.kz = pl->kz;
    a.adj_chunk = pl->adj_chunk;
    a.n_zgroups = (pl->nz + pl->kz - 1) / pl->kz;
    a.tiles_x = (pl->nx + kTile - 1) / kTile;
    a.tiles_y = (pl->ny + kTile - 1) / kTile;
    a.half_nr = 0.5f * (float)(pl->nr - 1);
    a.half_nu = 0.5f * (float)(pl->nu - 1);
    a.cx = 0.5f * (float)(pl->nx - 1);
    a.cy = 0.5f * (float)(pl->ny - 1);
    return a;
}

template <typename T>
static hipError_t launch_fwd(const mpi3d_plan *pl, const typename Texel<T>::V *vol, const FwdConfig &fc, float *rt,
                             int out_stride, hipStream_t st)
{
    ProjArgs a = base_args(pl);
    a.rt = rt;
    a.band_rows = fc.band_rows;
    a.n_bands = fc.n_bands;
    const size_t lds = (size_t)(fc.band_rows + 1) * proj_pitch(pl->nx) * sizeof(T);
    if (lds > 64 * 1024) {
        hipError_t e = hipFuncSetAttribute((const void *)proj_fwd_kernel<T>,
                                           hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds);
        if (e != hipSuccess) return e;
    }
    hipLaunchKernelGGL(proj_fwd_kernel<T>, dim3(fc.blocks), dim3(kFwdThreads), lds, st, a, vol, out_stride);
    return hipGetLastError();
}

template <class V>
static hipError_t launch_band(const mpi3d_plan *pl, const V *x, float *rt, int out_stride, hipStream_t st)
{
    ProjArgs a = base_args(pl);
    a.rt = rt;
    a.band_rows = pl->band.rows;
    a.band_cols = pl->band.cols;
    const int texels = std::max((a.band_rows + 1) * proj_pitch(a.nx), (a.ny + 2) * ((a.band_cols + 1) | 1));
    const int nm[2] = {a.n_steep, a.M - a.n_steep};
    for (int k = 0; k < 2; ++k) {
        a.parts[k] = pl->band.parts[k];
        if (nm[k] > 0 && (a.parts[k] < 1 || (long)((nm[k] + a.parts[k] - 1) / a.parts[k]) * a.nu > kFwdThreads * kBandRays))
            return hipErrorInvalidValue;
    }
    if (texels > kBandTexels) return hipErrorInvalidValue;
    const int lds = 16 * texels;
    hipError_t e = hipFuncSetAttribute((const void *)proj_fwd_band_kernel<V>,
                                       hipFuncAttributeMaxDynamicSharedMemorySize, lds);
    if (e != hipSuccess) return e;
    hipLaunchKernelGGL(proj_fwd_band_kernel<V>, dim3(pl->band.blocks), dim3(kFwdThreads), lds, st, a, x, out_stride);
    return hipGetLastError();
}

static hipError_t launch_fwd32(const mpi3d_plan *pl, const float *x, float *rt, int out_stride, hipStream_t st)
{
    if (pl->band.fp32) return launch_band(pl, x, rt, out_stride, st);
    if (pl->fwd32.slices == 2) return launch_fwd<float2>(pl, x, pl->fwd32, rt, out_stride, st);
    return launch_fwd<float>(pl, x, pl->fwd32, rt, out_stride, st);
}

hipError_t launch_project_strided(const mpi3d_plan *pl, const float *x, float *rt, int out_stride, hipStream_t st)
{
    return launch_fwd32(pl, x, rt, out_stride, st);
}

hipError_t launch_project(const mpi3d_plan *pl, const float *x, float *rt, hipStream_t st)
{
    hipError_t e = launch_fwd32(pl, x, rt, pl->nup, st);
    if (e == hipSuccess && pl->drive_axes == 2) e = launch_zlines(pl, rt, false, st);
    return e;
}

hipError_t launch_project16(const mpi3d_plan *pl, const float *x, const uint16_t *xb, float *rt, hipStream_t st)
{
    hipError_t e;
    if (pl->band.bf16)
        e = xb ? launch_band(pl, xb, rt, pl->nup, st)
               : launch_band(pl, reinterpret_cast<const Round16 *>(x), rt, pl->nup, st);
    else
        e = xb ? launch_fwd<uint32_t>(pl, xb, pl->fwd16, rt, pl->nup, st) : hipErrorInvalidValue;
    if (e == hipSuccess && pl->drive_axes == 2) e = launch_zlines(pl, rt, false, st);
    return e;
}

hipError_t launch_backproject_strided(const mpi3d_plan *pl, const float *rt, int in_stride, float *xo,
                                      const float *x_sub, double lambda, double *norm_parts, int *nparts,
                                      hipStream_t st, const float *x_add)
{
    ProjArgs a = base_args(pl);
    a.rt_in = rt;
    a.xo = xo;
    a.x_sub = x_sub;
    a.x_add = x_add;
    a.lambda = lambda;
    a.norm_parts = norm_parts;
    const int blocks = a.tiles_x * a.tiles_y * a.n_zgroups;
    if (nparts) *nparts = blocks;
    if (norm_parts && blocks > pl->max_parts) return hipErrorInvalidValue;
#define ADJ(KZ)                                                                                                   \
    case KZ:                                                                                                      \
        hipLaunchKernelGGL(proj_adj_kernel<KZ>, dim3(blocks), dim3(256), (adj_lds<KZ, false>(a.adj_chunk)), st, a, \
                           in_stride);                                                                            \
        break;
    switch (a.kz) {
        ADJ(4) ADJ(8) ADJ(16) ADJ(24) ADJ(32) ADJ(64)
    default: return hipErrorInvalidValue;
    }
#undef ADJ
    return hipGetLastError();
}

hipError_t launch_fold_zlines(const mpi3d_plan *pl, float *rt, hipStream_t st)
{
    return pl->drive_axes == 2 ? launch_zlines(pl, rt, true, st) : hipSuccess;
}

hipError_t launch_backproject16(const mpi3d_plan *pl, const uint16_t *rtb, const float *rtsc, float *xo,
                                const float *x_sub, double lambda, double *norm_parts, int *nparts, hipStream_t st,
                                const float *x_add)
{
    ProjArgs a = base_args(pl);
    a.xo = xo;
    a.x_sub = x_sub;
    a.x_add = x_add;
    a.lambda = lambda;
    a.norm_parts = norm_parts;
    a.kz = pl->kz16;
    a.adj_chunk = pl->adj_chunk16;
    a.n_zgroups = (pl->nz + a.kz - 1) / a.kz;
    const int blocks = a.tiles_x * a.tiles_y * a.n_zgroups;
    if (nparts) *nparts = blocks;
    if (norm_parts && blocks > pl->max_parts) return hipErrorInvalidValue;
#define ADJ(KZ)                                                                                                     \
    case KZ:                                                                                                        \
        hipLaunchKernelGGL(proj_adj_f16<KZ>, dim3(blocks), dim3(256), (adj_lds<KZ, true>(a.adj_chunk)), st, a, rtb, \
                           rtsc, pl->nup);                                                                          \
        break;
    switch (a.kz) {
        ADJ(8) ADJ(16) ADJ(24) ADJ(32) ADJ(64)
    default: return hipErrorInvalidValue;
    }
#undef ADJ
    return hipGetLastError();
}

hipError_t launch_backproject(const mpi3d_plan *pl, float *rt, float *xo, const float *x_sub, double lambda,
                              double *norm_parts, int *nparts, hipStream_t st, const float *x_add)
{
    if (pl->drive_axes == 2) {
        hipError_t e = launch_zlines(pl, rt, true, st);
        if (e != hipSuccess) return e;
    }
    return launch_backproject_strided(pl, rt, pl->nup, xo, x_sub, lambda, norm_parts, nparts, st, x_add);
}

}  // namespace mpi3d
