// Split reductions of the signal kernels and the CGLS vector/scalar steps.
//
// Every float64 norm is formed the same way: each block sums its elements'
// squares in float64 (fixed per-thread order, then a fixed tree), writes one
// partial, and whichever kernel needs the norm adds the partials in one fixed
// order.  Results therefore do not depend on timing, and the CGLS scalars
// (Sec. 3.3 solve of eq. nummodel; see the header for the recurrences) stay
// on the device: no host round trip per iteration.

#include <cmath>
#include <type_traits>

#include "device.h"

namespace mpi3d {

namespace {

constexpr int kThreads = 256;
constexpr int kVecBlocks = 1024;   // grid of the grid-stride vector kernels

__device__ __forceinline__ double block_sum(double v, double *red)
{
    for (int o = 32; o > 0; o >>= 1) v += __shfl_xor(v, o);
    const int w = threadIdx.x >> 6;
    if ((threadIdx.x & 63) == 0) red[w] = v;
    __syncthreads();
    double t = 0.0;
    if (threadIdx.x == 0)
        for (int i = 0; i < kThreads / 64; ++i) t += red[i];
    return t;  // valid in thread 0
}

// N consecutive floats as one word (4 N bytes aligned), N sums
template <int N>
struct Words {
    typedef float type __attribute__((ext_vector_type(N)));
};
template <>
struct Words<1> {
    typedef float type;
};
template <int N>
struct Sums {
    double v[N];
};
template <int N>
__device__ __forceinline__ float word(const typename Words<N>::type &w, int i)
{
    if constexpr (N == 1) return w;
    else return w[i];
}

// sum_s pp[s * stride] in float64, in split order, of N neighbours; eight
// loads in flight (a chain of rounds of loads, not bandwidth, is what many
// splits cost)
template <int N>
__device__ __forceinline__ Sums<N> sum_splits(const float *__restrict__ pp, int n, long stride)
{
    typedef typename Words<N>::type W;
    Sums<N> v{};
    int s = 0;
    auto block = [&](auto count) {
        constexpr int C = decltype(count)::value;
        W a[C];
#pragma unroll
        for (int j = 0; j < C; ++j) a[j] = *reinterpret_cast<const W *>(pp + (long)(s + j) * stride);
#pragma unroll
        for (int j = 0; j < C; ++j)
#pragma unroll
            for (int i = 0; i < N; ++i) v.v[i] += (double)word<N>(a[j], i);
        s += C;
    };
    while (s + 8 <= n) block(std::integral_constant<int, 8>{});
    while (s + 4 <= n) block(std::integral_constant<int, 4>{});
    while (s < n) block(std::integral_constant<int, 1>{});
    return v;
}

// Sum of the split partials of one output element, undoing the mixed path's
// per-line scale.  Without row coupling: the sum, divided by the line's own
// scale.  With the tensor PSF's passes (npass blocks of nparts / npass
// splits, pass e for offset e): forward, the line's passes e up to its
// coupling range, each divided by the scale of the symmetric sum that pass
// read (row_scale[e * lines + row]); adjoint, pass 0 of the line itself and
// pass e of the lines e before and after it within its angle, each divided
// by the scale of that line's data (row_scale[line]).  In pass order.
template <int N>
__device__ __forceinline__ Sums<N> sum_unscaled(const float *__restrict__ pp, int nparts, long stride, long row,
                                                const float *__restrict__ row_scale, RowPasses rp)
{
    if (rp.npass <= 1) {
        Sums<N> v = sum_splits<N>(pp, nparts, stride);
        if (row_scale)
#pragma unroll
            for (int i = 0; i < N; ++i) v.v[i] /= (double)row_scale[row];
        return v;
    }
    // passes: blocks of nparts / npass splits; the fused adjoint: every split
    // holds all passes, pass e at column offset e pass_cols of each line
    const int per = rp.pass_cols ? nparts : nparts / rp.npass;
    const long pass_off = rp.pass_cols ? (long)rp.pass_cols : (long)per * stride;
    const bool zl = row >= rp.zbase;
    const int nline = zl ? rp.nzc : rp.nz;
    const int R = min(zl ? rp.rz : rp.rx, rp.npass - 1);
    const int k = (int)(zl ? (row - rp.zbase) % rp.nzc : row % rp.nz);
    Sums<N> v{};
    for (int e = 0; e <= R; ++e) {
        const float *pe = pp + (long)e * pass_off;
        for (int sg = e == 0 || rp.fwd ? 1 : -1; sg <= 1; sg += 2) {
            const int d = rp.fwd ? 0 : sg * e;
            if (k + d < 0 || k + d >= nline) continue;
            const Sums<N> t = sum_splits<N>(pe + (long)d * rp.pitch, per, stride);
            const float *sc = row_scale ? row_scale + (rp.fwd ? (long)e * rp.lines + row : row + d) : nullptr;
#pragma unroll
            for (int i = 0; i < N; ++i) v.v[i] += sc ? t.v[i] / (double)*sc : t.v[i];
        }
    }
    return v;
}

// out[row][c] = sign * sum_s part[s][row][c] * col_scale[c] / row_scale[row] (+ b_sub);
// bcol (factored stage): column c = 2 j + part of bin j is column bcol[j] + part of part.
// N = 2: a bin's both parts a thread (out and b_sub 8-byte aligned), else one
// value.  I: the element index's type, 32 bits where it fits -- with 64-bit
// divisions and single values a 256 x 256 x 128 scan's 5 million values took
// 21 us, the bytes 10.
template <int N, class I>
__global__ __launch_bounds__(kThreads) void reduce_fwd_kernel(long rows, int nb2, int nbp2, int nparts,
                                                               long part_stride, const float *__restrict__ part,
                                                               const float *__restrict__ row_scale,
                                                               const float *__restrict__ col_scale, double scale,
                                                               const float *__restrict__ b_sub, float *out,
                                                               double *norm_parts, RowPasses rp,
                                                               const int *__restrict__ bcol)
{
    typedef typename Words<N>::type W;
    __shared__ double red[kThreads / 64];
    const I n = (I)(rows * nb2 / N), per = (I)(nb2 / N);
    double sq = 0.0;
    for (I idx = (I)blockIdx.x * kThreads + threadIdx.x; idx < n; idx += (I)gridDim.x * kThreads) {
        const I row = idx / per;
        const int c = N * (int)(idx - row * per);
        const int pc = bcol ? bcol[c >> 1] + (c & 1) : c;
        const Sums<N> v0 = sum_unscaled<N>(part + (long)row * nbp2 + pc, nparts, part_stride, row, row_scale, rp);
        W bs = {}, o;
        if (b_sub) bs = reinterpret_cast<const W *>(b_sub)[idx];
#pragma unroll
        for (int i = 0; i < N; ++i) {
            double v = v0.v[i] * scale;
            if (col_scale) v *= (double)col_scale[c + i];
            if (b_sub) v = (double)word<N>(bs, i) - v;
            const float f = (float)v;
            if constexpr (N == 1) o = f;
            else o[i] = f;
            sq += (double)f * (double)f;
        }
        reinterpret_cast<W *>(out)[idx] = o;
    }
    if (norm_parts) {
        const double t = block_sum(sq, red);
        if (threadIdx.x == 0) norm_parts[blockIdx.x] = t;
    }
}

// out[row][p] = scale * sum_s part[s][row][p] / row_scale[row]   (p < nu),
// N values a thread (out and its rows 4 N bytes aligned)
template <int N, class I>
__global__ __launch_bounds__(kThreads) void reduce_lines_kernel(long rows, int nu, int nup, int out_stride,
                                                                 int nparts, long part_stride,
                                                                 const float *__restrict__ part,
                                                                 const float *__restrict__ row_scale, double scale,
                                                                 float *out, RowPasses rp)
{
    typedef typename Words<N>::type W;
    const I n = (I)(rows * out_stride / N), per = (I)(out_stride / N);
    for (I idx = (I)blockIdx.x * kThreads + threadIdx.x; idx < n; idx += (I)gridDim.x * kThreads) {
        const I row = idx / per;
        const int p = N * (int)(idx - row * per);
        W o = {};
        if (p < nu) {
            const Sums<N> v = sum_unscaled<N>(part + (long)row * nup + p, nparts, part_stride, row, row_scale, rp);
#pragma unroll
            for (int i = 0; i < N; ++i) {
                const float f = p + i < nu ? (float)(v.v[i] * scale) : 0.f;
                if constexpr (N == 1) o = f;
                else o[i] = f;
            }
        }
        reinterpret_cast<W *>(out)[idx] = o;
    }
}

// The tensor PSF's forward pass inputs: sig[e][row] = rho(row + e) +
// rho(row - e) for the lines of row's angle (rows outside it count as zero;
// sig[0] = rho), zero for e beyond the row's coupling range and for columns
// past nu.
__global__ __launch_bounds__(kThreads) void sym_lines_kernel(const float *__restrict__ rho, int in_stride, int nu,
                                                              int nup, RowPasses rp, float *__restrict__ sig,
                                                              long pass_stride, long line_stride)
{
    const long n = (long)rp.npass * rp.lines * nup;
    for (long idx = (long)blockIdx.x * kThreads + threadIdx.x; idx < n; idx += (long)gridDim.x * kThreads) {
        const int p = (int)(idx % nup);
        const long t = idx / nup;
        const long row = t % rp.lines;
        const int e = (int)(t / rp.lines);
        const long o = e * pass_stride + row * line_stride + p;
        float v = 0.f;
        if (p < nu) {
            if (e == 0) {
                v = rho[row * in_stride + p];
            } else {
                const bool zl = row >= rp.zbase;
                const int nline = zl ? rp.nzc : rp.nz;
                const int R = zl ? rp.rz : rp.rx;
                const int k = (int)(zl ? (row - rp.zbase) % rp.nzc : row % rp.nz);
                if (e <= R) {
                    if (k + e < nline) v += rho[(row + e) * in_stride + p];
                    if (k - e >= 0) v += rho[(row - e) * in_stride + p];
                }
            }
        }
        sig[o] = v;
    }
}

// The mixed adjoint's lines as 16-bit operands of its backprojection: one
// wave per line forms the line's values -- the split sums as reduce_lines
// does, or (lines_in) fp32 lines already formed -- and a power-of-two scale
// s with max |v| s in [0.5, 1) (1 for a zero line; capped like the signal
// kernels' row scales), then writes fp16(v s) over nup columns (zero past
// nu) and 1/s.  Per-line scaling gives every line fp16's relative precision
// whatever its size.
constexpr int kLineSlots = 4;     // nup <= 256: at most 4 values per lane
__global__ __launch_bounds__(kThreads) void lines16_kernel(long rows, int nu, int nup, int nparts, long part_stride,
                                                            const float *__restrict__ part,
                                                            const float *__restrict__ row_scale, double scale,
                                                            RowPasses rp, const float *__restrict__ lines_in,
                                                            uint16_t *__restrict__ out16, float *__restrict__ inv_scale)
{
    const int lane = threadIdx.x & 63;
    const long row = (long)blockIdx.x * (kThreads / 64) + (threadIdx.x >> 6);
    if (row >= rows) return;
    float v[kLineSlots];
    float m = 0.f;
#pragma unroll
    for (int j = 0; j < kLineSlots; ++j) {
        const int p = lane + 64 * j;
        float o = 0.f;
        if (p < nu) {
            if (lines_in) {
                o = lines_in[row * nup + p];
            } else {
                const Sums<1> t = sum_unscaled<1>(part + row * nup + p, nparts, part_stride, row, row_scale, rp);
                o = (float)(t.v[0] * scale);
            }
        }
        v[j] = o;
        m = fmaxf(m, fabsf(o));
    }
    for (int o = 32; o > 0; o >>= 1) m = fmaxf(m, __shfl_xor(m, o));
    float s = 1.f;
    if (m > 0.f && isfinite(m)) {
        int e;
        frexpf(m, &e);
        s = ldexpf(1.f, min(-e, 120));
    }
    if (lane == 0) inv_scale[row] = 1.f / s;
#pragma unroll
    for (int j = 0; j < kLineSlots; ++j) {
        const int p = lane + 64 * j;
        if (p < nup) out16[row * nup + p] = __builtin_bit_cast(uint16_t, (_Float16)(v[j] * s));
    }
}

// Power-of-two line scales for the fp16 contractions: for each row,
// s = 2^-e with max_c |in[row][c] * col_scale[c]| in [2^(e-1), 2^e), so the
// scaled row's largest entry lies in [0.5, 1); 1 for an all-zero row.  With
// out16 the row is also written as the fp16 operand the signal kernels read,
// (in[row][c] * col_scale[c]) * s rounded to nearest, zero from column ncols
// to out16_cols.  One wave per row.
__global__ __launch_bounds__(kThreads) void row_scale_kernel(long rows, int ncols, int in_stride,
                                                              const float *__restrict__ in,
                                                              const float *__restrict__ col_scale, float *out,
                                                              uint16_t *__restrict__ out16, int out16_cols,
                                                              int out16_stride)
{
    const int lane = threadIdx.x & 63;
    const long row = (long)blockIdx.x * (kThreads / 64) + (threadIdx.x >> 6);
    if (row >= rows) return;
    const float *p = in + row * in_stride;
    float m = 0.f;
    for (int c = lane; c < ncols; c += 64) m = fmaxf(m, fabsf(col_scale ? p[c] * col_scale[c] : p[c]));
    for (int o = 32; o > 0; o >>= 1) m = fmaxf(m, __shfl_xor(m, o));
    float s = 1.f;
    if (m > 0.f && isfinite(m)) {
        // 2^-e brings the row maximum into [0.5, 1); capped so that rows
        // of subnormal size get a finite scale (and a normal 1/scale)
        int e;
        frexpf(m, &e);
        s = ldexpf(1.f, min(-e, 120));
    }
    if (lane == 0) out[row] = s;
    if (!out16) return;
    uint16_t *q = out16 + row * out16_stride;
    for (int c = lane; c < out16_cols; c += 64) {
        const float v = c < ncols ? (col_scale ? p[c] * col_scale[c] : p[c]) * s : 0.f;
        const _Float16 hv = (_Float16)v;
        q[c] = __builtin_bit_cast(uint16_t, hv);
    }
}

// Scalar slots (doubles) of one solve.
enum { S_GAMMA = 0, S_DELTA, S_ALPHA, S_BETA, S_BAD, S_GAMMA0, S_STEP, S_PREV, S_NSLOTS };

__device__ double sum_parts(const double *parts, int n, double *red)
{
    double v = 0.0;
#pragma unroll 8
    for (int i = threadIdx.x; i < n; i += kThreads) v += parts[i];
    return block_sum(v, red);
}

// The CGLS updates with their scalars.  Every block adds the norm partials
// itself, in the order one block would (some 2 us, in place of a launch of
// about 5 us in the iteration's serial chain; a 64^3 x 24-angle iteration:
// alpha 5.8 + update 4.5 -> 6.4 us, beta 3.0 + update 3.6 -> 4.9); block 0 writes
// the scalars, into slots that no block of the same launch reads: the update of
// x and r reads GAMMA and copies it to PREV, that of p reads PREV and writes
// GAMMA.

// delta = |q|^2 + lambda |p|^2, alpha = gamma / delta;
// x = x + alpha p, r = r - alpha q
__global__ __launch_bounds__(kThreads) void update_xr_kernel(float *__restrict__ x, const float *__restrict__ p,
                                                              float *__restrict__ r, const float *__restrict__ q,
                                                              long nvox, long ndata, double *scal,
                                                              const double *parts_q, int nq, const double *parts_p,
                                                              int np, double lambda, double *hist, int step)
{
    __shared__ double red[kThreads / 64];
    __shared__ double sh;
    const double qq = sum_parts(parts_q, nq, red);
    __syncthreads();
    const double pp = sum_parts(parts_p, np, red);
    if (threadIdx.x == 0) {
        const double gamma = scal[S_GAMMA], delta = qq + lambda * pp, alpha = gamma / delta;
        sh = alpha;
        if (blockIdx.x == 0) {
            scal[S_DELTA] = delta;
            scal[S_ALPHA] = alpha;
            scal[S_PREV] = gamma;
            if (!isfinite(alpha)) scal[S_BAD] = 1.0;
            if (hist) {
                hist[4 * step + 0] = gamma;
                hist[4 * step + 1] = delta;
                hist[4 * step + 2] = alpha;
            }
        }
    }
    __syncthreads();
    const float af = (float)sh;
    const long n = nvox + ndata;
    for (long idx = (long)blockIdx.x * kThreads + threadIdx.x; idx < n; idx += (long)gridDim.x * kThreads) {
        if (idx < nvox) x[idx] = fmaf(af, p[idx], x[idx]);
        else {
            const long j = idx - nvox;
            r[j] = fmaf(-af, q[j], r[j]);
        }
    }
}

// gamma' = |s|^2, beta = gamma' / gamma; p = s + beta p, optional bf16 shadow,
// partial |p|^2.  init (a restart; on the first, `first`, gamma0 = gamma'):
// beta = 0, p = s, and d and r (where given) are cleared.
__global__ __launch_bounds__(kThreads) void update_p_kernel(float *__restrict__ p, const float *__restrict__ s,
                                                             uint16_t *pb, long n, double *scal,
                                                             const double *parts_s, int ns, double *parts_p, int init,
                                                             int first, double *hist, int step, float *d, float *r,
                                                             long ndata)
{
    __shared__ double red[kThreads / 64];
    __shared__ double sh;
    if (!init || blockIdx.x == 0) {
        const double g = sum_parts(parts_s, ns, red);
        if (threadIdx.x == 0) {
            double beta = 0.0;
            if (!init) beta = g / scal[S_PREV];
            sh = beta;
            if (blockIdx.x == 0) {
                if (first) scal[S_GAMMA0] = g;
                scal[S_GAMMA] = g;
                scal[S_BETA] = beta;
                if (!isfinite(g) || !isfinite(beta)) scal[S_BAD] = 1.0;
                if (hist && !init) hist[4 * step + 3] = beta;
            }
        }
        __syncthreads();
    }
    const float bf = init ? 0.f : (float)sh;
    double sq = 0.0;
    for (long idx = (long)blockIdx.x * kThreads + threadIdx.x; idx < n; idx += (long)gridDim.x * kThreads) {
        const float v = init ? s[idx] : fmaf(bf, p[idx], s[idx]);
        p[idx] = v;
        sq += (double)v * (double)v;
        if (pb) pb[idx] = bf16_bits(v);
        if (d) d[idx] = 0.f;
    }
    if (r)
        for (long idx = (long)blockIdx.x * kThreads + threadIdx.x; idx < ndata; idx += (long)gridDim.x * kThreads)
            r[idx] = 0.f;
    const double t = block_sum(sq, red);
    if (threadIdx.x == 0) parts_p[blockIdx.x] = t;
}

// A solve's start from x = 0: x cleared, r = b, the scalars cleared (scal may be null).
__global__ __launch_bounds__(kThreads) void start_kernel(float *x, long nvox, float *r, const float *b, long ndata,
                                                          double *scal)
{
    if (scal && blockIdx.x == 0 && threadIdx.x < S_NSLOTS) scal[threadIdx.x] = 0.0;
    const long n = nvox + ndata;
    for (long idx = (long)blockIdx.x * kThreads + threadIdx.x; idx < n; idx += (long)gridDim.x * kThreads) {
        if (idx < nvox) x[idx] = 0.f;
        else r[idx - nvox] = b[idx - nvox];
    }
}

__global__ __launch_bounds__(kThreads) void to_bf16_kernel(long n, const float *x, uint16_t *xb)
{
    for (long idx = (long)blockIdx.x * kThreads + threadIdx.x; idx < n; idx += (long)gridDim.x * kThreads)
        xb[idx] = bf16_bits(x[idx]);
}

__global__ __launch_bounds__(kThreads) void clamp_kernel(float *x, long n)
{
    for (long idx = (long)blockIdx.x * kThreads + threadIdx.x; idx < n; idx += (long)gridDim.x * kThreads)
        x[idx] = fmaxf(x[idx], 0.f);
}

// x = x + d (refinement sweep end), optionally clamped at 0
__global__ __launch_bounds__(kThreads) void add_to_kernel(float *__restrict__ x, const float *__restrict__ d, long n,
                                                           int clamp)
{
    for (long idx = (long)blockIdx.x * kThreads + threadIdx.x; idx < n; idx += (long)gridDim.x * kThreads) {
        const float v = x[idx] + d[idx];
        x[idx] = clamp ? fmaxf(v, 0.f) : v;
    }
}

__global__ __launch_bounds__(kThreads) void fill_kernel(float *x, long n, float v)
{
    for (long idx = (long)blockIdx.x * kThreads + threadIdx.x; idx < n; idx += (long)gridDim.x * kThreads)
        x[idx] = v;
}

__global__ __launch_bounds__(kThreads) void copy_kernel(float *dst, const float *src, long n)
{
    for (long idx = (long)blockIdx.x * kThreads + threadIdx.x; idx < n; idx += (long)gridDim.x * kThreads)
        dst[idx] = src[idx];
}

// scal[S_GAMMA] = sum of the step partials (and S_GAMMA0 on the first step)
__device__ __forceinline__ void step_norm(double *scal, const double *parts, int n, int first, double *red)
{
    const double t = sum_parts(parts, n, red);
    if (threadIdx.x == 0) {
        scal[S_GAMMA] = t;
        if (first) scal[S_GAMMA0] = t;
        if (!isfinite(t)) scal[S_BAD] = 1.0;
    }
    __syncthreads();
}

// One step of the paper's iteration (eq. iters) after g = A^T (b - A y):
//   x_new = P(y + tau g - tau lambda T^T T y),  P = clamp at 0 when nonneg
//   y_new = x_new + beta (x_new - x)            (the next momentum point)
// T^T T y is the 7-point finite-difference Laplacian with no term across the
// volume boundary (fd = 1) or y itself (fd = 0).  y_new may alias g: every
// thread reads g only at its own voxel before writing y_new there.  A block
// partial of |x_new - y|^2 (the step) goes to parts; block 0 also adds the
// previous step's (prev, nprev of them; first: that was the first step), in
// place of a launch of its own.
template <class I>      // the voxel index's type: 32 bits where it fits (its divisions: 13.5 us of 128 x 128 x 64 in 64)
__global__ __launch_bounds__(kThreads) void momentum_kernel(const float *__restrict__ y, const float *g,
                                                             const float *__restrict__ x, float *__restrict__ x_new,
                                                             float *y_new, int nx, int ny, int nz, float tau,
                                                             float taulam, float beta, int fd, int nonneg,
                                                             double *parts, double *scal, const double *prev,
                                                             int nprev, int first)
{
    __shared__ double red[kThreads / 64];
    if (nprev > 0 && blockIdx.x == 0) step_norm(scal, prev, nprev, first, red);
    const I n = (I)nx * ny * nz;
    const I sxy = (I)nx * ny;
    double sq = 0.0;
    for (I idx = (I)blockIdx.x * kThreads + threadIdx.x; idx < n; idx += (I)gridDim.x * kThreads) {
        const float yc = y[idx];
        float ty = yc;
        if (fd) {
            const I line = idx / (I)nx;
            const int i = (int)(idx - line * (I)nx);
            const int k = (int)(line / (I)ny), j = (int)(line - (I)k * (I)ny);
            float acc = 0.f;
            if (i > 0) acc += yc - y[idx - 1];
            if (i + 1 < nx) acc += yc - y[idx + 1];
            if (j > 0) acc += yc - y[idx - nx];
            if (j + 1 < ny) acc += yc - y[idx + nx];
            if (k > 0) acc += yc - y[idx - sxy];
            if (k + 1 < nz) acc += yc - y[idx + sxy];
            ty = acc;
        }
        float v = fmaf(tau, g[idx], fmaf(-taulam, ty, yc));
        if (nonneg) v = fmaxf(v, 0.f);
        const float xo = x[idx];
        x_new[idx] = v;
        y_new[idx] = fmaf(beta, v - xo, v);
        const double dv = (double)v - (double)yc;
        sq += dv * dv;
    }
    const double t = block_sum(sq, red);
    if (threadIdx.x == 0) parts[blockIdx.x] = t;
}

__global__ __launch_bounds__(kThreads) void step_norm_kernel(double *scal, const double *parts, int n, int first)
{
    __shared__ double red[kThreads / 64];
    step_norm(scal, parts, n, first, red);
}

// Power iteration on A^T A: norms[k] = |z| from the partials of |z|^2.
__global__ __launch_bounds__(kThreads) void norm_record_kernel(const double *parts, int n, double *norms, int k)
{
    __shared__ double red[kThreads / 64];
    const double t = sum_parts(parts, n, red);
    if (threadIdx.x == 0) norms[k] = sqrt(t);
}

// v = z / norms[k]
__global__ __launch_bounds__(kThreads) void scale_by_kernel(float *__restrict__ v, const float *__restrict__ z, long n,
                                                             const double *norms, int k)
{
    const float inv = (float)(1.0 / norms[k]);
    for (long idx = (long)blockIdx.x * kThreads + threadIdx.x; idx < n; idx += (long)gridDim.x * kThreads)
        v[idx] = z[idx] * inv;
}

__global__ void scal_init_kernel(double *scal)
{
    if (threadIdx.x < S_NSLOTS) scal[threadIdx.x] = 0.0;
}

int grid_for(long n, int cap = kVecBlocks)
{
    long b = (n + kThreads - 1) / kThreads;
    if (b < 1) b = 1;
    if (b > cap) b = cap;
    return (int)b;
}

constexpr int kReduceBlocks = kMaxNormParts;   // the split reductions want many loads in flight

}  // namespace

int scal_slots() { return S_NSLOTS; }
int scal_slot_bad() { return S_BAD; }
int scal_slot_gamma() { return S_GAMMA; }
int scal_slot_gamma0() { return S_GAMMA0; }

hipError_t launch_reduce_fwd(long rows, int nb2, int nbp2, int nparts, long part_stride, const float *part,
                             const float *row_scale, const float *col_scale, double scale, const float *b_sub,
                             float *out, double *norm_parts, int *nnorm, hipStream_t st, RowPasses rp,
                             const int *bcol)
{
    // (wide words where they leave a block a CU: A^T A of a 32^3 scan with 8
    // angles 58.0 us with them, 57.3 without)
    const bool two = rows * nb2 >= 2 * 256 * kThreads && (uintptr_t)out % 8 == 0 && (uintptr_t)b_sub % 8 == 0 && nb2 % 2 == 0 && nbp2 % 2 == 0;
    const bool i32 = rows * nb2 < 0x70000000l;      // (and a grid's stride past it)
    const int g = grid_for(two ? rows * nb2 / 2 : rows * nb2, kReduceBlocks);
    if (nnorm) *nnorm = g;
    const auto k = two ? i32 ? reduce_fwd_kernel<2, unsigned> : reduce_fwd_kernel<2, long>
                       : i32 ? reduce_fwd_kernel<1, unsigned> : reduce_fwd_kernel<1, long>;
    hipLaunchKernelGGL(k, dim3(g), dim3(kThreads), 0, st, rows, nb2, nbp2, nparts, part_stride, part, row_scale,
                       col_scale, scale, b_sub, out, norm_parts, rp, bcol);
    return hipGetLastError();
}

hipError_t launch_reduce_lines_strided(long rows, int nu, int nup, int out_stride, int nparts, long part_stride,
                                       const float *part, const float *row_scale, double scale, float *out,
                                       hipStream_t st, RowPasses rp)
{
    const bool four = rows * out_stride >= 4 * 256 * kThreads && (uintptr_t)out % 16 == 0 && out_stride % 4 == 0;
    const bool i32 = rows * out_stride < 0x70000000l;
    const int g = grid_for(four ? rows * out_stride / 4 : rows * out_stride, kReduceBlocks);
    const auto k = four ? i32 ? reduce_lines_kernel<4, unsigned> : reduce_lines_kernel<4, long>
                        : i32 ? reduce_lines_kernel<1, unsigned> : reduce_lines_kernel<1, long>;
    hipLaunchKernelGGL(k, dim3(g), dim3(kThreads), 0, st, rows, nu, nup, out_stride, nparts, part_stride, part,
                       row_scale, scale, out, rp);
    return hipGetLastError();
}

hipError_t launch_lines16(long rows, int nu, int nup, int nparts, long part_stride, const float *part,
                          const float *row_scale, double scale, RowPasses rp, const float *lines_in, uint16_t *out16,
                          float *inv_scale, hipStream_t st)
{
    if (nup > 64 * kLineSlots) return hipErrorInvalidValue;
    const long blocks = (rows + kThreads / 64 - 1) / (kThreads / 64);
    hipLaunchKernelGGL(lines16_kernel, dim3((unsigned)blocks), dim3(kThreads), 0, st, rows, nu, nup, nparts,
                       part_stride, part, row_scale, scale, rp, lines_in, out16, inv_scale);
    return hipGetLastError();
}



hipError_t launch_sym_lines(const float *rho, int in_stride, int nu, int nup, RowPasses rp, float *sig,
                            long pass_stride, long line_stride, hipStream_t st)
{
    const int g = grid_for((long)rp.npass * rp.lines * nup, kReduceBlocks);
    hipLaunchKernelGGL(sym_lines_kernel, dim3(g), dim3(kThreads), 0, st, rho, in_stride, nu, nup, rp, sig,
                       pass_stride, line_stride);
    return hipGetLastError();
}

hipError_t launch_row_scale(long rows, int ncols, int in_stride, const float *in, const float *col_scale, float *out,
                            uint16_t *out16, int out16_cols, int out16_stride, hipStream_t st)
{
    const long blocks = (rows + kThreads / 64 - 1) / (kThreads / 64);
    hipLaunchKernelGGL(row_scale_kernel, dim3((unsigned)blocks), dim3(kThreads), 0, st, rows, ncols, in_stride, in,
                       col_scale, out, out16, out16_cols, out16_stride);
    return hipGetLastError();
}

hipError_t launch_to_bf16(long n, const float *x, uint16_t *xb, hipStream_t st)
{
    hipLaunchKernelGGL(to_bf16_kernel, dim3(grid_for(n)), dim3(kThreads), 0, st, n, x, xb);
    return hipGetLastError();
}

hipError_t launch_update_xr(float *x, const float *p, float *r, const float *q, long nvox, long ndata, double *scal,
                            const double *parts_q, int nq, const double *parts_p, int np, double lambda, double *hist,
                            int step, hipStream_t st)
{
    hipLaunchKernelGGL(update_xr_kernel, dim3(grid_for(nvox + ndata)), dim3(kThreads), 0, st, x, p, r, q, nvox,
                       ndata, scal, parts_q, nq, parts_p, np, lambda, hist, step);
    return hipGetLastError();
}

hipError_t launch_update_p(float *p, const float *s, uint16_t *pb, long n, double *scal, const double *parts_s, int ns,
                           double *parts_p, int *np_out, int init, int first, double *hist, int step, float *d,
                           float *r, long ndata, hipStream_t st)
{
    const int g = grid_for(n);
    if (np_out) *np_out = g;
    hipLaunchKernelGGL(update_p_kernel, dim3(g), dim3(kThreads), 0, st, p, s, pb, n, scal, parts_s, ns, parts_p, init,
                       first, hist, step, d, r, ndata);
    return hipGetLastError();
}

hipError_t launch_start(float *x, long nvox, float *r, const float *b, long ndata, double *scal, hipStream_t st)
{
    hipLaunchKernelGGL(start_kernel, dim3(grid_for(nvox + ndata)), dim3(kThreads), 0, st, x, nvox, r, b, ndata, scal);
    return hipGetLastError();
}

hipError_t launch_scal_init(double *scal, hipStream_t st)
{
    hipLaunchKernelGGL(scal_init_kernel, dim3(1), dim3(64), 0, st, scal);
    return hipGetLastError();
}

hipError_t launch_clamp(float *x, long n, hipStream_t st)
{
    hipLaunchKernelGGL(clamp_kernel, dim3(grid_for(n)), dim3(kThreads), 0, st, x, n);
    return hipGetLastError();
}

hipError_t launch_fill(float *x, long n, float v, hipStream_t st)
{
    hipLaunchKernelGGL(fill_kernel, dim3(grid_for(n)), dim3(kThreads), 0, st, x, n, v);
    return hipGetLastError();
}

hipError_t launch_copy(float *dst, const float *src, long n, hipStream_t st)
{
    hipLaunchKernelGGL(copy_kernel, dim3(grid_for(n)), dim3(kThreads), 0, st, dst, src, n);
    return hipGetLastError();
}

hipError_t launch_add_to(float *x, const float *d, long n, int clamp, hipStream_t st)
{
    hipLaunchKernelGGL(add_to_kernel, dim3(grid_for(n)), dim3(kThreads), 0, st, x, d, n, clamp);
    return hipGetLastError();
}

hipError_t launch_momentum(const float *y, const float *g, const float *x, float *x_new, float *y_new, int nx,
                           int ny, int nz, float tau, float taulam, float beta, int fd, int nonneg, double *parts,
                           int *nparts, double *scal, const double *prev, int nprev, int first, hipStream_t st)
{
    const long n = (long)nx * ny * nz;
    const int b = grid_for(n, kReduceBlocks);
    if (nparts) *nparts = b;
    hipLaunchKernelGGL(n < 0x70000000l ? momentum_kernel<unsigned> : momentum_kernel<long>, dim3(b), dim3(kThreads), 0, st, y, g, x, x_new, y_new, nx, ny, nz, tau,
                       taulam, beta, fd, nonneg, parts, scal, prev, nprev, first);
    return hipGetLastError();
}

hipError_t launch_step_norm(double *scal, const double *parts, int n, int first, hipStream_t st)
{
    hipLaunchKernelGGL(step_norm_kernel, dim3(1), dim3(kThreads), 0, st, scal, parts, n, first);
    return hipGetLastError();
}

hipError_t launch_norm_record(const double *parts, int n, double *norms, int k, hipStream_t st)
{
    hipLaunchKernelGGL(norm_record_kernel, dim3(1), dim3(kThreads), 0, st, parts, n, norms, k);
    return hipGetLastError();
}

hipError_t launch_scale_by(float *v, const float *z, long n, const double *norms, int k, hipStream_t st)
{
    hipLaunchKernelGGL(scale_by_kernel, dim3(grid_for(n)), dim3(kThreads), 0, st, v, z, n, norms, k);
    return hipGetLastError();
}

}  // namespace mpi3d
