// Plan creation: validation, float64 host tables, upload, workspace layout,
// and the operator entry points of the C ABI (forward, adjoint, stages).
//
// Tables follow the paper's factors:
//   cos/sin of the FFL angles           Sec. 2.2, eq. qtheta
//   ray-sample coordinate bases          eq. ptheta2 (unit-step Riemann sum)
//   PSF kernel K[n][p]                   eq. reals0 + Appendix B eq. PSF
//       = v_n L'((xi_n - u_p)/w) / w, xi_n = a sin(2 pi P n / T), v = xi'
//       (the global scale c_A is applied in fp64 when split sums are reduced,
//       so scans that differ only in c_A share identical line tables)
//   band DFT F[n][2j], F[n][2j+1]        Appendix A (+i, 1/sqrt(T)) on the kept
//       = Re/Im(D_j e^{+2 pi i (omega_j n mod T)/T}) / sqrt(T)   bins (eq. bcompress,
//                                        eq. DCmodel)
// All table values are computed in float64, then rounded once to fp32 or fp16, or
// split into a pair of fp16 numbers (the high one rounded, the low one the rest).

#include <algorithm>
#include <cmath>
#include <cstring>
#include <new>
#include <type_traits>
#include <vector>

#include "internal.h"

using namespace mpi3d;

namespace {

constexpr double kPi = 3.14159265358979323846264338327950288;

// L'(x) = 1/x^2 - 1/sinh^2 x.  For |x| < 0.5 the Maclaurin series
// sum_{n>=1} 2^{2n} B_{2n} (2n-1) x^{2n-2} / (2n)! (Bernoulli numbers B_{2n});
// for larger |x| the closed form, written with e^{-2|x|} so nothing overflows.
double langevin_deriv(double x)
{
    x = std::fabs(x);
    if (x < 0.5) {
        static const double bern[] = {1.0 / 6, -1.0 / 30, 1.0 / 42, -1.0 / 30, 5.0 / 66, -691.0 / 2730,
                                      7.0 / 6, -3617.0 / 510, 43867.0 / 798, -174611.0 / 330};
        double coef[10];
        double fact = 1.0, pow4 = 1.0;
        for (int n = 1; n <= 10; ++n) {
            fact *= (2.0 * n - 1) * (2.0 * n);
            pow4 *= 4.0;
            coef[n - 1] = pow4 * bern[n - 1] * (2.0 * n - 1) / fact;
        }
        double x2 = x * x, acc = 0.0;
        for (int n = 9; n >= 0; --n) acc = acc * x2 + coef[n];
        return acc;
    }
    double e = std::exp(-2.0 * x);
    return 1.0 / (x * x) - 4.0 * e / ((1.0 - e) * (1.0 - e));
}

// L(x) = coth x - 1/x.  For |x| < 0.5 the Maclaurin series
// sum_{n>=1} 2^{2n} B_{2n} x^{2n-1} / (2n)!; for larger |x| the closed form,
// where the two terms differ by at least 8% and nothing cancels badly.
double langevin(double x)
{
    const double ax = std::fabs(x);
    if (ax < 0.5) {
        static const double bern[] = {1.0 / 6, -1.0 / 30, 1.0 / 42, -1.0 / 30, 5.0 / 66, -691.0 / 2730,
                                      7.0 / 6, -3617.0 / 510, 43867.0 / 798, -174611.0 / 330};
        double coef[10];
        double fact = 1.0, pow4 = 1.0;
        for (int n = 1; n <= 10; ++n) {
            fact *= (2.0 * n - 1) * (2.0 * n);
            pow4 *= 4.0;
            coef[n - 1] = pow4 * bern[n - 1] / fact;
        }
        double x2 = x * x, acc = 0.0;
        for (int n = 9; n >= 0; --n) acc = acc * x2 + coef[n];
        return x * acc;
    }
    return 1.0 / std::tanh(x) - 1.0 / x;
}

// xx entry of the tensor PSF at in-plane offset (du, dz), dz != 0, with the
// gradient magnitude equal on both axes: L'(r/w)/w du^2/r^2 + L(r/w) dz^2/r^3.
double psf_xx(double du, double dz, double w)
{
    const double r2 = du * du + dz * dz, r = std::sqrt(r2);
    return langevin_deriv(r / w) / w * (du * du / r2) + langevin(r / w) * (dz * dz / (r2 * r));
}

// double -> fp16, rounded once (clang's _Float16 conversion is correctly rounded)
inline _Float16 to_f16(double v) { return (_Float16)v; }

// v (|v| < 2^15) as the nearest pair of fp16 numbers: hi = rn16(v), lo =
// rn16(v - hi).  By integer arithmetic on the double's bits, several times
// faster than the library conversion over a table's millions of entries.
inline uint16_t half_bits(double v, double *rounded)
{
    const double a = std::fabs(v);
    const uint16_t sign = std::signbit(v) ? 0x8000 : 0;
    if (a < 6.103515625e-05) {                     // below 2^-14: multiples of 2^-24
        const double q = (a * 16777216.0 + 4503599627370496.0) - 4503599627370496.0;
        *rounded = std::copysign(q / 16777216.0, v);
        return sign | (uint16_t)q;
    }
    uint64_t b;
    std::memcpy(&b, &a, 8);
    b += 0x1ffffffffffull + ((b >> 42) & 1);       // to 10 fraction bits, ties to even
    b &= ~0x3ffffffffffull;
    double r;
    std::memcpy(&r, &b, 8);
    *rounded = std::copysign(r, v);
    return sign | (uint16_t)((((b >> 52) - 1008) << 10) + ((b >> 42) & 0x3ff));
}
inline void half_pair(double v, uint16_t &hi, uint16_t &lo)
{
    double h, l;
    hi = half_bits(v, &h);
    lo = half_bits(v - h, &l);
}

// |D_j| of the receive filter (null: 1).
double bin_gain(const float *rx, int j) { return rx ? std::hypot((double)rx[2 * j], (double)rx[2 * j + 1]) : 1.0; }

// Exponents e_j with |D_j| scale 2^e_j in [2^14, 2^15) for bins j < nb, and the
// smallest of them (the strongest bin's).  A bin with D_j = 0 gets a large one:
// its data then drops out of an adjoint's lines.
std::vector<int> bin_exponents(const float *rx, int nb, double scale, int *least)
{
    constexpr int kNone = 5000;
    std::vector<int> ex(nb, kNone);
    *least = kNone;
    for (int j = 0; j < nb; ++j) {
        const double d = bin_gain(rx, j) * scale;
        if (!(d > 0)) continue;
        int e = 0;
        std::frexp(d * 1.0000001, &e);
        ex[j] = 15 - e;
        *least = std::min(*least, ex[j]);
    }
    return ex;
}

int round_up(int v, int m) { return (v + m - 1) / m * m; }
size_t align256(size_t v) { return (v + 255) & ~size_t(255); }

// Ray samples: smallest n >= sqrt(nx^2 + ny^2) with the parity of ny.
int ray_count(int nx, int ny)
{
    long d2 = (long)nx * nx + (long)ny * ny;
    int n = (int)std::floor(std::sqrt((double)d2));
    while ((long)n * n < d2) ++n;
    while (n > 0 && (long)(n - 1) * (n - 1) >= d2) --n;
    if ((n - ny) % 2) ++n;
    return n;
}

// Column groups of one precision's signal kernels for a band table of nct0
// 32-wide column tiles.  A pair covers 2 GH tiles of one group.  Narrow
// blocks (4 pairs, two waves per SIMD) hold at most 14 tiles per pair; wide
// blocks (2 pairs, one wave per SIMD: FP32 only) up to 22, so a table of 15 to
// 22 tiles needs one group instead of two -- each extra group repeats the
// first contraction (the time signal) for its lines.  Tables are zero-padded
// to the group width, so the kernels need no per-tile guards.
void column_groups(int nct0, bool fp32, mpi3d_plan::SigCfg &c)
{
    static const int widths[] = {6, 8, 12, 14};
    if (fp32 && nct0 > 14 && nct0 <= 22) {
        c.pairs = kWidePairs;
        c.ngroups = 1;
        c.gct = (nct0 + 1) / 2 * 2;
        return;
    }
    c.pairs = kWaves;
    c.ngroups = (nct0 + 13) / 14;
    const int want = (nct0 + c.ngroups - 1) / c.ngroups;
    c.gct = 0;
    for (int wdt : widths)
        if (!c.gct && wdt >= want) c.gct = wdt;
}

// Choose the T-split of one precision: (line tiles x splits x groups) blocks,
// one block resident per CU (narrow blocks need about 250 VGPRs a wave at two
// waves per SIMD, wide ones more than 256 at one).  Cost in seconds: rounds of
// blocks times chunks per block times one block's time per chunk, at the
// per-CU MFMA rate measured on MI355X (FP32 about 4.3e11 flop/s, fp16 about
// 2.3e12), plus each split's partial sums written and read back by the
// reduction at about 5 TB/s.
void choose_split(const mpi3d_plan *pl, bool fp32, mpi3d_plan::SigCfg &c, int nup, int passes)
{
    const int slots = 256;
    const int rows = kRowsPerWave * c.pairs;
    const long tiles = (pl->L + rows - 1) / rows;
    const double rate = fp32 ? 4.3e11 : 2.3e12;
    const double t_chunk = (double)rows * kChunk * 2.0 * (nup + kColTile * c.gct) / rate;
    const double split_bytes = 8.0 * passes * pl->L * std::max<double>(pl->nbp2, (double)c.ngroups * nup);
    int best_s = 1;
    double best = 1e30;
    for (int s = 1; s <= pl->nchunks; ++s) {
        int cps = (pl->nchunks + s - 1) / s;
        int used = (pl->nchunks + cps - 1) / cps;  // splits actually non-empty
        long blocks = tiles * used * c.ngroups;
        long rounds = (blocks + slots - 1) / slots;
        double cost = (double)rounds * cps * t_chunk + used * split_bytes / 5e12;
        if (cost < best * (1.0 - 1e-9)) {
            best = cost;
            best_s = used;
        }
    }
    c.cps = (pl->nchunks + best_s - 1) / best_s;
    c.nsplit = (pl->nchunks + c.cps - 1) / c.cps;
    c.tail_c0 = c.tail_tpb = 0;
    // FP32 wide blocks (one per CU): a tail split can even the load when the
    // tiles times the splits leave CUs idle -- s splits of w chunks per tile,
    // and the remaining r = nchunks - s w chunks of every tile gathered
    // tail_tpb tiles to a block, all in one round of blocks
    if (fp32 && c.pairs == kWidePairs) {
        const long per_group = slots / c.ngroups;
        for (int w = (int)((tiles * pl->nchunks + per_group - 1) / per_group); w < pl->nchunks; ++w) {
            const int s = pl->nchunks / w, r = pl->nchunks - s * w;
            if (r == 0) continue;
            const int tpb = std::max(1, w / r);
            const long blocks = (tiles * s + (tiles + tpb - 1) / tpb) * c.ngroups;
            if (blocks > slots) continue;
            const double cost = std::max(w, tpb * r) * t_chunk + (s + 1) * split_bytes / 5e12;
            if (cost < best * (1.0 - 1e-9)) {
                best = cost;
                c.cps = w;
                c.nsplit = s + 1;
                c.tail_c0 = s * w;
                c.tail_tpb = tpb;
            }
        }
    }
    // Serving launches merge the lines of several requests, so their time
    // split must not depend on the line count: a fixed split per line class.
    c.serve_nsplit = std::min(pl->nchunks, 16);
    c.serve_cps = (pl->nchunks + c.serve_nsplit - 1) / c.serve_nsplit;
    c.serve_nsplit = (pl->nchunks + c.serve_cps - 1) / c.serve_cps;
}

// Kernel configuration and time splits of the dense stage on fp16 pairs: the
// least estimated time.  Measured over all configurations and 2 to 32 splits at
// six scans: a block (one a CU) takes about 12 us besides its chunks; a chunk
// its products at 32 cycles each, 2.2 GHz, 80% busy with two waves a SIMD and
// 62% with one; each split costs the reduction
// one more partial sum (its chain of loads, about 0.1 us, and its bytes written
// and read at 4 TB/s).  Within 5% of each other, the forward takes ranges of at
// most 24 chunks (64^3, 24 angles, T = 4001: 18 chunks in place of 26, whose
// longer sums cost 4% more error than fp32 MFMA has).
// room: bytes for the partial sums.  Returns the time (1e30 where nothing fits).
double choose_dense_split(const mpi3d_plan *pl, bool fwd, double room, mpi3d_plan::Split::Dir &d)
{
    const int nct = pl->split.nct;
    double best = 1e30;
    for (int i = 0;; ++i) {
        int gt, waves;
        const int fits = split_config(i, pl->nup, &gt, &waves);
        if (fits < 0) break;
        if (!fits) continue;
        const int ng = (nct + gt - 1) / gt;
        long tg = 0;
        for (int gi = 0; gi < pl->n_line_groups; ++gi) tg += (pl->groups[gi].rows + 32 * waves - 1) / (32 * waves);
        const double chunk = (3.0 * pl->nup / 16 + 6.0 * gt) * 32 / 2.2e9 * (waves == 8 ? 2 / 0.80 : 1 / 0.62);
        const double per_split =
            fwd ? 1e-7 + 8.0 * pl->L * 32 * nct / 4e12 : ng * (1e-7 + 8.0 * pl->L * pl->nup / 4e12);
        for (int ns = 1; ns <= std::min(pl->nchunks, 128); ++ns) {
            const int len = (pl->nchunks + ns - 1) / ns;
            if (4.0 * pl->L * ns * (fwd ? 32 * nct : ng * pl->nup) > room) break;
            double t = (double)((tg * ng * ns + 255) / 256) * (12e-6 + len * chunk) + ns * per_split;
            if (fwd && waves == 4 && len > 24) t *= 1.05;
            if (t < best * (1.0 - 1e-9)) {
                best = t;
                d = {i, ng, ns};
            }
        }
    }
    return best;
}

// The operator workspace's layout (bytes from its base), with or without the
// factored FP32 stage or the dense one on fp16 pairs.
void op_layout(mpi3d_plan *pl, bool fac, bool split = false)
{
    const mpi3d_plan::Fac &f = pl->fac;
    const bool mixed = pl->precisions & (1 << MPI3D_MIXED);
    size_t o = 0;
    auto put = [&](size_t bytes) { o = align256(o); size_t r = o; o += bytes; return r; };
    pl->ws_rt = put(sizeof(float) * pl->L * pl->nup);
    size_t parts = 0;   // split partial sums: forward [splits][L][nbp2], adjoint [splits][groups][L][nup]
    for (int i = fac || split ? 1 : 0; i < 2; ++i) {
        if ((fac || split) && !mixed) break;
        const mpi3d_plan::SigCfg &c = pl->sc[i];
        parts = std::max(parts, (size_t)std::max(c.nsplit, c.serve_nsplit) *
                                    std::max<size_t>(pl->nbp2, (size_t)c.ngroups * pl->nup));
    }
    size_t part_floats = (size_t)pl->n_passes * pl->L * parts;
    if (pl->fused && !fac)   // one pass; adjoint lines of nupf
        part_floats = std::max(part_floats, (size_t)pl->L * std::max(pl->scf.nsplit, pl->scf.serve_nsplit) *
                                                std::max<size_t>(pl->nbp2, (size_t)pl->nupf));
    if (split)
        part_floats = std::max({part_floats, (size_t)pl->L * pl->split.fwd.nsplit * 32 * pl->split.nct,
                                (size_t)pl->L * pl->split.adj.nsplit * pl->split.adj.ngroups * pl->nup});
    size_t part_bytes = sizeof(float) * part_floats;
    pl->ws_part = align256(o);
    pl->ws_fac = pl->ws_lexp = pl->ws_part;
    if (fac) {
        // The factored stage's partial sums (adjoint: nsplit blocks of nup-column
        // lines; forward: psplit of 32 U columns) and phase sums lie where the mixed
        // operator has its partial sums: a request's calls follow one another, and
        // none leaves any of them for the next.  End to end they took a 192 x 192 x
        // 96 raster of 36 angles past the no-allocation scratch.
        const size_t own = sizeof(float) * pl->L * std::max(f.nsplit_adj * pl->n_passes * pl->nup, f.psplit * 32 * f.U);
        pl->ws_fac = align256(pl->ws_part + own);
        pl->ws_lexp = align256(pl->ws_fac + sizeof(uint32_t) * f.held_lines * f.P * 2 * f.zst);
        part_bytes = std::max(part_bytes, pl->ws_lexp + sizeof(int) * f.held_lines - pl->ws_part);
    }
    put(part_bytes);
    pl->ws_norm = put(sizeof(double) * pl->max_parts);
    // per tensor-PSF pass: the forward's symmetric line sums, their
    // scales and fp16 operands (one block each without coupling)
    const size_t np = pl->n_passes;
    pl->ws_rowscale = put(sizeof(float) * np * pl->L);
    pl->ws_xb = put(mixed ? sizeof(uint16_t) * pl->nvox : 0);
    pl->in16_cols = std::max(pl->nup, pl->nbp2);
    pl->ws_in16 = put(mixed ? sizeof(uint16_t) * np * pl->L * pl->in16_cols : 0);
    pl->ws_rtb = put(mixed ? sizeof(uint16_t) * pl->L * pl->nup : 0);
    pl->ws_rtsc = put(mixed ? sizeof(float) * pl->L : 0);
    pl->ws_sig = put(np > 1 ? sizeof(float) * np * pl->L * pl->nup : 0);
    pl->op_ws_bytes = align256(o);
}

// The dense stage on fp16 pairs: its splits within the workspace that the fp32 MFMA
// form takes, or the no-allocation entry point's scratch if that is more.  Returns
// the time of a forward and an adjoint, 1e30 for plans without such a stage: those
// with the mixed operator (for the reason given at the factored stage's choice),
// tensor PSFs, and where nothing fits.
double choose_pairs(mpi3d_plan *pl)
{
    const int precisions = pl->precisions;
    if (!(precisions & (1 << MPI3D_FP32)) || (precisions & (1 << MPI3D_MIXED)) || pl->n_passes > 1 ||
        (double)pl->nchunks * ((pl->nb2 + 31) / 32) * 4096 >= 2147483647.0 ||
        (double)pl->nchunks * pl->nup * 128 >= 2147483647.0)
        return 1e30;
    mpi3d_plan::Split &sp = pl->split;
    sp.nct = (pl->nb2 + 31) / 32;
    op_layout(pl, false);
    const double bound = std::max<double>(pl->op_ws_bytes, MPI3D_NOALLOC_SCRATCH_BYTES);
    const double room = bound - 512.0 - (double)(pl->op_ws_bytes - (pl->ws_norm - pl->ws_part));
    return choose_dense_split(pl, true, room, sp.fwd) + choose_dense_split(pl, false, room, sp.adj);
}

// Bytes of phase sums of a scan whose bins bunch, else 0: at most 24 residues mod C
// (32 or 64), and under 3/4 of the dense form's products in the factored form even
// with a pair of columns for every residue and fp32 products alone.  least: with a
// pair of columns for every residue, however few; else with the 16 pairs of columns
// that the kernels are for at least.
double bunched_phase_bytes(const mpi3d_plan *pl, const std::vector<long> &bins, bool least)
{
    if (pl->n_ktab > 1 || pl->n_line_groups > 1 || pl->n_passes > 1) return 0;
    const int T = pl->nt;
    double best = 0.75 * T * (pl->nup + pl->nbp2), bytes = 0;
    for (int C = 32; C <= T && C <= 64; C += 32) {
        if (T % C) continue;
        std::vector<int> cnt(C, 0);
        for (long b : bins) ++cnt[b % C];
        int R = 0, U = 0;
        for (int c : cnt) {
            R += c > 0;
            U += (c + 15) / 16;
        }
        if (R > 24 || *std::max_element(cnt.begin(), cnt.end()) > 24) continue;
        const int zst = (R + 3) / 4 * 4, P = T / C;
        const double cost = (double)T * (pl->nup + 32 * ((2 * zst + 31) / 32)) + 64.0 * ((P + 7) / 8 * 8) * U;
        if (cost < best) {
            best = cost;
            bytes = 8.0 * P * (least ? zst : std::max(16, zst)) * ((pl->L + 31) / 32 * 32 + 1);
        }
    }
    return bytes;
}

// Tiles a launch of the factored stage takes and the splits of its kernels: the
// least estimated time of a forward and an adjoint among those whose workspace
// stays within the bound: every line group in one launch where that fits, else group
// after group, in ranges of tiles.  The bound is the no-allocation entry point's
// scratch, or what the scan's dense form takes if that is more, so that a scan whose
// dense form fits the scratch does.  Scans whose bins bunch may take their phase sums
// on top where even the least number of them is past the scratch: ranges would cost
// them 3 to 9% (256 x 256 x 128 in two ranges, forward 489 -> 503 us, adjoint 416 ->
// 454; 192 x 192 x 96, A then A^T, 303 -> 329) and more where few angles leave CUs
// idle (32 x 32 x 152, 54 angles, T = 6144, 32 cycles, 22 harmonics: contraction
// 62 -> 108 us).  dense: the dense form's seconds a line and direction.  False where
// nothing fits, or where what was held back is estimated
// slower than a dense form (a 64 x 64 x 300 raster, 24 angles, T = 12288: in ranges of
// tiles 482 us for A and A^T, dense on fp16 pairs 300; 192 x 192 x 303, 12 angles, 491
// and 346, unbounded 384).
//
// The outer sums' forward waves are of two tiles and a slot, the adjoint's blocks of a
// tile; small launches also split the phase stages (8 and 16 phases) until about
// 2048 waves (256 blocks) run.  The line-tile kernels take 8 tiles a block, one block
// a CU: a block takes about 4 us to load its lines and first stages, then its phases
// at two waves a SIMD (MFMAs of 32 cycles at about 60% busy, 2.4 GHz); each phase
// range of the adjoint costs the reduction one more partial sum (its chain of loads,
// about 0.1 us, and the bytes at 4 TB/s).
bool choose_fac_ranges(mpi3d_plan *pl, const std::vector<long> &bins, double dense)
{
    mpi3d_plan::Fac &f = pl->fac;
    const int np = pl->n_passes, nup = pl->nup;
    const double t_phase = f.cj * (3.0 * nup / 16 + 6.0 * ((2 * f.zst + 31) / 32)) * 64 / 0.6 / 2.4e9;
    auto splits = [&](long groups, int most, double per_range, double &t) {
        int nbest = 1;
        t = 1e30;
        for (int ns = 1; ns <= std::min({f.P, 256, most}); ++ns) {
            const double tn = (double)((groups * ns + 255) / 256) * (4e-6 + (f.P + ns - 1) / ns * t_phase) + ns * per_range;
            if (tn < t * (1.0 - 1e-9)) {
                t = tn;
                nbest = ns;
            }
        }
        return nbest;
    };
    op_layout(pl, false);
    const double bunched = bunched_phase_bytes(pl, bins, false);
    double bound = std::max<double>(pl->op_ws_bytes, MPI3D_NOALLOC_SCRATCH_BYTES);
    if (pl->op_ws_bytes + bunched_phase_bytes(pl, bins, true) > bound) bound = pl->op_ws_bytes + bunched;
    const long tiles = (f.max_rows + 31) / 32;
    mpi3d_plan::Fac best = f;
    double tbest = 1e30;
    bool found = false, free = false;       // free: nothing was held back
    // n = 0: every line group in one launch; n > 0: group after group, in n ranges
    for (long n = pl->n_line_groups > 1 ? 0 : 1; n <= tiles; ++n) {
        f.together = n == 0;
        f.range = (int)(n > 1 ? (tiles + n - 1) / n : tiles);
        if (n > 1) f.range = (f.range + kFacWaves - 1) / kFacWaves * kFacWaves;
        if (n > 1 && (tiles + f.range - 1) / f.range < n) continue;      // as few ranges have this length
        long at_once = 0, tgroups = 0, fgroups = 0;     // tiles of a launch; blocks a phase range, adjoint and forward
        f.held_lines = 0;
        for (int gi = 0; gi < (f.together ? pl->n_line_groups : 1); ++gi) {
            const long t = f.together ? (pl->groups[gi].rows + 31) / 32 : f.range;
            at_once += t;
            tgroups += (t + kFacWaves - 1) / kFacWaves;
            fgroups += np * nup <= 256 ? (t + kFacWaves - 1) / kFacWaves : (t + 3) / 4;   // (tensor lines: blocks of 4 tiles)
            f.held_lines += 32 * t + 1;
        }
        if ((double)f.held_lines * f.P * 2 * f.zst >= 2147483647.0) continue;
        // what is left of the bound for the partial sums
        f.psplit = f.nsplit_adj = 0;
        op_layout(pl, true);
        const size_t rest = pl->op_ws_bytes - (pl->ws_norm - pl->ws_part);
        const double room = bound - 1024.0 - (double)rest - (double)(pl->ws_lexp + sizeof(int) * f.held_lines - pl->ws_part);
        const long most_out = (long)(room / (4.0 * pl->L * 32 * f.U)), most_adj = (long)(room / (4.0 * pl->L * nup * np));
        if (most_out < 1 || most_adj < 1) continue;
        const long psplit = std::max<long>(1, std::min<long>({8, 2048 / ((at_once + 1) / 2 * f.R), (f.P + 7) / 8}));
        f.psplit = (int)std::min(psplit, most_out);
        f.zsplit = (int)std::max<long>(1, std::min<long>({8, 256 / at_once, (f.P + 15) / 16}));
        // (tensor lines: the adjoint's blocks are np times as many)
        double tf, ta;
        f.nsplit = splits(fgroups, 256, 0.0, tf);
        f.nsplit_adj = splits(tgroups * np, (int)std::min<long>(most_adj, 256), 1e-7 + 8.0 * pl->L * nup * np / 4e12, ta);
        // the outer sums: their launches, the phase sums' bytes at 4 TB/s
        const double t = (f.together ? 1 : pl->n_line_groups * n) * (tf + ta + 10e-6) + 32.0 * f.P * f.zst * pl->L / 4e12;
        if (t < tbest) {
            tbest = t;
            best = f;
            found = true;
            free = n <= 1 && f.psplit == psplit && f.nsplit_adj < most_adj;
        }
        if (f.psplit == psplit && f.nsplit_adj < most_adj) break;
    }
    f = best;
    const double other = 2 * dense * pl->L + 30e-6;
    return found && (free || tbest < (bunched > 0 ? other : std::min(other, choose_pairs(pl))));
}

template <class T>
T *carve(char *base, size_t &off, size_t count)
{
    off = align256(off);
    T *p = reinterpret_cast<T *>(base + off);
    off += count * sizeof(T);
    return p;
}

}  // namespace

extern "C" const char *mpi3d_strerror(int status)
{
    switch (status) {
    case MPI3D_OK: return "ok";
    case MPI3D_EINVAL: return "invalid argument";
    case MPI3D_ENOMEM: return "out of device memory or workspace too small";
    case MPI3D_EDEVICE: return "HIP runtime error";
    case MPI3D_ENOTSUP: return "geometry not supported by the compiled kernels";
    case MPI3D_ENONFINITE: return "non-finite value in a solver norm";
    default: return "unknown status";
    }
}

extern "C" int mpi3d_plan_create(const mpi3d_geometry *g, int device, mpi3d_plan **out)
{
    if (!g || !out) return MPI3D_EINVAL;
    *out = nullptr;
    if (g->nx < 2 || g->ny < 2 || g->nz < 1 || g->n_angles < 1 || g->n_t < 32) return MPI3D_EINVAL;
    if (g->nx > 4096 || g->ny > 4096 || g->nz > 65535 || g->n_angles > 4096 || g->n_t > (1 << 22)) return MPI3D_EINVAL;
    int nu = g->n_u ? g->n_u : g->nx;
    if (nu < 2 || nu > 256) return MPI3D_ENOTSUP;
    if (!(g->drive_cycles > 0) || !(g->psf_width > 0) || !(g->op_scale >= 0)) return MPI3D_EINVAL;
    if (!(g->drive_amp >= 0)) return MPI3D_EINVAL;
    if (!std::isfinite(g->raster_sweep)) return MPI3D_EINVAL;
    const int n_classes = (g->raster_sweep != 0.0 && g->nz >= 2) ? 2 : 1;
    if (g->harm_lo < 1 || g->harm_hi < g->harm_lo || g->half_band < 0) return MPI3D_EINVAL;
    int precisions = g->precisions ? g->precisions : (1 << MPI3D_FP32);
    if (precisions & ~((1 << MPI3D_FP32) | (1 << MPI3D_MIXED) | (1 << MPI3D_PRECOMPOSED))) return MPI3D_EINVAL;
    // tensor PSF line coupling: every precision, without a raster
    if (g->psf_rows < 0) return MPI3D_EINVAL;
    const int psf_rows = std::min(g->psf_rows, g->nz - 1);
    if (psf_rows > 0 && n_classes > 1) return MPI3D_ENOTSUP;
    // dual drive: z-drive lines across the z-rows, as many entries as the
    // x-drive lines hold (nz <= n_u); under the tensor PSF they couple across
    // the detector columns of their angle
    const int drive_axes = g->drive_axes == 2 ? 2 : 1;
    if (g->drive_axes < 0 || g->drive_axes > 2 || !(g->drive_amp_z >= 0)) return MPI3D_EINVAL;
    if (drive_axes == 2 && (g->nz > nu || n_classes > 1)) return MPI3D_ENOTSUP;
    const int psf_cols = drive_axes == 2 && g->psf_rows > 0 ? std::min(g->psf_rows, nu - 1) : 0;
    const int n_ktab = drive_axes == 2 ? (psf_rows + 1) + (psf_cols + 1) : n_classes * (psf_rows + 1);

    // kept bins, validated
    std::vector<long> bins;
    for (int k = g->harm_lo; k <= g->harm_hi; ++k) {
        long c = (long)std::floor(k * g->drive_cycles + 0.5);
        for (int d = -g->half_band; d <= g->half_band; ++d) bins.push_back(c + d);
    }
    for (size_t i = 0; i < bins.size(); ++i) {
        if (bins[i] <= 0 || bins[i] >= g->n_t / 2) return MPI3D_EINVAL;
        if (i && bins[i] <= bins[i - 1]) return MPI3D_EINVAL;  // increasing => distinct
    }
    if (bins.size() > 2048) return MPI3D_ENOTSUP;

    hipError_t e = hipSetDevice(device);
    if (e != hipSuccess) return MPI3D_EINVAL;

    mpi3d_plan *pl = new (std::nothrow) mpi3d_plan();
    if (!pl) return MPI3D_ENOMEM;
    pl->device = device;
    pl->nx = g->nx; pl->ny = g->ny; pl->nz = g->nz; pl->M = g->n_angles;
    pl->nu = nu; pl->nt = g->n_t; pl->nr = ray_count(g->nx, g->ny);
    pl->nb = (int)bins.size();
    pl->harm_lo = g->harm_lo; pl->harm_hi = g->harm_hi; pl->half_band = g->half_band;
    pl->P = g->drive_cycles;
    pl->a = g->drive_amp > 0 ? g->drive_amp : nu / 2.0;
    pl->w = g->psf_width;
    pl->op_scale = g->op_scale;
    pl->precisions = precisions;
    pl->n_classes = n_classes;
    pl->psf_rows = psf_rows;
    pl->n_ktab = n_ktab;
    pl->pass_r = std::max(psf_rows, psf_cols);
    pl->n_passes = pl->pass_r + 1;
    pl->raster_sweep = g->raster_sweep;
    pl->nup = round_up(nu, 64);
    pl->ntp = round_up(g->n_t, kChunk);
    pl->nb2 = 2 * pl->nb;
    pl->nbp2 = round_up(pl->nb2, kColTile);
    pl->nct = pl->nbp2 / kColTile;
    pl->drive_axes = drive_axes;
    pl->a_z = g->drive_amp_z > 0 ? g->drive_amp_z : g->nz / 2.0;
    pl->Lx = (long)pl->M * pl->nz;
    pl->Lz = drive_axes == 2 ? (long)pl->M * nu : 0;
    pl->L = pl->Lx + pl->Lz;
    // line groups of a signal stage (each with its own PSF tables)
    if (n_classes > 1) {
        pl->n_line_groups = n_classes;
        for (int c = 0; c < n_classes; ++c) {
            const int per = (pl->nz - c + n_classes - 1) / n_classes;
            pl->groups[c] = {pl->M * per, per, pl->nz, c, n_classes, c, 0, pl->nz, 0};
        }
    } else if (drive_axes == 2) {
        pl->n_line_groups = 2;
        pl->groups[0] = {(int)pl->Lx, (int)pl->Lx, 0, 0, 1, 0, psf_rows, pl->nz, 0};
        pl->groups[1] = {(int)pl->Lz, (int)pl->Lz, 0, (int)pl->Lx, 1, psf_rows + 1, psf_cols, nu, pl->Lx};
    } else {
        pl->n_line_groups = 1;
        pl->groups[0] = {(int)pl->L, (int)std::max<long>(1, pl->L), 0, 0, 1, 0, psf_rows, pl->nz, 0};
    }
    pl->nvox = (long)pl->nx * pl->ny * pl->nz;
    pl->nchunks = pl->ntp / kChunk;

    // Column groups and time splits per precision; the band tables hold the
    // larger of the two paddings.
    {
        const int nct0 = pl->nct;
        column_groups(nct0, true, pl->sc[0]);
        column_groups(nct0, false, pl->sc[1]);
        pl->nct = pl->sc[0].ngroups * pl->sc[0].gct;
        if (precisions & (1 << MPI3D_MIXED)) pl->nct = std::max(pl->nct, pl->sc[1].ngroups * pl->sc[1].gct);
        // FP32 tensor PSF in one fused pass, where a kernel fits: every line
        // group coupled over the same R, a virtual line of a compiled width,
        // the band table in one wide group of 14 or 16 column tiles
        bool same_r = pl->pass_r > 0;
        for (int gi = 0; gi < pl->n_line_groups; ++gi) same_r = same_r && pl->groups[gi].coup == pl->pass_r;
        const int nupf = (pl->pass_r + 1) * pl->nup, gctf = 2 * std::max(7, (nct0 + 1) / 2);
        if (same_r && nct0 <= 16 && sig_fused_supported(nupf, gctf)) {
            pl->fused = true;
            pl->nupf = nupf;
            pl->scf = mpi3d_plan::SigCfg{kWidePairs, 1, gctf, 0, 0, 0, 0, 0, 0};
            pl->nct = std::max(pl->nct, gctf);
        }
        pl->nbp2 = pl->nct * kColTile;
    }
    {
        const mpi3d_plan::SigCfg &c0 = pl->sc[0], &c1 = pl->sc[1];
        if (!sig_fwd_supported(pl->nup, c0.gct, MPI3D_FP32, c0.pairs) ||
            !sig_adj_supported(pl->nup, c0.gct, MPI3D_FP32, c0.pairs) ||
            ((precisions & (1 << MPI3D_MIXED)) && (!sig_fwd_supported(pl->nup, c1.gct, MPI3D_MIXED, c1.pairs) ||
                                                   !sig_adj_supported(pl->nup, c1.gct, MPI3D_MIXED, c1.pairs)))) {
            delete pl;
            return MPI3D_ENOTSUP;
        }
    }
    choose_split(pl, true, pl->sc[0], pl->nup, pl->n_passes);
    choose_split(pl, false, pl->sc[1], pl->nup, pl->n_passes);
    if (pl->fused) choose_split(pl, true, pl->scf, pl->nupf, 1);

    // projection configuration
    {
        // Forward: a staged texel holds one or two slices (4 bytes: one fp32
        // slice or two bf16 slices; 8 bytes: two fp32 slices); a slice group
        // too large for 160 KB of LDS is staged in row bands (LDS rows =
        // band_rows + 1).  The fp32 path takes slice pairs only when a pair
        // fits in one band, since a band edge splits a wave's rays unevenly.
        // The ceil(nz / slices) * M (slice group, angle) units are split into
        // equal contiguous ranges, one per block (a block holds kFwdThreads *
        // fwd_rays_per_thread rays, nu per unit), in whole rounds of 256
        // blocks.
        auto fwd_config = [&](int slices, int texel_bytes, mpi3d::FwdConfig &fc) {
            const size_t lds = 160 * 1024;
            const int bases = pl->ny + 1;           // base rows -1 .. ny-1
            const int max_rows = (int)(lds / ((size_t)mpi3d::proj_pitch(pl->nx) * texel_bytes)) - 1;
            if (max_rows < 2) return false;
            fc.slices = slices;
            fc.n_bands = (bases + max_rows - 1) / max_rows;
            fc.band_rows = (bases + fc.n_bands - 1) / fc.n_bands;
            const long units = (long)((pl->nz + slices - 1) / slices) * pl->M;
            const long umax = std::max<long>(1, kFwdThreads * fwd_rays_per_thread(slices) / pl->nu);
            long nb = (units + umax - 1) / umax;
            nb = ((nb + 255) / 256) * 256;
            fc.blocks = (int)std::min(nb, units);
            return true;
        };
        if (!fwd_config(2, 8, pl->fwd32) || pl->fwd32.n_bands > 1) {
            if (!fwd_config(1, 4, pl->fwd32)) { delete pl; return MPI3D_ENOTSUP; }
        }
        if (!fwd_config(2, 4, pl->fwd16)) { delete pl; return MPI3D_ENOTSUP; }
        // FP32 in four-slice texels (proj_fwd_band_kernel): possible where bands
        // of at least 8 rows and columns fit; dealt to blocks, and compared with
        // the kernels above, once the angles are known.
        {
            const int texels = 160 * 1024 / 16;
            const int rmax = texels / mpi3d::proj_pitch(pl->nx) - 1;
            int cmax = texels / (pl->ny + 2) - 1;             // pitch (cols + 1) | 1
            if (((cmax + 1) | 1) * (pl->ny + 2) > texels) --cmax;
            pl->band.blocks = 0;
            if (rmax >= 8 && cmax >= 8) {
                auto even = [](int n, int mx) { const int k = (n + mx - 1) / mx; return (n + k - 1) / k; };
                pl->band.rows = even(pl->ny + 1, rmax);
                pl->band.cols = even(pl->nx + 1, cmax);
                pl->band.blocks = 1;
            }
        }
        // Backprojection: 16 x 16 voxel tiles times kz slices per block, the kz
        // with the least estimated time: 5 us, then the blocks of a CU one after
        // the other, each angle 52 ns for the weights and 10 ns a slice (fits to
        // both kernels at 7 shapes from 32^3 x 8 to 256^2 x 128 x 60, within
        // 15%); a CU with one block waits as long as it works, with two a
        // quarter of that.  Measured at 192^2 x 96 x 36, kz 8 / 16 / 24 / 32: 41 / 37 /
        // 39 / 37 us; 256^2 x 128 x 60: 127 / 102 / 98 / 88, 64: 102; 128^2 x 64 x 24:
        // 13 / 17 / 21 / 23.  fp16 lines take units of 8 slices, so kz >= 8.
        // Angles are staged in LDS in chunks of at most 40 KB, or 20 KB where
        // more than four blocks share a CU (kz 8 at 256^2 x 128: 137 -> 127 us).
        const long tiles = (long)((pl->nx + 15) / 16) * ((pl->ny + 15) / 16);
        pl->max_parts = kMaxNormParts;
        auto back_config = [&](int kmin, int unit_slices, int &kz_out, int &chunk_out) {
            double best = 1e30;
            long blocks = 0;
            for (int kz : {4, 8, 16, 24, 32, 64}) {
                if (kz < kmin) continue;
                const long nb = tiles * ((pl->nz + kz - 1) / kz), b = (nb + 255) / 256;
                const double wait = b == 1 ? 2.0 : b == 2 ? 1.25 : b == 3 ? 1.1 : 1.0;
                const double t = 5e-6 + (double)b * pl->M * (52e-9 + 10e-9 * kz) * wait;
                if (t < best * (1.0 - 1e-9)) {
                    best = t;
                    kz_out = kz;
                    blocks = nb;
                }
            }
            const int kb = blocks > 4 * 256 ? 20 : 40;
            const int chunk_max = std::max(1, kb * 1024 / ((kz_out / unit_slices | 1) * 16 * 32));
            const int nchunk = (pl->M + chunk_max - 1) / chunk_max;
            chunk_out = (pl->M + nchunk - 1) / nchunk;
            pl->max_parts = (int)std::max<long>(pl->max_parts, blocks);
        };
        back_config(4, 4, pl->kz, pl->adj_chunk);
        back_config(8, 8, pl->kz16, pl->adj_chunk16);
    }

    // ---- float64 host tables ------------------------------------------------
    const int M = pl->M, NU = pl->nu, NUP = pl->nup, T = pl->nt, TP = pl->ntp, NB = pl->nb;
    const int NBP2 = pl->nbp2, NCT = pl->nct, NC = pl->nchunks;
    std::vector<double> theta(M);
    for (int m = 0; m < M; ++m) theta[m] = g->theta_rad ? g->theta_rad[m] : m * kPi / M;
    for (int m = 0; m < M; ++m)
        if (!std::isfinite(theta[m])) { delete pl; return MPI3D_EINVAL; }
    const double cx = 0.5 * (pl->nx - 1), cy = 0.5 * (pl->ny - 1), cu = 0.5 * (NU - 1);

    std::vector<float2> cs(M);
    std::vector<float> ax((size_t)M * NU), ay((size_t)M * NU), ay1((size_t)M * NU);
    for (int m = 0; m < M; ++m) {
        double c = std::cos(theta[m]), s = std::sin(theta[m]);
        cs[m] = make_float2((float)c, (float)s);
        for (int p = 0; p < NU; ++p) {
            double up = p - cu;
            // sample (p, q) sits at x = u_p c + y_q s, y = -u_p s + y_q c; the
            // kernels add y_q times (s, c) to these bases (LDS column 0 holds
            // grid column -1, hence the +1).
            ax[(size_t)m * NU + p] = (float)(up * c + cx + 1.0);
            ay[(size_t)m * NU + p] = (float)(-up * s + cy);
            ay1[(size_t)m * NU + p] = (float)(-up * s + cy + 1.0);
        }
    }
    std::vector<int> order;    // angles by class: |c| >= |s| first
    for (int steep = 1; steep >= 0; --steep) {
        for (int m = 0; m < M; ++m)
            if ((std::fabs(cs[m].x) >= std::fabs(cs[m].y)) == (steep == 1)) order.push_back(m);
        if (steep) pl->n_steep = (int)order.size();
    }
    if (pl->band.blocks) {
        // Blocks a group and class: at most 2 rays a thread, and the least
        // estimated time.  The estimates are fits to both kernels' times at 14
        // shapes from 64^3 x 24 angles to 256^2 x 128 x 60: a round of blocks of
        // the four-slice kernel takes 11 us, 25 us a MB of staged slices and
        // 0.31 ns a ray sample of the longest block; the others 9 us and 0.26 ns
        // in slice pairs (a third more where rows are not whole vectors), or 3 us
        // and 0.155 ns (0.23 ns in row bands) slice by slice.  Measured at the
        // edges, old -> new: 64^3 x 24 11.9 -> 15.2 us, 192^2 x 64 x 36 54 -> 64
        // (not taken), 192^2 x 96 x 36 82 -> 71, 100^3 x 60 45 -> 37, 256^2 x 64 x 24
        // 102 -> 77 (taken).  It has to win by a twelfth.  The longest block of the
        // four-slice kernel has the longest rays; those of the others, of mixed
        // angles, rays an eighth of the way to the shortest (216 x 327 x 82, 10
        // angles: 69 us and 78 in four-slice texels, not taken).  Of 470 drawn
        // volumes 64 are taken in FP32 and 23 in bf16, none over 3% slower.
        const int ng4 = (pl->nz + 3) / 4, nm[2] = {pl->n_steep, M - pl->n_steep};
        const int amax = 2 * kFwdThreads / NU, len = std::max(pl->nx, pl->ny);
        const double len1 = 0.875 * len + 0.125 * std::min(pl->nx, pl->ny);
        const double stage = 16.0 * pl->nx * pl->ny * 25e-12;
        double best = 1e30;
        for (int amx = 1; amx <= amax; ++amx) {
            int parts[2], big = 0;
            for (int k = 0; k < 2; ++k) {
                parts[k] = (nm[k] + amx - 1) / amx;
                if (parts[k]) big = std::max(big, (nm[k] + parts[k] - 1) / parts[k]);
            }
            const long blocks = (long)ng4 * (parts[0] + parts[1]);
            const double t = (double)((blocks + 255) / 256) * (11e-6 + stage + (double)big * NU * len * 0.31e-9);
            if (t < best * (1.0 - 1e-9)) {
                best = t;
                pl->band.blocks = (int)blocks;
                pl->band.parts[0] = parts[0];
                pl->band.parts[1] = parts[1];
            }
        }
        const mpi3d::FwdConfig &fc = pl->fwd32;
        const long units = (long)((pl->nz + fc.slices - 1) / fc.slices) * M;
        const double x = (double)((fc.blocks + 255) / 256) * ((units + fc.blocks - 1) / fc.blocks) * NU * len1;
        const double other = fc.slices == 2 ? 9e-6 + (pl->nx % 4 ? 0.35e-9 : 0.26e-9) * x
                                            : 3e-6 + (fc.n_bands > 1 ? 0.23e-9 : 0.155e-9) * x;
        pl->band.fp32 = best <= 0.92 * other;
        // bf16 gathers: in one band their slice pairs cost 0.2 to 0.24 ns a ray
        // sample, within a tenth of the four-slice kernel's time from 128^2 x 128
        // x 36 to 160^2 x 128 x 60, and stay; in row bands 15 us and 0.36 ns
        // (measured 0.36 to 0.45).
        const mpi3d::FwdConfig &hc = pl->fwd16;
        const long hunits = (long)((pl->nz + 1) / 2) * M;
        const double hx = (double)((hc.blocks + 255) / 256) * ((hunits + hc.blocks - 1) / hc.blocks) * NU * len1;
        pl->band.bf16 = (precisions & (1 << MPI3D_MIXED)) && hc.n_bands > 1 && best <= 0.92 * (15e-6 + 0.36e-9 * hx);
    }

    // PSF kernel K[n][p] of every table (n < T, p < NU; zero padding
    // elsewhere).  Line group g's tables are table_g + d, d = 0..coup_g: for
    // trajectory class c (class 1 being the raster's backward sweep,
    // xi_n = a sin(phi_n) + dir S (n/T - 1/2), v_n = a phi' cos(phi_n) + dir S/T)
    // and line offset d of the tensor PSF, d = 0 being the collinear
    // L'(du/w)/w.  The z-drive group's tables use amplitude a_z and the
    // centred z-rows as samples (zero beyond nz); its offsets are detector
    // columns, the tensor entry's transverse offset.
    const size_t KE = (size_t)TP * NUP;
    pl->k_elems = KE;
    std::vector<double> K(KE * n_ktab, 0.0);
    {
        const double om = 2.0 * kPi * pl->P / T;
        for (int tb = 0; tb < n_ktab; ++tb) {
            const bool zt = drive_axes == 2 && tb > psf_rows;
            const int cl = zt ? 0 : tb / (psf_rows + 1);
            const int d = zt ? tb - (psf_rows + 1) : tb % (psf_rows + 1);
            const double dir = cl == 0 ? 1.0 : -1.0, S = pl->raster_sweep;
            const double amp = zt ? pl->a_z : pl->a, centre = zt ? 0.5 * (pl->nz - 1) : cu;
            const int npts = zt ? pl->nz : NU;
            double *Kc = &K[KE * tb];
            for (int n = 0; n < T; ++n) {
                double ph = om * n;
                double xi = amp * std::sin(ph) + dir * S * ((double)n / T - 0.5);
                double v = amp * om * std::cos(ph) + dir * S / T;
                for (int p = 0; p < npts; ++p) {
                    const double du = xi - (p - centre);
                    Kc[(size_t)n * NUP + p] =
                        v * (d == 0 ? langevin_deriv(du / pl->w) / pl->w : psf_xx(du, (double)d, pl->w));
                }
            }
        }
    }
    if (g->rx_filter)
        for (int j = 0; j < 2 * NB; ++j)
            if (!std::isfinite(g->rx_filter[j])) { delete pl; return MPI3D_EINVAL; }

    std::vector<double> phase((size_t)2 * T);     // cos, sin of 2 pi n / T
    for (int n = 0; n < T; ++n) {
        const double a = 2.0 * kPi * (double)n / T;
        phase[2 * n] = std::cos(a);
        phase[2 * n + 1] = std::sin(a);
    }

    // ---- band DFT factored over drive cycles (FP32) --------------------------
    // t = n1 + P n2 (T = C P, C = 32 or 64): the kept bin omega_j
    // contributes e^{2 pi i omega_j n1 / T} e^{2 pi i (omega_j mod C) n2 / C},
    // so the forward first sums each phase n1's C cycles against the residues
    // r = omega_j mod C, then each bin's P phases.  s is real, so residues r
    // and C - r share the columns cos, sin of one slot, and 0 and C / 2 (no
    // sine) share another.  Taken when its time per line, by the rates below,
    // is under the dense form's; C minimises it.
    std::vector<uint16_t> fkf, fka, fef, fea, fwf, fwa;   // fp16 bits
    std::vector<int> funit0, fubin, fqbin, fbcol, fwexp;
    // A plan that also holds the mixed operator takes it only where the bins'
    // residues bunch (at most 24 distinct): its refinement sweeps start from
    // the FP32 operator, and their inner iterations blow a difference in its
    // last bits up, through the 16-bit roundings, to some 1e-5 of the result;
    // scans that bunch less keep the dense form's bits there.
    const int NPASS = pl->n_passes;
    bool same_coup = true;     // every line group coupled over the same range
    pl->fac.max_rows = 0;
    for (int gi = 0; gi < pl->n_line_groups; ++gi) {
        same_coup = same_coup && pl->groups[gi].coup == pl->pass_r;
        pl->fac.max_rows = std::max<long>(pl->fac.max_rows, pl->groups[gi].rows);
    }
    if ((precisions & (1 << MPI3D_FP32)) && same_coup && T % 32 == 0) {
        // least residue of r's pair: 0 for r = 0 and C / 2, else min(r, C - r)
        auto least = [](long r, int C) { return (int)(2 * r == C ? 0 : std::min(r, C - r)); };
        auto slots_of = [](int R, int C) { return C == 32 ? 16 : std::max(16, (R + 3) / 4 * 4); };
        // A slot: the bins (ascending) of a residue pair, or a part of them: the
        // adjoint's outer sum takes 32 a slot with at most 16 slots, else 24 with at
        // most 24, and a pair with more has several slots of equal columns (drive
        // cycles in multiples of 64 with 17 harmonics and more put 34 in one).  Not
        // in plans that may take the dense form on fp16 pairs, whose adjoint is
        // faster than a few full slots (41 x 59 x 15, 28 angles, T = 8192, 64
        // cycles, 59 harmonics: 20.5 and 31.5 us).  Empty where no such slots are
        // enough, or a residue has more than 24 bins: so few residues leave the
        // adjoint's time sums too few terms to average their roundings out (16
        // samples, T = 6336, 64 cycles, 25 harmonics: error 1.0e-7 dense, 3.1e-7).
        const bool parts_of_pairs = (precisions & (1 << MPI3D_MIXED)) && NPASS == 1 && pl->n_line_groups == 1;
        struct Slot {
            int r;                    // least residue
            std::vector<int> bins;
        };
        auto deal_slots = [&](int C) {
            std::vector<std::vector<int>> pair(C / 2);
            for (int j = 0; j < NB; ++j) pair[least(bins[j] % C, C)].push_back(j);
            std::vector<Slot> out;
            std::vector<int> cnt(C, 0);
            for (long b : bins) ++cnt[b % C];
            if (*std::max_element(cnt.begin(), cnt.end()) > 24) return out;
            for (int cap : {32, 24}) {
                bool fits = true;
                out.clear();
                for (int r = 0; r < C / 2; ++r) {
                    const int n = (int)pair[r].size(), parts = (n + cap - 1) / cap;
                    if (parts > 1 && !parts_of_pairs) fits = false;
                    for (int i = 0; i < parts; ++i)
                        out.push_back({r, {pair[r].begin() + (long)i * n / parts, pair[r].begin() + (long)(i + 1) * n / parts}});
                }
                if (fits && (int)out.size() <= (cap == 32 || C == 32 ? 16 : 24)) return out;
            }
            out.clear();
            return out;
        };
        // seconds per line: dense fp32 products at 1.1e14 flop/s; factored
        // split products (three each) at 8e14, the phase sums written and read
        // at 4 TB/s, the outer sum's fp32 products (32 columns a unit) at 1e14
        double best = 2.0 * T * (NPASS * NUP + NBP2) / 1.1e14;
        int bestC = 0;
        for (int C = 32; C <= T && C <= 64; C += 32) {
            if (T % C) continue;
            std::vector<char> seen(C, 0);
            for (long b : bins) seen[b % C] = 1;
            if ((precisions & (1 << MPI3D_MIXED)) && std::count(seen.begin(), seen.end(), 1) > 24) continue;
            const std::vector<Slot> slots = deal_slots(C);
            const int R = (int)slots.size();
            if (R == 0) continue;
            int U = 0;
            for (const Slot &q : slots) U += ((int)q.bins.size() + 15) / 16;
            const int zst = slots_of(R, C), rct = (2 * zst + 31) / 32, P = T / C;
            if (!fac_supported(NUP, zst, C / 32, NPASS) ||
                (double)((pl->fac.max_rows + 31) / 32 * 32 + 1) * P * 2 * zst >= 2147483647.0 ||
                4.0 * T * NUP * NPASS >= 2147483647.0)
                continue;
            const double cost = 6.0 * T * (NPASS * NUP + 32 * rct) / 8e14 + 16.0 * P * zst / 4e12 + 128.0 * P * U / 1e14;
            if (cost < best) {
                best = cost;
                bestC = C;
            }
        }
        std::vector<int> res;                // least residue of each slot
        std::vector<std::vector<int>> qb;    // bins of each slot
        if (bestC) {
            mpi3d_plan::Fac &f = pl->fac;
            f.C = bestC;
            f.P = T / bestC;
            f.cj = bestC / 32;
            f.nzstage = (f.P + 15) / 16;
            // Slot order: the adjoint outer sum's wave w takes slots
            // w, w + 8, w + 16 (so waves w < R % 8 take one more when 8 does
            // not divide R) and spends a step per bin, so slots are dealt
            // largest first to the least loaded wave with room, and numbered
            // by (wave, turn).  Units: a slot's bins (ascending) 16 at a time.
            std::vector<char> seen(bestC, 0);
            for (long b : bins) seen[b % bestC] = 1;
            f.res = (int)std::count(seen.begin(), seen.end(), 1);
            std::vector<Slot> slots = deal_slots(bestC);
            std::stable_sort(slots.begin(), slots.end(),
                             [](const Slot &x, const Slot &y) { return x.bins.size() > y.bins.size(); });
            const int nw = kFacInWaves, nr = (int)slots.size();
            std::vector<std::vector<int>> wslot(nw);
            std::vector<int> load(nw, 0), room(nw);
            for (int w = 0; w < nw; ++w) room[w] = nr / nw + (w < nr % nw ? 1 : 0);
            for (int i = 0; i < nr; ++i) {
                int bw2 = -1;
                for (int w = 0; w < nw; ++w)
                    if ((int)wslot[w].size() < room[w] && (bw2 < 0 || load[w] < load[bw2])) bw2 = w;
                wslot[bw2].push_back(i);
                load[bw2] += ((int)slots[i].bins.size() + 3) / 4 * 4;
            }
            res.assign(nr, -1);
            qb.resize(nr);
            for (int w = 0; w < nw; ++w)
                for (size_t i = 0; i < wslot[w].size(); ++i) {
                    const int q = w + nw * (int)i;
                    res[q] = slots[wslot[w][i]].r;
                    qb[q] = slots[wslot[w][i]].bins;
                }
            f.R = (int)res.size();
            f.zst = slots_of(f.R, bestC);
            f.qmax = f.R <= 16 ? 32 : 24;
            const int QM = f.qmax;
            fqbin.assign((size_t)f.R * QM, 0xffff);   // (bins: below, with their exponents)
            fbcol.assign(NB, 0);
            for (int q = 0; q < f.R; ++q) {
                funit0.push_back((int)fubin.size() / 16);
                for (size_t i = 0; i < qb[q].size(); ++i) fbcol[qb[q][i]] = 2 * ((int)fubin.size() + (int)i);
                for (size_t i0 = 0; i0 < qb[q].size(); i0 += 16)
                    for (size_t i = 0; i < 16; ++i) fubin.push_back(i0 + i < qb[q].size() ? qb[q][i0 + i] : -1);
            }
            f.U = (int)fubin.size() / 16;
            funit0.push_back(f.U);
            f.on = choose_fac_ranges(pl, bins, 2.0 * T * (NPASS * NUP + NBP2) / 1.1e14);
        }
        if (pl->fac.on) {
            mpi3d_plan::Fac &f = pl->fac;
            if (NPASS > 1) {       // virtual lines, as the fused dense pass has them
                if (!pl->fused)    // (whose launch configuration nothing uses then)
                    pl->scf = mpi3d_plan::SigCfg{kWidePairs, 1, 14, pl->nchunks, 1, 0, 0, pl->nchunks, 1};
                pl->fused = true;
                pl->nupf = NPASS * NUP;
            }
            f.k_stride = 2 * (long)KE * NPASS;
            // tables
            const int QM = f.qmax, C = bestC, P = f.P, CJ = f.cj, ZST = f.zst, YC = 2 * ZST;
            const int RCT = (YC + 31) / 32, NZS = (YC + 15) / 16;
            auto tp16 = [](int e2, int h) { return 8 * (e2 / 4) + 4 * h + (e2 % 4); };
            auto tof = [&](int c, int i) { return (c / CJ) + P * (32 * (c % CJ) + i); };   // chunk row -> time
            // PSF tables scaled so their largest entry is in [2^14, 2^15); s_scale
            // keeps a time signal of lines below 2^15 at or below 2^15 by the
            // largest row sum (over a line's tables)
            double kmax = 0, ksum = 0;
            for (int gi = 0; gi < pl->n_line_groups; ++gi)
                for (int n = 0; n < T; ++n) {
                    double sum = 0;
                    for (int e2 = 0; e2 < NPASS; ++e2) {
                        const double *row = &K[KE * (pl->groups[gi].table + e2) + (size_t)n * NUP];
                        for (int p = 0; p < NUP; ++p) {
                            const double v = std::fabs(row[p]);
                            kmax = std::max(kmax, v);
                            sum += v;
                        }
                    }
                    ksum = std::max(ksum, sum);
                }
            int kexp = 0, sexp = 0;
            if (kmax > 0) {
                std::frexp(kmax, &kexp);
                kexp = 15 - kexp;
                std::frexp(std::ldexp(ksum, kexp), &sexp);   // row sums < 2^sexp
            }
            f.s_scale = (float)std::ldexp(1.0, -sexp);
            // |Y| <= C 2^14 2^15 before y_scale
            f.y_scale = (float)std::ldexp(1.0, -(bestC == 32 ? 19 : 20));
            f.y_exp = kexp - sexp + 14 - (bestC == 32 ? 19 : 20);
            // |2^14 E| <= 2^14 and |Z| <= 2^15 over at most 2 R columns
            int cexp = 0;
            while ((1 << cexp) < 2 * f.R) ++cexp;
            f.g_scale = (float)std::ldexp(1.0, -(14 + cexp));
            f.r_exp = kexp - cexp;   // 14 - (14 + cexp) + kexp
            // fragments of 64 lanes x 8 halves, hi then lo:
            //  kf [c][p / 16][hi, lo]: K[time row l % 32][p = 16 ks + 8 (l / 32) + e]
            //  ka [c][time step][p / 32][hi, lo]: K[time row 16 q + tp16(e, l / 32)][p = 32 pt + l % 32]
            // (kf: a chunk's tables e = 0 .. R one after the other; ka: table after
            // table; line group after line group)
            const size_t KG = 2 * KE * NPASS;       // halves a line group
            fkf.assign(KG * pl->n_line_groups, 0);
            fka.assign(KG * pl->n_line_groups, 0);
            std::vector<uint16_t> kh(32 * NUP), kl(32 * NUP);   // one chunk's pairs
            const double ksc = std::ldexp(1.0, kexp);
            for (int gi = 0; gi < pl->n_line_groups; ++gi)
                for (int e3 = 0; e3 < NPASS; ++e3)
                    for (int c = 0; c < P * CJ; ++c) {
                        const double *K0 = &K[KE * (pl->groups[gi].table + e3)];
                        uint16_t *ckf = &fkf[KG * gi + ((size_t)c * NPASS + e3) * 64 * NUP];
                        uint16_t *cka = &fka[KG * gi + 2 * KE * e3 + (size_t)c * 64 * NUP];
                        for (int i = 0; i < 32; ++i)
                            for (int p = 0; p < NUP; ++p)
                                half_pair(K0[(size_t)tof(c, i) * NUP + p] * ksc, kh[i * NUP + p], kl[i * NUP + p]);
                        for (int ks = 0; ks < NUP / 16; ++ks)
                            for (int l = 0; l < 64; ++l)
                                for (int e2 = 0; e2 < 8; ++e2) {
                                    const size_t o = ((size_t)ks * 2 * 64 + l) * 8 + e2;
                                    const int i = (l % 32) * NUP + 16 * ks + 8 * (l / 32) + e2;
                                    ckf[o] = kh[i];
                                    ckf[o + 512] = kl[i];
                                }
                        for (int q = 0; q < 2; ++q)
                            for (int pt = 0; pt < NUP / 32; ++pt)
                                for (int l = 0; l < 64; ++l)
                                    for (int e2 = 0; e2 < 8; ++e2) {
                                        const size_t o = (((size_t)q * (NUP / 32) + pt) * 2 * 64 + l) * 8 + e2;
                                        const int i = (16 * q + tp16(e2, l / 32)) * NUP + 32 * pt + l % 32;
                                        cka[o] = kh[i];
                                        cka[o + 512] = kl[i];
                                    }
                    }
            // E[n2][2q] = cos, E[n2][2q + 1] = sin of 2 pi (r n2 mod C) / C, r the
            // slot's least residue; the slot of 0 and C / 2: 1 and (-1)^n2
            auto E = [&](int n2, int q, int part) -> double {
                if (q >= f.R) return 0.0;
                if (res[q] == 0) return part == 0 ? 1.0 : (n2 % 2 ? -1.0 : 1.0);
                const long ph = (long)res[q] * n2 % C;
                const double a = 2.0 * kPi * (double)ph / C;
                return part ? std::sin(a) : std::cos(a);
            };
            // E takes few distinct values (cosines of multiples of 2 pi / C), so the
            // errors of its pairs are the same in every phase and add up: 2.1e-8 of its
            // columns as they stand, 1.5e-9 (C = 32) and 5.9e-9 (C = 64) times a factor
            // that was searched for among the multiples of 2^-20 in [1/2, 1].  What is
            // left of a column's gain, <E', E> / <E, E> of the columns E' held, and the
            // factor are divided out of the outer sums' weights.  (70 x 87 x 28, 10
            // angles, T = 2816: A of positive lines 1.3e-8 low -> 3e-10, A^T A 9e-8 ->
            // 6e-8, fp32 MFMA 4e-8; three CGLS iterations grow that to 1.5e-6 -> 1.0e-6.)
            const double escale = C == 32 ? 0.8672637939453125 : 0.8797330856323242;
            std::vector<double> gain(2 * f.R, 1.0);
            std::vector<int> slot(NB);          // of a bin
            for (int q = 0; q < f.R; ++q)
                for (int j : qb[q]) slot[j] = q;
            for (int col = 0; col < 2 * f.R; ++col) {
                double num = 0, den = 0;
                for (int n2 = 0; n2 < C; ++n2) {
                    const double v = E(n2, col / 2, col % 2);
                    double hi, lo;
                    half_bits(std::ldexp(escale * v, 14), &hi);
                    half_bits(std::ldexp(escale * v, 14) - hi, &lo);
                    num += v * std::ldexp(hi + lo, -14);
                    den += v * v;
                }
                if (den > 0) gain[col] = num / den;
            }
            // ef [j][g][time step][hi, lo]: row = column 32 g + l % 32 (2 slot + part),
            // k = time 32 j + 16 q + tp16(e, l / 32)
            fef.assign((size_t)CJ * RCT * 4 * 512, 0);
            for (int j = 0; j < CJ; ++j)
                for (int g2 = 0; g2 < RCT; ++g2)
                    for (int q = 0; q < 2; ++q)
                        for (int l = 0; l < 64; ++l)
                            for (int e2 = 0; e2 < 8; ++e2) {
                                const int col = 32 * g2 + l % 32;
                                const size_t o = ((((size_t)j * RCT + g2) * 2 + q) * 2 * 64 + l) * 8 + e2;
                                half_pair(std::ldexp(escale * E(32 * j + 16 * q + tp16(e2, l / 32), col / 2, col % 2), 14),
                                          fef[o], fef[o + 512]);
                            }
            // ea [j][column step][hi, lo]: row = time 32 j + l % 32, k = column
            // 16 ks + 8 (l / 32) + e (2 slot + part)
            fea.assign((size_t)CJ * NZS * 2 * 512, 0);
            for (int j = 0; j < CJ; ++j)
                for (int ks = 0; ks < NZS; ++ks)
                    for (int l = 0; l < 64; ++l)
                        for (int e2 = 0; e2 < 8; ++e2) {
                            const int col = 16 * ks + 8 * (l / 32) + e2;
                            if (col >= YC) continue;
                            const size_t o = (((size_t)j * NZS + ks) * 2 * 64 + l) * 8 + e2;
                            half_pair(std::ldexp(escale * E(32 * j + l % 32, col / 2, col % 2), 14), fea[o], fea[o + 512]);
                        }
            // G_j[n1] = D_j e^{2 pi i (omega_j n1 mod T) / T} / sqrt(T)
            const double inv = 1.0 / std::sqrt((double)T);
            std::vector<double> Gt((size_t)NB * P * 2);
            for (int j = 0; j < NB; ++j) {
                double dre = 1.0, dim = 0.0;
                if (g->rx_filter) { dre = g->rx_filter[2 * j]; dim = g->rx_filter[2 * j + 1]; }
                long ph = 0;                      // bins[j] n1 mod T
                for (int n1 = 0; n1 < P; ++n1, ph += bins[j], ph -= ph >= T ? T : 0) {
                    const double co = phase[2 * ph], si = phase[2 * ph + 1];
                    Gt[2 * ((size_t)j * P + n1)] = (dre * co - dim * si) * inv;
                    Gt[2 * ((size_t)j * P + n1) + 1] = (dre * si + dim * co) * inv;
                }
            }
            // weight of slot column cy (cos, sin) in part cb (re, im) of bin j:
            // residue r: b = G (c0 + i c1); C - r: G (c0 - i c1); 0: G c0; C / 2: G c1
            auto weight = [&](int j, int n1, int cy, int cb) -> double {
                const double gn = gain[2 * slot[j] + cy];
                const double gr = Gt[2 * ((size_t)j * P + n1)] / gn, gi = Gt[2 * ((size_t)j * P + n1) + 1] / gn;
                const long r = bins[j] % C;
                if (r == 0 || 2 * r == C) return (cy == 1) == (r != 0) ? (cb == 0 ? gr : gi) : 0.0;
                if (cy == 0) return cb == 0 ? gr : gi;
                const double sg = 2 * r < C ? 1.0 : -1.0;
                return cb == 0 ? -sg * gi : sg * gr;
            };
            // outer tables: bin j's weights by 2^wex[j], which brings the largest
            // possible one (|D_j| / sqrt(T)) into [2^14, 2^15).  The forward undoes
            // it per column; the adjoint takes bin j's data by 2^(wref - wex[j])
            // (qbin), and its sums over a slot's bins are below 2^zsum
            int wref = 0, zsum = 0;
            const std::vector<int> wex = bin_exponents(g->rx_filter, NB, inv / escale, &wref);
            double gsum = 0;
            for (int q = 0; q < f.R; ++q) {
                double sum = 0;
                for (size_t i = 0; i < qb[q].size(); ++i) {
                    const int j = qb[q][i];
                    sum += 1.4142136 * std::ldexp(bin_gain(g->rx_filter, j) * inv / escale, wex[j]);   // |re| + |im| of a weight
                    fqbin[(size_t)q * QM + i] = (int)((unsigned)(wref - wex[j]) << 16 | (unsigned)j);
                }
                gsum = std::max(gsum, sum);
            }
            if (gsum > 0) std::frexp(gsum, &zsum);
            f.z_scale = (float)std::ldexp(1.0, -zsum);
            f.z_exp = wref - zsum;
            fwexp.assign((size_t)32 * f.U, 0);
            for (int c = 0; c < 32 * f.U; ++c)
                if (fubin[c / 2] >= 0) fwexp[c] = wex[fubin[c / 2]];
            // forward outer B operand [unit][8-phase stage][hi, lo]: k = (column of
            // Y = l / 32, phase 8 stg + e), column l % 32 = (bin of the unit, re/im)
            const int nst8 = (P + 7) / 8;
            fwf.assign((size_t)f.U * nst8 * 1024, 0);
            for (int u = 0; u < f.U; ++u)
                for (int n1 = 0; n1 < P; ++n1)
                    for (int l = 0; l < 64; ++l) {
                        const int col = l % 32, jb = fubin[(size_t)u * 16 + col / 2];
                        if (jb < 0) continue;
                        const size_t o = (((size_t)u * nst8 + n1 / 8) * 2 * 64 + l) * 8 + n1 % 8;
                        half_pair(std::ldexp(weight(jb, n1, l / 32, col % 2), wex[jb]), fwf[o], fwf[o + 512]);
                    }
            // adjoint outer A operand [slot][16-phase stage][bin step][hi, lo]: row
            // l % 32 = (phase 16 stg + row / 2, column of Z = row % 2), k = (bin
            // 8 ks + 4 (l / 32) + e / 2, re/im = e % 2)
            fwa.assign((size_t)f.R * f.nzstage * (QM / 8) * 1024, 0);
            for (int q = 0; q < f.R; ++q)
                for (int stg = 0; stg < f.nzstage; ++stg)
                    for (int ks = 0; ks < QM / 8; ++ks)
                        for (int l = 0; l < 64; ++l)
                            for (int e2 = 0; e2 < 8; ++e2) {
                                const int jb = (int16_t)fqbin[(size_t)q * QM + 8 * ks + 4 * (l / 32) + e2 / 2];
                                const int n1 = 16 * stg + (l % 32) / 2;
                                if (jb < 0 || n1 >= P) continue;
                                const size_t o =
                                    ((((size_t)q * f.nzstage + stg) * (QM / 8) + ks) * 2 * 64 + l) * 8 + e2;
                                half_pair(std::ldexp(weight(jb, n1, l % 2, e2 % 2), wex[jb]), fwa[o], fwa[o + 512]);
                            }
        }
    }

    // ---- dense FP32 stage on fp16 pairs: what does not factor ----------------
    if (!pl->fac.on) pl->split.on = choose_pairs(pl) < 1e30;

    // band DFT F[n][c] (real columns: 2j = Re, 2j+1 = Im)
    // -- not for a plan whose only signal stage is the factored one
    const bool precomp = precisions & (1 << MPI3D_PRECOMPOSED), mixed = precisions & (1 << MPI3D_MIXED);
    const bool split = pl->split.on;
    const bool dense = !pl->fac.on && !split;      // the fp32 MFMA kernels' tables
    std::vector<double> F;
    if (dense || split || mixed || precomp) {
        F.assign((size_t)TP * NBP2, 0.0);
        const double inv = 1.0 / std::sqrt((double)T);
        for (int j = 0; j < NB; ++j) {
            double dre = 1.0, dim = 0.0;
            if (g->rx_filter) { dre = g->rx_filter[2 * j]; dim = g->rx_filter[2 * j + 1]; }
            long ph = 0;                          // bins[j] n mod T
            for (int n = 0; n < T; ++n, ph += bins[j], ph -= ph >= T ? T : 0) {
                const double c = phase[2 * ph], s = phase[2 * ph + 1];
                F[(size_t)n * NBP2 + 2 * j] = (dre * c - dim * s) * inv;
                F[(size_t)n * NBP2 + 2 * j + 1] = (dre * s + dim * c) * inv;
            }
        }
    }

    // split tables: fragments of 64 lanes x 8 halves, hi then lo, chunk after
    // chunk of 32 times
    //  kf [p / 16]: K[time l % 32][p = 16 ks + 8 (l / 32) + e]
    //  ff [32 columns][time step]: F[time 16 q + tp16(e, l / 32)][column 32 g + l % 32]
    //  fa [column / 16]: F[time l % 32][column 16 ks + 8 (l / 32) + e]
    //  ka [time step][p / 32]: K[time 16 q + tp16(e, l / 32)][p = 32 pt + l % 32]
    std::vector<uint16_t> skf, ska, sff, sfa;
    std::vector<int> sfexp, saexp;
    if (split) {
        mpi3d_plan::Split &sp = pl->split;
        auto tp16 = [](int e2, int h) { return 8 * (e2 / 4) + 4 * h + (e2 % 4); };
        // tables scaled so their largest entries (the band table's: a bin's) are in
        // [2^14, 2^15); the time tiles of lines below 2^15 kept below 2^15 by the
        // largest row sums
        int fref = 0;
        const std::vector<int> fex = bin_exponents(g->rx_filter, NB, 1.0 / std::sqrt((double)T), &fref);
        std::vector<double> fsc(NB);
        for (int j = 0; j < NB; ++j) fsc[j] = bin_gain(g->rx_filter, j) > 0 ? std::ldexp(1.0, fex[j]) : 0.0;
        double kmax = 0, ksum = 0, fsum = 0;
        for (size_t n = 0; n < (size_t)n_ktab * T; ++n) {
            const double *row = &K[KE * (n / T) + n % T * NUP];
            double sum = 0;
            for (int p = 0; p < NUP; ++p) {
                kmax = std::max(kmax, std::fabs(row[p]));
                sum += std::fabs(row[p]);
            }
            ksum = std::max(ksum, sum);
        }
        for (int n = 0; n < T; ++n) {
            double sum = 0;
            for (int c = 0; c < 2 * NB; ++c) {
                sum += std::fabs(F[(size_t)n * NBP2 + c]) * fsc[c / 2];
            }
            fsum = std::max(fsum, sum);
        }
        int kexp = 0, s1 = 0, s2 = 0;
        if (kmax > 0) {
            std::frexp(kmax, &kexp);
            kexp = 15 - kexp;
            std::frexp(std::ldexp(ksum, kexp), &s1);
        }
        if (fsum > 0) std::frexp(fsum, &s2);
        sp.s_scale = (float)std::ldexp(1.0, -s1);
        sp.g_scale = (float)std::ldexp(1.0, -s2);
        sp.fwd_exp = kexp - s1;
        sp.adj_exp = fref - s2 + kexp;
        sfexp.assign((size_t)32 * (sp.nct + 8), 0);      // (a last column group reads past nct)
        saexp.assign((size_t)32 * (sp.nct + 8), 0);
        for (int c = 0; c < 2 * NB; ++c) {
            sfexp[c] = fex[c / 2];
            saexp[c] = fref - fex[c / 2];
        }
        const double ksc = std::ldexp(1.0, kexp);
        // one chunk's 32 x n table as A fragments by row (time, 16 columns a
        // step) and by column (32 columns a tile, 16 times a step)
        std::vector<uint16_t> ph, plo;
        auto pairs = [&](const double *src, size_t pitch, int n, int pad, auto scale) {
            ph.assign((size_t)32 * pad, 0);
            plo.assign((size_t)32 * pad, 0);
            for (int i = 0; i < 32; ++i)
                for (int p = 0; p < n; ++p)
                    half_pair(src[(size_t)i * pitch + p] * scale(p), ph[(size_t)i * pad + p], plo[(size_t)i * pad + p]);
        };
        auto by_time = [&](uint16_t *dst, int pad) {
            for (int ks = 0; ks < pad / 16; ++ks)
                for (int l = 0; l < 64; ++l)
                    for (int e2 = 0; e2 < 8; ++e2) {
                        const size_t o = ((size_t)ks * 2 * 64 + l) * 8 + e2;
                        const size_t i = (size_t)(l % 32) * pad + 16 * ks + 8 * (l / 32) + e2;
                        dst[o] = ph[i];
                        dst[o + 512] = plo[i];
                    }
        };
        auto by_column = [&](uint16_t *dst, int pad, int tile_stride, int step_stride) {
            for (int g2 = 0; g2 < pad / 32; ++g2)
                for (int q = 0; q < 2; ++q)
                    for (int l = 0; l < 64; ++l)
                        for (int e2 = 0; e2 < 8; ++e2) {
                            const size_t o = ((size_t)(g2 * tile_stride + q * step_stride) * 2 * 64 + l) * 8 + e2;
                            const size_t i = (size_t)(16 * q + tp16(e2, l / 32)) * pad + 32 * g2 + l % 32;
                            dst[o] = ph[i];
                            dst[o + 512] = plo[i];
                        }
        };
        const int CP = 32 * sp.nct;
        skf.assign(2 * KE * n_ktab, 0);
        ska.assign(2 * KE * n_ktab, 0);
        sff.assign((size_t)2 * TP * CP, 0);
        sfa.assign((size_t)2 * TP * CP, 0);
        for (int c = 0; c < NC; ++c) {
            for (int tb = 0; tb < n_ktab; ++tb) {
                const size_t o = 2 * KE * tb + (size_t)c * 64 * NUP;
                pairs(&K[KE * tb + (size_t)32 * c * NUP], NUP, NUP, NUP, [&](int) { return ksc; });
                by_time(&skf[o], NUP);
                by_column(&ska[o], NUP, 1, NUP / 32);
            }
            pairs(&F[(size_t)32 * c * NBP2], NBP2, 2 * NB, CP, [&](int p) { return fsc[p / 2]; });
            by_column(&sff[(size_t)c * 64 * CP], CP, 2, 1);
            by_time(&sfa[(size_t)c * 64 * CP], CP);
        }
    }

    // precomposed line matrices Gt[p][c] = sum_n K[n][p] F[n][c] (the whole
    // A_DC of one line, c_A aside), one per PSF table, float64 accumulation
    std::vector<float> gt;
    pl->gt_elems = (size_t)NUP * 2 * NB;
    if (precomp) {
        const int NB2 = 2 * NB;
        gt.resize(pl->gt_elems * n_ktab);
        std::vector<double> acc(pl->gt_elems);
        for (int tb = 0; tb < n_ktab; ++tb) {
            std::fill(acc.begin(), acc.end(), 0.0);
            const double *Kc = &K[KE * tb];
            for (int n = 0; n < T; ++n) {
                const double *fr = &F[(size_t)n * NBP2];
                for (int p = 0; p < NU; ++p) {
                    const double k = Kc[(size_t)n * NUP + p];
                    double *row = &acc[(size_t)p * NB2];
                    for (int c = 0; c < NB2; ++c) row[c] += k * fr[c];
                }
            }
            for (size_t i = 0; i < acc.size(); ++i) gt[pl->gt_elems * tb + i] = (float)acc[i];
        }
    }

    // ---- table layout in one device allocation -----------------------------
    size_t off = 0;
    char *nullbase = nullptr;
    size_t o_cs, o_ax, o_ay, o_ay1, o_order, o_kf, o_ff, o_fa, o_ka, o_kf16 = 0, o_ff16 = 0, o_fa16 = 0, o_ka16 = 0, o_cols = 0, o_bands = 0;
    auto place = [&](size_t bytes) { off = align256(off); size_t o = off; off += bytes; return o; };
    o_cs = place(sizeof(float2) * M);
    o_ax = place(sizeof(float) * M * NU);
    o_ay = place(sizeof(float) * M * NU);
    o_ay1 = place(sizeof(float) * M * NU);
    o_order = place(sizeof(int) * M);
    o_kf = place(dense ? sizeof(float) * KE * n_ktab : 0);
    o_ff = place(dense ? sizeof(float) * (size_t)TP * NBP2 : 0);
    o_fa = place(dense ? sizeof(float) * (size_t)TP * NBP2 : 0);
    o_ka = place(dense ? sizeof(float) * KE * n_ktab : 0);
    const size_t KEF = KE * pl->n_passes * pl->n_line_groups;   // fused tables, all groups
    const size_t o_kff = pl->fused && dense ? place(sizeof(float) * KEF) : 0;
    const size_t o_kaf = pl->fused && dense ? place(sizeof(float) * KEF) : 0;
    const size_t o_gt = precomp ? place(sizeof(float) * gt.size()) : 0;
    const size_t o_gta = precomp ? place(sizeof(float) * gt.size()) : 0;
    const bool fac = pl->fac.on;
    const size_t o_fkf = fac ? place(sizeof(_Float16) * fkf.size()) : 0;
    const size_t o_fka = fac ? place(sizeof(_Float16) * fka.size()) : 0;
    const size_t o_fef = fac ? place(sizeof(_Float16) * fef.size()) : 0;
    const size_t o_fea = fac ? place(sizeof(_Float16) * fea.size()) : 0;
    const size_t o_fwf = fac ? place(sizeof(_Float16) * fwf.size()) : 0;
    const size_t o_fwa = fac ? place(sizeof(_Float16) * fwa.size()) : 0;
    const size_t o_funit0 = fac ? place(sizeof(int) * funit0.size()) : 0;
    const size_t o_fqbin = fac ? place(sizeof(int) * fqbin.size()) : 0;
    const size_t o_fbcol = fac ? place(sizeof(int) * fbcol.size()) : 0;
    const size_t o_fwexp = fac ? place(sizeof(int) * fwexp.size()) : 0;
    const size_t o_skf = split ? place(sizeof(_Float16) * skf.size()) : 0;
    const size_t o_ska = split ? place(sizeof(_Float16) * ska.size()) : 0;
    const size_t o_sff = split ? place(sizeof(_Float16) * sff.size()) : 0;
    const size_t o_sfa = split ? place(sizeof(_Float16) * sfa.size()) : 0;
    const size_t o_sfexp = split ? place(sizeof(int) * sfexp.size()) : 0;
    const size_t o_saexp = split ? place(sizeof(int) * saexp.size()) : 0;
    if (mixed) {
        o_kf16 = place(sizeof(__half) * KE * n_ktab);
        o_ff16 = place(sizeof(__half) * (size_t)TP * NBP2);
        o_fa16 = place(sizeof(__half) * (size_t)TP * NBP2);
        o_ka16 = place(sizeof(__half) * KE * n_ktab);
        o_cols = place(sizeof(float) * NBP2);
        o_bands = place(sizeof(float) * NBP2);
    }
    (void)nullbase;
    pl->table_bytes = align256(off);

    // Swizzled fp32 tables: every MFMA operand a lane needs for 4 consecutive
    // steps is one 16-byte load, and a wave's 64 loads are contiguous.
    //  kf: fwd GEMM1 A operand  K[t = 32c + l%32][p = 2st + l/32]    [c][st/4][l][st%4]
    //  ff: fwd GEMM2 B operand  F[t = 32c + tperm(s, l/32)][32ct + l%32]  [c][ct][s/4][l][s%4]
    //  fa: adj GEMM1 A operand  F[t = 32c + l%32][col = 2st + l/32]  [c][st/4][l][st%4]
    //  ka: adj GEMM2 B operand  K[t = 32c + tperm(s, l/32)][32pt + l%32]  [c][pt][s/4][l][s%4]
    // tperm(s, h) = 8(s/4) + 4h + s%4 is the time index that the 32x32 MFMA
    // result layout leaves in register s of lane half h.
    std::vector<float> kf(dense ? KE * n_ktab : 0), ff(dense ? (size_t)TP * NBP2 : 0), fa(ff.size()), ka(kf.size());
    auto tperm = [](int s, int h) { return 8 * (s / 4) + 4 * h + (s % 4); };
    for (int cl = 0; dense && cl < n_ktab; ++cl)
        for (int c = 0; c < NC; ++c) {
            const double *Kc = &K[KE * cl];
            float *kfc = &kf[KE * cl], *kac = &ka[KE * cl];
            for (int st = 0; st < NUP / 2; ++st)
                for (int l = 0; l < 64; ++l)
                    kfc[(((size_t)c * (NUP / 8) + st / 4) * 64 + l) * 4 + st % 4] =
                        (float)Kc[(size_t)(32 * c + l % 32) * NUP + 2 * st + l / 32];
            for (int pt = 0; pt < NUP / 32; ++pt)
                for (int s = 0; s < 16; ++s)
                    for (int l = 0; l < 64; ++l)
                        kac[((((size_t)c * (NUP / 32) + pt) * 4 + s / 4) * 64 + l) * 4 + s % 4] =
                            (float)Kc[(size_t)(32 * c + tperm(s, l / 32)) * NUP + 32 * pt + l % 32];
        }
    for (int c = 0; dense && c < NC; ++c) {
        for (int ct = 0; ct < NCT; ++ct)
            for (int s = 0; s < 16; ++s)
                for (int l = 0; l < 64; ++l)
                    ff[((((size_t)c * NCT + ct) * 4 + s / 4) * 64 + l) * 4 + s % 4] =
                        (float)F[(size_t)(32 * c + tperm(s, l / 32)) * NBP2 + 32 * ct + l % 32];
        for (int st = 0; st < NBP2 / 2; ++st)
            for (int l = 0; l < 64; ++l)
                fa[(((size_t)c * (NBP2 / 8) + st / 4) * 64 + l) * 4 + st % 4] =
                    (float)F[(size_t)(32 * c + l % 32) * NBP2 + 2 * st + l / 32];
    }

    // Mixed (fp16) tables with power-of-two scales.
    std::vector<_Float16> kf16, ff16, fa16, ka16;
    std::vector<float> col_scale, band_scale;
    if (mixed) {
        double kmax = 0, fmax = 0;
        for (double v : K) kmax = std::max(kmax, std::fabs(v));
        for (double v : F) fmax = std::max(fmax, std::fabs(v));
        int ek, ef;
        std::frexp(kmax > 0 ? kmax : 1.0, &ek);
        std::frexp(fmax > 0 ? fmax : 1.0, &ef);
        double ks = std::ldexp(1.0, -ek), fs = std::ldexp(1.0, -ef);  // scaled max in [0.5, 1)
        // Per-band adjoint scale: a band's share of the operator, measured as
        // its response to a unit source at each of a few detector positions.
        std::vector<double> bnorm(NB / (2 * pl->half_band + 1), 0.0);
        int nbands = (int)bnorm.size(), bw = 2 * pl->half_band + 1;
        for (int probe = 0; probe < 3 * n_ktab; ++probe) {
            const int p = (probe % 3 + 1) * NU / 4;
            const double *Kc = &K[KE * (probe / 3)];
            for (int j = 0; j < NB; ++j) {
                double re = 0, im = 0;
                for (int n = 0; n < T; ++n) {
                    double kv = Kc[(size_t)n * NUP + p];
                    re += kv * F[(size_t)n * NBP2 + 2 * j];
                    im += kv * F[(size_t)n * NBP2 + 2 * j + 1];
                }
                bnorm[j / bw] = std::max(bnorm[j / bw], std::sqrt(re * re + im * im));
            }
        }
        double bmax = *std::max_element(bnorm.begin(), bnorm.end());
        col_scale.assign(NBP2, (float)(1.0 / (ks * fs)));
        pl->adj_scale16 = (float)(1.0 / (ks * fs));
        band_scale.assign(NBP2, 1.0f);
        std::vector<double> fcol(NBP2, fs);
        for (int b = 0; b < nbands; ++b) {
            double rel = bnorm[b] > 0 && bmax > 0 ? bnorm[b] / bmax : 1.0;
            int e;
            std::frexp(rel, &e);                       // rel in [2^(e-1), 2^e)
            double bs = std::ldexp(1.0, std::min(-(e - 1), 14));  // lifts the band to [1, 2) x max
            for (int d = 0; d < bw; ++d)
                for (int h = 0; h < 2; ++h) {
                    int col = 2 * (b * bw + d) + h;
                    band_scale[col] = (float)bs;
                    fcol[col] = fs / bs;
                }
        }
        // fp16 layouts (8 halves per lane per MFMA step, 32x32x16):
        //  kf16: fwd GEMM1 A: K[t = 32c + l%32][p = 16st + 8(l/32) + e]          [c][st][l][e]
        //  ff16: fwd GEMM2 B: F[t = 32c + 16h + tperm16(e, l/32)][32ct + l%32]   [c][ct][h][l][e]
        //  fa16: adj GEMM1 A: F[t = 32c + l%32][col = 16st + 8(l/32) + e]        [c][st][l][e]
        //  ka16: adj GEMM2 B: K[t = 32c + 16h + tperm16(e, l/32)][32pt + l%32]   [c][pt][h][l][e]
        // tperm16(e, h) = 8(e/4) + 4h + e%4.
        auto tp16 = [](int e, int h) { return 8 * (e / 4) + 4 * h + (e % 4); };
        kf16.resize(KE * n_ktab);
        ff16.resize((size_t)TP * NBP2);
        fa16.resize((size_t)TP * NBP2);
        ka16.resize(KE * n_ktab);
        for (int cl = 0; cl < n_ktab; ++cl)
            for (int c = 0; c < NC; ++c) {
                const double *Kc = &K[KE * cl];
                _Float16 *kfc = &kf16[KE * cl], *kac = &ka16[KE * cl];
                for (int st = 0; st < NUP / 16; ++st)
                    for (int l = 0; l < 64; ++l)
                        for (int e2 = 0; e2 < 8; ++e2)
                            kfc[(((size_t)c * (NUP / 16) + st) * 64 + l) * 8 + e2] =
                                to_f16(Kc[(size_t)(32 * c + l % 32) * NUP + 16 * st + 8 * (l / 32) + e2] * ks);
                for (int pt = 0; pt < NUP / 32; ++pt)
                    for (int h = 0; h < 2; ++h)
                        for (int l = 0; l < 64; ++l)
                            for (int e2 = 0; e2 < 8; ++e2)
                                kac[((((size_t)c * (NUP / 32) + pt) * 2 + h) * 64 + l) * 8 + e2] = to_f16(
                                    Kc[(size_t)(32 * c + 16 * h + tp16(e2, l / 32)) * NUP + 32 * pt + l % 32] * ks);
            }
        for (int c = 0; c < NC; ++c) {
            for (int ct = 0; ct < NCT; ++ct)
                for (int h = 0; h < 2; ++h)
                    for (int l = 0; l < 64; ++l)
                        for (int e2 = 0; e2 < 8; ++e2)
                            ff16[((((size_t)c * NCT + ct) * 2 + h) * 64 + l) * 8 + e2] = to_f16(
                                F[(size_t)(32 * c + 16 * h + tp16(e2, l / 32)) * NBP2 + 32 * ct + l % 32] * fs);
            for (int st = 0; st < NBP2 / 16; ++st)
                for (int l = 0; l < 64; ++l)
                    for (int e2 = 0; e2 < 8; ++e2) {
                        int col = 16 * st + 8 * (l / 32) + e2;
                        fa16[(((size_t)c * (NBP2 / 16) + st) * 64 + l) * 8 + e2] =
                            to_f16(F[(size_t)(32 * c + l % 32) * NBP2 + col] * fcol[col]);
                    }
        }
        // undo factors applied to the adjoint: result = acc / (fs * ks * row_scale)
        (void)ef;
    }

    // ---- upload ------------------------------------------------------------
    e = hipMalloc(&pl->tables, pl->table_bytes);
    if (e != hipSuccess) { delete pl; return MPI3D_ENOMEM; }
    char *tb = (char *)pl->tables;
    pl->cs = (float2 *)(tb + o_cs);
    pl->ax = (float *)(tb + o_ax);
    pl->ay = (float *)(tb + o_ay);
    pl->ay1 = (float *)(tb + o_ay1);
    pl->order = (int *)(tb + o_order);
    if (dense) {
        pl->kf = (float *)(tb + o_kf);
        pl->ff = (float *)(tb + o_ff);
        pl->fa = (float *)(tb + o_fa);
        pl->ka = (float *)(tb + o_ka);
    }
    bool ok = hipMemcpy(pl->cs, cs.data(), sizeof(float2) * M, hipMemcpyHostToDevice) == hipSuccess;
    ok = ok && hipMemcpy(pl->ax, ax.data(), sizeof(float) * ax.size(), hipMemcpyHostToDevice) == hipSuccess;
    ok = ok && hipMemcpy(pl->ay, ay.data(), sizeof(float) * ay.size(), hipMemcpyHostToDevice) == hipSuccess;
    ok = ok && hipMemcpy(pl->ay1, ay1.data(), sizeof(float) * ay1.size(), hipMemcpyHostToDevice) == hipSuccess;
    ok = ok && hipMemcpy(pl->order, order.data(), sizeof(int) * M, hipMemcpyHostToDevice) == hipSuccess;
    ok = ok && (!dense || hipMemcpy(pl->kf, kf.data(), sizeof(float) * kf.size(), hipMemcpyHostToDevice) == hipSuccess);
    ok = ok && (!dense || hipMemcpy(pl->ff, ff.data(), sizeof(float) * ff.size(), hipMemcpyHostToDevice) == hipSuccess);
    ok = ok && (!dense || hipMemcpy(pl->fa, fa.data(), sizeof(float) * fa.size(), hipMemcpyHostToDevice) == hipSuccess);
    ok = ok && (!dense || hipMemcpy(pl->ka, ka.data(), sizeof(float) * ka.size(), hipMemcpyHostToDevice) == hipSuccess);
    if (pl->fused && dense) {
        // group g's tables table_g .. table_g + R side by side per time chunk:
        // a chunk of kf / ka holds NUP x 32 floats for detector samples (kf:
        // 8 per float4 step, ka: 32 per column tile) in the order the kernels
        // walk them, so concatenating the chunks of consecutive offsets is the
        // layout of one table of NUP (R + 1) samples
        std::vector<float> kff(KEF), kaf(KEF);
        const size_t CB = (size_t)NUP * 32;   // floats per chunk of one table
        const int NP = pl->n_passes;
        for (int gi = 0; gi < pl->n_line_groups; ++gi)
            for (int c = 0; c < NC; ++c)
                for (int e2 = 0; e2 < NP; ++e2) {
                    const size_t src = (size_t)(pl->groups[gi].table + e2) * KE + c * CB;
                    const size_t dst = ((size_t)gi * NP * NC + (size_t)c * NP + e2) * CB;
                    std::copy(&kf[src], &kf[src] + CB, &kff[dst]);
                    std::copy(&ka[src], &ka[src] + CB, &kaf[dst]);
                }
        pl->kff = (float *)(tb + o_kff);
        pl->kaf = (float *)(tb + o_kaf);
        ok = ok && hipMemcpy(pl->kff, kff.data(), sizeof(float) * KEF, hipMemcpyHostToDevice) == hipSuccess;
        ok = ok && hipMemcpy(pl->kaf, kaf.data(), sizeof(float) * KEF, hipMemcpyHostToDevice) == hipSuccess;
    }
    auto up = [&](auto *&dst, size_t o, const auto &v) {
        dst = reinterpret_cast<std::remove_reference_t<decltype(dst)>>(tb + o);
        ok = ok && hipMemcpy(dst, v.data(), sizeof(v[0]) * v.size(), hipMemcpyHostToDevice) == hipSuccess;
    };
    if (split) {
        up(pl->split.kf, o_skf, skf);
        up(pl->split.ka, o_ska, ska);
        up(pl->split.ff, o_sff, sff);
        up(pl->split.fa, o_sfa, sfa);
        up(pl->split.fexp, o_sfexp, sfexp);
        up(pl->split.aexp, o_saexp, saexp);
        if (std::all_of(saexp.begin(), saexp.end(), [](int e) { return e == 0; })) pl->split.aexp = nullptr;
    }
    if (fac) {
        mpi3d_plan::Fac &f = pl->fac;
        up(f.kf, o_fkf, fkf);
        up(f.ka, o_fka, fka);
        up(f.ef, o_fef, fef);
        up(f.ea, o_fea, fea);
        up(f.wf, o_fwf, fwf);
        up(f.wa, o_fwa, fwa);
        up(f.unit0, o_funit0, funit0);
        up(f.qbin, o_fqbin, fqbin);
        up(f.bcol, o_fbcol, fbcol);
        up(f.wexp, o_fwexp, fwexp);
    }
    if (precomp) {
        pl->gt = (float *)(tb + o_gt);
        pl->gta = (float *)(tb + o_gta);
        // G = (G^T)^T per table, [2nb][n_up]: the adjoint GEMM's operand rows
        std::vector<float> gta(gt.size());
        const size_t NB2 = 2 * (size_t)NB;
        for (int tb2 = 0; tb2 < n_ktab; ++tb2)
            for (size_t p = 0; p < (size_t)NUP; ++p)
                for (size_t c = 0; c < NB2; ++c)
                    gta[pl->gt_elems * tb2 + c * NUP + p] = gt[pl->gt_elems * tb2 + p * NB2 + c];
        ok = ok && hipMemcpy(pl->gt, gt.data(), sizeof(float) * gt.size(), hipMemcpyHostToDevice) == hipSuccess;
        ok = ok && hipMemcpy(pl->gta, gta.data(), sizeof(float) * gta.size(), hipMemcpyHostToDevice) == hipSuccess;
    }
    if (mixed) {
        pl->kf16 = (__half *)(tb + o_kf16);
        pl->ff16 = (__half *)(tb + o_ff16);
        pl->fa16 = (__half *)(tb + o_fa16);
        pl->ka16 = (__half *)(tb + o_ka16);
        pl->col_scale = (float *)(tb + o_cols);
        pl->band_scale = (float *)(tb + o_bands);
        ok = ok && hipMemcpy(pl->kf16, kf16.data(), sizeof(_Float16) * kf16.size(), hipMemcpyHostToDevice) == hipSuccess;
        ok = ok && hipMemcpy(pl->ff16, ff16.data(), sizeof(_Float16) * ff16.size(), hipMemcpyHostToDevice) == hipSuccess;
        ok = ok && hipMemcpy(pl->fa16, fa16.data(), sizeof(_Float16) * fa16.size(), hipMemcpyHostToDevice) == hipSuccess;
        ok = ok && hipMemcpy(pl->ka16, ka16.data(), sizeof(_Float16) * ka16.size(), hipMemcpyHostToDevice) == hipSuccess;
        ok = ok && hipMemcpy(pl->col_scale, col_scale.data(), sizeof(float) * NBP2, hipMemcpyHostToDevice) == hipSuccess;
        ok = ok && hipMemcpy(pl->band_scale, band_scale.data(), sizeof(float) * NBP2, hipMemcpyHostToDevice) == hipSuccess;
    }
    if (!ok) {
        (void)hipFree(pl->tables);
        delete pl;
        return MPI3D_EDEVICE;
    }

    // ---- workspace layouts -------------------------------------------------
    op_layout(pl, pl->fac.on, pl->split.on);
    {
        size_t o = 0;
        auto put = [&](size_t bytes) { o = align256(o); size_t r = o; o += bytes; return r; };
        long ndata = 2 * pl->L * pl->nb;
        pl->sw_op = put(pl->op_ws_bytes);
        pl->sw_r = put(sizeof(float) * ndata);
        pl->sw_q = put(sizeof(float) * ndata);
        pl->sw_s = put(sizeof(float) * pl->nvox);
        pl->sw_p = put(sizeof(float) * pl->nvox);
        pl->sw_scal = put(sizeof(double) * 64);
        pl->sw_parts = put(sizeof(double) * 3 * pl->max_parts);
        pl->sw_d = put(mixed ? sizeof(float) * pl->nvox : 0);   // refinement correction
        pl->sw_g = put(mixed ? sizeof(float) * pl->nvox : 0);   // FP32 gradient at the sweep start
        pl->sw_v = put(sizeof(float) * pl->nvox);                 // momentum solver: fourth volume
        pl->solve_ws_bytes = align256(o);
    }
    {
        // FNV-1a over the parameters that determine the line tables
        uint64_t h = 1469598103934665603ull;
        auto mix = [&](const void *p, size_t n) {
            const unsigned char *c = (const unsigned char *)p;
            for (size_t i = 0; i < n; ++i) { h ^= c[i]; h *= 1099511628211ull; }
        };
        int ints[] = {pl->nu, pl->nup, pl->nt, pl->harm_lo, pl->harm_hi, pl->half_band, pl->nbp2,
                      pl->sc[0].pairs, pl->sc[0].ngroups, pl->sc[0].gct, pl->sc[1].pairs, pl->sc[1].ngroups,
                      pl->sc[1].gct, precisions, n_classes, psf_rows, drive_axes, drive_axes == 2 ? pl->nz : 0,
                      pl->fused ? pl->nupf : 0, pl->fused ? pl->scf.gct : 0, pl->fac.on ? pl->fac.C : 0, pl->split.on};
        double dbl[] = {pl->P, pl->a, pl->w, pl->raster_sweep, drive_axes == 2 ? pl->a_z : 0.0};
        mix(ints, sizeof(ints));
        mix(dbl, sizeof(dbl));
        if (g->rx_filter) mix(g->rx_filter, sizeof(float) * 2 * pl->nb);
        pl->line_key = h;
    }
    // the no-allocation entry point's scratch address on this device (a
    // failure here is reported by that entry point itself)
    (void)scratch_setup(device);
    pl->norm_iters = 0;
    if (g->op_scale == 0.0) {
        // c_A = 1 / ||A||_2, estimated on the device
        double nrm = 0.0;
        int its = 0;
        const int rc = estimate_op_norm(pl, 1e-7, 1000, &nrm, &its);
        if (rc != MPI3D_OK) {
                (void)hipFree(pl->tables);
            delete pl;
            return rc;
        }
        pl->op_scale = 1.0 / nrm;
        pl->norm_iters = its;
    }
    *out = pl;
    return MPI3D_OK;
}

extern "C" void mpi3d_plan_destroy(mpi3d_plan *pl)
{
    if (!pl) return;
    int prev = 0;
    (void)hipGetDevice(&prev);
    (void)hipSetDevice(pl->device);
    (void)hipFree(pl->tables);
    (void)hipSetDevice(prev);
    delete pl;
}

extern "C" int mpi3d_plan_query(const mpi3d_plan *pl, mpi3d_plan_info *info)
{
    if (!pl || !info) return MPI3D_EINVAL;
    info->n_vox = pl->nvox;
    info->n_lines = pl->L;
    info->n_bins = pl->nb;
    info->n_data_floats = 2 * pl->L * pl->nb;
    info->n_proj_floats = pl->Lx * pl->nu;
    info->op_ws_bytes = (int64_t)pl->op_ws_bytes;
    info->solve_ws_bytes = (int64_t)pl->solve_ws_bytes;
    info->table_bytes = (int64_t)pl->table_bytes;
    info->history_doubles = 4;
    info->n_r = pl->nr;
    info->norm_iters = pl->norm_iters;
    info->op_scale = pl->op_scale;
    info->dft_cycles = pl->fac.on ? pl->fac.C : 0;
    info->dft_residues = pl->fac.on ? pl->fac.res : 0;
    return MPI3D_OK;
}
