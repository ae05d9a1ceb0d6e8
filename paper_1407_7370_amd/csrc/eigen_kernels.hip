// gfx950 kernels of the eigenvalue mode with full reorthogonalisation
// (Sec. 2: the Lanczos vectors are kept and every new vector is
// orthogonalised against all of them, twice where needed) and of the Ritz vectors
// (Sec. 2 eq. eigenvec_approx).
//
// Iteration i: z = H q_i - alpha_i q_i - beta_{i-1} q_{i-1} (k_eig_apply,
// k_local), then classical Gram-Schmidt, h = Q^H z, z -= Q h.  The projections of
// a pass all use the same z, so one pass is a tall-skinny product that streams
// the stored basis once; the modified form would stream it once per vector.
//
// A second pass follows where the first one removed anything to speak of:
// ||h|| > kAgain ||z|| (the test of Daniel, Gragg, Kaufman and Stewart 1976).  What a
// pass leaves along Q is (I - Q^H Q) h and its rounding, so with Q orthonormal to
// d it is at most d ||h|| + O(eps ||z||): after the local terms h is the rounding of
// H q_i (||h|| ~ eps ||H||) and one pass leaves O(eps), except near a breakdown,
// where ||z|| itself is that small.  Without the local terms first (h_i = alpha_i,
// far larger than ||z||) every iteration needed both passes.
//
// Bound by HBM bandwidth: the projection reads the i stored vectors and z, the
// update reads them again and rewrites z.  The projection walks the basis upwards
// and the update downwards, so that each finds what the other read last in the
// last-level cache (3 % at 1024^2, 5 % at 256^2).  256^2, 512 vectors (1 GB): k_proj
// 4.5 -> 5.7 TB/s, k_sub_q 5.8, a pass of 512 iterations with two Ritz vectors
// 236 ms with two pairs of kernels an iteration, 115 ms now.
// Reductions are per-workgroup partials folded in a fixed order, so results are
// bitwise reproducible.
//
// Vectors use the state layout (complex128, both spinor planes), vector j
// (0-based) of the basis at q + j * vstride bytes.
#include <hip/hip_runtime.h>

#include <algorithm>

#include "device_reduce.h"
#include "dl_internal.h"
#include "sweeps.h"

namespace dl {
namespace {

constexpr int kDotVecs = 16;  // basis vectors per workgroup of a projection
// workgroups of a projection (at most kProjTiles per vector chunk): one resident
// round of six per compute unit.  TB/s of 256^2 / 1024^2 (vector counts to 512 /
// 256): 1024 5.38 / 5.79, 1536 5.73 / 5.98, 2048 5.06 / 5.26, 8192 5.49 / 5.80
constexpr int kProjWorkgroups = 1536;
constexpr int kProjSecond = 512;  // of the second pass, most of whose launches return at once
// largest ||h|| / ||z|| of a pass that needs no second one
constexpr double kAgain = 1.0 / 128.0;
constexpr int kSubChunk = 256;  // coefficients staged in LDS per chunk of the update
static_assert(kSubChunk % kDotVecs == 0, "the update pads a chunk to whole groups of kDotVecs");
constexpr int kRitzChunk = 64;  // basis rows of t staged in LDS per chunk

__device__ __forceinline__ const double2 *qvec(const char *q, size_t vstride, int j)
{
    return reinterpret_cast<const double2 *>(q + (size_t)j * vstride);
}

// Sums of 2 N values over the wave's lanes: each step halves the values a lane
// holds and the lanes that share them (for 32 values 32 exchanges; a butterfly
// per value takes 192).  With 32 values lane l ends with the sum of value l >> 1.
template <int N, int S>
__device__ __forceinline__ double wave_sum_spread(double (&v)[2 * N])
{
    const bool up = ((int)threadIdx.x & S) != 0;
    double r[N];
#pragma unroll
    for (int k = 0; k < N; ++k) {
        const double keep = up ? v[k + N] : v[k], send = up ? v[k] : v[k + N];
        r[k] = keep + __shfl_xor(send, S, 64);
    }
    if constexpr (N > 1)
        return wave_sum_spread<N / 2, S / 2>(r);
    else
        return r[0] + __shfl_xor(r[0], S / 2, 64);
}

// w = H q (one site per thread and step), and this workgroup's partial of
// alpha = Re <q, w>.
__global__ __launch_bounds__(kBlock) void k_eig_apply(Op op, const double2 *__restrict__ q, double2 *__restrict__ w,
                                                      double *__restrict__ partials)
{
    const size_t sites = (size_t)op.nx * op.ny;
    double acc[1] = {0.0};
    for (size_t e = (size_t)blockIdx.x * kBlock + threadIdx.x; e < sites; e += (size_t)gridDim.x * kBlock) {
        const int j = (int)(e / (unsigned)op.nx), i = (int)(e - (size_t)j * op.nx);
        auto site = [&](int x, int y, bool in, bool periodic) {
            if (!in && !periodic) return sp_zero();
            const size_t g = (size_t)y * op.nx + x;
            const double2 a = q[g], b = q[sites + g];
            return Sp{a.x, a.y, b.x, b.y};
        };
        const Sp c = site(i, j, true, true);
        const Sp l = site(i > 0 ? i - 1 : op.nx - 1, j, i > 0, op.bcx), r = site(i + 1 < op.nx ? i + 1 : 0, j, i + 1 < op.nx, op.bcx);
        const Sp d = site(i, j > 0 ? j - 1 : op.ny - 1, j > 0, op.bcy), u = site(i, j + 1 < op.ny ? j + 1 : 0, j + 1 < op.ny, op.bcy);
        LaneGeo lg{};
        lg.colw = i;
        lg.inx = true;
        lg.x = op.xmin + i * op.hx;
        const double y = op.ymin + j * op.hy;
        const Sp o = hop(op, c, l, r, d, u, site_pot_row(op, lg, j, y), op.bq * y, -op.bqy * lg.x);
        w[e] = make_double2(o.r0, o.i0);
        w[sites + e] = make_double2(o.r1, o.i1);
        acc[0] += sp_redot(c, o);
    }
    store_partial(acc, partials, (int)blockIdx.x);
}

// alpha_i from the partials, and w -= alpha_i q_i + beta_{i-1} q_{i-1}.
__global__ __launch_bounds__(kBlock) void k_local(const double2 *__restrict__ q, const double2 *__restrict__ qm,
                                                  double2 *__restrict__ w, size_t nelem, int i, double *alpha,
                                                  const double *beta, const Scalars *sc,
                                                  const double *partials, int npart)
{
    __shared__ double red[kWaves][1];
    double tot[1];
    fold_partials(partials, npart, red, tot);
    const double al = tot[0], be = i > 1 ? beta[i - 1] : 0.0;
    if (blockIdx.x == 0 && threadIdx.x == 0 && sc->kstop >= i) alpha[i] = al;
    for (size_t e = (size_t)blockIdx.x * kBlock + threadIdx.x; e < nelem; e += (size_t)gridDim.x * kBlock) {
        const double2 a = q[e];
        double2 v = w[e];
        v.x -= al * a.x;
        v.y -= al * a.y;
        if (i > 1) {
            const double2 b = qm[e];
            v.x -= be * b.x;
            v.y -= be * b.y;
        }
        w[e] = v;
    }
}

// Partial projections.  Workgroup (t, c) accumulates conj(q_j) . z over the
// elements t*256 + tid + r * ntiles*256 for the 16 vectors j = 16c .. 16c+15
// (< nvec) and writes them to pproj[(j * ntiles + t) * 2 + {re, im}].
__global__ __launch_bounds__(kBlock) void k_proj(const char *__restrict__ q, size_t vstride, int nvec,
                                                 const double2 *__restrict__ z, size_t nelem,
                                                 double *__restrict__ pproj, int ntiles, const Scalars *sc,
                                                 int second)
{
    static_assert(kDotVecs == 16, "a wave sums 32 values");
    if (second && !sc->again) return;
    __shared__ double red[kWaves][2 * kDotVecs];
    const int t = blockIdx.x, j0 = blockIdx.y * kDotVecs;
    const int nj = min(kDotVecs, nvec - j0);
    double h[2 * kDotVecs];  // re, im per vector
#pragma unroll
    for (int jj = 0; jj < 2 * kDotVecs; ++jj) h[jj] = 0.0;
    for (size_t e = (size_t)t * kBlock + threadIdx.x; e < nelem; e += (size_t)ntiles * kBlock) {
        const double2 zv = z[e];
        // every load unconditional (a short last chunk re-reads its last
        // vector into accumulators that are never written out), so the 16
        // loads of a site are in flight together
#pragma unroll
        for (int jj = 0; jj < kDotVecs; ++jj) {
            const double2 qv = qvec(q, vstride, j0 + min(jj, nj - 1))[e];
            h[2 * jj] += qv.x * zv.x + qv.y * zv.y;
            h[2 * jj + 1] += qv.x * zv.y - qv.y * zv.x;
        }
    }
    const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
    const double sum = wave_sum_spread<16, 32>(h);
    if ((lane & 1) == 0) red[w][lane >> 1] = sum;
    __syncthreads();
    if (threadIdx.x < 2 * nj) {
        double a = red[0][threadIdx.x];
        for (int i = 1; i < kWaves; ++i) a += red[i][threadIdx.x];
        const int jj = threadIdx.x >> 1, part = threadIdx.x & 1;
        pproj[((size_t)(j0 + jj) * ntiles + t) * 2 + part] = a;
    }
}

// h_j = sum of the ntiles partials of vector j (workgroup j; fixed order).
__global__ __launch_bounds__(kBlock) void k_proj_fold(const double *__restrict__ pproj, int ntiles, double *h,
                                                      const Scalars *sc, int second)
{
    if (second && !sc->again) return;
    __shared__ double red[kWaves][2];
    const int j = blockIdx.x;
    double s[2] = {0.0, 0.0};
    for (int t = threadIdx.x; t < ntiles; t += kBlock) {
        s[0] += pproj[((size_t)j * ntiles + t) * 2];
        s[1] += pproj[((size_t)j * ntiles + t) * 2 + 1];
    }
    wave_sum(s);
    const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
    if (lane == 0) {
        red[w][0] = s[0];
        red[w][1] = s[1];
    }
    __syncthreads();
    if (threadIdx.x < 2) {
        double a = red[0][threadIdx.x];
        for (int i = 1; i < kWaves; ++i) a += red[i][threadIdx.x];
        h[2 * j + threadIdx.x] = a;
    }
}

// Scalar update of iteration i from ||z||^2 (alpha_i is there): beta_i = ||z||, the
// running scale max(|alpha_j|, beta_{j-1}) and the breakdown test beta_i <= 1e-13
// scale, which stops the recurrence with k_eff = i (the Krylov space is
// invariant).
__device__ __forceinline__ void norm_update(double zz, int i, const double *alpha, double *beta, Scalars *sc)
{
    if (sc->kstop < i) return;
    const double al = alpha[i];
    const double b = sqrt(zz);
    if (!isfinite(b) || !isfinite(al)) {
        sc->status = 3;
        sc->kstop = -1;
        return;
    }
    beta[i] = b;
    double scale = fmax(sc->scale, fabs(al));
    if (i > 1) scale = fmax(scale, beta[i - 1]);
    sc->scale = scale;
    sc->keff = i;
    if (b <= 1e-13 * scale) sc->kstop = i;
}

// z -= sum_j h_j q_j and ||z||^2; the last workgroup adds Re h_i (what rounding left
// along q_i) to alpha_i, decides whether a second pass follows, and else updates the
// scalars of iteration i = nvec.  The loop over element tiles has a workgroup-uniform
// trip count (the LDS staging of h needs every thread at the barriers).
__global__ __launch_bounds__(kBlock) void k_sub_q(const char *__restrict__ q, size_t vstride, int nvec,
                                                  const double *__restrict__ h, double2 *__restrict__ z,
                                                  size_t nelem, double *alpha, double *beta, Scalars *sc,
                                                  double *partials, int second)
{
    if (second && !sc->again) return;
    __shared__ double hs[2 * kSubChunk];
    double zz[1] = {0.0};
    const size_t step = (size_t)gridDim.x * kBlock;
    for (size_t base = (size_t)blockIdx.x * kBlock; base < nelem; base += step) {
        const size_t e = base + threadIdx.x;
        const bool live = e < nelem;
        double ar = 0.0, ai = 0.0;
        for (int j0 = (nvec - 1) / kSubChunk * kSubChunk; j0 >= 0; j0 -= kSubChunk) {
            const int nj = min(kSubChunk, nvec - j0);
            // coefficients padded with zeros to whole groups of kDotVecs, so
            // each group issues all its loads before the first use
            const int njp = (nj + kDotVecs - 1) / kDotVecs * kDotVecs;
            __syncthreads();
            for (int i = threadIdx.x; i < 2 * njp; i += kBlock) hs[i] = i < 2 * nj ? h[2 * (size_t)j0 + i] : 0.0;
            __syncthreads();
            if (live) {
                for (int jb = njp - kDotVecs; jb >= 0; jb -= kDotVecs) {
                    double2 qv[kDotVecs];
#pragma unroll
                    for (int u = 0; u < kDotVecs; ++u) qv[u] = qvec(q, vstride, j0 + min(jb + u, nj - 1))[e];
                    __builtin_amdgcn_sched_barrier(0);  // keep the loads ahead of the arithmetic
#pragma unroll
                    for (int u = 0; u < kDotVecs; ++u) {
                        const double hr = hs[2 * (jb + u)], hi = hs[2 * (jb + u) + 1];
                        ar += hr * qv[u].x - hi * qv[u].y;
                        ai += hr * qv[u].y + hi * qv[u].x;
                    }
                }
            }
        }
        if (live) {
            double2 zv = z[e];
            zv.x -= ar;
            zv.y -= ai;
            z[e] = zv;
            zz[0] += zv.x * zv.x + zv.y * zv.y;
        }
    }
    double tot[1];
    if (!grid_reduce(zz, partials, &sc->ticket, tot)) return;
    double hh = 0.0;
    if (!second) {
        double s[1] = {0.0};
        for (int j = threadIdx.x; j < 2 * nvec; j += kBlock) s[0] += h[j] * h[j];
        __shared__ double red[kWaves][1];
        double b[1];
        block_partial(s, red, b);
        hh = b[0];
    }
    if (threadIdx.x != 0) return;
    if (sc->kstop >= nvec) alpha[nvec] += h[2 * (nvec - 1)];
    sc->again = !second && hh > kAgain * kAgain * tot[0];
    if (!sc->again) norm_update(tot[0], nvec, alpha, beta, sc);
}

// beta_0 = ||psi|| (grid-wide fixed-order reduction); kstop = 0 for psi = 0,
// status 3 when the norm is not finite.
__global__ __launch_bounds__(kBlock) void k_first_norm(const double2 *__restrict__ psi, size_t nelem,
                                                       Scalars *sc, double *beta, double *partials)
{
    double s[1] = {0.0};
    for (size_t e = (size_t)blockIdx.x * kBlock + threadIdx.x; e < nelem; e += (size_t)gridDim.x * kBlock) {
        const double2 v = psi[e];
        s[0] += v.x * v.x + v.y * v.y;
    }
    double tot[1];
    if (!grid_reduce(s, partials, &sc->ticket, tot)) return;
    if (threadIdx.x == 0) {
        const double b = sqrt(tot[0]);
        beta[0] = b;
        sc->scale = 0.0;
        sc->keff = 0;
        if (!isfinite(b)) {
            sc->status = 3;
            sc->kstop = -1;
        } else {
            sc->kstop = b > 0.0 ? 0x40000000 : 0;
        }
    }
}

// out = in / beta[idx] while the recurrence goes on past iteration idx.
__global__ __launch_bounds__(kBlock) void k_scale_q(const double2 *__restrict__ in, size_t nelem,
                                                    double2 *__restrict__ out, const double *beta, int idx,
                                                    const Scalars *sc)
{
    if (sc->kstop <= idx) return;
    const double ib = 1.0 / beta[idx];
    for (size_t e = (size_t)blockIdx.x * kBlock + threadIdx.x; e < nelem; e += (size_t)gridDim.x * kBlock) {
        const double2 v = in[e];
        out[e] = make_double2(v.x * ib, v.y * ib);
    }
}

// Ritz values of T_k in (lo, hi], one workgroup per value (blockIdx.x): Sturm
// counts of kBlock shifts at a time, so that a pass gains eight bits, and the last
// component of the unit eigenvector z from the twisted factorisation of T - theta
// (Parlett and Dhillon, Linear Algebra Appl. 267 (1997) 247): pivots p_i from the
// top, m_i from the bottom, the twist r where |p_r + m_r - (d_r - theta)| is smallest;
// z_r = 1, (z_i / z_{i+1})^2 = e_i^2 / p_i^2 above it and (z_{i+1} / z_i)^2 = e_i^2 /
// m_{i+1}^2 below.
// A count is the sign changes of the leading minors, f_i = (d_i - x) f_{i-1} -
// e_{i-1}^2 f_{i-2} with T scaled by a power of two to norm <= 1 and both minors
// rescaled every kRows rows: four instructions a row and no division (the pivots'
// recurrence waits about 60 cycles a row for its reciprocal).
// Bound: the chain of rows, 141 us a checkpoint on average to k = 1600, against
// 1.5 ms on the host, which was longer than the 64 iterations (0.68 ms at 1024^2)
// that it ran beside.
__global__ __launch_bounds__(kBlock) void k_ritz_window(const double *__restrict__ alpha,
                                                        const double *__restrict__ beta, int k, double lo, double hi,
                                                        const Scalars *sc, double *out)
{
    constexpr int kRows = 16;
    extern __shared__ double2 td[];  // (d_i, e_i^2) of the scaled matrix, then the pivots
    double *const top = reinterpret_cast<double *>(td + k), *const bot = top + k;
    __shared__ double red[kWaves];
    __shared__ int cnt[kWaves];
    __shared__ double res[4];
    const int t = (int)threadIdx.x, lane = t & 63, w = t >> 6;
    if (sc->kstop <= k) return;  // the recurrence has ended: the host solves its last T
    // power of two that takes the norm to at most 1
    double tn = 0.0;
    for (int i = t; i < k; i += kBlock) {
        const double l = i > 0 ? fabs(beta[i - 1]) : 0.0, r = i + 1 < k ? fabs(beta[i]) : 0.0;
        tn = fmax(tn, fabs(alpha[i]) + l + r);
    }
#pragma unroll
    for (int s = 32; s >= 1; s >>= 1) tn = fmax(tn, __shfl_xor(tn, s, 64));
    if (lane == 0) red[w] = tn;
    __syncthreads();
    for (int i = 0; i < kWaves; ++i) tn = fmax(tn, red[i]);
    const int ex = tn > 0.0 ? ilogb(tn) + 1 : 0;
    for (int i = t; i < k; i += kBlock) {
        const double e = i + 1 < k ? ldexp(beta[i], -ex) : 0.0;
        td[i] = make_double2(ldexp(alpha[i], -ex), e * e);
    }
    __syncthreads();
    // eigenvalues at or below x
    auto count = [&](double x) {
        double f1 = 0.0, f = 1.0, e2 = 0.0;
        int n = 0, i = 0;
        uint32_t sign = 0;  // of f
        auto row = [&](uint32_t &bits) {
            const double2 r = td[i++];
            const double g = fma(r.x - x, f, -(e2 * f1));
            f1 = f;
            f = g;
            e2 = r.y;
            bits = (bits << 1) | ((uint32_t)__double2hiint(f) >> 31);
        };
        while (i + kRows <= k) {
            uint32_t bits = sign;
#pragma unroll
            for (int j = 0; j < kRows; ++j) row(bits);
            n += __popc((bits ^ (bits >> 1)) & ((1u << kRows) - 1u));
            sign = bits & 1u;
            const int sh = -ilogb(fmax(fmax(fabs(f), fabs(f1)), 1e-290));
            f = ldexp(f, sh);
            f1 = ldexp(f1, sh);
        }
        while (i < k) {
            uint32_t bits = sign;
            row(bits);
            n += (int)((bits ^ (bits >> 1)) & 1u);
            sign = bits & 1u;
        }
        // a zero minor changes sign once with the next; a last one is negative
        if (f == 0.0) n += (f1 < 0.0) == (sign != 0u);
        return n;
    };
    // x within the wave's reach of every thread: how many of the shifts have a
    // count of at most `target`
    auto below = [&](double x, int target) {
        const int c = __popcll(__ballot(count(x) <= target));
        __syncthreads();
        if (lane == 0) cnt[w] = c;
        __syncthreads();
        int s = 0;
        for (int i = 0; i < kWaves; ++i) s += cnt[i];
        return s;
    };
    // every value lies in [-1, 1]; bounds far outside would overflow the minors
    // between two rescalings
    const double slo = fmin(fmax(ldexp(lo, -ex), -2.0), 2.0), shi = fmin(fmax(ldexp(hi, -ex), -2.0), 2.0);
    if (w == 0) {
        const int c = count(lane == 0 ? slo : shi);
        if (lane < 2) cnt[lane] = c;
    }
    __syncthreads();
    const int clo = cnt[0], nw = cnt[1] - clo, v = (int)blockIdx.x;
    if (v == 0 && t == 0) {
        out[0] = nw > kRitzMax ? -1.0 : (double)max(nw, 0);
        out[kRitzLen - 1] = beta[k - 1];
    }
    if (nw > kRitzMax || v >= nw) return;
    double a = slo, b = shi;  // the value lies in (a, b]
    for (int pass = 0; pass < 200; ++pass) {
        const double mid = 0.5 * (a + b);
        if (b - a <= 4.440892098500626e-16 * fmax(fabs(a), fabs(b)) + 1e-290 || mid <= a || mid >= b) break;
        auto point = [&](int i) { return fmin(fmax(a + (b - a) * ((double)(i + 1) / (double)(kBlock + 1)), a), b); };
        const int f = below(point(t), clo + v);
        const double na = f > 0 ? point(f - 1) : a, nb = f < kBlock ? point(f) : b;
        a = na;
        b = nb;
    }
    const double theta = 0.5 * (a + b);
    // pivots: negligible ones taken as negative
    auto keep = [](double q) { return fabs(q) < 1e-280 ? -1e-280 : q; };
    if (w == 0) {
        double q = 1.0, e2 = 0.0;
#pragma unroll 8
        for (int i = 0; i < k; ++i) {
            const double2 r = td[i];
            q = keep((r.x - theta) - e2 * recip(q));
            e2 = r.y;
            if (lane == 0) top[i] = q;
        }
    } else if (w == 1) {
        double q = 1.0;
#pragma unroll 8
        for (int i = k - 1; i >= 0; --i) {
            const double2 r = td[i];
            q = keep((r.x - theta) - r.y * recip(q));
            if (lane == 0) bot[i] = q;
        }
    }
    __syncthreads();
    double best = INFINITY;
    int twist = k;
    for (int i = t; i < k; i += kBlock) {
        const double g = fabs(top[i] + bot[i] - (td[i].x - theta));
        if (g < best) {
            best = g;
            twist = i;
        }
    }
    auto better = [&](double g, int i) {
        if (g < best || (g == best && i < twist)) {
            best = g;
            twist = i;
        }
    };
#pragma unroll
    for (int s = 32; s >= 1; s >>= 1) better(__shfl_xor(best, s, 64), __shfl_xor(twist, s, 64));
    if (lane == 0) {
        red[w] = best;
        cnt[w] = twist;
    }
    __syncthreads();
    for (int i = 0; i < kWaves; ++i) better(red[i], cnt[i]);
    if (twist >= k) twist = k - 1;  // (non-finite chain: the call fails on its scalars)
    // squared ratios of neighbouring components, away from the twist
    for (int i = t; i < k; i += kBlock) {
        if (i < twist) {
            const double r = recip(top[i]);
            top[i] = td[i].y * r * r;
        } else if (i > twist) {
            const double r = recip(bot[i]);
            bot[i] = td[i - 1].y * r * r;
        }
    }
    __syncthreads();
    if (t == 0) {
        double s = 0.0;
#pragma unroll 8
        for (int i = 0; i < twist; ++i) s = top[i] * (1.0 + s);
        res[0] = s;
    } else if (t == 64) {
        double s = 0.0, last = 1.0;
#pragma unroll 8
        for (int i = k - 1; i > twist; --i) {
            s = bot[i] * (1.0 + s);
            last *= bot[i];
        }
        res[1] = s;
        res[2] = last;
    }
    __syncthreads();
    if (t == 0) {
        out[1 + v] = ldexp(theta, ex);
        out[1 + kRitzMax + v] = sqrt(res[2] / (1.0 + res[0] + res[1]));
    }
}

// Y[:, v] = sum_j t[j][v] q_j for v < r: the basis is streamed once for up to
// kRitzVecs vectors; rows of t are staged in LDS.
__global__ __launch_bounds__(kBlock) void k_ritz(const char *__restrict__ q, size_t vstride, int nvec,
                                                 const double *__restrict__ t, int r, double2 *__restrict__ y,
                                                 size_t nelem)
{
    __shared__ double ts[kRitzChunk][kRitzVecs];
    const size_t step = (size_t)gridDim.x * kBlock;
    for (size_t base = (size_t)blockIdx.x * kBlock; base < nelem; base += step) {
        const size_t e = base + threadIdx.x;
        const bool live = e < nelem;
        double ar[kRitzVecs], ai[kRitzVecs];
#pragma unroll
        for (int v = 0; v < kRitzVecs; ++v) ar[v] = ai[v] = 0.0;
        for (int j0 = 0; j0 < nvec; j0 += kRitzChunk) {
            const int nj = min(kRitzChunk, nvec - j0);
            __syncthreads();
            for (int i = threadIdx.x; i < nj * kRitzVecs; i += kBlock)
                ts[i / kRitzVecs][i % kRitzVecs] = t[(size_t)j0 * kRitzVecs + i];
            __syncthreads();
            if (live)
                for (int jj = 0; jj < nj; ++jj) {
                    const double2 qv = qvec(q, vstride, j0 + jj)[e];
#pragma unroll
                    for (int v = 0; v < kRitzVecs; ++v) {
                        ar[v] += ts[jj][v] * qv.x;
                        ai[v] += ts[jj][v] * qv.y;
                    }
                }
        }
        if (live)
#pragma unroll
            for (int v = 0; v < kRitzVecs; ++v)
                if (v < r) y[(size_t)v * nelem + e] = make_double2(ar[v], ai[v]);
    }
}

}  // namespace

void launch_lanczos_local(const Op &op, const double2 *q, const double2 *qm, double2 *w, int i, double *alpha,
                          const double *beta, const Scalars *sc, double *partials, int nblocks, hipStream_t st)
{
    const size_t sites = (size_t)op.nx * op.ny;
    const int na = (int)std::min<size_t>((sites + kBlock - 1) / kBlock, nblocks);
    hipLaunchKernelGGL(k_eig_apply, dim3(na), dim3(kBlock), 0, st, op, q, w, partials);
    hipLaunchKernelGGL(k_local, dim3(nblocks), dim3(kBlock), 0, st, q, qm, w, 2 * sites, i, alpha, beta, sc, partials, na);
}

void launch_orth(const char *q, size_t vstride, int nvec, double2 *z, size_t nelem, double *pproj, double *h,
                 double *alpha, double *beta, Scalars *sc, double *partials, int nblocks, bool second,
                 hipStream_t st)
{
    const int nchunk = (nvec + kDotVecs - 1) / kDotVecs;
    const int ntiles = std::max(1, std::min(proj_tiles(nelem), (second ? kProjSecond : kProjWorkgroups) / nchunk));
    hipLaunchKernelGGL(k_proj, dim3(ntiles, nchunk), dim3(kBlock), 0, st, q, vstride, nvec, z, nelem, pproj, ntiles,
                       sc, (int)second);
    hipLaunchKernelGGL(k_proj_fold, dim3(nvec), dim3(kBlock), 0, st, pproj, ntiles, h, sc, (int)second);
    hipLaunchKernelGGL(k_sub_q, dim3(second ? std::min(nblocks, kProjSecond) : nblocks), dim3(kBlock), 0, st, q, vstride,
                       nvec, h, z, nelem, alpha, beta, sc, partials, (int)second);
}

void launch_first_q(const double2 *psi, size_t nelem, double2 *q1, Scalars *sc, double *beta, double *partials,
                    int nblocks, hipStream_t st)
{
    hipLaunchKernelGGL(k_first_norm, dim3(nblocks), dim3(kBlock), 0, st, psi, nelem, sc, beta, partials);
    hipLaunchKernelGGL(k_scale_q, dim3(nblocks), dim3(kBlock), 0, st, psi, nelem, q1, beta, 0, sc);
}

hipError_t launch_ritz_window(const double *alpha, const double *beta, int k, double lo, double hi, const Scalars *sc,
                              double *out, hipStream_t st)
{
    const size_t lds = 32 * (size_t)k;
    const hipError_t e = hipFuncSetAttribute(reinterpret_cast<const void *>(k_ritz_window),
                                             hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds);
    if (e != hipSuccess) return e;
    hipLaunchKernelGGL(k_ritz_window, dim3(kRitzMax), dim3(kBlock), lds, st, alpha, beta, k, lo, hi, sc, out);
    return hipGetLastError();
}

void launch_next_q(const double2 *z, size_t nelem, int i, const double *beta, const Scalars *sc, double2 *qn,
                   int nblocks, hipStream_t st)
{
    hipLaunchKernelGGL(k_scale_q, dim3(nblocks), dim3(kBlock), 0, st, z, nelem, qn, beta, i, sc);
}

void launch_ritz(const char *q, size_t vstride, int nvec, const double *t, int r, double2 *y, size_t nelem,
                 int nblocks, hipStream_t st)
{
    hipLaunchKernelGGL(k_ritz, dim3(nblocks), dim3(kBlock), 0, st, q, vstride, nvec, t, r, y, nelem);
}

}  // namespace dl
