// Hermite pseudospectral discretisation (Sec. 5 of Beerwerth & Bauke,
// arXiv:1407.7370) on gfx950: each spinor component is held at the n x n
// collocation points (x_i, y_j) in the variables phi = sqrt(w_i w_j) psi, and
// the derivatives are dense n x n matrices, so H phi is a set of dense
// contractions -- the one matrix-shaped workload of the method.  They run on
// the FP64 matrix cores (v_mfma_f64_16x16x4f64).
//
// One workgroup (eight wave64, two per SIMD) owns one problem and runs the
// whole Lanczos recurrence of the eigenvalue mode (Sec. 2, Fig. 1 order) in a
// single launch.  The Lanczos vectors never leave the compute unit: z and q
// live in registers in the matrix-core output layout (each wave owns two
// 16 x 16 tiles of the n x n planes), and the matrix products read D and one
// component of q at a time from LDS.  A batch of problems (other Z, fields,
// chirality) runs on as many compute units.  For n = 32 and 64 the vectors are
// held in the parity basis (HermOp::split), where the products are half as long:
// 16 n^3 flops per iteration become 8 n^3.
// What bounds it: the matrix cores (n = 64: 6.9 us of an iteration at a compute
// unit's share of 78.6 TFLOP/s), then the two block sums and the staging of q.
// 256 problems x 1000 iterations: 22.0 ms with full products and the potential
// evaluated in every iteration, 13.8 in the parity basis, 12.2 with the potential
// in LDS and one barrier per block sum.
#include <hip/hip_runtime.h>

#include <cmath>

#include "device_reduce.h"
#include "dl_internal.h"

namespace dl {
namespace {

typedef double v4d __attribute__((ext_vector_type(4)));

__device__ __forceinline__ v4d mfma(double a, double b, v4d c)
{
    return __builtin_amdgcn_mfma_f64_16x16x4f64(a, b, c, 0, 0, 0);
}

constexpr int kHermMaxN = 64;
constexpr int kHermWaves = 8;
constexpr int kHermBlock = 64 * kHermWaves;
constexpr int kTilesPerWave = 16 / kHermWaves;  // (64/16)^2 tiles over the waves
// LDS row strides: lane (r, k) of an operand read hits bank group 4r + 2k
// (D, doubles) or r (a staged component, 16-byte values), so the 16 rows of
// a read are on distinct banks.
constexpr int kDStride = 66;
constexpr int kPStride = 65;

struct HermLds {
    double d[kHermMaxN * kDStride];    // D~ / scale
    double2 p[kHermMaxN * kPStride];   // one component of the vector being multiplied
    double x[kHermMaxN];               // scaled nodes
    double v[kHermMaxN * kHermMaxN];   // potential of the sites
    double red[2][kHermWaves];         // block sums, alternating
};

typedef v4d Tiles[kTilesPerWave][4];  // planes: Re phi_0, Im phi_0, Re phi_1, Im phi_1

__device__ __forceinline__ double herm_potential(const HermOp &op, double x, double y)
{
    if (op.pot_kind == 1) return -op.vz / sqrt(x * x + y * y + op.va2);
    return 0.0;
}

// Block-wide sum (fixed order: lane permutations in the wave, then waves in
// order).  Consecutive sums alternate between the rows of `red`, so that one
// barrier each is enough.
__device__ double block_sum(double v, double (&red)[2][kHermWaves], int &turn)
{
    v = lanes_sum(v);
    const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
    double *const r = red[turn];
    turn ^= 1;
    if (lane == 0) r[w] = v;
    __syncthreads();
    double t = 0.0;
#pragma unroll
    for (int i = 0; i < kHermWaves; ++i) t += r[i];
    return t;
}

// Visit every element of the wave's tiles: f(tt, r, row, col).  Tile t of
// wave w (t = w + kHermWaves tt) covers rows (y) 16 (t / nt) .. and columns (x)
// 16 (t mod nt) ..; element (i, j) of a tile sits in lane j + 16 (i mod 4),
// register i / 4 of the matrix-core output.
template <class F>
__device__ __forceinline__ void herm_tiles(const HermOp &op, F &&f)
{
    const int nt = op.n / 16, ntiles = nt * nt;
    const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
#pragma unroll
    for (int tt = 0; tt < kTilesPerWave; ++tt) {
        const int t = w + kHermWaves * tt;
        if (t >= ntiles) continue;
        const int r0 = 16 * (t / nt), c0 = 16 * (t % nt);
#pragma unroll
        for (int r = 0; r < 4; ++r) f(tt, r, r0 + 4 * r + (lane >> 4), c0 + (lane & 15));
    }
}

// Component s of the tiles' vector into the LDS staging plane.
__device__ __forceinline__ void herm_put(const HermOp &op, HermLds &L, const Tiles &q, int s)
{
    herm_tiles(op, [&](int tt, int r, int row, int col) {
        L.p[row * kPStride + col] = make_double2(q[tt][2 * s][r], q[tt][2 * s + 1][r]);
    });
}

// Derivative terms of the staged component into planes P, P + 1 of acc:
// c (-i) D_x phi (the x-derivative, phi D^T along rows) plus sy D_y phi (the
// y-derivative, D phi along columns), both with D = D~ / scale:
//   acc_P   += c Im(phi) D_x^T + sy D_y Re(phi)
//   acc_P+1 -= c Re(phi) D_x^T - sy D_y Im(phi)
template <int P>
__device__ __forceinline__ void herm_deriv(const HermOp &op, const HermLds &L, Tiles &acc, double sy)
{
    const int n = op.n, nt = n / 16, ntiles = nt * nt, nk = op.split ? n / 8 : n / 4;
    const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
    const int lr = lane & 15, lk = lane >> 4;
    const double c = op.c;
#pragma unroll
    for (int tt = 0; tt < kTilesPerWave; ++tt) {
        const int t = w + kHermWaves * tt;
        if (t >= ntiles) continue;
        const int r0 = 16 * (t / nt), c0 = 16 * (t % nt);
        // columns k of D that are not zero in this tile's rows: all, or the
        // half of the other parity
        const int kx = op.split && c0 < n / 2 ? n / 2 : 0, ky = op.split && r0 < n / 2 ? n / 2 : 0;
        const double2 *pa = L.p + (r0 + lr) * kPStride + kx + lk;    // A of the x-product: phi[r0 + lr][k]
        const double2 *pb = L.p + (ky + lk) * kPStride + c0 + lr;    // B of the y-product: phi[k][c0 + lr]
        const double *dx = L.d + (c0 + lr) * kDStride + kx + lk;     // B of the x-product: D[c0 + lr][k]
        const double *dy = L.d + (r0 + lr) * kDStride + ky + lk;     // A of the y-product: D[r0 + lr][k]
        v4d a0 = acc[tt][P], a1 = acc[tt][P + 1];
        // four operand groups at a time, their LDS reads ahead of the products
        // (nk is a multiple of four)
        for (int k4 = 0; k4 < nk; k4 += 4) {
            double2 fa[4], fb[4];
            double ex[4], ey[4];
#pragma unroll
            for (int u = 0; u < 4; ++u) {
                fa[u] = pa[4 * (k4 + u)];
                fb[u] = pb[4 * (k4 + u) * kPStride];
                ex[u] = dx[4 * (k4 + u)];
                ey[u] = dy[4 * (k4 + u)];
            }
#pragma unroll
            for (int u = 0; u < 4; ++u) {
                a0 = mfma(c * fa[u].y, ex[u], a0);
                a1 = mfma(-c * fa[u].x, ex[u], a1);
                a0 = mfma(ey[u], sy * fb[u].x, a0);
                a1 = mfma(ey[u], sy * fb[u].y, a1);
            }
        }
        acc[tt][P] = a0;
        acc[tt][P + 1] = a1;
    }
}

// Magnetic coupling of the staged component in the parity basis: x and y change
// the parity, so the factor multiplies the partner (the same node, the other
// parity) of the element.  Planes P, P + 1 of z += (gx -+ i chi gy) q_s, sign
// +1 for the lower component's coupling to the upper (P = 0), -1 for P = 2.
template <int P>
__device__ __forceinline__ void herm_field_split(const HermOp &op, const HermLds &L, Tiles &z)
{
    if (op.bq == 0.0) return;
    const int h = op.n / 2;
    herm_tiles(op, [&](int tt, int r, int row, int col) {
        const double2 fy = L.p[(row < h ? row + h : row - h) * kPStride + col];
        const double2 fx = L.p[row * kPStride + (col < h ? col + h : col - h)];
        const double gx = op.bq * L.x[row], gy = (P == 0 ? 1.0 : -1.0) * -op.bq * L.x[col] * op.chi;
        z[tt][P][r] += gx * fy.x + gy * fx.y;
        z[tt][P + 1][r] += gx * fy.y - gy * fx.x;
    });
}

// z += H q on the wave's tiles (q and z in the output layout):
//   (H q)_0 = (mc2 + V) q_0 + c [-i D_x q_1 - chi D_y q_1] - q c (A_x - i chi A_y) q_1
//   (H q)_1 = (V - mc2) q_1 + c [-i D_x q_0 + chi D_y q_0] - q c (A_x + i chi A_y) q_0
__device__ void herm_matvec(const HermOp &op, HermLds &L, const Tiles &q, Tiles &z)
{
    const double cchi = op.c * op.chi;
    __syncthreads();  // the staging plane is free
    herm_put(op, L, q, 1);
    __syncthreads();
    herm_deriv<0>(op, L, z, -cchi);
    if (op.split) herm_field_split<0>(op, L, z);
    __syncthreads();
    herm_put(op, L, q, 0);
    __syncthreads();
    herm_deriv<2>(op, L, z, cchi);
    if (op.split) herm_field_split<2>(op, L, z);
    // site terms (the potential is even in x and y)
    const double bq = op.split ? 0.0 : op.bq;
    herm_tiles(op, [&](int tt, int r, int row, int col) {
        const double x = L.x[col], y = L.x[row];
        const double v = L.v[row * op.n + col];
        const double d0 = op.mc2 + v, d1 = v - op.mc2;
        // g = -q c A with A = (B/2)(-y, x): gx = bq y, chi gy = -chi bq x
        // (bq = c q B / 2); coupling (gx -+ i chi gy) to the other component
        const double gx = bq * y, gy = -bq * x * op.chi;
        const double f0x = q[tt][0][r], f0y = q[tt][1][r], f1x = q[tt][2][r], f1y = q[tt][3][r];
        z[tt][0][r] += d0 * f0x + gx * f1x + gy * f1y;
        z[tt][1][r] += d0 * f0y + gx * f1y - gy * f1x;
        z[tt][2][r] += d1 * f1x + gx * f0x - gy * f0y;
        z[tt][3][r] += d1 * f1y + gx * f0y + gy * f0x;
    });
}

// Stage D~ / scale and the scaled nodes of a problem in LDS.
__device__ void herm_stage(const HermOp &op, HermLds &L)
{
    const int n = op.n;
    for (int i = threadIdx.x; i < n * n; i += kHermBlock) L.d[(i / n) * kDStride + (i % n)] = op.dmat[i];
    for (int i = threadIdx.x; i < n; i += kHermBlock) L.x[i] = op.x[i];
    __syncthreads();
    for (int i = threadIdx.x; i < n * n; i += kHermBlock) L.v[i] = herm_potential(op, L.x[i % n], L.x[i / n]);
    __syncthreads();
}

// A global spinor (layout (2, n, n)) at the wave's tile elements.
__device__ void herm_load(const HermOp &op, const double2 *__restrict__ v, Tiles &q)
{
    const size_t plane = (size_t)op.n * op.n;
#pragma unroll
    for (int tt = 0; tt < kTilesPerWave; ++tt)
#pragma unroll
        for (int p = 0; p < 4; ++p) q[tt][p] = v4d{0.0, 0.0, 0.0, 0.0};
    if (op.split) {
        // (f(i,j) +- f(i,J) +- f(I,j) + .. f(I,J)) / 2 with I, J the mirror nodes
        const int n = op.n, h = n / 2;
        herm_tiles(op, [&](int tt, int r, int row, int col) {
            const int i = row % h, j = col % h;
            const double sr = row < h ? 1.0 : -1.0, sc = col < h ? 1.0 : -1.0;
            const size_t s00 = (size_t)i * n + j, s01 = (size_t)i * n + (n - 1 - j), s10 = (size_t)(n - 1 - i) * n + j,
                         s11 = (size_t)(n - 1 - i) * n + (n - 1 - j);
#pragma unroll
            for (int c = 0; c < 2; ++c) {
                const double2 *f = v + (size_t)c * plane;
                const double2 a = f[s00], b = f[s01], d = f[s10], e = f[s11];
                q[tt][2 * c][r] = 0.5 * ((a.x + sc * b.x) + sr * (d.x + sc * e.x));
                q[tt][2 * c + 1][r] = 0.5 * ((a.y + sc * b.y) + sr * (d.y + sc * e.y));
            }
        });
        return;
    }
    herm_tiles(op, [&](int tt, int r, int row, int col) {
        const size_t s = (size_t)row * op.n + col;
        const double2 a = v[s], b = v[plane + s];
        q[tt][0][r] = a.x;
        q[tt][1][r] = a.y;
        q[tt][2][r] = b.x;
        q[tt][3][r] = b.y;
    });
}

__global__ __launch_bounds__(kHermBlock) void k_herm_apply(const HermOp *ops, const double2 *const *x,
                                                           double2 *const *y)
{
    __shared__ HermLds L;
    const HermOp op = ops[blockIdx.x];
    herm_stage(op, L);
    Tiles q, z;
    herm_load(op, x[blockIdx.x], q);
#pragma unroll
    for (int tt = 0; tt < kTilesPerWave; ++tt)
#pragma unroll
        for (int p = 0; p < 4; ++p) z[tt][p] = v4d{0.0, 0.0, 0.0, 0.0};
    herm_matvec(op, L, q, z);
    double2 *out = y[blockIdx.x];
    const size_t plane = (size_t)op.n * op.n;
    herm_tiles(op, [&](int tt, int r, int row, int col) {
        const size_t s = (size_t)row * op.n + col;
        out[s] = make_double2(z[tt][0][r], z[tt][1][r]);
        out[plane + s] = make_double2(z[tt][2][r], z[tt][3][r]);
    });
}

// The Lanczos recurrence of Fig. 1 (three vectors, no reorthogonalisation)
// on one problem per workgroup:
//   q_1 = b / ||b||; z = H q_1;
//   i = 1..k: alpha_i = Re <q_i, z>; z -= alpha_i q_i; beta_i = ||z||;
//             stop at k or on breakdown (beta_i <= 1e-13 max_j(|alpha_j|, beta_{j-1}));
//             q_{i+1} = z / beta_i; z = H q_{i+1} - beta_i q_i.
// Every element of the n x n planes belongs to exactly one lane and register
// of one wave, so the inner products are sums over the tiles.  Two vectors
// are live: q (q_i, then q_{i+1}) and z, which starts a product as -beta_i q_i.
__global__ __launch_bounds__(kHermBlock) void k_herm_lanczos(const HermOp *ops, HermRun *runs, int k_max)
{
    __shared__ HermLds L;
    const HermOp op = ops[blockIdx.x];
    HermRun &run = runs[blockIdx.x];
    herm_stage(op, L);
    Tiles qn, z;
    herm_load(op, run.b, qn);
    int turn = 0;
    double s = 0.0;
    herm_tiles(op, [&](int tt, int r, int, int) {
#pragma unroll
        for (int p = 0; p < 4; ++p) s += qn[tt][p][r] * qn[tt][p][r];
    });
    const double nb2 = block_sum(s, L.red, turn);
    if (!(nb2 > 0.0) || !isfinite(nb2)) {
        if (threadIdx.x == 0) run.keff = isfinite(nb2) ? 0 : -1;
        return;
    }
    const double inb = 1.0 / sqrt(nb2);
#pragma unroll
    for (int tt = 0; tt < kTilesPerWave; ++tt)
#pragma unroll
        for (int p = 0; p < 4; ++p) {
            qn[tt][p] *= inb;
            z[tt][p] = v4d{0.0, 0.0, 0.0, 0.0};
        }
    herm_matvec(op, L, qn, z);
    double scale = 0.0, beta_prev = 0.0;
    int keff = k_max;
    for (int i = 1; i <= k_max; ++i) {
        double pa = 0.0;
        herm_tiles(op, [&](int tt, int r, int, int) {
#pragma unroll
            for (int p = 0; p < 4; ++p) pa += qn[tt][p][r] * z[tt][p][r];
        });
        const double alpha = block_sum(pa, L.red, turn);
        double pn = 0.0;
        herm_tiles(op, [&](int tt, int r, int, int) {
#pragma unroll
            for (int p = 0; p < 4; ++p) {
                z[tt][p][r] -= alpha * qn[tt][p][r];
                pn += z[tt][p][r] * z[tt][p][r];
            }
        });
        const double beta = sqrt(block_sum(pn, L.red, turn));
        if (threadIdx.x == 0) {
            run.alpha[i - 1] = alpha;
            run.beta[i - 1] = beta;
        }
        if (!isfinite(alpha) || !isfinite(beta)) {
            keff = -1;
            break;
        }
        scale = fmax(scale, fabs(alpha));
        if (i > 1) scale = fmax(scale, beta_prev);
        if (i == k_max) break;
        if (beta <= 1e-13 * scale) {
            keff = i;
            break;
        }
        // q_{i+1} = z / beta_i; z = H q_{i+1} - beta_i q_i
        const double ib = 1.0 / beta;
#pragma unroll
        for (int tt = 0; tt < kTilesPerWave; ++tt)
#pragma unroll
            for (int p = 0; p < 4; ++p) {
                const v4d next = z[tt][p] * ib;
                z[tt][p] = -beta * qn[tt][p];
                qn[tt][p] = next;
            }
        herm_matvec(op, L, qn, z);
        beta_prev = beta;
    }
    if (threadIdx.x == 0) run.keff = keff;
}

// Ritz values of one leading block (blockIdx.y: checkpoint, the largest first) of
// one problem by one wave: T in LDS, Sturm counts of 64 shifts at a time (the
// signs of the pivots of the LDL^T factorisation of T - x, a negligible pivot
// taken as negative, as the host's bisection), the lanes shared out over the
// values of the window, so that a lone value gains six bits a pass.
// The last component of a value's eigenvector z comes from the twisted
// factorisation of T - theta (Parlett and Dhillon, Linear Algebra Appl. 267 (1997)
// 247): pivots p_i from the top, m_i from the bottom, the twist r where |p_r + m_r
// - (d_r - theta)| is smallest; z_r = 1, z_i / z_(i+1) = -e_i / p_i above it and
// z_(i+1) / z_i = -e_i / m_(i+1) below, so the squared components add up along
// either recurrence.
// Bound: chains of reciprocals (about 60 cycles a row and pass).  256 problems x
// 16 checkpoints of up to 1000 rows: 2.0 ms, 23 ms on the host's 16 threads.
__global__ __launch_bounds__(64) void k_herm_ritz(const HermRun *runs, const double *windows, int k_max, int every,
                                                  int ncheck, double *out)
{
    extern __shared__ double2 td[];                           // (alpha_i, beta_i)
    double *const piv = reinterpret_cast<double *>(td + k_max);  // pivots from the top
    const int prob = (int)blockIdx.x, c = ncheck - 1 - (int)blockIdx.y, lane = (int)threadIdx.x;
    const HermRun run = runs[prob];
    double *o = out + ((size_t)prob * ncheck + c) * kHermRitzLen;
    if (run.keff <= c * every) {  // no such block
        if (lane == 0) o[0] = 0.0;
        return;
    }
    const int k = min((c + 1) * every, run.keff);
    if (k < 2) {
        if (lane == 0) o[0] = -1.0;
        return;
    }
    double emax2 = 0.0;
    for (int i = lane; i < k; i += 64) {
        const double a = run.alpha[i], b = run.beta[i];
        td[i] = make_double2(a, b);
        if (i + 1 < k) emax2 = fmax(emax2, b * b);
    }
#pragma unroll
    for (int s = 32; s >= 1; s >>= 1) emax2 = fmax(emax2, __shfl_xor(emax2, s, 64));
    __syncthreads();
    const double pivmin = 1e-280 * fmax(1.0, emax2);  // (quotients by it stay finite)
    // eigenvalues at or below x
    auto count = [&](double x) {
        double2 t = td[0];
        double q = t.x - x;
        if (fabs(q) < pivmin) q = -pivmin;
        int n = q < 0.0;
#pragma unroll 4
        for (int i = 1; i < k; ++i) {
            const double b2 = t.y * t.y;
            t = td[i];
            q = (t.x - x) - b2 * recip(q);
            if (fabs(q) < pivmin) q = -pivmin;
            n += q < 0.0;
        }
        return n;
    };
    const double lo = windows[2 * prob], hi = windows[2 * prob + 1];
    const int cnt = count(lane == 0 ? lo : hi);
    const int clo = __shfl(cnt, 0, 64), nw = __shfl(cnt, 1, 64) - clo;
    if (nw <= 0 || nw > kHermRitzMax) {
        if (lane == 0) {
            o[0] = nw <= 0 ? 0.0 : -1.0;
            o[1] = td[k - 1].y;
        }
        return;
    }
    // 64 / groups lanes per value (groups: the power of two >= nw)
    int groups = 1;
    while (groups < nw) groups *= 2;
    const int per = 64 / groups, g = lane / per, r = lane % per;
    const int target = clo + min(g, nw - 1);
    const unsigned long long mask = (per == 64 ? ~0ull : ((1ull << per) - 1ull)) << (g * per);
    double a = lo, b = hi;  // the value of this group lies in (a, b]
    for (int pass = 0; pass < 1100; ++pass) {
        const double mid = 0.5 * (a + b);
        const bool open = !(b - a <= 4.440892098500626e-16 * fmax(fabs(a), fabs(b)) + 2.0 * pivmin || mid <= a || mid >= b);
        if (__ballot(open) == 0ull) break;
        const double x = fmin(fmax(a + (b - a) * ((double)(r + 1) / (double)(per + 1)), a), b);
        const unsigned long long above = __ballot(count(x) > target) & mask;
        // first point of the group above the value, and the point before it
        const int f = above ? __ffsll((long long)above) - 1 : (g + 1) * per;
        const double xf = __shfl(x, min(f, 63), 64), xb = __shfl(x, max(f - 1, 0), 64);
        if (open) {
            if (f > g * per) a = xb;
            if (f < (g + 1) * per) b = xf;
        }
    }
    const double theta_g = 0.5 * (a + b);
    if (lane == 0) {
        o[0] = (double)nw;
        o[1] = td[k - 1].y;
    }
    for (int v = 0; v < nw; ++v) {
        const double theta = __shfl(theta_g, v * per, 64);
        auto keep = [&](double q) { return fabs(q) < pivmin ? -pivmin : q; };
        double2 t = td[0];
        double q = keep(t.x - theta);
        if (lane == 0) piv[0] = q;
        for (int i = 1; i < k; ++i) {
            const double b2 = t.y * t.y;
            t = td[i];
            q = keep((t.x - theta) - b2 * recip(q));
            if (lane == 0) piv[i] = q;
        }
        __syncthreads();
        // from the bottom: squared components below row i (z_i = 1) and |z_k|
        double m = keep(td[k - 1].x - theta), below = 0.0, last = 1.0;
        double best = fabs(piv[k - 1]), best_below = 0.0, best_last = 1.0;
        int twist = k - 1;
        for (int i = k - 2; i >= 0; --i) {
            const double2 ti = td[i];
            const double s = ti.y * recip(m);
            below = s * s * (1.0 + below);
            last *= fabs(s);
            const double gamma = fabs(piv[i] - ti.y * s);
            m = keep((ti.x - theta) - ti.y * s);
            if (gamma < best) {
                best = gamma;
                best_below = below;
                best_last = last;
                twist = i;
            }
        }
        double above = 0.0;
        for (int i = 0; i < twist; ++i) {
            const double s = td[i].y * recip(piv[i]);
            above = s * s * (1.0 + above);
        }
        if (lane == 0) {
            o[2 + v] = theta;
            o[2 + kHermRitzMax + v] = best_last / sqrt(1.0 + above + best_below);
        }
        __syncthreads();
    }
}

}  // namespace

void launch_herm_ritz(const HermRun *runs, const double *windows, int n, int k_max, int every, int ncheck, double *out,
                      hipStream_t st)
{
    hipLaunchKernelGGL(k_herm_ritz, dim3(n, ncheck), dim3(64), (sizeof(double2) + sizeof(double)) * (size_t)k_max, st, runs,
                       windows, k_max, every, ncheck, out);
}

void launch_herm_apply(const HermOp *ops, const double2 *const *x, double2 *const *y, int n, hipStream_t st)
{
    hipLaunchKernelGGL(k_herm_apply, dim3(n), dim3(kHermBlock), 0, st, ops, x, y);
}

void launch_herm_lanczos(const HermOp *ops, HermRun *runs, int n, int k_max, hipStream_t st)
{
    hipLaunchKernelGGL(k_herm_lanczos, dim3(n), dim3(kHermBlock), 0, st, ops, runs, k_max);
}

}  // namespace dl
