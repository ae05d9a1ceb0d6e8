// Time steps of small and middle grids in one launch.  A sweep kernel per
// Lanczos iteration costs about 11 us on such grids whatever their size (the
// dispatch, the fold of the last iteration's partials, a chain of memory round
// trips), so here the whole propagation runs in a resident kernel: one
// workgroup per compute unit holds a tile of the grid in LDS and registers, and
// the workgroups exchange the reductions and the tile borders themselves.
//
// Per iteration p >= 2 a workgroup forms u_p on its tile and a one-site rim
// (from u_{p-1}, held in LDS with the rim and the sites at distance two, and
// u_{p-2}, held in registers by the thread that owns the site), publishes the
// border values that its neighbours need at distance two, applies A u_p on the
// tile and publishes its partial sums; it then collects all partial sums (folded
// in the same order by every workgroup, so all agree bit for bit on alpha_p and
// gamma_p and on every branch) and its own border.  This is the arithmetic of
// the sweeps (sweeps.h) per site; only the order of the reductions differs.
// Basis vectors are stored to memory for the recombination alone, which each
// thread does for its own sites; nothing waits for those stores.
//
// Exchange without flags or fences: every 8-byte word carries 32 bits of
// payload and the 32-bit epoch number it belongs to, is written with one
// device-scope 8-byte store and polled with device-scope 8-byte loads until the
// epoch matches, so data and validity arrive together (one store-to-load
// latency per iteration).  Words alternate between two buffers; a workgroup
// writes epoch e + 2 only after it has seen every partial of e + 1, which each
// workgroup sends after it has consumed epoch e.  Every call clears the words
// first (k_reset), and its launches have epoch numbers of their own
// (reserve_epochs), so neither what was in the memory before the call nor words
// of the call's earlier launches match.
//
// The partial sums of more than kDirect workgroups go through kLeaders of them
// (each adds its group's and posts the group's sum), because every workgroup
// polling every other's words saturates the few memory channels that hold them
// (512^2: 12.3 us an iteration, of which 6 us for the sums).
//
// All workgroups must be resident at once: the launch is cooperative.  Every
// wait is bounded in time (ResidentArgs::wait_ticks from the launch's start), after
// which the workgroups leave and the host runs what is left as sweeps.
//
// What bounds it: the latency chain of an iteration (partials and border
// through memory, workgroup barriers, the tile's arithmetic: 3.2 us at 64^2, 5.9
// at 512^2) on small grids, FP64 arithmetic and LDS traffic of a tile and the
// basis stores on the largest (13 us at 1024^2, of which 3 us are the stores).
// Measured per step, as sweeps before and here: 64^2 m = 10 124 -> 47 us, 512^2
// m = 12 161 -> 99 us, 1024^2 with potential and field m = 20 640 -> 461 us,
// 1001 x 777 complex64 m = 13 364 -> 184 us.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <atomic>

#include "sweeps.h"

namespace dl {
namespace {

constexpr int kRBlock = kResidentThreads;
constexpr int kRWaves = kRBlock / 64;
constexpr int kPollWave = kRWaves - 1;  // wave that collects the sums (no border slots: kResidentSlots)
static_assert(kResidentSlots <= 64 * kPollWave, "the polling wave has no border slots");
constexpr int kDirect = 64;   // workgroups whose sums every workgroup reads directly
constexpr int kLeaders = 16;  // groups beyond that,
constexpr int kGroup = 16;    // of at most 16 workgroups
constexpr int kCopies = 8;    // copies of the groups' sums
static_assert(kLeaders * kGroup >= kResidentWgs, "every workgroup has a group");
static_assert(kCommRed >= sizeof(unsigned long long) * 2 * 10 * (kLeaders * kGroup + kLeaders * kCopies),
              "the exchange buffers hold the sums");

__device__ __forceinline__ void put_word(unsigned long long *p, uint32_t payload, uint32_t epoch)
{
    __hip_atomic_store(p, ((unsigned long long)epoch << 32) | payload, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

__device__ __forceinline__ unsigned long long get_word(const unsigned long long *p)
{
    return __hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

__device__ __forceinline__ double join(unsigned long long lo, unsigned long long hi)
{
    return __hiloint2double((int)(uint32_t)hi, (int)(uint32_t)lo);
}

// Words of one published site: the four reals in storage precision.
template <class T>
constexpr int kSiteWords = sizeof(T) == 16 ? 8 : 4;

// Basis vectors that only this kernel reads are stored tile by tile, the tile's
// rows one after the other, complex128 ones in two planes per tile: a wave reads
// and writes whole lines and no line belongs to two workgroups (rows of the grid
// with 32 bytes a site: 1024^2 m = 20 429 us a step, 400 so; 724^2 m = 12 151 and 142;
// 512^2 and smaller the same).  Vectors that later kernels read (the adjoint's) are
// laid out as the sweeps write them.
template <class T, int POL>
__device__ __forceinline__ Raw<T> ld_site_at(__amdgpu_buffer_rsrc_t r, uint32_t off, uint32_t second)
{
    if constexpr (sizeof(T) == 8) {
        return ld16<Raw<T>, POL>(r, off);
    } else {
        Raw<T> v;
        v.a = ld16<T, POL>(r, off);
        v.b = ld16<T, POL>(r, off + second);
        return v;
    }
}
template <class T>
__device__ __forceinline__ void st_site(__amdgpu_buffer_rsrc_t r, uint32_t off, uint32_t second, const Raw<T> &v)
{
    if constexpr (sizeof(T) == 8) {
        st16<Raw<T>, kPolDefault>(r, off, v);
    } else {
        st16<T, kPolDefault>(r, off, v.a);
        st16<T, kPolDefault>(r, off + second, v.b);
    }
}

// Potential of a site, or zero terms, precomputed per thread.
template <int K, int TERMS>
struct SitePot {
    double v[K];
};
template <int K>
struct SitePot<K, 0> {};

// 1.0 where bit k of the mask is set, else 0.0.
__device__ __forceinline__ double bit_one(uint32_t mask, int k)
{
    return __hiloint2double(((int)(mask << (31 - k)) >> 31) & 0x3FF00000, 0);
}

struct ResidentShared {
    double part[kRWaves][5];  // partial sums of this workgroup's waves
    double tot[5];            // totals over the workgroups
    double al[kMaxM + 3], ga[kMaxM + 3];
    double coef[2 * (kMaxM + 2)];
    double wre[kMaxM], wim[kMaxM];
    double cabs;
    unsigned long long deadline;  // of this workgroup's waits
    int dead, scratch;
};

// The workgroup's LDS: one object for the kernel and the functions it calls, so
// that both address it as LDS (through a pointer argument it would be accessed
// by flat loads, which wait for the basis stores still in flight).
__device__ __forceinline__ ResidentShared &shared_state()
{
    __shared__ ResidentShared sh;
    return sh;
}
extern __shared__ double2 resident_tile[];

// The eigendecomposition of a wide spectrum, with the tile as scratch.  A call
// of its own, so that its registers are not the kernel's.
__device__ __attribute__((noinline)) void resident_qr(double d, double e, int k)
{
    ResidentShared &sh = shared_state();
    const int lane = (int)threadIdx.x & 63;
    double cr, ci;
    qr_exp_e1(d, e, k, lane, reinterpret_cast<double *>(resident_tile), sh.wre, sh.wim, cr, ci);
    wave_sync();
    if (lane < k) {
        sh.wre[lane] = cr;
        sh.wim[lane] = ci;
    }
    wave_sync();
}

// The small exponential of one step from the chain in LDS (one wave):
// coefficients c_j / gamma_j, |c_k| and whether the tile was overwritten.
__device__ __forceinline__ void resident_exp(ResidentShared &sh, int k, double sig)
{
    const int lane = (int)threadIdx.x & 63;
    const double d = lane < k ? sh.al[lane + 1] : 0.0, e = lane + 1 < k ? sh.ga[lane + 2] : 0.0;
    double em = from_left(e);
    if (lane == 0) em = 0.0;
    double cr = 0.0, ci = 0.0;
    const bool wide = !cheb_exp_e1(d, e, em, k, lane, cr, ci);
    if (wide) {
        resident_qr(d, e, k);
        if (lane < k) {
            cr = sh.wre[lane];
            ci = sh.wim[lane];
        }
    }
    if (lane == 0) sh.scratch = wide;
    if (lane < k) {
        double ss, cc;
        sincos(sig, &ss, &cc);
        const double g1 = sh.ga[1], ig = 1.0 / sh.ga[lane + 1];
        const double tr = g1 * (cr * cc + ci * ss), ti = g1 * (ci * cc - cr * ss);
        sh.coef[2 * (lane + 1)] = tr * ig;
        sh.coef[2 * (lane + 1) + 1] = ti * ig;
        if (lane == k - 1) sh.cabs = sqrt(tr * tr + ti * ti);
    }
}

__device__ __attribute__((noinline)) void resident_exp_call(int k, double sig) { resident_exp(shared_state(), k, sig); }

// An opaque copy: per-row masks and addresses derived from it are computed
// where they are used instead of being kept in registers over the whole launch
// (which spills).
template <class X>
__device__ __forceinline__ void opaque(X &x)
{
    asm volatile("" : "+v"(x));
}

// EIG: iterations p0 .. p1 of the plain recurrence of the eigen mode in place of
// time steps (ResidentEigen): no basis, no exponential; u_{p0-1} and u_{p0-2} are
// read from memory first and u_{p1}, u_{p1-1} written last.
template <class TO, int K, int TERMS, bool EIG>
__global__ __launch_bounds__(kRBlock) void k_resident(ResidentArgs a)
{
    double2 *const tile = resident_tile;
    ResidentShared &sh = shared_state();
    Scalars *sc = a.sc;
    if (sc->status != 0) return;
    if constexpr (EIG)
        if (sc->kstop < a.eig.p0) return;
    constexpr int NW = kSiteWords<TO>;
    // two tile buffers (u_p is formed into the one that does not hold u_{p-1})
    // where both fit, else one, exchanged with the registers between barriers
    constexpr bool kTwo = resident_two_buffers(K);
    const Op &op = a.op;
    const ResidentTiles &T = a.t;
    const int t = (int)threadIdx.x, lane = t & 63, wave = __builtin_amdgcn_readfirstlane(t >> 6);
    const int wg = (int)blockIdx.x, nwg = T.ntx * T.nty;
    const int tx = wg % T.ntx, ty = wg / T.ntx;
    const int x0 = T.x0(tx, op.nx), Tx = T.x0(tx + 1, op.nx) - x0;
    const int y0 = T.y0(ty, op.ny), Ty = T.y0(ty + 1, op.ny) - y0;
    const int W = T.tx + 4, P = W * (T.ty + 4);  // LDS row length and plane (sites)
    double2 *A0 = tile, *A1 = A0 + P + 1;  // site P of a plane takes the writes of rows not formed
    const int tile_words = (kTwo ? 4 : 2) * (P + 1);
    auto at = [&](int i, int j) { return (j + 2) * W + (i + 2); };
    auto get = [&](int s) {
        const double2 u = A0[s], v = A1[s];
        return Sp{u.x, u.y, v.x, v.y};
    };
    auto put = [&](int s, const Sp &v) {
        A0[s] = make_double2(v.r0, v.i0);
        A1[s] = make_double2(v.r1, v.i1);
    };
    // this thread's run of K rows of one column of the tile and its rim
    const int W1 = T.tx + 2;
    const int ci = t % W1 - 1, j0 = (t / W1) * K - 1;
    const int nk = ci <= Tx ? min(K, Ty + 1 - j0) : 0;  // rows of the run that exist (may be <= 0)
    // first site of the run, and the last that exists (rows beyond it compute on
    // its data and are masked, so that the rows need no branches)
    int s0 = nk > 0 ? at(ci, j0) : at(0, 0), s_last = nk > 0 ? s0 + (nk - 1) * W : s0;
    int gx = x0 + ci;  // wrapped column; rows likewise below
    const bool inx = gx >= 0 && gx < op.nx;
    if (!inx) gx = gx < 0 ? gx + op.nx : gx - op.nx;
    const bool ownx = ci >= 0 && ci < Tx;
    uint32_t form = 0, own = 0;  // rows of the run formed here; rows of the tile itself
#pragma unroll
    for (int k = 0; k < K; ++k) {
        const int j = j0 + k, g = y0 + j;
        const bool ring = !ownx && (j < 0 || j >= Ty);  // corners of the rim are received
        const bool dom = (inx || op.bcx) && ((g >= 0 && g < op.ny) || op.bcy);
        if (k < nk && !ring && dom) form |= 1u << k;
        if (k < nk && ownx && j >= 0 && j < Ty) own |= 1u << k;
    }
    int r0 = y0 + j0;  // row of the run's first site (unwrapped)
    auto grow = [&](int k) {
        const int g = r0 + k;
        return g < 0 ? g + op.ny : (g >= op.ny ? g - op.ny : g);
    };
    // index of the run's first row in a plane (rows of the tile itself never
    // wrap, so they are op.nx apart)
    int g0 = (y0 + j0) * op.nx + gx;
    const double xc = op.xmin + gx * op.hx;
    SitePot<K, TERMS> pot;
    if constexpr (TERMS & kTermPot) {
        LaneGeo lg{};
        lg.colw = gx;
        lg.inx = true;
        lg.x = xc;
#pragma unroll
        for (int k = 0; k < K; ++k) {
            __builtin_amdgcn_sched_barrier(0);
            pot.v[k] = 0.0;
            if (form >> k & 1u) pot.v[k] = site_pot_row(op, lg, grow(k), op.ymin + grow(k) * op.hy);
        }
    }
    auto vk = [&](int k) -> double {
        if constexpr (TERMS & kTermPot)
            return pot.v[k];
        else
            return 0.0;
    };
    // border exchange: slot t is published by this thread (psrc: its site in
    // LDS, -1 none), word block rsrc is received by it into site rdst
    const int NS = T.slots();
    int psrc = -1, rdst = -1;
    size_t rsrc = 0;
    {
        // slots: rows 1 and Ty-2, columns 1 and Tx-2, the four corners
        const int bx = T.tx, by = T.ty;
        if (t < bx) {
            if (t < Tx && Ty > 1) psrc = at(t, 1);
        } else if (t < 2 * bx) {
            if (t - bx < Tx && Ty > 1) psrc = at(t - bx, Ty - 2);
        } else if (t < 2 * bx + by) {
            if (t - 2 * bx < Ty && Tx > 1) psrc = at(1, t - 2 * bx);
        } else if (t < 2 * bx + 2 * by) {
            if (t - 2 * bx - by < Ty && Tx > 1) psrc = at(Tx - 2, t - 2 * bx - by);
        } else if (t < NS) {
            const int c = t - 2 * bx - 2 * by;
            psrc = at((c & 1) ? Tx - 1 : 0, (c & 2) ? Ty - 1 : 0);
        }
        // received sites, in the same order: rows -2 and Ty+1, columns -2 and
        // Tx+1, the corners of the rim
        int ri = 0, rj = 0, slot = -1, dx = 0, dy = 0;
        if (t < bx) {
            if (t < Tx) ri = t, rj = -2, dy = -1, slot = bx + t;
        } else if (t < 2 * bx) {
            if (t - bx < Tx) ri = t - bx, rj = Ty + 1, dy = 1, slot = t - bx;
        } else if (t < 2 * bx + by) {
            if (t - 2 * bx < Ty) rj = t - 2 * bx, ri = -2, dx = -1, slot = 2 * bx + by + rj;
        } else if (t < 2 * bx + 2 * by) {
            if (t - 2 * bx - by < Ty) rj = t - 2 * bx - by, ri = Tx + 1, dx = 1, slot = 2 * bx + rj;
        } else if (t < NS) {
            const int c = t - 2 * bx - 2 * by;
            dx = (c & 1) ? 1 : -1;
            dy = (c & 2) ? 1 : -1;
            ri = (c & 1) ? Tx : -1;
            rj = (c & 2) ? Ty : -1;
            slot = 2 * bx + 2 * by + (c ^ 3);  // the neighbour's opposite corner
        }
        if (slot >= 0) {
            int nx_ = tx + dx, ny_ = ty + dy;
            const bool okx = (nx_ >= 0 && nx_ < T.ntx) || op.bcx, oky = (ny_ >= 0 && ny_ < T.nty) || op.bcy;
            nx_ = (nx_ + T.ntx) % T.ntx;
            ny_ = (ny_ + T.nty) % T.nty;
            if (okx && oky) {
                rdst = at(ri, rj);
                rsrc = (size_t)(ny_ * T.ntx + nx_) * NW * NS + slot;
            }
        }
    }
    unsigned long long *const red = a.red, *const halo = a.halo;
    const size_t halo_buf = (size_t)NW * NS * nwg;
    uint32_t epoch = a.epoch;
    // whether this workgroup's waits are over.  The end is read from LDS where few
    // rows a thread leave the registers to the iterations (64^2 959 -> 974 us a call of 20
    // steps with it in registers), and kept in registers else (1024^2 2264 us a call of
    // five steps, from LDS 2294)
    const unsigned long long started = wall_clock64(), deadline = started + a.wait_ticks;
    auto late = [&] {
        if constexpr (kTwo)
            return wall_clock64() > sh.deadline;
        else
            return wall_clock64() > deadline;
    };

    const bool direct = nwg <= kDirect;
    // words of the sums, [group][word][member] with member wg / kLeaders of
    // group wg % kLeaders; the groups' sums (beyond kDirect) in kCopies copies,
    // [copy][word][group], so that fewer workgroups poll the same lines
    const int red_slot = (wg % kLeaders) * 10 * kGroup + wg / kLeaders;
    constexpr size_t red_buf = (size_t)10 * kGroup * kLeaders, red2_buf = (size_t)10 * kLeaders * kCopies;
    unsigned long long *const red2 = red + 2 * red_buf;
    // this workgroup's nv sums into the words of the current epoch (all
    // threads call it with their own parts)
    auto publish_sums = [&](double(&v)[5], auto nvc) {
        constexpr int nv = decltype(nvc)::value;
#pragma unroll
        for (int q = 0; q < nv; ++q) v[q] = lanes_sum(v[q]);
        if (lane == 0)
#pragma unroll
            for (int q = 0; q < nv; ++q) sh.part[wave][q] = v[q];
        __syncthreads();
        if (t < 2 * nv) {
            double s = sh.part[0][t >> 1];
#pragma unroll
            for (int w = 1; w < kRWaves; ++w) s += sh.part[w][t >> 1];
            put_word(red + (epoch & 1u) * red_buf + red_slot + t * kGroup,
                     (uint32_t)((t & 1) ? __double2hiint(s) : __double2loint(s)), epoch);
        }
    };
    // words q = 0 .. 2 nv - 1 of lane's slot (stride apart), once they are of the current
    // epoch, as nv doubles; lanes that are not `on` get zeros
    auto poll_sums = [&](const unsigned long long *p, size_t stride, bool on, auto nvc, double(&v)[5]) {
        constexpr int nv = decltype(nvc)::value;
        unsigned long long w[2 * nv];
#pragma unroll
        for (int q = 0; q < 2 * nv; ++q) w[q] = 0;
        if (on)
            for (;;) {
                bool ok = true;
#pragma unroll
                for (int q = 0; q < 2 * nv; ++q) w[q] = get_word(p + (size_t)q * stride);
#pragma unroll
                for (int q = 0; q < 2 * nv; ++q) ok &= (uint32_t)(w[q] >> 32) == epoch;
                if (ok) break;
                if (late()) {
                    sh.dead = 1;
                    break;
                }
            }
#pragma unroll
        for (int q = 0; q < nv; ++q) v[q] = join(w[2 * q], w[2 * q + 1]);
    };
    // the totals of all workgroups (and, with border, the border sites of the
    // current vector into LDS); false when a wait ran out of time
    auto collect = [&](double(&tot)[5], auto nvc, bool border) -> bool {
        constexpr int nv = decltype(nvc)::value;
        const size_t par = epoch & 1u;
        if (wave == kPollWave) {
            double v[5];
            if (direct) {
                poll_sums(red + par * red_buf + (lane % kLeaders) * 10 * kGroup + lane / kLeaders, kGroup, lane < nwg, nvc,
                          v);
#pragma unroll
                for (int q = 0; q < nv; ++q) v[q] = lanes_sum(v[q]);
            } else {
                if (wg < kLeaders) {  // leads group wg
                    poll_sums(red + par * red_buf + (size_t)wg * 10 * kGroup + lane, kGroup,
                              lane < kGroup && wg + kLeaders * lane < nwg, nvc, v);
                    // (after a wait that ran out of time the sum is not whole and is
                    // not sent, so that the others' waits end too)
                    const bool send = lane < kCopies && sh.dead == 0;
#pragma unroll
                    for (int q = 0; q < nv; ++q) {
                        v[q] = row_sum(v[q]);
                        if (send) {
                            unsigned long long *const o = red2 + par * red2_buf + (lane * 10 + 2 * q) * kLeaders + wg;
                            put_word(o, (uint32_t)__double2loint(v[q]), epoch);
                            put_word(o + kLeaders, (uint32_t)__double2hiint(v[q]), epoch);
                        }
                    }
                }
                poll_sums(red2 + par * red2_buf + (wg % kCopies) * 10 * kLeaders + lane, kLeaders, lane < kLeaders, nvc, v);
#pragma unroll
                for (int q = 0; q < nv; ++q) v[q] = row_sum(v[q]);
            }
            if (lane == 0)
#pragma unroll
                for (int q = 0; q < nv; ++q) sh.tot[q] = v[q];
        } else if (border && rdst >= 0) {
            const unsigned long long *const hp = halo + par * halo_buf + rsrc;
            unsigned long long h[NW];
            for (;;) {
                bool ok = true;
#pragma unroll
                for (int q = 0; q < NW; ++q) h[q] = get_word(hp + (size_t)q * NS);
#pragma unroll
                for (int q = 0; q < NW; ++q) ok &= (uint32_t)(h[q] >> 32) == epoch;
                if (ok) break;
                if (late()) {
                    sh.dead = 1;
                    break;
                }
            }
            Sp v;
            if constexpr (NW == 8)
                v = Sp{join(h[0], h[1]), join(h[2], h[3]), join(h[4], h[5]), join(h[6], h[7])};
            else
                v = Sp{(double)__uint_as_float((uint32_t)h[0]), (double)__uint_as_float((uint32_t)h[1]),
                       (double)__uint_as_float((uint32_t)h[2]), (double)__uint_as_float((uint32_t)h[3])};
            put(rdst, v);
        }
        __syncthreads();
#pragma unroll
        for (int q = 0; q < 5; ++q) tot[q] = q < nv ? sh.tot[q] : 0.0;
        return sh.dead == 0;
    };
    // this tile's share of a border exchange (LDS holds the new vector)
    auto publish_border = [&] {
        if (psrc < 0) return;
        unsigned long long *const hp = halo + (epoch & 1u) * halo_buf + (size_t)wg * NW * NS + t;
        const Sp v = get(psrc);
        const double c[4] = {v.r0, v.i0, v.r1, v.i1};
#pragma unroll
        for (int q = 0; q < 4; ++q) {
            if constexpr (NW == 8) {
                put_word(hp + (size_t)(2 * q) * NS, (uint32_t)__double2loint(c[q]), epoch);
                put_word(hp + (size_t)(2 * q + 1) * NS, (uint32_t)__double2hiint(c[q]), epoch);
            } else {
                put_word(hp + (size_t)q * NS, __float_as_uint((float)c[q]), epoch);
            }
        }
    };
    // the sites of a state within distance two of the tile, into LDS: written
    // by other workgroups (device-coherent loads)
    const uint32_t plane = (uint32_t)op.nx * (uint32_t)op.ny * 16u;
    const uint32_t vec_bytes = (uint32_t)op.nx * (uint32_t)op.ny * (uint32_t)sizeof(Raw<TO>);
    // in a basis vector: byte offset of the run's first row, strides of rows and
    // to the second component
    const uint32_t bsite = sizeof(TO) == 8 || !a.keep ? 16u : 32u;
    const uint32_t bsecond = a.keep ? 16u : (uint32_t)(Tx * Ty) * 16u, brow = (uint32_t)(a.keep ? op.nx : Tx) * bsite;
    uint32_t b0 = a.keep ? (uint32_t)g0 * bsite
                         : (uint32_t)(y0 * op.nx + x0 * Ty) * (uint32_t)sizeof(Raw<TO>) + (uint32_t)(j0 * Tx + ci) * bsite;
    // (paired: the components of a site side by side, else two planes)
    auto load_border = [&](const double2 *psi, bool paired) {
        const uint32_t stride = paired ? 32u : 16u, off1 = paired ? 16u : plane;
        const __amdgpu_buffer_rsrc_t d0 = row_rsrc(reinterpret_cast<const char *>(psi), 2u * plane);
        const int n = 4 * (Tx + Ty) + 4;
        for (int e = t; e < n; e += kRBlock) {
            int i, j;
            if (e < 4 * Tx) {
                const int r = e / Tx;
                i = e - r * Tx;
                j = r < 2 ? r - 2 : Ty + r - 2;
            } else if (e < 4 * (Tx + Ty)) {
                const int q = e - 4 * Tx, r = q / Ty;
                j = q - r * Ty;
                i = r < 2 ? r - 2 : Tx + r - 2;
            } else {
                const int c = e - 4 * (Tx + Ty);
                i = (c & 1) ? Tx : -1;
                j = (c & 2) ? Ty : -1;
            }
            int x = x0 + i, y = y0 + j;
            const bool ok = ((x >= 0 && x < op.nx) || op.bcx) && ((y >= 0 && y < op.ny) || op.bcy);
            x = x < 0 ? x + op.nx : (x >= op.nx ? x - op.nx : x);
            y = y < 0 ? y + op.ny : (y >= op.ny ? y - op.ny : y);
            if (!ok) continue;  // outside a Dirichlet domain: LDS keeps its zero
            const uint32_t off = ((uint32_t)y * (uint32_t)op.nx + (uint32_t)x) * stride;
            const int s = at(i, j);
            A0[s] = ld16<double2, kPolCoherent>(d0, off);
            A1[s] = ld16<double2, kPolCoherent>(d0, off + off1);
        }
    };
    // (A - shift) applied at the rows of the run from LDS: f(k, c, (A - shift) c)
    // per row k, c the row's value
    const double gxq = op.bq, gyq = op.bqy * xc;
    auto sweep_rows = [&](double gxh, double gyh, double shift, auto &&f) {
        const double gy = (TERMS & kTermB) ? gyh - gyq : gyh;
        Sp d = get(s0 - W), c = get(s0);
        auto row = [&](auto kc) {
            constexpr int k = decltype(kc)::value;
            // a few rows' loads in flight at a time (more would spill)
            if constexpr (k % 2 == 0) __builtin_amdgcn_sched_barrier(0);
            const int s = k == 0 ? s0 : min(s0 + k * W, s_last);
            const Sp u = get(s + W);
            double gx = gxh;
            if constexpr (TERMS & kTermB) gx = gxh + gxq * (op.ymin + grow(k) * op.hy);
            f(kc, c, hop(op, c, get(s - 1), get(s + 1), d, u, vk(k), gx, gy, shift));
            d = c;
            c = u;
        };
        unroll_steps(row, std::make_integer_sequence<int, K>{});
    };
    // see opaque()
    auto fresh = [&] {
        opaque(s0);
        opaque(s_last);
        opaque(form);
        opaque(own);
        opaque(r0);
        opaque(g0);
        opaque(b0);
    };
    // u_p = cw (A - sig) u_{p-1} - ca u_{p-1} - cb u_{p-2} from LDS and R into LDS,
    // u_{p-1} into R; store(k, u_p) per row
    auto advance = [&](double gxh, double gyh, double sig, double inv_g1, double ca, double cb, Sp(&R)[K],
                       auto &&store) {
        double2 *const B0 = kTwo ? tile + (A0 == tile ? 2 * (P + 1) : 0) : A0, *const B1 = B0 + P + 1;
        auto keep = [&](int k, const Sp &u, const Sp &old) {
            const int s = form >> k & 1u ? s0 + k * W : P;
            B0[s] = make_double2(u.r0, u.i0);
            B1[s] = make_double2(u.r1, u.i1);
            store(k, u);
            R[k] = old;
        };
        sweep_rows(gxh, gyh, sig, [&](auto kc, const Sp &c, const Sp &w) {
            constexpr int k = decltype(kc)::value;
            const double on = bit_one(form, k), cw = on * inv_g1, cc = on * ca, cu = on * cb;
            Sp u;
            u.r0 = cw * w.r0 - cc * c.r0 - cu * R[k].r0;
            u.i0 = cw * w.i0 - cc * c.i0 - cu * R[k].i0;
            u.r1 = cw * w.r1 - cc * c.r1 - cu * R[k].r1;
            u.i1 = cw * w.i1 - cc * c.i1 - cu * R[k].i1;
            u = stored_value<TO>(u);
            if constexpr (kTwo)
                keep(k, u, c);
            else
                R[k] = u;
        });
        if constexpr (kTwo) {
            A0 = B0;
            A1 = B1;
        } else {
            __syncthreads();
            fresh();
#pragma unroll
            for (int k = 0; k < K; ++k) {
                if (k % 2 == 0) __builtin_amdgcn_sched_barrier(0);
                keep(k, R[k], get(k == 0 ? s0 : min(s0 + k * W, s_last)));
            }
        }
        __syncthreads();
        fresh();
    };

    // zero the tile (sites outside a Dirichlet domain stay zero), then psi
    for (int s = t; s < tile_words; s += kRBlock) tile[s] = make_double2(0.0, 0.0);
    if (t == 0) {
        sh.dead = 0;
        sh.deadline = deadline;
    }
    __syncthreads();
    const double2 *in = EIG ? a.eig.u1 : a.state_in(0);
    const bool paired = EIG && a.eig.p0 > 2;  // u_1 is the start vector, in planes
    {
        const size_t sites = (size_t)op.nx * op.ny, stride = paired ? 2 : 1, off1 = paired ? 1 : sites;
#pragma unroll
        for (int k = 0; k < K; ++k)
            if (own >> k & 1u) {
                const size_t g = (size_t)(g0 + k * op.nx) * stride;
                A0[s0 + k * W] = in[g];
                A1[s0 + k * W] = in[off1 + g];
            }
    }
    load_border(in, paired);
    __syncthreads();

    // ticks per class since the last lap, by the first thread
    unsigned long long clk[5] = {0, 0, 0, 0, 0}, mark = started;
    auto lap = [&](int cls) {
        if (!a.ticks) return;
        const unsigned long long now = wall_clock64();
        clk[cls] += now - mark;
        mark = now;
    };
    bool timeout = false;
    if constexpr (EIG) {
        const int p0 = a.eig.p0, p1 = a.eig.p1;
        Sp R[K];  // u_{p-2} at the run's rows (rim included), then u_{p-1}
#pragma unroll
        for (int k = 0; k < K; ++k) {
            R[k] = sp_zero();
            if (p0 > 2 && (form >> k & 1u)) {
                const double2 *const v = a.eig.u2 + 2 * ((size_t)grow(k) * op.nx + gx);
                R[k] = Sp{v[0].x, v[0].y, v[1].x, v[1].y};
            }
        }
        double g_cur = a.eig.gamma[p0 - 1], g_prev = p0 > 2 ? a.eig.gamma[p0 - 2] : 0.0, al_cur = a.eig.alpha[p0 - 1];
        double scale = sc->scale;
        int p = p0;
        for (; p <= p1; ++p) {
            fresh();
            advance(0.0, 0.0, 0.0, 1.0 / g_cur, al_cur * (1.0 / g_cur), p > 2 ? g_cur / g_prev : 0.0, R,
                    [](int, const Sp &) {});
            ++epoch;
            if (p < p1) publish_border();
            double acc[5] = {0.0, 0.0, 0.0, 0.0, 0.0}, tot[5];
            sweep_rows(0.0, 0.0, 0.0, [&](auto kc, const Sp &c, const Sp &y) {
                constexpr int k = decltype(kc)::value;
                const double w = bit_one(own, k);
                acc[0] += w * sp_norm2(c);
                acc[1] += w * sp_redot(c, y);
                acc[2] += w * sp_redot(c, R[k]);
            });
            publish_sums(acc, IC<3>{});
            if (!collect(tot, IC<3>{}, p < p1)) {
                timeout = true;
                break;
            }
            // (never the last iteration of a step: beta_k is gamma_{k+1} here)
            constexpr int kNoLast = 0x7fffffff;
            const RecurTail o = recur_tail_eval(TailIn{kNoLast, g_cur, 0.0, scale, al_cur}, p, kNoLast, tot);
            if (wg == 0 && t == 0) recur_tail_store(sc, a.eig.alpha, a.eig.gamma, p, o);
            if (o.fail || o.breakdown) break;
            scale = o.scale;
            g_prev = g_cur;
            g_cur = o.gp;
            al_cur = o.al;
        }
        if (p > p1) {  // every workgroup has read its inputs: the buffers may be the same
#pragma unroll
            for (int k = 0; k < K; ++k)
                if (own >> k & 1u) {
                    const size_t g = 2 * (size_t)(g0 + k * op.nx);
                    const Sp u = get(s0 + k * W);
                    a.eig.o1[g] = make_double2(u.r0, u.i0);
                    a.eig.o1[g + 1] = make_double2(u.r1, u.i1);
                    a.eig.o2[g] = make_double2(R[k].r0, R[k].i0);
                    a.eig.o2[g + 1] = make_double2(R[k].r1, R[k].i1);
                }
        }
        if (timeout && t == 0) {  // (any workgroup: its tile of the outputs is missing)
            sc->status = kStatusTimeout;
            sc->kstop = -1;
        }
        return;
    }
    int step = 0;
    for (; step < a.n_steps; ++step) {
        in = a.state_in(step);
        double2 *out = a.state_out(step);
        char *basis = a.basis + (size_t)step * a.basis_step;
        const double *field = a.fields + (ptrdiff_t)step * a.field_stride;
        const double gxh = field[0], gyh = field[1];
        Sp R[K];  // u_{p-2} at the run's rows, then u_p, then u_{p-1}
#pragma unroll
        for (int k = 0; k < K; ++k) R[k] = sp_zero();
        // ---- iteration 1
        double acc[5] = {0.0, 0.0, 0.0, 0.0, 0.0}, tot[5];
        sweep_rows(gxh, gyh, 0.0, [&](auto kc, const Sp &c, const Sp &y) {
            const double w = bit_one(own, decltype(kc)::value);
            acc[0] += w * sp_norm2(c);
            acc[1] += w * sp_redot(c, y);
            acc[2] += w * sp_norm2(y);
        });
        ++epoch;
        publish_sums(acc, IC<3>{});
        if (!collect(tot, IC<3>{}, false)) {
            timeout = true;
            break;
        }
        lap(0);
        if (!isfinite(tot[0]) || !isfinite(tot[1]) || !isfinite(tot[2])) break;  // status 3 below
        // scalars of the recurrence, the same in every thread of the grid
        int keff = a.m;
        double sig = 0.0, scale = 0.0, beta_k = 0.0, g_prev = 0.0, g_cur = 0.0, al_cur = 0.0;
        if (tot[0] == 0.0) {
            keff = 0;
        } else {
            g_cur = sqrt(tot[0]);
            const double al = tot[1] / tot[0];
            sig = al;
            scale = fabs(al);
            beta_k = sqrt(fmax(tot[2] - tot[1] * (tot[1] / tot[0]), 0.0)) / g_cur;
        }
        if (t == 0) {
            sh.al[1] = 0.0;  // alpha'_1 of the shifted operator
            sh.ga[1] = g_cur;
        }
        // ---- iterations 2 .. m
        bool fail = false;
        if (keff > 0)
            for (int p = 2; p <= a.m; ++p) {
                fresh();
                const double inv_g1 = 1.0 / g_cur, ca = al_cur * inv_g1, cb = p > 2 ? g_cur / g_prev : 0.0;
                const __amdgpu_buffer_rsrc_t ub = row_rsrc(basis + (size_t)(p - 2) * a.vstride, vec_bytes);
                // u_p into LDS and (the tile itself) memory, u_{p-1} into the registers
                advance(gxh, gyh, sig, inv_g1, ca, cb, R, [&](int k, const Sp &u) {
                    st_site(ub, own >> k & 1u ? b0 + (uint32_t)k * brow : kOob, bsecond, to_raw<TO>(u));
                });
                const bool last = p == a.m;
                ++epoch;
                if (!last) publish_border();
#pragma unroll
                for (int q = 0; q < 5; ++q) acc[q] = 0.0;
                // the last iteration's two extra sums give beta_m
                bool ok;
                if (last) {
                    sweep_rows(gxh, gyh, sig, [&](auto kc, const Sp &c, const Sp &y) {
                        constexpr int k = decltype(kc)::value;
                        const double w = bit_one(own, k);
                        acc[0] += w * sp_norm2(c);
                        acc[1] += w * sp_redot(c, y);
                        acc[2] += w * sp_redot(c, R[k]);
                        acc[3] += w * sp_norm2(y);
                        acc[4] += w * sp_redot(y, R[k]);
                    });
                    publish_sums(acc, IC<5>{});
                    ok = collect(tot, IC<5>{}, false);
                } else {
                    sweep_rows(gxh, gyh, sig, [&](auto kc, const Sp &c, const Sp &y) {
                        constexpr int k = decltype(kc)::value;
                        const double w = bit_one(own, k);
                        acc[0] += w * sp_norm2(c);
                        acc[1] += w * sp_redot(c, y);
                        acc[2] += w * sp_redot(c, R[k]);
                    });
                    publish_sums(acc, IC<3>{});
                    ok = collect(tot, IC<3>{}, true);
                }
                if (!ok) {
                    timeout = true;
                    break;
                }
                const RecurTail o = recur_tail_eval(TailIn{a.m, g_cur, sig, scale, al_cur}, p, a.m, tot);
                lap(p <= 3 ? 2 : 1);
                if (o.fail) {
                    fail = true;
                    break;
                }
                if (o.breakdown) {
                    keff = p - 1;
                    beta_k = o.beta_k;
                    if (t == 0) sh.ga[p] = o.gp;
                    break;
                }
                scale = o.scale;
                g_prev = g_cur;
                g_cur = o.gp;
                al_cur = o.al;
                if (o.last) beta_k = o.beta_k;
                if (t == 0) {
                    sh.ga[p] = o.gp;
                    sh.al[p] = o.al;
                }
            }
        if (timeout || fail) break;
        __syncthreads();  // the chain is whole; LDS is free for the QR path
        // ---- the small exponential, by wave 0 of every workgroup
        double err = 0.0;
        if (wave == 0 && keff > 0) {
            // inside the kernel where registers allow (a call waits for the
            // basis stores in flight: 512^2 101.6 -> 97.9 us a step), else as a
            // call (1024^2: 503 -> 493 us, its registers would spill)
            if constexpr (kTwo && K > 1)
                resident_exp(sh, keff, sig);
            else
                resident_exp_call(keff, sig);
        }
        __syncthreads();
        if (keff > 0) {
            err = beta_k * sh.cabs;
            if (sh.scratch) {  // the tile was scratch: its outside sites are zero again
                for (int s = t; s < tile_words; s += kRBlock) tile[s] = make_double2(0.0, 0.0);
                __syncthreads();
            }
        }
        lap(3);
        // ---- the recombination of this thread's sites
        double nrm = 0.0;
        {
            fresh();
            const __amdgpu_buffer_rsrc_t i0 = row_rsrc(reinterpret_cast<const char *>(in), plane);
            const __amdgpu_buffer_rsrc_t i1 = row_rsrc(reinterpret_cast<const char *>(in) + plane, plane);
            const double c1r = keff >= 1 ? sh.coef[2] : 0.0, c1i = keff >= 1 ? sh.coef[3] : 0.0;
            const __amdgpu_buffer_rsrc_t o0 = row_rsrc(reinterpret_cast<const char *>(out), plane);
            const __amdgpu_buffer_rsrc_t o1 = row_rsrc(reinterpret_cast<const char *>(out) + plane, plane);
            // kPart rows at a time, two vectors' loads in flight (terms in the
            // order j = 2..k)
            constexpr int kPart = K <= 4 ? K : (K + 1) / 2;
#pragma unroll
            for (int kb = 0; kb < K; kb += kPart) {
                uint32_t site[kPart], boff[kPart];
                Sp c[kPart];
#pragma unroll
                for (int q = 0; q < kPart; ++q) {
                    const int k = kb + q;
                    const bool on = k < K && (own >> k & 1u);
                    site[q] = (uint32_t)(g0 + k * op.nx);
                    boff[q] = on ? b0 + (uint32_t)k * brow : kOob;
                    const uint32_t off = on ? site[q] * 16u : kOob;
                    const double2 p0 = ld16<double2>(i0, off), p1 = ld16<double2>(i1, off);
                    c[q].r0 = c1r * p0.x - c1i * p0.y;
                    c[q].i0 = c1r * p0.y + c1i * p0.x;
                    c[q].r1 = c1r * p1.x - c1i * p1.y;
                    c[q].i1 = c1r * p1.y + c1i * p1.x;
                }
                auto load = [&](int j, auto pol, Raw<TO>(&v)[kPart]) {
                    const __amdgpu_buffer_rsrc_t ub = row_rsrc(basis + (size_t)(j - 2) * a.vstride, vec_bytes);
#pragma unroll
                    for (int q = 0; q < kPart; ++q)
                        v[q] = ld_site_at<TO, decltype(pol)::value>(ub, boff[q], bsecond);
                };
                auto add = [&](int j, const Raw<TO>(&v)[kPart]) {
                    const double cr = sh.coef[2 * j], cim = sh.coef[2 * j + 1];
#pragma unroll
                    for (int q = 0; q < kPart; ++q) {
                        const Sp w = to_sp(v[q]);
                        c[q].r0 += cr * w.r0 - cim * w.i0;
                        c[q].i0 += cr * w.i0 + cim * w.r0;
                        c[q].r1 += cr * w.r1 - cim * w.i1;
                        c[q].i1 += cr * w.i1 + cim * w.r1;
                    }
                };
                auto terms = [&](auto pol) {
                    int j = 2;
                    for (; j + 1 <= keff; j += 2) {
                        Raw<TO> v0[kPart], v1[kPart];
                        load(j, pol, v0);
                        load(j + 1, pol, v1);
                        add(j, v0);
                        add(j + 1, v1);
                    }
                    if (j <= keff) {
                        Raw<TO> v[kPart];
                        load(j, pol, v);
                        add(j, v);
                    }
                };
                // a basis beyond the last-level cache is read with the
                // streaming hint (1024^2, 20 vectors: 174 -> 148 us), one inside
                // it is not (512^2, 12 vectors: 20 -> 25 us)
                if (a.stream_basis)
                    terms(IC<kPolStream>{});
                else
                    terms(IC<kPolDefault>{});
                // the new state: into LDS for the next step, and written through
                // to memory (neighbours read its border from there)
#pragma unroll
                for (int q = 0; q < kPart; ++q) {
                    const int k = kb + q;
                    if (k < K && (own >> k & 1u)) {
                        const uint32_t off = site[q] * 16u;
                        st16<double2, kPolCoherent>(o0, off, make_double2(c[q].r0, c[q].i0));
                        st16<double2, kPolCoherent>(o1, off, make_double2(c[q].r1, c[q].i1));
                        put(s0 + k * W, c[q]);
                        nrm += sp_norm2(c[q]);
                    }
                }
            }
        }
        // the stores are at the coherence point before this workgroup's sum is
        asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
        acc[0] = nrm;
        acc[1] = acc[2] = acc[3] = acc[4] = 0.0;
        ++epoch;
        publish_sums(acc, IC<1>{});
        if (!collect(tot, IC<1>{}, false)) {
            timeout = true;
            break;
        }
        if (wg == 0 && t == 0) {
            StepStat *st = a.stats + step;
            st->keff = keff;
            st->err_est = err;
            st->round_bound = 0.0;
            st->norm2 = tot[0];
        }
        // what later kernels read of this step: the chain (storage bound), and
        // for the adjoint the scalars and both arrays
        if (wg == 0 && wave == 1) {
            if (a.chain) {
                double *ch = a.chain + (size_t)step * kChainLen;
                if (lane == 0) ch[0] = (double)keff;
                if (lane < keff) {
                    ch[1 + lane] = sh.al[lane + 1];
                    ch[1 + kMaxM + lane] = sh.ga[lane + 1];
                }
            }
            if (a.keep) {
                char *kp = a.keep + (size_t)step * a.keep_step;
                Scalars *ks = reinterpret_cast<Scalars *>(kp);
                double *ka = reinterpret_cast<double *>(kp + a.keep_alpha), *kg = reinterpret_cast<double *>(kp + a.keep_gamma);
                if (lane == 0) {
                    ks->keff = keff;
                    ks->sigma = sig;
                    ks->status = 0;
                }
                for (int q = lane + 1; q <= a.m; q += 64) {
                    ka[q] = q <= keff ? sh.al[q] : 0.0;
                    kg[q] = q <= keff ? sh.ga[q] : 0.0;
                }
            }
        }
        if (!isfinite(tot[0])) break;
        if (wg == 0 && t == 0) sc->steps_done += 1;
        if (step + 1 < a.n_steps) load_border(out, false);
        __syncthreads();
        lap(4);
    }
    if (wg == 0 && t == 0) {
        if (step < a.n_steps) {  // left early: a non-finite sum, or a wait without an answer
            sc->status = timeout ? kStatusTimeout : 3;
            sc->kstop = -1;
        }
        if (a.ticks)
            for (int q = 0; q < 5; ++q) a.ticks[q] += clk[q];
    }
}

// The complex64 storage bound of steps 0 .. gridDim.x - 1 of a resident launch
// (one wave each), off the chain of its iterations.  first: completed steps of
// the call before the launch.
__global__ __launch_bounds__(64) void k_resident_bounds(const double *chain, const Scalars *sc, StepStat *stats,
                                                        int first, double reps, double rabs)
{
    __shared__ double lds[kBoundLds];
    const int step = (int)blockIdx.x, lane = (int)threadIdx.x;
    if (first + step >= sc->steps_done) return;
    const double *ch = chain + (size_t)step * kChainLen;
    const int k = (int)ch[0];
    if (k <= 0) return;
    const double d = lane < k ? ch[1 + lane] : 0.0, e = lane + 1 < k ? ch[1 + kMaxM + lane + 1] : 0.0;
    double em = from_left(e);
    if (lane == 0) em = 0.0;
    const double rb = storage_bound(d, e, em, k, lane, ch[1 + kMaxM], reps, rabs, lds);
    if (lane == 0) stats[step].round_bound = rb;
}

using ResidentKernel = void (*)(ResidentArgs);

template <class TO, int TERMS, bool EIG>
ResidentKernel pick_rows(int k)
{
    switch (k) {
    case 1: return k_resident<TO, 1, TERMS, EIG>;
    case 2: return k_resident<TO, 2, TERMS, EIG>;
    case 3: return k_resident<TO, 3, TERMS, EIG>;
    case 4: return k_resident<TO, 4, TERMS, EIG>;
    case 6: return k_resident<TO, 6, TERMS, EIG>;
    case 8: return k_resident<TO, 8, TERMS, EIG>;
    default: return k_resident<TO, 10, TERMS, EIG>;
    }
}

}  // namespace

// Epochs base + 1 .. base + n for one launch: never 0 (cleared buffers), and used
// again only after the 32-bit count has gone round, which no words outlast: every
// call clears them, and a launch writes each of them every few epochs.
static uint32_t reserve_epochs(uint32_t n)
{
    static std::atomic<uint32_t> last{0};
    uint32_t base;
    do
        base = last.fetch_add(n, std::memory_order_relaxed);
    while (base + n < base);
    return base;
}

static hipError_t launch_tiles(const ResidentArgs &a, int epochs, ResidentKernel kernel, hipStream_t st)
{
    const size_t lds = a.t.lds_bytes();
    hipError_t e = hipFuncSetAttribute(reinterpret_cast<const void *>(kernel), hipFuncAttributeMaxDynamicSharedMemorySize,
                                       (int)lds);
    if (e != hipSuccess) return e;
    ResidentArgs args = a;
    args.epoch = reserve_epochs((uint32_t)epochs);
    void *params[] = {&args};
    return hipLaunchCooperativeKernel(reinterpret_cast<const void *>(kernel), dim3(a.t.ntx * a.t.nty), dim3(kRBlock),
                                      params, (unsigned)lds, st);
}

hipError_t launch_resident(const ResidentArgs &a, bool mixed, hipStream_t st)
{
    constexpr int kAll = kTermPot | kTermB;
    const bool terms = op_terms(a.op) != 0;
    const int k = a.t.rows;
    // an epoch per iteration and one for the norm of the new state
    return launch_tiles(a, a.n_steps * (a.m + 1),
                        mixed ? (terms ? pick_rows<float2, kAll, false>(k) : pick_rows<float2, 0, false>(k))
                              : (terms ? pick_rows<double2, kAll, false>(k) : pick_rows<double2, 0, false>(k)),
                        st);
}

hipError_t launch_resident_eigen(const ResidentArgs &a, hipStream_t st)
{
    const int k = a.t.rows;
    return launch_tiles(a, a.eig.p1 - a.eig.p0 + 1,
                        op_terms(a.op) != 0 ? pick_rows<double2, kTermPot | kTermB, true>(k) : pick_rows<double2, 0, true>(k),
                        st);
}

void launch_resident_bounds(const double *chain, const Scalars *sc, StepStat *stats, int first, int n, double reps,
                            double rabs, hipStream_t st)
{
    hipLaunchKernelGGL(k_resident_bounds, dim3(n), dim3(64), 0, st, chain, sc, stats, first, reps, rabs);
}

}  // namespace dl
