// Device kernels of the hybrid symplectic hot path for gfx950 (MI355X).
//
// Paper: Mercury-Opal, arXiv 2601.19654.  Sec. 3.1 gives the five per-step
// blocks (force, Hamiltonian, drift, encounter check) and Sec. 3.2 the data
// kept on the device; Sec. 2.1.1 the coordinates (democratic heliocentric) and
// the Hill-radius based critical radius.  The kernels here are a new MI355X
// design, not a translation of the paper's OpenACC loops:
//   * state lives in HBM as FP64 structure-of-arrays planes for the whole run;
//   * pair kernels hold R targets per lane in VGPRs and stream sources through
//     LDS tiles read as wave-wide broadcasts; sources are split into chunks so a
//     single system fills all 256 CUs, and the chunk partials are summed in a
//     fixed order (bit-reproducible runs);
//   * O(N) phases run over blocks that never straddle two systems, with
//     per-system sums formed from per-block partials in a fixed order;
//   * no atomics touch floating-point data; the encounter list uses one
//     integer atomic per wave and is sorted afterwards.
#include "nb_internal.h"

#include <algorithm>
#include <cstddef>
#include <cstdint>
#include <float.h>
#include <math.h>
#include <type_traits>

namespace nb {

// ----------------------------------------------------------------------------
// small helpers
// ----------------------------------------------------------------------------

// Error-free sum (Knuth two-sum) accumulated into a (hi, lo) pair.
struct dd {
    double hi, lo;
};
__device__ __forceinline__ void dd_add(dd &a, double b)
{
    double s = a.hi + b;
    double bp = s - a.hi;
    double e = (a.hi - (s - bp)) + (b - bp);
    a.hi = s;
    a.lo += e;
}
__device__ __forceinline__ void dd_add(dd &a, const dd &b)
{
    dd_add(a, b.hi);
    a.lo += b.lo;
}

// 1/sqrt(x) in FP64 to the last bits (diagnostics): the hardware estimate y0
// (relative error at most 2^-24) corrected through (1-e)^(-1/2) = 1 + e/2 +
// 3e^2/8 + O(e^3), e = 1 - x y0^2: the dropped 5e^3/16 is below 2^-70, so the
// result carries the rounding of e and of the last operation only, which a
// further Newton step would carry again.
__device__ __forceinline__ double rsqrt64_acc(double x)
{
    const double y = __builtin_amdgcn_rsq(x);
    const double e = fma(-x * y, y, 1.0);
    return fma(y * e, fma(0.375, e, 0.5), y);
}

// Largest value over the wave, returned in a scalar register (every lane active).
__device__ __forceinline__ double wave_max(double v)
{
    for (int o = 32; o > 0; o >>= 1)
        v = fmax(v, __shfl_xor(v, o));
    const long long b = __double_as_longlong(v);
    const int lo = __builtin_amdgcn_readfirstlane((int)(b & 0xffffffffLL));
    const int hi = __builtin_amdgcn_readfirstlane((int)(b >> 32));
    return __longlong_as_double(((long long)hi << 32) | (unsigned int)lo);
}

// Deterministic block-wide sum of W doubles per thread (kBlock threads, fixed
// order): each wave's 64 values by an xor-shuffle butterfly (both lanes of a
// pair add the same two values, so every lane ends with the same bits), then
// the wave sums in wave order.  Every thread returns the block's sums.  (Threads
// past kBlock, which help elsewhere in a launch, add nothing.)
template <int W>
__device__ __forceinline__ void block_sum(double (&v)[W], double *sh)
{
    constexpr int NW = kBlock / 64;
    const int lane = threadIdx.x & 63, wv = threadIdx.x >> 6;
    // (a product is rounded before it is added, whichever launch sums it)
#pragma unroll
    for (int w = 0; w < W; ++w)
        __asm__("" : "+v"(v[w]));
#pragma unroll
    for (int w = 0; w < W; ++w)
        for (int o = 32; o > 0; o >>= 1)
            v[w] += __shfl_xor(v[w], o);
    if (lane == 0 && wv < NW) {
#pragma unroll
        for (int w = 0; w < W; ++w)
            sh[w * NW + wv] = v[w];
    }
    __syncthreads();
#pragma unroll
    for (int w = 0; w < W; ++w) {
        double t = sh[w * NW];
        for (int q = 1; q < NW; ++q)
            t += sh[w * NW + q];
        v[w] = t;
    }
    __syncthreads();
}

// Sum of the first W columns of the per-block partials of one system, in block order.
template <int W>
__device__ __forceinline__ void system_sum(const double *__restrict__ part, int stride, int first,
                                           int count, double (&out)[W], double *sh)
{
#pragma unroll
    for (int w = 0; w < W; ++w)
        out[w] = 0.0;
    for (int b = threadIdx.x; b < count && threadIdx.x < kBlock; b += kBlock)
#pragma unroll
        for (int w = 0; w < W; ++w)
            out[w] += part[(size_t)(first + b) * stride + w];
    block_sum<W>(out, sh);
}

// Changeover weight w = K/r^3 - (dK/dr)/r^2 for a pair at squared distance r2
// with pair critical radius rc (inner edge `inner` rc).  K = 0 below the inner
// edge, 1 beyond rc and y^2/(2y^2-2y+1) in between, y = (r - inner rc)/((1-inner) rc).
__device__ __forceinline__ double changeover_w_inl(double r2, double rc, double inner)
{
    if (!(r2 > 0.0))
        return 0.0;
    double r = sqrt(r2);
    if (r >= rc)
        return 1.0 / (r2 * r);
    double r_in = inner * rc;
    if (r <= r_in)
        return 0.0;
    double width = rc - r_in;
    double y = (r - r_in) / width;
    double q = 2.0 * y * (y - 1.0) + 1.0;
    double K = y * y / q;
    double dK = 2.0 * y * (1.0 - y) / (q * q * width);
    return (K / r - dK) / r2;
}

// Out of line: the pair loops call it only for the rare pairs inside rc.
__device__ __noinline__ double changeover_w(double r2, double rc, double inner)
{
    return changeover_w_inl(r2, rc, inner);
}

// K itself (diagnostics).
__device__ __forceinline__ double changeover_K(double r, double rc, double inner)
{
    if (r >= rc)
        return 1.0;
    double r_in = inner * rc;
    if (r <= r_in)
        return 0.0;
    double y = (r - r_in) / (rc - r_in);
    return y * y / (2.0 * y * (y - 1.0) + 1.0);
}

// ----------------------------------------------------------------------------
// fills, validation, transforms
// ----------------------------------------------------------------------------
__global__ void k_fill_i32(int *p, int n, int value)
{
    int i = blockIdx.x * blockDim.x + threadIdx.x;
    if (i < n)
        p[i] = value;
}

// flag bit 1: a non-finite value, a negative mass or m0 <= 0; bit 2: a small
// body (index >= off[s] + nbig[s]) with a nonzero mass.
__global__ void k_validate(int ntot, int nsys, const double *__restrict__ m0,
                           const double *__restrict__ m, const double *__restrict__ x,
                           const double *__restrict__ v, const int *__restrict__ sys_of,
                           const int *__restrict__ off, const int *__restrict__ nbig, int *flag,
                           unsigned long long *__restrict__ scale)
{
    int i = blockIdx.x * blockDim.x + threadIdx.x;
    int bad = 0;
    if (i < nsys)
        scale[i] = 0ull;
    if (i < ntot) {
        double mi = m[i];
        bad = (!isfinite(mi) || mi < 0.0) ? 1 : 0;
        for (int c = 0; c < 3; ++c)
            bad |= (!isfinite(x[(size_t)c * ntot + i]) || !isfinite(v[(size_t)c * ntot + i])) ? 1 : 0;
        const int s = sys_of[i];
        if (i - off[s] >= nbig[s] && mi != 0.0)
            bad |= 2;
    }
    if (i < nsys)
        bad |= (!(m0[i] > 0.0) || !isfinite(m0[i])) ? 1 : 0;
    if (bad)
        atomicOr(flag, bad);
}

// Per-block partial of sum m v (columns 0-2) and sum m (column 3).
__global__ void k_partial_mv(const RBlk *__restrict__ rblk, const double *__restrict__ m,
                             const double *__restrict__ vx, const double *__restrict__ vy,
                             const double *__restrict__ vz, double *__restrict__ part)
{
    __shared__ double sh[4 * kBlock];
    RBlk b = rblk[blockIdx.x];
    int i = b.start + threadIdx.x;
    double v[4] = {0.0, 0.0, 0.0, 0.0};
    if (i < b.end) {
        double mi = m[i];
        v[0] = mi * vx[i];
        v[1] = mi * vy[i];
        v[2] = mi * vz[i];
        v[3] = mi;
    }
    block_sum<4>(v, sh);
    if (threadIdx.x == 0)
        for (int w = 0; w < 4; ++w)
            part[(size_t)blockIdx.x * 4 + w] = v[w];
}

// Blocks of a system whose bodies set its unit of length (enc_inv_scale): a wave of each
// adds the sum of its bodies' exponents, shifted by kScaleShift, and their number.
constexpr int kScaleBlocks = 16, kScaleShift = 20;
static_assert(kScaleBlocks * kBlock < 1 << kScaleShift, "the number stays below the sum");

// Heliocentric -> DH: Q = x, V = v - sum m v / (m0 + sum m); or a plain copy.
__global__ void k_to_dh(const RBlk *__restrict__ rblk, const int *__restrict__ rb_first,
                        const int *__restrict__ rb_count, const double *__restrict__ m0,
                        const double *__restrict__ part, int ntot, const double *__restrict__ x,
                        const double *__restrict__ v, int helio, double *qx, double *qy,
                        double *qz, double *vx, double *vy, double *vz,
                        unsigned long long *__restrict__ scale)
{
    // scale: also the binary exponents of |Q|^2 of every system's bodies, summed over
    // up to kScaleBlocks of its blocks (cleared before; whole numbers, so that the sum
    // does not depend on the order): enc_inv_scale
    __shared__ double sh[4 * kBlock];
    RBlk b = rblk[blockIdx.x];
    double c[3] = {0.0, 0.0, 0.0};
    int e = 0, cnt = 0;
    if (helio) {
        double P[4];
        system_sum<4>(part, 4, rb_first[b.sys], rb_count[b.sys], P, sh);
        double M = m0[b.sys] + P[3];
        c[0] = P[0] / M;
        c[1] = P[1] / M;
        c[2] = P[2] / M;
    }
    int i = b.start + threadIdx.x;
    if (i < b.end) {
        const double x0 = x[i], x1 = x[(size_t)ntot + i], x2 = x[(size_t)2 * ntot + i];
        qx[i] = x0;
        qy[i] = x1;
        qz[i] = x2;
        vx[i] = v[i] - c[0];
        vy[i] = v[(size_t)ntot + i] - c[1];
        vz[i] = v[(size_t)2 * ntot + i] - c[2];
        const double r2 = x0 * x0 + x1 * x1 + x2 * x2;
        if (r2 > 0.0 && isfinite(r2)) {
            e = ilogb(r2);
            cnt = 1;
        }
    }
    const int nb = rb_count[b.sys], stride = (nb + kScaleBlocks - 1) / kScaleBlocks;
    if (((int)blockIdx.x - rb_first[b.sys]) % stride)
        return;
    for (int o = 32; o > 0; o >>= 1) {
        e += __shfl_xor(e, o);
        cnt += __shfl_xor(cnt, o);
    }
    if ((threadIdx.x & 63) == 0 && cnt)
        atomicAdd(&scale[b.sys], ((unsigned long long)(long long)e << kScaleShift) + (unsigned long long)cnt);
}

// DH -> heliocentric (v = V + P/m0) or DH copy, into plane-major x, v.
__global__ void k_from_dh(const RBlk *__restrict__ rblk, const int *__restrict__ rb_first,
                          const int *__restrict__ rb_count, const double *__restrict__ m0,
                          const double *__restrict__ part, int ntot, int helio,
                          const double *__restrict__ qx, const double *__restrict__ qy,
                          const double *__restrict__ qz, const double *__restrict__ vx,
                          const double *__restrict__ vy, const double *__restrict__ vz, double *x,
                          double *v)
{
    __shared__ double sh[4 * kBlock];
    RBlk b = rblk[blockIdx.x];
    double c[3] = {0.0, 0.0, 0.0};
    if (helio) {
        double P[3];
        system_sum<3>(part, 4, rb_first[b.sys], rb_count[b.sys], P, sh);
        double mm = m0[b.sys];
        c[0] = P[0] / mm;
        c[1] = P[1] / mm;
        c[2] = P[2] / mm;
    }
    int i = b.start + threadIdx.x;
    if (i < b.end) {
        x[i] = qx[i];
        x[(size_t)ntot + i] = qy[i];
        x[(size_t)2 * ntot + i] = qz[i];
        v[i] = vx[i] + c[0];
        v[(size_t)ntot + i] = vy[i] + c[1];
        v[(size_t)2 * ntot + i] = vz[i] + c[2];
    }
}

// ----------------------------------------------------------------------------
// Kick (Hamiltonian block loop 1), optionally with gas drag, and the partial
// sums of m V after it (the following stellar drift needs them).
// ----------------------------------------------------------------------------
struct DragP {
    double G, sigma0, h, cd, rho_p;
};

// Quadratic gas drag on one body (parity unpinned by the paper: Sec. 2.1 names
// aerodynamic drag, its disk model is elsewhere).  a = -k |u| u, u = v_helio -
// v_gas, k = 3 C_D rho_g / (8 rho_p s), s = (3 m/(4 pi rho_p))^(1/3),
// rho_g = Sigma0/R / (sqrt(2 pi) h R) exp(-z^2/(2 (h R)^2)),
// v_gas = sqrt(1 - 3 h^2) sqrt(G m0 / R) phi_hat, R cylindrical.
__device__ void drag_accel(const DragP &p, double m0, double mi, double x, double y, double z,
                           double ux, double uy, double uz, double &ax, double &ay, double &az)
{
    const double kPi = 3.141592653589793238462643;
    double R2 = x * x + y * y;
    double R = sqrt(R2);
    double H = p.h * R;
    double rho = p.sigma0 / R / (sqrt(2.0 * kPi) * H) * exp(-z * z / (2.0 * H * H));
    double vk = sqrt(p.G * m0 / R) * sqrt(1.0 - 3.0 * p.h * p.h);
    double gx = -vk * y / R, gy = vk * x / R;
    double wx = ux - gx, wy = uy - gy, wz = uz;
    double wm = sqrt(wx * wx + wy * wy + wz * wz);
    double s = cbrt(3.0 * mi / (4.0 * kPi * p.rho_p));
    double k = (mi > 0.0 && p.sigma0 > 0.0) ? 3.0 * p.cd * rho / (8.0 * p.rho_p * s) : 0.0;
    ax = -k * wm * wx;
    ay = -k * wm * wy;
    az = -k * wm * wz;
}

// One slice of a body's split partials: slots [k0, k1) of position i in order,
// eight loads of each component in flight.
template <typename P>
__device__ __forceinline__ void sum_slots(const P *__restrict__ fpart, int ntot, int maxs, int i,
                                          int k0, int k1, double &s0, double &s1, double &s2)
{
    const P *px = fpart + i, *py = px + (size_t)maxs * ntot, *pz = py + (size_t)maxs * ntot;
    int k = k0;
    for (; k + 8 <= k1; k += 8) {
        P ux[8], uy[8], uz[8];
#pragma unroll
        for (int u = 0; u < 8; ++u) {
            ux[u] = px[(size_t)(k + u) * ntot];
            uy[u] = py[(size_t)(k + u) * ntot];
            uz[u] = pz[(size_t)(k + u) * ntot];
        }
#pragma unroll
        for (int u = 0; u < 8; ++u) {
            s0 += (double)ux[u];
            s1 += (double)uy[u];
            s2 += (double)uz[u];
        }
    }
    for (; k < k1; ++k) {
        s0 += (double)px[(size_t)k * ntot];
        s1 += (double)py[(size_t)k * ntot];
        s2 += (double)pz[(size_t)k * ntot];
    }
}

// The sum of body i's partials times G by NSL threads per body, thread group g of
// kBlock threads slice g, in the arithmetic and order of k_force_finalize with as many
// slices; complete in group 0.  gs: 3 kBlock (NSL - 1) doubles.  Every thread calls.
template <int NSL, typename P>
__device__ __forceinline__ void slot_accel(const P *__restrict__ fpart, int ntot, int maxs, int i,
                                           bool in, int ns, double G, double *gs, double &s0,
                                           double &s1, double &s2)
{
    const int g = threadIdx.x / kBlock, t = threadIdx.x % kBlock;
    s0 = s1 = s2 = 0.0;
    if (in)
        sum_slots(fpart, ntot, maxs, i, g * ns / NSL, (g + 1) * ns / NSL, s0, s1, s2);
    if constexpr (NSL > 1) {
        if (g > 0) {
            double *o = gs + (size_t)(g - 1) * 3 * kBlock;
            o[t] = s0;
            o[kBlock + t] = s1;
            o[2 * kBlock + t] = s2;
        }
        __syncthreads();
        if (g == 0)
            for (int q = 0; q < NSL - 1; ++q) {
                const double *o = gs + (size_t)q * 3 * kBlock;
                s0 += o[t];
                s1 += o[kBlock + t];
                s2 += o[2 * kBlock + t];
            }
    }
    s0 *= G;
    s1 *= G;
    s2 *= G;
}

// A value the compiler cannot relate to the one it had: the expressions before and
// after are contracted to fused operations apart.
__device__ __forceinline__ void opaque(double &a)
{
    __asm__("" : "+v"(a));
}

// V += h a.  NSL > 0: a from the body's force partials first (slot_accel; stored), by
// kBlock NSL threads.  part_in: the per-block sums of m V, for gas drag (nullptr: none),
// whose kick depends on V; part_out: the sums after the kick.  Launch-bound: a step of
// 1001 bodies with drag was nine launches of 3-9 us in a chain, of which the sum of the
// partials and both sums of m V before a kick (the drift and the kick before leave them)
// are gone: 45 -> 38 us.
template <typename FP, int NSL>
__global__ __launch_bounds__(kBlock * (NSL ? NSL : 1)) void k_kick(
    const RBlk *__restrict__ rblk, double h, const double *__restrict__ m, double *__restrict__ ax,
    double *__restrict__ ay, double *__restrict__ az, double *vx, double *vy, double *vz,
    double *__restrict__ part_out, const double *__restrict__ part_in,
    const int *__restrict__ rb_first, const int *__restrict__ rb_count,
    const double *__restrict__ m0, const double *__restrict__ qx, const double *__restrict__ qy,
    const double *__restrict__ qz, DragP dp, const FP *__restrict__ fpart, int ntot, int maxs,
    const int *__restrict__ nsplit, double G)
{
    __shared__ double sh[4 * kBlock];
    __shared__ double gs[NSL > 1 ? (NSL - 1) * 3 * kBlock : 1];
    const RBlk b = rblk[blockIdx.x];
    const int i = b.start + (int)(threadIdx.x % kBlock);
    const bool on = i < b.end && threadIdx.x < kBlock;
    double s0 = 0.0, s1 = 0.0, s2 = 0.0;
    if constexpr (NSL > 0)
        slot_accel<NSL>(fpart, ntot, maxs, i, i < b.end, nsplit[b.sys], G, gs, s0, s1, s2);
    double P[3] = {0.0, 0.0, 0.0};
    double mm = 1.0;
    if (part_in) {
        system_sum<3>(part_in, 4, rb_first[b.sys], rb_count[b.sys], P, sh);
        mm = m0[b.sys];
    }
    double v[3] = {0.0, 0.0, 0.0};
    if (on) {
        double mi = m[i];
        if constexpr (NSL > 0) {
            ax[i] = s0;
            ay[i] = s1;
            az[i] = s2;
        } else {
            s0 = ax[i];
            s1 = ay[i];
            s2 = az[i];
        }
        double a0 = s0, a1 = s1, a2 = s2;
        double u0 = vx[i], u1 = vy[i], u2 = vz[i];
        if (part_in) {
            double d0, d1, d2;
            drag_accel(dp, mm, mi, qx[i], qy[i], qz[i], u0 + P[0] / mm, u1 + P[1] / mm,
                       u2 + P[2] / mm, d0, d1, d2);
            a0 += d0;
            a1 += d1;
            a2 += d2;
        }
        // fused multiply-add, as in k_force_finalize: two kicks there equal two here
        u0 = fma(h, a0, u0);
        u1 = fma(h, a1, u1);
        u2 = fma(h, a2, u2);
        vx[i] = u0;
        vy[i] = u1;
        vz[i] = u2;
        v[0] = mi * u0;
        v[1] = mi * u1;
        v[2] = mi * u2;
    }
    if (part_out) {
        block_sum<3>(v, sh);
        if (threadIdx.x == 0) {
            part_out[(size_t)blockIdx.x * 4 + 0] = v[0];
            part_out[(size_t)blockIdx.x * 4 + 1] = v[1];
            part_out[(size_t)blockIdx.x * 4 + 2] = v[2];
            part_out[(size_t)blockIdx.x * 4 + 3] = 0.0;
        }
    }
}

// ----------------------------------------------------------------------------
// Stellar drift Q += h P/m0 (Hamiltonian block loops 2-3), optionally followed
// by the critical radius rc = n_hill |Q| (m/(3 m0))^(1/3) (Sec. 2.1.1) and the
// FP32 hi/lo source records of the FP32C force.
// ----------------------------------------------------------------------------
// Per-system sums of the first three columns of the per-block partials (one
// workgroup per system, the same order as an inline system_sum), for systems with
// so many blocks that every block summing them again would read the partials
// quadratically often.
__global__ void k_sys_total(const int *__restrict__ rb_first, const int *__restrict__ rb_count,
                            const double *__restrict__ part, double *__restrict__ tot)
{
    __shared__ double sh[3 * kBlock];
    double P[3];
    system_sum<3>(part, 4, rb_first[blockIdx.x], rb_count[blockIdx.x], P, sh);
    if (threadIdx.x < 3)
        tot[(size_t)blockIdx.x * 4 + threadIdx.x] = P[threadIdx.x];
}

__global__ void k_sun_drift(const RBlk *__restrict__ rblk, const int *__restrict__ rb_first,
                            const int *__restrict__ rb_count, const double *__restrict__ m0,
                            const double *__restrict__ part, double h, double *qx, double *qy,
                            double *qz, int rcrit, const double *__restrict__ m, double n_hill,
                            double *__restrict__ rc, float4 *__restrict__ pk,
                            double *__restrict__ tile_rc2, double *__restrict__ copy_to,
                            const double *__restrict__ ptot, const int *__restrict__ rord,
                            float4 *__restrict__ rtb)
{
    // copy_to: this block's entry of `part` is copied there (nothing else reads
    // that array during the launch)
    if (copy_to && threadIdx.x < 4)
        copy_to[(size_t)blockIdx.x * 4 + threadIdx.x] = part[(size_t)blockIdx.x * 4 + threadIdx.x];
    __shared__ double sh[3 * kBlock];
    double rc2 = 0.0;
    RBlk b = rblk[blockIdx.x];
    // rord: the block's positions of the radial order (their bodies from
    // rord), each wave one tile of 64, whose bounds it writes to rtb
    const int pos = b.start + threadIdx.x;
    const bool on = pos < b.end;
    const int i = rord && on ? rord[pos] : pos;
    float tr = INFINITY, tR = 0.0f, tl = 0.0f, tc = 0.0f;
    // the body's position, loaded while the system's momentum is summed
    const double x0 = on ? qx[i] : 0.0, y0 = on ? qy[i] : 0.0, z0 = on ? qz[i] : 0.0;
    const double mi = on && rcrit ? m[i] : 0.0;
    double c[3] = {0.0, 0.0, 0.0};
    double mm = m0[b.sys];
    if (h != 0.0) {
        // the system's momentum: precomputed per system (ptot) or summed here
        double P[3];
        if (ptot) {
            P[0] = ptot[(size_t)b.sys * 4];
            P[1] = ptot[(size_t)b.sys * 4 + 1];
            P[2] = ptot[(size_t)b.sys * 4 + 2];
        } else {
            system_sum<3>(part, 4, rb_first[b.sys], rb_count[b.sys], P, sh);
        }
        c[0] = h * P[0] / mm;
        c[1] = h * P[1] / mm;
        c[2] = h * P[2] / mm;
    }
    if (on) {
        double x = x0 + c[0], y = y0 + c[1], z = z0 + c[2];
        // with h = 0 (critical radii only) Q is left as it is: the positions
        // may then be a caller's read-only input
        if (h != 0.0) {
            qx[i] = x;
            qy[i] = y;
            qz[i] = z;
        }
        if (rcrit) {
            double r = sqrt(x * x + y * y + z * z);
            double rci = n_hill * r * cbrt(mi / (3.0 * mm));
            rc[i] = rci;
            rc2 = rci * rci;
            if (pk) {
                float hx = (float)x, hy = (float)y, hz = (float)z;
                float lx = (float)(x - (double)hx), ly = (float)(y - (double)hy),
                      lz = (float)(z - (double)hz);
                // squared radius widened by 2^-9 so the FP32 zone test is a superset of
                // the FP64 one; never below 2^-80, so that pairs closer than 2^-40 (where
                // the FP32 weight r^-3 would overflow: massless bodies have rc = 0, and
                // 0 * inf is NaN) and coincident bodies take the FP64 path
                float r2 = (float)(rci * rci * (1.0 + 0x1p-9));
                r2 = fmaxf(r2, 0x1p-80f);
                pk[2 * (size_t)i] = make_float4(hx, hy, hz, (float)mi);
                pk[2 * (size_t)i + 1] = make_float4(lx, ly, lz, r2);
                if (rtb) {
                    // |xh| and |xl| in FP64 (products of floats are exact),
                    // widened by 2^-22 before rounding to nearest so that the
                    // floats bound them from the safe side
                    const double rh = sqrt((double)hx * hx + (double)hy * hy + (double)hz * hz);
                    const double rl = sqrt((double)lx * lx + (double)ly * ly + (double)lz * lz);
                    tr = (float)(rh * (1.0 - 0x1p-22));
                    tR = (float)(rh * (1.0 + 0x1p-22));
                    tl = (float)(rl * (1.0 + 0x1p-22));
                    tc = r2;
                }
            }
        }
    }
    if (rtb) {
        for (int o = 32; o > 0; o >>= 1) {
            tr = fminf(tr, __shfl_xor(tr, o));
            tR = fmaxf(tR, __shfl_xor(tR, o));
            tl = fmaxf(tl, __shfl_xor(tl, o));
            tc = fmaxf(tc, __shfl_xor(tc, o));
        }
        const int w = threadIdx.x >> 6;
        if ((threadIdx.x & 63) == 0 && b.start + 64 * w < b.end)
            rtb[b.rt0 + w] = make_float4(tr, tR, tl, tc);
    }
    if (rcrit) {
        // largest rc^2 of this block's bodies: the zone threshold of the ordered and
        // few-source force kernels (over the radial order, which only the symmetric
        // kernel uses, the bodies of the block's positions)
        for (int o = 32; o > 0; o >>= 1)
            rc2 = fmax(rc2, __shfl_xor(rc2, o));
        if ((threadIdx.x & 63) == 0)
            sh[threadIdx.x >> 6] = rc2;
        __syncthreads();
        if (threadIdx.x == 0) {
            double r = sh[0];
            for (int w = 1; w < kBlock / 64; ++w)
                r = fmax(r, sh[w]);
            tile_rc2[blockIdx.x] = r;
        }
    }
}

// ----------------------------------------------------------------------------
// Kepler drift (Sec. 2.1: WHFAST-derived drift; Sec. 3.1: one body per thread
// with a failure flag, positions and velocities copied first).  Universal
// variables: s solves r0 s + eta0 G2(s) + zeta0 G3(s) = dt with
// G_k(s) = s^k c_k(beta s^2), beta = 2 mu/r0 - v^2, zeta0 = mu - beta r0.
// ----------------------------------------------------------------------------
__host__ __device__ constexpr double inv_fact(int k)
{
    double f = 1.0;
    for (int i = 2; i <= k; ++i)
        f *= (double)i;
    return 1.0 / f;
}

// c_k(z) = sum_n (-z)^n/(2n+k)! by a fixed-length Horner polynomial (|z| <= 1).
template <int K>
__device__ __forceinline__ double stumpff_series(double mz)
{
    double p = inv_fact(2 * 11 + K);
#pragma unroll
    for (int n = 10; n >= 0; --n)
        p = fma(p, mz, inv_fact(2 * n + K));
    return p;
}

__device__ __forceinline__ void gfuncs(double beta, double s, double &G1, double &G2, double &G3)
{
    double z = beta * s * s;
    double c1, c2, c3;
    if (fabs(z) <= 1.0) {
        c1 = stumpff_series<1>(-z);
        c2 = stumpff_series<2>(-z);
        c3 = stumpff_series<3>(-z);
    } else if (z > 0.0) {
        double x = sqrt(z), sx, cx;
        sincos(x, &sx, &cx);
        c1 = sx / x;
        c2 = (1.0 - cx) / z;
        c3 = (1.0 - c1) / z;
    } else {
        double x = sqrt(-z);
        c1 = sinh(x) / x;
        c2 = (1.0 - cosh(x)) / z;
        c3 = (1.0 - c1) / z;
    }
    G1 = s * c1;
    G2 = s * s * c2;
    G3 = s * s * s * c3;
}

// Returns 0 on success; on failure the body is left unchanged.
__device__ int kepler_drift(double mu, double dt, double &x, double &y, double &z, double &u,
                            double &v, double &w)
{
    if (dt == 0.0)
        return 0;
    double r0 = sqrt(x * x + y * y + z * z);
    double v2 = u * u + v * v + w * w;
    double eta0 = x * u + y * v + z * w;
    double beta = 2.0 * mu / r0 - v2;
    double zeta0 = mu - beta * r0;
    if (!(r0 > 0.0) || !isfinite(r0 + v2))
        return 1;

    const double tol = 2.0 * DBL_EPSILON;   // 4 u
    // second-order starting value of s
    double s = dt / r0;
    double corr = 1.0 - 0.5 * eta0 * dt / (r0 * r0);
    if (corr > 0.5 && corr < 2.0)
        s *= corr;
    double lo = dt > 0.0 ? 0.0 : -INFINITY;
    double hi = dt > 0.0 ? INFINITY : 0.0;
    double G1, G2, G3;
    bool ok = false;
    for (int it = 0; it < 100; ++it) {
        gfuncs(beta, s, G1, G2, G3);
        double F = r0 * s + eta0 * G2 + zeta0 * G3 - dt;
        double dF = r0 + eta0 * G1 + zeta0 * G2;
        if (F == 0.0) {
            ok = true;
            break;
        }
        if (F < 0.0)
            lo = s;
        else
            hi = s;
        double sn = s - F / dF;
        if (!(sn > lo && sn < hi)) {
            if (isfinite(lo) && isfinite(hi))
                sn = 0.5 * (lo + hi);
            else if (isfinite(lo))
                sn = lo > 0.0 ? 2.0 * lo : fabs(dt / r0);
            else
                sn = hi < 0.0 ? 2.0 * hi : -fabs(dt / r0);
        }
        double ds = sn - s;
        s = sn;
        if (fabs(ds) <= tol * fabs(s) || (hi - lo) <= tol * fabs(s)) {
            ok = true;
            break;
        }
    }
    if (!ok)
        return 1;
    gfuncs(beta, s, G1, G2, G3);
    double r = r0 + eta0 * G1 + zeta0 * G2;
    double fm1 = -mu * G2 / r0;
    double g = dt - mu * G3;
    double fd = -mu * G1 / (r * r0);
    double gdm1 = -mu * G2 / r;
    double nx = x + (fm1 * x + g * u), ny = y + (fm1 * y + g * v), nz = z + (fm1 * z + g * w);
    double nu = u + (fd * x + gdm1 * u), nv = v + (fd * y + gdm1 * v), nw = w + (fd * z + gdm1 * w);
    if (!isfinite(nx + ny + nz + nu + nv + nw))
        return 1;
    x = nx;
    y = ny;
    z = nz;
    u = nu;
    v = nv;
    w = nw;
    return 0;
}

// What the encounter filters know of a pair.  The exact test's f(s) is the cubic of the
// squared distance with slopes 2 dt dQ0.dV0 and 2 dt dQ1.dV1.  With the relative midpoint M,
// chord c and endpoint velocity deviations e0 = dt dV0 - c, e1 = dt dV1 - c (half their
// difference d = dt (dV0 - dV1)/2, their mean p), the cubic reproduces the straight
// chord x(s) = M + (s - 1/2) c exactly and adds 2 h10 dQ0.e0 + 2 h11 dQ1.e1, h10 =
// s(1-s)^2, h11 = -s^2 (1-s):
//   f = |x|^2 + 2 sg d.x + 2 sg p.((1-2s) M - c/2),   sg = s(1-s), t = |1-2s| = sqrt(1 - 4 sg).
// With D = |M|, a = |c|/2 and X = D - a t <= |x|, where X >= sg |d|,
//   f >= X^2 - 2 sg |d| X - 2 sg |p| (t D + a).                                         (1)
// E = |d| + kEncP |p|; of two bodies, |d_j - d_i| + kEncP (|p_i| + |p_j|) is no less.
// (A) A pair with D > 2a + 3/4 E + rc stays outside rc: D = X + a t in (1), with al = 2 sg
// <= 1/2, be = al t <= 1/(3 sqrt 3), ga = al (1 + t^2) and X = u + rc, u >= (2-t) a + 3/4 |d| +
// 3/4 kEncP |p|, gives f - rc^2 >= X (X - al |d| - be |p|) - rc^2 - ga a |p| >=
// a |p| ((2-t)(3/2 kEncP - be) - ga) > 0, the last bracket at least 0.1.
// (B) Where D > a and g = (D-a)^2 - (D+a) E/2 > 0, f >= g: (1) minus g is at least
// a(1-t)(2D - a(1+t)) - (al - kEncP/2) a |p| (as kEncP/2 > be and al <= 1/2), and g > 0 bounds
// |p| by 2 (D-a)^2 / (kEncP (D+a)): with x = D/a >= 1 it is not negative where
// (1-t)(2x-1-t)(x+1) >= ((1-t^2)/kEncP - 1)(x-1)^2, which holds for every t in [0, 1].  (For
// g < 0 it can fail: p along c enters with sg a |p|, more than E/4 covers.)
// On an orbit d is the fall toward the star, about -dt^2/2 times the acceleration,
// which neighbours share, and p is of third order in dt: E is small where the largest
// |e| of either body is not.
constexpr double kEncP = 0.385;

__device__ __forceinline__ double norm3(double x, double y, double z)
{
    return sqrt(x * x + y * y + z * z);
}

__device__ __forceinline__ double norm1(double x, double y, double z)
{
    return fabs(x) + fabs(y) + fabs(z);
}

// A bound of sqrt(v) from above, within 2^-19 of it (the hardware estimate of
// 1/sqrt is good to 2^-24).
__device__ __forceinline__ double sqrt_up(double v)
{
    return v > 0.0 ? v * __builtin_amdgcn_rsq(v) * (1.0 + 0x1p-20) : v;
}

// A value to FP16 (over FP32: the split's low part takes what either rounding left).
__device__ __forceinline__ _Float16 to_half(double v)
{
    return (_Float16)(float)v;
}

// d and a bound of kEncP |p| of a step.
__device__ __forceinline__ double enc_deviation(double dt, const double (&v0)[3], const double (&v1)[3],
                                                const double (&c)[3], double (&d)[3])
{
    double p2 = 0.0;
#pragma unroll
    for (int k = 0; k < 3; ++k) {
        d[k] = 0.5 * dt * (v0[k] - v1[k]);
        const double p = 0.5 * dt * (v0[k] + v1[k]) - c[k];
        p2 += p * p;
    }
    return kEncP * sqrt_up(p2);
}

// The matrix-core filter of the direct encounter check (k_enc_direct): a pair can
// only be flagged when D <= C + 3/4 |d_j - d_i| + s_i + s_j with D, C the distances of
// the two chord midpoints M and chords c, and s = 3/4 kEncP |p| + rc.  As (x + y + z)^2
// <= 2 x^2 + 4 y^2 + 4 z^2, and with d' = sqrt(9/8) d, s' = sqrt 2 s, then
//   D^2 - 2 C^2 - 2 |d'_j - d'_i|^2 - 2 (s'_i + s'_j)^2 = al_i + al_j + sum_k g_k u_ik u_jk
// is not positive, with u = (M, c, d', s'), g = (-2 -2 -2 4 4 4 4 4 4 -4) and
// al = |M|^2 - 2|c|^2 - 2|d'|^2 - 2 s'^2: a product of two matrices.  M and c (in units
// of the system's scale L, a power of two) are split into two FP16 values, 22 bits,
// of whose four products the one of the two low values is left out; d' is rounded to
// one FP16 value, its rounding (2^-11 |d'| and 2^-25 a component, 1/sqrt 2 of it in
// units of s; with the sum of |d'|'s components) added to s; s' is rounded up to one.  al, from the rounded d' and s' and
// reduced by the body's share of the error bound, is split into two.  The 27 products
// of a pair are exact in the matrix core's FP32 sum.
// Bound of the error, with nn = |M|^2 + 2|c|^2 + 2|d'|^2 + 2 s'^2 (the terms' magnitudes
// add up to at most 2 (nn_i + nn_j)): splitting 2^-21 (nn_i + nn_j), the products left
// out 2^-22 (nn_i + nn_j), summing 32 terms (measured: 2^-21 of their magnitudes) 2^-20
// (nn_i + nn_j), FP16 values below 2^-14 in steps of 2^-24: 2^-22 (sqrt nn_i + sqrt
// nn_j) and 2^-31.  The shares below are at least four times that.
// The shares grow with L, so L is a typical distance, not the largest (enc_inv_scale),
// and a midpoint outside the ball of kEncBall L is moved to the ball's nearest point:
// the projection onto a convex set brings no two points further apart, so D only
// shrinks, and a body far out stays a candidate only of those near its direction at the
// ball's edge (and of those its own s reaches).  One body at 65000 AU beside 9990 at 1-3 AU: 602 us a check
// with the largest distance as L, 16 us now (13 us without it).  A body whose chord,
// deviation or s is outside 8 L (or not finite) gets a record that makes a candidate of
// each of its pairs.
constexpr double kEncK1 = 0x1p-17, kEncK2 = 0x1p-20, kEncK3 = 0x1p-28;
constexpr double kEncMax = 8.0;                 // largest component of u / L
constexpr double kEncBall = 7.5;                // largest |M| / L
constexpr double kEncAlUnit = 64.0;             // al is stored times this ...
constexpr double kEncAlOut = -60000.0;          // ... and this for a candidate of every pair
typedef _Float16 v8h __attribute__((ext_vector_type(8)));
typedef float v4f __attribute__((ext_vector_type(4)));

// 1/L of a system from the exponents of |Q|^2 of its bodies at the upload (k_to_dh): L
// about the power of two above the geometric mean of |Q| (1 when there is none).
__device__ __forceinline__ double enc_inv_scale(unsigned long long v)
{
    const int cnt = (int)(v & ((1ull << kScaleShift) - 1ull));
    if (cnt == 0)
        return 1.0;
    const float sum = (float)(int)((long long)v >> kScaleShift);
    const int e = (int)floorf(sum * __builtin_amdgcn_rcpf((float)cnt));      // the mean, rounded down
    return ldexp(1.0, -((e >> 1) + 1));
}

// The record of a body: (M_hi, c_hi, s', al_hi), (M_lo, c_lo, al_lo, 0), (d', 1/unit,
// 1/unit, al_hi, al_lo, 0).
constexpr int kEncRec = 3;
__device__ __forceinline__ void enc_record(double mx, double my, double mz, double cx, double cy,
                                           double cz, const double (&d)[3], double s, double inv_l,
                                           v8h *out)
{
    double u[6] = {mx * inv_l, my * inv_l, mz * inv_l, cx * inv_l, cy * inv_l, cz * inv_l};
    v8h A, B, D;
    const double R2 = u[0] * u[0] + u[1] * u[1] + u[2] * u[2];
    bool in = R2 <= DBL_MAX;
    if (R2 > kEncBall * kEncBall) {
        const double f = kEncBall / sqrt(R2);
        u[0] *= f;
        u[1] *= f;
        u[2] *= f;
    }
#pragma unroll
    for (int k = 0; k < 6; ++k) {
        in = in && fabs(u[k]) <= kEncMax;
        A[k] = to_half(u[k]);
        B[k] = to_half(u[k] - (double)A[k]);
    }
    double dd = 0.0, d2 = 0.0;
#pragma unroll
    for (int k = 0; k < 8; ++k) {
        const double w = k < 3 ? 0x1.0f876ccdf6cd9p+0 * inv_l * d[k < 3 ? k : 0] : 0.0;   // sqrt(9/8)
        in = in && fabs(w) <= kEncMax;
        D[k] = to_half(w);
        dd += fabs(w);
        d2 += (double)D[k] * (double)D[k];
    }
    const double sp = 0x1.6a09e667f3bcdp+0 * (s * inv_l) + 0x1.002p-11 * dd + 0x1p-23;   // sqrt 2
    in = in && sp <= 0.5 * kEncMax;
    A[6] = to_half(sp * (1.0 + 0x1p-10));
    const double M2 = u[0] * u[0] + u[1] * u[1] + u[2] * u[2];
    const double C2 = 2.0 * (u[3] * u[3] + u[4] * u[4] + u[5] * u[5] + d2 + (double)A[6] * (double)A[6]);
    const double nn = M2 + C2;
    const double al = (M2 - C2 - (kEncK1 * nn + kEncK2 * sqrt_up(nn) + kEncK3)) * kEncAlUnit;
    A[7] = to_half(al);
    B[6] = to_half(al - (double)A[7]);
    B[7] = (_Float16)0.0f;
    if (!in) {
        A = B = D = v8h{};
        A[7] = (_Float16)(float)kEncAlOut;
    }
    D[3] = D[4] = (_Float16)(float)(1.0 / kEncAlUnit);
    D[5] = A[7];
    D[6] = B[6];
    out[0] = A;
    out[1] = B;
    out[2] = D;
}

// Snapshot, drift, failure flags and counters, the encounter check's records,
// and the partial sums of m V after the drift (for the second stellar drift).
// The check clears its own list and flags, since it may run beside the next drift.
// NSL > 0: before the drift the sum of the body's force partials (FP: their type) by
// NSL threads per body and two kicks V += kick_h a, in the arithmetic and order of
// k_force_finalize with as many slices; the workgroup has kBlock NSL threads, and
// those past kBlock only sum.  It saves a launch (and the 96 bytes per body that
// the finalize and the drift pass through memory) inside a run.
// A step with the finalize apart / folded in: 300 bodies 29.8 / 27.5 us, 16 systems
// of 500 bodies 35.7 / 30.7, 3001 bodies (47 slots) 37.1 / 37.5, 5000 bodies (79
// slots) 47 / 50: hence kFinDriftSlots.
template <typename FP, int NSL, bool ISO>
__global__ __launch_bounds__(kBlock * (NSL ? NSL : 1)) void k_drift(const RBlk *__restrict__ rblk, const double *__restrict__ m0, double G,
                        double dt, const double *__restrict__ m, double *qx, double *qy,
                        double *qz, double *vx, double *vy, double *vz, double *__restrict__ q0x,
                        double *__restrict__ q0y, double *__restrict__ q0z,
                        double *__restrict__ v0x, double *__restrict__ v0y,
                        double *__restrict__ v0z, int *__restrict__ kflag,
                        DevStats *stats, double *__restrict__ part_out,
                        const double *__restrict__ rc, double *__restrict__ lnr_part,
                        double *__restrict__ q1x, double *__restrict__ q1y,
                        double *__restrict__ q1z, double *__restrict__ v1x,
                        double *__restrict__ v1y, double *__restrict__ v1z,
                        double *__restrict__ rc1, const double *__restrict__ part_in,
                        double sun_h, const int *__restrict__ rb_first,
                        const int *__restrict__ rb_count, const double *__restrict__ ptot,
                        v8h *__restrict__ eq, const unsigned long long *__restrict__ scale,
                        int *__restrict__ nce, const FP *__restrict__ fpart, int ntot, int maxs,
                        const int *__restrict__ nsplit, double kick_h)
{
    constexpr int NS1 = NSL > 1 ? NSL - 1 : 1;
    __shared__ double gs[NSL > 1 ? NS1 * 3 * kBlock : 1];
    // for the encounter check: eq (records of the direct check) or the ln R range
    // of the midpoints (sorted check).  nce: the count of the check that will read this set
    // of drift outputs, from zero.
    if (nce && blockIdx.x == 0 && threadIdx.x == 0)
        *nce = 0;
    __shared__ double sh[3 * kBlock];
    double lnr_lo = INFINITY, lnr_hi = -INFINITY;
    RBlk b = rblk[blockIdx.x];
    const int t = NSL > 1 ? threadIdx.x % kBlock : threadIdx.x;
    int i = b.start + t;
    const bool on = i < b.end && threadIdx.x < kBlock;
    // the body's state, loaded while the system's momentum is summed
    const double xs = on ? qx[i] : 0.0, ys = on ? qy[i] : 0.0, zs = on ? qz[i] : 0.0;
    double us = on ? vx[i] : 0.0, vs = on ? vy[i] : 0.0, ws = on ? vz[i] : 0.0;
    if constexpr (NSL > 0) {
        double s0, s1, s2;
        slot_accel<NSL>(fpart, ntot, maxs, i, i < b.end, nsplit[b.sys], G, gs, s0, s1, s2);
        us = fma(kick_h, s0, us);
        vs = fma(kick_h, s1, vs);
        ws = fma(kick_h, s2, ws);
        us = fma(kick_h, s0, us);
        vs = fma(kick_h, s1, vs);
        ws = fma(kick_h, s2, ws);
    }
    const double rci = on ? rc[i] : 0.0, mi = on ? m[i] : 0.0;
    double mu = G * m0[b.sys];
    bool fail = false;
    double pv[3] = {0.0, 0.0, 0.0};
    // the sun drift S(sun_h) that precedes the drift, from the per-block sums of
    // m V in part_in (same arithmetic as k_sun_drift)
    double sd[3] = {0.0, 0.0, 0.0};
    if (sun_h != 0.0) {
        // the system's momentum: precomputed per system (ptot) or summed here
        double P[3];
        if (ptot) {
            P[0] = ptot[(size_t)b.sys * 4];
            P[1] = ptot[(size_t)b.sys * 4 + 1];
            P[2] = ptot[(size_t)b.sys * 4 + 2];
        } else {
            system_sum<3>(part_in, 4, rb_first[b.sys], rb_count[b.sys], P, sh);
        }
        const double mm = m0[b.sys];
        sd[0] = sun_h * P[0] / mm;
        sd[1] = sun_h * P[1] / mm;
        sd[2] = sun_h * P[2] / mm;
    }
    if (on) {
        double x = xs + sd[0], y = ys + sd[1], z = zs + sd[2];
        double u = us, v = vs, w = ws;
        const double sx = x, sy = y, sz = z;
        q0x[i] = x;
        q0y[i] = y;
        q0z[i] = z;
        v0x[i] = u;
        v0y[i] = v;
        v0z[i] = w;
        // ISO (all but the full method, whose steps use one form of this launch): the solver
        // apart from the code around it, so that the forms give the same bits
        if constexpr (ISO)
            for (double *a : {&x, &y, &z, &u, &v, &w, &mu})
                opaque(*a);
        fail = kepler_drift(mu, dt, x, y, z, u, v, w) != 0;
        if constexpr (ISO)
            for (double *a : {&x, &y, &z, &u, &v, &w})
                opaque(*a);
        // Encounter data of this body over the step: chord c = Q1 - Q0 and midpoint M
        {
            const double c[3] = {x - sx, y - sy, z - sz};
            const double mx = sx + 0.5 * c[0], my = sy + 0.5 * c[1], mz = sz + 0.5 * c[2];
            if (eq) {
                const double e0[3] = {us, vs, ws}, e1[3] = {u, v, w};
                double d[3];
                const double p = enc_deviation(dt, e0, e1, c, d);
                // 2^-45 (|M| + |c|): the rounding of midpoint, chord and deviations
                const double s = 0.75 * p + rci + 0x1p-45 * (norm1(mx, my, mz) + norm1(c[0], c[1], c[2]));
                enc_record(mx, my, mz, c[0], c[1], c[2], d, s, enc_inv_scale(scale[b.sys]),
                           eq + kEncRec * (size_t)i);
            } else {
                const double lnr = log(fmax(sqrt(mx * mx + my * my), 1e-300));
                lnr_lo = lnr;
                lnr_hi = lnr;
            }
        }
        qx[i] = x;
        qy[i] = y;
        qz[i] = z;
        vx[i] = u;
        vy[i] = v;
        vz[i] = w;
        q1x[i] = x;
        q1y[i] = y;
        q1z[i] = z;
        v1x[i] = u;
        v1y[i] = v;
        v1z[i] = w;
        rc1[i] = rci;
        kflag[i] = fail ? 1 : 0;
        pv[0] = mi * u;
        pv[1] = mi * v;
        pv[2] = mi * w;
    }
    unsigned long long mask = __ballot(fail);
    if (mask && (threadIdx.x & 63) == (unsigned)(__ffsll((long long)mask) - 1)) {
        atomicAdd((unsigned long long *)&stats->kepler_fail, (unsigned long long)__popcll(mask));
        atomicAdd(&stats->cur_kfail, (int)__popcll(mask));
    }
    if (lnr_part) {
        // range of ln R over the block (the sorted encounter check bins by it)
        for (int o = 32; o > 0; o >>= 1) {
            lnr_lo = fmin(lnr_lo, __shfl_xor(lnr_lo, o));
            lnr_hi = fmax(lnr_hi, __shfl_xor(lnr_hi, o));
        }
        if ((threadIdx.x & 63) == 0 && threadIdx.x < kBlock) {
            sh[threadIdx.x >> 6] = lnr_lo;
            sh[kBlock / 64 + (threadIdx.x >> 6)] = lnr_hi;
        }
        __syncthreads();
        if (threadIdx.x == 0) {
            double lo = sh[0], hi = sh[kBlock / 64];
            for (int w = 1; w < kBlock / 64; ++w) {
                lo = fmin(lo, sh[w]);
                hi = fmax(hi, sh[kBlock / 64 + w]);
            }
            lnr_part[2 * (size_t)blockIdx.x] = lo;
            lnr_part[2 * (size_t)blockIdx.x + 1] = hi;
        }
        __syncthreads();
    }
    block_sum<3>(pv, sh);
    if (threadIdx.x == 0) {
        part_out[(size_t)blockIdx.x * 4 + 0] = pv[0];
        part_out[(size_t)blockIdx.x * 4 + 1] = pv[1];
        part_out[(size_t)blockIdx.x * 4 + 2] = pv[2];
        part_out[(size_t)blockIdx.x * 4 + 3] = 0.0;
    }
}

// ----------------------------------------------------------------------------
// Interaction force (Sec. 3.1 force block, loop 2): per target i the sum over
// sources j != i of m_j w(r_ij) (Q_j - Q_i); G is applied in the finalize pass.
// Pairs at or beyond rc_ij take the Newtonian term; pairs inside rc_ij take
// the exact changeover weight in a divergent branch.  The branch test is one
// compare per pair against a per-lane, per-tile threshold max(rc_i^2, max_j
// rc_j^2); the branch itself applies the exact pair test.
// ----------------------------------------------------------------------------

// m y^3 with y = 1/sqrt(r2): the hardware estimate y0 (worst relative error
// 2^-24.2 on gfx950) corrected through (1 - e)^(-3/2) = 1 + 3e/2 + O(e^2),
// e = 1 - r2 y0^2; the dropped 15e^2/8 term is below 2.1e-14.  m15 = 1.5 m.
__device__ __forceinline__ double m_rinv3(double m, double m15, double r2)
{
    double y0 = __builtin_amdgcn_rsq(r2);
    double y2 = y0 * y0;
    double e = fma(-r2, y2, 1.0);
    return (y0 * y2) * fma(m15, e, m);
}

// Work item layout shared by both force kernels: the block's 64*R targets are
// the same for its kBlock/64 waves; each source tile of kBlock bodies is staged
// in LDS and wave w takes its sources [64w, 64w+64).  The waves' sums are added
// in wave order through LDS at the end, so results do not depend on timing.
constexpr int kWaves = kBlock / 64;

template <int R>
__global__ __launch_bounds__(kBlock) void k_force64(const FWork *__restrict__ work,
                                                    const double *__restrict__ qx,
                                                    const double *__restrict__ qy,
                                                    const double *__restrict__ qz,
                                                    const double *__restrict__ m,
                                                    const double *__restrict__ rc,
                                                    const double *__restrict__ tile_rc2,
                                                    double *__restrict__ fpart, int ntot, int maxs,
                                                    double inner, DevStats *stats)
{
    __shared__ double4 sj[kBlock];
    __shared__ double2 sx[kBlock];                 // {1.5 m, rc}
    __shared__ double red[kWaves - 1][3 * R][64];
    const FWork wk = work[blockIdx.x];
    const int t = threadIdx.x, lane = t & 63, wv = t >> 6;
    double xi[R], yi[R], zi[R], rci[R], r2i[R], ax[R], ay[R], az[R];
    int near = 0;
#pragma unroll
    for (int k = 0; k < R; ++k) {
        int li = lane + 64 * k;
        int i = wk.i0 + (li < wk.ni ? li : 0);
        xi[k] = qx[i];
        yi[k] = qy[i];
        zi[k] = qz[i];
        rci[k] = rc[i];
        r2i[k] = fmax(rci[k] * rci[k], DBL_MIN);
        ax[k] = ay[k] = az[k] = 0.0;
    }
    const int jend = wk.j0 + wk.nj;
    int tile = wk.rb0;
    for (int jt = wk.j0; jt < jend; jt += kBlock, ++tile) {
        const int cnt = min(kBlock, jend - jt);
        __syncthreads();
        if (t < cnt) {
            int j = jt + t;
            double mj = m[j];
            sj[t] = make_double4(qx[j], qy[j], qz[j], mj);
            sx[t] = make_double2(1.5 * mj, rc[j]);
        }
        const double tmax = tile_rc2[tile];
        double thr[R];
#pragma unroll
        for (int k = 0; k < R; ++k)
            thr[k] = fmax(r2i[k], tmax);
        __syncthreads();
        // the waves take the tile's sources in turn (wave w: w, w + 4, ...), so a
        // short or ragged source range still splits evenly over the 4 waves
#pragma unroll 2
        for (int jj = wv; jj < cnt; jj += kWaves) {
            const double4 J = sj[jj];
            const double m15 = sx[jj].x;
#pragma unroll
            for (int k = 0; k < R; ++k) {
                double dx = J.x - xi[k], dy = J.y - yi[k], dz = J.z - zi[k];
                double r2 = fma(dz, dz, fma(dy, dy, dx * dx));
                double s = m_rinv3(J.w, m15, r2);
                if (r2 < thr[k]) {
                    double rcj = sx[jj].y;
                    if (r2 < fmax(r2i[k], fmax(rcj * rcj, DBL_MIN))) {
                        s = J.w * changeover_w(r2, fmax(rci[k], rcj), inner);
                        ++near;
                    }
                }
                ax[k] = fma(s, dx, ax[k]);
                ay[k] = fma(s, dy, ay[k]);
                az[k] = fma(s, dz, az[k]);
            }
        }
    }
    if (wv > 0) {
#pragma unroll
        for (int k = 0; k < R; ++k) {
            red[wv - 1][3 * k + 0][lane] = ax[k];
            red[wv - 1][3 * k + 1][lane] = ay[k];
            red[wv - 1][3 * k + 2][lane] = az[k];
        }
    }
    __syncthreads();
    if (wv == 0) {
#pragma unroll
        for (int k = 0; k < R; ++k) {
            for (int w = 0; w < kWaves - 1; ++w) {
                ax[k] += red[w][3 * k + 0][lane];
                ay[k] += red[w][3 * k + 1][lane];
                az[k] += red[w][3 * k + 2][lane];
            }
            int li = lane + 64 * k;
            if (li < wk.ni) {
                int i = wk.i0 + li;
                fpart[((size_t)0 * maxs + wk.slot) * ntot + i] = ax[k];
                fpart[((size_t)1 * maxs + wk.slot) * ntot + i] = ay[k];
                fpart[((size_t)2 * maxs + wk.slot) * ntot + i] = az[k];
            }
        }
    }
    // pairs evaluated in the changeover zone (self pairs included), one atomic per wave
    for (int o = 32; o > 0; o >>= 1)
        near += __shfl_xor(near, o);
    if (lane == 0 && near)
        atomicAdd((unsigned long long *)&stats->near_pairs, (unsigned long long)near);
}

// FP32C: pair terms in FP32 from hi/lo split positions (the difference of two
// hi parts is exact for nearby bodies, the lo parts restore the rest), summed
// in FP32 over runs of kMerge sources and merged by two-sum into a per-target
// (hi, lo) accumulator.  Pairs whose FP32 distance falls inside a widened
// critical radius are evaluated in FP64 from the FP64 state instead.
constexpr int kMerge = 32;

__device__ __forceinline__ void two_sum_f(float &hi, float &lo, float t)
{
    float s = hi + t;
    float bp = s - hi;
    float e = (hi - (s - bp)) + (t - bp);
    hi = s;
    lo += e;
}

template <int R>
__global__ __launch_bounds__(kBlock) void k_force32c(const FWork *__restrict__ work,
                                                     const float4 *__restrict__ pk,
                                                     const double *__restrict__ qx,
                                                     const double *__restrict__ qy,
                                                     const double *__restrict__ qz,
                                                     const double *__restrict__ m,
                                                     const double *__restrict__ rc,
                                                     const double *__restrict__ tile_rc2,
                                                     float *__restrict__ fpart, int ntot,
                                                     int maxs, double inner, DevStats *stats)
{
    __shared__ float4 sa[kBlock];
    __shared__ float4 sb[kBlock];
    __shared__ double red[kWaves - 1][3 * R][64];
    const FWork wk = work[blockIdx.x];
    const int t = threadIdx.x, lane = t & 63, wv = t >> 6;
    float xh[R], yh[R], zh[R], xl[R], yl[R], zl[R], r2i[R];
    float hx[R], hy[R], hz[R], lx[R], ly[R], lz[R], tx[R], ty[R], tz[R];
    double nx[R], ny[R], nz[R];
    int ii[R];
    int near = 0;
#pragma unroll
    for (int k = 0; k < R; ++k) {
        int li = lane + 64 * k;
        int i = wk.i0 + (li < wk.ni ? li : 0);
        ii[k] = i;
        float4 A = pk[2 * (size_t)i], B = pk[2 * (size_t)i + 1];
        xh[k] = A.x; yh[k] = A.y; zh[k] = A.z;
        xl[k] = B.x; yl[k] = B.y; zl[k] = B.z;
        r2i[k] = B.w;
        hx[k] = hy[k] = hz[k] = lx[k] = ly[k] = lz[k] = tx[k] = ty[k] = tz[k] = 0.0f;
        nx[k] = ny[k] = nz[k] = 0.0;
    }
    const int jend = wk.j0 + wk.nj;
    int tile = wk.rb0;
    for (int jt = wk.j0; jt < jend; jt += kBlock, ++tile) {
        const int cnt = min(kBlock, jend - jt);
        __syncthreads();
        if (t < cnt) {
            sa[t] = pk[2 * (size_t)(jt + t)];
            sb[t] = pk[2 * (size_t)(jt + t) + 1];
        }
        // widened like the per-body FP32 radii so the FP32 test stays a superset
        const float tmax = (float)(tile_rc2[tile] * (1.0 + 0x1p-9));
        float thr[R];
#pragma unroll
        for (int k = 0; k < R; ++k)
            thr[k] = fmaxf(r2i[k], tmax);
        __syncthreads();
        // the waves take the tile's sources in turn (wave w: w, w + 4, ...); each
        // run of kMerge of a wave's sources is summed in FP32, then merged
        for (int jb = wv; jb < cnt; jb += kWaves * kMerge) {
            const int jm = min(cnt, jb + kWaves * kMerge);
#pragma unroll 2
            for (int jj = jb; jj < jm; jj += kWaves) {
                const float4 A = sa[jj];
                const float4 B = sb[jj];
#pragma unroll
                for (int k = 0; k < R; ++k) {
                    float dx = (A.x - xh[k]) + (B.x - xl[k]);
                    float dy = (A.y - yh[k]) + (B.y - yl[k]);
                    float dz = (A.z - zh[k]) + (B.z - zl[k]);
                    float r2 = fmaf(dz, dz, fmaf(dy, dy, dx * dx));
                    float y = __builtin_amdgcn_rsqf(r2);
                    float s = (A.w * y) * (y * y);
                    if (r2 < thr[k]) {
                        if (r2 < fmaxf(r2i[k], B.w)) {
                            // FP64 changeover pair from the FP64 state
                            int i = ii[k], j = jt + jj;
                            double ex = qx[j] - qx[i], ey = qy[j] - qy[i], ez = qz[j] - qz[i];
                            double d2 = fma(ez, ez, fma(ey, ey, ex * ex));
                            double wgt = m[j] * changeover_w(d2, fmax(rc[i], rc[j]), inner);
                            nx[k] = fma(wgt, ex, nx[k]);
                            ny[k] = fma(wgt, ey, ny[k]);
                            nz[k] = fma(wgt, ez, nz[k]);
                            s = 0.0f;
                            ++near;
                        }
                    }
                    tx[k] = fmaf(s, dx, tx[k]);
                    ty[k] = fmaf(s, dy, ty[k]);
                    tz[k] = fmaf(s, dz, tz[k]);
                }
            }
#pragma unroll
            for (int k = 0; k < R; ++k) {
                two_sum_f(hx[k], lx[k], tx[k]);
                two_sum_f(hy[k], ly[k], ty[k]);
                two_sum_f(hz[k], lz[k], tz[k]);
                tx[k] = ty[k] = tz[k] = 0.0f;
            }
        }
    }
    double sx_[R], sy_[R], sz_[R];
#pragma unroll
    for (int k = 0; k < R; ++k) {
        sx_[k] = ((double)hx[k] + (double)lx[k]) + nx[k];
        sy_[k] = ((double)hy[k] + (double)ly[k]) + ny[k];
        sz_[k] = ((double)hz[k] + (double)lz[k]) + nz[k];
    }
    if (wv > 0) {
#pragma unroll
        for (int k = 0; k < R; ++k) {
            red[wv - 1][3 * k + 0][lane] = sx_[k];
            red[wv - 1][3 * k + 1][lane] = sy_[k];
            red[wv - 1][3 * k + 2][lane] = sz_[k];
        }
    }
    __syncthreads();
    if (wv == 0) {
#pragma unroll
        for (int k = 0; k < R; ++k) {
            for (int w = 0; w < kWaves - 1; ++w) {
                sx_[k] += red[w][3 * k + 0][lane];
                sy_[k] += red[w][3 * k + 1][lane];
                sz_[k] += red[w][3 * k + 2][lane];
            }
            int li = lane + 64 * k;
            if (li < wk.ni) {
                int i = wk.i0 + li;
                fpart[((size_t)0 * maxs + wk.slot) * ntot + i] = (float)sx_[k];
                fpart[((size_t)1 * maxs + wk.slot) * ntot + i] = (float)sy_[k];
                fpart[((size_t)2 * maxs + wk.slot) * ntot + i] = (float)sz_[k];
            }
        }
    }
    for (int o = 32; o > 0; o >>= 1)
        near += __shfl_xor(near, o);
    if (lane == 0 && near)
        atomicAdd((unsigned long long *)&stats->near_pairs, (unsigned long long)near);
}

// Few sources (every system's big bodies in one split): each wave owns the 64 R
// targets of a work item and sums over all of the system's sources.  These are the
// same for every lane and are read through the scalar cache, a few ahead: no staging,
// no LDS, so that registers alone bound the waves per SIMD.  Same pair arithmetic and
// per-target source order as the kernels above, no cross-wave reduction.  Bound by the
// pair arithmetic (about 100 cycles per wave and source in FP64).  100 big bodies and
// 1048576 small ones, one target a lane: with the sources in each wave's LDS 101 us
// (FP64) and 104 us (FP32C), now 83 and 71 us.
__device__ __forceinline__ void wave_lds_sync()
{
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

// The workgroup's changeover pairs to the counter: one atomic per workgroup, as those
// of the whole grid on one counter take turns (11 ns each).
__device__ __forceinline__ void add_near(int near, DevStats *stats)
{
    __shared__ int cnt[kWaves];
    for (int o = 32; o > 0; o >>= 1)
        near += __shfl_xor(near, o);
    if ((threadIdx.x & 63) == 0)
        cnt[threadIdx.x >> 6] = near;
    __syncthreads();
    if (threadIdx.x == 0) {
        int t = 0;
        for (int w = 0; w < kWaves; ++w)
            t += cnt[w];
        if (t)
            atomicAdd((unsigned long long *)&stats->near_pairs, (unsigned long long)t);
    }
}

template <int R>
__global__ __launch_bounds__(kBlock) void k_force64_few(const FWork *__restrict__ work, int nfw,
                                                        const double *__restrict__ qx,
                                                        const double *__restrict__ qy,
                                                        const double *__restrict__ qz,
                                                        const double *__restrict__ m,
                                                        const double *__restrict__ rc,
                                                        const double *__restrict__ tile_rc2,
                                                        double *__restrict__ fpart, int ntot, int maxs,
                                                        double inner, DevStats *stats)
{
    const int lane = threadIdx.x & 63, wv = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    int near = 0;
    for (int it = blockIdx.x * kWaves + wv; it < nfw; it += gridDim.x * kWaves) {
        const FWork wk = work[it];
        double xi[R], yi[R], zi[R], rci[R], r2i[R], thr[R], ax[R], ay[R], az[R];
        const double tmax = tile_rc2[wk.rb0];
#pragma unroll
        for (int k = 0; k < R; ++k) {
            const int li = lane + 64 * k;
            const int i = wk.i0 + (li < wk.ni ? li : 0);
            xi[k] = qx[i];
            yi[k] = qy[i];
            zi[k] = qz[i];
            rci[k] = rc[i];
            r2i[k] = fmax(rci[k] * rci[k], DBL_MIN);
            thr[k] = fmax(r2i[k], tmax);
            ax[k] = ay[k] = az[k] = 0.0;
        }
#pragma unroll 4
        for (int jj = 0; jj < wk.nj; ++jj) {
            const int j = wk.j0 + jj;
            const double Jx = qx[j], Jy = qy[j], Jz = qz[j], mj = m[j];
            const double m15 = 1.5 * mj;
#pragma unroll
            for (int k = 0; k < R; ++k) {
                double dx = Jx - xi[k], dy = Jy - yi[k], dz = Jz - zi[k];
                double r2 = fma(dz, dz, fma(dy, dy, dx * dx));
                double s = m_rinv3(mj, m15, r2);
                if (r2 < thr[k]) {
                    double rcj = rc[j];
                    if (r2 < fmax(r2i[k], fmax(rcj * rcj, DBL_MIN))) {
                        s = mj * changeover_w(r2, fmax(rci[k], rcj), inner);
                        ++near;
                    }
                }
                ax[k] = fma(s, dx, ax[k]);
                ay[k] = fma(s, dy, ay[k]);
                az[k] = fma(s, dz, az[k]);
            }
        }
#pragma unroll
        for (int k = 0; k < R; ++k) {
            const int li = lane + 64 * k;
            if (li < wk.ni) {
                const int i = wk.i0 + li;
                fpart[((size_t)0 * maxs + wk.slot) * ntot + i] = ax[k];
                fpart[((size_t)1 * maxs + wk.slot) * ntot + i] = ay[k];
                fpart[((size_t)2 * maxs + wk.slot) * ntot + i] = az[k];
            }
        }
    }
    add_near(near, stats);
}

template <int R>
__global__ __launch_bounds__(kBlock) void k_force32c_few(const FWork *__restrict__ work, int nfw,
                                                         const float4 *__restrict__ pk,
                                                         const double *__restrict__ qx,
                                                         const double *__restrict__ qy,
                                                         const double *__restrict__ qz,
                                                         const double *__restrict__ m,
                                                         const double *__restrict__ rc,
                                                         const double *__restrict__ tile_rc2,
                                                         float *__restrict__ fpart, int ntot,
                                                         int maxs, double inner, DevStats *stats)
{
    const int lane = threadIdx.x & 63, wv = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    int near = 0;
    for (int it = blockIdx.x * kWaves + wv; it < nfw; it += gridDim.x * kWaves) {
        const FWork wk = work[it];
        float xh[R], yh[R], zh[R], xl[R], yl[R], zl[R], r2i[R], thr[R];
        float hx[R], hy[R], hz[R], lx[R], ly[R], lz[R], tx[R], ty[R], tz[R];
        double nx[R], ny[R], nz[R];
        int ii[R];
        const float tmax = (float)(tile_rc2[wk.rb0] * (1.0 + 0x1p-9));
#pragma unroll
        for (int k = 0; k < R; ++k) {
            const int li = lane + 64 * k;
            const int i = wk.i0 + (li < wk.ni ? li : 0);
            ii[k] = i;
            const float4 A = pk[2 * (size_t)i], B = pk[2 * (size_t)i + 1];
            xh[k] = A.x; yh[k] = A.y; zh[k] = A.z;
            xl[k] = B.x; yl[k] = B.y; zl[k] = B.z;
            r2i[k] = B.w;
            thr[k] = fmaxf(r2i[k], tmax);
            hx[k] = hy[k] = hz[k] = lx[k] = ly[k] = lz[k] = tx[k] = ty[k] = tz[k] = 0.0f;
            nx[k] = ny[k] = nz[k] = 0.0;
        }
        for (int jb = 0; jb < wk.nj; jb += kMerge) {
            const int jm = min(wk.nj, jb + kMerge);
#pragma unroll 4
            for (int jj = jb; jj < jm; ++jj) {
                const float4 A = pk[2 * (size_t)(wk.j0 + jj)];
                const float4 B = pk[2 * (size_t)(wk.j0 + jj) + 1];
#pragma unroll
                for (int k = 0; k < R; ++k) {
                    float dx = (A.x - xh[k]) + (B.x - xl[k]);
                    float dy = (A.y - yh[k]) + (B.y - yl[k]);
                    float dz = (A.z - zh[k]) + (B.z - zl[k]);
                    float r2 = fmaf(dz, dz, fmaf(dy, dy, dx * dx));
                    float y = __builtin_amdgcn_rsqf(r2);
                    float s = (A.w * y) * (y * y);
                    if (r2 < thr[k]) {
                        if (r2 < fmaxf(r2i[k], B.w)) {
                            int i = ii[k], j = wk.j0 + jj;
                            double ex = qx[j] - qx[i], ey = qy[j] - qy[i], ez = qz[j] - qz[i];
                            double d2 = fma(ez, ez, fma(ey, ey, ex * ex));
                            double wgt = m[j] * changeover_w(d2, fmax(rc[i], rc[j]), inner);
                            nx[k] = fma(wgt, ex, nx[k]);
                            ny[k] = fma(wgt, ey, ny[k]);
                            nz[k] = fma(wgt, ez, nz[k]);
                            s = 0.0f;
                            ++near;
                        }
                    }
                    tx[k] = fmaf(s, dx, tx[k]);
                    ty[k] = fmaf(s, dy, ty[k]);
                    tz[k] = fmaf(s, dz, tz[k]);
                }
            }
#pragma unroll
            for (int k = 0; k < R; ++k) {
                two_sum_f(hx[k], lx[k], tx[k]);
                two_sum_f(hy[k], ly[k], ty[k]);
                two_sum_f(hz[k], lz[k], tz[k]);
                tx[k] = ty[k] = tz[k] = 0.0f;
            }
        }
#pragma unroll
        for (int k = 0; k < R; ++k) {
            const int li = lane + 64 * k;
            if (li < wk.ni) {
                const int i = wk.i0 + li;
                fpart[((size_t)0 * maxs + wk.slot) * ntot + i] = (float)(((double)hx[k] + (double)lx[k]) + nx[k]);
                fpart[((size_t)1 * maxs + wk.slot) * ntot + i] = (float)(((double)hy[k] + (double)ly[k]) + ny[k]);
                fpart[((size_t)2 * maxs + wk.slot) * ntot + i] = (float)(((double)hz[k] + (double)lz[k]) + nz[k]);
            }
        }
    }
    add_near(near, stats);
}

// Symmetric pairs (every body big): each unordered pair is evaluated once and
// applied to both bodies, a_i += m_j q d and a_j -= m_i q d with the mass-free
// weight q = K/r^3 - K'/r^2 (Newtonian q = 1/r^3 refined from the hardware
// estimate as in m_rinv3).  Bodies of a system form tiles of T = 64 R and
// super-tiles of G tiles.  A work item is a pair of super-tiles (I <= J),
// owned by a workgroup of G waves: wave w holds the R targets per lane of tile
// w of I in registers, the G tiles of J sit in LDS together with their
// accumulators, and in round k wave w meets tile (w + k) mod G of J, so that no
// two waves update one source tile at once.  Within a tile pair, at step k of
// sub-tile t, lane L pairs with source 64 t + (L xor k), so the 64 lanes touch
// 64 different sources and update their accumulators without atomics.  Item
// (I, J) writes super-tile I's sums to split slot J and super-tile J's sums to
// slot I (both to slot I on the diagonal, where each pair is met once), so
// every body receives exactly one partial per super-tile of its system, summed
// in slot order by the finalize pass: G times fewer partials than tiles, in a
// fixed order whatever the schedule.  The register budget keeps three waves
// per SIMD (two at R = 4), as with one wave per work item.
__device__ __forceinline__ double rinv3(double r2)
{
    const double y0 = __builtin_amdgcn_rsq(r2);
    const double y2 = y0 * y0;
    const double e = fma(-r2, y2, 1.0);
    return (y0 * y2) * fma(1.5, e, 1.0);
}

// max of two non-negative finite floats through their bit patterns (one
// integer instruction, no NaN handling needed)
__device__ __forceinline__ float max_nonneg(float a, float b)
{
    return __int_as_float(max(__float_as_int(a), __float_as_int(b)));
}

__device__ __forceinline__ float wave_max_nonneg(float v)
{
    for (int o = 32; o > 0; o >>= 1)
        v = max_nonneg(v, __shfl_xor(v, o));
    return __int_as_float(__builtin_amdgcn_readfirstlane(__float_as_int(v)));
}

// LDS addresses as 32-bit integers, for the rotating source index of the
// symmetric kernels: with a tile array aligned to 64 elements, the address of
// element 64 t + (lane xor k) is that of element 64 t + lane with k times the
// element size xored in.
typedef float lds_v4f __attribute__((ext_vector_type(4)));
typedef __attribute__((address_space(3))) lds_v4f lds_float4;
typedef __attribute__((address_space(3))) double lds_double;

__device__ __forceinline__ uint32_t lds_addr(float4 *p)
{
    return (uint32_t)(uintptr_t)(lds_float4 *)p;
}

__device__ __forceinline__ uint32_t lds_addr(double *p)
{
    return (uint32_t)(uintptr_t)(lds_double *)p;
}

__device__ __forceinline__ float4 lds_ld4(uint32_t a)
{
    const lds_v4f v = *(const lds_float4 *)(uintptr_t)a;
    return make_float4(v.x, v.y, v.z, v.w);
}

// x, y, z of a 16-byte record (the fourth word is neither read nor written)
typedef float lds_v3f __attribute__((ext_vector_type(3)));
typedef __attribute__((address_space(3))) lds_v3f lds_float3;

__device__ __forceinline__ lds_v3f lds_ld3(uint32_t a)
{
    return *(const lds_float3 *)(uintptr_t)a;
}

__device__ __forceinline__ void lds_st3(uint32_t a, float x, float y, float z)
{
    *(lds_float3 *)(uintptr_t)a = lds_v3f{x, y, z};
}

__device__ __forceinline__ double lds_ld8(uint32_t a)
{
    return *(const lds_double *)(uintptr_t)a;
}

__device__ __forceinline__ void lds_st8(uint32_t a, double v)
{
    *(lds_double *)(uintptr_t)a = v;
}

// Tile J of one wave in LDS, one array per component (consecutive lanes touch
// consecutive 8-byte words: no bank conflicts for the rotating accesses).
template <int T>
struct alignas(512) SymTile64 {
    double x[T], y[T], z[T], m[T];
    double r2[T];                      // max(rc^2, DBL_MIN)
    double rc[T];
    double ax[T], ay[T], az[T];        // tile J's sums
};
static_assert(offsetof(SymTile64<64>, m) == 8 * 3 * 64 && offsetof(SymTile64<64>, r2) == 8 * 4 * 64 &&
                  offsetof(SymTile64<64>, rc) == 8 * 5 * 64 && offsetof(SymTile64<64>, ax) == 8 * 6 * 64,
              "SymTile64 layout");

template <int R, bool DIAG, int T>
__device__ __forceinline__ void sym_tile64(SymTile64<T> &L, int lane, int i0, int ni, double inner,
                                           const double *__restrict__ rc, const double (&xi)[R],
                                           const double (&yi)[R], const double (&zi)[R],
                                           const double (&mi)[R], double tmi, double (&ax)[R],
                                           double (&ay)[R], double (&az)[R], int &near)
{
#pragma unroll 1
    for (int t = 0; t < R; ++t) {
        // Step k: lane L pairs its targets with source L xor k of sub-tile t,
        // so the lanes of a step touch distinct sources and each lane meets
        // every source once in 64 steps.  The sums a step reads were written by
        // another lane one step earlier: LDS operations of a wave complete in
        // issue order, and the compiler barrier keeps the read after that
        // write.  Sources are read-only and read one step ahead.
        // the largest rc^2 of the wave's targets and of the sub-tile's sources:
        // one compare per pair outside the rare branch
        const double thr = fmax(tmi, wave_max(L.r2[64 * t + lane]));
        // LDS address of x[64 t + lane]; the other arrays at fixed offsets
        const uint32_t self = lds_addr(&L.x[64 * t + lane]);
        uint32_t ac = self;
        double jxs = lds_ld8(ac), jys = lds_ld8(ac + 8 * T), jzs = lds_ld8(ac + 16 * T),
               jms = lds_ld8(ac + 24 * T);
#pragma unroll 2
        for (int k = 0; k < 64; ++k) {
            const uint32_t an = self ^ (uint32_t)(((k + 1) & 63) << 3);
            const double xn = lds_ld8(an), yn = lds_ld8(an + 8 * T), zn = lds_ld8(an + 16 * T),
                         mn = lds_ld8(an + 24 * T);
            double jx = lds_ld8(ac + 48 * T), jy = lds_ld8(ac + 56 * T), jz = lds_ld8(ac + 64 * T);
            // the R pairs' geometry first, then one branch for the rare ones,
            // so that the R chains share one basic block
            double dxr[R], dyr[R], dzr[R], r2r[R], qr[R];
            bool cand = false;
#pragma unroll
            for (int r = 0; r < R; ++r) {
                dxr[r] = jxs - xi[r];
                dyr[r] = jys - yi[r];
                dzr[r] = jzs - zi[r];
                r2r[r] = fma(dzr[r], dzr[r], fma(dyr[r], dyr[r], dxr[r] * dxr[r]));
                qr[r] = rinv3(r2r[r]);
                const bool on = !DIAG || (64 * r + lane < 64 * t + (lane ^ k));
                cand |= r2r[r] < thr && on;
                if (DIAG)
                    qr[r] = on ? qr[r] : 0.0;
            }
            if (cand) {
#pragma unroll
                for (int r = 0; r < R; ++r) {
                    const bool on = !DIAG || (64 * r + lane < 64 * t + (lane ^ k));
                    if (r2r[r] < thr && on) {
                        // rare: the target's rc from memory (a padded target is a copy
                        // of body i0), the source's rc^2 and rc from its LDS record
                        const int li = 64 * r + lane;
                        const double rci = rc[i0 + (li < ni ? li : 0)];
                        if (r2r[r] < fmax(fmax(rci * rci, DBL_MIN), lds_ld8(ac + 32 * T))) {
                            qr[r] = changeover_w(r2r[r], fmax(rci, lds_ld8(ac + 40 * T)), inner);
                            ++near;
                        }
                    }
                }
            }
#pragma unroll
            for (int r = 0; r < R; ++r) {
                const double dx = dxr[r], dy = dyr[r], dz = dzr[r], q = qr[r];
                const double wi = jms * q, wj = mi[r] * q;
                ax[r] = fma(wi, dx, ax[r]);
                ay[r] = fma(wi, dy, ay[r]);
                az[r] = fma(wi, dz, az[r]);
                jx = fma(-wj, dx, jx);
                jy = fma(-wj, dy, jy);
                jz = fma(-wj, dz, jz);
            }
            lds_st8(ac + 48 * T, jx);
            lds_st8(ac + 56 * T, jy);
            lds_st8(ac + 64 * T, jz);
            __asm__ __volatile__("" ::: "memory");
            ac = an;
            jxs = xn;
            jys = yn;
            jzs = zn;
            jms = mn;
        }
    }
}

// A double moved one lane down the wave: lane L gets lane (L + 1) mod 64's
// value (DPP wave rotate, one VALU per 32-bit half).
__device__ __forceinline__ double wave_rotl1(double v)
{
    const long long b = __double_as_longlong(v);
    const int lo = __builtin_amdgcn_mov_dpp((int)b, 0x134, 0xF, 0xF, false);
    const int hi = __builtin_amdgcn_mov_dpp((int)(b >> 32), 0x134, 0xF, 0xF, false);
    return __longlong_as_double(((long long)hi << 32) | (unsigned int)lo);
}

// Tile J of one wave for the FP64 loop with source sums in registers (R <= 2).
// Each sub-tile's source records are stored twice over (entry 64 + j repeats
// j), so that lane L reads source (L + k) mod 64 at entry L + k: a fixed
// offset from the lane's own entry, no wrap.  Only the FP64 totals of the
// sources' sums live here.
template <int R, int C = 1>
struct alignas(512) SymTile64R {
    struct Sub {
        double x[128], y[128], z[128], m[128];
    } s[R];
    double r2[64 * R];                 // max(rc^2, DBL_MIN)
    double rc[64 * R];
    double tot[C][3][64 * R];          // tile J's FP64 totals (C copies: sym_part)
};

// The waves of a workgroup that share one tile pair (H of them, one tile pair per
// workgroup) split its 64 R steps evenly: wave h takes the sub-tiles from t0 on,
// t1 not included, and of each the kSteps steps from k0 on.  Where the waves
// outnumber the sub-tiles, the kCopies waves of one sub-tile meet the same sources
// and each adds to totals of its own (copy c).
template <int R, int H>
struct SymPart {
    static constexpr int kCopies = H > R ? H / R : 1;
    static constexpr int kSteps = 64 / kCopies;
    int t0, t1, k0, c;
    __device__ __forceinline__ explicit SymPart(int h)
    {
        c = h % kCopies;
        t0 = h * R / H;
        t1 = H > R ? t0 + 1 : (h + 1) * R / H;
        k0 = c * kSteps;
    }
};

template <int R, int C>
__device__ __forceinline__ void put_src64(SymTile64R<R, C> &S, int e, double x, double y, double z,
                                          double m, double rcj)
{
    typename SymTile64R<R, C>::Sub &U = S.s[e / 64];
    const int j = e % 64;
    U.x[j] = U.x[j + 64] = x;
    U.y[j] = U.y[j + 64] = y;
    U.z[j] = U.z[j + 64] = z;
    U.m[j] = U.m[j + 64] = m;
    S.rc[e] = rcj;
    S.r2[e] = fmax(rcj * rcj, DBL_MIN);
#pragma unroll
    for (int c = 0; c < C; ++c)
        S.tot[c][0][e] = S.tot[c][1][e] = S.tot[c][2][e] = 0.0;
}

template <int T>
__device__ __forceinline__ void put_src64(SymTile64<T> &S, int e, double x, double y, double z,
                                          double m, double rcj)
{
    S.x[e] = x;
    S.y[e] = y;
    S.z[e] = z;
    S.m[e] = m;
    S.rc[e] = rcj;
    S.r2[e] = fmax(rcj * rcj, DBL_MIN);
    S.ax[e] = S.ay[e] = S.az[e] = 0.0;
}

// The tile pair of sym_tile64 with the sources' running sums in registers:
// in step k lane L pairs its targets with source (L + k) mod 64 of sub-tile t
// and holds that source's sums; after the step the sums move one lane down
// (wave_rotl1), where that source is met next.  After 64 steps every lane
// holds its own source's sums again and adds them to the FP64 totals.  The LDS
// then carries only the source records (32 B per lane and step instead of 80
// with the sums' read-modify-write), which keeps the FP64 loop off the LDS
// bandwidth limit; the moves cost 6 VALU per step.
template <int R, bool DIAG, int H, int C>
__device__ __forceinline__ void sym_tile64_rot(SymTile64R<R, C> &L, const SymPart<R, H> &part, int lane, int i0, int ni, int nj,
                                               double inner, const double *__restrict__ rc,
                                               const double (&xi)[R], const double (&yi)[R],
                                               const double (&zi)[R], const double (&mi)[R],
                                               double tmi, double (&ax)[R], double (&ay)[R],
                                               double (&az)[R], int &near)
{
#pragma unroll 1
    for (int t = part.t0; t < part.t1 && 64 * t < nj; ++t) {
        const double thr = fmax(tmi, wave_max(L.r2[64 * t + lane]));
        // LDS address of x[lane + k0] of sub-tile t; y, z, m at fixed offsets
        constexpr uint32_t kY = 8 * 128, kZ = 16 * 128, kM = 24 * 128;
        uint32_t ac = lds_addr(&L.s[t].x[lane + part.k0]);
        double jxs = lds_ld8(ac), jys = lds_ld8(ac + kY), jzs = lds_ld8(ac + kZ), jms = lds_ld8(ac + kM);
        double jx = 0.0, jy = 0.0, jz = 0.0;
#pragma unroll 2
        for (int kk = 0; kk < SymPart<R, H>::kSteps; ++kk) {
            const int k = part.k0 + kk;
            const uint32_t an = ac + 8;
            const double xn = lds_ld8(an), yn = lds_ld8(an + kY), zn = lds_ld8(an + kZ),
                         mn = lds_ld8(an + kM);
            double dxr[R], dyr[R], dzr[R], r2r[R], qr[R];
            bool cand = false;
#pragma unroll
            for (int r = 0; r < R; ++r) {
                dxr[r] = jxs - xi[r];
                dyr[r] = jys - yi[r];
                dzr[r] = jzs - zi[r];
                r2r[r] = fma(dzr[r], dzr[r], fma(dyr[r], dyr[r], dxr[r] * dxr[r]));
                qr[r] = rinv3(r2r[r]);
                const bool on = !DIAG || (64 * r + lane < 64 * t + ((lane + k) & 63));
                cand |= r2r[r] < thr && on;
                if (DIAG)
                    qr[r] = on ? qr[r] : 0.0;
            }
            if (cand) {
                const int sj = 64 * t + ((lane + k) & 63);
#pragma unroll
                for (int r = 0; r < R; ++r) {
                    const bool on = !DIAG || (64 * r + lane < sj);
                    if (r2r[r] < thr && on) {
                        const int li = 64 * r + lane;
                        const double rci = rc[i0 + (li < ni ? li : 0)];
                        if (r2r[r] < fmax(fmax(rci * rci, DBL_MIN), L.r2[sj])) {
                            qr[r] = changeover_w(r2r[r], fmax(rci, L.rc[sj]), inner);
                            ++near;
                        }
                    }
                }
            }
#pragma unroll
            for (int r = 0; r < R; ++r) {
                const double dx = dxr[r], dy = dyr[r], dz = dzr[r], q = qr[r];
                const double wi = jms * q, wj = mi[r] * q;
                ax[r] = fma(wi, dx, ax[r]);
                ay[r] = fma(wi, dy, ay[r]);
                az[r] = fma(wi, dz, az[r]);
                jx = fma(-wj, dx, jx);
                jy = fma(-wj, dy, jy);
                jz = fma(-wj, dz, jz);
            }
            jx = wave_rotl1(jx);
            jy = wave_rotl1(jy);
            jz = wave_rotl1(jz);
            ac = an;
            jxs = xn;
            jys = yn;
            jzs = zn;
            jms = mn;
        }
        // the sums in this lane are now those of the source it would meet next
        double (&tot)[3][64 * R] = L.tot[part.c];
        const int js = 64 * t + ((lane + part.k0 + SymPart<R, H>::kSteps) & 63);
        tot[0][js] += jx;
        tot[1][js] += jy;
        tot[2][js] += jz;
    }
}

template <int R, bool DIAG, int T, int H, int C>
__device__ __forceinline__ void sym_round64(SymTile64R<R, C> &L, const SymPart<R, H> &part, int lane,
                                            int i0, int ni, int nj, double inner,
                                            const double *__restrict__ rc, const double (&xi)[R],
                                            const double (&yi)[R], const double (&zi)[R],
                                            const double (&mi)[R], double tmi, double (&ax)[R],
                                            double (&ay)[R], double (&az)[R], int &near)
{
    sym_tile64_rot<R, DIAG>(L, part, lane, i0, ni, nj, inner, rc, xi, yi, zi, mi, tmi, ax, ay, az, near);
}

template <int R, bool DIAG, int T, int H>
__device__ __forceinline__ void sym_round64(SymTile64<T> &L, const SymPart<R, H> &, int lane, int i0,
                                            int ni, int, double inner,
                                            const double *__restrict__ rc, const double (&xi)[R],
                                            const double (&yi)[R], const double (&zi)[R],
                                            const double (&mi)[R], double tmi, double (&ax)[R],
                                            double (&ay)[R], double (&az)[R], int &near)
{
    sym_tile64<R, DIAG, T>(L, lane, i0, ni, inner, rc, xi, yi, zi, mi, tmi, ax, ay, az, near);
}

// Total c of source e of the tile, its copies in order.
template <int R, int C>
__device__ __forceinline__ double src_total(const SymTile64R<R, C> &S, int c, int e)
{
    double v = S.tot[0][c][e];
#pragma unroll
    for (int k = 1; k < C; ++k)
        v += S.tot[k][c][e];
    return v;
}

template <int T>
__device__ __forceinline__ double src_total(const SymTile64<T> &S, int c, int e)
{
    return c == 0 ? S.ax[e] : (c == 1 ? S.ay[e] : S.az[e]);
}

template <int R, int G, int H = 1>
__global__ __launch_bounds__(64 * G * H, R == 4 ? 2 : 3) void k_force64_sym(const FWork *__restrict__ work, int nitems,
                                                        const double *__restrict__ qx,
                                                        const double *__restrict__ qy,
                                                        const double *__restrict__ qz,
                                                        const double *__restrict__ m,
                                                        const double *__restrict__ rc,
                                                        double *__restrict__ fpart, int ntot, int maxs,
                                                        double inner, DevStats *stats)
{
    static_assert(H == 1 || (G == 1 && R <= 2), "only single tile pairs are shared");
    constexpr int T = 64 * R;
    // R <= 2: the sources' sums in registers, moved between lanes (LDS holds
    // the records only); R = 4 amortises the sums' LDS traffic over four
    // targets per lane and keeps them in LDS, within its LDS budget
    using Tile = typename std::conditional<(R <= 2), SymTile64R<R, SymPart<R, H>::kCopies>,
                                           SymTile64<T>>::type;
    __shared__ Tile tl[G];
    // H > 1: the waves' sums of the targets
    __shared__ double tgt[H > 1 ? H : 1][3][H > 1 ? T : 1];
    const int lane = threadIdx.x & 63, wv = H > 1 ? 0 : threadIdx.x >> 6;
    const int wh = threadIdx.x >> 6;
    const SymPart<R, H> part(H > 1 ? wh : 0);
    int near = 0;
    for (int it = blockIdx.x; it < nitems; it += gridDim.x) {
        const FWork wk = work[it];
        const bool diag = wk.i0 == wk.j0;
        // the G source tiles of super-tile J (nj real records from j0)
        for (int k = threadIdx.x; k < G * T; k += 64 * G * H) {
            // sources past the end: massless and far away (r^2 ~ 1e300, so
            // their weight underflows to 0 instead of meeting a target at r = 0)
            const bool ok = k < wk.nj;
            const int j = wk.j0 + (ok ? k : 0);
            put_src64(tl[k / T], k % T, ok ? qx[j] : 1e150, ok ? qy[j] : 1e150, ok ? qz[j] : 1e150,
                      ok ? m[j] : 0.0, ok ? rc[j] : 0.0);
        }
        __syncthreads();
        // this wave's target tile: tni bodies from ti0 (none when tni <= 0)
        const int ti0 = wk.i0 + wv * T;
        const int tni = min(T, wk.ni - wv * T);
        double xi[R], yi[R], zi[R], mi[R], ax[R], ay[R], az[R];
        double tmi = DBL_MIN;
#pragma unroll
        for (int r = 0; r < R; ++r) {
            const int li = 64 * r + lane;
            const bool ok = li < tni;
            const int i = ok ? ti0 + li : wk.i0;
            xi[r] = qx[i];
            yi[r] = qy[i];
            zi[r] = qz[i];
            // targets past the tile end are massless: they add nothing to the sources
            mi[r] = ok ? m[i] : 0.0;
            tmi = fmax(tmi, rc[i] * rc[i]);
            ax[r] = ay[r] = az[r] = 0.0;
        }
        tmi = wave_max(tmi);
        // rounds as in the FP32C kernel: wave w meets source tile (w + k) mod G
        const int nr = diag ? G / 2 + 1 : G;
        for (int k = 0; k < nr; ++k) {
            const int s = (wv + k) % G;
            const bool go = tni > 0 && s * T < wk.nj && !(diag && 2 * k == G && wv >= G / 2);
            if (go) {
                if (diag && k == 0)
                    sym_round64<R, true, T>(tl[s], part, lane, ti0, tni, wk.nj - s * T, inner, rc, xi, yi, zi, mi, tmi,
                                            ax, ay, az, near);
                else
                    sym_round64<R, false, T>(tl[s], part, lane, ti0, tni, wk.nj - s * T, inner, rc, xi, yi, zi, mi, tmi,
                                             ax, ay, az, near);
            }
            __syncthreads();
        }
        // super-tile I's sums to slot J (on the diagonal together with the same
        // bodies' sums as sources)
#pragma unroll
        for (int r = 0; r < R; ++r) {
            const int li = 64 * r + lane;
            if (li < tni) {
                double sx_ = ax[r], sy_ = ay[r], sz_ = az[r];
                if (H > 1) {
                    tgt[wh % H][0][li] = sx_;
                    tgt[wh % H][1][li] = sy_;
                    tgt[wh % H][2][li] = sz_;
                    continue;
                }
                if (diag) {
                    sx_ += src_total(tl[wv], 0, li);
                    sy_ += src_total(tl[wv], 1, li);
                    sz_ += src_total(tl[wv], 2, li);
                }
                const int i = ti0 + li;
                fpart[((size_t)0 * maxs + wk.slot) * ntot + i] = sx_;
                fpart[((size_t)1 * maxs + wk.slot) * ntot + i] = sy_;
                fpart[((size_t)2 * maxs + wk.slot) * ntot + i] = sz_;
            }
        }
        if (H > 1) {
            // the waves' sums in wave order
            __syncthreads();
            for (int e = threadIdx.x; e < tni; e += 64 * H)
#pragma unroll
                for (int c = 0; c < 3; ++c) {
                    double v = tgt[0][c][e];
#pragma unroll
                    for (int h = 1; h < H; ++h)
                        v += tgt[h][c][e];
                    if (diag)
                        v += src_total(tl[0], c, e);
                    fpart[((size_t)c * maxs + wk.slot) * ntot + ti0 + e] = v;
                }
        }
        if (!diag) {
            // super-tile J's sums to slot I
            for (int k = threadIdx.x; k < wk.nj; k += 64 * G * H) {
                const Tile &S = tl[k / T];
                const int e = k % T, j = wk.j0 + k;
                fpart[((size_t)0 * maxs + wk.pad) * ntot + j] = src_total(S, 0, e);
                fpart[((size_t)1 * maxs + wk.pad) * ntot + j] = src_total(S, 1, e);
                fpart[((size_t)2 * maxs + wk.pad) * ntot + j] = src_total(S, 2, e);
            }
        }
        __syncthreads();
    }
    for (int o = 32; o > 0; o >>= 1)
        near += __shfl_xor(near, o);
    if (lane == 0 && near)
        atomicAdd((unsigned long long *)&stats->near_pairs, (unsigned long long)near);
}

// FP32C form of the symmetric tile pairs.  Pair terms in FP32 from the hi/lo
// records.  Tile I's sums: FP32 runs of half a sub-tile round (32 steps)
// merged by two-sum into a (hi, lo) pair per target.  Tile J's sums: an FP32
// run sum per source over the same 32 steps (in registers that move between lanes, as
// in FP64, or at R = 4 and with the encounter test fused in, in LDS), added to the
// source's FP64 total when the run ends.  In registers: 8000 bodies in tiles of 64 37.3
// -> 29.7 us, 131072 bodies in tiles of 128 4955 -> 4770 us.  Changeover pairs in FP64 from the FP64 state: the
// target's part into its (hi, lo) pair, the source's part to its FP64 total.
// Each split partial is stored rounded to FP32: a rounding of at most 2^-24 of
// the partial, which is at most the sum of its terms' magnitudes, so all of a
// body's partials together add at most 2^-24 A_i (A_i the sum of the magnitudes
// of its pair terms), below the FP32 pair terms' own error.
// Aligned to 1024 bytes, so that the LDS address of a[64 t + (lane xor k)]
// is that of a[64 t + lane] with 16 k xored in (k < 64): one VALU per step
// addresses a[], b[] and run[] (fixed offsets 16 T and 32 T from a[]).
template <int T>
struct alignas(1024) SymTile32 {
    float4 a[T];                    // hi parts and mass
    float4 b[T];                    // lo parts and widened rc^2
    float4 run[T];                  // current FP32 run sums of tile J (x, y, z, -)
    double ax[T], ay[T], az[T];     // FP64 totals of tile J (consecutive planes)
};
static_assert(offsetof(SymTile32<64>, b) == 16 * 64 && offsetof(SymTile32<64>, run) == 32 * 64,
              "SymTile32 layout");
static_assert(offsetof(SymTile32<128>, b) == 16 * 128 && offsetof(SymTile32<128>, run) == 32 * 128,
              "SymTile32 layout");

// The target's FP64 part of a changeover pair (hit: the pair was one).
struct ChgPart {
    double x, y, z;
    int hit;
};

// The rare branch of the FP32C pair loop, out of line so that it adds nothing
// to the loop: target li of the item (position i0 + li, or a padded copy of
// position i0 when li >= ni) against source jj (position j0 + jj) at FP32 squared
// distance r2.  Positions are body indices, or with a sorted order
// (ord != nullptr) the bodies ord[position].
// Unless r2 is inside the pair's widened critical radius it returns hit = 0.
// Otherwise the pair is evaluated in FP64 from the FP64 state: -m_i w (Q_j - Q_i)
// goes to source jj's FP64 totals tot[jj], tot[T + jj], tot[2 T + jj], and the
// target's part m_j w (Q_j - Q_i) is returned (zero for a padded target).
__device__ __noinline__ ChgPart changeover_pair32(float r2, float r2j, const float4 *__restrict__ pk,
                                                  int i0, int li, int ni, int j0, int jj, int T,
                                                  double *tot,
                                                  const double *__restrict__ qx,
                                                  const double *__restrict__ qy,
                                                  const double *__restrict__ qz,
                                                  const double *__restrict__ m,
                                                  const double *__restrict__ rc, double inner,
                                                  const int *__restrict__ ord)
{
    ChgPart out{0.0, 0.0, 0.0, 0};
    const bool ok = li < ni;
    const int i = i0 + (ok ? li : 0);
    const int bi = ord ? ord[i] : i;
    if (!(r2 < max_nonneg(pk[2 * (size_t)bi + 1].w, r2j)))
        return out;
    out.hit = 1;
    const int bj = ord ? ord[j0 + jj] : j0 + jj;
    const double gx = qx[bj] - qx[bi], gy = qy[bj] - qy[bi], gz = qz[bj] - qz[bi];
    const double d2 = fma(gz, gz, fma(gy, gy, gx * gx));
    const double w = changeover_w_inl(d2, fmax(rc[bi], rc[bj]), inner);
    if (ok) {
        const double wi = m[bj] * w;
        out.x = wi * gx;
        out.y = wi * gy;
        out.z = wi * gz;
        const double wj = m[bi] * w;
        tot[jj] = fma(-wj, gx, tot[jj]);
        tot[T + jj] = fma(-wj, gy, tot[T + jj]);
        tot[2 * T + jj] = fma(-wj, gz, tot[2 * T + jj]);
    }
    return out;
}

// An FP64 term into a (hi, lo) FP32 accumulator: its leading float by two-sum,
// the float of the remainder into lo.
__device__ __forceinline__ void add_f64_to_pair(float &hi, float &lo, double v)
{
    const float vh = (float)v;
    two_sum_f(hi, lo, vh);
    lo += (float)(v - (double)vh);
}

// What the FP32C pair loop needs for the encounter test fused into it (sorted
// order): the sorted records, the step, and the list and flags to append to.
struct EncCtx {
    const SRec *srec;
    double dt;
    unsigned long long *keys;
    int cap;
    int *ce;
    DevStats *stats;
};

// Exact encounter test of two sorted positions, with the append of a flagged
// pair (defined with the encounter check).
__device__ __noinline__ void enc_candidate(const SRec *__restrict__ srec, double dt,
                                           unsigned long long *keys, int cap, int *ce,
                                           DevStats *stats, int pi, int pj);

// The tile of 64 R sources with, after the FP32C fields, each source's
// encounter records in FP32: chord midpoint M with the widened bound b' of
// 3/4 eps + rc (em), and chord c (ec).  The FP32C tile is a member, not a base:
// a base's tail padding may hold the derived members, while a member object
// keeps its whole size, so em[] starts exactly sizeof(SymTile32<T>) bytes after
// the tile's first record and ec[] 16 T bytes after that.
template <int T>
struct alignas(1024) SymTile32E {
    SymTile32<T> t;
    float4 em[T];
    float4 ec[T];
};
#pragma clang diagnostic push
#pragma clang diagnostic ignored "-Winvalid-offsetof"
static_assert(offsetof(SymTile32E<64>, em) == sizeof(SymTile32<64>) &&
                  offsetof(SymTile32E<128>, em) == sizeof(SymTile32<128>) &&
                  offsetof(SymTile32E<256>, em) == sizeof(SymTile32<256>) &&
                  offsetof(SymTile32E<64>, ec) == sizeof(SymTile32<64>) + 16 * 64 &&
                  offsetof(SymTile32E<128>, ec) == sizeof(SymTile32<128>) + 16 * 128 &&
                  offsetof(SymTile32E<256>, ec) == sizeof(SymTile32<256>) + 16 * 256,
              "SymTile32E: em[] and ec[] right after the FP32C tile");
#pragma clang diagnostic pop

// ENC: the encounter test fused in (sorted order).  Target r of sub-tile t is
// tested against the sources when bit t R + r of `live` is set (the tile pair
// survived the culling): the relative-chord filter in FP32 (midpoints emi[r],
// chords eci[r] and the source's em, ec records), and the pairs that pass go to
// the exact test.  The source records are read from the LDS tile at fixed
// offsets past the FP32C fields (em, ec of SymTile32E).
// FAR: bit t of `far` set means every target of the wave lies apart from every
// source of sub-tile t by more than 2^21 times their low parts' norms and
// outside their critical radii (the radial tile bounds prove it): those pairs
// take the differences of the high parts alone, with no changeover test.
template <int R, bool DIAG, int T, bool ENC = false, bool FAR = false>
__device__ __forceinline__ void sym_tile32c(SymTile32<T> &L, int lane, int i0, int ni, int j0,
                                            double inner, const float4 *__restrict__ pk,
                                            const double *__restrict__ qx,
                                            const double *__restrict__ qy,
                                            const double *__restrict__ qz,
                                            const double *__restrict__ m,
                                            const double *__restrict__ rc, const float (&xh)[R],
                                            const float (&yh)[R], const float (&zh)[R],
                                            const float (&xl)[R], const float (&yl)[R],
                                            const float (&zl)[R], const float (&mi)[R], float tmi,
                                            float (&hx)[R], float (&hy)[R], float (&hz)[R],
                                            float (&lx)[R], float (&ly)[R], float (&lz)[R],
                                            int &near, const int *__restrict__ ord,
                                            const EncCtx &ec, const float4 (&emi)[R],
                                            const float4 (&eci)[R], unsigned live,
                                            unsigned far = 0u)
{
#pragma unroll 1
    for (int t = 0; t < R; ++t) {
        const bool fart = FAR && !DIAG && ((far >> t) & 1u);
        // the largest widened rc^2 of the wave's targets and of the sub-tile's
        // sources: one compare per pair outside the rare branch
        const float thr = max_nonneg(tmi, wave_max_nonneg(L.b[64 * t + lane].w));
        // targets of this wave that meet sub-tile t in a tile pair the culling kept
        const unsigned livet = ENC ? (live >> (t * R)) & ((1u << R) - 1u) : 0u;
#pragma unroll 1
        for (int half = 0; half < 2; ++half) {
            float tx[R], ty[R], tz[R];
#pragma unroll
            for (int r = 0; r < R; ++r)
                tx[r] = ty[r] = tz[r] = 0.0f;
            // Step k: lane L pairs its targets with source L xor k of sub-tile t,
            // so the lanes of a step touch distinct sources and each lane meets
            // every source once in 64 steps.  The run sum a step reads was
            // written by another lane one step earlier: LDS operations of a
            // wave complete in issue order, and the compiler barrier keeps the
            // read after that write.  Source records are read-only and fetched
            // one step ahead.
            const int k0 = 32 * half;
            const uint32_t a0 = lds_addr(&L.a[0]);
            const uint32_t self = lds_addr(&L.a[64 * t + lane]);
            uint32_t ac = self ^ (uint32_t)(k0 << 4);
            if (fart) {
                // far sub-tile: high parts only, no changeover test, no low
                // records read
                float4 A = lds_ld4(ac);
#pragma unroll 2
                for (int kk = 0; kk < 32; ++kk) {
                    const uint32_t an = self ^ (uint32_t)(((k0 + kk + 1) & 63) << 4);
                    const float4 An = lds_ld4(an);
                    const lds_v3f S = lds_ld3(ac + 32 * T);
                    float jx = S.x, jy = S.y, jz = S.z;
#pragma unroll
                    for (int r = 0; r < R; ++r) {
                        const float dx = A.x - xh[r], dy = A.y - yh[r], dz = A.z - zh[r];
                        const float r2 = fmaf(dz, dz, fmaf(dy, dy, dx * dx));
                        const float y = __builtin_amdgcn_rsqf(r2);
                        const float q = y * (y * y);
                        const float wi = A.w * q, wj = mi[r] * q;
                        tx[r] = fmaf(wi, dx, tx[r]);
                        ty[r] = fmaf(wi, dy, ty[r]);
                        tz[r] = fmaf(wi, dz, tz[r]);
                        jx = fmaf(-wj, dx, jx);
                        jy = fmaf(-wj, dy, jy);
                        jz = fmaf(-wj, dz, jz);
                    }
                    lds_st3(ac + 32 * T, jx, jy, jz);
                    __asm__ __volatile__("" ::: "memory");
                    ac = an;
                    A = An;
                }
            } else {
            float4 A = lds_ld4(ac), B = lds_ld4(ac + 16 * T);
#pragma unroll 2
            for (int kk = 0; kk < 32; ++kk) {
                const uint32_t an = self ^ (uint32_t)(((k0 + kk + 1) & 63) << 4);
                const float4 An = lds_ld4(an), Bn = lds_ld4(an + 16 * T);
                const lds_v3f S = lds_ld3(ac + 32 * T);
                float jx = S.x, jy = S.y, jz = S.z;
                // the R pairs' geometry first, then one branch for the rare
                // ones, so that the R chains share one basic block
                float dxr[R], dyr[R], dzr[R], r2r[R], qr[R];
                bool cand = false;
#pragma unroll
                for (int r = 0; r < R; ++r) {
                    dxr[r] = (A.x - xh[r]) + (B.x - xl[r]);
                    dyr[r] = (A.y - yh[r]) + (B.y - yl[r]);
                    dzr[r] = (A.z - zh[r]) + (B.z - zl[r]);
                    r2r[r] = fmaf(dzr[r], dzr[r], fmaf(dyr[r], dyr[r], dxr[r] * dxr[r]));
                    const float y = __builtin_amdgcn_rsqf(r2r[r]);
                    qr[r] = y * (y * y);
                    const bool on = !DIAG || (64 * r + lane < 64 * t + (lane ^ (k0 + kk)));
                    cand |= r2r[r] < thr && on;
                    if (DIAG)
                        qr[r] = on ? qr[r] : 0.0f;
                }
                // fused encounter test: the relative-chord filter in FP32,
                // |dM|^2 <= 2 (|dc|^2 + (b'_i + b'_j + max(rc_i, rc_j))^2) with
                // the bounds b' widened for the FP32 rounding (padded targets
                // and sources carry NaN midpoints and never pass; every body is
                // big on this path, so no b' carries the small-body sign)
                bool encr[R] = {};
                bool ecand = false;
                if (ENC && livet) {
                    const float4 E = lds_ld4(ac + (uint32_t)sizeof(SymTile32<T>));
                    const float4 F = lds_ld4(ac + (uint32_t)(sizeof(SymTile32<T>) + 16 * T));
#pragma unroll
                    for (int r = 0; r < R; ++r) {
                        const float ex = E.x - emi[r].x, ey = E.y - emi[r].y, ez = E.z - emi[r].z;
                        const float cx = F.x - eci[r].x, cy = F.y - eci[r].y, cz = F.z - eci[r].z;
                        const float D2 = fmaf(ez, ez, fmaf(ey, ey, ex * ex));
                        const float C2 = fmaf(cz, cz, fmaf(cy, cy, cx * cx));
                        const float Sr = (E.w + emi[r].w) + fmaxf(F.w, eci[r].w);
                        const bool on = !DIAG || (64 * r + lane < 64 * t + (lane ^ (k0 + kk)));
                        encr[r] = ((livet >> r) & 1u) && on &&
                                  D2 <= fmaf(Sr, Sr, C2) * (2.0f * (1.0f + 0x1p-18f));
                        ecand |= encr[r];
                    }
                }
                if (cand || ecand) {
#pragma unroll
                    for (int r = 0; r < R; ++r) {
                        const bool on = !DIAG || (64 * r + lane < 64 * t + (lane ^ (k0 + kk)));
                        if (r2r[r] < thr && on) {
                            const ChgPart c = changeover_pair32(r2r[r], B.w, pk, i0, 64 * r + lane,
                                                                ni, j0, (int)((ac - a0) >> 4), T,
                                                                L.ax, qx, qy, qz, m, rc, inner,
                                                                ord);
                            if (c.hit) {
                                add_f64_to_pair(hx[r], lx[r], c.x);
                                add_f64_to_pair(hy[r], ly[r], c.y);
                                add_f64_to_pair(hz[r], lz[r], c.z);
                                qr[r] = 0.0f;
                                ++near;
                            }
                        }
                        if (ENC && encr[r])
                            enc_candidate(ec.srec, ec.dt, ec.keys, ec.cap, ec.ce, ec.stats,
                                          i0 + 64 * r + lane, j0 + (int)((ac - a0) >> 4));
                    }
                }
#pragma unroll
                for (int r = 0; r < R; ++r) {
                    const float dx = dxr[r], dy = dyr[r], dz = dzr[r], q = qr[r];
                    const float wi = A.w * q, wj = mi[r] * q;
                    tx[r] = fmaf(wi, dx, tx[r]);
                    ty[r] = fmaf(wi, dy, ty[r]);
                    tz[r] = fmaf(wi, dz, tz[r]);
                    jx = fmaf(-wj, dx, jx);
                    jy = fmaf(-wj, dy, jy);
                    jz = fmaf(-wj, dz, jz);
                }
                lds_st3(ac + 32 * T, jx, jy, jz);
                __asm__ __volatile__("" ::: "memory");
                ac = an;
                A = An;
                B = Bn;
            }
            }
#pragma unroll
            for (int r = 0; r < R; ++r) {
                two_sum_f(hx[r], lx[r], tx[r]);
                two_sum_f(hy[r], ly[r], ty[r]);
                two_sum_f(hz[r], lz[r], tz[r]);
            }
            // end of the run: every source of sub-tile t had its 32 steps; lane
            // L moves source 64 t + L's run sum into its FP64 total
            const int js = 64 * t + lane;
            const float4 S = L.run[js];
            L.ax[js] += (double)S.x;
            L.ay[js] += (double)S.y;
            L.az[js] += (double)S.z;
            L.run[js] = make_float4(0.0f, 0.0f, 0.0f, 0.0f);
            __asm__ __volatile__("" ::: "memory");
        }
    }
}

// Tile J of one wave for the FP32C loop with the source run sums in registers
// (R <= 2), as SymTile64R: records twice over, FP64 totals in C copies.
template <int R, int C>
struct alignas(512) SymTile32R {
    struct Sub {
        float4 a[128];              // hi parts and mass
        float4 b[128];              // lo parts and widened rc^2
    } s[R];
    double tot[C][3][64 * R];
};

template <int R, int C>
__device__ __forceinline__ void put_src32(SymTile32R<R, C> &S, int e, float4 a, float4 b)
{
    typename SymTile32R<R, C>::Sub &U = S.s[e / 64];
    const int j = e % 64;
    U.a[j] = U.a[j + 64] = a;
    U.b[j] = U.b[j + 64] = b;
#pragma unroll
    for (int c = 0; c < C; ++c)
        S.tot[c][0][e] = S.tot[c][1][e] = S.tot[c][2][e] = 0.0;
}

template <int T>
__device__ __forceinline__ void put_src32(SymTile32<T> &S, int e, float4 a, float4 b)
{
    S.a[e] = a;
    S.b[e] = b;
    S.run[e] = make_float4(0.0f, 0.0f, 0.0f, 0.0f);
    S.ax[e] = S.ay[e] = S.az[e] = 0.0;
}

template <int R, int C>
__device__ __forceinline__ double src_total(const SymTile32R<R, C> &S, int c, int e)
{
    double v = S.tot[0][c][e];
#pragma unroll
    for (int k = 1; k < C; ++k)
        v += S.tot[k][c][e];
    return v;
}

template <int T>
__device__ __forceinline__ double src_total(const SymTile32<T> &S, int c, int e)
{
    return c == 0 ? S.ax[e] : (c == 1 ? S.ay[e] : S.az[e]);
}

// A float moved one lane up the wave: lane L gets lane (L - 1) mod 64's value.
__device__ __forceinline__ float wave_rotr1(float v)
{
    return __int_as_float(__builtin_amdgcn_mov_dpp(__float_as_int(v), 0x13C, 0xF, 0xF, false));
}

// The tile pair of sym_tile32c with the sources' run sums in registers, as in
// sym_tile64_rot but downwards: in step k lane L meets source (L - k) mod 64 (entry
// 64 + L - k), and the sums move one lane up.  Over the radial order a close pair's
// bodies are few positions apart, the source behind the target, and so meet in the
// last steps: large terms at the end of a run lose the least (upwards the error of
// the bodies in close pairs is a sixth larger).
template <int R, bool DIAG, bool FAR, int H, int C>
__device__ __forceinline__ void sym_tile32c_rot(
    SymTile32R<R, C> &L, const SymPart<R, H> &part, int lane, int i0, int ni, int j0, int nj,
    double inner, const float4 *__restrict__ pk, const double *__restrict__ qx,
    const double *__restrict__ qy, const double *__restrict__ qz, const double *__restrict__ m,
    const double *__restrict__ rc, const float (&xh)[R], const float (&yh)[R], const float (&zh)[R],
    const float (&xl)[R], const float (&yl)[R], const float (&zl)[R], const float (&mi)[R],
    float tmi, float (&hx)[R], float (&hy)[R], float (&hz)[R], float (&lx)[R], float (&ly)[R],
    float (&lz)[R], int &near, const int *__restrict__ ord, unsigned far)
{
    constexpr int kRun = SymPart<R, H>::kSteps < 32 ? SymPart<R, H>::kSteps : 32;
    double(&tot)[3][64 * R] = L.tot[part.c];
#pragma unroll 1
    for (int t = part.t0; t < part.t1 && 64 * t < nj; ++t) {
        const bool fart = FAR && !DIAG && ((far >> t) & 1u);
        const float thr = max_nonneg(tmi, wave_max_nonneg(L.s[t].b[lane].w));
#pragma unroll 1
        for (int k0 = part.k0; k0 < part.k0 + SymPart<R, H>::kSteps; k0 += kRun) {
            float tx[R], ty[R], tz[R];
#pragma unroll
            for (int r = 0; r < R; ++r)
                tx[r] = ty[r] = tz[r] = 0.0f;
            float jx = 0.0f, jy = 0.0f, jz = 0.0f;
            // LDS address of a[64 + lane - k0] of sub-tile t; its b record 16 * 128 on
            uint32_t ac = lds_addr(&L.s[t].a[64 + lane - k0]);
            if (fart) {
                float4 A = lds_ld4(ac);
#pragma unroll 4
                for (int kk = 0; kk < kRun; ++kk) {
                    ac -= 16;
                    const float4 An = lds_ld4(ac);
#pragma unroll
                    for (int r = 0; r < R; ++r) {
                        const float dx = A.x - xh[r], dy = A.y - yh[r], dz = A.z - zh[r];
                        const float r2 = fmaf(dz, dz, fmaf(dy, dy, dx * dx));
                        const float y = __builtin_amdgcn_rsqf(r2);
                        const float q = y * (y * y);
                        const float wi = A.w * q, wj = mi[r] * q;
                        tx[r] = fmaf(wi, dx, tx[r]);
                        ty[r] = fmaf(wi, dy, ty[r]);
                        tz[r] = fmaf(wi, dz, tz[r]);
                        jx = fmaf(-wj, dx, jx);
                        jy = fmaf(-wj, dy, jy);
                        jz = fmaf(-wj, dz, jz);
                    }
                    jx = wave_rotr1(jx);
                    jy = wave_rotr1(jy);
                    jz = wave_rotr1(jz);
                    A = An;
                }
            } else {
                float4 A = lds_ld4(ac), B = lds_ld4(ac + 16 * 128);
#pragma unroll 2
                for (int kk = 0; kk < kRun; ++kk) {
                    ac -= 16;
                    const float4 An = lds_ld4(ac), Bn = lds_ld4(ac + 16 * 128);
                    // the R pairs' geometry first, then one branch for the rare
                    // ones, so that the R chains share one basic block
                    float dxr[R], dyr[R], dzr[R], r2r[R], qr[R];
                    bool cand = false;
#pragma unroll
                    for (int r = 0; r < R; ++r) {
                        dxr[r] = (A.x - xh[r]) + (B.x - xl[r]);
                        dyr[r] = (A.y - yh[r]) + (B.y - yl[r]);
                        dzr[r] = (A.z - zh[r]) + (B.z - zl[r]);
                        r2r[r] = fmaf(dzr[r], dzr[r], fmaf(dyr[r], dyr[r], dxr[r] * dxr[r]));
                        const float y = __builtin_amdgcn_rsqf(r2r[r]);
                        qr[r] = y * (y * y);
                        const bool on = !DIAG || (64 * r + lane < 64 * t + ((lane - k0 - kk) & 63));
                        cand |= r2r[r] < thr && on;
                        if (DIAG)
                            qr[r] = on ? qr[r] : 0.0f;
                    }
                    if (cand) {
                        const int sj = 64 * t + ((lane - k0 - kk) & 63);
#pragma unroll
                        for (int r = 0; r < R; ++r) {
                            const bool on = !DIAG || 64 * r + lane < sj;
                            if (r2r[r] < thr && on) {
                                const ChgPart c = changeover_pair32(
                                    r2r[r], B.w, pk, i0, 64 * r + lane, ni, j0, sj, 64 * R,
                                    &tot[0][0], qx, qy, qz, m, rc, inner, ord);
                                if (c.hit) {
                                    add_f64_to_pair(hx[r], lx[r], c.x);
                                    add_f64_to_pair(hy[r], ly[r], c.y);
                                    add_f64_to_pair(hz[r], lz[r], c.z);
                                    qr[r] = 0.0f;
                                    ++near;
                                }
                            }
                        }
                    }
#pragma unroll
                    for (int r = 0; r < R; ++r) {
                        const float dx = dxr[r], dy = dyr[r], dz = dzr[r], q = qr[r];
                        const float wi = A.w * q, wj = mi[r] * q;
                        tx[r] = fmaf(wi, dx, tx[r]);
                        ty[r] = fmaf(wi, dy, ty[r]);
                        tz[r] = fmaf(wi, dz, tz[r]);
                        jx = fmaf(-wj, dx, jx);
                        jy = fmaf(-wj, dy, jy);
                        jz = fmaf(-wj, dz, jz);
                    }
                    jx = wave_rotr1(jx);
                    jy = wave_rotr1(jy);
                    jz = wave_rotr1(jz);
                    A = An;
                    B = Bn;
                }
            }
#pragma unroll
            for (int r = 0; r < R; ++r) {
                two_sum_f(hx[r], lx[r], tx[r]);
                two_sum_f(hy[r], ly[r], ty[r]);
                two_sum_f(hz[r], lz[r], tz[r]);
            }
            // the sums in this lane are now those of the source it would meet next
            const int js = 64 * t + ((lane - k0 - kRun) & 63);
            tot[0][js] += (double)jx;
            tot[1][js] += (double)jy;
            tot[2][js] += (double)jz;
        }
    }
}

template <int R, bool DIAG, int T, bool FAR, int H, int C, class... A>
__device__ __forceinline__ void sym_round32(SymTile32R<R, C> &L, const SymPart<R, H> &part, int lane,
                                            int i0, int ni, int j0, int nj, unsigned far, A &&...a)
{
    sym_tile32c_rot<R, DIAG, FAR>(L, part, lane, i0, ni, j0, nj, a..., far);
}

template <int R, bool DIAG, int T, bool FAR, int H, class... A>
__device__ __forceinline__ void sym_round32(SymTile32<T> &L, const SymPart<R, H> &, int lane, int i0,
                                            int ni, int j0, int, unsigned far, A &&...a)
{
    const EncCtx noenc{};
    float4 noem[R];
    sym_tile32c<R, DIAG, T, false, FAR>(L, lane, i0, ni, j0, a..., noenc, noem, noem, 0u, far);
}

// Two 64-body tiles of the radial order are far apart for the FP32C pair loop
// when the gap between their shells, |xh_i| in [rmin, rmax] (records written
// by k_sun_drift with the FP32C records), exceeds 2^21 times the sum of their low parts' largest norms
// and its square exceeds both largest widened rc^2.  Then for i in one and j in
// the other |xh_j - xh_i| >= gap: dropping the low parts moves the pair's
// difference by at most 2^-21 of its length, and the pair lies outside the
// changeover zone (weight 1, no rare branch).  Margins of 2^-20 and 2^-18 cover
// the FP32 rounding of the test itself.
__device__ __forceinline__ bool far_tiles(float4 a, float4 b)
{
    const float gap = fmaxf(b.x - a.y, a.x - b.y) * (1.0f - 0x1p-20f);
    return gap >= 0x1p21f * (a.z + b.z) * (1.0f + 0x1p-20f) &&
           gap * gap >= fmaxf(a.w, b.w) * (1.0f + 0x1p-18f);
}

// SORT: the positions of the work items are positions of the radial order
// (ord: position -> body), whose tile bounds rtb (system s's tiles from
// rtf[s], 64 positions each from off[s]) mark the far sub-tile pairs.
// REG: the sources' run sums in registers, else in LDS.  In registers the loop is bound
// by the vector ALU alone, in LDS by both; but the far tile pairs of the radial order,
// whose steps are short, bear the moves between lanes worse than the LDS.  So wider
// workgroups over the radial order keep LDS.  The kernel / a step, registers against LDS,
// disk of 0.5-5 AU: 33000 bodies (workgroups of two) 324.8 / 289.7 us and 372.7 / 342.0 us, 65000
// 1147 / 1028 and 1272 / 1143, 131072 (of four) 4369 / 4109 and 4608 / 4313; a dense ring of
// 33000 341 / 340 and 397.3 / 396.3, of 131072 4656 / 4901 and 4989 / 5255.  (One wave per tile
// pair, 16384 bodies: 84.1 / 78.2 us, but a call of eight steps 989 / 1021 us.)
template <int R, int G, bool SORT = false, int H = 1, bool REG = (R <= 2 && !(SORT && G > 1))>
__global__ __launch_bounds__(64 * G * H, R == 4 ? 2 : 3) void k_force32c_sym(const FWork *__restrict__ work, int nitems,
                                                         const float4 *__restrict__ pk,
                                                         const double *__restrict__ qx,
                                                         const double *__restrict__ qy,
                                                         const double *__restrict__ qz,
                                                         const double *__restrict__ m,
                                                         const double *__restrict__ rc,
                                                         float *__restrict__ fpart, int ntot,
                                                         int maxs, double inner, DevStats *stats,
                                                         const int *__restrict__ ord = nullptr,
                                                         const float4 *__restrict__ rtb = nullptr,
                                                         const int *__restrict__ rtf = nullptr,
                                                         const int *__restrict__ off = nullptr)
{
    constexpr int T = 64 * R;
    static_assert(H == 1 || (G == 1 && REG), "only single tile pairs are shared");
    static_assert(!REG || R <= 2, "the register form's tiles");
    using Tile = typename std::conditional<REG, SymTile32R<R, SymPart<R, H>::kCopies>, SymTile32<T>>::type;
    __shared__ Tile tl[G];
    // H > 1: the waves' sums of the targets
    __shared__ double tgt[H > 1 ? H : 1][3][H > 1 ? T : 1];
    const int lane = threadIdx.x & 63, wv = H > 1 ? 0 : threadIdx.x >> 6;
    const int wh = threadIdx.x >> 6;
    const SymPart<R, H> part(H > 1 ? wh : 0);
    const size_t plane = (size_t)maxs * ntot;
    int near = 0;
    for (int it = blockIdx.x; it < nitems; it += gridDim.x) {
        const FWork wk = work[it];
        const bool diag = wk.i0 == wk.j0;
        // the G source tiles of super-tile J (nj real records from j0)
        for (int k = threadIdx.x; k < G * T; k += 64 * G * H) {
            // sources past the end: massless and far away (r^2 ~ 1e36, so the
            // weight underflows to 0 instead of meeting a target at r = 0)
            float4 A = make_float4(1e18f, 1e18f, 1e18f, 0.0f), B = make_float4(0.0f, 0.0f, 0.0f, 0.0f);
            if (k < wk.nj) {
                const int b = SORT ? ord[wk.j0 + k] : wk.j0 + k;
                A = pk[2 * (size_t)b];
                B = pk[2 * (size_t)b + 1];
            }
            put_src32(tl[k / T], k % T, A, B);
        }
        __syncthreads();
        // this wave's target tile: tni bodies from ti0 (none when tni <= 0)
        const int ti0 = wk.i0 + wv * T;
        const int tni = min(T, wk.ni - wv * T);
        float xh[R], yh[R], zh[R], xl[R], yl[R], zl[R], mi[R];
        float hx[R], hy[R], hz[R], lx[R], ly[R], lz[R];
        float tmi = 0.0f;
#pragma unroll
        for (int r = 0; r < R; ++r) {
            const int li = 64 * r + lane;
            const bool ok = li < tni;
            const int i = SORT ? ord[ok ? ti0 + li : wk.i0] : (ok ? ti0 + li : wk.i0);
            const float4 A = pk[2 * (size_t)i], B = pk[2 * (size_t)i + 1];
            xh[r] = A.x; yh[r] = A.y; zh[r] = A.z;
            xl[r] = B.x; yl[r] = B.y; zl[r] = B.z;
            // targets past the tile end are massless: they add nothing to the sources
            mi[r] = ok ? A.w : 0.0f;
            tmi = max_nonneg(tmi, B.w);
            hx[r] = hy[r] = hz[r] = lx[r] = ly[r] = lz[r] = 0.0f;
        }
        tmi = wave_max_nonneg(tmi);
        // Round k: wave w pairs its target tile with source tile (w + k) mod G, so
        // that the waves of a round update distinct source tiles.  Off the
        // diagonal G rounds cover the G x G tile pairs.  On the diagonal (I = J)
        // round 0 takes the pairs inside each tile, rounds 1 .. G/2 - 1 every
        // other tile pair once, and round G/2 (even G) only its first G/2 waves,
        // whose partners the other half would meet again.
        const int nr = diag ? G / 2 + 1 : G;
        for (int k = 0; k < nr; ++k) {
            const int s = (wv + k) % G;
            const bool go = tni > 0 && s * T < wk.nj && !(diag && 2 * k == G && wv >= G / 2);
            if (go) {
                if (diag && k == 0) {
                    sym_round32<R, true, T, false>(tl[s], part, lane, ti0, tni, wk.j0 + s * T,
                                                   wk.nj - s * T, 0u, inner, pk, qx, qy, qz, m, rc,
                                                   xh, yh, zh, xl, yl, zl, mi, tmi, hx, hy, hz, lx,
                                                   ly, lz, near, SORT ? ord : nullptr);
                } else {
                    // far source sub-tiles (radial order, no padded targets)
                    unsigned far = 0u;
                    if (SORT && tni == T) {
                        const int tb0 = rtf[wk.sys], o = off[wk.sys], sj0 = wk.j0 + s * T;
#pragma unroll
                        for (int t = 0; t < R; ++t) {
                            if (s * T + 64 * t >= wk.nj)
                                continue;
                            const float4 Bt = rtb[tb0 + (sj0 + 64 * t - o) / 64];
                            bool f = true;
#pragma unroll
                            for (int r = 0; r < R; ++r)
                                f = f && far_tiles(rtb[tb0 + (ti0 + 64 * r - o) / 64], Bt);
                            far |= f ? 1u << t : 0u;
                        }
                    }
                    sym_round32<R, false, T, SORT>(tl[s], part, lane, ti0, tni, wk.j0 + s * T,
                                                   wk.nj - s * T, far, inner, pk, qx, qy, qz, m,
                                                   rc, xh, yh, zh, xl, yl, zl, mi, tmi, hx, hy, hz,
                                                   lx, ly, lz, near, SORT ? ord : nullptr);
                }
            }
            __syncthreads();
        }
        // super-tile I's sums to slot J (on the diagonal together with the same
        // bodies' sums as sources)
#pragma unroll
        for (int r = 0; r < R; ++r) {
            const int li = 64 * r + lane;
            if (li < tni) {
                const int i = ti0 + li;
                double sx_ = (double)hx[r] + (double)lx[r];
                double sy_ = (double)hy[r] + (double)ly[r];
                double sz_ = (double)hz[r] + (double)lz[r];
                if (H > 1) {
                    tgt[wh % H][0][li] = sx_;
                    tgt[wh % H][1][li] = sy_;
                    tgt[wh % H][2][li] = sz_;
                    continue;
                }
                if (diag) {
                    sx_ += src_total(tl[wv], 0, li);
                    sy_ += src_total(tl[wv], 1, li);
                    sz_ += src_total(tl[wv], 2, li);
                }
                fpart[(size_t)wk.slot * ntot + i] = (float)sx_;
                fpart[plane + (size_t)wk.slot * ntot + i] = (float)sy_;
                fpart[2 * plane + (size_t)wk.slot * ntot + i] = (float)sz_;
            }
        }
        if (H > 1) {
            // the waves' sums in wave order
            __syncthreads();
            for (int e = threadIdx.x; e < tni; e += 64 * H)
#pragma unroll
                for (int c = 0; c < 3; ++c) {
                    double v = tgt[0][c][e];
#pragma unroll
                    for (int h = 1; h < H; ++h)
                        v += tgt[h][c][e];
                    if (diag)
                        v += src_total(tl[0], c, e);
                    fpart[c * plane + (size_t)wk.slot * ntot + ti0 + e] = (float)v;
                }
        }
        if (!diag) {
            // super-tile J's sums to slot I
            for (int k = threadIdx.x; k < wk.nj; k += 64 * G * H) {
                const Tile &S = tl[k / T];
                const int e = k % T, j = wk.j0 + k;
                fpart[((size_t)0 * maxs + wk.pad) * ntot + j] = (float)src_total(S, 0, e);
                fpart[((size_t)1 * maxs + wk.pad) * ntot + j] = (float)src_total(S, 1, e);
                fpart[((size_t)2 * maxs + wk.pad) * ntot + j] = (float)src_total(S, 2, e);
            }
        }
        __syncthreads();
    }
    for (int o = 32; o > 0; o >>= 1)
        near += __shfl_xor(near, o);
    if (lane == 0 && near)
        atomicAdd((unsigned long long *)&stats->near_pairs, (unsigned long long)near);
}

// a = G * sum over the body's split partials (fixed order); optionally `kicks`
// (1 or 2) kicks V += h a, rounded as that many k_kick launches.  A workgroup of
// kFinThreads threads takes B = kFinThreads / nsl bodies: thread group g (B
// threads) reads slice g of every body's partials (slots [g ns / nsl, (g + 1) ns
// / nsl) in order, eight loads in flight per lane), and the slice sums are added
// in slice order.  nsl (a power of two, at most 16) follows the largest split
// count, so that few-split systems do not leave most threads idle.  The sums of
// m V are not needed after it: the next S(h) takes the momentum from before the
// kicks.
constexpr int kFinThreads = 1024;

template <typename P>
__global__ __launch_bounds__(kFinThreads) void k_force_finalize(
    const int *__restrict__ sys_of, const int *__restrict__ nsplit, const P *__restrict__ fpart,
    int ntot, int maxs, int ns_all, int nsl, double G, double *__restrict__ ax,
    double *__restrict__ ay, double *__restrict__ az, double h, int kicks, double *vx, double *vy,
    double *vz, const int *__restrict__ ord, int count_cap, DevStats *stats)
{
    __shared__ double gs[3 * kFinThreads];
    // count_cap >= 0: also the encounter list's statistics (as k_enc_count), for
    // the check that ran inside the force pass before this launch
    if (count_cap >= 0 && blockIdx.x == 0 && threadIdx.x == 0) {
        const int count = stats->cur_nce;
        stats->total_nce += count;
        if (count > stats->max_nce)
            stats->max_nce = count;
        if (count > count_cap)
            stats->overflow_steps += 1;
    }
    const int B = kFinThreads / nsl;
    const int t = threadIdx.x % B, g = threadIdx.x / B;
    // i: the partials' position; bi: the body (the sorted order maps them)
    const int i = blockIdx.x * B + t;
    const int bi = ord && i < ntot ? ord[i] : i;
    double s0 = 0.0, s1 = 0.0, s2 = 0.0;
    // the velocities to kick, fetched while the partials load
    double v0 = 0.0, v1 = 0.0, v2 = 0.0;
    if (g == 0 && i < ntot && h != 0.0) {
        v0 = vx[bi];
        v1 = vy[bi];
        v2 = vz[bi];
    }
    if (i < ntot) {
        // ns_all != 0: every system has that split count
        const int ns = ns_all ? ns_all : nsplit[sys_of[i]];
        const int k0 = g * ns / nsl, k1 = (g + 1) * ns / nsl;
        sum_slots(fpart, ntot, maxs, i, k0, k1, s0, s1, s2);
    }
    if (g > 0) {
        double *o = gs + (size_t)(g - 1) * 3 * B;
        o[t] = s0;
        o[B + t] = s1;
        o[2 * B + t] = s2;
    }
    __syncthreads();
    if (g == 0 && i < ntot) {
        for (int q = 0; q < nsl - 1; ++q) {
            const double *o = gs + (size_t)q * 3 * B;
            s0 += o[t];
            s1 += o[B + t];
            s2 += o[2 * B + t];
        }
        s0 *= G;
        s1 *= G;
        s2 *= G;
        ax[bi] = s0;
        ay[bi] = s1;
        az[bi] = s2;
        if (h != 0.0) {
            double u0 = fma(h, s0, v0), u1 = fma(h, s1, v1), u2 = fma(h, s2, v2);
            if (kicks == 2) {
                u0 = fma(h, s0, u0);
                u1 = fma(h, s1, u1);
                u2 = fma(h, s2, u2);
            }
            vx[bi] = u0;
            vy[bi] = u1;
            vz[bi] = u2;
        }
    }
}

// ----------------------------------------------------------------------------
// Encounter check (Sec. 3.1, encounter block): every pair i<j of a system
// whose minimum separation over the step is <= rc_ij = max(rc_i, rc_j).  The
// squared separation over s in [0,1] is taken as the cubic Hermite through
// f0 = |dQ0|^2, f1 = |dQ1|^2 with slopes g0 = 2 dt dQ0.dV0, g1 = 2 dt dQ1.dV1.
// Its minimum is bounded below by min(f0,f1) - 4/27 (max(0,-g0) + max(0,g1)),
// which serves as a cheap conservative filter before the exact minimum.
// ----------------------------------------------------------------------------
__device__ double hermite_min(double f0, double f1, double g0, double g1)
{
    double b = 3.0 * (f1 - f0) - 2.0 * g0 - g1;   // s^2 coefficient
    double c = 2.0 * (f0 - f1) + g0 + g1;         // s^3 coefficient
    double best = fmin(f0, f1);
    // f'(s) = g0 + 2 b s + 3 c s^2
    double A = 3.0 * c, B = 2.0 * b, C = g0;
    double s1 = -1.0, s2 = -1.0;
    if (A != 0.0) {
        double disc = B * B - 4.0 * A * C;
        if (disc >= 0.0) {
            double q = -0.5 * (B + copysign(sqrt(disc), B));
            if (q != 0.0) {
                s1 = q / A;
                s2 = C / q;
            }
        }
    } else if (B != 0.0) {
        s1 = -C / B;
    }
    if (s1 > 0.0 && s1 < 1.0)
        best = fmin(best, f0 + s1 * (g0 + s1 * (b + s1 * c)));
    if (s2 > 0.0 && s2 < 1.0)
        best = fmin(best, f0 + s2 * (g0 + s2 * (b + s2 * c)));
    return fmax(best, 0.0);
}

// The exact test's fields of one record.
struct HRec {
    double q0[3], v0[3], q1[3], v1[3];
    double rc;
    int body;
};

// Exact encounter test of a pair (the Hermite bound, then the minimum over the
// step).  J: an HRec or a sorted record.
template <typename R>
__device__ __forceinline__ bool enc_hit(const HRec &I, const R &J, double dt)
{
    const double t2 = 2.0 * dt, k427 = 4.0 / 27.0;
    const double d0x = J.q0[0] - I.q0[0], d0y = J.q0[1] - I.q0[1], d0z = J.q0[2] - I.q0[2];
    const double d1x = J.q1[0] - I.q1[0], d1y = J.q1[1] - I.q1[1], d1z = J.q1[2] - I.q1[2];
    const double e0x = J.v0[0] - I.v0[0], e0y = J.v0[1] - I.v0[1], e0z = J.v0[2] - I.v0[2];
    const double e1x = J.v1[0] - I.v1[0], e1y = J.v1[1] - I.v1[1], e1z = J.v1[2] - I.v1[2];
    const double f0 = fma(d0z, d0z, fma(d0y, d0y, d0x * d0x));
    const double f1 = fma(d1z, d1z, fma(d1y, d1y, d1x * d1x));
    const double g0 = t2 * fma(d0z, e0z, fma(d0y, e0y, d0x * e0x));
    const double g1 = t2 * fma(d1z, e1z, fma(d1y, e1y, d1x * e1x));
    const double lower = fmin(f0, f1) - k427 * (fmax(0.0, -g0) + fmax(0.0, g1));
    const double rcij = fmax(I.rc, J.rc);
    const double thr = rcij * rcij;
    if (!(lower <= thr * (1.0 + 1e-6) + 1e-15 * (f0 + f1 + fabs(g0) + fabs(g1))))
        return false;
    return hermite_min(f0, f1, g0, g1) <= thr;
}

// A body's flag.  Stored only where it is not there yet: the stores of many pairs to
// one body's flag (embryos among many small bodies) take turns, about 10 ns each.
__device__ __forceinline__ void enc_mark(int *ce, int body, int tag)
{
    if (__hip_atomic_load(&ce[body], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP) != tag)
        __hip_atomic_store(&ce[body], tag, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

// The test and the append of a flagged pair (nce: the list's count; tag: the flag
// written to both bodies).
template <typename R>
__device__ __forceinline__ void enc_exact(const HRec &I, const R &J, double dt,
                                          unsigned long long *keys, int cap, int *ce, int *nce,
                                          int tag = kEncFlag)
{
    if (!enc_hit(I, J, dt))
        return;
    const int pos = atomicAdd(nce, 1);
    const int bi = I.body, bj = J.body;
    const unsigned lo = (unsigned)min(bi, bj), hi = (unsigned)max(bi, bj);
    if (pos < cap)
        keys[pos] = ((unsigned long long)lo << 32) | hi;
    enc_mark(ce, bi, tag);
    enc_mark(ce, bj, tag);
}

// The drift outputs the exact test reads, by body.
struct EncIn {
    const double *q0x, *q0y, *q0z, *v0x, *v0y, *v0z, *q1x, *q1y, *q1z, *v1x, *v1y, *v1z, *rc;
};

__device__ __forceinline__ HRec enc_load(const EncIn &E, int i)
{
    HRec r;
    r.q0[0] = E.q0x[i]; r.q0[1] = E.q0y[i]; r.q0[2] = E.q0z[i];
    r.v0[0] = E.v0x[i]; r.v0[1] = E.v0y[i]; r.v0[2] = E.v0z[i];
    r.q1[0] = E.q1x[i]; r.q1[1] = E.q1y[i]; r.q1[2] = E.q1z[i];
    r.v1[0] = E.v1x[i]; r.v1[1] = E.v1y[i]; r.v1[2] = E.v1z[i];
    r.rc = E.rc[i];
    r.body = i;
    return r;
}

// The exact test's bound in FP32 (k_enc_direct, where its filter keeps most pairs): the
// record in units of the system's scale, the velocities times 2 dt.  A pair the exact
// test's bound passes is never dropped: with u = 2^-24 the differences carry 2u (|x_i| +
// |x_j|), so f0, f1 an error of 14u (|Q_i|^2 + |Q_j|^2), g0, g1 of 14u (|Q|^2 + dt^2 |V|^2
// summed over both bodies), and the bound with its own rounding less than 32u of both
// bodies' |Q0|^2 + |Q1|^2 + dt^2 (|V0|^2 + |V1|^2): slack takes twice that.  rc is widened by 2^-18
// for its rounding and the exact test's own margin.
struct alignas(16) EncF {
    float q0[3], q1[3], v0[3], v1[3], rc, slack, pad[2];
};

__device__ __forceinline__ EncF enc_load32(const EncIn &E, int i, double dt, double inv_l)
{
    const HRec R = enc_load(E, i);
    EncF r;
    double w = 0.0;
#pragma unroll
    for (int k = 0; k < 3; ++k) {
        const double a = inv_l * R.q0[k], b = inv_l * R.q1[k], c = inv_l * dt * R.v0[k],
                     d = inv_l * dt * R.v1[k];
        r.q0[k] = (float)a;
        r.q1[k] = (float)b;
        r.v0[k] = (float)(2.0 * c);
        r.v1[k] = (float)(2.0 * d);
        w += a * a + b * b + c * c + d * d;
    }
    r.rc = (float)(inv_l * R.rc * (1.0 + 0x1p-18));
    r.slack = (float)(w * (0x1p-18 * (1.0 + 0x1p-20)));
    return r;
}

__device__ __forceinline__ bool enc_bound32(const EncF &I, const EncF &J)
{
    float f0 = 0.0f, f1 = 0.0f, g0 = 0.0f, g1 = 0.0f;
#pragma unroll
    for (int k = 0; k < 3; ++k) {
        const float a = J.q0[k] - I.q0[k], b = J.q1[k] - I.q1[k];
        f0 = fmaf(a, a, f0);
        f1 = fmaf(b, b, f1);
        g0 = fmaf(a, J.v0[k] - I.v0[k], g0);
        g1 = fmaf(b, J.v1[k] - I.v1[k], g1);
    }
    const float lower = fmaf(-4.0f / 27.0f, fmaxf(0.0f, -g0) + fmaxf(0.0f, g1), fminf(f0, f1));
    const float rc = fmaxf(I.rc, J.rc);
    // (a value that is not finite goes to the exact test)
    return !(lower > fmaf(rc, rc, I.slack + J.slack));
}

// Direct check of every pair i < j with a big member (i big): the filter of enc_record as
// a product of matrices, then the exact test of the pairs it keeps.
//
// A pair whose chord midpoints are further apart than its relative chord, 3/4 E and rc_ij
// together cannot be flagged (kEncP, A).  Bodies moving together (neighbours on similar orbits) have short relative
// chords and share their fall toward the star, so this keeps few pairs also when
// steps are long: 3.7e-5 of the pairs of 20011 bodies at 0.9-1.1 AU and steps of 0.04
// yr, as many of a 1-3 AU disk and 0.05 yr (with the sum of both bodies' largest
// deviations for E 1.1e-2 and 4.5e-4: the check alone 57 -> 23 us, and of 256 systems
// of 200-4000 bodies 104 -> 66 us).
//
// A wave owns a work item of up to 128 targets (eight groups of 16, the columns of
// its matrix products, held in registers) and its sources, 16 at a time (the
// rows, one 16-byte load per lane): eight 16x16x32 products test 2048 pairs, and
// the OR of their signs tells whether any is a candidate.  The FP32 pair test this
// replaces issued 17 operations per 64 pairs, this one about one and a half;
// candidates queue in LDS and take the exact test 64 at a time.
// Bound by the matrix products (128 of about 200 cycles per 2048 pairs); with few
// items, by the latency of the row loads.  The kernel: 100 bodies 22 -> 5.0 us, 16384
// bodies in 0.5-5 AU 14.4 us; the whole check at 1001 bodies 40 -> 10 us (nine launches
// before).
// With steps of most of a radian the relative chords are as long as the distances and
// the filter keeps most pairs.  A group of 16 rows where half of the lanes keep kEncDense
// or more of their 32 pairs waits for the end of the loop, where the targets are
// taken into registers and the group's sources into LDS and every pair meets the Hermite bound
// in FP32 (enc_bound32), which keeps few.  Every pair so costs about as much as one in
// twenty through the queue: a 0.9-1.1 AU ring of 9990 bodies and steps of 0.16 yr 73 us,
// by the queue alone 605 us, in the sorted check 220 us.
constexpr int kEncDense = 2;
__global__ __launch_bounds__(64, 3) void k_enc_direct(const PWork *__restrict__ work,
                                                   const v8h *__restrict__ eq, EncIn in, double dt,
                                                   unsigned long long *__restrict__ keys, int cap,
                                                   int *__restrict__ ce, int *__restrict__ nce,
                                                   int tag,
                                                   const unsigned long long *__restrict__ scale,
                                                   const int *__restrict__ sys_of)
{
    constexpr int NG = kEncTargets / 16;
    __shared__ int qe[128];
    // 16 sources of a group of many candidates
    __shared__ EncF sj[16];
    const PWork wk = work[blockIdx.x];
    const int lane = threadIdx.x, q = lane >> 4, r = lane & 15;
    // K slots 8q .. 8q + 7, rows against columns (g as in enc_record): q = 0 the high
    // parts, s' and the row's al_hi; q = 1 the rows' high and the columns' low parts; q = 2
    // the rows' low parts and al_lo and the columns' high parts; q = 3 d' and the
    // column's al
    const _Float16 one = (_Float16)(float)(1.0 / kEncAlUnit), zero = (_Float16)0.0f;
    const _Float16 g0 = (_Float16)(q == 3 ? 4.0f : -2.0f);
    const v8h g = {g0, g0, g0, (_Float16)4.0f, (_Float16)4.0f, (_Float16)4.0f, (_Float16)-4.0f, zero};
    const int cpart = q == 0 || q == 2 ? 0 : (q == 1 ? 1 : 2);
    const int rpart = q < 2 ? 0 : q - 1;
    int qn = 0;
    auto drain = [&](int n) {
        wave_lds_sync();
        if (lane < n) {
            const int e = qe[lane];
            const HRec I = enc_load(in, wk.i0 + (e & 255));
            enc_exact(I, enc_load(in, wk.j0 + (e >> 8)), dt, keys, cap, ce, nce, tag);
        }
    };
    // lanes' candidates (target i0 + ti, source j0 + sj) to the queue
    auto push = [&](bool cand, int ti, int sj) {
        const unsigned long long mk = __builtin_amdgcn_ballot_w64(cand);
        if (!mk)
            return;
        if (cand)
            qe[qn + __popcll(mk & ((1ull << lane) - 1ull))] = ti | (sj << 8);
        qn += __popcll(mk);
        if (qn >= 64) {
            drain(64);
            const int rest = qn - 64;
            const int e = lane < rest ? qe[64 + lane] : 0;
            wave_lds_sync();
            if (lane < rest)
                qe[lane] = e;
            qn = rest;
        }
    };
    v8h col[NG];
#pragma unroll
    for (int k = 0; k < NG; ++k) {
        const bool ok = 16 * k + r < wk.ni;
        const v8h raw = eq[kEncRec * (size_t)(wk.i0 + (ok ? 16 * k + r : 0)) + cpart];
        v8h c = raw * g;
        c[6] = q == 0 ? c[6] : (q == 2 ? one : zero);
        c[7] = q == 0 ? one : zero;
        c[3] = q == 3 ? raw[5] : c[3];
        c[4] = q == 3 ? raw[6] : c[4];
        c[5] = q == 3 ? zero : c[5];
        // columns past the targets: a large positive al and nothing else, so that
        // they never go below zero
        col[k] = c;
        if (!ok) {
            col[k] = v8h{};
            col[k][3] = q == 3 ? (_Float16)60000.0f : zero;
        }
    }
    auto rows = [&](int s) {
        return eq[kEncRec * (size_t)(wk.j0 + min(s + r, wk.nj - 1)) + rpart];
    };
    // the groups of many candidates, for after the loop (a work item has at most 64)
    unsigned long long dense = 0ull;
    // rows loaded two groups ahead
    v8h row = rows(0), next = rows(16);
    for (int s = 0; s < wk.nj; s += 16) {
        const v8h after = rows(s + 32);
        v4f f[NG];
#pragma unroll
        for (int k = 0; k < NG; ++k)
            f[k] = __builtin_amdgcn_mfma_f32_16x16x32_f16(row, col[k], v4f{}, 0, 0, 0);
        row = next;
        next = after;
        int any = 0;
#pragma unroll
        for (int k = 0; k < NG; ++k)
            any |= __float_as_int(f[k][0]) | __float_as_int(f[k][1]) | __float_as_int(f[k][2]) |
                   __float_as_int(f[k][3]);
        if (!__builtin_amdgcn_ballot_w64(any < 0))
            continue;
        // the signs as one mask per lane: bit 31 - (4k + v) for row 4q + v of group k
        unsigned m = 0u;
#pragma unroll
        for (int k = 0; k < NG; ++k)
#pragma unroll
            for (int v = 0; v < 4; ++v)
                m = __builtin_amdgcn_alignbit(m, (unsigned)__float_as_int(f[k][v]), 31);
        if (__builtin_expect(__popcll(__builtin_amdgcn_ballot_w64(__popc(m) >= kEncDense)) >= 32, 0)) {
            dense |= 1ull << (s >> 4);
            continue;
        }
        while (__builtin_amdgcn_ballot_w64(m != 0u)) {
            const int b = m ? __clz(m) : 0;
            const int sj = s + 4 * q + (b & 3), ti = 16 * (b >> 2) + r;
            const bool cand = m != 0u && sj < wk.nj && wk.j0 + sj > wk.i0 + ti;
            m &= ~(0x80000000u >> b);
            push(cand, ti, sj);
        }
    }
    if (__builtin_expect(dense != 0ull, 0)) {
        const double inv_l = enc_inv_scale(scale[sys_of[wk.i0]]);
        const bool two = wk.ni > 64, h0 = lane < wk.ni, h1 = 64 + lane < wk.ni;
        const EncF I0 = enc_load32(in, wk.i0 + (h0 ? lane : 0), dt, inv_l);
        const EncF I1 = enc_load32(in, wk.i0 + (h1 ? 64 + lane : 0), dt, inv_l);
        while (dense) {
            const int s = 16 * (__ffsll((long long)dense) - 1), jn = min(16, wk.nj - s);
            dense &= dense - 1ull;
            wave_lds_sync();
            if (lane < jn)
                sj[lane] = enc_load32(in, wk.j0 + s + lane, dt, inv_l);
            wave_lds_sync();
            for (int k = 0; k < jn; ++k) {
                const EncF J = sj[k];
                // source minus lane's first target
                const int d = wk.j0 + s + k - (wk.i0 + lane);
                const bool c0 = enc_bound32(I0, J) && h0 && d > 0;
                const bool c1 = two && enc_bound32(I1, J) && h1 && d > 64;
                if (!__builtin_amdgcn_ballot_w64(c0 || c1))
                    continue;
#pragma unroll 1
                for (int e = 0; e < 128; e += 64)
                    push(e ? c1 : c0, e + lane, s + k);
            }
        }
    }
    if (qn > 0)
        drain(qn);
}

// After the direct checks of a captured run (nsets steps, the k-th with set k's
// count and the flags kEncTag + k, each appending to the list from its start): the
// run's statistics, and the last check's count and flags as one check leaves them.
__global__ void k_enc_run_end(int ntot, int nsets, int cap, int *__restrict__ ce, DevStats *stats)
{
    const int i = blockIdx.x * blockDim.x + threadIdx.x;
    if (i < ntot)
        ce[i] = ce[i] == kEncTag + nsets - 1 ? kEncFlag : 0;
    if (i == 0) {
        for (int k = 0; k < nsets; ++k) {
            const int count = stats->set_nce[k];
            stats->total_nce += count;
            stats->max_nce = max(stats->max_nce, count);
            stats->overflow_steps += count > cap;
        }
        stats->cur_nce = stats->set_nce[nsets - 1];
    }
}

// Before the direct check: no encounter flag, an empty list.
__global__ void k_enc_clear(int ntot, int *__restrict__ ce, DevStats *stats)
{
    const int i = blockIdx.x * blockDim.x + threadIdx.x;
    if (i < ntot)
        ce[i] = 0;
    if (i == 0)
        stats->cur_nce = 0;
}

// ----------------------------------------------------------------------------
// Spatially sorted encounter check.  Each step the bodies of every system are
// binned by the chord midpoint's cylindrical (ln R, phi) into a power-of-two
// grid of about N_s/8 cells traversed in Morton order, counting-sorted, and
// cut into tiles of 64 consecutive bodies.  A tile carries the centre and
// radius of its chord midpoints M, chords c and endpoint velocity deviations
// (d, with kEncP |p| added to its radius).  For i in tile A and j in tile B
// f(s) >= Lmin^2 - Qmax Em / 2 where that is positive (kEncP, B), with
//   Lmin = D - sm_A - sm_B - Cm/2,  Qmax = D + sm_A + sm_B + Cm/2,
//   D = |cm_B - cm_A|, Cm = |cc_B - cc_A| + sc_A + sc_B, Em = |ce_B - ce_A| + se_A + se_B,
// so a tile pair whose bound exceeds max rc^2 holds no flagged pair.  Surviving
// tile pairs are tested pair by pair (k_enc_pairs).  The bodies of
// a cell are put in index order after the binning, so the sorted order does
// not depend on the timing of its atomics; the output list is sorted.
// ----------------------------------------------------------------------------
__device__ __forceinline__ unsigned morton2(unsigned band, int nb, unsigned pb, int np)
{
    unsigned code = 0;
    int k = 0, bit = 0;
    for (; k < nb || k < np; ++k) {
        if (k < np)
            code |= ((pb >> k) & 1u) << bit++;
        if (k < nb)
            code |= ((band >> k) & 1u) << bit++;
    }
    return code;
}

__global__ void k_cells(const RBlk *__restrict__ rblk, const int *__restrict__ rb_first,
                        const int *__restrict__ rb_count, const double *__restrict__ lnr_part,
                        const int *__restrict__ sys_cell_base, const int *__restrict__ sys_cell_cnt,
                        const double *__restrict__ q0x, const double *__restrict__ q0y,
                        const double *__restrict__ q1x, const double *__restrict__ q1y,
                        int *__restrict__ cell_cnt,
                        int *__restrict__ cell_of, int *__restrict__ slot_of, int *__restrict__ ce)
{
    __shared__ double sh[2 * kBlock];
    const RBlk b = rblk[blockIdx.x];
    // ln R range of the whole system, from its blocks' partials
    double lo = INFINITY, hi = -INFINITY;
    for (int k = threadIdx.x; k < rb_count[b.sys]; k += kBlock) {
        lo = fmin(lo, lnr_part[2 * (size_t)(rb_first[b.sys] + k)]);
        hi = fmax(hi, lnr_part[2 * (size_t)(rb_first[b.sys] + k) + 1]);
    }
    sh[threadIdx.x] = lo;
    sh[kBlock + threadIdx.x] = hi;
    __syncthreads();
    for (int st = kBlock / 2; st > 0; st >>= 1) {
        if ((int)threadIdx.x < st) {
            sh[threadIdx.x] = fmin(sh[threadIdx.x], sh[threadIdx.x + st]);
            sh[kBlock + threadIdx.x] = fmax(sh[kBlock + threadIdx.x], sh[kBlock + threadIdx.x + st]);
        }
        __syncthreads();
    }
    lo = sh[0];
    hi = sh[kBlock];
    const int C = sys_cell_cnt[b.sys];          // power of two
    int lc = 31 - __clz(C);
    // bands B x phi bins P = C with square cells in (ln R, phi): B ~ sqrt(C span / 2 pi)
    const double span = fmax(hi - lo, 0.0);
    int lb = 0;
    double bstar = sqrt((double)C * span / 6.283185307179586);
    if (bstar > 1.0)
        lb = min(lc, (int)floor(log2(bstar) + 0.5));
    const int lp = lc - lb;
    const int i = b.start + threadIdx.x;
    if (i < b.end) {
        // the chord midpoint, as in k_drift
        const double x0 = q0x[i], y0 = q0y[i];
        const double mx = x0 + 0.5 * (q1x[i] - x0), my = y0 + 0.5 * (q1y[i] - y0);
        double R = sqrt(mx * mx + my * my);
        double lnr = log(fmax(R, 1e-300));
        unsigned band = 0, pb = 0;
        if (span > 0.0)
            band = (unsigned)min((1 << lb) - 1, max(0, (int)((lnr - lo) / span * (double)(1 << lb))));
        double phi = atan2(my, mx);
        pb = (unsigned)min((1 << lp) - 1, max(0, (int)((phi + 3.141592653589793) *
                                                      (0.15915494309189535 * (double)(1 << lp)))));
        int cell = sys_cell_base[b.sys] + (int)morton2(band, lb, pb, lp);
        cell_of[i] = cell;
        slot_of[i] = atomicAdd(&cell_cnt[cell], 1);
        // no encounter flag yet (the check of this drift sets them)
        ce[i] = 0;
    }
}

// Exclusive scan of the cell counts (one workgroup), zeroing them for the next
// step, and reset of the surviving-tile-pair counter.
// 256 threads (one wave per SIMD): blocks this small still find room on a CU
// beside the force pass's waves, so the encounter check's scan need not wait
// for the force pass to drain a whole CU.
constexpr int kScanThreads = 256;
constexpr int kScanChunk = kScanChunkCells;    // cells per block pass, 4 per thread
static_assert(kScanChunk == 4 * kScanThreads, "four cells per scan thread");

// Exclusive scan over the kScanThreads threads of a block; *total gets the sum.
__device__ __forceinline__ int block_exscan(int v, int *sh, int &total)
{
    const int t = threadIdx.x, lane = t & 63, wv = t >> 6;
    int x = v;
    for (int o = 1; o < 64; o <<= 1) {
        int y = __shfl_up(x, o);
        if (lane >= o)
            x += y;
    }
    if (lane == 63)
        sh[wv] = x;
    __syncthreads();
    if (t < 64) {
        int w = t < kScanThreads / 64 ? sh[t] : 0;
        for (int o = 1; o < 64; o <<= 1) {
            int y = __shfl_up(w, o);
            if (lane >= o)
                w += y;
        }
        if (t < kScanThreads / 64)
            sh[32 + t] = w;               // inclusive wave totals
    }
    __syncthreads();
    total = sh[32 + kScanThreads / 64 - 1];
    const int before = wv > 0 ? sh[32 + wv - 1] : 0;
    __syncthreads();                      // sh is reused by the next call
    return before + x - v;
}

// Four consecutive cells of chunk `base` per thread, guarded at ncell.
__device__ __forceinline__ void load4(const int *__restrict__ cnt, int base, int ncell, int (&c)[4])
{
    const int k0 = base + 4 * (int)threadIdx.x;
#pragma unroll
    for (int q = 0; q < 4; ++q)
        c[q] = k0 + q < ncell ? cnt[k0 + q] : 0;
}

// Exclusive scan of one chunk with a carried offset: cell_off, counts cleared.
__device__ __forceinline__ int scan_chunk(int *__restrict__ cell_cnt, int *__restrict__ cell_off,
                                          int base, int ncell, int carry, int *sh)
{
    int c[4];
    load4(cell_cnt, base, ncell, c);
    int tot;
    int run = carry + block_exscan(c[0] + c[1] + c[2] + c[3], sh, tot);
    const int k0 = base + 4 * (int)threadIdx.x;
#pragma unroll
    for (int q = 0; q < 4; ++q) {
        if (k0 + q < ncell) {
            cell_off[k0 + q] = run;
            cell_cnt[k0 + q] = 0;
        }
        run += c[q];
    }
    return tot;
}

// Counting-sort offsets: cell_off = exclusive scan of cell_cnt (all systems'
// cells back to back), counts cleared for the next step.  One block walks
// the cells in chunks (up to kScanSerialChunks chunks); larger grids use
// k_scan_sums + k_scan_apply.
constexpr int kScanSerialChunks = 16;
__global__ __launch_bounds__(kScanThreads) void k_cell_scan(int *__restrict__ cell_cnt,
                                                            int *__restrict__ cell_off, int ncell,
                                                            DevStats *stats)
{
    __shared__ int sh[64];
    int carry = 0;
    for (int base = 0; base < ncell; base += kScanChunk)
        carry += scan_chunk(cell_cnt, cell_off, base, ncell, carry, sh);
    if (threadIdx.x == 0) {
        stats->cur_tp = 0;
        stats->cur_nce = 0;
    }
}

// Block b: sum of the counts of chunk b.
__global__ __launch_bounds__(kScanThreads) void k_scan_sums(const int *__restrict__ cell_cnt,
                                                            int ncell, int *__restrict__ part)
{
    __shared__ int sh[64];
    int c[4];
    load4(cell_cnt, blockIdx.x * kScanChunk, ncell, c);
    int tot;
    (void)block_exscan(c[0] + c[1] + c[2] + c[3], sh, tot);
    if (threadIdx.x == 0)
        part[blockIdx.x] = tot;
}

// Block b: exclusive offset of chunk b from the chunk sums (in order), then the
// chunk's own scan.  Block 0 also resets the tile-pair count.
__global__ __launch_bounds__(kScanThreads) void k_scan_apply(int *__restrict__ cell_cnt,
                                                             int *__restrict__ cell_off, int ncell,
                                                             const int *__restrict__ part,
                                                             DevStats *stats)
{
    __shared__ int sh[64];
    int pre = 0;
    for (int k = threadIdx.x; k < (int)blockIdx.x; k += kScanThreads)
        pre += part[k];
    int tot;
    (void)block_exscan(pre, sh, tot);
    (void)scan_chunk(cell_cnt, cell_off, blockIdx.x * kScanChunk, ncell, tot, sh);
    if (blockIdx.x == 0 && threadIdx.x == 0) {
        stats->cur_tp = 0;
        stats->cur_nce = 0;
    }
}

// Sorted position of every body: its cell's offset plus the slot the binning
// took (the order inside a cell follows the atomics' timing until
// k_cell_order puts it in index order).  slot_of[i] becomes the position.
__global__ void k_scatter(const RBlk *__restrict__ rblk, const int *__restrict__ cell_of,
                          int *__restrict__ slot_of, const int *__restrict__ cell_off,
                          int *__restrict__ ord)
{
    const RBlk b = rblk[blockIdx.x];
    const int i = b.start + threadIdx.x;
    if (i >= b.end)
        return;
    const int pos = cell_off[cell_of[i]] + slot_of[i];
    ord[pos] = i;
    slot_of[i] = pos;
}

// The bodies of every cell in index order, so that the sorted order, its tiles
// and the tile pairs are the same from run to run.  One wave per cell: a body's
// new slot is the number of smaller indices in its cell.  A cell of more than
// kCellSortMax bodies keeps the binning's order (its set is still right).
constexpr int kCellSortMax = 512;

__global__ __launch_bounds__(kBlock) void k_cell_order(const int *__restrict__ cell_off, int ncell,
                                                       int ntot, int *__restrict__ ord,
                                                       int *__restrict__ pos_of)
{
    __shared__ int sb[kBlock / 64][kCellSortMax];
    const int lane = threadIdx.x & 63, wv = threadIdx.x >> 6;
    const int c = blockIdx.x * (kBlock / 64) + wv;
    int start = 0, k = 0;
    if (c < ncell) {
        start = cell_off[c];
        k = (c + 1 < ncell ? cell_off[c + 1] : ntot) - start;
    }
    const bool go = k > 1 && k <= kCellSortMax;
    if (go)
        for (int e = lane; e < k; e += 64)
            sb[wv][e] = ord[start + e];
    __syncthreads();
    if (go)
        for (int e = lane; e < k; e += 64) {
            const int me = sb[wv][e];
            int rank = 0;
            for (int q = 0; q < k; ++q)
                rank += sb[wv][q] < me;
            ord[start + rank] = me;
            pos_of[me] = start + rank;
        }
}

// FP32 record of the pair filter: midpoint M and chord c, and the bound b' of
// 3/4 eps (e34) widened by 2^-21 (|M|_1 + |c|_1) for the FP32 rounding of M, c and
// their differences, and by 2^-18 relative for the rounding of the bound itself,
// negated (sign bit set) for a small body; the chord's fourth word is rc rounded
// up.  A pair's bound is |b'_i| + |b'_j| + max(rc_i, rc_j).
__device__ __forceinline__ void enc_record32(double mx, double my, double mz, double cx, double cy,
                                             double cz, double e34, double rc, bool big, float4 &M,
                                             float4 &C)
{
    const float w = (float)((e34 + 0x1p-21 * (fabs(mx) + fabs(my) + fabs(mz) + fabs(cx) + fabs(cy) +
                                              fabs(cz))) * (1.0 + 0x1p-18));
    M = make_float4((float)mx, (float)my, (float)mz, big ? w : -w);
    C = make_float4((float)cx, (float)cy, (float)cz, (float)(rc * (1.0 + 0x1p-20)));
}

// Chord midpoint M, chord c, deviation d and the bound p of the mean deviation
// (enc_deviation) of one record.
__device__ __forceinline__ void rec_geometry(const SRec &r, double dt, double (&M)[3],
                                             double (&c)[3], double (&d)[3], double &p)
{
    for (int k = 0; k < 3; ++k) {
        c[k] = r.q1[k] - r.q0[k];
        M[k] = r.q0[k] + 0.5 * c[k];
    }
    p = enc_deviation(dt, r.v0, r.v1, c, d);
}

// The sorted records from the drift outputs, body by body (coalesced reads),
// each written to the body's sorted position.
__global__ void k_srec(int ntot, const int *__restrict__ pos_of, const int *__restrict__ sys_of,
                       const double *__restrict__ q0x, const double *__restrict__ q0y,
                       const double *__restrict__ q0z, const double *__restrict__ v0x,
                       const double *__restrict__ v0y, const double *__restrict__ v0z,
                       const double *__restrict__ qx, const double *__restrict__ qy,
                       const double *__restrict__ qz, const double *__restrict__ vx,
                       const double *__restrict__ vy, const double *__restrict__ vz,
                       const double *__restrict__ rc, const int *__restrict__ off,
                       const int *__restrict__ nbig, SRec *__restrict__ srec,
                       float4 *__restrict__ em, float4 *__restrict__ eg, double dt, int fused)
{
    const int i = blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= ntot)
        return;
    const int pos = pos_of[i];
    const int sy = sys_of[i];
    SRec r;
    r.q0[0] = q0x[i]; r.q0[1] = q0y[i]; r.q0[2] = q0z[i];
    r.v0[0] = v0x[i]; r.v0[1] = v0y[i]; r.v0[2] = v0z[i];
    r.q1[0] = qx[i];  r.q1[1] = qy[i];  r.q1[2] = qz[i];
    r.v1[0] = vx[i];  r.v1[1] = vy[i];  r.v1[2] = vz[i];
    r.rc = rc[i];
    r.body = i;
    r.big = (i - off[sy]) < nbig[sy] ? 1 : 0;
    srec[pos] = r;
    double M[3], c[3], d[3], p;
    rec_geometry(r, dt, M, c, d, p);
    // the bound: 3/4 E's share of the body, with the deviation d apart (k_enc_pairs) or
    // its norm in it (the force pass with the encounter test in it, which has no d),
    // and 2^-45 (|M| + |c|) for the rounding of midpoint, chord and deviations
    const double e34 = 0.75 * (p + (fused ? norm3(d[0], d[1], d[2]) : 0.0)) * (1.0 + 0x1p-20) +
                       0x1p-21 * norm1(d[0], d[1], d[2]) +
                       0x1p-45 * (norm1(M[0], M[1], M[2]) + norm1(c[0], c[1], c[2]));
    enc_record32(M[0], M[1], M[2], c[0], c[1], c[2], e34, rc[i], r.big != 0, em[2 * (size_t)pos],
                 em[2 * (size_t)pos + 1]);
    eg[pos] = make_float4((float)d[0], (float)d[1], (float)d[2], (float)(p * (1.0 + 0x1p-20)));
}

__device__ __forceinline__ double wave_sum(double v)
{
    for (int o = 32; o > 0; o >>= 1)
        v += __shfl_xor(v, o);
    return v;
}

__device__ __forceinline__ double wave_maxd(double v)
{
    for (int o = 32; o > 0; o >>= 1)
        v = fmax(v, __shfl_xor(v, o));
    return v;
}

// One wave per tile: centres (means) and radii (maxima) of its bodies' geometry.
__global__ __launch_bounds__(kBlock) void k_tile_bounds(const Tile *__restrict__ tiles, int ntile,
                                                        const SRec *__restrict__ srec, double dt,
                                                        TileB *__restrict__ tileb)
{
    const int tw = blockIdx.x * (kBlock / 64) + (threadIdx.x >> 6);
    const int lane = threadIdx.x & 63;
    if (tw >= ntile)
        return;
    const Tile T = tiles[tw];
    const bool on = lane < T.count;
    double M[3] = {0, 0, 0}, c[3] = {0, 0, 0}, d[3] = {0, 0, 0}, p = 0.0, rc = 0.0;
    bool big = false;
    if (on) {
        const SRec r = srec[T.start + lane];
        rec_geometry(r, dt, M, c, d, p);
        rc = r.rc;
        big = r.big != 0;
    }
    const bool any_big = __any(big), all_big = __all(!on || big);
    const double inv = 1.0 / (double)T.count;
    double cm[3], cc[3], ce[3];
    for (int k = 0; k < 3; ++k) {
        cm[k] = wave_sum(M[k]) * inv;
        cc[k] = wave_sum(c[k]) * inv;
        ce[k] = wave_sum(d[k]) * inv;
    }
    double dm = 0.0, dc = 0.0, de = 0.0;
    if (on) {
        dm = norm3(M[0] - cm[0], M[1] - cm[1], M[2] - cm[2]);
        dc = norm3(c[0] - cc[0], c[1] - cc[1], c[2] - cc[2]);
        de = norm3(d[0] - ce[0], d[1] - ce[1], d[2] - ce[2]) + p;
    }
    // radii widened by 2^-20 to cover the rounding of the centres and norms
    const double wf = 1.0 + 0x1p-20;
    const double sm = wave_maxd(dm) * wf, sc = wave_maxd(dc) * wf, sde = wave_maxd(de) * wf;
    const double rcm = wave_maxd(rc);
    if (lane == 0) {
        TileB B;
        for (int k = 0; k < 3; ++k) {
            B.cm[k] = cm[k];
            B.cc[k] = cc[k];
            B.ce[k] = ce[k];
        }
        B.sm = sm;
        B.sc = sc;
        B.se = sde;
        B.rc = rcm;
        B.big = any_big ? 1 : 0;
        B.all_big = all_big ? 1 : 0;
        B.pad2[0] = B.pad2[1] = 0.0;
        tileb[tw] = B;
    }
}

// True when a pair between the two bounded sets may be flagged.  The rounding
// margin is relative to the squared scales involved.
__device__ __forceinline__ bool may_meet(const double cmA[3], double smA, const double ccA[3],
                                         double scA, const double ceA[3], double seA, double rcA,
                                         const TileB &B)
{
    double D = norm3(B.cm[0] - cmA[0], B.cm[1] - cmA[1], B.cm[2] - cmA[2]);
    double Cm = norm3(B.cc[0] - ccA[0], B.cc[1] - ccA[1], B.cc[2] - ccA[2]) + scA + B.sc;
    double Em = norm3(B.ce[0] - ceA[0], B.ce[1] - ceA[1], B.ce[2] - ceA[2]) + seA + B.se;
    double Lmin = D - smA - B.sm - 0.5 * Cm;
    double Qmax = D + smA + B.sm + 0.5 * Cm;
    double RC = fmax(rcA, B.rc);
    if (!(Lmin > 0.0))
        return true;
    double lhs = Lmin * Lmin - 0.5 * Qmax * Em;
    return !(lhs > RC * RC * (1.0 + 1e-6) + 1e-12 * Qmax * Qmax);
}

// One wave per culling unit (tile A against tiles [b0, b0 + 64) of the same
// system with B >= A; kTpWaves units per workgroup): its lanes test one tile B
// each and the pairs that may meet are appended.  The survivors are counted
// first and the workgroup reserves its whole range with one atomic (a counter
// that every wave of the grid hits is a serial point), then the test is
// repeated to write the pairs.
constexpr int kTpWaves = 4;

__device__ __forceinline__ bool tile_pair_kept(const Tile &TA, const TileB &BA,
                                               const TileB *__restrict__ tileb, int B)
{
    // two small bodies never interact: a pair of tiles without a big body is skipped
    return B <= TA.last && (BA.big || tileb[B].big) &&
           may_meet(BA.cm, BA.sm, BA.cc, BA.sc, BA.ce, BA.se, BA.rc, tileb[B]);
}

__global__ __launch_bounds__(64 * kTpWaves) void k_tile_pairs(const Tile *__restrict__ tiles,
                                                             const int2 *__restrict__ units,
                                                             int nunit,
                                                             const TileB *__restrict__ tileb,
                                                             int2 *__restrict__ tpairs, int tp_cap,
                                                             DevStats *stats)
{
    __shared__ int wcount[kTpWaves];
    __shared__ int wbase[kTpWaves];
    const int lane = threadIdx.x & 63, wv = threadIdx.x >> 6;
    const int u = blockIdx.x * kTpWaves + wv;
    const bool has = u < nunit;
    int A = 0, B = 0;
    bool ok = false;
    if (has) {
        const int2 U = units[u];
        A = U.x;
        B = U.y + lane;
        const Tile TA = tiles[A];
        const TileB BA = tileb[A];
        ok = tile_pair_kept(TA, BA, tileb, B);
    }
    const unsigned long long mask = __ballot(ok);
    if (lane == 0)
        wcount[wv] = (int)__popcll(mask);
    __syncthreads();
    if (threadIdx.x == 0) {
        int tot = 0;
        for (int w = 0; w < kTpWaves; ++w) {
            wbase[w] = tot;
            tot += wcount[w];
        }
        const int base = tot ? atomicAdd(&stats->cur_tp, tot) : 0;
        for (int w = 0; w < kTpWaves; ++w)
            wbase[w] += base;
    }
    __syncthreads();
    if (ok) {
        const int p = wbase[wv] + (int)__popcll(mask & ((1ull << lane) - 1ull));
        if (p < tp_cap)
            tpairs[p] = make_int2(A, B);
    }
}

// The record of a sorted position, every field read at once.
__device__ __forceinline__ HRec enc_load(const SRec &R)
{
    HRec I;
    for (int k = 0; k < 3; ++k) {
        I.q0[k] = R.q0[k];
        I.v0[k] = R.v0[k];
        I.q1[k] = R.q1[k];
        I.v1[k] = R.v1[k];
    }
    I.rc = R.rc;
    I.body = R.body;
    return I;
}

// The exact test of two sorted positions, and the append of a flagged pair.
__device__ __noinline__ void enc_candidate(const SRec *__restrict__ srec, double dt,
                                           unsigned long long *keys, int cap, int *ce,
                                           DevStats *stats, int pi, int pj)
{
    enc_exact(enc_load(srec[pi]), srec[pj], dt, keys, cap, ce, &stats->cur_nce);
}

// One wave per kept tile pair (A, B), the waves striding over the count: lane
// L holds the FP32 filter records of body L of tile A (midpoint with widened
// bound, chord with rc, deviation d with the bound of the mean deviation: 48 B),
// tile B's sit in the wave's LDS slice, and
// every lane meets the 64 sources in turn with the relative-chord filter in
// FP32 and the relative deviation in it (kEncP), a superset of the pairs that can be
// flagged (the widening covers the rounding).  A lane first meets tile B's bounds with
// the tile-pair test, as a tile of one body whose FP32 records stand for small balls
// around its FP64 values.  The pairs the filter keeps are queued in the wave's LDS and take the exact test
// from the sorted FP64 records in memory 64 at a time, one per lane (with steps of a
// radian most pairs of a dense ring pass the filter, and a test per pass would run on
// a few lanes); a tile pair reads 6 KB of filter records instead of the 112-byte
// records of both tiles.  W waves per workgroup (independent of each other): 10 KB of LDS
// each, so that the workgroup's size says where it fits beside the force's (launch_enc_test).
template <int W>
__global__ __launch_bounds__(64 * W) void k_enc_pairs(const Tile *__restrict__ tiles,
                                                      const TileB *__restrict__ tileb,
                                                      const int2 *__restrict__ tpairs, int tp_cap,
                                                      const SRec *__restrict__ srec,
                                                      const float4 *__restrict__ em,
                                                      const float4 *__restrict__ eg, double dt,
                                                      unsigned long long *__restrict__ keys,
                                                      int cap, int *__restrict__ ce,
                                                      DevStats *stats)
{
    const int wv = W > 1 ? __builtin_amdgcn_readfirstlane(threadIdx.x >> 6) : 0;
    __shared__ float4 sm_w[W][64], sc_w[W][64], sd_w[W][64];
    float4 (&sm_)[64] = sm_w[wv], (&sc_)[64] = sc_w[wv], (&sd_)[64] = sd_w[wv];
    // queued pairs (lane | source << 8), fewer than 64 between drains
    __shared__ int qe_w[W][128];
    int (&qe)[128] = qe_w[wv];
    // tile A's exact-test fields (q0, v0, q1, v1, rc by plane; body
    // index), staged at the tile pair's first full drain: a drain's 64 pairs
    // hold many targets and few sources
    __shared__ double ha_w[W][13][64];
    __shared__ int hb_w[W][64];
    double (&ha)[13][64] = ha_w[wv];
    int (&hb)[64] = hb_w[wv];
    const int lane = threadIdx.x & 63;
    const int npair = min(stats->cur_tp, tp_cap);
    const float qnan = __int_as_float(0x7fc00000);
    for (int p = blockIdx.x * W + wv; p < npair; p += gridDim.x * W) {
        const int2 AB = tpairs[p];
        Tile TA = tiles[AB.x], TB = tiles[AB.y];
        // uniform over the wave (one tile pair a wave): kept in scalar registers
        TA.start = __builtin_amdgcn_readfirstlane(TA.start);
        TA.count = __builtin_amdgcn_readfirstlane(TA.count);
        TB.start = __builtin_amdgcn_readfirstlane(TB.start);
        TB.count = __builtin_amdgcn_readfirstlane(TB.count);
        // tile B's FP32 filter records in the wave's LDS slice (padding: NaN
        // midpoints, which no test passes)
        if (lane < TB.count) {
            sm_[lane] = em[2 * (size_t)(TB.start + lane)];
            sc_[lane] = em[2 * (size_t)(TB.start + lane) + 1];
            sd_[lane] = eg[TB.start + lane];
        } else {
            sm_[lane] = make_float4(qnan, qnan, qnan, 0.0f);
            sc_[lane] = sd_[lane] = make_float4(0.0f, 0.0f, 0.0f, 0.0f);
        }
        wave_lds_sync();
        const bool on = lane < TA.count;
        const float4 Mi = on ? em[2 * (size_t)(TA.start + lane)] : make_float4(qnan, qnan, qnan, 0.0f);
        const float4 Ci = on ? em[2 * (size_t)(TA.start + lane) + 1] : make_float4(0.0f, 0.0f, 0.0f, 0.0f);
        // the lane against tile B's bounds with the tile-pair test, the lane a
        // tile of one body whose FP32 records stand for balls around them: 2^-23
        // of each vector's norm covers its rounding, se and rc are rounded up
        bool lane_ok = false;
        const float4 Gi = on ? eg[TA.start + lane] : make_float4(0.0f, 0.0f, 0.0f, 0.0f);
        if (on) {
            const double Mv[3] = {Mi.x, Mi.y, Mi.z}, cv[3] = {Ci.x, Ci.y, Ci.z},
                         ev[3] = {Gi.x, Gi.y, Gi.z};
            const double sM = 0x1p-23 * norm3(Mv[0], Mv[1], Mv[2]);
            const double sC = 0x1p-23 * norm3(cv[0], cv[1], cv[2]);
            const double sE = (double)Gi.w + 0x1p-23 * norm3(ev[0], ev[1], ev[2]);
            const TileB &BB = tileb[AB.y];
            lane_ok = (__float_as_int(Mi.w) >= 0 || BB.big) &&
                      may_meet(Mv, sM, cv, sC, ev, sE, (double)Ci.w, BB);
        }
        const bool diag = AB.x == AB.y;
        const int nj = __builtin_amdgcn_ballot_w64(lane_ok) ? TB.count : 0;
        const float wi = fabsf(Mi.w);
        int qn = 0;
        bool staged = false;
        // the exact test of queue entry e (this lane's): target from the staged
        // fields, source record from memory
        auto test_entry = [&](int e) {
            const int li = e & 255;
            HRec I;
            for (int k = 0; k < 3; ++k) {
                I.q0[k] = ha[k][li];
                I.v0[k] = ha[3 + k][li];
                I.q1[k] = ha[6 + k][li];
                I.v1[k] = ha[9 + k][li];
            }
            I.rc = ha[12][li];
            I.body = hb[li];
            enc_exact(I, srec[TB.start + (e >> 8)], dt, keys, cap, ce, &stats->cur_nce);
        };
        auto stage = [&]() {
            if (!staged) {
                if (on) {
                    const HRec R = enc_load(srec[TA.start + lane]);
                    for (int k = 0; k < 3; ++k) {
                        ha[k][lane] = R.q0[k];
                        ha[3 + k][lane] = R.v0[k];
                        ha[6 + k][lane] = R.q1[k];
                        ha[9 + k][lane] = R.v1[k];
                    }
                    ha[12][lane] = R.rc;
                    hb[lane] = R.body;
                }
                staged = true;
            }
        };
        // the pair loop, with the diagonal's order test and the small-small
        // test only where the tile pair needs them
        auto pair_loop = [&](auto diag_c, auto small_c) {
        constexpr bool DG = decltype(diag_c)::value, SM = decltype(small_c)::value;
        for (int jj = 0; jj < nj; ++jj) {
            // source jj's FP32 filter records (one broadcast read each)
            const float4 E = sm_[jj], F = sc_[jj], H = sd_[jj];
            // relative chord filter in FP32 (the bound's widening covers the
            // rounding), every lane without a branch
            const float ex = E.x - Mi.x, ey = E.y - Mi.y, ez = E.z - Mi.z;
            const float cx = F.x - Ci.x, cy = F.y - Ci.y, cz = F.z - Ci.z;
            const float D2 = fmaf(ez, ez, fmaf(ey, ey, ex * ex));
            const float C2 = fmaf(cz, cz, fmaf(cy, cy, cx * cx));
            const float hx = H.x - Gi.x, hy = H.y - Gi.y, hz = H.z - Gi.z;
            const float H2 = fmaf(hz, hz, fmaf(hy, hy, hx * hx));
            const float Sr = (fabsf(E.w) + wi) + max_nonneg(F.w, Ci.w);
            // D <= C + 3/4 |dd| + S, squared as in enc_record
            bool cand = lane_ok & (D2 <= fmaf(2.0f * Sr, Sr, fmaf(1.125f, H2, C2)) *
                                             (2.0f * (1.0f + 0x1p-18f)));
            if (DG)
                cand &= jj > lane;
            if (SM)
                cand &= (__float_as_int(E.w) & __float_as_int(Mi.w)) >= 0;
            // the pairs the filter keeps join the wave's queue; 64 of them at a
            // time take the exact test, one per lane
            const unsigned long long mk = __builtin_amdgcn_ballot_w64(cand);
            if (mk) {
                if ((mk >> lane) & 1ull)
                    qe[qn + __popcll(mk & ((1ull << lane) - 1ull))] = lane | (jj << 8);
                qn += __popcll(mk);
                if (qn >= 64) {
                    stage();
                    wave_lds_sync();
                    test_entry(qe[lane]);
                    const int rest = qn - 64;
                    const int v = lane < rest ? qe[64 + lane] : 0;
                    wave_lds_sync();
                    if (lane < rest)
                        qe[lane] = v;
                    wave_lds_sync();
                    qn = rest;
                }
            }
        }
        };
        // a small body in tile A (the sign of a lane's bound) or in tile B
        const bool small = __builtin_amdgcn_ballot_w64(on && __float_as_int(Mi.w) < 0) != 0 ||
                           !tileb[AB.y].all_big;
        if (diag) {
            if (small)
                pair_loop(std::true_type{}, std::true_type{});
            else
                pair_loop(std::true_type{}, std::false_type{});
        } else {
            if (small)
                pair_loop(std::false_type{}, std::true_type{});
            else
                pair_loop(std::false_type{}, std::false_type{});
        }
        if (qn > 0) {
            // the rest: from the staged fields if a full drain staged them, else
            // both records from memory (a tile pair with few pairs to test)
            wave_lds_sync();
            if (lane < qn) {
                const int e = qe[lane];
                if (staged)
                    test_entry(e);
                else
                    enc_candidate(srec, dt, keys, cap, ce, stats, TA.start + (e & 255),
                                  TB.start + (e >> 8));
            }
        }
        // the slices, the queue and the staged fields are refilled for the
        // next pair only after every lane's reads
        wave_lds_sync();
    }
}

// ----------------------------------------------------------------------------
// Force and encounter check in one pass over spatially sorted tiles (FP32C,
// every body big).  The symmetric force runs over super-tile pairs of sorted
// positions (sources and targets gathered through the sorted order, split
// partials by position, mapped back to bodies by the finalize).  In every
// round the wave bounds the tile pairs of its target sub-tiles and the source
// sub-tiles with the culling lemma of the sorted check (may_meet on the tiles
// of 64); where a tile pair may hold a flagged pair, each pair of it also gets
// the FP32 relative-chord filter, and the pairs it passes the exact Hermite
// test in FP64 from the sorted records.  Each unordered pair is met once, so
// each flagged pair is appended once.
// ----------------------------------------------------------------------------
// Tile of 64 sorted positions holding position p of system sy.
__device__ __forceinline__ int tile_of(const int *__restrict__ tile_first, const int *__restrict__ off,
                                       int sy, int p)
{
    return tile_first[sy] + (p - off[sy]) / 64;
}

template <int R, int G>
__global__ __launch_bounds__(64 * G, R == 4 ? 1 : 2) void k_force32c_fused(
    const FWork *__restrict__ work, int nitems, const int *__restrict__ ord,
    const float4 *__restrict__ pk, const float4 *__restrict__ em, const TileB *__restrict__ tileb,
    const int *__restrict__ tile_first, const int *__restrict__ off, const double *__restrict__ qx,
    const double *__restrict__ qy, const double *__restrict__ qz, const double *__restrict__ m,
    const double *__restrict__ rc, float *__restrict__ fpart, int ntot, int maxs, double inner,
    EncCtx ec)
{
    constexpr int T = 64 * R;
    __shared__ SymTile32E<T> tl[G];
    const int lane = threadIdx.x & 63, wv = threadIdx.x >> 6;
    const size_t plane = (size_t)maxs * ntot;
    const float qnan = __int_as_float(0x7fc00000);
    int near = 0;
    for (int it = blockIdx.x; it < nitems; it += gridDim.x) {
        const FWork wk = work[it];
        const bool diag = wk.i0 == wk.j0;
        // the G source tiles of super-tile J, gathered through the sorted order
        for (int k = threadIdx.x; k < G * T; k += 64 * G) {
            SymTile32<T> &S = tl[k / T].t;
            const int e = k % T;
            if (k < wk.nj) {
                const int b = ord[wk.j0 + k];
                S.a[e] = pk[2 * (size_t)b];
                S.b[e] = pk[2 * (size_t)b + 1];
                tl[k / T].em[e] = em[2 * (size_t)(wk.j0 + k)];
                tl[k / T].ec[e] = em[2 * (size_t)(wk.j0 + k) + 1];
            } else {
                S.a[e] = make_float4(1e18f, 1e18f, 1e18f, 0.0f);
                S.b[e] = make_float4(0.0f, 0.0f, 0.0f, 0.0f);
                tl[k / T].em[e] = make_float4(qnan, qnan, qnan, 0.0f);
                tl[k / T].ec[e] = make_float4(0.0f, 0.0f, 0.0f, 0.0f);
            }
            S.run[e] = make_float4(0.0f, 0.0f, 0.0f, 0.0f);
            S.ax[e] = S.ay[e] = S.az[e] = 0.0;
        }
        __syncthreads();
        const int ti0 = wk.i0 + wv * T;
        const int tni = min(T, wk.ni - wv * T);
        float xh[R], yh[R], zh[R], xl[R], yl[R], zl[R], mi[R];
        float hx[R], hy[R], hz[R], lx[R], ly[R], lz[R];
        float4 emi[R], eci[R];
        float tmi = 0.0f;
#pragma unroll
        for (int r = 0; r < R; ++r) {
            const int li = 64 * r + lane;
            const bool ok = li < tni;
            const int b = ord[ok ? ti0 + li : wk.i0];
            const float4 A = pk[2 * (size_t)b], B = pk[2 * (size_t)b + 1];
            xh[r] = A.x; yh[r] = A.y; zh[r] = A.z;
            xl[r] = B.x; yl[r] = B.y; zl[r] = B.z;
            mi[r] = ok ? A.w : 0.0f;
            tmi = max_nonneg(tmi, B.w);
            emi[r] = ok ? em[2 * (size_t)(ti0 + li)] : make_float4(qnan, qnan, qnan, 0.0f);
            eci[r] = ok ? em[2 * (size_t)(ti0 + li) + 1] : make_float4(0.0f, 0.0f, 0.0f, 0.0f);
            hx[r] = hy[r] = hz[r] = lx[r] = ly[r] = lz[r] = 0.0f;
        }
        tmi = wave_max_nonneg(tmi);
        const int nr = diag ? G / 2 + 1 : G;
        // The tile pairs that may hold a flagged pair, for every round at once:
        // lane (k R + t) R + r bounds target sub-tile r against sub-tile t of
        // round k's source tile (G R^2 <= 64 lanes), so the bounds' loads and
        // square roots are in flight together, once per item.
        unsigned long long livemask;
        {
            constexpr int RR = R * R;
            const int k = lane / RR, t = (lane % RR) / R, r = lane % R;
            const int s = (wv + k) % G;
            bool lv = false;
            if (k < nr && 64 * r < tni && s * T + 64 * t < wk.nj) {
                const TileB &A = tileb[tile_of(tile_first, off, wk.sys, ti0 + 64 * r)];
                lv = may_meet(A.cm, A.sm, A.cc, A.sc, A.ce, A.se, A.rc,
                              tileb[tile_of(tile_first, off, wk.sys, wk.j0 + s * T + 64 * t)]);
            }
            livemask = __ballot(lv);
        }
        for (int k = 0; k < nr; ++k) {
            const int s = (wv + k) % G;
            const bool go = tni > 0 && s * T < wk.nj && !(diag && 2 * k == G && wv >= G / 2);
            if (go) {
                // this round's bits: t R + r
                const int sj0 = wk.j0 + s * T;
                const unsigned live =
                    (unsigned)(livemask >> (k * R * R)) & (unsigned)((1ull << (R * R)) - 1ull);
                if (diag && k == 0)
                    sym_tile32c<R, true, T, true>(tl[s].t, lane, ti0, tni, sj0, inner, pk, qx, qy,
                                                  qz, m, rc, xh, yh, zh, xl, yl, zl, mi, tmi, hx,
                                                  hy, hz, lx, ly, lz, near, ord, ec, emi, eci,
                                                  live);
                else
                    sym_tile32c<R, false, T, true>(tl[s].t, lane, ti0, tni, sj0, inner, pk, qx, qy,
                                                   qz, m, rc, xh, yh, zh, xl, yl, zl, mi, tmi, hx,
                                                   hy, hz, lx, ly, lz, near, ord, ec, emi, eci,
                                                   live);
            }
            __syncthreads();
        }
#pragma unroll
        for (int r = 0; r < R; ++r) {
            const int li = 64 * r + lane;
            if (li < tni) {
                const int i = ti0 + li;
                double sx_ = (double)hx[r] + (double)lx[r];
                double sy_ = (double)hy[r] + (double)ly[r];
                double sz_ = (double)hz[r] + (double)lz[r];
                if (diag) {
                    sx_ += tl[wv].t.ax[li];
                    sy_ += tl[wv].t.ay[li];
                    sz_ += tl[wv].t.az[li];
                }
                fpart[(size_t)wk.slot * ntot + i] = (float)sx_;
                fpart[plane + (size_t)wk.slot * ntot + i] = (float)sy_;
                fpart[2 * plane + (size_t)wk.slot * ntot + i] = (float)sz_;
            }
        }
        if (!diag) {
            for (int k = threadIdx.x; k < wk.nj; k += 64 * G) {
                const SymTile32<T> &S = tl[k / T].t;
                const int e = k % T, j = wk.j0 + k;
                fpart[((size_t)0 * maxs + wk.pad) * ntot + j] = (float)S.ax[e];
                fpart[((size_t)1 * maxs + wk.pad) * ntot + j] = (float)S.ay[e];
                fpart[((size_t)2 * maxs + wk.pad) * ntot + j] = (float)S.az[e];
            }
        }
        __syncthreads();
    }
    for (int o = 32; o > 0; o >>= 1)
        near += __shfl_xor(near, o);
    if (lane == 0 && near)
        atomicAdd((unsigned long long *)&ec.stats->near_pairs, (unsigned long long)near);
}

// ----------------------------------------------------------------------------
// Persistent step launch: one workgroup owns one system and runs `nsteps`
// whole hybrid steps K S D C S F K without leaving the kernel (all phases at
// workgroup scope, separated by workgroup barriers).  Systems are handed out
// largest first.  FP64 pair arithmetic; every sum has a fixed order, so runs
// are bit-reproducible (the order differs from the per-phase launches, so the
// two paths agree to rounding, not bit for bit).
// ----------------------------------------------------------------------------
constexpr int kPJ = 256;    // sources staged in LDS per tile

template <int NT, int W>
__device__ __forceinline__ void pblock_sum(double (&v)[W], double *sh)
{
    const int t = threadIdx.x;
#pragma unroll
    for (int w = 0; w < W; ++w)
        sh[w * NT + t] = v[w];
    __syncthreads();
    for (int st = NT / 2; st > 0; st >>= 1) {
        if (t < st) {
#pragma unroll
            for (int w = 0; w < W; ++w)
                sh[w * NT + t] += sh[w * NT + t + st];
        }
        __syncthreads();
    }
#pragma unroll
    for (int w = 0; w < W; ++w)
        v[w] = sh[w * NT];
    __syncthreads();
}

// Sum of m V over the workgroup's system (each thread walks its own bodies).
template <int NT>
__device__ __forceinline__ void psys_momentum(int a, int n, const double *__restrict__ m,
                                              const double *vx, const double *vy,
                                              const double *vz, double (&P)[3], double *sh)
{
    P[0] = P[1] = P[2] = 0.0;
    for (int i = a + (int)threadIdx.x; i < a + n; i += NT) {
        double mi = m[i];
        P[0] += mi * vx[i];
        P[1] += mi * vy[i];
        P[2] += mi * vz[i];
    }
    pblock_sum<NT, 3>(P, sh);
}

template <int NT>
__device__ __forceinline__ void pkick(int a, int n, double h, double mm, const double (&P)[3],
                                      int drag, const DragP &dp, const double *__restrict__ m,
                                      const double *qx, const double *qy, const double *qz,
                                      const double *ax, const double *ay, const double *az,
                                      double *vx, double *vy, double *vz)
{
    for (int i = a + (int)threadIdx.x; i < a + n; i += NT) {
        double a0 = ax[i], a1 = ay[i], a2 = az[i];
        double u0 = vx[i], u1 = vy[i], u2 = vz[i];
        if (drag) {
            double d0, d1, d2;
            drag_accel(dp, mm, m[i], qx[i], qy[i], qz[i], u0 + P[0] / mm, u1 + P[1] / mm,
                       u2 + P[2] / mm, d0, d1, d2);
            a0 += d0;
            a1 += d1;
            a2 += d2;
        }
        vx[i] = u0 + h * a0;
        vy[i] = u1 + h * a1;
        vz[i] = u2 + h * a2;
    }
}

// Encounter record staged in LDS by the persistent launch.
struct PRec {
    double4 M;              // chord midpoint and reach
    double q0[3], v0[3], q1[3], v1[3];
    double rc, pad;
};
static_assert(sizeof(PRec) % sizeof(double) == 0, "PRec must be a whole number of doubles");

template <int NT>
__global__ __launch_bounds__(NT) void k_steps_persistent(
    const PSys *__restrict__ psys, int nsteps, double dt, double G, double n_hill, double inner,
    int drag, DragP dp, const double *__restrict__ m0, const double *__restrict__ m, double *qx,
    double *qy, double *qz, double *vx, double *vy, double *vz, double *ax, double *ay,
    double *az, double *rc, double *q0x, double *q0y, double *q0z, double *v0x, double *v0y,
    double *v0z, int *kflag, int *ce, double4 *mr, unsigned long long *keys, int cap,
    DevStats *stats, int *step_nce)
{
    // one LDS buffer, viewed per phase: block sums, encounter tile, force tile
    constexpr int kRecWords = (int)(sizeof(PRec) / sizeof(double));
    constexpr int kWords = (3 * NT > kPJ * kRecWords ? 3 * NT : kPJ * kRecWords);
    static_assert(kWords >= 2 * 4 * kPJ, "force tile must fit the buffer");
    __shared__ double lds[kWords];
    double *sh = lds;
    PRec *se = reinterpret_cast<PRec *>(lds);
    double4 *sj = reinterpret_cast<double4 *>(lds);
    double4 *sx = reinterpret_cast<double4 *>(lds) + kPJ;
    const PSys S = psys[blockIdx.x];
    const int a = S.start, n = S.n, nb = S.nbig, t = threadIdx.x, lane = t & 63;
    const int wave0 = t & ~63;             // first thread index of this wave
    const double mm = m0[S.sys], mu = G * mm, h = 0.5 * dt;
    const double t2 = 2.0 * dt, k427 = 4.0 / 27.0;
    for (int step = 0; step < nsteps; ++step) {
        const bool last = step == nsteps - 1;
        double P[3] = {0.0, 0.0, 0.0};
        // K(h); with drag the heliocentric velocity needs the current sum m V
        if (drag)
            psys_momentum<NT>(a, n, m, vx, vy, vz, P, sh);
        pkick<NT>(a, n, h, mm, P, drag, dp, m, qx, qy, qz, ax, ay, az, vx, vy, vz);
        // S(h)
        psys_momentum<NT>(a, n, m, vx, vy, vz, P, sh);
        for (int i = a + t; i < a + n; i += NT) {
            qx[i] += h * P[0] / mm;
            qy[i] += h * P[1] / mm;
            qz[i] += h * P[2] / mm;
        }
        // D(dt): snapshot, drift, failure flags, encounter reach, cleared flags
        int nf = 0;
        for (int i = a + t; i < a + n; i += NT) {
            double x = qx[i], y = qy[i], z = qz[i], u = vx[i], v = vy[i], w = vz[i];
            q0x[i] = x; q0y[i] = y; q0z[i] = z;
            v0x[i] = u; v0y[i] = v; v0z[i] = w;
            const double x0 = x, y0 = y, z0 = z, u0 = u, v0 = v, w0 = w;
            const bool fail = kepler_drift(mu, dt, x, y, z, u, v, w) != 0;
            nf += fail;
            qx[i] = x; qy[i] = y; qz[i] = z;
            vx[i] = u; vy[i] = v; vz[i] = w;
            kflag[i] = fail ? 1 : 0;
            ce[i] = 0;
            double cx = x - x0, cy = y - y0, cz = z - z0;
            double rho = 0.5 * sqrt(cx * cx + cy * cy + cz * cz);
            double ex0 = dt * u0 - cx, ey0 = dt * v0 - cy, ez0 = dt * w0 - cz;
            double ex1 = dt * u - cx, ey1 = dt * v - cy, ez1 = dt * w - cz;
            double eps = sqrt(fmax(ex0 * ex0 + ey0 * ey0 + ez0 * ez0, ex1 * ex1 + ey1 * ey1 + ez1 * ez1));
            double R = (2.0 * rho + 0.75 * eps + rc[i]) * (1.0 + 0x1p-20);
            mr[i] = make_double4(x0 + 0.5 * cx, y0 + 0.5 * cy, z0 + 0.5 * cz, R);
        }
        for (int o = 32; o > 0; o >>= 1)
            nf += __shfl_xor(nf, o);
        if (lane == 0 && nf)
            atomicAdd((unsigned long long *)&stats->kepler_fail, (unsigned long long)nf);
        double P2[3];
        psys_momentum<NT>(a, n, m, vx, vy, vz, P2, sh);   // also orders the drift's writes
        // C: ordered pairs (i, j) with i < j tested when i + j is even, i > j when
        // odd, so each unordered pair is tested once and every thread sees all j.
        for (int i0 = 0; i0 < n; i0 += NT) {
            const bool vi = i0 + t < n;
            const bool wave_on = i0 + wave0 < n;
            const int i = a + (vi ? i0 + t : 0);
            const double4 Mi = mr[i];
            const double a0[3] = {q0x[i], q0y[i], q0z[i]}, b0[3] = {v0x[i], v0y[i], v0z[i]};
            const double a1[3] = {qx[i], qy[i], qz[i]}, b1[3] = {vx[i], vy[i], vz[i]};
            const double rci = rc[i];
            for (int j0 = 0; j0 < n; j0 += kPJ) {
                const int cnt = min(kPJ, n - j0);
                __syncthreads();
                for (int k = t; k < cnt; k += NT) {
                    const int j = a + j0 + k;
                    PRec r;
                    r.M = mr[j];
                    r.q0[0] = q0x[j]; r.q0[1] = q0y[j]; r.q0[2] = q0z[j];
                    r.v0[0] = v0x[j]; r.v0[1] = v0y[j]; r.v0[2] = v0z[j];
                    r.q1[0] = qx[j];  r.q1[1] = qy[j];  r.q1[2] = qz[j];
                    r.v1[0] = vx[j];  r.v1[1] = vy[j];  r.v1[2] = vz[j];
                    r.rc = rc[j];
                    r.pad = 0.0;
                    se[k] = r;
                }
                __syncthreads();
                if (!wave_on)
                    continue;
                for (int jj = 0; jj < cnt; ++jj) {
                    const int j = a + j0 + jj;
                    const PRec &J = se[jj];
                    double dx = J.M.x - Mi.x, dy = J.M.y - Mi.y, dz = J.M.z - Mi.z;
                    double D2 = fma(dz, dz, fma(dy, dy, dx * dx));
                    double Sr = Mi.w + J.M.w;
                    // two small bodies (both at or past a + nb) never interact
                    bool mine = vi && j != i && ((i < j) == (((i + j) & 1) == 0)) &&
                                min(i, j) < a + nb;
                    bool cand = mine && D2 <= Sr * Sr;
                    if (!__any(cand))
                        continue;
                    bool hit = false;
                    if (cand) {
                        double d0x = J.q0[0] - a0[0], d0y = J.q0[1] - a0[1], d0z = J.q0[2] - a0[2];
                        double d1x = J.q1[0] - a1[0], d1y = J.q1[1] - a1[1], d1z = J.q1[2] - a1[2];
                        double e0x = J.v0[0] - b0[0], e0y = J.v0[1] - b0[1], e0z = J.v0[2] - b0[2];
                        double e1x = J.v1[0] - b1[0], e1y = J.v1[1] - b1[1], e1z = J.v1[2] - b1[2];
                        double f0 = fma(d0z, d0z, fma(d0y, d0y, d0x * d0x));
                        double f1 = fma(d1z, d1z, fma(d1y, d1y, d1x * d1x));
                        double g0 = t2 * fma(d0z, e0z, fma(d0y, e0y, d0x * e0x));
                        double g1 = t2 * fma(d1z, e1z, fma(d1y, e1y, d1x * e1x));
                        double lower = fmin(f0, f1) - k427 * (fmax(0.0, -g0) + fmax(0.0, g1));
                        double rcij = fmax(rci, J.rc);
                        double thr = rcij * rcij;
                        if (lower <= thr * (1.0 + 1e-6) + 1e-15 * (f0 + f1 + fabs(g0) + fabs(g1)))
                            hit = hermite_min(f0, f1, g0, g1) <= thr;
                    }
                    const unsigned long long mask = __ballot(hit);
                    if (mask) {
                        const int leader = __ffsll((long long)mask) - 1;
                        if (lane == leader)
                            atomicAdd(&step_nce[step], (int)__popcll(mask));
                        if (last) {
                            int base = 0;
                            if (lane == leader)
                                base = atomicAdd(&stats->cur_nce, (int)__popcll(mask));
                            base = __shfl(base, leader);
                            if (hit) {
                                const int pos = base + (int)__popcll(mask & ((1ull << lane) - 1ull));
                                const unsigned lo = (unsigned)min(i, j), hi = (unsigned)max(i, j);
                                if (pos < cap)
                                    keys[pos] = ((unsigned long long)lo << 32) | hi;
                            }
                        }
                        if (hit) {
                            __hip_atomic_store(&ce[i], 2, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
                            __hip_atomic_store(&ce[j], 2, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
                        }
                    }
                }
            }
        }
        __syncthreads();
        // S(h) and the critical radii at the new positions
        for (int i = a + t; i < a + n; i += NT) {
            double x = qx[i] + h * P2[0] / mm, y = qy[i] + h * P2[1] / mm, z = qz[i] + h * P2[2] / mm;
            qx[i] = x;
            qy[i] = y;
            qz[i] = z;
            rc[i] = n_hill * sqrt(x * x + y * y + z * z) * cbrt(m[i] / (3.0 * mm));
        }
        __syncthreads();
        // F: each thread sums its targets over every big source, tile by tile in order
        for (int i0 = 0; i0 < n; i0 += NT) {
            const bool vi = i0 + t < n;
            const bool wave_on = i0 + wave0 < n;
            const int i = a + (vi ? i0 + t : 0);
            const double xi = qx[i], yi = qy[i], zi = qz[i], rci = rc[i];
            const double r2i = fmax(rci * rci, DBL_MIN);
            double sx0 = 0.0, sy0 = 0.0, sz0 = 0.0;
            for (int j0 = 0; j0 < nb; j0 += kPJ) {
                const int cnt = min(kPJ, nb - j0);
                __syncthreads();
                for (int k = t; k < cnt; k += NT) {
                    const int j = a + j0 + k;
                    const double mj = m[j], rj = rc[j];
                    sj[k] = make_double4(qx[j], qy[j], qz[j], mj);
                    sx[k] = make_double4(1.5 * mj, rj, fmax(rj * rj, DBL_MIN), 0.0);
                }
                __syncthreads();
                if (!wave_on)
                    continue;
#pragma unroll 2
                for (int jj = 0; jj < cnt; ++jj) {
                    const double4 J = sj[jj];
                    const double4 X = sx[jj];
                    double dx = J.x - xi, dy = J.y - yi, dz = J.z - zi;
                    double r2 = fma(dz, dz, fma(dy, dy, dx * dx));
                    double w = m_rinv3(J.w, X.x, r2);
                    if (r2 < fmax(r2i, X.z))
                        w = J.w * changeover_w(r2, fmax(rci, X.y), inner);
                    sx0 = fma(w, dx, sx0);
                    sy0 = fma(w, dy, sy0);
                    sz0 = fma(w, dz, sz0);
                }
            }
            if (vi) {
                ax[i] = G * sx0;
                ay[i] = G * sy0;
                az[i] = G * sz0;
            }
        }
        __syncthreads();
        // K(h)
        if (drag)
            psys_momentum<NT>(a, n, m, vx, vy, vz, P, sh);
        pkick<NT>(a, n, h, mm, P, drag, dp, m, qx, qy, qz, ax, ay, az, vx, vy, vz);
        __syncthreads();
    }
}

// Small systems (at most kSmallMax bodies): a workgroup owns a system for many
// steps with every quantity on the chip: thread t keeps body t's state in
// registers, the pair phases read LDS.  As launches, a step of 100 bodies is five
// kernels of 3-7 us and the check's three beside them, each a single workgroup
// waiting for memory; here a step is three barriers.
//   body phase   kick, S(h), Kepler drift, the check's records to LDS, sum of m V
//   barrier      second S(h), critical radii, positions to LDS
//   barrier      pair phase: the NT threads are up to floor(NT / n) slices of the
//                sources for every target: FP64 pair sums; each unordered pair
//                once (j = i + k mod n, k <= n/2) through the FP32 filter of the
//                check, survivors through the exact test
//   barrier      each target's slice sums in slice order, closing kick
// Arithmetic of the per-phase kernels (FP64 pairs also for FP32C contexts); the
// last step leaves the drift outputs, flags and list the per-phase steps leave.
// Bound by latency: the Kepler solve's serial chain, then barriers and LDS reads.
// A step: 64 bodies 31 -> 5.9 us, 100 bodies 32 -> 8.8 us, 200 bodies 34 -> 20.7 us.
constexpr int kSmallSlices = 8;       // most slices (their sums are added one by one)

struct SmallArgs {
    const PSys *psys;
    int nsteps, drag, fp32c, unordered;   // unordered: near pairs counted once per pair
    double dt, G, n_hill, inner;
    DragP dp;
    const double *m0, *m;
    double *qx, *qy, *qz, *vx, *vy, *vz, *ax, *ay, *az, *rc;
    double *q0x, *q0y, *q0z, *v0x, *v0y, *v0z, *q1x, *q1y, *q1z, *v1x, *v1y, *v1z, *rc1;
    v8h *eq;
    const unsigned long long *scale;
    int *kflag, *ce;
    unsigned long long *keys;
    int cap;
    DevStats *stats;
    int *step_nce;
    double *mom;                          // per-block sums of m V: the first S(h)'s, replaced by the last step's
    const int *rb_first, *rb_count;
};

template <int NT, int NMAX>
__global__ __launch_bounds__(NT) void k_steps_small(SmallArgs A)
{
    static_assert(NMAX <= NT && NMAX % 64 == 0, "a thread per body");
    // sources: position and mass; rc and widened rc^2 (the zone test's superset)
    __shared__ double4 sj[NMAX];
    __shared__ double sr[NMAX], sw[NMAX];
    __shared__ double part[3][NT];
    __shared__ double red[3][NT / 64];
    __shared__ float4 em[NMAX], ec[NMAX];
    __shared__ double ex[13][NMAX];       // exact test: q0, v0, q1, v1, rc
    const PSys S = A.psys[blockIdx.x];
    const int a = S.start, n = S.n, nb = S.nbig, t = threadIdx.x, lane = t & 63, wv = t >> 6;
    const bool on = t < n;
    const int i = a + (on ? t : 0);
    const double mm = A.m0[S.sys], mu = A.G * mm, dt = A.dt, h = 0.5 * dt;
    // pair phase: target ti, slice sl of nsl
    const int nsl = min(NT / n, kSmallSlices), sl = t / n, ti = t - sl * n;
    const bool work = sl < nsl;
    double x = A.qx[i], y = A.qy[i], z = A.qz[i], u = A.vx[i], v = A.vy[i], w = A.vz[i];
    double ax = A.ax[i], ay = A.ay[i], az = A.az[i], rc = A.rc[i];
    const double mi = on ? A.m[i] : 0.0;
    const double hill = cbrt(mi / (3.0 * mm)), inv_l = enc_inv_scale(A.scale[S.sys]);
    const bool big = t < nb;
    double P[3] = {0.0, 0.0, 0.0};
    for (int b = 0; b < A.rb_count[S.sys]; ++b)
        for (int k = 0; k < 3; ++k)
            P[k] += A.mom[4 * (size_t)(A.rb_first[S.sys] + b) + k];
    int near = 0, nf = 0;
    // sum of m V (one barrier; every thread returns it; a second one before the next)
    auto momentum = [&](double (&out)[3]) {
        double p[3] = {mi * u, mi * v, mi * w};
#pragma unroll
        for (int k = 0; k < 3; ++k)
            p[k] = wave_sum(p[k]);
        if (lane == 0)
            for (int k = 0; k < 3; ++k)
                red[k][wv] = p[k];
        __syncthreads();
        for (int k = 0; k < 3; ++k) {
            out[k] = red[k][0];
            for (int q = 1; q < (n + 63) / 64; ++q)
                out[k] += red[k][q];
        }
    };
    auto kick = [&](const double (&Pk)[3]) {
        double a0 = ax, a1 = ay, a2 = az;
        if (A.drag) {
            double d0, d1, d2;
            drag_accel(A.dp, mm, mi, x, y, z, u + Pk[0] / mm, v + Pk[1] / mm, w + Pk[2] / mm, d0, d1, d2);
            a0 += d0;
            a1 += d1;
            a2 += d2;
        }
        u = fma(h, a0, u);
        v = fma(h, a1, v);
        w = fma(h, a2, w);
    };
    for (int step = 0; step < A.nsteps; ++step) {
        const bool last = step == A.nsteps - 1;
        // with drag the kick needs the current momentum, and so does S(h) after it
        if (A.drag) {
            momentum(P);
            __syncthreads();
        }
        if (on)
            kick(P);
        if (A.drag) {
            momentum(P);
            __syncthreads();
        }
        if (on) {
            x += h * P[0] / mm;
            y += h * P[1] / mm;
            z += h * P[2] / mm;
            const double x0 = x, y0 = y, z0 = z, u0 = u, v0 = v, w0 = w;
            const bool fail = kepler_drift(mu, dt, x, y, z, u, v, w) != 0;
            nf += fail;
            const double cx = x - x0, cy = y - y0, cz = z - z0;
            const double rho = 0.5 * sqrt(cx * cx + cy * cy + cz * cz);
            const double ax0 = dt * u0 - cx, ay0 = dt * v0 - cy, az0 = dt * w0 - cz;
            const double ax1 = dt * u - cx, ay1 = dt * v - cy, az1 = dt * w - cz;
            const double eps = sqrt(fmax(ax0 * ax0 + ay0 * ay0 + az0 * az0, ax1 * ax1 + ay1 * ay1 + az1 * az1));
            const double mx = x0 + 0.5 * cx, my = y0 + 0.5 * cy, mz = z0 + 0.5 * cz;
            const double e34 = 0.75 * eps * (1.0 + 0x1p-20) +
                               0x1p-45 * (sqrt(mx * mx + my * my + mz * mz) + 2.0 * rho);
            float4 M, C;
            enc_record32(mx, my, mz, cx, cy, cz, e34, rc, big, M, C);
            em[t] = M;
            ec[t] = C;
            ex[0][t] = x0; ex[1][t] = y0; ex[2][t] = z0;
            ex[3][t] = u0; ex[4][t] = v0; ex[5][t] = w0;
            ex[6][t] = x;  ex[7][t] = y;  ex[8][t] = z;
            ex[9][t] = u;  ex[10][t] = v; ex[11][t] = w;
            ex[12][t] = rc;
            if (last) {
                A.q0x[i] = x0; A.q0y[i] = y0; A.q0z[i] = z0;
                A.v0x[i] = u0; A.v0y[i] = v0; A.v0z[i] = w0;
                A.q1x[i] = x;  A.q1y[i] = y;  A.q1z[i] = z;
                A.v1x[i] = u;  A.v1y[i] = v;  A.v1z[i] = w;
                A.rc1[i] = rc;
                const double c3[3] = {cx, cy, cz}, e0[3] = {u0, v0, w0}, e1[3] = {u, v, w};
                double d[3];
                const double p = enc_deviation(dt, e0, e1, c3, d);
                enc_record(mx, my, mz, cx, cy, cz, d,
                           0.75 * p + rc + 0x1p-45 * (norm1(mx, my, mz) + norm1(cx, cy, cz)), inv_l,
                           A.eq + kEncRec * (size_t)i);
                A.kflag[i] = fail ? 1 : 0;
                A.ce[i] = 0;
            }
        }
        momentum(P);
        if (on) {
            x += h * P[0] / mm;
            y += h * P[1] / mm;
            z += h * P[2] / mm;
            rc = A.n_hill * sqrt(x * x + y * y + z * z) * hill;
            sj[t] = make_double4(x, y, z, mi);
            sr[t] = rc;
            // FP32C contexts count the pairs inside the radius their kernels widen
            const double r2 = rc * rc;
            sw[t] = A.fp32c ? fmax(r2 * (1.0 + 0x1p-9), 0x1p-80) : fmax(r2, DBL_MIN);
        }
        __syncthreads();
        if (work) {
            // C: pairs (ti, ti + k mod n), the slice's share of k = 1 .. n/2, kU of
            // them at a time (their LDS reads and chains overlap)
            constexpr int kU = 4;
            const int half = n / 2, k1 = 1 + (sl + 1) * half / nsl;
            const float4 Mi = em[ti], Ci = ec[ti];
            const float wi = fabsf(Mi.w);
            for (int k0 = 1 + sl * half / nsl; k0 < k1; k0 += kU) {
                unsigned cand = 0u;
#pragma unroll
                for (int q = 0; q < kU; ++q) {
                    int j = ti + min(k0 + q, k1 - 1);
                    j = j >= n ? j - n : j;
                    const float4 E = em[j], F = ec[j];
                    const float dx = E.x - Mi.x, dy = E.y - Mi.y, dz = E.z - Mi.z;
                    const float cx = F.x - Ci.x, cy = F.y - Ci.y, cz = F.z - Ci.z;
                    const float D2 = fmaf(dz, dz, fmaf(dy, dy, dx * dx));
                    const float C2 = fmaf(cz, cz, fmaf(cy, cy, cx * cx));
                    const float Sr = (fabsf(E.w) + wi) + max_nonneg(F.w, Ci.w);
                    cand |= D2 <= fmaf(Sr, Sr, C2) * (2.0f * (1.0f + 0x1p-18f)) ? 1u << q : 0u;
                }
                while (cand) {
                    const int k = k0 + __ffs(cand) - 1;
                    cand &= cand - 1u;
                    int j = ti + k;
                    j = j >= n ? j - n : j;
                    // not two small bodies; for even n the pairs half apart once
                    if (k >= k1 || min(ti, j) >= nb || (2 * k == n && ti >= k))
                        continue;
                    HRec I, J;
#pragma unroll
                    for (int c = 0; c < 3; ++c) {
                        I.q0[c] = ex[c][ti];
                        I.v0[c] = ex[3 + c][ti];
                        I.q1[c] = ex[6 + c][ti];
                        I.v1[c] = ex[9 + c][ti];
                        J.q0[c] = ex[c][j];
                        J.v0[c] = ex[3 + c][j];
                        J.q1[c] = ex[6 + c][j];
                        J.v1[c] = ex[9 + c][j];
                    }
                    I.rc = ex[12][ti];
                    J.rc = ex[12][j];
                    if (!enc_hit(I, J, dt))
                        continue;
                    atomicAdd(&A.step_nce[step], 1);
                    if (last) {
                        const int pos = atomicAdd(&A.stats->cur_nce, 1);
                        const unsigned lo = (unsigned)(a + min(ti, j)), hi = (unsigned)(a + max(ti, j));
                        if (pos < A.cap)
                            A.keys[pos] = ((unsigned long long)lo << 32) | hi;
                        __hip_atomic_store(&A.ce[lo], 2, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
                        __hip_atomic_store(&A.ce[hi], 2, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
                    }
                }
            }
            // F: the slice's share of the big sources, kU at a time with one branch
            // for the rare pairs in the changeover zone (the body itself is not one:
            // a wave meets one of its own bodies in most groups; ordered pairs'
            // counts include it)
            if (!A.unordered && sl == 0 && ti < nb)
                ++near;
            const double xi = sj[ti].x, yi = sj[ti].y, zi = sj[ti].z, wgt = sw[ti];
            double f0 = 0.0, f1 = 0.0, f2 = 0.0;
            const int j1 = (sl + 1) * nb / nsl;
            for (int j0 = sl * nb / nsl; j0 < j1; j0 += kU) {
                double dx[kU], dy[kU], dz[kU], r2[kU], g[kU], mj[kU];
                bool rare = false;
#pragma unroll
                for (int q = 0; q < kU; ++q) {
                    const int j = min(j0 + q, j1 - 1);
                    const double4 J = sj[j];
                    dx[q] = J.x - xi;
                    dy[q] = J.y - yi;
                    dz[q] = J.z - zi;
                    // without weight: the body itself, and past the slice's end
                    mj[q] = j0 + q < j1 && j != ti ? J.w : 0.0;
                    r2[q] = fma(dz[q], dz[q], fma(dy[q], dy[q], dx[q] * dx[q]));
                    g[q] = rinv3(r2[q]);
                    rare |= r2[q] < fmax(wgt, sw[j]) && j != ti;
                }
                if (rare) {
                    for (int q = 0; q < kU && j0 + q < j1; ++q) {
                        const int j = j0 + q;
                        double rq = r2[0], gq;
#pragma unroll
                        for (int e = 1; e < kU; ++e)
                            rq = q == e ? r2[e] : rq;
                        if (!(rq < fmax(wgt, sw[j])) || j == ti)
                            continue;
                        gq = changeover_w(rq, fmax(sr[ti], sr[j]), A.inner);
                        near += !A.unordered || ti < j;
#pragma unroll
                        for (int e = 0; e < kU; ++e)
                            g[e] = q == e ? gq : g[e];
                    }
                }
#pragma unroll
                for (int q = 0; q < kU; ++q) {
                    const double wq = r2[q] > 0.0 ? g[q] * mj[q] : 0.0;
                    f0 = fma(wq, dx[q], f0);
                    f1 = fma(wq, dy[q], f1);
                    f2 = fma(wq, dz[q], f2);
                }
            }
            part[0][t] = f0;
            part[1][t] = f1;
            part[2][t] = f2;
        }
        __syncthreads();
        if (on) {
            ax = part[0][t];
            ay = part[1][t];
            az = part[2][t];
            for (int q = 1; q < nsl; ++q) {
                ax += part[0][t + q * n];
                ay += part[1][t + q * n];
                az += part[2][t + q * n];
            }
            ax *= A.G;
            ay *= A.G;
            az *= A.G;
            kick(P);
        }
    }
    if (on) {
        A.qx[i] = x; A.qy[i] = y; A.qz[i] = z;
        A.vx[i] = u; A.vy[i] = v; A.vz[i] = w;
        A.ax[i] = ax; A.ay[i] = ay; A.az[i] = az;
        A.rc[i] = rc;
    }
    // the momentum the next step's first S(h) takes (drag: it sums its own)
    if (t == 0)
        for (int b = 0; b < A.rb_count[S.sys]; ++b)
            for (int k = 0; k < 3; ++k)
                A.mom[4 * (size_t)(A.rb_first[S.sys] + b) + k] = b ? 0.0 : P[k];
    for (int o = 32; o > 0; o >>= 1) {
        near += __shfl_xor(near, o);
        nf += __shfl_xor(nf, o);
    }
    if (lane == 0 && near)
        atomicAdd((unsigned long long *)&A.stats->near_pairs, (unsigned long long)near);
    if (lane == 0 && nf)
        atomicAdd((unsigned long long *)&A.stats->kepler_fail, (unsigned long long)nf);
}

// Per-step counts of one persistent launch into the run statistics (one workgroup).
__global__ __launch_bounds__(kBlock) void k_step_stats(int *__restrict__ step_nce, int nsteps,
                                                       int cap, DevStats *stats)
{
    __shared__ long long st[kBlock];
    __shared__ int mx[kBlock], ov[kBlock];
    long long tot = 0;
    int mxv = 0, ovc = 0;
    for (int k = threadIdx.x; k < nsteps; k += kBlock) {
        int c = step_nce[k];
        tot += c;
        mxv = max(mxv, c);
        ovc += c > cap;
        step_nce[k] = 0;
    }
    st[threadIdx.x] = tot;
    mx[threadIdx.x] = mxv;
    ov[threadIdx.x] = ovc;
    __syncthreads();
    for (int o = kBlock / 2; o > 0; o >>= 1) {
        if ((int)threadIdx.x < o) {
            st[threadIdx.x] += st[threadIdx.x + o];
            mx[threadIdx.x] = max(mx[threadIdx.x], mx[threadIdx.x + o]);
            ov[threadIdx.x] += ov[threadIdx.x + o];
        }
        __syncthreads();
    }
    if (threadIdx.x == 0) {
        stats->total_nce += st[0];
        stats->max_nce = max(stats->max_nce, mx[0]);
        stats->overflow_steps += ov[0];
    }
}

// Sort the encounter keys (one workgroup, bitonic) and split them into (ice,
// jce); `accumulate`: also fold the count into the run statistics.
constexpr int kSortThreads = 1024;
constexpr int kSortLds = 16384;  // 128 KiB of keys in LDS

// The check's totals: count, largest count and overflowing checks.  The list
// itself stays in append order until it is read (k_enc_sort).
__global__ void k_enc_count(int cap, DevStats *stats)
{
    if (threadIdx.x == 0) {
        const int count = stats->cur_nce;
        stats->total_nce += count;
        if (count > stats->max_nce)
            stats->max_nce = count;
        if (count > cap)
            stats->overflow_steps += 1;
    }
}

__global__ __launch_bounds__(kSortThreads) void k_enc_sort(unsigned long long *keys, int keys_p2,
                                                           int cap, int *__restrict__ ice,
                                                           int *__restrict__ jce, DevStats *stats,
                                                           int accumulate)
{
    __shared__ unsigned long long sk[kSortLds];
    const int t = threadIdx.x;
    const int count = stats->cur_nce;
    const int n = min(count, cap);
    if (t == 0 && accumulate) {
        stats->total_nce += count;
        if (count > stats->max_nce)
            stats->max_nce = count;
        if (count > cap)
            stats->overflow_steps += 1;
    }
    if (n <= 1) {
        if (n == 1 && t == 0) {
            ice[0] = (int)(keys[0] >> 32);
            jce[0] = (int)(keys[0] & 0xffffffffull);
        }
        return;
    }
    int P = 1;
    while (P < n)
        P <<= 1;
    const unsigned long long kMax = ~0ull;
    if (P <= kSortLds) {
        for (int k = t; k < P; k += kSortThreads)
            sk[k] = k < n ? keys[k] : kMax;
        __syncthreads();
        for (int size = 2; size <= P; size <<= 1) {
            for (int stride = size >> 1; stride > 0; stride >>= 1) {
                for (int k = t; k < P; k += kSortThreads) {
                    int l = k ^ stride;
                    if (l > k) {
                        bool up = (k & size) == 0;
                        unsigned long long a = sk[k], b = sk[l];
                        if ((a > b) == up) {
                            sk[k] = b;
                            sk[l] = a;
                        }
                    }
                }
                __syncthreads();
            }
        }
        for (int k = t; k < n; k += kSortThreads) {
            ice[k] = (int)(sk[k] >> 32);
            jce[k] = (int)(sk[k] & 0xffffffffull);
        }
    } else {
        // P <= keys_p2 by construction of the key buffer
        for (int k = n + t; k < P; k += kSortThreads)
            keys[k] = kMax;
        __syncthreads();
        for (int size = 2; size <= P; size <<= 1) {
            for (int stride = size >> 1; stride > 0; stride >>= 1) {
                for (int k = t; k < P; k += kSortThreads) {
                    int l = k ^ stride;
                    if (l > k) {
                        bool up = (k & size) == 0;
                        unsigned long long a = keys[k], b = keys[l];
                        if ((a > b) == up) {
                            keys[k] = b;
                            keys[l] = a;
                        }
                    }
                }
                __threadfence_block();
                __syncthreads();
            }
        }
        for (int k = t; k < n; k += kSortThreads) {
            ice[k] = (int)(keys[k] >> 32);
            jce[k] = (int)(keys[k] & 0xffffffffull);
        }
    }
}

// ----------------------------------------------------------------------------
// Diagnostics (Sec. 2.1.1 energy and momentum routine), FP64 with error-free
// accumulation: per pair work item the double-double sums of m_i m_j / r and of
// (K - 1) m_i m_j / r over the pairs inside the changeover zone; per body block
// kinetic, stellar potential, L and P; then one workgroup per system combines
// them in a fixed order.
//
// Bound by FP64 issue: 3 differences, 3 for r^2, 6 for the reciprocal root, one
// product and 7 for the error-free sum per pair.  K differs from 1 only for the
// few pairs inside rc_ij, so the second error-free sum takes only those pairs'
// differences, found by one compare per pair against the tile's largest rc^2
// and one branch per four sources (a branch per pair left every pair a
// dependent chain of its own).  Items of kDiagJ sources give a system of 16384
// bodies 2080 workgroups.  16384 bodies: 362 -> 139 us.
// ----------------------------------------------------------------------------
constexpr int kDiagU = 4;    // sources per branch

template <bool DIAG>
__device__ __forceinline__ void diag_tile(const double4 *sj, const double *srj, int cnt, int jt, int i,
                                          double xi, double yi, double zi, double rci, double thr,
                                          double inner, dd &acc, dd &chg)
{
    for (int j0 = 0; j0 < cnt; j0 += kDiagU) {
        double r2[kDiagU], y[kDiagU], u[kDiagU];
        bool rare = false;
#pragma unroll
        for (int k = 0; k < kDiagU; ++k) {
            const double4 J = sj[j0 + k];
            const double dx = J.x - xi, dy = J.y - yi, dz = J.z - zi;
            r2[k] = fma(dz, dz, fma(dy, dy, dx * dx));
            y[k] = rsqrt64_acc(r2[k]);
            u[k] = J.w * y[k];
            // on the diagonal only the pairs j > i
            const bool on = !DIAG || jt + j0 + k > i;
            if (DIAG)
                u[k] = on ? u[k] : 0.0;
            rare |= on && r2[k] < thr;
        }
        if (rare) {
#pragma unroll
            for (int k = 0; k < kDiagU; ++k) {
                const double rcij = fmax(rci, srj[j0 + k]);
                if (!(r2[k] > 0.0))
                    u[k] = 0.0;            // coincident bodies
                else if (r2[k] < rcij * rcij && (!DIAG || jt + j0 + k > i))
                    dd_add(chg, u[k] * (changeover_K(r2[k] * y[k], rcij, inner) - 1.0));
            }
        }
#pragma unroll
        for (int k = 0; k < kDiagU; ++k)
            dd_add(acc, u[k]);
    }
}

__global__ __launch_bounds__(kBlock) void k_diag_pairs(const PWork *__restrict__ work,
                                                       const double *__restrict__ qx,
                                                       const double *__restrict__ qy,
                                                       const double *__restrict__ qz,
                                                       const double *__restrict__ m,
                                                       const double *__restrict__ rc, double inner,
                                                       double *__restrict__ dpart)
{
    __shared__ double4 sj[kBlock];
    __shared__ double srj[kBlock];
    __shared__ double sh[4 * kBlock / 64];
    static_assert(kDiagJ <= kBlock, "a diagnostics item's sources are one LDS tile");
    const PWork wk = work[blockIdx.x];
    const int t = threadIdx.x;
    const bool has_i = t < wk.ni;
    const int i = wk.i0 + (has_i ? t : 0);
    const double xi = qx[i], yi = qy[i], zi = qz[i], rci = rc[i], mi = has_i ? m[i] : 0.0;
    // sources past the end, up to a whole group of kDiagU, are massless and far
    // away; the largest rc^2 of the tile, never below DBL_MIN (coincident bodies)
    double tmax = DBL_MIN;
    {
        const bool ok = t < wk.nj;
        const int j = wk.j0 + (ok ? t : 0);
        const double rcj = ok ? rc[j] : 0.0;
        sj[t] = ok ? make_double4(qx[j], qy[j], qz[j], m[j]) : make_double4(1e150, 1e150, 1e150, 0.0);
        srj[t] = rcj;
        tmax = wave_max(fmax(tmax, rcj * rcj));
        if ((t & 63) == 0)
            sh[t >> 6] = tmax;
    }
    __syncthreads();
    double thr = fmax(rci * rci, tmax);
    for (int w = 0; w < kBlock / 64; ++w)
        thr = fmax(thr, sh[w]);
    __syncthreads();
    dd acc = {0.0, 0.0}, chg = {0.0, 0.0};
    const int cnt = (wk.nj + kDiagU - 1) / kDiagU * kDiagU;
    if (wk.j0 < wk.i0 + wk.ni)
        diag_tile<true>(sj, srj, cnt, wk.j0, i, xi, yi, zi, rci, thr, inner, acc, chg);
    else
        diag_tile<false>(sj, srj, cnt, wk.j0, i, xi, yi, zi, rci, thr, inner, acc, chg);
    // m_i times the per-target sums, then a fixed-tree sum of the (hi, lo) parts
    double v[4] = {mi * acc.hi, mi * acc.lo, mi * chg.hi, mi * chg.lo};
    block_sum<4>(v, sh);
    if (t == 0)
        for (int w = 0; w < 4; ++w)
            dpart[(size_t)blockIdx.x * 4 + w] = v[w];
}

__global__ void k_diag_bodies(const RBlk *__restrict__ rblk, const double *__restrict__ m0,
                              const double *__restrict__ m, const double *__restrict__ qx,
                              const double *__restrict__ qy, const double *__restrict__ qz,
                              const double *__restrict__ vx, const double *__restrict__ vy,
                              const double *__restrict__ vz, double *__restrict__ bpart)
{
    __shared__ double sh[8 * kBlock];
    RBlk b = rblk[blockIdx.x];
    int i = b.start + threadIdx.x;
    double v[8] = {0, 0, 0, 0, 0, 0, 0, 0};
    if (i < b.end) {
        double mi = m[i];
        double x = qx[i], y = qy[i], z = qz[i], u = vx[i], w = vy[i], s = vz[i];
        v[0] = 0.5 * mi * (u * u + w * w + s * s);
        v[1] = -m0[b.sys] * mi / sqrt(x * x + y * y + z * z);   // G applied later
        v[2] = mi * (y * s - z * w);
        v[3] = mi * (z * u - x * s);
        v[4] = mi * (x * w - y * u);
        v[5] = mi * u;
        v[6] = mi * w;
        v[7] = mi * s;
    }
    block_sum<8>(v, sh);
    if (threadIdx.x == 0)
        for (int w = 0; w < 8; ++w)
            bpart[(size_t)blockIdx.x * 8 + w] = v[w];
}

// One workgroup per system: thread t takes every kBlock-th partial from t on,
// then the threads' double-double sums are added pairwise in a fixed tree.
// (One thread walking a system's partials in order took 106 us at 16384 bodies:
// one dependent chain of loads and error-free sums; now 7 us.)
__global__ __launch_bounds__(kBlock) void k_diag_final(
    const int *__restrict__ rb_first, const int *__restrict__ rb_count,
    const int *__restrict__ dw_first, const int *__restrict__ dw_count,
    const double *__restrict__ bpart, const double *__restrict__ dpart,
    const double *__restrict__ m0, double G, double *__restrict__ out)
{
    // columns 0-7: the body sums; 8: m m / r; 9: (K - 1) m m / r
    __shared__ dd sh[10][kBlock];
    const int s = blockIdx.x, t = threadIdx.x;
    dd q[10];
    for (int w = 0; w < 10; ++w)
        q[w] = {0.0, 0.0};
    for (int b = rb_first[s] + t, e = rb_first[s] + rb_count[s]; b < e; b += kBlock)
        for (int w = 0; w < 8; ++w)
            dd_add(q[w], bpart[(size_t)b * 8 + w]);
    for (int k = dw_first[s] + t, e = dw_first[s] + dw_count[s]; k < e; k += kBlock) {
        dd_add(q[8], dd{dpart[(size_t)k * 4 + 0], dpart[(size_t)k * 4 + 1]});
        dd_add(q[9], dd{dpart[(size_t)k * 4 + 2], dpart[(size_t)k * 4 + 3]});
    }
    for (int w = 0; w < 10; ++w)
        sh[w][t] = q[w];
    __syncthreads();
    for (int o = kBlock / 2; o > 0; o >>= 1) {
        // the o sums of each column, spread over the workgroup
        for (int k = t; k < 10 * o; k += kBlock) {
            const int w = k / o, e = k % o;
            dd_add(sh[w][e], sh[w][e + o]);
        }
        __syncthreads();
    }
    if (t != 0)
        return;
    for (int w = 0; w < 10; ++w)
        q[w] = sh[w][0];
    const double P0 = q[5].hi + q[5].lo, P1 = q[6].hi + q[6].lo, P2 = q[7].hi + q[7].lo;
    dd base = q[0];
    dd_add(base, G * q[1].hi);
    dd_add(base, G * q[1].lo);
    dd_add(base, (P0 * P0 + P1 * P1 + P2 * P2) / (2.0 * m0[s]));
    dd_add(base, -G * q[8].hi);
    dd_add(base, -G * q[8].lo);
    dd ek = base;
    dd_add(ek, -G * q[9].hi);
    dd_add(ek, -G * q[9].lo);
    double *o = out + (size_t)s * 8;
    o[0] = base.hi + base.lo;
    o[1] = ek.hi + ek.lo;
    o[2] = q[2].hi + q[2].lo;
    o[3] = q[3].hi + q[3].lo;
    o[4] = q[4].hi + q[4].lo;
    o[5] = P0;
    o[6] = P1;
    o[7] = P2;
}

// ----------------------------------------------------------------------------
// launchers
// ----------------------------------------------------------------------------
static inline int cdiv(int a, int b) { return (a + b - 1) / b; }

// Resolver transfers.  k_gather_pairs packs both ends of listed pairs
// [k0, k0 + n) (n capped by the step's count and the list): per pair two
// records of 10 doubles (m0, m, rc, Q0, V0, body index); k_scatter_members
// writes rows of 7 doubles (body index, Q, V) back, skipping rows that are not
// finite (a failed group keeps its drifted state).
__global__ __launch_bounds__(kBlock) void k_gather_pairs(
    const int *__restrict__ ice, const int *__restrict__ jce, int k0, int n, int cap,
    const DevStats *__restrict__ stats, const int *__restrict__ sys_of,
    const double *__restrict__ m0, const double *__restrict__ m, const double *__restrict__ rc,
    const double *__restrict__ q0x, const double *__restrict__ q0y, const double *__restrict__ q0z,
    const double *__restrict__ v0x, const double *__restrict__ v0y, const double *__restrict__ v0z,
    double *__restrict__ out)
{
    const int t = blockIdx.x * kBlock + threadIdx.x;
    const int k = k0 + t;
    if (t >= n || k >= min(stats->cur_nce, cap))
        return;
    const int body[2] = {ice[k], jce[k]};
    for (int e = 0; e < 2; ++e) {
        const int i = body[e];
        double *o = out + 20 * (size_t)t + 10 * e;
        o[0] = m0[sys_of[i]];
        o[1] = m[i];
        o[2] = rc[i];
        o[3] = q0x[i];
        o[4] = q0y[i];
        o[5] = q0z[i];
        o[6] = v0x[i];
        o[7] = v0y[i];
        o[8] = v0z[i];
        o[9] = (double)i;
    }
}

__global__ __launch_bounds__(kBlock) void k_scatter_members(const double *__restrict__ rows, int k,
                                                            int ntot, double *qx, double *qy,
                                                            double *qz, double *vx, double *vy,
                                                            double *vz)
{
    const int t = blockIdx.x * kBlock + threadIdx.x;
    if (t >= k)
        return;
    const double *r = rows + 7 * (size_t)t;
    const double a = r[1], b = r[2], c = r[3], u = r[4], v = r[5], w = r[6];
    const int i = (int)r[0];
    if (!isfinite(a + b + c + u + v + w) || i < 0 || i >= ntot)
        return;
    qx[i] = a;
    qy[i] = b;
    qz[i] = c;
    vx[i] = u;
    vy[i] = v;
    vz[i] = w;
}

hipError_t launch_gather_pairs(const Dev &d, int k0, int n, hipStream_t s)
{
    if (n <= 0)
        return hipSuccess;
    if (n > d.res_cap)
        return hipErrorInvalidValue;
    k_gather_pairs<<<cdiv(n, kBlock), kBlock, 0, s>>>(d.ice, d.jce, k0, n, d.enc_cap, d.stats, d.sys_of,
                                                       d.m0, d.m, d.rc, d.q0x, d.q0y, d.q0z, d.v0x,
                                                       d.v0y, d.v0z, d.res_buf);
    return hipGetLastError();
}

hipError_t launch_scatter_members(const Dev &d, int k, hipStream_t s)
{
    if (k <= 0)
        return hipSuccess;
    if (k > 2 * d.res_cap)
        return hipErrorInvalidValue;
    k_scatter_members<<<cdiv(k, kBlock), kBlock, 0, s>>>(d.res_rows, k, d.ntot, d.qx, d.qy, d.qz,
                                                          d.vx, d.vy, d.vz);
    return hipGetLastError();
}

// Tables of one system of n bodies for a force evaluation without a context:
// the O(N) blocks, the star's mass and the symmetric force's super-tile pairs
// (I <= J of nt super-tiles of ST bodies, row I's items from I nt - I (I - 1) / 2,
// in the layout the context's tables use; the order of the items does not
// change the sums, which the finalize takes in slot order).  Also clears the
// statistics block.
__global__ void k_single_tables(int n, int ST, int nt, double m0v, RBlk *__restrict__ rblk, int nrb,
                                double *__restrict__ m0, FWork *__restrict__ fw,
                                DevStats *__restrict__ stats)
{
    const int t = blockIdx.x * blockDim.x + threadIdx.x;
    if (t < nrb)
        rblk[t] = RBlk{0, t * kBlock, min(n, (t + 1) * kBlock), 0};
    if (t == 0) {
        m0[0] = m0v;
        *stats = DevStats{};
    }
    if (t < nt * nt) {
        const int I = t / nt, J = t % nt;
        if (J >= I) {
            const int at = I * nt - I * (I - 1) / 2 + (J - I);
            fw[at] = FWork{I * ST, min(ST, n - I * ST), J * ST, min(ST, n - J * ST), J, 0,
                           (J * ST) / kBlock, I};
        }
    }
}

hipError_t launch_single_tables(const Dev &d, int ST, int nt, double m0v, hipStream_t s)
{
    const int total = std::max(d.nrb, nt * nt);
    if (total <= 0)
        return hipSuccess;
    k_single_tables<<<cdiv(total, kBlock), kBlock, 0, s>>>(d.ntot, ST, nt, m0v, d.rblk, d.nrb, d.m0,
                                                           d.fwork, d.stats);
    return hipGetLastError();
}

hipError_t launch_fill_i32(int *p, int n, int value, hipStream_t s)
{
    if (n <= 0)
        return hipSuccess;
    k_fill_i32<<<cdiv(n, kBlock), kBlock, 0, s>>>(p, n, value);
    return hipGetLastError();
}

hipError_t launch_validate(const Dev &d, const double *m0, const double *m, const double *x,
                           const double *v, hipStream_t s)
{
    int n = d.ntot > d.nsys ? d.ntot : d.nsys;
    k_validate<<<cdiv(n, kBlock), kBlock, 0, s>>>(d.ntot, d.nsys, m0, m, x, v, d.sys_of, d.off,
                                                   d.nbig, d.flag, d.scale);
    return hipGetLastError();
}

hipError_t launch_to_dh(const Dev &d, const double *x, const double *v, int frame, hipStream_t s)
{
    if (d.nrb == 0)
        return hipSuccess;
    int helio = frame == 0;
    if (helio)
        k_partial_mv<<<d.nrb, kBlock, 0, s>>>(d.rblk, d.m, v, v + d.ntot, v + 2 * (size_t)d.ntot,
                                               d.rpart);
    k_to_dh<<<d.nrb, kBlock, 0, s>>>(d.rblk, d.rb_first, d.rb_count, d.m0, d.rpart, d.ntot, x, v,
                                      helio, d.qx, d.qy, d.qz, d.vx, d.vy, d.vz, d.scale);
    return hipGetLastError();
}

hipError_t launch_from_dh(const Dev &d, double *x, double *v, int frame, hipStream_t s)
{
    if (d.nrb == 0)
        return hipSuccess;
    int helio = frame == 0;
    if (helio)
        k_partial_mv<<<d.nrb, kBlock, 0, s>>>(d.rblk, d.m, d.vx, d.vy, d.vz, d.rpart);
    k_from_dh<<<d.nrb, kBlock, 0, s>>>(d.rblk, d.rb_first, d.rb_count, d.m0, d.rpart, d.ntot,
                                        helio, d.qx, d.qy, d.qz, d.vx, d.vy, d.vz, x, v);
    return hipGetLastError();
}

hipError_t launch_momentum(const Dev &d, double *part, hipStream_t s)
{
    if (d.nrb == 0)
        return hipSuccess;
    k_partial_mv<<<d.nrb, kBlock, 0, s>>>(d.rblk, d.m, d.vx, d.vy, d.vz, part);
    return hipGetLastError();
}

static DragP drag_params(const Params &p)
{
    DragP dp;
    dp.G = p.G;
    dp.sigma0 = p.sigma0;
    dp.h = p.h;
    dp.cd = p.cd;
    dp.rho_p = p.rho_p;
    return dp;
}

hipError_t launch_kick(const Dev &d, const Params &p, double h, hipStream_t s, double *part_in,
                       double *part_out, bool fin)
{
    if (d.nrb == 0)
        return hipSuccess;
    if (!part_out)
        part_out = d.rpart;
    if (p.drag && !part_in) {
        // partial sums of m V before the kick, for the heliocentric velocity
        part_in = d.rpart_drift();
        k_partial_mv<<<d.nrb, kBlock, 0, s>>>(d.rblk, d.m, d.vx, d.vy, d.vz, part_in);
    }
    if (!p.drag)
        part_in = nullptr;
    const int nsl = fin ? fin_slices(d.maxs, 4) : 0;
#define NB_KICK(FP_, NSL_, PART_)                                                                 \
    k_kick<FP_, NSL_><<<d.nrb, kBlock * (NSL_ ? NSL_ : 1), 0, s>>>(                               \
        d.rblk, h, d.m, d.ax, d.ay, d.az, d.vx, d.vy, d.vz, part_out, part_in, d.rb_first,        \
        d.rb_count, d.m0, d.qx, d.qy, d.qz, drag_params(p), PART_, d.ntot, d.maxs, d.nsplit, p.G)
#define NB_KICK_FIN(NSL_)                                                                         \
    do {                                                                                          \
        if (d.fpart32)                                                                            \
            NB_KICK(float, NSL_, d.fpart32);                                                      \
        else                                                                                      \
            NB_KICK(double, NSL_, d.fpart);                                                       \
    } while (0)
    if (nsl == 0)
        NB_KICK(double, 0, nullptr);
    else if (nsl == 1)
        NB_KICK_FIN(1);
    else if (nsl == 2)
        NB_KICK_FIN(2);
    else
        NB_KICK_FIN(4);
#undef NB_KICK_FIN
#undef NB_KICK
    return hipGetLastError();
}

hipError_t launch_sun_drift(const Dev &d, double h, int rcrit, const Params &p, const double *part,
                            double *copy_to, hipStream_t s)
{
    if (d.nrb == 0)
        return hipSuccess;
    const bool pre = h != 0.0 && d.sys_total;
    if (pre)
        k_sys_total<<<d.nsys, kBlock, 0, s>>>(d.rb_first, d.rb_count, part, d.ptot);
    // the FP32C records over the radial order, with its tile bounds
    const bool rs = p.mode == 1 && rcrit && d.force_rsort;
    k_sun_drift<<<d.nrb, kBlock, 0, s>>>(d.rblk, d.rb_first, d.rb_count, d.m0, part, h, d.qx,
                                          d.qy, d.qz, rcrit, d.m, p.n_hill, d.rc,
                                          p.mode == 1 ? d.pk : nullptr, d.tile_rc2, copy_to,
                                          pre ? d.ptot : nullptr, rs ? d.rord : nullptr,
                                          rs ? d.rtb : nullptr);
    return hipGetLastError();
}

hipError_t launch_drift(const Dev &d, const Params &p, double dt, double sun_h,
                        const double *part_in, hipStream_t s, bool fin)
{
    if (d.nrb == 0)
        return hipSuccess;
    const bool pre = sun_h != 0.0 && d.sys_total;
    if (pre)
        k_sys_total<<<d.nsys, kBlock, 0, s>>>(d.rb_first, d.rb_count, part_in, d.ptot);
    const int nsl = fin ? fin_slices(d.maxs, 4) : 0;
#define NB_DRIFT(FP_, NSL_, ISO_, PART_)                                                          \
    k_drift<FP_, NSL_, ISO_><<<d.nrb, kBlock * (NSL_ ? NSL_ : 1), 0, s>>>(                              \
        d.rblk, d.m0, p.G, dt, d.m, d.qx, d.qy, d.qz, d.vx, d.vy, d.vz, d.q0x, d.q0y, d.q0z,      \
        d.v0x, d.v0y, d.v0z, d.kflag, d.stats, d.rpart_drift(), d.rc,                             \
        d.enc_sorted ? d.lnr_part : nullptr, d.q1x, d.q1y, d.q1z, d.v1x, d.v1y, d.v1z, d.rc1,     \
        part_in, sun_h, d.rb_first, d.rb_count, pre ? d.ptot : nullptr, (v8h *)d.eq, d.scale,    \
        d.nce, PART_, d.ntot, d.maxs, d.nsplit, 0.5 * dt)
#define NB_DRIFT_FIN(NSL_)                                                                        \
    do {                                                                                          \
        if (d.fpart32)                                                                            \
            NB_DRIFT(float, NSL_, true, d.fpart32);                                                     \
        else                                                                                      \
            NB_DRIFT(double, NSL_, true, d.fpart);                                                      \
    } while (0)
    if (nsl == 0 && p.resolve)
        NB_DRIFT(double, 0, false, nullptr);
    else if (nsl == 0)
        NB_DRIFT(double, 0, true, nullptr);
    else if (nsl == 1)
        NB_DRIFT_FIN(1);
    else if (nsl == 2)
        NB_DRIFT_FIN(2);
    else
        NB_DRIFT_FIN(4);
#undef NB_DRIFT_FIN
#undef NB_DRIFT
    return hipGetLastError();
}

hipError_t launch_force(const Dev &d, const Params &p, hipStream_t s)
{
    if (d.nfw == 0)
        return hipSuccess;
    if (d.force_sym) {
        // one workgroup of G waves per super-tile pair
        const int grid = std::min(d.nfw, 1 << 22);
#define NB_SYM_ARGS d.fwork, d.nfw, d.qx, d.qy, d.qz, d.m, d.rc, d.fpart, d.ntot, d.maxs, \
                    p.inner, d.stats
#define NB_SYM32_ARGS d.fwork, d.nfw, d.pk, d.qx, d.qy, d.qz, d.m, d.rc, d.fpart32, d.ntot, \
                      d.maxs, p.inner, d.stats
#define NB_RSYM32_ARGS NB_SYM32_ARGS, d.rord, d.rtb, d.rtf, d.off
// G waves on G tile pairs each, or (H_ > 1) H_ waves on one tile pair
#define NB_SYM_GH(R_, G_, H_)                                                                 \
    do {                                                                                      \
        if (p.mode == 1 && d.force_rsort)                                                     \
            k_force32c_sym<R_, G_, true, H_><<<grid, 64 * G_ * H_, 0, s>>>(NB_RSYM32_ARGS);   \
        else if (p.mode == 1)                                                                 \
            k_force32c_sym<R_, G_, false, H_><<<grid, 64 * G_ * H_, 0, s>>>(NB_SYM32_ARGS);   \
        else                                                                                  \
            k_force64_sym<R_, G_, H_><<<grid, 64 * G_ * H_, 0, s>>>(NB_SYM_ARGS);             \
    } while (0)
#define NB_SYM_G(R_, HMAX_)                                                                   \
    do {                                                                                      \
        const int h = std::min(HMAX_, sym_waves(d.nfw, p));                                   \
        if (d.sym_g == 4)                                                                     \
            NB_SYM_GH(R_, 4, 1);                                                              \
        else if (d.sym_g == 2)                                                                \
            NB_SYM_GH(R_, 2, 1);                                                              \
        else if (HMAX_ >= 4 && h == 4)                                                        \
            NB_SYM_GH(R_, 1, (HMAX_ >= 4 ? 4 : 1));                                           \
        else if (HMAX_ >= 2 && h >= 2)                                                        \
            NB_SYM_GH(R_, 1, (HMAX_ >= 2 ? 2 : 1));                                           \
        else                                                                                  \
            NB_SYM_GH(R_, 1, 1);                                                              \
    } while (0)
        if (p.force_r == 1)
            NB_SYM_G(1, 4);
        else if (p.force_r == 4)
            NB_SYM_G(4, 1);
        else
            NB_SYM_G(2, 4);
#undef NB_SYM_G
#undef NB_SYM_GH
#undef NB_SYM_ARGS
#undef NB_RSYM32_ARGS
#undef NB_SYM32_ARGS
        return hipGetLastError();
    }
    if (d.force_few) {
        // one item a wave
        const int grid = std::min(cdiv(d.nfw, kWaves), 1 << 22);
#define NB_FEW_ARGS d.fwork, d.nfw, d.qx, d.qy, d.qz, d.m, d.rc, d.tile_rc2, d.fpart, d.ntot, d.maxs, \
                    p.inner, d.stats
#define NB_FEW32_ARGS d.fwork, d.nfw, d.pk, d.qx, d.qy, d.qz, d.m, d.rc, d.tile_rc2, d.fpart32, d.ntot, \
                      d.maxs, p.inner, d.stats
        if (p.mode == 1) {
            if (p.force_r == 1)
                k_force32c_few<1><<<grid, kBlock, 0, s>>>(NB_FEW32_ARGS);
            else if (p.force_r == 4)
                k_force32c_few<4><<<grid, kBlock, 0, s>>>(NB_FEW32_ARGS);
            else
                k_force32c_few<2><<<grid, kBlock, 0, s>>>(NB_FEW32_ARGS);
        } else {
            if (p.force_r == 1)
                k_force64_few<1><<<grid, kBlock, 0, s>>>(NB_FEW_ARGS);
            else if (p.force_r == 4)
                k_force64_few<4><<<grid, kBlock, 0, s>>>(NB_FEW_ARGS);
            else
                k_force64_few<2><<<grid, kBlock, 0, s>>>(NB_FEW_ARGS);
        }
#undef NB_FEW_ARGS
#undef NB_FEW32_ARGS
        return hipGetLastError();
    }
    if (p.mode == 1) {
        switch (p.force_r) {
        case 1:
            k_force32c<1><<<d.nfw, kBlock, 0, s>>>(d.fwork, d.pk, d.qx, d.qy, d.qz, d.m, d.rc,
                                                    d.tile_rc2, d.fpart32, d.ntot, d.maxs, p.inner, d.stats);
            break;
        case 4:
            k_force32c<4><<<d.nfw, kBlock, 0, s>>>(d.fwork, d.pk, d.qx, d.qy, d.qz, d.m, d.rc,
                                                    d.tile_rc2, d.fpart32, d.ntot, d.maxs, p.inner, d.stats);
            break;
        default:
            k_force32c<2><<<d.nfw, kBlock, 0, s>>>(d.fwork, d.pk, d.qx, d.qy, d.qz, d.m, d.rc,
                                                    d.tile_rc2, d.fpart32, d.ntot, d.maxs, p.inner, d.stats);
        }
    } else {
        switch (p.force_r) {
        case 1:
            k_force64<1><<<d.nfw, kBlock, 0, s>>>(d.fwork, d.qx, d.qy, d.qz, d.m, d.rc,
                                                   d.tile_rc2, d.fpart,
                                                   d.ntot, d.maxs, p.inner, d.stats);
            break;
        case 4:
            k_force64<4><<<d.nfw, kBlock, 0, s>>>(d.fwork, d.qx, d.qy, d.qz, d.m, d.rc,
                                                   d.tile_rc2, d.fpart,
                                                   d.ntot, d.maxs, p.inner, d.stats);
            break;
        default:
            k_force64<2><<<d.nfw, kBlock, 0, s>>>(d.fwork, d.qx, d.qy, d.qz, d.m, d.rc,
                                                   d.tile_rc2, d.fpart,
                                                   d.ntot, d.maxs, p.inner, d.stats);
        }
    }
    return hipGetLastError();
}

hipError_t launch_force_finalize(const Dev &d, const Params &p, double kick_h, int kicks,
                                 hipStream_t s, const int *ord, bool enc_count)
{
    if (d.ntot == 0)
        return hipSuccess;
    // about eight slots per slice at the largest split count; up to kFinDriftSlots at
    // most four slices, the order that the drift launch sums them in inside a run
    // (not over the radial order, whose partials only this kernel sums)
    const bool by4 = d.maxs <= kFinDriftSlots && !d.force_rsort && !ord;
    const int nsl = fin_slices(d.maxs, by4 ? 4 : 16);
    const int grid = cdiv(d.ntot, kFinThreads / nsl), cc = enc_count ? d.enc_cap : -1;
    // the radial order's partials are by position too
    if (!ord && d.force_rsort)
        ord = d.rord;
    if (d.fpart32)
        k_force_finalize<float><<<grid, kFinThreads, 0, s>>>(
            d.sys_of, d.nsplit, d.fpart32, d.ntot, d.maxs, d.ns_all, nsl, p.G, d.ax, d.ay, d.az,
            kick_h, kicks, d.vx, d.vy, d.vz, ord, cc, d.stats);
    else
        k_force_finalize<double><<<grid, kFinThreads, 0, s>>>(
            d.sys_of, d.nsplit, d.fpart, d.ntot, d.maxs, d.ns_all, nsl, p.G, d.ax, d.ay, d.az,
            kick_h, kicks, d.vx, d.vy, d.vz, ord, cc, d.stats);
    return hipGetLastError();
}

// Encounter check in two parts: the gather part bins the drift records and
// copies them into the sorted record array (sorted algorithm only), the test
// part tests pairs.  Both read only what the drift wrote (Q0, V0, the Q1, V1
// and rc copies, the midpoint and chord records), so the whole check may run
// beside the next S(h), force and kick.
hipError_t launch_enc_gather(const Dev &d, double dt, hipStream_t s)
{
    if (d.enc_sorted && d.nrb > 0) {
        k_cells<<<d.nrb, kBlock, 0, s>>>(d.rblk, d.rb_first, d.rb_count, d.lnr_part,
                                          d.sys_cell_base, d.sys_cell_cnt, d.q0x, d.q0y, d.q1x, d.q1y, d.cell_cnt,
                                          d.cell_of, d.slot_of, d.ce);
        const int nchunk = cdiv(d.ncell, kScanChunk);
        if (nchunk <= kScanSerialChunks) {
            k_cell_scan<<<1, kScanThreads, 0, s>>>(d.cell_cnt, d.cell_off, d.ncell, d.stats);
        } else {
            k_scan_sums<<<nchunk, kScanThreads, 0, s>>>(d.cell_cnt, d.ncell, d.scan_part);
            k_scan_apply<<<nchunk, kScanThreads, 0, s>>>(d.cell_cnt, d.cell_off, d.ncell,
                                                         d.scan_part, d.stats);
        }
        k_scatter<<<d.nrb, kBlock, 0, s>>>(d.rblk, d.cell_of, d.slot_of, d.cell_off, d.ord);
        k_cell_order<<<cdiv(d.ncell, kBlock / 64), kBlock, 0, s>>>(d.cell_off, d.ncell, d.ntot, d.ord,
                                                                    d.slot_of);
        k_srec<<<cdiv(d.ntot, kBlock), kBlock, 0, s>>>(d.ntot, d.slot_of, d.sys_of, d.q0x, d.q0y, d.q0z,
                                                       d.v0x, d.v0y, d.v0z, d.q1x, d.q1y, d.q1z,
                                                       d.v1x, d.v1y, d.v1z, d.rc1, d.off,
                                                       d.nbig, d.srec, d.em, d.eg, dt, d.enc_fused);
    }
    return hipGetLastError();
}

hipError_t launch_enc_test(const Dev &d, double dt, hipStream_t s, bool beside)
{
    if (d.enc_sorted) {
        if (d.ntile > 0) {
            k_tile_bounds<<<cdiv(d.ntile, kBlock / 64), kBlock, 0, s>>>(d.tiles, d.ntile, d.srec, dt,
                                                                         d.tileb);
            k_tile_pairs<<<cdiv(d.nunit, kTpWaves), 64 * kTpWaves, 0, s>>>(
                d.tiles, d.units, d.nunit, d.tileb, d.tpairs, d.tp_cap, d.stats);
            // one wave per kept tile pair, at most eight times as many as fit at once: they
            // take turns where pairs differ (steps of a radian, 20011 bodies of a ring: 986
            // us with 4096 waves, 743 with 16384, 707 with 32768)
            // Beside one system's force of one wave per tile pair (Dev::pair_waves), whose
            // workgroups hold most of a compute unit's LDS, single waves slip in wherever a
            // force workgroup ends and take its place; workgroups of four (over the radial
            // order of more than 16384 bodies two) mostly wait for the force's last, partly
            // idle round.  A step with 1 / 2 / 4 waves, disk of 0.5-5 AU: FP64 20011 bodies
            // 233.7 / 221.7 / 220.4 us, 26000 351.1 / 338.7 / 335.6; FP32C 20011 174.4 / 170.1
            // / 166.2, 26000 257.4 / 252.4 / 250.9; over the radial order 15000 101.4 / 103.1 /
            // 104.4, 16384 114.2 / 114.8 / 115.9, 18000 147.7 / 143.2 / 143.0, 26000 239.7 /
            // 235.7 / 241.1.  Beside wider force workgroups and beside a batch single waves are
            // as good or better (FP64 15000 bodies 135.6 / - / 137.3 us, a ring of 131072 in
            // FP32C 4967 / - / 5010 us, four systems of up to 12000 in FP32C 196.4 / - / 203.8 us),
            // and alone they are done sooner (steps of 0.2 yr, 40000 bodies at 1-3 AU, 524 /
            // 569 / 668 us).
            const int w = beside ? d.pair_waves : 1;
            const int grid = std::min(std::max(1, cdiv(d.tp_cap, w)), 32768 / w);
#define NB_ENC_PAIRS(W_)                                                                          \
    k_enc_pairs<W_><<<grid, 64 * W_, 0, s>>>(d.tiles, d.tileb, d.tpairs, d.tp_cap, d.srec, d.em,  \
                                             d.eg, dt, d.keys, d.enc_cap, d.ce, d.stats)
            if (w == 4)
                NB_ENC_PAIRS(4);
            else if (w == 2)
                NB_ENC_PAIRS(2);
            else
                NB_ENC_PAIRS(1);
#undef NB_ENC_PAIRS
        }
    } else if (d.new_ > 0) {
        const EncIn in{d.q0x, d.q0y, d.q0z, d.v0x, d.v0y, d.v0z, d.q1x, d.q1y, d.q1z, d.v1x, d.v1y, d.v1z,
                       d.rc1};
        k_enc_direct<<<d.new_, 64, 0, s>>>(d.ework, (const v8h *)d.eq, in, dt, d.keys, d.enc_cap, d.ce,
                                           &d.stats->cur_nce, kEncFlag, d.scale, d.sys_of);
    }
    k_enc_count<<<1, 64, 0, s>>>(d.enc_cap, d.stats);
    return hipGetLastError();
}

hipError_t launch_enc_prepare(const Dev &d, double dt, hipStream_t s)
{
    // the binning clears the flags, the cell scan the list count
    hipError_t e = launch_enc_gather(d, dt, s);
    if (e == hipSuccess && d.ntile > 0)
        k_tile_bounds<<<cdiv(d.ntile, kBlock / 64), kBlock, 0, s>>>(d.tiles, d.ntile, d.srec, dt,
                                                                     d.tileb);
    return e != hipSuccess ? e : hipGetLastError();
}

hipError_t launch_force_fused(const Dev &d, const Params &p, double dt, int count, hipStream_t s)
{
    if (d.nfw > 0) {
        const int grid = std::min(d.nfw, 1 << 22);
        const EncCtx ec{d.srec, dt, d.keys, d.enc_cap, d.ce, d.stats};
#define NB_FUSED_ARGS d.fwork, d.nfw, d.ord, d.pk, d.em, d.tileb, d.tile_first, d.off, d.qx, d.qy, \
                      d.qz, d.m, d.rc, d.fpart32, d.ntot, d.maxs, p.inner, ec
#define NB_FUSED_G(R_)                                                                        \
    do {                                                                                      \
        if (d.sym_g == 4)                                                                     \
            k_force32c_fused<R_, 4><<<grid, 256, 0, s>>>(NB_FUSED_ARGS);                      \
        else if (d.sym_g == 2)                                                                \
            k_force32c_fused<R_, 2><<<grid, 128, 0, s>>>(NB_FUSED_ARGS);                      \
        else                                                                                  \
            k_force32c_fused<R_, 1><<<grid, 64, 0, s>>>(NB_FUSED_ARGS);                       \
    } while (0)
        if (p.force_r == 1)
            NB_FUSED_G(1);
        else if (p.force_r == 4)
            NB_FUSED_G(4);
        else
            NB_FUSED_G(2);
#undef NB_FUSED_G
#undef NB_FUSED_ARGS
    }
    if (count)
        k_enc_count<<<1, 64, 0, s>>>(d.enc_cap, d.stats);
    return hipGetLastError();
}

hipError_t launch_encounters(const Dev &d, double dt, hipStream_t s, bool beside)
{
    // an empty list and no flags (the check may run beside the next drift, so
    // the drift does not clear them); the sorted check's binning clears the
    // flags and its scan the count
    hipError_t e = hipSuccess;
    if (!(d.enc_sorted && d.nrb > 0)) {
        k_enc_clear<<<cdiv(d.ntot, kBlock), kBlock, 0, s>>>(d.ntot, d.ce, d.stats);
        e = hipGetLastError();
    }
    if (e == hipSuccess)
        e = launch_enc_gather(d, dt, s);
    return e != hipSuccess ? e : launch_enc_test(d, dt, s, beside);
}

hipError_t launch_enc_in_run(const Dev &d, double dt, int set, hipStream_t s)
{
    if (d.new_ == 0)
        return hipSuccess;
    const EncIn in{d.q0x, d.q0y, d.q0z, d.v0x, d.v0y, d.v0z, d.q1x, d.q1y, d.q1z, d.v1x, d.v1y, d.v1z, d.rc1};
    k_enc_direct<<<d.new_, 64, 0, s>>>(d.ework, (const v8h *)d.eq, in, dt, d.keys, d.enc_cap, d.ce,
                                       &d.stats->set_nce[set], kEncTag + set, d.scale, d.sys_of);
    return hipGetLastError();
}

hipError_t launch_enc_run_end(const Dev &d, int nsets, hipStream_t s)
{
    k_enc_run_end<<<cdiv(d.ntot, kBlock), kBlock, 0, s>>>(d.ntot, nsets, d.enc_cap, d.ce, d.stats);
    return hipGetLastError();
}

hipError_t launch_enc_sort(const Dev &d, int accumulate, hipStream_t s)
{
    k_enc_sort<<<1, kSortThreads, 0, s>>>(d.keys, d.keys_p2, d.enc_cap, d.ice, d.jce, d.stats,
                                          accumulate);
    return hipGetLastError();
}

hipError_t launch_persistent_steps(const Dev &d, const Params &p, double dt, int nsteps,
                                   hipStream_t s)
{
    if (d.npsys == 0 || nsteps <= 0)
        return hipSuccess;
    // workgroup size from the largest system (psys[0] after the largest-first order)
#define NB_PERSIST_ARGS                                                                         \
    d.psys, nsteps, dt, p.G, p.n_hill, p.inner, p.drag, drag_params(p), d.m0, d.m, d.qx, d.qy, \
        d.qz, d.vx, d.vy, d.vz, d.ax, d.ay, d.az, d.rc, d.q0x, d.q0y, d.q0z, d.v0x, d.v0y,     \
        d.v0z, d.kflag, d.ce, d.mr, d.keys, d.enc_cap, d.stats, d.step_nce
    // (512 threads at most: 8 waves keep the full register budget without spills)
    if (d.pmax_n <= 128)
        k_steps_persistent<128><<<d.npsys, 128, 0, s>>>(NB_PERSIST_ARGS);
    else if (d.pmax_n <= 256)
        k_steps_persistent<256><<<d.npsys, 256, 0, s>>>(NB_PERSIST_ARGS);
    else
        k_steps_persistent<512><<<d.npsys, 512, 0, s>>>(NB_PERSIST_ARGS);
#undef NB_PERSIST_ARGS
    return hipGetLastError();
}

hipError_t launch_small_steps(const Dev &d, const Params &p, double dt, int nsteps, hipStream_t s)
{
    if (d.npsys == 0 || nsteps <= 0)
        return hipSuccess;
    const SmallArgs A{d.psys, nsteps, p.drag, p.mode == 1, d.force_sym, dt, p.G, p.n_hill, p.inner,
                      drag_params(p), d.m0, d.m, d.qx, d.qy, d.qz, d.vx, d.vy, d.vz, d.ax, d.ay,
                      d.az, d.rc, d.q0x, d.q0y, d.q0z, d.v0x, d.v0y, d.v0z, d.q1x, d.q1y, d.q1z,
                      d.v1x, d.v1y, d.v1z, d.rc1, (v8h *)d.eq, d.scale, d.kflag, d.ce, d.keys,
                      d.enc_cap, d.stats, d.step_nce, d.rpart_prev(), d.rb_first, d.rb_count};
    // 512 threads keep the whole state in registers; above 128 bodies the pair phase
    // is longer than what the 1024 threads' spills cost (100 bodies 8.8 / 11.4 us a
    // step, 200 bodies 25.8 / 20.7 us)
    if (d.pmax_n <= 128)
        k_steps_small<512, 128><<<d.npsys, 512, 0, s>>>(A);
    else
        k_steps_small<1024, kSmallMax><<<d.npsys, 1024, 0, s>>>(A);
    return hipGetLastError();
}

hipError_t launch_step_stats(const Dev &d, int nsteps, hipStream_t s)
{
    k_step_stats<<<1, kBlock, 0, s>>>(d.step_nce, nsteps, d.enc_cap, d.stats);
    return hipGetLastError();
}

// ----------------------------------------------------------------------------
// Collisions, star impacts, ejections and the removal of lost bodies (Sec.
// 2.1.1: physical radii, removal of lost bodies from the arrays; Sec. 2.1.2:
// planet-planet and planet-star collisions, ejections of bodies far from the
// star).  The paper gives the events and their schedule, not their arithmetic;
// the readings: physical radius R = (3 m/(4 pi rho))^(1/3); a star impact when
// the step's Kepler arc comes within r_star of the star (its mass joins the
// star, whose centre moves to the centre of mass of star and impactors); a
// collision when a flagged pair's minimum separation over the step (the
// encounter predicate's Hermite minimum) is at most R_i + R_j, bodies joined
// by colliding pairs merging perfectly into the smallest index; an ejection
// beyond r_eject, the body leaving with its momentum.  Applied in that order,
// on the state at the end of the step.  Lost bodies keep their slot with
// m = 0 and a nonzero flag until the compaction.
// ----------------------------------------------------------------------------
// Closest approach to the star along the Kepler arc of duration tau from
// (q0, v0) to (q1, v1), mu = G m0: the nearer end, or the pericentre distance
// h^2/(mu (1 + e)) when the arc passes a pericentre (bound orbits: a multiple
// of 2 pi between the mean anomalies at the ends; unbound orbits: the radial
// velocity changes sign from inward to outward along the direction of time).
__device__ double star_min_dist(double mu, double tau, const double (&q0)[3], const double (&v0)[3],
                                const double (&q1)[3], const double (&v1)[3])
{
    const double r0 = sqrt(q0[0] * q0[0] + q0[1] * q0[1] + q0[2] * q0[2]);
    const double r1 = sqrt(q1[0] * q1[0] + q1[1] * q1[1] + q1[2] * q1[2]);
    double rmin = fmin(r0, r1);
    const double eta0 = q0[0] * v0[0] + q0[1] * v0[1] + q0[2] * v0[2];
    const double eta1 = q1[0] * v1[0] + q1[1] * v1[1] + q1[2] * v1[2];
    const double hx = q0[1] * v0[2] - q0[2] * v0[1];
    const double hy = q0[2] * v0[0] - q0[0] * v0[2];
    const double hz = q0[0] * v0[1] - q0[1] * v0[0];
    const double h2 = hx * hx + hy * hy + hz * hz;
    const double vv = v0[0] * v0[0] + v0[1] * v0[1] + v0[2] * v0[2];
    const double alpha = 2.0 / r0 - vv / mu;        // 1/a
    const double e2 = 1.0 - h2 * alpha / mu;
    const double e = sqrt(fmax(e2, 0.0));
    bool passed;
    if (alpha > 0.0) {
        const double twopi = 6.283185307179586;
        const double esinE = eta0 * sqrt(alpha / mu), ecosE = 1.0 - r0 * alpha;
        const double M0 = atan2(esinE, ecosE) - esinE;
        const double M1 = M0 + sqrt(mu * alpha * alpha * alpha) * tau;
        const double lo = fmin(M0, M1), hi = fmax(M0, M1);
        passed = floor(hi / twopi) * twopi >= lo;
    } else {
        passed = tau >= 0.0 ? (eta0 < 0.0 && eta1 >= 0.0) : (eta1 < 0.0 && eta0 >= 0.0);
    }
    if (passed)
        rmin = fmin(rmin, h2 / (mu * (1.0 + e)));
    return rmin;
}

// Star impacts, per body: lost = 1 when the arc reaches r_star (r_star > 0);
// every flag cleared otherwise and every union-find parent set to the body.
// Per-block sums of the impactors' m, m Q and count into part (8 per block).
__global__ void k_ev_star(const RBlk *__restrict__ rblk, const double *__restrict__ m0, double G,
                          double tau, Snap a, const double *__restrict__ m,
                          const double *__restrict__ qx, const double *__restrict__ qy,
                          const double *__restrict__ qz, double r_star, int *__restrict__ lost,
                          int *__restrict__ root, double *__restrict__ part)
{
    __shared__ double sh[8 * kBlock / 64];
    const RBlk b = rblk[blockIdx.x];
    const int i = b.start + threadIdx.x;
    double w[5] = {0.0, 0.0, 0.0, 0.0, 0.0};
    if (i < b.end) {
        int flag = 0;
        if (r_star > 0.0) {
            const double q0[3] = {a.q0x[i], a.q0y[i], a.q0z[i]}, v0[3] = {a.v0x[i], a.v0y[i], a.v0z[i]};
            const double q1[3] = {a.q1x[i], a.q1y[i], a.q1z[i]}, v1[3] = {a.v1x[i], a.v1y[i], a.v1z[i]};
            flag = star_min_dist(G * m0[b.sys], tau, q0, v0, q1, v1) <= r_star;
        }
        lost[i] = flag;
        root[i] = i;
        if (flag) {
            const double mi = m[i];
            w[0] = mi;
            w[1] = mi * qx[i];
            w[2] = mi * qy[i];
            w[3] = mi * qz[i];
            w[4] = 1.0;
        }
    }
    block_sum<5>(w, sh);
    if (threadIdx.x < 5)
        part[(size_t)blockIdx.x * 8 + threadIdx.x] = w[threadIdx.x];
}

// One workgroup per system: the impactors join the star (m0 += their mass) and
// the star's centre moves to the centre of mass of star and impactors; the
// shift is kept in sys[8 s .. 8 s + 2] for the bodies.  cnt[0] += impacts.
__global__ void k_ev_star_sys(const int *__restrict__ rb_first, const int *__restrict__ rb_count,
                              const double *__restrict__ part, double *__restrict__ m0,
                              double *__restrict__ sys, int *__restrict__ cnt)
{
    __shared__ double sh[8 * kBlock / 64];
    double t[5];
    system_sum<5>(part + 0, 8, rb_first[blockIdx.x], rb_count[blockIdx.x], t, sh);
    if (threadIdx.x == 0) {
        double *o = sys + (size_t)blockIdx.x * 8;
        o[0] = o[1] = o[2] = 0.0;
        const int k = (int)t[4];
        if (k > 0) {
            const double mnew = m0[blockIdx.x] + t[0];
            o[0] = t[1] / mnew;
            o[1] = t[2] / mnew;
            o[2] = t[3] / mnew;
            m0[blockIdx.x] = mnew;
            atomicAdd(&cnt[0], k);
        }
        o[3] = (double)k;
    }
}

// Impactors lose their mass; every other body of a system with impacts moves
// by minus the star's shift (its heliocentric position is relative to the star).
__global__ void k_ev_star_apply(const RBlk *__restrict__ rblk, const double *__restrict__ sys,
                                const int *__restrict__ lost, double *__restrict__ m,
                                double *__restrict__ qx, double *__restrict__ qy,
                                double *__restrict__ qz)
{
    const RBlk b = rblk[blockIdx.x];
    const int i = b.start + threadIdx.x;
    if (i >= b.end)
        return;
    const double *o = sys + (size_t)b.sys * 8;
    if (o[3] == 0.0)
        return;
    if (lost[i]) {
        m[i] = 0.0;
    } else {
        qx[i] -= o[0];
        qy[i] -= o[1];
        qz[i] -= o[2];
    }
}

__device__ int uf_find(int *root, int i)
{
    while (root[i] != i)
        i = root[i];
    return i;
}

// Collisions among the step's listed pairs (sorted by (i, j); pairs with a
// lost member are skipped).  Every thread tests pairs: the Hermite minimum of
// the step's arcs against (R_i + R_j)^2.  Then thread 0 joins colliding pairs
// (union-find, the smaller root wins), lists the members in index order and
// merges every group into its smallest member: summed mass, mass-weighted
// position and velocity (compensated sums in index order); the others get
// lost = 2 and m = 0.  One workgroup; collisions are rare, and the member
// list is ordered by insertion (quadratic in the members of colliding pairs).
__global__ __launch_bounds__(kBlock) void k_ev_collide(
    const DevStats *__restrict__ stats, int cap, const int *__restrict__ ice,
    const int *__restrict__ jce, double tau, Snap a, double rho, int *__restrict__ lost,
    int *__restrict__ root, int *__restrict__ pflag, int *__restrict__ mem, double *m, double *qx,
    double *qy, double *qz, double *vx, double *vy, double *vz, int *__restrict__ cnt)
{
    const int nce = min(stats->cur_nce, cap);
    const double k3 = 3.0 / (4.0 * 3.141592653589793 * rho);
    const double t2 = 2.0 * tau;
    for (int p = threadIdx.x; p < nce; p += blockDim.x) {
        const int i = ice[p], j = jce[p];
        int hit = 0;
        if (!lost[i] && !lost[j]) {
            const double d0x = a.q0x[j] - a.q0x[i], d0y = a.q0y[j] - a.q0y[i], d0z = a.q0z[j] - a.q0z[i];
            const double d1x = a.q1x[j] - a.q1x[i], d1y = a.q1y[j] - a.q1y[i], d1z = a.q1z[j] - a.q1z[i];
            const double e0x = a.v0x[j] - a.v0x[i], e0y = a.v0y[j] - a.v0y[i], e0z = a.v0z[j] - a.v0z[i];
            const double e1x = a.v1x[j] - a.v1x[i], e1y = a.v1y[j] - a.v1y[i], e1z = a.v1z[j] - a.v1z[i];
            const double f0 = d0x * d0x + d0y * d0y + d0z * d0z;
            const double f1 = d1x * d1x + d1y * d1y + d1z * d1z;
            const double g0 = t2 * (d0x * e0x + d0y * e0y + d0z * e0z);
            const double g1 = t2 * (d1x * e1x + d1y * e1y + d1z * e1z);
            const double rr = cbrt(k3 * m[i]) + cbrt(k3 * m[j]);
            hit = hermite_min(f0, f1, g0, g1) <= rr * rr;
        }
        pflag[p] = hit;
    }
    __syncthreads();
    if (threadIdx.x != 0)
        return;
    int ncoll = 0, nm = 0;
    for (int p = 0; p < nce; ++p) {
        if (!pflag[p])
            continue;
        ++ncoll;
        const int i = ice[p], j = jce[p];
        const int ra = uf_find(root, i), rb = uf_find(root, j);
        if (ra != rb) {
            if (ra < rb)
                root[rb] = ra;
            else
                root[ra] = rb;
        }
        // members in increasing index order, each once
        for (int e = 0; e < 2; ++e) {
            const int b = e ? j : i;
            int k = nm;
            while (k > 0 && mem[k - 1] > b)
                --k;
            if (k > 0 && mem[k - 1] == b)
                continue;
            for (int q = nm; q > k; --q)
                mem[q] = mem[q - 1];
            mem[k] = b;
            ++nm;
        }
    }
    int merged = 0;
    for (int e = 0; e < nm; ++e) {
        const int r = mem[e];
        if (uf_find(root, r) != r)
            continue;
        dd sm{0, 0}, px{0, 0}, py{0, 0}, pz{0, 0}, ux{0, 0}, uy{0, 0}, uz{0, 0};
        for (int f = e; f < nm; ++f) {
            const int b = mem[f];
            if (uf_find(root, b) != r)
                continue;
            const double mb = m[b];
            dd_add(sm, mb);
            dd_add(px, mb * qx[b]);
            dd_add(py, mb * qy[b]);
            dd_add(pz, mb * qz[b]);
            dd_add(ux, mb * vx[b]);
            dd_add(uy, mb * vy[b]);
            dd_add(uz, mb * vz[b]);
        }
        const double M = sm.hi + sm.lo;
        if (M > 0.0) {
            qx[r] = (px.hi + px.lo) / M;
            qy[r] = (py.hi + py.lo) / M;
            qz[r] = (pz.hi + pz.lo) / M;
            vx[r] = (ux.hi + ux.lo) / M;
            vy[r] = (uy.hi + uy.lo) / M;
            vz[r] = (uz.hi + uz.lo) / M;
        }
        m[r] = M;
        for (int f = e + 1; f < nm; ++f) {
            const int b = mem[f];
            if (uf_find(root, b) == r) {
                lost[b] = 2;
                m[b] = 0.0;
                ++merged;
            }
        }
    }
    cnt[1] += ncoll;
    cnt[2] += merged;
}

// Ejections, per body not lost: lost = 3 beyond r_eject.  Per-block sums of
// the mass of the bodies not lost before this check, of the ejected mass, of
// the ejected momentum and of the count.
__global__ void k_ev_eject(const RBlk *__restrict__ rblk, double r_eject, int *__restrict__ lost,
                           const double *__restrict__ m, const double *__restrict__ qx,
                           const double *__restrict__ qy, const double *__restrict__ qz,
                           const double *__restrict__ vx, const double *__restrict__ vy,
                           const double *__restrict__ vz, double *__restrict__ part)
{
    __shared__ double sh[8 * kBlock / 64];
    const RBlk b = rblk[blockIdx.x];
    const int i = b.start + threadIdx.x;
    double w[6] = {0.0, 0.0, 0.0, 0.0, 0.0, 0.0};
    if (i < b.end && !lost[i]) {
        const double mi = m[i];
        w[0] = mi;
        const double r = sqrt(qx[i] * qx[i] + qy[i] * qy[i] + qz[i] * qz[i]);
        if (r > r_eject) {
            lost[i] = 3;
            w[1] = mi;
            w[2] = mi * vx[i];
            w[3] = mi * vy[i];
            w[4] = mi * vz[i];
            w[5] = 1.0;
        }
    }
    block_sum<6>(w, sh);
    if (threadIdx.x < 6)
        part[(size_t)blockIdx.x * 8 + threadIdx.x] = w[threadIdx.x];
}

// One workgroup per system: the ejected momentum leaves, so the barycentric
// velocities of the rest change by dv = sum m_e V_e / (m0 + sum m - sum m_e).
__global__ void k_ev_eject_sys(const int *__restrict__ rb_first, const int *__restrict__ rb_count,
                               const double *__restrict__ part, const double *__restrict__ m0,
                               double *__restrict__ sys, int *__restrict__ cnt)
{
    __shared__ double sh[8 * kBlock / 64];
    double t[6];
    system_sum<6>(part, 8, rb_first[blockIdx.x], rb_count[blockIdx.x], t, sh);
    if (threadIdx.x == 0) {
        double *o = sys + (size_t)blockIdx.x * 8;
        const int k = (int)t[5];
        o[0] = o[1] = o[2] = 0.0;
        if (k > 0) {
            const double rest = (m0[blockIdx.x] + t[0]) - t[1];
            o[0] = t[2] / rest;
            o[1] = t[3] / rest;
            o[2] = t[4] / rest;
            atomicAdd(&cnt[3], k);
        }
        o[3] = (double)k;
    }
}

__global__ void k_ev_eject_apply(const RBlk *__restrict__ rblk, const double *__restrict__ sys,
                                 const int *__restrict__ lost, double *__restrict__ m,
                                 double *__restrict__ vx, double *__restrict__ vy,
                                 double *__restrict__ vz)
{
    const RBlk b = rblk[blockIdx.x];
    const int i = b.start + threadIdx.x;
    if (i >= b.end)
        return;
    const double *o = sys + (size_t)b.sys * 8;
    if (o[3] == 0.0)
        return;
    const int f = lost[i];
    if (f == 3) {
        m[i] = 0.0;
    } else if (f == 0) {
        vx[i] += o[0];
        vy[i] += o[1];
        vz[i] += o[2];
    }
}

// Order-preserving compaction of the bodies with lost == 0: per-block kept
// counts, their exclusive scan over all blocks (systems are contiguous, so
// the scan is also each system's), then every kept body to its place.
__global__ void k_cmp_count(const RBlk *__restrict__ rblk, const int *__restrict__ lost,
                            int *__restrict__ kept)
{
    __shared__ int sh[kBlock / 64];
    const RBlk b = rblk[blockIdx.x];
    const int i = b.start + threadIdx.x;
    const int k = __popcll(__ballot(i < b.end && lost[i] == 0));
    if ((threadIdx.x & 63) == 0)
        sh[threadIdx.x >> 6] = k;
    __syncthreads();
    if (threadIdx.x == 0) {
        int t = 0;
        for (int w = 0; w < kBlock / 64; ++w)
            t += sh[w];
        kept[blockIdx.x] = t;
    }
}

// pos[b] = kept[0] + ... + kept[b-1], pos[n] = the total (one workgroup).
__global__ void k_cmp_scan(int n, const int *__restrict__ kept, int *__restrict__ pos)
{
    __shared__ int sh[kBlock];
    int carry = 0;
    for (int b0 = 0; b0 < n; b0 += kBlock) {
        const int b = b0 + threadIdx.x;
        const int v = b < n ? kept[b] : 0;
        sh[threadIdx.x] = v;
        __syncthreads();
        // inclusive Hillis-Steele scan of the chunk
        for (int o = 1; o < kBlock; o <<= 1) {
            const int t = threadIdx.x >= o ? sh[threadIdx.x - o] : 0;
            __syncthreads();
            sh[threadIdx.x] += t;
            __syncthreads();
        }
        if (b < n)
            pos[b] = carry + sh[threadIdx.x] - v;
        carry += sh[kBlock - 1];
        __syncthreads();
    }
    if (threadIdx.x == 0)
        pos[n] = carry;
}

// out: 7 planes of ntot (m, Q, V); idx[k] = the old index of kept body k.
__global__ void k_cmp_scatter(const RBlk *__restrict__ rblk, const int *__restrict__ lost,
                              const int *__restrict__ pos, int ntot, const double *__restrict__ m,
                              const double *__restrict__ qx, const double *__restrict__ qy,
                              const double *__restrict__ qz, const double *__restrict__ vx,
                              const double *__restrict__ vy, const double *__restrict__ vz,
                              double *__restrict__ out, int *__restrict__ idx)
{
    __shared__ int sh[kBlock / 64];
    const RBlk b = rblk[blockIdx.x];
    const int i = b.start + threadIdx.x;
    const int lane = threadIdx.x & 63, wv = threadIdx.x >> 6;
    const bool keep = i < b.end && lost[i] == 0;
    const unsigned long long mask = __ballot(keep);
    if (lane == 0)
        sh[wv] = __popcll(mask);
    __syncthreads();
    int before = 0;
    for (int w = 0; w < wv; ++w)
        before += sh[w];
    if (!keep)
        return;
    const int o = pos[blockIdx.x] + before + (int)__popcll(mask & ((1ull << lane) - 1ull));
    const size_t n = (size_t)ntot;
    out[o] = m[i];
    out[n + o] = qx[i];
    out[2 * n + o] = qy[i];
    out[3 * n + o] = qz[i];
    out[4 * n + o] = vx[i];
    out[5 * n + o] = vy[i];
    out[6 * n + o] = vz[i];
    idx[o] = i;
}

hipError_t launch_events(const Dev &d, const Params &p, double tau, double rho, double r_star,
                         double r_eject, hipStream_t s)
{
    if (d.nrb == 0)
        return hipSuccess;
    const Snap a = d.snap();
    k_fill_i32<<<1, 64, 0, s>>>(d.evcnt, 4, 0);
    k_ev_star<<<d.nrb, kBlock, 0, s>>>(d.rblk, d.m0, p.G, tau, a, d.m, d.qx, d.qy, d.qz, r_star,
                                        d.lost, d.evroot, d.evpart);
    k_ev_star_sys<<<d.nsys, kBlock, 0, s>>>(d.rb_first, d.rb_count, d.evpart, d.m0, d.evsys,
                                             d.evcnt);
    k_ev_star_apply<<<d.nrb, kBlock, 0, s>>>(d.rblk, d.evsys, d.lost, d.m, d.qx, d.qy, d.qz);
    k_ev_collide<<<1, kBlock, 0, s>>>(d.stats, d.enc_cap, d.ice, d.jce, tau, a, rho, d.lost,
                                       d.evroot, d.evflag, d.evmem, d.m, d.qx, d.qy, d.qz, d.vx,
                                       d.vy, d.vz, d.evcnt);
    if (r_eject > 0.0) {
        k_ev_eject<<<d.nrb, kBlock, 0, s>>>(d.rblk, r_eject, d.lost, d.m, d.qx, d.qy, d.qz, d.vx,
                                             d.vy, d.vz, d.evpart);
        k_ev_eject_sys<<<d.nsys, kBlock, 0, s>>>(d.rb_first, d.rb_count, d.evpart, d.m0, d.evsys,
                                                  d.evcnt);
        k_ev_eject_apply<<<d.nrb, kBlock, 0, s>>>(d.rblk, d.evsys, d.lost, d.m, d.vx, d.vy, d.vz);
    }
    return hipGetLastError();
}

hipError_t launch_compact(const Dev &d, double *out, int *idx, hipStream_t s)
{
    if (d.nrb == 0)
        return hipSuccess;
    k_cmp_count<<<d.nrb, kBlock, 0, s>>>(d.rblk, d.lost, d.evflag);
    k_cmp_scan<<<1, kBlock, 0, s>>>(d.nrb, d.evflag, d.cmp_pos);
    k_cmp_scatter<<<d.nrb, kBlock, 0, s>>>(d.rblk, d.lost, d.cmp_pos, d.ntot, d.m, d.qx, d.qy,
                                            d.qz, d.vx, d.vy, d.vz, out, idx);
    return hipGetLastError();
}

hipError_t launch_diagnostics(const Dev &d, const Params &p, hipStream_t s)
{
    if (d.ndw > 0)
        k_diag_pairs<<<d.ndw, kBlock, 0, s>>>(d.dwork, d.qx, d.qy, d.qz, d.m, d.rc, p.inner,
                                               d.dpart);
    if (d.nrb > 0)
        k_diag_bodies<<<d.nrb, kBlock, 0, s>>>(d.rblk, d.m0, d.m, d.qx, d.qy, d.qz, d.vx, d.vy,
                                                d.vz, d.bpart);
    const int *dw_first = d.nsplit + d.nsys;      // laid out after nsplit by the runtime
    const int *dw_count = dw_first + d.nsys;
    k_diag_final<<<d.nsys, kBlock, 0, s>>>(d.rb_first, d.rb_count, dw_first, dw_count, d.bpart,
                                           d.dpart, d.m0, p.G, d.diag);
    return hipGetLastError();
}

}  // namespace nb
