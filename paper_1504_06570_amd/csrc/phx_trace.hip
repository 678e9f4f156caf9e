// Photon trace kernels for gfx950 (MI355X).
//
// One photon per lane.  Photon state lives in registers (FP64 position, direction, wavelength,
// time); the optical prescription is read with uniform (scalar) loads; screens are gathered from
// global memory through L2 / Infinity Cache; image bins are 32-bit atomics, aggregated across the
// wavefront when several lanes hit the same pixel; per-(status, surface) counters are kept in LDS
// and flushed once per workgroup.
//
// Random numbers: Philox4x32-10 keyed by (seed, source) with counter (photon index lo, hi, block,
// stream), so each photon is reproducible alone.  Block/word map of stream 0:
//   block 0: pupil radius, pupil angle, time, wavelength
//   block 1: wavelength blur within an SED bin, Sersic angle, conversion length, unused
//   blocks 2-5: coating roulette of surfaces 4(b-2) .. 4(b-2)+3
//   block 6: diffusion normal pair
// Stream 1, block t: trial t of the Gamma sampler used by Sersic sources.
#include <hip/hip_runtime.h>

#include <mutex>

#include "phx_internal.h"
#include "phx_rng.h"

namespace phx {
namespace {

constexpr double kHcEvM = 1.2398419843320026e-6;  // h c / e in eV m
constexpr double kPi = 3.141592653589793;
// Newton stops once a step is at most 1e-12 m (the paper's criterion is 0.01 um).  The root is
// then exact to rounding (convergence is quadratic), but the slope that gives the surface normal
// is the one evaluated before the last step, a step away from the hit point: with a 1e-9 m stop
// the normal of the secondary carried an error of about c x 1e-9 rad, which moved the hit on the
// next mirror by up to 8e-10 m; at 1e-12 m that error is below 1e-13 m.
constexpr double kNewtonTol = 1e-12;             // m
constexpr int kNewtonMax = 16;
constexpr int kBlock = kThreads;

// Reciprocal and reciprocal square root for well-scaled operands (no zeros, infinities or
// denormals): the hardware estimate refined by two Newton steps, about 1 ulp; used for the
// continuous geometry.  Quotients whose operands a caller's constants or wavelengths can make zero or
// infinite (the index of silicon is infinite below 4.35 nm), and the pixel index, keep IEEE division.
__device__ __forceinline__ double rcp_fast(double x) {
    double r = __builtin_amdgcn_rcp(x);
    double e = fma(-x, r, 1.0);
    r = fma(r, e, r);
    e = fma(-x, r, 1.0);
    return fma(r, e, r);
}
__device__ __forceinline__ double rsq_fast(double x) {
    double y = __builtin_amdgcn_rsq(x);
    const double h = 0.5 * x;
    double e = fma(-h * y, y, 0.5);
    y = fma(y, e, y);
    e = fma(-h * y, y, 0.5);
    return fma(y, e, y);
}
// sqrt(x) for x >= 0 via the reciprocal square root (0 maps to 0).
__device__ __forceinline__ double sqrt_fast(double x) {
    const double r = x * rsq_fast(x);   // every lane: a select, not a branch
    return x > 0.0 ? r : 0.0;
}
// a / b for a constant b whose rounded reciprocal r comes from the host, rounded as IEEE division rounds
// it when a is finite and b is neither zero nor infinite (the correction of a quotient by a
// rounded reciprocal is the rounded quotient: Markstein, IBM J. Res. Dev. 34, 1990).
__device__ __forceinline__ double div_by(double a, double b, double r) {
    const double q = a * r;
    return fma(fma(-b, q, a), r, q);
}
// sqrt(x) rounded as the IEEE square root rounds it, for a well-scaled x > 0 (the coupled iteration
// for the root and half its reciprocal, as the compiler writes it between scalings).
__device__ __forceinline__ double sqrt_norm(double x) {
    const double y = __builtin_amdgcn_rsq(x);
    double g = x * y, h = 0.5 * y;
    const double r = fma(-h, g, 0.5);
    g = fma(g, r, g);
    h = fma(h, r, h);
    g = fma(fma(-g, g, x), h, g);
    return fma(fma(-g, g, x), h, g);
}

// a b + c d with the second product rounded.  The geometry names its fused operations: the compiler's own
// choice among the products of a sum depends on what else it shares a block with, and copies of one
// passage in different kernels would round differently.
__device__ __forceinline__ double dot2(double a, double b, double c, double d) {
    return fma(a, b, c * d);
}

// A table in device memory reached through a pointer that was itself loaded: named global, or its
// loads are flat ones, which also wait for the scalar and LDS counters.
template <class T>
using Global = const T __attribute__((address_space(1)))*;
typedef float Float4 __attribute__((ext_vector_type(4)));

struct Rng {
    uint32_t k0, k1, lo, hi;
    __device__ uint4 block(uint32_t b, uint32_t stream = 0) const {
        return philox(make_uint4(lo, hi, b, stream), k0, k1);
    }
    // The same inside a loop: the key is opaque there, or the compiler keeps the ten rounds' keys in
    // registers all through the loop.
    __device__ uint4 block_in_loop(uint32_t b) const {
        uint32_t a = k0, c = k1;
        asm volatile("" : "+v"(c));
        return philox(make_uint4(lo, hi, b, 0u), a, c);
    }
};

__device__ __forceinline__ double sellmeier(const DevParams& P, double lam) {
    const double lu = lam * 1e6, l2 = lu * lu;
    double s = 1.0;
#pragma unroll
    for (int i = 0; i < 3; ++i) s += P.sell_b[i] * l2 / fma(lu, lu, -P.sell_c[i]);
    return sqrt(s);
}

// Photon energy in eV.
__device__ __forceinline__ double energy_ev(double lam) { return kHcEvM / lam; }

__device__ __forceinline__ double n_silicon(double lam) {
    const double e = energy_ev(lam);
    return 3.36 + 0.211 * e + 2.79 * exp((e - 3.30) / 0.398);
}

// Rajkanan absorption coefficient in m^-1 (constants at the device temperature precomputed).  Eight of
// its quotients have constants for divisors: div_by (plain divisions took the optics stage of 1e9 photons
// from 14.2 to 14.5 ms).  An infinite divisor, at temperatures below 0.95 K, comes from the host as the
// largest double with reciprocal 0, so that its term is 0; what is left to turn a sum into a NaN are
// overflows and divisors of 0, where the quotient is infinite.
__device__ __forceinline__ double absorption(const DevParams& P, double lam) {
    const double e = energy_ev(lam);
    const double C[2] = {5.5, 4.0};
    const double A[2] = {3.231e2, 7.237e3};
    const double ep[2] = {1.827e-2, 5.773e-2};
    double alpha = 0.0;
#pragma unroll
    for (int i = 0; i < 2; ++i) {
#pragma unroll
        for (int j = 0; j < 2; ++j) {
            // (a term below its threshold is zero)
            const double a = fmax(e - P.eg[j] + ep[i], 0.0);
            const double b = fmax(e - P.eg[j] - ep[i], 0.0);
            const double term = div_by(a * a, P.absorb[i], P.inv_absorb[i]) +
                                div_by(b * b, P.emit[i], P.inv_emit[i]);
            alpha += C[i] * A[j] * term;
        }
    }
    if (e > P.egd) alpha += 1.052e6 * sqrt_norm(e - P.egd);
    return alpha == alpha ? alpha * 100.0 : INFINITY;   // (no operand is a NaN)
}

// ---------------------------------------------------------------------------------------------
// Surfaces.

// Zernike deformation as a bivariate polynomial of degree 4 in (u, v) = (x, y)/R: the host
// expands the Noll Z4..Z15 amplitudes into monomial coefficients c[] ordered (0,0) (1,0) (0,1)
// (2,0) (1,1) (0,2) (3,0) (2,1) (1,2) (0,3) (4,0) (3,1) (2,2) (1,3) (0,4).  Returns the value and
// the partial derivatives in u and v (Horner in u within each power of v).
__device__ __forceinline__ void zernike_poly(const double* c, double u, double v, double& s,
                                             double& du, double& dv) {
    const double p0 = c[0] + u * (c[1] + u * (c[3] + u * (c[6] + u * c[10])));
    const double p1 = c[2] + u * (c[4] + u * (c[7] + u * c[11]));
    const double p2 = c[5] + u * (c[8] + u * c[12]);
    const double p3 = c[9] + u * c[13];
    const double p4 = c[14];
    s = p0 + v * (p1 + v * (p2 + v * (p3 + v * p4)));
    const double q0 = c[1] + u * (2.0 * c[3] + u * (3.0 * c[6] + u * 4.0 * c[10]));
    const double q1 = c[4] + u * (2.0 * c[7] + u * 3.0 * c[11]);
    const double q2 = c[8] + u * 2.0 * c[12];
    const double q3 = c[13];
    du = q0 + v * (q1 + v * (q2 + v * q3));
    dv = p1 + v * (2.0 * p2 + v * (3.0 * p3 + v * 4.0 * p4));
}

// What every passage needs of a surface, read with one scalar load and held in scalar registers.
// The empty asm keeps the compiler from sinking each field's load to its first use, where the
// wavefront would wait for it alone: with about ten such waits per surface, 45 % of the optics
// kernel's wavefront time went into waiting (189 scalar loads per 64 photons; now 99, and 28 %
// with four wavefronts per SIMD in place of three).
struct SurfRegs {
    uint32_t bits;
    int32_t coating;
    double c, kappa1, kc2, r_in2, r_out2, tz;
    const float* coat;
};
__device__ __forceinline__ SurfRegs surf_regs(const DevSurface& s) {
    SurfRegs h{s.bits, s.coating, s.c, s.kappa1, s.kc2, s.r_in2, s.r_out2, s.tz, s.coat};
    asm volatile("" : "+s"(h.bits), "+s"(h.coating), "+s"(h.c), "+s"(h.kappa1), "+s"(h.kc2),
                      "+s"(h.r_in2), "+s"(h.r_out2), "+s"(h.tz), "+s"(h.coat));
    return h;
}
// Even aspheric coefficients alpha_4, alpha_6, alpha_8, alpha_10.
struct EvenTerms {
    double a4, a6, a8, a10;
};
__device__ __forceinline__ EvenTerms even_terms(const DevSurface& s) {
    EvenTerms e{s.alpha[1], s.alpha[3], s.alpha[5], s.alpha[7]};
    asm volatile("" : "+s"(e.a4), "+s"(e.a6), "+s"(e.a8), "+s"(e.a10));
    return e;
}

// Sag S(x, y) and g with (dS/dx, dS/dy) = (x g, y g) + zernike gradient.  Returns the conic's
// argument: negative outside its domain, where the rest is meaningless.
template <bool ZERN>
__device__ __forceinline__ double sag(const DevParams& P, const DevSurface& s, const SurfRegs& h,
                                      const EvenTerms& e, double x, double y, double& S,
                                      double& gx, double& gy) {
    const double r2 = dot2(x, x, y, y);
    const double arg = fma(-h.kc2, r2, 1.0);
    // conic: S = c r^2 / (1 + root), dS/dr / r = c / root, root = sqrt(arg); one reciprocal
    // square root and one reciprocal
    const double inv_root = rsq_fast(arg);
    const double root = arg * inv_root;
    S = h.c * r2 * rcp_fast(1.0 + root);
    double g = h.c * inv_root;
    if (h.bits & kSurfEven) {
        // even terms only: Horner in r^2
        S = fma(r2 * r2, fma(r2, fma(r2, fma(e.a10, r2, e.a8), e.a6), e.a4), S);
        g = fma(r2, fma(e.a4, 4.0, r2 * fma(e.a6, 6.0, r2 * fma(e.a8, 8.0, r2 * 10.0 * e.a10))), g);
    } else if (h.bits & kSurfGeneral) {
        // general: sum alpha_i r^i and sum i alpha_i r^(i-2), i = 3..10
        const double r = sqrt_fast(r2);
        double pw = r;          // r^(i-2) for i = 3
        double acc_s = 0.0, acc_g = 0.0;
#pragma unroll
        for (int i = 3; i <= 10; ++i) {
            const double a = s.alpha[i - 3];
            acc_g += (double)i * a * pw;
            acc_s += a * pw * r2;
            pw *= r;
        }
        S += acc_s;
        g += acc_g;
    }
    gx = x * g;
    gy = y * g;
    if (ZERN && (h.bits & kSurfZernike)) {
        double zs, zu, zv;
        zernike_poly(P.zern, x * P.zern_inv_r, y * P.zern_inv_r, zs, zu, zv);
        S += zs;
        gx += zu * P.zern_inv_r;
        gy += zv * P.zern_inv_r;
    }
    return arg;
}

// Intersection of the ray q + l d with the surface: exact conic root, then Newton on
// f(l) = q_z + l d_z - S(q_x + l d_x, q_y + l d_y).  Returns 0 or a status; gx, gy receive the
// sag gradient at the last evaluation.  Lanes whose ray misses run along to the end with
// meaningless values (the branches are on the surface's kind, the same in every lane): a branch for
// each way to miss would cut the arithmetic into pieces too short to fill its latencies.  SEARCH (the
// ghost branch's search): the conic's sums in the other order, as that branch rounds them.
template <bool ZERN, bool SEARCH = false>
__device__ __forceinline__ int intersect(const DevParams& P, const DevSurface& s, const SurfRegs& h,
                                         const double q[3], const double d[3], double& l,
                                         double& gx, double& gy, int& iters) {
    const bool zern = ZERN && (h.bits & kSurfZernike);
    gx = 0.0;
    gy = 0.0;
    if ((h.bits & kSurfPlane) && !zern) {
        // a plane (the conic root below with c = 0: l = q_z / -d_z), slope zero
        l = -q[2] * rcp_fast(d[2]);
        return d[2] == 0.0 ? PHX_MISSED : 0;
    }
    const double kq = h.kappa1 * q[2];
    constexpr int i = SEARCH ? 0 : 1, j = 1 - i;
    const double A = h.c * fma(d[2], h.kappa1 * d[2], dot2(d[i], d[i], d[j], d[j]));
    const double B = fma(h.c, fma(d[2], kq, dot2(q[i], d[i], q[j], d[j])), -d[2]);
    const double C = fma(h.c, fma(q[2], kq, dot2(q[i], q[i], q[j], q[j])), -2.0 * q[2]);
    const double disc = fma(B, B, -(A * C));
    const double sq = sqrt_fast(disc);
    const double den = B >= 0.0 ? B + sq : B - sq;
    l = -C * rcp_fast(den);
    int st = disc < 0.0 || den == 0.0 ? PHX_MISSED : 0;
    if (!(h.bits & (kSurfEven | kSurfGeneral)) && !zern) {
        // a plain conic: the root is the intersection (a Newton update would be rounding-sized,
        // far below the tolerance); only the slope at the hit point is needed
        const double x = fma(d[0], l, q[0]), y = fma(d[1], l, q[1]);
        const double arg = fma(-h.kc2, dot2(x, x, y, y), 1.0);
        const double g = h.c * rsq_fast(arg);
        gx = x * g;
        gy = y * g;
        return arg < 0.0 ? PHX_MISSED : st;
    }
    const EvenTerms e = even_terms(s);
    if (st == 0) {
        st = PHX_NONCONV;
#pragma unroll 1
        for (int it = 1; it <= kNewtonMax; ++it) {
            const double x = fma(d[0], l, q[0]), y = fma(d[1], l, q[1]);
            double S;
            const double arg = sag<ZERN>(P, s, h, e, x, y, S, gx, gy);
            const double fp = d[2] - dot2(gx, d[0], gy, d[1]);
            const double dz = fma(d[2], l, q[2]) - S, ifp = rcp_fast(fp), dl = dz * ifp;
            const bool out = arg < 0.0, flat = fp == 0.0;
            const bool step = !(out || flat);
            l = step ? fma(-dz, ifp, l) : l;
            iters += step;
            const bool conv = step && fabs(dl) <= kNewtonTol;
            st = out ? PHX_MISSED : conv ? 0 : PHX_NONCONV;
            if (!step || conv) break;
        }
    }
    return st;
}

// Position of a wavelength on the coating tables' uniform wavelength axis (clamped at the ends):
// column il and weight b of column il + 1.  Computed once per photon.
struct LamCol {
    int il;
    double b;
};
__device__ __forceinline__ LamCol lambda_column(const DevParams& P, double lam) {
    double fl = (lam - P.lam0) * P.inv_dlam;
    fl = fmin(fmax(fl, 0.0), (double)(P.n_lam - 1));
    const int il = min((int)floor(fl), P.n_lam - 2);
    return LamCol{il, fl - il};
}

// Coating transmission (section 2.4.2) from a coating's table: bilinear in s = sin^2(incidence) and
// wavelength.
__device__ __forceinline__ double coating(const DevParams& P, const float* table, double s,
                                          const LamCol& lc) {
    double fs = s * P.inv_s_step;
    fs = fmin(fmax(fs, 0.0), (double)(P.n_s - 1));
    const int is = min((int)floor(fs), P.n_s - 2);
    const double a = fs - is, b = lc.b;
    Global<float> r0 = (Global<float>)table +
                       ((uint64_t)(uint32_t)is * (uint32_t)P.n_lam + (uint32_t)lc.il);
    Global<float> r1 = r0 + P.n_lam;
    return (1.0 - a) * ((1.0 - b) * (double)r0[0] + b * (double)r0[1]) +
           a * ((1.0 - b) * (double)r1[0] + b * (double)r1[1]);
}
// The reflectance table of the coating whose transmission table is given (ghosts).
__device__ __forceinline__ const float* reflectance(const DevParams& P, const float* table) {
    return P.coat_r + (table - P.coat);
}

// The value of the other lane of a pair (lanes 2 i and 2 i + 1).
__device__ __forceinline__ uint32_t pair_swap(uint32_t v) {
    return (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0xb1, 0xf, 0xf, true);
}
__device__ __forceinline__ Float4 pair_swap(const Float4& v) {
    Float4 r;
    r.x = __uint_as_float(pair_swap(__float_as_uint(v.x)));
    r.y = __uint_as_float(pair_swap(__float_as_uint(v.y)));
    r.z = __uint_as_float(pair_swap(__float_as_uint(v.z)));
    r.w = __uint_as_float(pair_swap(__float_as_uint(v.w)));
    return r;
}

// Bilinear interpolation of one gradient screen at (sx, sy) in metres: one 32-byte record per cell
// holds the four corner gradients.  The cell index is taken modulo the screen's side (a power of two:
// every step is exact) in floating point; through 64-bit integers the two conversions take half of
// the lookup's instructions.
// Every lane of the wavefront has to call it: the lanes of a pair load the two halves of the even lane's
// record, then of the odd lane's, and exchange them.  Two loads of a lane from one record stall the
// first-level cache, which waits at the second for the first one's line and with that keeps no more than
// about one load's 64 lines on their way; a pair's halves are one request.  Sky stage of 2^26
// photons (8.8e6 traced) 1.48 -> 1.22 ms, for 5.6e7 lines from beyond the L2, 5.9 TB/s (six a photon, nearly
// all of the finest scale, which are of no use to another photon in flight).
__device__ __forceinline__ void screen_tap(const float4* g, uint32_t N, double side,
                                           double inv_side, double sx, double sy, double inv_pix,
                                           double& ax, double& ay) {
    const double fx = floor(sx * inv_pix), fy = floor(sy * inv_pix);
    const double a = fma(sx, inv_pix, -fx), b = fma(sy, inv_pix, -fy);
    const uint32_t i0 = (uint32_t)fma(-side, floor(fx * inv_side), fx);
    const uint32_t j0 = (uint32_t)fma(-side, floor(fy * inv_side), fy);
    const bool odd = __lane_id() & 1;
    const uint32_t cell = j0 * N + i0, other = pair_swap(cell);
    Global<Float4> half = (Global<Float4>)g + (odd ? 1 : 0);
    const Float4 ve = half[2 * (uint64_t)(odd ? other : cell)];   // of the even lane's record
    const Float4 vo = half[2 * (uint64_t)(odd ? cell : other)];   // of the odd lane's
    const Float4 we = pair_swap(ve), wo = pair_swap(vo);
    const Float4 lo = odd ? wo : ve, hi = odd ? vo : we;   // (i,j) (i+1,j) | (i,j+1) (i+1,j+1)
    const double a1 = 1.0 - a, b1 = 1.0 - b;
    ax = dot2(b1, dot2(a1, (double)lo.x, a, (double)lo.z), b, dot2(a1, (double)hi.x, a, (double)hi.z));
    ay = dot2(b1, dot2(a1, (double)lo.y, a, (double)lo.w), b, dot2(a1, (double)hi.y, a, (double)hi.w));
}

__device__ __forceinline__ void normalise(double n[3]) {
    const double inv = 1.0 / sqrt(n[0] * n[0] + n[1] * n[1] + n[2] * n[2]);
    n[0] *= inv; n[1] *= inv; n[2] *= inv;
}

// Gamma(shape) by Marsaglia & Tsang, trial t on stream 1 block t.
__device__ double gamma_sample(const Rng& rng, double shape) {
    const double a = shape < 1.0 ? shape + 1.0 : shape;
    const double dd = a - 1.0 / 3.0, cc = 1.0 / sqrt(9.0 * dd);
#pragma unroll 1
    for (uint32_t t = 0; t < 64; ++t) {
        const uint4 w = rng.block(t, 1);
        const double u0 = u01(w.x), u1 = u01(w.y), u2 = u01(w.z);
        const double x = sqrt(-2.0 * log(u0)) * cospi(2.0 * u1);
        double v = 1.0 + cc * x;
        if (v <= 0.0) continue;
        v = v * v * v;
        const double x2 = x * x;
        bool accept = u2 < 1.0 - 0.0331 * x2 * x2;
        if (!accept) accept = log(u2) < 0.5 * x2 + dd * (1.0 - v + log(v));
        if (accept) {
            double g = dd * v;
            if (shape < 1.0) g *= exp(log(u01(w.w)) / shape);
            return g;
        }
    }
    return shape;
}

// Wavelength (section 2.2): flat photon spectrum, or the SED's photon CDF (first bin k with
// CDF[k+1] > u, found by bisection between two entries of a guide table) blurred uniformly
// across the bin; then (1 + z).
__device__ __forceinline__ double wavelength(const DevParams& P, const DevSource& src,
                                             const uint4& w0, const uint4& w1) {
    double lam;
    if (src.sed < 0) {
        lam = src.lambda_lo + u01(w0.w) * src.lambda_span;
    } else {
        const double* cdf = P.sed_cdf + (size_t)src.sed * (P.sed_k + 1);
        const double u = u01(w0.w);
        // the answer lies between the guide entries around u (u kSedGuide is exact)
        const uint16_t* guide = P.sed_guide + (size_t)src.sed * (kSedGuide + 1);
        const int j = min((int)(u * kSedGuide), kSedGuide - 1);
        int lo = guide[j], hi = guide[j + 1];
        while (lo < hi) {
            const int mid = (lo + hi) >> 1;
            if (cdf[mid + 1] > u) hi = mid; else lo = mid + 1;
        }
        lam = P.sed_edges[lo] + u01(w1.x) * (P.sed_edges[lo + 1] - P.sed_edges[lo]);
    }
    return lam * src.redshift1;
}

// Pre-roll test (section 3.2): a photon is culled when a coated surface's roulette draw exceeds
// the largest transmission that coating has at this wavelength for any angle, so it cannot
// survive.  The coated surfaces are tested in order of decreasing selectivity.  preroll_draw
// gives the wavelength and block 0 (radius, angle and time words) from the photon's first Philox
// blocks.
__device__ __forceinline__ double preroll_draw(const DevParams& P, const Rng& rng,
                                               const DevSource& src, uint4& w0) {
    w0 = rng.block(0);
    uint4 w1 = make_uint4(0, 0, 0, 0);
    if (src.sed >= 0) w1 = rng.block(1);
    return wavelength(P, src, w0, w1);
}

__device__ __forceinline__ uint32_t word_of(const uint4& w, int m) {
    return m == 0 ? w.x : (m == 1 ? w.y : (m == 2 ? w.z : w.w));
}

// The first (most selective) test, at wavelength column il; only surfaces below k_lim are
// tested (with ghosts: the coated surfaces every photon passes sequentially).
template <bool GHOST>
__device__ __forceinline__ bool preroll_first(const DevParams& P, const Rng& rng, int il,
                                              int k_lim) {
    const int k = P.cull_order[0];
    if (GHOST && k >= k_lim) return false;
    const uint32_t wk = word_of(rng.block(2 + (k >> 2)), k & 3);
    return (int64_t)wk > P.coat_thr[(size_t)P.surf[k].coating * P.n_lam + il];
}

// Tests 1..n_tests-1 in order, stopping at the first that culls; a roulette block is drawn when
// the next test's surface needs a different one.
template <bool GHOST>
__device__ __forceinline__ bool preroll_rest(const DevParams& P, const Rng& rng, int il,
                                             int n_tests, int k_lim) {
    int blk = -1;
    uint4 w = make_uint4(0, 0, 0, 0);
    for (int j = 1; j < n_tests; ++j) {
        const int k = P.cull_order[j];
        if (GHOST && k >= k_lim) continue;
        if (2 + (k >> 2) != blk) {
            blk = 2 + (k >> 2);
            w = rng.block(blk);
        }
        if ((int64_t)word_of(w, k & 3) > P.coat_thr[(size_t)P.surf[k].coating * P.n_lam + il])
            return true;
    }
    return false;
}

// Pre-roll escape test (section 3.2 with the silicon stage): the photon converts deeper than the
// silicon whatever its path, since its conversion distance (the silicon stage's draw) times the
// smallest cosine a ray refracted into silicon can have exceeds the thickness.  The ray reaches
// silicon from vacuum or glass, so sin(theta) in silicon is at most n_in / n_Si with n_in the
// glass index when the optics hold glass; the relative margin 1e-12 covers the rounding of the
// optics stage's refracted direction.  Kept out of line: it runs for few photons, and inlined it
// raises the register count of the whole pre-roll.
__device__ __noinline__ bool escape_certain(const DevParams& P, double lam, uint32_t w_conv) {
    const double alpha = absorption(P, lam);
    const double L_conv = alpha > 0.0 ? -log(u01(w_conv)) / alpha : INFINITY;
    const double q = (P.has_glass ? sellmeier(P, lam) : 1.0) / n_silicon(lam);
    if (!(q < 1.0)) return false;
    const double cos_min = sqrt(1.0 - q * q);
    return L_conv * cos_min * (1.0 - 1e-12) > P.t_si;
}

// ---------------------------------------------------------------------------------------------
// Per-photon physics beyond the core path.  Only the sky and optics kernel instantiations with
// EXTRA = true contain this code (the launch picks them when one of its flags is set), so the
// registers and occupancy of the other instantiations do not depend on it.

__device__ __forceinline__ double3 unit3(double3 v) {
    const double inv = 1.0 / sqrt(v.x * v.x + v.y * v.y + v.z * v.z);
    return make_double3(v.x * inv, v.y * inv, v.z * inv);
}

// Atmospheric dispersion (section 2.3.3): the direction moves by R(lambda) - R(lambda0) along the
// zenith direction in (n_x, n_y), R = (n_air - 1) tan z, n_air from the Filippenko formula with
// its pressure-temperature and water factors precomputed; the difference of the dry brackets and
// of the water terms is taken before scaling, so no 1 + 3e-4 is formed.
__device__ __forceinline__ double3 disperse(const DevParams& P, double lam, double3 n) {
    const DevPhysics& X = P.ph;
    const double lu = lam * 1e6;
    const double s = 1.0 / (lu * lu);
    const double b = 64.328 + 29498.1 / (146.0 - s) + 255.4 / (41.0 - s);
    const double dR =
        1e-6 * (X.disp_pt * (b - X.disp_b0) + 0.000680 * X.disp_w * (s - X.disp_s0)) * X.disp_tanz;
    n.x += dR * X.disp_cx;
    n.y += dR * X.disp_cy;
    return unit3(n);
}

// Dome seeing and the micro-roughness halo (section 2.4.2), kicks of the direction on the start
// plane.  Dome: a normal kick of dome_sigma per axis (Box-Muller on block 8).  Halo: with
// probability f (block 7, word y) an angle r0 x toward the azimuth of block 7 word z; x has
// density proportional to x / (1 + x^n) on [0, x_max], drawn by rejection from the density
// x (1 + x^2)^(-n/2), whose CDF 1 - (1 + x^2)^(1 - n/2) inverts in closed form, keeping a trial
// when u < (1 + x^2)^(n/2) / (1 + x^n) / 2^(n/2 - 1) (the ratio's maximum, at x = 1); trial t
// reads stream 2 block t (proposal x, acceptance y); after 32 rejections no kick.
__device__ __forceinline__ double3 entrance_kicks(const DevParams& P, uint32_t flags, Rng rng,
                                               double3 n) {
    const DevPhysics& X = P.ph;
    if (flags & PHX_F_DOME) {
        const uint4 w = rng.block(8);
        const double rad = sqrt(-2.0 * log(u01(w.x)));
        double sa, ca;
        sincospi(2.0 * u01(w.y), &sa, &ca);
        n.x += X.dome_sigma * rad * ca;
        n.y += X.dome_sigma * rad * sa;
        n = unit3(n);
    }
    if (flags & PHX_F_HALO) {
        const uint4 w7 = rng.block(7);
        if (u01(w7.y) < X.halo_f) {
            double x = -1.0;
#pragma unroll 1
            for (uint32_t t = 0; t < 32; ++t) {
                const uint4 w = rng.block(t, 2);
                const double xt = sqrt(exp(log(1.0 - u01(w.x) * X.halo_fq) / X.halo_e) - 1.0);
                const double ratio =
                    exp(0.5 * X.halo_n * log(1.0 + xt * xt)) / (1.0 + exp(X.halo_n * log(xt)));
                if (u01(w.y) < ratio * X.halo_inv_m) {
                    x = xt;
                    break;
                }
            }
            if (x >= 0.0) {
                const double r = X.halo_r0 * x;
                double sa, ca;
                sincospi(2.0 * u01(w7.z), &sa, &ca);
                n.x += r * ca;
                n.y += r * sa;
                n = unit3(n);
            }
        }
    }
    return n;
}

// Second kick of the hybrid atmosphere at layer i (section 2.3.2): the long-exposure PSF of the
// layer's modes above kappa_crit, exp(-D/2) in the pupil, is the compound Poisson law of
// K ~ Poisson(s2_i) scatterings (count word wk; K = the smallest k whose cumulative probability
// exceeds the uniform, at most 8), each a deflection lambda_ref kappa / (2 pi) toward a uniform
// azimuth with kappa from the phase spectrum on [kappa_crit, kappa_max] by inverting
// (A(kappa_crit) - A(kappa)) / dA, A = (kappa^2 + kappa0^2)^(-5/6) (stream 3, block 8 i + j:
// wavenumber x, azimuth y).  Adds the deflection to (gx, gy).
__device__ __forceinline__ void second_kick(const DevParams& P, const Rng& rng, int i,
                                            uint32_t wk, double& gx, double& gy) {
    const DevPhysics& X = P.ph;
    const double uk = u01(wk);
    double p = X.kick_p0[i], cum = p;
    if (uk < cum) return;
    const double s2 = X.kick_s2[i];
    int K = 0;
    while (!(uk < cum) && K < 8) {
        ++K;
        p *= s2 / K;
        cum += p;
    }
#pragma unroll 1
    for (int j = 0; j < K; ++j) {
        const uint4 w = rng.block((uint32_t)(8 * i + j), 3);
        const double A = X.kick_A0 - u01(w.x) * X.kick_dA;
        const double kappa = sqrt(exp(-1.2 * log(A)) - X.kick_k02);
        const double th = P.lambda_ref * kappa / (2.0 * kPi);
        double sa, ca;
        sincospi(2.0 * u01(w.y), &sa, &ca);
        gx += th * ca;
        gy += th * sa;
    }
}

// Aerosol extinction (section 2.3.3) and the spider (sections 2.4.1-2.4.2) at the telescope
// entrance.  status 0: the photon lives (a ray that passes the spider is moved to the vanes'
// mid-height and turned); PHX_EXTINCT with p the start-plane point; PHX_OBSCURED with p the first
// point along the ray inside a vane.
struct Entry {
    double3 p, n;
    int status;
};

// One slab of the ray-box test: narrows [t0, t1] to the parameters where o + t d lies in [lo, hi].
__device__ __forceinline__ void slab(double o, double d, double lo, double hi, double& t0,
                                     double& t1, bool& inside) {
    if (d == 0.0) {
        if (o < lo || o > hi) inside = false;
        return;
    }
    double ta = (lo - o) / d, tb = (hi - o) / d;
    if (ta > tb) {
        const double tmp = ta;
        ta = tb;
        tb = tmp;
    }
    t0 = fmax(t0, ta);
    t1 = fmin(t1, tb);
}

// Aerosol: survival with probability exp(-tau sec z), tau = tau0 (lambda / 500 nm)^gamma (block 7
// word x).  Spider: vane k is the box u in [r_in, r_out], |v| <= w/2, z in [z_lo, z_hi] along
// u = (c_k, s_k, 0), v = (-s_k, c_k, 0).  A ray that passes every box turns by
// lambda / (4 pi max(d, lambda)) along +v or -v of the nearest vane (block 7 word w), d = the
// smallest distance between the ray's line and a vane's long edge (segment along u at v = +-w/2,
// z = z_lo or z_hi: the closest point of the infinite edge line, clamped to the segment, then its
// distance to the ray's line).
__device__ __forceinline__ Entry entrance_extra(const DevParams& P, uint32_t flags, Rng rng,
                                             double lam, double3 p, double3 n) {
    const DevPhysics& X = P.ph;
    const uint4 w7 = rng.block(7);
    if (flags & PHX_F_AEROSOL) {
        const double tau = X.tau0 * exp(X.gamma * log(lam / 500e-9)) * X.airmass;
        if (!(u01(w7.x) < exp(-tau))) return Entry{p, n, PHX_EXTINCT};
    }
    if ((flags & PHX_F_SPIDER) && X.vanes > 0) {
        double best = INFINITY, t_hit = INFINITY;
        int bk = -1;
#pragma unroll 1
        for (int k = 0; k < X.vanes; ++k) {
            const double c = X.vane_c[k], s = X.vane_s[k];
            double t0 = -INFINITY, t1 = INFINITY;
            bool inside = true;
            slab(p.x * c + p.y * s, n.x * c + n.y * s, X.vane_r0, X.vane_r1, t0, t1, inside);
            slab(-p.x * s + p.y * c, -n.x * s + n.y * c, -X.vane_hw, X.vane_hw, t0, t1, inside);
            slab(p.z, n.z, X.vane_z0, X.vane_z1, t0, t1, inside);
            if (inside && t0 <= t1 && t1 >= 0.0) {
                t_hit = fmin(t_hit, fmax(t0, 0.0));
                continue;
            }
            const double b = c * n.x + s * n.y;
            const double inv = 1.0 / (1.0 - b * b);
#pragma unroll
            for (int e = 0; e < 4; ++e) {
                const double ve = (e & 1) ? X.vane_hw : -X.vane_hw;
                const double ze = (e & 2) ? X.vane_z1 : X.vane_z0;
                const double w0x = -ve * s - p.x, w0y = ve * c - p.y, w0z = ze - p.z;
                const double dw = c * w0x + s * w0y;
                const double ew = n.x * w0x + n.y * w0y + n.z * w0z;
                const double sc = fmin(fmax((b * ew - dw) * inv, X.vane_r0), X.vane_r1);
                const double rx = w0x + sc * c, ry = w0y + sc * s, rz = w0z;
                const double rn = rx * n.x + ry * n.y + rz * n.z;
                const double cx = rx - rn * n.x, cy = ry - rn * n.y, cz = rz - rn * n.z;
                const double dist = sqrt(cx * cx + cy * cy + cz * cz);
                if (dist < best) {
                    best = dist;
                    bk = k;
                }
            }
        }
        if (t_hit < INFINITY)
            return Entry{make_double3(p.x + n.x * t_hit, p.y + n.y * t_hit, p.z + n.z * t_hit), n,
                         PHX_OBSCURED};
        if (bk >= 0) {
            const double l = (X.vane_zm - p.z) / n.z;
            p = make_double3(p.x + n.x * l, p.y + n.y * l, X.vane_zm);
            double delta = lam / (4.0 * kPi * fmax(best, lam));
            if (!(u01(w7.w) < 0.5)) delta = -delta;
            n.x -= delta * X.vane_s[bk];
            n.y += delta * X.vane_c[bk];
            n = unit3(n);
        }
    }
    return Entry{p, n, 0};
}

struct Outcome {
    int status, surface, newton;
    int pix_i, pix_j;
    double x, y, z, xe, ye, lam;
};

// The whole per-photon path.  `culled` photons return PHX_CULLED without being traced.
// Photon state at the start plane above the optics.
struct Front {
    double p[3], n[3], lam;
};

// Sky sampling (sections 2.2, 2.2.1) and the atmosphere (sections 2.3.1-2.3.2), ending on the
// start plane above every optic.
template <bool SERSIC, bool EXTRA>
__device__ void photon_front(const DevParams& P, const Launch& L, int si, uint64_t idx, Front& f) {
    const DevSource& src = P.src[si];
    const Rng rng{L.seed, (uint32_t)si, (uint32_t)idx, (uint32_t)(idx >> 32)};
    const uint4 w0 = rng.block(0);
    uint4 w1 = make_uint4(0, 0, 0, 0);
    if (src.sed >= 0 || (SERSIC && src.kind == 1)) w1 = rng.block(1);
    const double lam = wavelength(P, src, w0, w1);

    // direction (section 2.2) and extended-source perturbation (section 2.2.1)
    double n[3] = {src.xi, src.eta, src.nz};
    if (SERSIC && src.kind == 1) {
        const double g = gamma_sample(rng, 2.0 * src.sersic_n);
        const double rr = exp(src.sersic_n * log(g / src.sersic_bn));
        double sp, cp;
        sincospi(2.0 * u01(w1.y), &sp, &cp);
        const double dmaj = src.sersic_a * rr * cp, dmin = src.sersic_b * rr * sp;
        n[0] += dmaj * src.cos_pa - dmin * src.sin_pa;
        n[1] += dmaj * src.sin_pa + dmin * src.cos_pa;
        normalise(n);
    }
    if (EXTRA && (L.flags & PHX_F_DISPERSION)) {
        const double3 m = disperse(P, lam, make_double3(n[0], n[1], n[2]));
        n[0] = m.x; n[1] = m.y; n[2] = m.z;
    }
    const double t = L.exposure * u01(w0.z);

    // pupil sample on the first surface (section 2.2)
    double p[3];
    {
        const double ro = P.pupil_r_out + L.pupil_margin;
        const double ri = fmax(P.pupil_r_in - L.pupil_margin, 0.0);
        const double r = sqrt(u01(w0.x) * (ro * ro - ri * ri) + ri * ri);
        double sphi, cphi;
        sincospi(2.0 * u01(w0.y), &sphi, &cphi);
        p[0] = r * cphi;
        p[1] = r * sphi;
        const DevSurface& s0 = P.surf[0];
        const double r2 = p[0] * p[0] + p[1] * p[1];
        const double arg = 1.0 - s0.kc2 * r2;
        double z = s0.tz + (arg >= 0.0 ? s0.c * r2 / (1.0 + sqrt(arg)) : 0.0);
        if (s0.bits & (kSurfEven | kSurfGeneral)) {
            double pw = r * r2;
            for (int i = 3; i <= 10; ++i) {
                z += s0.alpha[i - 3] * pw;
                pw *= r;
            }
        }
        p[2] = z;
    }

    // atmosphere (sections 2.3.1-2.3.2): move up to the highest layer, then down layer by layer,
    // deflecting by the wind-shifted screen gradients scaled by (lambda/lambda_ref)^(-1/5)
    if ((L.flags & PHX_F_ATMOSPHERE) && P.n_layers > 0) {
        const double kick = exp(-0.2 * log(lam / P.lambda_ref));
        const uint32_t N = (uint32_t)P.screen_n;
        const double side = (double)P.screen_n, inv_side = 1.0 / side;
        const bool second = EXTRA && (L.flags & PHX_F_SECOND_KICK);
        uint4 kw0 = make_uint4(0, 0, 0, 0), kw1 = make_uint4(0, 0, 0, 0);
        if (second) {
            kw0 = rng.block(9);
            if (P.n_layers > 4) kw1 = rng.block(10);
        }
#pragma unroll 1
        for (int i = P.n_layers - 1; i >= 0; --i) {
            const double h = P.height[i];
            const double l = (h - p[2]) * rcp_fast(n[2]);
            p[0] += n[0] * l;
            p[1] += n[1] * l;
            p[2] = h;
            const double sx = p[0] - P.wind[i][0] * t;
            const double sy = p[1] - P.wind[i][1] * t;
            double gx = 0.0, gy = 0.0;
#pragma unroll 1
            for (int s = 0; s < P.n_scales; ++s) {
                const float4* g = P.grad + (size_t)(i * P.n_scales + s) * N * N * 2;
                double ax, ay;
                screen_tap(g, N, side, inv_side, sx, sy, P.inv_pix[s], ax, ay);
                gx += ax;
                gy += ay;
            }
            if (second) {
                // select by value: a select between the two blocks' addresses would keep them in
                // scratch memory
                const uint4 kw = i < 4 ? kw0 : kw1;
                second_kick(P, rng, i, word_of(kw, i & 3), gx, gy);
            }
            n[0] += kick * gx;
            n[1] += kick * gy;
            const double inv = rsq_fast(n[0] * n[0] + n[1] * n[1] + n[2] * n[2]);
            n[0] *= inv;
            n[1] *= inv;
            n[2] *= inv;
        }
    }
    {
        const double l = (P.z_start - p[2]) * rcp_fast(n[2]);
        p[0] += n[0] * l;
        p[1] += n[1] * l;
        p[2] = P.z_start;
    }
    if (EXTRA && (L.flags & (PHX_F_DOME | PHX_F_HALO))) {
        const double3 m = entrance_kicks(P, L.flags, rng, make_double3(n[0], n[1], n[2]));
        n[0] = m.x; n[1] = m.y; n[2] = m.z;
    }
    f.p[0] = p[0]; f.p[1] = p[1]; f.p[2] = p[2];
    f.n[0] = n[0]; f.n[1] = n[1]; f.n[2] = n[2];
    f.lam = lam;
}

// Field model of the diffusion width (section 2.4.3): sigma^2 interpolated linearly in the
// library's table against depth below the entrance surface (zero beyond the collection height);
// `slope` = d sigma / d depth of the interpolant.
__device__ __forceinline__ double field_sigma(const DevParams& P, double depth, double& slope) {
    const DevPhysics& X = P.ph;
    slope = 0.0;
    if (!(depth < X.sig2_dmax)) return 0.0;
    const double f = depth * X.sig2_inv_step;
    const int k = min((int)f, X.n_sig2 - 1);
    const double a = f - k;
    const double s2 = (1.0 - a) * X.sig2[k] + a * X.sig2[k + 1];
    if (!(s2 > 0.0)) return 0.0;
    const double sigma = sqrt(s2);
    slope = (X.sig2[k + 1] - X.sig2[k]) * X.sig2_inv_step / (2.0 * sigma);
    return sigma;
}

// Silicon (sections 2.4.2-2.4.3): conversion after a path of mean free path x Exp(1) along the
// refracted direction d; escape if deeper than the silicon; Gaussian diffusion with sigma
// proportional to the drift distance to the collecting surface.  With PHX_F_DEAD_LAYER an
// electron converted less than `dead` below the entrance surface is removed (section 2.4.2
// field-free layer).  Moves (xc, yc) from the landing point to the electron position; returns 0,
// PHX_ESCAPED or PHX_DEAD.  Inlined: a call would give the kernel a stack frame and register saves
// around it.
__device__ __forceinline__ int sensor_stage(const DevParams& P, const Launch& L, const Rng& rng,
                                         double lam, const double* d, double& xc, double& yc) {
    if (L.flags & PHX_F_SILICON) {
        const double alpha = absorption(P, lam);
        const double L_conv = alpha > 0.0 ? -log(u01(rng.block(1).z)) / alpha : INFINITY;
        const double depth = L_conv * fabs(d[2]);
        if (!(depth <= P.t_si)) return PHX_ESCAPED;
        if ((L.flags & PHX_F_DEAD_LAYER) && depth < P.ph.dead) return PHX_DEAD;
        xc += d[0] * L_conv;
        yc += d[1] * L_conv;
        if (L.flags & PHX_F_DIFFUSION) {
            const uint4 wd = rng.block(6);
            double slope;
            const double sigma = (L.flags & PHX_F_FIELD_DIFFUSION)
                                     ? field_sigma(P, depth, slope)
                                     : P.sigma_max * (P.t_si - depth) / P.t_si;
            const double rad = sqrt_norm(-2.0 * log(u01(wd.x)));
            double sa, ca;
            sincospi(2.0 * u01(wd.y), &sa, &ca);
            xc += sigma * rad * ca;
            yc += sigma * rad * sa;
        }
    }
    return 0;
}

// Central obscuration, the surfaces (sections 2.4.1-2.4.2), silicon (sections 2.4.2-2.4.3) and
// the pixel, from the start-plane state.
struct Hit {
    double q[3], d[3], N[3];
    double dn, l;
};

// Returned by hit_surface when a filter or anti-reflection coating reflects the photon (ghosts).
constexpr int kGhostReflect = 1000;

// Into and out of a surface's element frame.
__device__ __forceinline__ void to_element(const DevSurface& s, const SurfRegs& h, const double p[3],
                                           const double n[3], double q[3], double d[3]) {
    if (h.bits & kSurfMoved) {
        const double r0 = p[0] - s.t[0], r1 = p[1] - s.t[1], r2 = p[2] - s.t[2];
#pragma unroll
        for (int i = 0; i < 3; ++i) {
            q[i] = fma(s.R[6 + i], r2, dot2(s.R[i], r0, s.R[3 + i], r1));
            d[i] = fma(s.R[6 + i], n[2], dot2(s.R[i], n[0], s.R[3 + i], n[1]));
        }
    } else {
        q[0] = p[0]; q[1] = p[1]; q[2] = p[2] - h.tz;
        d[0] = n[0]; d[1] = n[1]; d[2] = n[2];
    }
}
__device__ __forceinline__ void to_global(const DevSurface& s, uint32_t bits, double tz,
                                          const double q[3], const double d[3], double p[3],
                                          double n[3]) {
    if (bits & kSurfMoved) {
#pragma unroll
        for (int i = 0; i < 3; ++i) {
            p[i] = fma(s.R[3 * i + 2], q[2], dot2(s.R[3 * i], q[0], s.R[3 * i + 1], q[1])) + s.t[i];
            n[i] = fma(s.R[3 * i + 2], d[2], dot2(s.R[3 * i], d[0], s.R[3 * i + 1], d[1]));
        }
    } else {
        p[0] = q[0]; p[1] = q[1]; p[2] = q[2] + tz;
        n[0] = d[0]; n[1] = d[1]; n[2] = d[2];
    }
}

__device__ __forceinline__ void advance(Hit& h, double l) {
#pragma unroll
    for (int i = 0; i < 3; ++i) h.q[i] = fma(h.d[i], l, h.q[i]);
}
// Reflection across the normal (section 2.4.2).
__device__ __forceinline__ void reflect_ray(Hit& h) {
#pragma unroll
    for (int i = 0; i < 3; ++i) h.d[i] = fma(-(2.0 * h.dn), h.N[i], h.d[i]);
}

// The normal at a hit point from the sag's slope, facing the incoming ray (SEARCH as in intersect).
template <bool ZERN, bool SEARCH = false>
__device__ __forceinline__ void hit_normal(uint32_t bits, double gx, double gy, Hit& h) {
    if ((bits & kSurfPlane) && !(ZERN && (bits & kSurfZernike))) {
        h.N[0] = 0.0; h.N[1] = 0.0; h.N[2] = 1.0;
    } else {
        const double inv = rsq_fast((SEARCH ? dot2(gy, gy, gx, gx) : dot2(gx, gx, gy, gy)) + 1.0);
        h.N[0] = -gx * inv; h.N[1] = -gy * inv; h.N[2] = inv;
    }
    constexpr int i = SEARCH ? 1 : 0, j = 1 - i;
    h.dn = fma(h.d[2], h.N[2], dot2(h.d[i], h.N[i], h.d[j], h.N[j]));
    if (h.dn > 0.0) { h.N[0] = -h.N[0]; h.N[1] = -h.N[1]; h.N[2] = -h.N[2]; h.dn = -h.dn; }
}

// Passage of surface k (the same in every lane): transform into its frame, intersect, clip to the
// clear aperture, take the normal (facing the incoming ray) and play the coating roulette
// (sections 2.4.1-2.4.2).  Returns 0 to continue or the photon's fate; a photon that misses keeps
// the position it came with.
template <bool ZERN, bool TAPE = false, bool GHOST = false>
__device__ __forceinline__ int hit_surface(const DevParams& P, const Launch& L, const Rng& rng,
                                           const SurfRegs& sr, int k, const double p[3],
                                           const double n[3], const LamCol& lc, uint4& wc,
                                           int& wc_block, Hit& h, int& newton) {
    const DevSurface& s = P.surf[k];
    to_element(s, sr, p, n, h.q, h.d);
    double l, gx, gy;
    int st = intersect<ZERN>(P, s, sr, h.q, h.d, l, gx, gy, newton);
    if (st == 0 && !(l > 0.0)) st = PHX_MISSED;
    if (TAPE) h.l = l;
    if (st != 0) l = 0.0;
    advance(h, l);
    const double rq2 = dot2(h.q[0], h.q[0], h.q[1], h.q[1]);
    if (st == 0 && (rq2 < sr.r_in2 || rq2 > sr.r_out2)) st = PHX_VIGNETTED;
    hit_normal<ZERN>(sr.bits, gx, gy, h);
    if ((L.flags & PHX_F_COATINGS) && sr.coating >= 0) {
        const int blk = 2 + (k >> 2);
        if (blk != wc_block) { wc = rng.block_in_loop(blk); wc_block = blk; }
        const uint32_t w = word_of(wc, k & 3);
        // (a lane that missed reads some entry of the table: the lookup clamps)
        const double T = coating(P, sr.coat, 1.0 - h.dn * h.dn, lc);
        const bool lost = !(u01(w) < T);
        if (GHOST) {
            if (st == 0 && lost) {
                st = PHX_ABSORBED;
                if ((L.flags & PHX_F_GHOSTS) && !(sr.bits & kSurfMirror) &&
                    u01(w) < T + coating(P, reflectance(P, sr.coat), 1.0 - h.dn * h.dn, lc))
                    st = kGhostReflect;
            }
        } else {
            st = st == 0 && lost ? PHX_ABSORBED : st;
        }
    }
    return st;
}

// Refraction by the vector form of Snell's law (section 2.4.2); false on total internal
// reflection.
__device__ __forceinline__ bool refract(Hit& h, double mu) {
    const double cosi = -h.dn;
    const double kk = fma(-fma(-cosi, cosi, 1.0), mu * mu, 1.0);
    const double f = fma(mu, cosi, -sqrt_fast(kk));
#pragma unroll
    for (int i = 0; i < 3; ++i) h.d[i] = fma(mu, h.d[i], f * h.N[i]);
    return !(kk < 0.0);   // (the direction of a totally reflected ray is not used)
}

// Tape of one surface passage for the adjoint: hit point and incoming direction in the
// element frame, and the path length from the previous surface, at tp[(k * kTapeFields + i) * ts].
__device__ __forceinline__ void tape_put(double* tp, uint64_t ts, int k, const Hit& h) {
    double* t = tp + (uint64_t)k * kTapeFields * ts;
    t[0] = h.q[0]; t[ts] = h.q[1]; t[2 * ts] = h.q[2];
    t[3 * ts] = h.d[0]; t[4 * ts] = h.d[1]; t[5 * ts] = h.d[2];
    t[6 * ts] = h.l;
}

// A photon between surfaces, in the global frame: position and direction.  The medium it travels in
// is a property of the surface it travels to (kSurfGlassIn), the same for every photon.
struct Ray {
    double p[3], n[3];
};

// Per-photon constants of the optics stage: the glass index and its reciprocal (when the surfaces
// ahead need them) and the coating tables' wavelength column at the photon's wavelength.
struct Optics {
    double lam, n_glass, inv_glass;
    LamCol lc;
};
__device__ __forceinline__ Optics optics_of(const DevParams& P, const Launch& L, double lam,
                                            bool glass = true) {
    Optics c;
    c.lam = lam;
    c.n_glass = c.inv_glass = 1.0;
    if (glass && P.has_glass) {
        c.n_glass = sellmeier(P, lam);
        c.inv_glass = 1.0 / c.n_glass;
    }
    c.lc = (L.flags & PHX_F_COATINGS) && P.n_lam > 1 ? lambda_column(P, lam) : LamCol{0, 0.0};
    return c;
}
// Index of the medium in front of a surface, and its ratio to the index behind it (media vacuum and
// glass: 1, n, 1/n; exact where the quotient is).
__device__ __forceinline__ double index_before(const Optics& oc, uint32_t bits) {
    return bits & kSurfGlassIn ? oc.n_glass : 1.0;
}
__device__ __forceinline__ double index_ratio(const Optics& oc, uint32_t bits) {
    if (bits & kSurfGlass) return bits & kSurfGlassIn ? 1.0 : oc.inv_glass;
    return bits & kSurfGlassIn ? oc.n_glass : 1.0;
}

__device__ __forceinline__ void outcome_init(Outcome& o, double lam) {
    o.status = PHX_MISSED; o.surface = -1; o.newton = 0; o.pix_i = -1; o.pix_j = -1;
    o.x = o.y = o.z = o.xe = o.ye = 0.0;
    o.lam = lam;
}

// Central obscuration (section 2.4.1): true, with the outcome filled, if the ray meets it.
__device__ __forceinline__ bool obscured(const DevParams& P, const Ray& ray, Outcome& o) {
    if (!(P.obsc_r > 0.0)) return false;
    const double l = (P.obsc_z - ray.p[2]) / ray.n[2];
    const double x = fma(ray.n[0], l, ray.p[0]), y = fma(ray.n[1], l, ray.p[1]);
    if (!(dot2(x, x, y, y) < P.obsc_s)) return false;   // sqrt(x^2 + y^2) < obsc_r
    o.status = PHX_OBSCURED;
    o.x = x; o.y = y; o.z = P.obsc_z;
    return true;
}

// Before the first surface: aerosol extinction and the spider (when their flags are set), then
// the central obscuration.  True while the photon lives, else the outcome is filled.
template <bool EXTRA>
__device__ __forceinline__ bool entrance(const DevParams& P, const Launch& L, const Rng& rng,
                                         Ray& ray, Outcome& o) {
    if (EXTRA && (L.flags & (PHX_F_AEROSOL | PHX_F_SPIDER))) {
        const Entry e = entrance_extra(P, L.flags, rng, o.lam,
                                       make_double3(ray.p[0], ray.p[1], ray.p[2]),
                                       make_double3(ray.n[0], ray.n[1], ray.n[2]));
        if (e.status != 0) {
            o.status = e.status;
            o.x = e.p.x; o.y = e.p.y; o.z = e.p.z;
            return false;
        }
        ray.p[0] = e.p.x; ray.p[1] = e.p.y; ray.p[2] = e.p.z;
        ray.n[0] = e.n.x; ray.n[1] = e.n.y; ray.n[2] = e.n.z;
    }
    return !obscured(P, ray, o);
}

// Surfaces k0..k1-1 before the detector (sections 2.4.1-2.4.2): returns true while the photon
// lives, else fills the outcome.  wc / wc_block cache the roulette block of the last coated
// surface (wc_block = -1: none).
// A ghost branch met in the surface loop, kept for later: the hit at the reflecting surface k
// (k = -1: none) and the refractive index of the medium the photon travelled in.  The optics
// kernel appends it to the chunk's ghost list; a second pass of the kernel runs the branches,
// started at different surfaces or by different photons, together.
struct GhostStart {
    Hit h;
    int k;
    double n_cur;
};

// The chunk's list of ghost starts in device memory: cap entries of kGhostFields 8-byte fields,
// field-major (field f of entry e at f * cap + e): the hit (q, d, N, dn), the index of the
// medium, the wavelength, (surface << 32 | Newton steps so far) and the photon's position in the
// survivor list.  ghost_get reads one entry.
__device__ __forceinline__ void ghost_get(const double* q, uint64_t cap, uint64_t e, GhostStart& gs,
                                          double& lam, uint32_t& r, int& newton) {
    const double* f = q + e;
#pragma unroll
    for (int i = 0; i < 3; ++i) {
        gs.h.q[i] = f[(0 + i) * cap];
        gs.h.d[i] = f[(3 + i) * cap];
        gs.h.N[i] = f[(6 + i) * cap];
    }
    gs.h.dn = f[9 * cap];
    gs.h.l = 0.0;   // not used by the branch
    gs.n_cur = f[10 * cap];
    lam = f[11 * cap];
    const uint64_t kn = (uint64_t)__double_as_longlong(f[12 * cap]);
    gs.k = (int)(kn >> 32);
    newton = (int)(uint32_t)kn;
    r = (uint32_t)__double_as_longlong(f[13 * cap]);
}
// Where the sequential pass leaves a lane's ghost start: the hit's fields are written to LDS at the
// reflecting surface, so that no register carries them out of the surface loop, and k records the
// surface (-1: none).  The first seven go to an entry of the wavefront's queue that is free at the
// time (field i at f[i * kQueue]), the others to the lane's column of a staging area (at g[i * 64]): with
// all in an area of their own two workgroups fitted a compute unit, now three (2.6e7 photons
// 3.0 -> 2.9 ms).
constexpr int kQueue = 128;               // queued photons per wavefront (64 + 63 carried)
constexpr int kGhostQueued = 7;           // q, d, N_x
constexpr int kGhostStage = 4;            // N_y, N_z, dn, index of the medium
struct GhostSink {
    double* f;
    double* g;
    int k;
};
__device__ __forceinline__ void ghost_stage(GhostSink* gs, const Hit& h, int k, double n_cur) {
#pragma unroll
    for (int i = 0; i < 3; ++i) {
        gs->f[(0 + i) * kQueue] = h.q[i];
        gs->f[(3 + i) * kQueue] = h.d[i];
    }
    gs->f[6 * kQueue] = h.N[0];
    gs->g[0 * 64] = h.N[1];
    gs->g[1 * 64] = h.N[2];
    gs->g[2 * 64] = h.dn;
    gs->g[3 * 64] = n_cur;
    gs->k = k;
}
// Appends the lanes holding a ghost start (gs.k >= 0) to the list.  A wavefront with many units ahead
// of it reserves kGhostReserve entries at a time (ctr[0] counts the reserved ones; an entry beyond cap, which the
// list's size rules out, is not written): an atomic for each append, all on one address, held the pass
// up (2.6e7 photons 2.9 ms, now 2.35; the unused entries cost the branch pass 0.3 of its 4.7).  One with few
// reserves what it appends (`reserve` 0): most of its block would stay unused, and the branch pass would
// start a wavefront for each (3e5 photons without the pre-roll 534 us, now 372; the line at 2, 4, 8 units:
// 2e6 photons with the pre-roll 1.27, 1.22, 1.22 ms, 4e6 without 2.33, 2.33, 2.46).  Every lane of the wavefront must call it.
struct GhostRoom {
    uint64_t next, end;   // the wavefront's reserved, not yet written entries
    uint64_t reserve;     // entries to reserve at a time, at least
};
__device__ __forceinline__ void ghost_append(double* q, uint64_t cap, unsigned long long* ctr,
                                             GhostRoom& room, const GhostSink& gs, const Outcome& o,
                                             uint32_t r) {
    const bool pend = gs.k >= 0;
    const uint64_t pm = __ballot(pend);
    if (!pm) return;
    const uint64_t n = (uint64_t)__popcll(pm), avail = room.end - room.next;
    const uint64_t rank = (uint64_t)__popcll(pm & ((1ull << __lane_id()) - 1ull));
    uint64_t e = room.next + rank;
    if (n > avail) {
        const uint64_t more = max(n - avail, room.reserve);
        unsigned long long b = 0;
        if (__lane_id() == 0) b = atomicAdd(&ctr[0], (unsigned long long)more);
        b = __shfl(b, 0);
        if (rank >= avail) e = b + (rank - avail);
        room.next = b + (n - avail);
        room.end = b + more;
    } else {
        room.next += n;
    }
    if (pend && e < cap) {
        double* f = q + e;
#pragma unroll
        for (int i = 0; i < kGhostQueued; ++i) f[i * cap] = gs.f[i * kQueue];
#pragma unroll
        for (int i = 0; i < kGhostStage; ++i) f[(kGhostQueued + i) * cap] = gs.g[i * 64];
        f[11 * cap] = o.lam;
        f[12 * cap] = __longlong_as_double((long long)(((uint64_t)(uint32_t)gs.k << 32) |
                                                       (uint32_t)o.newton));
        f[13 * cap] = __longlong_as_double((long long)r);
    }
}
// The entries that stay unused at the wavefront's end: surface -1.
__device__ __forceinline__ void ghost_close(double* q, uint64_t cap, const GhostRoom& room) {
    for (uint64_t e = room.next + __lane_id(); e < room.end && e < cap; e += 64)
        q[12 * cap + e] = __longlong_as_double(-1ll);
}

template <bool ZERN, bool TAPE = false, bool GHOST = false>
__device__ __forceinline__ bool trace_surfaces(const DevParams& P, const Launch& L, const Rng& rng,
                                               const Optics& oc, Ray& ray, int k0, int k1,
                                               uint4& wc, int& wc_block, Outcome& o,
                                               double* tp = nullptr, uint64_t ts = 0,
                                               GhostSink* gs = nullptr) {
    Hit h;
#pragma unroll 1
    for (int k = k0; k < k1; ++k) {
        const DevSurface& s = P.surf[k];
        const SurfRegs sr = surf_regs(s);
        int st = hit_surface<ZERN, TAPE, GHOST>(P, L, rng, sr, k, ray.p, ray.n, oc.lc, wc, wc_block,
                                                h, o.newton);
        if (GHOST && st == kGhostReflect) {   // GHOST callers pass gs
            ghost_stage(gs, h, k, index_before(oc, sr.bits));
            return false;
        }
        if (TAPE) tape_put(tp, ts, k, h);
        if (sr.bits & kSurfMirror) {
            reflect_ray(h);
        } else if (!refract(h, index_ratio(oc, sr.bits)) && st == 0) {
            st = PHX_TIR;
        }
        if (st != 0) {
            o.status = st; o.surface = k; o.x = h.q[0]; o.y = h.q[1]; o.z = h.q[2];
            return false;
        }
        to_global(s, sr.bits, sr.tz, h.q, h.d, ray.p, ray.n);
    }
    return true;
}

// Landing on the detector after its coating and the refraction into silicon: conversion,
// diffusion and the pixel (sections 2.4.2-2.4.3); fills the outcome.
__device__ __forceinline__ void land(const DevParams& P, const Launch& L, const Rng& rng,
                                     const Optics& oc, const Hit& h, Outcome& o) {
    o.surface = P.n_surf - 1;
    o.x = h.q[0]; o.y = h.q[1]; o.z = h.q[2];
    double xc = h.q[0], yc = h.q[1];
    const int ss = sensor_stage(P, L, rng, oc.lam, h.d, xc, yc);
    if (ss != 0) {
        o.status = ss;
        return;
    }
    o.xe = xc; o.ye = yc;
    // pixel quantisation (section 2.4.3)
    const double ix = floor((xc - P.chip_x0) / P.pixel);
    const double iy = floor((yc - P.chip_y0) / P.pixel);
    o.status = PHX_OFF_CHIP;
    if (ix >= 0.0 && ix < (double)P.nx && iy >= 0.0 && iy < (double)P.ny) {
        o.status = PHX_DETECTED;
        o.pix_i = (int)ix;
        o.pix_j = (int)iy;
    }
}

// Medium codes on either side of surface k in travel order and their indices.
__device__ __forceinline__ int medium_before(const DevParams& P, int k) {
    return k > 0 ? P.surf[k - 1].medium : PHX_VACUUM;
}
__device__ __forceinline__ double medium_index(const Optics& oc, int m) {
    return m == PHX_GLASS ? oc.n_glass : (m == PHX_SILICON ? n_silicon(oc.lam) : 1.0);
}

// A ghost (section 2.4.2): the photon was reflected by the coating of refracting surface k (hit
// h, element frame) and propagates backwards; from here on its next surface is the nearest one
// ahead along the ray among all surfaces but the current one (intersection distance above
// 1e-9 m), where it is transmitted into the medium on the other side, reflected (a mirror, or a
// coating's reflection), absorbed or vignetted, for at most kGhostMax interactions (interaction
// i draws its roulette word from stream 4, block i).  Reaching the detector it lands as usual.
// ghost_begin sets up the branch, ghost_step performs one interaction.
constexpr int kGhostMax = 16;
struct GhostRay {
    double p[3], n[3];   // global frame
    double n_cur;        // index of the medium the photon travels in
    int medium, from, inter;
};

__device__ __forceinline__ void ghost_begin(const DevParams& P, Hit h, int k, double n_cur,
                                            GhostRay& gr) {
    gr.medium = medium_before(P, k);
    gr.n_cur = n_cur;
    gr.from = k;
    gr.inter = 0;
    // reflect at k and return to the global frame
    reflect_ray(h);
    const DevSurface& s = P.surf[k];
    to_global(s, s.bits, s.tz, h.q, h.d, gr.p, gr.n);
}

// One interaction of a ghost branch; true when the photon's fate is settled (o filled).
template <bool ZERN>
__device__ __forceinline__ bool ghost_step(const DevParams& P, const Launch& L, const Rng& rng,
                                        const Optics& oc, GhostRay& gr, Outcome& o) {
    // the nearest surface ahead; the search keeps the best candidate's frame coordinates, path
    // length, slope and Newton steps, so that its hit is finished without intersecting again
    double best = INFINITY;
    int bk = -1;
    Hit h;
    double bgx = 0.0, bgy = 0.0;
    int bit = 0;
    if (gr.inter < kGhostMax) {
#pragma unroll 1
        for (int j = 0; j < P.n_surf; ++j) {
            if (j == gr.from) continue;
            const DevSurface& s = P.surf[j];
            const SurfRegs sr = surf_regs(s);
            double q[3], d[3];
            to_element(s, sr, gr.p, gr.n, q, d);
            double l, gx, gy;
            int it = 0;
            if (intersect<ZERN, true>(P, s, sr, q, d, l, gx, gy, it) == 0 && l > 1e-9 && l < best) {
                best = l;
                bk = j;
                h.q[0] = q[0]; h.q[1] = q[1]; h.q[2] = q[2];
                h.d[0] = d[0]; h.d[1] = d[1]; h.d[2] = d[2];
                bgx = gx;
                bgy = gy;
                bit = it;
            }
        }
    }
    if (bk < 0) {   // leaves the optics, or the interaction limit is reached
        o.status = PHX_MISSED;
        o.surface = gr.from;
        o.x = gr.p[0]; o.y = gr.p[1]; o.z = gr.p[2];
        return true;
    }
    const DevSurface& s = P.surf[bk];
    // the interaction: the hit point, aperture and normal (as the sequential passage takes
    // them), then the roulette with this interaction's own word
    o.newton += bit;
    advance(h, best);
    {
        const double rq2 = dot2(h.q[0], h.q[0], h.q[1], h.q[1]);
        if (rq2 < s.r_in2 || rq2 > s.r_out2) {
            o.status = PHX_VIGNETTED; o.surface = bk; o.x = h.q[0]; o.y = h.q[1]; o.z = h.q[2];
            return true;
        }
        hit_normal<ZERN, true>(s.bits, bgx, bgy, h);
    }
    bool reflect = s.kind == PHX_MIRROR;
    if ((L.flags & PHX_F_COATINGS) && s.coating >= 0) {
        const double u = u01(rng.block((uint32_t)gr.inter, 4).x);
        const double sv = 1.0 - h.dn * h.dn;
        const double T = coating(P, s.coat, sv, oc.lc);
        if (!(u < T)) {
            const double R = s.kind != PHX_MIRROR ? coating(P, reflectance(P, s.coat), sv, oc.lc) : 0.0;
            if (!(u < T + R)) {
                o.status = PHX_ABSORBED; o.surface = bk;
                o.x = h.q[0]; o.y = h.q[1]; o.z = h.q[2];
                return true;
            }
            reflect = true;
        }
    }
    const bool det = s.kind == PHX_DETECTOR;
    if (reflect) {
        reflect_ray(h);
    } else if (!det || (L.flags & PHX_F_SILICON)) {
        const int after = s.medium, before = medium_before(P, bk);
        const int m2 = gr.medium == after ? before : after;
        const double n2 = medium_index(oc, m2);
        if (!refract(h, gr.n_cur / n2)) {
            o.status = PHX_TIR; o.surface = bk; o.x = h.q[0]; o.y = h.q[1]; o.z = h.q[2];
            return true;
        }
        gr.n_cur = n2;
        gr.medium = m2;
    }
    if (det && !reflect) {
        land(P, L, rng, oc, h, o);
        return true;
    }
    to_global(s, s.bits, s.tz, h.q, h.d, gr.p, gr.n);
    gr.from = bk;
    gr.inter += 1;
    return false;
}

// The detector surface: its coating, the refraction into silicon, then the landing (sections
// 2.4.2-2.4.3); fills the outcome.  GHOST: a reflection by the detector's coating starts a ghost.
template <bool ZERN, bool TAPE = false, bool GHOST = false>
__device__ __forceinline__ void finish_detector(const DevParams& P, const Launch& L,
                                                const Rng& rng, const Optics& oc, Ray& ray,
                                                uint4& wc, int& wc_block, Outcome& o,
                                                double* tp = nullptr, uint64_t ts = 0,
                                                GhostSink* gs = nullptr) {
    const int kdet = P.n_surf - 1;
    Hit h;
    const SurfRegs sr = surf_regs(P.surf[kdet]);
    int st = hit_surface<ZERN, TAPE, GHOST>(P, L, rng, sr, kdet, ray.p, ray.n, oc.lc, wc, wc_block,
                                            h, o.newton);
    const double n_in = index_before(oc, sr.bits);
    if (GHOST && st == kGhostReflect) {   // GHOST callers pass gs
        ghost_stage(gs, h, kdet, n_in);
        return;
    }
    if (TAPE) tape_put(tp, ts, kdet, h);
    if (st == 0 && (L.flags & PHX_F_SILICON) && !refract(h, n_in / n_silicon(oc.lam)))
        st = PHX_TIR;
    if (st != 0) {
        o.status = st;
        o.surface = kdet;
        o.x = h.q[0]; o.y = h.q[1]; o.z = h.q[2];
        return;
    }
    land(P, L, rng, oc, h, o);
}

// Central obscuration, the surfaces (sections 2.4.1-2.4.2), silicon (sections 2.4.2-2.4.3) and
// the pixel, from the start-plane state.  With TAPE, every surface passage is recorded for the
// adjoint sweep.
template <bool ZERN, bool TAPE = false>
__device__ Outcome photon_back(const DevParams& P, const Launch& L, int si, uint64_t idx,
                               const Front& f, double* tp = nullptr, uint64_t ts = 0) {
    Outcome o;
    outcome_init(o, f.lam);
    const Rng rng{L.seed, (uint32_t)si, (uint32_t)idx, (uint32_t)(idx >> 32)};
    Ray ray{{f.p[0], f.p[1], f.p[2]}, {f.n[0], f.n[1], f.n[2]}};
    if (!entrance<true>(P, L, rng, ray, o)) return o;
    const Optics oc = optics_of(P, L, f.lam);
    uint4 wc = make_uint4(0, 0, 0, 0);
    int wc_block = -1;
    if (!trace_surfaces<ZERN, TAPE>(P, L, rng, oc, ray, 0, P.n_surf - 1, wc, wc_block, o, tp, ts))
        return o;
    finish_detector<ZERN, TAPE>(P, L, rng, oc, ray, wc, wc_block, o, tp, ts);
    return o;
}

// Wavefront-aggregated increment: lanes with the same pixel elect one leader that adds the
// group's count.  Every lane of the wavefront must call it.
__device__ __forceinline__ void bin_photon(uint32_t* image, int pix, bool active) {
    uint64_t pending = __ballot(active);
    const int lane = __lane_id();
    while (pending) {
        const int leader = __ffsll((unsigned long long)pending) - 1;
        const int key = __shfl(pix, leader);
        const uint64_t same = __ballot(active && pix == key);
        if (lane == leader) atomicAdd(&image[key], (uint32_t)__popcll(same));
        pending &= ~same;
    }
}

// Flattened launch index g -> (source, photon index).
__device__ __forceinline__ void decode(const Launch& L, uint64_t g, int& si, uint64_t& idx) {
    int s;
    uint64_t local;
    if (L.n_src == 1) {
        s = 0;
        local = g;
    } else if (L.uniform_count) {
        s = (int)(g / L.uniform_count);
        local = g - (uint64_t)s * L.uniform_count;
    } else {
        // largest s with prefix[s] <= g, between the sources of the guide blocks around g
        const uint64_t b = g >> L.guide_shift;
        int lo = L.src_guide[b], hi = L.src_guide[b + 1];
        while (lo < hi) {
            const int mid = (lo + hi + 1) >> 1;
            if (L.prefix[mid] <= g) lo = mid; else hi = mid - 1;
        }
        s = lo;
        local = g - L.prefix[s];
    }
    si = L.src_begin + s;
    idx = L.photon_begin + local;
}

__device__ __forceinline__ void write_event(const Launch& L, uint64_t g, int si, uint64_t idx,
                                            const Outcome& o) {
    phx_event& e = L.events[g / L.event_stride];
    e.photon = idx; e.source = si; e.status = o.status; e.surface = o.surface;
    e.pix_i = o.pix_i; e.pix_j = o.pix_j; e.newton = o.newton;
    e.x = o.x; e.y = o.y; e.z = o.z; e.xe = o.xe; e.ye = o.ye; e.lambda = o.lam;
}

// Book-keeping of one traced photon: event record; returns the pixel to bin (-1 for none).
__device__ __forceinline__ int account(const DevParams& P, const Launch& L, uint64_t g, int si,
                                       uint64_t idx, const Outcome& o) {
    if ((L.flags & PHX_F_EVENTS) && (g % L.event_stride) == 0) write_event(L, g, si, idx, o);
    return o.status == PHX_DETECTED ? o.pix_j * P.nx + o.pix_i : -1;
}

__device__ __forceinline__ int stat_slot(const Outcome& o) {
    return o.status * PHX_STAT_COLS + min(o.surface + 1, PHX_STAT_COLS - 1);
}

// Status count: one LDS atomic per photon (the LDS unit adds lanes of one address one after the
// other, beside the wavefronts' arithmetic; electing a leader per status took a hundred instructions).
__device__ __forceinline__ void count_stat(uint32_t* s_stats, int slot, bool active) {
    if (active) atomicAdd(&s_stats[slot], 1u);
}

// Exact per-source moments of converted photons.  Positions are quantised to 2^-44 m and the
// sums (count, X, Y, X^2, Y^2, XY) are accumulated as 128-bit integers, so the result is
// independent of the order in which photons arrive.  Lanes of the wavefront that hold the same
// source are summed with cross-lane shuffles first; the group's leader then adds the sums with
// one pair of 64-bit atomics per 128-bit word (the low word's carry goes into the high word).
// Every lane of the wavefront must call it.
__device__ __forceinline__ void wave_sum128(unsigned __int128& v) {
#pragma unroll
    for (int m = 1; m < 64; m <<= 1) {
        const uint64_t lo = __shfl_xor((unsigned long long)(uint64_t)v, m);
        const uint64_t hi = __shfl_xor((unsigned long long)(uint64_t)(v >> 64), m);
        v += ((unsigned __int128)hi << 64) | lo;
    }
}

__device__ __forceinline__ void atomic_add128(unsigned long long* w, unsigned __int128 v) {
    const unsigned long long lo = (unsigned long long)v, hi = (unsigned long long)(v >> 64);
    const unsigned long long old = atomicAdd(w, lo);
    const unsigned long long carry = old + lo < old ? 1ull : 0ull;
    if (hi + carry) atomicAdd(w + 1, hi + carry);
}

// Moments of one source are first gathered in a per-workgroup LDS record (the first source the
// workgroup meets, s_src); other sources, and the record at the end of the workgroup, go to the
// global words.  Without it every wavefront of a one-source launch would add to the same twelve
// global words.
struct MomentCache {
    unsigned long long w[PHX_MOMENT_WORDS];
    int src;
};

__device__ __forceinline__ void moment_cache_init(MomentCache* mc) {
    if (threadIdx.x < PHX_MOMENT_WORDS) mc->w[threadIdx.x] = 0ull;
    if (threadIdx.x == 0) mc->src = -1;
}

// Called by one thread after the workgroup's last add_moments (and a barrier).
__device__ __forceinline__ void moment_cache_flush(const Launch& L, MomentCache* mc) {
    if (mc->src < 0) return;
    unsigned long long* w = L.moments + (size_t)mc->src * PHX_MOMENT_WORDS;
    atomicAdd(w, mc->w[0]);
    for (int i = 0; i < 5; ++i)
        atomic_add128(w + 2 + 2 * i, ((unsigned __int128)mc->w[3 + 2 * i] << 64) | mc->w[2 + 2 * i]);
}

__device__ void add_moments(const Launch& L, int si, double xe, double ye, bool active,
                            MomentCache* mc) {
    uint64_t pending = __ballot(active);
    const int lane = __lane_id();
    while (pending) {
        const int leader = __ffsll((unsigned long long)pending) - 1;
        const int key = __shfl(si, leader);
        const bool mine = active && si == key;
        const uint64_t same = __ballot(mine);
        pending &= ~same;
        const double q = 17592186044416.0;   // 2^PHX_MOMENT_Q_LOG2
        const long long X = mine ? __double2ll_rn(xe * q) : 0;
        const long long Y = mine ? __double2ll_rn(ye * q) : 0;
        unsigned __int128 v[5] = {(unsigned __int128)(__int128)X, (unsigned __int128)(__int128)Y,
                                  (unsigned __int128)((__int128)X * X),
                                  (unsigned __int128)((__int128)Y * Y),
                                  (unsigned __int128)((__int128)X * Y)};
#pragma unroll
        for (int i = 0; i < 5; ++i) wave_sum128(v[i]);
        if (lane == leader) {
            int cached = mc->src;
            if (cached < 0) {
                const int prev = atomicCAS(&mc->src, -1, key);
                cached = prev < 0 ? key : prev;
            }
            unsigned long long* w = cached == key ? mc->w
                                                  : L.moments + (size_t)key * PHX_MOMENT_WORDS;
            atomicAdd(w, (unsigned long long)__popcll(same));
#pragma unroll
            for (int i = 0; i < 5; ++i) atomic_add128(w + 2 + 2 * i, v[i]);
        }
    }
}

__device__ __forceinline__ void stats_init(uint32_t* s_stats) {
    for (int i = threadIdx.x; i < PHX_STATS_LEN; i += blockDim.x) s_stats[i] = 0;
    __syncthreads();
}

__device__ __forceinline__ void stats_flush(const Launch& L, uint32_t* s_stats, uint32_t newton,
                                            uint32_t traced) {
    atomicAdd(&s_stats[PHX_STAT_NEWTON], newton);
    atomicAdd(&s_stats[PHX_STAT_TRACED], traced);
    __syncthreads();
    if (L.stats) {
        for (int i = threadIdx.x; i < PHX_STATS_LEN; i += blockDim.x)
            if (s_stats[i]) atomicAdd(&L.stats[i], (unsigned long long)s_stats[i]);
    }
}

// Pre-roll (section 3.2, dynamic transmission optimisation).  Each workgroup takes contiguous
// ranges of photons (range_log2).  Stage one draws every photon's wavelength and pupil radius, drops
// photons whose pupil sample cannot reach the primary's aperture (the annulus is sampled wider
// than the aperture to leave room for atmospheric displacement, which the host bounds) and
// applies the most selective coating test; its survivors are queued in LDS (offset, wavelength column,
// sort key) and stage two applies the remaining tests to them densely, so the many
// photons that fail the first test cost one test.  Stage two also flags the photons whose
// conversion word passes the escape filter, and stage three (only when any is flagged) runs the
// exact escape test on them out of the main loops' register budget.  Last, the survivors' ranks in
// the range's bitmap (photon order, whatever the queue's) give each its place: in the range's
// segment, with its sort key, for the sort to list; or straight in the list of photons to trace, behind
// the ranges that came before (any order of ranges; the images do not depend on it).
constexpr int kGenRange = 4096;         // photons per range at most (64 bitmap words)

// Sort key of a photon: pupil sector (the top bits of the angle word), class, time bucket (the
// top bits of the time word: the time stamp is t_e u01(w)).  Where all photons are of one class
// (the pre-roll without ghosts) the time takes its bit too.
template <bool CLASS>
__device__ __forceinline__ uint32_t sort_key(const uint4& w0, bool passes) {
    const uint32_t sector = (w0.y >> 29) << 7;
    return CLASS ? sector | (passes ? kSortClass : 0u) | (w0.z >> 26) : sector | (w0.z >> 25);
}

__device__ __forceinline__ void culled_event(const Launch& L, uint64_t g, int si, uint64_t idx,
                                             double lam) {
    if ((L.flags & PHX_F_EVENTS) && (g % L.event_stride) == 0) {
        Outcome o;
        o.status = PHX_CULLED; o.surface = -1; o.newton = 0; o.pix_i = o.pix_j = -1;
        o.x = o.y = o.z = o.xe = o.ye = 0.0;
        o.lam = lam;
        write_event(L, g, si, idx, o);
    }
}

// Photon r of a chunk: its flattened index, source and index within the source.  ONE: every photon
// of the chunk belongs to source one_si, whose first photon has flattened index `first` (the source
// index and the Philox key are then uniform over the workgroup).
template <bool ONE>
__device__ __forceinline__ void chunk_photon(const Launch& L, uint64_t begin, uint64_t r, int one_si,
                                             uint64_t first, uint64_t& g, int& si, uint64_t& idx) {
    g = begin + r;
    if constexpr (ONE) {
        si = one_si;
        idx = L.photon_begin + (g - first);
    } else {
        decode(L, g, si, idx);
    }
}

template <bool ONE, bool GHOST>
__global__ __launch_bounds__(kBlock) __attribute__((amdgpu_waves_per_eu(6))) void generate_kernel(const DevParams* __restrict__ Pg,
                                                          const Launch L, uint64_t begin,
                                                          uint64_t len, int one_si,
                                                          uint64_t first, int log2_range,
                                                          uint32_t* __restrict__ seg,
                                                          uint32_t* __restrict__ seg_n,
                                                          uint32_t* __restrict__ surv,
                                                          unsigned int* __restrict__ count) {
    __shared__ unsigned long long s_bits[kGenRange / 64];
    __shared__ uint32_t s_pre[kGenRange / 64];   // survivors before each bitmap word
    // queued photon: offset | wavelength column << 12 | escape test << 31; its sort key
    __shared__ uint32_t s_q[kGenRange];
    __shared__ uint16_t s_k[kGenRange];
    __shared__ unsigned int s_qn, s_esc, s_culled, s_base;
    const DevParams& P = *Pg;
    const int lane = __lane_id();
    // with ghosts a photon may leave the sequential path at a coated refracting surface, after
    // which the sequential roulette words no longer decide its fate: only the coated surfaces
    // ahead of the first coated refracting one (the mirrors) are tested then
    const int n_tests = P.n_cull;
    const int k_lim = GHOST ? P.ghost_cull_limit : PHX_MAX_SURF;
    // the chunk's one source, read once (the other case reads each photon's source record)
    DevSource one_src{};
    if constexpr (ONE) one_src = P.src[one_si];
    const int n_iter = 1 << (log2_range - 8);
    const uint64_t n_ranges = (len + (1ull << log2_range) - 1) >> log2_range;
    if (threadIdx.x == 0) s_culled = 0;
    for (uint64_t rg = blockIdx.x; rg < n_ranges; rg += gridDim.x) {   // workgroup-uniform
        const uint64_t r0 = rg << log2_range;
        if (threadIdx.x < kGenRange / 64) s_bits[threadIdx.x] = 0ull;
        if (threadIdx.x == 0) {
            s_qn = 0;
            s_esc = 0;
        }
        __syncthreads();
        // stage one: wavelength and the first test for every photon of the range
        for (int it = 0; it < n_iter; ++it) {
            const int rr = it * kBlock + threadIdx.x;
            const uint64_t r = r0 + rr;
            bool pass = false, culled = false;
            uint32_t entry = 0, key = 0;
            if (r < len) {
                uint64_t g, idx;
                int si;
                chunk_photon<ONE>(L, begin, r, one_si, first, g, si, idx);
                const Rng rng{L.seed, (uint32_t)si, (uint32_t)idx, (uint32_t)(idx >> 32)};
                uint4 w0;
                const double lam = preroll_draw(P, rng, ONE ? one_src : P.src[si], w0);
                // squared pupil radius as the sky stage samples it: outside the reachable annulus
                // the photon is vignetted at the primary whatever the atmosphere does (the bounds
                // carry a margin far above the rounding of the square root)
                const double ro = P.pupil_r_out + L.pupil_margin;
                const double ri = fmax(P.pupil_r_in - L.pupil_margin, 0.0);
                const double rp2 = u01(w0.x) * (ro * ro - ri * ri) + ri * ri;
                const int il = lambda_column(P, lam).il;
                culled = rp2 < L.cull_r2_lo || rp2 > L.cull_r2_hi ||
                         (n_tests > 0 && preroll_first<GHOST>(P, rng, il, k_lim));
                pass = !culled;
                if (culled) culled_event(L, g, si, idx, lam);
                entry = (uint32_t)rr | ((uint32_t)il << 12);
                key = sort_key<GHOST>(w0, true);
            }
            const uint64_t pm = __ballot(pass), cm = __ballot(culled);
            unsigned int base = 0;
            if (lane == 0) {
                if (pm) base = atomicAdd(&s_qn, (unsigned int)__popcll(pm));
                if (cm) atomicAdd(&s_culled, (unsigned int)__popcll(cm));
            }
            base = __shfl(base, 0);
            if (pass) {
                const unsigned int e = base + __popcll(pm & ((1ull << lane) - 1ull));
                s_q[e] = entry;
                s_k[e] = (uint16_t)key;
            }
        }
        __syncthreads();
        // stage two: the remaining tests for the queued photons
        const unsigned int qn = s_qn;
        for (unsigned int q0 = 0; q0 < qn; q0 += kBlock) {
            const unsigned int qi = q0 + threadIdx.x;
            bool culled = false;
            if (qi < qn) {
                const uint32_t entry = s_q[qi];
                const int rr = (int)(entry & 0xfffu);
                uint64_t g, idx;
                int si;
                chunk_photon<ONE>(L, begin, r0 + rr, one_si, first, g, si, idx);
                const Rng rng{L.seed, (uint32_t)si, (uint32_t)idx, (uint32_t)(idx >> 32)};
                const int il = (int)((entry >> 12) & 0x1fffu);
                culled = preroll_rest<GHOST>(P, rng, il, n_tests, k_lim);
                const uint32_t et = P.esc_thr && il >= P.esc_col0 ? P.esc_thr[il] : 0u;
                bool later = false;
                if (!culled && et && (L.flags & PHX_F_SILICON)) {
                    // escape: a quick filter on the conversion word here; the exact test in
                    // stage three, out of this loop's register budget
                    later = rng.block(1).z < et;
                    if (later) {
                        s_q[qi] = entry | (1u << 31);
                        s_esc = 1u;
                    }
                }
                // with ghosts the photons that the most selective coating turns back stay in: a
                // class of their own
                if (GHOST && !culled && n_tests > 0 &&
                    preroll_first<false>(P, rng, il, PHX_MAX_SURF))
                    s_k[qi] &= (uint16_t)~kSortClass;
                if (!culled && !later) {
                    atomicOr(&s_bits[rr >> 6], 1ull << (rr & 63));
                } else if ((L.flags & PHX_F_EVENTS) && (g % L.event_stride) == 0) {
                    uint4 w0;
                    culled_event(L, g, si, idx, preroll_draw(P, rng, ONE ? one_src : P.src[si], w0));
                }
            }
            const uint64_t cm = __ballot(culled);
            if (lane == 0 && cm) atomicAdd(&s_culled, (unsigned int)__popcll(cm));
        }
        // stage three: the exact escape test for the photons stage two flagged
        __syncthreads();
        if (s_esc) {
            for (unsigned int q0 = 0; q0 < qn; q0 += kBlock) {
                const unsigned int qi = q0 + threadIdx.x;
                const uint32_t entry = qi < qn ? s_q[qi] : 0u;
                bool culled = false;
                if (entry >> 31) {
                    const int rr = (int)(entry & 0xfffu);
                    uint64_t g, idx;
                    int si;
                    chunk_photon<ONE>(L, begin, r0 + rr, one_si, first, g, si, idx);
                    const Rng rng{L.seed, (uint32_t)si, (uint32_t)idx, (uint32_t)(idx >> 32)};
                    uint4 w0;
                    const double lam = preroll_draw(P, rng, ONE ? one_src : P.src[si], w0);
                    culled = escape_certain(P, lam, rng.block(1).z);
                    if (!culled)
                        atomicOr(&s_bits[rr >> 6], 1ull << (rr & 63));
                    else
                        culled_event(L, g, si, idx, lam);
                }
                const uint64_t cm = __ballot(culled);
                if (lane == 0 && cm) atomicAdd(&s_culled, (unsigned int)__popcll(cm));
            }
            __syncthreads();
        }
        // places: wavefront 0 scans the bitmap's counts
        if (threadIdx.x < 64) {
            const uint32_t n = (uint32_t)__popcll(s_bits[lane]);
            uint32_t v = n;
#pragma unroll
            for (int d = 1; d < 64; d <<= 1) {
                const uint32_t o = __shfl_up(v, d);
                if (lane >= d) v += o;
            }
            s_pre[lane] = v - n;
            if (lane == 63) {
                if (surv)
                    s_base = atomicAdd(count, v);
                else
                    seg_n[rg] = v;
            }
        }
        __syncthreads();
        for (unsigned int qi = threadIdx.x; qi < qn; qi += kBlock) {
            const uint32_t rr = s_q[qi] & 0xfffu;
            const unsigned long long w = s_bits[rr >> 6];
            if (!((w >> (rr & 63)) & 1ull)) continue;
            const uint32_t at = s_pre[rr >> 6] + (uint32_t)__popcll(w & ((1ull << (rr & 63)) - 1ull));
            if (surv)
                surv[s_base + at] = (uint32_t)r0 + rr;
            else
                seg[r0 + at] = rr | ((uint32_t)s_k[qi] << 12);
        }
        __syncthreads();
    }
    if (threadIdx.x == 0 && L.stats && s_culled)
        atomicAdd(&L.stats[PHX_CULLED * PHX_STAT_COLS], (unsigned long long)s_culled);
}

// Without the pre-roll every photon is traced: the sort's segments hold them all, classed by whether
// the most selective coating can let them pass.
template <bool ONE>
__global__ __launch_bounds__(kBlock) void list_kernel(const DevParams* __restrict__ Pg,
                                                      const Launch L, uint64_t begin, uint64_t len,
                                                      int one_si, uint64_t first, int log2_range,
                                                      uint32_t* __restrict__ seg,
                                                      uint32_t* __restrict__ seg_n) {
    const DevParams& P = *Pg;
    const uint64_t n = (uint64_t)gridDim.x * kBlock;
    for (uint64_t r = (uint64_t)blockIdx.x * kBlock + threadIdx.x; r < len; r += n) {
        uint64_t g, idx;
        int si;
        chunk_photon<ONE>(L, begin, r, one_si, first, g, si, idx);
        const Rng rng{L.seed, (uint32_t)si, (uint32_t)idx, (uint32_t)(idx >> 32)};
        uint4 w0;
        const double lam = preroll_draw(P, rng, P.src[si], w0);
        bool passes = true;
        if ((L.flags & PHX_F_COATINGS) && P.n_cull > 0)
            passes = !preroll_first<false>(P, rng, lambda_column(P, lam).il, PHX_MAX_SURF);
        const uint64_t rr = r & ((1ull << log2_range) - 1);
        seg[r] = (uint32_t)rr | (sort_key<true>(w0, passes) << 12);
        if (rr == 0) seg_n[r >> log2_range] = (uint32_t)min((uint64_t)1 << log2_range, len - r);
    }
}

// Without the pre-roll and without an atmosphere only the class matters, and photons of a source
// should stay together (the moments' sums of a wavefront): one pass lists the photons that the most
// selective coating can let pass from the front and the ones that it stops from the back, in pieces of a
// range each (1e7 photons 62 us; as a sort of two keys 213 us).  ctr: photons listed so far, from the front
// in the low half, from the back in the high half.
constexpr int kClassRange = 4096;

template <bool ONE>
__global__ __launch_bounds__(kBlock) void class_kernel(const DevParams* __restrict__ Pg,
                                                       const Launch L, uint64_t begin, uint64_t len,
                                                       int one_si, uint64_t first,
                                                       uint32_t* __restrict__ surv,
                                                       unsigned int* __restrict__ count,
                                                       unsigned long long* __restrict__ ctr) {
    __shared__ unsigned long long s_bits[kClassRange / 64];
    __shared__ uint32_t s_pre[kClassRange / 64];
    __shared__ unsigned long long s_base;
    const DevParams& P = *Pg;
    const int lane = __lane_id(), wave = threadIdx.x >> 6;
    if (blockIdx.x == 0 && threadIdx.x == 0) *count = (unsigned int)len;
    for (uint64_t r0 = (uint64_t)blockIdx.x * kClassRange; r0 < len;
         r0 += (uint64_t)gridDim.x * kClassRange) {   // workgroup-uniform
        const uint32_t n = (uint32_t)min((uint64_t)kClassRange, len - r0);
        for (int it = 0; it < kClassRange / kBlock; ++it) {
            const uint32_t rr = it * kBlock + threadIdx.x;
            bool passes = false;
            if (rr < n) {
                uint64_t g, idx;
                int si;
                chunk_photon<ONE>(L, begin, r0 + rr, one_si, first, g, si, idx);
                const Rng rng{L.seed, (uint32_t)si, (uint32_t)idx, (uint32_t)(idx >> 32)};
                uint4 w0;
                const double lam = preroll_draw(P, rng, P.src[si], w0);
                passes = !preroll_first<false>(P, rng, lambda_column(P, lam).il, PHX_MAX_SURF);
            }
            const unsigned long long b = __ballot(passes);
            if (lane == 0) s_bits[it * (kBlock / 64) + wave] = b;
        }
        __syncthreads();
        if (wave == 0) {
            const uint32_t c = (uint32_t)__popcll(s_bits[lane]);
            uint32_t v = c;
#pragma unroll
            for (int d = 1; d < 64; d <<= 1) {
                const uint32_t o = __shfl_up(v, d);
                if (lane >= d) v += o;
            }
            s_pre[lane] = v - c;
            if (lane == 63) s_base = atomicAdd(ctr, v | ((unsigned long long)(n - v) << 32));
        }
        __syncthreads();
        const uint64_t front = s_base & 0xffffffffull, back = len - 1 - (s_base >> 32);
        for (uint32_t rr = threadIdx.x; rr < n; rr += kBlock) {
            const unsigned long long w = s_bits[rr >> 6];
            const uint32_t at = s_pre[rr >> 6] + (uint32_t)__popcll(w & ((1ull << lane) - 1ull));
            surv[(w >> lane) & 1ull ? front + at : back - (rr - at)] = (uint32_t)r0 + rr;
        }
        __syncthreads();
    }
}

// The sort: a counting sort of a chunk's photons to trace by (pupil sector, class, time
// bucket), over groups of ranges (sort_group_log2).  What it is for:
//  - time: photons traced together see the same wind-shifted stretch of every phase screen;
//  - sector: workgroups go to the eight dies in turn and each die has its own L2, so the sky kernel gives
//    every die the photons of one eighth of the pupil, whose stretch of the screens is an eighth
//    as wide;
//  - class: photons that the most selective coating stops share wavefronts, which end there.
// sort_count: photons per group and key.  sort_scan: their prefixes over the groups, and the
// totals.  sort_scatter: each photon's place, from an LDS counter per wavefront and key.  STABLE (an
// adjoint, whose sums take this order): lanes of one key take their places in lane order, so
// that the list is the same on every run.  Otherwise the order within a key and wavefront is of
// no effect, and the plain atomic is cheaper beside the optics stage (1e9 photons 41.7 ms, with
// the ranking 42.4).
constexpr int kSortBlock = 512;
constexpr int kSortWaves = kSortBlock / 64;
constexpr int kSortBatch = 8;

// The active lanes of the wavefront that hold this lane's key.
__device__ __forceinline__ uint64_t same_key(uint32_t key) {
    uint64_t m = __ballot(1);
#pragma unroll
    for (int b = 0; b < kSortKeyBits; ++b) {
        const bool on = (key >> b) & 1u;
        const uint64_t v = __ballot(on);
        m &= on ? v : ~v;
    }
    return m;
}

// f(entry, range) for the photons of this wavefront's ranges, 64 at a time; kSortBatch loads are in flight
// together (one at a time, a wavefront waited out the memory's latency for every 64 photons).
template <class F>
__device__ __forceinline__ void for_each_listed(const uint32_t* seg, const uint32_t* seg_n,
                                                uint64_t n_ranges, int log2_range, int log2_group, F f) {
    const int lane = threadIdx.x & 63;
    const int per_wave = (1 << log2_group) / kSortWaves;
    const uint64_t rg0 = ((uint64_t)blockIdx.x << log2_group) + (threadIdx.x >> 6) * per_wave;
    for (int i = 0; i < per_wave; ++i) {
        const uint64_t rg = rg0 + i;
        if (rg >= n_ranges) break;
        const uint32_t n = seg_n[rg];
        const uint32_t* e = seg + (rg << log2_range);
        for (uint32_t k0 = 0; k0 < n; k0 += 64 * kSortBatch) {
            uint32_t v[kSortBatch];
#pragma unroll
            for (int j = 0; j < kSortBatch; ++j) {
                const uint32_t k = k0 + 64 * j + lane;
                v[j] = e[k < n ? k : n - 1];
            }
#pragma unroll
            for (int j = 0; j < kSortBatch; ++j)
                if (k0 + 64 * j + lane < n) f(v[j], rg);
        }
    }
}

__global__ __launch_bounds__(kSortBlock) void sort_count(const uint32_t* __restrict__ seg,
                                                         const uint32_t* __restrict__ seg_n,
                                                         uint64_t n_ranges, int log2_range,
                                                         int log2_group,
                                                         uint32_t* __restrict__ hist) {
    __shared__ uint32_t s_h[kSortKeys];
    for (int k = threadIdx.x; k < kSortKeys; k += kSortBlock) s_h[k] = 0;
    __syncthreads();
    for_each_listed(seg, seg_n, n_ranges, log2_range, log2_group,
                    [&](uint32_t e, uint64_t) { atomicAdd(&s_h[e >> 12], 1u); });
    __syncthreads();
    for (int k = threadIdx.x; k < kSortKeys; k += kSortBlock)
        hist[(uint64_t)blockIdx.x * kSortKeys + k] = s_h[k];
}

// One workgroup per 16 keys; 16 threads share a key's groups.
__global__ __launch_bounds__(kBlock) void sort_scan(uint32_t* __restrict__ hist, uint32_t n_groups,
                                                    uint32_t* __restrict__ tot) {
    __shared__ uint32_t s_sum[16][17];
    const int key = blockIdx.x * 16 + (threadIdx.x & 15), part = threadIdx.x >> 4;
    const uint32_t per = (n_groups + 15) / 16;
    const uint32_t a = min(n_groups, part * per), b = min(n_groups, a + per);
    uint32_t sum = 0;
#pragma unroll 8
    for (uint32_t g = a; g < b; ++g) sum += hist[(uint64_t)g * kSortKeys + key];
    s_sum[part][threadIdx.x & 15] = sum;
    __syncthreads();
    uint32_t run = 0, all = 0;
    for (int p = 0; p < 16; ++p) {
        const uint32_t v = s_sum[p][threadIdx.x & 15];
        if (p < part) run += v;
        all += v;
    }
#pragma unroll 8
    for (uint32_t g = a; g < b; ++g) {
        const uint32_t v = hist[(uint64_t)g * kSortKeys + key];
        hist[(uint64_t)g * kSortKeys + key] = run;
        run += v;
    }
    if (part == 0) tot[key] = all;
}

template <bool STABLE>
__global__ __launch_bounds__(kSortBlock) void sort_scatter(const uint32_t* __restrict__ seg,
                                                           const uint32_t* __restrict__ seg_n,
                                                           uint64_t n_ranges, int log2_range,
                                                           int log2_group,
                                                           const uint32_t* __restrict__ pre,
                                                           const uint32_t* __restrict__ tot,
                                                           uint32_t* __restrict__ surv,
                                                           unsigned int* __restrict__ count,
                                                           uint32_t* __restrict__ sect) {
    __shared__ uint32_t s_at[kSortWaves][kSortKeys];   // per wavefront: count, then next place
    __shared__ uint32_t s_wsum[kSortWaves];
    static_assert(kSortKeys == 2 * kSortBlock, "two keys per thread");
    const int wave = threadIdx.x >> 6, lane = threadIdx.x & 63;
    for (int w = 0; w < kSortWaves; ++w)
        for (int k = threadIdx.x; k < kSortKeys; k += kSortBlock) s_at[w][k] = 0;
    // where each key's photons start: a scan of the totals, two keys per thread
    const uint32_t t0 = tot[2 * threadIdx.x], t1 = tot[2 * threadIdx.x + 1];
    uint32_t v = t0 + t1;
#pragma unroll
    for (int d = 1; d < 64; d <<= 1) {
        const uint32_t o = __shfl_up(v, d);
        if (lane >= d) v += o;
    }
    if (lane == 63) s_wsum[wave] = v;
    __syncthreads();
    for_each_listed(seg, seg_n, n_ranges, log2_range, log2_group,
                    [&](uint32_t e, uint64_t) { atomicAdd(&s_at[wave][e >> 12], 1u); });
    uint32_t start = v - (t0 + t1);
    for (int w = 0; w < wave; ++w) start += s_wsum[w];
    if (blockIdx.x == 0) {
        const int k = 2 * threadIdx.x;
        if ((k & (kSortKeys / kSectors - 1)) == 0) sect[k / (kSortKeys / kSectors)] = start;
        if (threadIdx.x == kSortBlock - 1) {
            sect[kSectors] = start + t0 + t1;
            *count = start + t0 + t1;
        }
    }
    __syncthreads();
    const uint32_t* p = pre + (uint64_t)blockIdx.x * kSortKeys + 2 * threadIdx.x;
    uint32_t at[2] = {start + p[0], start + t0 + p[1]};
#pragma unroll
    for (int j = 0; j < 2; ++j)
        for (int w = 0; w < kSortWaves; ++w) {
            const uint32_t n = s_at[w][2 * threadIdx.x + j];
            s_at[w][2 * threadIdx.x + j] = at[j];
            at[j] += n;
        }
    __syncthreads();
    for_each_listed(seg, seg_n, n_ranges, log2_range, log2_group, [&](uint32_t e, uint64_t rg) {
        uint32_t at = 0;
        if constexpr (STABLE) {
            const uint64_t m = same_key(e >> 12);
            const int first = __ffsll((unsigned long long)m) - 1;
            if (first == lane) at = atomicAdd(&s_at[wave][e >> 12], (uint32_t)__popcll(m));
            at = __shfl(at, first) + (uint32_t)__popcll(m & ((1ull << lane) - 1ull));
        } else {
            at = atomicAdd(&s_at[wave][e >> 12], 1u);
        }
        surv[at] = (uint32_t)(rg << log2_range) + (e & 0xfffu);
    });
}

// Block-uniform work distribution over [0, n): static (tile = block, block + grid, ...), static within
// this die's pupil sector (sect: the sectors' starts; workgroup b runs on die b mod 8), or dynamic
// (tiles of kTileIters x blockDim elements claimed from a device counter).
struct Tiles {
    unsigned long long* ctr;   // null: static
    uint64_t tile, sub, n, base, step;
    __device__ Tiles(unsigned long long* c, const uint32_t* sect, uint64_t total)
        : ctr(c), tile(blockIdx.x), sub(0), n(total), base(0), step(gridDim.x) {
        if (sect) {
            const uint32_t s = blockIdx.x % kSectors;
            tile = blockIdx.x / kSectors;
            step = gridDim.x / kSectors;
            base = sect[s];
            n = sect[s + 1] - base;
        }
    }
    __device__ bool next(unsigned long long* s_tile) {
        if (!ctr) {
            if (sub) tile += step;
            sub = 1;
            return tile * blockDim.x < n;
        }
        if (sub == 0 || sub == kTileIters) {
            __syncthreads();
            if (threadIdx.x == 0) *s_tile = atomicAdd(ctr, 1ull);
            __syncthreads();
            tile = *s_tile * kTileIters;
            sub = 0;
        } else {
            tile += 1;
        }
        sub += 1;
        return tile * blockDim.x < n;
    }
    __device__ uint64_t last() const { return base + n - 1; }
    // this lane's element; false where the last tile is short
    __device__ bool element(uint64_t& r) const {
        const uint64_t k = tile * blockDim.x + threadIdx.x;
        r = base + k;
        return k < n;
    }
};

// Front half of the trace for the chunk's photons (the list, or every photon when surv is null): sky
// sampling and the atmosphere, leaving the start-plane state in SoA arrays
// st[0..5][i] = p_x, p_y, n_x, n_y, n_z, lambda (p_z is the start plane's height).
template <bool SERSIC, bool EXTRA>
__global__ __launch_bounds__(kBlock) void front_kernel(const DevParams* __restrict__ Pg,
                                                       const Launch L, uint64_t begin,
                                                       const uint32_t* __restrict__ surv,
                                                       const unsigned int* __restrict__ count,
                                                       uint64_t n_all, double* __restrict__ st,
                                                       uint64_t st_stride,
                                                       unsigned long long* tile_ctr,
                                                       const uint32_t* __restrict__ sect) {
    __shared__ unsigned long long s_tile;
    const DevParams& P = *Pg;
    Tiles T(tile_ctr, sect, surv ? (uint64_t)*count : n_all);
    while (T.next(&s_tile)) {
        uint64_t r;
        // every lane takes part in the screen lookups: past the end of a tile it repeats the last photon
        const bool valid = T.element(r);
        if (!valid) r = T.last();
        const uint64_t g = begin + (surv ? (uint64_t)surv[r] : r);
        int si;
        uint64_t idx;
        decode(L, g, si, idx);
        Front f;
        photon_front<SERSIC, EXTRA>(P, L, si, idx, f);
        if (!valid) continue;
        st[0 * st_stride + r] = f.p[0];
        st[1 * st_stride + r] = f.p[1];
        st[2 * st_stride + r] = f.n[0];
        st[3 * st_stride + r] = f.n[1];
        st[4 * st_stride + r] = f.n[2];
        st[5 * st_stride + r] = f.lam;
    }
}

// Book-keeping of finished photons, one per lane where act (every lane of the wavefront calls
// it): the event record, the pixel (through the workgroup's LDS window of win x win pixels placed
// at the first detection, else a wavefront-aggregated global atomic), the status count and the
// moment words.
__device__ __forceinline__ void book(const DevParams& P, const Launch& L, bool act, uint64_t g,
                                     int si, uint64_t idx, const Outcome& o, uint32_t* s_stats,
                                     uint32_t* s_win, int win, int* s_org, MomentCache* s_mc) {
    int pix = -1, slot = 0;
    bool m_on = false;
    if (act) {
        m_on = (L.flags & PHX_F_MOMENTS) && o.status <= PHX_OFF_CHIP;
        slot = stat_slot(o);
        if (account(P, L, g, si, idx, o) >= 0) {
            int org = *s_org;
            if (org < 0) {
                const int want = (max(o.pix_i - win / 2, 0) << 16) | max(o.pix_j - win / 2, 0);
                const int prev = atomicCAS(s_org, -1, want);
                org = prev < 0 ? want : prev;
            }
            const int wi = o.pix_i - (org >> 16), wj = o.pix_j - (org & 0xffff);
            if (wi >= 0 && wi < win && wj >= 0 && wj < win)
                atomicAdd(&s_win[wj * win + wi], 1u);
            else
                pix = o.pix_j * P.nx + o.pix_i;
        }
    }
    bin_photon(L.image, pix, pix >= 0);
    count_stat(s_stats, slot, act);
    if (L.flags & PHX_F_MOMENTS) add_moments(L, si, o.xe, o.ye, m_on, s_mc);
}

// Back half, the optics stage with refill (sections 2.4.1-2.4.3), from the start-plane state:
// each wavefront takes 64 photons at a time
// through the central obscuration and the first surface, queues the survivors in LDS, and runs
// the rest of the optics, the silicon and the pixel on 64 queued photons at a time, so lanes
// whose photon was vignetted or absorbed at the first surface are refilled instead of idling
// through the remaining surfaces.  Work units of 64 photons: static (unit w of the grid's
// wavefronts, then every grid-size-th unit) or from a device counter.
constexpr int kWin = 32;                  // LDS pixel window of the optics kernel
constexpr int kWaves = kBlock / 64;
// EXTRA: aerosol and the spider at the entrance.  GH, the ghost branch of the roulette (with
// ghosts the kernel runs twice per chunk): 0 none; 1 the sequential pass, which appends the
// photons a coating reflects to the chunk's ghost list (ghost_list, cap entries, ghost_ctr[0]
// their number) instead of booking them; 2 the branches of the listed photons, taken
// kGhostClaim at a time (ghost_ctr[1] counts the claimed ones), with every lane refilled from them as its photon is
// settled.  Keeping the branches out of the sequential pass keeps its registers those of the
// kernel without ghosts.
// Four wavefronts per SIMD (128 VGPRs; without the compiler's hoisting of constants out of the loop the
// kernel needs 119, with it 168 and spills): 8.6e6 photons 1.36 -> 1.04 ms with the compute units
// full.
template <bool ZERN, bool EXTRA, int GH>
__global__ __launch_bounds__(kBlock) __attribute__((amdgpu_waves_per_eu(4, 8))) void back_kernel(
        const DevParams* __restrict__ Pg, const Launch L, uint64_t begin,
        const uint32_t* __restrict__ surv, const unsigned int* __restrict__ count, uint64_t n_all,
        const double* __restrict__ st, uint64_t st_stride, unsigned long long* unit_ctr,
        double* __restrict__ ghost_list, uint64_t ghost_cap, unsigned long long* ghost_ctr) {
    constexpr bool GHOST = GH == 1;
    __shared__ uint32_t s_stats[PHX_STATS_LEN];
    __shared__ uint32_t s_win[kWin * kWin];
    __shared__ int s_org;   // window origin: (i0 << 16) | j0, or -1 before the first detection
    __shared__ MomentCache s_mc;
    __shared__ double s_q[kWaves][7][kQueue];   // p, n (global frame) and wavelength
    __shared__ uint32_t s_qr[kWaves][kQueue];   // position in the survivor list
    __shared__ int32_t s_qk[kWaves][kQueue];    // Newton steps so far
    // GH == 1: each wavefront's staging area of ghost starts (kGhostStage fields x 64 lanes; the
    // other fields go to the queue: to the lane's own entry, once read, in the second pass, to the upper
    // half, free then, in the first)
    __shared__ double s_gs[GH == 1 ? kWaves * kGhostStage * 64 : 1];
    for (int i = threadIdx.x; i < kWin * kWin; i += blockDim.x) s_win[i] = 0;
    if (threadIdx.x == 0) s_org = -1;
    moment_cache_init(&s_mc);
    stats_init(s_stats);   // ends with a barrier
    const DevParams& P = *Pg;
    const uint64_t n = surv ? (uint64_t)*count : n_all;
    const int wave = threadIdx.x >> 6, lane = __lane_id();
    double (*q)[kQueue] = s_q[wave];
    uint32_t* qr = s_qr[wave];
    int32_t* qk = s_qk[wave];
    const uint64_t n_units = (n + 63) / 64;
    const uint64_t n_waves = (uint64_t)gridDim.x * kWaves;
    uint64_t unit = (uint64_t)blockIdx.x * kWaves + wave;
    if (unit_ctr) {
        unsigned long long u = 0;
        if (lane == 0) u = atomicAdd(unit_ctr, 1ull);
        unit = __shfl(u, 0);
    }
    const int kdet = P.n_surf - 1;
    const int k_first = kdet < 1 ? kdet : 1;   // surfaces of the first pass: [0, k_first)
    int qn = 0;                                // queued photons (wavefront-uniform)
    uint32_t newton = 0, traced = 0;
    if (GH == 2) {
        // the branches: the wavefront takes kGhostClaim listed starts at a time; a lane whose photon is
        // settled takes the next claimed start, so that the lanes stay busy until the list is
        // exhausted
        const uint64_t total = min((uint64_t)ghost_ctr[0], ghost_cap);
        uint64_t wbase = 0, wend = 0;   // the wavefront's claimed, not yet started entries
        // a list of a few claims per wavefront is dealt out in turn
        const bool dealt = total <= kGhostDealt * n_waves * kGhostClaim;
        uint64_t next = ((uint64_t)blockIdx.x * kWaves + wave) * kGhostClaim;
        bool claims = true;
        bool busy = false;
        GhostRay gr;
        Outcome o;
        outcome_init(o, 0.0);
        Optics oc{0.0, 1.0, 1.0, LamCol{0, 0.0}};
        Rng rng{0u, 0u, 0u, 0u};
        uint64_t g = 0, idx = 0;
        int si = 0;
        for (;;) {
            const uint64_t idle = __ballot(!busy);
            if (claims && idle && wbase == wend) {
                unsigned long long b = next;
                if (dealt) {
                    next += n_waves * kGhostClaim;
                } else {
                    if (lane == 0) b = atomicAdd(&ghost_ctr[1], (unsigned long long)kGhostClaim);
                    b = __shfl(b, 0);
                }
                wbase = b < total ? b : total;
                wend = b + kGhostClaim < total ? b + kGhostClaim : total;
                claims = wbase < wend;
            }
            const uint64_t avail = wend - wbase;
            const int take = (int)min((uint64_t)__popcll(idle), avail);
            const int rank = __popcll(idle & ((1ull << lane) - 1ull));
            if (!busy && rank < take) {
                GhostStart gs;
                double lam;
                uint32_t r;
                int nw;
                ghost_get(ghost_list, ghost_cap, wbase + rank, gs, lam, r, nw);
                if (gs.k >= 0) {   // not an unused entry
                    g = begin + (surv ? (uint64_t)surv[r] : (uint64_t)r);
                    decode(L, g, si, idx);
                    rng = Rng{L.seed, (uint32_t)si, (uint32_t)idx, (uint32_t)(idx >> 32)};
                    outcome_init(o, lam);
                    o.newton = nw;
                    oc = optics_of(P, L, lam);
                    ghost_begin(P, gs.h, gs.k, gs.n_cur, gr);
                    busy = true;
                }
            }
            wbase += take;
            if (__ballot(busy) == 0) {   // nothing left, or only unused entries taken
                if (wbase == wend && !claims) break;
                continue;
            }
            bool fin = false;
            if (busy) fin = ghost_step<ZERN>(P, L, rng, oc, gr, o);
            if (fin) {
                newton += o.newton;
                busy = false;
            }
            book(P, L, fin, g, si, idx, o, s_stats, s_win, kWin, &s_org, &s_mc);
        }
    }
    GhostRoom room{0, 0, n_units >= kGhostUnits * n_waves ? kGhostReserve : 0};
    for (;;) {
        if (GH == 2) break;
        const bool more = unit < n_units;
        if (qn >= 64 || (!more && qn > 0)) {
            // second pass: up to 64 queued photons through the remaining surfaces
            const int take = qn < 64 ? qn : 64;
            const bool act = lane < take;
            Outcome o;
            outcome_init(o, 0.0);
            uint64_t g = 0, idx = 0;
            int si = 0;
            uint32_t r = 0;
            GhostSink gs{&q[0][max(qn - take + lane, 0)],
                         s_gs + (GH == 1 ? wave * kGhostStage * 64 + lane : 0), -1};
            if (act) {
                const int e = qn - take + lane;
                r = qr[e];
                g = begin + (surv ? (uint64_t)surv[r] : (uint64_t)r);
                decode(L, g, si, idx);
                const Rng rng{L.seed, (uint32_t)si, (uint32_t)idx, (uint32_t)(idx >> 32)};
                const double lam = q[6][e];
                outcome_init(o, lam);
                o.newton = qk[e];
                const Optics oc = optics_of(P, L, lam);
                Ray ray{{q[0][e], q[1][e], q[2][e]}, {q[3][e], q[4][e], q[5][e]}};
                uint4 wc = make_uint4(0, 0, 0, 0);
                int wc_block = -1;
                GhostSink* gp = GHOST ? &gs : nullptr;
                if (trace_surfaces<ZERN, false, GHOST>(P, L, rng, oc, ray, k_first, kdet, wc,
                                                       wc_block, o, nullptr, 0, gp))
                    finish_detector<ZERN, false, GHOST>(P, L, rng, oc, ray, wc, wc_block, o,
                                                        nullptr, 0, gp);
            }
            const bool fin = act && !(GHOST && gs.k >= 0);
            if (GHOST) ghost_append(ghost_list, ghost_cap, ghost_ctr, room, gs, o, r);
            if (fin) newton += o.newton;
            book(P, L, fin, g, si, idx, o, s_stats, s_win, kWin, &s_org, &s_mc);
            qn -= take;
            __builtin_amdgcn_wave_barrier();
            continue;
        }
        if (!more) break;
        // first pass: the next 64 photons through the central obscuration and the first surface
        const uint64_t r = unit * 64 + lane;
        const bool valid = r < n;
        bool alive = false;
        Outcome o;
        outcome_init(o, 0.0);
        uint64_t g = 0, idx = 0;
        int si = 0;
        Ray ray{{0.0, 0.0, 0.0}, {0.0, 0.0, 1.0}};
        GhostSink gs{&q[0][64 + lane], s_gs + (GH == 1 ? wave * kGhostStage * 64 + lane : 0), -1};
        if (valid) {
            g = begin + (surv ? (uint64_t)surv[r] : r);
            decode(L, g, si, idx);
            const double lam = st[5 * st_stride + r];
            outcome_init(o, lam);
            ray.p[0] = st[0 * st_stride + r];
            ray.p[1] = st[1 * st_stride + r];
            ray.p[2] = P.z_start;
            ray.n[0] = st[2 * st_stride + r];
            ray.n[1] = st[3 * st_stride + r];
            ray.n[2] = st[4 * st_stride + r];
            const Rng rng{L.seed, (uint32_t)si, (uint32_t)idx, (uint32_t)(idx >> 32)};
            if (entrance<EXTRA>(P, L, rng, ray, o)) {
                const Optics oc = optics_of(P, L, lam, !(P.surf[0].bits & kSurfMirror));
                uint4 wc = make_uint4(0, 0, 0, 0);
                int wc_block = -1;
                alive = trace_surfaces<ZERN, false, GHOST>(P, L, rng, oc, ray, 0, k_first, wc,
                                                           wc_block, o, nullptr, 0,
                                                           GHOST ? &gs : nullptr);
            }
            traced += 1;
        }
        if (GHOST) {
            ghost_append(ghost_list, ghost_cap, ghost_ctr, room, gs, o, (uint32_t)r);
            __builtin_amdgcn_wave_barrier();   // before the queue's upper half is written again
        }
        const uint64_t am = __ballot(alive);
        if (alive) {
            const int e = qn + __popcll(am & ((1ull << lane) - 1ull));
            q[0][e] = ray.p[0]; q[1][e] = ray.p[1]; q[2][e] = ray.p[2];
            q[3][e] = ray.n[0]; q[4][e] = ray.n[1]; q[5][e] = ray.n[2];
            q[6][e] = o.lam;
            qr[e] = (uint32_t)r;
            qk[e] = o.newton;
        }
        qn += __popcll(am);
        const bool done = valid && !alive && !(GHOST && gs.k >= 0);
        if (done) newton += o.newton;
        book(P, L, done, g, si, idx, o, s_stats, s_win, kWin, &s_org, &s_mc);
        if (unit_ctr) {
            unsigned long long u = 0;
            if (lane == 0) u = atomicAdd(unit_ctr, 1ull);
            unit = __shfl(u, 0);
        } else {
            unit += n_waves;
        }
        __builtin_amdgcn_wave_barrier();
    }
    if (GHOST) ghost_close(ghost_list, ghost_cap, room);
    stats_flush(L, s_stats, newton, traced);   // ends with a barrier
    if (threadIdx.x == 0 && (L.flags & PHX_F_MOMENTS)) moment_cache_flush(L, &s_mc);
    const int org = s_org;
    if (org >= 0) {
        const int i0 = org >> 16, j0 = org & 0xffff;
        for (int k = threadIdx.x; k < kWin * kWin; k += blockDim.x) {
            const uint32_t c = s_win[k];
            const int i = i0 + (k % kWin), j = j0 + (k / kWin);
            if (c && i < P.nx && j < P.ny) atomicAdd(&L.image[(size_t)j * P.nx + i], c);
        }
    }
}

// ---------------------------------------------------------------------------------------------
// Adjoint trace: pathwise derivative of per-source moments with respect to the rigid-body
// parameters of the two perturbation groups and the Zernike amplitudes of the primary, with
// every discrete decision (pupil, coatings, apertures, conversion, escape) held at its forward
// value.  Each converted photon is traced again with a tape of its surface passages, then swept
// from the electron position back to the primary: the intersection by the implicit-function
// rule (the path length solves q_z + l d_z = S(q_x + l d_x, q_y + l d_y)), the normal through
// the sag Hessian, reflection and Snell refraction through their Jacobians, and each group
// transform g = R q + t with t = pivot + R (vertex - pivot) + shift.

// Monomials u^a v^b of the Zernike expansion (order of zernike_poly).
__device__ constexpr int kMonoA[kNZernPoly] = {0, 1, 0, 2, 1, 0, 3, 2, 1, 0, 4, 3, 2, 1, 0};
__device__ constexpr int kMonoB[kNZernPoly] = {0, 0, 1, 0, 1, 2, 0, 1, 2, 3, 0, 1, 2, 3, 4};

__device__ __forceinline__ double ipow(const double* pw, int e) { return e > 0 ? pw[e] : 1.0; }

// Sag slopes and Hessian in the element frame at (x, y).
template <bool ZERN>
__device__ __forceinline__ void sag_hessian(const DevParams& P, const DevSurface& s, int k,
                                            double x, double y, double& Sx, double& Sy,
                                            double& Hxx, double& Hxy, double& Hyy) {
    const double r2 = x * x + y * y;
    const double arg = fmax(1.0 - s.kc2 * r2, 0.0);
    const double root = sqrt(arg);
    const double iroot = root > 0.0 ? 1.0 / root : 0.0;
    double g = s.c * iroot;                                       // dS/dr / r
    double gp = 0.5 * s.c * s.kappa1 * s.c * s.c * iroot * iroot * iroot;   // dg / d(r^2)
    if (s.bits & kSurfEven) {
        const double* a = s.alpha;
        g += r2 * (4.0 * a[1] + r2 * (6.0 * a[3] + r2 * (8.0 * a[5] + r2 * 10.0 * a[7])));
        gp += 4.0 * a[1] + r2 * (12.0 * a[3] + r2 * (24.0 * a[5] + r2 * 40.0 * a[7]));
    } else if (s.bits & kSurfGeneral) {
        const double r = sqrt(r2);
        const double ir = r > 0.0 ? 1.0 / r : 0.0;
        double pw = r;   // r^(i-2)
        for (int i = 3; i <= 10; ++i) {
            const double a = s.alpha[i - 3];
            g += (double)i * a * pw;
            gp += 0.5 * (double)(i * (i - 2)) * a * pw * ir * ir;   // i (i-2) a r^(i-4) / 2
            pw *= r;
        }
    }
    Sx = x * g;
    Sy = y * g;
    Hxx = g + 2.0 * x * x * gp;
    Hxy = 2.0 * x * y * gp;
    Hyy = g + 2.0 * y * y * gp;
    if (ZERN && k == 0 && (s.bits & kSurfZernike)) {
        const double ir = P.zern_inv_r;
        const double u = x * ir, v = y * ir;
        double pu[5], pv[5];
        pu[0] = pv[0] = 1.0;
        for (int e = 1; e < 5; ++e) { pu[e] = pu[e - 1] * u; pv[e] = pv[e - 1] * v; }
        double zu = 0, zv = 0, zuu = 0, zuv = 0, zvv = 0;
#pragma unroll
        for (int m = 0; m < kNZernPoly; ++m) {
            const int a = kMonoA[m], b = kMonoB[m];
            const double c = P.zern[m];
            if (a >= 1) zu += c * a * ipow(pu, a - 1) * pv[b];
            if (b >= 1) zv += c * b * pu[a] * ipow(pv, b - 1);
            if (a >= 2) zuu += c * a * (a - 1) * ipow(pu, a - 2) * pv[b];
            if (a >= 1 && b >= 1) zuv += c * a * b * ipow(pu, a - 1) * ipow(pv, b - 1);
            if (b >= 2) zvv += c * b * (b - 1) * pu[a] * ipow(pv, b - 2);
        }
        Sx += zu * ir;
        Sy += zv * ir;
        Hxx += zuu * ir * ir;
        Hxy += zuv * ir * ir;
        Hyy += zvv * ir * ir;
    }
}

__device__ __forceinline__ void group_rotation_derivs(const DevParams& P, int g, double dRx[9],
                                                      double dRy[9]) {
    const double cx = P.group_cs[g][0], sx = P.group_cs[g][1];
    const double cy = P.group_cs[g][2], sy = P.group_cs[g][3];
    // R = R_x(t_x) R_y(t_y) = [[cy, 0, sy], [sx sy, cx, -sx cy], [-cx sy, sx, cx cy]]
    dRx[0] = 0.0;      dRx[1] = 0.0; dRx[2] = 0.0;
    dRx[3] = cx * sy;  dRx[4] = -sx; dRx[5] = -cx * cy;
    dRx[6] = sx * sy;  dRx[7] = cx;  dRx[8] = -sx * cy;
    dRy[0] = -sy;      dRy[1] = 0.0; dRy[2] = cy;
    dRy[3] = sx * cy;  dRy[4] = 0.0; dRy[5] = sx * sy;
    dRy[6] = -cx * cy; dRy[7] = 0.0; dRy[8] = -cx * sy;
}

// The sweep for NC cotangent columns at once: seeds (xb, yb) of the electron position, results
// added to acc[c][0..kAdj).
template <bool ZERN, int NC>
__device__ void adjoint_sweep(const DevParams& P, const Launch& L, const Rng& rng, double lam,
                              const double* tp, uint64_t ts, const double* xb, const double* yb,
                              double (*acc)[kAdj]) {
    const int kdet = P.n_surf - 1;
    const double n_glass = P.has_glass ? sellmeier(P, lam) : 1.0;
    double pb[NC][3], nb[NC][3];   // global-frame cotangents of the ray leaving surface k
#pragma unroll 1
    for (int k = kdet; k >= 0; --k) {
        const DevSurface& s = P.surf[k];
        const double* t = tp + (uint64_t)k * kTapeFields * ts;
        const double q1[3] = {t[0], t[ts], t[2 * ts]};
        const double d0[3] = {t[3 * ts], t[4 * ts], t[5 * ts]};
        const double l = t[6 * ts];
        double Sx, Sy, Hxx, Hxy, Hyy;
        sag_hessian<ZERN>(P, s, k, q1[0], q1[1], Sx, Sy, Hxx, Hxy, Hyy);
        const double inv = 1.0 / sqrt(Sx * Sx + Sy * Sy + 1.0);
        const double Nr[3] = {-Sx * inv, -Sy * inv, inv};
        const double dnr = d0[0] * Nr[0] + d0[1] * Nr[1] + d0[2] * Nr[2];
        const double sg = dnr > 0.0 ? -1.0 : 1.0;
        const double N[3] = {sg * Nr[0], sg * Nr[1], sg * Nr[2]};
        const double dn = sg * dnr;
        const double n_in = (s.bits & kSurfGlassIn) ? n_glass : 1.0;
        // 0: no outgoing direction, 1: reflection, 2: refraction
        int mode;
        double mu = 1.0;
        if (k == kdet) {
            mode = (L.flags & PHX_F_SILICON) ? 2 : 0;
            mu = n_in / n_silicon(lam);
        } else if (s.kind == PHX_MIRROR) {
            mode = 1;
        } else {
            mode = 2;
            mu = n_in / (s.medium == PHX_GLASS ? n_glass : 1.0);
        }
        double d1[3] = {d0[0], d0[1], d0[2]};
        double f = 0.0, fpr = 0.0;
        if (mode == 1) {
#pragma unroll
            for (int i = 0; i < 3; ++i) d1[i] = d0[i] - 2.0 * dn * N[i];
        } else if (mode == 2) {
            const double cosi = -dn;
            const double kk = 1.0 - mu * mu * (1.0 - cosi * cosi);
            const double w = sqrt(fmax(kk, 0.0));
            f = mu * cosi - w;
            fpr = mu - (w > 0.0 ? mu * mu * cosi / w : 0.0);
#pragma unroll
            for (int i = 0; i < 3; ++i) d1[i] = mu * d0[i] + f * N[i];
        }
        double qb[NC][3], db[NC][3];
        double Rb[NC][9], tb[NC][3];
        const bool grp = s.group != 0;
#pragma unroll
        for (int c = 0; c < NC; ++c) {
#pragma unroll
            for (int i = 0; i < 9; ++i) Rb[c][i] = 0.0;
            tb[c][0] = tb[c][1] = tb[c][2] = 0.0;
        }
        if (k == kdet) {
            // electron position from the landing point (sections 2.4.2-2.4.3)
            double Lc = 0.0, kz = 0.0, ca = 0.0, sa = 0.0;
            if (L.flags & PHX_F_SILICON) {
                Lc = -log(u01(rng.block(1).z)) / absorption(P, lam);
                if (L.flags & PHX_F_DIFFUSION) {
                    const uint4 wd = rng.block(6);
                    const double rad = sqrt(-2.0 * log(u01(wd.x)));
                    sincospi(2.0 * u01(wd.y), &sa, &ca);
                    ca *= rad;
                    sa *= rad;
                    // d sigma / d d1z through the depth Lc |d1z|
                    double slope = -P.sigma_max / P.t_si;
                    if (L.flags & PHX_F_FIELD_DIFFUSION) field_sigma(P, Lc * fabs(d1[2]), slope);
                    kz = slope * Lc * (d1[2] >= 0.0 ? 1.0 : -1.0);
                }
            }
#pragma unroll
            for (int c = 0; c < NC; ++c) {
                qb[c][0] = xb[c]; qb[c][1] = yb[c]; qb[c][2] = 0.0;
                db[c][0] = Lc * xb[c]; db[c][1] = Lc * yb[c];
                db[c][2] = kz * (ca * xb[c] + sa * yb[c]);
            }
        } else {
            // leaving surface k: p' = R q1 + t, n' = R d1
#pragma unroll
            for (int c = 0; c < NC; ++c) {
#pragma unroll
                for (int j = 0; j < 3; ++j) {
                    qb[c][j] = s.R[j] * pb[c][0] + s.R[3 + j] * pb[c][1] + s.R[6 + j] * pb[c][2];
                    db[c][j] = s.R[j] * nb[c][0] + s.R[3 + j] * nb[c][1] + s.R[6 + j] * nb[c][2];
                }
                if (grp) {
#pragma unroll
                    for (int i = 0; i < 3; ++i) {
#pragma unroll
                        for (int j = 0; j < 3; ++j)
                            Rb[c][3 * i + j] += pb[c][i] * q1[j] + nb[c][i] * d1[j];
                        tb[c][i] += pb[c][i];
                    }
                }
            }
        }
        const double mv[3] = {-Sx, -Sy, 1.0};
        const double fpn = d0[2] - Sx * d0[0] - Sy * d0[1];
        double mono[kNZernPoly], mu_[kNZernPoly], mv_[kNZernPoly];
        if (k == 0) {
            const double ir = P.zern_inv_r;
            const double u = q1[0] * ir, v = q1[1] * ir;
            double pu[5], pv[5];
            pu[0] = pv[0] = 1.0;
            for (int e = 1; e < 5; ++e) { pu[e] = pu[e - 1] * u; pv[e] = pv[e - 1] * v; }
#pragma unroll
            for (int m = 0; m < kNZernPoly; ++m) {
                const int a = kMonoA[m], b = kMonoB[m];
                mono[m] = pu[a] * pv[b];
                mu_[m] = a >= 1 ? a * ipow(pu, a - 1) * pv[b] * ir : 0.0;
                mv_[m] = b >= 1 ? b * pu[a] * ipow(pv, b - 1) * ir : 0.0;
            }
        }
#pragma unroll
        for (int c = 0; c < NC; ++c) {
            // reflection / refraction: cotangents of the incoming direction and of the normal
            double d0b[3] = {0.0, 0.0, 0.0}, Nb[3] = {0.0, 0.0, 0.0};
            const double tN = N[0] * db[c][0] + N[1] * db[c][1] + N[2] * db[c][2];
            if (mode == 1) {
#pragma unroll
                for (int i = 0; i < 3; ++i) {
                    d0b[i] = db[c][i] - 2.0 * tN * N[i];
                    Nb[i] = -2.0 * (dn * db[c][i] + tN * d0[i]);
                }
            } else if (mode == 2) {
#pragma unroll
                for (int i = 0; i < 3; ++i) {
                    d0b[i] = mu * db[c][i] - tN * fpr * N[i];
                    Nb[i] = f * db[c][i] - tN * fpr * d0[i];
                }
            }
            // N = sg (-Sx, -Sy, 1) / sqrt(Sx^2 + Sy^2 + 1)
            const double nn = sg * (Nb[0] * Nr[0] + Nb[1] * Nr[1] + Nb[2] * Nr[2]);
            const double Sxb = -sg * Nb[0] * inv - nn * Sx * inv * inv;
            const double Syb = -sg * Nb[1] * inv - nn * Sy * inv * inv;
            double qc[3] = {qb[c][0] + Sxb * Hxx + Syb * Hxy, qb[c][1] + Sxb * Hxy + Syb * Hyy,
                            qb[c][2]};
            // intersection: q1 = q0 + l d0 with F(l) = q1_z - S(q1_x, q1_y) = 0
            const double lb = qc[0] * d0[0] + qc[1] * d0[1] + qc[2] * d0[2];
            const double coef = -lb / fpn;
            double q0b[3];
#pragma unroll
            for (int i = 0; i < 3; ++i) {
                q0b[i] = qc[i] + coef * mv[i];
                d0b[i] += l * qc[i] + coef * l * mv[i];
            }
            if (k == 0) {
#pragma unroll
                for (int m = 0; m < kNZernPoly; ++m)
                    acc[c][10 + m] += Sxb * mu_[m] + Syb * mv_[m] - coef * mono[m];
            }
            // entering surface k: q0 = R^T (p - t), d0 = R^T n
#pragma unroll
            for (int i = 0; i < 3; ++i) {
                pb[c][i] = s.R[3 * i] * q0b[0] + s.R[3 * i + 1] * q0b[1] + s.R[3 * i + 2] * q0b[2];
                nb[c][i] = s.R[3 * i] * d0b[0] + s.R[3 * i + 1] * d0b[1] + s.R[3 * i + 2] * d0b[2];
            }
            if (grp) {
                const double q0[3] = {q1[0] - l * d0[0], q1[1] - l * d0[1], q1[2] - l * d0[2]};
                double pt[3], nw[3];   // p - t = R q0 and n = R d0 (global frame)
#pragma unroll
                for (int i = 0; i < 3; ++i) {
                    pt[i] = s.R[3 * i] * q0[0] + s.R[3 * i + 1] * q0[1] + s.R[3 * i + 2] * q0[2];
                    nw[i] = s.R[3 * i] * d0[0] + s.R[3 * i + 1] * d0[1] + s.R[3 * i + 2] * d0[2];
                }
#pragma unroll
                for (int i = 0; i < 3; ++i) {
#pragma unroll
                    for (int j = 0; j < 3; ++j) Rb[c][3 * i + j] += pt[i] * q0b[j] + nw[i] * d0b[j];
                    tb[c][i] -= pb[c][i];
                }
                // t = pivot + R (vertex - pivot) + shift
                const double* Pv = P.group_pivot[s.group];
                const double vp[3] = {-Pv[0], -Pv[1], s.z_vertex - Pv[2]};
#pragma unroll
                for (int i = 0; i < 3; ++i)
#pragma unroll
                    for (int j = 0; j < 3; ++j) Rb[c][3 * i + j] += tb[c][i] * vp[j];
                double dRx[9], dRy[9];
                group_rotation_derivs(P, s.group, dRx, dRy);
                double gx = 0.0, gy = 0.0;
#pragma unroll
                for (int i = 0; i < 9; ++i) {
                    gx += Rb[c][i] * dRx[i];
                    gy += Rb[c][i] * dRy[i];
                }
                const int b = 5 * (s.group - 1);
                acc[c][b + 0] += tb[c][0];
                acc[c][b + 1] += tb[c][1];
                acc[c][b + 2] += gx;
                acc[c][b + 3] += gy;
                acc[c][b + 4] += tb[c][2];
            }
        }
    }
}

// Wavefront then workgroup sum of the per-lane accumulators in a fixed order; thread 0..kAdj-1
// write the workgroup's row.
__device__ void block_sum_rows(double* acc, double* row) {
    __shared__ double s_part[kBlock / 64][kAdj];
    const int lane = __lane_id(), wave = threadIdx.x / 64;
#pragma unroll
    for (int j = 0; j < kAdj; ++j) {
        double v = acc[j];
#pragma unroll
        for (int m = 32; m >= 1; m >>= 1) v += __shfl_xor(v, m);
        if (lane == 0) s_part[wave][j] = v;
    }
    __syncthreads();
    if (threadIdx.x < kAdj) {
        double v = 0.0;
        for (int w = 0; w < kBlock / 64; ++w) v += s_part[w][threadIdx.x];
        row[threadIdx.x] = v;
    }
}

template <bool ZERN, bool JAC>
__global__ __launch_bounds__(kBlock) void adjoint_kernel(const DevParams* __restrict__ Pg,
                                                         const Launch L, uint64_t begin,
                                                         const uint32_t* __restrict__ surv,
                                                         const unsigned int* __restrict__ count,
                                                         uint64_t n_all,
                                                         const double* __restrict__ st,
                                                         uint64_t st_stride, const Adjoint A,
                                                         uint64_t row0) {
    const DevParams& P = *Pg;
    const uint64_t n = surv ? (uint64_t)*count : n_all;
    const uint64_t tid = (uint64_t)blockIdx.x * blockDim.x + threadIdx.x;
    double* tp = A.tape + tid;
    const uint64_t ts = A.tape_stride;
    double acc[1][kAdj];
#pragma unroll
    for (int j = 0; j < kAdj; ++j) acc[0][j] = 0.0;
    for (uint64_t r = tid; r < n; r += (uint64_t)gridDim.x * blockDim.x) {
        const uint64_t g = begin + (surv ? (uint64_t)surv[r] : r);
        int si;
        uint64_t idx;
        decode(L, g, si, idx);
        Front f;
        f.p[0] = st[0 * st_stride + r];
        f.p[1] = st[1 * st_stride + r];
        f.p[2] = P.z_start;
        f.n[0] = st[2 * st_stride + r];
        f.n[1] = st[3 * st_stride + r];
        f.n[2] = st[4 * st_stride + r];
        f.lam = st[5 * st_stride + r];
        const Outcome o = photon_back<ZERN, true>(P, L, si, idx, f, tp, ts);
        const bool conv = o.status <= PHX_OFF_CHIP;
        const bool sampled = JAC && A.jac && (g % A.jac_stride) == 0;
        if (!conv) {
            if (sampled) {
                double* J = A.jac + (g / A.jac_stride) * 2 * PHX_N_THETA;
                for (int j = 0; j < 2 * PHX_N_THETA; ++j) J[j] = 0.0;
            }
            continue;
        }
        const double* sd = A.seed + (size_t)(si - L.src_begin) * 8;
        const double dx = o.xe - sd[5], dy = o.ye - sd[6];
        const double sxb = sd[0] + sd[2] * dx + sd[4] * dy;
        const double syb = sd[1] + sd[3] * dy + sd[4] * dx;
        const Rng rng{L.seed, (uint32_t)si, (uint32_t)idx, (uint32_t)(idx >> 32)};
        if (!JAC) {
            adjoint_sweep<ZERN, 1>(P, L, rng, o.lam, tp, ts, &sxb, &syb, acc);
        } else {
            double jl[2][kAdj];
#pragma unroll
            for (int c = 0; c < 2; ++c)
#pragma unroll
                for (int j = 0; j < kAdj; ++j) jl[c][j] = 0.0;
            const double xs[2] = {1.0, 0.0}, ys[2] = {0.0, 1.0};
            adjoint_sweep<ZERN, 2>(P, L, rng, o.lam, tp, ts, xs, ys, jl);
#pragma unroll
            for (int j = 0; j < kAdj; ++j) acc[0][j] += sxb * jl[0][j] + syb * jl[1][j];
            if (sampled) {
                double* J = A.jac + (g / A.jac_stride) * 2 * PHX_N_THETA;
                for (int c = 0; c < 2; ++c) {
                    for (int j = 0; j < 10; ++j) J[c * PHX_N_THETA + j] = jl[c][j];
                    for (int z = 0; z < kNZern; ++z) {
                        double v = 0.0;
                        for (int m = 0; m < kNZernPoly; ++m) v += P.zern_basis[z][m] * jl[c][10 + m];
                        J[c * PHX_N_THETA + 10 + z] = v;
                    }
                }
            }
        }
    }
    block_sum_rows(acc[0], A.partial + (row0 + blockIdx.x) * kAdj);
}

// Column sums of the partial rows (fixed order: each thread a strided share, then a tree).
__global__ __launch_bounds__(256) void adjoint_columns(const double* __restrict__ partial,
                                                       uint64_t rows, double* __restrict__ colsum) {
    __shared__ double s[256];
    const int j = blockIdx.x;
    double v = 0.0;
    for (uint64_t r = threadIdx.x; r < rows; r += blockDim.x) v += partial[r * kAdj + j];
    s[threadIdx.x] = v;
    __syncthreads();
    for (int h = 128; h >= 1; h >>= 1) {
        if (threadIdx.x < h) s[threadIdx.x] += s[threadIdx.x + h];
        __syncthreads();
    }
    if (threadIdx.x == 0) colsum[j] = s[0];
}

// Rigid-body columns as they are; monomial columns mapped to the Zernike amplitudes.
__global__ void adjoint_finish(const DevParams* __restrict__ Pg, const double* __restrict__ colsum,
                               double* __restrict__ grad) {
    const int j = threadIdx.x;
    if (j >= PHX_N_THETA) return;
    if (j < 10) {
        grad[j] = colsum[j];
        return;
    }
    double v = 0.0;
    for (int m = 0; m < kNZernPoly; ++m) v += Pg->zern_basis[j - 10][m] * colsum[10 + m];
    grad[j] = v;
}

__global__ void fill_u32(unsigned int* p, uint64_t n, unsigned int v) {
    const uint64_t i = (uint64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i < n) p[i] = v;
}

// Centred-difference gradients of periodic OPD screens (the refractive kick of section 2.3.2 is
// the phase gradient), single precision: g_x = (W[j][i+1] - W[j][i-1]) * (1/(2p)), likewise g_y.
// Thread (plane, j, i) writes the cell record: gradients at (i, j), (i+1, j), (i, j+1), (i+1, j+1).
__device__ __forceinline__ float2 grad_at(const float* w, int n, int i, int j, float f) {
    const int ip = i + 1 == n ? 0 : i + 1, im = i == 0 ? n - 1 : i - 1;
    const int jp = j + 1 == n ? 0 : j + 1, jm = j == 0 ? n - 1 : j - 1;
    const float dx = w[(int64_t)j * n + ip] - w[(int64_t)j * n + im];
    const float dy = w[(int64_t)jp * n + i] - w[(int64_t)jm * n + i];
    return make_float2(dx * f, dy * f);
}

// Also records, per screen, the largest gradient norm of any cell (as float bits: the order of
// non-negative floats is that of their bits), from which the host bounds how far the atmosphere
// can displace a photon at the primary.
__global__ void gradient_kernel(const float* __restrict__ opd, float4* __restrict__ grad, int n,
                                int n_scales, const float* inv2p, int64_t total,
                                unsigned int* __restrict__ gmax) {
    const int64_t id0 = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    const bool live = id0 < total;
    const int64_t id = live ? id0 : total - 1;
    const int64_t nn = (int64_t)n * n;
    const int64_t plane = id / nn;
    const int64_t r = id - plane * nn;
    const int j = (int)(r / n), i = (int)(r - (int64_t)j * n);
    const float* w = opd + plane * nn;
    const float f = inv2p[plane % n_scales];
    const int i1 = i + 1 == n ? 0 : i + 1, j1 = j + 1 == n ? 0 : j + 1;
    const float2 g00 = grad_at(w, n, i, j, f), g10 = grad_at(w, n, i1, j, f);
    const float2 g01 = grad_at(w, n, i, j1, f), g11 = grad_at(w, n, i1, j1, f);
    if (live) {
        grad[2 * id] = make_float4(g00.x, g00.y, g10.x, g10.y);
        grad[2 * id + 1] = make_float4(g01.x, g01.y, g11.x, g11.y);
    }
    if (!gmax) return;
    // a non-finite gradient (from a NaN or infinite optical path) records an infinite maximum
    // (fmaxf would drop a NaN), which the host refuses
    const bool finite = isfinite(g00.x) && isfinite(g00.y);
    float m = live ? (finite ? sqrtf(g00.x * g00.x + g00.y * g00.y) : INFINITY) : 0.0f;
    const int p0 = __shfl((int)plane, 0);
    if (__ballot((int)plane != p0) == 0) {   // the whole wavefront is on one screen
#pragma unroll
        for (int o = 32; o >= 1; o >>= 1) m = fmaxf(m, __shfl_xor(m, o));
        // most wavefronts see a maximum that another has already recorded: the read spares them the
        // atomic (3.4e5 of them on 21 addresses took 13 ms)
        if (__lane_id() == 0 &&
            __float_as_uint(m) > __hip_atomic_load(&gmax[plane], __ATOMIC_RELAXED,
                                                   __HIP_MEMORY_SCOPE_AGENT))
            atomicMax(&gmax[plane], __float_as_uint(m));
    } else if (live) {
        atomicMax(&gmax[plane], __float_as_uint(m));
    }
}

}  // namespace

// Workgroups for n units of work, at most per_cu per compute unit.
static dim3 grid_of(uint64_t n, int n_cu, int per_cu) {
    const uint64_t cap = (uint64_t)n_cu * per_cu;
    return dim3((unsigned)(n < cap ? n : cap));
}

// Pre-roll of one chunk: the survivors with their sort keys in the ranges' segments (seg, seg_n), or
// listed in surv (*count zero before) when the chunk is not sorted.
static void preroll_generate(const DevParams* dparams, const Launch& L, int n_cu,
                             const LaunchConfig& cfg, const ChunkSpan& sp, uint32_t* seg,
                             uint32_t* seg_n, uint32_t* surv, unsigned int* count,
                             hipStream_t stream) {
    const dim3 gg = grid_of(range_count(sp.len), n_cu, cfg.generate_per_cu);
    const bool ghost = (L.flags & PHX_F_GHOSTS) != 0, one = sp.src >= 0;
    const auto gk = one ? (ghost ? generate_kernel<true, true> : generate_kernel<true, false>)
                        : (ghost ? generate_kernel<false, true> : generate_kernel<false, false>);
    hipLaunchKernelGGL(gk, gg, dim3(kBlock), 0, stream, dparams, L, sp.begin, sp.len,
                       one ? L.src_begin + sp.src : 0, one ? sp.first : (uint64_t)0,
                       range_log2(sp.len), seg, seg_n, surv, count);
}

// Every photon of the chunk in the segments (a sorted chunk without the pre-roll).
static void list_photons(const DevParams* dparams, const Launch& L, int n_cu,
                         const LaunchConfig& cfg, const ChunkSpan& sp, uint32_t* seg,
                         uint32_t* seg_n, hipStream_t stream) {
    const dim3 gg = grid_of((sp.len + kBlock - 1) / kBlock, n_cu, cfg.generate_per_cu);
    const bool one = sp.src >= 0;
    hipLaunchKernelGGL(one ? list_kernel<true> : list_kernel<false>, gg, dim3(kBlock), 0, stream,
                       dparams, L, sp.begin, sp.len, one ? L.src_begin + sp.src : 0,
                       one ? sp.first : (uint64_t)0, range_log2(sp.len), seg, seg_n);
}

// Every photon of the chunk listed by class.
static void class_photons(const DevParams* dparams, const Launch& L, int n_cu,
                          const LaunchConfig& cfg, const ChunkSpan& sp, uint32_t* surv,
                          unsigned int* count, unsigned long long* ctr, hipStream_t stream) {
    const dim3 gg = grid_of((sp.len + kClassRange - 1) / kClassRange, n_cu, cfg.generate_per_cu);
    const bool one = sp.src >= 0;
    hipLaunchKernelGGL(one ? class_kernel<true> : class_kernel<false>, gg, dim3(kBlock), 0, stream,
                       dparams, L, sp.begin, sp.len, one ? L.src_begin + sp.src : 0,
                       one ? sp.first : (uint64_t)0, surv, count, ctr);
}

// The segments sorted into surv, their number in W.counts[c], the sectors' starts in W.sect.
static void sort_photons(const Workspace& W, const ChunkSpan& sp, uint64_t c, const uint32_t* seg,
                         const uint32_t* seg_n, uint32_t* surv, bool stable,
                         hipStream_t stream) {
    const uint64_t n_ranges = range_count(sp.len);
    const int lr = range_log2(sp.len);
    const int lg = sort_group_log2(n_ranges);
    const unsigned groups = (unsigned)((n_ranges + (1u << lg) - 1) >> lg);
    uint32_t* tot = W.hist + (uint64_t)groups * kSortKeys;
    hipLaunchKernelGGL(sort_count, dim3(groups), dim3(kSortBlock), 0, stream, seg, seg_n, n_ranges,
                       lr, lg, W.hist);
    hipLaunchKernelGGL(sort_scan, dim3(kSortKeys / 16), dim3(kBlock), 0, stream, W.hist, groups, tot);
    hipLaunchKernelGGL(stable ? sort_scatter<true> : sort_scatter<false>, dim3(groups),
                       dim3(kSortBlock), 0, stream, seg, seg_n, n_ranges, lr, lg,
                       (const uint32_t*)W.hist, (const uint32_t*)tot, surv, W.counts + c,
                       W.sect + 16 * c);
}

// Chunks are pipelined over two streams when the pipe gives a second one: the arithmetic-bound
// pre-roll and optics stage run on pipe.aux, in the order pre-roll(0), pre-roll(1),
// optics(0), pre-roll(2), optics(1), ..., and the sort and the bandwidth-bound
// sky stage on `stream`, so the two kinds of work share the compute units and neither stream
// carries much more than the other.  Segments, lists and states alternate
// between two buffers; events order the hand-offs (segments -> sort and sky -> optics, and
// buffer reuse: a chunk's sort waits for the optics stage two chunks back, and its segments (or, unsorted,
// its list) are rewritten only by the pre-roll issued after the optics stage that follows the sky
// stage that read them), the host issues every event record before the waits on it, and the caller's
// stream waits for the last optics stage before returning work to it.  Without a second stream
// each chunk's stages run in order on `stream`.
namespace {
struct Stages {
    const DevParams* dparams;
    const Launch& L;
    const Workspace& W;
    int n_cu;
    const LaunchConfig& cfg;
    hipStream_t stream;
    const Pipe& pipe;
    const Timing& T;
    const bool stable;   // the order of the lists has an effect (the adjoint's sums)
    // A launch of one chunk has nothing to overlap: its stages stay on the caller's stream (each
    // hand-off between the streams costs 10-12 us; 1e5 photons through the paraboloid 68 us with
    // them, 27 us without).
    bool piped() const { return pipe.aux && pipe.ev && W.n_plan > 1; }
    // events per chunk: 0 pre-roll done, 1 sky done, 2 optics done; then one fork event
    hipEvent_t ev(int kind, uint64_t c) const { return pipe.ev[3 * c + kind]; }
    void mark(int kind, int edge, hipStream_t s) const {
        if (T.on) T.record(T.self, kind, edge, s);
    }
    bool preroll() const { return (L.flags & PHX_F_CULL) && (L.flags & PHX_F_COATINGS); }
    hipStream_t arith() const { return piped() ? pipe.aux : stream; }
    uint64_t half(uint64_t c) const { return piped() ? c % 2 : 0; }
    uint32_t* surv_buf(uint64_t c) const { return W.survivors + half(c) * W.chunk; }
    double* state_buf(uint64_t c) const { return W.state + half(c) * kStateFields * W.chunk; }
    uint32_t* seg_buf(uint64_t c) const { return W.seg + half(c) * W.chunk; }
    uint32_t* seg_n_buf(uint64_t c) const { return W.seg_n + half(c) * max_ranges(W.chunk); }
    bool sorted(uint64_t c) const { return W.plan[c].sort == kListSort; }
    bool classed(uint64_t c) const { return W.plan[c].sort == kListClass; }
    bool listed(uint64_t c) const { return preroll() || sorted(c) || classed(c); }
    unsigned long long* class_ctr(uint64_t c) const {
        return (unsigned long long*)(W.sect + 16 * c);
    }
    const uint32_t* surv(uint64_t c) const { return listed(c) ? surv_buf(c) : nullptr; }
    const unsigned int* cnt(uint64_t c) const { return listed(c) ? W.counts + c : nullptr; }

    // pre-roll of chunk c
    void pre(uint64_t c) const {
        const hipStream_t s = arith();
        if (listed(c)) {
            mark(0, 0, s);
            if (preroll())
                preroll_generate(dparams, L, n_cu, cfg, W.plan[c],
                                 sorted(c) ? seg_buf(c) : nullptr, sorted(c) ? seg_n_buf(c) : nullptr,
                                 sorted(c) ? nullptr : surv_buf(c), W.counts + c, s);
            else if (classed(c))
                class_photons(dparams, L, n_cu, cfg, W.plan[c], surv_buf(c), W.counts + c,
                              class_ctr(c), s);
            else
                list_photons(dparams, L, n_cu, cfg, W.plan[c], seg_buf(c), seg_n_buf(c), s);
            mark(0, 1, s);
        }
        if (piped()) (void)hipEventRecord(ev(0, c), s);
    }
    // sort and sky stage of chunk c on `stream`
    void sky(uint64_t c, unsigned long long* ft) const {
        const ChunkSpan& sp = W.plan[c];
        if (piped()) {
            (void)hipStreamWaitEvent(stream, ev(0, c), 0);
            if (c >= 2) (void)hipStreamWaitEvent(stream, ev(2, c - 2), 0);
        }
        if (sorted(c)) {
            mark(3, 0, stream);
            sort_photons(W, sp, c, seg_buf(c), seg_n_buf(c), surv_buf(c), stable, stream);
            mark(3, 1, stream);
        }
        const dim3 fg = grid_of((sp.len + kBlock - 1) / kBlock, n_cu,
                                stage_groups(cfg, cfg.front_per_cu));
        // The dies take a pupil sector each where the grid covers them evenly (static schedule).  A chunk of
        // more photons than the grid has lanes (1.26e7 by default) always does; below, the grid is
        // ceil(len / 256) workgroups and one length in eight does: 39064 workgroups (1e7 photons) with
        // the pre-roll 537 us and without 2376, 39063 of them 585 and 2546.
        const uint32_t* sect = sorted(c) && (L.flags & PHX_F_ATMOSPHERE) && !ft &&
                                       fg.x % kSectors == 0 ? W.sect + 16 * c : nullptr;
        mark(1, 0, stream);
        const bool extra = (L.flags & kFrontExtra) != 0;
        const auto fk = L.any_sersic ? (extra ? front_kernel<true, true> : front_kernel<true, false>)
                                     : (extra ? front_kernel<false, true> : front_kernel<false, false>);
        hipLaunchKernelGGL(fk, fg, dim3(kBlock), 0, stream, dparams, L, sp.begin, surv(c), cnt(c),
                           sp.len, state_buf(c), W.chunk, ft, sect);
        mark(1, 1, stream);
        if (piped()) (void)hipEventRecord(ev(1, c), stream);
    }
    // the optics stage's stream after waiting for the sky stage of chunk c
    hipStream_t optics_begin(uint64_t c) const {
        if (piped()) (void)hipStreamWaitEvent(pipe.aux, ev(1, c), 0);
        return arith();
    }
    void optics_end(uint64_t c) const {
        if (piped()) (void)hipEventRecord(ev(2, c), pipe.aux);
    }
    void fork(uint64_t n_chunks) const {
        if (!piped()) return;
        (void)hipEventRecord(pipe.ev[3 * n_chunks], stream);
        (void)hipStreamWaitEvent(pipe.aux, pipe.ev[3 * n_chunks], 0);
    }
    void join(uint64_t n_chunks) const {
        if (piped() && n_chunks) (void)hipStreamWaitEvent(stream, ev(2, n_chunks - 1), 0);
    }
    bool valid() const {
        if (!W.state || !W.survivors || !W.counts) return false;
        if ((W.n_plan && !W.plan) || W.n_plan > W.n_chunks) return false;
        if (piped() && (W.buffers < 2 || pipe.n_ev < 3 * W.n_plan + 1)) return false;
        for (uint64_t c = 0; c < W.n_plan; ++c)
            if (W.plan[c].len > W.chunk || (classed(c) && (!W.sect || preroll())) ||
                (sorted(c) && (!W.seg || !W.seg_n || !W.hist || !W.sect)))
                return false;
        return true;
    }
    // Issue every chunk's stages; optics(c) is the caller's callback for the optics stage.
    template <class Optics>
    void run(uint64_t n_chunks, bool dynamic, Optics optics) const {
        bool direct = false, cls = false;   // counters that the kernels add to
        for (uint64_t c = 0; c < n_chunks; ++c) {
            direct |= preroll() && !sorted(c);
            cls |= classed(c);
        }
        if (cls)
            hipLaunchKernelGGL(fill_u32, dim3((unsigned)((16 * n_chunks + 255) / 256)), dim3(256), 0,
                               stream, W.sect, 16 * n_chunks, 0u);
        if (direct)
            hipLaunchKernelGGL(fill_u32, dim3((unsigned)((n_chunks + 255) / 256)), dim3(256), 0,
                               stream, W.counts, n_chunks, 0u);
        fork(n_chunks);
        if (!piped()) {
            for (uint64_t c = 0; c < n_chunks; ++c) {
                pre(c);
                sky(c, dynamic ? W.tiles + 2 * c : nullptr);
                optics(c, optics_begin(c));
                optics_end(c);
            }
            return;
        }
        for (uint64_t c = 0; c < n_chunks; ++c) {
            pre(c);
            sky(c, dynamic ? W.tiles + 2 * c : nullptr);
            if (c >= 1) {
                optics(c - 1, optics_begin(c - 1));
                optics_end(c - 1);
            }
        }
        if (n_chunks) {
            optics(n_chunks - 1, optics_begin(n_chunks - 1));
            optics_end(n_chunks - 1);
        }
        join(n_chunks);
    }
};
}  // namespace

hipError_t launch_trace(const DevParams* dparams, const Launch& L, const Workspace& W, int n_cu,
                        const LaunchConfig& cfg, hipStream_t stream, const Pipe& pipe,
                        const Timing& T) {
    if (L.total == 0) return hipSuccess;
    const Stages S{dparams, L, W, n_cu, cfg, stream, pipe, T, false};
    if (!S.valid()) return hipErrorInvalidValue;
    // with ghosts every chunk's traced photons may each leave one ghost start in the list
    if ((L.flags & PHX_F_GHOSTS) && (!W.ghost_list || !W.ghost_ctr ||
                                      W.ghost_cap < ghost_entries(W.chunk, n_cu, cfg.back_per_cu)))
        return hipErrorInvalidValue;
    const uint64_t n_chunks = W.n_plan;
    if (cfg.dynamic)
        hipLaunchKernelGGL(fill_u32, dim3((unsigned)((4 * n_chunks + 255) / 256)), dim3(256), 0,
                           stream, (unsigned int*)W.tiles, 4 * n_chunks, 0u);
    S.run(n_chunks, cfg.dynamic != 0, [&](uint64_t c, hipStream_t bs) {
        const ChunkSpan& sp = W.plan[c];
        const dim3 bg((unsigned)optics_groups(cfg, n_cu, sp.len));
        unsigned long long* bt = cfg.dynamic ? W.tiles + 2 * c + 1 : nullptr;
        S.mark(2, 0, bs);
        const bool extra = (L.flags & kBackExtra) != 0, ghost = (L.flags & PHX_F_GHOSTS) != 0;
        if (ghost) {
            // the sequential pass lists the chunk's ghost starts, the second pass runs them (the
            // list is reused by the next chunk, whose optics stage follows on this stream)
            hipLaunchKernelGGL(fill_u32, dim3(1), dim3(64), 0, bs, (unsigned int*)W.ghost_ctr, 4,
                               0u);
            const auto k1 = L.any_zernike ? back_kernel<true, true, 1> : back_kernel<false, true, 1>;
            const auto k2 = L.any_zernike ? back_kernel<true, true, 2> : back_kernel<false, true, 2>;
            hipLaunchKernelGGL(k1, bg, dim3(kBlock), 0, bs, dparams, L, sp.begin, S.surv(c),
                               S.cnt(c), sp.len, (const double*)S.state_buf(c), W.chunk, bt,
                               W.ghost_list, W.ghost_cap, W.ghost_ctr);
            const uint64_t claims = (ghost_entries(sp.len, n_cu, cfg.back_per_cu) + kGhostClaim - 1) /
                                    kGhostClaim;
            const dim3 gg = grid_of((claims + kWaves - 1) / kWaves, n_cu,
                                    stage_groups(cfg, cfg.back_per_cu));
            hipLaunchKernelGGL(k2, gg, dim3(kBlock), 0, bs, dparams, L,
                               sp.begin, S.surv(c), S.cnt(c), sp.len,
                               (const double*)S.state_buf(c), W.chunk,
                               (unsigned long long*)nullptr, W.ghost_list, W.ghost_cap,
                               W.ghost_ctr);
        } else {
            const auto bk = L.any_zernike
                                    ? (extra ? back_kernel<true, true, 0> : back_kernel<true, false, 0>)
                                    : (extra ? back_kernel<false, true, 0> : back_kernel<false, false, 0>);
            hipLaunchKernelGGL(bk, bg, dim3(kBlock), 0, bs, dparams, L, sp.begin, S.surv(c),
                               S.cnt(c), sp.len, (const double*)S.state_buf(c), W.chunk, bt,
                               (double*)nullptr, (uint64_t)0, (unsigned long long*)nullptr);
        }
        S.mark(2, 1, bs);
    });
    return hipGetLastError();
}

hipError_t launch_adjoint(const DevParams* dparams, const Launch& L, const Workspace& W, int n_cu,
                          const LaunchConfig& cfg, const Adjoint& A, double* colsum, double* grad,
                          hipStream_t stream, const Pipe& pipe, const Timing& T) {
    const Stages S{dparams, L, W, n_cu, cfg, stream, pipe, T, true};
    if (!S.valid()) return hipErrorInvalidValue;
    const uint64_t grid = (uint64_t)n_cu * A.per_cu;
    if (grid * kBlock > A.tape_stride) return hipErrorInvalidValue;
    const uint64_t n_chunks = W.n_plan;
    const bool jac = A.jac != nullptr;
    S.run(n_chunks, false, [&](uint64_t c, hipStream_t bs) {
        const ChunkSpan& sp = W.plan[c];
        const uint64_t row0 = c * grid;
        const dim3 ag((unsigned)grid);
        const double* cst = S.state_buf(c);
        const uint32_t* sv = S.surv(c);
        const unsigned int* cn = S.cnt(c);
        S.mark(2, 0, bs);
        if (L.any_zernike) {
            if (jac)
                hipLaunchKernelGGL((adjoint_kernel<true, true>), ag, dim3(kBlock), 0, bs, dparams,
                                   L, sp.begin, sv, cn, sp.len, cst, W.chunk, A, row0);
            else
                hipLaunchKernelGGL((adjoint_kernel<true, false>), ag, dim3(kBlock), 0, bs, dparams,
                                   L, sp.begin, sv, cn, sp.len, cst, W.chunk, A, row0);
        } else {
            if (jac)
                hipLaunchKernelGGL((adjoint_kernel<false, true>), ag, dim3(kBlock), 0, bs, dparams,
                                   L, sp.begin, sv, cn, sp.len, cst, W.chunk, A, row0);
            else
                hipLaunchKernelGGL((adjoint_kernel<false, false>), ag, dim3(kBlock), 0, bs,
                                   dparams, L, sp.begin, sv, cn, sp.len, cst, W.chunk, A, row0);
        }
        S.mark(2, 1, bs);
    });
    const uint64_t rows = n_chunks * grid;
    hipLaunchKernelGGL(adjoint_columns, dim3(kAdj), dim3(256), 0, stream, A.partial, rows, colsum);
    hipLaunchKernelGGL(adjoint_finish, dim3(1), dim3(64), 0, stream, dparams,
                       (const double*)colsum, grad);
    return hipGetLastError();
}

// Workspace of the entry point without allocation (phx_trace_noalloc), one per GPU for the life
// of the process.  Host code never passes this name to a kernel: it is a host-side stand-in for
// the symbol, and scratch_address gives the device address to use instead.
static __device__ __align__(256) unsigned char scratch[kScratchBytes];

hipError_t scratch_address(int device, void** out) {
    static std::mutex mu;
    static void* addr[64] = {};
    if (!out || device < 0 || device >= 64) return hipErrorInvalidValue;
    int cur = -1;
    hipError_t e = hipGetDevice(&cur);
    if (e != hipSuccess) return e;
    if (cur != device) return hipErrorInvalidDevice;
    std::lock_guard<std::mutex> lock(mu);
    if (!addr[device]) {
        void* p = nullptr;
        e = hipGetSymbolAddress(&p, HIP_SYMBOL(scratch));
        if (e != hipSuccess) return e;
        addr[device] = p;
    }
    *out = addr[device];
    return hipSuccess;
}

namespace {
// Exclusive prefix of the sources' photon counts: each of 256 lanes sums a contiguous slice, a
// workgroup scan of the slice sums gives each slice its start, and the lane writes its slice.
__global__ __launch_bounds__(256) void prefix_kernel(const DevSource* __restrict__ src,
                                                     int src_begin, int n_src,
                                                     uint64_t* __restrict__ prefix) {
    __shared__ uint64_t s_sum[256];
    const int t = threadIdx.x;
    const int per = (n_src + 255) / 256;
    const int a = min(n_src, t * per), b = min(n_src, a + per);
    uint64_t sum = 0;
    for (int i = a; i < b; ++i) sum += src[src_begin + i].n_photons;
    s_sum[t] = sum;
    __syncthreads();
    for (int o = 1; o < 256; o <<= 1) {
        const uint64_t v = t >= o ? s_sum[t - o] : 0;
        __syncthreads();
        s_sum[t] += v;
        __syncthreads();
    }
    uint64_t run = t ? s_sum[t - 1] : 0;
    for (int i = a; i < b; ++i) {
        prefix[i] = run;
        run += src[src_begin + i].n_photons;
    }
    if (t == 255) prefix[n_src] = s_sum[255];
}

// guide[b] = the source holding flattened photon b << shift: the number of j in [1, n_src) with
// prefix[j] <= b << shift (the prefix does not decrease); guide[n_blocks] = n_src - 1.
__global__ __launch_bounds__(256) void guide_kernel(const uint64_t* __restrict__ prefix,
                                                    int n_src, int32_t* __restrict__ guide,
                                                    uint64_t n_blocks, uint32_t shift) {
    const uint64_t b = (uint64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (b > n_blocks) return;
    if (b == n_blocks) {
        guide[b] = n_src - 1;
        return;
    }
    const uint64_t g = b << shift;
    int lo = 1, hi = n_src;   // first j in [1, n_src) with prefix[j] > g, else n_src
    while (lo < hi) {
        const int mid = (lo + hi) >> 1;
        if (prefix[mid] <= g) lo = mid + 1; else hi = mid;
    }
    guide[b] = lo - 1;
}
}  // namespace

hipError_t launch_prefix(const DevSource* src, int src_begin, int n_src, uint64_t* prefix,
                         int32_t* guide, uint64_t n_blocks, uint32_t shift, hipStream_t stream) {
    if (!src || !prefix || !guide || n_src < 1 || src_begin < 0) return hipErrorInvalidValue;
    hipLaunchKernelGGL(prefix_kernel, dim3(1), dim3(256), 0, stream, src, src_begin, n_src, prefix);
    hipLaunchKernelGGL(guide_kernel, dim3((unsigned)((n_blocks + 1 + 255) / 256)), dim3(256), 0,
                       stream, (const uint64_t*)prefix, n_src, guide, n_blocks, shift);
    return hipGetLastError();
}

hipError_t launch_gradients(const float* opd, float4* grad, int n_layers, int n_scales, int n,
                            const double* pixel, unsigned int* gmax, hipStream_t stream) {
    // inverse 2p per scale, rounded to float once (the same value for every texel)
    float h_inv2p[PHX_MAX_SCALES];
    for (int s = 0; s < n_scales; ++s) h_inv2p[s] = (float)(1.0 / (2.0 * pixel[s]));
    float* d_inv2p = nullptr;
    hipError_t e = hipMallocAsync((void**)&d_inv2p, sizeof(h_inv2p), stream);
    if (e != hipSuccess) return e;
    e = hipMemcpyAsync(d_inv2p, h_inv2p, sizeof(float) * n_scales, hipMemcpyHostToDevice, stream);
    if (e != hipSuccess) return e;
    const int64_t total = (int64_t)n_layers * n_scales * n * n;
    const int block = 256;
    const int64_t grid = (total + block - 1) / block;
    hipLaunchKernelGGL(gradient_kernel, dim3((unsigned)grid), dim3(block), 0, stream, opd, grad, n,
                       n_scales, d_inv2p, total, gmax);
    e = hipGetLastError();
    (void)hipFreeAsync(d_inv2p, stream);
    return e;
}

}  // namespace phx
