// Per-source centroids and second moments from the trace's exact moment words (the per-source
// outputs of the paper's section 3.1: counts and centroids of the sources; "weighted moments" of
// section 4 read as unweighted moments of the converted photons' electron positions), and the
// adjoint's per-photon cotangent coefficients from a loss gradient with respect to those moments.
//
// The words hold n and the 128-bit sums SX, SY, SXX, SYY, SXY of positions quantised to
// X = x 2^44.  Each result is a ratio of integers,
//   mean x = SX / (n 2^44),   Ixx = (n SXX - SX^2) / (n^2 2^88),   Ixy = (n SXY - SX SY) / (n^2 2^88),
// formed here in exact multiword integer arithmetic and rounded once to the nearest double (ties
// to even), so the small central moments of a far-off-axis source lose nothing to cancellation.
//
// One thread per source and result: with one thread per source the five divisions follow each
// other, and one bit of the quotient per step they took 162 us for one source and 187 us for 441.
// The kernels are latency-bound at any source count a catalogue has, so the chain is what counts: the
// numerator has at most 256 and the denominator at most 128 bits, every limb index is static (no
// scratch), and the 64-bit quotient comes from one 128 / 64-bit estimate that is at most two too
// large once the denominator's top bit is set (Knuth, TAOCP vol. 2, 4.3.1, theorem B).  4.3 us
// for one source and 5.7 us for 441.
#include <hip/hip_runtime.h>

#include "phx_internal.h"

namespace phx {
namespace {

struct U128 {
    uint64_t lo, hi;
};
struct U256 {
    uint64_t w[4];
};

__host__ __device__ __forceinline__ int top_bits(uint64_t x) {   // bit length
#ifdef __HIP_DEVICE_COMPILE__
    return 64 - __clzll((long long)x);
#else
    return x ? 64 - __builtin_clzll(x) : 0;
#endif
}

__host__ __device__ __forceinline__ U128 mul64(uint64_t a, uint64_t b) {
    const unsigned __int128 p = (unsigned __int128)a * b;
    return U128{(uint64_t)p, (uint64_t)(p >> 64)};
}

// a x b, 64 x 128 and 128 x 128 bits
__host__ __device__ __forceinline__ U256 mul_64_128(uint64_t a, U128 b) {
    const U128 p = mul64(a, b.lo), q = mul64(a, b.hi);
    const uint64_t m = p.hi + q.lo;
    return U256{{p.lo, m, q.hi + (m < p.hi), 0}};
}
__host__ __device__ __forceinline__ U256 mul_128(U128 a, U128 b) {
    const U256 p = mul_64_128(a.lo, b), q = mul_64_128(a.hi, b);   // p + q 2^64
    U256 r;
    r.w[0] = p.w[0];
    r.w[1] = p.w[1] + q.w[0];
    uint64_t c = r.w[1] < p.w[1];
    r.w[2] = p.w[2] + q.w[1];
    const uint64_t c1 = r.w[2] < p.w[2];
    r.w[2] += c;
    c = c1 + (r.w[2] < c);
    r.w[3] = q.w[2] + c;
    return r;
}

__host__ __device__ __forceinline__ U256 add256(const U256& a, const U256& b) {
    U256 r;
    uint64_t c = 0;
#pragma unroll
    for (int i = 0; i < 4; ++i) {
        const uint64_t v = a.w[i] + c;
        const uint64_t c1 = v < c;
        r.w[i] = v + b.w[i];
        c = c1 + (r.w[i] < v);
    }
    return r;
}

// a - b modulo 2^256; borrow: a < b
__host__ __device__ __forceinline__ U256 sub256(const U256& a, const U256& b, bool& borrow) {
    U256 r;
    uint64_t c = 0;
#pragma unroll
    for (int i = 0; i < 4; ++i) {
        const uint64_t v = a.w[i] - b.w[i];
        const uint64_t c1 = a.w[i] < b.w[i];
        r.w[i] = v - c;
        c = c1 + (v < c);
    }
    borrow = c != 0;
    return r;
}

// x shifted left by 0 <= s < 256
__host__ __device__ __forceinline__ U256 shl256(U256 x, int s) {
    if (s & 128) x = U256{{0, 0, x.w[0], x.w[1]}};
    if (s & 64) x = U256{{0, x.w[0], x.w[1], x.w[2]}};
    const int b = s & 63;
    if (b) {
        x.w[3] = (x.w[3] << b) | (x.w[2] >> (64 - b));
        x.w[2] = (x.w[2] << b) | (x.w[1] >> (64 - b));
        x.w[1] = (x.w[1] << b) | (x.w[0] >> (64 - b));
        x.w[0] <<= b;
    }
    return x;
}

// floor((hi : lo) / d) for hi < d with d's top bit set: two 32-bit quotient digits, each from a
// 64 / 32-bit estimate corrected at most twice.
__host__ __device__ __forceinline__ uint64_t div_128_64(uint64_t hi, uint64_t lo, uint64_t d) {
    const uint64_t d1 = d >> 32, d0 = d & 0xffffffffull;
    uint64_t q = 0;
#pragma unroll
    for (int k = 1; k >= 0; --k) {
        const uint64_t next = k ? lo >> 32 : lo & 0xffffffffull;
        uint64_t e = hi / d1, r = hi - e * d1;
#pragma unroll
        for (int t = 0; t < 2; ++t)
            if (r <= 0xffffffffull && (e > 0xffffffffull || e * d0 > ((r << 32) | next))) {
                e -= 1;
                r += d1;
            }
        hi = ((hi << 32) | next) - e * d;   // the partial remainder, below d
        q = (q << 32) | e;
    }
    return q;
}

// num / den x 2^e2 rounded once to the nearest double (ties to even), num, den > 0.  The quotient
// q = floor(num 2^sh / den) is formed with 63 or 64 bits; its bits below the double's 53 and the
// remainder decide the rounding.
__host__ __device__ __forceinline__ double ratio(const U256& num, U128 den, int e2) {
    const int ln = num.w[3] ? 192 + top_bits(num.w[3])
                            : num.w[2] ? 128 + top_bits(num.w[2])
                                       : num.w[1] ? 64 + top_bits(num.w[1]) : top_bits(num.w[0]);
    const int ld = den.hi ? 64 + top_bits(den.hi) : top_bits(den.lo);
    const int sh = 63 + ld - ln;
    // den shifted to 128 bits, num (shifted by sh with it) to 191: below den 2^64
    const U256 dn = shl256(U256{{den.lo, den.hi, 0, 0}}, 128 - ld);
    const int t = 191 - ln;   // negative: num's lowest -t bits go, and count as a remainder
    bool sticky = false;
    U256 n;
    if (t >= 0) {
        n = shl256(num, t);
    } else {
        const int k = -t;   // 1 .. 65, since num has at most 256 bits
        U256 m = num;
        if (k >= 64) {
            sticky = m.w[0] != 0;
            m = U256{{m.w[1], m.w[2], m.w[3], 0}};
        }
        const int b = k & 63;
        if (b) {
            sticky |= (m.w[0] & ((1ull << b) - 1ull)) != 0;
            m.w[0] = (m.w[0] >> b) | (m.w[1] << (64 - b));
            m.w[1] = (m.w[1] >> b) | (m.w[2] << (64 - b));
            m.w[2] = (m.w[2] >> b) | (m.w[3] << (64 - b));
            m.w[3] >>= b;
        }
        n = m;
    }
    uint64_t q = div_128_64(n.w[2], n.w[1], dn.w[1]);
    bool neg;
    U256 rem = sub256(n, mul_64_128(q, U128{dn.w[0], dn.w[1]}), neg);
#pragma unroll
    for (int i = 0; i < 2; ++i)
        if (neg) {
            q -= 1;
            rem = add256(rem, dn);
            neg = (rem.w[3] >> 63) != 0;
        }
    sticky |= (rem.w[0] | rem.w[1] | rem.w[2] | rem.w[3]) != 0;
    const int drop = top_bits(q) - 53;   // 10 or 11
    uint64_t m = q >> drop;
    const uint64_t low = q & ((1ull << drop) - 1), half = 1ull << (drop - 1);
    if ((low & half) && ((low & (half - 1)) != 0 || sticky || (m & 1u))) m += 1;
    return ldexp((double)m, e2 - sh + drop);   // m = 2^53 after a carry is still exact
}

struct Signed128 {
    bool neg;
    U128 mag;
};
__host__ __device__ __forceinline__ Signed128 s128(uint64_t lo, uint64_t hi) {
    Signed128 r{(hi >> 63) != 0, U128{lo, hi}};
    if (r.neg) {   // two's complement magnitude
        r.mag.lo = ~lo + 1;
        r.mag.hi = ~hi + (r.mag.lo == 0);
    }
    return r;
}

// Result i of a source's words: 0 the count, 1 mean x, 2 mean y, 3 Ixx, 4 Iyy, 5 Ixy.
__host__ __device__ __forceinline__ double source_moment(const unsigned long long* w, int i) {
    const uint64_t n = w[0];
    if (i == 0 || n == 0) return i == 0 ? (double)n : 0.0;
    constexpr int q = PHX_MOMENT_Q_LOG2;
    // the sums entering result i: numerator S (means) or n S - A B (second moments)
    const int ks = 2 * i;   // SX 2, SY 4, SXX 6, SYY 8, SXY 10
    const Signed128 S = s128(w[ks], w[ks + 1]);
    U256 num{{S.mag.lo, S.mag.hi, 0, 0}};
    bool neg = S.neg;
    U128 den{n, 0};
    if (i >= 3) {
        const int ka = i == 4 ? 4 : 2, kb = i == 3 ? 2 : 4;
        const Signed128 A = s128(w[ka], w[ka + 1]), B = s128(w[kb], w[kb + 1]);
        const U256 P = mul_64_128(n, S.mag), Q = mul_128(A.mag, B.mag);
        const bool pneg = S.neg, qneg = A.neg != B.neg;
        if (pneg != qneg) {
            num = add256(P, Q);
            neg = pneg;
        } else {
            bool less;
            num = sub256(P, Q, less);
            neg = pneg;
            if (less) {
                bool x;
                num = sub256(Q, P, x);
                neg = !pneg;
            }
        }
        den = mul64(n, n);
    }
    if ((num.w[0] | num.w[1] | num.w[2] | num.w[3]) == 0) return 0.0;
    const double v = ratio(num, den, i <= 2 ? -q : -2 * q);
    return neg ? -v : v;
}

constexpr int kPerSource = 8;   // threads per source (results 0..5)

__global__ __launch_bounds__(64) void moments_kernel(const unsigned long long* __restrict__ words,
                                                     int n_src, double* __restrict__ out) {
    const int t = blockIdx.x * blockDim.x + threadIdx.x;
    const int s = t / kPerSource, i = t % kPerSource;
    if (s >= n_src || i >= 6) return;
    out[(size_t)s * 6 + i] = source_moment(words + (size_t)s * PHX_MOMENT_WORDS, i);
}

// Cotangent coefficients of the adjoint for a loss L(mean x, mean y, Ixx, Iyy, Ixy) per source:
// d mean/d x_i = 1/n, d Ixx/d x_i = 2 (x_i - mean x)/n, d Ixy/d x_i = (y_i - mean y)/n, so that
// xbar_i = g0 + g2 (x_i - g5) + g4 (y_i - g6) and ybar_i = g1 + g3 (y_i - g6) + g4 (x_i - g5)
// with g = (dL/dmx, dL/dmy, 2 dL/dIxx, 2 dL/dIyy, dL/dIxy) / n and (g5, g6) the mean; a source
// without converted photons gets a zero row.  One thread per coefficient (214 us with one thread
// per source, of which the second moments it does not need were most; 5 us).
__global__ __launch_bounds__(64) void seed_kernel(const unsigned long long* __restrict__ words,
                                                  int n_src, const double* __restrict__ dmom,
                                                  double* __restrict__ seed) {
    const int t = blockIdx.x * blockDim.x + threadIdx.x;
    const int s = t / kPerSource, i = t % kPerSource;
    if (s >= n_src) return;
    const unsigned long long* w = words + (size_t)s * PHX_MOMENT_WORDS;
    const double n = (double)w[0];
    double g = 0.0;
    if (n != 0.0) {
        if (i < 5) {
            const double d = dmom[(size_t)s * 5 + i];
            g = (i == 2 || i == 3 ? 2.0 * d : d) * (1.0 / n);
        } else if (i < 7) {
            g = source_moment(w, i - 4);
        }
    }
    seed[(size_t)s * 8 + i] = g;
}

unsigned blocks_for(int n_src) {
    return (unsigned)(((uint64_t)n_src * kPerSource + 63) / 64);
}

}  // namespace

hipError_t launch_moments(const unsigned long long* words, int n_src, double* out,
                          hipStream_t stream) {
    if (n_src <= 0) return hipSuccess;
    hipLaunchKernelGGL(moments_kernel, dim3(blocks_for(n_src)), dim3(64), 0, stream,
                       words, n_src, out);
    return hipGetLastError();
}

hipError_t launch_seeds(const unsigned long long* words, int n_src, const double* dmom,
                        double* seed, hipStream_t stream) {
    if (n_src <= 0) return hipSuccess;
    hipLaunchKernelGGL(seed_kernel, dim3(blocks_for(n_src)), dim3(64), 0, stream,
                       words, n_src, dmom, seed);
    return hipGetLastError();
}

}  // namespace phx
