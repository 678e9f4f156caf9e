// Sensor readout chain (section 2.4.3 saturation and bleeding; section 2.5 electronic readout):
// bleeding along half-rows, dark current and defects, per-electron parallel and serial charge
// transfer, and digitisation with read noise, gain, non-linearity, bias and bit errors.
//
// Every random draw is keyed by the pixel (or packet, or output value) it belongs to, so the
// result does not depend on the launch shape.  Floating-point contraction is off in this file: the
// decisions that quantise (transfer delays, rounding of the dark current, the digitiser's floors)
// are taken with the plain IEEE operations written.
#include <hip/hip_runtime.h>
#include <stdint.h>

#include "phx_internal.h"
#include "phx_rng.h"

#pragma clang fp contract(off)

namespace phx {
namespace {

constexpr int kRoBlock = 256;
constexpr double kTwoPi = 6.283185307179586;

__device__ __forceinline__ uint4 ro_draw(uint32_t seed, uint32_t stage, uint64_t idx,
                                         uint32_t block) {
    return philox(make_uint4((uint32_t)idx, (uint32_t)(idx >> 32), block, 0u), seed, stage);
}

__device__ __forceinline__ uint32_t ro_word(const uint4& w, int k) {
    return k == 0 ? w.x : k == 1 ? w.y : k == 2 ? w.z : w.w;
}

// Step 1: one wavefront per half-row copies it (coalesced) into the work image; if a pixel exceeds
// the full well, the half-row is then bled: pixels in index order, each excess to the
// closest pixels below full well (ties toward the row's end), the rest removed once it is full.
// With `lds` the half-row is also staged in LDS (kRoBlock / 64 half-rows of nx / 2 words per
// workgroup), the wavefront bleeds it there and writes it back; a wider half-row is bled in place by
// one lane.
__device__ __forceinline__ void bleed_half_row(uint32_t* row, int64_t a, int64_t b, int half,
                                               uint64_t w) {
    for (int64_t p = a; p < b; ++p) {
        if (row[p] <= w) continue;
        uint64_t excess = row[p] - w;
        row[p] = (uint32_t)w;
        int64_t L = p - 1, R = p + 1;
        while (excess > 0) {
            while (L >= a && row[L] >= w) --L;
            while (R < b && row[R] >= w) ++R;
            const bool hl = L >= a, hr = R < b;
            if (!hl && !hr) break;
            int64_t t;
            if (hl && hr) {
                const int64_t dl = p - L, dr = R - p;
                t = dl != dr ? (dl < dr ? L : R) : (half == 0 ? L : R);
            } else {
                t = hl ? L : R;
            }
            const uint64_t room = w - row[t];
            const uint64_t put = excess < room ? excess : room;
            row[t] += (uint32_t)put;
            excess -= put;
        }
    }
}

__device__ __forceinline__ void wave_sync() {
    __builtin_amdgcn_fence(__ATOMIC_SEQ_CST, "wavefront");
    __builtin_amdgcn_wave_barrier();
}

// The same by the whole wavefront on n pixels in LDS: 64 pixels are looked at together for the next
// one above the full well and for the closest ones below it (a lane alone, which read every
// pixel in turn, kept the copy of 4096 x 4096 pixels at 187 us; now 49 us).
__device__ __forceinline__ void bleed_half_row_wave(uint32_t* row, int n, int half, uint32_t w) {
    const int lane = threadIdx.x & 63;
    for (int base = 0; base < n; base += 64) {
        uint64_t sat = __ballot(base + lane < n && row[base + lane] > w);
        while (sat) {
            const int p = base + __ffsll((unsigned long long)sat) - 1;
            sat &= sat - 1;
            uint32_t excess = row[p] - w;
            wave_sync();
            if (lane == 0) row[p] = w;
            wave_sync();
            int L = p - 1, R = p + 1;
            while (excess > 0) {
                while (L >= 0) {
                    const uint64_t m = __ballot(L - lane >= 0 && row[max(L - lane, 0)] < w);
                    if (m) {
                        L -= __ffsll((unsigned long long)m) - 1;
                        break;
                    }
                    L -= 64;
                }
                while (R < n) {
                    const uint64_t m = __ballot(R + lane < n && row[min(R + lane, n - 1)] < w);
                    if (m) {
                        R += __ffsll((unsigned long long)m) - 1;
                        break;
                    }
                    R += 64;
                }
                const bool hl = L >= 0, hr = R < n;
                if (!hl && !hr) break;
                int t;
                if (hl && hr) {
                    const int dl = p - L, dr = R - p;
                    t = dl != dr ? (dl < dr ? L : R) : (half == 0 ? L : R);
                } else {
                    t = hl ? L : R;
                }
                const uint32_t v = row[t], put = min(excess, w - v);
                wave_sync();
                if (lane == 0) row[t] = v + put;
                wave_sync();
                excess -= put;
            }
        }
    }
}

__global__ __launch_bounds__(kRoBlock) void ro_bleed(const ReadoutJob J, int lds) {
    extern __shared__ uint32_t s_half[];
    const int wave = threadIdx.x >> 6, lane = threadIdx.x & 63;
    const uint64_t h = (uint64_t)blockIdx.x * (kRoBlock / 64) + wave;
    if (h >= 2ull * (uint64_t)J.ny) return;
    const int64_t j = (int64_t)(h >> 1);
    const int half = (int)(h & 1);
    const int64_t a = half ? J.nx / 2 : 0, b = half ? J.nx : J.nx / 2;
    const uint64_t w = (uint64_t)J.p.full_well;
    const uint32_t* src = J.in + j * J.nx;
    uint32_t* row = J.work + j * J.nx;
    uint32_t* buf = s_half + (int64_t)wave * (J.nx / 2);   // buf[x - a] holds pixel x
    bool sat = false;
    for (int64_t x = a + lane; x < b; x += 64) {
        const uint32_t v = src[x];
        row[x] = v;
        if (lds) buf[x - a] = v;
        sat |= v > w;
    }
    if (__ballot(sat) == 0) return;
    if (lds) {
        wave_sync();
        bleed_half_row_wave(buf, (int)(b - a), half, (uint32_t)w);
        wave_sync();
        for (int64_t x = a + lane; x < b; x += 64) row[x] = buf[x - a];
    } else {
        __threadfence();
        __builtin_amdgcn_wave_barrier();
        if (lane == 0) bleed_half_row(row, a, b, half, w);
    }
}

// Normal deviates in 32 bits, for decisions that are taken again in 64 where they lie within kGaussErr
// of a boundary (in units of the deviate; over every word the radius is within 5.8e-7, sine and cosine
// within 1.2e-7, and the deviate, the radius being at most 6.8, within 1.8e-6): log u from the hardware's log2 below one half and
// from 1 - u (exact in whole numbers) above it, by 2 artanh(t / (2 - t)) to the 13th power; sine and cosine
// of the angle reduced in whole numbers to an eighth of a turn, by their series.
constexpr double kGaussErr = 2e-5;
struct Polar {
    float r, c, s;
};
__device__ __forceinline__ float gauss_radius(uint32_t w) {
    const float x = ((float)w + 0.5f) * 0x1p-32f;
    const float t = ((float)~w + 0.5f) * 0x1p-32f;
    const float z = t * __builtin_amdgcn_rcpf(2.0f - t), q = z * z;
    const float far = fmaf(q, fmaf(q, fmaf(q, fmaf(q, fmaf(q, fmaf(q, 1.0f / 13, 1.0f / 11), 1.0f / 9),
                                                   1.0f / 7), 1.0f / 5), 1.0f / 3), 1.0f) * (4.0f * z);
    const float near = -1.38629436f * __builtin_amdgcn_logf(x);
    return __builtin_amdgcn_sqrtf(w >> 31 ? far : near);
}
__device__ __forceinline__ void gauss_angle(uint32_t w, float& c, float& s) {
    const uint32_t k = (w + (1u << 29)) >> 30;
    const float a = ((float)(int)(w - (k << 30)) + 0.5f) * 1.46291808e-9f;   // 2 pi 2^-32
    const float q = a * a;
    const float sn = a * fmaf(q, fmaf(q, fmaf(q, fmaf(q, 1.0f / 362880, -1.0f / 5040), 1.0f / 120),
                                      -1.0f / 6), 1.0f);
    const float cs = fmaf(q, fmaf(q, fmaf(q, fmaf(q, 1.0f / 40320, -1.0f / 720), 1.0f / 24), -0.5f),
                          1.0f);
    const float u = k & 1 ? sn : cs, v = k & 1 ? cs : sn;
    c = (k + 1) & 2 ? -u : u;
    s = k & 2 ? -v : v;
}
__device__ __forceinline__ bool near_integer(double x, double margin) {
    return !(fabs(x - rint(x)) > margin);
}

// Step 2: dark current (normal with mean and variance mu, rounded, floored at zero), then hot
// pixels set to the full well and dead pixels emptied.  (4096 x 4096 pixels 134 -> 67 us by the deviate
// in 32 bits.)
__global__ __launch_bounds__(kRoBlock) void ro_defects(const ReadoutJob J) {
    const uint64_t n = (uint64_t)J.nx * J.ny;
    const double mu = J.p.dark_rate * J.p.exposure;
    const double root = sqrt(mu), margin = root * kGaussErr + 1e-12 * (1.0 + mu);
    const double fh = J.p.hot_fraction, fd = J.p.dead_fraction;
    const uint64_t w = (uint64_t)J.p.full_well;
    for (uint64_t i = (uint64_t)blockIdx.x * blockDim.x + threadIdx.x; i < n;
         i += (uint64_t)gridDim.x * blockDim.x) {
        const uint4 r = ro_draw(J.p.seed, 1, i, 0);
        uint64_t e = J.work[i];
        if (mu > 0.0) {
            float c, s;
            gauss_angle(r.w, c, s);
            double v = mu + root * (double)(gauss_radius(r.z) * c) + 0.5;
            if (near_integer(v, margin)) {
                const double g = sqrt(-2.0 * log(u01(r.z))) * cos(kTwoPi * u01(r.w));
                v = mu + root * g + 0.5;
            }
            const double d = floor(v);
            if (d > 0.0) e += (uint64_t)d;
        }
        const double u = u01(r.x);
        if (u < fh) e = w;
        else if (u < fh + fd) e = 0;
        J.work[i] = (uint32_t)(e > 0xffffffffull ? 0xffffffffull : e);
    }
}

// Step 2, hot columns: one wavefront per segment column draws the end flags of 64 rows at a
// time, walking away from the register; from the first end on, every pixel is set to the full
// well.
__global__ __launch_bounds__(kRoBlock) void ro_hot_columns(const ReadoutJob J) {
    const int lane = threadIdx.x & 63;
    const uint64_t t = (uint64_t)blockIdx.x * (kRoBlock / 64) + (threadIdx.x >> 6);
    if (t >= (uint64_t)J.nx * J.p.amp_ny) return;
    const int64_t x = (int64_t)(t % J.nx);
    const int half = (int)(t / J.nx);
    const int64_t sh = J.ny / J.p.amp_ny;
    const uint32_t w = (uint32_t)J.p.full_well;
    int64_t first = sh;
    for (int64_t r0 = 0; r0 < sh; r0 += 64) {
        const int64_t r = r0 + lane;
        bool end = false;
        if (r < sh) {
            const int64_t y = half == 0 ? r : J.ny - 1 - r;
            end = u01(ro_draw(J.p.seed, 2, (uint64_t)y * J.nx + x, 0).x) < J.p.hot_column_fraction;
        }
        const uint64_t mask = __ballot(end);
        if (mask) {
            first = r0 + __ffsll((unsigned long long)mask) - 1;
            break;
        }
    }
    for (int64_t r = first + lane; r < sh; r += 64) {
        const int64_t y = half == 0 ? r : J.ny - 1 - r;
        J.work[(uint64_t)y * J.nx + x] = w;
    }
}

// Failures before m successes of probability 1 - eps, by inversion of u above P(0) = p0 (at most
// 64).
__device__ __forceinline__ int ro_delay(double u, int64_t m, double eps, double p0) {
    double p = p0, cum = p0;
    int f = 0;
    while (!(u < cum) && f < 64) {
        ++f;
        p *= (double)(m + f - 1) / f * eps;
        cum += p;
    }
    return f;
}

// Number of 32-bit words w with u01(w) < c: ceil(c 2^32 - 1/2) clamped to [0, 2^32].
__device__ __forceinline__ uint64_t word_bound(double c) {
    const double x = ceil(c * 4294967296.0 - 0.5);
    return x <= 0.0 ? 0ull : (x >= 4294967296.0 ? 4294967296ull : (uint64_t)x);
}

// Before the transfers: their destinations and the heavy lists' counters zeroed, and the thresholds of
// every transfer count m (thr[m - 1] of steps 3 and 4): the first two cumulative probabilities of
// the delay, as the inversion forms them, and the words they imply: u01(w) = (w + 1/2) 2^-32 < c
// exactly when w < ceil(c 2^32 - 1/2) (every step exact in double), so the decisions are whole-number
// compares, w > a0 for any delay and w > a1 for more than one slot.  a0 > a1 marks a count whose
// first probability rounds to no word at all: there every word is inverted.
__global__ __launch_bounds__(kRoBlock) void ro_init(const ReadoutJob J, uint64_t n_par,
                                                    uint64_t n_ser, double ep, double es) {
    const uint64_t id = (uint64_t)blockIdx.x * blockDim.x + threadIdx.x;
    const uint64_t step = (uint64_t)gridDim.x * blockDim.x;
    if (id < 2) J.heavy_count[id] = 0;
    const uint64_t sh = J.ny / J.p.amp_ny, sw = J.nx / J.p.amp_nx;
    for (uint64_t k = id; k < sh + sw; k += step) {
        const int64_t m = (int64_t)(k < sh ? k : k - sh) + 1;
        const double eps = k < sh ? ep : es;
        const double p0 = pow(1.0 - eps, (double)m);
        const double cum1 = p0 + p0 * ((double)m / 1 * eps);
        const uint64_t t0 = word_bound(p0), t1 = word_bound(cum1);
        const bool all = t0 == 0 || t1 == 0;
        J.thr[k] = ReadoutThr{all ? 1u : (uint32_t)(t0 - 1), all ? 0u : (uint32_t)(t1 - 1), p0};
    }
    for (uint64_t i = id; i < n_par; i += step) J.par[i] = 0;
    for (uint64_t i = id; i < n_ser; i += step) J.ser[i] = 0;
}

// Steps 3 and 4: the electrons of one packet at transfer index m - 1 (m transfers), each drawn
// a delay; electron e reads word e % 4 of draw block e / 4.  Blocks b0, b0 + db, ... are handled
// here; the kept electrons and those delayed by one slot are counted (the caller adds them to
// slots m - 1 and m), longer delays are added one by one (rare).
struct Kept {
    uint32_t k0, k1;
};
struct Packet {
    uint32_t ne;
    int64_t m;
    uint32_t* dst;
    int64_t stride, n_slots;
    ReadoutThr thr;
};

// The first n words of a block one by one through the inversion: those above lim.
__device__ __forceinline__ Kept ro_delays(const Packet& k, const uint4& r, uint32_t n, uint32_t lim,
                                          bool all, double eps) {
    Kept d{0u, 0u};   // here: inverted, of these not delayed beyond one slot
    for (uint32_t q = 0; q < n; ++q) {
        const uint32_t w = ro_word(r, (int)q);
        if (!all && w <= lim) continue;
        d.k0 += 1;
        const int64_t s = k.m - 1 + ro_delay(u01(w), k.m, eps, k.thr.p0);
        if (s < k.n_slots) atomicAdd(k.dst + s * k.stride, 1u);
    }
    return d;
}

__device__ __forceinline__ Kept ro_transfer(const Packet& k, uint64_t idx, double eps, uint32_t seed,
                                            uint32_t stage, uint32_t b0, uint32_t db) {
    const uint32_t a0 = k.thr.a0, a1 = k.thr.a1, full = k.ne >> 2, rest = k.ne & 3;
    uint32_t late = 0, longer = 0, words = 0;
    uint32_t b = b0;
    if (a0 > a1) {   // every word inverted
        for (; b < (k.ne + 3) >> 2; b += db)
            ro_delays(k, ro_draw(seed, stage, idx, b), min(4u, k.ne - 4 * b), 0u, true, eps);
        return Kept{0u, 0u};
    }
    for (; b < full; b += db) {
        const uint4 r = ro_draw(seed, stage, idx, b);
        words += 4;
        late += (r.x > a0) + (r.y > a0) + (r.z > a0) + (r.w > a0);
        if (max(max(r.x, r.y), max(r.z, r.w)) > a1) longer += ro_delays(k, r, 4, a1, false, eps).k0;
    }
    if (b == full && rest) {
        const uint4 r = ro_draw(seed, stage, idx, b);
        words += rest;
        late += (r.x > a0) + (rest > 1 && r.y > a0) + (rest > 2 && r.z > a0);
        if (max(max(r.x, r.y), r.z) > a1) longer += ro_delays(k, r, rest, a1, false, eps).k0;
    }
    return Kept{words - late, late - longer};
}

// Packets with more electrons than some limit are handed to whole wavefronts (the heavy list): in the
// other kernel one of them holds up the 63 packets beside it, for one block of draws per four electrons.
// A wavefront weighs the two (light_limit): a limit t costs it up to (t - kHeavy) / 4 blocks more, a
// packet above the limit about kHeavyBlocks of them in the other kernel (0.97 ns a packet against 0.09 ns a
// wavefront's block on the filled chip).  So a bright pixel among dark ones goes to the list, and a
// background, with which all packets of the wavefront are as large, does not.  4096 x 4096 pixels of 300
// electrons take 5.7 ms (with every packet above 64 on the list 41.8; with up to 1024 never on it 8.7), of
// 1000 26 (53.7; 44.5); a field of 1e4 stars without a background 2.6 either way (4.5), at 1024 x 1024
// 0.33 (0.34; 0.72).  4 and 12 blocks gave the same within 3 % but for 1000 (4: 54 ms) and 2000 electrons
// (12: 34 ms, against 65) and the small dense field (12: 0.344 against 0.331).
constexpr uint32_t kHeavy = 64, kLightMax = 2048, kHeavyBlocks = 8;

__device__ __forceinline__ uint32_t light_limit(uint32_t ne) {
    uint32_t cost = kHeavyBlocks * (uint32_t)__popcll(__ballot(ne > kHeavy)), lim = kHeavy;
    if (cost == 0) return lim;   // the wavefront's
    for (uint32_t t = 2 * kHeavy; t <= kLightMax; t *= 2) {
        const uint32_t c = (t - kHeavy) / 4 + kHeavyBlocks * (uint32_t)__popcll(__ballot(ne > t));
        if (c < cost) {
            cost = c;
            lim = t;
        }
    }
    return lim;
}

__device__ __forceinline__ uint64_t div_by(uint64_t a, uint64_t b) {
    return (a | b) >> 32 ? a / b : (uint64_t)((uint32_t)a / (uint32_t)b);
}

// Packet i of a transfer stage, ne electrons: transfer count m, destination column or row, slot
// stride and count, thresholds.
template <int STAGE>
__device__ __forceinline__ Packet packet_of(const ReadoutJob& J, uint64_t i, uint32_t ne) {
    const int64_t sw = J.nx / J.p.amp_nx, sh = J.ny / J.p.amp_ny;
    const int64_t ph = sh + J.p.over_y, pw = sw + J.p.over_x;
    Packet k;
    if (STAGE == 3) {
        const int64_t y = (int64_t)div_by(i, J.nx), x = (int64_t)i - y * J.nx;
        const int64_t ax = (int32_t)x / (int32_t)sw, ay = (int32_t)y / (int32_t)sh;
        const int64_t amp = ay * J.p.amp_nx + ax, c = x - ax * sw;
        const int64_t r = ay == 0 ? y : J.ny - 1 - y;
        k = Packet{ne, r + 1, J.par + amp * ph * sw + c, sw, ph, J.thr[r]};
    } else {
        const int64_t rowi = (int64_t)div_by(i, sw), c = (int64_t)i - rowi * sw;   // amp ph + s
        k = Packet{ne, c + 1, J.ser + rowi * pw, 1, pw, J.thr[sh + c]};
    }
    return k;
}

template <int STAGE>
__device__ __forceinline__ uint32_t packet_electrons(const ReadoutJob& J, uint64_t i) {
    return STAGE == 3 ? J.work[i] : J.par[i];
}

// One thread per packet, `per` packets per workgroup (light_packets); packets above the wavefront's limit go
// to the heavy list instead, a workgroup's together: one atomic on the list's length each (one per packet
// serialised the kernel: 1.4e4 of them 0.46 ms, now 0.11).
constexpr uint32_t kPerBlock = 4096;

template <int STAGE>
__global__ __launch_bounds__(kRoBlock) void ro_transfer_light(const ReadoutJob J, uint64_t n,
                                                              uint32_t per, double eps) {
    __shared__ uint16_t s_list[kPerBlock];
    __shared__ uint32_t s_n, s_base;
    uint32_t* count = J.heavy_count + (STAGE - 3);
    for (uint64_t i0 = (uint64_t)blockIdx.x * per; i0 < n;
         i0 += (uint64_t)gridDim.x * per) {   // workgroup-uniform
        if (threadIdx.x == 0) s_n = 0;
        __syncthreads();
        constexpr int kBatch = 8;
        for (uint32_t c = 0; c < per; c += kBatch * kRoBlock) {
            const int batch = (int)min((uint32_t)kBatch, (per - c) / kRoBlock);
            uint32_t e[kBatch];
#pragma unroll
            for (int j = 0; j < kBatch; ++j) {
                const uint64_t i = i0 + c + j * kRoBlock + threadIdx.x;
                e[j] = j < batch && i < n ? packet_electrons<STAGE>(J, i) : 0u;
            }
#pragma unroll 1
            for (int j = 0; j < batch; ++j) {
                uint32_t ne = e[0];
#pragma unroll
                for (int q = 0; q + 1 < kBatch; ++q) e[q] = e[q + 1];
                const uint32_t lim = light_limit(ne);   // of every lane of the wavefront
                if (ne == 0) continue;
                const uint32_t o = c + j * kRoBlock + threadIdx.x;
                if (ne > lim && eps > 0.0) {
                    s_list[atomicAdd(&s_n, 1u)] = (uint16_t)o;
                    continue;
                }
                const uint64_t i = i0 + o;
                const Packet k = packet_of<STAGE>(J, i, ne);
                Kept kk{ne, 0u};
                if (eps > 0.0) kk = ro_transfer(k, i, eps, J.p.seed, STAGE, 0, 1);
                if (kk.k0) atomicAdd(k.dst + (k.m - 1) * k.stride, kk.k0);
                if (kk.k1 && k.m < k.n_slots) atomicAdd(k.dst + k.m * k.stride, kk.k1);
            }
        }
        __syncthreads();
        if (threadIdx.x == 0 && s_n) s_base = atomicAdd(count, s_n);
        __syncthreads();
        for (uint32_t q = threadIdx.x; q < s_n; q += kRoBlock)
            J.heavy[s_base + q] = (uint32_t)(i0 + s_list[q]);
        __syncthreads();
    }
}

// kSplit wavefronts per heavy packet: wavefront `sub` takes the draw blocks sub * 64 + lane +
// j * kSplit * 64, and each sums its kept electrons (a few hundred saturated pixels would
// otherwise leave most SIMDs with one long dependent chain each).
constexpr uint32_t kSplit = 4;
__device__ __forceinline__ uint32_t wave_sum(uint32_t v) {
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) v += __shfl_xor(v, o);
    return v;
}

template <int STAGE>
__global__ __launch_bounds__(kRoBlock) void ro_transfer_heavy(const ReadoutJob J, double eps) {
    const uint64_t n = (uint64_t)J.heavy_count[STAGE - 3] * kSplit;
    const int lane = threadIdx.x & 63;
    const uint64_t waves = (uint64_t)gridDim.x * (kRoBlock / 64);
    for (uint64_t t = (uint64_t)blockIdx.x * (kRoBlock / 64) + (threadIdx.x >> 6); t < n;
         t += waves) {
        // the packet is the wavefront's: scalar, and with it the parts of the draws that do not
        // depend on the block
        const uint32_t i = __builtin_amdgcn_readfirstlane(J.heavy[t / kSplit]);
        const uint32_t ne = __builtin_amdgcn_readfirstlane(packet_electrons<STAGE>(J, i));
        const uint32_t sub = (uint32_t)(t % kSplit);
        if (sub * 256u >= ne) continue;
        const Packet k = packet_of<STAGE>(J, i, ne);
        const Kept kk = ro_transfer(k, i, eps, J.p.seed, STAGE, sub * 64u + (uint32_t)lane,
                                    64u * kSplit);
        const uint32_t k0 = wave_sum(kk.k0), k1 = wave_sum(kk.k1);
        if (lane == 0) {
            if (k0) atomicAdd(k.dst + (k.m - 1) * k.stride, k0);
            if (k1 && k.m < k.n_slots) atomicAdd(k.dst + k.m * k.stride, k1);
        }
    }
}

// Step 5: read noise, gain, non-linearity, bias, clamp, bit errors, in the plain operations.
__device__ __forceinline__ uint16_t digitise_exact(const ReadoutJob& J, uint64_t i, int amp, uint32_t ne) {
    const double W = J.p.full_well;
    const uint4 r = ro_draw(J.p.seed, 5, i, 0);
    double e = (double)ne;
    e += J.p.read_noise[amp] * sqrt(-2.0 * log(u01(r.x))) * cos(kTwoPi * u01(r.y));
    double adu = e / (J.p.gain[amp] * (1.0 + J.p.nonlinearity * e / W)) + J.p.bias[amp];
    adu = adu < 0.0 ? 0.0 : (adu > 65535.0 ? 65535.0 : adu);
    uint32_t val = 0;
#pragma unroll 1
    for (int k = 0; k < 4; ++k) {
        double g[4] = {0.0, 0.0, 0.0, 0.0};
        // a block whose four widths are zero contributes nothing (0 x g): not drawn
        const bool need = J.p.bit_sigma[4 * k] > 0.0 || J.p.bit_sigma[4 * k + 1] > 0.0 ||
                          J.p.bit_sigma[4 * k + 2] > 0.0 || J.p.bit_sigma[4 * k + 3] > 0.0;
        if (need) {
            const uint4 v = ro_draw(J.p.seed, 5, i, 1 + k);
            const double r0 = sqrt(-2.0 * log(u01(v.x))), r1 = sqrt(-2.0 * log(u01(v.z)));
            g[0] = r0 * cos(kTwoPi * u01(v.y));
            g[1] = r0 * sin(kTwoPi * u01(v.y));
            g[2] = r1 * cos(kTwoPi * u01(v.w));
            g[3] = r1 * sin(kTwoPi * u01(v.w));
        }
#pragma unroll
        for (int q = 0; q < 4; ++q) {
            const int bit = 4 * k + q;
            // ldexp by -bit equals the division by 2^bit exactly
            const double a = ldexp(adu, -bit) + J.p.bit_sigma[bit] * g[q];
            const int64_t f = (int64_t)floor(a);
            if (((f % 2) + 2) % 2) val |= 1u << bit;
        }
    }
    return (uint16_t)val;
}

// The same with the deviates in 32 bits, which settle a value unless some floor lies within their
// error (about one value in 2000): then, or where the bounds do not hold (a value at the converter's
// limits, a strong non-linearity), the plain operations decide.  The bits without an error
// are those of the value's own floor.  One grid row per amplifier.  1.7e7 values 506 -> 313 us.
__global__ __launch_bounds__(kRoBlock) void ro_digitise(const ReadoutJob J) {
    const int64_t sw = J.nx / J.p.amp_nx, sh = J.ny / J.p.amp_ny;
    const uint64_t per_amp = (uint64_t)(sh + J.p.over_y) * (uint64_t)(sw + J.p.over_x);
    const int amp = blockIdx.y;
    const double rn = J.p.read_noise[amp], gain = J.p.gain[amp], bias = J.p.bias[amp];
    const double nl = J.p.nonlinearity / J.p.full_well;
    // error of the electrons, and of the value by its slope (at most 1 / (gain 0.89^2) where the
    // linearity term is at least 0.9 and its own error small), and the roundings of both forms of the
    // quotient (twelve of 2^-53 of a quotient that is at most 65536 + |bias| for a value in range)
    const double de = rn * kGaussErr, dv = 1.3 * de / gain + 2e-15 * (1e6 + fabs(bias));
    const bool bounded = nl * de < 0.01;
    uint32_t noisy = 0;
    for (int b = 0; b < 16; ++b) noisy |= J.p.bit_sigma[b] > 0.0 ? 1u << b : 0u;
    for (uint64_t p = (uint64_t)blockIdx.x * blockDim.x + threadIdx.x; p < per_amp;
         p += (uint64_t)gridDim.x * blockDim.x) {
        const uint64_t i = (uint64_t)amp * per_amp + p;
        const uint32_t ne = J.ser[i];
        const uint4 r = ro_draw(J.p.seed, 5, i, 0);
        float c, s;
        gauss_angle(r.y, c, s);
        const double e = (double)ne + rn * (double)(gauss_radius(r.x) * c);
        const double lin = 1.0 + nl * e;
        const double adu = e / (gain * lin) + bias;
        bool exact = !bounded || !(lin >= 0.9) || !(adu > dv) || !(adu < 65535.0 - dv) ||
                     near_integer(adu, dv);
        uint32_t val = exact ? 0u : (uint32_t)adu & ~noisy;
#pragma unroll
        for (int k = 0; k < 4; ++k) {
            if (!(noisy >> (4 * k) & 15u)) continue;
            const uint4 v = ro_draw(J.p.seed, 5, i, 1 + k);
#pragma unroll
            for (int h = 0; h < 2; ++h) {
                if (!(noisy >> (4 * k + 2 * h) & 3u)) continue;
                const float rad = gauss_radius(h ? v.z : v.x);
                gauss_angle(h ? v.w : v.y, c, s);
#pragma unroll
                for (int q = 0; q < 2; ++q) {
                    const int bit = 4 * k + 2 * h + q;
                    if (!(noisy >> bit & 1u)) continue;
                    const double inv = 1.0 / (double)(1u << bit), sig = J.p.bit_sigma[bit];
                    const double a = adu * inv + sig * (double)(rad * (q ? s : c));
                    exact |= near_integer(a, dv * inv + sig * kGaussErr);
                    if ((int64_t)floor(a) & 1) val |= 1u << bit;
                }
            }
        }
        J.out[i] = exact ? digitise_exact(J, i, amp, ne) : (uint16_t)val;
    }
}

unsigned grid_for(uint64_t n) {
    const uint64_t g = (n + kRoBlock - 1) / kRoBlock;
    return (unsigned)(g < (1ull << 20) ? (g ? g : 1) : (1ull << 20));
}

}  // namespace

hipError_t launch_readout(const ReadoutJob& J, hipStream_t s) {
    const uint64_t npix = (uint64_t)J.nx * J.ny;
    const int64_t sw = J.nx / J.p.amp_nx, sh = J.ny / J.p.amp_ny;
    const int64_t ph = sh + J.p.over_y, pw = sw + J.p.over_x;
    const uint64_t n_amp = (uint64_t)J.p.amp_nx * J.p.amp_ny;
    const uint64_t n_par = n_amp * ph * sw, n_ser = n_amp * ph * pw;
    const uint64_t half_rows = 2ull * (uint64_t)J.ny;
    const size_t lds_bytes = (size_t)(kRoBlock / 64) * (J.nx / 2) * sizeof(uint32_t);
    const int lds = lds_bytes <= 64 * 1024 ? 1 : 0;
    hipLaunchKernelGGL(ro_bleed, dim3((unsigned)((half_rows + 3) / 4)), dim3(kRoBlock),
                       lds ? lds_bytes : 0, s, J, lds);
    hipLaunchKernelGGL(ro_defects, dim3(grid_for(npix)), dim3(kRoBlock), 0, s, J);
    if (J.p.hot_column_fraction > 0.0)
        hipLaunchKernelGGL(ro_hot_columns,
                           dim3((unsigned)(((uint64_t)J.nx * J.p.amp_ny + 3) / 4)),
                           dim3(kRoBlock), 0, s, J);
    const double ep = 1.0 - J.p.cte_parallel, es = 1.0 - J.p.cte_serial;
    const unsigned heavy_grid = 2048;
    // Packets per workgroup: about sixteen workgroups per compute unit, of 256 to 4096 packets (more
    // workgroups are more appends to the heavy list).  With 4096 everywhere one workgroup held all of 64 x 64
    // pixels, 16 rounds of packets one after the other: with 30 electrons each 222 us, now 123; 1024 x 1024
    // of them 268 us, now 200; at 4096 x 4096 the rule gives the 4096.
    const auto light_packets = [](uint64_t n) {
        const uint64_t p = (n / 4096 + kRoBlock - 1) / kRoBlock * kRoBlock;
        return (uint32_t)(p < kRoBlock ? kRoBlock : p > kPerBlock ? kPerBlock : p);
    };
    const auto light_grid = [&](uint64_t n) {
        const uint64_t per = light_packets(n), g = (n + per - 1) / per;
        return dim3((unsigned)(g < (1ull << 20) ? g : 1ull << 20));
    };
    hipLaunchKernelGGL(ro_init, dim3(4096), dim3(kRoBlock), 0, s, J, n_par, n_ser, ep, es);
    hipLaunchKernelGGL(ro_transfer_light<3>, light_grid(npix), dim3(kRoBlock), 0, s, J, npix,
                       light_packets(npix), ep);
    hipLaunchKernelGGL(ro_transfer_heavy<3>, dim3(heavy_grid), dim3(kRoBlock), 0, s, J, ep);
    hipLaunchKernelGGL(ro_transfer_light<4>, light_grid(n_par), dim3(kRoBlock), 0, s, J, n_par,
                       light_packets(n_par), es);
    hipLaunchKernelGGL(ro_transfer_heavy<4>, dim3(heavy_grid), dim3(kRoBlock), 0, s, J, es);
    hipLaunchKernelGGL(ro_digitise, dim3(grid_for((uint64_t)ph * pw), (unsigned)n_amp),
                       dim3(kRoBlock), 0, s, J);
    return hipGetLastError();
}

}  // namespace phx
