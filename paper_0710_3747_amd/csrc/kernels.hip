// kernels.hip -- gfx950 kernels of the random-phase Trotter path.
//
//  k_init        random-phase state (counter-based SplitMix64 phases), or the
//                product state of M-1 random single-spin phases
//  k_init_members  2^c basis-state members of the ensemble stacked as one
//                state of M + c sites (member index on the top c bits)
//  k_accumulate  member sums of consecutive evolutions, in order
//  k_pass        one tiled sweep: a 2^k-amplitude tile per workgroup is held
//                in registers, whose stages apply the two-spin factors as
//                three-shear rotations and exchange through LDS; observables
//                are accumulated in FP64 and reduced per workgroup
//  k_resident    whole state in one workgroup's registers for every step
//  k_batch       many problems in one launch: whole ones in a workgroup, larger
//                ones by gangs of workgroups that meet after every pass
//  k_factor      one factor over the whole state (the unfused schedule)
//  k_observe     observable of a state as it is
//  k_reduce      fixed-order reduction of per-workgroup partial sums
#include <hip/hip_runtime.h>
#include <stdint.h>

#include "device_plan.hpp"
#include "kernels.hpp"

// The file is compiled once per part, in parallel: part 0 holds the small
// kernels and the launchers, the others one family of template kernels each.
#ifndef SPIN_PART
#error "compile with -DSPIN_PART=0..7 (see build.py)"
#endif

namespace spinqp {

template <typename T> struct CT;
template <> struct CT<float> {
    using c = float2;
    using v = float4;       // 16-byte global access: two amplitudes
    static constexpr int V = 2;
};
template <> struct CT<double> {
    using c = double2;
    using v = double2;      // 16-byte global access: one amplitude
    static constexpr int V = 1;
};

// ------------------------------------------------------------ SplitMix64
__device__ __forceinline__ uint64_t sm64_mix(uint64_t z) {
    z = (z ^ (z >> 30)) * 0xBF58476D1CE4E5B9ull;
    z = (z ^ (z >> 27)) * 0x94D049BB133111EBull;
    return z ^ (z >> 31);
}

// u(seed, r) = (z >> 11) 2^-53 with z output r+1 of the SplitMix64 stream
// started at `seed`, read directly at that counter.
__device__ __forceinline__ double sm64_uniform(uint64_t seed, uint64_t r) {
    const uint64_t z = sm64_mix(seed + (r + 1ull) * 0x9E3779B97F4A7C15ull);
    return double(z >> 11) * 0x1.0p-53;
}

// sin and cos of 2 pi u for u in [0, 1]: the nearest quarter turn is taken off
// exactly (u = q/4 + f, |f| <= 1/8), then the Taylor series in f^2, coefficients
// (2 pi)^k / k! (the first neglected terms are below 3e-20).  Each is within
// 1.1 ulp of the exact value (measured over 5e6 arguments).
__device__ __forceinline__ void sincos_turn(double u, double* s, double* c) {
    const double q = rint(4.0 * u);
    const double f = fma(-0.25, q, u), t = f * f;
    double a = 0x1.aaec32af93359p-4;
    a = fma(a, t, -0x1.6fadb9f155744p-1);
    a = fma(a, t, 0x1.e8f434d018d63p+1);
    a = fma(a, t, -0x1.e3074fde8871fp+3);
    a = fma(a, t, 0x1.50783487ee782p+5);
    a = fma(a, t, -0x1.32d2cce62bd86p+6);
    a = fma(a, t, 0x1.466bc6775aae2p+6);
    a = fma(a, t, -0x1.4abbce625be53p+5);
    a = fma(a, t, 0x1.1a62633145c07p-52);       // the rest of 2 pi
    a = fma(f, 0x1.921fb54442d18p+2, f * a);
    double b = 0x1.20c62c2f2d7f5p-2;
    b = fma(b, t, -0x1.b6e24f44b128fp+0);
    b = fma(b, t, 0x1.f9d38a3763cc3p+2);
    b = fma(b, t, -0x1.a6d1f2a204a8cp+4);
    b = fma(b, t, 0x1.e1f506891babbp+5);
    b = fma(b, t, -0x1.55d3c7e3cbffap+6);
    b = fma(b, t, 0x1.03c1f081b5ac4p+6);
    // 1 + C1 t with its rounding error and that of t carried along
    const double h = fma(t, -0x1.3bd3cc9be45dep+4, 1.0);
    const double e = fma(fma(f, f, -t), -0x1.3bd3cc9be45dep+4, fma(t, -0x1.3bd3cc9be45dep+4, 1.0 - h));
    b = h + fma(t * t, b, e);
    const int k = int(q);
    const double x = (k & 1) ? b : a, y = (k & 1) ? a : b;
    *s = (k & 2) ? -x : x;
    *c = ((k + 1) & 2) ? -y : y;
}

// Amplitude of basis state x of the random-phase state, FP64.
__device__ __forceinline__ void random_phase_amp(uint64_t x, int n, uint64_t seed, double scale,
                                                 double* re, double* im) {
    if ((x >> n) & 1ull) {
        *re = 0.0;
        *im = 0.0;
        return;
    }
    const uint64_t r = (x & ((1ull << n) - 1ull)) | ((x >> (n + 1)) << n);
    double s, c;
    sincos_turn(sm64_uniform(seed, r), &s, &c);      // phi = 2 pi u
    *re = c * scale;
    *im = s * scale;
}

// Amplitude of basis state x of the product state: site n up, every other
// site l in (|down> + exp(-i phi_l)|up>)/sqrt(2) with phi_l = 2 pi u(seed, l),
// so psi[x] = 2^-(M-1)/2 exp(-i 2 pi sum of u(seed, l) over the up sites l != n).
// `u` holds u(seed, l) for l < M (or is null: drawn here).
__device__ __forceinline__ void product_amp(uint64_t x, int M, int n, uint64_t seed,
                                            const double* u, double scale, double* re,
                                            double* im) {
    if ((x >> n) & 1ull) {
        *re = 0.0;
        *im = 0.0;
        return;
    }
    double acc = 0.0;
    for (int l = 0; l < M; ++l)
        if (l != n && !((x >> l) & 1ull)) acc += u ? u[l] : sm64_uniform(seed, uint64_t(l));
    acc -= floor(acc);               // the phase modulo 2 pi
    double s, c;
    sincos_turn(acc, &s, &c);
    *re = c * scale;
    *im = -s * scale;
}

// Initial amplitude of basis state x: init 1 = the random-phase state,
// init 2 = the basis state |seed> (one ensemble member of Eq. (1)), init 3 =
// the product state of the random phases of `seed`.
__device__ __forceinline__ void init_amp(uint64_t x, int M, int init, int polarized, uint64_t seed,
                                         double scale, double* re, double* im) {
    if (init == 2) {
        *re = x == seed ? 1.0 : 0.0;
        *im = 0.0;
    } else if (init == 3) {
        product_amp(x, M, polarized, seed, nullptr, scale, re, im);
    } else {
        random_phase_amp(x, polarized, seed, scale, re, im);
    }
}

// Both initial states hold zeros where site n is down, so a lane takes V
// consecutive free indices r (the bits of x but n) and stores their amplitudes
// and as many zeros, 16 bytes at a time; the phase generator alone would
// otherwise idle half of every wavefront's lanes.  The stride is a power of
// two, so the bits of r below it, and their part of the product state's phase,
// are the lane's for good.  M = 28, site 0 / 5, with the reduction of the
// phase above: random phases, complex64 766 / 720 -> 440 / 384 us (a fill takes
// 316), complex128 842 / 787 -> 750 / 737; product state, complex64 2048 / 2044
// -> 427 / 400, complex128 2037 / 2026 -> 870 / 766.  What is left above the
// fill is the FP64 series and the generator's 64-bit products.
template <typename T, bool PRODUCT>
__global__ __launch_bounds__(256) void k_init(typename CT<T>::c* __restrict__ psi, int M, int n,
                                              uint64_t seed, double scale) {
    using C = typename CT<T>::c;
    constexpr int V = CT<T>::V;
    __shared__ double u[64];
    if constexpr (PRODUCT) {
        if (threadIdx.x < 64) u[threadIdx.x] = sm64_uniform(seed, threadIdx.x);
        __syncthreads();
    }
    const uint64_t nfree = 1ull << (M - 1);
    const uint64_t stride = uint64_t(gridDim.x) * 256 * V, low = (1ull << n) - 1;
    uint64_t r = (uint64_t(blockIdx.x) * 256 + threadIdx.x) * V;
    const int lb = min(M - 1, 63 - __builtin_clzll(stride));      // bits of r below the stride
    double acc[V];
#pragma unroll
    for (int j = 0; j < V; ++j) {
        acc[j] = 0.0;
        if constexpr (PRODUCT)
            for (int b = 0; b < lb; ++b)
                if (!(((r + j) >> b) & 1ull)) acc[j] += u[b + (b >= n)];
    }
    for (; r < nfree; r += stride) {
        const uint64_t x = ((r & ~low) << 1) | (r & low);
        C v[V];
#pragma unroll
        for (int j = 0; j < V; ++j) {
            double sn, cs;
            if constexpr (PRODUCT) {
                double a = acc[j];
                for (int b = lb; b < M - 1; ++b)
                    if (!((r >> b) & 1ull)) a += u[b + (b >= n)];
                sincos_turn(a - floor(a), &sn, &cs);     // the phase modulo 2 pi
                sn = -sn;
            } else {
                sincos_turn(sm64_uniform(seed, r + j), &sn, &cs);
            }
            v[j].x = T(cs * scale);
            v[j].y = T(sn * scale);
        }
        if constexpr (V == 1) {
            psi[x] = v[0];
            psi[x | (1ull << n)] = C{};
        } else if (n == 0) {
            // x = 2 r: every amplitude has its zero beside it
            float4* out = reinterpret_cast<float4*>(psi) + r;
            out[0] = float4{v[0].x, v[0].y, 0.f, 0.f};
            if (r + 1 < nfree) out[1] = float4{v[1].x, v[1].y, 0.f, 0.f};
        } else {
            *reinterpret_cast<float4*>(psi + x) = float4{v[0].x, v[0].y, v[1].x, v[1].y};
            *reinterpret_cast<float4*>(psi + (x | (1ull << n))) = float4{};
        }
    }
}

// Amplitude of ensemble member r's basis state: 1, or in single precision a
// point of the unit circle at a phase of the member's own, which no observable
// sees.  With 1 in all of them the first factors round every member alike, and
// the mean keeps that rounding (ladder 2x7, 100 steps: norm 6.3e-8 off from the
// first steps on, with phases 1.2e-8).  Of 8 neighbouring points in single
// precision the one closest to the circle is taken (|x^2 + y^2 - 1| 3e-9, seldom
// 4e-8), at 0.5 us per call.  A mean over fewer than 64 members gains nothing from
// independent roundings (1.5e-7 of the norm each): they all start with 1.
__device__ __forceinline__ double2 member_amp(uint64_t r, double) { return double2{1.0, 0.0}; }
__device__ __forceinline__ float2 member_amp(uint64_t r, float) {
    const int first = __float_as_int(float(fma(0.5, sm64_uniform(0, r), 0.4)));
    float2 best{1.f, 0.f};
    double least = 1.0;
#pragma unroll
    for (int k = 0; k < 8; ++k) {
        const float x = __int_as_float(first + k);
        const double y2 = 1.0 - double(x) * double(x);
        const float y = sqrtf(float(y2));        // or a neighbour of the nearest
        const double off = fabs(double(y) * double(y) - y2);
        if (off < least) {
            least = off;
            best = float2{x, y};
        }
    }
    return best;
}

// Ensemble members stacked as one state of M + cbits sites: amplitude
// x = (m << M) | y is member_amp when m < count and y is the basis state of member
// first + m (its bits spread over the sites other than `polarized`, whose
// bit is 0: spin up), and 0 otherwise.
template <typename T>
__global__ __launch_bounds__(256) void k_init_members(typename CT<T>::c* __restrict__ psi, int M,
                                                      int cbits, int polarized, uint64_t first,
                                                      uint64_t count, bool phases) {
    const uint64_t dim = 1ull << (M + cbits);
    const uint64_t ymask = (1ull << M) - 1;
    const uint64_t low = (1ull << polarized) - 1;
    const uint64_t stride = uint64_t(gridDim.x) * blockDim.x;
    for (uint64_t x = uint64_t(blockIdx.x) * blockDim.x + threadIdx.x; x < dim; x += stride) {
        const uint64_t m = x >> M;
        const uint64_t r = first + m;
        const uint64_t basis = ((r & ~low) << 1) | (r & low);
        typename CT<T>::c v;
        v.x = v.y = T(0);
        if (m < count && (x & ymask) == basis) {
            if (phases) v = member_amp(r, T(0));
            else v.x = T(1);
        }
        psi[x] = v;
    }
}

#if SPIN_PART == 0
// acc[i] = (acc[i] + add[i]) * scale (add may be null), i < n.
__global__ void k_accumulate(double* __restrict__ acc, const double* __restrict__ add, int64_t n,
                             double scale) {
    for (int64_t i = int64_t(blockIdx.x) * blockDim.x + threadIdx.x; i < n;
         i += int64_t(gridDim.x) * blockDim.x)
        acc[i] = (acc[i] + (add ? add[i] : 0.0)) * scale;
}
#endif

// ---------------------------------------------------------- reductions
__device__ __forceinline__ double wave_sum(double v) {
#pragma unroll
    for (int off = 32; off >= 1; off >>= 1) v += __shfl_xor(v, off, 64);
    return v;
}

// Sum of (p, n) over the workgroup, fixed order; result valid in thread 0.
template <int NT>
__device__ __forceinline__ void block_sum2(double& p, double& n, double* red) {
    p = wave_sum(p);
    n = wave_sum(n);
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    if (lane == 0) {
        red[2 * wave] = p;
        red[2 * wave + 1] = n;
    }
    __syncthreads();
    if (threadIdx.x == 0) {
        double sp = 0.0, sn = 0.0;
        for (int w = 0; w < (NT + 63) / 64; ++w) {
            sp += red[2 * w];
            sn += red[2 * w + 1];
        }
        p = sp;
        n = sn;
    }
    __syncthreads();
}

// Workgroup sum of v (result valid in thread 0).
template <int NT>
__device__ __forceinline__ double block_sum1(double v, double* red) {
    v = wave_sum(v);
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    if (lane == 0) red[wave] = v;
    __syncthreads();
    double s = 0.0;
    if (threadIdx.x == 0)
        for (int w = 0; w < (NT + 63) / 64; ++w) s += red[w];
    __syncthreads();
    return s;
}

#if SPIN_PART == 0
// Profile partials [slot][nwg][M + 1] -> Pall[s * M + site], N[s]; one
// workgroup per (step, site or norm).
__global__ __launch_bounds__(256) void k_reduce_profile(const double* __restrict__ partials, int nwg,
                                                        int ch, int M, int64_t s0,
                                                        double* __restrict__ Pall,
                                                        double* __restrict__ N) {
    __shared__ double red[8];
    const int64_t s = s0 + blockIdx.x / (M + 1);
    const int site = int(blockIdx.x % (M + 1));
    const double* src = partials + (size_t)(s % ch) * nwg * (M + 1);
    double v = 0.0;
    for (int w = threadIdx.x; w < nwg; w += 256) v += src[(size_t)w * (M + 1) + site];
    v = block_sum1<256>(v, red);
    if (threadIdx.x == 0) {
        if (site < M) Pall[s * M + site] = v;
        else if (N) N[s] = v;
    }
}

// partials: [slot][nwg][2]; P/N for steps s0..s1-1, slot = s % ch.
template <int NT>
__global__ __launch_bounds__(NT) void k_reduce(const double* __restrict__ partials, int nwg, int ch,
                                                int64_t s0, double* __restrict__ P,
                                                double* __restrict__ N) {
    __shared__ double red[2 * (NT / 64)];
    const int64_t s = s0 + blockIdx.x;
    const double* base = partials + (size_t)(s % ch) * nwg * 2;
    double p = 0.0, n = 0.0;
    for (int w = threadIdx.x; w < nwg; w += NT) {
        p += base[2 * w];
        n += base[2 * w + 1];
    }
    block_sum2<NT>(p, n, red);
    if (threadIdx.x == 0) {
        P[s] = p;
        if (N) N[s] = n;
    }
}
#endif

// Reads the state once, so the loads in flight bound it: U = 4 16-byte loads per
// lane, a workgroup's 16 KiB contiguous.  M = 28: complex64 572 -> 348 us (6.2
// TB/s), complex128 738 -> 692 us; the same four loads a whole grid apart 412
// and 814 us.  complex128 states that stay in the last-level cache (256 MiB, M =
// 24) are read one load at a time: 40.9 us against 42.5, M = 23 23.1 against
// 23.6, M = 25 89.0 against 90.0, M = 26 176 against 175 (complex64 is faster
// with four at every size).
template <typename T, int U>
__global__ __launch_bounds__(256) void k_observe(const typename CT<T>::c* __restrict__ psi, int M,
                                                 int site, double* __restrict__ partials) {
    using Vec = typename CT<T>::v;
    constexpr int V = CT<T>::V;
    __shared__ double red[8];
    const Vec* __restrict__ in = reinterpret_cast<const Vec*>(psi);
    const uint64_t nvec = (1ull << M) / V;
    const uint64_t stride = uint64_t(gridDim.x) * 256;
    double p = 0.0, n = 0.0;
    auto add = [&](const Vec& v, uint64_t x) {
        double w = double(v.x) * double(v.x) + double(v.y) * double(v.y), d = w;
        if constexpr (V == 2) {
            const double w1 = double(v.z) * double(v.z) + double(v.w) * double(v.w);
            d = site == 0 ? w - w1 : w + w1;
            w += w1;
        }
        n += w;
        p += ((x * V) >> site) & 1ull ? -d : d;
    };
    for (uint64_t x = uint64_t(blockIdx.x) * 256 * U + threadIdx.x; x < nvec; x += U * stride) {
        Vec v[U];
#pragma unroll
        for (int k = 0; k < U; ++k) v[k] = x + k * 256 < nvec ? in[x + k * 256] : Vec{};
#pragma unroll
        for (int k = 0; k < U; ++k) add(v[k], x + k * 256);
    }
    block_sum2<256>(p, n, red);
    if (threadIdx.x == 0) {
        partials[2 * blockIdx.x] = p;
        partials[2 * blockIdx.x + 1] = n;
    }
}

// ------------------------------------------------------ unfused factor
// exp(-i tau H_ij) over the whole state; lane = one anti-aligned pair.
template <typename T>
__global__ __launch_bounds__(256) void k_factor(typename CT<T>::c* __restrict__ psi, int M, int lo,
                                                int hi, T t, T s, T pr, T pim, int zz) {
    using C = typename CT<T>::c;
    const uint64_t npairs = 1ull << (M - 2);
    const uint64_t stride = uint64_t(gridDim.x) * 256;
    for (uint64_t p = uint64_t(blockIdx.x) * 256 + threadIdx.x; p < npairs; p += stride) {
        uint64_t x = p;
        x = ((x >> lo) << (lo + 1)) | (x & ((1ull << lo) - 1ull));
        x = ((x >> hi) << (hi + 1)) | (x & ((1ull << hi) - 1ull));
        const uint64_t xa = x | (1ull << hi), xb = x | (1ull << lo);
        C a = psi[xa], b = psi[xb];
        // (a_re, b_im) rotate by [[c, s], [-s, c]]; (a_im, b_re) by [[c, -s], [s, c]]
        T u = a.x, v = b.y;
        u = fma(t, v, u); v = fma(-s, u, v); u = fma(t, v, u);
        a.x = u; b.y = v;
        u = a.y; v = b.x;
        u = fma(-t, v, u); v = fma(s, u, v); u = fma(-t, v, u);
        a.y = u; b.x = v;
        if (zz) {
            C a2, b2;
            a2.x = pr * a.x - pim * a.y; a2.y = pr * a.y + pim * a.x;
            b2.x = pr * b.x - pim * b.y; b2.y = pr * b.y + pim * b.x;
            a = a2; b = b2;
            C c0 = psi[x], c1 = psi[x | (1ull << lo) | (1ull << hi)];
            C d0, d1;
            d0.x = pr * c0.x + pim * c0.y; d0.y = pr * c0.y - pim * c0.x;
            d1.x = pr * c1.x + pim * c1.y; d1.y = pr * c1.y - pim * c1.x;
            psi[x] = d0;
            psi[x | (1ull << lo) | (1ull << hi)] = d1;
        }
        psi[xa] = a;
        psi[xb] = b;
    }
}

// ------------------------------------------------------- register ops
// Rotation of the anti-aligned pairs (bit A, bit B) = (0, 1) <-> (1, 0) of
// the register index: psi_x <- c psi_x - i s psi_y, psi_y <- -i s psi_x + c psi_y,
// done as two real three-shear rotations (exactly area preserving):
// (Re x, Im y) by [[c, s], [-s, c]] and (Im x, Re y) by [[c, -s], [s, c]],
// each as u += t v; v -= s u; u += t v with t = tan(theta/2).
template <int R, int A, int B, typename C, typename T>
__device__ __forceinline__ void reg_xy(C (&v)[1 << R], T t, T s) {
#pragma unroll
    for (int j = 0; j < (1 << R); ++j) {
        if (((j >> A) & 1) == 0 && ((j >> B) & 1) == 1) {
            const int k = j ^ (1 << A) ^ (1 << B);
            T u = v[j].x, w = v[k].y;
            u = fma(t, w, u); w = fma(-s, u, w); u = fma(t, w, u);
            v[j].x = u; v[k].y = w;
            u = v[j].y; w = v[k].x;
            u = fma(-t, w, u); w = fma(s, u, w); u = fma(-t, w, u);
            v[j].y = u; v[k].x = w;
        }
    }
}

// a <- (pr + i pim) a for two amplitudes and b <- (pr - i pim) b for two
// others.  In asm so that each result lands in the register of its input: left
// to itself the compiler computes the 2^R amplitudes into other registers and
// copies them back, half as many instructions again.  Four at a time because
// the compiler puts a wait state between two blocks.
template <typename C>
__device__ __forceinline__ void phase_quad(C& a0, C& a1, C& b0, C& b1, float pr, float pim) {
    float w, u;
    asm("v_mul_f32 %8, %11, %1\n\tv_mul_f32 %9, %11, %0\n\t"
        "v_fma_f32 %0, %10, %0, -%8\n\tv_fma_f32 %1, %10, %1, %9\n\t"
        "v_mul_f32 %8, %11, %3\n\tv_mul_f32 %9, %11, %2\n\t"
        "v_fma_f32 %2, %10, %2, -%8\n\tv_fma_f32 %3, %10, %3, %9\n\t"
        "v_mul_f32 %8, %11, %5\n\tv_mul_f32 %9, %11, %4\n\t"
        "v_fma_f32 %4, %10, %4, %8\n\tv_fma_f32 %5, %10, %5, -%9\n\t"
        "v_mul_f32 %8, %11, %7\n\tv_mul_f32 %9, %11, %6\n\t"
        "v_fma_f32 %6, %10, %6, %8\n\tv_fma_f32 %7, %10, %7, -%9"
        : "+v"(a0.x), "+v"(a0.y), "+v"(a1.x), "+v"(a1.y), "+v"(b0.x), "+v"(b0.y), "+v"(b1.x), "+v"(b1.y),
          "=&v"(w), "=&v"(u)
        : "s"(pr), "s"(pim));
}
template <typename C>
__device__ __forceinline__ void phase_quad(C& a0, C& a1, C& b0, C& b1, double pr, double pim) {
    double w, u;
    asm("v_mul_f64 %8, %11, %1\n\tv_mul_f64 %9, %11, %0\n\t"
        "v_fma_f64 %0, %10, %0, -%8\n\tv_fma_f64 %1, %10, %1, %9\n\t"
        "v_mul_f64 %8, %11, %3\n\tv_mul_f64 %9, %11, %2\n\t"
        "v_fma_f64 %2, %10, %2, -%8\n\tv_fma_f64 %3, %10, %3, %9\n\t"
        "v_mul_f64 %8, %11, %5\n\tv_mul_f64 %9, %11, %4\n\t"
        "v_fma_f64 %4, %10, %4, %8\n\tv_fma_f64 %5, %10, %5, -%9\n\t"
        "v_mul_f64 %8, %11, %7\n\tv_mul_f64 %9, %11, %6\n\t"
        "v_fma_f64 %6, %10, %6, %8\n\tv_fma_f64 %7, %10, %7, -%9"
        : "+v"(a0.x), "+v"(a0.y), "+v"(a1.x), "+v"(a1.y), "+v"(b0.x), "+v"(b0.y), "+v"(b1.x), "+v"(b1.y),
          "=&v"(w), "=&v"(u)
        : "s"(pr), "s"(pim));
}

// I^z I^z phase: anti-aligned amplitudes times (pr + i pi), aligned times
// its conjugate.
template <int R, int A, int B, typename C, typename T>
__device__ __forceinline__ void reg_zz(C (&v)[1 << R], T pr, T pim) {
    constexpr int a = 1 << A, b = 1 << B;
#pragma unroll
    for (int j = 0; j < (1 << R); ++j)
        if ((j & (a | b)) == 0) phase_quad(v[j | a], v[j | b], v[j], v[j | a | b], pr, pim);
}

// One op of a stage without register/lane exchanges.
template <int R, typename C, typename T>
__device__ __forceinline__ void reg_op(C (&v)[1 << R], int code, T t, T s) {
#define SPIN_CASE(A, B)                                        \
    case op_xy(A, B):                                          \
        if constexpr (B < R) reg_xy<R, A, B>(v, t, s);         \
        break;                                                 \
    case op_zz(A, B):                                          \
        if constexpr (B < R) reg_zz<R, A, B>(v, t, s);         \
        break;
    switch (code) {
        SPIN_CASE(0, 1) SPIN_CASE(0, 2) SPIN_CASE(1, 2) SPIN_CASE(0, 3) SPIN_CASE(1, 3)
        SPIN_CASE(2, 3) SPIN_CASE(0, 4) SPIN_CASE(1, 4) SPIN_CASE(2, 4) SPIN_CASE(3, 4)
        SPIN_CASE(0, 5) SPIN_CASE(1, 5) SPIN_CASE(2, 5) SPIN_CASE(3, 5) SPIN_CASE(4, 5)
        default: break;
    }
#undef SPIN_CASE
}

// sum of (sign * |psi|^2, |psi|^2) over the lane's registers, FP64
template <int R, typename C>
__device__ __forceinline__ void reg_observe(const C (&v)[1 << R], int sign, int mask, double& p,
                                            double& n) {
#pragma unroll
    for (int j = 0; j < (1 << R); ++j) {
        const double w = double(v[j].x) * double(v[j].x) + double(v[j].y) * double(v[j].y);
        n += w;
        const int neg = sign ^ ((j & mask) ? 1 : 0);
        p += neg ? -w : w;
    }
}

// LDS byte address of the lane's register 0 at the entry of stage S, over its
// NTB thread bits (offsets past the stage's own thread bits are zero).
template <int NTB>
__device__ __forceinline__ uint32_t stage_base(const DevStage& S, int tid) {
    uint32_t b = 0;
#pragma unroll
    for (int q = 0; q < NTB; ++q) b ^= S.tmask[q] & (0u - ((uint32_t(tid) >> q) & 1u));
    return b;
}

// Barrier for LDS traffic only: global loads in flight (the next tile's
// prefetch) stay in flight across it.
__device__ __forceinline__ void lds_barrier() {
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup", "local");
    __builtin_amdgcn_s_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "workgroup", "local");
}

// Ordering of a wave's own LDS scatter before its gather: the exchange
// moves amplitudes only between lanes of the wave, so no other wave reads
// the slots (LDS operations of one wave complete in issue order; the fences
// keep the compiler from moving the gather above the scatter).
__device__ __forceinline__ void wave_lds_sync() {
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront", "local");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront", "local");
}

// Deposit of the bits of `x` into the set bits of `mask`, lowest first.
__device__ __forceinline__ int64_t deposit(int64_t x, int64_t mask) {
    int64_t out = 0;
    while (x && mask) {
        const int64_t low = mask & -mask;
        if (x & 1) out |= low;
        mask ^= low;
        x >>= 1;
    }
    return out;
}

// Next value, in increasing order, among the submasks of `mask`.
__device__ __forceinline__ int64_t next_submask(int64_t cur, int64_t mask) {
    return ((cur | ~mask) + 1) & mask;
}

// Gather / scatter of a lane's 2^R registers in Gray-code order: register
// j = i ^ (i >> 1) sits at pb ^ (xor of rbit[q] over the set bits q of j),
// and consecutive Gray codes differ in bit ctz(i).
template <int R, typename C, typename Stage>
__device__ __forceinline__ void gather(C (&v)[1 << R], const char* lds, uint32_t pb,
                                       const Stage& S) {
    uint32_t a = pb;
    v[0] = *reinterpret_cast<const C*>(lds + a);
#pragma unroll
    for (int i = 1; i < (1 << R); ++i) {
        a ^= S.rbit[__builtin_ctz(i)];
        v[i ^ (i >> 1)] = *reinterpret_cast<const C*>(lds + a);
    }
}

template <int R, typename C, typename Stage>
__device__ __forceinline__ void scatter(const C (&v)[1 << R], char* lds, uint32_t pb,
                                        const Stage& S) {
    uint32_t a = pb;
    *reinterpret_cast<C*>(lds + a) = v[0];
#pragma unroll
    for (int i = 1; i < (1 << R); ++i) {
        a ^= S.rbit[__builtin_ctz(i)];
        *reinterpret_cast<C*>(lds + a) = v[i ^ (i >> 1)];
    }
}

// Exchange of 2^RW of a lane's registers, H * 2^RW and up (H: the half of a
// half-tile exchange, 0 otherwise).  Scatter: register i goes to row i, a
// constant offset from the lane's own slot.  Gather: Gray-code order over the
// RW register bits, one add or subtract per register.
template <int RW, int H, int ROW, typename C, int NR>
__device__ __forceinline__ void scatter_rows(const C (&v)[NR], char* own) {
#pragma unroll
    for (int i = 0; i < (1 << RW); ++i) *reinterpret_cast<C*>(own + i * ROW) = v[(H << RW) + i];
}

template <int RW, int H, typename C, int NR>
__device__ __forceinline__ void gather_rows(C (&v)[NR], const char* lds, uint32_t a, const uint32_t (&w)[RW]) {
    v[H << RW] = *reinterpret_cast<const C*>(lds + a);
#pragma unroll
    for (int i = 1; i < (1 << RW); ++i) {
        const int b = __builtin_ctz(i), j = i ^ (i >> 1);
        a = (j >> b) & 1 ? a + w[b] : a - w[b];
        v[(H << RW) + j] = *reinterpret_cast<const C*>(lds + a);
    }
}

// Register offsets of a stage read into scalar registers together with its
// lane offsets (one round trip for both before the gather).
template <int R>
struct RegBits {
    uint32_t rbit[R];
};

// An op record in the constant address space: with a pointer that steps
// through the table the compiler would otherwise use vector loads.
template <typename T>
using ConstOp = const __attribute__((address_space(4))) DevOp<T>;

template <typename T>
__device__ __forceinline__ ConstOp<T>* const_ops(const DevOp<T>* p) {
    return (ConstOp<T>*)(p);
}

// Runs a stage's ops from `op` up to the next observable, matrix or end
// record; returns that record and its code.  Each record is loaded one op
// ahead: the scalar load's latency hides behind the current op's arithmetic.
__device__ __forceinline__ bool leaves_loop(int code) { return (code & ~3) == kOpEnd; }

template <int R, typename C, typename T>
__device__ __forceinline__ ConstOp<T>* run_factors(C (&v)[1 << R], ConstOp<T>* op, int& code) {
    int c = op->code;
    T t = op->t, s = op->s;
    // The first record and the gathered registers have arrived before the loop:
    // otherwise every op waits for them there, and so for the next record's
    // load too.
    asm volatile("" ::"s"(t), "s"(s));
    while (!leaves_loop(c)) {
        ++op;
        const int cn = op->code;
        const T tn = op->t, sn = op->s;
        reg_op<R>(v, c, t, s);
        c = cn;
        t = tn;
        s = sn;
    }
    code = c;
    return op;
}

// ------------------------------------------------------- threaded op loop
// The same loop for stages with register/lane exchanges, in assembly: every
// handler sits at (op code << spS) behind .Lspin_ops and ends by jumping to the
// next op's.  Compiled from C++ (a switch), an op cost a tree of compares and
// four or five taken branches, about 310 clocks beside 24 to 48 FMAs when no
// other wave of the SIMD could fill them (2^12-amplitude tiles, M = 18: 20.5 us
// per pass of 50 factors and 21 exchanges); the jump costs about 80.  The
// registers are pinned: amplitude j of complex64 is v[spV + 2j] (re) and
// v[spV + 2j + 1] (im), complex128 takes two registers each.
//
// Scalars: s[72:79] the op's parameters, s[80:88] the next record (loaded when
// the op starts, waited for before the jump), s[90:91] .Lspin_ops, s[92:93] the
// jump's target, s[94:95] the record's address.  Handlers: op_xy does the
// three shears of reg_xy, each over all pairs before the next (a dependent FMA
// is 2^(R-1) instructions away); op_gate one v_permlane16/32_swap per 32-bit
// register pair, which trades the rows of its first operand that have the lane
// bit set for the rows of the second that have it clear; op_zz the phase of
// reg_zz.  At least the seven scalar instructions of the jump separate two
// handlers' vector instructions, more than the wait states a swap needs after
// a write of its operands.  A handler longer than its slots is an assembler
// error (.org backwards).
#define SPIN_ASM_COMMON                                            \
    ".set spR, %c[r]\n"                                            \
    ".set spN, 1<<spR\n"                                           \
    ".set spV, %c[vb]\n"                                           \
    ".set spS, %c[sh]\n"                                           \
    ".macro spin_slot n\n"                                         \
    ".org .Lspin_ops_%= + ((\\n)<<spS)\n"                          \
    ".endm\n"                                                      \
    ".macro spin_handler_xy a b\n"                                 \
    ".if \\b < spR\n"                                              \
    "spin_slot (\\b*(\\b-1)/2+\\a)\n"                              \
    "spin_head\n"                                                  \
    "spin_shear \\a \\b 1\n"                                       \
    "spin_shear \\a \\b 2\n"                                       \
    "spin_shear \\a \\b 1\n"                                       \
    "spin_next\n"                                                  \
    ".endif\n"                                                     \
    ".endm\n"                                                      \
    ".macro spin_handler_gate q\n"                                 \
    ".if \\q < spR\n"                                              \
    "spin_slot (16+2*\\q)\n"                                       \
    "spin_head\n"                                                  \
    "spin_swap \\q v_permlane16_swap_b32\n"                        \
    "spin_next\n"                                                  \
    "spin_slot (17+2*\\q)\n"                                       \
    "spin_head\n"                                                  \
    "spin_swap \\q v_permlane32_swap_b32\n"                        \
    "spin_next\n"                                                  \
    ".endif\n"                                                     \
    ".endm\n"                                                      \
    ".macro spin_handler_zz a b\n"                                 \
    ".if \\b < spR\n"                                              \
    "spin_slot (32+4*(\\b*(\\b-1)/2+\\a))\n"                       \
    "spin_head\n"                                                  \
    "spin_phase \\a \\b\n"                                         \
    "spin_next\n"                                                  \
    ".endif\n"                                                     \
    ".endm\n"
#define SPIN_ASM_RUN                                               \
    "s_mov_b64 s[94:95], %[op]\n"                                  \
    "s_getpc_b64 s[90:91]\n"                                       \
    ".Lspin_pc_%=:\n"                                              \
    "s_add_u32 s90, s90, .Lspin_ops_%=-.Lspin_pc_%=\n"             \
    "s_addc_u32 s91, s91, 0\n"                                     \
    "spin_load\n"                                                  \
    "spin_next\n"                                                  \
    ".p2align 6\n"                                                 \
    ".Lspin_ops_%=:\n"                                             \
    "spin_handler_xy 0 1\n"                                        \
    "spin_handler_xy 0 2\nspin_handler_xy 1 2\n"                   \
    "spin_handler_xy 0 3\nspin_handler_xy 1 3\nspin_handler_xy 2 3\n" \
    "spin_handler_xy 0 4\nspin_handler_xy 1 4\nspin_handler_xy 2 4\nspin_handler_xy 3 4\n" \
    "spin_handler_xy 0 5\nspin_handler_xy 1 5\nspin_handler_xy 2 5\nspin_handler_xy 3 5\nspin_handler_xy 4 5\n" \
    "spin_handler_gate 0\nspin_handler_gate 1\nspin_handler_gate 2\n" \
    "spin_handler_gate 3\nspin_handler_gate 4\nspin_handler_gate 5\n" \
    "spin_slot 28\ns_branch .Lspin_end_%=\n"                       \
    "spin_slot 29\ns_branch .Lspin_end_%=\n"                       \
    "spin_handler_zz 0 1\n"                                        \
    "spin_handler_zz 0 2\nspin_handler_zz 1 2\n"                   \
    "spin_handler_zz 0 3\nspin_handler_zz 1 3\nspin_handler_zz 2 3\n" \
    "spin_handler_zz 0 4\nspin_handler_zz 1 4\nspin_handler_zz 2 4\nspin_handler_zz 3 4\n" \
    "spin_handler_zz 0 5\nspin_handler_zz 1 5\nspin_handler_zz 2 5\nspin_handler_zz 3 5\nspin_handler_zz 4 5\n" \
    ".Lspin_end_%=:\n"                                             \
    "s_mov_b64 %[op], s[94:95]\n"                                  \
    ".purgem spin_slot\n.purgem spin_handler_xy\n.purgem spin_handler_gate\n.purgem spin_handler_zz\n" \
    ".purgem spin_head\n.purgem spin_load\n.purgem spin_next\n"    \
    ".purgem spin_shear\n.purgem spin_swap\n.purgem spin_phase\n"
#define SPIN_ASM_F32                                               \
    SPIN_ASM_COMMON                                                \
    ".macro spin_load\n"                                           \
    "s_load_dwordx8 s[80:87], s[94:95], 0x0\n"                     \
    ".endm\n"                                                      \
    ".macro spin_head\n"                                           \
    "s_add_u32 s94, s94, 32\n"                                     \
    "s_addc_u32 s95, s95, 0\n"                                     \
    "spin_load\n"                                                  \
    ".endm\n"                                                      \
    ".macro spin_next\n"                                           \
    "s_waitcnt lgkmcnt(0)\n"                                       \
    "s_lshl_b32 s92, s84, spS\n"                                   \
    "s_mov_b64 s[72:73], s[80:81]\n"                               \
    "s_mov_b64 s[74:75], s[82:83]\n"                               \
    "s_add_u32 s92, s92, s90\n"                                    \
    "s_addc_u32 s93, s91, 0\n"                                     \
    "s_setpc_b64 s[92:93]\n"                                       \
    ".endm\n"                                                      \
    ".macro spin_shear a b ph\n"                                   \
    ".set spj, 0\n"                                                \
    ".rept spN\n"                                                  \
    ".if (((spj>>\\a)&1)==0)&&(((spj>>\\b)&1)==1)\n"               \
    ".set spk, spj^(1<<\\a)^(1<<\\b)\n"                            \
    ".if \\ph == 2\n"                                              \
    "v_fmac_f32 v[spV+2*spk+1], s75, v[spV+2*spj]\n"               \
    "v_fmac_f32 v[spV+2*spk], s73, v[spV+2*spj+1]\n"               \
    ".else\n"                                                      \
    "v_fmac_f32 v[spV+2*spj], s72, v[spV+2*spk+1]\n"               \
    "v_fmac_f32 v[spV+2*spj+1], s74, v[spV+2*spk]\n"               \
    ".endif\n"                                                     \
    ".endif\n"                                                     \
    ".set spj, spj+1\n"                                            \
    ".endr\n"                                                      \
    ".endm\n"                                                      \
    ".macro spin_swap q op\n"                                      \
    ".set spj, 0\n"                                                \
    ".rept spN\n"                                                  \
    ".if ((spj>>\\q)&1)==0\n"                                      \
    ".set spk, spj|(1<<\\q)\n"                                     \
    "\\op v[spV+2*spj], v[spV+2*spk]\n"                            \
    "\\op v[spV+2*spj+1], v[spV+2*spk+1]\n"                        \
    ".endif\n"                                                     \
    ".set spj, spj+1\n"                                            \
    ".endr\n"                                                      \
    ".endm\n"                                                      \
    ".macro spin_phase a b\n"                                      \
    ".set spj, 0\n"                                                \
    ".rept spN/2\n"                                                \
    "v_mul_f32 %[w0], s73, v[spV+2*spj+1]\n"                       \
    "v_mul_f32 %[u0], s73, v[spV+2*spj]\n"                         \
    "v_mul_f32 %[w1], s73, v[spV+2*spj+3]\n"                       \
    "v_mul_f32 %[u1], s73, v[spV+2*spj+2]\n"                       \
    ".if ((spj>>\\a)^(spj>>\\b))&1\n"                              \
    "v_fma_f32 v[spV+2*spj], s72, v[spV+2*spj], -%[w0]\n"          \
    "v_fma_f32 v[spV+2*spj+1], s72, v[spV+2*spj+1], %[u0]\n"       \
    ".else\n"                                                      \
    "v_fma_f32 v[spV+2*spj], s72, v[spV+2*spj], %[w0]\n"           \
    "v_fma_f32 v[spV+2*spj+1], s72, v[spV+2*spj+1], -%[u0]\n"      \
    ".endif\n"                                                     \
    ".if (((spj+1)>>\\a)^((spj+1)>>\\b))&1\n"                      \
    "v_fma_f32 v[spV+2*spj+2], s72, v[spV+2*spj+2], -%[w1]\n"      \
    "v_fma_f32 v[spV+2*spj+3], s72, v[spV+2*spj+3], %[u1]\n"       \
    ".else\n"                                                      \
    "v_fma_f32 v[spV+2*spj+2], s72, v[spV+2*spj+2], %[w1]\n"       \
    "v_fma_f32 v[spV+2*spj+3], s72, v[spV+2*spj+3], -%[u1]\n"      \
    ".endif\n"                                                     \
    ".set spj, spj+2\n"                                            \
    ".endr\n"                                                      \
    ".endm\n"                                                      \
    SPIN_ASM_RUN                                                   \
    "s_mov_b32 %[code], s84\n"
#define SPIN_F64(n) "v[spV+4*" n ":spV+4*" n "+1]"
#define SPIN_G64(n) "v[spV+4*" n "+2:spV+4*" n "+3]"
#define SPIN_ASM_F64                                               \
    SPIN_ASM_COMMON                                                \
    ".macro spin_load\n"                                           \
    "s_load_dwordx8 s[80:87], s[94:95], 0x0\n"                     \
    "s_load_dword s88, s[94:95], 0x20\n"                           \
    ".endm\n"                                                      \
    ".macro spin_head\n"                                           \
    "s_add_u32 s94, s94, 48\n"                                     \
    "s_addc_u32 s95, s95, 0\n"                                     \
    "spin_load\n"                                                  \
    ".endm\n"                                                      \
    ".macro spin_next\n"                                           \
    "s_waitcnt lgkmcnt(0)\n"                                       \
    "s_lshl_b32 s92, s88, spS\n"                                   \
    "s_mov_b64 s[72:73], s[80:81]\n"                               \
    "s_mov_b64 s[74:75], s[82:83]\n"                               \
    "s_mov_b64 s[76:77], s[84:85]\n"                               \
    "s_mov_b64 s[78:79], s[86:87]\n"                               \
    "s_add_u32 s92, s92, s90\n"                                    \
    "s_addc_u32 s93, s91, 0\n"                                     \
    "s_setpc_b64 s[92:93]\n"                                       \
    ".endm\n"                                                      \
    ".macro spin_shear a b ph\n"                                   \
    ".set spj, 0\n"                                                \
    ".rept spN\n"                                                  \
    ".if (((spj>>\\a)&1)==0)&&(((spj>>\\b)&1)==1)\n"               \
    ".set spk, spj^(1<<\\a)^(1<<\\b)\n"                            \
    ".if \\ph == 2\n"                                              \
    "v_fmac_f64 " SPIN_G64("spk") ", s[78:79], " SPIN_F64("spj") "\n" \
    "v_fmac_f64 " SPIN_F64("spk") ", s[74:75], " SPIN_G64("spj") "\n" \
    ".else\n"                                                      \
    "v_fmac_f64 " SPIN_F64("spj") ", s[72:73], " SPIN_G64("spk") "\n" \
    "v_fmac_f64 " SPIN_G64("spj") ", s[76:77], " SPIN_F64("spk") "\n" \
    ".endif\n"                                                     \
    ".endif\n"                                                     \
    ".set spj, spj+1\n"                                            \
    ".endr\n"                                                      \
    ".endm\n"                                                      \
    ".macro spin_swap q op\n"                                      \
    ".set spj, 0\n"                                                \
    ".rept spN\n"                                                  \
    ".if ((spj>>\\q)&1)==0\n"                                      \
    ".set spk, spj|(1<<\\q)\n"                                     \
    "\\op v[spV+4*spj], v[spV+4*spk]\n"                            \
    "\\op v[spV+4*spj+1], v[spV+4*spk+1]\n"                        \
    "\\op v[spV+4*spj+2], v[spV+4*spk+2]\n"                        \
    "\\op v[spV+4*spj+3], v[spV+4*spk+3]\n"                        \
    ".endif\n"                                                     \
    ".set spj, spj+1\n"                                            \
    ".endr\n"                                                      \
    ".endm\n"                                                      \
    ".macro spin_phase a b\n"                                      \
    ".set spj, 0\n"                                                \
    ".rept spN\n"                                                  \
    "v_mul_f64 %[w0], s[74:75], " SPIN_G64("spj") "\n"             \
    "v_mul_f64 %[u0], s[74:75], " SPIN_F64("spj") "\n"             \
    ".if ((spj>>\\a)^(spj>>\\b))&1\n"                              \
    "v_fma_f64 " SPIN_F64("spj") ", s[72:73], " SPIN_F64("spj") ", -%[w0]\n" \
    "v_fma_f64 " SPIN_G64("spj") ", s[72:73], " SPIN_G64("spj") ", %[u0]\n"  \
    ".else\n"                                                      \
    "v_fma_f64 " SPIN_F64("spj") ", s[72:73], " SPIN_F64("spj") ", %[w0]\n"  \
    "v_fma_f64 " SPIN_G64("spj") ", s[72:73], " SPIN_G64("spj") ", -%[u0]\n" \
    ".endif\n"                                                     \
    ".set spj, spj+1\n"                                            \
    ".endr\n"                                                      \
    ".endm\n"                                                      \
    SPIN_ASM_RUN                                                   \
    "s_mov_b32 %[code], s88\n"
#define SPIN_CLOBBERS_F32                                                                               \
    "s72", "s73", "s74", "s75", "s80", "s81", "s82", "s83", "s84", "s85", "s86", "s87", "s90", "s91",   \
        "s92", "s93", "s94", "s95", "scc", "memory"
#define SPIN_CLOBBERS_F64 "s76", "s77", "s78", "s79", "s88", SPIN_CLOBBERS_F32

typedef float v8f __attribute__((ext_vector_type(8)));
typedef float v16f __attribute__((ext_vector_type(16)));
typedef float v32f __attribute__((ext_vector_type(32)));
typedef double v8d __attribute__((ext_vector_type(8)));
typedef double v16d __attribute__((ext_vector_type(16)));

// Handler slots of 2^shift bytes: the shears of 2^R registers or the swaps (4
// bytes each) and up to 60 bytes of scalars.
constexpr int op_slot_shift(int R) { return R <= 3 ? 7 : R == 4 ? 8 : 9; }

template <int R, typename T>
__device__ __forceinline__ ConstOp<T>* run_ops(typename CT<T>::c (&v)[1 << R], ConstOp<T>* op, int& code) {
    constexpr int NV = 2 << R;                                   // reals
    constexpr int W = NV * int(sizeof(T) / 4);                   // registers
    constexpr int VB = W <= 64 ? 64 : 128;
    constexpr int SH = op_slot_shift(R);
    constexpr int N = W < 32 ? NV : 32 / int(sizeof(T) / 4);     // reals of one operand
    auto get = [&](int i) { return i & 1 ? v[i / 2].y : v[i / 2].x; };
    auto put = [&](int i, T x) { if (i & 1) v[i / 2].y = x; else v[i / 2].x = x; };
    // uniform by construction; the compiler has to know it too
    const uint64_t q = reinterpret_cast<uint64_t>(op);
    uint64_t p = (uint64_t(uint32_t(__builtin_amdgcn_readfirstlane(int(uint32_t(q >> 32))))) << 32) |
                 uint32_t(__builtin_amdgcn_readfirstlane(int(uint32_t(q))));
    T w0, u0, w1, u1;
#define SPIN_RUN(TYPE, ...)                                                                      \
    asm volatile(SPIN_ASM_##TYPE : __VA_ARGS__, [op] "+s"(p), [code] "=&s"(code), [w0] "=&v"(w0),           \
                 [u0] "=&v"(u0), [w1] "=&v"(w1), [u1] "=&v"(u1)                                  \
                 : [r] "i"(R), [vb] "i"(VB), [sh] "i"(SH)                                        \
                 : SPIN_CLOBBERS_##TYPE)
#define SPIN_GET(X, B) _Pragma("unroll") for (int i = 0; i < N; ++i) X[i] = get((B) * N + i)
#define SPIN_PUT(X, B) _Pragma("unroll") for (int i = 0; i < N; ++i) put((B) * N + i, X[i])
    if constexpr (sizeof(T) == 4) {
        if constexpr (W == 8) {
            v8f a;
            SPIN_GET(a, 0);
            SPIN_RUN(F32, "+{v[64:71]}"(a));
            SPIN_PUT(a, 0);
        } else if constexpr (W == 16) {
            v16f a;
            SPIN_GET(a, 0);
            SPIN_RUN(F32, "+{v[64:79]}"(a));
            SPIN_PUT(a, 0);
        } else if constexpr (W == 32) {
            v32f a;
            SPIN_GET(a, 0);
            SPIN_RUN(F32, "+{v[64:95]}"(a));
            SPIN_PUT(a, 0);
        } else if constexpr (W == 64) {
            v32f a, b;
            SPIN_GET(a, 0); SPIN_GET(b, 1);
            SPIN_RUN(F32, "+{v[64:95]}"(a), "+{v[96:127]}"(b));
            SPIN_PUT(a, 0); SPIN_PUT(b, 1);
        } else {
            v32f a, b, c, d;
            SPIN_GET(a, 0); SPIN_GET(b, 1); SPIN_GET(c, 2); SPIN_GET(d, 3);
            SPIN_RUN(F32, "+{v[128:159]}"(a), "+{v[160:191]}"(b), "+{v[192:223]}"(c), "+{v[224:255]}"(d));
            SPIN_PUT(a, 0); SPIN_PUT(b, 1); SPIN_PUT(c, 2); SPIN_PUT(d, 3);
        }
    } else {
        if constexpr (W == 16) {
            v8d a;
            SPIN_GET(a, 0);
            SPIN_RUN(F64, "+{v[64:79]}"(a));
            SPIN_PUT(a, 0);
        } else if constexpr (W == 32) {
            v16d a;
            SPIN_GET(a, 0);
            SPIN_RUN(F64, "+{v[64:95]}"(a));
            SPIN_PUT(a, 0);
        } else if constexpr (W == 64) {
            v16d a, b;
            SPIN_GET(a, 0); SPIN_GET(b, 1);
            SPIN_RUN(F64, "+{v[64:95]}"(a), "+{v[96:127]}"(b));
            SPIN_PUT(a, 0); SPIN_PUT(b, 1);
        } else {
            v16d a, b, c, d;
            SPIN_GET(a, 0); SPIN_GET(b, 1); SPIN_GET(c, 2); SPIN_GET(d, 3);
            SPIN_RUN(F64, "+{v[128:159]}"(a), "+{v[160:191]}"(b), "+{v[192:223]}"(c), "+{v[224:255]}"(d));
            SPIN_PUT(a, 0); SPIN_PUT(b, 1); SPIN_PUT(c, 2); SPIN_PUT(d, 3);
        }
    }
#undef SPIN_RUN
#undef SPIN_GET
#undef SPIN_PUT
    return reinterpret_cast<ConstOp<T>*>(p);
}

// Weights of the exchange after a stage (see exchange_row_slots).
template <int RW, int NTB>
struct ExchangeWeights {
    uint32_t gr[RW], gw[NTB];
    int xnext;
    __device__ __forceinline__ void load(const DevStage& S) {
        xnext = S.xnext;
#pragma unroll
        for (int b = 0; b < RW; ++b) gr[b] = S.gr[b];
#pragma unroll
        for (int q = 0; q < NTB; ++q) gw[q] = S.gw[q];
    }
    // LDS byte address from which the lane gathers register 0.
    __device__ __forceinline__ uint32_t base(int tid) const {
        uint32_t a = 0;
#pragma unroll
        for (int q = 0; q < NTB; ++q) a += gw[q] & (0u - ((uint32_t(tid) >> q) & 1u));
        return a;
    }
};

// The exchange after a stage through per-lane slots (HALF: half 0 through the
// LDS, then half 1 through the same slots).  When both stages keep the same
// positions on the wave bits it moves amplitudes only within each wave and
// only the wave is ordered.  A lane scatters to slots of its own; after an
// exchange that crossed waves (prev_cross) other waves may still be gathering
// from them.
template <int R, int ROW, bool HALF, typename C, int RW, int NTB>
__device__ __forceinline__ void exchange(C (&v)[1 << R], char* ldsb, char* own, const ExchangeWeights<RW, NTB>& x,
                                         bool& prev_cross) {
    const bool xw = x.xnext != 0;
    auto sync = [&]() {
        if (xw) lds_barrier();
        else wave_lds_sync();
    };
    const uint32_t ga = x.base(threadIdx.x);
    if (prev_cross) lds_barrier();
    prev_cross = xw;
    scatter_rows<RW, 0, ROW>(v, own);
    sync();
    gather_rows<RW, 0>(v, ldsb, ga, x.gr);
    if constexpr (HALF) {
        sync();
        scatter_rows<RW, 1, ROW>(v, own);
        sync();
        gather_rows<RW, 1>(v, ldsb, ga, x.gr);
    }
}

// ------------------------------------------------------- matrix engine
// Dense 32 x 32 complex matrix U on the 32 registers of every lane, as the
// real product Y = W X with X = (Re v_0..Re v_31, Im v_0..Im v_31) per lane
// (column) and W = [[Re U, -Im U], [Im U, Re U]], on v_mfma_f32_32x32x2f32.
// A wave holds 64 columns.  One v_permlane32_swap per pair of rows (2p,
// 2p+1) turns the lane-per-column registers into the instruction's B
// operands (lane l: row 2p + l/32 of column 32h + l%32, h = 0, 1); the A
// operands are read from the matrix table (lane l: W[32b + l%32][2p + l/32]).
// The accumulators hold Y[32b + 8(r/4) + 4(l/32) + r%4][32h + l%32] in
// register r; one swap per register pair of h = 0, 1 returns them to the
// lane-per-column layout.
typedef float f32x16 __attribute__((ext_vector_type(16)));

template <typename C>
__device__ __forceinline__ float mat_row(const C (&v)[32], int m) {
    return m < 32 ? v[m].x : v[m - 32].y;
}
template <typename C>
__device__ __forceinline__ void mat_set(C (&v)[32], int m, float x) {
    if (m < 32) v[m].x = x;
    else v[m - 32].y = x;
}

template <typename C>
__device__ __forceinline__ void mfma_stage(C (&v)[32], const float* __restrict__ W) {
    const int lane = threadIdx.x & 63;
    float bop[64];
#pragma unroll
    for (int p = 0; p < 32; ++p) {
        const auto r = __builtin_amdgcn_permlane32_swap(__float_as_uint(mat_row(v, 2 * p)),
                                                        __float_as_uint(mat_row(v, 2 * p + 1)),
                                                        false, false);
        bop[2 * p] = __uint_as_float(r[0]);
        bop[2 * p + 1] = __uint_as_float(r[1]);
    }
    f32x16 d00 = {}, d01 = {}, d10 = {}, d11 = {};
#pragma unroll
    for (int p = 0; p < 32; ++p) {
        const float a0 = W[p * 64 + lane], a1 = W[(32 + p) * 64 + lane];
        d00 = __builtin_amdgcn_mfma_f32_32x32x2f32(a0, bop[2 * p], d00, 0, 0, 0);
        d01 = __builtin_amdgcn_mfma_f32_32x32x2f32(a0, bop[2 * p + 1], d01, 0, 0, 0);
        d10 = __builtin_amdgcn_mfma_f32_32x32x2f32(a1, bop[2 * p], d10, 0, 0, 0);
        d11 = __builtin_amdgcn_mfma_f32_32x32x2f32(a1, bop[2 * p + 1], d11, 0, 0, 0);
    }
#pragma unroll
    for (int r = 0; r < 16; ++r) {
        const int row = 8 * (r / 4) + r % 4;
        const auto s0 = __builtin_amdgcn_permlane32_swap(__float_as_uint(d00[r]), __float_as_uint(d01[r]),
                                                         false, false);
        mat_set(v, row, __uint_as_float(s0[0]));
        mat_set(v, row + 4, __uint_as_float(s0[1]));
        const auto s1 = __builtin_amdgcn_permlane32_swap(__float_as_uint(d10[r]), __float_as_uint(d11[r]),
                                                         false, false);
        mat_set(v, 32 + row, __uint_as_float(s1[0]));
        mat_set(v, 32 + row + 4, __uint_as_float(s1[1]));
    }
}

template <typename C>
__device__ __forceinline__ C& lds_at(char* lds, uint32_t byte) {
    return *reinterpret_cast<C*>(lds + byte);
}

// ------------------------------------------------------------ tiled pass
// One pass over the tiles of a group of G workgroups (G a power of two):
// member w takes the tiles whose index is w' + i*G (w' = w in the group's
// order), i = 0 .. tiles_per_member-1.  The first register stage of a tile
// is loaded straight from HBM (lanes along the low address bits, so the
// wave's accesses are contiguous runs) and the last one stored straight
// back, in the pass's output layout; the stages in between exchange through
// LDS, with a workgroup barrier where the exchange moves amplitudes between
// waves and a wave-level ordering where it does not.  Every wave has
// consumed its loads of a tile before the first workgroup barrier, so the
// stores after it cannot overtake another wave's loads; a pass without such
// a barrier keeps its wave positions and their address bits from the first
// stage to the last, so each wave stores only addresses it loaded itself.  A
// one-stage pass never touches LDS: its lanes store exactly the addresses
// they loaded (the planner only makes one-stage passes that keep the
// layout).  The next tile is prefetched into registers while
// the current one is worked on.  Observables accumulate into accP/accN per
// measurement slot of the pass.
// A lane's global accesses in Gray-code order over its register bits: the bits
// are disjoint, so a step adds or subtracts one (scalar) byte offset.
template <int R, typename C>
__device__ __forceinline__ void load_direct(C (&v)[1 << R], const C* __restrict__ psi, int64_t g,
                                            const int64_t* gr) {
    const char* a = reinterpret_cast<const char*>(psi + g);
    v[0] = *reinterpret_cast<const C*>(a);
#pragma unroll
    for (int i = 1; i < (1 << R); ++i) {
        const int b = __builtin_ctz(i), j = i ^ (i >> 1);
        const int64_t d = gr[b] * int64_t(sizeof(C));
        a += (j >> b) & 1 ? d : -d;
        v[j] = *reinterpret_cast<const C*>(a);
    }
}

template <int R, typename C>
__device__ __forceinline__ void store_direct(const C (&v)[1 << R], C* __restrict__ psi, int64_t g,
                                             const int64_t* gr) {
    char* a = reinterpret_cast<char*>(psi + g);
    *reinterpret_cast<C*>(a) = v[0];
#pragma unroll
    for (int i = 1; i < (1 << R); ++i) {
        const int b = __builtin_ctz(i), j = i ^ (i >> 1);
        const int64_t d = gr[b] * int64_t(sizeof(C));
        a += (j >> b) & 1 ? d : -d;
        *reinterpret_cast<C*>(a) = v[j];
    }
}

template <int NTB>
__device__ __forceinline__ int64_t lane_offset(const int64_t* gt, int tid) {
    int64_t o = 0;
#pragma unroll
    for (int q = 0; q < NTB; ++q) o ^= gt[q] & (int64_t(0) - int64_t((uint32_t(tid) >> q) & 1u));
    return o;
}

// Wave sum of a double, valid in lane 63: DPP adds over pairs, quads,
// half rows, rows, then rows 0+1 into row 1 and 2+3 into row 3
// (row_bcast:15), then rows 0..1 into rows 2..3 (row_bcast:31).
template <int CTRL, int ROW_MASK>
__device__ __forceinline__ double dpp_add(double v) {
    const uint64_t b = uint64_t(__double_as_longlong(v));
    const int lo = __builtin_amdgcn_update_dpp(0, int(uint32_t(b)), CTRL, ROW_MASK, 0xF, false);
    const int hi = __builtin_amdgcn_update_dpp(0, int(uint32_t(b >> 32)), CTRL, ROW_MASK, 0xF, false);
    return v + __longlong_as_double(int64_t((uint64_t(uint32_t(hi)) << 32) | uint32_t(lo)));
}

// Squared magnitudes of the lane's 2^R registers in FP64: their total and,
// for each register bit b, the half sum over registers with bit b set.
// Pairwise: the sums over bit b's pairs feed bit b+1 (2^R - 1 adds for the
// total, 2^R - 1 - R for the half sums).
template <int R, typename C>
__device__ __forceinline__ void reg_half_sums(const C (&v)[1 << R], double& tot, double (&half)[R]) {
    double w[1 << R];
#pragma unroll
    for (int j = 0; j < (1 << R); ++j)
        w[j] = double(v[j].x) * double(v[j].x) + double(v[j].y) * double(v[j].y);
#pragma unroll
    for (int b = 0; b < R; ++b) {
        const int n = (1 << R) >> (b + 1);    // pairs at this level
        double h = w[1];
#pragma unroll
        for (int i = 1; i < n; ++i) h += w[2 * i + 1];
        half[b] = h;
#pragma unroll
        for (int i = 0; i < n; ++i) w[i] = w[2 * i] + w[2 * i + 1];
    }
    tot = w[0];
}

// Same sums for kernels that share the CU with a second workgroup: the tree over
// the register bits is walked depth first, so that one partial sum per level is
// live, and every right branch is added to its level's half sum: two adds per
// amplitude (one accumulator per sum took 1 + R / 2): ladder
// 2x13, 26 sites, 24.2 -> 22.9 ms per 50 steps.
template <int R, int LEVEL, int J, typename C>
__device__ __forceinline__ double half_sum_tree(const C (&v)[1 << R], double (&half)[R]) {
    if constexpr (LEVEL == 0) {
        return double(v[J].x) * double(v[J].x) + double(v[J].y) * double(v[J].y);
    } else {
        const double l = half_sum_tree<R, LEVEL - 1, J>(v, half);
        const double r = half_sum_tree<R, LEVEL - 1, J + (1 << (LEVEL - 1))>(v, half);
        half[LEVEL - 1] += r;
        return l + r;
    }
}

template <int R, typename C>
__device__ __forceinline__ void reg_half_sums_seq(const C (&v)[1 << R], double& tot, double (&half)[R]) {
#pragma unroll
    for (int b = 0; b < R; ++b) half[b] = 0.0;
    tot = half_sum_tree<R, R, 0>(v, half);
}

__device__ __forceinline__ double wave_sum_last(double v) {
    v = dpp_add<0xB1, 0xF>(v);     // quad_perm [1,0,3,2]
    v = dpp_add<0x4E, 0xF>(v);     // quad_perm [2,3,0,1]
    v = dpp_add<0x141, 0xF>(v);    // row_half_mirror
    v = dpp_add<0x140, 0xF>(v);    // row_mirror
    v = dpp_add<0x142, 0xA>(v);    // row_bcast:15 into rows 1, 3
    v = dpp_add<0x143, 0xC>(v);    // row_bcast:31 into rows 2, 3
    return v;
}

// Observable of one site on the lane's registers: the sign of each amplitude
// follows the site's bit (thread bit, register bit or a bit of the tile base;
// see kOpMeas).
template <int R, typename C>
__device__ __forceinline__ void site_observe(const C (&v)[1 << R], int aux, int64_t base, double& p,
                                             double& n) {
    const int kind = (aux >> 6) & 3, idx = (aux >> 8) & 63;
    const int sign = kind == 0 ? ((int(threadIdx.x) >> idx) & 1)
                   : kind == 2 ? int((base >> idx) & 1) : 0;
    const int mask = kind == 1 ? (1 << idx) : 0;
    p = 0.0;
    n = 0.0;
    reg_observe<R>(v, sign, mask, p, n);
}

// Brings a pass's stage headers and ops into the scalar cache, several lines
// in flight, each wave its share.  Read in order they miss it once per stage
// and once per few ops, one miss after the other: on a one-tile workgroup
// (M <= 22) that is a microsecond of every pass.
template <typename T, int NT>
__device__ __forceinline__ void warm_tables(const DevPass& P, const DevStage* __restrict__ stages,
                                            const DevOp<T>* __restrict__ ops) {
    constexpr int kLine = 16, NW = NT / 64;     // words per 64-byte line; waves
    const int wave = __builtin_amdgcn_readfirstlane(int(threadIdx.x) / 64);
    const DevStage* S = stages + P.stage0;
    const DevStage& L = S[P.nstage - 1];
    const int* w = reinterpret_cast<const int*>(ops + S->op0);
    const int last = (L.op0 + L.nop + 1 - S->op0) * int(sizeof(DevOp<T>) / 4) - 1;
    for (int si = wave; si < P.nstage; si += NW) {
        // the first 3 lines of a stage hold what the stage loop reads
        const int* p = reinterpret_cast<const int*>(S + si);
        const int a = p[0], b = p[kLine], c = p[2 * kLine];
        asm volatile("" ::"s"(a), "s"(b), "s"(c));
    }
    for (int i = wave * 4 * kLine; i <= last; i += NW * 4 * kLine) {
        auto at = [&](int n) { return w[i + n * kLine < last ? i + n * kLine : last]; };
        const int a = at(0), b = at(1), c = at(2), d = at(3);
        asm volatile("" ::"s"(a), "s"(b), "s"(c), "s"(d));
    }
}

template <typename T, int R, int NT, bool WRITES, int ENGINE = 0, bool PROFILE = false>
__device__ __forceinline__ void pass_tiles(typename CT<T>::c* __restrict__ psi, const DevPass& P,
                                           const DevStage* __restrict__ stages,
                                           const DevOp<T>* __restrict__ ops, unsigned wperm,
                                           unsigned G, int64_t tiles_per_member, char* ldsb,
                                           double (&accP)[kMaxMeas], double (&accN)[kMaxMeas],
                                           const float* __restrict__ mats = nullptr,
                                           double* pacc = nullptr, double* nacc = nullptr) {
    using C = typename CT<T>::c;
    const int tid = threadIdx.x;
    const DevStage& S0 = stages[P.stage0];
    const DevStage& SL = stages[P.stage0 + P.nstage - 1];
    constexpr int NTB = __builtin_ctz(NT);
    const int64_t gin_t = lane_offset<NTB>(S0.gt_in, tid);
    const int64_t gout_t = lane_offset<NTB>(SL.gt_out, tid);

    // Tile bases: tile = wperm + i * G, so base = deposit(wperm) | (i-th
    // submask of the free bits above the lowest log2(G) ones).
    const int64_t base_w = deposit(wperm, P.free_mask);
    int64_t m_hi = P.free_mask;
    for (unsigned g = G; g > 1; g >>= 1) m_hi &= m_hi - 1;

    // The next tile's loads are issued into `pre` at the start of a tile and
    // always (the last tile re-reads itself), so every iteration ends with
    // the same memory ops outstanding -- prefetch loads, then stores -- and
    // the copy out of `pre` only waits for the loads.
    C pre[1 << R];
    int64_t hi = 0;
    load_direct<R>(pre, psi, base_w + gin_t, S0.gr_in);

    auto tile_body = [&](int64_t it_tile) {
        const int64_t base = base_w | hi;
        C v[1 << R];
#pragma unroll
        for (int j = 0; j < (1 << R); ++j) v[j] = pre[j];
        if (it_tile + 1 < tiles_per_member) hi = next_submask(hi, m_hi);
        load_direct<R>(pre, psi, (base_w | hi) + gin_t, S0.gr_in);

        for (int si = 0; si < P.nstage; ++si) {
            const DevStage& S = stages[P.stage0 + si];
            const uint32_t pb = stage_base<NTB>(S, tid);
            RegBits<R> rb;
#pragma unroll
            for (int b = 0; b < R; ++b) rb.rbit[b] = S.rbit[b];
            if (si > 0) gather<R>(v, ldsb, pb, rb);
            ConstOp<T>* op = const_ops<T>(ops + S.op0);
            while (true) {
                int code;
                if constexpr (ENGINE == 1) {
                    if (op->code == kOpMat) {
                        if constexpr (sizeof(T) == 4 && R == 5) mfma_stage(v, mats + size_t(op->aux) * kMatFloats);
                        ++op;
                        continue;
                    }
                    code = op->code;
                } else {
                    op = run_factors<R>(v, op, code);
                }
                if (code == kOpEnd) break;
                // observable of the state at this point
                if constexpr (PROFILE) {
                    // Every per-site observable at this point from the
                    // lane's total weight and its register-bit half sums,
                    // each squared once; wave sums go to the wave's LDS
                    // row (pacc / nacc), one row per wave.
                    double tot, half[R];
                    reg_half_sums<R>(v, tot, half);
                    const bool last = (tid & 63) == 63;
                    while (op->code == kOpMeas) {
                        const int aux = op->aux;
                        const int slot = aux & 63, kind = (aux >> 6) & 3, idx = (aux >> 8) & 63;
                        const int nslot = ((aux >> 14) & 7) - 1;
                        double p;
                        if (kind == 1) {
                            double h = half[0];
#pragma unroll
                            for (int b = 1; b < R; ++b)
                                if (b == idx) h = half[b];
                            p = tot - 2.0 * h;
                        } else {
                            const int neg = kind == 0 ? ((tid >> idx) & 1) : int((base >> idx) & 1);
                            p = neg ? -tot : tot;
                        }
                        p = wave_sum_last(p);
                        if (last) pacc[slot] += p;
                        if (nslot >= 0) {
                            const double n = wave_sum_last(tot);
                            if (last) nacc[nslot] += n;
                        }
                        ++op;
                    }
                } else {
                    const int slot = op->aux & 63;
                    double p, n;
                    site_observe<R>(v, op->aux, base, p, n);
#pragma unroll
                    for (int m = 0; m < kMaxMeas; ++m)
                        if (m == slot) { accP[m] += p; accN[m] += n; }
                    ++op;
                }
            }
            if (si + 1 < P.nstage) {
                // A lane scatters to exactly the LDS slots the next stage's
                // lanes gather after the barrier.  When both stages keep the
                // same positions on the wave bits, those slots belong to the
                // wave's own lanes and only the wave is ordered.
                scatter<R>(v, ldsb, pb, rb);
                if (S.xnext != 0) lds_barrier();
                else wave_lds_sync();
            }
        }
        if constexpr (WRITES) store_direct<R>(v, psi, base + gout_t, SL.gr_out);
        // the last gathers are done before the next tile's scatters, unless
        // the last and first stages keep the same wave positions (then every
        // wave's slots are its own across the tile boundary)
        if (P.tile_barrier) lds_barrier();
    };
    tile_body(0);
    for (int64_t it_tile = 1; it_tile < tiles_per_member; ++it_tile) tile_body(it_tile);
}

// Same for passes that exchange through per-lane slots (HALF: in two halves).
// No register prefetch: several workgroups share a CU and cover each other's
// loads (half of the next tile prefetched into the registers that are left
// gained 2 % with several tiles per workgroup and nothing with one).  What
// bounds it, per CU: M = 30 complex64 tiles of 2^14 take 3.5 ms per pass for the
// sweep alone, about 3 ms of VALU issue and 1.4 ms of LDS traffic, of which two
// workgroups overlap a part: 4.7 ms (star M = 28: VALU busy 70 % of the time);
// small tiles (M <= 20) take the sum of the three.
template <typename T, int R, int NT, bool WRITES, bool PROFILE, bool HALF>
__device__ __forceinline__ void slot_tiles(typename CT<T>::c* __restrict__ psi, const DevPass& P,
                                           const DevStage* __restrict__ stages,
                                           const DevOp<T>* __restrict__ ops, unsigned wperm, unsigned G,
                                           int64_t tiles_per_member, char* ldsb, double* pacc,
                                           double* nacc = nullptr, bool writes = true) {
    using C = typename CT<T>::c;
    const int tid = threadIdx.x;
    const int nstage = P.nstage;
    const DevStage* S0 = stages + P.stage0;
    const DevStage& SL = S0[nstage - 1];
    constexpr int NTB = __builtin_ctz(NT), RW = HALF ? R - 1 : R;
    constexpr int EB = sizeof(C), ROW = exchange_row_slots(NT, EB) * EB;
    char* own = ldsb + exchange_slot(tid, EB) * EB;
    bool prev_cross = false;
    const int64_t gin_t = lane_offset<NTB>(S0->gt_in, tid);
    const int64_t gout_t = lane_offset<NTB>(SL.gt_out, tid);
    const int64_t base_w = deposit(wperm, P.free_mask);
    int64_t m_hi = P.free_mask, hi = 0;
    for (unsigned g = G; g > 1; g >>= 1) m_hi &= m_hi - 1;

    for (int64_t it_tile = 0; it_tile < tiles_per_member; ++it_tile) {
        const int64_t base = base_w | hi;
        C v[1 << R];
        load_direct<R>(v, psi, base + gin_t, S0->gr_in);
        hi = next_submask(hi, m_hi);
        for (int si = 0; si < nstage; ++si) {
            const DevStage& S = S0[si];
            // read before the ops, which hide the loads' latency
            ExchangeWeights<RW, NTB> xw;
            xw.load(S);
            ConstOp<T>* op = const_ops<T>(ops + S.op0);
            while (true) {
                int code;
                op = run_ops<R, T>(v, op, code);
                if (code == kOpEnd) break;
                // observable of the state at this point
                if constexpr (PROFILE) {
                    // Every per-site observable at this point from the
                    // lane's total weight and its register-bit half sums,
                    // each squared once; wave sums go to the wave's LDS
                    // row (pacc / nacc), one row per wave.
                    double tot, half[R];
                    reg_half_sums_seq<R>(v, tot, half);
                    const bool last = (tid & 63) == 63;
                    while (op->code == kOpMeas) {
                        const int aux = op->aux;
                        const int slot = aux & 63, kind = (aux >> 6) & 3, idx = (aux >> 8) & 63;
                        const int nslot = ((aux >> 14) & 7) - 1;
                        double p;
                        if (kind == 1) {
                            double h = half[0];
#pragma unroll
                            for (int b = 1; b < R; ++b)
                                if (b == idx) h = half[b];
                            p = tot - 2.0 * h;
                        } else {
                            const int neg = kind == 0 ? ((tid >> idx) & 1) : int((base >> idx) & 1);
                            p = neg ? -tot : tot;
                        }
                        p = wave_sum_last(p);
                        if (last) pacc[slot] += p;
                        if (nslot >= 0) {
                            const double n = wave_sum_last(tot);
                            if (last) nacc[nslot] += n;
                        }
                        ++op;
                    }
                } else {
                    // wave sums into the wave's own LDS row (pacc: slot
                    // m holds P at 2m, N at 2m + 1), no accumulator
                    // registers
                    const int aux = op->aux, slot = aux & 63;
                    double p, n;
                    site_observe<R>(v, aux, base, p, n);
                    p = wave_sum_last(p);
                    n = wave_sum_last(n);
                    if ((tid & 63) == 63) {
                        pacc[2 * slot] += p;
                        pacc[2 * slot + 1] += n;
                    }
                    ++op;
                }
            }
            if (si + 1 < nstage) {
                // few instructions between two waits: they go before the other
                // workgroup's arithmetic (star M = 28 64.8 -> 64.0 ms)
                if constexpr (HALF) __builtin_amdgcn_s_setprio(2);
                exchange<R, ROW, HALF>(v, ldsb, own, xw, prev_cross);
                if constexpr (HALF) __builtin_amdgcn_s_setprio(0);
            }
        }
        if constexpr (WRITES)
            if (writes) store_direct<R>(v, psi, base + gout_t, SL.gr_out);
    }
}

// Workgroup sum of measurement slot m of the accumulators (thread 0).
template <int NT>
__device__ __forceinline__ void slot_sum(const double (&accP)[kMaxMeas],
                                         const double (&accN)[kMaxMeas], int m, double* red,
                                         double& p, double& n) {
    p = accP[0];
    n = accN[0];
#pragma unroll
    for (int mm = 1; mm < kMaxMeas; ++mm)
        if (mm == m) { p = accP[mm]; n = accN[mm]; }
    block_sum2<NT>(p, n, red);
}

// --------------------------------------------------------------- k_pass
// partials: [slot][nwg][2] (P, N), or with PROFILE [slot][nwg][M + 1] (P of
// every site, then N).
// X: exchanges through LDS (see ExchangeMode); all but kWholeTiles have no
// register prefetch and cap the registers so that several workgroups share a
// CU, as many as their LDS lets in, up to 4 waves per SIMD.
template <typename T, int R, int NT, int X>
__host__ __device__ constexpr int exchange_slots() {
    return X == kWholeTiles ? NT << R
                            : exchange_row_slots(NT, sizeof(typename CT<T>::c)) << (X == kHalfTiles ? R - 1 : R);
}
template <typename T, int R, int NT, int X>
__host__ __device__ constexpr int waves_per_eu() {
    if (X == kWholeTiles) return 1;
    const int wg = int((160 * 1024 - 8192) / (exchange_slots<T, R, NT, X>() * sizeof(typename CT<T>::c)));
    const int waves = (wg < 1 ? 1 : wg) * NT / 256;
    return waves > 4 ? 4 : waves < 1 ? 1 : waves;
}

template <typename T, int R, int NT, bool WRITES, int ENGINE, bool PROFILE, int X>
__global__ __launch_bounds__(NT, (waves_per_eu<T, R, NT, X>())) void k_pass(typename CT<T>::c* __restrict__ psi,
                                             const DevPass* __restrict__ passes,
                                             const DevStage* __restrict__ stages,
                                             const DevOp<T>* __restrict__ ops, int pass_index,
                                             int64_t tiles_per_wg, double* __restrict__ partials,
                                             int64_t step_offset, int ch, int nwg,
                                             const float* __restrict__ mats) {
    using C = typename CT<T>::c;
    __shared__ C lds[exchange_slots<T, R, NT, X>()];
    __shared__ double red[2 * (NT / 64)];
    const DevPass& P = passes[pass_index];
    double accP[kMaxMeas], accN[kMaxMeas];
#pragma unroll
    for (int m = 0; m < kMaxMeas; ++m) accP[m] = accN[m] = 0.0;
    // XCD-aware order: workgroups are dispatched round-robin over the 8
    // XCDs, so w and w + 8 share an L2.  They take adjacent tile indices,
    // i.e. tiles that differ only in the lowest non-tile address bit and so
    // share cache lines when the tile's contiguous runs are shorter than a
    // line.
    const unsigned G = gridDim.x, w = blockIdx.x;
    const unsigned wperm = (G >= 8) ? (w % 8u) * (G / 8u) + w / 8u : w;
    warm_tables<T, NT>(P, stages, ops);
    if constexpr (PROFILE) {
        // Per-wave accumulator rows; lane 63 of each wave owns its row.
        constexpr int NW = NT / 64;
        __shared__ double pacc[NW][kMaxMeasProfile];
        __shared__ double nacc[NW][kMaxMeas];
        const int wave = threadIdx.x / 64;
        if ((threadIdx.x & 63) == 63) {
            for (int m = 0; m < kMaxMeasProfile; ++m) pacc[wave][m] = 0.0;
            for (int m = 0; m < kMaxMeas; ++m) nacc[wave][m] = 0.0;
        }
        if constexpr (X != kWholeTiles)
            slot_tiles<T, R, NT, WRITES, true, X == kHalfTiles>(psi, P, stages, ops, wperm, G, tiles_per_wg,
                                                                reinterpret_cast<char*>(lds), pacc[wave],
                                                                nacc[wave]);
        else
            pass_tiles<T, R, NT, WRITES, ENGINE, true>(psi, P, stages, ops, wperm, G, tiles_per_wg,
                                                       reinterpret_cast<char*>(lds), accP, accN, mats,
                                                       pacc[wave], nacc[wave]);
        __syncthreads();
        const int M = P.k + P.nfree;
        auto dst = [&](int64_t step) {
            return partials + ((size_t)((step_offset + step) % ch) * nwg + blockIdx.x) * (M + 1);
        };
        // fixed-order sums over the waves
        for (int m = threadIdx.x; m < P.pmeas; m += NT) {
            double v = 0.0;
            for (int w = 0; w < NW; ++w) v += pacc[w][m];
            dst(P.pmeas_step[m])[P.pmeas_site[m]] = v;
        }
        if (threadIdx.x >= NT - kMaxMeas) {
            const int m = threadIdx.x - (NT - kMaxMeas);
            if (m < P.pnorm) {
                double v = 0.0;
                for (int w = 0; w < NW; ++w) v += nacc[w][m];
                dst(P.pmeas_step[P.pnorm_meas[m]])[M] = v;
            }
        }
        return;
    }
    if constexpr (X != kWholeTiles) {
        // per-wave observable rows; fixed-order sum over the waves
        constexpr int NW = NT / 64;
        __shared__ double wacc[NW][2 * kMaxMeas];
        const int wave = threadIdx.x / 64;
        if ((threadIdx.x & 63) == 63)
            for (int m = 0; m < 2 * kMaxMeas; ++m) wacc[wave][m] = 0.0;
        slot_tiles<T, R, NT, WRITES, false, X == kHalfTiles>(psi, P, stages, ops, wperm, G, tiles_per_wg,
                                                             reinterpret_cast<char*>(lds), wacc[wave]);
        __syncthreads();
        if (threadIdx.x < P.nmeas) {
            const int m = threadIdx.x;
            double p = 0.0, n = 0.0;
            for (int w = 0; w < NW; ++w) {
                p += wacc[w][2 * m];
                n += wacc[w][2 * m + 1];
            }
            const int64_t s = step_offset + P.meas_step[m];
            double* dst = partials + ((size_t)(s % ch) * nwg + blockIdx.x) * 2;
            dst[0] = p;
            dst[1] = n;
        }
        return;
    }
    pass_tiles<T, R, NT, WRITES, ENGINE, false>(psi, P, stages, ops, wperm, G, tiles_per_wg,
                                                       reinterpret_cast<char*>(lds), accP, accN, mats);
    for (int m = 0; m < P.nmeas; ++m) {
        double p, n;
        slot_sum<NT>(accP, accN, m, red, p, n);
        if (threadIdx.x == 0) {
            const int64_t s = step_offset + P.meas_step[m];
            double* dst = partials + ((size_t)(s % ch) * nwg + blockIdx.x) * 2;
            dst[0] = p;
            dst[1] = n;
        }
    }
}

// ------------------------------------------------------------ resident run
// One workgroup owns one whole state in its registers (2^M <= NT << R; the
// amplitudes past 2^M are zero and stay so) from the first step to the last
// and exchanges it through per-lane slots between stages; LDS also stages it
// between memory order and the registers.  A state this small is bound by the
// serial chain of its ops, not by any rate: about 80 clocks of scalar work and
// 2^R * 1.5 FMAs of 4 clocks per factor, 300 to 700 clocks per exchange, so 16
// amplitudes per lane (one wave at M <= 10, one per SIMD at M = 12).
// Observables: each wave's sums go to its row of a ring in LDS, written out
// with a fixed-order sum over the waves every kResidentRing values (a single
// wave writes its own).
constexpr int kResidentRing = 8;

template <int NW>
struct ResidentRing {
    double sum[kResidentRing][NW][2];
    double* dstP[kResidentRing];
    double* dstN[kResidentRing];
};

// Writes the first n entries of the ring (whole workgroup).
template <int NW>
__device__ __forceinline__ void flush_ring(const ResidentRing<NW>& ring, int n) {
    __syncthreads();
    if (int(threadIdx.x) < n) {
        const int e = threadIdx.x;
        double p = 0.0, q = 0.0;
        for (int w = 0; w < NW; ++w) {
            p += ring.sum[e][w][0];
            q += ring.sum[e][w][1];
        }
        *ring.dstP[e] = p;
        if (ring.dstN[e]) *ring.dstN[e] = q;
    }
    __syncthreads();
}

template <typename T, int R, int NT, bool PROFILE = false, int SLOTS>
__device__ __forceinline__ void resident_run(const ResidentJob& J, const DevStage* __restrict__ stages,
                                             const DevOp<T>* __restrict__ ops, int64_t n_steps,
                                             typename CT<T>::c (&lds)[SLOTS], ResidentRing<NT / 64>& ring,
                                             int* progress = nullptr) {
    using C = typename CT<T>::c;
    static_assert(SLOTS >= resident_slots(R, NT, int(sizeof(C))), "the state's rows do not fit the LDS buffer");
    constexpr int NTB = __builtin_ctz(NT), NW = NT / 64;
    constexpr int EB = sizeof(C), ROW = exchange_row_slots(NT, EB) * EB;
    const int tid = threadIdx.x;
    const int M = J.M;
    const uint32_t dim = 1u << M;
    C* psi = reinterpret_cast<C*>(J.psi);
    char* ldsb = reinterpret_cast<char*>(lds);
    char* own = ldsb + exchange_slot(tid, EB) * EB;
    // the state in memory order in LDS
    const double scale = 1.0 / sqrt(ldexp(1.0, M - 1));
    for (uint32_t x = tid; x < (uint32_t(NT) << R); x += NT) {
        C c;
        c.x = c.y = T(0);
        if (x < dim) {
            if (J.init) {
                double re, im;
                init_amp(x, M, J.init, J.polarized, J.seed, scale, &re, &im);
                c.x = T(re);
                c.y = T(im);
            } else {
                c = psi[x];
            }
        }
        lds[x] = c;
    }
    __syncthreads();
    // between memory order in LDS and an arrangement of the registers
    C v[1 << R];
    auto offset = [&](const int64_t* gt) { return uint32_t(lane_offset<NTB>(gt, tid)) * EB; };
    const int first = n_steps > 0 ? J.pro_stage0 : J.obs_stage0;
    {
        uint32_t w[R];
#pragma unroll
        for (int b = 0; b < R; ++b) w[b] = uint32_t(stages[first].gr_in[b]) * EB;
        gather_rows<R, 0>(v, ldsb, offset(stages[first].gt_in), w);
    }
    bool prev_cross = true;     // every wave gathers before the first scatter
    int nring = 0;
    int last_stage = first;
    for (int64_t k = 0; k <= n_steps; ++k) {
        const int st0 = k == 0 ? first : k < n_steps ? J.step_stage0 : J.last_stage0;
        // gangs that wait for this workgroup see that it moves (every 0.1 to 10 s)
        if (progress && (k & 0xffff) == 0 && tid == 0) atomicAdd(progress, 1);
        const int nst = k > 0 ? J.step_nstage : n_steps > 0 ? J.pro_nstage : 1;
        for (int si = 0; si < nst; ++si) {
            const DevStage& S = stages[st0 + si];
            ExchangeWeights<R, NTB> xw;
            xw.load(S);
            ConstOp<T>* op = const_ops<T>(ops + S.op0);
            while (true) {
                int code;
                op = run_ops<R, T>(v, op, code);
                if (code == kOpEnd) break;
                // observable of the state at this point
                const int aux = op->aux;
                double p, n;
                site_observe<R>(v, aux, 0, p, n);
                p = wave_sum_last(p);
                n = wave_sum_last(n);
                double* dstP = PROFILE ? J.Pall + k * M + ((aux >> 17) & 63) : J.P + k;
                double* dstN = J.N && (!PROFILE || ((aux >> 14) & 7)) ? J.N + k : nullptr;
                // sites past M belong to no site of the caller
                const bool own_site = !PROFILE || ((aux >> 17) & 63) < M;
                if constexpr (NW == 1) {
                    if (tid == 63 && own_site) {
                        *dstP = p;
                        if (dstN) *dstN = n;
                    }
                } else if (own_site) {
                    if ((tid & 63) == 63) {
                        ring.sum[nring][tid / 64][0] = p;
                        ring.sum[nring][tid / 64][1] = n;
                        if (tid == 63) {
                            ring.dstP[nring] = dstP;
                            ring.dstN[nring] = dstN;
                        }
                    }
                    if (++nring == kResidentRing) {
                        flush_ring<NW>(ring, nring);
                        nring = 0;
                    }
                }
                ++op;
            }
            last_stage = st0 + si;
            if (xw.xnext != kNoExchange && !(k == n_steps && si + 1 == nst))
                exchange<R, ROW, false>(v, ldsb, own, xw, prev_cross);
        }
    }
    if (NW > 1 && nring > 0) flush_ring<NW>(ring, nring);
    __syncthreads();            // every wave has gathered
    {
        uint32_t a = offset(stages[last_stage].gt_out);
        *reinterpret_cast<C*>(ldsb + a) = v[0];
#pragma unroll
        for (int i = 1; i < (1 << R); ++i) {
            const int b = __builtin_ctz(i), j = i ^ (i >> 1);
            const uint32_t w = uint32_t(stages[last_stage].gr_out[b]) * EB;
            a = (j >> b) & 1 ? a + w : a - w;
            *reinterpret_cast<C*>(ldsb + a) = v[j];
        }
    }
    __syncthreads();
    for (uint32_t x = tid; x < dim; x += NT) psi[x] = lds[x];
    __syncthreads();
}

template <typename T, int R, int NT, bool PROFILE>
__global__ __launch_bounds__(NT) void k_resident(ResidentJob job0,
                                                 const ResidentJob* __restrict__ jobs,
                                                 const DevStage* __restrict__ stages,
                                                 const DevOp<T>* __restrict__ ops,
                                                 int64_t n_steps) {
    using C = typename CT<T>::c;
    __shared__ C lds[resident_slots(R, NT, sizeof(C))];
    __shared__ ResidentRing<NT / 64> ring;
    ResidentJob J = jobs ? jobs[blockIdx.x] : job0;
    for (int32_t* f : {&J.M, &J.init, &J.obs_stage0, &J.pro_stage0, &J.pro_nstage, &J.step_stage0, &J.step_nstage,
                       &J.last_stage0})
        *f = __builtin_amdgcn_readfirstlane(*f);
    resident_run<T, R, NT, PROFILE>(J, stages, ops, n_steps, lds, ring);
}

// ---------------------------------------------------------------- k_batch
// Persistent batch: each workgroup runs its list of jobs in order.  A job
// is a whole problem held in registers (gang size 1, M < tile bits), or one
// member's share of a problem run as tiled passes by a gang of G
// workgroups that meet at a counter after every pass.  The host orders all
// job lists consistently (a global order of gang start times), so every
// wait is on members busy with earlier jobs: no cycle, no deadlock.  Each
// wait is bounded; on time-out the problem is flagged and its P set to NaN.
// A wait gives up when nothing in the launch has moved for kGangWaitTicks (the sum
// of its counters stands still), and at once when any workgroup has flagged an
// error.
__device__ __forceinline__ uint32_t launch_progress(const int* sync) {
    uint32_t sum = 0;
    for (int i = sync[kSyncCount]; --i >= kSyncProgress;)
        sum += uint32_t(__hip_atomic_load(sync + i, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT));
    return sum;
}

__device__ __forceinline__ bool gang_barrier(int* counter, uint32_t target, int* sync) {
    // Every wave waits until its stores are in the XCD's L2; after the barrier
    // one lane writes that back for all (release) and, when the gang has met,
    // invalidates what the CU and the L2 hold (acquire).  A release by every
    // wave wrote the L2 back four times: 32 stars of M = 14 to 20, 25 steps,
    // 20.5 -> 16.9 ms.
    asm volatile("s_waitcnt vmcnt(0) lgkmcnt(0)" ::: "memory");
    __syncthreads();
    __shared__ int ok_s;
    if (threadIdx.x == 0) {
        int ok = 1;
        __builtin_amdgcn_fence(__ATOMIC_RELEASE, "agent");
        atomicAdd(counter, 1);
        GangClock clock{uint64_t(wall_clock64())};
        for (int polls = 1;
             gang_waits(uint32_t(__hip_atomic_load(counter, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT)), target);
             ++polls) {
            __builtin_amdgcn_s_sleep(4);
            // the flag and the clock take as long to read as the counter: not
            // every time
            if (polls & 15) continue;
            const uint64_t now = uint64_t(wall_clock64());
            if (__hip_atomic_load(sync + kSyncError, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) != 0 ||
                (clock.due(now) && clock.stalled(now, launch_progress(sync)))) {
                atomicOr(sync + kSyncError, 1);
                ok = 0;
                break;
            }
        }
        __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "agent");
        ok_s = ok;
    }
    __syncthreads();
    return ok_s != 0;
}

// HALF: gangs run half-tile passes and two workgroups share a CU.  One-workgroup
// problems are at most half a tile either way, what the registers hold beside
// the gangs' tiles.
template <typename T, int R, int NT, bool HALF>
__global__ __launch_bounds__(NT, HALF ? 2 * NT / 256 : 1) void k_batch(const BatchProblem* __restrict__ probs,
                                              const BatchJob* __restrict__ jobs,
                                              const int* __restrict__ job_start,
                                              const DevPass* __restrict__ passes,
                                              const DevStage* __restrict__ stages,
                                              const DevOp<T>* __restrict__ ops,
                                              const int2* __restrict__ launches,
                                              double* __restrict__ partials,
                                              int* __restrict__ sync, int64_t n_steps) {
    using C = typename CT<T>::c;
    constexpr int K = R + __builtin_ctz(NT);
    constexpr int KL = K - 1;               // largest one-workgroup problem
    constexpr int NW = NT / 64;
    static_assert(R == batch_regs(sizeof(T) == 4, HALF) && NT == batch_lanes(HALF), "not the batch kernel's shape");
    __shared__ C lds[batch_lds_slots(sizeof(T) == 4, HALF)];
    __shared__ double red[2 * NW];
    __shared__ double wacc[HALF ? NW : 1][2 * kMaxMeas];
    __shared__ ResidentRing<NW> ring;
    const int tid = threadIdx.x;
    const int wave = tid / 64;
    for (int jb = job_start[blockIdx.x]; jb < job_start[blockIdx.x + 1]; ++jb) {
        const BatchJob job = jobs[jb];
        if (__hip_atomic_load(sync + kSyncError, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) != 0) break;
        const BatchProblem& B = probs[job.problem];
        if (B.gsize == 1 && B.M <= KL) {
            ResidentJob J{};
            J.psi = B.psi;
            J.P = B.P;
            J.N = B.N;
            J.seed = B.seed;
            J.M = B.M;
            J.polarized = B.polarized;
            J.init = B.init;
            J.obs_stage0 = B.obs_stage0;
            J.pro_stage0 = B.pro_stage0;
            J.pro_nstage = B.pro_nstage;
            J.step_stage0 = B.step_stage0;
            J.step_nstage = B.step_nstage;
            J.last_stage0 = B.last_stage0;
            int* progress = sync + kSyncProgress;
            // 16 amplitudes per lane, 32 (complex64) for the largest
            if constexpr (NT == 256) {
                if (B.M <= 12) resident_run<T, 4, NT>(J, stages, ops, n_steps, lds, ring, progress);
                else if constexpr (sizeof(T) == 4) resident_run<T, 5, NT>(J, stages, ops, n_steps, lds, ring, progress);
            } else {
                resident_run<T, 4, NT>(J, stages, ops, n_steps, lds, ring, progress);
            }
            continue;
        }
        // gang member `rank` of `gsize`
        C* psi = reinterpret_cast<C*>(B.psi);
        const unsigned G = unsigned(B.gsize), rank = unsigned(job.rank);
        int* ctr = sync + kSyncGangs + B.counter;
        uint32_t epoch = 0;
        bool ok = true;
        if (B.init) {
            const uint64_t dim = 1ull << B.M;
            const double scale = 1.0 / sqrt(ldexp(1.0, B.M - 1));
            for (uint64_t x = uint64_t(rank) * NT + tid; x < dim; x += uint64_t(G) * NT) {
                double re, im;
                init_amp(x, B.M, B.init, B.polarized, B.seed, scale, &re, &im);
                C c;
                c.x = T(re);
                c.y = T(im);
                psi[x] = c;
            }
            ok = gang_barrier(ctr, ++epoch * G, sync);
        }
        const int64_t tpm = B.ntiles / G;
        for (int l = 0; l < B.nlaunch && ok; ++l) {
            const int2 la = launches[B.launch0 + l];
            const DevPass& P = passes[B.pass0 + la.x];
            double accP[kMaxMeas], accN[kMaxMeas];
#pragma unroll
            for (int m = 0; m < kMaxMeas; ++m) accP[m] = accN[m] = 0.0;
            if constexpr (HALF) {
                // per-wave observable rows (as k_pass), summed over the
                // waves in a fixed order; the previous pass's reads of the
                // rows finished before the gang barrier
                if ((tid & 63) == 63)
                    for (int m = 0; m < 2 * kMaxMeas; ++m) wacc[wave][m] = 0.0;
                slot_tiles<T, R, NT, true, false, true>(psi, P, stages, ops, rank, G, tpm,
                                                        reinterpret_cast<char*>(lds), wacc[wave], nullptr,
                                                        P.writes != 0);
                __syncthreads();
                if (tid < P.nmeas) {
                    const int m = tid;
                    double p = 0.0, n = 0.0;
                    for (int w = 0; w < NW; ++w) {
                        p += wacc[w][2 * m];
                        n += wacc[w][2 * m + 1];
                    }
                    const int64_t s = int64_t(la.y) + P.meas_step[m];
                    double* dst = partials + B.part0 + ((s % kBatchRing) * G + rank) * 2;
                    dst[0] = p;
                    dst[1] = n;
                }
            } else {
                if (P.writes)
                    pass_tiles<T, R, NT, true>(psi, P, stages, ops, rank, G, tpm,
                                               reinterpret_cast<char*>(lds), accP, accN);
                else
                    pass_tiles<T, R, NT, false>(psi, P, stages, ops, rank, G, tpm,
                                                reinterpret_cast<char*>(lds), accP, accN);
                for (int m = 0; m < P.nmeas; ++m) {
                    double p, n;
                    slot_sum<NT>(accP, accN, m, red, p, n);
                    if (tid == 0) {
                        const int64_t s = int64_t(la.y) + P.meas_step[m];
                        double* dst = partials + B.part0 + ((s % kBatchRing) * G + rank) * 2;
                        dst[0] = p;
                        dst[1] = n;
                    }
                }
            }
            ok = gang_barrier(ctr, ++epoch * G, sync);
            if (rank == 0 && tid < 64 && ok) {
                for (int m = 0; m < P.nmeas; ++m) {
                    const int64_t s = int64_t(la.y) + P.meas_step[m];
                    const double* src = partials + B.part0 + (s % kBatchRing) * G * 2;
                    double p = 0.0, n = 0.0;
                    for (unsigned r = tid; r < G; r += 64) {
                        p += src[2 * r];
                        n += src[2 * r + 1];
                    }
                    p = wave_sum_last(p);
                    n = wave_sum_last(n);
                    if (tid == 63) {
                        B.P[s] = p;
                        if (B.N) B.N[s] = n;
                    }
                }
            }
        }
        if (!ok && rank == 0 && tid == 0)
            for (int64_t s = 0; s <= n_steps; ++s) B.P[s] = __builtin_nan("");
    }
}

#if SPIN_PART == 0
// Sync integers of a batch launch at its start (see kSyncError).
__global__ void k_sync_start(int* sync, int n) {
    for (int i = blockIdx.x * blockDim.x + threadIdx.x; i < n; i += gridDim.x * blockDim.x)
        sync[i] = i == kSyncCount ? n : 0;
}

// Folds a launch's error flag into the device's sticky batch status word.
__global__ void k_status_or(const int* err, int* status) {
    if (threadIdx.x == 0 && *err != 0) atomicOr(status, *err);
}

void launch_sync_start(int* sync, int n, hipStream_t st) {
    hipLaunchKernelGGL(k_sync_start, dim3((n + 255) / 256), dim3(256), 0, st, sync, n);
}

void launch_status_or(const int* err, int* status, hipStream_t st) {
    hipLaunchKernelGGL(k_status_or, dim3(1), dim3(64), 0, st, err, status);
}
#else
void launch_sync_start(int* sync, int n, hipStream_t st);
void launch_status_or(const int* err, int* status, hipStream_t st);
#endif

// Pass launches by kernel family (per-lane slots or one layout per tile), each
// compiled in its own part.
template <typename T>
hipError_t launch_pass_slots(const PassShape& sh, void* psi, const DevPass* passes, const DevStage* stages, const DevOp<T>* ops,
               int pass_index, int64_t tiles_per_wg, int nwg, double* partials, int64_t step_offset, int ch,
               hipStream_t st);
template <typename T>
hipError_t launch_pass_whole(const PassShape& sh, void* psi, const DevPass* passes, const DevStage* stages, const DevOp<T>* ops,
               int pass_index, int64_t tiles_per_wg, int nwg, double* partials, int64_t step_offset, int ch,
               hipStream_t st);

#if SPIN_PART == 0
// ------------------------------------------------------------- launchers
static inline int grid_for(uint64_t n, int per_block, int cap) {
    uint64_t g = (n + per_block - 1) / per_block;
    if (g > uint64_t(cap)) g = cap;
    if (g < 1) g = 1;
    return int(g);
}

template <typename T>
hipError_t launch_init(void* psi, int M, int n, uint64_t seed, hipStream_t st) {
    const double scale = 1.0 / sqrt(ldexp(1.0, M - 1));
    const int grid = grid_for((1ull << (M - 1)) / CT<T>::V, 256, 1 << 16);
    hipLaunchKernelGGL((k_init<T, false>), dim3(grid), dim3(256), 0, st,
                       reinterpret_cast<typename CT<T>::c*>(psi), M, n, seed, scale);
    return hipGetLastError();
}

template <typename T>
hipError_t launch_init_product(void* psi, int M, int n, uint64_t seed, hipStream_t st) {
    const double scale = 1.0 / sqrt(ldexp(1.0, M - 1));
    // lanes that each take several indices share the sum over the low sites:
    // M = 28 427 us, with 1 << 16 workgroups 482 us
    const int grid = grid_for((1ull << (M - 1)) / CT<T>::V, 256, 1 << 14);
    hipLaunchKernelGGL((k_init<T, true>), dim3(grid), dim3(256), 0, st,
                       reinterpret_cast<typename CT<T>::c*>(psi), M, n, seed, scale);
    return hipGetLastError();
}

template <typename T>
hipError_t launch_init_members(void* psi, int M, int cbits, int polarized, uint64_t first,
                               uint64_t count, bool phases, hipStream_t st) {
    const int grid = grid_for(1ull << (M + cbits), 256, 1 << 16);
    hipLaunchKernelGGL(k_init_members<T>, dim3(grid), dim3(256), 0, st,
                       reinterpret_cast<typename CT<T>::c*>(psi), M, cbits, polarized, first, count, phases);
    return hipGetLastError();
}

hipError_t launch_accumulate(double* acc, const double* add, int64_t n, double scale,
                             hipStream_t st) {
    const int grid = grid_for(uint64_t(n), 256, 1024);
    hipLaunchKernelGGL(k_accumulate, dim3(grid), dim3(256), 0, st, acc, add, n, scale);
    return hipGetLastError();
}

template <typename T>
hipError_t launch_observe(const void* psi, int M, int site, double* partials, int nblk,
                          hipStream_t st) {
    const auto* in = reinterpret_cast<const typename CT<T>::c*>(psi);
    if (sizeof(T) == 8 && M <= 25)
        hipLaunchKernelGGL((k_observe<T, 1>), dim3(nblk), dim3(256), 0, st, in, M, site, partials);
    else
        hipLaunchKernelGGL((k_observe<T, 4>), dim3(nblk), dim3(256), 0, st, in, M, site, partials);
    return hipGetLastError();
}

hipError_t launch_reduce_profile(const double* partials, int nwg, int ch, int M, int64_t s0,
                                 int64_t count, double* Pall, double* N, hipStream_t st) {
    if (count <= 0) return hipSuccess;
    hipLaunchKernelGGL(k_reduce_profile, dim3(unsigned(count * (M + 1))), dim3(256), 0, st, partials,
                       nwg, ch, M, s0, Pall, N);
    return hipGetLastError();
}

hipError_t launch_reduce(const double* partials, int nwg, int ch, int64_t s0, int64_t count,
                         double* P, double* N, hipStream_t st) {
    if (count <= 0) return hipSuccess;
    // one workgroup per step: a large one where it has many partial sums to read
    if (nwg > 4096)
        hipLaunchKernelGGL(k_reduce<1024>, dim3(unsigned(count)), dim3(1024), 0, st, partials, nwg, ch, s0, P, N);
    else
        hipLaunchKernelGGL(k_reduce<256>, dim3(unsigned(count)), dim3(256), 0, st, partials, nwg, ch, s0, P, N);
    return hipGetLastError();
}

template <typename T>
hipError_t launch_factor(void* psi, int M, int lo, int hi, double t, double s, double pr,
                         double pim, int zz, hipStream_t st) {
    const int grid = grid_for(1ull << (M - 2), 256, 1 << 16);
    hipLaunchKernelGGL(k_factor<T>, dim3(grid), dim3(256), 0, st,
                       reinterpret_cast<typename CT<T>::c*>(psi), M, lo, hi, T(t), T(s), T(pr),
                       T(pim), zz);
    return hipGetLastError();
}

bool pass_small_exists(bool f32, int r, int nt) {
    return (nt == 256 && r >= 2 && r <= 4) || (f32 && nt == 512 && r == 4);
}

bool pass_half_exists(bool f32, int r, int nt) {
    if (f32) return (r == 5 && nt == 512) || (r == 6 && nt == 256);
    return (r == 4 && nt == 512) || (r == 5 && nt == 256) || (r == 5 && nt == 512);
}

bool pass_shape_exists(bool f32, int r, int nt, int engine) {
    if (engine == 1) return f32 && r == 5 && nt == 512;
    if (engine != 0) return false;
    if (f32) return (r == 4 && nt == 256) || (r == 5 && nt == 256) || (r == 5 && nt == 512) ||
                    (r == 6 && nt == 256) || (r == 4 && nt == 512) || (r == 4 && nt == 1024);
    return (r == 4 && nt == 256) || (r == 5 && nt == 256) || (r == 4 && nt == 512) ||
           (r == 3 && nt == 512) || (r == 3 && nt == 1024);
}

template <typename T>
int batch_occupancy(bool half);

int batch_tile_bits(bool f32) { return f32 ? 14 : 13; }

// Launch shapes of the batch kernel: whole tiles 2^R x 512 lanes (one
// workgroup per CU); half tiles 2^(R+1) x 256 lanes (two per CU), whose
// larger register stages take fewer LDS exchanges on dense coupling graphs.
BatchShape batch_shape(bool f32, bool half) {
    return BatchShape{half, batch_regs(f32, half), batch_lanes(half)};
}

template hipError_t launch_init<float>(void*, int, int, uint64_t, hipStream_t);
template hipError_t launch_init<double>(void*, int, int, uint64_t, hipStream_t);
template hipError_t launch_init_product<float>(void*, int, int, uint64_t, hipStream_t);
template hipError_t launch_init_product<double>(void*, int, int, uint64_t, hipStream_t);
template hipError_t launch_init_members<float>(void*, int, int, int, uint64_t, uint64_t, bool, hipStream_t);
template hipError_t launch_init_members<double>(void*, int, int, int, uint64_t, uint64_t, bool, hipStream_t);
template hipError_t launch_observe<float>(const void*, int, int, double*, int, hipStream_t);
template hipError_t launch_observe<double>(const void*, int, int, double*, int, hipStream_t);
template hipError_t launch_factor<float>(void*, int, int, int, double, double, double, double, int,
                                         hipStream_t);
template hipError_t launch_factor<double>(void*, int, int, int, double, double, double, double,
                                          int, hipStream_t);

template <typename T>
hipError_t launch_pass(const PassShape& sh, void* psi, const DevPass* passes,
                       const DevStage* stages, const DevOp<T>* ops, int pass_index,
                       int64_t tiles_per_wg, int nwg, double* partials, int64_t step_offset,
                       int ch, hipStream_t st) {
    return (sh.exchange != kWholeTiles ? launch_pass_slots<T> : launch_pass_whole<T>)(sh, psi, passes, stages, ops, pass_index,
                                                                 tiles_per_wg, nwg, partials, step_offset, ch, st);
}
template hipError_t launch_pass<float>(const PassShape&, void*, const DevPass*, const DevStage*,
                                       const DevOp<float>*, int, int64_t, int, double*, int64_t,
                                       int, hipStream_t);
template hipError_t launch_pass<double>(const PassShape&, void*, const DevPass*, const DevStage*,
                                        const DevOp<double>*, int, int64_t, int, double*, int64_t,
                                        int, hipStream_t);

int batch_blocks_per_cu(bool f32, bool half) {
    return f32 ? batch_occupancy<float>(half) : batch_occupancy<double>(half);
}
#endif

#if SPIN_PART >= 2 && SPIN_PART <= 5
template <typename T, int R, int NT, int ENGINE = 0, bool PROFILE = false, int X = kWholeTiles>
static hipError_t pass_one(bool writes, void* psi, const DevPass* passes, const DevStage* stages,
                           const DevOp<T>* ops, int pass_index, int64_t tiles_per_wg, int nwg,
                           double* partials, int64_t step_offset, int ch, const float* mats,
                           hipStream_t st) {
    if (writes)
        hipLaunchKernelGGL((k_pass<T, R, NT, true, ENGINE, PROFILE, X>), dim3(nwg), dim3(NT), 0, st,
                           reinterpret_cast<typename CT<T>::c*>(psi), passes, stages, ops,
                           pass_index, tiles_per_wg, partials, step_offset, ch, nwg, mats);
    else
        hipLaunchKernelGGL((k_pass<T, R, NT, false, ENGINE, PROFILE, X>), dim3(nwg), dim3(NT), 0, st,
                           reinterpret_cast<typename CT<T>::c*>(psi), passes, stages, ops,
                           pass_index, tiles_per_wg, partials, step_offset, ch, nwg, mats);
    return hipGetLastError();
}
#endif

#if SPIN_PART == 2 || SPIN_PART == 3
template <typename T>
hipError_t launch_pass_slots(const PassShape& sh, void* psi, const DevPass* passes, const DevStage* stages, const DevOp<T>* ops,
               int pass_index, int64_t tiles_per_wg, int nwg, double* partials, int64_t step_offset, int ch,
               hipStream_t st) {
#define SPIN_SLOTS(RR, NTT, XX)                                                                   \
    if (sh.r == RR && sh.nt == NTT && sh.exchange == XX)                                          \
        return sh.profile                                                                         \
                   ? pass_one<T, RR, NTT, 0, true, XX>(sh.writes, psi, passes, stages, ops,       \
                                                       pass_index, tiles_per_wg, nwg, partials,   \
                                                       step_offset, ch, nullptr, st)              \
                   : pass_one<T, RR, NTT, 0, false, XX>(sh.writes, psi, passes, stages, ops,      \
                                                        pass_index, tiles_per_wg, nwg, partials,  \
                                                        step_offset, ch, nullptr, st);
    if constexpr (sizeof(T) == 4) {
        SPIN_SLOTS(5, 512, kHalfTiles) SPIN_SLOTS(6, 256, kHalfTiles)
        SPIN_SLOTS(2, 256, kSmallTiles) SPIN_SLOTS(3, 256, kSmallTiles) SPIN_SLOTS(4, 256, kSmallTiles)
        SPIN_SLOTS(4, 512, kSmallTiles)
    } else {
        SPIN_SLOTS(4, 512, kHalfTiles) SPIN_SLOTS(5, 256, kHalfTiles) SPIN_SLOTS(5, 512, kHalfTiles)
        SPIN_SLOTS(2, 256, kSmallTiles) SPIN_SLOTS(3, 256, kSmallTiles) SPIN_SLOTS(4, 256, kSmallTiles)
    }
#undef SPIN_SLOTS
    return hipErrorInvalidValue;
}
#endif

#if SPIN_PART == 4 || SPIN_PART == 5
template <typename T>
hipError_t launch_pass_whole(const PassShape& sh, void* psi, const DevPass* passes, const DevStage* stages, const DevOp<T>* ops,
               int pass_index, int64_t tiles_per_wg, int nwg, double* partials, int64_t step_offset, int ch,
               hipStream_t st) {
    if constexpr (sizeof(T) == 4) {
        if (sh.engine == 1) {
            if (sh.r == 5 && sh.nt == 512 && sh.mats)
                return pass_one<T, 5, 512, 1>(sh.writes, psi, passes, stages, ops, pass_index,
                                              tiles_per_wg, nwg, partials, step_offset, ch, sh.mats, st);
            return hipErrorInvalidValue;
        }
    }
    if (sh.engine != 0) return hipErrorInvalidValue;
#define SPIN_PASS(RR, NTT)                                                                   \
    if (sh.r == RR && sh.nt == NTT)                                                          \
        return sh.profile                                                                    \
                   ? pass_one<T, RR, NTT, 0, true>(sh.writes, psi, passes, stages, ops, pass_index, \
                                                   tiles_per_wg, nwg, partials, step_offset, ch,   \
                                                   nullptr, st)                                    \
                   : pass_one<T, RR, NTT>(sh.writes, psi, passes, stages, ops, pass_index,          \
                                          tiles_per_wg, nwg, partials, step_offset, ch, nullptr, st);
    if constexpr (sizeof(T) == 4) {
        SPIN_PASS(5, 256) SPIN_PASS(5, 512) SPIN_PASS(4, 256) SPIN_PASS(6, 256)
        SPIN_PASS(4, 512) SPIN_PASS(4, 1024)
    } else {
        SPIN_PASS(4, 256) SPIN_PASS(5, 256) SPIN_PASS(4, 512) SPIN_PASS(3, 512) SPIN_PASS(3, 1024)
    }
#undef SPIN_PASS
    return hipErrorInvalidValue;
}
#endif

#if SPIN_PART == 0 || SPIN_PART == 1
template <typename T, int R, int NT>
static hipError_t res_one(const ResidentJob& job0, const ResidentJob* jobs, int njobs,
                          const DevStage* stages, const DevOp<T>* ops, int64_t n_steps,
                          hipStream_t st) {
    if (!jobs && job0.Pall)    // one problem with the all-site profile
        hipLaunchKernelGGL((k_resident<T, R, NT, true>), dim3(njobs), dim3(NT), 0, st, job0, jobs,
                           stages, ops, n_steps);
    else
        hipLaunchKernelGGL((k_resident<T, R, NT, false>), dim3(njobs), dim3(NT), 0, st, job0, jobs,
                           stages, ops, n_steps);
    return hipGetLastError();
}

template <typename T>
hipError_t launch_resident(int bits, const ResidentJob& job0, const ResidentJob* jobs,
                           int njobs, const DevStage* stages, const DevOp<T>* ops,
                           int64_t n_steps, hipStream_t st) {
#define SPIN_RES(BITS)                                                                             \
    if (bits == BITS)                                                                              \
        return res_one<T, kResidentRegs, 1 << (BITS - kResidentRegs)>(job0, jobs, njobs, stages,   \
                                                                     ops, n_steps, st);
    SPIN_RES(10) SPIN_RES(11) SPIN_RES(12) SPIN_RES(13)
    if constexpr (sizeof(T) == 4) {
        SPIN_RES(14)
    }
#undef SPIN_RES
    return hipErrorInvalidValue;
}
#endif

#if SPIN_PART >= 6
template <typename T>
int batch_occupancy(bool half) {
    constexpr bool F = sizeof(T) == 4;
    int n = 0;
    const hipError_t e =
        half ? hipOccupancyMaxActiveBlocksPerMultiprocessor(&n, k_batch<T, F ? 6 : 5, 256, true>, 256, 0)
             : hipOccupancyMaxActiveBlocksPerMultiprocessor(&n, k_batch<T, F ? 5 : 4, 512, false>, 512, 0);
    return e == hipSuccess ? n : 0;
}

template <typename T>
hipError_t launch_batch(int nslots, bool half, const BatchProblem* probs, const BatchJob* jobs,
                        const int* job_start, const DevPass* passes, const DevStage* stages,
                        const DevOp<T>* ops, const int2* launches, double* partials, int* sync,
                        int ngangs, int* status, int64_t n_steps, hipStream_t st) {
    // a fill kernel, not a memset node, so the pair can sit in a captured graph
    launch_sync_start(sync, kSyncGangs + ngangs, st);
    constexpr bool F = sizeof(T) == 4;
    if (half)
        hipLaunchKernelGGL((k_batch<T, F ? 6 : 5, 256, true>), dim3(nslots), dim3(256), 0, st, probs,
                           jobs, job_start, passes, stages, ops, launches, partials, sync, n_steps);
    else
        hipLaunchKernelGGL((k_batch<T, F ? 5 : 4, 512, false>), dim3(nslots), dim3(512), 0, st, probs,
                           jobs, job_start, passes, stages, ops, launches, partials, sync, n_steps);
    launch_status_or(sync + kSyncError, status, st);
    return hipGetLastError();
}
#endif

// Instantiations of the template families of this part.
#define SPIN_INST_PASS(NAME, T)                                                                            \
    template hipError_t NAME<T>(const PassShape&, void*, const DevPass*, const DevStage*, const DevOp<T>*, \
                                int, int64_t, int, double*, int64_t, int, hipStream_t);
#define SPIN_INST_RESIDENT(T)                                                                             \
    template hipError_t launch_resident<T>(int, const ResidentJob&, const ResidentJob*, int,              \
                                           const DevStage*, const DevOp<T>*, int64_t, hipStream_t);
#define SPIN_INST_BATCH(T)                                                                                \
    template int batch_occupancy<T>(bool);                                                                \
    template hipError_t launch_batch<T>(int, bool, const BatchProblem*, const BatchJob*, const int*,      \
                                        const DevPass*, const DevStage*, const DevOp<T>*, const int2*,    \
                                        double*, int*, int, int*, int64_t, hipStream_t);
#if SPIN_PART == 0
SPIN_INST_RESIDENT(float)
#elif SPIN_PART == 1
SPIN_INST_RESIDENT(double)
#elif SPIN_PART == 2
SPIN_INST_PASS(launch_pass_slots, float)
#elif SPIN_PART == 3
SPIN_INST_PASS(launch_pass_slots, double)
#elif SPIN_PART == 4
SPIN_INST_PASS(launch_pass_whole, float)
#elif SPIN_PART == 5
SPIN_INST_PASS(launch_pass_whole, double)
#elif SPIN_PART == 6
SPIN_INST_BATCH(float)
#elif SPIN_PART == 7
SPIN_INST_BATCH(double)
#endif

}  // namespace spinqp
