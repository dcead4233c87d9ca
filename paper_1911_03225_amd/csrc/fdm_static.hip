// fdm_static.hip -- static problem of the layer case on the GPU.
//
// Layer-averaged shear stress tau13 at the layer nodes for given densities
// (Morin, Brenner & Suquet, arXiv:1911.03225, sec. 3.1.2 and 3.2.1): a
// periodic cell of homogeneous isotropic elasticity (mu, lambda), n3 voxels
// high, holds a layer of h voxels carrying U^p = phi(x1,x2) e1 (x) e3.  The
// homogeneous Green-operator solution sigma^ = (C:Gamma^ - I):C:U^p^ gives,
// for this ansatz,
//     sigma13^(xi) = -mu phi^ chi^(xi3) G(xi),
//     G = xi2^2/|xi|^2 + 2/(1-nu) xi1^2 xi3^2/|xi|^4,
// so the layer average folds x3 into a 2-D multiplier:
//     tau13^ = -mu K phi^,  K = (n3/h) sum_m3 |chi^[m3]|^2 G(xi1, xi2, xi3(m3)),
// and the mean is sigma_bar_13 = 2 mu eps_bar_13 - mu (h/n3) <phi>.
// phi^ comes from the densities: alpha12 = D1 phi, alpha11 = -D2 phi are
// forward differences on the staggered grid, with Fourier symbols
// d = (e^{i 2 pi m/n} - 1)/d, inverted in least squares:
//     phi^ = (conj(d1) alpha12^ - conj(d2) alpha11^) / (|d1|^2 + |d2|^2).
//
// Two ways through a solve:
//   * three kernels of this file, where a block's lines fit its LDS (see
//     line_shape): rows (both densities as one complex line), columns (the
//     transform, the multiplier, the transform back), rows back (two real
//     rows as one complex line) with the velocity law as they leave;
//   * rocFFT otherwise (see own_transforms): the densities side by side
//     (rocFFT may overwrite its input), a batched real-to-complex transform,
//     multiplier, complex-to-real transform, velocity law.
// K is built once per plan by a kernel (FP64 sum over m3).
#pragma clang fp contract(off)
#include <hip/hip_runtime.h>
#include <rocfft/rocfft.h>

#include <algorithm>
#include <cmath>
#include <mutex>
#include <new>
#include <string>
#include <vector>

#include "fdm_fft.h"
#include "fdm_static.h"

namespace fdm {
namespace {

// sin(pi a / b) and cos(pi a / b) of whole numbers, with the rounding of the
// quotient taken back to first order (it would cost up to five units in the
// last place of a root of unity, which the solve passes on to phi).
__device__ __forceinline__ void sincos_ratio(double a, double b, double *sn, double *cs)
{
    const double q = a / b, rest = M_PI * (fma(-q, b, a) / b);
    double s, c;
    sincospi(q, &s, &c);
    *sn = fma(rest, c, s);
    *cs = fma(-rest, s, c);
}

// Tables of a plan, in double first: the weights |chi^[m3]|^2 of h voxels
// out of n3 (a Dirichlet kernel; m3 and n3 - m3 together) and xi3^2, m3 = 0
// .. n3/2; the symbols of the forward differences along x (m1 = 0 .. nx/2)
// and y, whose real part -2 sin^2 keeps its digits at small m; and, where
// twx is given, the roots of unity of both axes.
template <typename T>
__global__ __launch_bounds__(256) void tables_kernel(int nx, int ny, double dx, double dy, int h, int n3, double *c2,
                                                     double *xi3sq, T *d1, T *d2, T *twx, T *twy)
{
    const int stride = gridDim.x * blockDim.x, first = blockIdx.x * blockDim.x + threadIdx.x;
    for (int m = first; m <= n3 / 2; m += stride) {
        double s, sh, c;
        sincos_ratio(m, n3, &s, &c);
        sincos_ratio(fmod((double)m * h, 2.0 * n3), n3, &sh, &c);
        const double chi = m == 0 ? (double)h : sh / s;
        c2[m] = chi * chi / ((double)n3 * n3) * (m == 0 || 2 * m == n3 ? 1.0 : 2.0);
        const double xi = 2.0 * M_PI * m / (n3 * dx);
        xi3sq[m] = xi * xi;
    }
    auto symbols = [&](T *d, int n, int count, double spacing) {
        for (int m = first; m < count; m += stride) {
            double s, c, im;
            sincos_ratio(m, n, &s, &c);
            d[2 * m] = (T)(-2.0 * s * s / spacing);
            sincos_ratio(2.0 * m, n, &im, &c);
            d[2 * m + 1] = (T)(im / spacing);
        }
    };
    symbols(d1, nx, nx / 2 + 1, dx);
    symbols(d2, ny, ny, dy);
    if (twx == nullptr) return;
    auto roots = [&](T *tw, int n) {
        for (int m = first; m < n; m += stride) {
            double s, c;
            sincos_ratio(2.0 * m, n, &s, &c);
            tw[2 * m] = (T)c;
            tw[2 * m + 1] = (T)-s;
        }
    };
    roots(twx, nx);
    roots(twy, ny);
}

// The multiplier over the half spectrum m1 = 0 .. nx/2, FP64 throughout.
// columns: K[m1 * ny + m2] = -mu/N K / (|d1|^2 + |d2|^2), what the difference
// symbols' numerator is multiplied by; otherwise K[m2 * nxh + m1] itself.
// One reciprocal a term (two Newton steps), halves of the sum folded: 14
// instructions a term where two divisions took 60 over twice the terms.
// Measured, 321 x 384 modes, n3 = 512, double: 29 us against 96.
template <typename T>
__global__ __launch_bounds__(256) void layer_multiplier_kernel(T *K, int nx, int ny, int nxh, double dx, double dy,
                                                                int n3, const double *c2, const double *xi3sq,
                                                                double two_over_1mnu, double n3_over_h, bool columns,
                                                                double neg_mu_over_n)
{
    const int64_t idx = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (idx >= (int64_t)nxh * ny) return;
    const int m1 = (int)(columns ? idx / ny : idx % nxh), m2 = (int)(columns ? idx % ny : idx / nxh);
    const int f1 = m1 <= nx - m1 ? m1 : nx - m1;          // |signed frequency|
    const int f2 = m2 <= ny - m2 ? m2 : ny - m2;
    const double x1 = 2.0 * M_PI * f1 / (nx * dx), x2 = 2.0 * M_PI * f2 / (ny * dy);
    const double x1s = x1 * x1, x2s = x2 * x2;
    double acc = 0.0;
    if (m1 != 0 || m2 != 0) {
        const double base = x1s + x2s, b = two_over_1mnu * x1s;
        for (int m3 = 0; m3 <= n3 / 2; ++m3) {
            const double z = xi3sq[m3], s = base + z;
            double y = __builtin_amdgcn_rcp(s);
            y = fma(y, fma(-s, y, 1.0), y);
            y = fma(y, fma(-s, y, 1.0), y);
            acc = fma(c2[m3], y * fma(b * z, y, x2s), acc);
        }
        acc *= n3_over_h;
        if (columns) {
            double s1, s2, c;
            sincos_ratio(m1, nx, &s1, &c);
            sincos_ratio(m2, ny, &s2, &c);
            s1 /= dx;
            s2 /= dy;
            acc *= neg_mu_over_n / (4.0 * (s1 * s1 + s2 * s2));   // |e^{it} - 1|^2 = 4 sin^2(t/2)
        }
    }
    K[idx] = (T)acc;
}

// --------------------------------------------------------- own transforms
//
// The densities travel as z = alpha12 + i alpha11: one complex transform
// gives both spectra, alpha12^(m) = (z^(m) + conj z^(-m)) / 2 and alpha11^(m)
// = (z^(m) - conj z^(-m)) / (2 i).  Between the kernels the array is
// transposed, spec[m1 * ny + k], so that the column kernel reads and writes
// whole lines; the row kernels touch runs of `rows` complex values of it.
//
// What bounds a solve: up to 1024^2 each kernel is launch, first loads,
// barriers and the passes' own latency (a block runs each pass once, on a
// lone wave per SIMD), so there are three kernels where the library's
// transforms with their pack, multiplier and law take eight.  Measured,
// 512^2 float: rows 5.2, columns 7.8, rows back 6.0 us, 19 together, against
// 31; a whole solve with its tables 89 us against 6.0 ms with rocFFT's plans.

constexpr int kLineThreads = 256;
constexpr int kMaxPairs = 4;   // column pairs a block takes at most

extern __shared__ __align__(16) unsigned char fft_lds_raw[];

// A table on its way from memory to LDS: a thread's first kAhead values load
// at once, before the lines' own loads, and are put down after the first
// pass (one trip to memory instead of two); longer tables follow then.
template <typename V> struct Table {
    static constexpr int kAhead = 4;
    V v[kAhead];
    template <typename Load> __device__ __forceinline__ void issue(int count, Load load)
    {
#pragma unroll
        for (int u = 0; u < kAhead; ++u)
            if (u * kLineThreads < count) v[u] = load(min(u * kLineThreads + (int)threadIdx.x, count - 1));
    }
    template <typename Load> __device__ __forceinline__ void put(V *lds, int count, Load load)
    {
#pragma unroll
        for (int u = 0; u < kAhead; ++u) {
            const int t = u * kLineThreads + (int)threadIdx.x;
            if (t < count) lds[t] = v[u];
        }
        for (int t = kAhead * kLineThreads + (int)threadIdx.x; t < count; t += kLineThreads) lds[t] = load(t);
    }
};

// The block's LDS: `lines` lines twice, then (copy) the roots of unity, then
// what the caller adds.
template <typename T> struct LineLds {
    FftLds<T> m;
    const Cx<T> *table;
    Cx<T> *roots;          // their place in LDS, or null
    unsigned char *rest;
    Table<Cx<T>> ahead;
    int n;
    __device__ __forceinline__ LineLds(const T *tw, bool copy, int n_, int lines) : n(n_)
    {
        Cx<T> *base = reinterpret_cast<Cx<T> *>(fft_lds_raw);
        const int half = lines * fft_line(n);
        table = reinterpret_cast<const Cx<T> *>(tw);
        roots = copy ? base + 2 * half : nullptr;
        rest = reinterpret_cast<unsigned char *>(base + 2 * half + (copy ? n : 0));
        m = FftLds<T>{base, base + half, copy ? roots : table};
        if (copy) ahead.issue(n, [&](int i) { return table[i]; });
    }
    __device__ __forceinline__ void put_roots()
    {
        if (roots) ahead.put(roots, n, [&](int i) { return table[i]; });
    }
};

template <typename T, bool POW2>
__global__ __launch_bounds__(kLineThreads) void rows_kernel(const T *__restrict__ a11, const T *__restrict__ a12,
                                                            T *__restrict__ spec, const T *__restrict__ tw, int nx,
                                                            int ny, int rows, bool copy, FftAxis ax, SlipArgs slip)
{
    // the previous coupled step's slip update in a block of its own, ahead of
    // every reader of the mean stress and slip (the later kernels)
    if (slip.cd != nullptr && blockIdx.x == gridDim.x - 1) {
        __shared__ double2 lds[256];
        coupled_slip_block(slip, lds);
        return;
    }
    const int k0 = (int)blockIdx.x * rows, nr = min(rows, ny - k0);
    LineLds<T> l(tw, copy, nx, rows);
    // (lines that fit LDS keep every index of these kernels in 32 bits)
    a11 += (int64_t)k0 * nx;
    a12 += (int64_t)k0 * nx;
    Cx<T> *out = reinterpret_cast<Cx<T> *>(spec) + k0;
    fft_lines<false, true, POW2>(
        l.m, ax, nr,
        [&](int r, int i) {
            const unsigned at = (unsigned)(r * nx + i);
            return Cx<T>{a12[at], a11[at]};
        },
        [&](int r, int i, Cx<T> v) { out[(unsigned)(i * ny + r)] = v; }, [&] { l.put_roots(); });
}

// Columns m1 and nx - m1 side by side (`pairs` of them a block): transform,
// T = multiplier times the numerator (sigma_bar at the mean), transform back
// into the column's place.  PHI: T + i P, P = phi^ / N, into both columns
// (their transforms back give tau + i phi).  A transform's rounding is that of
// its larger part, and tau and phi share one here: so P is taken in units of
// the power of two nearest below mu (phi_unit, which is exact; tau is of the
// size of mu times phi at most), and the means stay out of it and are added to
// the nodes.  With mu = 80e9 and P as it is, phi was off by 1e-5 of itself.
template <typename T, bool PHI, bool POW2>
__global__ __launch_bounds__(kLineThreads) void columns_kernel(T *__restrict__ spec, const T *__restrict__ K,
                                                               const T *__restrict__ d1, const T *__restrict__ d2,
                                                               const T *__restrict__ tw, int nx, int ny, int pairs,
                                                               bool copy, FftAxis ay, T unit_over_n,
                                                               const CoupledDev *cd, double sigma)
{
    const int nxh = nx / 2 + 1, p0 = (int)blockIdx.x * pairs, np = min(pairs, nxh - p0);
    LineLds<T> l(tw, copy, ny, 2 * pairs);
    // the multiplier and the symbols of the block's modes, put down in LDS
    // behind the roots (where those fit)
    Cx<T> *const sym = reinterpret_cast<Cx<T> *>(l.rest);
    T *const mult = reinterpret_cast<T *>(sym + ny);
    const Cx<T> *gsym = reinterpret_cast<const Cx<T> *>(d2);
    const T *gmult = K + (int64_t)p0 * ny;
    Table<Cx<T>> sym_ahead;
    Table<T> mult_ahead;
    // (early loads too: the mean stress, and the pairs' symbols)
    const T mean_tau = PHI ? T(0) : (T)(cd ? cd->sigma_bar : sigma);
    Cx<T> sym1[kMaxPairs];
#pragma unroll
    for (int q = 0; q < kMaxPairs; ++q) sym1[q] = reinterpret_cast<const Cx<T> *>(d1)[p0 + min(q, np - 1)];
    if (copy) {
        sym_ahead.issue(ny, [&](int i) { return gsym[i]; });
        mult_ahead.issue(np * ny, [&](int i) { return gmult[i]; });
    }
    Cx<T> *cx_spec = reinterpret_cast<Cx<T> *>(spec);
    auto place = [&](int line, int k) {
        const int p = p0 + (line >> 1);
        return (unsigned)(((line & 1) == 0 || p == 0 ? p : nx - p) * ny + k);
    };
    fft_lines<false, false, POW2>(
        l.m, ay, 2 * np, [&](int line, int k) { return cx_spec[place(line, k)]; },
        [&](int line, int k, Cx<T> v) { fft_put(l.m.dst, ny, line, k, v); },
        [&] {
            l.put_roots();
            if (copy) {
                sym_ahead.put(sym, ny, [&](int i) { return gsym[i]; });
                mult_ahead.put(mult, np * ny, [&](int i) { return gmult[i]; });
            }
        });
    __syncthreads();
    {
        Cx<T> *s = l.m.src;
        l.m.src = l.m.dst;
        l.m.dst = s;
    }
    const Cx<T> *const z = l.m.src;
    // the product at mode m2 of pair q
    auto product = [&](int q, int m2) {
        const int m1 = p0 + q, mm = m2 == 0 ? 0 : ny - m2;
        const Cx<T> zp = fft_get(z, ny, 2 * q, m2), zm = fft_get(z, ny, 2 * q + 1, mm);
        const T a12r = T(0.5) * (zp.re + zm.re), a12i = T(0.5) * (zp.im - zm.im);
        const T a11r = T(0.5) * (zp.im + zm.im), a11i = T(0.5) * (zm.re - zp.re);
        const Cx<T> s2 = copy ? sym[m2] : gsym[m2];
        const T f = copy ? mult[q * ny + m2] : gmult[q * ny + m2];
        Cx<T> s1 = sym1[0];
#pragma unroll
        for (int u = 1; u < kMaxPairs; ++u)
            if (q == u) s1 = sym1[u];
        const T d1r = s1.re, d1i = s1.im, d2r = s2.re, d2i = s2.im;
        // conj(d1) a12 - conj(d2) a11
        const T nr = (d1r * a12r + d1i * a12i) - (d2r * a11r + d2i * a11i);
        const T ni = (d1r * a12i - d1i * a12r) - (d2r * a11i - d2i * a11r);
        const bool mean = m1 == 0 && m2 == 0;
        struct Out {
            Cx<T> tau, phi;
        } o{{f * nr, f * ni}, {T(0), T(0)}};
        if (mean) o.tau = Cx<T>{mean_tau, T(0)};
        if constexpr (PHI) {
            const T g = unit_over_n / ((d1r * d1r + d1i * d1i) + (d2r * d2r + d2i * d2i));
            if (!mean) o.phi = Cx<T>{g * nr, g * ni};
        }
        return o;
    };
    if constexpr (PHI) {
        // line 2 q holds T + i P at m1, line 2 q + 1 its values at -m
        fft_lines<true, false, POW2>(
            l.m, ay, 2 * np,
            [&](int line, int i) {
                if ((line & 1) == 0) {
                    const auto o = product(line >> 1, i);
                    return Cx<T>{o.tau.re - o.phi.im, o.tau.im + o.phi.re};
                }
                const auto o = product(line >> 1, i == 0 ? 0 : ny - i);
                return Cx<T>{o.tau.re + o.phi.im, o.phi.re - o.tau.im};
            },
            [&](int line, int k, Cx<T> v) {
                // a pair that is one column (m1 = 0 or nx / 2) has one writer: its two
                // lines are equal in exact arithmetic, not in bits
                const int p = p0 + (line >> 1);
                if ((line & 1) != 0 && (p == 0 || 2 * p == nx)) return;
                cx_spec[place(line, k)] = v;
            },
            [] {});
    } else {
        fft_lines<true, false, POW2>(
            l.m, ay, np, [&](int q, int i) { return product(q, i).tau; },
            [&](int q, int k, Cx<T> v) { cx_spec[(unsigned)((p0 + q) * ny + k)] = v; }, [] {});
    }
}

// The celerity of one node (float32).
template <typename T> struct LawArgs {
    T tau0, mobility, tau_y, beta;
    const float *mfield;
};
template <typename T, bool WIGGLY>
__device__ __forceinline__ float law_celerity(const LawArgs<T> &L, T tau, T phi, int64_t i)
{
    const T m = L.mfield ? L.mobility * T(L.mfield[i]) : L.mobility;
    if constexpr (WIGGLY) {
        return (float)(m * (L.tau_y * cos(phi / L.beta) - tau));
    } else {
        const T a = fabs(tau) - L.tau0;
        return (float)-(m * (a > T(0) ? copysign(a, tau) : T(0)));
    }
}

// Block maximum of |v0| (NaN once a non-finite value is seen), 256 threads.
struct AbsMax {
    float m = 0.0f;
    bool bad = false;
    __device__ __forceinline__ void take(float v)
    {
        bad |= !isfinite(v);
        m = fmaxf(m, fabsf(v));
    }
    __device__ __forceinline__ void store(float *partial)
    {
        __shared__ float lds[4];
        if (bad) m = __builtin_nanf("");
        for (int o = 32; o > 0; o >>= 1) {
            const float other = __shfl_xor(m, o, 64);
            m = (isnan(m) || isnan(other)) ? __builtin_nanf("") : fmaxf(m, other);
        }
        if ((threadIdx.x & 63) == 0) lds[threadIdx.x >> 6] = m;
        __syncthreads();
        if (threadIdx.x == 0) {
            float r = lds[0];
            for (int w = 1; w < 4; ++w) r = (isnan(r) || isnan(lds[w])) ? __builtin_nanf("") : fmaxf(r, lds[w]);
            *partial = r;
        }
    }
};

// LAW_NONE: tau13 to `tau`; otherwise the celerity to v0 and a partial of
// its maximum per block.  Without phi the spectrum's rows are conjugate
// symmetric and two of them make one complex line (row k in the real part,
// row k + 1 in the imaginary one); with phi a line is tau + i phi, without
// their means and phi in units of 1 / per_unit (see columns_kernel).
enum : int { LAW_NONE = 0, LAW_SOFT = 1, LAW_WIGGLY = 2 };

template <typename T, int LAW, bool POW2>
__global__ __launch_bounds__(kLineThreads) void rows_back_kernel(const T *__restrict__ spec, T *__restrict__ tau,
                                                                 float *__restrict__ v0, const T *__restrict__ tw,
                                                                 int nx, int ny, int rows, int groups, bool copy,
                                                                 FftAxis ax, LawArgs<T> L, const CoupledDev *cd,
                                                                 T per_unit, float *__restrict__ partial)
{
    constexpr bool PHI = LAW == LAW_WIGGLY;
    const T sigma_bar = (T)(PHI ? cd->sigma_bar : 0.0), phi_mean = (T)(PHI ? cd->phi_mean : 0.0);
    const int lines = PHI ? rows : rows / 2;
    LineLds<T> l(tw, copy, nx, lines);
    const FftLds<T> m0 = l.m;
    const Cx<T> *cx_spec = reinterpret_cast<const Cx<T> *>(spec);
    AbsMax top;
    for (int g = blockIdx.x; g < groups; g += gridDim.x) {
        const int k0 = g * rows;
        l.m = m0;
        auto leave = [&](int k, int i, T x, T phi) {
            if (k >= ny) return;
            const unsigned at = (unsigned)(k * nx + i);
            if constexpr (LAW == LAW_NONE) {
                tau[at] = x;
            } else {
                const float c = law_celerity<T, PHI>(L, x, phi, at);
                v0[at] = c;
                top.take(c);
            }
        };
        fft_lines<true, true, POW2>(
            l.m, ax, lines,
            [&](int r, int i) {
                if constexpr (PHI) {
                    return cx_spec[(unsigned)(i * ny + min(k0 + r, ny - 1))];
                } else {
                    const int k = min(k0 + 2 * r, ny - 1), half = min(i, nx - i);
                    const unsigned at = (unsigned)(half * ny + k);
                    Cx<T> a = cx_spec[at], b = k + 1 < ny ? cx_spec[at + 1] : Cx<T>{T(0), T(0)};
                    if (i == 0 || 2 * i == nx) a.im = b.im = T(0);   // real up to rounding
                    if (2 * i > nx) {                                // conjugates of the mirrored mode
                        a.im = -a.im;
                        b.im = -b.im;
                    }
                    return Cx<T>{a.re - b.im, a.im + b.re};
                }
            },
            [&](int r, int i, Cx<T> v) {
                if constexpr (PHI) {
                    leave(k0 + r, i, v.re + sigma_bar, v.im * per_unit + phi_mean);
                } else {
                    leave(k0 + 2 * r, i, v.re, T(0));
                    leave(k0 + 2 * r + 1, i, v.im, T(0));
                }
            },
            [&] {
                if (g == (int)blockIdx.x) l.put_roots();
            });
        __syncthreads();   // the halves are free for the next group's lines
    }
    if constexpr (LAW != LAW_NONE) top.store(partial + blockIdx.x);
}

// ---------------------------------------------------------- rocFFT's way

// out[m] = -mu K[m] phi^[m] / N (m != 0), out[0] = sigma_bar; spec holds the
// two transforms alpha11^ then alpha12^ (interleaved complex).
template <typename T>
__global__ __launch_bounds__(256) void green_kernel(const T *spec, T *out, const T *K, const T *d1, const T *d2,
                                                     int nxh, int ny, T neg_mu_over_n, const CoupledDev *cd, double sigma, SlipArgs slip)
{
    // the previous coupled step's slip update by block 0, whose thread 0 is
    // the one reader of what it changes in this launch (the mean mode)
    if (slip.cd != nullptr && blockIdx.x == 0) {
        __shared__ double2 lds[256];
        coupled_slip_block(slip, lds);
    }
    const int64_t idx = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    const int64_t nmodes = (int64_t)nxh * ny;
    if (idx >= nmodes) return;
    const int m1 = (int)(idx % nxh), m2 = (int)(idx / nxh);
    const T a11r = spec[2 * idx], a11i = spec[2 * idx + 1];
    const T a12r = spec[2 * (nmodes + idx)], a12i = spec[2 * (nmodes + idx) + 1];
    const T d1r = d1[2 * m1], d1i = d1[2 * m1 + 1];
    const T d2r = d2[2 * m2], d2i = d2[2 * m2 + 1];
    T re, im;
    if (idx == 0) {
        re = (T)(cd ? cd->sigma_bar : sigma);
        im = T(0);
    } else {
        // conj(d1) a12 - conj(d2) a11
        const T nr = (d1r * a12r + d1i * a12i) - (d2r * a11r + d2i * a11i);
        const T ni = (d1r * a12i - d1i * a12r) - (d2r * a11i - d2i * a11r);
        const T den = (d1r * d1r + d1i * d1i) + (d2r * d2r + d2i * d2i);
        const T f = neg_mu_over_n * K[idx] / den;
        re = f * nr;
        im = f * ni;
    }
    out[2 * idx] = re;
    out[2 * idx + 1] = im;
}

template <typename T>
__global__ __launch_bounds__(256) void pack_kernel(T *dst, const T *a11, const T *a12, int64_t n)
{
    const int64_t stride = (int64_t)gridDim.x * blockDim.x;
    for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < n; i += stride) {
        dst[i] = a11[i];
        dst[n + i] = a12[i];
    }
}

// phi^ / N at every mode (phi_mean at the mean), for a complex-to-real
// transform; spec holds alpha11^ then alpha12^.
template <typename T>
__global__ __launch_bounds__(256) void phi_kernel(const T *spec, T *out, const T *d1, const T *d2, int nxh, int ny,
                                                   T inv_n, const CoupledDev *cd, SlipArgs slip)
{
    // the previous coupled step's slip update by block 0, whose thread 0 is
    // the one reader of what it changes in this launch (the mean mode)
    if (slip.cd != nullptr && blockIdx.x == 0) {
        __shared__ double2 lds[256];
        coupled_slip_block(slip, lds);
    }
    const int64_t idx = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    const int64_t nmodes = (int64_t)nxh * ny;
    if (idx >= nmodes) return;
    const int m1 = (int)(idx % nxh), m2 = (int)(idx / nxh);
    T re, im;
    if (idx == 0) {
        re = (T)cd->phi_mean;
        im = T(0);
    } else {
        const T a11r = spec[2 * idx], a11i = spec[2 * idx + 1];
        const T a12r = spec[2 * (nmodes + idx)], a12i = spec[2 * (nmodes + idx) + 1];
        const T d1r = d1[2 * m1], d1i = d1[2 * m1 + 1];
        const T d2r = d2[2 * m2], d2i = d2[2 * m2 + 1];
        const T nr = (d1r * a12r + d1i * a12i) - (d2r * a11r + d2i * a11i);
        const T ni = (d1r * a12i - d1i * a12r) - (d2r * a11i - d2i * a11r);
        const T den = (d1r * d1r + d1i * d1i) + (d2r * d2r + d2i * d2i);
        const T f = inv_n / den;
        re = f * nr;
        im = f * ni;
    }
    out[2 * idx] = re;
    out[2 * idx + 1] = im;
}

template <typename T, bool WIGGLY>
__global__ __launch_bounds__(256) void velocity_law_kernel(const T *tau, const T *phi, float *v0, int64_t n,
                                                            LawArgs<T> L, float *partial)
{
    AbsMax top;
    const int64_t stride = (int64_t)gridDim.x * blockDim.x;
    for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < n; i += stride) {
        const float v = law_celerity<T, WIGGLY>(L, tau[i], WIGGLY ? phi[i] : T(0), i);
        v0[i] = v;
        top.take(v);
    }
    top.store(partial + blockIdx.x);
}

std::once_flag g_rocfft_once;
rocfft_status g_rocfft_setup = rocfft_status_success;

const char *rocfft_message(rocfft_status s)
{
    switch (s) {
    case rocfft_status_success: return "success";
    case rocfft_status_failure: return "failure";
    case rocfft_status_invalid_arg_value: return "invalid argument value";
    case rocfft_status_invalid_dimensions: return "invalid dimensions";
    case rocfft_status_invalid_array_type: return "invalid array type";
    case rocfft_status_invalid_strides: return "invalid strides";
    case rocfft_status_invalid_distance: return "invalid distance";
    case rocfft_status_invalid_offset: return "invalid offset";
    case rocfft_status_invalid_work_buffer: return "invalid work buffer";
    default: return "unknown rocFFT status";
    }
}

// Whether the own transforms take a plan whose lines fit.
//   A single solve: rocFFT builds two plans for it, 5 to 14 ms; three kernels
// and their tables take 45 to 150 us up to 1024^2, 0.6 ms where a line's
// length is a prime.  There, two bounds: on all the direct sums (1021^2 3.4 ms
// against 20), and on those of a line, which one block does: float, 13 x 2503
// 6.0 ms against 12.4, 13 x 3001 11.0 / 13.4, but 13 x 3511 15.1 / 12.2 and
// 13 x 4099 28 / 11.4 (double lines of that length do not fit).
//   A coupled run pays for its plan once.  In double: 512^2 48 us a step
// against rocFFT's 67, 1024^2 122 / 137, 2048^2 315 / 366, 448^2 (a factor 7)
// 66 / 76, 496^2 (31) 106 / 151; primes of 11 to 17 are among rocFFT's radices
// and faster there (float, 528^2 74 / 78, 544^2 82 / 89), as are larger ones
// (61: 114 / 150).  In float the rounding of the transforms reaches the
// float32 celerities, their maximum and so the step, and a run is to give
// what it gave before: float keeps rocFFT.
bool own_transforms(const StaticParams &q, bool once)
{
    const int px = largest_prime(q.nx), py = largest_prime(q.ny), p = std::max(px, py);
    if (once)
        return (int64_t)q.nx * q.ny * p <= (int64_t)1 << 30 &&
               std::max((int64_t)q.nx * px, (int64_t)q.ny * py) <= (int64_t)1 << 23;
    return q.f64 && (p <= 7 || (p > 17 && p <= 31));
}

// How many rows / column pairs a block of the own transforms takes, and its
// LDS bytes; fits is false where a line is too long for it.
struct LineShape {
    int rows = 0, pairs = 0;
    size_t lds_rows = 0, lds_cols = 0;
    bool copy_rows = true, copy_cols = true;   // tables in LDS
    bool fits = false;
};

LineShape line_shape(int nx, int ny, bool f64, size_t lds_limit)
{
    const size_t es = 2 * (f64 ? sizeof(double) : sizeof(float));
    auto bytes = [&](int n, int lines, bool copy) {
        return es * ((copy ? (size_t)n : 0) + 2 * (size_t)lines * fft_line(n));
    };
    // columns: the roots, the symbols (complex) and the pairs' multipliers (real) too
    auto col_bytes = [&](int pairs, bool copy) {
        return bytes(ny, 2 * pairs, copy) + (copy ? es * ny + es / 2 * (size_t)pairs * ny : 0);
    };
    LineShape s;
    s.rows = bytes(nx, 4, true) > lds_limit ? 2 : 4;
    s.pairs = ny >= 256 ? 1 : ny >= 128 ? 2 : 4;
    s.copy_rows = bytes(nx, s.rows, true) <= lds_limit;
    s.copy_cols = col_bytes(s.pairs, true) <= lds_limit;
    s.lds_rows = bytes(nx, s.rows, s.copy_rows);
    s.lds_cols = col_bytes(s.pairs, s.copy_cols);
    s.fits = s.lds_rows <= lds_limit && s.lds_cols <= lds_limit;
    return s;
}

// Static LDS of the kernels beside their lines (the slip update's sums).
constexpr size_t kStaticLds = 256 * sizeof(double2) + 64;

}  // namespace

struct StaticPlan {
    int nx = 0, ny = 0, nxh = 0;
    bool f64 = false, own = false;
    double mu = 1.0;
    void *block = nullptr;   // one allocation, everything below points into it
    void *spec = nullptr;    // own: nx * ny complex, transposed; rocFFT: 2 spectra, 2 * ny * nxh complex
    void *K = nullptr;       // ny * nxh reals
    void *d1 = nullptr;      // nxh complex
    void *d2 = nullptr;      // ny complex
    // own transforms
    void *twx = nullptr, *twy = nullptr;
    LineShape shape;
    FftAxis ax, ay;
    // rocFFT
    rocfft_plan fwd = nullptr, inv = nullptr;
    rocfft_execution_info info = nullptr;
    void *work = nullptr;
    void *real2 = nullptr;   // packed densities, 2 * nx * ny reals
    void *tau = nullptr, *phi = nullptr;   // of coupled steps, nx * ny reals
};

#define ST_HIP(call)                                                                          \
    do {                                                                                      \
        hipError_t e_ = (call);                                                               \
        if (e_ != hipSuccess) {                                                               \
            err = std::string(#call) + ": " + hipGetErrorString(e_);                          \
            return e_ == hipErrorOutOfMemory ? StaticStatus::OutOfMemory : StaticStatus::Device; \
        }                                                                                     \
    } while (0)
#define ST_FFT(call)                                                                          \
    do {                                                                                      \
        rocfft_status r_ = (call);                                                            \
        if (r_ != rocfft_status_success) {                                                    \
            err = std::string(#call) + ": " + rocfft_message(r_);                             \
            return StaticStatus::Device;                                                      \
        }                                                                                     \
    } while (0)

void static_plan_destroy(StaticPlan *p)
{
    if (!p) return;
    if (p->fwd) (void)rocfft_plan_destroy(p->fwd);
    if (p->inv) (void)rocfft_plan_destroy(p->inv);
    if (p->info) (void)rocfft_execution_info_destroy(p->info);
    for (void *b : {p->work, p->block, p->tau, p->phi})
        if (b) (void)hipFree(b);
    delete p;
}

namespace {

// Allocates the plan's one block and builds its tables on s.
template <typename T> StaticStatus build_tables(StaticPlan *p, const StaticParams &q, hipStream_t s, std::string &err)
{
    const int64_t n = (int64_t)q.nx * q.ny, nm = (int64_t)p->nxh * q.ny;
    size_t at = 0;
    auto part = [&](size_t bytes) {
        const size_t here = at;
        at += (bytes + 255) / 256 * 256;
        return here;
    };
    const size_t o_spec = part(sizeof(T) * (p->own ? 2 * n : 4 * nm)), o_K = part(sizeof(T) * nm);
    const size_t o_d1 = part(sizeof(T) * 2 * p->nxh), o_d2 = part(sizeof(T) * 2 * q.ny);
    const size_t o_c2 = part(sizeof(double) * (q.n3 / 2 + 1)), o_x3 = part(sizeof(double) * (q.n3 / 2 + 1));
    const size_t o_tx = part(p->own ? sizeof(T) * 2 * q.nx : 0), o_ty = part(p->own ? sizeof(T) * 2 * q.ny : 0);
    const size_t o_real = part(p->own ? 0 : sizeof(T) * 2 * n);
    ST_HIP(hipMalloc(&p->block, at));
    char *b = static_cast<char *>(p->block);
    p->spec = b + o_spec;
    p->K = b + o_K;
    p->d1 = b + o_d1;
    p->d2 = b + o_d2;
    if (p->own) {
        p->twx = b + o_tx;
        p->twy = b + o_ty;
    } else {
        p->real2 = b + o_real;
    }
    double *c2 = reinterpret_cast<double *>(b + o_c2), *x3 = reinterpret_cast<double *>(b + o_x3);
    const int longest = std::max(std::max(q.nx, q.ny), q.n3);
    hipLaunchKernelGGL(tables_kernel<T>, dim3((unsigned)std::min((longest + 255) / 256, 256)), dim3(256), 0, s, q.nx,
                       q.ny, q.dx, q.dy, q.h, q.n3, c2, x3, (T *)p->d1, (T *)p->d2, (T *)p->twx, (T *)p->twy);
    ST_HIP(hipGetLastError());
    const double nu = q.lambda / (2.0 * (q.lambda + q.mu));
    hipLaunchKernelGGL(layer_multiplier_kernel<T>, dim3((unsigned)((nm + 255) / 256)), dim3(256), 0, s, (T *)p->K, q.nx,
                       q.ny, p->nxh, q.dx, q.dy, q.n3, (const double *)c2, (const double *)x3, 2.0 / (1.0 - nu),
                       (double)q.n3 / q.h, p->own, -q.mu / (double)n);
    ST_HIP(hipGetLastError());
    return StaticStatus::Ok;
}

StaticStatus build_rocfft(StaticPlan *p, const StaticParams &q, std::string &err)
{
    std::call_once(g_rocfft_once, [] { g_rocfft_setup = rocfft_setup(); });
    if (g_rocfft_setup != rocfft_status_success) {
        err = std::string("rocfft_setup: ") + rocfft_message(g_rocfft_setup);
        return StaticStatus::Device;
    }
    const rocfft_precision prec = q.f64 ? rocfft_precision_double : rocfft_precision_single;
    const size_t len[2] = {(size_t)q.nx, (size_t)q.ny};   // fastest first
    ST_FFT(rocfft_plan_create(&p->fwd, rocfft_placement_notinplace, rocfft_transform_type_real_forward, prec, 2, len,
                              2, nullptr));
    ST_FFT(rocfft_plan_create(&p->inv, rocfft_placement_notinplace, rocfft_transform_type_real_inverse, prec, 2, len,
                              1, nullptr));
    size_t w1 = 0, w2 = 0;
    ST_FFT(rocfft_plan_get_work_buffer_size(p->fwd, &w1));
    ST_FFT(rocfft_plan_get_work_buffer_size(p->inv, &w2));
    ST_FFT(rocfft_execution_info_create(&p->info));
    const size_t w = w1 > w2 ? w1 : w2;
    if (w > 0) {
        ST_HIP(hipMalloc(&p->work, w));
        ST_FFT(rocfft_execution_info_set_work_buffer(p->info, p->work, w));
    }
    return StaticStatus::Ok;
}

}  // namespace

StaticStatus static_plan_create(const StaticParams &q, bool once, hipStream_t s, StaticPlan **out, std::string &err)
{
    *out = nullptr;
    StaticPlan *p = new (std::nothrow) StaticPlan;
    if (!p) {
        err = "host allocation failed";
        return StaticStatus::OutOfMemory;
    }
    p->nx = q.nx;
    p->ny = q.ny;
    p->nxh = q.nx / 2 + 1;
    p->f64 = q.f64;
    p->mu = q.mu;
    int dev = 0, lds = 0;
    if (hipGetDevice(&dev) != hipSuccess ||
        hipDeviceGetAttribute(&lds, hipDeviceAttributeMaxSharedMemoryPerBlock, dev) != hipSuccess)
        lds = 0;
    p->shape = line_shape(q.nx, q.ny, q.f64, (size_t)std::max<int64_t>(0, lds - (int64_t)kStaticLds));
    p->own = p->shape.fits && own_transforms(q, once);
    if (p->own) {
        p->ax = fft_axis(q.nx);
        p->ay = fft_axis(q.ny);
    }
    StaticStatus st = q.f64 ? build_tables<double>(p, q, s, err) : build_tables<float>(p, q, s, err);
    if (st == StaticStatus::Ok && !p->own) st = build_rocfft(p, q, err);
    if (st != StaticStatus::Ok) {
        (void)hipStreamSynchronize(s);   // the tables' kernels write into the block
        static_plan_destroy(p);
        return st;
    }
    *out = p;
    return StaticStatus::Ok;
}

namespace {

int row_groups(const StaticPlan *p) { return (p->ny + p->shape.rows - 1) / p->shape.rows; }

// What a solve produces: tau13 (law null), or the celerity field.
struct SolveOut {
    void *tau = nullptr;
    const LawParams *law = nullptr;
    float *v0 = nullptr, *partial = nullptr;
};

template <typename T> LawArgs<T> law_args(const LawParams &L)
{
    return LawArgs<T>{(T)L.tau0, (T)L.mobility, (T)L.tau_y, (T)L.beta, L.mfield};
}

template <typename T>
StaticStatus run_own(StaticPlan *p, const void *a11, const void *a12, const SolveOut &out, const CoupledDev *cd,
                     double sigma, const SlipArgs *slip, hipStream_t s, std::string &err)
{
    SlipArgs sa{};
    if (slip) sa = *slip;
    const int nx = p->nx, ny = p->ny, groups = row_groups(p);
    const dim3 threads(kLineThreads);
    T *spec = (T *)p->spec;
    const bool px = fft_pow2(nx), py = fft_pow2(ny);
    auto forward = [&](auto kernel) {
        hipLaunchKernelGGL(kernel, dim3((unsigned)(groups + (slip ? 1 : 0))), threads, p->shape.lds_rows, s,
                           (const T *)a11, (const T *)a12, spec, (const T *)p->twx, nx, ny, p->shape.rows,
                           p->shape.copy_rows, p->ax, sa);
    };
    if (px) forward(rows_kernel<T, true>);
    else forward(rows_kernel<T, false>);
    ST_HIP(hipGetLastError());
    const bool wiggly = out.law && out.law->wiggly;
    const dim3 cols((unsigned)((p->nxh + p->shape.pairs - 1) / p->shape.pairs));
    // (an exponent that keeps 2^e and 2^-e finite)
    const int e = wiggly ? std::max(-1000, std::min(1000, std::ilogb(p->mu))) : 0;
    const T unit_over_n = (T)std::ldexp(1.0 / ((double)nx * (double)ny), e), per_unit = (T)std::ldexp(1.0, -e);
    auto columns = [&](auto kernel) {
        hipLaunchKernelGGL(kernel, cols, threads, p->shape.lds_cols, s, spec, (const T *)p->K, (const T *)p->d1,
                           (const T *)p->d2, (const T *)p->twy, nx, ny, p->shape.pairs, p->shape.copy_cols, p->ay,
                           unit_over_n, cd, sigma);
    };
    if (wiggly && py) columns(columns_kernel<T, true, true>);
    else if (wiggly) columns(columns_kernel<T, true, false>);
    else if (py) columns(columns_kernel<T, false, true>);
    else columns(columns_kernel<T, false, false>);
    ST_HIP(hipGetLastError());
    auto back = [&](auto kernel, const LawArgs<T> &L) {
        hipLaunchKernelGGL(kernel, dim3((unsigned)std::min(groups, kLawBlocks)), threads, p->shape.lds_rows, s,
                           (const T *)spec, (T *)out.tau, out.v0, (const T *)p->twx, nx, ny, p->shape.rows, groups,
                           p->shape.copy_rows, p->ax, L, cd, per_unit, out.partial);
    };
    const LawArgs<T> L = out.law ? law_args<T>(*out.law) : LawArgs<T>{};
    if (!out.law && px) back(rows_back_kernel<T, LAW_NONE, true>, L);
    else if (!out.law) back(rows_back_kernel<T, LAW_NONE, false>, L);
    else if (wiggly && px) back(rows_back_kernel<T, LAW_WIGGLY, true>, L);
    else if (wiggly) back(rows_back_kernel<T, LAW_WIGGLY, false>, L);
    else if (px) back(rows_back_kernel<T, LAW_SOFT, true>, L);
    else back(rows_back_kernel<T, LAW_SOFT, false>, L);
    ST_HIP(hipGetLastError());
    return StaticStatus::Ok;
}

int law_blocks(int64_t n) { return (int)std::min<int64_t>((n + 255) / 256, kLawBlocks); }

template <typename T>
StaticStatus run_rocfft(StaticPlan *p, const void *a11, const void *a12, const SolveOut &out, const CoupledDev *cd,
                        double sigma, const SlipArgs *slip, hipStream_t s, std::string &err)
{
    SlipArgs sa{};
    if (slip) sa = *slip;
    const int64_t n = (int64_t)p->nx * p->ny, nm = (int64_t)p->nxh * p->ny;
    const bool wiggly = out.law && out.law->wiggly;
    void *const tau = out.law ? p->tau : out.tau;
    ST_FFT(rocfft_execution_info_set_stream(p->info, s));
    const unsigned gb = (unsigned)((nm + 255) / 256);
    if (a11) {   // else the densities are in place already
        const unsigned pb = (unsigned)std::min<int64_t>((n + 255) / 256, 4096);
        hipLaunchKernelGGL(pack_kernel<T>, dim3(pb), dim3(256), 0, s, (T *)p->real2, (const T *)a11, (const T *)a12, n);
        ST_HIP(hipGetLastError());
    }
    void *in[1] = {p->real2}, *outb[1] = {p->spec};
    ST_FFT(rocfft_execute(p->fwd, in, outb, p->info));
    if (wiggly) {
        // phi^ into the (consumed) packed-input buffer, then to the nodes
        hipLaunchKernelGGL(phi_kernel<T>, dim3(gb), dim3(256), 0, s, (const T *)p->spec, (T *)p->real2,
                           (const T *)p->d1, (const T *)p->d2, p->nxh, p->ny, (T)(1.0 / (double)n), cd, sa);
        sa.cd = nullptr;   // taken
        ST_HIP(hipGetLastError());
        void *pin[1] = {p->real2}, *pout[1] = {p->phi};
        ST_FFT(rocfft_execute(p->inv, pin, pout, p->info));
    }
    // the product overwrites alpha11^ in place: each thread reads its own
    // mode of both spectra before writing that mode
    hipLaunchKernelGGL(green_kernel<T>, dim3(gb), dim3(256), 0, s, (const T *)p->spec, (T *)p->spec, (const T *)p->K,
                       (const T *)p->d1, (const T *)p->d2, p->nxh, p->ny, (T)(-p->mu / (double)n), cd, sigma, sa);
    ST_HIP(hipGetLastError());
    void *in2[1] = {p->spec}, *out2[1] = {tau};
    ST_FFT(rocfft_execute(p->inv, in2, out2, p->info));
    if (!out.law) return StaticStatus::Ok;
    const unsigned b = (unsigned)law_blocks(n);
    if (wiggly)
        hipLaunchKernelGGL((velocity_law_kernel<T, true>), dim3(b), dim3(256), 0, s, (const T *)p->tau,
                           (const T *)p->phi, out.v0, n, law_args<T>(*out.law), out.partial);
    else
        hipLaunchKernelGGL((velocity_law_kernel<T, false>), dim3(b), dim3(256), 0, s, (const T *)p->tau,
                           (const T *)nullptr, out.v0, n, law_args<T>(*out.law), out.partial);
    ST_HIP(hipGetLastError());
    return StaticStatus::Ok;
}

StaticStatus solve(StaticPlan *p, const void *a11, const void *a12, const SolveOut &out, const CoupledDev *cd,
                   double sigma, const SlipArgs *slip, hipStream_t s, std::string &err)
{
    if (p->own)
        return p->f64 ? run_own<double>(p, a11, a12, out, cd, sigma, slip, s, err)
                      : run_own<float>(p, a11, a12, out, cd, sigma, slip, s, err);
    return p->f64 ? run_rocfft<double>(p, a11, a12, out, cd, sigma, slip, s, err)
                  : run_rocfft<float>(p, a11, a12, out, cd, sigma, slip, s, err);
}

}  // namespace

static_assert(kLawBlocks <= kMaxPartials, "the stage kernels reduce at most kMaxPartials partials");
int static_plan_partials(const StaticPlan *p)
{
    return p->own ? std::min(row_groups(p), kLawBlocks) : law_blocks((int64_t)p->nx * p->ny);
}

StaticStatus static_plan_prepare(StaticPlan *p, const LawParams &law, std::string &err)
{
    if (p->own) return StaticStatus::Ok;
    const size_t bytes = (p->f64 ? sizeof(double) : sizeof(float)) * (size_t)p->nx * (size_t)p->ny;
    if (!p->tau) ST_HIP(hipMalloc(&p->tau, bytes));
    if (law.wiggly && !p->phi) ST_HIP(hipMalloc(&p->phi, bytes));
    return StaticStatus::Ok;
}

bool static_plan_input(StaticPlan *p, void **a11, void **a12)
{
    if (p->own) return false;
    const size_t es = p->f64 ? sizeof(double) : sizeof(float);
    *a11 = p->real2;
    *a12 = static_cast<char *>(p->real2) + es * (size_t)p->nx * (size_t)p->ny;
    return true;
}

StaticStatus static_plan_run(StaticPlan *p, const void *a11, const void *a12, void *tau13, double sigma_bar,
                             hipStream_t s, std::string &err)
{
    SolveOut out;
    out.tau = tau13;
    return solve(p, a11, a12, out, nullptr, sigma_bar, nullptr, s, err);
}

StaticStatus static_plan_celerity(StaticPlan *p, const void *a11, const void *a12, const LawParams &law,
                                  const CoupledDev *cd, const SlipArgs *slip, float *v0, float *partial,
                                  hipStream_t s, std::string &err)
{
    SolveOut out;
    out.law = &law;
    out.v0 = v0;
    out.partial = partial;
    return solve(p, a11, a12, out, cd, 0.0, slip, s, err);
}

}  // namespace fdm
