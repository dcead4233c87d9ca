// fdm_fft.h -- transforms of the static solve: one-dimensional complex FFTs
// of whole lines by one block, for any length whose lines fit its LDS.
//
// Stockham's autosort form: pass after pass reads n / r butterflies of radix
// r from one half of the LDS and writes them, sorted, to the other.  The
// first pass takes its inputs straight from where the caller has them and
// the last hands its outputs over (both in runs of consecutive indices), so
// a transform of k passes makes k - 1 trips through LDS.  Radices 8, 4, 2, 3
// and 5 are written out; any other prime is one pass of direct sums (each
// output a sum over the p inputs, in double), so there is no length that
// needs padding or convolution.  Twiddles come from one table of the n-th
// roots of unity, rounded once from double.
//
// LDS layout: complex values, one of padding after every eight, so that the
// first passes' strided writes (strides 1 .. 64 times the radix) spread over
// the banks.  A pass issues all its reads before the first is used.
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

// Products and sums of the transforms contract into fused multiply-adds.
#pragma clang fp contract(fast)

namespace fdm {

constexpr int kMaxPasses = 13;   // 2^13 is beyond what a line may hold

// Factors of a line's length, in the order of the passes.
struct FftAxis {
    int32_t n = 0, passes = 0;
    int32_t staged = 0;   // a prime radix, or a single pass: through LDS before and after
    int32_t radix[kMaxPasses];
};

inline int largest_prime(int n)
{
    int top = 1;
    for (int p = 2; (int64_t)p * p <= n; ++p)
        while (n % p == 0) {
            top = p;
            n /= p;
        }
    return n > 1 ? (n > top ? n : top) : top;
}

// n into radices 8, 4, 2, 3, 5 and remaining primes (largest radices first).
inline FftAxis fft_axis(int n)
{
    FftAxis a;
    a.n = n;
    int m = n;
    auto take = [&](int r) {
        while (m % r == 0 && a.passes < kMaxPasses) {
            a.radix[a.passes++] = r;
            m /= r;
        }
    };
    take(8);
    take(4);
    take(2);
    take(3);
    take(5);
    a.staged = m > 1 || a.passes < 2;
    for (int p = 7; m > 1 && p <= m; p += 2) take(p);
    return a;
}

// Complex values that one line takes in LDS: padded.
__host__ __device__ inline int fft_line(int n) { return n + (n >> 3) + 1; }
__device__ __forceinline__ int fft_at(int i) { return i + (i >> 3); }

template <typename T> struct alignas(2 * sizeof(T)) Cx {
    T re, im;
};
template <typename T> __device__ __forceinline__ Cx<T> operator+(Cx<T> a, Cx<T> b) { return {a.re + b.re, a.im + b.im}; }
template <typename T> __device__ __forceinline__ Cx<T> operator-(Cx<T> a, Cx<T> b) { return {a.re - b.re, a.im - b.im}; }
template <typename T> __device__ __forceinline__ Cx<T> mul(Cx<T> a, Cx<T> b)
{
    return {a.re * b.re - a.im * b.im, a.re * b.im + a.im * b.re};
}
// times -i (forward) or +i (inverse)
template <bool INV, typename T> __device__ __forceinline__ Cx<T> turn(Cx<T> a)
{
    return INV ? Cx<T>{-a.im, a.re} : Cx<T>{a.im, -a.re};
}

template <int R, bool INV, typename T> __device__ __forceinline__ void butterfly(Cx<T> (&v)[R])
{
    if constexpr (R == 2) {
        const Cx<T> a = v[0], b = v[1];
        v[0] = a + b;
        v[1] = a - b;
    } else if constexpr (R == 3) {
        const Cx<T> s = v[1] + v[2], d = turn<INV>(v[1] - v[2]);
        const T c = T(0.86602540378443864676);
        const Cx<T> m = {v[0].re - T(0.5) * s.re, v[0].im - T(0.5) * s.im};
        v[0] = v[0] + s;
        v[1] = {m.re + c * d.re, m.im + c * d.im};
        v[2] = {m.re - c * d.re, m.im - c * d.im};
    } else if constexpr (R == 4) {
        const Cx<T> a = v[0] + v[2], b = v[0] - v[2], c = v[1] + v[3], d = turn<INV>(v[1] - v[3]);
        v[0] = a + c;
        v[1] = b + d;
        v[2] = a - c;
        v[3] = b - d;
    } else if constexpr (R == 5) {
        const T c1 = T(0.30901699437494742410), c2 = T(-0.80901699437494742410);
        const T s1 = T(0.95105651629515357212), s2 = T(0.58778525229247312917);
        const Cx<T> p = v[1] + v[4], q = v[2] + v[3], d = turn<INV>(v[1] - v[4]), e = turn<INV>(v[2] - v[3]);
        const Cx<T> a = {v[0].re + c1 * p.re + c2 * q.re, v[0].im + c1 * p.im + c2 * q.im};
        const Cx<T> b = {v[0].re + c2 * p.re + c1 * q.re, v[0].im + c2 * p.im + c1 * q.im};
        const Cx<T> f = {s1 * d.re + s2 * e.re, s1 * d.im + s2 * e.im};
        const Cx<T> g = {s2 * d.re - s1 * e.re, s2 * d.im - s1 * e.im};
        v[0] = v[0] + p + q;
        v[1] = a + f;
        v[2] = b + g;
        v[3] = b - g;
        v[4] = a - f;
    } else {
        static_assert(R == 8, "radix");
        const T h = T(0.70710678118654752440);
        Cx<T> e[4] = {v[0], v[2], v[4], v[6]}, o[4] = {v[1], v[3], v[5], v[7]};
        butterfly<4, INV>(e);
        butterfly<4, INV>(o);
        // o[k] times the 8th root of unity to the k
        const Cx<T> t1 = turn<INV>(o[1]), t3 = turn<INV>(o[3]);
        o[1] = {h * (o[1].re + t1.re), h * (o[1].im + t1.im)};
        o[2] = turn<INV>(o[2]);
        o[3] = {h * (t3.re - o[3].re), h * (t3.im - o[3].im)};
#pragma unroll
        for (int k = 0; k < 4; ++k) {
            v[k] = e[k] + o[k];
            v[k + 4] = e[k] - o[k];
        }
    }
}

// floor(i / d) and the remainder for 0 <= i < 2^21 (a product with the
// rounded reciprocal is within 1/2 of a unit of i / d there)
__device__ __forceinline__ void div_small(int i, int d, float inv, int &q, int &r)
{
    q = (int)(((float)i + 0.5f) * inv);
    r = i - q * d;
}

// The lines of one block: `lines` of them, in two halves of LDS.
template <typename T> struct FftLds {
    Cx<T> *src, *dst;     // halves in use: lines * fft_line(n) values each
    const Cx<T> *tw;      // n roots of unity e^{-2 pi i k / n} (in LDS, or the
                          // plan's table where they do not fit)
};

template <typename T> __device__ __forceinline__ Cx<T> fft_get(const Cx<T> *half, int n, int line, int i)
{
    return half[line * fft_line(n) + fft_at(i)];
}
template <typename T> __device__ __forceinline__ void fft_put(Cx<T> *half, int n, int line, int i, Cx<T> v)
{
    half[line * fft_line(n) + fft_at(i)] = v;
}

// One pass.  FIRST takes load(line, i) instead of the source half, LAST
// gives store(line, i, value) instead of writing the other half.  LINES: the
// lines go fastest over the threads (for callers whose lines lie side by
// side in memory), else the butterflies.
enum : int { PASS_FIRST = 0, PASS_MID = 1, PASS_LAST = 2 };
template <int W> struct PassTag {
    static constexpr int value = W;
};

//
// EVEN: the strides between a butterfly's inputs, and between its outputs,
// are multiples of eight, so their padded places are evenly spaced too: one
// addition a value instead of four instructions (a lone wave per SIMD walks
// these passes, and addresses were half of what it issued).
template <int R, bool INV, int WHICH, bool LINES, bool EVEN, typename T, typename Load, typename Store>
__device__ __forceinline__ void fft_pass_as(const FftLds<T> &m, int n, int lines, int ns, Load load, Store store)
{
    const int per = n / R, step = per / ns;
    const float inv_major = 1.0f / (float)(LINES ? lines : per), inv_ns = 1.0f / (float)ns;
    for (int t = threadIdx.x; t < lines * per; t += blockDim.x) {
        int line, j, b = 0, k = 0;
        if constexpr (LINES) div_small(t, lines, inv_major, j, line);
        else div_small(t, per, inv_major, line, j);
        if constexpr (WHICH == PASS_MID) div_small(j, ns, inv_ns, b, k);
        if constexpr (WHICH == PASS_LAST) k = j;   // ns * R = n: one group
        Cx<T> v[R], w[R];
        const int at = line * fft_line(n), in0 = at + fft_at(j), in_step = per + (per >> 3);
#pragma unroll
        for (int q = 0; q < R; ++q) {
            if constexpr (WHICH == PASS_FIRST) v[q] = load(line, j + q * per);
            else if constexpr (EVEN) v[q] = m.src[in0 + q * in_step];
            else v[q] = m.src[at + fft_at(j + q * per)];
        }
        if constexpr (WHICH != PASS_FIRST) {
            const int e = k * step;
#pragma unroll
            for (int q = 1; q < R; ++q) w[q] = m.tw[q * e];
#pragma unroll
            for (int q = 1; q < R; ++q) v[q] = mul(v[q], INV ? Cx<T>{w[q].re, -w[q].im} : w[q]);
        }
        butterfly<R, INV>(v);
        const int o = WHICH == PASS_FIRST ? R * j : b * ns * R + k;
        const int out0 = at + fft_at(o), out_step = ns + (ns >> 3);
#pragma unroll
        for (int q = 0; q < R; ++q) {
            if constexpr (WHICH == PASS_LAST) store(line, o + q * ns, v[q]);
            else if constexpr (WHICH == PASS_FIRST && (R == 8 || R == 4 || R == 2)) m.dst[out0 + q] = v[q];
            else if constexpr (EVEN && WHICH == PASS_MID) m.dst[out0 + q * out_step] = v[q];
            else m.dst[at + fft_at(o + q * ns)] = v[q];
        }
    }
}

template <int R, bool INV, int WHICH, bool LINES, bool POW2, typename T, typename Load, typename Store>
__device__ __forceinline__ void fft_pass(const FftLds<T> &m, int n, int lines, int ns, Load load, Store store)
{
    if constexpr (WHICH == PASS_FIRST || POW2) {
        fft_pass_as<R, INV, WHICH, LINES, POW2>(m, n, lines, ns, load, store);
    } else {
        const int per = n / R;
        if ((per & 7) == 0 && (WHICH == PASS_LAST || (ns & 7) == 0))
            fft_pass_as<R, INV, WHICH, LINES, true>(m, n, lines, ns, load, store);
        else
            fft_pass_as<R, INV, WHICH, LINES, false>(m, n, lines, ns, load, store);
    }
}

// A prime radix p: each output of a butterfly on its own.
template <bool INV, typename T>
__device__ void fft_pass_prime(const FftLds<T> &m, int n, int lines, int ns, int p)
{
    const int per = n / p, step = per / ns;
    const float inv_n = 1.0f / (float)n, inv_per = 1.0f / (float)per, inv_ns = 1.0f / (float)ns;
    for (int t = threadIdx.x; t < lines * n; t += blockDim.x) {
        int line, u, q, j, b, k;
        div_small(t, n, inv_n, line, u);
        div_small(u, per, inv_per, q, j);
        div_small(j, ns, inv_ns, b, k);
        const int de = k * step + q * per;   // < n: the exponent's step over the inputs
        // eight interleaved sums: their chains overlap and round less than one
        constexpr int kSums = 8;
        double re[kSums] = {}, im[kSums] = {};
        int e = 0;
        for (int i = 0; i < p; i += kSums) {
#pragma unroll
            for (int u = 0; u < kSums; ++u) {
                if (i + u < p) {
                    const Cx<T> x = fft_get(m.src, n, line, j + (i + u) * per);
                    const Cx<T> w = m.tw[e];
                    const double c = w.re, s = INV ? -w.im : w.im;
                    re[u] += x.re * c - x.im * s;
                    im[u] += x.re * s + x.im * c;
                    e += de;
                    if (e >= n) e -= n;
                }
            }
        }
#pragma unroll
        for (int w = kSums / 2; w > 0; w >>= 1)
#pragma unroll
            for (int u = 0; u < w; ++u) {
                re[u] += re[u + w];
                im[u] += im[u + w];
            }
        fft_put(m.dst, n, line, b * ns * p + k + q * ns, Cx<T>{(T)re[0], (T)im[0]});
    }
}

// Transforms the block's lines from load(line, i) to store(line, i, value).
// after_first runs once between the first writes to LDS and the barrier
// behind them (for tables that have to be there from the second pass on).
// Ends without a barrier; load may read m.src and store write m.dst as they
// are when each is called.
//
// POW2: n is a power of two of at least 64, so every pass but the last has
// radix 8, the last 8, 4 or 2, and all strides are even (see EVEN).  A block
// runs through its code about once, so a good part of its time is fetching
// it: without the other radices 512^2 takes 5.4 / 7.7 / 5.9 us (rows, columns,
// rows back) instead of 5.9 / 9.2 / 6.8.
inline bool fft_pow2(int n) { return n >= 64 && (n & (n - 1)) == 0; }

template <bool INV, bool LINES, bool POW2, typename T, typename Load, typename Store, typename After>
__device__ __forceinline__ void fft_lines(FftLds<T> &m, const FftAxis &a, int lines, Load load, Store store,
                                          After after_first)
{
    auto swap = [&] {
        Cx<T> *s = m.src;
        m.src = m.dst;
        m.dst = s;
    };
    auto pass = [&](auto which, int r, int ns) {
        constexpr int W = decltype(which)::value;
        if constexpr (POW2) {
            if (W != PASS_LAST || r == 8) fft_pass<8, INV, W, LINES, true>(m, a.n, lines, ns, load, store);
            else if (r == 4) fft_pass<4, INV, W, LINES, true>(m, a.n, lines, ns, load, store);
            else fft_pass<2, INV, W, LINES, true>(m, a.n, lines, ns, load, store);
            return;
        } else
        switch (r) {
        case 8: fft_pass<8, INV, W, LINES, false>(m, a.n, lines, ns, load, store); break;
        case 4: fft_pass<4, INV, W, LINES, false>(m, a.n, lines, ns, load, store); break;
        case 2: fft_pass<2, INV, W, LINES, false>(m, a.n, lines, ns, load, store); break;
        case 3: fft_pass<3, INV, W, LINES, false>(m, a.n, lines, ns, load, store); break;
        case 5: fft_pass<5, INV, W, LINES, false>(m, a.n, lines, ns, load, store); break;
        default:
            if constexpr (W == PASS_MID) fft_pass_prime<INV>(m, a.n, lines, ns, r);
            break;
        }
    };
    int ns = 1, p = 0;
    if (!POW2 && a.staged) {
        const float inv = 1.0f / (float)(LINES ? lines : a.n);
        auto each = [&](auto f) {
            for (int t = threadIdx.x; t < lines * a.n; t += blockDim.x) {
                int line, i;
                if constexpr (LINES) div_small(t, lines, inv, i, line);
                else div_small(t, a.n, inv, line, i);
                f(line, i);
            }
        };
        each([&](int line, int i) { fft_put(m.dst, a.n, line, i, load(line, i)); });
        after_first();
        __syncthreads();
        swap();
        for (; p < a.passes; ++p) {
            pass(PassTag<PASS_MID>{}, a.radix[p], ns);
            ns *= a.radix[p];
            __syncthreads();
            swap();
        }
        each([&](int line, int i) { store(line, i, fft_get(m.src, a.n, line, i)); });
        return;
    }
    pass(PassTag<PASS_FIRST>{}, a.radix[0], 1);
    after_first();
    __syncthreads();
    swap();
    ns = a.radix[0];
    for (p = 1; p + 1 < a.passes; ++p) {
        pass(PassTag<PASS_MID>{}, a.radix[p], ns);
        ns *= a.radix[p];
        __syncthreads();
        swap();
    }
    pass(PassTag<PASS_LAST>{}, a.radix[p], ns);
}

}  // namespace fdm
#pragma clang fp contract(off)
