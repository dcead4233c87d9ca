// fdm_kernels.hip -- reductions and helpers of the transport hot path, and
// the precision dispatch of the stage kernels (fdm_stage_f32.hip,
// fdm_stage_f64.hip).
#include "fdm_internal.h"

namespace fdm {

hipError_t launch_stage_f32(const InstDev &I, int mode, hipStream_t s);
hipError_t launch_stage_batched_f32(const InstDev *d_inst, const int32_t *d_tile_inst, int64_t total_tiles,
                                    int mode, bool fd, hipStream_t s);
hipError_t launch_stage_f64(const InstDev &I, int mode, bool f64_state, hipStream_t s);
hipError_t launch_stage_batched_f64(const InstDev *d_inst, const int32_t *d_tile_inst, int64_t total_tiles,
                                    int mode, bool fd, bool f64_state, hipStream_t s);

hipError_t launch_fused_f32(const InstDev &I, int dir, int integ, hipStream_t s);
hipError_t launch_fused_f64(const InstDev &I, int dir, int integ, bool f64_state, hipStream_t s);

hipError_t launch_fused(const InstDev &I, int dir, int integ, int precision, hipStream_t s)
{
    if (precision == PREC_FP32) return launch_fused_f32(I, dir, integ, s);
    return launch_fused_f64(I, dir, integ, precision == PREC_FP64, s);
}

hipError_t launch_stage(const InstDev &I, int mode, int precision, hipStream_t s)
{
    if (precision == PREC_FP32) return launch_stage_f32(I, mode, s);
    return launch_stage_f64(I, mode, precision == PREC_FP64, s);
}

hipError_t launch_stage_batched(const InstDev *d_inst, const int32_t *d_tile_inst, int64_t total_tiles,
                                int mode, bool fd, int precision, hipStream_t s)
{
    if (precision == PREC_FP32) return launch_stage_batched_f32(d_inst, d_tile_inst, total_tiles, mode, fd, s);
    return launch_stage_batched_f64(d_inst, d_tile_inst, total_tiles, mode, fd, precision == PREC_FP64, s);
}

namespace {

// ---------------------------------------------------------------- reductions

// Error-free sum of two doubles folded into a compensated pair.
__device__ __forceinline__ void pair_add(double &s, double &c, double s2, double c2)
{
    const double t = s + s2;
    const double bp = t - s;
    const double e = (s - (t - bp)) + (s2 - bp);
    s = t;
    c = c + c2 + e;
}

__device__ __forceinline__ double shfl_xor_d(double v, int m)
{
    return __shfl_xor(v, m, 64);
}

// Fixed-order butterfly over the wave, then over the block's waves.
__device__ void block_reduce(StatsPartial &p, StatsPartial *lds)
{
    for (int m = 1; m < 64; m <<= 1) {
        double s11 = shfl_xor_d(p.s11, m), c11 = shfl_xor_d(p.c11, m);
        double s12 = shfl_xor_d(p.s12, m), c12 = shfl_xor_d(p.c12, m);
        double sab = shfl_xor_d(p.sab, m), cab = shfl_xor_d(p.cab, m);
        double mx = shfl_xor_d(p.maxn, m), nf = shfl_xor_d(p.nonfinite, m);
        // combine in lane order so both partners compute the same value
        const bool lower = (threadIdx.x & m) == 0;
        StatsPartial a = p, b;
        b.s11 = s11; b.c11 = c11; b.s12 = s12; b.c12 = c12; b.sab = sab; b.cab = cab;
        b.maxn = mx; b.nonfinite = nf;
        StatsPartial &x = lower ? a : b;
        StatsPartial &y = lower ? b : a;
        pair_add(x.s11, x.c11, y.s11, y.c11);
        pair_add(x.s12, x.c12, y.s12, y.c12);
        pair_add(x.sab, x.cab, y.sab, y.cab);
        x.maxn = fmax(x.maxn, y.maxn);
        x.nonfinite = x.nonfinite + y.nonfinite;
        p = x;
    }
    const int wave = threadIdx.x >> 6, nw = blockDim.x >> 6;
    if ((threadIdx.x & 63) == 0) lds[wave] = p;
    __syncthreads();
    if (threadIdx.x == 0) {
        StatsPartial r = lds[0];
        for (int w = 1; w < nw; ++w) {
            pair_add(r.s11, r.c11, lds[w].s11, lds[w].c11);
            pair_add(r.s12, r.c12, lds[w].s12, lds[w].c12);
            pair_add(r.sab, r.cab, lds[w].sab, lds[w].cab);
            r.maxn = fmax(r.maxn, lds[w].maxn);
            r.nonfinite += lds[w].nonfinite;
        }
        p = r;
    }
}

__device__ __forceinline__ void neumaier(double &s, double &c, double x)
{
    const double t = s + x;
    c += fabs(s) >= fabs(x) ? (s - t) + x : (x - t) + s;
    s = t;
}

// The diagnostics of one pair of arrays by the blocks 0 .. blocks-1 of a
// launch, each of kStatsThreads threads whatever the kernel, so the order of
// the sums follows from the number of nodes alone; the largest norm is kept as
// its square (the root of the largest is the largest root, correctly rounded
// either way).  A thread's next kAhead values load together, then add in order.
template <typename S>
__device__ __forceinline__ void stats_sum(const S *__restrict__ a11, const S *__restrict__ a12, int64_t n, int block,
                                          int blocks, StatsPartial *lds, StatsPartial &p)
{
    p = StatsPartial{0, 0, 0, 0, 0, 0, 0, 0};
    constexpr int kAhead = 4;
    const int64_t stride = (int64_t)blocks * kStatsThreads;
    auto add = [&](S x, S y, bool in) {   // (a value left out adds 0, which changes no bit)
        const bool finite = isfinite(x) && isfinite(y);
        const double dx = in && finite ? (double)x : 0.0, dy = in && finite ? (double)y : 0.0;
        p.nonfinite += in && !finite ? 1.0 : 0.0;
        neumaier(p.s11, p.c11, dx);
        neumaier(p.s12, p.c12, dy);
        neumaier(p.sab, p.cab, fabs(dx) + fabs(dy));
        p.maxn = fmax(p.maxn, dx * dx + dy * dy);
    };
    int64_t i = (int64_t)block * kStatsThreads + threadIdx.x;
    for (; i + (kAhead - 1) * stride < n; i += kAhead * stride) {
        S x[kAhead], y[kAhead];
#pragma unroll
        for (int u = 0; u < kAhead; ++u) {
            x[u] = a11[i + u * stride];
            y[u] = a12[i + u * stride];
        }
#pragma unroll
        for (int u = 0; u < kAhead; ++u) add(x[u], y[u], true);
    }
    if (i < n) {
        S x[kAhead], y[kAhead];
#pragma unroll
        for (int u = 0; u < kAhead; ++u) {
            const int64_t at = i + u * stride < n ? i + u * stride : i;
            x[u] = a11[at];
            y[u] = a12[at];
        }
#pragma unroll
        for (int u = 0; u < kAhead; ++u) add(x[u], y[u], i + u * stride < n);
    }
    block_reduce(p, lds);
}

__device__ __forceinline__ void stats_out(const StatsPartial &p, double *out)
{
    out[0] = p.s11 + p.c11;
    out[1] = p.s12 + p.c12;
    out[2] = p.sab + p.cab;
    out[3] = sqrt(p.maxn);
    out[4] = p.nonfinite;
}

// One block does a small grid alone and writes the five results itself.
template <typename S>
__global__ __launch_bounds__(kStatsThreads) void stats_small_kernel(const S *__restrict__ a11,
                                                                    const S *__restrict__ a12, int64_t n,
                                                                    double *__restrict__ out)
{
    __shared__ StatsPartial lds[kStatsThreads / 64];
    StatsPartial p;
    stats_sum<S>(a11, a12, n, 0, 1, lds, p);
    if (threadIdx.x == 0) stats_out(p, out);
}

template <typename S>
__global__ __launch_bounds__(kStatsThreads) void stats_partial_kernel(const S *__restrict__ a11,
                                                                      const S *__restrict__ a12, int64_t n,
                                                                      StatsPartial *__restrict__ out)
{
    __shared__ StatsPartial lds[kStatsThreads / 64];
    StatsPartial p;
    stats_sum<S>(a11, a12, n, blockIdx.x, gridDim.x, lds, p);
    if (threadIdx.x == 0) out[blockIdx.x] = p;
}

// Every instance of a batch in one launch: row y of the grid is instance y,
// whose first stats_blocks(nodes) blocks sum it.
template <typename S>
__global__ __launch_bounds__(kStatsThreads) void stats_batched_kernel(const InstDev *__restrict__ insts,
                                                                      StatsPartial *__restrict__ out)
{
    __shared__ StatsPartial lds[kStatsThreads / 64];
    const InstDev &I = insts[blockIdx.y];
    const int64_t n = (int64_t)I.nx * I.ny;
    const int blocks = stats_blocks(n);
    if ((int)blockIdx.x >= blocks) return;
    StatsPartial p;
    stats_sum<S>(static_cast<const S *>(I.a11), static_cast<const S *>(I.a12), n, blockIdx.x, blocks, lds, p);
    if (threadIdx.x == 0) out[I.stats_first + blockIdx.x] = p;
}

// One block folds the partials of one instance in fixed order: out = {sum11,
// sum12, sum_abs, max_norm, nonfinite}.  insts (a batch) may be null: then
// `blocks` partials of the one instance.
__global__ __launch_bounds__(kStatsBlocks) void stats_final_kernel(const StatsPartial *__restrict__ parts, int blocks,
                                                                   const InstDev *__restrict__ insts,
                                                                   double *__restrict__ out)
{
    __shared__ StatsPartial lds[kStatsBlocks / 64];
    int64_t first = 0;
    if (insts) {
        const InstDev &I = insts[blockIdx.x];
        first = I.stats_first;
        blocks = stats_blocks((int64_t)I.nx * I.ny);
    }
    StatsPartial p{0, 0, 0, 0, 0, 0, 0, 0};
    if ((int)threadIdx.x < blocks) p = parts[first + (int)threadIdx.x];
    block_reduce(p, lds);
    if (threadIdx.x == 0) stats_out(p, out + 5 * blockIdx.x);
}

// Largest |v| per block (NaN if the block saw a non-finite value).  Blocks
// of 1024 threads (16 waves per CU) read four float4 each per trip, so
// enough loads are in flight to stream the field at HBM rate; a misaligned
// pointer or the last n % 4 values take the scalar loop.
constexpr int kAbsmaxThreads = 1024;

__global__ __launch_bounds__(kAbsmaxThreads) void absmax_kernel(const float *__restrict__ v, int64_t n,
                                                                float *__restrict__ partial)
{
    __shared__ float lds[kAbsmaxThreads / 64];
    float m = 0.0f;
    bool bad = false;
    auto take = [&](float x) {
        bad |= !isfinite(x);
        m = fmaxf(m, fabsf(x));
    };
    const int64_t nt = (int64_t)gridDim.x * blockDim.x;
    const int64_t tid = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    const int64_t n4 = (reinterpret_cast<uintptr_t>(v) & 15) == 0 ? n / 4 : 0;
    const float4 *__restrict__ v4 = reinterpret_cast<const float4 *>(v);
    int64_t i = tid;
    for (; i + 3 * nt < n4; i += 4 * nt) {
        float4 q[4];
#pragma unroll
        for (int u = 0; u < 4; ++u) q[u] = v4[i + u * nt];
#pragma unroll
        for (int u = 0; u < 4; ++u) {
            take(q[u].x);
            take(q[u].y);
            take(q[u].z);
            take(q[u].w);
        }
    }
    for (; i < n4; i += nt) {
        const float4 q = v4[i];
        take(q.x);
        take(q.y);
        take(q.z);
        take(q.w);
    }
    for (int64_t j = 4 * n4 + tid; j < n; j += nt) take(v[j]);
    if (bad) m = __builtin_nanf("");
    for (int o = 32; o > 0; o >>= 1) {
        const float other = __shfl_xor(m, o, 64);
        m = (isnan(m) || isnan(other)) ? __builtin_nanf("") : fmaxf(m, other);
    }
    if ((threadIdx.x & 63) == 0) lds[threadIdx.x >> 6] = m;
    __syncthreads();
    if (threadIdx.x == 0) {
        float r = lds[0];
        for (int w = 1; w < kAbsmaxThreads / 64; ++w)
            r = (isnan(r) || isnan(lds[w])) ? __builtin_nanf("") : fmaxf(r, lds[w]);
        partial[blockIdx.x] = r;
    }
}

template <typename S>
__global__ __launch_bounds__(256) void copy_kernel(S *__restrict__ dst, const S *__restrict__ src, int64_t n)
{
    const int64_t stride = (int64_t)gridDim.x * blockDim.x;
    for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < n; i += stride) dst[i] = src[i];
}

// One block: the slip update of a coupled step, and the step's scalars to
// the host's pinned mirror.
__global__ __launch_bounds__(256) void coupled_slip_kernel(SlipArgs a, CoupledDev *mirror)
{
    __shared__ double2 lds[256];
    coupled_slip_block(a, lds);
    if (threadIdx.x == 0) *mirror = *a.cd;
}

}  // namespace

hipError_t launch_coupled_slip(const SlipArgs &a, CoupledDev *mirror, hipStream_t s)
{
    hipLaunchKernelGGL(coupled_slip_kernel, dim3(1), dim3(256), 0, s, a, mirror);
    return hipGetLastError();
}

hipError_t launch_absmax(const float *v, int64_t n, float *d_partial, hipStream_t s)
{
    hipLaunchKernelGGL(absmax_kernel, dim3(kAbsmaxBlocks), dim3(kAbsmaxThreads), 0, s, v, n, d_partial);
    return hipGetLastError();
}

template <typename S>
static void stats_launches(const void *a11, const void *a12, int64_t n, StatsPartial *parts, double *out, hipStream_t s)
{
    const S *x = static_cast<const S *>(a11), *y = static_cast<const S *>(a12);
    const int blocks = stats_blocks(n);
    if (blocks == 1) {
        hipLaunchKernelGGL(stats_small_kernel<S>, dim3(1), dim3(kStatsThreads), 0, s, x, y, n, out);
        return;
    }
    hipLaunchKernelGGL(stats_partial_kernel<S>, dim3(blocks), dim3(kStatsThreads), 0, s, x, y, n, parts);
    hipLaunchKernelGGL(stats_final_kernel, dim3(1), dim3(kStatsBlocks), 0, s, (const StatsPartial *)parts, blocks,
                       (const InstDev *)nullptr, out);
}

hipError_t launch_stats(const void *a11, const void *a12, int64_t n, int precision, StatsPartial *d_partials,
                        double *out, hipStream_t s)
{
    if (precision == PREC_FP64) stats_launches<double>(a11, a12, n, d_partials, out, s);
    else stats_launches<float>(a11, a12, n, d_partials, out, s);
    return hipGetLastError();
}

hipError_t launch_stats_batched(const InstDev *d_inst, int n_inst, int most_blocks, int precision,
                                StatsPartial *d_partials, double *out, hipStream_t s)
{
    constexpr int kMostRows = 32768;   // instances a launch: a device takes 65536 blocks along y
    for (int at = 0; at < n_inst; at += kMostRows) {
        const int rows = n_inst - at < kMostRows ? n_inst - at : kMostRows;
        const InstDev *insts = d_inst + at;
        const dim3 grid(most_blocks, rows);
        if (precision == PREC_FP64)
            hipLaunchKernelGGL(stats_batched_kernel<double>, grid, dim3(kStatsThreads), 0, s, insts, d_partials);
        else
            hipLaunchKernelGGL(stats_batched_kernel<float>, grid, dim3(kStatsThreads), 0, s, insts, d_partials);
        hipLaunchKernelGGL(stats_final_kernel, dim3(rows), dim3(kStatsBlocks), 0, s, (const StatsPartial *)d_partials,
                           0, insts, out + 5 * (int64_t)at);
        const hipError_t e = hipGetLastError();
        if (e != hipSuccess) return e;
    }
    return hipSuccess;
}

hipError_t launch_copy(void *dst, const void *src, int64_t n, int precision, hipStream_t s)
{
    int64_t blocks = (n + 255) / 256;
    if (blocks > 4096) blocks = 4096;
    if (blocks < 1) blocks = 1;
    if (precision == PREC_FP64)
        hipLaunchKernelGGL(copy_kernel<double>, dim3((unsigned)blocks), dim3(256), 0, s,
                           static_cast<double *>(dst), static_cast<const double *>(src), n);
    else
        hipLaunchKernelGGL(copy_kernel<float>, dim3((unsigned)blocks), dim3(256), 0, s,
                           static_cast<float *>(dst), static_cast<const float *>(src), n);
    return hipGetLastError();
}

}  // namespace fdm
