// fdm_line.hip -- several time steps of a one-dimensional problem (ny = 1) in
// one launch.
//
// On a single periodic row every y neighbour is the row itself, so a wave
// needs no walk and no stage buffer: it holds one column per lane, and with
// 2 halo lanes a side for every stage it can take several steps before it
// writes.  The stage kernels evaluate each row twice (the tile's extra row)
// and pay a launch per stage; what bounds a 1-D step there is the launch.
// The operations are those of the stage kernels (float: explicit multiply-
// adds; FP64: separate), so the results are the same bit for bit.
//
// kLineStages stages a launch: 16 halo lanes a side leave 32 of 64 columns
// to write.  A launch is 2.5 us of launch and first loads and a stage 0.2 us
// of a lone wave, so per stage 0.51 us at 8, 0.62 at 6, 0.41 at 12 (16 columns;
// twice the waves, which longer rows pay for).  Measured, 2048 nodes, 200
// Euler steps: 102 us against 690 with a launch per step.
#pragma clang fp contract(off)
#include "fdm_stage.h"

namespace fdm {
namespace {

constexpr int kLineStages = 8;

// Hhat (FP64 fully discrete: the node increment) at this lane's node.
template <typename R, typename S, int LK, int VK>
__device__ __forceinline__ R line_node(const InstDev &I, S wxs, S ys, R v0, R theta, R cx, R cy)
{
    constexpr bool kF64 = sizeof(R) == 8;
    constexpr bool kFD = (VK & VK_FD) != 0;
    constexpr int VH = VK & 1;
    const R V1 = R(I.V1), V2 = R(I.V2);
    const R wx = R(wxs), y = R(ys);
    const R s0 = limited_slope<LK>(y, y, y, theta);
    const R pyp = -madd(R(-0.5), s0, y), pym = -madd(R(0.5), s0, y);
    const R wl = from_left(wx), wr = from_right(wx);
    const R sx = limited_slope<LK>(wl, wx, wr, theta);
    const R pxp = madd(R(-0.5), sx, wx);
    const R pxm = from_left(madd(R(0.5), sx, wx));
    if constexpr (kFD) {
        const R sxm = from_left(sx);
        if constexpr (kF64)
            return fd_increment_ieee<VH>(wl, sxm, wx, sx, -y, -s0, -y, -s0, v0, V1, V2, I.dxd, I.dyd, I.dtd);
        else
            return fd_hamiltonian<VH>(pxm, pxp, pym, pyp, sxm, sx, -s0, -s0, v0, V1, V2, cx, cy);
    } else if constexpr (kF64 && VH == VK_LAW) {
        R hv;
        const bool ok = numerical_hamiltonian_shared(pxm, pxp, pym, pyp, v0, hv);
        if (!wave_all(both(ok, both(edge_in_range(wxs), edge_in_range(ys)))))
            hv = numerical_hamiltonian_ieee<VH>(pxm, pxp, pym, pyp, v0, V1, V2);
        return hv;
    } else if constexpr (kF64) {
        return numerical_hamiltonian_ieee<VH>(pxm, pxp, pym, pyp, v0, V1, V2);
    } else {
        return numerical_hamiltonian<VH>(pxm, pxp, pym, pyp, v0, V1, V2);
    }
}

// One stage's update of both components: a = from + dt L, from the rate at
// this node and the one to the right.  On one row Hhat does not change along
// y; the differences are taken all the same (a non-finite value stays one).
template <typename R, bool FD>
__device__ __forceinline__ void line_update(const InstDev &I, R hv, R half, R cx, R cy, R from12, R from11, R &n12,
                                            R &n11)
{
    R dx = from_right(hv) - hv, dy = hv - hv;
    if constexpr (sizeof(R) == 8 && FD) {
        dx /= I.dxd;
        dy /= I.dyd;
        n12 = from12 + dx;
        n11 = from11 - dy;
    } else if constexpr (sizeof(R) == 8) {
        divide_spacings(dx, dy, I);
        const R dt = half * I.dtd;
        n12 = from12 + dt * -dx;
        n11 = from11 + dt * dy;
    } else {
        n12 = madd(-(half * cx), dx, from12);
        n11 = madd(half * cy, dy, from11);
    }
}

template <typename R, typename S, int LK, int VK, bool FIELD>
__global__ __launch_bounds__(kWave) void line_kernel(InstDev I, int order, int steps, int halo, int dir)
{
    constexpr bool kF64 = sizeof(R) == 8;
    constexpr bool kFD = (VK & VK_FD) != 0;
    const S *s11 = static_cast<const S *>(dir ? I.w11 : I.a11), *s12 = static_cast<const S *>(dir ? I.w12 : I.a12);
    S *d11 = static_cast<S *>(dir ? I.a11 : I.w11), *d12 = static_cast<S *>(dir ? I.a12 : I.w12);
    const int lane = threadIdx.x, width = kWave - 2 * halo;
    const int64_t gcol = (int64_t)blockIdx.x * width - halo + lane;
    int col = (int)(gcol % I.nx);
    if (col < 0) col += I.nx;
    S x = s12[col], y = s11[col];
    const R v0 = FIELD ? R(I.v0f[col]) : R(I.v0);
    const R theta = kF64 ? R(I.thetad) : R(I.theta);
    const R cx = kF64 ? R(I.cxd) : R(I.cx), cy = kF64 ? R(I.cyd) : R(I.cy);
    for (int k = 0; k < steps; ++k) {
        const R b12 = R(x), b11 = R(y);
        R n12, n11;
        // first stage: all of the step, or half of it (midpoint)
        R hv = line_node<R, S, LK, VK>(I, x, y, v0, theta, cx, cy);
        line_update<R, kFD>(I, hv, order == 3 ? R(0.5) : R(1), cx, cy, b12, b11, n12, n11);
        x = S(n12);
        y = S(n11);
        if (order == 1) continue;
        hv = line_node<R, S, LK, VK>(I, x, y, v0, theta, cx, cy);
        const bool mid = order == 3;
        line_update<R, kFD>(I, hv, R(1), cx, cy, mid ? b12 : R(x), mid ? b11 : R(y), n12, n11);
        if (!mid) {
            n12 = madd(R(0.5), b12, R(0.5) * n12);
            n11 = madd(R(0.5), b11, R(0.5) * n11);
        }
        x = S(n12);
        y = S(n11);
    }
    if (lane >= halo && lane < kWave - halo && gcol < I.nx) {
        d12[col] = x;
        d11[col] = y;
    }
}

template <typename R, typename S>
hipError_t launch_line_t(const InstDev &I, int order, int steps, int dir, hipStream_t s)
{
    const int halo = 2 * (order == 1 ? 1 : 2) * steps, width = kWave - 2 * halo;
    const dim3 grid((unsigned)((I.nx + width - 1) / width)), block(kWave);
    return with_limiter<sizeof(R) == 4>(I.limiter, [&](auto t) -> hipError_t {
        constexpr int L = decltype(t)::value;
        const bool field = I.v0f != nullptr;
        auto go = [&](auto kernel) {
            hipLaunchKernelGGL(kernel, grid, block, 0, s, I, order, steps, halo, dir);
            return hipGetLastError();
        };
        switch (I.vkind) {
        case VK_PRESCRIBED: return go(line_kernel<R, S, L, VK_PRESCRIBED, false>);
        case VK_PRESCRIBED_FD: return go(line_kernel<R, S, L, VK_PRESCRIBED_FD, false>);
        case VK_LAW_FD:
            return field ? go(line_kernel<R, S, L, VK_LAW_FD, true>) : go(line_kernel<R, S, L, VK_LAW_FD, false>);
        default: return field ? go(line_kernel<R, S, L, VK_LAW, true>) : go(line_kernel<R, S, L, VK_LAW, false>);
        }
    });
}

}  // namespace

int line_steps(int order) { return order == 1 ? kLineStages : kLineStages / 2; }

hipError_t launch_line(const InstDev &I, int order, int steps, int dir, int precision, hipStream_t s)
{
    if (precision == PREC_FP32) return launch_line_t<float, float>(I, order, steps, dir, s);
    if (precision == PREC_FP64) return launch_line_t<double, double>(I, order, steps, dir, s);
    return launch_line_t<double, float>(I, order, steps, dir, s);
}

}  // namespace fdm
