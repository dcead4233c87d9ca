// fdm_host.hip -- host-side validation and set-up shared by the C-ABI entry
// points (declarations in fdm_host.h).
#include <hip/hip_runtime.h>

#include <algorithm>
#include <cfloat>
#include <cmath>
#include <climits>
#include <cstdio>
#include <cstring>

#include "fdm_host.h"

namespace fdm {
namespace host {

bool finite_pos(double v) { return std::isfinite(v) && v > 0.0; }

// Host-side validation of one descriptor (no HIP call).
std::string check_desc(const fdm_transport_desc &d)
{
    if (d.nx < 1 || d.ny < 1) return "nx and ny must be >= 1";
    if ((int64_t)d.nx * d.ny >= (int64_t)1 << 31) return "nx*ny must be < 2^31";
    if (d.nx >= 1 << 27) return "nx must be < 2^27 (a row of at most 1 GiB)";
    if (!finite_pos(d.dx) || !finite_pos(d.dy)) return "dx and dy must be finite and > 0";
    if (d.limiter < FDM_LIMITER_NONE || d.limiter > FDM_LIMITER_SUPERBEE) return "unknown limiter";
    if (d.limiter == FDM_LIMITER_THETA && !(d.theta >= 1.0 && d.theta <= 2.0))
        return "theta must lie in [1, 2]";
    if (d.time_order < 0 || d.time_order > 3) return "time_order must be 1, 2 or 3";
    if (d.scheme != FDM_SCHEME_SEMIDISCRETE && d.scheme != FDM_SCHEME_FULLY_DISCRETE) return "unknown scheme";
    if (d.scheme == FDM_SCHEME_FULLY_DISCRETE && d.time_order > 1)
        return "the fully discrete scheme is one pass per step: time_order must be 0 or 1";
    if (!(std::isfinite(d.dt) && d.dt >= 0.0 && d.dt <= (double)FLT_MAX))
        return "dt must be finite (as a float) and >= 0";
    if (d.dt == 0.0 && !(d.cfl > 0.0 && d.cfl <= 1.0)) return "cfl must lie in (0, 1]";
    if (d.velocity != FDM_VELOCITY_LAW && d.velocity != FDM_VELOCITY_PRESCRIBED)
        return "unknown velocity kind";
    // the kernels take velocities as float: they must stay finite there
    const auto float_finite = [](double v) { return std::isfinite(v) && std::fabs(v) <= (double)FLT_MAX; };
    if (d.velocity == FDM_VELOCITY_LAW && d.v0_field == nullptr && !float_finite(d.v0))
        return "v0 must be finite (as a float)";
    if (d.velocity == FDM_VELOCITY_PRESCRIBED && !(float_finite(d.V[0]) && float_finite(d.V[1])))
        return "V must be finite (as a float)";
    return "";
}

// Largest float not above x (x > 0).
float round_down_float(double x)
{
    float f = (float)x;
    if ((double)f > x) f = std::nextafter(f, 0.0f);
    return f;
}

// Stability bound of the step.  nu2 = dt (S1/dx + S2/dy) is the sum of the
// per-axis Courant numbers, S_i a bound on |dH/dp_i| over the grid (LAW:
// max |v0| on both axes, since |p_i| <= |p|; PRESCRIBED: |V_i|); an axis of
// one node has no differences along it and adds nothing.  Beyond nu2 = 1 the
// first-order upwind stage no longer writes each new value as a convex
// combination of old ones and is unstable in 2-D.  One forward-Euler stage
// with a limiter (time_order 1, or the fully discrete scheme) is held to
// nu2 <= 1/2, the bound of a limited (MUSCL) forward-Euler step; the paper's
// runs (Courant number 0.25 per axis, sec. 4.3-4.4) sit at exactly 1/2.
double courant_sum(const fdm_transport_desc &d, double dt, double smax_law)
{
    const double ax = d.nx > 1 ? 1.0 : 0.0, ay = d.ny > 1 ? 1.0 : 0.0;
    double s1 = smax_law, s2 = smax_law;
    if (d.velocity == FDM_VELOCITY_PRESCRIBED) {
        s1 = std::fabs((double)(float)d.V[0]);
        s2 = std::fabs((double)(float)d.V[1]);
    }
    return dt * (s1 / d.dx * ax + s2 / d.dy * ay);
}

double courant_limit(const fdm_transport_desc &d, int32_t order)
{
    return (order == 1 && d.limiter != FDM_LIMITER_NONE) ? 0.5 : 1.0;
}

// nu2 of the step a descriptor implies: a fixed dt with the given max |v0|
// (LAW), or the CFL-controlled step, for which dt max|v0| <= cfl min(dx, dy)
// whatever the celerity (LAW) and dt follows from V (PRESCRIBED).
double step_courant(const fdm_transport_desc &d, double smax_law)
{
    const double h = std::min(d.dx, d.dy);
    if (d.dt > 0.0) return courant_sum(d, (double)(float)d.dt, smax_law);
    if (d.velocity == FDM_VELOCITY_LAW) return courant_sum(d, d.cfl * h, 1.0);
    const double smax =
        std::max(std::fabs((double)(float)d.V[0]) / d.dx, std::fabs((double)(float)d.V[1]) / d.dy) * h;
    return courant_sum(d, (double)round_down_float(smax > 0.0 ? d.cfl * h / smax : d.cfl * h), 0.0);
}

// "" if the step is within the bound, else the reason.
std::string check_courant(const fdm_transport_desc &d, int32_t order, double smax_law)
{
    const double nu2 = step_courant(d, smax_law), lim = courant_limit(d, order);
    if (nu2 <= lim * (1.0 + 1e-12)) return "";
    char buf[256];
    std::snprintf(buf, sizeof(buf),
                  "dt (S1/dx + S2/dy) = %.6g exceeds %.3g (%s); lower %s", nu2, lim,
                  lim < 1.0 ? "one forward-Euler stage with a limiter" : "the 2-D Courant bound",
                  d.dt > 0.0 ? "dt" : "cfl");
    return buf;
}

// Rows per wave tile.  Each tile recomputes one extra row of Hhat and
// re-reads a few boundary rows, so long tiles are cheaper per row; but the
// launch should give every SIMD about six waves (6144 on 256 CUs x 4 SIMDs)
// to hide memory latency.  `strip_rows` is the number of (strip, row) pairs
// the launch covers (over all instances of a batched launch).  The result
// is that count / 6144 rounded up to a multiple of 4 and kept in [4, 16]
// (1024^2: 4 rows, 2048^2: 12, larger grids: 16).  The autotuner times
// fixed and SIMD-balanced heights beside it.
int pick_rows(int64_t strip_rows, int ny, int requested)
{
    if (requested > 0) return std::min(requested, ny);
    const int64_t target_waves = 256 * 4 * 6;
    int64_t rows = (strip_rows + target_waves - 1) / target_waves;
    rows = (rows + 3) / 4 * 4;
    // capped at 16: taller tiles lose on large grids (measured at 8192^2:
    // 32 rows 1.14e11, 16 rows 1.22e11, 4 rows 1.31e11 cell-updates/s; the
    // autotuner finds the last)
    rows = std::max<int64_t>(4, std::min<int64_t>(16, rows));
    return (int)std::min<int64_t>(rows, ny);
}

bool fused_applies(int32_t precision, int32_t order, bool fd)
{
    return precision == FDM_PRECISION_FP32 && (order == 2 || order == 3) && !fd;
}

// In float32 the fused kernel is faster at every size.  In the FP64 modes it
// issues 1.2 times the stage kernels' arithmetic (halo lanes and rows) at
// half their waves per SIMD, so it pays only where the two launches are bound
// by memory, that is where state, stage buffer and field exceed the 256 MB
// on-chip cache: 4096^2 with a field 330 us a step against 360 to 393
// (float32 state 297 against 316), but 1536^2 69 against 61.  One instance
// only: the batched FP64 launches have no fused form.
bool fused_by_default(const fdm_transport_desc *descs, int32_t n, int32_t precision, int32_t order)
{
    const fdm_transport_desc &d = descs[0];
    const bool fd = d.scheme == FDM_SCHEME_FULLY_DISCRETE;
    // Two single-stage steps a launch, us a step against a launch each: Euler
    // with a field 64^2 1.9 / 2.6, 512^2 3.0 / 4.0, 2048^2 13.1 / 15.6, 4096^2
    // 42 / 71; fully discrete 64^2 2.1 / 2.7, 512^2 3.5 / 4.2, 1009 x 757 6.0 /
    // 6.3, but 2048^2 17.7 / 17.1 (its arithmetic, 1.2 times as much fused,
    // bounds it there), 4096^2 61 / 60 (uniform celerities other than +-1).
    if (precision == FDM_PRECISION_FP32 && order == 1)
        return n == 1 && (!fd || (int64_t)d.nx * d.ny <= (int64_t)1 << 20);
    if (precision == FDM_PRECISION_FP32) return fused_applies(precision, order, fd);
    if (n > 1 || !fused_applies(FDM_PRECISION_FP32, order, fd)) return false;
    const bool field = d.velocity == FDM_VELOCITY_LAW && d.v0_field;
    const int64_t per_node = (precision == FDM_PRECISION_FP64 ? 32 : 16) + (field ? 4 : 0);
    return (int64_t)d.nx * d.ny * per_node > (int64_t)256 << 20;
}

int balanced_height(const std::function<int64_t(int)> &waves, int max_ny, int64_t limit)
{
    if (waves(max_ny) > limit) return -1;
    int lo = 1, hi = max_ny;
    while (lo < hi) {
        const int mid = lo + (hi - lo) / 2;
        if (waves(mid) <= limit) hi = mid;
        else lo = mid + 1;
    }
    return lo;
}

// As in fused_rows below: the SIMD with the most waves, w, sets the time of a
// launch that is resident at once, an iteration of a wave's row loop takes
// about as long again with each wave more (a lone wave also waits for its own
// results), and a tile of h rows costs h + 3 of them with its extra row and
// its first loads.  So the height is the smallest that fits w waves per SIMD
// for the w of 1 .. 8 with the least (h + 3)(1 + w).  Measured against
// pick_rows (us a step, uniform celerity other than +-1): fully discrete 64^2
// 2.77 / 3.64, 300 x 200 2.81 / 3.73, 512^2 4.28 / 4.49, 1009 x 757 6.29 / 6.86, 1536^2 12.2 / 13.0;
// float64 state, both stages, 64^2 7.5 / 11.5, 512^2 14.1 / 16.9, 1009 x 757
// 24.9 / 29.4, 1536^2 58.2 / 60.9.  Launches of more than 5 waves per SIMD at
// pick_rows' height keep it, the evenness matters less there: 2048^2 fully
// discrete 17.5 at its 12 rows against 17.7 at the balanced 18, 4096^2 61.0 at
// 16 against 62.6 at 36.
int stage_rows(const std::function<int64_t(int)> &waves, int64_t strip_rows, int max_ny, int64_t simds)
{
    const int large = pick_rows(strip_rows, max_ny, 0);
    if (waves(large) > 5 * simds) return large;
    int best = -1;
    int64_t least = 0;
    for (int w = 1; w <= 8; ++w) {
        const int h = balanced_height(waves, max_ny, w * simds);
        if (h < 0) continue;
        const int64_t t = ((int64_t)h + 3) * (1 + w);
        if (best < 0 || t < least) {
            best = h;
            least = t;
        }
    }
    return best > 0 ? best : large;
}

int stage_rows_of(const fdm_transport_desc &d, int64_t simds)
{
    const int64_t strips = (d.nx + kStrip - 1) / kStrip;
    return stage_rows([&](int h) { return strips * tiles_along_y(d.ny, h); }, strip_rows_of(d), d.ny, simds);
}

// A launch that is resident at once takes the time of the SIMD with the most
// waves, w, and a wave's time is linear in its height h.  Fitted over
// 300 x 200 to 4096^2 and 1 to 75 rows (minmod, uniform celerity other than
// +-1, us; those take 5% less at 2048^2 and choose the same heights to 1%):
//   3.4 + 0.75 w + (0.16 + 0.195 w) h,
// the first part the launch, the loads and the first stage's extra rows, the
// second the issue time of w waves (a lone wave also waits for its own
// results, hence 0.16).  For each w the smallest h that fits it is the best;
// at most seven waves are resident (66 to 72 registers).  Measured, this
// choice against the best of all heights: 300 x 200 3.99 / 3.99 us a step,
// 512^2 5.55 / 5.55, 1024^2 10.49 / 10.49, 1536^2 18.0 / 17.7, 2048^2
// 26.1 / 26.1, 3000 x 1000 20.3 / 20.3, 4096^2 80.1 / 78.9; the stage
// kernels' two launches take 7.09, 8.12, 13.7, -, 32.4, -, 165 at the sizes
// where they were timed beside it.
// Above 64 rows (beyond about 5000^2) the gain over 64 is under 2%.
int fused_rows(const std::function<int64_t(int)> &waves, int max_ny, int64_t simds)
{
    int best = -1;
    double least = 0.0;
    for (int w = 1; w <= 7; ++w) {
        const int h = balanced_height(waves, max_ny, w * simds);
        if (h < 0 || h > 64) continue;
        const double t = 3.4 + 0.75 * w + (0.16 + 0.195 * w) * h;
        if (best < 0 || t < least) {
            best = h;
            least = t;
        }
    }
    return best > 0 ? best : std::min(64, max_ny);
}

int launch_rows(int64_t strips, int ny, int rows)
{
    while (strips * tiles_along_y(ny, rows) > kMaxLaunchTiles && rows < ny)
        rows = (int)std::min<int64_t>(ny, 2 * (int64_t)rows);
    return rows;
}

int64_t strip_rows_of(const fdm_transport_desc &d)
{
    return (int64_t)((d.nx + kStrip - 1) / kStrip) * d.ny;
}

double smax_uniform(const fdm_transport_desc &d)
{
    const double h = std::min(d.dx, d.dy);
    if (d.velocity == FDM_VELOCITY_PRESCRIBED)   // the float32 velocity the kernels use
        return std::max(std::fabs((double)(float)d.V[0]) / d.dx, std::fabs((double)(float)d.V[1]) / d.dy) * h;
    return std::fabs((double)(float)d.v0);
}

float step_dt(const fdm_transport_desc &d, double smax)
{
    if (d.dt > 0.0) return (float)d.dt;
    const double h = std::min(d.dx, d.dy);
    return round_down_float(smax > 0.0 ? d.cfl * h / smax : d.cfl * h);
}

int spacing_kind(double dx, double dy)
{
    int ex = 0, ey = 0;
    const double mx = std::frexp(dx, &ex), my = std::frexp(dy, &ey);
    if (std::max(std::abs(ex), std::abs(ey)) <= 1000 && mx == 0.5 && my == 0.5) return SPACING_POW2;
    if (std::max(std::abs(ex), std::abs(ey)) < 100) return SPACING_SHARED;
    return SPACING_DIVIDE;
}

void fill_inst(InstDev &I, const fdm_transport_desc &d, float dt, void *w11, void *w12)
{
    std::memset(&I, 0, sizeof(I));
    I.w11 = w11;
    I.w12 = w12;
    I.v0f = d.velocity == FDM_VELOCITY_LAW ? d.v0_field : nullptr;
    I.nx = d.nx;
    I.ny = d.ny;
    I.v0 = (float)d.v0;
    I.V1 = (float)d.V[0];
    I.V2 = (float)d.V[1];
    I.dtd = (double)dt;
    I.dxd = d.dx;
    I.dyd = d.dy;
    I.rdxd = 1.0 / d.dx;
    I.rdyd = 1.0 / d.dy;
    I.spacing_kind = spacing_kind(d.dx, d.dy);
    I.cxd = (double)dt / d.dx;
    I.cyd = (double)dt / d.dy;
    I.thetad = d.limiter == FDM_LIMITER_MINMOD ? 1.0 : d.limiter == FDM_LIMITER_MC ? 2.0 : d.theta;
    I.cx = (float)I.cxd;
    I.cy = (float)I.cyd;
    I.theta = (float)I.thetad;
    I.limiter = d.limiter;
    I.vkind = d.velocity | (d.scheme == FDM_SCHEME_FULLY_DISCRETE ? VK_FD : 0);
}

int stage_modes(int32_t order, int32_t step, int modes[2])
{
    if (order == 2) {
        modes[0] = MODE_FWD;
        modes[1] = MODE_HEUN2;
        return 2;
    }
    if (order == 3) {
        modes[0] = MODE_MID1;
        modes[1] = MODE_MID2;
        return 2;
    }
    modes[0] = (step & 1) ? MODE_BWD : MODE_FWD;
    return 1;
}

// The same bits either way.  Two stages a step: a fused launch a step, in
// pairs; the stage kernels' pair on the last step of an odd count costs no
// more than a fused launch and the copy of both components back (2048^2: 32 us
// against 26 + 14; 512^2: 8.1 against 5.6 + 4).
// One stage a step (float): a fused launch takes two steps, and single steps
// (in either direction) fill up so that the last launch writes the state: an
// odd number of fused launches and then single ones back, or an even number.
FusedPlan fused_plan(int32_t order, int32_t n_steps)
{
    if (order != 1) return {n_steps - (n_steps & 1), n_steps & 1};
    // n mod 4: 0, pairs alone; 1, three singles; 2, two singles; 3, one
    const int32_t single = n_steps == 1 ? 1 : n_steps % 4 == 0 ? 0 : 4 - n_steps % 4;
    return {(n_steps - single) / 2, single};
}

int32_t fused_steps(int32_t order, int32_t n)
{
    const int32_t whole = order == 1 ? 4 : 2, up = (whole - n % whole) % whole;
    return n > INT32_MAX - up ? n : n + up;
}

InstDev stage_tiling(const InstDev &I, const fdm_transport_desc &d, int rows, int64_t simds)
{
    InstDev J = I;
    if (rows <= 0) J.rows = launch_rows(J.strips, d.ny, stage_rows_of(d, simds));
    J.chunks = tiles_along_y(d.ny, J.rows);
    return J;
}

hipError_t run_fused_steps(const InstDev &I, const InstDev &odd, int32_t order, int32_t precision, int32_t n_steps,
                           hipStream_t s)
{
    const FusedPlan plan = fused_plan(order, n_steps);
    const int integ = order == 1 ? FUSED_TWO_STEPS : order == 3 ? FUSED_MIDPOINT : FUSED_HEUN;
    hipError_t e = hipSuccess;
    for (int32_t k = 0; k < plan.fused && e == hipSuccess; ++k) e = launch_fused(I, k & 1, integ, precision, s);
    for (int32_t k = 0; k < plan.single && e == hipSuccess; ++k) {
        int modes[2];
        const int nm = stage_modes(order, plan.fused + k, modes);
        for (int m = 0; m < nm && e == hipSuccess; ++m) e = launch_stage(odd, modes[m], precision, s);
    }
    if (order == 1 && n_steps == 1) {
        const int64_t n = (int64_t)I.nx * I.ny;
        if (e == hipSuccess) e = launch_copy(I.a11, I.w11, n, precision, s);
        if (e == hipSuccess) e = launch_copy(I.a12, I.w12, n, precision, s);
    }
    return e;
}

hipError_t run_line_steps(const InstDev &I, int32_t order, int32_t precision, int32_t n_steps, hipStream_t s)
{
    const int32_t pair = 2 * line_steps(order);
    const int32_t launches = 2 * (int32_t)(((int64_t)n_steps + pair - 1) / pair);
    for (int32_t k = 0; k < launches; ++k) {
        const int32_t steps = n_steps / launches + (k < n_steps % launches ? 1 : 0);
        const hipError_t e = launch_line(I, order, steps, k & 1, precision, s);
        if (e != hipSuccess) return e;
    }
    return hipSuccess;
}

}  // namespace host
}  // namespace fdm
