// fdm_host.h -- host-side validation and set-up shared by the C-ABI entry
// points: descriptor checks, the step and its stability bound, the tiling
// and the stage sequence of an instance.
#pragma once

#include <stdint.h>

#include <functional>
#include <string>

#include "../../include/fdm.h"
#include "fdm_internal.h"

namespace fdm {
namespace host {

bool finite_pos(double v);

// "" if the descriptor is valid, else the reason (no HIP call).
std::string check_desc(const fdm_transport_desc &d);

// Largest float not above x (x > 0).
float round_down_float(double x);

// "" if the step the descriptor implies is within the stability bound
// (nu2 = dt (S1/dx + S2/dy) <= 1, or <= 1/2 for one limited forward-Euler
// stage, order 1), else the reason.  smax_law: max |v0| (LAW with a fixed
// dt; unused otherwise).
std::string check_courant(const fdm_transport_desc &d, int32_t order, double smax_law);

// max speed of a descriptor without a celerity field: |v0| (LAW, float32) or
// max(|V1|/dx, |V2|/dy) min(dx, dy) (PRESCRIBED).
double smax_uniform(const fdm_transport_desc &d);

// The float32 step: the given dt, or cfl min(dx,dy) / smax rounded down
// (the unit-speed step when smax = 0).
float step_dt(const fdm_transport_desc &d, double smax);

// How the FP64 update divides by the spacings (SPACING_*).
int spacing_kind(double dx, double dy);

// The device view of one instance with step dt and stage buffer (w11, w12);
// the state pointers and the tiling are left unset.
void fill_inst(InstDev &I, const fdm_transport_desc &d, float dt, void *w11, void *w12);

// Rows per wave tile of large launches: `requested`, or by the number of
// `strip_rows` (strip, row) pairs in the launch.
int pick_rows(int64_t strip_rows, int ny, int requested);

// Whether the fused schedule may be asked for: float32 state and arithmetic,
// two stages a step, semi-discrete scheme.
bool fused_applies(int32_t precision, int32_t order, bool fd);

// Whether the AUTO schedule takes the fused kernel.
bool fused_by_default(const fdm_transport_desc *descs, int32_t n, int32_t precision, int32_t order);

// Rows per tile of the stage kernels when no height was asked for; waves(h)
// is the number of tiles at height h, strip_rows the (strip, row) pairs.
int stage_rows(const std::function<int64_t(int)> &waves, int64_t strip_rows, int max_ny, int64_t simds);

// stage_rows for one instance.
int stage_rows_of(const fdm_transport_desc &d, int64_t simds);

// Rows per tile of the fused kernel when neither a height nor the fused
// schedule was asked for; waves(h) is the number of tiles at height h.
int fused_rows(const std::function<int64_t(int)> &waves, int max_ny, int64_t simds);

// Smallest tile height with at most `limit` tiles, or -1 if even one tile
// per strip exceeds it (waves falls as the height grows).
int balanced_height(const std::function<int64_t(int)> &waves, int max_ny, int64_t limit);

// Tiles (one wave64 each) of one launch: a dispatch holds fewer than 2^32
// work-items, and the grid rounds the tile count up by at most 31.
constexpr int64_t kMaxLaunchTiles = (int64_t)1 << 25;

// `rows`, doubled until a launch of one instance fits one dispatch.
int launch_rows(int64_t strips, int ny, int rows);

// (strip, row) pairs of one instance in the stage kernels' tiling.
int64_t strip_rows_of(const fdm_transport_desc &d);

// Stage launches of step number `step` for an integrator order (1 Euler,
// 2 Heun, 3 explicit midpoint): the modes in order, their count returned.
int stage_modes(int32_t order, int32_t step, int modes[2]);

// How n_steps of one instance are launched when it takes the fused kernel:
// `fused` launches from the state to the stage buffer and back, then `single`
// steps by the stage kernels.  The launches end in the state, unless the one
// step of a single-stage integrator is all there is.
struct FusedPlan {
    int32_t fused, single;
};
FusedPlan fused_plan(int32_t order, int32_t n_steps);

// The fewest steps, not below n, that are fused launches alone (n itself where
// that would pass the largest number of steps).
int32_t fused_steps(int32_t order, int32_t n);

// n_steps of one instance by that plan.  odd: the instance in the stage
// kernels' tiling, for the single steps.
hipError_t run_fused_steps(const InstDev &I, const InstDev &odd, int32_t order, int32_t precision, int32_t n_steps,
                           hipStream_t s);

// The instance in the stage kernels' tiling with `rows` rows a tile, or the
// default where that is 0.
InstDev stage_tiling(const InstDev &I, const fdm_transport_desc &d, int rows, int64_t simds);

// n_steps >= 2 of a one-row instance by launches of several steps each, an
// even number of them (the last writes the state).
hipError_t run_line_steps(const InstDev &I, int32_t order, int32_t precision, int32_t n_steps, hipStream_t s);

// Message of the last failed call without a context (fdm_last_error(NULL)).
void set_init_error(const std::string &msg);

}  // namespace host
}  // namespace fdm
