// fdm_static.h -- internal interface of the static (stress) solve of the
// layer case and of the coupled velocity law; see fdm_static.hip.
#pragma once
#include <hip/hip_runtime.h>

#include <cstdint>
#include <string>

#include "fdm_internal.h"

namespace fdm {

enum class StaticStatus { Ok, Device, OutOfMemory };

struct StaticParams {
    int nx, ny;
    double dx, dy;       // dx == dy: cubic voxels, x3 spacing dx
    double mu, lambda;
    int h, n3;           // layer and cell height in voxels, 1 <= h <= n3
    bool f64;            // double arrays and FFT, else float
};

struct StaticPlan;

// Builds the multiplier table and what the transforms need.  once: for a
// single solve (rather than every step of a run).
StaticStatus static_plan_create(const StaticParams &q, bool once, hipStream_t s, StaticPlan **out, std::string &err);
void static_plan_destroy(StaticPlan *p);

// Enqueues tau13 = layer average of sigma13 for densities (a11, a12) and the
// mean stress sigma_bar on s.  a11/a12 are read only; tau13 is written.
StaticStatus static_plan_run(StaticPlan *p, const void *a11, const void *a12, void *tau13, double sigma_bar,
                             hipStream_t s, std::string &err);

// Celerity at the nodes, written as float32, m = mobility * mfield[i] (mfield
// may be null):
//   wiggly = false: v0 = -m S_tau0(tau13), S the soft threshold;
//   wiggly = true:  v0 = m (tau_y cos(phi / beta) - tau13).
struct LawParams {
    bool wiggly;
    double tau0, mobility, tau_y, beta;
    const float *mfield;
};

// Allocates what static_plan_celerity needs with this law (kept with the
// plan), so that it only launches kernels and its steps can be captured.
StaticStatus static_plan_prepare(StaticPlan *p, const LawParams &law, std::string &err);

// Where a coupled step's solve reads its densities from, if not from the
// state itself: then the step's last stage also writes there, and
// static_plan_celerity is called with null densities (the first step of a
// run passes the state, which is copied there).
bool static_plan_input(StaticPlan *p, void **a11, void **a12);

// Enqueues a coupled step's celerity field on s: the static solve of the
// densities with the mean stress and slip of cd (device), phi at the nodes
// for the wiggly law, and the law.  slip (may be null): the previous step's
// pending slip update, run ahead of everything that reads the mean stress or
// slip.  Also writes static_plan_partials(p) partials of max |v0| (NaN marks
// a non-finite value) for the step size.  static_plan_prepare comes first.
StaticStatus static_plan_celerity(StaticPlan *p, const void *a11, const void *a12, const LawParams &law,
                                  const CoupledDev *cd, const SlipArgs *slip, float *v0, float *partial,
                                  hipStream_t s, std::string &err);
constexpr int kLawBlocks = 1024;   // at most this many partials
int static_plan_partials(const StaticPlan *p);

}  // namespace fdm
