// Launchers of the fused steps of small systems (k_step.hip).
#pragma once
#include "rod_internal.h"

namespace rodmx {

// Where a fused step writes: the next level's state planes and moments, or with
// `last` the closing level's state; the dipole field of the level gathered (or
// null). keep: the full-step velocities of the level are stored to d.v and d.w
// (a recorded run, whose levels have planes of their own).
struct StepOut {
  double *x, *v, *q, *w, *mu;
  float* muf;
  double* Bo;
  int last, keep;
};

constexpr int STEPS_MAX = 32;  // particles of a member that k_steps can serve

hipError_t launch_step(const Dev& d, int precision, const StepOut& o, hipStream_t s);
// n steps from the level in d.step[0] for every member, each of at most max_member <=
// STEPS_MAX particles; not for Hertz-Mindlin contact. With rec the levels after lvl0
// are recorded there, and the state and its level are left alone.
hipError_t launch_steps(const Dev& d, int precision, int max_member, long long lvl0, int n,
                        hipStream_t s, double* rec = nullptr, long rec_stride = 0);

}  // namespace rodmx
