// Register-resident agent kernels (resident.hip): plan and launch.
#pragma once

#include "internal.h"

namespace bi {

// launch_resident's answer for calls that it does not take.
constexpr int kNoPlan = 1;

// As launch_agent, for calls that the kernels declared here take (else
// kNoPlan, nothing enqueued).  staged: the kernels of agent.hip would hold the
// whole window's slices in LDS.
int launch_resident(const bi_model *m, int algo, int b, int T, bool staged, const int32_t *obs, const double *ll,
                    const int32_t *act, const float *prior, double tau, int iters, float *q, hipStream_t stream);

// The same choice as text (profile name of the kernel, its plan); false: no plan.
bool describe_resident(const bi_model *m, int algo, int b, int T, bool staged, char *buf, size_t cap);

}  // namespace bi
