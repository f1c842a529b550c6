// The table update with a phase of the coming mini-batch's preparation riding in its launch.
#include "apply_kernels.h"

void tn_launch_apply_update_riding(const ApplyArgs &a, const PrepPhase &rider, hipStream_t st)
{
    PhaseRider r;
    r.x = rider;
    launch_apply(a, r, st);
}
