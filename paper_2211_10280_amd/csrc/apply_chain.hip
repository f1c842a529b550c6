// The table update with the chaining of long rows in its launch, and maybe a phase of the coming mini-batch's preparation.
#include <string.h>

#include "apply_kernels.h"

void tn_launch_apply_update_chaining(const ApplyArgs &a, const PrepPhase *rider, const ChainWork &chain, hipStream_t st)
{
    ChainRider r;
    memset((void *)&r, 0, sizeof(r));
    if (rider) r.x = *rider;
    r.chain = chain;
    launch_apply(a, r, st);
}
