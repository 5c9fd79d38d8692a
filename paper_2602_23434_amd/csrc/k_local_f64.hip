// Self-grouping tile kernels, float64 form.
#include "k_local_impl.h"

namespace pl {

hipError_t launch_local_f64(Ctx *c, const ItemDesc *table, const ItemDesc *host, int nitems, const LocalPlan &pl,
                            unsigned sf, unsigned *counter)
{
    return launch_local_impl<PL_F64>(c, table, host, nitems, pl, sf, counter);
}

bool local_plan_f64(const Ctx *c, const ItemDesc *host, int nitems, bool push, bool deposit, LocalPlan &pl)
{
    return local_plan_impl<PL_F64>(c, host, nitems, push, deposit, pl);
}

}  // namespace pl
