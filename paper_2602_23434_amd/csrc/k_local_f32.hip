// Self-grouping tile kernels, float32 + cell-offset form.
#include "k_local_impl.h"

namespace pl {

hipError_t launch_local_f32(Ctx *c, const ItemDesc *table, const ItemDesc *host, int nitems, const LocalPlan &pl,
                            unsigned sf, unsigned *counter)
{
    return launch_local_impl<PL_F32_OFFSET>(c, table, host, nitems, pl, sf, counter);
}

bool local_plan_f32(const Ctx *c, const ItemDesc *host, int nitems, bool push, bool deposit, LocalPlan &pl)
{
    return local_plan_impl<PL_F32_OFFSET>(c, host, nitems, push, deposit, pl);
}

bool local_plan_f64(const Ctx *c, const ItemDesc *host, int nitems, bool push, bool deposit, LocalPlan &pl);

bool local_plan(const Ctx *c, const ItemDesc *host, int nitems, bool push, bool deposit, LocalPlan &pl)
{
    return c->d.prec == PL_F64 ? local_plan_f64(c, host, nitems, push, deposit, pl)
                               : local_plan_f32(c, host, nitems, push, deposit, pl);
}

}  // namespace pl
