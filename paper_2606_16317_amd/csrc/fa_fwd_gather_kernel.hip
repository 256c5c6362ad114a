// The kernels of a reordered call: those of fa_fwd_kernel.hip with queries and outputs taken
// through the gather map p.q_row, in a unit of their own (the reason stands at
// launch_fa_fwd_gather).

#define DSATTN_GATHER_KERNELS
#include "fa_fwd_kernel.hip"
