// Mask reuse, and the kernels of a reordered call: those of fa_fwd_kernel.hip with queries and
// outputs taken through the gather map p.q_row.  A unit of their own; the reason stands at
// launch_fa_fwd_gather.

#define DSATTN_SIDE_KERNELS
#include "fa_fwd_kernel.hip"
