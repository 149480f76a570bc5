// bf16, d = 104 .. 120 in steps of 8: the plainly written kernels at a padded width of 128 columns
// (namespace burst::d128x); and dK/dV at d = 128 for grouped heads whose slice is no multiple of 64 rows.
#define BURST_SMALL_D 128
#define BURST_SMALL_NS d128x
#define BURST_SMALL_PAD
// (eight wavefronts per dK/dV workgroup, K and V in LDS: see burst_bwd_dkv_d64_kernel)
#define BURST_SMALL_DKV_WAVES 8
#include "burst_plain_mfma.h"
