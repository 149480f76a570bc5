// bf16, d = 104 .. 120 in steps of 8: the plainly written kernels at a padded width of 128 columns
// (namespace burst::d128x); and dK/dV at d = 128 for grouped heads whose slice is no multiple of 64 rows.
#define BURST_SMALL_D 128
#define BURST_SMALL_NS d128x
#define BURST_SMALL_PAD
// (two wavefronts per dK/dV workgroup, as in the d = 128 build: four would spill)
#define BURST_SMALL_DKV_WAVES 2
#include "burst_plain_mfma.h"
