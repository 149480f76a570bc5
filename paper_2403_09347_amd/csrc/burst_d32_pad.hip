// bf16, d = 8 .. 32 in steps of 8: the plainly written kernels at a padded width of 32 columns
// (namespace burst::d32x).
#define BURST_SMALL_D 32
#define BURST_SMALL_NS d32x
#define BURST_SMALL_PAD
#include "burst_plain_mfma.h"
