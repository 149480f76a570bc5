// bf16, d = 40 .. 56 in steps of 8: the plainly written kernels at a padded width of 64 columns
// (namespace burst::d64x).
#define BURST_SMALL_D 64
#define BURST_SMALL_NS d64x
#define BURST_SMALL_PAD
#include "burst_plain_mfma.h"
