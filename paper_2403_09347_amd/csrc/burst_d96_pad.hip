// bf16, d = 72 .. 96 in steps of 8: the plainly written kernels at a padded width of 96 columns
// (namespace burst::d96x).
#define BURST_SMALL_D 96
#define BURST_SMALL_NS d96x
#define BURST_SMALL_PAD
#include "burst_plain_mfma.h"
