// The decode step's kernels for bf16 rows of 128 elements.
#define SSD_STEP_ONLY bf16_t, 128
#include "ssd_step.hip"
