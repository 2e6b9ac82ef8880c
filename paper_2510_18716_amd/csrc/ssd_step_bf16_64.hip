// The decode step's kernels for bf16 rows of 64 elements.
#define SSD_STEP_ONLY bf16_t, 64
#include "ssd_step.hip"
