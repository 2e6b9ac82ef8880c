// The decode step's kernels for f32 rows of 128 elements.
#define SSD_STEP_ONLY float, 128
#include "ssd_step.hip"
