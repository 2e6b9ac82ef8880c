// The decode step's kernels for f32 rows of 64 elements.
#define SSD_STEP_ONLY float, 64
#include "ssd_step.hip"
