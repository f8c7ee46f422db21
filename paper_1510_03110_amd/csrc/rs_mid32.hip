// The FP32 leaves of the column-owner kernels (mixed precision), compiled on
// their own so that the two element types build in parallel.
#define RS_MID_FP32 1
#include "rs_mid.hip"
