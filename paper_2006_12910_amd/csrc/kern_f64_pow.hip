// FP64 kernels with the power law of any exponent.  A file of its own because
// it is compiled without hoisting out of loops at the machine level: the
// constants of pow, in FP64 too wide for an operand, would wait for it in
// registers through all the steps of a launch, and the 128 that two workgroups
// a CU leave spilled 60.
#define LBK_ST lbk::ST_F64
#define LBK_GETTER kernels_f64_pow
#define LBK_GENERIC_POWER_FILE
#include "kernels_st.h"
