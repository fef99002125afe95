// Kernels with populations stored as f64; those with the power law of any
// exponent are in kern_f64_pow.hip.
#define LBK_ST lbk::ST_F64
#define LBK_GETTER kernels_f64
#define LBK_GENERIC_POWER kernels_f64_pow
#include "kernels_st.h"
