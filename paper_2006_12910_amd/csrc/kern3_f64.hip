// 3D sweeps with populations stored as f64.
#define LBK3_ST 0
#define LBK3_ENTRY sweep3_f64
#include "kern3_st.h"
