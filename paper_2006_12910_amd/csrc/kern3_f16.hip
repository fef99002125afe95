// 3D sweeps with populations stored as f16.
#define LBK3_ST 2
#define LBK3_ENTRY sweep3_f16
#include "kern3_st.h"
