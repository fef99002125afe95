// 3D sweeps with populations stored as bf16.
#define LBK3_ST 3
#define LBK3_ENTRY sweep3_bf16
#include "kern3_st.h"
