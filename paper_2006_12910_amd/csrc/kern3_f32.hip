// 3D sweeps with populations stored as f32.
#define LBK3_ST 1
#define LBK3_ENTRY sweep3_f32
#include "kern3_st.h"
