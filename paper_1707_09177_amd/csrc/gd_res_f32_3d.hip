// register-resident 3D kernels, F32
#define GD_RES_T float
#define GD_RES_NDIM 3
#define GD_RES_NAME kernels_f32_3d
#include "gd_res_inst.inc"
