// register-resident 2D kernels, F32
#define GD_RES_T float
#define GD_RES_NDIM 2
#define GD_RES_NAME kernels_f32_2d
#include "gd_res_inst.inc"
