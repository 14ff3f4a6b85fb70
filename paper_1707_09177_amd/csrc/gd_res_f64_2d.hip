// register-resident 2D kernels, F64
#define GD_RES_T double
#define GD_RES_NDIM 2
#define GD_RES_NAME kernels_f64_2d
#include "gd_res_inst.inc"
