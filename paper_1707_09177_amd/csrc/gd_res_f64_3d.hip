// register-resident 3D kernels, F64
#define GD_RES_T double
#define GD_RES_NDIM 3
#define GD_RES_NAME kernels_f64_3d
#include "gd_res_inst.inc"
