// Launchers of 2D resistive compressible MHD (all storages, D2Q5 and D2Q9).
#define LBM_FAST_CONTRACT               // one kernel per step only: the compiler may fuse across expressions
#include "step_kernels.hpp"

LBM_DEFINE_LAUNCHERS_2D(lbm_launchers_mhd, SysMHD)
