// The instantiations of dg_stage.hip that are compiled with -amdgpu-mfma-vgpr-form (build.py): MFMA
// results go to ordinary registers instead of accumulation registers, which saves the copies that
// the pointwise fluxes need (383 -> 204 per pass of the FP64 P3 kernel).
#define TDG_VGPR_FORM
#include "dg_stage.hip"
