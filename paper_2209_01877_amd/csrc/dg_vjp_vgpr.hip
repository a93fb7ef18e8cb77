// The instantiations of dg_vjp.hip that are compiled with -amdgpu-mfma-vgpr-form (build.py): MFMA
// results go to ordinary registers instead of accumulation registers, which saves the copies that
// the pointwise fluxes need (692 -> 320 per pass of the FP64 P2 kernel).
#define TDG_VGPR_FORM
#include "dg_vjp.hip"
