// The families of a call in one launch, 17 to 24 stages.
#include "chm_search_kernel.h"

int chmk_families_24(int sp, int s1, const FamiliesLaunch &a, uint32_t blocks, void *stream) {
#define CHM_CASE(SP, S1) if (sp == SP && s1 == S1) { hipLaunchKernelGGL((k_search_families<SP, S1>), dim3(blocks), dim3(BLOCK), 0, (hipStream_t)stream, a); return 0; }
  CHM_CASE(17, 16) CHM_CASE(18, 17) CHM_CASE(19, 18) CHM_CASE(20, 19) CHM_CASE(21, 20) CHM_CASE(22, 21)
  CHM_CASE(23, 22) CHM_CASE(24, 23)
#undef CHM_CASE
  return 1;
}
