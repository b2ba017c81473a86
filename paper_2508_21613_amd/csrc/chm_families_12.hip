// The families of a call in one launch, 9 to 12 stages.
#include "chm_search_kernel.h"

int chmk_families_12(int sp, int s1, const FamiliesLaunch &a, uint32_t blocks, void *stream) {
#define CHM_CASE(SP, S1) if (sp == SP && s1 == S1) { hipLaunchKernelGGL((k_search_families<SP, S1>), dim3(blocks), dim3(BLOCK), 0, (hipStream_t)stream, a); return 0; }
  CHM_CASE(9, 8) CHM_CASE(9, 7) CHM_CASE(10, 9) CHM_CASE(10, 8) CHM_CASE(11, 10) CHM_CASE(11, 9) CHM_CASE(12, 11)
  CHM_CASE(12, 10)
#undef CHM_CASE
  return 1;
}
