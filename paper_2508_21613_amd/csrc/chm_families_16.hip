// The families of a call in one launch, 13 to 16 stages.
#include "chm_search_kernel.h"

int chmk_families_16(int sp, int s1, const FamiliesLaunch &a, uint32_t blocks, void *stream) {
#define CHM_CASE(SP, S1) if (sp == SP && s1 == S1) { hipLaunchKernelGGL((k_search_families<SP, S1>), dim3(blocks), dim3(BLOCK), 0, (hipStream_t)stream, a); return 0; }
  CHM_CASE(13, 12) CHM_CASE(13, 11) CHM_CASE(14, 13) CHM_CASE(14, 12) CHM_CASE(15, 14) CHM_CASE(15, 13)
  CHM_CASE(16, 15) CHM_CASE(16, 14)
#undef CHM_CASE
  return 1;
}
