// The families of a call in one launch, 3 to 8 stages.
#include "chm_search_kernel.h"

int chmk_families_8(int sp, int s1, const FamiliesLaunch &a, uint32_t blocks, void *stream) {
#define CHM_CASE(SP, S1) if (sp == SP && s1 == S1) { hipLaunchKernelGGL((k_search_families<SP, S1>), dim3(blocks), dim3(BLOCK), 0, (hipStream_t)stream, a); return 0; }
  CHM_CASE(3, 2) CHM_CASE(4, 3) CHM_CASE(4, 2) CHM_CASE(5, 4) CHM_CASE(5, 3) CHM_CASE(6, 5) CHM_CASE(6, 4)
  CHM_CASE(7, 6) CHM_CASE(7, 5) CHM_CASE(8, 7) CHM_CASE(8, 6)
#undef CHM_CASE
  return 1;
}
