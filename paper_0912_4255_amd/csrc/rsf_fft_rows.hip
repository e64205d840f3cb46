// The first pass on general stages (rsf_pass_a.h) in workgroups of 128 and 256
// threads.  A source of its own because its twelve kernels take the compiler as
// long as all of rsf_fft.hip, which has the 512-thread ones.
#include "rsf_device.h"
#include "rsf_launch.h"
#include "rsf_pass_a.h"

namespace rsf {

#define RSF_GENERAL_FN(ORD, THR)                                               \
    {(const void*)rsf_fft_pass_a_k<ORD, false, GeneralStages<kFftEPT>, THR>,   \
     (const void*)rsf_fft_pass_a_k<ORD, true, GeneralStages<kFftEPT>, THR>}
#define RSF_GENERAL(THR) {RSF_GENERAL_FN(1, THR), RSF_GENERAL_FN(2, THR), RSF_GENERAL_FN(3, THR)}
// [threads][spindown order - 1][non-temporal spill]
const void* const kGeneralRowsSmall[2][3][2] = {RSF_GENERAL(128), RSF_GENERAL(256)};
#undef RSF_GENERAL
#undef RSF_GENERAL_FN

}  // namespace rsf
