// scan_one_f32.hip -- scan kernels for a bank of one template (timestamp groups over the lanes):
// FP32 compensated sums on F32 storage, the closed-form waveforms.
#include "sft_scan.h"

using namespace sftk;

ScanFn scan_pick_one_f32(int wf, int kern, int K, int nd)
{
  return wf == WF_PN35 ? pick_kern<float2, SFT_PREC_FP32_KAHAN, WF_PN35, 0, 1>(kern, K, nd)
                       : pick_kern<float2, SFT_PREC_FP32_KAHAN, WF_NEWTON, 0, 1>(kern, K, nd);
}
