// scan_one_f64.hip -- scan kernels for a bank of one template (timestamp groups over the lanes):
// FP64 sums on F64 storage, the closed-form waveforms.
#include "sft_scan.h"

using namespace sftk;

ScanFn scan_pick_one_f64(int wf, int kern, int K, int nd)
{
  return wf == WF_PN35 ? pick_kern<double2, SFT_PREC_FP64, WF_PN35, 0, 1>(kern, K, nd)
                       : pick_kern<double2, SFT_PREC_FP64, WF_NEWTON, 0, 1>(kern, K, nd);
}
