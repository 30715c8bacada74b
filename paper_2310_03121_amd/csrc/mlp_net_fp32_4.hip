// FP32 networks of hidden widths 160-128-96.
#include "mlp_net.h"

namespace nnp {

void launch_net_fp32_4(const NetArgs& a, int n_rows, int rows_cap, int members, hipStream_t st) {
  launch_net_w<float, 160, 128, 96>(a, n_rows, rows_cap, members, st);
}

}  // namespace nnp
