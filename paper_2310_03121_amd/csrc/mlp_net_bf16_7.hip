// BF16 networks of hidden widths 256-192-160.
#include "mlp_net.h"

namespace nnp {

void launch_net_bf16_7(const NetArgs& a, int n_rows, int rows_cap, int members, hipStream_t st) {
  launch_net_w<bf16_t, 256, 192, 160>(a, n_rows, rows_cap, members, st);
}

}  // namespace nnp
