// a3, bf16 operands: the launches whose last round of tiles is computed in halves (see tail_tile in moe_tile_order.h).  A file of its
// own: each of these kernels has the loops of the wide and of the narrow block, and they take minutes to compile.
#include "moe_ffn_gemm_bf16.h"

namespace moe {

int launch_gate_up_halves_bf16(const GemmParams& p, int R, int n_exp, hipStream_t st) { return launch_stages<0, 2, BM, true>(p, R, n_exp, st); }

int launch_down_halves_bf16(const GemmParams& p, int R, int n_exp, hipStream_t st) { return launch_stages<1, 2, BM, true>(p, R, n_exp, st); }

}  // namespace moe
