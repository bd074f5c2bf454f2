// a3, bf16 operands: the down launch with 128-wide column tiles whose last, or only, round is computed in tiles of 64 columns
// (launch_expert_ffn_bf16 has the rule).  A file of its own: the loops for every tile height take minutes to compile.
#include "moe_ffn_gemm_bf16.h"

namespace moe {

int launch_down_narrow_halves_bf16(const GemmParams& p, int R, int n_exp, hipStream_t st) { return launch_stages<1, 1, BM, true>(p, R, n_exp, st); }

}  // namespace moe
