// One-pass score kernels for head_dim 64, bf16 and FP8 keys (see score_once.h).
#include "score_once.h"

namespace codecomp {
template int launch_once<64, false>(const Plan&, const ScoreArgs&, hipStream_t);
template int launch_rows<64, false>(const Plan&, const ScoreArgs&, hipStream_t);
template int launch_once<64, true>(const Plan&, const ScoreArgs&, hipStream_t);
template int launch_rows<64, true>(const Plan&, const ScoreArgs&, hipStream_t);
}  // namespace codecomp
