// One-pass score kernels for head_dim 128, bf16 and FP8 keys (see score_once.h).
#include "score_once.h"

namespace codecomp {
template int launch_once<128, false>(const Plan&, const ScoreArgs&, hipStream_t);
template int launch_rows<128, false>(const Plan&, const ScoreArgs&, hipStream_t);
template int launch_once<128, true>(const Plan&, const ScoreArgs&, hipStream_t);
template int launch_rows<128, true>(const Plan&, const ScoreArgs&, hipStream_t);
}  // namespace codecomp
