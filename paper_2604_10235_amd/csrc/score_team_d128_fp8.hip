// Long requests in one pass by teams (see score_team.h): head_dim 128, FP8 keys.
#include "score_team.h"

namespace codecomp {
template bool team_fits<128, true>(const Plan&);
template int launch_team<128, true>(const Plan&, const ScoreArgs&, char*, hipStream_t);
}
