// C ABI of libcodecomp: argument validation, workspace layout and the enqueue order of the
// score -> select -> gather path.  Everything here runs on the host; validation happens before
// the first HIP call so that rejected arguments never reach a GPU.
#include <math.h>

#include "plan.h"

namespace codecomp {

static inline size_t align256(size_t x) { return (x + 255) & ~size_t(255); }

// A wave runs on SIMD (wave % 4) of its compute unit (consecutive waves of a workgroup go to consecutive
// SIMDs), and a score workgroup with more than four waves has a compute unit to itself.  The cost of a
// wave is its number of (row block, half tile) units: 2 for a block it computes for both halves of every
// tile, 1 for a block it shares with another wave.  Up to 8 blocks: pairs of blocks per wave, as many
// waves as that takes (several such workgroups share a compute unit).  More: eight waves, one block each,
// and the remaining blocks dealt out so that the four SIMDs carry the same number of units (+-1).
void assign_row_blocks(Plan* pl) {
  const int nb = pl->row_blocks;
  for (int b = 0; b < 2 * kMaxWaves; ++b) pl->rb_holder[b][0] = pl->rb_holder[b][1] = 255;
  for (int w = 0; w < kMaxWaves; ++w) pl->wave_desc[w] = 0;
  auto hold = [&](int rb, int wave, int slot) {
    uint8_t* h = pl->rb_holder[rb];
    h[h[0] == 255 ? 0 : 1] = (uint8_t)(wave * 2 + slot);
  };
  if (nb <= 8) {
    pl->waves = (nb + 1) / 2;
    for (int w = 0; w < pl->waves; ++w) {
      const int rb0 = 2 * w, rb1 = 2 * w + 1;
      hold(rb0, w, 0);
      if (rb1 < nb) { hold(rb1, w, 1); pl->wave_desc[w] = (uint32_t)rb0 | ((uint32_t)rb1 << 8) | (3u << 16); }
      else pl->wave_desc[w] = (uint32_t)rb0;
    }
    return;
  }
  pl->waves = kMaxWaves;
  int extra[kMaxWaves];                       // half-tile units of a second block per wave: 0, 1 or 2
  const int units = 2 * (nb - kMaxWaves);     // 2 .. 16
  for (int s = 0; s < 4; ++s) {
    const int e = units / 4 + (s < units % 4 ? 1 : 0);
    extra[s] = e < 2 ? e : 2;
    extra[s + 4] = e - extra[s];
  }
  int next = kMaxWaves;                       // next block to hand out
  for (int w = 0; w < kMaxWaves; ++w) {
    hold(w, w, 0);
    pl->wave_desc[w] = (uint32_t)w;
    if (extra[w] == 2) { hold(next, w, 1); pl->wave_desc[w] |= ((uint32_t)next << 8) | (3u << 16); ++next; }
  }
  int pending = -1;                           // wave that took the first half of block `next`
  for (int w = 0; w < kMaxWaves; ++w) {
    if (extra[w] != 1) continue;
    hold(next, w, 1);
    if (pending < 0) { pl->wave_desc[w] |= ((uint32_t)next << 8) | (1u << 16); pending = w; }
    else { pl->wave_desc[w] |= ((uint32_t)next << 8) | (2u << 16); pending = -1; ++next; }
  }
}

// Few rows: whether all rows of a problem at once (score_rows_kernel, a compute unit for each problem) are quicker than two passes, from
// what both take in us: a start, a time per problem and one per key, shared by 256 compute units; with all rows at once not less than
// the longest problem takes by itself, which may be the last to start where there are more problems than compute units.
static bool rows_quicker(int blocks, int d, bool fp8, int64_t problems, int64_t keys, int64_t most) {
  const float wide = (float)(d / 64), n = (float)problems, mean = (float)keys / n;
  const float longest = 1.5f * blocks + 0.0045f * wide * (float)most;
  const float shared = (n * (3.5f + 1.2f * blocks) + 0.0064f * wide * (float)keys) / 256.0f;
  const float last = n > 256.0f ? 0.0034f * wide * ((float)most - mean) : 0.0f;
  const float rows = 7.0f + fmaxf(longest, shared + last);
  const float passes = 11.0f + 2.0f * blocks + 1.5f * wide + (n * (1.7f + 0.4f * blocks) + (fp8 ? 0.0105f : 0.0117f) * wide * (float)keys) / 256.0f;
  return rows < passes;
}

// Are the teams quicker than the two passes, where none of the requests takes a route of its own?  Estimates in us, without what both need:
// a round takes its start and a time per pair of row blocks, however few of the 256 workgroups are in it; the passes take a time per key
// and pair, and one per key.  Measured, scores, both sides in turn in runs of 6 ms, 4 KV heads of 7 query heads, window 64 (448 rows),
// passes -> teams: 28 x 32K keys 890 -> 686 us (8-bit keys 826 -> 681), 28 x 20011 552 -> 466, 4 x 20011 89 -> 83, 16 x 8192 135 -> 104, 4 x 8192
// 53 -> 41, sixteen of 8K .. 48K 469 -> 409; 896 rows: 28 x 32K 1646 -> 1229, 28 x 5000 262 -> 229, 8 x 64K 954 -> 782; 8 KV heads, 256 rows: 8 x
// 64K 644 -> 550, 28 x 16K 574 -> 446; 224 rows: 4 x 32K 82 -> 69.  At the line: 224 rows 8 x 24000 112 -> 105; 4 KV heads of 4, 256 rows: 1 x 32K 39
// -> 34, 16 x 12000 124 -> 112.  Not taken, passes / teams: 1 x 8192 28 / 39, 1 x 16384 37 / 39, 2 x 20000 700 rows 79 / 82 (rounds that are nearly
// empty), 8 x 49152 402 / 403 (192 of 256 workgroups in a round), 28 x 50000 224 rows 824 / 801.
// The times are on the safe side: of 430 calls drawn over these ranges (1 to 32 layers, 1 to 16 requests, both key types) the rule takes 204,
// none of which gains less than 3 %, and leaves 84 that would gain more than 5, most of them of few rows or with 8-bit keys.  That pays for
// what it leaves out: places are emptied at 1.4 us a MB (up to 8 MB where lengths differ), 8-bit keys always take the kernel for 128 members
// (1.30 us a pair), and in calls one by one on an idle device, its clocks down, teams lose 3 to 7 % more than passes (8 x 24000 112 / 113).
static bool teams_quicker(int rounds, int pairs, int most, bool fp8, float keys) {
  const float teams = 4.0f + (float)rounds * (5.1f + (most <= 64 ? 1.27f : 1.35f) * (float)pairs);
  const float passes = keys / (256.0f * 512.0f) * (4.5f + 1.85f * (float)pairs) * (fp8 ? 0.93f : 1.0f);
  return teams < passes;
}

// Rounds of teams for calls whose requests all take the two passes otherwise: a request takes as many members as its keys need (one up to
// 512 keys), all problems the same time (they have the same rows), so a round is filled with teams, the largest first, and repeated while
// they last.  Scores with teams of one among them, passes -> teams, 448 rows: 6 layers of 32768 and 500 keys 189 -> 165 us (8-bit keys 183 ->
// 165), 28 layers of 5000 and eight times 500 310 -> 241 (266 -> 222).
static void schedule_teams(const codecomp_params* p, const Plan& pl, int64_t room, TeamSchedule* ts) {
  constexpr int nt = kTeamTiles;
  ts->steps = 0;
  const int LH = pl.L * pl.Hkv;
  struct Kind { int seq, chunks, left, next; } kind[kTeamEntries];
  int kinds = 0;
  int64_t keys = 0;
  for (int r = 0; r < pl.n_seqs; ++r) {
    const int n = p->cu_seqlens_host[r + 1] - p->cu_seqlens_host[r] - pl.key_trim;
    if (n <= 0) return;                                // nothing to do for it: left to the passes, which see to that
    keys += n;
    const int tiles = (n + 15) / 16, chunks = (tiles + 8 * nt - 1) / (8 * nt);
    // waves hold nt tiles or one less, the last wave of the last member nt: only a wave's tile nt - 1 may have places without a key
    if (chunks > kTeamMost || kinds == kTeamEntries || tiles / chunks <= 8 * (nt - 1)) return;
    int at = kinds++;
    for (; at > 0 && kind[at - 1].chunks < chunks; --at) kind[at] = kind[at - 1];
    kind[at] = {r, chunks, LH, 0};
  }
  struct Step { int rounds, used, first, count; } step[kTeamSteps];
  uint32_t entry[kTeamEntries][2];
  int steps = 0, entries = 0;
  for (;;) {
    Step s = {0, 0, entries, 0};
    for (int i = 0; i < kinds; ++i) {
      const int teams = kind[i].left < (kTeamMembers - s.used) / kind[i].chunks ? kind[i].left : (kTeamMembers - s.used) / kind[i].chunks;
      if (teams == 0) continue;
      if (entries == kTeamEntries) return;
      entry[entries][0] = (uint32_t)kind[i].seq | (uint32_t)teams << 16;
      entry[entries][1] = (uint32_t)kind[i].next | (uint32_t)kind[i].chunks << 16;
      ++entries; ++s.count;
      s.used += teams * kind[i].chunks;
      const int rounds = kind[i].left / teams;
      if (s.rounds == 0 || rounds < s.rounds) s.rounds = rounds;
    }
    if (s.count == 0) break;
    if (steps == kTeamSteps) return;
    for (int e = s.first, i = 0; e < entries; ++i)
      if ((int)(entry[e][0] & 0xFFFFu) == kind[i].seq) {
        const int done = (int)(entry[e][0] >> 16) * s.rounds;
        kind[i].left -= done; kind[i].next += done;
        ++e;
      }
    step[steps++] = s;
  }
  // fullest rounds first: a workgroup that has nothing to do in a round is through
  for (int i = 1; i < steps; ++i)
    for (int j = i; j > 0 && step[j - 1].used < step[j].used; --j) { const Step t = step[j]; step[j] = step[j - 1]; step[j - 1] = t; }
  int rounds = 0, n = 0;
  ts->most = kind[0].chunks;
  for (int i = 0; i < steps; ++i) {
    rounds += step[i].rounds;
    ts->step[i] = (uint32_t)step[i].rounds | (uint32_t)n << 16;
    for (int e = 0; e < step[i].count; ++e, ++n) { ts->entry[n][0] = entry[step[i].first + e][0]; ts->entry[n][1] = entry[step[i].first + e][1]; }
  }
  ts->step[steps] = (uint32_t)n << 16;
  ts->members = (step[0].used + 7) / 8 * 8;
  const int pairs = (pl.R + 31) / 32;
  ts->ring = kinds == 1;
  ts->line_pairs = ts->ring ? 16 : rounds * pairs;
  const int64_t counters = (int64_t)LH * pl.n_seqs * kTeamCounters * (int64_t)sizeof(uint32_t), per_problem = (int64_t)pairs * ts->most * 256;          // again, by half members; three at a time at least (team_tasks.h)
  ts->done_at = (room - counters) & ~(int64_t)255;
  if (room < counters || rounds > 0xFFFF || ts->done_at < (int64_t)ts->line_pairs * ts->members * 128 || ts->done_at < 3 * per_problem) return;
  ts->slots = (int)(ts->done_at / per_problem < LH * (int64_t)pl.n_seqs ? ts->done_at / per_problem : LH * (int64_t)pl.n_seqs);
  if (teams_quicker(rounds, pairs, ts->most, pl.kv_fp8, (float)(keys * LH))) ts->steps = steps;
}

int make_plan(const codecomp_params* p, Plan* pl) {
  if (!p) return CODECOMP_EINVAL_NULL;
  if (p->n_layers < 1 || p->n_seqs < 1 || p->n_seqs > 65535) return CODECOMP_EINVAL_SHAPE;
  if (p->select_mode != CODECOMP_SELECT_ADDITIVE && p->select_mode != CODECOMP_SELECT_TWO_STAGE) return CODECOMP_EINVAL_MODE;
  if (p->select_mode == CODECOMP_SELECT_TWO_STAGE &&
      (!(p->span_budget_ratio >= 0.0f) || !(p->span_budget_ratio <= 1.0f) || p->span_budget_min < 0))
    return CODECOMP_EINVAL_MODE;
  constexpr int kKnownVariants = CODECOMP_VARIANT_GROUP_SUM | CODECOMP_VARIANT_GROUP_MAX | CODECOMP_VARIANT_POOL_MAX |
                                 CODECOMP_VARIANT_SOFTMAX_PREFIX | CODECOMP_VARIANT_POOL_PREFIX | CODECOMP_VARIANT_NO_TEAMS |
                                 CODECOMP_VARIANT_TEAMS_APART;
  if ((p->score_variant & ~kKnownVariants) != 0) return CODECOMP_EINVAL_MODE;
  if (p->kv_dtype != CODECOMP_KV_BF16 && p->kv_dtype != CODECOMP_KV_FP8_E4M3) return CODECOMP_EINVAL_MODE;
  if ((p->score_variant & CODECOMP_VARIANT_GROUP_SUM) && (p->score_variant & CODECOMP_VARIANT_GROUP_MAX)) return CODECOMP_EINVAL_MODE;
  if ((p->score_variant & CODECOMP_VARIANT_NO_TEAMS) && (p->score_variant & CODECOMP_VARIANT_TEAMS_APART)) return CODECOMP_EINVAL_MODE;
  if ((int64_t)p->n_layers * p->n_kv_heads > 65535) return CODECOMP_EINVAL_SHAPE;   // one grid axis
  if (p->n_kv_heads < 1 || p->n_q_heads < 1 || p->n_q_heads % p->n_kv_heads != 0) return CODECOMP_EINVAL_HEADS;
  if (p->head_dim != 64 && p->head_dim != 128) return CODECOMP_EINVAL_HEADDIM;
  if (p->pool_kernel < 1 || p->pool_kernel % 2 == 0 || p->pool_kernel > 1025) return CODECOMP_EINVAL_POOL;
  if (!(p->prior_weight >= 0.0f) || !isfinite(p->prior_weight)) return CODECOMP_EINVAL_PRIOR;
  if (!(p->softmax_scale >= 0.0f) || !isfinite(p->softmax_scale)) return CODECOMP_EINVAL_PRIOR;
  if (!p->cu_seqlens_host || !p->cu_seqlens_dev || !p->cu_budgets_host || !p->cu_budgets_dev)
    return CODECOMP_EINVAL_NULL;
  if (p->window < 1) return CODECOMP_EINVAL_WINDOW;
  if (p->cu_seqlens_host[0] != 0 || p->cu_budgets_host[0] != 0) return CODECOMP_EINVAL_SEQLENS;
  int max_n = 0, max_b = 0;
  for (int r = 0; r < p->n_seqs; ++r) {
    int64_t n = (int64_t)p->cu_seqlens_host[r + 1] - p->cu_seqlens_host[r];
    int64_t b = (int64_t)p->cu_budgets_host[r + 1] - p->cu_budgets_host[r];
    if (n < 1 || b < 0) return CODECOMP_EINVAL_SEQLENS;
    if (p->window > n) return CODECOMP_EINVAL_WINDOW;
    if (b < p->window || b > n) return CODECOMP_EINVAL_BUDGET;
    if (n > max_n) max_n = (int)n;
    if (b > max_b) max_b = (int)b;
  }
  const int64_t strides[] = {p->q_stride_layer, p->q_stride_seq, p->q_stride_head, p->q_stride_tok,
                             p->kv_stride_layer, p->kv_stride_head, p->kv_stride_tok,
                             p->out_stride_layer, p->out_stride_head, p->out_stride_tok};
  for (int64_t s : strides)
    if (s < 0 || s % 8 != 0) return CODECOMP_EINVAL_SHAPE;   // rows are moved as 16-byte pieces
  if (p->kv_dtype == CODECOMP_KV_FP8_E4M3)                   // ... which hold 16 one-byte elements
    for (int i = 4; i < 10; ++i)
      if (strides[i] % 16 != 0) return CODECOMP_EINVAL_SHAPE;

  pl->L = p->n_layers; pl->Hq = p->n_q_heads; pl->Hkv = p->n_kv_heads; pl->G = pl->Hq / pl->Hkv;
  pl->d = p->head_dim; pl->W = p->window; pl->pool = p->pool_kernel; pl->n_seqs = p->n_seqs;
  pl->select_mode = p->select_mode;
  pl->variant = p->score_variant;
  pl->kv_fp8 = p->kv_dtype == CODECOMP_KV_FP8_E4M3 ? 1 : 0;
  pl->key_trim = (p->score_variant & CODECOMP_VARIANT_SOFTMAX_PREFIX) ? p->window : 0;
  pl->span_ratio = p->span_budget_ratio; pl->span_min = p->span_budget_min;
  // two-stage selection keeps the prior out of the scores: structure is handled by the selection itself
  pl->lambda = p->select_mode == CODECOMP_SELECT_TWO_STAGE ? 0.0f : p->prior_weight;
  pl->scale = p->softmax_scale > 0.0f ? p->softmax_scale : 1.0f / sqrtf((float)p->head_dim);
  pl->T = p->cu_seqlens_host[p->n_seqs];
  pl->TB = p->cu_budgets_host[p->n_seqs];
  pl->max_n = max_n;
  pl->max_b = max_b;
  int64_t R = (int64_t)pl->G * pl->W;
  if (R > (1 << 16)) return CODECOMP_EINVAL_SHAPE;
  pl->R = (int)R;
  const int max_rows = kMaxWaves * kRowsPerWave;
  pl->row_splits = (pl->R + max_rows - 1) / max_rows;
  int per = (pl->R + pl->row_splits - 1) / pl->row_splits;
  pl->row_blocks = (per + 31) / 32;
  assign_row_blocks(pl);
  // the largest head mass is taken per workgroup from whole row blocks: one head per block, all rows in one workgroup
  if ((pl->variant & CODECOMP_VARIANT_GROUP_MAX) && (pl->W % 32 != 0 || pl->row_splits != 1)) return CODECOMP_EINVAL_MODE;
  if (p->score_workgroups < 0 || p->score_lead_tiles > 64) return CODECOMP_EINVAL_SHAPE;
  pl->grid_override = p->score_workgroups;
  int64_t tiles = 0, keys = 0, tiles_short = 0, tiles_long = 0;          // short, long: of those that one pass could take
  int once_short = 0, once_long = 0;
  for (int r = 0; r < p->n_seqs; ++r) {
    int n = p->cu_seqlens_host[r + 1] - p->cu_seqlens_host[r] - pl->key_trim;     // >= 0: W <= N_r was checked
    const int t = (n + kTileKeys - 1) / kTileKeys;
    tiles += t;
    keys += n;
    if (n > 0 && n <= kOnceKeys / 2) { tiles_short += t; ++once_short; }
    else if (n > 0 && n <= kOnceKeys) { tiles_long += t; ++once_long; }
  }
  const int64_t problems = (int64_t)pl->L * pl->Hkv * pl->row_splits;
  const int automatic_lead = tiles > 0 && tiles * problems <= kNoLeadTiles ? 0 : kLeadTiles;
  pl->lead_tiles = p->score_lead_tiles == 0 ? automatic_lead : (p->score_lead_tiles < 0 ? 0 : p->score_lead_tiles);
  int64_t positions = tiles + (int64_t)pl->lead_tiles * pl->n_seqs;
  if (positions * problems > (1 << 30)) return CODECOMP_EINVAL_SHAPE;
  const int64_t LH64 = (int64_t)pl->L * pl->Hkv;
  const int64_t most = max_n - pl->key_trim;           // keys of the longest request
  const bool own_rules = !(pl->variant & CODECOMP_VARIANT_GROUP_MAX) && p->score_workgroups == 0 && p->score_lead_tiles == 0;
  const bool all_once = once_short + once_long > 0 && tiles_short + tiles_long == tiles;
  pl->rows_at_once = own_rules && pl->R <= kRowsMost && most > kOnceKeys && most <= 128 * rows_tiles((pl->R + 15) / 16) &&
                     LH64 * pl->n_seqs >= kRowsProblems && rows_quicker((pl->R + 15) / 16, pl->d, pl->kv_fp8 != 0, LH64 * pl->n_seqs, LH64 * keys, most);
  if (!own_rules || pl->rows_at_once) {
    once_short = once_long = 0;
  } else if (all_once) {
    if (pl->row_splits >= kOnceWide && (once_short + once_long) * LH64 <= kOnceWideProblems) once_short = once_long = 0;
  } else {
    const int64_t workgroups = LH64 * pl->row_splits;          // per request
    const bool few = pl->R <= kRowsMost;
    const float rounds = (float)(once_long * workgroups) / (float)kOnceFill;
    const bool long_pays = few ? once_long * workgroups >= kOnceMixedLongFew : rounds - kOnceRound * ceilf(rounds) >= kOnceAhead + kOnceStart / (2.0f * (float)pl->row_blocks);
    if (once_short * workgroups < (few ? kOnceMixedShortFew : kOnceMixedShort) || (few && 2 * tiles_short < 5 * once_short)) once_short = 0;
    if (!long_pays || (once_short == 0 && tiles_short > 0)) once_long = 0;
  }
  const bool once = once_short + once_long > 0;
  const int64_t once_problems = (once_short + once_long) * LH64;
  pl->once_keys = once_long > 0 ? kOnceKeys : once ? kOnceKeys / 2 : 0;
  pl->once_short = once_short;
  pl->once_long = once_long;
  pl->once_rows = pl->row_blocks * 32;
  pl->once_chunks = pl->row_splits;
  // statistics (one slot per segment and row split; slot numbers stay below (teams + problems) * row_splits) and merged row normalisers
  const int64_t stat_bytes = (kMaxScoreGrid + LH64 * pl->row_splits * pl->n_seqs) * (pl->waves * kRowsPerWave) * 2 * (int64_t)sizeof(float);
  const int64_t lse_bytes = LH64 * pl->n_seqs * pl->row_splits * pl->row_blocks * 32 * (int64_t)sizeof(float);
  if (once && all_once && once_problems < kOnceFill) {
    // few problems: smaller chunks of rows, of at least four blocks of 16, until the compute units are used
    const int blocks = (pl->R + 15) / 16;
    int64_t chunks = kOnceFill / once_problems;
    if (chunks > (blocks + 3) / 4) chunks = (blocks + 3) / 4;
    while (4 * chunks * chunks > kOnceArrays * blocks) --chunks;           // an array of masses each
    // More arrays than row splits lie over statistics and normalisers (below).  Requests without a key need no chunk, but every array
    // has a place for their tokens.
    const int64_t room = pl->row_splits + (stat_bytes + lse_bytes) / (LH64 * pl->T * (int64_t)sizeof(float));
    if (chunks > room) chunks = room;
    if (chunks < pl->row_splits) chunks = pl->row_splits;
    pl->once_rows = (int)((blocks + chunks - 1) / chunks) * 16;
    pl->once_chunks = (pl->R + pl->once_rows - 1) / pl->once_rows;
  }
  // how many of them a workgroup takes in turn: what fills the compute units best (figures at kOnceReload)
  pl->once_group = 1;
  if (once && pl->once_chunks > 1) {
    const float slots = once_long > 0 ? (float)kOnceFill : 2.0f * (float)kOnceFill;
    float best = INFINITY;
    for (int group = 1; group <= pl->once_chunks; ++group) {
      const float rounds = (float)(once_problems * ((pl->once_chunks + group - 1) / group)) / slots;
      const float cost = (rounds > 4.0f ? rounds + 0.5f : ceilf(rounds)) * ((float)group + kOnceReload);
      if (cost < best) { best = cost; pl->once_group = group; }
    }
  }
  pl->mass_parts = once && all_once ? pl->once_chunks : pl->row_splits;
  if (pl->rows_at_once) tiles = 0;
  if (once) {
    const int64_t taken = (once_short > 0 ? tiles_short : 0) + (once_long > 0 ? tiles_long : 0);
    tiles -= taken;
    positions -= taken + (int64_t)pl->lead_tiles * (once_short + once_long);
  }
  pl->tiles_per_problem = (int)positions;
  pl->total_tiles = (int)(positions * pl->L * pl->Hkv);      // the row splits of a problem walk the same positions
  pl->real_tiles = (int)(tiles * pl->L * pl->Hkv);

  const int64_t d = pl->d;
  pl->q_st = p->q_stride_tok ? p->q_stride_tok : d;
  pl->q_sh = p->q_stride_head ? p->q_stride_head : (int64_t)pl->W * d;
  pl->q_ss = p->q_stride_seq ? p->q_stride_seq : (int64_t)pl->Hq * pl->W * d;
  pl->q_sl = p->q_stride_layer ? p->q_stride_layer : (int64_t)pl->n_seqs * pl->Hq * pl->W * d;
  pl->kv_st = p->kv_stride_tok ? p->kv_stride_tok : d;
  pl->kv_sh = p->kv_stride_head ? p->kv_stride_head : (int64_t)pl->T * d;
  pl->kv_sl = p->kv_stride_layer ? p->kv_stride_layer : (int64_t)pl->Hkv * pl->T * d;
  pl->o_st = p->out_stride_tok ? p->out_stride_tok : d;
  pl->o_sh = p->out_stride_head ? p->out_stride_head : (int64_t)pl->TB * d;
  pl->o_sl = p->out_stride_layer ? p->out_stride_layer : (int64_t)pl->Hkv * pl->TB * d;
  if (pl->q_st < d || pl->kv_st < d || pl->o_st < d) return CODECOMP_EINVAL_SHAPE;
  if (pl->kv_st > (1 << 20)) return CODECOMP_EINVAL_SHAPE;   // tile staging keeps 32-bit byte offsets inside a tile
  pl->cu_seqlens_dev = p->cu_seqlens_dev;
  pl->cu_budgets_dev = p->cu_budgets_dev;

  // workspace: per-chunk softmax statistics, merged row normalisers, raw attention mass
  const size_t LH = (size_t)pl->L * pl->Hkv;
  size_t off = 0;
  pl->off_stats = off; off = align256(off + (size_t)stat_bytes);
  pl->off_lse = off;   off = align256(off + (size_t)lse_bytes);
  pl->off_uraw = off;  off = align256(off + (size_t)pl->row_splits * LH * pl->T * sizeof(float));
  pl->off_member = off; off = align256(off + (size_t)pl->T);
  pl->off_member_count = off; off = align256(off + (size_t)pl->n_seqs * sizeof(int32_t));
  // selection by parts: per (layer*head, part) the first-digit counts and the number of candidates admitted whatever
  // the cut; per (layer*head, request) what the parts agreed on.  The keys near the cut reuse the raw attention mass
  // (dead once the scores exist): one 32-bit word per token and layer*head, exactly its size.
  pl->sel_parts = 0;
  if (max_n - p->window > kSelectMaxCandidates) {
    int64_t parts = 0;
    for (int r = 0; r < p->n_seqs; ++r) {
      const int npre = p->cu_seqlens_host[r + 1] - p->cu_seqlens_host[r] - p->window;
      parts += npre > kPartChunk ? (npre + kPartChunk - 1) / kPartChunk : 1;
    }
    if (parts > (1 << 24)) return CODECOMP_EINVAL_SHAPE;
    pl->sel_parts = (int)parts;
    pl->off_part_hist = off; off = align256(off + LH * (size_t)parts * kFirstDigitBins * sizeof(uint16_t));
    pl->off_part_sure = off; off = align256(off + LH * (size_t)parts * sizeof(int32_t));
    pl->off_part_head = off; off = align256(off + LH * (size_t)pl->n_seqs * 8 * sizeof(uint32_t));
    pl->off_part_before = off; off = align256(off + LH * (size_t)parts * 2 * sizeof(int32_t));
  }
  pl->ws_bytes = off;
  pl->team.steps = 0;
  if (own_rules && !(pl->variant & CODECOMP_VARIANT_NO_TEAMS) && !once && !pl->rows_at_once && pl->R >= 192 && pl->R <= kTeamRows && pl->d == 128 &&
      LH64 * pl->n_seqs <= 65535 &&
      (int64_t)max_n * pl->kv_st * (pl->kv_fp8 ? 1 : 2) <= 0xFFFFFFFFll - 4096 &&
      ((int64_t)(pl->G - 1) * pl->q_sh + (int64_t)(pl->W - 1) * pl->q_st) / 8 <= 0xFFFF)
    schedule_teams(p, *pl, (int64_t)(pl->off_lse - pl->off_stats), &pl->team);
  // Calls without two-pass requests keep no statistics: more mass arrays than row splits take their place as well.  The number of chunks
  // is bounded by what fits.  Without requests that have no key it always does: problems * chunks <= kOnceFill and a problem has at most
  // R + kOnceKeys tokens, so the arrays beyond the row splits hold 4 * kOnceFill * (R + kOnceKeys) * (1 - splits / chunks) bytes at most,
  // which with chunks <= 1.5 * sqrt(R / 16) is below 5.9 MB (at R = 16384); the statistics have kMaxScoreGrid slots of 4 KB above 256
  // rows, and of 512 bytes per two blocks of 32 rows below.
  if (pl->mass_parts > pl->row_splits) pl->off_uraw = 0;
  return CODECOMP_OK;
}

int launch_compress(const Plan& pl, const void* q, const void* k, const void* v, const float* prior, float* scores, int32_t* idx,
                    void* k_out, void* v_out, void* workspace, hipStream_t stream) {
  if (fused_tail(pl)) {
    if (int rc = launch_score(pl, q, k, prior, scores, workspace, stream, CODECOMP_STAGE_ALL & ~CODECOMP_STAGE_FINISH)) return rc;
    if (int rc = launch_finish_select(pl, prior, scores, idx, k, v, k_out, v_out, workspace, stream)) return rc;
    if (fused_copy(pl)) return 0;
  } else {
    if (int rc = launch_score(pl, q, k, prior, scores, workspace, stream)) return rc;
    const int rc = pl.select_mode == CODECOMP_SELECT_TWO_STAGE ? launch_select_two_stage(pl, scores, prior, idx, workspace, stream)
                                                               : launch_select(pl, scores, idx, workspace, stream);
    if (rc) return rc;
  }
  return launch_gather(pl, k, v, idx, k_out, v_out, stream);
}

static int check_ws(const Plan& pl, const void* ws, size_t bytes) {
  if (!ws || ((uintptr_t)ws & 255) != 0 || bytes < pl.ws_bytes) return CODECOMP_EINVAL_WORKSPACE;
  return CODECOMP_OK;
}

static bool misaligned16(const void* p) { return ((uintptr_t)p & 15) != 0; }

}  // namespace codecomp

using namespace codecomp;

extern "C" {

size_t codecomp_workspace_bytes(const codecomp_params* params) {
  Plan pl;
  if (make_plan(params, &pl) != CODECOMP_OK) return 0;
  return pl.ws_bytes;
}

int codecomp_validate(const codecomp_params* params) {
  Plan pl;
  return make_plan(params, &pl);
}

int codecomp_score_layout(const codecomp_params* params, int32_t* row_splits, int32_t* row_blocks,
                          int32_t* waves, uint32_t* wave_desc) {
  Plan pl;
  if (int rc = make_plan(params, &pl)) return rc;
  if (row_splits) *row_splits = pl.row_splits;
  if (row_blocks) *row_blocks = pl.row_blocks;
  if (waves) *waves = pl.waves;
  if (wave_desc)
    for (int w = 0; w < kMaxWaves; ++w) wave_desc[w] = w < pl.waves ? pl.wave_desc[w] : 0u;
  return CODECOMP_OK;
}

int codecomp_score_route(const codecomp_params* params, int32_t* route, int32_t* row_chunks, int32_t* chunks_in_turn) {
  Plan pl;
  if (int rc = make_plan(params, &pl)) return rc;
  for (int r = 0; route && r < pl.n_seqs; ++r) {
    const int n = params->cu_seqlens_host[r + 1] - params->cu_seqlens_host[r] - pl.key_trim;
    route[r] = n <= 0 ? CODECOMP_ROUTE_TWO_PASSES : pl.rows_at_once ? CODECOMP_ROUTE_FEW_ROWS
             : n <= pl.once_keys ? CODECOMP_ROUTE_ONE_PASS : CODECOMP_ROUTE_TWO_PASSES;
  }
  if (row_chunks) *row_chunks = pl.once_keys > 0 ? pl.once_chunks : 0;
  if (chunks_in_turn) *chunks_in_turn = pl.once_keys > 0 ? pl.once_group : 0;
  return CODECOMP_OK;
}

int codecomp_score_teams(const codecomp_params* params, int32_t* members) {
  Plan pl;
  if (int rc = make_plan(params, &pl)) return rc;
  if (members) *members = pl.team.steps > 0 ? pl.team.most : 0;
  return CODECOMP_OK;
}

int codecomp_score(const void* q_obs, const void* k, const float* prior, const codecomp_params* params,
                   float* scores, void* workspace, size_t workspace_bytes, void* hip_stream) {
  if (!q_obs || !k || !prior || !params || !scores) return CODECOMP_EINVAL_NULL;
  Plan pl;
  if (int rc = make_plan(params, &pl)) return rc;
  if (misaligned16(q_obs) || misaligned16(k)) return CODECOMP_EINVAL_SHAPE;
  if (int rc = check_ws(pl, workspace, workspace_bytes)) return rc;
  return launch_score(pl, q_obs, k, prior, scores, workspace, (hipStream_t)hip_stream);
}

int codecomp_score_stages(const void* q_obs, const void* k, const float* prior, const codecomp_params* params,
                          float* scores, void* workspace, size_t workspace_bytes, unsigned stages,
                          void* hip_stream) {
  if (!q_obs || !k || !prior || !params || !scores) return CODECOMP_EINVAL_NULL;
  if (stages == 0 || (stages & ~(unsigned)CODECOMP_STAGE_ALL)) return CODECOMP_EINVAL_SHAPE;
  Plan pl;
  if (int rc = make_plan(params, &pl)) return rc;
  if (misaligned16(q_obs) || misaligned16(k)) return CODECOMP_EINVAL_SHAPE;
  if (int rc = check_ws(pl, workspace, workspace_bytes)) return rc;
  return launch_score(pl, q_obs, k, prior, scores, workspace, (hipStream_t)hip_stream, stages);
}

int codecomp_select(const float* scores, const codecomp_params* params, int32_t* idx, void* workspace,
                    size_t workspace_bytes, void* hip_stream) {
  if (!scores || !params || !idx) return CODECOMP_EINVAL_NULL;
  Plan pl;
  if (int rc = make_plan(params, &pl)) return rc;
  if (pl.select_mode != CODECOMP_SELECT_ADDITIVE) return CODECOMP_EINVAL_MODE;   // the prior is needed: other entry
  if (int rc = check_ws(pl, workspace, workspace_bytes)) return rc;
  return launch_select(pl, scores, idx, workspace, (hipStream_t)hip_stream);
}

int codecomp_select_two_stage(const float* scores, const float* prior, const codecomp_params* params, int32_t* idx,
                              void* workspace, size_t workspace_bytes, void* hip_stream) {
  if (!scores || !prior || !params || !idx) return CODECOMP_EINVAL_NULL;
  Plan pl;
  if (int rc = make_plan(params, &pl)) return rc;
  if (pl.select_mode != CODECOMP_SELECT_TWO_STAGE) return CODECOMP_EINVAL_MODE;
  if (int rc = check_ws(pl, workspace, workspace_bytes)) return rc;
  return launch_select_two_stage(pl, scores, prior, idx, workspace, (hipStream_t)hip_stream);
}

int codecomp_gather(const void* k, const void* v, const int32_t* idx, const codecomp_params* params,
                    void* k_out, void* v_out, void* hip_stream) {
  if (!k || !v || !idx || !params || !k_out || !v_out) return CODECOMP_EINVAL_NULL;
  Plan pl;
  if (int rc = make_plan(params, &pl)) return rc;
  if (misaligned16(k) || misaligned16(v) || misaligned16(k_out) || misaligned16(v_out)) return CODECOMP_EINVAL_SHAPE;
  return launch_gather(pl, k, v, idx, k_out, v_out, (hipStream_t)hip_stream);
}

int codecomp_compress(const void* q_obs, const void* k, const void* v, const float* prior,
                      const codecomp_params* params, float* scores, int32_t* idx, void* k_out, void* v_out,
                      void* workspace, size_t workspace_bytes, void* hip_stream) {
  if (!q_obs || !k || !v || !prior || !params || !scores || !idx || !k_out || !v_out) return CODECOMP_EINVAL_NULL;
  Plan pl;
  if (int rc = make_plan(params, &pl)) return rc;
  if (misaligned16(q_obs) || misaligned16(k) || misaligned16(v) || misaligned16(k_out) || misaligned16(v_out))
    return CODECOMP_EINVAL_SHAPE;
  if (int rc = check_ws(pl, workspace, workspace_bytes)) return rc;
  return launch_compress(pl, q_obs, k, v, prior, scores, idx, k_out, v_out, workspace, (hipStream_t)hip_stream);
}

const char* codecomp_status_string(int status) {
  switch (status) {
    case CODECOMP_OK: return "ok";
    case CODECOMP_EINVAL_NULL: return "a required pointer is NULL";
    case CODECOMP_EINVAL_SHAPE: return "bad shape, stride or alignment";
    case CODECOMP_EINVAL_WINDOW: return "window must satisfy 1 <= W <= N_r for every request";
    case CODECOMP_EINVAL_BUDGET: return "budget must satisfy W <= B_r <= N_r for every request";
    case CODECOMP_EINVAL_POOL: return "pool_kernel must be odd and >= 1";
    case CODECOMP_EINVAL_HEADS: return "n_q_heads must be a positive multiple of n_kv_heads";
    case CODECOMP_EINVAL_HEADDIM: return "head_dim must be 64 or 128";
    case CODECOMP_EINVAL_SEQLENS: return "cu_seqlens / cu_budgets must start at 0 and increase";
    case CODECOMP_EINVAL_WORKSPACE: return "workspace is NULL, not 256-byte aligned or too small";
    case CODECOMP_EINVAL_PRIOR: return "prior_weight / softmax_scale must be finite and >= 0";
    case CODECOMP_EINVAL_MODE: return "select_mode unknown or wrong for this call, or span budget out of range";
    default: return status > 0 ? "HIP runtime error (hipError_t value)" : "unknown status";
  }
}

int codecomp_version(void) { return 100; }

}  // extern "C"
