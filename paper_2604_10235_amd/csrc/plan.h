// Host-side launch plan shared by the translation units of libcodecomp (internal header).
#pragma once
#include <hip/hip_runtime.h>
#include <stddef.h>
#include <stdint.h>

#include "codecomp.h"

namespace codecomp {

constexpr int kRowsPerWave = 64;      // query rows (window x group) one wavefront can own: two blocks of 32
constexpr int kMaxWaves = 8;          // wavefronts per workgroup in the score kernels
constexpr int kTileKeys = 64;         // keys staged through LDS per pipeline step
// One pass over the logits (score_once.h): the keys of a request in the registers of one workgroup.  A call whose requests are all
// that short takes it (but for a few problems of very many rows, below): 1.1 to 2.4 times faster than two passes from one problem of
// 130 keys to 4096 of 760, head_dim 64 and 128, 32 to 896 rows (figures there).
constexpr int kOnceTiles = 6;           // most tiles of 16 keys a wave holds; with seven the eight-wave kernel spills inside its loop
constexpr int kOnceKeys = 16 * kOnceTiles * 8;      // keys of the longest request that takes one pass
constexpr int kOnceRows = 512;          // most query rows of a chunk
constexpr int kOnceFill = 256;          // workgroups that find a compute unit of their own at once: up to here a problem's rows are shared out
// In a call with longer requests too, the kernel runs after their two passes: one launch for requests of up to kOnceKeys / 2 keys
// (512 workgroups at a time), one for the others (256 at a time), each of 15 to 30 us however little it has to do, while the passes
// would have taken its requests along.  Workgroups counted as requests * heads * row splits, the shorter ones gain about half their
// time and pay from little more than one round on (kOnceMixedShort).  The others gain a fifth to a third, so that a begun round
// costs more than it brings unless there are many or it is nearly full (kOnceRound, kOnceAhead: 256 problems of 700 in one full round
// 98 -> 116 us), and the start costs about as much as kOnceStart blocks of 16 rows.  With few rows the passes' workgroups are small,
// many to a compute unit, and lose less to short requests: later lines, and requests of 128 keys or more on average.  One pass takes
// what is shorter than some length, so the longer ones go only with the shorter.
// Scores, all in two passes -> short ones apart: 28 query heads on 4, window 64: 520 short problems of 200 among 8 of 4000 85 -> 82 us,
// 520 of 700 133 -> 146, 512 of 600 among 512 of 5000 738 -> 700; window 128: 520 of 200 139 -> 121; 16 rows, 4000 of 20 among 96 of
// 4096, head_dim 128 88 -> 100; 40 rows, 1792 of 43 98 % as fast, 2064 of 260 84 -> 72, 7000 of 686 628 -> 479.  600 batches of 45 to
// 8192 short problems among longer ones, 16 to 896 rows: with one line at 512 short problems of any length 41 were slower than two
// passes by 3 % or more (the worst 0.75), with these 11 (0.91).
constexpr int kOnceMixedShort = 640;
constexpr float kOnceRound = 0.8f, kOnceAhead = 0.2f, kOnceStart = 3.0f;
constexpr int kOnceMixedShortFew = 2560, kOnceMixedLongFew = 1536;             // up to kRowsMost rows
// Each chunk has an array of masses of its own, which the pooling adds up: 0.3 to 0.5 us an array in a short call, against 0.9 us for
// each block of 16 rows that a chunk has more.  So at most 1.5 * sqrt(blocks) chunks (their square at most kOnceArrays / 4 * blocks),
// unless chunks of kOnceRows are more.  One request of 768 tokens, 4096 rows, scores: 64 chunks 45.1 us, 32 33.7, 16 32.6, 8 41.1.
constexpr int kOnceArrays = 9;
// From 1537 rows on, one or two problems take two passes, whose workgroups share out the keys, too.  Scores of 768 keys, two passes
// and one pass: one problem of 2048 rows 23.2 and 26.1 us, of 4096 25.6 and 32.6, of 16384 44.6 and 52.5; two 25.1 and 27.0, 27.9 and
// 33.2, 52.6 and 54.2; four 26.3 and 27.7, 33.9 and 33.9, 65.5 and 54.8; eight 32.5 and 28.3, 41.6 and 34.8, 81.8 and 56.5.
constexpr int kOnceWide = 4, kOnceWideProblems = 2;         // row splits, problems
// A workgroup may take several chunks of a problem in turn: the keys are loaded once.  That saves kOnceReload of a chunk's time and
// is taken only where it leaves no compute unit idle: 896 rows (two chunks), scores, a chunk each and two in turn: 256 problems of 768
// keys 76.9 and 70.0 us, 400 136 and 123, but 260 104 and 125.  (In turn wherever all chunks did not find a compute unit at once, 16
// problems of 16384 rows took 838 us, two passes 130; now 96.)
constexpr float kOnceReload = 0.16f;
// Few rows (up to kRowsMost): tiles of 16 keys per wave whose logits eight waves hold, by blocks of 16 rows; taken where a request is
// too long for its keys to stay in registers, the problems use the device and the longest request does not set the time (rows_quicker in
// api.hip).  Two passes -> all rows at once: 128 problems of 1000 keys, 16 rows, head_dim 64 20 -> 12 us (call), 32 rows, head_dim 128
// 31 -> 18, of 2500 47 -> 32; 4096 of 1000 and 2500, 32 rows, head_dim 64 263 -> 176, 583 -> 376.  With 4 to 32 problems it is 30 %
// faster to 30 % slower (2500 keys), and requests of up to kOnceKeys are up to twice as fast with their keys in registers.  Lengths mixed,
// 16 rows, 4 KV heads, scores: 50 requests of 100 to 4096 tokens, head_dim 128 52 -> 39 us, but 2000 of 100 and one of 1000 98 -> 140, 100 of
// 100 and one of 4096 27 -> 45.
constexpr int kRowsMost = 64, kRowsProblems = 96;
constexpr int rows_tiles(int blocks) { return blocks == 1 ? 32 : blocks == 2 ? 20 : blocks == 3 ? 12 : 8; }
// Long requests in one pass, by teams of workgroups (score_team.h).
constexpr int kTeamMembers = 256;     // workgroups of a launch, each with a compute unit of its own
// Most members of a team.  In every pair of row blocks each waits for the sums of all and adds them up: with 256 members a pair takes 1.87
// us instead of 1.3 (4 x 100000 keys, 896 rows 926 us, by two passes 723; 8 x 128K, 256 rows 1373 and 1265).
constexpr int kTeamMost = 128;
constexpr int kTeamTiles = 4;         // tiles of 16 keys per wave
constexpr int kTeamRows = 1024;       // most query rows
constexpr int kTeamCounters = 8;      // words of a problem that count what has been done again
constexpr int kTeamSteps = 48, kTeamEntries = 96;          // rounds that are alike, groups of teams in them
struct TeamSchedule {
  int steps;                          // 0: not taken
  int members, most;                  // workgroups; members of the largest team
  int ring;                           // 1: teams stay the same, the places of sums are used in turn
  int line_pairs;                     // places, in pairs of row blocks
  int slots;                          // problems whose sums have a place at a time when the work has to be done again
  int64_t done_at;                    // counters of that, in bytes from the places
  uint32_t step[kTeamSteps + 1];      // rounds | first entry << 16
  uint32_t entry[kTeamEntries][2];    // request | teams << 16, first (layer, head) | members of a team << 16
};
constexpr int kMaxScoreGrid = 2048;   // most workgroups a score pass is launched with
constexpr int kLeadTiles = 4;         // a segment start (query fragments, first K tile) costs about this many tiles
// Calls of up to this many (tile, row split) pairs get no leads: a workgroup then has one tile or two and nearly all of them start
// exactly one segment, so that a lead only leaves some workgroups idle and others with twice the tiles.  Scores, with -> without
// leads: one layer of 2000 tokens, head_dim 64 (128 pairs) 16.0 -> 15.3 us, 8192 of 28 query heads (512) 29.2 -> 27.4, 4096 with
// window 128 (512) 30.0 -> 28.2, 16 requests of 512 (512) 34.5 -> 33.1, 9000 of 2 KV heads (282) 28.0 -> 28.1.  Above the line one
// request still gains or stays (8192 x 2 layers (1024) 36.0 -> 34.7, 9000 (564) 29.2 -> 29.2, 20000 (1252) 36.4 -> 36.6), but
// many problems or requests of different lengths start two segments in some workgroups and lose: 28 layers of 2048 (3584)
// 76.4 -> 80.6, five requests of up to 5000 (596) 31.3 -> 39.8.  Such a batch loses below it too (298 pairs: 28.8 -> 36.6).
constexpr int kNoLeadTiles = 512;
// (layer, head, request) problems from which on smaller selection workgroups, several to a compute unit, are taken.  Selection with
// small -> with large ones: 256 problems of 8000 candidates 8.3 -> 7.3 us, of 16000 11.9 -> 10.4; 384 of 8000 9.9 -> 8.4, of 16000
// 15.6 -> 18.6; 512 of 8000 10.1 -> 8.6, of 12000 13.6 -> 17.0; 1024 of 4000 10.1 -> 10.9, of 8000 15.3 -> 15.4, of 16000
// 30.6 -> 38.8; 2048 of 2000 8.4 -> 10.4.  From two problems per compute unit on the small ones are ahead or (up to 8192
// candidates, 512 and 640 problems) up to 17 % behind.
constexpr int kSelectManyProblems = 512;
// Longer requests are selected by several workgroups each: parts of kPartChunk candidates, one 256-thread workgroup
// per part and step (first-digit counts, the candidates near the cut, the ordered output; between the last two one
// workgroup per request finds the cut among those candidates).
constexpr int kPartThreads = 256;
constexpr int kPartItems = 32;                             // candidates a thread holds
constexpr int kPartChunk = kPartThreads * kPartItems;      // candidates per part
constexpr int kSelectMaxCandidates = 65536;                // most candidates one workgroup keeps in registers (64 per thread)
// Up to there one workgroup per problem is quicker than parts, however few the problems.  Parts -> one workgroup: one problem of
// 16384 candidates 34.5 -> 9.9 us, of 65536 37.5 -> 29.1; 64 of 65536 49.6 -> 31.0; one of 65536 with a binary prior 45.2 ->
// 37.0, of one value only 128 -> 75; two-stage, 64 of 65536 107 -> 86.

// A workgroup that selects copies the kept rows, too, up to this many bytes of K and V (read): a launch less.  Whole call, own kernel ->
// copied along, 64 KB: 4 KV heads of 2048 tokens, head_dim 64, 256 kept 18.8 -> 17.8 us; head_dim 128, 2000 tokens, 128 kept 21.0 -> 20.1;
// 28 layers of them 24.9 -> 23.4 and 32.4 -> 31.1.  More: head_dim 64, 512 kept 20.0 -> 20.0, 1024 20.4 -> 22.6; head_dim 128, 512 kept
// 28.2 -> 31.0.
constexpr int64_t kCopyBytes = 65536;
constexpr int kFirstDigitBins = 2048;
constexpr int kFinishHalo = 512;      // largest supported (pool_kernel - 1) / 2

struct Plan {
  int L, Hq, Hkv, G, d, W, pool, n_seqs;
  float lambda, scale;
  int select_mode;           // CODECOMP_SELECT_*
  int variant;               // CODECOMP_VARIANT_* flags
  int key_trim;              // keys at the end of every request that the softmax leaves out (W or 0)
  int kv_fp8;                // 1: k, v and the compact cache hold one FP8 E4M3 code per element (else bf16)
  float span_ratio; int span_min;
  int T, TB;                 // total tokens / total output slots over the packed requests
  int max_n;                 // longest request
  int max_b;                 // largest budget
  int R;                     // G * W softmax rows per (layer, KV head, request)
  int row_splits;            // workgroups along the row axis (each <= kMaxWaves * kRowsPerWave rows)
  int row_blocks;            // blocks of 32 rows per split
  int waves;                 // wavefronts per workgroup of the score passes
  // Which row blocks each wave computes: block of slot 0 | block of slot 1 << 8 | halves << 16, where
  // slot 0 covers both 32-key halves of every tile and `halves` (bit 0 first, bit 1 second) says which
  // ones slot 1 covers (0: the wave has no slot 1).
  uint32_t wave_desc[kMaxWaves];
  uint8_t rb_holder[2 * kMaxWaves][2];   // per row block: wave * 2 + slot of its (one or two) owners, 255 = none
  bool rows_at_once;         // few rows and no request longer than their logits' place in registers: one kernel (score_rows_kernel)
  int once_keys;             // requests of up to this many keys take the one-pass kernel (0: none does)
  int once_short, once_long; // how many take it, of up to kOnceKeys / 2 keys and of more
  int once_rows, once_chunks;            // query rows of a chunk, chunks
  int once_group;            // chunks that one workgroup takes in turn
  int mass_parts;            // arrays of raw attention mass that add up: row splits, or chunks where every request takes one pass
  TeamSchedule team;         // all requests in one pass by teams of workgroups, where they would take two passes otherwise
  int grid_override;         // > 0: the caller fixed the number of workgroups of the score passes
  int lead_tiles;            // empty positions before each request's tiles in the sequence below: the cost of starting a segment
  int tiles_per_problem;     // sum over requests of (lead_tiles + ceil(N_r / kTileKeys)): positions of one (layer, head)
  int total_tiles;           // L * Hkv * tiles_per_problem, shared out evenly over the teams of row_splits workgroups
  int real_tiles;            // the same without the leads
  int64_t q_sl, q_ss, q_sh, q_st;
  int64_t kv_sl, kv_sh, kv_st;
  int64_t o_sl, o_sh, o_st;
  const int32_t* cu_seqlens_dev;
  const int32_t* cu_budgets_dev;
  // workspace layout (byte offsets, each 256-byte aligned)
  size_t off_stats, off_lse, off_uraw, off_member, off_member_count, ws_bytes;
  // selection by parts (a request beyond kSelectMaxCandidates; else 0 parts: one workgroup per request does it all)
  int sel_parts;             // sum over requests of max(1, ceil((N_r - W) / kPartChunk))
  size_t off_part_hist, off_part_sure, off_part_head, off_part_before;
};

// Spreads `row_blocks` blocks over the waves of a workgroup (fills waves, wave_desc, rb_holder).
void assign_row_blocks(Plan* plan);

// Validates `p` and fills `plan`.  Returns 0 or a CODECOMP_E* code.  Host only, no HIP calls.
int make_plan(const codecomp_params* p, Plan* plan);

// Tail of the score step: pooling and the prior.
struct FinishArgs {
  const float* uraw;
  const float* prior;
  const int32_t* cu_seqlens;
  float* scores;
  int n_seqs, T, LH, row_splits, pool;
  int mass_trim;      // window positions at the end of every request that hold no attention mass (prefix-only softmax)
  int pool_trim;      // window positions at the end of every request that pooling leaves out (prefix-only pooling)
  int pool_max;       // 1: max pooling
  float lambda, inv_pool;
};
FinishArgs finish_args(const Plan& pl, const float* prior, float* scores, void* workspace);

int launch_score(const Plan& pl, const void* q, const void* k, const float* prior, float* scores,
                 void* workspace, hipStream_t stream, unsigned stages = CODECOMP_STAGE_ALL);
int launch_select(const Plan& pl, const float* scores, int32_t* idx, void* workspace, hipStream_t stream);
int launch_select_two_stage(const Plan& pl, const float* scores, const float* prior, int32_t* idx, void* workspace,
                            hipStream_t stream);
// Score, select and gather in one go: the enqueue order behind codecomp_compress.
int launch_compress(const Plan& pl, const void* q, const void* k, const void* v, const float* prior, float* scores, int32_t* idx,
                    void* k_out, void* v_out, void* workspace, hipStream_t stream);
// Pooling, prior and selection of requests that one workgroup each can take (fused_tail says whether these parameters can).
bool fused_tail(const Plan& pl);
bool fused_copy(const Plan& pl);          // whether it copies the kept rows, too
int launch_finish_select(const Plan& pl, const float* prior, float* scores, int32_t* idx, const void* k, const void* v, void* k_out,
                         void* v_out, void* workspace, hipStream_t stream);
int launch_gather(const Plan& pl, const void* k, const void* v, const int32_t* idx, void* k_out, void* v_out,
                  hipStream_t stream);

}  // namespace codecomp
