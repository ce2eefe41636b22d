// Internal header: the score step of long requests in one pass over their logits, by teams of workgroups.
//
// The two passes of score_pass.h form every logit twice because a column of probabilities needs the normalisers of its rows, and
// those need all keys.  Here the workgroups that hold a request's keys between them (a team: 512 keys to each, in registers as
// MFMA fragments) take the query rows in step: each forms the logits and exponentials of 32 rows and its own keys, stores the 32
// sums over its keys to memory, goes on with the next rows, and some rows later adds up the sums of the whole team, which turn the
// exponentials, still in registers, into probabilities.  Every logit is formed once, every exponential taken once.
//
// Waiting for one another needs all workgroups of the launch on the device at once, which no launch promises: other streams and
// processes may hold compute units.  So every wait is bounded.  If a sum does not arrive in time, or a logit outruns its row's reference
// (the row's largest logit among 16 of its keys) by 69 nats, a word in the workspace says so (workgroups that see that a sum was missing
// leave at their start or with their problem), and the launch behind this one
// (score_team_again_kernel, which otherwise ends at once) does the same work, or that of the problems concerned, with the same
// arithmetic, bit for bit, without any wait for a workgroup that might not run: it hands out its tasks in an order in which a task
// only waits for tasks handed out before it.
//
// What bounds it: instructions issued.  Two waves on a SIMD take 32 rows and their 64 keys each in 1.25 .. 1.3 us (32 MFMAs, 32
// exponentials, and 32 each of scaling, summing and weighing to a wave, and 60 for everything else: the VALU is busy 55 % of the time, the
// matrix cores 28 %); the two passes take 1.85 us for the same.  Why this split: the sums of a pair of row blocks need 1.4 (32
// members) .. 1.7 us (256) from the first store to the last load, so the exponentials of three pairs wait in registers: 96 of them, beside
// 64 of keys, which leaves 4 tiles of 16 keys to a wave and one workgroup to a compute unit.  A round costs 5 us beyond its pairs (the two
// passes: 4.5): half of it while the next problem's keys are on their way to LDS, the rest where all waves take them up at once.
// Workgroups wait for counts in LDS, not at barriers: with a barrier in each block the slowest wave of every block was waited for.
// Measured, scores of 28 layers, 4 KV heads of 7 query heads, window 64, 32K keys: two passes 890 us, teams 686; window 128 1646 and 1229;
// 8-bit keys 826 and 681.  Error against 64 bits 7e-8 (2-norm), by two passes 3.4e-7.
#pragma once
#include "score_once.h"
#include "team_tasks.h"

namespace codecomp {

constexpr uint32_t kTeamEmpty = 0xFFFFFFFFu;       // a sum that is not there yet; sums are stored without their sign bit
constexpr int kTeamRing = 16;                      // pairs of row blocks whose sums have a place

enum { kTeamAbsent = 0, kTeamRange = 1, kTeamTicket = 32 };        // control words: a wait has failed; rows of some problems are out of range; tasks handed out
constexpr uint32_t kTeamOut = 1;                   // flag of a problem: the team kernel found rows out of range
constexpr uint32_t kTeamFine = 1, kTeamRedo = 2;   // its weights are there; it has rows out of range (found again)
// Words of a problem in score_team_again_kernel: tasks of a phase that are done, what is there; last, kTeamOut.
enum { kTeamSumsDone, kTeamWeighed, kTeamLargestDone, kTeamReferred, kTeamSumsAgainDone, kTeamWeighedAgain, kTeamMassesDone, kTeamFlags };

__device__ __forceinline__ uint32_t team_load(const uint32_t* p) { return __hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT); }
__device__ __forceinline__ void team_store(uint32_t* p, uint32_t v) { __hip_atomic_store(p, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT); }

struct TeamArgs {
  uint32_t* lines;             // [place of a pair of row blocks][member][32]: row sums over the member's keys
  uint32_t* ctl;
  uint32_t* done;              // [problem][kTeamCounters]; counters by position among the problems that are done, flags by problem
  int problems, slots, most;   // problems; how many of them have a place for their sums at a time there; members of the largest team
  int pairs;                   // of row blocks in a problem
  int members, ring, line_pairs, steps;
  int apart;                   // 1: kTeamAbsent is set from the start, so that score_team_again_kernel does it all
  uint32_t step[kTeamSteps + 1];
  uint32_t entry[kTeamEntries][2];
};
// Longest wait for a sum, in 10 ns.  Members that run answer within some us; what this bounds is the time lost where some do not.  A round of
// the most rows takes 48 us: a call that starts beside the last round of another one still waits for its compute units.
constexpr int64_t kTeamWait = 5000;

// One member's part of one problem.
struct TeamTask {
  int lz, seq, tok0, n;        // problem, its first token and its keys
  int first, chunks;           // place of the team's first member among the workgroups, members
  int tile0, tiles;            // this member's tiles of 16 keys
  int valid;
};
// ... and where its rows, references and masses lie.
struct TeamRows { const char* q; const float* ref; };
template <class Args>
__device__ __forceinline__ TeamRows team_rows(Args x, const TeamTask& t) {
  const int layer = divide(t.lz, x->a.Hkv, x->a.inv_heads), head = t.lz - layer * x->a.Hkv;
  return {reinterpret_cast<const char*>(x->a.q + (int64_t)layer * x->a.q_sl + (int64_t)t.seq * x->a.q_ss + (int64_t)(head * x->a.G) * x->a.q_sh),
          x->a.lse + ((int64_t)t.lz * x->a.n_seqs + t.seq) * x->a.lrows};
}

template <int D, int NT, bool K8, int ML>
struct Team {
  static_assert(D == 128, "what lies in LDS, and the order of MFMAs and exponentials, are laid out for head_dim 128");
  static constexpr int KS = D / 32;                    // MFMA k-steps
  static constexpr int NW = 8;
  static constexpr int DB = 6;                         // blocks of 16 rows whose exponentials are kept: what the registers hold
  static constexpr int LAG = DB / 2;                   // ... pairs
  static constexpr int PER = KS / (K8 ? 2 : 1);        // 16-byte pieces per lane of a tile of keys
  static constexpr int KP = NT * PER;                  // ... of a wave's keys
  // Pieces of the next problem's keys that find no room in LDS beside the rest.  They are loaded when the problem begins.
  static constexpr int DIRECT = K8 ? 0 : 2;
  static_assert(kTeamRing >= DB + 2, "a place is used again only when all have read it");
  struct Shared {
    u32x4 q[3][2][KS][64];       // query rows of three pairs of blocks, fragment order
    uint32_t poll[ML][32];       // row sums of the members, a share of the members to each wave
    float sums[NW][32];          // row sums of the waves over their own keys
    float team[LAG][NW][32];     // row sums of the team, each wave its share
    float ref[3][32];            // references of the rows of three pairs
    uint16_t row[kTeamRows + 64];          // where the query rows begin, in pieces of 16 bytes
    uint32_t summed[NW], ready[NW];        // pairs whose row sums a wave has left; ... whose team sums, and next query rows
    uint32_t quit, absent;       // a wave has waited in vain; control word kTeamAbsent, as seen last
    u32x4 k[NW][KP - DIRECT][64];          // the next problem's keys, 64 bytes of 16 keys a piece; last, the others are reached by offsets
  };
  static_assert(sizeof(Shared) <= 160 * 1024, "local memory");
};

template <class T>
__device__ __forceinline__ uint32_t lds_address(T* p) { return (uint32_t)(uintptr_t)(__attribute__((address_space(3))) void*)p; }

// Walks through the rounds of the plan: the tasks of workgroup `wg`, one a round.
struct TeamWalk {
  int step, round, rounds, stride;
  TeamTask t;
  template <class Args>
  __device__ __forceinline__ void find(Args x, int wg) {
    t.valid = 0;
    if (step >= x->t.steps) return;
    const uint32_t s = x->t.step[step];
    rounds = (int)(s & 0xFFFFu);
    int at = 0;
    for (int e = (int)(s >> 16); e < (int)(x->t.step[step + 1] >> 16); ++e) {
      const uint32_t kind = x->t.entry[e][0], size = x->t.entry[e][1];
      const int teams = (int)(kind >> 16), chunks = (int)(size >> 16);
      if (wg < at + teams * chunks) {
        const int team = (wg - at) / chunks;
        t.valid = 1;
        t.seq = (int)(kind & 0xFFFFu);
        t.chunks = chunks;
        t.first = at + team * chunks;
        t.lz = (int)(size & 0xFFFFu) + team;
        stride = teams;
        t.tok0 = x->a.cu_seqlens[t.seq];
        t.n = x->a.cu_seqlens[t.seq + 1] - t.tok0 - x->a.key_trim;
        const int all = (t.n + 15) >> 4, each = all / chunks, more = all - each * chunks, m = wg - t.first;
        t.tile0 = m * each + min(m, more);
        t.tiles = each + (m < more ? 1 : 0);
        return;
      }
      at += teams * chunks;
    }
  }
  template <class Args>
  __device__ __forceinline__ void start(Args x, int wg) {
    step = 0; round = 0; stride = 0;
    find(x, wg);
  }
  template <class Args>
  __device__ __forceinline__ void next(Args x, int wg) {
    if (!t.valid) return;
    if (++round < rounds) { t.lz += stride; return; }
    round = 0; ++step;
    find(x, wg);
  }
};

// What a wave holds of a task's keys: NT or NT - 1 tiles, one more to the last waves, so that only a wave's last tile can hold
// places without a key.
struct TeamShare { int key0, tiles; };
__device__ __forceinline__ TeamShare team_share(const TeamTask& t, int wave) {
  const int base = t.tiles >> 3, extra = t.tiles & 7;
  return {(t.tile0 + wave * base + max(0, wave - (8 - extra))) * 16, base + (wave >= 8 - extra ? 1 : 0)};
}

struct TeamKernelArgs { ScoreArgs a; TeamArgs t; };
// The arguments read anew, for code that few blocks come past: kept in registers they would cost the loop its own.
typedef const __attribute__((address_space(4))) TeamKernelArgs* team_args_t;
__device__ __forceinline__ team_args_t team_args() {
  team_args_t p = (team_args_t)__builtin_amdgcn_kernarg_segment_ptr();
  asm volatile("" : "+s"(p));
  return p;
}

// Halves of two registers exchanged: {own lower, other's lower}, {own upper, other's upper} (32 lanes, or every 16).
__device__ __forceinline__ void swap_halves(float x, float y, float& a, float& b) {
  const auto r = __builtin_amdgcn_permlane32_swap(__builtin_bit_cast(uint32_t, x), __builtin_bit_cast(uint32_t, y), false, false);
  a = __builtin_bit_cast(float, (uint32_t)r[0]); b = __builtin_bit_cast(float, (uint32_t)r[1]);
}
__device__ __forceinline__ void swap_rows(float x, float y, float& a, float& b) {
  const auto r = __builtin_amdgcn_permlane16_swap(__builtin_bit_cast(uint32_t, x), __builtin_bit_cast(uint32_t, y), false, false);
  a = __builtin_bit_cast(float, (uint32_t)r[0]); b = __builtin_bit_cast(float, (uint32_t)r[1]);
}

template <int D, int NT, bool K8, int ML>
__global__ __launch_bounds__(512, 2) void score_team_kernel(TeamKernelArgs args) {
  using O = Team<D, NT, K8, ML>;
  constexpr int KS = O::KS, NW = O::NW, DB = O::DB, LAG = O::LAG, PER = O::PER, ESZ = K8 ? 1 : 2;
  static_assert(LAG == 3, "the slots of query rows are counted along with the sets of exponentials");
  constexpr int STAGED = O::KP - O::DIRECT;
  constexpr int TC = 1;                                // tile of the odd block before which the team's sums are collected
  constexpr int TP = 1;                                // tile of the even block before which one wave reads the sums of all
  constexpr int LINE = 128;                            // bytes of a member's 32 sums
  __shared__ __attribute__((aligned(16))) typename O::Shared sh;
  const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int l16 = lane & 15, grp = lane >> 4, l32 = lane & 31, hf = lane >> 5;
  const float c = args.a.c;
  const int pairs = args.t.pairs;                      // of row blocks, per problem
  const int pair_bytes = args.t.members * LINE;
  // neighbours in a team share a die: workgroup b runs on die b % 8 (a multiple of 8 workgroups)
  const int wg = ((int)blockIdx.x & 7) * (args.t.members >> 3) + ((int)blockIdx.x >> 3);

  TeamWalk walk;
  walk.start(team_args(), wg);
  TeamTask cur = walk.t;
  if (!cur.valid) return;
  walk.next(team_args(), wg);
  const TeamTask& nxt = walk.t;                        // the one after

  // ---- loads that go straight into LDS: keys, query rows, references, sums.  They are counted by hand.
  const uint32_t k_to = lds_address(&sh.k[wave][0][0]);
  struct Keys { const unsigned char* from; int key0, last; } keys;     // of the problem whose keys are sent for
  auto keys_of = [&](const TeamTask& t) __attribute__((always_inline)) {
    const team_args_t x = team_args();
    const int layer = divide(t.lz, x->a.Hkv, x->a.inv_heads), head = t.lz - layer * x->a.Hkv;
    return Keys{x->a.k + ((int64_t)layer * x->a.kv_sl + (int64_t)head * x->a.kv_sh + (int64_t)t.tok0 * x->a.kv_st) * ESZ, team_share(t, wave).key0, t.n - 1};
  };
  const uint32_t key_bytes = (uint32_t)args.a.kv_st * ESZ;
  // Pieces are sent for two by two: they share the lane's offset.
  constexpr int UNIT = 2, UNITS = STAGED / UNIT;
  auto key_at = [&](int i) __attribute__((always_inline)) {            // of piece i, less what is the same in all lanes
    const uint32_t key = (uint32_t)min(keys.key0 + i / PER * 16 + l16, keys.last);
    return key * key_bytes + (uint32_t)(grp * 16);
  };
  auto stage = [&](int u) __attribute__((always_inline)) {             // unit u of this wave's keys
    // A unit is a cache line of each key, so that the pairs ask alike of memory (with a half of both lines at a time, every second pair
    // asked for everything: 8 x 64K keys, 256 rows 562 us, now 537); but of a tile that is not all in LDS the first half of both lines is
    // there, and what is loaded when the problem begins is found in the cache.
    const int i = u * UNIT;
    const bool parted = PER == 4 && STAGED % PER != 0 && i >= STAGED / PER * PER;
    const int apart = parted ? 128 : 64;
    const unsigned char* from = keys.from + (PER == 4 ? (u & 1) * (parted ? 64 : 128) : 0);
    const uint32_t at = key_at(i), to = k_to + (uint32_t)i * 1024u;
    asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %1, %2" ::"s"(to), "v"(at), "s"(from) : "memory", "m0");
    asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %1, %2" ::"s"(to + 1024u), "v"(at), "s"(from + apart) : "memory", "m0");
  };
  const uint32_t q_to = lds_address(&sh.q[0][0][0][0]) + (uint32_t)wave * 1024u;
  const uint32_t ref_to = lds_address(&sh.ref[0][0]);
  const int row_in = (wave / KS) * 16 + l16;           // this lane's row of a pair and piece of it
  const uint32_t piece_at = (uint32_t)((wave % KS) * 64 + grp * 16);
  TeamRows rows = team_rows(team_args(), cur);         // of the problem whose rows are sent for
  auto fetch = [&](uint32_t row_at, int pair, uint32_t slot) __attribute__((always_inline)) {
    if (wave == 7)                                     // first, so that the wait below counts no more for this wave than for the others
      asm volatile("s_mov_b32 m0, %0\n\ts_bfm_b64 exec, 32, 0\n\tglobal_load_lds_dword %1, %2\n\ts_mov_b64 exec, -1"
                   ::"s"(ref_to + slot * 128u), "v"(lane * 4), "s"(rows.ref + pair * 32) : "memory", "m0");
    asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %1, %2" ::"s"(q_to + slot * (2 * KS * 1024u)), "v"(row_at), "s"(rows.q) : "memory", "m0");
  };

  for (int r = tid; r < pairs * 32; r += 512) {        // rows past the end read the first one
    const int row = r < args.a.R ? r : 0, g = row_group(row, args.a.inv_w);
    sh.row[r] = (uint16_t)((uint32_t)g * ((uint32_t)args.a.q_sh / 8) + (uint32_t)(row - g * args.a.W) * ((uint32_t)args.a.q_st / 8));
  }
  if (tid < 8) sh.summed[tid] = sh.ready[tid] = 0;
  if (tid == 0) sh.quit = 0;
  // Where a wait has failed, the work so far counts for nothing, and who goes on only keeps the kernel behind from its own: workgroups that
  // start then leave at once, the others when their problem is through.
  auto look_for_absent = [&]() __attribute__((always_inline)) {
    if (wave == 0)
      asm volatile("s_mov_b32 m0, %0\n\ts_mov_b64 exec, 1\n\tglobal_load_lds_dword %1, %2 sc1\n\ts_mov_b64 exec, -1"
                   ::"s"(lds_address(&sh.absent)), "v"(0), "s"(team_args()->t.ctl + kTeamAbsent) : "memory", "m0");
  };
  for (int i = tid; i < ML * 32; i += 512) (&sh.poll[0][0])[i] = 0;
  asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory");
  keys = keys_of(cur);
  uint32_t row_at = sh.row[row_in] * 16u + piece_at;         // this lane's piece of the pair that is sent for next
  fetch(row_at, 0, 0);
  row_at = sh.row[32 + row_in] * 16u + piece_at;
  fetch(row_at, 1, 1);
  row_at = sh.row[64 + row_in] * 16u + piece_at;
  for (int u = 0; u < UNITS; ++u) stage(u);
  look_for_absent();

  u32x4 kf[NT][KS], qf[KS];
  f32x4 e[DB][NT], mass[NT];
  const f32x4 zero = {0.f, 0.f, 0.f, 0.f};
  auto take_tile = [&](int t) __attribute__((always_inline)) {         // keys of the problem that begins: from LDS, and what is not there
#pragma unroll
    for (int ks = 0; ks < KS; ++ks) {
      if constexpr (K8) {                              // a lane's 8 codes are half a piece of its row
        const unsigned char* piece = reinterpret_cast<const unsigned char*>(&sh.k[wave][t * PER + ks / 2][0]);
        kf[t][ks] = to_bf16x8(*reinterpret_cast<const u32x2*>(piece + (((ks & 1) * 2 + (grp >> 1)) * 16 + l16) * 16 + (grp & 1) * 8));
      } else {
        const int i = t * PER + (PER == 4 && t * PER + PER > STAGED ? (ks & 1) * 2 + (ks >> 1) : ks);
        kf[t][ks] = i < STAGED ? sh.k[wave][i < STAGED ? i : 0][lane] : *reinterpret_cast<const u32x4*>(keys.from + key_at(i) + ks * 64);
        if (i >= STAGED) pin(kf[t][ks]);               // waited for here: left to its use, every pair would wait for all loads there
      }
    }
  };
  TeamShare own = team_share(cur, wave);
  f32x4 pad;                                           // added to the logits of the wave's last tile: -inf in places without a key
  auto find_pad = [&]() __attribute__((always_inline)) {
#pragma unroll
    for (int v = 0; v < 4; ++v) pad[v] = own.tiles < NT || own.key0 + (NT - 1) * 16 + 4 * grp + v >= cur.n ? -INFINITY : 0.f;
    pin(pad);
  };
  find_pad();
  asm volatile("s_waitcnt vmcnt(0)\n\ts_barrier" ::: "memory");
  typedef volatile __attribute__((address_space(3))) uint32_t* word_t;
  const word_t quit = (word_t)&sh.quit, absent = (word_t)&sh.absent;
  if (__builtin_amdgcn_readfirstlane(*absent) != 0) return;
#pragma unroll
  for (int t = 0; t < NT; ++t) take_tile(t);
  asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
#pragma unroll
  for (int s = 0; s < DB; ++s)
#pragma unroll
    for (int t = 0; t < NT; ++t) e[s][t] = zero;
#pragma unroll
  for (int t = 0; t < NT; ++t) mass[t] = zero;
#pragma unroll
  for (int ks = 0; ks < KS; ++ks) qf[ks] = sh.q[0][0][ks][lane];

  // Pair q of the run is pair q - cur_start of the current problem.  Its rows are sent for two pairs earlier; its sums go out in pair
  // q + 1; those of the team are asked for and collected in pair q + LAG - 1, at whose end its weights are there; its exponentials are
  // then added to the masses while those of pair q + LAG take their place.  What does not happen in every pair is kept by the pair in
  // which it comes next, so that a pair comes past few questions: its instructions are what the kernel's time is made of.
  const uint16_t (*row_from)[32] = reinterpret_cast<const uint16_t (*)[32]>(&sh.row[64]);
  int q = 0, cur_start = 0;
  int event = 0;                                       // pair before which something happens (the first: it is found there)
  int flush_at = LAG - 1;                              // pair at whose end masses are complete
  int last = nxt.valid ? pairs - 1 : 0x7FFFFFFF;       // last pair of the current problem, where another one follows
  int rows_at = pairs - 2;                             // pair from which on the rows sent for are the next problem's
  int fpair = 2;                                       // pair of its problem that is sent for next
  bool more = true;                                    // there is one
  keys = keys_of(nxt);
  int staged = nxt.valid ? 0 : UNITS;                  // units of the next problem's keys that are on their way: one in a pair, two where too few are left before the last
  int on_way = 0;                                      // ... sent for in this pair
  int ask_lines = 0, ask_rows = 0;                     // members whose sums are collected; rows of that pair and the later ones of its problem, 0: no such pair
  const char* ask_from = reinterpret_cast<const char*>(args.t.lines);
  int ring_at = 0x7FFFFFFF;                            // pair before which the first place comes again
  int pub_at = wave + 1;                               // pair in which this wave stores the sums of the pair before
  bool over = false;
  int done_lz = -1, done_seq = 0, done_tok0 = 0, done_n = 0, split = 0;      // the problem, and its array of masses, that is added up
  TeamShare done_share = own;
  float ref = sh.ref[0][l16], ref_odd = sh.ref[0][16 + l16], ref_prev = 0.f;       // of the blocks of the pair; of the block before
  float sum = 0.f, sum_even = 0.f;                     // row sums in this lane: of the block at hand, of the even block of the pair
  float wa = 0.f, wb = 0.f;                            // weights of the pair of blocks that is added to the masses
  uint64_t bad = 0;                                    // lanes that have seen a row out of range
  bool patient = true;                                 // false: a wait has failed, none is waited out any more

  // What the waves leave for one another in LDS: data, then the count (LDS keeps a wave's order).  The counts are read ahead of the
  // data: all there, and the data is good.
  typedef volatile __attribute__((address_space(3))) uint32_t* count_t;
  const count_t summed = (count_t)&sh.summed[0], ready = (count_t)&sh.ready[0];
  uint32_t counts;
  auto leave = [&](count_t count) __attribute__((always_inline)) {
    asm volatile("" ::: "memory");
    *count = (uint32_t)q + 1;
    asm volatile("" ::: "memory");
  };
  auto look = [&](count_t count) __attribute__((always_inline)) {
    counts = *count;
    asm volatile("" ::: "memory");
  };
  auto late = [&]() __attribute__((always_inline)) { return __builtin_expect(__ballot(counts < (uint32_t)q + 1) != 0, 0); };
  auto await = [&](count_t count) __attribute__((always_inline)) {
    asm volatile("" ::: "memory");
    while (__ballot(*count < (uint32_t)q + 1) != 0) {}
    asm volatile("" ::: "memory");
  };
  float part[NW];
  auto gather_sums = [&]() __attribute__((always_inline)) {
#pragma unroll
    for (int w = 0; w < NW; ++w) part[w] = sh.sums[w][l32];
  };
  auto added = [&]() __attribute__((always_inline)) { return ((part[0] + part[1]) + (part[2] + part[3])) + ((part[4] + part[5]) + (part[6] + part[7])); };

  auto gather_team = [&](int slot) __attribute__((always_inline)) {
#pragma unroll
    for (int w = 0; w < NW; ++w) part[w] = sh.team[slot][w][l32];
  };
  // Sums of a pair of all members: this wave's share, eight members a load; lanes of members past the end of the team load nothing,
  // their places hold 0.
  constexpr int PL = ML / 8;                           // members a wave looks at
  const uint32_t ask_place = (uint32_t)(wave * PL * LINE + lane * 16), poll_to = lds_address(&sh.poll[wave * PL][0]);
  uint64_t ask_lanes[PL / 8] = {};
  auto ask = [&]() __attribute__((always_inline)) {
#pragma unroll
    for (int i = 0; i < PL / 8; ++i)
      asm volatile("s_mov_b32 m0, %0\n\ts_mov_b64 exec, %3\n\tglobal_load_lds_dwordx4 %1, %2 sc1\n\ts_mov_b64 exec, -1"
                   ::"s"(poll_to + i * 1024u), "v"(ask_place), "s"(ask_from + i * 1024), "s"(ask_lanes[i]) : "memory", "m0");
  };
  // ... added up: lane = row (l32), two lanes share the members.  A sum that is not there yet is a NaN.
  auto look_at_sums = [&]() __attribute__((always_inline)) {
    const float* from = reinterpret_cast<const float*>(&sh.poll[wave * PL + hf][l32]);
    float x[PL / 2];
#pragma unroll
    for (int i = 0; i < PL / 2; ++i) x[i] = from[i * 64];
#pragma unroll
    for (int n = PL / 4; n > 0; n /= 2)
#pragma unroll
      for (int i = 0; i < n; ++i) x[i] += x[i + n];
    return x[0];
  };
  auto any_missing = [&]() __attribute__((always_inline)) {
    uint32_t worst = 0;
    const uint32_t* from = &sh.poll[wave * PL + hf][l32];
#pragma unroll 1
    for (int i = 0; i < PL / 2; ++i) worst = max(worst, from[i * 64]);
    return __ballot(worst == kTeamEmpty) != 0;
  };
  auto collect = [&](int slot) __attribute__((always_inline)) {
    float got = look_at_sums();
    if (__builtin_expect(__ballot(!(got == got)) != 0, 0)) {
      const int64_t t0 = wall_clock64();
      while (any_missing()) {
        if (!patient || wall_clock64() - t0 > kTeamWait) {
          patient = false;
          if (lane == 0 && *quit == 0) {               // one wave says so: stores to one word take their turns, 10 .. 20 ns each
            team_store(team_args()->t.ctl + kTeamAbsent, 1);
            *quit = 1;
          }
          break;
        }
        ask();
        asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
      }
      got = look_at_sums();
    }
    float lo, hi;
    swap_halves(got, got, lo, hi);
    sh.team[slot][wave][l32] = lo + hi;               // two lanes the same to the same place
  };
  auto weigh = [&]() __attribute__((always_inline)) {
    const float total = added();
    const bool there = l32 < ask_rows;
    bad |= __ballot(!(total <= 1.0e30f));              // a logit outran the reference by 69 nats, or is NaN
    const float r0 = __builtin_amdgcn_rcpf(total);
    const float w = there ? __builtin_fmaf(__builtin_fmaf(-total, r0, 1.0f), r0, r0) : 0.f;
    swap_rows(w, w, wa, wb);                           // rows 0 .. 15 to all lane groups, rows 16 .. 31
  };
  // the row sums of pair q - 1 over this workgroup's keys, one wave for all: two stores always (the wait for this wave's loads counts
  // them), the sums, and the place of an earlier pair is empty again
  auto publish = [&]() __attribute__((always_inline)) {
    const team_args_t x = team_args();
    const int y = q - 1;
    const bool ring = x->t.ring != 0, again = ring && y >= DB;
    const int at = ring ? y & (kTeamRing - 1) : y, old = again ? (y - DB) & (kTeamRing - 1) : at;
    const uint32_t bits = __builtin_bit_cast(uint32_t, added()) & 0x7FFFFFFFu;
    char* line = reinterpret_cast<char*>(x->t.lines) + wg * LINE;
    // both halves of the wave hold the sums: the same to the same place
    team_store(reinterpret_cast<uint32_t*>(line + (int64_t)at * pair_bytes) + l32, bits);
    team_store(reinterpret_cast<uint32_t*>(line + (int64_t)old * pair_bytes) + l32, again ? kTeamEmpty : bits);
  };
  auto flush = [&]() __attribute__((always_inline)) {
    const team_args_t x = team_args();
    float* u = x->a.uraw + ((int64_t)split * x->a.LH + done_lz) * x->a.T + done_tok0;
    const float inv_g = x->a.inv_g;
    float mine = 0.f;                                  // a lane's key: tile l16 / 4, key l16 % 4 of its lane group
#pragma unroll
    for (int i = 0; i < NT; ++i) {
      const float m = mass_of_rows(mass[i], l16);
      mine = (l16 >> 2) == i ? m : mine;
      mass[i] = zero;
    }
    const int key = done_share.key0 + (l16 >> 2) * 16 + 4 * grp + (l16 & 3);
    if (done_lz >= 0 && (l16 >> 2) < done_share.tiles && key < done_n) u[key] = mine * inv_g;
    const bool end = q == cur_start + LAG - 1;         // all of the problem before, else one array of this one
    ++split;
    if (end) { done_lz = cur.lz; done_seq = cur.seq; done_tok0 = cur.tok0; done_n = cur.n; done_share = own; split = 0; over = !cur.valid; if (over) event = q + 1; }
    flush_at = cur_start + pairs + LAG - 1;
    if (x->a.row_splits > 1) flush_at = min(flush_at, q + x->a.nb);
  };

  auto block = [&](auto set, auto odd_c) __attribute__((always_inline)) {
    constexpr int SET = decltype(set)::value, BEFORE = (SET + DB - 1) % DB, NEXT = (SET + 1) % DB;
    constexpr int SLOT = SET / 2, SLOT_NEXT = (SET / 2 + 1) % LAG;
    constexpr bool ODD = decltype(odd_c)::value;
    const float w_now = ODD ? wb : wa;
    float r_a = 0.f, r_b = 0.f;
    const bool publisher = q == pub_at;
    auto take_next = [&]() __attribute__((always_inline)) {            // sums of the team, references of the next pair
      gather_team(SET / 2);
      r_a = sh.ref[SLOT_NEXT][l16]; r_b = sh.ref[SLOT_NEXT][16 + l16];
    };
    if constexpr (!ODD) {
      ask();
      fetch(row_at, fpair, (uint32_t)((SET / 2 + 2) % LAG));
      on_way = 0;
      if (staged < UNITS) {
        stage(staged++);
        on_way = UNIT;
        if (UNITS - staged > cur_start + pairs - 2 - q) { stage(staged++); on_way = 2 * UNIT; }
      }
    }
#pragma unroll
    for (int t = 0; t < NT; ++t) {
      if constexpr (ODD) {
        if (t == TC) {
          // the next pair's query rows and the sums asked for; the rows and keys sent for since, and the stores, may be on their way
          static_assert(UNIT <= 2, "waits");
          if (on_way == 0) {
            if (publisher) asm volatile("s_waitcnt vmcnt(3)" ::: "memory");
            else asm volatile("s_waitcnt vmcnt(1)" ::: "memory");
          } else if (on_way == UNIT) {
            if (publisher) asm volatile("s_waitcnt vmcnt(%0)" ::"i"(3 + UNIT) : "memory");
            else asm volatile("s_waitcnt vmcnt(%0)" ::"i"(1 + UNIT) : "memory");
          } else {
            if (publisher) asm volatile("s_waitcnt vmcnt(%0)" ::"i"(3 + 2 * UNIT) : "memory");
            else asm volatile("s_waitcnt vmcnt(%0)" ::"i"(1 + 2 * UNIT) : "memory");
          }
          collect(SET / 2);
          leave(ready + wave);
        }
        if (t == NT - 1) { look(ready + (lane & 7)); take_next(); }
      } else {
        if (t == TP && publisher) { look(summed + (lane & 7)); gather_sums(); }
        if (t == TP + 1 && publisher) {
          if (late()) { await(summed + (lane & 7)); gather_sums(); }
          publish();
        }
      }
      __builtin_amdgcn_sched_barrier(0);
      f32x4& prevl = t > 0 ? e[SET][t - 1] : e[BEFORE][NT - 1];
      const float rf = t > 0 ? (ODD ? ref_odd : ref) : ref_prev;
      f32x4 s = t == NT - 1 ? pad : zero;
#pragma unroll
      for (int ks = 0; ks < KS; ++ks) {
        s = once_mma(kf[t][ks], qf[ks], s);
        if (t == NT - 1) qf[ks] = ODD ? sh.q[SLOT_NEXT][0][ks][lane] : sh.q[SLOT][1][ks][lane];
      }
      if (t < NT - 1) {
#pragma unroll
        for (int v = 0; v < 4; ++v) mass[t + 1][v] = __builtin_fmaf(e[SET][t + 1][v], w_now, mass[t + 1][v]);
        pin(mass[t + 1]);
      }
#pragma unroll
      for (int v = 0; v < 4; ++v) {
        const float x = __builtin_amdgcn_exp2f(__builtin_fmaf(prevl[v], c, -rf));
        prevl[v] = x;
        if (t == 1 && v == 0) sum = x; else sum += x;
      }
      pin(prevl); pin(sum);
      e[SET][t] = s;
      if (t == 0) {
        if constexpr (ODD) {
          sum_even = sum;
        } else {
          float x, y, lo, hi;                          // sum_even: even block, sum: odd block; lanes below 32 take the even one
          swap_halves(sum_even, sum, x, y);
          swap_rows(x + y, x + y, lo, hi);
          sh.sums[wave][(hf << 4) + l16] = lo + hi;    // two lanes the same to the same place
          leave(summed + wave);
        }
      }
      if (t > 0) {
        // one MFMA at a time: the masses (nothing to wait for) beside the first, the exponentials beside the others
#pragma unroll
        for (int m = 0; m < KS; ++m) {
          __builtin_amdgcn_sched_group_barrier(0x008, 1, 0);
          if (t == NT - 1) __builtin_amdgcn_sched_group_barrier(0x100, 1, 0);
          if (m == 0) {
            if (t < NT - 1) __builtin_amdgcn_sched_group_barrier(0x002, 4, 0);
            continue;
          }
#pragma unroll
          for (int x = 0; x < (m == 1 ? 2 : 1); ++x) {
            __builtin_amdgcn_sched_group_barrier(0x002, 1, 0);
            __builtin_amdgcn_sched_group_barrier(0x400, 1, 0);
            if (m > 1 || x > 0) __builtin_amdgcn_sched_group_barrier(0x002, 1, 0);
          }
        }
        __builtin_amdgcn_sched_group_barrier(0x002, 1, 0);
        __builtin_amdgcn_sched_barrier(0);
      }
      if (t == NT - 1) {
        if constexpr (ODD) {
          if (late()) {                                // read again what was read too early
            await(ready + (lane & 7));
            take_next();
#pragma unroll
            for (int ks = 0; ks < KS; ++ks) qf[ks] = sh.q[SLOT_NEXT][0][ks][lane];
          }
          if (__builtin_expect(q == last, 0)) {        // the keys have done their part, the next problem's come
#pragma unroll
            for (int i = 0; i < NT; ++i) take_tile(i);
          }
          weigh();
          if (publisher) pub_at += 8;
          if (__builtin_expect(q == flush_at, 0)) flush();
        }
        const float w_next = ODD ? wa : wb;
#pragma unroll
        for (int v = 0; v < 4; ++v) mass[0][v] = __builtin_fmaf(e[NEXT][0][v], w_next, mass[0][v]);
        pin(mass[0]);
      }
    }
    if constexpr (ODD) { ref_prev = ref_odd; ref = r_a; ref_odd = r_b; }
    else ref_prev = ref;
  };

  // what happens before pair q
  auto turn = [&]() __attribute__((always_inline)) {
    if (over) return;
    if (q == cur_start + pairs && cur.valid) {         // the next problem, or none: then only the waiting exponentials are left
      if (__builtin_amdgcn_readfirstlane(*quit | *absent) != 0) {
        summed[wave] = ready[wave] = 0x7FFFFFFF;      // no wave waits for this one any more
        over = true;
        return;
      }
      cur = nxt;
      cur_start = q;
      if (cur.valid) {
        own = team_share(cur, wave);
        find_pad();
        walk.next(team_args(), wg);
        keys = keys_of(nxt);
        staged = nxt.valid ? 0 : UNITS;
        last = nxt.valid ? q + pairs - 1 : 0x7FFFFFFF;
        asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");     // the keys have left LDS
      } else {
        // the last sums go out in this pair, none after it
        if (pub_at > q) pub_at = 0x7FFFFFFF;
      }
    }
    if (q == rows_at && more) {                        // the rows sent for are the next problem's
      more = nxt.valid != 0;
      look_for_absent();                               // there when this pair's sums are, and looked at where the next problem begins
      if (more) rows = team_rows(team_args(), nxt);    // else: what is sent for, to keep the count, is not used
      fpair = 0;
      row_from = reinterpret_cast<const uint16_t (*)[32]>(&sh.row[0]);
      row_at = (*row_from)[row_in] * 16u + piece_at;
    }
    if (q == cur_start + LAG - 1) {                    // the pair whose sums are collected is the current problem's first
      const team_args_t x = team_args();
      // The problem before has rows out of range.  All waves of its team know; one says so (all of them, 512 stores to a word in every
      // problem, took the kernel from 0.75 to 2.1 ms where each of 112 problems of 32K keys had such rows).
      if (bad != 0 && lane == 0 && done_share.key0 == 0) {
        team_store(x->t.done + (int64_t)(done_seq * x->a.LH + done_lz) * kTeamCounters + kTeamFlags, kTeamOut);
        team_store(x->t.ctl + kTeamRange, 1);
      }
      bad = 0;
      const int lines_now = cur.valid ? cur.chunks : 0, p = q - LAG + 1, at = x->t.ring ? p & (kTeamRing - 1) : p;
      if (lines_now != ask_lines) {
        ask_lines = lines_now;
#pragma unroll
        for (int i = 0; i < PL / 8; ++i) {
          const int left = min(max(lines_now - wave * PL - i * 8, 0), 8);
          ask_lanes[i] = left == 8 ? ~0ull : (1ull << (left * 8)) - 1;
          *reinterpret_cast<u32x4*>(&sh.poll[wave * PL + i * 8][lane * 4]) = u32x4{0, 0, 0, 0};
        }
        asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
      }
      ask_rows = cur.valid ? x->a.R : 0;
      ask_from = reinterpret_cast<const char*>(x->t.lines) + (int64_t)at * pair_bytes + cur.first * LINE;
      ring_at = x->t.ring ? q + kTeamRing - at : 0x7FFFFFFF;
    }
    if (q == ring_at) {
      ask_from -= kTeamRing * (int64_t)pair_bytes;
      ring_at += kTeamRing;
    }
    // the next one
    event = 0x7FFFFFFF;
    auto soon = [&](int at) __attribute__((always_inline)) { if (at > q && at < event) event = at; };
    if (q >= cur_start && q == rows_at) rows_at = more ? cur_start + 2 * pairs - 2 : rows_at;
    soon(cur_start + pairs); soon(cur_start + LAG - 1); soon(rows_at); soon(ring_at);
  };

  auto pair = [&](auto s) __attribute__((always_inline)) {
    constexpr int S = decltype(s)::value;
    if (__builtin_expect(q == event, 0)) {
      turn();
      if (over) return false;
    }
    block(std::integral_constant<int, 2 * S>{}, std::false_type{});
    block(std::integral_constant<int, 2 * S + 1>{}, std::true_type{});
    ++q;
    ask_rows -= 32;
    ask_from += pair_bytes;
    ++fpair;
    ++row_from;
    row_at = (*row_from)[row_in] * 16u + piece_at;
    return true;
  };
  for (;;) {
    if (!pair(std::integral_constant<int, 0>{})) break;
    if (!pair(std::integral_constant<int, 1>{})) break;
    if (!pair(std::integral_constant<int, 2>{})) break;
  }
  asm volatile("s_waitcnt vmcnt(0)" ::: "memory");     // no load into LDS outlives the run
}

// Does the team kernel's work again where that could not be finished: the same sums in the same order, so the same bits, but without
// waiting for a workgroup that might not run.  Its tasks (team_tasks.h) are handed out by a counter; a task waits only for tasks with
// smaller numbers, which run or are done: one number is taken ahead, so a workgroup may hold two, and does the smaller one first.
// Where no wait has failed, only the problems with rows out of range are taken.
//
// Bound by instruction issue as the passes are, in twice the work of the team kernel: every logit is formed for the row sums and again
// for the masses.  The query rows come through LDS, four blocks of 16 at a time, the next four on their way in registers; the MFMAs of
// a block stand beside the exponentials of the one before.  A task is taken by half members, so that a compute unit holds two workgroups
// of four waves, of which one works while the other waits for keys (2 us), the next number (2) and counters: a third of a task's 22 us, in
// which its loop runs 14 (28 x 32K keys, 448 rows).  Measured, scores, by two passes / by teams / all of it by this kernel: 28 x 32K keys, 448
// rows 1009 / 663 / 1104 us (with eight waves, rows from memory to registers, a fence and the totals of all members in each task 6239); 896 rows
// 1659 / 1161 / 1990; 8 x 64K, 256 rows 661 / 534 / 957; sixteen requests of 8K .. 45K 473 / 373 / 686; 4 x 20011 95 / 89 / 140.  Teams and then a
// row of every problem out of range: 28 x 32K 2390 us (9409), 4 x 20011 304 (881).  Three workgroups a compute unit spill: 1790.
template <int D, int NT, bool K8, int ML>
__global__ __launch_bounds__(256, 2) void score_team_again_kernel(TeamKernelArgs args) {
  constexpr int KS = D / 32, ESZ = K8 ? 1 : 2, PL = ML / 8, kListed = 1024, NW = 4, kAhead = NW;
  using stage_t = std::conditional_t<K8, u32x2, u32x4>;
  const ScoreArgs& a = args.a;
  const TeamArgs& ta = args.t;
  const uint32_t absent = team_load(ta.ctl + kTeamAbsent), range = team_load(ta.ctl + kTeamRange);
  bool whole = absent != 0;
  if (!whole && range == 0) return;
  struct Shared {
    u32x4 q[2][kAhead][KS][64];                        // blocks of query rows, fragment order
    float part[kTeamRows / 32 + 1][NW][32];            // row sums (largest logits) of the waves; [0]: of the rows before the first
    float weight[32 + kTeamRows], ref[32 + kTeamRows];
    uint16_t list[kListed];
    struct { TeamTaskAt at; int problem, halves; } task[2];            // the task at hand and the next one
    int listed, out, last, redo;
  };
  __shared__ __attribute__((aligned(16))) Shared sh;
  const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int l16 = lane & 15, grp = lane >> 4, l32 = lane & 31, hf = lane >> 5;
  const int pairs = ta.pairs;
  const float c = a.c;
  const f32x4 zero = {0.f, 0.f, 0.f, 0.f};
  if (tid < 32) sh.weight[tid] = sh.ref[tid] = 0.f;
  if (!whole) {                                        // the problems with rows out of range, the same list in every workgroup
    if (wave == 0) {
      int count = 0;
      for (int at = 0; at < ta.problems; at += 64 * 8) {
        uint32_t flag[8];
#pragma unroll
        for (int i = 0; i < 8; ++i) flag[i] = team_load(ta.done + (int64_t)min(at + i * 64 + lane, ta.problems - 1) * kTeamCounters + kTeamFlags);
#pragma unroll
        for (int i = 0; i < 8; ++i) {
          const int problem = at + i * 64 + lane;
          const bool mine = problem < ta.problems && (flag[i] & kTeamOut) != 0;
          const uint64_t all = __ballot(mine);
          const int to = count + __popcll(all & ((1ull << lane) - 1));
          if (mine && to < kListed) sh.list[to] = (uint16_t)problem;
          count += __popcll(all);
        }
      }
      if (lane == 0) sh.listed = count;
    }
    __syncthreads();
    whole = __builtin_amdgcn_readfirstlane(sh.listed) > kListed;
  }
  const int problems = whole ? ta.problems : __builtin_amdgcn_readfirstlane(sh.listed);
  const int most = 2 * ta.most;                        // in half members
  const TeamTasks tasks = TeamTasks::make(problems, ta.slots, most, whole, (int)gridDim.x);
  auto problem_at = [&](int i) { return whole ? i : __builtin_amdgcn_readfirstlane((int)sh.list[i]); };
  auto halves_of = [&](int problem) {
    const int seq = problem / a.LH;
    return ((a.cu_seqlens[seq + 1] - a.cu_seqlens[seq] - a.key_trim + 15) / 16 + 8 * NT - 1) / (8 * NT) * 2;
  };
  // What a task leaves and takes in memory (sums, weights, references, counters) goes past the caches; here its stores are done.
  auto stored = [&]() __attribute__((always_inline)) { asm volatile("s_waitcnt vmcnt(0)" ::: "memory"); };
  auto await = [&](const uint32_t* count, uint32_t need) {
    if (tid == 0) while (team_load(count) < need) __builtin_amdgcn_s_sleep(2);
    asm volatile("" ::: "memory");
    __syncthreads();
  };
  // the next number that stands for half a member that there is
  auto next_number = [&]() { return (int)__hip_atomic_fetch_add(ta.ctl + kTeamTicket, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT); };
  auto take_number = [&](int to, int x) {
    for (;; x = next_number()) {
      const TeamTaskAt t = tasks.at(x);
      const int problem = t.at < 0 || whole ? t.at : (int)sh.list[t.at], halves = t.at < 0 ? 0 : halves_of(problem);
      if (t.at < 0 || t.first < halves) { sh.task[to] = {t, problem, halves}; return; }
    }
  };
  if (tid == 0) take_number(0, next_number());
  __syncthreads();
  for (int turn = 0;; turn ^= 1) {
    auto uniform = [](int x) __attribute__((always_inline)) { return __builtin_amdgcn_readfirstlane(x); };
    const int at = uniform(sh.task[turn].at.at);
    if (at < 0) return;
    const int phase = uniform(sh.task[turn].at.phase), first = uniform(sh.task[turn].at.first), problem = uniform(sh.task[turn].problem);
    const int halves = uniform(sh.task[turn].halves), chunks = halves >> 1, last = min(uniform(sh.task[turn].at.last), halves);
    uint32_t* const done = ta.done + (int64_t)at * kTeamCounters;
    const int seq = problem / a.LH, lz = problem - seq * a.LH;
    const int layer = divide(lz, a.Hkv, a.inv_heads), head = lz - layer * a.Hkv;
    uint32_t* const lines = ta.lines + (int64_t)(at % ta.slots) * pairs * most * 32;               // [pair][half member][32], weights in the first one's place
    uint32_t* const refs = reinterpret_cast<uint32_t*>(a.lse) + ((int64_t)lz * a.n_seqs + seq) * a.lrows;
    const uint16_t* const qb = a.q + (int64_t)layer * a.q_sl + (int64_t)seq * a.q_ss + (int64_t)(head * a.G) * a.q_sh + grp * 8;
    TeamTask t;
    t.lz = lz; t.seq = seq; t.chunks = chunks;
    t.tok0 = a.cu_seqlens[seq]; t.n = a.cu_seqlens[seq + 1] - t.tok0 - a.key_trim;
    const unsigned char* const kb = a.k + ((int64_t)layer * a.kv_sl + (int64_t)head * a.kv_sh + (int64_t)t.tok0 * a.kv_st) * ESZ + grp * 8 * ESZ;
    bool ahead = false;                                // the next number is taken

    // One phase of half members [first, last).  ready(): waits for what the phase needs beside keys and rows.
    auto pass = [&](auto phase_c, auto ready) __attribute__((always_inline)) {
      constexpr int KIND = decltype(phase_c)::value;
      u32x4 kf[NT][KS], st[KS];
      auto fetch_keys = [&](int half) __attribute__((always_inline)) {
        const int tiles = (t.n + 15) >> 4, each = tiles / chunks, more = tiles - each * chunks, member = half >> 1;
        t.tile0 = member * each + min(member, more); t.tiles = each + (member < more ? 1 : 0);
        const TeamShare own = team_share(t, (half & 1) * NW + wave);
#pragma unroll
        for (int i = 0; i < NT; ++i) {
          const unsigned char* from = kb + (int64_t)min(own.key0 + i * 16 + l16, t.n - 1) * a.kv_st * ESZ;
#pragma unroll
          for (int ks = 0; ks < KS; ++ks) kf[i][ks] = to_bf16x8(*reinterpret_cast<const stage_t*>(from + ks * 32 * ESZ));
        }
        return own;
      };
      auto fetch_rows = [&](int chunk) __attribute__((always_inline)) {        // rows past the end are the first one
        const int row = (chunk * kAhead + wave) * 16 + l16, r = row < a.R ? row : 0, g = row_group(r, a.inv_w);
        const uint16_t* from = qb + (int64_t)g * a.q_sh + (int64_t)(r - g * a.W) * a.q_st;
#pragma unroll
        for (int ks = 0; ks < KS; ++ks) st[ks] = *reinterpret_cast<const u32x4*>(from + ks * 32);
      };
      auto leave_rows = [&](int buf) __attribute__((always_inline)) {
#pragma unroll
        for (int ks = 0; ks < KS; ++ks) sh.q[buf][wave][ks][lane] = st[ks];
      };
      int number = 0;
      if (tid == 0) number = next_number();            // ahead of the loads: who waits for it does not wait for them
      TeamShare next = fetch_keys(first);
      fetch_rows(0);
      if (tid == 0) take_number(turn ^ 1, number);
      ahead = true;
      ready();
      if constexpr (KIND != kTeamLargest)
        for (int r = tid; r < pairs * 32; r += 64 * NW) {
          sh.ref[32 + r] = __builtin_bit_cast(float, team_load(refs + (r < a.R ? r : 0)));
          if constexpr (KIND == kTeamMasses) sh.weight[32 + r] = __builtin_bit_cast(float, team_load(lines + (int64_t)(r >> 5) * most * 32 + (r & 31)));
        }
      const int chunks_of_rows = (2 * pairs + kAhead - 1) / kAhead;
#pragma unroll 1
      for (int half = first; half < last; ++half) {
        const TeamShare own = next;
        leave_rows(0);
        f32x4 pad;                                     // added to the logits of the wave's last tile: -inf in places without a key
#pragma unroll
        for (int v = 0; v < 4; ++v) pad[v] = own.tiles < NT || own.key0 + (NT - 1) * 16 + 4 * grp + v >= t.n ? -INFINITY : 0.f;
        f32x4 mass[NT], s[2][NT];
#pragma unroll
        for (int i = 0; i < NT; ++i) { mass[i] = zero; s[1][i] = f32x4{-INFINITY, -INFINITY, -INFINITY, -INFINITY}; }
        auto flush = [&](int split) __attribute__((always_inline)) {
          float* u = a.uraw + ((int64_t)split * a.LH + lz) * a.T + t.tok0;
#pragma unroll
          for (int i = 0; i < NT; ++i) {
            const float m = mass_of_rows(mass[i], l16);
            const int key = own.key0 + i * 16 + 4 * grp + (l16 & 3);
            if (l16 >> 2 == i && i < own.tiles && key < t.n) u[key] = m * a.inv_g;     // the lane counts: they differ in the order of the sum
            mass[i] = zero;
          }
        };
        float of_even = 0.f;
        // the logits of one block of rows (row: this lane's): row sums, largest logits or masses
        auto take = [&](f32x4 (&x)[NT], int row, auto odd_c) __attribute__((always_inline)) {
          constexpr bool ODD = decltype(odd_c)::value;
          float of = 0.f;
          if constexpr (KIND == kTeamLargest) {
            of = x[0][0];
#pragma unroll
            for (int i = 0; i < NT; ++i)
#pragma unroll
              for (int v = 0; v < 4; ++v) of = fmaxf(of, x[i][v]);
          } else {
            const float rf = sh.ref[32 + row], w = KIND == kTeamMasses ? sh.weight[32 + row] : 0.f;
#pragma unroll
            for (int i = 0; i < NT; ++i)
#pragma unroll
              for (int v = 0; v < 4; ++v) {
                const float e = __builtin_amdgcn_exp2f(__builtin_fmaf(x[i][v], c, -rf));
                if constexpr (KIND == kTeamMasses) mass[i][v] = __builtin_fmaf(e, w, mass[i][v]);
                else if (i == 0 && v == 0) of = e;
                else of += e;
              }
          }
          if constexpr (KIND != kTeamMasses) {
            if constexpr (!ODD) {
              of_even = of;
            } else {                                   // both blocks: lanes below 32 take the even one
              float p, q, lo, hi;
              swap_halves(of_even, of, p, q);
              if constexpr (KIND == kTeamLargest) { p = fmaxf(p, q); swap_rows(p, p, lo, hi); lo = fmaxf(lo, hi); }
              else { swap_rows(p + q, p + q, lo, hi); lo = lo + hi; }
              sh.part[1 + (row >> 5)][wave][(hf << 4) + l16] = lo;
            }
          }
        };
        u32x4 qf[KS];
        auto form = [&](f32x4 (&to)[NT], const u32x4 (*from)[64]) __attribute__((always_inline)) {       // and the rows of the next block
#pragma unroll
          for (int i = 0; i < NT; ++i) {
            to[i] = i == NT - 1 ? pad : zero;
#pragma unroll
            for (int ks = 0; ks < KS; ++ks) to[i] = once_mma(kf[i][ks], qf[ks], to[i]);
          }
#pragma unroll
          for (int ks = 0; ks < KS; ++ks) qf[ks] = from[ks][lane];
        };
#pragma unroll 1
        for (int chunk = 0; chunk < chunks_of_rows; ++chunk) {
          __syncthreads();
          const int buf = chunk & 1, p0 = chunk * (kAhead / 2), p1 = min(p0 + kAhead / 2, pairs);
          fetch_rows(chunk + 1 < chunks_of_rows ? chunk + 1 : 0);        // the last time: for the next half member
#pragma unroll
          for (int ks = 0; ks < KS; ++ks) qf[ks] = sh.q[buf][0][ks][lane];
#pragma unroll 1
          for (int p = p0; p < p1; ++p) {
            const int b = 2 * (p - p0);
            form(s[0], sh.q[buf][b + 1]);
            take(s[1], (p - 1) * 32 + 16 + l16, std::true_type{});
            if constexpr (KIND == kTeamMasses)
              if (a.row_splits > 1 && p > 0 && p % a.nb == 0) flush(p / a.nb - 1);
            form(s[1], sh.q[buf][b + 2 < kAhead ? b + 2 : 0]);     // past the last block: not used
            take(s[0], p * 32 + l16, std::false_type{});
          }
          if (chunk + 1 < chunks_of_rows) leave_rows(buf ^ 1);
        }
        if (half + 1 < last) next = fetch_keys(half + 1);
        take(s[1], (pairs - 1) * 32 + 16 + l16, std::true_type{});
        if constexpr (KIND == kTeamMasses) flush((pairs - 1) / a.nb);
        __syncthreads();
        if constexpr (KIND != kTeamMasses) {
          for (int r = tid; r < pairs * 32; r += 64 * NW) {
            const float (&part)[NW][32] = sh.part[1 + (r >> 5)];
            const int i = r & 31;
            const float x = KIND == kTeamLargest ? fmaxf(fmaxf(part[0][i], part[1][i]), fmaxf(part[2][i], part[3][i])) * c : (part[0][i] + part[1][i]) + (part[2][i] + part[3][i]);
            team_store(lines + ((int64_t)(r >> 5) * most + half) * 32 + i, __builtin_bit_cast(uint32_t, x));
          }
        }
      }
    };
    // The references of the problem's rows become their largest logits.
    auto refer = [&]() __attribute__((always_inline)) {
      for (int r = tid; r < a.R; r += 64 * NW) {
        float m = __builtin_bit_cast(float, team_load(refs + r));
#pragma unroll 8
        for (int h = 0; h < halves; ++h) m = fmaxf(m, __builtin_bit_cast(float, team_load(lines + ((int64_t)(r >> 5) * most + h) * 32 + (r & 31))));
        team_store(refs + r, __builtin_bit_cast(uint32_t, m));
      }
      stored();
      __syncthreads();
    };
    // Weights of all rows of the problem from the sums of its members, in the team kernel's order; a wave has every fourth pair.  True if a row is out of range.
    auto weigh = [&]() __attribute__((always_inline)) {
      if (tid == 0) sh.out = 0;
      __syncthreads();
      for (int p = wave; p < pairs; p += NW) {
        float total = 0.f;                             // ((0 + 1) + (2 + 3)) + ((4 + 5) + (6 + 7)) of the waves' shares
#pragma unroll 1
        for (int half = 0; half < 8; half += 4) {
          float four = 0.f;
#pragma unroll 1
          for (int w = half; w < half + 4; w += 2) {
            float two[2];
#pragma unroll
            for (int j = 0; j < 2; ++j) {
              float x[PL / 2];
#pragma unroll
              for (int i = 0; i < PL / 2; ++i) {
                const int m = (w + j) * PL + hf + 2 * i;
                const uint32_t* of = lines + ((int64_t)p * most + 2 * min(m, chunks - 1)) * 32 + l32;
                const float v = __builtin_bit_cast(float, team_load(of)) + __builtin_bit_cast(float, team_load(of + 32));
                x[i] = m < chunks ? __builtin_bit_cast(float, __builtin_bit_cast(uint32_t, v) & 0x7FFFFFFFu) : 0.f;
              }
#pragma unroll
              for (int n = PL / 4; n > 0; n /= 2)
#pragma unroll
                for (int i = 0; i < n; ++i) x[i] += x[i + n];
              float lo, hi;
              swap_halves(x[0], x[0], lo, hi);
              two[j] = lo + hi;
            }
            four += two[0] + two[1];
          }
          total += four;
        }
        const bool there = p * 32 + l32 < a.R;
        const float r0 = __builtin_amdgcn_rcpf(total);
        const float w = there ? __builtin_fmaf(__builtin_fmaf(-total, r0, 1.0f), r0, r0) : 0.f;
        team_store(lines + (int64_t)p * most * 32 + l32, __builtin_bit_cast(uint32_t, w));
        if (there && !(total <= 1.0e30f)) sh.out = 1;
      }
      stored();
      __syncthreads();
      return __builtin_amdgcn_readfirstlane(sh.out) != 0;
    };
    // Counts the task; true for who has counted the last one of the problem's.
    auto count = [&](uint32_t* of, uint32_t all) __attribute__((always_inline)) {
      stored();
      __syncthreads();
      if (tid == 0) sh.last = __hip_atomic_fetch_add(of, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) + 1 == all;
      __syncthreads();
      return __builtin_amdgcn_readfirstlane(sh.last) != 0;
    };
    // Has the problem rows out of range?  Asked once in a task: `redo` is written again only behind the barriers at its end.
    auto far_out = [&]() {
      if (!whole) return true;
      if (tid == 0) {
        uint32_t word = team_load(done + kTeamWeighed);
        while (word == 0) { __builtin_amdgcn_s_sleep(2); word = team_load(done + kTeamWeighed); }
        sh.redo = word == kTeamRedo;
      }
      asm volatile("" ::: "memory");
      __syncthreads();
      return __builtin_amdgcn_readfirstlane(sh.redo) != 0;
    };

    // the place of a problem's sums is free when the problem that had it has its masses
    auto place = [&]() { if (at >= ta.slots) await(done - (int64_t)ta.slots * kTeamCounters + kTeamMassesDone, (uint32_t)tasks.tasks_of(halves_of(problem_at(at - ta.slots)), kTeamMasses)); };
    auto leave_word = [&](uint32_t* word, uint32_t what) { if (tid == 0) team_store(word, what); };

    if (phase == kTeamSums) {
      pass(std::integral_constant<int, kTeamSums>{}, place);
      if (count(done + kTeamSumsDone, (uint32_t)tasks.tasks_of(halves, phase))) {
        leave_word(done + kTeamWeighed, weigh() ? kTeamRedo : kTeamFine);
      }
    } else if (phase == kTeamMasses) {
      pass(std::integral_constant<int, kTeamMasses>{}, [&]() {
        if (far_out()) await(done + kTeamWeighedAgain, 1);
      });
      if (at + ta.slots < problems) {                  // somebody waits for the place
        stored();
        __syncthreads();
        if (tid == 0) __hip_atomic_fetch_add(done + kTeamMassesDone, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
      }
    } else {
      if (far_out()) {
        if (phase == kTeamLargest) {
          pass(std::integral_constant<int, kTeamLargest>{}, [&]() { if (!whole) place(); });
          if (count(done + kTeamLargestDone, (uint32_t)tasks.tasks_of(halves, phase))) {
            refer();
            leave_word(done + kTeamReferred, 1);
          }
        } else {
          pass(std::integral_constant<int, kTeamSumsAgain>{}, [&]() { await(done + kTeamReferred, 1); });
          if (count(done + kTeamSumsAgainDone, (uint32_t)tasks.tasks_of(halves, phase))) {
            weigh();
            leave_word(done + kTeamWeighedAgain, 1);
          }
        }
      }
    }
    // Not only for the next task: without a barrier here, what the first thread does at the end and at the start of a turn becomes one branch,
    // and the other lanes of its wave go round without it.
    __syncthreads();
    if (!ahead && tid == 0) take_number(turn ^ 1, next_number());
    __syncthreads();
  }
}

// References of the rows (their largest logit among 16 of the request's keys, times c), and what the team kernels find empty.
template <int D, bool K8>
__global__ __launch_bounds__(256) void score_team_prepare_kernel(ScoreArgs a, TeamArgs ta) {
  constexpr int KS = D / 32, ESZ = K8 ? 1 : 2;
  using stage_t = std::conditional_t<K8, u32x2, u32x4>;
  const int tid = threadIdx.x, lane = tid & 63, l16 = lane & 15, grp = lane >> 4;
  const int64_t at = ((int64_t)blockIdx.y * gridDim.x + blockIdx.x) * 256 + tid, all = (int64_t)gridDim.x * gridDim.y * 256;
  if (at < 64) ta.ctl[at] = at == kTeamAbsent && ta.apart ? 1 : 0;
  u32x4* lines = reinterpret_cast<u32x4*>(ta.lines);
  for (int64_t i = at; i < (int64_t)ta.line_pairs * ta.members * 8; i += all) lines[i] = u32x4{kTeamEmpty, kTeamEmpty, kTeamEmpty, kTeamEmpty};
  for (int64_t i = at; i < (int64_t)ta.problems * kTeamCounters; i += all) ta.done[i] = 0;
  const int p = blockIdx.y, lz = p / a.n_seqs, seq = p - lz * a.n_seqs;
  const int tok0 = a.cu_seqlens[seq], n = a.cu_seqlens[seq + 1] - tok0 - a.key_trim;
  const int block = blockIdx.x * 4 + (tid >> 6);
  if (n <= a.once_keys || n < 16 || block * 16 >= ta.pairs * 32) return;
  const int layer = lz / a.Hkv, head = lz - layer * a.Hkv;
  const int key = l16 < 8 ? l16 : n - 16 + l16;        // the first eight and the last eight keys
  const unsigned char* kp = a.k + ((int64_t)layer * a.kv_sl + (int64_t)head * a.kv_sh + (int64_t)(tok0 + key) * a.kv_st) * ESZ + grp * 8 * ESZ;
  const int row = block * 16 + l16, r = row < a.R ? row : 0, g = row_group(r, a.inv_w);
  const uint16_t* qp = a.q + (int64_t)layer * a.q_sl + (int64_t)seq * a.q_ss + (int64_t)(head * a.G + g) * a.q_sh + (int64_t)(r - g * a.W) * a.q_st + grp * 8;
  f32x4 s = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
  for (int ks = 0; ks < KS; ++ks)
    s = once_mma(to_bf16x8(*reinterpret_cast<const stage_t*>(kp + ks * 32 * ESZ)), *reinterpret_cast<const u32x4*>(qp + ks * 32), s);
  const float m = row_max4(fmaxf(fmaxf(s[0], s[1]), fmaxf(s[2], s[3])));
  if (lane < 16) a.lse[(int64_t)p * a.lrows + row] = m * a.c;          // rows past the end: the first one's
}

// The kernel for teams of up to so many members.  8-bit keys: with places for 64 the compiler runs out of registers in the loop (20 spilled;
// 4 layers of 32K keys 129 us, with places for 128 122 us).
template <bool K8, class F>
auto with_members(int most, F f) {
  if constexpr (!K8) if (most <= 64) return f(std::integral_constant<int, 64>{});
  return f(std::integral_constant<int, kTeamMost>{});
}

// Does the device hold all workgroups at once?  (Of its compute units each holds one.)
template <int D, bool K8>
bool team_fits(const Plan& pl) {
  return with_members<K8>(pl.team.most, [&](auto ml) {
    static std::atomic<int> cache[kMaxDevices];
    return resident_workgroups(score_team_kernel<D, kTeamTiles, K8, decltype(ml)::value>, 512, cache) >= pl.team.members;
  });
}

template <int D, bool K8>
int launch_team(const Plan& pl, const ScoreArgs& a, char* ws, hipStream_t stream) {
  constexpr int NT = kTeamTiles;
  TeamArgs ta;
  const TeamSchedule& s = pl.team;
  ta.lines = reinterpret_cast<uint32_t*>(ws + pl.off_stats);
  ta.ctl = reinterpret_cast<uint32_t*>(ws + pl.off_member);
  ta.pairs = (pl.R + 31) / 32;
  ta.problems = a.LH * a.n_seqs; ta.slots = s.slots; ta.most = s.most;
  ta.done = reinterpret_cast<uint32_t*>(ws + pl.off_stats + s.done_at);
  ta.apart = (pl.variant & CODECOMP_VARIANT_TEAMS_APART) != 0;
  ta.members = s.members; ta.ring = s.ring; ta.line_pairs = s.line_pairs; ta.steps = s.steps;
  for (int i = 0; i <= s.steps; ++i) ta.step[i] = s.step[i];
  for (int i = 0; i < (int)(s.step[s.steps] >> 16); ++i) { ta.entry[i][0] = s.entry[i][0]; ta.entry[i][1] = s.entry[i][1]; }
  score_team_prepare_kernel<D, K8><<<dim3((ta.pairs + 1) / 2, a.LH * a.n_seqs), dim3(256), 0, stream>>>(a, ta);
  if (hipError_t e = hipGetLastError()) return (int)e;
  const TeamKernelArgs args{a, ta};
  const dim3 grid(ta.members), block(512);
  return with_members<K8>(s.most, [&](auto ml) {
    constexpr int ML = decltype(ml)::value;
    score_team_kernel<D, NT, K8, ML><<<grid, block, 0, stream>>>(args);
    if (hipError_t e = hipGetLastError()) return (int)e;
    score_team_again_kernel<D, NT, K8, ML><<<dim3(2 * kTeamMembers), dim3(256), 0, stream>>>(args);
    return (int)hipGetLastError();
  });
}

}  // namespace codecomp
