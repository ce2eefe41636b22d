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
// (the row's largest logit among 16 of its keys) by 69 nats, a word in the workspace says so, and the launch behind this one
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
// Measured, scores of 28 layers, 4 KV heads of 7 query heads, window 64, 32K keys: two passes 873 us, teams 689; 1 layer 54 and 44; window
// 128 1648 and 1187; 8-bit keys 815 and 660.  Error against 64 bits 7e-8 (2-norm), by two passes 3.4e-7.
#pragma once
#include "score_once.h"

namespace codecomp {

constexpr uint32_t kTeamEmpty = 0xFFFFFFFFu;       // a sum that is not there yet; sums are stored without their sign bit
constexpr int kTeamRing = 16;                      // pairs of row blocks whose sums have a place

enum { kTeamAbsent = 0, kTeamRange = 1, kTeamTicket = 32 };        // control words: a wait has failed; rows of some problems are out of range; tasks handed out
constexpr uint32_t kTeamOut = 1, kTeamRedo = 2;    // a problem has rows out of range, as the team kernel found; as found again

__device__ __forceinline__ uint32_t team_load(const uint32_t* p) { return __hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT); }
__device__ __forceinline__ void team_store(uint32_t* p, uint32_t v) { __hip_atomic_store(p, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT); }

struct TeamArgs {
  uint32_t* lines;             // [place of a pair of row blocks][member][32]: row sums over the member's keys
  uint32_t* ctl;
  uint32_t* done;              // [problem][4] tasks of a phase that are done (score_team_again_kernel), then [problem] kTeamOut, kTeamRedo
  int problems, slots, most;   // problems; how many of them have a place for their sums at a time there; members of the largest team
  int pairs;                   // of row blocks in a problem
  int members, ring, line_pairs, steps;
  int apart;                   // 1: score_team_again_kernel does it all
  uint32_t step[kTeamSteps + 1];
  uint32_t entry[kTeamEntries][2];
};
// Longest wait for a sum, in 10 ns.  Members that run answer within some us; what this bounds is the time lost where some do not.
constexpr int64_t kTeamWait = 10000;

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
  static constexpr int KS = D / 32;                    // MFMA k-steps
  static constexpr int NW = 8;
  static constexpr int DB = 6;                         // blocks of 16 rows whose exponentials are kept: what the registers hold
  static constexpr int LAG = DB / 2;                   // ... pairs
  static constexpr int PER = KS / (K8 ? 2 : 1);        // 16-byte pieces per lane of a tile of keys
  static constexpr int KP = NT * PER;                  // ... of a wave's keys
  // Pieces of the next problem's keys that find no room in LDS beside the rest.  They are loaded when the problem begins.
  static constexpr int DIRECT = !K8 && D == 128 ? 2 : 0;
  static_assert(kTeamRing >= DB + 2, "a place is used again only when all have read it");
  struct Shared {
    u32x4 q[3][2][KS][64];       // query rows of three pairs of blocks, fragment order
    uint32_t poll[ML][32];       // row sums of the members, a share of the members to each wave
    float sums[NW][32];          // row sums of the waves over their own keys
    float team[LAG][NW][32];     // row sums of the team, each wave its share
    float ref[3][32];            // references of the rows of three pairs
    uint16_t row[kTeamRows + 64];          // where the query rows begin, in pieces of 16 bytes
    uint32_t summed[NW], ready[NW];        // pairs whose row sums a wave has left; ... whose team sums, and next query rows
    uint32_t quit;               // a wave has waited in vain
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
  // Pieces are sent for two by two (one by one where a tile has one): they share the lane's offset.
  constexpr int UNIT = PER > 1 ? 2 : 1, UNITS = STAGED / UNIT;
  auto key_at = [&](int i) __attribute__((always_inline)) {            // of piece i, less what is the same in all lanes
    const uint32_t key = (uint32_t)min(keys.key0 + i / PER * 16 + l16, keys.last);
    return key * key_bytes + (uint32_t)(grp * 16);
  };
  auto stage = [&](int u) __attribute__((always_inline)) {             // unit u of this wave's keys
    // A unit is a cache line of each key, so that the pairs ask alike of memory (with a half of both lines at a time, every second pair
    // asked for everything: 8 x 64K keys, 256 rows 544 us, now 526); but of a tile that is not all in LDS the first half of both lines is
    // there, and what is loaded when the problem begins is found in the cache.
    const int i = u * UNIT;
    const bool parted = PER == 4 && STAGED % PER != 0 && i >= STAGED / PER * PER;
    const int apart = parted ? 128 : 64;
    const unsigned char* from = keys.from + (PER == 4 ? (u & 1) * (parted ? 64 : 128) : UNIT == 2 ? 0 : (i & (PER - 1)) * 64);
    const uint32_t at = key_at(i), to = k_to + (uint32_t)i * 1024u;
    asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %1, %2" ::"s"(to), "v"(at), "s"(from) : "memory", "m0");
    if constexpr (UNIT == 2)
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
    if (D == 128 || wave < 2 * KS)
      asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %1, %2" ::"s"(q_to + slot * (2 * KS * 1024u)), "v"(row_at), "s"(rows.q) : "memory", "m0");
  };

  for (int r = tid; r < pairs * 32; r += 512) {        // rows past the end read the first one
    const int row = r < args.a.R ? r : 0, g = row_group(row, args.a.inv_w);
    sh.row[r] = (uint16_t)((uint32_t)g * ((uint32_t)args.a.q_sh / 8) + (uint32_t)(row - g * args.a.W) * ((uint32_t)args.a.q_st / 8));
  }
  if (tid < 8) sh.summed[tid] = sh.ready[tid] = 0;
  if (tid == 0) sh.quit = 0;
  for (int i = tid; i < ML * 32; i += 512) (&sh.poll[0][0])[i] = 0;
  asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory");
  keys = keys_of(cur);
  uint32_t row_at = sh.row[row_in] * 16u + piece_at;         // this lane's piece of the pair that is sent for next
  fetch(row_at, 0, 0);
  row_at = sh.row[32 + row_in] * 16u + piece_at;
  fetch(row_at, 1, 1);
  row_at = sh.row[64 + row_in] * 16u + piece_at;
  for (int u = 0; u < UNITS; ++u) stage(u);

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
          if (lane == 0) {
            team_store(team_args()->t.ctl + kTeamAbsent, 1);
            *(volatile __attribute__((address_space(3))) uint32_t*)&sh.quit = 1;
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
          for (int x = 0; x < (KS == 2 ? 4 : m == 1 ? 2 : 1); ++x) {
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
      if (__builtin_amdgcn_readfirstlane(*(volatile __attribute__((address_space(3))) uint32_t*)&sh.quit) != 0) {
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
      if (more) rows = team_rows(team_args(), nxt);    // else: what is sent for, to keep the count, is not used
      fpair = 0;
      row_from = reinterpret_cast<const uint16_t (*)[32]>(&sh.row[0]);
      row_at = (*row_from)[row_in] * 16u + piece_at;
    }
    if (q == cur_start + LAG - 1) {                    // the pair whose sums are collected is the current problem's first
      const team_args_t x = team_args();
      if (bad != 0 && lane == 0) {                     // the problem before has rows out of range
        team_store(x->t.done + x->t.problems * 4 + done_seq * x->a.LH + done_lz, kTeamOut);
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
// waiting for a workgroup that might not run.  Its tasks, one member's part of one problem in one of four phases, are handed out by a
// counter; a task waits only for tasks with smaller numbers, which run or are done.
//   0  row sums of the member, to memory          1  where a row of the problem is out of range: its largest logits become the references
//   2  ... and the sums are formed again          3  masses
// Where no wait has failed, only the problems with rows out of range are taken, without their phase 0.  The sums of some problems
// have a place at a time: their tasks come one phase after the other, and phase 0 of a problem waits for phase 3 of the one that had
// its place.
template <int D, int NT, bool K8, int ML>
__global__ __launch_bounds__(512, 2) void score_team_again_kernel(TeamKernelArgs args) {
  constexpr int KS = D / 32, ESZ = K8 ? 1 : 2, PL = ML / 8, kListed = 1024;
  using stage_t = std::conditional_t<K8, u32x2, u32x4>;
  const ScoreArgs& a = args.a;
  const TeamArgs& ta = args.t;
  bool whole = team_load(ta.ctl + kTeamAbsent) != 0;
  if (!whole && team_load(ta.ctl + kTeamRange) == 0) return;
  __shared__ float sums[kTeamRows / 32][8][32], weight[kTeamRows], ref[kTeamRows];
  __shared__ uint16_t list[kListed];
  __shared__ int ticket, listed, any;
  const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int l16 = lane & 15, grp = lane >> 4, l32 = lane & 31, hf = lane >> 5;
  const int pairs = ta.pairs;
  const float c = a.c;
  const f32x4 zero = {0.f, 0.f, 0.f, 0.f};
  if (!whole) {                                        // the problems with rows out of range, the same list in every workgroup
    if (wave == 0) {
      int count = 0;
      for (int at = 0; at < ta.problems; at += 64) {
        const bool mine = at + lane < ta.problems && (team_load(ta.done + (int64_t)ta.problems * 4 + at + lane) & kTeamOut) != 0;
        const uint64_t all = __ballot(mine);
        const int to = count + __popcll(all & ((1ull << lane) - 1));
        if (mine && to < kListed) list[to] = (uint16_t)(at + lane);
        count += __popcll(all);
      }
      if (lane == 0) listed = count;
    }
    __syncthreads();
    whole = __builtin_amdgcn_readfirstlane(listed) > kListed;
  }
  const int problems = whole ? ta.problems : __builtin_amdgcn_readfirstlane(listed);
  auto problem_at = [&](int i) { return whole ? i : __builtin_amdgcn_readfirstlane((int)list[i]); };
  auto members_of = [&](int problem) {
    const int seq = problem / a.LH;
    return ((a.cu_seqlens[seq + 1] - a.cu_seqlens[seq] - a.key_trim + 15) / 16 + 8 * NT - 1) / (8 * NT);
  };
  for (;;) {
    if (tid == 0) {
      ticket = (int)__hip_atomic_fetch_add(ta.ctl + kTeamTicket, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
      any = 0;
    }
    __syncthreads();
    // problems that have a place together, phase, problem, member: every problem counted with as many members as the largest has
    int x = __builtin_amdgcn_readfirstlane(ticket);
    const int first = x / (ta.slots * 4 * ta.most) * ta.slots, together = min(ta.slots, problems - first);
    x -= first * 4 * ta.most;
    if (together <= 0 || x >= together * 4 * ta.most) return;          // the last ones may be fewer
    const int phase = x / (together * ta.most);
    x -= phase * together * ta.most;
    const int at = first + x / ta.most, member = x % ta.most, problem = problem_at(at), chunks = members_of(problem);
    if (member >= chunks) { __syncthreads(); continue; }
    uint32_t* const done = ta.done + (int64_t)at * 4;
    uint32_t* const bad = ta.done + (int64_t)ta.problems * 4 + problem;
    {
      const bool place = phase == 0 && at >= ta.slots;
      const uint32_t need = place ? (uint32_t)members_of(problem_at(at - ta.slots)) : (uint32_t)chunks;
      const uint32_t* of = phase > 0 ? done + phase - 1 : done - (int64_t)ta.slots * 4 + 3;
      if (tid == 0) {
        if (place || phase > 0) while (team_load(of) < need) __builtin_amdgcn_s_sleep(4);
        __threadfence();
      }
    }
    __syncthreads();
    const int seq = problem / a.LH, lz = problem - seq * a.LH;
    TeamTask t;
    t.lz = lz; t.seq = seq; t.chunks = chunks;
    t.tok0 = a.cu_seqlens[seq]; t.n = a.cu_seqlens[seq + 1] - t.tok0 - a.key_trim;
    const int tiles = (t.n + 15) >> 4, each = tiles / chunks, more = tiles - each * chunks;
    t.tile0 = member * each + min(member, more); t.tiles = each + (member < more ? 1 : 0);
    const TeamShare own = team_share(t, wave);
    uint32_t* const lines = ta.lines + (int64_t)(at % ta.slots) * pairs * ta.most * 32;            // [pair][member][32]
    uint32_t* const refs = reinterpret_cast<uint32_t*>(a.lse) + ((int64_t)lz * a.n_seqs + seq) * a.lrows;

    bool redo = phase == 0 ? whole : true;
    if (phase == 2 && whole) redo = (__builtin_amdgcn_readfirstlane(team_load(bad)) & kTeamRedo) != 0;
    if (redo) for (int r = tid; r < pairs * 32; r += 512) ref[r] = __builtin_bit_cast(float, team_load(refs + (r < a.R ? r : 0)));
    if (phase == 3 || (phase == 1 && whole)) {
      // totals of the rows over the members, in the team kernel's order; a wave has every eighth pair
      for (int p = wave; p < pairs; p += 8) {
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
                const float v = __builtin_bit_cast(float, team_load(lines + ((int64_t)p * ta.most + min(m, chunks - 1)) * 32 + l32));
                x[i] = m < chunks ? v : 0.f;
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
        weight[p * 32 + l32] = there ? __builtin_fmaf(__builtin_fmaf(-total, r0, 1.0f), r0, r0) : 0.f;
        if (there && !(total <= 1.0e30f)) any = 1;
      }
    }
    __syncthreads();
    if (phase == 1 && whole) {                         // all members find the same
      redo = __builtin_amdgcn_readfirstlane(any) != 0;
      if (tid == 0 && redo) __hip_atomic_fetch_or(bad, kTeamRedo, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    }
    if (redo) {
      const int layer = divide(lz, a.Hkv, a.inv_heads), head = lz - layer * a.Hkv;
      const unsigned char* kb = a.k + ((int64_t)layer * a.kv_sl + (int64_t)head * a.kv_sh + (int64_t)t.tok0 * a.kv_st) * ESZ + grp * 8 * ESZ;
      const uint16_t* qb = a.q + (int64_t)layer * a.q_sl + (int64_t)seq * a.q_ss + (int64_t)(head * a.G) * a.q_sh + grp * 8;
      u32x4 kf[NT][KS];
#pragma unroll
      for (int i = 0; i < NT; ++i) {
        const unsigned char* from = kb + (int64_t)min(own.key0 + i * 16 + l16, t.n - 1) * a.kv_st * ESZ;
#pragma unroll
        for (int ks = 0; ks < KS; ++ks) kf[i][ks] = to_bf16x8(*reinterpret_cast<const stage_t*>(from + ks * 32 * ESZ));
      }
      f32x4 mass[NT];
#pragma unroll
      for (int i = 0; i < NT; ++i) mass[i] = zero;
      auto take_rows = [&](u32x4* to, int block) __attribute__((always_inline)) {      // rows past the end are the first one
        const int row = block * 16 + l16, r = row < a.R ? row : 0, g = row_group(r, a.inv_w);
        const uint16_t* from = qb + (int64_t)g * a.q_sh + (int64_t)(r - g * a.W) * a.q_st;
#pragma unroll
        for (int ks = 0; ks < KS; ++ks) to[ks] = *reinterpret_cast<const u32x4*>(from + ks * 32);
      };
      u32x4 qf[2][KS];
      take_rows(qf[0], 0);
      take_rows(qf[1], 1);
      for (int p = 0; p < pairs; ++p) {
        float sum_of[2] = {0.f, 0.f};
#pragma unroll
        for (int b = 0; b < 2; ++b) {
          const int row = p * 32 + b * 16 + l16;
          f32x4 s[NT];
#pragma unroll
          for (int i = 0; i < NT; ++i) {
            s[i] = zero;
#pragma unroll
            for (int ks = 0; ks < KS; ++ks) s[i] = once_mma(kf[i][ks], qf[b][ks], s[i]);
          }
          if (p + 1 < pairs) take_rows(qf[b], p * 2 + b + 2);
#pragma unroll
          for (int v = 0; v < 4; ++v)
            if (own.tiles < NT || own.key0 + (NT - 1) * 16 + 4 * grp + v >= t.n) s[NT - 1][v] = -INFINITY;
          if (phase == 1) {                            // the largest logits: of floats, as integers in the order of their sign
            float m = -INFINITY;
#pragma unroll
            for (int i = 0; i < NT; ++i)
#pragma unroll
              for (int v = 0; v < 4; ++v) m = fmaxf(m, s[i][v]);
            m = row_max4(m) * c;
            if (lane < 16 && row < a.R) {
              if (m >= 0.f) __hip_atomic_fetch_max(reinterpret_cast<int*>(refs + row), __builtin_bit_cast(int, m), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
              else if (m < 0.f) __hip_atomic_fetch_min(refs + row, __builtin_bit_cast(uint32_t, m), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            }
            continue;
          }
          const float rf = ref[row], w = phase == 3 ? weight[row] : 0.f;
          float sum = 0.f;
#pragma unroll
          for (int i = 0; i < NT; ++i)
#pragma unroll
            for (int v = 0; v < 4; ++v) {
              const float x = __builtin_amdgcn_exp2f(__builtin_fmaf(s[i][v], c, -rf));
              if (i == 0 && v == 0) sum = x; else sum += x;
              mass[i][v] = __builtin_fmaf(x, w, mass[i][v]);
            }
          sum_of[b] = sum;
        }
        if (phase == 0 || phase == 2) {
          float x, y, lo, hi;
          swap_halves(sum_of[0], sum_of[1], x, y);
          swap_rows(x + y, x + y, lo, hi);
          sums[p][wave][(hf << 4) + l16] = lo + hi;
        } else if (phase == 3 && (p + 1 == pairs || (a.row_splits > 1 && (p + 1) % a.nb == 0))) {
          float* u = a.uraw + ((int64_t)(p / a.nb) * a.LH + lz) * a.T + t.tok0;
#pragma unroll
          for (int i = 0; i < NT; ++i) {
            const float m = mass_of_rows(mass[i], l16);
            const int key = own.key0 + i * 16 + 4 * grp + (l16 & 3);
            if (l16 >> 2 == i && i < own.tiles && key < t.n) u[key] = m * a.inv_g;     // the lane counts: they differ in the order of the sum
            mass[i] = zero;
          }
        }
      }
      if (phase == 0 || phase == 2) {
        __syncthreads();
        for (int r = tid; r < pairs * 32; r += 512) {
          const float (&part)[8][32] = sums[r >> 5];
          const int i = r & 31;
          const float s = ((part[0][i] + part[1][i]) + (part[2][i] + part[3][i])) + ((part[4][i] + part[5][i]) + (part[6][i] + part[7][i]));
          team_store(lines + ((int64_t)(r >> 5) * ta.most + member) * 32 + i, __builtin_bit_cast(uint32_t, s) & 0x7FFFFFFFu);
        }
      }
    }
    __threadfence();
    __syncthreads();
    if (tid == 0) __hip_atomic_fetch_add(done + phase, 1u, __ATOMIC_RELEASE, __HIP_MEMORY_SCOPE_AGENT);
    // Not only for `ticket`: without a barrier here, what the first thread does at the end and at the start of a turn becomes one branch,
    // and the other lanes of its wave go round without it.
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
  for (int64_t i = at; i < (int64_t)ta.problems * 5; i += all) ta.done[i] = 0;
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
    if (!ta.apart) score_team_kernel<D, NT, K8, ML><<<grid, block, 0, stream>>>(args);
    if (hipError_t e = hipGetLastError()) return (int)e;
    score_team_again_kernel<D, NT, K8, ML><<<dim3(kTeamMembers), block, 0, stream>>>(args);
    return (int)hipGetLastError();
  });
}

}  // namespace codecomp
