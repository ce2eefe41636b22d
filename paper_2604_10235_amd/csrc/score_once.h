// Internal header: the score step of short requests in one pass over their logits.
//
// The two passes of score_pass.h form every logit twice because a request's keys are spread over workgroups and the row
// normalisers need all of them.  A request of up to kOnceKeys keys fits one workgroup: its keys stay in registers as MFMA
// fragments, its query rows come by in blocks of 16, and the exponentials of a block wait in registers until the block's row
// sums, exchanged between the waves through LDS, turn them into probabilities that are added to the keys' masses.  Every logit
// is formed once, every exponential taken once, every query row read once.
//
// v_mfma_f32_16x16x32_bf16, S^T = K Q^T: lane % 16 = query row, register and lane / 16 = key.  A wave owns NT tiles of 16 keys
// (K: D / 8 registers a tile), two sets of exponentials (4 registers a tile each: one is filled while the other waits for its
// weights) and the masses of its keys, one partial sum per lane (4 registers a tile), so that no value crosses lanes until the
// rows are through.  Blocks of 16 rows and not 32, as the two passes have: the waiting exponentials would take twice the
// registers, and half the keys would fit.
//
// Bound by instruction issue: 16 VALU instructions (fma, exponential, row sum, mass) and 4 MFMAs per tile and block.  A SIMD has 12
// tiles at most, six in each of its two waves: a block of 16 rows takes a compute unit 0.89 us for 768 keys (one workgroup of eight
// waves) and 0.97 us for two times 384 (two workgroups of four, which fill each other's waits), head_dim 128, that is 37 and 40 ns for a
// 32x32x16 MFMA's worth of logits; head_dim 64 0.68 and 0.72 us.  With its starts and unequal lengths a batch of chunks takes 62 and 56 ns,
// where the two passes together take 88.  Scores, two passes -> one pass: 28 query heads (window 128) on 4 KV heads, one request of 130
// tokens 22 -> 13 us, of 700 23 -> 21, 64 requests of 300 78 -> 31, of 760 122 -> 60, 16 layers of those 968 -> 470 and 1768 -> 1000; 28
// layers of 64 chunks of 135 to 1831 tokens (48 of them of up to 768) 2.73 -> 1.96 ms.
// Error against 64 bits (2-norm, 130 .. 768 keys): 5e-8 to 9e-8, of the two passes 1.8e-7 to 2.4e-7: the weight of a row is the
// reciprocal of its sum and not an exponent that was rounded.
#pragma once
#include "score_pass.h"

namespace codecomp {

typedef float f32x4 __attribute__((ext_vector_type(4)));

__device__ __forceinline__ f32x4 once_mma(u32x4 k, u32x4 q, f32x4 acc) {
  return __builtin_amdgcn_mfma_f32_16x16x32_bf16(frag(k), frag(q), acc, 0, 0, 0);
}

// x of this lane and of lane ^ 16 (lane ^ 32), in either order.
__device__ __forceinline__ void swap16(float x, float& a, float& b) {
  a = x; b = x;
  asm volatile("s_nop 1\n\tv_permlane16_swap_b32 %0, %1" : "+v"(a), "+v"(b));
}
__device__ __forceinline__ void swap32(float x, float& a, float& b) {
  a = x; b = x;
  asm volatile("s_nop 1\n\tv_permlane32_swap_b32 %0, %1" : "+v"(a), "+v"(b));
}
// Sum or largest of the four lanes that hold one query row (lane, lane ^ 16, lane ^ 32, lane ^ 48).
__device__ __forceinline__ float row_sum4(float x) {
  float a, b;
  swap16(x, a, b); swap32(a + b, a, b);
  return a + b;
}
__device__ __forceinline__ float row_max4(float x) {
  float a, b;
  swap16(x, a, b); swap32(fmaxf(a, b), a, b);
  return fmaxf(a, b);
}

// own + the other's value of the lane that the DPP control names (within 16 lanes).
template <int CTRL>
__device__ __forceinline__ float dpp_add(float own, float other) {
  return own + __builtin_bit_cast(float, __builtin_amdgcn_mov_dpp(__builtin_bit_cast(int, other), CTRL, 0xF, 0xF, true));
}

// The masses that a lane group holds of four keys, summed over its 16 rows: lane r gets key r % 4.
__device__ __forceinline__ float mass_of_rows(f32x4 mass, int l16) {
  const bool odd = l16 & 1, upper = l16 & 2;
  const float x0 = dpp_add<0xB1>(odd ? mass[1] : mass[0], odd ? mass[0] : mass[1]);      // with lane ^ 1
  const float x1 = dpp_add<0xB1>(odd ? mass[3] : mass[2], odd ? mass[2] : mass[3]);
  float x = dpp_add<0x4E>(upper ? x1 : x0, upper ? x0 : x1);                             // with lane ^ 2
  x = dpp_add<0x124>(x, x);                                                              // row_ror:4
  return dpp_add<0x128>(x, x);                                                           // row_ror:8
}

// Keeps a value where it is written: left alone, the compiler puts the masses off, so that both sets of exponentials live on beside
// new ones, and the exponentials behind the next wait, away from the MFMAs.
template <class T>
__device__ __forceinline__ void pin(T& x) { asm volatile("" : "+v"(x)); }

template <int D, int NW, bool K8>
struct Once {
  static constexpr int KS = D / 32;                 // MFMA k-steps
  static constexpr int ROUND = NW / KS;             // query blocks that the waves fetch together, one fragment each
  static constexpr int RING = 16;                   // query blocks in LDS
  static constexpr int AHEAD = RING / ROUND - 1;    // rounds on their way
  static constexpr int REFS = 4;                    // blocks whose references are found together, one wave each
  static constexpr int LATEST = AHEAD - (2 * REFS + ROUND - 1) / ROUND;   // rounds that may still be on their way in block b: block b + 8 is there
  static_assert(RING % ROUND == 0 && LATEST >= 1, "query ring");
  struct Shared {
    u32x4 q[RING][KS][64];                          // query blocks in fragment order
    float sums[2][16][NW];                          // row sums of the waves
    int64_t row[kOnceRows];          // where the query rows begin, in elements
    float ref[kOnceRows];            // per row: reference logit times c
  };
};

// One request and row split with NT tiles per wave.  `base` tiles to every wave, one more to the last `extra` waves, so that
// only the last tile of a wave can hold places without a key.
template <int D, int NW, bool K8, int NT>
__device__ __forceinline__ void once_run(const ScoreArgs& a, typename Once<D, NW, K8>::Shared& sh, int lz, int seq, int tok0, int n,
                                         int chunk0, int chunk1) {
  using O = Once<D, NW, K8>;
  constexpr int KS = O::KS, ESZ = K8 ? 1 : 2;
  using stage_t = std::conditional_t<K8, u32x2, u32x4>;
  const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int l16 = lane & 15, grp = lane >> 4;
  const int layer = lz / a.Hkv, head = lz - layer * a.Hkv;
  const int tiles = (n + 15) >> 4, base = tiles / NW, extra = tiles - base * NW;
  const int key0 = (wave * base + max(0, wave - (NW - extra))) * 16;       // this wave's first key
  const int mine = base + (wave >= NW - extra ? 1 : 0);                    // its tiles: NT or NT - 1
  const float c = a.c;

  auto barrier = [&]() __attribute__((always_inline)) { asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory"); };

  // ---- keys: fragments for the whole run; places without a key repeat the last one (masked below)
  const unsigned char* kb = a.k + ((int64_t)layer * a.kv_sl + (int64_t)head * a.kv_sh + (int64_t)tok0 * a.kv_st) * ESZ + grp * 8 * ESZ;
  u32x4 kf[NT][KS];
#pragma unroll
  for (int t = 0; t < NT; ++t) {
    const unsigned char* p = kb + (int64_t)min(key0 + t * 16 + l16, n - 1) * a.kv_st * ESZ;
#pragma unroll
    for (int ks = 0; ks < KS; ++ks) kf[t][ks] = to_bf16x8(*reinterpret_cast<const stage_t*>(p + ks * 32 * ESZ));
  }
  // start value of the last tile's logits: 0, or -inf where there is no key
  f32x4 mask;
#pragma unroll
  for (int v = 0; v < 4; ++v) mask[v] = mine == NT && key0 + (NT - 1) * 16 + 4 * grp + v < n ? 0.f : -INFINITY;
  const f32x4 zero = {0.f, 0.f, 0.f, 0.f};

  // ---- query rows
  const uint16_t* qb = a.q + (int64_t)layer * a.q_sl + (int64_t)seq * a.q_ss + (int64_t)(head * a.G) * a.q_sh;
  for (int chunk = chunk0; chunk < chunk1; ++chunk) {
  const int row0 = chunk * a.once_rows, rows = min(a.R - row0, a.once_rows);
  const int blocks = (rows + 15) >> 4;
  if (chunk > chunk0) barrier();                                           // every wave is through with the chunk before
  for (int r = tid; r < blocks * 16; r += NW * 64) {                       // rows past the end read the first one
    const int row = row0 + (r < rows ? r : 0);
    const int g = row_group(row, a.inv_w);
    sh.row[r] = (int64_t)g * a.q_sh + (int64_t)(row - g * a.W) * a.q_st;
  }
  barrier();
  // Query blocks go straight into LDS, one fragment (64 x 16 bytes, lane order) per wave and round.  The loads write no register;
  // they are counted by hand (before the barrier that makes a block visible, and all of them at the end of a run), because the
  // compiler would let every LDS read wait for all of them.  Nothing else in the loop loads from memory.  Through registers, a
  // block's rows arrived one block after they were asked for, and every block waited: 2.4 times as long.
  const uint32_t ring = (uint32_t)(uintptr_t)(__attribute__((address_space(3))) void*)&sh.q[0][0][0];
  const int fetch_ks = wave % KS;
  const uint32_t fetch_to = ring + (uint32_t)((wave / KS) * KS + fetch_ks) * 1024u;
  auto place = [&](int round) __attribute__((always_inline)) {
    return qb + sh.row[min(round * O::ROUND + wave / KS, blocks - 1) * 16 + l16] + (fetch_ks * 4 + grp) * 8;
  };
  auto fetch = [&](int round, const uint16_t* from) __attribute__((always_inline)) {
    const uint32_t to = fetch_to + (uint32_t)((round * O::ROUND) % O::RING) * (KS * 1024u);
    asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %1, off" ::"s"(to), "v"(from) : "memory", "m0");
  };
  const uint16_t* next_place;          // of the round to be sent for next: its rows are looked up a round ahead
  auto fetch_first = [&]() __attribute__((always_inline)) {
#pragma unroll 1
    for (int i = 0; i < O::AHEAD; ++i) fetch(i, place(i));
    next_place = place(O::AHEAD);
  };
  // The reference of a row is its largest logit among 16 of the request's keys: those of tile 0 of the wave whose turn it is.
  // Four blocks at a time, a wave each, four to seven blocks ahead.  (All of them before the loop: the query rows are read twice,
  // 8 % slower.  References of each lane's own: the sums then come with powers of two, 500 cycles a block more.)
  auto find_ref = [&](int b) __attribute__((always_inline)) {
    f32x4 s = zero;
#pragma unroll
    for (int ks = 0; ks < KS; ++ks) s = once_mma(kf[0][ks], sh.q[b % O::RING][ks][lane], s);
    const float m = row_max4(fmaxf(fmaxf(s[0], s[1]), fmaxf(s[2], s[3])));
    if (lane < 16) sh.ref[b * 16 + l16] = m * c;
  };

  f32x4 e[2][NT], mass[NT];
  u32x4 qf[KS];
  bool again = false;                  // second run, with the rows' largest logits as references
  for (;;) {
    fetch_first();
    asm volatile("s_waitcnt vmcnt(%0)" ::"i"(O::LATEST) : "memory");
    barrier();
    if (!again && wave < O::REFS && wave < blocks) find_ref(wave);
    barrier();
#pragma unroll
    for (int t = 0; t < NT; ++t) { mass[t] = zero; e[0][t] = zero; e[1][t] = zero; }
#pragma unroll
    for (int ks = 0; ks < KS; ++ks) qf[ks] = sh.q[0][ks][lane];
    float ref = sh.ref[l16], ref_prev = 0.f;       // of the block whose logits are formed, of the one before
    float sum = 0.f, w = 0.f;                      // row sum of a block in this lane; weight of the block that is added to the masses
    bool bad = false;

    // The row sums of a block, in three steps: every wave leaves its own; after a barrier all are read; they make the weight.
    float part[NW];
    auto sums_out = [&](auto par) __attribute__((always_inline)) {
      const float r = row_sum4(sum);
      if (lane < 16) sh.sums[decltype(par)::value][l16][wave] = r;
      sum = 0.f;
    };
    auto sums_in = [&](auto par) __attribute__((always_inline)) {
#pragma unroll
      for (int i = 0; i < NW; i += 4) *reinterpret_cast<float4*>(part + i) = *reinterpret_cast<const float4*>(&sh.sums[decltype(par)::value][l16][i]);
    };
    auto weigh = [&](int b) __attribute__((always_inline)) {
      float total = (part[0] + part[1]) + (part[2] + part[3]);
      if constexpr (NW == 8) total += (part[4] + part[5]) + (part[6] + part[7]);
      const bool row = b >= 0 && b * 16 + l16 < rows;
      // A logit outran the reference by 69 nats (or is NaN).  Rows past the end count: each repeats a row that may be in range, against
      // another reference, and its weight of 0 does not take away an infinite exponential.
      bad |= b >= 0 && !(total <= 1.0e30f);
      const float r0 = __builtin_amdgcn_rcpf(total);
      w = row ? __builtin_fmaf(__builtin_fmaf(-total, r0, 1.0f), r0, r0) : 0.f;
    };
    // Block b (set PAR): its logits are formed tile by tile; beside a tile's MFMAs the exponentials of the tile before it are
    // taken and the next place of the set gives up the probabilities of block b - 2.
    auto block = [&](int b, auto par) __attribute__((always_inline)) {
      constexpr int PAR = decltype(par)::value;
      float ref_next;
      const float w_now = w;
#pragma unroll
      for (int t = 0; t < NT; ++t) {
        // the barrier a step after the sums went out, where there is one before the next block's query rows are read
        if (t == (NT > 3 ? 2 : 1)) barrier();
        if (NT > 1 && t == NT - 1) {
          sums_in(par);
          ref_next = sh.ref[min(b + 1, blocks - 1) * 16 + l16];
        }
        __builtin_amdgcn_sched_barrier(0);
        f32x4& prev = t > 0 ? e[PAR][t - 1] : e[PAR ^ 1][NT - 1];
        const float rf = t > 0 ? ref : ref_prev;
        f32x4 s = t == NT - 1 ? mask : zero;
#pragma unroll
        for (int ks = 0; ks < KS; ++ks) {
          s = once_mma(kf[t][ks], qf[ks], s);
          if (NT > 1 && t == NT - 1) qf[ks] = sh.q[(b + 1) % O::RING][ks][lane];
        }
        if (t < NT - 1)
#pragma unroll
          for (int v = 0; v < 4; ++v) mass[t + 1][v] = __builtin_fmaf(e[PAR][t + 1][v], w_now, mass[t + 1][v]);
        if (t < NT - 1) pin(mass[t + 1]);
#pragma unroll
        for (int v = 0; v < 4; ++v) {
          const float x = __builtin_amdgcn_exp2f(__builtin_fmaf(prev[v], c, -rf));
          prev[v] = x;
          sum += x;
        }
        pin(prev); pin(sum);
        e[PAR][t] = s;
        if (t == 0) {
          if (b % O::ROUND == 0) {
            fetch(b / O::ROUND + O::AHEAD, next_place);
            next_place = place(b / O::ROUND + O::AHEAD + 1);
          }
          asm volatile("s_waitcnt vmcnt(%0)" ::"i"(O::LATEST) : "memory");
          sums_out(par);
          if (PAR == 0 && b % O::REFS == 0 && wave / O::REFS == (b / O::REFS) % (NW / O::REFS)) {
            const int next = b + O::REFS + wave % O::REFS;
            if (next < blocks && !again) find_ref(next);
          }
          if constexpr (NT == 1) {
            barrier();
            sums_in(par);
            ref_next = sh.ref[min(b + 1, blocks - 1) * 16 + l16];
#pragma unroll
            for (int ks = 0; ks < KS; ++ks) qf[ks] = sh.q[(b + 1) % O::RING][ks][lane];
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
            // an exponential's sum comes one instruction after it
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
          weigh(b - 1);
#pragma unroll
          for (int v = 0; v < 4; ++v) mass[0][v] = __builtin_fmaf(e[PAR ^ 1][0][v], w, mass[0][v]);
          pin(mass[0]);
        }
      }
      ref_prev = ref; ref = ref_next;
    };
    int b = 0;
    for (; b + 1 < blocks; b += 2) {
      block(b, std::integral_constant<int, 0>{});
      block(b + 1, std::integral_constant<int, 1>{});
    }
    // what is left: the masses of the last block but one (set LAST ^ 1, first place done), the exponentials of the last tile and
    // the masses of the last block
    auto finish = [&](auto last) __attribute__((always_inline)) {
      constexpr int LAST = decltype(last)::value;
#pragma unroll
      for (int t = 1; t < NT; ++t)
#pragma unroll
        for (int v = 0; v < 4; ++v) mass[t][v] = __builtin_fmaf(e[LAST ^ 1][t][v], w, mass[t][v]);
#pragma unroll
      for (int v = 0; v < 4; ++v) {
        const float x = __builtin_amdgcn_exp2f(__builtin_fmaf(e[LAST][NT - 1][v], c, -ref_prev));
        e[LAST][NT - 1][v] = x;
        sum += x;
      }
      sums_out(std::integral_constant<int, LAST ^ 1>{});
      barrier();
      sums_in(std::integral_constant<int, LAST ^ 1>{});
      weigh(blocks - 1);
#pragma unroll
      for (int t = 0; t < NT; ++t)
#pragma unroll
        for (int v = 0; v < 4; ++v) mass[t][v] = __builtin_fmaf(e[LAST][t][v], w, mass[t][v]);
    };
    if (b < blocks) {
      block(b, std::integral_constant<int, 0>{});
      finish(std::integral_constant<int, 0>{});
    } else {
      finish(std::integral_constant<int, 1>{});
    }
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");        // no load into LDS outlives the run
    if (again || __ballot(bad) == 0) break;      // all waves hold the same sums: all leave or none
    // ---- a logit far above its row's reference: the rows' largest logits, then everything again
    again = true;
    for (int b2 = 0; b2 < blocks; ++b2) {
      const uint16_t* qp = qb + sh.row[b2 * 16 + l16] + grp * 8;
#pragma unroll
      for (int ks = 0; ks < KS; ++ks) qf[ks] = *reinterpret_cast<const u32x4*>(qp + ks * 32);
      float m = -INFINITY;
#pragma unroll
      for (int t = 0; t < NT; ++t) {
        f32x4 s = t == NT - 1 ? mask : zero;
#pragma unroll
        for (int ks = 0; ks < KS; ++ks) s = once_mma(kf[t][ks], qf[ks], s);
        m = fmaxf(m, fmaxf(fmaxf(s[0], s[1]), fmaxf(s[2], s[3])));
      }
      m = row_max4(m);
      barrier();                                          // the sums of the block before have been read
      if (lane < 16) sh.sums[0][l16][wave] = m;
      barrier();
#pragma unroll
      for (int i = 0; i < NW; ++i) m = fmaxf(m, sh.sums[0][l16][i]);
      if (wave == 0 && lane < 16) sh.ref[b2 * 16 + l16] = m * c;
    }
      barrier();
  }

  // ---- masses, one store per tile
  float* u = a.uraw + ((int64_t)chunk * a.LH + lz) * a.T + tok0;
#pragma unroll
  for (int t = 0; t < NT; ++t) {
    const float x = mass_of_rows(mass[t], l16);
    const int key = key0 + t * 16 + 4 * grp + l16;
    if (l16 < 4 && t < mine && key < n) u[key] = x * a.inv_g;
  }
  }   // chunks
}

// Requests with more than n_above and at most n_most keys; a workgroup takes `group` row chunks of its problem in turn.  Heads and requests
// on axes of their own: one axis holds no more than 2^32 threads.
template <int D, int NW, bool K8>
__global__ __launch_bounds__(NW * 64, 2) void score_once_kernel(ScoreArgs a, int n_above, int n_most, int group) {
  __shared__ __attribute__((aligned(16))) typename Once<D, NW, K8>::Shared sh;
  const int chunk0 = (int)blockIdx.z * group, chunk1 = min(chunk0 + group, a.once_chunks);
  const int seq = (int)blockIdx.y, lz = (int)blockIdx.x;                      // neighbours are heads of one request: as much work on every die
  const int tok0 = a.cu_seqlens[seq];
  const int n = a.cu_seqlens[seq + 1] - tok0 - a.key_trim;
  if (n <= n_above || n > n_most) return;
  const int nt = ((n + 15) / 16 + NW - 1) / NW;
  switch (nt) {
    case 1: once_run<D, NW, K8, 1>(a, sh, lz, seq, tok0, n, chunk0, chunk1); break;
    case 2: once_run<D, NW, K8, 2>(a, sh, lz, seq, tok0, n, chunk0, chunk1); break;
    case 3: once_run<D, NW, K8, 3>(a, sh, lz, seq, tok0, n, chunk0, chunk1); break;
    case 4: once_run<D, NW, K8, 4>(a, sh, lz, seq, tok0, n, chunk0, chunk1); break;
    case 5: once_run<D, NW, K8, 5>(a, sh, lz, seq, tok0, n, chunk0, chunk1); break;
    case 6: once_run<D, NW, K8, 6>(a, sh, lz, seq, tok0, n, chunk0, chunk1); break;
  }
}

// The requests of a call that take one pass: up to kOnceKeys / 2 keys in workgroups of four waves, two to a compute unit, the
// others in workgroups of eight.  Where all workgroups find a compute unit at once, a second launch would only come after the first.
template <int D, bool K8>
int launch_once(const Plan& pl, const ScoreArgs& a, hipStream_t stream) {
  const dim3 grid(pl.L * pl.Hkv, pl.n_seqs, (pl.once_chunks + pl.once_group - 1) / pl.once_group);
  const bool together = pl.once_long && pl.once_short && (int64_t)grid.x * grid.y * grid.z <= kOnceFill;
  if (pl.once_long) {
    score_once_kernel<D, 8, K8><<<grid, dim3(512), 0, stream>>>(a, together ? 0 : kOnceKeys / 2, kOnceKeys, pl.once_group);
    if (hipError_t e = hipGetLastError()) return (int)e;
  }
  if (pl.once_short && !together) {
    score_once_kernel<D, 4, K8><<<grid, dim3(256), 0, stream>>>(a, 0, kOnceKeys / 2, pl.once_group);
    if (hipError_t e = hipGetLastError()) return (int)e;
  }
  return 0;
}

// ---------------------------------------------------------------------------------------------------------
// Few query rows: all of them at once.
// ---------------------------------------------------------------------------------------------------------
// Up to 64 rows leave room for all logits of a longer request in one workgroup's registers (RB blocks of 16 rows, TT tiles of 16
// keys per wave: 4 RB TT registers), so that the keys only pass through.  The rows' largest logits and sums are exchanged
// between the waves once each.  Bound by the memory round trips of a compute unit,
// then by issue; figures at kRowsProblems and rows_quicker (api.hip).
template <int RB>
struct Rows {
  static constexpr int TT = rows_tiles(RB);
  struct Shared {
    float largest[RB][16][8], sums[RB][16][8];
  };
};

template <int D, bool K8, int RB>
__global__ __launch_bounds__(512, 2) void score_rows_kernel(ScoreArgs a) {
  constexpr int KS = D / 32, ESZ = K8 ? 1 : 2, NW = 8, TT = Rows<RB>::TT;
  constexpr int GROUP = D == 128 && !K8 ? 2 : 4;   // tiles sent for together, a group ahead
  using stage_t = std::conditional_t<K8, u32x2, u32x4>;
  __shared__ __attribute__((aligned(16))) typename Rows<RB>::Shared sh;
  const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int l16 = lane & 15, grp = lane >> 4;
  const int seq = (int)blockIdx.y, lz = (int)blockIdx.x;
  const int tok0 = a.cu_seqlens[seq];
  const int n = a.cu_seqlens[seq + 1] - tok0 - a.key_trim;
  if (n <= 0 || n > TT * NW * 16) return;          // longer ones: the host has taken another kernel
  const int layer = lz / a.Hkv, head = lz - layer * a.Hkv;
  const int tiles = (n + 15) >> 4, base = tiles / NW, extra = tiles - base * NW;
  const int key0 = (wave * base + max(0, wave - (NW - extra))) * 16;
  const int mine = base + (wave >= NW - extra ? 1 : 0);
  const float c = a.c;

  const unsigned char* kb = a.k + ((int64_t)layer * a.kv_sl + (int64_t)head * a.kv_sh + (int64_t)tok0 * a.kv_st) * ESZ + grp * 8 * ESZ;
  stage_t kf[2][GROUP][KS];
  auto load = [&](int t0, stage_t (&dst)[GROUP][KS]) __attribute__((always_inline)) {
#pragma unroll
    for (int i = 0; i < GROUP; ++i) {
      const unsigned char* p = kb + (int64_t)min(key0 + (t0 + i) * 16 + l16, n - 1) * a.kv_st * ESZ;
#pragma unroll
      for (int ks = 0; ks < KS; ++ks) dst[i][ks] = *reinterpret_cast<const stage_t*>(p + ks * 32 * ESZ);
    }
  };
  load(0, kf[0]);
  u32x4 qf[RB][KS];
#pragma unroll
  for (int rb = 0; rb < RB; ++rb) {
    const int row = rb * 16 + l16 < a.R ? rb * 16 + l16 : 0;               // rows past the end read the first one
    const int g = row_group(row, a.inv_w);
    const uint16_t* p = a.q + (int64_t)layer * a.q_sl + (int64_t)seq * a.q_ss + (int64_t)(head * a.G + g) * a.q_sh +
                        (int64_t)(row - g * a.W) * a.q_st + grp * 8;
#pragma unroll
    for (int ks = 0; ks < KS; ++ks) qf[rb][ks] = *reinterpret_cast<const u32x4*>(p + ks * 32);
  }
  f32x4 e[TT][RB];
  const f32x4 zero = {0.f, 0.f, 0.f, 0.f};
  float m[RB];
#pragma unroll
  for (int rb = 0; rb < RB; ++rb) m[rb] = -INFINITY;
#pragma unroll
  for (int t0 = 0; t0 < TT; t0 += GROUP) {
    if (t0 < mine) {
      if (t0 + GROUP < TT && t0 + GROUP < mine) load(t0 + GROUP, kf[(t0 / GROUP + 1) & 1]);
#pragma unroll
      for (int i = 0; i < GROUP; ++i) {
        const int t = t0 + i;
        if (t >= TT) continue;
#pragma unroll
        for (int rb = 0; rb < RB; ++rb) {
          f32x4 s = zero;
#pragma unroll
          for (int ks = 0; ks < KS; ++ks) s = once_mma(to_bf16x8(kf[(t0 / GROUP) & 1][i][ks]), qf[rb][ks], s);
          if (t >= mine - 1) {                     // the wave's last tile may hold places without a key, those after it do not count
#pragma unroll
            for (int v = 0; v < 4; ++v) s[v] = t == mine - 1 && key0 + t * 16 + 4 * grp + v < n ? s[v] : -INFINITY;
          }
          e[t][rb] = s;
          m[rb] = fmaxf(fmaxf(m[rb], fmaxf(s[0], s[1])), fmaxf(s[2], s[3]));
        }
      }
    }
  }
#pragma unroll
  for (int rb = 0; rb < RB; ++rb) {
    const float x = row_max4(m[rb]);
    if (lane < 16) sh.largest[rb][l16][wave] = x;
  }
  __syncthreads();
  float sum[RB];
#pragma unroll
  for (int rb = 0; rb < RB; ++rb) {
    const float4 x = *reinterpret_cast<const float4*>(&sh.largest[rb][l16][0]), y = *reinterpret_cast<const float4*>(&sh.largest[rb][l16][4]);
    m[rb] = fmaxf(fmaxf(fmaxf(x.x, x.y), fmaxf(x.z, x.w)), fmaxf(fmaxf(y.x, y.y), fmaxf(y.z, y.w))) * c;
    sum[rb] = 0.f;
  }
#pragma unroll
  for (int t0 = 0; t0 < TT; t0 += GROUP) {
    if (t0 < mine) {
#pragma unroll
      for (int t = t0; t < t0 + GROUP && t < TT; ++t)
#pragma unroll
        for (int rb = 0; rb < RB; ++rb)
#pragma unroll
          for (int v = 0; v < 4; ++v) {
            const float x = __builtin_amdgcn_exp2f(__builtin_fmaf(e[t][rb][v], c, -m[rb]));
            e[t][rb][v] = x;
            sum[rb] += x;
          }
    }
  }
#pragma unroll
  for (int rb = 0; rb < RB; ++rb) {
    const float x = row_sum4(sum[rb]);
    if (lane < 16) sh.sums[rb][l16][wave] = x;
  }
  __syncthreads();
  float w[RB];
#pragma unroll
  for (int rb = 0; rb < RB; ++rb) {
    const float4 x = *reinterpret_cast<const float4*>(&sh.sums[rb][l16][0]), y = *reinterpret_cast<const float4*>(&sh.sums[rb][l16][4]);
    const float total = ((x.x + x.y) + (x.z + x.w)) + ((y.x + y.y) + (y.z + y.w));
    w[rb] = rb * 16 + l16 < a.R ? 1.0f / total : 0.f;
  }
  float* u = a.uraw + (int64_t)lz * a.T + tok0;
#pragma unroll
  for (int t = 0; t < TT; ++t) {
    if (t >= mine) continue;
    f32x4 mass = zero;
#pragma unroll
    for (int rb = 0; rb < RB; ++rb)
#pragma unroll
      for (int v = 0; v < 4; ++v) mass[v] = __builtin_fmaf(e[t][rb][v], w[rb], mass[v]);
    const float x = mass_of_rows(mass, l16);
    const int key = key0 + t * 16 + 4 * grp + l16;
    if (l16 < 4 && key < n) u[key] = x * a.inv_g;
  }
}

template <int D, bool K8>
int launch_rows(const Plan& pl, const ScoreArgs& a, hipStream_t stream) {
  const dim3 grid(pl.L * pl.Hkv, pl.n_seqs), block(512);
  switch ((pl.R + 15) / 16) {
    case 1: score_rows_kernel<D, K8, 1><<<grid, block, 0, stream>>>(a); break;
    case 2: score_rows_kernel<D, K8, 2><<<grid, block, 0, stream>>>(a); break;
    case 3: score_rows_kernel<D, K8, 3><<<grid, block, 0, stream>>>(a); break;
    default: score_rows_kernel<D, K8, 4><<<grid, block, 0, stream>>>(a); break;
  }
  if (hipError_t e = hipGetLastError()) return (int)e;
  return 0;
}

}  // namespace codecomp
