// Select step: per (layer, KV head, request) keep the last W tokens and the B - W best tokens
// of the prefix [0, N - W); equal scores go to the lower index; indices come out ascending
// (section "Attention-based KV Cache Compression": the best-scored context tokens are kept until the budget is used up).
//
// Counting rounds over order-preserving integer images of the float scores (LDS histograms) find the score of the last
// admitted token and how many tokens tied at that score are admitted; one ordered pass (prefix sums of "sure" and
// "tied" flags) then writes the indices already sorted.  No float is ever added, nothing depends on the order in which
// workgroups run: the result is the same bits on every call.
//
// Requests of at most 65536 candidates: one workgroup owns one (layer, head, request) problem; the candidates are read from
// memory once, all loads in flight together, and stay in registers until the indices are out.  In the fused call that
// workgroup also does the tail of the score step (finish_select_kernel).
// What bounds it is instruction issue and barriers of the one compute unit that works on a problem, so: few rounds, ballots
// instead of shuffles, register-to-register prefix sums, 16-byte loads and stores through buffer descriptors.  Measured
// (kernel times, the separate pooling kernel + the three-digit radix selection of 1024 threads before -> now): 2048 tokens
// x 4 problems 17.7 -> 4.6 us (binary prior: 5.6); 8192 x 8: 21.4 -> 7.7; 32768 x 112: 46.6 -> 26.4; 65536 x 256: 147 -> 69; sixteen requests
// of 8K .. 48K x 4 (by parts before): 67 -> 34; 64 requests of 135 .. 1831 x 112: 130 -> 31 us (142 .. 2313, next larger workgroup: 54).
// A batch with a longer request: every request is cut into parts of 8192 candidates and four kernels run one 256-thread
// workgroup per part (the third one per request), so that a problem is spread over as many compute units as it has parts:
//   counts  every part counts the first digit of its candidates (2048 bins) and stores the counts;
//   near    every part adds up the counts of its request, finds the bin that holds the cut, and appends its
//           candidates of that bin (keys only, in token order) to the request's list, at the place the
//           counts of the earlier parts give it; it also stores how many of its candidates lie above that bin;
//   resolve one workgroup per request finds the cut in the list (counting rounds in registers up to 16384 keys, two more
//           radix digits beyond; the list is short unless the scores crowd into one bin);
//   emit    every part counts what the earlier parts contribute and writes its own admitted indices at their
//           final places.
//
// Two selection rules share these pieces:
//   additive   : one selection on c = pooled attention + lambda * prior (the score kernel's output);
//   two-stage  : the paper's literal order - structure first, attention fills the rest
//                (sections "Span-Level Structural Protection" and "Attention-based KV Cache
//                Compression"): stage 1 keeps up to B_span = min(Bp, max(B_min, floor(rho * Bp)))
//                prefix tokens with prior > 0, largest prior first (ties: first in sequence, which for a
//                binary prior is the paper's rule for an overfull protected set: its first tokens),
//                Bp = B - W; stage 2 fills the remaining Bp - |P| slots with the best pooled-attention
//                tokens not in P.
#include <type_traits>

#include "cut_range.h"
#include "gather.h"

namespace codecomp {

constexpr uint32_t kForced = 0xFFFFFFFFu;      // key of a candidate that is admitted whatever the cut; 0: no candidate

// Monotone map float -> uint32 (larger float <=> larger key); -0 and +0 share a key.  Strictly between 0 and kForced,
// also for NaN.
__device__ __forceinline__ uint32_t order_key(float x) {
  x = x + 0.0f;   // -0 -> +0
  const uint32_t u = __float_as_uint(x);
  const uint32_t key = u ^ ((uint32_t)((int32_t)u >> 31) | 0x80000000u);      // negative: all bits flipped, else the sign bit set
  return min(max(key, 1u), kForced - 1u);
}

// ---------------------------------------------------------------------------------------------------------
// One workgroup per problem.
// ---------------------------------------------------------------------------------------------------------

constexpr int kCutList = 128;       // keys left to rank by comparing them with one another

// Slot s of thread tid holds candidate j = (s / 4) * 4 * NT + 4 * tid + s % 4: four consecutive candidates per thread and
// "quad" q = s / 4, the 256 candidates of a wave and quad consecutive too.
template <int NT> struct SelectShared {
  alignas(16) unsigned int hist[kCutBins];
  alignas(16) unsigned int list[kCutList];
  unsigned int list_n;
  unsigned int pick[3];
  alignas(16) unsigned int wave_a[NT / 64], wave_b[NT / 64];
  unsigned int chunk[NT / 4];       // per run of 256 consecutive candidates: admitted | tied << 16 (at most 16 quads)
};

// Rows are read and written through buffer descriptors: an access past `n` elements reads 0 and writes nothing, so that no
// index is clamped or compared and all loads of a thread are in flight together.  The whole byte offset is given as the
// vector offset, for that is what the bounds check covers: the builtins' scalar offset counts as outside of it.
typedef __amdgpu_buffer_rsrc_t rsrc_t;
template <class T>
__device__ __forceinline__ rsrc_t row_of(const T* p, int n) {
  return __builtin_amdgcn_make_buffer_rsrc(const_cast<void*>(static_cast<const void*>(p)), (short)0, max(n, 0) * (int)sizeof(T), 0x00020000);
}
__device__ __forceinline__ float4 row_f32x4(rsrc_t r, int byte) {
  return __builtin_bit_cast(float4, __builtin_amdgcn_raw_buffer_load_b128(r, byte, 0, 0));
}

// Prefix operations over the 64 lanes of a wave in six register-to-register steps (row shifts, then the last lane of a
// row of 16 and of the lower half broadcast upwards).
template <class Op>
__device__ __forceinline__ uint32_t wave_scan(uint32_t x, Op op) {
#define CODECOMP_DPP(CTRL, ROWS) \
  x = op(x, (uint32_t)__builtin_amdgcn_update_dpp((int)Op::kIdentity, (int)x, CTRL, ROWS, 0xf, false));
  CODECOMP_DPP(0x111, 0xf) CODECOMP_DPP(0x112, 0xf) CODECOMP_DPP(0x114, 0xf) CODECOMP_DPP(0x118, 0xf)
  CODECOMP_DPP(0x142, 0xa) CODECOMP_DPP(0x143, 0xc)
#undef CODECOMP_DPP
  return x;                         // lane i: op over lanes 0 .. i
}
struct OpAdd { static constexpr uint32_t kIdentity = 0u; __device__ uint32_t operator()(uint32_t a, uint32_t b) const { return a + b; } };
struct OpMin { static constexpr uint32_t kIdentity = ~0u; __device__ uint32_t operator()(uint32_t a, uint32_t b) const { return min(a, b); } };
struct OpMax { static constexpr uint32_t kIdentity = 0u; __device__ uint32_t operator()(uint32_t a, uint32_t b) const { return max(a, b); } };
__device__ __forceinline__ uint32_t last_lane(uint32_t x) { return (uint32_t)__builtin_amdgcn_readlane((int)x, 63); }

// op over the values that waves first .. last - 1 left in `of`; the same in every lane.
template <int NW, class Op>
__device__ __forceinline__ uint32_t over_waves(const unsigned int (&of)[NW], int first, int last, Op op) {
  uint32_t x = Op::kIdentity;
  if constexpr (NW <= 4) {
#pragma unroll
    for (int w = 0; w < NW; ++w) { const uint32_t o = of[w]; x = w >= first && w < last ? op(x, o) : x; }
    return (uint32_t)__builtin_amdgcn_readfirstlane((int)x);
  } else {
    const int lane = threadIdx.x & 63;
    if (lane < NW && lane >= first && lane < last) x = of[lane];
    return last_lane(wave_scan(x, op));
  }
}

// Runs body(s) for the slots in use, four at a time (a slot past them holds key 0, which nothing counts).
template <int ITEMS, class Body>
__device__ __forceinline__ void for_slots(int slots, Body body) {
  static_assert(ITEMS % 4 == 0, "groups of four slots");
#pragma unroll
  for (int g = 0; g < ITEMS; g += 4)
    if (g < slots) {
#pragma unroll
      for (int e = 0; e < 4; ++e) body(g + e);
    }
}

template <int NT>
__device__ __forceinline__ void hist_clear(SelectShared<NT>& sh) {
#pragma unroll
  for (int b = 0; b < kCutBins; b += NT) sh.hist[b + threadIdx.x] = 0;
}

// The bin that holds the `rank`-th largest counted key, its rank inside that bin and the bin's count (0: fewer than `rank`
// keys are counted).  Every thread sums its bins, prefix sums over lanes and waves find the one thread whose bins hold
// the rank.  All threads call it, behind a barrier after the last count.
template <int NT>
__device__ __forceinline__ void pick_bin(SelectShared<NT>& sh, uint32_t rank, uint32_t& bin, uint32_t& rank_in_bin, int& count) {
  constexpr int NW = NT / 64, PER = kCutBins / NT;
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  unsigned int own[PER], mine = 0;
#pragma unroll
  for (int i = 0; i < PER; ++i) { own[i] = sh.hist[tid * PER + i]; mine += own[i]; }
  const unsigned int incl = wave_scan(mine, OpAdd{}), total = last_lane(incl);
  if (lane == 0) sh.wave_a[wave] = total;
  if (tid == 0) sh.pick[2] = 0;                   // everyone has read the last pick: a barrier lies between
  __syncthreads();
  unsigned int higher = over_waves<NW>(sh.wave_a, wave + 1, NW, OpAdd{}) + total - incl;     // keys in the bins of higher waves and threads
  if (higher < rank && rank <= higher + mine) {
#pragma unroll
    for (int i = PER - 1; i >= 0; --i) {
      if (higher < rank && rank <= higher + own[i]) {
        sh.pick[0] = (unsigned int)(tid * PER + i); sh.pick[1] = rank - higher; sh.pick[2] = own[i];
      }
      higher += own[i];
    }
  }
  __syncthreads();
  bin = (uint32_t)__builtin_amdgcn_readfirstlane((int)sh.pick[0]);
  rank_in_bin = (uint32_t)__builtin_amdgcn_readfirstlane((int)sh.pick[1]);
  count = __builtin_amdgcn_readfirstlane((int)sh.pick[2]);
}

// The `need`-th largest competing key (1 <= need <= competing) and how many keys tied at it are admitted.  A thread
// holds keys[s], s < slots; 0 = no candidate, kForced = admitted whatever the cut, anything between competes.
//
// Counting rounds over the range [lo, hi] the cut is known to lie in, 2048 equal bins wide: the first range is that
// of the keys themselves (smallest to largest), so that the bins follow the scores wherever these sit; a fixed first digit
// (sign, exponent and two mantissa bits) put all of them into a few dozen bins, whose LDS atomics then wait for one another.
// The bin of the cut usually holds a handful of keys after one round: at most 128 are ranked by comparing all with all.
// From 16 candidates per thread on, the first round counts every eighth slot first and takes from that sample a bin that
// is almost surely below the cut: of the other slots only the keys from that bin up are counted (an LDS atomic
// costs by the number of lanes that take part).  Should the sample have misled, the rest is counted after all.
template <int NT, int ITEMS>
__device__ __forceinline__ void find_cut(SelectShared<NT>& sh, const uint32_t (&keys)[ITEMS], int slots, int competing, uint32_t need,
                                         uint32_t& tau, int& ties) {
  constexpr int NW = NT / 64;
  constexpr int kSampleEvery = 8;
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  uint32_t mn = 0xFFFFFFFFu, mx = 0u;                 // of key - 1 and key + 1: both kinds of non-competing keys drop out
  for_slots<ITEMS>(slots, [&](int s) { mn = min(mn, keys[s] - 1u); mx = max(mx, keys[s] + 1u); });
  mn = last_lane(wave_scan(mn, OpMin{}));
  mx = last_lane(wave_scan(mx, OpMax{}));
  if (lane == 0) { sh.wave_a[wave] = mn; sh.wave_b[wave] = mx; }
  hist_clear(sh);
  if (tid < kCutList) sh.list[tid] = 0;
  if (tid == 0) sh.list_n = 0;
  __syncthreads();
  uint32_t lo = over_waves<NW>(sh.wave_a, 0, NW, OpMin{}) + 1u;
  uint32_t hi = over_waves<NW>(sh.wave_b, 0, NW, OpMax{}) - 1u;
  // Which slots the next counting pass takes (bit 0: every eighth, bit 1: the others), the bins it counts, and the rank
  // that is looked up afterwards; one loop for all of them keeps the code short (it is fetched once per launch).
  enum { kSample = 1, kOthers = 2, kAll = 3, kRest = 6 };       // kRest: the others again, below the first bound
  int take = ITEMS >= 16 && slots > kSampleEvery ? kSample : kAll;
  uint32_t rank = need;
  uint32_t from = 0, span = hi - lo;             // counted: keys lo + from .. lo + from + span
  for (;;) {
    const uint32_t width = hi - lo;
    const int shift = cut_shift(width);
    for_slots<ITEMS>(slots, [&](int s) {
      if ((take >> (s % kSampleEvery != 0)) & 1) {
        const uint32_t d = keys[s] - lo;                      // 0 and kForced lie outside every range
        if (d - from <= span) atomicAdd(&sh.hist[d >> shift], 1u);
      }
    });
    __syncthreads();
    uint32_t bin, rank_in_bin, want = rank;
    int count;
    if (take == kSample) {       // the cut's rank in a sample of m of the n keys is about need * m / n: a tenth and three standard deviations more
      const float at = (float)need * (float)(((slots + kSampleEvery - 1) / kSampleEvery) * NT) / (float)competing;
      want = (uint32_t)(1.1f * at + 3.0f * __builtin_sqrtf(at) + 8.0f);
    }
    pick_bin<NT>(sh, want, bin, rank_in_bin, count);
    if (take == kSample) {
      from = count > 0 ? bin << shift : 0u;      // no such rank: the sample is smaller
      span = width - from;
      take = kOthers;
      continue;
    }
    if (take == kOthers && (count == 0 || (bin << shift) < from)) {             // misled: the bins below are needed after all
      span = from - 1u;
      from = 0;
      take = kRest;
      continue;
    }
    take = kAll;
    cut_narrow(lo, hi, bin, shift);
    rank = rank_in_bin;
    if (shift == 0) { tau = lo; ties = (int)rank; return; }
    if (count <= kCutList) {
      const uint32_t w = hi - lo;
      for_slots<ITEMS>(slots, [&](int s) {
        if (keys[s] - lo <= w) {                              // `count` entries, in any order
          const unsigned int at = atomicAdd(&sh.list_n, 1u);
          if (at < (unsigned int)kCutList) sh.list[at] = keys[s];              // always: belt and braces
        }
      });
      __syncthreads();
      if (tid < count) {
        const uint32_t k = sh.list[tid];
        unsigned int above = 0, equal = 0;
        for (int i = 0; i < count; i += 4) {           // (places past the last entry hold 0, below every key)
          const uint4 o = *reinterpret_cast<const uint4*>(&sh.list[i]);
          above += (o.x > k) + (o.y > k) + (o.z > k) + (o.w > k);
          equal += (o.x == k) + (o.y == k) + (o.z == k) + (o.w == k);
        }
        if (above < rank && rank <= above + equal) { sh.pick[0] = k; sh.pick[1] = rank - above; }   // equal keys write the same
      }
      __syncthreads();
      tau = (uint32_t)__builtin_amdgcn_readfirstlane((int)sh.pick[0]);
      ties = __builtin_amdgcn_readfirstlane((int)sh.pick[1]);
      return;
    }
    // Many keys in one bin are often one key many times (masses that are exactly 0), and every further round would have its
    // atomics wait for one another on that key's bin: the range is cut down to the keys in it first (65536 candidates, 97 % of
    // them 0: 183 us without, 80 with).  That pass is worth it only if one key makes up much of the bin, which is asked of the
    // first slot (15 % in one bin, nearly all different: 40.3 us with the pass always, 37.8 as it is).
    const uint32_t w = hi - lo;
    const bool many = count * 8 > slots * NT;
    if (many) {
      const unsigned long long in = __ballot(keys[0] - lo <= w);
      const uint32_t one = (uint32_t)__builtin_amdgcn_readlane((int)keys[0], in != 0 ? __ffsll(in) - 1 : 0);
      const int same = __popcll(__ballot(keys[0] == one) & in);
      if (lane == 0) sh.wave_a[wave] = (unsigned int)same;
    }
    hist_clear(sh);
    __syncthreads();
    if (many && over_waves<NW>(sh.wave_a, 0, NW, OpAdd{}) * 16u > (unsigned int)NT) {
      mn = 0xFFFFFFFFu, mx = 0u;
      for_slots<ITEMS>(slots, [&](int s) {
        const bool in = keys[s] - lo <= w;
        mn = in ? min(mn, keys[s]) : mn;
        mx = in ? max(mx, keys[s]) : mx;
      });
      mn = last_lane(wave_scan(mn, OpMin{}));
      mx = last_lane(wave_scan(mx, OpMax{}));
      __syncthreads();                             // wave_a has been read
      if (lane == 0) { sh.wave_a[wave] = mn; sh.wave_b[wave] = mx; }
      __syncthreads();
      lo = over_waves<NW>(sh.wave_a, 0, NW, OpMin{});
      hi = over_waves<NW>(sh.wave_b, 0, NW, OpMax{});
      if (lo == hi) { tau = lo; ties = (int)rank; return; }
    }
    from = 0;
    span = hi - lo;
  }
}

// The ordered output.  The counts of all runs of 256 consecutive candidates (wave and quad) are prefix-summed once;
// inside a run the lower lanes' candidates come first.  emit(j, admitted, pos) is called for the candidates, pos = number of
// admitted candidates before j: neighbouring lanes write neighbouring places.  ALL: also for those that are not admitted.
template <bool ALL, int NT, int ITEMS, class Emit>
__device__ __forceinline__ void emit_in_order(SelectShared<NT>& sh, const uint32_t (&keys)[ITEMS], int slots, int npre,
                                              uint32_t tau, int ties, Emit emit) {
  constexpr int NW = NT / 64, QUADS = ITEMS / 4;
  static_assert(QUADS <= 16 && QUADS * NW <= NT, "one run count per lane, one thread per run");
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  int mine = 0;
#pragma unroll
  for (int q = 0; q < QUADS; ++q) {
    if (4 * q >= slots) continue;
    int in = 0, tied = 0;
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      in += __popcll(__ballot(keys[4 * q + e] > tau));
      tied += __popcll(__ballot(keys[4 * q + e] == tau));
    }
    mine = lane == q ? in | tied << 16 : mine;
  }
  if (lane < QUADS) sh.chunk[lane * NW + wave] = (unsigned int)mine;       // quads not in use: 0
  __syncthreads();
  // fewer than 65536 candidates lie above the cut, so the low half never carries; all 65536 can be tied at it only
  // in the inclusive sum of the last run, which is not used
  const unsigned int x = tid < QUADS * NW ? sh.chunk[tid] : 0u;
  const unsigned int incl = wave_scan(x, OpAdd{});
  constexpr int SCANNED = (QUADS * NW + 63) / 64;                          // waves that hold a run's count
  if (SCANNED > 1) {
    if (lane == 63 && wave < SCANNED) sh.wave_b[wave] = incl;
    __syncthreads();
  }
  if (tid < QUADS * NW) {
    unsigned int before = incl - x;
#pragma unroll
    for (int w = 0; w < SCANNED - 1; ++w) before += w < wave ? sh.wave_b[w] : 0u;
    sh.chunk[tid] = before;
  }
  __syncthreads();
  const int base = lane < QUADS ? (int)sh.chunk[lane * NW + wave] : 0;
#pragma unroll
  for (int q = 0; q < QUADS; ++q) {
    if (4 * q >= slots) continue;
    const unsigned int b = (unsigned int)__builtin_amdgcn_readlane(base, q);
    int pos = (int)(b & 0xFFFFu), tb = (int)(b >> 16);
    unsigned long long any_tie = 0;
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      const unsigned long long m = __ballot(keys[4 * q + e] > tau);
      pos = (int)__builtin_amdgcn_mbcnt_hi((unsigned int)(m >> 32), __builtin_amdgcn_mbcnt_lo((unsigned int)m, (unsigned int)pos));
      any_tie |= __ballot(keys[4 * q + e] == tau);
    }
    if (any_tie != 0 && ties > 0) {
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        const unsigned long long m = __ballot(keys[4 * q + e] == tau);
        tb = (int)__builtin_amdgcn_mbcnt_hi((unsigned int)(m >> 32), __builtin_amdgcn_mbcnt_lo((unsigned int)m, (unsigned int)tb));
      }
    }
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      const int j = (q * NT + tid) * 4 + e;
      const bool in = keys[4 * q + e] > tau, tied = keys[4 * q + e] == tau;
      const bool admitted = in || (tied && tb < ties);
      if (ALL ? j < npre : admitted) emit(j, admitted, pos + min(tb, ties));
      pos += in;
      tb += tied;
    }
  }
}

struct SelectArgs {
  const float* scores;
  const float* prior;          // two-stage only
  const int32_t* cu_seqlens;
  const int32_t* cu_budgets;
  int32_t* idx;
  uint8_t* member;             // two-stage only: [T] 1 = token kept by stage 1
  int32_t* member_count;       // two-stage only: [n_seqs]
  int n_seqs, T, TB, W;
  float span_ratio;
  int span_min;
};

struct ScoreSource {            // additive rule: every prefix token competes on its fused score
  const float* sc;
  __device__ uint32_t key(int j) const { return order_key(sc[j]); }
  __device__ bool eligible(int) const { return true; }
  __device__ bool forced(int) const { return false; }
};
struct PriorSource {            // two-stage, stage 1: marked tokens compete on their prior
  const float* p;
  __device__ uint32_t key(int j) const { return order_key(p[j]); }
  __device__ bool eligible(int j) const { return p[j] > 0.f; }
  __device__ bool forced(int) const { return false; }
};
struct FillSource {             // two-stage, stage 2: protected tokens are in, the others compete on attention
  const float* sc;
  const uint8_t* member;
  __device__ uint32_t key(int j) const { return order_key(sc[j]); }
  __device__ bool eligible(int j) const { return member[j] == 0; }
  __device__ bool forced(int j) const { return member[j] != 0; }
};

// A row of floats into registers, all loads in flight together.
template <int NT, int ITEMS>
__device__ __forceinline__ void load_row(rsrc_t row, float (&x)[ITEMS]) {
#pragma unroll
  for (int s = 0; s < ITEMS; s += 4) {
    const float4 v = row_f32x4(row, ((int)threadIdx.x * 4 + s * NT) * 4);
    x[s] = v.x; x[s + 1] = v.y; x[s + 2] = v.z; x[s + 3] = v.w;
  }
}

// Slots that `count` candidates take per thread.
template <int NT>
__device__ __forceinline__ int slots_of(int count) { return (count + 4 * NT - 1) / (4 * NT) * 4; }

// Keys in registers -> indices of the `kept` tokens at `out`: the best `need` competing ones and the forced ones, or all.
template <int NT, int ITEMS>
__device__ __forceinline__ void select_and_emit(SelectShared<NT>& sh, const uint32_t (&keys)[ITEMS], int slots, int npre, int competing,
                                                int need, bool all, int kept, int32_t* out) {
  uint32_t tau = all ? 0u : kForced - 1u;       // every candidate / the forced ones only
  int ties = 0;
  if (!all && need > 0) find_cut<NT, ITEMS>(sh, keys, slots, competing, (uint32_t)need, tau, ties);
  const rsrc_t row = row_of(out, kept);         // pos < kept always; the descriptor is belt and braces
  emit_in_order<false, NT, ITEMS>(sh, keys, slots, npre, tau, ties, [&](int j, bool, int pos) {
    __builtin_amdgcn_raw_buffer_store_b32((uint32_t)j, row, pos * 4, 0, 0);
  });
}

// additive rule: one selection on the fused scores; two-stage rule, stage 2 (FILL): attention fills what stage 1 left
template <bool FILL, int NT, int ITEMS>
__global__ __launch_bounds__(NT) void select_kernel(SelectArgs a) {
  __shared__ SelectShared<NT> sh;
  const int tid = threadIdx.x;
  const int seq = blockIdx.x;
  const int lz = blockIdx.y;
  const int s0 = a.cu_seqlens[seq];
  const int npre = a.cu_seqlens[seq + 1] - s0 - a.W;   // candidates
  const int o0 = a.cu_budgets[seq];
  const int bp = a.cu_budgets[seq + 1] - o0 - a.W;     // how many of them are kept
  int32_t* out = a.idx + (int64_t)lz * a.TB + o0;
  for (int t = tid; t < a.W; t += NT) out[bp + t] = npre + t;      // the observation window is always kept
  if (bp <= 0 || npre > NT * ITEMS) return;            // the host picks ITEMS from the longest request: the latter cannot happen
  const int slots = slots_of<NT>(npre);
  const rsrc_t row = row_of(a.scores + (int64_t)lz * a.T + s0, npre);
  uint32_t keys[ITEMS];
  float x[ITEMS];
  uint8_t member[FILL ? ITEMS : 1];
  load_row<NT, ITEMS>(row, x);
  if constexpr (FILL) {
    const rsrc_t mrow = row_of(a.member + s0, npre);
#pragma unroll
    for (int s = 0; s < ITEMS; ++s) member[s] = __builtin_amdgcn_raw_buffer_load_b8(mrow, (s / 4 * NT + tid) * 4 + s % 4, 0, 0);
  }
#pragma unroll
  for (int s = 0; s < ITEMS; ++s) {
    keys[s] = (s / 4 * NT + tid) * 4 + s % 4 < npre ? order_key(x[s]) : 0u;
    if constexpr (FILL) keys[s] = member[s] ? kForced : keys[s];
  }
  const int members = FILL ? a.member_count[seq] : 0;
  select_and_emit<NT, ITEMS>(sh, keys, slots, npre, npre - members, bp - members, bp >= npre, bp, out);
}

constexpr int kFinishNear = 4;      // neighbours on a side that three 16-byte LDS reads cover

// The tail of the fused call in one kernel: the attention mass of a request is pooled, the prior added, the scores stored
// (what score_finish_kernel does, the same sums in the same order), and the selection goes on with the scores it holds in
// registers.  The masses pass through LDS, up to 32768 tokens at a time, so that a thread finds its neighbours there.
template <bool FILL, int NT, int ITEMS, int HALO, bool COPY>
__global__ __launch_bounds__(NT) void finish_select_kernel(SelectArgs a, FinishArgs f, GatherArgs g) {
  constexpr int BLOCK = ITEMS < 32768 / NT ? ITEMS : 32768 / NT;   // slots per LDS filling
  constexpr int NEAR = kFinishNear;
  static_assert(HALO % 4 == 0 && HALO >= NEAR, "16-byte LDS accesses");
  __shared__ __attribute__((aligned(16))) float mass[BLOCK * NT + 2 * HALO];
  __shared__ SelectShared<NT> sh;
  const int tid = threadIdx.x;
  const int seq = blockIdx.x;
  const int lz = blockIdx.y;
  const int s0 = a.cu_seqlens[seq];
  const int n = a.cu_seqlens[seq + 1] - s0;
  const int npre = n - a.W;                            // candidates
  const int o0 = a.cu_budgets[seq];
  const int bp = a.cu_budgets[seq + 1] - o0 - a.W;     // how many of them are kept
  int32_t* out = a.idx + (int64_t)lz * a.TB + o0;
  for (int t = tid; t < a.W; t += NT) out[bp + t] = npre + t;      // the observation window is always kept
  if (n > NT * ITEMS) return;                          // the host picks ITEMS from the longest request: cannot happen
  const int half = (f.pool - 1) >> 1;
  const int pooled_end = n - f.pool_trim;              // tokens from here on get no attention term
  const int mass_end = n - max(f.mass_trim, f.pool_trim);          // tokens from here on have no mass to pool
  const float* u = f.uraw + (int64_t)lz * f.T + s0;
  const int64_t split_stride = (int64_t)f.LH * f.T;
  const rsrc_t prior = row_of(f.prior + s0, n);
  const rsrc_t scores = row_of(f.scores + (int64_t)lz * f.T + s0, n);
  const rsrc_t members_row = row_of(a.member + s0, FILL ? npre : 0);
  float weight[NEAR + 1];                              // 1 for the neighbours that the pooling width reaches, else 0
#pragma unroll
  for (int t = 0; t <= NEAR; ++t) weight[t] = t <= half ? 1.f : 0.f;
  uint32_t keys[ITEMS];
#pragma unroll
  for (int s = 0; s < ITEMS; ++s) keys[s] = 0u;
#pragma unroll
  for (int b0 = 0; b0 < ITEMS; b0 += BLOCK) {
    const int width = b0 + BLOCK <= ITEMS ? BLOCK : ITEMS - b0;     // slots of this filling
    const int base = b0 * NT;
    if (base >= n) continue;                           // the same for every thread
    if (b0 > 0) __syncthreads();                       // the last filling has been read
    float4 v[BLOCK / 4];
    {
      const rsrc_t row = row_of(u, mass_end);
#pragma unroll
      for (int s = 0; s < BLOCK; s += 4)
        if (s < width) v[s / 4] = row_f32x4(row, (base + s * NT + tid * 4) * 4);
    }
    for (int sp = 1; sp < f.row_splits; ++sp) {        // added in the order of the splits
      const rsrc_t row = row_of(u + sp * split_stride, mass_end);
      float4 w[BLOCK / 4];
#pragma unroll
      for (int s = 0; s < BLOCK; s += 4)
        if (s < width) w[s / 4] = row_f32x4(row, (base + s * NT + tid * 4) * 4);
#pragma unroll
      for (int s = 0; s < BLOCK / 4; ++s)
        if (4 * s < width) { v[s].x += w[s].x; v[s].y += w[s].y; v[s].z += w[s].z; v[s].w += w[s].w; }
    }
    const int reach = max(half, NEAR);
    for (int i = tid; i < 2 * reach; i += NT) {        // the neighbours on both sides
      const int x = i < reach ? base - reach + i : base + width * NT + (i - reach);
      float val = 0.f;
      if (x >= 0 && x < mass_end)
        for (int sp = 0; sp < f.row_splits; ++sp) val += u[sp * split_stride + x];
      mass[HALO + x - base] = val;
    }
#pragma unroll
    for (int s = 0; s < BLOCK; s += 4)
      if (s < width) *reinterpret_cast<float4*>(&mass[HALO + (s / 4 * NT + tid) * 4]) = v[s / 4];
    __syncthreads();
#pragma unroll
    for (int s = 0; s < BLOCK; s += 4) {
      if (s >= width || base + s * NT >= n) continue;
      const int quad = base + s * NT + tid * 4;        // the first of four tokens
      float acc[4] = {0.f, 0.f, 0.f, 0.f};
      const float4 p4 = row_f32x4(prior, quad * 4);
      const float p[4] = {p4.x, p4.y, p4.z, p4.w};
      uint8_t member[4] = {0, 0, 0, 0};
      if constexpr (FILL) {
#pragma unroll
        for (int e = 0; e < 4; ++e) member[e] = __builtin_amdgcn_raw_buffer_load_b8(members_row, quad + e, 0, 0);
      }
      const float* m = mass + HALO + (s / 4 * NT + tid) * 4;
      if (half <= NEAR) {
        const float4 w0 = *reinterpret_cast<const float4*>(m - 4), w1 = *reinterpret_cast<const float4*>(m), w2 = *reinterpret_cast<const float4*>(m + 4);
        const float w[12] = {w0.x, w0.y, w0.z, w0.w, w1.x, w1.y, w1.z, w1.w, w2.x, w2.y, w2.z, w2.w};
        if (f.pool_max) {
#pragma unroll
          for (int t = -NEAR; t <= NEAR; ++t)
#pragma unroll
            for (int e = 0; e < 4; ++e) acc[e] = fmaxf(acc[e], weight[t < 0 ? -t : t] * w[4 + e + t]);           // masses are >= 0; NaN (0 * inf) loses
        } else {
#pragma unroll
          for (int t = -NEAR; t <= NEAR; ++t)
#pragma unroll
            for (int e = 0; e < 4; ++e) acc[e] = __builtin_fmaf(weight[t < 0 ? -t : t], w[4 + e + t], acc[e]);
          // 0 * inf has let a mass out of reach in as NaN, should there be infinite ones: once more without those out of reach
          if (__ballot(!(fabsf((acc[0] + acc[1]) + (acc[2] + acc[3])) < INFINITY)) != 0) {
#pragma unroll
            for (int e = 0; e < 4; ++e) acc[e] = 0.f;
#pragma unroll
            for (int t = -NEAR; t <= NEAR; ++t)
              if ((t < 0 ? -t : t) <= half)
#pragma unroll
                for (int e = 0; e < 4; ++e) acc[e] += w[4 + e + t];
          }
        }
      } else if (f.pool_max) {
        for (int t = -half; t <= half; ++t)
#pragma unroll
          for (int e = 0; e < 4; ++e) acc[e] = fmaxf(acc[e], m[e + t]);
      } else {
        for (int t = -half; t <= half; ++t)
#pragma unroll
          for (int e = 0; e < 4; ++e) acc[e] += m[e + t];
      }
      float c[4];
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        const int j = quad + e;
        const float pooled = f.pool_max ? acc[e] : acc[e] * f.inv_pool;
        c[e] = __builtin_fmaf(f.lambda, p[e], j < pooled_end ? pooled : 0.f);
        keys[b0 + s + e] = j < npre ? (member[e] ? kForced : order_key(c[e])) : 0u;
      }
      typedef unsigned int u32x4 __attribute__((ext_vector_type(4)));
      __builtin_amdgcn_raw_buffer_store_b128(__builtin_bit_cast(u32x4, make_float4(c[0], c[1], c[2], c[3])), scores, quad * 4, 0, 0);
    }
  }
  if (bp > 0) {
    const int slots = slots_of<NT>(npre);
    const int members = FILL ? a.member_count[seq] : 0;
    select_and_emit<NT, ITEMS>(sh, keys, slots, npre, npre - members, bp - members, bp >= npre, bp, out);
  }
  if constexpr (COPY) gather_request<NT>(g, lz, s0, n, o0, bp + a.W);
}

// two-stage rule, stage 1: once per request (the prior is shared by layers and heads)
template <int NT, int ITEMS>
__global__ __launch_bounds__(NT) void select_stage1_kernel(SelectArgs a) {
  __shared__ SelectShared<NT> sh;
  const int tid = threadIdx.x;
  const int seq = blockIdx.x;
  const int s0 = a.cu_seqlens[seq];
  const int npre = a.cu_seqlens[seq + 1] - s0 - a.W;
  const int bp = a.cu_budgets[seq + 1] - a.cu_budgets[seq] - a.W;           // slots of the prefix
  uint8_t* member = a.member + s0;
  for (int t = tid; t < a.W; t += NT) member[npre + t] = 0;
  if (npre <= 0 || npre > NT * ITEMS) {                                     // no candidate (more than fit cannot happen, as above)
    if (tid == 0) a.member_count[seq] = 0;
    return;
  }
  const int slots = slots_of<NT>(npre);
  const rsrc_t row = row_of(a.prior + s0, npre);
  uint32_t keys[ITEMS];
  float x[ITEMS];
  load_row<NT, ITEMS>(row, x);
#pragma unroll
  for (int s = 0; s < ITEMS; ++s) keys[s] = x[s] > 0.f ? order_key(x[s]) : 0u;       // past the row: 0, not marked
  // number of structurally marked prefix tokens
  int mine = 0;
  for_slots<ITEMS>(slots, [&](int s) { mine += __popcll(__ballot(keys[s] != 0u)); });
  if ((tid & 63) == 0) sh.chunk[tid >> 6] = (unsigned int)mine;
  __syncthreads();
  int flagged = 0;
#pragma unroll
  for (int w = 0; w < NT / 64; ++w) flagged += (int)sh.chunk[w];
  __syncthreads();
  int bspan = max(a.span_min, (int)floor((double)a.span_ratio * (double)bp));
  bspan = min(bp, bspan);
  const int need = min(bspan, flagged);
  if (tid == 0) a.member_count[seq] = max(need, 0);
  uint32_t tau = kForced - 1u;
  int ties = 0;
  if (need > 0) find_cut<NT, ITEMS>(sh, keys, slots, flagged, (uint32_t)need, tau, ties);
  emit_in_order<true, NT, ITEMS>(sh, keys, slots, npre, tau, ties, [&](int j, bool admitted, int) { member[j] = admitted ? 1 : 0; });
}

// ---------------------------------------------------------------------------------------------------------
// Selection by parts: several workgroups per problem, four kernels (see the head of this file).
// ---------------------------------------------------------------------------------------------------------

struct PartArgs {
  uint16_t* hist;        // [lz][part][2048] first-digit counts of each part (at most kPartChunk each)
  int32_t* sure;         // [lz][part] candidates of the part admitted whatever the cut: bins above the cut's, forced ones
  uint32_t* head;        // [lz][request][8]: mode, first digit of the cut, rank of the cut inside that bin, size of that bin,
                         //                   number of competing candidates admitted, key of the cut, ties admitted, 1 if `before` is filled in
  uint32_t* list;        // [lz][T] keys of the candidates in the cut's bin, per request from its first token on, in token order
  int32_t* before;       // [lz][part][2] candidates of the earlier parts in the cut's bin that lie above the cut / are tied at it
  int parts;             // parts of all requests together
};

enum { kModeNone = 0, kModeAll = 1, kModeSelect = 2 };   // no competing candidate admitted / all of them / a real selection

constexpr int kHistStride = 2049;     // odd stride: equal bins of different copies sit in different banks
constexpr int kPartCopies = 4;       // private copies of a histogram (lane % 4)
constexpr int kPartHistWords = 8 * (kFirstDigitBins / 2 + 1);   // 8 packed copies of the first-digit counts, or 4 plain copies of a digit
static_assert(kPartHistWords >= kPartCopies * kHistStride, "histogram storage of the part kernels");

struct PartShared {
  unsigned int hist[kPartHistWords];
  unsigned int prefix, need;
  int red[4][16];          // up to 16 waves (the resolve kernel)
  int found[4];
};

// The three rules as seen by the part kernels: where the candidates come from, how many of them are admitted, what
// is written for a candidate and for the window.
struct RuleAdditive {
  using Src = ScoreSource;
  __device__ static Src source(const SelectArgs& a, int lz, int s0) { return {a.scores + (int64_t)lz * a.T + s0}; }
  __device__ static int need(const SelectArgs& a, int, int budget, int npre, int, int& mode) {
    const int need = budget - a.W;
    mode = need <= 0 ? kModeNone : (need >= npre ? kModeAll : kModeSelect);
    return need;
  }
  __device__ static void emit(const SelectArgs& a, int lz, int, int o0, int j, bool admitted, int pos, int limit) {
    if (admitted && (unsigned)pos < (unsigned)limit) a.idx[(int64_t)lz * a.TB + o0 + pos] = j;   // pos < limit always: belt and braces
  }
  __device__ static void window(const SelectArgs& a, int lz, int, int, int o0, int budget, int npre, int, int t) {
    a.idx[(int64_t)lz * a.TB + o0 + (budget - a.W) + t] = npre + t;
  }
};
struct RuleStage1 {     // once per request: which marked tokens the span budget keeps
  using Src = PriorSource;
  __device__ static Src source(const SelectArgs& a, int, int s0) { return {a.prior + s0}; }
  __device__ static int need(const SelectArgs& a, int, int budget, int, int marked, int& mode) {
    const int bp = budget - a.W;
    int bspan = max(a.span_min, (int)floor((double)a.span_ratio * (double)bp));
    bspan = min(bp, bspan);
    const int need = min(bspan, marked);
    mode = need <= 0 ? kModeNone : kModeSelect;       // need == marked: the selection admits every marked token
    return need;
  }
  __device__ static void emit(const SelectArgs& a, int, int s0, int, int j, bool admitted, int, int) {
    a.member[s0 + j] = admitted ? 1 : 0;
  }
  __device__ static void window(const SelectArgs& a, int, int seq, int s0, int, int, int npre, int need, int t) {
    a.member[s0 + npre + t] = 0;
    if (t == 0) a.member_count[seq] = need > 0 ? need : 0;
  }
};
struct RuleStage2 {     // per (layer, head, request): attention fills what stage 1 left
  using Src = FillSource;
  __device__ static Src source(const SelectArgs& a, int lz, int s0) { return {a.scores + (int64_t)lz * a.T + s0, a.member + s0}; }
  __device__ static int need(const SelectArgs& a, int seq, int budget, int npre, int, int& mode) {
    const int bp = budget - a.W;
    if (bp <= 0) { mode = kModeNone; return 0; }
    if (bp >= npre) { mode = kModeAll; return bp; }
    const int need = bp - a.member_count[seq];
    mode = need > 0 ? kModeSelect : kModeNone;
    return need;
  }
  __device__ static void emit(const SelectArgs& a, int lz, int, int o0, int j, bool admitted, int pos, int limit) {
    if (admitted && (unsigned)pos < (unsigned)limit) a.idx[(int64_t)lz * a.TB + o0 + pos] = j;   // pos < limit always: belt and braces
  }
  __device__ static void window(const SelectArgs& a, int lz, int, int, int o0, int budget, int npre, int, int t) {
    a.idx[(int64_t)lz * a.TB + o0 + (budget - a.W) + t] = npre + t;
  }
};

__device__ __forceinline__ int parts_of(int npre) { return npre > kPartChunk ? (npre + kPartChunk - 1) / kPartChunk : 1; }

// Sum of one int over the workgroup (all threads call it; `slot` picks one of four scratch rows so that
// back-to-back calls need no barrier in between).
__device__ __forceinline__ int part_sum(PartShared& sh, int v, int slot) {
#pragma unroll
  for (int off = 32; off > 0; off >>= 1) v += __shfl_xor(v, off);
  if ((threadIdx.x & 63) == 0) sh.red[slot][threadIdx.x >> 6] = v;
  __syncthreads();
  int t = 0;
#pragma unroll
  for (int w = 0; w < kPartThreads / 64; ++w) t += sh.red[slot][w];
  return t;
}

// Exclusive prefix over the threads of the workgroup of two counts, and their totals (all threads call it).
__device__ __forceinline__ void part_scan2(PartShared& sh, int a, int b, int& before_a, int& before_b, int& tot_a, int& tot_b) {
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  int sa = a, sb = b;
#pragma unroll
  for (int off = 1; off < 64; off <<= 1) {
    const int oa = __shfl_up(sa, off), ob = __shfl_up(sb, off);
    if (lane >= off) { sa += oa; sb += ob; }
  }
  __syncthreads();                                 // the scratch rows may still be read from an earlier call
  if (lane == 63) { sh.red[0][wave] = sa; sh.red[1][wave] = sb; }
  __syncthreads();
  before_a = sa - a; before_b = sb - b; tot_a = 0; tot_b = 0;
#pragma unroll
  for (int w = 0; w < kPartThreads / 64; ++w) {
    if (w < wave) { before_a += sh.red[0][w]; before_b += sh.red[1][w]; }
    tot_a += sh.red[0][w]; tot_b += sh.red[1][w];
  }
}

// Which request and which of its parts workgroup `gp` of a launch works on; `first` = number of the request's first
// part.  All threads call it.  Up to 64 requests: every wave finds out by itself, one request a lane, without a barrier.
// More: every thread adds up the parts of a share of the requests, a prefix sum over the threads finds the share that
// holds gp, its owner walks it: four barriers before the first load of a candidate (16 problems of 131072 candidates,
// one request a call: counts 8.0 us with them, 7.1 without; near 11.2 and 10.9; emit 10.2 and 9.0).
__device__ __forceinline__ void locate_part(PartShared& sh, const int32_t* cu, int n_seqs, int W, int gp, int& seq, int& part, int& first) {
  const int tid = threadIdx.x;
  if (n_seqs <= 64) {
    const int lane = tid & 63;
    const int mine = lane < n_seqs ? parts_of(cu[lane + 1] - cu[lane] - W) : 0;
    const int end = (int)wave_scan((uint32_t)mine, OpAdd{});
    const uint64_t beyond = __ballot(gp < end);                     // never empty (grid = total parts)
    seq = beyond ? __builtin_ctzll(beyond) : n_seqs - 1;
    first = __builtin_amdgcn_readlane(end - mine, seq);
    part = gp - first;
    return;
  }
  const int per = (n_seqs + kPartThreads - 1) / kPartThreads;
  const int r0 = min(tid * per, n_seqs), r1 = min(r0 + per, n_seqs);
  int mine = 0;
  for (int r = r0; r < r1; ++r) mine += parts_of(cu[r + 1] - cu[r] - W);
  int before, dummy_b, total, dummy_t;
  part_scan2(sh, mine, 0, before, dummy_b, total, dummy_t);
  if (tid == 0) { sh.found[0] = n_seqs - 1; sh.found[1] = 0; }      // gp past the end never happens (grid = total parts)
  __syncthreads();
  if (gp >= before && gp < before + mine) {                         // exactly one thread
    int pos = before, r = r0;
    for (;; ++r) {
      const int np = parts_of(cu[r + 1] - cu[r] - W);
      if (gp < pos + np) break;
      pos += np;
    }
    sh.found[0] = r; sh.found[1] = pos;
  }
  __syncthreads();
  seq = sh.found[0]; first = sh.found[1]; part = gp - first;
  __syncthreads();                                                  // found[] and the scratch rows are reused
}

// Candidate in slot s of this thread: the part is cut into tiles of 4 * kPartThreads candidates, a thread holds 4
// consecutive candidates of every tile (the loads of a wave cover whole cache lines).
constexpr int kPartTile = 4 * kPartThreads;
constexpr int kPartTiles = kPartItems / 4;
__device__ __forceinline__ int part_index(int part, int s) {
  return part * kPartChunk + (s >> 2) * kPartTile + (int)threadIdx.x * 4 + (s & 3);
}

template <class Src>
__device__ __forceinline__ void part_load(const Src& src, int npre, int part, uint32_t (&keys)[kPartItems], unsigned& elig, unsigned& forc) {
  static_assert(kPartItems <= 32 && kPartItems % 4 == 0, "one flag bit per candidate, whole tiles");
  elig = 0; forc = 0;
  if (npre > 0) {
#pragma unroll
    for (int s = 0; s < kPartItems; ++s) {                          // unconditional, clamped: all loads in flight together
      const int j = part_index(part, s), jc = j < npre ? j : npre - 1;
      const uint32_t key = src.key(jc);
      const bool el = src.eligible(jc), fo = src.forced(jc);
      keys[s] = j < npre ? key : 0u;
      if (j < npre && el) elig |= 1u << s;
      if (j < npre && fo) forc |= 1u << s;
    }
  } else {
#pragma unroll
    for (int s = 0; s < kPartItems; ++s) keys[s] = 0u;
  }
}

// Places in token order.  In: per tile, a count (or two counts below 2^16 packed into the halves of a word) over this
// thread's 4 candidates of the tile.  Out: per tile, the same count(s) over all candidates of the part that come before
// them.  All threads call it.  The counts go through LDS as a [tile][thread] table, which is token order when read flat.
__device__ __forceinline__ void part_order(PartShared& sh, const unsigned int (&cnt)[kPartTiles], unsigned int (&before)[kPartTiles]) {
  unsigned int* table = sh.hist;                         // free at this point in both callers
  const int tid = threadIdx.x;
  __syncthreads();
#pragma unroll
  for (int t = 0; t < kPartTiles; ++t) table[t * kPartThreads + tid] = cnt[t];
  __syncthreads();
  unsigned int loc[kPartTiles], run = 0;
#pragma unroll
  for (int i = 0; i < kPartTiles; ++i) { loc[i] = run; run += table[tid * kPartTiles + i]; }
  int ba, bb, ta, tb;
  part_scan2(sh, (int)(run & 0xFFFFu), (int)(run >> 16), ba, bb, ta, tb);
  const unsigned int base = (unsigned int)ba | ((unsigned int)bb << 16);
#pragma unroll
  for (int i = 0; i < kPartTiles; ++i) table[tid * kPartTiles + i] = base + loc[i];
  __syncthreads();
#pragma unroll
  for (int t = 0; t < kPartTiles; ++t) before[t] = table[t * kPartThreads + tid];
  __syncthreads();
}

template <int NT = kPartThreads>
__device__ __forceinline__ void part_hist_clear(PartShared& sh, int nbins) {
  for (int b = threadIdx.x; b < (kPartCopies - 1) * kHistStride + nbins; b += NT) sh.hist[b] = 0;
  __syncthreads();
}

// counts: first digit of the part's competing candidates.  Every bin is stored, so nothing has to be cleared beforehand.
template <class Rule>
__global__ __launch_bounds__(kPartThreads) void part_counts_kernel(SelectArgs a, PartArgs c) {
  __shared__ PartShared sh;
  const int tid = threadIdx.x, gp = blockIdx.x, lz = blockIdx.y;
  int seq, part, first;
  locate_part(sh, a.cu_seqlens, a.n_seqs, a.W, gp, seq, part, first);
  const int s0 = a.cu_seqlens[seq];
  const int npre = a.cu_seqlens[seq + 1] - s0 - a.W;
  uint32_t keys[kPartItems];
  unsigned elig, forc;
  part_load(Rule::source(a, lz, s0), npre, part, keys, elig, forc);
  // A part holds at most kPartChunk < 2^16 candidates: two bins share a word, and there is room for 8 private copies
  // (lane % 8) of the table, which matters because the scores crowd into a few dozen bins.
  constexpr int COPIES = 8, STRIDE = kFirstDigitBins / 2 + 1;
  static_assert(COPIES * STRIDE <= kPartHistWords && kPartChunk < 65536, "packed first-digit counts");
  for (int b = tid; b < COPIES * STRIDE; b += kPartThreads) sh.hist[b] = 0;
  __syncthreads();
#pragma unroll
  for (int s = 0; s < kPartItems; ++s) {
    const uint32_t bin = keys[s] >> 21;
    if ((elig >> s) & 1u) atomicAdd(&sh.hist[(tid & (COPIES - 1)) * STRIDE + (bin >> 1)], 1u << (16 * (bin & 1u)));
  }
  __syncthreads();
  uint32_t* out = reinterpret_cast<uint32_t*>(c.hist + ((int64_t)lz * c.parts + gp) * kFirstDigitBins);
  for (int w = tid; w < kFirstDigitBins / 2; w += kPartThreads) {       // a sum below 2^16 per half: no carry between them
    unsigned int t = 0;
#pragma unroll
    for (int k = 0; k < COPIES; ++k) t += sh.hist[k * STRIDE + w];
    out[w] = t;
  }
}

// near: the bin that holds the cut, and the request's list of the candidates in that bin.
template <class Rule>
__global__ __launch_bounds__(kPartThreads) void part_near_kernel(SelectArgs a, PartArgs c) {
  __shared__ PartShared sh;
  const int tid = threadIdx.x, gp = blockIdx.x, lz = blockIdx.y;
  int seq, part, first;
  locate_part(sh, a.cu_seqlens, a.n_seqs, a.W, gp, seq, part, first);
  const int s0 = a.cu_seqlens[seq];
  const int npre = a.cu_seqlens[seq + 1] - s0 - a.W;
  const int budget = a.cu_budgets[seq + 1] - a.cu_budgets[seq];
  const int nparts = parts_of(npre);
  uint32_t keys[kPartItems];
  unsigned elig, forc;
  part_load(Rule::source(a, lz, s0), npre, part, keys, elig, forc);

  // counts of the 8 bins this thread owns (bins 8 * tid ...): over all parts of the request, in this part alone, and in the
  // parts before it (which say where this part's share of the list begins)
  constexpr int OWN = kFirstDigitBins / kPartThreads;
  static_assert(OWN == 8, "one 16-byte load per part and thread");
  unsigned int tot[OWN], own[OWN], early[OWN];
#pragma unroll
  for (int i = 0; i < OWN; ++i) { tot[i] = 0; own[i] = 0; early[i] = 0; }
  const uint16_t* hp = c.hist + ((int64_t)lz * c.parts + first) * kFirstDigitBins + tid * OWN;
  constexpr int BATCH = 8;                                // loads in flight
  for (int q0 = 0; q0 < nparts; q0 += BATCH) {
    uint4 v[BATCH];
#pragma unroll
    for (int u = 0; u < BATCH; ++u)
      v[u] = *reinterpret_cast<const uint4*>(hp + (int64_t)min(q0 + u, nparts - 1) * kFirstDigitBins);
#pragma unroll
    for (int u = 0; u < BATCH; ++u) {
      if (q0 + u >= nparts) continue;
      const unsigned int w[4] = {v[u].x, v[u].y, v[u].z, v[u].w};
#pragma unroll
      for (int i = 0; i < OWN; ++i) {
        const unsigned int x = (w[i >> 1] >> (16 * (i & 1))) & 0xFFFFu;
        tot[i] += x;
        if (q0 + u == part) own[i] = x;
        if (q0 + u < part) early[i] += x;
      }
    }
  }
  int mine = 0;
#pragma unroll
  for (int i = 0; i < OWN; ++i) mine += (int)tot[i];
  // candidates in the bins of higher threads (higher bins hold larger keys), and all competing candidates
  int below, dummy_b, total, dummy_t;
  part_scan2(sh, mine, 0, below, dummy_b, total, dummy_t);
  const int above = total - below - mine;
  int mode;
  const int need = Rule::need(a, seq, budget, npre, total, mode);
  if (tid == 0) { sh.found[0] = 0; sh.found[1] = 0; sh.found[2] = 0; sh.found[3] = 0; }
  __syncthreads();
  if (mode == kModeSelect && above < need && need <= above + mine) {   // exactly one thread: the cut lies in one of its bins
    int higher = above;
#pragma unroll
    for (int i = OWN - 1; i >= 0; --i) {
      if (higher < need && need <= higher + (int)tot[i]) {             // one bin of the 8
        sh.found[0] = tid * OWN + i; sh.found[1] = need - higher; sh.found[2] = (int)tot[i]; sh.found[3] = (int)early[i];
      }
      higher += (int)tot[i];
    }
  }
  __syncthreads();
  const int b0 = sh.found[0];
  if (part == 0 && tid == 0) {
    uint32_t* h = c.head + ((int64_t)lz * a.n_seqs + seq) * 8;
    h[0] = (uint32_t)mode; h[1] = (uint32_t)b0; h[2] = (uint32_t)sh.found[1]; h[3] = (uint32_t)sh.found[2];
    h[4] = (uint32_t)need;
  }
  // candidates of this part admitted whatever the cut: its bins above b0 (none when nothing is selected), forced ones
  int sure = __popc(forc);
  if (mode == kModeSelect) {
#pragma unroll
    for (int i = 0; i < OWN; ++i) sure += tid * OWN + i > b0 ? (int)own[i] : 0;
  }
  sure = part_sum(sh, sure, 2);
  if (tid == 0) c.sure[(int64_t)lz * c.parts + gp] = sure;
  if (mode != kModeSelect) return;                                     // the same for every thread
  const int off = sh.found[3];
  unsigned int cnt[kPartTiles], before[kPartTiles];
#pragma unroll
  for (int t = 0; t < kPartTiles; ++t) {
    cnt[t] = 0;
#pragma unroll
    for (int e = 0; e < 4; ++e) cnt[t] += ((elig >> (4 * t + e)) & 1u) && (int)(keys[4 * t + e] >> 21) == b0;
  }
  part_order(sh, cnt, before);
  uint32_t* list = c.list + (int64_t)lz * a.T + s0 + off;              // at most npre entries per request: inside its tokens
#pragma unroll
  for (int t = 0; t < kPartTiles; ++t) {
    unsigned int pos = before[t];
#pragma unroll
    for (int e = 0; e < 4; ++e)
      if (((elig >> (4 * t + e)) & 1u) && (int)(keys[4 * t + e] >> 21) == b0) list[pos++] = keys[4 * t + e];
  }
}

// One more digit of the radix select over the request's list (all NT threads of the workgroup call it).  Entries whose
// bits above the digit equal `prefix` take part; afterwards `prefix` has the digit filled in and `remaining` is the
// rank inside it.
template <int NT>
__device__ __forceinline__ void part_digit(PartShared& sh, const uint32_t* list, int m, int shift, int nbins, uint32_t himask,
                                           uint32_t& prefix, uint32_t& remaining) {
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  part_hist_clear<NT>(sh, nbins);
  constexpr int UNR = 8;                                  // loads in flight per thread
  for (int i0 = tid; i0 < m; i0 += NT * UNR) {
    uint32_t k[UNR];
#pragma unroll
    for (int u = 0; u < UNR; ++u) k[u] = list[min(i0 + u * NT, m - 1)];
#pragma unroll
    for (int u = 0; u < UNR; ++u)
      if (i0 + u * NT < m && (k[u] & himask) == prefix)
        atomicAdd(&sh.hist[(tid & (kPartCopies - 1)) * kHistStride + ((k[u] >> shift) & (uint32_t)(nbins - 1))], 1u);
  }
  __syncthreads();
  for (int b = tid; b < nbins; b += NT) {
    unsigned int t = 0;
#pragma unroll
    for (int k = 0; k < kPartCopies; ++k) t += sh.hist[k * kHistStride + b];
    sh.hist[b] = t;
  }
  __syncthreads();
  if (wave == 0) {                       // lane owns bins [lane * per, lane * per + per); higher bins hold larger keys
    const int per = nbins / 64;
    unsigned int mine = 0;
    for (int i = 0; i < per; ++i) mine += sh.hist[lane * per + i];
    unsigned int run = mine;             // inclusive suffix sum over lanes
#pragma unroll
    for (int off = 1; off < 64; off <<= 1) {
      const unsigned int o = __shfl_down(run, off);
      if (lane + off < 64) run += o;
    }
    const unsigned int above = run - mine;
    if (above < remaining && remaining <= above + mine) {        // exactly one lane
      unsigned int higher = above;
      for (int i = per - 1; i >= 0; --i) {
        const unsigned int cbin = sh.hist[lane * per + i];
        if (remaining <= higher + cbin) { sh.prefix = prefix | ((uint32_t)(lane * per + i) << shift); sh.need = remaining - higher; break; }
        higher += cbin;
      }
    }
  }
  __syncthreads();
  prefix = sh.prefix;
  remaining = sh.need;
  __syncthreads();
}

// resolve: one workgroup per problem finds the cut in the request's list and leaves its key and the number of candidates
// tied at it that are admitted.  A list of up to 16384 keys stays in registers and takes the counting rounds of the
// one-workgroup selection (find_cut): a prior that puts every marked token into one bin of the first digit leaves thousands
// of keys, most of them equal in the next digit too, whose LDS atomics then wait for one another.  Longer lists take two
// more radix digits.
// Bound by a chain of latencies in one workgroup, so what does not need the cut goes before it, with its loads beside the
// list's: where each part's stretch of the list ends, and which part each of a wave's reads begins in.  Counting per part
// then takes the keys from the registers that still hold them (16 problems of 131072 candidates, 13107 of them marked and in
// one bin: 16.5 -> 14.2 us).
constexpr int kResolveThreads = 1024;     // the list is read with 8 loads in flight per thread: many threads, few rounds
constexpr int kResolveItems = 16;
__global__ __launch_bounds__(kResolveThreads) void part_resolve_kernel(SelectArgs a, PartArgs c) {
  __shared__ PartShared sh;
  __shared__ SelectShared<kResolveThreads> cut;
  __shared__ unsigned int table[kPartHistWords];
  const int seq = blockIdx.x, lz = blockIdx.y;
  uint32_t* h = c.head + ((int64_t)lz * a.n_seqs + seq) * 8;
  const int s0 = a.cu_seqlens[seq];
  const int npre = a.cu_seqlens[seq + 1] - s0 - a.W;
  if ((int)h[0] != kModeSelect) return;                      // the same for every thread
  const uint32_t* list = c.list + (int64_t)lz * a.T + s0;
  const int b0 = (int)h[1], m = (int)h[3];
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const bool held = m <= kResolveThreads * kResolveItems;    // the same for every thread
  uint32_t keys[kResolveItems];
  if (held) {
    const rsrc_t row = row_of(list, m);
#pragma unroll
    for (int s = 0; s < kResolveItems; ++s)                  // past the list: 0, no candidate
      keys[s] = (uint32_t)__builtin_amdgcn_raw_buffer_load_b32(row, (s * kResolveThreads + tid) * 4, 0, 0);
  }
  // How many list entries of each part lie above the cut / are tied at it, as running totals over the parts: an
  // emitting part then knows what the earlier parts contribute without reading their stretch of the list again.
  const int nparts = parts_of(npre);
  const bool fits = 3 * nparts <= kPartHistWords;            // else the emitting parts count for themselves
  unsigned int* seg_end = table;                             // end of each part's stretch of the list
  unsigned int* n_above = table + nparts;
  unsigned int* n_tied = table + 2 * nparts;
  int first = 0;                                             // number of this request's first part
  // running totals over the parts, 64 at a time, by one wave
  auto running = [&](unsigned int* v, bool exclusive) __attribute__((always_inline)) {
    unsigned int carry = 0;
    for (int base = 0; base < nparts; base += 64) {
      const unsigned int x = base + lane < nparts ? v[base + lane] : 0u;
      unsigned int incl = x;
#pragma unroll
      for (int off = 1; off < 64; off <<= 1) {
        const unsigned int o = __shfl_up(incl, off);
        if (lane >= off) incl += o;
      }
      if (base + lane < nparts) v[base + lane] = carry + (exclusive ? incl - x : incl);
      carry += __shfl(incl, 63);
    }
  };
  if (fits) {                                                // the same for every thread
    if (seq > 0) {
      int mine = 0;
      for (int r = tid; r < seq; r += kResolveThreads) mine += parts_of(a.cu_seqlens[r + 1] - a.cu_seqlens[r] - a.W);
#pragma unroll
      for (int off = 32; off > 0; off >>= 1) mine += __shfl_xor(mine, off);
      if (lane == 0) sh.red[0][wave] = mine;
      __syncthreads();
#pragma unroll
      for (int w = 0; w < kResolveThreads / 64; ++w) first += sh.red[0][w];
    }
    for (int q = tid; q < nparts; q += kResolveThreads) {
      seg_end[q] = c.hist[((int64_t)lz * c.parts + first + q) * kFirstDigitBins + b0];
      n_above[q] = 0; n_tied[q] = 0;
    }
    __syncthreads();
    if (wave == 0) running(seg_end, false);
    __syncthreads();
  }
  auto part_of_entry = [&](int i) __attribute__((always_inline)) {      // first part whose stretch ends beyond entry i
    int lo = 0, hi = nparts - 1;
    while (lo < hi) {
      const int mid = (lo + hi) >> 1;
      if (seg_end[mid] > (unsigned int)i) hi = mid; else lo = mid + 1;
    }
    return lo;
  };
  // A wave's reads lie kResolveThreads entries apart: lane u looks up the part that its read u (of 64) begins in.
  int begins = fits && held ? part_of_entry(min(lane * kResolveThreads + wave * 64, m - 1)) : 0;
  uint32_t tau = (uint32_t)b0 << 21, remaining = h[2];
  if (held) {
    const int slots = ((m + kResolveThreads - 1) / kResolveThreads + 3) / 4 * 4;
    int ties;
    find_cut<kResolveThreads, kResolveItems>(cut, keys, slots, m, remaining, tau, ties);
    remaining = (uint32_t)ties;
  } else {
    part_digit<kResolveThreads>(sh, list, m, 10, 2048, 0xFFE00000u, tau, remaining);
    part_digit<kResolveThreads>(sh, list, m, 0, 1024, 0xFFFFFC00u, tau, remaining);
  }
  if (tid == 0) { h[5] = tau; h[6] = remaining; h[7] = fits ? 1u : 0u; }
  if (!fits) return;                                         // the same for every thread
  // The 64 entries of a read follow one another, so most of the time one part holds all of them: one round, two additions.
  auto count_read = [&](int i0, int part, uint32_t key) __attribute__((always_inline)) {
    const int end = min(i0 + 64, m);
    const uint64_t above = __ballot(i0 + lane < m && key > tau), tied = __ballot(i0 + lane < m && key == tau);
    for (int lo = i0; lo < end && part < nparts; ++part) {
      const int hi = min((int)__builtin_amdgcn_readfirstlane((int)seg_end[part]), end);
      if (hi <= lo) continue;                                // a part without entries in the list
      const uint64_t of_part = (~0ull >> (64 - (hi - lo))) << (lo - i0);
      const int na = __popcll(above & of_part), nt = __popcll(tied & of_part);
      if (lane == 0 && na > 0) atomicAdd(&n_above[part], (unsigned int)na);
      if (lane == 0 && nt > 0) atomicAdd(&n_tied[part], (unsigned int)nt);
      lo = hi;
    }
  };
  if (held) {
#pragma unroll
    for (int s = 0; s < kResolveItems; ++s) {
      const int i0 = s * kResolveThreads + wave * 64;
      if (i0 < m) count_read(i0, __builtin_amdgcn_readlane(begins, s), keys[s]);
    }
  } else {
    constexpr int UNR = 8;
    for (int w0 = wave * 64; w0 < m; w0 += kResolveThreads * UNR) {
      uint32_t k[UNR];
#pragma unroll
      for (int u = 0; u < UNR; ++u) k[u] = list[min(w0 + lane + u * kResolveThreads, m - 1)];
      begins = part_of_entry(min(w0 + (lane & (UNR - 1)) * kResolveThreads, m - 1));
#pragma unroll
      for (int u = 0; u < UNR; ++u) {
        const int i0 = w0 + u * kResolveThreads;
        if (i0 < m) count_read(i0, __builtin_amdgcn_readlane(begins, u), k[u]);
      }
    }
  }
  __syncthreads();
  if (wave == 0) running(n_above, true);
  if (wave == 1) running(n_tied, true);
  __syncthreads();
  for (int q = tid; q < nparts; q += kResolveThreads) {
    int32_t* out = c.before + ((int64_t)lz * c.parts + first + q) * 2;
    out[0] = (int32_t)n_above[q]; out[1] = (int32_t)n_tied[q];
  }
}

// emit: every part writes its admitted candidates at their final places.
template <class Rule>
__global__ __launch_bounds__(kPartThreads) void part_emit_kernel(SelectArgs a, PartArgs c) {
  __shared__ PartShared sh;
  const int tid = threadIdx.x, gp = blockIdx.x, lz = blockIdx.y;
  int seq, part, first;
  locate_part(sh, a.cu_seqlens, a.n_seqs, a.W, gp, seq, part, first);
  const int s0 = a.cu_seqlens[seq];
  const int npre = a.cu_seqlens[seq + 1] - s0 - a.W;
  const int o0 = a.cu_budgets[seq];
  const int budget = a.cu_budgets[seq + 1] - o0;
  uint32_t keys[kPartItems];
  unsigned elig, forc;
  part_load(Rule::source(a, lz, s0), npre, part, keys, elig, forc);
  int sure_before = 0;                                       // asked for beside the candidates
  for (int q = tid; q < part; q += kPartThreads) sure_before += c.sure[(int64_t)lz * c.parts + first + q];
  const uint32_t* h = c.head + ((int64_t)lz * a.n_seqs + seq) * 8;
  const int mode = (int)h[0], b0 = (int)h[1], need = (int)h[4];
  if (part == 0)
    for (int t = tid; t < a.W; t += kPartThreads) Rule::window(a, lz, seq, s0, o0, budget, npre, need, t);
  if (mode == kModeAll) {                                    // every candidate is kept at its own place
#pragma unroll
    for (int s = 0; s < kPartItems; ++s) {
      const int j = part_index(part, s);
      if (j < npre) Rule::emit(a, lz, s0, o0, j, true, j, budget - a.W);
    }
    return;
  }
  uint32_t tau = 0xFFFFFFFFu;
  int ties = 0, above_before = 0, ties_before = 0;
  if (mode == kModeSelect) {
    const uint32_t* list = c.list + (int64_t)lz * a.T + s0;
    tau = h[5];
    ties = (int)h[6];
    if (h[7] != 0u) {                                     // the resolve kernel has counted for every part
      const int32_t* bf = c.before + ((int64_t)lz * c.parts + gp) * 2;
      above_before = bf[0];
      ties_before = bf[1];
    } else {
      int ab = 0, tb = 0;
      // what the earlier parts hold of the list: their entries come first
      int off = 0;
      for (int q = tid; q < part; q += kPartThreads) off += c.hist[((int64_t)lz * c.parts + first + q) * kFirstDigitBins + b0];
      off = part_sum(sh, off, 2);
      constexpr int UNR = 8;
      for (int i0 = tid; i0 < off; i0 += kPartThreads * UNR) {
        uint32_t k[UNR];
#pragma unroll
        for (int u = 0; u < UNR; ++u) k[u] = list[min(i0 + u * kPartThreads, off - 1)];
#pragma unroll
        for (int u = 0; u < UNR; ++u)
          if (i0 + u * kPartThreads < off) { ab += k[u] > tau; tb += k[u] == tau; }
      }
      __syncthreads();
      above_before = part_sum(sh, ab, 3);
      __syncthreads();
      ties_before = part_sum(sh, tb, 2);
      __syncthreads();
    }
  }
  sure_before = part_sum(sh, sure_before, 3) + above_before;
  // classes of this thread's candidates: in whatever the cut / tied at the cut / out
  unsigned in2 = 0, in1 = 0;
  unsigned int cnt[kPartTiles], before[kPartTiles];
#pragma unroll
  for (int s = 0; s < kPartItems; ++s) {
    const bool el = (elig >> s) & 1u, fo = (forc >> s) & 1u;
    const bool two = fo || (el && mode == kModeSelect && keys[s] > tau);
    const bool one = !fo && el && mode == kModeSelect && keys[s] == tau;
    if (two) in2 |= 1u << s;
    if (one) in1 |= 1u << s;
  }
#pragma unroll
  for (int t = 0; t < kPartTiles; ++t) cnt[t] = __popc((in2 >> (4 * t)) & 15u) | (__popc((in1 >> (4 * t)) & 15u) << 16);
  part_order(sh, cnt, before);
#pragma unroll
  for (int t = 0; t < kPartTiles; ++t) {
    int ps = sure_before + (int)(before[t] & 0xFFFFu), pt = ties_before + (int)(before[t] >> 16);
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      const int s = 4 * t + e, j = part_index(part, s);
      const bool two = (in2 >> s) & 1u, one = (in1 >> s) & 1u;
      if (j < npre) Rule::emit(a, lz, s0, o0, j, two || (one && pt < ties), ps + min(pt, ties), budget - a.W);
      ps += two; pt += one;
    }
  }
}

// Calls launch(threads, candidates per thread) for requests of at most `longest` candidates.  Few problems: a workgroup has
// its compute unit to itself, and many threads with few candidates each are quickest (8192 tokens: 7.7 us with 1024 x 8 against
// 10.5 with 512 x 16; 4093: 6.1 with 1024 x 4 against 9.4 with 256 x 16; 2048: 4.6 with 512 x 4 against 6.8 with 1024 x 8).
// Many problems: smaller workgroups, of which several share a compute unit, spend less on barriers and on work that every
// wave repeats (7168 problems of 135 .. 1831 tokens: 31 us with 256 x 8; of 142 .. 2313: 54 with 256 x 16).
template <class Launch>
static void dispatch_items(int longest, int64_t problems, Launch launch) {
  auto with = [&](auto nt, auto items) { launch(nt, items); };
#define CODECOMP_WG(NT, ITEMS) if (longest <= NT * ITEMS) return with(std::integral_constant<int, NT>{}, std::integral_constant<int, ITEMS>{});
  if (problems >= kSelectManyProblems) {
    CODECOMP_WG(256, 8) CODECOMP_WG(256, 16) CODECOMP_WG(512, 16) CODECOMP_WG(512, 32)
  } else {
    CODECOMP_WG(256, 4) CODECOMP_WG(512, 4) CODECOMP_WG(1024, 4) CODECOMP_WG(1024, 8) CODECOMP_WG(1024, 16)
  }
  CODECOMP_WG(1024, 32) CODECOMP_WG(1024, 48)
  with(std::integral_constant<int, 1024>{}, std::integral_constant<int, 64>{});
#undef CODECOMP_WG
}

static PartArgs part_args(const Plan& pl, void* workspace) {
  char* ws = static_cast<char*>(workspace);
  PartArgs c;
  c.hist = reinterpret_cast<uint16_t*>(ws + pl.off_part_hist);
  c.sure = reinterpret_cast<int32_t*>(ws + pl.off_part_sure);
  c.head = reinterpret_cast<uint32_t*>(ws + pl.off_part_head);
  c.list = reinterpret_cast<uint32_t*>(ws + pl.off_uraw);       // the raw attention mass is dead once the scores exist
  c.before = reinterpret_cast<int32_t*>(ws + pl.off_part_before);
  c.parts = pl.sel_parts;
  return c;
}

template <class Rule>
static int launch_parts(const Plan& pl, const SelectArgs& a, const PartArgs& c, int lzs, hipStream_t stream) {
  const dim3 grid(pl.sel_parts, lzs), block(kPartThreads);
  part_counts_kernel<Rule><<<grid, block, 0, stream>>>(a, c);
  if (hipError_t e = hipGetLastError()) return (int)e;
  part_near_kernel<Rule><<<grid, block, 0, stream>>>(a, c);
  if (hipError_t e = hipGetLastError()) return (int)e;
  part_resolve_kernel<<<dim3(pl.n_seqs, lzs), dim3(kResolveThreads), 0, stream>>>(a, c);
  if (hipError_t e = hipGetLastError()) return (int)e;
  part_emit_kernel<Rule><<<grid, block, 0, stream>>>(a, c);
  if (hipError_t e = hipGetLastError()) return (int)e;
  return 0;
}

static SelectArgs select_args(const Plan& pl, const float* scores, const float* prior, int32_t* idx, void* workspace) {
  char* ws = static_cast<char*>(workspace);
  SelectArgs a = {};
  a.scores = scores; a.prior = prior; a.cu_seqlens = pl.cu_seqlens_dev; a.cu_budgets = pl.cu_budgets_dev; a.idx = idx;
  a.member = reinterpret_cast<uint8_t*>(ws + pl.off_member);
  a.member_count = reinterpret_cast<int32_t*>(ws + pl.off_member_count);
  a.n_seqs = pl.n_seqs; a.T = pl.T; a.TB = pl.TB; a.W = pl.W;
  a.span_ratio = pl.span_ratio; a.span_min = pl.span_min;
  return a;
}

static int launch_stage1(const Plan& pl, const SelectArgs& a, hipStream_t stream) {
  dispatch_items(pl.max_n - pl.W, (int64_t)pl.n_seqs, [&](auto nt, auto items) {
    select_stage1_kernel<nt(), items()><<<dim3(pl.n_seqs), dim3(nt()), 0, stream>>>(a);
  });
  if (hipError_t e = hipGetLastError()) return (int)e;
  return 0;
}

// One workgroup keeps a request's scores in registers (64 per thread of the large ones), if pooling leaves the fused kernel ahead.
// Up to nine neighbours it does, at every size.  Wider ones are read from LDS one by one, by the one compute unit that has the
// request (at about 24 tokens' reads of one neighbour per ns), where the pooling kernel spreads them over the device, for the
// price of a launch and a trip of the scores through memory (about 7 us).  So the fused kernel takes them while the neighbours
// that its busiest unit reads beyond an even share (of which the pooling kernel's halos and edges take back a quarter) cost less
// than that.  Separate -> fused: 4 problems of 4096 tokens, width 33 30.6 -> 28.4 us, 65 30.5 -> 34.0; of 8192, 13 30.7 -> 29.6,
// 25 30.4 -> 33.7; of 16384, 9 34.8 -> 34.1, 11 35.0 -> 39.2; of 65536, 1025 147 -> 2756;
// 256 of 4096, 129 113 -> 89; 256 of 32768, 25 595 -> 588, 129 675 -> 723; 1792 of 1000, 65 142 -> 131.
bool fused_tail(const Plan& pl) {
  constexpr int64_t kUnits = 256, kWideReads = 160000;
  if (pl.max_n > kSelectMaxCandidates) return false;
  if (pl.pool <= 2 * kFinishNear + 1) return true;
  const int64_t even = (int64_t)pl.L * pl.Hkv * pl.T / kUnits, busiest = even > pl.max_n ? even : pl.max_n;
  return pl.pool * (busiest - even * 3 / 4) <= kWideReads;
}

// Requests that keep little: the workgroup that selects the rows copies them too, and a launch is saved.
bool fused_copy(const Plan& pl) {
  const int64_t bytes = (int64_t)pl.max_b * pl.d * (pl.kv_fp8 ? 1 : 2) * 2;
  return fused_tail(pl) && bytes <= kCopyBytes;
}

int launch_finish_select(const Plan& pl, const float* prior, float* scores, int32_t* idx, const void* k, const void* v, void* k_out,
                         void* v_out, void* workspace, hipStream_t stream) {
  const SelectArgs a = select_args(pl, scores, prior, idx, workspace);
  const FinishArgs f = finish_args(pl, prior, scores, workspace);
  const GatherArgs g = gather_args(pl, k, v, idx, k_out, v_out);
  const bool fill = pl.select_mode == CODECOMP_SELECT_TWO_STAGE, copy = fused_copy(pl);
  if (fill)
    if (int rc = launch_stage1(pl, a, stream)) return rc;
  dispatch_items(pl.max_n, (int64_t)pl.n_seqs * pl.L * pl.Hkv, [&](auto nt, auto items) {
    const dim3 grid(pl.n_seqs, pl.L * pl.Hkv), block(nt());
    auto go = [&](auto filled, auto copied) {
      finish_select_kernel<filled(), nt(), items(), kFinishHalo, copied()><<<grid, block, 0, stream>>>(a, f, g);
    };
    if (copy) { if (fill) go(std::true_type{}, std::true_type{}); else go(std::false_type{}, std::true_type{}); }
    else { if (fill) go(std::true_type{}, std::false_type{}); else go(std::false_type{}, std::false_type{}); }
  });
  if (hipError_t e = hipGetLastError()) return (int)e;
  return 0;
}

int launch_select(const Plan& pl, const float* scores, int32_t* idx, void* workspace, hipStream_t stream) {
  const SelectArgs a = select_args(pl, scores, nullptr, idx, workspace);
  if (pl.sel_parts > 0) return launch_parts<RuleAdditive>(pl, a, part_args(pl, workspace), pl.L * pl.Hkv, stream);
  dispatch_items(pl.max_n - pl.W, (int64_t)pl.n_seqs * pl.L * pl.Hkv, [&](auto nt, auto items) {
    select_kernel<false, nt(), items()><<<dim3(pl.n_seqs, pl.L * pl.Hkv), dim3(nt()), 0, stream>>>(a);
  });
  if (hipError_t e = hipGetLastError()) return (int)e;
  return 0;
}

int launch_select_two_stage(const Plan& pl, const float* scores, const float* prior, int32_t* idx, void* workspace,
                            hipStream_t stream) {
  const SelectArgs a = select_args(pl, scores, prior, idx, workspace);
  if (pl.sel_parts > 0) {
    const PartArgs c = part_args(pl, workspace);
    if (int rc = launch_parts<RuleStage1>(pl, a, c, 1, stream)) return rc;
    return launch_parts<RuleStage2>(pl, a, c, pl.L * pl.Hkv, stream);
  }
  if (int rc = launch_stage1(pl, a, stream)) return rc;
  dispatch_items(pl.max_n - pl.W, (int64_t)pl.n_seqs * pl.L * pl.Hkv, [&](auto nt, auto items) {
    select_kernel<true, nt(), items()><<<dim3(pl.n_seqs, pl.L * pl.Hkv), dim3(nt()), 0, stream>>>(a);
  });
  if (hipError_t e = hipGetLastError()) return (int)e;
  return 0;
}

}  // namespace codecomp
