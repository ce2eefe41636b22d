// Score step, small kernels and entry: row merge between the two MFMA passes, pooling + prior, and the
// launch sequence.  The passes themselves live in score_pass.h and are instantiated per (head_dim, key
// type) in score_pass_*.hip.
#include "score_team.h"

namespace codecomp {

extern template int dispatch_waves<128, false>(const Plan&, const ScoreArgs&, hipStream_t, unsigned);
extern template int dispatch_waves<128, true>(const Plan&, const ScoreArgs&, hipStream_t, unsigned);
extern template int dispatch_waves<64, false>(const Plan&, const ScoreArgs&, hipStream_t, unsigned);
extern template int dispatch_waves<64, true>(const Plan&, const ScoreArgs&, hipStream_t, unsigned);
extern template int launch_team<128, false>(const Plan&, const ScoreArgs&, char*, hipStream_t);
extern template int launch_team<128, true>(const Plan&, const ScoreArgs&, char*, hipStream_t);
extern template bool team_fits<128, false>(const Plan&);
extern template bool team_fits<128, true>(const Plan&);
extern template int launch_once<128, false>(const Plan&, const ScoreArgs&, hipStream_t);
extern template int launch_rows<128, false>(const Plan&, const ScoreArgs&, hipStream_t);
extern template int launch_once<128, true>(const Plan&, const ScoreArgs&, hipStream_t);
extern template int launch_rows<128, true>(const Plan&, const ScoreArgs&, hipStream_t);
extern template int launch_once<64, false>(const Plan&, const ScoreArgs&, hipStream_t);
extern template int launch_rows<64, false>(const Plan&, const ScoreArgs&, hipStream_t);
extern template int launch_once<64, true>(const Plan&, const ScoreArgs&, hipStream_t);
extern template int launch_rows<64, true>(const Plan&, const ScoreArgs&, hipStream_t);

// Per (layer*head, request, row): log2-sum-exp over the segments (of the teams) that cover the request and over the (at
// most two) wave slots that hold a share of the row's keys.
// Bound by memory round trips, not by bytes: `ways` threads (a power of two, at most 16) share the segments of a row, each
// asks for four of them at once, and their sums meet in LDS.  Kernel time with one thread per row that walks the segments
// one after the other -> now: 2 layers of 8192 tokens (33 segments a row, 16 ways) 19.0 -> 4.7 us; one layer of 4093 tokens
// (W 128) 10.7 -> 4.2; 4 layers of 20011 tokens 11.9 -> 4; 7168 problems (one way) 38.6 -> 38.9.
constexpr int kMergeThreads = 256, kMergeMaxWays = 16;

__global__ __launch_bounds__(kMergeThreads) void score_merge_kernel(ScoreArgs a, int ways_log2) {
  __shared__ int part[kMergeThreads / 64];
  __shared__ float2 sums[kMergeThreads];
  const int tid = threadIdx.x;
  const int seq = blockIdx.y;
  const int lz = blockIdx.z;
  // One value of each cache line of arguments, all asked for at once: left to their uses, the later ones wait for the request's bounds
  // (4 layers of 20011 tokens: 5.05 -> 4.72 us).  Not volatile: the compiler would no longer trust the bounds to stay as they are.
  int lead = a.lead;
  asm("" : "+s"(lead) : "s"(a.stat_teams), "s"(a.rb_holder[0]), "s"(ways_log2));
  const TileRule rule = {a.key_trim, a.once_keys, lead};
  const int nt = tiles_of(a.cu_seqlens[seq + 1] - a.cu_seqlens[seq], rule);
  if (nt < 0) return;            // the one-pass kernel's: nothing reads its normalisers
  int tile_off = lead;
  if (a.n_seqs > 1) {            // positions of the earlier requests in a problem's sequence: summed by the whole workgroup
    int mine = 0;
    for (int r = tid; r < seq; r += kMergeThreads) mine += lead + tiles_of(a.cu_seqlens[r + 1] - a.cu_seqlens[r], rule);
#pragma unroll
    for (int off = 32; off > 0; off >>= 1) mine += __shfl_xor(mine, off);
    if ((tid & 63) == 0) part[tid >> 6] = mine;
    __syncthreads();
    tile_off += part[0] + part[1] + part[2] + part[3];
  }
  const int x0 = lz * a.tiles_per_problem + tile_off;
  const int g0 = wg_of_tile(x0, a.total_tiles, a.stat_teams);
  const int segments = nt == 0 ? 0 : wg_of_tile(x0 + nt - 1, a.total_tiles, a.stat_teams) - g0 + 1;
  const int p = lz * a.n_seqs + seq;
  const int ways = 1 << ways_log2, rows_per = kMergeThreads >> ways_log2;
  const int way = tid / rows_per, row_in = tid & (rows_per - 1);
  // a launch with many problems has one workgroup per problem (the rows in turns), else one per rows_per rows
  for (int row0 = blockIdx.x * rows_per; row0 < a.lrows; row0 += gridDim.x * rows_per) {
    const int row = row0 + row_in;
    float M = NEG_BIG, L = 0.f;
    if (row < a.lrows) {
      const int split = row / (a.nb * 32);
      const int rb = (row - split * a.nb * 32) >> 5;
      const int h0 = (int)(a.rb_holder[rb] & 255u), h1 = (int)(a.rb_holder[rb] >> 8);
      const int two = h1 != 255 ? 1 : 0;
      const int items = segments << two;           // (segment, holder) pairs of this row
      // the segment of team g in this problem and row split sits in slot (g + p) * row_splits + split
      const float2* st = reinterpret_cast<const float2*>(a.stats) + ((int64_t)(p + g0) * a.row_splits + split) * a.srows + (row & 31);
      const int64_t slot = (int64_t)a.row_splits * a.srows;
      for (int i = way; i < items; i += ways * kMergeBatch) {
        float2 s[kMergeBatch];
#pragma unroll
        for (int u = 0; u < kMergeBatch; ++u) {
          const int at = min(i + u * ways, items - 1);
          s[u] = st[(at >> two) * slot + ((at & two) ? h1 : h0) * 32];
        }
        float Mn = M;
#pragma unroll
        for (int u = 0; u < kMergeBatch; ++u) {
          if (i + u * ways >= items) s[u] = make_float2(NEG_BIG, 0.f);
          Mn = fmaxf(Mn, s[u].x);
        }
        L *= __builtin_amdgcn_exp2f(M - Mn);
#pragma unroll
        for (int u = 0; u < kMergeBatch; ++u) L += s[u].y * __builtin_amdgcn_exp2f(s[u].x - Mn);
        M = Mn;
      }
    }
    if (ways > 1) {
      sums[tid] = make_float2(M, L);
      __syncthreads();
      if (way == 0) {
        float Mn = M;
        for (int w = 1; w < ways; ++w) Mn = fmaxf(Mn, sums[w * rows_per + row_in].x);
        L *= __builtin_amdgcn_exp2f(M - Mn);
        for (int w = 1; w < ways; ++w) {
          const float2 o = sums[w * rows_per + row_in];
          L += o.y * __builtin_amdgcn_exp2f(o.x - Mn);
        }
        M = Mn;
      }
      __syncthreads();                             // the next rows reuse the places
    }
    // a request without a key to attend to: nothing reads this normaliser
    if (way == 0 && row < a.lrows) a.lse[(int64_t)p * a.lrows + row] = segments == 0 ? 0.f : M + log2f(L);
  }
}

// A workgroup of the finish kernel takes 256 * PER tokens.  It is a chain of latencies (bounds, masses, barrier, a sum over
// neighbours per token), so few problems take short ones that fill the device: from 512 workgroups of 2048 tokens on (one round
// or more of them) the long ones, which share the loads at the edges.  4 layers of 20011 tokens: 10.6 us as 160 workgroups of
// 2048 tokens, 4.8 as 640 of 512.
constexpr int kFinishLong = 8, kFinishShort = 2, kFinishFill = 512;

__device__ __forceinline__ int request_of(const int32_t* cu, int n_seqs, int j) {
  int lo = 0, hi = n_seqs;              // cu[lo] <= j < cu[lo+1]
  while (hi - lo > 1) {
    const int mid = (lo + hi) >> 1;
    if (cu[mid] <= j) lo = mid; else hi = mid;
  }
  return lo;
}

// scores[lz][j] = pool_{|delta| <= (k-1)/2, inside the request (or its prefix)} u[lz][j+delta] + lambda * prior[j],
// pool = sum / k (zero padding, divisor always k) or max.
// One workgroup stages its tokens of u (+ halo, row splits added) in LDS; every output is a direct sum.
// Everything that comes from memory (request bounds, prior, u) is asked for before the one barrier, so
// that a workgroup pays one memory round trip.  A tile that lies inside one request (the common case)
// takes that request's bounds once; otherwise every token looks its request up.
template <int PER>
__global__ __launch_bounds__(256) void score_finish_kernel(FinishArgs a) {
  constexpr int kTokens = 256 * PER;
  __shared__ float tile[kTokens + 2 * kFinishHalo];
  const int tid = threadIdx.x;
  const int lz = blockIdx.y;
  const int base = blockIdx.x * kTokens;
  const int half = (a.pool - 1) >> 1;
  const int last = min(base + kTokens, a.T) - 1;
  const int r_first = request_of(a.cu_seqlens, a.n_seqs, base), r_last = request_of(a.cu_seqlens, a.n_seqs, last);
  const bool one_request = r_first == r_last;
  int lo_[PER], hi_[PER];               // request bounds [lo, hi) of each of this thread's tokens
  float pr[PER];
  // A tile that meets fewer than 64 requests: every wave takes their upper bounds into one register (lane q: request
  // r_first + q) and each token counts the bounds at or below it - one load per wave instead of a binary search per token.
  const bool few_requests = !one_request && r_last - r_first < 64;
  const int bound = few_requests ? a.cu_seqlens[min(r_first + 1 + (tid & 63), a.n_seqs)] : 0;
  const int first_lo = a.cu_seqlens[r_first];
#pragma unroll
  for (int e = 0; e < PER; ++e) {
    const int j = base + e * 256 + tid;
    if (few_requests) {
      int k = 0;                          // requests of the tile that end at or before token j
      if (j < a.T)
        for (int q = 0; q < r_last - r_first; ++q) k += j >= __builtin_amdgcn_readlane(bound, q);
      hi_[e] = __shfl(bound, k);
      const int below = __shfl(bound, max(k - 1, 0));       // every lane takes part: a lane reads from lanes that are not in its request
      lo_[e] = k == 0 ? first_lo : below;
    } else {
      const int r = one_request || j >= a.T ? r_first : request_of(a.cu_seqlens, a.n_seqs, j);
      lo_[e] = a.cu_seqlens[r]; hi_[e] = a.cu_seqlens[r + 1];
    }
    pr[e] = j < a.T ? a.prior[j] : 0.f;
  }
  // the tile's own tokens: PER independent loads per thread (per row split), all in flight together
  float body[PER];
#pragma unroll
  for (int e = 0; e < PER; ++e) body[e] = 0.f;
  for (int sp = 0; sp < a.row_splits; ++sp) {
    const float* u = a.uraw + ((int64_t)sp * a.LH + lz) * a.T;
#pragma unroll
    for (int e = 0; e < PER; ++e) {
      const int j = base + e * 256 + tid;
      // the load does not wait for the request bounds (clamped: always in bounds); window positions were never
      // written by the mass pass when the softmax leaves them out, whatever they hold is dropped
      const float val = u[min(j, a.T - 1)];
      body[e] += j < min(a.T, hi_[e] - a.mass_trim) ? val : 0.f;
    }
  }
  // the halo on both sides: 2 * half tokens that belong to the neighbouring tiles
  for (int i = tid; i < 2 * half; i += 256) {
    const int x = i < half ? base - half + i : base + kTokens + (i - half);
    float val = 0.f;
    bool has_mass = x >= 0 && x < a.T;
    if (has_mass && a.mass_trim > 0)
      has_mass = x < a.cu_seqlens[request_of(a.cu_seqlens, a.n_seqs, x) + 1] - a.mass_trim;
    if (has_mass)
      for (int sp = 0; sp < a.row_splits; ++sp) val += a.uraw[((int64_t)sp * a.LH + lz) * a.T + x];
    tile[x - base + half] = val;
  }
#pragma unroll
  for (int e = 0; e < PER; ++e) tile[half + e * 256 + tid] = body[e];
  __syncthreads();
#pragma unroll
  for (int e = 0; e < PER; ++e) {
    const int j = base + e * 256 + tid;
    if (j >= a.T) continue;
    const int s0 = lo_[e], s1 = hi_[e] - a.pool_trim;     // pooling domain [s0, s1)
    const int b0 = max(s0, j - half), b1 = min(s1 - 1, j + half);
    float pooled = 0.f;
    if (j < s1) {
      if (a.pool_max) {
        for (int x = b0; x <= b1; ++x) pooled = fmaxf(pooled, tile[x - base + half]);      // masses are >= 0
      } else {
        for (int x = b0; x <= b1; ++x) pooled += tile[x - base + half];
        pooled *= a.inv_pool;
      }
    }
    a.scores[(int64_t)lz * a.T + j] = __builtin_fmaf(a.lambda, pr[e], pooled);
  }
}

FinishArgs finish_args(const Plan& pl, const float* prior, float* scores, void* workspace) {
  FinishArgs f;
  f.uraw = reinterpret_cast<const float*>(static_cast<char*>(workspace) + pl.off_uraw);
  f.prior = prior; f.cu_seqlens = pl.cu_seqlens_dev; f.scores = scores;
  f.n_seqs = pl.n_seqs; f.T = pl.T; f.LH = pl.L * pl.Hkv; f.row_splits = pl.mass_parts; f.pool = pl.pool;
  f.lambda = pl.lambda; f.inv_pool = 1.0f / (float)pl.pool;
  f.mass_trim = pl.key_trim;
  f.pool_trim = (pl.variant & CODECOMP_VARIANT_POOL_PREFIX) ? pl.W : 0;
  f.pool_max = (pl.variant & CODECOMP_VARIANT_POOL_MAX) ? 1 : 0;
  return f;
}

int launch_row_merge(const Plan& pl, const ScoreArgs& a, hipStream_t stream) {
  const int64_t problems = (int64_t)pl.n_seqs * pl.L * pl.Hkv;
  const bool many = problems >= 2048;     // enough workgroups for the device as it is
  // every request is met by about stat_teams / problems + 1 segments, most rows are held twice in each
  const int64_t items = 2 * (a.stat_teams / problems + 1);
  int ways_log2 = 0;
  while (!many && (1 << ways_log2) < kMergeMaxWays && ((int64_t)kMergeBatch << ways_log2) < items) ++ways_log2;
  const int rows_per = kMergeThreads >> ways_log2;
  const dim3 mgrid(many ? 1 : (a.lrows + rows_per - 1) / rows_per, pl.n_seqs, pl.L * pl.Hkv);
  score_merge_kernel<<<mgrid, dim3(kMergeThreads), 0, stream>>>(a, ways_log2);
  if (hipError_t e = hipGetLastError()) return (int)e;
  return 0;
}

int launch_score(const Plan& pl, const void* q, const void* k, const float* prior, float* scores,
                 void* workspace, hipStream_t stream, unsigned stages) {
  char* ws = static_cast<char*>(workspace);
  ScoreArgs a;
  a.q = static_cast<const uint16_t*>(q);
  a.k = static_cast<const unsigned char*>(k);
  a.cu_seqlens = pl.cu_seqlens_dev;
  a.stats = reinterpret_cast<float*>(ws + pl.off_stats);
  a.lse = reinterpret_cast<float*>(ws + pl.off_lse);
  a.uraw = reinterpret_cast<float*>(ws + pl.off_uraw);
  a.n_seqs = pl.n_seqs; a.Hkv = pl.Hkv; a.G = pl.G; a.W = pl.W; a.R = pl.R;
  a.row_splits = pl.row_splits; a.nb = pl.row_blocks; a.srows = pl.waves * kRowsPerWave;
  a.lrows = pl.row_splits * pl.row_blocks * 32;
  for (int w = 0; w < kMaxWaves; ++w) a.wave_desc[w] = pl.wave_desc[w];
  for (int b = 0; b < 2 * kMaxWaves; ++b) a.rb_holder[b] = (uint32_t)pl.rb_holder[b][0] | (uint32_t)pl.rb_holder[b][1] << 8;
  a.lead = pl.lead_tiles; a.tiles_per_problem = pl.tiles_per_problem; a.total_tiles = pl.total_tiles; a.stat_teams = 0; a.merge_in_mass = 0; a.T = pl.T;
  a.LH = pl.L * pl.Hkv;
  a.q_sl = pl.q_sl; a.q_ss = pl.q_ss; a.q_sh = pl.q_sh; a.q_st = pl.q_st;
  a.kv_sl = pl.kv_sl; a.kv_sh = pl.kv_sh; a.kv_st = pl.kv_st;
  a.c = pl.scale * 1.4426950408889634f;
  a.inv_g = (pl.variant & CODECOMP_VARIANT_GROUP_SUM) ? 1.0f : 1.0f / (float)pl.G;
  a.inv_w = 1.0f / (float)pl.W;
  a.inv_problem = 1.0f / (float)pl.tiles_per_problem; a.inv_heads = 1.0f / (float)pl.Hkv; a.inv_splits = 1.0f / (float)pl.row_splits;
  a.teams = a.tile_each = a.tile_left = a.by_die = 0; a.inv_teams = 0.f;
  a.key_trim = pl.key_trim;
  a.once_keys = pl.once_keys; a.once_rows = pl.once_rows; a.once_chunks = pl.once_chunks;
  a.blocks_per_head = (pl.variant & CODECOMP_VARIANT_GROUP_MAX) ? pl.W / 32 : 1;
  int rc;
  if (pl.team.steps > 0 && (pl.kv_fp8 ? team_fits<128, true>(pl) : team_fits<128, false>(pl))) {
    rc = !(stages & CODECOMP_STAGE_MASS) ? 0 : pl.kv_fp8 ? launch_team<128, true>(pl, a, ws, stream) : launch_team<128, false>(pl, a, ws, stream);
  } else if (pl.kv_fp8) rc = pl.d == 128 ? dispatch_waves<128, true>(pl, a, stream, stages) : dispatch_waves<64, true>(pl, a, stream, stages);
  else rc = pl.d == 128 ? dispatch_waves<128, false>(pl, a, stream, stages) : dispatch_waves<64, false>(pl, a, stream, stages);
  if (rc) return rc;
  if ((stages & CODECOMP_STAGE_MASS) && pl.rows_at_once) {
    if (pl.kv_fp8) rc = pl.d == 128 ? launch_rows<128, true>(pl, a, stream) : launch_rows<64, true>(pl, a, stream);
    else rc = pl.d == 128 ? launch_rows<128, false>(pl, a, stream) : launch_rows<64, false>(pl, a, stream);
    if (rc) return rc;
  }
  if ((stages & CODECOMP_STAGE_MASS) && pl.once_keys > 0) {
    if (pl.kv_fp8) rc = pl.d == 128 ? launch_once<128, true>(pl, a, stream) : launch_once<64, true>(pl, a, stream);
    else rc = pl.d == 128 ? launch_once<128, false>(pl, a, stream) : launch_once<64, false>(pl, a, stream);
    if (rc) return rc;
  }
  if (!(stages & CODECOMP_STAGE_FINISH)) return 0;

  const FinishArgs f = finish_args(pl, prior, scores, workspace);
  const int lh = pl.L * pl.Hkv;
  const int64_t long_ones = (int64_t)((pl.T + 256 * kFinishLong - 1) / (256 * kFinishLong)) * lh;
  if (long_ones >= kFinishFill) score_finish_kernel<kFinishLong><<<dim3((pl.T + 256 * kFinishLong - 1) / (256 * kFinishLong), lh), dim3(256), 0, stream>>>(f);
  else score_finish_kernel<kFinishShort><<<dim3((pl.T + 256 * kFinishShort - 1) / (256 * kFinishShort), lh), dim3(256), 0, stream>>>(f);
  if (hipError_t e = hipGetLastError()) return (int)e;
  return 0;
}

}  // namespace codecomp
