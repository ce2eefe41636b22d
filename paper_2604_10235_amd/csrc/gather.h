// Internal header: the row copies of the gather step, for its own kernel (gather.hip) and for the selection of short requests,
// which copies the rows it kept itself (select.hip).
#pragma once
#include "plan.h"

namespace codecomp {

struct GatherArgs {
  const unsigned char* k;
  const unsigned char* v;
  const int32_t* idx;
  const int32_t* cu_seqlens;
  const int32_t* cu_budgets;
  unsigned char* k_out;
  unsigned char* v_out;
  int n_seqs, Hkv, TB, pieces_log2;    // 16-byte pieces per row = d * element size / 16 (4, 8 or 16)
  int64_t kv_sl, kv_sh, kv_st, o_sl, o_sh, o_st;     // in bytes
};

typedef unsigned int u32x4 __attribute__((ext_vector_type(4)));

__device__ __forceinline__ u32x4 ld16(const unsigned char* p) { return *reinterpret_cast<const u32x4*>(p); }
__device__ __forceinline__ void st16(unsigned char* p, u32x4 v) { *reinterpret_cast<u32x4*>(p) = v; }

GatherArgs gather_args(const Plan& pl, const void* k, const void* v, const int32_t* idx, void* k_out, void* v_out);

// The rows that one request keeps in one (layer, head), by a workgroup of NT threads that has just written their indices.
template <int NT>
__device__ __forceinline__ void gather_request(const GatherArgs& a, int lz, int s0, int n, int o0, int kept) {
  constexpr int ROWS = 4;              // of K and of V a thread has in flight
  const int layer = lz / a.Hkv, head = lz - layer * a.Hkv;
  const int32_t* idx = a.idx + (int64_t)lz * a.TB + o0;
  const int piece = (threadIdx.x & ((1 << a.pieces_log2) - 1)) * 16, step = NT >> a.pieces_log2;
  const unsigned char* kb = a.k + layer * a.kv_sl + head * a.kv_sh + (int64_t)s0 * a.kv_st + piece;
  const unsigned char* vb = a.v + layer * a.kv_sl + head * a.kv_sh + (int64_t)s0 * a.kv_st + piece;
  unsigned char* ko = a.k_out + layer * a.o_sl + head * a.o_sh + (int64_t)o0 * a.o_st + piece;
  unsigned char* vo = a.v_out + layer * a.o_sl + head * a.o_sh + (int64_t)o0 * a.o_st + piece;
  asm volatile("s_waitcnt vmcnt(0)" ::: "memory");       // this thread's indices are out
  __syncthreads();
  for (int slot = threadIdx.x >> a.pieces_log2; slot < kept; slot += ROWS * step) {
    u32x4 kv[ROWS], vv[ROWS];
#pragma unroll
    for (int i = 0; i < ROWS; ++i) {
      const int64_t tok = min(max(idx[min(slot + i * step, kept - 1)], 0), n - 1);
      kv[i] = ld16(kb + tok * a.kv_st);
      vv[i] = ld16(vb + tok * a.kv_st);
    }
#pragma unroll
    for (int i = 0; i < ROWS; ++i)
      if (slot + i * step < kept) {
        st16(ko + (int64_t)(slot + i * step) * a.o_st, kv[i]);
        st16(vo + (int64_t)(slot + i * step) * a.o_st, vv[i]);
      }
  }
}

}  // namespace codecomp
