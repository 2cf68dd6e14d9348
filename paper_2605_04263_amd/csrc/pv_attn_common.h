// Device helpers shared by the bf16 MFMA attention kernels (gfx950).
#ifndef PV_ATTN_COMMON_H_
#define PV_ATTN_COMMON_H_

#include <type_traits>

#include "pv_internal.h"

namespace pv {

typedef __attribute__((ext_vector_type(8))) __bf16 bf16x8;
typedef __attribute__((ext_vector_type(2))) __bf16 bf16x2;
typedef __attribute__((ext_vector_type(2))) float f32x2;
typedef __attribute__((ext_vector_type(4))) float f32x4;
typedef __attribute__((ext_vector_type(16))) float f32x16;

__device__ __forceinline__ unsigned pack_bf16(float a, float b) {
  f32x2 v = {a, b};
  bf16x2 r = __builtin_convertvector(v, bf16x2);   // round to nearest even
  return __builtin_bit_cast(unsigned, r);
}
__device__ __forceinline__ float bf16_lo(unsigned u) { return __uint_as_float(u << 16); }
__device__ __forceinline__ float bf16_hi(unsigned u) { return __uint_as_float(u & 0xffff0000u); }

__device__ __forceinline__ bf16x8 as_bf16x8(uint4 u) { return __builtin_bit_cast(bf16x8, u); }

// Value held by the lane 32 away (both halves get the other's value via max/sum of the pair).
__device__ __forceinline__ float pair_max(float x) {
  const unsigned u = __float_as_uint(x);
  auto r = __builtin_amdgcn_permlane32_swap(u, u, false, false);
  return fmaxf(__uint_as_float(r[0]), __uint_as_float(r[1]));
}
__device__ __forceinline__ float pair_sum(float x) {
  const unsigned u = __float_as_uint(x);
  auto r = __builtin_amdgcn_permlane32_swap(u, u, false, false);
  return __uint_as_float(r[0]) + __uint_as_float(r[1]);
}

// 16-byte LDS read issued as inline assembly: the compiler neither tracks it nor orders it against
// the global->LDS staging loads (its own LDS reads would wait for every outstanding staging load).
// The caller must execute LDS_WAIT on the destination registers before using them.
template <int OFF>
__device__ __forceinline__ bf16x8 lds_read_b128(unsigned addr) {
  bf16x8 r;
  asm volatile("ds_read_b128 %0, %1 offset:%2" : "=v"(r) : "v"(addr), "n"(OFF));
  return r;
}
// The same read refilling `r` in place: the result is tied to the register that held the operand
// just consumed, so the allocator cannot spread a double-buffered operand over two register sets.
template <int OFF>
__device__ __forceinline__ void lds_refill_b128(bf16x8& r, unsigned addr) {
  asm volatile("ds_read_b128 %0, %1 offset:%2" : "+v"(r) : "v"(addr), "n"(OFF));
}
template <int I, int N, typename F>
__device__ __forceinline__ void static_for(F&& f) {
  if constexpr (I < N) {
    f(std::integral_constant<int, I>{});
    static_for<I + 1, N>(f);
  }
}

// (cos, sin) of the rotary angle pos * inv_freq.  Angles reach 1e5 rad, so the product is formed
// in fp64 and reduced there to a fraction of a revolution; the hardware cosine and sine take that
// fraction directly.  Measured against fp64 over the positions and frequencies in use: absolute
// error at most 2.6e-7, four orders below the bf16 rounding of what the result rotates.
__device__ __forceinline__ float2 rotary_cos_sin(int pos, double inv_freq) {
  const double rev = (double)pos * inv_freq * 0.15915494309189535;     // angle / (2 pi)
  const float fr = (float)(rev - floor(rev));
  return make_float2(__builtin_amdgcn_cosf(fr), __builtin_amdgcn_sinf(fr));
}

// Order in which a launch takes the work list (sorted longest first) when the whole grid is at most four
// workgroups to a compute unit, two of them resident: plain longest-first then pairs the longest items
// with each other and leaves some compute units one item more than others.  `a` tiles are one
// workgroup for each of the 256 compute units, x = tiles beyond two for each.
//   x <= 0, or a .. 2a     the second `a` tiles in reverse: a long first item gets a short partner
//   0 < x <= a             the x shortest first (in reverse), then the middle ones: the slots they free
//                          early take the middle ones, and no compute unit gets a fourth item
//   x > 2a                 longest first as listed
// Measured (32/8 heads of 128, launch of the main kernel, us, longest first / this order, bf16; FP8): 0.75
// workgroups per slot 32.3 / 30.6; 36.6 / 34.5 - 1.0: 43.5 / 41.3; 45.4 / 43.6 - 1.25: 63.6 / 62.7;
// 63.8 / 63.5 - 1.5: 79.3 / 75.0; 77.7 / 72.1 - 1.75: 102.0 / 98.5; 100.9 / 94.5 - 2.0: 128.1 / 124.5;
// 122.7 / 116.5 - beyond 2 within 1 % either way.  Whole passes, us, at other heads: 16/4 of 64, 0.8: 55.3 /
// 52.6 - 1.25: 86.5 / 83.6 - 1.6: 113.9 / 114.1 - 1.9: 150.3 / 149.0; 32/8 of 64, 0.8: 36.3 / 34.8 - 1.25:
// 50.0 / 49.0 - 1.6: 67.2 / 66.9 - 1.9: 86.5 / 86.2; 16/4 of 128, 1.6: 180.2 / 177.3.
// Returned: 0 as listed, a > 0 the second `a` reversed, -a the shortest first behind the first `a`.
inline int dispatch_order(int n_tiles, int hkv, int G) {
  const int a = 256 / hkv;
  if (G != 4 || a < 1) return 0;                        // other group sizes: not two such workgroups per unit
  const int x = n_tiles - 2 * a;
  if (n_tiles <= a || x > 2 * a) return 0;
  return x > 0 && x <= a ? -a : a;
}
__device__ __forceinline__ int dispatch_rank(int pos, int n, int order) {
  if (order == 0) return pos;
  const int a = order > 0 ? order : -order;
  if (pos < a) return pos;
  if (order > 0) {
    const int b = min(a, n - a);
    return pos < a + b ? a + b - 1 - (pos - a) : pos;
  }
  const int x = n - 2 * a;
  return pos < a + x ? n - 1 - (pos - a) : pos - x;
}

// caller_row of the 32 rows from `tok0` on (beyond rows_m1 the last one): lanes r and r + 32 look up row r, of() hands
// out the one of any row.  One round trip where a look-up per use, each behind the loads in front of it, is a chain of
// eight before the first product of an item and again before its last store.  Interleaved packing, passes, us, before /
// with it: 512 + 2048 tokens at 32/8 heads 88.8 / 87.1, at 64/8 heads 166.6 / 156.4; three requests of 1.5 to 4 K at
// 40/8 heads 434 / 413.
struct CallerRows {
  int mine;
  __device__ __forceinline__ CallerRows(const int32_t* plan, const PlanHeader& h, int64_t tok0, int rows_m1)
      : mine((int)caller_row(plan, h, tok0 + min((int)(threadIdx.x & 31), rows_m1))) {}
  __device__ __forceinline__ int64_t of(int row) const { return __shfl(mine, row); }
};

// The request that owns padded key row `row0` (requests are padded to multiples of 64 keys), for a preparation block.
// One request: everything is in the header, and a block starts with its loads instead of a round trip to the plan
// (passes, us, 352 tokens 22.8 / 21.4, 2.5 K tokens 70.8 / 70.1).
struct KeyBlock {
  int tok_base, n;        // first packed row of the request, its tokens
  int key0;               // row0 in the request
};
__device__ __forceinline__ KeyBlock key_block(const int32_t* plan, const PlanHeader& h, int row0) {
  if (h.batch == 1) return {0, h.total_tokens, row0};
  const int32_t* kp = plan + h.off_kpad_start;
  int lo = 0, hi = h.batch;
  while (hi - lo > 1) {
    const int mid = (lo + hi) >> 1;
    if (kp[mid] <= row0) lo = mid; else hi = mid;
  }
  const int tok_base = plan[h.off_tok_start + lo];
  return {tok_base, plan[h.off_tok_start + lo + 1] - tok_base, row0 - kp[lo]};
}

// s_waitcnt immediate (gfx9 encoding) that waits for vmcnt <= n only.
__host__ __device__ constexpr int vmcnt_imm(int n) { return 0x0f70 | (n & 15) | ((n >> 4) << 14); }

}  // namespace pv
#endif
