// FP8 K/V path of the masked attention for gfx950: K and V arrive as OCP FP8 E4M3 codes with one
// fp32 scale per kv head (the storage format of an FP8 serving stack; the keys are what a KV cache
// holds, i.e. already rotated), Q arrives in bf16 and is rotated here.  Both products run on the
// FP8 matrix instruction v_mfma_f32_32x32x64_f8f6f4 (64-deep, twice the bf16 rate), fp32 accumulate:
//   k_prep_fp8   K and V^T of every 64-key tile re-laid-out in MFMA operand order (plain byte moves,
//                no arithmetic on the codes), and the cos/sin table for Q
//   (rows that see at most PV_SHORT_ROW_KEYS keys are evaluated in plain fp32 by extra workgroups at the
//   end of k_attn_fp8's grid, one wave per row and query head)
//   k_attn_fp8   flash-style pass: one workgroup = one 32-token query tile x one kv head, wave w =
//                query head kvh*G + w (or four query tiles of one head); a step is one 64-key tile.  Q is rotated, scaled by a per-row
//                power of two and split into two E4M3 terms (the rounded value and 16 x the rounding
//                residual, the second product scaled by 2^-4 inside the instruction), which carries Q
//                at about bf16 precision through the FP8 pipe; probabilities are formed against a running
//                reference, scaled by 2^8 and rounded to E4M3; the row sum comes out of the matrix
//                pipe (a product with ones over the same codes), so the output is an exact convex
//                combination of V rows with the rounded weights.
// Operand layout of the instruction (checked on the device): lane l holds row (or column) l % 32 and
// the 32 consecutive depth indices 32 * (l / 32) .. + 31, byte j of its 32 bytes = depth offset j;
// the accumulator is laid out like the other 32x32 products (lane: column l % 32, register r: row
// 8 (r / 4) + 4 (l / 32) + r % 4).
#include "pv_attn_common.h"

namespace pv {

typedef __attribute__((ext_vector_type(8))) int i32x8;

constexpr int kStepKeys = 64;            // keys per step = depth of the second product

__device__ __forceinline__ f32x16 mfma_fp8(const i32x8& a, const i32x8& b, const f32x16& c) {
  return __builtin_amdgcn_mfma_scale_f32_32x32x64_f8f6f4(a, b, c, 0, 0, 0, 0, 0, 0);   // both operands E4M3, no block scales
}
// The same product with the B operand scaled by 2^-4 in the instruction (block scales are E8M0
// exponents, 0x7f = 1; checked on the device; byte 0 of the word scales A, byte 1 B, so that the two take one
// register): used for the low part of Q.
__device__ __forceinline__ f32x16 mfma_fp8_b_sixteenth(const i32x8& a, const i32x8& b, const f32x16& c) {
  return __builtin_amdgcn_mfma_scale_f32_32x32x64_f8f6f4(a, b, c, 0, 0, 0, 0x7b7f, 1, 0x7b7f);
}
// 16 x 16 x 128: lane l holds row (or column) l % 16 and the depth block l / 16; the accumulator has column
// l % 16, rows 4 (l / 16) ..
__device__ __forceinline__ f32x4 mfma_fp8_16(const i32x8& a, const i32x8& b, const f32x4& c) {
  return __builtin_amdgcn_mfma_scale_f32_16x16x128_f8f6f4(a, b, c, 0, 0, 0, 0, 0, 0);
}
__device__ __forceinline__ float fp8_byte(unsigned word, int byte) {
  switch (byte) {
    case 0: return __builtin_amdgcn_cvt_f32_fp8((int)word, 0);
    case 1: return __builtin_amdgcn_cvt_f32_fp8((int)word, 1);
    case 2: return __builtin_amdgcn_cvt_f32_fp8((int)word, 2);
    default: return __builtin_amdgcn_cvt_f32_fp8((int)word, 3);
  }
}
// four floats -> four E4M3 codes in one dword (round to nearest even; callers keep |x| <= 448)
__device__ __forceinline__ unsigned pack_fp8x4(float a, float b, float c, float d) {
  int w = 0;
  w = __builtin_amdgcn_cvt_pk_fp8_f32(a, b, w, false);
  w = __builtin_amdgcn_cvt_pk_fp8_f32(c, d, w, true);
  return (unsigned)w;
}

// ---------------------------------------------------------------- preparation
// One workgroup per (32 keys, kv head).  Workspace per kv head and tile (8 KB each for D = 128):
//   K:    16-byte chunk ((u * 2 + t) * 2 + c) * 64 + l  = features 64 t + 32 (l / 32) + 16 c .. + 15
//         of key 32 u + l % 32           (u: 32-key half, t: 64-feature half)
//   V^T:  16-byte chunk (db * 2 + c) * 64 + l            = feature 32 db + l % 32 at the 16 keys
//         32 c + 8 i + 4 (l / 32) + e, byte 4 i + e      (the key order in which the accumulator
//         registers of S^T hold keys, so probabilities go into the second product in place)
// Pad keys (beyond the request) are zero codes.  Latency bounds a small launch: half a tile to a workgroup is one load
// of K and of V and one chunk of V^T a thread, and the angles of its keys are shared out among the heads' workgroups and
// formed while the loads fly, where a whole tile with all its angles at the end of the first head's workgroups was a
// chain of its own.  Passes, us, before / with it: 3 K tokens at 32/8 heads 80.3 / 77.6, 4.5 K at 28/4 heads 138.7 /
// 136.3, ragged 23 K 518.5 / 519.5, 4 x 14 K at 64/8 heads 7132 / 7074.
template <int D>
__global__ __launch_bounds__(256) void k_prep_fp8(const int32_t* __restrict__ plan, PlanHeader h,
                                                  const uint8_t* __restrict__ k8,
                                                  const uint8_t* __restrict__ v8, RopeFreq f,
                                                  float2* __restrict__ cs, int hkv, bool rope,
                                                  uint8_t* __restrict__ kw, uint8_t* __restrict__ vw) {
  static_assert(D == 128, "the FP8 path is built for head_dim 128");
  constexpr int CPR = D / 16;                              // 16-byte chunks per key row
  constexpr int KB = 32;                                   // keys per block
  static_assert(KB * CPR == 256 && (D / 32) * 64 == 256, "one chunk of K, V and V^T a thread");
  __shared__ uint4 v_s[KB][CPR + 1];                       // V rows of the block, padded
  const int kvh = (int)blockIdx.x % hkv;
  const int row0 = (int)blockIdx.x / hkv * KB;             // first padded key row
  const KeyBlock own = key_block(plan, h, row0);
  const int tok_base = own.tok_base, n_b = own.n, key0 = own.key0;
  const int tid = threadIdx.x;
  const int half = (row0 / KB) & 1;                        // which half of the 64-key tile
  const int64_t tile_at = ((int64_t)kvh * h.padded_keys + (row0 & ~(kStepKeys - 1))) * D;
  const int key = tid / CPR, c16 = tid % CPR;
  uint4 kx = make_uint4(0, 0, 0, 0), vx = make_uint4(0, 0, 0, 0);
  if (key0 + key < n_b) {
    const int64_t src = (caller_row(plan, h, tok_base + key0 + key) * hkv + kvh) * D + c16 * 16;
    kx = *reinterpret_cast<const uint4*>(k8 + src);
    vx = *reinterpret_cast<const uint4*>(v8 + src);
  }
  if (rope) {
    for (int item = kvh * 256 + tid; item < KB * (D / 2); item += hkv * 256) {
      const int rkey = item / (D / 2), c = item % (D / 2);
      if (key0 + rkey < n_b) {
        const int64_t g = tok_base + key0 + rkey;
        cs[g * (D / 2) + c] = rotary_cos_sin(plan[h.off_pos + g], f.inv_freq[c]);
      }
    }
  }
  const int t = c16 >> 2, hh = (c16 >> 1) & 1, c = c16 & 1;
  reinterpret_cast<uint4*>(kw + tile_at)[((half * 2 + t) * 2 + c) * 64 + hh * 32 + key] = kx;
  v_s[key][c16] = vx;
  __syncthreads();
  const uint8_t* vb = reinterpret_cast<const uint8_t*>(&v_s[0][0]);
  constexpr int VROW = (CPR + 1) * 16;
  const int l = tid & 63, db = tid >> 6;
  const int feat = 32 * db + (l & 31), vhh = l >> 5;
  unsigned w[4];
#pragma unroll
  for (int i = 0; i < 4; ++i) {
    w[i] = 0;
#pragma unroll
    for (int e = 0; e < 4; ++e) w[i] |= (unsigned)vb[(8 * i + 4 * vhh + e) * VROW + feat] << (8 * e);
  }
  reinterpret_cast<uint4*>(vw + tile_at)[(db * 2 + half) * 64 + l] = make_uint4(w[0], w[1], w[2], w[3]);
}

// ---------------------------------------------------------------- rows with few keys, fp32
// One wave per (short row, query head); lane c owns the rotation pair (c, c + D/2).
template <int D>
__device__ void short_unit_fp8(const int32_t* __restrict__ plan, const PlanHeader& h,
                               const uint16_t* __restrict__ q, const uint8_t* __restrict__ k8,
                               const uint8_t* __restrict__ v8, const float* __restrict__ k_scale,
                               const float* __restrict__ v_scale, const float2* __restrict__ table,
                               int hq, int hkv, bool rope, float scale, void* __restrict__ out,
                               float* __restrict__ lse, bool out_f32, int unit, int lane) {
  constexpr int HALF = D / 2;
  const int4 desc = reinterpret_cast<const int4*>(plan + h.off_short)[unit / hq];
  const int head = unit % hq, kvh = head / (hq / hkv);
  const int g = desc.x, base = desc.y, i = g - base, a_end = desc.z, b_start = desc.w;
  const int n_a = min(a_end, (int)PV_SHORT_ROW_KEYS);
  const int b0 = max(b_start, a_end);
  const int n = min(n_a + max(i - b0 + 1, 0), (int)PV_SHORT_ROW_KEYS);
  const int c = lane;                                      // HALF == 64 lanes for D = 128
  const int64_t g_row = caller_row(plan, h, g);
  const uint16_t* qr = q + (g_row * hq + head) * D;
  const float xl = __uint_as_float((unsigned)qr[c] << 16), xh = __uint_as_float((unsigned)qr[c + HALF] << 16);
  float ql = xl, qh = xh;
  if (rope) {
    const float2 t = table[(int64_t)g * HALF + c];
    ql = xl * t.x - xh * t.y;
    qh = xh * t.x + xl * t.y;
  }
  const float ks = k_scale[kvh], vs = v_scale[kvh];
  float sc[PV_SHORT_ROW_KEYS], vl[PV_SHORT_ROW_KEYS], vh[PV_SHORT_ROW_KEYS];
  float m = -INFINITY;
#pragma unroll
  for (int e = 0; e < PV_SHORT_ROW_KEYS; ++e) {
    const int key = e < n_a ? e : b0 + (e - n_a);
    const int64_t row = (caller_row(plan, h, base + (e < n ? key : i)) * hkv + kvh) * D;
    const float kl = fp8_byte(k8[row + c], 0), kh = fp8_byte(k8[row + c + HALF], 0);
    vl[e] = fp8_byte(v8[row + c], 0);
    vh[e] = fp8_byte(v8[row + c + HALF], 0);
    float part = e < n ? ql * kl + qh * kh : 0.0f;
#pragma unroll
    for (int off = 32; off > 0; off >>= 1) part += __shfl_xor(part, off);
    sc[e] = e < n ? part * (scale * ks) : -INFINITY;
    m = fmaxf(m, sc[e]);
  }
  float l = 0.0f, ol = 0.0f, oh = 0.0f;
#pragma unroll
  for (int e = 0; e < PV_SHORT_ROW_KEYS; ++e) {
    const float p = expf(sc[e] - m);
    l += p;
    if (e < n) { ol = fmaf(p, vl[e], ol); oh = fmaf(p, vh[e], oh); }
  }
  const int64_t orow = (g_row * hq + head) * D;
  const float rl = ol * vs / l, rh = oh * vs / l;
  if (out_f32) {
    float* op = reinterpret_cast<float*>(out) + orow;
    op[c] = rl; op[c + HALF] = rh;
  } else {
    uint16_t* op = reinterpret_cast<uint16_t*>(out) + orow;
    op[c] = (uint16_t)(pack_bf16(rl, 0.0f) & 0xffffu);
    op[c + HALF] = (uint16_t)(pack_bf16(rh, 0.0f) & 0xffffu);
  }
  if (lse && lane == 0) lse[(int64_t)head * h.total_tokens + g_row] = m + logf(l);
}

// ---------------------------------------------------------------- main kernel
// 64 x 16 bytes straight from memory into LDS: lane l's 16 bytes at src + lane_off land at lds + 16 l.
// Inline assembly on purpose: the compiler orders its own LDS reads behind every global->LDS load it
// knows of, which would serialise the staging; the waits that are needed are placed by hand.
__device__ __forceinline__ void stage_1k(const uint8_t* src, unsigned lane_off, unsigned lds) {
  asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %1, %2"
               : : "s"(lds), "v"(lane_off), "s"(src) : "memory", "m0");
}
template <int N>
__device__ __forceinline__ void wait_loads() {            // at most N loads of this wave outstanding
  asm volatile("s_waitcnt vmcnt(%0)" : : "n"(N) : "memory");
}

// What bounds it: VALU issue.  A wave's step has 12 products of 64 matrix cycles and one of 32 (800), and ~115 VALU
// instructions of the softmax, 32 of them exponentials (16 cycles each): ~850 cycles of issue, and a product holds
// back VALU issue for about half its time.  Hence staging bypasses the registers, and every product of a step has its
// share of the softmax beside it: with the softmax of a tile beside S^T of the next and only the row maxima beside
// O^T, the two waves of a SIMD met the barrier in the same phase where they belong to one workgroup.  Passes, us,
// before / with it: 4 x (2048 + 8192) tokens, 64/8 heads 7057 / 6731; 4000 + 512, 28/4 heads 160.2 / 153.8;
// 1024 + 4096, 64/8 heads, no rotation 439 / 419; four waves to a workgroup: 512 + 2048, 32/8 heads 78.8 / 79.5, 8
// ragged requests 575.6 / 574.5, three requests at 40/8 heads 327.4 / 324.8.  Matrix pipe 52 / 59 % busy, 14.6 / 13.1 M
// cycles for the first of them.
// QT as in the bf16 kernel: the four waves are four consecutive query tiles of one query head; `tile` is
// the union of the four (it drives the key loop and the staging), `mine` the wave's own.
template <int D, int G, bool QT>
__global__ __launch_bounds__(G * 64, 2) __attribute__((amdgpu_waves_per_eu(2))) void k_attn_fp8(
    const int32_t* __restrict__ plan, PlanHeader h, const uint16_t* __restrict__ q,
    const uint8_t* __restrict__ kw, const uint8_t* __restrict__ vw, const float2* __restrict__ cs,
    const float* __restrict__ k_scale, const float* __restrict__ v_scale, void* __restrict__ out,
    float* __restrict__ lse, int hq, int hkv, float qscale, bool rope, bool out_f32,
    const uint8_t* __restrict__ k8, const uint8_t* __restrict__ v8, float scale, int n_short_blocks, int order) {
  static_assert(D == 128, "the FP8 path is built for head_dim 128");
  static_assert(!QT || G == 4, "query-tile workgroups have four waves");
  // The last n_short_blocks workgroups evaluate the rows with very few keys in fp32, one (row, query
  // head) per wave, from the caller's codes and the table of rotary angles: light work that starts
  // when every item of the grid has been taken, in the tail of the launch.
  if (n_short_blocks > 0 && blockIdx.x >= gridDim.x - (unsigned)n_short_blocks) {
    const int unit = (int)(blockIdx.x - (gridDim.x - (unsigned)n_short_blocks)) * G + ((int)threadIdx.x >> 6);
    if (unit < h.n_short_rows * hq)                        // whole waves leave together
      short_unit_fp8<D>(plan, h, q, k8, v8, k_scale, v_scale, cs, hq, hkv, rope, scale, out, lse, out_f32,
                        unit, (int)threadIdx.x & 63);
    return;
  }
  constexpr int NS = 4;                                    // slots per ring, one key tile each
  constexpr int TILE_BYTES = kStepKeys * D;                // 8 KB of K, the same of V^T
  constexpr int CH = TILE_BYTES / 16;                      // 16-byte chunks of a slot
  constexpr int NREP = (CH / 64 + G - 1) / G;              // staging instructions of a wave for one slot
  constexpr int RS = 2 * D + 16;                           // row stride of the epilogue's transposition
  constexpr int SMEM = (2 * NS * CH * 16 > G * 32 * RS ? 2 * NS * CH * 16 : G * 32 * RS) / 16;
  // K ring, then V^T ring; step j lives in slot j % NS of each.  QT: a slot of zeros behind them (72 KB, two
  // workgroups still fit a compute unit).
  constexpr int ZERO = 2 * NS * CH;
  __shared__ uint4 smem[SMEM + (QT ? CH : 0)];
  static_assert(!QT || SMEM == ZERO, "the slot of zeros starts behind the rings");

  const int tid = threadIdx.x, wave = tid >> 6, lane = tid & 63;
  const int wave_s = __builtin_amdgcn_readfirstlane(wave);
  const int qrow = lane & 31, hh = lane >> 5;
  int kvh, head;
  QTile tile, mine;
  if constexpr (QT) {
    head = (int)blockIdx.x % hq;
    kvh = head / (hq / hkv);
    tile = reinterpret_cast<const QTile*>(plan + h.off_quadwork)[(int)blockIdx.x / hq];
    mine = tile;                                           // a wave without a tile of its own: no row, never masks
    mine.t0 = tile.t0 + 32 * wave_s;
    mine.rows = 0;
    mine.n_full = 1 << 24;
    if (32 * wave_s < tile.rows)                           // tile.n_full: index of the group's first tile
      mine = reinterpret_cast<const QTile*>(plan + h.off_tiles)[tile.n_full + wave_s];
  } else {
    const int item = (int)blockIdx.x;
    kvh = item % hkv;
    head = kvh * G + wave;
    tile = reinterpret_cast<const QTile*>(plan + h.off_work)[dispatch_rank(item / hkv, h.n_q_tiles, order)];
    mine = tile;
  }
  const bool valid = qrow < mine.rows;
  // pad lanes repeat the last row (never stored)
  const int64_t g = (int64_t)tile.tok_base + tile.t0 + min((QT ? 32 * wave : 0) + qrow, tile.rows - 1);
  int a_end = 0, b_start = 0;
  if (valid) { a_end = plan[h.off_aend + g]; b_start = plan[h.off_bstart + g]; }

  // ---- staging.  The key tiles of the item are [0, n_a) then [jb0, jb1), one step each.  A wave moves
  // chunks wave * NREP .. of every slot (beyond the last chunk it repeats the last one: every wave issues
  // the same number of loads, so the waits are constants).  Steps beyond the last repeat the last one.
  const int n_steps = tile.n_a + (tile.jb1 - tile.jb0), last = n_steps - 1;
  const int64_t head_base = ((int64_t)kvh * h.padded_keys + tile.kpad_base) * D;     // bytes
  auto step_tile = [&](int j) { return j < tile.n_a ? j : tile.jb0 + (j - tile.n_a); };
  const unsigned lane16 = (unsigned)lane * 16;
  const unsigned smem_base = (unsigned)(uintptr_t)(__attribute__((address_space(3))) char*)(char*)&smem[0];
  auto stage_one = [&](const uint8_t* ring_src, unsigned ring, int j, int n) __attribute__((always_inline)) {
    const int c = min(wave_s * NREP + n, CH / 64 - 1);
    stage_1k(ring_src + head_base + (int64_t)step_tile(min(j, last)) * TILE_BYTES + c * 1024, lane16,
             smem_base + ring + (unsigned)(j & (NS - 1)) * TILE_BYTES + (unsigned)c * 1024);
  };
  auto stage_k = [&](int j) { for (int n = 0; n < NREP; ++n) stage_one(kw, 0u, j, n); };
  auto stage_v = [&](int j) { for (int n = 0; n < NREP; ++n) stage_one(vw, NS * TILE_BYTES, j, n); };

  // ---- Q: features 32 hh .. + 31 and 64 + 32 hh .. + 31 of this lane's row (the rotation pairs
  // (c, c + 64) sit in one lane), rotated, scaled by a power of two that brings the row's largest
  // magnitude into [128, 256), rounded to E4M3.
  i32x8 qf[2], qlo[2];                                     // Q = qf + qlo / 16, both E4M3
  float c_row;                                             // exponent argument per unit of S
  {
    const uint16_t* qr = q + (caller_row(plan, h, g) * hq + head) * D;
    uint4 raw[2][4], tab[16];
#pragma unroll
    for (int v4 = 0; v4 < 4; ++v4) {
      raw[0][v4] = reinterpret_cast<const uint4*>(qr + 32 * hh)[v4];
      raw[1][v4] = reinterpret_cast<const uint4*>(qr + 64 + 32 * hh)[v4];
    }
    if (rope) {
      const uint4* t = reinterpret_cast<const uint4*>(cs + g * (D / 2) + 32 * hh);
#pragma unroll
      for (int j = 0; j < 16; ++j) tab[j] = t[j];
    }
    __builtin_amdgcn_sched_barrier(0);
    stage_k(0);
    stage_k(1);
    __builtin_amdgcn_sched_barrier(0);
    float lo[32], hi[32];
#pragma unroll
    for (int v4 = 0; v4 < 4; ++v4) {
      const uint4 a = raw[0][v4], b = raw[1][v4];
      const unsigned aw[4] = {a.x, a.y, a.z, a.w}, bw[4] = {b.x, b.y, b.z, b.w};
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        lo[8 * v4 + 2 * e] = bf16_lo(aw[e]); lo[8 * v4 + 2 * e + 1] = bf16_hi(aw[e]);
        hi[8 * v4 + 2 * e] = bf16_lo(bw[e]); hi[8 * v4 + 2 * e + 1] = bf16_hi(bw[e]);
      }
    }
    if (rope) {
#pragma unroll
      for (int j = 0; j < 32; ++j) {
        const uint4 w4 = tab[j / 2];
        const float wc = __uint_as_float(j % 2 ? w4.z : w4.x), wsn = __uint_as_float(j % 2 ? w4.w : w4.y);
        const float l0 = lo[j], h0 = hi[j];
        // (spelled out: which product the compiler contracts shows in the codes of values next to a rounding
        // boundary, a change of 1e-4 of the output's norm from one build to another)
        lo[j] = __builtin_fmaf(l0, wc, -(h0 * wsn));
        hi[j] = __builtin_fmaf(l0, wsn, h0 * wc);
      }
    }
    stage_v(0); stage_k(2); stage_v(1); stage_k(3);
    float amax = 0.0f;
#pragma unroll
    for (int j = 0; j < 32; ++j) amax = fmaxf(amax, fmaxf(fabsf(lo[j]), fabsf(hi[j])));
    amax = pair_max(amax);
    // power of two f with 128 <= amax * f < 256 (exact scaling; 1 for an all-zero row)
    int e2 = (int)((__float_as_uint(amax) >> 23) & 255u) - 127;
    e2 = max(e2, -100);
    const float fac = amax > 0.0f ? __uint_as_float((unsigned)(127 + 7 - e2) << 23) : 1.0f;
    const float inv_fac = amax > 0.0f ? __uint_as_float((unsigned)(127 - 7 + e2) << 23) : 1.0f;
    auto split4 = [&](const float* x, int& top, int& rest) {   // four values -> rounded codes and residual codes
      const float x0 = x[0] * fac, x1 = x[1] * fac, x2 = x[2] * fac, x3 = x[3] * fac;
      const unsigned w = pack_fp8x4(x0, x1, x2, x3);
      top = (int)w;
      const f32x2 t0 = __builtin_amdgcn_cvt_pk_f32_fp8((int)w, false), t1 = __builtin_amdgcn_cvt_pk_f32_fp8((int)w, true);
      rest = (int)pack_fp8x4((x0 - t0[0]) * 16.0f, (x1 - t0[1]) * 16.0f, (x2 - t1[0]) * 16.0f, (x3 - t1[1]) * 16.0f);
    };
#pragma unroll
    for (int w = 0; w < 8; ++w) {
      int top, rest;
      split4(&lo[4 * w], top, rest);
      qf[0][w] = top; qlo[0][w] = rest;
      split4(&hi[4 * w], top, rest);
      qf[1][w] = top; qlo[1][w] = rest;
    }
    c_row = qscale * k_scale[kvh] * inv_fac;               // qscale = softmax scale * log2(e)
  }

  f32x16 o[4];
#pragma unroll
  for (int r = 0; r < 16; ++r) { o[0][r] = 0.0f; o[1][r] = 0.0f; o[2][r] = 0.0f; o[3][r] = 0.0f; }
  // Row sums: P^T as the B operand of the 16 x 16 x 128 product.  Its columns are l % 16, so the lanes of
  // queries c and c + 16 share a column and fill different depth blocks (l / 16): rows with ones in blocks 0
  // and 2 sum query c, rows with ones in blocks 1 and 3 query c + 16.  Row r takes the blocks of parity
  // (r / 4) % 2, which gives every lane its own query's sum in all four accumulators.
  float l_run = 0.0f;
  i32x8 ones;
  {
    int x = (lane >> 4 & 1) == (lane >> 2 & 1) ? 0x38383838 : 0;   // 1.0 in E4M3
#pragma unroll
    for (int w = 0; w < 8; ++w) { asm volatile("" : "+v"(x)); ones[w] = x; }
  }
  auto sum_product = [&](const i32x8& p) __attribute__((always_inline)) {
    const f32x4 zero = {0.0f, 0.0f, 0.0f, 0.0f};
    return mfma_fp8_16(ones, p, zero);
  };
  float mref = -INFINITY;                                  // reference of the exponent, log2 units

  // ---- pipeline.  Step j: O^T += V^T P^T of tile j and S^T of tile j + 2 on the matrix pipe, the probabilities of
  // tile j + 1 between them, so that every product has softmax work beside it.  Eight operands a step (a 32-key half
  // of K by 64 features, or 32 features of V^T) go through four register sets in the order of their use,
  //   K(u0,t0) V0 K(u0,t1) V1 K(u1,t0) K(u1,t1) V2 V3
  // and a set is refilled with the operand four places on as soon as it has been consumed.
  i32x8 op[4];
  i32x8 pA, pB;         // probabilities of two tiles, alternating roles from step to step
#pragma unroll
  for (int w = 0; w < 8; ++w) { pA[w] = 0; pB[w] = 0; }
  f32x16 sA[2], sB[2];  // score tiles (two 32-key halves each), likewise
  auto load_op = [&](i32x8& r, int chunk) __attribute__((always_inline)) {
    const uint4 a0 = smem[chunk], a1 = smem[chunk + 64];
    r[0] = (int)a0.x; r[1] = (int)a0.y; r[2] = (int)a0.z; r[3] = (int)a0.w;
    r[4] = (int)a1.x; r[5] = (int)a1.y; r[6] = (int)a1.z; r[7] = (int)a1.w;
  };
  auto k_chunk = [&](int j) { return (j & (NS - 1)) * CH + lane; };
  // QT: a key tile that only the other query tiles of the group read has probability zero throughout, and its
  // V^T is read from the slot of zeros: a NaN in it is not this tile's.  Every such tile is masked, so the test
  // sits with the mask, and a step in the open pays for a scalar select.  (Zeroing the operands instead, behind
  // a branch of its own, cost 1.5 to 3 % of the pass.)
  bool foreign = false, foreign_next = false;              // tile j, tile j + 1 is such a one
  auto v_chunk = [&](int j, bool zeros) { return (QT && zeros ? ZERO : (NS + (j & (NS - 1))) * CH) + lane; };
  constexpr auto koff = [](int u, int t) { return (2 * u + t) * 128; };
  // one of the eight products of S^T: half u of the keys, half t of the features, high or low term of Q
  auto mfma_qk = [&](f32x16 (&s)[2], const i32x8& a, auto u, auto t, auto lo) __attribute__((always_inline)) {
    constexpr int U = decltype(u)::value, T = decltype(t)::value, LO = decltype(lo)::value;
    if constexpr (T == 0 && LO == 0) {
#pragma unroll
      for (int r = 0; r < 16; ++r) s[U][r] = 0.0f;
    }
    if constexpr (LO) s[U] = mfma_fp8_b_sixteenth(a, qlo[T], s[U]);
    else s[U] = mfma_fp8(a, qf[T], s[U]);
  };
  // Row predicate: the keys of half u that this lane holds are key0 + 32 u + 4 hh + c,
  // c = 8 (r / 4) + r % 4; the row's visible ones among the 32 become a bit mask, and a score
  // is kept or replaced by -inf with one bit-field extract and one bit-field insert.
  auto apply_mask = [&](f32x16 (&s)[2], int key0) __attribute__((always_inline)) {
    auto low_bits = [](int n) {                            // bits [0, n) of 32, n clamped to [0, 32]
      const unsigned m = (1u << (n & 31)) - 1u;
      return n <= 0 ? 0u : n >= 32 ? 0xffffffffu : m;
    };
    // (4 hh and the row's index are formed anew from an opaque lane index: the register file is full, and what lives
    // through the loop for the sake of a rare path ends up in scratch memory)
    unsigned l16 = lane16;
    asm volatile("" : "+v"(l16));
    const int row = (int)((l16 >> 4) & 31u), i_loc = row < mine.rows ? mine.t0 + row : -1;
#pragma unroll
    for (int u = 0; u < 2; ++u) {
      const int base = key0 + 32 * u + 4 * (int)(l16 >> 9);
      const unsigned vis = low_bits(a_end - base) | (low_bits(i_loc - base + 1) & ~low_bits(b_start - base));
#pragma unroll
      for (int r = 0; r < 16; ++r) {
        const unsigned keep = (unsigned)__builtin_amdgcn_sbfe((int)vis, 8 * (r / 4) + (r % 4), 1);
        s[u][r] = __uint_as_float((__float_as_uint(s[u][r]) & keep) | (0xff800000u & ~keep));
      }
    }
  };
  // returns whether the tile is one that only other query tiles read
  auto mask_tile = [&](f32x16 (&s)[2], int jt) __attribute__((always_inline)) {
    bool other = false;
    if (__builtin_expect(jt >= mine.n_full, 0)) {
      if constexpr (QT) other = jt >= mine.n_a && (jt < mine.jb0 || jt >= mine.jb1);
      apply_mask(s, jt * kStepKeys);
    }
    return other;
  };
  // Running reference: moved up when a tile's largest exponent exceeds it by more than 0.75 octave
  // (probabilities scaled by 2^8 then stay below 2^8.75 = 431 < 448, the largest E4M3 value).  O and the row sum
  // follow one step later, when the tile before it, whose probabilities stand on the old reference, is in them.
  float bias = 0.0f;                                       // 8 - mref; 0 while no key has been seen (every S is -inf, p = 0)
  float alpha = 1.0f;                                      // what O and the row sum still have to be scaled by
  uint64_t rescale = 0;                                    // the lanes whose alpha is not 1
  auto apply_alpha = [&]() __attribute__((always_inline)) {
#pragma unroll
    for (int r = 0; r < 16; ++r) {
      o[0][r] *= alpha; o[1][r] *= alpha; o[2][r] *= alpha; o[3][r] *= alpha;
    }
    l_run *= alpha;
  };
  auto raise_to = [&](float mx) __attribute__((always_inline)) {   // mx: the tile's largest exponent
    const bool raise = mx > mref + 0.75f;                  // (mref = -inf: any visible key)
    const float m_new = raise ? mx : mref;
    alpha = mref == -INFINITY ? 0.0f : __builtin_amdgcn_exp2f(mref - m_new);   // 1 when unchanged
    mref = m_new;
    bias = mref == -INFINITY ? 0.0f : 8.0f - mref;
  };
  auto max3 = [](float a, float b, float c) __attribute__((always_inline)) { return fmaxf(fmaxf(a, b), c); };
  auto max_half = [&](const f32x16& s) __attribute__((always_inline)) {    // of elements 0 .. 14
    float mx = max3(s[0], s[1], s[2]);
    static_for<0, 6>([&](auto i) {
      constexpr int I = 3 + 2 * decltype(i)::value;
      mx = max3(mx, s[I], s[I + 1]);
    });
    return mx;
  };
  using c0 = std::integral_constant<int, 0>;
  using c1 = std::integral_constant<int, 1>;
  // The sum over a tile's probabilities.  A query's NaN (a NaN in its Q row, or in a key that its neighbour
  // does not see) meets the zeros of the query that shares its column: such a tile is summed from the codes.
  auto sum_codes = [&](const i32x8& p) __attribute__((always_inline)) {
    float rs = 0.0f;
#pragma unroll
    for (int w = 0; w < 8; ++w) {
      const unsigned c = (unsigned)p[w];
      rs += (fp8_byte(c, 0) + fp8_byte(c, 1)) + (fp8_byte(c, 2) + fp8_byte(c, 3));
    }
    return pair_sum(rs);
  };
  auto add_row_sum = [&](const f32x4& sum, const i32x8& p) __attribute__((always_inline)) {
    float rs = sum[0];
    if (__builtin_expect(__builtin_amdgcn_ballot_w64(rs != rs) != 0, 0)) rs = sum_codes(p);
    l_run += rs;
  };

  // PV, QK: which of the two products the step has.  Step -1 forms S^T of tile 1 beside the probabilities of tile 0,
  // step last - 1 has no tile left to score.
  auto step = [&](int j, f32x16 (&s_in)[2], f32x16 (&s_out)[2], i32x8& p_in, i32x8& p_out, auto with_pv,
                  auto with_qk) __attribute__((always_inline)) {
    constexpr bool PV = decltype(with_pv)::value, QK = decltype(with_qk)::value;
    const int kc = k_chunk(j + 2), vc = v_chunk(j, foreign), kc1 = k_chunk(j + 3), vc1 = v_chunk(j + 1, foreign_next);
    // Softmax share of group g: the exponentials of three scores, the arguments of the next group's, and the
    // rounding of the pairs that the group before completed, so that none waits for its input in front of a product.
    float ea[32], ex[32];
    auto v_arg = [&](auto i) {
      constexpr int I = decltype(i)::value;
      if constexpr (I < 32) ea[I] = __builtin_fmaf(s_in[I / 16][I % 16], c_row, bias);
    };
    auto v_exp = [&](auto i) {
      constexpr int I = decltype(i)::value;
      if constexpr (I < 32) {
        ex[I] = __builtin_amdgcn_exp2f(ea[I]);
        asm volatile("" :: "v"(ex[I]));                    // a use in this group: not sunk to the pack
      }
    };
    auto softmax = [&](auto g) {
      constexpr int GI = decltype(g)::value;
      static_for<0, 16>([&](auto e) {                      // pair e: scores 2 e and 2 e + 1
        constexpr int E = decltype(e)::value;
        if constexpr ((2 * E + 1) / 3 + 1 == GI) {
          if constexpr (E % 2 == 0) p_out[E / 2] = __builtin_amdgcn_cvt_pk_fp8_f32(ex[2 * E], ex[2 * E + 1], p_out[E / 2], false);
          else p_out[E / 2] = __builtin_amdgcn_cvt_pk_fp8_f32(ex[2 * E], ex[2 * E + 1], p_out[E / 2], true);
          asm volatile("" :: "v"(p_out[E / 2]));           // a use here: not sunk behind the branches below
        }
      });
      static_for<0, 3>([&](auto k) { v_exp(std::integral_constant<int, 3 * GI + decltype(k)::value>{}); });
      static_for<0, 3>([&](auto k) { v_arg(std::integral_constant<int, 3 * GI + 3 + decltype(k)::value>{}); });
      __builtin_amdgcn_sched_barrier(0);
    };
    auto mfma_done = [&]() { __builtin_amdgcn_sched_barrier(0); };   // the product first, its group's other work behind it
    auto stage = [&](auto x) {                             // K of tile j + 5, then V^T of tile j + 3
      constexpr int X = decltype(x)::value;
      if constexpr (X < NREP) stage_one(kw, 0u, j + 5, X);
      else if constexpr (X < 2 * NREP) stage_one(vw, NS * TILE_BYTES, j + 3, X - NREP);
    };
#define PV_G(n) std::integral_constant<int, n>{}
    static_for<0, 3>([&](auto k) { v_arg(k); });
    __builtin_amdgcn_sched_barrier(0);
    auto qk = [&](const i32x8& k, auto u, auto t, auto lo) {
      if constexpr (QK) { mfma_qk(s_out, k, u, t, lo); mfma_done(); }
    };
    auto pv = [&](auto x, const i32x8& v) {
      constexpr int X = decltype(x)::value;
      if constexpr (PV) { o[X] = mfma_fp8(v, p_in, o[X]); mfma_done(); }
    };
    qk(op[0], c0{}, c0{}, c0{}); softmax(PV_G(0));
    pv(PV_G(0), op[1]); if constexpr (QK) load_op(op[1], kc + koff(1, 1)); softmax(PV_G(1));
    qk(op[0], c0{}, c0{}, c1{}); if constexpr (QK) load_op(op[0], kc + koff(1, 0)); softmax(PV_G(2));
    qk(op[2], c0{}, c1{}, c0{}); softmax(PV_G(3));
    pv(PV_G(1), op[3]); if constexpr (PV) load_op(op[3], vc + 3 * 128); softmax(PV_G(4));
    qk(op[2], c0{}, c1{}, c1{}); if constexpr (PV) load_op(op[2], vc + 2 * 128); softmax(PV_G(5));
    qk(op[0], c1{}, c0{}, c0{}); softmax(PV_G(6));
    // K of tile j + 3 and V^T of tile j + 1 have to be there; younger: K(j+4), V^T(j+2).  Every wave is done with K of
    // tile j + 1 and V^T of tile j - 1, whose slots the loads below refill.
    wait_loads<2 * NREP>();
    __builtin_amdgcn_s_barrier();
    asm volatile("" ::: "memory");
    qk(op[0], c1{}, c0{}, c1{}); if constexpr (QK) { load_op(op[0], kc1 + koff(0, 0)); stage(PV_G(0)); } softmax(PV_G(7));
    qk(op[1], c1{}, c1{}, c0{}); if constexpr (QK) stage(PV_G(1)); softmax(PV_G(8));
    qk(op[1], c1{}, c1{}, c1{}); load_op(op[1], vc1); if constexpr (QK) stage(PV_G(2)); softmax(PV_G(9));
    pv(PV_G(2), op[2]); if constexpr (QK) { load_op(op[2], kc1 + koff(0, 1)); stage(PV_G(3)); } softmax(PV_G(10));
    softmax(PV_G(11));
#undef PV_G
    foreign = foreign_next;
    if constexpr (QK) foreign_next = mask_tile(s_out, step_tile(j + 2));
    f32x4 row_sum = {0.0f, 0.0f, 0.0f, 0.0f};
    if constexpr (PV) row_sum = sum_product(p_in);
    __builtin_amdgcn_sched_barrier(0);
    float m0 = 0.0f, mx = 0.0f;
    if constexpr (QK) {
      m0 = max_half(s_out[0]);
      asm volatile("" : "+v"(m0));                         // stays here, beside the products
    }
    __builtin_amdgcn_sched_barrier(0);
    if constexpr (PV) o[3] = mfma_fp8(op[3], p_in, o[3]);
    __builtin_amdgcn_sched_barrier(0);
    load_op(op[3], vc1 + 128);
    if constexpr (QK) mx = pair_max(fmaxf(max_half(s_out[1]), max3(s_out[1][15], s_out[0][15], m0))) * c_row;   // c_row > 0
    if constexpr (PV) {
      asm volatile("" :: "v"(row_sum));                    // (its unused elements are not handed to the maxima, which would wait)
      add_row_sum(row_sum, p_in);
      if (__builtin_expect(rescale != 0, 0)) apply_alpha();
    }
    if constexpr (QK) {
      rescale = __builtin_amdgcn_ballot_w64(mx > mref + 0.75f);
      if (__builtin_expect(rescale != 0, 0)) raise_to(mx);
    }
    __builtin_amdgcn_sched_barrier(0);
  };

  // ---- prologue: S^T of tile 0 and its reference
  if constexpr (QT) {
#pragma unroll
    for (int n = 0; n < CH / (G * 64); ++n) smem[ZERO + n * (G * 64) + tid] = make_uint4(0u, 0u, 0u, 0u);
    asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");     // the barrier below makes them everyone's
  }
  wait_loads<4 * NREP>();                                  // K of tiles 0 and 1
  __builtin_amdgcn_s_barrier();
  asm volatile("" ::: "memory");
  load_op(op[0], k_chunk(0) + koff(0, 0)); load_op(op[1], k_chunk(0) + koff(1, 0));
  load_op(op[2], k_chunk(0) + koff(0, 1)); load_op(op[3], k_chunk(0) + koff(1, 1));
  mfma_qk(sA, op[0], c0{}, c0{}, c0{}); mfma_qk(sA, op[1], c1{}, c0{}, c0{});
  mfma_qk(sA, op[0], c0{}, c0{}, c1{}); mfma_qk(sA, op[1], c1{}, c0{}, c1{});
  mfma_qk(sA, op[2], c0{}, c1{}, c0{}); mfma_qk(sA, op[3], c1{}, c1{}, c0{});
  mfma_qk(sA, op[2], c0{}, c1{}, c1{}); mfma_qk(sA, op[3], c1{}, c1{}, c1{});
  load_op(op[0], k_chunk(1) + koff(0, 0)); load_op(op[2], k_chunk(1) + koff(0, 1));
  foreign_next = mask_tile(sA, step_tile(0));
  {
    raise_to(pair_max(fmaxf(max3(max_half(sA[0]), sA[0][15], sA[1][15]), max_half(sA[1]))) * c_row);             // O and the row sum are still zero
  }
  constexpr std::true_type yes{};
  constexpr std::false_type no{};
  int j = 0;
  if (last >= 1) {
    step(-1, sA, sB, pB, pA, no, yes);
    for (; j + 3 <= last; j += 2) {
      step(j, sB, sA, pA, pB, yes, yes);
      step(j + 1, sA, sB, pB, pA, yes, yes);
    }
    if (j + 2 <= last) {
      step(j, sB, sA, pA, pB, yes, yes);
      sB[0] = sA[0]; sB[1] = sA[1];
      pA = pB;
      ++j;
    }
    step(j, sB, sA, pA, pB, yes, no);                      // j = last - 1
    pA = pB;
    ++j;
  } else {
    step(-1, sA, sB, pB, pA, no, no);
  }
  // the last tile's O^T: its probabilities in pA, two of its operands in op[1] and op[3]
  load_op(op[0], v_chunk(j, foreign) + 2 * 128);
  load_op(op[2], v_chunk(j, foreign) + 3 * 128);
  const f32x4 row_sum = sum_product(pA);
  o[0] = mfma_fp8(op[1], pA, o[0]);
  o[1] = mfma_fp8(op[3], pA, o[1]);
  o[2] = mfma_fp8(op[0], pA, o[2]);
  o[3] = mfma_fp8(op[2], pA, o[3]);
  add_row_sum(row_sum, pA);
  wait_loads<0>();
  __syncthreads();                                         // every wave is done with the rings

  // ---- epilogue: l_run holds the row sum of this lane's query.  The result is
  // transposed through LDS so that every row leaves in contiguous pieces.
  const float l_tot = l_run;
  {
    const float inv = v_scale[kvh] / l_tot;
    // (lane r < 32 holds the descriptor of row r); short rows come from the extra workgroups
    const unsigned stored_rows = (unsigned)__builtin_amdgcn_ballot_w64(
        valid && a_end + mine.t0 + qrow - b_start + 1 > PV_SHORT_ROW_KEYS);
    auto stored = [&](int row) { return ((stored_rows >> row) & 1u) != 0; };
    const int64_t tok0 = (int64_t)mine.tok_base + mine.t0;
    char* tr = reinterpret_cast<char*>(&smem[0]) + (size_t)wave * (32 * RS);
    if (out_f32) {
#pragma unroll
      for (int half = 0; half < 2; ++half) {
#pragma unroll
        for (int dbh = 0; dbh < 2; ++dbh)
#pragma unroll
          for (int i = 0; i < 4; ++i) {
            const f32x16& x = o[half * 2 + dbh];
            *reinterpret_cast<float4*>(tr + qrow * RS + (dbh * 32 + 8 * i + 4 * hh) * 4) =
                make_float4(x[4 * i] * inv, x[4 * i + 1] * inv, x[4 * i + 2] * inv, x[4 * i + 3] * inv);
          }
        constexpr int LPR = D / 8;                         // lanes per row: D/2 floats
#pragma unroll
        for (int it = 0; it < 32 * LPR / 64; ++it) {
          const int row = it * (64 / LPR) + lane / LPR, c = lane % LPR;
          const float4 w = *reinterpret_cast<const float4*>(tr + row * RS + c * 16);
          if (stored(row))
            *reinterpret_cast<float4*>(reinterpret_cast<float*>(out) +
                                       (caller_row(plan, h, tok0 + row) * hq + head) * D + half * (D / 2) + c * 4) = w;
        }
      }
    } else {
#pragma unroll
      for (int db = 0; db < 4; ++db)
#pragma unroll
        for (int i = 0; i < 4; ++i) {
          uint2 w;
          w.x = pack_bf16(o[db][4 * i] * inv, o[db][4 * i + 1] * inv);
          w.y = pack_bf16(o[db][4 * i + 2] * inv, o[db][4 * i + 3] * inv);
          *reinterpret_cast<uint2*>(tr + qrow * RS + (db * 32 + 8 * i + 4 * hh) * 2) = w;
        }
      constexpr int LPR = D / 8;                           // lanes per row: 2 D bytes
#pragma unroll
      for (int it = 0; it < 32 * LPR / 64; ++it) {
        const int row = it * (64 / LPR) + lane / LPR, c = lane % LPR;
        const uint4 w = *reinterpret_cast<const uint4*>(tr + row * RS + c * 16);
        if (stored(row))
          *reinterpret_cast<uint4*>(reinterpret_cast<uint16_t*>(out) +
                                    (caller_row(plan, h, tok0 + row) * hq + head) * D + c * 8) = w;
      }
    }
    if (lse && hh == 0 && stored(qrow))
      lse[(int64_t)head * h.total_tokens + caller_row(plan, h, g)] = (log2f(l_tot) - 8.0f + mref) * 0.6931471805599453f;
  }
}

// QT: one workgroup per (group of four tiles, query head), else one per (tile, kv head).
template <int G, bool QT>
static hipError_t launch_main_fp8(const int32_t* plan, const PlanHeader& h, const uint16_t* q, const uint8_t* kw,
                                  const uint8_t* vw, const float2* cs, const float* ks, const float* vs, void* out,
                                  float* lse, int hq, int hkv, float qscale, bool rope, bool out_f32,
                                  const uint8_t* k8, const uint8_t* v8, float scale, hipStream_t s) {
  dim3 grid;
  // one wave per (short row, query head), G of them to a workgroup, behind the items of the grid
  const int64_t n_short = ((int64_t)h.n_short_rows * hq + G - 1) / G;
  const int64_t items = QT ? (int64_t)h.n_quads * hq : (int64_t)h.n_q_tiles * hkv;
  if (n_short > 0x7fffffff || !grid_1d(items + n_short, G * 64, &grid)) return hipErrorInvalidConfiguration;
  k_attn_fp8<128, G, QT><<<grid, dim3(G * 64), 0, s>>>(plan, h, q, kw, vw, cs, ks, vs, out, lse, hq, hkv, qscale,
                                                       rope, out_f32, k8, v8, scale, (int)n_short,
                                                       QT ? 0 : dispatch_order(h.n_q_tiles, hkv, G));
  return hipGetLastError();
}

hipError_t launch_attn_fp8(const int32_t* plan_dev, const PlanHeader& h, const void* q, const void* k8,
                           const void* v8, const float* k_scale, const float* v_scale, void* out, float* lse,
                           int hq, int hkv, int d, int out_dtype, float scale, const RopeFreq& freq, bool rope,
                           char* ws, const AttnWorkspace& wl, hipEvent_t ev0, hipEvent_t ev1, hipStream_t s) {
  if (d != 128) return hipErrorInvalidValue;
  float2* cs = reinterpret_cast<float2*>(ws + wl.off_cs);
  uint8_t* kw = reinterpret_cast<uint8_t*>(ws + wl.off_krot);
  uint8_t* vw = reinterpret_cast<uint8_t*>(ws + wl.off_vt);
  const uint16_t* kq = reinterpret_cast<const uint16_t*>(q);
  const bool out_f32 = out_dtype == PV_F32;
  dim3 grid;
  if (!grid_1d((int64_t)(h.padded_keys / 32) * hkv, 256, &grid)) return hipErrorInvalidConfiguration;
  k_prep_fp8<128><<<grid, dim3(256), 0, s>>>(plan_dev, h, (const uint8_t*)k8, (const uint8_t*)v8, freq, cs, hkv, rope, kw, vw);
  hipError_t e = hipGetLastError();
  if (e != hipSuccess) return e;
  const float qscale = scale * 1.4426950408889634f;
  if (ev0) { e = hipEventRecord(ev0, s); if (e != hipSuccess) return e; }
#define PV_LAUNCH(GG, QT) launch_main_fp8<GG, QT>(plan_dev, h, kq, kw, vw, cs, k_scale, v_scale, out, lse, hq, hkv, qscale, rope, out_f32, (const uint8_t*)k8, (const uint8_t*)v8, scale, s)
  const int G = hq / hkv;
  if (group_uses_query_tiles(G) && h.n_quads > 0) e = PV_LAUNCH(4, true);
  else if (G == 4) e = PV_LAUNCH(4, false);
  else if (G == 7) e = PV_LAUNCH(7, false);
  else if (G == 8) e = PV_LAUNCH(8, false);
  else e = hipErrorInvalidValue;
#undef PV_LAUNCH
  if (e != hipSuccess) return e;
  if (ev1) { e = hipEventRecord(ev1, s); if (e != hipSuccess) return e; }
  return hipSuccess;
}

}  // namespace pv
