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
// exponents, 0x7f = 1; checked on the device): used for the low part of Q.
__device__ __forceinline__ f32x16 mfma_fp8_b_sixteenth(const i32x8& a, const i32x8& b, const f32x16& c) {
  return __builtin_amdgcn_mfma_scale_f32_32x32x64_f8f6f4(a, b, c, 0, 0, 0, 0x7f, 0, 0x7b);
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
// four floats -> four E4M3 codes in one dword (round to nearest even; callers keep |x| <= 448).  `old` is
// overwritten: a dead value that already sits in the result's register saves clearing it first.
__device__ __forceinline__ unsigned pack_fp8x4(float a, float b, float c, float d, int old = 0) {
  int w = old;
  w = __builtin_amdgcn_cvt_pk_fp8_f32(a, b, w, false);
  w = __builtin_amdgcn_cvt_pk_fp8_f32(c, d, w, true);
  return (unsigned)w;
}

// ---------------------------------------------------------------- preparation
// One workgroup per (64-key tile, kv head).  Workspace per kv head and tile (8 KB each for D = 128):
//   K:    16-byte chunk ((u * 2 + t) * 2 + c) * 64 + l  = features 64 t + 32 (l / 32) + 16 c .. + 15
//         of key 32 u + l % 32           (u: 32-key half, t: 64-feature half)
//   V^T:  16-byte chunk (db * 2 + c) * 64 + l            = feature 32 db + l % 32 at the 16 keys
//         32 c + 8 i + 4 (l / 32) + e, byte 4 i + e      (the key order in which the accumulator
//         registers of S^T hold keys, so probabilities go into the second product in place)
// Pad keys (beyond the request) are zero codes.
template <int D>
__global__ __launch_bounds__(256) void k_prep_fp8(const int32_t* __restrict__ plan, PlanHeader h,
                                                  const uint8_t* __restrict__ k8,
                                                  const uint8_t* __restrict__ v8, RopeFreq f,
                                                  float2* __restrict__ cs, int hkv, bool rope,
                                                  uint8_t* __restrict__ kw, uint8_t* __restrict__ vw) {
  static_assert(D == 128, "the FP8 path is built for head_dim 128");
  constexpr int CPR = D / 16;                              // 16-byte chunks per key row
  __shared__ uint4 v_s[kStepKeys][CPR + 1];                // V rows of the tile, padded
  const int tile = (int)blockIdx.x / hkv, kvh = (int)blockIdx.x % hkv;
  const int row0 = tile * kStepKeys;                       // first padded key row
  const int32_t* kp = plan + h.off_kpad_start;
  int lo = 0, hi = h.batch;
  while (hi - lo > 1) {
    const int mid = (lo + hi) >> 1;
    if (kp[mid] <= row0) lo = mid; else hi = mid;
  }
  const int b = lo;
  const int tok_base = plan[h.off_tok_start + b];
  const int n_b = plan[h.off_tok_start + b + 1] - tok_base;
  const int key0 = row0 - kp[b];
  const int tid = threadIdx.x;
  uint8_t* k_out = kw + ((int64_t)kvh * h.padded_keys + row0) * D;
  uint8_t* v_out = vw + ((int64_t)kvh * h.padded_keys + row0) * D;
#pragma unroll
  for (int it = 0; it < kStepKeys * CPR / 256; ++it) {
    const int ch = tid + it * 256, key = ch / CPR, c16 = ch % CPR;
    uint4 kx = make_uint4(0, 0, 0, 0), vx = make_uint4(0, 0, 0, 0);
    if (key0 + key < n_b) {
      const int64_t src = (caller_row(plan, h, tok_base + key0 + key) * hkv + kvh) * D + c16 * 16;
      kx = *reinterpret_cast<const uint4*>(k8 + src);
      vx = *reinterpret_cast<const uint4*>(v8 + src);
    }
    const int u = key >> 5, t = c16 >> 2, hh = (c16 >> 1) & 1, c = c16 & 1;
    reinterpret_cast<uint4*>(k_out)[((u * 2 + t) * 2 + c) * 64 + hh * 32 + (key & 31)] = kx;
    v_s[key][c16] = vx;
  }
  __syncthreads();
  const uint8_t* vb = reinterpret_cast<const uint8_t*>(&v_s[0][0]);
  constexpr int VROW = (CPR + 1) * 16;
#pragma unroll
  for (int it = 0; it < (D / 32) * 2 * 64 / 256; ++it) {
    const int ch = tid + it * 256, l = ch & 63, c = (ch >> 6) & 1, db = ch >> 7;
    const int feat = 32 * db + (l & 31), hh = l >> 5;
    unsigned w[4];
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      w[i] = 0;
#pragma unroll
      for (int e = 0; e < 4; ++e)
        w[i] |= (unsigned)vb[(32 * c + 8 * i + 4 * hh + e) * VROW + feat] << (8 * e);
    }
    reinterpret_cast<uint4*>(v_out)[(db * 2 + c) * 64 + l] = make_uint4(w[0], w[1], w[2], w[3]);
  }
  if (rope && kvh == 0) {
    for (int item = tid; item < kStepKeys * (D / 2); item += 256) {
      const int key = item / (D / 2), c = item % (D / 2);
      if (key0 + key < n_b) {
        const int64_t g = tok_base + key0 + key;
        cs[g * (D / 2) + c] = rotary_cos_sin(plan[h.off_pos + g], f.inv_freq[c]);
      }
    }
  }
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

// What bounds it: the matrix pipe, 12 products of 64 cycles and one of 32 per wave and step, and the issue of
// the ~120 VALU instructions of the softmax beside them; hence the products of one tile are issued between
// the softmax of its neighbour, and staging bypasses the registers.  Pass, us, against phases one after the
// other with staging through registers: 4 x (2048 + 8192) tokens, 64/8 heads 8272 / 6978; 512 + 2048, 32/8
// heads 91.3 / 80.0; three requests of 1.5 to 4 K, 40/8 heads (query tiles instead of one wave per head) 300 / 162.
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
  const int i_loc = valid ? mine.t0 + qrow : -1;
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
    stage_v(0); stage_k(2); stage_v(1); stage_k(3); stage_v(2);
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
      rest = (int)pack_fp8x4((x0 - fp8_byte(w, 0)) * 16.0f, (x1 - fp8_byte(w, 1)) * 16.0f,
                             (x2 - fp8_byte(w, 2)) * 16.0f, (x3 - fp8_byte(w, 3)) * 16.0f);
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
  float mref = -INFINITY;                                  // reference of the exponent, log2 units

  // ---- pipeline.  Step j: S^T of tile j + 1 beside the probabilities of tile j, then O^T += V^T P^T of
  // tile j beside the row maxima of tile j + 1.  One set of operand registers serves both products: an
  // operand of K is refilled with one of V^T as soon as it is consumed, and the other way round.
  i32x8 op[4];          // K operand (half u, features 64 t ..) is op[2 t + u]; V^T operand of features 32 db .. is op[db]
  i32x8 pb;             // probabilities of the current tile
#pragma unroll
  for (int w = 0; w < 8; ++w) pb[w] = 0;
  f32x16 sA[2], sB[2];  // score tiles (two 32-key halves each)
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
  bool foreign = false;                                    // the tile of the current scores is such a one
  auto v_chunk = [&](int j) { return (QT && foreign ? ZERO : (NS + (j & (NS - 1))) * CH) + lane; };
  constexpr int KOFF[4] = {0, 2 * 128, 1 * 128, 3 * 128};  // chunk of op[2 t + u]: (2 u + t) * 128
  // product x of the eight of S^T: t = x / 4, high or low term of Q = (x / 2) % 2, u = x % 2
  auto mfma_qk = [&](f32x16 (&s)[2], auto x) __attribute__((always_inline)) {
    constexpr int X = decltype(x)::value, t = X / 4, lo = (X / 2) % 2, u = X % 2;
    if constexpr (X < 2) {
#pragma unroll
      for (int r = 0; r < 16; ++r) s[u][r] = 0.0f;
    }
    if constexpr (lo) s[u] = mfma_fp8_b_sixteenth(op[2 * t + u], qlo[t], s[u]);
    else s[u] = mfma_fp8(op[2 * t + u], qf[t], s[u]);
  };
  // Row predicate: the keys of half u that this lane holds are key0 + 32 u + 4 hh + c,
  // c = 8 (r / 4) + r % 4; the row's visible ones among the 32 become a bit mask, and a score
  // is kept or replaced by -inf with one bit-field extract and one bit-field insert.
  auto apply_mask = [&](f32x16 (&s)[2], int key0) __attribute__((always_inline)) {
    auto low_bits = [](int n) {                            // bits [0, n) of 32, n clamped to [0, 32]
      const unsigned m = (1u << (n & 31)) - 1u;
      return n <= 0 ? 0u : n >= 32 ? 0xffffffffu : m;
    };
#pragma unroll
    for (int u = 0; u < 2; ++u) {
      const int base = key0 + 32 * u + 4 * hh;
      const unsigned vis = low_bits(a_end - base) | (low_bits(i_loc - base + 1) & ~low_bits(b_start - base));
#pragma unroll
      for (int r = 0; r < 16; ++r) {
        const unsigned keep = (unsigned)__builtin_amdgcn_sbfe((int)vis, 8 * (r / 4) + (r % 4), 1);
        s[u][r] = __uint_as_float((__float_as_uint(s[u][r]) & keep) | (0xff800000u & ~keep));
      }
    }
  };
  auto mask_tile = [&](f32x16 (&s)[2], int jt) __attribute__((always_inline)) {
    foreign = false;
    if (__builtin_expect(jt >= mine.n_full, 0)) {
      if constexpr (QT) foreign = jt >= mine.n_a && (jt < mine.jb0 || jt >= mine.jb1);
      apply_mask(s, jt * kStepKeys);
    }
  };
  // Running reference: moved up when a tile's largest exponent exceeds it by more than 0.75 octave
  // (probabilities scaled by 2^8 then stay below 2^8.75 = 431 < 448, the largest E4M3 value).
  auto raise_reference = [&](float mx) __attribute__((always_inline)) {
    mx = pair_max(mx) * c_row;                              // c_row > 0
    const bool raise = mx > mref + 0.75f;                   // (mref = -inf: any visible key)
    if (__builtin_amdgcn_ballot_w64(raise) != 0) {
      const float m_new = raise ? mx : mref;
      const float alpha = mref == -INFINITY ? 0.0f : __builtin_amdgcn_exp2f(mref - m_new);   // 1 when unchanged
      mref = m_new;
#pragma unroll
      for (int r = 0; r < 16; ++r) {
        o[0][r] *= alpha; o[1][r] *= alpha; o[2][r] *= alpha; o[3][r] *= alpha;
      }
      l_run *= alpha;
    }
  };
  auto max_of = [&](float mx, const f32x16& s, auto r0, auto n) __attribute__((always_inline)) {
    constexpr int R0 = decltype(r0)::value, N = decltype(n)::value;
    static_for<0, N / 2>([&](auto i) {
      constexpr int I = R0 + 2 * decltype(i)::value;
      mx = fmaxf(fmaxf(mx, s[I]), s[I + 1]);
    });
    return mx;
  };
  using c0 = std::integral_constant<int, 0>;
  using c8 = std::integral_constant<int, 8>;
  using c16 = std::integral_constant<int, 16>;

  // S^T of tile j + 1 into s_out (QK) and P of tile j from s_in.  The work is issued in groups of one
  // product and the softmax of four scores; exponent argument, exponential and rounding of a score sit in
  // consecutive groups, so that none waits for its input in front of a product.
  auto scores = [&](auto with_qk, int j, f32x16 (&s_in)[2], f32x16 (&s_out)[2]) __attribute__((always_inline)) {
    constexpr bool QK = decltype(with_qk)::value;
    const float bias = mref == -INFINITY ? 0.0f : 8.0f - mref;   // no key seen yet: every S is -inf, p = 0
    const int vc = v_chunk(j);
    float ea[8][4], ex[8][4];
    auto v_arg = [&](auto w) {
      constexpr int W = decltype(w)::value;
      if constexpr (W < 8)
        static_for<0, 4>([&](auto e) {
          constexpr int E = decltype(e)::value;
          ea[W][E] = __builtin_fmaf(s_in[W / 4][4 * (W % 4) + E], c_row, bias);
        });
    };
    v_arg(c0{});
    static_for<0, 8>([&](auto g8) {
      constexpr int X = decltype(g8)::value;
      if constexpr (QK) mfma_qk(s_out, g8);
      __builtin_amdgcn_sched_barrier(0);
      if constexpr (QK && X == 1) {
        // V^T of tile j and K of tile j + 2 have to be there; younger: V^T(j+1), K(j+3), V^T(j+2).  Every
        // wave is done with K of tile j and V^T of tile j - 1, whose slots the loads below refill.
        wait_loads<3 * NREP>();
        __builtin_amdgcn_s_barrier();
        asm volatile("" ::: "memory");
      }
      if constexpr (QK && X >= 2) {                        // K of tile j + 4, then V^T of tile j + 3
        static_for<0, 2 * NREP>([&](auto y) {
          constexpr int Y = decltype(y)::value;
          if constexpr (2 + Y * 6 / (2 * NREP) == X) {
            if constexpr (Y < NREP) stage_one(kw, 0u, j + NS, Y);
            else stage_one(vw, NS * TILE_BYTES, j + NS - 1, Y - NREP);
          }
        });
        if constexpr ((X / 2) % 2) load_op(op[2 * (X / 4) + X % 2], vc + (2 * (X / 4) + X % 2) * 128);
      }
      static_for<0, 4>([&](auto e) {
        constexpr int E = decltype(e)::value;
        ex[X][E] = __builtin_amdgcn_exp2f(ea[X][E]);
        asm volatile("" :: "v"(ex[X][E]));                 // a use in this group: not sunk to the pack
      });
      v_arg(std::integral_constant<int, X + 1>{});
      if constexpr (X > 0) pb[X - 1] = (int)pack_fp8x4(ex[X - 1][0], ex[X - 1][1], ex[X - 1][2], ex[X - 1][3], pb[X - 1]);
      __builtin_amdgcn_sched_barrier(0);
    });
    pb[7] = (int)pack_fp8x4(ex[7][0], ex[7][1], ex[7][2], ex[7][3], pb[7]);
  };
  // The sum over a tile's probabilities.  A query's NaN (a NaN in its Q row, or in a key that its neighbour
  // does not see) meets the zeros of the query that shares its column: such a tile is summed from the codes.
  auto add_row_sum = [&](const f32x4& d) __attribute__((always_inline)) {
    float rs = d[0];
    if (__builtin_expect(__builtin_amdgcn_ballot_w64(rs != rs) != 0, 0)) {
      rs = 0.0f;
#pragma unroll
      for (int w = 0; w < 8; ++w) {
        const unsigned c = (unsigned)pb[w];
        rs += (fp8_byte(c, 0) + fp8_byte(c, 1)) + (fp8_byte(c, 2) + fp8_byte(c, 3));
      }
      rs = pair_sum(rs);
    }
    l_run += rs;
  };
  const f32x4 zero4 = {0.0f, 0.0f, 0.0f, 0.0f};
  // O^T and the row sums (through a tile of ones) of tile j; then the reference for tile j + 1, whose
  // scores are s_next, and the K operands of tile j + 2.
  auto values = [&](int j, f32x16 (&s_next)[2]) __attribute__((always_inline)) {
    const int kc = k_chunk(j + 2);
    o[0] = mfma_fp8(op[0], pb, o[0]);
    __builtin_amdgcn_sched_barrier(0);
    load_op(op[0], kc + KOFF[0]);
    o[1] = mfma_fp8(op[1], pb, o[1]);
    __builtin_amdgcn_sched_barrier(0);
    load_op(op[1], kc + KOFF[1]);
    mask_tile(s_next, step_tile(j + 1));
    const f32x4 row_sum = mfma_fp8_16(ones, pb, zero4);
    __builtin_amdgcn_sched_barrier(0);
    float mx = max_of(s_next[0][0], s_next[0], c0{}, c16{});
    __builtin_amdgcn_sched_barrier(0);
    o[2] = mfma_fp8(op[2], pb, o[2]);
    __builtin_amdgcn_sched_barrier(0);
    load_op(op[2], kc + KOFF[2]);
    mx = max_of(mx, s_next[1], c0{}, c8{});
    __builtin_amdgcn_sched_barrier(0);
    o[3] = mfma_fp8(op[3], pb, o[3]);
    __builtin_amdgcn_sched_barrier(0);
    load_op(op[3], kc + KOFF[3]);
    mx = max_of(mx, s_next[1], c8{}, c8{});
    add_row_sum(row_sum);
    raise_reference(mx);
    __builtin_amdgcn_sched_barrier(0);
  };

  // prologue: S^T of tile 0, its reference, and the K operands of tile 1
  if constexpr (QT) {
#pragma unroll
    for (int n = 0; n < CH / (G * 64); ++n) smem[ZERO + n * (G * 64) + tid] = make_uint4(0u, 0u, 0u, 0u);
    asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");     // the barrier below makes them everyone's
  }
  wait_loads<5 * NREP>();
  __builtin_amdgcn_s_barrier();
  asm volatile("" ::: "memory");
  static_for<0, 4>([&](auto x) { load_op(op[decltype(x)::value], k_chunk(0) + KOFF[decltype(x)::value]); });
  static_for<0, 8>([&](auto x) { mfma_qk(sA, x); });
  static_for<0, 4>([&](auto x) { load_op(op[decltype(x)::value], k_chunk(1) + KOFF[decltype(x)::value]); });
  {
    mask_tile(sA, step_tile(0));
    float mx = max_of(sA[0][0], sA[0], c0{}, c16{});
    mx = max_of(mx, sA[1], c0{}, c16{});
    raise_reference(mx);
  }
  int j = 0;
  for (; j + 2 <= last; j += 2) {
    scores(std::true_type{}, j, sA, sB);
    values(j, sB);
    scores(std::true_type{}, j + 1, sB, sA);
    values(j + 1, sA);
  }
  if (j < last) {
    scores(std::true_type{}, j, sA, sB);
    values(j, sB);
    sA[0] = sB[0]; sA[1] = sB[1];
    ++j;
  }
  // the last tile: probabilities and O^T only
  wait_loads<0>();
  __builtin_amdgcn_s_barrier();
  asm volatile("" ::: "memory");
  static_for<0, 4>([&](auto x) { load_op(op[decltype(x)::value], v_chunk(j) + decltype(x)::value * 128); });
  scores(std::false_type{}, j, sA, sB);
  static_for<0, 4>([&](auto x) {
    constexpr int X = decltype(x)::value;
    o[X] = mfma_fp8(op[X], pb, o[X]);
  });
  add_row_sum(mfma_fp8_16(ones, pb, zero4));
  __syncthreads();                                         // every wave is done with the rings

  // ---- epilogue: l_run holds the row sum of this lane's query.  The result is
  // transposed through LDS so that every row leaves in contiguous pieces.
  const float l_tot = l_run;
  {
    const float inv = v_scale[kvh] / l_tot;
    // (lane r < 32 holds the descriptor of row r); short rows come from the extra workgroups
    const unsigned stored_rows = (unsigned)__builtin_amdgcn_ballot_w64(
        valid && a_end + i_loc - b_start + 1 > PV_SHORT_ROW_KEYS);
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
  if (!grid_1d((int64_t)(h.padded_keys / kStepKeys) * hkv, 256, &grid)) return hipErrorInvalidConfiguration;
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
