// Integer kernels: plan construction (row descriptors, positions, judge rows, tile work list),
// the optional dense mask, plan export and the readout.
#include "pv_internal.h"

namespace pv {

// ---------------------------------------------------------------- upload of the host image
constexpr int kUploadInts = 896;   // 3584 bytes of kernel arguments per launch
struct UploadChunk { int32_t v[kUploadInts]; };

__global__ __launch_bounds__(256) void k_upload(int32_t* dst, UploadChunk c, int n) {
  const int i = blockIdx.x * blockDim.x + threadIdx.x;
  if (i < n) dst[i] = c.v[i];
}

static hipError_t launch_upload(int32_t* plan_dev, const int32_t* host_ints, int n, hipStream_t s) {
  // The image travels in kernel arguments: they are captured at launch, so the host buffer can
  // be released immediately and no pageable-memory copy semantics are involved.
  for (int o = 0; o < n; o += kUploadInts) {
    UploadChunk c;
    const int m = (n - o) < kUploadInts ? (n - o) : kUploadInts;
    for (int i = 0; i < m; ++i) c.v[i] = host_ints[o + i];
    for (int i = m; i < kUploadInts; ++i) c.v[i] = 0;
    k_upload<<<dim3((m + 255) / 256), dim3(256), 0, s>>>(plan_dev + o, c, m);
    hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
  }
  return hipSuccess;
}

// ---------------------------------------------------------------- row descriptors
struct Req {
  int P, T, K, S, N;
  const int32_t* bounds;
};

__device__ inline Req load_req(const int32_t* plan, const PlanHeader& h, int b) {
  Req r;
  r.P = plan[h.off_prompt + b];
  r.T = plan[h.off_draft + b];
  r.K = plan[h.off_nseg + b];
  r.S = plan[h.off_seglen + b];
  r.N = r.P + r.T + r.K * r.S;
  r.bounds = plan + h.off_bounds + plan[h.off_seg_start + b];
  return r;
}

// Visible keys of local row i are [0, a_end) and [b_start, i].  Prompt and draft rows are plain
// causal (a_end = b_start = 0).  A row of segment k sees the prompt and the first p_k draft
// tokens (a_end = P + p_k) and its own segment up to itself (b_start = first row of the
// segment); its rotary position continues from the end of that prefix.
__device__ inline void row_desc(const Req& r, int i, int* pos, int* a_end, int* b_start) {
  const int c = r.P + r.T;
  if (i < c) {
    *pos = i; *a_end = 0; *b_start = 0;
  } else {
    const int k = (i - c) / r.S;
    const int a = (i - c) - k * r.S;
    *a_end = r.P + r.bounds[k];
    *b_start = c + k * r.S;
    *pos = *a_end + a;
  }
}

// Interleaved packing ("Parallel partial verify"): where local token i of the appended order
// [prompt | draft | segments] sits when every segment follows the draft tokens it judges.  A draft
// token is pushed back by the segments whose boundary does not exceed it; segment k comes after
// its p_k draft tokens and the k segments before it.
__device__ inline int interleaved_row(const Req& r, int i) {
  const int c = r.P + r.T;
  if (i < r.P) return i;
  if (i < c) {
    const int t = i - r.P;
    int lo = 0, hi = r.K;          // number of boundaries <= t
    while (lo < hi) {
      const int mid = (lo + hi) >> 1;
      if (r.bounds[mid] <= t) lo = mid + 1; else hi = mid;
    }
    return i + lo * r.S;
  }
  const int k = (i - c) / r.S;
  const int a = (i - c) - k * r.S;
  return r.P + r.bounds[k] + k * r.S + a;
}

// Largest b with start[b] <= x, for a non-decreasing start[0..n] with start[0] = 0 <= x < start[n].
__device__ inline int find_owner(const int32_t* start, int n, int x) {
  int lo = 0, hi = n;            // invariant: start[lo] <= x < start[hi]
  while (hi - lo > 1) {
    const int mid = (lo + hi) >> 1;
    if (start[mid] <= x) lo = mid; else hi = mid;
  }
  // skip empty owners (start[lo] == start[lo+1]) cannot happen for lo returned here because
  // start[lo] <= x < start[lo+1] after the loop.
  return lo;
}

// Row g of the packed batch (and, for g < total_segments, judge row g).  `img` is where the
// uploaded part of the plan is read from (the plan itself, or a copy in LDS).  causal_short: the rows with few
// keys are the first PV_SHORT_ROW_KEYS rows of every request and their list is written here.
__device__ inline void plan_token(int32_t* plan, const int32_t* img, const PlanHeader& h, int g, bool causal_short) {
  if (causal_short && g < h.n_short_rows) {
    const int base = img[h.off_tok_start + g / PV_SHORT_ROW_KEYS];
    reinterpret_cast<int4*>(plan + h.off_short)[g] = make_int4(base + g % PV_SHORT_ROW_KEYS, base, 0, 0);
  }
  if (g < h.total_tokens) {
    const int b = find_owner(img + h.off_tok_start, h.batch, g);
    const Req r = load_req(img, h, b);
    int pos, ae, bs;
    row_desc(r, g - img[h.off_tok_start + b], &pos, &ae, &bs);
    plan[h.off_pos + g] = pos;
    plan[h.off_aend + g] = ae;
    plan[h.off_bstart + g] = bs;
    if (h.layout == PV_LAYOUT_INTERLEAVED)
      plan[h.off_map + g] = img[h.off_tok_start + b] + interleaved_row(r, g - img[h.off_tok_start + b]);
  }
  if (g < h.total_segments) {
    const int b = find_owner(img + h.off_seg_start, h.batch, g);
    const Req r = load_req(img, h, b);
    const int k = g - img[h.off_seg_start + b];
    // the verdict of segment k is read at its last token (a row of the caller's tensors)
    const int last = r.P + r.T + (k + 1) * r.S - 1;
    plan[h.off_judge + g] = img[h.off_tok_start + b] +
                            (h.layout == PV_LAYOUT_INTERLEAVED ? interleaved_row(r, last) : last);
  }
}

// The up to h.tile_m rows from local row t0 of request b on as a query tile: the union of their visible key sets, in
// key-tile units.
__device__ inline QTile tile_at(const int32_t* plan, const PlanHeader& h, int b, const Req& r, int t0) {
  const int rows = min(h.tile_m, r.N - t0);
  const int bn = h.tile_n;
  int min_prefix = 0x7fffffff;   // min over rows of the length of the fully visible key prefix
  int max_low = 0;               // max over rows of the end of the low range
  int min_b = 0x7fffffff, max_i = -1;
  // The rows of a tile are consecutive, causal rows first.  Their low range ends at i + 1, which
  // grows with i; a segment row's ends at P + p_k and its second range starts at the segment's
  // first row, both non-decreasing in k because the boundaries are sorted.  The extremes over the
  // tile therefore sit at the first and last row of each kind.
  const int c = r.P + r.T, last = t0 + rows - 1;
  if (t0 < c) {
    min_prefix = t0 + 1;
    max_low = min(last, c - 1) + 1;
  }
  if (last >= c) {
    int pos, ae0, bs0, ae1, bs1;
    row_desc(r, max(t0, c), &pos, &ae0, &bs0);
    row_desc(r, last, &pos, &ae1, &bs1);
    min_prefix = min(min_prefix, ae0);
    max_low = max(max_low, ae1);
    min_b = bs0;
    max_i = last;
  }
  QTile q;
  q.tok_base = plan[h.off_tok_start + b];
  q.t0 = t0;
  q.rows = rows;
  q.n_full = min_prefix / bn;
  q.n_a = (max_low + bn - 1) / bn;
  if (max_i >= 0) {
    q.jb0 = max(q.n_a, min_b / bn);
    q.jb1 = max(q.jb0, max_i / bn + 1);
  } else {
    q.jb0 = q.n_a; q.jb1 = q.n_a;
  }
  q.kpad_base = plan[h.off_kpad_start + b];
  return q;
}

// Query tile t.  *seg_slot is its place in the list of tiles that hold segment rows (request after request), -1 if it
// holds none.
__device__ inline QTile plan_tile(const int32_t* plan, const PlanHeader& h, int t, int* seg_slot) {
  const int b = find_owner(plan + h.off_qtile_start, h.batch, t);
  const Req r = load_req(plan, h, b);
  const int t0 = (t - plan[h.off_qtile_start + b]) * h.tile_m;
  const QTile q = tile_at(plan, h, b, r, t0);
  const int c = r.P + r.T;
  *seg_slot = t0 + q.rows > c ? plan[h.off_segtile_start + b] + t0 / h.tile_m - c / h.tile_m : -1;
  return q;
}

// What the segment-only call evaluates in the place of the slot-th tile with segment rows.  Where segments are whole
// numbers of tiles long, the tiles are cut at the segments' first rows: a tile of two segments masks every key between
// their boundaries (a step of masked keys takes 0.8 us, one in the open 0.6), and there is one more of them (rows = 0
// in its place).  Segment rows of 32 tokens at 32/8 heads, us, as listed / cut anew: 16 ragged requests 390 / 361, 8 of
// 2.8 K tokens 152 / 134, 3 of them 78 / 67, one of 9 K 77 / 67.
__device__ inline QTile segment_tile(const int32_t* plan, const PlanHeader& h, int slot, int* listed_t0) {
  const int b = find_owner(plan + h.off_segtile_start, h.batch, slot);
  const Req r = load_req(plan, h, b);
  const int c = r.P + r.T, i = slot - plan[h.off_segtile_start + b];
  *listed_t0 = (c / h.tile_m + i) * h.tile_m;
  const int t0 = r.S % h.tile_m == 0 ? c + i * h.tile_m : *listed_t0;
  QTile q = tile_at(plan, h, b, r, min(t0, r.N - 1));
  if (t0 >= r.N) q.rows = 0;
  return q;
}
__device__ inline void plan_segment_tile(int32_t* plan, const int32_t* img, const PlanHeader& h, int slot) {
  int listed_t0;
  const QTile q = segment_tile(img, h, slot, &listed_t0);
  reinterpret_cast<QTile*>(plan + h.off_segtile)[(q.kpad_base + listed_t0) / h.tile_m] = q;
}

// Group qd of four consecutive query tiles of a request (the last group of a request may hold
// fewer): the union of their key-tile lists, for the launch whose workgroups take four query tiles
// of one head.  Every wave of such a workgroup masks with its own tile's descriptor, so key tiles
// that only some of the four need are simply fully masked for the others.  `n_full` of the result
// carries the index of the group's first tile in the tile list instead.  The groups of a request are
// listed last first (the last group has the longest key list).  Four neighbouring lanes take the four
// tiles (one thread after the other's tile is four chains of dependent reads and divisions); all four
// call this together, `lane4` = their place.
__device__ inline void plan_quad(int32_t* plan, const int32_t* img, const PlanHeader& h, int qd, int lane4) {
  const int b = find_owner(img + h.off_quad_start, h.batch, qd);
  const int q0 = img[h.off_quad_start + b], nq = img[h.off_quad_start + b + 1] - q0;
  const int ql = qd - q0;
  const int t_first = img[h.off_qtile_start + b] + 4 * ql;
  const int t = t_first + lane4, t_last = img[h.off_qtile_start + b + 1] - 1;
  int unused;
  QTile u = plan_tile(img, h, min(t, t_last), &unused);
  const bool two = u.jb1 > u.jb0;                // the tile has a second range
  int rows = t <= t_last ? u.rows : 0, n_a = u.n_a;
  int jb0 = two ? u.jb0 : 0x7fffffff, jb1 = two ? u.jb1 : -1;
#pragma unroll
  for (int off = 1; off < 4; off <<= 1) {
    rows += __shfl_xor(rows, off);
    n_a = max(n_a, __shfl_xor(n_a, off));
    jb0 = min(jb0, __shfl_xor(jb0, off));
    jb1 = max(jb1, __shfl_xor(jb1, off));
  }
  if (lane4 != 0) return;
  u.rows = rows;
  u.n_a = n_a;
  u.jb0 = jb1 >= 0 ? max(jb0, n_a) : n_a;
  u.jb1 = max(jb1, u.jb0);
  u.n_full = t_first;
  reinterpret_cast<QTile*>(plan + h.off_quadwork)[q0 + (nq - 1 - ql)] = u;
}

// Inclusive sum over the lanes of a wave, and sum and maximum over all of them, in every lane (non-negative numbers):
// shifts inside the rows of 16 lanes, then the rows' last lanes handed on.  A tenth of the time of exchanges through LDS,
// of which a plan would have a dozen in its longest chain.
__device__ __forceinline__ int wave_scan(int x) {
  x += __builtin_amdgcn_update_dpp(0, x, 0x111, 0xf, 0xf, true);     // row_shr 1, 2, 4, 8
  x += __builtin_amdgcn_update_dpp(0, x, 0x112, 0xf, 0xf, true);
  x += __builtin_amdgcn_update_dpp(0, x, 0x114, 0xf, 0xf, true);
  x += __builtin_amdgcn_update_dpp(0, x, 0x118, 0xf, 0xf, true);
  x += __builtin_amdgcn_update_dpp(0, x, 0x142, 0xa, 0xf, false);    // row_bcast 15 into rows 1 and 3
  x += __builtin_amdgcn_update_dpp(0, x, 0x143, 0xc, 0xf, false);    // row_bcast 31 into rows 2 and 3
  return x;
}
__device__ __forceinline__ int wave_sum(int x) { return __builtin_amdgcn_readlane(wave_scan(x), 63); }
__device__ __forceinline__ int wave_max(int x) {
  x = max(x, __builtin_amdgcn_update_dpp(0, x, 0x111, 0xf, 0xf, true));
  x = max(x, __builtin_amdgcn_update_dpp(0, x, 0x112, 0xf, 0xf, true));
  x = max(x, __builtin_amdgcn_update_dpp(0, x, 0x114, 0xf, 0xf, true));
  x = max(x, __builtin_amdgcn_update_dpp(0, x, 0x118, 0xf, 0xf, true));
  x = max(x, __builtin_amdgcn_update_dpp(0, x, 0x142, 0xa, 0xf, false));
  x = max(x, __builtin_amdgcn_update_dpp(0, x, 0x143, 0xc, 0xf, false));
  return __builtin_amdgcn_readlane(x, 63);
}

// The key pieces of the segment-only call, for a plan whose segment tiles alone would leave workgroup slots empty:
// pieces of nearly equal length, the shortest length L (at least kMinPiece key tiles) whose pieces fit the places.
// One workgroup of kPlanThreads; thread i has the i-th tile with segment rows, the waves try 64 lengths at a time.
// (Every tile in the same number of pieces leaves long ones, and a number rounded up so that they fill the slots a second
// round of workgroups.  Passes, us, before / with it: 64/8 heads, 3 K tokens 76.4 / 61.0; 28/4 heads 62.6 / 46.8; 40/8
// heads 65.4 / 55.5; 32/8 heads, 9 K tokens 90.5 / 77.5.  Pieces of 2 to 9 key tiles at least: the same.)
constexpr int kPlanThreads = 1024;
__device__ inline void plan_seg_units(int32_t* plan, const int32_t* img, const PlanHeader& h) {
  constexpr int W = kPlanThreads / 64, TRIES = 4 * W;  // lengths tried in a round, four a wave
  static_assert(TRIES == 64, "a lane each");
  __shared__ int cost_s[512], sum_s[TRIES];
  const int tid = (int)threadIdx.x, lane = tid & 63, wave = tid >> 6, n = h.n_seg_tiles, cap = h.n_seg_units;   // n < 512
  QTile q = {};
  int cost = 0;
  if (tid < n) {
    int unused;
    q = segment_tile(img, h, tid, &unused);
    cost = q.rows > 0 ? q.n_a + (q.jb1 - q.jb0) : 0;
  }
  if (tid < 512) cost_s[tid] = cost;
  __syncthreads();
  // min(ceil(c / len), 8) by the reciprocal: (c - 1/2) / len is at least 1 / (2 len) from a whole number, and below 8
  // the product's error is less for every len under 2^18 and c under len * 8
  auto pieces_of = [](int c, float rcp) { return c > 0 ? min((int)(((float)c - 0.5f) * rcp) + 1, kMaxPieces) : 0; };
  int hi = 1;
  for (int i = lane; i < n; i += 64) hi = max(hi, cost_s[i]);
  hi = wave_max(hi);
  int lo = min(kMinPiece, hi);                       // the answer is in [lo, hi]: pieces of length hi are the n tiles
  while (lo < hi) {
    const int step = (hi - lo + TRIES - 1) / TRIES;
    int total[2] = {0, 0};                           // two sums of at most 8 * 512 in a number
    float rcp[4];
#pragma unroll
    for (int k = 0; k < 4; ++k) rcp[k] = __builtin_amdgcn_rcpf((float)min(lo + (4 * wave + k) * step, hi));
    for (int i = lane; i < n; i += 64) {
      const int c = cost_s[i];
      total[0] += pieces_of(c, rcp[0]) + (pieces_of(c, rcp[1]) << 16);
      total[1] += pieces_of(c, rcp[2]) + (pieces_of(c, rcp[3]) << 16);
    }
    const int sum0 = wave_sum(total[0]), sum1 = wave_sum(total[1]);
    if (lane < 4) sum_s[4 * wave + lane] = ((lane & 2 ? sum1 : sum0) >> (16 * (lane & 1))) & 0xffff;
    __syncthreads();
    const int first = __popcll(__builtin_amdgcn_ballot_w64(sum_s[lane] > cap));   // the lengths that don't fit come first
    __syncthreads();
    const int lo0 = lo;
    lo = first > 0 ? min(lo0 + (first - 1) * step + 1, hi) : lo0;
    hi = first < TRIES ? min(lo0 + first * step, hi) : hi;
  }
  const int p = tid < n ? pieces_of(cost, __builtin_amdgcn_rcpf((float)lo)) : 0;
  const int at = wave_scan(p);                       // inclusive sum over the threads
  if (lane == 63) sum_s[wave] = at;
  __syncthreads();
  const int sum = lane < W ? sum_s[lane & (W - 1)] : 0;
  const int used = wave_sum(sum), before = wave_sum(lane < wave ? sum : 0);
  SegUnit* units = reinterpret_cast<SegUnit*>(plan + h.off_segunit);
  SegUnit u;
  u.tile = q;
  u.pieces = p;
  for (int c = 0; c < p; ++c) {
    u.piece = c;
    u.kt0 = c * cost / p;
    u.n_kt = (c + 1) * cost / p - u.kt0;
    units[before + at - p + c] = u;
  }
  for (int i = used + tid; i < cap; i += kPlanThreads) units[i].n_kt = 0;
}
// (a plan too large for plan_all)
__global__ __launch_bounds__(kPlanThreads) void k_plan_units(int32_t* plan, PlanHeader h) { plan_seg_units(plan, plan, h); }

// Threads, whole waves, in front of those of the tokens: the tiles of the segment-only call.
__host__ __device__ inline int segment_tile_threads(const PlanHeader& h) { return (h.n_seg_tiles + 63) & ~63; }

// The whole plan in one launch.  The request data (in the kernel arguments, or uploaded before) are copied to LDS by
// every workgroup, and no workgroup reads what another writes: a workgroup that ranks kRankTiles tiles, a wave each,
// forms the costs of all tiles itself.  That is two tiles a thread at 1 766 tiles (a tile is a chain of LDS reads and
// divisions of 0.7 us: with 256 threads to a workgroup and seven tiles a thread the launch took 11.5 us), against a
// launch of its own for the ranking and its wait for the tiles.  Longest first, ties in the order of the tiles: the
// cost, the tile's index from the end and whether it holds segment rows make one number.  Launches, us, in two or
// three kernels / with it: 16 ragged requests of 55 K tokens 22.5 / 7.3 (16 lanes to a tile 9.8: too few compute units
// with work); one workgroup that ranked all tiles / with it: 208 tiles 11.9 / 5.1, 96 tiles 5.6 / 5.0.
constexpr int kRankTiles = kPlanThreads / 64, kPlanTiles = 4096, kPlanData = 4096;   // (tiles and ints of request data in LDS)
__device__ inline void plan_all(int32_t* plan, const int32_t* img, unsigned* key_s, const PlanHeader& h, int rank_blocks,
                                int quad_blocks, bool causal_short) {
  const int tid = (int)threadIdx.x;
  int blk = (int)blockIdx.x;
  if (h.n_seg_units > 0 && blk-- == 0) {             // the longest chain first
    plan_seg_units(plan, img, h);
    return;
  }
  if (blk >= rank_blocks + quad_blocks) {
    const int x = (blk - rank_blocks - quad_blocks) * kPlanThreads + tid;
    const int seg_tiles = segment_tile_threads(h);
    if (x >= seg_tiles) plan_token(plan, img, h, x - seg_tiles, causal_short);
    else if (x < h.n_seg_tiles) plan_segment_tile(plan, img, h, x);
    return;
  }
  if (blk >= rank_blocks) {
    const int qd = (blk - rank_blocks) * (kPlanThreads / 4) + (tid >> 2);
    if (qd < h.n_quads) plan_quad(plan, img, h, qd, tid & 3);
    return;
  }
  const int n = h.n_q_tiles, n_padded = (n + 255) & ~255;
  static_assert((1 << 24) / kTileN + 8 < 1 << 19 && kPlanTiles <= 1 << 12, "cost, tile and flag fit 32 bits");
  __shared__ QTile mine_s[kRankTiles];
  for (int t = tid; t < n_padded; t += kPlanThreads) {
    unsigned key = 0u;               // a cost is at least 1: zero comes behind every tile
    if (t < n) {
      int seg_slot;
      const QTile q = plan_tile(img, h, t, &seg_slot);
      key = (unsigned)(q.n_a + (q.jb1 - q.jb0)) << 13 | (unsigned)(kPlanTiles - 1 - t) << 1 | (unsigned)(seg_slot >= 0);
      if (t / kRankTiles == blk) mine_s[t % kRankTiles] = q;
    }
    key_s[t] = key;
  }
  __syncthreads();
  const int t = blk * kRankTiles + (tid >> 6), lane = tid & 63;
  if (t >= n) return;
  const unsigned my_key = key_s[t];
  int rank = 0, seg_rank = 0;      // among all tiles, among those that hold segment rows
  for (int x = lane * 4; x < n_padded; x += 256) {
    const uint4 k4 = *reinterpret_cast<const uint4*>(key_s + x);
    const unsigned ks[4] = {k4.x, k4.y, k4.z, k4.w};
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      const unsigned before = ks[e] > my_key;
      rank += before;
      seg_rank += before & ks[e];
    }
  }
  rank = wave_sum(rank);
  seg_rank = wave_sum(seg_rank);
  if (lane == 0) {
    const QTile mine = mine_s[tid >> 6];
    reinterpret_cast<QTile*>(plan + h.off_tiles)[t] = mine;
    reinterpret_cast<QTile*>(plan + h.off_work)[rank] = mine;
    if (my_key & 1u) reinterpret_cast<QTile*>(plan + h.off_segwork)[seg_rank] = mine;
  }
}
// n_img ints of the arguments are the start of the plan (its last workgroup, one of tokens, writes them there).
__global__ __launch_bounds__(kPlanThreads) void k_plan_args(int32_t* plan, PlanHeader h, UploadChunk c, int n_img,
                                                            int rank_blocks, int quad_blocks, bool causal_short) {
  __shared__ int32_t img_s[kUploadInts];
  __shared__ __align__(16) unsigned key_s[kPlanTiles];
  for (int i = threadIdx.x; i < n_img; i += kPlanThreads) {
    const int32_t x = c.v[i];
    if (blockIdx.x == gridDim.x - 1) plan[i] = x;
    img_s[i] = x;
  }
  __syncthreads();
  plan_all(plan, img_s, key_s, h, rank_blocks, quad_blocks, causal_short);
}
// The request data are in the plan already.
__global__ __launch_bounds__(kPlanThreads) void k_plan_uploaded(int32_t* plan, PlanHeader h, int n_data,
                                                                int rank_blocks, int quad_blocks, bool causal_short) {
  __shared__ int32_t img_s[kPlanData];
  __shared__ __align__(16) unsigned key_s[kPlanTiles];
  for (int i = threadIdx.x; i < n_data; i += kPlanThreads) img_s[i] = plan[i];
  __syncthreads();
  plan_all(plan, img_s, key_s, h, rank_blocks, quad_blocks, causal_short);
}

// Beyond those limits (a workgroup for every 16 tiles would form too many costs): per-token arrays, tiles and groups
// of tiles in one launch, a range of workgroups for each, then the ranking.
__global__ __launch_bounds__(256) void k_plan_build(int32_t* plan, PlanHeader h, int tile_blocks, int quad_blocks,
                                                    bool causal_short) {
  const int blk = (int)blockIdx.x, tid = (int)threadIdx.x;
  if (blk < tile_blocks) {
    const int t = blk * 256 + tid;
    if (t < h.n_q_tiles) {
      int seg_slot;
      const QTile q = plan_tile(plan, h, t, &seg_slot);
      reinterpret_cast<QTile*>(plan + h.off_tiles)[t] = q;
      if (seg_slot >= 0) reinterpret_cast<QTile*>(plan + h.off_segwork)[h.n_seg_tiles + seg_slot] = q;   // sorted below
    }
  } else if (blk < tile_blocks + quad_blocks) {
    const int qd = (blk - tile_blocks) * 64 + (tid >> 2);
    if (qd < h.n_quads) plan_quad(plan, plan, h, qd, tid & 3);
  } else {
    const int x = (blk - tile_blocks - quad_blocks) * 256 + tid, seg_tiles = segment_tile_threads(h);
    if (x >= seg_tiles) plan_token(plan, plan, h, x - seg_tiles, causal_short);
    else if (x < h.n_seg_tiles) plan_segment_tile(plan, plan, h, x);
  }
}

// Longest-first order (stable) of the query tiles and of those that hold segment rows: rank = number of tiles that
// must run before this one.  One wave per four tiles; its lanes share the comparisons against all other tiles, whose
// costs they read eight at a time: one read per round trip and one tile per wave left the launch waiting for L2.
// (Segment rows of 16 ragged requests in the order of the requests: 2472 items of 7 to 78 key tiles on 512 slots
// leave 21 % of the launch to its tail; sorted, 2 %.)
constexpr int kSortTiles = 4, kSortReads = 8;
__global__ __launch_bounds__(256) void k_plan_sort(int32_t* plan, PlanHeader h, int tile_blocks) {
  const bool seg = (int)blockIdx.x >= tile_blocks;                 // the blocks behind those of all tiles
  const int n = seg ? h.n_seg_tiles : h.n_q_tiles, lane = threadIdx.x & 63;
  const int t0 = (((int)blockIdx.x - (seg ? tile_blocks : 0)) * 4 + ((int)threadIdx.x >> 6)) * kSortTiles;
  if (t0 >= n) return;                          // whole waves leave together
  QTile* dst = reinterpret_cast<QTile*>(plan + (seg ? h.off_segwork : h.off_work));
  const QTile* tiles = seg ? dst + n : reinterpret_cast<const QTile*>(plan + h.off_tiles);
  auto cost = [&](int t) { return tiles[t].n_a + (tiles[t].jb1 - tiles[t].jb0); };
  int mine[kSortTiles], rank[kSortTiles];
#pragma unroll
  for (int i = 0; i < kSortTiles; ++i) { mine[i] = cost(min(t0 + i, n - 1)); rank[i] = 0; }
  for (int u0 = lane; u0 < n; u0 += 64 * kSortReads) {
    int c[kSortReads];
#pragma unroll
    for (int r = 0; r < kSortReads; ++r) c[r] = cost(min(u0 + 64 * r, n - 1));
#pragma unroll
    for (int r = 0; r < kSortReads; ++r) {
      const int u = u0 + 64 * r;
#pragma unroll
      for (int i = 0; i < kSortTiles; ++i)
        rank[i] += u < n && (c[r] > mine[i] || (c[r] == mine[i] && u < t0 + i));
    }
  }
  int my_rank = 0;
#pragma unroll
  for (int i = 0; i < kSortTiles; ++i) {
#pragma unroll
    for (int off = 32; off > 0; off >>= 1) rank[i] += __shfl_xor(rank[i], off);
    if (lane == i) my_rank = rank[i];
  }
  if (lane < kSortTiles && t0 + lane < n) dst[my_rank] = tiles[t0 + lane];
}

// Dense mask from the stored row descriptors (what the attention kernels consume).
__global__ __launch_bounds__(256) void k_dense_mask(const int32_t* plan, PlanHeader h, uint8_t* mask) {
  const int g = blockIdx.x;      // packed row
  const int b = find_owner(plan + h.off_tok_start, h.batch, g);
  const int base = plan[h.off_tok_start + b];
  const int n = plan[h.off_tok_start + b + 1] - base;
  const int i = g - base;
  const int ae = plan[h.off_aend + g], bs = plan[h.off_bstart + g];
  const int64_t* mask_start = reinterpret_cast<const int64_t*>(plan + h.off_mask_start);
  // rows and columns of the mask follow the caller's row order
  uint8_t* row = mask + mask_start[b] + (caller_row(plan, h, g) - base) * n;
  for (int j = threadIdx.x; j < n; j += blockDim.x)
    row[caller_row(plan, h, base + j) - base] = (j < ae) || (j >= bs && j <= i) ? 1 : 0;
}

hipError_t launch_plan_kernels(int32_t* plan_dev, const PlanHeader& h, const int32_t* host_ints,
                               int n_img, bool causal_short, uint8_t* dense_mask, hipStream_t s) {
  hipError_t e = hipSuccess;
  const int n1 = h.total_tokens > h.total_segments ? h.total_tokens : h.total_segments;
  // The host image: all of it in the arguments of the launch that uses it, or the request data there and the rows
  // with few keys behind them written by the launch (the first ones of every request) or uploaded, or all uploaded.
  const bool in_args = h.off_short <= kUploadInts;
  const int n_args = n_img <= kUploadInts ? n_img : in_args ? h.off_short : 0;
  if (n_img <= kUploadInts) causal_short = false;
  const bool one_launch = h.n_q_tiles <= kPlanTiles && h.off_short <= kPlanData;
  const int n_upload = causal_short ? h.off_short : n_img, uploaded = one_launch ? n_args : 0;
  if (uploaded < n_upload) {
    e = launch_upload(plan_dev + uploaded, host_ints + uploaded, n_upload - uploaded, s);
    if (e != hipSuccess) return e;
  }
  if (one_launch) {
    const int rank_blocks = (h.n_q_tiles + kRankTiles - 1) / kRankTiles;
    const int quad_blocks = (4 * h.n_quads + kPlanThreads - 1) / kPlanThreads;
    const int token_blocks = (segment_tile_threads(h) + n1 + kPlanThreads - 1) / kPlanThreads;
    const dim3 grid((h.n_seg_units > 0 ? 1 : 0) + rank_blocks + quad_blocks + token_blocks);
    if (n_args > 0) {
      UploadChunk c;
      for (int i = 0; i < n_args; ++i) c.v[i] = host_ints[i];
      for (int i = n_args; i < kUploadInts; ++i) c.v[i] = 0;
      k_plan_args<<<grid, dim3(kPlanThreads), 0, s>>>(plan_dev, h, c, n_args, rank_blocks, quad_blocks, causal_short);
    } else {
      k_plan_uploaded<<<grid, dim3(kPlanThreads), 0, s>>>(plan_dev, h, h.off_short, rank_blocks, quad_blocks,
                                                          causal_short);
    }
    e = hipGetLastError();
    if (e != hipSuccess) return e;
  } else {
    const int tile_blocks = (h.n_q_tiles + 255) / 256, quad_blocks = (h.n_quads + 63) / 64;
    const dim3 grid(tile_blocks + quad_blocks + (segment_tile_threads(h) + n1 + 255) / 256);
    k_plan_build<<<grid, dim3(256), 0, s>>>(plan_dev, h, tile_blocks, quad_blocks, causal_short);
    e = hipGetLastError();
    if (e != hipSuccess) return e;
    constexpr int kPerBlock = 4 * kSortTiles;
    const int sort_blocks = (h.n_q_tiles + kPerBlock - 1) / kPerBlock, seg_blocks = (h.n_seg_tiles + kPerBlock - 1) / kPerBlock;
    k_plan_sort<<<dim3(sort_blocks + seg_blocks), dim3(256), 0, s>>>(plan_dev, h, sort_blocks);
    e = hipGetLastError();
    if (e != hipSuccess) return e;
    if (h.n_seg_units > 0) {
      k_plan_units<<<dim3(1), dim3(kPlanThreads), 0, s>>>(plan_dev, h);
      e = hipGetLastError();
      if (e != hipSuccess) return e;
    }
  }
  if (dense_mask) {
    dim3 grid;
    if (!grid_1d(h.total_tokens, 256, &grid)) return hipErrorInvalidConfiguration;
    k_dense_mask<<<grid, dim3(256), 0, s>>>(plan_dev, h, dense_mask);
    e = hipGetLastError();
  }
  return e;
}

// ---------------------------------------------------------------- export
__global__ __launch_bounds__(256) void k_export(const int32_t* plan, PlanHeader h, int32_t* pos,
                                                int32_t* aend, int32_t* bstart, int32_t* judge) {
  const int g = blockIdx.x * blockDim.x + threadIdx.x;
  if (g < h.total_tokens) {
    const int64_t row = caller_row(plan, h, g);
    if (pos) pos[row] = plan[h.off_pos + g];
    if (aend) aend[row] = plan[h.off_aend + g];
    if (bstart) bstart[row] = plan[h.off_bstart + g];
  }
  if (judge && g < h.total_segments) judge[g] = plan[h.off_judge + g];
}

hipError_t launch_plan_export(const int32_t* plan_dev, const PlanHeader& h, int32_t* pos,
                              int32_t* aend, int32_t* bstart, int32_t* judge, hipStream_t s) {
  const int n1 = h.total_tokens > h.total_segments ? h.total_tokens : h.total_segments;
  k_export<<<dim3((n1 + 255) / 256), dim3(256), 0, s>>>(plan_dev, h, pos, aend, bstart, judge);
  return hipGetLastError();
}

// ---------------------------------------------------------------- readout
// One wave per request: lane l takes segments l, l + 64, ..., so the logits of a request arrive
// in one round of loads; the three per-request quantities are then a min, a max and a sum over
// the wave.  A verdict is Correct iff the fp64 margin l_C - l_I is non-negative (ties count as
// Correct) and reaches the threshold.
__global__ __launch_bounds__(256) void k_first_reject(const int32_t* plan, PlanHeader h,
                                                      const float* logits, double thr, int mode,
                                                      int32_t* out) {
  const int b = blockIdx.x * 4 + (threadIdx.x >> 6), lane = threadIdx.x & 63;
  if (b >= h.batch) return;                     // whole waves leave together
  const int s0 = plan[h.off_seg_start + b];
  const int K = plan[h.off_nseg + b];
  const int32_t* bounds = plan + h.off_bounds + s0;
  int first = K, last_ok = -1, bad = 0;
  for (int k = lane; k < K; k += 64) {
    const float2 lg = reinterpret_cast<const float2*>(logits)[s0 + k];
    const double d = (double)lg.x - (double)lg.y;
    const bool ok = (d >= 0.0) && (d >= thr);
    if (ok) last_ok = k;                        // k grows: the last one written is the largest
    else { bad++; first = min(first, k); }
  }
#pragma unroll
  for (int off = 32; off > 0; off >>= 1) {
    first = min(first, __shfl_xor(first, off));
    last_ok = max(last_ok, __shfl_xor(last_ok, off));
    bad += __shfl_xor(bad, off);
  }
  if (lane == 0) {
    const int k_star = (mode == 0) ? first - 1 : last_ok;
    int4 o;
    o.x = first;
    o.y = k_star;
    o.z = k_star >= 0 ? bounds[k_star] : 0;
    o.w = bad;
    reinterpret_cast<int4*>(out)[b] = o;
  }
}

hipError_t launch_first_reject(const int32_t* plan_dev, const PlanHeader& h, const float* logits,
                               double thr, int mode, int32_t* out, hipStream_t s) {
  k_first_reject<<<dim3((h.batch + 3) / 4), dim3(256), 0, s>>>(plan_dev, h, logits, thr, mode, out);
  return hipGetLastError();
}

// ---------------------------------------------------------------- decision policy
// One thread per request; every comparison in fp64 on the margin l_C - l_I.
__global__ __launch_bounds__(64) void k_decide(const int32_t* plan, PlanHeader h, const float* logits,
                                               const float* full_logits, pv_policy pol,
                                               int32_t* out) {
  const int b = blockIdx.x * blockDim.x + threadIdx.x;
  if (b >= h.batch) return;
  const int s0 = plan[h.off_seg_start + b];
  const int K = plan[h.off_nseg + b];
  const int32_t* bounds = plan + h.off_bounds + s0;
  int first = K, bad = 0, trailing = 0, below = 0, argmin = -1;
  double dmin = 0.0;
  for (int k = 0; k < K; ++k) {
    const double d = (double)logits[2 * (s0 + k)] - (double)logits[2 * (s0 + k) + 1];
    const bool ok = (d >= 0.0) && (d >= pol.margin_chunk);
    if (ok) trailing = 0;
    else { bad++; trailing++; if (first == K) first = k; }
    if (d < pol.margin_chunk_relaxed) below++;
    if (argmin < 0 || d < dmin) { argmin = k; dmin = d; }
  }
  const int k_star = first - 1;
  const bool rejects = (K > 0 && (double)bad > pol.rho * (double)K) ||
                       (pol.kappa > 0 && trailing >= pol.kappa);
  const int m = (int)floor(fmax(0.0, (double)k_star + 1.0 - pol.eta));
  const int l_star = m >= 1 ? bounds[m - 1] : 0;
  const int handoff = l_star > 0 ? PV_LABEL_SM_LG : PV_LABEL_LG;
  int label, stage, v_full = -1;
  if (pol.premature) {
    const bool abort = rejects || below >= pol.relaxed_count_min;
    label = abort ? handoff : -1;
    stage = abort ? 1 : 0;
  } else {
    const double df = (double)full_logits[2 * b] - (double)full_logits[2 * b + 1];
    v_full = (df >= 0.0) && (df >= pol.margin_full);
    if (v_full) { label = PV_LABEL_SM; stage = 2; }
    else if (K >= 1 && K <= pol.n_short && df >= pol.margin_short[K - 1]) { label = PV_LABEL_SM; stage = 3; }
    else if (df >= pol.margin_full_relaxed && below == 0) { label = PV_LABEL_SM; stage = 5; }
    else { label = handoff; stage = 6; }
  }
  int32_t* o = out + 12 * b;
  o[0] = label; o[1] = stage; o[2] = l_star; o[3] = k_star; o[4] = first; o[5] = bad;
  o[6] = trailing; o[7] = rejects ? 1 : 0; o[8] = below; o[9] = v_full; o[10] = argmin; o[11] = K;
}

hipError_t launch_decide(const int32_t* plan_dev, const PlanHeader& h, const float* logits,
                         const float* full_logits, const pv_policy& pol, int32_t* out, hipStream_t s) {
  k_decide<<<dim3((h.batch + 63) / 64), dim3(64), 0, s>>>(plan_dev, h, logits, full_logits, pol, out);
  return hipGetLastError();
}

// ---------------------------------------------------------------- judge logits
// One wave per segment: lanes stride over the hidden dimension in 16-byte pieces, two fp32 dot
// products, then a fixed-order butterfly reduction (bit-reproducible).
__global__ __launch_bounds__(256) void k_judge_logits(const int32_t* plan, PlanHeader h,
                                                      const uint16_t* hidden, const uint16_t* w2,
                                                      int hs, float* logits) {
  const int seg = blockIdx.x * 4 + (threadIdx.x >> 6), lane = threadIdx.x & 63;
  if (seg >= h.total_segments) return;
  const int64_t row = plan[h.off_judge + seg];
  const uint4* hp = reinterpret_cast<const uint4*>(hidden + row * hs);
  const uint4* w0 = reinterpret_cast<const uint4*>(w2);
  const uint4* w1 = reinterpret_cast<const uint4*>(w2 + hs);
  float a0 = 0.0f, a1 = 0.0f;
  for (int c = lane; c < hs / 8; c += 64) {
    const uint4 x = hp[c], u = w0[c], v = w1[c];
    const unsigned xs[4] = {x.x, x.y, x.z, x.w}, us[4] = {u.x, u.y, u.z, u.w}, vs[4] = {v.x, v.y, v.z, v.w};
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      const float xl = __uint_as_float(xs[e] << 16), xh = __uint_as_float(xs[e] & 0xffff0000u);
      a0 = fmaf(xl, __uint_as_float(us[e] << 16), a0);
      a0 = fmaf(xh, __uint_as_float(us[e] & 0xffff0000u), a0);
      a1 = fmaf(xl, __uint_as_float(vs[e] << 16), a1);
      a1 = fmaf(xh, __uint_as_float(vs[e] & 0xffff0000u), a1);
    }
  }
#pragma unroll
  for (int off = 32; off > 0; off >>= 1) { a0 += __shfl_xor(a0, off); a1 += __shfl_xor(a1, off); }
  if (lane == 0) { logits[2 * seg] = a0; logits[2 * seg + 1] = a1; }
}

hipError_t launch_judge_logits(const int32_t* plan_dev, const PlanHeader& h, const void* hidden,
                               const void* w2, int hidden_size, float* logits, hipStream_t s) {
  if (h.total_segments == 0) return hipSuccess;
  dim3 grid;
  if (!grid_1d(((int64_t)h.total_segments + 3) / 4, 256, &grid)) return hipErrorInvalidConfiguration;
  k_judge_logits<<<grid, dim3(256), 0, s>>>(
      plan_dev, h, (const uint16_t*)hidden, (const uint16_t*)w2, hidden_size, logits);
  return hipGetLastError();
}

}  // namespace pv
