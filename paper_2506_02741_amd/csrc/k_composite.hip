// Tile compositing of view-tied Gaussians: forward (RGB, depth, silhouette)
// and its reverse-mode replay.
//
// One workgroup per (view, tile).  Each wave owns a square block of the
// tile (8x8 pixels, or 16x16 for 32-pixel tiles with four pixels per lane).
// The tile's depth-sorted list is walked in batches staged through LDS.
// Which entries reach which pixels is a matrix product (Coverage below): the
// conic's q(x, y) - q_cut is a polynomial in the pixel's tile coordinates,
// six coefficients per entry against six monomials per pixel, and the signs
// of the MFMA's results are every lane's bit mask of the entries that may
// reach its pixel.  The lanes then composite their own entries of a group of
// chunks (up to 512 entries) as one stream each, with the exact test, so a
// wave takes as many steps as its busiest lane has entries in the group.
//
// Forward, per pixel, front to back [splat of Sec. 3.3]:
//   q = d^T Q d with d = pixel - mu; skip q > q_cut
//   alpha = min(alpha_max, o exp(-q/2)); skip alpha < alpha_min
//   stop before T (1 - alpha) < t_min
//   C += c alpha T, D += z alpha T, T *= (1 - alpha)
//   out: C + T bg, D, 1 - T; keep T_final and the list position past the
//   last contributor for the backward.
//
// Backward replays the same list from the last contributor towards the
// front, recovering T_i = T_{i+1} / (1 - alpha_i).  What lies behind
// contributor i, normalised, is B_i = alpha_b x_b + (1 - alpha_b) B_b with
// b the next contributor behind it and x = (c, z, 1), and B = (bg, 0, 0) at
// the back; only g . (x_i - B_i) enters the gradient, carried per pixel by
// the difference recurrence
//   g.(x_i - B_i) = g.(x_i - x_b) + (1 - alpha_b) g.(x_b - B_b)
// (x_b = (bg, 0, 0) and the second term 0 at the back).  Neighbouring
// colours and depths are close, so their differences are exact or nearly,
// and the result keeps its relative accuracy where x_i and B_i agree (a
// surface seen through Gaussians of its own colour), which a running
// g . B subtracted from g . x_i would lose to cancellation.  Per
// contributing pair:
//   dL/dalpha = T [g_C.(c - B_C) + g_D (z - B_D) + g_S (1 - B_S)] = T g.(x - B)
//   dL/dc = alpha T g_C, dL/dz = alpha T g_D,
//   if o G <= alpha_max: dL/do = G dL/dalpha, dL/dq = -o G dL/dalpha / 2
// and q's dependence on the camera-frame centre p and the radius r
// (mu = proj(p), Sigma = r^2 J J^T + s I, w = Sigma^-1 d, t = J^T w):
//   dq/dr = -2 r |t|^2
//   dq/dp = (-2 t0 + k t0 t2, -2 t1 + k t1 t2, -2 t2 + k (t0^2 + t1^2 + 2 t2^2)),
//   k = 2 r^2 / p_z.
// Mode "twist": dL/dp is chained straight to the view's left twist
// (rho += dL/dp, phi += p x dL/dp) in registers, summed per tile.
// Mode "slots": each lane adds its (dL/dc, dL/do, dL/dr) -- and with
// geometry its dL/dp -- for an entry into its wave's own LDS accumulators
// (read and written back by the lane that claims the entry, LDS atomics for
// the lanes that lose, in the wave's program order); after a batch the four
// waves' sums go to the pair's (record, tile) slot, and a gather pass sums a
// record's slots.  Neither mode uses global
// atomics and no two waves share an accumulator, so both are deterministic.
#include <type_traits>

#include "vtgs_internal.h"

namespace vtgs {

namespace {

constexpr float kNegHalfLog2e = -0.72134752044448170368f;  // -log2(e) / 2

// Eq. 1 evaluated inside the tracking backward.
struct TrackArgs {
  float alpha, beta, sil_thr;
};

__device__ __forceinline__ float sgn(float x) { return (float)((x > 0.f) - (x < 0.f)); }

template <int TILE>
struct Shape {
  static constexpr int NT = TILE == 8 ? 64 : 256;
  static constexpr int PPT = TILE * TILE / NT;  // pixels per lane
  static constexpr int WB = TILE == 32 ? 16 : 8;  // side of a wave's block
};

// Pixel k of this lane, relative to the tile origin.
template <int TILE>
__device__ __forceinline__ void lane_pixel(int k, int &x, int &y) {
  const int w = threadIdx.x / kWave, l = threadIdx.x % kWave;
  if (TILE == 8) { x = l % 8; y = l / 8; return; }
  const int qx = (w % 2) * Shape<TILE>::WB, qy = (w / 2) * Shape<TILE>::WB;
  x = qx + l % 8 + 8 * (k % 2);
  y = qy + l / 8 + 8 * (k / 2);
}

// ---------------------------------------------------------------------------
// Coverage: which entries of a chunk reach which pixels of a wave's block
// ---------------------------------------------------------------------------
// With X, Y the pixel's integer offsets from the tile's middle (|X|, |Y| <=
// H = TILE / 2) and m the mean's,
//   q - q_cut = A X^2 + B X Y + C Y^2 + D X + E Y + F,
//   A = qa, B = 2 qb, C = qc, D = -(2 A mx + B my), E = -(B mx + 2 C my),
//   F = A mx^2 + B mx my + C my^2 - q_cut,
// a dot product of 16 bf16 terms: the monomials are exact in bf16 (products
// of integers up to 16 are at most 256), A, B, C enter as two bf16 pieces
// and D, E, F as three, the products are exact and their sum is FP32.  It
// errs by at most
//   |A X^2| .. : 2^-16 H^2 (|A| + |B| + |C|)        (two pieces)
//   the rest, and the FP32 q of the exact test: a few dozen roundings of
//   terms below (|A| + |B| + |C|) (|m| + H)^2 each, taken as 2^-18 of that
// and F is lowered by that much, so the sign is set for every pixel the exact
// test (FP32, q <= q_cut) accepts, and for few others (about one in a wave's
// life): the compositing step repeats the exact test and takes their bits
// back out.  A conic too large for the bound to be finite is tried at
// every pixel.  One v_alignbit per two (entry, 32 pixels) results moves the
// signs into the lanes' masks, so 64 entries against 64 pixels cost 4 MFMAs
// and ~80 VALU instructions; testing q per (entry, pixel) on the VALU took
// 12.75 for each entry whose cull circle met the block, ~380 per chunk.  With
// the compositing step's own instructions cut (48 from ~65) the forward of a
// 640x480 tracking frame went from 62 to 41 us, of 5 views of 8 keyframes from
// 1070 to 758, both still bound by VALU issue.
typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef float f32x16 __attribute__((ext_vector_type(16)));

// One entry's 16 bf16 coefficients, terms 0-7 in lo and 8-15 in hi (the
// halves the lower and upper 32 lanes of an MFMA operand hold).  absent: an
// entry past the list's end, or of an id out of range, reaches no pixel.
template <int TILE>
__device__ __forceinline__ void coverage_row(bool absent, float mx, float my, float A, float B,
                                             float C, float qcut, float cx, float cy, bf16x8 &lo,
                                             bf16x8 &hi) {
  constexpr float H = (float)(TILE / 2);
  mx -= cx;
  my -= cy;
  float D = -fmaf(2.0f * A, mx, B * my), E = -fmaf(2.0f * C, my, B * mx);
  const float S = fabsf(A) + fabsf(B) + fabsf(C);
  const float M = fmaxf(fabsf(mx), fabsf(my)) + H;
  const float slack = fmaf(S, fmaf(M * M, 0x1p-18f, H * H * 0x1p-16f), 1e-5f * qcut);
  float F = fmaf(-0.5f, fmaf(D, mx, E * my), -(qcut + slack));
  const bool bounded = slack < 1e30f;  // (false for NaN)
  const bool flat = absent || !bounded;
  A = flat ? 0.f : A; B = flat ? 0.f : B; C = flat ? 0.f : C;
  D = flat ? 0.f : D; E = flat ? 0.f : E;
  F = absent ? 1.0f : (bounded ? F : -1.0f);
  auto piece = [](float &x) {  // the leading bf16 of x, which keeps the rest
    const __bf16 b = (__bf16)x;
    x -= (float)b;
    return b;
  };
  lo[0] = piece(A); lo[1] = (__bf16)A;
  lo[2] = piece(B); lo[3] = (__bf16)B;
  lo[4] = piece(C); lo[5] = (__bf16)C;
  lo[6] = piece(F); lo[7] = piece(F);
  hi[0] = piece(D); hi[1] = piece(D); hi[2] = (__bf16)D;
  hi[3] = piece(E); hi[4] = piece(E); hi[5] = (__bf16)E;
  hi[6] = (__bf16)F; hi[7] = (__bf16)0.f;
}

// The monomials of pixel (l % 32) + 32 n of a lane's k-th 8x8 sub-block, in
// the order of coverage_row's terms (lanes 0-31 terms 0-7, 32-63 terms 8-15).
template <int TILE>
__device__ __forceinline__ bf16x8 coverage_pixel(int k, int n) {
  const int w = threadIdx.x / kWave, l = lane_id(), p = (l & 31) + 32 * n;
  const int qx = TILE == 8 ? 0 : (w % 2) * Shape<TILE>::WB, qy = TILE == 8 ? 0 : (w / 2) * Shape<TILE>::WB;
  const float X = (float)(qx + p % 8 + 8 * (k % 2) - TILE / 2);
  const float Y = (float)(qy + p / 8 + 8 * (k / 2) - TILE / 2);
  const bool lower = l < 32;
  const float a = lower ? X * X : X, c = lower ? Y * Y : Y, b = lower ? X * Y : X;
  const float d = lower ? X * Y : Y;
  bf16x8 r;
  r[0] = r[1] = (__bf16)a;
  r[2] = (__bf16)b; r[3] = (__bf16)d;
  r[4] = r[5] = (__bf16)c;
  r[6] = (__bf16)1.0f; r[7] = (__bf16)(lower ? 1.0f : 0.f);
  return r;
}

// Lane masks of 32 staged entries whose rows are `a` (coverage_entry gives
// the entry a lane loads): bit e is set where entry e may reach the lane's
// pixel of the sub-block with monomials pix.
__device__ __forceinline__ uint32_t coverage32(const bf16x8 &a, const bf16x8 (&pix)[2]) {
  const f32x16 zero = {};
  const f32x16 c0 = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a, pix[0], zero, 0, 0, 0);
  const f32x16 c1 = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a, pix[1], zero, 0, 0, 0);
  // result i of a lane is row 8 (i / 4) + 4 (l / 32) + i % 4, column l % 32:
  // the upper lanes hold the other rows of the same 32 pixels
  uint32_t b0 = 0u, b1 = 0u;
#pragma unroll
  for (int i = 15; i >= 0; i--) {
    b0 = __builtin_amdgcn_alignbit(b0, __float_as_uint(c0[i]), 31);
    b1 = __builtin_amdgcn_alignbit(b1, __float_as_uint(c1[i]), 31);
  }
  // b0's upper half (pixels 0-31) changes places with b1's lower half
  // (pixels 32-63): every lane then holds both masks of its own pixel
  const auto r = __builtin_amdgcn_permlane32_swap(b0, b1, false, false);
  return r[0] | (r[1] << 16);
}

// Entry of 32 whose row lane l loads: the rows a lane's results come from
// (above) are entries 0-15 in order for the lower lanes, 16-31 for the upper.
__device__ __forceinline__ int coverage_entry() {
  const int r = lane_id() & 31;
  return 16 * ((r >> 2) & 1) + 4 * (r >> 3) + (r & 3);
}

// Lanes as a scalar mask, and back.
__device__ __forceinline__ unsigned long long lanes(bool p) { return __builtin_amdgcn_ballot_w64(p); }
__device__ __forceinline__ bool in_lanes(unsigned long long m) {
  return __builtin_amdgcn_inverse_ballot_w64(m);
}

// First u64 of the lane bits of chunk c of the batch at list offset `boff`
// (a multiple of 64) of tile t, wave w of nw, ppt pixels per lane.  Chunks
// of consecutive tiles never share an index (the tile number is added to
// the list position / 64), and the index stays below cap / 64 + n_tiles + 1.
__device__ __forceinline__ int64_t chunk_word(int start, int boff, int c, int t, int w, int nw,
                                              int ppt) {
  const int64_t cid = (int64_t)(start >> 6) + (boff >> 6) + c + t;
  return ((cid * nw + w) * ppt) * kWave;
}

// q = d^T Q d (d = pixel - mu) in a fixed order, from a staged entry whose
// off-diagonal term is already doubled (e0.w = 2 qb, exact in FP32).
__device__ __forceinline__ float quad2(const float4 &e0, float qc, float px, float py) {
  const float dx = px - e0.x, dy = py - e0.y;
  float q = (e0.z * dx) * dx;
  q = fmaf(e0.w * dx, dy, q);
  q = fmaf(qc * dy, dy, q);
  return q;
}

// Chunks of 64 entries whose lane bits one phase-2 pass walks as a single
// stream per lane (a lane then steps once per entry that reaches its pixel,
// not once per entry of the busiest lane of every chunk).  Four pixels per
// lane keep one chunk per pass to bound the LDS words.
template <int TILE, int BATCH>
struct Group {
  static constexpr int NCB = BATCH / kWave;  // chunks of a full batch
  static constexpr int G = Shape<TILE>::PPT > 1 ? 1 : (NCB < 4 ? NCB : 4);
  // the forward's passes may be longer: it keeps no per-entry state
  static constexpr int GF = Shape<TILE>::PPT > 1 ? 1 : (NCB < 8 ? NCB : 8);
  static constexpr int NH = 2 * GF;          // 32-entry words of a forward pass
};

// Lowest set bit of a word, 31 for a zero word (an index that stays inside
// the group, read and then ignored).
__device__ __forceinline__ int low_bit(uint32_t v) { return __builtin_ctz(v | 0x80000000u); }

// Gather the record of entry `id` of the view.  No branch around the loads
// (so that nothing waits for them before their use): an id out of range,
// which a consistent list never holds, reads record 0 and clears `ok`, and
// the staging then leaves the entry out of every wave's mask.
__device__ __forceinline__ void fetch_record(const Ws &ws, int n_rec, int rec_base, uint32_t id,
                                             float4 &e0, float4 &e1, float4 &e2, bool &ok) {
  ok = id < (uint32_t)n_rec;
  const float4 *A = ws.recA + 3 * ((int64_t)rec_base + (ok ? id : 0u));
  e0 = A[0]; e1 = A[1]; e2 = A[2];
}

// Waves per SIMD the register budget leaves room for (tile 16: the blocks per
// CU its LDS allows); two or more also keep the MFMA results in VGPRs, which
// the sign extraction reads directly.
template <int TILE, int BATCH>
__global__ __attribute__((amdgpu_waves_per_eu(TILE == 16 ? 4 : 2))) __launch_bounds__(
    Shape<TILE>::NT) void k_fwd(Ws ws, float *out_rgb, float *out_depth, float *out_sil) {
  constexpr int NT = Shape<TILE>::NT, PPT = Shape<TILE>::PPT;
  constexpr int NW = NT / kWave;
  constexpr int PER = (BATCH + NT - 1) / NT;  // list entries each thread stages per batch
  constexpr int G = Group<TILE, BATCH>::GF, NH = Group<TILE, BATCH>::NH, NR = NW * PPT;
  // A batch that is one pass stages its coverage rows first and, once every
  // wave has its bits, the entries themselves in the same LDS (a barrier
  // more, but 512 entries fit four blocks per CU).
  constexpr bool kShare = BATCH / kWave == G;
  // staged entry: e0 (mx, my, qa, 2 qb), e2 (c, z), e1 (qc, o); 32 entries
  // more, never written, that a finished lane's last reads fall into
  constexpr int SE = BATCH + 32, kCov = kShare ? 0 : SE * 40;
  __shared__ __attribute__((aligned(16))) char lds[kShare ? SE * 40 : SE * 40 + BATCH * 32];
  float4 *e0s = (float4 *)lds, *e2s = e0s + SE;
  float2 *e1s = (float2 *)(e2s + SE);
  // coverage rows, terms 0-7, then terms 8-15
  bf16x8 *cov = (bf16x8 *)(lds + kCov);
  __shared__ uint32_t words[NH + 1][NR][kWave];  // the lanes' bits of a pass; the last row zero
  const int t = tile_of_block(ws);
  const DevView &vw = ws.views[find_view_by_tile(ws, t)];
  const int lt = t - vw.tile_base;
  const int ox = (lt % vw.tiles_x) * TILE, oy = (lt / vw.tiles_x) * TILE;
  const uint2 rg = ws.ranges[t];
  const int start = (int)rg.x, end = (int)rg.y;
  const int w = threadIdx.x / kWave;

  float px[PPT], py[PPT], T[PPT], C0[PPT], C1[PPT], C2[PPT], D[PPT];
  uint32_t last[PPT];
  bool valid[PPT];
  unsigned long long done[PPT];  // lanes whose pixel takes no more entries
#pragma unroll
  for (int k = 0; k < PPT; k++) {
    int x, y;
    lane_pixel<TILE>(k, x, y);
    px[k] = (float)(ox + x);
    py[k] = (float)(oy + y);
    valid[k] = (ox + x) < vw.width && (oy + y) < vw.height;
    done[k] = lanes(!valid[k]);
    T[k] = 1.f; C0[k] = C1[k] = C2[k] = D[k] = 0.f; last[k] = 0;
  }
  const float amin = ws.amin, amax = ws.amax, tmin = ws.tmin, qcut = ws.qcut;
  const float cx = (float)(ox + TILE / 2), cy = (float)(oy + TILE / 2);
  bf16x8 pix[PPT][2];
#pragma unroll
  for (int k = 0; k < PPT; k++) {
    pix[k][0] = coverage_pixel<TILE>(k, 0);
    pix[k][1] = coverage_pixel<TILE>(k, 1);
    words[NH][w * PPT + k][lane_id()] = 0u;
  }
  const bf16x8 *cov_row = cov + (lane_id() >> 5) * BATCH + coverage_entry();

  auto wave_done = [&]() {
    unsigned long long all = ~0ull;
#pragma unroll
    for (int k = 0; k < PPT; k++) all &= done[k];
    return all == ~0ull;
  };

  // the next batch's records are gathered into registers while the current
  // batch is composited, and the ids of the batch after it one batch ahead
  // (list positions are clamped to the list; the extra loads go unused)
  float4 p0[PER], p1[PER], p2[PER];
  bool pok[PER];
  uint32_t pid[PER];
  const int n_rec = vw.n_rec, rec_base = vw.rec_base;
  if (end > start) {
#pragma unroll
    for (int k = 0; k < PER; k++) pid[k] = ws.ids[min(start + (int)threadIdx.x + k * NT, end - 1)];
#pragma unroll
    for (int k = 0; k < PER; k++) fetch_record(ws, n_rec, rec_base, pid[k], p0[k], p1[k], p2[k], pok[k]);
#pragma unroll
    for (int k = 0; k < PER; k++)
      pid[k] = ws.ids[min(start + BATCH + (int)threadIdx.x + k * NT, end - 1)];
  }

  for (int b = start; b < end; b += BATCH) {
    if (__syncthreads_and(wave_done())) break;
    const int nb = min(BATCH, end - b);
    auto stage_entries = [&]() {
#pragma unroll
      for (int k = 0; k < PER; k++) {
        const int i = threadIdx.x + k * NT;
        if (i >= nb) continue;
        // the off-diagonal conic term is staged doubled (exact in FP32)
        e0s[i] = make_float4(p0[k].x, p0[k].y, p0[k].z, 2.0f * p0[k].w);
        e1s[i] = make_float2(p1[k].x, p1[k].y);
        e2s[i] = make_float4(p2[k].x, p2[k].y, p2[k].z, p1[k].z);
      }
    };
    // (past the last batch the clamped loads repeat the list's last entry)
    auto prefetch = [&]() {
#pragma unroll
      for (int k = 0; k < PER; k++) fetch_record(ws, n_rec, rec_base, pid[k], p0[k], p1[k], p2[k], pok[k]);
#pragma unroll
      for (int k = 0; k < PER; k++)
        pid[k] = ws.ids[min(b + 2 * BATCH + (int)threadIdx.x + k * NT, end - 1)];
    };
#pragma unroll
    for (int k = 0; k < PER; k++) {
      const int i = threadIdx.x + k * NT;
      if (BATCH % NT != 0 && i >= BATCH) continue;
      coverage_row<TILE>(i >= nb || !pok[k], p0[k].x, p0[k].y, p0[k].z, 2.0f * p0[k].w, p1[k].x,
                         qcut, cx, cy, cov[i], cov[BATCH + i]);
    }
    if (!kShare) stage_entries();
    __syncthreads();
    if (!kShare) prefetch();
    const uint32_t base = (uint32_t)(b - start + 1);
    const int nch = (nb + kWave - 1) / kWave;
    for (int g0 = 0; g0 < nch; g0 += G) {
      if (!kShare && wave_done()) break;
      // 1. which of the pass's entries may reach each of this lane's pixels:
      // a word per 32 entries, kept in LDS for the pass and in memory for the
      // backward, which replays the same chunks
      uint32_t nz[PPT];  // bit h: word h is not zero
#pragma unroll
      for (int k = 0; k < PPT; k++) nz[k] = 0u;
      const int cend = min(g0 + G, nch);
      for (int c = wave_done() ? cend : g0; c < cend; c++) {
        const bf16x8 r0 = cov_row[c * kWave], r1 = cov_row[c * kWave + 32];
        unsigned long long *dst = ws.lane_bits + chunk_word(start, b - start, c, t, w, NW, PPT);
        const int h = 2 * (c - g0);
#pragma unroll
        for (int k = 0; k < PPT; k++) {
          uint32_t lo = coverage32(r0, pix[k]), hi = coverage32(r1, pix[k]);
          lo = in_lanes(done[k]) ? 0u : lo;
          hi = in_lanes(done[k]) ? 0u : hi;
          words[h][w * PPT + k][lane_id()] = lo;
          words[h + 1][w * PPT + k][lane_id()] = hi;
          nz[k] |= (lo ? 1u << h : 0u) | (hi ? 2u << h : 0u);
          dst[k * kWave + lane_id()] = ((unsigned long long)hi << 32) | lo;
        }
      }
      if (odd_records(ws)[1] && !wave_done()) {
        // Plans with colours or depths that are not finite: a step that the
        // exact test refuses weighs 0, which would still put such a value into
        // the pixel's sums, so these entries take the exact test here.
        for (int c = g0; c < cend; c++) {
          const int n = min(nb - c * kWave, kWave);
          const uint32_t id = ws.ids[b + c * kWave + min(lane_id(), n - 1)];
          const float4 *A = ws.recA + 3 * ((int64_t)rec_base + (id < (uint32_t)n_rec ? id : 0u));
          const bool finite = all_finite(A[2].x, A[2].y, A[2].z, A[1].z);
          for (unsigned long long m = lanes(!finite && lane_id() < n); m; m &= m - 1ull) {
            const int e = __builtin_ctzll(m);
            const uint32_t i = (uint32_t)__builtin_amdgcn_readlane((int)id, e);
            const float4 *E = ws.recA + 3 * ((int64_t)rec_base + (i < (uint32_t)n_rec ? i : 0u));
            const float4 e0 = make_float4(E[0].x, E[0].y, E[0].z, 2.0f * E[0].w);
            const int h = 2 * (c - g0) + (e >> 5);
#pragma unroll
            for (int k = 0; k < PPT; k++) {
              uint32_t &word = words[h][w * PPT + k][lane_id()];
              if (!(quad2(e0, E[1].x, px[k], py[k]) <= qcut)) word &= ~(1u << (e & 31));
              if (word == 0u) nz[k] &= ~(1u << h);
              uint32_t *dst = (uint32_t *)(ws.lane_bits + chunk_word(start, b - start, c, t, w, NW, PPT));
              dst[2 * (k * kWave + lane_id()) + (e >> 5)] = word;
            }
          }
        }
      }
      if (kShare) {
        __syncthreads();
        stage_entries();
        __syncthreads();
        prefetch();
      }
      // 2. each lane composites its own entries of the pass in list order,
      // one step per entry; the wave runs until its last lane is through
#pragma unroll
      for (int k = 0; k < PPT; k++) {
        const int row = w * PPT + k;
        const int gb = g0 * kWave;
        // the lane's current word (index h) and next one (index hn, the zero
        // row after its last)
        auto first = [](uint32_t v) { return __builtin_ctz(v | (1u << NH)); };
        uint32_t left = nz[k];
        int h = first(left);
        left &= left - 1u;
        int hn = first(left);
        uint32_t cur = words[h][row][lane_id()], nxt = words[hn][row][lane_id()];
        int li = -1;  // the pass's last contributor
        struct Entry {
          float4 e0, e2;
          float2 e1;
          int i;
        };
        // the LDS reads of the lane's entry at the front of `cur`
        auto fetch = [&](Entry &E) {
          E.i = gb + (h << 5) + low_bit(cur);
          E.e0 = e0s[E.i];
          E.e1 = e1s[E.i];
          E.e2 = e2s[E.i];
        };
        // one step of the lanes that have an entry: issue the next entry's
        // reads into N, composite E; true where the pixel stops
        auto step = [&](const Entry &E, Entry &N) {
          cur &= cur - 1u;
          const bool z = cur == 0u;
          cur = z ? nxt : cur;
          h = z ? hn : h;
          left = z ? left & (left - 1u) : left;
          hn = first(left);
          nxt = words[hn][row][lane_id()];
          fetch(N);
          const float q = quad2(E.e0, E.e1.x, px[k], py[k]);
          const float gau = __builtin_amdgcn_exp2f(q * kNegHalfLog2e);
          const float a = fminf(amax, E.e1.y * gau);
          const bool ok = q <= qcut && a >= amin;
          const float Tn = T[k] * (1.0f - a);
          const bool stop = ok && Tn < tmin;
          const bool take = ok && !stop;
          const float wgt = take ? a * T[k] : 0.f;
          C0[k] = fmaf(E.e2.x, wgt, C0[k]);
          C1[k] = fmaf(E.e2.y, wgt, C1[k]);
          C2[k] = fmaf(E.e2.z, wgt, C2[k]);
          D[k] = fmaf(E.e2.w, wgt, D[k]);
          T[k] = take ? Tn : T[k];
          li = take ? E.i : li;
          const bool extra = !(q <= qcut);
          if (__builtin_expect(lanes(extra) != 0ull, 0)) {
            // (rare) the bit the backward reads goes: its streams hold the
            // entries of the exact test only.  The lane's own store of the
            // word is complete before its atomic.
            asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
            if (extra) {
              uint32_t *wd = (uint32_t *)(ws.lane_bits + chunk_word(start, b - start, E.i >> 6, t, w, NW, PPT) +
                                          k * kWave + lane_id()) + ((E.i >> 5) & 1);
              atomicAnd(wd, ~(1u << (E.i & 31)));
            }
          }
          return stop;
        };
        Entry A, B;
        fetch(A);
        // the lanes with an entry left (a scalar mask: the loop itself is
        // uniform, and the steps alternate between two register sets, so
        // that no entry is moved from one to the other)
        auto more = [&]() { return lanes(cur != 0u) & ~done[k]; };
        while (true) {
          unsigned long long live = more();
          if (live == 0ull) break;
          bool stop = false;
          if (in_lanes(live)) stop = step(A, B);
          done[k] |= lanes(stop);
          live = more();
          if (live == 0ull) break;
          stop = false;
          if (in_lanes(live)) stop = step(B, A);
          done[k] |= lanes(stop);
        }
        last[k] = li >= 0 ? base + (uint32_t)li : last[k];
      }
    }
  }
  const int64_t P = ws.P;
#pragma unroll
  for (int k = 0; k < PPT; k++) {
    if (!valid[k]) continue;
    const int64_t p = vw.pix_off + (int64_t)((int)py[k]) * vw.width + (int)px[k];
    if (out_rgb) {
      out_rgb[p] = fmaf(T[k], ws.bg[0], C0[k]);
      out_rgb[P + p] = fmaf(T[k], ws.bg[1], C1[k]);
      out_rgb[2 * P + p] = fmaf(T[k], ws.bg[2], C2[k]);
    }
    if (out_depth) out_depth[p] = D[k];
    if (out_sil) out_sil[p] = 1.0f - T[k];
    ws.t_final[p] = T[k];
    ws.last[p] = last[k];
  }
}

// Staging of one list entry for the backward to slots: the forward record,
// the camera-frame centre and learnable flag, the record's tile rectangle and
// first slot.  Gathered without branches, as in the forward.
struct BwdEntry {
  float4 e0, e1, e2;
  float2 eb;
  uint2 rc;
  uint32_t off;
  bool ok;
};

__device__ __forceinline__ void fetch_bwd_entry(const Ws &ws, int n_rec, int rec_base, uint32_t id,
                                                BwdEntry &E) {
  E.ok = id < (uint32_t)n_rec;
  const int64_t rec = (int64_t)rec_base + (E.ok ? id : 0u);
  const float4 *A = ws.recA + 3 * rec;
  E.e0 = A[0]; E.e1 = A[1]; E.e2 = A[2];
  E.eb = ws.recB[rec];
  E.rc = ws.rect[rec];
  E.off = ws.rec_off[rec];
}

// The (record, tile) slot of a staged entry of tile (tx, ty), or ~0u when
// it has none (an id out of range, or past the capacity after an overflow).
__device__ __forceinline__ uint32_t entry_slot(const Ws &ws, const BwdEntry &E, int tx, int ty) {
  const int x0 = E.rc.x & 0xffff, y0 = E.rc.x >> 16, x1 = E.rc.y & 0xffff;
  const uint32_t sl = E.off + (uint32_t)((ty - y0) * (x1 - x0 + 1) + (tx - x0));
  return E.ok && sl < (uint64_t)ws.cap ? sl : 0xffffffffu;
}

typedef float f32x4 __attribute__((ext_vector_type(4)));
// LDS pointers
#define LDS_AS __attribute__((address_space(3)))
// An empty statement that the compiler must take as reading and writing all
// memory: LDS accesses keep their program order across it (and the LDS
// keeps a wave's order).
__device__ __forceinline__ void kLdsOrder() { asm volatile("" ::: "memory"); }
// The accumulator floats past the first four: one (dL/dr) or, with
// geometry, four (dL/dr, dL/dp).
template <bool kGeo>
using AccB = typename std::conditional<kGeo, f32x4, float>::type;

// The per-pixel state of a backward: the forward's transmittance and last
// contributor, the upstream gradient (Eq. 1's where kTrack, alpha W |V - V'| +
// beta W |D - D'| with W = vis & (D > 0) & (S' > thr), and this lane's share
// of the tile's loss, else the caller's arrays) and the difference recurrence
// at the back: E = (1 - alpha_b) g.(x_b - B_b) of the contributor b behind (0),
// its colour and depth XP (the background and 0), and GS1 = g_S (1 - its
// coverage).
template <int PPT>
struct BwdPixels {
  float px[PPT], py[PPT], T[PPT], gC0[PPT], gC1[PPT], gC2[PPT], gD[PPT];
  float E[PPT], XP0[PPT], XP1[PPT], XP2[PPT], XPZ[PPT], GS1[PPT];
  uint32_t last[PPT];
  uint32_t mylast;
  float lsum;
};

template <int TILE, bool kTrack>
__device__ __forceinline__ void load_pixels(const Ws &ws, const DevView &vw, int ox, int oy,
                                            const float *g_rgb, const float *g_depth,
                                            const float *g_sil, const TrackArgs &tr,
                                            BwdPixels<Shape<TILE>::PPT> &S) {
  const int64_t P = ws.P;
  S.mylast = 0u;
  S.lsum = 0.f;
#pragma unroll
  for (int k = 0; k < Shape<TILE>::PPT; k++) {
    int x, y;
    lane_pixel<TILE>(k, x, y);
    S.px[k] = (float)(ox + x);
    S.py[k] = (float)(oy + y);
    const bool valid = (ox + x) < vw.width && (oy + y) < vw.height;
    const int64_t p = vw.pix_off + (int64_t)(oy + y) * vw.width + (ox + x);
    S.T[k] = valid ? ws.t_final[p] : 1.f;
    S.last[k] = valid ? ws.last[p] : 0u;
    float gS = 0.f;
    if constexpr (kTrack) {
      const int64_t lp = p - vw.pix_off;
      const int64_t Pv = (int64_t)vw.width * vw.height;
      float od = 0.f;
      bool W = false;
      if (valid) {
        od = vw.obs_depth[lp];
        W = (!vw.vis || vw.vis[lp] != 0) && od > 0.f && ws.img[4 * P + p] > tr.sil_thr;
      }
      const float r0 = valid ? vw.obs_rgb[lp] - ws.img[p] : 0.f;
      const float r1 = valid ? vw.obs_rgb[Pv + lp] - ws.img[P + p] : 0.f;
      const float r2 = valid ? vw.obs_rgb[2 * Pv + lp] - ws.img[2 * P + p] : 0.f;
      const float rd = valid ? od - ws.img[3 * P + p] : 0.f;
      S.gC0[k] = W ? -tr.alpha * sgn(r0) : 0.f;
      S.gC1[k] = W ? -tr.alpha * sgn(r1) : 0.f;
      S.gC2[k] = W ? -tr.alpha * sgn(r2) : 0.f;
      S.gD[k] = W ? -tr.beta * sgn(rd) : 0.f;
      S.lsum += W ? tr.alpha * ((fabsf(r0) + fabsf(r1)) + fabsf(r2)) + tr.beta * fabsf(rd) : 0.f;
    } else {
      S.gC0[k] = (valid && g_rgb) ? g_rgb[p] : 0.f;
      S.gC1[k] = (valid && g_rgb) ? g_rgb[P + p] : 0.f;
      S.gC2[k] = (valid && g_rgb) ? g_rgb[2 * P + p] : 0.f;
      S.gD[k] = (valid && g_depth) ? g_depth[p] : 0.f;
      gS = (valid && g_sil) ? g_sil[p] : 0.f;
    }
    S.E[k] = 0.f;
    S.XP0[k] = ws.bg[0]; S.XP1[k] = ws.bg[1]; S.XP2[k] = ws.bg[2]; S.XPZ[k] = 0.f;
    S.GS1[k] = gS;
    S.mylast = max(S.mylast, S.last[k]);
  }
}

// Per tile: the lanes' six twist sums and the Eq. 1 loss, wave by wave.
template <int NW>
__device__ __forceinline__ void store_twist(const Ws &ws, int t, const float (&tw)[6], float lsum,
                                            float (*red)[7]) {
  const int w = threadIdx.x / kWave;
#pragma unroll
  for (int c = 0; c < 6; c++) {
    const float s = wave_sum(tw[c]);
    if (lane_id() == 0) red[w][c] = s;
  }
  const float ls = wave_sum(lsum);
  if (lane_id() == 0) red[w][6] = ls;
  __syncthreads();
  if (threadIdx.x < 7) {
    float s = 0.f;
#pragma unroll
    for (int ww = 0; ww < NW; ww++) s += red[ww][threadIdx.x];
    ws.twist_part[8 * (int64_t)t + threadIdx.x] = s;
  }
}

// Backward to the twist alone (tracking): like the forward, a pass is a long
// stretch of the list (no per-entry state is kept: the twist is summed in
// registers) and its steps alternate between two register sets.  Staged
// entries hold the step's operands only, the list's last entry first:
//   e0 (mx, my, qa, 2 qb), e1 (qc, o, z, 2 r^2 / z), e2 (c, px),
//   e3 (py, 1/z, -fx px/z^2, -fy py/z^2).
// The operations and their order are the slots kernel's: a trajectory of L1
// steps amplifies any other rounding of the twist.  Against that kernel's form
// without slots, in 256-entry batches with five 16-byte reads a step: 640x480
// tracking frame 55 -> 49 us, 160x120 42 -> 31, a batch of served tracks 1166
// -> 1026; bound by VALU issue (72 %) and the waits of four waves per SIMD.
template <int TILE, int BATCH, bool kTrack>
__global__ __attribute__((amdgpu_waves_per_eu(TILE == 16 ? 4 : 2))) __launch_bounds__(
    Shape<TILE>::NT) void k_bwd_twist(Ws ws, const float *g_rgb, const float *g_depth,
                                      const float *g_sil, TrackArgs tr) {
  constexpr int NT = Shape<TILE>::NT, PPT = Shape<TILE>::PPT;
  constexpr int NW = NT / kWave;
  constexpr int PER = (BATCH + NT - 1) / NT;
  constexpr int NCB = BATCH / kWave, G = PPT > 1 ? 1 : NCB;  // chunks of a pass's stream
  constexpr int NH = 2 * G, NR = NW * PPT, SE = BATCH + 32;
  __shared__ float4 e0s[SE], e1s[SE], e2s[SE], e3s[SE];
  __shared__ uint32_t words[NH + 1][NR][kWave];  // the last row zero
  __shared__ int maxlast_s;
  __shared__ float red_s[NW][7];

  const int t = tile_of_block(ws);
  const DevView &vw = ws.views[find_view_by_tile(ws, t)];
  const int lt = t - vw.tile_base;
  const int ox = (lt % vw.tiles_x) * TILE, oy = (lt / vw.tiles_x) * TILE;
  const uint2 rg = ws.ranges[t];
  const int start = (int)rg.x;
  const int w = threadIdx.x / kWave;
  BwdPixels<PPT> S;
  if (threadIdx.x == 0) maxlast_s = 0;
  load_pixels<TILE, kTrack>(ws, vw, ox, oy, g_rgb, g_depth, g_sil, tr, S);
#pragma unroll
  for (int k = 0; k < PPT; k++) words[NH][w * PPT + k][lane_id()] = 0u;
  const int wlast = __builtin_amdgcn_readfirstlane(wave_max_i((int)S.mylast));
  __syncthreads();
  if (lane_id() == 0) atomicMax(&maxlast_s, wlast);
  __syncthreads();
  const int len = maxlast_s;

  float tw[6] = {0.f, 0.f, 0.f, 0.f, 0.f, 0.f};
  const float amin = ws.amin, amax = ws.amax;
  const float vfx = vw.fx, vfy = vw.fy;

  // the pass below is gathered while the current one is replayed, its ids one
  // pass ahead (positions clamped to the list, extra loads unused)
  float4 r0[PER], r1[PER], r2[PER];
  float2 rb[PER];
  uint32_t pid[PER];
  const int n_rec = vw.n_rec, rec_base = vw.rec_base;
  auto fetch_ids = [&](int top) {
#pragma unroll
    for (int k = 0; k < PER; k++)
      pid[k] = ws.ids[start + min(max(kWave * top - 1 - (int)threadIdx.x - k * NT, 0), len - 1)];
  };
  auto fetch_records = [&]() {
#pragma unroll
    for (int k = 0; k < PER; k++) {
      const int64_t rec = (int64_t)rec_base + (pid[k] < (uint32_t)n_rec ? pid[k] : 0u);
      const float4 *A = ws.recA + 3 * rec;
      r0[k] = A[0]; r1[k] = A[1]; r2[k] = A[2];
      rb[k] = ws.recB[rec];
    }
  };
  const int nchunk = (len + kWave - 1) / kWave;
  if (len > 0) {
    fetch_ids(nchunk);
    fetch_records();
    fetch_ids(nchunk - NCB);
  }
  for (int top = nchunk; top > 0; top -= NCB) {
    // the pass's lane bits, all loads issued at once (a chunk past the wave's
    // last contributor may hold anything: nothing below cuts it away)
    unsigned long long lb[G][PPT];
    auto fetch_bits = [&](int g0) {
#pragma unroll
      for (int j = 0; j < G; j++) {
        const unsigned long long *src =
            ws.lane_bits + chunk_word(start, 0, max(top - 1 - g0 - j, 0), t, w, NW, PPT);
#pragma unroll
        for (int k = 0; k < PPT; k++) lb[j][k] = src[k * kWave + lane_id()];
      }
    };
    fetch_bits(0);
    __syncthreads();
#pragma unroll
    for (int k = 0; k < PER; k++) {
      const int i = threadIdx.x + k * NT;
      if (BATCH % NT != 0 && i >= BATCH) continue;
      const float iz = 1.0f / r1[k].z;
      e0s[i] = make_float4(r0[k].x, r0[k].y, r0[k].z, 2.0f * r0[k].w);
      e1s[i] = make_float4(r1[k].x, r1[k].y, r1[k].z, 2.0f * r2[k].w * r2[k].w * iz);
      e2s[i] = make_float4(r2[k].x, r2[k].y, r2[k].z, rb[k].x);
      e3s[i] = make_float4(rb[k].y, iz, -vfx * rb[k].x * iz * iz, -vfy * rb[k].y * iz * iz);
    }
    __syncthreads();
    fetch_records();
    fetch_ids(top - 2 * NCB);
    for (int g0 = 0; g0 < min(top, NCB); g0 += G) {
      if (g0 > 0) fetch_bits(g0);
      // 1. the entries that reached each of this lane's pixels in the forward,
      // cut at the pixel's last contributor; the words go in bit-reversed,
      // top half first, so the lowest set bit is the next entry to the front
      uint32_t nz[PPT];
#pragma unroll
      for (int k = 0; k < PPT; k++) nz[k] = 0u;
#pragma unroll
      for (int j = 0; j < G; j++) {
        const int c = top - 1 - g0 - j;
#pragma unroll
        for (int k = 0; k < PPT; k++) {
          const int lim = c < 0 ? 0 : (int)S.last[k] - c * kWave;
          const unsigned long long below =
              lim >= kWave ? ~0ull : (lim <= 0 ? 0ull : (1ull << lim) - 1ull);
          const unsigned long long own = lb[j][k] & below;
          const uint32_t hi = __builtin_bitreverse32((uint32_t)(own >> 32));
          const uint32_t lo = __builtin_bitreverse32((uint32_t)own);
          words[2 * j][w * PPT + k][lane_id()] = hi;
          words[2 * j + 1][w * PPT + k][lane_id()] = lo;
          nz[k] |= (hi ? 1u << (2 * j) : 0u) | (lo ? 2u << (2 * j) : 0u);
        }
      }
      // 2. each lane replays its own entries of the pass, last to first, one
      // step per entry; the wave runs until its last lane is through
#pragma unroll
      for (int k = 0; k < PPT; k++) {
        const int row = w * PPT + k;
        auto first = [](uint32_t v) { return __builtin_ctz(v | (1u << NH)); };
        uint32_t left = nz[k];
        int h = first(left);
        left &= left - 1u;
        int hn = first(left);
        uint32_t cur = words[h][row][lane_id()], nxt = words[hn][row][lane_id()];
        struct Entry {
          float4 e0, e1, e2, e3;
        };
        auto fetch = [&](Entry &N) {
          const int i = g0 * kWave + (h << 5) + low_bit(cur);
          N.e0 = e0s[i]; N.e1 = e1s[i]; N.e2 = e2s[i]; N.e3 = e3s[i];
        };
        auto step = [&](const Entry &A, Entry &N) {
          cur &= cur - 1u;
          const bool z = cur == 0u;
          cur = z ? nxt : cur;
          h = z ? hn : h;
          left = z ? left & (left - 1u) : left;
          hn = first(left);
          nxt = words[hn][row][lane_id()];
          fetch(N);
          const float dx = S.px[k] - A.e0.x, dy = S.py[k] - A.e0.y;
          // q in the forward's order of operations
          const float ax = A.e0.z * dx, bx = A.e0.w * dx, cy = A.e1.x * dy;
          const float q = fmaf(cy, dy, fmaf(bx, dy, ax * dx));
          const float gau = __builtin_amdgcn_exp2f(q * kNegHalfLog2e);
          const float oG = A.e1.y * gau;
          const float a = fminf(amax, oG);
          const bool ok = a >= amin;
          const float om = 1.0f - a;
          const float Tk = ok ? S.T[k] * __builtin_amdgcn_rcpf(om) : S.T[k];
          S.T[k] = Tk;
          const float wgt = ok ? a * Tk : 0.f;
          // g . (x - B) for this Gaussian, x = (colour, depth, 1)
          const float back = kTrack ? S.E[k] : S.GS1[k] + S.E[k];
          const float gdi =
              fmaf(S.gC0[k], A.e2.x - S.XP0[k],
                   fmaf(S.gC1[k], A.e2.y - S.XP1[k],
                        fmaf(S.gC2[k], A.e2.z - S.XP2[k], fmaf(S.gD[k], A.e1.z - S.XPZ[k], back))));
          const float dLda = ok ? gdi * Tk : 0.f;
          S.E[k] = ok ? om * gdi : S.E[k];
          S.XP0[k] = ok ? A.e2.x : S.XP0[k];
          S.XP1[k] = ok ? A.e2.y : S.XP1[k];
          S.XP2[k] = ok ? A.e2.z : S.XP2[k];
          S.XPZ[k] = ok ? A.e1.z : S.XPZ[k];
          if (!kTrack) S.GS1[k] = ok ? 0.f : S.GS1[k];
          const float dLdq = oG <= amax ? -0.5f * oG * dLda : 0.f;
          // w = Q d (halving 2 qb is exact, also inside a product)
          const float w0 = fmaf(A.e0.z, dx, 0.5f * (A.e0.w * dy));
          const float w1 = fmaf(A.e0.w, 0.5f * dx, cy);
          const float t0 = (vfx * A.e3.y) * w0, t1 = (vfy * A.e3.y) * w1;
          const float t2 = fmaf(A.e3.z, w0, A.e3.w * w1);
          // dL/dp of this pair (camera-frame centre)
          const float kk = A.e1.w;
          const float g0v = dLdq * fmaf(kk * t0, t2, -2.0f * t0);
          const float g1v = dLdq * fmaf(kk * t1, t2, -2.0f * t1);
          const float s2 = fmaf(t0, t0, fmaf(t1, t1, 2.0f * t2 * t2));
          const float g2v = fmaf(dLdq, fmaf(kk, s2, -2.0f * t2), wgt * S.gD[k]);
          const float px = A.e2.w, py = A.e3.x, pz = A.e1.z;
          tw[0] += g0v; tw[1] += g1v; tw[2] += g2v;
          tw[3] += py * g2v - pz * g1v;
          tw[4] += pz * g0v - px * g2v;
          tw[5] += px * g1v - py * g0v;
        };
        Entry A, B;
        fetch(A);
        while (true) {  // (uniform; the lanes with an entry left step)
          unsigned long long live = lanes(cur != 0u);
          if (live == 0ull) break;
          if (in_lanes(live)) step(A, B);
          live = lanes(cur != 0u);
          if (live == 0ull) break;
          if (in_lanes(live)) step(B, A);
        }
      }
    }
  }
  store_twist<NW>(ws, t, tw, S.lsum, red_s);
}

// Backward to the slots (MODE bit 1), with the twist (bit 0) and geometry
// (bit 2) where asked.  Three waves per SIMD (the LDS allows three blocks per
// CU), two with geometry.  A step takes ~85 VALU instructions (115 before its
// register sets alternated) and 11 LDS ones; the LDS and the waits of three
// waves per SIMD bound it: 5 views over 8 keyframes 2629 -> 2496 us (with the
// twist 2895 -> 2721), 2 views over 3 with geometry 839 -> 810.
template <int TILE, int BATCH, int MODE>
__global__ __launch_bounds__(Shape<TILE>::NT, (MODE & 4) ? 2 : 3) void k_bwd(Ws ws, const float *g_rgb,
                                                         const float *g_depth,
                                                         const float *g_sil) {
  constexpr int NT = Shape<TILE>::NT, PPT = Shape<TILE>::PPT;
  constexpr int NW = NT / kWave;
  constexpr int PER = (BATCH + NT - 1) / NT;
  static_assert((MODE & 2) != 0, "the twist alone has its own kernel");
  constexpr bool kTwist = (MODE & 1) != 0;
  constexpr bool kGeo = (MODE & 4) != 0;  // slots also carry dL/dp
  constexpr int NA = kGeo ? 8 : 5;        // floats per slot
  constexpr int G = Group<TILE, BATCH>::G, NH = 2 * G, NR = NW * PPT;
  // staged entry, the batch's last first: e0 (mx, my, qa, 2 qb), e1 (qc, o, z,
  // qb), e2 (c, r), ej (fx/z, fy/z, -fx px/z^2, -fy py/z^2) and for dL/dp
  // ep (px, py, 2 r^2 / z); a finished lane's last reads fall up to 32
  // entries past an array, into the next one's or the 32 at the end
  constexpr bool kDp = kTwist || kGeo;
  __shared__ float4 entries[(kDp ? 5 : 4) * BATCH + 32];
  float4 *const e0s = entries, *const e1s = e0s + BATCH, *const e2s = e1s + BATCH;
  float4 *const ejs = e2s + BATCH, *const eps_ = ejs + (kDp ? BATCH : 0);
  // per-wave slot accumulators: floats 0-3 in accA, 4 (4-7 with geometry)
  // in accB, and the claim tags of their read-modify-write
  __shared__ f32x4 accA[NW][BATCH];
  __shared__ AccB<kGeo> accB[NW][BATCH];
  __shared__ uint8_t tag_s[NW][BATCH + kWave];  // + a tag per lane
  __shared__ int maxlast_s;
  __shared__ float red_s[NW][7];
  __shared__ uint32_t words[NH + 1][NR][kWave];  // the last row zero

  const int t = tile_of_block(ws);
  const DevView &vw = ws.views[find_view_by_tile(ws, t)];
  const int lt = t - vw.tile_base;
  const int tx = lt % vw.tiles_x, ty = lt / vw.tiles_x;
  const int ox = tx * TILE, oy = ty * TILE;
  const uint2 rg = ws.ranges[t];
  const int start = (int)rg.x, end = (int)rg.y;
  const int w = threadIdx.x / kWave;

  BwdPixels<PPT> S;
  load_pixels<TILE, false>(ws, vw, ox, oy, g_rgb, g_depth, g_sil, TrackArgs{}, S);
  auto &px = S.px, &py = S.py, &T = S.T, &gC0 = S.gC0, &gC1 = S.gC1, &gC2 = S.gC2, &gD = S.gD;
  auto &E = S.E, &XP0 = S.XP0, &XP1 = S.XP1, &XP2 = S.XP2, &XPZ = S.XPZ, &GS1 = S.GS1;
  auto &last = S.last;
  const uint32_t mylast = S.mylast;
#pragma unroll
  for (int k = 0; k < PPT; k++) words[NH][w * PPT + k][lane_id()] = 0u;
  if (threadIdx.x == 0) maxlast_s = 0;
  __syncthreads();
  atomicMax(&maxlast_s, (int)mylast);
  __syncthreads();
  const int stop = start + maxlast_s;
  // this wave's own last contributor: entries past it touch none of its lanes
  const int wstop = start + __builtin_amdgcn_readfirstlane(wave_max_i((int)mylast));

  float tw[6] = {0.f, 0.f, 0.f, 0.f, 0.f, 0.f};
  const float amin = ws.amin, amax = ws.amax;
  const float vfx = vw.fx, vfy = vw.fy;

  // batches walk the list from the block's last contributor towards the front
  // batches on the forward's grid (start + multiples of BATCH), so each
  // 64-entry chunk is the forward's chunk and its lane bits apply
  const int nbat = (stop - start + BATCH - 1) / BATCH;
  // the batch below is gathered while the current one is replayed, and its
  // ids one batch ahead (positions clamped to the list, extra loads unused)
  BwdEntry st[PER];
  uint32_t pid[PER], slot[PER];  // (slot: of the entry this thread staged)
  const int n_rec = vw.n_rec, rec_base = vw.rec_base;
  // position of this thread's entry k in the batch starting at `blo`,
  // clamped to the list (batches below the first repeat its first entry)
  auto bpos = [&](int blo, int k) {
    return max(blo + min((int)threadIdx.x + k * NT, BATCH - 1), start);
  };
  if (nbat > 0) {
    const int lo = start + (nbat - 1) * BATCH;
#pragma unroll
    for (int k = 0; k < PER; k++) pid[k] = ws.ids[min(lo + (int)threadIdx.x + k * NT, stop - 1)];
#pragma unroll
    for (int k = 0; k < PER; k++) fetch_bwd_entry(ws, n_rec, rec_base, pid[k], st[k]);
#pragma unroll
    for (int k = 0; k < PER; k++) pid[k] = ws.ids[bpos(lo - BATCH, k)];
  }
  for (int bi = nbat - 1; bi >= 0; bi--) {
    const int lo = start + bi * BATCH;
    const int nb = min(stop, lo + BATCH) - lo;
    __syncthreads();
#pragma unroll
    for (int k = 0; k < PER; k++) {
      const int i = threadIdx.x + k * NT, j = BATCH - 1 - i;
      slot[k] = 0xffffffffu;
      if (i >= nb) continue;
      const BwdEntry &E = st[k];
      // (the doubled off-diagonal conic term is exact)
      e0s[j] = make_float4(E.e0.x, E.e0.y, E.e0.z, 2.0f * E.e0.w);
      const uint32_t sl = entry_slot(ws, E, tx, ty);
      // no slot (only after a capacity overflow): the entry learns nothing
      const bool learn = sl != 0xffffffffu && __float_as_int(E.e1.w) >= 0;
      e1s[j] = make_float4(E.e1.x, E.e1.y, E.e1.z, E.e0.w);
      // (r is NaN where the entry does not learn; a record with tiles has a
      // finite one, of either sign)
      e2s[j] = make_float4(E.e2.x, E.e2.y, E.e2.z, learn ? E.e2.w : __builtin_nanf(""));
      const float iz = 1.0f / E.e1.z;
      ejs[j] = make_float4(vfx * iz, vfy * iz, -vfx * E.eb.x * iz * iz, -vfy * E.eb.y * iz * iz);
      if (kDp) eps_[j] = make_float4(E.eb.x, E.eb.y, 2.0f * E.e2.w * E.e2.w * iz, 0.f);
      slot[k] = learn ? sl : 0xffffffffu;
#pragma unroll
      for (int ww = 0; ww < NW; ww++) {
        accA[ww][j] = f32x4{0.f, 0.f, 0.f, 0.f};
        accB[ww][j] = AccB<kGeo>{};
      }
    }
    __syncthreads();
    // the batches below are full ones (below the first: clamped, unused)
#pragma unroll
    for (int k = 0; k < PER; k++) fetch_bwd_entry(ws, n_rec, rec_base, pid[k], st[k]);
#pragma unroll
    for (int k = 0; k < PER; k++) pid[k] = ws.ids[bpos(lo - 2 * BATCH, k)];
    // this wave's entries, last to first, below its own last contributor
    const int lim = min(nb, wstop - lo);
    const int ctop = (lim - 1) / kWave;
    for (int g0 = (ctop / G) * G; lim > 0 && g0 >= 0; g0 -= G) {
      // 1. the entries of the group's chunks that reached each of this lane's
      // pixels in the forward, cut at the pixel's last contributor; the words
      // go in bit-reversed, top half first, so the lowest set bit of a word is
      // the lane's next entry towards the front
      uint32_t nz[PPT];
#pragma unroll
      for (int k = 0; k < PPT; k++) nz[k] = 0u;
      // the group's lane bits, all loads issued at once (chunks past the top
      // one reload the top one's, unused)
      unsigned long long lb[G][PPT];
#pragma unroll
      for (int cc = 0; cc < G; cc++) {
        const unsigned long long *src =
            ws.lane_bits + chunk_word(start, lo - start, min(g0 + cc, ctop), t, w, NW, PPT);
#pragma unroll
        for (int k = 0; k < PPT; k++) lb[cc][k] = src[k * kWave + lane_id()];
      }
#pragma unroll
      for (int cc = G - 1; cc >= 0; cc--) {
        const int c = g0 + cc;
        if (c > ctop) continue;
        const int base = lo - start + c * kWave;
#pragma unroll
        for (int k = 0; k < PPT; k++) {
          const int lim_k = (int)last[k] - base;
          const unsigned long long below =
              lim_k >= kWave ? ~0ull : (lim_k <= 0 ? 0ull : (1ull << lim_k) - 1ull);
          const unsigned long long own = lb[cc][k] & below;
          const uint32_t hi = __builtin_bitreverse32((uint32_t)(own >> 32));
          const uint32_t lo = __builtin_bitreverse32((uint32_t)own);
          constexpr int kTop = 2 * (G - 1);
          words[kTop - 2 * cc][w * PPT + k][lane_id()] = hi;
          words[kTop - 2 * cc + 1][w * PPT + k][lane_id()] = lo;
          nz[k] |= (hi ? 1u << (kTop - 2 * cc) : 0u) | (lo ? 2u << (kTop - 2 * cc) : 0u);
        }
      }
      // 2. each lane replays its own entries of the group, last to first, one
      // step per entry; the wave runs until its last lane is through.  As in
      // the forward, steps alternate between two register sets.
#pragma unroll
      for (int k = 0; k < PPT; k++) {
        const int row = w * PPT + k;
        const int gb = BATCH - kWave * (g0 + G);
        auto first = [](uint32_t v) { return __builtin_ctz(v | (1u << NH)); };
        uint32_t left = nz[k];
        int h = first(left);
        left &= left - 1u;
        int hn = first(left);
        uint32_t cur = words[h][row][lane_id()], nxt = words[hn][row][lane_id()];
        const int me = lane_id();
        // Each lane's adds of a step go into its wave's accumulators by
        // read-modify-write.  The lanes that replay one entry in a step claim
        // it by writing their lane number to its tag; with the claim they
        // read the tag back and the accumulators.  The claim is settled in
        // the next step, after that step's arithmetic has covered the reads'
        // latency: the lane whose number stayed in the tag (one per entry)
        // adds what it read to its values and writes them back, and the
        // lanes that lost then add theirs with LDS float atomics (6 % of the
        // lane steps of a mapping wave, against all of them with atomics
        // alone, which the LDS runs at about a lane per three clocks).  A
        // lane's last claim is settled in the step after its last entry.
        // Compiler barriers (kLdsOrder) keep each claim and settle in its
        // step and in program order.
        struct Entry {
          float4 e0, e1, e2, ej, ep;
          int i;
        };
        struct Claim {  // a step's values for entry idx, and what its claim read
          f32x4 va, ra;
          AccB<kGeo> vb, rb;
          int idx, rt;
        };
        auto fetch = [&](Entry &N) {
          N.i = gb + (h << 5) + low_bit(cur);
          N.e0 = e0s[N.i]; N.e1 = e1s[N.i]; N.e2 = e2s[N.i]; N.ej = ejs[N.i];
          if (kDp) N.ep = eps_[N.i];
        };
        // tag slot `ti` claimed, then read back with entry j's accumulators
        auto claim = [&](int ti, int j, Claim &C) {
          uint8_t LDS_AS *tg = (uint8_t LDS_AS *)&tag_s[w][ti];
          *tg = (uint8_t)me;
          kLdsOrder();
          C.rt = *tg;
          C.ra = *(f32x4 LDS_AS *)&accA[w][j];
          C.rb = *(AccB<kGeo> LDS_AS *)&accB[w][j];
          C.idx = j;
          kLdsOrder();
        };
        // the arithmetic of one step: issue the next entry's reads into N,
        // replay A into C's values; true where A learns
        auto replay = [&](const Entry &A, Entry &N, Claim &C) {
          cur &= cur - 1u;
          const bool z = cur == 0u;
          cur = z ? nxt : cur;
          h = z ? hn : h;
          left = z ? left & (left - 1u) : left;
          hn = first(left);
          nxt = words[hn][row][lane_id()];
          fetch(N);
          const float dx = px[k] - A.e0.x, dy = py[k] - A.e0.y;
          // q in the forward's order of operations
          const float ax = A.e0.z * dx, cy = A.e1.x * dy;
          const float q = fmaf(cy, dy, fmaf(A.e0.w * dx, dy, ax * dx));
          const float gau = __builtin_amdgcn_exp2f(q * kNegHalfLog2e);
          const float oG = A.e1.y * gau;
          const float a = fminf(amax, oG);
          const bool ok = a >= amin;
          const float om = 1.0f - a;
          const float Tk = ok ? T[k] * __builtin_amdgcn_rcpf(om) : T[k];
          T[k] = Tk;
          const float wgt = ok ? a * Tk : 0.f;
          // g . (x - B) for this Gaussian, x = (colour, depth, 1)
          const float gdi = fmaf(
              gC0[k], A.e2.x - XP0[k],
              fmaf(gC1[k], A.e2.y - XP1[k],
                   fmaf(gC2[k], A.e2.z - XP2[k], fmaf(gD[k], A.e1.z - XPZ[k], GS1[k] + E[k]))));
          const float dLda = ok ? gdi * Tk : 0.f;
          E[k] = ok ? om * gdi : E[k];
          XP0[k] = ok ? A.e2.x : XP0[k];
          XP1[k] = ok ? A.e2.y : XP1[k];
          XP2[k] = ok ? A.e2.z : XP2[k];
          XPZ[k] = ok ? A.e1.z : XPZ[k];
          GS1[k] = ok ? 0.f : GS1[k];
          const bool pass = oG <= amax;
          const float dLdq = pass ? -0.5f * oG * dLda : 0.f;
          const float w0 = fmaf(A.e0.z, dx, A.e1.w * dy), w1 = fmaf(A.e1.w, dx, cy);
          const float t0 = A.ej.x * w0, t1 = A.ej.y * w1, t2 = fmaf(A.ej.z, w0, A.ej.w * w1);
          // dL/dp of this pair (camera-frame centre)
          float g0v = 0.f, g1v = 0.f, g2v = 0.f;
          if (kDp) {
            const float kk = A.ep.z;
            g0v = dLdq * fmaf(kk * t0, t2, -2.0f * t0);
            g1v = dLdq * fmaf(kk * t1, t2, -2.0f * t1);
            const float s2 = fmaf(t0, t0, fmaf(t1, t1, 2.0f * t2 * t2));
            g2v = fmaf(dLdq, fmaf(kk, s2, -2.0f * t2), wgt * gD[k]);
          }
          if (kTwist) {
            const float pz = A.e1.z;
            tw[0] += g0v; tw[1] += g1v; tw[2] += g2v;
            tw[3] += A.ep.y * g2v - pz * g1v;
            tw[4] += pz * g0v - A.ep.x * g2v;
            tw[5] += A.ep.x * g1v - A.ep.y * g0v;
          }
          const float tt = fmaf(t0, t0, fmaf(t1, t1, t2 * t2));
          C.va = f32x4{wgt * gC0[k], wgt * gC1[k], wgt * gC2[k], pass ? gau * dLda : 0.f};
          const float v4 = dLdq * (-2.0f * A.e2.w * tt);
          if constexpr (kGeo) C.vb = f32x4{v4, g0v, g1v, g2v};
          else C.vb = v4;
          // the settle waits for the previous claim's reads: after the step's
          // arithmetic (which this empty statement consumes)
          asm volatile("" ::"v"(C.va[0]), "v"(C.va[1]), "v"(C.va[2]), "v"(C.va[3]), "v"(v4) : "memory");
          return ok && !__builtin_isnan(A.e2.w);
        };
        // the claim O settled in the lanes `open`: the lane whose number
        // stayed in the tag writes its sum back; then the lanes that lost add
        // theirs with LDS atomics (after that write, in the LDS's order)
        auto settle = [&](const Claim &O, unsigned long long open) {
          const bool po = in_lanes(open), won = po && O.rt == me;
          if (won) {
            *(f32x4 LDS_AS *)&accA[w][O.idx] = O.ra + O.va;
            *(AccB<kGeo> LDS_AS *)&accB[w][O.idx] = O.rb + O.vb;
          }
          kLdsOrder();
          if (po && !won) {
            float *fa = (float *)&accA[w][O.idx];
            float *fb = (float *)&accB[w][O.idx];
            atomicAdd(fa + 0, O.va[0]);
            atomicAdd(fa + 1, O.va[1]);
            atomicAdd(fa + 2, O.va[2]);
            atomicAdd(fa + 3, O.va[3]);
            if constexpr (kGeo) {
#pragma unroll
              for (int c = 0; c < 4; c++) atomicAdd(fb + c, O.vb[c]);
            } else {
              atomicAdd(fb, O.vb);
            }
          }
          kLdsOrder();
        };
        // a step of the lanes `live`; every one claims (a lane with nothing
        // to add on its own tag), so that the LDS operations behind the next
        // entry's reads are the same on every path and the next step waits
        // for those reads only.  Returns the lanes whose claim is open.
        auto step = [&](const Entry &A, Entry &N, Claim &C, const Claim &O, unsigned long long live,
                        unsigned long long open) {
          bool learns = false;
          if (in_lanes(live)) learns = replay(A, N, C);
          settle(O, open);
          if (in_lanes(live)) claim(learns ? A.i : BATCH + me, A.i, C);
          return lanes(learns);
        };
        Entry A, B;
        Claim C, D;
        unsigned long long open = 0ull;
        fetch(A);
        claim(BATCH + me, 0, D);  // (as before every later step; not settled)
        while (true) {
          unsigned long long live = lanes(cur != 0u);
          if ((live | open) == 0ull) break;
          open = step(A, B, C, D, live, open);
          live = lanes(cur != 0u);
          if ((live | open) == 0ull) break;
          open = step(B, A, D, C, live, open);
        }
      }
    }
    __syncthreads();
#pragma unroll
    for (int k = 0; k < PER; k++) {
      if (slot[k] == 0xffffffffu) continue;
      const int j = BATCH - 1 - ((int)threadIdx.x + k * NT);
      float *o = ws.slots + NA * (int64_t)slot[k];
      f32x4 sa = accA[0][j];
      AccB<kGeo> sb = accB[0][j];
#pragma unroll
      for (int ww = 1; ww < NW; ww++) {
        sa = sa + accA[ww][j];
        sb = sb + accB[ww][j];
      }
#pragma unroll
      for (int c = 0; c < 4; c++) o[c] = sa[c];
      if constexpr (kGeo) {
#pragma unroll
        for (int c = 0; c < 4; c++) o[4 + c] = sb[c];
      } else {
        o[4] = sb;
      }
    }
  }
  // list entries past every pixel's last contributor: zero slots
  for (int i = stop + (int)threadIdx.x; i < end; i += NT) {
    BwdEntry E;
    fetch_bwd_entry(ws, n_rec, rec_base, ws.ids[i], E);
    const uint32_t sl = entry_slot(ws, E, tx, ty);
    if (sl == 0xffffffffu) continue;
    float *o = ws.slots + NA * (int64_t)sl;
#pragma unroll
    for (int c = 0; c < NA; c++) o[c] = 0.f;
  }
  if (kTwist) store_twist<NW>(ws, t, tw, 0.f, red_s);
}

template <int TILE, int BATCH>
hipError_t fwd_launch(const Ws &ws, float *rgb, float *depth, float *sil, hipStream_t st) {
  hipLaunchKernelGGL((k_fwd<TILE, BATCH>), dim3(ws.n_tiles), dim3(Shape<TILE>::NT), 0, st, ws,
                     rgb, depth, sil);
  return hipGetLastError();
}

template <int TILE, int BATCH>
hipError_t bwd_launch(const Ws &ws, const float *g_rgb, const float *g_depth, const float *g_sil,
                      int mode, hipStream_t st) {
  const dim3 g(ws.n_tiles), b(Shape<TILE>::NT);
  switch (mode) {
    case 2: hipLaunchKernelGGL((k_bwd<TILE, BATCH, 2>), g, b, 0, st, ws, g_rgb, g_depth, g_sil); break;
    case 3: hipLaunchKernelGGL((k_bwd<TILE, BATCH, 3>), g, b, 0, st, ws, g_rgb, g_depth, g_sil); break;
    case 6: hipLaunchKernelGGL((k_bwd<TILE, BATCH, 6>), g, b, 0, st, ws, g_rgb, g_depth, g_sil); break;
    case 7: hipLaunchKernelGGL((k_bwd<TILE, BATCH, 7>), g, b, 0, st, ws, g_rgb, g_depth, g_sil); break;
    default: return hipErrorInvalidValue;
  }
  return hipGetLastError();
}

template <int TILE, int BATCH>
hipError_t twist_launch(const Ws &ws, const float *g_rgb, const float *g_depth, const float *g_sil,
                        hipStream_t st, const vtgs_track_cfg *track) {
  const dim3 g(ws.n_tiles), b(Shape<TILE>::NT);
  if (track) {
    const TrackArgs tr{track->alpha, track->beta, track->sil_thr};
    hipLaunchKernelGGL((k_bwd_twist<TILE, BATCH, true>), g, b, 0, st, ws, nullptr, nullptr, nullptr, tr);
  } else {
    hipLaunchKernelGGL((k_bwd_twist<TILE, BATCH, false>), g, b, 0, st, ws, g_rgb, g_depth, g_sil,
                       TrackArgs{});
  }
  return hipGetLastError();
}

template <int TILE>
hipError_t fwd_tile(const Ws &ws, float *rgb, float *depth, float *sil, hipStream_t st) {
  switch (ws.batch) {
    case 128: return fwd_launch<TILE, 128>(ws, rgb, depth, sil, st);
    // 16-pixel tiles take the default batch as passes of 512 entries: a pass
    // twice as long takes fewer steps (a lane waits less for its wave's
    // busiest) and fewer barriers, and at four blocks per CU it still beats
    // 256 at five: 12 tiles 30 -> 22 us, 80 tiles 32 -> 23, 1,200 tiles 44 ->
    // 41, 6,000 tiles of 1,400 entries 848 -> 758.  Only large grids of lists that
    // fill no pass lose: 3,225 tiles of a stride-2 map 110 us in passes of 128,
    // 125 in these (139 before the coverage was a matrix product); batch 128
    // remains for them.
    case 256: return fwd_launch<TILE, TILE == 16 ? 512 : 256>(ws, rgb, depth, sil, st);
    case 512: return fwd_launch<TILE, 512>(ws, rgb, depth, sil, st);
  }
  return hipErrorInvalidValue;
}

template <int TILE>
hipError_t bwd_tile(const Ws &ws, const float *a, const float *b, const float *c, int mode,
                    hipStream_t st, const vtgs_track_cfg *track) {
  if (mode == 1) {
    switch (ws.batch) {
      case 128: return twist_launch<TILE, 128>(ws, a, b, c, st, track);
      // 384 entries a pass at four blocks per CU (1,200 tiles 49 us, 80 tiles
      // 31, a batch of served tracks 1026) against 256 at five (54, 40 and
      // 1096) and 512 at three (51, 30 and 1035)
      case 256: return twist_launch<TILE, TILE == 16 ? 384 : 256>(ws, a, b, c, st, track);
      case 512: return twist_launch<TILE, 512>(ws, a, b, c, st, track);
    }
    return hipErrorInvalidValue;
  }
  switch (ws.batch) {
    case 128: return bwd_launch<TILE, 128>(ws, a, b, c, mode, st);
    case 256: return bwd_launch<TILE, 256>(ws, a, b, c, mode, st);
    case 512: return bwd_launch<TILE, 512>(ws, a, b, c, mode, st);
  }
  return hipErrorInvalidValue;
}

}  // namespace

hipError_t launch_composite_fwd(const Ws &ws, float *rgb, float *depth, float *sil,
                                hipStream_t st) {
  if (ws.n_tiles == 0) return hipSuccess;
  switch (ws.tile) {
    case 8: return fwd_tile<8>(ws, rgb, depth, sil, st);
    case 16: return fwd_tile<16>(ws, rgb, depth, sil, st);
    case 32: return fwd_tile<32>(ws, rgb, depth, sil, st);
  }
  return hipErrorInvalidValue;
}

hipError_t launch_composite_bwd(const Ws &ws, const float *g_rgb, const float *g_depth,
                                const float *g_sil, int mode, hipStream_t st,
                                const vtgs_track_cfg *track) {
  if (ws.n_tiles == 0) return hipSuccess;
  if (((mode & 4) != 0) != (ws.slot_w == 8) && (mode & 2)) return hipErrorInvalidValue;
  if (track && mode != 1) return hipErrorInvalidValue;
  switch (ws.tile) {
    case 8: return bwd_tile<8>(ws, g_rgb, g_depth, g_sil, mode, st, track);
    case 16: return bwd_tile<16>(ws, g_rgb, g_depth, g_sil, mode, st, track);
    case 32: return bwd_tile<32>(ws, g_rgb, g_depth, g_sil, mode, st, track);
  }
  return hipErrorInvalidValue;
}

}  // namespace vtgs
