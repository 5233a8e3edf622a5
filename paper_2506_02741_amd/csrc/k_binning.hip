// Preprocessing and tile binning of view-tied Gaussians.
//
//  preprocess per (view, Gaussian): M_vk = T_v T_k^-1; back-project the tied
//             depth pixel with the keyframe pose (Sec. 3.2), move it to the
//             view camera, project, Sigma_2D = r^2 J J^T + lowpass*I, conic,
//             extent R = ceil(sqrt(q_cut * lambda_max)), tile rectangle; then
//             count the Gaussian in each tile it covers (wave-aggregated
//             atomics, whose old values are the wave's positions in those
//             tiles; rectangles of many tiles go into a list)
//  scan_tiles exclusive scan of the tile counts -> per-tile [start, end)
//             (small plans: in the fill)
//  fill_keys  write (depth bits << 32 | view-local id) into the tile slots
//  sort_tiles sort each tile's keys (ascending depth, ties by id) in LDS and
//             emit the id list the compositing kernels walk
//  scan_recs  exclusive scan of tiles per record (gradient slot offsets)
//
// Every floating-point operation that decides a tile or a record is
// written in a fixed order and compiled without contraction, so the tile
// lists are bit-identical to an IEEE single-precision evaluation of the same
// expressions.
#include "vtgs_internal.h"
#include "geom32.h"

#pragma clang fp contract(off)

namespace vtgs {

namespace {

constexpr int kNT = 256;

__global__ void k_fill_u32(uint32_t *p, uint32_t v, int64_t n) {
  const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i < n) p[i] = v;
}

__global__ void k_fill_f32(float *p, float v, int64_t n) {
  const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i < n) p[i] = v;
}

__device__ __forceinline__ int find_seg(const Ws &ws, int r) {
  int lo = 0, hi = ws.n_segs - 1;
  while (lo < hi) {
    const int mid = (lo + hi + 1) >> 1;
    if (ws.segs[mid].rec_start <= r) lo = mid; else hi = mid - 1;
  }
  return lo;
}

__device__ __forceinline__ void unpack_rect(uint2 rc, int &x0, int &y0, int &x1, int &y1) {
  x0 = rc.x & 0xffff; y0 = rc.x >> 16; x1 = rc.y & 0xffff; y1 = rc.y >> 16;
}

__device__ __forceinline__ uint2 pack_rect(int x0, int y0, int x1, int y1) {
  return make_uint2((uint32_t)x0 | ((uint32_t)y0 << 16), (uint32_t)x1 | ((uint32_t)y1 << 16));
}

// Tiles of a shared box: one per lane.  64 stride-1 records span 5-6 tiles of
// 16 in two or three rows, stride-2 records 9-10 in two or three, so a limit
// of 24 had left most waves of a stride-2 map to per-pair atomics: serving
// track batches 570 -> 273 us (preprocess) and 576 -> 104 us (fill), 5 views
// over 8 stride-1 keyframes 440 -> 412 and 243 -> 113.
constexpr int kBoxMax = 64;
// Tiles of a group's box for its counters in LDS: a group that does not share
// a box (a few large rectangles among it, or it goes on in the next row of
// the image) still issues one atomic per tile, not per pair.  Pair by pair,
// groups next to the camera plane queue for the same few tiles: 134 K such
// records among 2 M cost the preprocess 60 us and the fill 100 us.
constexpr int kMidBox = 512;

// Tiles covered by a wave's rectangles (a group of 64 consecutive records).
// When the whole wave belongs to one view and its rectangles fit in a
// bounding box of at most kBoxMax tiles, box tile j (row-major) is owned by
// lane j: the lanes count their tiles in LDS counters, and lane j issues the
// global atomic of tile j, so one instruction serves the whole box.
// Otherwise the group's records of up to kLaneTiles tiles are counted in LDS
// if their box has at most kMidBox tiles, else (mixed views, or a larger box)
// by the lanes that stand at the same tile together.
struct WaveBox {
  int bx0, by0, nx, area;
  int src;  // a lane with a rectangle (when shared): its view is the box's
  bool shared;
};

// Lane-wise minimum or maximum of two 16-bit fields over the wave, as a
// uniform value: row_ror 8, 4, 2, 1 within rows, then row_bcast:15 and :31.
typedef unsigned short u16x2 __attribute__((ext_vector_type(2)));
template <bool kMax>
__device__ __forceinline__ uint32_t wave_pair(uint32_t x) {
  auto step = [&](uint32_t y) {
    const u16x2 a = __builtin_bit_cast(u16x2, x), b = __builtin_bit_cast(u16x2, y);
    x = __builtin_bit_cast(uint32_t, kMax ? __builtin_elementwise_max(a, b) : __builtin_elementwise_min(a, b));
  };
  step((uint32_t)__builtin_amdgcn_update_dpp((int)x, (int)x, 0x128, 0xf, 0xf, false));
  step((uint32_t)__builtin_amdgcn_update_dpp((int)x, (int)x, 0x124, 0xf, 0xf, false));
  step((uint32_t)__builtin_amdgcn_update_dpp((int)x, (int)x, 0x122, 0xf, 0xf, false));
  step((uint32_t)__builtin_amdgcn_update_dpp((int)x, (int)x, 0x121, 0xf, 0xf, false));
  step((uint32_t)__builtin_amdgcn_update_dpp((int)x, (int)x, 0x142, 0xa, 0xf, false));
  step((uint32_t)__builtin_amdgcn_update_dpp((int)x, (int)x, 0x143, 0xc, 0xf, false));
  return (uint32_t)__builtin_amdgcn_readlane((int)x, kWave - 1);
}

// (views do not decrease from lane to lane; a lane past the last record gives
// that record's)
__device__ __forceinline__ WaveBox wave_box(bool has, int view, int x0, int y0, int x1, int y1,
                                            int most) {
  WaveBox b;
  const unsigned long long any = ballot64(has);
  const bool one_view = __builtin_amdgcn_readlane(view, 0) == __builtin_amdgcn_readlane(view, kWave - 1);
  const uint2 rc = pack_rect(x0, y0, x1, y1);
  const uint32_t lo = wave_pair<false>(has ? rc.x : 0xffffffffu), hi = wave_pair<true>(has ? rc.y : 0u);
  b.bx0 = (int)(lo & 0xffffu);
  b.by0 = (int)(lo >> 16);
  b.nx = (int)(hi & 0xffffu) - b.bx0 + 1;
  const long area = any ? (long)b.nx * (long)((int)(hi >> 16) - b.by0 + 1) : 0;
  b.shared = any && one_view && area <= most;
  b.area = b.shared ? (int)area : 0;
  b.src = (int)__builtin_ctzll(any | (1ull << 63));
  return b;
}

// An empty statement the compiler must take as reading and writing all
// memory: LDS accesses keep their program order across it, and the LDS
// executes a wave's accesses in that order.
__device__ __forceinline__ void lds_order() { asm volatile("" ::: "memory"); }

// Box tile j (row-major in the box) as a tile index of the box's view (tiles_x
// btx, first tile btb); tiles past the box are unused.
__device__ __forceinline__ int box_tile(const WaveBox &b, int j, int btx, int btb) {
  const int nx = max(b.nx, 1);
  const int q = j / nx;
  return btb + (b.by0 + q) * btx + (b.bx0 + (j - q * nx));
}

// The numbers of the wave's rectangles covering each box tile, in the wave's
// own LDS row `cnt`.
__device__ __forceinline__ void box_counts(const WaveBox &b, bool has, int x0, int y0, int x1, int y1,
                                           uint32_t *cnt) {
  for (int j = lane_id(); j < b.area; j += kWave) cnt[j] = 0u;
  lds_order();
  if (has) {
    for (int ty = y0; ty <= y1; ty++)
      for (int tx = x0; tx <= x1; tx++) atomicAdd(&cnt[(ty - b.by0) * b.nx + (tx - b.bx0)], 1u);
  }
  lds_order();
}

// Rectangles of a group without a shared box: a lane walks a small one by
// itself, one atomic per tile.  One of more than kLaneTiles tiles (a Gaussian
// close to the view's camera plane covers thousands) goes into a list of its
// own: it adds to its tiles' counts as the ends of its rows in a difference
// array over the tile indexes, which the tile scan sums up, and its pairs are
// stored tile by tile (fill_wide), at the ends of the tiles' lists.
// Measured on a section of 10 stride-2 keyframes in a 1200x680 view (3,225
// tiles), 2,400 of whose 2 M records cover more than 64 tiles, most of them
// all: preprocess and fill take 0.19 + 0.30 ms with the wave walking such a
// rectangle together, an atomic per pair (1.89 + 4.60 ms with its lane
// alone), 0.08 + 0.04 ms with the list and the counters of kMidBox.  The line:
// a listed record costs a test per tile of its view (1.2 ns in all for 3,225
// tiles, less where most have none), its pairs in a lane's walk 30 ps each; at
// 64 (81 tiles a record) the list is faster in plans of one to forty views.
constexpr int kLaneTiles = 64;

// The lanes standing at the same tile as this one: the first of them, their
// number and this lane's rank among them (all lanes of the wave call this;
// `on` where a lane stands at a tile).
struct SameTile {
  int first;
  uint32_t n, rank;
};
__device__ __forceinline__ SameTile same_tile(bool on, int t) {
  SameTile s = {0, 0u, 0u};
  unsigned long long todo = ballot64(on);
  while (todo) {
    const int src = (int)__builtin_ctzll(todo);
    const bool mine = on && t == __builtin_amdgcn_readlane(t, src);
    const unsigned long long m = ballot64(mine);
    if (mine) {
      s.first = src;
      s.n = (uint32_t)__popcll(m);
      s.rank = (uint32_t)__popcll(m & lanemask_lt());
    }
    todo &= ~m;
  }
  return s;
}

// One lane's walk over the tiles of its rectangle, row by row.
struct TileWalk {
  int tx, ty;
  __device__ __forceinline__ void next(int x0, int x1) {
    if (++tx > x1) { tx = x0; ty++; }
  }
};

__device__ __forceinline__ bool is_wide(bool has, int x0, int y0, int x1, int y1) {
  return has && (x1 - x0 + 1) * (y1 - y0 + 1) > kLaneTiles;
}

// The list: (record, depth bits, rectangle) in the buffer of the tile sort's
// runs, which is free until then.  Half of it is divided among the views by
// their records, so that a tile's wave reads its own view's alone (with one
// list for all views the fill grew by their square: 300 views of 300 tiles with
// 200 such records each took 2.11 ms, against 0.19; without any of them 0.10);
// the other half takes what a view's part does not (views of few records with
// many wide ones, in plans of little capacity).
__device__ __forceinline__ uint4 *wide_list(const Ws &ws) {
  return reinterpret_cast<uint4 *>(ws.keys_tmp);
}
struct WidePart {
  int64_t first;
  uint32_t n;
};
__device__ __forceinline__ WidePart wide_part(const Ws &ws, int64_t rec_base, int64_t n_rec) {
  const int64_t first = rec_base * ws.wide_part >> 16;
  return {first, (uint32_t)(((rec_base + n_rec) * ws.wide_part >> 16) - first)};
}
__device__ __forceinline__ WidePart wide_rest(const Ws &ws) {
  return {ws.cap / 4, (uint32_t)(ws.cap / 2 - ws.cap / 4)};
}
// The first word of n_wide: whether the pass has such records, and whether there
// were more than the rest holds.  Those past its end are left out: each has more
// than kLaneTiles pairs, so the pass is over the pair capacity anyway; it counts
// its pairs and leaves all lists empty.
constexpr uint32_t kWideAny = 1u, kWideFull = 2u;

// The wave's wide records into the list and their rows into the difference
// array, one interval for all rows of a rectangle as wide as the view.
__device__ __forceinline__ void add_wide(const Ws &ws, bool wide, int view, int r, uint32_t zbits, int x0,
                                         int y0, int x1, int y1, int tiles_x, int t0) {
  if (!wide) return;
  const SameTile sv = same_tile(true, view);
  uint32_t i = 0u;
  if (sv.rank == 0u) {
    i = atomicAdd(view_wide(ws, view), sv.n);
    if (i == 0u) atomicOr(ws.n_wide, kWideAny);
  }
  i = (uint32_t)__shfl((int)i, sv.first) + sv.rank;
  WidePart part = wide_part(ws, ws.views[view].rec_base, ws.views[view].n_rec);
  if (i >= part.n) {
    part = wide_rest(ws);
    i = atomicAdd(ws.n_wide + kWideRest, 1u);
    if (i == part.n) atomicOr(ws.n_wide, kWideFull);
  }
  const uint2 rc = pack_rect(x0, y0, x1, y1);
  if (i < part.n) wide_list(ws)[part.first + i] = make_uint4((uint32_t)r, zbits, rc.x, rc.y);
  const bool full = x0 == 0 && x1 == tiles_x - 1;
  const int rows = full ? 1 : y1 - y0 + 1, len = full ? (y1 - y0 + 1) * tiles_x : x1 - x0 + 1;
  for (int q = 0; q < rows; q++) {
    // (rectangles over all of the view begin and end at the same two tiles)
    const int a = t0 + (y0 + q) * tiles_x + x0, b = a + len;
    const SameTile sa = same_tile(true, a), sb = same_tile(b < ws.n_tiles, b);
    if (sa.rank == 0u) atomicAdd(ws.tile_fill + a, sa.n);
    if (b < ws.n_tiles && sb.rank == 0u) atomicSub(ws.tile_fill + b, sb.n);
  }
}

// The wide records' keys, at the ends of the lists of the tiles that they
// cover: a wave takes a tile, its lanes the list's records, 64 at a time, U
// of these chunks in flight, until the tile has as many as were counted.
template <int U, typename Range>
__device__ __forceinline__ void fill_wide(const Ws &ws, uint32_t n_rest, uint32_t n_first, int wave, int n_waves,
                                          Range range) {
  for (int t = wave; t < ws.n_tiles; t += n_waves) {
    const uint2 rg = range(t);
    // (of a list cut off at the capacity: the positions past the others)
    const uint32_t others = ws.tile_count[t] + ws.tile_count_ns[t];
    uint32_t left = rg.y - rg.x - min(rg.y - rg.x, others);
    if (!left) continue;
    uint32_t end = rg.y;
    int lo = 0, hi = ws.n_views - 1;
    while (lo < hi) {
      const int mid = (lo + hi + 1) >> 1;
      if (ws.views[mid].tile_base <= t) lo = mid; else hi = mid - 1;
    }
    const DevView &vw = ws.views[lo];
    const uint32_t r0 = vw.rec_base, r1 = r0 + vw.n_rec;
    const int tiles_x = vw.tiles_x, at = t - vw.tile_base;
    const int ty = at / tiles_x, tx = at - ty * tiles_x;
    auto walk = [&](const uint4 *list, uint32_t n) {
      for (uint32_t c = 0; c < n && left; c += U * kWave) {
        uint4 e[U];
#pragma unroll
        for (int u = 0; u < U; u++) e[u] = list[min(c + u * kWave + lane_id(), n - 1)];
#pragma unroll
        for (int u = 0; u < U; u++) {
          int x0, y0, x1, y1;
          unpack_rect(make_uint2(e[u].z, e[u].w), x0, y0, x1, y1);
          const bool in = c + u * kWave + lane_id() < n && e[u].x >= r0 && e[u].x < r1 && x0 <= tx &&
                          tx <= x1 && y0 <= ty && ty <= y1;
          const unsigned long long m = ballot64(in);
          const uint32_t rank = (uint32_t)__popcll(m & lanemask_lt());
          if (in && rank < left)
            ws.keys[end - 1u - rank] = ((unsigned long long)e[u].y << 32) | (e[u].x - r0);
          const uint32_t n_in = min(left, (uint32_t)__popcll(m));
          left -= n_in;
          end -= n_in;
        }
      }
    };
    const WidePart part = wide_part(ws, r0, vw.n_rec);
    walk(wide_list(ws) + part.first, min(lo ? *view_wide(ws, lo) : n_first, part.n));
    walk(wide_list(ws) + wide_rest(ws).first, n_rest);
  }
}

// A load through a descriptor's pointer, which addresses global memory:
// read as such (the compiler cannot tell, and would issue a flat load).
template <class T>
__device__ __forceinline__ T gload(const T *p, int64_t i) {
  return ((const __attribute__((address_space(1))) T *)p)[i];
}

// The same through the scalar cache, where the address is the wave's: for
// what no kernel writes while this one runs (descriptors' constants, poses).
template <class T>
__device__ __forceinline__ T uload(const T *p) {
  return *(const __attribute__((address_space(4))) T *)p;
}

constexpr int kViewLds = 256;  // view descriptors the key fill keeps in LDS

// A record's view and tiles.
struct Projected {
  int view, x0, y0, x1, y1, tiles_x, tile_base;
  uint32_t zbits;
  bool has;
};

// Column and row of pixel index pix in an image of width w: the quotient from
// a reciprocal, off by one at most (pix < 2^24, w >= 8: its error is below
// 0.4), then put right.
__device__ __forceinline__ void pixel_of(uint32_t pix, uint32_t w, int &u, int &v) {
  uint32_t q, r;
  if (w < 8u || ballot64(pix >= 1u << 24)) {
    q = pix / w;
    r = pix % w;
  } else {
    q = (uint32_t)((float)pix * __builtin_amdgcn_rcpf((float)w));
    r = pix - q * w;
    if ((int)r < 0) { r += w; q--; }
    if (r >= w) { r -= w; q++; }
  }
  u = (int)r;
  v = (int)q;
}

// Record r of segment seg.  kOneSeg: the segment is the block's (and the lanes
// past the last record run along): its descriptors and pointers stay in scalar
// registers, and three lanes form a row each of the relative pose.  Otherwise
// every lane reads its own.
template <bool kOneSeg>
__device__ __forceinline__ Projected project_record(const Ws &ws, int seg, int r, bool active) {
  Projected o = {0, 1, 0, 0, 0, 1, 0, 0u, false};
  const DevSeg &sg = ws.segs[seg];
  const int kfi = kOneSeg ? uload(&sg.kf) : sg.kf, rec_start = kOneSeg ? uload(&sg.rec_start) : sg.rec_start;
  o.view = kOneSeg ? uload(&sg.view) : sg.view;
  const DevKF &kf = ws.kfs[kfi];
  const DevView &vw = ws.views[o.view];
  // the descriptor fields used below, read up front (not inside branches)
  auto get = [](const auto &x) { return kOneSeg ? uload(&x) : x; };
  const float kfx = get(kf.fx), kfy = get(kf.fy), kcx = get(kf.cx), kcy = get(kf.cy);
  const float vfx = get(vw.fx), vfy = get(vw.fy), vcx = get(vw.cx), vcy = get(vw.cy);
  const int kwidth = get(kf.width), kn = get(kf.n), klearn = get(kf.learnable);
  const uint32_t *kpix = get(kf.pix);
  const float *kdepth = get(kf.depth), *kradius = get(kf.radius), *kopa = get(kf.opacity),
              *kcolor = get(kf.color);
  const float *vpose = get(vw.pose), *kpose = get(kf.pose);
  const int tiles_y = get(vw.tiles_y);
  o.tiles_x = get(vw.tiles_x);
  o.tile_base = get(vw.tile_base);
  // (a lane past the last record reads the segment's last one)
  const int i = min(r - rec_start, kn - 1);
  // the two poses and every per-Gaussian load issued together, before the
  // arithmetic (and before any store, which the compiler could not move
  // them past)
  const uint32_t pix = gload(kpix, i);
  const float d = gload(kdepth, i);
  const float rad = gload(kradius, i);
  const float opa = gload(kopa, i);
  const float c0 = gload(kcolor, i), c1 = gload(kcolor, (int64_t)kn + i), c2 = gload(kcolor, 2 * (int64_t)kn + i);
  float M[12];
  if (kOneSeg) {
    float tv[4], tk[12];
    const int row = min(lane_id() & 3, 2);
#pragma unroll
    for (int c = 0; c < 4; c++) tv[c] = gload(vpose, 4 * row + c);
#pragma unroll
    for (int c = 0; c < 12; c++) tk[c] = uload(kpose + c);
    float m[4];
    relative_pose_row(tv, tk, m);
#pragma unroll
    for (int c = 0; c < 12; c++)
      M[c] = __int_as_float(__builtin_amdgcn_readlane(__float_as_int(m[c % 4]), c / 4));
  } else {
    float tv[12], tk[12];
#pragma unroll
    for (int c = 0; c < 12; c++) { tv[c] = gload(vpose, c); tk[c] = gload(kpose, c); }
    relative_pose(tv, tk, M);
  }
  int u, v;
  pixel_of(pix, (uint32_t)kwidth, u, v);
  // back-projection of the tied depth pixel (keyframe camera), into the view
  float px, py, pz;
  backproject_move(M, kfx, kfy, kcx, kcy, u, v, d, px, py, pz);
  float mx = 0.f, my = 0.f, qa = 0.f, qb = 0.f, qc = 0.f, R = 0.f;
  if (active && pz > ws.znear) {
    mx = vfx * (px / pz) + vcx;
    my = vfy * (py / pz) + vcy;
    const float a = vfx / pz, b = vfy / pz;
    const float zz = pz * pz;
    const float jx = -(vfx * px) / zz, jy = -(vfy * py) / zz;
    const float r2 = rad * rad;
    const float s11 = r2 * (a * a + jx * jx) + ws.lowpass;
    const float s12 = r2 * (jx * jy);
    const float s22 = r2 * (b * b + jy * jy) + ws.lowpass;
    const float det = s11 * s22 - s12 * s12;
    if (det > 0.f) {
      const float mid = 0.5f * (s11 + s22);
      const float lmax = mid + sqrtf(fmaxf(0.f, mid * mid - det));
      R = ceilf(sqrtf(ws.qcut * lmax));
      if (__builtin_isfinite(mx) && __builtin_isfinite(my) && __builtin_isfinite(R)) {
        qa = s22 / det; qb = -s12 / det; qc = s11 / det;
        const float invB = 1.0f / (float)ws.tile;
        const float fx0 = fmaxf(floorf((mx - R) * invB), 0.f);
        const float fy0 = fmaxf(floorf((my - R) * invB), 0.f);
        const float fx1 = fminf(floorf((mx + R) * invB), (float)(o.tiles_x - 1));
        const float fy1 = fminf(floorf((my + R) * invB), (float)(tiles_y - 1));
        if (!(fx0 > fx1 || fy0 > fy1)) {
          o.x0 = (int)fx0; o.y0 = (int)fy0; o.x1 = (int)fx1; o.y1 = (int)fy1;
          o.has = true;
        }
      }
    }
  }
  if (!active) return o;
  o.zbits = __float_as_uint(pz);
  float4 *A = ws.recA + 3 * (int64_t)r;
  A[0] = make_float4(mx, my, qa, qb);
  // (R >= 0: its sign bit is free)
  A[1] = make_float4(qc, opa, pz, __builtin_copysignf(R, klearn ? 1.f : -1.f));
  A[2] = make_float4(c0, c1, c2, rad);
  if (o.has) ws.recB[r] = make_float2(px, py);
  if (o.has && !all_finite(c0, c1, c2, pz)) *odd_records(ws) = 1u;
  ws.rect[r] = pack_rect(o.x0, o.y0, o.x1, o.y1);
  // the depth again on its own, so that the key fill reads 4 B per record
  ws.zbits[r] = o.zbits;
  // the segment's relative pose, kept for the gradient gathers
  if (r == rec_start) {
#pragma unroll
    for (int c = 0; c < 12; c++) ws.segs[seg].M[c] = M[c];
  }
  return o;
}

// Bound by its stores, some 75 bytes a record (1.2 GB with the loads for 5
// views over 8 keyframes of 640x480, 12.3 M records: 290 us, a copy's 260).
// Nearly every block lies within one segment: then the descriptors are scalar
// loads and operands instead of 24 pose loads and 64-bit addresses per lane
// (410 us, the arithmetic alone 226; 2 M records: 82 -> 63).
__global__ __attribute__((amdgpu_waves_per_eu(8))) __launch_bounds__(kNT) void k_preprocess(Ws ws) {
  const int r = blockIdx.x * kNT + threadIdx.x;
  __shared__ uint32_t box_cnt[kNT / kWave][kMidBox];
  __shared__ uint32_t slot_cnt[kNT / kWave];
  const bool active = r < ws.n_rec;
  Projected o = {0, 1, 0, 0, 0, 1, 0, 0u, false};
  if (ws.n_rec > 0) {
    // the segment of the block's first record, found with scalar loads, and
    // the first record of the next one
    int lo = 0, hi = ws.n_segs - 1;
    const int b0 = blockIdx.x * kNT;
    while (lo < hi) {
      const int mid = (lo + hi + 1) >> 1;
      if (uload(&ws.segs[mid].rec_start) <= b0) lo = mid; else hi = mid - 1;
    }
    if (lo == ws.n_segs - 1 || uload(&ws.segs[lo + 1].rec_start) >= min(b0 + kNT, ws.n_rec))
      o = project_record<true>(ws, lo, r, active);
    else
      o = project_record<false>(ws, find_seg(ws, min(r, ws.n_rec - 1)), r, active);
  }
  // positions for this pass's key fill
  if (ws.tile_claim)
    for (int t = r; t < ws.n_tiles; t += (int)gridDim.x * kNT) ws.tile_claim[t] = 0u;
  // one more pass of the pipeline: the tracking update writes its loss at
  // this index, so a captured iteration needs no per-iteration argument
  if (r == 0) *ws.iter += 1u;
  const bool has = o.has;
  const int view = o.view, x0 = o.x0, y0 = o.y0, x1 = o.x1, y1 = o.y1, tiles_x = o.tiles_x,
            tile_base = o.tile_base;
  if (ws.slots) {
    // plans with gradients per Gaussian: the records' tiles, summed up to
    // and with this one over the block, for the slot offsets
    const uint32_t n = has ? (uint32_t)((x1 - x0 + 1) * (y1 - y0 + 1)) : 0u;
    const uint32_t before = block_exclusive_scan<kNT>(n, slot_cnt, nullptr);
    if (active) ws.rec_cnt[r] = before + n;
  }
  const WaveBox box = wave_box(has, view, x0, y0, x1, y1, kBoxMax);
  uint32_t *cnt = box_cnt[threadIdx.x / kWave];
  if (box.shared) {
    // the lanes count their tiles in the wave's LDS row, then lane j adds
    // box tile j's count with one atomic instruction for the whole box.
    // Lane j need not hold a record of the box's view (or any record), so
    // the tile index takes that view's geometry from a lane that does.
    const int btx = __builtin_amdgcn_readlane(tiles_x, box.src);
    const int btb = __builtin_amdgcn_readlane(tile_base, box.src);
    const int mt = box_tile(box, lane_id(), btx, btb);
    box_counts(box, has, x0, y0, x1, y1, cnt);
    const uint32_t mine = lane_id() < box.area ? cnt[lane_id()] : 0u;
    // the atomic's old value is the group's first position in box tile j:
    // kept for the key fill, which then claims nothing for this group
    if (mine) ws.wave_off[(r & ~(kWave - 1)) + lane_id()] = atomicAdd(ws.tile_count + mt, mine);
  } else {
    // the other groups' pairs take the positions after them, claimed by
    // the key fill
    const bool wide = is_wide(has, x0, y0, x1, y1), small = has && !wide;
    const WaveBox mid = wave_box(small, view, x0, y0, x1, y1, kMidBox);
    if (mid.shared) {
      const int btx = __builtin_amdgcn_readlane(tiles_x, mid.src);
      const int btb = __builtin_amdgcn_readlane(tile_base, mid.src);
      box_counts(mid, small, x0, y0, x1, y1, cnt);
      for (int j = lane_id(); j < mid.area; j += kWave)
        if (cnt[j]) atomicAdd(ws.tile_count_ns + box_tile(mid, j, btx, btb), cnt[j]);
    } else {
      const int last = small ? y1 : -1;
      for (TileWalk w = {x0, y0}; ballot64(w.ty <= last); w.next(x0, x1)) {
        const int t = tile_base + w.ty * tiles_x + w.tx;
        const SameTile s = same_tile(w.ty <= last, t);
        if (w.ty <= last && s.rank == 0u) atomicAdd(ws.tile_count_ns + t, s.n);
      }
    }
    add_wide(ws, wide, view, r, o.zbits, x0, y0, x1, y1, tiles_x, tile_base);
  }
}

// Longest lists of the tile sorts (keys in LDS): a 256-thread block takes up
// to kSmallSort, a 512-thread one up to kMidSort, a 1024-thread one the rest.
constexpr int kSmallSort = 1024, kMidSort = 4096;

// One block: tile counts -> ranges (clamped to the pair capacity), total
// pairs, capacity flag; lists longer than kSmallSort are queued for the
// long-list sorts, those over kMidSort from the queue array's end.
constexpr int kScanNT = 1024, kScanPer = 8;
constexpr int kOrderBuckets = 64;
// Bucket of a list of n entries in the longest-first order: 0 for the
// longest, eight per octave from 64 entries on, then one for shorter lists and
// one for empty ones.  (With two per octave the lists of a tracking frame, 590
// entries on average and 750 at most, shared one bucket.)
__device__ __forceinline__ int order_bucket(uint32_t n) {
  if (n < 64u) return kOrderBuckets - (n ? 2 : 1);
  const int bl = 32 - __clz((int)n);  // 7 ..
  return max(kOrderBuckets - 3 - (8 * (bl - 7) + (int)((n >> (bl - 4)) & 7u)), 0);
}

// Groups of records for the slot offsets: kRecBlocks blocks of the
// preprocess, whose sums the blocks of the tile scan past the first add up.
constexpr int kRecBlocks = 8, kRecGroup = kNT * kRecBlocks;

// The tiles of the kNT records from b on (0 past the end): the block's last
// running sum.
__device__ __forceinline__ uint32_t block_tiles(const Ws &ws, int64_t b) {
  return b < ws.n_rec ? ws.rec_cnt[min(b + kNT, (int64_t)ws.n_rec) - 1] : 0u;
}

// Sums of the record groups, one lane per preprocess block (the words lie 1 KB
// apart); block: the caller's index among the blocks doing this.
template <int NT>
__device__ __forceinline__ void group_sums(const Ws &ws, int block, int n_groups) {
  const int b = block * NT + threadIdx.x;
  uint32_t s = block_tiles(ws, (int64_t)b * kNT);
#pragma unroll
  for (int o = 1; o < kRecBlocks; o <<= 1) s += (uint32_t)__shfl_xor((int)s, o);
  if (b % kRecBlocks == 0 && b / kRecBlocks < n_groups) ws.scan_part[b / kRecBlocks] = s;
}

// The range of a list of n entries from pos, cut off at the capacity.
__device__ __forceinline__ uint2 list_range(unsigned long long pos, uint32_t n, unsigned long long cap) {
  return make_uint2((uint32_t)min(pos, cap), (uint32_t)min(pos + n, cap));
}

// The tile scan inside each block of the key fill (plans with a tile_claim:
// one view, at most kFillTiles tiles): every block sums up all counts for
// itself, the first one stores the results.  With 75 blocks and 80 tiles
// (160x120) the fill takes 4.8 us with or without it and the scan's launch
// (4.7 us) is saved; with 1,200 and 1,200 (640x480) it took 14.6 us instead of
// 4.8 + 5.9.  At the line, with about 510 blocks: a render of 512 tiles takes 44.0
// us, one of 520 with the scan 47.0 (stride 2, 125 blocks: 30.1 and 33.9).
constexpr int kFillPer = kFillTiles / kNT;
__device__ __forceinline__ void scan_in_fill(const Ws &ws, uint32_t n_wide, bool store, uint2 *range,
                                             uint32_t *lw) {
  const unsigned long long cap = n_wide & kWideFull ? 0 : ws.cap;
  const int i0 = threadIdx.x * kFillPer;
  uint32_t v[kFillPer], sum = 0u, tot;
#pragma unroll
  for (int k = 0; k < kFillPer; k++) {
    v[k] = i0 + k < ws.n_tiles ? ws.tile_count[i0 + k] + ws.tile_count_ns[i0 + k] : 0u;
    sum += v[k];
  }
  if (n_wide) {
    uint32_t d[kFillPer], w = 0u;
#pragma unroll
    for (int k = 0; k < kFillPer; k++) {
      d[k] = i0 + k < ws.n_tiles ? ws.tile_fill[i0 + k] : 0u;
      w += d[k];
    }
    w = block_exclusive_scan<kNT>(w, lw, nullptr);
#pragma unroll
    for (int k = 0; k < kFillPer; k++) {
      w += d[k];
      if (i0 + k < ws.n_tiles) { v[k] += w; sum += w; }
    }
  }
  unsigned long long pos = block_exclusive_scan<kNT>(sum, lw, &tot);
#pragma unroll
  for (int k = 0; k < kFillPer; k++) {
    const uint2 rg = list_range(pos, v[k], cap);
    range[i0 + k] = rg;
    if (store && i0 + k < ws.n_tiles) ws.ranges[i0 + k] = rg;
    pos += v[k];
  }
  if (store && threadIdx.x == 0) {
    *ws.n_pairs = tot;
    if (tot > (unsigned long long)ws.cap) atomicOr(ws.flags, kFlagCapacity);
  }
  __syncthreads();
}

__global__ __launch_bounds__(kScanNT) void k_scan_tiles(Ws ws, int n_groups) {
  if (blockIdx.x > 0) {
    group_sums<kScanNT>(ws, blockIdx.x - 1, n_groups);
    return;
  }
  __shared__ uint32_t lw[kScanNT / kWave];
  __shared__ unsigned long long carry_s;
  __shared__ uint32_t nlong_s, nhuge_s;
  __shared__ uint32_t bk[kOrderBuckets];
  __shared__ uint32_t wide_s;
  if (threadIdx.x == 0) { carry_s = 0; nlong_s = 0; nhuge_s = 0; wide_s = 0; }
  // wide records: their rows' ends in tile_fill become counts per tile
  const uint32_t n_wide = ws.n_wide[0];
  const unsigned long long cap = n_wide & kWideFull ? 0 : ws.cap;
  if (threadIdx.x < kOrderBuckets) bk[threadIdx.x] = 0u;
  __syncthreads();
  // a plan of one round keeps its tiles' buckets and their ranks there
  const bool one_round = ws.n_tiles <= kScanNT * kScanPer;
  int bucket[kScanPer];
  uint32_t rank[kScanPer];
  for (int base = 0; base < ws.n_tiles; base += kScanNT * kScanPer) {
    const int i0 = base + threadIdx.x * kScanPer;
    uint32_t v[kScanPer], vs[kScanPer], sum = 0;
    for (int k = 0; k < kScanPer; k++) {
      vs[k] = (i0 + k < ws.n_tiles) ? ws.tile_count[i0 + k] : 0u;
      v[k] = vs[k] + ((i0 + k < ws.n_tiles) ? ws.tile_count_ns[i0 + k] : 0u);
      sum += v[k];
    }
    uint32_t tot;
    if (n_wide) {
      uint32_t d[kScanPer], ds = 0;
      for (int k = 0; k < kScanPer; k++) {
        d[k] = (i0 + k < ws.n_tiles) ? ws.tile_fill[i0 + k] : 0u;
        ds += d[k];
      }
      uint32_t w = wide_s;
      w += block_exclusive_scan<kScanNT>(ds, lw, &tot);
      for (int k = 0; k < kScanPer; k++) {
        w += d[k];
        if (i0 + k < ws.n_tiles) { v[k] += w; sum += w; }
      }
      if (threadIdx.x == 0) wide_s += tot;
    }
    const uint32_t ex = block_exclusive_scan<kScanNT>(sum, lw, &tot);
    const unsigned long long c = carry_s;
    unsigned long long pos = c + ex;
    for (int k = 0; k < kScanPer; k++) {
      const int i = i0 + k;
      if (i < ws.n_tiles) {
        const uint2 rg = list_range(pos, v[k], cap);
        const uint32_t len = rg.y - rg.x;
        ws.ranges[i] = rg;
        if (len > (uint32_t)kMidSort)
          ws.long_tiles[(uint32_t)ws.n_tiles - 1u - atomicAdd(&nhuge_s, 1u)] = i;
        else if (len > (uint32_t)kSmallSort)
          ws.long_tiles[atomicAdd(&nlong_s, 1u)] = i;
        ws.tile_fill[i] = vs[k];
        if (ws.tile_order) {
          bucket[k] = order_bucket(len);
          rank[k] = atomicAdd(&bk[bucket[k]], 1u);
        }
      }
      pos += v[k];
    }
    __syncthreads();
    if (threadIdx.x == 0) carry_s = c + tot;
    __syncthreads();
  }
  if (threadIdx.x == 0) {
    *ws.n_pairs = carry_s;
    if (carry_s > (unsigned long long)ws.cap) atomicOr(ws.flags, kFlagCapacity);
    ws.n_long[0] = nlong_s;
    ws.n_long[1] = nhuge_s;
    ws.n_wide[1] = n_wide;
  }
  if (ws.tile_order) {
    // longest lists first: tiles bucketed by list length (eight buckets per
    // octave, longest first, empty lists last), so that the compositing
    // grid, dispatched in block order, starts its heaviest tiles first and
    // ends on light ones; the order within a bucket is whatever the atomics
    // give (each tile's results do not depend on it)
    // (the last round's barriers stand between the counts and here)
    if (threadIdx.x < kOrderBuckets) {
      const uint32_t c = bk[threadIdx.x];
      bk[threadIdx.x] = wave_incl_scan_u32(c) - c;
    }
    __syncthreads();
    if (one_round) {
      for (int k = 0; k < kScanPer; k++) {
        const int i = threadIdx.x * kScanPer + k;
        if (i < ws.n_tiles) ws.tile_order[bk[bucket[k]] + rank[k]] = (uint32_t)i;
      }
      return;
    }
    for (int i = threadIdx.x; i < ws.n_tiles; i += kScanNT)
      ws.tile_order[atomicAdd(&bk[order_bucket(ws.ranges[i].y - ws.ranges[i].x)], 1u)] = (uint32_t)i;
  }
}

// Keys into tile slots.  A thread takes RPT records, r = (block * RPT + k) *
// kNT + thread, so that each k is a group of 64 consecutive records, the
// preprocess's wave; the loads of all k are issued first, then every
// group's slot bases, then the key stores, so that a wave waits on one
// round trip per phase rather than one per group (large plans; the tracking
// frame, with ~5 waves per SIMD, takes one record per thread).  A group whose
// rectangles share a tile box recomputes the preprocess's box and takes the
// positions its atomics returned; the other groups claim positions after
// all of those with atomics here.  Either way a tile's keys land in no fixed
// order; the sort that follows fixes it.
//
// The grid: rec_blocks blocks of records, wide_blocks for the wide records
// and, with kScan (the tile scan is done here), blocks of record groups.
template <int RPT, bool kScan>
__global__ __launch_bounds__(kNT) void k_fill_keys(Ws ws, int rec_blocks, int wide_blocks, int n_groups) {
  __shared__ uint2 range_s[kScan ? kFillTiles : 1];
  __shared__ uint32_t lw[kNT / kWave];
  const uint32_t n_wide = kScan ? ws.n_wide[0] : ws.n_wide[1];
  if ((int)blockIdx.x >= rec_blocks + wide_blocks) {
    if (kScan) group_sums<kNT>(ws, blockIdx.x - rec_blocks - wide_blocks, n_groups);
    return;
  }
  auto range = [&](int t) { return kScan ? range_s[t] : ws.ranges[t]; };
  // n positions of tile t's list, after those of the shared boxes
  auto claim = [&](int t, uint32_t n) {
    return kScan ? ws.tile_count[t] + atomicAdd(ws.tile_claim + t, n) : atomicAdd(ws.tile_fill + t, n);
  };
  if ((int)blockIdx.x >= rec_blocks) {
    constexpr int kWaves = kNT / kWave;
    const uint32_t n_rest = ws.n_wide[kWideRest], n_first = *view_wide(ws, 0);
    if (!n_wide || n_wide & kWideFull) return;
    if (kScan) scan_in_fill(ws, n_wide, false, range_s, lw);
    fill_wide<4>(ws, n_rest, n_first, (blockIdx.x - rec_blocks) * kWaves + threadIdx.x / kWave,
                 wide_blocks * kWaves, range);
    return;
  }
  // the views' first records, tiles per row and first tiles, read by the
  // block at once beside its records' loads and then searched in LDS
  // (plans with more views search the descriptors in global memory, plans
  // with one read its descriptor without a search)
  __shared__ int3 vtab[kViewLds];
  __shared__ uint32_t fill_pos[kNT / kWave][kMidBox], fill_lim[kNT / kWave][kMidBox];
  const bool view_lds = ws.n_views > 1 && ws.n_views <= kViewLds;
  bool has[RPT];
  int x0[RPT], y0[RPT], x1[RPT], y1[RPT], tiles_x[RPT], tile_base[RPT], view[RPT];
  unsigned long long key[RPT];
  uint32_t zb[RPT];
  uint2 rc[RPT];
#pragma unroll
  for (int k = 0; k < RPT; k++) {
    const int r = (blockIdx.x * RPT + k) * kNT + threadIdx.x;
    const int rr = max(min(r, ws.n_rec - 1), 0);
    rc[k] = ws.rect[rr];
    zb[k] = ws.zbits[rr];
  }
  if (kScan) {
    scan_in_fill(ws, n_wide, blockIdx.x == 0, range_s, lw);
    if (ws.n_rec == 0) return;
  }
  if (view_lds) {
    for (int v = threadIdx.x; v < ws.n_views; v += kNT)
      vtab[v] = make_int3(ws.views[v].rec_base, ws.views[v].tiles_x, ws.views[v].tile_base);
    __syncthreads();
  }
#pragma unroll
  for (int k = 0; k < RPT; k++) {
    const int r = (blockIdx.x * RPT + k) * kNT + threadIdx.x;
    const int rr = min(r, ws.n_rec - 1);
    const bool active = r < ws.n_rec;
    unpack_rect(rc[k], x0[k], y0[k], x1[k], y1[k]);
    has[k] = active && x0[k] <= x1[k];
    if (!has[k]) { x0[k] = 1; y0[k] = 0; x1[k] = 0; y1[k] = 0; }
    int rec_base;
    if (view_lds) {
      int lo = 0, hi = ws.n_views - 1;
      while (lo < hi) {
        const int mid = (lo + hi + 1) >> 1;
        if (vtab[mid].x <= rr) lo = mid; else hi = mid - 1;
      }
      view[k] = lo;
      const int3 e = vtab[view[k]];
      rec_base = e.x; tiles_x[k] = e.y; tile_base[k] = e.z;
    } else {
      view[k] = find_view_by_record(ws, rr);
      const DevView &vw = ws.views[view[k]];
      rec_base = vw.rec_base; tiles_x[k] = vw.tiles_x; tile_base[k] = vw.tile_base;
    }
    key[k] = ((unsigned long long)zb[k] << 32) | (uint32_t)(r - rec_base);
  }
  // lane j of a group with a shared box: box tile j's first position and
  // end
  WaveBox box[RPT];
  uint32_t base[RPT], end[RPT];
#pragma unroll
  for (int k = 0; k < RPT; k++) {
    box[k] = wave_box(has[k], view[k], x0[k], y0[k], x1[k], y1[k], kBoxMax);
    base[k] = 0u; end[k] = 0u;
    if (!box[k].shared) continue;
    const int btx = __builtin_amdgcn_readlane(tiles_x[k], box[k].src);
    const int btb = __builtin_amdgcn_readlane(tile_base[k], box[k].src);
    if (lane_id() < box[k].area) {
      // the group's first position in box tile j, claimed by the
      // preprocess (unused, and never written, where no rectangle of the
      // group covers the tile)
      const uint2 rg = range(box_tile(box[k], lane_id(), btx, btb));
      const int g0 = (blockIdx.x * RPT + k) * kNT + (threadIdx.x & ~(kWave - 1));
      base[k] = rg.x + ws.wave_off[g0 + lane_id()];
      end[k] = rg.y;
    }
  }
  // stores: the next position and the end of each box tile's list lie in the
  // wave's LDS row; every lane then takes a position in each box tile its
  // rectangle covers (in whatever order the lanes come: the sort fixes it).
  // Groups without a shared box claim their tiles' positions first, and those
  // of no box store pair by pair.
  uint32_t *pos = fill_pos[threadIdx.x / kWave], *lim = fill_lim[threadIdx.x / kWave];
#pragma unroll
  for (int k = 0; k < RPT; k++) {
    auto put = [&](const WaveBox &b) {
      for (int ty = y0[k]; ty <= y1[k]; ty++)
        for (int tx = x0[k]; tx <= x1[k]; tx++) {
          const int j = (ty - b.by0) * b.nx + (tx - b.bx0);
          const uint32_t at = atomicAdd(&pos[j], 1u);
          if (at < lim[j]) ws.keys[at] = key[k];
        }
    };
    if (box[k].shared) {
      pos[lane_id()] = base[k];
      lim[lane_id()] = end[k];
      lds_order();
      if (has[k]) put(box[k]);
      lds_order();
      continue;
    }
    const bool small = has[k] && !is_wide(has[k], x0[k], y0[k], x1[k], y1[k]);
    const WaveBox mid = wave_box(small, view[k], x0[k], y0[k], x1[k], y1[k], kMidBox);
    if (mid.shared) {
      const int btx = __builtin_amdgcn_readlane(tiles_x[k], mid.src);
      const int btb = __builtin_amdgcn_readlane(tile_base[k], mid.src);
      box_counts(mid, small, x0[k], y0[k], x1[k], y1[k], pos);
      // (the claims of four tiles per lane in flight)
#pragma unroll 4
      for (int j = lane_id(); j < mid.area; j += kWave) {
        const uint32_t n = pos[j];
        const int t = box_tile(mid, j, btx, btb);
        const uint2 rg = range(t);
        if (n) pos[j] = rg.x + claim(t, n);
        lim[j] = rg.y;
      }
      lds_order();
      if (small) put(mid);
      lds_order();
    } else {
      const int last = small ? y1[k] : -1;
      for (TileWalk w = {x0[k], y0[k]}; ballot64(w.ty <= last); w.next(x0[k], x1[k])) {
        const bool on = w.ty <= last;
        const int t = on ? tile_base[k] + w.ty * tiles_x[k] + w.tx : 0;
        const SameTile s = same_tile(on, t);
        uint32_t at = 0u;
        if (on && s.rank == 0u) at = range(t).x + claim(t, s.n);
        at = (uint32_t)__shfl((int)at, s.first) + s.rank;
        if (on && at < range(t).y) ws.keys[at] = key[k];
      }
    }
  }
}

constexpr int kSortCap = 8192;

// One round of a merge sort over n keys held as sorted runs of `width`
// keys in `in`: each pair of neighbouring runs is merged into `out` (an odd
// run at the end is copied), written as D (u64: the keys, u32: the ids).
// Every thread takes an equal share of each merged pair's output, finds
// where its share starts by a binary search along the merge path, and
// merges its share serially.  Keys are unique and below ~0, so ~0 serves
// as the end of either run.
template <int NT, typename D>
__device__ void merge_round(const unsigned long long *in, D *out, int n, int width) {
  for (int lo = 0; lo < n; lo += 2 * width) {
    const int mid = min(lo + width, n), hi = min(lo + 2 * width, n);
    const unsigned long long *A = in + lo, *B = in + mid;
    const int la = mid - lo, lb = hi - mid, m = hi - lo;
    const int d0 = (int)((int64_t)m * threadIdx.x / NT);
    const int d1 = (int)((int64_t)m * (threadIdx.x + 1) / NT);
    // the first d0 outputs are A[0, i) and B[0, d0 - i)
    int a = max(0, d0 - lb), b = min(d0, la);
    while (a < b) {
      const int md = (a + b) >> 1;
      if (A[md] < B[d0 - md - 1]) a = md + 1;
      else b = md;
    }
    int i = a, j = d0 - a;
    unsigned long long va = i < la ? A[i] : ~0ull, vb = j < lb ? B[j] : ~0ull;
    for (int d = d0; d < d1; d++) {
      const bool ta = va < vb;
      out[lo + d] = (D)(ta ? va : vb);
      if (ta) { i++; va = i < la ? A[i] : ~0ull; }
      else { j++; vb = j < lb ? B[j] : ~0ull; }
    }
  }
}

// The LDS of a tile sort: the keys, the buckets and small tables (bins, coarse
// and cbase are also read four words at a time: 16 bytes, and sizes that keep
// the arrays before them at multiples of 16).
template <int NT, int E>
struct alignas(16) SortLds {
  static constexpr int CAP = NT * E;
  static_assert(CAP % 4 == 0, "bins, coarse and cbase begin at multiples of 16 bytes");
  unsigned long long buf[CAP];
  uint32_t bins[CAP + 4];
  uint32_t coarse[256], cbase[256];
  uint32_t wsum[NT / kWave], zlo[NT / kWave], zhi[NT / kWave], ilo[NT / kWave], ihi[NT / kWave];
};

constexpr uint32_t kMaxBucket = 48;  // keys of a bucket ranked by comparison
// A list whose depths differ by less than this many steps of a float is
// bucketed by depth and id together: on a plane seen face on, from its
// keyframe's own pose, whole tiles have one depth or a few neighbouring ones.
// (16 bits: with 16 of the id they fill a word; more steps than that already
// divide finer than the buckets.)  Sorts of flat frames, with it, without
// (every list bitonic) and by radix passes before there were buckets: one
// 640x480 keyframe 10, 35 and 15 us, six of them 72, 165 and 206, a 64x48 one 9,
// 24 and 10; frames of other depths take as long as without.
constexpr uint32_t kNearDepths = 1u << 16;

// Sort of one tile's n <= NT * E keys (depth bits << 32 | id, unique), written
// to dst in ascending key order as D (u32: the ids, u64: the keys), by two
// levels of buckets.  256 coarse buckets divide the list's own depth range
// evenly; a coarse bucket of c keys is divided evenly into c fine ones, so
// that surfaces that fill a small part of the range still get buckets of
// their own.  Both maps are monotone in the key, so a key's place is its
// fine bucket's start plus its rank among that bucket's few keys, counted by
// comparing whole keys.  Every pass is LDS atomics or independent reads, ~20
// VALU instructions per key in all, against five dependent radix passes of
// 23 or more before; a list of up to 1024 keys is spread over four waves, where one
// wave had sorted it alone: tracking frame 15.8 -> 6.8 us (9.3 with the clearing
// of the counters, which this kernel does too), 5 views over 8 keyframes (lists of ~1,400) 560 -> 138.  Returns false, with dst untouched,
// when a fine bucket holds more than kMaxBucket keys (many equal depths at a
// few values far apart, of a sensor's steps): a bitonic sort, which needs no
// registers to speak of, takes those lists (a room at 1 mm steps, lists of
// 620, 1,240 and 3,730 keys: 25, 92 and 215 us against 26, 933 and 608 of the
// radix passes).
template <int NT, int E, typename D>
__device__ __forceinline__ bool bucket_sort(const unsigned long long (&k)[E], D *dst, int n,
                                            SortLds<NT, E> &S) {
  constexpr int NW = NT / kWave;
  static_assert(E % 4 == 0, "fine buckets are scanned four at a time");
  const int t = threadIdx.x, l = lane_id(), w = t / kWave;
  // a word's range over the keys, wave by wave (the sign bit flipped: signed
  // comparisons in the keys' unsigned order)
  auto range = [&](int shift, uint32_t *lows, uint32_t *highs) {
    int lo = 0x7fffffff, hi = (int)0x80000000;
#pragma unroll
    for (int e = 0; e < E; e++) {
      const bool in = t + NT * e < n;
      const int z = (int)((uint32_t)(k[e] >> shift) ^ 0x80000000u);
      lo = in ? min(lo, z) : lo;
      hi = in ? max(hi, z) : hi;
    }
    lo = wave_min_i(lo);
    hi = wave_max_i(hi);
    if (l == 0) { lows[w] = (uint32_t)lo ^ 0x80000000u; highs[w] = (uint32_t)hi ^ 0x80000000u; }
  };
  range(32, S.zlo, S.zhi);
  if (t < 256) S.coarse[t] = 0u;
  uint4 *bins4 = (uint4 *)S.bins;
#pragma unroll
  for (int e = 0; e < E / 4; e++) bins4[t * (E / 4) + e] = make_uint4(0u, 0u, 0u, 0u);
  __syncthreads();
  uint32_t lo = S.zlo[0], hi = S.zhi[0];
#pragma unroll
  for (int i = 1; i < NW; i++) { lo = min(lo, S.zlo[i]); hi = max(hi, S.zhi[i]); }
  // a key's place in the list's range: its depth, and where the depths are near
  // each other its id behind it (ib bits of the id's own range)
  uint32_t ilo = 0u, most_place = hi - lo;
  int ib = 0, is = 31;
  if (hi - lo < kNearDepths) {
    range(0, S.ilo, S.ihi);
    __syncthreads();
    uint32_t ihi = S.ihi[0];
    ilo = S.ilo[0];
#pragma unroll
    for (int i = 1; i < NW; i++) { ilo = min(ilo, S.ilo[i]); ihi = max(ihi, S.ihi[i]); }
    const int bits = 32 - __clz((int)(ihi - ilo));
    ib = min(bits, 16);
    is = bits - ib;
    most_place = ((hi - lo) << ib) + ((ihi - ilo) >> is);
  }
  // (elsewhere no bit of the id is left: it is below 2^31)
  auto place = [&](unsigned long long key) {
    return (((uint32_t)(key >> 32) - lo) << ib) + (((uint32_t)key - ilo) >> is);
  };
  const int shift = max(0, 24 - __clz((int)most_place));  // most_place >> shift < 256
  // fine position within a coarse bucket: at most 16 bits of the place
  const int fb = min(shift, 16), fs = shift - fb;
#pragma unroll
  for (int e = 0; e < E; e++)
    if (t + NT * e < n) atomicAdd(&S.coarse[place(k[e]) >> shift], 1u);
  __syncthreads();
  if (w == 0) {  // exclusive scan of the 256 coarse counts
    const uint4 c = ((const uint4 *)S.coarse)[l];
    const uint32_t sum = c.x + c.y + c.z + c.w;
    const uint32_t ex = wave_incl_scan_u32(sum) - sum;
    ((uint4 *)S.cbase)[l] = make_uint4(ex, ex + c.x, ex + c.x + c.y, ex + c.x + c.y + c.z);
  }
  __syncthreads();
  uint32_t f[E], slot[E];
#pragma unroll
  for (int e = 0; e < E; e++) {
    if (t + NT * e >= n) continue;
    const uint32_t z = place(k[e]), c = z >> shift;
    const uint32_t part = (z & ((1u << shift) - 1u)) >> fs;
    f[e] = S.cbase[c] + ((part * S.coarse[c]) >> fb);
    slot[e] = atomicAdd(&S.bins[f[e]], 1u);
  }
  __syncthreads();
  // exclusive scan of the fine counts in place
  uint4 c[E / 4];
  uint32_t sum = 0u, most = 0u;
#pragma unroll
  for (int e = 0; e < E / 4; e++) {
    c[e] = bins4[t * (E / 4) + e];
    sum += (c[e].x + c[e].y) + (c[e].z + c[e].w);
    most = max(most, max(max(c[e].x, c[e].y), max(c[e].z, c[e].w)));
  }
  const uint32_t inc = wave_incl_scan_u32(sum);
  if (l == kWave - 1) S.wsum[w] = inc;
  if (__syncthreads_or(most > kMaxBucket)) return false;
  uint32_t run = inc - sum;
#pragma unroll
  for (int i = 0; i < NW; i++) run += i < w ? S.wsum[i] : 0u;
#pragma unroll
  for (int e = 0; e < E / 4; e++) {
    const uint4 o = make_uint4(run, run + c[e].x, run + c[e].x + c[e].y, run + c[e].x + c[e].y + c[e].z);
    run = o.w + c[e].w;
    bins4[t * (E / 4) + e] = o;
  }
  if (t == NT - 1) S.bins[NT * E] = run;
  __syncthreads();
#pragma unroll
  for (int e = 0; e < E; e++)
    if (t + NT * e < n) S.buf[S.bins[f[e]] + slot[e]] = k[e];
  __syncthreads();
#pragma unroll
  for (int e = 0; e < E; e++) {
    if (t + NT * e >= n) continue;
    const uint32_t b0 = S.bins[f[e]], b1 = S.bins[f[e] + 1];
    uint32_t r = b0;
    for (uint32_t j = b0; j < b1; j++) r += S.buf[j] < k[e] ? 1u : 0u;
    slot[e] = r;
  }
  __syncthreads();
  D *out = (D *)S.buf;
#pragma unroll
  for (int e = 0; e < E; e++)
    if (t + NT * e < n) out[slot[e]] = (D)k[e];
  __syncthreads();
  for (int i = t; i < n; i += NT) dst[i] = out[i];
  return true;
}

// Sort of one tile's n <= NT * E keys, written to dst in ascending key order
// as D (u32: the ids, u64: the keys).
template <int NT, int E, typename D>
__device__ __forceinline__ void sort_tile_keys(const unsigned long long *src, D *dst, int n,
                                               SortLds<NT, E> &S) {
  unsigned long long k[E];
  // coalesced loads (any starting arrangement sorts to the same result, the
  // keys being unique), every load first (clamped index), then the padding
#pragma unroll
  for (int e = 0; e < E; e++) k[e] = src[min((int)threadIdx.x + NT * e, n - 1)];
  if (bucket_sort<NT, E>(k, dst, n, S)) return;
  // bitonic sort in LDS of the next power of two, padded with ~0 (above every
  // key, a depth's bits being below the infinity bits)
  const int m = 2 << (31 - __clz(n - 1));
  __syncthreads();  // (the keys' LDS may still be read by the bucket sort)
#pragma unroll
  for (int e = 0; e < E; e++) {
    const int i = (int)threadIdx.x + NT * e;
    if (i < m) S.buf[i] = i < n ? k[e] : ~0ull;
  }
  for (int run = 2; run <= m; run *= 2)
    for (int d = run / 2; d > 0; d /= 2) {
      __syncthreads();
      for (int p = threadIdx.x; p < m / 2; p += NT) {
        const int i = 2 * p - (p & (d - 1)), j = i + d;
        const unsigned long long a = S.buf[i], b = S.buf[j];
        if ((a > b) == ((i & run) == 0)) { S.buf[i] = b; S.buf[j] = a; }
      }
    }
  __syncthreads();
  for (int i = threadIdx.x; i < n; i += NT) dst[i] = (D)S.buf[i];
}

// One block per tile: keys (depth bits << 32 | id) are unique within a tile,
// so ascending key order is the (depth, id) order.  Each variant handles the
// tiles whose length lies in (lo_n, hi_n], queue 0: every tile, 1 and 2: the
// scan's queues of mid and huge lists.  Blocks take their tiles by position:
// a shared cursor, one atomic per tile, cost the mid lists 20 us a turn (768
// blocks waiting for the same address).
template <int NT, int E>
__global__ __attribute__((amdgpu_waves_per_eu(NT == 256 ? 8 : NT == 512 ? 6 : 4)))
__launch_bounds__(NT) void k_sort_tiles(Ws ws, int lo_n, int hi_n, int queue) {
  constexpr int CAP = NT * E;
  __shared__ SortLds<NT, E> S;
  const int count = queue ? (int)ws.n_long[queue - 1] : ws.n_tiles;
  // the fill is done with the tile counters and the number of wide records:
  // cleared for the next pass, by blocks of their own (the mark of records
  // that are not finite goes to the compositors first)
  if (NT == 256 && (int)blockIdx.x >= ws.n_tiles) {
    const int i = ((int)blockIdx.x - ws.n_tiles) * NT + threadIdx.x;
    const int64_t pitch = counter_pitch(ws.n_tiles);
    for (int a = 0; a < 3; a++)
      if (i < ws.n_tiles) ws.tile_count[a * pitch + i] = 0u;
    if (i < ws.n_views) *view_wide(ws, i) = 0u;
    if (i == 0) {
      ws.n_wide[0] = 0u;
      ws.n_wide[kWideRest] = 0u;
      odd_records(ws)[1] = odd_records(ws)[0];
      odd_records(ws)[0] = 0u;
    }
    return;
  }
  const int blocks = NT == 256 ? ws.n_tiles : (int)gridDim.x;
  for (int q = blockIdx.x; q < count; q += blocks) {
    const int tile = queue == 0 ? q : (int)ws.long_tiles[queue == 1 ? q : ws.n_tiles - 1 - q];
    // ranges are clamped to the capacity, and every position of a clamped
    // range was written by the fill, so sorting stays in bounds on overflow
    const uint2 rg = ws.ranges[tile];
    const int n = (int)(rg.y - rg.x);
    if (n <= lo_n || n > hi_n || n <= 0) continue;
    const unsigned long long *src = ws.keys + rg.x;
    uint32_t *dst = ws.ids + rg.x;
    if (n == 1) {
      if (threadIdx.x == 0) dst[0] = (uint32_t)src[0];
      continue;
    }
    if (n <= CAP) {
      sort_tile_keys<NT, E>(src, dst, n, S);
    } else {
      // longer than the LDS holds: runs of CAP keys sorted in LDS into
      // keys_tmp, then merged pairwise, back and forth between keys_tmp and
      // the tile's own key range (free once its runs are sorted); the last
      // round writes the ids
      unsigned long long *runs = ws.keys_tmp + rg.x, *spare = ws.keys + rg.x;
      for (int lo = 0; lo < n; lo += CAP) {
        sort_tile_keys<NT, E>(src + lo, runs + lo, min(CAP, n - lo), S);
        __syncthreads();  // the LDS is reused by the next run
      }
      const unsigned long long *in = runs;
      unsigned long long *out = spare;
      int width = CAP;
      for (; 2 * width < n; width *= 2) {
        merge_round<NT>(in, out, n, width);
        __syncthreads();
        unsigned long long *nxt = const_cast<unsigned long long *>(in);
        in = out;
        out = nxt;
      }
      merge_round<NT>(in, dst, n, width);
    }
    __syncthreads();  // the LDS is reused by the block's next tile
  }
}

// Records' slot offsets: the exclusive sums of their tile counts over all
// records.  The preprocess leaves sums within its blocks, the tile scan adds
// up the groups of kRecGroup records; what is left is one pass over the
// records, in which each block adds up the groups before its own (at most
// 1024 blocks, so that this stays linear in the groups).  Scanning the counts
// themselves took three launches of 26 + 8 + 50 us at 12.3 M records, this
// one takes 26 us (98 MB).
__global__ __launch_bounds__(kNT) void k_scan_records(Ws ws, int n_groups, int per) {
  __shared__ uint32_t lw[kNT / kWave];
  const int g0 = blockIdx.x * per, g1 = min(g0 + per, n_groups);
  if (g0 >= n_groups) return;
  uint32_t s = 0, base;
  for (int g = threadIdx.x; g < g0; g += kNT) s += ws.scan_part[g];
  block_exclusive_scan<kNT>(s, lw, &base);
  for (int g = g0; g < g1; g++) {
    uint32_t before[kRecBlocks], sum[kRecBlocks];
#pragma unroll
    for (int k = 0; k < kRecBlocks; k++) {
      const int64_t b = ((int64_t)g * kRecBlocks + k) * kNT, r = b + threadIdx.x;
      before[k] = threadIdx.x > 0 && r < ws.n_rec ? ws.rec_cnt[r - 1] : 0u;
      sum[k] = block_tiles(ws, b);
    }
#pragma unroll
    for (int k = 0; k < kRecBlocks; k++) {
      const int64_t r = ((int64_t)g * kRecBlocks + k) * kNT + threadIdx.x;
      if (r < ws.n_rec) ws.rec_off[r] = base + before[k];
      base += sum[k];
    }
  }
  if (g1 == n_groups && threadIdx.x == 0) ws.rec_off[ws.n_rec] = base;
}

__global__ void k_debug_copy(Ws ws, float *records, int32_t *rect) {
  const int r = blockIdx.x * blockDim.x + threadIdx.x;
  if (r >= ws.n_rec) return;
  if (records) {
    const float4 a = ws.recA[3 * (int64_t)r], b = ws.recA[3 * (int64_t)r + 1],
                 c = ws.recA[3 * (int64_t)r + 2];
    float *o = records + 12 * (int64_t)r;
    o[0] = a.x; o[1] = a.y; o[2] = a.z; o[3] = a.w;
    o[4] = b.x; o[5] = b.y; o[6] = b.z; o[7] = fabsf(b.w);
    o[8] = c.x; o[9] = c.y; o[10] = c.z; o[11] = c.w;
  }
  if (rect) {
    int x0, y0, x1, y1;
    unpack_rect(ws.rect[r], x0, y0, x1, y1);
    int32_t *o = rect + 4 * (int64_t)r;
    o[0] = x0; o[1] = y0; o[2] = x1; o[3] = y1;
  }
}

inline unsigned blocks_for(int64_t n, int nt) { return (unsigned)((n + nt - 1) / nt); }

}  // namespace

hipError_t launch_fill_u32(uint32_t *p, uint32_t v, int64_t n, hipStream_t st) {
  if (n <= 0) return hipSuccess;
  hipLaunchKernelGGL(k_fill_u32, dim3(blocks_for(n, kNT)), dim3(kNT), 0, st, p, v, n);
  return hipGetLastError();
}

hipError_t launch_fill_f32(float *p, float v, int64_t n, hipStream_t st) {
  if (n <= 0) return hipSuccess;
  hipLaunchKernelGGL(k_fill_f32, dim3(blocks_for(n, kNT)), dim3(kNT), 0, st, p, v, n);
  return hipGetLastError();
}

hipError_t launch_preprocess(const Ws &ws, hipStream_t st) {
  // at least one block: it bumps the pass counter
  const int64_t nb = ws.n_rec > 0 ? blocks_for(ws.n_rec, kNT) : 1;
  hipLaunchKernelGGL(k_preprocess, dim3(nb), dim3(kNT), 0, st, ws);
  return hipGetLastError();
}


hipError_t launch_scan_tiles(const Ws &ws, hipStream_t st) {
  if (ws.tile_claim) return hipSuccess;  // part of the key fill
  const int ng = ws.slots ? (int)rec_scan_blocks(ws.n_rec) : 0;
  hipLaunchKernelGGL(k_scan_tiles, dim3(1 + blocks_for((int64_t)ng * kRecBlocks, kScanNT)), dim3(kScanNT), 0, st, ws, ng);
  return hipGetLastError();
}

hipError_t launch_fill_keys(const Ws &ws, hipStream_t st) {
  // a wave per tile for the wide records
  const int wide = (int)std::min(blocks_for(ws.n_tiles, kNT / kWave), 2048u);
  if (ws.tile_claim) {
    const int nb = std::max((int)blocks_for(ws.n_rec, kNT), 1);
    const int ng = ws.slots ? (int)rec_scan_blocks(ws.n_rec) : 0;
    hipLaunchKernelGGL((k_fill_keys<1, true>), dim3(nb + wide + blocks_for((int64_t)ng * kRecBlocks, kNT)),
                       dim3(kNT), 0, st, ws, nb, wide, ng);
    return hipGetLastError();
  }
  if (ws.n_rec == 0) return hipSuccess;
  // two records per thread once the grid holds several waves per SIMD at
  // that rate (1,024 SIMDs; 12.3 M records: 112 us with four, 102 with two, 103
  // with one, 2 M: 40, 41, 44)
  if (ws.n_rec >= (1 << 20)) {
    const int nb = (int)blocks_for(ws.n_rec, 2 * kNT);
    hipLaunchKernelGGL((k_fill_keys<2, false>), dim3(nb + wide), dim3(kNT), 0, st, ws, nb, wide, 0);
  } else {
    const int nb = (int)blocks_for(ws.n_rec, kNT);
    hipLaunchKernelGGL((k_fill_keys<1, false>), dim3(nb + wide), dim3(kNT), 0, st, ws, nb, wide, 0);
  }
  return hipGetLastError();
}

// Whether the records' expected pairs per tile (a Gaussian of extent ~4-5 px
// covers about (1 + 10 / B)^2 tiles of side B) make long lists the rule.
bool long_lists(double n_rec, double n_tiles, int tile) {
  const double per = (1.0 + 10.0 / tile) * (1.0 + 10.0 / tile);
  return per * n_rec > 1024.0 * n_tiles;
}

hipError_t launch_sort_tiles(const Ws &ws, hipStream_t st) {
  // Where long lists are the rule, lists of up to 1024 go to 256-thread blocks,
  // those of up to 4096, queued by the scan, to 512-thread blocks (three per
  // CU) and longer ones to 1024-thread blocks (one per CU; 8192 keys in LDS,
  // longer lists merged from runs), each grid a few rounds of the device's
  // blocks.  Otherwise the 256-thread blocks sort every list, a long one (the
  // odd one) as runs of 1024 merged in rounds, and no other kernel is launched
  // (an empty launch costs a tracking iteration ~5 us).
  const bool many = long_lists(ws.n_rec, ws.n_tiles, ws.tile);
  hipLaunchKernelGGL((k_sort_tiles<256, kSmallSort / 256>), dim3(ws.n_tiles + blocks_for(ws.n_tiles, 256)),
                     dim3(256), 0, st, ws, 0,
                     many ? kSmallSort : 0x7fffffff, 0);
  if (many) {
    hipLaunchKernelGGL((k_sort_tiles<512, kMidSort / 512>), dim3(std::min(ws.n_tiles, 3072)), dim3(512),
                       0, st, ws, kSmallSort, kMidSort, 1);
    hipLaunchKernelGGL((k_sort_tiles<1024, kSortCap / 1024>), dim3(std::min(ws.n_tiles, 256)),
                       dim3(1024), 0, st, ws, kMidSort, 0x7fffffff, 2);
  }
  return hipGetLastError();
}

hipError_t launch_scan_records(const Ws &ws, hipStream_t st) {
  const int ng = (int)rec_scan_blocks(ws.n_rec);
  if (ng == 0) return launch_fill_u32(ws.rec_off, 0u, 1, st);
  const int per = (ng + 1023) / 1024;
  hipLaunchKernelGGL(k_scan_records, dim3(blocks_for(ng, per)), dim3(kNT), 0, st, ws, ng, per);
  return hipGetLastError();
}

int64_t rec_scan_blocks(int64_t n_rec) { return (n_rec + kRecGroup - 1) / kRecGroup; }

hipError_t launch_debug_copy(const Ws &ws, float *records, int32_t *rect, hipStream_t st) {
  if (ws.n_rec == 0) return hipSuccess;
  hipLaunchKernelGGL(k_debug_copy, dim3(blocks_for(ws.n_rec, kNT)), dim3(kNT), 0, st, ws,
                     records, rect);
  return hipGetLastError();
}

}  // namespace vtgs
