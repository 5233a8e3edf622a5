// Keyframe ingestion: a view-tied Gaussian at every valid depth pixel of the
// stride grid (Sec. 3.2), radius initialised to stride * depth / focal
// length (App. A); the complement mask of pixels the current Gaussians leave
// uncovered (Sec. 3.4).  Stream compaction in row-major order: per-block counts,
// a single-block scan of the block counts, then an order-preserving fill.
#include "vtgs_internal.h"

namespace vtgs {

namespace {
constexpr int kNT = 256;
constexpr int kPer = 4;                 // grid cells per thread
constexpr int kCells = kNT * kPer;      // grid cells per block

// A wave's kPer x 64 consecutive cells, 64 at a time, so that its loads and
// the stores of its Gaussians lie next to each other: for a frame of 1200x680
// at stride 1 a thread with kPer cells of its own (and a 64-bit division each)
// took 23 us for the fill and 4.4 for the counts, this takes 9.6 and 3.9 (the
// fill moves 36 MB, 7.6 us).
struct Cells {
  uint32_t gx, gy, rows, cols;  // (rows, cols: 64 cells on, in a grid of nx columns)
  int64_t c;
  __device__ __forceinline__ Cells(int64_t first, int nx) : c(first + lane_id()) {
    // (an image has fewer than 2^31 pixels)
    gy = (uint32_t)c / (uint32_t)nx;
    gx = (uint32_t)c - gy * (uint32_t)nx;
    rows = (uint32_t)kWave / (uint32_t)nx;
    cols = (uint32_t)kWave - rows * (uint32_t)nx;
  }
  // (row by row, an image of one column took 15.3 us for the fill, this 5.3)
  __device__ __forceinline__ void next(int nx) {
    c += kWave;
    gx += cols;
    gy += rows;
    const bool over = gx >= (uint32_t)nx;
    gx -= over ? (uint32_t)nx : 0u;
    gy += over ? 1u : 0u;
  }
  __device__ __forceinline__ int64_t pixel(int W, int s) const {
    return (int64_t)((int)gy * s) * W + (int)gx * s;
  }
};

__device__ __forceinline__ bool valid_depth(float d) { return d > 0.f && d <= 3.402823466e38f; }

__device__ __forceinline__ int64_t first_cell() {
  return (int64_t)blockIdx.x * kCells + (threadIdx.x / kWave) * (kPer * kWave);
}

__global__ __launch_bounds__(kNT) void k_ingest_counts(const float *depth, const uint8_t *mask,
                                                       int H, int W, int s, int nx, int64_t M,
                                                       uint32_t *block_counts) {
  __shared__ uint32_t wave_n[kNT / kWave];
  uint32_t n = 0;
  Cells q(first_cell(), nx);
#pragma unroll
  for (int k = 0; k < kPer; k++) {
    const int64_t p = q.pixel(W, s);
    const bool ok = q.c < M && valid_depth(depth[p]) && (!mask || mask[p] != 0);
    n += (uint32_t)__popcll(ballot64(ok));
    q.next(nx);
  }
  if (lane_id() == 0) wave_n[threadIdx.x / kWave] = n;
  __syncthreads();
  if (threadIdx.x == 0) {
    uint32_t tot = 0;
    for (int w = 0; w < kNT / kWave; w++) tot += wave_n[w];
    block_counts[blockIdx.x] = tot;
  }
}

// One block: exclusive scan of the block counts, total to *count.
__global__ __launch_bounds__(1024) void k_ingest_scan(const uint32_t *block_counts, int nb,
                                                      uint32_t *block_off, int32_t *count) {
  __shared__ uint32_t lw[1024 / kWave];
  uint32_t carry = 0;
  for (int base = 0; base < nb; base += 1024) {
    const int i = base + threadIdx.x;
    const uint32_t v = i < nb ? block_counts[i] : 0u;
    uint32_t tot;
    const uint32_t ex = block_exclusive_scan<1024>(v, lw, &tot);
    if (i < nb) block_off[i] = carry + ex;
    carry += tot;
  }
  if (threadIdx.x == 0) *count = (int32_t)carry;
}

__global__ __launch_bounds__(kNT) void k_ingest_fill(const float *depth, const float *rgb,
                                                     const uint8_t *mask, int H, int W, int s,
                                                     int nx, int64_t M, float fx, float o_init,
                                                     const uint32_t *block_off, int n,
                                                     uint32_t *pix, float *dep, float *col,
                                                     float *opa, float *rad) {
  __shared__ uint32_t wave_n[kNT / kWave];
  unsigned long long ok[kPer];
  float d[kPer];
  uint32_t cnt = 0;
  const int w = threadIdx.x / kWave;
  Cells q(first_cell(), nx);
#pragma unroll
  for (int k = 0; k < kPer; k++) {
    const int64_t p = q.pixel(W, s);
    d[k] = q.c < M ? depth[p] : 0.f;
    ok[k] = ballot64(valid_depth(d[k]) && (!mask || mask[p] != 0));
    cnt += (uint32_t)__popcll(ok[k]);
    q.next(nx);
  }
  if (lane_id() == 0) wave_n[w] = cnt;
  __syncthreads();
  uint32_t i0 = block_off[blockIdx.x];
  for (int ww = 0; ww < w; ww++) i0 += wave_n[ww];
  const int64_t P = (int64_t)H * W;
  q = Cells(first_cell(), nx);
#pragma unroll
  for (int k = 0; k < kPer; k++) {
    const uint32_t i = i0 + (uint32_t)__popcll(ok[k] & lanemask_lt());
    if ((ok[k] >> lane_id() & 1ull) && (int)i < n) {
      const int64_t p = q.pixel(W, s);
      pix[i] = (uint32_t)p;
      dep[i] = d[k];
      if (rgb)
        for (int c = 0; c < 3; c++) col[(int64_t)c * n + i] = rgb[c * P + p];
      opa[i] = o_init;
      rad[i] = __fdiv_rn((float)s * d[k], fx);
    }
    i0 += (uint32_t)__popcll(ok[k]);
    q.next(nx);
  }
}

inline void grid_dims(int H, int W, int s, int *nx, int64_t *M, int *nb) {
  *nx = (W + s - 1) / s;
  const int ny = (H + s - 1) / s;
  *M = (int64_t)*nx * ny;
  *nb = (int)((*M + kCells - 1) / kCells);
}

// Complement initialisation (Sec. 3.4): a pixel is left uncovered by the
// current Gaussians when the silhouette of their rendering there is below
// thr, and gets a new Gaussian if its depth is valid.
__global__ __launch_bounds__(kNT) void k_uncovered(const float *sil, const float *depth, int64_t n,
                                                   float thr, uint8_t *mask) {
  const int64_t i = (int64_t)blockIdx.x * kNT + threadIdx.x;
  if (i >= n) return;
  const float d = depth[i];
  mask[i] = (uint8_t)(sil[i] < thr && d > 0.f && d <= 3.402823466e38f);
}
}  // namespace

hipError_t launch_uncovered(const float *sil, const float *depth, int64_t n, float thr,
                            uint8_t *mask, hipStream_t st) {
  if (n <= 0) return hipSuccess;
  hipLaunchKernelGGL(k_uncovered, dim3((unsigned)((n + kNT - 1) / kNT)), dim3(kNT), 0, st, sil,
                     depth, n, thr, mask);
  return hipGetLastError();
}

int64_t ingest_scratch_words(int H, int W, int s) {
  int nx, nb;
  int64_t M;
  grid_dims(H, W, s, &nx, &M, &nb);
  return 2 * (int64_t)nb + 2;
}

hipError_t launch_ingest_count(const float *depth, const uint8_t *mask, int H, int W, int s,
                               uint32_t *scratch, int32_t *count, hipStream_t st) {
  int nx, nb;
  int64_t M;
  grid_dims(H, W, s, &nx, &M, &nb);
  if (nb == 0) return hipSuccess;
  hipLaunchKernelGGL(k_ingest_counts, dim3(nb), dim3(kNT), 0, st, depth, mask, H, W, s, nx, M,
                     scratch);
  hipLaunchKernelGGL(k_ingest_scan, dim3(1), dim3(1024), 0, st, scratch, nb, scratch + nb, count);
  return hipGetLastError();
}

hipError_t launch_ingest_fill(const float *depth, const float *rgb, const uint8_t *mask, int H,
                              int W, int s, float fx, float o_init, const uint32_t *scratch,
                              int n, uint32_t *pix, float *dep, float *col, float *opa,
                              float *rad, hipStream_t st) {
  int nx, nb;
  int64_t M;
  grid_dims(H, W, s, &nx, &M, &nb);
  if (nb == 0) return hipSuccess;
  hipLaunchKernelGGL(k_ingest_fill, dim3(nb), dim3(kNT), 0, st, depth, rgb, mask, H, W, s, nx, M,
                     fx, o_init, scratch + nb, n, pix, dep, col, opa, rad);
  return hipGetLastError();
}

}  // namespace vtgs
