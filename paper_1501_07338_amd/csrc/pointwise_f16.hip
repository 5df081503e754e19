// Unpadded 1 x 1 layers in float as three dense products on the half-precision matrix cores (two f16 terms per operand,
// split_f16.h), both operands re-laid into fragment order first:
//     forward          y[n][m][p]  = sum_c w[m][c] * x[n][c][p]              (+ bias, sigma)
//     input gradient   dx[n][c][p] = sum_m w[m][c] * dy[n][m][p]
//     kernel gradient  dw[m][c]    = sum_n sum_p dy[n][m][p] * x[n][c][p]
// The float kernels ran at 60 % of the float matrix rate (16 512 49 49 -> 512, the three passes 0.66 ms); here that layer
// takes 0.47 ms: 87, 87 and 71 us of products, 50 us of a pass the scan and re-laying of the activations (bandwidth), 4.5 us
// a pass the float kernel behind the product, which leaves at once (split_f16.h).
#include <algorithm>

#include "common.h"
#include "elem.h"
#include "frag_product.h"

namespace vcnn {

static constexpr int kThreads = 256;
static constexpr int kXcds = 8;
static constexpr int kSteps = FragSlab<2>::STEPS;

struct PointwiseF16Args {
  const uint4* a;  // rows of the result: [n or 1][4 tiles_i][steps][64]
  const uint4* b;  // columns: [n][4 tiles_j][steps][64]
  int64_t a_term, b_term;
  const int32_t* image_exponent;  // the scales of the activations' images (kernel gradient: of all of them) ...
  const int32_t* exponent;        // ... and of the other operand
  Declined declined;              // images left to the float kernel
  const float* bias;
  float* y;        // [n][rows][P], or slices [splits][rows][cols]
  int n, rows, cols, tiles_i, tiles_j, steps;
  int total_slabs, slabs_per_split;  // kernel gradient
  int relu;
};

// Work item of a block: consecutive blocks go to the eight XCDs in turn; each XCD takes a contiguous eighth of the items, so
// that the row tiles of one column tile, which read the same activations, share an L2.
__device__ __forceinline__ int xcd_item(int block, int total) {
  const int per = total / kXcds;
  return block < per * kXcds ? (block % kXcds) * per + block / kXcds : block;
}

__global__ __launch_bounds__(kThreads, 2) void pointwise_f16_kernel(PointwiseF16Args a) {
  extern __shared__ uint4 smem16[];
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const int item = xcd_item(blockIdx.x, gridDim.x);
  const int it = item % a.tiles_i, tj = item / a.tiles_i;  // tj = (sample, column tile)
  const int n = tj / a.tiles_j, jt = tj - n * a.tiles_j;
  if (is_declined(a.declined, n)) return;
  const uint4* const src_a = a.a + (int64_t)(4 * it + wave) * a.steps * 64 + lane;
  const uint4* const src_b = a.b + ((int64_t)4 * tj + wave) * a.steps * 64 + lane;
  f32x16 acc[2][2];
  frag_product<2>(a.steps / kSteps, smem16, a.a_term, a.b_term, [&](int sl) { return src_a + sl * (kSteps * 64); },
                  [&](int sl) { return src_b + sl * (kSteps * 64); }, acc);
  const int descale = -(a.image_exponent[n] + *a.exponent);
  const int i0 = it * kFragTile + (wave & 1) * 64, j0 = jt * kFragTile + (wave >> 1) * 64;
  float* const yn = a.y + (int64_t)n * a.rows * a.cols;
#pragma unroll
  for (int ni = 0; ni < 2; ++ni) {
    const int p = j0 + ni * 32 + (lane & 31);
    if (p >= a.cols) continue;
#pragma unroll
    for (int mi = 0; mi < 2; ++mi)
#pragma unroll
      for (int q = 0; q < 16; ++q) {
        const int i = i0 + mi * 32 + acc_row(q, lane);
        if (i < a.rows) {
          float v = ldexpf(acc[mi][ni][q], descale);
          if (a.bias) v += a.bias[i];
          if (a.relu) v = fmaxf(v, 0.f);
          yn[(int64_t)i * a.cols + p] = v;
        }
      }
  }
}

// (blockIdx.y: the split, a run of slabs across the samples)
__global__ __launch_bounds__(kThreads, 2) void pointwise_f16_filter_kernel(PointwiseF16Args a) {
  if (!leave_all(a.declined)) return;
  extern __shared__ uint4 smem16[];
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const int it = blockIdx.x % a.tiles_i, jt = blockIdx.x / a.tiles_i;
  const int s0 = blockIdx.y * a.slabs_per_split, s1 = min(a.total_slabs, s0 + a.slabs_per_split);
  const int per_img = a.steps / kSteps;
  f32x16 acc[2][2];
  frag_product<2>(s1 - s0, smem16, a.a_term, a.b_term,
                  [&](int sl) {
                    const int n = (s0 + sl) / per_img, s = (s0 + sl) - n * per_img;
                    return a.a + (((int64_t)n * a.tiles_i + it) * 4 + wave) * a.steps * 64 + s * (kSteps * 64) + lane;
                  },
                  [&](int sl) {
                    const int n = (s0 + sl) / per_img, s = (s0 + sl) - n * per_img;
                    return a.b + (((int64_t)n * a.tiles_j + jt) * 4 + wave) * a.steps * 64 + s * (kSteps * 64) + lane;
                  },
                  acc);
  const int descale = -(*a.image_exponent + *a.exponent);
  const int i0 = it * kFragTile + (wave & 1) * 64, j0 = jt * kFragTile + (wave >> 1) * 64;
  float* const out = a.y + (int64_t)blockIdx.y * a.rows * a.cols;
#pragma unroll
  for (int ni = 0; ni < 2; ++ni) {
    const int j = j0 + ni * 32 + (lane & 31);
    if (j >= a.cols) continue;
#pragma unroll
    for (int mi = 0; mi < 2; ++mi)
#pragma unroll
      for (int q = 0; q < 16; ++q) {
        const int i = i0 + mi * 32 + acc_row(q, lane);
        if (i < a.rows) out[(int64_t)i * a.cols + j] = ldexpf(acc[mi][ni][q], descale);
      }
  }
}

static inline size_t align256(size_t b) { return (b + 255) & ~(size_t)255; }
static int whole_steps(int64_t depth) { return (int)(ceil_div(ceil_div(depth, 16), kSteps) * kSteps); }

bool pointwise_f16_plan(const ConvGeom& g, int pass, PointwiseF16Plan* p) {
  const bool filter = pass == VCNN_PASS_BWD_FILTER;
  const int64_t rows = pass == VCNN_PASS_BWD_DATA ? g.c : g.k, cols = filter ? g.c : g.P;
  const int64_t depth = filter ? g.P : (pass == VCNN_PASS_FWD ? g.c : g.k);
  p->tiles_i = (int)ceil_div(rows, kFragTile), p->tiles_j = (int)ceil_div(cols, kFragTile);
  p->steps = whole_steps(depth);
  if (4 * (int64_t)std::max(p->tiles_i, p->tiles_j) > 65535 || g.n > 65535 || g.P > (1 << 24)) return false;  // grid dimensions
  const size_t frag = (size_t)p->steps * 64 * 16;
  const int64_t tiles = (int64_t)p->tiles_i * p->tiles_j * (filter ? 1 : g.n);
  if (tiles > 0x7fffffffLL) return false;
  p->a_bytes = align256((filter ? (size_t)g.n : 1) * 4 * p->tiles_i * frag);
  p->b_bytes = align256((size_t)g.n * 4 * p->tiles_j * frag);
  const int64_t slabs = (int64_t)g.n * (p->steps / kSteps);
  if (slabs > 0x7fffffffLL) return false;
  p->splits = 1, p->slabs_per_split = (int)slabs, p->partial_bytes = 0;
  double blocks = (double)tiles, steps = p->steps;
  if (filter) {
    const int64_t want = std::min<int64_t>(std::max<int64_t>(ceil_div(512, tiles), 1), ceil_div(slabs, 4));
    p->slabs_per_split = (int)ceil_div(slabs, want);
    p->splits = (int)ceil_div(slabs, p->slabs_per_split);
    if (p->splits > 65535) return false;
    if (p->splits > 1) p->partial_bytes = align256((size_t)p->splits * g.M * g.K * sizeof(float));
    blocks = (double)tiles * p->splits, steps = (double)p->slabs_per_split * kSteps;
  }
  p->workspace_bytes = (filter ? 0 : split_scales_bytes(g.n)) + 2 * (p->a_bytes + p->b_bytes) + p->partial_bytes;
  // products at half the nominal rate on the busiest CU; the scan, the re-laying and the slices at 4.5 TB/s
  const double floats = 4.0 * (filter ? (double)g.M * g.N + (double)g.K * g.N : (double)g.M * g.K + (double)depth * g.N);
  p->est_seconds = std::max(std::ceil(blocks / 256.0), 1.5) * (steps * 12 * 32 * 1.9 / 2.4e9 + 1.5e-6) +
                   (2 * floats + 2.0 * (double)(p->a_bytes + p->b_bytes) + 2.0 * (double)p->partial_bytes) / 4.5e12 + 12e-6;
  return true;
}

vcnn_status launch_pointwise_f16(const PointwiseF16Plan& p, const ConvGeom& g, int pass, const float* w, const float* x,
                                 const float* bias, float* y, int relu, void* workspace, hipStream_t st) {
  const bool fwd = pass == VCNN_PASS_FWD;
  const int rows = fwd ? g.k : g.c, depth = fwd ? g.c : g.k, P = (int)g.P;
  const int64_t dp = (int64_t)depth * P;
  const SplitScales sc = split_scales(workspace, g.n, g.n, dp, g.M * g.K);
  char* const fa = (char*)workspace + split_scales_bytes(g.n);
  char* const fb = fa + 2 * p.a_bytes;
  PointwiseF16Args a{};
  a.a = (const uint4*)fa, a.b = (const uint4*)fb, a.a_term = (int64_t)(p.a_bytes / 16), a.b_term = (int64_t)(p.b_bytes / 16);
  a.image_exponent = sc.exponent[0], a.exponent = sc.exponent[1], a.declined = sc.declined();
  a.bias = bias, a.y = y, a.relu = relu;
  a.n = g.n, a.rows = rows, a.cols = P, a.tiles_i = p.tiles_i, a.tiles_j = p.tiles_j, a.steps = p.steps;
  if (vcnn_status e = launch_absmax(x, g.n, dp, w, g.M * g.K, sc, true, st)) return e;
  // w is [k][c]: its rows (forward) or its columns (input gradient) are the rows of the result
  if (vcnn_status e = launch_fragments({w, fa, a.a_term, rows, depth, fwd ? g.c : 1, fwd ? 1 : g.c, 0, 4 * p.tiles_i, 1, p.steps, 2, 1, 0}, sc, st)) return e;
  if (vcnn_status e = launch_fragments({x, fb, a.b_term, P, depth, 1, P, dp, 4 * p.tiles_j, g.n, p.steps, 2, 0, 1}, sc, st)) return e;
  (void)hipFuncSetAttribute(reinterpret_cast<const void*>(pointwise_f16_kernel), hipFuncAttributeMaxDynamicSharedMemorySize, (int)FragSlab<2>::LDS_BYTES);
  hipLaunchKernelGGL(pointwise_f16_kernel, dim3((unsigned)((int64_t)g.n * p.tiles_i * p.tiles_j)), dim3(kThreads), FragSlab<2>::LDS_BYTES, st, a);
  return check_launch("pointwise_f16");
}

vcnn_status launch_pointwise_f16_filter(const PointwiseF16Plan& p, const ConvGeom& g, const float* x, const float* dy, float* dw,
                                        void* workspace, void* scales, const FilterBehind& behind, hipStream_t st) {
  const int P = (int)g.P;
  const SplitScales sc = split_scales(scales, 1, 1, g.K * g.N, g.M * g.N);
  char* const fa = (char*)workspace;
  char* const fb = fa + 2 * p.a_bytes;
  float* const partial = (float*)(fb + 2 * p.b_bytes);
  PointwiseF16Args a{};
  a.a = (const uint4*)fa, a.b = (const uint4*)fb, a.a_term = (int64_t)(p.a_bytes / 16), a.b_term = (int64_t)(p.b_bytes / 16);
  a.image_exponent = sc.exponent[0], a.exponent = sc.exponent[1], a.declined = sc.declined();
  a.y = p.splits > 1 ? partial : dw;
  a.n = g.n, a.rows = (int)g.M, a.cols = (int)g.K, a.tiles_i = p.tiles_i, a.tiles_j = p.tiles_j, a.steps = p.steps;
  a.total_slabs = g.n * (p.steps / kSteps), a.slabs_per_split = p.slabs_per_split;
  if (vcnn_status e = launch_absmax(x, 1, g.K * g.N, dy, g.M * g.N, sc, true, st)) return e;
  if (vcnn_status e = launch_fragments({dy, fa, a.a_term, (int)g.M, P, P, 1, g.M * P, 4 * p.tiles_i, g.n, p.steps, 2, 1, 0}, sc, st)) return e;
  if (vcnn_status e = launch_fragments({x, fb, a.b_term, (int)g.K, P, P, 1, g.K * P, 4 * p.tiles_j, g.n, p.steps, 2, 0, 0}, sc, st)) return e;
  (void)hipFuncSetAttribute(reinterpret_cast<const void*>(pointwise_f16_filter_kernel), hipFuncAttributeMaxDynamicSharedMemorySize, (int)FragSlab<2>::LDS_BYTES);
  hipLaunchKernelGGL(pointwise_f16_filter_kernel, dim3((unsigned)(p.tiles_i * p.tiles_j), (unsigned)p.splits), dim3(kThreads), FragSlab<2>::LDS_BYTES, st, a);
  if (vcnn_status e = check_launch("pointwise_f16_filter")) return e;
  OtherSlices other{};
  if (vcnn_status e = launch_filter_behind(behind, dw, sc.declined(), st, &other)) return e;
  if (p.splits == 1 && other.splits == 0) return VCNN_OK;
  return launch_sum_slices(partial, nullptr, dw, VCNN_F32, g.M * g.K, p.splits > 1 ? p.splits : 0, 1, 1, 0, st, other);
}

}  // namespace vcnn
