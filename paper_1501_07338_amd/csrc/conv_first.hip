// Forward pass of layers with at most four input channels (the networks' first layers), y = act(bias + W (*) x) on the
// matrix cores with the kernel matrix held in registers.
//
// Such a layer contracts over few entries (C R S <= 128) and writes many: in the slab kernels a block's stages - kernel
// matrix, halo tile, products, stores - follow one another for each 256 pixels, and the matrix cores wait through most of
// them.  Here a block stages the kernel matrix in LDS once, every wave takes all of it into registers (32 TM rows, lane
// l holds rows l % 32 and the contraction index 2 t + l / 32 of each step t), the input rows under the block's pixels are
// staged once, and the waves walk their tiles of 32 pixels of one sample with no barrier: a step reads one float per lane
// from the halo tile at lane_base(pixel) + offset(t) for TM matrix instructions, and a tile's stores leave while the next
// tile's products run.  64 1 64 64 -> 64 9 9: 61 -> 42 us (28 of them products: 18 of matrix instructions at two waves a SIMD,
// then the stores of 67 MB and the staging of a block); 128 1 28 28 -> 20 5 5: 12 -> 8 us.  Halo reads a further group
// ahead: no change; 1024 blocks: slower.
//
// The contraction runs over (channel, kernel row, column pairs).  Where the kernel has an odd number of columns the second half has
// no entry in the last pair, and the steps compiled beyond those in use have none at all: their pixels are put to zero by one
// select a step, with the lanes' mask in scalar registers, since a zero weight times an infinity would be NaN (64 1 64 64 -> 64 9 9
// 42 -> 40 us with it, fewer registers; 16 3 184 90 -> 31 5 7 35 -> 37, 128 1 28 28 -> 20 5 5 8.1 -> 8.8).  The sums begin with the bias,
// which measures 0.89 to 1.0 of the error of adding it last (14 layers, eight seeds each).
#include <algorithm>
#include <type_traits>

#include "common.h"
#include "elem.h"
#include "mma_core.h"

namespace vcnn {

static constexpr int kThreads = 256;
static constexpr int kMaxSteps = 64;

struct FirstArgs {
  const void* x;
  const void* wgt;
  const float* bias;
  void* y;
  int c, h, w, m, r, s, ph, pw, oh, ow, P, K;
  int nr, wp, s2, steps;          // halo rows and pitch per channel; kernel columns in pairs; steps that carry something
  int tiles_per_img, tiles_per_wave, blocks_per_img, groups;
  int relu;
  unsigned magic_wp, magic_nr, magic_s2;  // ceil(2^32 / .): division by multiply-high, exact below 2^16
  uint16_t offset[kMaxSteps];     // of step t inside the halo tile
  uint64_t first, second;         // bit t: the first, the second half of step t has an entry
};

template <int TM, int STEPS, typename T>
__global__ __launch_bounds__(kThreads) void conv_first_kernel(FirstArgs a) {
  constexpr int PITCH = 2 * STEPS + 1;  // odd: the 32 rows of a read on different banks
  extern __shared__ float first_lds[];
  float* const ws = first_lds;                              // [32 TM][PITCH]
  float* const halo = ws + ((32 * TM * PITCH + 3) & ~3);    // [c][nr][wp]
  float* const bias = halo + a.c * a.nr * a.wp;             // [32 TM] (an absent second half may read its first word)
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6, l32 = lane & 31, half = lane >> 5;
  const int group = blockIdx.x % a.groups, rest = blockIdx.x / a.groups;
  const int n = rest / a.blocks_per_img, share = rest - n * a.blocks_per_img;
  const int i0 = group * 32 * TM;
  const int t0 = share * 4 * a.tiles_per_wave;  // the block's first tile
  const int oh_first = t0 * 32 / a.ow;

  // kernel matrix: [row][(channel, kernel row)][column, padded to pairs], zero beyond; and input rows oh_first - ph + [0, nr),
  // columns -pw + [0, wp), zero outside the image.  Loads in batches: one round trip each, not one per element
  const T* const wgt = (const T*)a.wgt;
  const T* const x = (const T*)a.x + (int64_t)n * a.c * a.h * a.w;
  constexpr int WU = 32 * TM * 2 * STEPS / kThreads, WB = WU <= 12 ? WU : (WU % 12 == 0 ? 12 : 8), HU = 8;
  static_assert(WU % WB == 0, "a batch that ran over would write rows past the matrix into the halo tile");
  const int total = a.c * a.nr * a.wp;
  auto halo_batch = [&](int e0, float (&v)[HU], unsigned& inside) {
    inside = 0;
#pragma unroll
    for (int u = 0; u < HU; ++u) {
      const int e = e0 + u * kThreads, row = (int)__umulhi((unsigned)e, a.magic_wp), rx = e - row * a.wp;
      const int cl = (int)__umulhi((unsigned)row, a.magic_nr), ry = row - cl * a.nr;
      const int ih = oh_first - a.ph + ry, iw = rx - a.pw;
      const bool ok = e < total && (unsigned)ih < (unsigned)a.h && (unsigned)iw < (unsigned)a.w;
      v[u] = ld(x + (unsigned)(ok ? (cl * a.h + ih) * a.w + iw : 0));
      inside |= ok ? 1u << u : 0;
    }
  };
  auto halo_put = [&](int e0, const float (&v)[HU], unsigned inside) {
#pragma unroll
    for (int u = 0; u < HU; ++u)
      if (e0 + u * kThreads < total) halo[e0 + u * kThreads] = inside >> u & 1 ? v[u] : 0.f;
  };
  float hv[HU];
  unsigned inside;
  halo_batch(tid, hv, inside);
#pragma unroll
  for (int u0 = 0; u0 < WU; u0 += WB) {
    float v[WB];
    unsigned ok = 0;
#pragma unroll
    for (int u = 0; u < WB; ++u) {
      const int e = tid + (u0 + u) * kThreads, row = e / (2 * STEPS), k = e % (2 * STEPS);
      const int cr = (int)__umulhi((unsigned)k, a.magic_s2), s = k - cr * a.s2;
      const bool in = i0 + row < a.m && cr < a.c * a.r && s < a.s;
      v[u] = ld(wgt + (unsigned)(in ? (i0 + row) * a.K + cr * a.s + s : 0));
      ok |= in ? 1u << u : 0;
    }
#pragma unroll
    for (int u = 0; u < WB; ++u) {
      const int e = tid + (u0 + u) * kThreads;
      ws[e / (2 * STEPS) * PITCH + e % (2 * STEPS)] = ok >> u & 1 ? v[u] : 0.f;
    }
  }
  if (tid < 32 * TM) bias[tid] = a.bias && i0 + tid < a.m ? a.bias[i0 + tid] : 0.f;
  halo_put(tid, hv, inside);
  for (int e0 = tid + HU * kThreads; e0 < total; e0 += HU * kThreads) {
    halo_batch(e0, hv, inside);
    halo_put(e0, hv, inside);
  }
  __syncthreads();
  float wr[TM][STEPS];
#pragma unroll
  for (int mi = 0; mi < TM; ++mi)
#pragma unroll
    for (int t = 0; t < STEPS; ++t) wr[mi][t] = ws[(mi * 32 + l32) * PITCH + 2 * t + half];

  f32x16 start[TM];  // the sums begin with the bias
#pragma unroll
  for (int mi = 0; mi < TM; ++mi)
#pragma unroll
    for (int e = 0; e < 16; ++e) start[mi][e] = bias[mi * 32 + acc_row(e, lane)];

  T* const y = (T*)a.y + ((int64_t)n * a.m + i0) * a.P;
  const bool whole = i0 + 32 * TM <= a.m;
  for (int q = 0; q < a.tiles_per_wave; ++q) {
    const int tile = t0 + q * 4 + wave;
    if (tile >= a.tiles_per_img) break;
    const int p = tile * 32 + l32, pc = min(p, a.P - 1), oy = pc / a.ow;
    const int base = (oy - oh_first) * a.wp + (pc - oy * a.ow) + half;
    f32x16 acc[TM];
    int first[2] = {(int)a.first, (int)(a.first >> 32)}, second[2] = {(int)a.second, (int)(a.second >> 32)};
    asm volatile("" : "+s"(first[0]), "+s"(first[1]), "+s"(second[0]), "+s"(second[1]));  // (else every step's mask is kept, in registers that spill)
    auto present = [&](float v, int t) {  // 0 in the lanes without an entry
      const uint64_t lanes = (uint64_t)(unsigned)__builtin_amdgcn_sbfe(second[t >> 5], t & 31, 1) << 32 | (unsigned)__builtin_amdgcn_sbfe(first[t >> 5], t & 31, 1);
      return __builtin_amdgcn_inverse_ballot_w64(lanes) ? v : 0.f;
    };
    // (eight steps' values requested while the eight before are multiplied)
    float b[2][8];
    auto request = [&](int t0, float (&v)[8]) {
#pragma unroll
      for (int u = 0; u < 8; ++u) v[u] = halo[base + a.offset[t0 + u]];
    };
    request(0, b[0]);
#pragma unroll
    for (int t = 0; t < STEPS; t += 8) {
      if (t + 8 < STEPS) request(t + 8, b[(t / 8 + 1) & 1]);
      __builtin_amdgcn_sched_barrier(0);
#pragma unroll
      for (int u = 0; u < 8; ++u)
#pragma unroll
        for (int mi = 0; mi < TM; ++mi) acc[mi] = __builtin_amdgcn_mfma_f32_32x32x2f32(wr[mi][t + u], present(b[(t / 8) & 1][u], t + u), t + u == 0 ? start[mi] : acc[mi], 0, 0, 0);
      __builtin_amdgcn_sched_barrier(0);
    }
    if (p >= a.P) continue;
    const unsigned at = 4 * half * a.P + p;  // of row 0 of the lane's half
    // (a mask and a branch for every value took as long as a sixth of the products)
    auto put = [&](auto masked, auto relu) {
#pragma unroll
      for (int mi = 0; mi < TM; ++mi)
#pragma unroll
        for (int e = 0; e < 16; ++e) {
          const int i = mi * 32 + acc_row(e, 0);
          if (decltype(masked)::value && i0 + i + 4 * half >= a.m) continue;
          st(y + (int64_t)i * a.P + at, decltype(relu)::value ? fmaxf(acc[mi][e], 0.f) : acc[mi][e]);
        }
    };
    if (whole && a.relu) put(std::false_type{}, std::true_type{});
    else if (whole) put(std::false_type{}, std::false_type{});
    else if (a.relu) put(std::true_type{}, std::true_type{});
    else put(std::true_type{}, std::false_type{});
  }
}

bool conv_first_plan(const ConvGeom& g, FirstPlan* p) {
  if (g.c > 4 || (int64_t)g.c * g.h * g.w > 0x7fffffffLL || g.P > (1 << 26)) return false;
  const int s2 = (g.s + 1) / 2 * 2, steps = g.c * g.r * s2 / 2;
  p->tm = g.k <= 32 ? 1 : 2;
  if (steps > (p->tm == 2 ? 48 : kMaxSteps)) return false;
  // with few tiles, 32 rows a wave and twice the waves: a wave's chain of products is half as long
  if ((int64_t)g.n * ceil_div(g.P, 32) * ceil_div(g.k, 32) <= 1024) p->tm = 1;
  p->steps = steps <= 16 ? 16 : (steps <= 32 ? 32 : (steps <= 48 ? 48 : 64));
  p->groups = (int)ceil_div(g.k, 32 * p->tm);
  p->tiles_per_img = (int)ceil_div(g.P, 32);
  const int64_t tiles = (int64_t)g.n * p->tiles_per_img * p->groups;
  if (tiles > 0x7fffffffLL) return false;
  // two blocks for each of 256 CUs where there is that much to do: what a block stages serves several tiles of each wave
  p->tiles_per_wave = (int)std::min<int64_t>(ceil_div(tiles, 4 * 512), 16);
  p->blocks_per_img = (int)ceil_div(p->tiles_per_img, 4 * p->tiles_per_wave);
  p->tiles_per_wave = (int)ceil_div(p->tiles_per_img, 4 * p->blocks_per_img);  // (an image's blocks alike)
  const int pixels = 128 * p->tiles_per_wave;
  p->nr = std::min(g.oh, (pixels + g.ow - 2) / g.ow + 1) + g.r - 1, p->wp = g.w + 2 * g.pw;
  const int64_t halo = (int64_t)g.c * p->nr * p->wp;
  if (halo > 0xffff || p->wp < 2 || p->nr < 2) return false;  // (offsets of 16 bits; divisors for which multiply-high is exact)
  p->lds_bytes = 4 * ((size_t)((32 * p->tm * (2 * p->steps + 1) + 3) & ~3) + 32 * p->tm + (size_t)halo);
  return p->lds_bytes <= 64 * 1024;
}

template <int TM, int STEPS, typename T>
static void launch_one(const FirstArgs& a, const FirstPlan& p, int n, hipStream_t st) {
  hipLaunchKernelGGL((conv_first_kernel<TM, STEPS, T>), dim3((unsigned)((int64_t)n * p.blocks_per_img * p.groups)), dim3(kThreads), p.lds_bytes, st, a);
}
template <typename T>
static void launch_typed(const FirstArgs& a, const FirstPlan& p, int n, hipStream_t st) {
  if (p.tm == 2) {
    if (p.steps == 16) launch_one<2, 16, T>(a, p, n, st);
    else if (p.steps == 32) launch_one<2, 32, T>(a, p, n, st);
    else launch_one<2, 48, T>(a, p, n, st);
  } else {
    if (p.steps == 16) launch_one<1, 16, T>(a, p, n, st);
    else if (p.steps == 32) launch_one<1, 32, T>(a, p, n, st);
    else if (p.steps == 48) launch_one<1, 48, T>(a, p, n, st);
    else launch_one<1, 64, T>(a, p, n, st);
  }
}

vcnn_status launch_conv_first(const FirstPlan& p, int dtype, const ConvGeom& g, const void* x, const void* w, const float* bias, void* y,
                              int relu, hipStream_t st) {
  FirstArgs a{};
  a.x = x, a.wgt = w, a.bias = bias, a.y = y;
  a.c = g.c, a.h = g.h, a.w = g.w, a.m = g.k, a.r = g.r, a.s = g.s, a.ph = g.ph, a.pw = g.pw, a.oh = g.oh, a.ow = g.ow;
  a.P = (int)g.P, a.K = (int)g.K;
  a.nr = p.nr, a.wp = p.wp, a.s2 = (g.s + 1) / 2 * 2, a.steps = g.c * g.r * a.s2 / 2;
  a.tiles_per_img = p.tiles_per_img, a.tiles_per_wave = p.tiles_per_wave, a.blocks_per_img = p.blocks_per_img, a.groups = p.groups;
  a.relu = relu;
  auto magic = [](int v) { return (unsigned)(((1ULL << 32) + v - 1) / v); };
  a.magic_wp = magic(p.wp), a.magic_nr = magic(p.nr), a.magic_s2 = magic(a.s2);
  for (int t = 0; t < a.steps; ++t) {
    const int cr = 2 * t / a.s2, s = 2 * t % a.s2;
    a.offset[t] = (uint16_t)((cr / g.r * p.nr + cr % g.r) * p.wp + s);
    a.first |= 1ULL << t, a.second |= (uint64_t)(s + 1 < g.s) << t;
  }
  if (dtype == VCNN_BF16) launch_typed<bf16>(a, p, g.n, st);
  else launch_typed<float>(a, p, g.n, st);
  return check_launch("conv_first");
}

}  // namespace vcnn
