// The float products of large layers on the half-precision matrix cores: which layers, the scales of the operands, and
// the workspace.  The terms and their precision are described in split_f16.h; the kernels that multiply them are the
// matrix-core kernels of the bfloat16 variant with two f16 terms per operand.
#include <algorithm>

#include "common.h"
#include "split_f16.h"

namespace vcnn {

static constexpr int kThreads = 256;

struct AbsMaxArgs {
  const float* src[2];
  int64_t count[2];  // floats per image, floats
  int image_blocks;  // blocks of operand 0; operand 1's follow
  int first;
  SplitScales sc;
};

// Largest magnitude (infinities and NaN above every finite one) of each block's share of the two operands, an image of
// the first at a time; the first block of a scale clears its counter and its word.  Bandwidth: read once, 16 bytes per
// load and four loads in flight per thread.
// BEHIND: behind another pass (a.sc.only).  (With the test in all of these kernels in place of an instance of their own, ordinary
// calls took 2 % longer: 64 64 64 64 -> 32 5 5 three passes 479 -> 490 us.)
template <bool BEHIND>
__global__ __launch_bounds__(kThreads) void absmax_kernel(AbsMaxArgs a) {
  const int op = (int)blockIdx.x >= a.image_blocks;
  const int image = op ? 0 : (int)blockIdx.x / a.sc.blocks;
  const int blocks = op ? kAbsMaxBlocks : a.sc.blocks;
  const int block = op ? (int)blockIdx.x - a.image_blocks : (int)blockIdx.x - image * a.sc.blocks;
  const int64_t count = a.count[op];
  const float* const p = a.src[op] + image * count;
  if (block == 0 && threadIdx.x == 0) {
    if (op == 0 && image == 0 && a.first) *a.sc.any = BEHIND && (a.sc.only.of || looks_at_none(a.sc.only)) ? kNotLookedAt : 0;
    a.sc.small[op][image] = 0;
    if (op) *a.sc.all = 0;
    else a.sc.image[image] = BEHIND && !looks_at(a.sc.only, image) ? kNotLookedAt : 0;
  }
  if (BEHIND && (op ? looks_at_none(a.sc.only) : !looks_at(a.sc.only, image))) return;
  const int head = (int)min((int64_t)((16 - ((uintptr_t)p & 15)) & 15) / 4, count);  // floats before a 16-byte boundary
  const uint4* const body = reinterpret_cast<const uint4*>(p + head);
  const int64_t quads = (count - head) / 4;
  uint32_t m = 0;
  auto take = [&](uint32_t bits) { m = max(m, bits & 0x7fffffffu); };
  const int64_t step = (int64_t)blocks * kThreads;
  int64_t i = (int64_t)block * kThreads + threadIdx.x;
  for (; i + 3 * step < quads; i += 4 * step) {
    uint4 v[4];
#pragma unroll
    for (int k = 0; k < 4; ++k) v[k] = body[i + k * step];
#pragma unroll
    for (int k = 0; k < 4; ++k) take(v[k].x), take(v[k].y), take(v[k].z), take(v[k].w);
  }
  for (; i < quads; i += step) {
    const uint4 v = body[i];
    take(v.x), take(v.y), take(v.z), take(v.w);
  }
  if (block == 0 && threadIdx.x < 8) {  // the floats around the 16-byte words
    const int64_t e = threadIdx.x < 4 ? (int64_t)threadIdx.x : head + quads * 4 + (threadIdx.x - 4);
    if (threadIdx.x < 4 ? e < head : e < count) take(__float_as_uint(p[e]));
  }
#pragma unroll
  for (int d = 32; d > 0; d >>= 1) m = max(m, (uint32_t)__shfl_xor((int)m, d));
  __shared__ uint32_t wave_max[4];
  if ((threadIdx.x & 63) == 0) wave_max[threadIdx.x >> 6] = m;
  __syncthreads();
  if (threadIdx.x == 0)
    a.sc.partial[op][op ? block : (int)blockIdx.x] = max(max(wave_max[0], wave_max[1]), max(wave_max[2], wave_max[3]));
}

vcnn_status launch_absmax(const float* a, int images, int64_t per_image, const float* b, int64_t nb, const SplitScales& sc,
                          bool first, hipStream_t st) {
  AbsMaxArgs args{{a, b}, {per_image, nb}, images * sc.blocks, first, sc};
  const dim3 grid((unsigned)(args.image_blocks + (nb ? kAbsMaxBlocks : 0)));
  if (sc.only.of_any) hipLaunchKernelGGL(absmax_kernel<true>, grid, dim3(kThreads), 0, st, args);
  else hipLaunchKernelGGL(absmax_kernel<false>, grid, dim3(kThreads), 0, st, args);
  return check_launch("absmax");
}

static inline size_t align256(size_t b) { return (b + 255) & ~(size_t)255; }

// Blocks that scan one of `images` images (whatever part of the batch they are, images x blocks <= images + kAbsMaxBlocks).
static int scan_blocks(int images) { return std::max(1, kAbsMaxBlocks / images); }

size_t split_scales_bytes(int images) {
  const size_t partial = (size_t)images + 2 * kAbsMaxBlocks, per_image = 3 * (size_t)images, others = 4;
  return align256((partial + per_image + others) * sizeof(uint32_t));
}

SplitScales split_scales(void* workspace, int images, int images_at_once, int64_t per_image, int64_t others, const Declined& only) {
  uint32_t* w = (uint32_t*)workspace;
  auto take = [&](size_t words) { uint32_t* const at = w; w += words; return at; };
  SplitScales sc{};
  sc.any = take(1), sc.all = take(1);
  sc.exponent[1] = (int32_t*)take(1), sc.small[1] = take(1);
  sc.exponent[0] = (int32_t*)take(images), sc.small[0] = take(images), sc.image = take(images);
  sc.partial[1] = take(kAbsMaxBlocks), sc.partial[0] = take((size_t)images + kAbsMaxBlocks);
  sc.blocks = scan_blocks(images_at_once);
  sc.only = only;
  // (at most half of a block's elements: a block of small ones then says so by itself, see note_small)
  auto limit = [](int64_t count) { return (uint32_t)std::min<int64_t>(count >> 13, 1024); };
  sc.limit[0] = limit(per_image), sc.limit[1] = limit(others);
  return sc;
}

Declined split_declined(const void* workspace, int images, const Declined& only) {
  return split_scales(const_cast<void*>(workspace), images, images, 0, 0, only).declined();
}

vcnn_status launch_filter_behind(const FilterBehind& b, float* dw, const Declined& only, hipStream_t st, OtherSlices* other) {
  other->declined = only.any, other->partial = b.workspace, other->of_any = only.of_any;
  if (b.halo) {
    other->splits = b.halo->splits > 1 ? b.halo->splits : 0;
    return launch_conv_halo_filter(*b.halo, VCNN_F32, *b.g, b.x, b.dy, dw, nullptr, b.workspace, st, only);
  }
  const int splits = bwd_filter_splits(*b.g);
  other->splits = splits > 1 ? splits : 0;
  return launch_bwd_filter_gemm_f32(*b.g, VCNN_F32, b.dy, nullptr, b.x, dw, b.workspace, st, only);
}

// The scales read both operands, the re-laying passes read them again and write the terms: at some 3.5 TB/s, and three
// launches.
static double relay_seconds(double float_bytes, double term_bytes) { return (2 * float_bytes + term_bytes) / 3.5e12 + 10e-6; }

// The plan for one part of n images.
static bool part_plan(const ConvGeom& whole, int pass, int n, int max_splits, F16x2Plan* p) {
  ConvGeom g = whole;
  g.n = n, g.N = (int64_t)n * g.P;
  const double x_bytes = 4.0 * g.n * g.c * g.h * g.w, w_bytes = 4.0 * (double)g.M * (double)g.K, y_bytes = 4.0 * (double)g.M * (double)g.N;
  if (pass == VCNN_PASS_BWD_FILTER) {
    if (!filter_grad_bf16_plan(g, &p->filter, 2, max_splits)) return false;
    const size_t terms = 2 * (p->filter.x8n_bytes + p->filter.dyf_bytes);
    // (later parts add to dw through the slice sum, which then needs one slice at least)
    const size_t slices = std::max(p->filter.partial_bytes, n < whole.n ? (size_t)g.M * g.K * sizeof(float) : (size_t)0);
    p->workspace_bytes = terms + align256(slices);  // (the scales have a place of their own)
    p->est_seconds = p->filter.est_seconds + relay_seconds(x_bytes + y_bytes, (double)terms);
    return true;
  }
  if (pass == VCNN_PASS_FWD) {
    if (!conv_halo_bf16_plan(g.n, g.c, g.h, g.w, g.k, g.r, g.s, g.ph, g.pw, &p->fwd, 2)) return false;
  } else {
    // the input gradient as a correlation of dy (k channels) with the flipped kernels
    const int ph = g.r - 1 - g.ph, pw = g.s - 1 - g.pw;
    if (ph < 0 || pw < 0 || !conv_halo_bf16_plan(g.n, g.k, g.oh, g.ow, g.c, g.r, g.s, ph, pw, &p->fwd, 2)) return false;
  }
  const size_t terms = 2 * (p->fwd.x8_bytes + p->fwd.wf_bytes);
  p->workspace_bytes = split_scales_bytes(whole.n) + terms;
  p->est_seconds = p->fwd.est_seconds + relay_seconds((pass == VCNN_PASS_FWD ? x_bytes : y_bytes) + w_bytes, (double)terms);
  return true;
}

bool conv_f16x2_plan(const ConvGeom& g, int pass, size_t budget, F16x2Plan* p) {
  const bool filter = pass == VCNN_PASS_BWD_FILTER;
  const int unit = filter ? 8 : 1;  // the kernel gradient takes images in groups of eight
  bool found = false;
  for (int max_splits = 0; max_splits <= 64; max_splits = max_splits ? 2 * max_splits : 4) {
    for (int parts = 1, next; parts <= 16; parts = next) {
      next = parts + 1;
      const int images = (int)std::min<int64_t>(ceil_div(ceil_div(g.n, parts), unit) * unit, g.n);
      if (parts > 1 && (int64_t)images * (parts - 1) >= g.n) continue;  // fewer parts of this size do
      F16x2Plan q{};
      if (!part_plan(g, pass, images, max_splits, &q)) return false;
      if (const int rest = g.n % images) {  // the shorter last part has a plan of its own
        F16x2Plan last{};
        if (!part_plan(g, pass, rest, max_splits, &last)) return false;
        q.workspace_bytes = std::max(q.workspace_bytes, last.workspace_bytes);
      }
      if (q.workspace_bytes > budget) {  // (the room a part takes falls about as the parts rise)
        next = std::max(next, (int)(0.8 * parts * (double)q.workspace_bytes / (double)std::max<size_t>(budget, 1)));
        continue;
      }
      q.parts = parts, q.images = images, q.max_splits = max_splits;
      q.est_seconds *= parts;
      if (!found || q.est_seconds < p->est_seconds) *p = q;
      found = true;
      break;
    }
    if (!filter || (found && p->parts == 1 && p->max_splits == 0)) break;
  }
  return found;
}

// Runs `part(first image, its geometry, its plan)` over the parts of the batch.
template <typename F>
static vcnn_status each_part(const F16x2Plan& p, const ConvGeom& whole, int pass, F part) {
  for (int n0 = 0; n0 < whole.n; n0 += p.images) {
    ConvGeom g = whole;
    g.n = std::min(p.images, whole.n - n0), g.N = (int64_t)g.n * g.P;
    if (g.n == p.images) {
      if (vcnn_status e = part(n0, g, p)) return e;
      continue;
    }
    // the shorter last part: its own plan, whose room the whole plan has counted in
    F16x2Plan last{};
    if (!part_plan(whole, pass, g.n, p.max_splits, &last) || last.workspace_bytes > p.workspace_bytes)
      return fail(VCNN_ERR_UNSUPPORTED, "conv: no plan for the last %d images", g.n);
    if (vcnn_status e = part(n0, g, last)) return e;
  }
  return VCNN_OK;
}

vcnn_status launch_conv_f16x2_fwd(const F16x2Plan& plan, const ConvGeom& whole, const float* x, const float* w,
                                  const float* bias, float* y, int relu, void* workspace, hipStream_t st, const Declined& only) {
  const int64_t chw = (int64_t)whole.c * whole.h * whole.w;
  char* const x8 = (char*)workspace + split_scales_bytes(whole.n);
  return each_part(plan, whole, VCNN_PASS_FWD, [&](int n0, const ConvGeom& g, const F16x2Plan& p) {
    const SplitScales sc = split_scales(workspace, whole.n, g.n, chw, g.M * g.K, only).from(n0);
    if (vcnn_status e = launch_absmax(x + n0 * chw, g.n, chw, w, g.M * g.K, sc, n0 == 0, st)) return e;
    return launch_conv_halo_f16x2(p.fwd, g.n, g.c, g.h, g.w, g.k, g.r, g.s, g.ph, g.pw, x + n0 * chw, w, g.K,
                                  (int64_t)g.r * g.s, 0, bias, y + n0 * g.M * g.P, relu, sc, x8, x8 + 2 * p.fwd.x8_bytes, nullptr,
                                  st);
  });
}

vcnn_status launch_conv_f16x2_bwd_data(const F16x2Plan& plan, const ConvGeom& whole, const float* w, const float* dy,
                                       float* dx, float* flipped, void* workspace, hipStream_t st, const Declined& only) {
  const int64_t mp = whole.M * whole.P;
  char* const x8 = (char*)workspace + split_scales_bytes(whole.n);
  return each_part(plan, whole, VCNN_PASS_BWD_DATA, [&](int n0, const ConvGeom& g, const F16x2Plan& p) {
    const SplitScales sc = split_scales(workspace, whole.n, g.n, mp, g.M * g.K, only).from(n0);
    if (vcnn_status e = launch_absmax(dy + n0 * mp, g.n, mp, w, g.M * g.K, sc, n0 == 0, st)) return e;
    return launch_conv_halo_f16x2(p.fwd, g.n, g.k, g.oh, g.ow, g.c, g.r, g.s, g.r - 1 - g.ph, g.s - 1 - g.pw, dy + n0 * mp, w,
                                  (int64_t)g.r * g.s, g.K, 1, nullptr, dx + (int64_t)n0 * g.c * g.h * g.w, 0, sc, x8,
                                  x8 + 2 * p.fwd.x8_bytes, flipped, st);
  });
}

vcnn_status launch_conv_f16x2_filter(const F16x2Plan& plan, const ConvGeom& whole, const float* x, const float* dy, float* dw,
                                     void* workspace, void* scales, const FilterBehind& behind, hipStream_t st, const Declined& only) {
  const int64_t chw = (int64_t)whole.c * whole.h * whole.w, mp = whole.M * whole.P;
  char* const x8n = (char*)workspace;
  return each_part(plan, whole, VCNN_PASS_BWD_FILTER, [&](int n0, const ConvGeom& g, const F16x2Plan& p) {
    const SplitScales sc = split_scales(scales, 1, 1, g.n * chw, g.n * mp, only);
    char* const dyf = x8n + 2 * p.filter.x8n_bytes;
    if (vcnn_status e = launch_absmax(x + n0 * chw, 1, g.n * chw, dy + n0 * mp, g.n * mp, sc, n0 == 0, st)) return e;
    return launch_filter_grad_f16x2(p.filter, g, x + n0 * chw, dy + n0 * mp, dw, sc, x8n, dyf,
                                    (float*)(dyf + 2 * p.filter.dyf_bytes), st, n0 > 0, n0 + g.n == whole.n ? &behind : nullptr);
  });
}

}  // namespace vcnn
