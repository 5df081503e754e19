// What the passes through the Fourier domain leave to the direct route behind them (spectral.h), decided before the
// transforms from the energy of every pixel of the operands: the sum of the squares over the channels (maps), in double.
//
// The error of such a pass is that of the spectra, rounded to float, and is spread evenly over a transform: about 2^-23 of the
// root mean square over the WHOLE transform of what is summed there.  An output is exact to that relative to what it sums
// itself only if its own samples are not much darker than the rest of the transform.  The windows looked at are the outputs'
// own, pixel by pixel, with what lies outside the plane left out.  The scan and the guard take 15 us of a forward pass over 10 MB, 32 us
// of an input gradient over 79 MB (16 38 64 64 -> 512 16 16: 671 -> 717 us in all).
#include <algorithm>

#include "elem.h"
#include "spectral.h"

namespace vcnn {

// ---- energies ------------------------------------------------------------------------------------------------------
struct EnergyArgs {
  EnergyJob job[2];
  int blocks[2];  // per image
  int first_blocks;
  uint32_t* words;
  int cleared;
};

// A block does 256 pixels of an image, four a lane (64 at a time, pieces of 128 and 256 bytes lie across cache lines that two
// blocks then fetch: 16 512 49 49 in bfloat16 36 us), a wave a share of the channels, 32 loads in flight.
static constexpr int kEnergyPixels = 256, kEnergyWaves = 16, kEnergyBatch = 8;
template <typename T>
__global__ __launch_bounds__(64 * kEnergyWaves) void energies_kernel(EnergyArgs a) {
  __shared__ double part[kEnergyWaves][kEnergyPixels];
  constexpr int PX = kEnergyPixels / 64;
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6, waves = blockDim.x >> 6;
  if (blockIdx.x == 0)
    for (int i = tid; i < a.cleared; i += blockDim.x) a.words[i] = 0;
  const bool second = (int)blockIdx.x >= a.first_blocks;
  const EnergyJob& job = a.job[second];
  const int id = (int)blockIdx.x - (second ? a.first_blocks : 0), blocks = a.blocks[second], image = id / blocks;
  const int64_t first = (int64_t)(id - image * blocks) * kEnergyPixels + lane;
  const int each = (job.channels + waves - 1) / waves, begin = wave * each, end = min(begin + each, job.channels);
  const T* const src = (const T*)job.src + (int64_t)image * job.channels * job.pixels;
  int64_t at[PX];
  double sum[PX];
#pragma unroll
  for (int k = 0; k < PX; ++k) at[k] = min(first + 64 * k, job.pixels - 1), sum[k] = 0;
  for (int c0 = begin; c0 < end; c0 += kEnergyBatch) {
    T t[kEnergyBatch][PX];
#pragma unroll
    for (int u = 0; u < kEnergyBatch; ++u)
#pragma unroll
      for (int k = 0; k < PX; ++k) t[u][k] = src[min(c0 + u, end - 1) * job.pixels + at[k]];
#pragma unroll
    for (int u = 0; u < kEnergyBatch; ++u)
#pragma unroll
      for (int k = 0; k < PX; ++k) {
        const double f = (double)ld(&t[u][k]);
        sum[k] += c0 + u < end ? f * f : 0.0;
      }
  }
#pragma unroll
  for (int k = 0; k < PX; ++k) part[wave][lane + 64 * k] = sum[k];
  __syncthreads();
  for (int i = tid; i < kEnergyPixels; i += blockDim.x) {
    const int64_t pixel = first - lane + i;
    if (pixel >= job.pixels) break;
    double e = 0;
    for (int k = 0; k < waves; ++k) e += part[k][i];
    job.energy[image * job.pixels + pixel] = e;
  }
}

vcnn_status launch_energies(int dtype, int images, const EnergyJob& first, const EnergyJob& second, uint32_t* words, int cleared,
                            hipStream_t st) {
  EnergyArgs a{};
  a.job[0] = first, a.job[1] = second, a.words = words, a.cleared = cleared;
  a.blocks[0] = (int)ceil_div(first.pixels, kEnergyPixels), a.blocks[1] = (int)ceil_div(second.pixels, kEnergyPixels);
  a.first_blocks = images * a.blocks[0];
  const int64_t waves = std::min<int64_t>(ceil_div(std::max(first.channels, second.channels), kEnergyBatch), kEnergyWaves);
  const dim3 grid((unsigned)(images * (a.blocks[0] + a.blocks[1]))), block((unsigned)(64 * waves));
  if (dtype == VCNN_BF16) hipLaunchKernelGGL(energies_kernel<bf16>, grid, block, 0, st, a);
  else hipLaunchKernelGGL(energies_kernel<float>, grid, block, 0, st, a);
  return check_launch("energies");
}

// ---- windows of outputs --------------------------------------------------------------------------------------------
// The sum over a block, by all its threads.
__device__ __forceinline__ double block_sum(double v, double* lds) {
#pragma unroll
  for (int d = 32; d > 0; d >>= 1) v += __shfl_xor(v, d);
  __syncthreads();
  if ((threadIdx.x & 63) == 0) lds[threadIdx.x >> 6] = v;
  __syncthreads();
  double sum = lds[0];
  for (int k = 1; k < (int)blockDim.x / 64; ++k) sum += lds[k];
  return sum;
}
// The bits any thread of a block has; `word` is zero before the last barrier.
__device__ __forceinline__ int block_or(int bits, int* word) {
  if (bits) atomicOr(word, bits);
  __syncthreads();
  return *word;
}
__device__ __forceinline__ bool is_finite(double v) { return v < __builtin_inf(); }  // (v >= 0 or NaN)

// Whether an output sums too little of its transform's energy (a sum of no energy at all is exact by itself).
__device__ __forceinline__ bool is_dark(const WindowGuard& g, double window, int samples, double total) {
  return window != 0 && !(window >= total * fmax(samples * g.mean, g.least));
}
// By one thread, for one transform.
__device__ __forceinline__ void note_transform(const WindowGuard& g, int64_t transform, int64_t image, double total, bool bad, bool zero) {
  g.totals[transform] = total;
  if (zero) *g.words.zeros = 1;
  if (bad || !is_finite(total)) g.words.image[image] = 1, *g.words.any = 1;
}
// Samples of the window of transform sample i (along one axis) that lie in the tensor, samples first .. last - 1 of the transform.
__device__ __forceinline__ int inside_window(int i, int taps, int back, int first, int last) {
  const int from = back ? i - taps + 1 : i;
  return max(0, min(from + taps, last) - max(from, first));
}
// The sums of `taps` values each from lane i on (back: up to lane i), of 64 in a wave, from those of powers of two of them.
template <int N>
__device__ __forceinline__ void wave_windows(double (&v)[N], int taps, int back) {
  const int lane = threadIdx.x & 63;
  auto shifted = [&](double f, int d) {
    const int from = back ? lane - d : lane + d;
    const double t = __shfl(f, from & 63);
    return (unsigned)from < 64u ? t : 0.0;
  };
  double sum[N];
#pragma unroll
  for (int k = 0; k < N; ++k) sum[k] = 0;
  for (int b = 0, done = 0; taps >> b; ++b) {
    if (taps >> b & 1) {
#pragma unroll
      for (int k = 0; k < N; ++k) sum[k] += shifted(v[k], done);
      done += 1 << b;
    }
#pragma unroll
    for (int k = 0; k < N; ++k) v[k] += shifted(v[k], 1 << b);
  }
#pragma unroll
  for (int k = 0; k < N; ++k) v[k] = sum[k];
}

// A block per transform, a wave per row and then per column.
static constexpr int kGuardThreads = 1024, kGuardEach = kFL * kFL / kGuardThreads;
__global__ __launch_bounds__(kGuardThreads) void guard_planes_kernel(WindowGuard g, SpectralTiles in, SpectralTiles out, int r, int s) {
  __shared__ double e[kFL][kFL + 1];
  __shared__ double red[kGuardThreads / 64];
  __shared__ int flags;
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6, tx = blockIdx.x % in.tiles_x, ty = blockIdx.x / in.tiles_x % in.tiles_y;
  const int n = blockIdx.x / in.tiles_x / in.tiles_y;
  const int y0 = ty * in.step_y + in.y0, x0 = tx * in.step_x + in.x0;  // the transform's first pixel
  double v[kGuardEach], sum = 0;
  if (tid == 0) flags = 0;
#pragma unroll
  for (int k = 0; k < kGuardEach; ++k) {
    const int py = y0 + wave * kGuardEach + k, px = x0 + lane;
    const bool ok = (unsigned)py < (unsigned)in.h && (unsigned)px < (unsigned)in.w;
    v[k] = ok ? g.energy[((int64_t)n * in.h + py) * in.w + px] : 0.0;
    sum += v[k];
  }
  wave_windows(v, s, g.back);
#pragma unroll
  for (int k = 0; k < kGuardEach; ++k) e[wave * kGuardEach + k][lane] = v[k];
  const double total = block_sum(sum, red);  // (and the rows are there)
#pragma unroll
  for (int k = 0; k < kGuardEach; ++k) v[k] = e[lane][wave * kGuardEach + k];
  wave_windows(v, r, g.back);
  const int y = lane, ly = y - out.y0, py = ty * out.step_y + ly;
  const bool row = ly >= 0 && ly < out.lim_y && py < out.h;
  const int rows = inside_window(y, r, g.back, -y0, in.h - y0);
  bool bad = false, zero = false;
  __syncthreads();
  uint64_t* const mask = reinterpret_cast<uint64_t*>(&e[0][0]);  // [column], a bit per row
#pragma unroll
  for (int k = 0; k < kGuardEach; ++k) {
    const int x = wave * kGuardEach + k, lx = x - out.x0, px = tx * out.step_x + lx;
    const bool valid = row && lx >= 0 && lx < out.lim_x && px < out.w;
    bad |= valid && is_dark(g, v[k], rows * inside_window(x, s, g.back, -x0, in.w - x0), total);
    const uint64_t zeros = __ballot(valid && v[k] == 0);
    zero |= zeros != 0;
    if (lane == 0) mask[x] = zeros;
  }
  const int any = block_or((bad ? 1 : 0) | (zero ? 2 : 0), &flags);
  if (tid < kFL) {  // turned: a word per row
    uint64_t w = 0;
    if (any & 2)
      for (int x = 0; x < kFL; ++x) w |= (mask[x] >> tid & 1) << x;
    g.zero[(int64_t)blockIdx.x * kFL + tid] = w;
  }
  if (tid == 0) note_transform(g, blockIdx.x, n, total, any & 1, any & 2);
}

// A thread per sample of four lines, again from the sums over powers of two of them.
static constexpr int kGuardLines = 4;
__global__ __launch_bounds__(kLL) void guard_lines_kernel(WindowGuard g, SpectralLines in, SpectralLines out, int taps) {
  __shared__ double e[2][kGuardLines][kLL];
  __shared__ double red[kGuardLines][kLL / 64];
  __shared__ int flags;
  const int i = threadIdx.x, lines = in.images * in.others * in.tiles, sign = g.back ? -1 : 1;
  double v[kGuardLines], window[kGuardLines];
  if (i == 0) flags = 0;
#pragma unroll
  for (int k = 0; k < kGuardLines; ++k) {
    const int line = min((int)blockIdx.x * kGuardLines + k, lines - 1), tile = line % in.tiles, o = line / in.tiles % in.others;
    const int64_t n = line / in.tiles / in.others;
    const int px = tile * in.step + in.x0 + i;
    v[k] = (unsigned)px < (unsigned)in.len ? g.energy[n * in.s_channel + o * in.s_other + px * in.s_along] : 0.0;
    window[k] = 0;
  }
#pragma unroll
  for (int k = 0; k < kGuardLines; ++k) {
    double sum = v[k];
#pragma unroll
    for (int d = 32; d > 0; d >>= 1) sum += __shfl_xor(sum, d);
    if ((i & 63) == 0) red[k][i >> 6] = sum;
    e[0][k][i] = v[k];
  }
  __syncthreads();
  for (int b = 0, done = 0; taps >> b; ++b) {
    auto at = [&](int k, int d) {
      const int from = i + sign * d;
      return (unsigned)from < (unsigned)kLL ? e[b & 1][k][from & (kLL - 1)] : 0.0;
    };
#pragma unroll
    for (int k = 0; k < kGuardLines; ++k) {
      if (taps >> b & 1) window[k] += at(k, done);
      v[k] += at(k, 1 << b);
      e[(b + 1) & 1][k][i] = v[k];
    }
    if (taps >> b & 1) done += 1 << b;
    __syncthreads();
  }
  int found = 0;
#pragma unroll
  for (int k = 0; k < kGuardLines; ++k) {
    const int line = blockIdx.x * kGuardLines + k, tile = line % in.tiles;
    const double total = (red[k][0] + red[k][1]) + (red[k][2] + red[k][3]);
    const int x0 = tile * in.step + in.x0, lx = i - out.x0;
    const bool valid = line < lines && lx >= 0 && lx < out.lim && tile * out.step + lx < out.len;
    const bool bad = valid && is_dark(g, window[k], inside_window(i, taps, g.back, -x0, in.len - x0), total);
    const uint64_t zeros = __ballot(valid && window[k] == 0);
    if ((i & 63) == 0 && line < lines) g.zero[(int64_t)line * 4 + (i >> 6)] = zeros;
    found |= (bad ? 1 << k : 0) | (zeros ? 16 << k : 0);
  }
  found = block_or(found, &flags);
  const int line = blockIdx.x * kGuardLines + i;
  if (i < kGuardLines && line < lines)
    note_transform(g, line, line / in.tiles / in.others, (red[i][0] + red[i][1]) + (red[i][2] + red[i][3]), found >> i & 1, found >> i & 16);
}

vcnn_status launch_guard_planes(const WindowGuard& g, const SpectralTiles& in, const SpectralTiles& out, int r, int s, hipStream_t st) {
  hipLaunchKernelGGL(guard_planes_kernel, dim3((unsigned)((int64_t)in.images * in.tiles_y * in.tiles_x)), dim3(kGuardThreads), 0, st, g, in, out, r, s);
  return check_launch("guard_planes");
}
vcnn_status launch_guard_lines(const WindowGuard& g, const SpectralLines& in, const SpectralLines& out, int taps, hipStream_t st) {
  const int64_t lines = (int64_t)in.images * in.others * in.tiles;
  hipLaunchKernelGGL(guard_lines_kernel, dim3((unsigned)ceil_div(lines, kGuardLines)), dim3(kLL), 0, st, g, in, out, taps);
  return check_launch("guard_lines");
}

}  // namespace vcnn
