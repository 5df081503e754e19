// What the passes through the Fourier domain leave to the direct route behind them (spectral.h), decided before the
// transforms from the energy of every pixel of the operands: the sum of the squares over the channels (maps), in double.
//
// The error of such a pass is that of the spectra, rounded to float, and is spread evenly over a transform: about 2^-23 of the
// root mean square over the WHOLE transform of what is summed there.  An output is exact to that relative to what it sums
// itself only if its own samples are not much darker than the rest of the transform.  The windows looked at are the outputs'
// own, pixel by pixel, with what lies outside the plane left out.  The scan and the guard take 15 us of a forward pass over 10 MB, 32 us
// of an input gradient over 79 MB and 32 us of a kernel gradient over both (16 38 64 64 -> 512 16 16: 672 -> 752 us in all, of which the
// direct routes would take 3240).
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

// A block does 256 pixels of an image, four a lane, a wave a share of the channels, 32 loads in flight.  (Smaller pieces lie across
// cache lines that two blocks then fetch: 16 512 49 49 takes 22 us, 24 with 128 pixels; in bfloat16 15, and 36 with 64.)
static constexpr int kEnergyWaves = 16, kEnergyPixels = 256, kEnergyBatch = 8;
template <typename T>
__global__ __launch_bounds__(64 * kEnergyWaves) void energies_kernel(EnergyArgs a) {
  constexpr int PX = kEnergyPixels / 64, PIXELS = kEnergyPixels, BATCH = kEnergyBatch;
  __shared__ double part[kEnergyWaves][PIXELS];
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6, waves = blockDim.x >> 6;
  if (blockIdx.x == 0)
    for (int i = tid; i < a.cleared; i += blockDim.x) a.words[i] = 0;
  const bool second = (int)blockIdx.x >= a.first_blocks;
  const EnergyJob& job = a.job[second];
  const int id = (int)blockIdx.x - (second ? a.first_blocks : 0), blocks = a.blocks[second], image = id / blocks;
  const int64_t first = (int64_t)(id - image * blocks) * PIXELS;
  const int each = (job.channels + waves - 1) / waves, begin = wave * each, end = min(begin + each, job.channels);
  const T* const src = (const T*)job.src + (int64_t)image * job.channels * job.pixels;
  int64_t at[PX];
  double sum[PX];
#pragma unroll
  for (int k = 0; k < PX; ++k) at[k] = min(first + lane + 64 * k, job.pixels - 1), sum[k] = 0;
  for (int c0 = begin; c0 < end; c0 += BATCH) {
    T t[BATCH][PX];
#pragma unroll
    for (int u = 0; u < BATCH; ++u)
#pragma unroll
      for (int k = 0; k < PX; ++k) t[u][k] = src[min(c0 + u, end - 1) * job.pixels + at[k]];
#pragma unroll
    for (int u = 0; u < BATCH; ++u)
#pragma unroll
      for (int k = 0; k < PX; ++k) {
        const double f = (double)ld(&t[u][k]);
        sum[k] += c0 + u < end ? f * f : 0.0;
      }
  }
#pragma unroll
  for (int k = 0; k < PX; ++k) part[wave][lane + 64 * k] = sum[k];
  __syncthreads();
  for (int i = tid; i < PIXELS && first + i < job.pixels; i += blockDim.x) {
    double e = 0;
    for (int k = 0; k < waves; ++k) e += part[k][i];
    job.energy[image * job.pixels + first + i] = e;
  }
}

// (the larger operand's blocks in front)
vcnn_status launch_energies(int dtype, int images, const EnergyJob& x, const EnergyJob& y, uint32_t* words, int cleared, hipStream_t st) {
  const bool turn = x.channels * x.pixels < y.channels * y.pixels;
  const EnergyJob &first = turn ? y : x, &second = turn ? x : y;
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

// ---- what meets at the taps of a kernel gradient ---------------------------------------------------------------------
// dW(tap) adds x(p + tap) dy(p); over the channels and maps its variance is the sum of the energies' products, M(tap).  The error is
// that of a correlation over the whole transform, sum over all shifts / samples = total(x) total(dy) / samples: the same for every
// tap, however little meets at it (black areas under all that is large in dy, for one).
//
// A transform with nothing or with something that is not finite in either operand: 0 or not finite in the totals' product.
__device__ __forceinline__ bool out_of_range(double energy, int depth) {
  if (energy == 0) return false;
  const int norm = ((__double2hiint(energy) >> 20) - 1023) >> 1;
  return norm + 1 > 110 || norm - depth < -90;
}

static constexpr int kThreads = 256;
// A block does a row of taps of some transforms, a thread four of them along one row of the plane.
__global__ __launch_bounds__(kThreads) void meet_planes_kernel(MeetGuard m, SpectralTiles tx, SpectralTiles tdy, int r, int s) {
  __shared__ double ex[kFL][kFL + 1], ey[kFL][kFL + 1];
  __shared__ double red[4], part[4][16];
  const int tid = threadIdx.x, q = blockIdx.x % r, chunk = blockIdx.x / r, tap = 4 * (tid & 3), row = tid >> 2;
  const int tiles = tx.images * tx.tiles_y * tx.tiles_x, taps = r * s;
  double acc[4] = {0, 0, 0, 0}, totals = 0;
  for (int t = chunk * m.per_chunk; t < min(tiles, (chunk + 1) * m.per_chunk); ++t) {
    const int ix = t % tx.tiles_x, iy = t / tx.tiles_x % tx.tiles_y;
    const int64_t n = t / tx.tiles_x / tx.tiles_y;
    const int x0 = ix * tx.step_x + tx.x0, y0 = iy * tx.step_y + tx.y0, dx0 = ix * tdy.step_x, dy0 = iy * tdy.step_y;
    double e[16], f[16], sum_x = 0, sum_y = 0;
#pragma unroll
    for (int k = 0; k < 16; ++k) {
      const int y = (tid >> 6) + 4 * k, x = tid & 63;
      const bool in = (unsigned)(y0 + y) < (unsigned)tx.h && (unsigned)(x0 + x) < (unsigned)tx.w;
      const bool out = y < tdy.lim_y && x < tdy.lim_x && dy0 + y < tdy.h && dx0 + x < tdy.w;
      e[k] = in ? m.x[(n * tx.h + y0 + y) * tx.w + x0 + x] : 0.0;
      f[k] = out ? m.dy[(n * tdy.h + dy0 + y) * tdy.w + dx0 + x] : 0.0;
    }
    __syncthreads();
#pragma unroll
    for (int k = 0; k < 16; ++k) {
      const int y = (tid >> 6) + 4 * k, x = tid & 63;
      ex[y][x] = e[k], ey[y][x] = f[k];
      sum_x += e[k], sum_y += f[k];
    }
    if (q == 0) {
      sum_x = block_sum(sum_x, red), sum_y = block_sum(sum_y, red);
      totals += sum_x * sum_y;
      if (tid == 0 && sum_x != 0 && sum_y != 0 && (out_of_range(sum_x, m.depth_x) || out_of_range(sum_y, m.depth_dy))) *m.words.any = 1;
    }
    __syncthreads();
    if (row < tdy.lim_y) {  // (row + q and, of the taps there are, x + tap lie in the transform)
      const double* const from = ex[(row + q) & 63];
      double a = from[tap], b = from[tap + 1], c = from[tap + 2];
      for (int x = 0; x < tdy.lim_x; ++x) {
        const double g = ey[row][x], d = from[min(x + tap + 3, kFL - 1)];
        acc[0] += g * a, acc[1] += g * b, acc[2] += g * c, acc[3] += g * d;
        a = b, b = c, c = d;
      }
    }
  }
#pragma unroll
  for (int k = 0; k < 4; ++k) {
#pragma unroll
    for (int d = 4; d < 64; d <<= 1) acc[k] += __shfl_xor(acc[k], d);
    if ((tid & 63) < 4) part[tid >> 6][tap + k] = acc[k];
  }
  __syncthreads();
  if (tid < s) m.partial[(int64_t)chunk * (taps + 1) + q * s + tid] = (part[0][tid] + part[1][tid]) + (part[2][tid] + part[3][tid]);
  if (tid == 0 && q == 0) m.partial[(int64_t)chunk * (taps + 1) + taps] = totals;
}

// Two threads a tap, each half of a line.
__global__ __launch_bounds__(kThreads) void meet_lines_kernel(MeetGuard m, SpectralLines tx, SpectralLines tdy, int taps) {
  __shared__ double ex[2 * kLL], ey[kLL];
  __shared__ double red[4], other[kLineTaps];
  const int tid = threadIdx.x, tap = tid & (kLineTaps - 1), from = (tid >> 7) * (kLL / 2);
  const int lines = tx.images * tx.others * tx.tiles;
  double acc = 0, totals = 0;
  ex[kLL + tid] = 0;
  for (int l = blockIdx.x * m.per_chunk; l < min(lines, ((int)blockIdx.x + 1) * m.per_chunk); ++l) {
    const int tile = l % tx.tiles, o = l / tx.tiles % tx.others;
    const int64_t n = l / tx.tiles / tx.others;
    const int px = tile * tx.step + tx.x0 + tid, py = tile * tdy.step + tid;
    const double e = (unsigned)px < (unsigned)tx.len ? m.x[n * tx.s_channel + o * tx.s_other + px * tx.s_along] : 0.0;
    const double f = tid < tdy.lim && py < tdy.len ? m.dy[n * tdy.s_channel + o * tdy.s_other + py * tdy.s_along] : 0.0;
    __syncthreads();
    ex[tid] = e, ey[tid] = f;
    const double sum_x = block_sum(e, red), sum_y = block_sum(f, red);
    totals += sum_x * sum_y;
    if (tid == 0 && sum_x != 0 && sum_y != 0 && (out_of_range(sum_x, m.depth_x) || out_of_range(sum_y, m.depth_dy))) *m.words.any = 1;
#pragma unroll 8
    for (int k = 0; k < kLL / 2; ++k) acc += ey[from + k] * ex[from + k + tap];
  }
  if (from) other[tap] = acc;
  __syncthreads();
  if (tid < taps) m.partial[(int64_t)blockIdx.x * (taps + 1) + tid] = acc + other[tid];
  if (tid == 0) m.partial[(int64_t)blockIdx.x * (taps + 1) + taps] = totals;
}

vcnn_status launch_meet_planes(const MeetGuard& m, const SpectralTiles& x, const SpectralTiles& dy, int r, int s, hipStream_t st) {
  hipLaunchKernelGGL(meet_planes_kernel, dim3((unsigned)(m.chunks * r)), dim3(kThreads), 0, st, m, x, dy, r, s);
  return check_launch("meet_planes");
}
vcnn_status launch_meet_lines(const MeetGuard& m, const SpectralLines& x, const SpectralLines& dy, int taps, hipStream_t st) {
  hipLaunchKernelGGL(meet_lines_kernel, dim3((unsigned)m.chunks), dim3(kThreads), 0, st, m, x, dy, taps);
  return check_launch("meet_lines");
}

}  // namespace vcnn
