// Real planes of 64 x 64 pixels to their spectra and back, in double (spectral.h).
//
// A transform of 64 points is 8 x 8: thread j of eight holds points j + 8 i, transforms over i, multiplies by the twiddles,
// hands values over in LDS (its own wave's: no barrier) and transforms again, which leaves it points k1 + 8 k2 of the
// result.  Two real rows share one complex transform, as its real and imaginary part.  One block of 256 threads does a
// plane: 32 pairs of rows, a transposition through LDS (one barrier on either side), 32 columns (the real columns 0 and 32
// share one).  Double costs the vector units no more than float and the LDS traffic twice as much; the kernels are bound by
// the memory the spectra take: 16.9 KB written (read) a plane, 8192 planes of 49 x 49 pixels (dY of 512 maps, batch 16) 67 us
// forward and 62 back, 608 planes 11 us, 19456 kernels of 16 x 16 (row spectra, 4.2 KB each) 28 us either way.
#include "elem.h"
#include "spectral.h"
#include "spectral_math.h"

namespace vcnn {

static constexpr int kThreads = 256;
static constexpr int kPitch = 65;  // of a row of 64 complex doubles in LDS: eight rows 16 bytes apart in their banks

// e^(-2 pi i j / 64), j < 8
__device__ const cd kRoot64[8] = {{1.0, -0.0},
                                  {0.99518472667219688624, -0.09801714032956060199},
                                  {0.98078528040323044913, -0.19509032201612826785},
                                  {0.95694033573220886494, -0.29028467725446236764},
                                  {0.92387953251128675613, -0.38268343236508977173},
                                  {0.88192126434835502971, -0.47139673682599764856},
                                  {0.83146961230254523708, -0.55557023301960222474},
                                  {0.77301045336273696081, -0.63439328416364549822}};
// v[k] *= w^k
__device__ __forceinline__ void twiddle(cd (&v)[8], cd w) {
  const cd w2 = w * w, w3 = w2 * w, w4 = w2 * w2;
  v[1] = v[1] * w, v[2] = v[2] * w2, v[3] = v[3] * w3, v[4] = v[4] * w4;
  v[5] = v[5] * (w4 * w), v[6] = v[6] * (w3 * w3), v[7] = v[7] * (w4 * w3);
}
// Between the two halves of a transform: thread j has v[k] and gets the v[j] of the eight threads, through its row of LDS.
__device__ __forceinline__ void exchange(cd (&v)[8], cd* row, int j) {
  wave_sync();
#pragma unroll
  for (int k = 0; k < 8; ++k) row[k * 8 + (j ^ k)] = v[k];
  wave_sync();
#pragma unroll
  for (int i = 0; i < 8; ++i) v[i] = row[j * 8 + (i ^ j)];
  wave_sync();
}
// The same hand-over of results rounded to float: the eight threads' points j + 8 k <-> 8 j + i of a column, so that they read
// and write its 512 bytes in whole lines.
__device__ __forceinline__ void exchange(float2 (&v)[8], float2* row, int j) {
  wave_sync();
#pragma unroll
  for (int k = 0; k < 8; ++k) row[k * 8 + (j ^ k)] = v[k];
  wave_sync();
#pragma unroll
  for (int i = 0; i < 8; ++i) v[i] = row[j * 8 + (i ^ j)];
  wave_sync();
}
// points j + 8 i in, k1 = j: points k1 + 8 k2 out; the inverse the other way round (unscaled)
__device__ __forceinline__ void fft64(cd (&v)[8], cd* row, int j, cd w) {
  dft8<false>(v);
  twiddle(v, w);
  exchange(v, row, j);
  dft8<false>(v);
}
__device__ __forceinline__ void ifft64(cd (&v)[8], cd* row, int j, cd w) {
  dft8<true>(v);
  twiddle(v, conj(w));
  exchange(v, row, j);
  dft8<true>(v);
}

// By one block of 256 threads (spectral.h).
__device__ void decide_meeting(const MeetDecision& m, uint64_t* zero) {
  const int tid = threadIdx.x, taps = m.r * m.s;
  if (tid < 16) zero[tid] = 0;
  __syncthreads();
  if (tid < taps) {
    double meets = 0, total = 0;
#pragma unroll 8
    for (int c = 0; c < m.chunks; ++c) meets += m.partial[(int64_t)c * (taps + 1) + tid], total += m.partial[(int64_t)c * (taps + 1) + taps];
    bool bad = !(total < __builtin_inf());
    if (total > 0) {
      const int norms = ((__double2hiint(total) >> 20) - 1023) >> 1;  // of the product of two of them
      bad |= norms + 1 + 24 + m.grow > 126 || norms < -80 || (meets != 0 && !(meets >= total * m.share));
    }
    if (bad) *m.words.any = 1;
    if (meets == 0) {
      const int row = m.r == 1 || m.s == 1 ? tid >> 6 : tid / m.s, bit = m.r == 1 || m.s == 1 ? tid & 63 : tid % m.s;
      atomicOr((unsigned long long*)zero + row, 1ull << bit);
      *m.words.zeros = 1;
    }
  }
  __syncthreads();
  if (tid < 16) m.zero[tid] = zero[tid];
}

// ---- planes ------------------------------------------------------------------------------------------------------
struct PlaneArgs {
  SpectralTiles t;
  const void* src;
  float2* spectra;
  double* sums;
  const uint32_t* declined;
  int per_image;
  int64_t planes;
  MeetDecision decide;
};

template <typename T>
__global__ __launch_bounds__(kThreads) void plane_spectra_kernel(PlaneArgs a) {
  __shared__ cd z[32 * kPitch];
  const int tid = threadIdx.x, j = tid & 7, q = tid >> 3;
  const int64_t p = blockIdx.x;
  if (p == a.planes) return decide_meeting(a.decide, reinterpret_cast<uint64_t*>(z));
  const SpectralTiles& t = a.t;
  const int c = (int)(p % t.count), tx = (int)(p / t.count % t.tiles_x), ty = (int)(p / t.count / t.tiles_x % t.tiles_y);
  const int64_t n = p / t.count / t.tiles_x / t.tiles_y;
  const uint32_t leaves = a.declined && !a.sums ? a.declined[a.per_image ? n : 0] : 0;  // (looked at where its latency is over)
  const T* const src = (const T*)a.src + (n * t.channels + t.first + c) * ((int64_t)t.h * t.w);
  const int y0 = ty * t.step_y + t.y0, x0 = tx * t.step_x + t.x0;
  // the pixels of the transform that lie in the tile and in the plane
  const int top = max(0, -y0), bottom = min(t.lim_y, t.h - y0), left = max(0, -x0), right = min(t.lim_x, t.w - x0);
  float lo[8], hi[8];
  const int at = (y0 + q) * t.w + x0 + j;
#pragma unroll
  for (int half = 0; half < 2; ++half)
#pragma unroll
    for (int i = 0; i < 8; ++i) {
      const int ly = q + 32 * half, lx = j + 8 * i;
      const bool in = ly >= top && ly < bottom && lx >= left && lx < right;
      (half ? hi : lo)[i] = ld(src + (unsigned)(in ? at + 32 * half * t.w + 8 * i : 0));
    }
  if (leaves) return;
#pragma unroll
  for (int half = 0; half < 2; ++half)  // (all loads in flight before the first is looked at)
#pragma unroll
    for (int i = 0; i < 8; ++i) {
      const int ly = q + 32 * half, lx = j + 8 * i;
      if (!(ly >= top && ly < bottom && lx >= left && lx < right)) (half ? hi : lo)[i] = 0.f;
    }
  const cd w = kRoot64[j];
  cd v[8];
#pragma unroll
  for (int i = 0; i < 8; ++i) v[i] = {(double)lo[i], (double)hi[i]};
  fft64(v, z + q * kPitch, j, w);  // rows q and q + 32
#pragma unroll
  for (int k = 0; k < 8; ++k) z[q * kPitch + j + 8 * k] = v[k];
  __syncthreads();
  // column `col` (0: columns 0 and 32 as real and imaginary part)
  const int col = q, other = col == 0 ? 32 : 64 - col;
#pragma unroll
  for (int i = 0; i < 4; ++i) {
    const cd A = z[(j + 8 * i) * kPitch + col], B = z[(j + 8 * i) * kPitch + other];
    if (col == 0) {
      v[i] = {A.x, B.x}, v[i + 4] = {A.y, B.y};
    } else {
      v[i] = {0.5 * (A.x + B.x), 0.5 * (A.y - B.y)};
      v[i + 4] = {0.5 * (A.y + B.y), 0.5 * (B.x - A.x)};
    }
  }
  __syncthreads();
  fft64(v, z + col * kPitch, j, w);
  auto put = [&](int column, const cd (&s)[8]) {
    float2 f[8];
#pragma unroll
    for (int k = 0; k < 8; ++k) f[k] = make_float2((float)s[k].x, (float)s[k].y);
    exchange(f, reinterpret_cast<float2*>(z + col * kPitch), j);
    float4* const out = reinterpret_cast<float4*>(a.spectra + ((int64_t)column * a.planes + p) * 64) + j;
#pragma unroll
    for (int rho = 0; rho < 4; ++rho) out[8 * rho] = make_float4(f[rho].x, f[rho].y, f[rho + 4].x, f[rho + 4].y);
  };
  if (a.sums && tid == 0) a.sums[p] = v[0].x;  // (additions only, also where an element is not finite)
  if (col == 0) {
    cd* const row = z;
    wave_sync();
#pragma unroll
    for (int k = 0; k < 8; ++k) row[j + 8 * k] = v[k];
    wave_sync();
    cd r[8];
#pragma unroll
    for (int k = 0; k < 8; ++k) {
      const cd B = row[(64 - j - 8 * k) & 63], A = v[k];
      v[k] = {0.5 * (A.x + B.x), 0.5 * (A.y - B.y)};
      r[k] = {0.5 * (A.y + B.y), 0.5 * (B.x - A.x)};
    }
    put(32, r);
  }
  put(col, v);
}

struct InverseArgs {
  SpectralTiles t;
  SpectralExcept except;
  const float2* spectra;
  int64_t slice, planes;
  int slices;
  void* dst;
  const float* bias;
  int relu;
};

template <typename T>
__global__ __launch_bounds__(kThreads) void plane_inverse_kernel(InverseArgs a) {
  __shared__ cd z[32 * kPitch];
  const int tid = threadIdx.x, j = tid & 7, q = tid >> 3;
  const int64_t p = blockIdx.x;
  const SpectralTiles& t = a.t;
  const int64_t tile = p / t.count, n = tile / t.tiles_x / t.tiles_y;
  // (looked at where their latency is over)
  const uint32_t leaves = a.except.declined ? a.except.declined[a.except.per_image ? n : 0] : 0, zeros = a.except.zero ? *a.except.zeros : 0;
  const cd w = kRoot64[j];
  const int col = q;
  cd v[8];
  auto get = [&](int column, cd (&s)[8]) {
    const float4* in = reinterpret_cast<const float4*>(a.spectra + ((int64_t)column * a.planes + p) * 64) + j;
    if (a.slices == 1) {
      float2 f[8];
#pragma unroll
      for (int rho = 0; rho < 4; ++rho) {
        const float4 t = in[8 * rho];
        f[rho] = make_float2(t.x, t.y), f[rho + 4] = make_float2(t.z, t.w);
      }
      exchange(f, reinterpret_cast<float2*>(z + col * kPitch), j);
#pragma unroll
      for (int k = 0; k < 8; ++k) s[k] = {(double)f[k].x, (double)f[k].y};
      return;
    }
#pragma unroll
    for (int k = 0; k < 8; ++k) s[k] = {0, 0};
    for (int l = 0; l < a.slices; ++l, in += a.slice / 2) {
#pragma unroll
      for (int rho = 0; rho < 4; ++rho) {
        const float4 t = in[8 * rho];
        s[rho] = s[rho] + cd{(double)t.x, (double)t.y}, s[rho + 4] = s[rho + 4] + cd{(double)t.z, (double)t.w};
      }
    }
    exchange(s, z + col * kPitch, j);
  };
  get(col, v);
  if (col == 0) {
    cd r[8];
    get(32, r);
#pragma unroll
    for (int k = 0; k < 8; ++k) v[k] = {v[k].x - r[k].y, v[k].y + r[k].x};
  }
  ifft64(v, z + col * kPitch, j, w);
  if (leaves) return;
  __syncthreads();
#pragma unroll
  for (int i = 0; i < 4; ++i) {
    cd* const row = z + (j + 8 * i) * kPitch;
    const cd lower = v[i], upper = v[i + 4];
    if (col == 0) {
      row[0] = {lower.x, upper.x}, row[32] = {lower.y, upper.y};
    } else {
      row[col] = {lower.x - upper.y, lower.y + upper.x};
      row[64 - col] = {lower.x + upper.y, upper.x - lower.y};
    }
  }
  __syncthreads();
#pragma unroll
  for (int k = 0; k < 8; ++k) v[k] = z[q * kPitch + j + 8 * k];
  ifft64(v, z + q * kPitch, j, w);
  const int c = (int)(p % t.count), tx = (int)(tile % t.tiles_x), ty = (int)(tile / t.tiles_x % t.tiles_y);
  const int64_t plane = (n * t.channels + t.first + c) * ((int64_t)t.h * t.w);
  T* const dst = (T*)a.dst + plane;
  const float bias = a.bias ? a.bias[t.first + c] : 0.f;
#pragma unroll
  for (int half = 0; half < 2; ++half) {
    const int ly = q + 32 * half - t.y0, y = ty * t.step_y + ly;
    if (ly < 0 || ly >= t.lim_y || y >= t.h) continue;
    const uint64_t zero = zeros ? a.except.zero[tile * kFL + q + 32 * half] >> j : 0;
#pragma unroll
    for (int i = 0; i < 8; ++i) {
      const int lx = j + 8 * i - t.x0, x = tx * t.step_x + lx;
      if (lx < 0 || lx >= t.lim_x || x >= t.w) continue;
      float r = zero >> 8 * i & 1 ? bias : (float)((half ? v[i].y : v[i].x) * (1.0 / 4096) + (double)bias);
      if (a.relu) r = fmaxf(r, 0.f);
      st(dst + (int64_t)y * t.w + x, r);
    }
  }
}

// ---- kernels -----------------------------------------------------------------------------------------------------
// Four kernels a block: pair b of a kernel's rows is (b, b + 8), of whose 64 points only the first 16 are not zero.
template <typename T>
__global__ __launch_bounds__(kThreads) void taps_spectra_kernel(const T* __restrict__ wgt, int64_t kernels, int r, int s,
                                                                float2* __restrict__ spectra, uint32_t* __restrict__ largest) {
  __shared__ cd z[32 * kPitch];
  __shared__ uint32_t wave_max[4];
  const int tid = threadIdx.x, j = tid & 7, q = tid >> 3;
  const int64_t first = (int64_t)blockIdx.x * 4, kernel = first + (q >> 3);
  const int row = q & 7;
  float f[2][2];
  uint32_t m = 0;
#pragma unroll
  for (int half = 0; half < 2; ++half)
#pragma unroll
    for (int i = 0; i < 2; ++i) {
      const int y = row + 8 * half, x = j + 8 * i;
      const float t = ld(wgt + (min(kernel, kernels - 1) * r + min(y, r - 1)) * s + min(x, s - 1));
      f[half][i] = kernel < kernels && y < r && x < s ? t : 0.f;
    }
#pragma unroll
  for (int half = 0; half < 2; ++half)
#pragma unroll
    for (int i = 0; i < 2; ++i) m = max(m, __float_as_uint(f[half][i]) & 0x7fffffffu);
#pragma unroll
  for (int d = 32; d > 0; d >>= 1) m = max(m, (uint32_t)__shfl_xor((int)m, d));
  if ((tid & 63) == 0) wave_max[tid >> 6] = m;
  const cd w = kRoot64[j], a{(double)f[0][0], (double)f[1][0]}, b{(double)f[0][1], (double)f[1][1]};
  constexpr double h = 0.70710678118654752440;
  const cd t1{h * (b.x + b.y), h * (b.y - b.x)}, t2{b.y, -b.x}, t3{h * (b.y - b.x), -h * (b.x + b.y)};
  cd v[8] = {a + b, a + t1, a + t2, a + t3, a - b, a - t1, a - t2, a - t3};
  twiddle(v, w);
  exchange(v, z + q * kPitch, j);
  dft8<false>(v);
#pragma unroll
  for (int k = 0; k < 8; ++k) z[q * kPitch + j + 8 * k] = v[k];
  __syncthreads();
  for (int i = tid; i < kFV * 16; i += kThreads) {  // rows b, b + 1 and b + 8, b + 9
    const int col = i >> 4, tr = 2 * (i & 15);
    if (first + (tr >> 3) >= kernels) continue;
    const cd* const row = z + tr * kPitch;
    const cd A = row[col], B = row[(64 - col) & 63], C = row[kPitch + col], D = row[kPitch + ((64 - col) & 63)];
    float4* const out = reinterpret_cast<float4*>(spectra + ((int64_t)col * kernels + first + (tr >> 3)) * 16 + (tr & 7));
    out[0] = make_float4((float)(0.5 * (A.x + B.x)), (float)(0.5 * (A.y - B.y)), (float)(0.5 * (C.x + D.x)), (float)(0.5 * (C.y - D.y)));
    out[4] = make_float4((float)(0.5 * (A.y + B.y)), (float)(0.5 * (B.x - A.x)), (float)(0.5 * (C.y + D.y)), (float)(0.5 * (D.x - C.x)));
  }
  if (tid == 0) largest[blockIdx.x] = max(max(wave_max[0], wave_max[1]), max(wave_max[2], wave_max[3]));
}

// db[m] = sums[m] + sums[maps + m] + ..., by a wave
__device__ __forceinline__ void add_sums(const double* sums, int count, int maps, int m, float* db) {
  if (m >= maps) return;
  double sum = 0;
  for (int i = threadIdx.x & 63; i < count; i += 64) sum += sums[(int64_t)i * maps + m];
#pragma unroll
  for (int d = 32; d > 0; d >>= 1) sum += __shfl_xor(sum, d);
  if ((threadIdx.x & 63) == 0) db[m] = (float)sum;
}

__global__ __launch_bounds__(kThreads) void taps_inverse_kernel(const float2* __restrict__ spectra, int64_t slice, int slices,
                                                                int64_t kernels, int r, int s, float* __restrict__ dw,
                                                                const double* __restrict__ sums, int sum_planes, int maps,
                                                                float* __restrict__ db, int blocks, SpectralExcept except) {
  __shared__ cd z[32 * kPitch];
  const int tid = threadIdx.x, j = tid & 7, q = tid >> 3;
  if ((int)blockIdx.x >= blocks) {  // the bias gradient
    add_sums(sums, sum_planes, maps, ((int)blockIdx.x - blocks) * 4 + (tid >> 6), db);
    return;
  }
  const uint32_t leaves = *except.declined, zeros = *except.zeros;  // (looked at where their latency is over)
  const int64_t first = (int64_t)blockIdx.x * 4;
  for (int i = tid; i < kFV * 32; i += kThreads) {
    const int col = i >> 5, tr = i & 31;
    cd lower{0, 0}, upper{0, 0};
    if (first + (tr >> 3) < kernels) {
      const float2* in = spectra + ((int64_t)col * kernels + first + (tr >> 3)) * 16 + (tr & 7);
      for (int l = 0; l < slices; ++l, in += slice) {
        const float2 f = in[0], g = in[8];
        lower = lower + cd{(double)f.x, (double)f.y}, upper = upper + cd{(double)g.x, (double)g.y};
      }
    }
    cd* const row = z + tr * kPitch;
    if (col == 0 || col == 32) {
      row[col] = {lower.x, upper.x};
    } else {
      row[col] = {lower.x - upper.y, lower.y + upper.x};
      row[64 - col] = {lower.x + upper.y, upper.x - lower.y};
    }
  }
  if (leaves) return;
  __syncthreads();
  const cd w = kRoot64[j];
  cd v[8];
#pragma unroll
  for (int k = 0; k < 8; ++k) v[k] = z[q * kPitch + j + 8 * k];
  ifft64(v, z + q * kPitch, j, w);
  const int64_t kernel = first + (q >> 3);
  if (kernel >= kernels) return;
#pragma unroll
  for (int half = 0; half < 2; ++half) {
    const int y = (q & 7) + 8 * half;
    const uint64_t zero = zeros ? except.zero[y] : 0;
#pragma unroll
    for (int i = 0; i < 2; ++i) {
      const int x = j + 8 * i;
      if (y < r && x < s) dw[(kernel * r + y) * s + x] = zero >> x & 1 ? 0.f : (float)((half ? v[i].y : v[i].x) * (1.0 / 4096));
    }
  }
}

// ---- lines -------------------------------------------------------------------------------------------------------
// 256 points as 16 x 16: sixteen threads a transform, two real lines each; 32 lines a block.
//
// The two lines of a transform may belong to two images, channels or maps of any magnitudes, and double keeps 53 bits of
// the larger one: each is scaled by a power of two to its own largest value first (exactly, and back as exactly), so that
// nothing of one shows in the other's spectrum; a line with an infinity or NaN takes part as zeros (its image, or the whole
// kernel gradient, is declined).
// e^(-2 pi i j / 256), j < 16
__device__ const cd kRoot256[16] = {{1.0, -0.0},
                                    {0.99969881869620422012, -0.02454122852291228803},
                                    {0.99879545620517239271, -0.04906767432741801426},
                                    {0.99729045667869021614, -0.07356456359966742352},
                                    {0.99518472667219688624, -0.09801714032956060199},
                                    {0.99247953459870999816, -0.12241067519921619849},
                                    {0.98917650996478097345, -0.14673047445536175166},
                                    {0.98527764238894124477, -0.17096188876030122636},
                                    {0.98078528040323044913, -0.19509032201612826785},
                                    {0.97570213003852854446, -0.21910124015686979722},
                                    {0.97003125319454399260, -0.24298017990326388994},
                                    {0.96377606579543986669, -0.26671275747489838633},
                                    {0.95694033573220886494, -0.29028467725446236764},
                                    {0.94952818059303666720, -0.31368174039889147666},
                                    {0.94154406518302077841, -0.33688985339222005069},
                                    {0.93299279883473888771, -0.35989503653498814878}};
__device__ __forceinline__ void twiddle(cd (&v)[16], cd w) {
  cd p[16];
  p[1] = w;
#pragma unroll
  for (int k = 2; k < 16; ++k) p[k] = p[k / 2] * p[k - k / 2];
#pragma unroll
  for (int k = 1; k < 16; ++k) v[k] = v[k] * p[k];
}
__device__ __forceinline__ void exchange(cd (&v)[16], cd* row, int j) {
  wave_sync();
#pragma unroll
  for (int k = 0; k < 16; ++k) row[k * 16 + (j ^ k)] = v[k];
  wave_sync();
#pragma unroll
  for (int i = 0; i < 16; ++i) v[i] = row[j * 16 + (i ^ j)];
  wave_sync();
}

// Where a line comes from and where its spectrum goes.
struct Line {
  int64_t at;      // of its first sample (before the tile's offset) in the tensor
  int64_t plane;   // index of its spectrum
  int64_t group;   // index of the lines of all channels it is one of
  int64_t cell;    // group by group
  int channel, start, image;
};
__device__ __forceinline__ Line line_of(const SpectralLines& t, unsigned id) {
  Line l;
  const unsigned rows = id / t.tiles, maps = rows / t.others;
  const int tile = id % t.tiles, o = rows % t.others, c = maps % t.count;
  const int64_t n = maps / t.count;
  l.at = (n * t.channels + t.first + c) * t.s_channel + o * t.s_other;
  l.plane = n * t.p_image + c * t.p_channel + (int64_t)o * t.tiles + tile;
  l.group = (n * t.others + o) * t.tiles + tile;
  l.cell = l.group * t.count + c;
  l.channel = t.first + c, l.start = tile * t.step, l.image = (int)n;
  return l;
}

struct LineArgs {
  LineJob job[2];
  int first_blocks;  // blocks of the first job
  int blocks;        // of both; another one decides
  MeetDecision decide;
};

template <typename T>
__global__ __launch_bounds__(kThreads) void line_spectra_kernel(LineArgs args) {
  __shared__ cd z[16 * 256];
  __shared__ int plane_of[32];
  __shared__ double unscale_of[32];
  const int tid = threadIdx.x, j = tid & 15, q = tid >> 4;
  if ((int)blockIdx.x >= args.blocks) return decide_meeting(args.decide, reinterpret_cast<uint64_t*>(z));
  const bool second = (int)blockIdx.x >= args.first_blocks;
  const LineJob& a = args.job[second];
  const SpectralLines& t = a.t;
  const int block = blockIdx.x - (second ? args.first_blocks : 0), first = block * 32 + 2 * q, lines = (int)t.lines();
  cd v[16];
  float f[2][16];
  Line l[2];
  double scale[2], spoilt_sum[2] = {0, 0};
  bool spoilt[2];
#pragma unroll
  for (int half = 0; half < 2; ++half) {
    l[half] = line_of(t, min(first + half, lines - 1));
    if (j == half) plane_of[2 * q + half] = (int)l[half].plane;
    const int x0 = l[half].start + t.x0;
    const T* const src = (const T*)a.src + l[half].at;
    const int left = max(0, -x0), right = first + half < lines ? min(t.lim, t.len - x0) : 0;
#pragma unroll
    for (int i = 0; i < 16; ++i) {
      const int x = j + 16 * i;
      f[half][i] = ld(src + (x >= left && x < right ? (int64_t)(x0 + x) * t.s_along : 0));
    }
  }
#pragma unroll
  for (int half = 0; half < 2; ++half) {
    const int x0 = l[half].start + t.x0, left = max(0, -x0), right = first + half < lines ? min(t.lim, t.len - x0) : 0;
    uint32_t m[16];
#pragma unroll
    for (int i = 0; i < 16; ++i) {
      const int x = j + 16 * i;
      if (!(x >= left && x < right)) f[half][i] = 0.f;
      m[i] = __float_as_uint(f[half][i]) & 0x7fffffffu;
    }
    uint32_t top = 0;  // the line's largest
#pragma unroll
    for (int i = 0; i < 16; ++i) top = max(top, m[i]);
    top = max(top, moved<kMirror16>(top));
    top = max(top, moved<kMirror8>(top));
    top = max(top, moved<kSwap2>(top));
    top = max(top, moved<kSwap1>(top));
    if (a.largest && first + half < lines && j == 0) a.largest[l[half].cell] = top;
    const bool finite = top < 0x7f800000u;
    spoilt[half] = !finite;
    if (a.sums && __any(!finite)) {  // the sum of such a line as it is
      double sum = 0;
#pragma unroll
      for (int i = 0; i < 16; ++i) sum += (double)f[half][i];
#pragma unroll
      for (int d = 8; d > 0; d >>= 1) sum += __shfl_xor(sum, d);
      spoilt_sum[half] = sum;
    }
    const int exponent = max((int)(top >> 23), 1) - 127;
    scale[half] = ldexp(1.0, -exponent);
    if (j == half) unscale_of[2 * q + half] = top == 0 || !finite ? 0.0 : ldexp(1.0, exponent);
#pragma unroll
    for (int i = 0; i < 16; ++i) f[half][i] = finite ? f[half][i] : 0.f;
  }
#pragma unroll
  for (int i = 0; i < 16; ++i) v[i] = {(double)f[0][i] * scale[0], (double)f[1][i] * scale[1]};
  cd* const row = z + q * 256;
  dft16<false>(v);
  twiddle(v, kRoot256[j]);
  exchange(v, row, j);
  dft16<false>(v);
#pragma unroll
  for (int k = 0; k < 16; ++k) row[j + 16 * k] = v[k];
  __syncthreads();
  if (a.sums && j == 0) {
    if (first < lines) a.sums[l[0].cell] = spoilt[0] ? spoilt_sum[0] : v[0].x * unscale_of[2 * q];
    if (first + 1 < lines) a.sums[l[1].cell] = spoilt[1] ? spoilt_sum[1] : v[0].y * unscale_of[2 * q + 1];
  }
  const int slot = tid & 127;
#pragma unroll 2
  for (int m = 0; m < 8; ++m) {
    const int tr = (tid >> 7) + 2 * m;
    const cd A = z[tr * 256 + slot], B = z[tr * 256 + (slot == 0 ? 128 : 256 - slot)];
    const double ua = unscale_of[2 * tr], ub = unscale_of[2 * tr + 1], ha = 0.5 * ua, hb = 0.5 * ub;
    const float2 lower = slot == 0 ? make_float2((float)(ua * A.x), (float)(ua * B.x)) : make_float2((float)(ha * (A.x + B.x)), (float)(ha * (A.y - B.y)));
    const float2 upper = slot == 0 ? make_float2((float)(ub * A.y), (float)(ub * B.y)) : make_float2((float)(hb * (A.y + B.y)), (float)(hb * (B.x - A.x)));
    const int id = block * 32 + 2 * tr;
    if (id < lines) a.spectra[((slot >> 6) * a.planes + plane_of[2 * tr]) * 64 + (slot & 63)] = lower;
    if (id + 1 < lines) a.spectra[((slot >> 6) * a.planes + plane_of[2 * tr + 1]) * 64 + (slot & 63)] = upper;
  }
}

struct LineInverseArgs {
  SpectralLines t;
  const float2* spectra;
  int64_t slice, lines, planes;
  int slices, blocks;
  void* dst;
  const float* bias;
  int relu;
  const double* sums;
  int sum_planes, maps;
  float* db;
  SpectralExcept except;
};

template <typename T>
__global__ __launch_bounds__(kThreads) void line_inverse_kernel(LineInverseArgs a) {
  __shared__ cd z[16 * 256];
  const int tid = threadIdx.x, j = tid & 15, q = tid >> 4;
  const SpectralLines& t = a.t;
  if ((int)blockIdx.x >= a.blocks) return add_sums(a.sums, a.sum_planes, a.maps, ((int)blockIdx.x - a.blocks) * 4 + (tid >> 6), a.db);
  __shared__ int plane_of[32];
  __shared__ uint32_t top_of[4][16];
  const uint32_t zeros = a.except.zero ? *a.except.zeros : 0;
  const int lines = (int)a.lines;
  if (tid < 32) plane_of[tid] = (int)line_of(t, min((int)blockIdx.x * 32 + tid, lines - 1)).plane;
  __syncthreads();
  const int slot = tid & 127;
  cd A[8], B[8];  // of the lines 2 tr and 2 tr + 1, tr = tid / 128 + 2 m
#pragma unroll
  for (int m = 0; m < 8; ++m) A[m] = B[m] = {0, 0};
  for (int s = 0; s < a.slices; ++s)
#pragma unroll
    for (int m = 0; m < 8; ++m) {
      const int tr = (tid >> 7) + 2 * m;
      const float2* const in = a.spectra + s * a.slice + (slot >> 6) * a.planes * 64 + (slot & 63);
      const float2 f = in[(int64_t)plane_of[2 * tr] * 64], g = in[(int64_t)plane_of[2 * tr + 1] * 64];
      A[m] = A[m] + cd{(double)f.x, (double)f.y}, B[m] = B[m] + cd{(double)g.x, (double)g.y};
    }
  {  // the largest value of each line, as the upper half of a double: half a line a wave, lane 2 m + half has that one's
    auto high = [](cd f) { return max((uint32_t)__double2hiint(f.x) & 0x7fffffffu, (uint32_t)__double2hiint(f.y) & 0x7fffffffu); };
    uint32_t t[16], b[8], c[4], e[2], top;
#pragma unroll
    for (int m = 0; m < 8; ++m) t[2 * m] = high(A[m]), t[2 * m + 1] = high(B[m]);
    keep_half<kMirror16, 8>(t, tid & 8, b);
    keep_half<kMirror8, 4>(b, tid & 4, c);
    keep_half<kSwap2, 2>(c, tid & 2, e);
    keep_half<kSwap1, 1>(e, tid & 1, &top);
    top = max(top, (uint32_t)__shfl_xor((int)top, 16));
    top = max(top, (uint32_t)__shfl_xor((int)top, 32));
    if ((tid & 63) < 16) top_of[tid >> 6][tid & 15] = top;
  }
  __syncthreads();
  auto top = [&](int tr, int half) { return max(top_of[2 * (tr & 1)][(tr & ~1) + half], top_of[2 * (tr & 1) + 1][(tr & ~1) + half]); };
  auto finite = [&](uint32_t high) { return high < 0x7ff00000u; };
  auto exponent = [&](uint32_t high) { return (int)(high >> 20) - 1023; };  // (sums of floats: never that of a denormal double)
#pragma unroll
  for (int m = 0; m < 8; ++m) {
    const int tr = (tid >> 7) + 2 * m;
    const uint32_t ta = top(tr, 0), tb = top(tr, 1);
    const double sa = ta ? ldexp(1.0, -exponent(ta)) : 0.0, sb = tb ? ldexp(1.0, -exponent(tb)) : 0.0;
    const cd lower = finite(ta) ? cd{sa * A[m].x, sa * A[m].y} : cd{0, 0}, upper = finite(tb) ? cd{sb * B[m].x, sb * B[m].y} : cd{0, 0};
    cd* const row = z + tr * 256;
    if (slot == 0) {
      row[0] = {lower.x, upper.x}, row[128] = {lower.y, upper.y};
    } else {
      row[slot] = {lower.x - upper.y, lower.y + upper.x};
      row[256 - slot] = {lower.x + upper.y, upper.x - lower.y};
    }
  }
  __syncthreads();
  cd* const row = z + q * 256;
  cd v[16];
#pragma unroll
  for (int k = 0; k < 16; ++k) v[k] = row[j + 16 * k];
  dft16<true>(v);
  twiddle(v, conj(kRoot256[j]));
  exchange(v, row, j);
  dft16<true>(v);
#pragma unroll
  for (int half = 0; half < 2; ++half) {
    const int id = blockIdx.x * 32 + 2 * q + half;
    if (id >= lines) continue;
    const Line l = line_of(t, id);
    if (a.except.declined && a.except.declined[a.except.per_image ? l.image : 0]) continue;
    T* const dst = (T*)a.dst + l.at;
    const float bias = a.bias ? a.bias[l.channel] : 0.f;
    const uint32_t high = top(q, half);
    const double unscale = high && finite(high) ? ldexp(1.0 / 256, exponent(high)) : 0.0;
    uint64_t zero[4];
#pragma unroll
    for (int k = 0; k < 4; ++k) zero[k] = zeros ? a.except.zero[(a.except.per_image ? l.group * 4 : 0) + k] >> j : 0;
#pragma unroll
    for (int i = 0; i < 16; ++i) {
      const int lx = j + 16 * i - t.x0, x = l.start + lx;
      if (lx < 0 || lx >= t.lim || x >= t.len) continue;
      float r = zero[i >> 2] >> 16 * (i & 3) & 1 ? bias : (float)((half ? v[i].y : v[i].x) * unscale + (double)bias);
      if (a.relu) r = fmaxf(r, 0.f);
      st(dst + (int64_t)x * t.s_along, r);
    }
  }
}

// ---- launches ----------------------------------------------------------------------------------------------------
vcnn_status launch_plane_spectra(const SpectralTiles& t, int dtype, const void* src, float2* spectra, double* sums,
                                 const uint32_t* declined, int per_image, const MeetDecision& decide, hipStream_t st) {
  PlaneArgs a{t, src, spectra, sums, declined, per_image, t.planes(), decide};
  const dim3 grid((unsigned)(a.planes + (decide.partial ? 1 : 0)));
  if (dtype == VCNN_BF16) hipLaunchKernelGGL(plane_spectra_kernel<bf16>, grid, dim3(kThreads), 0, st, a);
  else hipLaunchKernelGGL(plane_spectra_kernel<float>, grid, dim3(kThreads), 0, st, a);
  return check_launch("plane_spectra");
}
vcnn_status launch_plane_inverse(const SpectralTiles& t, int dtype, const float2* spectra, int64_t slice, int slices, void* dst,
                                 const float* bias, int relu, const SpectralExcept& except, hipStream_t st) {
  InverseArgs a{t, except, spectra, slice, t.planes(), slices, dst, bias, relu};
  if (dtype == VCNN_BF16) hipLaunchKernelGGL(plane_inverse_kernel<bf16>, dim3((unsigned)a.planes), dim3(kThreads), 0, st, a);
  else hipLaunchKernelGGL(plane_inverse_kernel<float>, dim3((unsigned)a.planes), dim3(kThreads), 0, st, a);
  return check_launch("plane_inverse");
}
vcnn_status launch_taps_spectra(int dtype, const void* w, int64_t kernels, int r, int s, float2* spectra, uint32_t* largest,
                                hipStream_t st) {
  const dim3 grid((unsigned)ceil_div(kernels, 4));
  if (dtype == VCNN_BF16)
    hipLaunchKernelGGL(taps_spectra_kernel<bf16>, grid, dim3(kThreads), 0, st, (const bf16*)w, kernels, r, s, spectra, largest);
  else hipLaunchKernelGGL(taps_spectra_kernel<float>, grid, dim3(kThreads), 0, st, (const float*)w, kernels, r, s, spectra, largest);
  return check_launch("taps_spectra");
}
vcnn_status launch_taps_inverse(const float2* spectra, int64_t slice, int slices, int64_t kernels, int r, int s, float* dw,
                                const double* sums, int sum_planes, int maps, float* db, const SpectralExcept& except, hipStream_t st) {
  const int blocks = (int)ceil_div(kernels, 4);
  hipLaunchKernelGGL(taps_inverse_kernel, dim3((unsigned)(blocks + (db ? ceil_div(maps, 4) : 0))), dim3(kThreads), 0, st,
                     spectra, slice, slices, kernels, r, s, dw, sums, sum_planes, maps, db, blocks, except);
  return check_launch("taps_inverse");
}

vcnn_status launch_line_spectra(int dtype, const LineJob& first, const LineJob& second, const MeetDecision& decide, hipStream_t st) {
  LineArgs a{{first, second}, (int)ceil_div(first.t.lines(), 32), 0, decide};
  a.blocks = (int)(a.first_blocks + ceil_div(second.t.lines(), 32));
  const dim3 grid((unsigned)(a.blocks + (decide.partial ? 1 : 0)));
  if (dtype == VCNN_BF16) hipLaunchKernelGGL(line_spectra_kernel<bf16>, grid, dim3(kThreads), 0, st, a);
  else hipLaunchKernelGGL(line_spectra_kernel<float>, grid, dim3(kThreads), 0, st, a);
  return check_launch("line_spectra");
}
vcnn_status launch_line_inverse(const SpectralLines& t, int64_t planes, int dtype, const float2* spectra, int64_t slice, int slices,
                                void* dst, const float* bias, int relu, const double* sums, int sum_planes, int maps, float* db,
                                const SpectralExcept& except, hipStream_t st) {
  LineInverseArgs a{t, spectra, slice, t.lines(), planes, slices, (int)ceil_div(t.lines(), 32), dst, bias, relu, sums, sum_planes, maps, db, except};
  const dim3 grid((unsigned)(a.blocks + (db ? ceil_div(maps, 4) : 0)));
  if (dtype == VCNN_BF16) hipLaunchKernelGGL(line_inverse_kernel<bf16>, grid, dim3(kThreads), 0, st, a);
  else hipLaunchKernelGGL(line_inverse_kernel<float>, grid, dim3(kThreads), 0, st, a);
  return check_launch("line_inverse");
}

}  // namespace vcnn
