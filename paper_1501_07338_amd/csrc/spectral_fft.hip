// Real planes of 64 x 64 pixels to their spectra and back, in double (spectral.h).
//
// A transform of 64 points is 8 x 8: thread j of eight holds points j + 8 i, transforms over i, multiplies by the twiddles,
// hands values over in LDS (its own wave's: no barrier) and transforms again, which leaves it points k1 + 8 k2 of the
// result.  Two real rows share one complex transform, as its real and imaginary part.  One block of 256 threads does a
// plane: 32 pairs of rows, a transposition through LDS (one barrier on either side), 32 columns (the real columns 0 and 32
// share one).  Double costs the vector units no more than float and the LDS traffic twice as much; the kernels are bound by
// the memory the spectra take.
#include "elem.h"
#include "spectral.h"

namespace vcnn {

static constexpr int kThreads = 256;
static constexpr int kPitch = 65;  // of a row of 64 complex doubles in LDS: eight rows 16 bytes apart in their banks

struct cd {
  double x, y;
};
__device__ __forceinline__ cd operator+(cd a, cd b) { return {a.x + b.x, a.y + b.y}; }
__device__ __forceinline__ cd operator-(cd a, cd b) { return {a.x - b.x, a.y - b.y}; }
__device__ __forceinline__ cd operator*(cd a, cd b) { return {fma(a.x, b.x, -a.y * b.y), fma(a.x, b.y, a.y * b.x)}; }
__device__ __forceinline__ cd conj(cd a) { return {a.x, -a.y}; }
// a * (-i) forward, a * i inverse
template <bool INV>
__device__ __forceinline__ cd turn(cd a) { return INV ? cd{-a.y, a.x} : cd{a.y, -a.x}; }

template <bool INV>
__device__ __forceinline__ void dft4(cd& a, cd& b, cd& c, cd& d) {
  const cd s = a + c, t = a - c, u = b + d, q = turn<INV>(b - d);
  a = s + u, b = t + q, c = s - u, d = t - q;
}
// v[k] = sum_n v[n] e^(-+ 2 pi i n k / 8)
template <bool INV>
__device__ __forceinline__ void dft8(cd (&v)[8]) {
  constexpr double h = 0.70710678118654752440;
  cd a[4], b[4];
#pragma unroll
  for (int i = 0; i < 4; ++i) a[i] = v[i] + v[i + 4], b[i] = v[i] - v[i + 4];
  const cd t1 = turn<INV>(b[1]), t3 = turn<INV>(b[3]);
  b[1] = {h * (b[1].x + t1.x), h * (b[1].y + t1.y)};
  b[2] = turn<INV>(b[2]);
  b[3] = {h * (t3.x - b[3].x), h * (t3.y - b[3].y)};
  dft4<INV>(a[0], a[1], a[2], a[3]);
  dft4<INV>(b[0], b[1], b[2], b[3]);
#pragma unroll
  for (int i = 0; i < 4; ++i) v[2 * i] = a[i], v[2 * i + 1] = b[i];
}

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
// Orders a wave's LDS accesses among its lanes (they execute in program order).
__device__ __forceinline__ void wave_sync() {
  __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
  __builtin_amdgcn_wave_barrier();
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

// ---- planes ------------------------------------------------------------------------------------------------------
struct PlaneArgs {
  SpectralTiles t;
  const void* src;
  float2* spectra;
  uint32_t* cells;
  double* sums;
  uint32_t* words;
  int64_t planes;
};

// The largest of v[0..7] over a wave: lane l gets that of v[((l >> 3) & 1) * 4 + (l >> 1 & 3)].  (Moves within 16 lanes cost the
// vector units one instruction; by general shuffles, of 16 values, this took 45 of 106 us on 8192 planes.)
template <int CTRL>
__device__ __forceinline__ uint32_t moved(uint32_t v) { return (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, CTRL, 0xf, 0xf, true); }
__device__ __forceinline__ uint32_t max_scatter(const uint32_t (&v)[8], int lane) {
  uint32_t a[4], b[2], c;
#pragma unroll
  for (int i = 0; i < 4; ++i) {  // row_mirror: lane ^ 15
    const uint32_t keep = lane & 8 ? v[i + 4] : v[i], give = lane & 8 ? v[i] : v[i + 4];
    a[i] = max(keep, moved<0x140>(give));
  }
#pragma unroll
  for (int i = 0; i < 2; ++i) {  // row_half_mirror: lane ^ 7
    const uint32_t keep = lane & 4 ? a[i + 2] : a[i], give = lane & 4 ? a[i] : a[i + 2];
    b[i] = max(keep, moved<0x141>(give));
  }
  const uint32_t keep = lane & 2 ? b[1] : b[0], give = lane & 2 ? b[0] : b[1];
  c = max(keep, moved<0x4e>(give));  // lane ^ 2
  c = max(c, moved<0xb1>(c));        // lane ^ 1
  c = max(c, (uint32_t)__shfl_xor((int)c, 16));
  return max(c, (uint32_t)__shfl_xor((int)c, 32));
}

template <typename T>
__global__ __launch_bounds__(kThreads) void plane_spectra_kernel(PlaneArgs a) {
  __shared__ cd z[32 * kPitch];
  const int tid = threadIdx.x, j = tid & 7, q = tid >> 3;
  const int64_t p = blockIdx.x;
  const SpectralTiles& t = a.t;
  const int c = (int)(p % t.count), tx = (int)(p / t.count % t.tiles_x), ty = (int)(p / t.count / t.tiles_x % t.tiles_y);
  const int64_t n = p / t.count / t.tiles_x / t.tiles_y;
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
#pragma unroll
  for (int half = 0; half < 2; ++half)  // (all loads in flight before the first is looked at)
#pragma unroll
    for (int i = 0; i < 8; ++i) {
      const int ly = q + 32 * half, lx = j + 8 * i;
      if (!(ly >= top && ly < bottom && lx >= left && lx < right)) (half ? hi : lo)[i] = 0.f;
    }
  if (a.words && p == 0 && tid < 2) a.words[tid] = 0;
  const cd w = kRoot64[j];
  cd v[8];
#pragma unroll
  for (int i = 0; i < 8; ++i) v[i] = {(double)lo[i], (double)hi[i]};
  {  // wave b holds the rows of cells b (lo) and b + 4 (hi); the columns j + 16 i and j + 8 + 16 i are those of a cell
    uint32_t m[8];
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      m[i] = max(__float_as_uint(lo[2 * i]) & 0x7fffffffu, __float_as_uint(lo[2 * i + 1]) & 0x7fffffffu);
      m[i + 4] = max(__float_as_uint(hi[2 * i]) & 0x7fffffffu, __float_as_uint(hi[2 * i + 1]) & 0x7fffffffu);
    }
    const int lane = tid & 63;
    const uint32_t largest = max_scatter(m, lane);
    if (lane < 16 && (lane & 1) == 0) a.cells[p * kFCells + ((tid >> 6) + 4 * (lane >> 3)) * 4 + (lane >> 1 & 3)] = largest;
  }
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
  const SpectralTiles& t = a.t;
  const int c = (int)(p % t.count), tx = (int)(p / t.count % t.tiles_x), ty = (int)(p / t.count / t.tiles_x % t.tiles_y);
  const int64_t n = p / t.count / t.tiles_x / t.tiles_y;
  const int64_t plane = (n * t.channels + t.first + c) * ((int64_t)t.h * t.w);
  T* const dst = (T*)a.dst + plane;
  const float bias = a.bias ? a.bias[t.first + c] : 0.f;
#pragma unroll
  for (int half = 0; half < 2; ++half) {
    const int ly = q + 32 * half - t.y0, y = ty * t.step_y + ly;
    if (ly < 0 || ly >= t.lim_y || y >= t.h) continue;
#pragma unroll
    for (int i = 0; i < 8; ++i) {
      const int lx = j + 8 * i - t.x0, x = tx * t.step_x + lx;
      if (lx < 0 || lx >= t.lim_x || x >= t.w) continue;
      float r = (float)((half ? v[i].y : v[i].x) * (1.0 / 4096) + (double)bias);
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

__global__ __launch_bounds__(kThreads) void taps_inverse_kernel(const float2* __restrict__ spectra, int64_t slice, int slices,
                                                                int64_t kernels, int r, int s, float* __restrict__ dw,
                                                                const double* __restrict__ sums, int sum_planes, int maps,
                                                                float* __restrict__ db, int blocks) {
  __shared__ cd z[32 * kPitch];
  const int tid = threadIdx.x, j = tid & 7, q = tid >> 3;
  if ((int)blockIdx.x >= blocks) {  // the bias gradient
    const int m = ((int)blockIdx.x - blocks) * kThreads + tid;
    if (m >= maps) return;
    double sum = 0;
    for (int i = 0; i < sum_planes; ++i) sum += sums[(int64_t)i * maps + m];
    db[m] = (float)sum;
    return;
  }
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
  __syncthreads();
  const cd w = kRoot64[j];
  cd v[8];
#pragma unroll
  for (int k = 0; k < 8; ++k) v[k] = z[q * kPitch + j + 8 * k];
  ifft64(v, z + q * kPitch, j, w);
  const int64_t kernel = first + (q >> 3);
  if (kernel >= kernels) return;
#pragma unroll
  for (int half = 0; half < 2; ++half)
#pragma unroll
    for (int i = 0; i < 2; ++i) {
      const int y = (q & 7) + 8 * half, x = j + 8 * i;
      if (y < r && x < s) dw[(kernel * r + y) * s + x] = (float)((half ? v[i].y : v[i].x) * (1.0 / 4096));
    }
}

// ---- launches ----------------------------------------------------------------------------------------------------
vcnn_status launch_plane_spectra(const SpectralTiles& t, int dtype, const void* src, float2* spectra, uint32_t* cells, double* sums,
                                 uint32_t* words, hipStream_t st) {
  PlaneArgs a{t, src, spectra, cells, sums, words, t.planes()};
  if (dtype == VCNN_BF16) hipLaunchKernelGGL(plane_spectra_kernel<bf16>, dim3((unsigned)a.planes), dim3(kThreads), 0, st, a);
  else hipLaunchKernelGGL(plane_spectra_kernel<float>, dim3((unsigned)a.planes), dim3(kThreads), 0, st, a);
  return check_launch("plane_spectra");
}
vcnn_status launch_plane_inverse(const SpectralTiles& t, int dtype, const float2* spectra, int64_t slice, int slices, void* dst,
                                 const float* bias, int relu, hipStream_t st) {
  InverseArgs a{t, spectra, slice, t.planes(), slices, dst, bias, relu};
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
                                const double* sums, int sum_planes, int maps, float* db, hipStream_t st) {
  const int blocks = (int)ceil_div(kernels, 4);
  hipLaunchKernelGGL(taps_inverse_kernel, dim3((unsigned)(blocks + (db ? ceil_div(maps, kThreads) : 0))), dim3(kThreads), 0, st,
                     spectra, slice, slices, kernels, r, s, dw, sums, sum_planes, maps, db, blocks);
  return check_launch("taps_inverse");
}

}  // namespace vcnn
