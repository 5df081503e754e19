// Complex arithmetic and short transforms in registers, for the passes through the Fourier domain.
#pragma once
#include <hip/hip_runtime.h>

#include <cstdint>

namespace vcnn {

template <typename T>
struct cx {
  T x, y;
};
typedef cx<double> cd;
typedef cx<float> cf;
template <typename T>
__device__ __forceinline__ cx<T> operator+(cx<T> a, cx<T> b) { return {a.x + b.x, a.y + b.y}; }
template <typename T>
__device__ __forceinline__ cx<T> operator-(cx<T> a, cx<T> b) { return {a.x - b.x, a.y - b.y}; }
template <typename T>
__device__ __forceinline__ cx<T> operator*(cx<T> a, cx<T> b) {
  return {__builtin_elementwise_fma(a.x, b.x, -a.y * b.y), __builtin_elementwise_fma(a.x, b.y, a.y * b.x)};
}
template <typename T>
__device__ __forceinline__ cx<T> conj(cx<T> a) { return {a.x, -a.y}; }
// a * (-i) forward, a * i inverse
template <bool INV, typename T>
__device__ __forceinline__ cx<T> turn(cx<T> a) { return INV ? cx<T>{-a.y, a.x} : cx<T>{a.y, -a.x}; }

template <bool INV, typename T>
__device__ __forceinline__ void dft4(cx<T>& a, cx<T>& b, cx<T>& c, cx<T>& d) {
  const cx<T> s = a + c, t = a - c, u = b + d, q = turn<INV>(b - d);
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
// v[4 k + i], i < 4, hold what first(v, i) makes of v[i + 4 n]; second(v, k) then leaves point k + 4 n of
// sum_m v[m] e^(-+ 2 pi i m p / 16) in v[4 k + n]
template <bool INV, typename T>
__device__ __forceinline__ void dft16_first(cx<T> (&v)[16], int i) {
  constexpr double c1 = 0.92387953251128675613, s1 = 0.38268343236508977173, h = 0.70710678118654752440;
  constexpr double c[10] = {1, c1, h, s1, 0, 0, -h, 0, 0, -c1}, s[10] = {0, s1, h, c1, 1, 0, h, 0, 0, -s1};
  dft4<INV>(v[i], v[4 + i], v[8 + i], v[12 + i]);
  if (i > 0) {
#pragma unroll
    for (int k = 1; k < 4; ++k) v[4 * k + i] = v[4 * k + i] * cx<T>{(T)c[i * k], (T)(INV ? s[i * k] : -s[i * k])};
  }
}
template <bool INV, typename T>
__device__ __forceinline__ void dft16_second(cx<T> (&v)[16], int k) { dft4<INV>(v[4 * k], v[4 * k + 1], v[4 * k + 2], v[4 * k + 3]); }
__device__ __forceinline__ constexpr int dft16_at(int p) { return 4 * (p & 3) + (p >> 2); }  // where point p is
// The same with the points in order.
template <bool INV, typename T>
__device__ __forceinline__ void dft16(cx<T> (&v)[16]) {
  cx<T> t[16];
#pragma unroll
  for (int i = 0; i < 4; ++i) dft16_first<INV>(v, i);
#pragma unroll
  for (int i = 0; i < 4; ++i) dft16_second<INV>(v, i);
#pragma unroll
  for (int i = 0; i < 16; ++i) t[i] = v[dft16_at(i)];
#pragma unroll
  for (int i = 0; i < 16; ++i) v[i] = t[i];
}

// Orders a wave's LDS accesses among its lanes (they execute in program order).
__device__ __forceinline__ void wave_sync() {
  __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
  __builtin_amdgcn_wave_barrier();
}

// A value from another lane of the same 16: one instruction of the vector units, where a general shuffle goes through LDS.
template <int CTRL>
__device__ __forceinline__ uint32_t moved(uint32_t v) { return (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, CTRL, 0xf, 0xf, true); }
static constexpr int kMirror16 = 0x140, kMirror8 = 0x141, kSwap2 = 0x4e, kSwap1 = 0xb1;  // lane ^ 15, ^ 7, ^ 2, ^ 1
// Of v[0 .. 2 N - 1] each lane keeps the half its bit chooses, the larger of its own and of the lane across.
template <int CTRL, int N>
__device__ __forceinline__ void keep_half(const uint32_t* v, bool up, uint32_t* out) {
#pragma unroll
  for (int i = 0; i < N; ++i) out[i] = max(up ? v[i + N] : v[i], moved<CTRL>(up ? v[i] : v[i + N]));
}

}  // namespace vcnn
