// Convolutions through the Fourier domain: products of spectra, the passes and their plans (spectral.h).
#include <algorithm>
#include <cmath>

#include "bf16_core.h"
#include "spectral.h"
#include "spectral_math.h"

namespace vcnn {

static constexpr int kThreads = 256;

// e^(-2 pi i q / 64), q = rho * r for the residues rho < 4 and kernel rows r < 16
__constant__ const float kRoots[4][16][2] = {
#define R0 {1.f, 0.f}
#define ROOT(c, s) {c, -(s)}
    {R0, R0, R0, R0, R0, R0, R0, R0, R0, R0, R0, R0, R0, R0, R0, R0},
    {R0, ROOT(0.99518472667219688624f, 0.09801714032956060199f), ROOT(0.98078528040323044913f, 0.19509032201612826785f),
     ROOT(0.95694033573220886494f, 0.29028467725446236764f), ROOT(0.92387953251128675613f, 0.38268343236508977173f),
     ROOT(0.88192126434835502971f, 0.47139673682599764856f), ROOT(0.83146961230254523708f, 0.55557023301960222474f),
     ROOT(0.77301045336273696081f, 0.63439328416364549822f), ROOT(0.70710678118654752440f, 0.70710678118654752440f),
     ROOT(0.63439328416364549822f, 0.77301045336273696081f), ROOT(0.55557023301960222474f, 0.83146961230254523708f),
     ROOT(0.47139673682599764856f, 0.88192126434835502971f), ROOT(0.38268343236508977173f, 0.92387953251128675613f),
     ROOT(0.29028467725446236764f, 0.95694033573220886494f), ROOT(0.19509032201612826785f, 0.98078528040323044913f),
     ROOT(0.09801714032956060199f, 0.99518472667219688624f)},
    {R0, ROOT(0.98078528040323044913f, 0.19509032201612826785f), ROOT(0.92387953251128675613f, 0.38268343236508977173f),
     ROOT(0.83146961230254523708f, 0.55557023301960222474f), ROOT(0.70710678118654752440f, 0.70710678118654752440f),
     ROOT(0.55557023301960222474f, 0.83146961230254523708f), ROOT(0.38268343236508977173f, 0.92387953251128675613f),
     ROOT(0.19509032201612826785f, 0.98078528040323044913f), ROOT(0.0f, 1.0f),
     ROOT(-0.19509032201612826785f, 0.98078528040323044913f), ROOT(-0.38268343236508977173f, 0.92387953251128675613f),
     ROOT(-0.55557023301960222474f, 0.83146961230254523708f), ROOT(-0.70710678118654752440f, 0.70710678118654752440f),
     ROOT(-0.83146961230254523708f, 0.55557023301960222474f), ROOT(-0.92387953251128675613f, 0.38268343236508977173f),
     ROOT(-0.98078528040323044913f, 0.19509032201612826785f)},
    {R0, ROOT(0.95694033573220886494f, 0.29028467725446236764f), ROOT(0.83146961230254523708f, 0.55557023301960222474f),
     ROOT(0.63439328416364549822f, 0.77301045336273696081f), ROOT(0.38268343236508977173f, 0.92387953251128675613f),
     ROOT(0.09801714032956060199f, 0.99518472667219688624f), ROOT(-0.19509032201612826785f, 0.98078528040323044913f),
     ROOT(-0.47139673682599764856f, 0.88192126434835502971f), ROOT(-0.70710678118654752440f, 0.70710678118654752440f),
     ROOT(-0.88192126434835502971f, 0.47139673682599764856f), ROOT(-0.98078528040323044913f, 0.19509032201612826785f),
     ROOT(-0.99518472667219688624f, -0.09801714032956060199f), ROOT(-0.92387953251128675613f, -0.38268343236508977173f),
     ROOT(-0.77301045336273696081f, -0.63439328416364549822f), ROOT(-0.55557023301960222474f, -0.83146961230254523708f),
     ROOT(-0.29028467725446236764f, -0.95694033573220886494f)}};
#undef ROOT
#undef R0

__device__ const float4 kZeros[8] = {};

// ---- what the magnitudes decline ---------------------------------------------------------------------------------
// By all 256 threads.
__device__ __forceinline__ uint32_t block_max(uint32_t m, uint32_t* lds) {
#pragma unroll
  for (int d = 32; d > 0; d >>= 1) m = max(m, (uint32_t)__shfl_xor((int)m, d));
  __syncthreads();
  if ((threadIdx.x & 63) == 0) lds[threadIdx.x >> 6] = m;
  __syncthreads();
  return max(max(lds[0], lds[1]), max(lds[2], lds[3]));
}
// What the magnitudes of a forward pass's or input gradient's operands decline, an image each block: of the image the energies that
// the guard of windows left, of the kernels the largest element of each few.
struct RangeArgs {
  SpectralWords words;
  const double* totals;     // [image][transform]
  int transforms;
  const uint32_t* largest;
  int largest_count;
  int grow;   // bits a sum of products may gain
  int depth;  // bits of the root of the number of channels (maps) added
};
__device__ void guard_range(const RangeArgs& g, int n, uint32_t* lds) {
  // (upper halves of doubles, none negative: ordered as integers)
  uint32_t most = 0, high = 0, low = 0;
#pragma unroll 8
  for (int i = threadIdx.x; i < g.largest_count; i += kThreads) most = max(most, g.largest[i]);
#pragma unroll 4
  for (int i = threadIdx.x; i < g.transforms; i += kThreads) {
    const uint32_t t = (uint32_t)__double2hiint(g.totals[(int64_t)n * g.transforms + i]);
    high = max(high, t), low = max(low, t ? ~t : 0u);
  }
  most = block_max(most, lds), high = block_max(high, lds), low = ~block_max(low, lds);
  const int eb = (int)(most >> 23) - 127;
  bool bad = eb == 128;  // infinity or NaN
  if (most && high) {
    // Norms of transforms (the root of the energy): below 2^top, 2^bottom or more.  A transform of 4096 samples gains 12 bits over
    // its largest, one of a kernel as many; a channel of them all alike has to stay far from the least float, and its product too.
    const int top = (((int)(high >> 20) - 1023) >> 1) + 1, bottom = ((int)(low >> 20) - 1023) >> 1;
    bad |= top + eb + 24 + g.grow > 126 || top > 110 || eb > 110;
    bad |= bottom - g.depth + eb < -80 || bottom - g.depth < -90 || eb < -90;
  }
  if (bad && threadIdx.x == 0) g.words.image[n] = 1, *g.words.any = 1;
}

// ---- products of spectra -------------------------------------------------------------------------------------------
// C(row, col) = sum_z A(row, z) B(z, col) at every frequency, A conjugated or not.  A block does 16 x 16 pairs at one column
// v of the spectrum, its wave rho the frequencies u = 4 a + rho: 16 complex products per step of four z on
// v_mfma_f32_16x16x4_f32, whose operands are one float per lane - lane (row, z) needs the 16 values of ITS plane, which lie
// together (128 bytes), and nothing another lane has.  They go through a swizzled LDS buffer of the wave's own, so that eight
// lanes fetch one plane's line together (by themselves every lane would touch 64 lines per load), straight from global memory
// and one step ahead; there is no barrier in the loop.
// TAPS operands are the row spectra of kernels: the lane transforms the 16 rows in registers (double) to its wave's 16
// frequencies, so that the kernels' spectra, four times as large, never reach memory; TAPS results are transformed back the
// same way, each wave's share of the rows, added over the four waves in LDS.
// 16 38 64 64 -> 512 16 16 does 5.3 GFLOP a pass (33 us of matrix instructions) in 105 us forward, 112 kernel gradient and
// 153 input gradient (matrix cores busy 45, 43, 32 % of the cycles): bound by a step's chain of loads, LDS reads and the kernels' transforms at two waves a SIMD, by a block's
// beginning and end (10 steps of four between them) and, with 1056 blocks on 512 slots, by a last round that is nearly empty; the
// input gradient by 0.67 GB between the L2s and memory, half of it the sums put away and fetched again every 32 products.  Stored
// by every lane for itself instead of through LDS, results cost 34 us more; the kernels' transform in front of the products
// instead of between them 13.
struct ProductArgs {
  const float2* A;
  const float2* B;
  float2* C;
  int rows, cols, depth;
  int64_t a_row, a_z, b_col, b_z, c_row, c_col;  // in planes (kernels)
  int64_t a_planes, b_planes, c_planes;          // per column v
  int64_t c_slice;                               // complex values
  int columns, tiles_r, tiles_c, splits, per_split;
  int flush;                                     // (spectra as results) so many products are added in a row, then to C
  int rows_inner;                                // tiles of rows follow each other (the columns' operand is the larger one)
  int blocks;                                    // of products; further blocks look at the magnitudes (range)
  const uint32_t* declined;                      // something is ...
  int col_images;                                // ... columns of one image (0, kernel gradient: then all is)
  RangeArgs range;
};
// Whether all images of a block's 16 columns are declined.
__device__ __forceinline__ bool leave_columns(const ProductArgs& a, int tc) {
  if (!*a.declined || a.col_images == 0) return *a.declined != 0;
  const int col = min(tc * 16 + ((int)threadIdx.x & 15), a.cols - 1);
  return __all(a.range.words.image[col / a.col_images] != 0);
}

__device__ __forceinline__ float4 add4(float4 a, float4 b) { return make_float4(a.x + b.x, a.y + b.y, a.z + b.z, a.w + b.w); }

template <bool TAPS_A, bool CONJ_A, bool TAPS_C, bool LINES>
__global__ __launch_bounds__(kThreads, 2) void spectral_product_kernel(ProductArgs a) {
  __shared__ __attribute__((aligned(128))) uint4 lds[4][1024];
  if ((int)blockIdx.x >= a.blocks) return guard_range(a.range, blockIdx.x - a.blocks, reinterpret_cast<uint32_t*>(&lds[0][0]));
  const int tid = threadIdx.x, lane = tid & 63, rho = __builtin_amdgcn_readfirstlane(tid >> 6);
  // blocks that share the larger operand's planes one after the other on the same XCD (blocks are dealt to the eight in turn)
  int id = blockIdx.x;
  {
    const int whole = a.blocks / 8, rest = a.blocks % 8, xcd = id % 8;
    id = xcd * whole + min(xcd, rest) + id / 8;
  }
  const int inner = a.rows_inner ? a.tiles_r : a.tiles_c, outer = a.rows_inner ? a.tiles_c : a.tiles_r;
  const int ti = id % inner, to = id / inner % outer;
  const int tr = a.rows_inner ? ti : to, tc = a.rows_inner ? to : ti;
  if (leave_columns(a, tc)) return;
  id /= inner * outer;
  const int split = id % a.splits, v = id / a.splits;
  const int z_begin = split * a.per_split, z_end = min(a.depth, z_begin + a.per_split);
  uint4* const la = lds[rho];
  uint4* const lb = lds[rho] + 512;

  // load j of a step: lane i fetches 16 bytes of plane 8 j + i / 8, that is of row 8 (j & 1) + i / 8 and z = j / 2
  const int piece = (lane & 7) ^ (lane >> 3);
  const uint4 *pa[2], *pb[2];
#pragma unroll
  for (int h = 0; h < 2; ++h) {
    const int row = min(tr * 16 + 8 * h + (lane >> 3), a.rows - 1), col = min(tc * 16 + 8 * h + (lane >> 3), a.cols - 1);
    if (TAPS_A) pa[h] = reinterpret_cast<const uint4*>(a.A + ((int64_t)v * a.a_planes + row * a.a_row) * 16) + piece;
    else pa[h] = reinterpret_cast<const uint4*>(a.A + ((int64_t)v * a.a_planes + row * a.a_row) * 64 + rho * 16) + piece;
    pb[h] = reinterpret_cast<const uint4*>(a.B + ((int64_t)v * a.b_planes + col * a.b_col) * 64 + rho * 16) + piece;
  }
  const int64_t za = a.a_z * (TAPS_A ? 8 : 32), zb = a.b_z * 32;
  auto fetch_a = [&](int z0) {
#pragma unroll
    for (int j = 0; j < 8; ++j) {
      const int z = z0 + (j >> 1);
      load_to_lds16(z < z_end ? pa[j & 1] + z * za : reinterpret_cast<const uint4*>(kZeros) + piece, la + 64 * j);
    }
  };
  auto fetch_b = [&](int z0) {
#pragma unroll
    for (int j = 0; j < 8; ++j) load_to_lds16(pb[j & 1] + min(z0 + (j >> 1), z_end - 1) * zb, lb + 64 * j);
  };
  f32x4 re[16], im[16];
  auto clear = [&]() {
#pragma unroll
    for (int i = 0; i < 16; ++i) re[i] = f32x4{0, 0, 0, 0}, im[i] = f32x4{0, 0, 0, 0};
  };
  const float(&root)[16][2] = kRoots[rho];

  // what a lane holds: column lane % 16, rows 4 (lane / 16) + e; `more`: C holds the sums before (never those of TAPS results)
  auto put = [&](bool more) {
    const int64_t slice = (int64_t)split * a.c_slice;
    if (!TAPS_C) {
      // eight lanes a line, through the LDS of the second operand
      float4* const turn = reinterpret_cast<float4*>(lb);
      int ln = lane;
      asm volatile("" : "+v"(ln));  // (or the addresses below are kept in registers throughout the loop: 62 spilled)
      const int which = ln >> 3, unit = ln & 7;
      char* const out = reinterpret_cast<char*>(a.C + slice + (int64_t)v * a.c_planes * 64 + rho * 16);
#pragma unroll
      for (int e = 0; e < 4; ++e) {
#pragma unroll
        for (int q = 0; q < 8; ++q)
          turn[ln * 8 + (q ^ unit)] = make_float4(re[2 * q][e], im[2 * q][e], re[2 * q + 1][e], im[2 * q + 1][e]);
        __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
        __builtin_amdgcn_wave_barrier();
#pragma unroll
        for (int j = 0; j < 8; ++j) {  // the values of lane 8 j + which
          const int row = tr * 16 + 4 * (j >> 1) + e, col = tc * 16 + 8 * (j & 1) + which;
          float4 f = turn[(8 * j + which) * 8 + (unit ^ which)];
          if (row >= a.rows || col >= a.cols) continue;
          float4* const to = reinterpret_cast<float4*>(out + (unsigned)((row * (int)a.c_row + col * (int)a.c_col) * 512 + unit * 16));
          if (more) f = add4(f, *to);
          *to = f;
        }
        __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
        __builtin_amdgcn_wave_barrier();
      }
    } else {
      float4* const share = reinterpret_cast<float4*>(&lds[0][0]);
#pragma unroll
      for (int round = 0; round < 2; ++round) {
        __syncthreads();
#pragma unroll
        for (int e2 = 0; e2 < 2; ++e2) {
          cf t[16];
#pragma unroll
          for (int i = 0; i < 16; ++i) t[i] = {re[i][2 * round + e2], im[i][2 * round + e2]};
#pragma unroll
          for (int i = 0; i < 4; ++i) dft16_first<true>(t, i);
#pragma unroll
          for (int i = 0; i < 4; ++i) dft16_second<true>(t, i);
#pragma unroll
          for (int q = 0; q < 8; ++q) {
            const cf f = t[dft16_at(2 * q)] * cf{root[2 * q][0], -root[2 * q][1]};
            const cf g = t[dft16_at(2 * q + 1)] * cf{root[2 * q + 1][0], -root[2 * q + 1][1]};
            share[rho * 1024 + (e2 * 64 + lane) * 8 + (q ^ (lane & 7))] = make_float4(f.x, f.y, g.x, g.y);
          }
        }
        __syncthreads();
#pragma unroll
        for (int m = 0; m < 4; ++m) {
          const int i = tid + 256 * m, q = i & 7, ln = (i >> 3) & 63, e2 = i >> 9;
          const int row = tr * 16 + 4 * (ln >> 4) + 2 * round + e2, col = tc * 16 + (ln & 15);
          const int at = (e2 * 64 + ln) * 8 + (q ^ (ln & 7));
          const float4 s0 = share[at], s1 = share[1024 + at], s2 = share[2048 + at], s3 = share[3072 + at];
          if (row >= a.rows || col >= a.cols) continue;
          float4* const out = reinterpret_cast<float4*>(a.C + slice + ((int64_t)v * a.c_planes + row * a.c_row + col * a.c_col) * 16) + q;
          *out = add4(add4(s0, s1), add4(s2, s3));
        }
      }
    }
  };

  // an operand's 16 values out of LDS (the next step's loads land in the same place)
  auto take = [&](const uint4* from, cf (&f)[16]) {
#pragma unroll
    for (int q = 0; q < 8; ++q) {
      const float4 t = __builtin_bit_cast(float4, from[lane * 8 + (q ^ (lane & 7))]);
      f[2 * q] = {t.x, t.y}, f[2 * q + 1] = {t.z, t.w};
    }
    asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
  };
  const bool pair = LINES && v == 0 && rho == 0;  // a line's first value: two real ones
  auto multiply = [&](cf x, cf y, int i) {
    float xi = CONJ_A ? -x.y : x.y, yr = y.x, yi = y.y;
    re[i] = __builtin_amdgcn_mfma_f32_16x16x4f32(x.x, y.x, re[i], 0, 0, 0);
    if (LINES && i == 0 && pair) yr = y.y, yi = 0, xi = x.y;
    im[i] = __builtin_amdgcn_mfma_f32_16x16x4f32(x.x, yi, im[i], 0, 0, 0);
    re[i] = __builtin_amdgcn_mfma_f32_16x16x4f32(-xi, yi, re[i], 0, 0, 0);
    im[i] = __builtin_amdgcn_mfma_f32_16x16x4f32(xi, yr, im[i], 0, 0, 0);
  };
  // a part in eight of a lane's transform of 16 kernel rows to the wave's frequencies
  auto transform = [&](cf (&t)[16], int part) {
    if (part < 4) {
#pragma unroll
      for (int r = part; r < 16; r += 4) t[r] = t[r] * cf{root[r][0], root[r][1]};
      dft16_first<false>(t, part);
    } else {
      dft16_second<false>(t, part - 4);
    }
  };

  // Loads complete in order, eight per operand and step: with eight still out, all but the last operand fetched are there.
  fetch_a(z_begin);
  fetch_b(z_begin);
  cf fa[16], fb[16];
  if (TAPS_A) {
    // The next step's transform runs between this step's products: waves that did one after the other did the same thing at
    // the same time.
    cf ga[16];
    asm volatile("s_waitcnt vmcnt(8)" ::: "memory");
    take(la, fa);
    fetch_a(z_begin + 4);
#pragma unroll
    for (int q = 0; q < 8; ++q) transform(fa, q);
    asm volatile("s_waitcnt vmcnt(8)" ::: "memory");
    take(lb, fb);
    fetch_b(z_begin + 4);
    auto step = [&](int z0, cf (&xa)[16], cf (&ya)[16], bool last) {
      asm volatile("s_waitcnt vmcnt(8)" ::: "memory");
      take(la, ya);
      fetch_a(z0 + 8);
#pragma unroll
      for (int q = 0; q < 8; ++q) {
        multiply(xa[dft16_at(2 * q)], fb[2 * q], 2 * q);
        multiply(xa[dft16_at(2 * q + 1)], fb[2 * q + 1], 2 * q + 1);
        transform(ya, q);
#pragma unroll
        for (int m = 0; m < 8; ++m) {
          __builtin_amdgcn_sched_group_barrier(0x008, 1, 0);  // one matrix instruction,
          __builtin_amdgcn_sched_group_barrier(0x002, 4, 0);  // four of the vector units
        }
        __builtin_amdgcn_sched_barrier(0);
      }
      asm volatile("s_waitcnt vmcnt(8)" ::: "memory");
      take(lb, fb);
      if (!last) fetch_b(z0 + 8);  // (the sums leave through its place)
    };
    for (int z_put = z_begin; z_put < z_end; z_put += a.flush) {
      const int z_next = min(z_put + a.flush, z_end);
      clear();
      for (int z0 = z_put;;) {
        step(z0, fa, ga, z0 + 4 >= z_next);
        z0 += 4;
        if (z0 >= z_next) {
#pragma unroll
          for (int i = 0; i < 16; ++i) fa[i] = ga[i];
          break;
        }
        step(z0, ga, fa, z0 + 4 >= z_next);
        z0 += 4;
        if (z0 >= z_next) break;
      }
      put(z_put > z_begin);
      asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
      if (z_next < z_end) fetch_b(z_next + 4);
    }
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");  // (the last fetch)
  } else {
    clear();
    int z_put = z_begin;
    for (int z0 = z_begin; z0 < z_end; z0 += 4) {
      asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
      take(la, fa);
      take(lb, fb);
      const bool another = z0 + 4 < z_end, last = !another || z0 + 4 - z_put >= a.flush;
      if (another) fetch_a(z0 + 4);
      if (!last) fetch_b(z0 + 4);
#pragma unroll
      for (int i = 0; i < 16; ++i) multiply(fa[i], fb[i], i);
      if (last) {
        put(z_put > z_begin);
        if (TAPS_C || !another) break;
        asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
        fetch_b(z0 + 4);
        clear();
        z_put = z0 + 4;
      }
    }
  }
}

// ---- plans ---------------------------------------------------------------------------------------------------------
static size_t align256(size_t b) { return (b + 255) & ~(size_t)255; }

namespace {
struct Layout {  // of the workspace
  size_t image, map, taps, words, energy, energy_dy;        // offsets
  size_t zero, totals, largest, meet, sums;                 // inside words
};
}  // namespace

static bool one_tile(const ConvGeom& g) { return g.h + 2 * g.ph <= kFL && g.w + 2 * g.pw <= kFL; }
// Tiles (lines: tiles of lines) of one channel of the whole batch.
static int64_t tiles_of(const ConvGeom& g, const SpectralPlan& p, int pass) {
  if (p.along == 0) return (int64_t)g.n * p.tiles_y * p.tiles_x;
  const bool data = pass == VCNN_PASS_BWD_DATA;
  return (int64_t)g.n * p.tiles_x * (p.along == 1 ? (data ? g.h : g.oh) : (data ? g.w : g.ow));
}

// Of both operands of a kernel gradient.
static size_t energy_bytes(const ConvGeom& g) { return 8 * ((size_t)g.n * g.h * g.w + (size_t)g.N); }
// Chunks of its transforms whose energies are multiplied at each tap.
static int meet_chunks(const SpectralPlan& p, int64_t tiles) { return (int)ceil_div(tiles, ceil_div(tiles, p.along ? 256 : 64)); }

static size_t lay_out(const ConvGeom& g, int pass, const SpectralPlan& p, Layout* l) {
  const int64_t tiles = tiles_of(g, p, pass);
  l->image = 0;
  l->map = l->image + p.image_bytes;
  l->taps = l->map + p.map_bytes;
  l->words = l->taps + p.taps_bytes;
  size_t at = l->words + align256(256 + 4 * (size_t)g.n);
  auto take = [&](size_t bytes) { const size_t from = at; at += align256(bytes); return from; };
  // (energies in the place of the result's spectra: at most 32 KB for a tile, which takes 16.5 KB of them for each of more than four
  // channels or maps, lines 2 and 1 KB; a kernel gradient's are as many as its kernels)
  l->energy = l->energy_dy = pass == VCNN_PASS_FWD ? l->map : l->image;
  if (pass != VCNN_PASS_BWD_FILTER) {
    l->zero = take((size_t)tiles * (p.along ? 32 : 8 * kFL));
    l->totals = take((size_t)tiles * 8);
    l->largest = take(p.along ? (size_t)g.k * g.c * 4 : (size_t)ceil_div((int64_t)g.k * g.c, 4) * 4);
  } else {
    l->energy = p.energy_in_taps ? l->taps : take(energy_bytes(g));
    l->energy_dy = l->energy + 8 * (size_t)g.n * g.h * g.w;
    l->zero = take(16 * 8);
    l->meet = take((size_t)meet_chunks(p, tiles) * (g.r * g.s + 1) * 8);
    l->sums = take((size_t)tiles * g.k * 8);
  }
  return at;
}
static Layout layout(const ConvGeom& g, int pass, const SpectralPlan& p) {
  Layout l{};
  lay_out(g, pass, p, &l);
  return l;
}

bool spectral_plan(const ConvGeom& g, int pass, size_t budget, SpectralPlan* p) {
  if (g.c <= 4 || g.k <= 4) return false;
  const bool data = pass == VCNN_PASS_BWD_DATA, filter = pass == VCNN_PASS_BWD_FILTER;
  SpectralPlan q{};
  int64_t spectrum, taps;  // bytes of a tile's spectrum, of a kernel's
  if (g.r == 1 || g.s == 1) {
    q.along = g.r == 1 ? 1 : 2;
    const int len = q.along == 1 ? g.w : g.h, pad = q.along == 1 ? g.pw : g.ph, size = g.r * g.s, out = q.along == 1 ? g.ow : g.oh;
    if (size > kLineTaps || (q.along == 1 ? g.ph : g.pw) != 0) return false;
    const bool one = len + 2 * pad <= kLL;
    q.tiles_y = 1, q.step_y = 1;
    q.step_x = one ? kLL : kLL - size + 1;
    q.tiles_x = one ? 1 : (int)ceil_div(data ? len : out, q.step_x);
    spectrum = taps = kLV * kFL * 8;
  } else {
    if (g.r > kFTaps || g.s > kFTaps) return false;
    if (one_tile(g)) {
      q.tiles_y = q.tiles_x = 1;
      q.step_y = q.step_x = kFL;
    } else {
      q.step_y = kFL - g.r + 1, q.step_x = kFL - g.s + 1;
      q.tiles_y = (int)ceil_div(data ? g.h : g.oh, q.step_y), q.tiles_x = (int)ceil_div(data ? g.w : g.ow, q.step_x);
    }
    spectrum = (int64_t)kFV * kFL * 8, taps = (int64_t)kFV * kFTaps * 8;
  }
  const int columns = q.along ? kLV : kFV;
  const int64_t tiles = tiles_of(g, q, pass);
  if (tiles * std::max(g.c, g.k) > (1 << 21) || (int64_t)g.c * g.k > (1 << 21)) return false;
  const size_t image = align256((size_t)(tiles * g.c * spectrum));
  const double rows = data ? g.c : g.k, cols = filter ? (double)g.c : (double)tiles, depth = filter ? (double)tiles : (data ? g.k : g.c);
  // No sum is longer than 32 complex products, 64 roundings of the float instruction (as one of 512, an input gradient over
  // 512 maps has an error of 4.6e-7, over 64 of 2.1e-7, the two-term product 1.9e-7): a block of an input gradient takes two
  // of them, a kernel gradient's sums are cut into slices, which the inverse transform adds in double.  A forward pass's
  // slices would be as large as its result; its blocks take every channel, and up to 64 in one sum.  An input gradient over fewer
  // maps competes with a transposed product whose own sums are shorter, and takes 16: the line lies where the two errors meet.
  // 16 38 64 64 -> k 16 16, error of that product / of sums of 32 (time of the pass) / of 16, in 1e-7: 96 maps 1.38 / 1.69 (112 us) / 1.38 (126),
  // 200 1.52 / 1.67 (156) / 1.37 (172), 300 1.66 / 1.67 (175) / 1.38 (199), 340 1.71 / 1.52 (202) / 1.39 (227), 400 1.77 / 1.60 (230)
  // / 1.40 (265), 512 1.89 / 1.61 (296) / 1.41 (348).  (Four more shapes, whose other routes have 2.8e-7 and more: 1.4 to 1.8 with 32, 1.2 to 1.6 with 16.)
  const int most = data || (filter && q.along) ? 64 : (filter ? 32 : 1 << 30);
  q.per_split = (int)std::min<double>(depth, most);
  if (data) {
    // where slices of 64 are more blocks than two for each CU, as few slices as fill those (16 38 64 64 -> 512 16 16: 792 blocks
    // in two rounds 165 us, 495 in one 105 us)
    const double blocks = columns * std::ceil(rows / 16) * std::ceil(cols / 16);
    if (blocks * std::ceil(depth / 64) > 512) q.per_split = (int)(std::ceil(depth / std::max(1.0, std::floor(512 / blocks)) / 4) * 4);
    q.per_split = (int)std::min<double>(depth, q.per_split);
  }
  q.splits = (int)std::ceil(depth / q.per_split);
  const int longest = q.along == 0 && pass == VCNN_PASS_FWD && g.c <= 64 ? 64 : (q.along == 0 && data && g.k < 320 ? 16 : 32);
  q.flush = (int)(ceil_div(ceil_div(q.per_split, ceil_div(q.per_split, longest)), 4) * 4);  // in chunks of about the same size
  q.part = g.k;
  q.image_bytes = image * (data ? q.splits : 1);
  q.taps_bytes = align256((size_t)((int64_t)g.k * g.c * taps)) * (filter ? q.splits : 1);
  q.map_bytes = align256((size_t)(tiles * g.k * spectrum));
  q.energy_in_taps = filter && energy_bytes(g) <= q.taps_bytes;
  SpectralPlan none = q;
  none.image_bytes = none.map_bytes = none.taps_bytes = 0;
  Layout l{};
  q.words_bytes = lay_out(g, pass, none, &l);
  if (pass == VCNN_PASS_FWD && q.image_bytes + q.map_bytes + q.taps_bytes + q.words_bytes > budget) {
    // as many maps at once as the budget holds, in whole tiles of 16
    int64_t maps = ceil_div(g.k, 16) * 16;
    do {
      maps -= 16;
      if (maps < 16) return false;
      q.part = (int)(ceil_div(ceil_div(g.k, 16), ceil_div(g.k, maps)) * 16);
      q.map_bytes = align256((size_t)(tiles * q.part * spectrum));
      q.taps_bytes = align256((size_t)((int64_t)q.part * g.c * taps));
    } while (q.image_bytes + q.map_bytes + q.taps_bytes + q.words_bytes > budget);
  }
  q.workspace_bytes = q.image_bytes + q.map_bytes + q.taps_bytes + q.words_bytes;
  if (q.workspace_bytes > budget) return false;
  // What the transforms read and write at 4.4 TB/s (the image spectra again for each part of a forward pass), and the products: blocks
  // of so many steps of four, two of them resident on each of 256 CUs at 2.7 us a step (3.4 where the larger operand is read
  // by every block; one alone 2.2 us), four steps' worth to begin and to end with; of that a share as fitted below; the scan of the energies, and 9 us for the guard
  // and for the launches of each part.  (229 passes of drawn layers, 40 us to 1.8 ms, with the launches behind: 0.9 to 1.1 times this in eight
  // of ten.)
  const double parts = (double)ceil_div(g.k, q.part), e = 4, x_pixels = (double)g.n * g.c * g.h * g.w, y_pixels = (double)g.n * g.k * g.P;
  const double result = data ? (double)image : (filter ? (double)g.k * g.c * taps : (double)tiles * g.k * spectrum), flushes = std::ceil(q.per_split / (double)q.flush) - 1;
  const double bytes = (x_pixels + y_pixels) * e + 2.0 * (double)(q.image_bytes + (size_t)(tiles * g.k * spectrum)) + 2.0 * flushes * result * q.splits * 0.75 +
                       2.0 * (double)g.k * g.c * taps * (filter ? q.splits : 1) + (double)g.M * g.K * e + (parts - 1) * (double)image;
  const double blocks = columns * std::ceil((data ? rows : (double)std::min<int64_t>(q.part, g.k)) / 16) * std::ceil(cols / 16) * q.splits, steps = std::ceil(q.per_split / 4.0) + 4;
  const double product = parts * (blocks <= 256 ? 2.2e-6 : std::ceil(blocks / 512) * (data ? 3.4e-6 : 2.7e-6)) * steps;
  const double share = filter ? (q.along ? 0.85 : 0.7) : (data ? (q.along ? 0.9 : 0.82) : (q.along ? 0.92 : 0.87));
  const double scanned = (filter ? x_pixels + y_pixels : (data ? y_pixels : x_pixels)) * e;
  q.est_seconds = share * (bytes / 4.4e12 + product) + scanned / 4e12 + 9e-6 * (1 + parts);
  *p = q;
  return true;
}

// ---- passes --------------------------------------------------------------------------------------------------------
template <bool TAPS_A, bool CONJ_A, bool TAPS_C, bool LINES>
static vcnn_status launch_product(ProductArgs a, int images, hipStream_t st) {  // (images: whose magnitudes are looked at)
  a.columns = LINES ? kLV : kFV;
  a.tiles_r = (int)ceil_div(a.rows, 16), a.tiles_c = (int)ceil_div(a.cols, 16);
  a.blocks = a.columns * a.tiles_r * a.tiles_c * a.splits;
  hipLaunchKernelGGL((spectral_product_kernel<TAPS_A, CONJ_A, TAPS_C, LINES>), dim3((unsigned)(a.blocks + images)), dim3(kThreads), 0, st, a);
  return check_launch("spectral_product");
}

static int bits_of(int64_t n) { return (int)std::ceil(std::log2((double)std::max<int64_t>(n, 1))); }

static SpectralTiles tiles_for(const ConvGeom& g, const SpectralPlan& p, int channels, int h, int w) {
  SpectralTiles t{};
  t.images = g.n, t.channels = channels, t.first = 0, t.count = channels;
  t.h = h, t.w = w;
  t.tiles_y = p.tiles_y, t.tiles_x = p.tiles_x, t.step_y = p.step_y, t.step_x = p.step_x;
  t.lim_y = t.lim_x = kFL;
  return t;
}
static SpectralWords words_at(void* workspace, const Layout& l) {
  uint32_t* const w = (uint32_t*)((char*)workspace + l.words);
  return {w, w + 2, w + 64};
}
// The guard of a forward pass's or input gradient's windows, and that of the magnitudes.
static WindowGuard window_guard(const ConvGeom& g, int pass, int dtype, const Layout& l, int samples, void* workspace) {
  const double share = (dtype == VCNN_BF16 ? kDarkBf16 : 1.0) / samples;
  return {(const double*)((char*)workspace + l.energy), pass == VCNN_PASS_BWD_DATA, kDarkMean * share, kDarkLeast * share,
          (uint64_t*)((char*)workspace + l.zero), (double*)((char*)workspace + l.totals), words_at(workspace, l)};
}
static RangeArgs range_guard(const ConvGeom& g, int pass, const SpectralPlan& p, const Layout& l, const void* workspace) {
  RangeArgs r{};
  r.words = words_at(const_cast<void*>(workspace), l);
  r.totals = (const double*)((const char*)workspace + l.totals), r.transforms = (int)(tiles_of(g, p, pass) / g.n);
  r.largest = (const uint32_t*)((const char*)workspace + l.largest);
  r.largest_count = (int)(p.along ? (int64_t)g.k * g.c : ceil_div((int64_t)g.k * g.c, 4));
  const int64_t depth = pass == VCNN_PASS_FWD ? g.c : g.k;
  r.grow = bits_of(depth * g.r * g.s), r.depth = (bits_of(depth) + 1) / 2;
  return r;
}
static MeetGuard meet_guard(const ConvGeom& g, const SpectralPlan& p, const Layout& l, void* workspace) {
  char* const ws = (char*)workspace;
  const int64_t tiles = tiles_of(g, p, VCNN_PASS_BWD_FILTER);
  MeetGuard m{};
  m.x = (const double*)(ws + l.energy), m.dy = (const double*)(ws + l.energy_dy);
  m.chunks = meet_chunks(p, tiles), m.per_chunk = (int)ceil_div(tiles, m.chunks), m.partial = (double*)(ws + l.meet);
  m.depth_x = (bits_of(g.c) + 1) / 2, m.depth_dy = (bits_of(g.k) + 1) / 2;
  m.words = words_at(workspace, l);
  return m;
}
static MeetDecision meet_decision(const ConvGeom& g, const SpectralPlan& p, const Layout& l, const MeetGuard& m, void* workspace) {
  return {m.partial, m.chunks, g.r, g.s, kDarkMeet / (p.along ? kLL : kFL * kFL), bits_of(g.N), (uint64_t*)((char*)workspace + l.zero), m.words};
}
static vcnn_status scan_both(const ConvGeom& g, int dtype, const Layout& l, const void* x, const void* dy, void* workspace, hipStream_t st) {
  char* const ws = (char*)workspace;
  return launch_energies(dtype, g.n, {x, g.c, (int64_t)g.h * g.w, (double*)(ws + l.energy)}, {dy, g.k, g.P, (double*)(ws + l.energy_dy)},
                         (uint32_t*)(ws + l.words), 64 + g.n, st);
}
static vcnn_status scan_energies(const ConvGeom& g, int pass, int dtype, const Layout& l, const void* src, void* workspace, hipStream_t st) {
  const bool fwd = pass == VCNN_PASS_FWD;
  const EnergyJob job{src, fwd ? g.c : g.k, fwd ? (int64_t)g.h * g.w : g.P, (double*)((char*)workspace + l.energy)};
  return launch_energies(dtype, g.n, job, {}, (uint32_t*)((char*)workspace + l.words), 64 + g.n, st);
}

// The lines of a tensor of `channels` channels of h x w, and of the kernels (one line each).
static SpectralLines lines_for(const ConvGeom& g, const SpectralPlan& p, int channels, int h, int w) {
  SpectralLines t{};
  t.images = g.n, t.channels = channels, t.first = 0, t.count = channels;
  t.len = p.along == 1 ? w : h, t.others = p.along == 1 ? h : w;
  t.tiles = p.tiles_x, t.step = p.step_x, t.lim = kLL;
  t.s_channel = (int64_t)h * w, t.s_other = p.along == 1 ? w : 1, t.s_along = p.along == 1 ? 1 : w;
  t.p_image = (int64_t)t.others * t.tiles, t.p_channel = g.n * t.p_image;  // the lines of a channel of all images together
  return t;
}
static SpectralLines kernel_lines(const ConvGeom& g, int maps) {
  SpectralLines t{};
  t.images = maps, t.channels = t.count = g.c;
  t.len = t.lim = g.r * g.s, t.others = t.tiles = t.step = 1;
  t.s_channel = g.r * g.s, t.s_other = 0, t.s_along = 1;
  t.p_image = g.c, t.p_channel = 1;
  return t;
}
// Tile offsets of the three tensors: x starts a tile `pad` before it.  In an input gradient pixel i of the padded line gets
// dy[i - q] w[q]: a whole line starts at dy's first pixel; a tile of a longer one starts `size` - 1 pixels before its results,
// of which the transform wraps that many.
static void place_dx(bool one, int size, int pad, int* dy0, int* dx0) { *dy0 = one ? 0 : pad - (size - 1), *dx0 = one ? pad : size - 1; }

static vcnn_status lines_fwd(const SpectralPlan& p, int dtype, const ConvGeom& g, const void* x, const void* w, const float* bias,
                             void* y, int relu, void* workspace, hipStream_t st) {
  const Layout l = layout(g, VCNN_PASS_FWD, p);
  char* const ws = (char*)workspace;
  float2 *const xs = (float2*)(ws + l.image), *const ys = (float2*)(ws + l.map), *const taps = (float2*)(ws + l.taps);
  uint32_t* const largest = (uint32_t*)(ws + l.largest);
  const WindowGuard guard = window_guard(g, VCNN_PASS_FWD, dtype, l, kLL, workspace);
  const SpectralExcept except{1, guard.words.image, guard.zero, guard.words.zeros};
  const int64_t tiles = tiles_of(g, p, VCNN_PASS_FWD);
  const int esize = dtype == VCNN_BF16 ? 2 : 4;
  SpectralLines tx = lines_for(g, p, g.c, g.h, g.w);
  tx.x0 = -(p.along == 1 ? g.pw : g.ph);
  SpectralLines ty = lines_for(g, p, g.k, g.oh, g.ow);
  ty.lim = std::min(p.step_x, ty.len);
  if (vcnn_status s = scan_energies(g, VCNN_PASS_FWD, dtype, l, x, workspace, st)) return s;
  if (vcnn_status s = launch_guard_lines(guard, tx, ty, g.r * g.s, st)) return s;
  for (int k0 = 0; k0 < g.k; k0 += p.part) {
    const int maps = std::min(p.part, g.k - k0);
    const bool last = k0 + maps == g.k;
    LineJob image{tx, tiles * g.c, x, xs, nullptr, nullptr};
    if (k0 > 0) image.t.count = 0;  // (they stay)
    const LineJob kernels{kernel_lines(g, maps), (int64_t)maps * g.c, (const char*)w + (int64_t)k0 * g.K * esize, taps, largest + (int64_t)k0 * g.c, nullptr};
    if (vcnn_status s = launch_line_spectra(dtype, image, kernels, {}, st)) return s;
    ProductArgs a{};
    a.A = taps, a.B = xs, a.C = ys;
    a.rows = maps, a.cols = (int)tiles, a.depth = g.c;
    a.a_row = g.c, a.a_z = 1, a.a_planes = (int64_t)maps * g.c;
    a.b_col = 1, a.b_z = tiles, a.b_planes = tiles * g.c;
    a.c_row = tiles, a.c_col = 1, a.c_planes = tiles * maps;
    a.splits = p.splits, a.per_split = p.per_split, a.flush = p.flush, a.rows_inner = 1;
    a.range = range_guard(g, VCNN_PASS_FWD, p, l, workspace), a.declined = guard.words.any, a.col_images = (int)(tiles / g.n);
    if (vcnn_status s = launch_product<false, true, false, true>(a, last ? g.n : 0, st)) return s;
    ty.first = k0, ty.count = maps;
    if (vcnn_status s = launch_line_inverse(ty, tiles * maps, dtype, ys, 0, 1, y, bias, relu, nullptr, 0, 0, nullptr, except, st)) return s;
  }
  return VCNN_OK;
}

static vcnn_status lines_bwd_data(const SpectralPlan& p, int dtype, const ConvGeom& g, const void* w, const void* dy, void* dx,
                                  void* workspace, hipStream_t st) {
  const Layout l = layout(g, VCNN_PASS_BWD_DATA, p);
  char* const ws = (char*)workspace;
  float2 *const xs = (float2*)(ws + l.image), *const ys = (float2*)(ws + l.map), *const taps = (float2*)(ws + l.taps);
  uint32_t* const largest = (uint32_t*)(ws + l.largest);
  const WindowGuard guard = window_guard(g, VCNN_PASS_BWD_DATA, dtype, l, kLL, workspace);
  const int64_t tiles = tiles_of(g, p, VCNN_PASS_BWD_DATA);
  const int pad = p.along == 1 ? g.pw : g.ph;
  SpectralLines tdy = lines_for(g, p, g.k, g.oh, g.ow), tdx = lines_for(g, p, g.c, g.h, g.w);
  place_dx(tdx.len + 2 * pad <= kLL, g.r * g.s, pad, &tdy.x0, &tdx.x0);
  tdx.lim = std::min(p.step_x, tdx.len);
  const LineJob image{tdy, tiles * g.k, dy, ys, nullptr, nullptr};
  const LineJob kernels{kernel_lines(g, g.k), (int64_t)g.k * g.c, w, taps, largest, nullptr};
  if (vcnn_status s = scan_energies(g, VCNN_PASS_BWD_DATA, dtype, l, dy, workspace, st)) return s;
  if (vcnn_status s = launch_guard_lines(guard, tdy, tdx, g.r * g.s, st)) return s;
  if (vcnn_status s = launch_line_spectra(dtype, image, kernels, {}, st)) return s;
  ProductArgs a{};
  a.A = taps, a.B = ys, a.C = xs;
  a.rows = g.c, a.cols = (int)tiles, a.depth = g.k;
  a.a_row = 1, a.a_z = g.c, a.a_planes = (int64_t)g.k * g.c;
  a.b_col = 1, a.b_z = tiles, a.b_planes = tiles * g.k;
  a.c_row = tiles, a.c_col = 1, a.c_planes = tiles * g.c;
  a.splits = p.splits, a.per_split = p.per_split, a.flush = p.flush, a.rows_inner = 1, a.c_slice = (int64_t)(p.image_bytes / p.splits / 8);
  a.range = range_guard(g, VCNN_PASS_BWD_DATA, p, l, workspace), a.declined = guard.words.any, a.col_images = (int)(tiles / g.n);
  if (vcnn_status s = launch_product<false, false, false, true>(a, g.n, st)) return s;
  return launch_line_inverse(tdx, tiles * g.c, dtype, xs, a.c_slice, p.splits, dx, nullptr, 0, nullptr, 0, 0, nullptr,
                             {1, guard.words.image, guard.zero, guard.words.zeros}, st);
}

static vcnn_status lines_filter(const SpectralPlan& p, int dtype, const ConvGeom& g, const void* x, const void* dy, float* dw,
                                float* db, void* workspace, hipStream_t st) {
  const Layout l = layout(g, VCNN_PASS_BWD_FILTER, p);
  char* const ws = (char*)workspace;
  float2 *const xs = (float2*)(ws + l.image), *const ys = (float2*)(ws + l.map), *const taps = (float2*)(ws + l.taps);
  double* const sums = (double*)(ws + l.sums);
  const MeetGuard meet = meet_guard(g, p, l, workspace);
  const MeetDecision decision = meet_decision(g, p, l, meet, workspace);
  const int64_t tiles = tiles_of(g, p, VCNN_PASS_BWD_FILTER);
  SpectralLines tx = lines_for(g, p, g.c, g.h, g.w), tdy = lines_for(g, p, g.k, g.oh, g.ow);
  tx.x0 = -(p.along == 1 ? g.pw : g.ph);
  tdy.lim = std::min(p.step_x, tdy.len);  // every output pixel in one tile
  const LineJob image{tx, tiles * g.c, x, xs, nullptr, nullptr}, map{tdy, tiles * g.k, dy, ys, nullptr, db ? sums : nullptr};
  if (vcnn_status s = scan_both(g, dtype, l, x, dy, workspace, st)) return s;
  if (vcnn_status s = launch_meet_lines(meet, tx, tdy, g.r * g.s, st)) return s;
  if (vcnn_status s = launch_line_spectra(dtype, image, map, decision, st)) return s;
  ProductArgs a{};
  a.A = ys, a.B = xs, a.C = taps;
  a.rows = g.k, a.cols = g.c, a.depth = (int)tiles;
  a.a_row = tiles, a.a_z = 1, a.a_planes = tiles * g.k;
  a.b_col = tiles, a.b_z = 1, a.b_planes = tiles * g.c;
  a.c_row = g.c, a.c_col = 1, a.c_planes = (int64_t)g.k * g.c;
  a.splits = p.splits, a.per_split = p.per_split, a.flush = p.flush, a.c_slice = (int64_t)(p.taps_bytes / p.splits / 8);
  a.declined = meet.words.any;
  if (vcnn_status s = launch_product<false, true, false, true>(a, 0, st)) return s;
  return launch_line_inverse(kernel_lines(g, g.k), (int64_t)g.k * g.c, VCNN_F32, taps, a.c_slice, p.splits, dw, nullptr, 0, sums,
                             (int)tiles, g.k, db, {0, meet.words.any, decision.zero, meet.words.zeros}, st);
}

vcnn_status launch_spectral_fwd(const SpectralPlan& p, int dtype, const ConvGeom& g, const void* x, const void* w, const float* bias,
                                void* y, int relu, void* workspace, hipStream_t st) {
  if (p.along) return lines_fwd(p, dtype, g, x, w, bias, y, relu, workspace, st);
  const Layout l = layout(g, VCNN_PASS_FWD, p);
  char* const ws = (char*)workspace;
  float2* const xs = (float2*)(ws + l.image);
  float2* const ys = (float2*)(ws + l.map);
  float2* const taps = (float2*)(ws + l.taps);
  uint32_t* const largest = (uint32_t*)(ws + l.largest);
  const WindowGuard guard = window_guard(g, VCNN_PASS_FWD, dtype, l, kFL * kFL, workspace);
  const SpectralExcept except{1, guard.words.image, guard.zero, guard.words.zeros};
  const int64_t tiles = tiles_of(g, p, VCNN_PASS_FWD);
  const int esize = dtype == VCNN_BF16 ? 2 : 4;
  SpectralTiles tx = tiles_for(g, p, g.c, g.h, g.w);
  tx.y0 = -g.ph, tx.x0 = -g.pw;
  SpectralTiles ty = tiles_for(g, p, g.k, g.oh, g.ow);
  ty.lim_y = std::min(p.step_y, g.oh), ty.lim_x = std::min(p.step_x, g.ow);
  if (vcnn_status s = scan_energies(g, VCNN_PASS_FWD, dtype, l, x, workspace, st)) return s;
  if (vcnn_status s = launch_guard_planes(guard, tx, ty, g.r, g.s, st)) return s;
  if (vcnn_status s = launch_plane_spectra(tx, dtype, x, xs, nullptr, guard.words.image, 1, {}, st)) return s;
  for (int k0 = 0; k0 < g.k; k0 += p.part) {
    const int maps = std::min(p.part, g.k - k0);
    const bool last = k0 + maps == g.k;
    if (vcnn_status s = launch_taps_spectra(dtype, (const char*)w + (int64_t)k0 * g.K * esize, (int64_t)maps * g.c, g.r, g.s, taps,
                                            largest + (int64_t)k0 * g.c / 4, st)) return s;
    ProductArgs a{};
    a.A = taps, a.B = xs, a.C = ys;
    a.rows = maps, a.cols = (int)tiles, a.depth = g.c;
    a.a_row = g.c, a.a_z = 1, a.a_planes = (int64_t)maps * g.c;
    a.b_col = g.c, a.b_z = 1, a.b_planes = tiles * g.c;
    a.c_row = 1, a.c_col = maps, a.c_planes = tiles * maps;
    a.splits = p.splits, a.per_split = p.per_split, a.flush = p.flush;
    a.range = range_guard(g, VCNN_PASS_FWD, p, l, workspace), a.declined = guard.words.any, a.col_images = (int)(tiles / g.n);
    if (vcnn_status s = launch_product<true, true, false, false>(a, last ? g.n : 0, st)) return s;
    ty.first = k0, ty.count = maps;
    if (vcnn_status s = launch_plane_inverse(ty, dtype, ys, 0, 1, y, bias, relu, except, st)) return s;
  }
  return VCNN_OK;
}

vcnn_status launch_spectral_bwd_data(const SpectralPlan& p, int dtype, const ConvGeom& g, const void* w, const void* dy, void* dx,
                                     void* workspace, hipStream_t st) {
  if (p.along) return lines_bwd_data(p, dtype, g, w, dy, dx, workspace, st);
  const Layout l = layout(g, VCNN_PASS_BWD_DATA, p);
  char* const ws = (char*)workspace;
  float2* const xs = (float2*)(ws + l.image);
  float2* const ys = (float2*)(ws + l.map);
  float2* const taps = (float2*)(ws + l.taps);
  uint32_t* const largest = (uint32_t*)(ws + l.largest);
  const WindowGuard guard = window_guard(g, VCNN_PASS_BWD_DATA, dtype, l, kFL * kFL, workspace);
  const int64_t tiles = tiles_of(g, p, VCNN_PASS_BWD_DATA);
  const bool one = one_tile(g);
  SpectralTiles tdy = tiles_for(g, p, g.k, g.oh, g.ow);
  SpectralTiles tdx = tiles_for(g, p, g.c, g.h, g.w);
  place_dx(one, g.r, g.ph, &tdy.y0, &tdx.y0);
  place_dx(one, g.s, g.pw, &tdy.x0, &tdx.x0);
  tdx.lim_y = std::min(p.step_y, g.h), tdx.lim_x = std::min(p.step_x, g.w);
  if (vcnn_status s = scan_energies(g, VCNN_PASS_BWD_DATA, dtype, l, dy, workspace, st)) return s;
  if (vcnn_status s = launch_guard_planes(guard, tdy, tdx, g.r, g.s, st)) return s;
  if (vcnn_status s = launch_plane_spectra(tdy, dtype, dy, ys, nullptr, guard.words.image, 1, {}, st)) return s;
  if (vcnn_status s = launch_taps_spectra(dtype, w, (int64_t)g.k * g.c, g.r, g.s, taps, largest, st)) return s;
  ProductArgs a{};
  a.A = taps, a.B = ys, a.C = xs;
  a.rows = g.c, a.cols = (int)tiles, a.depth = g.k, a.rows_inner = 1;
  a.a_row = 1, a.a_z = g.c, a.a_planes = (int64_t)g.k * g.c;
  a.b_col = g.k, a.b_z = 1, a.b_planes = tiles * g.k;
  a.c_row = 1, a.c_col = g.c, a.c_planes = tiles * g.c;
  a.splits = p.splits, a.per_split = p.per_split, a.flush = p.flush, a.c_slice = (int64_t)(p.image_bytes / p.splits / 8);
  a.range = range_guard(g, VCNN_PASS_BWD_DATA, p, l, workspace), a.declined = guard.words.any, a.col_images = (int)(tiles / g.n);
  if (vcnn_status s = launch_product<true, false, false, false>(a, g.n, st)) return s;
  return launch_plane_inverse(tdx, dtype, xs, a.c_slice, p.splits, dx, nullptr, 0, {1, guard.words.image, guard.zero, guard.words.zeros}, st);
}

vcnn_status launch_spectral_filter(const SpectralPlan& p, int dtype, const ConvGeom& g, const void* x, const void* dy, float* dw,
                                   float* db, void* workspace, hipStream_t st) {
  if (p.along) return lines_filter(p, dtype, g, x, dy, dw, db, workspace, st);
  const Layout l = layout(g, VCNN_PASS_BWD_FILTER, p);
  char* const ws = (char*)workspace;
  float2* const xs = (float2*)(ws + l.image);
  float2* const ys = (float2*)(ws + l.map);
  float2* const taps = (float2*)(ws + l.taps);
  const MeetGuard meet = meet_guard(g, p, l, workspace);
  const MeetDecision decision = meet_decision(g, p, l, meet, workspace);
  double* const sums = (double*)(ws + l.sums);
  const int64_t tiles = tiles_of(g, p, VCNN_PASS_BWD_FILTER);
  SpectralTiles tx = tiles_for(g, p, g.c, g.h, g.w);
  tx.y0 = -g.ph, tx.x0 = -g.pw;
  SpectralTiles tdy = tiles_for(g, p, g.k, g.oh, g.ow);
  tdy.lim_y = std::min(p.step_y, g.oh), tdy.lim_x = std::min(p.step_x, g.ow);  // every output pixel in one tile
  if (vcnn_status s = scan_both(g, dtype, l, x, dy, workspace, st)) return s;
  if (vcnn_status s = launch_meet_planes(meet, tx, tdy, g.r, g.s, st)) return s;
  if (vcnn_status s = launch_plane_spectra(tx, dtype, x, xs, nullptr, nullptr, 0, decision, st)) return s;
  if (vcnn_status s = launch_plane_spectra(tdy, dtype, dy, ys, db ? sums : nullptr, meet.words.any, 0, {}, st)) return s;
  ProductArgs a{};
  a.A = ys, a.B = xs, a.C = taps;
  a.rows = g.k, a.cols = g.c, a.depth = (int)tiles;
  a.a_row = 1, a.a_z = g.k, a.a_planes = tiles * g.k;
  a.b_col = 1, a.b_z = g.c, a.b_planes = tiles * g.c;
  a.c_row = g.c, a.c_col = 1, a.c_planes = (int64_t)g.k * g.c;
  a.splits = p.splits, a.per_split = p.per_split, a.flush = p.flush, a.c_slice = (int64_t)(p.taps_bytes / p.splits / 8);
  a.declined = meet.words.any;
  if (vcnn_status s = launch_product<false, true, true, false>(a, 0, st)) return s;
  return launch_taps_inverse(taps, a.c_slice, p.splits, (int64_t)g.k * g.c, g.r, g.s, dw, sums, (int)tiles, g.k, db,
                             {0, meet.words.any, decision.zero, meet.words.zeros}, st);
}

Declined spectral_declined(const ConvGeom& g, int pass, const SpectralPlan& p, const void* workspace) {
  const SpectralWords words = words_at(const_cast<void*>(workspace), layout(g, pass, p));
  return {nullptr, nullptr, nullptr, words.any, pass == VCNN_PASS_BWD_FILTER ? nullptr : words.image};
}

}  // namespace vcnn
