// Convolutions through the Fourier domain (planes of 64 x 64 pixels): what the transforms (spectral_fft.hip) and the
// products (spectral.hip) share.
//
// With xt a plane of at most 64 x 64 pixels and wt a kernel, both zero-extended to 64 x 64 and transformed,
//   forward         Y(u,v)  = sum_c X_c(u,v) conj(W_kc(u,v))    valid where the kernel lies inside the plane
//   input gradient  dX(u,v) = sum_k dY_k(u,v) W_kc(u,v)
//   kernel gradient dW(u,v) = sum_n X_nc(u,v) conj(dY_nk(u,v))  the first R x S elements
// so a pass costs 64 * 33 complex products per pair of planes where the direct sum costs R S oh ow real ones (16 x 16 taps
// on 64 x 64 pixels: 73 times fewer operations).  Larger planes are cut into tiles of 64 x 64 whose valid parts join.
//
// Precision.  The transforms run in double (the vector units do a double as fast as a float), spectra are stored as float,
// and the products add in float on the matrix cores over the channels (maps, images) only.  What is rounded to float is
// each spectrum once (rows of a kernel once more) and the short sums, so the result lies nearer the 64-bit one than that of
// the direct kernels, whose sums run over channels times taps.  The error is spread evenly over a transform, though, whatever
// the samples under an output's window: outputs whose window holds nothing but zeros are put to zero exactly, and an image with
// an output that sums too little of its transform's energy for that error (kDark...), with magnitudes whose products leave
// the range of a float, or with an infinity or NaN is DECLINED on the device (spectral_guard.hip) and computed by the
// direct route enqueued behind, which otherwise leaves at once.
#pragma once
#include "common.h"

namespace vcnn {

static constexpr int kFL = 64;        // transform length
static constexpr int kFV = 33;        // columns of a real plane's spectrum
static constexpr int kFTaps = 16;     // most kernel rows / columns
// A plane's spectrum is stored as columns v = 0..32, each of 64 complex floats in four residues rho = u mod 4 (one wave of
// the product each) of the 16 frequencies u = 4 a + rho in order.
// Layers whose kernels are one row (column) do the same with lines of 256 samples along it; a line's spectrum is two such
// columns of 64 values, frequencies 0..127, the first with those of 0 and 128 (both real) as its two parts.

static constexpr int kLL = 256, kLV = 2, kLineTaps = 128;  // lines: length, columns of 64 values, most taps
// A forward pass or input gradient declines an image where an output's window has, per sample of it, less energy (sum of squares
// over the channels) than this share of the mean over its transform, or in all less than that share of one mean sample: an
// error of some 1e-7 of the transform's mean output is then at most 16 times that of the output's own scale (short windows at
// the border of an input gradient: 4 sqrt(taps) times).
static constexpr double kDarkMean = 1.0 / 256, kDarkLeast = 1.0 / 16;
static constexpr double kDarkBf16 = 1.0 / 1024;  // of those, where the result is rounded to eight bits: 32 times the error
// A kernel gradient declines, all of it, where at a tap what meets - the energies of the two operands multiplied pixel by pixel -
// is less than this share of the mean over all shifts: an error of 6e-8 of the mean result at most four times that of the tap's own.
static constexpr double kDarkMeet = 1.0 / 16;

struct SpectralPlan {
  int along;               // 0: planes; kernels of one row (1) or one column (2): lines along the width or the height
  int tiles_y, tiles_x;    // tiles of a plane
  int step_y, step_x;      // distance of the tiles' valid parts
  int part;                // forward: output maps worked on at once (else all)
  int splits, per_split;   // slices of the contraction, summed by the inverse transform
  int flush;               // products in one sum
  int energy_in_taps;      // kernel gradient: the energies of the operands in the place of the result's spectra
  size_t image_bytes;      // spectra over the input channels (input gradient: one slice per split)
  size_t map_bytes;        // spectra over the output maps (of a part)
  size_t taps_bytes;       // row spectra of the kernels (of a part; kernel gradient: one slice per split)
  size_t words_bytes;      // energies, masks, maxima, sums and the words of Declined: behind everything else
  size_t workspace_bytes;
  double est_seconds;
};
bool spectral_plan(const ConvGeom& g, int pass, size_t budget, SpectralPlan* p);
vcnn_status launch_spectral_fwd(const SpectralPlan& p, int dtype, const ConvGeom& g, const void* x, const void* w, const float* bias,
                                void* y, int relu, void* workspace, hipStream_t st);
vcnn_status launch_spectral_bwd_data(const SpectralPlan& p, int dtype, const ConvGeom& g, const void* w, const void* dy, void* dx,
                                     void* workspace, hipStream_t st);
vcnn_status launch_spectral_filter(const SpectralPlan& p, int dtype, const ConvGeom& g, const void* x, const void* dy, float* dw,
                                   float* db, void* workspace, hipStream_t st);
// The images these passes leave to the route behind them.
Declined spectral_declined(const ConvGeom& g, int pass, const SpectralPlan& p, const void* workspace);

// ---- spectral_fft.hip -----------------------------------------------------------------------------------------------
// Planes of a tensor [images][channels][h][w], tile by tile: tile (ty, tx) starts at pixel (ty step_y + y0, tx step_x + x0)
// (what lies outside the plane is zero) and holds lim_y x lim_x pixels.  Spectra of plane (image, ty, tx, channel) in order.
struct SpectralTiles {
  int images, channels, first, count;  // channels first .. first + count - 1 of each image
  int h, w;
  int tiles_y, tiles_x, step_y, step_x, y0, x0, lim_y, lim_x;
  int64_t planes() const { return (int64_t)images * tiles_y * tiles_x * count; }
};
struct SpectralWords {  // cleared by launch_energies: 64 words and one for each image
  uint32_t* any;
  uint32_t* zeros;  // an output's window holds only zeros
  uint32_t* image;
};
// The decision about a kernel gradient from what meets at its taps (launch_meet_..), by one block of the transforms that follow: the
// word that declines, and a bit for each tap at which nothing meets (zero[16]: the rows of a kernel, of one row 64 taps each).
struct MeetDecision {
  const double* partial;  // null: nothing to decide
  int chunks, r, s;
  double share;
  int grow;
  uint64_t* zero;
  SpectralWords words;
};
// Also leaves each plane's sum (sums, nullable).  What is declined (nullable: a word for each image, or one) may be left out, where
// no sums are asked for; `decide` is done on the way.
vcnn_status launch_plane_spectra(const SpectralTiles& t, int dtype, const void* src, float2* spectra, double* sums,
                                 const uint32_t* declined, int per_image, const MeetDecision& decide, hipStream_t st);
// What an inverse transform does not write, and what it writes as zero (both nullable).
struct SpectralExcept {
  int per_image;             // the words are each image's, each transform's, or (0) one for all
  const uint32_t* declined;  // [image]
  const uint64_t* zero;      // a bit for each sample of a transform: [tile][64 rows], [line][4] ...
  const uint32_t* zeros;     // ... where this is set
};
// The spectra of planes back to pixels: pixel (y, x) of tile (ty, tx) is (ty step_y + y, tx step_x + x) of the plane and lies
// at (y + y0, x + x0) of the transform; `slices` spectra of a plane, `slice` complex values apart, are added first; bias per channel, nullable.
vcnn_status launch_plane_inverse(const SpectralTiles& t, int dtype, const float2* spectra, int64_t slice, int slices, void* dst,
                                 const float* bias, int relu, const SpectralExcept& except, hipStream_t st);
// Row spectra of kernels of r x s taps: [v][kernel][16 rows]; largest magnitude of each four kernels.
vcnn_status launch_taps_spectra(int dtype, const void* w, int64_t kernels, int r, int s, float2* spectra, uint32_t* largest,
                                hipStream_t st);
// And back; also, in blocks of their own, db[m] = sums[0][m] + sums[1][m] + ... (planes of `maps` maps; nullable).
vcnn_status launch_taps_inverse(const float2* spectra, int64_t slice, int slices, int64_t kernels, int r, int s, float* dw,
                                const double* sums, int sum_planes, int maps, float* db, const SpectralExcept& except, hipStream_t st);

// Lines of a tensor [images][channels][...]: sample x of line (image, channel, o) lies at o s_other + x s_along of the channel;
// tiles as above, in one dimension.  The spectrum of line (image, channel, o, tile) is number
// image p_image + channel p_channel + o tiles + tile.
struct SpectralLines {
  int images, channels, first, count;
  int len, others, tiles, step, x0, lim;
  int64_t s_channel, s_other, s_along;
  int64_t p_image, p_channel;
  __host__ __device__ int64_t lines() const { return (int64_t)images * count * others * tiles; }
};
struct LineJob {
  SpectralLines t;
  int64_t planes;    // spectra per column
  const void* src;
  float2* spectra;
  uint32_t* largest; // magnitude of each line, nullable
  double* sums;      // sums of the lines, nullable: [image][o][tile][channel]
};
// The lines of two tensors (the second may have none: all zero).
vcnn_status launch_line_spectra(int dtype, const LineJob& first, const LineJob& second, const MeetDecision& decide, hipStream_t st);
vcnn_status launch_line_inverse(const SpectralLines& t, int64_t planes, int dtype, const float2* spectra, int64_t slice, int slices,
                                void* dst, const float* bias, int relu, const double* sums, int sum_planes, int maps, float* db,
                                const SpectralExcept& except, hipStream_t st);

// ---- spectral_guard.hip ---------------------------------------------------------------------------------------------
struct EnergyJob {
  const void* src;  // [image][channels][pixels]
  int channels;
  int64_t pixels;
  double* energy;   // [image][pixels]: the sum of the squares over the channels
};
// (the second may have no pixels)
vcnn_status launch_energies(int dtype, int images, const EnergyJob& first, const EnergyJob& second, uint32_t* words, int cleared,
                            hipStream_t st);
struct WindowGuard {
  const double* energy;
  int back;            // the window of transform sample i: samples i and on (0), i and before (1)
  double mean, least;  // the least an output may sum, of its transform's energy: for each sample of its window, in all
  uint64_t* zero;      // left for the inverse transform
  double* totals;      // left for the guard of magnitudes: the energy of each transform
  SpectralWords words;
};
// in: the transforms of the operand with the energies; out: the outputs that the inverse transform keeps of them.
vcnn_status launch_guard_planes(const WindowGuard& g, const SpectralTiles& in, const SpectralTiles& out, int r, int s, hipStream_t st);
vcnn_status launch_guard_lines(const WindowGuard& g, const SpectralLines& in, const SpectralLines& out, int taps, hipStream_t st);
// What meets at each tap of a kernel gradient: partial[chunk][taps + 1] = the sums over some transforms of the products of the
// operands' energies, and of those of their totals.
struct MeetGuard {
  const double *x, *dy;  // energies [image][pixel]
  int chunks, per_chunk; // transforms
  double* partial;
  int depth_x, depth_dy; // bits of the root of the numbers of channels, of maps
  SpectralWords words;
};
vcnn_status launch_meet_planes(const MeetGuard& m, const SpectralTiles& x, const SpectralTiles& dy, int r, int s, hipStream_t st);
vcnn_status launch_meet_lines(const MeetGuard& m, const SpectralLines& x, const SpectralLines& dy, int taps, hipStream_t st);

}  // namespace vcnn
