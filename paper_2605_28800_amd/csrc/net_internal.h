// Kernels of the initial-state proposal network (3-D conv encoder-decoder)
// and their launchers, shared by net.hip and net_api.cpp.
//
// Tensors are BF16 (stored as uint16), channels-last: [position][channel],
// position = ((b * Z + z) * Y + y) * X + x, the channel count padded to a
// multiple of 16.  Grid sizes are powers of two (log2 in lx, ly, lz).
// Weights: plain, [cout_p][27 * cin_p] (k = tap * cin_p + ci; tap t =
// 9 (dz + 1) + 3 (dy + 1) + (dx + 1)), as the single-layer entry points take
// them, or packed in the order of the matrix operands, as the network keeps
// its forward weights and the backward-data copy (channels exchanged, tap
// mirrored): for every chunk c of 16 input channels and step s = 0..13 the
// 16-row blocks m as 64 lanes x 8 values, lane (kq, col) holding row 16 m + col,
// tap 2 s + kq / 2 (zero for tap 27), channels 16 c + 8 (kq % 2) + 0..7.
#pragma once
#include <hip/hip_runtime.h>
#include <cstddef>
#include <cstdint>

namespace tdgl_nn {

typedef uint16_t bf16_t;

constexpr float SLOPE = 0.125f;     // leaky ReLU slope for negative arguments (exact in BF16)

// epilogues of the implicit-GEMM convolution
enum ConvEpi {
  EPI_ACT = 0,        // out = act(acc + bias)
  EPI_ACT_SKIP = 1,   // out = act(acc + bias), out2 = out + aux
  EPI_P = 2,          // P (FP32, [b][3][z][y][x]) = film mask * (acc + bias)
  EPI_RAW = 3,        // out = acc
  EPI_RAW_D = 4,      // out = acc * act'(aux)
  EPI_RAW_AND_D = 5,  // out = acc, out2 = acc * act'(aux)
};

struct ConvArgs {
  const bf16_t *in;   // input tensor, cin_p channels (half resolution if in_up2)
  const bf16_t *w;    // plain or packed weights of cout_p rows, cin_p channels
  int packed;
  const float *bias;  // [cout_p] or null
  bf16_t *out, *out2; // [n][cout_p]
  const bf16_t *aux;  // [n][cout_p]: skip addend or activation
  float *P;           // EPI_P output
  const float *thick; // EPI_P: film thickness per dataset row
  const int *idx;     // EPI_P: dataset row of each sample (null: identity)
  int in_up2;         // input is the nearest-neighbour upsampling of a half grid
  int lx, ly, lz, nb; // output grid (log2) and samples
  int cin_p, cout_p;
};

constexpr size_t packed_size(int cin_p, int cout_p) { return (size_t)28 * cin_p * cout_p; }

struct WgradArgs {
  const bf16_t *g;    // [n][cout_p] gradient of the layer output (pre-activation)
  const bf16_t *in;   // layer input (half resolution if in_up2), cin_p channels
  float *part;        // [splits][cout_p][27 * cin_p]
  float *bpart;       // [splits][cout_p]
  int in_up2;
  int lx, ly, lz, nb;
  int cin_p, cout_p;
  // from wgrad_plan: the kernel, the splits, and per split the tiles (tiled) or
  // the positions, a multiple of 32
  int tiled, splits, chunk;
  int max_splits;     // no smaller batch of this layer has more splits
};

hipError_t launch_conv(int epi, const ConvArgs &a, hipStream_t s);
int conv_tile_code(const ConvArgs &a);    // 16 * channel blocks + rows per wave; 0: small grids
hipError_t launch_wgrad(const WgradArgs &a, hipStream_t s);
// from the grid and the channels; most: at most so many splits (0: as many as pay),
// for a tiled plan no fewer than wgrad_least_splits, which is what the kernel of small
// grids would use
void wgrad_plan(WgradArgs *a, int most = 0);
int wgrad_least_splits(const WgradArgs &planned);

// elementwise parts
// ops: per-sample in-plane symmetry op (bits: 1 mirror x, 2 mirror y, 4 swap
// x and y on square grids), or null for none
hipError_t launch_input(const float *T, const float *thick, const float *noise, const int *idx,
                        const int *ops, int lx, int ly, int lz, int nb, int noise_div, bf16_t *x0,
                        hipStream_t s);
hipError_t launch_pool(const bf16_t *in, int lx, int ly, int lz, int nb, int c_p, bf16_t *out,
                       hipStream_t s);
hipError_t launch_pool_bwd(const bf16_t *g, const bf16_t *add, const bf16_t *a, int lx, int ly,
                           int lz, int nb, int c_p, bf16_t *out, hipStream_t s);
hipError_t launch_up_bwd(const bf16_t *g, const bf16_t *a, int lx, int ly, int lz, int nb,
                         int c_p, bf16_t *out, hipStream_t s);
hipError_t launch_loss(const float *P, const float *target, const float *thick, const int *idx,
                       const int *ops, int lx, int ly, int lz, int nb, bf16_t *gy,
                       double *partials, int *nblocks, hipStream_t s);
hipError_t launch_sum_partials(const double *partials, int n, double *out, hipStream_t s);
hipError_t launch_reduce_grad(const float *part, const float *bpart, int splits, int cin,
                              int cout, int cin_p, int cout_p, float *grad, hipStream_t s);
// Adam step number t (from 1)
hipError_t launch_adam(float *master, float *m, float *v, const float *grad, long long n,
                       double lr, double b1, double b2, double eps, long long t, hipStream_t s);
hipError_t launch_cast_weights(const float *master, int cin, int cout, int cin_p, int cout_p,
                               bf16_t *w, bf16_t *wt, float *bias, hipStream_t s);

}  // namespace tdgl_nn

// For tests.  The tile of a convolution of these sizes (conv_tile_code), and a
// convolution with weights packed as the network packs them: W[cout][27][cin] and
// bias[cout] behind it (device FP32), into w and wt of packed_size BF16 each and
// bias of cout_p floats; mirror: the backward-data weights wt, from cout_p to cin_p
// channels.
extern "C" int tdgl_internal_conv_tile(int nb, int lx, int ly, int lz, int cin_p, int cout_p);
extern "C" int tdgl_internal_conv3_packed(int epi, const void *in, int in_up2, const float *W,
                                          int mirror, int cin, int cout, int nb, int lx, int ly,
                                          int lz, int cin_p, int cout_p, void *out, void *out2,
                                          const void *aux, void *w, void *wt, float *bias,
                                          void *hip_stream);
