// Kernels of the initial-state proposal network: implicit-GEMM 3x3x3
// convolutions on the BF16 matrix cores (v_mfma_f32_16x16x32_bf16, FP32
// accumulation), the weight gradient with an LDS transpose and split
// reduction, and the elementwise parts (input assembly, pooling, upsampling
// adjoint, loss, Adam).
//
// MFMA 16x16x32 operand layout (wave64): lane l holds A[m = l % 16][k = 8 (l / 16) + 0..7]
// and B[k = 8 (l / 16) + 0..7][n = l % 16]; the result D[m = 4 (l / 16) + i][n = l % 16],
// i = 0..3, sits in the lane's four accumulator registers.
#include "net_internal.h"

#include <cmath>

namespace tdgl_nn {

typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef float floatx4 __attribute__((ext_vector_type(4)));

__device__ inline float bf2f(bf16_t h) { return __uint_as_float((uint32_t)h << 16); }
// round to nearest, ties to even (one conversion instruction)
__device__ inline bf16_t f2bf(float f) {
  union { __bf16 h; bf16_t u; } v;
  v.h = (__bf16)f;
  return v.u;
}
__device__ inline float act(float z) { return fmaxf(z, SLOPE * z); }
__device__ inline float act_slope(bf16_t y) { return bf2f(y) > 0.f ? 1.f : SLOPE; }

__device__ inline bf16x8 load8(const bf16_t *p) { return *reinterpret_cast<const bf16x8 *>(p); }
__device__ inline bf16x8 zero8() {
  bf16x8 z;
  for (int i = 0; i < 8; ++i) z[i] = (__bf16)0.f;
  return z;
}

struct Pos {
  int b, z, y, x;
};
__device__ inline Pos decode(long long n, int lx, int ly, int lz) {
  Pos p;
  p.x = (int)(n & ((1 << lx) - 1));
  p.y = (int)((n >> lx) & ((1 << ly) - 1));
  p.z = (int)((n >> (lx + ly)) & ((1 << lz) - 1));
  p.b = (int)(n >> (lx + ly + lz));
  return p;
}

// element offset of the gathered input at (position p + tap d) of a conv
// whose output grid is (lx, ly, lz); -1 outside the grid
__device__ inline long long gather_index(const Pos &p, int dz, int dy, int dx, int lx, int ly,
                                         int lz, int up2) {
  const int z = p.z + dz, y = p.y + dy, x = p.x + dx;
  if ((unsigned)z >= (1u << lz) || (unsigned)y >= (1u << ly) || (unsigned)x >= (1u << lx))
    return -1;
  if (up2) {
    const int cx = lx - 1, cy = ly - 1, cz = lz - 1;
    return ((((long long)p.b << cz) + (z >> 1)) << (cy + cx)) + ((long long)(y >> 1) << cx) +
           (x >> 1);
  }
  return ((((long long)p.b << lz) + z) << (ly + lx)) + ((long long)y << lx) + x;
}

// ----------------------------------------------------------------- conv
// Small grids.  One work-group: 4 waves x 16 * NB output positions, 16 * MB
// output channels (blockIdx.y selects the channel block).  K = 27 * cin_p runs
// in steps of 32: each lane gathers 8 consecutive input channels of one tap
// for each of its NB position columns, and 8 consecutive weights per 16-row
// block; the operands of step k + 1 are loaded while step k's MFMAs run.
// wl: the weights of this lane's row (16 m + col of block m = 0); plain rows kp apart,
// packed ones co16 blocks of 16 rows a step
template <int MB, int NB, bool PACKED>
__device__ __forceinline__ void conv_operands(const ConvArgs &a, const bf16_t *wl, int kp, int co16,
                                              int lc, int k0, int kq, const Pos *p,
                                              const bool *inb, bf16x8 *av, bf16x8 *bv) {
  const int k = k0 + 8 * kq;
  const bool kv = k < kp;
  const int t = k >> lc, ci = k & (a.cin_p - 1);
  const int dz = t / 9 - 1, dy = (t / 3) % 3 - 1, dx = t % 3 - 1;
  const bf16_t *w = wl + k;
  int block = 16 * kp;
  if (PACKED) {
    w = wl + (size_t)((ci >> 4) * 14 + (t >> 1)) * co16 * 512 + (2 * (t & 1) + (ci >> 3 & 1)) * 128;
    block = 512;
  }
  for (int mb = 0; mb < MB; ++mb) av[mb] = kv ? load8(w + (size_t)mb * block) : zero8();
  for (int j = 0; j < NB; ++j) {
    long long src = -1;
    if (kv && inb[j]) src = gather_index(p[j], dz, dy, dx, a.lx, a.ly, a.lz, a.in_up2);
    bv[j] = src >= 0 ? load8(a.in + src * a.cin_p + ci) : zero8();
  }
}

typedef float floatx2 __attribute__((ext_vector_type(2)));
typedef __bf16 bf16x2 __attribute__((ext_vector_type(2)));
__device__ __forceinline__ uint32_t pack_bf16(float lo, float hi) {
  union { bf16x2 h; uint32_t u; } v;
  v.h = __builtin_convertvector((floatx2){lo, hi}, bf16x2);
  return v.u;
}

// Epilogue of one lane: channels co0 .. co0 + 3 of an output position, in three
// parts, so that a kernel loads the bias and the addends of all its positions
// before the first store (a load behind a store waits for it).  o: element
// offset of channel co0 at the position.
template <int EPI>
__device__ __forceinline__ floatx4 conv_bias(const ConvArgs &a, int co0) {
  if (EPI == EPI_ACT || EPI == EPI_ACT_SKIP || EPI == EPI_P) {
    typedef floatx4 floatx4_a4 __attribute__((aligned(4)));   // a caller's bias is an array of floats
    return *reinterpret_cast<const floatx4_a4 *>(a.bias + co0);
  }
  return floatx4{0.f, 0.f, 0.f, 0.f};
}

template <int EPI>
__device__ __forceinline__ uint2 conv_aux(const ConvArgs &a, size_t o) {
  if (EPI == EPI_ACT_SKIP || EPI == EPI_RAW_D || EPI == EPI_RAW_AND_D)
    return *reinterpret_cast<const uint2 *>(a.aux + o);
  return make_uint2(0u, 0u);
}

// (p, n: the position and its index; ls = log2 of the cells per sample)
template <int EPI>
__device__ __forceinline__ void conv_store(const ConvArgs &a, const Pos &p, long long n, int ls,
                                           int co0, size_t o, const floatx4 v,
                                           const floatx4 bias, const uint2 ax) {
  if (EPI == EPI_P) {
    if (co0 != 0) return;
    const int row = a.idx ? a.idx[p.b] : p.b;
    const float m = (float)p.z < a.thick[row] ? 1.f : 0.f;
    const long long r = n & ((1LL << ls) - 1);
    for (int c = 0; c < 3; ++c) a.P[(((long long)p.b * 3 + c) << ls) + r] = m * (v[c] + bias[c]);
    return;
  }
  float r[4];
  for (int i = 0; i < 4; ++i)
    r[i] = EPI == EPI_ACT || EPI == EPI_ACT_SKIP ? act(v[i] + bias[i]) : v[i];
  const uint2 w0 = make_uint2(pack_bf16(r[0], r[1]), pack_bf16(r[2], r[3]));
  if (EPI != EPI_RAW_D) *reinterpret_cast<uint2 *>(a.out + o) = w0;
  if (EPI == EPI_ACT_SKIP || EPI == EPI_RAW_D || EPI == EPI_RAW_AND_D) {
    const bf16_t xa[4] = {(bf16_t)(ax.x & 0xFFFF), (bf16_t)(ax.x >> 16), (bf16_t)(ax.y & 0xFFFF),
                          (bf16_t)(ax.y >> 16)};
    const bf16_t rr[4] = {(bf16_t)(w0.x & 0xFFFF), (bf16_t)(w0.x >> 16), (bf16_t)(w0.y & 0xFFFF),
                          (bf16_t)(w0.y >> 16)};
    float s[4];
    for (int i = 0; i < 4; ++i)
      s[i] = EPI == EPI_ACT_SKIP ? bf2f(rr[i]) + bf2f(xa[i]) : v[i] * act_slope(xa[i]);
    const uint2 w1 = make_uint2(pack_bf16(s[0], s[1]), pack_bf16(s[2], s[3]));
    *reinterpret_cast<uint2 *>((EPI == EPI_RAW_D ? a.out : a.out2) + o) = w1;
  }
}

template <int MB, int NB, int EPI, bool PACKED>
__global__ __launch_bounds__(256) void k_conv(ConvArgs a) {
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const int kq = lane >> 4, col = lane & 15;
  const int ls = a.lx + a.ly + a.lz;
  const long long npos = (long long)a.nb << ls;
  const int kp = 27 * a.cin_p;
  const int lc = __builtin_ctz(a.cin_p);
  const int co_blk = blockIdx.y * MB * 16;
  const long long nbase = ((long long)blockIdx.x * 4 + wave) * (16 * NB);

  Pos p[NB];
  bool inb[NB];
  for (int j = 0; j < NB; ++j) {
    const long long n = nbase + 16 * j + col;
    inb[j] = n < npos;
    p[j] = decode(inb[j] ? n : 0, a.lx, a.ly, a.lz);
  }

  floatx4 acc[MB][NB];
  for (int mb = 0; mb < MB; ++mb)
    for (int j = 0; j < NB; ++j) acc[mb][j] = floatx4{0.f, 0.f, 0.f, 0.f};

  const int co16 = a.cout_p >> 4;
  const bf16_t *wl = PACKED ? a.w + (size_t)(co_blk >> 4) * 512 + col * 8
                            : a.w + (size_t)(co_blk + col) * kp;
  bf16x8 av[MB], bv[NB];
  conv_operands<MB, NB, PACKED>(a, wl, kp, co16, lc, 0, kq, p, inb, av, bv);
  for (int k0 = 0; k0 < kp; k0 += 32) {
    bf16x8 an[MB], bn[NB];
    if (k0 + 32 < kp)
      conv_operands<MB, NB, PACKED>(a, wl, kp, co16, lc, k0 + 32, kq, p, inb, an, bn);
    for (int mb = 0; mb < MB; ++mb)
      for (int j = 0; j < NB; ++j)
        acc[mb][j] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(av[mb], bv[j], acc[mb][j], 0, 0, 0);
    for (int mb = 0; mb < MB; ++mb) av[mb] = an[mb];
    for (int j = 0; j < NB; ++j) bv[j] = bn[j];
  }

  // epilogue: this lane holds channels co0 .. co0 + 3 of position n
  for (int j = 0; j < NB; ++j) {
    if (!inb[j]) continue;
    const long long n = nbase + 16 * j + col;
    for (int mb = 0; mb < MB; ++mb) {
      const int co0 = co_blk + mb * 16 + 4 * kq;
      const size_t o = (size_t)n * a.cout_p + co0;
      conv_store<EPI>(a, p[j], n, ls, co0, o, acc[mb][j], conv_bias<EPI>(a, co0),
                      conv_aux<EPI>(a, o));
    }
  }
}

// LDS-tiled variant for grids with X >= 16, Y >= NR and Z >= 4: a
// work-group owns a 4 x NR x 16 (z, y, x) block, wave w the NR rows of
// plane w; per chunk of 16 input channels the 6 x (NR + 2) x 18 input halo
// of the block is staged in LDS once (direct loads), and all 27 taps read their
// operand from there, two taps of 16 channels per matrix step.  The next chunk's
// halo lands in a second buffer while this chunk is multiplied.  A halo position is 32
// bytes without padding: the 16 columns and the two halves of a tap cover 512
// contiguous bytes, free of bank conflicts.
// What bounds it: each step of a wave needs MB weight fragments (1 KB each,
// from L1/L2) and NR input fragments (from LDS) for MB * NR matrix
// instructions.  Plain weight rows put a fragment's 64 pieces of 16 bytes on 32
// cache lines, and those lookups held the matrix cores at a quarter of their
// rate; packed fragments (8 lines) do not.  Scheduling barriers keep the loads
// ahead of the matrix instructions that hide them: left alone, the compiler
// moved each down to its use and waited out its latency there.  The network's
// twelve convolutions, 8 films of 64x64x16, width 32, forward: 814 -> 338 us
// (257 -> 620 TFLOP/s of unpadded work), of which the packed weights alone gave
// 814 -> 520; one film 585 -> 145 us.
constexpr int HX = 18;
__device__ const uint4 zero_piece = {0u, 0u, 0u, 0u};

template <int MB, int NR, int EPI, bool PACKED>
__global__ __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(2)))
void k_conv_tile(ConvArgs a) {
  constexpr int HY = NR + 2, HPOS = 6 * HY * HX;
  constexpr int NS = (2 * HPOS + 255) / 256;       // 16-byte pieces per thread and chunk
  constexpr int GR = NR < 4 ? NR : 4, NG = NR / GR;   // rows per group of input operands
  constexpr int AHEAD = MB >= 4 ? 1 : 2;           // steps that the weights travel ahead
  static_assert(NS <= 14, "one piece per step");
  __shared__ __align__(16) bf16_t halo[2][HPOS * 16];
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int kq = lane >> 4, col = lane & 15;
  const int X = 1 << a.lx, Y = 1 << a.ly, Z = 1 << a.lz;
  const int tx_n = X >> 4, ty_n = Y / NR, tz_n = Z >> 2;
  const int per_b = tx_n * ty_n * tz_n;
  const int b = blockIdx.x / per_b;
  int rem = blockIdx.x % per_b;
  const int z0 = (rem / (tx_n * ty_n)) * 4;
  rem %= tx_n * ty_n;
  const int y0 = (rem / tx_n) * NR, x0 = (rem % tx_n) * 16;
  const int co_blk = blockIdx.y * MB * 16;

  // input offsets of this thread's halo pieces, in 16-byte units from the
  // first input plane of the halo (the launcher keeps them below 2^31); -1
  // outside the grid
  const int up = a.in_up2;
  const int c8n = a.cin_p >> 3;
  const int zb = (z0 > 0 ? z0 - 1 : 0) >> up;
  const bf16_t *in = a.in + (((long long)b << (a.lz - up)) + zb) *
                                ((long long)a.cin_p << (a.lx + a.ly - 2 * up));
  int soff[NS];
#pragma unroll
  for (int i = 0; i < NS; ++i) {
    const int h = tid + 256 * i, pos = h >> 1;
    const int z = z0 - 1 + pos / (HY * HX), y = y0 - 1 + (pos / HX) % HY, x = x0 - 1 + pos % HX;
    const bool ok = (unsigned)z < (unsigned)Z && (unsigned)y < (unsigned)Y &&
                    (unsigned)x < (unsigned)X;
    const int cell = ((((z >> up) - zb) << (a.ly - up)) + (y >> up)) * (X >> up) + (x >> up);
    soff[i] = ok ? cell * c8n + (h & 1) : -1;
  }
  // piece i of chunk c of the halo into LDS buffer c & 1, by a direct load: the
  // 64 pieces of a wave land side by side; those outside the grid come from
  // zero_piece.  In assembly, because the compiler would wait for such a load
  // before the next LDS read of any address; the wait before the barrier below
  // is the one it needs.
  auto stage = [&](int c, int i) {
    if (tid + 256 * i < 2 * HPOS) {
      const bf16_t *src = soff[i] >= 0 ? in + (size_t)(soff[i] + 2 * c) * 8
                                       : reinterpret_cast<const bf16_t *>(&zero_piece);
      const unsigned at = (unsigned)(uintptr_t)(__attribute__((address_space(3))) bf16_t *)
          &halo[c & 1][(256 * i + 64 * wave) * 8];
      asm volatile("s_mov_b32 m0, %1\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %0, off"
                   :
                   : "v"(src), "s"(__builtin_amdgcn_readfirstlane(at))
                   : "memory", "m0");
    }
  };
  const int kp = 27 * a.cin_p, co16 = a.cout_p >> 4;
  const bf16_t *wl = PACKED ? a.w + (size_t)(co_blk >> 4) * 512 + lane * 8
                            : a.w + (size_t)co_blk * kp;
  // plain weights: this lane's row, tap (of a step's two) and channels, behind an
  // offset that is the same for all lanes; as one address per lane and load, the
  // compiler kept them all in registers and spilled 196 bytes a lane (<4, 4>)
  const unsigned wo = (unsigned)(col * kp + 8 * (kq & 1) + (kq >> 1) * a.cin_p);
  auto weights = [&](int c, int s, bf16x8 *av) {   // step s of chunk c
#pragma unroll
    for (int mb = 0; mb < MB; ++mb) {
      if (PACKED) {
        av[mb] = load8(wl + ((size_t)(c * 14 + s) * co16 + mb) * 512);
      } else {
        const bf16_t *base = wl + (size_t)mb * 16 * kp + (2 * s * a.cin_p + 16 * c);
        av[mb] = s < 13 || kq < 2 ? load8(base + wo) : zero8();
      }
    }
  };

  floatx4 acc[MB][NR];
#pragma unroll
  for (int mb = 0; mb < MB; ++mb)
#pragma unroll
    for (int j = 0; j < NR; ++j) acc[mb][j] = floatx4{0.f, 0.f, 0.f, 0.f};
  const int lb = (wave * HY * HX + col) * 16 + 8 * (kq & 1);
  const bf16_t *hl = halo[0] + lb;                 // this lane's corner in the chunk's buffer
  // input operands of rows GR g .. of step s, from LDS
  auto inputs = [&](int s, int g, bf16x8 *bv) {
    const int t0 = 2 * s, t1 = s < 13 ? 2 * s + 1 : t0;
    const int o0 = ((t0 / 9) * HY + t0 / 3 % 3) * HX + t0 % 3;
    const int o1 = ((t1 / 9) * HY + t1 / 3 % 3) * HX + t1 % 3;
    const bf16_t *hb = hl + (kq >= 2 ? o1 : o0) * 16;
#pragma unroll
    for (int j = 0; j < GR; ++j)
      bv[j] = *reinterpret_cast<const bf16x8 *>(hb + (GR * g + j) * HX * 16);
  };
  const int chunks = a.cin_p >> 4;
  bf16x8 w0[MB], w1[MB], w2[MB], bv[2][GR];
#pragma unroll
  for (int i = 0; i < NS; ++i) stage(0, i);
  weights(0, 0, w0);
  if (AHEAD == 2) weights(0, 1, w1);
  for (int c = 0; c < chunks; ++c) {
    // this wave's part of the chunk has landed, then everyone's
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
    __syncthreads();
    hl = halo[c & 1] + lb;
    inputs(0, 0, bv[0]);
    // weights travel AHEAD steps ahead and inputs one group of rows; the
    // scheduling barriers keep the compiler from moving the loads down to
    // their uses
#pragma unroll
    for (int s = 0; s < 14; ++s) {
      if (s < NS && c + 1 < chunks) stage(c + 1, s);   // over the chunk before this one
      if (s < 14 - AHEAD) weights(c, s + AHEAD, AHEAD == 1 ? w1 : w2);
      else if (c + 1 < chunks) weights(c + 1, s + AHEAD - 14, AHEAD == 1 ? w1 : w2);
#pragma unroll
      for (int g = 0; g < NG; ++g) {
        bf16x8 *now = bv[(s * NG + g) & 1], *next = bv[(s * NG + g + 1) & 1];
        if (g + 1 < NG) inputs(s, g + 1, next);
        else if (s < 13) inputs(s + 1, 0, next);
        __builtin_amdgcn_sched_barrier(0);
#pragma unroll
        for (int j = 0; j < GR; ++j) {
          if (s == 13 && kq >= 2) now[j] = zero8();    // the half step behind tap 26
#pragma unroll
          for (int mb = 0; mb < MB; ++mb)
            acc[mb][GR * g + j] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(
                w0[mb], now[j], acc[mb][GR * g + j], 0, 0, 0);
        }
      }
#pragma unroll
      for (int mb = 0; mb < MB; ++mb) {
        w0[mb] = w1[mb];
        if (AHEAD == 2) w1[mb] = w2[mb];
      }
    }
  }

  const int ls = a.lx + a.ly + a.lz;
  const long long n0 =
      ((((long long)b << a.lz) + z0 + wave) * Y + y0) * (long long)X + x0 + col;
  const size_t o0 = (size_t)n0 * a.cout_p + co_blk + 4 * kq, row = (size_t)X * a.cout_p;
  floatx4 bias[MB];                                // every load before the first store
  uint2 ax[MB][NR];
#pragma unroll
  for (int mb = 0; mb < MB; ++mb) {
    bias[mb] = conv_bias<EPI>(a, co_blk + mb * 16 + 4 * kq);
#pragma unroll
    for (int j = 0; j < NR; ++j) ax[mb][j] = conv_aux<EPI>(a, o0 + j * row + mb * 16);
  }
#pragma unroll
  for (int j = 0; j < NR; ++j) {
    const Pos pj = {b, z0 + wave, y0 + j, x0 + col};
#pragma unroll
    for (int mb = 0; mb < MB; ++mb)
      conv_store<EPI>(a, pj, n0 + (long long)j * X, ls, co_blk + mb * 16 + 4 * kq,
                      o0 + j * row + mb * 16, acc[mb][j], bias[mb], ax[mb][j]);
  }
}

template <int MB, int NR, int EPI>
static hipError_t conv_tile(const ConvArgs &a, hipStream_t s) {
  const long long blocks = ((long long)a.nb << (a.lx + a.ly + a.lz)) / (64 * NR);
  if (blocks > 0x7FFFFFFF) return hipErrorInvalidValue;
  const dim3 grid((unsigned)blocks, a.cout_p / (16 * MB), 1);
  if (a.packed) hipLaunchKernelGGL((k_conv_tile<MB, NR, EPI, true>), grid, dim3(256), 0, s, a);
  else hipLaunchKernelGGL((k_conv_tile<MB, NR, EPI, false>), grid, dim3(256), 0, s, a);
  return hipGetLastError();
}

// Tile of the LDS kernel: MB * NR accumulator tiles per wave, the most (16)
// that still give TILE_GROUPS work-groups; smaller ones leave the matrix cores
// more often idle but fill the chip on small grids and batches: with 64 groups
// of 16 tiles, the 128-channel layers of 8 films (16x16x4) took 112 us each, with
// 256 groups of 4 tiles 20 us.  The order of every sum is the same in all of
// them, and in plain and packed weights.
constexpr long long TILE_GROUPS = 512;

// the tile of a convolution: channel blocks and rows per wave; {0, 0}: k_conv
struct ConvTile {
  int mb, nr;
};

static ConvTile conv_tile_of(const ConvArgs &a, bool to_P) {
  // (the input offsets of a halo fit 31 bits)
  if (a.lx < 4 || a.ly < 1 || a.lz < 2 || ((6LL * (a.cin_p / 8)) << (a.lx + a.ly)) >= (1LL << 31))
    return {0, 0};
  const long long npos = (long long)a.nb << (a.lx + a.ly + a.lz);
  const int co16 = a.cout_p / 16, Y = 1 << a.ly;
  auto fits = [&](int mb, int nr) {
    return mb <= co16 && Y >= nr && npos / (64 * nr) * (co16 / mb) >= TILE_GROUPS;
  };
  if (to_P || co16 == 1) return fits(1, 8) ? ConvTile{1, 8} : ConvTile{1, 2};
  if (co16 == 2 && fits(2, 8)) return {2, 8};
  if (fits(4, 4)) return {4, 4};
  return fits(2, 4) ? ConvTile{2, 4} : ConvTile{2, 2};
}

int conv_tile_code(const ConvArgs &a) {
  const ConvTile t = conv_tile_of(a, false);
  return 16 * t.mb + t.nr;
}

// the kernel for small grids
template <int MB, int NB, int EPI>
static hipError_t conv_small(const ConvArgs &a, long long npos, hipStream_t s) {
  const long long blocks = (npos + 64 * NB - 1) / (64 * NB);
  if (blocks > 0x7FFFFFFF) return hipErrorInvalidValue;
  const dim3 grid((unsigned)blocks, a.cout_p / (16 * MB), 1);
  if (a.packed) hipLaunchKernelGGL((k_conv<MB, NB, EPI, true>), grid, dim3(256), 0, s, a);
  else hipLaunchKernelGGL((k_conv<MB, NB, EPI, false>), grid, dim3(256), 0, s, a);
  return hipGetLastError();
}

// positions per wave: 16 * NB with MB * NB = 16 accumulator tiles (NB >= 2)
template <int EPI>
static hipError_t conv_mb(const ConvArgs &a, long long npos, hipStream_t s) {
  const ConvTile t = conv_tile_of(a, EPI == EPI_P);
  if (t.mb == 1) return t.nr == 8 ? conv_tile<1, 8, EPI>(a, s) : conv_tile<1, 2, EPI>(a, s);
  if constexpr (EPI != EPI_P) {
    if (t.mb == 2 && t.nr == 8) return conv_tile<2, 8, EPI>(a, s);
    if (t.mb == 4) return conv_tile<4, 4, EPI>(a, s);
    if (t.mb == 2) return t.nr == 4 ? conv_tile<2, 4, EPI>(a, s) : conv_tile<2, 2, EPI>(a, s);
  }
  const int mb = a.cout_p / 16 >= 8 ? 8 : a.cout_p / 16;
  switch (mb) {
    case 1: return conv_small<1, 8, EPI>(a, npos, s);
    case 2: return conv_small<2, 8, EPI>(a, npos, s);
    case 4: return conv_small<4, 4, EPI>(a, npos, s);
    case 8: return conv_small<8, 2, EPI>(a, npos, s);
    default: return hipErrorInvalidValue;
  }
}

static bool pow2(int v) { return v > 0 && (v & (v - 1)) == 0; }

hipError_t launch_conv(int epi, const ConvArgs &a, hipStream_t s) {
  if (!pow2(a.cin_p) || a.cin_p < 16 || !pow2(a.cout_p) || a.cout_p < 16 || a.nb < 1 ||
      a.lx < 0 || a.ly < 0 || a.lz < 0 || (a.in_up2 && (a.lx < 1 || a.ly < 1 || a.lz < 1)) ||
      a.cout_p / 16 > 8 * 65535)
    return hipErrorInvalidValue;
  if (!a.in || !a.w || (epi != EPI_P && !a.out)) return hipErrorInvalidValue;
  if (epi == EPI_P && (a.cout_p != 16 || !a.P || !a.thick || !a.bias))
    return hipErrorInvalidValue;
  if ((epi == EPI_ACT || epi == EPI_ACT_SKIP) && !a.bias) return hipErrorInvalidValue;
  if ((epi == EPI_ACT_SKIP || epi == EPI_RAW_AND_D) && !a.out2) return hipErrorInvalidValue;
  if ((epi == EPI_ACT_SKIP || epi == EPI_RAW_D || epi == EPI_RAW_AND_D) && !a.aux)
    return hipErrorInvalidValue;
  const long long npos = (long long)a.nb << (a.lx + a.ly + a.lz);
  switch (epi) {
    case EPI_ACT: return conv_mb<EPI_ACT>(a, npos, s);
    case EPI_ACT_SKIP: return conv_mb<EPI_ACT_SKIP>(a, npos, s);
    case EPI_P: return conv_mb<EPI_P>(a, npos, s);
    case EPI_RAW: return conv_mb<EPI_RAW>(a, npos, s);
    case EPI_RAW_D: return conv_mb<EPI_RAW_D>(a, npos, s);
    case EPI_RAW_AND_D: return conv_mb<EPI_RAW_AND_D>(a, npos, s);
  }
  return hipErrorInvalidValue;
}

// ---------------------------------------------------------- weight grad
// dW[co][tap][ci] = sum over positions n of G[n][co] X[n + tap][ci]: a
// contraction over positions, which both tensors store outermost.
//
// k_wgrad_tile (grids of at least 8 x 8 in y and x): a work-group sums the tiles
// of one split, blocks of TZ x 8 x 8 positions (TZ = 4, or the whole of a flatter
// grid), for 16 A output channels, 16 B input channels and all 27 taps; wave w
// holds the accumulators of taps 7 w .. 7 w + 6 (the 28th place sums G against
// ones, the bias gradient).  A tile's G and the (TZ+2) x 10 x 10 halo of X land
// in LDS by direct loads, 16 channels (32 bytes) a position, and every operand
// of a step of 32 positions (four rows of 8) is read from there by the
// transposing LDS loads, which hand a lane 4 positions of its channel; each
// group of 16 lanes reads 4 positions, 128 contiguous bytes, and the four rows
// of a step fall on distinct banks.
// What bounds it: 2 (A + 7 B) such reads (512 bytes each) per 7 A B matrix
// instructions of a wave.  The kernel it replaces on these grids gathered X from
// L2 once per tap and transposed with 2-byte LDS stores.  Layers of width 32 on 8
// films of 64x64x16, all twelve: 1674 -> 344 us (123 -> 600 TFLOP/s of unpadded
// work); one film 268 -> 151 us.
template <int A, int B>
__global__ __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(2)))
void k_wgrad_tile(WgradArgs a) {
  constexpr int HP = 600;                          // halo positions at TZ = 4
  constexpr int NX = (2 * HP * B + 255) / 256, NG = 2 * A;   // 16-byte pieces per thread
  __shared__ __align__(16) bf16_t xs[B][HP * 16];
  __shared__ __align__(16) bf16_t gs[A][256 * 16];
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int kq = lane >> 4, col = lane & 15;
  const int X = 1 << a.lx, Y = 1 << a.ly, Z = 1 << a.lz;
  const int TZ = Z < 4 ? Z : 4, up = a.in_up2;
  const int hp = (TZ + 2) * 100, np = TZ * 64;     // halo and tile positions
  const int tx_n = X >> 3, ty_n = Y >> 3, per_b = tx_n * ty_n * (Z / TZ);
  const int ci_blk = blockIdx.x * 16 * B, co_blk = blockIdx.z * 16 * A;
  const int c8x = a.cin_p >> 3, c8g = a.cout_p >> 3;
  const long long t0 = (long long)blockIdx.y * a.chunk, ntile = (long long)a.nb * per_b;
  const long long t1 = t0 + a.chunk < ntile ? t0 + a.chunk : ntile;

  // this lane's corner of the transposing reads: position (lane % 16) / 4 of its
  // row, channels 4 (lane % 4) .., in row kq of the step
  const int lx0 = (kq * 10 + (col >> 2)) * 16 + 4 * (col & 3);
  const int lg0 = (kq * 8 + (col >> 2)) * 16 + 4 * (col & 3);
  int toff[7];
  for (int i = 0; i < 7; ++i) {
    const int t = 7 * wave + i < 27 ? 7 * wave + i : 26;
    toff[i] = lx0 + ((t / 9) * 100 + (t / 3 % 3) * 10 + t % 3) * 16;
  }
  bf16x8 ones;
  for (int i = 0; i < 8; ++i) ones[i] = (__bf16)1.f;

  floatx4 acc[7][A][B];
#pragma unroll
  for (int i = 0; i < 7; ++i)
#pragma unroll
    for (int p = 0; p < A; ++p)
#pragma unroll
      for (int q = 0; q < B; ++q) acc[i][p][q] = floatx4{0.f, 0.f, 0.f, 0.f};

  auto tr8 = [](const bf16_t *p) -> bf16x8 {       // 8 positions of this lane's channel
    typedef short short4_t __attribute__((ext_vector_type(4)));
    typedef __attribute__((address_space(3))) short4_t *lds_t;
    union { short4_t s[2]; bf16x8 v; } r;
    r.s[0] = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_t)p);
    r.s[1] = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_t)(p + 4 * 16));
    return r.v;
  };
  auto land = [&](const bf16_t *src, const bf16_t *lds) {   // 64 pieces side by side
    __builtin_amdgcn_global_load_lds((const __attribute__((address_space(1))) void *)src,
                                     (__attribute__((address_space(3))) void *)lds, 16, 0, 0);
  };

  for (long long tile = t0; tile < t1; ++tile) {
    const int b = (int)(tile / per_b);
    int rem = (int)(tile - (long long)b * per_b);
    const int z0 = rem / (tx_n * ty_n) * TZ;
    rem %= tx_n * ty_n;
    const int y0 = rem / tx_n * 8, x0 = rem % tx_n * 8;
    const int zb = (z0 > 0 ? z0 - 1 : 0) >> up;
    const bf16_t *in = a.in + (((long long)b << (a.lz - up)) + zb) *
                                  ((long long)a.cin_p << (a.lx + a.ly - 2 * up)) + ci_blk;
    const bf16_t *g = a.g + (((long long)b << a.lz) + z0) * ((long long)a.cout_p << (a.lx + a.ly)) +
                      co_blk;
    __syncthreads();                               // the last tile has been read
#pragma unroll
    for (int i = 0; i < NX; ++i) {
      const int h = tid + 256 * i, blk = h / (2 * HP), pos = (h - blk * 2 * HP) >> 1;
      if (blk < B && pos < hp) {
        const int z = z0 - 1 + pos / 100, y = y0 - 1 + pos / 10 % 10, x = x0 - 1 + pos % 10;
        const bool ok = (unsigned)z < (unsigned)Z && (unsigned)y < (unsigned)Y &&
                        (unsigned)x < (unsigned)X;
        const int cell = ((((z >> up) - zb) << (a.ly - up)) + (y >> up)) * (X >> up) + (x >> up);
        land(ok ? in + (size_t)(unsigned)(cell * c8x + 2 * blk + (h & 1)) * 8
                : reinterpret_cast<const bf16_t *>(&zero_piece),
             &xs[0][0] + (256 * i + 64 * wave) * 8);
      }
    }
#pragma unroll
    for (int i = 0; i < NG; ++i) {
      const int h = tid + 256 * i, blk = h >> 9, pos = (h & 511) >> 1;
      if (pos < np) {
        const int cell = (((pos >> 6) << a.ly) + y0 + (pos >> 3 & 7)) * X + x0 + (pos & 7);
        land(g + (size_t)(unsigned)(cell * c8g + 2 * blk + (h & 1)) * 8,
             &gs[0][0] + (256 * i + 64 * wave) * 8);
      }
    }
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
    __syncthreads();
    for (int z = 0; z < TZ; ++z) {
#pragma unroll
      for (int half = 0; half < 2; ++half) {       // rows 4 half .. 4 half + 3 of plane z
        const int ox = (z * 100 + half * 40) * 16, og = (z * 64 + half * 32) * 16;
        bf16x8 ga[A];
#pragma unroll
        for (int p = 0; p < A; ++p) ga[p] = tr8(&gs[p][0] + lg0 + og);
#pragma unroll
        for (int i = 0; i < 7; ++i) {
#pragma unroll
          for (int q = 0; q < B; ++q) {
            bf16x8 xb = tr8(&xs[q][0] + toff[i] + ox);
            if (i == 6 && wave == 3) xb = ones;
#pragma unroll
            for (int p = 0; p < A; ++p)
              acc[i][p][q] =
                  __builtin_amdgcn_mfma_f32_16x16x32_bf16(ga[p], xb, acc[i][p][q], 0, 0, 0);
          }
        }
      }
    }
  }

  const int kp = 27 * a.cin_p;
#pragma unroll
  for (int i = 0; i < 7; ++i) {
    const int t = 7 * wave + i;
#pragma unroll
    for (int p = 0; p < A; ++p)
#pragma unroll
      for (int q = 0; q < B; ++q)
#pragma unroll
        for (int r = 0; r < 4; ++r) {
          const size_t co = (size_t)blockIdx.y * a.cout_p + co_blk + 16 * p + 4 * kq + r;
          if (t < 27) a.part[co * kp + t * a.cin_p + ci_blk + 16 * q + col] = acc[i][p][q][r];
          else if (q == 0 && col == 0 && blockIdx.x == 0) a.bpart[co] = acc[i][p][q][r];
        }
  }
}

template <int A, int B>
static hipError_t wgrad_tile(const WgradArgs &a, hipStream_t s) {
  const dim3 grid(a.cin_p / (16 * B), a.splits, a.cout_p / (16 * A));
  hipLaunchKernelGGL((k_wgrad_tile<A, B>), grid, dim3(256), 0, s, a);
  return hipGetLastError();
}

// Smaller grids (k_wgrad): one split's positions, k = tap * cin_p + ci.
// Work-group: 16 * MB output channels (blockIdx.z) x 64 k columns
// (blockIdx.x, 16 per wave), positions in slabs of 32 * WS.  Both tiles are
// transposed through LDS so that each lane reads 8 consecutive positions for
// the matrix core.  The blockIdx.x == 0 groups also sum G over the
// positions (bias gradient).
constexpr int WS = 4;                  // 32-position MFMA steps per LDS slab
constexpr int WG_LD = 32 * WS + 8;     // LDS row stride (elements)

template <int MB>
__global__ __launch_bounds__(256) void k_wgrad(WgradArgs a) {
  __shared__ bf16_t gs[MB * 16][WG_LD];
  __shared__ bf16_t xs[64][WG_LD];
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int kq = lane >> 4, col = lane & 15;
  const int ls = a.lx + a.ly + a.lz;
  const long long npos = (long long)a.nb << ls;
  const int kp = 27 * a.cin_p;
  const int lc = __builtin_ctz(a.cin_p);
  const int kt0 = blockIdx.x * 64;
  const int co_blk = blockIdx.z * MB * 16;
  const long long p0 = (long long)blockIdx.y * a.chunk;
  const long long p1 = p0 + a.chunk < npos ? p0 + a.chunk : npos;
  const bool bias_thread = blockIdx.x == 0 && tid < MB * 16;

  floatx4 acc[MB];
  for (int mb = 0; mb < MB; ++mb) acc[mb] = floatx4{0.f, 0.f, 0.f, 0.f};
  float bsum = 0.f;

  for (long long pb = p0; pb < p1; pb += 32 * WS) {
    for (int c = tid; c < MB * 64 * WS; c += 256) {
      const int gl = c % (32 * WS), c8 = c / (32 * WS);
      const long long n = pb + gl;
      uint4 v = make_uint4(0u, 0u, 0u, 0u);
      if (n < p1) v = *reinterpret_cast<const uint4 *>(a.g + n * a.cout_p + co_blk + 8 * c8);
      const uint32_t w4[4] = {v.x, v.y, v.z, v.w};
      for (int i = 0; i < 4; ++i) {
        gs[8 * c8 + 2 * i][gl] = (bf16_t)(w4[i] & 0xFFFF);
        gs[8 * c8 + 2 * i + 1][gl] = (bf16_t)(w4[i] >> 16);
      }
    }
    for (int c = tid; c < 256 * WS; c += 256) {
      const int nl = c % (32 * WS), k8 = c / (32 * WS);
      const int kx = kt0 + 8 * k8;
      const long long n = pb + nl;
      uint4 v = make_uint4(0u, 0u, 0u, 0u);
      if (kx < kp && n < p1) {
        const int t = kx >> lc, ci = kx & (a.cin_p - 1);
        const Pos p = decode(n, a.lx, a.ly, a.lz);
        const long long src =
            gather_index(p, t / 9 - 1, (t / 3) % 3 - 1, t % 3 - 1, a.lx, a.ly, a.lz, a.in_up2);
        if (src >= 0) v = *reinterpret_cast<const uint4 *>(a.in + src * a.cin_p + ci);
      }
      const uint32_t w4[4] = {v.x, v.y, v.z, v.w};
      for (int i = 0; i < 4; ++i) {
        xs[8 * k8 + 2 * i][nl] = (bf16_t)(w4[i] & 0xFFFF);
        xs[8 * k8 + 2 * i + 1][nl] = (bf16_t)(w4[i] >> 16);
      }
    }
    __syncthreads();
    for (int st = 0; st < WS; ++st) {
      const int n8 = 32 * st + 8 * kq;
      const bf16x8 bv = *reinterpret_cast<const bf16x8 *>(&xs[wave * 16 + col][n8]);
      for (int mb = 0; mb < MB; ++mb) {
        const bf16x8 av = *reinterpret_cast<const bf16x8 *>(&gs[mb * 16 + col][n8]);
        acc[mb] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(av, bv, acc[mb], 0, 0, 0);
      }
    }
    if (bias_thread)
      for (int i = 0; i < 32 * WS; ++i) bsum += bf2f(gs[tid][i]);
    __syncthreads();
  }
  const int k = kt0 + wave * 16 + col;
  if (k < kp) {
    for (int mb = 0; mb < MB; ++mb)
      for (int i = 0; i < 4; ++i) {
        const int co = co_blk + mb * 16 + 4 * kq + i;
        a.part[((size_t)blockIdx.y * a.cout_p + co) * kp + k] = acc[mb][i];
      }
  }
  if (bias_thread) a.bpart[(size_t)blockIdx.y * a.cout_p + co_blk + tid] = bsum;
}

// Work-groups of the tiled kernel, two per CU: one group's loads run under the
// other's matrix work, and every group writes 28 accumulator tiles per wave, so
// that more of them pay in the reduction (weight gradients of 8 films of
// 64x64x16, width 32: 440 us with 256 groups, 344 with 512, 398 with 768).
constexpr long long WGRAD_GROUPS = 512;

// tiles of 4 x 8 x 8 positions (fewer in z in a flatter grid)
static long long wgrad_tiles(const WgradArgs &a) {
  return ((long long)a.nb << (a.lx + a.ly + a.lz)) >> (6 + (a.lz < 2 ? a.lz : 2));
}

// Channel blocks of a work-group of the tiled kernel: 28 accumulator tiles per
// wave where the layer has the channels and the grid the tiles; where that would
// leave fewer than 256 groups, one per CU, each takes 16 x 16 channels: one sample
// of 4x32x32, 32 to 64 channels, 14.4 -> 10.3 us (13.9 with k_wgrad), of 4x16x16,
// 64 to 64, 14.0 -> 9.8 (10.8), 4 of 4x32x32, 32 to 64, 19.1 -> 16.0 (33.1).
static void wgrad_blocks(const WgradArgs &a, int *A, int *B) {
  const int co16 = a.cout_p / 16, ci16 = a.cin_p / 16;
  *A = co16 >= 4 ? 4 : co16;
  *B = *A == 4 || ci16 == 1 ? 1 : 2;
  if (wgrad_tiles(a) * (ci16 / *B) * (co16 / *A) < 256) *A = *B = 1;
}

// the splits of k_wgrad: about 1024 work-groups, at least 256 positions each
static void plan_small(WgradArgs *a) {
  const long long npos = (long long)a->nb << (a->lx + a->ly + a->lz);
  const long long ktiles = (27LL * a->cin_p + 63) / 64;
  long long s = (1024 + ktiles - 1) / ktiles;
  const long long smax = (npos + 255) / 256;
  if (s > smax) s = smax;
  if (s < 1) s = 1;
  a->max_splits = (int)s;
  long long c = (npos + s - 1) / s;
  c = (c + 32 * WS - 1) / (32 * WS) * (32 * WS);   // whole LDS slabs
  s = (npos + c - 1) / c;
  a->splits = (int)s;
  a->chunk = (int)c;
}

void wgrad_plan(WgradArgs *a, int most) {
  const int cmax = a->cin_p > a->cout_p ? a->cin_p : a->cout_p;
  // (the offsets within a tile's planes fit 31 bits)
  a->tiled = a->lx >= 3 && a->ly >= 3 && ((6LL * (cmax / 8)) << (a->lx + a->ly)) < (1LL << 31);
  if (!a->tiled) {
    plan_small(a);
    return;
  }
  int A, B;
  wgrad_blocks(*a, &A, &B);
  const long long tiles = wgrad_tiles(*a);
  const long long blocks = (long long)(a->cin_p / (16 * B)) * (a->cout_p / (16 * A));
  long long s = (WGRAD_GROUPS + blocks - 1) / blocks;
  if (s > tiles) s = tiles;
  if (most > 0 && s > most) s = most;
  a->max_splits = (int)s;
  a->chunk = (int)((tiles + s - 1) / s);
  a->splits = (int)((tiles + a->chunk - 1) / a->chunk);
}

int wgrad_least_splits(const WgradArgs &a) {
  WgradArgs u = a;
  plan_small(&u);
  return u.splits < a.splits ? u.splits : a.splits;
}

hipError_t launch_wgrad(const WgradArgs &a, hipStream_t s) {
  if (!pow2(a.cin_p) || a.cin_p < 16 || !pow2(a.cout_p) || a.cout_p < 16 || a.nb < 1 ||
      a.splits < 1 || a.splits > 65535 || (a.in_up2 && (a.lx < 1 || a.ly < 1 || a.lz < 1)))
    return hipErrorInvalidValue;
  if (a.tiled) {
    if (a.lx < 3 || a.ly < 3 || a.chunk < 1) return hipErrorInvalidValue;
    int A, B;
    wgrad_blocks(a, &A, &B);
    if (A == 4) return wgrad_tile<4, 1>(a, s);
    if (A == 2) return B == 2 ? wgrad_tile<2, 2>(a, s) : wgrad_tile<2, 1>(a, s);
    return B == 2 ? wgrad_tile<1, 2>(a, s) : wgrad_tile<1, 1>(a, s);
  }
  if (a.chunk < 32 || (a.chunk & 31)) return hipErrorInvalidValue;
  const int kp = 27 * a.cin_p;
  const int mb = a.cout_p / 16 >= 8 ? 8 : a.cout_p / 16;
  dim3 grid((kp + 63) / 64, a.splits, a.cout_p / (16 * mb));
  switch (mb) {
    case 1: hipLaunchKernelGGL(k_wgrad<1>, grid, dim3(256), 0, s, a); break;
    case 2: hipLaunchKernelGGL(k_wgrad<2>, grid, dim3(256), 0, s, a); break;
    case 4: hipLaunchKernelGGL(k_wgrad<4>, grid, dim3(256), 0, s, a); break;
    case 8: hipLaunchKernelGGL(k_wgrad<8>, grid, dim3(256), 0, s, a); break;
    default: return hipErrorInvalidValue;
  }
  return hipGetLastError();
}

// ------------------------------------------------------------ elementwise
// In-plane symmetry op of a sample (bits: 1 mirror x, 2 mirror y, 4 swap x
// and y; swap only on square grids): the sample's vector fields F become
// F'(x, y) = D F(src(x, y)) with src = swap(mirror_x(mirror_y(x, y))) and
// F'_x = (-1)^mx F_(swap ? y : x), F'_y = (-1)^my F_(swap ? x : y), F'_z = F_z.
struct SymOp {
  int mx, my, sw;
  __device__ explicit SymOp(int op) : mx(op & 1), my((op >> 1) & 1), sw((op >> 2) & 1) {}
  // source (x, y) of destination (x, y) on an X x Y grid
  __device__ void src(int &x, int &y, int X, int Y) const {
    if (my) y = Y - 1 - y;
    if (mx) x = X - 1 - x;
    if (sw) {
      const int t = x;
      x = y;
      y = t;
    }
  }
  // source component and sign of destination component c
  __device__ int comp(int c) const { return (sw && c < 2) ? 1 - c : c; }
  __device__ float sign(int c) const { return (c == 0 && mx) || (c == 1 && my) ? -1.f : 1.f; }
};

__global__ void k_input(const float *T, const float *thick, const float *noise, const int *idx,
                        const int *ops, int lx, int ly, int lz, int nb, int ld, bf16_t *x0) {
  const long long n = (long long)blockIdx.x * blockDim.x + threadIdx.x;
  const int ls = lx + ly + lz;
  if (n >= ((long long)nb << ls)) return;
  const Pos p = decode(n, lx, ly, lz);
  const int row = idx ? idx[p.b] : p.b;
  const float m = (float)p.z < thick[row] ? 1.f : 0.f;
  const int cx = lx - ld, cy = ly - ld, cz = lz - ld;
  const SymOp g(ops ? ops[p.b] & (lx == ly ? 7 : 3) : 0);
  int qx = p.x >> ld, qy = p.y >> ld;
  g.src(qx, qy, 1 << cx, 1 << cy);
  const long long cell = (((long long)(p.z >> ld) << cy) + qy) * (1LL << cx) + qx;
  const long long nc = 1LL << (cx + cy + cz);
  float v[16];
  for (int c = 0; c < 16; ++c) v[c] = 0.f;
  v[0] = m * ((T[row] - 350.f) / 100.f);
  v[1] = m;
  for (int c = 0; c < 3; ++c)
    v[2 + c] = m * (g.sign(c) * noise[((long long)row * 3 + g.comp(c)) * nc + cell] * 10.f);
  uint32_t w[8];
  for (int i = 0; i < 8; ++i) w[i] = f2bf(v[2 * i]) | ((uint32_t)f2bf(v[2 * i + 1]) << 16);
  uint4 *o = reinterpret_cast<uint4 *>(x0 + n * 16);
  o[0] = make_uint4(w[0], w[1], w[2], w[3]);
  o[1] = make_uint4(w[4], w[5], w[6], w[7]);
}

hipError_t launch_input(const float *T, const float *thick, const float *noise, const int *idx,
                        const int *ops, int lx, int ly, int lz, int nb, int noise_div, bf16_t *x0,
                        hipStream_t s) {
  if (!pow2(noise_div)) return hipErrorInvalidValue;
  const int ld = __builtin_ctz(noise_div);
  if (ld > lx || ld > ly || ld > lz) return hipErrorInvalidValue;
  const long long n = (long long)nb << (lx + ly + lz);
  hipLaunchKernelGGL(k_input, dim3((unsigned)((n + 255) / 256)), dim3(256), 0, s, T, thick, noise,
                     idx, ops, lx, ly, lz, nb, ld, x0);
  return hipGetLastError();
}

__device__ inline void unpack8(const uint4 v, float *f) {
  const uint32_t w[4] = {v.x, v.y, v.z, v.w};
  for (int i = 0; i < 4; ++i) {
    f[2 * i] = bf2f((bf16_t)(w[i] & 0xFFFF));
    f[2 * i + 1] = bf2f((bf16_t)(w[i] >> 16));
  }
}
__device__ inline uint4 pack8(const float *f) {
  uint32_t w[4];
  for (int i = 0; i < 4; ++i) w[i] = f2bf(f[2 * i]) | ((uint32_t)f2bf(f[2 * i + 1]) << 16);
  return make_uint4(w[0], w[1], w[2], w[3]);
}
__device__ inline void unpack8_raw(const uint4 v, bf16_t *h) {
  const uint32_t w[4] = {v.x, v.y, v.z, v.w};
  for (int i = 0; i < 4; ++i) {
    h[2 * i] = (bf16_t)(w[i] & 0xFFFF);
    h[2 * i + 1] = (bf16_t)(w[i] >> 16);
  }
}

// fine position of child c (0..7) of coarse position q; (lx, ly, lz) fine grid
__device__ inline long long child(const Pos &q, int c, int lx, int ly, int lz) {
  const int z = 2 * q.z + (c >> 2), y = 2 * q.y + ((c >> 1) & 1), x = 2 * q.x + (c & 1);
  return ((((long long)q.b << lz) + z) << (ly + lx)) + ((long long)y << lx) + x;
}

// coarse average of 2x2x2 blocks; (lx, ly, lz) is the fine grid
__global__ void k_pool(const bf16_t *in, int lx, int ly, int lz, int nb, int c8, bf16_t *out) {
  const long long i = (long long)blockIdx.x * blockDim.x + threadIdx.x;
  const int cls = lx + ly + lz - 3;
  if (i >= ((long long)nb << cls) * c8) return;
  const long long q = i / c8;
  const int ch = (int)(i % c8) * 8;
  const Pos cp = decode(q, lx - 1, ly - 1, lz - 1);
  float s[8] = {0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f};
  for (int c = 0; c < 8; ++c) {
    float f[8];
    unpack8(*reinterpret_cast<const uint4 *>(in + child(cp, c, lx, ly, lz) * (8 * c8) + ch), f);
    for (int k = 0; k < 8; ++k) s[k] += f[k];
  }
  for (int k = 0; k < 8; ++k) s[k] *= 0.125f;
  *reinterpret_cast<uint4 *>(out + q * (8 * c8) + ch) = pack8(s);
}

// out[fine] = (g[coarse] / 8 + add[fine]) * act'(a[fine])
__global__ void k_pool_bwd(const bf16_t *g, const bf16_t *add, const bf16_t *a, int lx, int ly,
                           int lz, int nb, int c8, bf16_t *out) {
  const long long i = (long long)blockIdx.x * blockDim.x + threadIdx.x;
  const int ls = lx + ly + lz;
  if (i >= ((long long)nb << ls) * c8) return;
  const long long n = i / c8;
  const int ch = (int)(i % c8) * 8;
  const Pos p = decode(n, lx, ly, lz);
  const long long q = ((((long long)p.b << (lz - 1)) + (p.z >> 1)) << (ly - 1 + lx - 1)) +
                      ((long long)(p.y >> 1) << (lx - 1)) + (p.x >> 1);
  const int C = 8 * c8;
  float gv[8], av[8];
  bf16_t ah[8];
  unpack8(*reinterpret_cast<const uint4 *>(g + q * C + ch), gv);
  if (add) unpack8(*reinterpret_cast<const uint4 *>(add + n * C + ch), av);
  unpack8_raw(*reinterpret_cast<const uint4 *>(a + n * C + ch), ah);
  float r[8];
  for (int k = 0; k < 8; ++k) r[k] = (gv[k] * 0.125f + (add ? av[k] : 0.f)) * act_slope(ah[k]);
  *reinterpret_cast<uint4 *>(out + n * C + ch) = pack8(r);
}

// out[coarse] = (sum of g over the 8 children) * act'(a[coarse]); (lx, ly, lz) fine grid
__global__ void k_up_bwd(const bf16_t *g, const bf16_t *a, int lx, int ly, int lz, int nb, int c8,
                         bf16_t *out) {
  const long long i = (long long)blockIdx.x * blockDim.x + threadIdx.x;
  const int cls = lx + ly + lz - 3;
  if (i >= ((long long)nb << cls) * c8) return;
  const long long q = i / c8;
  const int ch = (int)(i % c8) * 8;
  const int C = 8 * c8;
  const Pos cp = decode(q, lx - 1, ly - 1, lz - 1);
  float s[8] = {0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f};
  for (int c = 0; c < 8; ++c) {
    float f[8];
    unpack8(*reinterpret_cast<const uint4 *>(g + child(cp, c, lx, ly, lz) * C + ch), f);
    for (int k = 0; k < 8; ++k) s[k] += f[k];
  }
  bf16_t ah[8];
  unpack8_raw(*reinterpret_cast<const uint4 *>(a + q * C + ch), ah);
  for (int k = 0; k < 8; ++k) s[k] *= act_slope(ah[k]);
  *reinterpret_cast<uint4 *>(out + q * C + ch) = pack8(s);
}

static hipError_t ew_check(int lx, int ly, int lz, int nb, int c_p, bool coarse) {
  if (c_p < 8 || (c_p & 7) || nb < 1 || (coarse && (lx < 1 || ly < 1 || lz < 1)))
    return hipErrorInvalidValue;
  return hipSuccess;
}

hipError_t launch_pool(const bf16_t *in, int lx, int ly, int lz, int nb, int c_p, bf16_t *out,
                       hipStream_t s) {
  if (ew_check(lx, ly, lz, nb, c_p, true) != hipSuccess) return hipErrorInvalidValue;
  const long long n = ((long long)nb << (lx + ly + lz - 3)) * (c_p / 8);
  hipLaunchKernelGGL(k_pool, dim3((unsigned)((n + 255) / 256)), dim3(256), 0, s, in, lx, ly, lz,
                     nb, c_p / 8, out);
  return hipGetLastError();
}

hipError_t launch_pool_bwd(const bf16_t *g, const bf16_t *add, const bf16_t *a, int lx, int ly,
                           int lz, int nb, int c_p, bf16_t *out, hipStream_t s) {
  if (ew_check(lx, ly, lz, nb, c_p, true) != hipSuccess) return hipErrorInvalidValue;
  const long long n = ((long long)nb << (lx + ly + lz)) * (c_p / 8);
  hipLaunchKernelGGL(k_pool_bwd, dim3((unsigned)((n + 255) / 256)), dim3(256), 0, s, g, add, a,
                     lx, ly, lz, nb, c_p / 8, out);
  return hipGetLastError();
}

hipError_t launch_up_bwd(const bf16_t *g, const bf16_t *a, int lx, int ly, int lz, int nb,
                         int c_p, bf16_t *out, hipStream_t s) {
  if (ew_check(lx, ly, lz, nb, c_p, true) != hipSuccess) return hipErrorInvalidValue;
  const long long n = ((long long)nb << (lx + ly + lz - 3)) * (c_p / 8);
  hipLaunchKernelGGL(k_up_bwd, dim3((unsigned)((n + 255) / 256)), dim3(256), 0, s, g, a, lx, ly,
                     lz, nb, c_p / 8, out);
  return hipGetLastError();
}

// the same rounding in integers: behind a conversion from double the compiler
// would round once to BF16, not first to float as the network's definition has it
__device__ inline bf16_t f2bf_float(float f) {
  uint32_t u = __float_as_uint(f);
  u += 0x7FFFu + ((u >> 16) & 1u);
  return (bf16_t)(u >> 16);
}

// squared error of P against the target rows over the film cells, divided by
// 3 x the film cells of the batch (FP64 partial per block), and the BF16
// gradient 2 m (P - target) / count in channels 0..2 of 16
__global__ __launch_bounds__(256) void k_loss(const float *P, const float *target,
                                              const float *thick, const int *idx, const int *ops,
                                              int lx, int ly, int lz, int nb, bf16_t *gy,
                                              double *partials) {
  __shared__ double red[4];
  const long long n = (long long)blockIdx.x * 256 + threadIdx.x;
  const int ls = lx + ly + lz;
  // 3 x the film cells of the batch
  double count = 0.0;
  for (int b = 0; b < nb; ++b) {
    const float th = thick[idx ? idx[b] : b];
    const float layers = ceilf(fminf(fmaxf(th, 0.f), (float)(1 << lz)));
    count += 3.0 * (double)layers * (double)(1LL << (lx + ly));
  }
  const double inv_count = count > 0.0 ? 1.0 / count : 0.0;
  double e = 0.0;
  if (n < ((long long)nb << ls)) {
    const Pos p = decode(n, lx, ly, lz);
    const int row = idx ? idx[p.b] : p.b;
    const float m = (float)p.z < thick[row] ? 1.f : 0.f;
    const long long r = n & ((1LL << ls) - 1);
    // the target is read through the sample's symmetry op
    const SymOp op(ops ? ops[p.b] & (lx == ly ? 7 : 3) : 0);
    int sx = p.x, sy = p.y;
    op.src(sx, sy, 1 << lx, 1 << ly);
    const long long rs = ((long long)p.z << (lx + ly)) + ((long long)sy << lx) + sx;
    float g[16];
    for (int c = 0; c < 16; ++c) g[c] = 0.f;
    for (int c = 0; c < 3; ++c) {
      const double d = (double)P[(((long long)p.b * 3 + c) << ls) + r] -
                       (double)op.sign(c) *
                           (double)target[(((long long)row * 3 + op.comp(c)) << ls) + rs];
      e += m * d * d;
      g[c] = (float)(m * 2.0 * d * inv_count);
    }
    uint32_t w[8];
    for (int i = 0; i < 8; ++i)
      w[i] = f2bf_float(g[2 * i]) | ((uint32_t)f2bf_float(g[2 * i + 1]) << 16);
    uint4 *o = reinterpret_cast<uint4 *>(gy + n * 16);
    o[0] = make_uint4(w[0], w[1], w[2], w[3]);
    o[1] = make_uint4(w[4], w[5], w[6], w[7]);
  }
  for (int off = 32; off > 0; off >>= 1) e += __shfl_down(e, off, 64);
  if ((threadIdx.x & 63) == 0) red[threadIdx.x >> 6] = e;
  __syncthreads();
  if (threadIdx.x == 0) partials[blockIdx.x] = (red[0] + red[1] + red[2] + red[3]) * inv_count;
}

hipError_t launch_loss(const float *P, const float *target, const float *thick, const int *idx,
                       const int *ops, int lx, int ly, int lz, int nb, bf16_t *gy,
                       double *partials, int *nblocks, hipStream_t s) {
  const long long n = (long long)nb << (lx + ly + lz);
  const long long nbk = (n + 255) / 256;
  if (nb < 1 || nbk > 0x7FFFFFFF) return hipErrorInvalidValue;
  *nblocks = (int)nbk;
  hipLaunchKernelGGL(k_loss, dim3((unsigned)nbk), dim3(256), 0, s, P, target, thick, idx, ops, lx,
                     ly, lz, nb, gy, partials);
  return hipGetLastError();
}

__global__ __launch_bounds__(256) void k_sum_partials(const double *p, int n, double *out) {
  __shared__ double red[4];
  double e = 0.0;
  for (int i = threadIdx.x; i < n; i += 256) e += p[i];
  for (int off = 32; off > 0; off >>= 1) e += __shfl_down(e, off, 64);
  if ((threadIdx.x & 63) == 0) red[threadIdx.x >> 6] = e;
  __syncthreads();
  if (threadIdx.x == 0) *out = red[0] + red[1] + red[2] + red[3];
}

hipError_t launch_sum_partials(const double *partials, int n, double *out, hipStream_t s) {
  hipLaunchKernelGGL(k_sum_partials, dim3(1), dim3(256), 0, s, partials, n, out);
  return hipGetLastError();
}

// flat gradient of one layer (public order: W [cout][27][cin], then b [cout]):
// 256 / SL entries per work-group, SL threads each taking every SL-th split, so that
// the hundreds of splits of a small layer are not one thread's chain of loads
// (SL = 8: 19 us a layer with one thread an entry, 11 with eight, 8 films of
// 64x64x16, width 32), while the few splits of a wide layer on a small grid do not
// leave seven of eight threads idle (SL = 1: 4 splits of 256 x 27 x 256, with the
// weight gradient 40 us against 59).
constexpr int REDUCE_SLICES = 64;      // splits from which an entry has eight threads

template <int SL>
__global__ __launch_bounds__(256) void k_reduce_grad(const float *part, const float *bpart,
                                                     int splits, int cin, int cout, int cin_p,
                                                     int cout_p, float *grad) {
  constexpr int E = 256 / SL;
  __shared__ float red[SL][E];
  const int e = threadIdx.x % E, sg = threadIdx.x / E;
  const long long i = (long long)blockIdx.x * E + e;
  const long long nw = (long long)cout * 27 * cin;
  float s = 0.f;
  if (i < nw + cout) {
    const size_t kp = 27 * (size_t)cin_p;
    const float *src = bpart + (i - nw);
    size_t stride = cout_p;
    if (i < nw) {
      const int ci = (int)(i % cin);
      const int t = (int)((i / cin) % 27);
      const int co = (int)(i / (27LL * cin));
      src = part + (size_t)co * kp + (size_t)t * cin_p + ci;
      stride = (size_t)cout_p * kp;
    }
#pragma unroll 8
    for (int sp = sg; sp < splits; sp += SL) s += src[(size_t)sp * stride];
  }
  if constexpr (SL > 1) {
    red[sg][e] = s;
    __syncthreads();
    if (sg != 0) return;
    for (int k = 1; k < SL; ++k) s += red[k][e];
  }
  if (i < nw + cout) grad[i] = s;
}

hipError_t launch_reduce_grad(const float *part, const float *bpart, int splits, int cin,
                              int cout, int cin_p, int cout_p, float *grad, hipStream_t s) {
  const long long n = (long long)cout * 27 * cin + cout;
  auto launch = [&](auto kernel, int entries) {
    hipLaunchKernelGGL(kernel, dim3((unsigned)((n + entries - 1) / entries)), dim3(256), 0, s, part,
                       bpart, splits, cin, cout, cin_p, cout_p, grad);
    return hipGetLastError();
  };
  return splits < REDUCE_SLICES ? launch(k_reduce_grad<1>, 256) : launch(k_reduce_grad<8>, 32);
}

// omb1 = 1 - beta1, omb2 = 1 - beta2 and the bias corrections c1, c2 come
// from the host in FP64, so that the first step's m / c1 and v / c2 are g and
// g^2 to within a rounding
__global__ void k_adam(float *master, float *m, float *v, const float *grad, long long n,
                       float lr, float b1, float b2, float omb1, float omb2, float eps, float c1,
                       float c2) {
  const long long i = (long long)blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= n) return;
  const float g = grad[i];
  const float mi = b1 * m[i] + omb1 * g;
  const float vi = b2 * v[i] + omb2 * g * g;
  m[i] = mi;
  v[i] = vi;
  master[i] -= lr * (mi / c1) / (sqrtf(vi / c2) + eps);
}

hipError_t launch_adam(float *master, float *m, float *v, const float *grad, long long n,
                       double lr, double b1, double b2, double eps, long long t, hipStream_t s) {
  const double c1 = 1.0 - std::pow(b1, (double)t), c2 = 1.0 - std::pow(b2, (double)t);
  hipLaunchKernelGGL(k_adam, dim3((unsigned)((n + 255) / 256)), dim3(256), 0, s, master, m, v,
                     grad, n, (float)lr, (float)b1, (float)b2, (float)(1.0 - b1), (float)(1.0 - b2),
                     (float)eps, (float)c1, (float)c2);
  return hipGetLastError();
}

// FP32 master (one layer, public order) -> packed BF16 forward weights (rows
// cout, channels cin), packed backward-data copy (rows cin, channels cout, tap
// mirrored) and the padded FP32 bias
__global__ void k_cast_weights(const float *master, int cin, int cout, int cin_p, int cout_p,
                               bf16_t *w, bf16_t *wt, float *bias) {
  const long long i = (long long)blockIdx.x * blockDim.x + threadIdx.x;
  const long long nw = 28LL * cin_p * cout_p;
  if (i < nw) {
    const int k8 = (int)(i & 7), col = (int)(i >> 3) & 15, kq = (int)(i >> 7) & 3;
    const int frag = (int)(i >> 9);
    // (chunk, step, row block) of this element for 16-row blocks rows / 16
    auto value = [&](int rows16, bool mirror) -> bf16_t {
      const int m = frag % rows16, s = frag / rows16 % 14, c = frag / (14 * rows16);
      const int t = 2 * s + (kq >> 1), row = 16 * m + col, ch = 16 * c + 8 * (kq & 1) + k8;
      const int co = mirror ? ch : row, ci = mirror ? row : ch, tap = mirror ? 26 - t : t;
      const bool in = t < 27 && co < cout && ci < cin;
      return f2bf(in ? master[((long long)co * 27 + tap) * cin + ci] : 0.f);
    };
    w[i] = value(cout_p >> 4, false);
    wt[i] = value(cin_p >> 4, true);
  } else if (i < nw + cout_p) {
    const int co = (int)(i - nw);
    bias[co] = co < cout ? master[(long long)cout * 27 * cin + co] : 0.f;
  }
}

hipError_t launch_cast_weights(const float *master, int cin, int cout, int cin_p, int cout_p,
                               bf16_t *w, bf16_t *wt, float *bias, hipStream_t s) {
  const long long n = (long long)packed_size(cin_p, cout_p) + cout_p;
  hipLaunchKernelGGL(k_cast_weights, dim3((unsigned)((n + 255) / 256)), dim3(256), 0, s, master,
                     cin, cout, cin_p, cout_p, w, wt, bias);
  return hipGetLastError();
}

}  // namespace tdgl_nn
