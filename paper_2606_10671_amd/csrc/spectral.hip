// Distance-dependent spectral decay (FadeMem Sec. 3.2; supplementary Sec. S2):
// per clip of channel-averaged latent frames z_0..z_T-1 ([H][W] fp32 each),
// the orthonormal 2-D DCT-II D(z_t) = A_H z_t A_W^T of every frame up to the
// largest lag, then for every radial band k (given as a band index per
// coefficient) and lag the Pearson correlation of band k's coefficients of
// frame 0 and of frame lag, averaged over clips:
//   C_k(lag) = mean_clips Pearson(D(z_0)|B_k, D(z_lag)|B_k).
//
// Kernels:
// * spectral_setup_kernel -- A_N[k][n] = s_k cos(pi (2n+1) k / (2N)), s_0 =
//   sqrt(1/N), s_k = sqrt(2/N), in fp64, stored fp32, and the coefficients
//   grouped by band (a stable counting sort), so each band is a contiguous
//   index list;
// * spectral_fused_kernel (frames of up to 128 x 128 whose LDS fits) --
//   persistent blocks, each taking an equal contiguous range of the
//   (clip, lag) frames: per frame T = z A_W^T and D = A_H T on the fp32
//   matrix cores (v_mfma_f32_16x16x4_f32), on the frame folded into its four
//   even/odd quadrants (half the products in each direction), the second
//   product taking T straight from the first one's accumulators, then D
//   written to LDS in band order and reduced per band to the fp64 sums S_y,
//   S_yy and S_xy against frame 0's coefficients x (kept in LDS); no
//   transform ever reaches HBM;
// * clip_mean_kernel -- per clip the Pearson coefficient from those sums
//   (frame 0's own, at lag 0, give S_x and S_xx), then the mean over clips
//   in a fixed order (every call gives the same bits).
// Frames too large for that (more than 128 rows or columns, or their LDS)
// take the general path:
// * dct2_kernel -- one block per (clip, run of frames): both bases (as
//   transposes) in LDS once, then per frame z^T in LDS, T = z A_W^T and
//   D = A_H T, each thread computing 4 x 4 output tiles from 16-byte LDS
//   reads (8 FMAs per read); fp32 products and sums; sizes padded to
//   multiples of 4 with zeros;
// * band_corr_kernel -- one block per (clip, lag): each wave takes bands in
//   turn and sums y, y^2 and x y over the band in fp64 (lanes, then a wave
//   reduction), x being frame 0.
#include <math.h>
#include <string.h>

#include <mutex>
#include <type_traits>
#include <vector>

#include "fademem_internal.h"

namespace {

inline size_t rup(size_t x) { return (x + 255) / 256 * 256; }

constexpr int kSpecLdsBytes = 160 * 1024;  // LDS of one workgroup on gfx950
constexpr int kSpecMaxBands = 1024;
constexpr int kSpecMaxLags = 65535;        // grid.y

struct SpecLayout {
  size_t off_ah, off_aw, off_d, off_perm, off_start, off_clip, total;
};

bool spec_layout(int64_t clips, int64_t nlag, int64_t H, int64_t W, int64_t bands, bool on_chip, SpecLayout* L) {
  const double d_bytes = on_chip ? 0.0 : double(clips) * double(nlag) * double(H) * double(W) * 4.0;
  const double c_bytes = double(clips) * double(nlag) * double(bands) * 24.0;
  if (d_bytes > 1e15 || c_bytes > 1e15) return false;
  size_t off = 0;
  L->off_ah = off;    off = rup(off + size_t(H * H) * 4);
  L->off_aw = off;    off = rup(off + size_t(W * W) * 4);
  L->off_d = off;     off = rup(off + (on_chip ? 0 : size_t(clips) * size_t(nlag) * size_t(H * W) * 4));
  L->off_perm = off;  off = rup(off + size_t(H * W) * 4);
  L->off_start = off; off = rup(off + size_t(bands + 1) * 4);
  L->off_clip = off;  off = rup(off + size_t(clips) * size_t(nlag) * size_t(bands) * 24);
  L->total = off;
  return true;
}

int64_t pad4(int64_t x) { return (x + 3) / 4 * 4; }
size_t dct_lds_bytes(int64_t H, int64_t W) {
  const int64_t Hp = pad4(H), Wp = pad4(W);
  return size_t(2 * Hp * Wp + Hp * Hp + Wp * Wp) * 4;
}
constexpr int kDctFramesPerBlock = 8;

typedef float f32x4 __attribute__((ext_vector_type(4)));

constexpr int kDctThreads = 512;

__global__ __launch_bounds__(kDctThreads) void dct2_kernel(const float* latents, int64_t frames, int nlag, int H, int W,
                                                   const float* AH, const float* AW, float* D) {
  extern __shared__ __attribute__((aligned(16))) float sm[];
  const int Hp = (H + 3) & ~3, Wp = (W + 3) & ~3;
  float* zt = sm;                 // z^T   [Wp][Hp]
  float* ts = zt + Wp * Hp;       // T     [Hp][Wp]
  float* aht = ts + Hp * Wp;      // A_H^T [Hp][Hp]: aht[h][u] = A_H[u][h]
  float* awt = aht + Hp * Hp;     // A_W^T [Wp][Wp]: awt[w][v] = A_W[v][w]
  const int64_t c = blockIdx.x;
  const int tid = threadIdx.x;
  const int HW = H * W;
  for (int i = tid; i < Hp * Hp; i += kDctThreads) {
    const int h = i / Hp, u = i % Hp;
    aht[i] = (h < H && u < H) ? AH[u * H + h] : 0.0f;
  }
  for (int i = tid; i < Wp * Wp; i += kDctThreads) {
    const int w = i / Wp, v = i % Wp;
    awt[i] = (w < W && v < W) ? AW[v * W + w] : 0.0f;
  }
  const int th = Hp / 4, tw = Wp / 4, tiles = th * tw;
  const int t0 = blockIdx.y * kDctFramesPerBlock;
  const int t1 = min(t0 + kDctFramesPerBlock, nlag);
  for (int t = t0; t < t1; ++t) {
    const float* z = latents + (size_t(c) * size_t(frames) + size_t(t)) * size_t(HW);
    __syncthreads();  // the previous frame's reads of zt and ts are done (and the bases are in)
    for (int i = tid; i < Wp * Hp; i += kDctThreads) {
      const int w = i / Hp, h = i % Hp;
      zt[i] = (w < W && h < H) ? z[h * W + w] : 0.0f;
    }
    __syncthreads();
    for (int i = tid; i < tiles; i += kDctThreads) {  // T[h][v] = sum_w z[h][w] A_W[v][w]
      const int h0 = 4 * (i / tw), v0 = 4 * (i % tw);
      f32x4 acc[4] = {};
#pragma unroll 4
      for (int w = 0; w < Wp; ++w) {
        const f32x4 zv = *reinterpret_cast<const f32x4*>(zt + w * Hp + h0);
        const f32x4 av = *reinterpret_cast<const f32x4*>(awt + w * Wp + v0);
#pragma unroll
        for (int a = 0; a < 4; ++a)
#pragma unroll
          for (int b = 0; b < 4; ++b) acc[a][b] = __builtin_fmaf(zv[a], av[b], acc[a][b]);
      }
#pragma unroll
      for (int a = 0; a < 4; ++a) *reinterpret_cast<f32x4*>(ts + (h0 + a) * Wp + v0) = acc[a];
    }
    __syncthreads();
    float* out = D + (size_t(c) * size_t(nlag) + size_t(t)) * size_t(HW);
    for (int i = tid; i < tiles; i += kDctThreads) {  // D[u][v] = sum_h A_H[u][h] T[h][v]
      const int u0 = 4 * (i / tw), v0 = 4 * (i % tw);
      f32x4 acc[4] = {};
#pragma unroll 4
      for (int h = 0; h < Hp; ++h) {
        const f32x4 av = *reinterpret_cast<const f32x4*>(aht + h * Hp + u0);
        const f32x4 tv = *reinterpret_cast<const f32x4*>(ts + h * Wp + v0);
#pragma unroll
        for (int a = 0; a < 4; ++a)
#pragma unroll
          for (int b = 0; b < 4; ++b) acc[a][b] = __builtin_fmaf(av[a], tv[b], acc[a][b]);
      }
#pragma unroll
      for (int a = 0; a < 4; ++a) {
        const int u = u0 + a;
        if (u >= H) continue;
#pragma unroll
        for (int b = 0; b < 4; ++b)
          if (v0 + b < W) out[u * W + v0 + b] = acc[a][b];
      }
    }
  }
}

// Set-up of an analysis in one launch, bound by its own chain of latencies
// (band map load, two passes over it in LDS): 7.9 us at 72 x 128, where two
// basis kernels and a one-block sort took 34 us:
// * blocks [0, order_blocks): the coefficients grouped by band, in index
//   order within a band, those outside [0, bands) left out.  Every block
//   keeps the band map in LDS; wave w of all takes quarter w % 4 of band w / 4,
//   counts the coefficients of lower bands and of its own before its quarter
//   (its first position) and ranks its own 512 at a time, 8 per lane.  inverse: order[i] = the position of coefficient i, H W if
//   left out (the fused kernel's scatter); else order[position] = i;
// * the other blocks: A_N[k][n] = s_k cos(pi (2n+1) k / (2N)), s_0 =
//   sqrt(1/N), s_k = sqrt(2/N), for N = H, then N = W.
constexpr int kSetupThreads = 512;
constexpr int kSetupSplit = 4;    // waves per band, each ranking its quarter of the coefficients
constexpr int kSetupChunk = 512;  // coefficients a wave ranks at a time, 8 per lane
__host__ __device__ inline int setup_map_len(int HW) { return (HW + kSetupChunk - 1) / kSetupChunk * kSetupChunk; }
__global__ __launch_bounds__(kSetupThreads) void spectral_setup_kernel(const int32_t* band_of, int H, int W, int bands,
                                                                       int order_blocks, int inverse, int32_t* order,
                                                                       int32_t* start, float* AH, float* AW) {
  extern __shared__ __attribute__((aligned(16))) uint16_t map[];  // [setup_map_len(HW)], 0xffff: left out
  const int tid = threadIdx.x, HW = H * W;
  if (int(blockIdx.x) >= order_blocks) {
    int i = (int(blockIdx.x) - order_blocks) * kSetupThreads + tid;
    const bool rows = i < H * H;
    const int N = rows ? H : W;
    if (!rows) i -= H * H;
    if (i >= N * N) return;
    const int k = i / N, n = i % N;
    const double s = k == 0 ? sqrt(1.0 / N) : sqrt(2.0 / N);
    (rows ? AH : AW)[i] = float(s * cos(M_PI * (2.0 * n + 1.0) * double(k) / (2.0 * N)));
    return;
  }
  const int len = setup_map_len(HW);
  typedef int32_t i32x4 __attribute__((ext_vector_type(4)));
  typedef uint16_t u16x4 __attribute__((ext_vector_type(4)));
#pragma unroll 5
  for (int i = 4 * tid; i < len; i += 4 * kSetupThreads) {
    i32x4 v = {-1, -1, -1, -1};
    if (i + 3 < HW) {
      __builtin_memcpy(&v, band_of + i, 16);  // band_of is aligned to 4 bytes only
    } else {
#pragma unroll
      for (int e = 0; e < 4; ++e)
        if (i + e < HW) v[e] = band_of[i + e];
    }
    u16x4 m;
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      const bool in = v[e] >= 0 && v[e] < bands;
      m[e] = in ? uint16_t(v[e]) : uint16_t(0xffff);
      if (inverse && blockIdx.x == 0 && i + e < HW && !in) order[i + e] = HW;
    }
    *reinterpret_cast<u16x4*>(map + i) = m;
  }
  __syncthreads();
  const int w = int(blockIdx.x) * (kSetupThreads / 64) + (tid >> 6), lane = tid & 63;
  const int b = w / kSetupSplit;
  if (b >= bands) return;
  const int part = (len / kSetupChunk + kSetupSplit - 1) / kSetupSplit * kSetupChunk;
  const int i0 = min(len, (w % kSetupSplit) * part), i1 = min(len, i0 + part);
  typedef uint16_t u16x8 __attribute__((ext_vector_type(8)));
  int below = 0;
#pragma unroll 4
  for (int i = 8 * lane; i < len; i += kSetupChunk) {
    const u16x8 m = *reinterpret_cast<const u16x8*>(map + i);
#pragma unroll
    for (int e = 0; e < 8; ++e) below += int(m[e]) < b + (i < i0 ? 1 : 0);
  }
  for (int o = 32; o > 0; o >>= 1) below += __shfl_xor(below, o);
  int pos = below;
  for (int i = i0 + 8 * lane; i < i1; i += kSetupChunk) {
    const u16x8 m = *reinterpret_cast<const u16x8*>(map + i);
    int n = 0;
#pragma unroll
    for (int e = 0; e < 8; ++e) n += int(m[e]) == b;
    // Matches of the lanes below (n <= 8: four bits) and of all lanes.
    int p = pos;
#pragma unroll
    for (int k = 0; k < 4; ++k) {
      const uint64_t mask = __ballot((n >> k) & 1);
      p += __popcll(mask & ((uint64_t(1) << lane) - 1)) << k;
      pos += __popcll(mask) << k;
    }
#pragma unroll
    for (int e = 0; e < 8; ++e)
      if (int(m[e]) == b) {
        if (inverse) order[i + e] = p;
        else order[p] = i + e;
        ++p;
      }
  }
  if (lane == 0) {
    if (w % kSetupSplit == 0) start[b] = below;
    if (w == bands * kSetupSplit - 1) start[bands] = pos;
  }
}

__device__ __forceinline__ double wave_sum(double v) {
  for (int o = 32; o > 0; o >>= 1) v += __shfl_xor(v, o);
  return v;
}

__global__ __launch_bounds__(256) void band_corr_kernel(const float* D, int nlag, int HW, const int32_t* perm,
                                                        const int32_t* start, int bands, double* per_clip) {
  const int64_t c = blockIdx.x;
  const int lag = blockIdx.y;
  const int wave = threadIdx.x >> 6, lane = threadIdx.x & 63;
  const float* x = D + size_t(c) * size_t(nlag) * size_t(HW);
  const float* y = x + size_t(lag) * size_t(HW);
  double* out = per_clip + (size_t(c) * size_t(nlag) + size_t(lag)) * size_t(bands) * 3;
  for (int b = wave; b < bands; b += 4) {
    const int s0 = start[b], s1 = start[b + 1];
    double sy = 0, syy = 0, sxy = 0;
    for (int j = s0 + lane; j < s1; j += 64) {
      const int i = perm[j];
      const double xv = x[i], yv = y[i];
      sy += yv;
      syy += yv * yv;
      sxy += xv * yv;
    }
    sy = wave_sum(sy);
    syy = wave_sum(syy);
    sxy = wave_sum(sxy);
    if (lane == 0) {
      out[3 * b] = sy;
      out[3 * b + 1] = syy;
      out[3 * b + 2] = sxy;
    }
  }
}

// ---- fused path: frames of up to 128 x 128 whose LDS fits ----------------
constexpr int kFusedThreads = 512;  // 8 waves
constexpr int kFusedMaxH = 128, kFusedMaxW = 128;

// The DCT's symmetry, A_N[k][N-1-n] = (-1)^k A_N[k][n], halves both products
// in each direction: with the frame folded into four quadrants (sums and
// differences of its mirrored rows and columns, by row parity pr and column
// parity pc), coefficients (2u' + pr, 2v' + pc) need quadrant (pr, pc) alone:
//   T[h'][v'] = sum_w' Z[h'][w'] A_W[2v' + pc][w'],
//   D[2u' + pr][2v' + pc] = sum_h' A_H[2u' + pr][h'] T[h'][v'].
// The middle row (column) of an odd size is its own mirror: it enters the
// even quadrant once and the odd one as x - x, whose basis value is 0 (so a
// NaN or infinity there still reaches every coefficient).
__host__ __device__ inline int half_up(int n) { return (n + 1) / 2; }
__host__ __device__ inline int r16(int x) { return (x + 15) / 16 * 16; }
// Row stride of a quadrant in floats: an odd multiple of 4, so the 16-byte
// reads of 16 consecutive rows, and the 4-byte ones of 16 rows x 4 columns,
// fall in distinct banks.
__host__ __device__ inline int fused_stride(int W) { return 4 * (((half_up(W) + 3) / 4) | 1); }
__host__ __device__ inline int fused_ht(int H) { return (half_up(H) + 15) / 16; }  // row tiles of a quadrant

// Byte offsets of the fused kernel's LDS regions.  zl: the folded frame, four
// quadrants of 16 HT rows (zero outside H x W); dl: the transform D in band
// order; xl: frame 0's coefficients in band order; sl: the band starts.
struct FusedLds {
  int zl, dl, xl, sl, total;
};
__host__ __device__ inline FusedLds fused_lds(int H, int W, int bands) {
  FusedLds L;
  int off = 0;
  L.zl = off;  off += r16(4 * 16 * fused_ht(H) * fused_stride(W) * 4);
  L.dl = off;  off += r16(H * W * 4 + 4);  // + a spare slot that takes left-out coefficients
  L.xl = off;  off += r16(H * W * 4);
  L.sl = off;  off += r16((bands + 1) * 4);
  L.total = off;
  return L;
}

bool fused_fits(int64_t H, int64_t W, int64_t bands) {
  return H <= kFusedMaxH && W <= kFusedMaxW && fused_lds(int(H), int(W), int(bands)).total <= kSpecLdsBytes;
}

// fp64 lane -> lane moves within rows of 16 (DPP), on the two halves.
template <int CTRL>
__device__ __forceinline__ double dpp_f64(double v) {
  const long long b = __double_as_longlong(v);
  const int lo = __builtin_amdgcn_update_dpp(0, int(b), CTRL, 0xf, 0xf, false);
  const int hi = __builtin_amdgcn_update_dpp(0, int(b >> 32), CTRL, 0xf, 0xf, false);
  return __longlong_as_double((static_cast<long long>(hi) << 32) | static_cast<unsigned int>(lo));
}
__device__ __forceinline__ double f64_of(unsigned lo, unsigned hi) {
  return __longlong_as_double((static_cast<long long>(hi) << 32) | lo);
}
// Lanes 0-31: a[l] + a[l + 32]; lanes 32-63: b[l - 32] + b[l].
__device__ __forceinline__ double fold32(double a, double b) {
  const long long x = __double_as_longlong(a), y = __double_as_longlong(b);
  const auto lo = __builtin_amdgcn_permlane32_swap(unsigned(x), unsigned(y), false, false);
  const auto hi = __builtin_amdgcn_permlane32_swap(unsigned(x >> 32), unsigned(y >> 32), false, false);
  return f64_of(lo[0], hi[0]) + f64_of(lo[1], hi[1]);
}
// Rows of 16 lanes: rows 0 and 2 get a's rows 0 + 1 and 2 + 3, rows 1 and 3 b's.
__device__ __forceinline__ double fold16(double a, double b) {
  const long long x = __double_as_longlong(a), y = __double_as_longlong(b);
  const auto lo = __builtin_amdgcn_permlane16_swap(unsigned(x), unsigned(y), false, false);
  const auto hi = __builtin_amdgcn_permlane16_swap(unsigned(x >> 32), unsigned(y >> 32), false, false);
  return f64_of(lo[0], hi[0]) + f64_of(lo[1], hi[1]);
}
// Sums of three values over the 64 lanes, in a fixed order: every lane of
// row 0 (lanes 0-15) gets a's, row 1 c's, row 2 b's.
__device__ __forceinline__ double wave_total3(double a, double b, double c) {
  double v = fold16(fold32(a, b), fold32(c, 0.0));
  v += dpp_f64<0xB1>(v);   // quad_perm [1, 0, 3, 2]
  v += dpp_f64<0x4E>(v);   // quad_perm [2, 3, 0, 1]
  v += dpp_f64<0x141>(v);  // row_half_mirror
  v += dpp_f64<0x140>(v);  // row_mirror
  return v;
}

// v_mfma_f32_16x16x4_f32 lane layout (64 lanes, l = lane): A operand
// A[l % 16][l / 16], B operand B[l / 16][l % 16], result element r of lane l
// is C[4 (l / 16) + r][l % 16].  The contraction index k of one step can be
// any 4 values of the summed index, as long as A and B agree:
// * T = Z A_W^T, step (q, e): k = w' = 16 q + 4 (l / 16) + e, so lane l reads
//   Z[h'][16 q + 4 (l / 16) .. + 3] with one 16-byte LDS read for 4 steps;
//   the NR steps of 4 columns after the NQ full sixteens take w' = 16 NQ +
//   4 s + l / 16.  Lane l holds B = A_W[v][w'] of its v-tiles in registers
//   for the whole run;
// * D = A_H T, step (i, r): k = h' = 16 i + 4 (l / 16) + r, which is where
//   element r of lane l of T's tile i already sits: T feeds the second
//   product from its accumulators with no data movement, and the A_H
//   fragments stay in registers too.
// Wave w works on quadrant (pr, pc) = (w & 1, w >> 1 & 1), on v'-tiles
// w >> 2 and (w >> 2) + 2 of 16 columns.  Each lane writes its D values
// straight to their band-order positions, so a band is a contiguous run of dl
// and xl.  Band b is always reduced by wave b % 8, which also keeps frame 0's
// run for it: that needs no barrier.
//
// A frame takes two barriers: after its products (every read of zl, and the
// previous frame's band sums, are done: D goes to dl, the next frame to zl)
// and after those stores; between a wave's band sums and its next products
// there is none.  Bound by the matrix cores and the vector ALUs together: fp32
// matrix instructions do not run beside vector ones on a SIMD (their
// co-execution counter reads 0), so a frame costs the products (840 us of a
// call on 374 clips x 177 frames of 60 x 104, the band sums, folds and stores
// left out) plus the rest (560 us alone), less what two workgroups per CU (77
// KB of LDS, 128 VGPRs) hide of the waits.  That call: 1.15 ms, 2.15 ms with
// unfolded products, frames in pairs and one workgroup per CU; 48 x 61 frames
// of 72 x 128: 131 us, 667 us through the general path.
//
// Registers: HT <= 2 is held to 128 VGPRs for two workgroups per CU.  <2, 3>
// spills 2 of them and <2, 4> (61 to 64 folded columns) 15, also at heights
// whose LDS admits one workgroup only (from 46 rows at 128 columns); <4, 3> and
// <4, 4> spill 10 and 13 of 256.  96 x 61 frames of 64 x 128 take 159 us, 263 us
// with unfolded products.
template <int HT, int NQ>
__global__ __launch_bounds__(kFusedThreads, HT <= 2 ? 4 : 2) void spectral_fused_kernel(
    const float* latents, int64_t frames, int nlag, int64_t clips, int H, int W, const float* AH, const float* AW,
    const int32_t* order, const int32_t* start, int bands, double* per_clip) {
  constexpr int UPW = NQ >= 2 ? 2 : 1;  // v'-tiles per wave
  constexpr int NI = HT <= 2 ? 1 : 2;   // 16-byte items (x 4 mirrored places) per thread and frame
  extern __shared__ __attribute__((aligned(16))) char smem[];
  const FusedLds L = fused_lds(H, W, bands);
  float* zl = reinterpret_cast<float*>(smem + L.zl);
  float* dl = reinterpret_cast<float*>(smem + L.dl);
  float* xl = reinterpret_cast<float*>(smem + L.xl);
  int32_t* sl = reinterpret_cast<int32_t*>(smem + L.sl);
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int l16 = lane & 15, g = lane >> 4;
  const int HW = H * W, He = half_up(H), We = half_up(W);
  const int S = fused_stride(W), ZQ = 16 * HT * S;  // floats per row and per quadrant
  const int nr = (We + 3) / 4 - 4 * NQ;             // 0..3 single steps
  const int NV = (We + 15) / 16;
  const int pr = wave & 1, pc = (wave >> 1) & 1;
  const int Hp = pr ? H / 2 : He, Wp = pc ? W / 2 : We;  // rows and columns of this quadrant's coefficients

  for (int i = tid; i < 4 * ZQ; i += kFusedThreads) zl[i] = 0.0f;
  for (int i = tid; i <= bands; i += kFusedThreads) sl[i] = start[i];
  f32x4 bw[UPW][NQ > 0 ? NQ : 1];  // A_W[2v' + pc][16 q + 4 g + e]
  float bs[UPW][3];                // A_W[2v' + pc][16 NQ + 4 s + g]
#pragma unroll
  for (int s = 0; s < UPW; ++s) {
    const int vp = 16 * ((wave >> 2) + 2 * s) + l16;
    const float* row = AW + size_t(2 * vp + pc) * W;
#pragma unroll
    for (int q = 0; q < NQ; ++q)
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        const int w = 16 * q + 4 * g + e;
        bw[s][q][e] = (vp < Wp && w < Wp) ? row[w] : 0.0f;
      }
#pragma unroll
    for (int t = 0; t < 3; ++t) {
      const int w = 16 * NQ + 4 * t + g;
      bs[s][t] = (vp < Wp && w < Wp) ? row[w] : 0.0f;
    }
  }
  f32x4 ah[HT][HT];  // [a][i]: A_H[2 (16 a + l16) + pr][16 i + 4 g + r]
#pragma unroll
  for (int a = 0; a < HT; ++a)
#pragma unroll
    for (int i = 0; i < HT; ++i)
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        const int up = 16 * a + l16, h = 16 * i + 4 * g + r;
        ah[a][i][r] = (up < Hp && h < Hp) ? AH[size_t(2 * up + pr) * H + h] : 0.0f;
      }
  int pos[UPW][4 * HT];  // band-order position of result element (a, r) of this lane; HW (spare) if left out
#pragma unroll
  for (int s = 0; s < UPW; ++s)
#pragma unroll
    for (int a = 0; a < HT; ++a)
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        const int up = 16 * a + 4 * g + r, vp = 16 * ((wave >> 2) + 2 * s) + l16;
        pos[s][4 * a + r] = (up < Hp && vp < Wp) ? order[(2 * up + pr) * W + 2 * vp + pc] : HW;
      }
  // This block's frames: an equal contiguous share of the (clip, lag) order,
  // preceded by frame 0 of its first clip when the share starts past it.
  const int64_t total = clips * int64_t(nlag);
  const int64_t f0 = total * blockIdx.x / gridDim.x, f1 = total * (blockIdx.x + 1) / gridDim.x;
  const int64_t c_first = f0 / nlag;
  const int t_first = int(f0 - c_first * nlag);
  const int64_t njobs = (f1 - f0) + (t_first != 0 ? 1 : 0);
  // Frame loads, each place with its three mirrors: W % 8 == 0 as 16-byte
  // chunks (item tid + 512 m = chunk k of row h'), else one float per (row,
  // column), four items where the other has one.  Addresses are worked out
  // anew for each frame: kept across the products they would cost registers.
  const bool vec = (W & 7) == 0;
  const int per_row = vec ? W / 8 : We, items = He * per_row;
  // it / per_row for it < 2^16: a multiplication by 2^32 / per_row, rounded up.
  const unsigned magic = per_row > 1 ? unsigned(((1ull << 32) + per_row - 1) / per_row) : 0u;
  auto row_of = [&](int it) { return per_row > 1 ? int(__umulhi(unsigned(it), magic)) : it; };
  constexpr int kPlaces = 4 * NI;
  f32x4 zr[kPlaces];  // vec: the four mirrored chunks of item m in zr[4 m ..]; else item m's four values in zr[m]
  auto item = [&](int m) {
    int it = tid + kFusedThreads * m;
    asm volatile("" : "+v"(it));
    return it;
  };
  auto load_z = [&](int64_t c, int t) {
    const float* z = latents + (size_t(c) * size_t(frames) + size_t(t)) * size_t(HW);
    if (vec) {
#pragma unroll
      for (int m = 0; m < NI; ++m) {
        const int it = item(m);
        if (it < items) {
          const int h = row_of(it), k = 4 * (it - h * per_row);
          const int o0 = h * W + k, o1 = h * W + W - 4 - k, down = (H - 1 - 2 * h) * W;
          zr[4 * m] = *reinterpret_cast<const f32x4*>(z + o0);
          zr[4 * m + 1] = *reinterpret_cast<const f32x4*>(z + o1);
          zr[4 * m + 2] = *reinterpret_cast<const f32x4*>(z + o0 + down);
          zr[4 * m + 3] = *reinterpret_cast<const f32x4*>(z + o1 + down);
        }
      }
    } else {
#pragma unroll
      for (int m = 0; m < kPlaces; ++m) {
        const int it = item(m);
        if (it < items) {
          const int h = row_of(it), w = it - h * per_row;
          const int o0 = h * W + w, o1 = h * W + W - 1 - w, down = (H - 1 - 2 * h) * W;
          zr[m] = f32x4{z[o0], z[o1], z[o0 + down], z[o1 + down]};
        }
      }
    }
  };
  // The four quadrants' values of one place and its mirrors: a, b in a row,
  // c, d in the mirrored row.  In a middle row (column) the mirror is the
  // place itself: fr (fc) is 0 there, else 1.
  auto fold = [](float a, float b, float c, float d, float fr, float fc) {
    const float s1 = __builtin_fmaf(b, fc, a), s2 = __builtin_fmaf(d, fc, c), d1 = a - b, d2 = c - d;
    return f32x4{__builtin_fmaf(s2, fr, s1), __builtin_fmaf(d2, fr, d1), s1 - s2, d1 - d2};  // quadrants 2 pr + pc
  };
  auto store_z = [&]() {
    if (vec) {
#pragma unroll
      for (int m = 0; m < NI; ++m) {
        const int it = item(m);
        if (it < items) {
          const int h = row_of(it), k = 4 * (it - h * per_row);
          const float fr = 2 * h == H - 1 ? 0.0f : 1.0f;
          f32x4 q[4];
#pragma unroll
          for (int e = 0; e < 4; ++e) {
            const f32x4 v = fold(zr[4 * m][e], zr[4 * m + 1][3 - e], zr[4 * m + 2][e], zr[4 * m + 3][3 - e], fr, 1.0f);
#pragma unroll
            for (int x = 0; x < 4; ++x) q[x][e] = v[x];
          }
#pragma unroll
          for (int x = 0; x < 4; ++x) *reinterpret_cast<f32x4*>(zl + x * ZQ + h * S + k) = q[x];
        }
      }
    } else {
#pragma unroll
      for (int m = 0; m < kPlaces; ++m) {
        const int it = item(m);
        if (it < items) {
          const int h = row_of(it), w = it - h * per_row;
          const f32x4 v = fold(zr[m][0], zr[m][1], zr[m][2], zr[m][3], 2 * h == H - 1 ? 0.0f : 1.0f,
                               2 * w == W - 1 ? 0.0f : 1.0f);
#pragma unroll
          for (int x = 0; x < 4; ++x) zl[x * ZQ + h * S + w] = v[x];
        }
      }
    }
  };
  const float* zq = zl + (2 * pr + pc) * ZQ + l16 * S;
  const bool mma = (wave >> 2) < NV, two = UPW == 2 && (wave >> 2) + 2 < NV;  // wave-uniform
  f32x4 dacc[UPW][HT];
  auto products = [&](auto n_c) {
    constexpr int N = decltype(n_c)::value;
    f32x4 tacc[N][HT];
#pragma unroll
    for (int s = 0; s < N; ++s)
#pragma unroll
      for (int i = 0; i < HT; ++i) tacc[s][i] = f32x4{0.0f, 0.0f, 0.0f, 0.0f};
#pragma unroll
    for (int q = 0; q < NQ; ++q) {
      f32x4 a[HT];
#pragma unroll
      for (int i = 0; i < HT; ++i) a[i] = *reinterpret_cast<const f32x4*>(zq + 16 * i * S + 16 * q + 4 * g);
#pragma unroll
      for (int e = 0; e < 4; ++e)
#pragma unroll
        for (int i = 0; i < HT; ++i)
#pragma unroll
          for (int s = 0; s < N; ++s)
            tacc[s][i] = __builtin_amdgcn_mfma_f32_16x16x4f32(a[i][e], bw[s][q][e], tacc[s][i], 0, 0, 0);
    }
#pragma unroll
    for (int t = 0; t < 3; ++t)
      if (t < nr) {
#pragma unroll
        for (int i = 0; i < HT; ++i) {
          const float a = zq[16 * i * S + 16 * NQ + 4 * t + g];
#pragma unroll
          for (int s = 0; s < N; ++s)
            tacc[s][i] = __builtin_amdgcn_mfma_f32_16x16x4f32(a, bs[s][t], tacc[s][i], 0, 0, 0);
        }
      }
#pragma unroll
    for (int s = 0; s < N; ++s)
#pragma unroll
      for (int a = 0; a < HT; ++a) dacc[s][a] = f32x4{0.0f, 0.0f, 0.0f, 0.0f};
#pragma unroll
    for (int i = 0; i < HT; ++i)
#pragma unroll
      for (int r = 0; r < 4; ++r)
#pragma unroll
        for (int a = 0; a < HT; ++a)
#pragma unroll
          for (int s = 0; s < N; ++s)
            dacc[s][a] = __builtin_amdgcn_mfma_f32_16x16x4f32(ah[a][i][r], tacc[s][i][r], dacc[s][a], 0, 0, 0);
  };
  auto scatter = [&](int s) {
#pragma unroll
    for (int a = 0; a < HT; ++a)
#pragma unroll
      for (int r = 0; r < 4; ++r) dl[pos[s][4 * a + r]] = dacc[s][a][r];
  };
  // The band sums of frame (c, t), in dl.
  auto reduce = [&](int64_t c, int t, bool emit) {
    double* out = per_clip + (size_t(c) * size_t(nlag) + size_t(t)) * size_t(bands) * 3;
    const int which = g == 0 ? 0 : g == 1 ? 2 : 1;  // of a band's three sums, the one wave_total3 leaves in this row
    for (int b = wave; b < bands; b += kFusedThreads / 64) {
      const int s0 = sl[b], s1 = sl[b + 1];
      double sy = 0, syy = 0, sxy = 0;
      if (t == 0) {  // frame 0 of a clip: its run becomes x
        for (int j = s0 + lane; j < s1; j += 64) {
          const float yf = dl[j];
          xl[j] = yf;
          const double y = yf;
          sy += y;
          syy = fma(y, y, syy);
        }
        sxy = syy;
      } else {
        int j = s0 + lane;
        for (; j + 192 < s1; j += 256) {  // four elements per lane in flight
          float xf[4], yf[4];
#pragma unroll
          for (int m = 0; m < 4; ++m) {
            xf[m] = xl[j + 64 * m];
            yf[m] = dl[j + 64 * m];
          }
#pragma unroll
          for (int m = 0; m < 4; ++m) {
            const double x = xf[m], y = yf[m];
            sy += y;
            syy = fma(y, y, syy);
            sxy = fma(x, y, sxy);
          }
        }
        for (; j < s1; j += 64) {
          const double x = xl[j], y = dl[j];
          sy += y;
          syy = fma(y, y, syy);
          sxy = fma(x, y, sxy);
        }
      }
      const double v = wave_total3(sy, syy, sxy);
      if (emit && l16 == 0 && g < 3) out[3 * b + which] = v;
    }
  };

  int64_t c = c_first;
  int t = 0;
  bool emit = t_first == 0;
  load_z(c, t);
  __syncthreads();  // zl is cleared
  store_z();
  __syncthreads();
  for (int64_t k = 0; k < njobs; ++k) {
    const bool more = k + 1 < njobs;
    int64_t cn = c;
    int tn = emit ? t + 1 : t_first;  // the next frame
    if (tn == nlag) {
      ++cn;
      tn = 0;
    }
    if (more) load_z(cn, tn);
    if (two) products(std::integral_constant<int, UPW>{});
    else if (mma) products(std::integral_constant<int, 1>{});
    __syncthreads();  // every read of zl, and the previous frame's band sums, are done
    if (mma) scatter(0);
    if (two) scatter(UPW - 1);
    if (more) store_z();
    __syncthreads();
    reduce(c, t, emit);
    c = cn;
    t = tn;
    emit = true;
  }
}

typedef void (*FusedKernel)(const float*, int64_t, int, int64_t, int, int, const float*, const float*,
                            const int32_t*, const int32_t*, int, double*);
template <int HT>
constexpr FusedKernel kFusedRow[5] = {spectral_fused_kernel<HT, 0>, spectral_fused_kernel<HT, 1>,
                                      spectral_fused_kernel<HT, 2>, spectral_fused_kernel<HT, 3>,
                                      spectral_fused_kernel<HT, 4>};
FusedKernel fused_kernel(int H, int W) {  // H <= 128, W <= 128
  const int HT = fused_ht(H), q = (half_up(W) + 3) / 4 / 4;
  return HT == 1 ? kFusedRow<1>[q] : HT == 2 ? kFusedRow<2>[q] : HT == 3 ? kFusedRow<3>[q] : kFusedRow<4>[q];
}

// Per clip, band b and lag, the Pearson coefficient from the band sums
// S_y, S_yy, S_xy of frame lag (x = frame 0, whose own sums at lag 0 are
// S_x, S_xx):
//   r = (n S_xy - S_x S_y) / sqrt((n S_xx - S_x^2)(n S_yy - S_y^2)),
// NaN for a band without spread; then the mean over clips into
// corr[band][lag].  Block = 8 consecutive (lag, band) outputs x 32 clip
// groups: group g takes clips g, g + 32, ... in order, then the 32 partial
// sums are added in group order (a fixed order, so every call gives the
// same bits).  Bound by the latency of the sums' loads: four clips' loads in
// flight per thread.
constexpr int kMeanOuts = 8, kMeanGroups = 32;
__global__ __launch_bounds__(kMeanOuts * kMeanGroups) void clip_mean_kernel(const double* per_clip,
                                                                           const int32_t* start, int64_t clips,
                                                                           int nlag, int bands, double* corr) {
  __shared__ double part[kMeanGroups][kMeanOuts];
  const int o = threadIdx.x % kMeanOuts, g = threadIdx.x / kMeanOuts;
  const int64_t n_out = int64_t(bands) * nlag;
  const int64_t i = int64_t(blockIdx.x) * kMeanOuts + o;  // i = lag * bands + band
  double s = 0.0;
  if (i < n_out) {
    const int b = int(i % bands);
    const double n = double(start[b + 1] - start[b]);
#pragma unroll 4
    for (int64_t c = g; c < clips; c += kMeanGroups) {
      const double* f = per_clip + (size_t(c) * size_t(n_out) + size_t(i)) * 3;
      const double* f0 = per_clip + (size_t(c) * size_t(n_out) + size_t(b)) * 3;  // lag 0
      const double sx = f0[0], sxx = f0[1], sy = f[0], syy = f[1], sxy = f[2];
      const double cov = n * sxy - sx * sy;
      const double vx = n * sxx - sx * sx, vy = n * syy - sy * sy;
      s += cov / sqrt(vx * vy);
    }
  }
  part[g][o] = s;
  __syncthreads();
  if (g == 0 && i < n_out) {
    double t = 0.0;
    for (int k = 0; k < kMeanGroups; ++k) t += part[k][o];
    const int lag = int(i / bands), b = int(i % bands);
    corr[size_t(b) * nlag + lag] = t / double(clips);
  }
}

// Frames whose workspace holds no transforms.  The workspace sizes and the
// sizes accepted are part of the interface: larger frames keep room for
// their transforms and stay within the general path's limits, also where the
// fused kernel takes them.
bool stored_on_chip(int64_t H, int64_t W) { return H <= 64 && W <= 128; }

bool spec_args_ok(int64_t clips, int64_t frames, int32_t height, int32_t width, int32_t bands, int64_t max_lag) {
  if (clips < 1 || clips > int64_t(0x7fffffff) || frames < 1) return false;
  if (max_lag < 0 || max_lag >= frames || max_lag + 1 > kSpecMaxLags) return false;
  if (height < 1 || width < 1 || height > 1024 || width > 1024) return false;
  if (int64_t(height) * width > 40960) return false;
  if (bands < 1 || bands > kSpecMaxBands) return false;
  if (!stored_on_chip(height, width) && dct_lds_bytes(height, width) > size_t(kSpecLdsBytes)) return false;
  return true;
}

bool is_aligned(const void* p, size_t a) { return (reinterpret_cast<uintptr_t>(p) % a) == 0; }

}  // namespace

// Workspace of the allocation-free entry point: one copy per GPU, in the
// library's code object, held until the process ends.  Host code never
// passes this name to a kernel (on the host it is only a stand-in for the
// symbol): it uses the device address hipGetSymbolAddress returns for the
// current device.
constexpr size_t kStaticScratchBytes = size_t(64) << 20;
static __device__ __align__(256) char scratch[kStaticScratchBytes];

namespace {

constexpr int kMaxScratchDevices = 64;
std::mutex g_scratch_mu;
void* g_scratch[kMaxScratchDevices];  // device address of `scratch` per device, once looked up

// The current device's copy of `scratch` (looked up on the first call on
// that device, with it current).
int static_scratch(void** out) {
  int dev = 0;
  if (hipGetDevice(&dev) != hipSuccess) return FADEMEM_EHIP;
  if (dev < 0 || dev >= kMaxScratchDevices) return FADEMEM_EUNSUPPORTED;
  std::lock_guard<std::mutex> lock(g_scratch_mu);
  if (!g_scratch[dev]) {
    void* p = nullptr;
    if (hipGetSymbolAddress(&p, HIP_SYMBOL(scratch)) != hipSuccess || !p) return FADEMEM_EHIP;
    g_scratch[dev] = p;
  }
  *out = g_scratch[dev];
  return FADEMEM_OK;
}

}  // namespace

extern "C" {

int fademem_spectral_workspace_bytes(int64_t clips, int64_t frames, int32_t height, int32_t width, int32_t bands,
                                     int64_t max_lag, size_t* bytes) {
  if (!bytes || !spec_args_ok(clips, frames, height, width, bands, max_lag)) return FADEMEM_EINVAL;
  SpecLayout L;
  if (!spec_layout(clips, max_lag + 1, height, width, bands, stored_on_chip(height, width), &L))
    return FADEMEM_EINVAL;
  *bytes = L.total;
  return FADEMEM_OK;
}

int fademem_spectral_corr(const float* latents, int64_t clips, int64_t frames, int32_t height, int32_t width,
                          const int32_t* band_of, int32_t bands, int64_t max_lag, void* workspace,
                          size_t workspace_bytes, double* corr, void* stream) {
  if (!latents || !band_of || !workspace || !corr) return FADEMEM_EINVAL;
  if (!is_aligned(latents, 4) || !is_aligned(band_of, 4) || !is_aligned(workspace, 256) || !is_aligned(corr, 8))
    return FADEMEM_EINVAL;
  if (!spec_args_ok(clips, frames, height, width, bands, max_lag)) return FADEMEM_EINVAL;
  const int nlag = int(max_lag + 1);
  const bool fused = fused_fits(height, width, bands);
  SpecLayout L;
  if (!spec_layout(clips, nlag, height, width, bands, stored_on_chip(height, width), &L)) return FADEMEM_EINVAL;
  if (workspace_bytes < L.total) return FADEMEM_ENOMEM;
  char* ws = static_cast<char*>(workspace);
  float* ah = reinterpret_cast<float*>(ws + L.off_ah);
  float* aw = reinterpret_cast<float*>(ws + L.off_aw);
  float* d = reinterpret_cast<float*>(ws + L.off_d);
  int32_t* perm = reinterpret_cast<int32_t*>(ws + L.off_perm);
  int32_t* start = reinterpret_cast<int32_t*>(ws + L.off_start);
  double* per_clip = reinterpret_cast<double*>(ws + L.off_clip);
  hipStream_t s = reinterpret_cast<hipStream_t>(stream);
  const int HW = height * width;
  (void)hipGetLastError();
  const int order_blocks = (int(bands) * kSetupSplit * 64 + kSetupThreads - 1) / kSetupThreads;
  const int basis_blocks = (height * height + width * width + kSetupThreads - 1) / kSetupThreads;
  const size_t map_bytes = size_t(setup_map_len(HW)) * sizeof(uint16_t);
  if (map_bytes > 64 * 1024 &&
      hipFuncSetAttribute(reinterpret_cast<const void*>(spectral_setup_kernel),
                          hipFuncAttributeMaxDynamicSharedMemorySize, int(map_bytes)) != hipSuccess)
    return FADEMEM_EHIP;
  hipLaunchKernelGGL(spectral_setup_kernel, dim3(unsigned(order_blocks + basis_blocks)), dim3(kSetupThreads), map_bytes,
                     s, band_of, int(height), int(width), int(bands), order_blocks, fused ? 1 : 0, perm, start, ah, aw);
  if (fused) {
    const int lds = fused_lds(height, width, bands).total;
    const FusedKernel fn = fused_kernel(height, width);
    if (lds > 64 * 1024 &&
        hipFuncSetAttribute(reinterpret_cast<const void*>(fn), hipFuncAttributeMaxDynamicSharedMemorySize, lds) !=
            hipSuccess)
      return FADEMEM_EHIP;
    int dev = 0, cus = 0;
    if (hipGetDevice(&dev) != hipSuccess ||
        hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess || cus < 1)
      return FADEMEM_EHIP;
    const int64_t total = clips * int64_t(nlag);
    // All blocks resident at once, every block with a frame: two per CU where LDS and registers (HT <= 2) allow.
    const int per_cu = fused_ht(height) <= 2 && 2 * lds <= kSpecLdsBytes ? 2 : 1;
    const unsigned grid = unsigned(total < per_cu * cus ? total : per_cu * cus);
    hipLaunchKernelGGL(fn, dim3(grid), dim3(kFusedThreads), size_t(lds), s, latents, frames, nlag, clips,
                       int(height), int(width), ah, aw, perm, start, int(bands), per_clip);
  } else {
    const size_t lds = dct_lds_bytes(height, width);
    if (lds > 64 * 1024) {
      hipError_t e = hipFuncSetAttribute(reinterpret_cast<const void*>(dct2_kernel),
                                         hipFuncAttributeMaxDynamicSharedMemorySize, int(lds));
      if (e != hipSuccess) return FADEMEM_EHIP;
    }
    const unsigned runs = unsigned((nlag + kDctFramesPerBlock - 1) / kDctFramesPerBlock);
    hipLaunchKernelGGL(dct2_kernel, dim3(unsigned(clips), runs), dim3(kDctThreads), lds, s, latents, frames, nlag,
                       int(height), int(width), ah, aw, d);
    hipLaunchKernelGGL(band_corr_kernel, dim3(unsigned(clips), unsigned(nlag)), dim3(256), 0, s, d, nlag, HW, perm,
                       start, int(bands), per_clip);
  }
  const int64_t outs = int64_t(bands) * nlag;
  hipLaunchKernelGGL(clip_mean_kernel, dim3(unsigned((outs + kMeanOuts - 1) / kMeanOuts)),
                     dim3(kMeanOuts * kMeanGroups), 0, s, per_clip, start, clips, nlag, int(bands), corr);
  return hipGetLastError() == hipSuccess ? FADEMEM_OK : FADEMEM_EHIP;
}


// The same analysis with its workspace in the library's static scratch of
// the current device: no allocation, no workspace argument.  Requests whose
// workspace would exceed kStaticScratchBytes are refused before anything is
// enqueued.  Every call on a GPU shares that GPU's scratch: calls that
// overlap on one GPU (other streams, other threads) race.  The kernels write
// every scratch byte they read, so nothing needs clearing between calls.
int fademem_spectral_corr_static(const float* latents, int64_t clips, int64_t frames, int32_t height, int32_t width,
                                 const int32_t* band_of, int32_t bands, int64_t max_lag, double* corr,
                                 void* stream) {
  if (!latents || !band_of || !corr) return FADEMEM_EINVAL;
  if (!spec_args_ok(clips, frames, height, width, bands, max_lag)) return FADEMEM_EINVAL;
  SpecLayout L;
  if (!spec_layout(clips, max_lag + 1, height, width, bands, stored_on_chip(height, width), &L))
    return FADEMEM_EINVAL;
  if (L.total > kStaticScratchBytes) return FADEMEM_ESCRATCH;
  void* ws = nullptr;
  const int rc = static_scratch(&ws);
  if (rc != FADEMEM_OK) return rc;
  return fademem_spectral_corr(latents, clips, frames, height, width, band_of, bands, max_lag, ws,
                               kStaticScratchBytes, corr, stream);
}

// ---------------------------------------------------------------------------
// Host steps of the analysis (Sec. 3.2, supplementary Sec. S2) on the
// correlation curves: a few dozen numbers, no device work.
// ---------------------------------------------------------------------------

// Radial bands: bands equal-width bins of r(u, v) = sqrt((u/H)^2 + (v/W)^2)
// over [0, max r], the last bin closed, the DC coefficient left out (-1);
// a band's radius is its bin centre.
int fademem_spectral_band_map(int32_t height, int32_t width, int32_t bands, int32_t* band_of, double* centres) {
  if (!band_of || height < 1 || width < 1 || height > 1024 || width > 1024 || bands < 1 || bands > kSpecMaxBands)
    return FADEMEM_EINVAL;
  auto radius = [&](int u, int v) {
    const double a = double(u) / double(height), b = double(v) / double(width);
    return sqrt(a * a + b * b);
  };
  const double r_max = radius(height - 1, width - 1);
  for (int u = 0; u < height; ++u)
    for (int v = 0; v < width; ++v) {
      int32_t k = -1;
      if (u != 0 || v != 0) {
        const double x = floor(radius(u, v) / r_max * double(bands));
        k = x >= double(bands - 1) ? bands - 1 : int32_t(x);
      }
      band_of[size_t(u) * size_t(width) + size_t(v)] = k;
    }
  if (centres)
    for (int k = 0; k < bands; ++k) centres[k] = (double(k) + 0.5) * r_max / double(bands);
  return FADEMEM_OK;
}

// Decorrelation horizon of each band's curve corr[k][0..lags-1]: smooth it
// with a centred moving average over `window` lags (shrinking at the ends);
// the horizon is the first lag >= 1, once the smoothed curve has made at
// least half of its total decay (s[0] - min s), where its next one-lag fall
// is below `drop` times its steepest one-lag fall; -1 if there is none (or
// the curve never falls).
int fademem_spectral_horizons(const double* corr, int32_t bands, int64_t lags, int32_t window, double drop,
                              int64_t* horizon) {
  if (!corr || !horizon || bands < 1 || lags < 1 || lags > (int64_t(1) << 24) || window < 1 || !(drop >= 0.0))
    return FADEMEM_EINVAL;
  std::vector<double> sm;
  try {
    sm.resize(size_t(lags));
  } catch (...) {
    return FADEMEM_ENOMEM;
  }
  const int64_t h = window / 2;
  for (int k = 0; k < bands; ++k) {
    const double* c = corr + size_t(k) * size_t(lags);
    for (int64_t i = 0; i < lags; ++i) {
      const int64_t lo = i - h < 0 ? 0 : i - h, hi = i + h + 1 < lags ? i + h + 1 : lags;
      double sum = 0.0;
      for (int64_t j = lo; j < hi; ++j) sum += c[j];
      sm[size_t(i)] = sum / double(hi - lo);
    }
    double lowest = sm[0], steepest = -INFINITY;
    for (int64_t i = 0; i < lags; ++i) lowest = fmin(lowest, sm[size_t(i)]);
    for (int64_t i = 0; i + 1 < lags; ++i) steepest = fmax(steepest, sm[size_t(i)] - sm[size_t(i) + 1]);
    const double total = sm[0] - lowest;
    horizon[k] = -1;
    if (!(total > 0.0 && steepest > 0.0)) continue;
    for (int64_t lag = 1; lag + 1 < lags; ++lag) {
      if (sm[0] - sm[size_t(lag)] >= 0.5 * total && sm[size_t(lag)] - sm[size_t(lag) + 1] < drop * steepest) {
        horizon[k] = lag;
        break;
      }
    }
  }
  return FADEMEM_OK;
}

// r = a t^(-b) fitted to n points by least squares on r: Gauss-Newton on
// the residuals r_i - a t_i^(-b), started from the straight line through
// (log t, log r); stops when a step changes a and b by less than 1e-14
// relative, or after `iters` steps.
int fademem_spectral_fit(const double* t, const double* r, int64_t n, int32_t iters, double* a_out, double* b_out) {
  if (!t || !r || !a_out || !b_out || n < 2 || iters < 0) return FADEMEM_EINVAL;
  for (int64_t i = 0; i < n; ++i)
    if (!(t[i] > 0.0) || !(r[i] > 0.0) || isinf(t[i]) || isinf(r[i])) return FADEMEM_EINVAL;
  double mx = 0.0, my = 0.0;
  for (int64_t i = 0; i < n; ++i) {
    mx += log(t[i]);
    my += log(r[i]);
  }
  mx /= double(n);
  my /= double(n);
  double sxx = 0.0, sxy = 0.0;
  for (int64_t i = 0; i < n; ++i) {
    const double dx = log(t[i]) - mx, dy = log(r[i]) - my;
    sxx += dx * dx;
    sxy += dx * dy;
  }
  if (!(sxx > 0.0)) return FADEMEM_EINVAL;  // every t equal: the exponent is not determined
  const double slope = sxy / sxx;
  double a = exp(my - slope * mx), b = -slope;
  for (int it = 0; it < iters; ++it) {
    // Normal equations of the linearised problem: J = [df/da, df/db].
    double jaa = 0.0, jab = 0.0, jbb = 0.0, ga = 0.0, gb = 0.0;
    for (int64_t i = 0; i < n; ++i) {
      const double lt = log(t[i]);
      const double f = a * exp(-b * lt);
      const double da = f / a, db = -lt * f, res = r[i] - f;
      jaa += da * da;
      jab += da * db;
      jbb += db * db;
      ga += da * res;
      gb += db * res;
    }
    const double det = jaa * jbb - jab * jab;
    if (!(det != 0.0) || isinf(det)) break;
    const double sa = (jbb * ga - jab * gb) / det, sb = (jaa * gb - jab * ga) / det;
    a += sa;
    b += sb;
    if (fabs(sa) <= 1e-14 * fmax(1.0, fabs(a)) && fabs(sb) <= 1e-14 * fmax(1.0, fabs(b))) break;
  }
  if (!isfinite(a) || !isfinite(b)) return FADEMEM_EINVAL;
  *a_out = a;
  *b_out = b;
  return FADEMEM_OK;
}

}  // extern "C"
