// Attention of a chunk's queries over FadeMem's exposed cache, fp32 in and
// out (FadeMem Sec. 3.1, Sec. 4.1): O_h = softmax(scale * Q_h K_h^T) V_h,
// keys/values = [memory entries in memory order || current chunk].
//
// Flash attention on the fp32 matrix cores (v_mfma_f32_32x32x2_f32: fp32
// products and sums throughout).  A workgroup of 8 waves takes one head and
// QW x 32 queries over a range of the key tiles; wave w runs queries
// 32 (w % QW) .. + 31 over key split w / QW, the range's tiles of 32 keys
// being dealt round-robin to the KS = 8 / QW splits.
// * Transposed scores: S^T = K Q^T leaves 16 keys of one query in each lane
//   (lane = query l % 32, half l / 32), so row max and sum need one lane-pair
//   exchange, and a lane's weight of key r is already the B operand of
//   O^T = V^T P^T, step r covering the two halves' keys r.
// * The summed index of an MFMA step may be any two values as long as both
//   operands agree: with d = 8 j + 4 (l / 32) + e in step (j, e) of S^T, a
//   lane's K operands of four steps are one 16-byte LDS read; V is read row by
//   row, 4 bytes per lane.
// * Sums stay short: scores in two chains, a tile's weights and O^T summed
//   from zero and then added to the running ones (one FMA per element, 3% of
//   the MFMAs' time).
// * K/V tiles go from global memory straight into LDS; K's 16-byte chunks are
//   XOR-swizzled by row so that 16 rows' reads fall in distinct banks.  With
//   QW = 4 they are double-buffered (each buffer its own LDS object, so the
//   compiler can tell its reads from the loads in flight into the other), one
//   barrier per tile; with QW = 2, for calls too small to give each split
//   more than a few tiles, one buffer and four splits.
// * Rows past the last key are zero in LDS and score -inf.
// * At the end the splits' partial (O, max, sum) are combined through LDS;
//   split 0 writes O and the LSE or, where the key axis is cut into ranges,
//   the range's partial result to its slot, and attend_f32_combine_kernel
//   combines a query tile's ranges in order.
// Bound by the matrix cores (a tile of 32 keys x 32 queries is 2 x 64 MFMAs
// of 64 cycles at D = 128) and, since fp32 matrix instructions do not run
// beside vector ones on a SIMD, by the vector work of the softmax and the
// loads' addresses: 12 heads x 1170 queries over 5850 keys take 420-425 us (99
// TFLOP/s of the 157 peak; 1100-1140 us on the vector ALUs with K/V broadcast
// from LDS), and the error against 64 bits falls from 3.1e-7 to 1.6e-7.
#include <algorithm>
#include <mutex>

#include "fademem_internal.h"

namespace fademem {
namespace {

typedef float f32x4 __attribute__((ext_vector_type(4)));
typedef float f32x16 __attribute__((ext_vector_type(16)));
#define LDS_AS __attribute__((address_space(3)))

constexpr int kThreads = 512;
constexpr int kWaves = kThreads / 64;
constexpr int kTile = 32;  // keys per tile
constexpr float kLog2e = 1.4426950408889634f;
constexpr float kLn2 = 0.6931471805599453f;

__device__ __forceinline__ float pair_add(float x) {
  auto r = __builtin_amdgcn_permlane32_swap(__float_as_uint(x), __float_as_uint(x), false, false);
  return __uint_as_float(r[0]) + __uint_as_float(r[1]);
}
__device__ __forceinline__ float pair_max(float x) {
  auto r = __builtin_amdgcn_permlane32_swap(__float_as_uint(x), __float_as_uint(x), false, false);
  return fmaxf(__uint_as_float(r[0]), __uint_as_float(r[1]));
}

// Floats of a partial result: O of every query, then its row max and row sum.
__host__ __device__ constexpr size_t part_floats(int queries, int head_dim) {
  return size_t(queries) * size_t(head_dim + 2);
}

template <int D, int QW>
struct Shape {
  static constexpr int KS = kWaves / QW;           // key splits
  static constexpr int NBUF = QW == 4 ? 2 : 1;     // tile buffers
  static constexpr int QT = 32 * QW;               // queries per workgroup
  static constexpr int DB = D / 32;                // 32-row blocks of O^T
  static constexpr int CH = D / 4;                 // 16-byte chunks per row
  static constexpr int TILE = kTile * D;           // floats per tile
  static constexpr int LOADS = kTile * CH / (64 * QW);  // 16-byte loads per lane and tile, for K and for V
  static constexpr int COMB = 64 * (16 * DB + 2);  // floats a wave leaves for the combine
  static constexpr int OBJ = KS * TILE;            // floats per LDS object
  static constexpr int PER_OBJ = (kWaves - QW) / (2 * NBUF);  // waves' combine areas per object
  static_assert(LOADS * 64 * QW == kTile * CH, "tile split");
  static_assert(PER_OBJ * 2 * NBUF == kWaves - QW && PER_OBJ * COMB <= OBJ, "combine areas fit");
};

template <int D, int QW>
__global__ __launch_bounds__(kThreads, 2) void attend_f32_kernel(AttendArgs args, int q_tiles, int parts) {
  using S = Shape<D, QW>;
  constexpr int KS = S::KS, DB = S::DB;
  __shared__ __attribute__((aligned(16))) float k_lds0[S::OBJ];
  __shared__ __attribute__((aligned(16))) float v_lds0[S::OBJ];
  __shared__ __attribute__((aligned(16))) float k_lds1[S::NBUF == 2 ? S::OBJ : 4];
  __shared__ __attribute__((aligned(16))) float v_lds1[S::NBUF == 2 ? S::OBJ : 4];
  // K and V addresses of row 0 (this head) of each exposed entry, the current
  // chunk as entry n_entries.
  extern __shared__ __attribute__((aligned(16))) const char* rows_s[];

  const int part = blockIdx.x % parts;
  const int h = (blockIdx.x / parts) / q_tiles;
  const int qt = (blockIdx.x / parts) % q_tiles;
  const int tid = threadIdx.x;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int lane = tid & 63;
  const int l32 = lane & 31, hh = lane >> 5;
  const int qw = wave % QW, split = wave / QW;
  const int H = args.heads;
  const int n_entries = int(args.n_entries);
  const int N = int(args.tokens_per_block);
  const int mem_rows = n_entries * N;
  const int Lk = mem_rows + int(args.cur_tokens);
  const int Lq = int(args.q_tokens);
  const int q_row = qt * S::QT + 32 * qw + l32;
  const size_t row_bytes = size_t(H) * D * 4;
  const size_t head_off = size_t(h) * D * 4;

  for (int e = tid; e <= n_entries; e += kThreads) {
    const char* kr = static_cast<const char*>(args.k_cur);
    const char* vr = static_cast<const char*>(args.v_cur);
    if (e < n_entries) {
      kr = args.k_base + size_t(args.k_order ? args.k_order[e] : e) * args.k_stride;
      vr = args.v_base + size_t(args.v_order[e]) * args.v_stride;
    }
    rows_s[2 * e] = kr + head_off;
    rows_s[2 * e + 1] = vr + head_off;
  }

  // Query l32, elements 8 j + 4 hh + e, times the power of two in the scale (in
  // the log2 domain), which rounds nothing; the rest of it, c in [1, 2), enters
  // where a score's distance to the row max is taken, in one rounding.
  const float c2 = args.scale * kLog2e;
  const float cp = fmaxf(__uint_as_float(__float_as_uint(c2) & 0x7f800000u), 0x1p-126f), c = c2 / cp;
  f32x4 q[D / 8];
  {
    const char* qp = static_cast<const char*>(args.q) + size_t(q_row < Lq ? q_row : Lq - 1) * row_bytes + head_off;
#pragma unroll
    for (int j = 0; j < D / 8; ++j) q[j] = *reinterpret_cast<const f32x4*>(qp + 32 * j + 16 * hh) * cp;
  }
  f32x16 o[DB];
#pragma unroll
  for (int db = 0; db < DB; ++db)
#pragma unroll
    for (int r = 0; r < 16; ++r) o[db][r] = 0.0f;
  float m_run = -INFINITY, l_run = 0.0f;
  const bool active = qt * S::QT + 32 * qw < Lq;  // wave-uniform: the wave has a query
  __syncthreads();                                // the entry table is in

  // Key tiles [t_begin, t_end) of this workgroup; round i gives this split
  // tile t_begin + i * KS + split.
  const int n_tiles = (Lk + kTile - 1) / kTile;
  const int t_begin = int(int64_t(n_tiles) * part / parts), t_end = int(int64_t(n_tiles) * (part + 1) / parts);
  const int rounds = (t_end - t_begin + KS - 1) / KS;
  auto issue = [&](int round, float* kb, float* vb) {
    const int tile = t_begin + round * KS + split;
    if (tile >= t_end) return;
    kb += split * S::TILE;
    vb += split * S::TILE;
    int ln = lane;  // kept from one tile to the next, the addresses would cost registers
    asm volatile("" : "+v"(ln));
    // The tile's first row: entry e0, row r0 of it (a division per tile; a
    // row of its own only where entries are shorter than a tile).
    const int k0 = tile * kTile;
    const bool in_mem = k0 < mem_rows;
    const int e0 = in_mem ? k0 / N : n_entries, r0 = in_mem ? k0 - e0 * N : k0 - mem_rows;
#pragma unroll
    for (int i = 0; i < S::LOADS; ++i) {
      const int idx = (i * QW + qw) * 64 + ln;  // destination chunk
      const int row = idx / S::CH, pos = idx % S::CH;
      if (k0 + row < Lk) {
        int e = e0, r = r0 + row;
        if (N >= kTile) {
          if (in_mem && r >= N) {
            r -= N;
            ++e;
          }
        } else if (k0 + row < mem_rows) {
          e = (k0 + row) / N;
          r = k0 + row - e * N;
        } else {
          e = n_entries;
          r = k0 + row - mem_rows;
        }
        const size_t off = size_t(r) * row_bytes;
        __builtin_amdgcn_global_load_lds(rows_s[2 * e] + off + (pos ^ (row & 15)) * 16,
                                         (LDS_AS void*)(kb + (i * QW + qw) * 256), 16, 0, 0);
        __builtin_amdgcn_global_load_lds(rows_s[2 * e + 1] + off + pos * 16,
                                         (LDS_AS void*)(vb + (i * QW + qw) * 256), 16, 0, 0);
      } else {
        *reinterpret_cast<f32x4*>(kb + idx * 4) = f32x4{0.0f, 0.0f, 0.0f, 0.0f};
        *reinterpret_cast<f32x4*>(vb + idx * 4) = f32x4{0.0f, 0.0f, 0.0f, 0.0f};
      }
    }
  };
  auto compute = [&](int round, const float* kb, const float* vb) {
    const int tile = t_begin + round * KS + split;
    if (tile >= t_end || !active) return;
    const float* kr = kb + split * S::TILE + l32 * D;
    int swz = (l32 & 15) ^ hh;  // worked out anew for each tile, as in issue()
    asm volatile("" : "+v"(swz));
    const float* vr = vb + split * S::TILE;
    f32x16 zero;
#pragma unroll
    for (int r = 0; r < 16; ++r) zero[r] = 0.0f;
    f32x16 s, s1;  // two chains of D / 4 steps
#pragma unroll
    for (int j = 0; j < D / 8; ++j) {
      const f32x4 kf = *reinterpret_cast<const f32x4*>(kr + ((2 * j) ^ swz) * 4);
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        if (e % 2 == 0) s = __builtin_amdgcn_mfma_f32_32x32x2f32(kf[e], q[j][e], j + e == 0 ? zero : s, 0, 0, 0);
        else s1 = __builtin_amdgcn_mfma_f32_32x32x2f32(kf[e], q[j][e], j + e == 1 ? zero : s1, 0, 0, 0);
      }
    }
#pragma unroll
    for (int r = 0; r < 16; ++r) s[r] += s1[r];
    const int left = Lk - tile * kTile;
    if (left < kTile) {
#pragma unroll
      for (int r = 0; r < 16; ++r)
        if (8 * (r >> 2) + 4 * hh + (r & 3) >= left) s[r] = -INFINITY;
    }
    float mx = s[0];
#pragma unroll
    for (int r = 1; r < 16; ++r) mx = fmaxf(mx, s[r]);
    const float m_new = fmaxf(m_run, pair_max(mx) * c);
    const float m_ref = m_new == -INFINITY ? 0.0f : m_new;  // every score -inf so far: weights 0, not NaN
    const float alpha = exp2f(m_run - m_ref);
    m_run = m_new;
    float least = 0.0f, l_tile = 0.0f;
#pragma unroll
    for (int r = 0; r < 16; ++r) {
      s[r] = __builtin_fmaf(s[r], c, -m_ref);
      least = fminf(least, s[r]);
    }
    // The instruction alone makes weights below 2^-126 zero, exp2f does not: it
    // is taken for the tiles that hold such weights (the test for them costs 1%
    // of a long call at D = 128, 2% at D = 64).
    if (__any(least < -126.0f)) {
#pragma unroll
      for (int r = 0; r < 16; ++r) s[r] = exp2f(s[r]);
    } else {
#pragma unroll
      for (int r = 0; r < 16; ++r) s[r] = __builtin_amdgcn_exp2f(s[r]);
    }
#pragma unroll
    for (int r = 0; r < 16; ++r) l_tile += s[r];
    l_run = l_run * alpha + l_tile;
    // The tile's own O^T, one block at a time, from zero, then added to the
    // running one: its 32 keys round at the tile's size, not at the whole
    // sum's.  With QW = 2 in two chains of 16 keys: small calls, whose sums
    // are short, keep the error of one pass over 16 keys per split.
#pragma unroll
    for (int db = 0; db < DB; ++db) {
      const float* vp = vr + 4 * hh * D + 32 * db + l32;
      f32x16 t;
#pragma unroll
      for (int r = 0; r < 16; ++r) t[r] = 0.0f;
      if constexpr (QW == 2) {
        f32x16 t1 = t;
#pragma unroll
        for (int r = 0; r < 8; ++r) {
          t = __builtin_amdgcn_mfma_f32_32x32x2f32(vp[(8 * (r >> 2) + (r & 3)) * D], s[r], t, 0, 0, 0);
          t1 = __builtin_amdgcn_mfma_f32_32x32x2f32(vp[(8 * (r >> 2) + (r & 3) + 16) * D], s[r + 8], t1, 0, 0, 0);
        }
#pragma unroll
        for (int r = 0; r < 16; ++r) o[db][r] = __builtin_fmaf(o[db][r], alpha, t[r] + t1[r]);
      } else {
#pragma unroll
        for (int r = 0; r < 16; ++r)
          t = __builtin_amdgcn_mfma_f32_32x32x2f32(vp[(8 * (r >> 2) + (r & 3)) * D], s[r], t, 0, 0, 0);
#pragma unroll
        for (int r = 0; r < 16; ++r) o[db][r] = __builtin_fmaf(o[db][r], alpha, t[r]);
      }
      __builtin_amdgcn_sched_barrier(0);  // the next block's V reads stay behind: 256 VGPRs do not hold them too
    }
  };

  if constexpr (S::NBUF == 2) {
    issue(0, k_lds0, v_lds0);
    for (int i = 0; i < rounds; i += 2) {
      __builtin_amdgcn_s_waitcnt(0);
      __syncthreads();  // round i's tiles landed for every wave; the other buffers are free
      if (i + 1 < rounds) issue(i + 1, k_lds1, v_lds1);
      compute(i, k_lds0, v_lds0);
      if (i + 1 >= rounds) break;
      __builtin_amdgcn_s_waitcnt(0);
      __syncthreads();
      if (i + 2 < rounds) issue(i + 2, k_lds0, v_lds0);
      compute(i + 1, k_lds1, v_lds1);
    }
  } else {
    for (int i = 0; i < rounds; ++i) {
      if (i > 0) __syncthreads();  // the previous round's reads are done
      issue(i, k_lds0, v_lds0);
      __builtin_amdgcn_s_waitcnt(0);
      __syncthreads();
      compute(i, k_lds0, v_lds0);
    }
  }
  // The row sum of both halves' keys (the row max is the pair's already).
  l_run = pair_add(l_run);

  // Combine the splits into split 0.
  auto area = [&](int w) {  // combine area of wave w >= QW
    const int i = w - QW, obj = i / S::PER_OBJ;
    float* base = obj == 0 ? k_lds0 : obj == 1 ? v_lds0 : obj == 2 ? k_lds1 : v_lds1;
    return base + (i % S::PER_OBJ) * S::COMB + lane;
  };
  __syncthreads();  // the last round's reads are done
  if (split > 0) {
    float* dst = area(wave);
#pragma unroll
    for (int db = 0; db < DB; ++db)
#pragma unroll
      for (int r = 0; r < 16; ++r) dst[64 * (16 * db + r)] = o[db][r];
    dst[64 * 16 * DB] = m_run;
    dst[64 * (16 * DB + 1)] = l_run;
  }
  __syncthreads();
  if (split > 0 || !active) return;
#pragma unroll
  for (int x = 1; x < KS; ++x) {
    const float* src = area(x * QW + qw);
    const float m_o = src[64 * 16 * DB];
    const float m_new = fmaxf(m_run, m_o);
    if (m_new == -INFINITY) continue;  // both empty: nothing to add
    const float a = exp2f(m_run - m_new), b = exp2f(m_o - m_new);
    l_run = l_run * a + src[64 * (16 * DB + 1)] * b;
#pragma unroll
    for (int db = 0; db < DB; ++db)
#pragma unroll
      for (int r = 0; r < 16; ++r) o[db][r] = o[db][r] * a + src[64 * (16 * db + r)] * b;
    m_run = m_new;
  }

  // Query l32's elements 32 db + 8 (r / 4) + 4 hh + r % 4.
  auto write = [&](float* row, float f) {
#pragma unroll
    for (int db = 0; db < DB; ++db)
#pragma unroll
      for (int r = 0; r < 16; r += 4)
        *reinterpret_cast<f32x4*>(row + 32 * db + 2 * r + 4 * hh) =
            f32x4{o[db][r] * f, o[db][r + 1] * f, o[db][r + 2] * f, o[db][r + 3] * f};
  };
  if (parts > 1) {  // this range's partial result: unnormalised O, row max and row sum per query
    float* slot = args.ws + size_t(blockIdx.x) * part_floats(S::QT, D);
    const int qi = 32 * qw + l32;
    write(slot + size_t(qi) * D, 1.0f);
    if (hh == 0) {
      slot[S::QT * D + qi] = m_run;
      slot[S::QT * (D + 1) + qi] = l_run;
    }
    return;
  }
  if (q_row < Lq) {
    write(reinterpret_cast<float*>(static_cast<char*>(args.out) + size_t(q_row) * row_bytes + head_off), 1.0f / l_run);
    if (args.lse && hh == 0) args.lse[size_t(h) * Lq + q_row] = (m_run + log2f(l_run)) * kLn2;
  }
}

// Combine the `parts` key ranges of a (head, query tile) of `qt_rows`
// queries: a thread takes four elements of one query, and adds the ranges in
// order with weights 2^(m_p - max_p m_p).  grid = (queries of a tile / per
// block, heads * q_tiles).
constexpr int kCombThreads = 256;
template <int D>
__global__ __launch_bounds__(kCombThreads) void attend_f32_combine_kernel(AttendArgs args, int q_tiles, int parts,
                                                                         int qt_rows) {
  constexpr int CH = D / 4;
  const int h = blockIdx.y / q_tiles, qt = blockIdx.y % q_tiles;
  const int qi = blockIdx.x * (kCombThreads / CH) + threadIdx.x / CH, c = threadIdx.x % CH;
  const int q_row = qt * qt_rows + qi;
  const int Lq = int(args.q_tokens);
  if (q_row >= Lq) return;
  const size_t step = part_floats(qt_rows, D);
  const float* base = args.ws + size_t(blockIdx.y) * size_t(parts) * step;
  const float* mp = base + size_t(qt_rows) * D + qi;
  float m_max = -INFINITY;
#pragma unroll 8
  for (int p = 0; p < parts; ++p) m_max = fmaxf(m_max, mp[p * step]);
  f32x4 o = {0.0f, 0.0f, 0.0f, 0.0f};
  float l = 0.0f;
#pragma unroll 8
  for (int p = 0; p < parts; ++p) {
    const float w = exp2f(mp[p * step] - m_max);
    l += mp[p * step + qt_rows] * w;
    o += *reinterpret_cast<const f32x4*>(base + p * step + size_t(qi) * D + 4 * c) * w;
  }
  float* out = reinterpret_cast<float*>(static_cast<char*>(args.out)) + (size_t(q_row) * args.heads + h) * D + 4 * c;
  *reinterpret_cast<f32x4*>(out) = o * (1.0f / l);
  if (args.lse && c == 0) args.lse[size_t(h) * Lq + q_row] = (m_max + log2f(l)) * kLn2;
}

typedef void (*F32Kernel)(AttendArgs, int, int);
typedef void (*F32Combine)(AttendArgs, int, int, int);

// Bytes of entry table a workgroup can hold beside its tiles (128 KB at
// D = 128): the largest memory, M + staged frames, fits.
constexpr size_t kMaxTable = 20 * 1024;
static_assert((kMaxBudget + kMaxPlanFrames + 1) * 2 * sizeof(const char*) <= kMaxTable, "entry table fits");

// Key tiles times 32-query blocks of a call from which four query waves
// share a tile (two splits, double-buffered) rather than two (four splits):
// 8 heads x 200 queries over 1600 keys (2800) 27.2 us with two, 31.0 with
// four; 5 x 300 over 3900 at D = 64 (6100) 35.3 and 38.1; 6 x 600 over 7800
// (27816) the same; above, two would read every K/V tile twice as often.
constexpr int64_t kWideFrom = 8192;

hipError_t launch_f32(F32Kernel wide, F32Kernel narrow, F32Combine combine, std::once_flag& attr_once,
                      const AttendArgs& a, hipStream_t stream) {
  const size_t shmem = size_t(a.n_entries + 1) * 2 * sizeof(const char*);  // entry table; tile buffers are static
  if (shmem > kMaxTable) return hipErrorInvalidValue;
  const int64_t lk = a.n_entries * a.tokens_per_block + a.cur_tokens;
  const int n_tiles = int((lk + kTile - 1) / kTile);
  const int64_t wave_tiles = (a.q_tokens + 31) / 32 * a.heads * n_tiles;
  const int QW = wave_tiles >= kWideFrom ? 4 : 2, KS = kWaves / QW, qt_rows = 32 * QW;
  const int64_t q_tiles64 = (a.q_tokens + qt_rows - 1) / qt_rows;
  if (q_tiles64 * a.heads > int64_t(0x7fffffff)) return hipErrorInvalidValue;
  const int q_tiles = int(q_tiles64);
  const int total = q_tiles * a.heads;
  const int most = std::min<int64_t>(f32_ws_bytes(a.head_dim) / sizeof(float) / part_floats(qt_rows, a.head_dim) / total,
                                     (n_tiles + KS - 1) / KS);
  // Key ranges: as many as finish first, up to a tile for every split and the
  // slots there are, in rounds of one workgroup per CU.  In units of 70 ns, a
  // key tile of a split takes D, a workgroup's start and end 128, the combine
  // 40 and, as few workgroups wait for one slot after another, 9 per range
  // (measured: 8.7 us a tile and 0.65 us a range at D = 128, 4.7 and 0.62 at
  // D = 64).  So one head of 128 queries over 65536 keys takes 128 ranges, 164
  // us (64 ranges 192, 256 ranges 212).
  int parts = 1;
  int64_t best = INT64_MAX;
  for (int p = 1; p <= std::max(1, most) && 9 * p < best; ++p) {
    const int rounds = int((int64_t(total) * p + 255) / 256), per = (n_tiles + p * KS - 1) / (p * KS);
    const int64_t cost = int64_t(rounds) * (int64_t(per) * a.head_dim + 128) + (p > 1 ? 40 + 9 * p : 0);
    if (cost < best) {
      best = cost;
      parts = p;
    }
  }
  hipError_t e = hipSuccess;
  std::call_once(attr_once, [&] {
    for (F32Kernel k : {wide, narrow})
      if (e == hipSuccess)
        e = hipFuncSetAttribute(reinterpret_cast<const void*>(k), hipFuncAttributeMaxDynamicSharedMemorySize,
                                int(kMaxTable));
  });
  if (e != hipSuccess) return e;
  hipLaunchKernelGGL(QW == 4 ? wide : narrow, dim3(unsigned(total) * unsigned(parts)), dim3(kThreads), shmem, stream, a,
                     q_tiles, parts);
  if ((e = hipGetLastError()) != hipSuccess) return e;
  if (parts > 1) {
    const int per_block = kCombThreads / (a.head_dim / 4);
    hipLaunchKernelGGL(combine, dim3(unsigned(qt_rows / per_block), unsigned(total)), dim3(kCombThreads), 0, stream, a,
                       q_tiles, parts, qt_rows);
    e = hipGetLastError();
  }
  return e;
}

std::once_flag attr_f32_d128, attr_f32_d64;

}  // namespace

hipError_t launch_attend_f32(const AttendArgs& a, hipStream_t stream) {
  if (a.head_dim == 128)
    return launch_f32(attend_f32_kernel<128, 4>, attend_f32_kernel<128, 2>, attend_f32_combine_kernel<128>,
                      attr_f32_d128, a, stream);
  if (a.head_dim == 64)
    return launch_f32(attend_f32_kernel<64, 4>, attend_f32_kernel<64, 2>, attend_f32_combine_kernel<64>, attr_f32_d64,
                      a, stream);
  return hipErrorInvalidValue;
}

}  // namespace fademem
