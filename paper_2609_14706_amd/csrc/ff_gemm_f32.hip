// General fp32 product on the fp32 matrix cores (v_mfma_f32_32x32x2_f32).
//
// The smaller fp32 products: the tree of the triangular inverse of a factor,
// smaller fp32 layers.  64 x 64 output tiles, four waves of one 32 x 32
// matrix-core tile, 64-wide k slices staged through double-buffered LDS (such
// products are latency bound: few, large slices).  Products that fill the GPU
// with larger tiles go to ff_gemm_split.hip.  Any shape and
// either operand transpose; k ranges can be clipped to the non-zero triangle
// of a triangular operand, k can run over segments (the stacked samples), and
// k can be split over the grid into partial outputs.  When every operand is
// 16-byte aligned with leading dimensions divisible by 4, global loads are
// 16-byte vectors (edge vectors fall back to element loads).
#include <algorithm>

#include "ff_common.hpp"
#include "ff_kernels.hpp"

namespace ff {
namespace {

// k range per workgroup above which products use two-level accumulation
constexpr int64_t kDeepK = 16384;

constexpr int BT = 64;  // tile rows and columns
constexpr int BK = 64;  // k per LDS slice

// Offset of k in a k axis made of segments of kseg, seg apart (kseg == 0:
// one contiguous axis, no division).
__device__ __forceinline__ int64_t seg_off(int64_t k, int64_t kseg, int64_t seg) {
  return kseg ? (k / kseg) * seg + (k % kseg) : k;
}

// One operand slice: 64 "outer" indices (rows of op(A) or columns of op(B))
// x 64 k.  KMAJ: the operand is contiguous along k (element (o, k) at
// P[o * ld + koff(k)]); otherwise contiguous along o (at P[koff(k) * ld + o]).
// Each thread fetches NQ 4-element groups; slice[k][o] is written to LDS.
// FAST: the whole slice is in bounds and 16-byte vectors can be used.
template <bool KMAJ, bool FAST>
struct SliceLoader {
  static constexpr int NQ = BT * BK / 4 / 256;  // 4-element groups per thread
  static constexpr int OQ = BT / 4;             // 4-element groups per k row (non-k-major)
  f32x4 v[NQ];
  __device__ __forceinline__ void load(const float* P, int64_t ld, int64_t o0, int64_t olim,
                                       int64_t k0, int64_t khi, int64_t kseg, int64_t seg,
                                       int tid) {
#pragma unroll
    for (int q = 0; q < NQ; ++q) {
      const int idx = tid + 256 * q;
      const int o = KMAJ ? idx / (BK / 4) : (idx % OQ) * 4;
      const int k = KMAJ ? (idx % (BK / 4)) * 4 : idx / OQ;
      const int64_t go = o0 + o, gk = k0 + k;
      if (FAST) {
        const int64_t ko = seg_off(gk, kseg, seg);
        v[q] = KMAJ ? *reinterpret_cast<const f32x4*>(P + go * ld + ko)
                    : *reinterpret_cast<const f32x4*>(P + ko * ld + go);
      } else {
        f32x4 r = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
        for (int e = 0; e < 4; ++e) {
          const int64_t eo = KMAJ ? go : go + e, ek = KMAJ ? gk + e : gk;
          if (eo < olim && ek < khi) {
            const int64_t ko = seg_off(ek, kseg, seg);
            r[e] = KMAJ ? P[eo * ld + ko] : P[ko * ld + eo];
          }
        }
        v[q] = r;
      }
    }
  }
  __device__ __forceinline__ void store(float (*S)[BT + 4], int tid) const {
#pragma unroll
    for (int q = 0; q < NQ; ++q) {
      const int idx = tid + 256 * q;
      if (KMAJ) {
        const int o = idx / (BK / 4), k = (idx % (BK / 4)) * 4;
#pragma unroll
        for (int e = 0; e < 4; ++e) S[k + e][o] = v[q][e];
      } else {
        const int k = idx / OQ, o = (idx % OQ) * 4;
        *reinterpret_cast<f32x4*>(&S[k][o]) = v[q];
      }
    }
  }
};

struct TileLDS {
  float a[2][BK][BT + 4];
  float b[2][BK][BT + 4];
};

// acc += op(A)[i0.., klo..khi) op(B)[klo..khi), j0..) for one tile (each wave
// one 32 x 32 quadrant).
// DEEP: two-level accumulation (see below), for long k ranges only: its
// second set of accumulators halves the waves a CU can hold.
template <bool AK, bool BKM, bool FAST, bool DEEP>
__device__ __forceinline__ void tile_product(const GemmF32& p, const float* A, const float* B,
                                             int64_t i0, int64_t j0, int64_t klo, int64_t khi,
                                             TileLDS& sm, f32x16& acc) {
  const int tid = threadIdx.x, wave = tid >> 6, lane = tid & 63;
  const int wm = wave >> 1, wn = wave & 1;
  SliceLoader<AK, FAST> la;
  SliceLoader<BKM, FAST> lb;
  la.load(A, p.lda, i0, p.M, klo, khi, p.kseg, p.segA, tid);
  lb.load(B, p.ldb, j0, p.N, klo, khi, p.kseg, p.segB, tid);
  la.store(sm.a[0], tid);
  lb.store(sm.b[0], tid);
  __syncthreads();
  // Two-level accumulation: the products of up to CHUNK slices go into a
  // fresh accumulator that is then added to acc.  Long k ranges (the
  // stacked samples, hundreds of thousands deep) thus round each output
  // element about CHUNK * BK / 2 + K / (CHUNK * BK) times instead of K / 2.
  constexpr int CHUNK = 8;
  f32x16 loc;
#pragma unroll
  for (int r = 0; r < 16; ++r) loc[r] = 0.0f;
  int cnt = 0;
  int cur = 0;
  for (int64_t k0 = klo; k0 < khi; k0 += BK) {
    const bool more = k0 + BK < khi;
    if (more) {
      la.load(A, p.lda, i0, p.M, k0 + BK, khi, p.kseg, p.segA, tid);
      lb.load(B, p.ldb, j0, p.N, k0 + BK, khi, p.kseg, p.segB, tid);
    }
    __builtin_amdgcn_sched_barrier(0);
    // operands of k-step s + 1 are read while the products of step s run
    float fa[2], fb[2];
    fa[0] = sm.a[cur][lane >> 5][wm * 32 + (lane & 31)];
    fb[0] = sm.b[cur][lane >> 5][wn * 32 + (lane & 31)];
#pragma unroll
    for (int s = 0; s < BK / 2; ++s) {
      if (s + 1 < BK / 2) {
        const int kr = 2 * (s + 1) + (lane >> 5);
        fa[(s + 1) & 1] = sm.a[cur][kr][wm * 32 + (lane & 31)];
        fb[(s + 1) & 1] = sm.b[cur][kr][wn * 32 + (lane & 31)];
      }
      __builtin_amdgcn_sched_barrier(0);  // keep the reads ahead of the products
      if constexpr (DEEP) loc = __builtin_amdgcn_mfma_f32_32x32x2f32(fa[s & 1], fb[s & 1], loc, 0, 0, 0);
      else acc = __builtin_amdgcn_mfma_f32_32x32x2f32(fa[s & 1], fb[s & 1], acc, 0, 0, 0);
    }
    if (DEEP && (++cnt == CHUNK || !more)) {
      acc += loc;
#pragma unroll
      for (int r = 0; r < 16; ++r) loc[r] = 0.0f;
      cnt = 0;
    }
    __builtin_amdgcn_sched_barrier(0);
    if (more) {
      la.store(sm.a[cur ^ 1], tid);
      lb.store(sm.b[cur ^ 1], tid);
    }
    __syncthreads();
    cur ^= 1;
  }
}

template <int TA, int TBT, bool VEC, bool DEEP>
__global__ __launch_bounds__(256) void k_gemm_f32(GemmF32 p) {
  if (ff_halted(p.st)) return;
  // With a triangular operand the k range, hence the work, of a tile grows
  // along one tile index: walk the tiles with that index slowest and from the
  // long end, so that the longest workgroups start first.
  int64_t bx = blockIdx.x, by = blockIdx.y;
  if (p.flags & (kKHiRow | kKLoRow)) {
    const int64_t lin = bx + (int64_t)gridDim.x * by;
    bx = lin / gridDim.y;
    by = lin % gridDim.y;
    if (p.flags & kKHiRow) bx = gridDim.x - 1 - bx;
  } else if (p.flags & (kKHiCol | kKLoCol)) {
    if (p.flags & kKHiCol) by = gridDim.y - 1 - by;
  }
  const int64_t i0 = bx * BT, j0 = by * BT;
  if ((p.flags & kCLower) && j0 > i0 + BT - 1) return;
  const float* A = p.A;
  const float* B = p.B;
  float* C = p.C;
  int64_t klo = 0, khi = p.K;
  if (p.flags & kKHiRow) khi = min(khi, i0 + BT);
  if (p.flags & kKLoRow) klo = max(klo, i0);
  if (p.flags & kKHiCol) khi = min(khi, j0 + BT);
  if (p.flags & kKLoCol) klo = max(klo, j0);
  if (p.ksplit > 1) {
    const int64_t span = khi > klo ? khi - klo : 0;
    const int64_t chunk = ((span + p.ksplit - 1) / p.ksplit + BK - 1) / BK * BK;
    klo = klo + (int64_t)blockIdx.z * chunk;
    khi = min(khi, klo + chunk);
    C += (int64_t)blockIdx.z * p.sC;
  } else {
    A += (int64_t)blockIdx.z * p.sA;
    B += (int64_t)blockIdx.z * p.sB;
    C += (int64_t)blockIdx.z * p.sC;
  }
  __shared__ __align__(16) TileLDS sm;
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const int wm = wave >> 1, wn = wave & 1;
  f32x16 acc;
#pragma unroll
  for (int r = 0; r < 16; ++r) acc[r] = 0.0f;
  if (klo < khi) {
    const bool fast = VEC && i0 + BT <= p.M && j0 + BT <= p.N && (khi - klo) % BK == 0;
    if (fast) tile_product<TA == 0, TBT != 0, VEC, DEEP>(p, A, B, i0, j0, klo, khi, sm, acc);
    else tile_product<TA == 0, TBT != 0, false, DEEP>(p, A, B, i0, j0, klo, khi, sm, acc);
  }
  const bool lower = (p.flags & kCLower) != 0;
  const bool use_beta = p.ksplit <= 1 && p.beta != 0.0f;
#pragma unroll
  for (int r = 0; r < 16; ++r) {
    const int64_t i = i0 + wm * 32 + 8 * (r >> 2) + 4 * (lane >> 5) + (r & 3);
    const int64_t j = j0 + wn * 32 + (lane & 31);
    if (i < p.M && j < p.N && (!lower || i >= j)) {
      float v = p.alpha * acc[r];
      if (use_beta) v += p.beta * C[i * p.ldc + j];
      C[i * p.ldc + j] = v;
    }
  }
}

__global__ __launch_bounds__(256) void k_reduce_rowmajor(const float* __restrict__ P, int splits,
                                                         int64_t dim_p, float* __restrict__ F,
                                                         int64_t dim, float scale, const int* st) {
  if (ff_halted(st)) return;
  const int64_t idx = (int64_t)blockIdx.x * 256 + threadIdx.x;
  if (idx >= dim * dim) return;
  const int64_t i = idx / dim, j = idx % dim;
  if (j > i) return;
  // the partials in order, sixteen loads at a time (one at a time, a 64-wide
  // factor's 128 partials took 38 us)
  const float* p = P + i * dim_p + j;
  const int64_t step = dim_p * dim_p;
  float s = 0.0f;
  int z = 0;
  for (; z + 16 <= splits; z += 16) {
    float v[16];
#pragma unroll
    for (int e = 0; e < 16; ++e) v[e] = p[(z + e) * step];
#pragma unroll
    for (int e = 0; e < 16; ++e) s += v[e];
  }
  for (; z < splits; ++z) s += p[z * step];
  s *= scale;
  F[i * dim + j] = s;
  F[j * dim + i] = s;
}

bool aligned16(const void* p) { return ((uintptr_t)p & 15u) == 0; }

}  // namespace

hipError_t launch_tiles(const GemmF32& p, int batch, bool vec, bool deep, hipStream_t s) {
  const int64_t gx = (p.M + BT - 1) / BT, gy = (p.N + BT - 1) / BT;
  const int gz = p.ksplit > 1 ? p.ksplit : batch;
  if (gx > 0x7fffffff || gy > 65535 || gz > 65535) return hipErrorInvalidValue;
  const dim3 grid((uint32_t)gx, (uint32_t)gy, (uint32_t)gz);
  const int sel = (p.transA ? 1 : 0) | (p.transB ? 2 : 0) | (vec ? 4 : 0) | (deep ? 8 : 0);
  switch (sel) {
#define FF_GEMM_CASE(c, ta, tb, v, dp) \
    case c: hipLaunchKernelGGL((k_gemm_f32<ta, tb, v, dp>), grid, dim3(256), 0, s, p); break;
    FF_GEMM_CASE(0, 0, 0, false, false)
    FF_GEMM_CASE(1, 1, 0, false, false)
    FF_GEMM_CASE(2, 0, 1, false, false)
    FF_GEMM_CASE(3, 1, 1, false, false)
    FF_GEMM_CASE(4, 0, 0, true, false)
    FF_GEMM_CASE(5, 1, 0, true, false)
    FF_GEMM_CASE(6, 0, 1, true, false)
    FF_GEMM_CASE(7, 1, 1, true, false)
    FF_GEMM_CASE(8, 0, 0, false, true)
    FF_GEMM_CASE(9, 1, 0, false, true)
    FF_GEMM_CASE(10, 0, 1, false, true)
    FF_GEMM_CASE(11, 1, 1, false, true)
    FF_GEMM_CASE(12, 0, 0, true, true)
    FF_GEMM_CASE(13, 1, 0, true, true)
    FF_GEMM_CASE(14, 0, 1, true, true)
    default: hipLaunchKernelGGL((k_gemm_f32<1, 1, true, true>), grid, dim3(256), 0, s, p); break;
#undef FF_GEMM_CASE
  }
  return hipGetLastError();
}

// Which route is faster, from the work that the busiest CU gets in each, in
// units of one k of a 64 x 64 tile (25 ns; 35 where its loads are checked):
//  * 64 x 64 tiles: one k each, rounds of 256 tiles, triangular ranges evened
//    out over the rounds;
//  * 256 x 128 tiles of three-part products: three units a k and about 128 k
//    to begin and end, rounds of 256 tiles, the first of which has the longest
//    range.
// Partly empty tiles and rounds count in full on both sides, so many products
// smaller than a large tile stay with the small ones.  Measured, us, 64 x 64
// tiles against 256 x 128: dense 1408 square 71 / 112, 1500 square 175 / 132,
// 2048 square 194 / 159, 2000 x 3000 618 / 238; eight of 1024 square 196 / 92; 2048
// of 64 square 24 / 114, 2048 of 16 square 22 / 95, 1024 of 128 square 65 / 84;
// triangular 2304 square 150 / 174, 2600 square 241 / 205; 65536 whitened rows of
// 64 14 / 21, of 192 57 / 58, of 256 86 / 67, of 512 273 / 198; symmetric from 65536 k in
// parts, 192 wide 58 / 85, 256 wide 143 / 87, 1024 wide 1869 / 675.
bool gemm_takes_split(const GemmF32& p, int batch, bool vec) {
  const bool lower = (p.flags & kCLower) != 0;
  if (p.tile == 64 || (lower && p.M != p.N) || p.lda > kSplitMaxLd || p.ldb > kSplitMaxLd) return false;
  if (p.M <= 128) return false;  // half of every large tile or more is empty
  auto parts = [](int64_t x, int64_t t) { return (x + t - 1) / t; };
  const int64_t z = p.ksplit > 1 ? p.ksplit : batch;
  const int64_t m64 = parts(p.M, 64), m256 = parts(p.M, 256), n128 = parts(p.N, 128);
  int64_t small = m64 * parts(p.N, 64), large = m256 * n128;
  if (lower) {
    small = m64 * (m64 + 1) / 2;
    large = 0;
    for (int64_t b = 1; b <= m256; ++b) large += std::min<int64_t>(2 * b, n128);
  }
  const double k = p.ksplit > 1 ? (double)parts(p.K, p.ksplit) : (double)p.K;
  const bool row = (p.flags & (kKHiRow | kKLoRow)) != 0, col = (p.flags & (kKHiCol | kKLoCol)) != 0;
  // mean ranges of the tiles
  const double k_small = row || col ? std::min(k, (k + 64) / 2) : k;
  const double k_large = row ? std::min(k, (k + 256) / 2) : col ? std::min(k, (k + 128) / 2) : k;
  const double r_small = (double)parts(small * z, 256), r_large = (double)parts(large * z, 256);
  const bool whole = vec && p.ksplit <= 1 && p.M % 64 == 0 && p.N % 64 == 0 && p.K % 64 == 0;
  return r_small * k_small * (whole ? 1.0 : 1.4) > 3.0 * (std::max(k, r_large * k_large) + 128.0 * r_large);
}

hipError_t launch_gemm_f32(const GemmF32& p, int batch, hipStream_t s) {
  if (p.M < 0 || p.N < 0 || p.K < 0 || batch < 1) return hipErrorInvalidValue;
  if (p.ksplit > 1 && batch != 1) return hipErrorInvalidValue;
  if (p.M == 0 || p.N == 0) return hipSuccess;
  const bool segmented = p.kseg < p.K;
  // two-level accumulation when a workgroup's k range is long (the stacked samples)
  const int64_t kwg = p.ksplit > 1 ? (p.K + p.ksplit - 1) / p.ksplit : p.K;
  const bool deep = kwg > kDeepK;
  const bool vec = aligned16(p.A) && aligned16(p.B) && p.lda % 4 == 0 && p.ldb % 4 == 0 &&
                   (batch == 1 || (p.sA % 4 == 0 && p.sB % 4 == 0)) &&
                   (!segmented || (p.kseg % 4 == 0 && p.segA % 4 == 0 && p.segB % 4 == 0));
  GemmF32 q = p;
  if (!segmented) q.kseg = 0;  // plain k axis: the kernels skip the segment arithmetic
  if (gemm_takes_split(p, batch, vec)) return launch_gemm_split(q, batch, vec, deep, s);
  return launch_tiles(q, batch, vec, deep, s);
}

hipError_t launch_reduce_rowmajor(const float* P, int splits, int64_t dim_p, float* F,
                                  int64_t dim, double scale, const int* st, hipStream_t s) {
  if (dim <= 0 || dim > dim_p || splits < 1) return hipErrorInvalidValue;
  const int64_t blocks = (dim * dim + 255) / 256;
  hipLaunchKernelGGL(k_reduce_rowmajor, dim3((uint32_t)blocks), dim3(256), 0, s, P, splits, dim_p,
                     F, dim, (float)scale, st);
  return hipGetLastError();
}

}  // namespace ff
