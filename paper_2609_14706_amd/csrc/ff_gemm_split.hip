// Large fp32 products on the bf16 matrix cores: every fp32 operand entry is
// split into three bf16 parts, x = h + m + l (each what is left, rounded to
// nearest: together all 24 significant bits), and
//     a b = ah bh + (ah bm + am bh) + (ah bl + am bm + al bh) + ...
// is summed over the six products written; the dropped ones have random
// signs and are together at most 2^-24 |a b|.  Products of two bf16 numbers
// are exact in fp32 and one matrix instruction adds 32 of them per rounding
// (the fp32 matrix instructions 2), so sums over many k are nearer to the
// exact ones than theirs: 2-norm errors of 2048-wide dense products 3.9e-7
// against 1.07e-6.  Where one term makes up the sum (a diagonal factor) the
// dropped products show: 3.7e-8 against 3.6e-8, the largest error 1.6e-7 against
// 1.2e-7 (with h truncated instead of rounded 4.9e-8 and 3.9e-7).  With the two
// larger dropped products as well the errors are those of the fp32
// instructions, and 8 products of 3000 x 2000 take 2.98 ms instead of 2.55; sums
// of more than one term gain nothing from them.
//
// 256 x 128 output tiles, four waves of 128 x 64 (8 x 4 tiles of
// v_mfma_f32_16x16x32_bf16), one workgroup per CU.  k goes in slices of 32:
// fp32 from global memory into registers two slices ahead, split one slice
// ahead, the parts through two LDS buffers (144 KB).  All of it stands
// between the products: within a slice's 192 matrix instructions (16 cycles
// each) every one is followed by a few others (the splitting takes about 340,
// the LDS reads and writes 54), in a fixed program order.  The slice's one
// barrier comes before its last 34 products, which hide the reads of the next
// slice's first fragments.  What bounds it is the instructions that the lone
// wave of each SIMD can issue: about 590 vector and 54 LDS instructions a slice
// in some 6000 cycles, the matrix cores busy for half of them (counters, 4096
// square triangular products at 2.0 GHz, 0.38 to 0.44 ms each), so every further
// instruction in the loop shows.  256 vector and 256 accumulator registers are
// in use: 0 to 21 values (the loop's operand addresses first) are kept in
// scratch memory.
#include <math.h>

#include <type_traits>
#include <utility>

#include "ff_common.hpp"
#include "ff_kernels.hpp"

namespace ff {
namespace {

constexpr int BM = 256, BN = 128;  // tile rows and columns
constexpr int BK = 32;             // k per slice
constexpr int CHUNK = 32;          // slices per fresh accumulator (DEEP)
constexpr int FP32_CHUNK = 8;      // the same of fp32 products
constexpr int ROWB = BK * 2;       // bytes of a row of one part in LDS
constexpr int PA = BM * ROWB, PB = BN * ROWB;  // bytes of one part of an operand slice
constexpr int BUF = 3 * (PA + PB);             // bytes of a slice's parts

typedef __attribute__((ext_vector_type(4))) uint32_t u32x4;
typedef __attribute__((ext_vector_type(2))) __bf16 bf16x2;
typedef __attribute__((ext_vector_type(2))) float f32x2;

// Parts of a slice: first operand h, m, l, second operand h, m, l; rows of 64
// bytes: row r starts at bank 16 (r & 3), and its 16-byte chunk c (8 k) sits
// at position c ^ ((r >> 2) & 3), so the 16 lanes of a pass (16 consecutive
// rows, one chunk) cover all banks.
struct __align__(16) SplitLDS {
  char p[2 * BUF];
  uint32_t big;  // bits of the largest magnitude of the tile's entries (if tiny)
  int tiny;      // set if a nonzero entry is below kTiny
  int wide;      // set if the tile has to be computed from the fp32 numbers
};

// LDS row of column o of the second operand: within each 64-column half,
// column 4 c + j sits in row 16 j + c, so that a lane's four 16-column tiles
// are four consecutive columns (one 16-byte store); the low two row bits are
// rotated by j to keep the writes of four consecutive columns in distinct
// banks.
__device__ __forceinline__ int col_row(int o) {
  const int j = o & 3, c = (o >> 2) & 15;
  return (o & 64) + 16 * j + (c & 12) + ((c + j) & 3);
}

__device__ __forceinline__ uint32_t chunk_at(int row, int c) {
  return (uint32_t)row * ROWB + 16u * (uint32_t)(c ^ ((row >> 2) & 3));
}

// Offset of k in a k axis made of segments of kseg, seg apart (kseg == 0:
// one contiguous axis).
__device__ __forceinline__ int64_t seg_off(int64_t k, int64_t kseg, int64_t seg) {
  return kseg ? (k / kseg) * seg + (k % kseg) : k;
}

__device__ __forceinline__ uint32_t pack2(float a, float b) {  // round to nearest even
  const f32x2 v = {a, b};
  return __builtin_bit_cast(uint32_t, __builtin_convertvector(v, bf16x2));
}

// Where three bf16 parts do not hold an entry, the tile is computed again from
// the fp32 numbers themselves on the fp32 matrix cores (fp32_slice), as is a
// last slice of fewer than 32 k:
//  * entries above the largest bf16 number or infinite: an infinite part
//    would meet the zero or opposite parts of finite factors and give NaN;
//  * nonzero entries below 2^-100, whose lower parts may be subnormal or below
//    every bf16 number, off by at most 2^-126 (all of the subnormal range):
//    only if an output of the tile is so small that k products of that with
//    the largest entry reach 2^-25 of it.  Tiny entries among ordinary ones
//    (gradients of a saturated softmax) so cost a look at the outputs, no
//    more.  Entries below 2^-133, subnormal fp32 numbers that round to a bf16
//    zero, are not noticed and count as zeros.
// Noticing them takes three instructions per two entries, which fit between
// the products (8 products of 3000 x 2000: 2.55 ms with and without); with 32-bit
// minima in place of the packed 16-bit ones 2.66.
constexpr float kWide = 3.3895313e38f;
constexpr float kTinyReach = 0x1p-101f;

// Range of the entries a thread has split.
struct Range {
  float big = 0.0f;             // largest magnitude (NaNs drop out)
  uint32_t least = 0xffffffffu;  // in each half the least 2 h - 1 of nonzero h, as 16-bit patterns
  __device__ __forceinline__ bool wide() const { return big > kWide; }
  __device__ __forceinline__ bool tiny() const {
    constexpr uint32_t t = 2u * ((127u - 100u) << 7) - 1u;  // of 2^-100
    return (least & 0xffffu) < t || (least >> 16) < t;
  }
};

// A thread's share of a slice: groups of eight consecutive k of one row of
// op(A) (four groups) or one column of op(B) (two).  KMAJ: the operand is
// contiguous along k (four threads share a row's 128 bytes); otherwise along
// the rows or columns (a wave reads 64 of them at one k).
template <bool KMAJ>
__device__ __forceinline__ int outer_a(int g, int tid) { return KMAJ ? (tid >> 2) + 64 * g : tid; }
template <bool KMAJ>
__device__ __forceinline__ int chunk_a(int g, int tid) { return KMAJ ? tid & 3 : g; }
template <bool KMAJ>
__device__ __forceinline__ int outer_b(int g, int tid) { return KMAJ ? (tid >> 2) + 64 * g : tid & 127; }
template <bool KMAJ>
__device__ __forceinline__ int chunk_b(int g, int tid) { return KMAJ ? tid & 3 : (tid >> 7) + 2 * g; }

// Splitting of two entries in four steps, spread between products.
struct Split {
  float a, b, ra, rb;
  uint32_t H[4], M[4], L[4];
  __device__ __forceinline__ void step(int st, const float (&v)[8], int q, Range& rg) {
    if (st == 0) {
      a = v[2 * q];
      b = v[2 * q + 1];
      H[q] = pack2(a, b);
      ra = a - __uint_as_float(H[q] << 16);
      rb = b - __uint_as_float(H[q] & 0xffff0000u);
    } else if (st == 1) {
      // one instruction (fmaxf would quiet its operands first); NaNs drop out
      asm("v_max3_f32 %0, |%1|, |%2|, %0" : "+v"(rg.big) : "v"(a), "v"(b));
      M[q] = pack2(ra, rb);
      // 2 h - 1 of both halves (the sign drops out, a zero wraps around to the largest)
      uint32_t t;
      asm("v_pk_mad_u16 %0, %1, 2, -1 op_sel_hi:[1,0,1]" : "=v"(t) : "v"(H[q]));
      asm("v_pk_min_u16 %0, %1, %0" : "+v"(rg.least) : "v"(t));
    } else if (st == 2) {
      ra -= __uint_as_float(M[q] << 16);
      rb -= __uint_as_float(M[q] & 0xffff0000u);
    } else if (st == 3) {
      L[q] = pack2(ra, rb);
    }
  }
};

// A slice of fp32 numbers in LDS: rows of 128 bytes, the first operand's 256,
// then the second's 128 (col_row); a row's 16-byte chunk c (4 k) sits at
// position c ^ (row & 7).
__device__ __forceinline__ uint32_t fp32_at(int row, int c) {
  return (uint32_t)row * (BK * 4) + 16u * (uint32_t)(c ^ (row & 7));
}

template <bool AK, bool BKM, bool VEC>
struct Stage {
  float v[6][8];        // A groups 0..3, B groups 4, 5
  uint32_t off[6];      // element offset of the group from the slice's base
  uint32_t at_a, at_b;  // byte offset of groups 0 and 4's chunk in its part in LDS
  __device__ __forceinline__ void setup(const GemmF32& p, int64_t i0, int64_t j0, int tid) {
#pragma unroll
    for (int g = 0; g < 4; ++g) {
      // rows beyond the operand repeat its last one (their results are not stored)
      const uint32_t o = (uint32_t)min<int64_t>(outer_a<AK>(g, tid), p.M - 1 - i0);
      off[g] = AK ? o * (uint32_t)p.lda + 8 * chunk_a<AK>(g, tid) : 8 * chunk_a<AK>(g, tid) * (uint32_t)p.lda + o;
    }
#pragma unroll
    for (int g = 0; g < 2; ++g) {
      const uint32_t o = (uint32_t)min<int64_t>(outer_b<BKM>(g, tid), p.N - 1 - j0);
      off[4 + g] = BKM ? o * (uint32_t)p.ldb + 8 * chunk_b<BKM>(g, tid)
                       : 8 * chunk_b<BKM>(g, tid) * (uint32_t)p.ldb + o;
    }
    at_a = chunk_at(outer_a<AK>(0, tid), chunk_a<AK>(0, tid));
    at_b = 3 * PA + chunk_at(col_row(outer_b<BKM>(0, tid)), chunk_b<BKM>(0, tid));
  }
  // group g of the whole slice whose k axis starts at a (A) / b (B)
  __device__ __forceinline__ void load(int g, const float* a, const float* b, int64_t lda, int64_t ldb) {
    const float* s = (g < 4 ? a : b) + off[g];
    const bool km = g < 4 ? AK : BKM;
    const int64_t ld = g < 4 ? lda : ldb;
    if (km && VEC) {
      const f32x4 x = reinterpret_cast<const f32x4*>(s)[0], y = reinterpret_cast<const f32x4*>(s)[1];
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        v[g][e] = x[e];
        v[g][4 + e] = y[e];
      }
    } else {
#pragma unroll
      for (int e = 0; e < 8; ++e) v[g][e] = km ? s[e] : s[e * ld];
    }
  }
  // group g of a slice that ends before k0 + 32 or lies in several segments;
  // k at or beyond khi are zero
  __device__ __forceinline__ void load_checked(int g, const GemmF32& p, const float* A, const float* B, int64_t i0,
                                               int64_t j0, int64_t k0, int64_t khi, int tid) {
    const bool is_a = g < 4, km = is_a ? AK : BKM;
    const int64_t o = is_a ? i0 + min<int64_t>(outer_a<AK>(g, tid), p.M - 1 - i0)
                           : j0 + min<int64_t>(outer_b<BKM>(g - 4, tid), p.N - 1 - j0);
    const int64_t k = k0 + 8 * (is_a ? chunk_a<AK>(g, tid) : chunk_b<BKM>(g - 4, tid));
    const float* P = is_a ? A : B;
    const int64_t ld = is_a ? p.lda : p.ldb, seg = is_a ? p.segA : p.segB;
    // the eight k lie in one segment when its length is a multiple of 8 (k is one)
    const bool one = p.kseg % 8 == 0 && k + 7 < khi;
    const int64_t k8 = one ? seg_off(k, p.kseg, seg) : 0;
#pragma unroll
    for (int e = 0; e < 8; ++e) {
      const int64_t ko = one ? k8 + e : seg_off(min(k + e, khi - 1), p.kseg, seg);
      const float x = km ? P[o * ld + ko] : P[ko * ld + o];
      v[g][e] = k + e < khi ? x : 0.0f;
    }
  }
  // all groups as fp32 numbers (fp32_at)
  __device__ __forceinline__ void store_fp32(char* buf, int tid) const {
#pragma unroll
    for (int g = 0; g < 6; ++g) {
      const int row = g < 4 ? outer_a<AK>(g, tid) : BM + col_row(outer_b<BKM>(g - 4, tid));
      const int c = 2 * (g < 4 ? chunk_a<AK>(g, tid) : chunk_b<BKM>(g - 4, tid));
#pragma unroll
      for (int t = 0; t < 2; ++t)
        *reinterpret_cast<f32x4*>(buf + fp32_at(row, c + t)) =
            f32x4{v[g][4 * t], v[g][4 * t + 1], v[g][4 * t + 2], v[g][4 * t + 3]};
    }
  }
  __device__ __forceinline__ void put(int g, char* buf, int part, const uint32_t (&w)[4]) const {
    // KMAJ: 64 rows further down; otherwise the same row's chunk g (A) or
    // (tid / 128) + 2 g (B), whose number is xored into its position
    const uint32_t at = g < 4 ? (AK ? at_a + (uint32_t)g * 64 * ROWB : at_a ^ (16u * (uint32_t)g))
                              : (BKM ? at_b + (uint32_t)(g - 4) * 64 * ROWB : at_b ^ (32u * (uint32_t)(g - 4)));
    *reinterpret_cast<u32x4*>(buf + at + part * (g < 4 ? PA : PB)) = u32x4{w[0], w[1], w[2], w[3]};
  }
  __device__ __forceinline__ void move(uint32_t d) {  // to the other buffer
    at_a += d;
    at_b += d;
  }
  // split and store all groups (outside the pipelined loop)
  __device__ __forceinline__ void store_all(char* buf, Range& rg) const {
    Split s;
#pragma unroll
    for (int g = 0; g < 6; ++g) {
#pragma unroll
      for (int q = 0; q < 4; ++q)
#pragma unroll
        for (int st = 0; st < 4; ++st) s.step(st, v[g], q, rg);
      put(g, buf, 0, s.H);
      put(g, buf, 1, s.M);
      put(g, buf, 2, s.L);
    }
  }
};

typedef f32x4 Acc[8][4];
typedef bf16x8 FragA[3];     // the parts of one 16-row tile
typedef bf16x8 FragB[3][4];  // the parts of the wave's four 16-column tiles

struct FragAt {
  uint32_t a, b[4];  // byte offsets of the h parts: row tile 0, the column tiles
  __device__ __forceinline__ FragAt plus(uint32_t d) const { return FragAt{a + d, {b[0] + d, b[1] + d, b[2] + d, b[3] + d}}; }
};

__device__ __forceinline__ bf16x8 frag(const char* buf, uint32_t at) {
  return __builtin_bit_cast(bf16x8, *reinterpret_cast<const u32x4*>(buf + at));
}
__device__ __forceinline__ bf16x8 frag_a(const char* buf, const FragAt& f, int i, int s) {
  return frag(buf, f.a + (uint32_t)(s * PA + i * 16 * ROWB));
}
__device__ __forceinline__ bf16x8 frag_b(const char* buf, const FragAt& f, int j, int s) {
  return frag(buf, f.b[j] + (uint32_t)(s * PB));
}

// Product q of the six: parts of the two operands, in the order that frees
// the second operand's parts one after the other, the leading product last.
constexpr int NP = 6;
constexpr int kPartA[NP] = {0, 0, 1, 1, 2, 0}, kPartB[NP] = {2, 1, 1, 0, 0, 0};
constexpr int PT = 4 * NP;  // products per row tile

__device__ __forceinline__ void lds_barrier() {
  __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup", "local");
  __builtin_amdgcn_s_barrier();
  __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "workgroup", "local");
}

__device__ __forceinline__ void clear(Acc& acc) {
#pragma unroll
  for (int i = 0; i < 8; ++i)
#pragma unroll
    for (int j = 0; j < 4; ++j) acc[i][j] = f32x4{0.0f, 0.0f, 0.0f, 0.0f};
}

// acc += the slice of fp32 numbers in buf: element e of the four lane groups'
// eight consecutive k are the four k of one 16x16x4 instruction.
__device__ __forceinline__ void fp32_slice(const char* buf, int wm, int wn, int lane, Acc& acc) {
  const int r = lane & 15, c = 2 * (lane >> 4);
  auto eight = [&](int row, f32x4 (&v)[2]) {
#pragma unroll
    for (int t = 0; t < 2; ++t) v[t] = *reinterpret_cast<const f32x4*>(buf + fp32_at(row, c + t));
  };
  f32x4 b[4][2];
#pragma unroll
  for (int j = 0; j < 4; ++j) eight(BM + col_row(wn * 64 + 4 * r + j), b[j]);
#pragma unroll
  for (int i = 0; i < 8; ++i) {
    f32x4 a[2];
    eight(wm * 128 + i * 16 + r, a);
#pragma unroll
    for (int j = 0; j < 4; ++j)
#pragma unroll
      for (int e = 0; e < 8; ++e)
        acc[i][j] = __builtin_amdgcn_mfma_f32_16x16x4f32(a[e >> 2][e & 3], b[j][e >> 2][e & 3], acc[i][j], 0, 0, 0);
  }
}

// f(0), ..., f(N - 1) with the index a constant (as integral_constant).
template <class F, int... I>
__device__ __forceinline__ void static_for_seq(const F& f, std::integer_sequence<int, I...>) {
  (f(std::integral_constant<int, I>()), ...);
}
template <int N, class F>
__device__ __forceinline__ void static_for(const F& f) {
  static_for_seq(f, std::make_integer_sequence<int, N>());
}

// One slice of the pipelined loop: the 192 products of the slice that f
// points at, in program order, and between them the reads of its other row
// tiles, the splitting of the staged slice into the buffer that sg points at,
// the loads of the slice at (na, nb) into the stage, the barrier, and the reads
// of the next slice's first fragments (fn), each over one whose last product is issued: on entry a[0] and
// parts 2 and 1 of b hold this slice's (part 0 is read here), on return the
// next one's.
template <bool AK, bool BKM, bool VEC>
__device__ __forceinline__ void pipelined_slice(SplitLDS& sm, const FragAt& f, const FragAt& fn,
                                                Stage<AK, BKM, VEC>& sg, Range& rg, const float* na, const float* nb,
                                                int64_t lda, int64_t ldb, FragA (&a)[2], FragB& b, Acc& hi, Acc& lo) {
  char* buf = sm.p;
  Split sp;
  static_for<8 * PT>([&](auto mc) {
    constexpr int m = decltype(mc)::value;
    constexpr int i = m / PT, q = (m % PT) / 4, j = m % 4;
    constexpr int last = m - 7 * PT;  // product of the last row tile
    f32x4& c = kPartA[q] + kPartB[q] == 0 ? hi[i][j] : lo[i][j];
    c = __builtin_amdgcn_mfma_f32_16x16x32_bf16(a[i & 1][kPartA[q]], b[kPartB[q]][j], c, 0, 0, 0);
    if constexpr (m < 4) b[0][m] = frag_b(buf, f, m, 0);
    // the next row tile's parts, in the order of their use
    if constexpr (i < 7 && m % 4 == 1 && m % PT < 12) {
      constexpr int s = m % PT / 4;
      a[(i + 1) & 1][s] = frag_a(buf, f, i + 1, s);
    }
    if constexpr (m < 24 * NP) {  // NP products per two entries
      constexpr int pr = m / NP, st = m % NP, g = pr / 4, e = pr % 4;
      sp.step(st, sg.v[g], e, rg);
      if constexpr (e == 3 && st == 1) sg.put(g, buf, 0, sp.H);
      if constexpr (e == 3 && st == 3) sg.put(g, buf, 1, sp.M);
      if constexpr (e == 3 && st == 4) sg.put(g, buf, 2, sp.L);
      if constexpr (e == 3 && st == 5) sg.load(g, na, nb, lda, ldb);
    }
    if constexpr (last == -11) lds_barrier();  // every read of buf but the last wave's a tile has landed
    if constexpr (last == 1 || last == 3 || last == 5) a[0][last / 2] = frag_a(buf, fn, 0, last / 2);
    if constexpr (last >= 4 && last < 8) b[2][last - 4] = frag_b(buf, fn, last - 4, 2);
    if constexpr (last >= 12 && last < 16) b[1][last - 12] = frag_b(buf, fn, last - 12, 1);
    __builtin_amdgcn_sched_barrier(0);
  });
}

// Tile of workgroup b of one batch entry or k split.  Workgroups go round
// robin to the 8 XCDs; each XCD takes whole tile rows (columns when the k
// range depends on the column), so that its L2 serves the row's operand to
// all of its workgroups.  The rows are dealt longest first (with a triangular
// operand the k range grows along them) and back and forth, so that the
// XCDs' shares are alike; those left over after the last full eight go round
// robin by tile.
__device__ __forceinline__ void tile_of(uint32_t b, uint32_t gx, uint32_t gy, int flags, uint32_t& bx,
                                        uint32_t& by) {
  const bool cols = (flags & (kKHiCol | kKLoCol)) != 0;
  const uint32_t no = cols ? gy : gx, ni = cols ? gx : gy;
  const uint32_t full = no / 8;
  uint32_t rank, in;
  if (b < full * 8 * ni) {
    const uint32_t x = b & 7, idx = b >> 3, g = idx / ni;
    rank = g * 8 + ((g & 1) ? 7 - x : x);
    in = idx % ni;
  } else {
    const uint32_t u = b - full * 8 * ni, rest = no - full * 8;
    rank = full * 8 + u % rest;
    in = u / rest;
  }
  if (flags & (kKHiRow | kKHiCol)) rank = no - 1 - rank;
  bx = cols ? in : rank;
  by = cols ? rank : in;
}

template <bool AK, bool BKM, bool VEC, bool DEEP>
__global__ __launch_bounds__(256, 1) void k_gemm_split(GemmF32 p, uint32_t gx, uint32_t gy) {
  if (ff_halted(p.st)) return;
  uint32_t bx, by;
  if (p.flags & kCLower) {
    // square output: 2 (bx + 1) column tiles reach the lower triangle of row tile bx
    const uint32_t b = xcd_remap(blockIdx.x, gridDim.x);
    bx = (uint32_t)((sqrtf(4.0f * (float)b + 1.0f) - 1.0f) * 0.5f);
    while (bx * (bx + 1) > b) --bx;
    while ((bx + 1) * (bx + 2) <= b) ++bx;
    by = b - bx * (bx + 1);
    if (by >= gy) return;
  } else {
    tile_of(blockIdx.x, gx, gy, p.flags, bx, by);
  }
  const int64_t i0 = (int64_t)bx * BM, j0 = (int64_t)by * BN;
  const float* A = p.A;
  const float* B = p.B;
  float* C = p.C;
  int64_t klo = 0, khi = p.K;
  if (p.flags & kKHiRow) khi = min(khi, i0 + BM);
  if (p.flags & kKLoRow) klo = max(klo, i0);
  if (p.flags & kKHiCol) khi = min(khi, j0 + BN);
  if (p.flags & kKLoCol) klo = max(klo, j0);
  if (p.ksplit > 1) {
    const int64_t span = khi > klo ? khi - klo : 0;
    const int64_t chunk = ((span + p.ksplit - 1) / p.ksplit + BK - 1) / BK * BK;
    klo = klo + (int64_t)blockIdx.y * chunk;
    khi = min(khi, klo + chunk);
    C += (int64_t)blockIdx.y * p.sC;
  } else {
    A += (int64_t)blockIdx.y * p.sA;
    B += (int64_t)blockIdx.y * p.sB;
    C += (int64_t)blockIdx.y * p.sC;
  }
  __shared__ SplitLDS sm;
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int wm = wave >> 1, wn = wave & 1;
  Acc acc;
  clear(acc);
  if (klo < khi) {
    FragAt f;
    f.a = chunk_at(wm * 128 + (lane & 15), lane >> 4);
#pragma unroll
    for (int j = 0; j < 4; ++j) f.b[j] = 3 * PA + chunk_at(col_row(wn * 64 + 4 * (lane & 15) + j), lane >> 4);
    Stage<AK, BKM, VEC> sg;
    sg.setup(p, i0, j0, tid);
    // whole slices, each in one segment (otherwise all take the checked path)
    const bool segs = p.kseg == 0 || p.kseg % BK == 0;
    const int n = segs ? (int)((khi - klo) / BK) : 0;
    if (tid == 0) {
      sm.big = 0u;
      sm.tiny = sm.wide = 0;
    }
    lds_barrier();
    if (n > 0) {
      Range rg;
      // base of the slice to load next, moved along until the last one
      int64_t in = klo;
      const float* na = A + (AK ? i0 * p.lda : i0);
      const float* nb = B + (BKM ? j0 * p.ldb : j0);
      const int64_t ka = AK ? 1 : p.lda, kb = BKM ? 1 : p.ldb;
      if (p.kseg) {
        in = klo % p.kseg;
        na += (in + (klo / p.kseg) * p.segA) * ka;
        nb += (in + (klo / p.kseg) * p.segB) * kb;
      } else {
        na += klo * ka;
        nb += klo * kb;
      }
      int at = 0;
      auto advance = [&]() {
        if (++at >= n) return;  // the last slice is loaded again, for nothing
        in += BK;
        na += BK * ka;
        nb += BK * kb;
        if (p.kseg && in >= p.kseg) {
          in -= p.kseg;
          na += (p.segA - p.kseg) * ka;
          nb += (p.segB - p.kseg) * kb;
        }
      };
#pragma unroll
      for (int g = 0; g < 6; ++g) sg.load(g, na, nb, p.lda, p.ldb);
      advance();
      sg.store_all(sm.p, rg);
#pragma unroll
      for (int g = 0; g < 6; ++g) sg.load(g, na, nb, p.lda, p.ldb);
      advance();
      lds_barrier();
      FragA a[2];
      FragB b;
#pragma unroll
      for (int t = 0; t < 3; ++t) {
        a[0][t] = frag_a(sm.p, f, 0, t);
        if (t > 0)
#pragma unroll
          for (int j = 0; j < 4; ++j) b[t][j] = frag_b(sm.p, f, j, t);
      }
      uint32_t d = BUF;  // from the buffer in use to the other one
      FragAt fc = f;
      if constexpr (DEEP) {
        // a fresh accumulator per CHUNK slices, added to the total
        for (int s = 0; s < n;) {
          Acc loc;
          clear(loc);
          const int e = min(n, s + CHUNK);
          for (; s < e; ++s) {
            const FragAt fn = fc.plus(d);
            sg.move(d);
            pipelined_slice(sm, fc, fn, sg, rg, na, nb, p.lda, p.ldb, a, b, loc, loc);
            advance();
            fc = fn;
            d = 0u - d;
          }
#pragma unroll
          for (int i = 0; i < 8; ++i)
#pragma unroll
            for (int j = 0; j < 4; ++j) acc[i][j] += loc[i][j];
        }
      } else {
        // the products with a lower part, at most 2^-7 of the leading ones,
        // go into an accumulator of their own, so that the total is rounded
        // once per 32 k
        Acc lo;
        clear(lo);
        for (int s = 0; s < n; ++s) {
          const FragAt fn = fc.plus(d);
          sg.move(d);
          pipelined_slice(sm, fc, fn, sg, rg, na, nb, p.lda, p.ldb, a, b, acc, lo);
          advance();
          fc = fn;
          d = 0u - d;
        }
#pragma unroll
        for (int i = 0; i < 8; ++i)
#pragma unroll
          for (int j = 0; j < 4; ++j) acc[i][j] += lo[i][j];
      }
      if (__any(rg.wide())) sm.wide = 1;
      if (__any(rg.tiny())) sm.tiny = 1;
      lds_barrier();
      if (__builtin_amdgcn_readfirstlane(sm.tiny) != 0) {
        atomicMax(&sm.big, __float_as_uint(rg.big));
        lds_barrier();
        const float reach = kTinyReach * (float)(khi - klo) * __uint_as_float(sm.big);
        float least = INFINITY;
#pragma unroll
        for (int i = 0; i < 8; ++i)
#pragma unroll
          for (int j = 0; j < 4; ++j)
#pragma unroll
            for (int r = 0; r < 4; ++r) least = fminf(least, fabsf(acc[i][j][r]));
        if (__any(!(least >= reach))) sm.wide = 1;
        lds_barrier();
      }
    }
    int64_t k = klo + (int64_t)n * BK;
    if (__builtin_amdgcn_readfirstlane(sm.wide) != 0) {
      clear(acc);
      k = klo;
    }
    auto fp32_part = [&](int64_t ke, Acc& c) {
      for (; k < ke; k += BK) {
#pragma unroll
        for (int g = 0; g < 6; ++g) sg.load_checked(g, p, A, B, i0, j0, k, khi, tid);
        sg.store_fp32(sm.p, tid);
        lds_barrier();
        fp32_slice(sm.p, wm, wn, lane, c);
        lds_barrier();
      }
    };
    if constexpr (DEEP) {
      while (k < khi) {
        Acc loc;
        clear(loc);
        fp32_part(min(khi, k + FP32_CHUNK * BK), loc);
#pragma unroll
        for (int i = 0; i < 8; ++i)
#pragma unroll
          for (int j = 0; j < 4; ++j) acc[i][j] += loc[i][j];
      }
    } else {
      fp32_part(khi, acc);
    }
  }
  // lane c of a row of 16 holds columns 4 c .. 4 c + 3 of the wave's half
  const bool lower = (p.flags & kCLower) != 0;
  const bool use_beta = p.ksplit <= 1 && p.beta != 0.0f;
  const bool vec_c = p.ldc % 4 == 0 && (reinterpret_cast<uintptr_t>(C) & 15) == 0;
  const int64_t j = j0 + wn * 64 + 4 * (lane & 15);
#pragma unroll
  for (int t = 0; t < 8; ++t)
#pragma unroll
    for (int r = 0; r < 4; ++r) {
      const int64_t i = i0 + wm * 128 + t * 16 + 4 * (lane >> 4) + r;
      if (i >= p.M || j >= p.N || (lower && i < j)) continue;
      float* c = C + i * p.ldc + j;
      f32x4 v = {acc[t][0][r], acc[t][1][r], acc[t][2][r], acc[t][3][r]};
      v *= p.alpha;
      if (vec_c && j + 3 < p.N && (!lower || i >= j + 3)) {
        if (use_beta) v += p.beta * *reinterpret_cast<const f32x4*>(c);
        *reinterpret_cast<f32x4*>(c) = v;
      } else {
#pragma unroll
        for (int e = 0; e < 4; ++e)
          if (j + e < p.N && (!lower || i >= j + e)) c[e] = use_beta ? v[e] + p.beta * c[e] : v[e];
      }
    }
}

}  // namespace

hipError_t launch_gemm_split(const GemmF32& p, int batch, bool vec, bool deep, hipStream_t s) {
  const bool lower = (p.flags & kCLower) != 0;
  // 32-bit element offsets within a tile's slice
  if ((lower && p.M != p.N) || p.lda > kSplitMaxLd || p.ldb > kSplitMaxLd) return hipErrorInvalidValue;
  const int64_t gx = (p.M + BM - 1) / BM, gy = (p.N + BN - 1) / BN;
  const int gz = p.ksplit > 1 ? p.ksplit : batch;
  const int64_t tiles = lower ? gx * (gx + 1) : gx * gy;
  if (tiles > 0x7fffffff || gz > 65535) return hipErrorInvalidValue;
  const dim3 grid((uint32_t)tiles, (uint32_t)gz);
  switch ((p.transA ? 1 : 0) | (p.transB ? 2 : 0) | (vec ? 4 : 0) | (deep ? 8 : 0)) {
#define FF_SPLIT_CASE(c, ak, bk, v, d)                                                                     \
    case c:                                                                                                \
      hipLaunchKernelGGL((k_gemm_split<ak, bk, v, d>), grid, dim3(256), 0, s, p, (uint32_t)gx, (uint32_t)gy); \
      break;
    FF_SPLIT_CASE(0, true, false, false, false)
    FF_SPLIT_CASE(1, false, false, false, false)
    FF_SPLIT_CASE(2, true, true, false, false)
    FF_SPLIT_CASE(3, false, true, false, false)
    FF_SPLIT_CASE(4, true, false, true, false)
    FF_SPLIT_CASE(5, false, false, true, false)
    FF_SPLIT_CASE(6, true, true, true, false)
    FF_SPLIT_CASE(7, false, true, true, false)
    FF_SPLIT_CASE(8, true, false, false, true)
    FF_SPLIT_CASE(9, false, false, false, true)
    FF_SPLIT_CASE(10, true, true, false, true)
    FF_SPLIT_CASE(11, false, true, false, true)
    FF_SPLIT_CASE(12, true, false, true, true)
    FF_SPLIT_CASE(13, false, false, true, true)
    FF_SPLIT_CASE(14, true, true, true, true)
    default:
      hipLaunchKernelGGL((k_gemm_split<false, true, true, true>), grid, dim3(256), 0, s, p, (uint32_t)gx, (uint32_t)gy);
      break;
#undef FF_SPLIT_CASE
  }
  return hipGetLastError();
}

}  // namespace ff
