// Dense and convolution layers as one MFMA GEMM kernel on fp32 operands (gfx950).
//
// C[M][N] = sum_k A[m][k] B[k][n].  The fp32 matrix instructions of gfx950 run
// at a sixteenth of the bfloat16 ones' rate (157 TFLOP/s against 2.5 PFLOP/s),
// so each fp32 value is split, exactly, into three bfloat16 pieces h + m + l
// and x y is the sum of the six largest piece products, accumulated in fp32:
// a ceiling of 416 TFLOP/s instead of 157.  The result is closer to the exact
// one than fp32 products gave, because the matrix instruction rounds its
// accumulator once per 16 terms instead of at each: relative error at a
// reduction of 1024, 4.9e-7 in one accumulator and half of that with the small
// products in a second one, against 5.7e-7; at 5 terms, 2.7e-8 against 4.4e-8.
// For a single term it is not (2.60e-8 against 2.53e-8): reductions of up to
// kFewTerms terms use fp32 products, in kernels of their own.
// 12288 x 1024 x 4096: 0.80 ms (129 TFLOP/s) with fp32 products, 0.57 ms (180)
// split; at that rate the card's power limit holds the clock at 1.8 GHz, and
// a large library product in bfloat16 reaches 1280 TFLOP/s, 213 in these units.
//
// A 256-thread workgroup computes a tile of C (128 x 128 in general; shapes
// below); each of its four wave64s owns a part of it made of 32 x 32 blocks.
// K is walked in tiles of 32 through one LDS buffer: every thread has its
// values of tile t+1 in flight from global memory while the waves multiply
// tile t, then splits and stores them between two barriers.  Two or three
// workgroups share a CU, so that one multiplies while another splits.
//
// Operands reach LDS through loaders, one per way the operand sits in
// memory: plain row-major matrices (contiguous along k, or along m / n) and
// the implicit-GEMM views of NHWC convolutions (forward: the input patches;
// input gradient: the output gradient gathered through the filter taps;
// filter gradient: the input patches seen along the batch-pixel axis).  A
// loader zero-fills everything outside the matrix, so no shape needs
// padding.  A convolution whose channel count is a multiple of 32 has
// every K tile inside one filter tap (uniform over the workgroup), and the
// remaining index splits use multiply-high division by invariant integers.
// The input gradient of a strided convolution is computed per stride class
// of input pixels (h mod st, w mod st), each class a GEMM over only the taps
// that reach it.
//
// Split-K: the filter gradients reduce over N P Q pixels or over the rows of
// a dense layer (up to millions), so the grid's second dimension cuts that
// axis into slices whose partial tiles go to separate buffers and are summed
// afterwards in slice order.  A dense layer's bias gradient (the column sums
// of dY) is summed in fp32 from the values the workgroups of the first tile
// column load for A, slice by slice like dW.  No atomics anywhere: results
// do not depend on scheduling or addresses.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <cstdint>
#include <type_traits>

#include "kernels.h"

namespace ooc {

namespace {

constexpr int BK = 32;
constexpr int THREADS = 256;
constexpr uint32_t kXcds = 8;   // accelerator complex dies of an MI355X, one L2 each

typedef float floatx16 __attribute__((ext_vector_type(16)));
typedef float floatx2 __attribute__((ext_vector_type(2)));
typedef __bf16 bf16x2 __attribute__((ext_vector_type(2)));
typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));

__device__ inline float4 zero4() { return make_float4(0.f, 0.f, 0.f, 0.f); }

// ---------------------------------------------------------------- loaders
// A loader feeds one operand tile of extent E (tile rows along m or n) by 32
// along k.  init(mn0, MN) runs once per workgroup (mn0 = tile origin, MN =
// extent of the matrix), fetch(k0, kend, r) loads this thread's E / 8 values
// of the K tile starting at k0 as E / 32 float4.  Values at k >= kend are zero
// (they enter every dot product), also where the whole tile lies past kend.
//
// The common views load through buffer descriptors: a base that is uniform
// over the workgroup and moves with the K tile, a 32-bit byte offset per lane
// that does not, and the descriptor's length.  What lies past the length reads
// as zero without a memory access, so a lane with nothing to load takes the
// offset kNone, and the rows past a matrix's last need no test at all.  Loads
// are 16 bytes wide at any 4-byte alignment.  Against 64-bit addresses with a
// select per load this saves 20 to 40 registers a lane, and rows that are not
// multiples of 4 need no scalar loads (1379 x 765 x 3067: 0.120 ms with them,
// 0.060 without).  Rows and columns past M or N that are in bounds read their
// neighbours: they only reach C entries that are never stored.  The general views
// (matrices with rows of more than kMaxLd values, images too large for 32-bit
// offsets, gradient taps of channel counts that are not multiples of 4) form
// 64-bit addresses per value; their masked lanes load from a block of zeros.
constexpr uint32_t kNone = 0x80000000u;   // past the length of every descriptor
constexpr int64_t kMaxLd = int64_t(1) << 21;   // 255 rows of it stay below 2^31 bytes

// `values` floats from p on (at most 2^29, the length that kNone is past)
__device__ inline __amdgpu_buffer_rsrc_t buffer(const float* p, int64_t values) {
  const int64_t n = values < 0 ? 0 : values > (int64_t(1) << 29) ? (int64_t(1) << 29) : values;
  return __builtin_amdgcn_make_buffer_rsrc(const_cast<float*>(p), 0, (int)((uint32_t)n * 4u),
                                           0x00020000);
}
__device__ inline float4 ldb(__amdgpu_buffer_rsrc_t r, uint32_t off) {
  return __builtin_bit_cast(float4, __builtin_amdgcn_raw_buffer_load_b128(r, (int)off, 0, 0));
}
__device__ inline float ldb1(__amdgpu_buffer_rsrc_t r, uint32_t off) {
  return __builtin_bit_cast(float, __builtin_amdgcn_raw_buffer_load_b32(r, (int)off, 0, 0));
}

// What masked lanes of the general views load (never written).
__device__ __attribute__((aligned(16))) float g_zero[64] = {};

__device__ inline float4 ld4(const float* p) { return *reinterpret_cast<const float4*>(p); }

// Pins v in a register at this point.  The compiler would otherwise move an
// address computation that only a masked select uses into a branch around
// it, which is what the loaders avoid.
template <class T>
__device__ inline void keep(T& v) {
  asm volatile("" : "+v"(v));
}

// ---------------------------------------------------------------- split operands
// x 2^40 = h + m + l, each a bfloat16: h = bf16(x'), m = bf16(x' - h), l = x' - h - m.
// Rounding to nearest leaves remainders of at most 16 and then 8 bits, so the
// split is exact; the scale puts the smallest subnormal x at 2^-109, so that
// no piece is a subnormal bfloat16.  |x| >= 2^87 overflows; the kernel then
// recomputes its tile (see gemm_kernel).  The remainders are single two-term
// dot products with (-1, 0) and (0, -1): 4.5 vector instructions per value.
//
// The matrix instruction aligns its 16 products and the accumulator to the largest and cuts off
// what falls below: of the accumulator towards minus infinity, of each product towards zero, at
// 2^-24 of the largest (seen on single products).  Each result is closer to the exact one than
// fp32 products give, but such errors share a sign, and sums over many of them show it.
//
// The accumulator's: about 5e-8 of a typical result; a sum over 8192 rows (a bias or normalisation
// gradient) came out 5e-6 off instead of 6e-7.  So odd rows of either operand are negated (scale
// -2^40) and odd outputs (row + column) negated back: with the signs alternating along both
// directions it cancels in such sums.
//
// The products': h h has 16 bits, so every product below 2^-8 of the largest is cut, and where the
// terms of a column share a sign (inputs behind a ReLU, gradients that a mask has thinned out) the
// cuts of a column do too, whatever the outputs' signs: about 5e-10 of a typical result, which in
// sums over a convolution's pixels outgrows the rounding of fp32 products.  Sums of 200704 products
// of non-negative rows at K = 64 were off by 2.5e-7 sqrt(rows) of a typical result instead of
// 1.0e-7, the shift gradient of a batch normalisation behind a 7 x 7 convolution by 7.0e-5 instead
// of 4.6e-5.  Convolutions therefore give one operand's h only 6 bits (NARROW; h is rounded half
// away from zero, which leaves remainders of 17 bits and then 8: still exact), so that products
// have 14: 0.95e-7, 5.6e-5, and gradients of the network's other layers at 0.5 to 1.0 of the error
// of fp32 products.  Two instructions a value more for that operand: steps of convolution networks
// 0.98 to 1.01 times as long.  The rows of dense layers are fewer and their sums don't cancel.
constexpr float kSplitScale = 0x1p40f, kSplitUnscale = 0x1p-80f;
constexpr int kPieces = 3;
// At 2 terms the split's error is 2.6e-8 (3.4e-8 with a 6-bit h) and that of fp32 products 3.1e-8, at
// 3 2.7e-8 (3.4e-8) and 3.6e-8; four are what one step of fp32 instructions takes.
constexpr int kFewTerms = 4;

template <bool NARROW>
__device__ __forceinline__ void split2(float x, float y, float scale, uint32_t (&o)[kPieces]) {
  // (-1, 0) and (0, -1) as register operands: as constants, the compiler would encode one of them
  // as an inline -1.0, which this instruction does not read as a pair (wrong results measured)
  uint32_t c0 = 0x0000bf80u, c1 = 0xbf800000u;
  asm("" : "+s"(c0), "+s"(c1));
  const bf16x2 first = __builtin_bit_cast(bf16x2, c0), second = __builtin_bit_cast(bf16x2, c1);
  x *= scale;
  y *= scale;
  bf16x2 h;
  if constexpr (NARROW) {   // rounded half away from zero; an infinity stays one
    const uint32_t hx = (__builtin_bit_cast(uint32_t, x) + 0x00020000u) & 0xfffc0000u;
    const uint32_t hy = (__builtin_bit_cast(uint32_t, y) + 0x00020000u) & 0xfffc0000u;
    h = __builtin_bit_cast(bf16x2, __builtin_amdgcn_perm(hy, hx, 0x07060302u));
    x -= __builtin_bit_cast(float, hx);
    y -= __builtin_bit_cast(float, hy);
  } else {
    h = __builtin_convertvector((floatx2){x, y}, bf16x2);
    x = __builtin_amdgcn_fdot2_f32_bf16(h, first, x, false);
    y = __builtin_amdgcn_fdot2_f32_bf16(h, second, y, false);
  }
  const bf16x2 m = __builtin_convertvector((floatx2){x, y}, bf16x2);
  x = __builtin_amdgcn_fdot2_f32_bf16(m, first, x, false);
  y = __builtin_amdgcn_fdot2_f32_bf16(m, second, y, false);
  const bf16x2 l = __builtin_convertvector((floatx2){x, y}, bf16x2);
  o[0] = __builtin_bit_cast(uint32_t, h);
  o[1] = __builtin_bit_cast(uint32_t, m);
  o[2] = __builtin_bit_cast(uint32_t, l);
}

__device__ inline float comp(const float4& v, int t) {
  return t == 0 ? v.x : t == 1 ? v.y : t == 2 ? v.z : v.w;
}

// fp32 row-of-k tiles [E][32] keep k quad q of row i in slot q ^ (i mod 8).
__device__ inline int rowk_index(int i, int k) { return i * BK + ((((k >> 2) ^ i) & 7) << 2) + (k & 3); }

// Split tiles: three pieces of E rows x 32 k of bfloat16, 64 bytes a row in
// four 16-byte octets of k.  octet(r, o) is the byte offset of octet o of row
// r in its piece; the octets are swizzled within the row so that the 16 rows
// of any 256 bytes' worth of reads, and the writes of either thread map, cover
// all banks.  Row-of-m tiles also order rows by r mod 4 first, because their
// threads write rows 4 q + e for consecutive q.
template <int E>
struct RowK {
  static constexpr bool kRowOfK = true;
  static constexpr bool kPixels = false;
  static constexpr int kN = E / 32;
  static constexpr int kLds = E * BK;            // floats of the fp32 tile
  static constexpr int kPiece = E * BK * 2;      // bytes of one piece
  __device__ static int row(int j) { return (threadIdx.x >> 3) + 32 * j; }
  __device__ static int koff() { return (threadIdx.x & 7) * 4; }
  __device__ static void store(float* lds, const float4 (&r)[kN]) {
#pragma unroll
    for (int j = 0; j < kN; ++j)
      *reinterpret_cast<float4*>(&lds[rowk_index(row(j), koff())]) = r[j];
  }
  __device__ static int octet(int r, int o) { return r * 64 + (((o ^ (r >> 2)) & 3) << 4); }
  template <bool NARROW>
  __device__ static void split_store(char* lds, const float4 (&r)[kN]) {
    const int q = threadIdx.x & 7;
    const float scale = row(0) & 1 ? -kSplitScale : kSplitScale;   // the same parity for every j
#pragma unroll
    for (int j = 0; j < kN; ++j) {
      uint32_t u[kPieces], v[kPieces];
      split2<NARROW>(r[j].x, r[j].y, scale, u);
      split2<NARROW>(r[j].z, r[j].w, scale, v);
      char* d = lds + octet(row(j), q >> 1) + (q & 1) * 8;
#pragma unroll
      for (int p = 0; p < kPieces; ++p) *reinterpret_cast<uint2*>(d + p * kPiece) = make_uint2(u[p], v[p]);
    }
  }
};
// A thread loads kItems blocks of four consecutive m by kR consecutive k, so
// that it can write kR consecutive k of a row at once; value j of a thread is
// k row krow(j) at m offset moff(j).
template <int E>
struct RowM {
  static constexpr bool kRowOfK = false;
  static constexpr bool kPixels = false;
  static constexpr int kN = E / 32;
  static constexpr int kItems = E == 192 ? 3 : 1;
  static constexpr int kR = kN / kItems;
  static constexpr int kLds = BK * E;
  static constexpr int kPiece = E * BK * 2;
  static_assert(kR == 1 || kR == 2 || kR == 4 || kR == 8, "k rows per thread");
  __device__ static int item(int j) { return (int)threadIdx.x + 256 * (j / kR); }
  __device__ static int krow(int j) { return item(j) / (E / 4) * kR + j % kR; }
  __device__ static int moff(int j = 0) { return item(j) % (E / 4) * 4; }
  __device__ static void store(float* lds, const float4 (&r)[kN]) {
#pragma unroll
    for (int j = 0; j < kN; ++j) *reinterpret_cast<float4*>(&lds[krow(j) * E + moff(j)]) = r[j];
  }
  __device__ static int octet(int r, int o) {
    return ((r >> 2) + (r & 3) * (E / 4)) * 64 + (((o ^ r ^ (r >> 4)) & 3) << 4);
  }
  template <bool NARROW>
  __device__ static void split_store(char* lds, const float4 (&r)[kN]) {
#pragma unroll
    for (int i = 0; i < kItems; ++i) {
      const int k = krow(i * kR), m = moff(i * kR);
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        char* d = lds + octet(m + e, k >> 3) + (k & 7) * 2;
        uint32_t u[(kR + 1) / 2][kPieces];
#pragma unroll
        for (int j = 0; j < (kR + 1) / 2; ++j)
          split2<NARROW>(comp(r[i * kR + 2 * j], e), kR > 1 ? comp(r[i * kR + 2 * j + (kR > 1)], e) : 0.f,
                 e & 1 ? -kSplitScale : kSplitScale, u[j]);
#pragma unroll
        for (int p = 0; p < kPieces; ++p) {
          char* dp = d + p * kPiece;
          if constexpr (kR == 1)
            *reinterpret_cast<uint16_t*>(dp) = (uint16_t)u[0][p];
          else if constexpr (kR == 2)
            *reinterpret_cast<uint32_t*>(dp) = u[0][p];
          else if constexpr (kR == 4)
            *reinterpret_cast<uint2*>(dp) = make_uint2(u[0][p], u[1][p]);
          else
            *reinterpret_cast<uint4*>(dp) = make_uint4(u[0][p], u[1][p], u[2][p], u[3][p]);
        }
      }
    }
  }
};

// x / d for 0 <= x < 2^31 and an invariant d >= 1 with one multiply-high
// (Granlund and Montgomery, division by invariant integers using
// multiplication, 1994): with l = ceil(log2 d) and m = floor(2^(31+l) / d) + 1,
// 2^(31+l) < m d <= 2^(31+l) + 2^l, hence floor(x m / 2^(31+l)) = floor(x / d)
// for every x < 2^31, and m < 2^32.  d = 1 takes m = 2^32 - 1 and adds one
// to x first: floor((x + 1)(2^32 - 1) / 2^32) = x for x + 1 <= 2^32.  Both
// cases are the same instructions, so a division never branches.
struct FastDiv {
  uint32_t d = 1, m = 0xffffffffu, s = 0, a = 1;
  static FastDiv make(int64_t dv) {
    FastDiv f;
    f.d = (uint32_t)dv;
    if (dv <= 1) return f;
    uint32_t l = 0;
    while ((1ull << l) < (uint64_t)dv) ++l;
    f.m = (uint32_t)((1ull << (31 + l)) / (uint64_t)dv + 1);
    f.s = l - 1;
    f.a = 0;
    return f;
  }
  __device__ int div(int x) const { return (int)(__umulhi((uint32_t)x + a, m) >> s); }
};

constexpr int kFar = -(1 << 29);   // coordinate of a row past the matrix: fails every bounds check

__device__ inline bool inside(int v, int n) { return (unsigned)v < (unsigned)n; }

// X[i][k] = p[i * ld + k] (contiguous along k), kdim values in every row
template <int E>
struct MatK : RowK<E> {
  using Base = RowK<E>;
  const float* p;
  int64_t ld, kdim;
  int64_t end;                // values from the tile's first row on
  uint32_t off_[Base::kN];    // bytes from the tile's first row, at this lane's k offset
  __device__ void init(int64_t mn0, int64_t MN) {
    p += mn0 * ld;
    end = (MN - 1 - mn0) * ld + kdim;
#pragma unroll
    for (int j = 0; j < Base::kN; ++j) off_[j] = (uint32_t)((Base::row(j) * ld + Base::koff()) * 4);
  }
  __device__ void fetch(int64_t k0, int64_t kend, float4 (&r)[Base::kN]) const {
    const auto b = buffer(p + k0, k0 < kend ? end - k0 : 0);
#pragma unroll
    for (int j = 0; j < Base::kN; ++j) r[j] = ldb(b, off_[j]);
    if (k0 + BK > kend) {   // the last tile: what follows kend in the row is not zero
      const int left = (int)(kend - k0) - Base::koff();
#pragma unroll
      for (int j = 0; j < Base::kN; ++j) {
        r[j].x = left > 0 ? r[j].x : 0.f;
        r[j].y = left > 1 ? r[j].y : 0.f;
        r[j].z = left > 2 ? r[j].z : 0.f;
        r[j].w = left > 3 ? r[j].w : 0.f;
      }
    }
  }
};

// X[i][k] = p[k * ld + i] (contiguous along m or n).  The descriptor ends with row kend - 1.
template <int E>
struct MatM : RowM<E> {
  using Base = RowM<E>;
  const float* p;
  int64_t ld, kdim;
  int64_t cols;               // values of a row from the tile's first column on
  uint32_t off_[Base::kN];
  __device__ void init(int64_t mn0, int64_t MN) {
    p += mn0;
    cols = MN - mn0;
#pragma unroll
    for (int j = 0; j < Base::kN; ++j) off_[j] = (uint32_t)((Base::krow(j) * ld + Base::moff(j)) * 4);
  }
  __device__ void fetch(int64_t k0, int64_t kend, float4 (&r)[Base::kN]) const {
    const auto b = buffer(p + k0 * ld, k0 < kend ? (kend - 1 - k0) * ld + cols : 0);
#pragma unroll
    for (int j = 0; j < Base::kN; ++j) r[j] = ldb(b, off_[j]);
  }
};

// The pixel operand of a 1 x 1 convolution, which is a plain matrix
template <int E>
struct PixelK : MatK<E> {
  static constexpr bool kPixels = true;
};
template <int E>
struct PixelM : MatM<E> {
  static constexpr bool kPixels = true;
};

// The same two views with 64-bit addresses, for ld > kMaxLd
template <int E>
struct MatKFar : RowK<E> {
  using Base = RowK<E>;
  const float* p;
  int64_t ld, kdim;
  int64_t off_[Base::kN];   // (row, clamped to the matrix) * ld + this lane's k offset
  __device__ void init(int64_t mn0, int64_t MN) {
#pragma unroll
    for (int j = 0; j < Base::kN; ++j) {
      const int64_t i = mn0 + Base::row(j);
      off_[j] = (i < MN ? i : 0) * ld + Base::koff();
    }
  }
  __device__ void fetch(int64_t k0, int64_t kend, float4 (&r)[Base::kN]) const {
    const int64_t k = k0 + Base::koff();
#pragma unroll
    for (int j = 0; j < Base::kN; ++j) {
      const float* q = p + off_[j] + k0;
      r[j].x = *(k + 0 < kend ? q + 0 : g_zero);
      r[j].y = *(k + 1 < kend ? q + 1 : g_zero);
      r[j].z = *(k + 2 < kend ? q + 2 : g_zero);
      r[j].w = *(k + 3 < kend ? q + 3 : g_zero);
    }
  }
};
template <int E>
struct MatMFar : RowM<E> {
  using Base = RowM<E>;
  const float* p;
  int64_t ld, kdim;
  int64_t mn0_, rows;       // tile origin, MN
  __device__ void init(int64_t mn0, int64_t MN) {
    mn0_ = mn0;
    rows = MN;
  }
  __device__ void fetch(int64_t k0, int64_t kend, float4 (&r)[Base::kN]) const {
#pragma unroll
    for (int j = 0; j < Base::kN; ++j) {
      const int64_t k = k0 + Base::krow(j);
      float v[4];
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        const int64_t i = mn0_ + Base::moff(j) + e;
        v[e] = *(k < kend ? p + k * ld + (i < rows ? i : 0) : g_zero);
      }
      r[j] = make_float4(v[0], v[1], v[2], v[3]);
    }
  }
};

// Loader modes of the convolution views.  Row-of-k views: TAP when the
// reduced channel count is a multiple of 32 (a K tile lies inside one filter
// tap, uniform over the workgroup), VEC4 when it is a multiple of 4 (each lane
// splits its own k index, four consecutive channels per load), VEC1 (one load
// per value) otherwise.  Row-of-m views: VEC4 when each float4 lies in one tap,
// VEC1 otherwise.  These take byte offsets from the first image row that the
// tile can touch; the launchers check that they fit (window_fits).  SCALAR, a
// 64-bit address per value, is for images too large for that and, among the
// gradient taps, for channel counts that are not multiples of 4.  7 x 7 stride 2
// on 64 x 224 x 224 x 3, 64-bit addresses and VEC1: forward 208 and 175 us,
// filter gradient 240 and 221.
enum { SCALAR = 0, VEC4 = 1, TAP = 2, VEC1 = 3 };

__device__ inline int clampi(int v, int lo, int hi) { return min(max(v, lo), hi); }

// Convolution forward, A = input patches: A[m = (n, p, q)][kk = (r, s, c)] =
// X[n][p st - pad + r][q st - pad + s][c]   (row-of-k)
template <int E, int MODE>
struct ConvPatch : RowK<E> {
  using Base = RowK<E>;
  static constexpr bool kPixels = true;
  const float* x;
  int H, W, C, S, st, pad;
  FastDiv dQ, dPQ, dC, dS, dSC;   // by Q, P Q, C, S, S C
  int64_t far_[MODE == SCALAR ? Base::kN : 1];   // offset of X[n][h0][w0][0]
  int base_[MODE == SCALAR ? 1 : Base::kN];      // the same from the tile's first image row, bytes
  int h_[Base::kN], w_[Base::kN];                // h0 = p st - pad, w0 = q st - pad
  __device__ void split(int m, int& n, int& p, int& q) const {
    n = dPQ.div(m);
    const int rem = m - n * (int)dPQ.d;
    p = dQ.div(rem);
    q = rem - p * (int)dQ.d;
  }
  __device__ void init(int64_t mn0, int64_t M) {
    int n0 = 0, hb = 0;
    if constexpr (MODE != SCALAR) {
      int p0, q0;
      split((int)mn0, n0, p0, q0);
      hb = clampi(p0 * st - pad, 0, H - 1);
      x += ((int64_t)n0 * H + hb) * W * C;
    }
#pragma unroll
    for (int j = 0; j < Base::kN; ++j) {
      const int64_t m = mn0 + Base::row(j);
      int n = 0, p = 0, q = 0;
      if (m < M) split((int)m, n, p, q);
      h_[j] = m < M ? p * st - pad : kFar;
      w_[j] = q * st - pad;
      if constexpr (MODE == SCALAR)
        far_[j] = m < M ? (((int64_t)n * H + h_[j]) * W + w_[j]) * C : 0;
      else
        base_[j] = m < M ? (((n - n0) * H + h_[j] - hb) * W + w_[j]) * C * 4 : 0;
    }
  }
  // value at (row j, column kk) or 0 when kk >= kend or outside the image
  __device__ float at(int j, int kk, int64_t kend) const {
    const bool kin = kk < kend;
    const int kc = kin ? kk : 0;
    const int r = dSC.div(kc);
    const int rem = kc - r * (int)dSC.d;
    const int s = dC.div(rem), c = rem - s * C;
    const bool ok = kin & inside(h_[j] + r, H) & inside(w_[j] + s, W);
    return *(ok ? x + far_[j] + ((int64_t)r * W + s) * C + c : g_zero);
  }
  __device__ void fetch(int64_t k0, int64_t kend, float4 (&r)[Base::kN]) const {
    const int kk = (int)k0 + Base::koff();
    if constexpr (MODE == SCALAR) {
#pragma unroll
      for (int j = 0; j < Base::kN; ++j)
        r[j] = make_float4(at(j, kk, kend), at(j, kk + 1, kend), at(j, kk + 2, kend),
                           at(j, kk + 3, kend));
    } else if constexpr (MODE == VEC1) {
      const auto b = buffer(x, k0 < kend ? int64_t(1) << 29 : 0);
      float v[Base::kN][4];
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        const int rr = dSC.div(kk + e);
        const int rem = kk + e - rr * (int)dSC.d;
        const int s = dC.div(rem);
        const int toff = ((rr * W + s) * C + rem - s * C) * 4;
#pragma unroll
        for (int j = 0; j < Base::kN; ++j) {
          const bool ok = (kk + e < kend) & inside(h_[j] + rr, H) & inside(w_[j] + s, W);
          v[j][e] = ldb1(b, ok ? (uint32_t)(base_[j] + toff) : kNone);
        }
      }
#pragma unroll
      for (int j = 0; j < Base::kN; ++j) r[j] = make_float4(v[j][0], v[j][1], v[j][2], v[j][3]);
    } else {
      int rr, s, c;
      bool kin = true;
      if constexpr (MODE == TAP) {   // uniform tap
        const int tap = dC.div((int)k0);
        rr = dS.div(tap);
        s = tap - rr * S;
        c = (int)k0 - tap * C + Base::koff();
      } else {
        rr = dSC.div(kk);
        const int rem = kk - rr * (int)dSC.d;
        s = dC.div(rem);
        c = rem - s * C;
        kin = kk < kend;
      }
      const int toff = ((rr * W + s) * C + c) * 4;
      const auto b = buffer(x, k0 < kend ? int64_t(1) << 29 : 0);
#pragma unroll
      for (int j = 0; j < Base::kN; ++j) {
        const bool ok = kin & inside(h_[j] + rr, H) & inside(w_[j] + s, W);
        r[j] = ldb(b, ok ? (uint32_t)(base_[j] + toff) : kNone);
      }
    }
  }
};

// Convolution input gradient for the input pixels of one stride class,
// h = st hh + ph and w = st ww + pw (hh < Hc, ww < Wc).  Only the taps
// r = r0 + st i (i < nR) and s = s0 + st j (j < nS) reach them, from the
// output position p = hh + a - i, q = ww + b - j (a = (ph + pad - r0) / st,
// b = (pw + pad - s0) / st); A is the output gradient gathered that way:
// A[m = (n, hh, ww)][kk = (i, j, k)] = dY[n][hh + a - i][ww + b - j][k], zero
// outside the output.  Stride 1 is the single class r0 = s0 = 0, a = b = pad.
// Row-of-k; the mode refers to the output channels K.
template <int E, int MODE>
struct ConvGradTap : RowK<E> {
  using Base = RowK<E>;
  static constexpr bool kPixels = true;
  const float* dy;
  int P, Q, K, nR, nS, a, b;
  FastDiv dWc, dHWc, dK, dnS, dSK;   // by Wc, Hc Wc, K, nS, nS K
  int64_t far_[MODE == SCALAR ? Base::kN : 1];   // offset of dY[n][hh + a][ww + b][0]
  int base_[MODE == SCALAR ? 1 : Base::kN];      // from the tile's first row of dY, bytes
  int p_[Base::kN], q_[Base::kN];                // hh + a, ww + b
  __device__ void split(int m, int& n, int& hh, int& ww) const {
    n = dHWc.div(m);
    const int rem = m - n * (int)dHWc.d;
    hh = dWc.div(rem);
    ww = rem - hh * (int)dWc.d;
  }
  __device__ void init(int64_t mn0, int64_t M) {
    int n0 = 0, pb = 0;
    if constexpr (MODE != SCALAR) {
      int h0, w0;
      split((int)mn0, n0, h0, w0);
      pb = clampi(h0 + a - (nR - 1), 0, P - 1);
      dy += ((int64_t)n0 * P + pb) * Q * K;
    }
#pragma unroll
    for (int j = 0; j < Base::kN; ++j) {
      const int64_t m = mn0 + Base::row(j);
      int n = 0, hh = 0, ww = 0;
      if (m < M) split((int)m, n, hh, ww);
      p_[j] = m < M ? hh + a : kFar;
      q_[j] = ww + b;
      if constexpr (MODE == SCALAR)
        far_[j] = m < M ? (((int64_t)n * P + p_[j]) * Q + q_[j]) * K : 0;
      else
        base_[j] = m < M ? (((n - n0) * P + p_[j] - pb) * Q + q_[j]) * K * 4 : 0;
    }
  }
  __device__ float at(int j, int kk, int64_t kend) const {
    const bool kin = kk < kend;
    const int kc = kin ? kk : 0;
    const int i = dSK.div(kc);
    const int rem = kc - i * (int)dSK.d;
    const int jj = dK.div(rem), k = rem - jj * K;
    const bool ok = kin & inside(p_[j] - i, P) & inside(q_[j] - jj, Q);
    return *(ok ? dy + far_[j] - ((int64_t)i * Q + jj) * K + k : g_zero);
  }
  __device__ void fetch(int64_t k0, int64_t kend, float4 (&r)[Base::kN]) const {
    const int kk = (int)k0 + Base::koff();
    if constexpr (MODE == SCALAR) {
#pragma unroll
      for (int j = 0; j < Base::kN; ++j)
        r[j] = make_float4(at(j, kk, kend), at(j, kk + 1, kend), at(j, kk + 2, kend),
                           at(j, kk + 3, kend));
    } else {
      int i, jj, k;
      bool kin = true;
      if constexpr (MODE == TAP) {   // uniform tap
        const int tap = dK.div((int)k0);
        i = dnS.div(tap);
        jj = tap - i * nS;
        k = (int)k0 - tap * K + Base::koff();
      } else {
        i = dSK.div(kk);
        const int rem = kk - i * (int)dSK.d;
        jj = dK.div(rem);
        k = rem - jj * K;
        kin = kk < kend;
      }
      const int toff = (k - (i * Q + jj) * K) * 4;
      const auto bf = buffer(dy, k0 < kend ? int64_t(1) << 29 : 0);
#pragma unroll
      for (int j = 0; j < Base::kN; ++j) {
        const bool ok = kin & inside(p_[j] - i, P) & inside(q_[j] - jj, Q);
        r[j] = ldb(bf, ok ? (uint32_t)(base_[j] + toff) : kNone);
      }
    }
  }
};

// Convolution input gradient, B = filter at the class's taps:
// B[kk = (i, j, k)][c] = W[k][r0 + st i][s0 + st j][c]   (row-of-m; C % 4 == 0)
template <int E, int MODE>
struct ConvFilterTap : RowM<E> {
  using Base = RowM<E>;
  const float* w;
  int C, K, S, st, r0, s0, nS;
  int64_t RSC;
  FastDiv dK, dnS, dSK;
  int c0;                     // the tile's first channel
  uint32_t off_[MODE == TAP ? Base::kN : 1];   // bytes from the K tile's first filter row
  __device__ void init(int64_t mn0, int64_t) {
    c0 = (int)mn0;
    if constexpr (MODE == TAP) {
#pragma unroll
      for (int j = 0; j < Base::kN; ++j)
        off_[j] = (uint32_t)((Base::krow(j) * RSC + Base::moff(j)) * 4);
    }
  }
  __device__ void fetch(int64_t k0, int64_t kend, float4 (&r)[Base::kN]) const {
    if constexpr (MODE == TAP) {   // uniform tap
      const int tap = dK.div((int)k0);
      const int i = dnS.div(tap), jj = tap - i * nS;
      const int64_t at = ((int64_t)k0 - (int64_t)tap * K) * RSC +
                         ((int64_t)(r0 + st * i) * S + s0 + st * jj) * C + c0;
      const auto b = buffer(w + at, k0 < kend ? K * RSC - at : 0);
#pragma unroll
      for (int j = 0; j < Base::kN; ++j) r[j] = ldb(b, off_[j]);
    } else {
      const int cc = c0 + Base::moff() < C ? c0 + Base::moff() : 0;   // clamped to the filter
#pragma unroll
      for (int j = 0; j < Base::kN; ++j) {
        const int kk = (int)k0 + Base::krow(j);
        const bool ok = kk < kend;
        const int kc = ok ? kk : 0;
        const int i = dSK.div(kc);
        const int rem = kc - i * (int)dSK.d;
        const int jj = dK.div(rem), k = rem - jj * K;
        int64_t off = (int64_t)k * RSC + ((int64_t)(r0 + st * i) * S + s0 + st * jj) * C + cc;
        keep(off);
        r[j] = ld4(ok ? w + off : g_zero);
      }
    }
  }
};

// Convolution filter gradient, B = input patches along the pixel axis:
// B[kk = (n, p, q)][col = (r, s, c)] = X[n][p st - pad + r][q st - pad + s][c]
// (row-of-m).  A lane's columns are clamped to the matrix, then split into
// taps at set-up: one per float4 (VEC4) or one per value.  A lane's
// kR pixels are consecutive: the first one's position is split from its index,
// the others step from it.
template <int E, int MODE>
struct ConvPixelPatch : RowM<E> {
  using Base = RowM<E>;
  static constexpr bool kPixels = true;
  using Off = std::conditional_t<MODE == SCALAR, int64_t, int>;
  static constexpr int kPer = MODE == VEC4 ? 1 : 4;   // taps per float4
  static constexpr int kT = kPer * Base::kItems;
  const float* x;
  int H, W, C, st, pad;
  int h_end, w_end;       // P st - pad, Q st - pad
  int64_t row_step;       // from the pixel after a row's last one to the next row's first
  int64_t img_step;       // from the row after an image's last one to the next image's first
  FastDiv dQ, dPQ, dC, dSC;
  int toff_[kT];          // (r W + s) C + c of each tap entry
  int r_[kT], s_[kT];
  __device__ void init(int64_t mn0, int64_t RSC) {
#pragma unroll
    for (int e = 0; e < kT; ++e) {
      const int col = (int)mn0 + Base::moff(e / kPer * Base::kR) + e % kPer;
      const int cc = col < RSC ? col : 0;
      const int r = dSC.div(cc);
      const int rem = cc - r * (int)dSC.d;
      const int s = dC.div(rem), c = rem - s * C;
      r_[e] = r;
      s_[e] = s;
      toff_[e] = (r * W + s) * C + c;
    }
  }
  __device__ void split(int m, int& n, int& p, int& q) const {
    n = dPQ.div(m);
    const int rem = m - n * (int)dPQ.d;
    p = dQ.div(rem);
    q = rem - p * (int)dQ.d;
  }
  __device__ void fetch(int64_t k0, int64_t kend, float4 (&r)[Base::kN]) const {
    int n0 = 0, hb0 = 0;      // the image row that 32-bit offsets count from
    if constexpr (MODE != SCALAR) {
      int p0, q0;
      split(k0 < kend ? (int)k0 : 0, n0, p0, q0);
      hb0 = clampi(p0 * st - pad, 0, H - 1);
    }
    const auto b = buffer(x + ((int64_t)n0 * H + hb0) * W * C, k0 < kend ? int64_t(1) << 29 : 0);
#pragma unroll
    for (int i = 0; i < Base::kItems; ++i) {
      const int kk = (int)k0 + Base::krow(i * Base::kR);
      int n, p, q;
      split(kk < kend ? kk : 0, n, p, q);
      int hb = p * st - pad, wb = q * st - pad;
      Off po = (((Off)(n - n0) * H + hb - hb0) * W + wb) * C;
#pragma unroll
      for (int j = 0; j < Base::kR; ++j) {
        keep(po);
        const bool kin = kk + j < kend;
        if constexpr (MODE == VEC4) {
          const bool ok = kin & inside(hb + r_[i], H) & inside(wb + s_[i], W);
          r[i * Base::kR + j] = ldb(b, ok ? (uint32_t)(po + toff_[i]) * 4u : kNone);
        } else {
          float v[4];
#pragma unroll
          for (int e = 0; e < 4; ++e) {
            const int u = 4 * i + e;
            const bool ok = kin & inside(hb + r_[u], H) & inside(wb + s_[u], W);
            if constexpr (MODE == VEC1)
              v[e] = ldb1(b, ok ? (uint32_t)(po + toff_[u]) * 4u : kNone);
            else
              v[e] = *(ok ? x + po + toff_[u] : g_zero);
          }
          r[i * Base::kR + j] = make_float4(v[0], v[1], v[2], v[3]);
        }
        if (j + 1 < Base::kR) {
          wb += st;
          const bool row_done = wb >= w_end;
          hb += row_done ? st : 0;
          const bool img_done = hb >= h_end;
          po += st * C + (row_done ? (Off)row_step : 0) + (img_done ? (Off)img_step : 0);
          wb = row_done ? -pad : wb;
          hb = img_done ? -pad : hb;
        }
      }
    }
  }
};

// Where row m of C goes: m * ldc, or the NHWC input pixel of a stride class
struct DenseOut {
  int64_t ldc;
  __device__ int64_t row(int64_t m) const { return m * ldc; }
};
struct ClassOut {
  int H, W, C, st, ph, pw;
  FastDiv dWc, dHWc;
  __device__ int64_t row(int64_t m) const {
    const int n = dHWc.div((int)m);
    const int rem = (int)m - n * (int)dHWc.d;
    const int hh = dWc.div(rem), ww = rem - hh * (int)dWc.d;
    return (((int64_t)n * H + st * hh + ph) * W + st * ww + pw) * C;
  }
};

// ---------------------------------------------------------------- kernel
template <class L>
__device__ inline float4 read_op(const float* lds, int i, int k) {
  if (L::kRowOfK) return *reinterpret_cast<const float4*>(&lds[rowk_index(i, k)]);
  constexpr int ld = L::kLds / BK;
  return make_float4(lds[(k + 0) * ld + i], lds[(k + 1) * ld + i], lds[(k + 2) * ld + i],
                     lds[(k + 3) * ld + i]);
}

// Batched problems (grid z): batch z = (zo, zi) with zi = z mod inner; operand
// and result pointers move by zo * outer stride + zi * inner stride.  causal:
// see BatchStrides.
struct Batch {
  int64_t inner;
  int64_t a_o, a_i, b_o, b_i, c_o, c_i;
  int64_t causal;
};

template <class L>
__device__ inline void shift(L& l, int64_t d) {
  l.p += d;
}

// The wave grid of a BM x BN tile: the four waves form WM x WN, 4 x 1 for
// 32-wide and 256 x 64 tiles, 1 x 4 for 32-tall ones, else 2 x 2; each wave
// owns MB x NB MFMA 32 x 32 blocks.
template <int BM, int BN>
struct WaveGrid {
  static constexpr int WM = (BN == 32 || (BM == 256 && BN == 64)) ? 4 : BM == 32 ? 1 : 2;
  static constexpr int WN = 4 / WM;
  static constexpr int MB = BM / (32 * WM), NB = BN / (32 * WN);
  static_assert(MB >= 1 && NB >= 1 && MB * 32 * WM == BM && NB * 32 * WN == BN, "tile shape");
  // waves per SIMD, the compiler's register budget: 3, or what the LDS tile (192 bytes a row)
  // or two accumulators for three or more blocks leave room for
  static constexpr int kWaves =
      MB * NB >= 3 ? 2 : std::min(3, 160 * 1024 / ((BM + BN) * 192 + 256));
};

// One K tile of split operands into the accumulators: two k steps of 16, each
// six products of pieces.  m l, l m and l l are left out: together at most 2^-24
// of x y (|m| <= 2^-8, |l| <= 2^-17 of the operand's power of two), 5.6e-9 in the
// root mean square, or 2^-22 and 2.3e-8 where one operand's h is narrow.  h h
// goes to acc, the five smaller products to low: next to an accumulator that one
// large term has raised, the matrix instruction drops the last bits of every
// small term, always the same ones for operands that repeat.  In one accumulator,
// column sums of (softmax - onehot) W came out
// 1.8e-6 off instead of 5.6e-7.
template <class LA, class LB, int MB, int NB>
__device__ __forceinline__ void mma_split(floatx16 (&acc)[MB][NB], floatx16 (&low)[MB][NB],
                                          const char* A, const char* B, const int (&aoff)[MB],
                                          const int (&boff)[NB]) {
  auto read = [&](bf16x8(&x)[MB], int p, int ks) {
#pragma unroll
    for (int mb = 0; mb < MB; ++mb)
      x[mb] = *reinterpret_cast<const bf16x8*>(A + p * LA::kPiece + (aoff[mb] ^ (ks << 5)));
  };
  auto readb = [&](bf16x8(&x)[NB], int p, int ks) {
#pragma unroll
    for (int nb = 0; nb < NB; ++nb)
      x[nb] = *reinterpret_cast<const bf16x8*>(B + p * LB::kPiece + (boff[nb] ^ (ks << 5)));
  };
  auto mma = [&](floatx16(&c)[MB][NB], const bf16x8(&x)[MB], const bf16x8(&y)[NB]) {
#pragma unroll
    for (int mb = 0; mb < MB; ++mb)
#pragma unroll
      for (int nb = 0; nb < NB; ++nb)
        c[mb][nb] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(x[mb], y[nb], c[mb][nb], 0, 0, 0);
  };
#pragma unroll
  for (int ks = 0; ks < 2; ++ks) {
    bf16x8 ah[MB], al[MB], am[MB], bh[NB], bl[NB], bm[NB];
    read(ah, 0, ks);
    readb(bl, 2, ks);
    read(al, 2, ks);
    readb(bh, 0, ks);
    mma(low, ah, bl);
    mma(low, al, bh);
    read(am, 1, ks);
    readb(bm, 1, ks);
    mma(acc, ah, bh);
    mma(low, am, bm);
    mma(low, am, bh);
    mma(low, ah, bm);
  }
}

// One fp32 K tile from LDS into the accumulators: STEPS k steps of 4 per
// half-wave (the lower half's are k = 0 .. 4 STEPS - 1), each a round of LDS
// reads feeding MB x NB x 4 MFMAs.
template <int BM, int BN, class LA, class LB, int STEPS, int MB, int NB>
__device__ __forceinline__ void mma_ktile(floatx16 (&acc)[MB][NB], const float* A, const float* B,
                                          int wm, int wn, int half, int li) {
  using G = WaveGrid<BM, BN>;
#pragma unroll
  for (int j = 0; j < STEPS; ++j) {
    const int kq = half * 16 + 4 * j;
    float4 a[G::MB], b[G::NB];
#pragma unroll
    for (int mb = 0; mb < G::MB; ++mb) a[mb] = read_op<LA>(A, wm * (BM / G::WM) + mb * 32 + li, kq);
#pragma unroll
    for (int nb = 0; nb < G::NB; ++nb) b[nb] = read_op<LB>(B, wn * (BN / G::WN) + nb * 32 + li, kq);
#pragma unroll
    for (int s = 0; s < 4; ++s)
#pragma unroll
      for (int mb = 0; mb < G::MB; ++mb)
#pragma unroll
        for (int nb = 0; nb < G::NB; ++nb)
          acc[mb][nb] = __builtin_amdgcn_mfma_f32_32x32x2f32(comp(a[mb], s), comp(b[nb], s),
                                                            acc[mb][nb], 0, 0, 0);
  }
}

// The accumulators (times even for the tile's even rows, odd for the others) of the tile at
// (m0, n0) into C, plus the column's bias.
template <int BM, int BN, class OM, bool BIAS, int MB, int NB>
__device__ __forceinline__ void store_tile(const floatx16 (&acc)[MB][NB], float even, float odd,
                                           float* out, const OM& om, const float* bias, int64_t m0, int64_t n0,
                                           int64_t M, int64_t N, int wm, int wn, int half, int li) {
  using G = WaveGrid<BM, BN>;
#pragma unroll
  for (int mb = 0; mb < G::MB; ++mb)
#pragma unroll
    for (int nb = 0; nb < G::NB; ++nb) {
      const int64_t col = n0 + wn * (BN / G::WN) + nb * 32 + li;
      if (col >= N) continue;
      const float bv = BIAS ? bias[col] : 0.f;
#pragma unroll
      for (int r = 0; r < 16; ++r) {
        const int64_t row = m0 + wm * (BM / G::WM) + mb * 32 + 8 * (r >> 2) + 4 * half + (r & 3);
        if (row < M) out[om.row(row) + col] = acc[mb][nb][r] * (r & 1 ? odd : even) + bv;
      }
    }
}

template <int MB, int NB>
__device__ __forceinline__ void clear(floatx16 (&acc)[MB][NB]) {
#pragma unroll
  for (int a = 0; a < MB; ++a)
#pragma unroll
    for (int b = 0; b < NB; ++b)
#pragma unroll
      for (int r = 0; r < 16; ++r) acc[a][b][r] = 0.f;
}

// ROWSUM: rowsum[slice][m] = sum over this slice's k of A[m][k].  FEW: K <= kFewTerms, fp32
// products only.
template <int BM, int BN, class LA, class LB, class OM, bool BIAS, bool BATCHED, bool ROWSUM,
          bool FEW>
__global__ __launch_bounds__(THREADS, (WaveGrid<BM, BN>::kWaves)) void gemm_kernel(
    LA la, LB lb, float* __restrict__ c, OM om, int64_t slice_stride,
    const float* __restrict__ bias, int64_t M, int64_t N, int64_t K, int64_t k_slice, int tiles_m,
    int tiles_n, Batch bt, float* __restrict__ rowsum) {
  using G = WaveGrid<BM, BN>;
  constexpr int MB = G::MB, NB = G::NB;
  constexpr bool kNarrow = LA::kPixels || LB::kPixels;
  constexpr bool kNarrowA = kNarrow && LA::kN < LB::kN;   // the side with fewer values to split
  // Workgroup (tile, slice, batch) from an XCD-aware order: the hardware hands
  // linear workgroup h to XCD h mod 8, so logical ids are laid out so that each
  // XCD (with its own L2) gets one contiguous run of them, and neighbouring
  // tiles, which share operand rows, share an L2.
  const uint32_t gx = gridDim.x, gy = gridDim.y;
  const uint32_t total = gx * gy * gridDim.z;
  const uint32_t h = blockIdx.x + gx * (blockIdx.y + gy * blockIdx.z);
  const uint32_t q = total / kXcds, rem = total % kXcds, xcd = h % kXcds, local = h / kXcds;
  const uint32_t L = xcd < rem ? xcd * (q + 1) + local : rem * (q + 1) + (xcd - rem) * q + local;
  const int t = (int)(L % gx);
  const int64_t slice = (L / gx) % gy;
  if constexpr (BATCHED) {
    const int64_t z = L / (gx * gy), zo = z / bt.inner, zi = z % bt.inner;
    shift(la, zo * bt.a_o + zi * bt.a_i);
    shift(lb, zo * bt.b_o + zi * bt.b_i);
    c += zo * bt.c_o + zi * bt.c_i;
  }
  __shared__ __attribute__((aligned(16))) char lds[kPieces * (LA::kPiece + LB::kPiece)];
  char* const As = lds;
  char* const Bs = lds + kPieces * LA::kPiece;

  // grouped tile order: 8 tile-rows share their B tiles in L2
  const int group = 8;
  const int per_group = group * tiles_n;
  const int g = t / per_group;
  const int first_m = g * group;
  const int gsize = min(tiles_m - first_m, group);
  const int tm = first_m + (t % per_group) % gsize;
  const int tn = (t % per_group) / gsize;
  const int64_t m0 = (int64_t)tm * BM, n0 = (int64_t)tn * BN;
  int64_t kb = slice * k_slice;
  int64_t ke = min(K, kb + k_slice);
  if constexpr (BATCHED) {
    // the whole workgroup leaves together
    if (bt.causal == BatchStrides::kUpperC && n0 >= m0 + BM) return;
    if (bt.causal == BatchStrides::kLowerA) ke = min(ke, m0 + BM);
    if (bt.causal == BatchStrides::kLowerAT) kb = max(kb, m0);
  }

  la.init(m0, M);
  lb.init(n0, N);
  float4 ra[LA::kN], rb[LB::kN];
  floatx16 acc[MB][NB], low[MB][NB];
  clear(acc);
  clear(low);

  const bool sums = ROWSUM && tn == 0;
  float4 rs = zero4();

  const int lane = threadIdx.x & 63;
  const int wave = threadIdx.x >> 6;
  const int wm = wave % G::WM, wn = wave / G::WM;
  const int half = lane >> 5;
  const int li = lane & 31;
  int aoff[MB], boff[NB];
#pragma unroll
  for (int mb = 0; mb < MB; ++mb) aoff[mb] = LA::octet(wm * (BM / G::WM) + mb * 32 + li, half);
#pragma unroll
  for (int nb = 0; nb < NB; ++nb) boff[nb] = LB::octet(wn * (BN / G::WN) + nb * 32 + li, half);

  la.fetch(kb, ke, ra);
  lb.fetch(kb, ke, rb);
  if constexpr (FEW) {
    float* const Af = reinterpret_cast<float*>(lds);
    float* const Bf = Af + LA::kLds;
    LA::store(Af, ra);
    LB::store(Bf, rb);
    if constexpr (ROWSUM) {
      if (sums) {
#pragma unroll
        for (int j = 0; j < LA::kN; ++j) {
          rs.x += ra[j].x;
          rs.y += ra[j].y;
          rs.z += ra[j].z;
          rs.w += ra[j].w;
        }
      }
    }
    __syncthreads();
    mma_ktile<BM, BN, LA, LB, (kFewTerms + 3) / 4>(acc, Af, Bf, wm, wn, half, li);
    __syncthreads();
  }
  for (int64_t k0 = FEW ? ke : kb; k0 < ke; k0 += BK) {
    __syncthreads();   // every wave has read the previous tile
    LA::template split_store<kNarrowA>(As, ra);
    LB::template split_store<kNarrow && !kNarrowA>(Bs, rb);
    if constexpr (ROWSUM) {
      if (sums) {
#pragma unroll
        for (int j = 0; j < LA::kN; ++j) {
          rs.x += ra[j].x;
          rs.y += ra[j].y;
          rs.z += ra[j].z;
          rs.w += ra[j].w;
        }
      }
    }
    __syncthreads();
    // in flight while this tile is multiplied; past the last tile, the loads
    // read zeros without touching memory
    la.fetch(k0 + BK, ke, ra);
    lb.fetch(k0 + BK, ke, rb);
    __builtin_amdgcn_sched_barrier(0);
    mma_split<LA, LB>(acc, low, As, Bs, aoff, boff);
  }

  // A value of 2^87 or more, an infinity, a NaN or a sum of 2^48 or more leaves an accumulator
  // that is not finite: such a tile is computed again by fp32 products.
  float check = 0.f;
#pragma unroll
  for (int a = 0; a < MB; ++a)
#pragma unroll
    for (int b = 0; b < NB; ++b)
#pragma unroll
      for (int r = 0; r < 16; ++r) {
        acc[a][b][r] += low[a][b][r];
        check = fmaf(acc[a][b][r], 0.f, check);
      }
  float even = li & 1 ? -kSplitUnscale : kSplitUnscale, odd = -even;
  if constexpr (FEW) even = odd = 1.f;
  if (!FEW && __syncthreads_or(check != 0.f)) {
    even = odd = 1.f;
    clear(acc);
    float* const Af = reinterpret_cast<float*>(lds);
    float* const Bf = Af + LA::kLds;
    for (int64_t k0 = kb; k0 < ke; k0 += BK) {
      la.fetch(k0, ke, ra);
      lb.fetch(k0, ke, rb);
      LA::store(Af, ra);
      LB::store(Bf, rb);
      __syncthreads();
      mma_ktile<BM, BN, LA, LB, 4>(acc, Af, Bf, wm, wn, half, li);
      __syncthreads();
    }
  }
  if constexpr (ROWSUM) {
    if (sums) {   // uniform over the workgroup; every wave is past its reads of the tiles
      float* red = reinterpret_cast<float*>(lds);   // [k group][BM]
      constexpr int kGroups = THREADS / (BM / 4);
      *reinterpret_cast<float4*>(&red[threadIdx.x / (BM / 4) * BM + LA::moff()]) = rs;
      __syncthreads();
      if ((int)threadIdx.x < BM && m0 + threadIdx.x < M) {
        float v = 0.f;
#pragma unroll
        for (int j = 0; j < kGroups; ++j) v += red[j * BM + threadIdx.x];
        rowsum[slice * M + m0 + threadIdx.x] = v;
      }
    }
  }
  store_tile<BM, BN, OM, BIAS>(acc, even, odd, c + slice * slice_stride, om, bias, m0, n0, M, N, wm,
                               wn, half, li);
}

// Tiles of a launch: a grid's threads along x are counted in 32 bits, and a launch of more runs
// the remainder without an error.
constexpr int64_t kMaxTiles = (int64_t(1) << 32) / THREADS - 1;

template <int BM, int BN, class LA, class LB, class OM, bool BIAS, bool BATCHED = false,
          bool ROWSUM = false, bool FEW = false>
hipError_t run_gemm(const LA& la, const LB& lb, float* c, OM om, int64_t slice_stride,
                    const float* bias, int64_t M, int64_t N, int64_t K, int64_t slices,
                    hipStream_t s, int64_t batches = 1, Batch bt = Batch{1, 0, 0, 0, 0, 0, 0, 0},
                    float* rowsum = nullptr) {
  const int64_t tiles_m = (M + BM - 1) / BM, tiles_n = (N + BN - 1) / BN;
  if (tiles_m * tiles_n > kMaxTiles || slices > 65535 || batches > 65535 || batches < 1 ||
      tiles_m * tiles_n * slices * batches > INT32_MAX)
    return hipErrorInvalidValue;
  int64_t k_slice = (K + slices - 1) / slices;
  k_slice = (k_slice + BK - 1) / BK * BK;
  if (ROWSUM != (rowsum != nullptr) || (FEW && K > kFewTerms)) return hipErrorInvalidValue;
  dim3 grid((unsigned)(tiles_m * tiles_n), (unsigned)slices, (unsigned)batches);
  hipLaunchKernelGGL((gemm_kernel<BM, BN, LA, LB, OM, BIAS, BATCHED, ROWSUM, FEW>), grid, dim3(THREADS), 0, s,
                     la, lb, c, om, slice_stride, bias, M, N, K, k_slice, (int)tiles_m,
                     (int)tiles_n, bt, rowsum);
  return hipGetLastError();
}

// Tile shape of a product with `copies` batches or slices: the one of least
// modelled time.  A CU takes k = ceil(tiles / CUs) tiles, up to `resident` of
// them side by side (LDS and registers bound it); n side by side run at rate[n]
// of what two 128 x 128 tiles reach together, so smaller tiles only pay where
// the large ones leave CUs idle or alone.  Rates measured on convolutions and
// dense products from 32 x 256 x 256 to 12288 x 4096 x 1024, each run with
// every shape.  Of 25 such products the rule's shape is within 2 % of the best
// in 23 (56 x 56 1 x 1 256 -> 128 at batch 64: 117 us on 64 x 64 tiles, 107 on
// 128 x 64); us with 128 x 128, 128 x 64 and 64 x 64 tiles:
//   256 x 1024 x 1024     66   45   30      12288 x 1024 x 4096  676  746  806
//   1379 x 765 x 3067     78   69   64      7 x 7 3 x 3 512, batch 64  264  188  167
//   8192 x 512 x 1536    101  100  102      28 x 28 3 x 3 128, batch 64  112  137  133
enum Shape { S128x128, S128x64, S64x128, S256x64, S64x64 };
struct ShapeRate {
  int bm, bn, resident;
  double rate[6];   // [n - 1], n tiles side by side
};
constexpr ShapeRate kShapes[] = {
    {128, 128, 2, {0.72, 1.0}},
    {128, 64, 3, {0.52, 0.74, 0.84}},
    {64, 128, 3, {0.51, 0.73, 0.83}},
    {256, 64, 2, {0.66, 0.92}},
    {64, 64, 5, {0.36, 0.54, 0.60, 0.63, 0.78}},
};
double shape_time(const ShapeRate& r, int64_t M, int64_t N, int64_t copies) {
  constexpr int64_t kCUs = 256;
  const int64_t tiles = ((M + r.bm - 1) / r.bm) * ((N + r.bn - 1) / r.bn) * copies;
  const int64_t k = (tiles + kCUs - 1) / kCUs, rem = k % r.resident;
  return r.bm * r.bn * ((k - rem) / r.rate[r.resident - 1] + (rem ? rem / r.rate[rem - 1] : 0.0));
}
// K is the reduction of one copy.  256 x 64 tiles are for at most 64 columns
// and long reductions (64-channel 3 x 3 convolutions: 6 % faster than 128 x 64
// at K = 576, 10 % slower at K = 256).
Shape pick_shape(int64_t M, int64_t N, int64_t K, int64_t copies) {
  int best = S128x128;
  for (int i = S128x64; i <= S64x64; ++i) {
    if (i == S256x64 && (N > 64 || K < 512)) continue;
    if (shape_time(kShapes[i], M, N, copies) < shape_time(kShapes[best], M, N, copies)) best = i;
  }
  return (Shape)best;
}

// Runs the GEMM with loader templates A<E>, B<E> instantiated for the chosen
// tile shape; `fa(a)` / `fb(b)` fill them in.  Row m of C starts at om.row(m);
// split-K slices of C are slice_stride floats apart.
template <template <int> class LAT, template <int> class LBT, bool BIAS, bool BATCHED = false,
          bool ROWSUM = false, class FA, class FB, class OM>
hipError_t dispatch(FA fa, FB fb, float* c, OM om, int64_t slice_stride, const float* bias,
                    int64_t M, int64_t N, int64_t K, int64_t slices, hipStream_t s,
                    int64_t batches = 1, Batch bt = Batch{1, 0, 0, 0, 0, 0, 0, 0},
                    float* rowsum = nullptr) {
  if (K <= kFewTerms) {
    LAT<128> a{};
    LBT<64> b{};
    fa(a);
    fb(b);
    return run_gemm<128, 64, LAT<128>, LBT<64>, OM, BIAS, BATCHED, ROWSUM, true>(
        a, b, c, om, slice_stride, bias, M, N, K, slices, s, batches, bt, rowsum);
  }
  switch (pick_shape(M, N, K / slices, slices * batches)) {
    case S256x64:
      if constexpr (!BATCHED) {
        LAT<256> a{};
        LBT<64> b{};
        fa(a);
        fb(b);
        return run_gemm<256, 64, LAT<256>, LBT<64>, OM, BIAS, false, ROWSUM>(
            a, b, c, om, slice_stride, bias, M, N, K, slices, s, 1, bt, rowsum);
      }
      [[fallthrough]];
    case S128x64: {
      LAT<128> a{};
      LBT<64> b{};
      fa(a);
      fb(b);
      return run_gemm<128, 64, LAT<128>, LBT<64>, OM, BIAS, BATCHED, ROWSUM>(
          a, b, c, om, slice_stride, bias, M, N, K, slices, s, batches, bt, rowsum);
    }
    case S64x128: {
      LAT<64> a{};
      LBT<128> b{};
      fa(a);
      fb(b);
      return run_gemm<64, 128, LAT<64>, LBT<128>, OM, BIAS, BATCHED, ROWSUM>(
          a, b, c, om, slice_stride, bias, M, N, K, slices, s, batches, bt, rowsum);
    }
    case S64x64: {
      LAT<64> a{};
      LBT<64> b{};
      fa(a);
      fb(b);
      return run_gemm<64, 64, LAT<64>, LBT<64>, OM, BIAS, BATCHED, ROWSUM>(
          a, b, c, om, slice_stride, bias, M, N, K, slices, s, batches, bt, rowsum);
    }
    default: {
      LAT<128> a{};
      LBT<128> b{};
      fa(a);
      fb(b);
      return run_gemm<128, 128, LAT<128>, LBT<128>, OM, BIAS, BATCHED, ROWSUM>(
          a, b, c, om, slice_stride, bias, M, N, K, slices, s, batches, bt, rowsum);
    }
  }
}

// row-major C with leading dimension ldc
template <template <int> class LAT, template <int> class LBT, bool BIAS, bool BATCHED = false,
          bool ROWSUM = false, class FA, class FB>
hipError_t dispatch_dense(FA fa, FB fb, float* c, int64_t ldc, const float* bias, int64_t M,
                          int64_t N, int64_t K, int64_t slices, hipStream_t s,
                          int64_t batches = 1, Batch bt = Batch{1, 0, 0, 0, 0, 0, 0, 0},
                          float* rowsum = nullptr) {
  return dispatch<LAT, LBT, BIAS, BATCHED, ROWSUM>(fa, fb, c, DenseOut{ldc}, M * ldc, bias, M, N, K,
                                                   slices, s, batches, bt, rowsum);
}

// A product whose rows are those of plain matrices, in launches of as many rows as one takes: at
// most kMaxTiles of the smallest tiles, 64 x 64.  (Convolutions have fewer than 2^31 pixels, and at
// most 64 columns where these fill memory: fewer than 2^24 tiles of 128 x 64.)
template <template <int> class LAT, template <int> class LBT, bool BIAS, class FB>
hipError_t dispatch_rows(const float* A, FB fb, float* c, const float* bias, int64_t M, int64_t N,
                         int64_t K, hipStream_t s) {
  const int64_t cols = (N + 63) / 64;
  // whole tiles of any shape
  const int64_t rows = std::max<int64_t>(1, kMaxTiles / cols / 4) * 256;
  for (int64_t m = 0; m < M; m += rows) {
    const auto fa = [=](auto& l) { l.p = A + m * K; l.ld = K; l.kdim = K; };
    const hipError_t e = dispatch_dense<LAT, LBT, BIAS>(fa, fb, c + m * N, N, bias,
                                                        std::min(rows, M - m), N, K, 1, s);
    if (e != hipSuccess) return e;
  }
  return hipSuccess;
}

// one explicit tile shape, loaders instantiated at its extents (reductions of few terms: dispatch)
template <int BM, int BN, template <int> class LAT, template <int> class LBT, class FA, class FB,
          class OM>
hipError_t dispatch_shape(FA fa, FB fb, float* c, OM om, int64_t slice_stride, int64_t M,
                          int64_t N, int64_t K, int64_t slices, hipStream_t s) {
  if (K <= kFewTerms)
    return dispatch<LAT, LBT, false>(fa, fb, c, om, slice_stride, nullptr, M, N, K, slices, s);
  LAT<BM> a{};
  LBT<BN> b{};
  fa(a);
  fb(b);
  return run_gemm<BM, BN, LAT<BM>, LBT<BN>, OM, false>(a, b, c, om, slice_stride, nullptr, M, N, K,
                                                       slices, s);
}

template <int E> using ConvPatchT = ConvPatch<E, TAP>;
template <int E> using ConvPatchV = ConvPatch<E, VEC4>;
template <int E> using ConvPatch1 = ConvPatch<E, VEC1>;
template <int E> using ConvPatchS = ConvPatch<E, SCALAR>;
template <int E> using ConvGradTapT = ConvGradTap<E, TAP>;
template <int E> using ConvGradTapV = ConvGradTap<E, VEC4>;
template <int E> using ConvGradTapS = ConvGradTap<E, SCALAR>;
template <int E> using ConvFilterTapT = ConvFilterTap<E, TAP>;
template <int E> using ConvFilterTapG = ConvFilterTap<E, VEC4>;
template <int E> using ConvPixelPatchV = ConvPixelPatch<E, VEC4>;
template <int E> using ConvPixelPatch1 = ConvPixelPatch<E, VEC1>;
template <int E> using ConvPixelPatchS = ConvPixelPatch<E, SCALAR>;

// the GEMM sizes of the convolution views index with 32-bit arithmetic
bool fits31(int64_t v) { return v >= 0 && v < (int64_t(1) << 31) - 512; }

// Tile of a filter gradient (M = output channels, N = RSC), first rule that
// applies:
//   32 x 256 for M <= 32 (no empty tile rows; 32 columns of one tap a thread
//            when C % 32 == 0);
//   64 x 192 for M <= 64 when that leaves fewer padded RSC columns than
//            64 x 128 (RSC = 576 for a 3 x 3 x 64 filter: 3 full tiles, not 4.5);
//   otherwise the general shapes.
// Both only for M and C that are multiples of 4, those they were measured with.
enum class WgradTile { k32x256, k64x192, kGeneral };
WgradTile wgrad_tile(int64_t M, int64_t N, int64_t C) {
  if (M % 4 != 0 || C % 4 != 0) return WgradTile::kGeneral;
  if (M <= 32) return WgradTile::k32x256;
  const int64_t pad128 = (N + 127) / 128 * 128 - N, pad192 = (N + 191) / 192 * 192 - N;
  if (M <= 64 && pad192 < pad128) return WgradTile::k64x192;
  return WgradTile::kGeneral;
}

// ---------------------------------------------------------------- small kernels
// out[j] = sum over slices of part[s][j].  A workgroup covers 64 consecutive
// j, one per lane; wave w takes the slices s = w mod 4 in eight interleaved
// chains (s / 4 mod 8), so that each lane has eight loads in flight, and the
// partial sums are added in a fixed order: the result does not depend on
// timing.
constexpr int SUM_J = 64;
__global__ __launch_bounds__(256) void slice_sum_kernel(const float* __restrict__ part,
                                                        float* __restrict__ out, int64_t n,
                                                        int64_t slices) {
  __shared__ float red[4][SUM_J];
  const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
  const int64_t j = (int64_t)blockIdx.x * SUM_J + lane;
  float a[8] = {0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f};
  if (j < n) {
    int64_t s = w;
    for (; s + 28 < slices; s += 32) {
      float v[8];
#pragma unroll
      for (int u = 0; u < 8; ++u) v[u] = part[(s + 4 * u) * n + j];
#pragma unroll
      for (int u = 0; u < 8; ++u) a[u] += v[u];
    }
#pragma unroll
    for (int u = 0; u < 7; ++u)
      if (s + 4 * u < slices) a[u] += part[(s + 4 * u) * n + j];
  }
  red[w][lane] = ((a[0] + a[1]) + (a[2] + a[3])) + ((a[4] + a[5]) + (a[6] + a[7]));
  __syncthreads();
  if (w == 0 && j < n) out[j] = (red[0][lane] + red[1][lane]) + (red[2][lane] + red[3][lane]);
}

hipError_t slice_sum(const float* part, float* out, int64_t n, int64_t slices, hipStream_t s) {
  hipLaunchKernelGGL(slice_sum_kernel, dim3((unsigned)((n + SUM_J - 1) / SUM_J)), dim3(256), 0, s,
                     part, out, n, slices);
  return hipGetLastError();
}

// The input-gradient pixels of a stride class that no filter tap reaches are
// zeros (a 1 x 1 filter with stride 2 reaches one class of four).  Rows
// m0 .. m0 + rows of the class, q = C / 4 float4 each; rows * q < 2^31.
__global__ __launch_bounds__(256) void class_zero_kernel(float* __restrict__ dx, ClassOut om,
                                                         int64_t m0, int rows, int q,
                                                         FastDiv dq) {
  const int n = rows * q;
  for (int i = blockIdx.x * 256 + threadIdx.x; i < n; i += gridDim.x * 256) {
    const int r = dq.div(i);
    *reinterpret_cast<float4*>(dx + om.row(m0 + r) + 4 * (i - r * q)) = make_float4(0, 0, 0, 0);
  }
}

hipError_t class_zero(float* dx, const ClassOut& om, int64_t M, int64_t C, hipStream_t s) {
  const int64_t q = C / 4;
  const int64_t per = std::max<int64_t>(1, (int64_t(1) << 30) / q);   // rows per launch
  for (int64_t m0 = 0; m0 < M; m0 += per) {
    const int64_t rows = std::min(per, M - m0);
    const int64_t blocks = std::min<int64_t>((rows * q + 255) / 256, 16384);
    hipLaunchKernelGGL(class_zero_kernel, dim3((unsigned)blocks), dim3(256), 0, s, dx, om, m0,
                       (int)rows, (int)q, FastDiv::make(q));
    const hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
  }
  return hipSuccess;
}

}  // namespace

// ---------------------------------------------------------------- launchers
namespace {
// Fills a dense view
auto dense(const float* p, int64_t ld, int64_t kdim) {
  return [=](auto& l) { l.p = p; l.ld = ld; l.kdim = kdim; };
}

// Whether the bytes between the first image row and the last that `pixels`
// consecutive pixels of an (N, rows, cols) grid can touch fit a buffer
// descriptor: pixel (h, w) reads rows h st + [-back, taps) of (imgH, imgW, C)
// images.
bool window_fits(int64_t pixels, int64_t rows, int64_t cols, int64_t st, int64_t taps,
                 int64_t imgH, int64_t imgW, int64_t C) {
  const int64_t lines = (pixels + cols - 1) / cols + 1;          // grid rows touched
  const int64_t images = (lines + rows - 1) / rows + 1;          // images touched
  const int64_t skip = std::max<int64_t>(0, imgH - (rows - 1) * st);   // at each change of image
  const int64_t span = std::min(images * imgH, lines * st + taps + images * (skip + taps));
  return span < (int64_t(1) << 29) / C / imgW;
}
}  // namespace

hipError_t linear_fwd(const float* X, const float* W, const float* b, float* Y, int64_t M,
                      int64_t K, int64_t N, hipStream_t s) {
  const auto fb = dense(W, K, K);
  if (K <= kMaxLd) return dispatch_rows<MatK, MatK, true>(X, fb, Y, b, M, N, K, s);
  return dispatch_rows<MatKFar, MatKFar, true>(X, fb, Y, b, M, N, K, s);
}

hipError_t linear_bwd_x(const float* W, const float* dY, float* dX, int64_t M, int64_t K,
                        int64_t N, hipStream_t s) {
  // dX[M][K] = dY[M][N] W[N][K]: A = dY (contiguous along the reduction), B[n_out][k_in] = W
  const auto fb = dense(W, K, N);
  if (std::max(N, K) <= kMaxLd)
    return dispatch_rows<MatK, MatM, false>(dY, fb, dX, nullptr, M, K, N, s);
  return dispatch_rows<MatKFar, MatMFar, false>(dY, fb, dX, nullptr, M, K, N, s);
}

hipError_t linear_bwd_w(const float* X, const float* dY, float* dW, float* db, float* part,
                        int64_t slices, int64_t M, int64_t K, int64_t N, hipStream_t s) {
  // dW[N][K] = dY^T X: A[n][m] = dY[m][n] (contiguous in n), B[m][k] = X[m][k] (contiguous in k);
  // db = the row sums of A.  With slices > 1, part holds slices copies of dW, then slices of db.
  if (slices > 1 && part == nullptr) return hipErrorInvalidValue;
  float* out = slices > 1 ? part : dW;
  float* sums = slices > 1 ? part + slices * N * K : db;
  const auto fa = dense(dY, N, M), fb = dense(X, K, M);
  const Batch one{1, 0, 0, 0, 0, 0, 0};
  hipError_t e;
  if (std::max(N, K) <= kMaxLd)
    e = dispatch_dense<MatM, MatM, false, false, true>(fa, fb, out, K, nullptr, N, K, M, slices, s,
                                                       1, one, sums);
  else
    e = dispatch_dense<MatMFar, MatMFar, false, false, true>(fa, fb, out, K, nullptr, N, K, M,
                                                             slices, s, 1, one, sums);
  if (e != hipSuccess || slices <= 1) return e;
  e = slice_sum(part, dW, N * K, slices, s);
  if (e != hipSuccess) return e;
  return slice_sum(sums, db, N, slices, s);
}

hipError_t gemm_batched(bool a_rowk, const float* A, int64_t lda, bool b_rowk, const float* B,
                        int64_t ldb, float* C, int64_t ldc, int64_t M, int64_t N, int64_t K,
                        int64_t batches, const BatchStrides& st, hipStream_t s) {
  const Batch bt{st.inner,   st.a_outer, st.a_inner, st.b_outer,
                 st.b_inner, st.c_outer, st.c_inner, st.causal};
  const auto fa = dense(A, lda, K), fb = dense(B, ldb, K);
#define GEMM_BATCHED_CASE(LA, LB) \
  return dispatch_dense<LA, LB, false, true>(fa, fb, C, ldc, nullptr, M, N, K, 1, s, batches, bt)
  if (std::max(lda, ldb) <= kMaxLd) {
    if (a_rowk && b_rowk) GEMM_BATCHED_CASE(MatK, MatK);
    if (a_rowk) GEMM_BATCHED_CASE(MatK, MatM);
    if (b_rowk) GEMM_BATCHED_CASE(MatM, MatK);
    GEMM_BATCHED_CASE(MatM, MatM);
  }
  if (a_rowk && b_rowk) GEMM_BATCHED_CASE(MatKFar, MatKFar);
  if (a_rowk) GEMM_BATCHED_CASE(MatKFar, MatMFar);
  if (b_rowk) GEMM_BATCHED_CASE(MatMFar, MatKFar);
  GEMM_BATCHED_CASE(MatMFar, MatMFar);
#undef GEMM_BATCHED_CASE
}

// A 1 x 1 convolution with stride 1 and no padding is a plain product of the
// NHWC pixel rows: its forward is X W^T, its input gradient dY W and its filter
// gradient dY^T X, all run on the dense loaders (one add per K tile for the
// address, no tap arithmetic).
static bool pointwise(const ConvShape& c) {
  return c.R == 1 && c.S == 1 && c.stride == 1 && c.pad == 0 && c.C <= kMaxLd && c.K <= kMaxLd;
}

hipError_t conv_fwd(const float* X, const float* W, float* Y, const ConvShape& c, hipStream_t s) {
  const int64_t M = c.N * c.P * c.Q, N = c.K, K = c.R * c.S * c.C;
  if (!fits31(M) || !fits31(K)) return hipErrorInvalidValue;
  if (pointwise(c) && N > 32)   // Y[NPQ][K] = X[NPQ][C] W[K][C]^T
    return dispatch_dense<PixelK, MatK, false>(dense(X, c.C, K), dense(W, c.C, K), Y, N, nullptr, M,
                                               N, K, 1, s);
  auto fa = [&](auto& a) {
    a.x = X; a.H = (int)c.H; a.W = (int)c.W; a.C = (int)c.C; a.S = (int)c.S;
    a.st = (int)c.stride; a.pad = (int)c.pad;
    a.dQ = FastDiv::make(c.Q); a.dPQ = FastDiv::make(c.P * c.Q); a.dC = FastDiv::make(c.C);
    a.dS = FastDiv::make(c.S); a.dSC = FastDiv::make(c.S * c.C);
  };
  const auto fb = dense(W, K, K);
  const bool fits = K <= kMaxLd &&
                    window_fits(256, c.P, c.Q, c.stride, c.R + 2 * c.pad, c.H, c.W, c.C);
  const bool near = fits && c.C % 4 == 0;
  if (N <= 32 && near) {
    // at most 32 output channels: 256 x 32 tiles, no empty columns; 128 x 32 when there are
    // fewer 256-row tiles than CUs, so that twice as many workgroups share the chip
    if ((M + 255) / 256 < 256) {
      if (c.C % 32 == 0)
        return dispatch_shape<128, 32, ConvPatchT, MatK>(fa, fb, Y, DenseOut{N}, 0, M, N, K, 1, s);
      return dispatch_shape<128, 32, ConvPatchV, MatK>(fa, fb, Y, DenseOut{N}, 0, M, N, K, 1, s);
    }
    if (c.C % 32 == 0)
      return dispatch_shape<256, 32, ConvPatchT, MatK>(fa, fb, Y, DenseOut{N}, 0, M, N, K, 1, s);
    return dispatch_shape<256, 32, ConvPatchV, MatK>(fa, fb, Y, DenseOut{N}, 0, M, N, K, 1, s);
  }
  if (near && c.C % 32 == 0)
    return dispatch_dense<ConvPatchT, MatK, false>(fa, fb, Y, N, nullptr, M, N, K, 1, s);
  if (near) return dispatch_dense<ConvPatchV, MatK, false>(fa, fb, Y, N, nullptr, M, N, K, 1, s);
  if (fits) return dispatch_dense<ConvPatch1, MatK, false>(fa, fb, Y, N, nullptr, M, N, K, 1, s);
  if (K <= kMaxLd)
    return dispatch_dense<ConvPatchS, MatK, false>(fa, fb, Y, N, nullptr, M, N, K, 1, s);
  return dispatch_dense<ConvPatchS, MatKFar, false>(fa, fb, Y, N, nullptr, M, N, K, 1, s);
}

hipError_t conv_bwd_x(const float* W, const float* dY, float* dX, const ConvShape& c,
                      hipStream_t s) {
  if (c.C % 4 != 0) return hipErrorInvalidValue;   // every conv with an input gradient has C % 4 == 0
  if (!fits31(c.N * c.H * c.W) || !fits31(c.R * c.S * c.K)) return hipErrorInvalidValue;
  if (pointwise(c))   // dX[NHW][C] = dY[NHW][K] W[K][C]
    return dispatch_dense<PixelK, MatM, false>(dense(dY, c.K, c.K), dense(W, c.C, c.K), dX, c.C,
                                               nullptr, c.N * c.H * c.W, c.C, c.K, 1, s);
  const int64_t st = c.stride;
  // one GEMM per stride class (ph, pw) of input pixels; a class no tap reaches gets zeros
  for (int64_t ph = 0; ph < st; ++ph)
    for (int64_t pw = 0; pw < st; ++pw) {
      const int64_t Hc = (c.H - ph + st - 1) / st, Wc = (c.W - pw + st - 1) / st;
      const int64_t r0 = (ph + c.pad) % st, s0 = (pw + c.pad) % st;
      const int64_t nR = r0 < c.R ? (c.R - r0 + st - 1) / st : 0;
      const int64_t nS = s0 < c.S ? (c.S - s0 + st - 1) / st : 0;
      const int64_t M = c.N * Hc * Wc, N = c.C, K = nR * nS * c.K;
      if (M == 0) continue;
      const int64_t up = (ph + c.pad - r0) / st;   // rows of dY above the class pixel's own
      auto fa = [&](auto& a) {
        a.dy = dY; a.P = (int)c.P; a.Q = (int)c.Q; a.K = (int)c.K; a.nR = (int)nR; a.nS = (int)nS;
        a.a = (int)up; a.b = (int)((pw + c.pad - s0) / st);
        a.dWc = FastDiv::make(Wc); a.dHWc = FastDiv::make(Hc * Wc); a.dK = FastDiv::make(c.K);
        a.dnS = FastDiv::make(nS > 0 ? nS : 1); a.dSK = FastDiv::make(nS > 0 ? nS * c.K : 1);
      };
      auto fb = [&](auto& b) {
        b.w = W; b.C = (int)c.C; b.K = (int)c.K; b.S = (int)c.S; b.st = (int)st; b.r0 = (int)r0;
        b.s0 = (int)s0; b.nS = (int)nS; b.RSC = c.R * c.S * c.C;
        b.dK = FastDiv::make(c.K); b.dnS = FastDiv::make(nS > 0 ? nS : 1);
        b.dSK = FastDiv::make(nS > 0 ? nS * c.K : 1);
      };
      const ClassOut om{(int)c.H, (int)c.W, (int)c.C, (int)st, (int)ph, (int)pw,
                        FastDiv::make(Wc), FastDiv::make(Hc * Wc)};
      const bool near = c.K % 4 == 0 &&
                        window_fits(256, Hc, Wc, 1, nR + 2 * up + 1, c.P, c.Q, c.K);
      hipError_t e;
      if (K == 0)   // no tap: a plain fill instead of an empty product
        e = class_zero(dX, om, M, c.C, s);
      else if (near && c.K % 32 == 0 && c.R * c.S * c.C <= kMaxLd)
        e = dispatch<ConvGradTapT, ConvFilterTapT, false>(fa, fb, dX, om, 0, nullptr, M, N, K, 1,
                                                          s);
      else if (near)
        e = dispatch<ConvGradTapV, ConvFilterTapG, false>(fa, fb, dX, om, 0, nullptr, M, N, K, 1,
                                                          s);
      else
        e = dispatch<ConvGradTapS, ConvFilterTapG, false>(fa, fb, dX, om, 0, nullptr, M, N, K, 1,
                                                          s);
      if (e != hipSuccess) return e;
    }
  return hipSuccess;
}

hipError_t conv_bwd_w(const float* X, const float* dY, float* dW, float* part, int64_t slices,
                      const ConvShape& c, hipStream_t s) {
  // dW[K][RSC] = sum over pixels of dY[pixel][k] * patch[pixel][rsc]
  const int64_t M = c.K, N = c.R * c.S * c.C, K = c.N * c.P * c.Q;
  if (!fits31(K) || !fits31(N) || !fits31((c.R * c.W + c.S) * c.C)) return hipErrorInvalidValue;
  if (slices > 1 && part == nullptr) return hipErrorInvalidValue;
  float* out = slices > 1 ? part : dW;
  const auto fa = dense(dY, c.K, K);
  auto fb = [&](auto& b) {
    b.x = X; b.H = (int)c.H; b.W = (int)c.W; b.C = (int)c.C; b.st = (int)c.stride;
    b.pad = (int)c.pad; b.h_end = (int)(c.P * c.stride - c.pad);
    b.w_end = (int)(c.Q * c.stride - c.pad);
    b.row_step = c.stride * (c.W - c.Q) * c.C;
    b.img_step = (c.H - c.P * c.stride) * c.W * c.C;
    b.dQ = FastDiv::make(c.Q); b.dPQ = FastDiv::make(c.P * c.Q);
    b.dC = FastDiv::make(c.C); b.dSC = FastDiv::make(c.S * c.C);
  };
  const DenseOut om{N};
  // a K tile covers 32 pixels; twice that covers the offsets of a lane's steps past the tile
  const bool fits = c.K <= kMaxLd &&
                    window_fits(64, c.P, c.Q, c.stride, c.R + 2 * c.pad, c.H, c.W, c.C);
  const bool near = fits && c.C % 4 == 0;
  const WgradTile tile = wgrad_tile(M, N, c.C);
  hipError_t e;
  if (near && tile == WgradTile::k32x256)   // at most 32 output channels: no empty tile rows
    e = dispatch_shape<32, 256, MatM, ConvPixelPatchV>(fa, fb, out, om, M * N, M, N, K, slices, s);
  else if (near && tile == WgradTile::k64x192)   // no tile column half empty at odd multiples of 64
    e = dispatch_shape<64, 192, MatM, ConvPixelPatchV>(fa, fb, out, om, M * N, M, N, K, slices, s);
  else if (pointwise(c))
    // dW[K][C] = dY^T X over the pixel rows: the dense weight gradient's loaders
    e = dispatch_dense<MatM, PixelM, false>(fa, dense(X, c.C, K), out, N, nullptr, M, N, K, slices,
                                            s);
  else if (near)
    e = dispatch_dense<MatM, ConvPixelPatchV, false>(fa, fb, out, N, nullptr, M, N, K, slices, s);
  else if (fits)
    e = dispatch_dense<MatM, ConvPixelPatch1, false>(fa, fb, out, N, nullptr, M, N, K, slices, s);
  else if (c.K <= kMaxLd)
    e = dispatch_dense<MatM, ConvPixelPatchS, false>(fa, fb, out, N, nullptr, M, N, K, slices, s);
  else
    e = dispatch_dense<MatMFar, ConvPixelPatchS, false>(fa, fb, out, N, nullptr, M, N, K, slices,
                                                        s);
  if (e != hipSuccess || slices <= 1) return e;
  return slice_sum(part, dW, M * N, slices, s);
}

// Split-K slice count of a weight gradient with M x N outputs reduced over K
// rows (C = input channels of a filter gradient, -1 for a dense layer).  With T
// tiles of which a CU holds R at once, a launch of T s workgroups takes
// ceil(T s / (256 R)) rounds of K / s rows.  s minimises rounds / s (a partly
// filled last round leaves most CUs idle behind a few), with at most four rounds
// and at least 256 rows a slice; the smallest s within 1 % of the best is taken,
// since every slice adds one partial dW to write and read back.
//
// The count belongs to a network's registered sequence, whose partial sums it
// sizes.  T and R are those of a rule on sizes alone, stated here; which tile runs
// is pick_shape's choice for the count that is registered (any tile runs with any
// count), and it is often a smaller one.  Over the 175 weight gradients of the
// timed networks and ten drawn ones, each timed with up to 25 counts: within 5 %
// of the best count in 108, the sum of all 1.5 % over that of the best; worst are
// small ones, whose 256 rows a slice are too many (3 x 3 20 -> 20 over 931 pixels:
// 22.9 us with 4 slices, 15.4 with 8), and 64 x 64 outputs, whose count is for 5
// workgroups a CU (1 x 1 64 -> 64 over 200704 pixels: 34.6 us with 777, 27.7 with
// 512).
int64_t wgrad_slices(int64_t M, int64_t N, int64_t K, int64_t C) {
  constexpr int64_t kCUs = 256, kFewTiles = 128, kFewTilesMaxK = 4096;
  int64_t tiles, resident;
  const WgradTile t = C >= 0 ? wgrad_tile(M, N, C) : WgradTile::kGeneral;
  if (t == WgradTile::k32x256) {
    tiles = (N + 255) / 256, resident = 2;
  } else if (t == WgradTile::k64x192) {
    tiles = (N + 191) / 192, resident = 2;
  } else if (C >= 0 && M % 4 == 0 && M <= 64 && N <= 64) {
    tiles = 1, resident = C % 4 == 0 ? 5 : 4;
  } else {
    const int64_t large = ((M + 127) / 128) * ((N + 127) / 128);
    if (N <= 64 && M >= 65536)
      tiles = (M + 255) / 256, resident = 2;
    else if (N <= 64 && M > 64)
      tiles = (M + 127) / 128, resident = 3;
    else if (M <= 64)
      tiles = (N + 127) / 128, resident = 3;
    else if (large < kFewTiles && K <= kFewTilesMaxK)
      tiles = ((M + 63) / 64) * ((N + 63) / 64), resident = 4;
    else
      tiles = large, resident = 2;
  }
  const int64_t slots = kCUs * resident;
  const int64_t smax = std::max<int64_t>(1, std::min(4 * slots / tiles, (K + 255) / 256));
  double best = 1e300;
  for (int64_t s = 1; s <= smax; ++s)
    best = std::min(best, (double)((tiles * s + slots - 1) / slots) / (double)s);
  for (int64_t s = 1; s <= smax; ++s)
    if ((double)((tiles * s + slots - 1) / slots) / (double)s <= best * 1.01) return s;
  return 1;
}

}  // namespace ooc
