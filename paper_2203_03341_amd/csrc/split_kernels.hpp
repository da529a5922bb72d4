// Step 1 of the error-corrected SGEMM: element split + repack, HBM-bandwidth bound.
//
// FP16 mode (Eqs. corr-1-1024 .. corr-4-1024):  v16 = toFP16(v),  dv16 = toFP16((v - toFP32(v16)) * 2^11)
// BF16 mode (three exact terms, stands in for the paper's TF32 pair on hardware without a TF32
// matrix instruction):  b0 = toBF16(v), b1 = toBF16(v - b0), b2 = toBF16(v - b0 - b1)
// Conversions round to nearest even (the hardware converts) and saturate: a finite input never
// yields an infinite part.  An infinite input keeps only its high part.  SplitKind lists the other
// splits the kernels can produce for the paper's comparison methods.
//
// Output layout ("fragment order"), 16-bit elements:
//     packed[row_block][k_step][part][lane][8],  row_block = r / 32, k_step = k / 16,
//     lane = ((k % 16) / 8) * 32 + r % 32, element = k % 8
// so that one 1 KiB chunk is exactly what the 64 lanes of a wave feed to one
// v_mfma_f32_32x32x16 operand, and a block tile is a run of whole chunks.  Rows are padded to
// kRowPad and depth to kDepthPad with zeros, which makes every tile of the product kernel full.
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

namespace ecgemm {

constexpr int kRowPad = 256;
constexpr int kDepthPad = 32;
constexpr int kChunkElems = 512;  // 64 lanes x 8 elements

typedef _Float16 half8_t __attribute__((ext_vector_type(8)));
typedef __bf16 bf16x8_t __attribute__((ext_vector_type(8)));
typedef unsigned short ushort8_t __attribute__((ext_vector_type(8)));

__device__ __forceinline__ float saturate_finite(float v, float limit) {
  // leaves Inf and NaN alone, clamps everything finite into [-limit, limit]
  return (__builtin_fabsf(v) <= 3.402823466e+38f) ? __builtin_fminf(__builtin_fmaxf(v, -limit), limit) : v;
}

// What a value is split into.  The first two are the method; the others exist to reproduce the paper's
// comparisons (Markidis' unscaled residual, and plain conversion with no residual at all).
enum SplitKind {
  kSplitFp16Scaled = 0,    // v16, (v - v16) * 2^11      Eqs. corr-elm-1, corr-elm-2-1024 ("halfhalf")
  kSplitBf16x3 = 1,        // three exact BF16 terms
  kSplitFp16Unscaled = 2,  // v16, v - v16               Eqs. corr-elm-1, corr-elm-2 ("Markidis' halfhalf")
  kSplitFp16Plain = 3,     // v16 only
  kSplitBf16Plain = 4,     // toBF16(v) only
  kSplitFp32 = 5           // v itself, repacked for the FP32 matrix instruction (the baseline the method is set against)
};

// 1 KiB chunks per (32 rows x 16 k).  kSplitFp32 has two as well, but they are the two 8-deep halves of the k step,
// 32 rows x 8 k of 32-bit elements each, not two parts of every element.
__host__ __device__ constexpr int parts_of_split(int kind) {
  return kind == kSplitBf16x3 ? 3 : (kind == kSplitFp16Plain || kind == kSplitBf16Plain) ? 1 : 2;
}
__host__ __device__ constexpr bool split_is_bf16(int kind) { return kind == kSplitBf16x3 || kind == kSplitBf16Plain; }

constexpr float kBf16Max = 3.3895313892515355e+38f;  // largest finite BF16

// 2^e for a per-row scaling exponent e in [-126, 127]
__device__ __forceinline__ float row_scale_factor(int e) { return __builtin_bit_cast(float, (unsigned)(e + 127) << 23); }

template <int KIND>
struct Splitter {
  static constexpr int kParts = parts_of_split(KIND);
  __device__ static __forceinline__ void split(float v, unsigned short (&out)[kParts]) {
    if constexpr (!split_is_bf16(KIND)) {
      const _Float16 hi = (_Float16)saturate_finite(v, 65504.0f);
      out[0] = __builtin_bit_cast(unsigned short, hi);
      if constexpr (kParts == 2) {
        float residual = v - (float)hi;                                  // exact
        // exact; a residual beyond +-32 saturates the low part anyway, and cutting it there first keeps the
        // multiplication from overflowing FP32 for inputs of magnitude 2^117 and more
        if constexpr (KIND == kSplitFp16Scaled) residual = saturate_finite(residual, 32.0f) * 2048.0f;
        const _Float16 lo = (_Float16)saturate_finite(residual, 65504.0f);
        // an infinite input keeps only its high part (selected on the bits: no branch around the conversion)
        const unsigned short keep = (__builtin_bit_cast(unsigned short, hi) & 0x7fffu) == 0x7c00u ? 0u : 0xffffu;
        out[1] = __builtin_bit_cast(unsigned short, lo) & keep;
      }
    } else {
      const __bf16 b0 = (__bf16)saturate_finite(v, kBf16Max);
      out[0] = __builtin_bit_cast(unsigned short, b0);
      if constexpr (kParts == 3) {
        const float r1 = v - (float)b0;
        const __bf16 b1 = (__bf16)saturate_finite(r1, kBf16Max);
        const float r2 = r1 - (float)b1;
        const __bf16 b2 = (__bf16)saturate_finite(r2, kBf16Max);
        const unsigned short keep = (out[0] & 0x7fffu) == 0x7f80u ? 0u : 0xffffu;  // infinite input: high part only
        out[1] = __builtin_bit_cast(unsigned short, b1) & keep;
        out[2] = __builtin_bit_cast(unsigned short, b2) & keep;
      }
    }
  }
};

// The split for values that need no care, two at a time (the two 16-bit results of a part share a register: out[q]
// holds part q of v0 in its low half and of v1 in its high half).  It has none of Splitter's clamps and masks; on a
// value whose high part comes out finite both give the same bits: the high part is then at most the largest finite
// number of the format whether or not the value was clamped to it first, the residuals are at most half a unit of
// its last place, far inside the range of the low parts, and nothing is masked.  A value that Splitter treats
// differently (beyond the format's range, where it saturates; infinite; NaN) is one whose high part is infinite or NaN.
typedef float fused_float2_t __attribute__((ext_vector_type(2)));
typedef _Float16 fused_half2_t __attribute__((ext_vector_type(2)));
typedef __bf16 fused_bf16x2_t __attribute__((ext_vector_type(2)));
template <int KIND>
struct FastSplit {
  static constexpr int kParts = parts_of_split(KIND);
  // `scaled0`, `scaled1`: the same two values times 2^11 (used by kSplitFp16Scaled only), so that the scaled residual
  // is one fused multiply-add on the packed high part: hi * -2^11 + v * 2^11 = (v - hi) * 2^11, exact like the
  // two-step form (v * 2^11 overflows only for values whose high part is not finite, which do not end up here).
  __device__ static __forceinline__ void split2(float v0, float v1, float scaled0, float scaled1, unsigned (&out)[kParts]) {
    if constexpr (!split_is_bf16(KIND)) {
      const fused_half2_t hi = __builtin_convertvector(fused_float2_t{v0, v1}, fused_half2_t);
      out[0] = __builtin_bit_cast(unsigned, hi);
      if constexpr (KIND == kSplitFp16Scaled) {
        // (the multiply-add in 32 bits and one packed conversion: the form that delivers a half by itself takes 8 cycles
        // where the others take 4, and holds up the matrix instructions of other waves; hence the empty statement.  FP16 calls
        // with that form / with this one: 1024^3 NN 14.2 / 13.9 us, NT 14.5 / 14.0, TN 13.8 / 13.9, 512^3 7.4 / 7.2, 256^3 6.1 /
        // 5.9, and behind where blocks walk a long way with little else to do, 192 x 1920 x 62912 NN 308 / 315, NT 319 / 321)
        float r0 = __builtin_fmaf((float)hi[0], -2048.0f, scaled0), r1 = __builtin_fmaf((float)hi[1], -2048.0f, scaled1);
        asm("" : "+v"(r0), "+v"(r1));
        out[1] = __builtin_bit_cast(unsigned, __builtin_convertvector(fused_float2_t{r0, r1}, fused_half2_t));
      } else if constexpr (kParts == 2) {
        const fused_float2_t residual = {v0 - (float)hi[0], v1 - (float)hi[1]};  // exact
        out[1] = __builtin_bit_cast(unsigned, __builtin_convertvector(residual, fused_half2_t));
      }
    } else {
      const fused_bf16x2_t b0 = __builtin_convertvector(fused_float2_t{v0, v1}, fused_bf16x2_t);
      out[0] = __builtin_bit_cast(unsigned, b0);
      if constexpr (kParts == 3) {
        const fused_float2_t r1 = {v0 - (float)b0[0], v1 - (float)b0[1]};
        const fused_bf16x2_t b1 = __builtin_convertvector(r1, fused_bf16x2_t);
        const fused_float2_t r2 = {r1[0] - (float)b1[0], r1[1] - (float)b1[1]};
        out[1] = __builtin_bit_cast(unsigned, b1);
        out[2] = __builtin_bit_cast(unsigned, __builtin_convertvector(r2, fused_bf16x2_t));
      }
    }
  }
  // The test for that, one instruction for two values: `largest` starts at 0 and is raised to their magnitudes (a NaN
  // stays one); every high part is finite if ordinary(largest).
  __device__ static __forceinline__ void raise(float& largest, float v0, float v1) {
    largest = __builtin_elementwise_maximum(__builtin_elementwise_maximum(largest, __builtin_fabsf(v0)), __builtin_fabsf(v1));
  }
  __device__ static __forceinline__ bool ordinary(float largest) {
    return largest < (split_is_bf16(KIND) ? 0x1.ffp127f : 65520.0f);  // from here on a value rounds to infinity
  }
};

// What the automatic mode choice needs to know about an operand: how much of it the FP16 pair loses, and how many
// elements of a row carry its weight.  Per thread, then per block: the sums of (x - (v16 + dv16 2^-11))^2, of x^2 and
// of |x| over the elements handled, in FP64.
struct SplitStats {
  double err2 = 0.0, norm2 = 0.0, abs1 = 0.0;
};
constexpr int kStatsPerBlock = 3;  // doubles a block leaves: err2, norm2, abs1

// The criterion of the automatic mode choice (see choose_mode_kernel) on the sums (err2, norm2, abs1) of A and of B.
__device__ __forceinline__ bool choice_fits(const double* a, double rows_a, const double* b, double rows_b, double tolerance2,
                                            double min_terms) {
  const bool represented = a[0] <= tolerance2 * a[1] && b[0] <= tolerance2 * b[1];
  // (sum |x|)^2 >= min_terms rows sum x^2, for either operand; an all-zero operand has nothing to lose
  const bool spread = a[2] * a[2] >= min_terms * rows_a * a[1] || b[2] * b[2] >= min_terms * rows_b * b[1] ||
                      a[1] == 0.0 || b[1] == 0.0;
  return represented && spread;
}

// What measure_rows_kernel leaves: per block kMeasureSums sums, err2, norm2, abs1 as they are (see SplitStats), then with
// the rows scaled; and what is made of them.
constexpr int kMeasureSums = 6;
struct RowSums {
  const double* a;
  const double* b;
  unsigned blocks_a, blocks_b;
  double rows_a, rows_b, tolerance, min_terms;
  int if_fits, if_fits_scaled, if_not;
  int* choice;
};
// The choice by the criterion above for either candidate: if_fits, else if_fits_scaled, else if_not.  Called by every
// thread of a block of at least 256; every sum in a fixed order, so that every block comes to the same choice.
__device__ __forceinline__ int choose_from_rows(const RowSums& sums, bool publish) {
  __shared__ double partial[4][kMeasureSums];
  const int t = threadIdx.x, wave = t >> 6;
  if (t < 256) {
    const bool second = t >= 128;  // two waves per operand
    const double* from = second ? sums.b : sums.a;
    const unsigned blocks = second ? sums.blocks_b : sums.blocks_a;
    double sum[kMeasureSums] = {};
#pragma unroll 2
    for (unsigned i = t & 127; i < blocks; i += 128)
#pragma unroll
      for (int q = 0; q < kMeasureSums; ++q) sum[q] += from[kMeasureSums * (size_t)i + q];
#pragma unroll
    for (int q = 0; q < kMeasureSums; ++q) {
#pragma unroll
      for (int d = 32; d >= 1; d >>= 1) sum[q] += __shfl_xor(sum[q], d, 64);
      if ((t & 63) == 0) partial[wave][q] = sum[q];
    }
  }
  __syncthreads();
  const double t2 = sums.tolerance * sums.tolerance;
  auto fits = [&](int at) {
    double a[kStatsPerBlock], b[kStatsPerBlock];
#pragma unroll
    for (int q = 0; q < kStatsPerBlock; ++q) a[q] = partial[0][at + q] + partial[1][at + q], b[q] = partial[2][at + q] + partial[3][at + q];
    return choice_fits(a, sums.rows_a, b, sums.rows_b, t2, sums.min_terms);
  };
  const int choice = fits(0) ? sums.if_fits : fits(kStatsPerBlock) ? sums.if_fits_scaled : sums.if_not;
  if (publish && t == 0) *sums.choice = choice;
  return __builtin_amdgcn_readfirstlane(choice);
}

// Binary exponent of a non-zero finite value, FP32 subnormals counted as -127; INT_MIN for zero, infinities and NaN
// (the elements that the per-row scaling exponents ignore).
__device__ __forceinline__ int finite_exponent(float v) {
  const unsigned bits = __builtin_bit_cast(unsigned, v) & 0x7fffffffu;
  return (bits != 0 && bits < 0x7f800000u) ? (int)(bits >> 23) - 127 : -0x7fffffff - 1;
}
// max of finite_exponent over eight values (before any pre-scaling)
__device__ __forceinline__ int finite_exponent8(const float (&v)[8]) {
  int hi = -0x7fffffff - 1;
#pragma unroll
  for (int e = 0; e < 8; ++e) hi = max(hi, finite_exponent(v[e]));
  return hi;
}
// Four neighbouring lanes hold values of one row: the row's maximum goes to row_max[r] from the first of them.
__device__ __forceinline__ void publish_row_exponent_of_4_lanes(int* __restrict__ row_max, int64_t r, bool row_exists, int hi) {
  hi = max(hi, __shfl_xor(hi, 1, 64));
  hi = max(hi, __shfl_xor(hi, 2, 64));
  if ((threadIdx.x & 3) == 0 && row_exists && hi != -0x7fffffff - 1) atomicMax(&row_max[r], hi);
}

// Writes the eight consecutive-k values `v` of row r (global indices) to their place in `packed`.
template <int KIND, bool STATS = false>
__device__ __forceinline__ void store_fragment_row(unsigned short* __restrict__ packed, int64_t k_steps_total,
                                                   int64_t r, int64_t k, const float (&v)[8], SplitStats* stats = nullptr) {
  if constexpr (KIND == kSplitFp32) {
    // v_mfma_f32_32x32x2_f32 takes one float per lane: lane l supplies row l % 32 and k = l / 32 of a 2-deep step.
    // A 1 KiB chunk holds four such steps, 16 bytes per lane: element k % 8 of the row goes to lane
    // (k % 2) * 32 + r % 32, float (k % 8) / 2.
    typedef float native4 __attribute__((ext_vector_type(4)));
    const int64_t chunk_index = ((r >> 5) * k_steps_total + (k >> 4)) * 2 + ((k >> 3) & 1);
    float* chunk = reinterpret_cast<float*>(packed) + chunk_index * (kChunkElems / 2) + (int)(r & 31) * 4;
    native4 even = {v[0], v[2], v[4], v[6]}, odd = {v[1], v[3], v[5], v[7]};
    *reinterpret_cast<native4*>(chunk) = even;
    *reinterpret_cast<native4*>(chunk + 32 * 4) = odd;
    return;
  }
  constexpr int NP = Splitter<KIND>::kParts;
  ushort8_t parts[NP];
  // The short split where every value of the wave is ordinary: 4 vector instructions per element against about 20, which
  // operands that come from the caches and the measuring split (with its sums in 64 bits) wait for.  Whole calls with
  // the general one throughout / with this: FP16 2048^3 58.4 / 57.2 us, 1024 x 1024 x 65536 527 / 523 us, the automatic
  // mode at 8192^3 on a wide range (two measuring splits) 2707 / 2679 us; the others within 0.3 %.  A wave that does hold
  // a value beyond the format pays for both: a 2048 x 2048 operand full of them, split by itself, 5.8 / 6.3 us, and the
  // product of it, 2048^3, 51.6 / 50.8 with the rest of the call.
  constexpr bool kShort = (KIND == kSplitFp16Scaled || KIND == kSplitBf16x3);
  bool done = false;
  if constexpr (kShort) {
    unsigned words[4][NP];
    float largest = 0.0f;
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      FastSplit<KIND>::raise(largest, v[2 * e], v[2 * e + 1]);
      FastSplit<KIND>::split2(v[2 * e], v[2 * e + 1], v[2 * e] * 2048.0f, v[2 * e + 1] * 2048.0f, words[e]);
    }
    done = __builtin_amdgcn_ballot_w64(!FastSplit<KIND>::ordinary(largest)) == 0;  // wave-uniform
    typedef unsigned uint4_t __attribute__((ext_vector_type(4)));
#pragma unroll
    for (int p = 0; p < NP; ++p)
      parts[p] = __builtin_bit_cast(ushort8_t, uint4_t{words[0][p], words[1][p], words[2][p], words[3][p]});
  }
  if (!done)
#pragma unroll
  for (int e = 0; e < 8; ++e) {
    unsigned short s[NP];
    Splitter<KIND>::split(v[e], s);
#pragma unroll
    for (int p = 0; p < NP; ++p) parts[p][e] = s[p];
  }
  if constexpr (STATS && KIND == kSplitFp16Scaled) {
#pragma unroll
    for (int e = 0; e < 8; ++e) {
      // (every step exact where nothing saturates: what is lost is a multiple of the last place of v)
      const float residual = v[e] - (float)__builtin_bit_cast(_Float16, (unsigned short)parts[0][e]);
      const double lost = (double)__builtin_fmaf((float)__builtin_bit_cast(_Float16, (unsigned short)parts[1][e]), -0x1p-11f, residual);
      const double x = (double)v[e];
      stats->err2 += lost * lost;
      stats->norm2 += x * x;
      stats->abs1 += __builtin_fabs(x);
    }
  }
  const int64_t row_block = r >> 5, k_step = k >> 4;
  const int lane = (int)((k >> 3) & 1) * 32 + (int)(r & 31);
  unsigned short* chunk = packed + ((row_block * k_steps_total + k_step) * NP) * kChunkElems + lane * 8;
#pragma unroll
  for (int p = 0; p < NP; ++p) *reinterpret_cast<ushort8_t*>(chunk + p * kChunkElems) = parts[p];
}

constexpr int kSplitDeepTiles = 4;

// One operand to split: X = op(src), rows x depth, into `packed`.
struct SplitJob {
  const float* src;
  int64_t ld, rows, depth;
  int64_t k_steps_total;      // padded depth / 16
  float prescale;             // a power of two chosen by the caller (1 by default): exact
  const int* row_log2_scale;  // optional per-row exponents, applied on top of prescale
  unsigned short* packed;
  unsigned fast_tiles;        // tiles along the direction in which the blocks are numbered first
  unsigned blocks;
  int variant;                // SplitVariant
  bool streamed;              // kSplitRContiguousWide: non-temporal loads of the source (operands larger than the memory-side cache)
  bool runs;                  // the blocks of one XCD take one contiguous run of the tiles (see tile_of_block)
  // Automatic mode choice only, else null: block b leaves its SplitStats at stats[kStatsPerBlock b ...]
  double* stats;
  // Automatic mode choice only, else null: the kernel does nothing unless *gate == gate_value
  const int* gate;
  int gate_value;
  // Automatic mode choice only, else null (STATS kernels): row_max[r] is raised to the largest finite_exponent of row
  // r's elements as they are in `src` (the caller has set every entry to INT_MIN), so that the scaling exponents of
  // ecgemm_row_scales need no pass of their own
  int* row_max;
};

// Sums the threads' statistics over the block in a fixed order and stores them (all 256 threads call this).
__device__ __forceinline__ void store_block_stats(const SplitStats& mine, double* __restrict__ out, double* scratch12) {
  double e = mine.err2, n = mine.norm2, a = mine.abs1;
#pragma unroll
  for (int d = 32; d >= 1; d >>= 1) {
    e += __shfl_xor(e, d, 64);
    n += __shfl_xor(n, d, 64);
    a += __shfl_xor(a, d, 64);
  }
  const int wave = threadIdx.x >> 6;
  if ((threadIdx.x & 63) == 0) scratch12[3 * wave] = e, scratch12[3 * wave + 1] = n, scratch12[3 * wave + 2] = a;
  __syncthreads();
  if (threadIdx.x < kStatsPerBlock)
    out[threadIdx.x] = (scratch12[threadIdx.x] + scratch12[3 + threadIdx.x]) + (scratch12[6 + threadIdx.x] + scratch12[9 + threadIdx.x]);
}
enum SplitVariant { kSplitKContiguous = 0, kSplitKContiguousDeep = 1, kSplitRContiguous = 2, kSplitRContiguousWide = 3 };

// Four values of the source, at any multiple of 4 bytes.  STREAMED: non-temporal, so that an operand that is too large to
// be found in the memory-side cache by anyone later does not push out of it what was just packed.
typedef float source4_t __attribute__((ext_vector_type(4)));
template <bool STREAMED>
__device__ __forceinline__ source4_t load_source4(const float* from) {
  typedef float any4_t __attribute__((ext_vector_type(4), aligned(4)));
  const any4_t* at = reinterpret_cast<const any4_t*>(from);
  return STREAMED ? __builtin_nontemporal_load(at) : *at;
}
// x[behind .. 3] and zeros after it
__device__ __forceinline__ source4_t shift_or_zero(const source4_t& x, int64_t behind) {
  source4_t y;
#pragma unroll
  for (int i = 0; i < 4; ++i) {
    y[i] = behind == 0 ? x[i] : 0.0f;
#pragma unroll
    for (int d = 1; i + d < 4; ++d) y[i] = behind == d ? x[i + d] : y[i];
  }
  return y;
}
// line[at .. at + 3] of a line of `count` >= 4 values, zero behind its end: one load inside the line, whatever `at` >= 0
template <bool STREAMED>
__device__ __forceinline__ source4_t load_source4_or_zero(const float* line, int64_t at, int64_t count) {
  const int64_t inside = at < count - 4 ? at : count - 4;
  return shift_or_zero(load_source4<STREAMED>(line + inside), at - inside);
}

// Source with k contiguous, X(r, k) = src[k + r * ld].  One block: 64 rows x 32 k, 256 threads, thread t handles row
// t / 4 and the 8 values starting at k = 8 * (t % 4), two 16-byte loads; or TILES such tiles next to each other in k, whose
// loads are all requested before the first is split (kernels of their own: one tile takes 24 to 34 registers, four 58 to
// 61, which leaves eight waves on a SIMD).  Blocks are numbered with k fastest.  The memory path takes 16 bytes at any
// multiple of four, so rows that start on no alignment (lda = 5003) are read like the others: 4095 x 5003 FP16 31.1 us /
// 25.3 and BF16 36.4 / 32.1 with lanes along k, one value each, handed to the row's thread through LDS / so; 9001 x 9001
// 161 / 118 and 195 / 149.
template <int KIND, int TILES, bool STATS>
__device__ __forceinline__ void split_tiles_k_contiguous(const SplitJob& job, unsigned block, SplitStats* stats) {
  const int t = threadIdx.x;
  const int64_t r = (int64_t)(block / job.fast_tiles) * 64 + (t >> 2);
  const int64_t k0 = (int64_t)(block % job.fast_tiles) * (32 * TILES) + (t & 3) * 8;
  // A block of nothing but padding (the same for all its threads) has nothing to load: 64 x 31936 FP16 9.1 us / 8.0 with the
  // clamped loads below / so.  (It returns: a path without loads that joined the others would make every block wait for
  // all of its loads at the join, 2048 x 4096 FP16 12.4 us / 12.8.)
  if (r - (t >> 2) >= job.rows) {
    const float zeros[8] = {};
#pragma unroll
    for (int s = 0; s < TILES; ++s)
      if (k0 + 32 * s < job.k_steps_total * 16) store_fragment_row<KIND>(job.packed, job.k_steps_total, r, k0 + 32 * s, zeros);
    return;
  }
  float prescale = job.prescale;
  if (job.row_log2_scale != nullptr && r < job.rows) prescale *= row_scale_factor(job.row_log2_scale[r]);
  const float* src = job.src;
  float v[TILES][8];
  if (r - (t >> 2) + 64 <= job.rows && k0 - (t & 3) * 8 + 32 * TILES <= job.depth) {  // the same for the block
    // (without a condition of its own for every tile: the compiler waits for a tile's loads where their branches join)
    const float* from = src + r * job.ld + k0;
    source4_t lo[TILES], hi[TILES];
#pragma unroll
    for (int s = 0; s < TILES; ++s) lo[s] = load_source4<false>(from + 32 * s), hi[s] = load_source4<false>(from + 32 * s + 4);
#pragma unroll
    for (int s = 0; s < TILES; ++s)
#pragma unroll
      for (int e = 0; e < 4; ++e) v[s][e] = lo[s][e], v[s][4 + e] = hi[s][e];
  } else if (job.depth >= 4) {
    const float* line = src + (r < job.rows ? r : job.rows - 1) * job.ld;
    const int64_t count = job.depth;
    // (two tiles at a time: the clamped loads of four would take 70 registers and a wave of every SIMD, 2048 x 4096 FP16
    // 12.0 us / 11.7 so, BF16 level)
    constexpr int GROUP = TILES > 1 ? TILES / 2 : 1;
#pragma unroll
    for (int g = 0; g < TILES; g += GROUP) {
      source4_t x[2 * GROUP];
#pragma unroll
      for (int s = 0; s < 2 * GROUP; ++s) x[s] = load_source4_or_zero<false>(line, k0 + 32 * (g + s / 2) + 4 * (s % 2), count);
#pragma unroll
      for (int s = 0; s < 2 * GROUP; ++s)
#pragma unroll
        for (int e = 0; e < 4; ++e) v[g + s / 2][4 * (s % 2) + e] = r < job.rows ? x[s][e] : 0.0f;
      if (TILES > 1) __builtin_amdgcn_sched_barrier(0);
    }
  } else {
#pragma unroll
    for (int s = 0; s < TILES; ++s) {
      const int64_t k = k0 + 32 * s;
#pragma unroll
      for (int e = 0; e < 8; ++e) v[s][e] = (r < job.rows && k + e < job.depth) ? src[r * job.ld + k + e] : 0.0f;
    }
  }
  if constexpr (STATS) {
    if (job.row_max != nullptr) {
      int hi = -0x7fffffff - 1;
#pragma unroll
      for (int s = 0; s < TILES; ++s) hi = max(hi, finite_exponent8(v[s]));
      publish_row_exponent_of_4_lanes(job.row_max, r, r < job.rows, hi);
    }
  }
#pragma unroll
  for (int s = 0; s < TILES; ++s) {
    const int64_t k = k0 + 32 * s;
    if (TILES > 1 && k >= job.k_steps_total * 16) break;  // (the padded depth is a multiple of 32: the same for the block)
#pragma unroll
    for (int e = 0; e < 8; ++e) v[s][e] *= prescale;
    store_fragment_row<KIND, STATS>(job.packed, job.k_steps_total, r, k, v[s], stats);
  }
}
// Source with r contiguous: X(r, k) = src[r + k * ld], any alignment.  One block: 64 rows x 32 k.  Lanes run along r,
// so a thread reads the 8 consecutive-k values of its row directly and each read instruction of a wave is a 256-byte
// run.  Blocks are numbered with the row tile fastest: neighbours in the launch order read neighbouring runs.
template <int KIND, bool STATS = false>
__device__ __forceinline__ void split_block_r_contiguous(const SplitJob& job, unsigned block, SplitStats* stats = nullptr) {
  const int t = threadIdx.x, lane = t & 63, wave = __builtin_amdgcn_readfirstlane(t >> 6);
  const int64_t r0 = (int64_t)(block % job.fast_tiles) * 64, r = r0 + lane;
  const int64_t k = (int64_t)(block / job.fast_tiles) * 32 + wave * 8;
  if (r0 >= job.rows) {  // nothing but padding (the same for the block)
    const float zeros[8] = {};
    store_fragment_row<KIND>(job.packed, job.k_steps_total, r, k, zeros);
    return;
  }
  float prescale = job.prescale;
  if (job.row_log2_scale != nullptr && r < job.rows) prescale *= row_scale_factor(job.row_log2_scale[r]);
  // Addresses clamped into the operand and zeros selected, in every block: a condition at a load, in a path of its own for
  // the blocks at the edge, makes that path wait for the loads before it (calls with a kept operand, such a path / so: BF16
  // 65 x 9379 x 686 27.5 us / 26.9, 4847 x 192 x 311 24.3 / 24.0, 75 x 1539 x 7700 32.1 / 31.5).
  const unsigned row = (unsigned)(r < job.rows ? lane : job.rows - 1 - r0);
  const int64_t behind = job.depth - 1 - k;
  const int last = (int)(behind < 0 ? -1 : behind < 7 ? behind : 7);  // of the eight k inside the depth
  const float* line = job.src + r0 + (behind < 0 ? job.depth - 1 : k) * job.ld;
  float v[8];
#pragma unroll
  for (int e = 0; e < 8; ++e) {
    v[e] = line[row];
    line += e < last ? job.ld : 0;
  }
  __builtin_amdgcn_sched_barrier(0);
#pragma unroll
  for (int e = 0; e < 8; ++e) {
    asm("" : "+v"(v[e]));  // (a load whose value is selected once would otherwise move under the condition)
    v[e] = r < job.rows && e <= last ? v[e] : 0.0f;
  }
  if constexpr (STATS) {
    const int hi = finite_exponent8(v);
    if (job.row_max != nullptr && r < job.rows && hi != -0x7fffffff - 1) atomicMax(&job.row_max[r], hi);
  }
#pragma unroll
  for (int e = 0; e < 8; ++e) v[e] *= prescale;
  store_fragment_row<KIND, STATS>(job.packed, job.k_steps_total, r, k, v, stats);
}

// Source with r contiguous.  One block: 256 rows x 32 k through 32 KiB of LDS (`tile`).  A wave reads one k line of 256
// rows per instruction (1 KiB runs, 16 bytes per lane), all eight of its lines before it waits for the first; after the
// barrier thread t owns row t and picks its 8-value groups out of LDS along k (lanes on consecutive words: no bank
// conflicts).  5.4 TB/s at 16384^2 against 3.9 TB/s for the 64-row kernel above.  FP16 2048 x 2048 6.6 us / 5.8, 4096 x
// 4096 25.2 / 21.3, 1024 x 65536 91.7 / 80.4 with each line waited for before the next / so.
template <bool STREAMED>
__device__ __forceinline__ void stage_r_contiguous_wide(const SplitJob& job, unsigned block, float* tile) {
  const int t = threadIdx.x, lane = t & 63, wave = t >> 6;
  const int64_t r0 = (int64_t)(block % job.fast_tiles) * 256, k0 = (int64_t)(block / job.fast_tiles) * 32;
  const float* src = job.src;
  if (r0 + 256 <= job.rows && k0 + 32 <= job.depth) {  // the same for the block
    // (without a condition of its own for every load: the compiler waits for a load where its branches join)
    const float* from = src + r0 + 4 * lane + (k0 + wave) * job.ld;
    source4_t x[8];
#pragma unroll
    for (int j = 0; j < 8; ++j) x[j] = load_source4<STREAMED>(from + 4 * j * job.ld);
#pragma unroll
    for (int j = 0; j < 8; ++j) *reinterpret_cast<source4_t*>(&tile[(wave + 4 * j) * 256 + 4 * lane]) = x[j];
  } else if (job.rows >= 4) {
    source4_t x[8];
#pragma unroll
    for (int j = 0; j < 8; ++j) {
      const int64_t k = k0 + wave + 4 * j;
      x[j] = load_source4_or_zero<STREAMED>(src + (k < job.depth ? k : job.depth - 1) * job.ld, r0 + 4 * lane, job.rows);
    }
#pragma unroll
    for (int j = 0; j < 8; ++j) {
      const source4_t zero = {0.0f, 0.0f, 0.0f, 0.0f};
      *reinterpret_cast<source4_t*>(&tile[(wave + 4 * j) * 256 + 4 * lane]) = k0 + wave + 4 * j < job.depth ? x[j] : zero;
    }
  } else {
#pragma unroll
    for (int j = 0; j < 8; ++j) {
      const int64_t k = k0 + wave + 4 * j;
#pragma unroll
      for (int e = 0; e < 4; ++e)
        tile[(wave + 4 * j) * 256 + 4 * lane + e] = r0 + 4 * lane + e < job.rows && k < job.depth ? src[r0 + 4 * lane + e + k * job.ld] : 0.0f;
    }
  }
}
template <int KIND, bool STATS = false>
__device__ __forceinline__ void split_block_r_contiguous_wide(const SplitJob& job, unsigned block, float* tile, SplitStats* stats = nullptr) {
  const int t = threadIdx.x;
  const int64_t r0 = (int64_t)(block % job.fast_tiles) * 256, k0 = (int64_t)(block / job.fast_tiles) * 32;
  if (!STATS && job.streamed) stage_r_contiguous_wide<true>(job, block, tile);
  else stage_r_contiguous_wide<false>(job, block, tile);
  __syncthreads();
  float prescale = job.prescale;
  if (job.row_log2_scale != nullptr && r0 + t < job.rows) prescale *= row_scale_factor(job.row_log2_scale[r0 + t]);
  int row_hi = -0x7fffffff - 1;
#pragma unroll
  for (int g = 0; g < 4; ++g) {
    float v[8];
#pragma unroll
    for (int e = 0; e < 8; ++e) v[e] = tile[(8 * g + e) * 256 + t];
    if constexpr (STATS) row_hi = max(row_hi, finite_exponent8(v));
#pragma unroll
    for (int e = 0; e < 8; ++e) v[e] *= prescale;
    store_fragment_row<KIND, STATS>(job.packed, job.k_steps_total, r0 + t, k0 + 8 * g, v, stats);
  }
  if constexpr (STATS)
    if (job.row_max != nullptr && r0 + t < job.rows && row_hi != -0x7fffffff - 1) atomicMax(&job.row_max[r0 + t], row_hi);
}

// Workgroups are dealt round-robin to the 8 XCDs, each with its own L2.  Block b of n takes the tile at this position
// where every XCD is to work through one contiguous run of the tile list.
__device__ __forceinline__ unsigned xcd_run_position(unsigned b, unsigned n) {
  const unsigned per = n / 8, rem = n % 8, x = b % 8;
  return x * per + (x < rem ? x : rem) + b / 8;
}

// The tile of block b.  With `runs`, neighbouring tiles, which share cache lines at their common edge where a source's
// lines start anywhere, meet in one L2 instead of being fetched by two.  (make_split_job in ecgemm.hip decides.)
__device__ __forceinline__ unsigned tile_of_block(const SplitJob& job, unsigned b) { return job.runs ? xcd_run_position(b, job.blocks) : b; }

// Whether a gated kernel is to run (automatic mode choice: both candidates' kernels are enqueued, and the ones of the
// mode not chosen return at once).
__device__ __forceinline__ bool gate_open(const int* gate, int gate_value) {
  return gate == nullptr || *gate == gate_value;
}

// One operand per launch; VARIANT is fixed at compile time so that only the kernels that stage through LDS hold any.
// STATS (automatic mode choice): block b also leaves its SplitStats at job.stats[kStatsPerBlock b ...].
template <int KIND, int VARIANT, bool STATS = false>
__global__ void __launch_bounds__(256) split_kernel(const SplitJob job) {
  if (!gate_open(job.gate, job.gate_value)) return;
  SplitStats stats;
  if constexpr (VARIANT == kSplitRContiguousWide) {
    __shared__ float tile[32 * 256];
    split_block_r_contiguous_wide<KIND, STATS>(job, tile_of_block(job, blockIdx.x), tile, &stats);
  } else if constexpr (VARIANT == kSplitRContiguous) {
    split_block_r_contiguous<KIND, STATS>(job, blockIdx.x, &stats);
  } else {
    split_tiles_k_contiguous<KIND, VARIANT == kSplitKContiguousDeep ? kSplitDeepTiles : 1, STATS>(job, tile_of_block(job, blockIdx.x), &stats);
  }
  if constexpr (STATS) {
    __shared__ double sums[12];
    // (indexed by the launch's block number: the choice adds all blocks of an operand, in that order)
    store_block_stats(stats, job.stats + kStatsPerBlock * (size_t)blockIdx.x, sums);
  }
}

// Both operands of a product in one launch, for operands up to a size at which the second launch no longer shows: blocks
// 0 .. a.blocks - 1 split A, the rest split B.  DEEP: kSplitKContiguousDeep may be among the variants.
template <int KIND, bool DEEP, bool STATS = false>
__global__ void __launch_bounds__(256) split_pair_kernel(const SplitJob a, const SplitJob b) {
  if (!gate_open(a.gate, a.gate_value)) return;
  __shared__ float tile[32 * 256];
  const bool second = blockIdx.x >= a.blocks;  // block-uniform
  const SplitJob& job = second ? b : a;
  const unsigned block = second ? blockIdx.x - a.blocks : blockIdx.x;
  SplitStats stats;
  // (The order of the branches moves the measuring instance, whose code is larger than the instruction cache: automatic
  // mode, 1024 x 1024 x 16384 NN, wide beside deep, 163.4 us in this order, 164 to 168 in five others.)
  if (!STATS && job.variant == kSplitRContiguous) {  // (measured, not one of a pair)
    split_block_r_contiguous<KIND, STATS>(job, block, &stats);
  } else if (job.variant == kSplitKContiguous) {
    split_tiles_k_contiguous<KIND, 1, STATS>(job, tile_of_block(job, block), &stats);
  } else if (DEEP && job.variant == kSplitKContiguousDeep) {
    split_tiles_k_contiguous<KIND, kSplitDeepTiles, STATS>(job, tile_of_block(job, block), &stats);
  } else {
    split_block_r_contiguous_wide<KIND, STATS>(job, tile_of_block(job, block), tile, &stats);
  }
  if constexpr (STATS) {
    __shared__ double sums[12];
    store_block_stats(stats, job.stats + kStatsPerBlock * (size_t)block, sums);
  }
}

}  // namespace ecgemm
