// The one-launch arrangement (fused_kernel.hpp) for products of ordinary size in FP16 mode: steps 1 to 5 on the caller's
// FP32 operands in blocks of 128 x 128, one per compute unit.  It carries out a plan of the split-first kernels, the same
// tiles' elements over the same slices of the depth in the same order, and gives their bits; what it leaves out is the
// split pass and its trip through memory.
//
// One block: four waves that fetch and split, one per SIMD, and beside them four that multiply, 64 x 64 of the tile each
// (two accumulators of 2 x 2 matrix instructions: 128 registers of the 256 that two waves per SIMD leave each).  Depth is
// walked in chunks of 64 through two LDS buffers, one barrier per chunk, as in fused_kernel.hpp.  What a chunk costs, in
// cycles: a multiplying wave 48 matrix instructions, 1536; a splitting wave 64 values per lane at 3 vector instructions
// each next to them, 800 alone on its SIMD, and its 16 loads and 16 writes; the LDS 64 KiB of parts in and 128 KiB of
// fragments out, 1536 at 128 bytes per cycle.  Measured 1.41 us a chunk with all units busy (2048 x 2048, between 512 and
// 2048 deep), where the product kernels, which the chip's power limits, take 1.21 to 1.27 us for the same products and the
// split pass comes on top; 0.8 us on 100 units.  What brought it there from 1.75 us: no instruction in the loop that writes
// halves (FastSplit::split2), no test in it (below), buffer loads with constant offsets, registers refilled as they become
// free, the first conversion of a chunk in front of the barrier, priority for the multiplying waves (1 to 2 %).  Left out one
// at a time (2048 x 2048, us a chunk): the matrix instructions 1.08, the loads 1.25, loads and matrix instructions 0.86.
#pragma once
#include "fused_kernel.hpp"

namespace ecgemm {

constexpr int kWideTile = 128, kWideSplitWaves = 4, kWideThreads = 512;
constexpr int64_t kWideLargestLd = (int64_t)1 << 21;  // every value of a chunk lies well within 2^32 bytes of its first

struct WideParams {
  const float* A;  // device, column-major, as passed to ecgemm_sgemm
  const float* B;
  int64_t lda, ldb;      // at most kWideLargestLd
  int64_t M, N, K, ldc;  // M, N >= kWideTile, K >= 4
  int tiles_m, tiles_n;
  float alpha, beta;
  float* C;
  // slices > 1: a block takes one tile over one slice of the depth, slice_depth deep (the last one what is left, at least
  // 1), and leaves its sums, before alpha / beta, in partials[slice][tile][n][m] for reduce_tail_kernel
  int slices;
  int64_t slice_depth;
  float* partials;
};

// Where the eight values k = 8 octet .. + 7 of a row of the tile lie in an operand's region of LDS, part 0 (bytes):
// fragment order, [row / 32][k step][part] blocks of 1 KiB, each two halves (octet % 2) of 32 rows x 16 bytes.  The rows of
// a half are taken four apart (place_in_half), then rotated by the octet: the lanes of one write hold either rows four
// apart of one octet or the eight octets of one row, and go to different banks either way, while a fragment read takes
// a whole half.  The matrix instruction's row (or column) i is then row_at_place(i) of the 32.
__device__ __forceinline__ int place_in_half(int row) { return (row & 3) * 8 + (row >> 2); }
__device__ __forceinline__ int row_at_place(int place) { return 4 * (place & 7) + (place >> 3); }
template <int NP>
__device__ __forceinline__ int wide_lds_slot(int row_block, int place, int octet) {
  return (row_block * 4 + (octet >> 1)) * NP * 1024 + (octet & 1) * 512 + ((place + octet) & 31) * 16;
}

// One operand of the block.  A splitting thread t of 256 holds four units of a row and an octet each, in eight 16-byte
// loads at any multiple of four bytes:
//   !DEPTH (rows contiguous)   rows 4 (t % 32) + u, octet t / 32; load j is k = 8 octet + j of all four
//   DEPTH (depth contiguous)   rows t / 8 + 32 u, octet t % 8; loads 2 u and 2 u + 1 are the halves of unit u
template <int KIND, bool DEPTH>
struct WideOperand {
  static constexpr int NP = parts_of_split(KIND);
  static constexpr int REGION_BYTES = (kWideTile / 32) * 4 * NP * 1024;
  static_assert(KIND == kSplitFp16Scaled, "conversions that saturate (MODE.FP16_OVFL) stand in for Splitter's clamps");

  const float* tile;      // &X(first row of the tile, first k of the slice), the same for the block
  const float* lane_ptr;  // this lane's part of it: row 4 (t % 32) or t / 8, k = 0
  int64_t ld, K;          // K: depth of the slice
  unsigned lane_bytes;    // from the chunk's first value to this lane's first load
  int octet;
  int lds_offset[4];

  __device__ __forceinline__ void init(const float* first, int64_t ld_, int64_t K_, int t) {
    tile = first, ld = ld_, K = K_;
    octet = DEPTH ? t & 7 : t >> 5;
    const int row = DEPTH ? t >> 3 : 4 * (t & 31);
    lane_ptr = first + (DEPTH ? row * ld : (int64_t)row);
    lane_bytes = (unsigned)((DEPTH ? row * ld + 8 * octet : 8 * octet * ld + row) * 4);
#pragma unroll
    for (int u = 0; u < 4; ++u) {
      const int unit_row = DEPTH ? row + 32 * u : row + u;
      lds_offset[u] = wide_lds_slot<NP>(unit_row >> 5, place_in_half(unit_row & 31), octet);
    }
  }

  // Requests loads FIRST .. FIRST + COUNT - 1 of chunk c, which lies inside the depth: buffer loads, whose address is the
  // chunk's plus an offset per lane that never changes plus a scalar offset per load that does not either.
  template <int FIRST = 0, int COUNT = 8>
  __device__ __forceinline__ void fetch(source4_t (&x)[8], int c) const {
    const float* first = tile + (DEPTH ? (int64_t)c * 64 : (int64_t)c * 64 * ld);
    const auto buffer = __builtin_amdgcn_make_buffer_rsrc(const_cast<float*>(first), 0, -1, 0x00020000);
    const unsigned step = (unsigned)(DEPTH ? 128 * ld : 4 * ld);
#pragma unroll
    for (int j = FIRST; j < FIRST + COUNT; ++j)
      x[j] = __builtin_bit_cast(source4_t, __builtin_amdgcn_raw_buffer_load_b128(buffer, (int)(lane_bytes + (DEPTH ? (j & 1) * 16 : 0)), (int)((DEPTH ? (j >> 1) : j) * step), 0));
  }
  // The same for the chunk in which the depth ends: every address is inside the operand, complete() does the rest.
  __device__ __forceinline__ void fetch_last(source4_t (&x)[8], int c) {
    const int64_t k0 = (int64_t)c * 64 + 8 * octet;
#pragma unroll
    for (int j = 0; j < 8; ++j) {
      const int64_t k = k0 + (DEPTH ? 4 * (j & 1) : j), inside = DEPTH ? (k < K - 4 ? k : K - 4) : (k < K - 1 ? k : K - 1);
      x[j] = load_source4<false>(lane_ptr + (DEPTH ? (int64_t)(32 * (j >> 1)) * ld + inside : inside * ld));
    }
  }
  // k behind the depth counts as zero
  __device__ __forceinline__ void complete(source4_t (&x)[8], int c) const {
    const int64_t k0 = (int64_t)c * 64 + 8 * octet;
#pragma unroll
    for (int j = 0; j < 8; ++j) {
      const int64_t k = k0 + (DEPTH ? 4 * (j & 1) : j);
      if constexpr (DEPTH) {
        x[j] = shift_or_zero(x[j], k - (k < K - 4 ? k : K - 4));
      } else {
#pragma unroll
        for (int u = 0; u < 4; ++u) x[j][u] = k < K ? x[j][u] : 0.0f;
      }
    }
  }

  __device__ __forceinline__ static float value(const source4_t (&x)[8], int u, int e) { return DEPTH ? x[2 * u + (e >> 2)][e & 3] : x[e][u]; }

  typedef unsigned uint4_t __attribute__((ext_vector_type(4)));
  // The parts of unit u, by the short split without a test for the values it does not take: see wide_kernel.
  __device__ __forceinline__ static void convert(const source4_t (&x)[8], int u, uint4_t (&parts)[NP]) {
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      const float v0 = value(x, u, 2 * e), v1 = value(x, u, 2 * e + 1);
      unsigned words[NP];
      FastSplit<KIND>::split2(v0, v1, v0 * 2048.0f, v1 * 2048.0f, words);
#pragma unroll
      for (int q = 0; q < NP; ++q) parts[q][e] = words[q];
    }
  }
  __device__ __forceinline__ void write(const uint4_t (&parts)[NP], int u, char* region) const {
#pragma unroll
    for (int q = 0; q < NP; ++q) *reinterpret_cast<uint4_t*>(region + lds_offset[u] + q * 1024) = parts[q];
  }
  // Splits units FIRST .. 3 and writes their parts to `region`.  REFILL: chunk `next`, which lies inside the depth, is
  // requested into the registers as they become free (those of the units before FIRST at once).
  template <bool REFILL, int FIRST>
  __device__ __forceinline__ void deposit(source4_t (&x)[8], char* region, int next) const {
    if constexpr (REFILL && DEPTH && FIRST > 0) {
      fetch<0, 2 * FIRST>(x, next);
      __builtin_amdgcn_sched_barrier(0);
    }
    static_for<4 - FIRST>([&](auto u_c) {
      constexpr int u = FIRST + decltype(u_c)::value;
      uint4_t parts[NP];
      convert(x, u, parts);
      write(parts, u, region);
      if constexpr (REFILL && DEPTH) {
        __builtin_amdgcn_sched_barrier(0);
        fetch<2 * u, 2>(x, next);
        __builtin_amdgcn_sched_barrier(0);
      }
    });
    if constexpr (REFILL && !DEPTH) {
      __builtin_amdgcn_sched_barrier(0);
      fetch(x, next);
      __builtin_amdgcn_sched_barrier(0);
    }
  }
  // The same for any value: unit by unit, the short split where no lane of the wave holds one that it does not take.
  // (2048^3 NT with one NaN, 16 of whose 256 blocks go through the depth again, 170 us with Splitter throughout / 111; with a
  // million of them, every block, 167 / 147; 1024 x 1024 x 65536 NT 900 / 660 and 1460 / 1290.)
  __device__ __forceinline__ void deposit_with_care(const source4_t (&x)[8], char* region) const {
    static_for<4>([&](auto u_c) {
      constexpr int u = decltype(u_c)::value;
      uint4_t parts[NP];
      convert(x, u, parts);
      float largest = 0.0f;
#pragma unroll
      for (int e = 0; e < 4; ++e) FastSplit<KIND>::raise(largest, value(x, u, 2 * e), value(x, u, 2 * e + 1));
      if (__builtin_amdgcn_ballot_w64(!(largest <= 0x1p116f)) != 0) {
#pragma unroll
        for (int e = 0; e < 4; ++e) {
          unsigned short even[NP], odd[NP];
          Splitter<KIND>::split(value(x, u, 2 * e), even);
          Splitter<KIND>::split(value(x, u, 2 * e + 1), odd);
#pragma unroll
          for (int q = 0; q < NP; ++q) parts[q][e] = (unsigned)even[q] | ((unsigned)odd[q] << 16);
        }
      }
      write(parts, u, region);
      __builtin_amdgcn_sched_barrier(0);
    });
  }
};

template <int METHOD, bool DEPTH_A, bool DEPTH_B>
__global__ void __launch_bounds__(kWideThreads, 1) wide_kernel(const WideParams p) {
  constexpr int KIND = split_kind_of(METHOD), NP = parts_of_split(KIND), PRODUCTS = products_of(METHOD), ELEM = element_kind_of(METHOD);
  typedef WideOperand<KIND, DEPTH_A> OperandA;
  typedef WideOperand<KIND, DEPTH_B> OperandB;
  constexpr int REGION_BYTES = OperandA::REGION_BYTES, STAGE_BYTES = 2 * REGION_BYTES;
  typedef typename Mfma<ELEM>::frag_t frag_t;
  __shared__ __attribute__((aligned(1024))) char lds[2 * STAGE_BYTES + 4 * sizeof(int)];
  int* not_finite = reinterpret_cast<int*>(lds + 2 * STAGE_BYTES);  // one word per multiplying wave

  const int t = threadIdx.x, lane = t & 63;
  const int wave = __builtin_amdgcn_readfirstlane(t >> 6);
  // each XCD takes a contiguous run of the tiles, whose patch shares rows of A and columns of B in its L2
  const int tiles = p.tiles_m * p.tiles_n, position = (int)xcd_run_position(blockIdx.x, gridDim.x);
  const int slice = position / tiles, tile_index = position - slice * tiles;
  int tile_m, tile_n;
  tile_coordinates(tile_index, p.tiles_m, p.tiles_n, 4, 1, tile_m, tile_n);
  // (a last tile that is not whole is moved back to be whole and stores what is its own)
  const int64_t m_tile = (int64_t)tile_m * kWideTile, n_tile = (int64_t)tile_n * kWideTile;
  const int64_t m0 = m_tile < p.M - kWideTile ? m_tile : p.M - kWideTile, n0 = n_tile < p.N - kWideTile ? n_tile : p.N - kWideTile;
  const int64_t k_begin = slice * p.slice_depth;
  const int64_t K = p.slices == 1 ? p.K : p.K - k_begin < p.slice_depth ? p.K - k_begin : p.slice_depth;
  const int chunks = (int)((K + 63) / 64);  // >= 1

  auto block_barrier = [&]() {
    __builtin_amdgcn_sched_barrier(0);
    asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
    __builtin_amdgcn_s_barrier();
    asm volatile("" ::: "memory");
    __builtin_amdgcn_sched_barrier(0);
  };

  // Every wave passes `chunks` barriers: a splitting wave one after each chunk it has written, a multiplying wave one
  // before each chunk it reads, having read the chunk before it to the end.  Chunk c lives in buffer c % 2.
  //
  // The short split takes every value up to 2^116: its conversions run with the mode bit that makes an overflow the
  // largest finite number, which is what Splitter's clamps do.  What it does not take, infinities, NaN and values for
  // which the scaled one overflows FP32, leaves an infinity or a NaN among the parts, and with it in every element of the
  // row or column of the tile.  So nothing is tested in the loop; a block whose sums are not all finite goes through the
  // depth once more, with a test and with Splitter where it takes one.
  if (wave < kWideSplitWaves) {
    OperandA a;
    OperandB b;
    a.init(p.A + (DEPTH_A ? m0 * p.lda + k_begin : m0 + k_begin * p.lda), p.lda, K, t);
    b.init(p.B + (DEPTH_B ? n0 * p.ldb + k_begin : n0 + k_begin * p.ldb), p.ldb, K, t);
    const int whole = (int)(K / 64);
    __builtin_amdgcn_s_setreg(1 | (23 << 6), 1);  // MODE.FP16_OVFL
    source4_t xa[2][8], xb[2][8];
    auto request = [&](auto r_c, int c) {
      constexpr int r = decltype(r_c)::value;
      if (c < whole) a.fetch(xa[r], c), b.fetch(xb[r], c);
      else if (c < chunks) a.fetch_last(xa[r], c), b.fetch_last(xb[r], c);
    };
    request(std::integral_constant<int, 0>{}, 0);
    __builtin_amdgcn_sched_barrier(0);
    request(std::integral_constant<int, 1>{}, 1);
    __builtin_amdgcn_sched_barrier(0);
    int c = 0;
    // The bulk of the depth: chunks that lie inside it, and so do those requested behind them (no condition at a load).
    // The first unit of a chunk is converted in front of the barrier that lets it be written, while the writes before it
    // are on their way.
    typename OperandA::uint4_t ahead[NP];
    if (c + 4 <= whole) OperandA::convert(xa[0], 0, ahead);
    for (; c + 4 <= whole; c += 2) {
      static_for<2>([&](auto r_c) {
        constexpr int r = decltype(r_c)::value;
        a.write(ahead, 0, lds + r * STAGE_BYTES);
        a.template deposit<true, 1>(xa[r], lds + r * STAGE_BYTES, c + r + 2);
        b.template deposit<true, 0>(xb[r], lds + r * STAGE_BYTES + REGION_BYTES, c + r + 2);
        OperandA::convert(xa[r ^ 1], 0, ahead);
        block_barrier();
      });
    }
    for (; c < chunks; c += 2) {
      static_for<2>([&](auto r_c) {
        constexpr int r = decltype(r_c)::value;
        if (c + r < chunks) {
          if (c + r >= whole) a.complete(xa[r], c + r), b.complete(xb[r], c + r);
          a.template deposit<false, 0>(xa[r], lds + r * STAGE_BYTES, 0);
          b.template deposit<false, 0>(xb[r], lds + r * STAGE_BYTES + REGION_BYTES, 0);
          __builtin_amdgcn_sched_barrier(0);
          request(r_c, c + r + 2);
          block_barrier();
        }
      });
    }
    block_barrier();  // the multiplying waves' words are there
    if ((not_finite[0] | not_finite[1] | not_finite[2] | not_finite[3]) == 0) return;
    for (c = 0; c < chunks; ++c) {
      char* stage = lds + (c & 1) * STAGE_BYTES;
      a.fetch_last(xa[0], c), b.fetch_last(xb[0], c);
      a.complete(xa[0], c), b.complete(xb[0], c);
      a.deposit_with_care(xa[0], stage);
      b.deposit_with_care(xb[0], stage + REGION_BYTES);
      block_barrier();
    }
    return;
  }

  // ---- multiplying waves: rows wave_m 64 .. + 63 and columns wave_n 64 .. + 63 of the tile
  __builtin_amdgcn_s_setprio(2);  // (what is free beside them is the splitting waves')
  const int wave_m = wave & 1, wave_n = (wave >> 1) & 1;
  float16_t acc_main[2][2], acc_corr[2][2];
  int lane_off[4];  // of this lane's 16 bytes within a 1 KiB block of k step ks
#pragma unroll
  for (int ks = 0; ks < 4; ++ks) lane_off[ks] = wide_lds_slot<NP>(0, lane & 31, 2 * ks + (lane >> 5));
  // Fragments of a k step in the order in which its matrix instructions first need them, two sets: one is read while the
  // other is multiplied.
  frag_t fa[2][2][NP], fb[2][2][NP];
  constexpr int READS = 4 * NP, MFMAS = 4 * PRODUCTS;
  auto read_fragment = [&](auto set_c, auto r_c, const char* stage, int off) {
    constexpr int set = decltype(set_c)::value, r = decltype(r_c)::value, part = r / 4, which = r % 4;  // a0 b0 b1 a1 of part 0, b0 b1 a0 a1 of part 1
    constexpr bool from_b = part == 0 ? (which == 1 || which == 2) : which < 2;
    constexpr int index = part == 0 ? (which >= 2 ? 1 : 0) : which & 1;
    if constexpr (from_b)
      fb[set][index][part] = *reinterpret_cast<const frag_t*>(stage + REGION_BYTES + (wave_n * 2 + index) * 4 * NP * 1024 + part * 1024 + off);
    else
      fa[set][index][part] = *reinterpret_cast<const frag_t*>(stage + (wave_m * 2 + index) * 4 * NP * 1024 + part * 1024 + off);
  };
  // Multiplies set SET, term by term over the four 32 x 32 blocks (neighbours never share an accumulator), and reads the
  // other set behind its first instructions.
  auto step = [&](auto set_c, const char* stage, int off) {
    constexpr int SET = decltype(set_c)::value;
    static_for<MFMAS>([&](auto m_c) {
      constexpr int m = decltype(m_c)::value;
      constexpr ProductTerm term = product_term(METHOD, m / 4);
      constexpr int i = (m % 4) / 2, j = m % 2;
      if constexpr (term.correction)
        acc_corr[i][j] = Mfma<ELEM>::run(fb[SET][j][term.qb], fa[SET][i][term.qa], acc_corr[i][j]);
      else
        acc_main[i][j] = Mfma<ELEM>::run(fb[SET][j][term.qb], fa[SET][i][term.qa], acc_main[i][j]);
      if constexpr (m < READS) read_fragment(std::integral_constant<int, SET ^ 1>{}, m_c, stage, off);
      __builtin_amdgcn_sched_barrier(0);
    });
  };
  typedef std::integral_constant<int, 0> set0_t;
  typedef std::integral_constant<int, 1> set1_t;
  for (int pass = 0;; ++pass) {
#pragma unroll
    for (int i = 0; i < 2; ++i)
#pragma unroll
      for (int j = 0; j < 2; ++j)
#pragma unroll
        for (int v = 0; v < 16; ++v) acc_main[i][j][v] = 0.0f, acc_corr[i][j][v] = 0.0f;
    block_barrier();  // chunk 0 is there
    static_for<READS>([&](auto r_c) { read_fragment(set0_t{}, r_c, lds, lane_off[0]); });
    auto chunk_and_next = [&](const char* stage, const char* next) {
      step(set0_t{}, stage, lane_off[1]);
      step(set1_t{}, stage, lane_off[2]);
      step(set0_t{}, stage, lane_off[3]);
      block_barrier();  // this chunk has been read to the end, the next one is there
      step(set1_t{}, next, lane_off[0]);
    };
    int left = chunks - 1;  // chunks to multiply before the last one
    for (; left >= 2; left -= 2) {  // (two at a time: a jump leaves the matrix pipe idle for three instructions)
      chunk_and_next(lds, lds + STAGE_BYTES);
      chunk_and_next(lds + STAGE_BYTES, lds);
    }
    if (left == 1) chunk_and_next(lds, lds + STAGE_BYTES);
    const int buffer = ((chunks - 1) & 1) * STAGE_BYTES;  // of the last chunk
    step(set0_t{}, lds + buffer, lane_off[1]);
    step(set1_t{}, lds + buffer, lane_off[2]);
    step(set0_t{}, lds + buffer, lane_off[3]);
    step(set1_t{}, lds + buffer, lane_off[0]);  // (what it reads is not used)
    // main + correction, in the accumulators of the leading product
    float largest = 0.0f;
#pragma unroll
    for (int i = 0; i < 2; ++i)
#pragma unroll
      for (int j = 0; j < 2; ++j)
#pragma unroll
        for (int v = 0; v < 16; ++v) {
          acc_main[i][j][v] = acc_main[i][j][v] + acc_corr[i][j][v] * 0x1p-11f;  // (the residuals carry 2^11)
          largest = __builtin_elementwise_maximum(largest, __builtin_fabsf(acc_main[i][j][v]));
        }
    if (pass == 1) break;
    const bool redo = __builtin_amdgcn_ballot_w64(!(largest <= 3.402823466e+38f)) != 0;
    if (lane == 0) not_finite[wave - kWideSplitWaves] = redo;
    block_barrier();
    if ((not_finite[0] | not_finite[1] | not_finite[2] | not_finite[3]) == 0) break;  // the same for the block
  }

  // ---- epilogue, as in product_kernel: a lane owns one row per 32 x 32 block; register v of it is the matrix
  // instruction's column 8 (v / 4) + 4 (lane / 32) + v % 4
  const int tile_row = wave_m * 64 + row_at_place(lane & 31);
  auto tile_column = [&](int j, int v) { return wave_n * 64 + j * 32 + row_at_place(8 * (v / 4) + 4 * (lane >> 5) + v % 4); };
  float* partial = p.slices > 1 ? p.partials + ((int64_t)slice * tiles + tile_index) * (kWideTile * kWideTile) : nullptr;
  const int m_skip = (int)(m_tile - m0), n_skip = (int)(n_tile - n0);  // rows and columns of the moved tile that are its neighbour's
#pragma unroll
  for (int i = 0; i < 2; ++i) {
    const int row = tile_row + i * 32;
#pragma unroll
    for (int j = 0; j < 2; ++j) {
      float c[16];
#pragma unroll
      for (int v = 0; v < 16; ++v) c[v] = acc_main[i][j][v];
      if (row < m_skip) continue;
      auto store_all = [&](auto whole_c) {  // whole: the tile is nobody else's (the same for the block)
        constexpr bool whole = decltype(whole_c)::value;
        if (partial != nullptr) {
#pragma unroll
          for (int v = 0; v < 16; ++v)
            if (whole || tile_column(j, v) >= n_skip) store_partial(partial + (tile_column(j, v) - n_skip) * kWideTile + (row - m_skip), c[v]);
          return;
        }
        float* dst = p.C + (m0 + row) + n0 * p.ldc;
        if (p.beta != 0.0f) {
          float c_in[16];
#pragma unroll
          for (int v = 0; v < 16; ++v) c_in[v] = whole || tile_column(j, v) >= n_skip ? load_global(dst + tile_column(j, v) * p.ldc) : 0.0f;
#pragma unroll
          for (int v = 0; v < 16; ++v)
            if (whole || tile_column(j, v) >= n_skip) store_result(dst + tile_column(j, v) * p.ldc, scaled_sum(p.alpha, c[v], p.beta, c_in[v]));
        } else {
#pragma unroll
          for (int v = 0; v < 16; ++v)
            if (whole || tile_column(j, v) >= n_skip) store_result(dst + tile_column(j, v) * p.ldc, p.alpha * c[v]);
        }
      };
      if (n_skip == 0) store_all(std::true_type{});
      else store_all(std::false_type{});
    }
  }
}

}  // namespace ecgemm
