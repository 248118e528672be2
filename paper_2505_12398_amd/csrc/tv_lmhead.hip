// LM head with fused row statistics for gfx950: logits = hidden * weight^T on
// bf16 MFMA, rounded to bf16, and in the same kernel the statistics of every
// row of the rounded logits that the verifier's tempered softmax needs (the
// row maximum and the sum of exp((z - max) / T)), so that no pass over the
// logits is needed to compute them (the distributions M_b and M_s of the
// problem statement, Alg. 3 REQUIRE, are softmax(logits / T) per row).
//
// What bounds it. Many rows: the matrix cores, and behind them the card's
// power limit. Under products of random bf16 values the clock falls below
// 2.0 GHz, so energy per product counts, not only issue slots. On register
// operands of normal values v_mfma_f32_16x16x32_bf16 reaches 2.03 PFLOP/s where
// v_mfma_f32_32x32x16_bf16 reaches 1.77 (same card; its accumulators move twice
// as often per product; with zeros or ones both reach 2.42), hence 16 x 16
// blocks; loads straight into LDS save the passage through registers. Few rows:
// the one read of the weight from HBM.
//
// Tiling. A workgroup of 4 wavefronts (2 x 2, one per SIMD) computes a
// 32 MB x 256 tile of logits, each wavefront 16 MB x 128 of it as MB x 8
// blocks of 16 x 16. K advances 64 at a time through a ring of LDS slices
// filled by buffer loads that write LDS directly. A slice row is 128 bytes in
// eight 16-byte chunks, chunk c of row r at position c ^ ((r >> 1) & 7): a
// load instruction still fetches whole 128-byte lines, and the sixteen lanes
// that read one chunk of sixteen rows touch sixteen different bank groups.
// Both operands are K-contiguous (hidden [M][K], weight [N][K]), so an MFMA
// operand is one 16-byte LDS read. The weight is the first operand: a lane
// then holds four consecutive columns of one logits row.
//
// The workgroups are persistent and the ring runs on across tiles: while a
// tile's last products are formed, the next tile's first slices are loaded,
// and they land during the epilogue.
//
// Epilogue, in registers: accumulators are rounded to bf16 (round to nearest
// even, by the hardware conversion); lanes exchange halves so that each stores
// 16 bytes; each row's maximum and sum of 2^((z - max) k), k = log2(e)/T, in
// fp32, are reduced over the four lanes and two wavefronts that hold the row:
// one (max, sum) partial per row and column tile (per column range where there
// is one row of tiles, its tiles' sums added in fp64). A second kernel merges a
// row's partials in fp64, each moved to the frame of the row maximum.
#include <hip/hip_runtime.h>
#include <math.h>
#include <stdint.h>

#include <mutex>
#include <type_traits>
#include <utility>

#include "tv.h"
#include "tv_launch.h"

namespace {

constexpr int kBN = tv::kLmheadTileN, kBK = 64;
constexpr int kNB = kBN / 32;             // 16-column blocks per wavefront
constexpr int kThreads = 256;
constexpr int kRowBytes = kBK * 2;        // one row of a slice
constexpr int kLdsBytes = 160 * 1024;     // LDS of a CU
constexpr int kXcds = 8;
constexpr size_t kLastLevelCache = size_t{256} << 20;
constexpr int kGroupN = 8;                // column tiles per group of the tile order
static_assert(kBN == 256 && kRowBytes == 128, "the chunk positions and the wave layout assume these");

typedef __attribute__((ext_vector_type(8))) __bf16 bf16x8;
typedef __attribute__((ext_vector_type(4))) float f32x4;
typedef __attribute__((ext_vector_type(4))) int i32x4;
typedef __attribute__((ext_vector_type(4))) unsigned u32x4;
typedef __attribute__((address_space(3))) uint8_t lds_byte;

struct LmParams {
  const uint16_t* x;      // [M][K] bf16 bits
  const uint16_t* w;      // [N][K] bf16 bits
  uint16_t* logits;       // [M][N] bf16 bits
  float* part_max;        // [M][parts]
  float* part_sum;        // [M][parts], in the frame of part_max
  float* row_max;         // [M]
  double* row_sum;        // [M]
  int M, K, N, tiles_m, tiles_n;
  int per_xcd;            // workgroups per XCD
  int parts;              // partials per row: tiles_n, or the column ranges of a single row of tiles
  float k32;              // log2(e) / T rounded to fp32
};

// LDS slices a tile height has room for. A slice must be complete one
// 32-deep step before its products start, and a buffer is refilled as soon as
// its last fragments are read, so two buffers keep a slice in flight; tiles of
// up to 160 rows, which read the weight faster than they multiply, have three
// or four (72 to 108 KB in flight per CU).
constexpr int slice_bytes(int mb) { return (32 * mb + kBN) * kRowBytes; }
// per row the right half's (max, sum), and a range's (max, fp64 sum) so far
constexpr int merge_bytes(int mb) { return 32 * mb * (8 + 4 + 8); }
constexpr int stages(int mb) {
  const int s = (kLdsBytes - merge_bytes(mb)) / slice_bytes(mb);
  return s < 4 ? s : 4;
}

// Tile i of the launch's order: groups of kGroupN column tiles, in a group row
// by row. The 32 tiles an XCD runs at once are then four rows by eight columns
// that share their slices through its L2, and all XCDs read the same eight
// column tiles of the weight at about the same time, where the last-level cache
// can serve all but the first. (With each XCD on a contiguous eighth of all
// tiles, the XCDs sat at different columns: 13.8 against 12.5 ms at 16640 x
// 4096 x 128256; groups of 4 or 16 columns 13.1 and 12.2 against 12.1 ms. What
// leaves the L2s is the same, 32 GB read; no counter here tells the last-level
// cache's part of it from the memory's.)
__device__ __forceinline__ void tile_at(const LmParams& P, int i, int& tm, int& tn) {
  const int per = kGroupN * P.tiles_m;
  const int g = i / per, in = i - g * per;
  const int w = min(kGroupN, P.tiles_n - kGroupN * g);
  tm = in / w;
  tn = kGroupN * g + in - tm * w;
}

// A single row of tiles: workgroup i takes the columns [range_start(i),
// range_start(i + 1)), multiples of 8 but for the end. Against whole tiles dealt
// out, every CU has the same share of the weight, and the ranges' rows, often a
// power of two of bytes apart, start at odd multiples of that: tiles of 256 rows
// each had all CUs wait for the same memory channels (65 x 4096 x 128256: 245
// against 188 us).
__device__ __forceinline__ int range_start(const LmParams& P, int i) {
  const long long n8 = (P.N + 7) / 8;
  return min(P.N, 8 * static_cast<int>(n8 * i / P.parts));
}

// acc += a * b. Written in assembly with the accumulator tied to its
// registers: left to the compiler, a loop that fills all 256 accumulation
// registers is allocated with copies around half of its products. Its inputs
// come from LDS reads, whose waits the compiler inserts for assembly as for
// any reader; the accumulators are settled by settle() before other
// instructions touch them.
__device__ __forceinline__ void mfma(f32x4& acc, const bf16x8& a, const bf16x8& b) {
  asm volatile("v_mfma_f32_16x16x32_bf16 %0, %1, %2, %0" : "+a"(acc) : "v"(a), "v"(b));
}

// f(0), ..., f(N - 1) with constant arguments (fully unrolled whatever the size)
template <class F, int... I>
__device__ __forceinline__ void unrolled(F&& f, std::integer_sequence<int, I...>) {
  (f(std::integral_constant<int, I>{}), ...);
}
template <int N, class F>
__device__ __forceinline__ void unrolled(F&& f) {
  unrolled(f, std::make_integer_sequence<int, N>{});
}

// f(i) for the i < N whose turn comes at slot J, when N things are spread
// evenly over SLOTS slots: those with i * SLOTS / N == J
constexpr int turn(int j, int n, int slots) { return (j * n + slots - 1) / slots; }
template <int J, int N, int SLOTS, class F>
__device__ __forceinline__ void at_slot(F&& f) {
  if constexpr (J >= 0 && J < SLOTS) {
    constexpr int i0 = turn(J, N, SLOTS), i1 = turn(J + 1, N, SLOTS);
    unrolled<i1 - i0>([&](auto i) { f(std::integral_constant<int, i0 + i.value>{}); });
  }
}

// Wait states between vector writes or reads of accumulators and the products:
// at most 18 for a product's result (8 passes), 2 before one reads.
__device__ __forceinline__ void settle(f32x4 (&a)[8]) {
  asm volatile("s_nop 15\n\ts_nop 7"
               : "+a"(a[0]), "+a"(a[1]), "+a"(a[2]), "+a"(a[3]), "+a"(a[4]), "+a"(a[5]),
                 "+a"(a[6]), "+a"(a[7]));
}

// Keeps what is computed from a row of blocks behind this point.
__device__ __forceinline__ void pin(f32x4 (&a)[8]) {
  asm volatile("" : "+a"(a[0]), "+a"(a[1]), "+a"(a[2]), "+a"(a[3]), "+a"(a[4]), "+a"(a[5]),
                    "+a"(a[6]), "+a"(a[7]));
}

// 64 lanes' 16 bytes from the buffer `rs` at byte offsets voff + soff into LDS
// at dst + 16 * lane. A voff past the buffer's range writes zeros. kOnce: with
// the non-temporal hint, for data that no one reads again. m0 is reserved, which
// the compiler warns of; declared, it is set again by whoever else uses it.
// The hazard recogniser does not look into assembly. The wait state between m0
// and the load is here. The five between a scalar that the vector unit wrote (a
// spilled one read back) and a load that reads it are not (with them 13.85 ms
// against 13.4 at 16640 x 4096 x 128256): in the build such a scalar is read
// much later, and a test of the generated code holds that, as it does the two
// states between a vector write and the product that reads it (mfma above).
#pragma clang diagnostic push
#pragma clang diagnostic ignored "-Winline-asm"
template <bool kOnce>
__device__ __forceinline__ void load_to_lds(const i32x4& rs, int voff, int soff, int dst) {
  if constexpr (kOnce)
    asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tbuffer_load_dwordx4 %1, %2, %3 offen nt lds"
                 :: "s"(dst), "v"(voff), "s"(rs), "s"(soff) : "memory", "m0");
  else
    asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tbuffer_load_dwordx4 %1, %2, %3 offen lds"
                 :: "s"(dst), "v"(voff), "s"(rs), "s"(soff) : "memory", "m0");
}
#pragma clang diagnostic pop

constexpr int kPastRange = 0x40000000;   // more than any tile's bytes (256 rows of 2^16 bf16)

// bf16 rounding of two accumulators into one word (v_cvt_pk_bf16_f32)
__device__ __forceinline__ uint32_t pack2(float lo, float hi) {
  return static_cast<uint32_t>(__builtin_bit_cast(uint16_t, static_cast<__bf16>(lo))) |
         static_cast<uint32_t>(__builtin_bit_cast(uint16_t, static_cast<__bf16>(hi))) << 16;
}

// the largest of three (in assembly: fmaxf would first quiet each operand)
__device__ __forceinline__ float max3(float a, float b, float c) {
  float r;
  asm("v_max3_f32 %0, %1, %2, %3" : "=v"(r) : "v"(a), "v"(b), "v"(c));
  return r;
}

// (m, s) merged with (m2, s2): maxima and sums in the frames of their maxima (0
// where there is no finite value). A frame is the product -m k rounded to fp32,
// as the sum's terms were formed in it, so the products are rounded before they
// are subtracted: contracted into an fma, the side that holds the maximum would
// move by the rounding of its own frame, 2^-24 |m| k (T = 0.001: sums 1e-3 off).
__device__ __forceinline__ void merge_stats(float& m, float& s, float m2, float s2, float k) {
#pragma clang fp contract(off)
  const float top = fmaxf(m, m2);
  const float c = top > -INFINITY ? -top * k : 0.0f;
  const float f = m > -INFINITY ? __builtin_amdgcn_exp2f(c - -m * k) : 1.0f;
  const float f2 = m2 > -INFINITY ? __builtin_amdgcn_exp2f(c - -m2 * k) : 1.0f;
  s = s * f + s2 * f2;
  m = top;
}

// the sum s in the frame of m, moved to the frame of top >= m (as it is where
// there is no finite value: 0 or NaN)
__device__ __forceinline__ double moved(double s, float m, float top, float k) {
  return m > -INFINITY
             ? s * exp2(static_cast<double>(-top * k) - static_cast<double>(-m * k))
             : s;
}

template <int MB, bool kRange, bool kOnce>
__global__ void __launch_bounds__(kThreads, 1) lmhead_kernel(LmParams P) {
  constexpr int S = stages(MB);
  constexpr int kBM = 32 * MB;
  constexpr int kXBytes = kBM * kRowBytes;          // hidden rows of a slice, then the weight's
  constexpr int kSlice = slice_bytes(MB);
  constexpr int kLoads = MB + kNB;                  // load instructions per slice and wavefront
  constexpr int kProds = MB * kNB;                  // products per 32-deep step
  static_assert(S >= 2, "two slices");
  __shared__ __attribute__((aligned(1024))) uint8_t smem[S * kSlice + merge_bytes(MB)];
  lds_byte* const lds = (lds_byte*)smem;
  const int lds0 = static_cast<int>(reinterpret_cast<uintptr_t>(lds));
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int wm = wave >> 1, wn = wave & 1;
  const int nk = (P.K + kBK - 1) / kBK;
  // Workgroups are dealt to the XCDs in turn, and each XCD has per_xcd
  // consecutive ones: in every round of tiles, or of the ranges.
  const int wg = static_cast<int>(blockIdx.x % kXcds) * P.per_xcd +
                 static_cast<int>(blockIdx.x / kXcds);
  const int r0 = kRange ? range_start(P, wg) : 0, r1 = kRange ? range_start(P, wg + 1) : 0;
  const int ntiles = kRange ? (r1 - r0 + kBN - 1) / kBN : P.tiles_m * P.tiles_n;
  const int step = kRange ? 1 : kXcds * P.per_xcd;
  int t = kRange ? 0 : wg;
  if (kRange ? wg >= P.parts || r0 >= r1 : t >= ntiles) return;
  // first row, first column and columns of tile i
  auto tile = [&](int i, int& m0, int& n0, int& nw) {
    if constexpr (kRange) {
      m0 = 0;
      n0 = r0 + kBN * i;
      nw = min(kBN, r1 - n0);
    } else {
      int tm, tn;
      tile_at(P, i, tm, tn);
      m0 = tm * kBM;
      n0 = tn * kBN;
      nw = min(kBN, P.N - n0);
    }
  };

  // Loads. Instruction q of this wavefront fills eight rows of the slice: lane
  // l row l / 8, position l % 8. Rows past the matrix read its last row
  // (their results are not stored); chunks past the last column read zeros.
  const int lrow = lane >> 3, lpos = lane & 7;
  int vx[MB], vw[kNB];
  i32x4 rx, rw;
  // Chunks past the last column: before the last slice of a tile is loaded
  // their offsets go past the range. (A bit set per load, in every slice, took
  // 13.0 against 12.5 ms at 16640 x 4096 x 128256.)
  const bool ragged = P.K % kBK != 0;
  auto mask_last = [&]() {
    asm volatile("" : "+v"(vx[0]));   // a branch of its own, not selects in every slice
#pragma unroll
    for (int o = 0; o < 2; ++o) {     // groups of eight rows, even and odd
      const int col = 8 * (lpos ^ (4 * o + (lrow >> 1)));
      const int past = (nk - 1) * kBK + col >= P.K ? kPastRange : 0;
#pragma unroll
      for (int q = 0; q < MB; ++q)
        if (((MB * wave + q) & 1) == o) vx[q] |= past;
#pragma unroll
      for (int q = o; q < kNB; q += 2) vw[q] |= past;
    }
  };
  auto load_tile = [&](int i) {
    int m0, n0, nw;
    tile(i, m0, n0, nw);
    const int nx = min(kBM, P.M - m0);
#pragma unroll
    for (int q = 0; q < MB; ++q) {
      const int g = MB * wave + q;    // group of eight rows
      const int col = 8 * (lpos ^ (4 * (g & 1) + (lrow >> 1)));
      vx[q] = (min(8 * g + lrow, nx - 1) * P.K + col) * 2;
    }
#pragma unroll
    for (int q = 0; q < kNB; ++q) {
      const int col = 8 * (lpos ^ (4 * (q & 1) + (lrow >> 1)));
      vw[q] = (min(8 * (kNB * wave + q) + lrow, nw - 1) * P.K + col) * 2;
    }
    const uint64_t bx = reinterpret_cast<uint64_t>(P.x + static_cast<size_t>(m0) * P.K);
    const uint64_t bw = reinterpret_cast<uint64_t>(P.w + static_cast<size_t>(n0) * P.K);
    rx = i32x4{static_cast<int>(bx), static_cast<int>(bx >> 32) & 0xffff, nx * P.K * 2, 0x00020000};
    rw = i32x4{static_cast<int>(bw), static_cast<int>(bw >> 32) & 0xffff, nw * P.K * 2, 0x00020000};
  };
  load_tile(t);
  int lt = t, lk = 0, lbuf = 0;       // tile, slice and LDS buffer to load next
  if (ragged && nk == 1) mask_last();
  auto load_i = [&](auto c) {         // load instruction c of the slice
    constexpr int i = c.value;
    const int soff = lk * kRowBytes;
    if constexpr (i < kNB)
      load_to_lds<kOnce>(rw, vw[i], soff, lds0 + lbuf * kSlice + kXBytes + (kNB * wave + i) * 1024);
    else
      load_to_lds<false>(rx, vx[i - kNB], soff,
                         lds0 + lbuf * kSlice + (MB * wave + i - kNB) * 1024);
  };
  auto load_next = [&]() {            // on to the next slice (of this workgroup's next tile)
    lbuf = lbuf + 1 == S ? 0 : lbuf + 1;
    if (++lk == nk) {
      lk = 0;
      lt += step;
      if (lt < ntiles) {
        load_tile(lt);
      } else {                        // nothing left: every load is past the range
        rx[2] = 0;
        rw[2] = 0;
      }
    }
    if (ragged && lk == nk - 1) mask_last();
  };
  for (int s = 0; s < S; ++s) {
    unrolled<kLoads>(load_i);
    load_next();
  }
  // Slice 0 complete. (Loads complete in order: all but the later slices'.)
  asm volatile("s_waitcnt vmcnt(%0)\n\ts_barrier" :: "n"((S - 1) * kLoads) : "memory");

  // Fragments: lane l reads row l % 16 of a block, chunk l / 16 of the step.
  const int fr = lane & 15, fg = lane >> 4;
  const int fpos = (fg ^ ((fr >> 1) & 7)) * 16;
  const int fx0 = (wm * 16 * MB + fr) * kRowBytes + fpos;
  const int fw0 = kXBytes + (wn * 16 * kNB + fr) * kRowBytes + fpos;
  bf16x8 fx[2][MB], fw[2][kNB];
  // fragment i of a step, the weight's first; step 1's chunks are 4 further,
  // so their positions differ in bit 2
  auto read_i = [&](auto st, auto c, int buf) {
    constexpr int step = st.value, i = c.value;
    const int base = buf * kSlice;
    if constexpr (i < kNB)
      fw[step][i] = __builtin_bit_cast(
          bf16x8, *(const __attribute__((address_space(3))) i32x4*)(
                      lds + (fw0 ^ (64 * step)) + base + i * 16 * kRowBytes));
    else
      fx[step][i - kNB] = __builtin_bit_cast(
          bf16x8, *(const __attribute__((address_space(3))) i32x4*)(
                      lds + (fx0 ^ (64 * step)) + base + (i - kNB) * 16 * kRowBytes));
  };
  constexpr std::integral_constant<int, 0> kStep0{};
  constexpr std::integral_constant<int, 1> kStep1{};
  unrolled<kLoads>([&](auto i) { read_i(kStep0, i, 0); });

  int buf = 0;                        // the slice being multiplied
  for (; t < ntiles; t += step) {
    f32x4 acc[MB][kNB];
#pragma unroll
    for (int a = 0; a < MB; ++a)
#pragma unroll
      for (int b = 0; b < kNB; ++b) acc[a][b] = f32x4{0.0f, 0.0f, 0.0f, 0.0f};
    settle(acc[0]);
    for (int kt = 0; kt < nk; ++kt) {
      const int nxt = buf + 1 == S ? 0 : buf + 1;
      // Step 0, while step 1's fragments are read. The products walk the
      // blocks in a serpentine, so that consecutive ones share an operand.
      unrolled<kProds>([&](auto jc) {
        constexpr int j = jc.value, a = j / kNB, b = a & 1 ? kNB - 1 - j % kNB : j % kNB;
        at_slot<j, kLoads, kProds / 2>([&](auto i) { read_i(kStep1, i, buf); });
        mfma(acc[a][b], fw[0][b], fx[0][a]);
      });
      // This wavefront has read its last fragments of the slice, and its loads
      // of the next slice are complete (those of later slices may be in
      // flight); past the barrier that holds for all four.
      asm volatile("s_waitcnt vmcnt(%0) lgkmcnt(0)\n\ts_barrier" :: "n"((S - 2) * kLoads)
                   : "memory");
      // Step 1, while the buffer is refilled and the next slice's first
      // fragments are read. The loads are spread over the step: issued closer
      // together they fill the address unit's queue and hold up the products
      // behind them (one load per 2 products 12.6 ms, per 4 12.1 ms at 16640 x
      // 4096 x 128256; per 6, into the next slice, 12.4 ms).
      unrolled<kProds>([&](auto jc) {
        constexpr int j = jc.value, a = j / kNB, b = a & 1 ? kNB - 1 - j % kNB : j % kNB;
        at_slot<j, kLoads, kProds>(load_i);
        at_slot<j - kProds / 4, kLoads, kProds / 2>([&](auto i) { read_i(kStep0, i, nxt); });
        mfma(acc[a][b], fw[1][b], fx[1][a]);
      });
      load_next();
      buf = nxt;
    }
    settle(acc[MB - 1]);

    // Epilogue. Lane l's accumulator r of block (a, b) is row 16 a + l % 16,
    // column 16 b + 4 (l / 16) + r of the wavefront's part of the tile.
    int el = lane;
    asm volatile("" : "+v"(el));      // lane arithmetic stays out of the K loop's registers
    const int er = el & 15, eg = el >> 4;
    int m0, n0, cols;
    tile(t, m0, n0, cols);
    const int slot = kRange ? wg : n0 / kBN;
    m0 += wm * 16 * MB;
    n0 += wn * 16 * kNB;
    cols -= wn * 16 * kNB;            // of this wavefront's part (may be negative)
    const bool wide = (P.N & 7) == 0 && (reinterpret_cast<uintptr_t>(P.logits) & 15) == 0;
    const int merge = S * kSlice;     // (max, sum) of the tile's rows from the right half
    // One row of blocks; FULL: every row and column exists and rows are stored
    // in 16-byte vectors.
    auto rows16 = [&](auto ac, auto full) {
      constexpr int a = ac.value;
      constexpr bool kFull = full.value;
      pin(acc[a]);                    // nothing of the row is formed before its turn
      uint32_t z[kNB][2];
#pragma unroll
      for (int b = 0; b < kNB; ++b) {
        z[b][0] = pack2(acc[a][b][0], acc[a][b][1]);
        z[b][1] = pack2(acc[a][b][2], acc[a][b][3]);
      }
      const int left = cols - 4 * eg; // column 16 b + r of the lane exists if below
      auto value = [&](int b, int r) {
        const uint32_t u = z[b][r >> 1];
        const float v = __uint_as_float(r & 1 ? u & 0xffff0000u : u << 16);
        return kFull || 16 * b + r < left ? v : -INFINITY;
      };
      // Statistics of the row's 32 columns in this lane, then over the four
      // lanes that hold the row. The hardware exp2 gives 0 for -inf; a row
      // with no finite value keeps the frame 0, so its terms are 0 as well.
      // NaN or +inf propagate into the sum (the maximum passes over NaN,
      // which surfaces there; +inf makes the frame -inf and its term NaN).
      float mx = -INFINITY;
      if constexpr (kFull) {
        // of the unrounded values: rounding keeps their order
#pragma unroll
        for (int b = 0; b < kNB; ++b) {
          mx = max3(mx, acc[a][b][0], acc[a][b][1]);
          mx = max3(mx, acc[a][b][2], acc[a][b][3]);
        }
        mx = __uint_as_float(pack2(0.0f, mx) & 0xffff0000u);
      } else {
#pragma unroll
        for (int b = 0; b < kNB; ++b)
#pragma unroll
          for (int r = 0; r < 4; ++r) mx = fmaxf(mx, value(b, r));
      }
      mx = fmaxf(mx, __shfl_xor(mx, 16, 64));
      mx = fmaxf(mx, __shfl_xor(mx, 32, 64));
      const float c = mx > -INFINITY ? -mx * P.k32 : 0.0f;
      float sm[4] = {0.0f, 0.0f, 0.0f, 0.0f};
#pragma unroll
      for (int b = 0; b < kNB; ++b)
#pragma unroll
        for (int r = 0; r < 4; ++r)
          sm[r] += __builtin_amdgcn_exp2f(fmaf(value(b, r), P.k32, c));
      float s = (sm[0] + sm[1]) + (sm[2] + sm[3]);
      s += __shfl_xor(s, 16, 64);
      s += __shfl_xor(s, 32, 64);
      typedef __attribute__((ext_vector_type(2))) float f32x2;
      if (wn == 1) {
        if (eg == 0)
          *(__attribute__((address_space(3))) f32x2*)(
              lds + merge + (wm * 16 * MB + 16 * a + er) * 8) = f32x2{mx, s};
      } else {
        // kept in the block's accumulators until the right half's are there
        acc[a][0][0] = mx;
        acc[a][0][1] = s;
      }
      // Logits. Blocks b and b + 1 exchange the odd 16-lane rows of one with
      // the even ones of the other: lane group g then holds eight consecutive
      // columns, 16 (b + g % 2) + 8 (g / 2). Non-temporal: they are not read
      // again here and should not displace the slices in L2.
      const int m = m0 + 16 * a + er;
      uint16_t* out = P.logits + static_cast<size_t>(m) * P.N + n0;
      if (kFull || wide) {
        out += 16 * (eg & 1) + 8 * (eg >> 1);
        const int cleft = cols - (16 * (eg & 1) + 8 * (eg >> 1));
#pragma unroll
        for (int b = 0; b < kNB; b += 2) {
          const auto lo = __builtin_amdgcn_permlane16_swap(z[b][0], z[b + 1][0], false, false);
          const auto hi = __builtin_amdgcn_permlane16_swap(z[b][1], z[b + 1][1], false, false);
          if (kFull || (m < P.M && 16 * b < cleft))
            __builtin_nontemporal_store(u32x4{lo[0], hi[0], lo[1], hi[1]},
                                        reinterpret_cast<u32x4*>(out + 16 * b));
        }
      } else if (m < P.M) {
#pragma unroll
        for (int b = 0; b < kNB; ++b)
#pragma unroll
          for (int r = 0; r < 4; ++r)
            if (16 * b + r < left)
              out[16 * b + 4 * eg + r] = static_cast<uint16_t>(z[b][r >> 1] >> (16 * (r & 1)));
      }
      __builtin_amdgcn_sched_barrier(0);
    };
    if (wide && m0 + 16 * MB <= P.M && cols >= 16 * kNB)
      unrolled<MB>([&](auto a) { rows16(a, std::true_type{}); });
    else
      unrolled<MB>([&](auto a) { rows16(a, std::false_type{}); });
    // The two halves of every row; the K loop's barriers keep the next tile's
    // writes behind these reads.
    asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory");
    if (wn == 0 && eg == 0) {
#pragma unroll
      for (int a = 0; a < MB; ++a) {
        typedef __attribute__((ext_vector_type(2))) float f32x2;
        const f32x2 o = *(const __attribute__((address_space(3))) f32x2*)(
            lds + merge + (wm * 16 * MB + 16 * a + er) * 8);
        float mx = acc[a][0][0], s = acc[a][0][1];
        merge_stats(mx, s, o[0], o[1], P.k32);
        if constexpr (kRange) {
          // those of the range so far, kept by this lane: the tiles' fp32 sums
          // are added in fp64, as the merge kernel adds those of whole tiles
          const int r = wm * 16 * MB + 16 * a + er;
          auto* run_s = (__attribute__((address_space(3))) double*)(lds + merge + 32 * MB * 8 +
                                                                    r * 8);
          auto* run_m = (__attribute__((address_space(3))) float*)(lds + merge + 32 * MB * 16 +
                                                                   r * 4);
          if (ntiles > 1) {
            double sum = static_cast<double>(s);
            if (t > 0) {
              const float m = *run_m;
              const double before = *run_s;
              const bool up = mx > m;   // the side with the smaller maximum moves
              sum = (up ? sum : before) +
                    moved(up ? before : sum, fminf(mx, m), fmaxf(mx, m), P.k32);
              mx = fmaxf(mx, m);
            }
            *run_m = mx;
            *run_s = sum;
            s = static_cast<float>(sum);
          }
        }
        const int m = m0 + 16 * a + er;
        if (m < P.M && (!kRange || t + 1 == ntiles)) {
          P.part_max[static_cast<size_t>(m) * P.parts + slot] = mx;
          P.part_sum[static_cast<size_t>(m) * P.parts + slot] = s;
        }
      }
    }
  }
  // no load of this workgroup may write LDS after it has ended
  asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
}

// Merges the column-tile partials of one row per wavefront (fp64 sum, each
// partial moved from its frame to the row maximum's by 2^(frame difference),
// evaluated in fp64).
__global__ void __launch_bounds__(kThreads) lmhead_merge_kernel(LmParams P) {
  const int lane = threadIdx.x & 63;
  const int row = static_cast<int>(blockIdx.x) * (kThreads / 64) + (threadIdx.x >> 6);
  if (row >= P.M) return;
  const float* pm = P.part_max + static_cast<size_t>(row) * P.parts;
  const float* ps = P.part_sum + static_cast<size_t>(row) * P.parts;
  float m = -INFINITY;
  for (int t = lane; t < P.parts; t += 64) m = fmaxf(m, pm[t]);
#pragma unroll
  for (int off = 32; off > 0; off >>= 1) m = fmaxf(m, __shfl_xor(m, off, 64));
  // each partial is in the frame -max_t * k (an fp32 product): move it to the
  // row's frame -m * k by 2 to the difference of the two frames
  const double cm = static_cast<double>(-m * P.k32);
  double s = 0.0;
  for (int t = lane; t < P.parts; t += 64) {
    const float mt = pm[t];
    const double st = static_cast<double>(ps[t]);
    s += (mt > -INFINITY && m > -INFINITY)
             ? st * exp2(cm - static_cast<double>(-mt * P.k32))
             : st;
  }
#pragma unroll
  for (int off = 32; off > 0; off >>= 1) s += __shfl_xor(s, off, 64);
  if (lane == 0) {
    // from the frame -m * k rounded to fp32 to the exact frame of the maximum,
    // so that row_sum is sum exp((z - m) / T) as defined
    P.row_max[row] = m;
    P.row_sum[row] = m > -INFINITY && isfinite(m)
                         ? s * exp2(-(cm + static_cast<double>(m) * static_cast<double>(P.k32)))
                         : s;
  }
}

// Rows per tile. A tile of 32 MB rows costs about 256 MB cycles of products per
// slice and as long as 40 (MB + 8) cycles' worth of LDS and cache traffic, and the
// tiles run in whole rounds over the CUs; the cheapest MB wins (at equal cost
// the larger one, which reads the weight less often). 1040 rows at V = 128256:
// five tiles of 224 rows instead of 256; 200 rows at V = 32000: four of 64,
// which fill the CUs that one of 224 would leave idle.
// With rows of more than 24 KB the slices of the tiles in flight outgrow the
// caches, and a lower tile saves less than that: 256 rows there unless another
// height is 1/16 cheaper (256 against 224 rows, us: 4000 x 16384 x 70001 7282,
// 7961; x 14336 6156, 6516; x 12288 5330, 5388; 1040 x 16384 x 128256, 12%
// cheaper with 224, 3873, 3780).
constexpr int kLongRow = 12288;
int tile_height(int rows, int tiles_n, int hidden, int cus) {
  int best = 1;
  long long best_cost = -1, tall_cost = 0;
  for (int mb = 8; mb >= 1; --mb) {
    const long long tiles = static_cast<long long>((rows + 32 * mb - 1) / (32 * mb)) * tiles_n;
    const long long rounds = (tiles + cus - 1) / cus;
    const long long cost = rounds * (256 * mb + 40 * (mb + kNB));
    if (mb == 8) tall_cost = cost;
    if (best_cost < 0 || cost < best_cost) {
      best_cost = cost;
      best = mb;
    }
  }
  if (hidden > kLongRow && 17 * best_cost > 16 * tall_cost) best = 8;
  return best;
}

template <int MB>
hipError_t run_tiles(LmParams& P, int cus, hipStream_t stream) {
  P.tiles_m = (P.M + 32 * MB - 1) / (32 * MB);
  if (P.tiles_m == 1) {
    // The columns in equal ranges, a workgroup each (as many as the partials
    // have room for). The weight is then read once, and one that the last-level
    // cache cannot hold until the next call is read past the caches (65 x
    // 4096 x 128256, 1.05 GB: 169 against 188 us; 32 x 3000 x 32000, 192 MB: 72
    // against 42 us, so not there).
    P.parts = P.tiles_n < cus ? P.tiles_n : cus;
    P.per_xcd = (P.parts + kXcds - 1) / kXcds;
    const dim3 grid(static_cast<unsigned>(kXcds * P.per_xcd));
    if (static_cast<size_t>(P.N) * P.K * 2 > kLastLevelCache)
      hipLaunchKernelGGL((lmhead_kernel<MB, true, true>), grid, dim3(kThreads), 0, stream, P);
    else
      hipLaunchKernelGGL((lmhead_kernel<MB, true, false>), grid, dim3(kThreads), 0, stream, P);
  } else {
    // as many workgroups as the rounds need, the same number on every XCD
    const int tiles = P.tiles_m * P.tiles_n;
    const int rounds = (tiles + cus - 1) / cus;
    P.parts = P.tiles_n;
    P.per_xcd = (tiles + rounds * kXcds - 1) / (rounds * kXcds);
    hipLaunchKernelGGL((lmhead_kernel<MB, false, false>),
                       dim3(static_cast<unsigned>(kXcds * P.per_xcd)), dim3(kThreads), 0, stream,
                       P);
  }
  return hipGetLastError();
}

// CUs of the current device, rounded down to whole XCDs; 0 on failure.
int device_cus() {
  constexpr int kMaxDevices = 64;
  static int cus[kMaxDevices];
  static std::mutex mu;
  int dev = 0, n = 0;
  if (hipGetDevice(&dev) != hipSuccess || dev < 0) return 0;
  std::lock_guard<std::mutex> lock(mu);
  if (dev < kMaxDevices && cus[dev]) return cus[dev];
  if (hipDeviceGetAttribute(&n, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess) return 0;
  n = n < kXcds ? kXcds : n / kXcds * kXcds;
  if (dev < kMaxDevices) cus[dev] = n;
  return n;
}

}  // namespace

namespace tv {

int launch_lmhead(const LmheadArgs& a, void* workspace, hipStream_t stream) {
  const LmheadLayout L = lmhead_layout(a.rows, a.vocab);
  LmParams P{};
  P.x = static_cast<const uint16_t*>(a.hidden);
  P.w = static_cast<const uint16_t*>(a.weight);
  P.logits = static_cast<uint16_t*>(a.logits);
  P.part_max = reinterpret_cast<float*>(static_cast<uint8_t*>(workspace) + L.off_max);
  P.part_sum = reinterpret_cast<float*>(static_cast<uint8_t*>(workspace) + L.off_sum);
  P.row_max = a.row_max;
  P.row_sum = a.row_sum;
  P.M = a.rows;
  P.K = a.hidden_size;
  P.N = a.vocab;
  P.tiles_n = L.tiles_n;
  P.k32 = static_cast<float>(1.4426950408889634 / static_cast<double>(a.temperature));
  const int cus = device_cus();
  if (!cus) return TV_ERR_HIP;
  hipError_t e = hipErrorInvalidValue;
  switch (tile_height(a.rows, L.tiles_n, a.hidden_size, cus)) {
    case 1: e = run_tiles<1>(P, cus, stream); break;
    case 2: e = run_tiles<2>(P, cus, stream); break;
    case 3: e = run_tiles<3>(P, cus, stream); break;
    case 4: e = run_tiles<4>(P, cus, stream); break;
    case 5: e = run_tiles<5>(P, cus, stream); break;
    case 6: e = run_tiles<6>(P, cus, stream); break;
    case 7: e = run_tiles<7>(P, cus, stream); break;
    case 8: e = run_tiles<8>(P, cus, stream); break;
  }
  if (e != hipSuccess) return TV_ERR_HIP;
  hipLaunchKernelGGL(lmhead_merge_kernel, dim3(static_cast<unsigned>((a.rows + 3) / 4)),
                     dim3(kThreads), 0, stream, P);
  return hipGetLastError() == hipSuccess ? TV_OK : TV_ERR_HIP;
}

}  // namespace tv
