// Layer-output error of a weight-activation quantized linear layer (Section 3.2,
// layer analysis: A_out = W * A_in with both inputs quantized):
//
//     E_f = sum_{t,o} ( Y[t,o] - sx_f * sw_f[o] * (Qx_f Qw_f^T)[t,o] )^2 ,  P = sum Y^2 ,
//     Y = X W^T .
//
// One kernel computes, per output tile, the reference product on the bf16
// matrix cores, then up to two quantized products (for W8A8: the INT8 code product on the
// int8 matrix cores and the FP8-E4M3 code product), one after the other: each product is a K loop of its own over its own
// operand arrays, the reference accumulators stay in registers for the whole kernel and
// the quantized accumulators are reduced against them (squared differences in fp64) as
// soon as their loop ends.  Y is never written to memory.
//
// Why the products run in sequence and not side by side: the loop is bound by the
// texture path (one 128-byte line every ~2.2 clocks per compute unit, whatever part of
// the line is used), by LDS bandwidth and by how many bytes can be in flight from L2
// into LDS.  One product at a time lets a stage hold whole 128-byte lines of every
// operand row (48 KB, three stages resident) and keeps a wave at two accumulator sets
// (128 registers for its 64x64 share), so that eight waves, two per SIMD, fit: while
// one waits at the stage barrier or for its fragments the other keeps the matrix core
// busy.  The 256x128 workgroup tile needs 25 % fewer operand bytes per flop than
// 128x128.  (That is for grids that fill the chip; wa_gemm_plan has the tiles of smaller ones.)  The weight-only metric's
// products have X in common and run side by side instead (wa_gemm_shared_kernel).
//
// What bounds it on full grids: power.  The part holds 1.73 GHz with the matrix cores busy for 0.67 of the clocks
// (2048 x 11008 x 4096, three bf16 products, 456 us); four waves of 128 x 64, with a quarter less LDS traffic, run at 1.87 GHz
// and 0.62 and take as long; without the deposits, at 1.89 GHz and 0.72, it takes 387 us.  On small grids: the latency of a
// step (0.2 us of deposit, barrier and fragment reads with one workgroup on a compute unit).
//
// Exactness: bf16 x bf16 products are exact in fp32 and are accumulated in fp32;
// int8 products are accumulated exactly in int32 (|sum| <= 32768*127*127 < 2^31).
// A quantized product is one of four kinds:
//   WA_INT8      : int8 codes on the int8 matrix cores (exact);
//   WA_GRID_BF16 : grid values stored as bf16 (exact for 4-bit and 8-bit grids) on the
//                  bf16 matrix cores, products exact, fp32 accumulation -- the products
//                  of the weight-only layer-output metric, where the "quantized" input is
//                  the 16-bit input itself (scale 1);
//   WA_GRID_FP8  : the same product from e4m3 codes, widened in registers: half the bytes
//                  deposited, kept in LDS and read as fragments, and no bf16 copies of the
//                  operands to write.  It meets the 1e-5 tolerance on the error sum, which
//                  the fp8 matrix cores by themselves do not.  The three products of a layer, with their
//                  inputs' passes, from the stored bf16 values and so: 2048 x 11008 x 4096
//                  469 -> 436 us, 1024 x 4096 x 4096 117 -> 111, 64 x 4096 x 4096 53 -> 47;
//                  a block of 4096 x 10624 at 2048 tokens 2099 -> 1923;
//   WA_FP8       : e4m3 codes on the fp8 matrix cores (the low-bit matmul units the WA
//                  case of Algorithm 1 targets).  Measured on the part with single
//                  instructions: the 8 products of each group of 8 consecutive k are
//                  aligned to the group's largest exponent sum (operand exponents added,
//                  whatever the mantissas) and bits more than 13 places below it are
//                  dropped towards zero; the group sums and the accumulator are then added
//                  like fp32 numbers.  On tensors with outlier channels that shifts the
//                  error sum by 1e-6 .. 3e-5 relative, more where a layer's largest outliers
//                  stretch its scales further, plus a random part that falls with the
//                  number of outputs (a few 1e-5 at some ten thousand outputs).  A caller can
//                  keep the outlier columns out of this product (zeros in the X operand) and
//                  hand their grid values over as a second part (QProd::xs / ws): one K step
//                  on the bf16 matrix cores into the same accumulators, which brings the sum
//                  to within 4e-7 at full size.
#include <algorithm>
#include <type_traits>

#include "mofq_device.h"
#include "mofq_internal.h"

namespace mofq {

namespace {

typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef float f32x16 __attribute__((ext_vector_type(16)));
typedef int i32x16 __attribute__((ext_vector_type(16)));
typedef int i32x2 __attribute__((ext_vector_type(2)));
typedef int i32x4 __attribute__((ext_vector_type(4)));
typedef float f32x4 __attribute__((ext_vector_type(4)));
typedef int i32x8 __attribute__((ext_vector_type(8)));

constexpr int SIDE_K = kWaSideCols;             // K extent of a product's optional second part: one 16-bit stage

// The K loops of a tile run one after the other as one sequence of stages, in this order.
enum : int { SEG_REF = 0, SEG_Q = 1, SEG_SIDE = 2, N_SEG = 5 };   // the reference, then (product, its side part) twice
struct Segment {
  const void* x; const void* w;                 // rows of X and W
  int64_t xrow, wrow;                           // bytes from row to row
  int32_t stages;                               // 0: not there
  int32_t half;                                 // the last stage holds half a line per row (8-bit, K % 128 == 64)
};
struct GemmArgs {
  Segment seg[N_SEG];
  const float* sx[2]; const float* sw[2];       // scales: sx one value or null (= 1); sw one value or [N]
  double* part[3];                              // [blocks]: errors of the two products (or null), sum of Y^2
  int32_t w_per_channel;
  int32_t M, N;
  int32_t tiles_m, tiles_n;
  // products cut into pieces (PIECES): accumulators [piece][tile][wave][TI * TJ * 4][lane][4], and the first piece of
  // the reference, of each product, and the end
  float* partial;
  int32_t piece0[4];
};

// ---- LDS stage ----------------------------------------------------------------------
// A stage holds one K slab of both operand tiles: TM rows of X then TN rows of W, each
// row ROW_B = 128 bytes (64 sixteen-bit or 128 eight-bit elements, one cache line), i.e.
// 8 chunks of 16 bytes, no padding.  Stages are filled by global_load_lds (each lane of a wave
// instruction deposits 16 bytes at consecutive LDS addresses), so the layout is chosen
// through WHICH global chunk a lane fetches: chunk slot p of row R holds logical chunk
// p ^ swz(R).  A 128-bit LDS read is served 16 lanes (256 bytes, all 64 banks) per
// clock; the 16 lanes of one pass read the same logical chunk of 16 consecutive rows,
// which by themselves cover 2 distinct 128-byte offsets, so the rotation advances once
// every 2 rows.
constexpr int ROW_B = 128;
constexpr int CH = ROW_B / 16;                  // chunks per row
constexpr int NST = 3;                          // stages resident
MOFQ_DEV constexpr int swz(int row) { return (row >> 1) & (CH - 1); }

// One wave instruction: lane l fetches 16 bytes at base + its own offset and deposits
// them at LDS address lds_addr + 16*l.  Written as inline assembly so that the compiler
// does not serialise later LDS reads of OTHER buffers behind the deposit; completion is
// tracked by hand with s_waitcnt vmcnt (deposits of a wave retire in order).
// (64-bit offsets: for row strides beyond 2^32 bytes per tile.)
MOFQ_DEV void lds_deposit(const char* base, uint64_t off, uint32_t lds_addr) {
  asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %1, off"
               :
               : "s"(__builtin_amdgcn_readfirstlane(lds_addr)), "v"(base + off)
               : "memory");
}
MOFQ_DEV void lds_deposit(const char* base, uint32_t off, uint32_t lds_addr) {
  asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %1, %2"
               :
               : "s"(__builtin_amdgcn_readfirstlane(lds_addr)), "v"(off), "s"(base)
               : "memory");   // m0 is not otherwise used by these kernels
}

// s_waitcnt: all LDS reads done, at most N vector-memory operations in flight (6 bits, split field).
template <int N> MOFQ_DEV void wait_deposits_and_reads() {
  __builtin_amdgcn_s_waitcnt((N & 15) | (7 << 4) | (0 << 8) | ((N >> 4) << 14));
}

// 8 e4m3 codes as bf16 (exact)
MOFQ_DEV i32x4 widened(int lo, int hi) {
  i32x4 o;
#pragma unroll
  for (int d = 0; d < 2; ++d) {
    o[2 * d] = __builtin_bit_cast(int, __builtin_amdgcn_cvt_scalef32_pk_bf16_fp8(d ? hi : lo, 1.0f, false));
    o[2 * d + 1] = __builtin_bit_cast(int, __builtin_amdgcn_cvt_scalef32_pk_bf16_fp8(d ? hi : lo, 1.0f, true));
  }
  return o;
}

enum : int { K_REF = 100, K_GRID = WA_GRID_BF16, K_I8 = WA_INT8, K_F8 = WA_FP8, K_G8 = WA_GRID_FP8 };   // K_REF: the 16-bit inputs themselves

template <int TM_, int TN_, int WM_, int WN_> struct Tile {
  static constexpr int TM = TM_, TN = TN_;                  // workgroup tile
  static constexpr int WM = WM_, WN = WN_;                  // wave tile: matrix-core tiles of 32 x 32
  static constexpr int NW = (TM / WM) * (TN / WN);          // waves per workgroup
  static constexpr int STAGE = (TM + TN) * ROW_B;           // bytes
  static constexpr int PER_CU = (160 * 1024) / (NST * STAGE + 1024);   // workgroups that LDS lets a compute unit hold
  static constexpr int PER_SIMD = PER_CU * NW / 4;          // their waves on a SIMD
};

// Workgroup -> tile.  Consecutive workgroup ids go to different XCDs (8 of them, each
// with its own L2), so ids are first regrouped so that one XCD works on a contiguous
// range of tiles (of pieces of tiles), and a range is walked in bands of 4 tile rows: the 32 workgroups
// resident on an XCD then share 4 X tiles and 8 W tiles.
MOFQ_DEV int regrouped(int id, int total) {
  const int per_xcd = total / 8;
  return id < per_xcd * 8 ? (id & 7) * per_xcd + (id >> 3) : id;
}
MOFQ_DEV void tile_of(const GemmArgs& a, int t, int& bm, int& bn) {
  constexpr int BAND = 4;
  const int band = t / (BAND * a.tiles_n);
  const int first_m = band * BAND;
  const int rows_in_band = (a.tiles_m - first_m) < BAND ? (a.tiles_m - first_m) : BAND;
  const int in_band = t - band * BAND * a.tiles_n;
  bm = first_m + in_band % rows_in_band;
  bn = in_band / rows_in_band;
}

// The layers of a launch.  Layers one launch after the other leave compute units idle in each one's last round (688 tiles of
// 2048 x 11008 x 4096 are 2.69 rounds); together they have one last round.  The XCDs' ranges are those of each layer by itself.
template <int N> struct GemmBatch {
  GemmArgs a[N];
  int32_t first[N];   // first workgroup of a layer; unused entries: INT_MAX
  MOFQ_DEV int layer_of(uint32_t block) const {
    int layer = 0;
#pragma unroll
    for (int i = 1; i < N; ++i) layer += static_cast<int>(block) >= first[i] ? 1 : 0;
    return layer;
  }
};

template <typename T, int KIND1, int KIND2, bool PIECES, bool WIDE, int N>
__global__ __launch_bounds__(T::NW * 64) __attribute__((amdgpu_waves_per_eu(T::PER_SIMD, T::PER_SIMD))) void wa_gemm_kernel(const GemmBatch<N> batch) {
  const int layer = batch.layer_of(blockIdx.x);
  const GemmArgs& a = batch.a[layer];
  constexpr int TM = T::TM, TN = T::TN, WM = T::WM, WN = T::WN, NW = T::NW;
  constexpr int TI = WM / 32, TJ = WN / 32;
  constexpr int STAGE = T::STAGE;
  constexpr int DEP = STAGE / 1024 / NW;        // deposits per wave per stage
  constexpr int FIRST = DEP / 4;                // of which the first ones are issued a step ahead
  constexpr int STEP = NW * 8;                  // rows from one deposit of a wave to the next
  static_assert(DEP * NW * 1024 == STAGE && TM % STEP == 0 && STEP % 16 == 0, "deposits");
  __shared__ __attribute__((aligned(1024))) unsigned char s_buf[NST * STAGE];
  __shared__ double s_red[3][NW];

  const uint32_t lds0 = static_cast<uint32_t>(reinterpret_cast<uintptr_t>((__attribute__((address_space(3))) unsigned char*)s_buf));
  const int tid = threadIdx.x;
  const int lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int wm = wave / (TN / WN), wn = wave % (TN / WN);
  const int r = lane & 31, g = lane >> 5;

  const int tiles = a.tiles_m * a.tiles_n;
  int t = regrouped(static_cast<int>(blockIdx.x) - (N > 1 ? batch.first[layer] : 0), PIECES ? tiles * a.piece0[3] : tiles), piece = 0;
  if constexpr (PIECES) { piece = t / tiles; t -= piece * tiles; }
  int bm, bn;
  tile_of(a, t, bm, bn);
  const int m0 = bm * TM, n0 = bn * TN;

  // LDS byte offsets of this lane's fragment rows inside a stage, and of the chunks it
  // reads: lane (r, g) supplies row r of a 32-row operand tile and the g-th half of the
  // instruction's K range, for A and B alike.
  const int sw = swz(r);                                   // same for all of the lane's rows (multiples of 32 apart)
  const int row_a = (wm * WM + r) * ROW_B;                 // + i * 32 * ROW_B
  const int row_b = (TM + wn * WN + r) * ROW_B;            // + j * 32 * ROW_B
  int ch_k[CH / 2], ch_h[CH / 2], ch_f[CH / 2];
#pragma unroll
  for (int q = 0; q < CH / 2; ++q) {
    ch_k[q] = ((2 * q + g) ^ sw) * 16;                       // K slice q of a stage, 16 bytes per lane
    // 16-bit elements: the columns that half a slice of widened codes holds; in the weight-only metric's products as wa_gemm_shared_kernel
    ch_h[q] = KIND1 == K_GRID ? ch_k[q] : ((4 * (q / 2) + 2 * g + q % 2) ^ sw) * 16;
    ch_f[q] = ((4 * (q >> 1) + 2 * g + (q & 1)) ^ sw) * 16;  // fp8 instruction q/2: 32 bytes per lane, half q%2
  }

  // ---- the deposits' position in the sequence of stages ----------------------------------
  // Deposit d of a stage covers the rows d STEP + 8 wave + lane / 8 (multiples of 16 apart, so the lane fetches the
  // same chunk of each).  The tile's first row and the stage are in the scalar bases, a lane's row and chunk in `off`:
  // nothing is computed per deposit (with 64-bit addresses per lane, five vector instructions each, these cases took 4 to
  // 6 % longer: 2048 x 11008 x 4096, three bf16 products, 535 -> 511 us a call, 2048 x 4096 x 4096 196 -> 184.5).  Rows past the edge repeat the last one (masked later).
  // The deposits run up to three stages ahead of the matrix instructions, across the ends of the products: what the last
  // steps of one product fetch are the first stages of the next, so a product does not begin with an empty pipeline
  // (777 x 3000 x 5056, large tiles: 156 -> 154 us).
  const int row0 = wave * 8 + (lane >> 3), kc = (lane & 7) ^ swz(row0);
  using off_t = std::conditional_t<WIDE, uint64_t, uint32_t>;
  off_t off[DEP];
  const char* dep_x = nullptr;
  const char* dep_w = nullptr;
  int dep_left = 0, dep_half = 0, dep_seg = -1;
  // A piece: some stages of one product, with the side part behind its last ones.  (Widened codes': the columns of the reference
  // product's piece, which may begin and end at half a line.)
  int mine = SEG_REF, piece_byte = 0, piece_stages = 0, piece_half = 0;
  bool last_piece = false;
  if constexpr (PIECES) {
    const int q = (piece >= a.piece0[1]) + (piece >= a.piece0[2]);
    mine = q == 0 ? static_cast<int>(SEG_REF) : SEG_Q + 2 * (q - 1);
    const int n = a.piece0[q + 1] - a.piece0[q], i = piece - a.piece0[q];
    last_piece = i == n - 1;
    const bool widened_codes = (KIND1 == K_G8 && q == 1) || (KIND2 == K_G8 && q == 2);
    const int total = a.seg[widened_codes ? static_cast<int>(SEG_REF) : mine].stages, first = total * i / n, count = total * (i + 1) / n - first;
    piece_byte = first * (widened_codes ? ROW_B / 2 : ROW_B);
    piece_stages = widened_codes ? (count + 1) / 2 : count;
    piece_half = widened_codes ? count % 2 : a.seg[mine].half && last_piece;
    dep_seg = mine - 1;
  }
  const int end_seg = PIECES ? (mine != SEG_REF && last_piece ? mine + 2 : mine + 1) : static_cast<int>(N_SEG);
  auto next_segment = [&]() {
    int s = dep_seg + 1;
    while (s < end_seg && a.seg[s].stages == 0) ++s;
    if (s == end_seg) {       // past the last stage: it is fetched again, unused
      dep_x -= ROW_B;
      dep_w -= ROW_B;
      dep_left = 1;
      dep_half = 0;
      return;
    }
    dep_seg = s;
    const Segment& sg = a.seg[s];
    dep_x = static_cast<const char*>(sg.x) + m0 * sg.xrow;
    dep_w = static_cast<const char*>(sg.w) + n0 * sg.wrow;
    dep_left = sg.stages;
    dep_half = sg.half;
    if constexpr (PIECES) {
      if (s == mine) {
        dep_x += piece_byte;
        dep_w += piece_byte;
        dep_left = piece_stages;
        dep_half = piece_half;
      }
    }
#pragma unroll
    for (int d = 0; d < DEP; ++d) {
      const bool x = d * STEP < TM;
      const int row = row0 + (x ? d * STEP : d * STEP - TM), last = (x ? a.M - m0 : a.N - n0) - 1;
      off[d] = static_cast<off_t>(row < last ? row : last) * static_cast<off_t>(x ? sg.xrow : sg.wrow) + kc * 16;
    }
  };
  auto next_stage = [&]() {
    dep_left -= 1;
    dep_x += ROW_B;
    dep_w += ROW_B;
    if (dep_left <= 1) {
      if (dep_left <= 0) next_segment();
      // The last stage of an 8-bit product may hold half a line per row: the missing half fetches
      // the valid one again (addresses stay inside the row) and is not multiplied.
      if (dep_left == 1 && dep_half) {
#pragma unroll
        for (int d = 0; d < DEP; ++d) off[d] -= kc >= CH / 2 ? ROW_B / 2 : 0;
      }
    }
  };
  auto issue = [&](int buf, int lo, int hi) {   // deposits [lo, hi) of the current stage into the buffer at byte `buf`
#pragma unroll
    for (int d = 0; d < DEP; ++d)
      if (d >= lo && d < hi) lds_deposit(d * STEP < TM ? dep_x : dep_w, off[d], lds0 + static_cast<uint32_t>(buf + (wave + NW * d) * 1024));
  };

  // Stages 0 and 1 and the first deposits of stage 2.
  int b0 = 0, b1 = STAGE, b2 = 2 * STAGE;   // buffers of the stages k, k + 1, k + 2
  static_assert(NST == 3, "three buffers in turn");
  next_stage();
  issue(b0, 0, DEP);
  next_stage();
  issue(b1, 0, DEP);
  wait_deposits_and_reads<DEP>();
  __builtin_amdgcn_s_barrier();
  asm volatile("" ::: "memory");
  next_stage();
  issue(b2, 0, FIRST);

  // ---- one product (or side part): a loop over its stages ---------------------------------
  // KIND selects element size and matrix instruction; acc is f32x16 or i32x16.
  auto product = [&](auto kind_c, auto& acc, const int stages, const bool half) {
    constexpr int KIND = decltype(kind_c)::value;
    constexpr bool WIDENED = KIND == K_G8, EIGHT = KIND == K_I8 || KIND == K_F8 || WIDENED;
    constexpr int NG = (KIND == K_F8) ? CH / 4 : CH / 2;            // matrix groups per stage (TI*TJ instructions each)
    // Fragments of group gi of a stage: f[0 .. TI) = A tiles, f[TI ..) = B tiles.
    using frag_t = std::conditional_t<KIND == K_F8, i32x8, i32x4>;
    auto load_frag = [&](const unsigned char* row, int gi) {
      if constexpr (KIND == K_F8) {
        const i32x4 lo = *reinterpret_cast<const i32x4*>(row + ch_f[2 * gi]), hi = *reinterpret_cast<const i32x4*>(row + ch_f[2 * gi + 1]);
        return __builtin_shufflevector(lo, hi, 0, 1, 2, 3, 4, 5, 6, 7);
      } else {
        return *reinterpret_cast<const i32x4*>(row + (EIGHT ? ch_k[gi] : ch_h[gi]));
      }
    };
    auto load_group = [&](const unsigned char* st, int gi, frag_t (&f)[TI + TJ]) {
#pragma unroll
      for (int i = 0; i < TI; ++i) f[i] = load_frag(st + row_a + i * 32 * ROW_B, gi);
#pragma unroll
      for (int j = 0; j < TJ; ++j) f[TI + j] = load_frag(st + row_b + j * 32 * ROW_B, gi);
    };
    // E4M3 codes for the bf16 matrix cores (grid values have 4 significant bits: the same operands as if they had been stored as
    // bf16).  A lane's 16 codes of a fragment are the operands of two instructions, 8 each; the 16-bit products take their columns in the
    // same order (ch_h), so that values on the grid leave an error of exactly 0.  (Exchanging codes between lanes for the other
    // order costs 2 to 4 % of a call.)  They are widened (4 conversions to 8 codes) between the matrix instructions before: the second
    // half of a group's during its first half, the next group's first half (of `next`) during its second.
    bf16x8 wide[2][TI + TJ];
    auto widen = [](const auto& v, int h) { return __builtin_bit_cast(bf16x8, widened(v[2 * h], v[2 * h + 1])); };
    // The matrix instructions of one group, with the deposits [lo, hi) of the current stage
    // spread between them: a wave issues in order, so a burst of deposits (each occupies
    // the texture path for ~18 clocks, and all waves share it) would hold back the
    // matrix instructions behind it while the matrix pipe runs dry.
    // `then` (the next group's fragment reads) follows the first instruction: what that one waits for is its own
    // group's fragments alone.
    auto run_group = [&](const frag_t (&f)[TI + TJ], const frag_t (&next)[TI + TJ], int buf, int lo, int hi, auto then) {
      if constexpr (WIDENED) {
        constexpr int PER = TI * TJ;
#pragma unroll
        for (int m = 0; m < 2 * PER; ++m) {
          const int h = m / PER, i = m % PER / TJ, j = m % TJ, n = hi - lo;
          __builtin_amdgcn_sched_barrier(0);
          if (m == (PER > 1 ? 1 : 0)) then();
          issue(buf, lo + m * n / (2 * PER), lo + (m + 1) * n / (2 * PER));
#pragma unroll
          for (int q = 0; q < TI + TJ; ++q)
            if (q >= (m % PER) * (TI + TJ) / PER && q < (m % PER + 1) * (TI + TJ) / PER) wide[1 - h][q] = h == 0 ? widen(f[q], 1) : widen(next[q], 0);
          __builtin_amdgcn_sched_barrier(0);
          acc[i][j] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(wide[h][i], wide[h][TI + j], acc[i][j], 0, 0, 0);
        }
      } else {
#pragma unroll
        for (int i = 0; i < TI; ++i)
#pragma unroll
          for (int j = 0; j < TJ; ++j) {
            {
              const int m = i * TJ + j, n = hi - lo;
              __builtin_amdgcn_sched_barrier(0);
              if (m == (TI * TJ > 1 ? 1 : 0)) then();
              issue(buf, lo + m * n / (TI * TJ), lo + (m + 1) * n / (TI * TJ));
              __builtin_amdgcn_sched_barrier(0);
            }
            if constexpr (KIND == K_REF || KIND == K_GRID) {
              acc[i][j] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(bf16x8, f[i]), __builtin_bit_cast(bf16x8, f[TI + j]), acc[i][j], 0, 0, 0);
            } else if constexpr (KIND == K_I8) {
              acc[i][j] = __builtin_amdgcn_mfma_i32_32x32x32_i8(f[i], f[TI + j], acc[i][j], 0, 0, 0);
            } else {
              // format selectors 0 = E4M3 for both operands; block scales 2^0 (exponent byte 127)
              acc[i][j] = __builtin_amdgcn_mfma_scale_f32_32x32x64_f8f6f4(f[i], f[TI + j], acc[i][j], 0, 0, 0, 127, 0, 127);
            }
          }
      }
    };
    // One K step.  Its last group is preceded by a barrier that makes stage k+1 visible to everyone and tells
    // everyone that stage k is no longer read (its last fragments are in registers): the fragments of the next step's
    // first group are requested there, ahead of a whole group of matrix instructions, and the deposits of
    // stage k+NST may begin to overwrite stage k.  So no step starts by waiting for LDS, and up to three
    // stages are on their way or unread.  Inside the step the fragments of group g+1 are requested before the matrix
    // instructions of group g are issued, and the deposits are spread over the groups so
    // that the texture path works while the matrix cores do.
    // (Straight-line code away from the ends: with the ends' branch in every step 2048 x 11008 x 4096 takes 532 us.)
    frag_t f[2][TI + TJ];
    auto step = [&](auto inside_c, auto last_c, const bool drop) {   // last step, drop: the second half of the stage counts nothing
#pragma unroll
      for (int gi = 0; gi < NG; ++gi) {
        if constexpr (decltype(last_c)::value && EIGHT) {
          if (gi >= NG / 2) {
#pragma unroll
            for (int i = 0; i < TI; ++i) {
              f[gi & 1][i] = drop ? frag_t{} : f[gi & 1][i];
              if constexpr (WIDENED) wide[0][i] = drop ? bf16x8{} : wide[0][i];
            }
          }
        }
        if (gi + 1 < NG) {
          run_group(f[gi & 1], f[(gi + 1) & 1], b2, FIRST + gi * (DEP - FIRST) / (NG - 1), FIRST + (gi + 1) * (DEP - FIRST) / (NG - 1),
                    [&] { load_group(s_buf + b0, gi + 1, f[(gi + 1) & 1]); });
        } else {
          // this wave's deposits of stage k+1 have landed, its fragment reads are done; stage k+2 may stay in flight
          wait_deposits_and_reads<DEP>();
          __builtin_amdgcn_s_barrier();
          asm volatile("" ::: "memory");     // LDS reads below must not move above the barrier
          if constexpr (decltype(inside_c)::value) {
            dep_left -= 1;
            dep_x += ROW_B;
            dep_w += ROW_B;
          } else {
            next_stage();
          }
          // (behind the last step: the next product's, which it reads again as its own kind)
          run_group(f[gi & 1], f[(gi + 1) & 1], b0, 0, FIRST, [&] { load_group(s_buf + b1, 0, f[(gi + 1) & 1]); });
        }
      }
      const int b = b0;
      b0 = b1;
      b1 = b2;
      b2 = b;
    };
    load_group(s_buf + b0, 0, f[0]);
    if constexpr (WIDENED) {
#pragma unroll
      for (int q = 0; q < TI + TJ; ++q) wide[0][q] = widen(f[0][q], 0);
    }
    using yes = std::true_type;
    using no = std::false_type;
    int k = EIGHT ? 1 : 0;
    // the deposits' next stage is inside the product, and not its last
    for (; k < stages - 4; ++k) step(yes{}, no{}, false);
    for (; k < stages; ++k) step(no{}, no{}, false);
    if constexpr (EIGHT) step(no{}, yes{}, half);
  };

  // ---- squared differences in fp64.  Accumulator value e of a lane in one 32x32 tile is
  // output (row 8*(e/4) + 4*g + e%4, column lane%32) of that tile; rows and columns past
  // the matrix edge hold repeats of the last row and are skipped.  The first reduction
  // also sums Y^2.
  f32x16 acc_r[TI][TJ];
  double p = 0.0;
  auto sq_diff = [&](auto with_p_c, const auto& acc_q, const float* sx, const float* sw_) {
    constexpr bool WITH_P = decltype(with_p_c)::value;
    __builtin_amdgcn_sched_barrier(0);
    const double sxd = sx ? static_cast<double>(*sx) : 1.0;
    double e_q = 0.0;
    // rows of this lane's accumulators that exist: 32 i + 8 (e/4) + e%4 < row_lim.  Opaque,
    // so that each reduction computes its own masks instead of keeping 128 of them live.
    int row_lim = a.M - (m0 + wm * WM + 4 * g);
    asm volatile("" : "+v"(row_lim));
#pragma unroll
    for (int j = 0; j < TJ; ++j) {
      const int n = n0 + wn * WN + j * 32 + r;
      const bool col_ok = n < a.N;
      const int ns = (a.w_per_channel && col_ok) ? n : 0;
      const double cq = sxd * static_cast<double>(sw_[ns]);
#pragma unroll
      for (int i = 0; i < TI; ++i)
#pragma unroll
        for (int e = 0; e < 16; ++e) {
          const bool ok = col_ok && (i * 32 + 8 * (e / 4) + (e % 4)) < row_lim;
          // Opaque copy, ordered after the previous element's sum.  Without it the fp64
          // image of all 128 reference values is kept (spilled) across the next product's
          // K loop for reuse in its reduction, and the conversions of all elements are
          // hoisted ahead of the two summation chains, which spills as well: every
          // register is in use here.
          float yf = acc_r[i][j][e];
          asm volatile("" : "+v"(yf) : "v"(e_q));
          const double y = ok ? static_cast<double>(yf) : 0.0;
          const double q = ok ? static_cast<double>(acc_q[i][j][e]) : 0.0;
          const double d = __builtin_fma(-cq, q, y);
          e_q = __builtin_fma(d, d, e_q);
          if constexpr (WITH_P) p = __builtin_fma(y, y, p);
        }
    }
    // Pin the sums here: otherwise the Y^2 chain is sunk to the end of the kernel and
    // its 128 fp64 inputs are spilled across the next product.
    asm volatile("" : "+v"(e_q), "+v"(p));
    __builtin_amdgcn_sched_barrier(0);   // and keep the next product's set-up out of this reduction
    return wave_sum(e_q);
  };

  auto clear = [&](auto& acc) {
#pragma unroll
    for (int i = 0; i < TI; ++i)
#pragma unroll
      for (int j = 0; j < TJ; ++j)
#pragma unroll
        for (int e = 0; e < 16; ++e) acc[i][j][e] = 0;
  };
  if constexpr (PIECES) {
    auto store = [&](const auto& acc) {
      f32x4* const to = reinterpret_cast<f32x4*>(a.partial) + ((static_cast<int64_t>(piece) * tiles + bm * a.tiles_n + bn) * NW + wave) * (TI * TJ * 4 * 64) + lane;
#pragma unroll
      for (int i = 0; i < TI; ++i)
#pragma unroll
        for (int j = 0; j < TJ; ++j)
#pragma unroll
          for (int q = 0; q < 4; ++q) {
            i32x4 v;
#pragma unroll
            for (int x = 0; x < 4; ++x) {
              const auto one = acc[i][j][4 * q + x];
              v[x] = __builtin_bit_cast(int, one);
            }
            to[((i * TJ + j) * 4 + q) * 64] = __builtin_bit_cast(f32x4, v);
          }
    };
    auto run = [&](auto kind_c) {
      constexpr int KIND = decltype(kind_c)::value;
      if constexpr (KIND != WA_NONE) {
        using acc_t = std::conditional_t<KIND == K_I8, i32x16, f32x16>;
        acc_t acc[TI][TJ];
        clear(acc);
        product(kind_c, acc, piece_stages, piece_half != 0);
        if constexpr (KIND == K_F8) product(std::integral_constant<int, K_GRID>{}, acc, last_piece ? a.seg[mine + 1].stages : 0, false);
        store(acc);
      }
    };
    if (mine == SEG_REF) run(std::integral_constant<int, K_REF>{});
    else if (mine == SEG_Q) run(std::integral_constant<int, KIND1>{});
    else run(std::integral_constant<int, KIND2>{});
    wait_deposits_and_reads<0>();   // LDS is given back with the workgroup: the unused deposits have to have landed
    return;
  }
  clear(acc_r);
  product(std::integral_constant<int, K_REF>{}, acc_r, a.seg[SEG_REF].stages, false);
  double e_q[2] = {0.0, 0.0};
  auto quantized = [&](auto kind_c, auto slot_c) {
    constexpr int KIND = decltype(kind_c)::value;
    constexpr int SLOT = decltype(slot_c)::value;
    if constexpr (KIND != WA_NONE) {
      using acc_t = std::conditional_t<KIND == K_I8, i32x16, f32x16>;
      acc_t acc_q[TI][TJ];
      clear(acc_q);
      product(kind_c, acc_q, a.seg[SEG_Q + 2 * SLOT].stages, a.seg[SEG_Q + 2 * SLOT].half != 0);
      // The columns split off from an fp8-unit product: one K step from their grid values on
      // the bf16 matrix cores into the same accumulators (both accumulate in fp32).
      if constexpr (KIND == K_F8) product(std::integral_constant<int, K_GRID>{}, acc_q, a.seg[SEG_SIDE + 2 * SLOT].stages, false);
      // the first reduction also sums Y^2
      e_q[SLOT] = sq_diff(std::integral_constant<bool, SLOT == 0>{}, acc_q, a.sx[SLOT], a.sw[SLOT]);
    }
  };
  quantized(std::integral_constant<int, KIND1>{}, std::integral_constant<int, 0>{});
  quantized(std::integral_constant<int, KIND2>{}, std::integral_constant<int, 1>{});
  p = wave_sum(p);
  wait_deposits_and_reads<0>();   // LDS is given back with the workgroup: the unused deposits have to have landed
  if (lane == 0) { s_red[0][wave] = e_q[0]; s_red[1][wave] = e_q[1]; s_red[2][wave] = p; }
  __syncthreads();
  if (tid == 0) {
    const int out = bm * a.tiles_n + bn;
    double t[3] = {0.0, 0.0, 0.0};
    for (int q = 0; q < 3; ++q)
      for (int w = 0; w < NW; ++w) t[q] += s_red[q][w];   // fixed order
    for (int q = 0; q < 3; ++q)
      if (a.part[q]) a.part[q][out] = t[q];
  }
}

// The sums of a tile whose products were cut into pieces: fp32 (int32) partial sums in the order of K, then the
// squared differences as above.
template <typename T, int KIND1, int KIND2, int N>
__global__ __launch_bounds__(T::NW * 64) void wa_pieces_kernel(const GemmBatch<N> batch) {
  const int layer = batch.layer_of(blockIdx.x);
  const GemmArgs& a = batch.a[layer];
  const int tile = static_cast<int>(blockIdx.x) - (N > 1 ? batch.first[layer] : 0);
  constexpr int NW = T::NW, TI = T::WM / 32, TJ = T::WN / 32;
  __shared__ double s_red[3][NW];
  const int lane = threadIdx.x & 63;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int bm = tile / a.tiles_n, bn = tile - bm * a.tiles_n;
  const int m = bm * T::TM + wave / (T::TN / T::WN) * T::WM + 4 * (lane >> 5), n0 = bn * T::TN + wave % (T::TN / T::WN) * T::WN + (lane & 31);
  const int64_t piece = static_cast<int64_t>(a.tiles_m * a.tiles_n) * NW * (TI * TJ * 4 * 64);   // f32x4 from piece to piece
  const f32x4* const from = reinterpret_cast<const f32x4*>(a.partial) + (static_cast<int64_t>(tile) * NW + wave) * (TI * TJ * 4 * 64) + lane;
  double e[2] = {0.0, 0.0}, p = 0.0;
#pragma unroll
  for (int j = 0; j < TJ; ++j) {
    const int n = n0 + j * 32;
    const bool col_ok = n < a.N;
    double c[2];
#pragma unroll
    for (int s = 0; s < 2; ++s)
      c[s] = (s == 0 || KIND2 != WA_NONE) ? (a.sx[s] ? static_cast<double>(*a.sx[s]) : 1.0) * static_cast<double>(a.sw[s][a.w_per_channel && col_ok ? n : 0]) : 0.0;
#pragma unroll
    for (int i = 0; i < TI; ++i) {
      const f32x4* const at = from + (i * TJ + j) * 4 * 64;
      auto sum = [&](auto kind_c, int q, double (&v)[16]) {
        using vec = std::conditional_t<decltype(kind_c)::value == K_I8, i32x4, f32x4>;
        vec s[4] = {};
        for (int k = a.piece0[q]; k < a.piece0[q + 1]; ++k)
#pragma unroll
          for (int h = 0; h < 4; ++h) s[h] += __builtin_bit_cast(vec, at[k * piece + h * 64]);
#pragma unroll
        for (int x = 0; x < 16; ++x) v[x] = static_cast<double>(s[x / 4][x % 4]);
      };
      double y[16], v[16];
      sum(std::integral_constant<int, K_REF>{}, 0, y);
      auto add = [&](int s) {
#pragma unroll
        for (int x = 0; x < 16; ++x) {
          const bool ok = col_ok && m + i * 32 + 8 * (x / 4) + x % 4 < a.M;
          const double d = ok ? __builtin_fma(-c[s], v[x], y[x]) : 0.0;
          e[s] = __builtin_fma(d, d, e[s]);
          if (s == 0) p = ok ? __builtin_fma(y[x], y[x], p) : p;
        }
      };
      sum(std::integral_constant<int, KIND1>{}, 1, v);
      add(0);
      if constexpr (KIND2 != WA_NONE) {
        sum(std::integral_constant<int, KIND2>{}, 2, v);
        add(1);
      }
    }
  }
  const double w[3] = {wave_sum(e[0]), wave_sum(e[1]), wave_sum(p)};
  if (lane < 3) s_red[lane][wave] = lane == 0 ? w[0] : (lane == 1 ? w[1] : w[2]);
  __syncthreads();
  if (threadIdx.x < 3 && a.part[threadIdx.x]) {
    double t = 0.0;
    for (int k = 0; k < NW; ++k) t += s_red[threadIdx.x][k];   // fixed order
    a.part[threadIdx.x][tile] = t;
  }
}

// ---- bf16 products that share X (weight-only layer output) -------------------------------------------------
// X W^T, X G1^T and X G2^T (of a format alone, NQ = 1, the first two) in one K loop: a stage holds one line of K of TM rows of X
// and of TN rows of W, G1 and G2 each, so X is deposited and its fragments are read once instead of three times: for a 256x128 tile 640 rows a step of 64
// of K instead of 1152, and 8 fragments for 12 matrix instructions instead of 12.  A lane of a 64x64 share then holds 192
// accumulators, 247 registers in all, so two waves still fit a SIMD.  A stage of 80 KB (PAIR: 64) leaves room for two in LDS;
// as a step lasts three times as long as one of wa_gemm_kernel, a stage has as long to arrive if its deposits are issued early in the
// step before: over its first third (FIRST, SPREAD; over two thirds of it 2048 x 11008 x 4096 474 us a call instead of 467, 1536 x
// 11008 x 8192 913 instead of 885).  Measured, layer selection with INT4 and E2M1, us, one product after the other -> here:
// 2048 x 11008 x 4096 (tokens x rows x columns) 516 -> 467, 1536 x 11008 x 8192 1009 -> 885, 2048 x 4096 x 4096 186 -> 167, 1024 x 11008 x 4096
// 349 -> 314, 512 x 4096 x 4096 100 -> 82, 777 x 3000 x 5056 118 -> 109, 64 x 4096 x 1024 39.8 -> 35.  Bound by power and LDS as
// wa_gemm_kernel.  Medium tiles have eight waves of 64x32 (four of 64x64 are 1 % slower).
//
// PAIR: two 4-bit formats' grid values come as e4m3 codes in one array (grid_fp8_at) and are widened to bf16, exactly, while the product
// before runs: 512 rows a step instead of 640, fragments of 6 x 16 bytes for 12 matrix instructions instead of 8, and half the
// bytes for the scoring pass to write.  A lane holds one format's codes of a group at a time (both formats' take more registers than
// two waves of a SIMD have: 5 spilled, 458 us for the first shape).  As bf16 -> so, us: 2048 x 11008 x 4096 443 -> 426 (1.50 PFLOP/s in
// the kernel), 1536 x 11008 x 8192 840 -> 797, 2048 x 4096 x 4096 161 -> 159, 1024 x 11008 x 4096 299 -> 250, 512 x 4096 x 4096 77 -> 71, 777 x 3000 x
// 5056 106 -> 97, 64 x 4096 x 1024 34.2 -> 30.4.  The bf16 form serves 8-bit formats and scales with several ratios, whose
// values leave the emission pass.
//
// All forms add up a product in one order (wa_gemm_kernel's pieces of one too) and divide a tile among the same waves: a format's error
// is the same number, bit for bit, with another candidate beside it and alone.  Alone (mofq_score), us, wa_gemm_kernel -> here: 2048 x
// 11008 x 4096 354 -> 331, 2048 x 4096 x 4096 136 -> 127, 777 x 3000 x 5056 90.2 -> 92.4, 512 x 4096 x 4096 73.6 -> 67.4.
template <int TM_, int TN_, int WM_, int WN_, int NQ_, bool PAIR_> struct SharedTile {
  static constexpr int NQ = NQ_;        // quantized products
  static constexpr bool PAIR = PAIR_;   // their operands: one array of e4m3 codes, else bf16
  static constexpr int NB = PAIR_ ? 2 : 1 + NQ_;   // arrays beside X
  static constexpr int TM = TM_, TN = TN_, WM = WM_, WN = WN_;
  static constexpr int NW = (TM / WM) * (TN / WN);
  static constexpr int STAGE = (TM + NB * TN) * ROW_B;
  static constexpr int PER_CU = (160 * 1024) / (2 * STAGE);
  static constexpr int PER_SIMD = PER_CU * NW / 4;
};

template <typename T>
__global__ __launch_bounds__(T::NW * 64) __attribute__((amdgpu_waves_per_eu(T::PER_SIMD, T::PER_SIMD))) void wa_gemm_shared_kernel(const GemmArgs a) {
  constexpr int TM = T::TM, TN = T::TN, WM = T::WM, WN = T::WN, NW = T::NW;
  constexpr int TI = WM / 32, TJ = WN / 32, STAGE = T::STAGE, STEP = NW * 8;
  constexpr bool PAIR = T::PAIR;
  constexpr int NB = T::NB, NP = 1 + T::NQ;                    // products
  constexpr int DX = TM / STEP, DW = TN / STEP, DEP = DX + NB * DW;   // deposits per wave per stage
  constexpr int NG = CH / 2, NSUB = NP * NG;                         // groups of 16 of K; a group of one product
  constexpr int FIRST = NB == 2 ? DEP / 4 : DEP / 5, SPREAD = 4;                   // deposits issued behind the barrier; over how many parts the others go
  static_assert(TM % STEP == 0 && TN % STEP == 0 && STEP % 16 == 0, "deposits");
  static_assert(SPREAD < NSUB && (!PAIR || NP == 3), "parts of a step");
  __shared__ __attribute__((aligned(1024))) unsigned char s_buf[2 * STAGE];

  const uint32_t lds0 = static_cast<uint32_t>(reinterpret_cast<uintptr_t>((__attribute__((address_space(3))) unsigned char*)s_buf));
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int wm = wave / (TN / WN), wn = wave % (TN / WN);
  const int r = lane & 31, g = lane >> 5;
  int bm, bn;
  tile_of(a, regrouped(blockIdx.x, gridDim.x), bm, bn);
  const int m0 = bm * TM, n0 = bn * TN;

  const int sw = swz(r);
  const int row_a = (wm * WM + r) * ROW_B, row_b = (TM + wn * WN + r) * ROW_B;
  int ch_k[NG];
#pragma unroll
  for (int q = 0; q < NG; ++q) ch_k[q] = ((2 * q + g) ^ sw) * 16;

  // deposits: the tile's first row and the stage in scalar bases, a lane's row and chunk in 32-bit offsets
  const int row0 = wave * 8 + (lane >> 3), kc = (lane & 7) ^ swz(row0);
  uint32_t off_x[DX], off_w[DW], off_g[DW];
  const Segment& sr = a.seg[SEG_REF];
  const Segment& s1 = a.seg[SEG_Q];
  const Segment& s2 = a.seg[SEG_Q + 2];
  const auto offset = [&](int row, int last, int64_t pitch) { return static_cast<uint32_t>(row < last ? row : last) * static_cast<uint32_t>(pitch) + kc * 16; };
#pragma unroll
  for (int d = 0; d < DX; ++d) off_x[d] = offset(row0 + d * STEP, a.M - m0 - 1, sr.xrow);
#pragma unroll
  for (int d = 0; d < DW; ++d) {
    off_w[d] = offset(row0 + d * STEP, a.N - n0 - 1, sr.wrow);
    off_g[d] = offset(row0 + d * STEP, a.N - n0 - 1, s1.wrow);
  }
  const char* dep_x = static_cast<const char*>(sr.x) + m0 * sr.xrow;
  const char* dep_w[3] = {static_cast<const char*>(sr.w) + n0 * sr.wrow, static_cast<const char*>(s1.w) + n0 * s1.wrow, static_cast<const char*>(s2.w) + n0 * s2.wrow};
  const int stages = sr.stages;
  int dep_left = stages - 1;       // stages behind the one that is being deposited; past the last it is fetched again, unused
  auto next_stage = [&]() {
    const int by = dep_left > 0 ? ROW_B : 0;
    dep_left -= 1;
    dep_x += by;
#pragma unroll
    for (int q = 0; q < NB; ++q) dep_w[q] += by;
  };
  auto issue = [&](int buf, int lo, int hi) {
#pragma unroll
    for (int d = 0; d < DEP; ++d)
      if (d >= lo && d < hi) {
        const uint32_t at = lds0 + static_cast<uint32_t>(buf + (wave + NW * d) * 1024);
        if (d < DX) lds_deposit(dep_x, off_x[d], at);
        else if ((d - DX) / DW == 0) lds_deposit(dep_w[0], off_w[(d - DX) % DW], at);
        else lds_deposit(dep_w[(d - DX) / DW], off_g[(d - DX) % DW], at);
      }
  };

  f32x16 acc[NP][TI][TJ];
#pragma unroll
  for (int q = 0; q < NP; ++q)
#pragma unroll
    for (int i = 0; i < TI; ++i)
#pragma unroll
      for (int j = 0; j < TJ; ++j)
#pragma unroll
        for (int e = 0; e < 16; ++e) acc[q][i][j][e] = 0.0f;

  int b0 = 0, b1 = STAGE;
  issue(b0, 0, DEP);
  next_stage();
  issue(b1, 0, FIRST);
  wait_deposits_and_reads<FIRST>();
  __builtin_amdgcn_s_barrier();
  asm volatile("" ::: "memory");

  i32x4 fa[2][TI], fb[2][TJ];
  auto load_a = [&](int buf, int gi) {
#pragma unroll
    for (int i = 0; i < TI; ++i) fa[gi & 1][i] = *reinterpret_cast<const i32x4*>(s_buf + buf + row_a + ch_k[gi] + i * 32 * ROW_B);
  };
  auto load_b = [&](int buf, int sub) {   // sub = NP * group + product
#pragma unroll
    for (int j = 0; j < TJ; ++j) fb[sub & 1][j] = *reinterpret_cast<const i32x4*>(s_buf + buf + row_b + ch_k[sub / NP] + (sub % NP * TN + j * 32) * ROW_B);
  };
  // PAIR: a group's 8 codes of each format, widened into fb while the product before runs
  const int row_q = (TM + TN + wn * WN + r) * ROW_B, half_q = ((g ^ (r >> 4)) & 1) * 8;
  i32x2 fq[TJ];
  auto load_q = [&](int buf, int gi, int f) {
#pragma unroll
    for (int j = 0; j < TJ; ++j) fq[j] = *reinterpret_cast<const i32x2*>(s_buf + buf + row_q + ((4 * f + gi) ^ sw) * 16 + half_q + j * 32 * ROW_B);
  };
  load_a(b0, 0);
  load_b(b0, 0);
  if constexpr (PAIR) load_q(b0, 0, 0);
  for (int k = 0; k < stages; ++k) {
#pragma unroll
    for (int sub = 0; sub < NSUB; ++sub) {
      const int gi = sub / NP, q = sub % NP;
      int lo = 0, hi = 0, buf = b1;
      if (sub < SPREAD) {
        lo = FIRST + sub * (DEP - FIRST) / SPREAD;
        hi = FIRST + (sub + 1) * (DEP - FIRST) / SPREAD;
      }
      if (sub == NSUB - 1) {
        // the next stage has landed, and nobody reads this one any more: its last fragments are in registers
        wait_deposits_and_reads<0>();
        __builtin_amdgcn_s_barrier();
        asm volatile("" ::: "memory");
        next_stage();
        lo = 0;
        hi = FIRST;
        buf = b0;
      }
#pragma unroll
      for (int i = 0; i < TI; ++i)
#pragma unroll
        for (int j = 0; j < TJ; ++j) {
          const int m = i * TJ + j, n = hi - lo;
          __builtin_amdgcn_sched_barrier(0);
          if (m == (TI * TJ > 1 ? 1 : 0)) {
            if (sub + 1 < NSUB) {
              if (q == NP - 1) load_a(b0, gi + 1);
              if (!PAIR || q == NP - 1) load_b(b0, sub + 1);
              if (PAIR && q == NP - 1) load_q(b0, gi + 1, 0);
            } else {
              load_a(b1, 0);
              load_b(b1, 0);
              if (PAIR) load_q(b1, 0, 0);
            }
          }
          if (PAIR && q < 2) {
#pragma unroll
            for (int t = 0; t < TJ; ++t)
              if (m == (t + 1 < TI * TJ ? t + 1 : TI * TJ - 1)) fb[(sub + 1) & 1][t] = widened(fq[t][0], fq[t][1]);
            if (q == 0 && m == (TJ < TI * TJ ? TJ : TI * TJ - 1)) load_q(b0, gi, 1);
          }
          issue(buf, lo + m * n / (TI * TJ), lo + (m + 1) * n / (TI * TJ));
          __builtin_amdgcn_sched_barrier(0);
          acc[q][i][j] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(bf16x8, fa[gi & 1][i]), __builtin_bit_cast(bf16x8, fb[sub & 1][j]), acc[q][i][j], 0, 0, 0);
        }
    }
    const int b = b0;
    b0 = b1;
    b1 = b;
  }

  // squared differences in fp64 (the layout and the order of wa_gemm_kernel's)
  double e[2] = {0.0, 0.0}, p = 0.0;
  const int row_lim = a.M - (m0 + wm * WM + 4 * g);
#pragma unroll
  for (int j = 0; j < TJ; ++j) {
    const int n = n0 + wn * WN + j * 32 + r;
    const bool col_ok = n < a.N;
    const int ns = a.w_per_channel && col_ok ? n : 0;
    const double c0 = static_cast<double>(a.sw[0][ns]), c1 = NP == 3 ? static_cast<double>(a.sw[1][ns]) : 0.0;
#pragma unroll
    for (int i = 0; i < TI; ++i)
#pragma unroll
      for (int x = 0; x < 16; ++x) {
        const bool ok = col_ok && (i * 32 + 8 * (x / 4) + (x % 4)) < row_lim;
        const double y = ok ? static_cast<double>(acc[0][i][j][x]) : 0.0;
        const double d0 = __builtin_fma(-c0, ok ? static_cast<double>(acc[1][i][j][x]) : 0.0, y);
        e[0] = __builtin_fma(d0, d0, e[0]);
        if constexpr (NP == 3) {
          const double d1 = __builtin_fma(-c1, ok ? static_cast<double>(acc[2][i][j][x]) : 0.0, y);
          e[1] = __builtin_fma(d1, d1, e[1]);
        }
        p = __builtin_fma(y, y, p);
      }
  }
  const double w[3] = {wave_sum(e[0]), wave_sum(e[1]), wave_sum(p)};
  wait_deposits_and_reads<0>();   // the unused deposits have landed: the sums lie over the stages
  __syncthreads();
  double (*const s_red)[NW] = reinterpret_cast<double (*)[NW]>(s_buf);
  if (lane < 3) s_red[lane][wave] = lane == 0 ? w[0] : (lane == 1 ? w[1] : w[2]);
  __syncthreads();
  if (tid < 3 && a.part[tid]) {
    double t = 0.0;
    for (int k = 0; k < NW; ++k) t += s_red[tid][k];   // fixed order
    a.part[tid][bm * a.tiles_n + bn] = t;
  }
}

using Large = Tile<256, 128, 64, 64>;    // one workgroup per compute unit, two waves per SIMD
using Medium = Tile<128, 128, 64, 64>;   // one, one wave per SIMD
using Small = Tile<64, 64, 32, 32>;      // three
template <int NQ, bool PAIR> using SharedLarge = SharedTile<256, 128, 64, 64, NQ, PAIR>;
template <int NQ, bool PAIR> using SharedMedium = SharedTile<128, 128, 64, 32, NQ, PAIR>;
template <int NQ, bool PAIR> using SharedSmall = SharedTile<64, 64, 32, 32, NQ, PAIR>;

}  // namespace

// The tile by the time a K step takes, in units of one of a full grid of large tiles, on the MI355X's 256 compute units (a
// number of its own here, not the current device's: the plan sets the size of the workspace and the order of the sums,
// which are the same wherever and whenever they are asked for): a round of
// large tiles 1, of medium ones 0.6, of small ones 0.38, 0.51 and 0.7 with one, two and three on a compute unit.
// Measured, layer selection with INT8 and exact E4M3 products, us, large / medium / small: tokens x rows x columns
// 2048 x 4096 x 4096 194 / 212 / 289; 1024 x 4096 x 4096 134 / 127 / 168; 777 x 3000 x 5056 155 / 121 / 159;
// 512 x 4096 x 4096 128 / 101 / 102; 384 x 4096 x 4096 126 / 99 / 95; 384 x 11008 x 4096 202 / 225 / 233;
// 1536 x 11008 x 4096 458 / 472 / 611; 1024 x 11008 x 4096 340 / 333 / 418.
// Up to 256 small tiles leave compute units idle, and a tile's three products follow each other: there the products and,
// with fewer tiles yet, parts of K are workgroups of their own and a second kernel takes the sums.  Small tiles
// whole / cut to 40 / to 20 stages: 64 x 1024 x 4096 (16 tiles) 66 / 40 / 38; 64 x 512 x 8192 (8) 96 / 42 / 41;
// 64 x 4096 x 4096 (64) 76 / 56 / 58; 128 x 4096 x 11008 (128) 217 / 166 / 182; 256 x 4096 x 11008 (256) 227 / 232 / 256,
// into the products alone 226; 256 x 1024 x 4096 (64) 65 / 42 / 43; 1024 x 1024 x 4096 (256) 71 / 69 / 73.  The second
// launch costs what short products save: 64 x 1024 x 1024 29.4 / - / 30.2, 128 x 8192 x 1024 40 / 44 / 44.
//
// Products that share X (wa_gemm_shared_kernel) take the same tiles, and are cut up to 160 small tiles only: into the products
// alone / whole 256 x 4096 x 4096 75.8 / 73.0 us, 300 x 3000 x 2048 45.1 / 43.9, 64 x 11008 x 2560 88.7 / 83.8, but 64 x 10240 x 2560
// (160 tiles) 77.7 / 81.6, 64 x 4096 x 2048 (64) 35.4 / 42.8.
constexpr int64_t kUnits = 256, kProductsOnly = 160;
WaPlan wa_gemm_plan(int64_t M, int64_t N, int64_t K, int64_t ldx, int64_t ldw) {
  auto tiles = [&](auto t) { using T = decltype(t); return ((M + T::TM - 1) / T::TM) * ((N + T::TN - 1) / T::TN); };
  const int64_t large = tiles(Large{}), medium = tiles(Medium{}), small = tiles(Small{});
  const int64_t stages = K / 64;
  // rows whose offsets fit 32 bits
  const int64_t rows = ((int64_t{1} << 32) - 1 - 2 * K) / (2 * std::max(std::max(ldx, ldw), K)) + 1;
  WaPlan p{};
  if (rows < Small::TM) {
    p.tile = WaPlan::kWide;
  } else {
    const auto rounds = [](int64_t n) { return static_cast<double>((n + kUnits - 1) / kUnits); };
    const double per_cu = rounds(small), t_large = rounds(large), t_medium = 0.6 * rounds(medium);
    const double t_small = per_cu == 1.0 ? 0.38 : (per_cu == 2.0 ? 0.51 : 0.235 * per_cu);
    p.tile = WaPlan::kSmall;
    if (rows >= Medium::TM && t_medium < t_small) p.tile = WaPlan::kMedium;
    if (rows >= Large::TM && t_large <= std::min(t_medium, t_small)) p.tile = WaPlan::kLarge;
  }
  p.blocks = static_cast<int>(p.tile == WaPlan::kLarge ? large : (p.tile == WaPlan::kMedium ? medium : small));
  if (p.tile == WaPlan::kSmall && small <= kUnits && stages >= 20) {
    // (at most 16 or 8 pieces of a product, which bounds the scratch: 40 MB or 64 MB)
    const int64_t run = small <= 48 ? std::max(std::min<int64_t>(20, (stages + 1) / 2), (stages + 15) / 16)
                                    : (small <= kProductsOnly ? std::max<int64_t>(40, (stages + 7) / 8) : stages);
    p.run = static_cast<int>(run);
    p.partial_bytes = static_cast<size_t>(3 * ((stages + run - 1) / run) * small) * (Small::TM * Small::TN * sizeof(float));
  }
  p.shared = p.tile != WaPlan::kWide && (p.run == 0 || p.blocks > kProductsOnly);
  return p;
}

namespace {

// Kernel arguments of a layer but for its tiles.
int gemm_args(const WaGemmParams& p, GemmArgs& a) {
  if (p.K % 64 != 0) return MOFQ_ERR_UNSUPPORTED;
  if (p.q[0].kind == WA_NONE) return MOFQ_ERR_INVALID_ARG;   // the first slot carries the Y^2 sum
  a = GemmArgs{};
  const int32_t lines8 = static_cast<int32_t>((p.K + 127) / 128), lines16 = static_cast<int32_t>(p.K / 64);
  a.seg[SEG_REF] = Segment{p.x, p.w, p.ldx * 2, p.ldw * 2, lines16, 0};
  for (int i = 0; i < 2; ++i) {
    const WaProduct& q = p.q[i];
    if ((q.xs != nullptr) != (q.ws != nullptr)) return MOFQ_ERR_INVALID_ARG;
    if (q.xs && q.kind != WA_FP8) return MOFQ_ERR_INVALID_ARG;
    if (q.kind == WA_NONE) continue;
    const bool eight = q.kind != WA_GRID_BF16 && q.kind != WA_PAIR_FP8;   // (a pair: two bytes a column)
    const int64_t row = eight ? p.K : 2 * p.K;
    a.seg[SEG_Q + 2 * i] = Segment{q.x, q.w, row, row, eight ? lines8 : lines16, eight && p.K % 128 != 0};
    if (q.xs) a.seg[SEG_SIDE + 2 * i] = Segment{q.xs, q.ws, 2 * SIDE_K, 2 * SIDE_K, 1, 0};
    a.sx[i] = q.sx;
    a.sw[i] = q.sw;
    a.part[i] = q.part;
  }
  a.w_per_channel = p.w_per_channel;
  a.M = static_cast<int32_t>(p.M); a.N = static_cast<int32_t>(p.N);
  a.part[2] = p.part_p;
  return MOFQ_OK;
}
// Products in pieces of up to `run` stages (of widened codes as many as the reference product's): returns their number.
int set_pieces(const WaGemmParams& p, GemmArgs& a, int run) {
  for (int q = 0; q < 3; ++q) {
    const int stages = q == 0 || p.q[q - 1].kind == WA_GRID_FP8 ? a.seg[SEG_REF].stages : a.seg[SEG_Q + 2 * (q - 1)].stages;
    a.piece0[q + 1] = a.piece0[q] + (stages + run - 1) / run;
  }
  a.partial = static_cast<float*>(p.partial);
  return a.piece0[3];
}
template <typename T> void set_tiles(const WaGemmParams& p, GemmArgs& a) {
  a.tiles_m = static_cast<int32_t>((p.M + T::TM - 1) / T::TM);
  a.tiles_n = static_cast<int32_t>((p.N + T::TN - 1) / T::TN);
}

}  // namespace

int launch_wa_gemm(const WaGemmParams& p, hipStream_t st) {
  GemmBatch<1> batch{};
  GemmArgs& a = batch.a[0];
  const int rc = gemm_args(p, a);
  if (rc != MOFQ_OK) return rc;
  const int k1 = p.q[0].kind, k2 = p.q[1].kind;
  const WaPlan plan = wa_gemm_plan(p.M, p.N, p.K, p.ldx, p.ldw);
  auto launch = [&](auto k1_c, auto k2_c) {
    constexpr int K1 = decltype(k1_c)::value, K2 = decltype(k2_c)::value;
    auto tiled = [&](auto tile_c, auto kernel, int pieces = 1) {
      using T = decltype(tile_c);
      set_tiles<T>(p, a);
      hipLaunchKernelGGL(kernel, dim3(static_cast<unsigned>(plan.blocks * pieces)), dim3(T::NW * 64), 0, st, batch);
    };
    auto shared = [&](auto tile_c, auto kernel) {
      using T = decltype(tile_c);
      set_tiles<T>(p, a);
      hipLaunchKernelGGL(kernel, dim3(static_cast<unsigned>(plan.blocks)), dim3(T::NW * 64), 0, st, a);
    };
    constexpr bool PAIR = K1 == WA_PAIR_FP8, SHARED = K1 == WA_GRID_BF16 || PAIR;
    if constexpr (SHARED) {   // all products take the unquantized X
      constexpr int NQ = K2 == WA_NONE ? 1 : 2;
      for (int i = 0; i < NQ; ++i)
        if (p.q[i].x != p.x || p.q[i].sx) return static_cast<int>(MOFQ_ERR_UNSUPPORTED);
      if (p.ldx != p.K) return static_cast<int>(MOFQ_ERR_UNSUPPORTED);
      if (PAIR && (!plan.shared || p.q[0].w != p.q[1].w)) return static_cast<int>(MOFQ_ERR_UNSUPPORTED);
      // (a single format where products are workgroups of their own, each a whole one: there the sums are the same, and
      // 256 x 4096 x 4096 takes 55.5 us instead of 63.4)
      if (NQ == 2 ? plan.shared : plan.shared && plan.run == 0) {
        switch (plan.tile) {
          case WaPlan::kLarge: shared(SharedLarge<NQ, PAIR>{}, wa_gemm_shared_kernel<SharedLarge<NQ, PAIR>>); break;
          case WaPlan::kMedium: shared(SharedMedium<NQ, PAIR>{}, wa_gemm_shared_kernel<SharedMedium<NQ, PAIR>>); break;
          default: shared(SharedSmall<NQ, PAIR>{}, wa_gemm_shared_kernel<SharedSmall<NQ, PAIR>>);
        }
        return hip_status(hipGetLastError());
      }
    }
    if constexpr (!PAIR) {
      if (plan.tile == WaPlan::kWide) {
        tiled(Small{}, wa_gemm_kernel<Small, K1, K2, false, true, 1>);
      } else if (plan.run) {
        tiled(Small{}, wa_gemm_kernel<Small, K1, K2, true, false, 1>, set_pieces(p, a, plan.run));
        hipLaunchKernelGGL((wa_pieces_kernel<Small, K1, K2, 1>), dim3(static_cast<unsigned>(plan.blocks)), dim3(Small::NW * 64), 0, st, batch);
      } else if constexpr (!SHARED) {
        switch (plan.tile) {
          case WaPlan::kLarge: tiled(Large{}, wa_gemm_kernel<Large, K1, K2, false, false, 1>); break;
          case WaPlan::kMedium: tiled(Medium{}, wa_gemm_kernel<Medium, K1, K2, false, false, 1>); break;
          default: tiled(Small{}, wa_gemm_kernel<Small, K1, K2, false, false, 1>);
        }
      }
    }
    return hip_status(hipGetLastError());
  };
#define MOFQ_WA(A, B) \
  if (k1 == (A) && k2 == (B)) return launch(std::integral_constant<int, A>{}, std::integral_constant<int, B>{});
  MOFQ_WA(WA_INT8, WA_GRID_FP8) MOFQ_WA(WA_INT8, WA_FP8) MOFQ_WA(WA_INT8, WA_NONE)
  MOFQ_WA(WA_GRID_BF16, WA_NONE) MOFQ_WA(WA_GRID_FP8, WA_NONE) MOFQ_WA(WA_FP8, WA_NONE) MOFQ_WA(WA_GRID_BF16, WA_GRID_BF16)
  MOFQ_WA(WA_PAIR_FP8, WA_PAIR_FP8)
#undef MOFQ_WA
  return MOFQ_ERR_UNSUPPORTED;
}

// Layers of one tile, with whole products or with pieces, share a launch, the longest loops first.
int launch_wa_gemms(const WaGemmParams* p, int n, hipStream_t st) {
  if (!p || n < 1 || n > kWaGroup) return MOFQ_ERR_INVALID_ARG;
  bool done[kWaGroup] = {};
  for (int kind = 0; kind < 4; ++kind) {
    const bool pieces = kind == 3;
    const int tile = kind == 0 ? WaPlan::kLarge : (kind == 1 ? WaPlan::kMedium : WaPlan::kSmall);
    int list[kWaGroup], m = 0;
    for (int i = 0; i < n; ++i) {
      const WaPlan plan = wa_gemm_plan(p[i].M, p[i].N, p[i].K, p[i].ldx, p[i].ldw);
      const bool pair = p[i].q[0].kind == WA_INT8 && (p[i].q[1].kind == WA_FP8 || p[i].q[1].kind == WA_GRID_FP8) && p[i].q[1].kind == p[0].q[1].kind;
      if (plan.tile == tile && (plan.run > 0) == pieces && pair) list[m++] = i;
    }
    if (m < 2) continue;
    std::stable_sort(list, list + m, [&](int i, int j) { return p[i].K > p[j].K; });
    GemmBatch<kWaGroup> batch{};
    static_assert(sizeof(batch) <= 4096, "kernel arguments");
    int64_t blocks = 0, sums = 0;
    int32_t first_sum[kWaGroup];
    for (int i = 0; i < kWaGroup; ++i) batch.first[i] = first_sum[i] = INT32_MAX;
    for (int i = 0; i < m; ++i) {
      const int rc = gemm_args(p[list[i]], batch.a[i]);
      if (rc != MOFQ_OK) return rc;
      const WaGemmParams& q = p[list[i]];
      const int n_pieces = pieces ? set_pieces(q, batch.a[i], wa_gemm_plan(q.M, q.N, q.K, q.ldx, q.ldw).run) : 1;
      switch (tile) {
        case WaPlan::kLarge: set_tiles<Large>(p[list[i]], batch.a[i]); break;
        case WaPlan::kMedium: set_tiles<Medium>(p[list[i]], batch.a[i]); break;
        default: set_tiles<Small>(p[list[i]], batch.a[i]);
      }
      const int64_t tiles = static_cast<int64_t>(batch.a[i].tiles_m) * batch.a[i].tiles_n;
      batch.first[i] = static_cast<int32_t>(blocks);
      first_sum[i] = static_cast<int32_t>(sums);
      blocks += tiles * n_pieces;
      sums += tiles;
    }
    if (blocks >= (int64_t{1} << 31)) continue;
    auto launch = [&](auto k2_c) {
      constexpr int K2 = decltype(k2_c)::value;
      const dim3 grid(static_cast<unsigned>(blocks));
      if (pieces) {
        hipLaunchKernelGGL((wa_gemm_kernel<Small, WA_INT8, K2, true, false, kWaGroup>), grid, dim3(Small::NW * 64), 0, st, batch);
        std::copy(first_sum, first_sum + kWaGroup, batch.first);
        hipLaunchKernelGGL((wa_pieces_kernel<Small, WA_INT8, K2, kWaGroup>), dim3(static_cast<unsigned>(sums)), dim3(Small::NW * 64), 0, st, batch);
        return;
      }
      switch (tile) {
        case WaPlan::kLarge: hipLaunchKernelGGL((wa_gemm_kernel<Large, WA_INT8, K2, false, false, kWaGroup>), grid, dim3(Large::NW * 64), 0, st, batch); break;
        case WaPlan::kMedium: hipLaunchKernelGGL((wa_gemm_kernel<Medium, WA_INT8, K2, false, false, kWaGroup>), grid, dim3(Medium::NW * 64), 0, st, batch); break;
        default: hipLaunchKernelGGL((wa_gemm_kernel<Small, WA_INT8, K2, false, false, kWaGroup>), grid, dim3(Small::NW * 64), 0, st, batch);
      }
    };
    if (p[0].q[1].kind == WA_FP8) launch(std::integral_constant<int, WA_FP8>{});
    else launch(std::integral_constant<int, WA_GRID_FP8>{});
    if (hipGetLastError() != hipSuccess) return MOFQ_ERR_HIP;
    for (int i = 0; i < m; ++i) done[list[i]] = true;
  }
  for (int i = 0; i < n; ++i)
    if (!done[i]) {
      const int rc = launch_wa_gemm(p[i], st);
      if (rc != MOFQ_OK) return rc;
    }
  return MOFQ_OK;
}

}  // namespace mofq
