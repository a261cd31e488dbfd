// mfma2.hip -- 2-way tallies on the matrix cores (fp4 or int8 operands): the
// one-shot kernels over the triangle (ccc_2way) or the rectangle
// (ccc_2way_block).  The tile bodies and their design notes are in tile2o.h
// (fp4, on the operands of the pre-pass) and tile2.h (packed rows: int8, and
// fp4 where the operands find no room).
#include "tile2.h"
#include "tile2o.h"

namespace ccc {

namespace {

// *flag = id if some row of A or B misses an entry, else 0 (one workgroup;
// its threads read the counts with a stride).  For calls on packed rows; the
// pre-pass of the operands sets the flag itself.
__global__ __launch_bounds__(1024) void complete_flag_kernel(const int32_t* __restrict__ ca,
                                                             int64_t n_a,
                                                             const int32_t* __restrict__ cb,
                                                             int64_t n_b, int64_t n_f,
                                                             unsigned long long* __restrict__ flag,
                                                             unsigned long long id) {
  bool ok = n_f > 0;
  for (int64_t r = threadIdx.x; r < n_a && ok; r += blockDim.x)
    ok = reinterpret_cast<const v4i*>(ca)[r].z == n_f;
  for (int64_t r = threadIdx.x; r < n_b && ok; r += blockDim.x)
    ok = reinterpret_cast<const v4i*>(cb)[r].z == n_f;
  ok = __syncthreads_and(ok ? 1 : 0) != 0;
  if (threadIdx.x == 0) *flag = ok ? 0ull : id;
}

// Tile index of this workgroup (launch_slices): the XCDs take contiguous runs.
__device__ __forceinline__ int64_t launch_tile(const Pair2Args& a) {
  return a.tile_base + xcd_unit(blockIdx.x, gridDim.x);
}

// Launch a kernel over `tiles` workgroups of 256 threads.
template <typename Kernel, typename... Rest>
hipError_t launch_tiles(Kernel kernel, int64_t tiles, Pair2Args a, hipStream_t stream,
                        Rest... rest) {
  if (tiles > 0x7FFFFFFF) return hipErrorInvalidValue;
  return launch_slices(tiles, 256, [&](int64_t base, dim3 grid) {
    a.tile_base = base;
    hipLaunchKernelGGL(kernel, grid, dim3(256), 0, stream, a, rest...);
  });
}

// Workgroup tile (I, J) of `b` in a grid of tiles of BM x BN pairs.  A
// triangle is cut into squares of the larger side, each a few whole tiles,
// the squares in strips of H square rows.
template <int BM, int BN, int H = kStripRows>
__device__ __forceinline__ void tile_of(const Pair2Args& a, int64_t b, int64_t tiles_side,
                                        int64_t tiles_n, int64_t& I, int64_t& J) {
  constexpr int S = BM > BN ? BM : BN, PARTS = S / (BM > BN ? BN : BM);
  static_assert(S % BM == 0 && S % BN == 0, "a square splits into whole tiles");
  if (a.tri) {
    int64_t sq_i, sq_j;
    strip_square(b / PARTS, tiles_side, a.row_begin / S, (a.row_end + S - 1) / S, sq_i, sq_j, H);
    I = BM < BN ? PARTS * sq_i + b % PARTS : sq_i;
    J = BM < BN ? sq_j : PARTS * sq_j + b % PARTS;
  } else {
    I = b / tiles_n;
    J = b % tiles_n;
  }
}

// Square rows per strip of the complete-data kernels' triangle order, whose
// squares are twice the height of the general kernel's.  On operands, strips of
// 2 / 4 / 8 take 16384 x 8000 1.78 / 1.87 / 1.85 ms, 16000 x 40000 2.81 / 2.88 /
// 2.86, 32768 x 65536 15.33 / 15.44 / 15.72 (one run each, which differ by up to
// 3%).
constexpr int kCompleteStripRows = 4;
// ... and of the kernels on operands: fewer rows in flight than the packed
// kernel's strips of 8 write their output in fewer, longer runs (16384 x
// 2000: 1.62 -> 1.55 ms, 16384 x 32768: 5.81 -> 5.66 ms; with 2 the latter
// takes 5.90 ms).
constexpr int kOperandStripRows = 4;

// Calls whose every row is complete: 2 x 2 waves of (16 WM) x (16 WN) pairs
// (mfma2_complete_wave_tile); a workgroup exits at once when the flag says
// that some row is not complete (mfma2_kernel then covers the call).
template <int WM, int WN, bool F4>
__global__ __launch_bounds__(256, 2) void mfma2_complete_kernel(Pair2Args a,
                                                                int64_t tiles_side,
                                                                int64_t tiles_n) {
  if (*a.flag == a.id) return;  // uniform: some row is not complete
  constexpr int BM = 32 * WM, BN = 32 * WN, NB = 2 * WM + 2 * WN;
  const int wave = threadIdx.x >> 6;
  int64_t I, J;
  tile_of<BM, BN, kCompleteStripRows>(a, launch_tile(a), tiles_side, tiles_n, I, J);
  __shared__ u4 stage[2][NB][64];
  __shared__ u4 outs[4][128];
  tile2::mfma2_complete_wave_tile<WM, WN, F4>(a, I * BM + (wave & 1) * 16 * WM,
                                              J * BN + (wave >> 1) * 16 * WN, stage, outs[wave]);
}

// The general kernel: 2 x 2 waves of (16 WM) x (16 WN) pairs.  Workgroups
// of the 128 x 64 shape whose rows are all complete compute their tile
// together in the one-plane form (mfma2_coop_complete).
template <int WM, int WN, bool F4, int MIN_WG>
__global__ __launch_bounds__(256, MIN_WG) void mfma2_kernel(Pair2Args a, int64_t tiles_side,
                                                            int64_t tiles_n) {
  if (a.flag && *a.flag != a.id) return;  // uniform: mfma2_complete_kernel covers the call
  constexpr int BM = 32 * WM, BN = 32 * WN, NB = 2 * WM + 2 * WN;
  constexpr bool kCoop = WM == 4 && WN == 2;
  const int wave = threadIdx.x >> 6;
  // XCD-contiguous runs of tiles (triangle: in strip order, so that a run
  // shares row and column blocks in one L2)
  int64_t I, J;
  tile_of<BM, BN>(a, launch_tile(a), tiles_side, tiles_n, I, J);
  // the cooperative form's partial tiles (64 KB), or else the workgroup's
  // two stage buffers of NB row blocks
  __shared__ u4 smem[kCoop ? 4 * 16 * 64 : 2 * NB * 64];
  static_assert(sizeof(smem) >= 2 * NB * 64 * sizeof(u4), "stage buffers fit");
  if constexpr (kCoop) {
    if (tile2::workgroup_complete<WM, WN>(a, I * BM, J * BN)) {
      tile2::mfma2_coop_complete<WM, WN, F4>(a, I * BM, J * BN,
                                             reinterpret_cast<v4i(*)[16][64]>(smem));
      return;
    }
  }
  tile2::mfma2_wave_tile<WM, WN, F4>(a, I * BM + (wave & 1) * 16 * WM,
                                     J * BN + (wave >> 1) * 16 * WN,
                                     reinterpret_cast<u4(*)[NB][64]>(smem));
}

// Calls whose every row is complete, on operands (tile2o.h).
template <tile2::Out OUT, int WM, int WN>
__global__ __launch_bounds__(256, 2) void mfma2_complete_operand_kernel(Pair2Args a,
                                                                        int64_t tiles_side,
                                                                        int64_t tiles_n) {
  if (*a.flag == a.id) return;  // uniform: some row is not complete
  constexpr int BM = 32 * WM, BN = 32 * WN;
  int64_t I, J;
  tile_of<BM, BN, kCompleteStripRows>(a, launch_tile(a), tiles_side, tiles_n, I, J);
  __shared__ u4 stage[3][2 * WM + 2 * WN][64];
  tile2::complete_tile<OUT, WM, WN>(a, I * BM, J * BN, stage);
}

// The general kernel on operands: workgroup tiles of (32 WM) x (32 WN).
template <tile2::Out OUT, int WM, int WN, int MIN_WG>
__global__ __launch_bounds__(256, MIN_WG) void mfma2_operand_kernel(Pair2Args a,
                                                                    int64_t tiles_side,
                                                                    int64_t tiles_n) {
  if (a.flag && *a.flag != a.id) return;  // uniform: the complete-data kernel covers the call
  constexpr int BM = 32 * WM, BN = 32 * WN;
  int64_t I, J;
  tile_of<BM, BN, kOperandStripRows>(a, launch_tile(a), tiles_side, tiles_n, I, J);
  __shared__ u4 stage[3][2 * WM + 2 * WN][64];
  tile2::staged_tile<OUT, WM, WN>(a, I * BM, J * BN, stage);
}

// The field-split kernel on operands: 32 x 32 tiles, each by `splits`
// workgroups that take a share of the super-steps.  With one, the workgroup
// emits its tile; with more, the partial sums go to a.part, [tile][split]
// [block][plane][lane], and mfma2_split_finish_kernel adds and emits them.
using tile2::kSplitTile;
__device__ __forceinline__ void split_tile_of(const Pair2Args& a, int64_t t, int64_t tiles_side,
                                              int64_t tiles_n, int64_t& I0, int64_t& J0) {
  int64_t I, J;
  tile_of<kSplitTile, kSplitTile, kOperandStripRows>(a, t, tiles_side, tiles_n, I, J);
  I0 = I * kSplitTile;
  J0 = J * kSplitTile;
}

using tile2::SplitSides;

template <tile2::Out OUT>
__global__ __launch_bounds__(256, 3) void mfma2_split_kernel(Pair2Args a, int64_t tiles_side,
                                                             int64_t tiles_n, int splits,
                                                             int complete_only) {
  if (complete_only && *a.flag == a.id) return;  // uniform: another kernel covers the call
  __shared__ v4i red[4][4][64];
  __shared__ SplitSides sides;
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const int64_t b = launch_tile(a), t = b / splits;
  const int sp = (int)(b % splits);
  int64_t I0, J0;
  split_tile_of(a, t, tiles_side, tiles_n, I0, J0);
  if (splits == 1 && threadIdx.x >= 192)  // one wave; the barriers of the sums cover it
    tile2::load_sides<OUT>(a, I0, J0, sides, threadIdx.x - 192, 64);
  tile2::split_tile(
      a, I0, J0, a.steps * sp / splits, a.steps * (sp + 1) / splits, red,
      [&] { return tile2::wave_complete<kSplitTile, kSplitTile>(a, I0, J0); },
      [&](auto general, const auto& s) {
        if (splits == 1) {
          tile2::split_emit<OUT, general.value>(a, I0, J0, s, sides);
        } else {
          v4i* part = reinterpret_cast<v4i*>(a.part) + ((b * 4 + wave) * 4) * 64 + lane;
          tile2::static_for<general.value ? 4 : 1>(
              [&](auto p) { part[64 * p.value] = s[0][p.value]; });
        }
      });
}

template <tile2::Out OUT>
__global__ __launch_bounds__(256) void mfma2_split_finish_kernel(Pair2Args a, int64_t tiles_side,
                                                                 int64_t tiles_n, int splits) {
  __shared__ SplitSides sides;
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const int64_t t = launch_tile(a);
  int64_t I0, J0;
  split_tile_of(a, t, tiles_side, tiles_n, I0, J0);
  const bool whole = tile2::wave_complete<kSplitTile, kSplitTile>(a, I0, J0);
  tile2::load_sides<OUT>(a, I0, J0, sides, threadIdx.x, 256);
  __syncthreads();
  const v4i* part = reinterpret_cast<const v4i*>(a.part) + ((t * splits * 4 + wave) * 4) * 64 + lane;
  auto run = [&](auto general, auto& s) {
    constexpr int NP = general.value ? 4 : 1;
    tile2::static_for<NP>([&](auto p) { s[0][p.value] = part[64 * p.value]; });
#pragma unroll 4
    for (int k = 1; k < splits; ++k)
      tile2::static_for<NP>([&](auto p) { s[0][p.value] += part[(k * 16 + p.value) * 64]; });
    tile2::split_emit<OUT, general.value>(a, I0, J0, s, sides);
  };
  if (whole) {
    v4i s[1][1];
    run(std::false_type{}, s);
  } else {
    v4i s[1][4];
    run(std::true_type{}, s);
  }
}

// Grid of BM x BN workgroup tiles: tiles along a side (rows, columns; for a
// triangle squares) and the tile count (triangle: the squares of the row
// range, a few tiles each); 0 tiles when there is nothing to do.
template <int BM, int BN>
int64_t tile_grid(const Pair2Args& a, int64_t& tm, int64_t& tn) {
  constexpr int S = BM > BN ? BM : BN, PARTS = S / (BM > BN ? BN : BM);
  if (!a.tri) {
    tm = (a.n_a + BM - 1) / BM;
    tn = (a.n_b + BN - 1) / BN;
    return tm * tn;
  }
  tm = tn = (a.n_a + S - 1) / S;
  const int64_t s0 = a.row_begin / S, s1 = (a.row_end + S - 1) / S;
  return PARTS * (s1 * tm - s1 * (s1 - 1) / 2 - (s0 * tm - s0 * (s0 - 1) / 2));
}

template <int WM, int WN, bool F4, int MIN_WG>
hipError_t launch_shape(const Pair2Args& a, hipStream_t stream) {
  int64_t tm, tn;
  const int64_t ntiles = tile_grid<32 * WM, 32 * WN>(a, tm, tn);
  return launch_tiles(mfma2_kernel<WM, WN, F4, MIN_WG>, ntiles, a, stream, tm, tn);
}

// Shapes of the general kernel, picked per call by the kernel-shape table
// (kind oneshot): 0 = 128 x 64 workgroup tiles (waves 64 x 32), 1 = 64 x 32
// (32 x 16), 2 = 64 x 64 (32 x 32).  Smaller tiles give small calls more
// workgroups.
constexpr int kOneShotVariants = 3;

template <bool F4>
hipError_t launch_general(const Pair2Args& a, hipStream_t stream) {
  const int64_t n = a.n_a > a.n_b ? a.n_a : a.n_b;
  switch (tune_pick(kTuneOneShot, n, a.n_f, kOneShotVariants).variant) {
    case 1: return launch_shape<2, 1, F4, 4>(a, stream);
    case 2: return launch_shape<2, 2, F4, 2>(a, stream);
    default: return launch_shape<4, 2, F4, 2>(a, stream);
  }
}

// The complete-data kernel's wave tile: 128 x 64 pairs (8 x 4 blocks of 16).
constexpr int kCWM = 8, kCWN = 4;
// ... and on operands: 64 x 128, for the longer stretches of a row.
constexpr int kCOM = 4, kCON = 8;

template <bool F4>
hipError_t launch_complete(const Pair2Args& a, hipStream_t stream) {
  int64_t tm, tn;
  const int64_t ntiles = tile_grid<32 * kCWM, 32 * kCWN>(a, tm, tn);
  return launch_tiles(mfma2_complete_kernel<kCWM, kCWN, F4>, ntiles, a, stream, tm, tn);
}

template <bool F4>
hipError_t launch_f(const Pair2Args& a, hipStream_t stream) {
  if (a.flag) {
    // the flag first, then both kernels: each exits at once unless the flag
    // picks it
    hipLaunchKernelGGL(complete_flag_kernel, dim3(1), dim3(1024), 0, stream, a.counts_a, a.n_a,
                       a.counts_b, a.n_b, a.n_f, a.flag, a.id);
    hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
    if ((e = launch_complete<F4>(a, stream)) != hipSuccess) return e;
  }
  return launch_general<F4>(a, stream);
}

// Shapes on operands: 0 = 64 x 128 staged tiles, 1 = field-split 32 x 32
// tiles, 2 = 64 x 64 staged tiles, 3 = the packed rows' kernel (the
// complete-data kernel on operands all the same).
struct OperandShape {
  int variant;
  int splits;  // workgroups per tile (variant 1)
};

int64_t split_tiles(const Pair2Args& a, int64_t& tm, int64_t& tn) {
  return tile_grid<kSplitTile, kSplitTile>(a, tm, tn);
}

OperandShape operand_shape(const Pair2Args& a) {
  int64_t tm, tn;
  const int64_t tiles = split_tiles(a, tm, tn);
  OperandShape s{0, 1};
  const int forced = tune_forced_oneshot(kOneShotVariants);
  if (forced >= 0 && a.n_f <= tile2::kStagedMaxFields)
    s.variant = forced;
  else
    s.variant = operand_variant(tiles, a.n_f, a.tri && a.ccc && !a.sel.count,
                                a.sel.count || a.accumulate);
  if (s.variant == 1 && tiles > 0) {
    // Enough workgroups for two per CU, but no share below 16 super-steps:
    // the sums' way through memory and the second launch cost about 5 us
    // (384 x 250007: 173 us with 1 split, 94 with 3, 83 with 6, 85 with 12;
    // 700 x 50000: 48, 44 with 2, 46 with 6; 700 x 5000: 18, 20 with 2).
    int64_t n = 512 / tiles < a.steps / 16 ? 512 / tiles : a.steps / 16;
    if (const int forced = tune_forced_split(); forced > 0) n = forced < a.steps ? forced : a.steps;
    s.splits = n > 1 ? (int)n : 1;
  }
  return s;
}

template <tile2::Out OUT, int WM, int WN, int MIN_WG>
hipError_t launch_operand_shape(const Pair2Args& a, hipStream_t stream) {
  int64_t tm, tn;
  const int64_t ntiles = tile_grid<32 * WM, 32 * WN>(a, tm, tn);
  return launch_tiles(mfma2_operand_kernel<OUT, WM, WN, MIN_WG>, ntiles, a, stream, tm, tn);
}

template <tile2::Out OUT>
hipError_t launch_split(const Pair2Args& a, int splits, hipStream_t stream,
                        bool complete_only = false) {
  int64_t tm, tn;
  const int64_t ntiles = split_tiles(a, tm, tn);
  const hipError_t e =
      launch_tiles(mfma2_split_kernel<OUT>, ntiles * splits, a, stream, tm, tn, splits,
                   complete_only ? 1 : 0);
  if (e != hipSuccess || splits == 1) return e;
  return launch_tiles(mfma2_split_finish_kernel<OUT>, ntiles, a, stream, tm, tn, splits);
}

// Whether the complete-data tiles stream their tables.  Long fields bind them by
// their operand reads, which a plain output stream pushes out of L2; short
// ones by the output, whose lines plain stores let L2 join (triangles, plain /
// streamed: 16000 x 40000 3.20 / 2.87 ms, 16384 x 16384 2.26 / 2.19, 16384 x
// 2000 1.71 / 2.06).  In a rectangle whose rows start on multiples of 64 bytes
// there is little to join (us, 12000 x 12000: x 1500 1356 / 1386, x 3000 1430 /
// 1412, x 4000 1470 / 1391, x 9000 1649 / 1511; 12000 x 12004 x 4000 1570 / 1504;
// but 12000 x 12001 x 4000 1825 / 2131).
bool stream_tables(const Pair2Args& a) {
  return a.n_f >= (!a.tri && a.n_b % 4 == 0 ? 3000 : 12288);
}

// Whether complete data takes the 32 x 32 tiles where other data takes the
// staged ones: as long as the 128 x 256 one-plane tiles are few, or short and
// bound by CCC rows (us, complete data, 32 x 32 / 128 x 256 tiles: 1700 x 1700 x
// 1000 38 / 48, x 9000 65 / 80, 2200 x 2200 x 4000 equal; selection 3000 x 1000 42 /
// 48, 2400 x 16000 63 / 108, but 5000 x 1000 93 / 63; tables alone 2400 x 16000 60 /
// 91, 3000 x 1000 38 / 33, 3200 x 16000 86 / 99; with CCC 6000 x 6000 x 1000 310 /
// 362, x 2000 375 / 373, 4000 x 32000 x 1000 0.84 of the time, but 4096 x 50000 x 1000
// 2306 / 1955 and 1000000 x 200 x 1000 2720 / 2135).
bool complete_by_split(const Pair2Args& a, int64_t tiles) {
  if (a.sel.count) return tiles < 6000;
  if (!a.ccc) return tiles < 4000 || (tiles < 6000 && a.n_f > 8192);
  return tiles < 6000 ||
         (a.n_f <= 1024 && (a.tri || (a.n_a <= 65536 && a.n_b <= 40000)));
}

template <tile2::Out OUT>
hipError_t launch_operand_kernels(Pair2Args a, hipStream_t stream) {
  OperandShape s = operand_shape(a);
  int64_t tm, tn;
  if (s.variant == 1 && s.splits > 1 && mfma2_part_bytes(a) > a.part_bytes) s.splits = 1;
  if (s.variant == 1) return launch_split<OUT>(a, s.splits, stream);  // its tiles vote
  if constexpr (OUT != tile2::kAccumulate) {  // (whose counts are running totals)
    hipError_t e = hipSuccess;
    if (complete_by_split(a, split_tiles(a, tm, tn))) {
      e = launch_split<OUT>(a, 1, stream, true);
    } else {
      const int64_t n = tile_grid<32 * kCOM, 32 * kCON>(a, tm, tn);
      auto* kernel = mfma2_complete_operand_kernel<OUT, kCOM, kCON>;
      if constexpr (OUT == tile2::kDense)
        if (stream_tables(a)) kernel = mfma2_complete_operand_kernel<tile2::kStream, kCOM, kCON>;
      e = launch_tiles(kernel, n, a, stream, tm, tn);
    }
    if (e != hipSuccess) return e;
  }
  return s.variant == 3   ? launch_general<true>(a, stream)
         : s.variant == 2 ? launch_operand_shape<OUT, 2, 2, 4>(a, stream)
                          : launch_operand_shape<OUT, 2, 4, 2>(a, stream);
}

hipError_t launch_operands_out(const Pair2Args& a, hipStream_t stream) {
  if (a.sel.count) return launch_operand_kernels<tile2::kSelect>(a, stream);
  if (a.accumulate) return launch_operand_kernels<tile2::kAccumulate>(a, stream);
  return launch_operand_kernels<tile2::kDense>(a, stream);
}

}  // namespace

// The shape by the number of 32 x 32 tiles (n^2 / 2048 for a triangle) and
// fields, from timings of whole calls.  Small tiles give a small call more
// workgroups and a shorter chain each; large ones read their operands less
// often.
//
// Dense triangles with CCC rows (us for shapes 1 / 2 / 0, 1% missing): 1500 x
// 9000 39 / 51 / 56, 2600 x 6000 69 / 65 / 70, 2600 x 20000 128 / 134 / 144,
// 3500 x 4000 92 / 94 / 105, 4500 x 15000 273 / 249 / 298, 8000 x 10000 656 /
// 569 / 586, 12000 x 4000 980 / 893 / 872, 16384 x 32768 6570 / 5880 / 5660.
// With very short fields such a call is its output, 48 bytes a pair in rows
// that start anywhere in a line, and the 32 x 32 tiles, one block per wave,
// start storing at once: 12000 x 1000 719 / 862 / 835, complete data 9000 x
// 1000 406 / 536 / 547.
//
// Every other form puts out less (selections, tables alone), reads what it
// adds to, or writes rows of a rectangle that start on whole 16 bytes times
// n_b, so the operands' reads weigh more, however short the fields: selection
// 3000 x 300 48 / 32 / 38, 30000 x 1000 3547 / 1814 / 1988, 2400 x 300 34 / 24,
// but 2100 x 20000 89 / 109; tables alone 4000 x 1000 67 / 38 / 47; rectangles
// 4000 x 1024 x 4000 77 / 62 / 64, 256 x 1000000 x 1000 3528 / 2590 / 2585;
// accumulating 8000 x 8000 x 256 616 / 400 / 546, 8000 x 8000 x 8192 1076 /
// 783 / 934, but 1500 x 1500 x 8192 49 / 57 / 71.  Selections and accumulating
// calls (`mixed`) keep the 64 x 64 tile for longer: 12000 x 12000 x 8192
// accumulating 2418 / 1836 / 2061, selection 12000 x 8009 957 / 1000 (2 / 0).
int operand_variant(int64_t tiles, int64_t n_f, bool dense_ccc, bool mixed) {
  // Past kStagedMaxFields fields the staged tiles' sums are not exact.  Those of
  // the field-split tiles are, each wave having a quarter of the fields, but
  // many such tiles read the operands too often, while the packed rows' kernel
  // and the one-plane tiles of complete data stay exact to kF4MaxFields (ms,
  // field-split / packed: 2000 rows x 1,900,000 6.8 / 11.2, 3000 rows 13.9 /
  // 15.6, 12000 x 4,000,000 500 / 365; complete data, field-split / packed /
  // one-plane tiles on operands: 2000 x 1,900,000 5.1 / 9.0, 3000 x 1,900,000
  // 13.4 / 9.1 / 7.5, 12000 x 4,000,000 567 / 156 / 119).
  if (n_f > tile2::kStagedMaxFields) return tiles < 3000 ? 1 : 3;
  if (dense_ccc ? tiles < 6000 || n_f <= 1024 : tiles < 2500) return 1;
  return tiles < 50000 || (mixed && n_f < 16384) ? 2 : 0;
}

bool operands_serve(const Pair2Args& a) {
  int64_t tm, tn;
  return !a.accumulate || operand_variant(split_tiles(a, tm, tn), a.n_f, false, true) != 3;
}

size_t mfma2_part_bytes(const Pair2Args& a) {
  const OperandShape s = operand_shape(a);
  if (s.variant != 1 || s.splits == 1) return 0;
  int64_t tm, tn;
  return (size_t)(split_tiles(a, tm, tn) * s.splits) * 16 * 64 * sizeof(v4i);
}

hipError_t launch_mfma2(const Pair2Args& a, hipStream_t stream) {
  if (a.flag && a.accumulate) return hipErrorInvalidValue;
  timing_begin("mfma2", stream);
  const hipError_t e = a.f4 ? (a.za ? launch_operands_out(a, stream) : launch_f<true>(a, stream))
                            : launch_f<false>(a, stream);
  timing_end(stream);
  return e;
}

}  // namespace ccc
