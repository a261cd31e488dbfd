// kernels.h -- host-side launchers of the CCC kernels (internal to the library).
#pragma once

#include <hip/hip_runtime.h>
#include <math.h>
#include <stdint.h>

namespace ccc {

// Threshold selection: instead of dense tables, keep every pair (triple)
// with a CCC value >= threshold as (index, CCC values[, table]) records at
// slots taken from a device counter; slots past `cap` are counted, not stored.
struct Select {
  unsigned long long* count;  // device counter (zeroed before the tally kernel)
  int64_t cap;
  double threshold;
  int64_t* index;             // [cap] pair (triple) index
  double* ccc;                // [cap][4] or [cap][8]
  int32_t* tables;            // [cap][4] or [cap][8], may be null
};

// Arguments of one 2-way tally launch: either the upper triangle (i < j) of
// one vector set (tri = 1, va == vb) or the full rectangle A x B (tri = 0).
struct Pair2Args {
  const uint8_t* va;
  int64_t lda, n_a;
  const uint8_t* vb;
  int64_t ldb, n_b;
  int64_t n_f;
  int f4;                     // MFMA operands: fp4 (1, needs n_f <= kF4MaxFields) or int8 (0)
  int tri;
  int accumulate;             // tables += result (rectangle only)
  int32_t* tables;            // may be null when ccc is set
  double* ccc;                // may be null
  const int32_t* counts_a;    // [n_a][4]
  const int32_t* counts_b;    // [n_b][4]
  // this call's own 1-way counts of its n_f fields (the same arrays as
  // counts_a / counts_b unless accumulating, where those are running totals)
  const int32_t* chunk_a;
  const int32_t* chunk_b;
  double gamma;
  // rows of A whose pairs are produced; pair (i, j) goes to entry p(i,j) - p_base
  int64_t row_begin, row_end;
  int64_t p_base;
  int64_t sq_offset;          // first square tile of the row range (triangle)
  int64_t tile_base;          // tile of the launch's first workgroup (launch_slices)
  Select sel;                 // threshold selection (sel.count != null) instead of dense output
  // Device flag that holds `id` when some row of A or B misses an entry (any
  // other value: every row has all n_f fields present); null: no such check
  // (each tile votes for itself).  Only for calls that do not accumulate.
  unsigned long long* flag;
  unsigned long long id;
  // The rows as operands (operands.h), in super-steps of 256 fields; null:
  // the kernels read the packed rows.
  const void* za;
  const void* zb;
  int64_t steps;
  // Workspace for the partial sums of field-split tiles, and its size
  void* part;
  size_t part_bytes;
};

// Rows for which the pre-pass of the fp4 kernels writes operands and counts.
struct OperandSet {
  const uint8_t* v;
  int64_t ld, n;
  uint32_t blocks;  // (n + 15) / 16, or 0: no such set
  uint32_t first;   // first block to lay out; those before are only counted
  void* z;          // [blocks - first][steps][1024 bytes]
  int32_t* counts;  // [n][4] or null; added to when accumulating
  int32_t* chunk;   // [n][4] or null: this call's own counts
};
struct OperandJob {
  OperandSet set[2];
  int64_t n_f, steps;  // steps = ceil(n_f / 256)
  int accumulate;
  unsigned long long* zero;  // a counter to clear, or null
  unsigned long long* flag;  // set to `id` when some row misses an entry, or null
  unsigned long long id;
  int shares;  // workgroups along the fields of a block (one set only; see below)
  int2* part;  // [shares][n]: their counts, when shares > 1
};
inline int64_t operand_steps(int64_t n_f) { return (n_f + 255) / 256; }
inline int64_t operand_blocks(int64_t n) { return (n + 15) / 16; }
inline int64_t operand_bytes(int64_t n, int64_t n_f) {
  return operand_blocks(n) * operand_steps(n_f) * 1024;
}

// HIP launches fewer than 2^32 work-items along a dimension, so a kernel with
// more is launched in slices: launch(first workgroup, workgroups), in order.
// Slices are whole multiples of 2048 workgroups, which keeps the kernels'
// mapping of workgroups to XCDs.
constexpr int64_t slice_workgroups(int threads) { return 0xFFFFFFFFll / threads / 2048 * 2048; }
template <typename Launch>
hipError_t launch_slices(int64_t count, int threads, Launch launch) {
  const int64_t most = slice_workgroups(threads);
  for (int64_t base = 0; base < count; base += most) {
    launch(base, dim3((unsigned)(count - base < most ? count - base : most)));
    const hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
  }
  return hipSuccess;
}

// Largest n_f for which the MFMA kernels may take fp4 operands (their fp32
// sums of quarter-multiples, at most n_f, stay exact); int8 beyond.
constexpr int64_t kF4MaxFields = int64_t(1) << 22;

// Row tile of the 3-way work units (one-j units and the complete-data
// kernel's runs), and of the fp4 general kernel's runs of middle vectors.
constexpr int64_t kUnitTile = 64;
constexpr int64_t kRunTile = 32;

// Tetrahedral work units of the 3-way kernels.  Rows are cut into b-row
// tiles; a unit is (I tile it, K tile kt, middle vectors j .. j + run - 1)
// with it <= kt and covers every triple i < j < k with i in tile it (and in
// the staged range [i_begin, i_end)) and k in tile kt, for its run of
// consecutive middle vectors (cut from the pair's j range; the last run of
// a pair may be shorter).  Units are ordered by tile pair (it major, then
// kt) and, within a pair, by j: consecutive units share both row tiles, so
// a run of them on one XCD reads the tiles from its L2 once.
struct UnitGrid {
  int64_t n, b, i_begin, i_end;
  int64_t it0, it1;  // I tiles [it0, it1)
  int64_t nt;        // tiles of all n rows
  int64_t run;       // middle vectors per unit
};

__host__ __device__ __forceinline__ UnitGrid unit_grid(int64_t n, int64_t b, int64_t i_begin,
                                                       int64_t i_end, int64_t run = 1) {
  UnitGrid g;
  g.n = n;
  g.b = b;
  g.run = run;
  g.i_begin = i_begin;
  g.i_end = i_end;
  g.it0 = i_begin / b;
  g.it1 = i_end > i_begin ? (i_end + b - 1) / b : g.it0;
  g.nt = (n + b - 1) / b;
  return g;
}

// Number of tile pairs (it, kt), it0 <= it < it1, it <= kt < nt.
__host__ __device__ __forceinline__ int64_t grid_pairs(const UnitGrid& g) {
  int64_t p = 0;
  if (g.it1 > g.it0) {
    const int64_t rows = g.it1 - g.it0;  // sum of (nt - it) over the I tiles
    p = rows * g.nt - (g.it1 * (g.it1 - 1) / 2 - g.it0 * (g.it0 - 1) / 2);
  }
  return p;
}

// First pair index of I tile it.
__host__ __device__ __forceinline__ int64_t grid_row_start(const UnitGrid& g, int64_t it) {
  return (it - g.it0) * g.nt - (it * (it - 1) / 2 - g.it0 * (g.it0 - 1) / 2);
}

// Middle vectors [jlo, jhi) of tile pair (it, kt): j above the first row of
// tile it in the range, and below the last row of tile kt.
__host__ __device__ __forceinline__ void pair_j_range(const UnitGrid& g, int64_t it, int64_t kt,
                                                      int64_t& jlo, int64_t& jhi) {
  jlo = (it * g.b > g.i_begin ? it * g.b : g.i_begin) + 1;
  jhi = (kt + 1) * g.b - 1;
  if (jhi > g.n - 1) jhi = g.n - 1;
  if (jhi < jlo) jhi = jlo;
}

// Units of tile pair (it, kt): its j range in runs of g.run.
__host__ __device__ __forceinline__ int64_t pair_units(const UnitGrid& g, int64_t it,
                                                       int64_t kt) {
  int64_t jlo, jhi;
  pair_j_range(g, it, kt, jlo, jhi);
  return (jhi - jlo + g.run - 1) / g.run;
}

// Tile pair of pair index p.
__host__ __device__ __forceinline__ void pair_tiles(const UnitGrid& g, int64_t p, int64_t& it,
                                                    int64_t& kt) {
  int64_t lo = g.it0, hi = g.it1;  // row_start(lo) <= p < row_start(hi)
  while (hi - lo > 1) {
    const int64_t mid = (lo + hi) >> 1;
    if (grid_row_start(g, mid) <= p) lo = mid; else hi = mid;
  }
  it = lo;
  kt = it + (p - grid_row_start(g, it));
}

// Unit u -> (first middle vector j of its run, I tile, K tile), given
// offs[p] = units of all pairs before p (p = 0..pairs).
// The host tests hold unit_at to it.
__host__ __device__ __forceinline__ void unit_coords(int64_t u, const UnitGrid& g,
                                                     const int64_t* __restrict__ offs,
                                                     int64_t& j, int64_t& it, int64_t& kt) {
  int64_t lo = 0, hi = grid_pairs(g);  // offs[lo] <= u < offs[hi]
  while (hi - lo > 1) {
    const int64_t mid = (lo + hi) >> 1;
    if (offs[mid] <= u) lo = mid; else hi = mid;
  }
  pair_tiles(g, lo, it, kt);
  int64_t jlo, jhi;
  pair_j_range(g, it, kt, jlo, jhi);
  j = jlo + g.run * (u - offs[lo]);
}

// The same without the table of offsets.  With s = jlo(it) the first middle
// vector of I tile it (the same for all its K tiles) and every tile but the
// last whole, pair (it, it + d) has (d + 1) b/run - f units, f = floor((2 +
// delta) / run) and delta how far the range begins inside the tile (first I
// tile only), and the last K tile ceil((n - 1 - s) / run).  So the units
// before a pair are a quadratic in d, and those before an I tile a cubic,
// searched by halving: no dependent loads, no kernel that writes a table.
// (Only d = 0 can come out negative, -1 with run = 1; it is then 0.)
struct UnitRow {
  int64_t q, f, fix, last, tail;  // b / run, f, units added back at d = 0, last d, its units
};
__host__ __device__ __forceinline__ UnitRow unit_row(const UnitGrid& g, int64_t it) {
  const int64_t first = it * g.b, delta = g.i_begin > first ? g.i_begin - first : 0;
  UnitRow r;
  r.q = g.b / g.run;
  r.f = (2 + delta) / g.run;
  r.fix = r.q < r.f ? r.f - r.q : 0;
  r.last = g.nt - 1 - it;
  const int64_t js = g.n - 1 - (first + delta + 1);  // middle vectors of the last K tile
  r.tail = js > 0 ? (js + g.run - 1) / g.run : 0;
  return r;
}
// Units of the pairs (it, it) .. (it, it + d - 1), d <= last.
__host__ __device__ __forceinline__ int64_t row_units_before(const UnitRow& r, int64_t d) {
  return r.q * (d * (d + 1) / 2) - d * r.f + (d > 0 ? r.fix : 0);
}
// Units of I tiles it0 .. it - 1.
__host__ __device__ __forceinline__ int64_t tile_units_before(const UnitGrid& g, int64_t it) {
  if (it <= g.it0) return 0;
  const UnitRow r0 = unit_row(g, g.it0);
  const int64_t head = row_units_before(r0, r0.last) + r0.tail;
  // the whole tiles after the first: rows x = it0 + 1 .. it - 1 with D = nt -
  // 1 - x whole pairs and a tail of ceil((n - 2 - x b) / run)
  const int64_t lo = g.it0 + 1, cnt = it - lo, q = g.b / g.run, f = 2 / g.run;
  const int64_t D1 = g.nt - 1 - lo, D0 = D1 - cnt;  // D runs D1 .. D0 + 1
  const int64_t pairs = (D1 * (D1 + 1) - D0 * (D0 + 1)) / 2;                          // sum of D
  const int64_t tets = (D1 * (D1 + 1) * (D1 + 2) - D0 * (D0 + 1) * (D0 + 2)) / 6;     // D(D+1)/2
  const int64_t rows = (lo + it - 1) * cnt / 2;                                       // sum of x
  return head + q * tets - f * pairs + cnt * ((g.n - 2 + g.run - 1) / g.run) - q * rows;
}
__host__ __device__ __forceinline__ int64_t grid_unit_count(const UnitGrid& g) {
  return tile_units_before(g, g.it1);
}
__host__ __device__ __forceinline__ void unit_at(int64_t u, const UnitGrid& g, int64_t& j,
                                                 int64_t& it, int64_t& kt) {
  int64_t lo = g.it0, hi = g.it1;  // tile_units_before(lo) <= u < tile_units_before(hi)
  while (hi - lo > 1) {
    const int64_t mid = (lo + hi) >> 1;
    if (tile_units_before(g, mid) <= u) lo = mid; else hi = mid;
  }
  it = lo;
  u -= tile_units_before(g, it);
  const UnitRow r = unit_row(g, it);
  lo = 0, hi = r.last + 1;  // row_units_before(lo) <= u
  while (hi - lo > 1) {
    const int64_t mid = (lo + hi) >> 1;
    if (row_units_before(r, mid) <= u) lo = mid; else hi = mid;
  }
  kt = it + lo;
  int64_t jlo, jhi;
  pair_j_range(g, it, kt, jlo, jhi);
  j = jlo + g.run * (u - row_units_before(r, lo));
}

// Workgroup b of a grid of `count` -> unit index, so that the workgroups the
// dispatcher sends to one of the 8 XCDs (b mod 8) take one contiguous run of
// units, in order.
__host__ __device__ __forceinline__ int64_t xcd_unit(int64_t b, int64_t count) {
  const int64_t q = count >> 3, r = count & 7, x = b & 7;
  return x * q + (x < r ? x : r) + (b >> 3);
}

// Strip order of the squares of a 2-way triangle launch, so that the
// consecutive squares an XCD has in flight (xcd_unit hands each XCD a
// contiguous run) share both their row and their column blocks: strips of
// kStripRows square rows, walked column by column, rows ascending within a
// column.  (A rectangle keeps the row-major order, which measured faster.)
constexpr int64_t kStripRows = 8;

// Triangle: square t of the squares (I, J), s0 <= I < s1, I <= J < T, in
// strips of H square rows.  A strip of h rows r0 .. r1 - 1 holds
// h (h - 1) / 2 squares in its first h - 1 columns (column r0 + c has c + 1)
// and h in each of the T - r1 + 1 columns after them; the strips before the
// last are full, so the squares before strip k number
// k A - H^2 k (k + 1) / 2 with A = H (H - 1) / 2 + H (T - s0 + 1).
__host__ __device__ inline void strip_square(int64_t t, int64_t T, int64_t s0, int64_t s1,
                                             int64_t& I, int64_t& J,
                                             int64_t H = kStripRows) {
  const int64_t nstrips = (s1 - s0 + H - 1) / H;
  const int64_t A = H * (H - 1) / 2 + H * (T - s0 + 1);
  auto before = [&](int64_t k) { return k * A - H * H * k * (k + 1) / 2; };
  const double bq = (double)A - 0.5 * (double)(H * H);
  const double disc = bq * bq - 2.0 * (double)(H * H) * (double)t;
  int64_t k = (int64_t)((bq - sqrt(disc > 0.0 ? disc : 0.0)) / (double)(H * H));
  if (k < 0) k = 0;
  if (k > nstrips - 1) k = nstrips - 1;
  while (k > 0 && before(k) > t) --k;
  while (k + 1 < nstrips && before(k + 1) <= t) ++k;
  const int64_t r0 = s0 + k * H, r1 = r0 + H < s1 ? r0 + H : s1, h = r1 - r0;
  const int64_t u = t - before(k), diag = h * (h - 1) / 2;
  if (u < diag) {  // column r0 + c holds rows r0 .. r0 + c
    int64_t c = (int64_t)((sqrt(8.0 * (double)u + 1.0) - 1.0) * 0.5);
    while (c > 0 && c * (c + 1) / 2 > u) --c;
    while ((c + 1) * (c + 2) / 2 <= u) ++c;
    J = r0 + c;
    I = r0 + (u - c * (c + 1) / 2);
  } else {
    J = r1 - 1 + (u - diag) / h;
    I = r0 + (u - diag) % h;
  }
}

// Arguments of one 3-way tally launch over all triples i < j < k.
struct Triple3Args {
  const uint8_t* v;
  int64_t ld, n, n_f;
  int f4;         // MFMA operands: fp4 (1, needs n_f <= kF4MaxFields) or int8 (0)
  int32_t* tables;
  double* ccc;
  const int32_t* counts;
  double gamma;
  // triples whose first index lies in [i_begin, i_end); triple t goes to entry t - t_base
  int64_t i_begin, i_end;
  int64_t t_base;
  Select sel;
  // Dense rho(1) Gram matrix of rows [g0, g0 + ng) (workspace), filled by the
  // MFMA launcher; null turns the complete-data path off.
  int32_t* gram;
  int64_t g0, ng;
  // Complete-data flag (fp4 MFMA with a Gram matrix only; null: every unit
  // votes for itself): holds `id` when some row of [g0, n) misses an entry.
  unsigned long long* flag;
  unsigned long long id;
};

enum Path { kPathPopcount = 1, kPathMfma = 2 };

// Kernel-shape table (tune.hip): kinds of launch, and the variant the table
// picks for a problem of n_v vectors over n_f fields (0 .. n_variants - 1).
enum TuneKind { kTuneManyMfma = 0, kTuneManyPopcount = 1, kTuneOneShot = 2 };
struct TuneChoice {
  int variant;    // tile variant, in [0, n_variants)
  int wg_per_cu;  // persistent workgroups per compute unit; 0: the launcher's default
};
// The one-shot variant that the environment forces (0 .. n_variants - 1), or -1.
int tune_forced_oneshot(int n_variants);
// Workgroups per field-split tile that the environment forces (1 .. 64), or -1.
int tune_forced_split();
// Shape of a 2-way call on operands by its 32 x 32 tiles and fields: 0 = 64 x
// 128 staged tiles, 1 = field-split 32 x 32 tiles, 2 = 64 x 64 staged tiles, 3 =
// packed rows (mfma2.hip).  dense_ccc: a dense triangle with CCC rows; mixed: a selection or
// an accumulating call.
int operand_variant(int64_t tiles, int64_t n_f, bool dense_ccc, bool mixed);
TuneChoice tune_pick(int kind, int64_t n_v, int64_t n_f, int n_variants);

// Optional event timing around the main kernel of a launcher (no-ops unless
// enabled through ccc_timing_enable).
void timing_begin(const char* name, hipStream_t stream);
void timing_end(hipStream_t stream);
// A host-side duration under `name` (recorded only while timing is enabled).
void timing_host(const char* name, double ms);

hipError_t launch_count1(const uint8_t* v, int64_t ld, int64_t n, int64_t n_f, int32_t* counts,
                         int accumulate, hipStream_t stream);
// count1 that also zeroes a selection counter (a kernel store, graph safe) and
// sets *flag = id when some row from flag_from on misses an entry
hipError_t launch_count1_zero(const uint8_t* v, int64_t ld, int64_t n, int64_t n_f,
                              int32_t* counts, int accumulate, unsigned long long* zero,
                              hipStream_t stream, unsigned long long* flag = nullptr,
                              unsigned long long id = 0, int64_t flag_from = 0);
hipError_t launch_operands(OperandJob job, hipStream_t stream);
// First 16-row block that the tiles of a triangle's rows from i_begin on read:
// no tile is larger than 256 rows.
inline int64_t operand_first(int64_t i_begin) { return i_begin / 256 * 16; }
// Whether a 2-way call has a use for operands (an accumulating one whose tiles
// would all read the packed rows has not).
bool operands_serve(const Pair2Args& a);
// Most operands that the library holds on a device (api.hip).
int64_t operand_limit();
// Room for a batch's operands beside the workspaces', and the account of those
// that the batches hold (api.hip).
bool batch_operands_fit(int dev, size_t bytes);
void hold_batch_operands(int dev, int64_t bytes);
// Shares of the fields for the pass over one set: few blocks of long rows are
// bound by the memory path of the few CUs that hold them (24 blocks x 977
// super-steps: 39 us in one share), but the counts' second launch costs 5 us.
inline int operand_shares(int64_t n, int64_t n_f) {
  const int64_t blocks = operand_blocks(n), steps = operand_steps(n_f);
  if (blocks <= 0 || blocks > 128 || steps < 256) return 1;
  const int64_t a = 512 / blocks, b = steps / 32, s = a < b ? a : b;
  return (int)(s < 16 ? s : 16);
}
inline size_t operand_part_bytes(int64_t n, int64_t n_f) {
  const int s = operand_shares(n, n_f);
  return s > 1 ? ((size_t)s * n * sizeof(int2) + 255) / 256 * 256 : 0;
}
// Bytes of partial sums that launch_mfma2 wants for a call (0: it will not
// split the fields).
size_t mfma2_part_bytes(const Pair2Args& a);
hipError_t launch_pop2(const Pair2Args& a, hipStream_t stream);
hipError_t launch_mfma2(const Pair2Args& a, hipStream_t stream);
hipError_t launch_mfma3(const Triple3Args& a, hipStream_t stream);
hipError_t launch_pop3(const Triple3Args& a, hipStream_t stream);
// Multi-allelic 2-way (one byte per field, s = 2..4 states): counts are
// [n][8] = (n(0), n(1), n(2), n(3), m, 0, 0, 0); tables / ccc [pairs][s*s].
hipError_t launch_multi_count(const uint8_t* v, int64_t ld, int64_t n, int64_t n_f, int s,
                              int32_t* counts, hipStream_t stream);
hipError_t launch_multi2(const uint8_t* v, int64_t ld, int64_t n, int64_t n_f, int s,
                         int32_t* tables, double* ccc, const int32_t* counts, double gamma,
                         int f4, const void* z, hipStream_t stream);
// The count pass that also writes the rows as fp4 operands (multi2.hip) to z,
// multi_operand_bytes of them; launch_multi2 reads them when z is given.
size_t multi_operand_bytes(int64_t n, int64_t n_f, int s);
hipError_t launch_multi_operands(const uint8_t* v, int64_t ld, int64_t n, int64_t n_f, int s,
                                 int32_t* counts, void* z, hipStream_t stream);

}  // namespace ccc
