// tile2o.h -- 2-way tally tiles on fp4 operands that the pre-pass has laid out
// (operands.h): device bodies of the one-shot kernels (mfma2.hip) and the
// batched ones (many.hip).
//
// A tile needs the four sums of the planes W = rho(1) + 3 [missing], the
// 2-bit code of the layout as it lies, and M = [missing]:
//   WW = sum W_i W_j, WM = sum W_i M_j, MW = sum M_i W_j, MM = sum M_i M_j,
// each 4x its fp32 accumulator (operands are halves; multiples of 1/4, and
// exact while 9 n_f <= 2^24, kStagedMaxFields).  With the call's own 1-way
// counts, rho(1) = W - 3M, P = 1 - M and rho(0) = 2P - rho(1) they give the
// table.  M is nearly all zeros in real data, and rows that miss nothing
// need WW alone.
#pragma once

#include "tile2.h"

namespace ccc {
namespace tile2 {

// Largest n_f whose sums an fp32 accumulator holds exactly.
constexpr int64_t kStagedMaxFields = (int64_t(1) << 24) / 9;

// The MFMA operands W and (GENERAL) M of 32 fields per lane, words w0 and w1:
// even fields in registers 0 and 2, odd ones in 1 and 3, e2m1 value = plane
// / 2.  Eleven operations, or five for W alone.  Truth table 0x80 = a & b & c.
// The paired shifts carry w1's bits 0, 0-1, 0-2 into bits 31, 30-31, 29-31 of
// the w0 results, which no mask keeps.
template <bool GENERAL>
__device__ __forceinline__ void operands32(unsigned w0, unsigned w1, v8i& w, v8i& m) {
  unsigned c0, c1;
  shr_pair<2>(w0, w1, c0, c1);
  w = v8i{(int)(w0 & kNib2), (int)(c0 & kNib2), (int)(w1 & kNib2), (int)(c1 & kNib2), 0, 0, 0, 0};
  if constexpr (GENERAL) {
    constexpr unsigned k = 0x11111111u;
    unsigned b0, b1, d0, d1;
    shr_pair<1>(w0, w1, b0, b1);
    shr_pair<3>(w0, w1, d0, d1);
    m = v8i{(int)__builtin_amdgcn_bitop3_b32(w0, b0, k, 0x80),
            (int)__builtin_amdgcn_bitop3_b32(c0, d0, k, 0x80),
            (int)__builtin_amdgcn_bitop3_b32(w1, b1, k, 0x80),
            (int)__builtin_amdgcn_bitop3_b32(c1, d1, k, 0x80), 0, 0, 0, 0};
  }
}

// acc[n][..] += the products of row operands (aw, am) with the WN column
// operands: the four sums, or WW alone.
template <bool GENERAL, int WN, int NP>
__device__ __forceinline__ void multiply_row(const v8i& aw, const v8i& am, const v8i (&bw)[WN],
                                             const v8i (&bm)[WN], v4f (&acc)[WN][NP]) {
#pragma unroll
  for (int n = 0; n < WN; ++n) {
    acc[n][0] = mfma_f4(aw, bw[n], acc[n][0]);
    if constexpr (GENERAL) {
      acc[n][1] = mfma_f4(aw, bm[n], acc[n][1]);
      acc[n][2] = mfma_f4(am, bw[n], acc[n][2]);
      acc[n][3] = mfma_f4(am, bm[n], acc[n][3]);
    }
  }
}

// Table (entry 2a+b) from the four sums over n_f fields: with
//   S = sum rho_i rho_j = WW - 3 WM - 3 MW + 9 MM,
//   T = sum rho_i P_j = n_i(1) - (WM - 3 MM), U = sum P_i rho_j likewise,
//   V = sum P_i P_j = m_i + m_j - n_f + MM.
__device__ __forceinline__ v4i table_wm(int ww, int wm, int mw, int mm, int n1i, int mi, int n1j,
                                        int mj, int n_f) {
  const int S = ww - 3 * (wm + mw) + 9 * mm;
  const int T = n1i - wm + 3 * mm, U = n1j - mw + 3 * mm, V = mi + mj - n_f + mm;
  return v4i{4 * V - 2 * T - 2 * U + S, 2 * U - S, 2 * T - S, S};
}

// How a kernel puts its pairs out, fixed at compile time: the epilogue is
// unrolled over a tile's blocks, and with its forms behind run-time
// branches each copy is four times the code.
enum Out {
  kDense,
  kAccumulate,
  kSelect,
  kStream  // dense, the tables by streaming stores (complete-data tiles, see mfma2.hip)
};

// What the epilogue needs of one row or column: its factors, this call's own
// counts n(1) and m, and for a row the first column of its run (columns from
// jmin on are pairs to put out; none: past every column) and the entry of
// column 0 of its run in the output.
struct SideIn {
  double w[2];
  int jmin, n1, m, pad;
};
static_assert(sizeof(SideIn) == 32, "two 16-byte halves");
template <int NR, int NC>
struct Sides {
  SideIn s[NR + NC];
  int64_t entry[NR];
};

// Sides of rows row0 .. row0 + NR - 1 and columns col0 .. col0 + NC - 1, by
// `threads` threads from thread t on.
template <Out OUT, int NR, int NC>
__device__ __forceinline__ void load_sides(const Pair2Args& a, int64_t row0, int64_t col0,
                                           Sides<NR, NC>& out, int t, int threads) {
  for (; t < NR + NC; t += threads) {
    const bool is_row = t < NR;
    const int64_t x = is_row ? row0 + t : col0 + (t - NR), nx = is_row ? a.n_a : a.n_b;
    SideIn si;
    side_factors(a, is_row ? 0 : 1, x, si.w);
    const v4i c = reinterpret_cast<const v4i*>(is_row ? a.chunk_a : a.chunk_b)[x < nx ? x : nx - 1];
    si.n1 = c.y;
    si.m = c.z;
    si.pad = 0;
    si.jmin = 0;
    if (is_row) {
      const bool in = x < a.n_a && x >= a.row_begin && x < a.row_end;
      si.jmin = in ? (a.tri ? (int)x + 1 : 0) : 0x7FFFFFFF;
      // p(i, j) is affine in j
      out.entry[t] = (a.tri ? pair_index(a.n_a, x, 0) : x * a.n_b) - (OUT == kSelect ? 0 : a.p_base);
    }
    out.s[t] = si;
  }
}

// Every row of the (NR rows) x (NC columns) tile has all n_f fields present;
// uniform over the wave.  Never in an accumulating call, whose counts are
// running totals.
template <int NR, int NC>
__device__ __forceinline__ bool wave_complete(const Pair2Args& a, int64_t row0, int64_t col0) {
  if (a.accumulate || a.n_f <= 0) return false;
  const int lane = threadIdx.x & 63;
  bool ok = true;
  for (int t = lane; t < NR + NC; t += 64) {
    const bool is_row = t < NR;
    const int64_t x = is_row ? row0 + t : col0 + (t - NR), nx = is_row ? a.n_a : a.n_b;
    ok = ok && reinterpret_cast<const v4i*>(is_row ? a.counts_a : a.counts_b)[x < nx ? x : nx - 1]
                       .z == a.n_f;
  }
  return __all(ok ? 1 : 0) != 0;
}

// Base address of super-step 0 of row block b (clamped) of a side.
__device__ __forceinline__ gbytes block_base(const void* z, int64_t b, int64_t n, int64_t steps) {
  const int64_t last = (n + 15) / 16 - 1;
  return (gbytes)z + (b < last ? b : last) * steps * 1024;
}

// Byte offset of an LDS address.
__device__ __forceinline__ uint32_t lds_offset(const void* p) {
  return (uint32_t)(uintptr_t)(__attribute__((address_space(3))) const void*)p;
}

// Asynchronous copy of 1 KB into LDS: lane l's 16 bytes at base + off go to
// dst + 16 l (base and dst uniform; the wave's vector-memory counter covers
// it).  In asm, so that the compiler does not put a wait for every copy in
// flight before the next LDS read, as it does with the builtin whatever the
// addresses; callers wait themselves (ring_loop).  It has no output register,
// and its inputs are read as it issues.
__device__ __forceinline__ void copy_async(gbytes base, uint32_t off, uint32_t dst) {
  asm volatile("s_nop 0\n\tglobal_load_lds_dwordx4 %0, %1"
               :
               : "v"(off), "s"(base), "{m0}"(dst)
               : "memory");
}

// Steps 0 .. n - 1 of a workgroup of four waves whose ND pieces of 1 KB per
// step travel into a ring of three LDS buffers, two steps ahead, split over
// the waves: wave w copies pieces DPW w + t from base[t] + s * stride.  One
// barrier per step says that every piece of the step has landed and that the
// buffer read one step earlier is free.  Every wave must call it; body(buf)
// multiplies a step.  Two steps ahead, not one: a step is some 1100 to 2200
// cycles of a SIMD, and a copy takes about that long to arrive when a CU's
// two workgroups have theirs in flight.
template <int ND, typename Body>
__device__ __forceinline__ void ring_loop(const gbytes (&base)[ND / 4], int64_t n,
                                          u4 (*stage)[ND][64], Body body,
                                          uint32_t stride = 1024) {
  constexpr int DPW = ND / 4;
  const int lane = threadIdx.x & 63;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);  // uniform
  constexpr uint32_t kBuf = ND * 1024;
  const uint32_t dst0 = __builtin_amdgcn_readfirstlane(lds_offset(&stage[0][DPW * wave][0]));
  gbytes cur[DPW];
#pragma unroll
  for (int t = 0; t < DPW; ++t) {
    // uniform already; read from lane 0 so that the compiler knows it
    const uint64_t b = (uint64_t)base[t];
    cur[t] = (gbytes)(((uint64_t)(uint32_t)__builtin_amdgcn_readfirstlane((int)(b >> 32)) << 32) |
                      (uint32_t)__builtin_amdgcn_readfirstlane((int)b));
  }
  auto issue = [&](uint32_t buf) {
#pragma unroll
    for (int t = 0; t < DPW; ++t) {
      copy_async(cur[t], 16 * lane,
                 __builtin_amdgcn_readfirstlane(dst0 + buf * kBuf + 1024 * t));
      cur[t] += stride;
    }
  };
  if (n > 0) issue(0);
  if (n > 1) issue(1);
  uint32_t buf = 0;
  for (int64_t s = 0; s < n; ++s) {
    // this wave's pieces of step s have landed (those of s + 1 may fly on)
    // and its reads of the last buffer are done; then every wave's
    if (s + 1 < n)
      asm volatile("s_waitcnt vmcnt(%0) lgkmcnt(0)\n\ts_barrier" : : "n"(DPW) : "memory");
    else
      asm volatile("s_waitcnt vmcnt(0) lgkmcnt(0)\n\ts_barrier" : : : "memory");
    if (s + 2 < n) issue(buf == 0 ? 2 : buf - 1);
    body(stage[buf]);
    buf = buf == 2 ? 0 : buf + 1;
  }
}

// Super-step loop of a workgroup of 2 x 2 waves of (16 WM) x (16 WN) pairs
// over its 2 WM + 2 WN row blocks.  GENERAL: the four sums, else WW alone.
// Every wave must call it; inactive ones only copy and meet the barriers.
template <int WM, int WN, bool GENERAL, int NP>
__device__ __forceinline__ void staged_loop(const Pair2Args& a, int64_t I0, int64_t J0,
                                            bool active, u4 (*stage)[2 * WM + 2 * WN][64],
                                            v4f (&acc)[WM][WN][NP]) {
  constexpr int ND = 2 * WM + 2 * WN, DPW = ND / 4;  // 1 KB pieces per step, per wave
  static_assert(ND % 4 == 0, "pieces split evenly over the waves");
  static_assert(NP == (GENERAL ? 4 : 1), "sums");
  const int lane = threadIdx.x & 63;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);  // uniform
  gbytes base[DPW];
#pragma unroll
  for (int t = 0; t < DPW; ++t) {
    const int blk = DPW * wave + t;
    base[t] = blk < 2 * WM ? block_base(a.za, I0 / 16 + blk, a.n_a, a.steps)
                           : block_base(a.zb, J0 / 16 + blk - 2 * WM, a.n_b, a.steps);
  }
  const int ma = (wave & 1) * WM, nb = 2 * WM + (wave >> 1) * WN;  // first pieces
  if (!active) {
    ring_loop<ND>(base, a.steps, stage, [](const u4 (&)[ND][64]) {});
    return;
  }
#pragma unroll
  for (int m = 0; m < WM; ++m)
#pragma unroll
    for (int n = 0; n < WN; ++n)
#pragma unroll
      for (int p = 0; p < NP; ++p) acc[m][n][p] = v4f{0, 0, 0, 0};
  ring_loop<ND>(base, a.steps, stage, [&](const u4 (&buf)[ND][64]) {
    u4 xa[WM], xb[WN];
#pragma unroll
    for (int n = 0; n < WN; ++n) xb[n] = buf[nb + n][lane];
#pragma unroll
    for (int m = 0; m < WM; ++m) xa[m] = buf[ma + m][lane];
#pragma unroll
    for (int h = 0; h < 2; ++h) {
      v8i bw[WN], bm[WN];
#pragma unroll
      for (int n = 0; n < WN; ++n)
        operands32<GENERAL>(word_of(xb[n], 2 * h), word_of(xb[n], 2 * h + 1), bw[n], bm[n]);
#pragma unroll
      for (int m = 0; m < WM; ++m) {
        v8i aw, am;
        operands32<GENERAL>(word_of(xa[m], 2 * h), word_of(xa[m], 2 * h + 1), aw, am);
        multiply_row<GENERAL>(aw, am, bw, bm, acc[m]);
      }
    }
  });
}

// Put out the 16 x (16 WN) pairs of rows r0 .. and columns c0 .. of the sides
// (first column j0): lane holds rows 4g + e of column rl of each block.
// GENERAL: the four sums; else WW alone (every row complete).  Plain stores,
// and a row's blocks one after the other: the 256- and 512-byte stretches of
// a row start anywhere in a line, and L2 joins their ends if they come close
// together.  (Stores alone, 64 x 64 tiles: tables 4.8 TB/s plain and 2.8
// streaming, CCC rows 4.8 and 1.6; both together 4.3 TB/s in this order and
// 3.4 block by block.)
__device__ __forceinline__ int count_of(const v4f& x, int e) { return f4_count(x[e]); }
__device__ __forceinline__ int count_of(const v4i& x, int e) { return x[e]; }
template <Out OUT, bool GENERAL, typename V, int NP, int WN, int NR, int NC>
__device__ __forceinline__ void emit_blocks(const Pair2Args& a, const Sides<NR, NC>& sides, int r0,
                                            int c0, int64_t j0, const V (&s)[WN][NP]) {
  const int lane = threadIdx.x & 63, g = lane >> 4, rl = lane & 15;
  const int n_f = (int)a.n_f;
  static_for<4>([&](auto ec) {
    constexpr int e = decltype(ec)::value;
    const SideIn si = sides.s[r0 + 4 * g + e];
    const int64_t entry = sides.entry[r0 + 4 * g + e];
    static_for<WN>([&](auto nc) {
      constexpr int n = decltype(nc)::value;
      const int64_t j = j0 + 16 * n + rl, p = entry + j;
      const SideIn sj = sides.s[NR + c0 + 16 * n + rl];
      const bool valid = j >= si.jmin && j < a.n_b;
      v4i t;
      if constexpr (GENERAL)
        t = table_wm(count_of(s[n][0], e), count_of(s[n][1], e), count_of(s[n][2], e),
                     count_of(s[n][3], e), si.n1, si.m, sj.n1, sj.m, n_f);
      else
        t = table_wm(count_of(s[n][0], e), 0, 0, 0, si.n1, si.m, sj.n1, sj.m, n_f);
      if constexpr (OUT == kSelect) {
        double r[4] = {0.0, 0.0, 0.0, 0.0};
        bool keep = false;
        if (valid) {
          pair_ccc(t, si.w, sj.w, r);
          keep = r[0] >= a.sel.threshold || r[1] >= a.sel.threshold ||
                 r[2] >= a.sel.threshold || r[3] >= a.sel.threshold;
        }
        select_pair(a.sel, keep, p, t, r);
      } else if (valid) {
        if (a.tables) {
          v4i* out = reinterpret_cast<v4i*>(a.tables) + p;
          if constexpr (OUT == kAccumulate) t = t + *out;
          if constexpr (OUT == kStream)
            __builtin_nontemporal_store(t, out);
          else
            *out = t;
        }
        if (a.ccc) {
          double r[4];
          pair_ccc(t, si.w, sj.w, r);
          double2* out = reinterpret_cast<double2*>(a.ccc) + 2 * p;
          out[0] = double2{r[0], r[1]};
          out[1] = double2{r[2], r[3]};
        }
      }
    });
  });
}

// One workgroup's tile of (32 WM) x (32 WN) pairs at (I0, J0), 2 x 2 waves;
// `stage` is its LDS (three buffers), reused for the epilogue's inputs.  Bound
// by MFMA issue (matrix cores 69% busy at 16384 x 32768, where power holds the
// clock at 2.03 GHz, 73% and 2.13 at 32768 x 65536), then by the output.
// 16384 x 32768: 6.50 ms from
// packed rows, 5.69 here; 32768 x 65536: 45.2-48.1 and 41.2.
template <Out OUT, int WM, int WN>
__device__ __forceinline__ void staged_tile(const Pair2Args& a, int64_t I0, int64_t J0,
                                            u4 (*stage)[2 * WM + 2 * WN][64]) {
  const int lane = threadIdx.x & 63;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);  // uniform
  const int64_t row0 = I0 + (wave & 1) * 16 * WM, col0 = J0 + (wave >> 1) * 16 * WN;
  const bool active = row0 < a.n_a && col0 < a.n_b && !(a.tri && row0 >= col0 + 16 * WN - 1);
  using S = Sides<16 * WM, 16 * WN>;
  static_assert(4 * sizeof(S) <= sizeof(u4) * 3 * (2 * WM + 2 * WN) * 64,
                "the epilogue's inputs fit in the stage");
  S& sides = reinterpret_cast<S*>(&stage[0][0][0])[wave];
  auto finish = [&](auto general, auto& acc) {
    // the epilogue's inputs are read before its first store (a wait for a
    // load also waits for every store issued before it)
    __syncthreads();  // every wave is done with the stage
    if (!active) return;
    load_sides<OUT>(a, row0, col0, sides, lane, 64);
    static_for<WM>([&](auto m) {
      emit_blocks<OUT, general.value>(a, sides, 16 * m.value, 0, col0, acc[m.value]);
    });
  };
  // uniform over the workgroup: every wave takes the same loop
  bool whole = wave_complete<16 * WM, 16 * WN>(a, row0, col0);
  whole = __syncthreads_and(whole || !active ? 1 : 0) != 0;
  if (whole && !a.accumulate && a.n_f > 0) {
    v4f acc[WM][WN][1];
    staged_loop<WM, WN, false>(a, I0, J0, active, stage, acc);
    finish(std::false_type{}, acc);
  } else {
    v4f acc[WM][WN][4];
    staged_loop<WM, WN, true>(a, I0, J0, active, stage, acc);
    finish(std::true_type{}, acc);
  }
}

// Tile of a call whose every row is complete: WW alone, so the accumulators
// of a (16 WM) x (16 WN) wave tile are a quarter of the general form's and
// the tile four times the size.  Bound by its operands' reads past L2 beside
// the output stream.  16000 x 40000: 3.55 ms from packed rows, 2.83 here;
// 32768 x 65536: 19.4-20.5 and 15.7.
template <Out OUT, int WM, int WN>
__device__ __forceinline__ void complete_tile(const Pair2Args& a, int64_t I0, int64_t J0,
                                              u4 (*stage)[2 * WM + 2 * WN][64]) {
  const int lane = threadIdx.x & 63;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);  // uniform
  const int64_t row0 = I0 + (wave & 1) * 16 * WM, col0 = J0 + (wave >> 1) * 16 * WN;
  const bool active = row0 < a.n_a && col0 < a.n_b && !(a.tri && row0 >= col0 + 16 * WN - 1);
  using S = Sides<16 * WM, 16 * WN>;
  static_assert(4 * sizeof(S) <= sizeof(u4) * 3 * (2 * WM + 2 * WN) * 64,
                "the epilogue's inputs fit in the stage");
  S& sides = reinterpret_cast<S*>(&stage[0][0][0])[wave];
  v4f acc[WM][WN][1];
  staged_loop<WM, WN, false>(a, I0, J0, active, stage, acc);
  __syncthreads();  // every wave is done with the stage
  if (!active) return;
  load_sides<OUT>(a, row0, col0, sides, lane, 64);
  static_for<WM>([&](auto m) {
    emit_blocks<OUT, false>(a, sides, 16 * m.value, 0, col0, acc[m.value]);
  });
}

constexpr int kSplitTile = 32;
using SplitSides = Sides<kSplitTile, kSplitTile>;

// Field-split tile: 32 x 32 pairs at (I0, J0) whose super-steps [s0, s1) are
// shared out over the workgroup's four waves, each multiplying the whole tile
// over its quarter from registers (1 KB contiguous loads, no barrier), so
// that a call with few tiles still fills the chip and a short chain of steps
// ends early.  The four partial sums, whole numbers, meet in LDS (`red`,
// 16 KB), after which wave w holds block (w & 1, w >> 1) of the tile, given to
// done(general, sums).  A wave's own sum stays exact up to 4 kStagedMaxFields
// fields.  These tiles are short (a few dozen steps at most), so what a wave
// waits for at the start goes out together: the counts of the vote `whole()`
// (every row of the tile complete) and the first two steps' loads.  Bound by
// the latency of that chain, and of the launches before it: 384 x 250007 481
// us from packed rows and 61.5 here, 200 x 1337 24 and 14.
template <typename Vote, typename Done>
__device__ __forceinline__ void split_tile(const Pair2Args& a, int64_t I0, int64_t J0, int64_t s0,
                                           int64_t s1, v4i (*red)[4][64], Vote whole, Done done) {
  const int lane = threadIdx.x & 63;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);  // uniform
  gbytes base[4];
#pragma unroll
  for (int t = 0; t < 4; ++t)
    base[t] = t < 2 ? block_base(a.za, I0 / 16 + t, a.n_a, a.steps)
                    : block_base(a.zb, J0 / 16 + t - 2, a.n_b, a.steps);
  typedef const __attribute__((address_space(1))) u4* gu4;
  auto load = [&](int64_t s, u4 (&x)[4]) {
#pragma unroll
    for (int t = 0; t < 4; ++t) x[t] = *(gu4)(base[t] + s * 1024 + 16 * lane);
  };
  const int64_t len = s1 - s0, b = s0 + len * wave / 4, e = s0 + len * (wave + 1) / 4;
  u4 x[4], y[4];
  if (b < e) load(b, x);
  auto sums = [&](auto general) {
    constexpr bool GENERAL = decltype(general)::value;
    constexpr int NP = GENERAL ? 4 : 1;
    v4f acc[2][2][NP];
#pragma unroll
    for (int m = 0; m < 2; ++m)
#pragma unroll
      for (int n = 0; n < 2; ++n)
#pragma unroll
        for (int p = 0; p < NP; ++p) acc[m][n][p] = v4f{0, 0, 0, 0};
    auto multiply = [&](const u4 (&x)[4]) {
#pragma unroll
      for (int h = 0; h < 2; ++h) {
        v8i bw[2], bm[2];
#pragma unroll
        for (int n = 0; n < 2; ++n)
          operands32<GENERAL>(word_of(x[2 + n], 2 * h), word_of(x[2 + n], 2 * h + 1), bw[n],
                              bm[n]);
#pragma unroll
        for (int m = 0; m < 2; ++m) {
          v8i aw, am;
          operands32<GENERAL>(word_of(x[m], 2 * h), word_of(x[m], 2 * h + 1), aw, am);
          multiply_row<GENERAL>(aw, am, bw, bm, acc[m]);
        }
      }
    };
    int64_t s = b;
    for (; s + 1 < e; s += 2) {
      load(s + 1, y);
      multiply(x);
      if (s + 2 < e) load(s + 2, x);
      multiply(y);
    }
    if (s < e) multiply(x);
    // block k = 2n + m of plane p from every wave, added by wave k
    v4i out[1][NP];
#pragma unroll
    for (int p = 0; p < NP; ++p) {
#pragma unroll
      for (int k = 0; k < 4; ++k) {
        const v4f f = acc[k & 1][k >> 1][p];
        red[wave][k][lane] = v4i{f4_count(f[0]), f4_count(f[1]), f4_count(f[2]), f4_count(f[3])};
      }
      __syncthreads();
      out[0][p] = red[0][wave][lane] + red[1][wave][lane] + red[2][wave][lane] + red[3][wave][lane];
      __syncthreads();
    }
    done(general, out);
  };
  if (whole())
    sums(std::false_type{});
  else
    sums(std::true_type{});
}

// This wave's block of the tile: its sums `s` to the output.  The workgroup
// has filled `sides` before its last barrier.
template <Out OUT, bool GENERAL, int NP>
__device__ __forceinline__ void split_emit(const Pair2Args& a, int64_t I0, int64_t J0,
                                           const v4i (&s)[1][NP], const SplitSides& sides) {
  const int wave = threadIdx.x >> 6, m = wave & 1, n = wave >> 1;
  const int64_t i0 = I0 + 16 * m, j0 = J0 + 16 * n;
  if (i0 >= a.n_a || j0 >= a.n_b || (a.tri && i0 >= j0 + 15)) return;  // no pair
  emit_blocks<OUT, GENERAL>(a, sides, 16 * m, 16 * n, j0, s);
}

}  // namespace tile2
}  // namespace ccc
