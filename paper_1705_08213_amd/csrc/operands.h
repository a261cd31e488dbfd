// operands.h -- the pre-pass of the fp4 MFMA kernels (device code; kernels in
// operands.hip and many.hip): one read of the packed rows gives the 1-way
// counts and the rows as matrix-core operands.
//
// Layout: rows in blocks of 16, fields in super-steps of 256; super-step s of
// block b is the 1 KB at z + (b * steps + s) * 1024.  Lane (g, rl) = 16 g + rl
// of an MFMA wave has the 16 bytes at 16 * lane there, 64 fields of row
// 16 b + rl: two bits each, 0, 1, 2 = rho(1) and 3 = missing.  A lane's words
// 0-1 are its part of one 16x16x128 operand, words 2-3 of the next.  Fields
// past n_f and rows past n are 0.
//
// Why: every tile of the tally reads its row blocks again.  From packed rows
// such a block is 16 pieces of 64 bytes, one per row, and a 1 KB copy of them
// into LDS or registers holds a CU's memory path for 65 cycles; a contiguous
// 1 KB takes 16.7 (both measured, source in L2).  Nibbles, which need fewer
// operations to become operands (6 instead of 11 per 32 fields), are twice
// the bytes, and the complete-data kernel is bound by those.
#pragma once

#include <type_traits>

#include "common.h"
#include "kernels.h"

namespace ccc {
namespace {

// 1-way counts of one row to where they go: n(1) = a, m missing fields.
__device__ __forceinline__ void put_counts(const OperandJob& job, const OperandSet& s, int64_t r,
                                           int a, int m) {
  const int present = (int)job.n_f - m;
  const v4i c = v4i{2 * present - a, a, present, 0};
  if (s.chunk) reinterpret_cast<v4i*>(s.chunk)[r] = c;
  if (s.counts) {
    v4i* out = reinterpret_cast<v4i*>(s.counts) + r;
    v4i t = c;
    if (job.accumulate) {
      const v4i old = *out;
      t = v4i{old.x + c.x, old.y + c.y, old.z + c.z, 0};
    }
    *out = t;
  }
  if (m > 0 && job.flag) *job.flag = job.id;  // some row is not complete
}

// Share `share` of block b of 16 rows of set s, by the whole workgroup (up to
// 16 waves, which take the share's super-steps in turn).  LAY: not of a block
// before s.first, which is only counted.
template <bool LAY>
__device__ __forceinline__ void operand_block(const OperandJob& job, const OperandSet& s,
                                              int64_t b, int share, int (*part)[16][2]) {
  const int lane = threadIdx.x & 63, g = lane >> 4, rl = lane & 15;
  const int wave = threadIdx.x >> 6, waves = blockDim.x >> 6;
  const int64_t n_f = job.n_f, row = 16 * b + rl;
  const int64_t begin = job.steps * share / job.shares;
  const int64_t end = job.steps * (share + 1) / job.shares;
  const bool have = row < s.n;
  const uint8_t* p = s.v + (have ? row : s.n - 1) * s.ld + 16 * g;
  u4* z = reinterpret_cast<u4*>(s.z) + (b - s.first) * job.steps * 64 + lane;
  int n1 = 0, miss = 0;
  auto put = [&](int64_t st, const u4& x) {
    u4 o;
#pragma unroll
    for (int q = 0; q < 4; ++q) {
      const unsigned hi = (x[q] >> 1) & kEven, c = x[q] ^ hi;  // 00, 01, 11, 10 -> 0, 1, 2, 3
      const unsigned ms = c & hi, two = hi & ~c;
      n1 += __popc(c & kEven & ~hi) + 2 * __popc(two);
      miss += __popc(ms);
      o[q] = c;
    }
    if constexpr (LAY) z[st * 64] = o;
  };
  const u4 none = u4{0u, 0u, 0u, 0u};
  const int64_t whole = n_f / 256, nfull = end < whole ? end : whole;
  int64_t st = begin + wave;
  // many loads in flight: with few row blocks the pass is bound by their
  // latency
  auto batch = [&](auto count) {
    constexpr int N = decltype(count)::value;
    for (; st + (N - 1) * waves < nfull; st += N * waves) {
      u4 x[N];
#pragma unroll
      for (int t = 0; t < N; ++t)
        x[t] = have ? *reinterpret_cast<const u4*>(p + (st + t * waves) * 64) : none;
#pragma unroll
      for (int t = 0; t < N; ++t) put(st + t * waves, x[t]);
    }
  };
  batch(std::integral_constant<int, 8>{});
  batch(std::integral_constant<int, 2>{});
  for (; st < nfull; st += waves)
    put(st, have ? *reinterpret_cast<const u4*>(p + st * 64) : none);
  if (st == nfull && nfull < end) {  // the padded last step
    u4 x = none;
    const int64_t q0 = nfull * 256 + 64 * g, left = n_f - q0;
    if (have && left > 0) {
      x = *reinterpret_cast<const u4*>(p + nfull * 64);
      // fields past n_f become code 00
#pragma unroll
      for (int q = 0; q < 4; ++q) {
        const int64_t v = left - 16 * q;
        if (v <= 0)
          x[q] = 0u;
        else if (v < 16)
          x[q] &= (1u << (2 * (int)v)) - 1u;
      }
    }
    put(nfull, x);
  }
  // counts: the four lanes of a row, then the waves
#pragma unroll
  for (int o = 16; o < 64; o <<= 1) {
    n1 += __shfl_xor(n1, o);
    miss += __shfl_xor(miss, o);
  }
  if (lane < 16) {
    part[wave][lane][0] = n1;
    part[wave][lane][1] = miss;
  }
  __syncthreads();
  if (threadIdx.x < 16 && 16 * b + threadIdx.x < s.n) {
    const int64_t r = 16 * b + threadIdx.x;
    int a = 0, m = 0;
    for (int w = 0; w < waves; ++w) {
      a += part[w][threadIdx.x][0];
      m += part[w][threadIdx.x][1];
    }
    if (job.shares == 1)
      put_counts(job, s, r, a, m);
    else
      job.part[(int64_t)share * job.set[0].n + r] = make_int2(a, m);
  }
}

}  // namespace
}  // namespace ccc
