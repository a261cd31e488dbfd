// The asynchronous copy of tile2o.h (in asm) between two builtin copies to one
// LDS address: compiled only, to look at what the compiler keeps in m0.
#include "../../paper_1705_08213_amd/csrc/tile2o.h"

using namespace ccc;

__global__ void async_copy_mix(const uint8_t* p, unsigned* out) {
  __shared__ u4 a[2][64];
  tile2::stage_row(p + 16 * threadIdx.x, a[1]);
  tile2::copy_async((gbytes)p, 16 * threadIdx.x, tile2::lds_offset(a[0]));
  tile2::stage_row(p + 4096 + 16 * threadIdx.x, a[1]);
  __syncthreads();
  out[threadIdx.x] = a[0][threadIdx.x].x + a[1][threadIdx.x].x;
}
