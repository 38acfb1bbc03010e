// The 128x128 tiles of gemm_mid.h: two workgroups per CU, so one's epilogue
// runs beside the other's K loop; the shorter K and the finer grid.
#include "gemm_mid.h"

namespace adept {

adept_status gemm_mid_128x128(GP p, int epi, const char* name, float* ws, size_t ws_bytes,
                              hipStream_t s) {
  return gemm_mid<Geo<128, 128>>(p, epi, name, ws, ws_bytes, s);
}

}  // namespace adept
