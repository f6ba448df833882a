// The products for a few right-hand sides (endor_gemv.hip), as the small-batch product's entry point calls them.
#ifndef ENDOR_GEMV_H_
#define ENDOR_GEMV_H_

#include <hip/hip_runtime.h>

#include <cstdint>

namespace endor_gemv {

struct SmallProduct {
    const uint64_t *bitmap;
    const uint16_t *values;
    const uint32_t *chunk_total, *tile_off;  // the offset table
    const uint16_t *x;
    float *y;
    int64_t rows, cols, nnz, ldx;
    int nb;
};

// y of those products; the arguments are checked.
void small_product(const SmallProduct &p, hipStream_t s);

// count zeros
void zero(float *y, int64_t count, hipStream_t s);

}  // namespace endor_gemv

#endif  // ENDOR_GEMV_H_
