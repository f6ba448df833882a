// The products for a few right-hand sides (endor_gemv.hip), as the small-batch product's entry point calls them.
#ifndef ENDOR_GEMV_H_
#define ENDOR_GEMV_H_

#include <hip/hip_runtime.h>

#include <cstdint>

namespace endor_gemv {

constexpr int kMaxRhs = 4;

struct SmallProduct {
    const uint64_t *bitmap;
    const uint16_t *values;
    const uint32_t *chunk_total, *tile_off;  // the offset table
    const uint16_t *x;
    float *y;
    int64_t rows, cols, nnz, ldx;
    int nb;
};

// Whether the vector form is the faster one for nb right-hand sides.  Measured, us, the form on the matrix
// cores / this one:
//  - short rows, many of them: 36864 x 768 and one right-hand side 18.6 / 19 to 21, 131072 x 256 22 / 104;
//    12000 x 600 13 / 9.5, 20000 x 1200 24 / 16, 36864 x 1500 with two 29.6 / 27.4, with three 29.6 / 30.2;
//  - all of x has to fit LDS: two right-hand sides 4096 x 20000 39 / 28, 8192 x 28672 74 / 82; three
//    2000 x 16000 21.7 / 19.2, 4096 x 20000 39 / 46;
//  - four only pay on small matrices: 4096 x 4096 15 / 12, 12000 x 2500 27 / 22, 16384 x 4096 27 / 29,
//    36864 x 9216 107 / 117;
//  - else 28672 x 8192 with one to three 75 / 52, 59, 70; 4099 x 5005, three in ten kept, 18 / 12, 14, 15.
//  cols >= 8: shorter vectors are read element by element, which is there for one right-hand side only.
constexpr bool takes(int64_t rows, int64_t cols, int nb) {
    if (cols < 8 || nb > kMaxRhs || cols * nb > 48 * 1024) return false;
    if (nb == 4 && rows * cols > int64_t(1) << 25) return false;
    return rows <= 16384 || cols >= 1024 * (nb == 1 ? 1 : nb == 2 ? 1.4 : 2);
}

// y of those products; the arguments are checked.
void small_product(const SmallProduct &p, hipStream_t s);

// count zeros
void zero(float *y, int64_t count, hipStream_t s);

}  // namespace endor_gemv

#endif  // ENDOR_GEMV_H_
