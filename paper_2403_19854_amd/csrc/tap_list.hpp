// tap_list.hpp -- the variants of the direct tap kernels that are built: basis
// (dimension, degree), radius, mode and coefficient rows.  The linear bases
// keep M in their records, so one variant serves any number of rows.
#pragma once
#include "tapconv.hpp"

#define FC_TAP_LIN(X, T, U, DIM, MODE) X(T, U, DIM, 1, 1, MODE, DIM) X(T, U, DIM, 1, 2, MODE, DIM) X(T, U, DIM, 1, 3, MODE, DIM)
#define FC_TAP_K_LIN(X, T, U) FC_TAP_LIN(X, T, U, 3, TAP_K)
#define FC_TAP_F32(X) FC_TAP_K_LIN(X, float, float)
#define FC_TAP_F64(X) FC_TAP_K_LIN(X, double, double)
#define FC_TAP_MIX(X) FC_TAP_K_LIN(X, float, double)

#define FC_TAP_EXTERN(T, U, DIM, DEG, R, MODE, ROWS) \
    extern template void tap_go<T, U, TapBasis<DIM, DEG>, R, MODE, ROWS>(const TapArgs<T>&, dim3, hipStream_t);
#define FC_TAP_BUILD(T, U, DIM, DEG, R, MODE, ROWS) \
    template void tap_go<T, U, TapBasis<DIM, DEG>, R, MODE, ROWS>(const TapArgs<T>&, dim3, hipStream_t);

namespace fcrkpm {
FC_TAP_F32(FC_TAP_EXTERN)
FC_TAP_F64(FC_TAP_EXTERN)
FC_TAP_MIX(FC_TAP_EXTERN)
}  // namespace fcrkpm
