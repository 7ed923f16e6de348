// tap_list.hpp -- the variants of the direct tap kernels that are built: basis
// (dimension, degree), radius, mode and coefficient rows.  The linear bases
// keep M in their records, so one variant serves any number of rows; the
// others take K's rows (dim), the consistent mass's one and the dim + 1 of
// c_m M + c_k K.  Radii: a basis of degree n needs n + 1 nodes per axis in the
// corner of a box, so R >= n.
#pragma once
#include "tapconv.hpp"

#define FC_TAP_LIN(X, T, U, DIM) \
    X(T, U, DIM, 1, 1, TAP_K, DIM) X(T, U, DIM, 1, 2, TAP_K, DIM) X(T, U, DIM, 1, 3, TAP_K, DIM)
#define FC_TAP_R2(X, T, U, DIM, DEG, ROWS) X(T, U, DIM, DEG, 2, TAP_K, ROWS)
#define FC_TAP_R3(X, T, U, DIM, DEG, ROWS) X(T, U, DIM, DEG, 3, TAP_K, ROWS)
// 1D and 2D
#define FC_TAP_LOW(X, T, U)                                                                                     \
    FC_TAP_LIN(X, T, U, 1) FC_TAP_LIN(X, T, U, 2)                                                               \
    FC_TAP_R2(X, T, U, 1, 2, 1) FC_TAP_R3(X, T, U, 1, 2, 1) FC_TAP_R2(X, T, U, 1, 2, 2)                         \
    FC_TAP_R3(X, T, U, 1, 2, 2) FC_TAP_R2(X, T, U, 2, 2, 1) FC_TAP_R3(X, T, U, 2, 2, 1)                         \
    FC_TAP_R2(X, T, U, 2, 2, 2) FC_TAP_R3(X, T, U, 2, 2, 2) FC_TAP_R2(X, T, U, 2, 2, 3)                         \
    FC_TAP_R3(X, T, U, 2, 2, 3) FC_TAP_R3(X, T, U, 1, 3, 1) FC_TAP_R3(X, T, U, 1, 3, 2)                         \
    FC_TAP_R3(X, T, U, 2, 3, 1) FC_TAP_R3(X, T, U, 2, 3, 2) FC_TAP_R3(X, T, U, 2, 3, 3)
// 3D
#define FC_TAP_3D(X, T, U)                                                                                      \
    FC_TAP_LIN(X, T, U, 3)                                                                                      \
    FC_TAP_R2(X, T, U, 3, 2, 1) FC_TAP_R2(X, T, U, 3, 2, 3) FC_TAP_R2(X, T, U, 3, 2, 4)                         \
    FC_TAP_R3(X, T, U, 3, 2, 1) FC_TAP_R3(X, T, U, 3, 2, 3) FC_TAP_R3(X, T, U, 3, 2, 4)

#define FC_TAP_F32(X) FC_TAP_LOW(X, float, float) FC_TAP_3D(X, float, float)
#define FC_TAP_F64(X) FC_TAP_LOW(X, double, double) FC_TAP_3D(X, double, double)
#define FC_TAP_MIX(X) FC_TAP_LOW(X, float, double) FC_TAP_3D(X, float, double)

#define FC_TAP_EXTERN(T, U, DIM, DEG, R, MODE, ROWS) \
    extern template void tap_go<T, U, TapBasis<DIM, DEG>, R, MODE, ROWS>(const TapArgs<T>&, dim3, hipStream_t);
#define FC_TAP_BUILD(T, U, DIM, DEG, R, MODE, ROWS) \
    template void tap_go<T, U, TapBasis<DIM, DEG>, R, MODE, ROWS>(const TapArgs<T>&, dim3, hipStream_t);

namespace fcrkpm {
FC_TAP_F32(FC_TAP_EXTERN)
FC_TAP_F64(FC_TAP_EXTERN)
FC_TAP_MIX(FC_TAP_EXTERN)
}  // namespace fcrkpm
