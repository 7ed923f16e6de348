// tap_list.hpp -- the variants of the direct tap kernels that are built: basis
// (dimension, degree), radius, mode and coefficient rows.  The linear bases
// keep M in their records, so one variant serves any number of rows; the
// others take K's rows (dim), the consistent mass's one and the dim + 1 of
// c_m M + c_k K.  Radii: a basis of degree n needs n + 1 nodes per axis in the
// corner of a box, so R >= n.
#pragma once
#include "tapconv.hpp"

// X(T, U, dimension, degree, radius, mode, rows) for every basis and radius
#define FC_TAP_LIN(X, T, U, DIM, MODE, ROWS) \
    X(T, U, DIM, 1, 1, MODE, ROWS) X(T, U, DIM, 1, 2, MODE, ROWS) X(T, U, DIM, 1, 3, MODE, ROWS)
#define FC_TAP_QUAD(X, T, U, DIM, MODE, ROWS) X(T, U, DIM, 2, 2, MODE, ROWS) X(T, U, DIM, 2, 3, MODE, ROWS)
#define FC_TAP_CUB(X, T, U, DIM, MODE, ROWS) X(T, U, DIM, 3, 3, MODE, ROWS)
#define FC_TAP_ALL(X, T, U, MODE, R1, R2, R3)                                                                  \
    FC_TAP_LIN(X, T, U, 1, MODE, R1) FC_TAP_LIN(X, T, U, 2, MODE, R2) FC_TAP_LIN(X, T, U, 3, MODE, R3)          \
    FC_TAP_QUAD(X, T, U, 1, MODE, R1) FC_TAP_QUAD(X, T, U, 2, MODE, R2) FC_TAP_QUAD(X, T, U, 3, MODE, R3)       \
    FC_TAP_CUB(X, T, U, 1, MODE, R1) FC_TAP_CUB(X, T, U, 2, MODE, R2)
// K's rows, then the mass's and the shifted operator's of the higher bases
#define FC_TAP_KS(X, T, U, MODE)                                                                               \
    FC_TAP_ALL(X, T, U, MODE, 1, 2, 3)                                                                         \
    FC_TAP_QUAD(X, T, U, 2, MODE, 1) FC_TAP_QUAD(X, T, U, 3, MODE, 1) FC_TAP_CUB(X, T, U, 2, MODE, 1)          \
    FC_TAP_QUAD(X, T, U, 1, MODE, 2) FC_TAP_QUAD(X, T, U, 2, MODE, 3) FC_TAP_QUAD(X, T, U, 3, MODE, 4)         \
    FC_TAP_CUB(X, T, U, 1, MODE, 2) FC_TAP_CUB(X, T, U, 2, MODE, 3)
#define FC_TAP_NODE(X, T, U) FC_TAP_ALL(X, T, U, TAP_UH, 1, 1, 1) FC_TAP_ALL(X, T, U, TAP_LOAD, 1, 1, 1)
// the gradient force and the implicit gradient run in FP64 (in 1D the gradient
// has the one row of u^h)
#define FC_TAP_GRADS(X, T, U)                                                                                  \
    FC_TAP_ALL(X, T, U, TAP_KN, 1, 2, 3)                                                                       \
    FC_TAP_LIN(X, T, U, 2, TAP_UH, 2) FC_TAP_QUAD(X, T, U, 2, TAP_UH, 2) FC_TAP_CUB(X, T, U, 2, TAP_UH, 2)     \
    FC_TAP_LIN(X, T, U, 3, TAP_UH, 3) FC_TAP_QUAD(X, T, U, 3, TAP_UH, 3)

// one list per translation unit
#define FC_TAP_F32(X) FC_TAP_KS(X, float, float, TAP_K) FC_TAP_NODE(X, float, float)
#define FC_TAP_F64(X) FC_TAP_KS(X, double, double, TAP_K)
#define FC_TAP_F64N(X) FC_TAP_NODE(X, double, double) FC_TAP_GRADS(X, double, double)
#define FC_TAP_MIX(X) FC_TAP_KS(X, float, double, TAP_K)
#define FC_TAP_CG32(X) FC_TAP_KS(X, float, float, TAP_CG)
#define FC_TAP_CG64(X) FC_TAP_KS(X, double, double, TAP_CG)

// moments: the basis of twice the degree, in FP64
#define FC_TAP_MOM1(X, DIM, DEG, R) X(double, double, DIM, DEG, R, TAP_MOM, 1)
#define FC_TAP_MOM(X)                                                                                          \
    FC_TAP_MOM1(X, 1, 2, 1) FC_TAP_MOM1(X, 1, 2, 2) FC_TAP_MOM1(X, 1, 2, 3) FC_TAP_MOM1(X, 1, 4, 2)             \
    FC_TAP_MOM1(X, 1, 4, 3) FC_TAP_MOM1(X, 1, 6, 3) FC_TAP_MOM1(X, 2, 2, 1) FC_TAP_MOM1(X, 2, 2, 2)             \
    FC_TAP_MOM1(X, 2, 2, 3) FC_TAP_MOM1(X, 2, 4, 2) FC_TAP_MOM1(X, 2, 4, 3) FC_TAP_MOM1(X, 2, 6, 3)             \
    FC_TAP_MOM1(X, 3, 2, 1) FC_TAP_MOM1(X, 3, 2, 2) FC_TAP_MOM1(X, 3, 2, 3) FC_TAP_MOM1(X, 3, 4, 2)             \
    FC_TAP_MOM1(X, 3, 4, 3)

#define FC_TAP_EXTERN(T, U, DIM, DEG, R, MODE, ROWS) \
    extern template void tap_go<T, U, TapBasis<DIM, DEG>, R, MODE, ROWS>(const TapArgs<T>&, dim3, bool, hipStream_t);
#define FC_TAP_BUILD(T, U, DIM, DEG, R, MODE, ROWS) \
    template void tap_go<T, U, TapBasis<DIM, DEG>, R, MODE, ROWS>(const TapArgs<T>&, dim3, bool, hipStream_t);

namespace fcrkpm {
FC_TAP_F32(FC_TAP_EXTERN)
FC_TAP_F64(FC_TAP_EXTERN)
FC_TAP_F64N(FC_TAP_EXTERN)
FC_TAP_MIX(FC_TAP_EXTERN)
FC_TAP_CG32(FC_TAP_EXTERN)
FC_TAP_CG64(FC_TAP_EXTERN)
FC_TAP_MOM(FC_TAP_EXTERN)
}  // namespace fcrkpm
