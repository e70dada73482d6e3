// Which instances of the matrix-core kernel templates the library holds.  The host file (ftk_api.hip) sees them
// as `extern template` declarations; ftk_instances.hip defines them, one translation unit per (kernel family,
// order) -- selected with -DFTK_INST_FAMILY / -DFTK_INST_ORDER -- so that the build can compile them side by side.
#pragma once
#include "ftk_kernels_mfma16.hpp"
#include "ftk_kernels_tiled.hpp"
#include "ftk_kernels_errors.hpp"
#include "ftk_kernels_owners.hpp"
#include "ftk_kernels_wide.hpp"

// J_n = R = 16 kernel, order N: both sampling rules x the passes, the core phase (a kernel of its own), and the evaluation pass;
// orders 2 to 5 also with two samples of ranks up to 8 side by side
#define FTK_MFMA16_INSTANCES_P(X, XC, N, P)                                               \
    X(N, false, ftk::kSyncPass, P) X(N, false, ftk::kInPlacePass, P) X(N, false, ftk::kFactorPhase, P) XC(N, false, P) \
    X(N, true, ftk::kSyncPass, P) X(N, true, ftk::kInPlacePass, P) X(N, true, ftk::kFactorPhase, P) XC(N, true, P)
#define FTK_MFMA16_INSTANCES(X, XC, XE, N) FTK_MFMA16_INSTANCES_P(X, XC, N, 1) XE(N)
#define FTK_PAIR8_INSTANCES(X, XC, N) FTK_MFMA16_INSTANCES_P(X, XC, N, 2)
// general matrix-core kernel, order N, ranks padded to 16 P (WAVES waves per workgroup): one pass and the two phases of the
// mode-by-mode order, for ranks that are multiples of four and for any; the row-owner form for the former; the evaluation
// pass with rows fetched 16 bytes per lane or float by float
#define FTK_TILED_INSTANCES_P(X, XE, N, P, WAVES)                                                    \
    X(N, P, WAVES, true, false, ftk::kSyncPass) X(N, P, WAVES, false, false, ftk::kSyncPass)          \
    X(N, P, WAVES, true, true, ftk::kSyncPass)                                                        \
    X(N, P, WAVES, true, false, ftk::kFactorPhase) X(N, P, WAVES, false, false, ftk::kFactorPhase)    \
    X(N, P, WAVES, true, false, ftk::kCorePhase) X(N, P, WAVES, false, false, ftk::kCorePhase)        \
    XE(N, P, true) XE(N, P, false)
#define FTK_TILED_INSTANCES(X, XE, N) \
    FTK_TILED_INSTANCES_P(X, XE, N, 1, 8) FTK_TILED_INSTANCES_P(X, XE, N, 2, 8) FTK_TILED_INSTANCES_P(X, XE, N, 4, 4)
// ranks above 32 at orders 2 and 3: the pass of the synchronous and the fused in-place step on a kernel of its own as well
#define FTK_WIDE_INSTANCES(X, N) X(N, true) X(N, false)
#define FTK_GRAD_WIDE(N, X4) template __global__ void ftk::grad_wide_kernel<N, X4>(ftk::TiledArgs);
// orders 9 and 10 (the end of the paper's order sweep): ranks up to 16 only
#define FTK_TILED_INSTANCES_HIGH(X, XE, N) FTK_TILED_INSTANCES_P(X, XE, N, 1, 8)

// evaluation pass over projected rows, order N: 1, 2, 4, 8 or 16 lanes per entry
#define FTK_ROWS_INSTANCES(X, N) X(N, 1) X(N, 2) X(N, 4) X(N, 8) X(N, 16)
#define FTK_HOT_INSTANCES(X, N) X(N, 1) X(N, 2) X(N, 4)   // with the frequent rows in LDS

// row owners, order N >= 2: 1 or 2 lanes per sample
#define FTK_APPEND_INSTANCES(X, N) X(N, 1) X(N, 2)

#define FTK_APPEND(N, G) template __global__ void ftk::append_lists_kernel<N, G>(ftk::AppendArgs);
#define FTK_ERRORS_ROWS(N, G) template __global__ void ftk::errors_rows_kernel<N, G, false>(ftk::Coo, uint64_t, ftk::ErrorRows, double*);
#define FTK_ERRORS_HOT(N, G) template __global__ void ftk::errors_rows_kernel<N, G, true>(ftk::Coo, uint64_t, ftk::ErrorRows, double*);
#define FTK_GRAD_MFMA16(N, T, M, P) template __global__ void ftk::grad_mfma16_kernel<N, T, M, P>(ftk::Mfma16Args);
#define FTK_CORE_MFMA16(N, T, P) template __global__ void ftk::core_phase_mfma16_kernel<N, T, P>(ftk::Mfma16Args);
#define FTK_ERRORS_MFMA16(N) \
    template __global__ void ftk::errors_mfma16_kernel<N>(ftk::Coo, uint64_t, const float*, const float*, ftk::Layout, ftk::ModeBytes, double*);
#define FTK_GRAD_TILED(N, P, W, X4, R, M) template __global__ void ftk::grad_tiled_kernel<N, P, W, X4, R, M>(ftk::TiledArgs);
#define FTK_ERRORS_TILED(N, P, X4) \
    template __global__ void ftk::errors_tiled_kernel<N, P, X4>(ftk::Coo, uint64_t, const float*, const float*, ftk::Layout, ftk::TiledModeBytes, double*);

#define FTK_ALL_INSTANCES(PREFIX_GM, PREFIX_CM, PREFIX_EM, PREFIX_GT, PREFIX_ET)                          \
    FTK_MFMA16_INSTANCES(PREFIX_GM, PREFIX_CM, PREFIX_EM, 1) FTK_MFMA16_INSTANCES(PREFIX_GM, PREFIX_CM, PREFIX_EM, 2)           \
    FTK_MFMA16_INSTANCES(PREFIX_GM, PREFIX_CM, PREFIX_EM, 3) FTK_MFMA16_INSTANCES(PREFIX_GM, PREFIX_CM, PREFIX_EM, 4)           \
    FTK_MFMA16_INSTANCES(PREFIX_GM, PREFIX_CM, PREFIX_EM, 5) FTK_MFMA16_INSTANCES(PREFIX_GM, PREFIX_CM, PREFIX_EM, 6)           \
    FTK_TILED_INSTANCES(PREFIX_GT, PREFIX_ET, 1) FTK_TILED_INSTANCES(PREFIX_GT, PREFIX_ET, 2)         \
    FTK_TILED_INSTANCES(PREFIX_GT, PREFIX_ET, 3) FTK_TILED_INSTANCES(PREFIX_GT, PREFIX_ET, 4)         \
    FTK_TILED_INSTANCES(PREFIX_GT, PREFIX_ET, 5) FTK_TILED_INSTANCES(PREFIX_GT, PREFIX_ET, 6)             \
    FTK_TILED_INSTANCES(PREFIX_GT, PREFIX_ET, 7) FTK_TILED_INSTANCES(PREFIX_GT, PREFIX_ET, 8)             \
    FTK_TILED_INSTANCES_HIGH(PREFIX_GT, PREFIX_ET, 9) FTK_TILED_INSTANCES_HIGH(PREFIX_GT, PREFIX_ET, 10)

#ifdef FTK_INSTANCES_EXTERN
// the host file: every instance is defined elsewhere
#define FTK_X_GM(N, T, M, P) extern FTK_GRAD_MFMA16(N, T, M, P)
#define FTK_X_CM(N, T, P) extern FTK_CORE_MFMA16(N, T, P)
#define FTK_X_EM(N) extern FTK_ERRORS_MFMA16(N)
#define FTK_X_GT(N, P, W, X4, R, M) extern FTK_GRAD_TILED(N, P, W, X4, R, M)
#define FTK_X_ET(N, P, X4) extern FTK_ERRORS_TILED(N, P, X4)
FTK_ALL_INSTANCES(FTK_X_GM, FTK_X_CM, FTK_X_EM, FTK_X_GT, FTK_X_ET)
FTK_PAIR8_INSTANCES(FTK_X_GM, FTK_X_CM, 2) FTK_PAIR8_INSTANCES(FTK_X_GM, FTK_X_CM, 3)
FTK_PAIR8_INSTANCES(FTK_X_GM, FTK_X_CM, 4) FTK_PAIR8_INSTANCES(FTK_X_GM, FTK_X_CM, 5)
#define FTK_X_GW(N, X4) extern FTK_GRAD_WIDE(N, X4)
FTK_WIDE_INSTANCES(FTK_X_GW, 2) FTK_WIDE_INSTANCES(FTK_X_GW, 3)
#define FTK_X_ER(N, G) extern FTK_ERRORS_ROWS(N, G)
#define FTK_X_EH(N, G) extern FTK_ERRORS_HOT(N, G)
FTK_HOT_INSTANCES(FTK_X_EH, 1) FTK_HOT_INSTANCES(FTK_X_EH, 2) FTK_HOT_INSTANCES(FTK_X_EH, 3) FTK_HOT_INSTANCES(FTK_X_EH, 4)
FTK_HOT_INSTANCES(FTK_X_EH, 5) FTK_HOT_INSTANCES(FTK_X_EH, 6) FTK_HOT_INSTANCES(FTK_X_EH, 7) FTK_HOT_INSTANCES(FTK_X_EH, 8)
FTK_HOT_INSTANCES(FTK_X_EH, 9) FTK_HOT_INSTANCES(FTK_X_EH, 10)
FTK_ROWS_INSTANCES(FTK_X_ER, 1) FTK_ROWS_INSTANCES(FTK_X_ER, 2) FTK_ROWS_INSTANCES(FTK_X_ER, 3) FTK_ROWS_INSTANCES(FTK_X_ER, 4)
FTK_ROWS_INSTANCES(FTK_X_ER, 5) FTK_ROWS_INSTANCES(FTK_X_ER, 6) FTK_ROWS_INSTANCES(FTK_X_ER, 7) FTK_ROWS_INSTANCES(FTK_X_ER, 8)
FTK_ROWS_INSTANCES(FTK_X_ER, 9) FTK_ROWS_INSTANCES(FTK_X_ER, 10)
#define FTK_X_AP(N, G) extern FTK_APPEND(N, G)
FTK_APPEND_INSTANCES(FTK_X_AP, 2) FTK_APPEND_INSTANCES(FTK_X_AP, 3) FTK_APPEND_INSTANCES(FTK_X_AP, 4)
FTK_APPEND_INSTANCES(FTK_X_AP, 5) FTK_APPEND_INSTANCES(FTK_X_AP, 6) FTK_APPEND_INSTANCES(FTK_X_AP, 7)
FTK_APPEND_INSTANCES(FTK_X_AP, 8) FTK_APPEND_INSTANCES(FTK_X_AP, 9) FTK_APPEND_INSTANCES(FTK_X_AP, 10)
#endif
