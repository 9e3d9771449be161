// Internal declarations of the s-step GMRES kernels.
#pragma once

#include <hip/hip_runtime.h>

#include <algorithm>
#include <cstdint>

#include "sko_internal.h"

namespace sko {

struct BatchSys;

// A matrix whose nonzeros lie on at most kMaxDiags diagonals, in diagonal storage: value k of
// row i (column i + off[k], off ascending) at val[k * ld + i], zero where the row has none.
constexpr int kMaxDiags = 16;
constexpr int64_t kDiaMinVectors = 4;  // shortest solve whose set-up looks for diagonals
struct DiaView {
    const void* val = nullptr;  // MPK operator values (double or float); null: not in this form
    int64_t ld = 0;
    int nd = 0;
    int32_t off[kMaxDiags] = {};
};

// Words csr_check writes: [0] nonzero if the structure is invalid, [1] nonzero if some row's
// columns are not strictly ascending or there are more than kMaxDiags diagonals, [2..] the
// diagonals' offsets plus 2^31 (unsigned) in no order, 0 where unused.  All zero before the
// launch.
constexpr int kScanWords = 2 + kMaxDiags;
// Diagonals of a scanned matrix (ascending in d.off, d.nd of them); false where diagonal storage
// does not pay: eb bytes a value on every row and diagonal against the CSR form's values,
// column indices and row pointers.  A 7-point stencil moves 56 + 16 bytes per row instead of
// 88 + 16 (FP64), a matrix with many part-filled diagonals would move more.  The line lies at 0.85 of
// the CSR bytes: an SpMV still gains beyond it at 2^20 rows (us, CSR | diagonals, FP64: 9 diagonals at
// 0.87 30.6 | 21.0, 13 at 1.02 34.2 | 27.6) but not at 2^16 (13 at 1.02 6.5 | 7.1), the storage grows
// with it, and so does the set-up.
bool scan_diagonals(const int32_t* words, int64_t n, int64_t nnz, int eb, DiaView& d);

// CSR operand: structure + FP64 values of A (explicit residual) and the values used by
// the matrix-powers kernel (A D^{-1} in double or float, or A itself).
struct CsrView {
    int64_t n;
    int64_t nnz;
    const int32_t* rowptr;
    const int32_t* colind;
    const double* val;     // A, double
    const void* val_op;    // MPK operator values (double or float)
    DiaView dia;           // the same values by diagonals (dia.val null: not)
};

// y = A x, or with a Newton step (na != null) y = A x - (*na) x + (*nb) z (na, nb: device
// scalars; z: the basis vector before x, read only where *nb != 0).
hipError_t launch_spmv(const CsrView& A, bool f32, const void* x, void* y, int grid_cap, hipStream_t st,
                       const double* na = nullptr, const double* nb = nullptr, const void* z = nullptr);
// Mixed precision: one matrix-powers step of the FP64 panel (FP32 operator values, FP64
// vectors), and the widening copy of an FP32 basis column into the panel.
hipError_t launch_spmv_panel(const CsrView& A, const double* x, double* y, int grid_cap, hipStream_t st,
                             const double* na = nullptr, const double* nb = nullptr, const double* z = nullptr);
hipError_t launch_widen(int64_t n, const float* x, double* y, int grid_cap, hipStream_t st);
int residual_grid(int64_t n, int grid_cap);
hipError_t launch_residual(const CsrView& A, const double* x, const double* b, bool f32, void* r, double* partials,
                           int grid, hipStream_t st);
hipError_t launch_update(int64_t n, bool f32, const void* Q, int64_t ldq, int k, const double* y,
                         const double* dinv, double* x, hipStream_t st);
// `words`: kScanWords ints, zero.  scan: look for the diagonals too (without it words[1] is set).
hipError_t launch_csr_check(int64_t n, int64_t nnz, const int32_t* rowptr, const int32_t* colind, bool scan,
                            int* words, hipStream_t st);
// d.val from the CSR values (scaled by dinv[column] if given).
hipError_t launch_fill_diagonals(int64_t n, int64_t nnz, const int32_t* rowptr, const int32_t* colind,
                                 const double* val, const double* dinv, bool f32, const DiaView& d, hipStream_t st);
// Whether a matrix's rows are staged in two halves (more entries per row than one part holds);
// `halves` below: whether any system's are.
bool long_rows(int64_t n, int64_t nnz);
// The set-up of many systems in one launch each: system i's row of the device table `sys` (a
// system with n = 0 is left alone), its check words at words + 32 i, its status word (Jacobi)
// i * pitch bytes behind status0.
hipError_t launch_csr_check_batched(int nsys, int64_t max_n, const BatchSys* sys, bool scan, bool halves, int* words,
                                    hipStream_t st);
hipError_t launch_jacobi_setup_batched(int nsys, int64_t max_n, const BatchSys* sys, void* status0, int64_t pitch,
                                       hipStream_t st);
hipError_t launch_fill_diagonals_batched(int nsys, int64_t max_n, const BatchSys* sys, bool f32, bool halves,
                                         hipStream_t st);
hipError_t launch_jacobi_setup(int64_t n, int64_t nnz, const int32_t* rowptr, const int32_t* colind,
                               const double* val, double* dinv, int* status, hipStream_t st);
hipError_t launch_scale_values(int64_t nnz, const int32_t* colind, const double* val, const double* dinv, bool f32,
                               void* out, hipStream_t st);

enum GmOp : int {
    GM_INIT = 0,      // T_in = T_out = 0, g = beta e_1
    GM_BLOCK = 1,     // rewrite the boundary vector kk, store an s-step block, optional LSQ
    GM_BIGCLOSE = 2,  // express the closed big panel in the final basis, then LSQ
};

struct GmSmallArgs {
    int op;
    int m, s;
    int kk;            // GM_BLOCK: basis index of the block's start vector
    int k0;            // two-stage: first column of the current big panel
    int two_stage;
    int do_lsq;
    int Wb, kend;      // GM_BIGCLOSE: big-panel width and the basis size after it
    double* Tin;       // (m+1) x m
    double* Tout;      // (m+1) x m
    double* g;         // m+1
    double* gw;        // m+1 scratch
    double* H;         // (m+1) x m scratch
    double* y;         // m
    double* res;       // 1: implicit residual norm
    const double* beta;  // GM_INIT
    double* coef;      // (m+1) x (s+1) block coefficients (ld m+1)
    const double* Cpan;  // two-stage: k0 x (s+1) projection coefficients of the panel
    const double* Rh;  // GM_BIGCLOSE: Wb x Wb
    const double* Rt;  // GM_BIGCLOSE: Wb x Wb or null (identity)
    const double* C2;  // GM_BIGCLOSE: k0 x Wb or null
    // GM_BLOCK with the Newton basis: recurrence coefficients a (s) then b (s); null: monomial
    const double* newton;
    // GM_BLOCK with least squares, one system: mapped host words that receive the implicit
    // residual ([0]) and the status word (int at [1]) when the step ends (null: none)
    double* host_res;
    const int* status_in;
};

hipError_t launch_gm_small(const GmSmallArgs& a, hipStream_t st, const BatchReloc* br = nullptr);
// Ritz values of the leading k x k Hessenberg matrix (k <= 64) -> Newton coefficients (2 s).
hipError_t launch_ritz(const GmSmallArgs& a, int k, double* newton, hipStream_t st);

// Batched forms (batch.h): one launch for every active system; x, y, r and Q are template
// basis addresses, partials and y template workspace addresses.
// Rows one workgroup iteration of the batched SpMV covers for this value type and mean row
// length; the flat launch's BatchReloc::chunk is a multiple of it.
int spmv_flat_unit(bool f32, double avg_nnz, bool dia);
hipError_t launch_spmv_batched(bool f32, double avg_nnz, bool dia, int64_t max_n, const void* x, void* y, int grid_cap,
                               hipStream_t st, const BatchReloc& br);
hipError_t launch_residual_batched(bool f32, double avg_nnz, void* r, double* partials, int grid, hipStream_t st,
                                   const BatchReloc& br);
hipError_t launch_update_batched(bool f32, int64_t max_n, const void* Q, int max_k, const double* y, hipStream_t st,
                                 const BatchReloc& br);

}  // namespace sko
