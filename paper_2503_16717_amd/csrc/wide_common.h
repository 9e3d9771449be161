// Device helpers shared by the wide-block kernels (wide_kernels.hip, wide_fused.hip): the
// row operation's solve and element addressing, and the 4-row operand pieces of the FP64
// MFMA 16 x 16 x 4 tiles.
#pragma once
#include <hip/hip_runtime.h>

#include <cstdint>
#include <type_traits>

#include "sko_internal.h"
#include "uniform.h"

namespace sko {
namespace wide {

template <typename T>
__device__ __forceinline__ double ldv(const T* p) {
    return static_cast<double>(*p);
}
// The row operation's input and output columns stream through it once: non-temporal.
template <typename T>
__device__ __forceinline__ double ldv_nt(const T* p) {
    return static_cast<double>(__builtin_nontemporal_load(p));
}
template <typename T>
__device__ __forceinline__ void stv_nt(T* p, T v) {
    __builtin_nontemporal_store(v, p);
}

constexpr int ROW_NT = 256;

struct RowopArgs {
    int64_t n;
    int w;
    const void* Y;
    int64_t ldy;
    const void* Qu;
    int64_t ldqu;
    int pu;
    const double* Cu;
    const double* Rpk;   // packed factor: w reciprocal diagonal entries, then column c's c
                         // strictly upper entries at w + c(c-1)/2
    void* X;
    int64_t ldx;
    // further factors, solved with after Rpk in this order (same packed form)
    const double* Rpk2 = nullptr;
    const double* Rpk3 = nullptr;
    int pw = 0;  // FP32 storage: panel width of Rpk's columns (solve_cols)
};

// v - sum_{q < c} x[q] Rc[q] for column c of a triangular solve, the factor entries loaded
// in chunks of 8 (one chunk ahead of the FMAs that use it) so that only two chunks occupy
// SGPRs at a time.
template <int WB, int C>
__device__ __forceinline__ double solve_col(const double (&x)[WB], CD Rc, double v) {
    constexpr int NCH = (C + 7) / 8;
    if constexpr (NCH > 0) {
        double r[2][8];
#pragma unroll
        for (int u = 0; u < 8; ++u)
            if (u < C) r[0][u] = Rc[u];
#pragma unroll
        for (int k = 0; k < NCH; ++k) {
            if (k + 1 < NCH) {
#pragma unroll
                for (int u = 0; u < 8; ++u)
                    if (8 * (k + 1) + u < C) r[(k + 1) & 1][u] = Rc[8 * (k + 1) + u];
            }
            __builtin_amdgcn_sched_barrier(0);
#pragma unroll
            for (int u = 0; u < 8; ++u)
                if (8 * k + u < C) v -= x[8 * k + u] * r[k & 1][u];
            __builtin_amdgcn_sched_barrier(0);
        }
    }
    return v;
}

template <typename T, int WB, int CNT>
__device__ __forceinline__ void round_cols(double (&x)[WB]) {
    if constexpr (sizeof(T) == 4) {
#pragma unroll
        for (int q = 0; q < CNT; ++q) x[q] = static_cast<double>(static_cast<T>(x[q]));
    }
}

// PW (FP32 storage, panel width pw, bnd = pw): a panel's columns are rounded to the storage type
// when the next panel begins, as panels stored one by one are.  The branch per column that this
// takes stays out of the other solves (61 FP32 columns, 7.1 million rows: 1.12 against 0.91 ms).
template <typename T, int WB, int C, bool PW>
__device__ __forceinline__ void solve_cols(double (&x)[WB], CD Rs, int w, const double* sD, int pw, int bnd) {
    if constexpr (C < WB) {
        if (C < w) {
            if constexpr (PW && sizeof(T) == 4 && C > 0) {
                if (C == bnd) {
                    round_cols<T, WB, C>(x);
                    bnd += pw;
                }
            }
            x[C] = solve_col<WB, C>(x, Rs + w + C * (C - 1) / 2, x[C]) * sD[C];
            solve_cols<T, WB, C + 1, PW>(x, Rs, w, sD, pw, bnd);
        }
    }
}

// x R1^{-1} [R2^{-1} [R3^{-1}]]; between the factors the row is rounded to the storage type, so
// a chain gives what storing and loading the rows between the solves gives.
template <typename T, int WB, int TRSM, bool PW>
__device__ __forceinline__ void solve_chain(double (&x)[WB], CD R1, CD R2, CD R3, int w, const double* sD, int pw) {
    if constexpr (TRSM >= 1) solve_cols<T, WB, 0, PW>(x, per_strip(R1), w, sD, pw, pw);
    if constexpr (TRSM >= 2) {
        round_cols<T, WB, WB>(x);
        solve_cols<T, WB, 0, false>(x, per_strip(R2), w, sD + WB, 0, 0);
    }
    if constexpr (TRSM >= 3) {
        round_cols<T, WB, WB>(x);
        solve_cols<T, WB, 0, false>(x, per_strip(R3), w, sD + 2 * WB, 0, 0);
    }
}

// The reciprocal diagonals of the TRSM factors of ra into LDS, WB apart.
template <int WB, int TRSM>
__device__ __forceinline__ void stage_diagonals(const RowopArgs& ra, double* sD) {
    for (int i = threadIdx.x; i < TRSM * WB; i += ROW_NT) {
        const int t = i / WB, c = i - t * WB;
        if (c < ra.w) sD[i] = (t == 0 ? ra.Rpk : t == 1 ? ra.Rpk2 : ra.Rpk3)[c];
    }
}

// The element a lane handles in a column, given the column's address at the strip's first
// row (the same for the whole workgroup, so it is formed in SGPRs) and the lane's byte
// offset in the strip (one VGPR shared by every column).
template <typename T>
__device__ __forceinline__ T* lane_elem(T* strip_col, uint32_t lane_bytes) {
    using B = typename std::conditional<std::is_const<T>::value, const char, char>::type;
    return reinterpret_cast<T*>(reinterpret_cast<B*>(strip_col) + lane_bytes);
}

constexpr int GT = 256;   // threads (4 waves)
static_assert(16 * (GT / 64) == kGemmUnitRows, "a workgroup index covers 16 rows per wave");

typedef double double4_t __attribute__((ext_vector_type(4)));

struct GemmArgs {
    int64_t n;
    const void* A;
    int64_t lda;
    int ma;
    const void* B;
    int64_t ldb;
    int nb;
    double* partials;
    int64_t stride;
};

// Rows row0..row0+3 of one column into v (zero past n or for a column past the block).
template <typename T>
__device__ __forceinline__ void load_piece(const T* col, bool live, int64_t row0, int64_t n, double (&v)[4]) {
    if (live && row0 + 3 < n) {
        load4(col + row0, v);
    } else {
#pragma unroll
        for (int u = 0; u < 4; ++u) v[u] = (live && row0 + u < n) ? ldv(col + row0 + u) : 0.0;
    }
}

// The four pieces (16-column tiles t) of one operand for a group of 16 rows.  In a full
// group every lane loads every piece without a branch: a column past m reads column m - 1
// (lines already requested) and is zeroed after the loads, so all loads of the group are in
// flight together.  A branch per piece would wait for each load in turn.  The group at the
// end of the rows keeps the guarded loads.
template <typename T, int NTL>
__device__ __forceinline__ void load_pieces(const T* base, int64_t ld, int m, int ci, bool full, int64_t row0,
                                            int64_t n, double (&v)[NTL][4]) {
    if (full) {
#pragma unroll
        for (int t = 0; t < NTL; ++t) {
            const int c = 16 * t + ci;
            load4(base + (int64_t)(c < m ? c : m - 1) * ld + row0, v[t]);
        }
#pragma unroll
        for (int t = 0; t < NTL; ++t)
            if (16 * t + ci >= m) v[t][0] = v[t][1] = v[t][2] = v[t][3] = 0.0;
    } else {
#pragma unroll
        for (int t = 0; t < NTL; ++t) {
            const int c = 16 * t + ci;
            load_piece(base + (int64_t)(c < m ? c : 0) * ld, c < m, row0, n, v[t]);
        }
    }
}

}  // namespace wide
}  // namespace sko
