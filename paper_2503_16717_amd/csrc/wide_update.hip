// The wide update X = Y - Q C of a big panel (up to 64 columns) against p previous columns,
// optionally with the Gram matrix X^T X in the same sweep (Fig. 6: the BCGS steps of the
// two-stage scheme).
//
// Work per row: p + w columns read, w written, p w FMAs; 36 columns on 36 move 108 x 8 bytes
// for 2592 flops, so the sweep is HBM-bound.  The product runs on v_mfma_f64_16x16x4 with the
// panel's columns as the tile's rows: a wave takes 32 rows, lane l rows 2 (l % 16) and
// 2 (l % 16) + 1, and
//   B operand  Q[row][4s + l / 16], one 16-byte load for both row halves (256 bytes of a column
//              per 16 lanes, 1 KiB per wave instruction);
//   A operand  -C[4s + l / 16][16t + l % 16], staged once per workgroup in LDS;
//   D          columns 16t + l / 16 + 4e of the lane's rows: Y loads straight into it and X
//              stores straight from it, with the same 256-byte column segments.
// A lane so keeps 8 values per 16-column tile where one row per thread keeps the whole row
// (72 VGPRs at 36 columns) and waits for scalar loads of C: at n = 2^24, 36 columns on 36,
// that form took 3.34 ms (4.3 TB/s) and its Gram matrix another 1.11 ms.
//
// Gram: D holds rows across lanes, the contraction over rows wants columns across lanes, so
// each wave passes its 16-row halves through LDS (column stride 18 doubles, as the fused row
// solve does).  Columns past the panel width repeat its last column; they only reach output
// entries that are never written.
#include <algorithm>

#include "batch.h"
#include "sko_internal.h"
#include "uniform.h"
#include "wide_common.h"

namespace sko {
namespace {

using namespace wide;

struct UpdateArgs {
    int64_t n;
    int w;
    const void* Y;
    int64_t ldy;
    const void* Q;
    int64_t ldq;
    int p;
    const double* C;  // p x w, column-major, ld p
    void* X;
    int64_t ldx;
    double* partials;  // Gram: w * w per workgroup
    int64_t stride;
};

constexpr int SLD = 18;  // staged column stride in doubles (16 rows + 2)
constexpr int NW = GT / 64;

__device__ __forceinline__ void wave_sync() {
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

// Rows row0, row0 + 1 of a column; the guarded form reads zero at or beyond n.
template <typename T>
__device__ __forceinline__ typename Unaligned<T>::v2 load_pair(const T* col, int64_t row0, int64_t n, bool full) {
    typedef typename Unaligned<T>::v2 V;
    if (full) return __builtin_nontemporal_load(reinterpret_cast<const V*>(col + row0));
    V v;
    v.x = row0 < n ? col[row0] : T(0);
    v.y = row0 + 1 < n ? col[row0 + 1] : T(0);
    return v;
}

constexpr int KG = 4;  // k-steps (of 4 columns of Q) loaded ahead

template <typename T, int TX, bool GRAM>
__device__ __forceinline__ void update_body(const UpdateArgs& ua, const int wg, const int nwg) {
    typedef typename Unaligned<T>::v2 V;
    extern __shared__ double upd_lds[];
    constexpr int LC = 16 * TX;
    const int64_t n = ua.n;
    const int w = ua.w, p = ua.p;
    const int ksteps = (p + 3) / 4;
    const T* Y = static_cast<const T*>(ua.Y);
    const T* Q = static_cast<const T*>(ua.Q);
    T* X = static_cast<T*>(ua.X);
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6, ci = lane & 15, g = lane >> 4;
    double* sc = upd_lds;  // -C, 4 ksteps rows of LC, zero outside p x w
    for (int i = tid; i < 4 * ksteps * LC; i += GT) {
        const int k = i / LC, c = i - k * LC;
        sc[i] = (k < p && c < w) ? -ua.C[k + (int64_t)c * p] : 0.0;
    }
    __syncthreads();
    double* st = upd_lds + 4 * ksteps * LC + wave * (LC * SLD);
    double4_t gacc[GRAM ? TX : 1][GRAM ? TX : 1];
    if constexpr (GRAM) {
#pragma unroll
        for (int i = 0; i < TX; ++i)
#pragma unroll
            for (int j = 0; j < TX; ++j) gacc[i][j] = double4_t{0.0, 0.0, 0.0, 0.0};
    }

    const int64_t ngroups = (n + 31) / 32;
    for (int64_t grp = (int64_t)wg * NW + wave; grp < ngroups; grp += (int64_t)nwg * NW) {
        const int64_t row0 = grp * 32 + 2 * ci;
        const bool full = grp * 32 + 32 <= n;
        // Y into the accumulators' layout, and the first columns of Q behind it
        double4_t acc[2][TX];
        V y[TX][4];
#pragma unroll
        for (int t = 0; t < TX; ++t)
#pragma unroll
            for (int e = 0; e < 4; ++e) {
                const int c = 16 * t + g + 4 * e;
                y[t][e] = load_pair(Y + (int64_t)(c < w ? c : w - 1) * ua.ldy, row0, n, full);
            }
        V q[2][KG];
        auto load_q = [&](V(&d)[KG], int s0) {
#pragma unroll
            for (int s = 0; s < KG; ++s) {
                const int k = 4 * (s0 + s) + g;
                d[s] = load_pair(Q + (int64_t)(k < p ? k : p - 1) * ua.ldq, row0, n, full);
            }
            __builtin_amdgcn_sched_barrier(0);
        };
        auto steps = [&](const V(&d)[KG], int s0) {
#pragma unroll
            for (int s = 0; s < KG; ++s) {
                if (s0 + s < ksteps) {
#pragma unroll
                    for (int t = 0; t < TX; ++t) {
                        const double cv = sc[(4 * (s0 + s) + g) * LC + 16 * t + ci];
                        acc[0][t] = __builtin_amdgcn_mfma_f64_16x16x4f64(cv, (double)d[s].x, acc[0][t], 0, 0, 0);
                        acc[1][t] = __builtin_amdgcn_mfma_f64_16x16x4f64(cv, (double)d[s].y, acc[1][t], 0, 0, 0);
                    }
                }
            }
        };
        load_q(q[0], 0);
#pragma unroll
        for (int t = 0; t < TX; ++t)
#pragma unroll
            for (int e = 0; e < 4; ++e) {
                acc[0][t][e] = (double)y[t][e].x;
                acc[1][t][e] = (double)y[t][e].y;
            }
        int s0 = 0;
        while (true) {
            const bool more = s0 + KG < ksteps;
            if (more) load_q(q[1], s0 + KG);
            steps(q[0], s0);
            s0 += KG;
            if (!more) break;
            const bool more2 = s0 + KG < ksteps;
            if (more2) load_q(q[0], s0 + KG);
            steps(q[1], s0);
            s0 += KG;
            if (!more2) break;
        }
#pragma unroll
        for (int t = 0; t < TX; ++t)
#pragma unroll
            for (int e = 0; e < 4; ++e) {
                const int c = 16 * t + g + 4 * e;
                V v;
                v.x = static_cast<T>(acc[0][t][e]);
                v.y = static_cast<T>(acc[1][t][e]);
                if (c < w) {
                    T* col = X + (int64_t)c * ua.ldx + row0;
                    if (full) {
                        __builtin_nontemporal_store(v, reinterpret_cast<V*>(col));
                    } else {
                        if (row0 < n) col[0] = v.x;
                        if (row0 + 1 < n) col[1] = v.y;
                    }
                }
                if constexpr (GRAM) {  // reduce what was stored (FP32 storage: rounded)
                    acc[0][t][e] = (double)v.x;
                    acc[1][t][e] = (double)v.y;
                }
            }
        if constexpr (GRAM) {
#pragma unroll
            for (int h = 0; h < 2; ++h) {
#pragma unroll
                for (int t = 0; t < TX; ++t)
#pragma unroll
                    for (int e = 0; e < 4; ++e) st[(16 * t + g + 4 * e) * SLD + ci] = acc[h][t][e];
                wave_sync();
                double xb[TX][4];
#pragma unroll
                for (int t = 0; t < TX; ++t) {
                    const double2* sp = reinterpret_cast<const double2*>(st + (16 * t + ci) * SLD + 4 * g);
                    const double2 v0 = sp[0], v1 = sp[1];
                    xb[t][0] = v0.x;
                    xb[t][1] = v0.y;
                    xb[t][2] = v1.x;
                    xb[t][3] = v1.y;
                }
#pragma unroll
                for (int u = 0; u < 4; ++u)
#pragma unroll
                    for (int i = 0; i < TX; ++i)
#pragma unroll
                        for (int j = i; j < TX; ++j)
                            gacc[i][j] = __builtin_amdgcn_mfma_f64_16x16x4f64(xb[i][u], xb[j][u], gacc[i][j], 0, 0, 0);
                wave_sync();
            }
        }
    }

    if constexpr (GRAM) {
        // D[r][c] of a tile sits in lane c + 16 (r % 4), element r / 4; the waves' tiles are
        // summed through LDS in wave order and written once per workgroup
        __syncthreads();
        double* red = upd_lds + 4 * ksteps * LC;
        double* out = ua.partials + (int64_t)wg * ua.stride;
#pragma unroll
        for (int i = 0; i < TX; ++i)
#pragma unroll
            for (int j = i; j < TX; ++j) {
#pragma unroll
                for (int r = 0; r < 4; ++r) red[(wave * 4 + r) * 64 + lane] = gacc[i][j][r];
                __syncthreads();
                if (wave == 0) {
#pragma unroll
                    for (int r = 0; r < 4; ++r) {
                        double v = 0.0;
                        for (int w2 = 0; w2 < NW; ++w2) v += red[(w2 * 4 + r) * 64 + lane];
                        const int ca = 16 * i + g + 4 * r, cb = 16 * j + ci;
                        if (ca < w && cb < w) out[ca + (int64_t)cb * w] = v;
                    }
                }
                __syncthreads();
            }
    }
}

template <typename T, int TX, bool GRAM>
__global__ void __launch_bounds__(GT) wide_update_kernel(const UpdateArgs ua) {
    update_body<T, TX, GRAM>(ua, blockIdx.x, gridDim.x);
}

// Many systems at once (blockIdx.y); workgroups past a system's rows write no partial sums
// (the batched reduction reads the first ceil(n / kUpdateUnitRows) of them).
template <typename T, int TX, bool GRAM>
__global__ void __launch_bounds__(GT) wide_update_kernel_batched(const UpdateArgs t, const BatchReloc br) {
    const int sys = batch_system(br);
    const BatchSys& d = br.sys[sys];
    if ((int64_t)blockIdx.x * kUpdateUnitRows >= d.n) return;
    UpdateArgs ua = t;
    ua.n = d.n;
    ua.Y = batch_ptr(br, sys, d, t.Y);
    ua.ldy = batch_ld(br, d, t.ldy);
    ua.Q = batch_ptr(br, sys, d, t.Q);
    ua.ldq = batch_ld(br, d, t.ldq);
    ua.C = batch_ptr(br, sys, d, t.C);
    ua.X = batch_ptr(br, sys, d, t.X);
    ua.ldx = batch_ld(br, d, t.ldx);
    ua.partials = batch_ptr(br, sys, d, t.partials);
    update_body<T, TX, GRAM>(ua, blockIdx.x, gridDim.x);
}

size_t update_lds(int w, int p, bool gram) {
    const size_t lc = 16 * (size_t)((w + 15) / 16);
    return sizeof(double) * (4 * (size_t)((p + 3) / 4) * lc + (gram ? NW * lc * SLD : 0));
}

template <typename T, int TX, bool GRAM>
hipError_t update_launch(const UpdateArgs& ua, int* grid, hipStream_t st, const BatchReloc* br) {
    static_assert(NW * 16 * TX * SLD >= 4 * 64 * NW, "the staging area also holds the cross-wave sums");
    const size_t lds = update_lds(ua.w, ua.p, GRAM);
    if (br) {
        hipLaunchKernelGGL((wide_update_kernel_batched<T, TX, GRAM>), dim3(*grid, br->nact), dim3(GT), lds, st, ua, *br);
        return hipGetLastError();
    }
    // one system: the resident workgroups, each walking its 32-row groups
    const int64_t units = (ua.n + kUpdateUnitRows - 1) / kUpdateUnitRows;
    int64_t cap = resident_grid(reinterpret_cast<const void*>(&wide_update_kernel<T, TX, GRAM>), GT, lds);
    if (cap < 1) cap = 512;
    if (GRAM) cap = std::min<int64_t>(cap, skinny_gemm_grid_cap());  // what the partial-sum buffers hold
    *grid = (int)std::max<int64_t>(1, std::min<int64_t>(units, cap));
    hipLaunchKernelGGL((wide_update_kernel<T, TX, GRAM>), dim3(*grid), dim3(GT), lds, st, ua);
    return hipGetLastError();
}

template <typename T, int TX>
hipError_t update_gram(const UpdateArgs& ua, bool gram, int* grid, hipStream_t st, const BatchReloc* br) {
    return gram ? update_launch<T, TX, true>(ua, grid, st, br) : update_launch<T, TX, false>(ua, grid, st, br);
}

template <typename T>
hipError_t update_dispatch(const UpdateArgs& ua, bool gram, int* grid, hipStream_t st, const BatchReloc* br) {
    switch ((ua.w + 15) / 16) {
        case 1: return update_gram<T, 1>(ua, gram, grid, st, br);
        case 2: return update_gram<T, 2>(ua, gram, grid, st, br);
        case 3: return update_gram<T, 3>(ua, gram, grid, st, br);
        default: return update_gram<T, 4>(ua, gram, grid, st, br);
    }
}

}  // namespace

bool wide_update_fits(int W, int p, bool gram) { return p >= 1 && update_lds(W, p, gram) <= 64 * 1024; }

hipError_t launch_wide_update(int64_t n, int W, bool f32, const void* Y, int64_t ldy, const void* Q, int64_t ldq,
                              int p, const double* C, void* X, int64_t ldx, double* partials, int* grid,
                              hipStream_t st, const BatchReloc* br) {
    const bool gram = partials != nullptr;
    if (W < 1 || W > 64 || n < 1 || !grid || !wide_update_fits(W, p, gram)) return hipErrorInvalidValue;
    if (br && (br->nact < 1 || *grid < 1)) return hipErrorInvalidValue;
    const UpdateArgs ua{n, W, Y, ldy, Q, ldq, p, C, X, ldx, partials, (int64_t)W * W};
    return f32 ? update_dispatch<float>(ua, gram, grid, st, br) : update_dispatch<double>(ua, gram, grid, st, br);
}

}  // namespace sko
