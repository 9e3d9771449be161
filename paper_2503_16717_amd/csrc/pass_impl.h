// Row-strip streaming pass kernel template for tall-skinny blocks on gfx950.
//
// A workgroup (4 waves of 64) walks strips of consecutive rows (grid-stride over strips).
// Phase A gives each thread RPT consecutive rows (two for float storage, read and written
// as one 8-byte access per column, so a wave moves 512 bytes per load as it does for
// double storage; not for wide float blocks with triangular solves, which would not fit the
// registers): the rows are loaded with coalesced accesses, updated, triangular-solved
// and written back; the result is staged in LDS column-major (padded leading dimension,
// so column reads across lanes do not collide in the LDS banks).  Phase B computes the pass's
// one reduction from the staged strip:
//
//  * projection Q^T x and the dense sketch Theta^T x: FP64 MFMA tiles of 16 output rows
//    (v_mfma_f64_16x16x4, for up to 12 columns v_mfma_f64_4x4x4).  The waves split the strip's
//    16-row groups; per group every lane supplies 4 consecutive rows of one output row's operand
//    (Q or Theta, read as one 32-byte piece per lane, so 16 lanes use each 128-byte line whole)
//    and the matching 4 rows of x from LDS, and issues 4 MFMAs per tile.  A 16 x 16 accumulator
//    is 4 doubles per lane, so one launch covers up to 16 * MT output rows; the waves' tiles are
//    summed through LDS once at the end.
//  * sparse-sign sketch: no MFMA; every lane owns one or two sketch rows and adds the staged rows
//    that the masks built from the rows' hashes select for it.
//  * Gram x^T x: blocks of up to 8 columns, and wider FP32 ones without an update, on FP64 FMAs
//    (lanes own strip rows, waves own output rows, register accumulators); the others and the
//    two-block passes on MFMA tiles with both operands from LDS.
//
// Every tall operand is read from HBM once per pass; partial sums stay in registers for the
// whole sweep and are written once per workgroup at the end.
#pragma once
#include <type_traits>
#include "batch.h"
#include "sko_internal.h"
#include "uniform.h"

namespace sko {
namespace passk {

typedef double double4_t __attribute__((ext_vector_type(4)));

// Block width from which the Gram matrix runs on MFMA tiles: below, the vector form's W / 4
// accumulator rows per wave are few; at 11 columns they take 66 VGPRs and 14 LDS reads per 64
// rows and wave.  us, vector | MFMA: after one solve, FP64, 2^22 rows: 7 columns 55 | 47, 8 61 | 54, 9 69 | 61,
// 11 82 | 69, 16 151 | 100; 300 007 rows: 8 18.7 | 9.7, 11 27.9 | 11.5.  Behind two solves and the update of a
// block, FP32, 2^22 rows: 8 columns 180 | 170, 9 222 | 241, 10 242 | 249, 11 327 | 301, 12 251 | 205, 16 399 | 268;
// 300 007 rows: 8 27 | 19, 9 38 | 27, 11 49 | 31.  (7 and 8 columns would gain too; at 9 and 10 the small row
// counts decide.)
constexpr int kGramMfmaW = 9;

// Per-(width, reduction) launch configuration.
template <int W, int RED>
struct Cfg {
    static constexpr bool SK = RED == RED_SKETCH_SPARSE || RED == RED_SKETCH_DENSE;
    // reductions on MFMA tiles: the projection and both sketches
    static constexpr bool MF = RED == RED_PROJ || SK;
    static constexpr int NT = 256;
    static constexpr int NWAVE = NT / 64;
    // Gram: output rows per wave (accumulators per lane = MAXA * W), spread over all waves
    static constexpr int MAXA = (W + NWAVE - 1) / NWAVE;
    // MFMA tiles of 16 output rows held by every wave (a dense sketch up to 64 rows in one
    // launch; projections up to 128 previous columns); a sparse sketch covers 16 MT rows too,
    // on row masks (MT = 4: one sketch row per lane, 8: two).  Fewer tiles are instantiated
    // for launches that need fewer (more resident waves).
    static constexpr int MT = RED == RED_SKETCH_DENSE ? 4 : 8;
    static constexpr int ROWS = MF ? 16 * MT : NWAVE * MAXA;
};

// The tall operands stream through a pass once: loads and stores are non-temporal (the two-row
// forms' 8-byte accesses are ordinary ones).
template <typename T>
__device__ __forceinline__ double ldv(const T* p) {
    return static_cast<double>(__builtin_nontemporal_load(p));
}
template <typename T>
__device__ __forceinline__ void stv(T* p, double v) {
    __builtin_nontemporal_store(static_cast<T>(v), p);
}

// SplitMix64 output number c+1 of the stream started at `seed` (Steele, Lea, Flood 2014).
__device__ __forceinline__ uint64_t splitmix64(uint64_t seed, uint64_t c) {
    uint64_t z = seed + (c + 1ull) * 0x9E3779B97F4A7C15ull;
    z = (z ^ (z >> 30)) * 0xBF58476D1CE4E5B9ull;
    z = (z ^ (z >> 27)) * 0x94D049BB133111EBull;
    return z ^ (z >> 31);
}

__device__ __forceinline__ double wave_sum(double v) {
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) v += __shfl_xor(v, o, 64);
    return v;
}

// Four consecutive staged rows of one column (16-byte aligned).
template <typename D>
__device__ __forceinline__ void lds4(const double* p, D* v) {
    const double2 a = reinterpret_cast<const double2*>(p)[0], b = reinterpret_cast<const double2*>(p)[1];
    v[0] = (D)a.x;
    v[1] = (D)a.y;
    v[2] = (D)b.x;
    v[3] = (D)b.y;
}
template <typename D>
__device__ __forceinline__ void lds4(const float* p, D* v) {
    const float4 a = *reinterpret_cast<const float4*>(p);
    v[0] = (D)a.x;
    v[1] = (D)a.y;
    v[2] = (D)a.z;
    v[3] = (D)a.w;
}

// Loads rows row0..row0+3 of one operand column (Q or a dense Theta) into av; rows at or
// beyond n read as zero.  `full`: all four rows lie below n.
template <typename TA>
__device__ __forceinline__ void load_col4(const TA* q, bool full, int64_t row0, int64_t n, double (&av)[4]) {
    if (full) {
        load4(q, av);
    } else {
#pragma unroll
        for (int u = 0; u < 4; ++u) av[u] = (row0 + u < n) ? ldv(q + u) : 0.0;
    }
}

// Rows row0..row0+R-1 of one column (zero at or beyond n).
template <int R, typename T>
__device__ __forceinline__ void load_rows(const T* col, int64_t row0, int64_t n, double v[R]) {
    if constexpr (R == 2) {
        if (row0 + 1 < n) {
            const RawRows<2, T> p = load_raw<2>(col + row0);
            v[0] = p.v[0];
            v[1] = p.v[1];
            return;
        }
    }
#pragma unroll
    for (int r = 0; r < R; ++r) v[r] = (row0 + r < n) ? ldv(col + row0 + r) : 0.0;
}

template <int R, typename T>
__device__ __forceinline__ void store_rows(T* col, int64_t row0, int64_t n, const double v[R]) {
    if constexpr (R == 2) {
        if (row0 + 1 < n) {
            typedef typename Unaligned<T>::v2 V;
            *reinterpret_cast<V*>(col + row0) = V{static_cast<T>(v[0]), static_cast<T>(v[1])};
            return;
        }
    }
#pragma unroll
    for (int r = 0; r < R; ++r)
        if (row0 + r < n) stv(col + row0 + r, v[r]);
}

// Transposes 64 x 64 bits held one row per lane (lo, hi: bits 0..31 and 32..63): afterwards bit r
// of lane l is what bit l of lane r was.  Six exchanges between lanes whose numbers differ in one
// bit, 32 first; all 64 lanes take part.
struct BitTranspose {
    unsigned p16, p8, m4, r4, m2, r2, m1, r1;  // this lane's byte selectors, kept bits and rotations
    __device__ __forceinline__ void init(int lane) {
        p16 = (lane & 16) ? 0x07060302u : 0x05040100u;
        p8 = (lane & 8) ? 0x03070105u : 0x06020400u;
        m4 = (lane & 4) ? 0xf0f0f0f0u : 0x0f0f0f0fu;
        r4 = (lane & 4) ? 4u : 28u;
        m2 = (lane & 2) ? 0xccccccccu : 0x33333333u;
        r2 = (lane & 2) ? 2u : 30u;
        m1 = (lane & 1) ? 0xaaaaaaaau : 0x55555555u;
        r1 = (lane & 1) ? 1u : 31u;
    }
    template <int CTRL>
    __device__ __forceinline__ static unsigned from(unsigned x) {
        return (unsigned)__builtin_amdgcn_mov_dpp((int)x, CTRL, 0xf, 0xf, true);
    }
    __device__ __forceinline__ static unsigned merge(unsigned m, unsigned x, unsigned p, unsigned r) {
        return (x & m) | (__builtin_amdgcn_alignbit(p, p, r) & ~m);
    }
    __device__ __forceinline__ unsigned low(unsigned x) const {
        const auto w = __builtin_amdgcn_permlane16_swap(x, x, false, false);
        x = __builtin_amdgcn_perm(w[1], w[0], p16);
        x = __builtin_amdgcn_perm(from<0x128>(x), x, p8);             // row_ror:8
        x = merge(m4, x, from<0x1b>(from<0x141>(x)), r4);             // row_half_mirror, quad_perm 3210
        x = merge(m2, x, from<0x4e>(x), r2);                          // quad_perm 2301
        return merge(m1, x, from<0xb1>(x), r1);                       // quad_perm 1032
    }
    __device__ __forceinline__ void run(unsigned& lo, unsigned& hi) const {
        const auto w = __builtin_amdgcn_permlane32_swap(lo, hi, false, false);
        lo = low(w[0]);
        hi = low(w[1]);
    }
};

// Element types of a pass: TY the input block Y, TQ the basis operand (Qu of the update,
// Qp of the projection), TX the written block X.  Plain passes use one storage type for
// all three; the mixed-precision GMRES panel reads an FP64 panel against the FP32 basis.
template <typename TY_, typename TQ_, typename TX_>
struct Tys {
    using TY = TY_;
    using TQ = TQ_;
    using TX = TX_;
};

// One pass over the rows of `a` by workgroup wg of nwg.
// W columns per block; WR columns staged and reduced.
template <int W, typename TS, int RED, bool UPD, int NTRSM, bool WRITE, int MTX, int PAIR = PAIR_NONE>
__device__ __forceinline__ void pass_body(const PassArgs& a, const int wg, const int nwg) {
    using TY = typename TS::TY;
    using TQ = typename TS::TQ;
    using TX = typename TS::TX;
    using C = Cfg<W, RED>;
    constexpr int NT = C::NT;
    constexpr bool F32 = sizeof(TY) == 4 && sizeof(TQ) == 4 && sizeof(TX) == 4;
    // rows per thread in phase A: two for float storage (8-byte accesses), except for wide
    // blocks with triangular solves or updates, whose two rows would not fit the registers
    constexpr bool TWO = PAIR == PAIR_PROJ || PAIR == PAIR_UPD || PAIR == PAIR_LEAD || PAIR == PAIR_CROSS;
    constexpr int WR = (PAIR == PAIR_PROJ || PAIR == PAIR_UPD) ? 2 * W : W;
    // the Gram of a pair runs on MFMA tiles as a projection does, with its W rows read from LDS
    // (PAIR_CROSS stages x as well, behind the reduced columns y)
    // and so does the Gram of a block of 9 or more columns, except in FP32 without an update
    // (11 columns after one solve, 2^24 rows: 0.245 ms vector, 0.257 ms MFMA)
    constexpr bool GMF = PAIR == PAIR_UPD || PAIR == PAIR_CROSS ||
                         (RED == RED_GRAM && W >= kGramMfmaW && (!F32 || UPD || PAIR == SOLO_UPD));
    constexpr int WS = PAIR == PAIR_CROSS ? 2 * W : WR;
    constexpr int GA0 = PAIR == PAIR_CROSS ? W : 0;  // staged column of the Gram's first row
    // (one in the two-block and solve-first passes of float blocks up to 8 columns too: fewer bytes in
    // flight per thread than with two rows, but two columns of traffic less; orth_blocks of 12 x 4, 12 x 6
    // and 8 x 8 FP32 columns, 2^24 rows: 17.2, 27.4, 18.8 ms; block by block with two rows 21.7, 34.3, 24.2)
    constexpr int RPT = PAIR != PAIR_NONE ? 1 : (F32 && (W <= 8 || (NTRSM == 0 && !UPD))) ? 2 : 1;
    constexpr int STRIP = NT * RPT;
    constexpr int RPL = STRIP / 64;
    constexpr int MAXA = C::MAXA;
    constexpr int MT = GMF ? 1 : MTX > 0 ? MTX : C::MT;  // MFMA tiles held (fewer: more waves per SIMD)
    constexpr bool MF = C::MF || GMF;
    constexpr bool WAVE_LOCAL = C::SK;  // sketch tiles reduce each wave's own rows
    constexpr bool HAS_RED = RED != RED_NONE;
    constexpr bool GRAM = RED == RED_GRAM && !GMF;
    // the strip in LDS, in the storage type: float storage reduces the rounded values it
    // stores (and halves the LDS)
    using XS = typename std::conditional<sizeof(typename std::conditional<WRITE, TX, TY>::type) == 4, float,
                                         double>::type;
    // padded LDS leading dimension of the strip: columns 16 bytes apart modulo the banks, so the
    // MFMA operands read four rows of 16 columns as 16-byte vectors without bank conflicts
    constexpr int LDX = STRIP + 16 / (int)sizeof(XS);
    __shared__ __align__(16) XS xs[HAS_RED ? WS * LDX : 1];
    __shared__ uint64_t hs[RED == RED_SKETCH_SPARSE ? STRIP : 1];
    // two-block projections of 16 to 24 columns: one 16 x 16 x 4 tile column for the first 16, 4 x
    // 4 x 4 blocks for the others (a B operand register per row and 16 columns instead of four).
    // us on up to 64 columns, FP32, 2^22 rows, blocks | tile and blocks: two blocks of 8 197 | 146, 9 202 | 197,
    // 10 215 | 192, 12 290 | 236; FP64 the same within 1 % at every width
    constexpr bool HYB = PAIR == PAIR_PROJ && WR >= 16;
    constexpr int C16 = HYB ? 16 : 0;           // columns on 16 x 16 x 4
    constexpr int CB = (WR - C16 + 3) / 4;      // 4-column blocks
    constexpr int PC = CB > 4 ? CB : 4;
    __shared__ double pred[MF ? PC * 64 * C::NWAVE : 1];  // cross-wave tile sums

    const int tid = threadIdx.x;
    const int lane = tid & 63;
    const int wave = tid >> 6;
    const int64_t n = a.n;

    // triangular factors (W x W, column-major) and update coefficients (pu x W)
    const CD gR0[2] = {as_uniform(a.R1), as_uniform(a.R2)};
    const CD gC0 = as_uniform(a.Cu);
    const int ldcu = a.ldcu ? a.ldcu : a.pu;
    // their diagonals' reciprocals: in registers, or for wide blocks in LDS, read again per
    // strip (two solves of 11 columns would hold 44 registers of them for the whole sweep:
    // 144 against 101 VGPRs, 3 against 4 waves, for the FP32 solve + projection on 64 columns,
    // 0.88 against 0.79 ms at 2^24 rows; one solve + Gram of 13 FP32 columns 207 against 178 us at 2^23
    // rows).  One solve behind an update of 10 or more columns keeps them in registers: there the LDS
    // form's higher occupancy does not pay (solve into the FP32 basis behind 55 columns, 192^3 rows: 10
    // columns 322 us in LDS, 311 in registers; 11: 357, 345; 12: 365, 346; 16: 467, 447; but 9: 299, 306).
    constexpr bool RINV_LDS = NTRSM > 0 && W >= 9 && !(UPD && W >= 10);
    __shared__ double srinv[RINV_LDS ? NTRSM * W : 1];
    double rinv[NTRSM > 0 && !RINV_LDS ? NTRSM * W : 1];
    if constexpr (RINV_LDS) {
        for (int i = tid; i < NTRSM * W; i += NT) {
            const int t = i / W, c = i - t * W;
            srinv[i] = 1.0 / (t == 0 ? a.R1 : a.R2)[c * W + c];
        }
        __syncthreads();
    } else if constexpr (NTRSM > 0) {
#pragma unroll
        for (int t = 0; t < NTRSM; ++t)
#pragma unroll
            for (int c = 0; c < W; ++c) rinv[t * W + c] = uniform_d(1.0 / gR0[t][c * W + c]);
    }

    // Gram: this wave accumulates output rows [a_lo, a_lo + MAXA)
    const int a_lo = wave * MAXA;
    double acc[GRAM ? MAXA : 1][WR];
#pragma unroll
    for (int i = 0; i < (GRAM ? MAXA : 1); ++i)
#pragma unroll
        for (int c = 0; c < WR; ++c) acc[i][c] = 0.0;
    // MFMA accumulators: tile m covers output rows 16m..16m+15 of this launch
    // The projection and dense sketch of blocks up to 12 columns run on v_mfma_f64_4x4x4 (four independent 4 x 4 x 4 blocks per instruction, the same FP64
    // rate as 16 x 16 x 4): a block covers 4 output rows x 4 columns of x, so narrow blocks
    // do not pay for 16 padded columns (three instructions of a quarter of the time instead
    // of one 16 x 16 x 4 for 11 columns).  Instruction (m, cb) holds the output rows
    // 16m..16m+15 (block b: rows 16m + 4b..+3) and the columns 4cb..4cb+3.  The A operand
    // uses the lane mapping of the 16 x 16 x 4 tile (lane l: output row 16m + l % 16, data
    // row l / 16), so the same pieces feed both forms.
    // sparse-sign sketches on row masks (no MFMA): lane l accumulates the launch's sketch rows
    // l and, for launches of up to 128 rows, l + 64
    constexpr bool SPM = RED == RED_SKETCH_SPARSE;
    constexpr int SPR = MT / 4;
    constexpr bool B4 = MF && !SPM && (W <= 12 || TWO);
    double4_t dacc[(MF && !SPM && (!B4 || HYB)) ? MT : 1];
    double acc4[B4 && CB > 0 ? MT * CB : 1];
#pragma unroll
    for (int i = 0; i < (B4 && CB > 0 ? MT * CB : 1); ++i) acc4[i] = 0.0;
    const int ntiles = (a.red_rows + 15) / 16;
#pragma unroll
    for (int m = 0; m < (MF ? MT : 1); ++m) dacc[m] = double4_t{0.0, 0.0, 0.0, 0.0};

    // Sparse sketch on row masks (SPM): lane l accumulates sketch row g = red_row0 + l (and
    // g + 64), which is slot j of hash byte t; byte b selects slot floor((b >> 1) B / 128) of its
    // B = k / zeta and carries the sign in bit 0.  Per 64 staged rows each lane sets the bits of its
    // own row's sketch rows in a word, and the wave transposes the 64 x 64 bits: lane l then has the
    // mask of the rows that sketch row l takes.  (The rows' signs in a byte are one ballot, which the
    // lanes of the byte's sketch rows keep.)  It adds those rows into its W sums in ascending row
    // order.  Only the rows with a nonzero in the lane's sketch row are touched: zeta W products per
    // row instead of k W on MFMA blocks.
    // The masks take a third of the instructions where few rows fall to a lane, and uniform values
    // held for them across the sweep overflow the scalar registers (spills to lanes of vector
    // registers).  us with masks from ballots of every slot bit | masks and signs transposed, up to 185
    // spills | now, none in the plain sketches: 11 FP64 columns, 128 rows, zeta = 8, 7 077 889 rows
    // 209 | 209 | 194; 6 FP32 columns, 64 rows, 2^22 rows 87.8 | 93.4 | 79.5; 8 FP32 columns 104 | 119 |
    // 96; 6 FP64 columns 68.4 | 67.1 | 65.2.  Where ballots of a single bit did (k = 2 zeta, zeta = 1) FP64
    // sketches take 1 to 5 % more than with them.
    double sacc[SPM ? SPR : 1][SPM ? W : 1];
#pragma unroll
    for (int q = 0; q < (SPM ? SPR : 1); ++q)
#pragma unroll
        for (int c = 0; c < (SPM ? W : 1); ++c) sacc[q][c] = 0.0;
    BitTranspose bt;
    if constexpr (SPM) bt.init(lane);

    const int64_t nstrips = (n + STRIP - 1) / STRIP;
    for (int64_t s = wg; s < nstrips; s += nwg) {
        const int64_t base = s * STRIP;
        // wide blocks load the factor and coefficient entries again per strip (w(w-1)/2 per
        // factor would not fit the SGPRs for the whole sweep); narrow blocks may hold them
        CD gR[2] = {gR0[0], gR0[1]};
        CD gC = gC0;
        if constexpr (W >= 10) {
            gR[0] = per_strip(gR[0]);
            gR[1] = per_strip(gR[1]);
            gC = per_strip(gC);
        }
        const int ri0 = RINV_LDS ? per_strip(0) : 0;
        auto rdiag = [&](int i) {
            if constexpr (RINV_LDS)
                return srinv[ri0 + i];
            else
                return rinv[i];
        };
        // ---------------- phase A: RPT consecutive rows per thread ----------------
        if constexpr (PAIR != PAIR_NONE) {
            // x solved (and rounded as a stored x would be), then the updates of both blocks
            const int64_t row = base + tid;
            constexpr int WZ = TWO ? 2 * W : W;
            double za[1][WZ];
            double(&z)[WZ] = za[0];
            if (row < n) {
                const TY* Y = static_cast<const TY*>(a.Y);
#pragma unroll
                for (int c = 0; c < W; ++c) z[c] = ldv(Y + row + c * a.ldy);
                if constexpr (TWO) {
                    const TY* Y2 = static_cast<const TY*>(a.Y2);
#pragma unroll
                    for (int c = 0; c < W; ++c) z[W + c] = ldv(Y2 + row + c * a.ldy2);
                }
#pragma unroll
                for (int t = 0; t < NTRSM; ++t) {
                    const CD R = gR[t];
#pragma unroll
                    for (int c = 0; c < W; ++c) {
                        double v = z[c];
#pragma unroll
                        for (int q = 0; q < c; ++q) v -= z[q] * R[q + c * W];
                        z[c] = v * rdiag(t * W + c);
                    }
                }
                if constexpr (sizeof(TX) == 4) {
#pragma unroll
                    for (int c = 0; c < W; ++c) z[c] = static_cast<double>(static_cast<TX>(z[c]));
                }
                TX* X = static_cast<TX*>(a.X);
                TX* X2 = static_cast<TX*>(a.X2);
                const TQ* Qr = static_cast<const TQ*>(a.Qu) + row;
                if constexpr (PAIR == PAIR_UPD) {
                    update_rows<WZ, 1, TQ>(za, Qr, a.ldqu, a.pu, gC, ldcu);
                } else if constexpr (PAIR == SOLO_UPD) {
                    double xa[1][W];
#pragma unroll
                    for (int c = 0; c < W; ++c) xa[0][c] = z[c];
                    update_rows<W, 1, TQ>(xa, Qr, a.ldqu, a.pu, gC, ldcu);
#pragma unroll
                    for (int c = 0; c < W; ++c) z[c] = xa[0][c];
                } else if constexpr (PAIR == PAIR_LEAD) {
#pragma unroll
                    for (int c = 0; c < W; ++c) {
                        double v = z[W + c];
#pragma unroll
                        for (int q = 0; q < W; ++q) v -= z[q] * gC[q + c * ldcu];
                        z[W + c] = v;
                    }
                }
                if constexpr (WRITE) {
#pragma unroll
                    for (int c = 0; c < W; ++c) stv(X + row + c * a.ldx, z[c]);
                }
                if constexpr (PAIR == PAIR_LEAD) {
#pragma unroll
                    for (int c = 0; c < W; ++c) stv(X2 + row + c * a.ldx2, z[W + c]);
                } else if constexpr (PAIR == PAIR_UPD) {
                    if (X2) {
#pragma unroll
                        for (int c = 0; c < W; ++c) stv(X2 + row + c * a.ldx2, z[W + c]);
                    }
                }
                if constexpr (RED == RED_SKETCH_SPARSE) hs[tid] = splitmix64(a.sk_seed, (uint64_t)row);
            } else {
#pragma unroll
                for (int c = 0; c < WZ; ++c) z[c] = 0.0;
                if constexpr (RED == RED_SKETCH_SPARSE) hs[tid] = 0;
            }
            constexpr int Z0 = PAIR == PAIR_LEAD || PAIR == PAIR_CROSS ? W : 0;
#pragma unroll
            for (int c = 0; c < WS; ++c) xs[c * LDX + tid] = static_cast<XS>(z[(Z0 + c) % WZ]);
        }
        else if constexpr (RPT == 1)
        {
            const int64_t row = base + tid;
            double xa[1][W];
            double(&x)[W] = xa[0];
            if (row < n) {
                const TY* Y = static_cast<const TY*>(a.Y);
#pragma unroll
                for (int c = 0; c < W; ++c) x[c] = ldv(Y + row + c * a.ldy);
                if constexpr (UPD) update_rows<W, 1, TQ>(xa, static_cast<const TQ*>(a.Qu) + row, a.ldqu, a.pu, gC, ldcu);
#pragma unroll
                for (int t = 0; t < NTRSM; ++t) {
                    const CD R = gR[t];
#pragma unroll
                    for (int c = 0; c < W; ++c) {
                        double v = x[c];
#pragma unroll
                        for (int q = 0; q < c; ++q) v -= x[q] * R[q + c * W];
                        x[c] = v * rdiag(t * W + c);
                    }
                }
                if constexpr (WRITE) {
                    TX* X = static_cast<TX*>(a.X);
#pragma unroll
                    for (int c = 0; c < W; ++c) stv(X + row + c * a.ldx, x[c]);
                }
                if constexpr (RED == RED_SKETCH_SPARSE) hs[tid] = splitmix64(a.sk_seed, (uint64_t)row);
            } else {
#pragma unroll
                for (int c = 0; c < W; ++c) x[c] = 0.0;
                if constexpr (RED == RED_SKETCH_SPARSE) hs[tid] = 0;
            }
            if constexpr (HAS_RED) {
#pragma unroll
                for (int c = 0; c < W; ++c) xs[c * LDX + tid] = static_cast<XS>(x[c]);
            }
        }
        else
        {
            const int64_t row0 = base + (int64_t)RPT * tid;
            double x[RPT][W];
            if (row0 < n) {
                const TY* Y = static_cast<const TY*>(a.Y);
#pragma unroll
                for (int c = 0; c < W; ++c) {
                    double v[RPT];
                    load_rows<RPT>(Y + (int64_t)c * a.ldy, row0, n, v);
#pragma unroll
                    for (int r = 0; r < RPT; ++r) x[r][c] = v[r];
                }
                if constexpr (UPD) {
                    // the last row alone (an odd n) updates its single row
                    if (row0 + RPT - 1 < n) {
                        update_rows<W, RPT, TQ>(x, static_cast<const TQ*>(a.Qu) + row0, a.ldqu, a.pu, gC, ldcu);
                    } else {
                        const TQ* Q = static_cast<const TQ*>(a.Qu) + row0;
                        for (int j = 0; j < a.pu; ++j) {
                            const double q = ldv(Q + (int64_t)j * a.ldqu);
#pragma unroll
                            for (int c = 0; c < W; ++c) x[0][c] -= q * gC[j + c * ldcu];
                        }
                    }
                }
#pragma unroll
                for (int t = 0; t < NTRSM; ++t) {
                    const CD R = gR[t];
#pragma unroll
                    for (int c = 0; c < W; ++c) {
#pragma unroll
                        for (int r = 0; r < RPT; ++r) {
                            double v = x[r][c];
#pragma unroll
                            for (int q = 0; q < c; ++q) v -= x[r][q] * R[q + c * W];
                            x[r][c] = v * rdiag(t * W + c);
                        }
                    }
                }
                if constexpr (WRITE) {
                    TX* X = static_cast<TX*>(a.X);
#pragma unroll
                    for (int c = 0; c < W; ++c) {
                        double v[RPT];
#pragma unroll
                        for (int r = 0; r < RPT; ++r) v[r] = x[r][c];
                        store_rows<RPT>(X + (int64_t)c * a.ldx, row0, n, v);
                    }
                }
                // rows past n (a partial last pair) contribute zero to the reduction
#pragma unroll
                for (int r = 1; r < RPT; ++r)
                    if (row0 + r >= n)
#pragma unroll
                        for (int c = 0; c < W; ++c) x[r][c] = 0.0;
                if constexpr (RED == RED_SKETCH_SPARSE) {
#pragma unroll
                    for (int r = 0; r < RPT; ++r)
                        hs[RPT * tid + r] = (row0 + r < n) ? splitmix64(a.sk_seed, (uint64_t)(row0 + r)) : 0;
                }
            } else {
#pragma unroll
                for (int r = 0; r < RPT; ++r)
#pragma unroll
                    for (int c = 0; c < W; ++c) x[r][c] = 0.0;
                if constexpr (RED == RED_SKETCH_SPARSE) {
#pragma unroll
                    for (int r = 0; r < RPT; ++r) hs[RPT * tid + r] = 0;
                }
            }
            if constexpr (HAS_RED) {
#pragma unroll
                for (int c = 0; c < W; ++c)
#pragma unroll
                    for (int r = 0; r < RPT; ++r) xs[c * LDX + RPT * tid + r] = static_cast<XS>(x[r][c]);
            }
        }
        if constexpr (HAS_RED) {
            // Sketches: each wave reduces the rows it staged itself, so only the wave's own LDS
            // writes must be visible (no workgroup barrier: the waves drift apart and one
            // wave's MFMA tiles overlap another's loads).  Projections and the Gram share the
            // whole strip across the waves (the projection's Q reads then cover each column's
            // strip segment at once, which the HBM pages favour).
            if constexpr (WAVE_LOCAL) {
                __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
                __builtin_amdgcn_wave_barrier();
                __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
            } else {
                __syncthreads();
            }
            if constexpr (SPM) {
                // ---------------- phase B, sparse-sign sketch on row masks ----------------
                constexpr int WROWS = STRIP / C::NWAVE;  // rows this wave staged (64 per thread row)
                const int B0 = a.sk_k / a.sk_zeta;
                // masks of the wave's RPT groups of 64 rows, formed side by side (their chains of
                // lane exchanges overlap)
                unsigned ml[RPT][SPR], mh[RPT][SPR], sl[RPT][SPR], sh[RPT][SPR];
                uint64_t h[RPT];
#pragma unroll
                for (int u = 0; u < RPT; ++u) h[u] = hs[wave * WROWS + u * 64 + lane];
                // uniform operands derived again here: held for the sweep, the bytes' offsets and
                // conditions overflow the scalar registers
                const int B = per_strip(B0), zeta = per_strip(a.sk_zeta);
#pragma unroll
                for (int q = 0; q < SPR; ++q) {
#pragma unroll
                    for (int u = 0; u < RPT; ++u) ml[u][q] = mh[u][q] = sl[u][q] = sh[u][q] = 0u;
                    int o = per_strip(-a.red_row0) - 64 * q;  // the byte's first sketch row among the lanes'
#pragma unroll
                    for (int t = 0; t < 8; ++t) {
                        if (t < zeta && o < 64 && o + B > 0) {
                            const bool at = lane >= o;
                            unsigned bit[RPT];
                            int pos[RPT];
#pragma unroll
                            for (int u = 0; u < RPT; ++u) {
                                const unsigned b8 = (unsigned)(h[u] >> (8 * t)) & 0xffu;
                                pos[u] = ((int)__umul24(b8 >> 1, (unsigned)B) + o * 128) >> 7;  // B <= 128
                                bit[u] = 1u << (pos[u] & 31);
                                const uint64_t sg = __ballot(b8 & 1u);
                                sl[u][q] = at ? (unsigned)sg : sl[u][q];
                                sh[u][q] = at ? (unsigned)(sg >> 32) : sh[u][q];
                            }
                            if ((o & 31) + B <= 32) {  // all of the byte's rows in one half
#pragma unroll
                                for (int u = 0; u < RPT; ++u) {
                                    if (o & 32)
                                        mh[u][q] |= bit[u];
                                    else
                                        ml[u][q] |= bit[u];
                                }
                            } else {
#pragma unroll
                                for (int u = 0; u < RPT; ++u) {
                                    ml[u][q] |= (unsigned)pos[u] < 32u ? bit[u] : 0u;
                                    mh[u][q] |= (unsigned)(pos[u] - 32) < 32u ? bit[u] : 0u;
                                }
                            }
                        }
                        o += B;
                    }
#pragma unroll
                    for (int u = 0; u < RPT; ++u) bt.run(ml[u][q], mh[u][q]);
                }
#pragma unroll
                for (int u = 0; u < RPT; ++u) {
                    const int rb = wave * WROWS + u * 64;  // strip-local row of mask bit 0
                    const uint64_t vm = __ballot(base + rb + lane < n);
#pragma unroll
                    for (int q = 0; q < SPR; ++q) {
                        ml[u][q] &= (unsigned)vm;
                        mh[u][q] &= (unsigned)(vm >> 32);
                    }
                    // one sketch row per lane: each mask in two 32-row halves (the lowest set bit,
                    // its clearing and the sign are single 32-bit operations); two rows per lane:
                    // whole 64-row masks (four half loops would each run to their own longest
                    // half, and the sparser masks of larger sketches leave them short)
                    constexpr int NH = SPR == 1 ? 2 : 1;
#pragma unroll
                    for (int q = 0; q < SPR; ++q) {
#pragma unroll
                        for (int hf = 0; hf < NH; ++hf) {
                            using MW = typename std::conditional<NH == 2, unsigned, uint64_t>::type;
                            MW msk, sgm;
                            if constexpr (NH == 2) {
                                msk = hf ? mh[u][q] : ml[u][q];
                                sgm = hf ? sh[u][q] : sl[u][q];
                            } else {
                                msk = ((uint64_t)mh[u][q] << 32) | ml[u][q];
                                sgm = ((uint64_t)sh[u][q] << 32) | sl[u][q];
                            }
                            const int rh = rb + 32 * hf;
                            while (msk) {
                                const int bit = NH == 2 ? __builtin_ctz((unsigned)msk) : __builtin_ctzll((uint64_t)msk);
                                msk &= msk - 1u;
                                // +-1.0 from the row's sign bit for this byte
                                const unsigned sb = (unsigned)(sgm >> bit) & 1u;
                                const double sgn = __hiloint2double((int)((sb << 31) | 0x3FF00000u), 0);
#pragma unroll
                                for (int c = 0; c < W; ++c)
                                    sacc[q][c] = fma(sgn, (double)xs[c * LDX + rh + bit], sacc[q][c]);
                            }
                        }
                    }
                }
            } else if constexpr (MF) {
                // ---------------- phase B, MFMA tiles ----------------
                const int g = lane >> 4, ci = lane & 15;
                const TQ* Qp = static_cast<const TQ*>(a.Qp);
                const double* Th = a.theta;
                // rows per group: 16 (4 per lane), or 32 (8 per lane) for projections against an
                // FP32 basis on 4 x 4 x 4 blocks: a 4-byte piece load moves half the bytes of a
                // double one, so each lane loads two per column, as many bytes in flight as the
                // FP64 form (the staged operand stays in float until its MFMA)
                constexpr int UR = (RED == RED_PROJ && sizeof(TQ) == 4 && sizeof(XS) == 4 && B4) ? 8 : 4;
                constexpr int GR = 4 * UR;
                constexpr int GPW = STRIP / GR / C::NWAVE;  // row groups per wave
                static_assert(STRIP % (GR * C::NWAVE) == 0, "row groups must tile the strip");
                const int g0 = WAVE_LOCAL ? wave * GPW : wave, gstep = WAVE_LOCAL ? 1 : C::NWAVE;
                // not unrolled: the unrolled groups hold more loads and tiles at once and cost a
                // resident wave
#pragma unroll 1
                for (int gam = g0, it = 0; it < GPW; gam += gstep, ++it) {
                    const int r0 = gam * GR + UR * g;  // strip-local rows r0..r0+UR-1 for this lane
                    const bool full = base + r0 + 3 < n;
                    const bool gfull = base + (gam + 1) * GR <= n;  // the whole group lies below n
                    // B operands: 16 x 16 x 4 tiles take column ci of the 4 rows; 4 x 4 x 4 blocks
                    // take column 4cb + lane % 4
                    double bv[B4 && !HYB ? 1 : UR];
                    // (the two-block passes' 2W columns meet every tile: converted once)
                    using BT = typename std::conditional<TWO, double, XS>::type;
                    BT bq[B4 && CB > 0 ? CB : 1][UR];
                    if constexpr (HYB) {
#pragma unroll
                        for (int u = 0; u < UR; u += 4) lds4(xs + ci * LDX + r0 + u, bv + u);
                    }
                    if constexpr (B4) {
#pragma unroll
                        for (int cb = 0; cb < CB; ++cb) {
                            const int col = C16 + 4 * cb + (lane & 3);
#pragma unroll
                            for (int u = 0; u < UR; u += 4) {
                                if (col < WR) {
                                    lds4(xs + col * LDX + r0 + u, &bq[cb][u]);
                                } else {
                                    bq[cb][u] = bq[cb][u + 1] = bq[cb][u + 2] = bq[cb][u + 3] = BT(0);
                                }
                            }
                        }
                    } else {
                        bv[0] = bv[1] = bv[2] = bv[3] = 0.0;
                        if (ci < W) lds4(xs + ci * LDX + r0, bv);
                    }
#pragma unroll
                    for (int m = 0; m < MT; ++m) {
                        if (m < ntiles) {
                            const int col = 16 * m + ci;
                            if constexpr (UR == 8) {
                                // the 8 pieces stay in float until their MFMA; a lane past the last
                                // output row reads that row's column (its own row is never written)
                                typedef Unaligned<float>::v4 V4;
                                const float* qc = reinterpret_cast<const float*>(Qp) +
                                                  (int64_t)(col < a.red_rows ? col : a.red_rows - 1) * a.ldqp + base + r0;
                                V4 v0, v1;
                                if (gfull) {
                                    v0 = *reinterpret_cast<const V4*>(qc);
                                    v1 = *reinterpret_cast<const V4*>(qc + 4);
                                } else {
                                    const int64_t rr = base + r0;
#pragma unroll
                                    for (int u = 0; u < 4; ++u) {
                                        v0[u] = (rr + u < n) ? qc[u] : 0.0f;
                                        v1[u] = (rr + 4 + u < n) ? qc[4 + u] : 0.0f;
                                    }
                                }
#pragma unroll
                                for (int u = 0; u < 8; ++u) {
                                    const double au = (double)(u < 4 ? v0[u & 3] : v1[u & 3]);
                                    if constexpr (HYB)
                                        dacc[m] = __builtin_amdgcn_mfma_f64_16x16x4f64(au, bv[u], dacc[m], 0, 0, 0);
#pragma unroll
                                    for (int cb = 0; cb < CB; ++cb)
                                        acc4[m * CB + cb] = __builtin_amdgcn_mfma_f64_4x4x4f64(
                                            au, (double)bq[cb][u], acc4[m * CB + cb], 0, 0, 0);
                                }
                                continue;
                            }
                            double av[4] = {0.0, 0.0, 0.0, 0.0};
                            if (col < a.red_rows) {
                                if constexpr (GMF) {
                                    lds4(xs + (GA0 + ci) * LDX + r0, av);
                                } else if constexpr (RED == RED_PROJ)
                                    load_col4(Qp + (int64_t)col * a.ldqp + base + r0, full, base + r0, n, av);
                                else
                                    load_col4(Th + (int64_t)col * a.ldtheta + base + r0, full, base + r0, n, av);
                            }
                            if constexpr (B4) {
#pragma unroll
                                for (int u = 0; u < 4; ++u) {
                                    if constexpr (HYB)
                                        dacc[m] = __builtin_amdgcn_mfma_f64_16x16x4f64(av[u], bv[u], dacc[m], 0, 0, 0);
#pragma unroll
                                    for (int cb = 0; cb < CB; ++cb)
                                        acc4[m * CB + cb] = __builtin_amdgcn_mfma_f64_4x4x4f64(
                                            av[u], (double)bq[cb][u], acc4[m * CB + cb], 0, 0, 0);
                                }
                            } else {
#pragma unroll
                                for (int u = 0; u < 4; ++u)
                                    dacc[m] = __builtin_amdgcn_mfma_f64_16x16x4f64(av[u], bv[u], dacc[m], 0, 0, 0);
                            }
                        }
                    }
                }
            } else if constexpr (GRAM) {
                // ---------------- phase B, lanes over rows, waves over output rows ----------------
#pragma unroll 2
                for (int r = 0; r < RPL; ++r) {
                    const int rr = r * 64 + lane;
                    double x[WR];
#pragma unroll
                    for (int c = 0; c < WR; ++c) x[c] = xs[c * LDX + rr];
#pragma unroll
                    for (int i = 0; i < MAXA; ++i) {
                        const int al = a_lo + i;
                        if (al < a.red_rows) {
                            const double xa = xs[(a.red_row0 + al) * LDX + rr];
#pragma unroll
                            for (int c = 0; c < WR; ++c) acc[i][c] += xa * x[c];
                        }
                    }
                }
            }
            // the next strip's phase A overwrites the staged rows
            if constexpr (WAVE_LOCAL) {
                __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
                __builtin_amdgcn_wave_barrier();
            } else {
                __syncthreads();
            }
        }
    }

    if constexpr (SPM) {
        // lane l holds sketch rows red_row0 + l + 64 q; the waves' sums are added through LDS in
        // wave order, four columns at a time
        double* out = a.partials + (int64_t)wg * a.part_stride;
#pragma unroll
        for (int q = 0; q < SPR; ++q) {
            const int r = lane + 64 * q;
#pragma unroll
            for (int c0 = 0; c0 < W; c0 += 4) {
#pragma unroll
                for (int cc = 0; cc < 4; ++cc)
                    if (c0 + cc < W) pred[(wave * 4 + cc) * 64 + lane] = sacc[q][c0 + cc];
                __syncthreads();
                if (wave == 0 && r < a.red_rows) {
#pragma unroll
                    for (int cc = 0; cc < 4; ++cc) {
                        if (c0 + cc < W) {
                            double v = 0.0;
                            for (int w2 = 0; w2 < C::NWAVE; ++w2) v += pred[(w2 * 4 + cc) * 64 + lane];
                            out[(a.red_row0 + r) + (int64_t)(c0 + cc) * a.part_rows_total] = v;
                        }
                    }
                }
                __syncthreads();
            }
        }
    } else if constexpr (MF) {
        // Output layouts (measured on gfx950).  v_mfma_f64_4x4x4: D[i][j] of block b sits in lane
        // 4b + j + 16i, so lane l holds output row 16m + 4((l % 16) / 4) + l / 16 and column
        // 4cb + l % 4 of instruction (m, cb).  v_mfma_f64_16x16x4: D[i][j] of a tile sits in lane
        // j + 16 * (i % 4), element i / 4.  The waves' values are summed through LDS in wave order.
        double* out = a.partials + (int64_t)wg * a.part_stride;
        // K values per lane summed over the waves; put(k, value) on wave 0
        auto wave_sums = [&](auto kc, auto&& val, auto&& put) {
            constexpr int K = decltype(kc)::value;
#pragma unroll
            for (int k = 0; k < K; ++k) pred[(wave * PC + k) * 64 + lane] = val(k);
            __syncthreads();
            if (wave == 0) {
#pragma unroll
                for (int k = 0; k < K; ++k) {
                    double v = 0.0;
                    for (int w2 = 0; w2 < C::NWAVE; ++w2) v += pred[(w2 * PC + k) * 64 + lane];
                    put(k, v);
                }
            }
            __syncthreads();
        };
#pragma unroll
        for (int m = 0; m < MT; ++m) {
            if (m >= ntiles) break;
            if constexpr (B4 && CB > 0) {
                const int r = 16 * m + 4 * ((lane & 15) >> 2) + (lane >> 4);
                wave_sums(std::integral_constant<int, CB>{}, [&](int k) { return acc4[m * CB + k]; },
                          [&](int k, double v) {
                              const int c = C16 + 4 * k + (lane & 3);
                              if (r < a.red_rows && c < WR) out[(a.red_row0 + r) + (int64_t)c * a.part_rows_total] = v;
                          });
            }
            if constexpr (!B4 || HYB) {
                const int c = lane & 15;
                wave_sums(std::integral_constant<int, 4>{}, [&](int k) { return dacc[m][k]; },
                          [&](int k, double v) {
                              const int r = 16 * m + (lane >> 4) + 4 * k;
                              if (r < a.red_rows && c < WR) out[(a.red_row0 + r) + (int64_t)c * a.part_rows_total] = v;
                          });
            }
        }
    } else if constexpr (GRAM) {
        double* out = a.partials + (int64_t)wg * a.part_stride;
#pragma unroll
        for (int i = 0; i < MAXA; ++i) {
            const int al = a_lo + i;
#pragma unroll
            for (int c = 0; c < WR; ++c) {
                const double v = wave_sum(acc[i][c]);
                if (lane == 0 && al < a.red_rows)
                    out[(a.red_row0 + al) + (int64_t)c * a.part_rows_total] = v;
            }
        }
    }
}

template <int W, typename T, int RED, bool UPD, int NTRSM, bool WRITE, int MTX = 0>
__global__ void __launch_bounds__((Cfg<W, RED>::NT)) pass_kernel(const PassArgs a) {
    pass_body<W, Tys<T, T, T>, RED, UPD, NTRSM, WRITE, MTX>(a, blockIdx.x, gridDim.x);
}

// FP64 panel (Y) against the FP32 basis (Q), written as TX.
template <int W, typename TX, int RED, bool UPD, int NTRSM, bool WRITE, int MTX = 0>
__global__ void __launch_bounds__((Cfg<W, RED>::NT)) pass_kernel_panel(const PassArgs a) {
    pass_body<W, Tys<double, float, TX>, RED, UPD, NTRSM, WRITE, MTX>(a, blockIdx.x, gridDim.x);
}

// Batched form: the template arguments are moved to the system of blockIdx.y.
template <int W, typename T, int RED, bool UPD, int NTRSM, bool WRITE, int MTX = 0>
__global__ void __launch_bounds__((Cfg<W, RED>::NT)) pass_kernel_batched(const PassArgs t, const BatchReloc br) {
    const int sys = batch_system(br);
    const BatchSys& d = br.sys[sys];
    PassArgs a = t;
    a.n = d.n;
    a.Y = batch_ptr(br, sys, d, t.Y);
    a.ldy = batch_ld(br, d, t.ldy);
    a.Qu = batch_ptr(br, sys, d, t.Qu);
    a.ldqu = batch_ld(br, d, t.ldqu);
    a.Cu = batch_ptr(br, sys, d, t.Cu);
    a.R1 = batch_ptr(br, sys, d, t.R1);
    a.R2 = batch_ptr(br, sys, d, t.R2);
    a.X = batch_ptr(br, sys, d, t.X);
    a.ldx = batch_ld(br, d, t.ldx);
    a.Qp = batch_ptr(br, sys, d, t.Qp);
    a.ldqp = batch_ld(br, d, t.ldqp);
    a.partials = batch_ptr(br, sys, d, t.partials);
    a.sk_seed = d.seed;
    pass_body<W, Tys<T, T, T>, RED, UPD, NTRSM, WRITE, MTX>(a, blockIdx.x, gridDim.x);
}

// The two-block and solve-first passes (PairKind).  All stay HBM-bound: at n = 2^24, 6 FP64 columns,
// averaged over 36 previous ones, the projection of both blocks runs at 5.9 TB/s (1.02 ms), their
// update at 5.5 TB/s (1.31 ms), the leading pass at 5.2 TB/s (0.62 ms); one block at a time, with
// Q read for each, the same work took 0.99 + 1.23 ms (projections), 1.22 + 1.24 ms (updates) and
// 0.29 ms.  In FP32 at 11 columns the projection of both blocks is held to 3.5 TB/s by its 22
// columns' MFMAs and conversions.
template <int W, typename T, int RED, int PAIR, int MTX = 0>
__global__ void __launch_bounds__((Cfg<W, RED>::NT)) pass_kernel_pair(const PassArgs a) {
    constexpr int NTRSM = PAIR == PAIR_LEAD || PAIR == PAIR_CROSS ? 1 : 2;
    constexpr bool WRITE = PAIR != PAIR_PROJ && PAIR != SOLO_PROJ;
    pass_body<W, Tys<T, T, T>, RED, false, NTRSM, WRITE, MTX, PAIR>(a, blockIdx.x, gridDim.x);
}

using KernelPtr = void (*)(const PassArgs);
using BatchedKernelPtr = void (*)(const PassArgs, const BatchReloc);

// The pass variants the orchestration launches: (reduction, update, solves, write).
template <int W, typename T>
KernelPtr select_w(const PassKey& k) {
    const int r = k.red;
    const bool u = k.upd, wr = k.write;
    const int t = k.ntrsm;
    // projections: the fewest accumulator tiles that hold the launch's rows
    const int mt = (k.tiles >= 1 && k.tiles <= 4) ? 4 : (k.tiles >= 5 && k.tiles <= 6) ? 6 : 8;
    if (!u && t == 0 && !wr) {
        if (r == RED_PROJ)
            return mt == 4   ? &pass_kernel<W, T, RED_PROJ, false, 0, false, 4>
                   : mt == 6 ? &pass_kernel<W, T, RED_PROJ, false, 0, false, 6>
                             : &pass_kernel<W, T, RED_PROJ, false, 0, false>;
        if (r == RED_GRAM) return &pass_kernel<W, T, RED_GRAM, false, 0, false>;
        if (r == RED_SKETCH_SPARSE)
            return mt == 4 ? &pass_kernel<W, T, RED_SKETCH_SPARSE, false, 0, false, 4>
                           : &pass_kernel<W, T, RED_SKETCH_SPARSE, false, 0, false>;
        if (r == RED_SKETCH_DENSE) return &pass_kernel<W, T, RED_SKETCH_DENSE, false, 0, false>;
    }
    if (u && t == 0 && wr) {
        if (r == RED_NONE) return &pass_kernel<W, T, RED_NONE, true, 0, true>;
        if (r == RED_GRAM) return &pass_kernel<W, T, RED_GRAM, true, 0, true>;
        if (r == RED_SKETCH_SPARSE)
            return mt == 4 ? &pass_kernel<W, T, RED_SKETCH_SPARSE, true, 0, true, 4>
                           : &pass_kernel<W, T, RED_SKETCH_SPARSE, true, 0, true>;
        if (r == RED_SKETCH_DENSE) return &pass_kernel<W, T, RED_SKETCH_DENSE, true, 0, true>;
    }
    if (!u && t == 1 && !wr && r == RED_GRAM) return &pass_kernel<W, T, RED_GRAM, false, 1, false>;
    if (!u && t == 2 && wr && r == RED_GRAM) return &pass_kernel<W, T, RED_GRAM, false, 2, true>;
    if (r == RED_NONE && t == 1 && wr) {
        if (!u) return &pass_kernel<W, T, RED_NONE, false, 1, true>;
        return &pass_kernel<W, T, RED_NONE, true, 1, true>;
    }
    return nullptr;
}

// The two-block passes of the one-stage block QR and the solve-first passes of a single block.
template <int W, typename T>
KernelPtr select_w_pair(const PassKey& k) {
    const int mt = (k.tiles >= 1 && k.tiles <= 4) ? 4 : (k.tiles >= 5 && k.tiles <= 6) ? 6 : 8;
    if (k.pair == SOLO_PROJ && k.red == RED_PROJ)
        return mt == 4   ? &pass_kernel_pair<W, T, RED_PROJ, SOLO_PROJ, 4>
               : mt == 6 ? &pass_kernel_pair<W, T, RED_PROJ, SOLO_PROJ, 6>
                         : &pass_kernel_pair<W, T, RED_PROJ, SOLO_PROJ>;
    if (k.pair == SOLO_UPD && k.red == RED_GRAM) return &pass_kernel_pair<W, T, RED_GRAM, SOLO_UPD>;
    if constexpr (W <= kMaxPairW) {
        if (k.pair == PAIR_PROJ && k.red == RED_PROJ)
            return mt == 4   ? &pass_kernel_pair<W, T, RED_PROJ, PAIR_PROJ, 4>
                   : mt == 6 ? &pass_kernel_pair<W, T, RED_PROJ, PAIR_PROJ, 6>
                             : &pass_kernel_pair<W, T, RED_PROJ, PAIR_PROJ>;
        if constexpr (sizeof(T) == 4) {
            if (k.pair == PAIR_CROSS && k.red == RED_GRAM) return &pass_kernel_pair<W, T, RED_GRAM, PAIR_CROSS>;
        } else {
            if (k.pair == PAIR_UPD && k.red == RED_GRAM) return &pass_kernel_pair<W, T, RED_GRAM, PAIR_UPD>;
            if (k.pair == PAIR_LEAD) {
                if (k.red == RED_GRAM) return &pass_kernel_pair<W, T, RED_GRAM, PAIR_LEAD>;
                if (k.red == RED_SKETCH_DENSE) return &pass_kernel_pair<W, T, RED_SKETCH_DENSE, PAIR_LEAD>;
                if (k.red == RED_SKETCH_SPARSE)
                    return mt == 4 ? &pass_kernel_pair<W, T, RED_SKETCH_SPARSE, PAIR_LEAD, 4>
                                   : &pass_kernel_pair<W, T, RED_SKETCH_SPARSE, PAIR_LEAD>;
            }
        }
    }
    return nullptr;
}

// The variants of the mixed-precision GMRES panel step: panel 1 reads the FP64 panel
// against the FP32 basis and writes the panel (projection; update + sketch); panel 2 writes
// the finished columns into the FP32 basis (update + solve).
template <int W>
KernelPtr select_w_panel(const PassKey& k) {
    const int r = k.red;
    const bool u = k.upd, wr = k.write;
    const int t = k.ntrsm;
    const int mt = (k.tiles >= 1 && k.tiles <= 4) ? 4 : (k.tiles >= 5 && k.tiles <= 6) ? 6 : 8;
    if (k.panel == 1) {
        if (!u && t == 0 && !wr && r == RED_PROJ)
            return mt == 4   ? &pass_kernel_panel<W, double, RED_PROJ, false, 0, false, 4>
                   : mt == 6 ? &pass_kernel_panel<W, double, RED_PROJ, false, 0, false, 6>
                             : &pass_kernel_panel<W, double, RED_PROJ, false, 0, false>;
        if (u && t == 0 && wr) {
            if (r == RED_SKETCH_SPARSE)
                return mt == 4 ? &pass_kernel_panel<W, double, RED_SKETCH_SPARSE, true, 0, true, 4>
                               : &pass_kernel_panel<W, double, RED_SKETCH_SPARSE, true, 0, true>;
            if (r == RED_SKETCH_DENSE) return &pass_kernel_panel<W, double, RED_SKETCH_DENSE, true, 0, true>;
        }
    }
    if (k.panel == 2 && r == RED_NONE && t == 1 && wr)
        return u ? &pass_kernel_panel<W, float, RED_NONE, true, 1, true>
                 : &pass_kernel_panel<W, float, RED_NONE, false, 1, true>;
    return nullptr;
}

// The batched variants the lock-step two-stage solver launches.
template <int W, typename T>
BatchedKernelPtr select_w_batched(const PassKey& k) {
    const int r = k.red;
    const bool u = k.upd, wr = k.write;
    const int t = k.ntrsm;
    const bool few = k.tiles >= 1 && k.tiles <= 4;
    if (!u && t == 0 && !wr) {
        if (r == RED_PROJ)
            return few ? &pass_kernel_batched<W, T, RED_PROJ, false, 0, false, 4>
                       : &pass_kernel_batched<W, T, RED_PROJ, false, 0, false>;
        if (r == RED_SKETCH_SPARSE)
            return few ? &pass_kernel_batched<W, T, RED_SKETCH_SPARSE, false, 0, false, 4>
                       : &pass_kernel_batched<W, T, RED_SKETCH_SPARSE, false, 0, false>;
    }
    if (u && t == 0 && wr && r == RED_SKETCH_SPARSE)
        return few ? &pass_kernel_batched<W, T, RED_SKETCH_SPARSE, true, 0, true, 4>
                   : &pass_kernel_batched<W, T, RED_SKETCH_SPARSE, true, 0, true>;
    if (r == RED_NONE && t == 1 && wr) {
        if (!u) return &pass_kernel_batched<W, T, RED_NONE, false, 1, true>;
        return &pass_kernel_batched<W, T, RED_NONE, true, 1, true>;
    }
    return nullptr;
}

template <int W>
int rows_w(int red) {
    switch (red) {
        case RED_PROJ: return Cfg<W, RED_PROJ>::ROWS;
        case RED_GRAM: return Cfg<W, RED_GRAM>::ROWS;
        case RED_SKETCH_SPARSE: return Cfg<W, RED_SKETCH_SPARSE>::ROWS;
        case RED_SKETCH_DENSE: return Cfg<W, RED_SKETCH_DENSE>::ROWS;
        default: return 0;
    }
}

template <int W>
int threads_w(int red) {
    switch (red) {
        case RED_SKETCH_SPARSE: return Cfg<W, RED_SKETCH_SPARSE>::NT;
        case RED_SKETCH_DENSE: return Cfg<W, RED_SKETCH_DENSE>::NT;
        case RED_PROJ: return Cfg<W, RED_PROJ>::NT;
        case RED_GRAM: return Cfg<W, RED_GRAM>::NT;
        default: return Cfg<W, RED_NONE>::NT;
    }
}

}  // namespace passk

// Per-width selectors, one translation unit each (pass_wNN.hip).
struct PassSel {
    passk::KernelPtr fn;
    passk::BatchedKernelPtr fnb;  // batched form (null where not instantiated)
    int threads;  // workgroup size (= strip rows)
    int rows;     // reduction rows one launch can produce
};
PassSel select_pass_w1(const PassKey& k);
PassSel select_pass_w2(const PassKey& k);
PassSel select_pass_w3(const PassKey& k);
PassSel select_pass_w4(const PassKey& k);
PassSel select_pass_w5(const PassKey& k);
PassSel select_pass_w6(const PassKey& k);
PassSel select_pass_w7(const PassKey& k);
PassSel select_pass_w8(const PassKey& k);
PassSel select_pass_w9(const PassKey& k);
PassSel select_pass_w10(const PassKey& k);
PassSel select_pass_w11(const PassKey& k);
PassSel select_pass_w12(const PassKey& k);
PassSel select_pass_w13(const PassKey& k);
PassSel select_pass_w14(const PassKey& k);
PassSel select_pass_w15(const PassKey& k);
PassSel select_pass_w16(const PassKey& k);

}  // namespace sko
