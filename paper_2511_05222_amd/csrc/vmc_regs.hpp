// vmc_regs.hpp -- wavefront register-level helpers (gfx950): lane reads and
// the in-register Gauss-Jordan inversion shared by the sweep and the
// measurement.
#pragma once

#include <hip/hip_runtime.h>

#include "vmc_device.hpp"

namespace vmcx {

__device__ inline void wave_sync_s() {
    __builtin_amdgcn_fence(__ATOMIC_SEQ_CST, "wavefront");
    __builtin_amdgcn_wave_barrier();
}

__device__ inline double readlane_d(double v, int src) {
    const long long b = __double_as_longlong(v);
    const int lo = __builtin_amdgcn_readlane((int)b, src);
    const int hi = __builtin_amdgcn_readlane((int)(b >> 32), src);
    return __longlong_as_double(((long long)hi << 32) | (long long)(unsigned)lo);
}

__device__ inline float readlane_t(float v, int src) {
    return __int_as_float(__builtin_amdgcn_readlane(__float_as_int(v), src));
}
__device__ inline double readlane_t(double v, int src) { return readlane_d(v, src); }

// Maximum over each row of 16 lanes, in all of them.
__device__ inline unsigned row16_max_u32(unsigned v) {
    v = max(v, (unsigned)__builtin_amdgcn_update_dpp(0, (int)v, 0xB1, 0xF, 0xF, false));    // quad [1,0,3,2]
    v = max(v, (unsigned)__builtin_amdgcn_update_dpp(0, (int)v, 0x4E, 0xF, 0xF, false));    // quad [2,3,0,1]
    v = max(v, (unsigned)__builtin_amdgcn_update_dpp(0, (int)v, 0x141, 0xF, 0xF, false));   // half-row mirror
    return max(v, (unsigned)__builtin_amdgcn_update_dpp(0, (int)v, 0x140, 0xF, 0xF, false));   // row mirror
}

// Maximum of an unsigned value over the wavefront (uniform result): the four
// row results by lane reads.
__device__ inline unsigned wave_max_u32(unsigned v) {
    v = row16_max_u32(v);
    const unsigned a = __builtin_amdgcn_readlane(v, 0), b = __builtin_amdgcn_readlane(v, 16),
                   c = __builtin_amdgcn_readlane(v, 32), d = __builtin_amdgcn_readlane(v, 48);
    return max(max(a, b), max(c, d));
}

// In-register Gauss-Jordan inversion (FP64) of one spin block by one
// wavefront, with partial pivoting by implicit row choice.  The matrix is
// B = A^T of the block (row c = orbital c, column k = electron k), padded to
// KN x KN with an identity block and spread over all 64 lanes: lane (g, m),
// g = lane / 16, m = lane % 16, holds rows c = m + 16 s (s < KN/16) and
// columns k = 4 q + g (q < KN/4) as Br[s * KN/4 + q].
// Step k eliminates column k, which a rotation every four steps keeps in the
// registers q = 0 of group k % 4.  The column goes through LDS to the other
// groups (which hold the same rows), the pivot row's entries to the lanes of
// their own group (which hold the same columns); every lane then updates its
// KN^2 / 64 entries.  Bound: the latency of a step's chain (two LDS round trips,
// a maximum, a reciprocal): about 600 of a SIMD's cycles a step at KN = 48 with
// three wavefronts, of which 310 issue, 166 of them the 36 FMAs.  (A lane to each row, the pivot row broadcast by
// two lane reads per entry, issues 3 instructions for each of KN entries a step
// instead of 1 for KN^2 / 64, on KN of the 64 lanes.  A rebuild of all walkers
// within the FP32 sweep of 65536 walkers, 21 atoms: 1.47 -> 0.77 ms; within the
// FP64 sweep of 16384: 0.41 -> 0.26 ms; k_dense<float, 48> with rebuilds, 8192
// walkers: 1.59 -> 1.13 ms.)
// The pivot of step k is an unused row with the largest |B[.][k]| compared on
// a 32-bit key: |B| rounded to FP32 with its six low mantissa bits replaced by
// (63 - row), so that values within 2^-17 of each other count as equal and the
// lowest such row wins (any such pivot is a partial-pivoting choice; NaN and 0
// rank lowest among the unused rows).  With p_k the pivot row of step k the
// result is B[p_k][j] -> K[p_j][k]: row p_k holds column k of K = A^-1, its
// column j orbital p_j.  On return sig[s] = k on the row that was p_k.  The
// block counts as singular (bad set) when a pivot is no larger than tol
// (gj_tol below: 2^-40 of the block's largest entry), so a row that is a
// linear combination of the others to working precision, e.g. two coincident
// same-spin electrons, or an all-zero row is reported.  A NaN pivot is not: it
// leaves non-finite results, reported as such.  With LOGDET, logabs =
// log|prod_k pivot_k| = log|det B| (the identity padding adds 0).
// ws: gj_ws_bytes<KN>() of 16-byte aligned LDS of the wavefront's own.
template <int KN>
constexpr int gj_ws_bytes() { return KN * 8 + 4 * (KN / 4 + 2) * 8; }

template <int KN, bool LOGDET>
__device__ inline void gj_regs(double (&Br)[KN * KN / 64], int (&sig)[KN / 16], bool &bad, double &logabs,
                               double tol, double *ws) {
    constexpr int RR = KN / 16, CC = KN / 4;
    typedef double V2 __attribute__((ext_vector_type(2)));
    const int lane = threadIdx.x & 63, m = lane & 15, g = lane >> 4;
    double *col = ws;                                // [KN] the eliminated column
    double *prow = ws + KN + g * (CC + 2);           // the pivot row's entries of this group
    // per row: the low key bits, and the key's mask, cleared once it was a pivot
    unsigned low[RR], open[RR];
    double mant = 1.0;
    int expo = 0;
#pragma unroll
    for (int s = 0; s < RR; ++s) {
        sig[s] = 0;
        low[s] = 63u - (unsigned)(m + 16 * s);
        open[s] = ~0u;
    }
    for (int q0 = 0; q0 < CC; ++q0) {
#pragma unroll
        for (int gk = 0; gk < 4; ++gk) {
            if (g == gk)
#pragma unroll
                for (int s = 0; s < RR; ++s) col[m + 16 * s] = Br[s * CC];
            wave_sync_s();
            double a0[RR];
#pragma unroll
            for (int s = 0; s < RR; ++s) a0[s] = col[m + 16 * s];
            unsigned key = 0u;
#pragma unroll
            for (int s = 0; s < RR; ++s) {
                // (the maximum with 0 ranks a NaN as 0)
                const unsigned fb = __float_as_uint(fmaxf((float)fabs(a0[s]), 0.0f));
                key = max(key, max((fb & ~63u) | low[s], 64u | low[s]) & open[s]);
            }
            const int p = 63 - (int)(row16_max_u32(key) & 63u);   // every row of 16 lanes holds all rows
            const int pu = __builtin_amdgcn_readfirstlane(p);
#pragma unroll
            for (int s = 0; s < RR; ++s)
                if (m + 16 * s == pu) {
#pragma unroll
                    for (int q = 0; q < CC; q += 2) *(V2 *)(prow + q) = V2{Br[s * CC + q], Br[s * CC + q + 1]};
                    open[s] = 0u;
                    sig[s] = 4 * q0 + gk;
                }
            wave_sync_s();
            const double piv = col[pu];
            if (fabs(piv) <= tol) bad = true;
            if (LOGDET) {
                mant *= __builtin_amdgcn_frexp_mant(piv);
                expo += __builtin_amdgcn_frexp_exp(piv);
            }
            const double inv = rcp_nr(piv);   // a few ulp; a zero pivot is flagged above
            // other rows: B[i][j] - (B[i][k] / piv) B[p][j];  pivot row: B[p][j] / piv,
            // formed by the same fma as B[p][j] - (1 - 1/piv) B[p][j] (its own
            // row; relative error |piv - 1| 2^-53 from rounding 1 - 1/piv)
            double ga[RR], G[RR];
#pragma unroll
            for (int s = 0; s < RR; ++s) {
                ga[s] = a0[s] * inv;
                G[s] = m + 16 * s == pu ? 1.0 - inv : ga[s];
            }
            V2 P[CC / 2];
#pragma unroll
            for (int q = 0; q < CC / 2; ++q) P[q] = *(const V2 *)(prow + 2 * q);
#pragma unroll
            for (int s = 0; s < RR; ++s) {
                double *R = Br + s * CC;
                double x0 = fma(-G[s], P[0][0], R[0]);
                if (g == gk) x0 = m + 16 * s == pu ? inv : -ga[s];
                // (after the group's last column of four the registers move down by one)
                if (gk < 3) R[0] = x0;
#pragma unroll
                for (int q = 1; q < CC; ++q) R[gk < 3 ? q : q - 1] = fma(-G[s], P[q / 2][q & 1], R[q]);
                if (gk == 3) R[CC - 1] = x0;
            }
        }
    }
    if (LOGDET) logabs = log(fabs(mant)) + (double)expo * 0.69314718055994531;
}

// The rows of gj_regs' result from its layout to one row to a lane, 16 columns
// at a time (so that the two layouts are not both whole in registers): lane c <
// KN gets row c (column k in Kr[k]) and its sig; lanes >= KN zeros and their
// own number.  buf: gj_row_bytes<T, KN>() of the wavefront's LDS (may be ws).
template <typename T, int KN>
constexpr int gj_row_bytes() { return KN * (16 + 16 / (int)sizeof(T)) * (int)sizeof(T); }

template <typename T, int KN>
__device__ inline void gj_to_rows(const double (&Br)[KN * KN / 64], const int (&sig)[KN / 16], T (&Kr)[KN],
                                  int &sig1, T *buf) {
    constexpr int RR = KN / 16, CC = KN / 4, VL = 16 / sizeof(T), LD = 16 + VL;
    typedef T V __attribute__((ext_vector_type(VL)));
    const int lane = threadIdx.x & 63, m = lane & 15, g = lane >> 4;
    const T *row = buf + min(lane, KN - 1) * LD;
    sig1 = lane;
#pragma unroll
    for (int s = 0; s < RR; ++s) {
        // (lane c = m + 16 s: row c of group s)
        if (g == s) sig1 = sig[s];
    }
#pragma unroll
    for (int c0 = 0; c0 < KN; c0 += 16) {
        wave_sync_s();
#pragma unroll
        for (int q = 0; q < 4; ++q)
#pragma unroll
            for (int s = 0; s < RR; ++s) buf[(m + 16 * s) * LD + 4 * q + g] = (T)Br[s * CC + c0 / 4 + q];
        wave_sync_s();
#pragma unroll
        for (int r = 0; r < 16; r += VL) {
            const V v = *(const V *)(row + r);
#pragma unroll
            for (int u = 0; u < VL; ++u) Kr[c0 + r + u] = lane < KN ? v[u] : T(0);
        }
    }
    wave_sync_s();
}

// Singularity threshold of gj_regs from each lane's largest |entry| of the
// block (padding excluded): 2^-40 of the block's largest entry, i.e. a pivot
// that lost 40 of the 53 significant bits.  The wavefront maximum is taken
// on the high words of the non-negative doubles (monotonic in the value),
// rounded up; NaN entries must be left out by the caller (fmax does).
__device__ inline double gj_tol(double lane_max) {
    const unsigned hi = wave_max_u32((unsigned)__double2hiint(lane_max));
    return __hiloint2double((int)hi, -1) * 0x1p-40;
}

}  // namespace vmcx
