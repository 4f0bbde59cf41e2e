// vmc_mo.hip -- MO rows of every (walker, electron) on the matrix cores.
//
//   out[row][c][i] = sum_mu AO_c(r_row)[mu] C[mu][i],   c < NC
//   (NC = 1: values;  NC = 5: value, gradient, Laplacian)
//
// A block owns 64 rows (one 16-row tile per wavefront) and all n orbitals
// (NT tiles of 16 columns).  C is read from a copy padded to 64 columns and
// 16 extra zero rows (k_prepare), one 16-byte vector per thread and tile.  The
// AO tile is zeroed once: its AOs past the tile's last one then hold finite
// values of earlier tiles, which meet zero rows of the C tile.  AO tiles of whole shells (<= 16 AOs) are
// produced in LDS by a GTO evaluation that gives each wavefront one shell at
// all 64 rows (uniform angular momentum) and consumed in k-steps of
// 4 AOs by 16x16x4 MFMA (FP64: v_mfma_f64_16x16x4_f64; FP32:
// v_mfma_f32_16x16x4_f32), accumulating in the arithmetic type T.
//
// Bound: FP32 and FP64 MFMA run on the vector ALUs' multipliers, so a SIMD's
// time is the sum of its MFMA cycles (33 per 16x16x4 in FP32) and its other
// VALU cycles (FP32 2 to 3, FP64 4 to 5, exponential 9 per instruction); the
// two do not overlap.  At 21 atoms, 3.1e6 measurement rows in FP32: MFMA 2.3
// of 4.1 ms.  What the evaluation reads of a shell is one 128-byte record
// loaded one shell ahead (a chain of table lookups before), an atom's shells
// share its displacement, the component factors are constants, the tile's
// shells are dealt to the wavefronts by cost, and the occupancy target keeps
// the accumulators in VGPRs at three wavefronts per SIMD (FP32, five
// components).  Per launch at 21 atoms: FP32 measurement rows 4.84 -> 4.14 ms
// (32768 walkers), FP32 proposals 2.81 -> 1.97 ms (65536 walkers; k_mo_values
// below), FP64 4.51 -> 3.90 ms and 1.60 -> 1.11 ms (16384 walkers).
#include <algorithm>

#include "vmc_mfma.hpp"
#include "vmc_pipeline.hpp"
#include "vmc_regs.hpp"

namespace vmcx {

// What the row kernels read of (C, R): C padded to [M + 16][64] with zero rows
// and columns (FP64 Cp; with Cpf also FP32, and the plain FP32 copy Cf of C),
// and the shell records at the nuclei R.
__global__ __launch_bounds__(256) void k_prepare(const double *__restrict__ C, int M, int n,
                                                 const double *__restrict__ R, const ShellRec *__restrict__ src,
                                                 int n_rec, double *__restrict__ Cp, float *__restrict__ Cpf,
                                                 float *__restrict__ Cf, ShellRec *__restrict__ rec) {
    const int k = blockIdx.x * 256 + threadIdx.x;
    if (k < n_rec) {
        ShellRec q = src[k];
        q.x = R[3 * q.atom];
        q.y = R[3 * q.atom + 1];
        q.z = R[3 * q.atom + 2];
        rec[k] = q;
    }
    if (k >= (M + 16) * 64) return;
    const int mu = k >> 6, i = k & 63;
    const bool in = mu < M && i < n;
    const double v = in ? C[(size_t)mu * n + i] : 0.0;
    Cp[k] = v;
    if (Cpf) {
        Cpf[k] = (float)v;
        if (in) Cf[(size_t)mu * n + i] = (float)v;
    }
}

// Wavefronts per SIMD: FP32 with five components takes three up to 48 orbitals
// (168 VGPRs; four spill: 5.7 instead of 4.1 ms per launch); FP64 values four
// (1.11 against 1.39 ms).
template <typename T, int NC, int NT>
constexpr int mo_waves() {
    return sizeof(T) == 4 ? (NC == 1 ? 6 : (NT <= 3 ? 3 : 2)) : (NC == 1 ? 4 : 2);
}

template <typename T, int NC, int NT>
__global__ __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(mo_waves<T, NC, NT>()))) void k_mo_rows_mfma(int n, const T *__restrict__ Cp, ShellTiles tiles,
                                                      const double *__restrict__ pos, int64_t n_rows,
                                                      T *__restrict__ out, const int *__restrict__ rows_dev) {
    constexpr int RB = 64, MT = 16;
    constexpr int RS = MT * NC + 1;    // odd row stride of the AO tile
    typedef typename std::conditional<NC == 5, double, T>::type W;   // type of the evaluation
    constexpr int CS = 80;             // row stride of the C tile (lane groups hit disjoint banks)
    __shared__ T aot[RB * RS];
    __shared__ T ct[MT * CS];
    typedef Mfma<T> MF;
    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int64_t row0 = (int64_t)blockIdx.x * RB;
    // (a row count known only on the device: the blocks past it leave)
    if (rows_dev) n_rows = min(n_rows, (int64_t)*rows_dev);
    if (row0 >= n_rows) return;
    // this lane's row of the evaluation (rows past the end repeat the last)
    const double *pr = pos + 3 * min(row0 + lane, n_rows - 1);
    const double px = pr[0], py = pr[1], pz = pr[2];
    // which wavefront's share of a tile's shells this one evaluates: turned
    // from block to block, so that the four SIMDs of a CU get equal work
    const int turn = (wave + (int)blockIdx.x) & 3;
    for (int k = tid; k < RB * RS; k += 256) aot[k] = T(0);
    typename MF::acc_t acc[NC][NT];
#pragma unroll
    for (int c = 0; c < NC; ++c)
#pragma unroll
        for (int t = 0; t < NT; ++t) acc[c][t] = MF::zero();
    const int ar = wave * 16 + (lane & 15);   // A-operand row of this lane
    const int ak = lane >> 4;                 // A-operand k (AO within the k-step)
    ShellDisp<W> sd;
    for (int tile = 0; tile < tiles.n_tiles; ++tile) {
        const TileHdr hd = ldc(tiles.hdr + tile);
        const int mu0 = hd.x, nmu = hd.y;
        __syncthreads();
        // a wavefront evaluates one shell at the block's 64 rows at a time, so
        // the angular momentum (and the shell's record) are uniform over it
        const int q1 = (hd.w >> (8 * turn)) & 255, q0 = turn ? (hd.w >> (8 * turn - 8)) & 255 : 0;
        RecVals<W> rc = rec_load<W>(tiles.rec + hd.z + q0);
        for (int q = q0; q < q1; ++q) {
            const RecVals<W> cur = rc;
            rc = rec_load<W>(tiles.rec + hd.z + q + 1);   // (one record past the last is there)
            shell_rec_eval<NC, T, W>(tiles, cur, sd, px, py, pz, aot + lane * RS);
        }
        // C tile: rows of the tile's AOs, zero rows past its last AO
        constexpr int VW = 16 / sizeof(T);
        typedef T V __attribute__((ext_vector_type(VW)));
        for (int p = tid; p < MT * 64 / VW; p += 256) {
            const int m = p / (64 / VW), i = (p - m * (64 / VW)) * VW;
            const V v = *(const V *)(Cp + (size_t)(mu0 + m) * 64 + i);
            *(V *)(ct + m * CS + i) = m < nmu ? v : V(T(0));
        }
        __syncthreads();
        const int ksteps = (nmu + 3) >> 2;
        for (int ks = 0; ks < ksteps; ++ks) {
            const int m = ks * 4 + ak;
            T a[NC], b[NT];
#pragma unroll
            for (int c = 0; c < NC; ++c) a[c] = aot[ar * RS + m * NC + c];
#pragma unroll
            for (int t = 0; t < NT; ++t) b[t] = ct[m * CS + t * 16 + (lane & 15)];
#pragma unroll
            for (int c = 0; c < NC; ++c)
#pragma unroll
                for (int t = 0; t < NT; ++t) acc[c][t] = MF::fma(a[c], b[t], acc[c][t]);
        }
    }
    const int col = lane & 15;
#pragma unroll
    for (int v = 0; v < 4; ++v) {
        const int64_t row = row0 + wave * 16 + MF::row(lane, v);
        if (row >= n_rows) continue;
#pragma unroll
        for (int c = 0; c < NC; ++c)
#pragma unroll
            for (int t = 0; t < NT; ++t) {
                const int i = t * 16 + col;
                if (i < n) out[(row * NC + c) * n + i] = acc[c][t][v];
            }
    }
}

// Values only (the sweep's proposals and MO matrix), many rows: a wavefront
// owns 64 rows, evaluates every shell of a tile at them (lane = row) into its
// own part of LDS and multiplies all four row tiles itself, its entries of C
// in registers, so no wavefront waits for another: while one waits for its loads
// or LDS, the others of its SIMD evaluate or multiply.
template <typename T, int NT>
__global__ __launch_bounds__(256) void k_mo_values(int n, const T *__restrict__ Cp, ShellTiles tiles,
                                                   const double *__restrict__ pos, int64_t n_rows,
                                                   T *__restrict__ out) {
    constexpr int MT = 16, RS = MT + 1;
    __shared__ T aot[4][64 * RS];
    typedef Mfma<T> MF;
    const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int64_t row0 = ((int64_t)blockIdx.x * 4 + wave) * 64;
    if (row0 >= n_rows) return;   // no block barrier in this kernel
    const double *pr = pos + 3 * min(row0 + lane, n_rows - 1);
    const double px = pr[0], py = pr[1], pz = pr[2];
    T *at = aot[wave];
    for (int k = lane; k < 64 * RS; k += 64) at[k] = T(0);
    typename MF::acc_t acc[4][NT];
#pragma unroll
    for (int r = 0; r < 4; ++r)
#pragma unroll
        for (int t = 0; t < NT; ++t) acc[r][t] = MF::zero();
    const int ml = lane & 15, kg = lane >> 4;
    RecVals<T> rc = rec_load<T>(tiles.rec + ldc(tiles.hdr).z);
    ShellDisp<T> sd;
    for (int tile = 0; tile < tiles.n_tiles; ++tile) {
        const TileHdr hd = ldc(tiles.hdr + tile);
        const int mu0 = hd.x, nmu = hd.y, nsh = (hd.w >> 24) & 255;
        // C entries of the tile's AOs, zero past its last one
        T b[4][NT];
#pragma unroll
        for (int ks = 0; ks < 4; ++ks)
#pragma unroll
            for (int t = 0; t < NT; ++t) {
                const T v = Cp[(size_t)(mu0 + 4 * ks + kg) * 64 + 16 * t + ml];
                b[ks][t] = 4 * ks + kg < nmu ? v : T(0);
            }
        for (int q = 0; q < nsh; ++q) {
            const RecVals<T> cur = rc;
            rc = rec_load<T>(tiles.rec + hd.z + q + 1);   // (one record past the last is there)
            shell_rec_eval<1, T, T>(tiles, cur, sd, px, py, pz, at + lane * RS);
        }
        wave_sync_s();
#pragma unroll
        for (int ks = 0; ks < 4; ++ks)
#pragma unroll
            for (int r = 0; r < 4; ++r) {
                const T a = at[(16 * r + ml) * RS + 4 * ks + kg];
#pragma unroll
                for (int t = 0; t < NT; ++t) acc[r][t] = MF::fma(a, b[ks][t], acc[r][t]);
            }
        wave_sync_s();
    }
#pragma unroll
    for (int r = 0; r < 4; ++r)
#pragma unroll
        for (int v = 0; v < 4; ++v) {
            const int64_t row = row0 + 16 * r + MF::row(lane, v);
            if (row >= n_rows) continue;
#pragma unroll
            for (int t = 0; t < NT; ++t)
                if (16 * t + ml < n) out[row * n + 16 * t + ml] = acc[r][t][v];
        }
}

// Rows from which k_mo_values is the faster one in FP32 (21 atoms, block
// kernel against k_mo_values: 131600 rows 72 / 85 us, 385024 rows 158 / 157 us;
// 18 atoms, 606134 rows 184 / 190 us; 21 atoms, 6.2e6 rows 2.15 / 1.97 ms): its
// blocks take four times the rows, so that fewer rows leave SIMDs without a
// wavefront.  In FP64 the block kernel is faster at every size (five wavefronts
// against two to a SIMD; 1.54e6 rows 1.11 / 1.19 ms).
constexpr int64_t MO_VALUES_ROWS = 1 << 20;

template <typename T, int NC>
static hipError_t launch_nc(int n, const T *Cp, const ShellTiles &tiles, const double *pos, int64_t n_rows, T *out,
                            const int *rows_dev, hipStream_t st) {
    const dim3 g((unsigned)((n_rows + 63) / 64)), b(256);
    switch ((n + 15) / 16) {
        case 1: hipLaunchKernelGGL((k_mo_rows_mfma<T, NC, 1>), g, b, 0, st, n, Cp, tiles, pos, n_rows, out, rows_dev); break;
        case 2: hipLaunchKernelGGL((k_mo_rows_mfma<T, NC, 2>), g, b, 0, st, n, Cp, tiles, pos, n_rows, out, rows_dev); break;
        case 3: hipLaunchKernelGGL((k_mo_rows_mfma<T, NC, 3>), g, b, 0, st, n, Cp, tiles, pos, n_rows, out, rows_dev); break;
        default: hipLaunchKernelGGL((k_mo_rows_mfma<T, NC, 4>), g, b, 0, st, n, Cp, tiles, pos, n_rows, out, rows_dev); break;
    }
    return hipGetLastError();
}

template <typename T>
hipError_t launch_mo_rows_mfma(const SysDev &S, const Prepared &P, const double *pos, int64_t n_rows, T *out, int nc,
                               hipStream_t st, const int *rows_dev) {
    if (S.n_occ > 64) return hipErrorInvalidValue;
    const T *Cp;
    if constexpr (sizeof(T) == 4)
        Cp = P.Cpf;
    else
        Cp = P.Cp;
    if constexpr (sizeof(T) == 4)
        if (nc == 1 && rows_dev == nullptr && n_rows >= MO_VALUES_ROWS) {
            const dim3 g((unsigned)((n_rows + 255) / 256)), b(256);
            const int n = S.n_occ;
            switch ((n + 15) / 16) {
                case 1: hipLaunchKernelGGL((k_mo_values<T, 1>), g, b, 0, st, n, Cp, P.mo, pos, n_rows, out); break;
                case 2: hipLaunchKernelGGL((k_mo_values<T, 2>), g, b, 0, st, n, Cp, P.mo, pos, n_rows, out); break;
                case 3: hipLaunchKernelGGL((k_mo_values<T, 3>), g, b, 0, st, n, Cp, P.mo, pos, n_rows, out); break;
                default: hipLaunchKernelGGL((k_mo_values<T, 4>), g, b, 0, st, n, Cp, P.mo, pos, n_rows, out); break;
            }
            return hipGetLastError();
        }
    return nc == 1 ? launch_nc<T, 1>(S.n_occ, Cp, P.mo, pos, n_rows, out, rows_dev, st)
                   : launch_nc<T, 5>(S.n_occ, Cp, P.mo, pos, n_rows, out, rows_dev, st);
}

hipError_t launch_prepare(const double *C, int M, int n, const double *R, const ShellRec *src, int n_rec, double *Cp,
                          float *Cpf, float *Cf, ShellRec *rec, hipStream_t st) {
    const int np = std::max((M + 16) * 64, n_rec);
    hipLaunchKernelGGL(k_prepare, dim3((unsigned)((np + 255) / 256)), dim3(256), 0, st, C, M, n, R, src, n_rec, Cp, Cpf,
                       Cf, rec);
    return hipGetLastError();
}

template hipError_t launch_mo_rows_mfma<double>(const SysDev &, const Prepared &, const double *, int64_t, double *,
                                                int, hipStream_t, const int *);
template hipError_t launch_mo_rows_mfma<float>(const SysDev &, const Prepared &, const double *, int64_t, float *, int,
                                               hipStream_t, const int *);

}  // namespace vmcx
