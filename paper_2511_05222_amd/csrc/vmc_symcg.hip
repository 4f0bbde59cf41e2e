// vmc_symcg.hip -- conjugate gradients H z_j = -b_j with a symmetric H, reading
// its lower triangle only (gfx950).
//
// H is read in tiles of 64 x 64, and every tile below the diagonal serves both
// its rows (Y[r] += H[r][c] P[c]) and its columns (Y[c] += H[r][c] P[r]).  Up
// to 32 right-hand sides run in lockstep, the columns of the FP64 16x16x4
// matrix-core products (one or two on the vector units).  Vectors are stored
// with the right-hand sides side by side.
//
// A block takes TB x TB tiles (rows of block bi, columns of block bj <= bi); its
// sums over columns go to slot bj of Y, those over rows to slot bi + 1, so that
// every element of H P is the sum of the nb + 1 slots, added in order: the
// result does not depend on the order in which blocks run.
//
// Bound: one or two right-hand sides, HBM: 4 d^2 bytes an iteration plus the
// slots ((nb + 1) d doubles per right-hand side, written and read); 66 us at d =
// 8836 (4.7 TB/s) where reading all of H took 113.  Up to 16, the matrix cores
// and the LDS reads of their operands: 112 us against 247.  Odd iterations take
// the blocks in the opposite order, so that what the last iteration read last
// is still in the memory-side cache (2 %).
#include <algorithm>

#include "vmc_kernels.hpp"
#include "vmc_mfma.hpp"
#include "vmc_regs.hpp"

namespace vmcx {

namespace {

constexpr int TS = 64;         // rows and columns of a tile
constexpr int TL = TS + 4;     // LDS row stride of a tile (doubles): the row fragments without bank conflicts

// red[j] = the sum of v over the threads (q, j), q < 256 / n, thread q n + j
// (the rest hold nothing), by halves.  red: 256 doubles.
__device__ inline void tree_sum(double v, int n, double *red) {
    const int per = 256 / n, q = threadIdx.x / n;
    __syncthreads();
    red[threadIdx.x] = v;
    for (int off = 128; off > 0; off >>= 1) {
        if (off >= per) continue;
        __syncthreads();
        if (q < off && q + off < per) red[threadIdx.x] += red[threadIdx.x + off * n];
    }
    __syncthreads();
}

// out[j] = sum_i src[i * n + j], i < len, for j < n <= 64, the same in every
// block: thread (q, j) takes i = q, q + 256 / n, ....  Ends with a barrier.
__device__ inline void sums_by_rhs(const double *src, int64_t len, int n, double *red, double *out) {
    const int per = 256 / n, j = threadIdx.x % n, q = threadIdx.x / n;
    double v = 0.0;
    if (q < per) {
        int64_t i = q;
        for (; i + 7 * per < len; i += 8 * per) {
            double x[8];
#pragma unroll
            for (int u = 0; u < 8; ++u) x[u] = src[(i + u * per) * n + j];
#pragma unroll
            for (int u = 0; u < 8; ++u) v += x[u];
        }
        for (; i < len; i += per) v += src[i * n + j];
    }
    tree_sum(v, n, red);
    if (threadIdx.x < n) out[threadIdx.x] = red[threadIdx.x];
    __syncthreads();
}

// This block's sums over its threads of two values per right-hand side (thread
// (q, j) as above), to part[block][j] and part[blocks + block][j].
__device__ inline void block_sums(double a, double b, int n, double *red, double *part) {
    for (int c = 0; c < 2; ++c) {
        tree_sum(c ? b : a, n, red);
        if (threadIdx.x < n) part[((int64_t)c * gridDim.x + blockIdx.x) * n + threadIdx.x] = red[threadIdx.x];
    }
}

// Block u of the lower triangle of blocks: u = bi (bi + 1) / 2 + bj.
__device__ inline void block_of(int u, int &bi, int &bj) {
    // (the square root is the vector unit's: back to a scalar)
    bi = __builtin_amdgcn_readfirstlane((int)((sqrtf(8.0f * (float)u + 1.0f) - 1.0f) * 0.5f));
    while ((bi + 1) * (bi + 2) / 2 <= u) ++bi;
    while (bi * (bi + 1) / 2 > u) --bi;
    bj = u - bi * (bi + 1) / 2;
}

}  // namespace

// *differs is set where H is not symmetric to the last bit (or holds a NaN).
// Blocks that start after it is set read nothing: an H with rounding in its two
// halves is found out within the first of them.
__global__ __launch_bounds__(256) void k_sym_check(const double *__restrict__ H, int64_t d, int *differs) {
    __shared__ double t[TS][TS + 1];
    if (blockIdx.x > blockIdx.y) return;
    if (__syncthreads_or(__hip_atomic_load(differs, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT))) return;
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const int64_t r0 = (int64_t)blockIdx.y * TS, c0 = (int64_t)blockIdx.x * TS;
    double v[16];
#pragma unroll
    for (int q = 0; q < 16; ++q)
        v[q] = H[min(r0 + 16 * wave + q, d - 1) * d + min(c0 + lane, d - 1)];
#pragma unroll
    for (int q = 0; q < 16; ++q) t[16 * wave + q][lane] = v[q];
#pragma unroll
    for (int q = 0; q < 16; ++q)
        v[q] = H[min(c0 + 16 * wave + q, d - 1) * d + min(r0 + lane, d - 1)];
    __syncthreads();
    bool bad = false;
#pragma unroll
    for (int q = 0; q < 16; ++q)
        bad = bad || (r0 + lane < d && c0 + 16 * wave + q < d && !(v[q] == t[lane][16 * wave + q]));
    if (__any(bad) && lane == 0) atomicOr(differs, 1);
}

// x = 0, r = -b, dinv = 1 / H_kk (or 1), p = dinv r (zero rows past d, zero
// columns past n), and this block's sums of r.r and r.(dinv r).
__global__ __launch_bounds__(256) void k_sym_setup(const double *__restrict__ H, const double *__restrict__ b,
                                                   int64_t d, int64_t d_pad, int n, int G, int jacobi,
                                                   double *__restrict__ X,
                                                   double *__restrict__ R, double *__restrict__ dinv,
                                                   double *__restrict__ P, double *__restrict__ part) {
    __shared__ double red[256];
    const int per = 256 / n, j = threadIdx.x % n, q = threadIdx.x / n;
    const int64_t k0 = (int64_t)blockIdx.x * per, k = k0 + q;
    double rr = 0.0, rz = 0.0;
    if (q < per && k < d) {
        const double rk = -b[(int64_t)j * d + k], di = jacobi ? 1.0 / H[k * d + k] : 1.0;
        X[k * n + j] = 0.0;
        R[k * n + j] = rk;
        if (j == 0) dinv[k] = di;
        rr = rk * rk;
        rz = rk * (di * rk);
    }
    for (int i = threadIdx.x; i < per * G; i += 256) {
        const int64_t kk = k0 + i / G;
        const int jj = i % G;
        double v = 0.0;
        if (kk < d && jj < n) v = (jacobi ? 1.0 / H[kk * d + kk] : 1.0) * -b[(int64_t)jj * d + kk];
        if (kk < d_pad) P[kk * G + jj] = v;
    }
    block_sums(rr, rz, n, red, part);
}

__global__ __launch_bounds__(256) void k_sym_init(const double *__restrict__ part, int64_t blocks, int n, double rtol,
                                                  int maxit, CgState *cs, int *differs) {
    __shared__ double rr[64], rz[64], red[256];
    if (threadIdx.x == 0) *differs = 0;
    sums_by_rhs(part, blocks, n, red, rr);
    sums_by_rhs(part + blocks * n, blocks, n, red, rz);
    const int j = threadIdx.x;
    if (j >= n) return;
    cs[j].rz = rz[j];
    cs[j].tol2 = rtol * rtol * rr[j];
    cs[j].maxit = maxit;
    cs[j].it = 0;
    cs[j].done = !(std::isfinite(rr[j]) && std::isfinite(rz[j])) ? CG_NONFINITE : (rr[j] == 0.0 ? CG_CONVERGED : 0);
}

// The slots of H P (see the top) and, per block and right-hand side, its part
// of p.(H p).  P has rows up to the next multiple of TS.
template <int NRT, int TB>
__global__ __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(NRT == 1 ? 3 : 2))) void k_sym_matvec(const double *H, const double *P,
                                                    double *Y, double *php, int64_t d,
                                                    int n, int reverse, const CgState *cs) {
    typedef Mfma<double> MF;
    constexpr int G = 16 * NRT;
    extern __shared__ __align__(16) double lds[];
    double *Hs = lds, *Pr = Hs + TS * TL, *Pc = Pr + TS * G;   // a tile of H; P at its rows and at its columns
    __shared__ double red[4][G];
    int running = 0;
    for (int k = 0; k < n; ++k) running |= cs[k].done == 0;
    if (!running) return;
    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int ml = lane & 15, kg = lane >> 4;
    int bi, bj;
    const int u = reverse ? (int)(gridDim.x - 1 - blockIdx.x) : (int)blockIdx.x;
    block_of(u, bi, bj);
    const int nt = (int)((d + TS - 1) / TS), rows = min(TB, nt - TB * bi);   // tile rows of this block
    // tile columns of tile row ti: those below or on the diagonal
    auto cols = [&](int ti) { return bi > bj ? TB : ti + 1; };
    double hr[16], pn[4 * NRT];
    auto load = [&](int ti, int tj) {
        const double *pc = P + (int64_t)(TB * bj + tj) * TS * G + tid;
#pragma unroll
        for (int q = 0; q < 4 * NRT; ++q) pn[q] = pc[256 * q];
        // (rows and columns past the end repeat the last: they meet zeros of P,
        // or results that are not kept)
        const int64_t r0 = (int64_t)(TB * bi + ti) * TS + 16 * wave;
        const unsigned c = (unsigned)min((int64_t)(TB * bj + tj) * TS + lane, d - 1) * 8u;
#pragma unroll
        for (int q = 0; q < 16; ++q) hr[q] = *(const double *)((const char *)(H + min(r0 + q, d - 1) * d) + c);
    };
    typename MF::acc_t ac[TB][NRT];
#pragma unroll
    for (int t = 0; t < TB; ++t)
#pragma unroll
        for (int r = 0; r < NRT; ++r) ac[t][r] = MF::zero();
    double pp[NRT];
#pragma unroll
    for (int r = 0; r < NRT; ++r) pp[r] = 0.0;
    // a 16 x 16 result of rows x0 + kg + 4 v and right-hand sides 16 r + ml:
    // into the slot, and its product with P
    auto flush = [&](const typename MF::acc_t &a, int64_t x0, int r, int64_t slot) {
        const int j = 16 * r + ml;
#pragma unroll
        for (int v = 0; v < 4; ++v) {
            const int64_t k = x0 + kg + 4 * v;
            if (k < d && j < n) {
                Y[(slot * d + k) * n + j] = a[v];
                pp[r] += a[v] * P[k * G + j];
            }
        }
    };
    load(0, 0);
    for (int ti = 0; ti < rows; ++ti) {
        const int64_t r0 = (int64_t)(TB * bi + ti) * TS;
        typename MF::acc_t ar[NRT];
#pragma unroll
        for (int r = 0; r < NRT; ++r) ar[r] = MF::zero();
        // (the barrier before the tile's writes has passed every read of the last row's P)
        bool first = true;
        const int nc = cols(ti);
#pragma unroll 1
        for (int tj = 0; tj < nc; ++tj) {
            const bool below = bi > bj || tj < ti;
            __syncthreads();
#pragma unroll
            for (int q = 0; q < 16; ++q) Hs[(16 * wave + q) * TL + lane] = hr[q];
#pragma unroll
            for (int q = 0; q < 4 * NRT; ++q) Pc[tid + 256 * q] = pn[q];
            if (first) {
#pragma unroll
                for (int q = 0; q < 4 * NRT; ++q) Pr[tid + 256 * q] = P[r0 * G + tid + 256 * q];
                first = false;
            }
            __syncthreads();
            if (tj + 1 < nc)
                load(ti, tj + 1);
            else if (ti + 1 < rows)
                load(ti + 1, 0);
            const double *ha = Hs + (16 * wave + ml) * TL + kg, *hc = Hs + kg * TL + 16 * wave + ml;
#pragma unroll 4
            for (int k = 0; k < 16; ++k) {
                const double a = ha[4 * k];
#pragma unroll
                for (int r = 0; r < NRT; ++r)
                    ar[r] = MF::fma(a, Pc[(4 * k + kg) * G + 16 * r + ml], ar[r]);
            }
            if (below) {
                // (the column's accumulators by a uniform choice: tj is not a
                // constant, so that this body exists once)
                typename MF::acc_t x[NRT];
#pragma unroll
                for (int t = 0; t < TB; ++t)
                    if (t == tj)
#pragma unroll
                        for (int r = 0; r < NRT; ++r) x[r] = ac[t][r];
#pragma unroll 4
                for (int k = 0; k < 16; ++k) {
                    const double a = hc[4 * k * TL];
#pragma unroll
                    for (int r = 0; r < NRT; ++r)
                        x[r] = MF::fma(a, Pr[(4 * k + kg) * G + 16 * r + ml], x[r]);
                }
#pragma unroll
                for (int t = 0; t < TB; ++t)
                    if (t == tj)
#pragma unroll
                        for (int r = 0; r < NRT; ++r) ac[t][r] = x[r];
            }
        }
#pragma unroll
        for (int r = 0; r < NRT; ++r) flush(ar[r], r0 + 16 * wave, r, bj);
    }
#pragma unroll
    for (int tj = 0; tj < TB; ++tj)
#pragma unroll
        for (int r = 0; r < NRT; ++r) flush(ac[tj][r], (int64_t)(TB * bj + tj) * TS + 16 * wave, r, bi + 1);
#pragma unroll
    for (int r = 0; r < NRT; ++r) {
        pp[r] += __shfl_xor(pp[r], 16, 64);
        pp[r] += __shfl_xor(pp[r], 32, 64);
        if (kg == 0) red[wave][16 * r + ml] = pp[r];
    }
    __syncthreads();
    if (tid < n) php[(int64_t)u * n + tid] = (red[0][tid] + red[1][tid]) + (red[2][tid] + red[3][tid]);
}

// The same for one or two right-hand sides on the vector units (the matrix
// cores would use one of their 16 columns): a wavefront takes 16 rows of a tile
// at a time, lane = column, so that H goes from memory to the FMAs without LDS
// or barriers; rows are summed over the lanes at the end of a tile row, columns
// over the block's wavefronts at the end.
template <int NV, int TB>
__global__ __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(NV == 1 && TB == 2 ? 3 : 2))) void k_sym_matvec_few(
    const double *H, const double *P, double *Y, double *php, int64_t d, int reverse, const CgState *cs) {
    // (P is [k][NV] here)
    constexpr int LD = TS + 1;
    __shared__ double tr[4][16 * LD], yc[4][TB][TS][NV], red[4][NV];
    int running = 0;
    for (int k = 0; k < NV; ++k) running |= cs[k].done == 0;
    if (!running) return;
    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    int bi, bj;
    const int u = reverse ? (int)(gridDim.x - 1 - blockIdx.x) : (int)blockIdx.x;
    block_of(u, bi, bj);
    const int nt = (int)((d + TS - 1) / TS), rows = min(TB, nt - TB * bi);
    double hr[16];
    auto load = [&](int ti, int tj) {
        // (rows and columns past the end repeat the last: they meet zeros of P,
        // or results that are not kept)
        const int64_t r0 = (int64_t)(TB * bi + ti) * TS + 16 * wave;
        const unsigned c = (unsigned)min((int64_t)(TB * bj + tj) * TS + lane, d - 1) * 8u;
#pragma unroll
        for (int q = 0; q < 16; ++q)
            hr[q] = *(const double *)((const char *)(H + min(r0 + q, d - 1) * d) + c);
    };
    double ac[TB][NV], pc[TB][NV], pp[NV];
#pragma unroll
    for (int t = 0; t < TB; ++t)
#pragma unroll
        for (int j = 0; j < NV; ++j) {
            ac[t][j] = 0.0;
            const int64_t c = (int64_t)(TB * bj + t) * TS + lane;
            pc[t][j] = c < (int64_t)nt * TS ? P[c * NV + j] : 0.0;
        }
#pragma unroll
    for (int j = 0; j < NV; ++j) pp[j] = 0.0;
    load(0, 0);
    for (int ti = 0; ti < rows; ++ti) {
        const int64_t r0 = (int64_t)(TB * bi + ti) * TS + 16 * wave;
        const int nc = bi > bj ? TB : ti + 1;
        // P of the wavefront's rows: scalar loads (not written by this kernel)
        double s[16][NV], pr[16][NV];
#pragma unroll
        for (int q = 0; q < 16; ++q)
#pragma unroll
            for (int j = 0; j < NV; ++j) {
                s[q][j] = 0.0;
                pr[q][j] = ldc(P + (r0 + q) * NV + j);
            }
#pragma unroll
        for (int tj = 0; tj < TB; ++tj) {
            if (tj >= nc) continue;
            double h[16];
#pragma unroll
            for (int q = 0; q < 16; ++q) h[q] = hr[q];
            if (tj + 1 < nc)
                load(ti, tj + 1);
            else if (ti + 1 < rows)
                load(ti + 1, 0);
            const bool below = bi > bj || tj < ti;
#pragma unroll
            for (int q = 0; q < 16; ++q)
#pragma unroll
                for (int j = 0; j < NV; ++j) {
                    s[q][j] = fma(h[q], pc[tj][j], s[q][j]);
                    if (below) ac[tj][j] = fma(h[q], pr[q][j], ac[tj][j]);
                }
        }
        // the rows' sums over the lanes, through LDS: lane 4 q + part takes 16
        // of row q's 64 values
#pragma unroll
        for (int j = 0; j < NV; ++j) {
            wave_sync_s();
#pragma unroll
            for (int q = 0; q < 16; ++q) tr[wave][q * LD + lane] = s[q][j];
            wave_sync_s();
            const double *x = tr[wave] + (lane >> 2) * LD + 16 * (lane & 3);
            double v = 0.0;
#pragma unroll
            for (int i = 0; i < 16; ++i) v += x[i];
            v += __shfl_xor(v, 1, 64);
            v += __shfl_xor(v, 2, 64);
            const int64_t k = r0 + (lane >> 2);
            if ((lane & 3) == 0 && k < d) {
                Y[((int64_t)bj * d + k) * NV + j] = v;
                pp[j] += v * P[k * NV + j];
            }
        }
    }
#pragma unroll
    for (int t = 0; t < TB; ++t)
#pragma unroll
        for (int j = 0; j < NV; ++j) yc[wave][t][lane][j] = ac[t][j];
    __syncthreads();
    for (int i = tid; i < TB * TS * NV; i += 256) {
        const int j = i % NV, l = (i / NV) % TS, t = i / (NV * TS);
        const int64_t k = (int64_t)(TB * bj + t) * TS + l;
        const double v = (yc[0][t][l][j] + yc[1][t][l][j]) + (yc[2][t][l][j] + yc[3][t][l][j]);
        if (k < d) {
            Y[((int64_t)(bi + 1) * d + k) * NV + j] = v;
            // (256 is a multiple of NV: j is the thread's own)
            const double x = v * P[k * NV + j];
#pragma unroll
            for (int jj = 0; jj < NV; ++jj) pp[jj] += jj == j ? x : 0.0;
        }
    }
#pragma unroll
    for (int j = 0; j < NV; ++j) {
        const double v = wave_sum_dpp(pp[j]);
        if (lane == 0) red[wave][j] = v;
    }
    __syncthreads();
    if (tid < NV) php[(int64_t)u * NV + tid] = (red[0][tid] + red[1][tid]) + (red[2][tid] + red[3][tid]);
}

// alpha = rz / p.Hp; x += alpha p; r -= alpha Hp; this block's sums of r.r and
// r.(dinv r).  Right-hand sides that have ended stay as they are.
__global__ __launch_bounds__(256) void k_sym_update(const double *__restrict__ Y, const double *__restrict__ php,
                                                    int64_t units, int slots, const double *__restrict__ P,
                                                    const double *__restrict__ dinv, int64_t d, int n, int G,
                                                    double *__restrict__ X, double *__restrict__ R,
                                                    double *__restrict__ part, const CgState *__restrict__ cs) {
    __shared__ double red[256], ph[64];
    int running = 0;
    for (int k = 0; k < n; ++k) running |= cs[k].done == 0;
    if (!running) return;
    const int per = 256 / n, j = threadIdx.x % n, q = threadIdx.x / n;
    const int64_t k = (int64_t)blockIdx.x * per + q;
    const bool on = q < per && k < d && cs[j].done == 0;
    // the slots' sum in order, their loads a dozen at a time
    double hp = 0.0;
    if (on) {
        const double *y = Y + k * n + j;
        const int64_t step = d * n;
        int s = 0;
        for (; s + 12 <= slots; s += 12) {
            double x[12];
#pragma unroll
            for (int u = 0; u < 12; ++u) x[u] = y[(s + u) * step];
#pragma unroll
            for (int u = 0; u < 12; ++u) hp += x[u];
        }
        for (; s < slots; ++s) hp += y[s * step];
    }
    sums_by_rhs(php, units, n, red, ph);
    double rr = 0.0, rz = 0.0;
    if (on) {
        const double alpha = cs[j].rz / ph[j];
        X[k * n + j] += alpha * P[k * G + j];
        const double rk = R[k * n + j] - alpha * hp;
        R[k * n + j] = rk;
        rr = rk * rk;
        rz = rk * (dinv[k] * rk);
    }
    block_sums(rr, rz, n, red, part);
}

// The stopping tests, beta = rz_new / rz and p = dinv r + beta p.  Every block
// forms the same sums; block 0 writes the state that the next iteration reads
// (cs -> next).
__global__ __launch_bounds__(256) void k_sym_direction(const double *__restrict__ part, int64_t blocks,
                                                       const double *__restrict__ R, const double *__restrict__ dinv,
                                                       int64_t d, int n, int G, double *__restrict__ P,
                                                       const CgState *__restrict__ cs, CgState *__restrict__ next) {
    __shared__ double rr[64], rz[64], beta[64], red[256];
    int running = 0;
    for (int k = 0; k < n; ++k) running |= cs[k].done == 0;
    if (running) {
        sums_by_rhs(part, blocks, n, red, rr);
        sums_by_rhs(part + blocks * n, blocks, n, red, rz);
    }
    if (threadIdx.x < n) {
        const int j = threadIdx.x;
        CgState s = cs[j];
        beta[j] = 0.0;
        if (!s.done) {
            s.it += 1;
            if (!(std::isfinite(rr[j]) && std::isfinite(rz[j]))) s.done = CG_NONFINITE;
            else if (rr[j] <= s.tol2) s.done = CG_CONVERGED;
            else if (s.it >= s.maxit) s.done = CG_MAXIT;
            beta[j] = rz[j] / s.rz;
            s.rz = rz[j];
        }
        rr[j] = s.done ? 1.0 : 0.0;   // (read: ended)
        if (blockIdx.x == 0) next[j] = s;
    }
    __syncthreads();
    const int per = 256 / n, j = threadIdx.x % n, q = threadIdx.x / n;
    const int64_t k = (int64_t)blockIdx.x * per + q;
    if (q < per && k < d && rr[j] == 0.0) P[k * G + j] = dinv[k] * R[k * n + j] + beta[j] * P[k * G + j];
}

// z[j][k] = X[k][j]
__global__ void k_sym_out(const double *__restrict__ X, int64_t d, int n, double *__restrict__ z) {
    const int64_t t = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (t >= d * n) return;
    z[t] = X[(t % d) * n + t / d];
}

// ---------------------------------------------------------------------------
// host side
// ---------------------------------------------------------------------------
SymCgPlan symcg_plan(int64_t d, int n) {
    SymCgPlan p{};
    // Where reading every element is the faster way (us an iteration, full /
    // triangle): one right-hand side d = 3500 33 / 35, 4256 47 / 39, 8836 135 /
    // 86; two d = 2048 32 / 31, 2834 49 / 32, 8836 259 / 96; 12 d = 2048 39 /
    // 42, 2834 54 / 46, 8836 285 / 143; 24 d = 2834 68 / 63, 8836 / 276; 40 d =
    // 8836 490 / 863 (four times 16 columns of accumulators spill).
    if (n < 1 || n > SYM_RHS || d < (n == 1 ? 4000 : 2400)) return p;
    p.G = n <= 2 ? n : (n <= 16 ? 16 : 32);
    // Larger blocks write fewer slots, smaller ones fill the chip sooner (us an
    // iteration, 2 / 4 tiles a side): one or two right-hand sides d = 3500 36 /
    // 43, 4256 49 / 45; 12 d = 7000 97 / 107, 8836 about equal; 24 d = 5000 109
    // / 121, 5661 133 / 130.
    p.tb = d >= (n <= 2 ? 4000 : (n <= 16 ? 8192 : 5600)) ? 4 : 2;
    const int64_t nt = (d + TS - 1) / TS, nb = (nt + p.tb - 1) / p.tb;
    p.units = nb * (nb + 1) / 2;
    p.slots = (int)(nb + 1);
    const int per = 256 / n;   // rows of an update block (they cover the padded rows of P too)
    p.blocks = (nt * TS + per - 1) / per;
    int64_t at = 0;
    auto take = [&](int64_t len) {
        const int64_t o = at;
        at += (len + 1) & ~(int64_t)1;
        return o;
    };
    p.oP = take(nt * TS * p.G);
    p.oR = take(d * n);
    p.oX = take(d * n);
    p.oD = take(d);
    p.oY = take(p.slots * d * n);
    p.oH = take(p.units * n);
    p.oS = take(p.blocks * n * 2);
    p.oC = take((int64_t)(2 * n * sizeof(CgState) + sizeof(int) + 7) / 8);
    if (n == 1 && at > SYM_ONE_DOUBLES) return SymCgPlan{};
    p.doubles = at;
    return p;
}

hipError_t launch_symcg_setup(const SymCgPlan &p, const double *H, const double *b, int64_t d, int n, int jacobi,
                              double rtol, int maxit, double *ws, hipStream_t st) {
    CgState *cs = (CgState *)(ws + p.oC);
    int *flag = (int *)(cs + 2 * n);
    const unsigned nt = (unsigned)((d + TS - 1) / TS);
    hipLaunchKernelGGL(k_sym_setup, dim3((unsigned)p.blocks), dim3(256), 0, st, H, b, d, (int64_t)nt * TS, n, p.G, jacobi,
                       ws + p.oX, ws + p.oR, ws + p.oD, ws + p.oP, ws + p.oS);
    hipLaunchKernelGGL(k_sym_init, dim3(1), dim3(256), 0, st, ws + p.oS, p.blocks, n, rtol, maxit, cs,
                       flag);
    hipLaunchKernelGGL(k_sym_check, dim3(nt, nt), dim3(256), 0, st, H, d, flag);
    return hipGetLastError();
}

hipError_t launch_symcg_iteration(const SymCgPlan &p, const double *H, int64_t d, int n, int it, double *ws,
                                  hipStream_t st) {
    // the state alternates between its two copies
    CgState *cs = (CgState *)(ws + p.oC) + (it & 1) * n, *next = (CgState *)(ws + p.oC) + (1 - (it & 1)) * n;
    const dim3 g((unsigned)p.units), b(256);
    double *P = ws + p.oP, *Y = ws + p.oY, *ph = ws + p.oH;
    const int rev = it & 1;
#define SYM_MV(NRT, TB)                                                                                          \
    hipLaunchKernelGGL((k_sym_matvec<NRT, TB>), g, b, sizeof(double) * TS * (TL + 2 * p.G), st, H, P, Y, ph, d, n,  \
                       rev, cs)
#define SYM_FEW(NV, TB) hipLaunchKernelGGL((k_sym_matvec_few<NV, TB>), g, b, 0, st, H, P, Y, ph, d, rev, cs)
    if (n == 1) {
        if (p.tb == 4) SYM_FEW(1, 4);
        else SYM_FEW(1, 2);
    } else if (n == 2) {
        if (p.tb == 4) SYM_FEW(2, 4);
        else SYM_FEW(2, 2);
    } else if (p.tb == 4) {
        if (p.G == 16) SYM_MV(1, 4);
        else SYM_MV(2, 4);
    } else {
        if (p.G == 16) SYM_MV(1, 2);
        else SYM_MV(2, 2);
    }
#undef SYM_MV
#undef SYM_FEW
    hipLaunchKernelGGL(k_sym_update, dim3((unsigned)p.blocks), b, 0, st, Y, ph, p.units, p.slots, P, ws + p.oD, d, n,
                       p.G, ws + p.oX, ws + p.oR, ws + p.oS, cs);
    hipLaunchKernelGGL(k_sym_direction, dim3((unsigned)p.blocks), b, 0, st, ws + p.oS, p.blocks, ws + p.oR,
                       ws + p.oD, d, n, p.G, P, cs, next);
    return hipGetLastError();
}

hipError_t launch_symcg_out(const SymCgPlan &p, const double *ws, int64_t d, int n, double *z, hipStream_t st) {
    hipLaunchKernelGGL(k_sym_out, dim3((unsigned)((d * n + 255) / 256)), dim3(256), 0, st, ws + p.oX, d, n, z);
    return hipGetLastError();
}

}  // namespace vmcx
