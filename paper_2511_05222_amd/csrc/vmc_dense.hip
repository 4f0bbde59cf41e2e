// vmc_dense.hip -- per-walker dense part of one measurement (gfx950).
//
// One block of four wavefronts per walker (eight from 49 orbitals on where both
// inverses are held).
//   phase A  waves 0 and 1: the inverse K of the up and down Slater blocks by
//            in-register Gauss-Jordan (FP64, partial pivoting), log|det|; or,
//            after a sweep, the sweep's inverse of the block followed by one
//            FP64 Newton step K + K (I - A K) on MFMA (then without log|det|);
//            every wave: Jastrow gradient g_e, Laplacian and value, e-e and
//            e-n potentials, each electron pair evaluated once (in rounds,
//            the partner's gradient share gathered per wavefront) and
//            combined in a fixed order.
//   phase B  per spin block, one wavefront per electron row: the determinant
//            gradient b_e = sum_i K[i][e] grad phi_i(r_e), lap D/D likewise,
//            and (with the adjoint) X[e][i] = lap phi_i + 2 g_e . grad phi_i;
//            then on 16x16x4 FP64 MFMA T = X K and
//            Abar = 1/2 (K X K)^T = 1/2 T^T K^T, written with K~[e][i] = K[i][e].
//            Abar is the sensitivity of E_L to the orbital values, so its
//            largest magnitude is the key by which the mixed path picks the
//            walkers it measures again in FP64 (formed, not stored, when
//            only that key is wanted).
//   phase C  block sums: E_L, ln|Psi| = log|det up| + log|det dn| + J.
// K, X and T stay FP64; K~ and Abar are stored in the arithmetic type T.
//
// Bound: the latency of a walker's chain of phases (barriers, loads of the MO
// rows, FP64 products): at 37 orbitals the matrix cores are busy 27 % of the
// cycles and 0.11 other vector instructions issue a cycle (2.6 cycles each as
// integer, 4.6 as FP64 ones).  Hence small blocks, as many on a CU as fit: from 33 orbitals on,
// after a sweep, one inverse at a time is held and loaded by the whole block,
// three walkers a CU instead of two (32768 walkers of 47 orbitals FP32 3.39 ->
// 2.76 ms, 16384 FP64 1.90 -> 1.61).  Blocks of six or eight wavefronts gained
// nothing there (4.6 and 3.3 ms: six do not pair up on the four SIMDs, eight
// spill).  The pairs of 26 electrons use all wavefronts (groups of 32 lanes),
// and a row's four sums over the orbitals halve the values a lane holds (13
// orbitals, 16384 walkers FP64 335 -> 276 us).
#include <cfloat>

#include "vmc_mfma.hpp"
#include "vmc_pipeline.hpp"
#include "vmc_regs.hpp"

namespace vmcx {

// The maximum / sum of v over a block of NW wavefronts, in a fixed order.
template <int NW>
__device__ inline double block_max(double v, double *red) {
#pragma unroll
    for (int off = 32; off > 0; off >>= 1) v = fmax(v, __shfl_xor(v, off, 64));
    const int lane = threadIdx.x & 63, wid = threadIdx.x >> 6;
    __syncthreads();
    if (lane == 0) red[wid] = v;
    __syncthreads();
    v = red[0];
#pragma unroll
    for (int q = 1; q < NW; ++q) v = fmax(v, red[q]);
    return v;
}

template <int NW>
__device__ inline double block_sum(double v, double *red) {
    v = wave_sum_dpp(v);
    const int lane = threadIdx.x & 63, wid = threadIdx.x >> 6;
    __syncthreads();
    if (lane == 0) red[wid] = v;
    __syncthreads();
    v = red[0];
#pragma unroll
    for (int q = 1; q < NW; ++q) v += red[q];
    return v;
}

// STATE: the spin blocks' inverses come from the sweep (mb.kst) unless stale.
// From 33 orbitals on only one is then held at a time, so that three blocks
// (two from 49 orbitals on) fit on a CU; otherwise wavefronts 0 and 1 load or form
// both at the start.
template <typename T, int KN, bool STATE>
__global__ __launch_bounds__(64 * dense_waves(KN, STATE)) __attribute__((amdgpu_waves_per_eu(STATE && KN == 48 ? 3 : 2)))
void k_dense(SysDev S, const double *__restrict__ R, MeasBufs<T> mb, WalkerOut out, int *status, DenseLayout L) {
    constexpr int NW = dense_waves(KN, STATE), NT = 64 * NW;   // wavefronts, threads
    constexpr int GL = dense_pair_lanes(KN), NG = NT / GL, NTAB = NG > NW ? NG : NW;
    typedef Mfma<double> MF;
    constexpr int RTS = KN / 16;                    // 16-row tiles of a spin block
    constexpr int TPW = (RTS * RTS + NW - 1) / NW;  // output tiles per wavefront
    constexpr bool BOTH = !(STATE && KN >= 48);     // both inverses held
    extern __shared__ __align__(16) unsigned char smem[];
    const int w = blockIdx.x;
    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int N = S.N, nu = S.n_up, nd = S.n_dn, n = S.n_occ, A = S.A;
    const int ldk = L.ldk;
    double *p = (double *)(smem + L.off_p);      // [N][3]
    double *g = (double *)(smem + L.off_g);      // [N][3] Jastrow gradient
    int *perm = (int *)(smem + L.off_perm);      // [2][64]
    double *red = (double *)(smem + L.off_red);  // [24]
    double *Xs = (double *)(smem + L.off_x);     // [KN][ldk]     X, then T
    double *Ks = (double *)(smem + L.off_k);     // [BOTH ? 2 : 1][KN][ldk]  K[i][e]
    const T *ph = mb.phi + (size_t)w * N * 5 * n;
    for (int i = tid; i < 3 * N; i += NT) p[i] = mb.pos[(size_t)w * N * 3 + i];
    __syncthreads();
    double el_part = 0.0, j_part = 0.0;
    bool bad = false;
    // The inverse of spin block b from its MO matrix by one wavefront, and
    // log|det| into red[4 + b].
    auto invert = [&](int b, double *K) {
        const int off = b ? nu : 0, nb = b ? nd : nu;
        int *pm = perm + 64 * b;
        double la = 0.0;
        // B = A^T of the block in the layout of gj_regs (clamped,
        // unconditional loads: a guarded load per register would be issued
        // and waited for one at a time)
        constexpr int CC = KN / 4;
        int lz = lane;
        asm volatile("" : "+v"(lz));
        const int m = lz & 15, g = lz >> 4;
        T av[RTS * CC];
#pragma unroll
        for (int q = 0; q < CC; ++q)
#pragma unroll
            for (int s = 0; s < RTS; ++s)
                av[s * CC + q] = ph[(size_t)(off + min(4 * q + g, nb - 1)) * 5 * n + min(m + 16 * s, nb - 1)];
        double Br[RTS * CC];
        double mx = 0.0;
#pragma unroll
        for (int s = 0; s < RTS; ++s)
#pragma unroll
            for (int q = 0; q < CC; ++q) {
                const int c = m + 16 * s, k = 4 * q + g;
                const bool in = c < nb && k < nb;
                const double v = in ? (double)av[s * CC + q] : (c == k ? 1.0 : 0.0);   // identity padding
                Br[s * CC + q] = v;
                mx = fmax(mx, in ? fabs(v) : 0.0);
            }
        int sg[RTS];
        gj_regs<KN, true>(Br, sg, bad, la, gj_tol(mx), K);   // (K's place in LDS is still free)
        // natural layout: row p_k holds column k, its column j orbital p_j
        if (g == 0)
#pragma unroll
            for (int s = 0; s < RTS; ++s) pm[sg[s]] = m + 16 * s;
        wave_sync_s();
#pragma unroll
        for (int q = 0; q < CC; ++q) {
            const int row = pm[4 * q + g] * ldk;
#pragma unroll
            for (int s = 0; s < RTS; ++s) K[row + sg[s]] = Br[s * CC + q];
        }
        if (lane == 0) red[4 + b] = la;
    };
    if (BOTH && wave < 2) {
        double *K = Ks + (size_t)wave * KN * ldk;
        if (STATE && mb.kstale[2 * w + wave] == 0) {
            // the sweep's inverse, in its register layout: lane p_k holds
            // column k with register j = orbital p_j
            int *pm = perm + 64 * wave;
            const T *kk = mb.kst + ((size_t)w * 2 + wave) * KN * KN + min(lane, KN - 1);
            T kr[KN];
#pragma unroll
            for (int r = 0; r < KN; ++r) kr[r] = kk[r * KN];
            const int sig = (int)mb.ksig[((size_t)w * 2 + wave) * KN + min(lane, KN - 1)];
            if (lane < KN) pm[sig] = lane;
            wave_sync_s();
            if (lane < KN)
#pragma unroll
                for (int j = 0; j < KN; ++j) K[pm[j] * ldk + sig] = (double)kr[j];
        } else {
            invert(wave, K);
        }
    }
    // Jastrow and potential, each electron pair once.  Round s pairs electron
    // e with k = (e + s) mod N; rounds 1 .. N/2 cover every pair once (in
    // round N/2 of an even N only e < N/2 takes part).  Groups of GL threads
    // (GL >= N), one electron each, share the rounds.  The pair's gradient
    // term f (r_e - r_k) is odd under exchange, bit for bit: e keeps it, and
    // k's share is gathered in a table of the wavefront (or of the group: all
    // of a table's lanes are in the same round, so their slots differ; reads
    // and writes in program order).  The even terms (Laplacian, potential, J)
    // enter the block sums once per pair with weight 2 relative to the
    // per-electron form.  The tables share their place with X, which comes
    // later.
    double *jp = Xs;              // [NG][N][3] own gradient partials
    double *bw = jp + NG * 3 * N; // [NTAB][N][3] partners' gradient partials
    {
        const int h = tid / GL, e = tid % GL;
        double *bme = bw + (size_t)(GL < 64 ? h : wave) * 3 * N;
        for (int i = GL < 64 ? e : lane; i < 3 * N; i += GL < 64 ? GL : 64) bme[i] = 0.0;
        wave_sync_s();
        const int per = (N / 2 + NG - 1) / NG, sb = 1 + h * per, se = min(N / 2, sb + per - 1);
        if (e < N) {
            const double x = p[3 * e], y = p[3 * e + 1], z = p[3 * e + 2];
            double gx = 0.0, gy = 0.0, gz = 0.0;
            for (int s = sb; s <= se; ++s) {
                if (2 * s == N && e >= s) break;
                int k = e + s;
                if (k >= N) k -= N;
                const double dx = x - p[3 * k], dy = y - p[3 * k + 1], dz = z - p[3 * k + 2];
                const double d2 = dx * dx + dy * dy + dz * dz;
                const double ir = rsqrt_nr(d2), r = d2 * ir;
                double u, u1, u2;
                if (S.ee_form == 1) {
                    const double ex = exp(-S.ee_F * r);
                    u1 = S.ee_a * ex;
                    u2 = -S.ee_F * u1;
                    u = S.ee_a * (1.0 - ex) / S.ee_F;
                } else {
                    const double q = rcp_nr(1.0 + S.ee_F * r);
                    u1 = S.ee_a * q * q;
                    u2 = -2.0 * S.ee_F * u1 * q;
                    u = S.ee_a * r * q;
                }
                const double f = u1 * ir;
                const double tx = f * dx, ty = f * dy, tz = f * dz;
                gx += tx;
                gy += ty;
                gz += tz;
                bme[3 * k] -= tx;
                bme[3 * k + 1] -= ty;
                bme[3 * k + 2] -= tz;
                el_part += ir - (u2 + 2.0 * f);
                j_part += u;
                // the next round's partner slot of lane e - 1 is this round's
                // of lane e: keep the rounds' LDS accesses in order
                wave_sync_s();
            }
            for (int a = h; a < A; a += NG) {
                const double ax = x - R[3 * a], ay = y - R[3 * a + 1], az = z - R[3 * a + 2];
                el_part -= S.Z[a] * rsqrt_nr(ax * ax + ay * ay + az * az);
            }
            double *o = jp + 3 * ((size_t)h * N + e);
            o[0] = gx;
            o[1] = gy;
            o[2] = gz;
        }
    }
    __syncthreads();
    for (int e = tid; e < N; e += NT) {
        double gq[3];
#pragma unroll
        for (int c = 0; c < 3; ++c) {
            double own = 0.0, others = 0.0;
#pragma unroll
            for (int q = 0; q < NG; ++q) own += jp[3 * (q * N + e) + c];
#pragma unroll
            for (int q = 0; q < NTAB; ++q) others += bw[3 * (q * N + e) + c];
            gq[c] = own + others;
        }
        if (mb.jg) {
            // one-/three-body terms: gradient into the total, Laplacian
            const double *jg = mb.jg + ((size_t)w * N + e) * 4;
#pragma unroll
            for (int c = 0; c < 3; ++c) gq[c] += jg[c];
            el_part += -0.5 * jg[3];
        }
        g[3 * e] = gq[0];
        g[3 * e + 1] = gq[1];
        g[3 * e + 2] = gq[2];
        el_part += -0.5 * (gq[0] * gq[0] + gq[1] * gq[1] + gq[2] * gq[2]);
    }
    __syncthreads();
    // (a block that starts from the sweep's inverse leaves ln|det| unknown)
    const bool have_ld = !STATE || (mb.kstale[2 * w] != 0 && mb.kstale[2 * w + 1] != 0);
    const bool full = mb.ktil != nullptr;
    // Abar is also formed, not stored, when it decides the FP64 re-measurement
    const bool need_abar = full || mb.promote_key != nullptr;
    double abar_max = 0.0;
    double *gb = mb.gb + (size_t)w * N * 6;
#pragma unroll 1
    for (int b = 0; b < 2; ++b) {
        const int nb = b ? nd : nu, off = b ? nu : 0;
        // (opaque here: otherwise every index made of them is kept in a
        // register of its own across the spin blocks)
        int tid = threadIdx.x;
        asm volatile("" : "+v"(tid));
        const int lane = tid & 63, ml = lane & 15, kg = lane >> 4;
        double *K = Ks + (BOTH ? (size_t)b * KN * ldk : (size_t)0);
        if constexpr (STATE) {
            if (mb.kstale[2 * w + b] != 0) {
                if constexpr (!BOTH) {
                    if (wave == 0) invert(b, K);
                    __syncthreads();
                }
            } else {
                // one FP64 Newton step K <- K + K (I - A K) on the matrix
                // cores (quadratic in the drift)
                // (all of this thread's loads first: one latency, not one per element)
                constexpr int PER = (KN * KN + NT - 1) / NT;
                T av[PER], kv[PER];
                const T *kk = mb.kst + ((size_t)w * 2 + b) * KN * KN;
#pragma unroll
                for (int q = 0; q < PER; ++q) {
                    const int idx = min(tid + NT * q, KN * KN - 1);
                    const int e = idx / KN, i = idx - (idx / KN) * KN;
                    if (!BOTH) kv[q] = kk[idx];
                    av[q] = ph[(size_t)(off + min(e, nb - 1)) * 5 * n + min(i, nb - 1)];
                }
                // the sweep's inverse, in its register layout: lane p_k holds
                // column k with register j = orbital p_j (row j, column lane)
                int *pm = perm, *sg = perm + 64;
                if (!BOTH) {
                    if (tid < KN) {
                        const int sig = (int)mb.ksig[((size_t)w * 2 + b) * KN + tid];
                        sg[tid] = sig;
                        pm[sig] = tid;
                    }
                    __syncthreads();
                }
#pragma unroll
                for (int q = 0; q < PER; ++q) {
                    const int idx = tid + NT * q;
                    if (idx < KN * KN) {
                        const int e = idx / KN, i = idx - (idx / KN) * KN;
                        const bool in = e < nb && i < nb;
                        Xs[e * ldk + i] = in ? (double)av[q] : (e == i ? 1.0 : 0.0);
                        if (!BOTH) K[pm[e] * ldk + sg[i]] = (double)kv[q];
                    }
                }
                __syncthreads();
                MF::acc_t tacc[TPW];
#pragma unroll
                for (int q = 0; q < TPW; ++q) {
                    const int t = wave + NW * q;
                    tacc[q] = MF::zero();
                    if (t < RTS * RTS) {
                        const int rt = t / RTS, ct = t - (t / RTS) * RTS;
                        const double *xa = Xs + (16 * rt + ml) * ldk + kg;
                        const double *kb = K + kg * ldk + 16 * ct + ml;
#pragma unroll
                        for (int ks = 0; ks < KN / 4; ++ks) tacc[q] = MF::fma(xa[4 * ks], kb[4 * ks * ldk], tacc[q]);
                    }
                }
                __syncthreads();   // A is read: R = I - A K replaces it
#pragma unroll
                for (int q = 0; q < TPW; ++q) {
                    const int t = wave + NW * q;
                    if (t < RTS * RTS) {
                        const int rt = t / RTS, ct = t - (t / RTS) * RTS;
#pragma unroll
                        for (int v = 0; v < 4; ++v) {
                            const int r = 16 * rt + MF::row(lane, v), c = 16 * ct + ml;
                            Xs[r * ldk + c] = (r == c ? 1.0 : 0.0) - tacc[q][v];
                        }
                    }
                }
                __syncthreads();
#pragma unroll
                for (int q = 0; q < TPW; ++q) {
                    const int t = wave + NW * q;
                    tacc[q] = MF::zero();
                    if (t < RTS * RTS) {
                        const int rt = t / RTS, ct = t - (t / RTS) * RTS;
                        const double *ka = K + (16 * rt + ml) * ldk + kg;
                        const double *rb = Xs + kg * ldk + 16 * ct + ml;
#pragma unroll
                        for (int ks = 0; ks < KN / 4; ++ks) tacc[q] = MF::fma(ka[4 * ks], rb[4 * ks * ldk], tacc[q]);
                    }
                }
                __syncthreads();   // K is read: add the correction
#pragma unroll
                for (int q = 0; q < TPW; ++q) {
                    const int t = wave + NW * q;
                    if (t < RTS * RTS) {
                        const int rt = t / RTS, ct = t - (t / RTS) * RTS;
#pragma unroll
                        for (int v = 0; v < 4; ++v) K[(16 * rt + MF::row(lane, v)) * ldk + 16 * ct + ml] += tacc[q][v];
                    }
                }
                __syncthreads();
            }
        }
        // one wavefront per electron row j of the block (rows nb..KN-1:
        // zeros).  The wavefront's gradient and Laplacian rows are loaded
        // together first (clamped, unconditional loads), so that their
        // latency is paid once rather than once per row.
        constexpr int JPW = KN / NW;
        T rG[JPW][4];
        const int lc = min(lane, n - 1);
#pragma unroll
        for (int q = 0; q < JPW; ++q) {
            const T *row = ph + (size_t)(off + min(wave + NW * q, nb - 1)) * 5 * n + lc;
#pragma unroll
            for (int c = 0; c < 4; ++c) rG[q][c] = row[(c + 1) * n];
        }
#pragma unroll
        for (int q = 0; q < JPW; ++q) {
            const int j = wave + NW * q;
            if (j >= nb) {
                if (lane < KN) Xs[j * ldk + lane] = 0.0;
                continue;
            }
            const int e = off + j;
            const double gx = g[3 * e], gy = g[3 * e + 1], gz = g[3 * e + 2];
            double bx = 0.0, by = 0.0, bz = 0.0, lp = 0.0, xv = 0.0;
            if (lane < n) {
                const double Gx = (double)rG[q][0], Gy = (double)rG[q][1], Gz = (double)rG[q][2],
                             Lp = (double)rG[q][3];
                xv = Lp + 2.0 * (gx * Gx + gy * Gy + gz * Gz);
                if (lane < nb) {
                    const double kk = K[lane * ldk + j];
                    bx = kk * Gx;
                    by = kk * Gy;
                    bz = kk * Gz;
                    lp = kk * Lp;
                }
            }
            if (lane < KN) Xs[j * ldk + lane] = xv;
            // lane m of the first four: bx, by, bz or lp
            const double t4[4] = {bx, by, bz, lp};
            const double sum = wave_sum4(t4, lane);
            const double gm = lane == 0 ? gx : (lane == 1 ? gy : gz);
            if (lane < 3) {
                gb[6 * e + lane] = gm;
                gb[6 * e + 3 + lane] = sum;
            }
            if (lane < 4) el_part -= lane == 3 ? 0.5 * sum : sum * gm;
        }
        if (!need_abar) continue;
        __syncthreads();
        // T = X K  (rows e', columns e)
        MF::acc_t tacc[TPW];
#pragma unroll
        for (int q = 0; q < TPW; ++q) {
            const int t = wave + NW * q;
            tacc[q] = MF::zero();
            if (t < RTS * RTS) {
                const int rt = t / RTS, ct = t - (t / RTS) * RTS;
                const double *xa = Xs + (16 * rt + ml) * ldk + kg;
                const double *kb = K + kg * ldk + 16 * ct + ml;
#pragma unroll
                for (int ks = 0; ks < KN / 4; ++ks) tacc[q] = MF::fma(xa[4 * ks], kb[4 * ks * ldk], tacc[q]);
            }
        }
        __syncthreads();   // every read of X is done: T replaces it
#pragma unroll
        for (int q = 0; q < TPW; ++q) {
            const int t = wave + NW * q;
            if (t < RTS * RTS) {
                const int rt = t / RTS, ct = t - (t / RTS) * RTS;
#pragma unroll
                for (int v = 0; v < 4; ++v) Xs[(16 * rt + MF::row(lane, v)) * ldk + 16 * ct + ml] = tacc[q][v];
            }
        }
        __syncthreads();
        // Abar[e][i] = 1/2 sum_e' T[e'][e] K[i][e']
        T *abw = full ? mb.abar + ((size_t)w * N + off) * n : nullptr;
        T *ktw = full ? mb.ktil + ((size_t)w * N + off) * n : nullptr;
#pragma unroll
        for (int q = 0; q < TPW; ++q) {
            const int t = wave + NW * q;
            if (t < RTS * RTS) {
                const int rt = t / RTS, ct = t - (t / RTS) * RTS;
                const double *ta = Xs + kg * ldk + 16 * rt + ml;
                const double *kb = K + (16 * ct + ml) * ldk + kg;
                MF::acc_t acc = MF::zero();
#pragma unroll
                for (int ks = 0; ks < KN / 4; ++ks) acc = MF::fma(ta[4 * ks * ldk], kb[4 * ks], acc);
                const int i = 16 * ct + ml;
#pragma unroll
                for (int v = 0; v < 4; ++v) {
                    const int e = 16 * rt + MF::row(lane, v);
                    if (e < nb && i < n) {
                        abar_max = fmax(abar_max, fabs(0.5 * acc[v]));
                        if (full) {
                            abw[(size_t)e * n + i] = (T)(0.5 * acc[v]);
                            ktw[(size_t)e * n + i] = (T)K[i * ldk + e];
                        }
                    }
                }
            }
        }
        __syncthreads();   // the next block rewrites X
    }
    if (mb.promote_key) abar_max = block_max<NW>(abar_max, red + 16);
    // nuclear repulsion: the A^2 ordered pairs spread over the block
    double vnn = 0.0;
    for (int q = tid; q < A * A; q += NT) {
        const int a = q / A, c = q - (q / A) * A;
        if (c <= a) continue;
        const double dx = R[3 * a] - R[3 * c], dy = R[3 * a + 1] - R[3 * c + 1], dz = R[3 * a + 2] - R[3 * c + 2];
        vnn += S.Z[a] * S.Z[c] / sqrt(dx * dx + dy * dy + dz * dz);
    }
    const double logdet = have_ld ? red[4] + red[5] : 0.0;   // (before the sums below take red)
    const double EL = block_sum<NW>(el_part + vnn, red);
    const double J = block_sum<NW>(j_part, red) + (mb.ju ? mb.ju[w] : 0.0);
    const int anybad = __syncthreads_or(bad ? 1 : 0);
    if (tid == 0) {
        if (mb.promote_key) mb.promote_key[w] = abar_max <= DBL_MAX ? abar_max : __builtin_inf();
        if (out.EL) out.EL[w] = EL;
        if (out.lnpsi) out.lnpsi[w] = have_ld ? logdet + J : __builtin_nan("");
        if (anybad) atomicOr(status, STATUS_SINGULAR);
        if (!isfinite(EL) || !isfinite(J) || (have_ld && !isfinite(logdet))) atomicOr(status, STATUS_NONFINITE);
    }
}

template <typename T>
hipError_t launch_dense(const SysDev &S, const double *R, const MeasBufs<T> &mb, const WalkerOut &out, int *status,
                        const DenseLayout &L, int W, hipStream_t st) {
    const int kn = sweep_kn(S.n_occ);
    const bool state = mb.kst != nullptr;
    // Where one inverse is held at a time, the second block's replaces the
    // first's behind the barriers of the Abar part only: a block without that
    // part would overwrite an inverse that other wavefronts still read.
    if (state && kn >= 48 && !mb.ktil && !mb.promote_key) return hipErrorInvalidValue;
    const dim3 g((unsigned)W), b((unsigned)(64 * dense_waves(kn, state)));
#define DENSE(KN)                                                                                                     \
    case KN:                                                                                                          \
        if (state)                                                                                                    \
            hipLaunchKernelGGL((k_dense<T, KN, true>), g, b, kn >= 48 ? L.bytes_one : L.bytes, st, S, R, mb, out, status, L);            \
        else                                                                                                          \
            hipLaunchKernelGGL((k_dense<T, KN, false>), g, b, L.bytes, st, S, R, mb, out, status, L);                 \
        break
    switch (kn) {
        DENSE(16);
        DENSE(32);
        DENSE(48);
        DENSE(64);
    }
#undef DENSE
    return hipGetLastError();
}

template <typename T>
hipError_t configure_dense(size_t lds) {
    const void *f[8] = {(const void *)k_dense<T, 16, false>, (const void *)k_dense<T, 32, false>,
                        (const void *)k_dense<T, 48, false>, (const void *)k_dense<T, 64, false>,
                        (const void *)k_dense<T, 16, true>,  (const void *)k_dense<T, 32, true>,
                        (const void *)k_dense<T, 48, true>,  (const void *)k_dense<T, 64, true>};
    for (const void *g : f) {
        const hipError_t e = hipFuncSetAttribute(g, hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds);
        if (e != hipSuccess) return e;
    }
    return hipSuccess;
}

template hipError_t launch_dense<double>(const SysDev &, const double *, const MeasBufs<double> &, const WalkerOut &,
                                         int *, const DenseLayout &, int, hipStream_t);
template hipError_t configure_dense<double>(size_t);

template hipError_t launch_dense<float>(const SysDev &, const double *, const MeasBufs<float> &, const WalkerOut &,
                                        int *, const DenseLayout &, int, hipStream_t);
template hipError_t configure_dense<float>(size_t);

}  // namespace vmcx
