// vmc_adjoint.hip -- AO-space adjoint of one measurement on the matrix cores.
//
// One block per walker; the block's wavefronts take 16-AO sub-tiles in turn.
// For a sub-tile (AOs mu) and 16-electron row tile (electrons e):
//   kappa[e][mu] = sum_i K~[e][i] C[mu][i],  a[e][mu] = sum_i Abar[e][i] C[mu][i]
// on 16x16x4 MFMA (A = K~ or Abar from LDS, B = C held in registers).  The
// accumulator of that product holds, in every lane, the (e, mu) pairs that
// the lane then evaluates (AO value, gradient, Hessian, grad-Laplacian):
//   t_k = a d_k psi - kappa (sum_d g_d d_k d_d psi + 1/2 d_k lap psi)
//   s_k = kappa d_k psi,   q = -g . grad psi - 1/2 lap psi
// and those per-lane values are exactly the A operand (rows mu, k = e) of the
// outer products
//   O[mu][i] = sum_e psi[e][mu] K~[e][i]
//   G[mu][i] = sum_e psi[e][mu] Abar[e][i] + q[e][mu] K~[e][i]
// whose B operand (K~, Abar rows e) comes from LDS.  Per AO the electron sums
// of t_k and s_k go to tao; per electron the AO sums of t_k (dE_L/dr_e, the
// determinant part) go to dedr_part, in a fixed order.
//
// Bound: issue (the matrix cores and the vector units of a SIMD take turns): at
// 47 orbitals, FP32, the matrix cores are busy 38 % of the cycles and 0.166
// other vector instructions issue a cycle (at 2.6 cycles 43 %); FP64 34 % and
// 0.100 (at 4.6 cycles 46 %), the rest latency that two wavefronts a SIMD do not
// hide.
//   FP64: an AO's lane used to form its shell's radial sums itself, each
// shell's 2.3 times over with exponents read from memory; now four or eight
// lanes a shell form them once (SHARED), in LDS until the AOs' lanes read them.
// With shorter algebra for t_k and one LDS update per sum (below): 235 AOs, 94
// electrons, 8192 walkers 3.87 -> 3.42 ms; 75 AOs, 26 electrons, 16384 walkers
// 1.17 -> 0.66 (there also from four wavefronts a block for 5 sub-tiles); H2 30
// -> 11 us.
//   FP32: radial sums are cheap and in registers; shared they cost more in
// LDS round trips than they save (6.50 against 6.08 ms, 235 AOs, 32768
// walkers).
#include "vmc_pipeline.hpp"
#include "vmc_mfma.hpp"
#include "vmc_regs.hpp"

namespace vmcx {

// The shell of one lane of the radial phase (FP64).
struct ShellLane {
    static constexpr int NP = 3;   // primitives held in registers
    double x, y, z, al[NP], cp[NP];
    int np, p0;
};

__device__ inline void shell_lane_load(const SysDev &S, const double *R, int s, ShellLane &L) {
    const int a = S.basis.shell_atom[s];
    L.x = R[3 * a];
    L.y = R[3 * a + 1];
    L.z = R[3 * a + 2];
    L.np = S.basis.shell_np[s];
    L.p0 = S.basis.shell_p0[s];
#pragma unroll
    for (int k = 0; k < ShellLane::NP; ++k) {
        const int p = L.p0 + max(min(k, L.np - 1), 0);
        L.al[k] = S.basis.prim_exp[p];
        L.cp[k] = k < L.np ? S.basis.prim_cp[p] : 0.0;   // padded primitives carry cp = 0
    }
}

// R0, u1, u2, u3 of ao_lane_radial for the lane's shell.
__device__ inline void shell_lane_radial(const ShellLane &L, const BasisDev &B, double rho, double *o) {
    double r0 = 0.0, r1 = 0.0, r2 = 0.0, r3 = 0.0;
    auto add = [&](double al, double cp) {
        const double e = cp * exp(-al * rho), al2 = al * al, al3 = al2 * al;
        r0 += e;
        r1 = fma(-al, e, r1);
        r2 = fma(al2, e, r2);
        r3 = fma(-al3, e, r3);
    };
#pragma unroll
    for (int k = 0; k < ShellLane::NP; ++k) add(L.al[k], L.cp[k]);
    for (int k = ShellLane::NP; k < L.np; ++k) add(B.prim_exp[L.p0 + k], B.prim_cp[L.p0 + k]);
    o[0] = r0;
    o[1] = 2.0 * r1;
    o[2] = 4.0 * r2;
    o[3] = 8.0 * r3;
}

// The lane's monomial P = eta x^a y^b z^c at (x, y, z): its gradient, its
// Hessian times g and its Laplacian.
template <typename T, int NPR>
__device__ inline void ao_lane_monomial(const AoLane<T, NPR> &L, T x, T y, T z, T gx, T gy, T gz, T &P, T *dP,
                                        T *HPg, T &lapP) {
    const T r[3] = {x, y, z};
    T f[3], f1[3];
#pragma unroll
    for (int q = 0; q < 3; ++q) {
        const T h = fma(L.c2[q], r[q], L.c1[q]);
        f[q] = fma(h, r[q], L.c0[q]);
        f1[q] = fma(L.c2[q], r[q], h);
    }
    const T fyz = f[1] * f[2], fxz = f[0] * f[2], fxy = f[0] * f[1];
    P = f[0] * fyz;
    dP[0] = f1[0] * fyz;
    dP[1] = f1[1] * fxz;
    dP[2] = f1[2] * fxy;
    const T Pxx = L.c22[0] * fyz, Pyy = L.c22[1] * fxz, Pzz = L.c22[2] * fxy;
    const T Pxy = f1[0] * f1[1] * f[2], Pxz = f1[0] * f1[2] * f[1], Pyz = f1[1] * f1[2] * f[0];
    lapP = Pxx + Pyy + Pzz;
    HPg[0] = fma(Pxx, gx, fma(Pxy, gy, Pxz * gz));
    HPg[1] = fma(Pxy, gx, fma(Pyy, gy, Pyz * gz));
    HPg[2] = fma(Pxz, gx, fma(Pyz, gy, Pzz * gz));
}

// Sums of 3 or 6 values over the 16 lanes of a DPP row, one value a lane, by
// halving what a lane holds at each step: lane m (of the row) returns the value
// row16_which<NV>(m).  The pairs added are those of row16_sum_last (neighbours,
// then twos, fours, eights).
template <int NV>
__device__ inline int row16_which(int m) {
    return NV == 3 ? ((m & 2) ? 2 : (m & 1)) : ((m & 4) ? 4 : (m & 2)) + (m & 1);
}
template <typename T>
__device__ inline T row16_sums(const T (&t)[3], int m) {
    const T q0 = add_xor<1>((m & 1) ? t[1] : t[0], (m & 1) ? t[0] : t[1]), q1 = add_xor<1>(t[2], t[2]);
    T u = add_xor<2>((m & 2) ? q1 : q0, (m & 2) ? q0 : q1);
    u = add_xor<4>(u, u);
    return add_xor<8>(u, u);
}
template <typename T>
__device__ inline T row16_sums(const T (&t)[6], int m) {
    T q[3], s[2];
#pragma unroll
    for (int p = 0; p < 3; ++p)
        q[p] = add_xor<1>((m & 1) ? t[2 * p + 1] : t[2 * p], (m & 1) ? t[2 * p] : t[2 * p + 1]);
    s[0] = add_xor<2>((m & 2) ? q[1] : q[0], (m & 2) ? q[0] : q[1]);
    s[1] = add_xor<2>(q[2], q[2]);
    const T u = add_xor<4>((m & 4) ? s[1] : s[0], (m & 4) ? s[0] : s[1]);
    return add_xor<8>(u, u);
}

template <typename T, int NT, bool SHARED>
__global__ __launch_bounds__(512) __attribute__((amdgpu_waves_per_eu(sizeof(T) == 4 ? (NT == 1 ? 4 : 3) : 2)))
void k_adjoint_mfma(SysDev S, const T *__restrict__ C, const double *__restrict__ R, MeasBufs<T> mb, WalkerOut out,
                    AdjLayout L) {
    typedef Mfma<T> MF;
    constexpr int KS = 4 * NT;        // k-steps over orbitals (4 per step)
    constexpr int NPR = SHARED ? 0 : (sizeof(T) == 4 ? 3 : 0);   // primitives an AO's lane holds
    typedef T V4 __attribute__((ext_vector_type(4), aligned(16)));
    extern __shared__ __align__(16) unsigned char smem[];
    const int w = blockIdx.x;
    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6), nw = blockDim.x >> 6;
    const int N = S.N, n = S.n_occ, M = S.M;
    const int ldk = L.ldk, RT = L.rt;
    T *Ks = (T *)(smem + L.off_k);    // [RT*16][ldk]  K~[e][i]
    T *As = (T *)(smem + L.off_a);    // [RT*16][ldk]  Abar[e][i]
    double *sp = (double *)(smem + L.off_p);    // [N][3]
    T *sg = (T *)(smem + L.off_g);              // [N][3] Jastrow gradient (arithmetic type)
    double *dpw = (double *)(smem + L.off_d);   // [nw][dst] per-wave dE_L/dr_e partials [N][3]
    const int dst = (3 * N + 1) & ~1;
    const T *ktw = mb.ktil + (size_t)w * N * n;
    const T *abw = mb.abar + (size_t)w * N * n;
    // K~ and Abar into LDS, eight elements per thread in flight (clamped,
    // unconditional loads; the padding is selected afterwards)
    for (int k0 = tid; k0 < RT * 16 * ldk; k0 += 8 * (int)blockDim.x) {
        T kv[8], av[8];
#pragma unroll
        for (int u = 0; u < 8; ++u) {
            const int k = k0 + u * (int)blockDim.x;
            const int e = min(k / ldk, N - 1), i = min(k - (k / ldk) * ldk, n - 1);
            kv[u] = ktw[(size_t)e * n + i];
            av[u] = abw[(size_t)e * n + i];
        }
#pragma unroll
        for (int u = 0; u < 8; ++u) {
            const int k = k0 + u * (int)blockDim.x;
            if (k < RT * 16 * ldk) {
                const int e = k / ldk, i = k - (k / ldk) * ldk;
                const bool on = e < N && i < n;
                Ks[k] = on ? kv[u] : T(0);
                As[k] = on ? av[u] : T(0);
            }
        }
    }
    for (int k = tid; k < 3 * N; k += blockDim.x) {
        sp[k] = mb.pos[(size_t)w * N * 3 + k];
        sg[k] = (T)mb.gb[(size_t)w * N * 6 + 6 * (k / 3) + (k - (k / 3) * 3)];
    }
    for (int k = tid; k < nw * dst; k += blockDim.x) dpw[k] = 0.0;
    __syncthreads();
    // One block of eight wavefronts a CU: the wavefronts left without a last
    // sub-tile differ from block to block (2.5 % at 15 sub-tiles; smaller
    // blocks, several a CU, lose by it).  The partials are kept by share: the
    // order of their sum is the same in every block.
    const int share = nw == 8 ? (wave + (w >> 3) + (w >> 8)) & 7 : wave;
    double *dw = dpw + share * dst;
    V4 *xr = (V4 *)(dpw + nw * dst) + wave * 8 * ADJ_XS;   // radial sums, [4 VU electrons][XS shells]
    const int ml = lane & 15, kg = lane >> 4;
    // Evaluations a turn, and the dE_L/dr sum this lane gets of a turn's: two
    // take fewer lane moves a sum, one fewer registers.  Two / one, 4096 walkers:
    // FP32 with 20, 32, 37 and 47 orbitals 200 / 203, 369 / 387, 539 / 552 and
    // 808 / 823 us, with 13 and 56 (both spill) 123 / 94 and 1318 / 1238; FP64
    // with 13 and 32 171 / 198 and 650 / 705, with 37, 47, 56 and 64 (all spill)
    // 1072 / 1025, 1770 / 1717, 2605 / 2400 and 3003 / 2700.
    constexpr int VU = sizeof(T) == 8 ? (NT <= 2 ? 2 : 1) : (NT == 2 || NT == 3 ? 2 : 1);
    const int dq = row16_which<3 * VU>(ml), de = MF::row(lane, dq / 3), dc = dq % 3;
    const bool dmine = VU == 2 ? (ml & 8) == 0 && (ml & 6) != 6 : ml < 3;
    // the electron (of 4 VU) and shell (of XS) of this lane in the radial phase
    constexpr int XS = 2 * ADJ_XS / VU;
    const int ri = lane % (4 * VU), rj = lane / (4 * VU), re = MF::row(16 * (ri / VU), ri % VU);
    const int n_sub = (M + 15) >> 4;
    for (int st = share; st < n_sub; st += nw) {
        const int mu = 16 * st + ml;
        const bool vm = mu < M;
        // this lane's AO: monomial (and primitives) in registers for the sub-tile
        AoLane<T, NPR> al;
        ao_lane_load<T, NPR>(S.basis, vm ? mu : M - 1, al);
        if (!vm) al.c0[0] = al.c1[0] = al.c2[0] = al.c22[0] = T(0);   // no AO: every component 0
        const int shell = S.basis.ao_shell[vm ? mu : M - 1], atom = S.basis.shell_atom[shell];
        const double Rx = R[3 * atom], Ry = R[3 * atom + 1], Rz = R[3 * atom + 2];
        // the sub-tile's shells, this lane's AO's among them
        const int s0 = ldc(S.basis.ao_shell + 16 * st), ns = ldc(S.basis.ao_shell + min(16 * st + 15, M - 1)) - s0 + 1;
        const int sj = shell - s0;
        ShellLane sl;
        if constexpr (SHARED) shell_lane_load(S, R, s0 + min(rj, ns - 1), sl);
        T cB[KS];
#pragma unroll
        for (int ks = 0; ks < KS; ++ks) {
            const int i = 4 * ks + kg;
            cB[ks] = (vm && i < n) ? C[(size_t)mu * n + i] : T(0);
        }
        typename MF::acc_t accO[NT], accG[NT];
#pragma unroll
        for (int it = 0; it < NT; ++it) accO[it] = accG[it] = MF::zero();
        // per-AO sums over this lane's 4 RT electrons in T, then over the
        // four row groups in FP64
        T tl[6] = {T(0), T(0), T(0), T(0), T(0), T(0)};
        for (int rt = 0; rt < RT; ++rt) {
            typename MF::acc_t kap = MF::zero(), aa = MF::zero();
            const T *kr = Ks + (16 * rt + ml) * ldk + kg;
            const T *ar = As + (16 * rt + ml) * ldk + kg;
#pragma unroll
            for (int ks = 0; ks < KS; ++ks) {
                kap = MF::fma(kr[4 * ks], cB[ks], kap);
                aa = MF::fma(ar[4 * ks], cB[ks], aa);
            }
            // One evaluation (e, mu) at a time (interleaved, several would be
            // live).  Every lane evaluates: past the last AO all
            // components are 0, past the last electron (position of electron
            // N - 1) kappa, a and the K~ / Abar rows are 0, so nothing of it
            // reaches a sum.
#pragma unroll 1
            for (int h = 0; h < 4; h += VU) {
                V4 rs[VU];
                if constexpr (SHARED) {
                    // radial sums of the sub-tile's shells, XS at a time, at the
                    // turn's electrons, then to the lanes of their AOs
                    const int ec = min(16 * rt + MF::row(0, h) + re, N - 1);
                    const double px = sp[3 * ec], py = sp[3 * ec + 1], pz = sp[3 * ec + 2];
                    for (int q = 0; q < ns; q += XS) {
                        if (ns > XS) shell_lane_load(S, R, s0 + min(q + rj, ns - 1), sl);
                        const double dx = px - sl.x, dy = py - sl.y, dz = pz - sl.z;
                        double o[4];
                        shell_lane_radial(sl, S.basis, dx * dx + dy * dy + dz * dz, o);
                        wave_sync_s();
                        if (rj < XS) xr[XS * ri + rj] = V4{o[0], o[1], o[2], o[3]};
                        wave_sync_s();
                        const V4 *r = xr + XS * VU * kg + max(0, min(sj - q, XS - 1));
#pragma unroll
                        for (int v = 0; v < VU; ++v) {
                            const V4 x = r[XS * v];
                            if (sj >= q) rs[v] = x;
                        }
                    }
                }
                T t[3 * VU];
#pragma unroll
                for (int v = 0; v < VU; ++v) {
                    const int e = 16 * rt + MF::row(lane, h) + MF::row(0, v), ec = min(e, N - 1);
                    const double dx = sp[3 * ec] - Rx, dy = sp[3 * ec + 1] - Ry, dz = sp[3 * ec + 2] - Rz;
                    const double rho_d = dx * dx + dy * dy + dz * dz;
                    const T x = (T)dx, y = (T)dy, z = (T)dz, rho = (T)rho_d;
                    T R0, u1, u2, u3;
                    if constexpr (SHARED) {
                        R0 = rs[v][0], u1 = rs[v][1], u2 = rs[v][2], u3 = rs[v][3];
                    } else {
                        ao_lane_radial<T, NPR>(al, S.basis, rho_d, R0, u1, u2, u3);
                    }
                    const T gx = sg[3 * ec], gy = sg[3 * ec + 1], gz = sg[3 * ec + 2];
                    const T kv = kap[v], av = aa[v], half = T(0.5);
                    T psi, q;
                    if constexpr (sizeof(T) == 8) {
                        // (95 FP64 operations where the 14 components and their
                        // products with g take 125)
                        T P, dP[3], HPg[3], lapP;
                        ao_lane_monomial<T, NPR>(al, x, y, z, gx, gy, gz, P, dP, HPg, lapP);
                        const T PR1 = P * u1, PR2 = P * u2, kR = kv * R0, kP = kv * PR1;
                        const T xg = fma(x, gx, fma(y, gy, z * gz)), Pg = fma(dP[0], gx, fma(dP[1], gy, dP[2] * gz));
                        // d_k psi = dP_k R + x_k 2 P R'
                        // (H g)_k = (HP g)_k R + dP_k xg 2 R' + x_k (Pg 2 R' + xg 4 P R'') + g_k 2 P R'
                        // d_k lap psi = x_k S1 + dP_k S2
                        const T A = fma(Pg, u1, xg * PR2);
                        const T S1 = fma(lapP, u1, fma(al.h820, PR2, rho * P * u3)), S2 = fma(al.h46, u1, rho * u2);
                        const T cP = fma(av, R0, -kv * fma(xg, u1, half * S2)), cD = fma(av, PR1, -kv * fma(half, S1, A));
                        const T r[3] = {x, y, z}, g[3] = {gx, gy, gz};
#pragma unroll
                        for (int c = 0; c < 3; ++c) {
                            const T tk = fma(cP, dP[c], fma(cD, r[c], -fma(kR, HPg[c], kP * g[c])));
                            t[3 * v + c] = tk;
                            tl[c] += tk;
                            tl[3 + c] = fma(kR, dP[c], fma(kP, r[c], tl[3 + c]));
                        }
                        psi = P * R0;
                        q = -fma(Pg, R0, xg * PR1) - half * fma(lapP, R0, fma(al.h46, PR1, rho * PR2));
                    } else {
                        T d[14];
                        ao_lane_components<T, NPR>(al, x, y, z, rho, R0, u1, u2, u3, d);
                        const T hgx = gx * d[5] + gy * d[6] + gz * d[7];
                        const T hgy = gx * d[6] + gy * d[8] + gz * d[9];
                        const T hgz = gx * d[7] + gy * d[9] + gz * d[10];
                        const T t6[6] = {av * d[1] - kv * (hgx + half * d[11]), av * d[2] - kv * (hgy + half * d[12]),
                                         av * d[3] - kv * (hgz + half * d[13]), kv * d[1], kv * d[2], kv * d[3]};
                        psi = d[0];
                        q = -(gx * d[1] + gy * d[2] + gz * d[3]) - half * d[4];
#pragma unroll
                        for (int c = 0; c < 6; ++c) tl[c] += t6[c];
#pragma unroll
                        for (int c = 0; c < 3; ++c) t[3 * v + c] = t6[c];
                    }
                    const T *kb = Ks + e * ldk + ml;
                    const T *ab = As + e * ldk + ml;
#pragma unroll
                    for (int it = 0; it < NT; ++it) {
                        const T bk = kb[16 * it], ba = ab[16 * it];
                        accO[it] = MF::fma(psi, bk, accO[it]);
                        accG[it] = MF::fma(psi, ba, accG[it]);
                        accG[it] = MF::fma(q, bk, accG[it]);
                    }
                    __builtin_amdgcn_sched_barrier(0);
                }
                // AO sums of t_k over the 16 lanes of a row group (a DPP row),
                // added to the electron's by one lane each
                const double dd = (double)row16_sums<T>(t, ml);
                const int e = 16 * rt + MF::row(0, h) + de;
                if (dmine && e < N) dw[3 * e + dc] += dd;
#pragma unroll
                for (int v = 0; v + VU < 4; ++v) kap[v] = kap[v + VU], aa[v] = aa[v + VU];
            }
        }
        // outer products of the walker for this sub-tile
#pragma unroll
        for (int v = 0; v < 4; ++v) {
            const int mr = 16 * st + MF::row(lane, v);
            if (mr >= M) continue;
#pragma unroll
            for (int it = 0; it < NT; ++it) {
                const int i = 16 * it + ml;
                if (i < n) {
                    const size_t o = ((size_t)w * M + mr) * n + i;
                    if (out.O) out.O[o] = (double)accO[it][v];
                    if (out.G) out.G[o] = (double)accG[it][v];
                    if (out.Of) out.Of[o] = (float)accO[it][v];
                    if (out.Gf) out.Gf[o] = (float)accG[it][v];
                }
            }
        }
        // electron sums per AO: add the four row groups
        double td[6];
#pragma unroll
        for (int c = 0; c < 6; ++c) {
            td[c] = (double)tl[c];
            td[c] += __shfl_xor(td[c], 16, 64);
            td[c] += __shfl_xor(td[c], 32, 64);
        }
        if (kg == 0 && vm)
#pragma unroll
            for (int c = 0; c < 6; ++c) mb.tao[((size_t)w * M + mu) * 6 + c] = td[c];
    }
    __syncthreads();
    // dE_L/dr_e (determinant part): the wavefronts' partials in a fixed order
    double *dpart = mb.dedr_part + (size_t)w * N * 3;
    for (int k = tid; k < 3 * N; k += blockDim.x) {
        double acc = 0.0;
        for (int q = 0; q < nw; ++q) acc += dpw[q * dst + k];
        dpart[k] = acc;
    }
}

template <typename T>
hipError_t launch_adjoint(const SysDev &S, const T *C, const double *R, const MeasBufs<T> &mb,
                          const WalkerOut &out, const AdjLayout &L, int W, hipStream_t st) {
    const dim3 g((unsigned)W), b((unsigned)(64 * L.waves));
    constexpr bool SH = sizeof(T) == 8;
#define ADJ(NT, SHARED) hipLaunchKernelGGL((k_adjoint_mfma<T, NT, SHARED>), g, b, L.bytes, st, S, C, R, mb, out, L)
    switch ((S.n_occ + 15) / 16) {
        case 1: ADJ(1, SH); break;
        case 2: ADJ(2, SH); break;
        case 3: ADJ(3, SH); break;
        default:
            if (SH && L.shared)
                ADJ(4, SH);
            else
                ADJ(4, false);
            break;
    }
#undef ADJ
    return hipGetLastError();
}

template <typename T>
hipError_t configure_adjoint(size_t lds) {
    constexpr bool SH = sizeof(T) == 8;
    const void *f[5] = {(const void *)k_adjoint_mfma<T, 1, SH>, (const void *)k_adjoint_mfma<T, 2, SH>,
                        (const void *)k_adjoint_mfma<T, 3, SH>, (const void *)k_adjoint_mfma<T, 4, SH>,
                        (const void *)k_adjoint_mfma<T, 4, false>};
    for (const void *g : f) {
        const hipError_t e = hipFuncSetAttribute(g, hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds);
        if (e != hipSuccess) return e;
    }
    return hipSuccess;
}

template hipError_t launch_adjoint<double>(const SysDev &, const double *, const double *, const MeasBufs<double> &,
                                           const WalkerOut &, const AdjLayout &, int, hipStream_t);
template hipError_t configure_adjoint<double>(size_t);

template hipError_t launch_adjoint<float>(const SysDev &, const float *, const double *, const MeasBufs<float> &,
                                          const WalkerOut &, const AdjLayout &, int, hipStream_t);
template hipError_t configure_adjoint<float>(size_t);

}  // namespace vmcx
