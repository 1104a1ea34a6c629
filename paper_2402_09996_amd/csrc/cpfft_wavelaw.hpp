// The FP64 law of the Table 1 systems with four lanes per voxel.
//
// One wave integrates tiles of 16 voxels: lane (g, n) = (lane / 16,
// lane % 16) holds the systems of slip plane g of voxel n, three slip
// systems (slots 0, 1 superdislocations, 2 ordinary) and the plane's twin
// (slot 3).  That is the accumulator layout of the 16x16x4 matrix
// instruction, which contracts over the 16 systems of a voxel without
// moving them between lanes.  The strain enters once per load step
// (T0 = P C (eps_n - ep_n), dT = P C (eps - eps_n)); within it the resolved
// stresses are tau = T0 + f dT - H G, where G is the sum of the weighted
// signed slip increments since the step began and H = P C P^T, and the
// plastic strain is contracted once per substep.
//
// What bounds it.  With a lane per voxel (cpfft_device.hpp) the FP64 law
// keeps 6 + 2 S state values, three RK4 copies of them and Newton columns
// per lane: 338 registers and 106 KB of LDS per block, one wave per SIMD,
// VALU 49 % busy.  Here a lane holds a quarter of the systems: 168 registers
// and 53 KB at 128 points, three waves per SIMD, VALU 58 % and matrix units
// 14 % busy at 128^3 (the FP64 matrix and vector instructions share the SIMD's
// FP64 units: measured together they take the sum of their times, so the
// matrix form saves the exchange between lanes, not arithmetic).  128^3, 16
// systems, 4 substeps, per launch over four load steps: 3882 us before, 2195
// now; 64^3 847 / 600, 16^3 (12 systems, 10-16 substeps) 226 / 79.  FP32 keeps
// a lane per voxel: three of its blocks run per CU as it is, and the exchange
// between lanes here adds instructions (128^3: 822 us with its Newton solves
// of that time, against 1169).
#pragma once
#include "cpfft_device.hpp"

namespace cpf {

typedef double Acc4 __attribute__((ext_vector_type(4)));

// D = A B + C of one wave: A [16][4] (lane: row lane % 16, column lane / 16),
// B [4][16] (row lane / 16, column lane % 16), C and D [16][16] (column
// lane % 16, rows wl_row(lane / 16, element)).
__device__ __forceinline__ Acc4 wl_mma(double a, double b, Acc4 c)
{
    return __builtin_amdgcn_mfma_f64_16x16x4f64(a, b, c, 0, 0, 0);
}
// Matrix row of accumulator element r in lane group g.
__host__ __device__ constexpr int wl_row(int g, int r) { return 4 * r + g; }
// System of slot r in lane group g (Table 1 order: planes of three slip
// systems, then the four twins).
__host__ __device__ constexpr int wl_sys(int g, int r) { return r < 3 ? 3 * g + r : 12 + g; }

// Matrices of the law as A operands, one value per lane; filled on the host
// from the problem's Schmid tensors and stiffness.
constexpr int WL_H = 0;     // 4: -P C P^T, columns = slot j of each lane group
constexpr int WL_PT = 4;    // 4: P^T, rows = strain components, columns as WL_H
constexpr int WL_PC = 8;    // 2: P C, columns = strain components 0-3 and 4-7 (6, 7 empty)
constexpr int WL_TAB = 10;
constexpr int WL_LDS_TAB = 4;   // the first of them (every stage's) lie in LDS

// LDS rows: elastic strain at the start of the step [6] and strain increment
// [6] in the crystal frame, one column per voxel of the block; on return
// the elastic strain at the end and the plastic strain increment.
constexpr int WL_ROWS = 12;
constexpr int WL_STRIDE = 256;
constexpr size_t WL_ROWS_BYTES = (size_t)WL_ROWS * WL_STRIDE * sizeof(double);

// Root-solve list of one wave: at most 256 active systems.  In: overstress
// with the sign of the slip, root and rate of the previous stage; out: rate
// with that sign, root.
struct WlItem {
    double o, y, g;
};
constexpr size_t WL_LIST_BYTES = 256 * sizeof(WlItem);

// A value that is the same in every lane, into scalar registers.
__device__ __forceinline__ double wl_uniform(double x)
{
    const uint64_t b = __builtin_bit_cast(uint64_t, x);
    const uint32_t lo = (uint32_t)__builtin_amdgcn_readfirstlane((int)(uint32_t)b);
    const uint32_t hi = (uint32_t)__builtin_amdgcn_readfirstlane((int)(uint32_t)(b >> 32));
    return __builtin_bit_cast(double, (uint64_t)hi << 32 | lo);
}

__device__ __forceinline__ int wl_uniform(int x) { return __builtin_amdgcn_readfirstlane(x); }
template <typename T>
__device__ __forceinline__ T *wl_uniform(T *x)
{
    return reinterpret_cast<T *>(__builtin_bit_cast(uint64_t, wl_uniform(__builtin_bit_cast(double, x))));
}

// The lane's index, computed anew where it is called: opaque to the
// compiler, which would otherwise compute the addresses that follow from it
// once per kernel and hold them (the rows of the state alone: 32 registers)
// through the law.
__device__ __forceinline__ int wl_lane()
{
    int l;
    asm volatile("v_mbcnt_lo_u32_b32 %0, -1, 0\n\tv_mbcnt_hi_u32_b32 %0, -1, %0" : "=v"(l));
    return l;
}

// y^p for a uniform integer p >= 1, by the bits of p from the top (the empty
// asm keeps the product under a branch: a select would cost two instructions
// whether or not the bit is set).
__device__ __forceinline__ double wl_powu(double y, int p)
{
    double r = y;
#pragma unroll 1
    for (int b = 30 - __builtin_clz((unsigned)p); b >= 0; --b) {
        r *= r;
        if ((p >> b) & 1) {
            asm volatile("");
            r *= y;
        }
    }
    return r;
}

// y^(n-1).  UNI: the families' exponents are one integer n >= 2 (nm1_uni >=
// 1).  The software log2 and exp2 of the other case take 45 registers more,
// hence a kernel of its own (two blocks per CU).
template <bool UNI>
__device__ __forceinline__ double wl_pow(double y, double nm1, const LawP<double> &P)
{
    if constexpr (UNI) return wl_powu(y, P.nm1_uni);
    else return ex2(nm1 * lg2(y));
}

// Root of phi(y) = K y + etaA y^n - o, o > 0 (see newton_solve).  With a
// root y of the previous stage (y = 0: none) and its rate g, so that
// K y + eta g was the overstress there, the iteration starts from the
// second-order change of the root with the overstress,
//   y (1 + u - a u^2), u = (o - K y - eta g) / S, a = n (n-1)/2 eta g / S,
//   S = K y + n eta g = y phi',
// while |u| is below u_max: 0.06, beyond n = 10 0.6 / n, since the series is
// one in n u (at n = 100 and u = 0.06 it ends a third below the root, from
// where a step leads far above it and 40 iterations do not lead back).
// Otherwise, and without a root, it starts from the upper bounds of
// newton_solve, whatever the exponent at most 2^(1/n) above the root.  So
// at most 6 iterations are needed at n = 10 and 9 at n = 600 (16 and more
// than 40 from y itself).  A step's reciprocal is the hardware's estimate
// (relative error below 1e-7) refined once: an error d of it leaves an error
// d step in the root, of which (o - K y)/eta makes up to d of the rate where
// K y is nearly o.  The family's constants are uniform.
template <bool UNI>
__device__ __forceinline__ double wl_newton(double o, double A, double y, double g, double K, double n, double nm1,
                                            double u_max, const LawP<double> &P, int &nnewt)
{
    const double etaA = P.eta * A;
    const double q = P.eta * g, nq = n * q, Ky = K * y;
    const double rS = __builtin_amdgcn_rcp(Ky + nq);
    const double u = ((o - Ky) - q) * rS;
    const bool far = !(fabs(u) < u_max);   // no root: u is infinite
    double z = y + y * (u - 0.5 * nm1 * nq * rS * u * u);
    if (__any(far)) {
        asm volatile("");
        // an upper bound is enough: FP32, raised by 1e-5 (newton_solve);
        // where it underflows o/K is taken, since the logarithm of a
        // start at 0 would be infinite (0^0 for n = 1: NaN)
        const double yk = o / K;
        const float w = (float)o * __builtin_amdgcn_rcpf((float)etaA);
        const double yc = (double)ex2(lg2(w) * __builtin_amdgcn_rcpf((float)n)) * (1.0 + 1e-5);
        if (far) z = yk < yc || !(yc > 0.0) ? yk : yc;
    }
#pragma unroll 1
    for (int it = 0; it < 40; ++it) {
        const double w = etaA * wl_pow<UNI>(z, nm1, P);
        const double phi = (K + w) * z - o;
        const double dphi = K + n * w, r = __builtin_amdgcn_rcp(dphi);
        const double step = phi * fma(r, fma(-dphi, r, 1.0), r);
        z -= step;
        ++nnewt;
        if (fabs(step) <= P.newton_rtol * z) break;
    }
    return z;
}

// Sum over the four lane groups of each voxel.
__device__ __forceinline__ double wl_sum4(double x)
{
    x += __shfl_xor(x, 16, 64);
    return x + __shfl_xor(x, 32, 64);
}

// E[k] exp(-x[k]) into e, where the lanes of the wave mostly have |x| <= 1/64:
// Taylor sums, remainder |x|^7 / 5040 < 5e-17.  With larger |x| in some lane
// (of either sign: a law may have b < 0), by 18 terms up to |x| = 1, and
// beyond by halving x and squaring; past |x| = 1100 the factor is 0 or
// infinite.
template <int NSL>
__device__ __forceinline__ void wl_decay(const double (&E)[NSL], const double (&x)[NSL], double (&e)[NSL])
{
    double xm = 0.0;
#pragma unroll
    for (int k = 0; k < NSL; ++k) xm = fmax(xm, fabs(x[k]));
    if (!__any(xm > 1.0 / 64.0)) {
#pragma unroll
        for (int k = 0; k < NSL; ++k) {
            double p = fma(-x[k], 1.0 / 720.0, 1.0 / 120.0);
            p = fma(-x[k], p, 1.0 / 24.0);
            p = fma(-x[k], p, 1.0 / 6.0);
            p = fma(-x[k], p, 0.5);
            p = fma(-x[k], p, 1.0);
            e[k] = E[k] * fma(-x[k], p, 1.0);
        }
        return;
    }
    int m = 0;
    xm = fmin(xm, 1100.0);
    while (__any(xm > 1.0)) {
        xm *= 0.5;
        ++m;
    }
    const double f = ldexp(1.0, -m);
#pragma unroll
    for (int k = 0; k < NSL; ++k) {
        const double z = x[k] * f;
        double p = 1.0;
#pragma unroll 1
        for (int i = 18; i > 0; --i) p = 1.0 - z * p / (double)i;
        for (int i = 0; i < m; ++i) p *= p;
        if (x[k] > 1100.0) p = 0.0;
        if (x[k] < -1100.0) p = INFINITY;
        e[k] = E[k] * p;
    }
}

// Work of one wave: 16 voxels of the block (columns v0 .. v0 + 15 of the
// rows, those below nv exist) integrated over the load step.  tab: the
// matrices in global memory, htab: H in LDS.  st_in and st_out: the committed
// and the trial state [6 + 2 S][N] (rows v and alpha only; S = 12 or 16
// systems), vox0: the grid's voxel of column 0.  Sums over the voxels are
// added to vs (accumulated slip) and ft (twin fractions), the work counters
// to nact and nnewt (nnewt per lane, the others uniform).  Called by whole
// waves.
//
// The saturation terms: each slot carries E = exp(-b v) of the substep's
// start and multiplies it by the short series of exp(-b dv), dv the slip
// since (8 instructions in place of the 25 of the software exponential).
template <int NSL, bool UNI>
__device__ __forceinline__ void wave_law(const LawP<double> &P, const double *tab, const double *htab, double *rows,
                                         int v0, int nv, const double *st_in, double *st_out, long N, long vox0,
                                         double dt, int M, WlItem *list, double &vs, double &ft, int &nact,
                                         int &nnewt)
{
    constexpr int S = NSL == 4 ? 16 : 12;
    const int lane = wl_lane();
    const double *hl = htab + lane;   // this lane's value of H
    const Acc4 zero = {0.0, 0.0, 0.0, 0.0};

    // one list when twins obey the slip systems' rate law; otherwise the
    // lanes solve their twins in a pass of their own
    const bool one_list = NSL == 3 || (P.twin_mode == 0 && P.fs.K == P.ft.K && P.fs.n == P.ft.n);

    // per slot: v, alpha; E = exp(-b v); root and rate of the previous stage
    double v[NSL], al[NSL], E[NSL], y[NSL], gp[NSL];
    // resolved stresses: at the start of the substep, change over the load step
    Acc4 TB, dT;
    {
        const int g = lane >> 4, col = v0 + (lane & 15);
        const bool in = col < nv;
        const long vox = vox0 + col;
        const double *rc = rows + col, *pc = tab + WL_PC * 64 + lane;
#pragma unroll
        for (int k = 0; k < NSL; ++k) {
            // a column without a voxel has the back strain NaN: no system of
            // it is active then, with a negative initial resistance neither,
            // and it adds nothing to the sums
            v[k] = in ? st_in[(6 + wl_sys(g, k)) * N + vox] : 0.0;
            al[k] = in ? st_in[(6 + S + wl_sys(g, k)) * N + vox] : __builtin_nan("");
            E[k] = ex2(-(k < 3 ? P.fs.bl2e : P.ft.bl2e) * v[k]);
            y[k] = gp[k] = 0.0;
        }
        TB = wl_mma(pc[0], rc[g * WL_STRIDE], zero);
        dT = wl_mma(pc[0], rc[(6 + g) * WL_STRIDE], zero);
        TB = wl_mma(pc[64], g < 2 ? rc[(4 + g) * WL_STRIDE] : 0.0, TB);
        dT = wl_mma(pc[64], g < 2 ? rc[(10 + g) * WL_STRIDE] : 0.0, dT);
    }
    const double h = wl_uniform(dt / (double)M), invM = wl_uniform(1.0 / (double)M);
    const double t0[4] = {P.tau0k[1], P.tau0k[1], P.tau0k[0], P.tau0k[2]};
    // plastic strain since the step began: this lane's matrix rows below 6
    // (the first two elements)
    double dep[2] = {0.0, 0.0};

#pragma unroll 1
    for (int j = 0; j < M; ++j) {
        // stage values: e1 = exp(-b v), tf the twin's slip, tal; sums over
        // the stages: dv, aal, Gs
        double e1[NSL], tf = NSL == 4 ? v[NSL - 1] : 0.0, tal[NSL], dv[NSL], aal[NSL], Gs[NSL];
        Acc4 tau = TB;
        bool slipped = false;
#pragma unroll
        for (int k = 0; k < NSL; ++k) {
            e1[k] = E[k];
            tal[k] = aal[k] = al[k];
            dv[k] = Gs[k] = 0.0;
        }
#pragma unroll 1
        for (int st = 0; st < 4; ++st) {
            const double wacc = wl_uniform((st == 0 || st == 3) ? h * (1.0 / 6.0) : h * (1.0 / 3.0));
            const double cnext = wl_uniform((st == 2) ? h : h * 0.5);
            const double fr = wl_uniform((st == 2) ? invM : 0.5 * invM);
            // overstresses; the active ones go to the list
            WlItem *item[NSL];
            bool on[NSL];
            int nl = 0, n1 = 0;
            double wslip = 1.0, Atw = 1.0;
            {
                double hs[NSL], Hs, Ht = 0.0;
#pragma unroll
                for (int k = 0; k < NSL; ++k) hs[k] = 1.0 - e1[k];
                Hs = P.fs.QL * wl_sum4(hs[0] + hs[1] + hs[2]);
                if constexpr (NSL == 4) {
                    Ht = P.ft.QL * wl_sum4(hs[3]);
                    const double f = P.inv_gT * wl_sum4(tf);
                    wslip = 1.0 - f;
                    if (P.twin_mode) Atw = P.Kc_gT * (P.fm - f);
                }
#pragma unroll
                for (int k = 0; k < NSL; ++k) {
                    if (k == 3) n1 = nl;
                    const double r = (t0[k] + (k < 3 ? Hs : Ht)) + (k < 3 ? P.fs.QD : P.ft.QD) * hs[k];
                    const double tx = tau[k] - (k < 3 ? P.fs.c : P.ft.c) * tal[k];
                    const double o = (k < 3 ? fabs(tx) : tx) - r;
                    on[k] = o > 0.0;
                    if (k == 3) on[k] = on[k] && Atw > 0.0;
                    const uint64_t b = __ballot(on[k]);
                    item[k] = list + nl +
                              __builtin_amdgcn_mbcnt_hi((uint32_t)(b >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)b, 0u));
                    nl += __popcll(b);
                    // an active slip system has |tx| > r >= 0: the sign of tx is the slip's
                    if (on[k]) *item[k] = WlItem{k < 3 ? copysign(o, tx) : o, y[k], gp[k]};
                }
            }
            nact += nl;
            if (nl != 0) {
                __builtin_amdgcn_wave_barrier();
                // passes over the list; in the last one, with twins of their
                // own rate law, every lane takes its own
                const int ns = one_list ? nl : n1;
                const int nb = (ns + 63) & ~63;
                const int end = NSL == 4 && ns < nl ? nb + 64 : nb;
                for (int b = 0; b < end; b += 64) {
                    const bool tw = NSL == 4 && b == nb;
                    WlItem *it = tw ? item[NSL - 1] : list + b + lane;
                    if (tw ? on[NSL - 1] : b + lane < ns) {
                        const double os = it->o, o = fabs(os), A = tw ? Atw : 1.0;
                        const double K = tw ? P.ft.K : P.fs.K, nm1 = tw ? P.ft.nm1 : P.fs.nm1;
                        const double z = wl_newton<UNI>(o, A, it->y, it->g, K, tw ? P.ft.n : P.fs.n, nm1,
                                                        tw ? P.ft.u_max : P.fs.u_max, P, nnewt);
                        it->y = z;
                        double rate = (o - K * z) * P.inv_eta;
                        if (!(P.eta > 0.0)) rate = A * z * wl_pow<UNI>(z, nm1, P);
                        it->o = copysign(rate, os);
                    }
                }
                __builtin_amdgcn_wave_barrier();
                tau = TB + fr * dT;
                double x[NSL];
#pragma unroll
                for (int k = 0; k < NSL; ++k) {
                    double gd = 0.0;
                    y[k] = 0.0;
                    if (on[k]) {
                        gd = item[k]->o;
                        y[k] = item[k]->y;
                    }
                    const double ag = fabs(gd);
                    gp[k] = ag;
                    const double dal = gd - (k < 3 ? P.fs.d : P.ft.d) * ag * tal[k];
                    dv[k] += wacc * ag;
                    aal[k] += wacc * dal;
                    tal[k] = al[k] + cnext * dal;
                    x[k] = cnext * ag;
                    const double wg = NSL == 4 && k < 3 ? wslip * gd : gd;
                    Gs[k] += wacc * wg;
                    tau = wl_mma(hl[(WL_H + k) * 64], cnext * wg, tau);
                }
                if constexpr (NSL == 4) tf = v[3] + x[3];
#pragma unroll
                for (int k = 0; k < NSL; ++k) x[k] *= k < 3 ? P.fs.b : P.ft.b;
                wl_decay<NSL>(E, x, e1);
                slipped = true;
            } else {
                tau = TB + fr * dT;
#pragma unroll
                for (int k = 0; k < NSL; ++k) {
                    y[k] = gp[k] = 0.0;
                    tal[k] = al[k];
                    e1[k] = E[k];
                }
                if constexpr (NSL == 4) tf = v[3];
            }
        }
        TB += invM * dT;
        if (slipped) {
            double x[NSL];
            Acc4 d = zero;
            const double *tl = tab + lane;
            d[0] = dep[0];
            d[1] = dep[1];
#pragma unroll
            for (int k = 0; k < NSL; ++k) {
                v[k] += dv[k];
                al[k] = aal[k];
                TB = wl_mma(hl[(WL_H + k) * 64], Gs[k], TB);
                d = wl_mma(tl[(WL_PT + k) * 64], Gs[k], d);
                x[k] = (k < 3 ? P.fs.b : P.ft.b) * dv[k];
            }
            wl_decay<NSL>(E, x, E);
            dep[0] = d[0];
            dep[1] = d[1];
        }
    }
    const int lane1 = wl_lane();
    const int g = lane1 >> 4, col = v0 + (lane1 & 15);
    const long vox = vox0 + col;
    double *rc = rows + col;
#pragma unroll
    for (int k = 0; k < 2; ++k) {
        const int c = wl_row(g, k);
        if (c < 6) {
            rc[c * WL_STRIDE] += rc[(6 + c) * WL_STRIDE] - dep[k];
            rc[(6 + c) * WL_STRIDE] = dep[k];
        }
    }
    if (col < nv) {
#pragma unroll
        for (int k = 0; k < NSL; ++k) {
            st_out[(6 + wl_sys(g, k)) * N + vox] = v[k];
            st_out[(6 + S + wl_sys(g, k)) * N + vox] = al[k];
        }
    }
    double a = 0.0;
#pragma unroll
    for (int k = 0; k < 3; ++k) a += (double)v[k];
    vs = wl_uniform(vs + wave_sum(a));
    if constexpr (NSL == 4) ft = wl_uniform(ft + wave_sum((double)v[3] * (double)P.inv_gT));
}

}  // namespace cpf
