// Collision of one cell, shared by every step kernel (one step per launch and
// several steps per launch): moments (a2), fluctuation-form flux (a3),
// shifted equilibrium (a4), sources (a5) and relaxation (a6) from the cell's
// pulled populations to its post-collision populations.
//
// Expressions are contracted to fused multiply-adds only within one source
// expression (the pragma below and in the headers this one includes), so the
// update rounds alike in every kernel it is inlined into: a run advanced
// several steps per launch is bit for bit the run advanced step by step.
#pragma once

#include <hip/hip_runtime.h>

#include <type_traits>

#include "device_common.hpp"

#ifndef LBM_FAST_CONTRACT
#pragma clang fp contract(on)
#endif

// collision operators of the step kernels
enum { COLL_BGK = 0, COLL_TRT = 1, COLL_REG = 2 };

// c2 e_i + w_i s for i >= 1, in double: the equilibrium of zeroth moment q
// and first moment G = lam dPhi scaled by c2, plus the source's part.
template <class L>
__device__ inline void wide_feq(double c2, double q, const double *G, double s, double *e)
{
    const double m = fma(c2, q, s);
    if constexpr (L::Q == 9) {
        const double A = m * (1.0 / 36), A4 = m * (1.0 / 9), k = c2 * (1.0 / 12);
        const double hx = k * G[0], hy = k * G[1], sp = hx + hy, sm = hy - hx;
        e[1] = fma(4.0, hx, A4); e[2] = fma(4.0, hy, A4); e[3] = fma(-4.0, hx, A4); e[4] = fma(-4.0, hy, A4);
        e[5] = A + sp; e[6] = A + sm; e[7] = A - sp; e[8] = A - sm;
    } else {
        const double A = m * L::w[1], h = 0.5 * c2;
#pragma unroll
        for (int i = 1; i < L::Q; ++i) {
            const int a = L::cx[i] != 0 ? 0 : (L::cy[i] != 0 ? 1 : 2);
            e[i] = fma(lat_c<L>(i, a) > 0 ? h : -h, G[a], A);
        }
    }
}

// Readers of a cell's coefficient field and explicit source ([.][C] arrays of
// F, the cell at byte offset off).
// EXT false: known to have neither.
template <class F, class I, bool EXT = true>
struct CellFields {
    static constexpr bool ext = EXT;
    const F *cb, *cs;
    size_t C;
    I off;
    __device__ F b(int a) const { return *byte_at(cb + a * C, off); }
    __device__ F s(int k) const { return *byte_at(cs + k * C, off); }
};

template <class Sys, class Lat, class St, int COLL>
struct Cell {
    static constexpr int K = Sys::K, Q = Lat::Q, D = Lat::D;
    static constexpr bool F16 = std::is_same<St, _Float16>::value;
    // Single-precision storage of the precise systems computes in double:
    // every operation on the stored values is then exact to far below their
    // rounding, and post is rounded once, at the store.  On this part a
    // double add, multiply or fma issues at 0.6 of the float rate (530 against
    // 865-915 G wave instructions/s measured), while the float-float form of
    // the same accuracy takes six to eight float operations for each: 886 ->
    // 412 vector instructions per wave for shallow water on D2Q9, 635 -> 327
    // for Euler on D2Q5 (150 x 101 shallow water: 5.6 -> 4.6 us per step).
    // The other systems evaluate their flux in float, as their registers
    // allow, and form moments, equilibria and relaxation in double (WIDEQ: 3D
    // NSF 3714 -> 2407 vector instructions, 75 x 66 x 50: 40.0 -> 37.5 us per
    // step; at 256^3, bound by memory, 2745 -> 2780).
    static constexpr bool WIDE = Sys::precise && std::is_same<St, float>::value;
    // The 3D velocity-gradient trackers need the accuracy: they see the
    // momentum's rounding amplified by |u| / |du| and by 1 / (k dx), and with
    // plain-float equilibria their distance to the FP64 oracle reached 3x the
    // binary32 storage floor at 128^3.
    static constexpr bool WIDEQ = !Sys::precise && std::is_same<St, float>::value;
    using F = typename Store<St>::R;                                    // type of the per-cell fields
    using P = typename std::conditional<WIDE, Wd, F>::type;             // type of the parameters
    using X = typename std::conditional<WIDE, double, F>::type;         // type of fluxes and sources
    using CT = CoefTraits<Sys>;
    static constexpr int NB = CT::NB > 3 ? CT::NB : 3;

    // Post-collision populations from the pulled ones f (the stored values;
    // binary16 unscaled), handed to emit(k, i, value) in the stored type as
    // they are formed; dQ: the moment deviations (a history's entries).
    // ex: the cell's readers of its coefficients, ex.b(a), and its explicit
    // source, ex.s(k) (called where attached), Smms: the in-kernel forcing of
    // the conserved rows.
    template <class Ext, class Emit>
    __device__ __forceinline__ static void update(const KParams<P> &p, const F (*f)[Q], const Ext &ex,
                                                  const F *Smms, F *dQ, Emit &&emit)
    {
        if constexpr (WIDE || WIDEQ)
            wide(p, f, ex, Smms, dQ, emit);
        else
            plain(p, f, ex, Smms, dQ, emit);
    }

    // The moment sums convert every population to double, the relaxation needs
    // them in double again.  With more than about 30 populations keeping the
    // doubles would fill the registers: the value is converted a second time
    // (the empty asm keeps the compiler from reusing the first conversion).
    __device__ __forceinline__ static F again(F v)
    {
        if constexpr (K * Q > 30) asm("" : "+v"(v));
        return v;
    }

    // per-cell coefficients (default values when none is attached)
    template <class Ext, class B>
    __device__ __forceinline__ static void coefficients(const KParams<P> &p, const Ext &ex, B *bl)
    {
#pragma unroll
        for (int a = 0; a < NB; ++a) bl[a] = B(CT::dflt(a));
        if (Ext::ext && p.b) {
#pragma unroll
            for (int a = 0; a < CT::NB; ++a) bl[a] = B(ex.b(a));
        }
    }

    template <class Ext, class Emit>
    __device__ __forceinline__ static void wide(const KParams<P> &p, const F (*f)[Q], const Ext &ex, const F *Smms, F *dQ,
                                                Emit &emit)
    {
        double q[K];
#pragma unroll
        for (int k = 0; k < K; ++k) {
            q[k] = (double)f[k][0];
#pragma unroll
            for (int i = 1; i < Q; ++i) q[k] += (double)f[k][i];
            dQ[k] = (F)q[k];
        }
        X dPhi[K][D], Sk[K];
        P bl[NB];
        coefficients(p, ex, bl);
        if constexpr (CT::in_flux)
            Sys::template flux_delta_b<F, F>(p.phys, dQ, bl, dPhi);
        else if constexpr (WIDE)
            Sys::template flux_delta<double, Wd>(p.phys, q, dPhi);
        else
            Sys::template flux_delta<F, F>(p.phys, dQ, dPhi);
        if constexpr (WIDE)
            Sys::template source<double, Wd>(p.phys, q, bl, Sk);
        else
            Sys::template source<F, F>(p.phys, dQ, bl, Sk);
        if (Ext::ext && p.sext) {
#pragma unroll
            for (int k = 0; k < K; ++k) Sk[k] += (X)ex.s(k);
        }
        if constexpr (Sys::id == SYS_NSF17) {
#pragma unroll
            for (int k = 0; k < 5; ++k) Sk[k] += (X)Smms[k];
        }
#pragma unroll
        for (int k = 0; k < K; ++k) {
            const double c1 = p.c1[k], c2 = p.c2[k], dts = (double)p.dt * (double)Sk[k];
            double G[D], e[Q], fd[Q];
            F fk[Q];
#pragma unroll
            for (int i = 1; i < Q; ++i) {
                fk[i] = again(f[k][i]);
                fd[i] = (double)fk[i];
            }
#pragma unroll
            for (int a = 0; a < D; ++a) G[a] = (double)p.lam * (double)dPhi[k][a];
            F acc = (F)dts;
            // post_i = e_i + c1 (e_i - f_i) + dt w_i S with c1 = omega - 1; TRT
            // and regularized as in plain()
            if constexpr (COLL == COLL_BGK) {
                wide_feq<Lat>(c2, q[k], G, dts, e);
            } else if constexpr (COLL == COLL_TRT) {
                const double tb = p.tb[k];
                double z[Q], b[Q];
                wide_feq<Lat>(1.0, q[k], G, 0.0, z);
                wide_feq<Lat>(c2, q[k], G, dts, e);
#pragma unroll
                for (int i = 1; i < Q; ++i) b[i] = tb * (z[i] - fd[i]);
#pragma unroll
                for (int i = 1; i < Q; ++i) e[i] += b[Lat::opp[i]];
            } else {
                double P1[D];
                wide_feq<Lat>(1.0, q[k], G, 0.0, e);
#pragma unroll
                for (int a = 0; a < D; ++a) P1[a] = 0.0;
#pragma unroll
                for (int i = 1; i < Q; ++i)
#pragma unroll
                    for (int a = 0; a < D; ++a)
                        if (lat_c<Lat>(i, a) != 0) P1[a] += lat_c<Lat>(i, a) * (fd[i] - e[i]);
#pragma unroll
                for (int i = 1; i < Q; ++i) {
                    double cp = 0.0;
#pragma unroll
                    for (int a = 0; a < D; ++a) cp += lat_c<Lat>(i, a) * P1[a];
                    e[i] += (-c1) * (cp * (double(Lat::Wn[i]) / Lat::Fden)) + dts * Lat::w[i];
                }
            }
#pragma unroll
            for (int i = 1; i < Q; ++i) {
                const F post = COLL == COLL_REG ? (F)e[i] : (F)fma(-c1, fd[i], e[i]);
                emit(k, i, (St)post);
                acc += fk[i] - post;
            }
            emit(k, 0, (St)(f[k][0] + acc));
        }
    }

    template <class Ext, class Emit>
    __device__ __forceinline__ static void plain(const KParams<F> &p, const F (*f)[Q], Ext &ex,
                                                 const F *Smms, F *dQ, Emit &emit)
    {
#include "collide_plain.inc"
    }
};
