// FP16 storage of the deviation from the sender's local equilibrium
// (storage LBM_F16NE).
//
// The paper stores the populations shifted by the background equilibrium
// (Sec. 2.5.2).  In binary16 that leaves a rounding of ~2^-12 |f*| per
// population per step, which over thousands of steps dominates fields that
// start at zero.  This storage keeps, for every cell y, its pre-collision
// moment deviations M(y) in FP32 and stores in binary16 only
//     g_i(y) = post_i(y) - e_i(M(y)),
// the deviation of each post-collision population from the cell's own
// (shifted, exact-moment) equilibrium e_i(M) = w_i M + (w_i/cs^2) c_i.(dt/dx)
// dPhi(M).  With post = e + (omega - 1)(e - f) + dt w_i S the stored value is
// g_i = (omega - 1)(e_i - f_i) + dt w_i S (the non-equilibrium part), formed
// without cancellation.  The receiver x = y + c_i rebuilds
//     f_i(x) = g_i(x - c_i) + e_i(M(x - c_i))
// by re-evaluating the flux at the sender's stored moments (the same float
// computation as the sender's).  Per cell update this moves K Q 2 bytes of
// populations and K 4 bytes of moments each way.
//
// Buffer layout (each of A and B): the binary16 deviations in the
// tile-blocked layout of the step kernels ([tiles][K][Q][kTile], the cells
// padded to whole tiles), padded to 256 bytes, then moments [K][cells]
// float.
#include <hip/hip_runtime.h>

#include <cmath>
#include <cstring>

#include "march.hpp"

inline size_t ne_pop_bytes(long long C, int K, int Q)
{
    return (((size_t)K * Q * (size_t)padded_plane(C) * 2) + 255) & ~(size_t)255;
}

// Collision of one cell from its pulled populations: emit(k, i, deviation in
// the stored form, the cell's own equilibrium e_i); dQ: the moments.
template <class Sys, class Lat, class Emit>
__device__ __forceinline__ void ne_collide(const KParams<float> &p, const float (&f)[Sys::K][Lat::Q], const float *bl,
                                           float *dQ, Emit &&emit)
{
    constexpr int K = Sys::K, Q = Lat::Q, D = Lat::D;
#pragma unroll
    for (int k = 0; k < K; ++k) {
        float s = f[k][0];
#pragma unroll
        for (int i = 1; i < Q; ++i) s += f[k][i];
        dQ[k] = s;
    }
    float dPhi[K][D], Sk[K];
    Sys::template flux_delta<float, float>(p.phys, dQ, dPhi);
    Sys::template source<float, float>(p.phys, dQ, bl, Sk);
#pragma unroll
    for (int k = 0; k < K; ++k) {
        float G[D], e[Q], s[Q];
#pragma unroll
        for (int a = 0; a < D; ++a) G[a] = p.lam * dPhi[k][a];
        ExactEq<Lat>::feq(dQ[k], 0.0f, G, e);
        const float e0 = ExactEq<Lat>::rest(dQ[k]);
        const float dts = p.dt * Sk[k];
        ExactEq<Lat>::zeroth(dts, s);
        float acc = dts;
#pragma unroll
        for (int i = 1; i < Q; ++i) {
            const float d = e[i] - f[k][i];
            const _Float16 hv = (_Float16)(fmaf(p.c1[k], d, s[i]) * p.scale[k]);
            emit(k, i, hv, e[i]);
            // f - e is exactly -d and hv / scale is exact: the closure's
            // (f - e) - hv / scale is -(d + hv / scale), rounded once
            acc -= fmaf((float)hv, p.inv_scale[k], d);
        }
        const float g0 = (f[k][0] - e0) + acc;
        emit(k, 0, (_Float16)(g0 * p.scale[k]), e0);
    }
}

// The step works on a tile of kNeTX x kNeTY cells whose senders (the tile
// and a one-cell halo, periodic) first put the parts of their equilibrium
// into LDS: the stored moment divided by 9 (D2Q9) or 3 (D2Q5) and the two
// components of lam dPhi(M) times w_1 / cs^2 (ExactEq::parts).  The flux and
// the weight divisions of each sender are evaluated once per workgroup
// instead of once per pulled population (Q - 1 times per cell); the
// receiver finishes each pulled population's equilibrium from LDS with two
// or three operations (ExactEq::dir), bit for bit the sender-side
// definition above.
constexpr int kNeTX = 64, kNeTY = 4;

// periodic index of a halo row or column v in [-1, n + kNeTX]: one
// conditional step where the tile fits the grid, a division only on grids
// narrower than a tile
__device__ inline int pmod(int v, int n)
{
    const int r = v < 0 ? v + n : v;
    return r < n ? r : (r < 2 * n ? r - n : r % n);
}

template <class Sys, class Lat, bool NT, bool O32>
__global__ __launch_bounds__(kNeTX * kNeTY) void k_step_ne(const _Float16 *__restrict__ gin,
                                                           const float *__restrict__ Min,
                                                           _Float16 *__restrict__ gout, float *__restrict__ Mout,
                                                           const KParams<float> p)
{
    using I = typename Index<O32>::T;
    constexpr int K = Sys::K, Q = Lat::Q, D = Lat::D;
    constexpr int HX = kNeTX + 2, HY = kNeTY + 2, NH = HX * HY, NTH = kNeTX * kNeTY;
    static_assert(D == 2, "binary16 deviation storage is built for the 2D lattices");
    __shared__ float sP[K][3][NH];
    const size_t C = (size_t)p.C;
    const int tilesx = (p.nx + kNeTX - 1) / kNeTX;
    const unsigned t = (unsigned)xcd_tile(blockIdx.x, gridDim.x);
    const int tx0 = (int)(t % (unsigned)tilesx) * kNeTX, ty0 = (int)(t / (unsigned)tilesx) * kNeTY;
    const int lx = (int)threadIdx.x % kNeTX, ly = (int)threadIdx.x / kNeTX;
    const int x = tx0 + lx, y = ty0 + ly;
    const bool live = x < p.nx && y < p.ny;
    // Each thread evaluates one or two halo senders (h and h + NTH).  The
    // first sender's stored moments are loaded first, then this cell's
    // pulled binary16 deviations, which the halo work does not need: the
    // load counter retires in issue order, so the first halo flux
    // evaluation waits only for its sender's moments while the deviations
    // are still in flight.
    static_assert(NTH <= NH && NH <= 2 * NTH, "one or two halo senders per thread");
    const int h0 = (int)threadIdx.x, h1 = h0 + NTH;
    auto sender = [&](int h) {
        const int hy = h / HX, hx = h - hy * HX;
        return (size_t)pmod(ty0 + hy - 1, p.ny) * p.nx + pmod(tx0 + hx - 1, p.nx);
    };
    float M0[K];
    {
        const size_t c0 = sender(h0);
#pragma unroll
        for (int k = 0; k < K; ++k) M0[k] = Min[(size_t)k * C + c0];
    }
    // two binary16 values per register: the deviations then hold 27 of the
    // kernel's registers instead of 54 (four waves per SIMD, not three)
    typedef _Float16 h2 __attribute__((ext_vector_type(2)));
    h2 gr[K][(Q + 1) / 2];
    if (live) {
#pragma unroll
        for (int i = 0; i < Q; ++i) {
            const I src = tile_offset<K, Q>((I)wrapi(y - Lat::cy[i], p.ny) * (I)p.nx + (I)wrapi(x - Lat::cx[i], p.nx));
#pragma unroll
            for (int k = 0; k < K; ++k) gr[k][i / 2][i % 2] = *byte_at(gin + (size_t)(k * Q + i) * kTile, src * (I)2);
        }
    }
    auto halo = [&](int h, const float *My) {
        float P[K][D];
        Sys::template flux_delta<float, float>(p.phys, My, P);
#pragma unroll
        for (int k = 0; k < K; ++k) {
            float G[D], Pt[3];
#pragma unroll
            for (int a = 0; a < D; ++a) G[a] = p.lam * P[k][a];
            ExactEq<Lat>::parts(My[k], G, Pt);
#pragma unroll
            for (int j = 0; j < 3; ++j) sP[k][j][h] = Pt[j];
        }
    };
    halo(h0, M0);
    if (h1 < NH) {
        float M1[K];
        const size_t c1 = sender(h1);
#pragma unroll
        for (int k = 0; k < K; ++k) M1[k] = Min[(size_t)k * C + c1];
        halo(h1, M1);
    }
    __syncthreads();
    if (!live) return;                                  // no barrier follows
    const long long cell = (long long)y * p.nx + x;
    const I own = tile_offset<K, Q>((I)cell) * (I)2;
    float f[K][Q];
#pragma unroll
    for (int i = 0; i < Q; ++i) {
        const int h = (ly + 1 - Lat::cy[i]) * HX + (lx + 1 - Lat::cx[i]);
#pragma unroll
        for (int k = 0; k < K; ++k) {
            float Pt[3];
#pragma unroll
            for (int j = 0; j < 3; ++j) Pt[j] = sP[k][j][h];
            const float ei = i == 0 ? ExactEq<Lat>::rest_parts(Pt) : ExactEq<Lat>::dir(Pt, i);
            f[k][i] = fmaf((float)gr[k][i / 2][i % 2], p.inv_scale[k], ei);      // the scaling is exact
        }
    }
    float dQ[K], bl[3] = {0.0f, 0.0f, 0.0f};
    if (p.b) {
#pragma unroll
        for (int a = 0; a < D; ++a) bl[a] = ((const float *)p.b)[(size_t)a * C + cell];
    }
    ne_collide<Sys, Lat>(p, f, bl, dQ, [&](int k, int i, _Float16 v, float) {
        st_pop<NT>(byte_at(gout + (size_t)(k * Q + i) * kTile, own), v);
    });
#pragma unroll
    for (int k = 0; k < K; ++k) st_pop<NT>(Mout + (size_t)k * C + cell, dQ[k]);
}

// Several steps per launch, as k_march (march.hpp) does for the other
// storages, with one stage more: stage 0 takes a row's deviations and moments
// as stored, both from the cell itself, and forms the populations that the
// cell sent, g_i + e_i(M) with one flux evaluation per cell; from there on a
// sent population is the same sum of the stage's own values, rounded through
// binary16 like a stored one.  So T steps take T flux evaluations and one more
// per cell, where T launches of k_step_ne take 2.55 T, and the deviations and
// moments cross memory once.  Bit for bit the steps of k_step_ne.
template <class Sys, class Lat> constexpr int ne_march_lds(int T)
{
    return (T * march_slots<Lat>() * Sys::K * 64 + 2) * (int)sizeof(float);
}
// steps per launch that leave five wavefronts a CU their LDS (neo-Hookean
// D2Q9 two, shallow water D2Q9 and the smaller D2Q5 states four)
template <class Sys, class Lat> constexpr int ne_march_most()
{
    int T = 4;
    while (T > 1 && 5 * ne_march_lds<Sys, Lat>(T) > kLdsPerCu) --T;
    return T;
}

template <class Sys, class Lat, int T, bool EXT>
__global__ __launch_bounds__(64) void k_march_ne(const _Float16 *__restrict__ gin, const float *__restrict__ Min,
                                                 _Float16 *__restrict__ gout, float *__restrict__ Mout,
                                                 const KParams<float> p, int rows, int strips)
{
    constexpr int K = Sys::K, Q = Lat::Q, D = Lat::D, HALO = T;
    const int lane = (int)threadIdx.x;
    const unsigned g = (unsigned)xcd_tile(blockIdx.x, gridDim.x);
    const int strip = (int)(g % (unsigned)strips);
    const int y0 = (int)(g / (unsigned)strips) * rows, y1 = segment_end(y0, rows, p.ny);
    const int xo = strip * (64 - 2 * HALO) + lane - HALO;                 // unwrapped column
    const bool mine = lane >= HALO && lane < 64 - HALO && xo < p.nx;      // column stored by this lane
    int xw = xo % p.nx;
    xw = xw < 0 ? xw + p.nx : xw;
    const size_t C = (size_t)p.C;
    int yn = (y0 - HALO) % p.ny;                                          // the row that stage 0 loads next
    yn = yn < 0 ? yn + p.ny : yn;
    const int last = y1 - y0 + 2 * HALO - 1;
    // two rows of stored values: one at work, the next on its way (see k_march)
    _Float16 gi[2][K][Q];
    float mi[2][K];
    auto load = [&](_Float16 (&gt)[K][Q], float (&mt)[K], bool more) {
        const size_t c = (size_t)yn * (size_t)p.nx;
        const unsigned off = tile_offset<K, Q>((unsigned)(c % kTile) + (unsigned)xw) * 2u;
        const auto rg = rsrc_of(gin + c / kTile * (size_t)(K * Q * kTile));
#pragma unroll
        for (int k = 0; k < K; ++k) mt[k] = ld_buf<float>(rsrc_of(Min + k * C + c), (unsigned)xw * 4u, 0);
#pragma unroll
        for (int k = 0; k < K; ++k)
#pragma unroll
            for (int i = 0; i < Q; ++i) gt[k][i] = ld_buf<_Float16>(rg, off, (k * Q + i) * kTile * 2);
        yn = more ? wrapi(yn + 1, p.ny) : yn;
    };
    // populations on their way between stages, as in k_march
    constexpr int NU = Lat::Q == 9 ? 3 : 1, NW = march_slots<Lat>();
    __shared__ float carry[ne_march_lds<Sys, Lat>(T) / sizeof(float)];
    float *const wait = &carry[1 + lane];
    constexpr auto slot = [](int s, int k, int i, int par) {
        int n = Lat::cy[i] > 0 ? par * NU : 2 * NU;
        for (int j = 0; j < i; ++j) n += Lat::cy[j] == Lat::cy[i];
        return ((s * NW + n) * K + k) * 64;
    };
    // one row of the march with stages 0 to NS at work
    auto row = [&](auto ns, auto parity, int j) {
        constexpr int NS = decltype(ns)::value, par = decltype(parity)::value;
        load(gi[par ^ 1], mi[par ^ 1], j + 1 < last);
        __builtin_amdgcn_sched_barrier(0);
        float post[K][Q], f[K][Q];
        {
            float P[K][D];
            Sys::template flux_delta<float, float>(p.phys, mi[par], P);
#pragma unroll
            for (int k = 0; k < K; ++k) {
                float G[D], e[Q];
#pragma unroll
                for (int a = 0; a < D; ++a) G[a] = p.lam * P[k][a];
                ExactEq<Lat>::feq(mi[par][k], 0.0f, G, e);
                e[0] = ExactEq<Lat>::rest(mi[par][k]);
#pragma unroll
                for (int i = 0; i < Q; ++i) post[k][i] = fmaf((float)gi[par][k][i], p.inv_scale[k], e[i]);
            }
        }
#pragma unroll
        for (int s = 0; s < NS; ++s) {
            // the populations sent by stage s arrive a row below; what the rows
            // below left is read before this row takes its place
#pragma unroll
            for (int k = 0; k < K; ++k)
#pragma unroll
                for (int i = 0; i < Q; ++i)
                    f[k][i] = Lat::cy[i] < 0 ? lane_pull<Lat>(post[k][i], i) : wait[slot(s, k, i, par) - Lat::cx[i]];
            wave_fence();
#pragma unroll
            for (int k = 0; k < K; ++k)
#pragma unroll
                for (int i = 0; i < Q; ++i)
                    if (Lat::cy[i] >= 0) wait[slot(s, k, i, par)] = post[k][i];
            wave_fence();
            const int yu = y0 - HALO + j - s - 1;                         // this stage's row, unwrapped
            float dQ[K], bl[3] = {0.0f, 0.0f, 0.0f};
            if (EXT) {
                int y = yu % p.ny;
                y = y < 0 ? y + p.ny : y;
#pragma unroll
                for (int a = 0; a < D; ++a)
                    bl[a] = ((const float *)p.b)[a * C + (size_t)y * (size_t)p.nx + (unsigned)xw];
            }
            if (s == T - 1) {                                             // rows y0 to y1 only: none wraps
                const size_t c = (size_t)yu * (size_t)p.nx;
                const unsigned off = mine ? tile_offset<K, Q>((unsigned)(c % kTile) + (unsigned)xw) * 2u : 0x80000000u;
                const auto rg = rsrc_of(gout + c / kTile * (size_t)(K * Q * kTile));
                ne_collide<Sys, Lat>(p, f, bl, dQ, [&](int k, int i, _Float16 v, float) {
                    st_masked(rg, off, (k * Q + i) * kTile * 2, v);
                });
#pragma unroll
                for (int k = 0; k < K; ++k) st_masked(rsrc_of(Mout + k * C + c), mine ? (unsigned)xw * 4u : 0x80000000u, 0, dQ[k]);
            } else {
                ne_collide<Sys, Lat>(p, f, bl, dQ, [&](int k, int i, _Float16 v, float e) {
                    post[k][i] = fmaf((float)v, p.inv_scale[k], e);
                });
            }
        }
        if constexpr (NS < T) {                                           // the next stage has not begun
#pragma unroll
            for (int k = 0; k < K; ++k)
#pragma unroll
                for (int i = 0; i < Q; ++i)
                    if (Lat::cy[i] >= 0) wait[slot(NS, k, i, par)] = post[k][i];
            wave_fence();
        }
    };
    constexpr std::integral_constant<int, 0> even{};
    constexpr std::integral_constant<int, 1> odd{};
    load(gi[0], mi[0], true);
    // fill: a stage joins two rows after the one before it
    auto fill = [&](auto self, auto ns) {
        constexpr int NS = decltype(ns)::value;
        if constexpr (NS < T) {
            row(ns, even, 2 * NS);
            row(ns, odd, 2 * NS + 1);
            self(self, std::integral_constant<int, NS + 1>());
        }
    };
    fill(fill, even);
    constexpr std::integral_constant<int, T> all{};
    for (int j = 2 * HALO;; j += 2) {
        row(all, even, j);
        if (j == last) break;
        row(all, odd, j + 1);
        if (j + 1 == last) break;
    }
}

// ---- kernels around the step: initialisation, moments, reductions ----
// A cell's populations are its senders' deviations and equilibria.  TILED: a
// workgroup takes 64 x 4 cells and forms each sender's equilibrium once, in LDS
// (as k_step_ne does).  Else it takes 256 consecutive cells and each forms its
// senders' by itself: three to six times the flux evaluations, but no lane is
// idle on grids narrower than the tiles and nothing waits for a barrier.
constexpr int kNeHX = kNeTX + 2, kNeHY = kNeTY + 2, kNeHalo = kNeHX * kNeHY, kNeThreads = kNeTX * kNeTY;
template <class Sys, bool TILED> constexpr int ne_parts() { return TILED ? Sys::K * 3 * kNeHalo : 1; }

template <class Sys, class Lat, bool TILED>
struct NeCells {
    static constexpr int K = Sys::K, D = Lat::D;
    const KParams<float> &p;
    float *parts;                       // [K][3][kNeHalo]
    int x, y, lx, ly;
    size_t cell;
    bool live;

    // The cells of tile t; moment(k, c): the stored moments of cell c.  Ends with
    // a barrier (TILED).
    template <class Moment>
    __device__ __forceinline__ void enter(unsigned t, Moment &&moment)
    {
        if constexpr (TILED) {
            const unsigned tilesx = (unsigned)(p.nx - 1) / kNeTX + 1;
            const int tx0 = (int)(t % tilesx) * kNeTX, ty0 = (int)(t / tilesx) * kNeTY;
            lx = (int)threadIdx.x % kNeTX;
            ly = (int)threadIdx.x / kNeTX;
            x = tx0 + lx;
            y = ty0 + ly;
            live = x < p.nx && y < p.ny;
            cell = (size_t)y * p.nx + x;
            for (int h = (int)threadIdx.x; h < kNeHalo; h += kNeThreads) {
                const int hy = h / kNeHX, hx = h - hy * kNeHX;
                const size_t c = (size_t)pmod(ty0 + hy - 1, p.ny) * p.nx + pmod(tx0 + hx - 1, p.nx);
                float M[K], P[K][D];
#pragma unroll
                for (int k = 0; k < K; ++k) M[k] = moment(k, c);
                Sys::template flux_delta<float, float>(p.phys, M, P);
#pragma unroll
                for (int k = 0; k < K; ++k) {
                    float G[D], Pt[3];
#pragma unroll
                    for (int a = 0; a < D; ++a) G[a] = p.lam * P[k][a];
                    ExactEq<Lat>::parts(M[k], G, Pt);
#pragma unroll
                    for (int j = 0; j < 3; ++j) parts[(k * 3 + j) * kNeHalo + h] = Pt[j];
                }
            }
            __syncthreads();
        } else {
            cell = (size_t)t * kNeThreads + threadIdx.x;
            live = cell < (size_t)p.C;
            // a 64-bit quotient is a long function
            y = (int)(p.C < 1ll << 32 ? (unsigned)cell / (unsigned)p.nx : cell / (unsigned)p.nx);
            x = (int)(cell - (size_t)y * p.nx);
        }
    }
    // take(k, i, e_i of field k of the sender x - c_i), every field's i in order.
    // TILED: field by field, which keeps one field's values at a time (direction
    // by direction k_moments_ne takes 100 registers in place of 72 for the
    // neo-Hookean D2Q9, one wavefront a SIMD fewer: 171 against 155 us at 2048^2).
    template <class Moment, class Take>
    __device__ __forceinline__ void each(Moment &&moment, Take &&take) const
    {
        if constexpr (TILED) {
#pragma unroll
            for (int k = 0; k < K; ++k) {
                const float *const part = parts + k * 3 * kNeHalo;
#pragma unroll
                for (int i = 0; i < Lat::Q; ++i) {
                    const int h = (ly + 1 - Lat::cy[i]) * kNeHX + (lx + 1 - Lat::cx[i]);
                    const float Pt[3] = {part[h], part[kNeHalo + h], part[2 * kNeHalo + h]};
                    take(k, i, i == 0 ? ExactEq<Lat>::rest_parts(Pt) : ExactEq<Lat>::dir(Pt, i));
                }
            }
        } else {
#pragma unroll
            for (int i = 0; i < Lat::Q; ++i) {
                float e[K];
                sent(i, moment, e);
#pragma unroll
                for (int k = 0; k < K; ++k) take(k, i, e[k]);
            }
        }
    }
    // e_i of the sender x - c_i, every field, from its moments
    template <class Moment>
    __device__ __forceinline__ void sent(int i, Moment &&moment, float *e) const
    {
        const size_t c = (size_t)wrapi(y - Lat::cy[i], p.ny) * p.nx + wrapi(x - Lat::cx[i], p.nx);
        float M[K], P[K][D];
#pragma unroll
        for (int k = 0; k < K; ++k) M[k] = moment(k, c);
        if (i == 0) {
#pragma unroll
            for (int k = 0; k < K; ++k) e[k] = ExactEq<Lat>::rest(M[k]);
            return;
        }
        Sys::template flux_delta<float, float>(p.phys, M, P);
#pragma unroll
        for (int k = 0; k < K; ++k) {
            float G[D], all[Lat::Q];
#pragma unroll
            for (int a = 0; a < D; ++a) G[a] = p.lam * P[k][a];
            ExactEq<Lat>::feq(M[k], 0.0f, G, all);
            e[k] = all[i];
        }
    }
    // before the next tile's enter
    __device__ __forceinline__ static void leave()
    {
        if constexpr (TILED) __syncthreads();
    }
    // the cell's moments, summed in double from its rebuilt populations
    template <class Moment>
    __device__ __forceinline__ void moments(const _Float16 *__restrict__ g, Moment &&moment, double *q) const
    {
        size_t src[Lat::Q];
        pulled_places_of<K, Lat, unsigned long long>(x, y, 0, p.nx, p.ny, 1, src);
#pragma unroll
        for (int k = 0; k < K; ++k) q[k] = 0.0;
        each(moment, [&](int k, int i, float e) __attribute__((always_inline)) {
            q[k] += (double)fmaf((float)g[src[i] + (size_t)(k * Lat::Q * kTile)], p.inv_scale[k], e);
        });
    }
};

// Initial state: M(y) = Q(y) - Q0 rounded to float and, in the pull layout,
// g_i(y) = f*eq_i(Q(y + c_i)) - e_i(M(y)) with the equilibrium of the
// receiver's initial fields in double and e_i(M) as the step kernel forms it.
// A thread is a receiver: it forms its equilibrium once and writes what each of
// its senders stores.  SCALE: only the largest |g| per field of the workgroup,
// to part[k][block]; else the state, and where part is given the largest wave
// speed of the workgroup, from the moments of the values as stored.
// Neo-Hookean 2048^2: 363 + 524 us with the receivers' equilibria formed by
// every sender, and 825 us for the speeds read back.
template <class Sys, class Lat, bool SCALE, bool TILED>
__global__ __launch_bounds__(kNeThreads) void k_init_ne(const double *__restrict__ Qin, _Float16 *__restrict__ g,
                                                        float *__restrict__ M, double *__restrict__ part,
                                                        const KParams<double> pd, const KParams<float> pf, unsigned tiles)
{
    constexpr int K = Sys::K, Q = Lat::Q, D = Lat::D;
    __shared__ float parts[ne_parts<Sys, TILED>()];
    __shared__ double sh[kBlock / 64];
    static_assert(kNeThreads == kBlock, "block reductions");
    const size_t C = (size_t)pd.C;
    NeCells<Sys, Lat, TILED> at = {pf, parts};
    const auto moment = [&](int k, size_t c) { return (float)(Qin[(size_t)k * C + c] - pd.phys.Q0[k]); };
    double mx[K], fastest = 0.0;
#pragma unroll
    for (int k = 0; k < K; ++k) mx[k] = 0.0;
    for (unsigned t = blockIdx.x; t < tiles; t += gridDim.x) {
        at.enter(t, moment);
        if (at.live) {
            double dq[K], P[K][D], q[K];
#pragma unroll
            for (int k = 0; k < K; ++k) dq[k] = Qin[(size_t)k * C + at.cell] - pd.phys.Q0[k];
            Sys::template flux_delta<double, double>(pd.phys, dq, P);
            size_t dst[Q];
            pulled_places_of<K, Lat, unsigned long long>(at.x, at.y, 0, pd.nx, pd.ny, 1, dst);
#pragma unroll
            for (int k = 0; k < K; ++k) q[k] = 0.0;
            at.each(moment, [&](int k, int i, float e) __attribute__((always_inline)) {
                double cd = 0.0;
#pragma unroll
                for (int a = 0; a < D; ++a) cd += lat_c<Lat>(i, a) * P[k][a];
                const double gv = Lat::w[i] * (dq[k] + pd.lam_cs2 * cd) - (double)e;
                if constexpr (SCALE) {
                    mx[k] = fabs(gv) > mx[k] ? fabs(gv) : mx[k];
                } else {
                    const _Float16 v = (_Float16)(gv * (double)pf.scale[k]);
                    g[dst[i] + (size_t)(k * Q * kTile)] = v;
                    q[k] += (double)fmaf((float)v, pf.inv_scale[k], e);
                }
            });
            if constexpr (!SCALE) {
#pragma unroll
                for (int k = 0; k < K; ++k) {
                    M[(size_t)k * C + at.cell] = (float)dq[k];
                    q[k] += pd.phys.Q0[k];
                }
                if (part) {
                    const double v = Sys::template max_speed<double>(pd.phys, q);
                    fastest = v > fastest ? v : fastest;
                }
            }
        }
        at.leave();
    }
    if constexpr (SCALE) {
        for (int k = 0; k < K; ++k) {
            const double r = block_reduce_max(mx[k], sh);
            if (threadIdx.x == 0) part[(size_t)k * gridDim.x + blockIdx.x] = r;
        }
    } else if (part) {
        const double r = block_reduce_max(fastest, sh);
        if (threadIdx.x == 0) part[blockIdx.x] = r;
    }
}

template <class Sys, class Lat, class Out, bool TILED>
__global__ __launch_bounds__(kNeThreads) void k_moments_ne(const _Float16 *__restrict__ g, const float *__restrict__ M,
                                                           Out *__restrict__ out, const KParams<float> p,
                                                           const KParams<double> pd, int absolute)
{
    constexpr int K = Sys::K;
    __shared__ float parts[ne_parts<Sys, TILED>()];
    const size_t C = (size_t)p.C;
    NeCells<Sys, Lat, TILED> at = {p, parts};
    const auto moment = [&](int k, size_t c) { return M[(size_t)k * C + c]; };
    at.enter((unsigned)xcd_tile(blockIdx.x, gridDim.x), moment);
    if (!at.live) return;
    double q[K];
    at.moments(g, moment, q);
#pragma unroll
    for (int k = 0; k < K; ++k) out[(size_t)k * C + at.cell] = (Out)(absolute ? q[k] + pd.phys.Q0[k] : q[k]);
}

template <class Sys, class Lat, bool TILED>
__global__ __launch_bounds__(kNeThreads) void k_reduce1_ne(const _Float16 *__restrict__ g, const float *__restrict__ M,
                                                           const double *__restrict__ ref, double *__restrict__ part,
                                                           const KParams<float> p, const KParams<double> pd, int what,
                                                           unsigned tiles)
{
    constexpr int K = Sys::K, Q = Lat::Q;
    __shared__ float parts[ne_parts<Sys, TILED>()];
    __shared__ double sh[kBlock / 64];
    const size_t C = (size_t)p.C;
    const unsigned nb = gridDim.x;
    if (what == 4) {
        // a wavefront takes a tile of deviations, a lane one cell; then the
        // moments (the padding of the last tile is never read)
        double cnt = 0.0;
        const size_t T = (C + kTile - 1) / kTile, waves = (size_t)nb * (kBlock / 64);
        for (size_t t = (size_t)blockIdx.x * (kBlock / 64) + (threadIdx.x >> 6); t < T; t += waves) {
            const unsigned lane = threadIdx.x & 63u;
            if (t * kTile + lane >= C) continue;
            const _Float16 *cell = g + t * (size_t)(K * Q * kTile) + lane;
            int bad = 0;
#pragma unroll
            for (int j = 0; j < K * Q; ++j) bad += isfinite((float)cell[(size_t)j * kTile]) ? 0 : 1;
            cnt += bad;
        }
        for (size_t j = (size_t)blockIdx.x * kBlock + threadIdx.x; j < (size_t)K * C; j += (size_t)nb * kBlock)
            cnt += isfinite(M[j]) ? 0.0 : 1.0;
        const double r = block_reduce_sum(cnt, sh);
        if (threadIdx.x == 0) part[blockIdx.x] = r;
        return;
    }
    NeCells<Sys, Lat, TILED> at = {p, parts};
    const auto moment = [&](int k, size_t c) { return M[(size_t)k * C + c]; };
    double a0[K], a1[K];
#pragma unroll
    for (int k = 0; k < K; ++k) a0[k] = a1[k] = 0.0;
    for (unsigned t = blockIdx.x; t < tiles; t += nb) {
        at.enter(t, moment);
        if (at.live) {
            double q[K];
            at.moments(g, moment, q);
#pragma unroll
            for (int k = 0; k < K; ++k) q[k] += pd.phys.Q0[k];
            if (what == 0) {
#pragma unroll
                for (int k = 0; k < K; ++k) a0[k] += q[k];
            } else if (what == 1) {
#pragma unroll
                for (int k = 0; k < K; ++k) {
                    const double r = ref[(size_t)k * C + at.cell];
                    a0[k] += (q[k] - r) * (q[k] - r);
                    a1[k] += r * r;
                }
            } else if (what == 2) {
#pragma unroll
                for (int k = 0; k < K; ++k) {
                    const double r = ref[(size_t)k * C + at.cell];
                    const double e = fabs(q[k] - r);
                    a0[k] = e > a0[k] ? e : a0[k];
                    a1[k] = fabs(r) > a1[k] ? fabs(r) : a1[k];
                }
            } else {
                const double sp = Sys::template max_speed<double>(pd.phys, q);
                a0[0] = sp > a0[0] ? sp : a0[0];
            }
        }
        at.leave();
    }
    const int nslot = (what == 3) ? 1 : (what == 0 ? K : 2 * K);
    for (int j = 0; j < nslot; ++j) {
        const double v = j < K ? a0[j] : a1[j - K];
        const double r = (what == 2 || what == 3) ? block_reduce_max(v, sh) : block_reduce_sum(v, sh);
        if (threadIdx.x == 0) part[(size_t)j * nb + blockIdx.x] = r;
    }
}

__global__ __launch_bounds__(kBlock) void k_reduce2_ne(const double *__restrict__ part, double *__restrict__ out,
                                                       int nslot, int nb, int is_max)
{
    __shared__ double sh[kBlock / 64];
    for (int j = blockIdx.x; j < nslot; j += gridDim.x) {
        double v = 0.0;
        for (int b = threadIdx.x; b < nb; b += kBlock) {
            const double w = part[(size_t)j * nb + b];
            v = is_max ? (w > v ? w : v) : v + w;
        }
        const double r = is_max ? block_reduce_max(v, sh) : block_reduce_sum(v, sh);
        if (threadIdx.x == 0) out[j] = r;
    }
}

template <class Sys, class Lat>
struct ImplNE {
    static unsigned step_grid(const lbm_state_impl &h)
    {
        return (unsigned)(((h.nx + kNeTX - 1) / kNeTX) * (long long)((h.ny + kNeTY - 1) / kNeTY));
    }
    static const _Float16 *gp(const lbm_state_impl &, const void *buf) { return (const _Float16 *)buf; }
    static const float *mp(const lbm_state_impl &h, const void *buf)
    {
        return (const float *)((const char *)buf + ne_pop_bytes(h.C, Sys::K, Lat::Q));
    }

    template <bool NT, bool O32>
    static void launch(const lbm_state_impl &h, const void *fin, void *fout, const KParams<float> &p, hipStream_t s)
    {
        hipLaunchKernelGGL((k_step_ne<Sys, Lat, NT, O32>), dim3(step_grid(h)), dim3(kNeTX * kNeTY), 0, s, gp(h, fin),
                           mp(h, fin), (_Float16 *)fout, (float *)mp(h, fout), p);
    }
    static hipError_t step(const lbm_state_impl &h, const void *fin, void *fout, void *qhist, hipStream_t s)
    {
        if (qhist) return hipErrorInvalidValue;
        const KParams<float> p = h.kparams<float>(h.t0 + (h.nsteps + 0.5) * h.dt);
        const bool nt = 2 * (ne_pop_bytes(h.C, Sys::K, Lat::Q) + (size_t)Sys::K * h.C * 4) > kLastLevelCacheBytes;
        // 32-bit byte offsets when the deviations stay below 4 GiB
        const bool o32 = ne_pop_bytes(h.C, Sys::K, Lat::Q) <= 0xffffffffull;
        if (nt)
            o32 ? launch<true, true>(h, fin, fout, p, s) : launch<true, false>(h, fin, fout, p, s);
        else
            o32 ? launch<false, true>(h, fin, fout, p, s) : launch<false, false>(h, fin, fout, p, s);
        return hipGetLastError();
    }
    // several steps per launch (k_march_ne) where that pays (march_plan.hpp)
    static constexpr int kMost = ne_march_most<Sys, Lat>();
    static int steps_per_launch(const lbm_state_impl &h, int want, int run)
    {
        const StepState s = {3, Sys::K, Lat::Q, false, h.field_b != nullptr};
        return march_steps(s, kMost, ne_march_lds<Sys, Lat>(kMost), ne_march_lds<Sys, Lat>(2), [](int T) { return T; }, want,
                           run, h.nx, h.ny);
    }
    template <int T>
    static hipError_t launch_march(const lbm_state_impl &h, const void *fin, void *fout, hipStream_t s)
    {
        const KParams<float> p = h.kparams<float>(h.t0);
        const int strips = march_strips(T, h.nx);
        const int rows = march_rows(T, ne_march_lds<Sys, Lat>(T), Sys::K * Lat::Q, h.nx, h.ny);
        const dim3 blocks((unsigned)(strips * march_segments(h.ny, rows)));
        auto go = [&](auto kern) {
            hipLaunchKernelGGL(kern, blocks, dim3(64), 0, s, gp(h, fin), mp(h, fin), (_Float16 *)fout,
                               (float *)mp(h, fout), p, rows, strips);
        };
        h.field_b ? go(k_march_ne<Sys, Lat, T, true>) : go(k_march_ne<Sys, Lat, T, false>);
        return hipGetLastError();
    }
    static hipError_t multi(const lbm_state_impl &h, int steps, const void *fin, void *fout, void *qhist, hipStream_t s)
    {
        if (qhist) return hipErrorInvalidValue;
        if constexpr (kMost >= 2)
            if (steps == 2) return launch_march<2>(h, fin, fout, s);
        if constexpr (kMost > 2)
            if (steps == kMost) return launch_march<kMost>(h, fin, fout, s);
        return hipErrorInvalidValue;
    }
    static void combine(double *part, int nslot, unsigned nb, int is_max, hipStream_t s)
    {
        hipLaunchKernelGGL(k_reduce2_ne, dim3(nslot), dim3(kBlock), 0, s, part, part + (size_t)2 * LBM_MAXK * kRedBlocks,
                           nslot, (int)nb, is_max);
    }
    // Tiles of a kernel around the step (TILED), or its runs of 256 cells.  Tiles
    // pay where they save D2Q9's eight flux evaluations and are at least four
    // fifths full: below, idle lanes take what they save (cells / tiles, us:
    // moments of shallow water D2Q9 1500^2 51 / 34, 20000 x 65 32 / 36, 200^2 6.7 /
    // 8.3; initialisation of neo-Hookean D2Q9 200000 x 1 167 / 1942), and where
    // every CU has one or the state is large (64^2: 6.0 / 6.6).  D2Q5's four
    // evaluations are as fast as the barrier and the LDS they would save, except
    // for the moments of three to six fields (neo-Hookean 700^2 18.2 / 15.2; sums
    // of the 7-field flow 1000 x 1100 72 / 113).
    struct Around {
        bool tiled;
        unsigned tiles;
    };
    static constexpr bool kTiledMoments = Sys::K > 1 && (Lat::Q == 9 || (Sys::K >= 3 && Sys::K <= 6));
    static constexpr bool kTiled = Sys::K > 1 && Lat::Q == 9;
    static Around around(const lbm_state_impl &h, bool may)
    {
        const long long tiles = (long long)((h.nx - 1) / kNeTX + 1) * ((h.ny - 1) / kNeTY + 1);
        const long long runs = (h.C + kNeThreads - 1) / kNeThreads;
        const bool tiled = may && 5 * h.C >= 4 * kNeThreads * tiles && tiles < 1ll << 24 && (tiles >= kSimds / 4 || Sys::K >= 6);
        return {tiled, (unsigned)(tiled ? tiles : runs)};
    }
    static hipError_t init(const lbm_state_impl &h, const double *Q, void *fout, double *speed, hipStream_t s)
    {
        const Around a = around(h, kTiled);
        const unsigned nb = std::min(a.tiles, (unsigned)kInitBlocks);
        auto go = [&](auto kern) {
            hipLaunchKernelGGL(kern, dim3(nb), dim3(kNeThreads), 0, s, Q, (_Float16 *)fout, (float *)mp(h, fout), speed,
                               h.kparams<double>(h.t0), h.kparams<float>(h.t0), a.tiles);
        };
        a.tiled ? go(k_init_ne<Sys, Lat, false, kTiled>) : go(k_init_ne<Sys, Lat, false, false>);
        if (speed) combine(speed, 1, nb, 1, s);
        return hipGetLastError();
    }
    static hipError_t init_absmax(const lbm_state_impl &h, const double *Q, double *part, hipStream_t s)
    {
        const Around a = around(h, kTiled);
        const unsigned nb = std::min(a.tiles, (unsigned)(2 * kRedBlocks));
        auto go = [&](auto kern) {
            hipLaunchKernelGGL(kern, dim3(nb), dim3(kNeThreads), 0, s, Q, (_Float16 *)nullptr, (float *)nullptr, part,
                               h.kparams<double>(h.t0), h.kparams<float>(h.t0), a.tiles);
        };
        a.tiled ? go(k_init_ne<Sys, Lat, true, kTiled>) : go(k_init_ne<Sys, Lat, true, false>);
        combine(part, Sys::K, nb, 1, s);
        return hipGetLastError();
    }
    static hipError_t moments(const lbm_state_impl &h, const void *fin, void *out, int absolute, int out_dtype,
                              hipStream_t s)
    {
        const Around a = around(h, kTiledMoments);
        auto go = [&](auto kern, auto *to) {
            hipLaunchKernelGGL(kern, dim3(a.tiles), dim3(kNeThreads), 0, s, gp(h, fin), mp(h, fin), to,
                               h.kparams<float>(h.t0), h.kparams<double>(h.t0), absolute);
        };
        if (out_dtype == 0)
            a.tiled ? go(k_moments_ne<Sys, Lat, double, kTiledMoments>, (double *)out)
                    : go(k_moments_ne<Sys, Lat, double, false>, (double *)out);
        else
            a.tiled ? go(k_moments_ne<Sys, Lat, float, kTiledMoments>, (float *)out)
                    : go(k_moments_ne<Sys, Lat, float, false>, (float *)out);
        return hipGetLastError();
    }
    static hipError_t reduce(const lbm_state_impl &h, const void *fin, int what, const double *ref, double *aux,
                             hipStream_t s)
    {
        const int nslot = (what == 3 || what == 4) ? 1 : (what == 0 ? Sys::K : 2 * Sys::K);
        const int is_max = (what == 2 || what == 3) ? 1 : 0;
        const Around a = around(h, kTiled);
        const unsigned nb = std::min(a.tiles, (unsigned)std::min(2 * kRedBlocks, 2 * LBM_MAXK * kRedBlocks / nslot));
        auto go = [&](auto kern) {
            hipLaunchKernelGGL(kern, dim3(nb), dim3(kNeThreads), 0, s, gp(h, fin), mp(h, fin), ref, aux,
                               h.kparams<float>(h.t0), h.kparams<double>(h.t0), what, a.tiles);
        };
        a.tiled ? go(k_reduce1_ne<Sys, Lat, kTiled>) : go(k_reduce1_ne<Sys, Lat, false>);
        combine(aux, nslot, nb, is_max, s);
        return hipGetLastError();
    }
    static const Launchers *get()
    {
        static const Launchers L = {Sys::K, Lat::Q, Lat::D, 2, steps_per_launch, step, multi, init, init_absmax, moments,
                                    reduce, nullptr, nullptr, nullptr};
        return &L;
    }
};

const Launchers *lbm_launchers_ne(int sys, int lat)
{
    switch (sys) {
    case SYS_SWE:
        if (lat == LAT_D2Q5) return ImplNE<SysSWE, D2Q5>::get();
        if (lat == LAT_D2Q9) return ImplNE<SysSWE, D2Q9>::get();
        break;
    case SYS_ADVDIFF:
        if (lat == LAT_D2Q5) return ImplNE<SysAdvDiff, D2Q5>::get();
        if (lat == LAT_D2Q9) return ImplNE<SysAdvDiff, D2Q9>::get();
        break;
    case SYS_NEOHOOKE:
        if (lat == LAT_D2Q5) return ImplNE<SysNeoHooke, D2Q5>::get();
        if (lat == LAT_D2Q9) return ImplNE<SysNeoHooke, D2Q9>::get();
        break;
    case SYS_BURGERS:
        if (lat == LAT_D2Q5) return ImplNE<SysBurgers, D2Q5>::get();
        if (lat == LAT_D2Q9) return ImplNE<SysBurgers, D2Q9>::get();
        break;
    case SYS_EULER:
        if (lat == LAT_D2Q5) return ImplNE<SysEuler, D2Q5>::get();
        if (lat == LAT_D2Q9) return ImplNE<SysEuler, D2Q9>::get();
        break;
    case SYS_MAXWELL:
        if (lat == LAT_D2Q5) return ImplNE<SysMaxwell, D2Q5>::get();
        if (lat == LAT_D2Q9) return ImplNE<SysMaxwell, D2Q9>::get();
        break;
    case SYS_ALLENCAHN:
        if (lat == LAT_D2Q5) return ImplNE<SysAllenCahn, D2Q5>::get();
        if (lat == LAT_D2Q9) return ImplNE<SysAllenCahn, D2Q9>::get();
        break;
    case SYS_RELHYDRO:
        if (lat == LAT_D2Q5) return ImplNE<SysRelHydro, D2Q5>::get();
        if (lat == LAT_D2Q9) return ImplNE<SysRelHydro, D2Q9>::get();
        break;
    case SYS_NSE:
        if (lat == LAT_D2Q5) return ImplNE<SysNSE, D2Q5>::get();
        if (lat == LAT_D2Q9) return ImplNE<SysNSE, D2Q9>::get();
        break;
    case SYS_CNSF2D:
        if (lat == LAT_D2Q5) return ImplNE<SysCNSF2D, D2Q5>::get();
        break;
    }
    return nullptr;
}
