// Several collide-and-stream steps of a 2D grid in one launch.
//
// A step by itself moves every population through HBM once each way, and the
// 2D steps spend their time on that.  Here a wavefront marches up a strip of
// 64 columns, row by row: stage 1 pulls a row of populations from the buffer
// and collides it, stage 2 collides the row below from the stage-1 rows
// around it, and so on; only the last stage's rows are stored, T steps on.
// The intermediate rows live on the chip: a population moving up waits two
// rows and one moving along the row waits one, in this wavefront's own part
// of LDS, where a neighbouring column is a neighbouring word; one moving down
// is used at once, pulled from the neighbouring lane by a wave-wide DPP shift.
// Wavefronts share nothing and meet no barrier.
//
// Price: T - 1 lanes at each end of the strip and T - 1 rows at each end of
// the march are computed but not stored (stage t needs T - t of them), so a
// wavefront stores 64 - 2 (T - 1) columns of every row of its segment.  Those
// are no whole cache lines: the stores are plain ones, so that L2 joins the
// parts of two strips (non-temporal stores: 19% slower at 2048^2).
//
// Bound: with one or two wavefronts a SIMD the vector units issue for about
// two thirds of the time (shallow water 2048^2, four stages: 40 of 61 us per
// step); the rest is the partial cache lines' stores (misaligned stores alone
// cost 18 us at three stages, misaligned loads nothing).
#pragma once

#include "collide.hpp"
#include "march_plan.hpp"

static_assert(kTile == kMarchLanes, "a strip is a tile wide");

// The value of lane l - 1 (C = +1) or l + 1 (C = -1); zero past the ends.
template <int C>
__device__ __forceinline__ float lane_pull(float v)
{
    if constexpr (C == 0) return v;
    return __int_as_float(__builtin_amdgcn_mov_dpp(__float_as_int(v), C > 0 ? 0x138 : 0x130, 0xf, 0xf, true));
}
template <int C>
__device__ __forceinline__ double lane_pull(double v)
{
    if constexpr (C == 0) return v;
    return __hiloint2double(__builtin_amdgcn_mov_dpp(__double2hiint(v), C > 0 ? 0x138 : 0x130, 0xf, 0xf, true),
                            __builtin_amdgcn_mov_dpp(__double2loint(v), C > 0 ? 0x138 : 0x130, 0xf, 0xf, true));
}
template <class Lat, class F>
__device__ __forceinline__ F lane_pull(F v, int i)      // i a constant after unrolling
{
    return Lat::cx[i] > 0 ? lane_pull<1>(v) : (Lat::cx[i] < 0 ? lane_pull<-1>(v) : v);
}

// Buffer descriptor of the 2^31 - 1 bytes from base on (march_fits keeps a
// row within them): offsets at and beyond 2^31 are out of range for every access.
__device__ __forceinline__ __amdgpu_buffer_rsrc_t rsrc_of(const void *base)
{
    return __builtin_amdgcn_make_buffer_rsrc((void *)base, 0, 0x7fffffff, 0x00027000);
}

// A cell's coefficients, already loaded, and the reader of its explicit source
// (see CellFields).
template <class F, bool EXT>
struct RowFields {
    static constexpr bool ext = EXT;
    const F *cb, *cs;
    size_t C, cell;
    __device__ F b(int a) const { return cb[a]; }
    __device__ F s(int k) const { return cs[k * C + cell]; }
};

// A buffer store whose lanes with off >= 2^31 are dropped by the range check,
// so the marching loop has no branch around its stores.
template <class T>
__device__ __forceinline__ void st_masked(__amdgpu_buffer_rsrc_t r, unsigned off, int base, T v)
{
    constexpr int aux = 0;
    if constexpr (sizeof(T) == 8) {
        typedef int v2 __attribute__((ext_vector_type(2)));
        __builtin_amdgcn_raw_buffer_store_b64(__builtin_bit_cast(v2, v), r, off, base, aux);
    } else if constexpr (sizeof(T) == 4) {
        __builtin_amdgcn_raw_buffer_store_b32(__builtin_bit_cast(int, v), r, off, base, aux);
    } else {
        __builtin_amdgcn_raw_buffer_store_b16(__builtin_bit_cast(short, v), r, off, base, aux);
    }
}

// A load through a buffer descriptor: uniform base, one 32-bit offset per lane.
template <class T>
__device__ __forceinline__ T ld_buf(__amdgpu_buffer_rsrc_t r, unsigned off, int base)
{
    if constexpr (sizeof(T) == 8)
        return __builtin_bit_cast(T, __builtin_amdgcn_raw_buffer_load_b64(r, off, base, 0));
    else if constexpr (sizeof(T) == 4)
        return __builtin_bit_cast(T, __builtin_amdgcn_raw_buffer_load_b32(r, off, base, 0));
    else
        return __builtin_bit_cast(T, __builtin_amdgcn_raw_buffer_load_b16(r, off, base, 0));
}

// Keeps the compiler from moving LDS accesses of one lane across those of
// others in the wavefront (which executes them in order).
__device__ __forceinline__ void wave_fence()
{
    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront", "local");
    __builtin_amdgcn_wave_barrier();
}

// Populations of a field that wait between two stages, and the LDS that a
// wavefront of T stages keeps.
template <class Lat> constexpr int march_slots() { return Lat::Q == 9 ? 9 : 5; }
template <class Sys, class Lat, class St>
constexpr int march_lds(int T) { return ((T - 1) * march_slots<Lat>() * Sys::K * 64 + 2) * (int)sizeof(St); }

// Steps per launch of a large grid: four, where that leaves seven wavefronts
// a CU their LDS, else three or two.  Shallow water 2048^2, D2Q9, float, us
// per step: 152 one step per launch, 120, 86, 61 two, three and four; five
// (five wavefronts a CU) 66.
template <class Sys, class Lat, class St>
constexpr int march_most()
{
    int T = 4;
    while (T > 2 && 7 * march_lds<Sys, Lat, St>(T) > kLdsPerCu) --T;
    return T;
}

// Whether two stages leave eight wavefronts a CU (two a SIMD) their LDS, and
// a state fits the registers of two wavefronts a SIMD.
template <class Sys, class Lat, class St>
constexpr bool marches()
{
    return Lat::D == 2 && Sys::K <= 7 && 8 * march_lds<Sys, Lat, St>(2) <= kLdsPerCu;
}

template <class Sys, class Lat, class St, int T, bool EXT, bool REC, int COLL>
__global__ __launch_bounds__(64) void k_march(const St *__restrict__ fin, St *__restrict__ fout,
                                              const KParams<typename Cell<Sys, Lat, St, COLL>::P> p,
                                              typename Store<St>::R *__restrict__ qhist, int rows, int strips)
{
    using C = Cell<Sys, Lat, St, COLL>;
    using F = typename Store<St>::R;
    constexpr int K = Sys::K, Q = Lat::Q, KQ = K * Q;
    constexpr int HALO = T - 1, WOUT = 64 - 2 * HALO;
    const int lane = (int)threadIdx.x;                                    // one wavefront per workgroup
    const unsigned g = (unsigned)xcd_tile(blockIdx.x, gridDim.x);
    const int strip = (int)(g % (unsigned)strips);
    const int y0 = (int)(g / (unsigned)strips) * rows, y1 = segment_end(y0, rows, p.ny);
    const int xo = strip * WOUT + lane - HALO;                            // unwrapped column
    const bool mine = lane >= HALO && lane < 64 - HALO && xo < p.nx;      // column stored by this lane
    int xw = xo % p.nx;
    xw = xw < 0 ? xw + p.nx : xw;
    const int xs[3] = {wrapi(xw - 1, p.nx), xw, wrapi(xw + 1, p.nx)};

    // Offsets of a row: its first cell y nx lies b cells into tile a; the
    // tile's part is uniform, a lane's part stays below 2^31.
    struct Row {
        size_t base;            // elements to tile a
        unsigned b;             // y nx - 64 a
    };
    auto row_of = [&](int y) {
        const size_t c = (size_t)y * (size_t)p.nx;
        return Row{c / kTile * (size_t)(KQ * kTile), (unsigned)(c % kTile)};
    };
    auto lane_off = [&](const Row &r, int x) { return tile_offset<K, Q>(r.b + (unsigned)x) * (unsigned)sizeof(St); };

    // the row that stage 1 loads next
    int yn = (y0 - HALO) % p.ny;
    yn = yn < 0 ? yn + p.ny : yn;
    const int last = y1 - y0 + 2 * HALO - 1;
    // Two rows of populations: one at work, the next on its way from memory.
    // The march alternates between them, so that no register copy waits for
    // the loads; past the last row it loads that row again.
    St in[2][K][Q];
    // With EXT the coefficients of every stage's next row come along: read
    // where they are used, each stage would wait for memory once a row (shallow
    // water 512^2 with topography: 35.5 -> 32.7 us per four steps).  Without an
    // attached field the loads take populations, which nobody uses.
    constexpr int NC = EXT && Sys::id == SYS_SWE ? CoefTraits<Sys>::NB : 0;
    const F *const coef = p.b ? (const F *)p.b : (const F *)fin;
    F cf[2][T][2];
    int yc = yn;                                                          // stage 1's row, wrapped
    auto below = [&](int y, int s) {                                      // y - s wrapped, s < T <= 4
        y -= s;
#pragma unroll
        for (int n = 1; n < T; ++n) y = y < 0 ? y + p.ny : y;
        return y;
    };
    auto load_coef = [&](F (&to)[T][2], int first) {
#pragma unroll
        for (int s = 0; s < T; ++s) {
            const int y = below(first, s);
#pragma unroll
            for (int a = 0; a < NC; ++a)
                to[s][a] = ld_buf<F>(rsrc_of(coef + a * (size_t)p.C + (size_t)y * (size_t)p.nx),
                                     (unsigned)xw * (unsigned)sizeof(F), 0);
        }
    };
    auto load = [&](St (&to)[K][Q], bool more) {
        const Row rw[3] = {row_of(wrapi(yn - 1, p.ny)), row_of(yn), row_of(wrapi(yn + 1, p.ny))};
#pragma unroll
        for (int i = 0; i < Q; ++i) {
            const Row &r = rw[1 - Lat::cy[i]];
            const auto rs = rsrc_of(fin + r.base);
            const unsigned off = lane_off(r, xs[1 - Lat::cx[i]]);
#pragma unroll
            for (int k = 0; k < K; ++k) to[k][i] = ld_buf<St>(rs, off, (k * Q + i) * kTile * (int)sizeof(St));
        }
        yn = more ? wrapi(yn + 1, p.ny) : yn;
    };
    // Stage s's populations on their way: slots of 64 words, two rows of those
    // moving up (by the row's parity), then those moving along the row.  Lane
    // 0's left and lane 63's right neighbour are other slots' words: lanes at
    // the ends are not stored.
    constexpr int NU = Lat::Q == 9 ? 3 : 1, NW = march_slots<Lat>();
    static_assert(NW == 2 * NU + 3, "two rows of those moving up, one of those along it");
    __shared__ St carry[march_lds<Sys, Lat, St>(T) / sizeof(St)];
    St *const wait = &carry[1 + lane];
    // slot of population i of field k after stage s, parity of its row
    constexpr auto slot = [](int s, int k, int i, int par) {
        int n = Lat::cy[i] > 0 ? par * NU : 2 * NU;
        for (int j = 0; j < i; ++j) n += Lat::cy[j] == Lat::cy[i];
        return ((s * NW + n) * K + k) * 64;
    };
    // one row of the march with the first NS stages at work; the last stage of
    // a full march stores row y0 + j - 2 HALO
    auto row = [&](auto ns, auto parity, int j) {
        constexpr int NS = decltype(ns)::value, par = decltype(parity)::value;
        F f[K][Q];
        load(in[par ^ 1], j + 1 < last);
        load_coef(cf[par ^ 1], wrapi(yc + 1, p.ny));
        __builtin_amdgcn_sched_barrier(0);
#pragma unroll
        for (int k = 0; k < K; ++k)
#pragma unroll
            for (int i = 0; i < Q; ++i) f[k][i] = (F)in[par][k][i];
#pragma unroll
        for (int s = 0; s < NS; ++s) {
            const int yu = y0 - HALO + j - s;                             // this stage's row, unwrapped
            const int y = EXT || REC ? below(yc, s) : yu;
            const RowFields<F, EXT> ex = {cf[par][s], (const F *)p.sext, (size_t)p.C,
                                          (size_t)y * (size_t)p.nx + (unsigned)xw};
            F dQ[K];
            St post[K][Q];
            if (s == HALO) {                                              // rows y0 to y1 only: none wraps
                const Row out = row_of(yu);
                const auto rs = rsrc_of(fout + out.base);
                const unsigned off = mine ? lane_off(out, xw) : 0x80000000u;
                C::update(p, f, ex, nullptr, dQ, [&](int k, int i, St v) {
                    st_masked(rs, off, (k * Q + i) * kTile * (int)sizeof(St), v);
                });
            } else {
                C::update(p, f, ex, nullptr, dQ, [&](int k, int i, St v) { post[k][i] = v; });
                // read what the rows below left before this row takes its place
#pragma unroll
                for (int k = 0; k < K; ++k)
#pragma unroll
                    for (int i = 0; i < Q; ++i)
                        f[k][i] = Lat::cy[i] < 0 ? lane_pull<Lat>((F)post[k][i], i)
                                                 : (F)wait[slot(s, k, i, par) - Lat::cx[i]];
                wave_fence();
#pragma unroll
                for (int k = 0; k < K; ++k)
#pragma unroll
                    for (int i = 0; i < Q; ++i)
                        if (Lat::cy[i] >= 0) wait[slot(s, k, i, par)] = post[k][i];
                wave_fence();
            }
            if constexpr (REC) {
                const unsigned off = mine && yu >= y0 && yu < y1 ? (unsigned)xw * (unsigned)sizeof(F) : 0x80000000u;
#pragma unroll
                for (int k = 0; k < K; ++k)
                    st_masked(rsrc_of(qhist + (s * (size_t)K + k) * (size_t)p.C + (size_t)y * (size_t)p.nx), off, 0, dQ[k]);
            }
        }
        yc = wrapi(yc + 1, p.ny);
    };
    constexpr std::integral_constant<int, 0> even{};
    constexpr std::integral_constant<int, 1> odd{};
    load(in[0], true);
    load_coef(cf[0], yc);
    // fill: stage s + 1 joins two rows after stage s
    auto fill = [&](auto self, auto ns) {
        constexpr int NS = decltype(ns)::value;
        if constexpr (NS < T) {
            row(ns, even, 2 * NS - 2);
            row(ns, odd, 2 * NS - 1);
            self(self, std::integral_constant<int, NS + 1>());
        }
    };
    fill(fill, std::integral_constant<int, 1>());
    constexpr std::integral_constant<int, T> all{};
    for (int j = 2 * HALO;; j += 2) {
        row(all, even, j);
        if (j == last) break;
        row(all, odd, j + 1);
        if (j + 1 == last) break;
    }
}

// ---------------------------------------------------------- small grids ----
// On a grid that leaves most of the chip idle a step's time is the launch and
// one cell's chain of loads and arithmetic.  Here a workgroup takes a square of
// kSquare^2 cells, one per thread (a wavefront per SIMD), through `steps`
// steps: the populations pass between the threads through LDS, and the middle
// cells of the square, steps - 1 away from its edge, are stored (after t steps
// a cell t - 1 away from the edge is right; the others hold what is used by
// nobody).
//
// Bound: latency.  A launch takes about 2.5 us beside its steps (kernel start,
// addresses, loads, stores) and a step 1 us (a double chain of about 400
// instructions of one wavefront, LDS, two barriers).  Neighbouring squares run
// on one XCD, so that most of a square's loads hit the L2 that the last launch
// wrote (in dispatch order: 150 x 101 2.13 against 1.65 us per step, 160^2 2.72
// against 1.70).  us per step with 1 (k_step) / 2 / 3 / 4 / 5 / 6 / 7 steps a
// launch: shallow water 64^2, D2Q9, float 2.9 / 2.35 / 1.89 / 1.64 / 1.43 /
// 1.43 / 1.39; advection-diffusion 64^2, D2Q5, double 3.2 / 2.56 / 2.14 / 1.91
// / 1.72 / 1.70 / 1.67.
constexpr int kSquare = 16;
constexpr int kSquareMost = 5;
inline int square_out(int steps) { return kSquare - 2 * (steps - 1); }
// Whether a square's moving populations fit 64 KiB of LDS.
template <class Sys, class Lat, class St>
constexpr bool squares()
{
    return marches<Sys, Lat, St>()
           && (Sys::K * (Lat::Q - 1) * kSquare * kSquare + 2 * (kSquare + 1)) * (int)sizeof(St) <= 64 * 1024;
}

template <class Sys, class Lat, class St, bool EXT, bool REC, int COLL>
__global__ __launch_bounds__(kSquare * kSquare) void k_square(const St *__restrict__ fin, St *__restrict__ fout,
                                                              const KParams<typename Cell<Sys, Lat, St, COLL>::P> p,
                                                              typename Store<St>::R *__restrict__ qhist, int steps,
                                                              int across)
{
    using C = Cell<Sys, Lat, St, COLL>;
    using F = typename Store<St>::R;
    constexpr int K = Sys::K, Q = Lat::Q, W = kSquare, N = W * W;
    const int halo = steps - 1, out = W - 2 * halo;
    const int tid = (int)threadIdx.x, lx = tid % W, ly = tid / W;
    const int g = (int)xcd_tile(blockIdx.x, gridDim.x);
    const int xu = g % across * out - halo + lx, yu = g / across * out - halo + ly;
    const bool mine = lx >= halo && lx < W - halo && ly >= halo && ly < W - halo && xu < p.nx && yu < p.ny;
    int x = xu % p.nx, y = yu % p.ny;
    x = x < 0 ? x + p.nx : x;
    y = y < 0 ? y + p.ny : y;
    const unsigned cell = (unsigned)y * (unsigned)p.nx + (unsigned)x;
    F f[K][Q];
#pragma unroll
    for (int i = 0; i < Q; ++i) {
        const int xs = wrapi(x - Lat::cx[i], p.nx), ys = wrapi(y - Lat::cy[i], p.ny);
        const unsigned off = tile_offset<K, Q>((unsigned)ys * (unsigned)p.nx + (unsigned)xs) * (unsigned)sizeof(St);
#pragma unroll
        for (int k = 0; k < K; ++k) f[k][i] = Store<St>::ld(byte_at(fin + (k * Q + i) * kTile, off));
    }
    constexpr int NB = CoefTraits<Sys>::NB > 0 ? CoefTraits<Sys>::NB : 1;
    F cf[NB];
    if (EXT && p.b) {
#pragma unroll
        for (int a = 0; a < CoefTraits<Sys>::NB; ++a) cf[a] = ((const F *)p.b)[a * (size_t)p.C + cell];
    }
    const RowFields<F, EXT> ex = {cf, (const F *)p.sext, (size_t)p.C, (size_t)cell};
    __shared__ St mid[K * (Q - 1) * N + 2 * (W + 1)];                     // a neighbour's word is in bounds for every thread
    St *const here = &mid[W + 1 + tid];
    St post[K][Q];
    for (int s = 0;; ++s) {
        F dQ[K];
        C::update(p, f, ex, nullptr, dQ, [&](int k, int i, St v) { post[k][i] = v; });
        if constexpr (REC) {
            if (mine) {
#pragma unroll
                for (int k = 0; k < K; ++k) qhist[(s * (size_t)K + k) * (size_t)p.C + cell] = dQ[k];
            }
        }
        if (s == halo) break;
#pragma unroll
        for (int k = 0; k < K; ++k)
#pragma unroll
            for (int i = 1; i < Q; ++i) here[(k * (Q - 1) + i - 1) * N] = post[k][i];
        __syncthreads();
#pragma unroll
        for (int k = 0; k < K; ++k) {
            f[k][0] = (F)post[k][0];
#pragma unroll
            for (int i = 1; i < Q; ++i)
                f[k][i] = (F)here[(k * (Q - 1) + i - 1) * N - Lat::cx[i] - W * Lat::cy[i]];
        }
        __syncthreads();
    }
    if (mine) {
        const unsigned own = tile_offset<K, Q>(cell) * (unsigned)sizeof(St);
#pragma unroll
        for (int k = 0; k < K; ++k)
#pragma unroll
            for (int i = 0; i < Q; ++i) *byte_at(fout + (k * Q + i) * kTile, own) = post[k][i];
    }
}
