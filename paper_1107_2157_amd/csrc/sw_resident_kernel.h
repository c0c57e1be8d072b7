// The resident time loop: every step of a call in one launch, the state of
// the grid in registers from the first step to the last.
//
// A grid belongs to a team of workgroups (all of them resident at once, see
// sw_resident.cpp).  A wave holds a patch of up to R rows by 62 columns in
// registers, one column per lane and a halo column in the lanes beside them.
// Per step it marches up its rows with the fused kernel's arithmetic
// (sw_tile.h), operation for operation, so the states are bitwise those of
// the per-step launches.
// Between two steps only what a neighbour needs moves:
//   rows      between waves of a workgroup through LDS, between workgroups
//             through memory;
//   columns   (the patch's first and last) through memory;
//   max speed one word per workgroup, read by every workgroup of the team.
// A word in memory is 8 bytes, 32 bits of value and a 32-bit tag that names
// the step, written and read with relaxed device-scope atomics: a reader
// polls the word it needs until its tag is right, so one trip through memory
// orders and carries the data, no fence or counter is needed and no cache is
// written back or invalidated.  Words are doubled by step parity: a workgroup
// overwrites a word two steps later, when it has seen the reader's word of
// the step between, which the reader wrote after it had read.
#pragma once
#include "sw_resident.h"
#include "sw_tile_tr.h"

#include <utility>

using namespace sw;
using namespace sw::tile;

namespace {

typedef unsigned long long u64;

// On the kernel's lambdas: inlined before any other optimisation, so that the
// patch is split into registers before its rows are selected by address.
#define SW_INLINE __attribute__((always_inline))

__device__ __forceinline__ void put(u64 *p, u64 v) { __hip_atomic_store(p, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT); }
__device__ __forceinline__ u64 get(const u64 *p) { return __hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT); }

template <typename T> constexpr int words_of() { return sizeof(T) / 4; }
__device__ __forceinline__ void put_value(char *p, unsigned tag, float v) {
    put((u64 *)p, ((u64)tag << 32) | __float_as_uint(v));
}
__device__ __forceinline__ void put_value(char *p, unsigned tag, double v) {
    put((u64 *)p, ((u64)tag << 32) | (unsigned)__double2loint(v));
    put((u64 *)p + 1, ((u64)tag << 32) | (unsigned)__double2hiint(v));
}
// The words of the value at p, to be looked at later (several polls are then in flight at once).
template <typename T> struct Words { u64 w[words_of<T>()]; };
template <typename T> __device__ __forceinline__ Words<T> get_words(const char *p) {
    Words<T> r;
#pragma unroll
    for (int k = 0; k < words_of<T>(); ++k) r.w[k] = get((const u64 *)p + k);
    return r;
}
__device__ __forceinline__ bool is_tagged(const Words<float> &r, unsigned tag) { return (unsigned)(r.w[0] >> 32) == tag; }
__device__ __forceinline__ bool is_tagged(const Words<double> &r, unsigned tag) {
    return (unsigned)(r.w[0] >> 32) == tag && (unsigned)(r.w[1] >> 32) == tag;
}
__device__ __forceinline__ float value_of(const Words<float> &r) { return __uint_as_float((unsigned)r.w[0]); }
__device__ __forceinline__ double value_of(const Words<double> &r) {
    return __hiloint2double((int)(unsigned)r.w[1], (int)(unsigned)r.w[0]);
}

// Lane l receives x from lane l + 1 / l - 1; the wave's edge lane, never an
// owned cell, receives 0 (in FP32 the move then folds into its consumer).
__device__ __forceinline__ float next_lane(float x) {
    return __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(x), 0x130, 0xf, 0xf, true));
}
__device__ __forceinline__ float prev_lane(float x) {
    return __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(x), 0x138, 0xf, 0xf, true));
}
__device__ __forceinline__ double next_lane(double x) { return from_next_lane(x, x); }
__device__ __forceinline__ double prev_lane(double x) { return from_prev_lane(x, x); }

// The larger of a and b, b where a is not a number (one instruction in
// FP32: fmax would first quiet the carried operand).
__device__ __forceinline__ float max_of(float a, float b) { return __builtin_amdgcn_fmed3f(a, b, __builtin_inff()); }
__device__ __forceinline__ double max_of(double a, double b) { return fmax(a, b); }

// Wave-wide maximum of non-negative values, in every lane (uniform): lane
// moves by DPP (a shuffle through LDS takes several times as long, and the
// step waits for this one).
template <int CTRL> __device__ __forceinline__ float dpp_move(float x) {
    return __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(x), CTRL, 0xf, 0xf, true));
}
template <int CTRL> __device__ __forceinline__ double dpp_move(double x) {
    return __hiloint2double(__builtin_amdgcn_update_dpp(0, __double2hiint(x), CTRL, 0xf, 0xf, true),
                            __builtin_amdgcn_update_dpp(0, __double2loint(x), CTRL, 0xf, 0xf, true));
}
__device__ __forceinline__ float lane63(float x) { return __int_as_float(__builtin_amdgcn_readlane(__float_as_int(x), 63)); }
__device__ __forceinline__ double lane63(double x) {
    return __hiloint2double(__builtin_amdgcn_readlane(__double2hiint(x), 63),
                            __builtin_amdgcn_readlane(__double2loint(x), 63));
}
template <typename T> __device__ __forceinline__ T wave_max_t(T v) {
    v = fmax(v, dpp_move<0x111>(v));   // row_shr:1, 2, 4, 8: lane 15 of each row of 16 has the row's maximum
    v = fmax(v, dpp_move<0x112>(v));
    v = fmax(v, dpp_move<0x114>(v));
    v = fmax(v, dpp_move<0x118>(v));
    v = fmax(v, dpp_move<0x142>(v));   // row_bcast:15, then 31: lane 63 has the wave's
    v = fmax(v, dpp_move<0x143>(v));
    return lane63(v);
}

// Workgroup barrier for data in LDS alone: stores and loads of memory stay
// in flight (__syncthreads waits for the words just published to be written,
// a trip through memory per step).
__device__ __forceinline__ void lds_barrier() {
    asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory");
}

// LDS written by some lanes of a wave, read by others of the same wave.
__device__ __forceinline__ void wave_sync() {
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

// f(integral_constant<int, 0>), f(<1>), ... f(<N - 1>) while it returns true.
template <typename F, int... I> __device__ __forceinline__ void each_of(F &&f, std::integer_sequence<int, I...>) {
    (f(std::integral_constant<int, I>{}), ...);
}
// f(integral_constant<int, 0>) ... f(<N - 1>): a loop whose index is a constant from the start, so that an array it
// indexes is registers from the start (unrolled later, rows were selected by address and the patch went to scratch).
template <int N, typename F> __device__ __forceinline__ void each(F &&f) { each_of(f, std::make_integer_sequence<int, N>{}); }
template <typename F, int... I> __device__ __forceinline__ void chain(F &&f, std::integer_sequence<int, I...>) {
    (void)(f(std::integral_constant<int, I>{}) && ...);
}

// Flags lie 32 bytes apart and the first poll of a step waits kResPollFirst
// (0.5 us).  Measured, us per step (f32 64x48 / f64 128^2 / f32 512^2 / f32
// 1024^2): flags packed and polled at once 3.66 / 5.03 / 4.96 / 7.18, packed
// and polled after 0.43 us 2.93 / 3.78 / 4.15 / 6.87, 32 bytes apart and after
// 0.53 us 3.02 / 3.57 / 3.85 / 6.26, 64 bytes apart 3.03 / 3.76 / 3.84 / 6.11.
constexpr int kFlagWords = kResFlagWords;

template <typename T> struct Coef { T lx, ly, mx, my, lx4, ly4; };

// A poll that outlives every step by far (seconds): the data cannot come any
// more.  The wave goes on, waits for nothing further, and the run is flagged
// unstable.
constexpr int kPollMost = 1 << 22;

// All steps of one grid by one workgroup through the two buffers in memory,
// with the fused tile body: what is left to do when a team could not be
// brought together (the resident launch then has written nothing).
template <typename T> struct Serial {
    T *P[2][3];
    int64_t pitch;
    int nx, ny, bcx, bcy, cur, nsteps;
    double g, dx, dy, cfl, dt_fixed;
    double t, last_dt;   // in and out: the simulated time; out: the last dt
    bool bad;
};
template <typename T, bool TR> __device__ __attribute__((noinline)) void serial_steps(Serial<T> &z, T *lmax) {
    const int64_t pitch = z.pitch;
    const int nx = z.nx, ny = z.ny, bcx = z.bcx, bcy = z.bcy, nsteps = z.nsteps;
    const double g = z.g, dx = z.dx, dy = z.dy, cfl = z.cfl, dt_fixed = z.dt_fixed;
    T *(&P)[2][3] = z.P;
    int cur = z.cur;
    double t = z.t, last_dt = 0.0;
    bool bad = false;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), nw = blockDim.x >> 6;
    const int nstrips = (nx + 63) / 64, rows = 8, nrb = (ny + rows - 1) / rows;
    T smax = T(0);
    auto sync_memory = [] {
        __threadfence();
        __syncthreads();
        __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "agent");
    };
    auto cell = [&](T *const *B, int i, int j) {
        const int64_t o = (int64_t)j * pitch + i;
        return U3<T>{B[0][o], B[1][o], B[2][o]};
    };
    for (int64_t idx = threadIdx.x; idx < (int64_t)nx * ny; idx += blockDim.x) {
        const int j = (int)(idx / nx), i = (int)(idx - (int64_t)j * nx);
        const U3<T> c = cell(P[cur], i, j);
        const T s = signal_speed(c, (T)g);
        bad |= !(s <= finite_max<T>());
        smax = fmax(smax, s);
        if (i == 0 || i == nx - 1 || j == 0 || j == ny - 1) write_ghosts(P[cur], pitch, nx, ny, bcx, bcy, i, j, c);
    }
    for (int n = 0; n < nsteps; ++n) {
        smax = wave_max_t(smax);
        if ((threadIdx.x & 63) == 0) lmax[wave] = smax;
        sync_memory();
        T m = lmax[0];
        for (int k = 1; k < nw; ++k) m = fmax(m, lmax[k]);
        const double dt = dt_fixed > 0 ? dt_fixed : cfl * fmin(dx, dy) / (double)m;
        t += dt;
        last_dt = dt;
        smax = T(0);
        __syncthreads();
        for (int tile = wave; tile < nstrips * nrb; tile += nw) {
            TileArgs ta;
            for (int k = 0; k < 3; ++k) {
                ta.in[k] = P[cur][k];
                ta.out[k] = P[cur ^ 1][k];
            }
            ta.pitch = pitch;
            ta.nx = nx; ta.ny = ny; ta.bc_x = bcx; ta.bc_y = bcy;
            ta.s = tile % nstrips; ta.rb = tile / nstrips; ta.rows = rows;
            double used;
            if constexpr (TR) fused_tile_tr<T, 1, 1>(ta, [&] { return dt; }, g, dx, dy, smax, bad, used);
            else fused_tile_dir<T, 1, 1, false>(ta, [&] { return dt; }, g, dx, dy, smax, bad, used);
        }
        cur ^= 1;
    }
    z.t = t;
    z.last_dt = last_dt;
    z.bad |= bad;
}

__device__ __forceinline__ int uni(int v) { return __builtin_amdgcn_readfirstlane(v); }
__device__ __forceinline__ int64_t uni(int64_t v) {
    return ((int64_t)uni((int)(v >> 32)) << 32) | (unsigned)uni((int)v);
}
__device__ __forceinline__ float uni(float v) { return __int_as_float(uni(__float_as_int(v))); }
__device__ __forceinline__ double uni(double v) { return __longlong_as_double(uni((int64_t)__double_as_longlong(v))); }

template <int R, bool TR> constexpr int col_values() { return (3 * R + (TR ? 6 : 0) + 3) & ~3; }

// What bounds it: from about a million cells the VALU issue rate (70 to 80
// instructions per row of 64 lanes and step, five of them quarter-rate
// reciprocals and square roots: 1536^2 FP32 8.5 us a step, 278
// Gcell-updates/s, 19.1 us as per-step launches that read and write the state;
// the issue slots are 0.54 full, the rest is the exchange); below that the
// step's one trip of words through memory, 1.4 us of the 2.6 us that a step of
// 64^2 takes (4.8 us as per-step launches).  1024^2 FP32 12.1 -> 5.9 us, 2048^2
// 24.5 -> 14.8, 1024^2 FP64 16.3 -> 10.7, 1531x1087 FP64 transverse 26.2 ->
// 15.8.
//
// EXACT: every wave has R or R - 1 rows, so that the row above the patch
// stands at one of two places known at compile time (otherwise 1 to R rows).
template <typename T, int R, bool TR, int NW, bool EXACT>
__global__ __launch_bounds__(64 * NW) void k_resident(const SwResArgs a) {
    constexpr int VW = words_of<T>();
    constexpr int CV = col_values<R, false>();  // staged values of one side of a patch
    constexpr int HV = col_values<R, TR>();     // received ones (with the corners' rows)
    constexpr int KC = (2 * (3 * R + (TR ? 6 : 0)) + 63) / 64;
    constexpr int KF = 4;                       // flags a lane polls at once
    extern __shared__ char smem[];
    const int nw = blockDim.x >> 6;
    const int lane = threadIdx.x & 63, w = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    Coef<T> *lcoef = (Coef<T> *)smem;
    int *lgo = (int *)(smem + 64);
    T *lmax = (T *)(smem + 80);
    T *lrow = (T *)(smem + 256);                                    // [nw][2][3][64]: a wave's first and last row
    T *lcol = lrow + nw * 384 + w * 2 * (CV + HV);                  // this wave's: staged [2][CV], received [2][HV]
    T *lhal = lcol + 2 * CV;

    const int ti = a.teams ? uni(a.wg_team[blockIdx.x]) : 0;
    SwResTeam t = a.one;
    if (a.teams) {
        const SwResTeam &m = a.teams[ti];
        t.wg0 = uni(m.wg0); t.nwg = uni(m.nwg); t.ns = uni(m.ns); t.ws = uni(m.ws); t.nb = uni(m.nb);
        t.waves = uni(m.waves); t.base = uni(m.base); t.rem = uni(m.rem); t.nx = uni(m.nx); t.ny = uni(m.ny);
        t.pitch = uni(m.pitch); t.words = (uint64_t)uni((int64_t)m.words);
    }
    const int member = (int)blockIdx.x - t.wg0;
    const int b = member / t.ns, s = member - b * t.ns;
    const int nx = t.nx, ny = t.ny;
    const int gw = b * nw + w;                                      // wave of the strip
    const bool active = gw < t.waves;
    const int rr0 = active ? t.base + (gw < t.rem ? 1 : 0) : 0;     // rows j0 .. j0 + rr0 - 1
    const int j0 = gw * t.base + min(gw, t.rem);
    const int c0 = s * t.ws, wn = min(t.ws, nx - c0);               // columns c0 .. c0 + wn - 1 in lanes 1 .. wn
    const bool perx = a.bc_x == 1, pery = a.bc_y == 1;
    auto plane = [&](int q, int k) SW_INLINE -> T * {
        if (!a.teams) return (T *)a.plane[q][k];
        return (T *)(intptr_t)uni((int64_t)(intptr_t)a.grids[ti].plane[q][k]);
    };
    SwResCtl *ctl = a.ctl + ti;
    const unsigned tag0 = (unsigned)uni((int)ctl->epoch) + 1;

    // Exchange words of the team: [2] by step parity, each flags [nwg], rows
    // [nb][2][3][nx] (a workgroup's first and last row) and columns
    // [ns][waves][2][cvt] (a wave's first and last column).  Offsets are in
    // bytes, fit 31 bits (sw_res_cut) and are formed once.
    const int cvt = 3 * (t.base + (t.rem ? 1 : 0));
    constexpr unsigned VB = VW * 8, FB = kFlagWords * 8;
    const unsigned rows_at = (unsigned)t.nwg * FB, cols_at = rows_at + (unsigned)(t.nb * 6 * nx) * VB;
    const unsigned par_bytes = cols_at + (unsigned)(t.ns * t.waves * 2 * cvt) * VB;
    char *const words = (char *)(a.words + t.words);
    // the strips beside and the waves below and above (-1: a wall)
    const int sl = s > 0 ? s - 1 : (perx ? t.ns - 1 : -1), sr = s + 1 < t.ns ? s + 1 : (perx ? 0 : -1);
    const int gb = gw > 0 ? gw - 1 : (pery ? t.waves - 1 : -1), ga = gw + 1 < t.waves ? gw + 1 : (pery ? 0 : -1);
    const bool lds_b = gb >= 0 && gb / nw == b, lds_a = ga >= 0 && ga / nw == b;   // the neighbour is in this workgroup
    const bool far_b = active && gb >= 0 && !lds_b, far_a = active && ga >= 0 && !lds_a;
    const unsigned plane_bytes = (unsigned)nx * VB;
    auto row_words = [&](int blk, int side) SW_INLINE {      // of this lane's column (lanes beside the strip: its nearest)
        return rows_at + (unsigned)((blk * 2 + side) * 3 * nx + c0 + min(max(lane - 1, 0), wn - 1)) * VB;
    };
    const unsigned out_b = row_words(b, 0), out_a = row_words(b, 1);
    const unsigned in_b = row_words(far_b ? gb / nw : 0, 1), in_a = row_words(far_a ? ga / nw : 0, 0);
    auto col_words = [&](int strip, int wave, int side, int v) SW_INLINE {
        return cols_at + (unsigned)(((strip * t.waves + wave) * 2 + side) * cvt + v) * VB;
    };
    // The lane's column values v = lane + 64 q: out, values of the left column
    // and then of the right one; in, of the strip to the left and then of the
    // one to the right (TR: then those beside the rows below and above).
    // ~0: none.  *_lds: where they stand in the wave's LDS area.
    unsigned out_at[KC], in_at[KC];
    unsigned short out_lds[KC], in_lds[KC];
#pragma unroll
    for (int q = 0; q < KC; ++q) {
        const int v = lane + 64 * q, no = 3 * rr0, ni = active ? no + (TR ? 6 : 0) : 0;
        {
            const int side = v >= no, x = v - side * no;
            const bool on = v < 2 * no && (side ? sr : sl) >= 0;
            out_at[q] = on ? col_words(s, gw, side, x) : ~0u;
            out_lds[q] = (unsigned short)(on ? side * CV + x : 0);
        }
        const int side = v >= ni, x = v - side * ni, strip = side ? sr : sl;
        unsigned p = ~0u;
        if (v < 2 * ni && strip >= 0) {
            if (!TR || x < no) {
                p = col_words(strip, gw, side ^ 1, x);
            } else {
                const int at = x - no, up = at >= 3, wave = up ? ga : gb;
                if (wave >= 0)
                    p = col_words(strip, wave, side ^ 1, up ? at - 3 : (t.base + (wave < t.rem ? 1 : 0) - 1) * 3 + at);
            }
        }
        in_at[q] = p;
        in_lds[q] = (unsigned short)(p != ~0u ? 2 * CV + side * HV + x : 0);
    }

    T U[R + 1][3];
    const T kg = (T)(0.5 * a.g), g = (T)a.g;
    T smax = T(0), broken = T(0);   // broken: 0, or not a number once a cell's speed was not finite
    bool bad = false, late = false;
    each<R + 1>([&](auto ic) SW_INLINE {
        constexpr int i = decltype(ic)::value;
        U[i][0] = T(1);
        U[i][1] = U[i][2] = T(0);
    });
    if (lane >= 1 && lane <= wn) {
        const T *I[3] = {plane(a.cur, 0), plane(a.cur, 1), plane(a.cur, 2)};
        each<R>([&](auto ic) SW_INLINE {
            constexpr int i = decltype(ic)::value;
            if (i < rr0) {
                const int64_t o = (int64_t)(j0 + i) * t.pitch + c0;
                each<3>([&](auto kc) SW_INLINE { constexpr int k = decltype(kc)::value; U[i][k] = (I[k] + o)[lane - 1]; });
            }
        });
        each<R>([&](auto ic) SW_INLINE {
            constexpr int i = decltype(ic)::value;
            if (i < rr0) {
                const T sp = signal_speed(U3<T>{U[i][0], U[i][1], U[i][2]}, g);
                bad |= !(sp <= finite_max<T>());
                smax = fmax(smax, sp);
            }
        });
    }
    __builtin_amdgcn_s_waitcnt(0x0f70);             // the loads are in: no wait for them (and for words put since) in the loop
    const bool keeper = member == 0 && w == 0;      // the wave that keeps the grid's books
    double time = 0.0, last_dt = 0.0;
    if (keeper) time = a.teams ? a.bsc[ti].t : a.sc->t;

    bool go = true;
    for (int n = 0; n < a.nsteps; ++n) {
        const unsigned tag = tag0 + (unsigned)n;
        char *const wp = words + (n & 1 ? par_bytes : 0u);
        // (opaque copies: comparisons and offsets derived from them are formed anew each step instead of being
        // kept in registers over the whole loop)
        int rr = rr0, ln = lane;
        asm volatile("" : "+s"(rr), "+v"(ln));
        const int lane = ln;
        const bool own = lane >= 1 && lane <= wn;
        // row i is the patch's (EXACT), or stands in a group of four with such a row: the rest of a group is carried
        // along and its results dropped, so that the rows are not cut into a basic block each
        auto has = [&](int i) SW_INLINE { return EXACT ? i < R - 1 || rr == R : (i & ~3) < rr; };
        auto ends = [&](int i) SW_INLINE { return i == R || (EXACT ? !has(i) : (i & 3) == 3 && i >= rr); };   // nothing after row i
        auto last_row = [&](T v[3]) SW_INLINE {
            each<3>([&](auto kc) SW_INLINE { constexpr int k = decltype(kc)::value; v[k] = U[EXACT ? R - 1 : 0][k]; });
            if constexpr (EXACT && R > 1) {
                if (rr != R) {
                    each<3>([&](auto kc) SW_INLINE { constexpr int k = decltype(kc)::value; v[k] = U[R - 2][k]; });
                }
            } else if constexpr (!EXACT) {
                // (values selected, not branches taken: the compiler would merge those into one indexed access)
                each<R>([&](auto ic) SW_INLINE {
                    constexpr int i = decltype(ic)::value;
                    each<3>([&](auto kc) SW_INLINE { constexpr int k = decltype(kc)::value; v[k] = i == rr - 1 ? U[i][k] : v[k]; });
                });
            }
        };
        // ---- what the neighbours need of U^n
        if (active) {
            auto stage = [&](T *to) SW_INLINE {
                each<R>([&](auto ic) SW_INLINE {
                    constexpr int i = decltype(ic)::value;
                    if (has(i)) {
                        each<3>([&](auto kc) SW_INLINE { constexpr int k = decltype(kc)::value; to[i * 3 + k] = U[i][k]; });
                    }
                });
            };
            if (lane == 1 || lane == wn) stage(lane == 1 ? lcol : lcol + CV);
            if (wn == 1 && lane == 1) stage(lcol + CV);
            wave_sync();
#pragma unroll
            for (int q = 0; q < KC; ++q)
                if (out_at[q] != ~0u) put_value(wp + out_at[q], tag, lcol[out_lds[q]]);
            T last[3];
            last_row(last);
#pragma unroll
            for (int k = 0; k < 3; ++k) {
                lrow[((w * 2 + 0) * 3 + k) * 64 + lane] = U[0][k];
                lrow[((w * 2 + 1) * 3 + k) * 64 + lane] = last[k];
            }
            if (far_b && own) {
                each<3>([&](auto kc) SW_INLINE {
                    constexpr int k = decltype(kc)::value;
                    put_value(wp + (out_b + k * plane_bytes), tag, U[0][k]);
                });
            }
            if (far_a && own) {
                each<3>([&](auto kc) SW_INLINE {
                    constexpr int k = decltype(kc)::value;
                    put_value(wp + (out_a + k * plane_bytes), tag, last[k]);
                });
            }
        }
        const bool want_dt = a.dt_fixed <= 0 || n == 0;
        if (want_dt) {
            const T m = wave_max_t(own ? smax : T(0));
            if (lane == 0) lmax[w] = m;
        }
        lds_barrier();
        // ---- the halo of the patch: rows below (into D) and above (into A), columns beside (into U); wave 0 also
        // takes the step's dt from the maximum over the team, one word per workgroup.  All words a wave needs are
        // polled together, so that a step waits for one trip through memory.
        T D[3], A[3];
        const bool keeps_dt = want_dt && w == 0;
        T top = T(0);
        if (keeps_dt) {
            top = wave_max_t(lane < nw ? lmax[lane] : T(0));
            if (lane == 0) put_value(wp + (unsigned)member * FB, tag, top);
        }
        int verdict = 1;
        // flags [m0, m0 + 64 KF) of the team: folded into `top` once all are there
        auto get_flags = [&](int m0, Words<T> f[KF]) SW_INLINE {
#pragma unroll
            for (int k = 0; k < KF; ++k) f[k] = get_words<T>(wp + (unsigned)min(m0 + 64 * k + lane, t.nwg - 1) * FB);
        };
        auto take_flags = [&](const Words<T> f[KF]) SW_INLINE {
            bool ok = true;
            T m = T(0);
#pragma unroll
            for (int k = 0; k < KF; ++k) {
                ok = ok && is_tagged(f[k], tag);
                m = fmax(m, value_of(f[k]));
            }
            ok = __all(ok);
            if (ok) top = fmax(top, m);
            return ok;
        };
        auto gather = [&]() SW_INLINE {                     // n = 0: is the whole team there?  Give up together if it does not come
            const long long began = wall_clock64();
            if (a.patience < 0 && lane == 0) (void)atomicCAS(&ctl->state, 0u, 2u);   // (asked not to wait at all)
            for (int m0 = 0; m0 < t.nwg && verdict; m0 += 64 * KF) {
                for (;;) {
                    Words<T> f[KF];
                    get_flags(m0, f);
                    if (take_flags(f)) break;
                    const unsigned st = __hip_atomic_load(&ctl->state, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
                    if (st == 2u) { verdict = 0; break; }
                    if (st == 0u && wall_clock64() - began > a.patience) {
                        unsigned was = 0u;
                        if (lane == 0) was = atomicCAS(&ctl->state, 0u, 2u);
                        if (uni((int)was) != 1) { verdict = 0; break; }
                    }
                    __builtin_amdgcn_s_sleep(1);
                }
            }
            if (verdict) {
                unsigned was = 0u;
                if (lane == 0) was = atomicCAS(&ctl->state, 0u, 1u);
                verdict = uni((int)was) != 2;
            }
        };
        auto fetch = [&](bool with_flags) SW_INLINE {
            Words<T> cw[KC], bw[3], aw[3], fw[KF];
            // A poll that comes too early costs a whole further trip, and many of them hold up the words they
            // wait for: the first goes out about when the neighbours' words, put at the same time as this wave's,
            // can be there.
            for (int z = 0; z < a.poll_first; ++z) __builtin_amdgcn_s_sleep(2);
            for (int it = 0;; ++it) {
#pragma unroll
                for (int q = 0; q < KC; ++q) cw[q] = get_words<T>(wp + (in_at[q] != ~0u ? in_at[q] : 0u));
                if (far_b) {
                    each<3>([&](auto kc) SW_INLINE {
                        constexpr int k = decltype(kc)::value;
                        bw[k] = get_words<T>(wp + (in_b + k * plane_bytes));
                    });
                }
                if (far_a) {
                    each<3>([&](auto kc) SW_INLINE {
                        constexpr int k = decltype(kc)::value;
                        aw[k] = get_words<T>(wp + (in_a + k * plane_bytes));
                    });
                }
                if (with_flags) get_flags(0, fw);
                bool ok = true;
#pragma unroll
                for (int q = 0; q < KC; ++q) ok = ok && (in_at[q] == ~0u || is_tagged(cw[q], tag));
                if (far_b) ok = ok && is_tagged(bw[0], tag) && is_tagged(bw[1], tag) && is_tagged(bw[2], tag);
                if (far_a) ok = ok && is_tagged(aw[0], tag) && is_tagged(aw[1], tag) && is_tagged(aw[2], tag);
                ok = __all(ok);
                if (with_flags) ok = ok && take_flags(fw);
                if (ok) break;
                if (late || it >= kPollMost) { late = true; break; }
                for (int z = 0; z < a.poll_next; ++z) __builtin_amdgcn_s_sleep(2);
            }
            if (with_flags) {
                for (int m0 = 64 * KF; m0 < t.nwg; m0 += 64 * KF)
                    for (int it = 0;; ++it) {
                        get_flags(m0, fw);
                        if (take_flags(fw)) break;
                        for (int z = 0; z < a.poll_next; ++z) __builtin_amdgcn_s_sleep(2);
                        if (late || it >= kPollMost) { late = true; break; }
                    }
            }
#pragma unroll
            for (int q = 0; q < KC; ++q)
                if (in_at[q] != ~0u) lcol[in_lds[q]] = value_of(cw[q]);
            T got[2][3];
#pragma unroll
            for (int k = 0; k < 3; ++k) {
                got[0][k] = far_b ? value_of(bw[k]) : T(0);
                got[1][k] = far_a ? value_of(aw[k]) : T(0);
            }
#pragma unroll
            for (int side = 0; side < 2; ++side)          // 0: below, 1: above
                if (side ? lds_a : lds_b) {
                    const int ow = (side ? ga : gb) - b * nw;
                    each<3>([&](auto kc) SW_INLINE {
                        constexpr int k = decltype(kc)::value;
                        got[side][k] = lrow[((ow * 2 + (side ^ 1)) * 3 + k) * 64 + lane];
                    });
                }
            wave_sync();
            // columns: the lanes beside the strip; at a wall the mirror image of the wall cell
            const bool beside = lane == 0 || lane == wn + 1;
            {
                const int side = lane != 0;
                const bool wall = (side ? sr : sl) < 0;
                const T *src = wall ? lcol + side * CV : lhal + side * HV;
                const T sg = wall ? T(-1) : T(1);
                each<R>([&](auto ic) SW_INLINE {
                    constexpr int i = decltype(ic)::value;
                    if (has(i)) {
                        const T h = src[i * 3], p = src[i * 3 + 1], q = src[i * 3 + 2];
                        U[i][0] = beside ? h : U[i][0];
                        U[i][1] = beside ? sg * p : U[i][1];
                        U[i][2] = beside ? q : U[i][2];
                    }
                });
                if (TR && beside && !wall) {                // corners: beside the rows below and above
#pragma unroll
                    for (int up = 0; up < 2; ++up) {
                        if ((up ? ga : gb) < 0) continue;
                        each<3>([&](auto kc) SW_INLINE { constexpr int k = decltype(kc)::value; got[up][k] = src[3 * rr + up * 3 + k]; });
                    }
                }
            }
            if (TR) {   // corners at an x wall: the mirror image of the neighbour row's wall cell
#pragma unroll
                for (int up = 0; up < 2; ++up) {
                    if ((up ? ga : gb) < 0) continue;
                    T fromn[3], fromp[3];
#pragma unroll
                    for (int k = 0; k < 3; ++k) {
                        fromn[k] = from_next_lane(got[up][k], got[up][k]);
                        fromp[k] = from_prev_lane(got[up][k], got[up][k]);
                    }
                    if (lane == 0 && sl < 0) { got[up][0] = fromn[0]; got[up][1] = -fromn[1]; got[up][2] = fromn[2]; }
                    if (lane == wn + 1 && sr < 0) { got[up][0] = fromp[0]; got[up][1] = -fromp[1]; got[up][2] = fromp[2]; }
                }
            }
            // at a y wall the mirror image of the wall row (halo lanes included)
            if (gb < 0) {
                D[0] = U[0][0]; D[1] = U[0][1]; D[2] = -U[0][2];
            } else {
                each<3>([&](auto kc) SW_INLINE { constexpr int k = decltype(kc)::value; D[k] = got[0][k]; });
            }
            if (ga < 0) {
                last_row(A);
                A[2] = -A[2];
            } else {
                each<3>([&](auto kc) SW_INLINE { constexpr int k = decltype(kc)::value; A[k] = got[1][k]; });
            }
        };
        if (n == 0) {
            if (w == 0) {
                gather();
                if (lane == 0) *lgo = verdict;
            }
            lds_barrier();
            go = *lgo != 0;
            if (!go) break;
        }
        if (active) fetch(keeps_dt && n > 0);
        if (keeps_dt) {
            const T m = wave_max_t(top);
            const double dt = a.dt_fixed > 0 ? a.dt_fixed : a.cfl * fmin(a.dx, a.dy) / (double)m;
            // x / dx as x * (1 / dx) where dx is a power of two (the same bits, without the division's latency)
            const double rx = a.rdx != 0.0 ? dt * a.rdx : dt / a.dx, ry = a.rdy != 0.0 ? dt * a.rdy : dt / a.dy;
            if (lane == 0)
                *lcoef = Coef<T>{(T)(0.5 * rx), (T)(0.5 * ry), (T)rx, (T)ry, (T)(0.125 * rx), (T)(0.125 * ry)};
            last_dt = dt;
        }
        lds_barrier();
        time += last_dt;
        const Coef<T> cl = *lcoef;
        const Coef<T> cf = {uni(cl.lx), uni(cl.ly), uni(cl.mx), uni(cl.my), uni(cl.lx4), uni(cl.ly4)};
        if (!active) continue;
        // ---- the step: rows below, 0 .. rr - 1 and above in turn (the row above sits in U[rr])
        if constexpr (EXACT) {
            if (R == 1 || rr == R) {
                each<3>([&](auto kc) SW_INLINE { constexpr int k = decltype(kc)::value; U[R][k] = A[k]; });
            } else {
                each<3>([&](auto kc) SW_INLINE { constexpr int k = decltype(kc)::value; U[R > 1 ? R - 1 : 0][k] = A[k]; });
            }
        } else {
            each<R + 1>([&](auto ic) SW_INLINE {
                constexpr int i = decltype(ic)::value;
                each<3>([&](auto kc) SW_INLINE { constexpr int k = decltype(kc)::value; U[i][k] = i == rr ? A[k] : U[i][k]; });
            });
        }
        smax = T(0);
        const T lx = cf.lx, ly = cf.ly, mx = cf.mx, my = cf.my;
        if constexpr (!TR) {
            T S[3], B[3], G[3];
            {
                const T rc = fast_rcp(D[0]);
                const T u = D[1] * rc, v = D[2] * rc, kh = kg * D[0];
                (void)u;
                B[0] = fma(ly, D[2], T(0.5) * D[0]);
                B[1] = fma(ly, D[2] * (D[1] * rc), T(0.5) * D[1]);
                B[2] = fma(ly, fma(kh, D[0], D[2] * v), T(0.5) * D[2]);
            }
            auto row = [&](auto ic) SW_INLINE {
                constexpr int i = decltype(ic)::value;
                const T h = U[i][0], p = U[i][1], q = U[i][2];
                const T rc = fast_rcp(h);
                const T u = p * rc, v = q * rc, kh = kg * h;
                const T fp = fma(kh, h, p * u), fq = q * u, gq = fma(kh, h, q * v);
                const T hh = T(0.5) * h, hp = T(0.5) * p, hq = T(0.5) * q;
                T f[3];
                yface_flux<T>(B[0] + fma(-ly, q, hh), B[1] + fma(-ly, fq, hp), B[2] + fma(-ly, gq, hq), kg, f);
                if constexpr (i > 0) {
                    T *o = U[i - 1];
                    each<3>([&](auto kc) SW_INLINE { constexpr int k = decltype(kc)::value; o[k] = fma(-my, f[k] - G[k], S[k]); });
                    T sp = signal_speed(U3<T>{o[0], o[1], o[2]}, g);
                    if constexpr (!EXACT) sp = i <= rr ? sp : T(0);
                    broken = fma(sp, T(0), broken);
                    smax = max_of(sp, smax);
                }
                each<3>([&](auto kc) SW_INLINE { constexpr int k = decltype(kc)::value; G[k] = f[k]; });
                if (ends(i)) return false;
                B[0] = fma(ly, q, hh);
                B[1] = fma(ly, fq, hp);
                B[2] = fma(ly, gq, hq);
                T fr[3];
                xface_flux<T>(fma(lx, p, hh) + next_lane(fma(-lx, p, hh)), fma(lx, fp, hp) + next_lane(fma(-lx, fp, hp)),
                              fma(lx, fq, hq) + next_lane(fma(-lx, fq, hq)), kg, fr);
                each<3>([&](auto kc) SW_INLINE { constexpr int k = decltype(kc)::value; S[k] = fma(-mx, fr[k] - prev_lane(fr[k]), U[i][k]); });
                return true;
            };
            chain(row, std::make_integer_sequence<int, R + 1>{});
        } else {
            const T lx4 = cf.lx4, ly4 = cf.ly4;
            // carried (sw_tile_tr.h): row i - 1's flux parts, row i - 2's G, the face contribution and flux below
            T Rfp, Rfq, Rgq, Gm[3], B[3], G[3];
            auto parts = [&](const T *c3, T &fp, T &fq, T &gq, T C[3]) SW_INLINE {
                const T rc = fast_rcp(c3[0]);
                const T u = c3[1] * rc, v = c3[2] * rc, kh = kg * c3[0];
                fp = fma(kh, c3[0], c3[1] * u);
                fq = c3[2] * u;
                gq = fma(kh, c3[0], c3[2] * v);
                C[0] = prev_lane(c3[1]) - next_lane(c3[1]);
                C[1] = prev_lane(fp) - next_lane(fp);
                C[2] = prev_lane(fq) - next_lane(fq);
            };
            T C[3];
            parts(D, Rfp, Rfq, Rgq, C);
            B[0] = fma(lx4, C[0], fma(ly, D[2], T(0.5) * D[0]));
            B[1] = fma(lx4, C[1], fma(ly, Rfq, T(0.5) * D[1]));
            B[2] = fma(lx4, C[2], fma(ly, Rgq, T(0.5) * D[2]));
            T below_q = D[2];
            auto row = [&](auto ic) SW_INLINE {
                constexpr int i = decltype(ic)::value;
                const T h = U[i][0], p = U[i][1], q = U[i][2];
                T fp, fq, gq;
                parts(U[i], fp, fq, gq, C);
                const T hh = T(0.5) * h, hp = T(0.5) * p, hq = T(0.5) * q;
                T f[3];
                yface_flux<T>(B[0] + fma(lx4, C[0], fma(-ly, q, hh)), B[1] + fma(lx4, C[1], fma(-ly, fq, hp)),
                              B[2] + fma(lx4, C[2], fma(-ly, gq, hq)), kg, f);
                if constexpr (i > 0) {
                    T *o = U[i - 1];                              // row i - 1: its x faces, then its update
                    const T d0 = Gm[0] - q, d1 = Gm[1] - fq, d2 = Gm[2] - gq;
                    const T oh = T(0.5) * o[0], op = T(0.5) * o[1], oq = T(0.5) * o[2];
                    T fr[3];
                    xface_flux<T>(fma(ly4, d0, fma(lx, o[1], oh)) + next_lane(fma(ly4, d0, fma(-lx, o[1], oh))),
                                  fma(ly4, d1, fma(lx, Rfp, op)) + next_lane(fma(ly4, d1, fma(-lx, Rfp, op))),
                                  fma(ly4, d2, fma(lx, Rfq, oq)) + next_lane(fma(ly4, d2, fma(-lx, Rfq, oq))), kg, fr);
                    Gm[0] = o[2];
#pragma unroll
                    for (int k = 0; k < 3; ++k)
                        o[k] = fma(-my, f[k] - G[k], fma(-mx, fr[k] - prev_lane(fr[k]), o[k]));
                    T sp = signal_speed(U3<T>{o[0], o[1], o[2]}, g);
                    if constexpr (!EXACT) sp = i <= rr ? sp : T(0);
                    broken = fma(sp, T(0), broken);
                    smax = max_of(sp, smax);
                } else {
                    Gm[0] = below_q;
                }
                Gm[1] = Rfq;
                Gm[2] = Rgq;
                Rfp = fp;
                Rfq = fq;
                Rgq = gq;
                each<3>([&](auto kc) SW_INLINE { constexpr int k = decltype(kc)::value; G[k] = f[k]; });
                if (ends(i)) return false;
                B[0] = fma(lx4, C[0], fma(ly, q, hh));
                B[1] = fma(lx4, C[1], fma(ly, fq, hp));
                B[2] = fma(lx4, C[2], fma(ly, gq, hq));
                return true;
            };
            chain(row, std::make_integer_sequence<int, R + 1>{});
        }
    }

    if (go && lane >= 1 && lane <= wn) {
        const int f = a.cur ^ (a.nsteps & 1), c = c0 + lane - 1;
        T *O[3] = {plane(f, 0), plane(f, 1), plane(f, 2)};
        each<R>([&](auto ic) SW_INLINE {
            constexpr int i = decltype(ic)::value;
            if (i < rr0) {
                const int j = j0 + i;
                const int64_t o = (int64_t)j * t.pitch + c0;
                each<3>([&](auto kc) SW_INLINE { constexpr int k = decltype(kc)::value; (O[k] + o)[lane - 1] = U[i][k]; });
                if (c == 0 || c == nx - 1 || j == 0 || j == ny - 1)
                    write_ghosts(O, t.pitch, nx, ny, a.bc_x, a.bc_y, c, j, U3<T>{U[i][0], U[i][1], U[i][2]});
            }
        });
    }
    bad |= late || (broken != broken && lane >= 1 && lane <= wn && rr0 > 0);
    // the team's last workgroup to end readies the words for the next launch,
    // after it has done the steps by itself if the team never came together
    __syncthreads();
    if (threadIdx.x == 0) *lgo = atomicAdd(&ctl->exits, 1u) + 1u == (unsigned)t.nwg ? 1 : 0;
    __syncthreads();
    const bool last_one = *lgo != 0;
    bool books = keeper && go;
    if (!go && last_one) {
        Serial<T> z;
        for (int q = 0; q < 2; ++q)
            for (int k = 0; k < 3; ++k) z.P[q][k] = plane(q, k);
        z.pitch = t.pitch;
        z.nx = nx; z.ny = ny; z.bcx = a.bc_x; z.bcy = a.bc_y; z.cur = a.cur; z.nsteps = a.nsteps;
        z.g = a.g; z.dx = a.dx; z.dy = a.dy; z.cfl = a.cfl; z.dt_fixed = a.dt_fixed;
        z.t = a.teams ? a.bsc[ti].t : a.sc->t;
        z.bad = false;
        __syncthreads();                            // (the books below are written after everyone has read them)
        serial_steps<T, TR>(z, lmax);
        time = z.t;
        last_dt = z.last_dt;
        bad |= z.bad;
        books = w == 0;
    }
    const u64 anybad = __ballot(bad);
    if (lane == 0) {
        if (a.teams) {
            SwBatchScalars *sc = a.bsc + ti;
            if (anybad) atomicOr(&sc->unstable, 1u);
            if (books) { sc->t = time; sc->last_dt = last_dt; sc->steps += a.nsteps; sc->alone += !go; }
        } else {
            if (anybad) atomicOr(&a.sc->unstable, 1u);
            if (books) { a.sc->t = time; a.sc->last_dt = last_dt; a.sc->steps += a.nsteps; a.sc->alone += !go; }
        }
    }
    if (last_one && threadIdx.x == 0) {
        ctl->epoch = tag0 + (unsigned)a.nsteps - 1u;
        ctl->state = 0u;
        ctl->exits = 0u;
    }
}

template <typename T, int R, bool TR> size_t lds_bytes(int nw) {
    return 256 + sizeof(T) * ((size_t)nw * 384 + (size_t)nw * 2 * (col_values<R, false>() + col_values<R, TR>()));
}

template <typename T, int R, bool TR, int NW, bool EXACT>
hipError_t launch(const SwResArgs &a, int nw, int nwg, hipStream_t s) {
    k_resident<T, R, TR, NW, EXACT><<<(unsigned)nwg, 64 * nw, lds_bytes<T, R, TR>(nw), s>>>(a);
    return hipGetLastError();
}

template <typename T, bool TR>
hipError_t launch_rows(const SwResArgs &a, int rows, bool exact, int nw, int nwg, hipStream_t s) {
    // FP32 patches up to 16 rows fit 128 registers (16 waves to a CU), though
    // those of 10 rows and more spill a little: they have an instance with
    // twice the registers too, for workgroups of up to 8 waves
    constexpr int NW = sizeof(T) == 4 ? 16 : 8;
    const bool roomy = sizeof(T) == 4 && nw <= 8 && rows >= kResRoomy;
#define SW_RES_CASE(R) \
    case R: return launch<T, R, TR, NW, true>(a, nw, nwg, s);
#define SW_RES_CASE8(R) \
    case R: return launch<T, R, TR, 8, true>(a, nw, nwg, s);
    if (exact && roomy) {
        if constexpr (sizeof(T) == 4) switch (rows) {
                SW_RES_ROOMY(SW_RES_CASE8) SW_RES_TALL(SW_RES_CASE8)
            }
    } else if (exact) {
        switch (rows) {
            SW_RES_ROWS(SW_RES_CASE)
        }
    }
#undef SW_RES_CASE
#undef SW_RES_CASE8
    if (rows <= 4) return launch<T, 4, TR, NW, false>(a, nw, nwg, s);
    if (rows < kResRoomy) return launch<T, kResRoomy - 1, TR, NW, false>(a, nw, nwg, s);
    if constexpr (sizeof(T) == 4) {
        if (roomy) return rows <= 20 ? launch<T, 20, TR, 8, false>(a, nw, nwg, s)
                                     : launch<T, kResRowsTall, TR, 8, false>(a, nw, nwg, s);
    }
    if constexpr (sizeof(T) == 8) return launch<T, kResRows, TR, NW, false>(a, nw, nwg, s);   // (FP32 with 16 waves: exact cuts alone)
    return hipErrorInvalidValue;
}

}  // namespace
