// Host side of the resident time loop: how a grid is cut up, and the
// admission of its launches.
//
// The workgroups of a team wait for each other, so all of them have to be
// resident at once.  Two things see to that.  (1) A grid is cut into at most
// one workgroup per compute unit, and a launch is ordered (by event waits on
// its stream) behind the resident launches of this process whose compute
// units it takes over (sw_admission.h), so that those that can run at the same
// time have room together.  Other
// kernels on the device only delay a team: they end by themselves.  A batch
// launches more workgroups than fit: workgroups start in order of their
// index (on each XCD), so the teams of the lowest indices are complete first
// and end, and so on.  (2) Where a team does not come together all the same
// (another process holds the device), its workgroups give up together
// before anything is written and the last of them does the steps alone.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <climits>
#include <cmath>
#include <map>
#include <mutex>
#include <numeric>
#include <vector>

#include "sw_admission.h"
#include "sw_resident.h"

bool sw_res_cut(int dtype, int nx, int ny, int64_t pitch, int nw, int max_rows, int max_wg, bool spread, SwResPlan *out) {
    SwResPlan p{};
    SwResTeam &t = p.team;
    t.nx = nx;
    t.ny = ny;
    t.pitch = pitch;
    t.ns = (nx + kResStrip - 1) / kResStrip;
    t.ws = (nx + t.ns - 1) / t.ns;
    t.ns = (nx + t.ws - 1) / t.ws;
    const int64_t waves = ((int64_t)ny + max_rows - 1) / max_rows;      // (each with as many rows, give or take one)
    const int64_t nb = (waves + nw - 1) / nw;
    if (nb * t.ns > max_wg) return false;
    t.waves = (int)(spread ? std::min<int64_t>(nb * nw, ny) : waves);
    t.base = ny / t.waves;
    t.rem = ny - t.base * t.waves;
    t.nb = (t.waves + nw - 1) / nw;
    t.nwg = t.nb * t.ns;
    p.rows = t.base + (t.rem ? 1 : 0);
    if (spread && !sw_res_has_rows(p.rows)) {                                    // fewer, taller waves of a listed height
        int r = p.rows;
        while (r < max_rows && !sw_res_has_rows(r)) ++r;
        t.waves = (ny + r - 1) / r;
        t.base = ny / t.waves;
        t.rem = ny - t.base * t.waves;
        t.nb = (t.waves + nw - 1) / nw;
        t.nwg = t.nb * t.ns;
        p.rows = t.base + (t.rem ? 1 : 0);
    }
    p.nw = nw;
    p.exact = sw_res_has_rows(p.rows);
    const uint64_t vw = dtype ? 2 : 1;
    p.nwords = 2ull * kResFlagWords * t.nwg + vw * (12ull * t.nb * nx + 12ull * t.ns * t.waves * p.rows);
    if (p.nwords > 0x0fffffffull) return false;                        // 32-bit offsets in the kernel
    if (!sw_res_shape_ok(dtype, p.rows, nw)) return false;
    *out = p;
    return true;
}

static double us_per_row(int dtype) { return dtype ? 0.37 : 0.135; }   // of a wave that has its SIMD to itself

// The cut with the least work per step on a CU's busiest SIMD, in rows: the
// patches' rows and about 1.5 more each for the halo rows and the exchange,
// times the waves that share the SIMD, which run at 1 / 1.35 and 1 / 1.1 of
// the rate when there are only one or two of them (measured, us per step,
// FP32: 512^2 4 waves of 5 rows 3.64, 8 of 3 3.89, 16 of 2 4.00; 768^2 8 of 6
// 4.46, 16 of 3 4.64, 4 of 18 5.80; 1280^2 16 of 8 7.27, 4 of 28 8.22, 8 of 18
// 8.41; 1536^2 8 of 20 8.72, 16 of 10 8.86), a tenth more where 16 FP32 waves
// of 10 rows or more spill (1280^2: 8 of 14 7.25, 16 of 10 8.31; 1800^2: 8 of
// 32 12.7, 16 of 16 14.7).
bool sw_res_plan(int dtype, int nx, int ny, int64_t pitch, int cus, SwResPlan *out) {
    double best = 0.0;
    bool found = false;
    for (int nw = 4; nw <= (dtype ? 8 : 16); nw *= 2) {
        for (int rows = 1; rows <= (dtype || nw > 8 ? kResRows : kResRowsTall); ++rows) {
            SwResPlan p;
            if (!sw_res_has_rows(rows) || !sw_res_cut(dtype, nx, ny, pitch, nw, rows, cus, true, &p) || !p.exact) continue;
            double cost = (nw == 4 ? 1.35 : nw == 8 ? 2.2 : 4.0) * (p.rows + 1.5);
            if (nw == 16 && p.rows >= kResRoomy) cost *= 1.1;
            if (!found || cost < best) {
                *out = p;
                best = cost;
                found = true;
            }
        }
    }
    // (time per step as sw_res_plan_batch estimates it)
    if (found) out->most_steps = (int)std::max(64.0, kResLaunchUs / (us_per_row(dtype) * best + 2.5));
    return found;
}

// Workgroups of four waves that a CU holds at once.
static int batch_wgs_per_cu(int dtype, int rows) { return dtype || rows >= kResRoomy ? 2 : 4; }

// All grids of a batch in patches of the same greatest height, four waves to
// a workgroup, workgroups in order of their grid's size (largest first).
static bool cut_batch(int dtype, int n, const int *nx, const int *ny, const int64_t *pitch, int nw, int rows, int cus,
                      const std::vector<int> &order, SwResBatchPlan *out) {
    SwResBatchPlan &p = *out;
    const int max_team = cus * batch_wgs_per_cu(dtype, rows);   // a team must find room on the device as a whole
    p.nw = nw;
    p.teams.assign(n, SwResTeam{});
    p.wg_team.clear();
    p.nwords = 0;
    p.rows = 1;
    for (int g : order) {
        SwResPlan one;
        if (!sw_res_cut(dtype, nx[g], ny[g], pitch[g], p.nw, rows, max_team, false, &one)) return false;
        one.team.wg0 = (int32_t)p.wg_team.size();
        one.team.words = p.nwords;
        p.teams[g] = one.team;
        p.nwords += (one.nwords + 31) / 32 * 32;
        p.wg_team.insert(p.wg_team.end(), (size_t)one.team.nwg, g);
        if (p.wg_team.size() > (size_t)1 << 26) return false;
        p.rows = std::max(p.rows, one.rows);
    }
    p.exact = dtype ? p.rows <= kResRows && sw_res_has_rows(p.rows) : sw_res_has_rows(p.rows);
    for (const SwResTeam &t : p.teams) p.exact = p.exact && t.base >= p.rows - 1;
    return true;
}

// The fewest steps of a call from which the resident loop takes less time
// than the per-step launches.  It reads and writes every state once a call,
// workgroup by workgroup, and in a batch of more workgroups than fit the next
// teams start only when whole teams have ended; per-step launches stream
// through the states and pay for it every step.  Measured, us a call of 1 / 4
// / 20 steps, resident against per-step (FP32): 16 grids of 256^2 32 / 49 /
// 143 against 35 / 84 / 357; 256 of 256^2 283 / 437 / 1318 against 190 / 431 /
// 1690; 16 of 1024^2 301 / 438 / 1271 against 172 / 392 / 1550; FP64, 60 of
// 512^2 575 / 792 / 2440 against 305 / 731 / 2810.  us: the resident loop's
// estimated time a step in the paper's scheme.  The constants are fitted to
// 109 batches of 4 to 1024 grids of 16 to 1024 a side: over calls of 1 to 20
// steps the form picked took 0.5 % more than the faster one on average, at
// most 21 %.
static int batch_from_steps(int dtype, int scheme, int n, const int *nx, const int *ny, int cus, double us,
                            const SwResBatchPlan &p) {
    double cells = 0.0, padded = 0.0;
    bool even = true;
    for (int i = 0; i < n; ++i) {
        cells += (double)nx[i] * ny[i];
        padded += (double)((nx[i] + 127) / 128 * 128) * ((ny[i] + 15) / 16 * 16);   // in whole tiles
        even = even && nx[i] == nx[0] && ny[i] == ny[0];
    }
    cells *= 1e-6;
    padded *= 1e-6;
    const bool split = n >= 2 && cells >= 4.194304;             // two chains of launches
    const double work = cells + 0.45 * (padded - cells);
    double step_p, step_r = us * (dtype ? (scheme ? 1.0 : 0.84) : (scheme ? 1.38 : 1.08));
    if (split) step_p = (5.0 + work * (dtype ? 8.9 : 4.5)) * (scheme ? (dtype ? 1.06 : 1.12) : 1.0) * (even ? 1.0 : 1.08);
    else if (dtype) step_p = std::max((21.4 + 2.9 * work) * (scheme ? 1.05 : 1.0), 5.0 + 11.5 * work);
    else step_p = std::max(15.2 + 1.7 * work, 5.0 + 6.0 * work) * (scheme ? 1.2 : 1.0);
    step_r = step_r * (p.exact ? 1.0 : 1.33) + 1.2;
    const double rounds = (double)p.wg_team.size() / ((double)cus * batch_wgs_per_cu(dtype, p.rows));
    const double team = std::min((double)p.wg_team.size() / n, 128.0);
    const double call_p = split ? 55.0 + cells * (dtype ? 6.0 : 2.8) : 18.0 + cells * (dtype ? 4.0 : 2.0);
    // (teams of different heights do not end and start together)
    const double call_r = 13.0 + cells * (dtype ? 18.0 : 9.0) + (p.exact ? 0.3 * team * std::max(0.0, rounds - 1.0) : 0.0);
    if (call_r + step_r <= call_p + step_p) return 1;
    if (step_r >= step_p) return INT_MAX;
    return (int)std::min(std::ceil((call_r - call_p) / (step_p - step_r)), 1e9);
}

bool sw_res_plan_batch(int dtype, int scheme, int n, const int *nx, const int *ny, const int64_t *pitch, int cus,
                       SwResBatchPlan *out) {
    std::vector<int> order(n);
    std::iota(order.begin(), order.end(), 0);
    std::stable_sort(order.begin(), order.end(),
                     [&](int x, int y) { return (int64_t)nx[x] * ny[x] > (int64_t)nx[y] * ny[y]; });
    // Time per step (us) of the per-step launches and of the resident loop in
    // each patch height.  The latter in bins of teams that are resident
    // together: rows and 1.5 more per wave, times the waves that share a SIMD
    // at the rate measured for so many, and a step's exchange, which only
    // other teams of the bin hide.  (Measured, FP32 / FP64, resident against
    // per-step: 16 grids of 256^2 7.0 / 18.2 us, 256 of 256^2 63 / 87, 60 of
    // 512^2 58 / 76, 16 of 1024^2 62 / 78; 64 of 256^2 42 / 48 and 4 of
    // 1024^2 53 / 44 in FP64, whose patches are so low that one such team
    // fills the device.)
    int64_t cells = 0;
    for (int i = 0; i < n; ++i) cells += (int64_t)nx[i] * ny[i];
    double best = 0.97 * std::max(16.0, 5.0 + (double)cells / (dtype ? 105e3 : 215e3));
    bool found = false;
    for (int rows : {1, 2, 4, 6, 8, 10, 12, 16, 20, 24, 32, 40}) {
        if (rows > (dtype ? kResRows : kResRowsTall)) break;
        SwResBatchPlan p;
        if (!cut_batch(dtype, n, nx, ny, pitch, 4, rows, cus, order, &p)) continue;
        const int64_t slots = (int64_t)cus * batch_wgs_per_cu(dtype, rows);
        double us = 0.0;
        int64_t used = 0;
        int teams = 0;
        auto close = [&] {
            static const double at[5] = {0.0, 1.35, 2.2, 3.7, 5.2};
            us += us_per_row(dtype) * at[(used + cus - 1) / cus] * (p.rows + 1.5) + 2.5 / teams;
            used = teams = 0;
        };
        for (int g : order) {
            if (used + p.teams[g].nwg > slots) close();
            used += p.teams[g].nwg;
            ++teams;
        }
        close();
        if (us < best) {
            *out = std::move(p);
            best = us;
            found = true;
        }
    }
    if (!found) return false;
    out->from_steps = batch_from_steps(dtype, scheme, n, nx, ny, cus, best, *out);
    out->most_steps = (int)std::max(64.0, kResBatchLaunchUs / best);
    return out->from_steps < INT_MAX;
}

// For the tests (not in sw.h): the cut of a batch.  out: rows, waves per
// workgroup, workgroups, those of the largest team, from_steps, most_steps,
// exact; returns 0 where the per-step launches are kept.
extern "C" int sw_internal_plan_batch(int dtype, int scheme, int n, const int *nx, const int *ny, int cus, int *out) {
    SwResBatchPlan p;
    const std::vector<int64_t> pitch((size_t)n, 0);
    if (!sw_res_plan_batch(dtype, scheme, n, nx, ny, pitch.data(), cus, &p)) return 0;
    int team = 0;
    for (const SwResTeam &t : p.teams) team = std::max(team, t.nwg);
    const int got[7] = {p.rows, p.nw, (int)p.wg_team.size(), team, p.from_steps, p.most_steps, p.exact};
    std::copy(got, got + 7, out);
    return 1;
}
// The same of a single grid: rows, waves per workgroup, workgroups, most_steps.
extern "C" int sw_internal_plan_grid(int dtype, int nx, int ny, int cus, int *out) {
    SwResPlan p;
    if (!sw_res_plan(dtype, nx, ny, 0, cus, &p)) return 0;
    const int got[4] = {p.rows, p.nw, p.team.nwg, p.most_steps};
    std::copy(got, got + 4, out);
    return 1;
}

bool sw_res_stream_ok(hipStream_t s, int cus) {
    hipStreamCaptureStatus cs = hipStreamCaptureStatusNone;
    if (hipStreamIsCapturing(s, &cs) != hipSuccess) {
        (void)hipGetLastError();
        return false;
    }
    if (cs != hipStreamCaptureStatusNone) return false;
    if ((uintptr_t)s <= (uintptr_t)hipStreamPerThread) return true;   // a default stream: no handle to ask, and no mask
    constexpr int kWords = 32;
    uint32_t mask[kWords] = {};
    const int words = (cus + 31) / 32;
    if (words > kWords) return false;
    if (hipExtStreamGetCUMask(s, (uint32_t)words, mask) != hipSuccess) {
        (void)hipGetLastError();
        return false;
    }
    int on = 0;
    for (int k = 0; k < words; ++k) on += __builtin_popcount(mask[k]);
    return on >= cus;
}

// For the tests (not in sw.h): the calling thread's next sw_res_alloc finds no
// memory.
static thread_local bool t_deny = false;
extern "C" void sw_internal_deny_alloc() { t_deny = true; }

hipError_t sw_res_alloc(void **p, size_t bytes) {
    *p = nullptr;
    const bool deny = t_deny;
    t_deny = false;
    const hipError_t e = deny ? hipErrorOutOfMemory : hipMalloc(p, bytes);
    if (e != hipErrorOutOfMemory) return e;
    (void)hipGetLastError();
    *p = nullptr;
    return hipSuccess;
}

hipError_t sw_res_launch_f32(const SwResArgs &a, int rows, bool exact, int nw, int nwg, hipStream_t s);
hipError_t sw_res_launch_f64(const SwResArgs &a, int rows, bool exact, int nw, int nwg, hipStream_t s);
hipError_t sw_res_launch_f32_tr(const SwResArgs &a, int rows, bool exact, int nw, int nwg, hipStream_t s);
hipError_t sw_res_launch_f64_tr(const SwResArgs &a, int rows, bool exact, int nw, int nwg, hipStream_t s);

hipError_t sw_res_launch(const SwResArgs &a, int dtype, int scheme, int rows, bool exact, int nw, int nwg, hipStream_t s) {
    if (nwg < 1 || a.nsteps < 1 || !sw_res_shape_ok(dtype, rows, nw)) return hipErrorInvalidValue;
    if (dtype) return scheme ? sw_res_launch_f64_tr(a, rows, exact, nw, nwg, s) : sw_res_launch_f64(a, rows, exact, nw, nwg, s);
    return scheme ? sw_res_launch_f32_tr(a, rows, exact, nw, nwg, s) : sw_res_launch_f32(a, rows, exact, nw, nwg, s);
}

namespace {

// Compute units a launch of nwg workgroups takes: workgroups go to the XCDs
// in turn, so a launch has one more on some of them than on others, and the
// units it holds must cover it on each (9 and 247 workgroups are 2 and 31 on
// the first of 8 XCDs of 32 units).
constexpr int kXcds = 8;
int units_of(int nwg, int cus) { return std::min(((int64_t)nwg + kXcds - 1) / kXcds * kXcds, (int64_t)cus); }

struct Device {
    SwCuPool<hipStream_t, hipEvent_t> pool;
    std::vector<hipEvent_t> spare;
};
std::mutex g_mutex;
std::map<int, Device> &devices() {
    static auto *d = new std::map<int, Device>();   // never destroyed: the HIP runtime may go first at exit
    return *d;
}

}  // namespace

hipError_t sw_res_launch_admitted(const SwResArgs &a, int dtype, int scheme, int rows, bool exact, int nw, int nwg,
                                  int device, int cus, hipStream_t s) {
    std::lock_guard<std::mutex> hold(g_mutex);
    Device &d = devices().try_emplace(device, Device{SwCuPool<hipStream_t, hipEvent_t>(cus), {}}).first->second;
    const int want = units_of(nwg, cus);
    hipError_t e = hipSuccess;
    hipEvent_t done;
    if (!d.spare.empty()) {
        done = d.spare.back();
        d.spare.pop_back();
    } else if ((e = hipEventCreateWithFlags(&done, hipEventDisableTiming)) != hipSuccess) {
        return e;
    }
    auto drop = [&](hipEvent_t ev) { d.spare.push_back(ev); };
    if (!d.pool.take(want, s, [&](hipEvent_t ev) { return (e = hipStreamWaitEvent(s, ev, 0)) == hipSuccess; }, drop)) {
        d.spare.push_back(done);
        return e != hipSuccess ? e : hipErrorInvalidValue;
    }
    e = sw_res_launch(a, dtype, scheme, rows, exact, nw, nwg, s);
    const hipError_t r = hipEventRecord(done, s);     // (also where the launch failed: behind what it waited for)
    if (r == hipSuccess) {
        d.pool.lend(want, s, done);
    } else {
        d.pool.put_back(want);
        d.spare.push_back(done);
    }
    return e != hipSuccess ? e : r;
}

// For the tests (not in sw.h): n launches in turn, none of which ends, of nwg[i] workgroups on stream[i], on a device
// of `cus` compute units; waits[i * n + k] is set where launch i is ordered behind launch k.  Returns the most shares
// kept at a time.
extern "C" int sw_internal_admission(int cus, int n, const int *nwg, const int *stream, unsigned char *waits) {
    SwCuPool<int, int> pool(cus);
    size_t most = 0;
    for (int i = 0; i < n; ++i) {
        const int want = units_of(nwg[i], cus);
        if (!pool.take(want, stream[i], [&](int k) { return waits[i * n + k] = 1, true; }, [](int) {})) return -1;
        pool.lend(want, stream[i], i);
        most = std::max(most, pool.shares());
    }
    return (int)most;
}
