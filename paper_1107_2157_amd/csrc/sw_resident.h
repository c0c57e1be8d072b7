// Internal interface of the resident time loop (sw_resident_kernel.h, sw_resident.cpp):
// all steps of a call in one launch, the state held in registers throughout.
#pragma once
#include <hip/hip_runtime.h>
#include <cmath>
#include <cstdint>
#include <vector>

#include "sw_batch_internal.h"

// Launch control of one team (the workgroups of one grid), zero between
// launches except for the epoch.
struct SwResCtl {
    unsigned epoch;   // exchange tags of a launch are epoch + 1 ... epoch + nsteps
    unsigned state;   // 0 gathering, 1 every workgroup of the team is resident, 2 given up
    unsigned exits;   // workgroups that are done
    unsigned pad;
};

// How one grid is cut up.  Strips of ws columns (one lane each, plus a halo
// lane on either side); per strip `waves` waves hold consecutive runs of
// rows, base + 1 rows each for the first rem of them and base for the rest;
// a workgroup is nw consecutive waves of one strip.
struct SwResTeam {
    int32_t wg0, nwg;        // workgroups [wg0, wg0 + nwg), block-major: member = block * ns + strip
    int32_t ns, ws, nb;
    int32_t waves, base, rem;
    int32_t nx, ny;
    int64_t pitch;
    uint64_t words;          // first exchange word of the team
};

struct SwResArgs {
    SwResTeam one;           // the team of a single grid (teams == nullptr)
    void *plane[2][3];       // its planes at interior cell (0, 0)
    SwScalars *sc;
    const SwResTeam *teams;  // batch: per grid
    const int32_t *wg_team;  // batch: workgroup -> team
    const SwBatchGrid *grids;
    SwBatchScalars *bsc;
    unsigned long long *words;
    SwResCtl *ctl;           // per team
    int32_t cur, nsteps;
    int32_t bc_x, bc_y;
    double g, dx, dy, cfl, dt_fixed;
    double rdx, rdy;         // 1 / dx, 1 / dy where they are powers of two, else 0
    int32_t poll_first, poll_next;   // waits before a step's first poll and between polls, in 128 cycles
    int64_t patience;        // 100 MHz ticks a workgroup waits for the rest of its team to start
};

// A cut of one grid that fits the device, and what it needs.
struct SwResPlan {
    int rows;                // most rows of a wave
    int nw;                  // waves per workgroup
    bool exact;              // every active wave has rows or rows - 1, and there is an instance for that
    SwResTeam team;          // wg0 and words are the caller's
    uint64_t nwords;         // exchange words (8 bytes)
    int most_steps;          // steps of one launch at most (sw_res_plan)
};

constexpr int64_t kResPatience = 500000000;   // 5 s in ticks of the 100 MHz clock
// Estimated time of one launch at most (us); longer calls are several
// launches.  In a batch of more workgroups than fit a team waits for the teams
// before it, a whole launch at worst, and must not run out of patience; and
// where a team gives up, what one workgroup then does alone is a launch, not
// the call.  A launch costs 20 us beside its steps, in a batch a reading and
// writing of all states: longer there.
constexpr double kResLaunchUs = 20e3, kResBatchLaunchUs = 100e3;
constexpr int kResFlagWords = 4;   // exchange words from one workgroup's flag to the next (32 bytes)
constexpr int kResPollFirst = 9;   // 128 cycles each: 0.5 us
// Between polls: none is the fastest, but for the few cycles that asking takes
// (dam break of 128^2 FP64, 100 steps: 319.0 us; without the question 320.0;
// 1024^2 FP32: 562.5 / 565.3, with 64 cycles 565.5).
constexpr int kResPollNext = 0;
constexpr int kResStrip = 62;      // most columns of a strip
constexpr int kResRows = 16;       // most rows of a wave with 16 (FP32) or 8 (FP64) waves to a CU
constexpr int kResRoomy = 10;      // FP32 patches from this height take twice the registers where nw <= 8
constexpr int kResRowsTall = 40;   // FP32 with 8 waves to a CU (twice the registers each)

// The instantiated exact row counts.
#define SW_RES_ROWS(X) X(1) X(2) X(3) X(4) X(5) X(6) X(8) X(10) X(12) X(14) X(16)
#define SW_RES_ROOMY(X) X(10) X(12) X(14) X(16)
#define SW_RES_TALL(X) X(18) X(20) X(22) X(24) X(28) X(32) X(36) X(40)

inline bool sw_res_has_rows(int rows) {
#define SW_RES_IS(R) if (rows == R) return true;
    SW_RES_ROWS(SW_RES_IS) SW_RES_TALL(SW_RES_IS)
#undef SW_RES_IS
    return false;
}
// Whether waves of `rows` rows, nw to a workgroup, have an instance.
inline bool sw_res_shape_ok(int dtype, int rows, int nw) {
    if (rows < 1 || nw < 1) return false;
    if (rows <= kResRows) return nw <= (dtype ? 8 : 16);
    return !dtype && rows <= kResRowsTall && nw <= 8;
}

// Cut an nx x ny grid into patches of at most max_rows rows for workgroups
// of nw waves, at most max_wg of them (wg0 and words are left 0); false if
// it does not fit.  spread: over all the waves of those workgroups, in a
// height that has an exact instance if possible; otherwise over as few waves
// as max_rows allows.
bool sw_res_cut(int dtype, int nx, int ny, int64_t pitch, int nw, int max_rows, int max_wg, bool spread, SwResPlan *out);
// The cut for a grid that has the device to itself.
bool sw_res_plan(int dtype, int nx, int ny, int64_t pitch, int cus, SwResPlan *out);

// The cut of a batch: teams in order of size, largest first.
struct SwResBatchPlan {
    std::vector<SwResTeam> teams;      // per grid
    std::vector<int32_t> wg_team;      // workgroup -> grid
    uint64_t nwords;
    int rows, nw;
    bool exact;
    int from_steps;                    // calls of fewer steps are faster as per-step launches
    int most_steps;                    // steps of one launch at most
};
// False where the per-step launches are the faster form, or a grid does not fit.
bool sw_res_plan_batch(int dtype, int scheme, int n, const int *nx, const int *ny, const int64_t *pitch, int cus,
                       SwResBatchPlan *out);

// Steps of the next launch of a call with `left` steps to go: as many launches
// as `most` asks for, of about equal length.
inline int sw_res_next_steps(int left, int most) {
    const int launches = (int)(((int64_t)left + most - 1) / most);
    return (int)(((int64_t)left + launches - 1) / launches);
}

// Whether resident launches may go to the stream: it is not under capture (or
// cannot be asked), and its kernels may use every compute unit (a team cut for
// the device would never find room on a stream created with a mask of fewer,
// and wait out its patience each call).
bool sw_res_stream_ok(hipStream_t s, int cus);

// 1 / x where that is exact for every product with it, else 0.
inline double sw_res_exact_inverse(double x) {
    int e = 0;
    return std::frexp(x, &e) == 0.5 && e > -1000 && e < 1000 ? 1.0 / x : 0.0;
}

// Device memory that a context or batch can do without (it then takes the
// per-step launches): null where there is not enough.
hipError_t sw_res_alloc(void **p, size_t bytes);

// Launch nwg workgroups of nw waves.  rows: the most rows of any wave; exact:
// every active wave has rows or rows - 1.
hipError_t sw_res_launch(const SwResArgs &a, int dtype, int scheme, int rows, bool exact, int nw, int nwg, hipStream_t s);
// The same behind the admission of resident launches (sw_resident.cpp):
// enqueued on s after as many earlier ones as have to be done for all its
// workgroups to find room.  Not for streams under capture.
hipError_t sw_res_launch_admitted(const SwResArgs &a, int dtype, int scheme, int rows, bool exact, int nw, int nwg,
                                  int device, int cus, hipStream_t s);
