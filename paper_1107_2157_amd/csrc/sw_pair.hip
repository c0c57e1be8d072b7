// Two consecutive 3x3 convolution layers of the surrogate in one launch, the
// activations between them in LDS only (gfx950, v_mfma_f32_16x16x32_bf16).
//
// A layer at a time, every 32-channel activation goes through memory once
// out and once in, 128 bytes per pixel and layer at 37 kFLOP: bound by
// memory at 0.28 of the matrix cores' rate.  Here a workgroup owns a run of
// rows of one image, as wide as the image (W = 64 G columns, G = 1 .. 4), and
// marches down it a row per step.  Half of its waves (role a) compute the
// first layer, half (role b) the second, a wave 64 columns; a ring of input
// rows comes in by LDS DMA, role a's rows go to a second ring, which role b
// reads a step later.  Per step a wave reads each 16-pixel operand of the new
// row from LDS once per column tap (three times) and feeds it to the three
// output rows it belongs to, whose accumulators it holds (nine reads per
// row otherwise: at 32 channels the LDS reads would take as long as the MFMAs
// at their peak).  Each accumulator still sums its taps in the order of the
// single-layer kernels (sw_conv.hip), so all results are bitwise theirs.
//
// At the top and bottom of a run role a computes one row more on either side
// (the next run computes it too); hidden rows outside the image are zero.
// The weights' rows are dealt to the MFMA's 16-row blocks so that a lane ends
// with 8 consecutive channels of a pixel: 16-byte stores to LDS and to
// memory, without a pass through LDS to gather them.
#include "sw_conv.h"
#include "sw_conv_dev.h"
#include "sw_dma.h"

#include <algorithm>
#include <type_traits>

namespace {

constexpr int kRing = 5;   // input rows in LDS

enum { FIRST_DENSE = 0, FIRST_PLANES = 1, RESID = 2 };   // role a: first layer (8-channel input or planes), residual block
                                                         // role b: residual block, or the output layer (OUT)

// relu(acc + bias) of a lane's 8 channels.
__device__ __forceinline__ void relu8(const f32x4 &lo, const f32x4 &hi, const float bias[8], float v[8]) {
#pragma unroll
    for (int q = 0; q < 4; ++q) {
        v[q] = fmaxf(lo[q] + bias[q], 0.f);
        v[4 + q] = fmaxf(hi[q] + bias[4 + q], 0.f);
    }
}
// MIDS: 0, role a's rows stay on chip; 1, they are stored; 2, they and the
// backward pass's masks are.
template <int A, bool OUT, int G, int MIDS>
__global__ __launch_bounds__(128 * G, 2) void k_conv_pair(SwPairArgs a, int rows, int nseg) {
    constexpr int W = 64 * G, PX = W + 2;
    constexpr int SLOTS = A == RESID ? PX * 4 : PX;          // 16-byte slots of an input row
    constexpr int NI = (SLOTS + 63) / 64;                    // DMA instructions per row
    constexpr int NWV = 2 * G;
    constexpr int PERW = (NI + NWV - 1) / NWV;               // per wave
    constexpr int IN_ROW = NI * 64 * 8;                      // BF16 elements (padded to whole instructions)
    constexpr int AHEAD = A == RESID ? 3 : 2;                // rows brought in ahead of the one being read
    constexpr int MBB = OUT ? 1 : 2;
    __shared__ __attribute__((aligned(16))) __bf16 in[kRing][IN_ROW];
    __shared__ __attribute__((aligned(16))) __bf16 mid[3][PX * 32];

    const int lane = threadIdx.x & 63, w = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int g = lane >> 4, n = lane & 15;
    const int role = w / G, grp = w - role * G;
    const int img = blockIdx.x / nseg, seg = blockIdx.x - img * nseg;
    const int H = a.H;
    const int ys = seg * rows, ye = min(ys + rows, H);
    if (ys >= ye) return;                                     // uniform per workgroup
    const int nsteps = ye - ys + 5;
    const int64_t img_row = (int64_t)img * (H + 2);           // first halo row of the image in a tensor

    // ---- input rows: DMA of the row whose step is s (image row ys - 2 + s) into ring slot s % kRing
    const char *const X = (const char *)a.x;
    // (every wave the same number of instructions, i = w + NWV k, so that the waits below are constants: past the
    // row's last it repeats one; the last's lanes past the row's end bring a slot of it into the padding again)
    unsigned soff[PERW], ldst[PERW];
#pragma unroll
    for (int k = 0; k < PERW; ++k) {
        const int i = (w + NWV * k) % NI;
        int sl = i * 64 + lane;
        if (sl >= SLOTS) sl = lane;
        ldst[k] = (unsigned)(i * 1024);
        const int p = A == RESID ? sl >> 2 : sl, c = A == RESID ? (sl & 3) ^ ((p >> 1) & 3) : 0;
        soff[k] = (unsigned)(A == RESID ? p * 64 + c * 16 : p * 16);
    }
    auto issue = [&](int s) {
        if constexpr (A == FIRST_PLANES) return;
        const int m = min(max(ys - 1 + s, 0), H + 1);         // tensor row (the image's row + 1); rows outside feed nothing
        const char *base = X + (img_row + m) * PX * (A == RESID ? 64 : 16);
        const unsigned l0 = lds_addr(&in[0][0]) + (unsigned)((s % kRing) * IN_ROW * 2);
#pragma unroll
        for (int k = 0; k < PERW; ++k) lds_dma16(base, soff[k], l0 + ldst[k]);
    };
    // planes: this wave's pixels of a row, read as floats and normalised (role a; its last wave also takes the last two)
    float pl[2][3];
    auto load_planes = [&](int s) {
        if constexpr (A != FIRST_PLANES) return;
        const SwBatchGrid &gd = a.grids[img];
        const int y = min(max(ys - 2 + s, -1), H);
#pragma unroll
        for (int k = 0; k < 2; ++k) {
            const int p = k ? W + lane : grp * 64 + lane;     // pixel of the row (column p - 1)
            if (k && (grp != G - 1 || lane > 1)) break;
            const int64_t off = (int64_t)y * gd.pitch + p - 1;
#pragma unroll
            for (int c = 0; c < 3; ++c) pl[k][c] = ((const float *)gd.plane[a.cur][c])[off];
        }
    };
    auto store_planes = [&](int s) {
        if constexpr (A != FIRST_PLANES) return;
#pragma unroll
        for (int k = 0; k < 2; ++k) {
            const int p = k ? W + lane : grp * 64 + lane;
            if (k && (grp != G - 1 || lane > 1)) break;
            *reinterpret_cast<bf16x8 *>(&in[s % kRing][p * 8]) =
                bf16x8{(__bf16)((pl[k][0] - a.nrm.in_off[0]) / a.nrm.in_scale[0]),
                       (__bf16)((pl[k][1] - a.nrm.in_off[1]) / a.nrm.in_scale[1]),
                       (__bf16)((pl[k][2] - a.nrm.in_off[2]) / a.nrm.in_scale[2]),
                       (__bf16)0.f, (__bf16)0.f, (__bf16)0.f, (__bf16)0.f, (__bf16)0.f};
        }
    };

    // the halo columns of the rows between the layers are zero
    if (threadIdx.x < 24) {
        const int r = threadIdx.x >> 3, e = threadIdx.x & 7;
        *reinterpret_cast<bf16x8 *>(&mid[r][chunk_off(e < 4 ? 0 : PX - 1, e & 3)]) = bf16x8{};
    }
    if (A == FIRST_PLANES && a.clear_stats && seg == 0 && threadIdx.x == 0) {
        SwGateStats &st = a.clear_stats[img];
        st.mass_old = 0.0;
        st.mass_new = 0.0;
        st.hmin = 3.0e38f;
        st.nonfinite = 0u;
    }

    // LDS offsets of this lane's operand: chunk g of pixel grp * 64 + n + dx (+ 16 per block)
    int off[3];
#pragma unroll
    for (int dx = 0; dx < 3; ++dx) off[dx] = chunk_off(grp * 64 + n + dx, g);
    const int64_t px0 = grp * 64 + n;
    // End of step s: row s + 1 is in.  It was issued at the start of step s + 1 - AHEAD; newer are the rows issued
    // since and the stores of AHEAD steps (ST of them a step from step `first` on, dropped ones too; vector memory
    // operations end in order).  The first rows were waited for before the first step; rows past the last are issued
    // all the same.
    auto land = [&](auto st, int s, int first) {
        if constexpr (A != FIRST_PLANES) {
            constexpr int ST = decltype(st)::value;
            if (s >= first + AHEAD - 1) asm volatile("s_waitcnt vmcnt(%0)" ::"n"((AHEAD - 1) * PERW + AHEAD * ST) : "memory");
            else if (s >= AHEAD - 1) asm volatile("s_waitcnt vmcnt(%0)" ::"n"((AHEAD - 1) * PERW) : "memory");
        }
        lds_barrier();
    };
    if constexpr (A != FIRST_PLANES)
        for (int s = 0; s < AHEAD; ++s) issue(s);

    if (role == 0) {
        // ---- role a
        constexpr int KS = A == RESID ? 9 : 3, KP = KS * 32;
        bf16x8 wt[KS][2];
        float bias[8];
#pragma unroll
        for (int ks = 0; ks < KS; ++ks)
#pragma unroll
            for (int mb = 0; mb < 2; ++mb)
                wt[ks][mb] = *reinterpret_cast<const bf16x8 *>((const __bf16 *)a.wa + (8 * (n >> 2) + 4 * mb + (n & 3)) * KP +
                                                               ks * 32 + 8 * g);
#pragma unroll
        for (int q = 0; q < 8; ++q) bias[q] = a.ba[8 * g + q];
        if constexpr (A == FIRST_PLANES) {
            for (int s = 0; s < 2; ++s) {
                load_planes(s);
                store_planes(s);
            }
        } else {
            wait_vm_upto<0>(0);
        }
        lds_barrier();
        f32x4 acc[A == RESID ? 3 : 1][2][4];
#pragma unroll
        for (int r = 0; r < (A == RESID ? 3 : 1); ++r)
#pragma unroll
            for (int mb = 0; mb < 2; ++mb)
#pragma unroll
                for (int pb = 0; pb < 4; ++pb) acc[r][mb][pb] = f32x4{0.f, 0.f, 0.f, 0.f};
        auto step = [&](auto phase, int s) {
            constexpr int P = decltype(phase)::value, NXT = (P + 1) % 3, MID = P, FIN = (P + 2) % 3;
            constexpr int SLOT = (P + 1) % 3, E = A == RESID ? FIN : 0;
            const int yi = ys - 2 + s, r = yi - 1;            // the new row; the row it finishes
            issue(s + AHEAD);
            load_planes(s + AHEAD);
            const bool inside = r >= 0 && r < H, keep = r >= ys && r < ye;   // else zero; else not stored
            const int64_t row = ((img_row + r + 1) * PX + 1) * 64;
            const rsrc_t ry = row_rsrc((char *)a.ya + (MIDS ? row : 0), MIDS && keep, W * 64);
            unsigned bits = 0;
            auto done = [&](int pb) {
                float v[8];
                relu8(acc[E][0][pb], acc[E][1][pb], bias, v);
                if (MIDS == 2) bits = mask_push(bits, __builtin_bit_cast(u32x4, to_bf16(v)));
                if (A == RESID) {
                    const bf16x8 xin = *reinterpret_cast<const bf16x8 *>(&in[(s + kRing - 1) % kRing][off[1] + pb * 512]);
#pragma unroll
                    for (int q = 0; q < 8; ++q) v[q] += (float)xin[q];
                }
                u32x4 o = __builtin_bit_cast(u32x4, to_bf16(v));
#pragma unroll
                for (int q = 0; q < 4; ++q) o[q] = inside ? o[q] : 0u;
                *reinterpret_cast<u32x4 *>(&mid[SLOT][off[1] + pb * 512]) = o;
                if (MIDS >= 1) store_row(ry, (int)px0 * 64 + g * 16 + pb * 1024, o);
            };
            if constexpr (A == RESID) {
                conv_row<2, NXT, MID, FIN>(in[s % kRing], off, wt, acc, done);
            } else {
                // 8 channels: four taps per K step, three rows of the ring
                const __bf16 *rowp[3] = {in[(s + kRing - 2) % kRing], in[(s + kRing - 1) % kRing], in[s % kRing]};
                const __bf16 *T[3];
                bool live[3];
#pragma unroll
                for (int ks = 0; ks < 3; ++ks) {
                    const int tap = 4 * ks + g;
                    live[ks] = tap < 9;
                    const int dy = live[ks] ? tap / 3 : 1, dx = live[ks] ? tap % 3 : 1;
                    T[ks] = (dy == 0 ? rowp[0] : dy == 1 ? rowp[1] : rowp[2]) + ((int)px0 + dx) * 8;
                }
#pragma unroll
                for (int pb = 0; pb < 4; ++pb) {
#pragma unroll
                    for (int ks = 0; ks < 3; ++ks) {
                        bf16x8 xb = *reinterpret_cast<const bf16x8 *>(T[ks] + pb * 128);
                        if (ks == 2 && !live[ks]) xb = bf16x8{};
#pragma unroll
                        for (int mb = 0; mb < 2; ++mb)
                            acc[0][mb][pb] = mfma(wt[ks][mb], xb, ks == 0 ? f32x4{0.f, 0.f, 0.f, 0.f} : acc[0][mb][pb]);
                    }
                    if (pb > 0) done(pb - 1);
                }
                done(3);
            }
            if constexpr (MIDS == 2)
                store_word(row_rsrc((char *)a.ma + ((int64_t)img * H + r) * W * 4, keep, W * 4), grp * 256 + lane * 4, bits);
            store_planes(s + AHEAD);
            land(std::integral_constant<int, MIDS == 0 ? 0 : MIDS == 2 ? 5 : 4>{}, s, 0);
        };
        // (what the last step would compute, nobody reads)
        for (int s = 0; s < nsteps - 1; s += 3) {
            step(std::integral_constant<int, 0>{}, s);
            if (s + 1 < nsteps - 1) step(std::integral_constant<int, 1>{}, s + 1);
            if (s + 2 < nsteps - 1) step(std::integral_constant<int, 2>{}, s + 2);
        }
        lds_barrier();
    } else {
        // ---- role b
        bf16x8 wt[9][MBB];
        float bias[8];
#pragma unroll
        for (int ks = 0; ks < 9; ++ks)
#pragma unroll
            for (int mb = 0; mb < MBB; ++mb)
                wt[ks][mb] = *reinterpret_cast<const bf16x8 *>(
                    (const __bf16 *)a.wb + (OUT ? n : 8 * (n >> 2) + 4 * mb + (n & 3)) * 288 + ks * 32 + 8 * g);
#pragma unroll
        for (int q = 0; q < 8; ++q) bias[q] = OUT ? (q < 3 ? a.bb[q] : 0.f) : a.bb[8 * g + q];
        if constexpr (A != FIRST_PLANES) wait_vm_upto<0>(0);
        lds_barrier();
        f32x4 acc[3][MBB][4];
#pragma unroll
        for (int r = 0; r < 3; ++r)
#pragma unroll
            for (int mb = 0; mb < MBB; ++mb)
#pragma unroll
                for (int pb = 0; pb < 4; ++pb) acc[r][mb][pb] = f32x4{0.f, 0.f, 0.f, 0.f};
        auto step = [&](auto phase, int s) {
            constexpr int P = decltype(phase)::value, NXT = (P + 1) % 3, MID = P, FIN = (P + 2) % 3;
            const int o = ys - 5 + s;                         // the row finished: the row above the one read
            issue(s + AHEAD);
            const bool keep = o >= ys;                        // (o < ye: nsteps ends there)
            if constexpr (OUT) {
                const int64_t row = ((int64_t)img * H + o) * W * 16;
                const rsrc_t r1 = row_rsrc((char *)a.yf + row, keep, W * 16);
                const rsrc_t r2 = row_rsrc((char *)a.yf2 + row, keep && a.yf2, W * 16);
                const int at = g == 0 ? (int)px0 * 16 : 0x40000000;   // the channels are in lanes 0 .. 15
                double dh = 0.0;
                conv_row<MBB, NXT, MID, FIN>(mid[P], off, wt, acc, [&](int pb) {
                    f32x4 v = acc[FIN][0][pb];
#pragma unroll
                    for (int q = 0; q < 4; ++q) v[q] = q < 3 ? v[q] + bias[q] : 0.f;
                    store_row(r1, at + pb * 256, v);
                    store_row(r2, at + pb * 256, v);
                    dh += (double)v[0];
                });
                if (a.dh_part && keep) {                      // fixed-order sum of the wave's 64 pixels
                    if (g != 0) dh = 0.0;
#pragma unroll
                    for (int k = 32; k > 0; k >>= 1) dh += __shfl_xor(dh, k);
                    if (lane == 0) a.dh_part[((int64_t)img * H + o) * G + grp] = dh;
                }
            } else {
                const int64_t row = ((img_row + o + 1) * PX + 1) * 64;
                const rsrc_t ry = row_rsrc((char *)a.yb + row, keep, W * 64);
                unsigned bits = 0;
                conv_row<MBB, NXT, MID, FIN>(mid[P], off, wt, acc, [&](int pb) {
                    float v[8];
                    relu8(acc[FIN][0][pb], acc[FIN][MBB - 1][pb], bias, v);
                    if (MIDS == 2) bits = mask_push(bits, __builtin_bit_cast(u32x4, to_bf16(v)));
                    const bf16x8 xin = *reinterpret_cast<const bf16x8 *>(&mid[(P + 2) % 3][off[1] + pb * 512]);
#pragma unroll
                    for (int q = 0; q < 8; ++q) v[q] += (float)xin[q];
                    store_row(ry, (int)px0 * 64 + g * 16 + pb * 1024, to_bf16(v));
                });
                if constexpr (MIDS == 2)
                    store_word(row_rsrc((char *)a.mb + ((int64_t)img * H + o) * W * 4, keep, W * 4), grp * 256 + lane * 4, bits);
            }
            land(std::integral_constant<int, OUT ? 8 : MIDS == 2 ? 5 : 4>{}, s, 3);
        };
        // (role a's first row of use is there in step 3)
        for (int s = 0; s < 3; ++s) {
            issue(s + AHEAD);
            land(std::integral_constant<int, 0>{}, s, 3);
        }
        for (int s = 3; s < nsteps; s += 3) {
            step(std::integral_constant<int, 0>{}, s);
            if (s + 1 < nsteps) step(std::integral_constant<int, 1>{}, s + 1);
            if (s + 2 < nsteps) step(std::integral_constant<int, 2>{}, s + 2);
        }
    }
    wait_vm_upto<0>(0);                                       // no DMA into this workgroup's LDS outlives it
}

// Rows per run: the runs fill the device in as few rounds as possible, and
// each costs 5 steps beside its rows.
template <int A, bool OUT, int G, int MIDS> hipError_t launch(const SwPairArgs &a, hipStream_t s) {
    static const int resident = [] {
        int r = 0;
        return hipOccupancyMaxActiveBlocksPerMultiprocessor(&r, k_conv_pair<A, OUT, G, MIDS>, 128 * G, 0) == hipSuccess && r > 0 ? r : 1;
    }();
    int nseg;
    const int rows = conv_run_rows(a.B, a.H, (int64_t)sw_device_cus() * resident, 5, &nseg);
    k_conv_pair<A, OUT, G, MIDS><<<(unsigned)((int64_t)a.B * nseg), 128 * G, 0, s>>>(a, rows, nseg);
    return hipGetLastError();
}

template <int A, bool OUT, int MIDS> hipError_t launch_w(const SwPairArgs &a, hipStream_t s) {
    switch (a.W) {
        case 64: return launch<A, OUT, 1, MIDS>(a, s);
        case 128: return launch<A, OUT, 2, MIDS>(a, s);
        case 192: return launch<A, OUT, 3, MIDS>(a, s);
        case 256: return launch<A, OUT, 4, MIDS>(a, s);
    }
    return hipErrorInvalidValue;
}

template <int A, bool OUT> hipError_t launch_mids(const SwPairArgs &a, hipStream_t s) {
    if (!a.ya) return a.ma || a.mb ? hipErrorInvalidValue : launch_w<A, OUT, 0>(a, s);
    if (!a.ma && !a.mb) return launch_w<A, OUT, 1>(a, s);
    if (!a.ma || (a.mb != nullptr) == OUT) return hipErrorInvalidValue;
    return launch_w<A, OUT, 2>(a, s);
}

}  // namespace

bool sw_conv_pair_fits(int H, int W) { return H >= 1 && W >= 64 && W <= 256 && W % 64 == 0; }

hipError_t sw_conv_pair(const SwPairArgs &a, int pair, hipStream_t s) {
    if (a.B < 1 || !sw_conv_pair_fits(a.H, a.W) || (int64_t)a.B * a.H > (int64_t)1 << 30 || !a.wa || !a.wb || !a.ba || !a.bb)
        return hipErrorInvalidValue;
    if (pair == SW_PAIR_OUT ? !a.yf || !a.x : !a.yb) return hipErrorInvalidValue;
    if (pair == SW_PAIR_FIRST && a.grids) {
        if (a.ma || a.mb) return hipErrorInvalidValue;
        return a.ya ? launch_w<FIRST_PLANES, false, 1>(a, s) : launch_w<FIRST_PLANES, false, 0>(a, s);
    }
    if (pair == SW_PAIR_FIRST) return a.x ? launch_mids<FIRST_DENSE, false>(a, s) : hipErrorInvalidValue;
    if (!a.x) return hipErrorInvalidValue;
    return pair == SW_PAIR_OUT ? launch_mids<RESID, true>(a, s) : launch_mids<RESID, false>(a, s);
}

// For the tests (not in sw.h).
extern "C" int sw_internal_run_rows(int B, int H, long long slots, int extra, int *nseg, int *trials) {
    return conv_run_rows(B, H, slots, extra, nseg, trials);
}
