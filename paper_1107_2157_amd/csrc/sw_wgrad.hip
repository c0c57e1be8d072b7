// Weight gradients of the surrogate's layers (gfx950,
// v_mfma_f32_16x16x32_bf16):
//     dW[co][tap][ci] = sum over pixels p of dZ[p][co] A[p + tap][ci],   db[co] = sum dZ[p][co]
// GEMMs with the pixels as K.  Bound by memory: dZ and A are read once, 128
// bytes a pixel for 18 kFLOP.
//
// A workgroup marches down a run of rows of one image and one group of up to
// 256 columns; wave w has 32 of the columns, one K step a row.  At the step
// of A's row r the wave reads that row's operands from LDS once (shifted by
// the three column taps) and multiplies them with dZ's rows r + 1, r and
// r - 1, the first just read, the others kept in registers: all nine taps
// are sums the wave holds, and a row of A and of dZ comes in once (with
// tiles of 4 rows, taps dealt to the waves, A came in 1.5 times and its
// operands were read from LDS three times).  Rows come in by LDS DMA, three
// ahead.  Both tensors lie pixel-major, the operands are channel-major:
// transposing LDS reads.  The waves' sums meet in LDS at the end of the run
// (FP32), the workgroups' in k_wgrad_reduce (FP64, a fixed order).
// Measured at 32 images of 256^2: 63 us (4.3 TB/s) for 32 -> 32 channels, 45
// for the first and last layer, against 87 and 66 with tiles of 4 rows (the
// gradients of 48 images in all 1.54 -> 1.42 ms).
#include "sw_conv.h"
#include "sw_conv_dev.h"
#include "sw_dma.h"

#include <algorithm>
#include <type_traits>

namespace {

typedef short i16x4 __attribute__((ext_vector_type(4)));

// Offset (BF16 elements) of 16-byte chunk c (channels 8c .. 8c + 7) of pixel
// p in a row of 32-channel pixels.  The chunk index is XORed with pixel bits
// 1-2 (the same chunk of 8 consecutive pixels covers all bank quads) and with
// pixel bit 3 into chunk bit 1 (a transposing read takes two chunks of pixels
// p .. p + 3 and p + 8 .. p + 11 in one pass; they then fall on disjoint
// banks).
__device__ __forceinline__ int tr_chunk(int p, int c) { return ((c ^ ((p >> 1) & 3) ^ ((p >> 2) & 2)) << 3) + p * 32; }

__device__ __forceinline__ i16x4 read_tr(const __bf16 *p) {
    return __builtin_amdgcn_ds_read_tr16_b64_v4i16((__attribute__((address_space(3))) i16x4 *)p);
}

// Channel-major reads of a pixel-major row with ds_read_b64_tr_b16 (gfx950):
// within each group of 16 lanes, lane i reads 4 16-bit elements and lane j
// receives element (j & 3) of the reads of lanes 4 e + (j >> 2), e = 0..3
// (probed on MI355X).  With lane i reading column quad i & 3 of pixel
// p0 + (i >> 2), lane j of the group receives column j of pixels p0 .. p0 + 3;
// two reads give the 8 consecutive pixels of one column that an MFMA operand
// lane holds (i: the lane's index in its group).  Columns: 32 channels, c0 ..
// c0 + 15; 8 channels, the channels of the pixel and those of the next.
template <int CH> __device__ __forceinline__ bf16x8 pixels8(const __bf16 *row, int p0, int c0, int i) {
    i16x4 v[2];
#pragma unroll
    for (int h = 0; h < 2; ++h) {
        const int p = p0 + 4 * h + (i >> 2), ch = c0 + 4 * (i & 3);
        v[h] = read_tr(CH == 32 ? row + tr_chunk(p, ch >> 3) + (ch & 7) : row + p * 8 + 4 * (i & 3));
    }
    return __builtin_bit_cast(bf16x8, v);
}

// The rows of a run, step after step: output rows t .. t1 - 1 counted down
// the columns of groups (group u = t / H: image u / cg, columns u % cg), each
// stretch within a group from the row of A above it to the row below it.
struct Walk {
    int t, t1, H;
    int u, r, ya, yb;   // the group, A's row, the stretch's output rows ya .. yb - 1
    __device__ __forceinline__ void stretch() {
        u = t / H;
        ya = t - u * H;
        yb = min(H, ya + t1 - t);
        r = ya - 1;
    }
    __device__ __forceinline__ void next() {   // past the last step it stays there
        if (r < yb) {
            ++r;
        } else if (t + yb - ya < t1) {
            t += yb - ya;
            stretch();
        }
    }
    __device__ __forceinline__ bool has(int y) const { return y >= ya && y < yb; }
};

// CIN, COUT: channels of A and dZ as stored (8 or 32); CG: columns of a group / 64.
template <int CIN, int COUT, int CG>
__global__ __launch_bounds__(128 * CG, 2) void k_wgrad(const __bf16 *dz, const __bf16 *x, int cout, int cin, int H, int W,
                                                       int groups, int total, int per, float *partial, int nent) {
    constexpr int NWV = 2 * CG, COLS = 64 * CG;
    constexpr int MB = COUT / 16 > 0 ? COUT / 16 : 1;        // 16-row blocks of output channels
    constexpr int CB = CIN == 32 ? 2 : 1;                    // 16-column blocks of input channels
    constexpr int NT = CIN == 32 ? 3 : 2;                    // operands of a row of taps (8 channels: taps 0 and 1 in one)
    constexpr int XS = (COLS + 2) * CIN / 8, ZS = COLS * COUT / 8;   // 16-byte slots of a row
    constexpr int XNI = (XS + 63) / 64, ZNI = ZS / 64, NI = XNI + ZNI;   // DMA instructions
    constexpr int PERW = (NI + NWV - 1) / NWV;               // most of one wave
    constexpr int ROW = NI * 64 * 8;                         // BF16 elements of a ring slot: A's row, then dZ's
    constexpr int AHEAD = 3, RING = AHEAD + 1;
    constexpr int NACC = CB * MB * NT * 4;                   // a lane's sums of one row of taps
    static_assert(ZS % 64 == 0, "dZ rows are whole instructions");
    constexpr int RINGB = RING * ROW * 2 + 16, SUMB = NWV * 64 * (NACC + MB * 4) * 4;   // (dZ of 8 channels: read to a pixel past its row)
    __shared__ __attribute__((aligned(16))) char lds[RINGB > SUMB ? RINGB : SUMB];

    const int lane = threadIdx.x & 63, w = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int n = lane & 15, kg = lane >> 4;
    const int Wp = W + 2;
    const int t0 = blockIdx.x * per, t1 = min(total, t0 + per);
    if (t0 >= t1) return;                                     // uniform per workgroup
    const int nsteps = t1 - t0 + 2 * ((t1 - 1) / H - t0 / H + 1);

    // this wave's DMA instructions i = w + NWV k (k < nw): per lane the slot's byte offset from the row's first pixel
    // (lanes past the row's end bring a slot of it into the padding again)
    const int nw = (NI - w + NWV - 1) / NWV;
    unsigned soff[PERW];
#pragma unroll
    for (int k = 0; k < PERW; ++k) {
        const int i = w + NWV * k;
        const bool isx = i < XNI;
        int sl = (isx ? i : i - XNI) * 64 + lane;
        if (isx && sl >= XS) sl = lane;
        const bool wide = (isx ? CIN : COUT) == 32;
        const int p = wide ? sl >> 2 : sl, c = wide ? (sl & 3) ^ ((p >> 1) & 3) ^ ((p >> 2) & 2) : 0;
        soff[k] = (unsigned)(wide ? p * 64 + c * 16 : p * 16);
    }
    const unsigned lds0 = lds_addr(&lds[0]);
    Walk ahead{t0, t1, H, 0, 0, 0, 0};
    ahead.stretch();
    auto issue = [&](int s) {                                 // step s's rows (of `ahead`) into ring slot s % RING
        const int img = ahead.u / groups, x0 = (ahead.u - img * groups) * COLS;
        const int64_t top = (int64_t)img * (H + 2);
        const int y = min(max(ahead.r + 1, 0), H - 1);        // dZ's row (a row outside the stretch is not used)
        const char *xb = (const char *)(x + ((top + ahead.r + 1) * Wp + x0) * CIN);
        const char *zb = (const char *)(dz + ((top + y + 1) * Wp + x0 + 1) * COUT);
        const unsigned l0 = lds0 + (unsigned)(s % RING) * (ROW * 2);
#pragma unroll
        for (int k = 0; k < PERW; ++k)
            if (k < nw) lds_dma16(w + NWV * k < XNI ? xb : zb, soff[k], l0 + (unsigned)((w + NWV * k) * 1024));
        ahead.next();
    };
    // the rows of the oldest step in flight are in (no other vector memory operation is in flight)
    auto land = [&] {
        if (nw == PERW) asm volatile("s_waitcnt vmcnt(%0)" ::"n"((AHEAD - 1) * PERW) : "memory");
        else asm volatile("s_waitcnt vmcnt(%0)" ::"n"((AHEAD - 1) * (PERW - 1)) : "memory");
        lds_barrier();
    };

    f32x4 acc[3][MB][CB][NT], accb[MB];
    bf16x8 z[3][MB];                                          // dZ's last three rows
#pragma unroll
    for (int mb = 0; mb < MB; ++mb) {
        accb[mb] = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
        for (int dy = 0; dy < 3; ++dy) {
            z[dy][mb] = bf16x8{};
#pragma unroll
            for (int cb = 0; cb < CB; ++cb)
#pragma unroll
                for (int t = 0; t < NT; ++t) acc[dy][mb][cb][t] = f32x4{0.f, 0.f, 0.f, 0.f};
        }
    }
    const u32x4 one = {0x3F803F80u, 0x3F803F80u, 0x3F803F80u, 0x3F803F80u};   // BF16 1.0 pairs
    const bf16x8 ones = __builtin_bit_cast(bf16x8, one);

    Walk at{t0, t1, H, 0, 0, 0, 0};
    at.stretch();
    for (int s = 0; s < AHEAD; ++s) issue(s);
    land();
    const int j0 = w * 32 + 8 * kg;
    auto step = [&](auto phase, int s) {
        constexpr int P = decltype(phase)::value;             // z[P] takes row r + 1; z[P - 1] holds r, z[P - 2] r - 1
        issue(s + AHEAD);
        const __bf16 *X = reinterpret_cast<const __bf16 *>(lds + (s % RING) * (ROW * 2)), *Z = X + XNI * 64 * 8;
        // row r meets dZ's row r + 1 - dy in the taps of dy (A zero where that row is none of the run's, too: values that
        // are no finite numbers must not reach sums they are no part of)
        const bool on[3] = {at.has(at.r + 1), at.has(at.r), at.has(at.r - 1)};
#pragma unroll
        for (int mb = 0; mb < MB; ++mb) z[P][mb] = on[0] ? pixels8<COUT>(Z, j0, mb * 16, n) : bf16x8{};
#pragma unroll
        for (int cb = 0; cb < CB; ++cb)
#pragma unroll
            for (int t = 0; t < NT; ++t) {
                const bf16x8 b = pixels8<CIN>(X, j0 + (CIN == 32 ? t : 2 * t), cb * 16, n);
#pragma unroll
                for (int dy = 0; dy < 3; ++dy) {
                    const bf16x8 bd = on[dy] ? b : bf16x8{};
#pragma unroll
                    for (int mb = 0; mb < MB; ++mb)
                        acc[dy][mb][cb][t] = mfma(z[(P + 3 - dy) % 3][mb], bd, acc[dy][mb][cb][t]);
                }
            }
#pragma unroll
        for (int mb = 0; mb < MB; ++mb) accb[mb] = mfma(z[P][mb], ones, accb[mb]);
        at.next();
        land();
    };
    for (int s = 0; s < nsteps; s += 3) {
        step(std::integral_constant<int, 0>{}, s);
        if (s + 1 < nsteps) step(std::integral_constant<int, 1>{}, s + 1);
        if (s + 2 < nsteps) step(std::integral_constant<int, 2>{}, s + 2);
    }
    wait_vm_upto<0>(0);
    __syncthreads();                                          // all DMA has ended: the ring is free for the sums

    // the waves' sums, a row of taps at a time: [wave][sum][lane]; D[m][n] is in lane n + 16 (m / 4), element m % 4
    float *const S = reinterpret_cast<float *>(lds);
    float *const P = partial + (int64_t)blockIdx.x * nent;
#pragma unroll
    for (int dy = 0; dy < 3; ++dy) {
        constexpr int NS = NACC + MB * 4;
        float *mine = S + w * NS * 64 + lane;
#pragma unroll
        for (int mb = 0; mb < MB; ++mb)
#pragma unroll
            for (int q = 0; q < 4; ++q) {
#pragma unroll
                for (int cb = 0; cb < CB; ++cb)
#pragma unroll
                    for (int t = 0; t < NT; ++t) mine[(((mb * CB + cb) * NT + t) * 4 + q) * 64] = acc[dy][mb][cb][t][q];
                if (dy == 0) mine[(NACC + mb * 4 + q) * 64] = accb[mb][q];
            }
        __syncthreads();
        const int ne = (dy == 0 ? NS : NACC) * 64;
        for (int e = threadIdx.x; e < ne; e += 128 * CG) {
            float v = 0.f;
#pragma unroll
            for (int k = 0; k < NWV; ++k) v += S[k * NS * 64 + e];
            const int l = e & 63, i = e >> 6, q = i & 3, col = l & 15;
            if (i < NACC) {
                const int t = (i >> 2) % NT, cb = (i >> 2) / NT % CB, mb = (i >> 2) / (NT * CB);
                const int co = mb * 16 + 4 * (l >> 4) + q;
                const int ci = CIN == 32 ? cb * 16 + col : col & 7, dx = CIN == 32 ? t : 2 * t + (col >> 3);
                if (co < cout && ci < cin && dx < 3) P[(co * 9 + 3 * dy + dx) * cin + ci] = v;
            } else {
                const int co = (i - NACC) / 4 * 16 + 4 * (l >> 4) + q;
                if (co < cout && col == 0) P[cout * 9 * cin + co] = v;
            }
        }
        __syncthreads();
    }
}

// Sum of the workgroups' partials per entry: 64 entries per block, kParts
// partial sums per entry over interleaved workgroups, combined in LDS (FP64).
// A thread's loads are what takes the time: with 4 parts 7.5 us at 256
// workgroups, with 16 5.0 us.
constexpr int kParts = 16;
__global__ __launch_bounds__(64 * kParts) void k_wgrad_reduce(const float *partial, int nblocks, int nent, int nw,
                                                              float *grad_w, float *grad_b) {
    const int e = blockIdx.x * 64 + (threadIdx.x & 63), part = threadIdx.x >> 6;
    double acc = 0.0;
    if (e < nent) {
        int k = part;
        for (; k + 3 * kParts < nblocks; k += 4 * kParts) {
            const float a0 = partial[(int64_t)k * nent + e], a1 = partial[(int64_t)(k + kParts) * nent + e];
            const float a2 = partial[(int64_t)(k + 2 * kParts) * nent + e], a3 = partial[(int64_t)(k + 3 * kParts) * nent + e];
            acc += ((double)a0 + (double)a1) + ((double)a2 + (double)a3);
        }
        for (; k < nblocks; k += kParts) acc += partial[(int64_t)k * nent + e];
    }
    __shared__ double red[kParts][64];
    red[part][threadIdx.x & 63] = acc;
    __syncthreads();
    if (part == 0 && e < nent) {
        double sum = 0.0;
#pragma unroll
        for (int k = 0; k < kParts; ++k) sum += red[k][threadIdx.x];
        if (e < nw) grad_w[e] = (float)sum;
        else grad_b[e - nw] = (float)sum;
    }
}

// Workgroups of one round, at least four rows each (fewer rows would be less
// work than the two steps and the sums that a run costs beside them).
template <int CIN, int COUT, int CG>
hipError_t launch(const __bf16 *dz, const __bf16 *x, int cout, int cin, int B, int H, int W, float *partial, int maxblocks,
                  int nent, int *used, hipStream_t s) {
    static const int resident = [] {
        int r = 0;
        return hipOccupancyMaxActiveBlocksPerMultiprocessor(&r, k_wgrad<CIN, COUT, CG>, 128 * CG, 0) == hipSuccess && r > 0 ? r : 1;
    }();
    const int groups = W / (64 * CG);
    const int64_t total = (int64_t)B * groups * H;
    if (total > (int64_t)1 << 30) return hipErrorInvalidValue;
    const int64_t most = std::min<int64_t>({(total + 3) / 4, (int64_t)sw_device_cus() * resident, (int64_t)maxblocks});
    const int per = (int)((total + most - 1) / most);
    *used = (int)((total + per - 1) / per);
    k_wgrad<CIN, COUT, CG><<<(unsigned)*used, 128 * CG, 0, s>>>(dz, x, cout, cin, H, W, groups, (int)total, per, partial, nent);
    return hipGetLastError();
}

template <int CIN, int COUT>
hipError_t launch_w(const __bf16 *dz, const __bf16 *x, int cout, int cin, int B, int H, int W, float *partial, int maxblocks,
                    int nent, int *used, hipStream_t s) {
    if (W % 256 == 0) return launch<CIN, COUT, 4>(dz, x, cout, cin, B, H, W, partial, maxblocks, nent, used, s);
    if (W % 192 == 0) return launch<CIN, COUT, 3>(dz, x, cout, cin, B, H, W, partial, maxblocks, nent, used, s);
    if (W % 128 == 0) return launch<CIN, COUT, 2>(dz, x, cout, cin, B, H, W, partial, maxblocks, nent, used, s);
    return launch<CIN, COUT, 1>(dz, x, cout, cin, B, H, W, partial, maxblocks, nent, used, s);
}

}  // namespace

hipError_t sw_sur_wgrad(const void *dzv, int coutp, int cout, const void *av, int cinp, int cin, int B, int H, int W,
                        float *partial, int nblocks, float *grad_w, float *grad_b, hipStream_t s) {
    if (B < 1 || H < 1 || W < 64 || W % 64 != 0 || nblocks < 1 || cout > coutp || cin > cinp) return hipErrorInvalidValue;
    const int nent = cout * 9 * cin + cout;
    const __bf16 *dz = (const __bf16 *)dzv, *a = (const __bf16 *)av;
    int used = 0;
    hipError_t e = hipErrorInvalidValue;
    if (cinp == 32 && coutp == 32) e = launch_w<32, 32>(dz, a, cout, cin, B, H, W, partial, nblocks, nent, &used, s);
    else if (cinp == 8 && coutp == 32) e = launch_w<8, 32>(dz, a, cout, cin, B, H, W, partial, nblocks, nent, &used, s);
    else if (cinp == 32 && coutp == 8) e = launch_w<32, 8>(dz, a, cout, cin, B, H, W, partial, nblocks, nent, &used, s);
    if (e != hipSuccess) return e;
    k_wgrad_reduce<<<(nent + 63) / 64, 64 * kParts, 0, s>>>(partial, used, nent, cout * 9 * cin, grad_w, grad_b);
    return hipGetLastError();
}
