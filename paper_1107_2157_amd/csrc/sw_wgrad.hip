// Weight gradients of the surrogate's layers (gfx950,
// v_mfma_f32_16x16x32_bf16):
//     dW[co][tap][ci] = sum over pixels p of dZ[p][co] A[p + tap][ci],   db[co] = sum dZ[p][co]
// GEMMs with the pixels as K.  Bound by memory: dZ and A are read once, 128
// bytes a pixel for 18 kFLOP.  Two forms:
//
// Rows (k_wgrad_rows), images of a multiple of 256 columns in large batches.
// A workgroup marches down a run of rows of one image's group of 256 columns;
// a wave has 32 of the columns, one K step a row.  At the step of A's row r
// the wave reads that row's operands from LDS once (shifted by the three
// column taps) and multiplies them with dZ's rows r + 1, r and r - 1, the
// first just read, the others kept in registers: all nine taps are sums the
// wave holds, and a row of A and of dZ comes in once.  Rows come in by LDS
// DMA, three ahead.
//
// Tiles (k_wgrad, k_wgrad_dma), the rest: the taps dealt to the waves, A
// brought in 1.5 times.
//
// Both tensors lie pixel-major, the operands are channel-major: transposing
// LDS reads.  The workgroups' sums (FP32) meet in k_wgrad_reduce (FP64, a
// fixed order).  Measured at 32 images of 256^2, rows against tiles: 63 us
// (4.3 TB/s) / 87 for 32 -> 32 channels, 45 / 66 for the first and last layer.
#include "sw_conv.h"
#include "sw_conv_dev.h"
#include "sw_dma.h"

#include <algorithm>

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

// CIN, COUT: channels of A and dZ as stored (8 or 32).
constexpr int kRowWaves = 8, kRowCols = 32 * kRowWaves;
template <int CIN, int COUT>
__global__ __launch_bounds__(64 * kRowWaves, 2) void k_wgrad_rows(const __bf16 *dz, const __bf16 *x, int cout, int cin, int H, int W,
                                                       int groups, int total, int per, float *partial, int nent) {
    constexpr int NWV = kRowWaves, COLS = kRowCols;
    constexpr int MB = COUT / 16 > 0 ? COUT / 16 : 1;        // 16-row blocks of output channels
    constexpr int CB = CIN == 32 ? 2 : 1;                    // 16-column blocks of input channels
    constexpr int NT = CIN == 32 ? 3 : 2;                    // operands of a row of taps (8 channels: taps 0 and 1 in one)
    constexpr int XS = (COLS + 2) * CIN / 8, ZS = COLS * COUT / 8;   // 16-byte slots of a row
    constexpr int XNI = (XS + 63) / 64, ZNI = ZS / 64, NI = XNI + ZNI;   // DMA instructions
    constexpr int PERW = (NI + NWV - 1) / NWV;               // most of one wave
    constexpr int ROW = NI * 64 * 8;                         // BF16 elements of a ring slot: A's row, then dZ's
    constexpr int AHEAD = 3, RING = AHEAD + 1;
    static_assert(ZS % 64 == 0, "dZ rows are whole instructions");
    constexpr int RINGB = RING * ROW * 2 + 16, SUMB = NWV * 64 * (CB * MB * NT + MB) * 16;   // (dZ of 8 channels: read to a pixel past its row)
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
    bf16x8 z[3][MB];                                          // dZ's last three rows, r + 1 first
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
#pragma unroll 1
    for (int s = 0; s < AHEAD; ++s) issue(s);
    land();
    const int j0 = w * 32 + 8 * kg;
    // (one body for all steps: dZ's rows move through z; unrolled threefold to leave them in place, the code was 30 KB)
#pragma unroll 1
    for (int s = 0; s < nsteps; ++s) {
        issue(s + AHEAD);
        const __bf16 *X = reinterpret_cast<const __bf16 *>(lds + (s % RING) * (ROW * 2)), *Z = X + XNI * 64 * 8;
        // row r meets dZ's row r + 1 - dy in the taps of dy (A zero where that row is none of the run's, too: values that
        // are no finite numbers must not reach sums they are no part of)
        const bool on[3] = {at.has(at.r + 1), at.has(at.r), at.has(at.r - 1)};
#pragma unroll
        for (int mb = 0; mb < MB; ++mb) {
            z[2][mb] = z[1][mb];
            z[1][mb] = z[0][mb];
            z[0][mb] = on[0] ? pixels8<COUT>(Z, j0, mb * 16, n) : bf16x8{};
        }
#pragma unroll
        for (int cb = 0; cb < CB; ++cb)
#pragma unroll
            for (int t = 0; t < NT; ++t) {
                const bf16x8 b = pixels8<CIN>(X, j0 + (CIN == 32 ? t : 2 * t), cb * 16, n);
#pragma unroll
                for (int dy = 0; dy < 3; ++dy) {
                    const bf16x8 bd = on[dy] ? b : bf16x8{};
#pragma unroll
                    for (int mb = 0; mb < MB; ++mb) acc[dy][mb][cb][t] = mfma(z[dy][mb], bd, acc[dy][mb][cb][t]);
                }
            }
#pragma unroll
        for (int mb = 0; mb < MB; ++mb) accb[mb] = mfma(z[0][mb], ones, accb[mb]);
        at.next();
        land();
    }
    wait_vm_upto<0>(0);
    __syncthreads();                                          // all DMA has ended: the ring is free for the sums

    // the waves' sums, a row of taps at a time: [wave][four sums][lane]; D[m][n] is in lane n + 16 (m / 4), element
    // m % 4.  Wave w adds up the quadruples w, w + NWV, ... (with the bias's in the first round).
    constexpr int NQ = MB * CB * NT, NQB = NQ + MB;
    f32x4 *const S = reinterpret_cast<f32x4 *>(lds);
    float *const P = partial + (int64_t)blockIdx.x * nent;
#pragma unroll
    for (int dy = 0; dy < 3; ++dy) {
        f32x4 *mine = S + w * NQB * 64 + lane;
#pragma unroll
        for (int mb = 0; mb < MB; ++mb) {
#pragma unroll
            for (int cb = 0; cb < CB; ++cb)
#pragma unroll
                for (int t = 0; t < NT; ++t) mine[((mb * CB + cb) * NT + t) * 64] = acc[dy][mb][cb][t];
            if (dy == 0) mine[(NQ + mb) * 64] = accb[mb];
        }
        lds_barrier();
#pragma unroll 1
        for (int i = w; i < (dy == 0 ? NQB : NQ); i += NWV) {
            f32x4 v = S[i * 64 + lane];
#pragma unroll
            for (int k = 1; k < NWV; ++k) v += S[(k * NQB + i) * 64 + lane];
            const int mb = i < NQ ? i / (NT * CB) : i - NQ, cb = i / NT % CB, t = i % NT;
            const int ci = CIN == 32 ? cb * 16 + n : n & 7, dx = CIN == 32 ? t : 2 * t + (n >> 3);
#pragma unroll
            for (int q = 0; q < 4; ++q) {
                const int co = mb * 16 + 4 * kg + q;
                if (co >= cout) continue;
                if (i >= NQ) {
                    if (n == 0) P[cout * 9 * cin + co] = v[q];
                } else if (ci < cin && dx < 3) {
                    P[(co * 9 + 3 * dy + dx) * cin + ci] = v[q];
                }
            }
        }
        if (dy < 2) lds_barrier();
    }
}

// ---- small batches: tiles

// Weight gradient partials on MFMA (v_mfma_f32_16x16x32_bf16), K = pixels:
//     dW[co][(tap, ci)] = sum_p dZ[p][co] A[p + off(tap)][ci]
// read from the NHWC tensors.  Persistent blocks walk contiguous runs of
// 4-row x 64-pixel tiles, numbered down the columns of tiles (the next tile's
// halo rows are still in L2), and keep dW in registers.  A tile's dZ (4 x 64
// pixels) and input rows (6 x 66 pixels, halo included) are staged in LDS
// transposed, channel-major with the pixels contiguous, so 8 consecutive
// pixels of one channel are one 16-byte LDS read (row strides padded so the
// reads of 16 channels are conflict free); the next tile's global loads are
// in flight during the MFMAs.  A K step is 32 pixels of one row: lane
// (n, kg) = (lane % 16, lane / 16) takes pixels j0 = 8 kg .. + 7 of the step.
// Wave w owns input row dy = w / CH and, for CINP = 32, channel half w % CH,
// i.e. the taps (dy, 0..2) of 16 input channels: two aligned reads give all
// three column shifts (dx = 1 by a 16-bit funnel shift, dx = 2 by a dword
// shift).  For CINP = 8 a 16-wide N tile holds two taps of 8 channels.  Wave
// 0 also forms db with an all-ones operand.

__device__ __forceinline__ bf16x8 as_bf16x8(u32x4 v) { return __builtin_bit_cast(bf16x8, v); }

constexpr int kWgRows = 4, kWgCols = 64;

template <int CINP, int COUTP>
__global__ __launch_bounds__(CINP == 32 ? 384 : 192) void k_wgrad(const __bf16 *dz, const __bf16 *a, int cout, int cin,
                                                                  int H, int W, int tiles_y, int tiles_x, int ntiles,
                                                                  float *partial, int nent) {
    constexpr int CH = CINP == 32 ? 2 : 1;
    constexpr int NTH = 64 * 3 * CH;
    constexpr int MB = (COUTP + 15) / 16;
    constexpr int NT = CINP == 32 ? 3 : 2;
    constexpr int DZS = kWgRows * kWgCols + 8;               // per output channel (padded)
    constexpr int AROW = 72, AS = (kWgRows + 2) * AROW + 8;  // per input channel (padded)
    constexpr int NKO = COUTP / 8, NKI = CINP / 8;
    constexpr int DZ_CH = kWgRows * NKO * kWgCols, A_CH = (kWgRows + 2) * NKI * (kWgCols + 2);
    constexpr int DZ_PER = (DZ_CH + NTH - 1) / NTH, A_PER = (A_CH + NTH - 1) / NTH;
    __shared__ __attribute__((aligned(16))) __bf16 dzT[COUTP * DZS];
    __shared__ __attribute__((aligned(16))) __bf16 aT[CINP * AS];

    const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
    const int n = lane & 15, kg = lane >> 4;
    const int dy = w / CH, chalf = w % CH;
    const int ci = CINP == 32 ? chalf * 16 + n : (n & 7);
    const int Wp = W + 2;
    const int per_block = (ntiles + gridDim.x - 1) / gridDim.x;
    const int t0 = blockIdx.x * per_block, t1 = min(ntiles, t0 + per_block);
    const u32x4 ones = {0x3F803F80u, 0x3F803F80u, 0x3F803F80u, 0x3F803F80u};   // bf16 1.0 pairs

    f32x4 acc[MB][NT], accb[MB];
#pragma unroll
    for (int mb = 0; mb < MB; ++mb) {
        accb[mb] = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
        for (int t = 0; t < NT; ++t) acc[mb][t] = f32x4{0.f, 0.f, 0.f, 0.f};
    }

    bf16x8 sdz[DZ_PER], sa[A_PER];
    auto load_tile = [&](int t) {
        const int b = t / (tiles_y * tiles_x);
        const int r = t - b * tiles_y * tiles_x;
        const int tx = r / tiles_y, ty = r - tx * tiles_y;   // column-major: the next tile is the one below
#pragma unroll
        for (int k = 0; k < DZ_PER; ++k) {   // chunk c = (row * NKO + part) * 64 + p
            const int c = threadIdx.x + k * NTH;
            const int p = c % kWgCols, rp = c / kWgCols;
            const int row = rp / NKO, part = rp - row * NKO;
            const int y = ty * kWgRows + row;
            sdz[k] = bf16x8{};
            if (c < DZ_CH && y < H)
                sdz[k] = *reinterpret_cast<const bf16x8 *>(
                    dz + (((int64_t)b * (H + 2) + y + 1) * Wp + tx * kWgCols + 1 + p) * COUTP + part * 8);
        }
#pragma unroll
        for (int k = 0; k < A_PER; ++k) {    // chunk c = (row * NKI + part) * 66 + p, halo coordinates
            const int c = threadIdx.x + k * NTH;
            const int p = c % (kWgCols + 2), rp = c / (kWgCols + 2);
            const int row = rp / NKI, part = rp - row * NKI;
            const int yy = ty * kWgRows + row;
            sa[k] = bf16x8{};
            if (c < A_CH && yy < H + 2)
                sa[k] = *reinterpret_cast<const bf16x8 *>(
                    a + (((int64_t)b * (H + 2) + yy) * Wp + tx * kWgCols + p) * CINP + part * 8);
        }
    };
    auto store_tile = [&]() {   // transposing writes: lanes of a wave take consecutive pixels
#pragma unroll
        for (int k = 0; k < DZ_PER; ++k) {
            const int c = threadIdx.x + k * NTH;
            if (c >= DZ_CH) continue;
            const int p = c % kWgCols, rp = c / kWgCols;
            const int row = rp / NKO, part = rp - row * NKO;
#pragma unroll
            for (int e = 0; e < 8; ++e) dzT[(part * 8 + e) * DZS + row * kWgCols + p] = sdz[k][e];
        }
#pragma unroll
        for (int k = 0; k < A_PER; ++k) {
            const int c = threadIdx.x + k * NTH;
            if (c >= A_CH) continue;
            const int p = c % (kWgCols + 2), rp = c / (kWgCols + 2);
            const int row = rp / NKI, part = rp - row * NKI;
#pragma unroll
            for (int e = 0; e < 8; ++e) aT[(part * 8 + e) * AS + row * AROW + p] = sa[k][e];
        }
    };

    if (t0 < t1) load_tile(t0);
    for (int t = t0; t < t1; ++t) {
        __syncthreads();                  // the previous tile's reads of LDS are done
        store_tile();
        __syncthreads();
        if (t + 1 < t1) load_tile(t + 1); // in flight during the MFMAs below
#pragma unroll
        for (int kc = 0; kc < 2 * kWgRows; ++kc) {
            const int r = kc >> 1, j0 = (kc & 1) * 32 + 8 * kg;
            bf16x8 aop[MB];
#pragma unroll
            for (int mb = 0; mb < MB; ++mb) {
                const int co = mb * 16 + n;
                aop[mb] = co < COUTP ? *reinterpret_cast<const bf16x8 *>(&dzT[co * DZS + r * kWgCols + j0]) : bf16x8{};
            }
            const __bf16 *row = &aT[ci * AS + (r + dy) * AROW + j0];
            const u32x4 v0 = *reinterpret_cast<const u32x4 *>(row);
            const u32x4 v1 = *reinterpret_cast<const u32x4 *>(row + 8);
            // staged pixel j0 + dx + e is input pixel x0 + j0 + e + dx - 1: dx = 0, 1, 2
            const u32x4 s1 = {__builtin_amdgcn_alignbit(v0[1], v0[0], 16), __builtin_amdgcn_alignbit(v0[2], v0[1], 16),
                              __builtin_amdgcn_alignbit(v0[3], v0[2], 16), __builtin_amdgcn_alignbit(v1[0], v0[3], 16)};
            const u32x4 s2 = {v0[1], v0[2], v0[3], v1[0]};
            bf16x8 bop[NT];
            if (CINP == 32) {
                bop[0] = as_bf16x8(v0);
                bop[1] = as_bf16x8(s1);
                bop[2] = as_bf16x8(s2);
            } else {
                bop[0] = as_bf16x8(n < 8 ? v0 : s1);
                bop[1] = n < 8 ? as_bf16x8(s2) : bf16x8{};
            }
#pragma unroll
            for (int mb = 0; mb < MB; ++mb) {
#pragma unroll
                for (int tt = 0; tt < NT; ++tt)
                    acc[mb][tt] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(aop[mb], bop[tt], acc[mb][tt], 0, 0, 0);
                if (w == 0) accb[mb] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(aop[mb], as_bf16x8(ones), accb[mb], 0, 0, 0);
            }
        }
    }
    // D[m][n] in lane n + 16 (m / 4), element m % 4
    float *P = partial + (int64_t)blockIdx.x * nent;
#pragma unroll
    for (int mb = 0; mb < MB; ++mb)
#pragma unroll
        for (int q = 0; q < 4; ++q) {
            const int co = mb * 16 + 4 * kg + q;
            if (co >= cout) continue;
#pragma unroll
            for (int tt = 0; tt < NT; ++tt) {
                int tap, cc;
                if (CINP == 32) {
                    tap = 3 * dy + tt;
                    cc = ci;
                } else {
                    tap = 3 * dy + (tt == 0 ? (n >> 3) : 2);
                    cc = n & 7;
                    if (tt == 1 && n >= 8) continue;
                }
                if (cc < cin) P[(co * 9 + tap) * cin + cc] = acc[mb][tt][q];
            }
            if (w == 0 && n == 0) P[cout * 9 * cin + co] = accb[mb][q];
        }
}

// Weight gradient of a 32 -> 32 layer: k_wgrad's tile walk and MFMA
// operands for 32 channels, with the tiles brought in by LDS DMA,
// pixel-major as they lie in HBM, three buffers deep (two tiles' loads in
// flight while one is computed; one workgroup per CU, the buffers fill 123 KB
// of LDS), and the operands read channel-major with transposing LDS reads
// instead of staged transposed.  12 waves: wave w takes input row dy = u / 2
// and channel half u % 2 (u = w % 6) of the K steps over pixel half w / 6 of
// each tile row (three waves per SIMD hide each other's LDS latency); the
// two halves' sums meet in LDS at the end.  A tile's 16-byte slots: dZ (4 x
// 64 pixels) then the input (6 x 66 pixels, padded to whole DMA
// instructions; padding lanes reload a slot of the window and land past its
// end); slot s holds chunk (s & 3) ^ swizzle of pixel s >> 2 (tr_chunk).  dZ
// rows below the image (the last tile row of an image whose height is not a
// multiple of 4) are loaded from its last row and their K steps skipped;
// input rows below the bottom halo row feed only those steps.  The loop
// issues no vector memory operation other than the DMA, so waiting for all
// but the newest tile's DMA instructions leaves exactly that tile in flight.
__global__ __launch_bounds__(768) void k_wgrad_dma(const __bf16 *dz, const __bf16 *a, int cout, int cin, int H, int W,
                                                    int tiles_y, int tiles_x, int ntiles, float *partial, int nent) {
    constexpr int NWV = 12, MB = 2, NT = 3;
    constexpr int DZ_SLOTS = kWgRows * kWgCols * 4;
    constexpr int A_SLOTS = (kWgRows + 2) * (kWgCols + 2) * 4;
    constexpr int DZ_NI = DZ_SLOTS / 64;
    constexpr int A_NI = (A_SLOTS + 63) / 64;
    constexpr int NI = DZ_NI + A_NI;                 // DMA instructions per tile
    constexpr int BUF = NI * 64 * 8;                 // bf16 per buffer
    constexpr int PERW = (NI + NWV - 1) / NWV;       // most instructions of one wave
    constexpr int NBUF = 3;
    constexpr int NACC = MB * NT * 4 + MB * 4;       // a lane's sums (with the bias's)
    static_assert(6 * 64 * NACC * 4 <= NBUF * BUF * 2, "the halves' sums fit the tile buffers");
    __shared__ __attribute__((aligned(16))) __bf16 tiles[NBUF][BUF];

    const int lane = threadIdx.x & 63, w = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int n = lane & 15, kg = lane >> 4;
    const int u = w % 6, half = w / 6;
    const int dy = u >> 1, chalf = u & 1;
    const bool bias_wave = u == 0;
    const int Wp = W + 2;
    const int per_block = (ntiles + gridDim.x - 1) / gridDim.x;
    const int t0 = blockIdx.x * per_block, t1 = min(ntiles, t0 + per_block);
    const u32x4 ones = {0x3F803F80u, 0x3F803F80u, 0x3F803F80u, 0x3F803F80u};   // bf16 1.0 pairs

    f32x4 acc[MB][NT], accb[MB];
#pragma unroll
    for (int mb = 0; mb < MB; ++mb) {
        accb[mb] = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
        for (int t = 0; t < NT; ++t) acc[mb][t] = f32x4{0.f, 0.f, 0.f, 0.f};
    }

    // this wave's DMA instructions i = w + 12 k (k < nw): per lane the slot's
    // byte offset from its window's first pixel, and its window row
    const int nw = (NI - w + NWV - 1) / NWV;
    unsigned soff[PERW];
    int srow[PERW];
#pragma unroll
    for (int k = 0; k < PERW; ++k) {
        const int i = w + NWV * k;
        const bool isdz = i < DZ_NI;
        const int cols = isdz ? kWgCols : kWgCols + 2;
        int sl = (isdz ? i : i - DZ_NI) * 64 + lane;
        if (!isdz && sl >= A_SLOTS) sl = lane;
        const int p = sl >> 2, c = (sl & 3) ^ ((p >> 1) & 3) ^ ((p >> 2) & 2);
        const int row = p / cols, col = p - row * cols;
        soff[k] = (unsigned)(((row * Wp + col) * 32 + c * 8) * 2);
        srow[k] = row;
    }
    const unsigned lds0 = lds_addr(&tiles[0][0]);
    auto issue = [&](int t, int buf) {
        const int b = t / (tiles_y * tiles_x);
        const int r = t - b * tiles_y * tiles_x;
        const int tx = r / tiles_y, ty = r - tx * tiles_y;   // column-major: the next tile is the one below
        const char *zb = (const char *)(dz + ((((int64_t)b * (H + 2) + ty * kWgRows + 1) * Wp + tx * kWgCols + 1) * 32));
        const char *ab = (const char *)(a + ((((int64_t)b * (H + 2) + ty * kWgRows) * Wp + tx * kWgCols) * 32));
        const int rz = H - 1 - ty * kWgRows, ra = H + 1 - ty * kWgRows;   // last window rows inside the image
        const unsigned l0 = lds0 + (unsigned)(buf * BUF * 2);
#pragma unroll
        for (int k = 0; k < PERW; ++k) {
            if (k < nw) {
                const int i = w + NWV * k;
                const bool isdz = i < DZ_NI;
                const int rm = isdz ? rz : ra;
                const unsigned off = srow[k] > rm ? soff[k] - (unsigned)((srow[k] - rm) * Wp * 64) : soff[k];
                lds_dma16(isdz ? zb : ab, off, l0 + (unsigned)(i * 1024));
            }
        }
    };

    if (t0 < t1) {
        issue(t0, 0);
        if (t0 + 1 < t1) issue(t0 + 1, 1);
        wait_vm_upto<PERW>(t0 + 1 < t1 ? nw : 0);      // tile t0 has landed
    }
    __syncthreads();
    for (int t = t0; t < t1; ++t) {
        const int buf = (t - t0) % NBUF;
        if (t + 2 < t1) issue(t + 2, (t - t0 + 2) % NBUF);   // its buffer was last read before the barrier
        const int r0 = t - (t / (tiles_y * tiles_x)) * tiles_y * tiles_x;
        const int ty = r0 - (r0 / tiles_y) * tiles_y;
        const int rows = min(kWgRows, H - ty * kWgRows);
        const __bf16 *DZ = tiles[buf];
        const __bf16 *AT = tiles[buf] + DZ_SLOTS * 8;
#pragma unroll
        for (int r = 0; r < kWgRows; ++r) {
            if (r >= rows) break;
            const int j0 = half * 32 + 8 * kg;
            bf16x8 aop[MB], bop[NT];
            // dZ: channel mb * 16 + n of pixels j0 .. j0 + 7 of row r; the
            // input: channel 16 chalf + n of staged pixels j0 + dx .. + 7 of row r + dy
#pragma unroll
            for (int mb = 0; mb < MB; ++mb) aop[mb] = pixels8<32>(DZ, r * kWgCols + j0, mb * 16, n);
#pragma unroll
            for (int dx = 0; dx < NT; ++dx) bop[dx] = pixels8<32>(AT, (r + dy) * (kWgCols + 2) + j0 + dx, chalf * 16, n);
#pragma unroll
            for (int mb = 0; mb < MB; ++mb) {
#pragma unroll
                for (int tt = 0; tt < NT; ++tt)
                    acc[mb][tt] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(aop[mb], bop[tt], acc[mb][tt], 0, 0, 0);
                if (bias_wave)
                    accb[mb] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(aop[mb], as_bf16x8(ones), accb[mb], 0, 0, 0);
            }
        }
        if (t + 1 < t1) wait_vm_upto<PERW>(t + 2 < t1 ? nw : 0);   // tile t + 1 has landed
        __syncthreads();
    }
    // the second pixel half's sums join the first's (the tile buffers are free)
    float *X = reinterpret_cast<float *>(&tiles[0][0]) + (u * 64 + lane) * NACC;
    if (half == 1) {
#pragma unroll
        for (int mb = 0; mb < MB; ++mb) {
#pragma unroll
            for (int tt = 0; tt < NT; ++tt)
#pragma unroll
                for (int q = 0; q < 4; ++q) X[(mb * NT + tt) * 4 + q] = acc[mb][tt][q];
#pragma unroll
            for (int q = 0; q < 4; ++q) X[MB * NT * 4 + mb * 4 + q] = accb[mb][q];
        }
    }
    __syncthreads();
    if (half == 1) return;
#pragma unroll
    for (int mb = 0; mb < MB; ++mb) {
#pragma unroll
        for (int tt = 0; tt < NT; ++tt)
#pragma unroll
            for (int q = 0; q < 4; ++q) acc[mb][tt][q] += X[(mb * NT + tt) * 4 + q];
#pragma unroll
        for (int q = 0; q < 4; ++q) accb[mb][q] += X[MB * NT * 4 + mb * 4 + q];
    }
    // D[m][n] in lane n + 16 (m / 4), element m % 4
    float *P = partial + (int64_t)blockIdx.x * nent;
    const int ci = chalf * 16 + n;
#pragma unroll
    for (int mb = 0; mb < MB; ++mb)
#pragma unroll
        for (int q = 0; q < 4; ++q) {
            const int co = mb * 16 + 4 * kg + q;
            if (co >= cout) continue;
#pragma unroll
            for (int tt = 0; tt < NT; ++tt)
                if (ci < cin) P[(co * 9 + 3 * dy + tt) * cin + ci] = acc[mb][tt][q];
            if (bias_wave && n == 0) P[cout * 9 * cin + co] = accb[mb][q];
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

// Workgroups of one round, at least four rows each (a run costs two steps and
// its sums beside its rows).
template <int CIN, int COUT>
hipError_t launch_rows(const __bf16 *dz, const __bf16 *x, int cout, int cin, int B, int H, int W, float *partial,
                       int maxblocks, int nent, int *used, hipStream_t s) {
    static const int resident = [] {
        int r = 0;
        return hipOccupancyMaxActiveBlocksPerMultiprocessor(&r, k_wgrad_rows<CIN, COUT>, 64 * kRowWaves, 0) == hipSuccess && r > 0 ? r : 1;
    }();
    const int groups = W / kRowCols;
    const int64_t total = (int64_t)B * groups * H;
    if (total > (int64_t)1 << 30) return hipErrorInvalidValue;
    const int64_t most = std::min<int64_t>({(total + 3) / 4, (int64_t)sw_device_cus() * resident, (int64_t)maxblocks});
    const int per = (int)((total + most - 1) / most);
    *used = (int)((total + per - 1) / per);
    k_wgrad_rows<CIN, COUT><<<(unsigned)*used, 64 * kRowWaves, 0, s>>>(dz, x, cout, cin, H, W, groups, (int)total, per, partial, nent);
    return hipGetLastError();
}

template <int CINP, int COUTP>
hipError_t launch_wgrad(const __bf16 *dz, const __bf16 *a, int cout, int cin, int B, int H, int W, float *partial,
                        int maxblocks, int nent, int *used, hipStream_t s) {
    constexpr int threads = CINP == 32 ? 384 : 192;
    static const int resident = [] {   // blocks of this instance that fit on one CU at once
        int r = 0;
        return hipOccupancyMaxActiveBlocksPerMultiprocessor(&r, k_wgrad<CINP, COUTP>, threads, 0) == hipSuccess && r > 0
                   ? r
                   : 1;
    }();
    const int cus = sw_device_cus();
    const int tiles_y = (H + kWgRows - 1) / kWgRows, tiles_x = W / kWgCols;
    const int64_t ntiles = (int64_t)B * tiles_y * tiles_x;
    if (ntiles > (int64_t)1 << 30) return hipErrorInvalidValue;
    const int nb = (int)std::min<int64_t>({ntiles, (int64_t)cus * resident, (int64_t)maxblocks});
    k_wgrad<CINP, COUTP><<<nb, threads, 0, s>>>(dz, a, cout, cin, H, W, tiles_y, tiles_x, (int)ntiles, partial, nent);
    *used = nb;
    return hipGetLastError();
}

hipError_t launch_wgrad_dma(const __bf16 *dz, const __bf16 *a, int cout, int cin, int B, int H, int W, float *partial,
                            int maxblocks, int nent, int *used, hipStream_t s) {
    const int tiles_y = (H + kWgRows - 1) / kWgRows, tiles_x = W / kWgCols;
    const int64_t ntiles = (int64_t)B * tiles_y * tiles_x;
    if (ntiles > (int64_t)1 << 30) return hipErrorInvalidValue;
    const int nb = (int)std::min<int64_t>({ntiles, (int64_t)sw_device_cus(), (int64_t)maxblocks});   // one per CU (LDS)
    k_wgrad_dma<<<nb, 768, 0, s>>>(dz, a, cout, cin, H, W, tiles_y, tiles_x, (int)ntiles, partial, nent);
    *used = nb;
    return hipGetLastError();
}

// Rows for groups of 256 columns from 600 000 pixels on: below, a run's start
// and its sums at the end (eight waves') take longer than a tile walk.
// Measured, gradients in all, rows / tiles: 48 images of 256^2 1412 / 1487 us,
// 16 of 400x256 783 / 819, 4 of 400x256 326 / 315, one of 40x256 179 / 145.  In
// groups of 64, 128 or 192 columns rows were never faster by more than 2 %
// (40 of 400x192 1446 / 1427 us, 58 of 400x128 1353 / 1377, 110 of 400x64 1353 / 1335).
bool use_rows(int B, int H, int W) { return W % kRowCols == 0 && (int64_t)B * H * W >= 600000; }

}  // namespace

hipError_t sw_sur_wgrad(const void *dzv, int coutp, int cout, const void *av, int cinp, int cin, int B, int H, int W,
                        float *partial, int nblocks, float *grad_w, float *grad_b, hipStream_t s) {
    if (B < 1 || H < 1 || W < 64 || W % 64 != 0 || nblocks < 1 || cout > coutp || cin > cinp) return hipErrorInvalidValue;
    const int nent = cout * 9 * cin + cout;
    const __bf16 *dz = (const __bf16 *)dzv, *a = (const __bf16 *)av;
    int used = 0;
    hipError_t e = hipErrorInvalidValue;
    auto run = [&](auto rows, auto tiles) {
        e = use_rows(B, H, W) ? rows(dz, a, cout, cin, B, H, W, partial, nblocks, nent, &used, s)
                              : tiles(dz, a, cout, cin, B, H, W, partial, nblocks, nent, &used, s);
    };
    if (cinp == 32 && coutp == 32) run(launch_rows<32, 32>, launch_wgrad_dma);
    else if (cinp == 8 && coutp == 32) run(launch_rows<8, 32>, launch_wgrad<8, 32>);
    else if (cinp == 32 && coutp == 8) run(launch_rows<32, 8>, launch_wgrad<32, 8>);
    if (e != hipSuccess) return e;
    k_wgrad_reduce<<<(nent + 63) / 64, 64 * kParts, 0, s>>>(partial, used, nent, cout * 9 * cin, grad_w, grad_b);
    return hipGetLastError();
}
