// The rollout's whole network in one kernel: each workgroup takes a TH x TW
// output tile and runs all six layers on it with the activations in LDS, so
// the only HBM traffic of a jump's forward pass is the state read once (with
// a 6-pixel border) and the FP32 prediction written once.
//
// Layer l (1..6) is evaluated over the tile grown by 6 - l pixels on every
// side, so that layer l + 1 finds all its 3x3 inputs: the input region is
// (TH + 12) x (TW + 12) pixels, layer 1 writes (TH + 10) x (TW + 10), ...,
// layer 6 only the tile.  Hidden activations outside the grid are set to
// zero, which is the zero padding of the layer that reads them; the input's
// one-pixel ring outside the grid comes from the state's ghost cells (the
// boundary conditions), as in the per-layer path.  Every MFMA takes the same
// operands in the same order as the per-layer kernel (k_conv3x3): weights as
// the 16-row A operand per K step, 16 pixels as the B operand, FP32
// accumulation tap by tap, then bias, ReLU, the residual add and the BF16
// rounding in the same expression order.  The prediction is therefore
// bitwise that of the per-layer path; only the recomputed border costs
// extra (1.77x the flops at 16 x 16 tiles, 1.54x at 16 x 32).
//
// LDS regions are row-major: X (input, 8 channels, 16 B per pixel), A (layers
// 1, 3, 5) and B (layers 2, 4), 32 channels (64 B per pixel, its 16-byte
// chunks swizzled by chunk_off), with rows of a multiple of 8 pixels, so that
// the swizzle, and with it a tap's address, is the same in every row.  X and
// B share one area (X is dead once layer 1 has run).
//
// At the sizes it runs at a CU has one tile, in eight waves that barriers
// keep in step: what a layer takes is the latency of its operands and the
// vector instructions around its MFMAs.  Hence a layer's weights stay in
// registers; the waves take their pixel blocks two at a time, one pair's
// epilogue among the next one's MFMAs; the weights' rows are dealt to the
// MFMA's 16-row blocks so that a lane ends with 8 consecutive channels of a
// pixel, the ones of its operand of the middle tap, which is the residual
// block's skip; and the barriers wait for LDS alone, not for the next layer's
// weights.  Measured, the network of one grid of 256^2: 21.8 -> 20.0 us, of
// which about 13 are its layers' (their MFMAs and, as long, their operands'
// LDS reads would take 4.6); a rollout of 4 grids (16 x 32 tiles, 64 steps):
// 575 -> 513 us.  (The weights two K steps ahead and all of a wave's blocks at
// once before; a layer's weights ahead with the old order of blocks was 5 %
// slower than that.)
#include "sw_conv.h"
#include "sw_conv_dev.h"

#include <algorithm>

namespace {

constexpr int kBorder = 6;   // one pixel per 3x3 layer

template <int TH, int TW> struct Geo {
    static constexpr int h(int l) { return TH + 2 * (kBorder - l); }   // rows of layer l's region (l = 0: input)
    static constexpr int w(int l) { return TW + 2 * (kBorder - l); }
    static constexpr int s(int l) { return (w(l) + 7) / 8 * 8; }            // its row stride in LDS, pixels
    static constexpr int X_ELEMS = h(0) * s(0) * 8;
    static constexpr int A_ELEMS = h(1) * s(1) * 32;
    static constexpr int B_ELEMS = h(2) * s(2) * 32;
    // X is read only by layer 1 and B first written by layer 2: they share one area
    static constexpr int XB_ELEMS = X_ELEMS > B_ELEMS ? X_ELEMS : B_ELEMS;
};

// The A operand of M block mb, K step ks of a layer with KS K steps (forward
// layout: KS * 32 elements a row).  32 output channels: rows dealt so that
// lane (g, n) ends with channels 8 g + 4 mb .. + 3 of pixel n.
template <int KS>
__device__ __forceinline__ bf16x8 load_wk(const void *wk, int mb, int ks, int n, int g, bool out) {
    return *reinterpret_cast<const bf16x8 *>((const __bf16 *)wk + (out ? n : 8 * (n >> 2) + 4 * mb + (n & 3)) * (KS * 32) +
                                             ks * 32 + 8 * g);
}

// One layer over its region.  Wave w owns the 16-pixel blocks w, w + NW, ...
// (NB of them, the last possibly a padding block that stores nothing), two at
// a time.  wt: the layer's weights; once the last blocks' MFMAs of K step ks
// are issued, next(ks) loads what takes their place in the following layer.
// Each accumulator sums its K steps in order, as the per-layer kernel does.
// MODE 0: A = relu(Z) (first layer), 1: A = A_prev + relu(Z) (residual
// blocks), 2: FP32 Z to the prediction (output layer, channels 0..2; returns
// this lane's sum of channel 0 over the pixels it stored).  WOUT x HOUT: the
// region; SIN, SOUT: row strides of the source and destination regions.
// (gy0, gx0): grid coordinates of the region's first pixel; bias: the layer's
// biases in LDS.  at_last() issues the caller's own loads (the next tile's
// input) before the last blocks.
template <int CIN, int COUT, int MODE, int WOUT, int HOUT, int SIN, int SOUT, int NW, typename Next, typename AtLast>
__device__ __forceinline__ double run_layer(const __bf16 *src, __bf16 *dst, const bf16x8 (&wt)[9][2], Next &&next,
                                            const float *bias, int gy0, int gx0, int H, int W, float *out,
                                            int64_t out_row0, AtLast &&at_last) {
    constexpr int KS = CIN == 32 ? 9 : 3;
    constexpr int MB = (COUT + 15) / 16;
    constexpr int NPIX = WOUT * HOUT;
    constexpr int NB = ((NPIX + 15) / 16 + NW - 1) / NW;     // blocks per wave
    static_assert(CIN == 8 || SIN % 8 == 0, "a tap's swizzle must not depend on the row");
    const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int g = lane >> 4, n = lane & 15;
    float bl[8];
#pragma unroll
    for (int q = 0; q < 8; ++q) bl[q] = bias[MODE == 2 ? q & 3 : 8 * g + q];
    double dh = 0.0;
    struct Block {
        f32x4 acc[MB];
        bf16x8 skip;
        int p, r, c;
    };
    auto finish = [&](const Block &v) {
        if (v.p >= NPIX) return;
        const int gy = gy0 + v.r, gx = gx0 + v.c;
        if constexpr (MODE == 2) {
            if (g != 0 || gy >= H) return;                   // lanes of group 0 hold channels 0..3
            f32x4 o = v.acc[0];
#pragma unroll
            for (int q = 0; q < 4; ++q) o[q] = q < COUT ? o[q] + bl[q] : 0.f;
            *reinterpret_cast<f32x4 *>(out + (out_row0 + (int64_t)v.r * W + v.c) * 4) = o;
            dh += (double)o[0];
        } else {
            const bool inside = gy >= 0 && gy < H && gx >= 0 && gx < W;
            float f[8];
#pragma unroll
            for (int q = 0; q < 8; ++q) {
                f[q] = fmaxf(v.acc[q >> 2][q & 3] + bl[q], 0.f);
                if (MODE == 1) f[q] += (float)v.skip[q];
            }
            u32x4 o = __builtin_bit_cast(u32x4, to_bf16(f));
#pragma unroll
            for (int q = 0; q < 4; ++q) o[q] = inside ? o[q] : 0u;
            *reinterpret_cast<u32x4 *>(dst + chunk_off(v.r * SOUT + v.c, g)) = o;
        }
    };
    Block blk[2][2];                                         // the pair at hand and the one before
#pragma unroll
    for (int k = 0; k < NB; k += 2) {
        Block(&cur)[2] = blk[(k >> 1) & 1];
        const int m = k + 1 < NB ? 2 : 1;
        const bool last = k + 2 >= NB;
        if (last) at_last();
        const __bf16 *at[2][3];
#pragma unroll
        for (int i = 0; i < m; ++i) {
            cur[i].p = (wave + (k + i) * NW) * 16 + n;
            const int pc = min(cur[i].p, NPIX - 1);          // padding lanes read a real pixel, store nothing
            cur[i].r = pc / WOUT;
            cur[i].c = pc - cur[i].r * WOUT;
            const int sb = cur[i].r * SIN + cur[i].c;
#pragma unroll
            for (int d = 0; d < 3; ++d) {
                if (CIN == 32) {
                    at[i][d] = src + chunk_off(sb + d, g);   // column tap d of row tap 0
                } else {                                     // K step d: tap 4 d + g
                    const int tap = min(4 * d + g, 8);
                    at[i][d] = src + (sb + tap / 3 * SIN + tap % 3) * 8;
                }
            }
#pragma unroll
            for (int mb = 0; mb < MB; ++mb) cur[i].acc[mb] = f32x4{0.f, 0.f, 0.f, 0.f};
        }
#pragma unroll
        for (int ks = 0; ks < KS; ++ks) {
            bf16x8 x[2];
#pragma unroll
            for (int i = 0; i < m; ++i) {
                x[i] = *reinterpret_cast<const bf16x8 *>(CIN == 32 ? at[i][ks % 3] + ks / 3 * (SIN * 32) : at[i][ks]);
                if (CIN == 8 && ks == 2 && g != 0) x[i] = bf16x8{};   // taps 9 .. 11 do not exist
                if (MODE == 1 && ks == 4) cur[i].skip = x[i];
            }
#pragma unroll
            for (int i = 0; i < m; ++i)
#pragma unroll
                for (int mb = 0; mb < MB; ++mb) cur[i].acc[mb] = mfma(wt[ks][mb], x[i], cur[i].acc[mb]);
            if (last) next(ks);
            if (ks == KS / 3 && k > 0)
#pragma unroll
                for (int i = 0; i < 2; ++i) finish(blk[((k >> 1) & 1) ^ 1][i]);
        }
    }
#pragma unroll
    for (int i = 0; i < (NB % 2 ? 1 : 2); ++i) finish(blk[((NB - 1) >> 1) & 1][i]);
    return dh;
}

// NW waves per workgroup.
template <int TH, int TW, int NW>
__global__ __launch_bounds__(64 * NW) void k_net_fused(SwNetFusedArgs a, int tiles_y, int tiles_x, int ntiles) {
    using G = Geo<TH, TW>;
    __shared__ __attribute__((aligned(16))) __bf16 sa[G::A_ELEMS];
    __shared__ __attribute__((aligned(16))) __bf16 sxb[G::XB_ELEMS];
    __bf16 *const sx = sxb, *const sbf = sxb;   // input (layer 1 reads it), then layers 2 and 4
    __shared__ double s_dh[NW];
    __shared__ float s_bias[6][32];
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    for (int i = threadIdx.x; i < 6 * 32; i += 64 * NW) {   // the layers' biases (output layer: 3)
        const int l = i >> 5, co = i & 31;
        s_bias[l][co] = (l < 5 || co < 3) ? a.bias[l][co] : 0.f;
    }
    const int H = a.H, W = a.W;

    // the input of tile tt: raw state values of this thread's pixels of the
    // (TH + 12) x (TW + 12) region, loaded into registers ahead of use (the
    // ghost ring of the grid included; pixels further out are zero)
    constexpr int NPIN = G::h(0) * G::w(0);
    constexpr int PER = (NPIN + 64 * NW - 1) / (64 * NW);
    float rh[PER], rp[PER], rq[PER];
    unsigned ok = 0u;
    auto stage_load = [&](int tt) {
        const int b = tt / (tiles_y * tiles_x);
        const int rem = tt - b * tiles_y * tiles_x;
        const int ty = rem / tiles_x, tx = rem - ty * tiles_x;
        const SwBatchGrid &gd = a.grids[b];
        const float *P0 = (const float *)gd.plane[a.cur][0], *P1 = (const float *)gd.plane[a.cur][1],
                    *P2 = (const float *)gd.plane[a.cur][2];
        ok = 0u;
#pragma unroll
        for (int j = 0; j < PER; ++j) {
            const int i = threadIdx.x + j * 64 * NW;
            const int r = i / G::w(0), c = i - r * G::w(0);
            const int gy = ty * TH - kBorder + r, gx = tx * TW - kBorder + c;
            rh[j] = rp[j] = rq[j] = 0.f;
            if (i < NPIN && gy >= -1 && gy <= H && gx >= -1 && gx <= W) {
                const int64_t off = (int64_t)gy * gd.pitch + gx;
                rh[j] = P0[off];
                rp[j] = P1[off];
                rq[j] = P2[off];
                ok |= 1u << j;
            }
        }
    };
    auto stage_store = [&] {
#pragma unroll
        for (int j = 0; j < PER; ++j) {
            const int i = threadIdx.x + j * 64 * NW;
            if (i >= NPIN) continue;
            bf16x8 v = bf16x8{};
            if (ok >> j & 1u)
                v = bf16x8{(__bf16)((rh[j] - a.nrm.in_off[0]) / a.nrm.in_scale[0]),
                           (__bf16)((rp[j] - a.nrm.in_off[1]) / a.nrm.in_scale[1]),
                           (__bf16)((rq[j] - a.nrm.in_off[2]) / a.nrm.in_scale[2]),
                           (__bf16)0.f, (__bf16)0.f, (__bf16)0.f, (__bf16)0.f, (__bf16)0.f};
            const int r = i / G::w(0);
            *reinterpret_cast<bf16x8 *>(sx + (r * G::s(0) + i - r * G::w(0)) * 8) = v;
        }
    };
    auto nothing = [] {};
    const int lane16 = lane & 15, g4 = lane >> 4;
    // weights of the layer that runs; the first layer has only 3 K steps, the rest of the second's are loaded before it
    bf16x8 wt[9][2];
    auto load_first = [&](int ks) {
#pragma unroll
        for (int mb = 0; mb < 2; ++mb)
            if (ks < 3) wt[ks][mb] = load_wk<3>(a.wk[0], mb, ks, lane16, g4, false);
    };
    auto load_of = [&](int l) {                               // layer l's (1 .. 5)
        return [&, l](int ks) {
#pragma unroll
            for (int mb = 0; mb < 2; ++mb)
                if (l < 5 || mb == 0) wt[ks][mb] = load_wk<9>(a.wk[l], mb, ks, lane16, g4, l == 5);
        };
    };
    if (blockIdx.x < ntiles) stage_load(blockIdx.x);
#pragma unroll
    for (int ks = 0; ks < 3; ++ks) load_first(ks);

    for (int t = blockIdx.x; t < ntiles; t += gridDim.x) {   // uniform per block
        const int b = t / (tiles_y * tiles_x);
        const int rem = t - b * tiles_y * tiles_x;
        const int ty = rem / tiles_x, tx = rem - ty * tiles_x;
        const int y0 = ty * TH, x0 = tx * TW;               // tile origin in the grid
        if (a.clear_stats && ty == 0 && tx == 0 && threadIdx.x == 0) {   // the grid's first tile clears its statistics
            SwGateStats &st = a.clear_stats[b];
            st.mass_old = 0.0;
            st.mass_new = 0.0;
            st.hmin = 3.0e38f;
            st.nonfinite = 0u;
        }
        stage_store();
        lds_barrier();
#pragma unroll
        for (int ks = 3; ks < 9; ++ks) load_of(1)(ks);
        run_layer<8, 32, 0, G::w(1), G::h(1), G::s(0), G::s(1), NW>(sx, sa, wt, load_of(1), s_bias[0], y0 - 5, x0 - 5, H,
                                                        W, nullptr, 0, nothing);
        lds_barrier();
        run_layer<32, 32, 1, G::w(2), G::h(2), G::s(1), G::s(2), NW>(sa, sbf, wt, load_of(2), s_bias[1], y0 - 4, x0 - 4,
                                                         H, W, nullptr, 0, nothing);
        lds_barrier();
        run_layer<32, 32, 1, G::w(3), G::h(3), G::s(2), G::s(3), NW>(sbf, sa, wt, load_of(3), s_bias[2], y0 - 3, x0 - 3,
                                                         H, W, nullptr, 0, nothing);
        lds_barrier();
        run_layer<32, 32, 1, G::w(4), G::h(4), G::s(3), G::s(4), NW>(sa, sbf, wt, load_of(4), s_bias[3], y0 - 2, x0 - 2,
                                                         H, W, nullptr, 0, nothing);
        lds_barrier();
        run_layer<32, 32, 1, G::w(5), G::h(5), G::s(4), G::s(5), NW>(sbf, sa, wt, load_of(5), s_bias[4], y0 - 1, x0 - 1,
                                                         H, W, nullptr, 0, nothing);
        lds_barrier();
        const int tn = t + gridDim.x;
        double dh = run_layer<32, 3, 2, TW, TH, G::s(5), TW, NW>(sa, nullptr, wt, load_first, s_bias[5], y0, x0, H, W,
                                                          a.delta, ((int64_t)b * H + y0) * W + x0, [&] {
                                                              if (tn < ntiles) stage_load(tn);
                                                          });
        // the tile's sum of predicted dh in a fixed order: lanes, then waves
#pragma unroll
        for (int o = 32; o > 0; o >>= 1) dh += __shfl_xor(dh, o);
        if (lane == 0) s_dh[wave] = dh;
        lds_barrier();                                       // also: the next tile's staging may overwrite sx / sa
        if (threadIdx.x == 0 && a.dh_tile) {
            double s = 0.0;
            for (int k = 0; k < NW; ++k) s += s_dh[k];
            a.dh_tile[(int64_t)b * tiles_y * tiles_x + rem] = s;
        }
    }
}

#ifndef SW_NET_WAVES
#define SW_NET_WAVES 8
#endif
constexpr int kNetWaves = SW_NET_WAVES;

template <int TH, int TW>
hipError_t launch_net(const SwNetFusedArgs &a, hipStream_t s) {
    const int tiles_y = (a.H + TH - 1) / TH, tiles_x = a.W / TW;
    const int64_t ntiles = (int64_t)a.B * tiles_y * tiles_x;
    if (ntiles > (int64_t)1 << 30) return hipErrorInvalidValue;
    static const int resident = [] {   // workgroups that fit on one CU at once (LDS and registers)
        int r = 0;
        return hipOccupancyMaxActiveBlocksPerMultiprocessor(&r, k_net_fused<TH, TW, kNetWaves>, 64 * kNetWaves,
                                                            0) == hipSuccess &&
                       r > 0
                   ? r
                   : 1;
    }();
    int64_t blocks = std::min<int64_t>(ntiles, (int64_t)sw_device_cus() * resident);
    if (a.max_blocks > 0) blocks = std::min<int64_t>(blocks, a.max_blocks);
    k_net_fused<TH, TW, kNetWaves><<<(unsigned)blocks, 64 * kNetWaves, 0, s>>>(a, tiles_y, tiles_x, (int)ntiles);
    return hipGetLastError();
}

}  // namespace

// Tile shape: 16 x 32 when the batch has at least two such tiles per CU
// (less recomputed border), else 16 x 16 (more workgroups for small batches).
#ifndef SW_NET_WIDE
#define SW_NET_WIDE 1
#endif
void sw_net_fused_tile(int B, int H, int W, int *th, int *tw) {
    const int64_t wide = (int64_t)B * ((H + 15) / 16) * (W / 32);
    *th = 16;
    *tw = SW_NET_WIDE && wide >= 2 * (int64_t)sw_device_cus() ? 32 : 16;
}

hipError_t sw_net_fused(const SwNetFusedArgs &a, hipStream_t s) {
    if (a.B < 1 || a.H < 1 || a.W < 64 || a.W % 64 != 0 || !a.grids || a.cur < 0 || a.cur > 1 || !a.delta)
        return hipErrorInvalidValue;
    for (int l = 0; l < 6; ++l)
        if (!a.wk[l] || !a.bias[l]) return hipErrorInvalidValue;
    int th, tw;
    sw_net_fused_tile(a.B, a.H, a.W, &th, &tw);
    return tw == 32 ? launch_net<16, 32>(a, s) : launch_net<16, 16>(a, s);
}
