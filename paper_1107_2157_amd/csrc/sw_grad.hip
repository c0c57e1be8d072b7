// Two consecutive layers of the surrogate's input gradient in one launch, as
// sw_pair.hip runs two layers forward (gfx950, v_mfma_f32_16x16x32_bf16):
//     Ga = conv(x) + add,  za = Ga where ma,  Gb = conv(za) + Ga,  zb = Gb where mb
// with add the gradient at the upper layer's output, and x its masked part.
//
// A layer at a time a pixel costs 320 bytes of memory traffic (x, add and a
// 64-byte mask in, G and z out); here Ga never leaves the chip, the masks are
// a bit per value, and a pair costs 328 bytes (264 where Gb is not wanted).
// Half of a workgroup's waves (role a) compute the upper layer's rows, half
// (role b) the lower's, a step behind, on a run of rows of one image as wide
// as the image.  x's rows and the masks come in by LDS DMA, which role b
// issues alone: role a reads `add` a step ahead into registers with ordinary
// loads, whose waits the compiler counts, and it does not see DMA
// instructions (issued by the same wave they would be waited for too).
// za goes to role b through two rows of LDS, Ga, which is added two steps
// later, through three.  At the ends of a run role a computes one row more.
// The accumulators sum their taps in the order of the single-layer kernel and
// every value is rounded where it rounds: all results are bitwise its own.
// Measured at 32 images of 256^2: 143 us a pair, 111 without Gb (4.8 and 5.0
// TB/s: memory), against 320 for its two layers singly, whose masks then
// were 64 bytes a pixel (the gradients of 48 images in all 2.23 -> 1.54 ms).
#include "sw_conv.h"
#include "sw_conv_dev.h"
#include "sw_dma.h"

#include <type_traits>

namespace {

template <int G, bool GB>
__global__ __launch_bounds__(128 * G, 2) void k_grad_pair(SwGradPairArgs a, int rows, int nseg) {
    constexpr int W = 64 * G, PX = W + 2;
    // rows brought in ahead of the one being read (at 128 columns two, with which two workgroups fit on a CU)
    constexpr int kAhead = G == 2 ? 2 : 3, kRing = kAhead + 1;
    constexpr int SLOTS = PX * 4;                            // 16-byte slots of a row
    constexpr int NX = (SLOTS + 63) / 64, NI = NX + 2;       // DMA instructions: of a row, of a step (with the masks')
    constexpr int PERW = (NI + G - 1) / G;                   // per wave of role b
    constexpr int IN_ROW = NX * 64 * 8;                      // BF16 elements (padded to whole instructions)
    __shared__ __attribute__((aligned(16))) __bf16 in[kRing][IN_ROW];
    __shared__ __attribute__((aligned(16))) __bf16 zmid[2][PX * 32];
    __shared__ __attribute__((aligned(16))) __bf16 gmid[3][W * 32];
    __shared__ __attribute__((aligned(16))) unsigned mask[kRing][2][256];   // of role a's and role b's row

    const int lane = threadIdx.x & 63, w = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int g = lane >> 4, n = lane & 15;
    const int role = w / G, grp = w - role * G;
    const int img = blockIdx.x / nseg, seg = blockIdx.x - img * nseg;
    const int H = a.H;
    const int ys = seg * rows, ye = min(ys + rows, H);
    if (ys >= ye) return;                                     // uniform per workgroup
    const int nsteps = ye - ys + 5;
    const int64_t img_row = (int64_t)img * (H + 2);           // first halo row of the image in a tensor

    // the halo columns of za are zero
    if (threadIdx.x < 16) {
        const int r = threadIdx.x >> 3, e = threadIdx.x & 7;
        *reinterpret_cast<bf16x8 *>(&zmid[r][chunk_off(e < 4 ? 0 : PX - 1, e & 3)]) = bf16x8{};
    }
    int off[3];                                               // chunk g of pixel grp * 64 + n + dx (+ 16 per block)
#pragma unroll
    for (int dx = 0; dx < 3; ++dx) off[dx] = chunk_off(grp * 64 + n + dx, g);
    const int px0 = grp * 64 + n, goff = chunk_off(px0, g);

    bf16x8 wt[9][2];
    const __bf16 *const wsrc = (const __bf16 *)(role == 0 ? a.wa : a.wb);
#pragma unroll
    for (int ks = 0; ks < 9; ++ks)
#pragma unroll
        for (int mb = 0; mb < 2; ++mb)
            wt[ks][mb] = *reinterpret_cast<const bf16x8 *>(wsrc + (8 * (n >> 2) + 4 * mb + (n & 3)) * 288 + ks * 32 + 8 * g);
    f32x4 acc[3][2][4];
#pragma unroll
    for (int r = 0; r < 3; ++r)
#pragma unroll
        for (int mb = 0; mb < 2; ++mb)
#pragma unroll
            for (int pb = 0; pb < 4; ++pb) acc[r][mb][pb] = f32x4{0.f, 0.f, 0.f, 0.f};

    if (role == 0) {
        // ---- role a: reads row ys - 2 + s of x, finishes row r = ys - 3 + s
        bf16x8 add[4];
        auto add_row = [&](int s) {
            const int m = min(max(ys - 2 + s, 0), H + 1);     // tensor row of r; rows outside the image are not used
            return (const __bf16 *)a.add + (img_row + m) * PX * 32 + (px0 + 1) * 32 + 8 * g;
        };
        {
            const __bf16 *p = add_row(0);
#pragma unroll
            for (int pb = 0; pb < 4; ++pb) add[pb] = *reinterpret_cast<const bf16x8 *>(p + pb * 512);
        }
        lds_barrier();
        auto step = [&](auto phase, int s) {
            constexpr int P = decltype(phase)::value, NXT = (P + 1) % 3, MID = P, FIN = (P + 2) % 3;
            const int r = ys - 3 + s;
            const bool inside = r >= 0 && r < H, keep = r >= ys && r < ye;   // else zero; else not stored
            const rsrc_t rz = row_rsrc((char *)a.za + ((img_row + r + 1) * PX + 1) * 64, keep, W * 64);
            const unsigned m = mask[s % kRing][0][grp * 64 + lane];
            const __bf16 *next = add_row(s + 1);
            conv_row<2, NXT, MID, FIN>(in[s % kRing], off, wt, acc, [&](int pb) {
                float v[8];
#pragma unroll
                for (int q = 0; q < 4; ++q) {
                    v[q] = acc[FIN][0][pb][q] + (float)add[pb][q];
                    v[4 + q] = acc[FIN][1][pb][q] + (float)add[pb][4 + q];
                }
                add[pb] = *reinterpret_cast<const bf16x8 *>(next + pb * 512);
                const bf16x8 ga = to_bf16(v);
                *reinterpret_cast<bf16x8 *>(&gmid[P][goff + pb * 512]) = ga;
                u32x4 z = mask_keep(__builtin_bit_cast(u32x4, ga), m, pb);
#pragma unroll
                for (int q = 0; q < 4; ++q) z[q] = inside ? z[q] : 0u;
                *reinterpret_cast<u32x4 *>(&zmid[s & 1][off[1] + pb * 512]) = z;
                store_row(rz, px0 * 64 + g * 16 + pb * 1024, z);
            });
            lds_barrier();
        };
        // (what the last step would compute, nobody reads)
        for (int s = 0; s < nsteps - 1; s += 3) {
            step(std::integral_constant<int, 0>{}, s);
            if (s + 1 < nsteps - 1) step(std::integral_constant<int, 1>{}, s + 1);
            if (s + 2 < nsteps - 1) step(std::integral_constant<int, 2>{}, s + 2);
        }
        lds_barrier();
        return;
    }
    // ---- role b: reads row ys - 4 + s of za, finishes row o = ys - 5 + s
    // DMA of step s's row of x and masks into ring slot s % kRing; every wave issues the same number of
    // instructions i = grp + G k, so that the waits are constants (past the last it repeats one; lanes past a
    // row's end bring a slot of it into the padding again)
    unsigned soff[PERW], ldst[PERW];
    int kind[PERW];                                           // 0 x, 1 / 2 mask of role a's / role b's row
#pragma unroll
    for (int k = 0; k < PERW; ++k) {
        const int i = (grp + G * k) % NI;
        kind[k] = i < NX ? 0 : i - NX + 1;
        int sl = i * 64 + lane;
        if (sl >= SLOTS) sl = lane;
        const int p = sl >> 2, c = (sl & 3) ^ ((p >> 1) & 3);
        soff[k] = (unsigned)(kind[k] ? lane % (16 * G) * 16 : p * 64 + c * 16);
        ldst[k] = kind[k] ? lds_addr(&mask[0][kind[k] - 1][0]) : lds_addr(&in[0][0]) + (unsigned)(i * 1024);
    }
    auto issue = [&](int s) {
        const int m = min(max(ys - 1 + s, 0), H + 1);         // tensor row (the image's row + 1); rows outside feed nothing
        const int ra = min(max(ys - 3 + s, 0), H - 1), rb = min(max(ys - 5 + s, 0), H - 1);
        const char *const xr = (const char *)a.x + (img_row + m) * PX * 64;
        const char *const mra = (const char *)a.ma + ((int64_t)img * H + ra) * W * 4;
        const char *const mrb = (const char *)a.mb + ((int64_t)img * H + rb) * W * 4;
        const unsigned slot = (unsigned)(s % kRing);
#pragma unroll
        for (int k = 0; k < PERW; ++k)
            lds_dma16(kind[k] == 0 ? xr : kind[k] == 1 ? mra : mrb, soff[k],
                      ldst[k] + slot * (unsigned)(kind[k] ? sizeof(mask[0]) : sizeof(in[0])));
    };
    // End of step s: step s + 1's row and masks are in.  They were issued at the start of step s + 1 - kAhead; newer are
    // those issued since and the stores of kAhead steps (ST a step from step 3 on; vector memory operations end in
    // order).  The first were waited for before the first step; rows past the last are issued all the same.
    auto land = [&](auto st, int s) {
        constexpr int ST = decltype(st)::value;
        if (s >= kAhead + 2) asm volatile("s_waitcnt vmcnt(%0)" ::"n"((kAhead - 1) * PERW + kAhead * ST) : "memory");
        else if (s >= kAhead - 1) asm volatile("s_waitcnt vmcnt(%0)" ::"n"((kAhead - 1) * PERW) : "memory");
        lds_barrier();
    };
    for (int s = 0; s < kAhead; ++s) issue(s);
    wait_vm_upto<0>(0);
    lds_barrier();
    auto step = [&](auto phase, int s) {
        constexpr int P = decltype(phase)::value, NXT = (P + 1) % 3, MID = P, FIN = (P + 2) % 3;
        const int o = ys - 5 + s;
        issue(s + kAhead);
        const bool keep = o >= ys;                            // (o < ye: nsteps ends there)
        const int64_t row = ((img_row + o + 1) * PX + 1) * 64;
        const rsrc_t rz = row_rsrc((char *)a.zb + row, keep, W * 64);
        const rsrc_t ry = row_rsrc((char *)a.yb + (GB ? row : 0), GB && keep, W * 64);
        const unsigned m = mask[s % kRing][1][grp * 64 + lane];
        conv_row<2, NXT, MID, FIN>(zmid[(s + 1) & 1], off, wt, acc, [&](int pb) {
            const bf16x8 ga = *reinterpret_cast<const bf16x8 *>(&gmid[(P + 1) % 3][goff + pb * 512]);   // written two steps ago
            float v[8];
#pragma unroll
            for (int q = 0; q < 4; ++q) {
                v[q] = acc[FIN][0][pb][q] + (float)ga[q];
                v[4 + q] = acc[FIN][1][pb][q] + (float)ga[4 + q];
            }
            const u32x4 gb = __builtin_bit_cast(u32x4, to_bf16(v));
            if (GB) store_row(ry, px0 * 64 + g * 16 + pb * 1024, gb);
            store_row(rz, px0 * 64 + g * 16 + pb * 1024, mask_keep(gb, m, pb));
        });
        land(std::integral_constant<int, GB ? 8 : 4>{}, s);
    };
    // (role a's first row of use is there in step 3)
    for (int s = 0; s < 3; ++s) {
        issue(s + kAhead);
        land(std::integral_constant<int, 0>{}, s);
    }
    for (int s = 3; s < nsteps; s += 3) {
        step(std::integral_constant<int, 0>{}, s);
        if (s + 1 < nsteps) step(std::integral_constant<int, 1>{}, s + 1);
        if (s + 2 < nsteps) step(std::integral_constant<int, 2>{}, s + 2);
    }
    wait_vm_upto<0>(0);                                       // no DMA into this workgroup's LDS outlives it
}

template <int G, bool GB> hipError_t launch(const SwGradPairArgs &a, hipStream_t s) {
    static const int resident = [] {
        int r = 0;
        return hipOccupancyMaxActiveBlocksPerMultiprocessor(&r, k_grad_pair<G, GB>, 128 * G, 0) == hipSuccess && r > 0 ? r : 1;
    }();
    int nseg;
    const int rows = conv_run_rows(a.B, a.H, (int64_t)sw_device_cus() * resident, 5, &nseg);
    k_grad_pair<G, GB><<<(unsigned)((int64_t)a.B * nseg), 128 * G, 0, s>>>(a, rows, nseg);
    return hipGetLastError();
}

template <bool GB> hipError_t launch_w(const SwGradPairArgs &a, hipStream_t s) {
    switch (a.W) {
        case 64: return launch<1, GB>(a, s);
        case 128: return launch<2, GB>(a, s);
        case 192: return launch<3, GB>(a, s);
        case 256: return launch<4, GB>(a, s);
    }
    return hipErrorInvalidValue;
}

}  // namespace

hipError_t sw_grad_pair(const SwGradPairArgs &a, hipStream_t s) {
    if (a.B < 1 || !sw_conv_pair_fits(a.H, a.W) || (int64_t)a.B * a.H > (int64_t)1 << 30 || !a.x || !a.add || !a.wa || !a.wb ||
        !a.ma || !a.mb || !a.za || !a.zb)
        return hipErrorInvalidValue;
    return a.yb ? launch_w<true>(a, s) : launch_w<false>(a, s);
}
