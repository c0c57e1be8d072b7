// Device code that the surrogate's convolution kernels share (included by
// .hip sources only): the LDS layout of 32-channel pixels, the backward
// masks, and the step of the kernels that march down an image.
#pragma once
#include <hip/hip_runtime.h>

#include <algorithm>
#include <cstdint>

namespace {

typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef float f32x4 __attribute__((ext_vector_type(4)));
typedef unsigned int u32x4 __attribute__((ext_vector_type(4)));
typedef __amdgpu_buffer_rsrc_t rsrc_t;

// Offset (BF16 elements) of 16-byte chunk c (channels 8c .. 8c + 7) of pixel
// p in an LDS area of 32-channel pixels.  The chunk index is XORed with bits
// 1-2 of the pixel index.  A ds_read_b128 is served 8 lanes (128 bytes, 32
// banks) at a time, and 8 lanes of an MFMA operand read the same chunk of 8
// consecutive pixels: at a plain 64-byte pixel stride those fall on 2 of the
// 8 bank quads, a 4-way conflict (measured: about 70 % of the convolutions'
// LDS cycles were bank-conflict cycles); swizzled they cover all 8.
__device__ __forceinline__ int chunk_off(int p, int c) { return p * 32 + ((c ^ ((p >> 1) & 3)) << 3); }

// The backward pass needs of a ReLU only where it is positive: one bit per
// value, a word per lane for 64 pixels of a row: word 16 c + n of the row's
// 64 pixels covers chunk c of pixels n, n + 16, n + 32, n + 48 (4 KB per 1024
// pixels, where the 32 channels in BF16 are 64 KB).  mask_push appends the
// next of a lane's four chunks (in order); mask_keep returns chunk pb of
// `v` with the values whose bit is clear set to zero.
__device__ __forceinline__ unsigned mask_push(unsigned m, u32x4 relu) {
#pragma unroll
    for (int q = 0; q < 4; ++q) m = (m >> 1) | (((relu[q] | 0x80008000u) - 0x00010001u) & 0x80008000u);
    return m;
}
__device__ __forceinline__ u32x4 mask_keep(u32x4 v, unsigned m, int pb) {
#pragma unroll
    for (int q = 0; q < 4; ++q) v[q] &= __umul24((m >> (4 * pb + q)) & 0x00010001u, 0xffffu);
    return v;
}

__device__ __forceinline__ f32x4 mfma(bf16x8 w, bf16x8 x, f32x4 c) {
    return __builtin_amdgcn_mfma_f32_16x16x32_bf16(w, x, c, 0, 0, 0);
}

__device__ __forceinline__ bf16x8 to_bf16(const float v[8]) {
    return bf16x8{(__bf16)v[0], (__bf16)v[1], (__bf16)v[2], (__bf16)v[3], (__bf16)v[4], (__bf16)v[5], (__bf16)v[6], (__bf16)v[7]};
}

// 16 bytes (or a word) at byte offset `at` of the row r; dropped outside it
// (a row that is not to be stored has length 0, so that a step has no branch
// around its stores).  Non-temporal: GB-sized tensors.
__device__ __forceinline__ rsrc_t row_rsrc(void *row, bool keep, int bytes) {
    return __builtin_amdgcn_make_buffer_rsrc(row, (short)0, keep ? bytes : 0, 0x00020000);
}
template <typename V> __device__ __forceinline__ void store_row(rsrc_t r, int at, const V &v) {
    __builtin_amdgcn_raw_buffer_store_b128(__builtin_bit_cast(u32x4, v), r, at, 0, 2);
}
__device__ __forceinline__ void store_word(rsrc_t r, int at, unsigned v) {
    __builtin_amdgcn_raw_buffer_store_b32(v, r, at, 0, 2);
}

__device__ __forceinline__ void lds_barrier() { asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory"); }

// One step of a 32-channel layer: the new row T (LDS) into the accumulators
// of the rows below (first contribution), beside and above it, a block of 16
// pixels at a time.  done(pb) is called once block pb's last row is complete
// and the next block's MFMAs are underway: its vector instructions fill the
// matrix core's 16 cycles per MFMA (done after all MFMAs, both waves of a
// SIMD, in step by the barrier, left the matrix cores idle meanwhile).
template <int MB, int NXT, int MID, int FIN, typename Done>
__device__ __forceinline__ void conv_row(const __bf16 *T, const int off[3], const bf16x8 (&wt)[9][MB],
                                         f32x4 (&acc)[3][MB][4], Done &&done) {
#pragma unroll
    for (int pb = 0; pb < 4; ++pb) {
#pragma unroll
        for (int dx = 0; dx < 3; ++dx) {
            const bf16x8 xb = *reinterpret_cast<const bf16x8 *>(T + off[dx] + pb * 512);
#pragma unroll
            for (int mb = 0; mb < MB; ++mb)
                acc[FIN][mb][pb] = mfma(wt[6 + dx][mb], xb, acc[FIN][mb][pb]);
#pragma unroll
            for (int mb = 0; mb < MB; ++mb) {
                acc[NXT][mb][pb] = mfma(wt[dx][mb], xb, dx == 0 ? f32x4{0.f, 0.f, 0.f, 0.f} : acc[NXT][mb][pb]);
                acc[MID][mb][pb] = mfma(wt[3 + dx][mb], xb, acc[MID][mb][pb]);
            }
        }
        if (pb > 0) done(pb - 1);
    }
    done(3);
}

}  // namespace

// Rows per run of a kernel that gives each workgroup a run of rows of one of
// B images of H rows (`slots` workgroups at a time, `extra` steps beside a
// run's rows): the runs, at least four rows each, that take the fewest steps.
// *nseg: runs per image; *trials (may be null): run lengths looked at.  For
// each number of rounds the shortest runs that need no more are the best, and
// a number of rounds costs `extra` steps each beside the rows themselves: the
// search ends where that alone exceeds the best (a few dozen lengths, where
// trying all down to four rows took milliseconds a launch for tall images).
inline int conv_run_rows(int B, int H, int64_t slots, int extra, int *nseg, int *trials = nullptr) {
    const int most = std::max(1, (H + 3) / 4);                // runs per image
    int best = H, n = 0;
    *nseg = 1;
    int64_t best_cost = -1;
    for (int64_t rounds = (B + slots - 1) / slots;; ++rounds) {
        if (best_cost >= 0 && rounds * extra + (int64_t)B * H / slots >= best_cost) break;
        const int64_t k = std::min<int64_t>(rounds * slots / B, most);
        const int rows = (int)((H + k - 1) / k), segs = (H + rows - 1) / rows;
        const int64_t cost = ((int64_t)B * segs + slots - 1) / slots * (rows + extra);
        ++n;
        if (best_cost < 0 || cost < best_cost) {
            best_cost = cost;
            best = rows;
            *nseg = segs;
        }
        if (k == most) break;
    }
    if (trials) *trials = n;
    return best;
}
