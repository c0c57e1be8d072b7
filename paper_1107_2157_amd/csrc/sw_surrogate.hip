// Learned-surrogate kernels other than the convolution: input preparation,
// loss and its gradient seed, Adam with the BF16 weight re-layout, and the
// gated rollout (apply, gate statistics, accept).
#include <algorithm>

#include "sw_common.h"
#include "sw_conv.h"

using namespace sw;

namespace {

typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));

__device__ __forceinline__ float wave_sum_f(float v) {
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) v += __shfl_xor(v, o);
    return v;
}
__device__ __forceinline__ double wave_sum_d(double v) {
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) v += __shfl_xor(v, o);
    return v;
}

// Source cell of halo pixel index t in [0, n + 2) along one axis (halo
// coordinates): interior t - 1, or the boundary image; *flip = -1 where the
// reflective wall negates that axis' momentum.
__device__ __forceinline__ int src_index(int t, int n, int bc, float *flip) {
    *flip = 1.f;
    if (t == 0) {
        if (bc) return n - 1;
        *flip = -1.f;
        return 0;
    }
    if (t == n + 1) {
        if (bc) return 0;
        *flip = -1.f;
        return n - 1;
    }
    return t - 1;
}

__device__ __forceinline__ void store_x0(__bf16 *x0, float a, float b, float c) {
    bf16x8 v = {(__bf16)a, (__bf16)b, (__bf16)c, (__bf16)0.f, (__bf16)0.f, (__bf16)0.f, (__bf16)0.f, (__bf16)0.f};
    *reinterpret_cast<bf16x8 *>(x0) = v;
}

__global__ __launch_bounds__(256) void k_prep_dense(const float *u, const float *u8, int B, int H, int W, int bcx,
                                                    int bcy, SwNorm nrm, __bf16 *x0, float *target) {
    const int Wp = W + 2, Hp = H + 2;
    const int64_t n = (int64_t)B * Hp * Wp;
    for (int64_t idx = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; idx < n; idx += (int64_t)gridDim.x * blockDim.x) {
        const int b = (int)(idx / ((int64_t)Hp * Wp));
        const int r = (int)(idx - (int64_t)b * Hp * Wp);
        const int yy = r / Wp, xx = r - yy * Wp;
        float fx, fy;
        const int x = src_index(xx, W, bcx, &fx), y = src_index(yy, H, bcy, &fy);
        const int64_t plane = (int64_t)H * W;
        const float *ub = u + (int64_t)b * 3 * plane + (int64_t)y * W + x;
        const float h = ub[0], hu = fx * ub[plane], hv = fy * ub[2 * plane];
        const float c0 = (h - nrm.in_off[0]) / nrm.in_scale[0], c1 = (hu - nrm.in_off[1]) / nrm.in_scale[1],
                    c2 = (hv - nrm.in_off[2]) / nrm.in_scale[2];
        store_x0(x0 + idx * 8, c0, c1, c2);
        if (target && xx >= 1 && xx <= W && yy >= 1 && yy <= H) {
            const float *vb = u8 + (int64_t)b * 3 * plane + (int64_t)y * W + x;
            float *tg = target + (((int64_t)b * H + y) * W + x) * 4;
            tg[0] = (vb[0] - ub[0]) / nrm.out_scale[0];
            tg[1] = (vb[plane] - ub[plane]) / nrm.out_scale[1];
            tg[2] = (vb[2 * plane] - ub[2 * plane]) / nrm.out_scale[2];
            tg[3] = 0.f;
        }
    }
}

__global__ __launch_bounds__(256) void k_loss(const float *pred, const float *target, int B, int H, int W,
                                              float *partial, __bf16 *dz) {
    const int64_t n = (int64_t)B * H * W;
    const float scale = 2.f / (3.f * (float)n);
    float acc = 0.f;
    for (int64_t p = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; p < n; p += (int64_t)gridDim.x * blockDim.x) {
        const float4 pr = *reinterpret_cast<const float4 *>(pred + p * 4);
        const float4 tg = *reinterpret_cast<const float4 *>(target + p * 4);
        const float d0 = pr.x - tg.x, d1 = pr.y - tg.y, d2 = pr.z - tg.z;
        acc += d0 * d0 + d1 * d1 + d2 * d2;
        const int b = (int)(p / ((int64_t)H * W));
        const int r = (int)(p - (int64_t)b * H * W);
        const int y = r / W, x = r - y * W;
        const float g0 = scale * d0, g1 = scale * d1, g2 = scale * d2;
        store_x0(dz + (((int64_t)b * (H + 2) + y + 1) * (W + 2) + x + 1) * 8, g0, g1, g2);
    }
    __shared__ float red[4];
    acc = wave_sum_f(acc);
    if ((threadIdx.x & 63) == 0) red[threadIdx.x >> 6] = acc;
    __syncthreads();
    if (threadIdx.x == 0) partial[blockIdx.x] = (red[0] + red[1] + red[2] + red[3]) / (3.f * (float)n);
}

__global__ void k_reduce_sum(const float *partial, int n, float *out) {
    double acc = 0.0;
    for (int i = threadIdx.x; i < n; i += blockDim.x) acc += partial[i];
    __shared__ double red[4];
    acc = wave_sum_d(acc);
    if ((threadIdx.x & 63) == 0) red[threadIdx.x >> 6] = acc;
    __syncthreads();
    if (threadIdx.x == 0) out[0] = (float)(red[0] + red[1] + red[2] + red[3]);
}

__global__ void k_adam(float *master, float *m, float *v, const float *grad, int64_t n, SwAdam ad) {
    const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= n) return;
    const float g = grad[i];
    const float mi = ad.beta1 * m[i] + (1.f - ad.beta1) * g;
    const float vi = ad.beta2 * v[i] + (1.f - ad.beta2) * g * g;
    m[i] = mi;
    v[i] = vi;
    master[i] -= ad.lr * (mi * ad.c1) / (sqrtf(vi * ad.c2) + ad.eps);
}

// One thread per weight of every layer: write its BF16 copies.
__global__ void k_relayout(const float *master, const SwLayerDesc *layers, int nlayers, int64_t total) {
    int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= total) return;
    int l = 0;
    while (l < nlayers) {
        const int64_t nw = (int64_t)layers[l].cout * 9 * layers[l].cin;
        if (i < nw) break;
        i -= nw;
        ++l;
    }
    if (l >= nlayers) return;
    const SwLayerDesc &L = layers[l];
    const int ci = (int)(i % L.cin), tap = (int)((i / L.cin) % 9), co = (int)(i / (9 * L.cin));
    const float w = master[L.w_off + i];
    reinterpret_cast<__bf16 *>(L.wk)[(int64_t)co * L.kp + tap * L.cinp + ci] = (__bf16)w;
    if (L.wd) reinterpret_cast<__bf16 *>(L.wd)[(int64_t)ci * L.kpd + (8 - tap) * L.cdp + co] = (__bf16)w;
}

// Per grid (blockIdx.y): U' = U + denorm(delta) (less the mean dh when
// projecting) into buffer cur ^ 1 with its ghosts, and the gate statistics.
// The mean dh comes from the output layer's per-row sums, added by every
// block in the same fixed order (so every block, and every run, gets the
// same value).
__global__ __launch_bounds__(256) void k_apply(const float *delta, const double *dh_part, int nparts,
                                               const SwBatchGrid *grids, int cur, int H, int W, SwNorm nrm, int project,
                                               int bcx, int bcy, SwGateStats *st, SwApplyPart *part,
                                               unsigned *ticket) {
    const int b = blockIdx.y;
    const SwBatchGrid &g = grids[b];
    const int64_t n = (int64_t)H * W;
    const float *U[3] = {(const float *)g.plane[cur][0], (const float *)g.plane[cur][1], (const float *)g.plane[cur][2]};
    float *O[3] = {(float *)g.plane[cur ^ 1][0], (float *)g.plane[cur ^ 1][1], (float *)g.plane[cur ^ 1][2]};
    // a thread's pixels in pairs, a pair's loads issued together (the first
    // pair's before the projection's sum, which they do not need)
    struct Px {
        float4 d;
        float h, hu, hv;
        int x, y;
        int64_t off;
        bool live;
    };
    auto fetch = [&](int64_t q, Px &v) {
        v.live = q < n;
        if (!v.live) return;
        if (n <= 0x7fffffff) {
            v.y = (int)q / W;
            v.x = (int)q - v.y * W;
        } else {
            v.y = (int)(q / W);
            v.x = (int)(q - (int64_t)v.y * W);
        }
        v.off = (int64_t)v.y * g.pitch + v.x;
        v.d = *reinterpret_cast<const float4 *>(delta + ((int64_t)b * n + q) * 4);
        v.h = U[0][v.off];
        v.hu = U[1][v.off];
        v.hv = U[2][v.off];
    };
    const int64_t stride = (int64_t)gridDim.x * blockDim.x;
    int64_t p = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    Px pa, pb;
    fetch(p, pa);
    fetch(p + stride, pb);
    float dh_mean = 0.f;
    if (project) {
        __shared__ double s_part[4];
        const double *part = dh_part + (int64_t)b * nparts;
        double acc = 0.0;
        for (int k = threadIdx.x; k < nparts; k += blockDim.x) acc += part[k];
        acc = wave_sum_d(acc);
        if ((threadIdx.x & 63) == 0) s_part[threadIdx.x >> 6] = acc;
        __syncthreads();
        dh_mean = (float)(((s_part[0] + s_part[1]) + (s_part[2] + s_part[3])) / (double)n);
    }
    double mo = 0.0, mn = 0.0;
    float hmin = 3.0e38f;
    bool bad = false;
    auto emit = [&](const Px &v) {
        U3<float> c = {v.h + (v.d.x - dh_mean) * nrm.out_scale[0], v.hu + v.d.y * nrm.out_scale[1],
                       v.hv + v.d.z * nrm.out_scale[2]};
        O[0][v.off] = c.h;
        O[1][v.off] = c.p;
        O[2][v.off] = c.q;
        if (v.x == 0 || v.x == W - 1 || v.y == 0 || v.y == H - 1) write_ghosts(O, g.pitch, W, H, bcx, bcy, v.x, v.y, c);
        mo += v.h;
        mn += c.h;
        hmin = fminf(hmin, c.h);
        bad |= !(fabsf(c.h) <= 3.0e38f) || !(fabsf(c.p) <= 3.0e38f) || !(fabsf(c.q) <= 3.0e38f);
    };
    while (pa.live) {
        emit(pa);
        if (!pb.live) break;
        emit(pb);
        p += 2 * stride;
        fetch(p, pa);
        fetch(p + stride, pb);
    }
    mo = wave_sum_d(mo);
    mn = wave_sum_d(mn);
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) hmin = fminf(hmin, __shfl_xor(hmin, o));
    const unsigned long long anybad = __ballot(bad);
    // The four waves' partial results meet in LDS; each block then publishes
    // its partials in its own slot with device-scope atomic exchanges
    // (performed where every XCD sees them) and takes a ticket; the block
    // with the last ticket sums the slots in block order and writes the
    // grid's statistics, then clears the ticket.  Per grid that is one
    // contended atomic per block, where atomics on the statistics themselves
    // (four per block, one cache line) serialised into microseconds for the
    // few grids of a small batch.
    __shared__ double s_mo[4], s_mn[4];
    __shared__ float s_hmin[4];
    __shared__ int s_bad[4];
    __shared__ int s_last;
    const int w = threadIdx.x >> 6;
    if ((threadIdx.x & 63) == 0) {
        s_mo[w] = mo;
        s_mn[w] = mn;
        s_hmin[w] = hmin;
        s_bad[w] = anybad != 0;
    }
    __syncthreads();
    const unsigned nb = gridDim.x;
    SwApplyPart *P = part + (int64_t)b * nb;
    if (threadIdx.x == 0) {
        const double bmo = (s_mo[0] + s_mo[1]) + (s_mo[2] + s_mo[3]);
        const double bmn = (s_mn[0] + s_mn[1]) + (s_mn[2] + s_mn[3]);
        const float hm = fminf(fminf(s_hmin[0], s_hmin[1]), fminf(s_hmin[2], s_hmin[3]));
        const unsigned bd = (unsigned)(s_bad[0] | s_bad[1] | s_bad[2] | s_bad[3]);
        unsigned long long r = atomicExch(&P[blockIdx.x].mo, (unsigned long long)__double_as_longlong(bmo));
        r ^= atomicExch(&P[blockIdx.x].mn, (unsigned long long)__double_as_longlong(bmn));
        r ^= atomicExch(&P[blockIdx.x].hmin_bad, ((unsigned long long)__float_as_uint(hm) << 32) | bd);
        // the exchanges have returned (so are performed) before the ticket is taken
        asm volatile("" : "+v"(r)::"memory");
        const unsigned t = atomicAdd(&ticket[b], 1u);
        s_last = t == nb - 1;
    }
    __syncthreads();
    if (!s_last) return;                              // uniform per block
    // every block's slot is published: per thread a strided run of slots in
    // block order, then the waves and the block in a fixed order
    double tmo = 0.0, tmn = 0.0;
    float thm = 3.0e38f;
    unsigned tbad = 0u;
    for (unsigned k = threadIdx.x; k < nb; k += blockDim.x) {
        tmo += __longlong_as_double((long long)atomicAdd(&P[k].mo, 0ull));
        tmn += __longlong_as_double((long long)atomicAdd(&P[k].mn, 0ull));
        const unsigned long long hb = atomicAdd(&P[k].hmin_bad, 0ull);
        thm = fminf(thm, __uint_as_float((unsigned)(hb >> 32)));
        tbad |= (unsigned)hb;
    }
    tmo = wave_sum_d(tmo);
    tmn = wave_sum_d(tmn);
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) thm = fminf(thm, __shfl_xor(thm, o));
    const unsigned long long wbad = __ballot(tbad != 0u);
    __syncthreads();                                  // the LDS slots are reused
    if ((threadIdx.x & 63) == 0) {
        s_mo[w] = tmo;
        s_mn[w] = tmn;
        s_hmin[w] = thm;
        s_bad[w] = wbad != 0ull;
    }
    __syncthreads();
    if (threadIdx.x == 0) {
        st[b].mass_old = (s_mo[0] + s_mo[1]) + (s_mo[2] + s_mo[3]);
        st[b].mass_new = (s_mn[0] + s_mn[1]) + (s_mn[2] + s_mn[3]);
        const float hm = fminf(fminf(s_hmin[0], s_hmin[1]), fminf(s_hmin[2], s_hmin[3]));
        st[b].hmin = hm > 0.f ? hm : 0.f;             // a non-positive depth is recorded as 0
        st[b].nonfinite = (unsigned)(s_bad[0] | s_bad[1] | s_bad[2] | s_bad[3]);
        atomicExch(&ticket[b], 0u);                   // ready for the next launch
    }
}

// Per grid (blockIdx.y): the gate's verdict on the jump from its statistics
// (mass drift, least depth, non-finite values; every block derives it, block
// 0 records it in active, st and fallbacks), then for a rejected grid the
// whole halo'd rectangle of buffer cur copied into cur ^ 1.
__global__ __launch_bounds__(256) void k_gate_restore(const SwBatchGrid *grids, int cur, int H, int W, SwGateStats *st,
                                                      double mass_tol, double hmin, int *active, int *fallbacks) {
    const int b = blockIdx.y;
    const double mass_old = st[b].mass_old, mass_new = st[b].mass_new;
    const double drift = fabs(mass_new - mass_old) / fabs(mass_old);
    const int reject = !(drift <= mass_tol) || !((double)st[b].hmin > hmin) || st[b].nonfinite != 0u;
    if (blockIdx.x == 0 && threadIdx.x == 0) {
        st[b].fallback = reject;
        active[b] = reject;
        if (fallbacks) fallbacks[b] += reject;
    }
    if (!reject) return;
    const SwBatchGrid &g = grids[b];
    const int64_t n = (int64_t)(H + 2) * (W + 2);
    for (int64_t p = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; p < n; p += (int64_t)gridDim.x * blockDim.x) {
        const int yy = (int)(p / (W + 2)), xx = (int)(p - (int64_t)yy * (W + 2));
        const int64_t off = (int64_t)(yy - 1) * g.pitch + (xx - 1);
#pragma unroll
        for (int k = 0; k < 3; ++k) ((float *)g.plane[cur ^ 1][k])[off] = ((const float *)g.plane[cur][k])[off];
    }
}

// Judge, before the rollout: remember every grid's time and step count and
// clear the sums.
__global__ void k_judge_begin(const SwBatchScalars *sc, int B, SwJudge *j) {
    const int b = blockIdx.x * blockDim.x + threadIdx.x;
    if (b >= B) return;
    j[b].d2 = 0.0;
    j[b].r2 = 0.0;
    j[b].t0 = sc[b].t;
    j[b].steps0 = sc[b].steps;
}

// Per grid (blockIdx.y): sums of (h - h_ref)^2 and h_ref^2 over the interior.
__global__ __launch_bounds__(256) void k_judge_sums(const SwBatchGrid *ga, int cur_a, const SwBatchGrid *gr,
                                                    int cur_r, int H, int W, SwJudge *j) {
    const int b = blockIdx.y;
    const float *A = (const float *)ga[b].plane[cur_a][0];
    const float *R = (const float *)gr[b].plane[cur_r][0];
    const int64_t pa = ga[b].pitch, pr = gr[b].pitch, n = (int64_t)H * W;
    double d2 = 0.0, r2 = 0.0;
    for (int64_t p = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; p < n; p += (int64_t)gridDim.x * blockDim.x) {
        const int y = (int)(p / W), x = (int)(p - (int64_t)y * W);
        const double r = R[y * pr + x], d = (double)A[y * pa + x] - r;
        d2 += d * d;
        r2 += r * r;
    }
    d2 = wave_sum_d(d2);
    r2 = wave_sum_d(r2);
    if ((threadIdx.x & 63) == 0) {
        atomicAdd(&j[b].d2, d2);
        atomicAdd(&j[b].r2, r2);
    }
}

__global__ void k_judge_decide(SwJudge *j, int B, SwBatchScalars *sc, const SwBatchScalars *rsc, double l2_tol,
                               int jumps, int *reject, int *fallbacks, double *l2) {
    const int b = blockIdx.x * blockDim.x + threadIdx.x;
    if (b >= B) return;
    const double e = sqrt(j[b].d2 / j[b].r2);
    const int rej = !(e <= l2_tol);
    reject[b] = rej;
    if (l2) l2[b] = e;
    if (rej) {
        if (fallbacks) fallbacks[b] = jumps;
        sc[b].t = j[b].t0 + rsc[b].t;
        sc[b].last_dt = rsc[b].last_dt;
        sc[b].steps = j[b].steps0 + rsc[b].steps;
        sc[b].unstable = rsc[b].unstable;   // the rollout's history is discarded
    }
}

// Rejected grids: copy the solver's halo'd rectangle (buffer cur) over the rollout's.
__global__ __launch_bounds__(256) void k_judge_copy(const SwBatchGrid *ga, int cur_a, const SwBatchGrid *gr,
                                                    int cur_r, int H, int W, const int *reject) {
    const int b = blockIdx.y;
    if (!reject[b]) return;
    const int64_t n = (int64_t)(H + 2) * (W + 2);
    for (int64_t p = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; p < n; p += (int64_t)gridDim.x * blockDim.x) {
        const int yy = (int)(p / (W + 2)), xx = (int)(p - (int64_t)yy * (W + 2));
        const int64_t oa = (int64_t)(yy - 1) * ga[b].pitch + (xx - 1), orr = (int64_t)(yy - 1) * gr[b].pitch + (xx - 1);
#pragma unroll
        for (int k = 0; k < 3; ++k) ((float *)ga[b].plane[cur_a][k])[oa] = ((const float *)gr[b].plane[cur_r][k])[orr];
    }
}

unsigned grid_for(int64_t n, int cap = 16384) {
    int64_t b = (n + 255) / 256;
    if (b > cap) b = cap;
    if (b < 1) b = 1;
    return (unsigned)b;
}

}  // namespace

hipError_t sw_sur_prep_dense(const float *u, const float *u8, int B, int H, int W, int bc_x, int bc_y, SwNorm nrm,
                             void *x0, float *target, hipStream_t s) {
    k_prep_dense<<<grid_for((int64_t)B * (H + 2) * (W + 2)), 256, 0, s>>>(u, u8, B, H, W, bc_x, bc_y, nrm,
                                                                           (__bf16 *)x0, u8 ? target : nullptr);
    return hipGetLastError();
}


hipError_t sw_sur_loss(const float *pred, const float *target, int B, int H, int W, float *partial, int nblocks,
                       void *dz, hipStream_t s) {
    k_loss<<<nblocks, 256, 0, s>>>(pred, target, B, H, W, partial, (__bf16 *)dz);
    return hipGetLastError();
}

hipError_t sw_sur_reduce_sum(const float *partial, int n, float *out, hipStream_t s) {
    k_reduce_sum<<<1, 256, 0, s>>>(partial, n, out);
    return hipGetLastError();
}

hipError_t sw_sur_adam(float *master, float *m, float *v, const float *grad, int64_t n, SwAdam ad, hipStream_t s) {
    k_adam<<<(unsigned)((n + 255) / 256), 256, 0, s>>>(master, m, v, grad, n, ad);
    return hipGetLastError();
}

hipError_t sw_sur_relayout(const float *master, const SwLayerDesc *layers, int nlayers, int64_t total_weights,
                           hipStream_t s) {
    k_relayout<<<(unsigned)((total_weights + 255) / 256), 256, 0, s>>>(master, layers, nlayers, total_weights);
    return hipGetLastError();
}

// Blocks per grid of the per-grid passes: up to one element per thread for
// small batches (their few grids would otherwise leave most CUs idle and
// walk the pixels serially), 64 per grid from 256 grids up.
unsigned per_grid_blocks(int64_t n, int B) {
    const int cap = B >= 256 ? 64 : std::max(64, 16384 / std::max(B, 1));
    return grid_for(n, cap);
}


unsigned sw_sur_apply_slots(int64_t pixels, int B) { return per_grid_blocks(pixels, 1) * (unsigned)B; }

hipError_t sw_sur_apply(const float *delta, const double *dh_part, int nparts, const SwBatchGrid *grids, int cur,
                        int B, int H, int W, SwNorm nrm, int project, int bcx, int bcy, SwGateStats *st,
                        SwApplyPart *part, unsigned *ticket, hipStream_t s) {
    if (project && (!dh_part || nparts < 1)) return hipErrorInvalidValue;
    if (!part || !ticket) return hipErrorInvalidValue;
    // at most 128 blocks per grid (two pixels per thread on a 256^2 grid), and
    // few more than two per CU in all: a block's three exchanges and its
    // ticket, performed in memory, take longer than its pixels (32 grids of
    // 256^2, a 64-step rollout: 128 blocks per grid 2235 us, 64 2090, 32 1982,
    // 16 1960; 64 grids 3927 with 128, 3592 with 32, 3620 with 8)
    const unsigned most = std::max(8u, std::min(128u, 512u / (unsigned)B));
    dim3 grid(std::min(per_grid_blocks((int64_t)H * W, B), most), B);
    k_apply<<<grid, 256, 0, s>>>(delta, dh_part, nparts, grids, cur, H, W, nrm, project, bcx, bcy, st, part, ticket);
    return hipGetLastError();
}

hipError_t sw_sur_gate_restore(const SwBatchGrid *grids, int cur, int B, int H, int W, SwGateStats *st,
                               double mass_tol, double hmin, int *active, int *fallbacks, hipStream_t s) {
    dim3 grid(per_grid_blocks((int64_t)(H + 2) * (W + 2), B), B);
    k_gate_restore<<<grid, 256, 0, s>>>(grids, cur, H, W, st, mass_tol, hmin, active, fallbacks);
    return hipGetLastError();
}

hipError_t sw_sur_judge_begin(const SwBatchScalars *sc, int B, SwJudge *j, hipStream_t s) {
    k_judge_begin<<<(B + 255) / 256, 256, 0, s>>>(sc, B, j);
    return hipGetLastError();
}

hipError_t sw_sur_judge(const SwBatchGrid *a, int cur_a, const SwBatchGrid *ref, int cur_ref, int B, int H, int W,
                        SwJudge *j, SwBatchScalars *sc, const SwBatchScalars *ref_sc, double l2_tol, int jumps,
                        int *reject, int *fallbacks, double *l2, hipStream_t s) {
    k_judge_sums<<<dim3(grid_for((int64_t)H * W, 64), B), 256, 0, s>>>(a, cur_a, ref, cur_ref, H, W, j);
    hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
    k_judge_decide<<<(B + 255) / 256, 256, 0, s>>>(j, B, sc, ref_sc, l2_tol, jumps, reject, fallbacks, l2);
    if ((e = hipGetLastError()) != hipSuccess) return e;
    k_judge_copy<<<dim3(grid_for((int64_t)(H + 2) * (W + 2), 64), B), 256, 0, s>>>(a, cur_a, ref, cur_ref, H, W, reject);
    return hipGetLastError();
}
