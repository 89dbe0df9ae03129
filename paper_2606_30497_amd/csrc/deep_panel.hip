// deep_panel.hip -- the L-hidden-layer path for nets up to 256 units wide, a few
// launches a step however deep the net (the sequence of GEMM launches in deep.hip
// serves wider nets; the step's equations are stated there).
//
// A panel of 16, 32 or 64 batch rows needs no other rows for its forward pass, its
// output and its back-propagation down to G_1, and its activations fit in LDS. So
// one workgroup takes a panel through all of it (k_panel), streaming every layer's
// weights from L2:
//   - the weights come split into three bf16 parts (bf16x3.h), in the order the
//     matrix cores take them (one 16-byte load per lane, part and 16 x 32 block; no
//     conversion, no LDS), written once per step by the update kernel;
//   - a product computes Z^T: the weights are the MFMA's A operand, the
//     activations its B operand, so a lane holds four consecutive units of one row,
//     which it splits and stores to LDS as 8-byte words in the layout the next
//     layer's B operand reads;
//   - the activations H_l and gradients G_l go to memory once, in fp32, for
// k_panel_wgrad, which forms every dW_l = H_{l-1}^T G_l (64 x 64 tiles, row chunks;
// each wave loads 64 units of 32 rows of either operand as 16-byte loads along the
// units and splits them in registers), and k_panel_apply, which sums the chunk
// partials, applies eq. 19, splits the new weights for the next step and gathers
// its rows.
// Every sum runs in a fixed order: results are bitwise reproducible.
#include <hip/hip_runtime.h>

#include <stdint.h>
#include <string.h>

#include "bf16x3.h"
#include "deep_internal.h"
#include "lanes.h"
#include "mlp.h"
#include "mlp_internal.h"

namespace mlp {

typedef __amdgpu_buffer_rsrc_t rsrc_t;

// ---- split weights -----------------------------------------------------------
// 16-byte words: block (x tile of 16, k block of 32) of a matrix holds, per part,
// lane (li, lq)'s eight values k = 8 lq .. 8 lq + 7 of row x = li:
//   word ((xt * nkb + kb) * 3 + part) * 64 + lane.
// Forward operand of W_l: x = output unit, k = input; backward: x = input unit,
// k = output unit. Order: forward W_1, forward W_2 .. W_L, backward W_2 .. W_L.
__host__ __device__ inline int64_t frag_w1(int h) { return 12 * (int64_t)h; }
__host__ __device__ inline int64_t frag_wl(int h) { return (int64_t)h * h * 3 / 8; }
__host__ __device__ inline int64_t frag_fwd(int h, int l) {
    return l == 1 ? 0 : frag_w1(h) + (l - 2) * frag_wl(h);
}
__host__ __device__ inline int64_t frag_bwd(int h, int L, int l) {
    return frag_w1(h) + (L - 1 + l - 2) * frag_wl(h);
}

// Weight tiles of 8 inputs x 64 units: W_1's, then each W_l's.
__host__ __device__ inline int weight_tiles(int h, int L) {
    return (D_IN / 8) * (h / 64) + (L - 1) * (h / 8) * (h / 64);
}
struct WeightTile {
    int l, i0, j0;
};
__device__ __forceinline__ WeightTile weight_tile(int t, int h) {
    const int nj = h / 64, n1 = (D_IN / 8) * nj, nl = (h / 8) * nj;
    WeightTile w;
    w.l = t < n1 ? 1 : 2 + (t - n1) / nl;
    if (t >= n1) t = (t - n1) % nl;
    w.i0 = 8 * (t / nj);
    w.j0 = 64 * (t % nj);
    return w;
}

constexpr int WT_S = 68;   // LDS row stride of a weight tile (floats)

// The split words of a weight tile in LDS: wave 0 the forward operand's (a lane's
// eight inputs of one unit), wave 1 the backward operand's (eight units of one input).
__device__ __forceinline__ void write_frags(const float *tl, const WeightTile &w, int h, int L,
                                            u4v *__restrict__ frag) {
    const int tid = threadIdx.x;
    float v[8];
    int64_t at;
    if (tid < 64) {
        const int j = w.j0 + tid, nkb = w.l == 1 ? 1 : h / 32;
#pragma unroll
        for (int t = 0; t < 8; ++t) v[t] = tl[t * WT_S + tid];
        at = frag_fwd(h, w.l) + ((int64_t)(j / 16) * nkb + w.i0 / 32) * 192 + ((w.i0 % 32) / 8) * 16 + j % 16;
    } else if (tid < 128 && w.l > 1) {
        const int i = tid & 7, jb = (tid - 64) >> 3, j = w.j0 + 8 * jb;
#pragma unroll
        for (int t = 0; t < 8; ++t) v[t] = tl[i * WT_S + 8 * jb + t];
        at = frag_bwd(h, L, w.l) + ((int64_t)((w.i0 + i) / 16) * (h / 32) + j / 32) * 192 +
             ((j % 32) / 8) * 16 + (w.i0 + i) % 16;
    } else {
        return;
    }
    uint32_t q[4][3];
#pragma unroll
    for (int t = 0; t < 4; ++t) split_pair(v[2 * t], v[2 * t + 1], q[t]);
#pragma unroll
    for (int p = 0; p < 3; ++p) frag[at + 64 * p] = u4v{q[0][p], q[1][p], q[2][p], q[3][p]};
}

// Before a call's first step (or its forward pass): the weights split, and, in
// the workgroups past the weight tiles, the first batch gathered.
__global__ __launch_bounds__(256) void k_panel_prepare(const float *__restrict__ params, int h, int L,
                                                       int ntiles, u4v *__restrict__ frag,
                                                       const GatherArgs rows) {
    __shared__ float tl[8 * WT_S];
    if ((int)blockIdx.x >= ntiles) {
        gather_one(rows, (int64_t)((int)blockIdx.x - ntiles) * 256 + threadIdx.x);
        return;
    }
    const WeightTile w = weight_tile(blockIdx.x, h);
    const int i = threadIdx.x >> 5, j = 2 * (threadIdx.x & 31);
    const float *src = params + (w.l == 1 ? 0 : (int64_t)D_IN * h + (int64_t)(w.l - 2) * h * h) +
                       (int64_t)(w.i0 + i) * h + w.j0 + j;
    tl[i * WT_S + j] = src[0];
    tl[i * WT_S + j + 1] = src[1];
    __syncthreads();
    write_frags(tl, w, h, L, frag);
}

// ---- the panel ----------------------------------------------------------------

struct PanelArgs {
    const float *X;          // rows (through idx when it is not null)
    int64_t n_rows;
    const int32_t *idx;
    int64_t nb;              // rows of the call or batch
    const u4v *frag;
    int64_t words;           // of frag
    const float *wo;
    int L;
    int32_t *err;
    float *ypred;            // forward pass
    const float *Yb;         // the rest: training
    float scale;             // 2 / nb
    float *sq;               // squared residuals
    float *H;                // H_l, l < L, at H + (l - 1) hstride
    int64_t hstride;
    float *G[DEEP_MAX_LAYERS];
    float *dwo;              // [workgroups][h]
};

// Workgroups go to the XCDs in turn. A launch of 128 n workgroups takes its panels
// in groups of 16 on one XCD (n groups on each), the rows of one wgrad chunk at
// batch 4096, which then reads them where they were written.
__device__ __forceinline__ int64_t panel_of(int b, int grid) {
    if (grid % 128) return b;
    const int xcd = b & 7, slot = b >> 3;
    return (int64_t)(xcd + 8 * (slot >> 4)) * 16 + (slot & 15);
}

template <int H>
struct PanelShape {
    static constexpr int NW = H == 64 ? 4 : H == 192 ? 6 : 8;   // waves
    static constexpr int NUT = H / 16 / NW;                      // unit tiles per wave
    static constexpr int KB = H / 32;                            // k blocks of a hidden layer
    static constexpr int LS = H + 8;                             // LDS row stride (bf16)
    static_assert(NUT * NW * 16 == H && NUT <= 2, "panel shape");
};

// 16 RT rows. What bounds it: with 16 rows the weights' stream from L2 (h = 256,
// L = 2: 836 KB a workgroup, about 50 bytes a clock into each CU, 7 us) and the
// latency of the layers' epilogues and barriers; with 64 rows the matrix cores. A
// step of 32-256x2-1 at 4,096 rows takes 27.0 us in a training run against 39.5 as
// GEMM launches (under the profiler, which adds up to a microsecond a launch, 15.2 us
// of this, 10.1 of k_panel_wgrad and 4.3 of k_panel_apply); 1M rows through 32-256x3-1
// 1.20-1.26 ms, as the card's clock allows (221-232 TFLOP/s of fp32 work), against 6.9.
// Panels of 64 rows in training spill 52 registers at 256 units and 20 at 192, and
// remain the faster: 32-256x2-1 at 16,384 rows 72 us a step, 94 as GEMM launches.
template <int H, int RT, bool TRAIN>
__global__ __launch_bounds__((64 * PanelShape<H>::NW)) void k_panel(const PanelArgs a) {
    using S = PanelShape<H>;
    constexpr int NW = S::NW, NUT = S::NUT, KB = S::KB, LS = S::LS, ROWS = 16 * RT;
    extern __shared__ __attribute__((aligned(16))) uint16_t act[];   // [3][ROWS][LS]: activations, split
    __shared__ float part[NW][ROWS];
    __shared__ uint32_t mk[TRAIN ? DEEP_MAX_LAYERS : 1][64 * NW];    // ReLU masks of layers below L

    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int li = lane & 15, lq = lane >> 4;
    const int L = a.L;
    // D k blocks of weights in flight. The scheduler may not move a block's loads
    // (sched_barrier): left to itself it sinks them to their first use, and the
    // stream from L2 stops at every block.
    constexpr int D = KB < 4 || RT > 1 ? 2 : 3;
    u4v w[D][NUT][3];
    const rsrc_t frag = __builtin_amdgcn_make_buffer_rsrc(const_cast<u4v *>(a.frag), (short)0,
                                                          (int)(16 * a.words), 0x00020000);
    const uint32_t lane16 = 16u * (uint32_t)lane;
    auto wload = [&](int64_t base, int nkb, int kb, u4v (&d)[NUT][3]) __attribute__((always_inline)) {
#pragma unroll
        for (int u = 0; u < NUT; ++u)
#pragma unroll
            for (int p = 0; p < 3; ++p)
                // a scalar offset per (unit tile, k block): no address registers per load
                d[u][p] = __builtin_amdgcn_raw_buffer_load_b128(
                    frag, lane16 + 1024u * p, (int)(16 * base) + ((wave * NUT + u) * nkb + kb) * 3072, 0);
    };
    auto prefetch = [&](int64_t base) __attribute__((always_inline)) {
#pragma unroll
        for (int kb = 0; kb < D; ++kb) wload(base, KB, kb, w[kb]);
        __builtin_amdgcn_sched_barrier(0);
    };
    // six part products of one k block: a0 b0 into hi, the smaller five into lo
    constexpr int PA[5] = {2, 1, 0, 1, 0}, PB[5] = {0, 1, 2, 0, 1};
    auto block = [&](const u4v (&wk)[NUT][3], const u4v (&b)[3], int r, f4 (&hi)[NUT][RT],
                     f4 (&lo)[NUT][RT]) __attribute__((always_inline)) {
#pragma unroll
        for (int q = 0; q < 5; ++q)
#pragma unroll
            for (int u = 0; u < NUT; ++u) lo[u][r] = mfma_bf16(wk[u][PA[q]], b[PB[q]], lo[u][r]);
#pragma unroll
        for (int u = 0; u < NUT; ++u) hi[u][r] = mfma_bf16(wk[u][0], b[0], hi[u][r]);
    };
    // hi = the layer's product with the activations in LDS, for the wave's units;
    // its first D k blocks of weights are in flight already
    auto product = [&](int64_t base, f4 (&hi)[NUT][RT]) __attribute__((always_inline)) {
        f4 lo[NUT][RT];
#pragma unroll
        for (int u = 0; u < NUT; ++u)
#pragma unroll
            for (int r = 0; r < RT; ++r) hi[u][r] = lo[u][r] = f4{0.f, 0.f, 0.f, 0.f};
        // the next activations are read from LDS while a block is multiplied
        u4v b[2][3];
        auto bload = [&](int t, u4v (&d)[3]) __attribute__((always_inline)) {
            const int kb = t / RT, r = t % RT;
#pragma unroll
            for (int p = 0; p < 3; ++p)
                d[p] = *reinterpret_cast<const u4v *>(act + (p * ROWS + 16 * r + li) * LS + 32 * kb + 8 * lq);
        };
        bload(0, b[0]);
#pragma unroll
        for (int kb = 0; kb < KB; ++kb) {
#pragma unroll
            for (int r = 0; r < RT; ++r) {
                const int t = kb * RT + r;
                if (t + 1 < KB * RT) bload(t + 1, b[(t + 1) & 1]);
                block(w[kb % D], b[t & 1], r, hi, lo);
            }
            __builtin_amdgcn_sched_barrier(0);
            if (kb + D < KB) wload(base, KB, kb + D, w[kb % D]);
            __builtin_amdgcn_sched_barrier(0);
        }
#pragma unroll
        for (int u = 0; u < NUT; ++u)
#pragma unroll
            for (int r = 0; r < RT; ++r) hi[u][r] += lo[u][r];
    };
    // the wave's values (units ut(u) + 4 lq + v of row li) split into LDS
    auto put = [&](const f4 (&v)[NUT][RT]) __attribute__((always_inline)) {
#pragma unroll
        for (int u = 0; u < NUT; ++u)
#pragma unroll
            for (int r = 0; r < RT; ++r) {
                uint32_t q0[3], q1[3];
                split_pair(v[u][r][0], v[u][r][1], q0);
                split_pair(v[u][r][2], v[u][r][3], q1);
#pragma unroll
                for (int p = 0; p < 3; ++p)
                    *reinterpret_cast<u2v *>(act + (p * ROWS + 16 * r + li) * LS + (wave * NUT + u) * 16 + 4 * lq) =
                        u2v{q0[p], q1[p]};
            }
    };

    float4 wov[NUT];
#pragma unroll
    for (int u = 0; u < NUT; ++u) wov[u] = *reinterpret_cast<const float4 *>(a.wo + (wave * NUT + u) * 16 + 4 * lq);
    float dwo[NUT];
#pragma unroll
    for (int u = 0; u < NUT; ++u) dwo[u] = 0.0f;

    // The weights were written by another launch's XCDs, so each XCD's first read of
    // them misses its L2; the XCD's workgroups (every eighth) read a share each into
    // it at once, instead of waiting on the misses block by block.
    constexpr int WARM = 2;   // a word of every 64 bytes: 2 MB over an XCD's 32 workgroups
    uint32_t warm[WARM];
    {
        const int slots = ((int)gridDim.x + 7) / 8, slot = (int)blockIdx.x / 8;
#pragma unroll
        for (int k = 0; k < WARM; ++k)   // past the buffer's end: no access
            warm[k] = __builtin_amdgcn_raw_buffer_load_b32(
                frag, (uint32_t)((k * slots + slot) * (64 * 64 * NW) + 64 * tid), 0, 0);
    }

    const int64_t npanel = (a.nb + ROWS - 1) / ROWS;
    for (int64_t pn = panel_of(blockIdx.x, gridDim.x); pn < npanel; pn += gridDim.x) {
        const int64_t r0 = pn * ROWS;
        // ---- layer 1: the rows split in registers -------------------------------
        f4 hv[NUT][RT];
        float yt[RT];   // targets
        {
            wload(0, 1, 0, w[0]);
            float4 x[RT][2];
#pragma unroll
            for (int r = 0; r < RT; ++r) {
                const int64_t t = r0 + 16 * r + li;
                const bool in = t < a.nb;
                if constexpr (TRAIN) yt[r] = a.Yb[in ? t : 0];
                int64_t row = in ? t : 0;
                if (a.idx) {
                    row = a.idx[in ? t : a.nb - 1];
                    if (row < 0 || row >= a.n_rows) {
                        __hip_atomic_store(a.err, (int32_t)MLP_ERR_INDEX, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
                        row = 0;
                    }
                }
                x[r][0] = ld4(in, a.X + row * D_IN + 8 * lq);
                x[r][1] = ld4(in, a.X + row * D_IN + 8 * lq + 4);
            }
            f4 lo[NUT][RT];
#pragma unroll
            for (int u = 0; u < NUT; ++u)
#pragma unroll
                for (int r = 0; r < RT; ++r) hv[u][r] = lo[u][r] = f4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
            for (int r = 0; r < RT; ++r) {
                uint32_t q[4][3];
                split_pair(x[r][0].x, x[r][0].y, q[0]);
                split_pair(x[r][0].z, x[r][0].w, q[1]);
                split_pair(x[r][1].x, x[r][1].y, q[2]);
                split_pair(x[r][1].z, x[r][1].w, q[3]);
                u4v b[3];
#pragma unroll
                for (int p = 0; p < 3; ++p) b[p] = u4v{q[0][p], q[1][p], q[2][p], q[3][p]};
                block(w[0], b, r, hv, lo);
            }
#pragma unroll
            for (int k = 0; k < WARM; ++k) asm volatile("" ::"v"(warm[k]));   // the loads are kept
#pragma unroll
            for (int u = 0; u < NUT; ++u)
#pragma unroll
                for (int r = 0; r < RT; ++r) hv[u][r] += lo[u][r];
        }
        // ---- ReLU of layer l (eq. 12; a NaN passes, so that a diverged step reaches
        // the loss), its mask, and H_l to memory (training) and LDS ------------------
        uint32_t mask = 0;
        for (int l = 1;; ++l) {
            // the next product's weights (the last layer of a forward pass or of a
            // one-layer net has none: its loads are not used)
            prefetch(l < L ? frag_fwd(H, l + 1) : TRAIN && L > 1 ? frag_bwd(H, L, L) : 0);
            mask = 0;
#pragma unroll
            for (int u = 0; u < NUT; ++u)
#pragma unroll
                for (int r = 0; r < RT; ++r)
#pragma unroll
                    for (int v = 0; v < 4; ++v) {
                        const float z = hv[u][r][v];
                        hv[u][r][v] = z <= 0.0f ? 0.0f : z;
                        if constexpr (TRAIN) mask |= (hv[u][r][v] > 0.0f ? 1u : 0u) << ((u * RT + r) * 4 + v);
                    }
            if (l == L) break;
            if constexpr (TRAIN) {
                mk[l - 1][tid] = mask;
                float *Hl = a.H + (l - 1) * a.hstride;
#pragma unroll
                for (int u = 0; u < NUT; ++u)
#pragma unroll
                    for (int r = 0; r < RT; ++r) {
                        const int64_t t = r0 + 16 * r + li;
                        if (t < a.nb)
                            *reinterpret_cast<f4 *>(Hl + t * H + (wave * NUT + u) * 16 + 4 * lq) = hv[u][r];
                    }
            }
            put(hv);
            __syncthreads();   // H_l in LDS
            product(frag_fwd(H, l + 1), hv);
            __syncthreads();   // every wave has read it
        }
        // ---- output layer (eq. 13) -----------------------------------------------
        float y[RT];
#pragma unroll
        for (int r = 0; r < RT; ++r) {
            float s = 0.0f;
#pragma unroll
            for (int u = 0; u < NUT; ++u) {
                s = fmaf(hv[u][r][0], wov[u].x, s);
                s = fmaf(hv[u][r][1], wov[u].y, s);
                s = fmaf(hv[u][r][2], wov[u].z, s);
                s = fmaf(hv[u][r][3], wov[u].w, s);
            }
            s = xadd32(xadd16(s));
            if (lq == 0) part[wave][16 * r + li] = s;
        }
        __syncthreads();
#pragma unroll
        for (int r = 0; r < RT; ++r) {
            y[r] = part[0][16 * r + li];
#pragma unroll
            for (int q = 1; q < NW; ++q) y[r] += part[q][16 * r + li];
        }
        if constexpr (!TRAIN) {
            if (wave == 0 && lq == 0)
#pragma unroll
                for (int r = 0; r < RT; ++r)
                    if (r0 + 16 * r + li < a.nb) a.ypred[r0 + 16 * r + li] = y[r];
        } else {
            // residual, dZ_o (eqs. 14-15), the dw_o share (eq. 16) and G_L (eq. 17)
            float g[RT];
#pragma unroll
            for (int r = 0; r < RT; ++r) {
                const int64_t t = r0 + 16 * r + li;
                const bool in = t < a.nb;
                const float res = in ? y[r] - yt[r] : 0.0f;
                g[r] = a.scale * res;
                if (wave == 0 && lq == 0 && in) a.sq[t] = res * res;
            }
            f4 gv[NUT][RT];
#pragma unroll
            for (int u = 0; u < NUT; ++u) {
                float d[4] = {0.f, 0.f, 0.f, 0.f};
                const float wq[4] = {wov[u].x, wov[u].y, wov[u].z, wov[u].w};
#pragma unroll
                for (int r = 0; r < RT; ++r)
#pragma unroll
                    for (int v = 0; v < 4; ++v) {
                        d[v] = fmaf(hv[u][r][v], g[r], d[v]);
                        gv[u][r][v] = (mask >> ((u * RT + r) * 4 + v)) & 1u ? g[r] * wq[v] : 0.0f;
                    }
                dwo[u] += rsum16x4(d, li);
            }
            // back-propagation, eq. 17 one layer down at a time
            for (int l = L;; --l) {
                float *Gl = a.G[l - 1];
#pragma unroll
                for (int u = 0; u < NUT; ++u)
#pragma unroll
                    for (int r = 0; r < RT; ++r) {
                        const int64_t t = r0 + 16 * r + li;
                        if (t < a.nb)
                            *reinterpret_cast<f4 *>(Gl + t * H + (wave * NUT + u) * 16 + 4 * lq) = gv[u][r];
                    }
                if (l == 1) break;
                put(gv);
                __syncthreads();   // G_l in LDS
                product(frag_bwd(H, L, l), gv);
                if (l > 2) prefetch(frag_bwd(H, L, l - 1));
                const uint32_t m = mk[l - 2][tid];
#pragma unroll
                for (int u = 0; u < NUT; ++u)
#pragma unroll
                    for (int r = 0; r < RT; ++r)
#pragma unroll
                        for (int v = 0; v < 4; ++v)
                            gv[u][r][v] = (m >> ((u * RT + r) * 4 + v)) & 1u ? gv[u][r][v] : 0.0f;
                __syncthreads();   // every wave has read it
            }
        }
        __syncthreads();   // part and act are free for the next panel
    }
    if constexpr (TRAIN) {
        // lane li holds unit 4 lq + (li >> 2) of each tile
        if ((li & 3) == 0)
#pragma unroll
            for (int u = 0; u < NUT; ++u)
                a.dwo[(int64_t)blockIdx.x * H + (wave * NUT + u) * 16 + 4 * lq + (li >> 2)] = dwo[u];
    }
}

// ---- weight gradients -----------------------------------------------------------

struct WgradArgs {
    const float *A[DEEP_MAX_LAYERS];   // H_{l-1} (X for l = 1), [nb x h] ([nb x 32])
    const float *G[DEEP_MAX_LAYERS];   // G_l, [nb x h]
    float *out[DEEP_MAX_LAYERS];       // partials of dW_l, partial z at z * size
    int h, L, chunks;
    int64_t nb, kc;                    // rows, rows per chunk (a multiple of 256)
};

// 8 rows x N units of the lane: rows r .. r + 7, N consecutive units at x. Through a
// buffer resource that ends at the chunk's last row: rows past it read zeros, and a
// load needs no 64-bit address.
__device__ __forceinline__ rsrc_t rows_rsrc(const float *P, int64_t rows, int ld) {
    return __builtin_amdgcn_make_buffer_rsrc(const_cast<float *>(P), (short)0, (int)(uint32_t)(rows * ld * 4),
                                             0x00020000);
}
template <int N>
__device__ __forceinline__ void load_rows8(float (&v)[8][N], rsrc_t P, int ld, int64_t r, int x) {
    const uint32_t at = (uint32_t)(r * ld + x) * 4u;
#pragma unroll
    for (int t = 0; t < 8; ++t) {
        if constexpr (N == 1) {
            v[t][0] = __uint_as_float(__builtin_amdgcn_raw_buffer_load_b32(P, at + (uint32_t)(t * ld) * 4u, 0, 0));
        } else if constexpr (N == 4) {
            const u4v q = __builtin_amdgcn_raw_buffer_load_b128(P, at + (uint32_t)(t * ld) * 4u, 0, 0);
#pragma unroll
            for (int n = 0; n < 4; ++n) v[t][n] = __uint_as_float(q[n]);
        } else {
            const u2v q = __builtin_amdgcn_raw_buffer_load_b64(P, at + (uint32_t)(t * ld) * 4u, 0, 0);
            v[t][0] = __uint_as_float(q[0]);
            v[t][1] = __uint_as_float(q[1]);
        }
    }
}
template <int N>
__device__ __forceinline__ void split_unit(const float (&v)[8][N], int n, u4v (&o)[3]) {
    uint32_t q[4][3];
#pragma unroll
    for (int t = 0; t < 4; ++t) split_pair(v[2 * t][n], v[2 * t + 1][n], q[t]);
#pragma unroll
    for (int p = 0; p < 3; ++p) o[p] = u4v{q[0][p], q[1][p], q[2][p], q[3][p]};
}

// c += sum over the lanes' eight rows: a and b of one unit each, six part products
__device__ __forceinline__ f4 mfma6(const u4v (&a)[3], const u4v (&b)[3], f4 c) {
    c = mfma_bf16(a[2], b[0], c);
    c = mfma_bf16(a[1], b[1], c);
    c = mfma_bf16(a[0], b[2], c);
    c = mfma_bf16(a[1], b[0], c);
    c = mfma_bf16(a[0], b[1], c);
    return mfma_bf16(a[0], b[0], c);
}

constexpr int WG_W = 8;                            // waves
constexpr int WG_T = 64 * 64, WG_T1 = 32 * 16;     // outputs of a W_l tile and of a W_1 tile
constexpr int WG_LDS = WG_W * (WG_T + WG_T1) * 4;

// A 64 x 64 tile (tm, tn) of dW_l over one row chunk: wave w takes the chunk's
// 32-row blocks w, w + 8, ..., and the eight waves' sums meet in LDS. MFMA tile
// (i, j) takes units 4 li + i and 4 li + j of the lanes, so that the operands load
// along the units and the outputs leave as 16-byte stores. The workgroups of l = 2
// (of a one-layer net: all) also form the chunk's dW_1 for the units
// 64 tn + 16 g .. + 15, g = tm, tm + h / 64, ... < 4, first, while the tile's
// operands load. (As workgroups of their own those tiles left a fifth of the CUs
// with two workgroups, done 2 us after the others.) Bound by latency: the loads 1.4
// us, splits and products of one block a wave 1.8, the sums in LDS 1.2 of a launch.
// Grid: tiles(h, L) per chunk, chunks rounded up to a multiple of 8: chunk z's tiles
// are all on XCD z % 8, whose L2 then fetches the chunk's rows once.
static inline int wgrad_tiles(int h, int L) { return (L > 1 ? L - 1 : 1) * (h / 64) * (h / 64); }

__global__ __launch_bounds__(64 * WG_W) void k_panel_wgrad(const WgradArgs a) {
    extern __shared__ __attribute__((aligned(16))) float lds[];   // [8][64][64], then [8][32][16]
    const int h = a.h, nt = h / 64, n2 = nt * nt, T = (a.L > 1 ? a.L - 1 : 1) * n2;
    int b = blockIdx.x;
    const int z = (b / (8 * T)) * 8 + (b & 7);
    if (z >= a.chunks) return;
    b = (b % (8 * T)) >> 3;
    const int l = 2 + b / n2;
    b %= n2;
    const int tm = b / nt, tn = b % nt;
    const bool main = a.L > 1;
    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int li = lane & 15, lq = lane >> 4;
    const int64_t rb = (int64_t)z * a.kc, re = rb + a.kc < a.nb ? rb + a.kc : a.nb;
    const int64_t r0 = rb + 32 * wave;

    // the tile's operands (a one-layer net has none: X is read and not used)
    const int lm = main ? l : 1, lda = main ? h : D_IN;
    const rsrc_t A = rows_rsrc(a.A[lm - 1], re, lda), G = rows_rsrc(a.G[lm - 1], re, h);
    float va[8][4], vg[8][4];
    load_rows8<4>(vg, G, h, r0 + 8 * lq, 64 * tn + 4 * li);
    load_rows8<4>(va, A, lda, r0 + 8 * lq, 64 * tm + 4 * li);
    __builtin_amdgcn_sched_barrier(0);
    if (l == 2) {
        const rsrc_t X = rows_rsrc(a.A[0], re, D_IN), G1 = rows_rsrc(a.G[0], re, h);
        float *l1 = lds + WG_W * WG_T;
        for (int g = tm; g < 4; g += nt) {
            f4 acc[2] = {f4{0.f, 0.f, 0.f, 0.f}, f4{0.f, 0.f, 0.f, 0.f}};
            for (int64_t r = r0; r < re; r += 32 * WG_W) {
                float vx[8][2], v1[8][1];
                load_rows8<2>(vx, X, D_IN, r + 8 * lq, 2 * li);
                load_rows8<1>(v1, G1, h, r + 8 * lq, 64 * tn + 16 * g + li);
                u4v q[3], x[3];
                split_unit<1>(v1, 0, q);
#pragma unroll
                for (int i = 0; i < 2; ++i) {
                    split_unit<2>(vx, i, x);
                    acc[i] = mfma6(x, q, acc[i]);
                }
            }
            // lane (li, lq): inputs 2 (4 lq + v) + i, unit li of the group
#pragma unroll
            for (int i = 0; i < 2; ++i)
#pragma unroll
                for (int v = 0; v < 4; ++v) l1[wave * WG_T1 + (2 * (4 * lq + v) + i) * 16 + li] = acc[i][v];
            __syncthreads();
            {
                float s = l1[tid];
#pragma unroll
                for (int w = 1; w < WG_W; ++w) s += l1[w * WG_T1 + tid];
                a.out[0][(int64_t)z * D_IN * h + (int64_t)(tid >> 4) * h + 64 * tn + 16 * g + (tid & 15)] = s;
            }
            __syncthreads();
        }
    }
    if (!main) return;
    f4 acc[4][4];
#pragma unroll
    for (int i = 0; i < 4; ++i)
#pragma unroll
        for (int j = 0; j < 4; ++j) acc[i][j] = f4{0.f, 0.f, 0.f, 0.f};
    auto multiply = [&](const float (&xa)[8][4], const float (&xg)[8][4]) __attribute__((always_inline)) {
        u4v q[4][3];
#pragma unroll
        for (int j = 0; j < 4; ++j) split_unit<4>(xg, j, q[j]);
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            u4v x[3];
            split_unit<4>(xa, i, x);
            constexpr int PA[6] = {2, 1, 0, 1, 0, 0}, PB[6] = {0, 1, 2, 0, 1, 0};
#pragma unroll
            for (int p = 0; p < 6; ++p)
#pragma unroll
                for (int j = 0; j < 4; ++j) acc[i][j] = mfma_bf16(x[PA[p]], q[j][PB[p]], acc[i][j]);
        }
    };
    multiply(va, vg);   // zeros for a wave past the chunk's rows
    for (int64_t r = r0 + 32 * WG_W; r < re; r += 32 * WG_W) {
        float xa[8][4], xg[8][4];
        load_rows8<4>(xg, G, h, r + 8 * lq, 64 * tn + 4 * li);
        load_rows8<4>(xa, A, lda, r + 8 * lq, 64 * tm + 4 * li);
        multiply(xa, xg);
    }
    // lane (li, lq): rows 4 (4 lq + v) + i, columns 4 li .. 4 li + 3
    float *mine = lds + wave * WG_T;
#pragma unroll
    for (int i = 0; i < 4; ++i)
#pragma unroll
        for (int v = 0; v < 4; ++v)
            *reinterpret_cast<f4 *>(mine + (4 * (4 * lq + v) + i) * 64 + 4 * li) =
                f4{acc[i][0][v], acc[i][1][v], acc[i][2][v], acc[i][3][v]};
    __syncthreads();
    float *out = a.out[l - 1] + (int64_t)z * h * h;
#pragma unroll
    for (int q = 0; q < 2; ++q) {
        const int e = q * 2048 + 4 * tid;
        f4 s = *reinterpret_cast<const f4 *>(lds + e);
#pragma unroll
        for (int w = 1; w < WG_W; ++w) s += *reinterpret_cast<const f4 *>(lds + w * WG_T + e);
        *reinterpret_cast<f4 *>(out + (int64_t)(64 * tm + (e >> 6)) * h + 64 * tn + (e & 63)) = s;
    }
}

// ---- update ---------------------------------------------------------------------

struct PanelApply {
    const float *part[DEEP_MAX_LAYERS];   // dW_l partials
    int chunks;                           // of each
    const float *dwo;
    int ndwo;
    int h, L, ntiles;
    float *params, *dparams;
    float lr;
    int sgd;
    u4v *frag;        // null: no further step in this call
    const float *sq;
    int64_t nb;
};

// Workgroups [0, ntiles): a weight tile each (a thread two columns of one row):
// its chunk partials summed in order, eq. 19 (or the gradient out), the new weights
// split for the next step. Then h / 16 workgroups for w_o (16 slices of the
// panels' shares a unit), one for the loss, and the next step's gather.
__global__ __launch_bounds__(256) void k_panel_apply(const PanelApply a, const ReduceArgs ra,
                                                     const GatherArgs next) {
    __shared__ float tl[8 * WT_S];
    const int tid = threadIdx.x;
    int b = blockIdx.x;
    const int h = a.h;
    constexpr int U = 16;   // partial loads in flight (twice as many while they last)
    if (b < a.ntiles) {
        const WeightTile w = weight_tile(b, h);
        const int i = tid >> 5, j = 2 * (tid & 31);
        const int64_t size = (int64_t)(w.l == 1 ? D_IN : h) * h;
        const int64_t e = (int64_t)(w.i0 + i) * h + w.j0 + j;
        const int64_t pe = (w.l == 1 ? 0 : (int64_t)D_IN * h + (int64_t)(w.l - 2) * h * h) + e;
        const float *q = a.part[w.l - 1] + e;
        const float w0 = a.sgd ? a.params[pe] : 0.0f, w1 = a.sgd ? a.params[pe + 1] : 0.0f;
        const int n = a.chunks;
        float2 s = make_float2(0.f, 0.f);
        int z0 = 0;
        for (; z0 + 2 * U <= n; z0 += 2 * U) {
            float2 x[2 * U];
#pragma unroll
            for (int t = 0; t < 2 * U; ++t) x[t] = *reinterpret_cast<const float2 *>(q + (z0 + t) * size);
#pragma unroll
            for (int t = 0; t < 2 * U; ++t) {
                s.x += x[t].x;
                s.y += x[t].y;
            }
        }
        for (; z0 < n; z0 += U) {
            float2 x[U];
#pragma unroll
            for (int t = 0; t < U; ++t) {
                const int z = z0 + t < n ? z0 + t : n - 1;
                x[t] = *reinterpret_cast<const float2 *>(q + z * size);
            }
#pragma unroll
            for (int t = 0; t < U; ++t)
                if (z0 + t < n) {
                    s.x += x[t].x;
                    s.y += x[t].y;
                }
        }
        if (!a.sgd) {
            a.dparams[pe] = s.x;
            a.dparams[pe + 1] = s.y;
            return;
        }
        const float n0 = w0 - a.lr * s.x, n1 = w1 - a.lr * s.y;
        a.params[pe] = n0;
        a.params[pe + 1] = n1;
        if (!a.frag) return;
        tl[i * WT_S + j] = n0;
        tl[i * WT_S + j + 1] = n1;
        __syncthreads();
        write_frags(tl, w, h, a.L, a.frag);
        return;
    }
    b -= a.ntiles;
    if (b < h / 16) {
        const int u = 16 * b + (tid & 15), sl = tid >> 4;
        float s = 0.0f;
        for (int z0 = sl; z0 < a.ndwo; z0 += 16 * 16) {
            float x[16];
#pragma unroll
            for (int t = 0; t < 16; ++t) {
                const int z = z0 + 16 * t < a.ndwo ? z0 + 16 * t : a.ndwo - 1;
                x[t] = a.dwo[(int64_t)z * h + u];
            }
#pragma unroll
            for (int t = 0; t < 16; ++t)
                if (z0 + 16 * t < a.ndwo) s += x[t];
        }
        tl[tid] = s;
        __syncthreads();
        if (tid >= 16) return;
        float d = tl[tid];
#pragma unroll
        for (int t = 1; t < 16; ++t) d += tl[16 * t + tid];
        const int64_t pe = (int64_t)D_IN * h + (int64_t)(a.L - 1) * h * h + u;
        if (a.sgd) a.params[pe] -= a.lr * d;
        else a.dparams[pe] = d;
        return;
    }
    b -= h / 16;
    if (b == 0) {
        batch_loss(a.sq, a.nb, ra);
        return;
    }
    gather_one(next, (int64_t)(b - 1) * 256 + tid);
}

// ---------------------------------------------------------------------------
// Host side
// ---------------------------------------------------------------------------

static int64_t frag_words(int h, int L) { return frag_w1(h) + 2 * (L - 1) * frag_wl(h); }
// G_l buffers beyond the context's two and H_L's slot (which the panel path does
// not use for H_L)
static int extra_g(int L) { return L > 3 ? L - 3 : 0; }

// Workspace of the panel path past the GEMM path's (floats).
size_t panel_ws_floats(int h, int L, int64_t mb) {
    if (h > PANEL_MAX_H) return 0;
    return pad64f(4 * (size_t)frag_words(h, L)) + pad64f((size_t)PANEL_WGS_MAX * h) +
           extra_g(L) * pad64f((size_t)mb * h);
}

void panel_carve(DeepCtx &c, float *p) {
    const int h = c.hidden, L = c.layers;
    c.frag = reinterpret_cast<u4v *>(p);
    p += pad64f(4 * (size_t)frag_words(h, L));
    c.dwo_part = p;
    p += pad64f((size_t)PANEL_WGS_MAX * h);
    for (int l = 1; l <= L; ++l) {
        if (l <= 2) {
            c.PG[l - 1] = c.G[l - 1];
        } else if (l == 3) {
            c.PG[l - 1] = c.H + (int64_t)(L - 1) * c.max_batch * h;
        } else {
            c.PG[l - 1] = p;
            p += pad64f((size_t)c.max_batch * h);
        }
    }
}

// Where a step is faster here than as GEMM launches (us a step, GEMM / panel):
//   three or more layers: always up to 192 units (4 layers of 64 at 16 rows
//     35.1 / 19.1); at 256 from 256 rows (48.1 / 47.9; 59.2 / 47.2 at 1,024,
//     89.0 / 55.5 at 4,096; 45.8 / 47.2 at 16), below which a few workgroups read
//     all the weights alone;
//   two layers: 64 units from 4,096 rows (21.6 / 20.7; 19.5 / 20.7 at 1,024), else
//     from 512 (256 units 26.2 / 25.5, 40.9 / 28.1 at 4,096; 24.8 / 25.4 at 384);
//   one layer: at most 64 rows (64 units 14.4 / 13.8; 14.0 / 16.0 at 256), and at 128
//     units or more from 2,048 to 8,192 (256: 19.7 / 15.9 at 4,096; 26.0 / 28.3 at
//     16,384).
// (A training run's; single steps of more rows: two layers of 64 26.0 / 26.5 at 8,192
// and 38.7 / 33.2 at 16,384; of 256 63.5 / 38.4, 94 / 72, and 333 / 232 at 65,536, where
// three of 256 take 586 / 378 and eight of 192 1,170 / 716.)
bool panel_pays(const DeepCtx &c, int64_t nb) {
    if (!c.frag) return false;
    const int h = c.hidden;
    if (c.layers == 1) return nb <= 64 || (h >= 128 && nb >= 2048 && nb <= 8192);
    if (c.layers == 2) return nb >= (h == 64 ? 4096 : 512);
    return h <= 192 || nb >= 256;
}

// Row tiles of 16 per panel and the grid: the fewest rounds of workgroups, a round
// weighted by its time.
static int panel_rt(int64_t nb, int cap) {
    static const double cost[3] = {1.0, 1.3, 2.0};
    int best = 1;
    double bc = 0.0;
    for (int k = 0, rt = 1; k < 3; ++k, rt *= 2) {
        const int64_t panels = (nb + 16 * rt - 1) / (16 * rt);
        const double t = (double)((panels + cap - 1) / cap) * cost[k];
        if (k == 0 || t < bc) {
            best = rt;
            bc = t;
        }
    }
    return best;
}

template <int H, int RT, bool TRAIN>
static hipError_t launch_panel(hipStream_t st, const PanelArgs &a, int grid) {
    const size_t lds = sizeof(uint16_t) * 3 * 16 * RT * PanelShape<H>::LS;
    hipLaunchKernelGGL((k_panel<H, RT, TRAIN>), dim3(grid), dim3(64 * PanelShape<H>::NW), lds, st, a);
    return hipGetLastError();
}

// Returns the grid through *wgs.
template <bool TRAIN>
static hipError_t panel(hipStream_t st, int h, const PanelArgs &a, int *wgs) {
    const int cap = 256;
    const int rt = panel_rt(a.nb, cap);
    const int64_t panels = (a.nb + 16 * rt - 1) / (16 * rt);
    const int grid = (int)(panels < cap ? panels : cap);
    *wgs = grid;
    switch (h) {
#define PANEL_CASE(H)                                                          \
    case H:                                                                    \
        if (rt == 1) return launch_panel<H, 1, TRAIN>(st, a, grid);            \
        if (rt == 2) return launch_panel<H, 2, TRAIN>(st, a, grid);            \
        return launch_panel<H, 4, TRAIN>(st, a, grid);
        PANEL_CASE(64) PANEL_CASE(128) PANEL_CASE(192) PANEL_CASE(256)
#undef PANEL_CASE
    }
    return hipErrorInvalidValue;
}

static hipError_t prepare(const DeepCtx &c, const GatherArgs *rows) {
    GatherArgs none;
    memset(&none, 0, sizeof(none));
    const int nt = weight_tiles(c.hidden, c.layers);
    const unsigned ng = rows ? blocks_of(rows->nb * (D_IN / 4), 256) : 0;
    hipLaunchKernelGGL(k_panel_prepare, dim3(nt + ng), dim3(256), 0, c.stream, c.params, c.hidden,
                       c.layers, nt, c.frag, rows ? *rows : none);
    return hipGetLastError();
}

static PanelArgs panel_args(const DeepCtx &c, int64_t nb) {
    PanelArgs a;
    memset(&a, 0, sizeof(a));
    a.nb = nb;
    a.frag = c.frag;
    a.words = frag_words(c.hidden, c.layers);
    a.wo = c.params + layer_offset(c.hidden, c.layers + 1);
    a.L = c.layers;
    a.err = &c.ctl->err;
    return a;
}

// Any number of rows straight from X: no activations in memory, no chunks.
hipError_t panel_forward(const DeepCtx &c, const float *X, int64_t n_rows, const int32_t *idx,
                         int64_t B, float *ypred) {
    const hipError_t e = prepare(c, nullptr);
    if (e != hipSuccess) return e;
    PanelArgs a = panel_args(c, B);
    a.X = X;
    a.n_rows = n_rows;
    a.idx = idx;
    a.ypred = ypred;
    int wgs;
    return panel<false>(c.stream, c.hidden, a, &wgs);
}

// One step or gradient. ready: the weights are split and the rows gathered (by the
// previous step of the call); next: the rows of the following step.
hipError_t panel_step(const DeepCtx &c, const GatherArgs &rows, int64_t nb, const ReduceArgs &ra,
                      float *dparams, bool ready, const GatherArgs *next) {
    const int h = c.hidden, L = c.layers;
    hipError_t e = hipSuccess;
    if (!ready) e = prepare(c, &rows);
    if (e != hipSuccess) return e;
    PanelArgs a = panel_args(c, nb);
    a.X = c.Xb;
    a.n_rows = nb;
    a.Yb = c.Yb;
    a.scale = 2.0f / (float)nb;   // eq. 15
    a.sq = c.sq;
    a.H = c.H;
    a.hstride = c.max_batch * h;
    for (int l = 0; l < L; ++l) a.G[l] = c.PG[l];
    a.dwo = c.dwo_part;
    PanelApply ap;
    memset(&ap, 0, sizeof(ap));
    e = panel<true>(c.stream, h, a, &ap.ndwo);
    if (e != hipSuccess) return e;

    // Row chunks of at least 256 rows, at most what the partial buffers (sized for
    // the GEMM path's plan) hold.
    WgradArgs g;
    memset(&g, 0, sizeof(g));
    int64_t chunks = (nb + 255) / 256;
    for (int s = 0; s < L; ++s) {
        const int64_t most = seg_chunks(h, L, nb, s);
        if (chunks > most) chunks = most;
    }
    g.h = h;
    g.L = L;
    g.nb = nb;
    g.kc = ((nb + chunks - 1) / chunks + 255) / 256 * 256;
    g.chunks = (int)((nb + g.kc - 1) / g.kc);
    for (int l = 1; l <= L; ++l) {
        g.A[l - 1] = l == 1 ? c.Xb : c.H + (int64_t)(l - 2) * c.max_batch * h;
        g.G[l - 1] = c.PG[l - 1];
        g.out[l - 1] = c.part + c.part_off[l - 1];
        ap.part[l - 1] = g.out[l - 1];
    }
    hipLaunchKernelGGL(k_panel_wgrad, dim3((unsigned)((g.chunks + 7) / 8 * 8 * wgrad_tiles(h, L))),
                       dim3(64 * WG_W), WG_LDS, c.stream, g);
    e = hipGetLastError();
    if (e != hipSuccess) return e;

    ap.chunks = g.chunks;
    ap.dwo = c.dwo_part;
    ap.h = h;
    ap.L = L;
    ap.ntiles = weight_tiles(h, L);
    ap.params = c.params;
    ap.dparams = dparams;
    ap.lr = ra.lr;
    ap.sgd = ra.sgd;
    ap.frag = next ? c.frag : nullptr;
    ap.sq = c.sq;
    ap.nb = nb;
    GatherArgs none;
    memset(&none, 0, sizeof(none));
    const unsigned ng = next ? blocks_of(next->nb * (D_IN / 4), 256) : 0;
    hipLaunchKernelGGL(k_panel_apply, dim3((unsigned)(ap.ntiles + h / 16 + 1) + ng), dim3(256), 0, c.stream, ap, ra,
                       next ? *next : none);
    return hipGetLastError();
}

}  // namespace mlp
