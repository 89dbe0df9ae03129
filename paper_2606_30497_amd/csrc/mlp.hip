// mlp.hip -- HIP (gfx950) implementation of the C ABI in include/mlp.h:
// fused mini-batch SGD for the d-h-1 ReLU/MSE network of the paper's
// Sec. III (eqs. 11-19), d = 32, no biases.
//
// Kernels in this file (the "tile" path: every gradient, single step and training
// batch the persistent trainer does not take):
//   k_batch<H, WR, ONE>  a workgroup holds every hidden unit and takes a share of
//                        the batch's rows: forward, residual and backward on the
//                        matrix cores, Z1, the mask and P = X^T (dZ2 (.) mask) in
//                        registers. It writes its partial of P and of the sum of
//                        squared residuals to its slot; with ONE (a batch one
//                        workgroup takes alone) it finishes the step itself.
//   k_batch_reduce<H>    sums the slots in a fixed order, forms dW1 = P diag(W2)
//                        and dW2_j = sum_k W1_kj P_kj (equal to eqs. 16-18), then
//                        either writes dW1/dW2/loss or applies W -= lr dW (eq. 19)
//                        and records the step and epoch loss.
// The persistent single-launch trainer lives in train_persistent.hip, the
// forward pass of mlp_forward in forward.hip.
#include <hip/hip_runtime.h>

#include <math.h>
#include <stdint.h>
#include <stdlib.h>
#include <string.h>

#include "bf16x3.h"
#include "lanes.h"
#include "mlp.h"
#include "mlp_internal.h"

namespace mlp {

// ---------------------------------------------------------------------------
// Tile kernels
// ---------------------------------------------------------------------------

// WR waves along rows (32 rows each) x WU along units; NUT unit tiles of 16 a wave.
template <int H, int WR_>
struct BatchShape {
    static constexpr int WR = WR_;
    static constexpr int WU = H == 32 ? 2 : H == 64 ? 4 : 8;
    static constexpr int NUT = H / 16 / WU;
    static constexpr int NW = WR * WU, NT = 64 * NW;
    static constexpr int RB = 32 * WR;                 // rows of one pass
    static constexpr int ITEMS = RB * 8;               // (row pair, input pair) staging items
    static constexpr int IPT = ITEMS > NT ? ITEMS / NT : 1;   // items per staging thread
    static constexpr int NST = ITEMS / IPT;            // staging threads (whole waves)
    static constexpr int XS = 40;                      // bf16 row stride of a staged X part
    static constexpr int GS = RB + 8;                  // bf16 row stride of a staged (g X)^T part
    static_assert(NUT >= 1 && WU * NUT * 16 == H && NST % 64 == 0 && NST <= NT, "shape");
};

// One (row pair, input pair) item of a pass: X[r][2c .. 2c+1] of rows r and
// r + 1, their targets, and whether each row exists.
struct BatchItem {
    float2 a, b;
    float ya, yb;
};

// A step on nb rows (batch position t: row idx[off + t], or off + t). The products
// are fp32 products on the bf16 matrix cores (bf16x3.h). Per pass of RB rows:
//   forward   Z1 = X W1 from the split rows in LDS and the wave's split weights in
//             registers; ReLU, the W2 product and the mask stay in registers, the
//             waves' shares of Ypred meet in LDS (barrier);
//   residual  each staging thread forms dZ2 = (2/n_b) r (eq. 15) of its two rows
//             and scales its own inputs by it: (dZ2 (.) X)^T goes to LDS in three
//             parts, and the rows of the next pass beside it (barrier);
//   backward  P_kj += sum_r (dZ2_r X_rk) [Z1_rj > 0]: the mask is exact in one bf16
//             part, so a product costs three MFMAs, not six.
// What bounds it: at the sizes it serves a workgroup runs one to a few passes, so
// a call is the latency of the gather, the weights' load and split, and two
// launches; the matrix work of 20,001 rows at h = 256 is about 3 us of it. Against
// the vector-ALU kernel it replaced (one unit a thread): the gradient of 20,001
// gathered rows at h = 256 128 -> 14.4 us, training steps of 1,000 rows at h = 64
// 39 -> 7.2 us and of 2,048 at h = 512 78 -> 12.4 us. At 1024 units a wave holds eight
// unit tiles and spills 52-57 registers: 32 rows take 13.2 us there, 7.2 at 512.
template <int H, int WR, bool ONE>
__global__ __launch_bounds__((BatchShape<H, WR>::NT)) void k_batch(
    const float *__restrict__ X, int64_t n_rows, const float *__restrict__ Y,
    const int32_t *__restrict__ idx, int64_t idx_off, int64_t nb, float *__restrict__ partial,
    int64_t slot_stride, const ReduceArgs ra) {
    using S = BatchShape<H, WR>;
    constexpr int NUT = S::NUT, WU = S::WU, RB = S::RB, IPT = S::IPT, XS = S::XS, GS = S::GS;
    __shared__ __attribute__((aligned(16))) uint16_t XR[3 * RB * XS];   // rows, split
    __shared__ __attribute__((aligned(16))) uint16_t GT[3 * 32 * GS];   // (g X)^T, split
    __shared__ __attribute__((aligned(16))) float part[WU][RB];         // shares of Ypred
    __shared__ float red[S::NW];
    // the row waves' partials of P, added at the end ([H][36], k inner)
    __shared__ __attribute__((aligned(16))) float psum[WR > 1 ? (WR - 1) * H * 36 : 4];

    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int li = lane & 15, lq = lane >> 4;
    const int wu = wave % WU, wr = wave / WU;
    const int64_t npass = (nb + RB - 1) / RB;
    const int64_t G = gridDim.x;
    const float scale = 2.0f / (float)nb;
    const bool stager = tid < S::NST;
    int32_t *err = &ra.ctl->err;

    // ---- rows: item q of this thread covers rows 2 rp, 2 rp + 1 and inputs 2 c, 2 c + 1
    auto item_row = [&](int q) { return 2 * ((tid + q * S::NST) >> 4); };
    const int c = tid & 15;
    struct Idx2 { int32_t a, b; };
    auto clamp_t = [&](int64_t t) { return t < nb ? t : nb - 1; };
    auto load_idx = [&](int64_t p, Idx2 (&ix)[IPT]) {
#pragma unroll
        for (int q = 0; q < IPT; ++q) {
            const int64_t t = p * RB + item_row(q);
            if (idx) {
                ix[q].a = idx[idx_off + clamp_t(t)];
                ix[q].b = idx[idx_off + clamp_t(t + 1)];
            }
        }
    };
    auto row_of = [&](int64_t t, int32_t ix) {
        int64_t r = idx ? (int64_t)ix : idx_off + clamp_t(t);
        if (r < 0 || r >= n_rows) {
            __hip_atomic_store(err, (int32_t)MLP_ERR_INDEX, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            r = 0;
        }
        return r;
    };
    // rows past the batch load its last row and are zeroed when they are staged
    auto load_rows = [&](int64_t p, const Idx2 (&ix)[IPT], BatchItem (&it)[IPT]) {
#pragma unroll
        for (int q = 0; q < IPT; ++q) {
            const int64_t t = p * RB + item_row(q);
            const int64_t r0 = row_of(t, ix[q].a), r1 = row_of(t + 1, ix[q].b);
            it[q].a = *reinterpret_cast<const float2 *>(X + r0 * D_IN + 2 * c);
            it[q].b = *reinterpret_cast<const float2 *>(X + r1 * D_IN + 2 * c);
            it[q].ya = Y[r0];
            it[q].yb = Y[r1];
        }
    };
    auto stage = [&](int64_t p, BatchItem (&it)[IPT]) {
#pragma unroll
        for (int q = 0; q < IPT; ++q) {
            const int r = item_row(q);
            const int64_t t = p * RB + r;
            if (t >= nb) it[q].a = make_float2(0.f, 0.f);
            if (t + 1 >= nb) it[q].b = make_float2(0.f, 0.f);
            uint32_t wa[3], wb[3];
            split_pair(it[q].a.x, it[q].a.y, wa);
            split_pair(it[q].b.x, it[q].b.y, wb);
#pragma unroll
            for (int s = 0; s < 3; ++s) {
                uint32_t *d = reinterpret_cast<uint32_t *>(XR + (s * RB + r) * XS + 2 * c);
                d[0] = wa[s];
                d[XS / 2] = wb[s];
            }
        }
    };

    int64_t p = blockIdx.x;
    Idx2 ix[IPT];
    BatchItem cur[IPT], nxt[IPT];
    if (stager) {
        load_idx(p, ix);
        load_rows(p, ix, cur);
        load_idx(p + G, ix);
    }
    // the wave's weights, for its whole life: the parts of W1[8 lq + t][unit]
    // (t = 0..7) of unit 16 (wu NUT + u) + li, and W2[unit]
    const float *__restrict__ W1 = ra.W1;
    u4v w1p[NUT][3];
    float w2v[NUT];
#pragma unroll
    for (int u = 0; u < NUT; ++u) {
        const int unit = 16 * (wu * NUT + u) + li;
        uint32_t w[4][3];
#pragma unroll
        for (int t = 0; t < 4; ++t)
            split_pair(W1[(8 * lq + 2 * t) * H + unit], W1[(8 * lq + 2 * t + 1) * H + unit], w[t]);
#pragma unroll
        for (int s = 0; s < 3; ++s) w1p[u][s] = u4v{w[0][s], w[1][s], w[2][s], w[3][s]};
        w2v[u] = ra.W2[unit];
    }
    f4 pacc[2][NUT];   // P[16 kt + 4 lq + v][unit]
#pragma unroll
    for (int kt = 0; kt < 2; ++kt)
#pragma unroll
        for (int u = 0; u < NUT; ++u) pacc[kt][u] = f4{0.f, 0.f, 0.f, 0.f};
    float sse = 0.0f;
    if (stager) {
        stage(p, cur);
        load_rows(p + G, ix, nxt);
        load_idx(p + 2 * G, ix);
    }
    __syncthreads();

    for (; p < npass; p += G) {
        // ---- forward: Z1 tiles (eq. 11), mask words, shares of Ypred (eqs. 12-13)
        uint32_t mw[NUT][4];   // the mask of rows 4 lq + 0..1, + 2..3 of tiles 0 and 1 as bf16 pairs
        {
            u4v xp[2][3];
#pragma unroll
            for (int i = 0; i < 2; ++i)
#pragma unroll
                for (int s = 0; s < 3; ++s)
                    xp[i][s] = *reinterpret_cast<const u4v *>(XR + (s * RB + wr * 32 + 16 * i + li) * XS + 8 * lq);
            float yp[2][4] = {{0.f, 0.f, 0.f, 0.f}, {0.f, 0.f, 0.f, 0.f}};
            constexpr int UG = NUT < 4 ? NUT : NUT == 4 ? 4 : 2;   // unit tiles in flight (to bound registers)
            constexpr int PA[6] = {2, 1, 0, 1, 0, 0}, PB[6] = {0, 1, 2, 0, 1, 0};
#pragma unroll
            for (int ug = 0; ug < NUT; ug += UG) {
                f4 acc[UG][2];
#pragma unroll
                for (int u = 0; u < UG; ++u) acc[u][0] = acc[u][1] = f4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
                for (int q = 0; q < 6; ++q)
#pragma unroll
                    for (int u = 0; u < UG; ++u)
#pragma unroll
                        for (int i = 0; i < 2; ++i)
                            acc[u][i] = mfma_bf16(xp[i][PA[q]], w1p[ug + u][PB[q]], acc[u][i]);
#pragma unroll
                for (int u = 0; u < UG; ++u)
#pragma unroll
                    for (int i = 0; i < 2; ++i) {
#pragma unroll
                        for (int h = 0; h < 2; ++h)   // [z > 0] as bf16 1.0 or 0 (ReLU'(0) = 0)
                            mw[ug + u][2 * i + h] = (acc[u][i][2 * h] > 0.0f ? 0x00003F80u : 0u) |
                                                    (acc[u][i][2 * h + 1] > 0.0f ? 0x3F800000u : 0u);
#pragma unroll
                        for (int v = 0; v < 4; ++v) {
                            // ReLU as an integer max on the bits (forward.hip)
                            const float z = __int_as_float(max(__float_as_int(acc[u][i][v]), 0));
                            yp[i][v] = fmaf(z, w2v[ug + u], yp[i][v]);
                        }
                    }
            }
#pragma unroll
            for (int i = 0; i < 2; ++i) {
                const float rowv = rsum16x4(yp[i], li);   // row 4 lq + (li >> 2) of the tile
                if ((li & 3) == 0) part[wu][wr * 32 + 16 * i + 4 * lq + (li >> 2)] = rowv;
            }
        }
        __syncthreads();   // shares of Ypred written; the forward's reads of XR done
        // ---- residuals; (g X)^T and the next pass's rows into LDS -----------------
        if (stager) {
#pragma unroll
            for (int q = 0; q < IPT; ++q) {
                const int r = item_row(q);
                const int64_t t = p * RB + r;
                float2 y = *reinterpret_cast<const float2 *>(&part[0][r]);
#pragma unroll
                for (int w = 1; w < WU; ++w) {
                    const float2 z = *reinterpret_cast<const float2 *>(&part[w][r]);
                    y.x += z.x;
                    y.y += z.y;
                }
                const float ea = t < nb ? y.x - cur[q].ya : 0.0f, eb = t + 1 < nb ? y.y - cur[q].yb : 0.0f;
                if (c == 0) sse = fmaf(eb, eb, fmaf(ea, ea, sse));   // eq. 14
                const float ga = scale * ea, gb = scale * eb;       // eq. 15
                uint32_t w0[3], w1[3];
                split_pair(ga * cur[q].a.x, gb * cur[q].b.x, w0);
                split_pair(ga * cur[q].a.y, gb * cur[q].b.y, w1);
                // column of row r of its 32-row block: the order of the mask words,
                // 8 lq + 4 i + v for row 16 i + 4 lq + v
                const int rl = r & 31;
                const int col = (r & ~31) + 8 * ((rl & 15) >> 2) + 4 * (rl >> 4) + (rl & 3);
#pragma unroll
                for (int s = 0; s < 3; ++s) {
                    uint32_t *d = reinterpret_cast<uint32_t *>(GT + (s * 32 + 2 * c) * GS + col);
                    d[0] = w0[s];
                    d[GS / 2] = w1[s];
                }
            }
            if (p + G < npass) {
#pragma unroll
                for (int q = 0; q < IPT; ++q) cur[q] = nxt[q];
                stage(p + G, cur);
                load_rows(p + 2 * G, ix, nxt);
                load_idx(p + 3 * G, ix);
            }
        }
        __syncthreads();   // (g X)^T and the next rows written
        // ---- backward: P += (g X)^T mask over the wave's 32 rows --------------------
#pragma unroll
        for (int kt = 0; kt < 2; ++kt) {
            u4v a[3];
#pragma unroll
            for (int s = 0; s < 3; ++s)
                a[s] = *reinterpret_cast<const u4v *>(GT + (s * 32 + 16 * kt + li) * GS + wr * 32 + 8 * lq);
#pragma unroll
            for (int s = 2; s >= 0; --s)
#pragma unroll
                for (int u = 0; u < NUT; ++u)
                    pacc[kt][u] = mfma_bf16(a[s], u4v{mw[u][0], mw[u][1], mw[u][2], mw[u][3]}, pacc[kt][u]);
        }
    }

    // ---- the workgroup's P (row waves added in order) and sum of squares --------
    {
        const float s = sum64(sse);
        if (lane == 0) red[wave] = s;
    }
    if constexpr (WR > 1) {
        if (wr > 0)
#pragma unroll
            for (int kt = 0; kt < 2; ++kt)
#pragma unroll
                for (int u = 0; u < NUT; ++u)
                    *reinterpret_cast<f4 *>(psum + ((wr - 1) * H + 16 * (wu * NUT + u) + li) * 36 + 16 * kt + 4 * lq) =
                        pacc[kt][u];
    }
    __syncthreads();
    if constexpr (WR > 1) {
        if (wr > 0) return;
#pragma unroll
        for (int w = 0; w < WR - 1; ++w)
#pragma unroll
            for (int kt = 0; kt < 2; ++kt)
#pragma unroll
                for (int u = 0; u < NUT; ++u)
                    pacc[kt][u] += *reinterpret_cast<const f4 *>(
                        psum + (w * H + 16 * (wu * NUT + u) + li) * 36 + 16 * kt + 4 * lq);
    }
    float tot = red[0];
#pragma unroll
    for (int w = 1; w < S::NST / 64; ++w) tot += red[w];
    if constexpr (!ONE) {
        float *slot = partial + (int64_t)blockIdx.x * slot_stride;   // [H][32], k inner, then the sum of squares
#pragma unroll
        for (int kt = 0; kt < 2; ++kt)
#pragma unroll
            for (int u = 0; u < NUT; ++u)
                *reinterpret_cast<f4 *>(slot + (16 * (wu * NUT + u) + li) * 32 + 16 * kt + 4 * lq) = pacc[kt][u];
        if (tid == 0) slot[32 * H] = tot;
    } else {
#pragma unroll
        for (int u = 0; u < NUT; ++u) {
            const int j = 16 * (wu * NUT + u) + li;
            float w1[2][4], d2 = 0.0f;
#pragma unroll
            for (int kt = 0; kt < 2; ++kt)
#pragma unroll
                for (int v = 0; v < 4; ++v) {
                    w1[kt][v] = W1[(16 * kt + 4 * lq + v) * H + j];
                    d2 = fmaf(w1[kt][v], pacc[kt][u][v], d2);   // dW2_j = sum_k W1_kj P_kj
                }
            d2 = xadd32(xadd16(d2));
#pragma unroll
            for (int kt = 0; kt < 2; ++kt)
#pragma unroll
                for (int v = 0; v < 4; ++v) {
                    const int e = (16 * kt + 4 * lq + v) * H + j;
                    const float d1 = w2v[u] * pacc[kt][u][v];   // dW1_kj = W2_j P_kj
                    if (ra.sgd) ra.W1[e] = w1[kt][v] - ra.lr * d1;   // eq. 19
                    else ra.dW1[e] = d1;
                }
            if (lq == 0) {
                if (ra.sgd) ra.W2[j] = w2v[u] - ra.lr * d2;
                else ra.dW2[j] = d2;
            }
        }
        if (tid == 0) record_loss(ra, tot);
    }
}

// Fixed-order reduction of G <= TILE_SLOTS slots: workgroup j sums unit j's 32
// words of P (32 threads' slices of slots, eight lanes of four words each; the
// slices s, s + 32, ... of a thread in order, then a fixed tree) and finishes the
// unit; workgroup H takes the loss. All of a thread's loads are in flight together.
template <int H>
__global__ __launch_bounds__(256) void k_batch_reduce(const float *__restrict__ partial, int G,
                                                      int64_t slot_stride, const ReduceArgs ra) {
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int j = blockIdx.x;
    __shared__ __attribute__((aligned(16))) float red[4][32];
    if (j == H) {
        float s = tid < G ? partial[(int64_t)tid * slot_stride + 32 * H] : 0.0f;
        s = sum64(s);
        if (lane == 0) red[0][wave] = s;
        __syncthreads();
        if (tid == 0) record_loss(ra, ((red[0][0] + red[0][1]) + red[0][2]) + red[0][3]);
        return;
    }
    constexpr int N = TILE_SLOTS / 32;
    const int kc = tid & 7, s0 = tid >> 3;
    // read before the sums, so that every load of the workgroup is in flight at once
    const int k = tid & 31;
    const float w1 = ra.W1[k * H + j], w2 = ra.W2[j];
    f4 x[N];
#pragma unroll
    for (int q = 0; q < N; ++q) {
        const int g = s0 + 32 * q < G ? s0 + 32 * q : G - 1;   // always a written slot
        x[q] = *reinterpret_cast<const f4 *>(partial + (int64_t)g * slot_stride + 32 * j + 4 * kc);
    }
    f4 s = f4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int q = 0; q < N; ++q)
        if (s0 + 32 * q < G) s += x[q];
#pragma unroll
    for (int v = 0; v < 4; ++v) s[v] = xadd32(xadd16(xadd8(s[v])));   // the wave's eight slices
    if (lane < 8) *reinterpret_cast<f4 *>(&red[wave][4 * lane]) = s;
    __syncthreads();
    if (tid >= 64) return;
    const float pk = ((red[0][k] + red[1][k]) + red[2][k]) + red[3][k];   // P_kj, in both half waves
    const float d1 = w2 * pk;                             // dW1_kj = W2_j P_kj
    const float d2 = xadd16(rsum16(w1 * pk));             // dW2_j = sum_k W1_kj P_kj
    if (tid < 32) {
        if (ra.sgd) ra.W1[k * H + j] = w1 - ra.lr * d1;   // eq. 19
        else ra.dW1[k * H + j] = d1;
        if (tid == 0) {
            if (ra.sgd) ra.W2[j] = w2 - ra.lr * d2;
            else ra.dW2[j] = d2;
        }
    }
}

__global__ void k_fill(float *p, int64_t n, float v) {
    const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i < n) p[i] = v;
}

__global__ void k_clear_ctl(Control *c) {
    if (blockIdx.x == 0) {
        if (threadIdx.x == 0) {
            c->err = 0;
            c->abort = 0;
            c->epoch_sse = 0.0;
        }
        c->reg[threadIdx.x] = 0;   // 64 threads
    }
}

// ---------------------------------------------------------------------------
// Host-side launchers for the tile path
// ---------------------------------------------------------------------------

#define MLP_DISPATCH_H(h, ...)                 \
    switch (h) {                                \
    case 32: { constexpr int HH = 32; __VA_ARGS__; }   \
    case 64: { constexpr int HH = 64; __VA_ARGS__; }   \
    case 128: { constexpr int HH = 128; __VA_ARGS__; } \
    case 256: { constexpr int HH = 256; __VA_ARGS__; } \
    case 512: { constexpr int HH = 512; __VA_ARGS__; } \
    case 1024: { constexpr int HH = 1024; __VA_ARGS__; } \
    default: return hipErrorInvalidValue;       \
    }

// Passes of RB rows over at most TILE_SLOTS workgroups; a batch of at most
// ONE_ROWS rows is one workgroup's, in one launch.
template <int H, int WR>
static hipError_t launch_batch(const Ctx &c, const float *X, int64_t n_rows, const float *Y,
                               const int32_t *idx, int64_t idx_off, int64_t nb, const ReduceArgs &a) {
    using S = BatchShape<H, WR>;
    const int G = tile_workgroups(c.hidden, nb);
    if (G == 1) {
        hipLaunchKernelGGL((k_batch<H, WR, true>), dim3(1), dim3(S::NT), 0, c.stream, X, n_rows, Y,
                           idx, idx_off, nb, c.slots, c.slot_stride, a);
        return hipGetLastError();
    }
    hipLaunchKernelGGL((k_batch<H, WR, false>), dim3(G), dim3(S::NT), 0, c.stream, X, n_rows, Y, idx,
                       idx_off, nb, c.slots, c.slot_stride, a);
    const hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
    hipLaunchKernelGGL((k_batch_reduce<H>), dim3(H + 1), dim3(256), 0, c.stream, c.slots, G,
                       c.slot_stride, a);
    return hipGetLastError();
}

// One workgroup runs up to this many rows itself (two passes of 32). Steps of 33 to 64
// rows so, and on two workgroups with the reduction's launch: 5.0 us and 8.5 at
// h <= 128, 6.4 and 8.7 at 256, 9.3 and 10.7 at 512. At 1024, where a pass is longest,
// the two launches would be 4 % faster (17.7 us against 18.5); the line is one for all.
constexpr int64_t ONE_ROWS = 64;

// Workgroups of a batch of nb rows: one per pass of RB rows (64 at h = 32, else
// 32), at most TILE_SLOTS.
int tile_workgroups(int hidden, int64_t nb) {
    if (nb <= ONE_ROWS) return 1;
    const int rb = hidden == 32 ? 64 : 32;
    const int64_t g = (nb + rb - 1) / rb;
    return (int)(g < TILE_SLOTS ? g : TILE_SLOTS);
}

hipError_t tile_step(const Ctx &c, const float *X, int64_t n_rows, const float *Y,
                     const int32_t *idx, int64_t idx_off, int64_t nb, const ReduceArgs &a) {
    MLP_DISPATCH_H(c.hidden, {
        return (launch_batch<HH, HH == 32 ? 2 : 1>(c, X, n_rows, Y, idx, idx_off, nb, a));
    });
}

hipError_t clear_control(const Ctx &c) {
    hipLaunchKernelGGL(k_clear_ctl, dim3(1), dim3(64), 0, c.stream, c.ctl);
    return hipGetLastError();
}

__global__ void k_zero64(uint64_t *p, int64_t n) {
    for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < n;
         i += (int64_t)gridDim.x * blockDim.x)
        p[i] = 0;
}

hipError_t clear_words(const Ctx &c, uint64_t *p, int64_t n) {
    if (n <= 0) return hipSuccess;
    hipLaunchKernelGGL(k_zero64, dim3(1024), dim3(256), 0, c.stream, p, n);
    return hipGetLastError();
}

hipError_t fill(const Ctx &c, float *p, int64_t n, float v) {
    if (n <= 0) return hipSuccess;
    hipLaunchKernelGGL(k_fill, dim3((unsigned)((n + 255) / 256)), dim3(256), 0, c.stream, p, n, v);
    return hipGetLastError();
}

}  // namespace mlp
