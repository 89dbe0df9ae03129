// forward.hip -- the forward pass over many rows (eqs. 11-13), for inference
// and full-dataset evaluation (mlp_forward), with fp32 products formed on the
// bf16 matrix cores.
//
// Per sample the pass is 2 * 32 * h FLOP of the layer-1 contraction plus 2 h
// of the output product against 132 bytes of HBM traffic (an X row and its
// output; 4 more with a row index).
//
// The 32-deep contraction of a 16-row tile with a 16-unit tile is one
// v_mfma_f32_16x16x32_bf16 per part product: X and W1 are split into three
// bf16 parts each (bf16x3.h) and the six part products with i + j <= 2 are
// accumulated in fp32, smallest first -- six 16-cycle MFMAs where fp32 MFMA
// takes eight of 32 cycles, and a bf16 MFMA does not hold up the other waves
// of its SIMD.
//
// A wave keeps the split weights of up to 128 hidden units in registers for its
// whole life (three parts of W1[8 lq .. 8 lq + 7][unit] per unit tile, 12
// VGPRs, plus one W2 value) and streams 16-row tiles of X:
//   lane (li, lq) = (lane % 16, lane / 16) loads X[row li][8 lq .. 8 lq + 7]
//   (two 16-byte loads), which is its A operand of the MFMA, and splits it; the
//   MFMAs accumulate Z1[4 lq + v][unit 16 u + li] of unit tile u in acc[u][v];
//   ReLU and the W2 product stay in registers (eqs. 12-13), and a DPP
//   butterfly sums each row's 16 unit lanes.
// For h > 128 the waves of a workgroup split the units of one row tile and add
// their partial outputs in LDS in a fixed order. The next tile's rows are
// loaded while the current tile is on the matrix cores.
#include <hip/hip_runtime.h>

#include <stdint.h>

#include "bf16x3.h"
#include "lanes.h"
#include "mlp.h"
#include "mlp_internal.h"

namespace mlp {

template <int H>
struct FwdShape {
    static constexpr int UW = H < 128 ? H : 128;   // units per wave
    static constexpr int NUT = UW / 16;            // unit tiles per wave
    static constexpr int WPT = H / UW;             // waves per row tile: 1, 2, 4 or 8
    static constexpr int WAVES = WPT > 4 ? WPT : 4;   // waves per workgroup
    static constexpr int TPI = WAVES / WPT;        // row-tile slots per workgroup iteration
    // row tiles per slot and iteration: the HBM-bound h = 32 keeps four tiles
    // of loads in flight per wave (at four waves a SIMD)
    static constexpr int RT = H == 32 ? 4 : 1;
    // waves per SIMD the register budget allows (a wave holds 13 registers per
    // unit tile of weights and 4 of accumulators, about 40 more, and 8 per row
    // tile in flight): small nets need enough row loads outstanding; at
    // 128 units a wave, three (168 registers, a few of them spilled) beat two
    // (172) where a workgroup's waves fit three times, i.e. except at h = 1024
    // (eight waves a workgroup)
    static constexpr int WAVES_PER_SIMD = NUT <= 4 ? 4 : WPT == 8 ? 2 : 3;
    static_assert(H % 16 == 0 && WPT * UW == H && WPT <= 8, "shape");
};

// Rows of one 16-row tile as MFMA A operands: lane (li, lq) holds
// X[r_t][8 lq .. 8 lq + 7] of batch position t = r0 + li (zeros past B).
struct RowTile {
    float x[8];
};

// The batch index of tile row t, loaded ahead of the rows it selects (an
// unconditional load from a clamped address; only read for t < B).
__device__ __forceinline__ int32_t load_index(const int32_t *__restrict__ idx, int64_t B, int64_t t) {
    return idx ? idx[t < B ? t : B - 1] : 0;
}
// Rows r0 + li (t < B) of X, through the index ix loaded for them.
__device__ __forceinline__ RowTile load_rows(const float *__restrict__ X, int64_t n_rows,
                                             const int32_t *__restrict__ idx, int64_t B, int64_t r0,
                                             int32_t ix, int li, int lq, int32_t *err) {
    RowTile rt;
    const int64_t t = r0 + li;
    float4 a = make_float4(0.f, 0.f, 0.f, 0.f), b = a;
    if (t < B) {
        int64_t r = idx ? (int64_t)ix : t;
        if (r < 0 || r >= n_rows) {
            __hip_atomic_store(err, (int32_t)MLP_ERR_INDEX, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            r = 0;
        }
        const float4 *p = reinterpret_cast<const float4 *>(X + r * D_IN + 8 * lq);
        a = p[0];
        b = p[1];
    }
    rt.x[0] = a.x; rt.x[1] = a.y; rt.x[2] = a.z; rt.x[3] = a.w;
    rt.x[4] = b.x; rt.x[5] = b.y; rt.x[6] = b.z; rt.x[7] = b.w;
    return rt;
}

template <int H>
__global__ __launch_bounds__(64 * FwdShape<H>::WAVES, FwdShape<H>::WAVES_PER_SIMD) void k_forward(
    const float *__restrict__ X, int64_t n_rows, const int32_t *__restrict__ idx, int64_t B,
    const float *__restrict__ W1, const float *__restrict__ W2, float *__restrict__ ypred,
    int32_t *err) {
    using S = FwdShape<H>;
    constexpr int NUT = S::NUT, WPT = S::WPT, TPI = S::TPI, RT = S::RT;
    __shared__ float part[S::WAVES][16];   // partial outputs of the waves of a row tile (WPT > 1)

    const int lane = threadIdx.x & 63;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int li = lane & 15, lq = lane >> 4;
    const int wt = wave / WPT;   // row-tile slot within an iteration
    const int wu = wave % WPT;   // unit block: units [wu * UW, wu * UW + UW)

    // the wave's weights, for its whole life: the parts of W1[8 lq + t][unit]
    // (t = 0..7), and W2[unit]
    u4v w1p[NUT][3];
    float w2v[NUT];
#pragma unroll
    for (int u = 0; u < NUT; ++u) {
        const int unit = wu * S::UW + 16 * u + li;
        uint32_t w[4][3];
#pragma unroll
        for (int t = 0; t < 4; ++t)
            split_pair(W1[(8 * lq + 2 * t) * H + unit], W1[(8 * lq + 2 * t + 1) * H + unit], w[t]);
#pragma unroll
        for (int p = 0; p < 3; ++p) w1p[u][p] = u4v{w[0][p], w[1][p], w[2][p], w[3][p]};
        w2v[u] = W2[unit];
    }

    // one 16-row tile rt at batch row r0: eq. 11 (the six part products
    // smallest first, every unit tile's product of one part pair back to back),
    // ReLU and the W2 product in registers (eqs. 12-13), the row sums out
    auto tile = [&](const RowTile &rt, int64_t r0) __attribute__((always_inline)) {
        u4v xp[3];
        {
            uint32_t w[4][3];
#pragma unroll
            for (int t = 0; t < 4; ++t) split_pair(rt.x[2 * t], rt.x[2 * t + 1], w[t]);
#pragma unroll
            for (int p = 0; p < 3; ++p) xp[p] = u4v{w[0][p], w[1][p], w[2][p], w[3][p]};
        }
        constexpr int PA[6] = {2, 1, 0, 1, 0, 0}, PB[6] = {0, 1, 2, 0, 1, 0};
        f4 acc[NUT];
#pragma unroll
        for (int u = 0; u < NUT; ++u) acc[u] = f4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
        for (int q = 0; q < 6; ++q)
#pragma unroll
            for (int u = 0; u < NUT; ++u) acc[u] = mfma_bf16(xp[PA[q]], w1p[u][PB[q]], acc[u]);
        // the lane's share of Ypred for rows 4 lq + v, units ascending
        float yp[4] = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
        for (int u = 0; u < NUT; ++u)
#pragma unroll
            for (int v = 0; v < 4; ++v) {
                // ReLU as an integer max on the bits: every negative float
                // (-0 included) has a negative pattern and becomes +0, every
                // positive one stays; one instruction, where the float form
                // costs two (a canonicalizing max first)
                const float z = __int_as_float(max(__float_as_int(acc[u][v]), 0));
                yp[v] = fmaf(z, w2v[u], yp[v]);
            }
        // lane li ends with row 4 lq + (li >> 2) summed over the 16 unit lanes
        const float rowv = rsum16x4(yp, li);
        const int rr = 4 * lq + (li >> 2);
        if constexpr (WPT == 1) {
            if ((li & 3) == 0 && r0 + rr < B) ypred[r0 + rr] = rowv;
        } else {
            if ((li & 3) == 0) part[wave][rr] = rowv;
            __syncthreads();
            if (wu == 0 && lane < 16 && r0 + lane < B) {
                float s = 0.0f;
#pragma unroll
                for (int w = 0; w < WPT; ++w) s += part[wt * WPT + w][lane];
                ypred[r0 + lane] = s;
            }
            __syncthreads();
        }
    };

    // iteration it: tiles (it TPI + wt) RT + j, j < RT, of this wave
    const int64_t ntiles = (B + 15) / 16;
    const int64_t iters = (ntiles + TPI * RT - 1) / (TPI * RT);
    auto row0 = [&](int64_t i, int j) { return ((i * TPI + wt) * RT + j) * 16; };
    int64_t it = blockIdx.x;
    RowTile cur[RT];
    int32_t ixn[RT];
#pragma unroll
    for (int j = 0; j < RT; ++j) {
        cur[j] = load_rows(X, n_rows, idx, B, row0(it, j), load_index(idx, B, row0(it, j) + li), li, lq, err);
        ixn[j] = load_index(idx, B, row0(it + gridDim.x, j) + li);
    }
    __builtin_amdgcn_s_waitcnt(0x0F70);   // vmcnt(0)
    for (; it < iters; it += gridDim.x) {
        // the next iteration's rows, in flight while these tiles are computed,
        // and the indices of the iteration after it
        RowTile nxt[RT];
#pragma unroll
        for (int j = 0; j < RT; ++j) {
            nxt[j] = load_rows(X, n_rows, idx, B, row0(it + gridDim.x, j), ixn[j], li, lq, err);
            ixn[j] = load_index(idx, B, row0(it + 2 * (int64_t)gridDim.x, j) + li);
        }
#pragma unroll
        for (int j = 0; j < RT; ++j) tile(cur[j], row0(it, j));
#pragma unroll
        for (int j = 0; j < RT; ++j) cur[j] = nxt[j];
    }
}

template <int H>
static hipError_t launch_forward_h(const Ctx &c, const float *X, int64_t n_rows,
                                   const int32_t *idx, int64_t B, float *ypred) {
    using S = FwdShape<H>;
    const int64_t ntiles = (B + 15) / 16;
    const int64_t iters = (ntiles + S::TPI * S::RT - 1) / (S::TPI * S::RT);
    // resident workgroups: WAVES_PER_SIMD waves on each of a CU's four SIMDs
    const int64_t cap = (int64_t)S::WAVES_PER_SIMD * 4 / S::WAVES * (c.num_cu > 0 ? c.num_cu : 256);
    const int grid = (int)(iters < cap ? iters : cap);
    hipLaunchKernelGGL((k_forward<H>), dim3(grid), dim3(64 * S::WAVES), 0, c.stream, X, n_rows, idx,
                       B, c.W1, c.W2, ypred, &c.ctl->err);
    return hipGetLastError();
}

// ---- many rows through 256 units or more ------------------------------------------
//
// A wave takes 128 units (four tiles of 32) and 32 rows a pass, as Z1^T: the weights
// are the A operand of v_mfma_f32_32x32x16_bf16, the rows its B operand, so lane l
// holds row l % 32 and, in its registers, units: ReLU, the W2 product and the sum
// over the wave's units stay in the lane, and one exchange in LDS ends them. The
// vector work of a pass (its epilogues and the next rows' splits, about five
// instructions an MFMA) is issued between the MFMAs, one unit tile behind: on a bare
// loop with constant operands 24 of these MFMAs and 160 vector instructions take 467
// ns interleaved and 510 in two blocks, 48 16x16x32 ones 520 and 570.
// Bound by the card's power: 10M rows through 256 units always take 1.26M clocks, three
// quarters of them with the matrix cores busy, but at 1.7 GHz and, run after run, less
// (705-800 us; of zeros, which draw less, 527 us: 2.4 GHz). That is 210-235 TFLOP/s of
// fp32 work, 1,270-1,400 of bf16; a large library bf16 product reaches 1,430 on the same
// card, and 1,800 of zeros. Against k_forward on one box, 4M rows: 256 units 341 -> 317
// us, 512 642 -> 602, 1024 1,303 -> 1,159 (before the 64-bit sums below).
template <int H>
struct WideShape {
    static constexpr int UW = 128;                    // units per wave
    static constexpr int NUT = UW / 32;               // unit tiles per wave
    static constexpr int WPT = H / UW;                // waves per row tile
    static constexpr int WAVES = WPT > 4 ? WPT : 4;   // waves per workgroup
    static constexpr int TPI = WAVES / WPT;           // row tiles per workgroup pass
    static constexpr int WAVES_PER_SIMD = 2;
    static_assert(WPT * UW == H && WPT >= 2 && WPT <= 8, "shape");
};

template <int H, bool IDX>
__global__ __launch_bounds__(64 * WideShape<H>::WAVES, WideShape<H>::WAVES_PER_SIMD) void k_forward_wide(
    const float *__restrict__ X, int64_t n_rows, const int32_t *__restrict__ idx, int64_t B,
    const float *__restrict__ W1, const float *__restrict__ W2, float *__restrict__ ypred,
    int32_t *err) {
    using S = WideShape<H>;
    constexpr int NUT = S::NUT, WPT = S::WPT, TPI = S::TPI;
    __shared__ __attribute__((aligned(16))) float w2s[H];
    __shared__ float part[2][S::WAVES][64];   // the lanes' shares of a pass, by its parity

    const int lane = threadIdx.x & 63;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int lr = lane & 31, lh = lane >> 5;
    const int wt = wave / WPT, wu = wave % WPT;

    const int64_t ntiles = (B + 31) / 32;
    const int64_t iters = (ntiles + TPI - 1) / TPI;
    const int64_t stride = gridDim.x;
    auto row0 = [&](int64_t i) { return (i * TPI + wt) * 32; };
    // a pass's row of this lane; past the batch its last row, which is not stored
    auto index_of = [&](int64_t i) -> int32_t {
        const int64_t t = row0(i) + lr;
        return IDX ? idx[t < B ? t : B - 1] : 0;
    };
    bool bad = false;   // an index out of range (its row reads row 0), raised at the end
    // the row's inputs 8 lh .. + 7 at p[0..1], 16 + 8 lh .. + 7 at p[4..5]
    auto row_at = [&](int64_t i, int32_t ix) {
        const int64_t t = row0(i) + lr;
        int64_t r = t < B ? t : B - 1;
        if constexpr (IDX) {
            const bool out = ix < 0 || ix >= n_rows;
            bad |= out;
            r = out ? 0 : ix;
        }
        return reinterpret_cast<const float4 *>(X + r * D_IN + 8 * lh);
    };
    constexpr int OFF[4] = {0, 1, 4, 5};

    int64_t it = blockIdx.x;
    float4 raw[4];
    {
        const float4 *p = row_at(it, index_of(it));
#pragma unroll
        for (int q = 0; q < 4; ++q) raw[q] = p[OFF[q]];
    }
    int32_t ix = index_of(it + stride);
    for (int j = threadIdx.x; j < H; j += 64 * S::WAVES) w2s[j] = W2[j];
    // the wave's weights, for its whole life: unit wu UW + 32 u + lr, inputs
    // 16 k + 8 lh .. + 7
    u4v w[NUT][2][3];
#pragma unroll
    for (int u = 0; u < NUT; ++u)
#pragma unroll
        for (int k = 0; k < 2; ++k) {
            const float *c = W1 + (16 * k + 8 * lh) * H + wu * S::UW + 32 * u + lr;
            uint32_t q[4][3];
#pragma unroll
            for (int t = 0; t < 4; ++t) split_pair(c[2 * t * H], c[(2 * t + 1) * H], q[t]);
#pragma unroll
            for (int p = 0; p < 3; ++p) w[u][k][p] = u4v{q[0][p], q[1][p], q[2][p], q[3][p]};
        }
    // parts of the current rows: word t of part p of half k holds inputs 2 t, 2 t + 1
    uint32_t xp[2][3][4];
#pragma unroll
    for (int k = 0; k < 2; ++k)
#pragma unroll
        for (int t = 0; t < 4; ++t) {
            const float4 v = raw[2 * k + t / 2];
            uint32_t q[3];
            if (t % 2 == 0) split_pair(v.x, v.y, q);
            else split_pair(v.z, v.w, q);
#pragma unroll
            for (int p = 0; p < 3; ++p) xp[k][p][t] = q[p];
        }
    {
        const float4 *p = row_at(it + stride, ix);
#pragma unroll
        for (int q = 0; q < 4; ++q) raw[q] = p[OFF[q]];
    }
    ix = index_of(it + 2 * stride);
    __syncthreads();   // w2s

    // eqs. 12-13 of register j of unit tile c: the lane's unit 8 (j / 4) + 4 lh + j % 4,
    // summed by j % 4. ReLU as an integer max on the bits: every negative float (-0
    // included) has a negative pattern and becomes +0, every positive one stays; one
    // instruction, where the float form costs two (a canonicalizing max first)
    auto unit = [&](const f16v &c, int j, const float4 (&w2)[4], float (&y)[4]) __attribute__((always_inline)) {
        const float4 q = w2[j / 4];
        const float ws[4] = {q.x, q.y, q.z, q.w};
        y[j % 4] = fmaf(__int_as_float(max(__float_as_int(c[j]), 0)), ws[j % 4], y[j % 4]);
    };
    auto load_w2 = [&](int u, float4 (&w2)[4]) __attribute__((always_inline)) {
#pragma unroll
        for (int q = 0; q < 4; ++q)
            w2[q] = *reinterpret_cast<const float4 *>(w2s + wu * S::UW + 32 * u + 8 * q + 4 * lh);
    };
    // a pass's outputs: the row's sum over the lane's units, then in 64 bits over the two
    // lanes of each wave and the waves (past two waves a half-wave takes half of them).
    // The 64 bits make up for k_forward's shorter chains: with 32 the outputs were 3-4 %
    // farther from exact than k_forward's, so they are 2 % nearer at 256 units and 15 % at
    // 1024, for 0.2-0.4 % of the time (eight sums a lane: 7 and 19 %, for 0.4-0.8 %).
    auto finish = [&](int64_t i, int par, const float (&y)[4]) __attribute__((always_inline)) {
        const int64_t r = row0(i) + lr;
        part[par][wave][lane] = (y[0] + y[1]) + (y[2] + y[3]);
        __syncthreads();   // a wave is at most one pass ahead: the other parity's words
        if (wu == 0) {
            constexpr int NQ = WPT == 2 ? 2 : WPT / 2;   // waves a lane adds
            const float *p = part[par][wt * WPT + (WPT == 2 ? 0 : lh * NQ)];
            double v = (double)p[lr] + (double)p[32 + lr];
#pragma unroll
            for (int q = 1; q < NQ; ++q) v += (double)p[64 * q + lr] + (double)p[64 * q + 32 + lr];
            if constexpr (WPT > 2) v = xadd32(v);
            if (lh == 0 && r >= 0 && r < B) ypred[r] = (float)v;
        }
    };

    // A value is computed where it stands: the compiler otherwise sinks what only the
    // next pass uses past the end of this one, out of the MFMAs' shadow.
    auto pin = [](auto &v) __attribute__((always_inline)) { asm volatile("" : "+v"(v)); };
    // the previous pass's last unit tile and its sums so far (before the first pass,
    // of rows below 0: not stored)
    f16v prev = {0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f};
    float y[4] = {0.f, 0.f, 0.f, 0.f};
    float4 w2[4];
    load_w2(NUT - 1, w2);
    int par = 0;
    for (; it < iters; it += stride) {
        const float4 *pn = row_at(it + 2 * stride, ix);   // the rows two passes on
        ix = index_of(it + 3 * stride);
        uint32_t nx[2][3][4];
        float yn[4] = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
        for (int u = 0; u < NUT; ++u) {
            constexpr int PX[6] = {2, 1, 0, 1, 0, 0}, PW[6] = {0, 1, 2, 0, 1, 0};
            f16v c = {0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f};
            float ra = 0.f, rb = 0.f;   // what a split has left
            // one MFMA and its share of the vector work at a time: Z1 of unit tile u (eq. 11,
            // the six part products smallest first); two registers of the tile before it a
            // slot; then the splits of the next rows
#pragma unroll
            for (int s = 0; s < 12; ++s) {
                const int q = s / 2, k = s % 2;
                c = mfma_bf16_32(w[u][k][PW[q]],
                                 u4v{xp[k][PX[q]][0], xp[k][PX[q]][1], xp[k][PX[q]][2], xp[k][PX[q]][3]}, c);
                if (s < 8) {
                    float(&ys)[4] = u == 0 ? y : yn;
                    unit(prev, 2 * s, w2, ys);
                    unit(prev, 2 * s + 1, w2, ys);
                    pin(ys[(2 * s) % 4]);
                    pin(ys[(2 * s + 1) % 4]);
                } else {   // a pair in two slots
                    const int pr = 2 * u + (s - 8) / 2, kk = pr / 4, t = pr % 4;
                    const float4 v = raw[pr / 2];
                    if (s % 2 == 0) {
                        ra = pr % 2 == 0 ? v.x : v.z;
                        rb = pr % 2 == 0 ? v.y : v.w;
                        nx[kk][0][t] = bf16_pair(ra, rb);
                        ra -= __uint_as_float(nx[kk][0][t] << 16);
                        rb -= __uint_as_float(nx[kk][0][t] & 0xFFFF0000u);
                        pin(ra);
                        pin(rb);
                    } else {
                        nx[kk][1][t] = bf16_pair(ra, rb);
                        ra -= __uint_as_float(nx[kk][1][t] << 16);
                        rb -= __uint_as_float(nx[kk][1][t] & 0xFFFF0000u);
                        nx[kk][2][t] = bf16_pair(ra, rb);
                        pin(nx[kk][1][t]);
                        pin(nx[kk][2][t]);
                    }
                }
                __builtin_amdgcn_sched_barrier(0);
            }
            // the inputs just split are free: the rows two passes on
            raw[u] = pn[OFF[u]];
            load_w2(u, w2);
            prev = c;
            __builtin_amdgcn_sched_barrier(0);
        }
        finish(it - stride, par, y);
        par ^= 1;
#pragma unroll
        for (int v = 0; v < 4; ++v) y[v] = yn[v];
#pragma unroll
        for (int k = 0; k < 2; ++k)
#pragma unroll
            for (int p = 0; p < 3; ++p)
#pragma unroll
                for (int t = 0; t < 4; ++t) xp[k][p][t] = nx[k][p][t];
    }
#pragma unroll
    for (int j = 0; j < 16; ++j) unit(prev, j, w2, y);
    finish(it - stride, par, y);
    if (IDX && bad)
        __hip_atomic_store(err, (int32_t)MLP_ERR_INDEX, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

template <int H>
static hipError_t launch_forward_wide(const Ctx &c, const float *X, int64_t n_rows,
                                      const int32_t *idx, int64_t B, float *ypred) {
    using S = WideShape<H>;
    const int64_t iters = ((B + 31) / 32 + S::TPI - 1) / S::TPI;
    const int64_t cap = (int64_t)S::WAVES_PER_SIMD * 4 / S::WAVES * (c.num_cu > 0 ? c.num_cu : 256);
    const int grid = (int)(iters < cap ? iters : cap);
    if (idx)
        hipLaunchKernelGGL((k_forward_wide<H, true>), dim3(grid), dim3(64 * S::WAVES), 0, c.stream, X, n_rows,
                           idx, B, c.W1, c.W2, ypred, &c.ctl->err);
    else
        hipLaunchKernelGGL((k_forward_wide<H, false>), dim3(grid), dim3(64 * S::WAVES), 0, c.stream, X, n_rows,
                           idx, B, c.W1, c.W2, ypred, &c.ctl->err);
    return hipGetLastError();
}

// Fewer rows leave k_forward_wide's longer passes a few waves (1,777 rows through 1024
// units: 5.4 us here, 6.7 there; 20,000 rows 11.0 and 10.7, 256 units 6.9 and 6.4), and
// at 64 and 128 units it is no faster (4M rows through 128: 183 and 188).
constexpr int64_t WIDE_ROWS = 16384;

hipError_t launch_forward(const Ctx &c, const float *X, int64_t n_rows, const int32_t *idx,
                          int64_t B, float *ypred) {
    if (B >= WIDE_ROWS) {
        switch (c.hidden) {
        case 256: return launch_forward_wide<256>(c, X, n_rows, idx, B, ypred);
        case 512: return launch_forward_wide<512>(c, X, n_rows, idx, B, ypred);
        case 1024: return launch_forward_wide<1024>(c, X, n_rows, idx, B, ypred);
        }
    }
    switch (c.hidden) {
    case 32: return launch_forward_h<32>(c, X, n_rows, idx, B, ypred);
    case 64: return launch_forward_h<64>(c, X, n_rows, idx, B, ypred);
    case 128: return launch_forward_h<128>(c, X, n_rows, idx, B, ypred);
    case 256: return launch_forward_h<256>(c, X, n_rows, idx, B, ypred);
    case 512: return launch_forward_h<512>(c, X, n_rows, idx, B, ypred);
    case 1024: return launch_forward_h<1024>(c, X, n_rows, idx, B, ypred);
    }
    return hipErrorInvalidValue;
}

}  // namespace mlp
