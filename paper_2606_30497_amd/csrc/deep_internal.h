// deep_internal.h -- shared declarations of the L-hidden-layer path: its context,
// the batch gather and the batch loss (deep.hip, deep_panel.hip).
#pragma once

#include <hip/hip_runtime.h>

#include <stdint.h>

#include "bf16x3.h"
#include "mlp.h"
#include "mlp_internal.h"

namespace mlp {

constexpr int DEEP_MAX_LAYERS = 8;
constexpr int PANEL_MAX_H = 256;      // widest net of the panel path
constexpr int PANEL_WGS_MAX = 512;    // most workgroups of a panel launch (dw_o partials)

struct DeepCtx {
    int hidden = 0, layers = 0;
    int64_t max_batch = 0, np = 0;
    float *params = nullptr;
    Control *ctl = nullptr;
    float *Xb = nullptr, *Yb = nullptr, *sq = nullptr;
    float *H = nullptr;       // [layers][max_batch x hidden]
    float *G[2] = {nullptr, nullptr};
    float *part = nullptr;    // gradient partials, segment s at part_off[s] (plan of max_batch)
    int64_t part_off[DEEP_MAX_LAYERS + 1] = {};
    // panel path (null: the workspace does not hold it, or the net is wider)
    u4v *frag = nullptr;      // split weights in operand order (panel_frag_words)
    float *dwo_part = nullptr;             // [PANEL_WGS_MAX][hidden]
    float *PG[DEEP_MAX_LAYERS] = {};       // G_l at PG[l - 1], [max_batch x hidden]
    hipStream_t stream = nullptr;
    bool profile = false, ev_valid = false;
    hipEvent_t ev0 = nullptr, ev1 = nullptr;
};

// Sixteen zero bytes in device memory: a lane whose value lies outside its
// operand loads these instead. The choice is made on the address, before the
// load, and the loaded registers are not touched again until they are written
// to LDS. (A load under a lane condition compiles to a branch and an immediate
// wait for that load; a select of zero after the load is consumed, and so
// waited for, wherever the scheduler places it, often among the MFMAs of an
// earlier chunk. Either way the next chunks' loads stop overlapping the current
// chunk's MFMAs.)
static __device__ __attribute__((aligned(16))) float g_zero16[4] = {0.f, 0.f, 0.f, 0.f};

__device__ __forceinline__ float4 ld4(bool ok, const float *p) {
    return *reinterpret_cast<const float4 *>(ok ? p : g_zero16);
}
__device__ __forceinline__ float ld1(bool ok, const float *p) { return *(ok ? p : g_zero16); }

// Xb[t][k] = X[r_t][k], Yb[t] = Y[r_t], r_t = idx[off + t] (or off + t);
// out-of-range rows read row 0 and raise the sticky error.
struct GatherArgs {
    const float *X, *Y;
    int64_t n_rows;
    const int32_t *idx;
    int64_t off, nb;
    float *Xb, *Yb;
    int32_t *err;
};

// Element e of the gather: float4 e % 8 of batch row e / 8.
__device__ __forceinline__ void gather_one(const GatherArgs &g, int64_t e) {
    if (e >= g.nb * (D_IN / 4)) return;
    const int64_t t = e / (D_IN / 4);
    const int q = (int)(e % (D_IN / 4));
    int64_t r = g.idx ? (int64_t)g.idx[g.off + t] : g.off + t;
    if (r < 0 || r >= g.n_rows) {
        __hip_atomic_store(g.err, (int32_t)MLP_ERR_INDEX, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        r = 0;
    }
    reinterpret_cast<float4 *>(g.Xb)[t * (D_IN / 4) + q] =
        reinterpret_cast<const float4 *>(g.X)[r * (D_IN / 4) + q];
    if (q == 0) g.Yb[t] = g.Y ? g.Y[r] : 0.0f;
}

// The batch loss (eq. 14) of nb squared residuals by one workgroup of 256
// threads: thread i sums rows i, i + 256, ... (32 loads in flight), then a fixed
// binary tree; step and epoch loss as in the one-layer paths.
__device__ __forceinline__ void batch_loss(const float *sq, int64_t nb, const ReduceArgs &ra) {
    constexpr int U = 32;
    __shared__ float red[256];
    const int i = threadIdx.x;
    float v = 0.0f;
    for (int64_t t0 = i; t0 < nb; t0 += 256 * U) {
        float x[U];
#pragma unroll
        for (int j = 0; j < U; ++j) {
            const int64_t t = t0 + 256 * j;
            x[j] = sq[t < nb ? t : nb - 1];
        }
#pragma unroll
        for (int j = 0; j < U; ++j)
            if (t0 + 256 * j < nb) v += x[j];
    }
    red[i] = v;
    __syncthreads();
    for (int w = 128; w >= 1; w >>= 1) {
        if (i < w) red[i] += red[i + w];
        __syncthreads();
    }
    if (i == 0) record_loss(ra, red[0]);
}

inline int64_t deep_np(int h, int L) { return (int64_t)D_IN * h + (int64_t)(L - 1) * h * h + h; }
inline int64_t layer_offset(int h, int l) {   // W_l, l = 1..L; w_o at l = L + 1
    return l == 1 ? 0 : (int64_t)D_IN * h + (int64_t)(l - 2) * h * h;
}
inline size_t pad64f(size_t n) { return (n + 63) / 64 * 64; }
inline unsigned blocks_of(int64_t n, int per) { return (unsigned)((n + per - 1) / per); }
int64_t seg_chunks(int h, int L, int64_t nb, int s);

// ---- panel path (deep_panel.hip) ----
size_t panel_ws_floats(int h, int L, int64_t mb);
void panel_carve(DeepCtx &c, float *p);
hipError_t panel_forward(const DeepCtx &c, const float *X, int64_t n_rows, const int32_t *idx,
                         int64_t B, float *ypred);
bool panel_pays(const DeepCtx &c, int64_t nb);   // steps of nb rows take the panel path
hipError_t panel_step(const DeepCtx &c, const GatherArgs &rows, int64_t nb, const ReduceArgs &ra,
                      float *dparams, bool ready, const GatherArgs *next);

}  // namespace mlp
