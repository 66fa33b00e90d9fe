// fff_wide.hip -- GENERIC mode for rows of whole 16-byte vectors (fff_wide.hpp): the fused descent of
// fff_kernels.hip with the row length a run-time value.  A group of 16, 32 or 64 lanes per token keeps x in
// registers, walks each tree (top levels from LDS, deeper rows by 16-byte loads) and accumulates the
// visited W_out rows, one row in flight ahead of the FMAs.
//
// What bounds it: as the fused descent, the D+1 dependent row gathers.  Against the kernel it stands in
// for (one wave per token, an element per lane and load; us, buffers rotating): hidden 512, depth 10,
// 9001 tokens, bf16 126.8 -> 16.2; hidden 512, depth 9, 65536 tokens, fp32 808 -> 132; hidden 2048,
// depth 9, 100 / 4001 tokens, bf16 124 / 245 -> 9.6 / 21.6; hidden 200, depth 4, 1 / 16384 tokens, fp32
// 9.6 / 44.1 -> 9.1 / 12.0.
#include "fff_common.hpp"
#include "fff_device.hpp"
#include "fff_internal.hpp"
#include "fff_wide.hpp"

#include <hip/hip_runtime.h>

namespace fff {

namespace {

constexpr int WIDE_BLOCK = 256;

// LayerNorm of a token in the wide layout: as layer_norm_regs, the vectors past the row kept at zero.
template <int LANES, int NV, bool WBF>
__device__ __forceinline__ void wide_layer_norm(float* f, const Params& p, int rowv, int sl) {
    constexpr int EV = WBF ? 8 : 4, E = NV * EV;
    const float H = float(p.hidden);
    float s = 0.0f;
#pragma unroll
    for (int i = 0; i < E; ++i) s += f[i];
    const float mean = group_sum<LANES>(s) / H;
    float q = 0.0f;
#pragma unroll
    for (int c = 0; c < NV; ++c)
#pragma unroll
        for (int e = 0; e < EV; ++e) {
            float& v = f[c * EV + e];
            v = c * LANES + sl < rowv ? v - mean : 0.0f;
            q = __builtin_fmaf(v, v, q);
        }
    const float rstd = 1.0f / sqrtf(group_sum<LANES>(q) / H + p.norm_eps);
#pragma unroll
    for (int c = 0; c < NV; ++c) {
        const int v = c * LANES + sl;
        if (v >= rowv) continue;
#pragma unroll
        for (int e = 0; e < EV; ++e)
            f[c * EV + e] = __builtin_fmaf(f[c * EV + e] * rstd, p.gamma ? p.gamma[v * EV + e] : 1.0f,
                                           p.beta ? p.beta[v * EV + e] : 0.0f);
    }
}

// XDOT: bf16 x and W, no LayerNorm (x kept as bf16 pairs); otherwise x in fp32 registers, whatever
// its storage.  LDS: [T][2^K - 1][2][LANES NV] vectors, W_in row then W_out row, zeros past the row.
template <int LANES, int NV, bool XDOT, bool WBF>
__global__ __launch_bounds__(WIDE_BLOCK) void wide_kernel(Params p, int rowv) {
    using S = Shape<LANES, NV, XDOT, WBF>;
    constexpr int WAVES = WIDE_BLOCK / 64;
    extern __shared__ uint4 lds_rows[];
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const int sl = lane % LANES, sub = lane / LANES;
    const int T = p.n_trees, D = p.depth, K = p.lds_levels, Nk = (1 << K) - 1;
    const int KD = K < D + 1 ? K : D + 1;
    const int64_t N = p.n_nodes;
    const uint32_t rowb = uint32_t(rowv) * 16;
    WideRows<LANES, NV> win, wout;
    const int64_t wbytes = int64_t(T) * N * rowb;
    win.init(p.w_in, wbytes, rowv, sl);
    wout.init(p.w_out, wbytes, rowv, sl);
    if (K > 0) {
        for (int i = threadIdx.x; i < T * Nk * 2 * S::ROWV; i += WIDE_BLOCK) {
            const int v = i % S::ROWV, r = i / S::ROWV;
            const int m = r & 1, tn = r >> 1, t = tn / Nk, node = tn - t * Nk;
            const uint4* src = static_cast<const uint4*>(m ? p.w_out : p.w_in) + (t * N + node) * rowv;
            lds_rows[i] = v < rowv ? src[v] : make_uint4(0, 0, 0, 0);
        }
        __syncthreads();
    }
    const int64_t groups = (p.n_tokens + S::TPW - 1) / S::TPW;
    for (int64_t g = int64_t(blockIdx.x) * WAVES + wave; g < groups; g += int64_t(gridDim.x) * WAVES) {
        const int64_t slot = g * S::TPW + sub;
        const bool valid = slot < p.n_tokens;
        const int64_t tok = valid ? slot : p.n_tokens - 1;  // idle groups redo the last token, store nothing
        XRegs<LANES, NV, XDOT, WBF> xr;
        if constexpr (XDOT) {
#pragma unroll
            for (int c = 0; c < NV; ++c) {
                const int v = c * LANES + sl;
                xr.v[c] = v < rowv ? static_cast<const uint4*>(p.x)[tok * rowv + v] : make_uint4(0, 0, 0, 0);
            }
        } else {
            wide_load_f32<LANES, NV, WBF>(xr.f, p.x, p.x_bf16, tok, rowv, sl);
            if (p.norm) wide_layer_norm<LANES, NV, WBF>(xr.f, p, rowv, sl);
        }
        float acc[S::E];
#pragma unroll
        for (int e = 0; e < S::E; ++e) acc[e] = 0.0f;
        for (int t = 0; t < T; ++t) {
            const uint4* lrows = lds_rows + t * Nk * 2 * S::ROWV + sl;
            const uint32_t tree = uint32_t(t) * uint32_t(N) * rowb;
            LevelRegs<LANES> lv;
            lv.clear();
            uint32_t n = 0;
            auto visit = [&](int l, const uint4* w) {
                const float logit = group_sum<LANES>(wide_dot<NV, XDOT, WBF>(xr, w));
                lv.park(l, sl, logit);
                if (l < D) n = 2 * n + 1 + (logit > 0.0f ? 1u : 0u);
            };
            for (int l = 0; l < KD; ++l) {
                uint4 w[NV];
                const uint4* row = lrows + n * 2 * S::ROWV;
#pragma unroll
                for (int c = 0; c < NV; ++c) w[c] = row[c * LANES];
                visit(l, w);
            }
            for (int l = KD; l <= D; ++l) {
                uint4 w[NV];
                win.load(tree + n * rowb, w);
                visit(l, w);
            }
            const uint32_t leaf1 = n + 1;
            LevelRegs<LANES> av;
#pragma unroll
            for (int r = 0; r < LevelRegs<LANES>::NR; ++r) av.v[r] = activation(lv.v[r], p.act);
            if ((p.nodes_out || p.logits_out) && valid)
                write_records<LANES>(p.nodes_out, p.logits_out, p, lv, leaf1, tok, t, sl);
            auto node = [&](int l) { return (leaf1 >> (D - l)) - 1; };
            // the W_out rows of the path, one in flight ahead of the FMAs (as emit_levels)
            uint4 cur[NV], nxt[NV];
            float a_cur = 0.0f, a_nxt = 0.0f;
            auto load = [&](uint4* dst, float& a, int l) {
                wout.load(tree + node(l) * rowb, dst);
                a = av.get(l, lane);
            };
            if (KD <= D) load(cur, a_cur, KD);
            __builtin_amdgcn_sched_barrier(0);
            for (int l = 0; l < KD; ++l) {
                uint4 w[NV];
                const uint4* row = lrows + node(l) * 2 * S::ROWV + S::ROWV;
#pragma unroll
                for (int c = 0; c < NV; ++c) w[c] = row[c * LANES];
                axpy<NV, WBF>(acc, av.get(l, lane), w);
            }
            if (KD <= D)
                for (int l = KD;; l += 2) {
                    load(nxt, a_nxt, l + 1 <= D ? l + 1 : D);
                    __builtin_amdgcn_sched_barrier(0);
                    axpy<NV, WBF>(acc, a_cur, cur);
                    if (l + 1 > D) break;
                    load(cur, a_cur, l + 2 <= D ? l + 2 : D);
                    __builtin_amdgcn_sched_barrier(0);
                    axpy<NV, WBF>(acc, a_nxt, nxt);
                    if (l + 2 > D) break;
                }
        }
        const bool res = p.out_mode == OUT_RESIDUAL, accum = p.out_mode == OUT_ACCUMULATE;
        if (valid)
            wide_store<LANES, NV, WBF>(p.y, p.y_bf16, res ? p.x : accum ? p.y : nullptr, res ? p.x_bf16 : p.y_bf16, acc,
                                       tok, rowv, sl);
    }
}

}  // namespace

bool wide_plan(const Params& p, WidePlan* w) {
    const int rowv = wide_vecs(p.hidden, p.w_bf16, int64_t(p.n_trees) * p.n_nodes);
    if (!rowv) return false;
    w->rowv = rowv;
    auto fill = [&](auto lanes, auto nv, auto xdot, auto wbf) {
        constexpr int L = decltype(lanes)::value, NV = decltype(nv)::value;
        w->lanes = L;
        w->row_vecs = L * NV;
        w->block = WIDE_BLOCK;
        w->kernel = reinterpret_cast<const void*>(&wide_kernel<L, NV, decltype(xdot)::value, decltype(wbf)::value>);
        return true;
    };
    using std::true_type, std::false_type;
    if (!p.w_bf16) return wide_class<false>(rowv, [&](auto l, auto v) { return fill(l, v, false_type{}, false_type{}); });
    if (p.x_bf16 && !p.norm) return wide_class<false>(rowv, [&](auto l, auto v) { return fill(l, v, true_type{}, true_type{}); });
    return wide_class<true>(rowv, [&](auto l, auto v) { return fill(l, v, false_type{}, true_type{}); });
}

}  // namespace fff
