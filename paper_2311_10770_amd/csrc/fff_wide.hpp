// fff_wide.hpp -- the register layout of a hidden size without kernels of its own: a row of whole
// 16-byte vectors (hidden a multiple of 8 with bf16 W, of 4 with fp32 W) held by LANES lanes of NV
// vectors, LANES NV at least the row's vectors.  Lane sl owns vectors c LANES + sl as in
// fff_common.hpp; those past the row are zeros, never loaded and never stored.
#pragma once

#include "fff_common.hpp"

#include <type_traits>

namespace fff {

constexpr uint32_t WIDE_NO_VEC = 0x80000000u;  // past the end of any matrix below 2^31 bytes
typedef uint32_t wide_u4 __attribute__((ext_vector_type(4)));

// One weight matrix, rows through a buffer resource: an offset past its end reads zeros without a
// memory access, so a lane's vectors past the row need no branch.
template <int LANES, int NV>
struct WideRows {
    __amdgpu_buffer_rsrc_t rsrc;
    uint32_t off[NV];  // this lane's vectors within a row, bytes
    __device__ void init(const void* w, int64_t bytes, int rowv, int sl) {
        rsrc = __builtin_amdgcn_make_buffer_rsrc(const_cast<void*>(w), 0, int(bytes), 0x00020000);
        set_lane(rowv, sl);
    }
    __device__ void set_lane(int rowv, int sl) {
#pragma unroll
        for (int c = 0; c < NV; ++c) {
            const int v = c * LANES + sl;
            off[c] = v < rowv ? uint32_t(v) * 16 : WIDE_NO_VEC;
        }
    }
    // row: the row's first byte
    __device__ void load(uint32_t row, uint4* dst) const {
#pragma unroll
        for (int c = 0; c < NV; ++c) {
            const wide_u4 v = __builtin_amdgcn_raw_buffer_load_b128(rsrc, int(off[c] + row), 0, 0);
            dst[c] = make_uint4(v[0], v[1], v[2], v[3]);
        }
    }
};

// Token tok of a [B, 4 EV-vector] matrix into fp32 registers (EV values per vector), zeros past the row.
template <int LANES, int NV, bool WBF>
__device__ __forceinline__ void wide_load_f32(float* f, const void* x, bool xbf, int64_t tok, int rowv, int sl) {
    constexpr int EV = WBF ? 8 : 4;
#pragma unroll
    for (int c = 0; c < NV; ++c) {
        const int v = c * LANES + sl;
        const int64_t e = (tok * rowv + v) * EV;
#pragma unroll
        for (int h = 0; h < EV / 4; ++h) {
            float4 a = make_float4(0.f, 0.f, 0.f, 0.f);
            if (v < rowv) {
                if (xbf) {
                    const uint2 u = *reinterpret_cast<const uint2*>(static_cast<const uint16_t*>(x) + e + 4 * h);
                    a = make_float4(bf16_lo(u.x), bf16_hi(u.x), bf16_lo(u.y), bf16_hi(u.y));
                } else {
                    a = *reinterpret_cast<const float4*>(static_cast<const float*>(x) + e + 4 * h);
                }
            }
            f[c * EV + 4 * h + 0] = a.x; f[c * EV + 4 * h + 1] = a.y;
            f[c * EV + 4 * h + 2] = a.z; f[c * EV + 4 * h + 3] = a.w;
        }
    }
}

// Stores one token's slice (fp32 or bf16 rows), after adding the fp32 or bf16 row src where there is one.
template <int LANES, int NV, bool WBF>
__device__ __forceinline__ void wide_store(void* y, bool ybf, const void* src, bool sbf, const float* acc, int64_t tok,
                                           int rowv, int sl) {
    constexpr int EV = WBF ? 8 : 4;
#pragma unroll
    for (int c = 0; c < NV; ++c) {
        const int v = c * LANES + sl;
        if (v >= rowv) continue;
        const int64_t e = (tok * rowv + v) * EV;
        float o[EV];
#pragma unroll
        for (int i = 0; i < EV; ++i) o[i] = acc[c * EV + i];
        if (src) {
#pragma unroll
            for (int h = 0; h < EV; h += 4) {
                if (sbf) {
                    const uint2 u = *reinterpret_cast<const uint2*>(static_cast<const uint16_t*>(src) + e + h);
                    o[h] += bf16_lo(u.x); o[h + 1] += bf16_hi(u.x); o[h + 2] += bf16_lo(u.y); o[h + 3] += bf16_hi(u.y);
                } else {
                    const float4 u = *reinterpret_cast<const float4*>(static_cast<const float*>(src) + e + h);
                    o[h] += u.x; o[h + 1] += u.y; o[h + 2] += u.z; o[h + 3] += u.w;
                }
            }
        }
#pragma unroll
        for (int h = 0; h < EV; h += 4) {
            if (ybf)
                *reinterpret_cast<uint2*>(static_cast<uint16_t*>(y) + e + h) =
                    make_uint2(pack_bf16x2(o[h], o[h + 1]), pack_bf16x2(o[h + 2], o[h + 3]));
            else
                *reinterpret_cast<float4*>(static_cast<float*>(y) + e + h) = make_float4(o[h], o[h + 1], o[h + 2], o[h + 3]);
        }
    }
}

// This lane's part of the dot product of a row in registers (x, in the layout of Shape<LANES, NV, XDOT, WBF>)
// with a W row: a sum per four elements (eight bf16 x), the sums added in pairs.  One chain over all of a
// lane's elements (up to 64) loses against a wave per token, whose lanes hold one in 64: hidden 512, fp32 x
// with bf16 W, logits off by 1.16e-7 (relative, 2-norm) so, 8.5e-8 there, 8.2e-8 here.
template <int NV, bool XDOT, bool WBF, class X>
__device__ __forceinline__ float wide_dot(const X& x, const uint4* w) {
    float s[NV], zero = 0.0f;
#pragma unroll
    for (int c = 0; c < NV; ++c) {
        float h[2] = {zero, zero};
#pragma unroll
        for (int j = 0; j < 4; ++j) {
            const uint32_t u = word(w[c], j);
            if constexpr (XDOT) {
                h[0] = dot2_bf16(word(x.v[c], j), u, h[0]);
            } else if constexpr (WBF) {
                h[j / 2] = __builtin_fmaf(x.f[c * 8 + 2 * j], bf16_lo(u), h[j / 2]);
                h[j / 2] = __builtin_fmaf(x.f[c * 8 + 2 * j + 1], bf16_hi(u), h[j / 2]);
            } else {
                h[0] = __builtin_fmaf(x.f[c * 4 + j], __uint_as_float(u), h[0]);
            }
        }
        s[c] = WBF && !XDOT ? h[0] + h[1] : h[0];
        // the sums in order, each while the vectors after it arrive (interleaved, most wait for the last one):
        // the next one starts from a zero that this one's end hands out
        asm volatile("" : "+v"(s[c]), "+v"(zero));
    }
#pragma unroll
    for (int d = 1; d < NV; d *= 2)
#pragma unroll
        for (int c = 0; c + d < NV; c += 2 * d) s[c] += s[c + d];
    return s[0];
}

// The (LANES, NV) classes: f(lanes, nv), integral constants, for the smallest that holds rowv vectors
// (at most WIDE_MAX_VECS).  Sixteen lanes up to six vectors each (heavy layouts, 16 fp32 registers per
// vector and lane besides the row: up to four), then 32 and 64.  Two waves per SIMD or more, except rows
// past 384 vectors of bf16 W with x or dy widened: one (296 registers; 332 in the backward).
constexpr int WIDE_MAX_VECS = 512;
template <bool HEAVY, class F>
auto wide_class(int rowv, F&& f) {
    using std::integral_constant;
    if (rowv <= 32) return f(integral_constant<int, 16>{}, integral_constant<int, 2>{});
    if (rowv <= 64) return f(integral_constant<int, 16>{}, integral_constant<int, 4>{});
    if constexpr (!HEAVY)
        if (rowv <= 96) return f(integral_constant<int, 16>{}, integral_constant<int, 6>{});
    if (rowv <= 128) return f(integral_constant<int, 32>{}, integral_constant<int, 4>{});
    if constexpr (!HEAVY)
        if (rowv <= 192) return f(integral_constant<int, 32>{}, integral_constant<int, 6>{});
    if (rowv <= 256) return f(integral_constant<int, 64>{}, integral_constant<int, 4>{});
    if (rowv <= 384) return f(integral_constant<int, 64>{}, integral_constant<int, 6>{});
    return f(integral_constant<int, 64>{}, integral_constant<int, 8>{});
}

// Vectors of a W row, or 0 where the layout does not apply.
inline int wide_vecs(int64_t hidden, bool w_bf16, int64_t w_rows) {
    const int ev = w_bf16 ? 8 : 4;
    if (hidden % ev || hidden / ev > WIDE_MAX_VECS || w_rows * hidden * (w_bf16 ? 2 : 4) >= (int64_t(1) << 31)) return 0;
    return int(hidden / ev);
}

}  // namespace fff
