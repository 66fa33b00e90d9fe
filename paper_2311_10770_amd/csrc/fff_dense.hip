// fff_dense.hip -- the dense form of TILED mode (bf16 weights, one tree, at most
// twelve levels, large batches): the walk and the output accumulation as dense
// MFMA products over small subtrees.
//
// A token walks one node per level, but the logits of ALL nodes of a subtree of
// up to six levels (63 nodes) are one 64-column product x W_in[subtree]^T, which
// the matrix cores do in less time than the token's rows take to arrive.  So the
// tree is cut at level s:
//   top pass (dense_top_kernel): the logits of levels 0 .. s-1 for tokens in
//     order; each token descends through its row of logits in LDS, and leaves
//     its activations, its node at level s (the group) and, per workgroup, how
//     many of its tokens went to each group;
//   subtree pass (dense_sub_kernel): a workgroup takes up to DS_TOK (384) tokens
//     of one group (found from those counts, in token order: no atomics), gathers
//     their x rows, does the same for levels s .. D of the group's subtree, and then
//     forms the tokens' whole output
//         Y[tokens, H] = A[tokens, s + 63] W_out[s ancestors and 63 subtree nodes, H],
//     A holding a token's activation at its visited nodes and zeros elsewhere.
// With D < 6 there is no top pass: the one group is the whole tree.
//
// Every bf16 x bf16 product is exact and the sums are fp32, but in chains of hidden / 32 matrix products:
// at hidden 768 the logits are off by 1.57e-7 (relative, 2-norm) where the walk's lanes end at 6.9e-8.
// That is far below what bf16 outputs show (1.66e-3 either way); a call that asks for the logits
// themselves takes the walk.  An activation is split into two bf16 parts
// (relative error 2^-17, as in the leaf tiles of a bf16 y).  A row's result does not depend on the
// other rows of its tile, so the output bits do not depend on how tokens fall into tiles.
//
// What bounds it: HBM and MALL traffic, x twice and y once.  At 65536 tokens, depth 11, hidden 768,
// buffers rotating so that nothing is warm: top pass 24 us (19 where no dirty rows of y are being
// written back), subtree pass 52 us, of which 16 gather x (6.3 TB/s), 17 store y (5.9 TB/s), 6
// look the tokens up, 2 evaluate the activations and 3 transpose W_out; 81.6 us per forward against
// 94.7 us for the walk and the leaf tiles.  First forms of the subtree pass: four waves per
// workgroup, x rows loaded straight into the MFMA operand layout, W_out fetched one block ahead of
// its use: 94 us (a quad of lanes then reads four rows, and the loads waited for the stores issued
// before them); x through LDS, three workgroups per CU: 71 us.
#include "fff_common.hpp"
#include "fff_device.hpp"
#include "fff_gemm.hpp"
#include "fff_internal.hpp"

#include <hip/hip_runtime.h>

#include <algorithm>
#include <type_traits>

namespace fff {

namespace {

// Top pass: 128 tokens per workgroup of four waves, two 16-token tiles each.  Subtree pass: eight
// waves of up to three tiles.
constexpr int DT_WAVES = 4, DT_MT = 2, DT_TOK = 16 * DT_WAVES * DT_MT;
constexpr int DS_WAVES = 8, DS_THREADS = 64 * DS_WAVES, DS_MT = 3, DS_TOK = 16 * DS_WAVES * DS_MT;
constexpr int DN_MAX_LEVELS = 6;             // levels of a subtree: at most 64 columns
constexpr int DN_REC = 8;                    // floats per token of the top pass's activations
constexpr int DN_MAX_HIDDEN = 1024;          // W_out of a subtree fits LDS
constexpr int DN_SC = 65;                    // floats per token of the logits in LDS (odd: lanes read one column)
// Most tokens per pair of passes: however they fall into 64 groups, workgroups of DS_TOK tokens are no more
// than a round of 256 CUs (below).  Larger batches: as many equal chunks as it takes.
constexpr int64_t DN_CHUNK = 69632;
static_assert(DN_CHUNK / DS_TOK + (1 << DN_MAX_LEVELS) <= 256, "one round of subtree workgroups");

// What the two passes hand over, carved from the workspace.
struct DenseArgs {
    float* rec;        // [B, DN_REC] activations of levels 0 .. s-1
    uint8_t* gid;      // [B] the token's node at level s, counted within the level
    uint8_t* hist;     // [2^s, hist_ld] tokens per (group, top workgroup)
    int32_t hist_ld;   // top workgroups, rounded up to 16
    int32_t top_wgs;
    int32_t s;         // levels of the top pass (0: none)
    int32_t levels;    // levels of the subtree pass
    int32_t item;      // most tokens of a subtree workgroup (s == 0), or the least such bound
    int32_t round;     // subtree workgroups that run at once
    float* act;        // [B, DN_REC] activations of levels s .. D and, last, the subtree column of the leaf
};

// Steps of the logit loop: 64 elements of every x row and of the subtree's W_in rows (128 bytes each),
// written straight to LDS (lds_dma16), the next step's in flight while one is multiplied.  The
// 16-byte vectors of LDS row r are stored in the order c ^ swz(r % 16) (free of bank conflicts).
template <int NT, int MT, int WAVES> struct DStep {
    static constexpr int KC = 64, ROW = 2 * KC;
    static constexpr int XBYTES = WAVES * MT * 16 * ROW, STAGE = XBYTES + NT * 16 * ROW;
    static constexpr int LX = MT * 2;              // x loads per wave: eight rows each
    static constexpr int WLOADS = NT * 2;          // W_in loads of the workgroup, likewise
    static constexpr int LW = WLOADS >= WAVES ? WLOADS / WAVES : 1;
    static constexpr int S = 2;                    // stages
};

// Heap node of column c of the subtree of group g at level s: column 1 is its root, the children of
// c are 2c and 2c + 1; unused columns (0, and past the subtree) stand for the root.
__device__ __forceinline__ int64_t dn_node(int c, int g, int s, int levels) {
    if (c < 1 || c >= (1 << levels)) c = 1;
    const int l = 31 - __builtin_clz(uint32_t(c));
    return (((int64_t(1) << s) + g) << l) + (c - (1 << l)) - 1;
}

// Two values in two bf16 parts each: hi = bf16(v), mid = bf16(v - hi).
__device__ __forceinline__ void dn_split2(float a, float b, uint32_t& hi, uint32_t& mid) {
    hi = pack_bf16x2(a, b);
    mid = pack_bf16x2(a - bf16_lo(hi), b - bf16_hi(hi));
}

// f(integral_constant<n>) with n = min(tiles, MT), nothing for no tiles.
template <int MT, class F>
__device__ __forceinline__ void dn_tiles(int tiles, F&& f) {
    if (tiles >= MT) f(std::integral_constant<int, MT>{});
    else if constexpr (MT > 1) dn_tiles<MT - 1>(tiles, f);
}

// acc[mt][j] = logits of the wave's tiles at columns 16 j + n of the subtree of `levels` levels
// under node g of level s.  Tile mt of wave w is tile w + WAVES mt of the workgroup, its tokens
// list[16 (w + WAVES mt) + 0 .. 15] (list holds a token for every row of the tiles of every wave); the
// wave's first `tiles` tiles are computed.  lds: S stages.  Ends with every wave past its last read of
// the stages.
template <int NT, int MT, int WAVES>
__device__ __forceinline__ void dn_logits(const Params& p, int g, int s, int levels, const int32_t* list, int tiles,
                                          unsigned char* lds, tile_v4f (&acc)[MT][NT]) {
    using S = DStep<NT, MT, WAVES>;
    const int tid = threadIdx.x, lane = tid & 63, n = lane & 15, q = lane >> 4;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int64_t H = p.hidden;
    const int steps = p.hidden / S::KC;
    const uint32_t lds0 = uint32_t(uintptr_t((__attribute__((address_space(3))) unsigned char*)lds));
    // x: this wave's own rows, eight lanes each
    const char* gx[S::LX];
#pragma unroll
    for (int i = 0; i < S::LX; ++i) {
        const int r = 8 * (i & 1) + (lane >> 3);
        gx[i] = static_cast<const char*>(p.x) + int64_t(list[16 * (wave + WAVES * (i >> 1)) + r]) * H * 2 +
                ((lane & 7) ^ swz(r)) * 16;
    }
    // W_in: eight lanes per row; with fewer loads than waves some waves repeat one
    const char* gw[S::LW];
#pragma unroll
    for (int i = 0; i < S::LW; ++i) {
        const int r = ((wave * S::LW + i) % S::WLOADS) * 8 + (lane >> 3);
        gw[i] = static_cast<const char*>(p.w_in) + dn_node(r, g, s, levels) * H * 2 + ((lane & 7) ^ swz(r & 15)) * 16;
    }
    auto issue = [&](int step) {
        const uint32_t st = lds0 + uint32_t(step % S::S) * S::STAGE;
#pragma unroll
        for (int i = 0; i < S::LX; ++i)
            if ((i >> 1) < tiles) lds_dma16(gx[i] + step * S::ROW, st + (wave * S::LX + i) * 1024);
#pragma unroll
        for (int i = 0; i < S::LW; ++i)
            lds_dma16(gw[i] + step * S::ROW, st + S::XBYTES + ((wave * S::LW + i) % S::WLOADS) * 1024);
    };
#pragma unroll
    for (int mt = 0; mt < MT; ++mt)
#pragma unroll
        for (int j = 0; j < NT; ++j) acc[mt][j] = tile_v4f{0.f, 0.f, 0.f, 0.f};
    const int key = swz(n);
    auto compute = [&](const unsigned char* st, auto mts) {
        constexpr int M = decltype(mts)::value;
        const unsigned char* const xr = st + (wave * MT * 16 + n) * S::ROW;
        const unsigned char* const wr = st + S::XBYTES + n * S::ROW;
#pragma unroll
        for (int k = 0; k < S::KC / 32; ++k) {
            const int off = ((4 * k + q) ^ key) * 16;
            bf16x8_t fa[M];
#pragma unroll
            for (int mt = 0; mt < M; ++mt)
                fa[mt] = __builtin_bit_cast(bf16x8_t, *reinterpret_cast<const uint4*>(xr + mt * 16 * S::ROW + off));
#pragma unroll
            for (int j = 0; j < NT; ++j) {
                const bf16x8_t fb = __builtin_bit_cast(bf16x8_t, *reinterpret_cast<const uint4*>(wr + 16 * j * S::ROW + off));
#pragma unroll
                for (int mt = 0; mt < M; ++mt)
                    acc[mt][j] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(fa[mt], fb, acc[mt][j], 0, 0, 0);
            }
        }
    };
    issue(0);
    for (int k = 0; k < steps; ++k) {
        wait_vmem<0>();
        __syncthreads();  // step k is in LDS for every wave; every wave is done with step k - 1
        if (k + 1 < steps) issue(k + 1);
        const unsigned char* const st = lds + (k % S::S) * S::STAGE;
        dn_tiles<MT>(tiles, [&](auto m) { compute(st, m); });  // wave-uniform
    }
    __syncthreads();
}

// A wave's logits to its LDS scratch (16 MT rows of DN_SC floats).
template <int MT, int NT>
__device__ __forceinline__ void dn_put_logits(const tile_v4f (&acc)[MT][NT], float* sc) {
    const int lane = threadIdx.x & 63, n = lane & 15, q = lane >> 4;
#pragma unroll
    for (int mt = 0; mt < MT; ++mt)
#pragma unroll
        for (int j = 0; j < NT; ++j)
#pragma unroll
            for (int r = 0; r < 4; ++r) sc[(mt * 16 + 4 * q + r) * DN_SC + 16 * j + n] = acc[mt][j][r];
}

// Orders a wave's LDS accesses before it against those after.
__device__ __forceinline__ void dn_wave_sync() {
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

// One token's descent through its row of logits: lg[l] of the subtree's levels; returns the column
// of the last node, one level further (branch of the last logit included) when `out` is set.
__device__ __forceinline__ int dn_descend(const float* row, int levels, bool out, float (&lg)[DN_MAX_LEVELS]) {
    int c = 1;
#pragma unroll
    for (int l = 0; l < DN_MAX_LEVELS; ++l) {
        lg[l] = 0.0f;
        if (l < levels) {
            lg[l] = row[c];
            if (l + 1 < levels || out) c = 2 * c + (lg[l] > 0.0f ? 1 : 0);
        }
    }
    return c;
}

__device__ __forceinline__ void dn_record(const Params& p, int64_t tok, int level, int64_t node) {
    p.nodes_out[tok * (p.depth + 1) + level] = int32_t(node);
}

// ----------------------------------------------------------------------------
// top pass
// ----------------------------------------------------------------------------

// LDS of the top pass: the stages, then the logits.
template <int NT> constexpr size_t dense_top_lds() {
    using S = DStep<NT, DT_MT, DT_WAVES>;
    constexpr size_t sc = DT_TOK * DN_SC * 4, work = S::S * S::STAGE;
    return work > sc ? work : sc;
}

template <int NT>
__global__ __launch_bounds__(64 * DT_WAVES, 3) void dense_top_kernel(Params p, DenseArgs a) {
    extern __shared__ __align__(16) unsigned char lds[];
    __shared__ int32_t s_hist[1 << DN_MAX_LEVELS];
    __shared__ int32_t s_list[DT_TOK];
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int64_t base = int64_t(blockIdx.x) * DT_TOK;
    if (tid < (1 << DN_MAX_LEVELS)) s_hist[tid] = 0;
    if (tid < DT_TOK) {
        const int64_t t = base + tid;
        s_list[tid] = int32_t(t < p.n_tokens ? t : p.n_tokens - 1);
    }
    __syncthreads();
    tile_v4f acc[DT_MT][NT];
    dn_logits<NT, DT_MT, DT_WAVES>(p, 0, 0, a.s, s_list, DT_MT, lds, acc);
    float* const sc = reinterpret_cast<float*>(lds) + wave * 16 * DT_MT * DN_SC;
    dn_put_logits<DT_MT, NT>(acc, sc);
    dn_wave_sync();
    // lanes l and l + 32 walk row l, and take three levels' activations each
    const int row = lane & 31, half = lane >> 5;
    float lg[DN_MAX_LEVELS];
    const int c = dn_descend(sc + row * DN_SC, a.s, true, lg);
    const int64_t t = base + 16 * (wave + DT_WAVES * (row >> 4)) + (row & 15);
    if (t < p.n_tokens) {
#pragma unroll
        for (int l = 0; l < DN_MAX_LEVELS; ++l)
            if (l / 3 == half && l < a.s) {
                a.rec[t * DN_REC + l] = activation(lg[l], p.act);
                if (p.nodes_out) dn_record(p, t, l, (c >> (a.s - l)) - 1);
            }
        if (half == 0) {
            const int g = c - (1 << a.s);
            a.gid[t] = uint8_t(g);
            atomicAdd(&s_hist[g], 1);
        }
    }
    __syncthreads();
    if (tid < (1 << a.s)) {
        uint8_t* h = a.hist + int64_t(tid) * a.hist_ld;
        h[blockIdx.x] = uint8_t(s_hist[tid]);
        if (blockIdx.x == gridDim.x - 1)
            for (int i = a.top_wgs; i < a.hist_ld; ++i) h[i] = 0;
    }
}

// ----------------------------------------------------------------------------
// subtree pass
// ----------------------------------------------------------------------------

// Sum of the four bytes of each word of v.
__device__ __forceinline__ uint32_t bytes_sum(const uint4& v) {
    uint32_t s = 0;
#pragma unroll
    for (int j = 0; j < 4; ++j) s = __builtin_amdgcn_sad_u8(word(v, j), 0u, s);
    return s;
}

// Inclusive sum over the wave.
__device__ __forceinline__ int wave_scan(int v, int lane) {
#pragma unroll
    for (int d = 1; d < 64; d <<= 1) {
        const int u = __shfl_up(v, d, 64);
        if (lane >= d) v += u;
    }
    return v;
}

// Sizes of the subtree pass.  LDS: the token lookup, then the stages of the logit loop, then per wave
// its logits and its part of A, then W_out of the ancestors and the subtree, transposed, all columns
// at once (so that no load follows a store of y: vector memory operations retire in order, and a wait
// for such a load would wait for the stores).
template <int NT> struct DSub {
    static constexpr int CH = 1 + 2 * NT;             // eight-node chunks: the ancestors, then columns 8i .. 8i+7
    static constexpr int KSO = (2 * CH + 3) / 4;      // MFMA steps of the output product: four (part, chunk) pairs each
    static constexpr int AROW = KSO * 64 + 16;        // bytes per token of A (an odd number of 16-byte units)
    static constexpr int WROW = CH * 16;              // bytes per column of W_out^T (likewise)
    static constexpr int SC = 16 * DS_MT * DN_SC * 4, AB = 16 * DS_MT * AROW;
    static constexpr int PW = ((SC > AB ? SC : AB) + 15) / 16 * 16;  // per wave
    using S = DStep<NT, DS_MT, DS_WAVES>;
    // 64 group sizes, the group's prefix sums, wave totals, all counts
    static constexpr size_t LOOKUP = 64 * 4 + 4 * DS_THREADS * 4 + 8 * 4 + (size_t(DN_CHUNK / DT_TOK) << DN_MAX_LEVELS);
    static size_t lds(int hidden) {
        return std::max({size_t(S::S) * S::STAGE, size_t(DS_WAVES) * PW, size_t(hidden) * WROW, LOOKUP});
    }
};

// SRC: a bf16 source row (p.tile_src) is added to each output row.
template <int NT, bool SRC>
__global__ __launch_bounds__(DS_THREADS, 2) void dense_sub_kernel(Params p, DenseArgs a) {
    using Z = DSub<NT>;
    constexpr int MT = DS_MT, TOK = DS_TOK, CH = Z::CH, KSO = Z::KSO, AROW = Z::AROW, WROW = Z::WROW;
    extern __shared__ __align__(16) unsigned char lds[];
    __shared__ int32_t s_list[TOK];
    __shared__ int32_t s_bad[DN_MAX_HIDDEN / 128];  // column blocks whose weights hold inf or nan
    const int tid = threadIdx.x, lane = tid & 63, n = lane & 15, q = lane >> 4;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int s = a.s, levels = a.levels, D = p.depth;
    int g = 0, count;
    if (tid < DN_MAX_HIDDEN / 128) s_bad[tid] = 0;
    // W_out on its way to LDS: unit u (sixteen lanes) is (chunk u / blocks, 128-column block u % blocks),
    // a lane taking eight rows' 16 bytes; two units per sixteen lanes are in flight from here on
    const int64_t H = p.hidden;
    const int blocks = p.hidden / 128, units = CH * blocks, u16 = tid & 15;
    const uint32_t rblocks = 65536u / uint32_t(blocks) + 1;  // u / blocks = u rblocks >> 16 for u < 256
    uint4 wr[2][8];
    auto fetch = [&](int u, uint4 (&w)[8]) {
        if (u < units) {
            const int uc = int((uint32_t(u) * rblocks) >> 16), cb = u - uc * blocks;
            const uint32_t col = uint32_t(cb * 256 + u16 * 16), rowb = uint32_t(p.hidden) * 2;
            const uint32_t g1 = (1u << s) + uint32_t(g);  // the subtree root, counted from 1
            // chunk 0: the ancestors; 1: columns 1 .. 7 (levels 0 to 2); from 2 on eight nodes of one level
            const uint32_t c0 = uint32_t(8 * uc - 8), l0 = 31 - __builtin_clz(c0 | 1u);
            const bool whole = uc >= 2 && c0 < (1u << levels);
#pragma unroll
            for (int i = 0; i < 8; ++i) {
                constexpr int lvl1[8] = {0, 0, 1, 1, 2, 2, 2, 2};
                const uint32_t anc = g1 >> (i < s ? s - i : 0);
                const uint32_t top = i > 0 && lvl1[i] < levels ? (g1 << lvl1[i]) + uint32_t(i) - (1u << lvl1[i]) : g1;
                const uint32_t sub = whole ? (g1 << l0) + c0 + uint32_t(i) - (1u << l0) : g1;
                const uint32_t node = (uc == 0 ? anc : uc == 1 ? top : sub) - 1;  // heap node (rows at most 2 KB: 32 bits)
                w[i] = *reinterpret_cast<const uint4*>(static_cast<const char*>(p.w_out) + node * rowb + col);
            }
        }
    };
    if (s == 0) {
        fetch(tid >> 4, wr[0]);
        fetch((tid >> 4) + DS_THREADS / 16, wr[1]);
        __builtin_amdgcn_sched_barrier(0);
        const int64_t b0 = int64_t(blockIdx.x) * a.item;
        count = int(p.n_tokens - b0 < a.item ? p.n_tokens - b0 : a.item);
        if (tid < TOK) s_list[tid] = int32_t(b0 + (tid < count ? tid : count - 1));
    } else {
        // tokens per group, eight threads per group; the counts stay in LDS
        int32_t* s_cnt = reinterpret_cast<int32_t*>(lds);
        int32_t* s_pre = s_cnt + 64;  // [4 * DS_THREADS] tokens of this group in earlier top workgroups
        int32_t* s_tot = s_pre + 4 * DS_THREADS;
        uint4* s_hist = reinterpret_cast<uint4*>(s_tot + 8);  // [2^s][hist_ld / 16]
        {
            constexpr int UN = (DN_CHUNK / DT_TOK / 16 + 7) / 8;  // 16-byte vectors per thread
            const int gg = tid >> 3, hv = a.hist_ld / 16;
            const bool live = gg < (1 << s);
            const uint4* h = reinterpret_cast<const uint4*>(a.hist + int64_t(live ? gg : 0) * a.hist_ld);
            uint4 v[UN];
#pragma unroll
            for (int j = 0; j < UN; ++j) {
                const int c = (tid & 7) + 8 * j;
                v[j] = live && c < hv ? h[c] : make_uint4(0, 0, 0, 0);
            }
            uint32_t sum = 0;
#pragma unroll
            for (int j = 0; j < UN; ++j) {
                const int c = (tid & 7) + 8 * j;
                sum += bytes_sum(v[j]);
                if (live && c < hv) s_hist[gg * hv + c] = v[j];
            }
#pragma unroll
            for (int d = 1; d < 8; d <<= 1) sum += __shfl_xor(sum, d, 64);
            if ((tid & 7) == 0) s_cnt[gg] = int32_t(sum);
        }
        __syncthreads();
        // items: ceil(count / most) per group, groups in order, with the smallest bound (a multiple of 16, from
        // a.item up) whose items all run at once: the groups' sizes are the routing's, and one item more than
        // the CUs take would cost a second round (a.item alone, an eighth over the mean: depth 11,
        // hidden 768, 57344 / 61440 / 65536 tokens 102 / 107 / 80 us a forward; so 75 / 78 / 82).  XCD x
        // (blockIdx % 8) takes a contiguous eighth of them, so that a group's rows are read through one L2
        const int cnt = s_cnt[lane];
        int lo16 = a.item / 16, hi16 = TOK / 16;
        const int cnt16 = (cnt + 15) / 16;
        auto items_of = [&](int m) {  // ceil(cnt16 / m): the quotient is 0.5 / m or more from the next integer
            return int((float(cnt16 + m - 1) + 0.5f) * __builtin_amdgcn_rcpf(float(m)));
        };
        for (int m = lo16; lo16 < hi16; m = (lo16 + hi16) / 2) {  // the first bound fits as a rule
            if (int(group_sum<64>(float(items_of(m)))) <= a.round) hi16 = m;
            else lo16 = m + 1;
            lo16 = __builtin_amdgcn_readfirstlane(lo16);
            hi16 = __builtin_amdgcn_readfirstlane(hi16);
        }
        const int items = items_of(lo16);
        const int incl = wave_scan(items, lane);
        const int total = __builtin_amdgcn_readlane(incl, 63);
        const int x = int(blockIdx.x % XCDS), i = int(blockIdx.x / XCDS);
        const int i0 = int(int64_t(total) * x / XCDS), i1 = int(int64_t(total) * (x + 1) / XCDS);
        if (i >= i1 - i0) return;  // workgroup-uniform
        const int item = i0 + i;
        g = __builtin_ctzll(__ballot(incl > item));
        const int gc = __builtin_amdgcn_readlane(cnt, g), gi = __builtin_amdgcn_readlane(items, g);
        const int sl = item - (__builtin_amdgcn_readlane(incl, g) - gi);
        const int lo = int(int64_t(gc) * sl / gi), hi = int(int64_t(gc) * (sl + 1) / gi);
        count = hi - lo;
        fetch(tid >> 4, wr[0]);
        fetch((tid >> 4) + DS_THREADS / 16, wr[1]);
        __builtin_amdgcn_sched_barrier(0);
        // tokens lo .. hi-1 of the group, in token order
        typedef uint32_t __attribute__((may_alias)) u32a;
        uint32_t hw = 0;
        if (4 * tid < a.hist_ld) hw = *reinterpret_cast<const u32a*>(reinterpret_cast<unsigned char*>(s_hist) + g * a.hist_ld + 4 * tid);
        const int mine = int(__builtin_amdgcn_sad_u8(hw, 0u, 0u));
        const int scan = wave_scan(mine, lane);
        if (lane == 63) s_tot[wave] = scan;
        __syncthreads();
        int pre = scan - mine;
        for (int w = 0; w < wave; ++w) pre += s_tot[w];
#pragma unroll
        for (int j = 0; j < 4; ++j) {
            s_pre[4 * tid + j] = pre;
            pre += int((hw >> (8 * j)) & 0xffu);
        }
        __syncthreads();
        // first and last top workgroup holding any of them: the last whose prefix is <= lo (hi - 1)
        int f0 = 0, f1 = 0;
#pragma unroll
        for (int b = 512; b > 0; b >>= 1) {
            if (f0 + b < a.top_wgs && s_pre[f0 + b] <= lo) f0 += b;
            if (f1 + b < a.top_wgs && s_pre[f1 + b] <= hi - 1) f1 += b;
        }
        // eight threads per top workgroup, 16 tokens each; four rounds' loads at once
        static_assert(DT_TOK == 128, "eight threads of 16 tokens per top workgroup");
        constexpr int RW = DS_THREADS / 8, UN = 4;
        for (int r0 = f0; r0 <= f1; r0 += RW * UN) {
            uint4 v[UN];
#pragma unroll
            for (int j = 0; j < UN; ++j) {
                const int w = r0 + j * RW + (tid >> 3);
                v[j] = *reinterpret_cast<const uint4*>(a.gid + int64_t(w <= f1 ? w : f1) * DT_TOK + 16 * (tid & 7));
            }
#pragma unroll
            for (int j = 0; j < UN; ++j) {
                if (r0 + j * RW > f1) break;  // uniform
                const int w = r0 + j * RW + (tid >> 3);
                const bool live = w <= f1;
                const int t0 = w * DT_TOK + 16 * (tid & 7);
                uint32_t mask = 0;
#pragma unroll
                for (int b = 0; b < 16; ++b)
                    mask |= (((word(v[j], b / 4) >> (8 * (b % 4))) & 0xffu) == uint32_t(g) ? 1u : 0u) << b;
                const int left = int(p.n_tokens) - t0;  // gid is padded to whole workgroups
                if (left < 16) mask &= left > 0 ? (1u << left) - 1 : 0u;
                if (!live) mask = 0;
                int incl8 = __popc(mask);
#pragma unroll
                for (int d = 1; d < 8; d <<= 1) {
                    const int u = __shfl_up(incl8, d, 8);
                    if ((tid & 7) >= d) incl8 += u;
                }
                int pos = live ? s_pre[w] + incl8 - __popc(mask) - lo : 0;
                while (mask) {
                    const int b = __builtin_ctz(mask);
                    mask &= mask - 1;
                    if (pos >= 0 && pos < count) s_list[pos] = t0 + b;
                    ++pos;
                }
            }
        }
        __syncthreads();
        if (tid >= count && tid < TOK) s_list[tid] = s_list[count - 1];  // rows past the count: loaded, never stored
    }
    __syncthreads();
    const int all_tiles = (count + 15) / 16;
    const int tiles = (all_tiles - wave + DS_WAVES - 1) / DS_WAVES;  // of this wave (all_tiles - wave > -DS_WAVES)
    // lane i < 16 MT handles the path of row i % 16 of tile i / 16
    const bool worker = lane < 16 * MT;
    const int mine = 16 * (wave + DS_WAVES * (worker ? lane >> 4 : 0)) + n;
    const bool valid = worker && mine < count;
    const int64_t mtok = s_list[mine];
    float tp[DN_REC];  // activations of the levels above the subtree
#pragma unroll
    for (int j = 0; j < DN_REC; j += 4) {
        const float4 v = s > j ? *reinterpret_cast<const float4*>(a.rec + mtok * DN_REC + j) : make_float4(0.f, 0.f, 0.f, 0.f);
#pragma unroll
        for (int e = 0; e < 4; ++e) tp[j + e] = j + e < s ? fword(v, e) : 0.0f;
    }

    tile_v4f acc[MT][NT];
    dn_logits<NT, MT, DS_WAVES>(p, g, s, levels, s_list, tiles, lds, acc);

    // Output tiles per store: eight (16 bytes of a row per lane: column c of a 128-column block is MFMA
    // column n of tile j with c = 8 n + j), or four where source rows take registers (8 bytes, two
    // rounds per block: c = 64 (j / 4) + 4 n + j % 4).
    constexpr int NB = SRC ? 4 : 8, HB = 8 / NB;
    auto put = [&](int u, const uint4 (&w)[8]) {
        if (u >= units) return;
        const int uc = int((uint32_t(u) * rblocks) >> 16), cb = u - uc * blocks;
        unsigned char* const buf = lds + size_t(cb) * 128 * WROW + uc * 16;
        typedef uint16_t us2 __attribute__((ext_vector_type(2)));
        us2 big = {0, 0};
#pragma unroll
        for (int i = 0; i < 8; ++i)
#pragma unroll
            for (int j = 0; j < 4; ++j)
                big = __builtin_elementwise_max(big, __builtin_bit_cast(us2, word(w[i], j) & 0x7fff7fffu));
        if (big.x >= 0x7f80 || big.y >= 0x7f80) s_bad[cb] = 1;
#pragma unroll
        for (int e = 0; e < 8; ++e) {
            uint32_t w4[4];
#pragma unroll
            for (int k = 0; k < 4; ++k) {
                const uint32_t l = word(w[2 * k], e / 2), h = word(w[2 * k + 1], e / 2);
                w4[k] = (e & 1) ? (l >> 16) | (h & 0xffff0000u) : (l & 0xffffu) | (h << 16);
            }
            const int c = 8 * u16 + e;
            const int slot = NB == 8 ? e * 16 + u16 : ((c >> 6) * 4 + (e & 3)) * 16 + ((c & 63) >> 2);
            *reinterpret_cast<uint4*>(buf + slot * WROW) = make_uint4(w4[0], w4[1], w4[2], w4[3]);
        }
    };
    unsigned char* const pw = lds + wave * Z::PW;
    dn_put_logits<MT, NT>(acc, reinterpret_cast<float*>(pw));
    dn_wave_sync();
    float lg[DN_MAX_LEVELS];
    const int leaf = dn_descend(reinterpret_cast<const float*>(pw) + (worker ? lane : 0) * DN_SC, levels, false, lg);
    dn_wave_sync();
    // A: [token][part * CH + chunk] of eight bf16; chunk 0 the ancestors by level, chunk 1 + i the
    // columns 8i .. 8i+7
    for (int i = lane; i < 16 * MT * AROW / 16; i += 64) reinterpret_cast<uint4*>(pw)[i] = make_uint4(0, 0, 0, 0);
    dn_wave_sync();
    if (worker) {
        typedef uint4 __attribute__((may_alias)) u4a;
        typedef uint16_t __attribute__((may_alias)) u16a;
        unsigned char* const row = pw + lane * AROW;
        uint32_t h4[4], m4[4];
#pragma unroll
        for (int j = 0; j < 4; ++j) dn_split2(tp[2 * j], tp[2 * j + 1], h4[j], m4[j]);
        *reinterpret_cast<u4a*>(row) = make_uint4(h4[0], h4[1], h4[2], h4[3]);
        *reinterpret_cast<u4a*>(row + CH * 16) = make_uint4(m4[0], m4[1], m4[2], m4[3]);
        float av[DN_REC] = {};
#pragma unroll
        for (int l = 0; l < DN_MAX_LEVELS; ++l)
            if (l < levels) {
                av[l] = activation(lg[l], p.act);
                const int c = leaf >> (levels - 1 - l);
                uint32_t hi, mid;
                dn_split2(av[l], 0.0f, hi, mid);
                unsigned char* const e = row + 16 + 2 * c;  // chunk 1 + c / 8, element c % 8
                *reinterpret_cast<u16a*>(e) = uint16_t(hi);
                *reinterpret_cast<u16a*>(e + CH * 16) = uint16_t(mid);
                if (valid && p.nodes_out) dn_record(p, mtok, s + l, dn_node(c, g, s, levels));
            }
        av[DN_REC - 1] = __int_as_float(leaf);
        if (valid) {
            float4* const act = reinterpret_cast<float4*>(a.act + mtok * DN_REC);
            act[0] = make_float4(av[0], av[1], av[2], av[3]);
            act[1] = make_float4(av[4], av[5], av[6], av[7]);
        }
    }
    dn_wave_sync();
    bf16x8_t fa[MT][KSO];
#pragma unroll
    for (int mt = 0; mt < MT; ++mt)
#pragma unroll
        for (int k = 0; k < KSO; ++k)
            fa[mt][k] = __builtin_bit_cast(bf16x8_t, *reinterpret_cast<const uint4*>(pw + (mt * 16 + n) * AROW + (4 * k + q) * 16));
    // this lane's chunk in each step (pairs past the last repeat chunk 0: their part of A is zero)
    uint32_t boff[KSO];
#pragma unroll
    for (int k = 0; k < KSO; ++k) {
        const int e = 4 * k + q;
        boff[k] = uint32_t(n * WROW + (e < 2 * CH ? e % CH : 0) * 16);
    }
    int32_t rtok[MT][4];  // the tokens of this lane's result rows, -1 for none
#pragma unroll
    for (int mt = 0; mt < MT; ++mt)
#pragma unroll
        for (int r = 0; r < 4; ++r) {
            const int i = 16 * (wave + DS_WAVES * mt) + 4 * q + r;
            rtok[mt][r] = i < count ? s_list[i] : -1;
        }
    __syncthreads();  // every wave has read its part of A: W_out overwrites it
    constexpr int UR = DS_THREADS / 16;  // units per round
    put(tid >> 4, wr[0]);
    put((tid >> 4) + UR, wr[1]);
    for (int u0 = 2 * UR; u0 < units; u0 += UR) {
        fetch(u0 + (tid >> 4), wr[0]);
        put(u0 + (tid >> 4), wr[0]);
    }
    __syncthreads();
    struct Src { uint2 v[MT][4]; };  // the source's four columns of each result row
    auto at_of = [&](int mt, int r, int it) {
        return int64_t(rtok[mt][r] >= 0 ? rtok[mt][r] : s_list[0]) * H + int64_t(it / HB) * 128 +
               (NB == 8 ? 8 * n : 64 * (it % HB) + 4 * n);
    };
    const uint16_t* const src = static_cast<const uint16_t*>(p.tile_src);
    uint16_t* const y = static_cast<uint16_t*>(p.y);
    auto load_src = [&](int it, Src& sr) {
#pragma unroll
        for (int mt = 0; mt < MT; ++mt)
#pragma unroll
            for (int r = 0; r < 4; ++r) sr.v[mt][r] = *reinterpret_cast<const uint2*>(src + at_of(mt, r, it));
    };
    auto block = [&](int it, const Src& sr, auto mts) {
        constexpr int M = decltype(mts)::value;
        const unsigned char* const buf = lds + size_t(it / HB) * 128 * WROW + (it % HB) * NB * 16 * WROW;
        tile_v4f o[M][NB];
#pragma unroll
        for (int j = 0; j < NB; ++j) {
#pragma unroll
            for (int mt = 0; mt < M; ++mt) o[mt][j] = tile_v4f{0.f, 0.f, 0.f, 0.f};
#pragma unroll
            for (int k = 0; k < KSO; ++k) {
                const bf16x8_t fb = __builtin_bit_cast(bf16x8_t, *reinterpret_cast<const uint4*>(buf + j * 16 * WROW + boff[k]));
#pragma unroll
                for (int mt = 0; mt < M; ++mt)
                    o[mt][j] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(fa[mt][k], fb, o[mt][j], 0, 0, 0);
            }
        }
#pragma unroll
        for (int mt = 0; mt < M; ++mt)
#pragma unroll
            for (int r = 0; r < 4; ++r) {
                if (rtok[mt][r] < 0) continue;
                const int64_t at = at_of(mt, r, it);
                float v[NB];
#pragma unroll
                for (int j = 0; j < NB; ++j) v[j] = o[mt][j][r];
                if constexpr (SRC) {
                    const uint2 u = sr.v[mt][r];
                    v[0] += bf16_lo(u.x); v[1] += bf16_hi(u.x); v[2] += bf16_lo(u.y); v[3] += bf16_hi(u.y);
                }
                if constexpr (NB == 8)
                    *reinterpret_cast<uint4*>(y + at) = make_uint4(pack_bf16x2(v[0], v[1]), pack_bf16x2(v[2], v[3]),
                                                                   pack_bf16x2(v[4], v[5]), pack_bf16x2(v[6], v[7]));
                else
                    *reinterpret_cast<uint2*>(y + at) = make_uint2(pack_bf16x2(v[0], v[1]), pack_bf16x2(v[2], v[3]));
            }
    };
    // Infinite or nan weights among a block's rows: a zero activation times such a weight would reach
    // tokens that do not visit the node, so the block's outputs are summed per token along its path.
    auto block_by_path = [&](int cb) {
        __threadfence();
        for (int i = 0; i < 16 * tiles; ++i) {
            const int w = 16 * (wave + DS_WAVES * (i >> 4)) + (i & 15);
            if (w >= count) break;
            const int64_t t = s_list[w];
            const float* const act = a.act + t * DN_REC;
            const int64_t leaf1 = dn_node(__float_as_int(act[DN_REC - 1]), g, s, levels) + 1;
            for (int c = lane; c < 128; c += 64) {
                const int64_t col = int64_t(cb) * 128 + c;
                float v = 0.0f;
                for (int l = 0; l <= D; ++l)
                    v = __builtin_fmaf(l < s ? a.rec[t * DN_REC + l] : act[l - s],
                                       bf16_to_f32(static_cast<const uint16_t*>(p.w_out)[((leaf1 >> (D - l)) - 1) * H + col]), v);
                const int64_t at = t * H + col;
                if (SRC) v += bf16_to_f32(src[at]);
                y[at] = f32_to_bf16(v);
            }
        }
    };
    auto run = [&](int it, const Src& sr) {
        if (s_bad[it / HB] == 0) dn_tiles<MT>(tiles, [&](auto m) { block(it, sr, m); });  // wave-uniform
        else if (it % HB == 0) block_by_path(it / HB);
    };
    const int its = blocks * HB;
    if constexpr (!SRC) {
        const Src none{};
        for (int it = 0; it < its; ++it) run(it, none);
    } else {
        // the source rows of the next tiles are loaded before this one's stores
        static_assert(!SRC || HB == 2, "an even number of rounds");
        Src s0, s1;
        load_src(0, s0);
        for (int it = 0; it < its; it += 2) {
            load_src(it + 1, s1);
            __builtin_amdgcn_sched_barrier(0);
            run(it, s0);
            load_src(it + 2 < its ? it + 2 : it + 1, s0);
            __builtin_amdgcn_sched_barrier(0);
            run(it + 1, s1);
        }
    }
}

size_t align256(size_t v) { return (v + 255) & ~size_t(255); }

}  // namespace

int dense_top_levels(int32_t depth) {
    const int levels = depth + 1;
    return levels <= DN_MAX_LEVELS ? 0 : levels <= 2 * (DN_MAX_LEVELS - 1) ? levels / 2 : DN_MAX_LEVELS;
}

bool dense_shape(const Params& p) {
    return p.x_bf16 && p.w_bf16 && p.y_bf16 && !p.norm && !p.logits_out && p.n_trees == 1 && p.depth < 2 * DN_MAX_LEVELS &&
           p.hidden % 128 == 0 && p.hidden <= DN_MAX_HIDDEN;
}

size_t dense_workspace_bytes(int64_t n_tokens) {
    const size_t n = size_t(std::min(n_tokens, DN_CHUNK));
    const size_t wgs = (n + DT_TOK - 1) / DT_TOK, ld = (wgs + 15) / 16 * 16;
    return 2 * align256(n * DN_REC * sizeof(float)) + align256(wgs * DT_TOK) + align256(ld << DN_MAX_LEVELS);
}

constexpr int DN_ITEM_MIN = 16 * DS_WAVES;  // a tile per wave

// The least bound on a subtree workgroup's tokens (a multiple of 16): the mean group over as many workgroups as
// fill the CUs, with an eighth to spare for the usual spread of the groups' sizes.
static int dense_item_least(int64_t n_tokens, int s, int cu_count) {
    const double mean = double(n_tokens) / double(int64_t(1) << s);
    const int64_t per = std::max<int64_t>(1, cu_count >> s);  // workgroups per group
    const int64_t item = int64_t(mean * 1.125 / double(per) / 16.0 + 1.0) * 16;
    return int(std::min<int64_t>(std::max<int64_t>(item, DN_ITEM_MIN), DS_TOK));
}

// Tokens of a workgroup without a top pass (a multiple of 16): the batch over a number of workgroups that
// fills the CUs.
static int dense_item(int64_t n_tokens, int cu_count) {
    int64_t item = DS_TOK + 1;
    for (int64_t k = cu_count; item > DS_TOK; k += cu_count) item = (n_tokens / k / 16 + 1) * 16;
    return int(std::max<int64_t>(item, DN_ITEM_MIN));
}

// Equal chunks of at most DN_CHUNK tokens.
int64_t dense_chunk(int64_t n_tokens) {
    const int64_t chunks = std::max<int64_t>(1, (n_tokens + DN_CHUNK - 1) / DN_CHUNK);
    return (n_tokens + chunks - 1) / chunks;
}

int dense_launches(const Params& p, int64_t n_tokens, int cu_count, Launch* L) {
    const int s = dense_top_levels(p.depth), sub = p.depth + 1 - s;
    int n = 0;
    if (s) {
        L[n].kernel = s > 5 ? reinterpret_cast<const void*>(&dense_top_kernel<4>) : reinterpret_cast<const void*>(&dense_top_kernel<2>);
        L[n].grid = int((n_tokens + DT_TOK - 1) / DT_TOK);
        L[n].block = 64 * DT_WAVES;
        L[n++].lds_bytes = s > 5 ? dense_top_lds<4>() : dense_top_lds<2>();
    }
    const bool src = p.out_mode != OUT_STORE;
    L[n].kernel = sub > 5 ? (src ? reinterpret_cast<const void*>(&dense_sub_kernel<4, true>)
                                 : reinterpret_cast<const void*>(&dense_sub_kernel<4, false>))
                          : (src ? reinterpret_cast<const void*>(&dense_sub_kernel<2, true>)
                                 : reinterpret_cast<const void*>(&dense_sub_kernel<2, false>));
    L[n].block = DS_THREADS;
    L[n].lds_bytes = sub > 5 ? DSub<4>::lds(p.hidden) : DSub<2>::lds(p.hidden);
    if (s) {
        // at most one item per whole `most` tokens and one partly filled per group: a round of them, or with
        // the bound at its least or its most
        const int64_t groups = int64_t(1) << s;
        const int64_t items = std::min(n_tokens / DN_ITEM_MIN + groups, std::max<int64_t>(cu_count, n_tokens / DS_TOK + groups));
        L[n++].grid = int((items + XCDS - 1) / XCDS * XCDS);
    } else {
        const int item = dense_item(n_tokens, cu_count);
        L[n++].grid = int((n_tokens + item - 1) / item);
    }
    return n;
}

hipError_t run_dense(const Params& p, void* workspace, int cu_count, hipStream_t stream) {
    const int levels = p.depth + 1, s = dense_top_levels(p.depth), sub = levels - s;
    const int64_t H = p.hidden;
    // pairs of passes over equal chunks
    const int64_t chunk = dense_chunk(p.n_tokens);
    for (int64_t c0 = 0; c0 < p.n_tokens; c0 += chunk) {
        Params c = p;
        c.n_tokens = std::min(chunk, p.n_tokens - c0);
        c.x = static_cast<const uint16_t*>(p.x) + c0 * H;
        c.y = static_cast<uint16_t*>(p.y) + c0 * H;
        if (p.nodes_out) c.nodes_out = p.nodes_out + c0 * levels;
        c.tile_src = p.out_mode == OUT_RESIDUAL ? c.x : p.out_mode == OUT_ACCUMULATE ? c.y : nullptr;
        const int64_t wgs = (c.n_tokens + DT_TOK - 1) / DT_TOK;
        DenseArgs a{};
        char* ws = static_cast<char*>(workspace);
        a.rec = reinterpret_cast<float*>(ws);
        ws += align256(size_t(c.n_tokens) * DN_REC * sizeof(float));
        a.act = reinterpret_cast<float*>(ws);
        ws += align256(size_t(c.n_tokens) * DN_REC * sizeof(float));
        a.gid = reinterpret_cast<uint8_t*>(ws);
        ws += align256(size_t(wgs) * DT_TOK);
        a.hist = reinterpret_cast<uint8_t*>(ws);
        a.top_wgs = int32_t(wgs);
        a.hist_ld = int32_t((wgs + 15) / 16 * 16);
        a.s = s;
        a.levels = sub;
        a.item = s ? dense_item_least(c.n_tokens, s, cu_count) : dense_item(c.n_tokens, cu_count);
        a.round = cu_count;
        void* args[] = {&c, &a};
        Launch L[2];
        const int n = dense_launches(c, c.n_tokens, cu_count, L);
        for (int i = 0; i < n; ++i) {
            const hipError_t e = hipLaunchKernel(L[i].kernel, dim3(unsigned(L[i].grid)), dim3(unsigned(L[i].block)), args,
                                                 L[i].lds_bytes, stream);
            if (e != hipSuccess) return e;
        }
    }
    return hipSuccess;
}

}  // namespace fff
