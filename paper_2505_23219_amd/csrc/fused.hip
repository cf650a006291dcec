// The attention kernel (see attention_impl.h), the set-up kernel and the dispatch of the
// persistent kernels.
#include "attention_impl.h"

namespace ghd {


// The first twelve words are what the first requests of the cache need (see AttnFirst); `source`: see mask_source.  With
// those read from the argument block and the shares worked out by integer divisions the first request went out
// 2.2 to 2.8 us after the start of a call's last launch.  us a call, then and now: 24 heads of 128, 48 rows, 3001 cached
// 18.3 and 17.4; 32 heads of 128, 1 row, 2048 cached 13.3 and 12.7; 16 heads, 32 rows, 8000 cached 22.7 and 21.6; 8 heads of 64,
// 100 rows, 1000 cached 11.4 and 11.0.
constexpr int kAttM = 0, kAttNh = 8, kAttGx = 17, kAttParents = 23, kAttFar = 24;    // bits of `flags`: M, nh, workgroups per XCD, ...
static_assert(kRangeWgs / 8 < 64 && GHD_MAX_M < 256, "fits its bits");
template <int MT, int D, bool ALONE>
__global__ __launch_bounds__(kFT) void k_attention(const half_t* k, const half_t* v, const void* source, uint32_t k_head8,
                                                   uint32_t v_head8, uint32_t st_tok, uint32_t st_ch, int T, uint32_t flags,
                                                   const FusedArgs)
{
    extern __shared__ __attribute__((aligned(16))) char lds[];
    const int M = flags >> kAttM & 255, nh = flags >> kAttNh & 511, Gx = flags >> kAttGx & 63;
    Ctx cx;
    cx.G = 8 * Gx;
    cx.j = (blockIdx.x & 7) * Gx + (blockIdx.x >> 3);
    cx.lds = lds;
    cx.parents = flags >> kAttParents & 1;
    if constexpr (ALONE) mask_source<(MT > 4)>(cx, source, M);
    AttnFirst f = {k, v, (int64_t)k_head8 * 8, (int64_t)v_head8 * 8, st_tok, st_ch, T, M, nh};
    if (flags >> kAttFar & 1) {              // (heads 64 GiB apart)
        f.k_head = late_args()->stride_head;
        f.v_head = late_args()->v_stride_head;
    }
    const AttnPlan plan = attn_plan(nh, (T + 63) >> 6, ALONE ? 0 : AttnOf<MT, D>::TMIN, blockIdx.x & 7, blockIdx.x >> 3, Gx);
    const auto late = []() -> const FusedArgs& { return *(const FusedArgs*)late_args(); };
    attn_phase<MT, D, false, ALONE>(f, late, cx, plan);
    if (ALONE && blockIdx.x == 0 && threadIdx.x == 0) carry_status(late().sync);
    wait_loads<0>();       // (nothing is on its way to the LDS when the workgroup ends)
}

// ---------------------------------------------------------------------------
// host side
// ---------------------------------------------------------------------------
template <int MT, int D, bool ALONE>
static ghd_status launch_attention_t(const FusedArgs& a, hipStream_t st)
{
    int G = 0;
    const size_t lds = sizeof(typename AttnOf<MT, D>::Lds);
    ghd_status s = launch_resident_checked((const void*)k_attention<MT, D, ALONE>, kFT, lds, &G);
    if (s) return s;
    if (ALONE) G = 8 * ceil_div(a.nh, 8) < G ? 8 * ceil_div(a.nh, 8) : G;
    // (strides are multiples of 8, and inside a head they fit 32 bits: checked where the call came in)
    const bool far = ((a.stride_head | a.v_stride_head) >> 35) != 0;
    const bool parents = ALONE && a.att_parent;
    const uint32_t flags = (uint32_t)a.M << kAttM | (uint32_t)a.nh << kAttNh | (uint32_t)(G / 8) << kAttGx | (uint32_t)parents << kAttParents | (uint32_t)far << kAttFar;
    const void* source = parents ? (const void*)a.att_parent : (const void*)a.mask;
    hipLaunchKernelGGL((k_attention<MT, D, ALONE>), dim3(G), dim3(kFT), lds, st, a.att_k, a.att_v, source, (uint32_t)(a.stride_head >> 3),
                       (uint32_t)(a.v_stride_head >> 3), (uint32_t)a.stride_tok, (uint32_t)a.v_stride_ch, a.kv_len + a.M, flags, a);
    return check_launch();
}

template <int D, bool ALONE>
static ghd_status launch_attention_d(const FusedArgs& a, hipStream_t st)
{
    // (above 32 rows the attention has wavefronts for 4 or 8 row tiles)
    switch (layout_tiles(row_tiles(a.M))) {
    case 1: return launch_attention_t<1, D, ALONE>(a, st);
    case 2: return launch_attention_t<2, D, ALONE>(a, st);
    case 4: return launch_attention_t<4, D, ALONE>(a, st);
    default: return launch_attention_t<8, D, ALONE>(a, st);
    }
}

// a.mode selects the kernel; the row-tile count of M selects the instantiation
ghd_status launch_fused(const FusedArgs& a, hipStream_t st)
{
    if (a.mode == MODE_LINEAR) return launch_linear(a, st);
    if (a.mode == MODE_QKV_ATTN) return launch_qkv_attn(a, st);
    if (a.att_alone) return a.d == 64 ? launch_attention_d<64, true>(a, st) : launch_attention_d<128, true>(a, st);
    return a.d == 64 ? launch_attention_d<64, false>(a, st) : launch_attention_d<128, false>(a, st);
}

thread_local int host_recip_ulps = 0;

// The attention's work shares on the host: for workgroup j and head `head`,
// out[0..5] = first part, number of parts, this part's index, t0, t1, and whether `head` is
// one of j's heads at all (otherwise the first five are -1).
void attn_share_on_host(int nh, int ntile, int tmin, int j, int G, int head, int* out)
{
    const int Gx = G / 8;        // (a grid that 8 does not divide, which no launch has, counts as the first of 8 XCDs)
    const AttnHeads hs = G % 8 ? attn_heads(8 * nh, 0, j, G) : attn_heads(nh, j / Gx, j % Gx, Gx);
    for (int i = 0; i < 6; ++i) out[i] = -1;
    out[5] = 0;
    const int hl = head - hs.hx0;
    if (hl < hs.h_lo || hl >= hs.h_hi) return;
    const AttnTiles ts = attn_tiles(hs, hl, ntile, tmin);
    out[0] = ts.first;
    out[1] = ts.np;
    out[2] = ts.me;
    out[3] = ts.t0;
    out[4] = ts.t1;
    out[5] = 1;
}

// An attention call whose heads are one workgroup's each needs no counter and so no launch before its own (3 us of
// the host's time, which makes two launches 10.5 us at least where calls are made one by one).  Against that stands one
// workgroup's way through all of a head's keys, where up to 32 of them share it otherwise.  The line was drawn with calls made one
// by one, of earlier kernels.  With the present ones, 8 heads under a tree, from a graph, us in two launches and in one (2 and 32
// heads differ by 0.3 us or less), below the line and past it:
//   d = 64:  8 rows, 12 tiles of 64 keys 8.5 and 8.9, 13 8.5 and 9.4; 32 rows, 12 tiles 10.2 and 10.1, 13 9.9 and 10.6;
//            64 rows, 4 tiles 8.5 and 7.2, 5 8.5 and 7.9, 6 8.4 and 8.7; 65 rows, 3 tiles 8.6 and 8.3, 4 8.4 and 9.6;
//            128 rows, 3 tiles 9.6 and 8.3, 4 9.2 and 9.6
//   d = 128: 8 rows, 6 tiles 10.1 and 9.7, 7 10.8 and 10.6, 8 11.0 and 11.4; 32 rows, 6 tiles 14.2 and 12.7, 7 14.6 and
//            13.8, 8 14.9 and 14.7; 64 rows, 4 tiles 10.5 and 9.4, 5 10.5 and 10.4, 6 10.5 and 11.3; 72 rows, 2 tiles 11.3
//            and 9.2, 3 10.5 and 11.0; 80 rows, 3 tiles 11.0 and 10.7; 88 rows, 3 tiles 11.3 and 11.0, 4 10.8 and 12.6;
//            128 rows, 3 tiles 12.9 and 10.9, 4 12.2 and 12.5
// So it lies right or a tile short: 5 tiles of 64 channels at 33 to 64 rows and 7 of 128 up to 32 rows would gain up to 0.8 us.
bool attention_alone(int M, int kv_len, int d)
{
    const int64_t ntile = ((int64_t)kv_len + M + 63) / 64;
    if (M <= 32) return ntile * d <= 6 * 128;
    if (M <= 64) return ntile <= 4;
    return ntile <= (d == 128 && M <= 80 ? 2 : 3);
}

// ---- setup kernel ------------------------------------------------------------
// Blocks 0..kRopeBlocks-1: the rotary table, a thread per element (the double-precision sine and cosine
// behind the node's depth are the longest chain of the launch); the next one: the ancestor masks.  The next kZeroBlocks
// blocks zero the sync block.  Further blocks: one per 16-column tile of the residual stream,
// writing x = widen(x_in), the tile's sums of squares and the gain-scaled fp16 image.
constexpr int kRopeBlocks = 32;      // a thread per element of the largest rotary table
static_assert(kRopeBlocks * 256 >= GHD_MAX_M * 64, "128 rows of 64 pairs");
constexpr int kTreeBlocks = kRopeBlocks + 1;
constexpr int kZeroBlocks = 64;

__global__ __launch_bounds__(256) void k_fused_setup(uint32_t* __restrict__ sync,
                                                     const int32_t* __restrict__ parent, int M,
                                                     int Mpad, int kv_len, int d, float rope_base,
                                                     uint64_t* __restrict__ mask,
                                                     float2* __restrict__ rope, float* __restrict__ x,
                                                     const half_t* __restrict__ x_in16, int H,
                                                     float* __restrict__ ss,
                                                     const half_t* __restrict__ gain,
                                                     half_t* __restrict__ xg16)
{
    int tid = threadIdx.x;
    if (blockIdx.x < kRopeBlocks) {
        const int half = d / 2, e = blockIdx.x * 256 + tid;
        if (!parent || !rope || blockIdx.x * 256 >= M * half) return;
        // This thread's element: its frequency base^(-2j/d), in double, while parent[] is on its way.
        const int row = e / half;
        const double freq = exp2(-2.0 / d * log2((double)rope_base) * (e - row * half));
        const int lane = tid & 63;
        const TreeNodes<2> t = tree_nodes<2, false>(parent[min(lane, M - 1)], parent[min(lane + 64, M - 1)], M, lane);
        const int depth = t.depth(row);
        if (e >= M * half) return;
        const double ang = (double)(kv_len + depth) * freq;
        double sn, cs;
        sincos(ang, &sn, &cs);
        rope[e] = make_float2((float)cs, (float)sn);
        return;
    }
    if (blockIdx.x < kTreeBlocks) {
        if (!parent || tid >= 64) return;
        store_masks(tree_nodes<2, true>(parent[min(tid, M - 1)], parent[min(tid + 64, M - 1)], M, tid), M, tid, mask);
        return;
    }
    if (blockIdx.x < kTreeBlocks + kZeroBlocks) {
        zero_sync<kZeroBlocks>(sync, blockIdx.x - kTreeBlocks);
        return;
    }
    // residual stream tiles: thread -> (row m, four columns of the 16-wide tile)
    const int col = (blockIdx.x - kTreeBlocks - kZeroBlocks) * 16 + (tid & 3) * 4;
    half4 g = {0, 0, 0, 0};
    if (xg16) g = *(const half4*)(gain + col);
#pragma unroll
    for (int i = 0; i < GHD_MAX_M / 64; ++i) {
        const int m = i * 64 + (tid >> 2);
        if (m >= Mpad) break;
        floatx4 v = {0.f, 0.f, 0.f, 0.f};
        if (m < M) {
            if (x_in16) {
                const half4 h = *(const half4*)(x_in16 + (size_t)m * H + col);
#pragma unroll
                for (int r = 0; r < 4; ++r) v[r] = (float)h[r];
                *(floatx4*)(x + (size_t)m * H + col) = v;
            } else {
                v = *(const floatx4*)(x + (size_t)m * H + col);
            }
            if (xg16) {
                half4 o;
#pragma unroll
                for (int r = 0; r < 4; ++r) o[r] = (half_t)(v[r] * (float)g[r] * kXgScale);
                *(half4*)(xg16 + xpk_index(m, col, Mpad >> 4)) = o;
            }
        }
        float s = (v[0] * v[0] + v[1] * v[1]) + (v[2] * v[2] + v[3] * v[3]);
        s += __shfl_xor(s, 1);
        s += __shfl_xor(s, 2);
        if ((tid & 3) == 0) ss[(size_t)(col >> 4) * Mpad + m] = s;
    }
}

ghd_status launch_fused_setup(uint32_t* sync, const int32_t* parent, int M, int Mpad, int kv_len, int d,
                              float rope_base, uint64_t* mask, float2* rope, float* x,
                              const half_t* x_in16, int H, float* ss, const half_t* gain,
                              half_t* xg16, hipStream_t st)
{
    int blocks = kTreeBlocks + kZeroBlocks + (ss ? H / 16 : 0);
    hipLaunchKernelGGL(k_fused_setup, dim3(blocks), dim3(256), 0, st, sync, parent, M, Mpad, kv_len, d,
                       rope_base, mask, rope, x, x_in16, H, ss, gain, xg16);
    return check_launch();
}

}  // namespace ghd
