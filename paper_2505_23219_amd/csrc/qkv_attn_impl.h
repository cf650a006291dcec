// The QKV linear layer and the tree attention of one decoder layer in one launch.
//
// The attention of head h needs q, k and v of head h only (Ghidorah, section 2.2.2: the
// heads are independent), and with the packed QKV rows grouped by XCD (see qkv_row) the
// workgroups that produce them are the ones that run that head's attention: all on one
// XCD.  So instead of ending the launch after the QKV layer, the 32 workgroups of an XCD
// meet at a counter in their L2 once their rotated queries and cache rows are stored, and go
// on with the attention of their XCD's heads.  What is saved is a launch boundary per
// layer: the dispatch gap and the start-up of the attention kernel.
#pragma once
#include "attention_impl.h"
#include "linear_impl.h"

namespace ghd {

template <int MT, int R, int D>
__global__ __launch_bounds__(kFT) void k_qkv_attn(const half8* W, const half_t* x, uint64_t aux, int nks, int K,
                                                  int ntiles, int cut, uint32_t magic, uint32_t flags,
                                                  const FusedArgs a)
{
    extern __shared__ __attribute__((aligned(16))) char lds[];
    const LinHead h = {W, x, aux, nks, K, ntiles, cut, magic, flags};
    int c0, c1;
    tile_range(ntiles, cut, magic, blockIdx.x, &c0, &c1);
    const int lane = threadIdx.x & 63, xcd = blockIdx.x & 7, Gx = cut;
    Ctx cx;
    cx.G = 8 * Gx;
    cx.j = xcd * Gx + (blockIdx.x >> 3);
    cx.lds = lds;
    AttnPlan plan;
    auto make_plan = [&]() {       // (while the first weights are on their way)
        const ArgPtr la = late_args();
        plan = attn_plan(la->nh, (la->kv_len + la->M + 63) >> 6, AttnOf<MT, D>::TMIN, xcd, blockIdx.x >> 3, Gx);
    };
    if (c0 >= c1) make_plan();
    else
        gemm_group<MT, R, 8, false, stretches_whole(MT, R), 0, 1>(
            h, lds, c0, c1 - c0, 0, nks, 0, make_plan,
            [&](ArgPtr la, auto&, auto& v, auto& m, auto& n0, const float* s_rinv) { epilogue(la, v, m, n0, lane, s_rinv); });
    // ---- the XCD's workgroups meet.  Every one of them counts itself in once its part of
    //      q16 and of the cache rows is acknowledged by the L2 they share (the wait below
    //      covers loads too, so it comes before the attention requests anything) ...
    //      The counter's line is for the arrivals alone, with thirty-two workgroups looking at it as
    //      well a 64-row step of 32 layers took 3873 us instead of 3860: the workgroup that arrives last
    //      passes the sum of the XCD numbers on to the others, each on a line of its own, with the
    //      number of the layer in place of the count.
    uint32_t* const cnt = a.sync + kCntXcd + xcd * kCntStride;
    uint32_t* const go = a.sync + kCntGo;
    const uint32_t round = a.att_epoch + 1;
    wait_own_stores();
    __syncthreads();       // also: the linear phase's use of the LDS is over
    bool last = false;
    uint32_t word = 0;
    if (threadIdx.x < 64) {
        // (a line a lane: one lane storing to all of them kept the others waiting 1.5 us longer)
        if (lane == 0) word = arrive(epoch_word(cnt, a.att_epoch));
        word = (uint32_t)__builtin_amdgcn_readfirstlane((int)word);
        last = (word & 0xffffu) == (uint32_t)Gx;
        if (last) {
            if (lane < Gx)
                __hip_atomic_store(go + (xcd * Gx + lane) * kCntStride, (word & 0xffff0000u) | round, __ATOMIC_RELAXED,
                                   __HIP_MEMORY_SCOPE_AGENT);
            if (lane == 0) clear_next(cnt, a.att_epoch);
        }
    }
    // ... and waits for the others at the attention's gate, after it has set up its indices
    //     and requested the cache rows of earlier steps that it starts with.  (Counting in
    //     only after that set-up was measured slower: it is the stores that make a workgroup
    //     late, and everybody waits for the last.)
    auto gate = [&]() -> bool {
        int* s_ok = &reinterpret_cast<typename AttnOf<MT, D>::Lds*>(cx.lds)->wait_ok;
        if (threadIdx.x == 0)
            *s_ok = last ? same_xcd(a.sync, word, (uint32_t)Gx)
                        : bounded_wait(a.sync, go + cx.j * kCntStride, ld_relaxed(go + cx.j * kCntStride), round, (uint32_t)Gx, 3000u);
        barrier_lds();
        if (!*s_ok) return false;
        // Nothing of q16 or of the tree's cache rows should be in this compute unit's L1 (it
        // has not read them in this launch); dropping the L1's contents makes that independent
        // of what the L1 does with this workgroup's own stores.  The L1 only: an agent-scope
        // acquire would also walk the L2, which every workgroup of the XCD is streaming through.
        invalidate_l1();
        return true;
    };
    const AttnFirst f = {a.att_k, a.att_v, a.stride_head, a.v_stride_head, (uint32_t)a.stride_tok, (uint32_t)a.v_stride_ch, a.kv_len + a.M, a.M, a.nh};
    const auto late = [&]() -> const FusedArgs& { return a; };
    attn_phase<MT, D, true, false>(f, late, cx, plan, gate);
    wait_loads<0>();       // (nothing is on its way to the LDS when the workgroup ends)
}

// the instantiations for one number of row tiles of x: head dim 128, wide QKV matrices of 3
// to 6 row tiles per workgroup (7B- to 70B-shaped layers)
template <int MT, int R>
ghd_status launch_qkv_attn_r(const FusedArgs& a, const LinCut& cut, hipStream_t st)
{
    if (a.d != 128 || !cut.whole) return GHD_ERR_SHAPE;
    if (cut.tiles == R) {
        static_assert(waves_of(MT, R) * 64 == kFT, "the attention works with eight wavefronts");
        constexpr size_t l1 = LinShape<MT, R, 8>::template lds_bytes<(stretches_whole(MT, R) > 1)>, l2 = sizeof(typename AttnOf<MT, 128>::Lds);
        return launch_linear_kernel(k_qkv_attn<MT, R, 128>, a, cut, kFT, l1 > l2 ? l1 : l2, st);
    }
    if constexpr (R < (MT <= 4 ? 6 : 4)) return launch_qkv_attn_r<MT, R + 1>(a, cut, st);
    return GHD_ERR_SHAPE;
}

ghd_status launch_qkv_attn_mt1(const FusedArgs& a, const LinCut& cut, hipStream_t st);
ghd_status launch_qkv_attn_mt2(const FusedArgs& a, const LinCut& cut, hipStream_t st);
ghd_status launch_qkv_attn_mt3(const FusedArgs& a, const LinCut& cut, hipStream_t st);
ghd_status launch_qkv_attn_mt4(const FusedArgs& a, const LinCut& cut, hipStream_t st);
ghd_status launch_qkv_attn_mt6(const FusedArgs& a, const LinCut& cut, hipStream_t st);
ghd_status launch_qkv_attn_mt8(const FusedArgs& a, const LinCut& cut, hipStream_t st);

}  // namespace ghd
