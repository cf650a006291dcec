// Tree attention of the verification step: the device code shared by the attention kernel
// and the fused QKV + attention kernel.
//
// A head's 64-key tiles are split over a run of workgroups of one XCD.  S^T = K q^T puts one
// query row in each lane column, so softmax statistics are per-lane scalars and the fp16
// probabilities come out in B-operand layout for O^T += V^T P^T; the V cache is kept channel-major,
// so V^T rows are read as they lie.  The ancestor mask (Ghidorah, section 2.3) is only looked at
// where keys reach into the tree rows, and keys no row can see are skipped.  The wavefronts'
// states are merged inside the workgroup, the workgroups of a head through one partial state each,
// with the online-softmax rescale of section 3.2.2.  Two ways through a workgroup's tiles:
//
// Up to 32 query rows (attn_direct), a wavefront works on 32-key units by itself: it loads a unit's
// K and V^T straight into MFMA operand registers, with no LDS and no barrier in between.  At
// 2048 cached tokens there are some eight units, one for each wavefront, so everything is
// requested at once and what is left is a chain of latencies (first loads out after 1.4 us, units done
// at 5.7, merged at 7.4, exchanged at 7.8).  7B-shaped layer at 2048 cached tokens, 1 row: the
// launch with the QKV layer 30.8 us staged, 27.6 us this way.  (The loads take 64 bytes of a
// row at a time, so they must not carry the non-temporal hint: the other half of the line is
// then fetched again, 30.2 us.)
//
// Above (attn_staged), the workgroup shares tiles through LDS, where they are loaded without passing
// through registers: a ring of buffers, a barrier a tile, and one copy of the code for a tile.  With up to
// 64 rows wavefronts 0-3 take the first 32 keys of a tile, 4-7 the last 32, each for its own 16 rows; with
// more a wavefront takes 16 rows and all keys.  What bounds it: at many tiles per workgroup HBM (13B-shaped
// layer, 8192 cached tokens: 1.2 us a tile of 32 KB on each compute unit, 6.9 TB/s); at few the chain of latencies around
// the tiles.  The same through registers, four tiles ahead, took seven copies of a tile's code (28 KB, each
// fetched when it is first run) and a final merge of a row per wavefront: attention of 24 heads, 48
// rows, 3001 cached tokens 20.5 us a call, 17.9 through the ring when it came in and 17.0 now; launch with the QKV layer and
// 128 rows at 2048 cached tokens 61 us, 52 and 50.  Each wavefront reading units by itself was slower there: the states of eight
// wavefronts with all rows take 4 us to merge, and with the rows split over groups of wavefronts every unit is
// read once per group (13B-shaped layer, 64 rows, 8192 cached tokens, launch with the QKV layer: 10 and 20 us more).
#pragma once
#include "persist.h"

#include <type_traits>

namespace ghd {

// ---------------------------------------------------------------------------
// tree attention
// ---------------------------------------------------------------------------
// Work shares of the attention (see attn_phase): which heads workgroup j works on, and for
// one of them which workgroups share it and which key tiles are this workgroup's.
struct AttnHeads {
    int Gx, x, w;      // workgroups per XCD, this workgroup's XCD and its index inside it
    int hx0, Hx;       // first head and number of heads of the XCD
    int h_lo, h_hi;    // this workgroup's heads, local to the XCD (empty if h_lo == h_hi)
};

// (of workgroup w of XCD x, which has Gx of them)
__host__ __device__ __forceinline__ AttnHeads attn_heads(int nh, int x, int w, int Gx)
{
    AttnHeads s;
    s.Gx = Gx;
    s.x = x;
    s.w = w;
    s.hx0 = nh * x >> 3;
    s.Hx = (nh * (x + 1) >> 3) - s.hx0;
    s.h_lo = s.h_hi = 0;
    if (s.Hx == 0) return s;
    if (s.Hx >= Gx) {
        s.h_lo = div_small(s.Hx * w, Gx);
        s.h_hi = div_small(s.Hx * (w + 1), Gx);
    } else {
        s.h_lo = div_small((w + 1) * s.Hx - 1, Gx);    // the head whose run of workgroups contains w
        s.h_hi = s.h_lo + 1;
    }
    return s;
}

struct AttnTiles {
    int first, np, me;   // the head's parts are workgroups first .. first + np - 1; this one is part `me`
    int t0, t1;          // its key tiles (empty, with me >= np, when there are more workgroups than tiles)
};

// tmin: tiles a part should have at least (0: a head is one part).  A part's wavefronts work in parallel, so splitting a
// head further than a unit for each of them only adds to the exchange.
__host__ __device__ __forceinline__ AttnTiles attn_tiles(const AttnHeads& s, int hl, int ntile, int tmin)
{
    AttnTiles t;
    t.first = s.x * s.Gx + s.w;
    t.np = 1;
    t.me = 0;
    if (s.Hx < s.Gx) {
        const int wl0 = div_small(s.Gx * hl, s.Hx);        // head hl's run of local workgroups
        const int wl1 = div_small(s.Gx * (hl + 1), s.Hx);
        t.first = s.x * s.Gx + wl0;
        const int most = tmin == 0 ? 1 : tmin == 1 ? ntile : (ntile + tmin - 1) / tmin;
        t.np = (wl1 - wl0 < most) ? wl1 - wl0 : most;
        t.me = s.w - wl0;
    }
    // boundaries ntile * me / np rounded up: when the tiles do not divide evenly the longer ranges come first,
    // and the last workgroup, whose range ends with the (costlier) tree tile, gets a shorter one
    t.t0 = t.t1 = 0;
    if (t.me < t.np) {
        // ntile = q * np + r.  (The products of the boundaries do not fit div_small.  ntile does - it is below 2^19, since offsets
        // inside a head of 64 channels or more fit 31 bits, which every entry point checks - but with it, fifteen
        // instructions less, calls came out up to 1.5% slower: 40 heads of 64, 33 rows, 6000 cached 18.2 us and 18.5.)
        const int guess = (int)((float)ntile * recip(t.np)), left = ntile - guess * t.np;
        const int more = (int)floorf(((float)left + 0.5f) * recip(t.np));
        const int q = guess + more, r = left - more * t.np;
        t.t0 = q * t.me + div_small(r * t.me + t.np - 1, t.np);
        t.t1 = q * (t.me + 1) + div_small(r * (t.me + 1) + t.np - 1, t.np);
    }
    return t;
}

// A workgroup's heads and its tiles of the first of them.  (The launch that shares itself with the QKV layer has it
// done while its first weights are on their way.)
struct AttnPlan {
    AttnHeads heads;
    AttnTiles tiles;
};
__host__ __device__ __forceinline__ AttnPlan attn_plan(int nh, int ntile, int tmin, int x, int w, int Gx)
{
    AttnPlan p;
    p.heads = attn_heads(nh, x, w, Gx);
    p.tiles = p.heads.h_lo < p.heads.h_hi ? attn_tiles(p.heads, p.heads.h_lo, ntile, tmin) : AttnTiles{};
    return p;
}

// What a launch needs for its first requests of the cache; the rest is in the argument block, read behind them.
struct AttnFirst {
    const half_t *k, *v;
    int64_t k_head, v_head;          // elements from head to head
    uint32_t st_tok, st_ch;          // ... from key to key of K, and from channel to channel of V
    int T, M, nh;                    // keys with the tree's, rows, heads
};

// 2^x for x <= 0 (softmax weights): the hardware instruction; results below the smallest
// normal number flush to zero, which is what a weight that small should be.
__device__ __forceinline__ float fast_exp2(float x) { return __builtin_amdgcn_exp2f(x); }

// op over the four lanes that share lane % 16, in all of them: by swaps of rows of lanes, which leave the
// LDS alone (a shuffle through it waits behind the operands that it is reading: 0.15 us a tile)
template <class Op>
__device__ __forceinline__ float over_groups(float x, Op op)
{
    typedef uint32_t pair __attribute__((ext_vector_type(2)));
    const uint32_t u = __float_as_uint(x);
    const pair a = __builtin_amdgcn_permlane16_swap(u, u, false, false);
    const uint32_t v = __float_as_uint(op(__uint_as_float(a[0]), __uint_as_float(a[1])));
    const pair b = __builtin_amdgcn_permlane32_swap(v, v, false, false);
    return op(__uint_as_float(b[0]), __uint_as_float(b[1]));
}
__device__ __forceinline__ float max_over_groups(float x) { return over_groups(x, [](float a, float b) { return fmaxf(a, b); }); }
__device__ __forceinline__ float sum_over_groups(float x) { return over_groups(x, [](float a, float b) { return a + b; }); }

// Depths, and ancestor sets where they are wanted, by pointer doubling: after round k a node knows how many edges lead to
// its farthest known ancestor, which is up to 2^k edges up, the node above that one (-1 past the root), and which nodes
// lie between.  As many rounds as the deepest node needs; a parent that is not an earlier
// node is taken as "no parent".  A wavefront does it by itself, one or two nodes a lane (i and i + 64), with exchanges of
// lanes instead of LDS arrays and two barriers a round.  Nodes from 64 on double among themselves; what lies above the
// node at which they leave for the first 64 is added at the end (both halves in one: 20 exchanges a round instead of 6, and
// calls of 65 to 128 rows under a chain 0.7 us slower than with barriers).
template <int NODES>
struct TreeNodes {
    int link[NODES];          // depth << 8 | up + 1
    uint64_t own[NODES];      // ancestors-or-self among the node's own 64
    uint64_t first;           // ... and, of the second node, among the first 64
    __device__ __forceinline__ int depth(int node) const
    {
        const int a = __shfl(link[0], node & 63), b = __shfl(link[NODES - 1], node & 63);
        return (node < 64 ? a : b) >> 8;
    }
};
// (up0, up1: parent[lane] and parent[lane + 64]; what they are from M on is not looked at)
template <int NODES, bool SETS>
__device__ __forceinline__ TreeNodes<NODES> tree_nodes(int up0, int up1, int M, int lane)
{
    static_assert(GHD_MAX_M == 128, "two nodes a lane; up + 1 fits 8 bits");
    TreeNodes<NODES> t;
    t.first = 0;
    bool on[NODES], any = false;                 // whether the node above is one of the same 64
    auto look = [&]() {
        any = false;
#pragma unroll
        for (int u = 0; u < NODES; ++u) {
            on[u] = (t.link[u] & 255) > u * 64;
            any = any || on[u];
        }
    };
#pragma unroll
    for (int u = 0; u < NODES; ++u) {
        const int i = u * 64 + lane, up = u ? up1 : up0;
        t.link[u] = i < M && up >= 0 && up < i ? 1 << 8 | (up + 1) : 0;
        t.own[u] = 1ull << lane;
    }
    for (look(); __ballot(any); look()) {
#pragma unroll
        for (int u = 0; u < NODES; ++u) {
            const int from = on[u] ? (t.link[u] & 255) - 1 - u * 64 : 0, o = __shfl(t.link[u], from);
            if constexpr (SETS) {
                const uint64_t more = __shfl(t.own[u], from);
                if (on[u]) t.own[u] |= more;
            }
            if (on[u]) t.link[u] = ((t.link[u] & ~255) + (o & ~255)) | (o & 255);
        }
    }
    if constexpr (NODES > 1) {
        const int up = t.link[1] & 255, from = up ? up - 1 : 0, o = __shfl(t.link[0], from);
        if (up) t.link[1] += o & ~255;
        if constexpr (SETS) {
            const uint64_t more = __shfl(t.own[0], from);
            if (up) t.first = more;
        }
    }
    return t;
}

// Node `lane` (and lane + 64) to its mask (low and high word)
template <int NODES, class Mask>
__device__ __forceinline__ void store_masks(const TreeNodes<NODES>& t, int M, int lane, Mask mask)
{
#pragma unroll
    for (int u = 0; u < NODES; ++u) {
        const int i = u * 64 + lane;
        if (i >= M) continue;
        mask[2 * i] = u ? t.first : t.own[0];
        mask[2 * i + 1] = u ? t.own[u] : 0;
    }
}

// A call in one launch gets what its masks are made from before anything else, and has it when
// it requests queries and cache (the work shares are worked out in between): the masks are then made while those are on
// their way.  Loads return in order: requested behind the cache, parent[] came back behind it, and the
// rounds of the doubling began when all else was there.  Masks: a word a thread; parent[]: the first wavefront has all of it.
template <bool TWO>
__device__ __forceinline__ void mask_source(Ctx& cx, const void* source, int M)
{
    const int tid = threadIdx.x, n = cx.parents ? min(M, 64) : M * 4;
    const auto words = gp((const uint32_t*)source);
    cx.source[0] = tid < n ? (int)words[tid] : 0;
    cx.source[1] = TWO && cx.parents && tid < 64 && tid + 64 < M ? (int)words[tid + 64] : 0;
}
// (The first wavefront makes a tree's masks in registers: reads of LDS arrays would wait for all that is on its way to the
// LDS.  us a call under a wide tree, from a graph, with the doubling in LDS arrays and now: 32 heads of 128, 4 rows, 120
// cached 6.5 and 6.3; 32 of 64, 64 rows, 128 cached 7.2 and 6.5; 8 of 128, 128 rows, 60 cached 11.7 and 11.1, under a
// chain 12.1 and 11.7)
template <bool TWO>
__device__ __forceinline__ void masks_from_source(bool parents, int M, const int (&word)[2], uint64_t* mask)
{
    const int tid = threadIdx.x;
    if (!parents) {
        if (tid < M * 4) ((uint32_t*)mask)[tid] = (uint32_t)word[0];
    } else if (tid < 64) {
        constexpr int NODES = TWO ? 2 : 1;
        store_masks(tree_nodes<NODES, true>(word[0], word[1], M, tid), M, tid, mask);
    }
}

// Which of the eight keys from `key` on a row sees, a bit each, by its mask in the LDS (four words; bits from M on are
// never looked at): committed keys, and of the tree's rows those of the mask; none from T on.  (One shift across two
// words for the eight instead of one of 64 bits and two choices for each: an instruction here is a wait of the whole
// call.  40 heads of 128, 4 rows, 300 cached 9.14 us and 9.49; a 7B-shaped layer of 16 rows 87.3 and 87.9.)
__device__ __forceinline__ uint32_t seen_keys(const uint32_t* mask, int key, int kv_len, int T)
{
    const int jn = key - kv_len, at = max(jn, 0), w = min(at >> 5, 3);
    const uint32_t lo = mask[w], hi = w < 3 ? mask[min(w + 1, 3)] : 0u;
    uint32_t bits = __builtin_amdgcn_alignbit(hi, lo, (uint32_t)at);       // (by at modulo 32)
    if (jn < 0) bits = jn <= -8 ? 0xffu : bits << -jn | ((1u << -jn) - 1);
    return bits & ((1u << min(max(T - key, 0), 8)) - 1);
}

// `gate` is called once by every workgroup (all threads), before the first read of q or of a
// cache row from kv_len on; it returns false if the launch is to be abandoned.  A kernel that
// produces those in the same launch waits there for their producers; with PREFETCH a
// wavefront's first unit is requested before the gate if it lies wholly below kv_len (rows of
// earlier steps), so that it arrives while the workgroup waits.
struct NoGate {
    __device__ __forceinline__ bool operator()() const { return true; }
};

// Adds a unit of 32 keys to a running state: scores s (times log2 e; -inf where a row does not see the key), their
// largest `tmax` in all four lanes of a row, V^T operands vf.  The probabilities of the product are fp16, and the
// largest of those that share a maximum is exactly 1, so the more keys share one the more is rounded.  APART:
// the unit's probabilities are taken against its own maximum and its product is added to the state in fp32.
// So do calls in one launch, since a head split over workgroups would have given each unit a state of its own:
// without it their outputs were 0.7% (up to 32 rows) and 1.1% (33 to 64) further from 64 bits than in two
// launches, 4% at the worst.  (32 heads of 128: 48 rows, 4 tiles 10.3 -> 10.6 us a call, in two launches 11.6;
// 128 rows, 3 tiles 12.4 -> 12.9 and 14.5; 32 rows, 6 tiles 13.8 -> 14.3 and 15.6.)
template <int DT, bool APART>
__device__ __forceinline__ void add_unit(float& mrun, float& lrun, floatx4 (&oacc)[DT], const floatx4 (&s)[2],
                                         const half8 (&vf)[DT], float tmax)
{
    const float mnew = fmaxf(mrun, tmax);
    const float muse = (mnew == -INFINITY) ? 0.f : mnew;
    const float alpha = fast_exp2(mrun - muse);
    const float mine = APART && tmax != -INFINITY ? tmax : muse;
    mrun = mnew;
    float lsum = 0.f;
    half8 pf;
#pragma unroll
    for (int i = 0; i < 8; ++i) {
        const float pv = fast_exp2(s[i >> 2][i & 3] - mine);
        lsum += pv;
        pf[i] = (half_t)pv;
    }
    // (the maximum of most rows settles early: usually nothing has to be rescaled)
    if (__ballot(alpha != 1.0f)) {
#pragma unroll
        for (int e = 0; e < DT; ++e) oacc[e] *= alpha;
    }
    if constexpr (APART) {
        const float beta = fast_exp2(mine - muse);
        lrun = lrun * alpha + lsum * beta;
#pragma unroll
        for (int e = 0; e < DT; ++e) {
            const floatx4 o = __builtin_amdgcn_mfma_f32_16x16x32_f16(vf[e], pf, (floatx4){0.f, 0.f, 0.f, 0.f}, 0, 0, 0);
            oacc[e] += o * beta;
        }
    } else {
        lrun = lrun * alpha + lsum;
#pragma unroll
        for (int e = 0; e < DT; ++e) oacc[e] = __builtin_amdgcn_mfma_f32_16x16x32_f16(vf[e], pf, oacc[e], 0, 0, 0);
    }
}

// ---- up to 32 query rows: every wavefront works on units of its own ----------------------
// a part should have a unit for each of the eight wavefronts
constexpr int kDirectTiles = 4;

template <int MT, int D>
struct DirectLds {
    floatx4 o[8][MT][D / 16][64];                    // the wavefronts' outputs, when they are merged
    float m[8][MT][16], l[8][MT][16];                // ... and their softmax statistics
    uint64_t mask[MT * 16][2];
    int wait_ok;                                     // thread 0's verdict on a bounded wait, for the whole workgroup
};

// v, of which the compiler then knows nothing: what is worked out from it is worked out where
// it is used, not ahead of a loop in registers that the loop needs
__device__ __forceinline__ int hidden(int v)
{
    asm volatile("" : "+v"(v));
    return v;
}

// four columns of a row of the attention's output
__device__ __forceinline__ void store_attn_out(const FusedArgs& a, GLOBAL half_t* out, int m, int col, floatx4 v)
{
    const half4 h = {(half_t)v[0], (half_t)v[1], (half_t)v[2], (half_t)v[3]};
    const size_t at = a.att_out_packed ? xpk_index(m, col, a.Mpad >> 4) : (size_t)m * a.nh * a.d + col;
    *(GLOBAL half4*)(out + at) = h;
}

// The end of a head that the workgroups first .. first + np - 1 share, of which this is number `me`: once
// the partial states of all are stored, each merges its share of the rows.  Returns false if they never
// came.
template <int D>
__device__ __forceinline__ bool finish_parts(const FusedArgs& a, GLOBAL half_t* out, int head, int first, int np, int me,
                                             uint32_t epoch, int* wait_ok)
{
    const int tid = hidden(threadIdx.x), M = a.M, Mpad = a.Mpad;
    const auto o_part = gp(a.o_part), ml_part = gp(a.ml_part);
    wait_own_stores();
    __syncthreads();   // partial state acknowledged by the L2
    uint32_t* const cnt = a.sync + kCntAttn + head * kCntStride;
    const int r0 = M * me / np, r1 = M * (me + 1) / np;        // the rows this part merges
    if (tid == 0) {
        uint32_t* const word = epoch_word(cnt, epoch);
        const uint32_t seen = arrive(word);
        if (r0 < r1) *wait_ok = bounded_wait(a.sync, word, seen, (uint32_t)np, (uint32_t)np, 2000u);
        if (me == 0) clear_next(cnt, epoch);
    }
    if (r0 >= r1) return true;
    __syncthreads();
    if (!*wait_ok) return false;    // the other parts never arrived: nothing sensible to write
    // a thread per four channels of a row; parts in index order, eight of them in flight
    constexpr int CH = D / 4;
    for (int i = tid; i < (r1 - r0) * CH; i += kFT) {
        const int m = r0 + i / CH, ch = i % CH * 4;
        float mx = -INFINITY, den = 0.f;
        floatx4 num = {0.f, 0.f, 0.f, 0.f};
        for (int p0 = 0; p0 < np; p0 += 8) {
            floatx2 ml[8];
            floatx4 o[8];
#pragma unroll
            for (int p = 0; p < 8; ++p) {
                const size_t row = (size_t)(first + min(p0 + p, np - 1)) * Mpad + m;
                ml[p] = *(GLOBAL const floatx2*)(ml_part + row * 2);
                o[p] = *(GLOBAL const floatx4*)(o_part + row * D + ch);
            }
            float mnew = mx;
#pragma unroll
            for (int p = 0; p < 8; ++p) mnew = fmaxf(mnew, ml[p][0]);
            const float w0 = (mx == -INFINITY) ? 0.f : fast_exp2(mx - mnew);
            mx = mnew;
            num *= w0;
            den *= w0;
#pragma unroll
            for (int p = 0; p < 8; ++p) {
                const float w = (p0 + p >= np || ml[p][0] == -INFINITY) ? 0.f : fast_exp2(ml[p][0] - mx);
                den += w * ml[p][1];
                num += w * o[p];
            }
        }
        // (a row that sees no key at all, possible with a caller's mask and an empty cache, gets zeros)
        store_attn_out(a, out, m, head * D + ch, den > 0.f ? num / den : (floatx4){0.f, 0.f, 0.f, 0.f});
    }
    return true;
}

template <int MT, int D, bool PREFETCH, bool ALONE, class Late, class Gate>
__device__ __forceinline__ bool attn_direct(const AttnFirst& f, Late late, Ctx& cx, const AttnPlan& plan, Gate gate)
{
    constexpr int DS = D / 32, DT = D / 16;
    DirectLds<MT, D>& sm = *reinterpret_cast<DirectLds<MT, D>*>(cx.lds);

    const int tid = threadIdx.x;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int M = f.M, nh = f.nh, T = f.T, kv_len = T - M;
    constexpr int Mpad = MT * 16;
    const auto kc = gp(f.k), vc = gp(f.v);
    const int ntile = (T + 63) >> 6, nunit = (T + 31) >> 5;
    const uint32_t st_tok = f.st_tok, st_ch = f.st_ch;

    // Work shares.  Heads are dealt to the 8 XCDs in contiguous blocks.  Inside an XCD a
    // workgroup works on one head at a time: with fewer heads than workgroups, every head
    // gets its own run of workgroups, each taking a contiguous range of the head's key
    // tiles; otherwise every workgroup takes whole heads.  A head is therefore always
    // finished inside one XCD (partial states go through that XCD's L2).
    const AttnHeads hs = plan.heads;
    const int hx0 = hs.hx0, h_lo = hs.h_lo, h_hi = hs.h_hi;
    // (bits from M on, which a caller's mask may have set, are never looked at: a mask bit is
    // only consulted for keys kv_len <= key < kv_len + M)
    uint64_t mask_lo = 0, mask_hi = 0;
    auto request_masks = [&]() {
        const auto mask = gp(late().mask);
        if (tid < M && !ALONE) {
            mask_lo = mask[2 * tid];
            mask_hi = mask[2 * tid + 1];
        }
    };
    if constexpr (PREFETCH) request_masks();

    bool gated = false;
    for (int hl = h_lo; hl < (PREFETCH ? min(h_hi, h_lo + 1) : h_hi); ++hl) {
        const int lane = hidden(threadIdx.x & 63), c = lane & 15, g4 = lane >> 4;
        const int head = hx0 + hl;
        // the workgroups first .. first + np - 1 split this head's tiles
        const AttnTiles ts = hl == h_lo ? plan.tiles : attn_tiles(hs, hl, ntile, kDirectTiles);
        const int first = ts.first, np = ts.np, me = ts.me;
        if (me >= np) continue;                            // more workgroups than parts
        const auto kh = kc + (int64_t)head * f.k_head;
        const auto vh = vc + (int64_t)head * f.v_head;
        const int u1 = min(2 * ts.t1, nunit);
        int u = 2 * ts.t0 + wave;                          // this wavefront's unit

        // A unit's K: row i of S^T's 16-key tile jx is key (i / 4) * 8 + jx * 4 + i % 4, so that
        // lane group g4 gets the scores of keys g4 * 8 .. + 7 in order.  Rows past the last key
        // read the last one.  V^T: 8 keys of a channel; pieces past the capacity, which hold no
        // key, read the last piece.
        // (Offsets inside a head fit 32 bits: checked on the host.)
        half8 kf[2][DS], vf[DT];
        auto load16 = [&](GLOBAL const char* base, uint32_t off) {
            return *(GLOBAL const half8*)(base + off);
        };
        auto load_k = [&](int unit) {
#pragma unroll
            for (int jx = 0; jx < 2; ++jx) {
                const int key = min(unit * 32 + (c >> 2) * 8 + jx * 4 + (c & 3), T - 1);
                const uint32_t off = ((uint32_t)key * st_tok + g4 * 8) * 2;
#pragma unroll
                for (int ds = 0; ds < DS; ++ds) kf[jx][ds] = load16((GLOBAL const char*)kh + ds * 64, off);
            }
        };
        auto load_v = [&](int unit) {
            const uint32_t off = (c * st_ch + min((uint32_t)(unit * 32 + g4 * 8), st_ch - 8)) * 2;
#pragma unroll
            for (int e = 0; e < DT; ++e) vf[e] = load16((GLOBAL const char*)vh + (size_t)(e * 16 * st_ch) * 2, off);
        };
        // Requests, in order: [a unit known before the gate] gate, queries, [the unit otherwise].  Without a gate the
        // first unit is requested before the argument block is read.  With one, no
        // cache line of a unit that ends 64 rows or more below kv_len can hold a row that this
        // launch writes, whatever the strides and the alignment of the cache.
        const bool early = !gated && u < u1 && (!PREFETCH || u * 32 + 96 <= kv_len);
        if (early) {
            load_k(u);
            load_v(u);
            pin_order();
        }
        if (!gated) {
            if (!gate()) return false;
            if constexpr (!PREFETCH) request_masks();
            gated = true;
        }
        const FusedArgs& a = late();
        const float scale_log2e = a.scale_log2e;
        const auto q = gp(a.att_q);
        const auto out = gp(a.att_out);
        const auto o_part = gp(a.o_part), ml_part = gp(a.ml_part);
        int source[2] = {0, 0};
        if constexpr (ALONE) {
            source[0] = hidden(cx.source[0]);              // (it is there)
            if constexpr (MT > 4) source[1] = hidden(cx.source[1]);
            pin_order();
        }
        half8 qf[MT][DS];
#pragma unroll
        for (int t = 0; t < MT; ++t) {
            const int row = t * 16 + c;
#pragma unroll
            for (int ds = 0; ds < DS; ++ds) {
                half8 v = {0, 0, 0, 0, 0, 0, 0, 0};
                if (row < M) v = *(GLOBAL const half8*)(q + ((size_t)row * nh + head) * D + ds * 32 + g4 * 8);
                qf[t][ds] = v;
            }
        }
        pin_order();
        if (!early && u < u1) {
            load_k(u);
            load_v(u);
        }
        pin_order();           // (all requests are out before the first of them is waited for)
        if constexpr (ALONE) masks_from_source<false>(cx.parents, M, source, &sm.mask[0][0]);
        else if (tid < MT * 16) {
            sm.mask[tid][0] = mask_lo;
            sm.mask[tid][1] = mask_hi;
        }

        // running state of this head
        float mrun[MT], lrun[MT];
        floatx4 oacc[MT][DT];
#pragma unroll
        for (int t = 0; t < MT; ++t) {
            mrun[t] = -INFINITY;
            lrun[t] = 0.f;
#pragma unroll
            for (int e = 0; e < DT; ++e) oacc[t][e] = (floatx4){0.f, 0.f, 0.f, 0.f};
        }
        __syncthreads();                                   // the masks are in LDS

        for (; u < u1; u += 8) {
            const int c = hidden(lane) & 15, g4 = hidden(lane) >> 4;
            const int key0 = u * 32;
            const bool committed = key0 + 32 <= kv_len;    // every key visible to every row
            floatx4 s[MT][2];
#pragma unroll
            for (int t = 0; t < MT; ++t) {
#pragma unroll
                for (int jx = 0; jx < 2; ++jx) {
                    s[t][jx] = (floatx4){0.f, 0.f, 0.f, 0.f};
#pragma unroll
                    for (int ds = 0; ds < DS; ++ds)
                        s[t][jx] = __builtin_amdgcn_mfma_f32_16x16x32_f16(kf[jx][ds], qf[t][ds], s[t][jx], 0, 0, 0);
                }
            }
            if (u + 8 < u1) load_k(u + 8);
            if (key0 + 32 > T) {
                // keys from T on hold no data: zero them, a stray NaN times a zero weight is a NaN
                const int nvalid = T - key0 - g4 * 8;
#pragma unroll
                for (int e = 0; e < DT; ++e)
#pragma unroll
                    for (int i = 0; i < 8; ++i)
                        if (i >= nvalid) vf[e][i] = (half_t)0;
            }
#pragma unroll
            for (int t = 0; t < MT; ++t) {
                float tmax = -INFINITY;
                bool any = true;
                if (committed) {
#pragma unroll
                    for (int jx = 0; jx < 2; ++jx) {
                        s[t][jx] *= scale_log2e;
                        tmax = fmaxf(tmax, fmaxf(fmaxf(s[t][jx][0], s[t][jx][1]), fmaxf(s[t][jx][2], s[t][jx][3])));
                    }
                } else {
                    const int row = t * 16 + c;
                    const uint32_t seen = seen_keys((const uint32_t*)sm.mask[row], key0 + g4 * 8, kv_len, T);
                    const bool mine = seen != 0 && row < M;
#pragma unroll
                    for (int i = 0; i < 8; ++i) {
                        const float v = seen >> i & 1 ? s[t][i >> 2][i & 3] * scale_log2e : -INFINITY;
                        s[t][i >> 2][i & 3] = v;
                        tmax = fmaxf(tmax, v);
                    }
                    any = __ballot(mine) != 0ull;          // no row of the tile sees the unit: leave it out
                }
                if (!any) continue;
                add_unit<DT, ALONE>(mrun[t], lrun[t], oacc[t], s[t], vf, max_over_groups(tmax));
            }
            if (u + 8 < u1) load_v(u + 8);
        }

        // ---- the wavefronts' states meet in LDS and are merged in wavefront order; a head in one
        //      part is finished by that
        const int lane_ = hidden(lane);
        {
        const int lane = lane_, c = lane & 15, g4 = lane >> 4;
#pragma unroll
        for (int t = 0; t < MT; ++t) {
            const float l = sum_over_groups(lrun[t]);
            if (lane < 16) {
                sm.m[wave][t][c] = mrun[t];
                sm.l[wave][t][c] = l;
            }
        }
#pragma unroll
        for (int t = 0; t < MT; ++t)
#pragma unroll
            for (int e = 0; e < DT; ++e) sm.o[wave][t][e][lane] = oacc[t][e];
        __syncthreads();
        for (int i = wave; i < MT * DT; i += 8) {
            const int e = i % DT, t = i / DT, m = t * 16 + c;
            float mw[8], mx = -INFINITY, l = 0.f;
#pragma unroll
            for (int k = 0; k < 8; ++k) {
                mw[k] = sm.m[k][t][c];
                mx = fmaxf(mx, mw[k]);
            }
            floatx4 o = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
            for (int k = 0; k < 8; ++k) {
                const float w = (mw[k] == -INFINITY) ? 0.f : fast_exp2(mw[k] - mx);
                l += sm.l[k][t][c] * w;
                o += sm.o[k][t][e][lane] * w;
            }
            if (m >= M) continue;
            if (np == 1) {
                // (a row that sees no key at all, possible with a caller's mask and an empty
                // cache, gets zeros)
                store_attn_out(a, out, m, head * D + e * 16 + g4 * 4, l > 0.f ? o / l : (floatx4){0.f, 0.f, 0.f, 0.f});
            } else {
                const size_t row = (size_t)cx.j * Mpad + m;
                *(GLOBAL floatx4*)(o_part + row * D + e * 16 + g4 * 4) = o;
                if (e == 0 && g4 == 0) *(GLOBAL floatx2*)(ml_part + row * 2) = (floatx2){mx, l};
            }
        }
        }
        if (np > 1 && !finish_parts<D>(a, out, head, first, np, me, a.att_epoch, &sm.wait_ok)) return false;
        // a workgroup that goes on to another head reuses its LDS and its partial-state slot
        // (a workgroup with several heads has them to itself: np = 1)
        if (hl + 1 < h_hi) __syncthreads();
    }
    // a workgroup without a share of any head still checks in
    if (!gated && !gate()) return false;
    return true;
}

// ---- more query rows: tiles in LDS, shared by the wavefronts -----------------------------------
template <int MT, int D>
struct StagedLds {
    static constexpr int NB = D == 128 ? 4 : 8;        // tile buffers
    static constexpr uint32_t KB = 64 * D * 2;         // bytes of a tile's K, and of its V^T
    char tile[NB][2 * KB];
    alignas(8) uint32_t mask[GHD_MAX_M * 4];
    int wait_ok;                                       // thread 0's verdict on a bounded wait, for the whole workgroup
    // what the two wavefronts of a row tile exchange when a head ends: their softmax statistics and, in a
    // tile buffer that is free then, half of their output fragments
    float m[4][2][16], l[4][2][16];
    typedef floatx4 HalfOut[4][2][D / 32][64];
    static_assert(sizeof(HalfOut) <= 2 * KB, "fits a buffer");
};

// 16 bytes a lane from base + off straight into the LDS, lane after lane from `lds` on (the same for all
// lanes): no registers.  The waits for it are written out (wait_loads, then a barrier).
typedef __attribute__((address_space(3))) void* LdsPtr;
__device__ __forceinline__ void to_lds(GLOBAL const char* base, uint32_t off, uint32_t lds)
{
    __builtin_amdgcn_global_load_lds((GLOBAL void*)(base + off), (LdsPtr)(uintptr_t)lds, 16, 0, 0);
}
__device__ __forceinline__ void to_lds_nt(GLOBAL const char* base, uint32_t off, uint32_t lds)     // non-temporal
{
    __builtin_amdgcn_global_load_lds((GLOBAL void*)(base + off), (LdsPtr)(uintptr_t)lds, 16, 0, 2);
}
__device__ __forceinline__ void to_lds_word(GLOBAL const char* base, uint32_t off, uint32_t lds)   // 4 bytes a lane
{
    __builtin_amdgcn_global_load_lds((GLOBAL void*)(base + off), (LdsPtr)(uintptr_t)lds, 4, 0, 0);
}
// waits until at most n of this wavefront's loads are on their way
template <int N>
__device__ __forceinline__ void wait_loads()
{
    static_assert(N < 64, "six bits");
    __builtin_amdgcn_s_waitcnt(0x0F70 | (N & 15) | (N >> 4) << 14);
}

// ... until all but its youngest n tiles are there (n <= MOST; uniform)
template <int PER_TILE, int MOST>
__device__ __forceinline__ void wait_tiles_of(int n)
{
    if constexpr (MOST > 0) {
        if (n < MOST) return wait_tiles_of<PER_TILE, MOST - 1>(n);
    }
    wait_loads<PER_TILE * MOST>();
}

template <int MT, int D, bool PREFETCH, bool ALONE, class Late, class Gate>
__device__ __forceinline__ bool attn_staged(const AttnFirst& f, Late late, Ctx& cx, const AttnPlan& plan, Gate gate)
{
    constexpr int DS = D / 32, DT = D / 16;
    constexpr int HALVES = MT <= 4 ? 2 : 1;            // wavefronts that share a row tile, each for its keys
    constexpr int UNITS = 2 / HALVES;                  // 32-key units of a tile that a wavefront works on
    constexpr int PIECES = D / 64;                     // 1 KiB pieces of a tile's K that a wavefront requests (as many of V)
    constexpr int LPT = 2 * PIECES;                    // loads per tile
    // Masked units by seen_keys(), except with 128 channels up to 64 rows: there the loop over the other tiles comes out
    // slower beside it, and calls of many tiles lose what those of few win.  us a call, by the masks' words and by seen_keys:
    // 4 heads, 48 rows, 16000 cached 19.5 and 19.8; 24, 3001 cached 15.4 and 15.5; 32, 64 rows, 2048 cached 15.6 and 15.7, 120
    // cached 9.15 and 8.7; 64, 900 cached 15.5 and 15.3; 2, 40 rows, 1000 cached 10.4 and 10.1.  Elsewhere: 8 heads of
    // 128, 128 rows, 60 cached 12.5 and 11.4; 16, 3000 cached 19.0 and 18.8; 16 heads of 64, 64 rows, 700 cached 10.0 and
    // 9.6; 40, 33 rows, 6000 cached 19.0 and 18.9.
    constexpr bool COMPACT = HALVES == 1 || D == 64;
    using L = StagedLds<MT, D>;
    constexpr int NB = L::NB;
    constexpr uint32_t KB = L::KB, TB = 2 * KB;
    L& sm = *reinterpret_cast<L*>(cx.lds);
    const uint32_t lds0 = (uint32_t)(uintptr_t)(__attribute__((address_space(3))) char*)cx.lds;

    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int c = lane & 15, g4 = lane >> 4;
    const int wq = HALVES == 2 ? wave & 3 : wave, half = HALVES == 2 ? wave >> 2 : 0;    // row tile, key half
    const int M = f.M, nh = f.nh, T = f.T, kv_len = T - M;
    constexpr int Mpad = MT * 16;
    const auto kc = gp(f.k), vc = gp(f.v);
    const int ntile = (T + 63) >> 6;
    const int mrow = wq * 16 + c;
    const bool mok = mrow < M, wave_active = wq * 16 < M;
    const AttnHeads hs = plan.heads;
    const int hx0 = hs.hx0, h_lo = hs.h_lo, h_hi = hs.h_hi;

    // What this lane requests of every tile.  A KiB of the LDS is 8 (or 4) consecutive rows of a tile: K
    // rows are keys, V^T rows channels.  The 16-byte pieces of a row lie in an order of their own
    // (piece p of row r in place p ^ f(r)), so that the 16 rows that an MFMA operand takes the same
    // piece of are spread over all banks.
    constexpr int KR = 512 / D;                        // K rows of a KiB: 4 or 8
    const uint32_t st_tok2 = f.st_tok * 2, st_ch2 = f.st_ch * 2;
    const int k_row = wave * PIECES * KR + lane / (D / 8);                   // (piece i: i * KR rows on)
    const uint32_t k_piece = D == 128 ? (uint32_t)((lane & 15) ^ ((lane >> 4) | (wave & 3) << 2)) * 16
                                      : (uint32_t)((lane & 7) ^ (((lane >> 4) & 1) | (wave & 3) << 1)) * 16;
    const int v_ch = wave * PIECES * 8 + (lane >> 3);                        // (piece i: i * 8 channels on)
    const uint32_t v_last = st_ch2 - 16;
    // where it finds the operands of its MFMAs (see attn_direct: row i of S^T's 16-key tile jx is key
    // (i / 4) * 8 + jx * 4 + i % 4 of a unit)
    uint32_t k_at[DS], v_at[2];
#pragma unroll
    for (int ds = 0; ds < DS; ++ds)
        k_at[ds] = (uint32_t)((c >> 2) * 8 + (c & 3)) * (D * 2) + (uint32_t)((ds * 4 + g4) ^ (D == 128 ? c : c >> 1)) * 16;
#pragma unroll
    for (int un = 0; un < 2; ++un) v_at[un] = KB + (uint32_t)c * 128 + (uint32_t)((un * 4 + g4) ^ (c >> 1)) * 16;

    // the masks of all rows, four words each: a word a thread (rows past the last read the last word;
    // bits from M on, which a caller's mask may have set, are never looked at)
    auto request_masks = [&]() {
        to_lds_word((GLOBAL const char*)gp(late().mask), (uint32_t)min(tid, M * 4 - 1) * 4, lds0 + (uint32_t)offsetof(L, mask) + wave * 256);
    };

    bool gated = false;
    for (int hl = h_lo; hl < (PREFETCH ? min(h_hi, h_lo + 1) : h_hi); ++hl) {
        const int head = hx0 + hl;
        // the workgroups first .. first + np - 1 split this head's tiles
        const AttnTiles ts = hl == h_lo ? plan.tiles : attn_tiles(hs, hl, ntile, 1);
        const int first = ts.first, np = ts.np, me = ts.me, t0 = ts.t0, t1 = ts.t1;
        if (me >= np) continue;                            // more workgroups than tiles
        const auto kh = (GLOBAL const char*)(kc + (int64_t)head * f.k_head);
        const auto vh = (GLOBAL const char*)(vc + (int64_t)head * f.v_head);

        // Keys from T on read the last one; V^T pieces past the capacity, which hold no key, the last
        // piece.  (Offsets inside a head fit 32 bits: checked on the host.)
        auto request = [&](int tile) {
            const uint32_t at = lds0 + (uint32_t)((tile - t0) & (NB - 1)) * TB + (uint32_t)wave * (PIECES * 1024);
#pragma unroll
            for (int i = 0; i < PIECES; ++i)
                to_lds_nt(kh, (uint32_t)min(tile * 64 + k_row + i * KR, T - 1) * st_tok2 + k_piece, at + i * 1024);
#pragma unroll
            for (int i = 0; i < PIECES; ++i) {
                const int ch = v_ch + i * 8;
                const uint32_t key2 = (uint32_t)tile * 128 + (uint32_t)((lane & 7) ^ ((ch >> 1) & 7)) * 16;
                to_lds_nt(vh, (uint32_t)ch * st_ch2 + min(key2, v_last), at + KB + i * 1024);
            }
        };
        // Requests, in order: [tiles known before the gate] gate, queries, [the rest].  Without a gate the first tile is
        // requested before the argument block is read.  With one, a tile is known
        // if it ends at least 64 rows below kv_len: no cache line of it holds a row that this launch
        // writes, whatever the strides and the alignment of the cache.  The queries take the last
        // buffer until its first tile is requested; every wavefront brings its own.
        const int up_front = min(t1 - t0, NB - 1);
        int n_pre = 0;
        if (!gated) {
            // (loads return in order: the wavefront that polls at the gate requests nothing before)
            const bool polls = PREFETCH && wave == 0;
            if constexpr (!PREFETCH) request(t0), n_pre = 1, pin_order();
            if (!polls && !ALONE) request_masks();
            if constexpr (PREFETCH)
                for (; !polls && n_pre < up_front && (t0 + n_pre) * 64 + 128 <= kv_len; ++n_pre) request(t0 + n_pre);
            if (!gate()) return false;
            gated = true;
            if (polls) request_masks();
        }
        const FusedArgs& a = late();
        const float scale_log2e = a.scale_log2e;
        const auto q = gp(a.att_q);
        const auto out = gp(a.att_out);
        const auto o_part = gp(a.o_part), ml_part = gp(a.ml_part);
        int source[2] = {0, 0};
        if constexpr (ALONE) {
            source[0] = hidden(cx.source[0]);              // (it is there)
            if constexpr (MT > 4) source[1] = hidden(cx.source[1]);
            pin_order();
        }
        {
            const uint32_t at = lds0 + (NB - 1) * TB + (uint32_t)wave * (DS * 1024);
            const uint32_t off = ((uint32_t)min(mrow, M - 1) * (uint32_t)nh + (uint32_t)head) * (D * 2) + g4 * 16;
#pragma unroll
            for (int ds = 0; ds < DS; ++ds) to_lds((GLOBAL const char*)q, off + ds * 64, at + ds * 1024);
        }
        for (int n = n_pre; n < up_front; ++n) request(t0 + n);

        if constexpr (ALONE) masks_from_source<(MT > 4)>(cx.parents, M, source, (uint64_t*)sm.mask);

        // waits for all but the youngest n tiles
        auto wait_tiles = [&](int n) {
            wait_tiles_of<LPT, NB - 2>(n);
            pin_order();
        };
        // running state of this head: one for each unit of a tile, which come together when the head ends
        // (one for both rounds more, see add_unit: outputs 1.8% further from 64 bits at 65 to 128 rows, and a
        // 7B-shaped layer of 128 rows took 0.3 us of 152 less)
        constexpr int STATES = ALONE ? 1 : UNITS;
        float mrun[STATES], lrun[STATES];
        floatx4 oacc[STATES][DT];
#pragma unroll
        for (int uu = 0; uu < STATES; ++uu) {
            mrun[uu] = -INFINITY;
            lrun[uu] = 0.f;
#pragma unroll
            for (int e = 0; e < DT; ++e) oacc[uu][e] = (floatx4){0.f, 0.f, 0.f, 0.f};
        }
        wait_tiles(up_front - max(n_pre, 1));              // the queries and the first tile are there
        half8 qf[DS];
        {
            const char* at = sm.tile[NB - 1] + wave * (DS * 1024) + lane * 16;
#pragma unroll
            for (int ds = 0; ds < DS; ++ds) qf[ds] = *(const half8*)(at + ds * 1024);
        }

        for (int tile = t0; tile < t1; ++tile) {
            // A barrier a tile: the tile is there for everybody, and everybody is done with the one before,
            // whose buffer is requested into.
            if (tile > t0) wait_tiles(min(t1 - 1 - tile, NB - 2));
            barrier_lds();
            if (tile + NB - 1 < t1) request(tile + NB - 1);
            if (!wave_active) continue;
            const char* const buf = sm.tile[(tile - t0) & (NB - 1)];
#pragma unroll STATES
            for (int uu = 0; uu < UNITS; ++uu) {
                const int un = HALVES == 2 ? half : uu, key0 = tile * 64 + un * 32;
                const char* const kp = buf + un * (32 * D * 2);
                const char* const vp = buf + (un ? v_at[1] : v_at[0]);
                // (all of K is read before the first product: left to itself the compiler waits for it in two goes;
                // 30 heads of 64, 43 rows, 6442 cached 18.65 us and 18.4, 24 of 128, 48 rows, 3001 cached 16.5 and 16.1)
                half8 kf[2][DS];
#pragma unroll
                for (int ds = 0; ds < DS; ++ds)
#pragma unroll
                    for (int jx = 0; jx < 2; ++jx) kf[jx][ds] = *(const half8*)(kp + k_at[ds] + jx * (4 * D * 2));
                __builtin_amdgcn_sched_barrier(0);
                floatx4 s[2];
#pragma unroll
                for (int jx = 0; jx < 2; ++jx) {
                    s[jx] = (floatx4){0.f, 0.f, 0.f, 0.f};
#pragma unroll
                    for (int ds = 0; ds < DS; ++ds) s[jx] = __builtin_amdgcn_mfma_f32_16x16x32_f16(kf[jx][ds], qf[ds], s[jx], 0, 0, 0);
                }
                half8 vf[DT];
#pragma unroll
                for (int e = 0; e < DT; ++e) vf[e] = *(const half8*)(vp + e * 2048);
                float tmax = -INFINITY;
                if (key0 + 32 <= kv_len) {                 // every key visible to every row
#pragma unroll
                    for (int jx = 0; jx < 2; ++jx) {
                        s[jx] *= scale_log2e;
                        tmax = fmaxf(tmax, fmaxf(fmaxf(s[jx][0], s[jx][1]), fmaxf(s[jx][2], s[jx][3])));
                    }
                } else {
                    bool mine = false;
                    if constexpr (COMPACT) {
                        const uint32_t seen = seen_keys(sm.mask + mrow * 4, key0 + g4 * 8, kv_len, T);
                        mine = seen != 0 && mok;
#pragma unroll
                        for (int i = 0; i < 8; ++i) s[i >> 2][i & 3] = seen >> i & 1 ? s[i >> 2][i & 3] * scale_log2e : -INFINITY;
                    } else {
                        const uint32_t* mw = sm.mask + mrow * 4;
                        const uint64_t lo = mw[0] | (uint64_t)mw[1] << 32, hi = mw[2] | (uint64_t)mw[3] << 32;
#pragma unroll
                        for (int i = 0; i < 8; ++i) {
                            const int key = key0 + g4 * 8 + i, jn = key - kv_len;
                            bool vis = key < kv_len;
                            if (jn >= 0 && key < T) vis = ((jn < 64 ? lo >> jn : hi >> (jn - 64)) & 1ull) != 0;
                            mine = mine || (vis && mok);
                            s[i >> 2][i & 3] = vis ? s[i >> 2][i & 3] * scale_log2e : -INFINITY;
                        }
                    }
#pragma unroll
                    for (int i = 0; i < 8; ++i) tmax = fmaxf(tmax, s[i >> 2][i & 3]);
                    if (__ballot(mine) == 0ull) continue;  // no row of the tile sees the unit: leave it out
                    // keys from T on hold no data: zero them, a stray NaN times a zero weight is a NaN
                    const int nvalid = T - key0 - g4 * 8;
                    if (key0 + 32 > T) {
#pragma unroll
                        for (int e = 0; e < DT; ++e)
#pragma unroll
                            for (int i = 0; i < 8; ++i)
                                if (i >= nvalid) vf[e][i] = (half_t)0;
                    }
                }
                add_unit<DT, ALONE>(mrun[uu % STATES], lrun[uu % STATES], oacc[uu % STATES], s, vf, max_over_groups(tmax));
            }
        }

        // ---- end of this workgroup's share of the head.  The two wavefronts of a row tile exchange half of
        //      their output fragments each and merge the other half (online-softmax rescale); a head in
        //      one part is finished by that
        // (fixed order: the first half's share comes first)
        const auto merge = [](float& ma, float mb, float& wa, float& wb) {
            const float mx = fmaxf(ma, mb);
            wa = (ma == -INFINITY) ? 0.f : fast_exp2(ma - mx);
            wb = (mb == -INFINITY) ? 0.f : fast_exp2(mb - mx);
            ma = mx;
        };
        float m = mrun[0], l = sum_over_groups(lrun[0]);
        if constexpr (STATES == 2) {
            float wa, wb;
            merge(m, mrun[1], wa, wb);
            l = l * wa + sum_over_groups(lrun[1]) * wb;
#pragma unroll
            for (int e = 0; e < DT; ++e) oacc[0][e] = oacc[0][e] * wa + oacc[1][e] * wb;
        }
        const auto state = o_part + ((size_t)cx.j * Mpad + mrow) * D + g4 * 4;
        auto store = [&](auto n, int e0, const floatx4* o) {
            if (!mok) return;
            if (np > 1) {
#pragma unroll
                for (int e = 0; e < decltype(n)::value; ++e) *(GLOBAL floatx4*)(state + (e0 + e) * 16) = o[e];
            } else {
#pragma unroll
                for (int e = 0; e < decltype(n)::value; ++e)
                    store_attn_out(a, out, mrow, head * D + (e0 + e) * 16 + g4 * 4, l > 0.f ? o[e] / l : (floatx4){0.f, 0.f, 0.f, 0.f});
            }
        };
        if constexpr (HALVES == 2) {
            // (the buffer after the last tile's: everybody was done with it at the last barrier)
            auto& other = *reinterpret_cast<typename L::HalfOut*>(sm.tile[(t1 - t0) & (NB - 1)]);
            constexpr int HE = DT / 2;
            if (wave_active) {
#pragma unroll
                for (int e = 0; e < HE; ++e) other[wq][half][e][lane] = half ? oacc[0][e] : oacc[0][HE + e];
                if (lane < 16) {
                    sm.m[wq][half][c] = m;
                    sm.l[wq][half][c] = l;
                }
            }
            __syncthreads();
            if (wave_active) {
                const float mb = sm.m[wq][half ^ 1][c], lb = sm.l[wq][half ^ 1][c];
                float wa, wb;
                merge(m, mb, wa, wb);
                l = half ? lb * wb + l * wa : l * wa + lb * wb;
                floatx4 o[HE];
#pragma unroll
                for (int e = 0; e < HE; ++e) o[e] = (half ? oacc[0][HE + e] : oacc[0][e]) * wa + other[wq][half ^ 1][e][lane] * wb;
                store(std::integral_constant<int, HE>{}, half * HE, o);
            }
        } else {
            store(std::integral_constant<int, DT>{}, 0, oacc[0]);
        }
        if (np > 1) {
            if (mok && half == 0 && g4 == 0) *(GLOBAL floatx2*)(ml_part + ((size_t)cx.j * Mpad + mrow) * 2) = (floatx2){m, l};
            if (!finish_parts<D>(a, out, head, first, np, me, a.att_epoch, &sm.wait_ok)) return false;
        }
        // a workgroup that goes on to another head reuses its LDS (it has its heads to itself: np = 1)
        if (hl + 1 < h_hi) __syncthreads();
    }
    // a workgroup without a share of any head still checks in
    if (!gated && !gate()) return false;
    return true;
}

// ---- the attention of a launch ---------------------------------------------------------------
// MT: 16-row tiles of queries.
template <int MT, int D>
struct AttnOf {
    static constexpr bool DIRECT = MT <= 2;
    static constexpr int TMIN = DIRECT ? kDirectTiles : 1;         // tiles that a part has at least
    static_assert((kDirectTiles & (kDirectTiles - 1)) == 0, "divided by");
    using Lds = std::conditional_t<DIRECT, DirectLds<MT, D>, StagedLds<layout_tiles(MT), D>>;
};

// ALONE: no head is shared and there was no set-up launch (see attention_alone).  `late` gives the argument block.
template <int MT, int D, bool PREFETCH = false, bool ALONE = false, class Late, class Gate = NoGate>
__device__ __forceinline__ bool attn_phase(const AttnFirst& f, Late late, Ctx& cx, const AttnPlan& plan, Gate gate = Gate())
{
    if constexpr (AttnOf<MT, D>::DIRECT) return attn_direct<MT, D, PREFETCH, ALONE>(f, late, cx, plan, gate);
    else return attn_staged<layout_tiles(MT), D, PREFETCH, ALONE>(f, late, cx, plan, gate);
}

}  // namespace ghd
