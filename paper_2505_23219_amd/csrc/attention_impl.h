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
// Above (attn_staged), the workgroup shares tiles through LDS; wavefronts 0-3 take the first 32
// keys of a tile, 4-7 the last 32, each for its own 16 (or 32) rows.  Each wavefront reading units by
// itself was slower there: the states of eight wavefronts with all rows take 4 us to merge, and
// with the rows split over groups of wavefronts every unit is read once per group (13B-shaped layer,
// 64 rows, 8192 cached tokens, launch with the QKV layer: 75.7 us staged, 86 and 96 us).
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

__host__ __device__ __forceinline__ AttnHeads attn_heads(int nh, int j, int G)
{
    AttnHeads s;
    const int nx = (G % 8 == 0) ? 8 : 1;
    s.Gx = G / nx;
    s.x = j / s.Gx;
    s.w = j - s.x * s.Gx;
    s.hx0 = nh * s.x / nx;
    s.Hx = nh * (s.x + 1) / nx - s.hx0;
    s.h_lo = s.h_hi = 0;
    if (s.Hx == 0) return s;
    if (s.Hx >= s.Gx) {
        s.h_lo = s.Hx * s.w / s.Gx;
        s.h_hi = s.Hx * (s.w + 1) / s.Gx;
    } else {
        s.h_lo = ((s.w + 1) * s.Hx - 1) / s.Gx;    // the head whose run of workgroups contains w
        s.h_hi = s.h_lo + 1;
    }
    return s;
}

struct AttnTiles {
    int first, np, me;   // the head's parts are workgroups first .. first + np - 1; this one is part `me`
    int t0, t1;          // its key tiles (empty, with me >= np, when there are more workgroups than tiles)
};

// tmin: tiles a part should have at least.  A part's wavefronts work in parallel, so splitting a
// head further than a unit for each of them only adds to the exchange.
__host__ __device__ __forceinline__ AttnTiles attn_tiles(const AttnHeads& s, int hl, int ntile, int tmin)
{
    AttnTiles t;
    t.first = s.x * s.Gx + s.w;
    t.np = 1;
    t.me = 0;
    if (s.Hx < s.Gx) {
        int wl0 = s.Gx * hl / s.Hx;                        // head hl's run of local workgroups
        int wl1 = s.Gx * (hl + 1) / s.Hx;
        t.first = s.x * s.Gx + wl0;
        const int most = (ntile + tmin - 1) / tmin;
        t.np = (wl1 - wl0 < most) ? wl1 - wl0 : most;
        t.me = s.w - wl0;
    }
    // boundaries rounded up: when the tiles do not divide evenly the longer ranges come first,
    // and the last workgroup, whose range ends with the (costlier) tree tile, gets a shorter one
    t.t0 = t.t1 = 0;
    if (t.me < t.np) {
        t.t0 = (ntile * t.me + t.np - 1) / t.np;
        t.t1 = (ntile * (t.me + 1) + t.np - 1) / t.np;
    }
    return t;
}

// 2^x for x <= 0 (softmax weights): the hardware instruction; results below the smallest
// normal number flush to zero, which is what a weight that small should be.
__device__ __forceinline__ float fast_exp2(float x) { return __builtin_amdgcn_exp2f(x); }

// `gate` is called once by every workgroup (all threads), before the first read of q or of a
// cache row from kv_len on; it returns false if the launch is to be abandoned.  A kernel that
// produces those in the same launch waits there for their producers; with PREFETCH a
// wavefront's first unit is requested before the gate if it lies wholly below kv_len (rows of
// earlier steps), so that it arrives while the workgroup waits.
struct NoGate {
    __device__ __forceinline__ bool operator()() const { return true; }
};

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

template <int MT, int D, bool PREFETCH, class Gate>
__device__ __forceinline__ bool attn_direct(const FusedArgs& a, Ctx& cx, const half_t* q_, const half_t* kc_,
                                            const half_t* vc_, half_t* out_, uint32_t epoch, Gate gate)
{
    constexpr int DS = D / 32, DT = D / 16;
    DirectLds<MT, D>& sm = *reinterpret_cast<DirectLds<MT, D>*>(cx.lds);

    const int tid = threadIdx.x;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int M = a.M, nh = a.nh, kv_len = a.kv_len, T = a.kv_len + a.M, Mpad = a.Mpad;
    const float scale_log2e = a.scale_log2e;
    uint32_t* const sync = a.sync;
    const auto q = gp(q_), kc = gp(kc_), vc = gp(vc_);
    const auto out = gp(out_);
    const auto o_part = gp(a.o_part), ml_part = gp(a.ml_part);
    const int ntile = (T + 63) >> 6, nunit = (T + 31) >> 5;
    const uint32_t st_tok = (uint32_t)a.stride_tok, st_ch = (uint32_t)a.v_stride_ch;

    // Work shares.  Heads are dealt to the 8 XCDs in contiguous blocks.  Inside an XCD a
    // workgroup works on one head at a time: with fewer heads than workgroups, every head
    // gets its own run of workgroups, each taking a contiguous range of the head's key
    // tiles; otherwise every workgroup takes whole heads.  A head is therefore always
    // finished inside one XCD (partial states go through that XCD's L2).
    const AttnHeads hs = attn_heads(nh, cx.j, cx.G);
    const int hx0 = hs.hx0, h_lo = hs.h_lo, h_hi = hs.h_hi;
    // (bits from M on, which a caller's mask may have set, are never looked at: a mask bit is
    // only consulted for keys kv_len <= key < kv_len + M)
    uint64_t mask_lo = 0, mask_hi = 0;
    {
        const auto mask = gp(a.mask);
        if (tid < M) {
            mask_lo = mask[2 * tid];
            mask_hi = mask[2 * tid + 1];
        }
    }

    bool gated = false;
    for (int hl = h_lo; hl < h_hi; ++hl) {
        const int lane = hidden(threadIdx.x & 63), c = lane & 15, g4 = lane >> 4;
        const int head = hx0 + hl;
        // the workgroups first .. first + np - 1 split this head's tiles
        const AttnTiles ts = attn_tiles(hs, hl, ntile, kDirectTiles);
        const int first = ts.first, np = ts.np, me = ts.me;
        if (me >= np) continue;                            // more workgroups than parts
        const auto kh = kc + (size_t)head * a.stride_head;
        const auto vh = vc + (size_t)head * a.v_stride_head;
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
        // Requests, in order: [a unit of earlier steps] gate, queries, [the unit otherwise].  No
        // cache line of a unit that ends 64 rows or more below kv_len can hold a row that this
        // launch writes, whatever the strides and the alignment of the cache.
        const bool early = PREFETCH && !gated && u < u1 && u * 32 + 96 <= kv_len;
        if (early) {
            load_k(u);
            load_v(u);
        }
        if (!gated) {
            if (!gate()) return false;
            gated = true;
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
        if (tid < MT * 16) {
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
                    const uint64_t lo = sm.mask[row][0], hi = sm.mask[row][1];
                    bool mine = false;
#pragma unroll
                    for (int i = 0; i < 8; ++i) {
                        const int key = key0 + g4 * 8 + i, jn = key - kv_len;
                        bool vis = key < kv_len;
                        if (jn >= 0 && key < T) vis = ((jn < 64 ? lo >> jn : hi >> (jn - 64)) & 1ull) != 0;
                        mine = mine || (vis && row < M);
                        const float v = vis ? s[t][i >> 2][i & 3] * scale_log2e : -INFINITY;
                        s[t][i >> 2][i & 3] = v;
                        tmax = fmaxf(tmax, v);
                    }
                    any = __ballot(mine) != 0ull;          // no row of the tile sees the unit: leave it out
                }
                if (!any) continue;
                tmax = fmaxf(tmax, __shfl_xor(tmax, 16));
                tmax = fmaxf(tmax, __shfl_xor(tmax, 32));
                const float mnew = fmaxf(mrun[t], tmax);
                const float muse = (mnew == -INFINITY) ? 0.f : mnew;
                const float alpha = fast_exp2(mrun[t] - muse);
                mrun[t] = mnew;
                float lsum = 0.f;
                half8 pf;
#pragma unroll
                for (int i = 0; i < 8; ++i) {
                    const float pv = fast_exp2(s[t][i >> 2][i & 3] - muse);
                    lsum += pv;
                    pf[i] = (half_t)pv;
                }
                lrun[t] = lrun[t] * alpha + lsum;
                // (the maximum of most rows settles early: usually nothing has to be rescaled)
                if (__ballot(alpha != 1.0f)) {
#pragma unroll
                    for (int e = 0; e < DT; ++e) oacc[t][e] *= alpha;
                }
#pragma unroll
                for (int e = 0; e < DT; ++e) {
                    oacc[t][e] = __builtin_amdgcn_mfma_f32_16x16x32_f16(vf[e], pf, oacc[t][e], 0, 0, 0);
                }
            }
            if (u + 8 < u1) load_v(u + 8);
        }

        // ---- the wavefronts' states meet in LDS and are merged in wavefront order; a head in one
        //      part is finished by that
        const int lane_ = hidden(lane);
        auto store_out = [&](int m, int col, floatx4 v) {
            const half4 h = {(half_t)v[0], (half_t)v[1], (half_t)v[2], (half_t)v[3]};
            const size_t at = a.att_out_packed ? xpk_index(m, col, Mpad >> 4) : (size_t)m * nh * D + col;
            *(GLOBAL half4*)(out + at) = h;
        };
        {
        const int lane = lane_, c = lane & 15, g4 = lane >> 4;
#pragma unroll
        for (int t = 0; t < MT; ++t) {
            float l = lrun[t];
            l += __shfl_xor(l, 16);
            l += __shfl_xor(l, 32);
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
                store_out(m, head * D + e * 16 + g4 * 4, l > 0.f ? o / l : (floatx4){0.f, 0.f, 0.f, 0.f});
            } else {
                const size_t row = (size_t)cx.j * Mpad + m;
                *(GLOBAL floatx4*)(o_part + row * D + e * 16 + g4 * 4) = o;
                if (e == 0 && g4 == 0) *(GLOBAL floatx2*)(ml_part + row * 2) = (floatx2){mx, l};
            }
        }
        }
        if (np > 1) {
            const int tid = hidden(threadIdx.x);
            wait_own_stores();
            __syncthreads();   // partial state acknowledged by the L2
            uint32_t* const cnt = sync + kCntAttn + head * kCntStride;
            const int r0 = M * me / np, r1 = M * (me + 1) / np;        // the rows this part merges
            if (tid == 0) {
                uint32_t* const word = epoch_word(cnt, epoch);
                arrive(word);
                if (r0 < r1) sm.wait_ok = bounded_wait(sync, word, (uint32_t)np, (uint32_t)np, 2000u);
                if (me == 0) clear_next(cnt, epoch);
            }
            if (r0 < r1) {
                __syncthreads();
                if (!sm.wait_ok) return false;    // the other parts never arrived: nothing sensible to write
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
                    store_out(m, head * D + ch, den > 0.f ? num / den : (floatx4){0.f, 0.f, 0.f, 0.f});
                }
            }
        }
        // a workgroup that goes on to another head reuses its LDS and its partial-state slot
        // (a workgroup with several heads has them to itself: np = 1)
        if (hl + 1 < h_hi) __syncthreads();
    }
    // a workgroup without a share of any head still checks in
    if (!gated && !gate()) return false;
    return true;
}

// ---- more query rows: tiles staged through LDS, shared by the wavefronts ----------------------
template <int MT, int D>
struct StagedLds {
    static constexpr int MTW = (MT + 3) / 4;
    static constexpr int KS = D + 8;    // halves per K row (padded)
    static constexpr int VS = 64 + 8;   // halves per V^T row (padded, rows stay 16-byte aligned)
    // two tile buffers: while one tile is being multiplied, the next one is staged
    half_t k[2][64 * KS];
    half_t vt[2][D * VS];
    // state of the wavefronts working on the second key half, handed to their partners on
    // the first half when a head ends: [row-tile slot][tile][fragment][lane]
    floatx4 o2[4][MTW][D / 16][64];
    float m2[4][MTW][64];
    float l2[4][MTW][64];
    int wait_ok;      // thread 0's verdict on a bounded wait, for the whole workgroup
};

template <int MT, int D, bool PREFETCH, class Gate>
__device__ __forceinline__ bool attn_staged(const FusedArgs& a, Ctx& cx, const half_t* q, const half_t* kc,
                                            const half_t* vc, half_t* out, uint32_t epoch, Gate gate)
{
    constexpr int MTW = (MT + 3) / 4;   // 16-row tiles per wavefront
    constexpr int DS = D / 32, DT = D / 16, CPR = D / 8;
    constexpr int NLD = 64 * CPR / kFT; // 16-byte pieces per thread per tile, for K and for V alike
    constexpr int NT = (MT <= 4) ? 4 : 2;   // tiles in flight
    using L = StagedLds<MT, D>;
    L& sm = *reinterpret_cast<L*>(cx.lds);

    const int tid = threadIdx.x, wave = tid >> 6, lane = tid & 63;
    const int c = lane & 15, g4 = lane >> 4;
    const int kh = wave >> 2, wq = wave & 3;   // key half of the tile, row-tile slot
    // scalars of the argument block used inside the loops, as plain locals
    const int M = a.M, nh = a.nh, kv_len = a.kv_len, T = a.kv_len + a.M, Mpad = a.Mpad;
    const float scale_log2e = a.scale_log2e;
    uint32_t* const sync = a.sync;
    float* const o_part = a.o_part;
    float* const ml_part = a.ml_part;
    const int ntile = (T + 63) >> 6;

    // Work shares.  Heads are dealt to the 8 XCDs in contiguous blocks.  Inside an XCD a
    // workgroup works on one head at a time: with fewer heads than workgroups, every head
    // gets its own run of workgroups, each taking a contiguous range of the head's key
    // tiles; otherwise every workgroup takes whole heads.  A head is therefore always
    // finished inside one XCD (partial states go through that XCD's L2), and the tile loop
    // of a head has no head change in it.
    const AttnHeads hs = attn_heads(nh, cx.j, cx.G);
    const int hx0 = hs.hx0, h_lo = hs.h_lo, h_hi = hs.h_hi;

    // per-wave query rows
    int mrow[MTW];
    bool mok[MTW];
    uint64_t alo[MTW], ahi[MTW];
    bool wave_active = false;
#pragma unroll
    for (int t = 0; t < MTW; ++t) {
        int mt = wq * MTW + t;
        mrow[t] = mt * 16 + c;
        mok[t] = mrow[t] < M;
        wave_active = wave_active || (mt * 16 < M);
        alo[t] = mok[t] ? a.mask[2 * mrow[t]] : 0;
        ahi[t] = mok[t] ? a.mask[2 * mrow[t] + 1] : 0;
        // (bits from M on, which a caller's mask may have set, are never looked at: a mask bit
        // is only consulted for keys kv_len <= key < kv_len + M)
    }
    // K piece id -> (row id / CPR, 8 channels id % CPR); V^T piece id -> (channel id / 8,
    // 8 keys id % 8).  Offsets inside a head fit 32 bits (checked on the host).
    int k_off[NLD], v_off[NLD], k_row[NLD];
#pragma unroll
    for (int i = 0; i < NLD; ++i) {
        int id = tid + kFT * i;
        k_row[i] = id / CPR;
        k_off[i] = (id % CPR) * 8;
        v_off[i] = (id >> 3) * (int)a.v_stride_ch + (id & 7) * 8;
    }
    const int v_last = (int)a.v_stride_ch - 8, st_tok = (int)a.stride_tok;
    const std::integral_constant<int, 0> s0;
    const std::integral_constant<int, 1> s1;
    const std::integral_constant<int, NT == 4 ? 2 : 0> s2;
    const std::integral_constant<int, NT == 4 ? 3 : 1> s3;

    bool gated = false;
    for (int hl = h_lo; hl < h_hi; ++hl) {
        const int head = hx0 + hl;
        // the workgroups first .. first + np - 1 split this head's tiles
        const AttnTiles ts = attn_tiles(hs, hl, ntile, 1);
        const int first = ts.first, np = ts.np, me = ts.me, t0 = ts.t0, t1 = ts.t1;
        if (me >= np) continue;                            // more workgroups than tiles
        const half_t* kh_ = kc + (size_t)head * a.stride_head;
        const half_t* vh_ = vc + (size_t)head * a.v_stride_head;

        // running state of this head
        float mrun[MTW], lrun[MTW];
        floatx4 oacc[MTW][DT];
#pragma unroll
        for (int t = 0; t < MTW; ++t) {
            mrun[t] = -INFINITY;
            lrun[t] = 0.f;
#pragma unroll
            for (int e = 0; e < DT; ++e) oacc[t][e] = (floatx4){0.f, 0.f, 0.f, 0.f};
        }

        // NT tiles in flight: registers of set (tile - t0) % NT hold a tile until it is
        // staged.  A workgroup has few tiles (about 4 at 2048 cached tokens), so the time to
        // the first byte dominates unless all of them are requested at once.  The loads
        // are unconditional: past the last tile they all read one valid 16-byte piece (a
        // broadcast), which keeps the wait counts of the loop exact.
        half8 kreg[NT][NLD], vreg[NT][NLD];
        int l_tile = t0;                                   // next tile to request
        auto load_tile = [&](auto set) {
            constexpr int S = decltype(set)::value;
            const bool real = l_tile < t1;
#pragma unroll
            for (int i = 0; i < NLD; ++i) {
                int key = min(l_tile * 64 + k_row[i], T - 1);
                const half_t* kp = kh_ + key * st_tok + k_off[i];
                // keys past the capacity are never touched: the last piece is read instead
                // and zeroed when it is staged
                int over = max(l_tile * 64 + (int)((tid + kFT * i) & 7) * 8 - v_last, 0);
                const half_t* vp = vh_ + v_off[i] + l_tile * 64 - over;
                kreg[S][i] = __builtin_nontemporal_load((const half8*)(real ? kp : kc));
                vreg[S][i] = __builtin_nontemporal_load((const half8*)(real ? vp : vc));
            }
            ++l_tile;
        };
        auto store_tile = [&](auto set, int tile) {
            constexpr int S = decltype(set)::value;
#pragma unroll
            for (int i = 0; i < NLD; ++i) {
                int id = tid + kFT * i;
                *(half8*)(&sm.k[S & 1][k_row[i] * L::KS + k_off[i]]) = kreg[S][i];
                int vch = id >> 3, seg = id & 7;
                half8 v = vreg[S][i];
                int nvalid = T - (tile * 64 + seg * 8);  // rows from T on hold no data: zero them,
                if (nvalid < 8) {                        // a stray NaN times a zero weight is a NaN
#pragma unroll
                    for (int e = 0; e < 8; ++e)
                        if (e >= nvalid) v[e] = (half_t)0;
                }
                *(half8*)(&sm.vt[S & 1][vch * L::VS + seg * 8]) = v;
            }
        };
        // Requests, in tile order: [tiles known before the gate] gate [queries] [the rest].
        int n_pre = 0;
        if (!gated) {
            if constexpr (PREFETCH) {
                // past this share's last tile (a dummy load), or at least 64 rows below
                // kv_len: no cache line of such a tile holds a row that this launch writes,
                // whatever the strides and the alignment of the cache
                auto early = [&]() { return l_tile >= t1 || l_tile * 64 + 128 <= kv_len; };
                if (early()) {
                    load_tile(s0);
                    n_pre = 1;
                    if (early()) {
                        load_tile(s1);
                        n_pre = 2;
                        if constexpr (NT == 4) {
                            if (early()) {
                                load_tile(s2);
                                n_pre = 3;
                                if (early()) {
                                    load_tile(s3);
                                    n_pre = 4;
                                }
                            }
                        }
                    }
                }
            }
            if (!gate()) return false;
            gated = true;
        }
        half8 qf[MTW][DS];
#pragma unroll
        for (int t = 0; t < MTW; ++t) {
#pragma unroll
            for (int s = 0; s < DS; ++s) {
                half8 v = {0, 0, 0, 0, 0, 0, 0, 0};
                if (mok[t]) v = *(const half8*)(q + ((size_t)mrow[t] * nh + head) * D + s * 32 + g4 * 8);
                qf[t][s] = v;
            }
        }
        if (n_pre < 1) load_tile(s0);
        if (n_pre < 2) load_tile(s1);
        if constexpr (NT == 4) {
            if (n_pre < 3) load_tile(s2);
            if (n_pre < 4) load_tile(s3);
        }
        // The tiles alternate between the two LDS buffers (register set S goes to buffer
        // S & 1: the number of sets is even).  While tile i is multiplied out of one buffer,
        // tile i + 1 is staged into the other and its registers are refilled - one barrier
        // per tile.  Past the share's last tile the staged data is a dummy nobody reads.
        int p_tile = t0;                                   // the tile being processed
        store_tile(s0, t0);
        load_tile(s0);
        auto do_tile = [&](auto set, auto next) {
            constexpr int B = decltype(set)::value & 1;
            const int tile = p_tile++;
            __syncthreads();            // tile staged by everybody; the other buffer is free
            store_tile(next, tile + 1);
            load_tile(next);
        if (!wave_active) return;
        const int key0 = tile * 64 + kh * 32;    // this wavefront's 32 keys
        const bool committed = key0 + 32 <= kv_len;   // every key visible to every row
#pragma unroll
        for (int t = 0; t < MTW; ++t) {
            floatx4 s[2];
            float tmax = -INFINITY;
            if (committed) {
#pragma unroll
                for (int jx = 0; jx < 2; ++jx) {
                    s[jx] = (floatx4){0.f, 0.f, 0.f, 0.f};
#pragma unroll
                    for (int ds = 0; ds < DS; ++ds) {
                        half8 kf = *(const half8*)(&sm.k[B][(kh * 32 + jx * 16 + c) * L::KS + ds * 32 + g4 * 8]);
                        s[jx] = __builtin_amdgcn_mfma_f32_16x16x32_f16(kf, qf[t][ds], s[jx], 0, 0, 0);
                    }
                    s[jx] *= scale_log2e;
                    tmax = fmaxf(tmax, fmaxf(fmaxf(s[jx][0], s[jx][1]), fmaxf(s[jx][2], s[jx][3])));
                }
            } else {
                bool sub_any[2];
#pragma unroll
                for (int jx = 0; jx < 2; ++jx) {
                    const int kbase = key0 + jx * 16;
                    bool vis_any;
                    if (kbase + 16 <= kv_len) {
                        vis_any = true;
                    } else {
                        bool mine = false;
#pragma unroll
                        for (int r = 0; r < 4; ++r) {
                            int key = kbase + g4 * 4 + r;
                            bool vis = key < kv_len;
                            if (key >= kv_len && key < T) {
                                int jn = key - kv_len;
                                vis = (jn < 64 ? (alo[t] >> jn) : (ahi[t] >> (jn - 64))) & 1ull;
                            }
                            mine = mine || (vis && mok[t]);
                        }
                        vis_any = __ballot(mine) != 0ull;
                    }
                    sub_any[jx] = vis_any;
                    s[jx] = (floatx4){0.f, 0.f, 0.f, 0.f};
                    if (vis_any) {
#pragma unroll
                        for (int ds = 0; ds < DS; ++ds) {
                            half8 kf = *(const half8*)(&sm.k[B][(kh * 32 + jx * 16 + c) * L::KS + ds * 32 + g4 * 8]);
                            s[jx] = __builtin_amdgcn_mfma_f32_16x16x32_f16(kf, qf[t][ds], s[jx], 0, 0, 0);
                        }
                    }
                }
                if (!(sub_any[0] || sub_any[1])) continue;
#pragma unroll
                for (int jx = 0; jx < 2; ++jx) {
                    const int kbase = key0 + jx * 16;
#pragma unroll
                    for (int r = 0; r < 4; ++r) {
                        int key = kbase + g4 * 4 + r;
                        bool vis = sub_any[jx] && key < kv_len;
                        if (sub_any[jx] && key >= kv_len && key < T) {
                            int jn = key - kv_len;
                            vis = (jn < 64 ? (alo[t] >> jn) : (ahi[t] >> (jn - 64))) & 1ull;
                        }
                        float v = vis ? s[jx][r] * scale_log2e : -INFINITY;
                        s[jx][r] = v;
                        tmax = fmaxf(tmax, v);
                    }
                }
            }
            tmax = fmaxf(tmax, __shfl_xor(tmax, 16));
            tmax = fmaxf(tmax, __shfl_xor(tmax, 32));
            float mnew = fmaxf(mrun[t], tmax);
            float muse = (mnew == -INFINITY) ? 0.f : mnew;
            float alpha = fast_exp2(mrun[t] - muse);
            mrun[t] = mnew;
            float lsum = 0.f;
            half8 pf;
#pragma unroll
            for (int jx = 0; jx < 2; ++jx)
#pragma unroll
                for (int r = 0; r < 4; ++r) {
                    float pv = fast_exp2(s[jx][r] - muse);
                    lsum += pv;
                    pf[jx * 4 + r] = (half_t)pv;
                }
            lrun[t] = lrun[t] * alpha + lsum;
#pragma unroll
            for (int e = 0; e < DT; ++e) {
                oacc[t][e] *= alpha;
                const half_t* vrow = &sm.vt[B][(e * 16 + c) * L::VS + kh * 32];
                half4 a0 = *(const half4*)(vrow + g4 * 4);
                half4 a1 = *(const half4*)(vrow + 16 + g4 * 4);
                half8 vf = {a0[0], a0[1], a0[2], a0[3], a1[0], a1[1], a1[2], a1[3]};
                oacc[t][e] = __builtin_amdgcn_mfma_f32_16x16x32_f16(vf, pf, oacc[t][e], 0, 0, 0);
            }
        }
    };
        // Whole groups of NT tiles run in a branch-free loop; the rest is a chain of nested
        // conditions, so every tile is only reachable through its predecessor and the number
        // of loads younger than the one being waited for is known.
        {
            int u = t0;
            if constexpr (NT == 4) {
                for (; u + 3 < t1; u += 4) {
                    do_tile(s0, s1);
                    do_tile(s1, s2);
                    do_tile(s2, s3);
                    do_tile(s3, s0);
                }
                if (u < t1) {
                    do_tile(s0, s1);
                    if (u + 1 < t1) {
                        do_tile(s1, s2);
                        if (u + 2 < t1) do_tile(s2, s3);
                    }
                }
            } else {
                for (; u + 1 < t1; u += 2) {
                    do_tile(s0, s1);
                    do_tile(s1, s0);
                }
                if (u < t1) do_tile(s0, s1);
            }
        }

        // ---- end of this workgroup's share of the head: the wavefronts of the second key
        //      half hand their state over through LDS, their partners merge it into their
        //      own (online-softmax rescale) and store the workgroup's partial state
#pragma unroll
        for (int t = 0; t < MTW; ++t) {
            float l = lrun[t];
            l += __shfl_xor(l, 16);
            l += __shfl_xor(l, 32);
            lrun[t] = l;
        }
        if (kh == 1 && wave_active) {
#pragma unroll
            for (int t = 0; t < MTW; ++t) {
#pragma unroll
                for (int e = 0; e < DT; ++e) sm.o2[wq][t][e][lane] = oacc[t][e];
                sm.m2[wq][t][lane] = mrun[t];
                sm.l2[wq][t][lane] = lrun[t];
            }
        }
        __syncthreads();
        if (kh == 0 && wave_active) {
#pragma unroll
            for (int t = 0; t < MTW; ++t) {
                float mb = sm.m2[wq][t][lane], lb = sm.l2[wq][t][lane];
                float mx = fmaxf(mrun[t], mb);
                float wa = (mrun[t] == -INFINITY) ? 0.f : fast_exp2(mrun[t] - mx);
                float wb = (mb == -INFINITY) ? 0.f : fast_exp2(mb - mx);
                float l = lrun[t] * wa + lb * wb;
                if (!mok[t]) continue;
                size_t row = (size_t)cx.j * Mpad + mrow[t];
#pragma unroll
                for (int e = 0; e < DT; ++e) {
                    floatx4 ob = sm.o2[wq][t][e][lane];
                    *(floatx4*)(o_part + row * D + e * 16 + g4 * 4) = oacc[t][e] * wa + ob * wb;
                }
                if (g4 == 0) {
                    ml_part[row * 2] = mx;
                    ml_part[row * 2 + 1] = l;
                }
            }
        }
        wait_own_stores();
        __syncthreads();   // partial state acknowledged by the L2; hand-over buffers free again

        // ---- merge: every workgroup of the head combines its share of the rows
        if (tid == 0) {
            uint32_t* const cnt = sync + kCntAttn + head * kCntStride;
            uint32_t* const word = epoch_word(cnt, epoch);
            arrive(word);
            sm.wait_ok = bounded_wait(sync, word, (uint32_t)np, (uint32_t)np, 2000u);
            if (me == 0) clear_next(cnt, epoch);
        }
        __syncthreads();
        if (!sm.wait_ok) return false;    // the other parts never arrived: nothing sensible to write
        int r0 = M * me / np, r1 = M * (me + 1) / np;
        for (int m = r0 + wave; m < r1; m += 8) {
            // lane p holds the statistics of part p (np <= 64: one XCD's workgroups)
            float mq = -INFINITY, lq = 0.f;
            size_t rowq = 0;
            if (lane < np) {
                rowq = (size_t)(first + lane) * Mpad + m;
                mq = ml_part[rowq * 2];
                lq = ml_part[rowq * 2 + 1];
            }
            float mx = mq;
            for (int off = 32; off > 0; off >>= 1) mx = fmaxf(mx, __shfl_xor(mx, off));
            float wq_ = (mq == -INFINITY) ? 0.f : fast_exp2(mq - mx);
            float den = wq_ * lq;
            for (int off = 32; off > 0; off >>= 1) den += __shfl_xor(den, off);
            // weighted sum of the parts' outputs, parts in index order, 8 loads in flight
            float num[D / 64];
#pragma unroll
            for (int e = 0; e < D / 64; ++e) num[e] = 0.f;
            for (int q0 = 0; q0 < np; q0 += 8) {
                float t[8][D / 64], w8[8];
#pragma unroll
                for (int qi = 0; qi < 8; ++qi) {
                    int qq = min(q0 + qi, np - 1);
                    size_t row = (size_t)__shfl((long long)rowq, qq);
                    w8[qi] = (q0 + qi < np) ? __shfl(wq_, qq) : 0.f;
#pragma unroll
                    for (int e = 0; e < D / 64; ++e) t[qi][e] = o_part[row * D + e * 64 + lane];
                }
#pragma unroll
                for (int qi = 0; qi < 8; ++qi)
#pragma unroll
                    for (int e = 0; e < D / 64; ++e) num[e] += w8[qi] * t[qi][e];
            }
#pragma unroll
            for (int e = 0; e < D / 64; ++e) {
                // a row that sees no key at all (possible with a caller's mask and an empty
                // cache) gets zeros
                const int col = head * D + e * 64 + lane;
                const size_t at = a.att_out_packed ? xpk_index(m, col, Mpad >> 4) : (size_t)m * nh * D + col;
                out[at] = (half_t)(den > 0.f ? num[e] / den : 0.f);
            }
        }
        // a workgroup that goes on to another head reuses its partial-state slot: wait until
        // the other parts have read it
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
    using Lds = std::conditional_t<DIRECT, DirectLds<MT, D>, StagedLds<layout_tiles(MT), D>>;
};

template <int MT, int D, bool PREFETCH = false, class Gate = NoGate>
__device__ __forceinline__ bool attn_phase(const FusedArgs& a, Ctx& cx, const half_t* q, const half_t* kc,
                                           const half_t* vc, half_t* out, uint32_t epoch, Gate gate = Gate())
{
    if constexpr (AttnOf<MT, D>::DIRECT) return attn_direct<MT, D, PREFETCH>(a, cx, q, kc, vc, out, epoch, gate);
    else return attn_staged<layout_tiles(MT), D, PREFETCH>(a, cx, q, kc, vc, out, epoch, gate);
}

}  // namespace ghd
