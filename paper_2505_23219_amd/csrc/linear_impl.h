// The skinny linear layer: y[M, N] = x[M, K] W[N, K]^T with M <= 128 rows, one launch.
//
// The step re-reads every weight once per decoding step and is bound by that stream
// (Ghidorah, sections 2.1 and 2.2.2), so the kernel is built around it.  A workgroup has a
// group of up to R row tiles (16 output features each) and a k range.  Its wavefronts
// (eight) take the range's k-steps in turn; each wavefront streams its k-steps of ALL the group's
// tiles (W is the MFMA A operand, fetched with non-temporal 128-bit loads straight into
// registers, a few k-steps ahead) together with the matching x fragments (the B operand,
// from the L2), and keeps one fp32 accumulator fragment per (row tile, 16 rows of x).  There
// is no LDS staging, and up to 64 rows no barrier inside the stream: the wavefronts run independently until
// the range ends (above, a barrier in every turn keeps them together, see keeps_step).  Then the partial fragments of every tile are added up through LDS,
// in pairs of pairs of wavefronts, and the reducing wavefront runs the layer's element-wise epilogue
// (residual add + sums of squares for the next RMSNorm, rotary embedding + KV append, SwiGLU).
// Where the accumulators would leave one of eight wavefronts no registers for a load ring
// (above 64 rows of x), the workgroup has four wavefronts of twice the registers.
//
// Two ways of dealing a matrix out (chosen on the host, see choose_cut).  Whole tiles: a
// workgroup has a run of consecutive tiles over the whole k range; nothing is exchanged
// between workgroups, every workgroup reads all of x - or, where tiles are few, all of some of its rows: groups
// of workgroups have the same tiles and different rows.  Parts: a workgroup has 1/S of the k
// range of a block of R tiles; it reads only that part of x, stores the block's partial sums,
// and the S workgroups of a block, which run on one XCD, finish it jointly at the end of the
// launch, parts added in index order, so results never depend on timing.
#pragma once
#include "persist.h"

#include <type_traits>

namespace ghd {

// What a wavefront needs before it can request its first weights: twelve words that the
// hardware puts into scalar registers at the start of the kernel (kernel argument preloading),
// so the first loads go out some forty instructions after a wavefront starts instead of
// waiting for the argument block (host memory: 0.6 us) and for index arithmetic.  Everything
// else is in FusedArgs behind them and only read when those loads are on their way.
struct LinHead {
    const half8* W;
    const half_t* x;     // packed activation layout, or row-major (ROWS)
    uint64_t aux;        // packed: the sums of squares (0: none); ROWS: elements from row to row
    int nks, K, ntiles;
    int cut;             // whole tiles: workgroups per XCD; parts: S
    uint32_t magic;      // whole tiles: 2^32 / cut + 1; parts: 2^16 / cut + 1
    uint32_t flags;      // see kHead*
};
constexpr int kHeadBlk = 0;      // bits 0-3: log2 of the tiles per storage block
constexpr int kHeadMtp = 4;      // bits 4-7: row tiles of the packed activation layout (Mpad / 16)
constexpr int kHeadM = 8;        // bits 8-15: rows of x
constexpr int kHeadSolo = 16;    // bit 16: a call of its own, without a set-up kernel
constexpr int kHeadLong = 17;    // bit 17: chains of sums are cut short (see folded)
static_assert(sizeof(LinHead) == kTailAt && alignof(FusedArgs) == 8, "kernel argument layout");

// wavefronts of a workgroup
__host__ __device__ constexpr int waves_of(int MT, int R) { return MT > 4 && R * MT > 32 ? 4 : 8; }

#ifndef GHD_RING_REGS
#define GHD_RING_REGS 88     // registers the load ring of a wavefront may take: two k-steps of three tiles
                             // by 128 rows of x (one, with 80: [9000, 13824] 91.7 us instead of 87.9)
#endif
#ifndef GHD_RING_KIB
#define GHD_RING_KIB 4       // weight bytes it keeps in flight, in KiB (more was measured slower)
#endif
// k-steps in flight per wavefront: limited by registers (accumulators + the ring) and by
// what the stream needs (a few KiB per wavefront: loads return in issue order, and a long
// queue only delays the x fragments behind it)
__host__ __device__ constexpr int pd_of(int MT, int R, int NW)
{
    const bool four = NW == 4;
    const int regs = (four ? 304 : 200) - R * MT * 4;       // beside the accumulators
    int by_regs = (four || regs < GHD_RING_REGS ? regs : GHD_RING_REGS) / ((R + MT) * 4);
    int by_bytes = ((four ? 8 : GHD_RING_KIB) + R - 1) / R;
    int pd = by_regs < by_bytes ? by_regs : by_bytes;
    return pd < 1 ? 1 : (pd > 8 ? 8 : pd);
}

// How sums are kept short.  The rounding error of a chain of MFMAs grows with its length (measured:
// squared relative error 4.4e-15 + 1.3e-15 per k-step of a wavefront's chain), so a cut whose
// chains come out long must not leave them in one piece (see long_chains).  Two ways:
//   FOLDED: a second set of accumulators; after every two to four k-steps the first is added to
//   it and begins anew (an addition rounds a quarter as badly as an MFMA);
//   STRETCHES, where there are no registers for that: a wavefront's range is taken in halves, and the
//   sums of the first are set aside, in the LDS that the reduction uses later and in what registers
//   are left; the last fragments of the largest groups are added up step by step instead.
// And in row groups SINGLE: every k-step's product is added to one of four sets of sums in turn, which
// are added in pairs at the end.  Groups then round less than the parts they stand in for ([300, 3416] at 64 rows:
// 8.4e-8, in parts 9.4e-8), and stand in for more of them ([1280, 1280] at 64 rows: 7.0 us, in parts 10.0).  Without
// groups it only costs: [3457, 4872] at 27 rows took 14.1 us instead of 13.7.
// [2048, 13824] at 1 row: 2.8e-7 of the result in one chain, 1.2e-7 folded (weights from HBM 13.1 and 13.3 us);
// [22016, 4096] at 128 rows, four wavefronts: 2.1e-7 in one chain, 1.5e-7 in halves (45.3 and 48.0 us).
constexpr int kFoldSteps = 2;
__host__ __device__ constexpr bool folded(int MT, int R) { return R * MT <= (R <= 3 ? 18 : 16); }
__host__ __device__ constexpr bool grouped(int MT, int R) { return R == 1 && (MT == 1 || MT == 2 || MT == 4); }
constexpr int kSingleSets = 4;       // (one for each k-step of the ring)
// Stretches that a range is taken in: two halves, or three where the chains of an even deal are less
// than half as long.  (Of more than three whole tiles on eight wavefronts only wide matrices are dealt
// out, whose chains are never long.)
__host__ __device__ constexpr int stretches_whole(int MT, int R)
{
    return folded(MT, R) ? 1 : waves_of(MT, R) == 4 ? 2 : R <= 3 ? 3 : 1;
}
__host__ __device__ constexpr int stretches_parts(int MT, int R) { return folded(MT, R) ? 1 : 2; }

// The wavefronts of a workgroup take the k-steps in turn, so that together they read one run of a tile
// block from front to back; with a range of its own each (the first of a SIMD's two got 18/32, since
// it gets its data sooner) the memory saw eight runs per workgroup at a time.  us a call, weights from HBM:
//   rows   matrix           ranges   in turn
//      1   [22016, 4096]     28.6     27.4
//     16   [32000, 4096]     40.9     38.9
//     64   [32000, 4096]     48.8     48.1
//     16   7B-shaped layer   89.9     87.0
// Above 64 rows x takes more of the way into a compute unit than weights do, the wavefronts drift apart
// over it, and a barrier in every turn of the ring keeps them together (it waits for no load):
//     96   [32000, 4096]     60.3     61.0, with the barrier 58.8
//     96   [20480, 4096]     40.5     40.0                   39.1
//     96   [16384, 4096]     36.3     35.0                   33.5
//    128   [27648, 4096]     64.6     65.2                   62.7
//    128   [22016, 4096]     52.2     52.5                   48.1
//    128   [16384, 4096]     40.2     39.5                   36.5
//    128   [4096, 11008]     34.6     34.7                   33.7
//    128   [32000, 4096]     68.1     68.3                   74.9
// The last, 8 tiles by 128 rows, is the one that is slower with it, so it has none.  (Its ring holds one k-step, but so do
// those of 7 tiles by 128 rows and of 4, 5 and 8 by 96; it adds 22 fragments up step by step, 7 tiles 6, the others none: see
// NSTEP.)  Up to 64 rows it costs 0 to 1%.
__host__ __device__ constexpr bool keeps_step(int MT, int R) { return MT > 4 && R * MT <= 56; }

// A workgroup of one whole tile takes a single KiB out of every four of a block and, where x is read as it lies, 64 bytes of a
// row for each: with turns of one k-step, neighbours of a memory page and the halves of a line of x go to
// different wavefronts. So its wavefronts take four consecutive k-steps in their turn (as many as their ring holds), and
// what is left over after whole rounds in runs of one to three, so that no chain gets longer. us a call, weights in the cache:
//   rows   matrix           ranges   turns of one   of four
//      8   [4096, 11008]    16.3     17.6           16.0
//      9   [3311, 4960]      8.1      8.8            7.9
//     16   [4096, 4096]      8.7      9.0            8.1
//     18   [2879, 3680]      9.6      9.9            9.9
// (From HBM, over 121 calls of 56 k-steps and more, ranges taken as 1: turns of one 0.94 to 1.12, of four 0.90 to 1.05.)  Below
// 56 k-steps there are rounds too few: turns of one 2% faster from the cache, of four 2% from HBM.
__host__ __device__ constexpr int run_of(int MT, int R) { return R == 1 && MT <= 4 ? 4 : 1; }
constexpr int kRunSteps = 56;
static inline int run_of_launch(const LinCut& cut, int nks) { return cut.whole && nks >= kRunSteps ? run_of(cut.mt, cut.tiles) : 1; }

// What the residual epilogue reads: four columns of a row of the residual stream and of the next
// norm's gain.  (Requested behind the stream's first loads they delay the weights behind them by more
// than they save: 0.9% of a 64-row step.)
struct ResidOperands {
    floatx4 x;
    half4 g;
};
__device__ __forceinline__ ResidOperands resid_operands(ArgPtr a, int m, int n0)
{
    ResidOperands r = {{0.f, 0.f, 0.f, 0.f}, {0, 0, 0, 0}};
    if (m < a->M && n0 < a->lin_N) {
        r.x = *(GLOBAL const floatx4*)(gp((const float*)a->lin_y) + (size_t)m * a->lin_ldy + n0);
        if (a->lin_gnext) r.g = *(GLOBAL const half4*)(gp(a->lin_gnext) + n0);
    }
    return r;
}

constexpr int kNoRow = 1 << 20;      // m of a fragment that is not there

// ---------------------------------------------------------------------------
// epilogue of NB 16x16 output fragments: lane (c, g4) holds y[m][n0 .. n0+3] of each; m past the last row
// stands for no fragment.  What is worked out is worked out for all of them before any is stored: with one
// or two wavefronts on a SIMD a fragment by itself is one chain of latencies.
// ---------------------------------------------------------------------------
template <int NB>
__device__ __forceinline__ void epilogue(ArgPtr a, floatx4 (&v)[NB], int (&m)[NB], int (&n0)[NB], int lane, const float* s_rinv,
                                         const ResidOperands* ahead = nullptr)
{
    // Everything below depends on the fragments' positions: the (empty) asm keeps the compiler
    // from working parts of it out ahead of the weight stream, before the kernel's first loads.
#pragma unroll
    for (int i = 0; i < NB; ++i) asm volatile("" : "+v"(m[i]), "+v"(n0[i]));
    const int M = a->M, mtp = a->Mpad >> 4, N = a->lin_N, epi = a->lin_epi;
    const int64_t ldo = a->lin_ldy;
    if (a->lin_rscale) {
#pragma unroll
        for (int i = 0; i < NB; ++i) v[i] *= s_rinv[m[i] == kNoRow ? m[0] : m[i]];      // (the first one is there)
    }
    if (epi == EPI_STORE_F32) {
        if (a->lin_amax) {
            // the row's best output among a tile's 16 columns: (largest value, lowest column).
            // Greedy acceptance (section 2.3) only needs the row argmax, so the finish of the
            // LM head leaves one candidate per tile and row instead of (or besides) the logits.
#pragma unroll
            for (int i = 0; i < NB; ++i) {
                float bv = -INFINITY;
                int bi = 0x7fffffff;
#pragma unroll
                for (int r = 0; r < 4; ++r)
                    if (n0[i] + r < N && v[i][r] > bv) {
                        bv = v[i][r];
                        bi = n0[i] + r;
                    }
#pragma unroll
                for (int off = 16; off < 64; off <<= 1) {
                    const float ov = __shfl_xor(bv, off);
                    const int oi = __shfl_xor(bi, off);
                    if (ov > bv || (ov == bv && oi < bi)) {
                        bv = ov;
                        bi = oi;
                    }
                }
                if (lane < 16 && m[i] < M) {
                    const floatx2 best = {bv, __int_as_float(bi)};
                    *(GLOBAL floatx2*)(gp((float*)a->lin_amax) + ((size_t)(n0[i] >> 4) * a->Mpad + m[i]) * 2) = best;
                }
            }
        }
        if (!a->lin_y) return;
#pragma unroll
        for (int i = 0; i < NB; ++i) {
            if (m[i] >= M) continue;
            auto o = gp((float*)a->lin_y) + (size_t)m[i] * ldo + n0[i];
            if (n0[i] + 3 < N && (ldo & 3) == 0) *(GLOBAL floatx4*)o = v[i];
            else
                for (int r = 0; r < 4; ++r)
                    if (n0[i] + r < N) o[r] = v[i][r];
        }
    } else if (epi == EPI_STORE_F16) {
#pragma unroll
        for (int i = 0; i < NB; ++i) {
            if (m[i] >= M) continue;
            auto o = gp((half_t*)a->lin_y) + (size_t)m[i] * ldo + n0[i];
            for (int r = 0; r < 4; ++r)
                if (n0[i] + r < N) o[r] = (half_t)v[i][r];
        }
    } else if (epi == EPI_RESID) {
        // x += y; sums of squares of the new x over a tile's 16 columns, per row
        ResidOperands ops[NB];
#pragma unroll
        for (int i = 0; i < NB; ++i) ops[i] = ahead ? ahead[i] : resid_operands(a, m[i], n0[i]);
        floatx4 xn[NB];
        half4 o[NB];
        float sq[NB];
#pragma unroll
        for (int i = 0; i < NB; ++i) {
            xn[i] = ops[i].x + v[i];
            sq[i] = m[i] < M && n0[i] < N ? xn[i][0] * xn[i][0] + xn[i][1] * xn[i][1] + xn[i][2] * xn[i][2] + xn[i][3] * xn[i][3] : 0.f;
#pragma unroll
            for (int q = 0; q < 4; ++q) o[i][q] = (half_t)(xn[i][q] * (float)ops[i].g[q] * kXgScale);
            sq[i] += __shfl_xor(sq[i], 16);
            sq[i] += __shfl_xor(sq[i], 32);
        }
#pragma unroll
        for (int i = 0; i < NB; ++i) {
            if (n0[i] < N && m[i] < M) {
                *(GLOBAL floatx4*)(gp((float*)a->lin_y) + (size_t)m[i] * ldo + n0[i]) = xn[i];
                if (a->lin_gnext) *(GLOBAL half4*)(gp(a->xg16) + xpk_index(m[i], n0[i], mtp)) = o[i];
            }
            // (rows past M too, of the tiles that there are: the next norm adds them up)
            if (lane < 16 && n0[i] < N && m[i] < a->Mpad) gp(a->ss)[(size_t)(n0[i] >> 4) * a->Mpad + m[i]] = sq[i];
        }
    } else if (epi == EPI_SWIGLU) {
        // packed rows: (gate f, gate f+1, up f, up f+1)
        // silu with the hardware's exp2 and reciprocal: a few ulp, far below the fp16 rounding
        // of the result (and 0.3 us per launch on the critical path)
        half2_ h[NB];
#pragma unroll
        for (int i = 0; i < NB; ++i) {
            const float a0 = __fdividef(v[i][0], 1.0f + __expf(-v[i][0])) * v[i][2];
            const float a1 = __fdividef(v[i][1], 1.0f + __expf(-v[i][1])) * v[i][3];
            h[i] = (half2_){(half_t)a0, (half_t)a1};
        }
#pragma unroll
        for (int i = 0; i < NB; ++i) {
            const int f = (n0[i] >> 4) * 8 + ((n0[i] & 15) >> 2) * 2;
            if (m[i] < M && f < a->F) *(GLOBAL half2_*)(gp((half_t*)a->lin_y) + xpk_index(m[i], f, mtp)) = h[i];
        }
    } else {   // EPI_QKV: packed rows of a head: (j, j+1, j+d/2, j+1+d/2)
        const int nh = a->nh, d = a->d, H = nh * d, hd = d >> 1;
        QkvRow qr[NB];
        floatx4 cs[NB];
#pragma unroll
        for (int i = 0; i < NB; ++i) {
            qr[i] = qkv_row_fast(n0[i], nh, d);
            // (cos, sin) of channels jj and jj + 1 (jj is even: 16 bytes, aligned)
            cs[i] = (floatx4){1.f, 0.f, 1.f, 0.f};
            if (m[i] < M && qr[i].part < 2)
                cs[i] = *(GLOBAL const floatx4*)(gp((const float*)a->rope) + ((size_t)m[i] * hd + (qr[i].ph >> 2) * 2) * 2);
        }
#pragma unroll
        for (int i = 0; i < NB; ++i) {
            if (m[i] >= M || n0[i] >= N) continue;
            const int part = qr[i].part, head = qr[i].head, jj = (qr[i].ph >> 2) * 2;
            if (part == 2) {
                // V is kept channel-major: row kv_len + m of channels jj, jj+1, jj+d/2, jj+1+d/2
                auto col = gp(a->lin_vc) + (size_t)head * a->v_stride_head + (size_t)(a->kv_len + m[i]);
                col[(size_t)jj * a->v_stride_ch] = (half_t)v[i][0];
                col[(size_t)(jj + 1) * a->v_stride_ch] = (half_t)v[i][1];
                col[(size_t)(jj + hd) * a->v_stride_ch] = (half_t)v[i][2];
                col[(size_t)(jj + 1 + hd) * a->v_stride_ch] = (half_t)v[i][3];
                continue;
            }
            const float o0 = v[i][0] * cs[i][0] - v[i][2] * cs[i][1], o2 = v[i][2] * cs[i][0] + v[i][0] * cs[i][1];
            const float o1 = v[i][1] * cs[i][2] - v[i][3] * cs[i][3], o3 = v[i][3] * cs[i][2] + v[i][1] * cs[i][3];
            auto dst = (part == 0)
                           ? gp(a->q16) + (size_t)m[i] * H + head * d + jj
                           : gp(a->lin_kc) + (size_t)head * a->stride_head + (size_t)(a->kv_len + m[i]) * a->stride_tok + jj;
            *(GLOBAL half2_*)dst = (half2_){(half_t)o0, (half_t)o1};
            *(GLOBAL half2_*)(dst + hd) = (half2_){(half_t)o2, (half_t)o3};
        }
    }
}

template <int MT, int R, int NW>
struct LinShape {
    static constexpr int THREADS = NW * 64;
    static constexpr int NF = R * MT;                        // accumulator fragments of a wavefront
    static constexpr int CAP = 128 / NW;                     // ... reduced per round through LDS, at most
    static constexpr int ROUNDS = (NF + CAP - 1) / CAP;
    static constexpr int FR = (NF + ROUNDS - 1) / ROUNDS;    // ... and per round
    static constexpr int NB = NW == 4 ? 4 : FR > NW ? 2 : 1; // that a wavefront finishes at a time
    static constexpr size_t small_bytes = (128 + 1024 + 4) * sizeof(float);
    // HALVED: fragments of the first half that a wavefront keeps in the LDS; the rest stay in registers
    static constexpr int ROOM = (160 * 1024 - (int)small_bytes) / (NW * 1024);
    static constexpr int ASIDE = NF < ROOM ? NF : ROOM;
    // LDS of a launch, and where the small arrays begin
    template <bool HALVED>
    static constexpr size_t red_bytes = (size_t)NW * (HALVED && ASIDE > FR ? ASIDE : FR) * 1024;
    template <bool HALVED>
    static constexpr size_t lds_bytes = red_bytes<HALVED> + small_bytes;
};

// One workgroup's share: the tiles first .. first + count - 1 (count <= R; the other slots
// re-read the first tile, and what they accumulate is never looked at) over the k-steps
// k0 .. k1 - 1, for the row tiles rt0 .. rt0 + MT - 1 of x.  `finish(a, f, v, m, n0, s_rinv)` is called by one wavefront for every
// fragment f = slot * MT + row tile with the workgroup's sum v, LinShape::NB fragments at a time: one, two, or four
// in workgroups of four wavefronts (one that is not there has a row past all others); `early()` runs between
// the stream's first loads and its first wait.
//
// ROWS: x is row-major and read as it lies (16 rows x 64 bytes per load), which saves a
// separate packing launch; columns from K on are not read.  STRETCHES: see folded().  RUN: k-steps of a wavefront's turn
// (more than one: at least NW * RUN k-steps).
template <int MT, int R, int NW, bool ROWS, int STRETCHES, int SETS, int RUN, class Early, class Finish>
__device__ __forceinline__ void gemm_group(const LinHead& h, char* lds, int first, int count, int k0, int k1, int rt0,
                                           Early early, Finish finish)
{
    using S = LinShape<MT, R, NW>;
    constexpr int NF = S::NF, FR = S::FR;
    constexpr int PD = pd_of(MT, R, NW);
    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int c = lane & 15, g4 = lane >> 4;
    const uint32_t lane16 = lane * 16;                     // this lane's 16 bytes of a 1 KiB block
    floatx4* red = (floatx4*)lds;                          // [NW][FR][64]
    float* s_rinv = (float*)(lds + S::template red_bytes<(STRETCHES > 1)>);    // 128 floats
    float* s_tmp = s_rinv + 128;                           // 1024 floats
    const half8 zero8 = {0, 0, 0, 0, 0, 0, 0, 0};

    // this wavefront's k-steps, i < we: k0 + turn + i * NW.  (The turns go round so that what is left
    // over after the last whole round is spread over the pairs that the reduction adds up, and sums of
    // unlike size meet late: in the order of the wavefronts K = 136 and 320 rounded 5% worse.)  RUN > 1: see run_of.
    const int turn = NW == 8 ? (wave & 1) << 2 | (wave & 2) | wave >> 2 : (wave & 1) << 1 | wave >> 1;
    const int n = k1 - k0;
    // RUN > 1, at least RUN k-steps for everybody: `runs` of them in whole rounds, then what is left in shorter runs
    constexpr uint32_t ROUND = NW * RUN;
    const int left = (uint32_t)n % ROUND, tail = (left + NW - 1) / NW, runs = (uint32_t)n / ROUND * RUN;
    const int we = RUN == 1 ? (n - turn + NW - 1) / NW : runs + min(max(left - turn * tail, 0), tail);
    const int i_hi = max(we - 1, 0);                  // loads never go past the wavefront's last k-step
    const int kw = min(k0 + turn * RUN, k1 - 1);      // (a wavefront without a k-step requests the last one)
    // the wavefront's k-step i, which takes a place of the ring (RUN > 1: i % RUN); `last`: it may be one of those left
    auto step_of = [&](auto slot, int i, auto last) {
        constexpr int p = decltype(slot)::value;
        if constexpr (RUN == 1) return kw + i * NW;
        else if (decltype(last)::value && i - p >= runs) return k0 + runs * NW + turn * tail + p;
        else return kw + (i - p) * NW + p;
    };
    const int blk_sh = (h.flags >> kHeadBlk) & 15;
    const int mtp = ROWS ? 0 : (h.flags >> kHeadMtp) & 15;

    const char* wbase[R];                   // the slot's block of k-step 0
#pragma unroll
    for (int t = 0; t < R; ++t) {
        const int tile = first + (t < count ? t : 0);
        const int blk = (tile >> blk_sh) * (h.nks << blk_sh) + (tile & ((1 << blk_sh) - 1));
        wbase[t] = (const char*)h.W + ((size_t)(uint32_t)blk << 10);
    }
    const half_t* xrow[MT];                 // ROWS: this lane's rows of x
    if constexpr (ROWS) {
        const int M = (h.flags >> kHeadM) & 255;
#pragma unroll
        for (int b = 0; b < MT; ++b) xrow[b] = h.x + (int64_t)min((rt0 + b) * 16 + c, M - 1) * (int64_t)h.aux;
    }

    half8 wr[PD][R], xr[PD][MT];
    constexpr bool SINGLE = SETS > 0, FOLDED = folded(MT, R) && !SINGLE, HALVED = STRETCHES > 1;
    static_assert(!(FOLDED && HALVED), "one way or the other");
    static_assert(!SINGLE || SETS == PD, "a set for each k-step of the ring");
    static_assert(RUN == 1 || (RUN == PD && NW * RUN <= kRunSteps && !keeps_step(MT, R)), "a run is a turn of the ring");
    // What came before: FOLDED: the sums of earlier k-steps; HALVED: those of the first half that
    // stay in registers, as many as there are registers for.  The last NSTEP fragments are not set
    // aside but added up step by step, before the others of a step, which cover the wait for their
    // products ([32000, 4096] at 128 rows: 64 us with 22 of them; 78 with all 26 that the LDS does not
    // hold, after the others).
    constexpr int NSTEP = HALVED && NF - S::ASIDE > 13 ? NF - S::ASIDE - (NF > 60 ? 4 : 12) : 0;
    constexpr int NB = FOLDED ? NF : HALVED ? NF - S::ASIDE - NSTEP : 0;
    floatx4 acc[R][MT], before[NB > 0 ? NB : 1];
    const floatx4 zero4 = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int f = 0; f < NF; ++f) acc[f / MT][f % MT] = zero4;
#pragma unroll
    for (int f = 0; f < NB; ++f) before[f] = zero4;
    floatx4 sums[SINGLE ? SETS : 1][SINGLE ? NF : 1];
    if constexpr (SINGLE) {
#pragma unroll
        for (int i = 0; i < SETS * NF; ++i) sums[i / NF][i % NF] = zero4;
    }
    const bool long_chains = (h.flags >> kHeadLong) & 1;
    auto fold = [&]() {
        if (!long_chains) return;              // (uniform)
#pragma unroll
        for (int f = 0; f < NB; ++f) {
            before[f] += acc[f / MT][f % MT];
            acc[f / MT][f % MT] = zero4;
        }
    };
    floatx4* const aside = red + (size_t)wave * S::ASIDE * 64 + lane;      // HALVED; this lane's alone
    auto set_aside = [&](bool again) {
#pragma unroll
        for (int f = 0; f < NF - NSTEP; ++f) {
            const bool more = STRETCHES > 2 && again;
            if (f < S::ASIDE) aside[f * 64] = more ? aside[f * 64] + acc[f / MT][f % MT] : acc[f / MT][f % MT];
            else if (STRETCHES > 2) before[f - S::ASIDE] += acc[f / MT][f % MT];
            else before[f - S::ASIDE] = acc[f / MT][f % MT];
            acc[f / MT][f % MT] = zero4;
            if (f % 8 == 7) pin_order();       // (few registers at a time)
        }
    };

    auto load = [&](auto slot, int i, auto last) {
        constexpr int p = decltype(slot)::value;
        const int s = step_of(slot, i, last);
        if constexpr (ROWS) {
            const int col = min(s * 32 + g4 * 8, h.K - 8);
#pragma unroll
            for (int b = 0; b < MT; ++b) xr[p][b] = *(const half8*)(xrow[b] + col);
        } else {
            const char* xq = (const char*)h.x + ((size_t)(uint32_t)(s * mtp + rt0) << 10);
#pragma unroll
            for (int b = 0; b < MT; ++b) xr[p][b] = *(const half8*)(xq + (b << 10) + lane16);
        }
#pragma unroll
        for (int t = 0; t < R; ++t) {
            const char* wq = wbase[t] + ((size_t)(uint32_t)(s << blk_sh) << 10);
            wr[p][t] = __builtin_nontemporal_load((const half8*)(wq + lane16));
        }
    };
    // MASKED: columns from K on count as zeros (the x fragments are zeroed: one select for all slots)
    auto compute = [&](auto masked, auto slot, int i, auto last) {
        constexpr int p = decltype(slot)::value;
        constexpr bool MASKED = decltype(masked)::value;
        half8 xf[MT];
        if constexpr (MASKED) {
            const bool use = step_of(slot, i, last) * 32 + g4 * 8 < h.K;
#pragma unroll
            for (int b = 0; b < MT; ++b) xf[b] = use ? xr[p][b] : zero8;
        } else {
#pragma unroll
            for (int b = 0; b < MT; ++b) xf[b] = xr[p][b];
        }
#pragma unroll
        for (int tt = 0; tt < R; ++tt)
#pragma unroll
            for (int bb = 0; bb < MT; ++bb) {
                const int t = NSTEP ? R - 1 - tt : tt, b = NSTEP ? MT - 1 - bb : bb;
                if constexpr (SINGLE) sums[p % SETS][t * MT + b] += __builtin_amdgcn_mfma_f32_16x16x32_f16(wr[p][t], xf[b], zero4, 0, 0, 0);
                else if (t * MT + b >= NF - NSTEP) acc[t][b] += __builtin_amdgcn_mfma_f32_16x16x32_f16(wr[p][t], xf[b], zero4, 0, 0, 0);
                else acc[t][b] = __builtin_amdgcn_mfma_f32_16x16x32_f16(wr[p][t], xf[b], acc[t][b], 0, 0, 0);
            }
    };
    auto prologue = [&](auto self, auto slot) {
        constexpr int p = decltype(slot)::value;
        if constexpr (p < PD) {
            load(slot, RUN == 1 ? min(p, i_hi) : p, std::false_type{});
            pin_order();
            self(self, std::integral_constant<int, p + 1>{});
        }
    };
    const int common = n / NW;              // k-steps that every wavefront has
    auto ring = [&](auto self, auto slot, int s) {
        constexpr int p = decltype(slot)::value;
        if constexpr (p < PD) {
            if constexpr (p == 0 && keeps_step(MT, R)) {
                // (a turn that every wavefront takes: all come to as many barriers)
                if (s + 2 * PD <= common) {
                    __builtin_amdgcn_s_barrier();
                    pin_order();
                }
            }
            compute(std::false_type{}, slot, s + p, std::false_type{});
            pin_order();
            load(slot, s + p + PD, std::false_type{});
            pin_order();
            self(self, std::integral_constant<int, p + 1>{}, s);
        }
    };
    // the last steps, PD of which are in the ring already: nothing is requested past the range
    auto drain = [&](auto self, auto slot, int s) {
        constexpr int p = decltype(slot)::value;
        if constexpr (p < 2 * PD - 1) {
            auto step = [&]() {
                compute(std::true_type{}, std::integral_constant<int, p % PD>{}, s + p, std::bool_constant<(p >= PD)>{});
                pin_order();
                if constexpr (FOLDED && p % kFoldSteps == kFoldSteps - 1) fold();
                if constexpr (p < PD - 1) {
                    if (s + p + PD < we) load(std::integral_constant<int, p % PD>{}, s + p + PD, std::true_type{});
                    pin_order();
                }
            };
            // (nested conditions leave the loop sooner; four wavefronts' accumulators would be
            // copied at every exit)
            if constexpr (NW == 8) {
                if (s + p < we) {
                    step();
                    self(self, std::integral_constant<int, p + 1>{}, s);
                }
            } else {
                if (s + p < we) step();
                self(self, std::integral_constant<int, p + 1>{}, s);
            }
        }
    };

    prologue(prologue, std::integral_constant<int, 0>{});
    early();
    const ArgPtr a = late_args();

    // RMSNorm factor per row from the per-tile sums of squares ss[tile][Mpad], in two steps.
    // Early, here, where the stream's first loads are waited for anyway: thread (rq, part) adds 4
    // rows of every P-th tile and the lanes of a wavefront that share rq are combined by
    // shuffles.  Late, when the stream is over and the workgroup meets anyway: the wavefronts'
    // sums are added through LDS.  Fixed order throughout.
    constexpr int MTP = layout_tiles(MT), RQ = MTP * 4, P = S::THREADS / RQ;
    floatx4 rs4 = {0.f, 0.f, 0.f, 0.f};
    const bool rscale = !ROWS && h.aux != 0;
    if (rscale) {
        const auto ss = gp((const float*)h.aux);
        const int n_ss = h.K >> 4, rq = tid % RQ;
        for (int t0 = tid / RQ; t0 < n_ss; t0 += 8 * P) {
            floatx4 sst[8];
#pragma unroll
            for (int q = 0; q < 8; ++q)
                sst[q] = *(GLOBAL const floatx4*)(ss + (size_t)min(t0 + q * P, n_ss - 1) * (mtp * 16) + rt0 * 16 + rq * 4);
#pragma unroll
            for (int q = 0; q < 8; ++q)
                if (t0 + q * P < n_ss) rs4 += sst[q];
        }
        for (int off = RQ; off < 64; off <<= 1) {
#pragma unroll
            for (int r = 0; r < 4; ++r) rs4[r] += __shfl_xor(rs4[r], off);
        }
    }

    if (we > 0) {
        int s = 0;
        if constexpr (FOLDED) {
            constexpr int ROUNDS = (kFoldSteps + PD - 1) / PD;
            for (; s + (ROUNDS + 1) * PD <= we; s += ROUNDS * PD) {
#pragma unroll
                for (int r = 0; r < ROUNDS; ++r) ring(ring, std::integral_constant<int, 0>{}, s + r * PD);
                fold();
            }
            if constexpr (ROUNDS > 1) {
                for (; s + 2 * PD <= we; s += PD) ring(ring, std::integral_constant<int, 0>{}, s);
                fold();
            }
        } else {
            auto stream = [&](int end) {
                for (; s + 2 * PD <= we && s < end; s += PD) ring(ring, std::integral_constant<int, 0>{}, s);
            };
            if constexpr (STRETCHES == 2 && NW == 8) {
                // (written out twice, what is set aside needs no registers in the first stretch)
                if (long_chains) {
                    stream(we / 2);
                    set_aside(false);
                }
                stream(we);
            } else {
                // (once: the code is fetched while it runs)
                const int stretches = long_chains ? STRETCHES : 1;
                for (int i = 1;; ++i) {
                    stream(i == stretches ? we : we * i / STRETCHES);
                    if (i == stretches) break;
                    set_aside(i > 1);
                }
            }
        }
        drain(drain, std::integral_constant<int, 0>{}, s);
    }
    if constexpr (SINGLE) {
#pragma unroll
        for (int f = 0; f < NF; ++f) {
#pragma unroll
            for (int d = 1; d < SETS; d *= 2)
#pragma unroll
                for (int i = 0; i + d < SETS; i += 2 * d) sums[i][f] += sums[i + d][f];
            acc[f / MT][f % MT] = sums[0][f];
        }
    }
    if constexpr (FOLDED) {
        if (long_chains) {
#pragma unroll
            for (int f = 0; f < NB; ++f) acc[f / MT][f % MT] += before[f];
        }
    }
    if constexpr (HALVED) {
        if (long_chains) {
            if (we > 0) {
#pragma unroll
                for (int f = 0; f < NF - NSTEP; ++f) {
                    if (f < S::ASIDE) acc[f / MT][f % MT] += aside[f * 64];
                    else acc[f / MT][f % MT] += before[f - S::ASIDE];
                    if (f % 8 == 7) pin_order();
                }
            }
            __syncthreads();       // (the reduction lays the same LDS out in another way)
        }
    }

    // ---- the wavefronts' k slices are added up through LDS, FR fragments of every wavefront
    //      per round, in a fixed order; wavefront w has sums w, w + NW, ... of the round
    if (rscale) {
        if (lane < RQ) *(floatx4*)(s_tmp + (wave * RQ + lane) * 4) = rs4;
        __syncthreads();
        if (tid < MTP * 16) {
            float tot = 0.f;
            for (int w = 0; w < NW; ++w) tot += s_tmp[(w * RQ + (tid >> 2)) * 4 + (tid & 3)];
            s_rinv[tid] = (1.0f / kXgScale) / sqrtf(tot / (float)h.K + a->eps);
        }
        // (the first barrier of the reduction makes s_rinv visible)
    }
#pragma unroll
    for (int r0 = 0; r0 < NF; r0 += FR) {
        if (r0) __syncthreads();
#pragma unroll
        for (int ff = 0; ff < FR; ++ff)
            if (r0 + ff < NF) red[(wave * FR + ff) * 64 + lane] = acc[(r0 + ff) / MT][(r0 + ff) % MT];
        __syncthreads();
        constexpr int NB = S::NB;
#pragma unroll 1
        for (int f0 = 0; f0 < FR; f0 += NB * NW) {
            if (f0 + wave >= FR || r0 + f0 + wave >= NF || (r0 + f0 + wave) / MT >= count) break;     // (nor any later one)
            floatx4 v[NB], part[NB][NW];
            int f[NB], m[NB], n0[NB];
#pragma unroll
            for (int i = 0; i < NB; ++i) {
                const int ff = f0 + i * NW + wave;
                f[i] = r0 + ff;
                const int t = f[i] / MT, b = f[i] % MT;
                m[i] = ff < FR && f[i] < NF && t < count ? (rt0 + b) * 16 + c : kNoRow;
                n0[i] = (first + t) * 16 + g4 * 4;
                // (what is read for a fragment that is not there is not looked at)
#pragma unroll
                for (int w = 0; w < NW; ++w) part[i][w] = red[(w * FR + min(ff, FR - 1)) * 64 + lane];
            }
            // (pairs of pairs: half the roundings of one sum after the other)
#pragma unroll
            for (int i = 0; i < NB; ++i) {
#pragma unroll
                for (int d = 1; d < NW; d *= 2)
#pragma unroll
                    for (int w = 0; w < NW; w += 2 * d) part[i][w] += part[i][w + d];
                v[i] = part[i][0];
            }
            finish(a, f, v, m, n0, s_rinv - rt0 * 16);
        }
    }
}

// The tiles [c0, c1) of workgroup i (i % 8 stands for its XCD) when `ntiles` tiles are dealt to the 8
// XCDs in contiguous blocks, x * ntiles / 8 and on, and an XCD's U tiles to its gx workgroups in
// contiguous runs, w * U / gx and on (single tiles to the first U if U < gx), without a division:
// magic = 2^32 / gx + 1, gx > 1; exact while U times gx stays below 2^32 / gx.
__host__ __device__ __forceinline__ void tile_range(int ntiles, int gx, uint32_t magic, int i, int* c0, int* c1)
{
    const int x = i & 7, w = i >> 3;
    const int i0 = (int)((unsigned)ntiles * (unsigned)x >> 3), U = (int)((unsigned)ntiles * (unsigned)(x + 1) >> 3) - i0;
    if (U < gx) {
        *c0 = i0 + (w < U ? w : U);
        *c1 = i0 + (w + 1 < U ? w + 1 : U);
    } else {
        *c0 = i0 + (int)(((uint64_t)((unsigned)U * (unsigned)w) * magic) >> 32);
        *c1 = i0 + (int)(((uint64_t)((unsigned)U * (unsigned)(w + 1)) * magic) >> 32);
    }
}

// ---- whole tiles ----------------------------------------------------------------------
// GROUPS: of workgroups, with the same tiles and different rows of x.  RUN: see run_of.
template <int MT, int R, bool ROWS, bool GROUPS, int RUN>
__global__ __launch_bounds__(waves_of(MT, R) * 64) void k_linear(const half8* W, const half_t* x, uint64_t aux, int nks, int K,
                                                    int ntiles, int cut, uint32_t magic, uint32_t flags,
                                                    const FusedArgs)
{
    extern __shared__ __attribute__((aligned(16))) char lds[];
    const LinHead h = {W, x, aux, nks, K, ntiles, cut, magic, flags};
    // the group of rows, and the workgroup's number in it
    const int w = blockIdx.x >> 3, group = GROUPS ? (int)(((uint64_t)(uint32_t)w * magic) >> 32) : 0;
    int c0, c1;
    tile_range(ntiles, cut, magic, (w - group * cut) << 3 | (blockIdx.x & 7), &c0, &c1);
    // A call of its own that is dealt out in whole tiles needs nothing that a set-up kernel
    // prepares; the workspace's status words are brought up to date here (nothing else in
    // the launch touches them).
    auto solo = [&]() {
        if (((flags >> kHeadSolo) & 1) && blockIdx.x == 0 && threadIdx.x == 0) carry_status(late_args()->sync);
    };
    if (c0 >= c1) {
        solo();
        return;
    }
    const int lane = threadIdx.x & 63;
    gemm_group<MT, R, waves_of(MT, R), ROWS, stretches_whole(MT, R), GROUPS ? kSingleSets : 0, RUN>(
        h, lds, c0, c1 - c0, 0, nks, group * MT, solo,
        [&](ArgPtr a, auto&, auto& v, auto& m, auto& n0, const float* s_rinv) { epilogue(a, v, m, n0, lane, s_rinv); });
}

// ---- parts --------------------------------------------------------------------------
// Workgroups i with the same i % 8 run on one XCD (checked, see arrive); of those, S consecutive
// ones are the parts of one block of R tiles, and the blocks are dealt to the XCDs in turn.
template <int MT, int R>
__global__ __launch_bounds__(512) void k_linear_parts(const half8* W, const half_t* x, uint64_t aux, int nks, int K,
                                                      int ntiles, int cut, uint32_t magic, uint32_t flags,
                                                      const FusedArgs)
{
    extern __shared__ __attribute__((aligned(16))) char lds[];
    const LinHead h = {W, x, aux, nks, K, ntiles, cut, magic, flags};
    const int S = cut, xcd = blockIdx.x & 7, w = blockIdx.x >> 3;
    const int bx = (int)(((uint32_t)w * magic) >> 16), part = w - bx * S;
    const int first = (bx * 8 + xcd) * R;
    if (first >= ntiles) return;
    const int count = min(R, ntiles - first);
    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int k0 = nks * part / S, k1 = nks * (part + 1) / S;
    constexpr int NF = R * MT;
    const int f0 = count * MT * part / S, f1 = count * MT * (part + 1) / S;     // what this part finishes

    // partial sums: one slot of NF fragments per workgroup; the block's parts are eight
    // workgroups apart
    const int slot0 = bx * S * 8 + xcd;
    gemm_group<MT, R, 8, false, stretches_parts(MT, R), 0, 1>(
        h, lds, first, count, k0, k1, 0, []() {},
        [&](ArgPtr a, auto& f, auto& v, auto& m, auto&, const float*) {
            for (int i = 0; i < (int)(sizeof(f) / sizeof(f[0])); ++i)
                if (m[i] != kNoRow) *(GLOBAL floatx4*)(gp(a->part) + ((size_t)(slot0 + part * 8) * NF + f[i]) * 256 + lane * 4) = v[i];
        });
    const ArgPtr a = late_args();
    const float* s_rinv = (const float*)(lds + LinShape<MT, R, 8>::template red_bytes<(stretches_parts(MT, R) > 1)>);
    int* s_wait_ok = (int*)(s_rinv + 128 + 1024);
    const int c = lane & 15, g4 = lane >> 4;
    const auto position = [&](int f, int* m, int* n0) {
        *m = (f % MT) * 16 + c;
        *n0 = (first + f / MT) * 16 + g4 * 4;
    };
    wait_own_stores();                       // the partials are in the L2
    __syncthreads();
    // What the residual epilogue reads is requested while the workgroup waits, where there is much of it, but not by
    // the wavefront that polls (loads return in order: its polls would come back behind them): the last
    // wavefront has the first fragment.  [5120, 13824] at 64 rows and [4096, 11008]: 0.5 us a launch.
    constexpr bool AHEAD = MT > 2;
    const int mine = f0 + (AHEAD ? 7 - wave : wave);
    ResidOperands ops[1] = {};
    int m[1], n0[1];
    if (AHEAD && wave != 0 && mine < f1 && a->lin_epi == EPI_RESID) {
        position(mine, m, n0);
        ops[0] = resid_operands(a, m[0], n0[0]);
    }
    uint32_t* const cnt = a->sync + a->lin_cnt + slot0 * kCntStride;
    if (tid == 0) {
        uint32_t* const word = epoch_word(cnt, a->lin_epoch);
        const uint32_t seen = arrive(word);
        *s_wait_ok = bounded_wait(a->sync, word, seen, (uint32_t)S, (uint32_t)S, 1000u + a->lin_epi);
        if (part == 0) clear_next(cnt, a->lin_epoch);
    }
    __syncthreads();
    if (!*s_wait_ok) return;                 // the other parts never arrived: nothing sensible to write
    for (int f = mine; f < f1; f += 8) {
        // the parts in index order (fixed order: the result does not depend on timing), eight
        // loads in flight at a time
        const auto src = gp((const float*)a->part) + ((size_t)slot0 * NF + f) * 256 + lane * 4;
        position(f, m, n0);
        if ((!AHEAD || wave == 0 || f != mine) && a->lin_epi == EPI_RESID) ops[0] = resid_operands(a, m[0], n0[0]);
        floatx4 v[1] = {{0.f, 0.f, 0.f, 0.f}};
        for (int p0 = 0; p0 < S; p0 += 8) {
            floatx4 t[8];
#pragma unroll
            for (int q = 0; q < 8; ++q)
                if (p0 + q < S) t[q] = *(GLOBAL const floatx4*)(src + (size_t)(p0 + q) * (8 * NF * 256));
#pragma unroll
            for (int q = 0; q < 8; ++q)
                if (p0 + q < S) v[0] += t[q];
        }
        epilogue(a, v, m, n0, lane, s_rinv, ops);
    }
}

// ---- launches -----------------------------------------------------------------------
static inline LinHead head_of(const FusedArgs& a, const LinCut& cut)
{
    const WLayout lay = w_layout(a.lin_N, a.lin_K);
    LinHead h;
    h.W = a.lin_W;
    h.x = a.lin_x;
    h.aux = cut.rows ? (uint64_t)a.lin_ldx : a.lin_rscale ? (uint64_t)(uintptr_t)a.ss : 0;
    h.nks = lay.nks;
    h.K = a.lin_K;
    h.ntiles = lay.ntiles;
    h.cut = cut.whole ? cut.grid / 8 / cut.groups : cut.parts;
    h.magic = (uint32_t)((cut.whole ? 0x100000000ull : 0x10000ull) / (uint64_t)h.cut + 1);
    h.flags = (uint32_t)(lay.blk == kWideBlock ? 3 : 2) << kHeadBlk | (uint32_t)(a.Mpad / 16) << kHeadMtp |
              (uint32_t)a.M << kHeadM | (uint32_t)(a.lin_solo != 0) << kHeadSolo;
    static_assert(kWideBlock == 8 && kRbNarrow == 4, "storage blocks of 8 or 4 tiles");
    return h;
}

// Are a cut's chains (k-steps of a wavefront) longer than an even deal over all compute units, eight
// wavefronts each, would make them: of whole tiles for wide matrices, of the k-steps of four-tile
// blocks for narrow ones?  Pairwise sums of the wavefronts make up for half a k-step, with four of
// them for a whole one.
static inline bool long_chains(const WLayout& lay, const LinCut& cut, int waves)
{
    const double chain = (double)ceil_div(lay.nks, cut.parts) / waves;
    double even = lay.nks / 8.0;
    if (lay.rb != 1) {
        const double share = (double)lay.nitems / kRangeWgs;
        even *= share;
        // (a run of k-steps that goes over a block's end is two chains)
        if (kRangeWgs % lay.nitems != 0) even *= 1.0 - share / 3.0;
    }
    return chain >= 2.0 && chain > even + (waves == 8 ? 0.5 : 1.0);
}

template <class Kernel>
static ghd_status launch_linear_kernel(Kernel kernel, const FusedArgs& a, const LinCut& cut, int threads, size_t lds,
                                       hipStream_t st)
{
    ghd_status s = launch_resident_checked((const void*)kernel, threads, lds);
    if (s) return s;
    LinHead h = head_of(a, cut);
    if (long_chains(w_layout(a.lin_N, a.lin_K), cut, threads / 64)) h.flags |= 1u << kHeadLong;
    hipLaunchKernelGGL(kernel, dim3(cut.grid), dim3(threads), lds, st, h.W, h.x, h.aux, h.nks, h.K, h.ntiles, h.cut,
                       h.magic, h.flags, a);
    return check_launch();
}

// the instantiations for one number of row tiles of x
template <int MT, int R>
ghd_status launch_linear_r(const FusedArgs& a, const LinCut& cut, hipStream_t st)
{
    if (cut.tiles == R && cut.whole) {
        constexpr int threads = waves_of(MT, R) * 64;
        constexpr size_t lds = LinShape<MT, R, waves_of(MT, R)>::template lds_bytes<(stretches_whole(MT, R) > 1)>;
        constexpr int RUN = run_of(MT, R);
        const bool runs = run_of_launch(cut, w_layout(a.lin_N, a.lin_K).nks) > 1;
        if constexpr (grouped(MT, R))
            if (cut.groups > 1) {
                if (runs)
                    return launch_linear_kernel(cut.rows ? k_linear<MT, R, true, true, RUN> : k_linear<MT, R, false, true, RUN>, a, cut,
                                                threads, lds, st);
                return launch_linear_kernel(cut.rows ? k_linear<MT, R, true, true, 1> : k_linear<MT, R, false, true, 1>, a, cut,
                                            threads, lds, st);
            }
        if (cut.groups > 1) return GHD_ERR_SHAPE;
        if constexpr (MT <= kRowsMaxMT)
            if (cut.rows)
                return launch_linear_kernel(runs ? k_linear<MT, R, true, false, RUN> : k_linear<MT, R, true, false, 1>, a, cut, threads,
                                            lds, st);
        if (cut.rows) return GHD_ERR_SHAPE;
        return launch_linear_kernel(runs ? k_linear<MT, R, false, false, RUN> : k_linear<MT, R, false, false, 1>, a, cut, threads, lds,
                                    st);
    }
    if constexpr (R <= parts_max_tiles(MT))
        if (cut.tiles == R)
            return launch_linear_kernel(k_linear_parts<MT, R>, a, cut, 512, LinShape<MT, R, 8>::template lds_bytes<(stretches_parts(MT, R) > 1)>, st);
    if constexpr (R < 8) return launch_linear_r<MT, R + 1>(a, cut, st);
    return GHD_ERR_SHAPE;
}

ghd_status launch_linear_mt1(const FusedArgs& a, const LinCut& cut, hipStream_t st);
ghd_status launch_linear_mt2(const FusedArgs& a, const LinCut& cut, hipStream_t st);
ghd_status launch_linear_mt3(const FusedArgs& a, const LinCut& cut, hipStream_t st);
ghd_status launch_linear_mt4(const FusedArgs& a, const LinCut& cut, hipStream_t st);
ghd_status launch_linear_mt6(const FusedArgs& a, const LinCut& cut, hipStream_t st);
ghd_status launch_linear_mt8(const FusedArgs& a, const LinCut& cut, hipStream_t st);

}  // namespace ghd
