// The drafting side of a decoding step (Ghidorah, section 2.1: tokens for several future
// slots are predicted, then verified in one pass; section 2.3: with self-drafting the
// predictions come from extra heads at the tail of the model, several candidates per head;
// section 3.3.1: the candidates are combined into the verification tree).
//   k_embed       : hidden states of the tree's tokens, rows of the embedding table;
//   k_pick_norm   : the final hidden state of the last accepted node, RMS-normalised with
//                   the final gain, as the fp16 input row of the heads' linear layer (the
//                   K heads are one stacked [K*V, H] matrix: one skinny linear launch);
//   k_topk_segment, k_topk_tokens : the R best candidates of every head, best first, lowest
//                   index on ties, and the tokens of the next tree: the root carries the
//                   token the model has just produced, a node at depth t candidate rank[i]
//                   of head t - 1.
// Also the host-side tree design from head accuracies (section 3.3.1).
#include "common.h"

#include <queue>
#include <vector>

namespace ghd {

__global__ __launch_bounds__(256) void k_embed(half8* __restrict__ x, const half8* __restrict__ table,
                                               const int32_t* __restrict__ tokens, int H8, int V)
{
    const int i = blockIdx.x;
    int t = tokens[i];
    t = t < 0 ? 0 : (t >= V ? V - 1 : t);     // a corrupt token cannot reach outside the table
    for (int j = threadIdx.x; j < H8; j += 256) x[(size_t)i * H8 + j] = table[(size_t)t * H8 + j];
}

constexpr int kPickThreads = 1024;

// One workgroup.  Bound by its chain of latencies: argument block, accepted length, last node, that node's row, sum, stores.
// A thread has four consecutive channels at a time, and keeps the first two of these pieces between the sum and the scaling
// (4096 channels 5.4 us, one channel at a time and read twice, and 5.1).
__global__ __launch_bounds__(kPickThreads) void k_pick_norm(const float* __restrict__ x_final,
                                                            const int32_t* __restrict__ res, int M, int H,
                                                            const half_t* __restrict__ g, float eps,
                                                            half_t* __restrict__ n16)
{
    __shared__ float s_part[kPickThreads / 64];
    constexpr int kKeep = 2;
    const int tid = threadIdx.x, H4 = H >> 2;              // (H is a multiple of 8, and all rows are 16-byte aligned)
    half4 gain[kKeep];
#pragma unroll
    for (int u = 0; u < kKeep; ++u) gain[u] = ((const half4*)g)[min(tid + u * kPickThreads, H4 - 1)];
    int len = res[0];
    len = len < 1 ? 1 : (len > M ? M : len);
    int last = res[2 + len - 1];
    last = last < 0 ? 0 : (last >= M ? M - 1 : last);
    const floatx4* row = (const floatx4*)(x_final + (size_t)last * H);
    floatx4 x[kKeep];
#pragma unroll
    for (int u = 0; u < kKeep; ++u) x[u] = row[min(tid + u * kPickThreads, H4 - 1)];
    auto squares = [](floatx4 v) { return (v[0] * v[0] + v[1] * v[1]) + (v[2] * v[2] + v[3] * v[3]); };
    float s = 0.f;
#pragma unroll
    for (int u = 0; u < kKeep; ++u)
        if (tid + u * kPickThreads < H4) s += squares(x[u]);
    for (int j = tid + kKeep * kPickThreads; j < H4; j += kPickThreads) s += squares(row[j]);
    for (int off = 32; off > 0; off >>= 1) s += __shfl_xor(s, off);
    if ((tid & 63) == 0) s_part[tid >> 6] = s;
    __syncthreads();
    float tot = 0.f;
    for (int w = 0; w < kPickThreads / 64; ++w) tot += s_part[w];
    const float rinv = 1.0f / sqrtf(tot / (float)H + eps);
    auto scaled = [&](floatx4 v, half4 gv) {
        half4 o;
#pragma unroll
        for (int e = 0; e < 4; ++e) o[e] = (half_t)(v[e] * rinv * (float)gv[e]);
        return o;
    };
#pragma unroll
    for (int u = 0; u < kKeep; ++u)
        if (tid + u * kPickThreads < H4) ((half4*)n16)[tid + u * kPickThreads] = scaled(x[u], gain[u]);
    for (int j = tid + kKeep * kPickThreads; j < H4; j += kPickThreads)
        ((half4*)n16)[j] = scaled(row[j], ((const half4*)g)[j]);
}

// ---- the R best candidates of every head, then the next tree's tokens ----------------------
// Bound by latency: the K heads' logits are 640 KB at 5 x 32000, far less than a microsecond of
// HBM time, so what counts is how many compute units look at them and how long the chain of R
// dependent picks is.  One workgroup per head with R passes over its whole row took 80 us there.
// Now every head's row is cut into segments of kSegLen entries, one workgroup each: a
// wavefront holds 512 entries in registers, in order in every lane, picks its R best in R rounds (a DPP
// maximum over the lanes' first ones, no LDS and no barrier), a candidate's place among the four wavefronts' is
// counted, and one last workgroup merges the segments' lists, a wavefront per head, and
// writes the tokens.  At 5 x 32000, R = 10: 80 + 4.6 us in the beginning, 7.3 + 6.4 with rounds over all of a lane's keys
// in 64 bits and a second set of rounds for the four lists, 7.0 + 4.9 now.
//
// A candidate is one 64-bit key whose unsigned order is the order of the picks: larger value
// first, lower index first among equal values (-0 equals +0).  0 stands for "none": a NaN
// compares with nothing and is never picked.
constexpr int kSegWaves = 4;                     // wavefronts of a segment's workgroup
constexpr int kPerLane = 8;                      // entries a lane holds
constexpr int kSegLen = kSegWaves * 64 * kPerLane;
constexpr int kMaxPicks = 32;                    // R (checked on the host)

__device__ __forceinline__ uint64_t cand_key(float v, int idx)
{
    uint32_t b = __float_as_uint(v + 0.0f);
    b ^= (uint32_t)((int32_t)b >> 31) | 0x80000000u;
    return v == v ? ((uint64_t)b << 32) | (uint32_t)~idx : 0ull;
}
__device__ __forceinline__ int cand_index(uint64_t key) { return (int)~(uint32_t)key; }

// v's maximum with the lane that the DPP control word names (the lane itself where there is none)
template <int CTRL>
__device__ __forceinline__ uint32_t max_dpp(uint32_t v)
{
    const uint32_t o = (uint32_t)__builtin_amdgcn_update_dpp((int)v, (int)v, CTRL, 0xf, 0xf, false);
    return o > v ? o : v;
}

// maximum over the wavefront, uniform
__device__ __forceinline__ uint32_t wave_max(uint32_t v)
{
    v = max_dpp<0xB1>(v);      // quad_perm 1,0,3,2
    v = max_dpp<0x4E>(v);      // quad_perm 2,3,0,1
    v = max_dpp<0x141>(v);     // row_half_mirror
    v = max_dpp<0x140>(v);     // row_mirror: every lane has its row's maximum
    v = max_dpp<0x142>(v);     // row_bcast15
    v = max_dpp<0x143>(v);     // row_bcast31: lane 63 has the wavefront's
    return (uint32_t)__builtin_amdgcn_readlane((int)v, 63);
}

// a lane's keys, largest first (Batcher's merge exchange, for any E)
template <int E>
__device__ __forceinline__ void sort_keys(uint64_t (&key)[E])
{
#pragma unroll
    for (int p = 1; p < E; p *= 2)
#pragma unroll
        for (int k = p; k >= 1; k /= 2)
#pragma unroll
            for (int i = 0; i + k < E; ++i) {
                // (pairs i, i + k of a run of k from j = k % p on, 2 k apart, inside one block of 2 p)
                const int from = i - k % p;
                if (from < 0 || from / k % 2 != 0 || i / (2 * p) != (i + k) / (2 * p)) continue;
                const uint64_t a = key[i], b = key[i + k];
                const bool swap = b > a;
                key[i] = swap ? b : a;
                key[i + k] = swap ? a : b;
            }
}

// lane r (r < R <= 64) gets the r-th best of the wavefront's keys, 0 when there are fewer.  With its keys in order
// a lane offers its first one; the maximum is taken over the values, and over the indexes only where lanes
// tie (a maximum over all of a lane's keys, 64 bits wide, and a look at each of them took twice the instructions a round).
template <int E>
__device__ __forceinline__ uint64_t wave_topk(uint64_t (&key)[E], int R, int lane)
{
    sort_keys(key);
    uint64_t mine = 0;
    for (int r = 0; r < R; ++r) {
        const uint32_t value = (uint32_t)(key[0] >> 32), index = (uint32_t)key[0];
        const uint32_t best = wave_max(value);
        if (best == 0) break;                  // (no number's upper word is 0)
        const uint64_t with = __ballot(value == best);
        const uint32_t first = (with & (with - 1)) == 0
                                   ? (uint32_t)__builtin_amdgcn_readlane((int)index, __builtin_ctzll(with))
                                   : wave_max(value == best ? index : 0u);
        if (lane == r) mine = ((uint64_t)best << 32) | first;
        const bool taken = value == best && index == first;
#pragma unroll
        for (int e = 0; e < E; ++e) key[e] = taken ? (e + 1 < E ? key[e + 1 < E ? e + 1 : e] : 0ull) : key[e];
    }
    return mine;
}

// one workgroup per (head, segment): lists[head][segment][R]
__global__ __launch_bounds__(kSegWaves * 64) void k_topk_segment(const float* __restrict__ logits, int V, int R,
                                                                 int nseg, uint64_t* __restrict__ lists)
{
    __shared__ __attribute__((aligned(16))) uint64_t s_list[kSegWaves * kMaxPicks];
    __shared__ int s_n[kSegWaves];
    const int head = blockIdx.x / nseg, seg = blockIdx.x - head * nseg;
    const int tid = threadIdx.x, wave = tid >> 6, lane = tid & 63;
    const float* row = logits + (size_t)head * V;
    const int at = seg * kSegLen + wave * (64 * kPerLane) + lane;
    float v[kPerLane];
#pragma unroll
    for (int e = 0; e < kPerLane; ++e) v[e] = row[min(at + e * 64, V - 1)];
    uint64_t key[kPerLane];
#pragma unroll
    for (int e = 0; e < kPerLane; ++e) key[e] = at + e * 64 < V ? cand_key(v[e], at + e * 64) : 0ull;
    const uint64_t mine = wave_topk(key, R, lane);
    if (lane < R) s_list[wave * R + lane] = mine;
    const int n = __popcll(__ballot(mine != 0));
    if (lane == 0) s_n[wave] = n;
    __syncthreads();
    // The four lists in one: a candidate's place is the number of larger ones.
    uint64_t* const out = lists + ((size_t)head * nseg + seg) * R;
    if (lane >= R) return;
    int place = 0, all = 0;
#pragma unroll 4
    for (int j = 0; j < kSegWaves * R; ++j) place += s_list[j] > mine;
#pragma unroll
    for (int w = 0; w < kSegWaves; ++w) all += s_n[w];
    if (mine != 0 && place < R) out[place] = mine;
    if (wave == 0 && lane >= all) out[lane] = 0;
}

constexpr int kPickWaves = 16;                   // K (checked on the host)
constexpr int kFewPerLane = 3;                   // (19 segments of 10 candidates: putting 9 keys in order takes 28 exchanges, 3 take 3)

// a lane's entries of a list of n from c0 on, 0 past its end
template <int E>
__device__ __forceinline__ void list_keys(const uint64_t* __restrict__ list, int c0, int n, int lane, uint64_t (&key)[E])
{
#pragma unroll
    for (int e = 0; e < E; ++e) key[e] = list[min(c0 + e * 64 + lane, n - 1)];
#pragma unroll
    for (int e = 0; e < E; ++e)
        if (c0 + e * 64 + lane >= n) key[e] = 0;
}

constexpr int kNodeThreads = GHD_MAX_M;

// one workgroup: wavefront k merges head k's lists, while the last wavefronts, a thread per node, find the nodes'
// depths, each from a copy of parent[] of its own; then the nodes' tokens are written
__global__ __launch_bounds__(kPickWaves * 64) void k_topk_tokens(const uint64_t* __restrict__ lists, int nseg,
                                                                 int32_t* __restrict__ tokens,
                                                                 const int32_t* __restrict__ parent,
                                                                 const int32_t* __restrict__ rank, int M,
                                                                 int32_t* __restrict__ topk, int K, int R,
                                                                 const int32_t* __restrict__ res, int V)
{
    __shared__ int32_t s_parent[kNodeThreads / 64][GHD_MAX_M];
    __shared__ int32_t s_top[kPickWaves * kMaxPicks];
    const int tid = threadIdx.x, wave = __builtin_amdgcn_readfirstlane(tid >> 6), lane = tid & 63;
    const int i = tid - (kPickWaves * 64 - kNodeThreads);          // the thread's node, if 0 <= i < M
    const int copy = wave - (kPickWaves - kNodeThreads / 64);
    int my_rank = 0, root = 0;
    if (copy >= 0) {
        int up[GHD_MAX_M / 64];
#pragma unroll
        for (int u = 0; u < GHD_MAX_M / 64; ++u) up[u] = parent[min(u * 64 + lane, M - 1)];
        if (i < M) {
            my_rank = rank[i];
            root = res[1];
        }
#pragma unroll
        for (int u = 0; u < GHD_MAX_M / 64; ++u) s_parent[copy][u * 64 + lane] = up[u];
    }
    if (wave < K) {
        const uint64_t* list = lists + (size_t)wave * nseg * R;
        const int n = nseg * R;
        uint64_t mine = 0;
        if (n <= 64 * kFewPerLane) {
            uint64_t key[kFewPerLane];
            list_keys(list, 0, n, lane, key);
            mine = wave_topk(key, R, lane);
        } else {
            for (int c0 = 0; c0 < n; c0 += 64 * kPerLane) {
                uint64_t key[kPerLane + 1];
                list_keys(list, c0, n, lane, reinterpret_cast<uint64_t(&)[kPerLane]>(key));
                key[kPerLane] = mine;                // what the entries before these left
                mine = wave_topk(key, R, lane);
            }
        }
        // Fewer than R entries that compare (NaNs): the last pick is repeated once (0 if there
        // is none), what follows is marked with the largest index.
        const int n_ok = __popcll(__ballot(mine != 0));
        const int last = __shfl(cand_index(mine), max(n_ok - 1, 0));
        const int idx = lane < n_ok ? cand_index(mine) : lane > n_ok ? 0x7fffffff : n_ok ? last : 0;
        if (lane < R) {
            s_top[wave * R + lane] = idx;
            topk[wave * R + lane] = idx;
        }
    }
    int dep = 0;
    if (copy >= 0 && i < M) {
        __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
        for (int j = i, step = 0; step < M; ++step) {
            const int p = s_parent[copy][j];
            if (p < 0 || p >= j) break;
            j = p;
            ++dep;
        }
    }
    __syncthreads();
    if (i < 0 || i >= M) return;
    int t;
    if (i == 0) {
        t = root;
    } else {
        // clamped: a tree deeper than the heads or a rank past R cannot read outside the table
        int head = dep < 1 ? 0 : (dep > K ? K - 1 : dep - 1);
        int r = my_rank;
        r = r < 0 ? 0 : (r >= R ? R - 1 : r);
        t = s_top[head * R + r];
    }
    tokens[i] = t < 0 ? 0 : (t >= V ? V - 1 : t);
}

ghd_status launch_embed(void* x16, const void* table16, const int32_t* tokens, int M, int H, int V,
                        hipStream_t st)
{
    hipLaunchKernelGGL(k_embed, dim3(M), dim3(256), 0, st, (half8*)x16, (const half8*)table16, tokens,
                       H / 8, V);
    return check_launch();
}

ghd_status launch_pick_norm(const float* x_final, const int32_t* res, int M, int H, const void* g,
                            float eps, void* n16, hipStream_t st)
{
    hipLaunchKernelGGL(k_pick_norm, dim3(1), dim3(kPickThreads), 0, st, x_final, res, M, H,
                       (const half_t*)g, eps, (half_t*)n16);
    return check_launch();
}

size_t topk_list_entries(int K, int V, int R) { return (size_t)K * R * ceil_div(V, kSegLen); }

ghd_status launch_topk_tokens(const float* logits, int K, int V, int R, uint64_t* lists, int32_t* topk,
                              int32_t* tokens, const int32_t* parent, const int32_t* rank, int M,
                              const int32_t* res, hipStream_t st)
{
    static_assert(GHD_MAX_M <= kPickWaves * 64 && GHD_MAX_M % 64 == 0, "a thread per node, in whole wavefronts");
    const int nseg = ceil_div(V, kSegLen);
    if (K > kPickWaves || R > kMaxPicks) return GHD_ERR_SHAPE;
    hipLaunchKernelGGL(k_topk_segment, dim3(K * nseg), dim3(kSegWaves * 64), 0, st, logits, V, R, nseg, lists);
    hipLaunchKernelGGL(k_topk_tokens, dim3(1), dim3(kPickWaves * 64), 0, st, (const uint64_t*)lists, nseg, tokens,
                       parent, rank, M, topk, K, R, res, V);
    return check_launch();
}

// ---- tree design (host) -------------------------------------------------------
// The expected acceptance length of a tree is 1 + the sum over its nodes of the product of
// the accuracies along the node's path (section 3.3.1); since accuracies are at most 1 a
// node never scores above its parent, so taking the best-scoring open candidate M - 1 times
// gives the best tree of M nodes.  Open candidates sit in a heap ordered by (score, lower
// parent, lower rank); a node's R children are opened when it is inserted.
int tree_build_host(const double* acc, int K, int R, int M, int32_t* parent, int32_t* rank,
                    double* expect)
{
    struct Cand {
        double score;
        int parent, rank;
    };
    auto worse = [](const Cand& a, const Cand& b) {
        if (a.score != b.score) return a.score < b.score;
        if (a.parent != b.parent) return a.parent > b.parent;
        return a.rank > b.rank;
    };
    std::priority_queue<Cand, std::vector<Cand>, decltype(worse)> open(worse);
    std::vector<double> score(M);
    std::vector<int> depth(M);
    parent[0] = -1;
    rank[0] = 0;
    score[0] = 1.0;
    depth[0] = 0;
    double e = 1.0;
    int n = 1;
    auto open_children = [&](int u) {
        if (depth[u] >= K) return;
        for (int r = 0; r < R; ++r) open.push({score[u] * acc[(size_t)depth[u] * R + r], u, r});
    };
    open_children(0);
    while (n < M && !open.empty()) {
        Cand c = open.top();
        open.pop();
        parent[n] = c.parent;
        rank[n] = c.rank;
        score[n] = c.score;
        depth[n] = depth[c.parent] + 1;
        e += c.score;
        open_children(n);
        ++n;
    }
    if (expect) *expect = e;
    return n;
}

}  // namespace ghd
