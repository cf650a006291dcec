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

__global__ __launch_bounds__(kPickThreads) void k_pick_norm(const float* __restrict__ x_final,
                                                            const int32_t* __restrict__ res, int M, int H,
                                                            const half_t* __restrict__ g, float eps,
                                                            half_t* __restrict__ n16)
{
    __shared__ float s_part[kPickThreads / 64];
    __shared__ float s_rinv;
    const int tid = threadIdx.x;
    int len = res[0];
    len = len < 1 ? 1 : (len > M ? M : len);
    int last = res[2 + len - 1];
    last = last < 0 ? 0 : (last >= M ? M - 1 : last);
    const float* row = x_final + (size_t)last * H;
    float s = 0.f;
    for (int j = tid; j < H; j += kPickThreads) s += row[j] * row[j];
    for (int off = 32; off > 0; off >>= 1) s += __shfl_xor(s, off);
    if ((tid & 63) == 0) s_part[tid >> 6] = s;
    __syncthreads();
    if (tid == 0) {
        float tot = 0.f;
        for (int w = 0; w < kPickThreads / 64; ++w) tot += s_part[w];
        s_rinv = 1.0f / sqrtf(tot / (float)H + eps);
    }
    __syncthreads();
    const float rinv = s_rinv;
    for (int j = tid; j < H; j += kPickThreads) n16[j] = (half_t)(row[j] * rinv * (float)g[j]);
}

// ---- the R best candidates of every head, then the next tree's tokens ----------------------
// Bound by latency: the K heads' logits are 640 KB at 5 x 32000, far less than a microsecond of
// HBM time, so what counts is how many compute units look at them and how long the chain of R
// dependent picks is.  One workgroup per head with R passes over its whole row took 80 us there.
// Now every head's row is cut into segments of kSegLen entries, one workgroup each: a
// wavefront holds 512 entries in registers, picks its R best in R rounds (a register maximum,
// a DPP maximum over the lanes, no LDS and no barrier), the four wavefronts' lists are merged
// the same way, and one last workgroup merges the segments' lists, a wavefront per head, and
// writes the tokens.  Measured at 5 x 32000, R = 10: 80 + 4.6 us before, 7.5 + 6.1 us now.
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
__device__ __forceinline__ uint64_t max_dpp(uint64_t v)
{
    const int lo = (int)(uint32_t)v, hi = (int)(uint32_t)(v >> 32);
    const uint32_t olo = (uint32_t)__builtin_amdgcn_update_dpp(lo, lo, CTRL, 0xf, 0xf, false);
    const uint32_t ohi = (uint32_t)__builtin_amdgcn_update_dpp(hi, hi, CTRL, 0xf, 0xf, false);
    const uint64_t o = ((uint64_t)ohi << 32) | olo;
    return o > v ? o : v;
}

// maximum over the wavefront, uniform
__device__ __forceinline__ uint64_t wave_max(uint64_t v)
{
    v = max_dpp<0xB1>(v);      // quad_perm 1,0,3,2
    v = max_dpp<0x4E>(v);      // quad_perm 2,3,0,1
    v = max_dpp<0x141>(v);     // row_half_mirror
    v = max_dpp<0x140>(v);     // row_mirror: every lane has its row's maximum
    v = max_dpp<0x142>(v);     // row_bcast15
    v = max_dpp<0x143>(v);     // row_bcast31: lane 63 has the wavefront's
    const uint32_t lo = (uint32_t)__builtin_amdgcn_readlane((int)(uint32_t)v, 63);
    const uint32_t hi = (uint32_t)__builtin_amdgcn_readlane((int)(uint32_t)(v >> 32), 63);
    return ((uint64_t)hi << 32) | lo;
}

// lane r (r < R <= 64) gets the r-th best of the wavefront's keys, 0 when there are fewer
template <int E>
__device__ __forceinline__ uint64_t wave_topk(uint64_t (&key)[E], int R, int lane)
{
    uint64_t mine = 0;
    for (int r = 0; r < R; ++r) {
        uint64_t best = key[0];
#pragma unroll
        for (int e = 1; e < E; ++e) best = key[e] > best ? key[e] : best;
        best = wave_max(best);
        if (best == 0) break;
        if (lane == r) mine = best;
#pragma unroll
        for (int e = 0; e < E; ++e) key[e] = key[e] == best ? 0ull : key[e];
    }
    return mine;
}

// one workgroup per (head, segment): lists[head][segment][R]
__global__ __launch_bounds__(kSegWaves * 64) void k_topk_segment(const float* __restrict__ logits, int V, int R,
                                                                 int nseg, uint64_t* __restrict__ lists)
{
    __shared__ uint64_t s_list[kSegWaves * kMaxPicks];
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
    __syncthreads();
    if (wave) return;
    constexpr int E2 = kSegWaves * kMaxPicks / 64;
    uint64_t k2[E2];
#pragma unroll
    for (int e = 0; e < E2; ++e) k2[e] = lane + e * 64 < kSegWaves * R ? s_list[lane + e * 64] : 0ull;
    const uint64_t best = wave_topk(k2, R, lane);
    if (lane < R) lists[((size_t)head * nseg + seg) * R + lane] = best;
}

constexpr int kPickWaves = 16;                   // K (checked on the host)

// one workgroup: wavefront k merges head k's lists, then a thread per node writes its token
__global__ __launch_bounds__(kPickWaves * 64) void k_topk_tokens(const uint64_t* __restrict__ lists, int nseg,
                                                                 int32_t* __restrict__ tokens,
                                                                 const int32_t* __restrict__ parent,
                                                                 const int32_t* __restrict__ rank, int M,
                                                                 int32_t* __restrict__ topk, int K, int R,
                                                                 const int32_t* __restrict__ res, int V)
{
    __shared__ int32_t s_parent[GHD_MAX_M];
    __shared__ int32_t s_top[kPickWaves * kMaxPicks];
    const int i = threadIdx.x, wave = i >> 6, lane = i & 63;
    int my_rank = 0, root = 0;
    if (i < M) {
        s_parent[i] = parent[i];
        my_rank = rank[i];
        root = res[1];
    }
    if (wave < K) {
        const uint64_t* list = lists + (size_t)wave * nseg * R;
        const int n = nseg * R;
        uint64_t mine = 0;
        for (int c0 = 0; c0 < n; c0 += 64 * kPerLane) {
            uint64_t key[kPerLane + 1];
#pragma unroll
            for (int e = 0; e < kPerLane; ++e) key[e] = list[min(c0 + e * 64 + lane, n - 1)];
#pragma unroll
            for (int e = 0; e < kPerLane; ++e)
                if (c0 + e * 64 + lane >= n) key[e] = 0;
            key[kPerLane] = mine;                // what the entries before these left
            mine = wave_topk(key, R, lane);
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
    __syncthreads();
    if (i >= M) return;
    int t;
    if (i == 0) {
        t = root;
    } else {
        int dep = 0;
        for (int j = i, step = 0; step < M; ++step) {
            int p = s_parent[j];
            if (p < 0 || p >= j) break;
            j = p;
            ++dep;
        }
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
    static_assert(GHD_MAX_M <= kPickWaves * 64, "a thread per node");
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
