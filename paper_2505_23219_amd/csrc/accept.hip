// Greedy acceptance: after the verification pass the longest root path that the model
// itself would have produced is kept (Ghidorah, section 2.3).  Two launches:
//   k_row_argmax : every row of the logits is cut into kArgSeg segments; a workgroup
//                  finds the (largest value, lowest index) of one segment with a
//                  wavefront-level reduction;
//   k_accept     : merges the segments into amax[i] (lowest index on ties); a node is
//                  valid iff every edge (p -> c) on its root path has
//                  tokens[c] == amax[p]; the deepest valid node (lowest index on
//                  ties) wins and its root path is written out.
#include "common.h"

#include <mutex>

namespace ghd {

constexpr int kCommitMaxLayers = 48;

__device__ inline void argmax_merge(float& v, int& i, float ov, int oi)
{
    if (ov > v || (ov == v && oi < i)) {
        v = ov;
        i = oi;
    }
}

constexpr int kArgSeg = 8;   // segments per row

__global__ __launch_bounds__(256) void k_row_argmax(const float* __restrict__ logits, int V,
                                                    float* __restrict__ seg_v,
                                                    int32_t* __restrict__ seg_i)
{
    __shared__ float s_v[4];
    __shared__ int s_i[4];
    const int rowi = blockIdx.x / kArgSeg, seg = blockIdx.x % kArgSeg;
    const float* row = logits + (size_t)rowi * V;
    const int lo = (int)((long)V * seg / kArgSeg), hi = (int)((long)V * (seg + 1) / kArgSeg);
    int tid = threadIdx.x;
    float bv = -INFINITY;
    int bi = 0x7fffffff;
    // The entries before the segment's first 16-byte boundary and after its last one by the
    // first threads; between them 16 bytes at a time, four loads in flight (rows of an odd V, or a
    // caller's array, start at any 4 bytes).
    const int head = min((int)(((16 - ((uintptr_t)(row + lo) & 15)) & 15) >> 2), hi - lo);
    const int v0 = lo + head, nv = (hi - v0) >> 2, t0 = v0 + nv * 4;
    float edge = -INFINITY;
    const int at = tid < head ? lo + tid : t0 + tid - head;
    if (at < hi && (tid < head || tid < head + 3)) edge = row[at];
    for (int q = tid; q < nv; q += 1024) {
        floatx4 v[4];
#pragma unroll
        for (int u = 0; u < 4; ++u) v[u] = *(const floatx4*)(row + v0 + 4 * min(q + 256 * u, nv - 1));
#pragma unroll
        for (int u = 0; u < 4; ++u)
            if (q + 256 * u < nv)
#pragma unroll
                for (int e = 0; e < 4; ++e) argmax_merge(bv, bi, v[u][e], v0 + 4 * (q + 256 * u) + e);
    }
    if (at < hi && tid < head + 3) argmax_merge(bv, bi, edge, at);
    for (int off = 32; off > 0; off >>= 1) {
        float ov = __shfl_xor(bv, off);
        int oi = __shfl_xor(bi, off);
        argmax_merge(bv, bi, ov, oi);
    }
    if ((tid & 63) == 0) {
        s_v[tid >> 6] = bv;
        s_i[tid >> 6] = bi;
    }
    __syncthreads();
    if (tid == 0) {
        for (int w = 1; w < 4; ++w) argmax_merge(bv, bi, s_v[w], s_i[w]);
        seg_v[rowi * kArgSeg + seg] = bv;
        seg_i[rowi * kArgSeg + seg] = bi;
    }
}

// Row argmax from the per-tile candidates the LM-head finish leaves: one workgroup per row
// merges `ntiles` (value, column) pairs, lowest column on ties.
__global__ __launch_bounds__(256) void k_amax_merge(const float2* __restrict__ tbl, int ntiles, int Mpad,
                                                    int32_t* __restrict__ amax)
{
    __shared__ float s_v[4];
    __shared__ int s_i[4];
    const int row = blockIdx.x, tid = threadIdx.x;
    float bv = -INFINITY;
    int bi = 0x7fffffff;
    for (int t0 = tid; t0 < ntiles; t0 += 1024) {
        float2 c[4];
#pragma unroll
        for (int u = 0; u < 4; ++u) c[u] = tbl[(size_t)min(t0 + 256 * u, ntiles - 1) * Mpad + row];
#pragma unroll
        for (int u = 0; u < 4; ++u)
            if (t0 + 256 * u < ntiles) argmax_merge(bv, bi, c[u].x, __float_as_int(c[u].y));
    }
    for (int off = 32; off > 0; off >>= 1) {
        float ov = __shfl_xor(bv, off);
        int oi = __shfl_xor(bi, off);
        argmax_merge(bv, bi, ov, oi);
    }
    if ((tid & 63) == 0) {
        s_v[tid >> 6] = bv;
        s_i[tid >> 6] = bi;
    }
    __syncthreads();
    if (tid == 0) {
        for (int w = 1; w < 4; ++w) argmax_merge(bv, bi, s_v[w], s_i[w]);
        amax[row] = bi;
    }
}

// amax_in != nullptr: the row argmaxes are given (seg_v, seg_i unused)
__global__ __launch_bounds__(128) void k_accept(const float* __restrict__ seg_v,
                                                const int32_t* __restrict__ seg_i,
                                                const int32_t* __restrict__ amax_in,
                                                const int32_t* __restrict__ tokens,
                                                const int32_t* __restrict__ parent, int M,
                                                int32_t* __restrict__ res,
                                                int32_t* __restrict__ amax_out)
{
    __shared__ int32_t s_amax[GHD_MAX_M], s_up[GHD_MAX_M], s_depth[GHD_MAX_M];
    __shared__ uint64_t s_lo[GHD_MAX_M], s_hi[GHD_MAX_M];
    __shared__ int s_key[2];
    const int i = threadIdx.x;
    int par = -1, tok = 0, bi = 0x7fffffff;
    if (i < M) {
        par = parent[i];
        tok = tokens[i];
        if (amax_in) bi = amax_in[i];
        else {
            float bv = -INFINITY;
            float sv[kArgSeg];
            int si[kArgSeg];
#pragma unroll
            for (int sg = 0; sg < kArgSeg; ++sg) {
                sv[sg] = seg_v[i * kArgSeg + sg];
                si[sg] = seg_i[i * kArgSeg + sg];
            }
#pragma unroll
            for (int sg = 0; sg < kArgSeg; ++sg) argmax_merge(bv, bi, sv[sg], si[sg]);
        }
        s_amax[i] = bi;
        if (amax_out) amax_out[i] = bi;
    }
    __syncthreads();
    // Root paths by pointer doubling: after a round a node knows, of twice as many edges up as
    // before, whether all of them are valid, how many there are, which nodes they pass, and
    // the node above them.  As many rounds as the deepest node needs; a parent that is not an
    // earlier node is taken as "no parent".
    int up = -1, depth = 0;
    bool ok = true;
    uint64_t lo = 0, hi = 0;
    if (i < M) {
        if (par >= 0 && par < i) {
            up = par;
            depth = 1;
            ok = tok == s_amax[par];
        }
        if (i < 64) lo = 1ull << i;
        else hi = 1ull << (i - 64);
    }
    while (__syncthreads_or(up >= 0)) {
        s_up[i] = up;
        s_depth[i] = ok ? depth : -1 - depth;
        s_lo[i] = lo;
        s_hi[i] = hi;
        __syncthreads();
        if (up >= 0) {
            const int d = s_depth[up], a = up;
            ok = ok && d >= 0;
            depth += d >= 0 ? d : -1 - d;
            lo |= s_lo[a];
            hi |= s_hi[a];
            up = s_up[a];
        }
    }
    // key orders candidates by depth first, then by lower node index
    int key = i < M && ok ? depth * 256 + (255 - i) : -1;
    for (int off = 32; off > 0; off >>= 1) key = max(key, __shfl_xor(key, off));
    if ((i & 63) == 0) s_key[i >> 6] = key;
    s_depth[i] = depth;
    s_lo[i] = lo;
    s_hi[i] = hi;
    __syncthreads();
    const int best = max(s_key[0], s_key[1]), node = 255 - (best & 255);
    if (i == 0) {
        res[0] = (best >> 8) + 1;
        res[1] = s_amax[node];
    }
    if (i < M && (((i < 64 ? s_lo[node] >> i : s_hi[node] >> (i - 64)) & 1ull) != 0)) res[2 + depth] = i;
}

// ---- commit of the accepted path ---------------------------------------------
// One workgroup per (layer, head).  The K rows (and the V columns: V is channel-major) of
// the accepted nodes are read, and only after a barrier written to rows kv_len + j, so no
// source can have been overwritten before it is read.  Rows that are where they belong are left
// alone: the root always is, and with it as much of the path as follows the node order.  What
// has to move usually fits the registers, K and V at once; longer paths go through LDS.  The path
// comes from the device result of the acceptance kernel; its entries are clamped, so that
// whatever that buffer holds no access leaves the tree rows.
// Bound by the lines it touches: V is channel-major, so a row that moves costs a 128-byte line of
// every channel, 17 MB read and as much written back for 32 layers x 32 heads x 128 channels (6.5 us at
// a copy's rate).  8.5 us there in four dependent steps with K and V one after the other, 7.3 us now.
struct CommitArgs {
    half_t* k[kCommitMaxLayers];
    half_t* v[kCommitMaxLayers];
    const int32_t* res;
    int nh, d, cap, kv_len, M;
};

__global__ __launch_bounds__(256) void k_commit_path(const CommitArgs a)
{
    __shared__ __attribute__((aligned(16))) half_t s_rows[GHD_MAX_M * 128];
    __shared__ int32_t s_path[GHD_MAX_M];
    __shared__ int s_moved;
    const int tid = threadIdx.x, layer = blockIdx.x / a.nh, head = blockIdx.x % a.nh;
    const int d = a.d, len = min(max(a.res[0], 0), a.M);
    if (tid == 0) s_moved = a.M;
    // (the path's entries only: a result that ends with them is as good as one of 2 + M words)
    int at = 0;
    if (tid < len) at = min(max(a.res[2 + tid], 0), a.M - 1);
    __syncthreads();
    if (tid < len) {
        s_path[tid] = at;
        if (at != tid) atomicMin(&s_moved, tid);
    }
    __syncthreads();
    const int j0 = s_moved, n = len - j0;                          // rows j0 .. len - 1 move
    if (n <= 0) return;
    const int32_t* path = s_path + j0;
    half_t* kh = a.k[layer] + (size_t)head * a.cap * d + (size_t)a.kv_len * d;
    half_t* vh = a.v[layer] + (size_t)head * d * a.cap + a.kv_len;
    const int cpr = d / 8;
    constexpr int kMove = 16;                                      // rows that fit the registers
    if (n <= kMove) {
        constexpr int NK = kMove * 16 / 256, NV = kMove * 128 / 256;
        half8 kr[NK];
        half_t vr[NV];
#pragma unroll
        for (int i = 0; i < NK; ++i) {
            const int idx = tid + 256 * i;
            if (idx < n * cpr) kr[i] = *(const half8*)(kh + (size_t)path[idx / cpr] * d + idx % cpr * 8);
        }
#pragma unroll
        for (int i = 0; i < NV; ++i) {
            const int idx = tid + 256 * i;
            if (idx < d * n) vr[i] = vh[(size_t)(idx / n) * a.cap + path[idx % n]];
        }
        __syncthreads();
#pragma unroll
        for (int i = 0; i < NK; ++i) {
            const int idx = tid + 256 * i;
            if (idx < n * cpr) *(half8*)(kh + (size_t)(j0 + idx / cpr) * d + idx % cpr * 8) = kr[i];
        }
#pragma unroll
        for (int i = 0; i < NV; ++i) {
            const int idx = tid + 256 * i;
            if (idx < d * n) vh[(size_t)(idx / n) * a.cap + j0 + idx % n] = vr[i];
        }
        return;
    }
    for (int idx = tid; idx < n * cpr; idx += 256) {
        int j = idx / cpr, c = idx % cpr;
        *(half8*)(s_rows + idx * 8) = *(const half8*)(kh + (size_t)path[j] * d + c * 8);
    }
    __syncthreads();
    for (int idx = tid; idx < n * cpr; idx += 256) {
        int j = idx / cpr, c = idx % cpr;
        *(half8*)(kh + (size_t)(j0 + j) * d + c * 8) = *(const half8*)(s_rows + idx * 8);
    }
    __syncthreads();
    for (int idx = tid; idx < d * n; idx += 256) {
        int ch = idx / n, j = idx % n;
        s_rows[idx] = vh[(size_t)ch * a.cap + path[j]];
    }
    __syncthreads();
    for (int idx = tid; idx < d * n; idx += 256) {
        int ch = idx / n, j = idx % n;
        vh[(size_t)ch * a.cap + j0 + j] = s_rows[idx];
    }
}

ghd_status launch_commit_path(void* const* k, void* const* v, int L, int nh, int d, int cap,
                              int kv_len, int M, const int32_t* res, hipStream_t st)
{
    CommitArgs a;
    for (int l = 0; l < L; ++l) {
        a.k[l] = (half_t*)k[l];
        a.v[l] = (half_t*)v[l];
    }
    a.res = res;
    a.nh = nh;
    a.d = d;
    a.cap = cap;
    a.kv_len = kv_len;
    a.M = M;
    hipLaunchKernelGGL(k_commit_path, dim3(L * nh), dim3(256), 0, st, a);
    return check_launch();
}

size_t accept_workspace_bytes() { return (size_t)GHD_MAX_M * kArgSeg * 8; }

// ---- acceptance without a caller's workspace ------------------------------------
// The per-segment maxima of ghd_accept_greedy_static live in this array instead of a
// workspace: GHD_MAX_M rows x kArgSeg segments x (value, index) = 8 KiB, one copy per GPU
// the library runs on, held until the process ends.  The name is a host-side stand-in; the
// device address is looked up once per device and only that pointer is handed to kernels.
constexpr size_t kStaticScratchBytes = (size_t)GHD_MAX_M * kArgSeg * 8;
static __device__ __align__(256) unsigned char scratch[kStaticScratchBytes];

constexpr int kScratchDevices = 64;
static void* g_scratch_ptr[kScratchDevices] = {};
static std::mutex g_scratch_mu;

// device address of `scratch` on the current device (looked up on first use)
static ghd_status static_scratch(void** out)
{
    int dev = -1;
    hipError_t e = hipGetDevice(&dev);
    if (e != hipSuccess) return hip_fail(e);
    if (dev < 0 || dev >= kScratchDevices) return hip_fail(hipErrorInvalidDevice);
    std::lock_guard<std::mutex> lock(g_scratch_mu);
    if (!g_scratch_ptr[dev]) {
        void* p = nullptr;
        e = hipGetSymbolAddress(&p, HIP_SYMBOL(scratch));
        if (e != hipSuccess) return hip_fail(e);
        if (!p) return hip_fail(hipErrorInvalidSymbol);
        g_scratch_ptr[dev] = p;
    }
    *out = g_scratch_ptr[dev];
    return GHD_OK;
}

ghd_status launch_accept_static(const float* logits, const int32_t* tokens, const int32_t* parent, int M,
                                int V, int32_t* res, int32_t* amax_out, hipStream_t st)
{
    if ((size_t)M * kArgSeg * 8 > kStaticScratchBytes) return GHD_ERR_SHAPE;
    void* ws = nullptr;
    ghd_status s = static_scratch(&ws);
    if (s) return s;
    // every entry the second kernel reads (rows < M) is written by the first: nothing to clear
    return launch_accept(logits, tokens, parent, M, V, res, amax_out, ws, st);
}

ghd_status launch_accept(const float* logits, const int32_t* tokens, const int32_t* parent, int M,
                         int V, int32_t* res, int32_t* amax_out, void* ws, hipStream_t st)
{
    // workspace: per-segment maxima [GHD_MAX_M][kArgSeg] float, then their indices
    float* seg_v = (float*)ws;
    int32_t* seg_i = (int32_t*)(seg_v + GHD_MAX_M * kArgSeg);
    hipLaunchKernelGGL(k_row_argmax, dim3(M * kArgSeg), dim3(256), 0, st, logits, V, seg_v, seg_i);
    hipLaunchKernelGGL(k_accept, dim3(1), dim3(128), 0, st, (const float*)seg_v,
                       (const int32_t*)seg_i, (const int32_t*)nullptr, tokens, parent, M, res, amax_out);
    return check_launch();
}

ghd_status launch_amax_merge(const void* tbl, int ntiles, int Mpad, int M, int32_t* amax, hipStream_t st)
{
    hipLaunchKernelGGL(k_amax_merge, dim3(M), dim3(256), 0, st, (const float2*)tbl, ntiles, Mpad, amax);
    return check_launch();
}

ghd_status launch_accept_path(const int32_t* amax, const int32_t* tokens, const int32_t* parent, int M,
                              int32_t* res, hipStream_t st)
{
    hipLaunchKernelGGL(k_accept, dim3(1), dim3(128), 0, st, (const float*)nullptr, (const int32_t*)nullptr,
                       amax, tokens, parent, M, res, (int32_t*)nullptr);
    return check_launch();
}

}  // namespace ghd
