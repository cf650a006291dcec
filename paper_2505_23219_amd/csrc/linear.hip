// Host side of the skinny linear layers (how an operation is cut into work shares, kernel
// selection) and the two packing kernels (weights, activations).
#include "linear_impl.h"
#include "qkv_attn_impl.h"

#include <cstdlib>
#include <mutex>
#include <vector>

namespace ghd {

// ---- per-device facts ------------------------------------------------------------
constexpr int kMaxDevices = 64;
static int g_num_cu[kMaxDevices] = {};

static int current_device()
{
    int dev = -1;
    if (hipGetDevice(&dev) != hipSuccess || dev < 0 || dev >= kMaxDevices) return -1;
    return dev;
}

int fused_grid_size()
{
    const int dev = current_device();
    if (dev < 0) return 0;
    if (g_num_cu[dev] == 0) {
        hipDeviceProp_t prop;
        if (hipGetDeviceProperties(&prop, dev) != hipSuccess) return 0;
        g_num_cu[dev] = prop.multiProcessorCount;
    }
    return g_num_cu[dev];
}

// Workgroups of a launch that wait for each other must all be resident: one per compute
// unit.  The first launch of a kernel on a device raises its dynamic LDS limit and checks
// that a workgroup fits; *grid = compute units.
ghd_status launch_resident_checked(const void* kernel, int threads, size_t lds, int* grid)
{
    static std::mutex mu;
    static std::vector<const void*> checked[kMaxDevices];
    const int dev = current_device();
    const int G = fused_grid_size();
    // the hand-off of partial results is laid out for 8 XCDs of G / 8 compute units
    // and for at most kRangeWgs workgroups (their counters in the sync block)
    if (dev < 0 || G < 16 || G > kRangeWgs || (G % 8) != 0) return hip_fail(hipErrorInvalidDevice);
    if (grid) *grid = G;
    std::lock_guard<std::mutex> lock(mu);
    for (const void* k : checked[dev])
        if (k == kernel) return GHD_OK;
    hipError_t e = hipFuncSetAttribute(kernel, hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds);
    if (e != hipSuccess) return hip_fail(e);
    int per_cu = 0;
    e = hipOccupancyMaxActiveBlocksPerMultiprocessor(&per_cu, kernel, threads, lds);
    if (e != hipSuccess) return hip_fail(e);
    if (per_cu < 1) return hip_fail(hipErrorLaunchOutOfResources);
    checked[dev].push_back(kernel);
    return GHD_OK;
}

// ---- which linear layers are taken ---------------------------------------------------
// Any narrow matrix; a wide one that at most 8 passes over the compute units deal out in whole
// tiles, 8 of them a workgroup at up to 64 rows of x, 4 above (the launch itself would take 8 there
// too).  How a launch is cut is choose_cut's.
bool linear_admitted(int M, int N, int K, int G)
{
    const WLayout lay = w_layout(N, K);
    return lay.rb != 1 || ceil_div(lay.ntiles, 8) <= (M <= 64 ? 8 : 4) * (G / 8) * kMaxPasses;
}

// partial-sum slots of the parts cut: one per workgroup, up to 8 tiles of fragments each
size_t linear_part_floats(int M, int G)
{
    static_assert(parts_max_tiles(1) <= 8, "a slot holds a block's fragments");
    return (size_t)G * 8 * layout_tiles(row_tiles(M)) * 256;
}

// ---- how a launch is cut ----------------------------------------------------------------
// The estimate (microseconds) that chooses among the ways; its terms were fitted to launches
// at 1 to 128 rows of 1280 x 1280 to 5120 x 13824 matrices, which it meets within 5 to 10%:
//   weights: at what HBM streams, or the longest share's at what one compute unit gets;
//   x: comes on top, not beside it - a compute unit's vector memory path keeps some 16 KB on
//   their way, in order, so x from the L2 waits its turn among weights from HBM.  [4096, 11008] at
//   64 rows: 31 us whole-tile (1.4 MB of x per workgroup), 26 in parts of 2 tiles (0.7 MB), 22.6
//   of 4 (0.34 MB), 23.3 of 8;
//   parts: the exchange, its partial sums, and a little for every part;
//   whole tiles of a narrow matrix: that one tile's KiB out of every four that lie together are read, which counts
//   up to 16 rows (and is not asked of calls of their own, which have a launch less in whole tiles); and, at 17 to 32
//   rows, what workgroups with a tile more than others need alone.  us a layer, in whole tiles and in parts: [2560, 6904]
//   at 1 to 16 rows 53.5 to 55.1 and 51.9 to 53.4; [2048, 5504] 45.1 to 46.7 and 44.1 to 45.2; [5120, 5120] at 24
//   to 32 rows 130.0 to 131.6 and 126.3 to 127.3; [4096, 4096] at 1 row 84.2 and 85.2, in whole tiles still.  (At 65 rows
//   and more the same allowance made layers of 8 to 17 heads of 128 4% slower: their gate|up comes out in parts.)
//   Calls of their own at 17 to 32 rows, us in whole tiles and in parts: where both pack x ([5120, 5120] at 24 rows 16.7 and
//   13.8, [9375, 6256] at 26 25.6 and 23.9) as in a step; where whole tiles read x as it lies (up to 97 k-steps), parts are a
//   launch more, and what whole tiles lose grows with the rows that there are: [4539, 2096] at 18 rows 7.5 and 8.9, [4478, 2384]
//   at 19 8.7 and 9.6, [4173, 2616] at 21 9.7 and 9.9, [5454, 3080] at 24 12.0 and 11.1, [4478, 2616] at 29 10.9 and 10.1,
//   [5027, 3080] at 32 13.4 and 10.9; with three tiles a workgroup [8748, 2848] at 17 11.7 and 13.6, [8931, 3080] at 29 16.2
//   and 14.5.  (The estimate is off by up to a tenth: [4313, 2144] at 30 rows, 8.9 and 9.5, comes out in parts.)
// Whole tiles read all of x in every workgroup, so they are for wide matrices, and for narrow
// ones where x is small; parts divide x with the k range; groups of workgroups divide its rows, and exchange
// nothing.  (Layers of 20 heads of 64 at 37 rows 41.6 us without groups, 39.9 with them; 5 heads of 128 at 128 rows
// 44.7 and 40.4; 4 heads of 64 at 128 rows 35.4 and 30.1.)  A call of its own pays one launch
// more for parts (counters have to be zeroed, and x packed); with whole tiles it can read x
// as it lies, which costs about twice the x time (64-byte pieces of 128-byte lines), where
// that is less than the launch.
constexpr double kStreamBytesPerUs = 6.4e6;    // what a launch of 0.1 to 0.2 GB streams from HBM (measured)
constexpr double kCuStreamBytesPerUs = 40e3;
constexpr double kCuReadBytesPerUs = 55e3;
constexpr double kXBytesPerUs = 80e3;
constexpr double kPartsUs = 1.6, kPartsFragmentUs = 0.1, kPartsPartUs = 0.25;
constexpr double kNarrowWholeUs = 1.0, kUnevenStepUs = 0.03;     // (the latter a k-step)
constexpr double kPrepareUs = 2.5;

// How often a cut's sums are rounded, in k-steps of one chain (see folded; an addition counts for a quarter of
// one): a wavefront's chain, cut short where it is long, and the additions of sets and of parts.
static double chain_steps(const WLayout& lay, const LinCut& cut)
{
    const int waves = cut.whole ? waves_of(cut.mt, cut.tiles) : 8;
    const double chain = (double)ceil_div(lay.nks, cut.parts) / waves, more = cut.parts > 1 ? cut.parts / 4.0 : 0.0;
    double cut_short = chain;
    if (cut.groups > 1) cut_short = 1.0 + chain / kSingleSets / 4.0 + 0.5;      // (two additions bring the sets together)
    else if (long_chains(lay, cut, waves))
        cut_short = folded(cut.mt, cut.tiles) ? kFoldSteps + chain / kFoldSteps / 4.0 : chain / 2.0 + 0.25;
    return (cut_short < chain ? cut_short : chain) + more;
}

LinCut choose_cut(int M, int N, int K, int G, bool solo)
{
    const WLayout lay = w_layout(N, K);
    const int mt = row_tiles(M), Gx = G / 8;
    const double hbm = 2.0 * N * K / kStreamBytesPerUs;
    // a share of w tiles and x row tiles over ks k-steps
    auto share_us = [&](double w, double x, double ks) {
        const double wb = w * ks * 1024, xb = x * ks * 1024;
        const double stream = wb / kCuStreamBytesPerUs;
        const double a = (stream > hbm ? stream : hbm) + xb / kXBytesPerUs, b = (wb + xb) / kCuReadBytesPerUs;
        return a > b ? a : b;
    };
    LinCut best = {};
    const int U = ceil_div(lay.ntiles, 8);       // tiles of the fullest XCD
    int P = 1;
    while (U > 8 * Gx * P) ++P;
    best.whole = 1;
    best.tiles = U <= Gx * P ? 1 : ceil_div(U, Gx * P);
    best.parts = 1;
    best.grid = 8 * Gx * P;
    best.mt = mt;
    best.groups = 1;
    // (up to 16 rows only the rows that there are get read)
    const double row_cost = mt == 1 ? M / 8.0 : 2.0;
    best.rows = solo && mt <= kRowsMaxMT && (row_cost - 1.0) * mt * P * lay.nks * 1024.0 / kXBytesPerUs < kPrepareUs;
    const bool uneven = mt == 2 && U > Gx;
    // (of x as it lies, at 17 to 32 rows in uneven shares too, the rows that there are: see above)
    const double x_cost = !best.rows ? 1.0 : uneven ? M / 16.0 : row_cost;
    double best_us = share_us(best.tiles * P, mt * P * x_cost, lay.nks) + (solo && !best.rows ? kPrepareUs : 0.0);
    if (lay.rb == 1) return best;
    if (mt == 1 && U <= Gx && !solo) best_us += kNarrowWholeUs;
    if (uneven) best_us += (best.tiles * P - (double)U / Gx) * lay.nks * kUnevenStepUs;
    for (int r = 1; r <= parts_max_tiles(mt); ++r) {
        const int per_xcd = ceil_div(ceil_div(lay.ntiles, r), 8);
        if (per_xcd > Gx) continue;
        int S = Gx / per_xcd;
        if (S > lay.nks / 8) S = lay.nks / 8;    // a k-step for each wavefront
        if (S < 2) continue;
        const double us = share_us(r, mt, ceil_div(lay.nks, S)) + kPartsUs + kPartsFragmentUs * r * mt + kPartsPartUs * S +
                          (solo ? kPrepareUs : 0.0);
        if (us < best_us) {
            best_us = us;
            best = LinCut{0, r, S, per_xcd * S * 8, 0, mt, 1};
        }
    }
    // Groups of workgroups with some of the rows each (1, 2 or 4 row tiles, of which the packed activation layout
    // holds a whole number), while that leaves a tile at most for each.  Weights are then read once per group,
    // from the L2 but for the first, and x once in all.  Not where that would round sums more often than
    // the cut it stands in for (parts have shorter chains; the count is rough, so more than half a step less is
    // asked for), nor for less than half a microsecond instead of parts ([1280, 3416] at 64 rows: 0.6 us slower).
    const double steps = chain_steps(lay, best) - (best.whole ? 0.0 : 0.6), us_to_beat = best_us - (best.whole ? 0.0 : 0.5);
    for (int m = 1; m < mt && m <= 4; m *= 2) {
        const int groups = ceil_div(ceil_div(M, 16), m), gx = Gx / groups;
        if (groups < 2 || gx < 2 || U > gx) continue;
        for (int rows = 0; rows <= (solo && M <= 64 ? 1 : 0); ++rows) {
            const double us = share_us(1, m * (rows ? 2.0 : 1.0), lay.nks) + (solo && !rows ? kPrepareUs : 0.0);
            const LinCut cut = {1, 1, 1, 8 * gx * groups, rows, m, groups};
            if (us < best_us && us < us_to_beat && chain_steps(lay, cut) <= steps) {
                best_us = us;
                best = cut;
            }
        }
    }
    return best;
}

ghd_status launch_linear(const FusedArgs& a, hipStream_t st)
{
    const int G = fused_grid_size();
    if (G <= 0) return hip_fail(hipErrorInvalidDevice);
    const LinCut cut = choose_cut(a.M, a.lin_N, a.lin_K, G, a.lin_row_major != 0);
    switch (cut.mt) {
    case 1: return launch_linear_mt1(a, cut, st);
    case 2: return launch_linear_mt2(a, cut, st);
    case 3: return launch_linear_mt3(a, cut, st);
    case 4: return launch_linear_mt4(a, cut, st);
    case 6: return launch_linear_mt6(a, cut, st);
    default: return launch_linear_mt8(a, cut, st);
    }
}

// The QKV layer and the attention share a launch when the packed QKV rows are grouped by
// XCD, the matrix is a wide one whose tiles fit one workgroup per compute unit, and a kernel
// was built for the shape.
bool qkv_attn_available(int M, int d, int nh)
{
    if (!qkv_grouped(nh) || d != 128) return false;
    const WLayout lay = w_layout(3 * nh * d, nh * d);
    const int G = fused_grid_size();
    if (lay.rb != 1 || G < 8) return false;
    const int slots = ceil_div(lay.ntiles, G);
    return slots >= 3 && slots <= (row_tiles(M) <= 4 ? 6 : 4);
}

ghd_status launch_qkv_attn(const FusedArgs& a, hipStream_t st)
{
    const int G = fused_grid_size();
    if (G <= 0) return hip_fail(hipErrorInvalidDevice);
    const LinCut cut = choose_cut(a.M, a.lin_N, a.lin_K, G, false);
    switch (row_tiles(a.M)) {
    case 1: return launch_qkv_attn_mt1(a, cut, st);
    case 2: return launch_qkv_attn_mt2(a, cut, st);
    case 3: return launch_qkv_attn_mt3(a, cut, st);
    case 4: return launch_qkv_attn_mt4(a, cut, st);
    case 6: return launch_qkv_attn_mt6(a, cut, st);
    default: return launch_qkv_attn_mt8(a, cut, st);
    }
}

// The kernels' arithmetic evaluated on the host, for tests of its invariants.
// (row tiles of a workgroup, groups of rows) of a cut
void groups_on_host(int M, int N, int K, int G, bool solo, int* out)
{
    const LinCut cut = choose_cut(M, N, K, G, solo);
    out[0] = cut.mt;
    out[1] = cut.groups;
}

int run_on_host(int M, int N, int K, int G, bool solo) { return run_of_launch(choose_cut(M, N, K, G, solo), w_layout(N, K).nks); }

void tile_range_on_host(int ntiles, int gx, int i, int* out)
{
    tile_range(ntiles, gx, (uint32_t)(0x100000000ull / (uint64_t)gx + 1), i, out, out + 1);
}

// One line's counting over the launches of a call, with the very words that the kernels form:
// workgroup i of epoch e runs on XCD xcd[e * n + i]; ok[e] = how many of the n take the exchange
// to be whole and on their own XCD.
void exchange_on_host(const int* xcd, int epochs, int n, int* ok)
{
    uint32_t line[2] = {0, 0};
    for (int e = 0; e < epochs; ++e, xcd += n) {
        uint32_t* const word = epoch_word(&line[0], (uint32_t)e);
        for (int i = 0; i < n; ++i) *word += arrival_of((uint32_t)xcd[i]);
        *epoch_word(&line[0], (uint32_t)e + 1) = 0;
        ok[e] = 0;
        for (int i = 0; i < n; ++i) ok[e] += (*word & 0xffffu) == (uint32_t)n && all_from(*word, (uint32_t)xcd[i], (uint32_t)n);
    }
}

// ---- weight packing ------------------------------------------------------------
// One thread per 16-byte piece of the packed image.  Packed row p of the matrix maps
// to a source row through the permutation of its kind:
//   PLAIN    p
//   QKV      inside every head the rows are ordered (j, j+1, j+d/2, j+1+d/2), j even,
//            so the two rotary pairs of a quad sit in one lane of the GEMM output; heads
//            grouped by XCD when their number is a multiple of 8 (see qkv_row)
//   GATE_UP  (gate f, gate f+1, up f, up f+1): source holds gate rows [0,F) then up rows
__global__ void k_pack2(half8* __restrict__ dst, const half_t* __restrict__ src, int N, int K,
                        int kind, int d, WLayout lay)
{
    size_t id = (size_t)blockIdx.x * blockDim.x + threadIdx.x;
    size_t total = w_pieces(lay);
    if (id >= total) return;
    int lane = (int)(id & 63);
    size_t blk = id >> 6;
    int tin = (int)(blk % lay.blk);
    size_t bk = blk / lay.blk;
    int ks = (int)(bk % lay.nks);
    int block = (int)(bk / lay.nks);
    int p = (block * lay.blk + tin) * 16 + (lane & 15);
    int k = ks * 32 + (lane >> 4) * 8;
    int srow = -1;
    if (kind == PACK_PLAIN) {
        if (p < N) srow = p;
    } else if (kind == PACK_QKV) {
        if (p < N) {
            const int H = N / 3;
            const QkvRow qr = qkv_row(p, H / d, d);
            srow = qr.part * H + qr.head * d + qkv_channel(qr.ph, d);
        }
    } else {
        int F = N / 2;
        int f = (p >> 4) * 8 + ((p & 15) >> 2) * 2 + (p & 1);
        bool up = (p & 3) >= 2;
        if (f < F) srow = (up ? F : 0) + f;
    }
    half8 v;
    for (int e = 0; e < 8; ++e)
        v[e] = (srow >= 0 && k + e < K) ? src[(size_t)srow * K + k + e] : (half_t)0;
    dst[id] = v;
}

size_t packed_bytes2(int N, int K)
{
    return w_pieces(w_layout(N, K)) * 16;
}

ghd_status launch_pack2(void* dst, const void* src, int N, int K, int kind, int d, hipStream_t st)
{
    const WLayout lay = w_layout(N, K);
    size_t total = w_pieces(lay);
    hipLaunchKernelGGL(k_pack2, dim3((unsigned)((total + 255) / 256)), dim3(256), 0, st, (half8*)dst,
                       (const half_t*)src, N, K, kind, d, lay);
    return check_launch();
}

// ---- activation packing -----------------------------------------------------------
// One thread per 16-byte piece of the packed image: row-major [M, ldx] -> B-operand blocks.
// Rows from M on and columns from K on are written as zeros.  With `sync`, the first
// kPackZeroBlocks workgroups zero the sync block (the parts cut counts on it).
constexpr int kPackZeroBlocks = 64;

__global__ __launch_bounds__(256) void k_pack_x(uint32_t* __restrict__ sync, half8* __restrict__ dst,
                                                const half_t* __restrict__ src, int M, int mtp, int K, int64_t ldx)
{
    int block = blockIdx.x;
    if (sync) {
        if (block < kPackZeroBlocks) {
            zero_sync<kPackZeroBlocks>(sync, block);
            return;
        }
        block -= kPackZeroBlocks;
    }
    size_t id = (size_t)block * blockDim.x + threadIdx.x;
    size_t total = (size_t)((K + 31) / 32) * mtp * 64;
    if (id >= total) return;
    int lane = (int)(id & 63);
    size_t blk = id >> 6;
    int b = (int)(blk % mtp);
    int ks = (int)(blk / mtp);
    int m = b * 16 + (lane & 15), k = ks * 32 + (lane >> 4) * 8;
    half8 v = {0, 0, 0, 0, 0, 0, 0, 0};
    if (m < M && k < K) v = *(const half8*)(src + (size_t)m * ldx + k);
    dst[id] = v;
}

ghd_status launch_pack_x(uint32_t* sync, half_t* dst, const half_t* src, int M, int Mpad, int K, int64_t ldx, hipStream_t st)
{
    const int mtp = Mpad / 16;
    size_t total = (size_t)((K + 31) / 32) * mtp * 64;
    hipLaunchKernelGGL(k_pack_x, dim3((unsigned)((total + 255) / 256) + (sync ? kPackZeroBlocks : 0)), dim3(256), 0, st,
                       sync, (half8*)dst, src, M, mtp, K, ldx);
    return check_launch();
}

}  // namespace ghd
