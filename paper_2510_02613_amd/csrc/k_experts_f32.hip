// Grouped SwiGLU expert GEMMs of fp32 layers on the fp32 matrix cores.
//
// The same computation as the bf16 kernels (the expert FFN of Sec. 2.1 of the paper over slot-grouped rows; the
// slot comes from the M-tile list or, for few tokens, from the selection kernel's block masks), every product a
// true fp32 product, fp32 accumulation.
//
// What bounds it: a layer of a few megabytes is latency, a chain of memory round trips per launch, so as many of a
// task's loads as possible go out together; large batches are bound by the fp32 matrix rate (k_expert_f32_tile, below, serves
// them).  A task is 16 gate rows and the 16 matching up rows (GEMM-1) or 32 W2 rows (GEMM-2) of one M-tile, one workgroup of
// four wavefronts that each walk a quarter of the contraction; the four sums are added in K order through LDS.  Operands go straight from
// global memory into the layout of v_mfma_f32_16x16x4_f32: lane (n = l % 16, q = l / 16) reads 16 bytes, k = 4q .. 4q+3,
// of row n per 16 k, and the contraction does not care that MFMA i takes element i of every lane as long as weight
// and token rows agree.  A tile has up to 32 token rows, which a weight row read once serves; the next 16 k are
// in flight while 16 are multiplied.
// Measured against 32 x 64 tiles staged through LDS without overlap: 64 tokens of the 128 x 64 layer, GEMM-1 21 -> 5 us.
#include <type_traits>

#include "moe_internal.h"
#include "self_tiles.h"

namespace emoe {
namespace {

typedef float f32x4 __attribute__((ext_vector_type(4)));

constexpr int kSplit = 4;         // wavefronts that share a task's contraction
constexpr int kKC = 16;           // k per chunk: with the 128 bytes of 32 k, a 264-wide contraction left a wavefront without work (264 x 264 layer,
                                  // 1500 tokens, whole pass: 75 -> 70 us)
constexpr int kWRows = 32;        // weight rows per task
constexpr int kGridRow = 1 << 23; // tasks per row of the grid: a launch takes less than 2^32 threads in one dimension

struct Run { f32x4 v[kKC / 16]; };   // a lane's share of one row of a chunk

__device__ __forceinline__ void load_run(Run &r, const float *row, int k0, int q, int K)
{
#pragma unroll
    for (int j = 0; j < kKC / 16; ++j) {
        const int k = k0 + j * 16 + q * 4;
        r.v[j] = k < K ? *(const f32x4 *)(row + k) : (f32x4){0.f, 0.f, 0.f, 0.f};   // K % 8 == 0
    }
}

// The part of a task behind the tile lookup, for a tile with up to NT groups of 16 rows; src: this lane's row of x or h
// per group.
template <bool kFirst, int NT, int TT>
__device__ __forceinline__ void task_body(const Pass &p, const MTile &mt, int n0, const int (&src)[TT], f32x4 *part)
{
    const int K = kFirst ? p.H : p.I, N = kFirst ? p.I : p.H;
    const int lane = threadIdx.x & 63, ks = (int)(threadIdx.x >> 6), n = lane & 15, q = lane >> 4;
    const float *W = (const float *)(kFirst ? p.w13 : p.w2) + (size_t)mt.slot * (kFirst ? 2 : 1) * (size_t)p.I * p.H;
    const float *A = (const float *)(kFirst ? p.x : p.h);
    const int ra = min(n0 + n, N - 1), rb = kFirst ? p.I + ra : min(n0 + 16 + n, N - 1);
    const float *wa = W + (size_t)ra * K, *wb = W + (size_t)rb * K;
    const float *xr[NT];
#pragma unroll
    for (int c = 0; c < NT; ++c) xr[c] = A + (size_t)src[c] * K;
    const int chunks = (K + kKC - 1) / kKC, per = (chunks + kSplit - 1) / kSplit;
    const int kbeg = min(ks * per, chunks) * kKC, kend = min(min((ks + 1) * per, chunks) * kKC, K);
    f32x4 aa[NT], ab[NT];
#pragma unroll
    for (int c = 0; c < NT; ++c) aa[c] = ab[c] = (f32x4){0.f, 0.f, 0.f, 0.f};
    Run ca, cb, na, nb, cx[NT], nx[NT];
    auto load = [&](int k0, Run &a, Run &b, Run (&x)[NT]) {
        load_run(a, wa, k0, q, K);
        load_run(b, wb, k0, q, K);
#pragma unroll
        for (int c = 0; c < NT; ++c) load_run(x[c], xr[c], k0, q, K);
    };
    if (kbeg < kend) load(kbeg, ca, cb, cx);
    for (int k0 = kbeg; k0 < kend; k0 += kKC) {
        if (k0 + kKC < kend) load(k0 + kKC, na, nb, nx);
        __builtin_amdgcn_sched_barrier(0);   // the prefetch goes out before this chunk's MFMAs, not after
#pragma unroll
        for (int j = 0; j < kKC / 16; ++j)
#pragma unroll
            for (int i = 0; i < 4; ++i)
#pragma unroll
                for (int c = 0; c < NT; ++c) {
                    aa[c] = __builtin_amdgcn_mfma_f32_16x16x4f32(ca.v[j][i], cx[c].v[j][i], aa[c], 0, 0, 0);
                    ab[c] = __builtin_amdgcn_mfma_f32_16x16x4f32(cb.v[j][i], cx[c].v[j][i], ab[c], 0, 0, 0);
                }
        ca = na; cb = nb;
#pragma unroll
        for (int c = 0; c < NT; ++c) cx[c] = nx[c];
    }
    // the parts' sums meet in LDS; wavefront c adds those of row group c in K order and stores them
#pragma unroll
    for (int c = 0; c < NT; ++c) {
        part[((ks * NT + c) * 2) * 64 + lane] = aa[c];
        part[((ks * NT + c) * 2 + 1) * 64 + lane] = ab[c];
    }
    __syncthreads();
    const int m = ks * 16 + n;                    // the lane's row of the tile, weight rows 4q .. 4q+3 of both blocks
    if (ks >= NT || m >= mt.rows) return;
    f32x4 sa = part[(ks * 2) * 64 + lane], sb = part[(ks * 2 + 1) * 64 + lane];
#pragma unroll
    for (int s = 1; s < kSplit; ++s) {
        sa += part[((s * NT + ks) * 2) * 64 + lane];
        sb += part[((s * NT + ks) * 2 + 1) * 64 + lane];
    }
    float *O = (float *)(kFirst ? p.h : p.y) + (size_t)(mt.row_begin + m) * N;
    const int c0 = n0 + 4 * q, c1 = n0 + 16 + 4 * q;
    if (kFirst) {
        f32x4 h;
#pragma unroll
        for (int r = 0; r < 4; ++r) h[r] = sa[r] / (1.f + expf(-sa[r])) * sb[r];
        if (c0 < N) *(f32x4 *)(O + c0) = h;
    } else {
        if (c0 < N) *(f32x4 *)(O + c0) = sa;
        if (c1 < N) *(f32x4 *)(O + c1) = sb;
    }
}

// kRows: the grid has several rows of kGridRow tasks.
template <bool kFirst, int TT, bool kSelf, bool kRows>
__global__ __launch_bounds__(64 * kSplit) void k_expert_f32(Pass p)
{
    static_assert(!kSelf || kFirst, "only GEMM-1 derives its tiles itself");
    constexpr int TR = 16 * TT, COLS = kFirst ? kWRows / 2 : kWRows;
    __shared__ f32x4 part[kSplit * TT * 2 * 64];
    static_assert(sizeof part >= kSelfTableBytes, "the table workgroup borrows the partial sums' LDS");
    const int N = kFirst ? p.I : p.H;
    const int groups = (N + COLS - 1) / COLS;               // tasks per M-tile
    const int lane = threadIdx.x & 63, n = lane & 15;
    std::conditional_t<kRows, long long, int> task = blockIdx.x;
    if (kRows) task += (long long)blockIdx.y * kGridRow;
    if (kSelf) {
        if (task == 0) { self_tables(p, TR, part); return; }
        task -= 1;
    }
    const int tile = (int)(task / groups), n0 = (int)(task % groups) * COLS;
    MTile mt;
    int src[TT];                                            // rows past the tile's end re-read its last row; their outputs are dropped
    if (kSelf) {
        unsigned long long tokens;
        int first;
        if (!self_tile(p, lane, tile, TR, &mt, &tokens, &first)) return;
#pragma unroll
        for (int c = 0; c < TT; ++c) src[c] = nth_set_bit(tokens, first + min(c * 16 + n, mt.rows - 1));
    } else {
        if (tile >= *p.n_tiles) return;
        mt = p.tiles[tile];
#pragma unroll
        for (int c = 0; c < TT; ++c) {
            const int r = mt.row_begin + min(c * 16 + n, mt.rows - 1);
            src[c] = kFirst ? p.perm[r] : r;
        }
    }
    if constexpr (TT >= 2) {
        if (mt.rows > 16) { task_body<kFirst, 2>(p, mt, n0, src, part); return; }
    }
    task_body<kFirst, 1>(p, mt, n0, src, part);
}

// Tiles of up to 64 token rows, for slots that expect more than 32: a workgroup multiplies them with 16 gate rows and the 16
// matching up rows (GEMM-1) or 32 W2 rows (GEMM-2), wavefront g the rows [16 g, 16 g + 16).  The matrix pipes bound this size (an MFMA of
// 2048 flops takes 32 cycles), if the operands get there: loaded straight into MFMA layout, as in the kernel above, a load
// touches half a line of 16 rows and every wavefront loads all of the tile's token rows.  Here both operands travel as whole 128-byte
// lines, once per workgroup, into an LDS tile of 32 k (registers in between: a ragged contraction is zero filled there), the
// next tile's loads in flight during this one's MFMAs.  Tasks are small, so that a launch has several per compute unit to deal
// out (64 weight rows: +4 %); two K-steps of loads in flight instead of one changed nothing (+-2 %).  One LDS tile of 12 KB and a second
// barrier a step, not two tiles: seven tasks run beside each other instead of six (72 registers a lane are the limit now; a launch bound of eight spills), and whoever
// waits at a barrier has six others to wait beside (whole pass, us, two tiles -> one: 1500 tokens 57.9 -> 56.2, 400 38.3 -> 37.4, 2500 76.1 -> 75.2, 512 x 256, 1500 tokens 82.4 -> 80.2).
// Not multiplying the half of the last K-step that a ragged contraction leaves empty changed nothing: it is the loads that bound it.
// An XCD takes a contiguous run of tasks (GEMM-2 20.5 -> 18.2 us).
// The contraction is summed in the same four parts as above (a flush every quarter), so both kernels give the same bits.
// Measured (264 x 264 layer, 30 of 40 experts, top-4, us with two events): 1500 tokens GEMM-1 32.8 -> 28.7, GEMM-2 26.7 -> 18.4, whole
// pass 71 -> 59.5; 400 tokens 41.8 -> 38.5, 2500: 93 -> 77; 512 x 256, 1500 tokens 92 -> 82.  That is 85 TFLOP/s in GEMM-2
// at 2500 tokens; the tile's ragged rows and columns cost 20 % more MFMAs than the flops of the layer.
constexpr int kTileRows = 64, kTileK = 32;

template <bool kFirst, bool kRows>
__global__ __launch_bounds__(256) void k_expert_f32_tile(Pass p)
{
    constexpr int COLS = kFirst ? kWRows / 2 : kWRows;
    constexpr int XL = kTileRows * 8 / 256;                   // 16-byte loads of token rows per thread and K-step; one of weight rows
    static_assert(kWRows * 8 == 256, "one 16-byte load of weight rows per thread");
    __shared__ f32x4 xs[kTileRows * 8], ws[kWRows * 8];
    const int K = kFirst ? p.H : p.I, N = kFirst ? p.I : p.H;
    const int groups = (N + COLS - 1) / COLS;
    // workgroups are dealt round-robin to the 8 XCDs: each takes a contiguous run of the tasks, so that a tile's token rows and
    // a slot's weights are fetched into one L2
    using Index = std::conditional_t<kRows, long long, int>;
    Index b = blockIdx.x;
    if (kRows) b += (long long)blockIdx.y * kGridRow;
    const Index tasks = (Index)*p.n_tiles * groups, run = (tasks + 7) / 8, task = (b & 7) * run + (b >> 3);
    if ((b >> 3) >= run || task >= tasks) return;
    const int tile = (int)(task / groups), n0 = (int)(task % groups) * COLS;
    const MTile mt = p.tiles[tile];
    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6), n = lane & 15, q = lane >> 4;
    const float *W = (const float *)(kFirst ? p.w13 : p.w2) + (size_t)mt.slot * (kFirst ? 2 : 1) * (size_t)p.I * p.H;
    const float *A = (const float *)(kFirst ? p.x : p.h);
    // ---- staging: thread -> rows tid / 8 + 32 i, 16-byte chunk tid % 8; rows past the end re-read the last one, their outputs are dropped ----
    const int row = tid >> 3, ch = tid & 7;
    const float *xsrc[XL];
    int xat[XL];
#pragma unroll
    for (int i = 0; i < XL; ++i) {
        const int r = row + 32 * i, m = mt.row_begin + min(r, mt.rows - 1);
        xsrc[i] = A + (size_t)(kFirst ? p.perm[m] : m) * K;
        xat[i] = r * 8 + (ch ^ swz8(r));
    }
    const int wrow = kFirst ? min(n0 + (row & 15), N - 1) + (row < 16 ? 0 : p.I) : min(n0 + row, N - 1);
    const float *wsrc = W + (size_t)wrow * K;
    const int wat = row * 8 + (ch ^ swz8(row));
    f32x4 xr[XL], wr;
    auto load = [&](int k0) {
        const int k = k0 + ch * 4;
        const bool in = k < K;                                        // K % 8 == 0: the 4 elements are all in or all out
#pragma unroll
        for (int i = 0; i < XL; ++i) xr[i] = in ? *(const f32x4 *)(xsrc[i] + k) : (f32x4){0.f, 0.f, 0.f, 0.f};
        wr = in ? *(const f32x4 *)(wsrc + k) : (f32x4){0.f, 0.f, 0.f, 0.f};
    };
    auto store = [&]() {
#pragma unroll
        for (int i = 0; i < XL; ++i) xs[xat[i]] = xr[i];
        ws[wat] = wr;
    };
    // ---- this wavefront's products: a group of 16 rows x both weight blocks ----
    const bool live = wave * 16 < mt.rows;
    f32x4 acc[2], sum[2];
#pragma unroll
    for (int a = 0; a < 2; ++a) acc[a] = sum[a] = (f32x4){0.f, 0.f, 0.f, 0.f};
    const int chunks = (K + kKC - 1) / kKC, per = (chunks + kSplit - 1) / kSplit;
    int left = per;                                                   // chunks of 16 k until the part's end
    auto flush = [&]() {
#pragma unroll
        for (int a = 0; a < 2; ++a) { sum[a] += acc[a]; acc[a] = (f32x4){0.f, 0.f, 0.f, 0.f}; }
    };
    auto multiply = [&]() {
        constexpr int J = kTileK / kKC;
        f32x4 xv[J], wv[J][2];
        const int r = wave * 16 + n;
#pragma unroll
        for (int j = 0; j < J; ++j) {
            xv[j] = xs[r * 8 + ((j * 4 + q) ^ swz8(r))];
#pragma unroll
            for (int a = 0; a < 2; ++a) wv[j][a] = ws[(a * 16 + n) * 8 + ((j * 4 + q) ^ swz8(a * 16 + n))];
        }
#pragma unroll
        for (int j = 0; j < J; ++j) {
#pragma unroll
            for (int i = 0; i < 4; ++i)
#pragma unroll
                for (int a = 0; a < 2; ++a) acc[a] = __builtin_amdgcn_mfma_f32_16x16x4f32(wv[j][a][i], xv[j][i], acc[a], 0, 0, 0);
            if (--left == 0) { flush(); left = per; }                 // past the last chunk: zeros are added
        }
    };
    const int KT = (K + kTileK - 1) / kTileK;
    load(0);
    for (int kt = 0; kt < KT; ++kt) {
        store();
        if (kt + 1 < KT) load((kt + 1) * kTileK);
        __syncthreads();
        if (live) multiply();
        __syncthreads();
    }
    if (!live) return;
    if (left != per) flush();
    // lane holds token n of the group, weight rows 4q .. 4q+3 of both blocks
    const int m = wave * 16 + n, c0 = n0 + 4 * q, c1 = n0 + 16 + 4 * q;
    if (m >= mt.rows) return;
    float *O = (float *)(kFirst ? p.h : p.y) + (size_t)(mt.row_begin + m) * N;
    if (kFirst) {
        f32x4 h;
#pragma unroll
        for (int r = 0; r < 4; ++r) h[r] = sum[0][r] / (1.f + expf(-sum[0][r])) * sum[1][r];
        if (c0 < N) *(f32x4 *)(O + c0) = h;
    } else {
        if (c0 < N) *(f32x4 *)(O + c0) = sum[0];
        if (c1 < N) *(f32x4 *)(O + c1) = sum[1];
    }
}

template <bool kFirst>
void launch_tile(const Pass &p, hipStream_t st)
{
    long long tasks = (long long)p.max_tiles * (kFirst ? (p.I + kWRows / 2 - 1) / (kWRows / 2) : (p.H + kWRows - 1) / kWRows);
    tasks = (tasks + 7) / 8 * 8;
    if (tasks <= kGridRow) hipLaunchKernelGGL((k_expert_f32_tile<kFirst, false>), dim3((unsigned)tasks), dim3(256), 0, st, p);
    else hipLaunchKernelGGL((k_expert_f32_tile<kFirst, true>), dim3(kGridRow, (unsigned)((tasks + kGridRow - 1) / kGridRow)), dim3(256), 0, st, p);
}

template <bool kFirst, int TT, bool kSelf>
void launch_tasks(const Pass &p, long long tasks, hipStream_t st)
{
    const dim3 block(64 * kSplit);
    if (tasks <= kGridRow) hipLaunchKernelGGL((k_expert_f32<kFirst, TT, kSelf, false>), dim3((unsigned)tasks), block, 0, st, p);
    else hipLaunchKernelGGL((k_expert_f32<kFirst, TT, kSelf, true>), dim3(kGridRow, (unsigned)((tasks + kGridRow - 1) / kGridRow)), block, 0, st, p);
}

template <int TT>
void launch_tt(const Pass &p, int which, hipStream_t st)
{
    if (which == 0) {
        const long long tasks = (long long)p.max_tiles * ((p.I + kWRows / 2 - 1) / (kWRows / 2));
        if (p.self_tiles) launch_tasks<true, TT, true>(p, tasks + 1, st);
        else              launch_tasks<true, TT, false>(p, tasks, st);
    } else {
        launch_tasks<false, TT, false>(p, (long long)p.max_tiles * ((p.H + kWRows - 1) / kWRows), st);
    }
}

}  // namespace

// Rows per M-tile: what a slot can expect (its share of the routed assignments), so that a weight row read once
// serves the slot's rows and small groups are not multiplied with padding.  64 rows: k_expert_f32_tile, which reads its tiles
// from the list; up to 64 tokens there may be none (GEMM-1 derives its tiles).
int f32_tile_rows(const Pass &p)
{
    const long long r = ((long long)p.T * p.k + p.E - 1) / p.E;
    return r <= 16 ? 16 : r <= 32 || p.T <= 64 ? 32 : 64;
}

hipError_t launch_experts_f32(const Pass &p, int tile_rows, int which, hipStream_t st)
{
    if (tile_rows == 16)      launch_tt<1>(p, which, st);
    else if (tile_rows == 32) launch_tt<2>(p, which, st);
    else if (which == 0)      launch_tile<true>(p, st);
    else                      launch_tile<false>(p, st);
    return hipGetLastError();
}

}  // namespace emoe
