// Gating: logits, scores, (group limited) top-k, renormalised weights.
//
// The paper (Sec. 2.1) only says that a gating function picks a few experts per
// token; the rules implemented here are the two its evaluated model families use:
// softmax over all experts then top-k, and sigmoid scores with group-limited
// top-k (group score = sum of the group's two best), both with optional
// renormalisation over the k selected and a constant scale.
//
// Two kernels: logits (matrix cores, fp32 accumulation), then selection, one 64-lane wavefront per token (gate_select.h; small
// routers: one kernel for both; a token to four: GEMM-1 selects): scores live in registers up to 512 experts and in LDS above,
// every arg-max is a wavefront reduction in which ties go to the lower index exactly as the ordering rule demands.
#include <type_traits>

#include "gate_select.h"
#include "gate_small.h"
#include "moe_internal.h"
#include "wave_ops.h"

namespace emoe {

namespace {

constexpr int kThreads = 256;  // 4 wavefronts

// ---------------------------------------------------------------------------------
// k_gate_logits.  A workgroup owns 16 tokens x 16 experts (its logits go to the workspace in fp32).  Both MFMA
// operands are read straight from global memory in operand layout (no LDS): for a K-chunk of 128, lane (n = l%16,
// q = l/16) reads 32 of the 128 k of row n, interleaved with the other three lanes of the row in units of 8, and
// feeds them to the matrix core 8 (bf16) or 1 (fp32) at a time.  The contraction does not care which k a lane group
// carries as long as the router row and the token row use the same assignment, which they do.
//   bf16 x bf16:      v_mfma_f32_16x16x32_bf16, fp32 accumulate.
//   otherwise:        bf16 operands widened to fp32 (exact), v_mfma_f32_16x16x4_f32: every product is a true fp32
//                     product.
// The next chunk's loads are issued before the current chunk's MFMAs.  The contraction is shared out over the
// workgroup's 4 wavefronts (partial sums meet in LDS, added in wavefront order) and, for few tokens, over gridDim.z
// workgroups (partial-sum planes): the router matrix must be streamed by many workgroups at once.
// fp32 layers run it at every batch size (64 tokens of a 128-wide layer: 14 us in a kernel that staged both operands
// through LDS -> 4 us; 1500 tokens of a 264-wide layer with 40 experts: 32 -> 7 us).
//
// k_gate_select.  One wavefront per token: scores, group limiting, top-k, weights
// (select_token in gate_select.h).  Its reductions are latency chains, so it runs as many small
// workgroups as possible and lets occupancy hide them.
template <typename WT> struct RouterRun;           // the lane's 32 k of one row
template <> struct RouterRun<uint16_t> { uint4 v[4]; };
template <> struct RouterRun<float> { uint4 v[8]; };

// Loads the lane's 32 elements of a 128-wide K chunk.  Element (jj, i) of the lane in k-group q
// is k0 + jj*32 + q*8 + i (jj < 4, i < 8): the four lanes of a row then read one contiguous
// 64-byte (bf16) or 128-byte (fp32) span per pair of load instructions.
template <typename WT>
__device__ __forceinline__ void load_run(RouterRun<WT> &r, const WT *row, int k0, int q, int kend)
{
    constexpr int per16 = 16 / sizeof(WT);  // elements per 16-byte load: 8 or 4
    constexpr int parts = 8 / per16;         // loads per 8 elements: 1 or 2
#pragma unroll
    for (int jj = 0; jj < 4; ++jj) {
        const int k = k0 + jj * 32 + q * 8;
        const bool ok = k < kend;  // kend % 8 == 0: the 8 elements are all in or all out
#pragma unroll
        for (int h = 0; h < parts; ++h)
            r.v[jj * parts + h] = ok ? *(const uint4 *)(row + k + h * per16) : make_uint4(0, 0, 0, 0);
    }
}

__device__ __forceinline__ void widen(const RouterRun<uint16_t> &r, float (&f)[32])
{
#pragma unroll
    for (int j = 0; j < 4; ++j) {
        const uint32_t *u = (const uint32_t *)&r.v[j];
#pragma unroll
        for (int e = 0; e < 4; ++e) {
            f[j * 8 + 2 * e] = __uint_as_float(u[e] << 16);
            f[j * 8 + 2 * e + 1] = __uint_as_float(u[e] & 0xffff0000u);
        }
    }
}
__device__ __forceinline__ void widen(const RouterRun<float> &r, float (&f)[32])
{
#pragma unroll
    for (int e = 0; e < 32; ++e) f[e] = ((const float *)&r.v[0])[e];
}

template <typename XT, typename WT>
__global__ __launch_bounds__(kThreads) void k_gate_logits(Pass p)
{
    constexpr bool kBf16 = sizeof(XT) == 2 && sizeof(WT) == 2;
    __shared__ float part[4 * 256];
    const int E = p.E, H = p.H;
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int n = lane & 15, q = lane >> 4;
    const int t0 = blockIdx.x * 16, e0 = blockIdx.y * 16;
    // K range of this wavefront (whole chunks of 128): workgroup z of gridDim.z takes an equal share of the chunks
    // (its sums go to plane z of the logits buffer), its wavefronts a quarter of that each
    const int chunks = (H + 127) / 128;
    const int c0 = (int)((long long)blockIdx.z * chunks / gridDim.z), c1 = (int)((long long)(blockIdx.z + 1) * chunks / gridDim.z);
    const int per = (c1 - c0 + 3) / 4;
    const int kbeg = min(H, min(c1, c0 + wave * per) * 128), kend = min(H, min(c1, c0 + (wave + 1) * per) * 128);

    const XT *xrow = (const XT *)p.x + (size_t)min(t0 + n, p.T - 1) * H;
    const WT *wrow = (const WT *)p.router_w + (size_t)min(e0 + n, E - 1) * H;
    f32x4 acc = {0.f, 0.f, 0.f, 0.f};
    RouterRun<XT> xc, xn;
    RouterRun<WT> wc, wn;
    if (kbeg < kend) {
        load_run<XT>(xc, xrow, kbeg, q, kend);
        load_run<WT>(wc, wrow, kbeg, q, kend);
    }
    for (int k0 = kbeg; k0 < kend; k0 += 128) {
        if (k0 + 128 < kend) {
            load_run<XT>(xn, xrow, k0 + 128, q, kend);
            load_run<WT>(wn, wrow, k0 + 128, q, kend);
        }
        __builtin_amdgcn_sched_barrier(0);  // the prefetch must be issued before this chunk's MFMAs, not after
        if constexpr (kBf16) {
#pragma unroll
            for (int j = 0; j < 4; ++j) acc = __builtin_amdgcn_mfma_f32_16x16x32_bf16(*(bf16x8 *)&wc.v[j], *(bf16x8 *)&xc.v[j], acc, 0, 0, 0);
        } else {
            float xf[32], wf[32];
            widen(xc, xf);
            widen(wc, wf);
#pragma unroll
            for (int e = 0; e < 32; ++e) acc = __builtin_amdgcn_mfma_f32_16x16x4f32(wf[e], xf[e], acc, 0, 0, 0);
        }
        xc = xn;
        wc = wn;
    }
#pragma unroll
    for (int r = 0; r < 4; ++r) part[wave * 256 + r * 64 + lane] = acc[r];
    __syncthreads();
    if (wave != 0) return;
    // lane holds token n, experts 4q + r
    float *plane = p.logits + (size_t)blockIdx.z * p.T * E;
    const float *bias = blockIdx.z == 0 ? p.logit_bias : nullptr;   // added once
    const int t = t0 + n, e = e0 + 4 * q;   // E may be any size: guard each of the 4
    if (t >= p.T) return;
#pragma unroll
    for (int r = 0; r < 4; ++r) {
        float s = 0.f;
#pragma unroll
        for (int w = 0; w < 4; ++w) s += part[w * 256 + r * 64 + lane];
        if (e + r < E) plane[(size_t)t * E + e + r] = s + (bias ? bias[e + r] : 0.f);
    }
}

// LDS-tiled logits kernel for prefill-sized batches.  A workgroup owns 16*TBT tokens x 64*EBT
// experts; the token tile and the router tile of a K-step of 64 are staged once in LDS (global ->
// registers -> LDS, next step's loads in flight during this step's MFMAs) and shared by the four
// wavefronts, wavefront w taking expert tiles w*EBT .. of 16 experts each.  Tile rows are 128
// bytes with their 16-byte chunks XOR-swizzled so that the 16 rows a half-wavefront reads for one
// operand fall into 16 distinct bank groups.
// fp32 router weights are split on the fly into three bf16 planes hi + mid + lo (each the
// truncated top 8 mantissa bits of what is left: the split is exact), so that x . w is three bf16
// MFMAs whose products are all exact and whose sum is accumulated in fp32: the same products and
// the same accumulator width as an fp32 multiply-add chain.
__device__ __forceinline__ int gate_swz(int row) { return ((row >> 1) & 3) | (((row ^ (row >> 3)) & 1) << 2); }

template <typename WT, int TBT, int EBT>
__global__ __launch_bounds__(kThreads) void k_gate_logits_lds(Pass p)
{
    constexpr int P = sizeof(WT) == 2 ? 1 : 3;          // bf16 planes per router tile
    constexpr int TB = 16 * TBT, EB = 64 * EBT;
    constexpr int XCH = TB * 8, WCH = EB * 8;           // 16-byte chunks per tile (per plane)
    constexpr int XL = (XCH + kThreads - 1) / kThreads; // staging loads per thread
    constexpr int WL = WCH / kThreads * (P == 3 ? 2 : 1);   // fp32: 8 floats = 2 loads per 8-element chunk
    constexpr int WCL = WCH / kThreads;                 // 8-element chunks per thread
    __shared__ uint4 lds[2][XCH + P * WCH];
    const int E = p.E, H = p.H;
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int t0 = blockIdx.x * TB, e0 = blockIdx.y * EB;
    const uint16_t *x = (const uint16_t *)p.x;
    const WT *wr = (const WT *)p.router_w;

    uint4 xa[XL], wa[WL], xb[XL], wb[WL];   // two register stages: K-steps kt+1 and kt+2 are in flight
    auto load_global = [&](int k0, uint4 *xreg, uint4 *wreg) {
#pragma unroll
        for (int i = 0; i < XL; ++i) {
            const int c = tid + i * kThreads, row = c >> 3, ch = c & 7;
            const int k = k0 + ch * 8;
            xreg[i] = (c < XCH && k < H) ? *(const uint4 *)(x + (size_t)min(t0 + row, p.T - 1) * H + k) : make_uint4(0, 0, 0, 0);
        }
#pragma unroll
        for (int i = 0; i < WCL; ++i) {
            const int c = tid + i * kThreads, row = c >> 3, ch = c & 7;
            const int k = k0 + ch * 8;
            const WT *src = wr + (size_t)min(e0 + row, E - 1) * H + k;
            if constexpr (P == 1) {
                wreg[i] = (k < H) ? *(const uint4 *)src : make_uint4(0, 0, 0, 0);
            } else {
                wreg[2 * i] = (k < H) ? *(const uint4 *)src : make_uint4(0, 0, 0, 0);
                wreg[2 * i + 1] = (k < H) ? *(const uint4 *)(src + 4) : make_uint4(0, 0, 0, 0);
            }
        }
    };
    auto store_lds = [&](int buf, const uint4 *xreg, const uint4 *wreg) {
#pragma unroll
        for (int i = 0; i < XL; ++i) {
            const int c = tid + i * kThreads, row = c >> 3, ch = c & 7;
            if (c < XCH) lds[buf][row * 8 + (ch ^ gate_swz(row))] = xreg[i];
        }
#pragma unroll
        for (int i = 0; i < WCL; ++i) {
            const int c = tid + i * kThreads, row = c >> 3, ch = c & 7;
            const int at = XCH + row * 8 + (ch ^ gate_swz(row));
            if constexpr (P == 1) {
                lds[buf][at] = wreg[i];
            } else {
                const uint32_t *f = (const uint32_t *)&wreg[2 * i];   // 8 fp32 bit patterns
                uint32_t hi[8], mid[8], lo[8];
#pragma unroll
                for (int e = 0; e < 8; ++e) {
                    hi[e] = f[e] & 0xffff0000u;
                    const float r1 = __uint_as_float(f[e]) - __uint_as_float(hi[e]);
                    mid[e] = __float_as_uint(r1) & 0xffff0000u;
                    const float r2 = r1 - __uint_as_float(mid[e]);
                    lo[e] = __float_as_uint(r2);   // at most 8 significant bits left: already a bf16 value
                }
                auto pack = [](const uint32_t *v) {
                    return make_uint4((v[0] >> 16) | v[1], (v[2] >> 16) | v[3], (v[4] >> 16) | v[5], (v[6] >> 16) | v[7]);
                };
                uint32_t lom[8];
#pragma unroll
                for (int e = 0; e < 8; ++e) lom[e] = lo[e] & 0xffff0000u;
                lds[buf][at] = pack(hi);
                lds[buf][at + WCH] = pack(mid);
                lds[buf][at + 2 * WCH] = pack(lom);
            }
        }
    };

    f32x4 acc[EBT][TBT];
#pragma unroll
    for (int a = 0; a < EBT; ++a)
#pragma unroll
        for (int tb = 0; tb < TBT; ++tb) acc[a][tb] = (f32x4){0.f, 0.f, 0.f, 0.f};
    const int n = lane & 15, q = lane >> 4;

    auto multiply = [&](int buf) {
#pragma unroll
        for (int ks = 0; ks < 2; ++ks) {
            const int ch = ks * 4 + q;
            bf16x8 xf[TBT];
#pragma unroll
            for (int tb = 0; tb < TBT; ++tb) {
                const int row = tb * 16 + n;
                const uint4 v = lds[buf][row * 8 + (ch ^ gate_swz(row))];
                xf[tb] = *(const bf16x8 *)&v;
            }
#pragma unroll
            for (int a = 0; a < EBT; ++a) {
                const int row = (wave * EBT + a) * 16 + n;
#pragma unroll
                for (int pl = 0; pl < P; ++pl) {
                    const uint4 v = lds[buf][XCH + pl * WCH + row * 8 + (ch ^ gate_swz(row))];
                    const bf16x8 wf = *(const bf16x8 *)&v;
#pragma unroll
                    for (int tb = 0; tb < TBT; ++tb)
                        acc[a][tb] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(wf, xf[tb], acc[a][tb], 0, 0, 0);
                }
            }
        }
    };
    // Loads past the end of K are predicated off (they return zeros), so the pipeline needs no tail code.
    const int KT = (H + 63) / 64;
    load_global(0, xa, wa);
    load_global(64, xb, wb);
    store_lds(0, xa, wa);
    load_global(128, xa, wa);
    __syncthreads();
    for (int kt = 0; kt < KT; kt += 2) {
        multiply(0);                          // K-step kt
        store_lds(1, xb, wb);                 // K-step kt+1 (loaded one whole iteration ago)
        load_global((kt + 3) * 64, xb, wb);
        __syncthreads();
        if (kt + 1 < KT) multiply(1);         // K-step kt+1
        store_lds(0, xa, wa);                 // K-step kt+2
        load_global((kt + 4) * 64, xa, wa);
        __syncthreads();
    }
    // lane holds token n of each token tile, experts 4q + r of each of its expert tiles
#pragma unroll
    for (int a = 0; a < EBT; ++a)
#pragma unroll
        for (int tb = 0; tb < TBT; ++tb) {
            const int t = t0 + tb * 16 + n;
            const int e = e0 + (wave * EBT + a) * 16 + 4 * q;
            if (t < p.T) {
#pragma unroll
                for (int r = 0; r < 4; ++r)
                    if (e + r < E) p.logits[(size_t)t * E + e + r] = acc[a][tb][r] + (p.logit_bias ? p.logit_bias[e + r] : 0.f);
            }
        }
}

template <typename WT, int TBT, int EBT>
hipError_t launch_gate_logits_lds(const Pass &p, hipStream_t st)
{
    dim3 grid((p.T + 16 * TBT - 1) / (16 * TBT), (p.E + 64 * EBT - 1) / (64 * EBT));
    hipLaunchKernelGGL((k_gate_logits_lds<WT, TBT, EBT>), grid, dim3(kThreads), 0, st, p);
    return hipGetLastError();
}

__global__ __launch_bounds__(kThreads) void k_gate_select(Pass p)
{
    extern __shared__ float smem[];
    const int stride = select_stride(p.E);
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const int t = blockIdx.x * 4 + wave;
    if (t >= p.T) return;
    float *lg = smem + wave * 2 * stride;
    select_one<4>(p, t, lg, lg + stride, lane, [] {});
}

// The selection kernel with the first step of the routing bookkeeping fused in: a workgroup of 16
// wavefronts owns kFusedTokens = 16 consecutive tokens, one per wavefront.  After the selection every
// lane j < k + n_shared holds one assignment of its token; its slot is looked up in the expert table and
// the workgroup builds, per slot, the 16-bit mask of its tokens that have a row in the slot (a token's
// assignments go to distinct slots: distinct experts, one-to-one table), from which an assignment's rank
// among the block's earlier rows of the slot is a population count -- deterministic, token order.
// Word [slot][block] of blk_hist: the mask, and above it (bits 16..21) the selection position of the
// block's first row in the slot (with the token it makes the group's first-assignment key); byte
// [slot][block] of blk_cnt: the number of rows, i.e. of mask bits.
// The block's token masks from its assignments' slots, and every assignment's rank.  All threads call it.
__device__ __forceinline__ void rank_block(const Pass &p, int n_blocks, uint32_t *blkmask, int t, int slot, int lane, int wave)
{
    if (slot >= 0) atomicOr(&blkmask[slot], 1u << wave);
    __syncthreads();
    int rank = 0;
    if (slot >= 0) {
        rank = __popc(blkmask[slot] & ((1u << wave) - 1u));
        if (rank == 0) atomicOr(&blkmask[slot], (uint32_t)lane << 16);   // one such lane per slot
    }
    if (t < p.T && lane < p.kk) p.slot_rank[(size_t)t * p.kk + lane] = slot >= 0 ? ((slot << 12) | rank) : -1;
    __syncthreads();
    for (int s = threadIdx.x; s < p.S; s += kFusedTokens * 64) {
        const uint32_t m = blkmask[s];
        p.blk_hist[(size_t)s * fused_row_stride(n_blocks) + blockIdx.x] = (int32_t)m;
        p.blk_cnt[(size_t)s * fused_row_stride(n_blocks) + blockIdx.x] = (uint8_t)__popc(m & 0xffffu);   // what the placing kernel adds up
    }
}

// kMany: batches that fill the chip; two workgroups per compute unit then matter more than a token's latency.
template <bool kMany, typename Table>
__global__ __launch_bounds__(kFusedTokens * 64) __attribute__((amdgpu_waves_per_eu(kMany ? 8 : 4))) void k_gate_select_hist(Pass p, int n_blocks, Table tab)
{
    extern __shared__ float smem[];
    const int S = p.S, stride = select_stride(p.E);
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    float *lg = smem + wave * 2 * stride;
    uint32_t *blkmask = (uint32_t *)(smem + kFusedTokens * 2 * stride);   // [S]
    int32_t *map = (int32_t *)(blkmask + S);                              // [E + n_shared]: looked up right after the selection
    // Staged behind the request for the logits where the launch does not fill the chip (gate phase, us, before it -> behind it: 16 tokens of the Qwen3 shape 13.5 -> 13.2, 333 16.0 -> 15.6,
    // DeepSeek-V3-shaped rank 512 tokens 20.5 -> 20.1; 8192 tokens 69.5 -> 70.0, Qwen3 shape 4096 25.1 -> 25.4).
    auto stage = [&]() {
        for (int s = threadIdx.x; s < S; s += kFusedTokens * 64) blkmask[s] = 0u;
        stage_table(p, tab, map, kFusedTokens * 64);
    };
    const int t = blockIdx.x * kFusedTokens + wave;
    int id = 0, slot = -1;
    if (kMany) stage();
    if (t < p.T) id = kMany ? select_one<4>(p, t, lg, lg + stride, lane, [] {}) : select_one<kGatePlanes>(p, t, lg, lg + stride, lane, stage);
    else if (!kMany) stage();
    __syncthreads();
    if (t < p.T) slot = slot_of_lane(p, map, t, lane, id);
    rank_block(p, n_blocks, blkmask, t, slot, lane, wave);
}

// Logits and selection in one kernel, for routers that a workgroup can multiply its own 16 tokens with (up to 64 experts,
// 512 wide: at most 128 KB, out of L2): such a layer is a chain of launches, and this is one less.  Wavefront w
// multiplies expert tile w mod n_et with its share of the contraction, the shares are added in K order.
// 64 tokens of the 128 x 64 fp32 layer: 8.3 us in two launches -> 5 us.
// kRank = false: the selection alone (the bookkeeping of the pass is separate).
template <typename XT, typename WT, typename Table, bool kRank>
__global__ __launch_bounds__(kFusedTokens * 64) void k_gate_small(Pass p, int n_blocks, Table tab)
{
    __shared__ float part[kFusedTokens * 256];
    __shared__ float lgs[kFusedTokens * 128];
    __shared__ int32_t map[kSmallExperts + 4];
    extern __shared__ uint32_t blkmask[];   // [S]
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6, t0 = blockIdx.x * kFusedTokens;
    if (kRank) {
        for (int s = threadIdx.x; s < p.S; s += kFusedTokens * 64) blkmask[s] = 0u;
        stage_table(p, tab, map, kFusedTokens * 64);
    }
    const SmallShare sh(p, wave, false);
    f32x4 acc[1];
    small_products<1, XT, WT>(p, t0, sh, lane, acc);
#pragma unroll
    for (int r = 0; r < 4; ++r) part[wave * 256 + r * 64 + lane] = acc[0][r];
    __syncthreads();
    const int t = t0 + wave;
    int slot = -1;
    if (t < p.T) {
        float v[1] = {small_logit(p, sh, part, wave, lane)};
        const int id = select_regs<1>(p, t, v, lgs + wave * 128, lgs + wave * 128 + 64, lane);
        if (kRank) slot = slot_of_lane(p, map, t, lane, id);
    }
    if (kRank) rank_block(p, n_blocks, blkmask, t, slot, lane, wave);
}

template <typename XT, typename WT>
hipError_t launch_gate_logits(const Pass &p, int planes, hipStream_t st)
{
    hipLaunchKernelGGL((k_gate_logits<XT, WT>), dim3((p.T + 15) / 16, (p.E + 15) / 16, planes), dim3(kThreads), 0, st, p);
    return hipGetLastError();
}

// planes for the few-token logits kernel: 4 chunks of 128 (one per wavefront) or more per workgroup
int few_token_planes(int T, int H)
{
    if (T > kGateFewTokens) return 1;
    const int z = (H + 127) / 128 / 4;
    return z < 1 ? 1 : z > kGatePlanes ? kGatePlanes : z;
}

template <typename WT>
hipError_t launch_logits_bf16(const Pass &p, int *planes, hipStream_t st)
{
    // Up to a hundred or so tokens there are too few (token, expert) tiles for the LDS-tiled kernels: the
    // K-split kernel reads both operands straight into registers, 16 tokens x 16 experts per workgroup, and
    // shares the contraction out over its wavefronts and over workgroups.  Up to 128 tokens it is ahead of the direct-to-LDS kernel (gate phase, us, this kernel -> that one)
    //  * for one block of tokens, whatever the router's size (512 experts on rows of 8192, fp32, one token 14.3 -> 18.4, 16 tokens 19.1 -> 22.4; 1024 on rows of 7168, bf16, 1 and 16
    //    34.6 -> 34.9, 42.6 -> 42.2);
    //  * while the router, which it reads once per block, comes to 16 MB (256 on rows of 7168, bf16, 32 tokens 14.2 -> 15.2, 64, 15 MB, 15.8 -> 15.4, 80, 18 MB, 17.8 -> 15.4, 128 19.2 -> 15.6; 128 on rows of 2048,
    //    fp32, 128, 8 MB, 13.1 -> 13.7; 256 on rows of 4096, fp32, 64, 16 MB, 15.8 -> 16.3, 65, 20 MB, 17.3 -> 16.4);
    //  * with an fp32 router, which the other one splits into three planes, while blocks of tokens times experts come to 1024 at most (rows of 7168, 256 experts, 64 tokens 19.0 -> 19.4, 65 21.6 -> 19.6; 384, 32
    //    21.1 -> 21.6, 33 23.3 -> 21.9; 128, 96 17.8 -> 18.2; 512 on rows of 8192, 32 22.1 -> 22.8, 33 25.5 -> 23.4).
    // (Without the direct-to-LDS kernel -- H not a multiple of 64 -- it stays ahead until the router re-reads reach about 128 MB.)
    const int blocks = (p.T + 15) / 16;
    const size_t router_rereads = (size_t)blocks * p.E * p.H * (p.router_bf16 ? 2 : 4);
    const bool few = blocks == 1 || router_rereads <= (size_t)16 << 20 || (!p.router_bf16 && blocks * p.E <= 1024);
    const bool small = gate_dma_supports(p) ? p.T <= 128 && few : (p.T <= kGateFewTokens || router_rereads <= (size_t)128 << 20);
    *planes = 1;
    if (!p.gate_tiled && small) {
        *planes = few_token_planes(p.T, p.H);
        return launch_gate_logits<uint16_t, WT>(p, *planes, st);
    }
    if (gate_dma_supports(p))      return launch_gate_logits_dma(p, planes, st);    // LDS ring filled by direct copies
    if (p.E > 64 && p.T >= 8192)   return launch_gate_logits_lds<WT, 4, 2>(p, st);   // 64 tokens x 128 experts
    return launch_gate_logits_lds<WT, 2, 1>(p, st);                                  // 32 tokens x 64 experts
}

template <bool kMany, typename Table>
hipError_t launch_select_hist(const Pass &p, const Table &tab, hipStream_t st)
{
    const int nb = (p.T + kFusedTokens - 1) / kFusedTokens;
    const size_t smem = sizeof(float) * kFusedTokens * 2 * (size_t)select_stride(p.E) + sizeof(uint32_t) * (p.S + p.E + p.n_shared);
    if (smem > 64 * 1024) {
        const hipError_t e = hipFuncSetAttribute((const void *)k_gate_select_hist<kMany, Table>, hipFuncAttributeMaxDynamicSharedMemorySize, (int)smem);
        if (e != hipSuccess) return e;
    }
    hipLaunchKernelGGL((k_gate_select_hist<kMany, Table>), dim3(nb), dim3(kFusedTokens * 64), smem, st, p, nb, tab);
    return hipGetLastError();
}

template <typename XT, typename WT>
hipError_t launch_small_t(const Pass &p, hipStream_t st)
{
    const int nb = (p.T + kFusedTokens - 1) / kFusedTokens;
    const size_t smem = sizeof(uint32_t) * p.S;
    if (!p.fused_hist) hipLaunchKernelGGL((k_gate_small<XT, WT, NoTable, false>), dim3(nb), dim3(kFusedTokens * 64), smem, st, p, nb, NoTable{});
    else if (p.host_table) hipLaunchKernelGGL((k_gate_small<XT, WT, TableArg, true>), dim3(nb), dim3(kFusedTokens * 64), smem, st, p, nb, fill_table(p));
    else hipLaunchKernelGGL((k_gate_small<XT, WT, NoTable, true>), dim3(nb), dim3(kFusedTokens * 64), smem, st, p, nb, NoTable{});
    return hipGetLastError();
}

hipError_t launch_gate_small(const Pass &p, hipStream_t st)
{
    if (p.act_bf16) return p.router_bf16 ? launch_small_t<uint16_t, uint16_t>(p, st) : launch_small_t<uint16_t, float>(p, st);
    return p.router_bf16 ? launch_small_t<float, uint16_t>(p, st) : launch_small_t<float, float>(p, st);
}

hipError_t launch_select(const Pass &p, hipStream_t st)
{
    if (p.fused_hist) {
        // the two forms are alike up to 4096 tokens (logits and selection of 256 experts 21.7 us both); 5000: 32.9 against 30.7,
        // 8192: 31.0 against 29.0
        const bool many = p.T > 2048;
        if (p.host_table) return many ? launch_select_hist<true>(p, fill_table(p), st) : launch_select_hist<false>(p, fill_table(p), st);
        return many ? launch_select_hist<true>(p, NoTable{}, st) : launch_select_hist<false>(p, NoTable{}, st);
    }
    const size_t smem = sizeof(float) * 4 * 2 * (size_t)select_stride(p.E);
    hipLaunchKernelGGL(k_gate_select, dim3((p.T + 3) / 4), dim3(kThreads), smem, st, p);
    return hipGetLastError();
}

}  // namespace

int gate_f32_planes(int T, int H) { return few_token_planes(T, H); }

// Whether logits and selection go in one kernel.  Its workgroups read the whole router per 16 tokens, so where the direct
// copies of k_gate_logits_dma serve the layer, those are ahead again once tokens x router is large (whole pass, us, one kernel
// -> separate, 64 experts on rows of 512: bf16 router 8192 tokens 56.2 -> 56.4, 20000: 78.1 -> 72.3, 60000: 179 -> 160; fp32
// router, where the separate selection ranks the assignments too, 2500: 40.2 -> 43.0, 5000: 47.7 -> 45.0, 8192: 60.6 -> 56.7,
// and where it does not, 10000: 60.8 -> 62.2, 20000: 87.1 -> 82.2).  The other logits kernels are not, or by 2 percent
// (rows of 264, 60000 tokens 125 -> 137; of 504, fp32 router, 184 -> 181).
bool one_gate_kernel(const Pass &p)
{
    if (p.gate_tiled || p.E > kSmallExperts || p.H > kSmallHidden) return false;
    const long long work = (long long)p.T * p.E * p.H;
    return !gate_dma_supports(p) || work <= (p.router_bf16 || p.T > kFusedMaxTokens ? 600000000ll : 150000000ll);
}

// Logits and selection of the tokens that the logits' memory holds, then of the next ones.
static hipError_t launch_gate_in_parts(const Pass &p, hipStream_t st)
{
    for (int t = 0; t < p.T; t += p.logit_tokens) {
        Pass q = p;
        q.T = p.T - t < p.logit_tokens ? p.T - t : p.logit_tokens;
        q.x = (const char *)p.x + (size_t)t * p.H * (p.act_bf16 ? 2 : 4);
        q.ids = p.ids + (size_t)t * p.k;
        q.w = p.w + (size_t)t * p.k;
        const hipError_t e = launch_gate(q, st);
        if (e != hipSuccess) return e;
    }
    return hipSuccess;
}

hipError_t launch_gate(Pass &p, hipStream_t st)
{
    hipError_t e;
    if (one_gate_kernel(p)) return launch_gate_small(p, st);
    if (p.act_bf16) {
        e = p.router_bf16 ? launch_logits_bf16<uint16_t>(p, &p.logit_planes, st) : launch_logits_bf16<float>(p, &p.logit_planes, st);
    } else {
        if (p.T > p.logit_tokens) return launch_gate_in_parts(p, st);
        const int room = p.logit_tokens / p.T, planes = gate_f32_planes(p.T, p.H);
        p.logit_planes = planes < room ? planes : room;
        e = p.router_bf16 ? launch_gate_logits<float, uint16_t>(p, p.logit_planes, st) : launch_gate_logits<float, float>(p, p.logit_planes, st);
    }
    return e == hipSuccess && !p.self_select ? launch_select(p, st) : e;
}

}  // namespace emoe
