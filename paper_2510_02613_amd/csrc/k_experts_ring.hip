// Weight-streaming expert kernels for small groups of rows whose contractions are whole K-steps (bf16, H and I
// multiples of 64).
//
// The memory-bound regime of the layer of Sec. 2.1 of the paper: a handful of rows per expert, every active expert's
// weights read once, slots without rows never touched (the tile list, or the selection kernel's block masks, only name
// slots that have rows; Sec. 3.2 / 4.6: placement is data, not layout).
//
// What bounds it: bytes on their way from HBM.  Weights travel as in the large-tile kernels, global memory straight into
// an LDS ring (global_load_lds_dwordx4, whole 128-byte lines, 8 rows per instruction, non-temporal when nobody else reads
// the slot), which holds more of them in flight than registers can and costs none; but a task is 128 weight rows and up to
// 32 or 64 token rows on four wavefronts in 80 KB of LDS, so that a compute unit runs two (120 KB in flight), one's first and
// last steps run beside the other's, and the end of a launch is dealt out in small pieces.  A wavefront stages and
// multiplies its own 32 weight rows; the token rows (4 KB per step and 32 rows) are shared.  Tiles of 33 to 64 rows have a ring of
// three stages instead of four.  Products are v_mfma_f32_16x16x32_bf16 over the 16-row token tiles that have rows: next to the
// 32x32x16 form on 32-row tiles, whole pass, us: Qwen3 shape 48 tokens 188.8 -> 187.6, DeepSeek-V3-shaped rank 8 tokens 184.8 -> 180 .. 184,
// 30 tokens 381 -> 380, 64 tokens 471 -> 470.
// Against weights and token rows loaded into registers in MFMA layout (k_expert_decode, which serves contractions that are
// no whole K-steps): see the dispatch in moe_api.hip.
#include <type_traits>

#include "moe_internal.h"
#include "self_tiles.h"

namespace emoe {
namespace {

typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef float f32x4 __attribute__((ext_vector_type(4)));

constexpr int kWaves = 4, kThreads = 64 * kWaves;
constexpr int kBN = 128;                     // weight rows per task, 32 per wavefront
constexpr int kBK = 64;                      // K-step: 128 bytes of every row
constexpr int kWStage = kBN * kBK * 2;       // 16 KB
constexpr int kWPieces = kWStage / 1024 / kWaves;   // 1 KB copies (8 rows) of weights per wavefront and step
constexpr int kRows = 32;                    // token rows per token tile
constexpr int kLds = 80 * 1024;              // two workgroups per compute unit
// a stage: the step's weight rows, then TT x 32 token rows (4 KB each); as many stages as fit (one multiplied, the others on their way)
template <int TT> struct Ring {
    static constexpr int kStage = kWStage + TT * 4096, kDepth = kLds / kStage;
    static_assert(kDepth == 3 || kDepth == 4, "the waits of the K loop");
};

__device__ __forceinline__ uint32_t lds_addr(const void *p)
{
    return (uint32_t)(uintptr_t)(__attribute__((address_space(3))) const void *)p;
}

// global -> LDS copy of one 1 KB piece (lane i's 16 bytes land at lds + 16 i), in inline assembly so that the compiler
// does not wait for it before later LDS reads; completion is awaited in the K loop
template <bool kStream>
__device__ __forceinline__ void copy_piece(const void *base, uint32_t byte_off, uint32_t lds)
{
    if (kStream) asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %1, %2 nt" ::"s"(lds), "v"(byte_off), "s"(base) : "memory", "m0");
    else         asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %1, %2" ::"s"(lds), "v"(byte_off), "s"(base) : "memory", "m0");
}

template <int n>
__device__ __forceinline__ void wait_loads()
{
    __builtin_amdgcn_s_waitcnt((n & 15) | ((n >> 4) << 14) | (7 << 4) | (15 << 8));   // vmcnt only
}
// Wait until at most kSteps steps' copies are on their way, of a wavefront with xlive pieces of token rows per step (the count is
// an immediate of the instruction).
template <int kSteps, int TT>
__device__ __forceinline__ void wait_younger(int xlive)
{
    if (TT == 2 && xlive == 2) wait_loads<kSteps * (kWPieces + 2)>();
    else if (xlive)            wait_loads<kSteps * (kWPieces + 1)>();
    else                       wait_loads<kSteps * kWPieces>();
}

// The part of a task behind the tile lookup, for a tile of up to 16 HT rows; tokens, tok0 (kSelf) or tok (LDS, not NULL): the tile's rows where
// GEMM-1 derived them.
template <bool kFirst, bool kSelf, int HT>
__device__ __forceinline__ void task_body(const Pass &p, const MTile &mt, int slice, int slices, unsigned long long tokens, int tok0, const int32_t *tok, char *ring)
{
    constexpr int TT = (HT + 1) / 2;
    using R = Ring<TT>;
    constexpr int BNO = kFirst ? kBN / 2 : kBN;             // output columns per task
    constexpr int kDepth = R::kDepth;
    const int K = kFirst ? p.H : p.I, N = kFirst ? p.I : p.H, n0 = slice * BNO;
    const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);

    // ---- what this lane copies: byte offsets from the matrix base at k = 0 ----
    const uint16_t *W = (const uint16_t *)(kFirst ? p.w13 : p.w2) + (size_t)mt.slot * (kFirst ? 2 : 1) * (size_t)p.I * p.H;
    const uint16_t *A = (const uint16_t *)(kFirst ? p.x : p.h);
    uint32_t woff[kWPieces], xoff[TT];
#pragma unroll
    for (int i = 0; i < kWPieces; ++i) {
        const int within = i * 8 + (lane >> 3), row = wave * 32 + within;     // weight row of the task
        int g;
        if (kFirst) {   // a wavefront's 32 rows: 16 gate rows, then the 16 matching up rows
            const int col = n0 + wave * 16 + (within & 15);
            g = within < 16 ? col : p.I + col;
        } else {
            g = min(n0 + row, N - 1);
        }
        woff[i] = ((uint32_t)g * K + ((lane & 7) ^ swz8(row)) * 8) * 2;
    }
    // pieces of token rows (8 rows each) that hold rows: pieces wave and wave + 4
    const int xlive = (wave * 8 < mt.rows) + (TT == 2 && (wave + kWaves) * 8 < mt.rows);
#pragma unroll
    for (int i = 0; i < TT; ++i) {
        xoff[i] = 0;
        if (i >= xlive) continue;
        const int row = (wave + kWaves * i) * 8 + (lane >> 3), r = min(row, mt.rows - 1);
        const int src = kSelf ? nth_set_bit(tokens, tok0 + r) : !kFirst ? mt.row_begin + r : tok ? tok[r] : p.perm[mt.row_begin + r];
        xoff[i] = ((uint32_t)src * K + ((lane & 7) ^ swz8(row)) * 8) * 2;
    }
    const int KT = K / kBK;
    // the slices of a tile start spread over K (see the large-tile kernels: memory channels)
    const int first = slice * KT / slices;
    const uint32_t ring_a = lds_addr(ring);
    auto issue = [&](int i) {                               // step i in this task's order
        const int k0 = (i + first < KT ? i + first : i + first - KT) * kBK;
        const uint32_t st = ring_a + (i % kDepth) * R::kStage;
        if (mt.single) {
#pragma unroll
            for (int j = 0; j < kWPieces; ++j) copy_piece<true>(W + k0, woff[j], st + (wave * kWPieces + j) * 1024);
        } else {
#pragma unroll
            for (int j = 0; j < kWPieces; ++j) copy_piece<false>(W + k0, woff[j], st + (wave * kWPieces + j) * 1024);
        }
#pragma unroll
        for (int j = 0; j < TT; ++j)
            if (j < xlive) copy_piece<false>(A + k0, xoff[j], st + kWStage + (wave + kWaves * j) * 1024);
    };
    // ---- operand rows of this lane: 16-row tiles, two of weights, HT of tokens ----
    const int l15 = lane & 15, quad = lane >> 4, wr = wave * 32 + l15;
    uint32_t wo[2], xo[2];
#pragma unroll
    for (int ks = 0; ks < 2; ++ks) {
        wo[ks] = wr * 128 + (((ks * 4 + quad) ^ swz8(wr)) << 4);
        xo[ks] = kWStage + l15 * 128 + (((ks * 4 + quad) ^ swz8(l15)) << 4);
    }
    f32x4 acc[2][HT];
#pragma unroll
    for (int a = 0; a < 2; ++a)
#pragma unroll
        for (int t = 0; t < HT; ++t) acc[a][t] = (f32x4){0.f, 0.f, 0.f, 0.f};
    for (int s = 0; s < kDepth - 1 && s < KT; ++s) issue(s);
    for (int kt = 0; kt < KT; ++kt) {
        // step kt has landed when at most the copies of the younger steps (kDepth - 2 at most) are still on their way
        const int younger = min(kDepth - 2, KT - 1 - kt);
        if (younger == kDepth - 2)               wait_younger<kDepth - 2, TT>(xlive);
        else if (kDepth == 4 && younger == 1)    wait_younger<1, TT>(xlive);
        else                                     wait_loads<0>();
        __syncthreads();   // everyone's pieces of step kt are in LDS; everyone is done reading step kt-1
        if (kt + kDepth - 1 < KT) issue(kt + kDepth - 1);
        const char *st = ring + (kt % kDepth) * R::kStage;
        uint4 w[2][2], x[2][HT];
#pragma unroll
        for (int ks = 0; ks < 2; ++ks) {
#pragma unroll
            for (int a = 0; a < 2; ++a) w[ks][a] = *(const uint4 *)(st + wo[ks] + a * 2048);
#pragma unroll
            for (int t = 0; t < HT; ++t) x[ks][t] = *(const uint4 *)(st + xo[ks] + t * 2048);
        }
        __builtin_amdgcn_sched_barrier(0);   // all reads go out before the first product waits for its own
#pragma unroll
        for (int ks = 0; ks < 2; ++ks)
#pragma unroll
            for (int t = 0; t < HT; ++t)
#pragma unroll
                for (int a = 0; a < 2; ++a)
                    acc[a][t] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(*(const bf16x8 *)&w[ks][a], *(const bf16x8 *)&x[ks][t], acc[a][t], 0, 0, 0);
    }
    // lane holds token rows 16 t + l15, weight rows 16 a + 4 quad + 0..3 of this wavefront's 32
#pragma unroll
    for (int t = 0; t < HT; ++t) {
        const int m = 16 * t + l15;
        if (m >= mt.rows) continue;
        uint16_t *O = (uint16_t *)(kFirst ? p.h : p.y) + (size_t)(mt.row_begin + m) * N;
#pragma unroll
        for (int a = 0; a < (kFirst ? 1 : 2); ++a) {
            const int col = n0 + wave * (kFirst ? 16 : 32) + a * 16 + quad * 4;
            if (col >= N) continue;
            uint16_t o[4];
#pragma unroll
            for (int e = 0; e < 4; ++e) o[e] = f32_to_bf16(kFirst ? silu_mul(acc[0][t][e], acc[1][t][e]) : acc[a][t][e]);
            *(uint2 *)(O + col) = make_uint2((uint32_t)o[0] | ((uint32_t)o[1] << 16), (uint32_t)o[2] | ((uint32_t)o[3] << 16));
        }
    }
}

// GEMM-1 that reads the bookkeeping kernels' tile list: an instance of its own, without the code that derives tiles, which spills 56 scalars (in front of its K loops).
// One kernel for both cost routed passes 0.3 to 0.7 % (whole pass, us, both in one -> this: DeepSeek-V2-Lite shape, 180 tokens on 32 experts 126.4 -> 125.7, on 16 78.7 -> 78.3, 120 on
// 32 121.9 -> 121.1, Qwen3 shape 200 on 32 63.1 -> 62.9).
struct TileList {};

// kTiles: the most token tiles of 32 rows an M-tile has.
// How GEMM-1 comes by its tiles: TileList; NoTable or TableArg: a token to four, it selects the experts too (see k_experts_decode.hip); none: kSelf up to 64 tokens, else up
// to 1024.  Selection, whole pass, us, selection kernel -> here: Qwen3
// shape two tokens 39.7 -> 36.9, four 63.7 -> 61.0, four on half of its experts 36.0 -> 33.3; DeepSeek-V2-Lite shape three tokens 68.7 -> 66.2, four
// 75.2 -> 72.5.  The limit on the workgroups is the register kernels', measured for both there.
template <bool kFirst, bool kSelf, int kTiles, typename... How>
__global__ __launch_bounds__(kThreads, 2) void k_expert_ring(Pass p, How... how)
{
    constexpr bool kList = !kFirst || (std::is_same_v<How, TileList> || ...), kSelect = sizeof...(How) == 1 && !kList, kMany = !kSelf && !kList;
    static_assert(!kSelect || (kSelf && kSelectTokens == kWaves), "a GEMM-1 that selects derives its tiles too, a wavefront selects a token");
    static_assert(!kSelf || (kFirst && !kList), "only GEMM-1 derives its tiles itself");
    constexpr int BNO = kFirst ? kBN / 2 : kBN;             // output columns per task
    __shared__ __attribute__((aligned(1024))) char ring[kLds];
    const int N = kFirst ? p.I : p.H;
    const int slices = (N + BNO - 1) / BNO;
    int task = blockIdx.x;
    std::conditional_t<kSelect, SelfLds, SelfTables> src;
    static_assert(sizeof(SelectLds) <= kLds - 16384 && kSelfTableBytes <= 16384, "the selection borrows the ring, the tables are put together in front of it");
    if constexpr (kSelect) src = select_few(p, *(SelectLds *)(ring + 16384), how...);
    // The tiles of up to 1024 tokens too are derived here: a launch and its tables' round trips less, for
    // 1 to 2 us in front of a workgroup's stream (whole pass, us, k_scan_place -> here: 32 Qwen3 experts, 65 tokens 68.2 -> 65.6, 320 75.9 -> 73.1, 128 experts, 100 tokens 207.8 -> 203.0; DeepSeek-V2-Lite
    // shape 64 tokens 205.0 -> 201.7, 213 224.0 -> 218.1; 16 experts of 512, 1020 tokens 58.6 -> 55.8; where it costs more than it saves: self_table_blocks).
    if constexpr (!kList) {
        const int tables = kMany ? p.table_blocks : 1;
        if (task < tables) {
            if constexpr (kMany) many_tables(p, kTiles * kRows, task, ring);
            else                 self_tables(p, kRows, ring, src);
            return;
        }
        task -= tables;
    }
    const int tile = task / slices, slice = task - tile * slices;
    MTile mt;
    unsigned long long tokens = 0;
    int tok0 = 0;
    // in the last 8 KB, which the first copies leave alone: a ring of two token tiles ends before them, one of one copies there behind the first barrier
    int32_t *tok = kMany ? (int32_t *)(ring + kLds - 8192) + (threadIdx.x >> 6) * (kTiles * kRows) : nullptr;
    static_assert(3 * Ring<2>::kStage <= kLds - 8192 && 3 * Ring<1>::kStage <= kLds - 8192, "what is copied before that barrier");
    if constexpr (kMany) {
        if (!many_tile(p, threadIdx.x & 63, tile, kTiles * kRows, &mt, tok)) return;
    } else if constexpr (kSelf) {
        if (!self_tile(p, threadIdx.x & 63, tile, kRows, &mt, &tokens, &tok0, src)) return;
        if (kSelect) __syncthreads();   // everyone has read the masks: the ring is free
    } else {
        if (tile >= *p.n_tiles) return;
        mt = p.tiles[tile];
    }
    if constexpr (kTiles == 2) {
        if (mt.rows > 48) { task_body<kFirst, kSelf, 4>(p, mt, slice, slices, tokens, tok0, tok, ring); return; }
        if (mt.rows > 32) { task_body<kFirst, kSelf, 3>(p, mt, slice, slices, tokens, tok0, tok, ring); return; }
    }
    if (mt.rows > 16) task_body<kFirst, kSelf, 2>(p, mt, slice, slices, tokens, tok0, tok, ring);
    else              task_body<kFirst, kSelf, 1>(p, mt, slice, slices, tokens, tok0, tok, ring);
}

}  // namespace

int ring_tile_rows(bool large) { return large ? 2 * kRows : kRows; }

int ring_blocks(const Pass &p) { return p.max_tiles * ((p.I + kBN / 2 - 1) / (kBN / 2)); }

// Every wavefront of GEMM-1 adds up the count bytes of all slots: 16-byte loads of a lane, one per 64 slots and 256 tokens, in each workgroup.  With rows of 1024 and more they
// hide behind the weight stream (whole pass, us, k_scan_place -> derived: 256 slots of 2048 x 768, 576 tokens 399 -> 392, of 2048 x 64, 1024 76 -> 73 and 78 -> 77; 250 of 1024 x 192, 700 76.0 -> 74.9,
// 1024 78.4 -> 78.6).  Shorter rows end too soon for that: up to 5500 loads of all workgroups' lanes derived (256 slots of 128 x 128, 512 tokens, 4600 loads 28.0 -> 26.3, of 512 x 64, 1024, 5100 36.8 -> 36.1; 128 of
// 320 x 192, 1024, 4600 33.5 -> 31.0), above list (128 slots of 256 x 256, 784 tokens, 5700 loads 31.9 -> 32.4, 640 x 256, 1024, 6100 47.3 -> 48.2; 256 of 128 x 128, 640, 7100 28.1 -> 29.2, 320 x 320, 1024, 25600
// 56.0 -> 61.8, 256 x 256 43.3 -> 48.9).  What that leaves: up to 512 tokens some would gain further up (256 slots of 192 x 192, 6900 loads 34.8 -> 33.8; 256 x 256, 9200 41.0 -> 42.8).
constexpr int kLongRow = 1024, kManyLoads = 5500;

// (sums of rows are kept in 15 bits)
int self_table_blocks(const Pass &p)
{
    if (!p.fused_hist || p.S > kSelfMaxSlots || p.T > kManyBlocks * kFusedTokens || p.T * p.kk >= (1 << 15)) return 0;
    const int loads = (p.S + 63) / 64 * ((p.T + 16 * kFusedTokens - 1) / (16 * kFusedTokens));
    return p.H >= kLongRow || ring_blocks(p) * loads <= kManyLoads ? table_blocks(p) : 0;
}

hipError_t launch_experts_ring(const Pass &p, int tile_rows, int which, hipStream_t st)
{
    const dim3 block(kThreads), grid(which == 0 ? ring_blocks(p) + (p.table_blocks > 0 ? p.table_blocks : p.self_tiles ? 1 : 0) : p.max_tiles * ((p.H + kBN - 1) / kBN));
    const bool many = p.table_blocks > 0;
    if (tile_rows > kRows) {
        if (which != 0) hipLaunchKernelGGL((k_expert_ring<false, false, 2>), grid, block, 0, st, p);
        else if (many)  hipLaunchKernelGGL((k_expert_ring<true, false, 2>), grid, block, 0, st, p);
        else            hipLaunchKernelGGL((k_expert_ring<true, false, 2, TileList>), grid, block, 0, st, p, TileList{});
    } else if (which == 0) {
        if (p.self_select && p.host_table) {
            hipLaunchKernelGGL((k_expert_ring<true, true, 1, TableArg>), grid, block, 0, st, p, fill_table(p));
        } else if (p.self_select) {
            hipLaunchKernelGGL((k_expert_ring<true, true, 1, NoTable>), grid, block, 0, st, p, NoTable{});
        } else if (many) {
            hipLaunchKernelGGL((k_expert_ring<true, false, 1>), grid, block, 0, st, p);
        } else if (p.self_tiles) {
            hipLaunchKernelGGL((k_expert_ring<true, true, 1>), grid, block, 0, st, p);
        } else {
            hipLaunchKernelGGL((k_expert_ring<true, false, 1, TileList>), grid, block, 0, st, p, TileList{});
        }
    } else {
        hipLaunchKernelGGL((k_expert_ring<false, false, 1>), grid, block, 0, st, p);
    }
    return hipGetLastError();
}

}  // namespace emoe
