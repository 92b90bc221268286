// Weight-streaming expert kernels for decode-sized batches whose contractions are whole K-steps (bf16, H and I
// multiples of 64).
//
// The memory-bound regime of the layer of Sec. 2.1 of the paper: a handful of rows per expert, every active expert's
// weights read once, slots without rows never touched (the tile list, or the selection kernel's block masks, only name
// slots that have rows; Sec. 3.2 / 4.6: placement is data, not layout).
//
// What bounds it: bytes on their way from HBM.  Weights travel as in the large-tile kernels, global memory straight into
// an LDS ring (global_load_lds_dwordx4, whole 128-byte lines, 8 rows per instruction, non-temporal when nobody else reads
// the slot), which holds more of them in flight than registers can and costs none; but a task is 128 weight rows and up to
// 32 token rows on four wavefronts in 80 KB of LDS, so that a compute unit runs two (120 KB in flight), one's first and
// last steps run beside the other's, and the end of a launch is dealt out in small pieces.  A wavefront stages and
// multiplies its own 32 weight rows; the token rows (4 KB per step at most) are shared.
// Against weights and token rows loaded into registers in MFMA layout (k_expert_decode, which serves contractions that are
// no whole K-steps): see the dispatch in moe_api.hip.
#include "moe_internal.h"
#include "self_tiles.h"

namespace emoe {
namespace {

typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef float f32x16 __attribute__((ext_vector_type(16)));

constexpr int kWaves = 4, kThreads = 64 * kWaves;
constexpr int kBN = 128;                     // weight rows per task, 32 per wavefront
constexpr int kBK = 64;                      // K-step: 128 bytes of every row
constexpr int kRows = 32;                    // token rows per tile
constexpr int kWStage = kBN * kBK * 2, kXStage = kRows * kBK * 2, kStage = kWStage + kXStage;   // 16 + 4 KB
constexpr int kDepth = 4;                    // stages: one multiplied, three on their way
constexpr int kWPieces = kWStage / 1024 / kWaves;   // 1 KB copies (8 rows) of weights per wavefront and step
static_assert(2 * kDepth * kStage <= 160 * 1024, "two workgroups per compute unit");
static_assert(kXStage / 1024 == kWaves, "a wavefront copies at most one piece of token rows");

// 16-byte slot of a 128-byte row in LDS: conflict-free operand reads (the large-tile kernels' swizzle)
__device__ __forceinline__ int swz8(int row) { return ((row >> 1) & 3) | (((row ^ (row >> 3)) & 1) << 2); }

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

template <bool kFirst, bool kSelf>
__global__ __launch_bounds__(kThreads, 2) void k_expert_ring(Pass p)
{
    static_assert(!kSelf || kFirst, "only GEMM-1 derives its tiles itself");
    constexpr int BNO = kFirst ? kBN / 2 : kBN;             // output columns per task
    __shared__ __attribute__((aligned(1024))) char ring[kDepth * kStage];
    const int K = kFirst ? p.H : p.I, N = kFirst ? p.I : p.H;
    const int slices = (N + BNO - 1) / BNO;
    const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    int task = blockIdx.x;
    if (kSelf) {
        if (task == 0) { self_tables(p, kRows, ring); return; }
        task -= 1;
    }
    const int tile = task / slices, slice = task - tile * slices, n0 = slice * BNO;
    MTile mt;
    unsigned long long tokens = 0;
    int tok0 = 0;
    if (kSelf) {
        if (!self_tile(p, lane, tile, kRows, &mt, &tokens, &tok0)) return;
    } else {
        if (tile >= *p.n_tiles) return;
        mt = p.tiles[tile];
    }

    // ---- what this lane copies: byte offsets from the matrix base at k = 0 ----
    const uint16_t *W = (const uint16_t *)(kFirst ? p.w13 : p.w2) + (size_t)mt.slot * (kFirst ? 2 : 1) * (size_t)p.I * p.H;
    const uint16_t *A = (const uint16_t *)(kFirst ? p.x : p.h);
    uint32_t woff[kWPieces], xoff = 0;
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
    const bool xload = wave * 8 < mt.rows;                  // this wavefront's piece of the token rows holds rows
    if (xload) {
        const int row = wave * 8 + (lane >> 3), r = min(row, mt.rows - 1);
        const int src = kSelf ? nth_set_bit(tokens, tok0 + r) : kFirst ? p.perm[mt.row_begin + r] : mt.row_begin + r;
        xoff = ((uint32_t)src * K + ((lane & 7) ^ swz8(row)) * 8) * 2;
    }
    const int KT = K / kBK;
    // the slices of a tile start spread over K (see the large-tile kernels: memory channels)
    const int first = slice * KT / slices;
    const uint32_t ring_a = lds_addr(ring);
    auto issue = [&](int i) {                               // step i in this task's order
        const int k0 = (i + first < KT ? i + first : i + first - KT) * kBK;
        const uint32_t st = ring_a + (i % kDepth) * kStage;
        if (mt.single) {
#pragma unroll
            for (int j = 0; j < kWPieces; ++j) copy_piece<true>(W + k0, woff[j], st + (wave * kWPieces + j) * 1024);
        } else {
#pragma unroll
            for (int j = 0; j < kWPieces; ++j) copy_piece<false>(W + k0, woff[j], st + (wave * kWPieces + j) * 1024);
        }
        if (xload) copy_piece<false>(A + k0, xoff, st + kWStage + wave * 1024);
    };
    // ---- operand rows of this lane ----
    const int l31 = lane & 31, khalf = lane >> 5, wr = wave * 32 + l31;
    uint32_t wo[4], xo[4];
#pragma unroll
    for (int ks = 0; ks < 4; ++ks) {
        wo[ks] = wr * 128 + (((ks * 2 + khalf) ^ swz8(wr)) << 4);
        xo[ks] = kWStage + l31 * 128 + (((ks * 2 + khalf) ^ swz8(l31)) << 4);
    }
    f32x16 acc;
#pragma unroll
    for (int r = 0; r < 16; ++r) acc[r] = 0.f;
    for (int s = 0; s < kDepth - 1 && s < KT; ++s) issue(s);
    for (int kt = 0; kt < KT; ++kt) {
        // step kt has landed when at most the copies of the younger steps (two at most) are still on their way
        const int younger = min(kDepth - 2, KT - 1 - kt);
        if (younger == 2)      { if (xload) wait_loads<2 * kWPieces + 2>(); else wait_loads<2 * kWPieces>(); }
        else if (younger == 1) { if (xload) wait_loads<kWPieces + 1>(); else wait_loads<kWPieces>(); }
        else                   wait_loads<0>();
        __syncthreads();   // everyone's pieces of step kt are in LDS; everyone is done reading step kt-1
        if (kt + kDepth - 1 < KT) issue(kt + kDepth - 1);
        const char *st = ring + (kt % kDepth) * kStage;
#pragma unroll
        for (int ks = 0; ks < 4; ++ks) {
            const uint4 w = *(const uint4 *)(st + wo[ks]), x = *(const uint4 *)(st + xo[ks]);
            acc = __builtin_amdgcn_mfma_f32_32x32x16_bf16(*(const bf16x8 *)&w, *(const bf16x8 *)&x, acc, 0, 0, 0);
        }
    }
    // lane holds token row l31, weight rows 8 q + 4 khalf + 0..3 of this wavefront's 32
    if (l31 >= mt.rows) return;
    uint16_t *O = (uint16_t *)(kFirst ? p.h : p.y) + (size_t)(mt.row_begin + l31) * N;
#pragma unroll
    for (int q = 0; q < (kFirst ? 2 : 4); ++q) {
        const int col = n0 + wave * (kFirst ? 16 : 32) + q * 8 + khalf * 4;
        if (col >= N) continue;
        uint16_t o[4];
#pragma unroll
        for (int e = 0; e < 4; ++e) o[e] = f32_to_bf16(kFirst ? silu_mul(acc[q * 4 + e], acc[(q + 2) * 4 + e]) : acc[q * 4 + e]);
        *(uint2 *)(O + col) = make_uint2((uint32_t)o[0] | ((uint32_t)o[1] << 16), (uint32_t)o[2] | ((uint32_t)o[3] << 16));
    }
}

}  // namespace

int ring_tile_rows() { return kRows; }

hipError_t launch_experts_ring(const Pass &p, int which, hipStream_t st)
{
    if (which == 0) {
        const int blocks = p.max_tiles * ((p.I + kBN / 2 - 1) / (kBN / 2));
        if (p.self_tiles) hipLaunchKernelGGL((k_expert_ring<true, true>), dim3(blocks + 1), dim3(kThreads), 0, st, p);
        else              hipLaunchKernelGGL((k_expert_ring<true, false>), dim3(blocks), dim3(kThreads), 0, st, p);
    } else {
        const int blocks = p.max_tiles * ((p.H + kBN - 1) / kBN);
        hipLaunchKernelGGL((k_expert_ring<false, false>), dim3(blocks), dim3(kThreads), 0, st, p);
    }
    return hipGetLastError();
}

}  // namespace emoe
