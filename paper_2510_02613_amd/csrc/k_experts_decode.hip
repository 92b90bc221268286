// Weight-streaming expert kernels for decode-sized batches (bf16): operands in registers, small tasks.  They serve what the
// LDS-ring kernels leave: contractions that are no whole K-steps, passes with too few of the ring's 128-row tasks for the
// chip, and passes with a little more than one of them per compute unit (the dispatch in moe_api.hip has the counts).
//
// With a few tokens per step most resident experts receive 0-4 rows (the
// memory-bound regime of the layer of Sec. 2.1 of the paper under expert
// parallelism): the work is reading every ACTIVE expert's weights once, and the
// right measure is HBM bandwidth.  Slots without rows are never touched -- the
// tile list, built from the active expert map (Sec. 3.2 / 4.6: placement is data,
// not layout), only names slots that have rows.
//
// A task is a block of weight rows of one M-tile (<= 16 grouped rows): GEMM-1 takes 16
// gate rows and the 16 matching up rows (so silu(g)*u is formed in registers), GEMM-2
// 32 consecutive W2 rows.  A task is one workgroup of four wavefronts, each walking a
// quarter of the contraction.  Weights and token rows go straight from global memory
// into MFMA operand layout, as in the gate kernel: for a K-chunk of 128, lane
// (n = l%16, q = l/16) reads the 32 k {jj*32 + q*8 + i} of row n with four 16-byte
// loads issued back to back, so every row contributes a contiguous 256-byte run per
// chunk.  v_mfma_f32_16x16x32_bf16 with the weights as first operand gives lane
// (j = l%16, q) the outputs of token j for weight rows 4q..4q+3: one 8-byte store.
// The next chunk's loads are in flight during the current chunk's MFMAs: 8 KB of weights (and 4 KB of token rows, which mostly
// come from L2) per wavefront, 96 to 128 KB of weights per compute unit with 12 to 16 wavefronts, 192 KB with 8 that are three chunks ahead (the forms below).
#include <type_traits>

#include "moe_internal.h"
#include "self_tiles.h"

namespace emoe {
namespace {

typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef float f32x4 __attribute__((ext_vector_type(4)));

constexpr int kThreads = 64;    // a wavefront; a workgroup is one task: the kSplit wavefronts that share its contraction
constexpr int kTileRows = 16;   // grouped rows per M-tile (one MFMA N dimension)
constexpr int kWRows = 32;      // weight rows per wavefront

struct Run { uint4 v[4]; };     // a lane's 32 k of one row of a 128-wide K chunk

__device__ __forceinline__ void load_run(Run &r, const uint16_t *row, int k0, int q, int K)
{
#pragma unroll
    for (int jj = 0; jj < 4; ++jj) {
        const int k = k0 + jj * 32 + q * 8;
        r.v[jj] = (k < K) ? *(const uint4 *)(row + k) : make_uint4(0, 0, 0, 0);  // K % 8 == 0
    }
}

constexpr int kBlocks2 = 2;   // 16-row weight blocks per task in GEMM-2
// Wavefronts that share a task's contraction: each takes a contiguous quarter of the K-chunks, the first adds
// the four sums in K order (through LDS) and stores.  A wavefront's stream is latency bound (one chunk or three in
// flight), so a launch ends with a tail as long as one task in which ever fewer wavefronts stream; with four
// wavefronts per task that tail is a quarter as long, and the tasks of a launch (several rounds of the chip's
// wavefront slots in GEMM-2) are dealt to the compute units in finer pieces.  Measured on the DeepSeek-V3-shaped
// rank with 64 tokens: GEMM-1 291 -> 277 us, GEMM-2 161 -> 140 us (2 or 8 wavefronts per task: slower).
constexpr int kSplit1 = 4;
constexpr int kSplit2 = 4;

// The K loop is unrolled over the chunk multiplied and those requested ahead of it, so that a chunk's registers are where the MFMAs read
// them (copied from the prefetched chunk's after every step before: whole pass, us, copied -> unrolled, one ahead: one token of the
// Qwen3 shape 30.7 -> 30.1, of the DeepSeek-V3-shaped rank 48.7 -> 46.3, two 50.9 -> 47.5, five on 16 of its experts 68.0 -> 65.3).
// Three forms, by the length of the contraction:
//  * kShort: one chunk ahead on four wavefronts per SIMD.  kMiddle: the same on three (134 to 138 registers; never more, should a compiler find fewer).  With one to three chunks a wavefront
//    there is little to request ahead, and what hides a task's first loads is another task; with more the fourth wavefront only makes
//    more rows be walked at a time.  128 experts, T tokens, us, one ahead on three -> on four wavefronts.  GEMM-2, rows of I: 264 wide, T = 16, H = 2056 20.4 ->
//    19.1, T = 48 30.7 -> 27.6; 520, T = 16, H = 1032 21.6 -> 20.5, H = 2056 35.4 -> 35.2, T = 48 50.5 -> 51.5; 760 and more 48.2 -> 50.0, 70.9 -> 75.2
//    (nothing between 520 and 760).  GEMM-1, rows of H: 264, T = 48 14.8 -> 14.2; 776 22.9 -> 22.2; 1032, I = 264 28.9 -> 28.2, I = 1032, T = 16 80.2 -> 79.3;
//    1544, I = 264, T = 48 42.4 -> 43.5; 2056, I = 760 153 -> 158 (nothing between 1032 and 1544).  Whole pass, copied -> three everywhere -> the forms: 520 x 264, T = 48 40.7 -> 41.7
//    -> 40.2; 2056 x 264 100.1 -> 101.3 -> 98.0; 2056 x 760 247.4 -> 237.4 -> 237.6.  What is left: 1032 x 520, T = 6 44.4 -> 43.2 -> 43.9; a little over one round of
//    four (the Qwen3 shape, 32 of its experts, T = 16 to 28) 48.9 -> 49.3 -> 49.3, where GEMM-2 on four would be 48.4, but three tokens 54.2 -> 54.4 and five 78.1 -> 78.7.
//  * kLong: three chunks ahead on two wavefronts per SIMD, GEMM-1 only.  Rows of 7168: one token 46.3 -> 44.6, five on 16 experts 66.7 -> 65.3, 64 tokens, I = 2040, 513 -> 508;
//    6152, 24 tokens 550 -> 530; 5128 460 -> 445; 4104 339 -> 326; 3080 283 -> 274, but rows of 4096 and three tokens 78.1 -> 79.9, of 3072
//    71.6 -> 75.2, of 2048 54.0 -> 58.5: what few tokens lose there is more than what many gain.  Workgroups that
//    find no tile take their turn two to a compute unit: where none of a token's or two's experts are here, 15.6 -> 16.4, 18.2 -> 19.8 (on three wavefronts 15.9, 18.8).
enum Form { kShort, kMiddle, kLong };
constexpr int kShort1 = 1280, kLong1 = 4096;   // GEMM-1: the last H of kShort and of kMiddle
constexpr int kShort2 = 640;                   // GEMM-2: the last I of kShort
constexpr int waves_of(int form) { return form == kShort ? 4 : form == kMiddle ? 3 : 2; }

// Table (NoTable or TableArg, or none): GEMM-1 of a token to four selects its experts, behind the logits kernel alone.  The selection kernel is nothing but latency then (one
// workgroup between two launches).  Every workgroup selects all tokens itself instead, a wavefront each, and workgroup 0 leaves the ids,
// the weights and (tab) the placement in the workspace.  Whole pass, us, selection kernel -> here: one token of the Qwen3 shape 30.5 ->
// 27.4, three 55.3 -> 53.6, four on 32 of its experts 32.4 -> 29.1 (1536 workgroups); DeepSeek-V2-Lite shape two tokens 52.3 -> 50.3, on
// 16 of its experts one 27.4 -> 25.1, four 38.4 -> 36.7 (1760 workgroups).  A workgroup pays 1 to 2 us for it, one that finds no tile too, so
// there is a limit on their number.  Rows of 2048, 16 experts of 128 here, so that most workgroups find no tile: 1728 workgroups 32.5 -> 31.8, 2048 29.2 -> 29.2, 2304 33.0 ->
// 36.7, 2560 31.3 -> 35.0, 3456 42.7 -> 49.6; all 128 here, whose weight stream hides it: 2112 94.2 -> 92.1, 3072 125.4 -> 123.6, 4096 151.0 -> 150.1.  The ring
// kernels, the same line: 1536 workgroups, all experts here 187 -> 182, 1088, 16 experts here 58.9 -> 56.7; 2048, all here 273.6 -> 270.6, half of them 103.2 -> 105.0, 4096 185 -> 200.  Group-limited gates take several times as long to select (DeepSeek-V3-shaped
// rank one token 45.0 -> 45.0, two 46.2 -> 55.4): they keep their kernel, and so do
// more than 128 experts (256 in GEMM-1, four scores a lane, not taken up: rows of 2048, one token 30.7 -> 27.6, four 64.9 -> 61.9, on 32 of them one 21.0 -> 18.8, four 25.0 -> 25.5) and
// more tokens: two a wavefront made five tokens of the DeepSeek-V2-Lite shape 90.5 -> 95.3, eight on 32 Qwen3 experts 34.9 -> 43.0.
constexpr long long kSelectBlocks = 1760;
template <bool kFirst, bool kSelf, int kForm, typename... Table>
__global__ __launch_bounds__(kFirst ? kThreads * kSplit1 : kThreads * kSplit2) __attribute__((amdgpu_waves_per_eu(kForm == kShort ? waves_of(kForm) : 1, waves_of(kForm)))) void k_expert_decode(Pass p, Table... tab)
{
    constexpr bool kSelect = sizeof...(Table) == 1;
    static_assert(!kSelf || kFirst, "only GEMM-1 derives its tiles itself");
    static_assert(!kSelect || kSelf, "a GEMM-1 that selects derives its tiles too");
    constexpr int NS = kFirst ? kSplit1 : kSplit2;                // wavefronts of this workgroup (one task)
    const int K = kFirst ? p.H : p.I;
    const int N = kFirst ? p.I : p.H;                       // output columns
    constexpr bool kTwo = kFirst || kBlocks2 == 2;          // two weight rows per lane
    constexpr int COLS = kFirst ? kWRows / 2 : 16 * kBlocks2;   // output columns per wavefront
    const int groups = (N + COLS - 1) / COLS;               // wavefront tasks per M-tile
    const int lane = threadIdx.x & 63;
    const int ks = NS > 1 ? (int)(threadIdx.x >> 6) : 0;    // which part of the contraction
    int task = blockIdx.x;
    std::conditional_t<kSelect, SelfLds, SelfTables> src;
    if constexpr (kSelect) {
        static_assert(kSelectTokens == NS, "a wavefront selects a token");
        __shared__ SelectLds sel;
        src = select_few(p, sel, tab...);
    }
    if (kSelf) {
        __shared__ int32_t lds[kSelfTableBytes / 4];
        if (task == 0) { self_tables(p, kTileRows, lds, src); return; }
        task -= 1;
    }
    const int tile = task / groups;
    const int n = lane & 15, q = lane >> 4;
    MTile mt;
    int self_token = 0;                                     // kSelf: the token of this lane's row
    if (kSelf) {
        unsigned long long tokens;
        int first;
        if (!self_tile(p, lane, tile, kTileRows, &mt, &tokens, &first, src)) return;
        self_token = nth_set_bit(tokens, first + min(n, mt.rows - 1));
    } else {
        if (tile >= *p.n_tiles) return;
        mt = p.tiles[tile];
    }
    const int n0 = (task % groups) * COLS;

    const uint16_t *W = (const uint16_t *)(kFirst ? p.w13 : p.w2) + (size_t)mt.slot * (kFirst ? 2 : 1) * (size_t)p.I * p.H;
    // two weight rows per lane: (gate, up) of one h column, or two W2 rows 16 apart
    const int ra = min(n0 + n, N - 1);
    const int rb = kFirst ? p.I + ra : min(n0 + 16 + n, N - 1);
    const uint16_t *wa = W + (size_t)ra * K, *wb = W + (size_t)rb * K;
    // token row of this lane (rows past the tile's end re-read its last row; their outputs are dropped)
    const int tr = mt.row_begin + min(n, mt.rows - 1);
    const uint16_t *xr = (const uint16_t *)(kFirst ? p.x : p.h) + (size_t)(kSelf ? self_token : kFirst ? p.perm[tr] : tr) * K;

    // this wavefront's K-chunks: [kbeg, kend)
    const int chunks = (K + 127) >> 7, per = (chunks + NS - 1) / NS;
    const int kbeg = min(ks * per, chunks) * 128, kend = min(min((ks + 1) * per, chunks) * 128, K), kstep = 128;
    f32x4 acc_a = {0.f, 0.f, 0.f, 0.f}, acc_b = {0.f, 0.f, 0.f, 0.f};
    constexpr int kAhead = kForm == kLong ? 3 : 1, D = kAhead + 1;
    Run ca[D], cb[D], cx[D];
    auto load_chunk = [&](int u, int k) {
        load_run(ca[u], wa, k, q, K);
        if (kTwo) load_run(cb[u], wb, k, q, K);
        load_run(cx[u], xr, k, q, K);
    };
#pragma unroll
    for (int u = 0; u < kAhead; ++u)
        if (u == 0 || kbeg + u * kstep < kend) load_chunk(u, kbeg + u * kstep);
    for (int k0 = kbeg; k0 < kend; k0 += D * kstep) {
#pragma unroll
        for (int u = 0; u < D; ++u) {
            const int k = k0 + u * kstep;
            if (k >= kend) break;
            if (k + kAhead * kstep < kend) load_chunk((u + kAhead) % D, k + kAhead * kstep);
            __builtin_amdgcn_sched_barrier(0);  // the prefetch must be issued before this chunk's MFMAs, not after
#pragma unroll
            for (int jj = 0; jj < 4; ++jj) {
                acc_a = __builtin_amdgcn_mfma_f32_16x16x32_bf16(*(bf16x8 *)&ca[u].v[jj], *(bf16x8 *)&cx[u].v[jj], acc_a, 0, 0, 0);
                if (kTwo) acc_b = __builtin_amdgcn_mfma_f32_16x16x32_bf16(*(bf16x8 *)&cb[u].v[jj], *(bf16x8 *)&cx[u].v[jj], acc_b, 0, 0, 0);
            }
        }
    }

    if constexpr (NS > 1) {   // the parts' sums, added in K order by the first wavefront
        __shared__ f32x4 part[NS - 1 > 0 ? NS - 1 : 1][kTwo ? 2 : 1][64];
        if (ks > 0) { part[ks - 1][0][lane] = acc_a; if (kTwo) part[ks - 1][kTwo ? 1 : 0][lane] = acc_b; }
        __syncthreads();
        if (ks > 0) return;
#pragma unroll
        for (int s = 0; s < NS - 1; ++s) {
            const f32x4 a = part[s][0][lane];
            acc_a[0] += a[0]; acc_a[1] += a[1]; acc_a[2] += a[2]; acc_a[3] += a[3];
            if (kTwo) { const f32x4 b = part[s][kTwo ? 1 : 0][lane]; acc_b[0] += b[0]; acc_b[1] += b[1]; acc_b[2] += b[2]; acc_b[3] += b[3]; }
        }
    }
    // lane holds token n, weight rows 4q..4q+3 of each of its two row blocks
    if (n >= mt.rows) return;
    uint16_t *O = (uint16_t *)(kFirst ? p.h : p.y) + (size_t)(mt.row_begin + n) * N;
    auto pack = [](float a, float b, float c, float d) {
        return make_uint2((uint32_t)f32_to_bf16(a) | ((uint32_t)f32_to_bf16(b) << 16),
                          (uint32_t)f32_to_bf16(c) | ((uint32_t)f32_to_bf16(d) << 16));
    };
    if (kFirst) {
        const int col = n0 + 4 * q;
        if (col < N) {
            float h[4];
#pragma unroll
            for (int r = 0; r < 4; ++r) h[r] = silu_mul(acc_a[r], acc_b[r]);
            *(uint2 *)(O + col) = pack(h[0], h[1], h[2], h[3]);
        }
    } else {
        const int c0 = n0 + 4 * q, c1 = n0 + 16 + 4 * q;
        if (c0 < N) *(uint2 *)(O + c0) = pack(acc_a[0], acc_a[1], acc_a[2], acc_a[3]);
        if (kTwo && c1 < N) *(uint2 *)(O + c1) = pack(acc_b[0], acc_b[1], acc_b[2], acc_b[3]);
    }
}

// GEMM-1 with its table, if it selects
template <bool kSelf, typename... Table>
void launch_first(const Pass &p, dim3 grid, dim3 block, hipStream_t st, const Table &...tab)
{
    if (p.H <= kShort1)     hipLaunchKernelGGL((k_expert_decode<true, kSelf, kShort, Table...>), grid, block, 0, st, p, tab...);
    else if (p.H <= kLong1) hipLaunchKernelGGL((k_expert_decode<true, kSelf, kMiddle, Table...>), grid, block, 0, st, p, tab...);
    else                    hipLaunchKernelGGL((k_expert_decode<true, kSelf, kLong, Table...>), grid, block, 0, st, p, tab...);
}

}  // namespace

int decode_tile_rows() { return kTileRows; }

bool gemm1_selects(const Pass &p, int blocks)
{
    return p.self_tiles && p.gate == MOE_GATE_SOFTMAX_TOPK && p.T <= kSelectTokens && p.E <= kSelectExperts && blocks <= kSelectBlocks;
}
int decode_blocks(const Pass &p) { return p.max_tiles * ((p.I + kWRows / 2 - 1) / (kWRows / 2)); }

hipError_t launch_experts_decode(const Pass &p, int which, hipStream_t st)
{
    if (which == 0) {
        const int groups = (p.I + kWRows / 2 - 1) / (kWRows / 2);
        const int blocks = p.max_tiles * groups;
        const dim3 grid(blocks + (p.self_tiles ? 1 : 0)), block(kThreads * kSplit1);
        if (p.self_select && p.host_table) launch_first<true>(p, grid, block, st, fill_table(p));
        else if (p.self_select)            launch_first<true>(p, grid, block, st, NoTable{});
        else if (p.self_tiles)             launch_first<true>(p, grid, block, st);
        else                               launch_first<false>(p, grid, block, st);
    } else {
        const int groups = (p.H + 16 * kBlocks2 - 1) / (16 * kBlocks2);
        const int blocks = p.max_tiles * groups;
        if (p.I <= kShort2) hipLaunchKernelGGL((k_expert_decode<false, false, kShort>), dim3(blocks), dim3(kThreads * kSplit2), 0, st, p);
        else                hipLaunchKernelGGL((k_expert_decode<false, false, kMiddle>), dim3(blocks), dim3(kThreads * kSplit2), 0, st, p);
    }
    return hipGetLastError();
}

}  // namespace emoe
