// Large-tile grouped SwiGLU expert GEMMs for prefill-sized groups (bf16, H and I multiples of 64).
//
// Same computation as the 4-wavefront kernels (the expert FFN of Sec. 2.1 of the
// paper over slot-grouped rows, weights addressed by slot so that a re-placement of
// experts -- Sec. 3.2 / 4.6 -- costs nothing here); what changes is the tile shape
// and the staging, chosen for three facts of this chip and this workload:
//
//  * Every expert's weights are used by only ~256 rows, so the layer streams all
//    resident weights from HBM once per pass: the kernel must keep HBM busy.  A
//    compute unit has to hold ~48 KB of weight bytes in flight to cover HBM latency
//    at full bandwidth, and whole 128-byte lines travel much faster than half lines
//    (also out of L2: a copy instruction that touches 16 half lines costs the issuing
//    wavefront twice one that touches 8 whole lines).  Both operands therefore travel
//    in steps of 64 k -- one full line per row: 32 KB of weight rows, up to 40 KB of
//    token rows per step -- through a ring each, as deep as LDS allows for the tile's
//    number of token rows (see Ring), with their own loader wavefronts.
//  * A compute unit pulls ~64 B/clk from L2 but retires 4096 bf16 flops/clk, so a
//    tile must reuse staged bytes >= 64 times: up to 320 token rows x 256 weight
//    rows gives 114-142 (a 128 x 128 tile gives exactly 64 and is bandwidth bound).
//    Measured, staged bytes are the scarce resource of this kernel: a group's weights
//    should be staged once, and token rows that do not exist not at all.
//  * Groups are ragged (tokens per expert are binomial): the tile list carries
//    chunks of <= 320 rows balanced in units of 32 (one chunk for all but the
//    largest groups), token rows that do not exist are neither staged nor multiplied:
//    above 128 rows they are staged by 8 and multiplied by 16 (all by 32 -> so, whole pass, us: Qwen3 shape 200
//    rows a slot 314.7 -> 308, 266 rows 361.7 -> 351.5; DeepSeek-V2-Lite shape 166 rows 264.7 -> 260.7; DeepSeek-V3-shaped, 32 experts,
//    264 rows 748 -> 730).  Tiles of up to 128 rows, which wait for weights, go by 32: twice as many loop bodies
//    there made 20 rows a slot 0.6 % slower.
//
// Workgroup: 8 wavefronts as 2 (token) x 4 (weight).  Wavefront (wm, wn) owns weight
// rows [wn*64, wn*64+64) and token tiles wm, wm+2, ... (interleaved so that a ragged
// tile count splits evenly): up to 4 x 10 accumulators of 16x16 = 160 registers, two
// wavefronts per SIMD so that one's LDS waits hide under the other's MFMAs.
//
// v_mfma_f32_16x16x32_bf16, not 32x32x16.  With hundreds of token rows a slot this chip runs at its power limit
// (whole passes draw 1350 to 1397 W of 1400), so that part of a kernel's time follows from the energy it spends: on zero operands, at 960 to 1120 W, GEMM-1 of the
// Qwen3 shape, 256 rows, takes 170 us instead of 206, of the DeepSeek-V3-shaped rank 478 instead of 518, of the DeepSeek-V2-Lite shape, 167 rows, 187 instead of 203.
// Per product the 16x16x32 form reads and writes half as many accumulators: a register-only stream of it on
// the layer's operands sustains 2.14 PFLOP/s at 1326 W, one of the 32x32x16 form 1.88 at 1300 W.  LDS operand
// reads per product are the same.  Whole pass of routed tokens, the same rows in every slot, us, 32x32x16 -> 16x16x32: Qwen3
// shape 64 rows 235 -> 235, 128 269.5 -> 265, 192 326 -> 304, 256 358 -> 342.5, 288 383 -> 367; DeepSeek-V2-Lite shape 162
// rows 276 -> 265; DeepSeek-V3-shaped, 32 experts, 256 rows 735 -> 680, 288 rows 800 -> 752.  The sums come out the same to the bit.
//
// Staging: global_load_lds_dwordx4 -- global memory straight into LDS, 16 bytes per
// lane, no VGPR round trip, no ds_write.  One instruction fills 1 KB: 8 rows of
// 128 bytes (token rows or weight rows); lane i lands in 16-byte slot i of the
// piece, so it FETCHES the chunk that belongs there: the XOR swizzle that keeps the
// 16-byte operand reads conflict free is applied on the global side.
//
// GEMM-1 stages 16 gate rows and then the 16 matching up rows, and so on: a lane holds
// the gate value and the up value of the same (token, column) in the same element of two
// neighbouring accumulators, so silu(g)*u needs no shuffles.
//
// Epilogue: every wavefront transposes its accumulators through a private LDS
// region (row stride = row bytes + 16: rows stay 16-byte aligned for the copy out, the
// 8-byte writes meet two to a bank) and writes whole contiguous row segments, 16 bytes
// per lane, so global stores are full cache lines.  The epilogue is instruction bound
// (3 us of a workgroup): 16-byte rather than 8-byte copies out halve its longest loop.
#include <type_traits>

#include "moe_internal.h"

namespace emoe {
namespace {

typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef float f32x4 __attribute__((ext_vector_type(4)));

constexpr int kBK = 64;                    // K-step: 128 bytes per tile row, one whole cache line, for both operands
constexpr int kThreads = 512;
constexpr int kWaves = 8;
constexpr int kBN = 256;                   // weight rows per workgroup
constexpr int kMaxTT = 10;                 // token tiles (32 rows) per workgroup
constexpr int kBM = kMaxTT * 32;           // 320: a whole group with its ragged tail in the usual case
constexpr int kBKW = 64;                   // weight K-step: 128 bytes per row = one whole cache line
constexpr int kWStage = kBN * kBKW * 2;    // 32 KB of weight rows per weight step
constexpr int kXTile = 32 * kBK * 2;       // 4 KB: a token tile's share of a K-step
constexpr int kWPieces = kWStage / 1024 / 4;   // 8: 1 KB pieces (8 rows x 128 B) per weight-loader wavefront per weight step
constexpr int kXPieces = kMaxTT * kXTile / 1024 / 4;   // 10: 1 KB pieces (8 rows x 128 B) per token-loader wavefront per K-step
constexpr int kLdsBytes = 160 * 1024;      // all of a compute unit's LDS: the rings below, then the epilogue's staging
constexpr int kXcds = 8;
constexpr int kMaxPartialSets = 256;        // partial-sum sets the workspace has room for: one round of a 256-unit chip
constexpr int kTC = kMaxTT / 2;            // token tiles per wavefront
constexpr int kWT = 4;                     // 16-row weight tiles per wavefront
// A workgroup's eight wavefronts as WM (token) x 8 / WM (weight): 2 x 4, or 4 x 2 on half an N-slice
constexpr int pieces_of(int wm) { return kWPieces * 2 / wm; }                // of weight rows per loader and step
constexpr int acc_tiles(int wm) { return 2 * ((kMaxTT + wm - 1) / wm); }     // 16-row token tiles of a wavefront
constexpr int kEpiStride1 = 2 * kWT * 8 + 16;  // GEMM-1: 32 h columns per wavefront, bytes per staged row (rows stay 16-byte aligned)
constexpr int kEpiStride2 = 2 * kWT * 16 + 16;  // GEMM-2: 64 y columns per wavefront
constexpr int kEpiBytes = 32 * kEpiStride2;     // one token tile of one wavefront
static_assert(kWaves * kEpiBytes <= kLdsBytes, "epilogue staging reuses the ring");
static_assert(kMaxTT == 10, "the dispatch on token tiles below lists 1..10");

// Everything one wavefront needs for its K loop.
struct WaveCtx {
    const uint16_t *wbase, *abase;        // slot's weight matrix, activation matrix
    uint32_t off[kXPieces > kWPieces ? kXPieces : kWPieces];               // this lane's byte offset (from the matrix base) of each piece it stages, k = 0
    uint32_t woff[kBKW / 32], xoff[kBK / 32]; // LDS byte offsets (inside a stage) of this lane's operand rows per sub-step
    int wave, lane, wm, wn, n_tt;
    bool stream_w;                        // this tile's weight rows are read by no other tile: copy them non-temporally
    int xlive;                            // token-loader wavefronts: how many of their pieces (8 rows each) are staged
};

// LDS byte address of a __shared__ object (LDS pointers are 32-bit offsets in address space 3).
__device__ __forceinline__ uint32_t lds_addr(const void *p)
{
    return (uint32_t)(uintptr_t)(__attribute__((address_space(3))) const void *)p;
}

// Direct global -> LDS copy of one 1 KB piece: lane i's 16 bytes land at m0_base + 16*i.
// The global address is a wave-uniform base (SGPR pair) plus this lane's 32-bit byte offset.
// Issued as inline assembly on purpose: the compiler's wait-count insertion would otherwise
// hold every later LDS read until these loads (which belong to a LATER stage) have returned.
// Completion is awaited explicitly (wait_loads) before the step's barrier.
// kStream: the line is marked non-temporal -- read once and not worth a place in L2.  Used for the weight
// rows of a slot whose rows are a single chunk (no other tile reads them): the weight stream then does not
// push out what is read again -- the chunk's token rows (once per N-slice), h between the two GEMMs, and the
// rows y that the combine kernel reads back right after.  A slot with several chunks keeps the default
// policy, so that the later chunks find the weights in L2.
template <bool kStream>
__device__ __forceinline__ void dma_piece(const void *base, uint32_t byte_off, uint32_t lds_byte_addr)
{
    if (kStream) asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %1, %2 nt" ::"s"(lds_byte_addr), "v"(byte_off), "s"(base) : "memory", "m0");
    else         asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %1, %2" ::"s"(lds_byte_addr), "v"(byte_off), "s"(base) : "memory", "m0");
}

// Loader roles: wavefronts 0-3 stream the weight rows (8 pieces each per K-step), wavefronts 4-7
// the token rows (up to 10 pieces each per K-step, only those whose rows exist).  The two kinds go
// out at different moments of a K-step (see k_loop), which one wavefront issuing both could not do
// without making the token copies wait for the weight copies ahead of them: a wavefront's loads
// complete in order.
template <int WM>
__device__ __forceinline__ void issue_step(const WaveCtx &c, uint32_t slot_addr, int k0)
{
    constexpr int WP = pieces_of(WM);
    if (c.wave < 4) {
        const uint16_t *b = c.wbase + k0;
        if (c.stream_w) {
#pragma unroll
            for (int i = 0; i < WP; ++i) dma_piece<true>(b, c.off[i], slot_addr + (c.wave * WP + i) * 1024);
        } else {
#pragma unroll
            for (int i = 0; i < WP; ++i) dma_piece<false>(b, c.off[i], slot_addr + (c.wave * WP + i) * 1024);
        }
    } else {
        const uint16_t *b = c.abase + k0;
#pragma unroll
        for (int i = 0; i < kXPieces; ++i)
            if (i < c.xlive) dma_piece<false>(b, c.off[i], slot_addr + ((c.wave & 3) + 4 * i) * 1024);
    }
}

// Orders this wavefront's own LDS traffic (writes before, reads after) WITHOUT waiting for its
// global stores: LDS instructions of one wavefront execute in order, so all that is needed is
// that the compiler keeps the order and that outstanding LDS operations have retired.  (A
// release/acquire fence here would also drain the vector-memory counter, i.e. stall every token
// tile of the epilogue on the round trip of the previous tile's stores.)
__device__ __forceinline__ void wave_lds_sync()
{
    asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
    __builtin_amdgcn_wave_barrier();
}

// Wait until at most n of this wavefront's loads are still in flight (they complete in order).
template <int n>
__device__ __forceinline__ void wait_loads()
{
    // s_waitcnt simm16: vmcnt = bits [3:0] and [15:14], expcnt [6:4] = 7, lgkmcnt [11:8] = 15 (no wait)
    static_assert(n < 64, "vmcnt has 6 bits");
    __builtin_amdgcn_s_waitcnt((n & 15) | ((n >> 4) << 14) | (7 << 4) | (15 << 8));
}

// One K-step (64 k) of this wavefront: NT token tiles of 16 rows x 4 weight tiles x 2 sub-steps of 32 k.  The
// (sub-step, token tile) pairs run as one software pipeline: the token operand of pair s+2 and the
// weight operands of the next sub-step are requested from LDS before the MFMAs of pair s.  Every other token tile takes
// its weight tiles backwards, so that an MFMA always has one operand of the one before it (0.6 to 1 % of the whole pass).
// `mid` is called once, half way through.
template <int NT, int WM, typename Mid>
__device__ __forceinline__ void multiply_stage(const WaveCtx &c, const char *Ws, const char *Xs, f32x4 (&acc)[kWT][acc_tiles(WM)], Mid mid)
{
    if constexpr (NT > 0) {
        constexpr int KS = kBK / 32, STEPS = KS * NT, D = 2;
        bf16x8 wf[2][kWT], xf[D + 1];
        auto fetch_w = [&](int ks) {
#pragma unroll
            for (int a = 0; a < kWT; ++a) {
                const uint4 v = *(const uint4 *)(Ws + c.woff[ks] + a * 16 * 128);
                wf[ks & 1][a] = *(const bf16x8 *)&v;
            }
        };
        auto fetch_x = [&](int step) {
            const int ks = step / NT, t = step % NT;
            const uint4 v = *(const uint4 *)(Xs + c.xoff[ks] + (t >> 1) * WM * 32 * 128 + (t & 1) * 16 * 128);
            xf[step % (D + 1)] = *(const bf16x8 *)&v;
        };
        fetch_w(0);
#pragma unroll
        for (int s0 = 0; s0 < D && s0 < STEPS; ++s0) fetch_x(s0);
#pragma unroll
        for (int step = 0; step < STEPS; ++step) {
            const int ks = step / NT, t = step % NT;
            if (step == STEPS / 2) mid();
            if (t == 0 && ks + 1 < KS) fetch_w(ks + 1);
            if (step + D < STEPS) fetch_x(step + D);
#pragma unroll
            for (int i = 0; i < kWT; ++i) {
                const int a = t & 1 ? kWT - 1 - i : i;
                acc[a][t] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(wf[ks & 1][a], xf[step % (D + 1)], acc[a][t], 0, 0, 0);
            }
            __builtin_amdgcn_sched_barrier(0);  // keep the written order: the prefetch depth is the register budget
        }
    } else {
        mid();
    }
}

// Ring geometry of a workgroup: NW stages of weight rows (32 KB each), then NX stages of TT token tiles (4 KB
// each).  What bounds this kernel is how many bytes a compute unit has on their way: a step's copies come back a
// memory latency after they were issued, so a ring that holds only the next step is a burst and a wait.  The
// fewer token tiles a workgroup has, the more weight stages fit beside them, and the shorter its multiply --
// which is what covers the wait -- so the ring is chosen by the tile's size:
//   1-2 token tiles   4 weight + 4 token stages   three steps in flight
//   3-4               3 + 4                       two
//   5-8               3 + 2                       weights two steps ahead
//   9-10              2 + 2                       one (a third weight stage does not fit)
// kMid: a weight step is issued half way through a multiply instead of at its start.  A compute unit returns
// copies in issue order and accepts about 64 KB of them before the issuing wavefronts stand still: with many
// token tiles the token copies (L2 hits, needed one step later) go first and alone, and the weight copies follow
// when those have landed.
// Measured against two stages of each for every size (whole pass, us): Qwen3 shape 333 tokens 279 -> 238, 1000
// tokens 298 -> 274, 3500 tokens 367 -> 362; DeepSeek-V3-shaped rank 512 tokens 600 -> 517, 2000 tokens
// 674 -> 597, 6500 tokens 885 -> 839; 1777 routed tokens of the DeepSeek-V2-Lite shape 367 -> 340.
template <int NW_, int NX_, int TT_, bool kMid_>
struct Ring {
    static constexpr int NW = NW_, NX = NX_, TT = TT_, XStage = TT_ * kXTile, XBase = NW_ * kWStage;
    static constexpr bool kMid = kMid_;
    static_assert((NX_ == 2 || (NX_ == 4 && TT_ <= 4)) && NW_ >= 2 && NW_ <= 4, "the waits of the K loop");
    static_assert(XBase + NX_ * XStage <= kLdsBytes, "LDS budget");
};
using Ring2 = Ring<4, 4, 2, false>;
using Ring4 = Ring<3, 4, 4, false>;
using Ring8 = Ring<3, 2, 8, true>;
using Ring10 = Ring<2, 2, kMaxTT, true>;

// K-step number i in the order this workgroup walks its KT steps: it starts at step `first` and wraps around.
__device__ __forceinline__ int step_at(int i, int first, int KT) { return i + first < KT ? i + first : i + first - KT; }

// KT K-steps of 64 of this wavefront.  The caller issued the first depth - 1 steps of the ring this wavefront loads.
template <int NT, typename R, int WM>
__device__ __forceinline__ void k_loop(const WaveCtx &c, const char *ring, int KT, int first, f32x4 (&acc)[kWT][acc_tiles(WM)])
{
    constexpr int WP = pieces_of(WM);
    const bool wloader = c.wave < 4;
    const uint32_t wring = lds_addr(ring), xring = wring + R::XBase;
    const int depth = wloader ? R::NW : R::NX;
    int ws = 0, xs = 0, fill = depth - 1;
    for (int kt = 0; kt < KT; ++kt) {
        // This wavefront's share of step kt has landed when only the copies of the younger steps (depth - 2 at most) are on their way: 8 a step
        // for a weight loader; for a token loader the 32-row tiles that exist, which with a ring of four are as many as the ring is for or
        // one fewer.  The count is an immediate of the instruction; a switch over it was slower (whole pass, us, switch -> here:
        // DeepSeek-V3-shaped, 32 experts, 264 rows 716.5 -> 710, Qwen3 shape 266 rows 348 -> 345, 128 rows 266 -> 265.4, 64 rows 235.6 -> 234.6).
        if (wloader) {
            if (kt + R::NW - 2 < KT)                  wait_loads<(R::NW - 2) * WP>();
            else if (R::NW == 4 && kt + 1 < KT)       wait_loads<WP>();
            else                                      wait_loads<0>();
        } else if (R::NX == 2 || kt + 1 >= KT) {
            wait_loads<0>();
        } else if (kt + 2 < KT) {
            if (c.xlive == R::TT) wait_loads<2 * R::TT>(); else wait_loads<2 * (R::TT - 1)>();
        } else {
            if (c.xlive == R::TT) wait_loads<R::TT>(); else wait_loads<R::TT - 1>();
        }
        __syncthreads();   // everyone's share of step kt is in LDS; everyone is done reading step kt-1
        auto issue = [&]() {
            if (kt + depth - 1 >= KT) return;
            issue_step<WM>(c, wloader ? wring + fill * kWStage : xring + fill * R::XStage, step_at(kt + depth - 1, first, KT) * kBK);
            fill = fill + 1 == depth ? 0 : fill + 1;
        };
        if (!wloader || !R::kMid) issue();
        multiply_stage<NT, WM>(c, ring + ws * kWStage, ring + R::XBase + xs * R::XStage, acc, [&]() { if (wloader && R::kMid) issue(); });
        ws = ws + 1 == R::NW ? 0 : ws + 1;
        xs = xs + 1 == R::NX ? 0 : xs + 1;
    }
}

// Partial sums of a tile whose contraction is shared out over several workgroups (the tail of a
// launch, see the kernel): floats per set, and where a wavefront's accumulator registers go.
constexpr int kPartialFloats = kWaves * kWT * 2 * kTC * 4 * 64;   // 81920 = 320 KB
__device__ __forceinline__ float *partial_at(float *set, int wave, int a, int t, int lane)
{
    return set + (((wave * kWT + a) * 2 * kTC + t) * 64 + lane) * 4;   // 16 bytes per lane, 1 KB per instruction
}

// Epilogue of one 32-row token tile of a wavefront: accumulators (both halves of token tile t of the wavefront, its kWT weight
// tiles) -> the wavefront's private LDS region [token row][column] -> coalesced rows of h (with SwiGLU) or y.
template <bool kFirst, int WM>
__device__ __forceinline__ void emit_token_tile(const Pass &p, const WaveCtx &c, const MTile &mt, int n0, int N, char *ring, int t,
                                                const f32x4 (&v)[2][kWT])
{
    constexpr int COLS = kFirst ? kWT * 8 : kWT * 16;      // output columns of this wavefront
    constexpr int STRIDE = kFirst ? kEpiStride1 : kEpiStride2;
    char *mine = ring + c.wave * kEpiBytes;
    const int l15 = c.lane & 15, quad = c.lane >> 4;
    constexpr int LPR = COLS / 8;                           // copy out: 16 bytes per lane, LPR lanes per row,
    constexpr int RPI = 64 / LPR;                           // 64/LPR rows per instruction
    static_assert(STRIDE % 16 == 0 && kEpiBytes % 16 == 0 && 32 % RPI == 0, "16-byte reads of the staged rows");
    uint16_t *O = (uint16_t *)(kFirst ? p.h : p.y);
    const int ncol0 = n0 + c.wn * COLS;
    const int lr = c.lane / LPR, lc = (c.lane % LPR) * 8;
#pragma unroll
    for (int half = 0; half < 2; ++half) {
        char *row = mine + (half * 16 + l15) * STRIDE;
#pragma unroll
        for (int a = 0; a < kWT; a += kFirst ? 2 : 1) {
            uint16_t o[4];
#pragma unroll
            for (int e = 0; e < 4; ++e) {
                float g = v[half][a][e];
                if (kFirst) g = silu_mul(g, v[half][a + (kFirst ? 1 : 0)][e]);
                o[e] = f32_to_bf16(g);
            }
            const int col = (kFirst ? a / 2 : a) * 16 + quad * 4;
            *(uint2 *)(row + col * 2) = make_uint2((uint32_t)o[0] | ((uint32_t)o[1] << 16), (uint32_t)o[2] | ((uint32_t)o[3] << 16));
        }
    }
    wave_lds_sync();
#pragma unroll
    for (int r0 = 0; r0 < 32; r0 += RPI) {
        const int rr = r0 + lr;                       // row inside the token tile
        const int m = (WM * t + c.wm) * 32 + rr;       // row inside the chunk
        const uint4 w = *(const uint4 *)(mine + rr * STRIDE + lc * 2);
        if (m < mt.rows && ncol0 + lc < N)   // N is a multiple of 64: the lane's 8 columns exist together
            *(uint4 *)(O + (size_t)(mt.row_begin + m) * N + ncol0 + lc) = w;
    }
    wave_lds_sync();  // the region is rewritten by the next token tile
}

// kPhase 0: a whole tile.  1: the partial sums of one of n_parts K ranges of a tile, left in
// p.partials (phase 2, sum_body below, adds them up).
// (Letting the last of a tile's workgroups to finish do the adding, in the same launch, was
// measured and is slower: the device-wide fence it needs costs more than the third launch.)
template <bool kFirst, int NT, int kPhase, typename R, int WM>
__device__ __forceinline__ void wave_body(const Pass &p, const WaveCtx &c, const MTile &mt, int n0, int N, int KT, int first, char *ring,
                                          float *tile_sets, int part)
{
    f32x4 acc[kWT][acc_tiles(WM)];
#pragma unroll
    for (int a = 0; a < kWT; ++a)
#pragma unroll
        for (int t = 0; t < acc_tiles(WM); ++t)
#pragma unroll
            for (int r = 0; r < 4; ++r) acc[a][t][r] = 0.f;
    k_loop<NT, R, WM>(c, ring, KT, first, acc);
    __syncthreads();  // all operand reads are done: the ring becomes the epilogue staging area
    if (kPhase == 1) {
        float *mine = tile_sets + (size_t)part * kPartialFloats;
#pragma unroll
        for (int a = 0; a < kWT; ++a)
#pragma unroll
            for (int t = 0; t < NT; ++t) *(f32x4 *)partial_at(mine, c.wave, a, t, c.lane) = acc[a][t];
        return;
    }
#pragma unroll
    for (int t = 0; t < (NT + 1) / 2; ++t) {
        f32x4 v[2][kWT];
#pragma unroll
        for (int a = 0; a < kWT; ++a) { v[0][a] = acc[a][2 * t]; v[1][a] = acc[a][2 * t + 1]; }
        emit_token_tile<kFirst, WM>(p, c, mt, n0, N, ring, t, v);
    }
}

// Phase 2: the sum of a tile's partial sums, in K order, for token tile t of this wavefront, then the
// same epilogue as a whole tile.  The sets of four parts are requested together (32 loads of 16 bytes
// per lane in flight: the launch is one round of the chip, its length is that of one workgroup) and
// added one after the other.  A 16-row half that holds no rows was not written by phase 1: what is read in its place is summed and not emitted.
template <bool kFirst>
__device__ __forceinline__ void sum_body(const Pass &p, const WaveCtx &c, const MTile &mt, int n0, int N, char *ring,
                                         float *tile_sets, int n_parts, int t)
{
    f32x4 s[2][kWT];
#pragma unroll
    for (int h = 0; h < 2; ++h)
#pragma unroll
        for (int a = 0; a < kWT; ++a) s[h][a] = (f32x4){0.f, 0.f, 0.f, 0.f};
    for (int q0 = 0; q0 < n_parts; q0 += 4) {
        f32x4 v[4][2][kWT];
#pragma unroll
        for (int u = 0; u < 4; ++u) {
            if (q0 + u >= n_parts) continue;               // uniform
            float *set = tile_sets + (size_t)(q0 + u) * kPartialFloats;
#pragma unroll
            for (int h = 0; h < 2; ++h)
#pragma unroll
                for (int a = 0; a < kWT; ++a) v[u][h][a] = *(const f32x4 *)partial_at(set, c.wave, a, 2 * t + h, c.lane);
        }
#pragma unroll
        for (int u = 0; u < 4; ++u) {
            if (q0 + u >= n_parts) continue;
#pragma unroll
            for (int h = 0; h < 2; ++h)
#pragma unroll
                for (int a = 0; a < kWT; ++a) s[h][a] += v[u][h][a];
        }
    }
    emit_token_tile<kFirst, 2>(p, c, mt, n0, N, ring, t, s);
}

// kSpread: units of more than four token tiles start spread over K (the launcher's choice, see `first`).
// kTailWM: 4 or 8 where the N-slices of a last round that fills half or a quarter of the chip run as two or four workgroups each.  An instance
// of its own: with both kinds in every launch those without such a round were 0.3 to 0.6 % slower (50 instead of 32 spilled scalars).
template <bool kFirst, int kPhase, bool kSpread = false, int kTailWM = 2>
__global__ __launch_bounds__(kThreads, 1) void k_expert_gemm_mfma8(Pass p)
{
    constexpr int kTailParts = kTailWM / 2;
    const int K = kFirst ? p.H : p.I;
    const int N = kFirst ? p.I : p.H;                  // output columns
    constexpr int BNO = kFirst ? kBN / 2 : kBN;        // output columns per workgroup

    // Work is dealt to the 8 XCDs in UNITS: a tile (chunk) of the size-ordered list with a run of its
    // N-slices.  The unit list of this GEMM was written by the bookkeeping kernel in rows of 8 -- entry
    // 8 i + x is the i-th unit of XCD x, largest tiles first on every XCD, loads equal to within one unit,
    // the tiles of one slot one behind the other on one XCD -- and workgroup ids are dealt round-robin to
    // the XCDs by the hardware, so workgroup b works for XCD b % 8 and takes that XCD's units in order,
    // the N-slices of a unit on consecutive workgroups (they share the tile's token rows in that XCD's L2).
    const UnitHdr hdr = p.unit_hdr[kFirst ? 0 : 1];
    const int spp = hdr.spp;                           // N-slices per unit

    // The tail of the launch.  Workgroups run in rounds of one per compute unit; with long
    // contractions a launch is only a few rounds deep, and a last round that fills a fraction of the
    // chip costs a whole round.  When the launch allows it (p.k_split), the workgroups of that last
    // round are run separately: each tile's contraction is shared out over n_parts workgroups
    // (phase 1, partial sums to p.partials), which a third launch adds up in K order (phase 2).  The
    // split is a function of the unit list alone, so all three launches agree on it, and of an ordered one only
    // (the launcher's choice), so that it does not follow from the slots that the experts sit in.
    const int rows_total = hdr.n_rows;                 // rows of 8 workgroups, holes at the ends of the columns included
    const int rows_round = min(p.n_cus, kMaxPartialSets) / kXcds;
    int tail_rows = 0, n_parts = 1;
    if (p.k_split && rows_total >= rows_round) {
        const int tr = rows_total % rows_round;
        int parts = tr ? rows_round / tr : 1;
        parts = min(parts, min(8, K / kBKW / 8));       // eight weight steps or more per part
        if (parts >= 2) { tail_rows = tr; n_parts = parts; }
    }
    // Where the contraction is not shared out, the last round's N-slices are: kTailParts workgroups each multiply the tile with their part
    // of the slice's weight rows, their wavefronts as kTailWM (token) x 8 / kTailWM (weight).  Whole output elements, summed as in
    // a whole slice: the same bits.  The host chooses it (parts_of) from an even load, here it is what the unit list has.
    int fine_rows = 0, sub = -1;
    if (kTailParts > 1 && !(p.k_split && rows_total >= rows_round)) {
        const int tr = rows_total % rows_round;
        if (kTailParts * tr <= rows_round) fine_rows = tr;
    }
    const int head_blocks = (rows_total - tail_rows - fine_rows) * kXcds;
    int b, part = 0;
    if (kPhase == 0) {
        b = blockIdx.x;
        if (b >= head_blocks) {
            const int r = (b - head_blocks) / kXcds;       // the parts of a slice on one XCD, one behind the other
            if (r >= kTailParts * fine_rows) return;
            sub = r % kTailParts;
            b = head_blocks + r / kTailParts * kXcds + b % kXcds;
        }
    } else if (kPhase == 1) {
        const int tail_blocks = tail_rows * kXcds;
        if (tail_blocks == 0) return;
        part = blockIdx.x / tail_blocks;
        if (part >= n_parts) return;
        b = head_blocks + blockIdx.x % tail_blocks;     // consecutive workgroups keep their XCDs (tail_blocks is a multiple of 8)
    } else {
        if ((int)blockIdx.x >= tail_rows * kXcds) return;
        b = head_blocks + blockIdx.x;
    }
    float *tile_sets = kPhase == 0 ? nullptr : p.partials + (size_t)((b - head_blocks) * n_parts) * kPartialFloats;
    const int j = b / kXcds;
    const MUnit un = p.units[kFirst ? 0 : 1][(j / spp) * kXcds + b % kXcds];
    if (un.rows == 0) return;                          // a hole at the end of this XCD's column
    MTile mt;
    mt.slot = un.slot; mt.row_begin = un.row_begin; mt.rows = un.rows; mt.single = un.info & 1;
    const int slice = (un.info >> 1) + j % spp, n0 = slice * BNO + (sub > 0 ? sub * (BNO / kTailParts) : 0);
    if (sub > 0 && n0 >= N) return;

    __shared__ __attribute__((aligned(1024))) char ring[kPhase == 2 ? kWaves * kEpiBytes : kLdsBytes];   // phase 2 only stages its epilogue
    WaveCtx c;
    c.lane = threadIdx.x & 63;
    c.wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    c.wn = sub < 0 ? c.wave & 3 : c.wave & (8 / kTailWM - 1);
    c.wm = sub < 0 ? c.wave >> 2 : c.wave / (8 / kTailWM);
    c.n_tt = (mt.rows + 31) >> 5;                      // token tiles that exist
    c.stream_w = mt.single != 0;                       // the slot's rows are one chunk: nobody else reads these weights (known from the tile itself: no further lookup before the first weight copies)
    // pieces w, w + 4, ... that hold rows; up to 128 rows all of a 32-row tile's
    c.xlive = c.wave < 4 ? 0 : c.n_tt <= 4 ? c.n_tt : (((mt.rows + 7) >> 3) - (c.wave & 3) + 3) >> 2;

    // ---- staging plan ----
    // this workgroup's K range: everything, or (phase 1) weight steps [w0, w1) of the tile
    const int wsteps = K / kBKW;
    const int w0 = kPhase == 1 ? (int)((long long)part * wsteps / n_parts) : 0;
    const int w1 = kPhase == 1 ? (int)((long long)(part + 1) * wsteps / n_parts) : wsteps;
    const uint16_t *W = (const uint16_t *)(kFirst ? p.w13 : p.w2) + (size_t)mt.slot * (kFirst ? 2 : 1) * (size_t)p.I * p.H;
    const uint16_t *A = (const uint16_t *)(kFirst ? p.x : p.h);
    c.wbase = W + w0 * kBKW;      // rows are K-contiguous: the piece offsets below are relative to the range's first k
    c.abase = A + w0 * kBKW;
    if (c.wave < 4) {
#pragma unroll
        for (int i = 0; i < kWPieces; ++i) {
            // weight piece: rows [8*pc, 8*pc+8) of the weight tile, 128 bytes each
            const int pc = c.wave * (sub < 0 ? pieces_of(2) : pieces_of(kTailWM)) + i;   // (a part of a slice: its loaders copy the first ones)
            const int row = pc * 8 + (c.lane >> 3);
            const int chunk = (c.lane & 7) ^ swz8(row);
            int g;
            if (kFirst) {
                const int tile = row >> 5, within = row & 31;
                const int col = min(n0 + tile * 16 + (within & 15), N - 1);
                g = (within < 16) ? col : p.I + col;
            } else {
                g = min(n0 + row, N - 1);
            }
            c.off[i] = ((uint32_t)g * K + chunk * 8) * 2;
        }
    } else {
#pragma unroll
        for (int i = 0; i < kXPieces; ++i) {
            // token piece: rows [8*pc, 8*pc+8) of the token tile, 128 bytes each (rows past the chunk re-read its last row)
            const int pc = (c.wave & 3) + 4 * i;   // interleaved over the 4 loaders so that live pieces are shared evenly
            const int row = pc * 8 + (c.lane >> 3);
            const int chunk = (c.lane & 7) ^ swz8(row);
            const int r = min(row, mt.rows - 1);
            const int sr = kFirst ? p.perm[mt.row_begin + r] : mt.row_begin + r;
            c.off[i] = ((uint32_t)sr * K + chunk * 8) * 2;
        }
    }
    {   // operand rows of this lane: weight row wn*64 + l15 (+16a), token row wm*32 + l15 (+64 per 32-row token tile, +16 for its second half)
        const int l15 = c.lane & 15, quad = c.lane >> 4;
        const int wr = c.wn * kWT * 16 + l15, xr = c.wm * 32 + l15;
#pragma unroll
        for (int ks = 0; ks < kBKW / 32; ++ks) c.woff[ks] = wr * 128 + (((ks * 4 + quad) ^ swz8(wr)) << 4);
#pragma unroll
        for (int ks = 0; ks < kBK / 32; ++ks) c.xoff[ks] = xr * 128 + (((ks * 4 + quad) ^ swz8(xr)) << 4);
    }

    const int KT = w1 - w0;
    // All workgroups of a launch walk K at the same pace, 128 bytes of rows that lie a row length apart: started at the
    // same K-step they ask the same few memory channels at a time (a row length of 4096 bytes is the worst case, and
    // how bad it gets then changes with where the pool lies).  So they start spread over K.
    // Tiles with few token rows: every N-slice at its own step.  Qwen3 shape (rows of 4096 bytes) 333 tokens 236 .. 254 -> 228 us,
    // 1000 tokens 263 .. 281 -> 251 us; rows of 14336 bytes +-0.
    // Tiles with many: their rows are shared through L2 by slices at the same step, so a unit's slices start together and the units are
    // spread by their place in the list (kSpread: launch_experts_mfma8), 5 steps from one to the next (1 and 3: the same within 1 %).
    // Not the chunks of one slot, which share its weights the same way.
    const int first = kPhase != 0 ? 0 : c.n_tt <= 4 ? slice * KT / p.n_slices[kFirst ? 0 : 1] : kSpread && mt.single ? ((j / spp) * kXcds + b % kXcds) * 5 % KT : 0;
    // 32-row token tiles this wavefront multiplies: wm, wm+2, ... < n_tt.  The whole rest of the
    // wavefront's work is specialised on their number, above 128 rows on that of their 16-row halves, so that its K loop is straight-line code.
    const int ntc = sub < 0 ? (c.n_tt - c.wm + 1) >> 1 : (c.n_tt - c.wm + kTailWM - 1) / kTailWM;
    if constexpr (kPhase == 2) {
        // phase 2 is spread over the token tiles too: a workgroup adds up one per wavefront
        if ((int)blockIdx.y < ntc) sum_body<kFirst>(p, c, mt, n0, N, ring, tile_sets, n_parts, (int)blockIdx.y);
    } else {
        auto run_on = [&](auto geometry, auto tiles, auto wm) __attribute__((always_inline)) {
            using R = decltype(geometry);
            constexpr int WM = decltype(wm)::value;
            const uint32_t wring = lds_addr(ring), xring = wring + R::XBase;
            const int depth = c.wave < 4 ? R::NW : R::NX;
            for (int s = 0; s < depth - 1 && s < KT; ++s) issue_step<WM>(c, c.wave < 4 ? wring + s * kWStage : xring + s * R::XStage, step_at(s, first, KT) * kBK);
            wave_body<kFirst, decltype(tiles)::value, kPhase, R, WM>(p, c, mt, n0, N, KT, first, ring, tile_sets, part);
        };
        using std::integral_constant;
        auto run = [&](auto geometry, auto tiles) __attribute__((always_inline)) { run_on(geometry, tiles, integral_constant<int, 2>{}); };
        if constexpr (kTailParts > 1) {
            if (sub >= 0) {
                // whole 32-row tiles: `most` of them where a wavefront has that many, else one fewer
                auto pick2 = [&](auto geometry, auto most) __attribute__((always_inline)) {
                    constexpr int m = decltype(most)::value;
                    if (ntc >= m) run_on(geometry, integral_constant<int, 2 * m>{}, integral_constant<int, kTailWM>{});
                    else          run_on(geometry, integral_constant<int, 2 * m - 2>{}, integral_constant<int, kTailWM>{}); };
                if (c.n_tt <= 2)      pick2(Ring2{}, integral_constant<int, 1>{});
                else if (c.n_tt <= 4) pick2(Ring4{}, integral_constant<int, 1>{});
                else if (c.n_tt <= 8) pick2(Ring8{}, integral_constant<int, (8 + kTailWM - 1) / kTailWM>{});
                else                  pick2(Ring10{}, integral_constant<int, (kMaxTT + kTailWM - 1) / kTailWM>{});
                return;
            }
        }
        // the body for nt, n .. most: the numbers of 16-row token tiles that a wavefront of this geometry can have
        auto pick = [&](auto self, auto geometry, auto n, auto most, int nt) __attribute__((always_inline)) {
            constexpr int v = decltype(n)::value;
            if constexpr (v == decltype(most)::value) run(geometry, n);
            else if (nt == v) run(geometry, n);
            else self(self, geometry, integral_constant<int, v + 1>{}, most, nt);
        };
        if (c.n_tt <= 2)      { if (ntc == 1) run(Ring2{}, integral_constant<int, 2>{}); else run(Ring2{}, integral_constant<int, 0>{}); return; }
        if (c.n_tt <= 4)      { if (ntc == 2) run(Ring4{}, integral_constant<int, 4>{}); else run(Ring4{}, integral_constant<int, 2>{}); return; }
        // the last 32-row tile's owner leaves its second half out when it has no rows
        const int nt = __builtin_amdgcn_readfirstlane(2 * ntc - (((mt.rows + 15) >> 4) & ((c.n_tt - 1) == 2 * (ntc - 1) + c.wm)));
        if (c.n_tt <= 8)      pick(pick, Ring8{}, integral_constant<int, 4>{}, integral_constant<int, 8>{}, nt);
        else                  pick(pick, Ring10{}, integral_constant<int, 8>{}, integral_constant<int, 10>{}, nt);
    }
}

// Into how many workgroups the N-slices of a last round that is not full are to be split (1, 2 or 4), from the tiles of an even load; rows of 8
// workgroups, `round` of them run at a time.  A launch takes as long as its fullest compute unit: 1.5 rounds cost what two do,
// and 48 workgroups, a fifth of the chip, what a whole round does.  A part of a slice reads all of the tile's token rows for fewer weight rows, so that it
// takes more than its share of the time (rows + 128 or rows + 64 of rows + 256): worth it where there are compute units left over.
// us a pass, whole slices -> in two -> in four.  Under one round: 8 Qwen3 experts, 1000 tokens 67.8 -> 55.3 -> 49.0, 10, 3000 97.0 -> 82.3 -> 78.1,
// 16, 3000 98.6 -> 86.0 (too many for four), 32, 3000 tokens, 192 workgroups: whole.  More than one: 48, 1500 142.3 -> 132.1 -> 128.6, 3000 170.0 -> 160.9 -> 156.2, 64, 4096
// 208 -> 205; DeepSeek-V2-Lite shape, 1777 tokens 332.9 -> 328.4 -> 328.4, 16 experts, 1000 127.1 -> 118.2 -> 112.8; DeepSeek-V3-shaped, 16 experts, 6000 505 -> 496 -> 493.
//  * In four up to 224 rows a tile: above, the token rows that are read four times tell (DeepSeek-V2-Lite shape, 281 rows 294.7 -> 289.3 -> 294.8, DeepSeek-V3-shaped, 250
//    588 -> 579 -> 584; Qwen3 shape, 231 rows, 10 experts 96.8 -> 79.2 -> 82.3; 281 rows 208.7 -> 198.1 -> 200.5, though on 10 experts 119 -> 104 -> 100).
//  * Slots with several tiles, whose weights are read out of L2 as it is, only under one round (Qwen3 shape, 6000 tokens, 8 experts 103.4 -> 93.6, 4 101.3 -> 86.8;
//    32 experts, 1.5 rounds, 189.4 -> 195.4).
//  * A long contraction of more than a round is shared out instead (k_split).  Under one round it cannot be (DeepSeek-V3-shaped, 4 experts, 4000 tokens 240 -> 201).
int parts_of(const Pass &p, int n_slices, int round)
{
    if (p.tiles_expected <= 0) return 1;
    const int runs = mfma8_runs(p.tiles_expected, n_slices);
    const int rows = (p.tiles_expected * runs + kXcds - 1) / kXcds * (n_slices / runs), tail = rows % round;
    if (tail == 0 || 2 * tail > round || (rows >= round && (p.k_split || p.slot_tiles_expected > 1))) return 1;
    return 4 * tail > round || p.tile_rows_expected > 224 ? 2 : 4;
}

template <bool kFirst, int kTailWM>
void launch_phase0(const Pass &p, bool spread, int grid, hipStream_t st)
{
    if (spread) hipLaunchKernelGGL((k_expert_gemm_mfma8<kFirst, 0, true, kTailWM>), dim3(grid), dim3(kThreads), 0, st, p);
    else        hipLaunchKernelGGL((k_expert_gemm_mfma8<kFirst, 0, false, kTailWM>), dim3(grid), dim3(kThreads), 0, st, p);
}
void launch_whole(const Pass &p, bool first, int parts, bool spread, int grid, hipStream_t st)
{
    if (first) parts == 1 ? launch_phase0<true, 2>(p, spread, grid, st) : parts == 2 ? launch_phase0<true, 4>(p, spread, grid, st) : launch_phase0<true, 8>(p, spread, grid, st);
    else       parts == 1 ? launch_phase0<false, 2>(p, spread, grid, st) : parts == 2 ? launch_phase0<false, 4>(p, spread, grid, st) : launch_phase0<false, 8>(p, spread, grid, st);
}

}  // namespace

int mfma8_tile_rows() { return kBM; }

// usable when both contraction lengths are whole K-steps (direct-to-LDS loads cannot zero fill)
// Whole K-steps only (the copies cannot zero fill), and the copies address their rows with 32-bit byte
// offsets from the matrix base: x by token index, h by grouped row, a slot's weights by weight row.
bool mfma8_supports(const Pass &p)
{
    const size_t lim = (size_t)1 << 32;
    return p.act_bf16 && p.H % kBKW == 0 && p.I % kBKW == 0 &&
           (size_t)p.T * p.H * 2 < lim && (size_t)p.T * p.kk * p.I * 2 < lim && (size_t)2 * p.I * p.H * 2 < lim;
}

size_t mfma8_partial_bytes() { return (size_t)kMaxPartialSets * kPartialFloats * sizeof(float); }

int mfma8_n_slices(int H, int I, int which) { return which == 0 ? (I + kBN / 2 - 1) / (kBN / 2) : (H + kBN - 1) / kBN; }

// Rows of 8 workgroups a launch provides (and unit rows x N-slices per unit its unit list has room for):
// every tile's N-slices, dealt evenly (rounded up to whole units), plus kUnitSlack units per column for columns
// of unequal length when the tiles of a slot are kept on one XCD.
int mfma8_grid_rows(int max_tiles, int n_slices) { return (max_tiles * n_slices + kXcds - 1) / kXcds + (kUnitSlack + 1) * n_slices; }

hipError_t launch_experts_mfma8(const Pass &p0, int which, hipStream_t st)
{
    // compute units of the CURRENT device (looked up once per device: a process may drive several)
    static int cus_of[64] = {};
    int dev = 0;
    hipError_t e = hipGetDevice(&dev);
    if (e != hipSuccess) return e;
    int cus = dev >= 0 && dev < 64 ? cus_of[dev] : 0;
    if (cus == 0) {
        int n = 0;
        e = hipDeviceGetAttribute(&n, hipDeviceAttributeMultiprocessorCount, dev);
        if (e != hipSuccess) return e;
        cus = n >= kXcds ? n : kXcds;
        if (dev >= 0 && dev < 64) cus_of[dev] = cus;
    }
    Pass p = p0;
    p.n_cus = cus;
    // sharing out the contraction of the last round's tiles pays when a tile is long: 64 weight steps or more
    const int K = which == 0 ? p.H : p.I;
    // a list in slot order would let the slots decide which tiles fall into the last round, and with that how their rows are summed
    // (300 tiles in 1800 slots, rows of 4096, split -> not: 64 wide, 300 workgroups, 552 -> 555 us the whole pass; 192 wide 764 -> 757)
    p.k_split = p.partials != nullptr && K / kBKW >= 64 && tile_list_sorted(p);
    if (!p.units[0] || !p.unit_hdr) return hipErrorInvalidValue;   // the bookkeeping kernel must have been asked for unit lists
    const int nt = p.n_slices[which];
    int grid = mfma8_grid_rows(p.max_tiles, nt) * kXcds;      // and the parts of a last round's slices
    const int round_blocks = (cus < kMaxPartialSets ? cus : kMaxPartialSets) / kXcds * kXcds;
    // K starts of many-row units spread over K (see the kernel): where rows are a multiple of 4096 bytes, and the order of the tile
    // list does not follow from the slots the experts sit in -- a row's sum would.
    // us, together -> spread: GEMM-1, rows of 4096 bytes, Qwen3 shape 1700 tokens 141 -> 142, 2500 tokens 165 -> 158, 4096 tokens
    // 198 -> 198, 2500 tokens on 64 of its experts 112 -> 90, Zipf(1.2) 180 -> 180; DeepSeek-V2-Lite shape without shared rows 1777 tokens
    // 185 -> 160; rows of 8192 and 12288 bytes, 32 experts, 1500 tokens 130 -> 107 and 338 -> 324, of 6144 153 -> 154; GEMM-2, rows of
    // 4096 bytes, DeepSeek-V3-shaped rank 5000 tokens 262 -> 224, 8192 tokens 292 -> 280; of 8192 237 -> 235.
    // A shared expert with several chunks reads the same token rows as everybody: DeepSeek-V2-Lite shape with the whole batch,
    // GEMM-1 of 1000 tokens 166 -> 168, 1777 tokens 194.5 -> 198.6, 3000 tokens 270 -> 259.  There the starts stay together.
    const bool spread = K % 2048 == 0 && tile_list_sorted(p) && !(which == 0 && p.shared_end - p.shared_begin > kBM);
    const int parts = parts_of(p, nt, round_blocks / kXcds);
    if (parts > 1) grid += (parts - 1) * (round_blocks / kXcds / parts) * kXcds;
    launch_whole(p, which == 0, parts, spread, grid, st);
    if (p.k_split) {
        if (which == 0) {
            hipLaunchKernelGGL((k_expert_gemm_mfma8<true, 1>), dim3(round_blocks), dim3(kThreads), 0, st, p);
            hipLaunchKernelGGL((k_expert_gemm_mfma8<true, 2>), dim3(round_blocks / 2, kTC), dim3(kThreads), 0, st, p);
        } else {
            hipLaunchKernelGGL((k_expert_gemm_mfma8<false, 1>), dim3(round_blocks), dim3(kThreads), 0, st, p);
            hipLaunchKernelGGL((k_expert_gemm_mfma8<false, 2>), dim3(round_blocks / 2, kTC), dim3(kThreads), 0, st, p);
        }
    }
    return hipGetLastError();
}

}  // namespace emoe
