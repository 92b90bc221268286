// Gate logits for prefill-sized batches, staged by direct global -> LDS copies.
//
// logits[t, e] = sum_h x[t, h] * Wr[e, h] (+ logit_bias[e]) in fp32 -- step 1 of the gate of the
// layer of Sec. 2.1 of the paper; scores and the top-k selection follow in k_gate_select.
//
// The contraction is small (2*T*H*E flops); what costs is moving its operands into the compute
// units: a workgroup owns a tile of tokens x experts and walks K in steps of 64 through LDS rings
// filled by global_load_lds_dwordx4 (no register round trip), waiting only for the oldest step
// in flight.  The NW wavefronts form a WM x (NW/WM) grid: wavefront (wt, we) multiplies token
// tiles wt*TBT .. +TBT-1 (16 tokens each) with expert tiles we*EBT .. +EBT-1 (16 experts each),
// v_mfma_f32_16x16x32_bf16.
//
// * The bytes a workgroup pulls are (tokens + experts of its tile) * H: large tiles (up to 128
//   tokens x 256 experts) cut them, and the contraction is then split over gridDim.z workgroups
//   so that the chip stays full.  Split z writes its partial sums to plane z of the logits
//   buffer; the selection kernel adds the planes in order.
// * Issuing a copy instruction costs a wavefront on the order of a hundred cycles, during which
//   it multiplies nothing: the large tiles run on 8 wavefronts (two per SIMD, one issuing while
//   the other multiplies).
// * Accumulators go out through LDS as whole row segments (stored from registers, every
//   instruction would touch 16 rows of the plane, 64 bytes each: a third of the kernel's time).
//
// Rows are 128 bytes (bf16) or 256 bytes (fp32 router) with their 16-byte chunks XOR-swizzled on
// the global side of the copy, so that the 16 rows a quarter-wavefront reads for one operand fall
// into 16 distinct bank groups.  An fp32 router row is split when it is READ from LDS into three
// bf16 planes hi + mid + lo (each the truncated top 8 mantissa bits of what is left: the split is
// exact), so that x . w is three bf16 MFMAs whose products are all exact and whose sum is
// accumulated in fp32 -- the same products and the same accumulator width as an fp32 chain.
#include "moe_internal.h"

namespace emoe {
namespace {

typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef float f32x4 __attribute__((ext_vector_type(4)));

constexpr int kBK = 64;   // K-step
constexpr int kChain = 8;   // K-steps that are added up in the matrix cores' accumulators before they go to a sum

__device__ __forceinline__ uint32_t lds_addr(const void *p)
{
    return (uint32_t)(uintptr_t)(__attribute__((address_space(3))) const void *)p;
}

// global -> LDS copy of one 1 KB piece: lane i's 16 bytes land at lds_byte_addr + 16*i.  Inline
// assembly on purpose: the compiler's wait-count insertion would otherwise hold every later LDS
// read until these copies (which belong to a LATER K-step) have landed.
__device__ __forceinline__ void dma_piece(const void *base, uint32_t byte_off, uint32_t lds_byte_addr)
{
    asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %1, %2" ::"s"(lds_byte_addr), "v"(byte_off), "s"(base) : "memory", "m0");
}

template <int n>
__device__ __forceinline__ void wait_loads()
{
    static_assert(n >= 0 && n < 64, "vmcnt has 6 bits");
    __builtin_amdgcn_s_waitcnt((n & 15) | ((n >> 4) << 14) | (7 << 4) | (15 << 8));   // vmcnt only
}

// exact split of 8 fp32 values (two 16-byte loads) into three bf16 planes
__device__ __forceinline__ void split3(const uint4 &lo4, const uint4 &hi4, bf16x8 &ph, bf16x8 &pm, bf16x8 &pl)
{
    const uint32_t f[8] = {lo4.x, lo4.y, lo4.z, lo4.w, hi4.x, hi4.y, hi4.z, hi4.w};
    uint32_t h[8], m[8], l[8];
#pragma unroll
    for (int e = 0; e < 8; ++e) {
        h[e] = f[e] & 0xffff0000u;
        const float r1 = __uint_as_float(f[e]) - __uint_as_float(h[e]);
        m[e] = __float_as_uint(r1) & 0xffff0000u;
        const float r2 = r1 - __uint_as_float(m[e]);
        l[e] = __float_as_uint(r2) & 0xffff0000u;   // at most 8 significant bits are left: already a bf16 value
    }
    auto pack = [](const uint32_t *v) {
        const uint4 u = make_uint4((v[0] >> 16) | v[1], (v[2] >> 16) | v[3], (v[4] >> 16) | v[5], (v[6] >> 16) | v[7]);
        return *(const bf16x8 *)&u;
    };
    ph = pack(h); pm = pack(m); pl = pack(l);
}

// One ring of NS stages, a stage = the step's token rows + router rows.  Every wavefront copies its share of both, so one count, an immediate of
// the instruction, says that a step has landed.  Copies complete in order: a deeper ring for the token rows alone (each read once, from HBM; the router rows
// come from L2) keeps no more of them on their way, unless half of the wavefronts copy token rows and half router rows.  In the largest tilings (three
// stages of 48 KB) neither pays: gate phase, us, this -> four token stages, all wavefronts copying both -> four token stages, separate loaders:
// DeepSeek-V3-shaped rank 8192 tokens 69.5 -> 70.0 -> 70.0, with 16 experts 67.0 -> 68.7 -> 69.0, 2500 tokens 37.2 -> 37.2 -> 37.4; Qwen3 shape 4096 tokens
// 25.4 -> 25.6 -> 25.5; an fp32 router of 256 experts on rows of 7168, 4096 tokens 62.3 -> 63.9 -> 63.1.
template <typename WT, int TBT, int EBT, int NS, int NW, int WM>
__global__ __launch_bounds__(NW * 64) void k_gate_logits_dma(Pass p)
{
    constexpr bool F32 = sizeof(WT) == 4;
    constexpr int kWaves = NW, WE = NW / WM;
    constexpr int TB = 16 * TBT * WM, EB = 16 * EBT * WE;
    constexpr int XBYTES = TB * 128, WROW = F32 ? 256 : 128, WBYTES = EB * WROW, STAGE = XBYTES + WBYTES;
    constexpr int XP = XBYTES / 1024, WP = WBYTES / 1024;   // 1 KB pieces: 8 rows of 128 B, or 4 rows of 256 B
    constexpr int PW = (XP + WP) / kWaves;                  // pieces per wavefront per K-step
    static_assert((XP + WP) % kWaves == 0, "pieces are dealt evenly to the wavefronts");
    static_assert(NS >= 2 && (NS - 2) * PW < 64, "load counter");
    constexpr int LDS = NS * STAGE;
    static_assert(LDS <= 160 * 1024, "the ring fits LDS");
    __shared__ __attribute__((aligned(1024))) char ring[LDS];   // a stage: token rows, then router rows

    const int E = p.E, H = p.H;
    const int lane = threadIdx.x & 63;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int wt = wave / WE, we = wave % WE;
    const int t0 = blockIdx.x * TB, e0 = blockIdx.y * EB;
    // this workgroup's share of the K-steps
    const int kt0 = (int)((long long)blockIdx.z * (H / kBK) / gridDim.z), kt1 = (int)((long long)(blockIdx.z + 1) * (H / kBK) / gridDim.z);
    const char *xbase = (const char *)p.x;
    const char *wbase = (const char *)p.router_w;

    // ---- this lane's share of every K-step: its pieces, their global byte offsets at k = 0 ----
    uint32_t src[PW];
    uint32_t dst[PW];   // wave-uniform LDS offset of the piece inside its stage
    bool isx[PW];
#pragma unroll
    for (int i = 0; i < PW; ++i) {
        // piece wave + NW i of a step's XP pieces of token rows and WP of router rows
        int pc = wave + kWaves * i;
        isx[i] = pc < XP;
        if (!isx[i]) pc -= XP;
        if (isx[i]) {
            const int row = pc * 8 + (lane >> 3);
            const int chunk = (lane & 7) ^ ((row >> 1) & 7);
            src[i] = (uint32_t)min(t0 + row, p.T - 1) * (uint32_t)H * 2u + chunk * 16;
        } else if (!F32) {
            const int row = pc * 8 + (lane >> 3);
            const int chunk = (lane & 7) ^ ((row >> 1) & 7);
            src[i] = (uint32_t)min(e0 + row, E - 1) * (uint32_t)H * 2u + chunk * 16;
        } else {
            const int row = pc * 4 + (lane >> 4);
            const int chunk = (lane & 15) ^ (row & 15);
            src[i] = (uint32_t)min(e0 + row, E - 1) * (uint32_t)H * 4u + chunk * 16;
        }
        dst[i] = pc * 1024;
    }
    const uint32_t ring_a = lds_addr(ring);
    // this wavefront's copies for K-step kt into stage `slot`
    auto issue = [&](int kt, int slot) {
#pragma unroll
        for (int i = 0; i < PW; ++i) {
            const char *b = isx[i] ? xbase + (size_t)kt * (kBK * 2) : wbase + (size_t)kt * (kBK * (F32 ? 4 : 2));
            dma_piece(b, src[i], ring_a + slot * STAGE + (isx[i] ? 0 : XBYTES) + __builtin_amdgcn_readfirstlane(dst[i]));
        }
    };

    // ---- operand reads: lane (n = l % 16, q = l / 16) holds k = 8q .. 8q+7 of row n of a 16-row tile ----
    const int n = lane & 15, q = lane >> 4;
    uint32_t xoff[2], woff[2][F32 ? 2 : 1];
#pragma unroll
    for (int ks = 0; ks < 2; ++ks) {
        const int ch = ks * 4 + q;
        xoff[ks] = n * 128 + ((ch ^ ((n >> 1) & 7)) << 4);
        if (F32) {
            woff[ks][0] = n * 256 + (((2 * ch) ^ n) << 4);
            woff[ks][F32 ? 1 : 0] = n * 256 + (((2 * ch + 1) ^ n) << 4);
        } else {
            woff[ks][0] = xoff[ks];
        }
    }

    // sum: what every kChain K-steps leave, so that a logit's error does not grow with the K-steps of a split
    f32x4 acc[EBT][TBT], sum[EBT][TBT];
#pragma unroll
    for (int a = 0; a < EBT; ++a)
#pragma unroll
        for (int tb = 0; tb < TBT; ++tb) acc[a][tb] = sum[a][tb] = (f32x4){0.f, 0.f, 0.f, 0.f};
    auto flush = [&]() {
#pragma unroll
        for (int a = 0; a < EBT; ++a)
#pragma unroll
            for (int tb = 0; tb < TBT; ++tb) { sum[a][tb] += acc[a][tb]; acc[a][tb] = (f32x4){0.f, 0.f, 0.f, 0.f}; }
    };

    auto multiply = [&](int slot) {
        const char *X = ring + slot * STAGE + wt * TBT * 16 * 128;
        const char *W = ring + slot * STAGE + XBYTES + we * EBT * 16 * WROW;
#pragma unroll
        for (int ks = 0; ks < 2; ++ks) {
            bf16x8 xf[TBT];
#pragma unroll
            for (int tb = 0; tb < TBT; ++tb) {
                const uint4 v = *(const uint4 *)(X + xoff[ks] + tb * 16 * 128);
                xf[tb] = *(const bf16x8 *)&v;
            }
#pragma unroll
            for (int a = 0; a < EBT; ++a) {
                if constexpr (F32) {
                    const uint4 v0 = *(const uint4 *)(W + woff[ks][0] + a * 16 * WROW);
                    const uint4 v1 = *(const uint4 *)(W + woff[ks][1] + a * 16 * WROW);
                    bf16x8 ph, pm, pl;
                    split3(v0, v1, ph, pm, pl);
#pragma unroll
                    for (int tb = 0; tb < TBT; ++tb) {
                        acc[a][tb] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(ph, xf[tb], acc[a][tb], 0, 0, 0);
                        acc[a][tb] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(pm, xf[tb], acc[a][tb], 0, 0, 0);
                        acc[a][tb] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(pl, xf[tb], acc[a][tb], 0, 0, 0);
                    }
                } else {
                    const uint4 v = *(const uint4 *)(W + woff[ks][0] + a * 16 * WROW);
                    const bf16x8 wf = *(const bf16x8 *)&v;
#pragma unroll
                    for (int tb = 0; tb < TBT; ++tb)
                        acc[a][tb] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(wf, xf[tb], acc[a][tb], 0, 0, 0);
                }
            }
        }
    };

    // ---- K loop: steps kt+1 .. kt+NS-1 are in flight while step kt is multiplied ----
    for (int s = 0; s < NS - 1 && kt0 + s < kt1; ++s) issue(kt0 + s, s);
    int slot = 0, fill = NS - 1;
    for (int kt = kt0; kt < kt1;) {
        const int end = min(kt + kChain, kt1);
        for (; kt < end; ++kt) {
            // Behind step kt's copies those of NS - 2 steps were issued and may stay on their way; the last steps wait for all.  (Counted down
            // exactly, by a switch over the immediates of the instruction, it was slower.)
            if (kt + NS - 2 < kt1) wait_loads<(NS - 2) * PW>();
            else                   wait_loads<0>();
            __syncthreads();   // everyone's pieces of step kt have landed; everyone is done reading step kt-1
            if (kt + NS - 1 < kt1) issue(kt + NS - 1, fill);
            multiply(slot);
            slot = slot + 1 == NS ? 0 : slot + 1;
            fill = fill + 1 == NS ? 0 : fill + 1;
        }
        flush();
    }

    // ---- epilogue: accumulators -> this wavefront's LDS region [token][expert] -> whole row segments ----
    // A lane holds token n of each token tile and experts 4q .. 4q+3 of each of its expert tiles:
    // stored straight from registers every instruction would touch 16 rows, 64 bytes each.
    __syncthreads();   // all operand reads are done: the ring becomes the staging area
    float *plane = p.logits + (size_t)blockIdx.z * p.T * E;
    const float *bias = blockIdx.z == 0 ? p.logit_bias : nullptr;   // added once
    constexpr int COLS = EBT * 16, STRIDE = COLS + 4;   // floats; +4 keeps the 16 rows of a store apart on the banks
    static_assert(NW * TBT * 16 * STRIDE * 4 <= LDS, "staging fits the ring");
    float *stg = (float *)ring + wave * (TBT * 16 * STRIDE);
#pragma unroll
    for (int a = 0; a < EBT; ++a)
#pragma unroll
        for (int tb = 0; tb < TBT; ++tb)
            *(f32x4 *)(stg + (tb * 16 + n) * STRIDE + a * 16 + 4 * q) = sum[a][tb];
    asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
    __builtin_amdgcn_wave_barrier();
    constexpr int LPR = COLS / 4, RPI = 64 / LPR;        // lanes per row, rows per instruction
    const int lr = lane / LPR, lc = (lane % LPR) * 4;
    const int ecol = e0 + we * COLS + lc;
    f32x4 bv = {0.f, 0.f, 0.f, 0.f};
    if (bias) {
#pragma unroll
        for (int r = 0; r < 4; ++r) bv[r] = ecol + r < E ? bias[ecol + r] : 0.f;
    }
    const bool vec = (E & 3) == 0;                        // rows of the plane are 16-byte aligned
#pragma unroll
    for (int r0 = 0; r0 < TBT * 16; r0 += RPI) {
        const int row = r0 + lr;
        const int t = t0 + wt * TBT * 16 + row;
        f32x4 v = *(const f32x4 *)(stg + row * STRIDE + lc);
        v += bv;
        if (t < p.T) {
            float *dst = plane + (size_t)t * E + ecol;
            if (vec && ecol + 3 < E) {
                *(f32x4 *)dst = v;
            } else {
#pragma unroll
                for (int r = 0; r < 4; ++r)
                    if (ecol + r < E) dst[r] = v[r];
            }
        }
    }
}

template <typename WT, int TBT, int EBT, int NS, int NW, int WM>
hipError_t launch_t(const Pass &p, int planes, hipStream_t st)
{
    constexpr int TB = 16 * TBT * WM, EB = 16 * EBT * (NW / WM);
    dim3 grid((p.T + TB - 1) / TB, (p.E + EB - 1) / EB, planes);
    hipLaunchKernelGGL((k_gate_logits_dma<WT, TBT, EBT, NS, NW, WM>), grid, dim3(NW * 64), 0, st, p);
    return hipGetLastError();
}

// The tilings: tokens x experts of a workgroup, and the us that one of its K-steps takes (bf16, fp32 router), measured on 150 to 8000 tokens of 64, 128 and 256
// experts on rows of 2048 and 7168.  Two workgroups of the first one with a bf16 router have their LDS on a compute unit (72 KB each; of all others one): alone one takes 0.16 us a step, two
// together 0.30.  Its 0.21 stands for both, and a launch of it that is counted as two rounds is in truth one of pairs.
struct Tiling { int tokens, experts[2]; float step[2]; };
constexpr Tiling kTilings[3] = {{32, {64, 64}, {0.21f, 0.45f}}, {64, {128, 128}, {0.38f, 0.8f}}, {128, {256, 128}, {0.95f, 1.1f}}};
constexpr int kChipUnits = 256;                            // the step times are of a whole chip; on a part of one only the choice would be another
constexpr float kTileUs = 0.5f, kPlaneBytesPerUs = 6e6f;   // a workgroup's start and end; the planes' way out and back

}  // namespace

// whole K-steps only (the copies cannot zero fill), and 32-bit byte offsets into x and the router
bool gate_dma_supports(const Pass &p)
{
    return p.act_bf16 && p.H % kBK == 0 && p.H >= kBK && (size_t)p.T * p.H * 2 < ((size_t)1 << 32) && (size_t)p.E * p.H * 4 < ((size_t)1 << 32);
}

// Writes *planes partial-sum planes [T,E] to p.logits.
hipError_t launch_gate_logits_dma(const Pass &p, int *planes, hipStream_t st)
{
    // The tiling and the K split (at most kGatePlanes, at least 4 K-steps each) with the shortest time by that measure: rounds of the chip's compute units, each with one workgroup, times
    // K-steps, and what the planes cost.  What matters is that a launch is one round: the largest tiling that filled the chip, split into ceil(256 / tiles), was
    // a little more than one round nearly everywhere.  Gate phase, us, that -> this: 128 experts on rows of 2048 (fp32 router) 333 tokens 15.3 -> 13.7, 1100 21.1 -> 17.2, 2200 28.8 -> 18.7,
    // 3000 28.7 -> 20.2, 6000 37.4 -> 29.1, where it was one round 4096 22.0 -> 22.0; 256 on rows of 7168 (bf16) 512 tokens 20.3 -> 20.3, 700 28.0 -> 22.5, 2500 37.1 -> 29.7,
    // 5000 62.4 -> 45.0, 8000 81.2 -> 61.4; 64 on rows of 2048 2500 20.4 -> 16.7.  The best of all (tiling, split) pairs is 0.3 % faster on average over 47 such sizes,
    // and 0.7 % over 168: 130 to 8000 tokens of 14 routers, 60 to 512 experts on rows of 1024 to 7168 (at worst 11 %, 128 experts on rows of 2048, bf16, 2200 tokens 17.6 us -> 15.9).  Counting the pairs above
    // (0.16, 0.30) comes to 0.6 %, six of seven changed choices 1 to 10 % faster, but 384 experts on rows of 7168, 333 tokens 23.3 -> 25.3: not taken.
    const int KT = p.H / kBK, f32 = p.router_bf16 ? 0 : 1;
    int cfg = 0, z = 1;
    float best = 0.f;
    for (int c = 0; c < 3; ++c) {
        const Tiling &t = kTilings[c];
        if (c > 0 && p.E <= t.experts[f32] / 2) continue;      // mostly padding
        const long long tiles = (long long)((p.T + t.tokens - 1) / t.tokens) * ((p.E + t.experts[f32] - 1) / t.experts[f32]);
        for (int n = 1; n <= kGatePlanes && (n == 1 || KT / n >= 4); ++n) {
            const float us = (float)((tiles * n + kChipUnits - 1) / kChipUnits) * (kTileUs + (float)((KT + n - 1) / n) * t.step[f32]) + (float)n * (float)p.T * (float)p.E * 8.f / kPlaneBytesPerUs;
            if ((c == 0 && n == 1) || us < best) { best = us; cfg = c; z = n; }
        }
    }
    *planes = z;
    // 128 x 256 (bf16 router) or 128 x 128 (fp32 router) on 8 wavefronts (2 x 4), 64 x 128 on 8, 32 x 64 on 4
    if (p.router_bf16) return cfg == 2 ? launch_t<uint16_t, 4, 4, 3, 8, 2>(p, z, st) : cfg == 1 ? launch_t<uint16_t, 2, 2, 6, 8, 2>(p, z, st) : launch_t<uint16_t, 2, 1, 6, 4, 1>(p, z, st);
    return cfg == 2 ? launch_t<float, 4, 2, 3, 8, 2>(p, z, st) : cfg == 1 ? launch_t<float, 4, 1, 4, 8, 1>(p, z, st) : launch_t<float, 2, 1, 6, 4, 1>(p, z, st);
}

}  // namespace emoe
