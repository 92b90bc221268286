// Launches saved where a pass is a chain of them: everything behind the gate of a pass of few tokens through a small layer in one
// launch (k_token_experts), the gate too where all tokens can be selected at once, GEMM-2 and combine of a token or two in one (k_gemm2_combine, at the end).
//
// The expert FFN of Sec. 2.1 of the paper and its weighted combine, token by token: a workgroup reads its token's k + n_shared
// experts (the slot comes from the selection kernel's table of assignments; Sec. 3.2 / 4.6: placement is data), keeps h
// and y in LDS and adds them up.
//
// What bounds it: nothing but latency.  As GEMM-1, GEMM-2 and combine such a pass is three launches of 3 to 5 us, each a chain of
// memory round trips; nothing is left of two of them when a token's rows need not meet the other tokens' of the same expert.  The
// price is that an expert's weights are read once per token instead of once per tile, out of L2, by one compute unit: the host
// takes this kernel while that is at most 256 KB per token (kTokenBytes) and there is a compute unit per token (kTokens).
// Whole pass, us, three launches -> this one: 128 x 64 fp32 layer, top-2, 1 token 14.3 -> 11.2, 64 tokens 16.4 -> 12.6, 256
// tokens 22.0 -> 16.8, in bf16 14.2 -> 11.4, 18.8 -> 16.1, 23.5 -> 18.0; at the limit of the bytes (512 x 16, fp32) 64 tokens 18.9 -> 18.6,
// 256 tokens 27.5 -> 23.0.
// Rows of the weights are dotted by quarter wavefronts (16 lanes x 16 bytes), several of them requested together; no matrix
// instruction, the contractions are too short to fill one.  Sums: a lane's products in order, then the 16 lanes' by halves.
// Workgroup 0 writes the tables (offsets, permutation, tile list) as in the other kernels that derive their tiles, and h and y go to the
// workspace too.
#include <algorithm>

#include "gate_small.h"
#include "moe_internal.h"
#include "self_tiles.h"
#include "wave_ops.h"

namespace emoe {
namespace {

constexpr int kThreads = 1024, kGroups = kThreads / 16;   // groups of 16 lanes, a weight row each
constexpr int kMaxKK = 36;                                // top_k <= 32 plus <= 4 shared experts
constexpr int kTokens = 256;                              // a workgroup per token: one round of the chip
constexpr long long kTokenBytes = 256 * 1024;

template <typename T> struct Vec;
template <> struct Vec<float> { static constexpr int n = 4; };
template <> struct Vec<uint16_t> { static constexpr int n = 8; };

// sum over the 16 lanes of a row of the wavefront, in its lane 15
__device__ __forceinline__ float row_sum(float v)
{
    v += __int_as_float(dpp_i32<0x118, 0xf>(0, __float_as_int(v)));   // row_shr 8, 4, 2, 1
    v += __int_as_float(dpp_i32<0x114, 0xf>(0, __float_as_int(v)));
    v += __int_as_float(dpp_i32<0x112, 0xf>(0, __float_as_int(v)));
    v += __int_as_float(dpp_i32<0x111, 0xf>(0, __float_as_int(v)));
    return v;
}

// acc[u] += rows[u] . v over this lane's share: elements l V + 16 V c .. of K (K % 8 == 0), v in LDS as floats.  (Two c's loads
// together: no faster, rows of 512 2 % slower.)
template <typename T, int U>
__device__ __forceinline__ void dot_rows(float (&acc)[U], const T *const (&rows)[U], const float *const (&v)[U], int K, int l)
{
    constexpr int V = Vec<T>::n;
    for (int k = l * V; k < K; k += 16 * V) {
        uint4 raw[U];
#pragma unroll
        for (int u = 0; u < U; ++u) raw[u] = *(const uint4 *)(rows[u] + k);
#pragma unroll
        for (int u = 0; u < U; ++u) {
            const T *w = (const T *)&raw[u];
#pragma unroll
            for (int i = 0; i < V; ++i) acc[u] = fmaf(load_f32<T>(w, i), v[u][k + i], acc[u]);
        }
    }
}

template <typename T> __device__ __forceinline__ float silu_up(float g, float u);
template <> __device__ __forceinline__ float silu_up<float>(float g, float u) { return g / (1.f + expf(-g)) * u; }
template <> __device__ __forceinline__ float silu_up<uint16_t>(float g, float u) { return silu_mul(g, u); }
// v as it is stored in the activation type
template <typename T> __device__ __forceinline__ float stored(float v);
template <> __device__ __forceinline__ float stored<float>(float v) { return v; }
template <> __device__ __forceinline__ float stored<uint16_t>(float v) { return bf16_to_f32(f32_to_bf16(v)); }

// Rows of the slots before s and of s in the blocks of tokens before t's (all lanes of a wavefront, each with its own s)
__device__ __forceinline__ int rows_before(const Pass &p, int lane, int t, int s, const SelfScan &sc)
{
    const int owner = s / sc.spl, mine = s - owner * sc.spl;
    int row = __shfl(sc.incl - sc.own, owner, 64) >> 16;
#pragma unroll
    for (int i = 0; i < kSelfLaneSlots; ++i) {
        const uint32_t w = (uint32_t)__shfl((int)sc.w[i], owner, 64);
        if (i < mine) row += rows_of(w);
        if (i == mine) row += rows_of(w & ((1u << (8 * (t / kFusedTokens))) - 1u));
    }
    return row;
}

// A token behind its selection: h and y of its n local experts (slots; x [H], h [n][I], y [n][H] in LDS) and their sum, all threads of the
// workgroup.  rows: where h and y go in the workspace; written by the first wavefront before it comes here, read behind the first barrier.
template <typename T>
__device__ __forceinline__ void token_ffn(const Pass &p, int t, int n, const int32_t *slots, const int32_t *rows, const float *wts, const float *x, float *h, float *y)
{
    const int H = p.H, I = p.I, tid = threadIdx.x, l = tid & 15, g = tid >> 4;
    // ---- h = silu(x . Wg) * (x . Wu): a group of lanes takes columns g, g + 64, ... of all experts, two of them together ----
    const size_t s13 = 2 * (size_t)I * H, s2 = (size_t)H * I;
    for (int c0 = g; c0 < n * I; c0 += 2 * kGroups) {
        const T *w[4];
        const float *v[4];
        int task[2];
#pragma unroll
        for (int u = 0; u < 2; ++u) {
            task[u] = min(c0 + u * kGroups, n * I - 1);          // past the end: the last one again, not stored
            const int j = task[u] / I, col = task[u] - j * I;
            w[2 * u] = (const T *)p.w13 + (size_t)slots[j] * s13 + (size_t)col * H;
            w[2 * u + 1] = w[2 * u] + (size_t)I * H;
            v[2 * u] = v[2 * u + 1] = x;
        }
        float acc[4] = {0.f, 0.f, 0.f, 0.f};
        dot_rows<T, 4>(acc, w, v, H, l);
#pragma unroll
        for (int u = 0; u < 2; ++u) {
            const float gate = row_sum(acc[2 * u]), up = row_sum(acc[2 * u + 1]);
            if (l == 15 && c0 + u * kGroups < n * I) h[task[u]] = stored<T>(silu_up<T>(gate, up));
        }
    }
    __syncthreads();
    for (int c = tid; c < n * I; c += kThreads) store_f32<T>((T *)p.h + (size_t)rows[c / I] * I, c % I, h[c]);
    // ---- y = h . W2 ----
    for (int c0 = g; c0 < n * H; c0 += 4 * kGroups) {
        const T *w[4];
        const float *v[4];
        int task[4];
#pragma unroll
        for (int u = 0; u < 4; ++u) {
            task[u] = min(c0 + u * kGroups, n * H - 1);
            const int j = task[u] / H, col = task[u] - j * H;
            w[u] = (const T *)p.w2 + (size_t)slots[j] * s2 + (size_t)col * I;
            v[u] = h + j * I;
        }
        float acc[4] = {0.f, 0.f, 0.f, 0.f};
        dot_rows<T, 4>(acc, w, v, I, l);
#pragma unroll
        for (int u = 0; u < 4; ++u) {
            const float s = row_sum(acc[u]);
            if (l == 15 && c0 + u * kGroups < n * H) y[task[u]] = stored<T>(s);
        }
    }
    __syncthreads();
    for (int c = tid; c < n * H; c += kThreads) store_f32<T>((T *)p.y + (size_t)rows[c / H] * H, c % H, y[c]);
    // ---- combine, in selection order ----
    for (int c = tid; c < H; c += kThreads) {
        float o = 0.f;
        for (int j = 0; j < n; ++j) o = fmaf(wts[j], y[(size_t)j * H + c], o);
        store_f32<T>((T *)p.out + (size_t)t * H, c, o);
    }
}

template <typename T, bool kSelf>
__global__ __launch_bounds__(kThreads) void k_token_experts(Pass p, int tile_rows)
{
    extern __shared__ float sm[];             // x [H], h [n][I], y [n][H]; or workgroup 0's tables
    __shared__ int32_t slots[kMaxKK], rows[kMaxKK], n_local;
    __shared__ float wts[kMaxKK];
    if (kSelf && blockIdx.x == 0) { self_tables(p, tile_rows, sm); return; }
    const int t = blockIdx.x - (kSelf ? 1 : 0), H = p.H, I = p.I, tid = threadIdx.x, lane = tid & 63;
    float *x = sm, *h = x + H, *y = h + (size_t)p.kk * I;
    for (int c = tid; c < H; c += kThreads) x[c] = load_f32<T>((const T *)p.x + (size_t)t * H, c);
    if (tid < 64) {   // first wavefront: the token's local assignments, compacted, in selection order
        int slot = -1, row = 0;
        float wv = 0.f;
        if (lane < p.kk) {
            const int a = t * p.kk + lane;
            wv = lane < p.k ? p.w[(size_t)t * p.k + lane] : 1.0f;
            if (kSelf) {
                row = p.slot_rank[a];
                slot = row >> 12;
            } else {
                row = p.inv[a];
                slot = slot_of(p, a);
            }
        }
        if (kSelf) {   // the row among all rows: those of the slots before, of the slot in earlier blocks of tokens, the rank
            row = (row & 0xfff) + rows_before(p, lane, t, max(slot, 0), self_scan(p, lane, (p.T + kFusedTokens - 1) / kFusedTokens, tile_rows));
        }
        const unsigned long long m = __ballot(slot >= 0);
        if (slot >= 0) {
            const int at = __popcll(m & ((1ull << lane) - 1ull));
            slots[at] = slot;
            rows[at] = row;
            wts[at] = wv;
        }
        if (lane == 0) n_local = __popcll(m);
    }
    __syncthreads();
    token_ffn<T>(p, t, n_local, slots, rows, wts, x, h, y);
}

// The whole pass of a small layer, the gate too, in one launch (up to 64 tokens; routers as in k_gate_small).  A workgroup per token, and one that writes the tables, ids
// and weights.  Every one of them multiplies and selects ALL tokens, since where a token's h and y go in the workspace follows from the
// others' selections, and nothing waits for another workgroup; its own token's experts follow as above.  What bounds it: latency, as above; what it saves is a
// launch and the round trips of the tables.  NTT tiles of 16 tokens, NTT tokens a wavefront, on 64 / NTT lanes each: a wavefront that selects
// one after the other takes 1.2 us for each (64 tokens of the 128 x 64 layer 12.1 -> 13.4).
template <typename T, typename WT, int NTT, typename Table>
__global__ __launch_bounds__(kThreads) void k_token_experts(Pass p, int tile_rows, Table tab)
{
    extern __shared__ float sm[];             // x [H]; then partial logits [NTT][wavefronts with a share][256], behind them h [n][I], y [n][H], or the tables and ranks
    __shared__ uint32_t masks[NTT * kSelfMaxSlots];
    __shared__ int32_t map[kSmallExperts + 4];
    __shared__ float scratch[NTT == 1 ? kThreads / 64 * 128 : 1];
    __shared__ int32_t slots[kMaxKK], rows[kMaxKK], n_local;
    __shared__ float all_w[kMaxKK], wts[kMaxKK];
    static_assert(kThreads == 64 * kFusedTokens, "a wavefront per token of a tile");
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6, t = (int)blockIdx.x - 1, H = p.H;
    const bool tables = blockIdx.x == 0;
    float *x = sm, *rest = sm + H;
    if (!tables)
        for (int c = tid; c < H; c += kThreads) x[c] = load_f32<T>((const T *)p.x + (size_t)t * H, c);
    for (int s = tid; s < NTT * kSelfMaxSlots; s += kThreads) masks[s] = 0u;
    stage_table(p, tab, map, kThreads);
    const SmallShare sh(p, wave, true);
    f32x4 acc[NTT];
    small_products<NTT, T, WT>(p, 0, sh, lane, acc);
    if (wave < sh.waves()) {
#pragma unroll
        for (int i = 0; i < NTT; ++i)
#pragma unroll
            for (int r = 0; r < 4; ++r) rest[(i * sh.waves() + wave) * 256 + r * 64 + lane] = acc[i][r];
    }
    __syncthreads();
    // ---- selection: lanes of a token, its assignment `sub` ----
    constexpr int L = 64 / NTT;
    const int sub = lane & (L - 1), tok = wave * NTT + lane / L, tile = tok / kFusedTokens, in_tile = tok % kFusedTokens;
    const bool own = tok == t;
    const float logit = small_logit(p, sh, rest + tile * sh.waves() * 256, in_tile, sub);
    int slot = -1;
    if (wave * NTT < p.T) {                                // uniform
        int id;
        if constexpr (NTT == 1) {
            float v[1] = {logit};
            id = select_regs<1>(p, tok, v, scratch + wave * 128, scratch + wave * 128 + 64, lane, tables, own ? all_w : nullptr);
        } else {
            id = select_lanes<L>(p, tok, logit, lane, tok < p.T, tables, own ? all_w : nullptr);
        }
        if (tok < p.T) slot = slot_of_lane(p, map, tok, sub, id);
        if (slot >= 0) atomicOr(&masks[tile * kSelfMaxSlots + slot], 1u << in_tile);
        wave_sync();
        const uint64_t here = __ballot(slot >= 0) >> (lane & (64 - L)) & (~0ull >> (64 - L));
        if (own) {                                         // the local assignments, compacted, in selection order
            if (slot >= 0) {
                const int at = __popcll(here & ((1ull << sub) - 1ull));
                slots[at] = slot;
                wts[at] = sub < p.k ? all_w[sub] : 1.0f;
            }
            if (sub == 0) n_local = __popcll(here);
        }
    }
    __syncthreads();
    SelfBlocks<NTT> src;
    src.masks = masks;
    src.ranks = nullptr;
    if (tables) {
        int32_t *ranks = (int32_t *)(rest + kSelfTableBytes / 4);
        if (tok < p.T && sub < p.kk)
            ranks[tok * p.kk + sub] = slot >= 0 ? (slot << 12) | __popc(masks[tile * kSelfMaxSlots + slot] & ((1u << in_tile) - 1u)) : -1;
        src.ranks = ranks;                                // read behind self_tables' barrier
        self_tables(p, tile_rows, rest, src);
        return;
    }
    const int n = n_local;
    if (tid < 64) {
        const int s = lane < n ? slots[lane] : 0, b = t / kFusedTokens;
        const int before = rows_before(p, lane, t, s, self_scan(p, lane, (p.T + kFusedTokens - 1) / kFusedTokens, tile_rows, src));
        if (lane < n) rows[lane] = before + __popc(masks[b * kSelfMaxSlots + s] & ((1u << (t % kFusedTokens)) - 1u));
    }
    float *h = rest, *y = h + (size_t)p.kk * p.I;
    token_ffn<T>(p, t, n, slots, rows, wts, x, h, y);
}

// GEMM-2 and combine of a token or two (bf16): a token's experts share no rows with another token's worth speaking of, so
// a workgroup takes 8 columns of out for one token, wavefront j its j-th local expert (and the j + 8-th): 8 rows of W2, all
// of a row's loads a lane has in flight together, dotted without matrix instructions, y rounded as it is stored, added up in
// selection order.  What bounds it: the weights' way from HBM and the launch; the combine by itself was 4 us of latency behind it.
// One token of the Qwen3 shape (8 experts, 25 MB of W2): GEMM-2 7.1 us and combine 4.3 us -> 8.4 us.  (When it pays: moe_api.hip.)
constexpr int kCols = 8, kColWaves = 8;
__global__ __launch_bounds__(64 * kColWaves) void k_gemm2_combine(Pass p)
{
    __shared__ float y[kMaxKK][kCols];
    const int t = blockIdx.y, n0 = blockIdx.x * kCols, H = p.H, I = p.I, lane = threadIdx.x & 63;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    int slot = -1, row = 0;
    if (lane < p.kk) {
        slot = slot_of(p, t * p.kk + lane);
        row = p.inv[(size_t)t * p.kk + lane];
    }
    unsigned long long left = __ballot(slot >= 0);           // local assignments, in selection order
    const int n = __popcll(left);
    for (int i = 0; i < n; ++i, left &= left - 1) {
        if (i % kColWaves != wave) continue;                 // uniform
        const int j = __ffsll((long long)left) - 1, s = __builtin_amdgcn_readlane(slot, j), r = __builtin_amdgcn_readlane(row, j);
        const uint16_t *w = (const uint16_t *)p.w2 + (size_t)s * H * I + (size_t)n0 * I, *h = (const uint16_t *)p.h + (size_t)r * I;
        float acc[kCols] = {};
        for (int k0 = 0; k0 < I; k0 += 1024) {               // two pieces of 512: one 16-byte load per row, lane and piece
            uint4 raw[2][kCols], hv[2];
#pragma unroll
            for (int c = 0; c < 2; ++c) {
                const int k = k0 + c * 512 + lane * 8;
                const bool in = k < I;                       // I % 8 == 0
                hv[c] = in ? *(const uint4 *)(h + k) : make_uint4(0, 0, 0, 0);
#pragma unroll
                for (int q = 0; q < kCols; ++q) raw[c][q] = in ? *(const uint4 *)(w + (size_t)q * I + k) : make_uint4(0, 0, 0, 0);
            }
            __builtin_amdgcn_sched_barrier(0);               // all loads go out before the first product
#pragma unroll
            for (int c = 0; c < 2; ++c)
#pragma unroll
                for (int q = 0; q < kCols; ++q)
#pragma unroll
                    for (int e = 0; e < 8; ++e)
                        acc[q] = fmaf(load_f32<uint16_t>((const uint16_t *)&raw[c][q], e), load_f32<uint16_t>((const uint16_t *)&hv[c], e), acc[q]);
        }
        float mine = 0.f;
#pragma unroll
        for (int q = 0; q < kCols; ++q) {
            const float sum = wave_sum_f32(acc[q]);
            mine = lane == q ? sum : mine;
        }
        if (lane < kCols) {
            const uint16_t b = f32_to_bf16(mine);
            ((uint16_t *)p.y)[(size_t)r * H + n0 + lane] = b;
            y[i][lane] = bf16_to_f32(b);
        }
    }
    __syncthreads();
    if (threadIdx.x >= 64) return;
    unsigned long long m = __ballot(slot >= 0);
    const float wv = lane < p.k ? p.w[(size_t)t * p.k + lane] : 1.0f;
    float o = 0.f;
    for (int i = 0; i < n; ++i, m &= m - 1) {
        const float wj = __int_as_float(__builtin_amdgcn_readlane(__float_as_int(wv), __ffsll((long long)m) - 1));
        if (lane < kCols) o = fmaf(wj, y[i][lane], o);
    }
    if (lane < kCols) ((uint16_t *)p.out)[(size_t)t * H + n0 + lane] = f32_to_bf16(o);
}

template <typename T, typename WT, int NTT, typename Table>
hipError_t launch_pass_t(const Pass &p, int tile_rows, const Table &tab, hipStream_t st)
{
    const int n_et = (p.E + 15) / 16, parts = kFusedTokens / n_et, chunks = (p.H + 31) / 32, per = (chunks + parts - 1) / parts;
    const size_t logits = (size_t)NTT * ((chunks + per - 1) / per * n_et) * 256, ffn = (size_t)p.kk * (p.I + p.H), tables = kSelfTableBytes / 4 + (size_t)p.T * p.kk;
    const size_t lds = sizeof(float) * (p.H + std::max(logits, std::max(ffn, tables)));
    if (lds > 48 * 1024) {       // beside the static part
        const hipError_t e = hipFuncSetAttribute((const void *)k_token_experts<T, WT, NTT, Table>, hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds);
        if (e != hipSuccess) return e;
    }
    hipLaunchKernelGGL((k_token_experts<T, WT, NTT, Table>), dim3(p.T + 1), dim3(kThreads), lds, st, p, tile_rows, tab);
    return hipGetLastError();
}

template <typename T, typename WT>
hipError_t launch_pass(const Pass &p, int tile_rows, hipStream_t st)
{
    if (p.T <= 16) return p.host_table ? launch_pass_t<T, WT, 1>(p, tile_rows, fill_table(p), st) : launch_pass_t<T, WT, 1>(p, tile_rows, NoTable{}, st);
    if (p.T <= 32) return p.host_table ? launch_pass_t<T, WT, 2>(p, tile_rows, fill_table(p), st) : launch_pass_t<T, WT, 2>(p, tile_rows, NoTable{}, st);
    return p.host_table ? launch_pass_t<T, WT, 4>(p, tile_rows, fill_table(p), st) : launch_pass_t<T, WT, 4>(p, tile_rows, NoTable{}, st);
}

}  // namespace

// Whether the gate goes into the launch too.  Every workgroup then reads all token rows and the router, which costs it about 30 GB/s worth of time; whole
// pass, us, gate in a launch of its own (bf16 with more than 4 E assignments: two, bookkeeping) -> in this one, KB of both: 128 x 64 fp32, 8 experts, top-2, 1 token 11.1 -> 7.8, 16 12.1 -> 8.4, 17 (20
// KB) 12.2 -> 8.4, 64 (36 KB) 12.1 -> 9.4, in bf16 15.8 -> 9.4; 256 x 32, 64 tokens, 16 experts (80 KB) 15.3 -> 13.4, 32, 24 experts (56 KB) 15.3 -> 13.4; 512 x 16 bf16, 32 tokens, 32
// experts (96 KB) 22.2 -> 21.1; 512 x 8 fp32, 32 of them (128 KB) 21.2 -> 21.5, 64 tokens, 16 experts (160 KB) 19.1 -> 20.2.  With one token tile the gate's own launch reads
// as much: 512 x 8, 16 tokens, 64 experts (160 KB) 24.9 -> 22.4, 512 x 16 bf16, grouped gate 23.2 -> 20.1.
bool token_pass_supports(const Pass &p)
{
    if (!p.self_tiles || !token_experts_supports(p) || !one_gate_kernel(p)) return false;
    if (p.T <= 16) return true;
    const int tiles = p.T <= 32 ? 2 : 4, lanes = 64 / tiles;     // of 16 tokens; that select a token
    return p.n_group == 1 && p.E <= lanes && p.kk <= lanes && (tiles * 16 * (p.act_bf16 ? 2 : 4) + p.E * (p.router_bf16 ? 2 : 4)) * p.H <= 96 * 1024;
}

hipError_t launch_token_pass(const Pass &p, int tile_rows, hipStream_t st)
{
    if (p.act_bf16) return p.router_bf16 ? launch_pass<uint16_t, uint16_t>(p, tile_rows, st) : launch_pass<uint16_t, float>(p, tile_rows, st);
    return p.router_bf16 ? launch_pass<float, uint16_t>(p, tile_rows, st) : launch_pass<float, float>(p, tile_rows, st);
}

// H % 8 == 0 as everywhere
hipError_t launch_gemm2_combine(const Pass &p, hipStream_t st)
{
    hipLaunchKernelGGL(k_gemm2_combine, dim3(p.H / kCols, p.T), dim3(64 * kColWaves), 0, st, p);
    return hipGetLastError();
}

bool token_experts_supports(const Pass &p)
{
    return p.T <= kTokens && 3ll * p.kk * p.H * p.I * (p.act_bf16 ? 2 : 4) <= kTokenBytes;
}

hipError_t launch_token_experts(const Pass &p, int tile_rows, hipStream_t st)
{
    const size_t smem = sizeof(float) * ((size_t)p.H + (size_t)p.kk * (p.I + p.H));   // at most 44 KB with kTokenBytes of weights and I >= 8
    const size_t lds = smem > (size_t)kSelfTableBytes ? smem : (size_t)kSelfTableBytes;
    const dim3 grid(p.T + (p.self_tiles ? 1 : 0)), block(kThreads);
    if (p.act_bf16) {
        if (p.self_tiles) hipLaunchKernelGGL((k_token_experts<uint16_t, true>), grid, block, lds, st, p, tile_rows);
        else              hipLaunchKernelGGL((k_token_experts<uint16_t, false>), grid, block, lds, st, p, tile_rows);
    } else {
        if (p.self_tiles) hipLaunchKernelGGL((k_token_experts<float, true>), grid, block, lds, st, p, tile_rows);
        else              hipLaunchKernelGGL((k_token_experts<float, false>), grid, block, lds, st, p, tile_rows);
    }
    return hipGetLastError();
}

}  // namespace emoe
