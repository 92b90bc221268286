// Tiles derived by the expert GEMM-1 itself: for passes of at most 64 tokens, shared by the weight-streaming bf16
// kernels (registers and LDS ring), the fp32 kernel and the token-by-token one, and for up to 1024 by the LDS ring (many_*, below).
#pragma once
#include "gate_select.h"
#include "moe_internal.h"

namespace emoe {

// Self-derived tiles (GEMM-1 of passes with at most 64 tokens and 256 slots whose selection kernel left per-block
// slot masks): with so few tokens the offsets / permutation / tile-list kernel is pure latency in front of the
// weight stream, and everything a GEMM-1 workgroup needs from it follows from 4 count bytes per slot.  So that
// kernel is not launched: every wavefront adds up the counts itself (lane l = up to four consecutive slots), finds
// the slot and chunk of its tile with a wavefront scan, and reads its rows' tokens off the slot's block masks;
// workgroup 0 of the same launch writes the tables that GEMM-2, the combine and the workspace view read, while the
// others stream.
constexpr int kSelfLaneSlots = 4, kSelfMaxSlots = 64 * kSelfLaneSlots;

// position of the r-th (0-based) set bit of m; m has more than r bits set
__device__ __forceinline__ int nth_set_bit(unsigned long long m, int r)
{
    int pos = 0;
#pragma unroll
    for (int w = 32; w >= 1; w >>= 1) {
        const int cnt = __popcll(m & ((1ull << w) - 1ull));
        if (r >= cnt) { r -= cnt; m >>= w; pos += w; }
    }
    return pos;
}

// Where the masks come from.  The selection kernel's tables:
struct SelfTables {
    // the count bytes of slot s that exist (blocks past nb hold nothing defined)
    __device__ __forceinline__ uint32_t counts(const Pass &p, int s, int nb) const
    {
        const uint32_t w = *(const uint32_t *)(p.blk_cnt + (size_t)s * fused_row_stride(nb));
        return nb >= 4 ? w : w & ((1u << (8 * nb)) - 1u);
    }
    __device__ __forceinline__ uint32_t mask(const Pass &p, int s, int b, int nb) const { return (uint32_t)p.blk_hist[(size_t)s * fused_row_stride(nb) + b]; }
    __device__ __forceinline__ int slot_rank(const Pass &p, int a) const { return p.slot_rank[a]; }
};
// or LDS, where the workgroup has selected the (at most kSelectTokens) tokens' experts itself:
struct SelfLds {
    const uint32_t *masks;     // per slot
    const int32_t *ranks;      // per assignment: slot << 12 | rank, or -1 (the workgroup that writes the tables)
    __device__ __forceinline__ uint32_t counts(const Pass &, int s, int) const { return (uint32_t)__popc(masks[s]); }
    __device__ __forceinline__ uint32_t mask(const Pass &, int s, int, int) const { return masks[s]; }
    __device__ __forceinline__ int slot_rank(const Pass &, int a) const { return ranks[a]; }
};

// or LDS, for all of up to 64 tokens, where a workgroup has selected them itself:
template <int NB>
struct SelfBlocks {
    const uint32_t *masks;     // [NB][kSelfMaxSlots]
    const int32_t *ranks;      // per assignment: slot << 12 | rank in the block of 16 tokens, or -1 (the workgroup that writes the tables)
    __device__ __forceinline__ uint32_t counts(const Pass &, int s, int) const
    {
        uint32_t w = 0;
#pragma unroll
        for (int b = 0; b < NB; ++b) w |= (uint32_t)__popc(masks[b * kSelfMaxSlots + s]) << (8 * b);
        return w;
    }
    __device__ __forceinline__ int slot_rank(const Pass &, int a) const { return ranks[a]; }
};

// Lane l of a wavefront: the count bytes of its slots l * spl + i, i < spl = ceil(S / 64), and the sums over all
// slots up to and including its own (rows in the high half, tiles of tile_rows in the low one).
struct SelfScan {
    uint32_t w[kSelfLaneSlots];   // count bytes (one per block of 16 tokens)
    int own, incl, spl;
};
__device__ __forceinline__ int rows_of(uint32_t count_bytes) { return (int)__builtin_amdgcn_sad_u8(count_bytes, 0u, 0u); }
template <typename Src = SelfTables>
__device__ __forceinline__ SelfScan self_scan(const Pass &p, int lane, int nb, int tile_rows, const Src &src = Src())
{
    SelfScan r;
    r.spl = (p.S + 63) >> 6;
    r.own = 0;
#pragma unroll
    for (int i = 0; i < kSelfLaneSlots; ++i) {
        const int s = lane * r.spl + i;
        r.w[i] = i < r.spl && s < p.S ? src.counts(p, s, nb) : 0u;
    }
#pragma unroll
    for (int i = 0; i < kSelfLaneSlots; ++i) {
        const int c = rows_of(r.w[i]);
        r.own += (c << 16) | ((c + tile_rows - 1) / tile_rows);
    }
    r.incl = r.own;
#pragma unroll
    for (int off = 1; off < 64; off <<= 1) {
        const int o = __shfl_up(r.incl, off, 64);
        if (lane >= off) r.incl += o;
    }
    return r;
}

// Workgroup 0: counts, offsets, tile list (slot order, chunks of tile_rows), permutation and its inverse --
// the tables of the bookkeeping kernels, for the few-token case.  All threads of the workgroup (256 or 1024); lds: kSelfTableBytes of LDS.
constexpr int kSelfTableBytes = kSelfMaxSlots * 8;
template <typename Src = SelfTables>
__device__ inline void self_tables(const Pass &p, int tile_rows, void *lds, const Src &src = Src())
{
    uint32_t *s_cb = (uint32_t *)lds;                        // count bytes of slot s
    int32_t *s_off = (int32_t *)(s_cb + kSelfMaxSlots);
    const int tid = threadIdx.x, nb = (p.T + kFusedTokens - 1) / kFusedTokens;
    if (tid < 64) {
        const SelfScan sc = self_scan(p, tid, nb, tile_rows, src);
        int row = (sc.incl - sc.own) >> 16, tl = (sc.incl - sc.own) & 0xffff;
#pragma unroll
        for (int i = 0; i < kSelfLaneSlots; ++i) {
            const int s = tid * sc.spl + i, c = rows_of(sc.w[i]);
            if (i >= sc.spl || s >= p.S) continue;
            const int nt = (c + tile_rows - 1) / tile_rows;
            s_cb[s] = sc.w[i];
            s_off[s] = row;
            p.counts[s] = c;
            p.offs[s] = row;
            for (int j = 0; j < nt; ++j, ++tl)
                if (tl < p.max_tiles) {
                    MTile mt;
                    mt.slot = s; mt.row_begin = row + j * tile_rows; mt.rows = min(tile_rows, c - j * tile_rows); mt.single = nt == 1;
                    p.tiles[tl] = mt;
                }
            row += c;
        }
        if (tid == 63) {
            p.offs[p.S] = sc.incl >> 16;
            *p.n_tiles = min(sc.incl & 0xffff, p.max_tiles);
        }
    }
    __syncthreads();
    for (int a = tid; a < p.T * p.kk; a += blockDim.x) {
        const int sr = src.slot_rank(p, a);
        int row = -1;
        if (sr >= 0) {
            const int slot = sr >> 12, rank = sr & 0xfff, t = a / p.kk, b = t / kFusedTokens;
            // rows of the slot in the blocks before the token's
            row = s_off[slot] + rank + rows_of(s_cb[slot] & ((1u << (8 * b)) - 1u));
            p.perm[row] = t;
        }
        p.inv[a] = row;
    }
}

// The tile of a task of a GEMM-1 that derives its tiles, the same in every wavefront; false past the last tile.
// *tokens: the slot's tokens, ascending, as a bit mask; *first: the tile's first row among them.
template <typename Src = SelfTables>
__device__ __forceinline__ bool self_tile(const Pass &p, int lane, int tile, int tile_rows, MTile *mt, unsigned long long *tokens, int *first, const Src &src = Src())
{
    const int nb = (p.T + kFusedTokens - 1) / kFusedTokens;
    const SelfScan sc = self_scan(p, lane, nb, tile_rows, src);
    const unsigned long long owners = __ballot((sc.incl & 0xffff) > tile);
    if (owners == 0) return false;
    const int l = __ffsll((long long)owners) - 1;
    int before = __builtin_amdgcn_readlane(sc.incl - sc.own, l), cs = 0, s = l * sc.spl;
#pragma unroll
    for (int i = 0; i < kSelfLaneSlots; ++i) {          // which of the lane's slots (uniform)
        const int c = rows_of((uint32_t)__builtin_amdgcn_readlane((int)sc.w[i], l)), nt = (c + tile_rows - 1) / tile_rows;
        if (cs == 0) {
            if ((before & 0xffff) + nt > tile) { cs = c; s += i; }
            else before += (c << 16) | nt;
        }
    }
    const int chunk = tile - (before & 0xffff);
    mt->slot = s;
    mt->row_begin = (before >> 16) + chunk * tile_rows;
    mt->rows = min(tile_rows, cs - chunk * tile_rows);
    mt->single = cs <= tile_rows;
    // bit t of the block masks side by side
    unsigned long long m = 0;
    for (int b = 0; b < nb; ++b) m |= (unsigned long long)(src.mask(p, s, b, nb) & 0xffffu) << (16 * b);
    *tokens = m;
    *first = chunk * tile_rows;
    return true;
}

// The same for more tokens (k_expert_ring): up to kManyBlocks blocks of 16.  A slot's count bytes are one 16-byte load per 16 blocks then, lane b has
// the mask of block b, and the tile's tokens go through LDS.
constexpr int kManyBlocks = 64;
static_assert(fused_row_stride(kManyBlocks) == kManyBlocks, "rows of count bytes are one line");
// rows of slot s in the blocks before b (16-byte words 0 .. n16 - 1 of its count bytes, n16 = 1 .. 4)
__device__ __forceinline__ int rows_in_blocks(const uint4 (&v)[4], int n16, int b)
{
    int sum = 0;
#pragma unroll
    for (int j = 0; j < 4; ++j) {
        if (j >= n16) continue;                             // uniform
        const uint32_t w[4] = {v[j].x, v[j].y, v[j].z, v[j].w};
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            const int n = b - 16 * j - 4 * i;               // bytes of the word that count
            sum += rows_of(n >= 4 ? w[i] : n <= 0 ? 0u : w[i] & ((1u << (8 * n)) - 1u));
        }
    }
    return sum;
}
__device__ __forceinline__ void load_counts(const Pass &p, int s, int n16, uint4 (&v)[4])
{
#pragma unroll
    for (int j = 0; j < 4; ++j)
        if (j < n16) v[j] = ((const uint4 *)(p.blk_cnt + (size_t)s * kManyBlocks))[j];
}
struct ManyScan { int c[kSelfLaneSlots], own, incl, spl; };   // as SelfScan, with the slots' rows instead of their count bytes
__device__ __forceinline__ ManyScan many_scan(const Pass &p, int lane, int nb, int tile_rows)
{
    ManyScan r;
    const int n16 = (nb + 15) >> 4;
    r.spl = (p.S + 63) >> 6;
    uint4 v[kSelfLaneSlots][4];
#pragma unroll
    for (int i = 0; i < kSelfLaneSlots; ++i)
        if (i < r.spl) load_counts(p, min(lane * r.spl + i, p.S - 1), n16, v[i]);
    r.own = 0;
#pragma unroll
    for (int i = 0; i < kSelfLaneSlots; ++i) {
        r.c[i] = 0;
        if (i < r.spl && lane * r.spl + i < p.S) r.c[i] = rows_in_blocks(v[i], n16, nb);
        r.own += (r.c[i] << 16) | ((r.c[i] + tile_rows - 1) / tile_rows);
    }
    r.incl = wave_incl_scan_i32(r.own);
    return r;
}
// As self_tile; tok (LDS, tile_rows entries of the wavefront's own): the tile's tokens
__device__ __forceinline__ bool many_tile(const Pass &p, int lane, int tile, int tile_rows, MTile *mt, int32_t *tok)
{
    const int nb = (p.T + kFusedTokens - 1) / kFusedTokens;
    const ManyScan sc = many_scan(p, lane, nb, tile_rows);
    const unsigned long long owners = __ballot((sc.incl & 0xffff) > tile);
    if (owners == 0) return false;
    const int l = __ffsll((long long)owners) - 1;
    int before = __builtin_amdgcn_readlane(sc.incl - sc.own, l), cs = 0, s = l * sc.spl;
#pragma unroll
    for (int i = 0; i < kSelfLaneSlots; ++i) {              // which of the lane's slots (uniform)
        const int c = __builtin_amdgcn_readlane(sc.c[i], l), nt = (c + tile_rows - 1) / tile_rows;
        if (cs == 0) {
            if ((before & 0xffff) + nt > tile) { cs = c; s += i; }
            else before += (c << 16) | nt;
        }
    }
    const int first = (tile - (before & 0xffff)) * tile_rows;
    mt->slot = s;
    mt->row_begin = (before >> 16) + first;
    mt->rows = min(tile_rows, cs - first);
    mt->single = cs <= tile_rows;
    uint32_t m = lane < nb ? (uint32_t)p.blk_hist[(size_t)s * kManyBlocks + lane] & 0xffffu : 0u;
    int at = wave_incl_scan_i32(__popc(m)) - __popc(m) - first;
    for (; m; m &= m - 1, ++at)
        if (at >= 0 && at < mt->rows) tok[at] = lane * kFusedTokens + __ffs((int)m) - 1;
    wave_sync();
    return true;
}
// Workgroup `part` of those that write the tables: the permutation and its inverse for kTableAssign assignments each, the first one everything else
constexpr int kTableAssign = 1024;
inline int table_blocks(const Pass &p) { return (p.T * p.kk + kTableAssign - 1) / kTableAssign; }
__device__ inline void many_tables(const Pass &p, int tile_rows, int part, void *lds)
{
    int32_t *s_off = (int32_t *)lds;                         // [kSelfMaxSlots]
    const int tid = threadIdx.x, nb = (p.T + kFusedTokens - 1) / kFusedTokens, n16 = (nb + 15) >> 4;
    if (tid < 64) {
        const ManyScan sc = many_scan(p, tid, nb, tile_rows);
        int row = (sc.incl - sc.own) >> 16, tl = (sc.incl - sc.own) & 0xffff;
#pragma unroll
        for (int i = 0; i < kSelfLaneSlots; ++i) {
            const int s = tid * sc.spl + i, c = sc.c[i], nt = (c + tile_rows - 1) / tile_rows;
            if (i >= sc.spl || s >= p.S) continue;
            s_off[s] = row;
            if (part == 0) {
                p.counts[s] = c;
                p.offs[s] = row;
                for (int j = 0; j < nt; ++j, ++tl)
                    if (tl < p.max_tiles) {
                        MTile mt;
                        mt.slot = s; mt.row_begin = row + j * tile_rows; mt.rows = min(tile_rows, c - j * tile_rows); mt.single = nt == 1;
                        p.tiles[tl] = mt;
                    }
            }
            row += c;
        }
        if (part == 0 && tid == 63) {
            p.offs[p.S] = sc.incl >> 16;
            *p.n_tiles = min(sc.incl & 0xffff, p.max_tiles);
        }
    }
    __syncthreads();
    for (int a = part * kTableAssign + tid; a < min((part + 1) * kTableAssign, p.T * p.kk); a += blockDim.x) {
        const int sr = p.slot_rank[a];
        int row = -1;
        if (sr >= 0) {
            const int slot = sr >> 12, t = a / p.kk;
            uint4 v[4];
            load_counts(p, slot, n16, v);
            row = s_off[slot] + (sr & 0xfff) + rows_in_blocks(v, n16, t / kFusedTokens);
            p.perm[row] = t;
        }
        p.inv[a] = row;
    }
}

// A token to four behind the logits kernel alone, selected by a GEMM-1's workgroup of four wavefronts, one a token: their masks and (workgroup 0, which
// also leaves the ids, the weights and what `tab` brings in the workspace) ranks in LDS.
constexpr int kSelectTokens = 4, kSelectExperts = 128, kSelectKK = 36;   // top_k <= 32 plus <= 4 shared experts
struct SelectLds {
    float scores[kSelectTokens][2 * kSelectExperts];
    uint32_t masks[kSelfMaxSlots];
    int32_t ranks[kSelectTokens * kSelectKK], map[kSelectExperts + 4];
};
template <typename Table>
__device__ __forceinline__ SelfLds select_few(const Pass &p, SelectLds &s, const Table &tab)
{
    const int lane = threadIdx.x & 63, t = (int)(threadIdx.x >> 6);
    const bool first = blockIdx.x == 0;
    for (int i = threadIdx.x; i < kSelfMaxSlots; i += kSelectTokens * 64) s.masks[i] = 0u;
    stage_table(p, tab, s.map, kSelectTokens * 64);
    __syncthreads();   // (requesting the logits first, as in the selection kernel, was no faster here: one token of the Qwen3 shape 27.1 -> 27.3)
    int slot = -1;
    if (t < p.T) {
        float *lg = s.scores[t], *cs = lg + kSelectExperts;
        const int id = p.E <= 64 ? select_from_planes<1, kGatePlanes>(p, t, lg, cs, lane, first, [] {})
                                 : select_from_planes<2, kGatePlanes>(p, t, lg, cs, lane, first, [] {});
        slot = slot_of_lane(p, s.map, t, lane, id);
        if (slot >= 0) atomicOr(&s.masks[slot], 1u << t);
    }
    __syncthreads();
    if (first && t < p.T && lane < p.kk) s.ranks[t * p.kk + lane] = slot >= 0 ? (slot << 12) | __popc(s.masks[slot] & ((1u << t) - 1u)) : -1;
    SelfLds src;
    src.masks = s.masks;
    src.ranks = s.ranks;
    return src;
}

}  // namespace emoe
