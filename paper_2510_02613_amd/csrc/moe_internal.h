// Internal declarations shared by the translation units of libelasticmoe.so.
// Host-side launch wrappers only; every kernel lives in its own .hip file.
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

#include "elasticmoe.h"

namespace emoe {

// One M-tile of the grouped GEMMs: `rows` consecutive grouped rows starting at
// `row_begin`, all belonging to weight slot `slot`.
struct MTile {
    int32_t slot;
    int32_t row_begin;
    int32_t rows;
    int32_t single;   // 1 when the tile is all of its slot's rows (nobody else reads the slot's weights in this pass)
};

// One work unit of the large-tile GEMMs: an M-tile with a run of its N-slices.  The unit list of a GEMM is
// read as rows of 8: entry 8 i + x is the i-th unit of XCD x (workgroup b serves XCD b mod 8), so which
// column a unit sits in decides where it runs; rows == 0 marks a hole at the end of a column.
struct MUnit {
    int32_t slot;
    int32_t row_begin;
    int32_t rows;
    int32_t info;     // first N-slice of the run << 1 | the tile's single flag
};
struct UnitHdr {
    int32_t n_rows;   // rows of 8 workgroups the launch has to run: unit rows x spp
    int32_t spp;      // N-slices per unit
    int32_t n_units;  // entries of the list, holes included (a multiple of 8)
    int32_t runs;     // runs a tile's N-slices are split into
};

constexpr int kUnitSlack = 2;   // units by which an XCD's column of the unit list may exceed an even deal

// Runs a tile's N-slices are split into so that the units deal out evenly to the 8 XCDs: the smallest
// divisor d of n_slices with at most 5 % of an XCD's share idle if all units were alike, else n_slices.
__host__ __device__ inline int mfma8_runs(int n_chunks, int n_slices)
{
    for (int d = 1; d < n_slices; ++d) {
        const int units = n_chunks * d, dealt = (units + 7) / 8 * 8;
        if (n_slices % d == 0 && (dealt - units) * 20 <= units) return d;
    }
    return n_slices;
}

// Everything the kernels need to know about one forward pass.  Plain device
// pointers into caller-owned memory (x/out/weights) and the caller's workspace.
struct Pass {
    // layer
    int32_t T, H, I, E, k, S, kk;  // kk = k + n_shared : assignment columns per token
    int32_t n_shared;
    int32_t act_bf16, router_bf16;
    int32_t gate, n_group, topk_group, renormalize;
    float routed_scale;
    int32_t shared_begin, shared_end;
    // caller buffers
    const void *x;
    void *out;
    const void *router_w;
    const float *logit_bias, *select_bias;
    const void *w13, *w2;
    // workspace
    const int32_t *map;  // [E + n_shared] active table, shared slots last
    float *logits;       // [logit_planes][T,E] gate logits: the planes are partial sums over K ranges
    int32_t logit_planes;
    int32_t logit_tokens;   // tokens the logits' memory holds with one plane; fewer than T (fp32 layers): the gate takes a part of the batch at a time, fused_hist is off
    int32_t *ids;        // [T,k]
    float *w;            // [T,k]
    int32_t *slot_rank;  // [T*kk] (slot << 12 | rank-in-block) or -1
    int32_t *blk_hist;   // [NB,S] per-block histogram, then per-block exclusive base (fused bookkeeping: [S][row stride] token masks)
    uint8_t *blk_cnt;    // fused bookkeeping: [S][row stride] rows per slot and block of 16 tokens
    int32_t *counts;     // [S]
    int32_t *offs;       // [S+1]
    int32_t *perm;       // [A]
    int32_t *inv;        // [T,kk]
    MTile *tiles;        // [max_tiles]
    int32_t *n_tiles;    // [1]
    MUnit *units[2];     // large-tile GEMMs only: the unit lists of GEMM-1 and GEMM-2, unit_cap entries each (else NULL)
    UnitHdr *unit_hdr;   // [2]
    int32_t unit_cap;
    int32_t n_slices[2]; // N-slices of a tile in GEMM-1 and GEMM-2
    int32_t tiles_expected, slot_tiles_expected, tile_rows_expected;   // large-tile GEMMs, for an even load: tiles in all, of a slot, rows of a tile
    void *h;             // [A,I]
    void *y;             // [A,H]
    int32_t max_tiles;
    int32_t gate_tiled;  // the LDS-tiled gate logits kernel is forced (testing aid)
    int32_t self_tiles;  // weight-streaming and fp32 GEMM-1 and k_token_experts only: their workgroups derive their tile from the selection kernel's per-block counts and
                         // masks (self_select, and k_token_experts with the gate: from their own selection) themselves, and workgroup 0 of the launch writes the tables (offsets, permutation, tile list) beside them
    int32_t table_blocks; // self_tiles, k_expert_ring with tiles of 64 rows or more than 64 tokens: as many workgroups write the tables; else 0
    int32_t self_select; // GEMM-1 selects the experts itself from the logits (a token to four): no selection kernel
    int32_t fused_hist;  // the selection kernel also ranks the assignments (blocks of kFusedTokens tokens, blk_hist [S][blocks]
                         // of token masks); the scan-and-place kernel finishes the bookkeeping
    float *partials;     // partial sums of the large-tile GEMMs' split tiles, or NULL (no room: never split)
    const int32_t *host_table;   // HOST address of the expert table when the kernel that selects (selection kernel, k_gate_small, GEMM-1 of a token to four) is to carry it in as an argument (moe_forward_static), else NULL
    int32_t n_cus;       // compute units of the device (set by the large-tile launcher)
    int32_t k_split;     // this launch may share the contraction of its last round's tiles out (set by the launcher)
};

constexpr int kSortMax = 2048;         // tile lists of the large-tile kernels that may get this long are ordered by size and first assignment, longer ones by slot
inline __host__ __device__ bool tile_list_sorted(const Pass &p) { return p.max_tiles <= kSortMax; }
constexpr int kTableArg = 512;         // expert-table entries that travel in one kernel argument
constexpr int kGatePlanes = 8;         // most partial-sum planes of the gate logits
constexpr int kGateFewTokens = 256;    // up to here the few-token logits kernel shares the contraction out over workgroups
constexpr int kAssignPerBlock = 1024;  // assignments ranked by one block of the slot histogram kernel
constexpr int kFusedTokens = 16;       // tokens per workgroup of the fused selection + ranking kernel (one per wavefront)
constexpr int kFusedMaxTokens = 8192;  // largest batch the fused bookkeeping serves: every placing workgroup reads all block masks
// words between the rows of blk_hist [S][blocks] in the fused bookkeeping: whole groups of 64 blocks
__host__ __device__ constexpr int fused_row_stride(int n_blocks) { return (n_blocks + 63) / 64 * 64; }

hipError_t launch_write_map(int32_t *dst, const int32_t *host_vals, int n, hipStream_t st);
hipError_t launch_fill_slot(void *dst13, const void *src13, size_t bytes13, void *dst2, const void *src2, size_t bytes2, int blocks, hipStream_t st);  // bytes % 16 == 0
hipError_t launch_gate(Pass &p, hipStream_t st);   // sets logit_planes
bool one_gate_kernel(const Pass &p);                 // logits and selection are one kernel
bool gemm1_selects(const Pass &p, int blocks);       // a GEMM-1 of that many workgroups that derives its tiles does the selection too
int decode_blocks(const Pass &p);                    // workgroups of the GEMM-1 of k_expert_decode, of k_expert_ring (one that writes the tables aside)
int ring_blocks(const Pass &p);
int gate_f32_planes(int T, int H);   // partial-sum planes of the gate logits of fp32 layers
hipError_t launch_gate_logits_dma(const Pass &p, int *planes, hipStream_t st);   // logits only, bf16 activations
bool gate_dma_supports(const Pass &p);
hipError_t launch_permute(const Pass &p, int tile_rows, bool sort_tiles, hipStream_t st);
// which: 0 = first GEMM (gather + SwiGLU), 1 = second GEMM
hipError_t launch_experts_generic(const Pass &p, int which, hipStream_t st);
hipError_t launch_experts_mfma(const Pass &p, int which, hipStream_t st);
int mfma_tile_rows();
// 8-wavefront large-tile variant (needs H % 64 == 0 and I % 64 == 0)
hipError_t launch_experts_mfma8(const Pass &p, int which, hipStream_t st);
int mfma8_tile_rows();
bool mfma8_supports(const Pass &p);
int mfma8_n_slices(int H, int I, int which);   // N-slices of a tile in GEMM-1 (which = 0) or GEMM-2
int mfma8_grid_rows(int max_tiles, int n_slices);   // rows of 8 workgroups a launch provides
size_t mfma8_partial_bytes();   // workspace for the partial sums of tiles whose contraction is shared out
hipError_t launch_ceiling_mfma(int blocks, int iters, int random_operands, float *sink, hipStream_t st);
double ceiling_mfma_flops(int blocks, int iters);
hipError_t launch_ceiling_stream(const void *buf, size_t bytes, float *sink, hipStream_t st);
hipError_t launch_ceiling_tile_stream(const void *buf, int n_tiles, size_t row_bytes, int non_temporal, hipStream_t st);
// weight-streaming variant for decode-sized batches (M-tiles of 16 rows)
hipError_t launch_experts_decode(const Pass &p, int which, hipStream_t st);
int decode_tile_rows();
// the same for contractions that are whole K-steps (H and I multiples of 64)
hipError_t launch_experts_ring(const Pass &p, int tile_rows, int which, hipStream_t st);
int ring_tile_rows(bool large);   // large: 64 rows, for a dozen or two a slot and for more on few slots
// fp32 layers, M-tiles of 16, 32 or 64 rows
hipError_t launch_experts_f32(const Pass &p, int tile_rows, int which, hipStream_t st);
int f32_tile_rows(const Pass &p);
// GEMM-1 of these can derive its tiles itself (Pass::self_tiles) when the selection kernel left per-block masks for
// at most 4 blocks of tokens and 256 slots: no bookkeeping kernel in front of it
inline bool self_tiles_possible(const Pass &p) { return p.fused_hist && p.S <= 256 && p.T <= 4 * 16; }
int self_table_blocks(const Pass &p);   // k_expert_ring, up to 64 blocks: workgroups that write the tables, 0: not possible, or slower than the bookkeeping kernel (max_tiles is set)
// everything behind the gate and the bookkeeping in one launch, for few tokens of small layers
bool token_experts_supports(const Pass &p);
hipError_t launch_token_experts(const Pass &p, int tile_rows, hipStream_t st);
bool token_pass_supports(const Pass &p);             // and the gate too (self_tiles is set)
hipError_t launch_token_pass(const Pass &p, int tile_rows, hipStream_t st);
hipError_t launch_gemm2_combine(const Pass &p, hipStream_t st);   // GEMM-2 and combine of a token or two (bf16)
hipError_t launch_identity_experts(const Pass &p, hipStream_t st);
hipError_t launch_combine(const Pass &p, hipStream_t st);

// A layer that was told which page pools its weights live in (moe_layer_bind_vpools) checks on the host that
// every slot a placement names has a page under it; the pool tells the layer when it goes away.
bool vpool_backed(const moe_vpool *pool, int32_t slot);          // moe_vpool.hip
void vpool_bind(moe_vpool *pool, moe_layer *layer);
void vpool_unbind(moe_vpool *pool, moe_layer *layer);
void layer_drop_vpool(moe_layer *layer, const moe_vpool *pool);  // moe_api.hip

constexpr int kGenericTileRows = 32;  // M-tile of the plain expert kernels

// ---- small device helpers ---------------------------------------------------
__device__ __forceinline__ float bf16_to_f32(uint16_t b) { return __uint_as_float(((uint32_t)b) << 16); }

// slot of assignment a (token a / kk, column a % kk), or -1 when it is not this rank's
__device__ __forceinline__ int slot_of(const Pass &p, int a)
{
    if (a >= p.T * p.kk) return -1;
    const int t = a / p.kk, j = a - t * p.kk;
    if (j < p.k) {
        // ids come from the gate, or from the caller when the routing is given: an id outside
        // [0, E) is an assignment that does not exist
        const int id = p.ids[(size_t)t * p.k + j];
        if ((unsigned)id >= (unsigned)p.E) return -1;
        const int m = p.map[id];
        if (m >= -1) return m;
        // replicated expert: -2 - m is where its copy list (count R >= 2, then R slots) starts behind
        // the E + n_shared entries; token t uses copy t mod R
        const int32_t *copies = p.map + p.E + p.n_shared + (-2 - m);
        return copies[1 + t % copies[0]];
    }
    if (t >= p.shared_begin && t < p.shared_end) return p.map[p.E + (j - p.k)];
    return -1;
}

// 16-byte slot swizzle of a 128-byte tile row: slot = chunk ^ swz8(row).  An LDS read of 16 bytes
// per lane is served 16 lanes at a time over 64 four-byte banks (256 bytes, i.e. 2 rows): the
// 16 consecutive rows a half-wavefront reads for one MFMA operand must therefore hit 16 distinct
// 16-byte bank groups.  Row bits (1, 2, 0^3) do that.
__device__ __forceinline__ int swz8(int row) { return ((row >> 1) & 3) | (((row ^ (row >> 3)) & 1) << 2); }

// fp32 -> bf16, round to nearest even (one v_cvt_pk_bf16_f32 per pair on gfx950)
__device__ __forceinline__ uint16_t f32_to_bf16(float f)
{
    const __bf16 b = (__bf16)f;
    return __builtin_bit_cast(uint16_t, b);
}

// silu(g) * u with the hardware exp2 / reciprocal (about 1 ulp each): g * u / (1 + exp(-g))
__device__ __forceinline__ float silu_mul(float g, float u)
{
    return g * __builtin_amdgcn_rcpf(1.f + __expf(-g)) * u;
}

template <typename T> __device__ __forceinline__ float load_f32(const T *p, size_t i);
template <> __device__ __forceinline__ float load_f32<float>(const float *p, size_t i) { return p[i]; }
template <> __device__ __forceinline__ float load_f32<uint16_t>(const uint16_t *p, size_t i) { return bf16_to_f32(p[i]); }

template <typename T> __device__ __forceinline__ void store_f32(T *p, size_t i, float v);
template <> __device__ __forceinline__ void store_f32<float>(float *p, size_t i, float v) { p[i] = v; }
template <> __device__ __forceinline__ void store_f32<uint16_t>(uint16_t *p, size_t i, float v) { p[i] = f32_to_bf16(v); }

}  // namespace emoe
