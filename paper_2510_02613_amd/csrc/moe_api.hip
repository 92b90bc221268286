// Host side of libelasticmoe.so: argument checking, workspace carving, the
// expert-map switch and the launch sequence of one forward pass.
//
// The library owns no device memory (the paper's execution processes only hold
// references to tensors kept by the memory daemon, Sec. 3.2 "Decoupled Memory and
// Execution Layers"); all intermediates live in the caller's workspace, which is
// carved once at create time, so no later call can allocate.
#include <atomic>
#include <chrono>
#include <cmath>
#include <cstdarg>
#include <cstdio>
#include <cstring>
#include <mutex>
#include <new>
#include <vector>

#include "moe_internal.h"

using namespace emoe;

// Scratch of moe_forward_static: the whole workspace of its pass lives here, so that the call needs no
// device memory from anybody.  One copy per GPU the library is loaded on, held until the process ends.
// In host code this name is only a handle for hipGetSymbolAddress, never a device address.
static __device__ __align__(256) unsigned char scratch[MOE_STATIC_SCRATCH_BYTES];

namespace {
thread_local char g_err[512] = "";
}

namespace emoe {
// the message moe_last_error() returns on this thread (shared by every translation unit of the library)
moe_status_t set_error(moe_status_t st, const char *fmt, va_list ap)
{
    vsnprintf(g_err, sizeof g_err, fmt, ap);
    return st;
}
}  // namespace emoe

namespace {

moe_status_t fail(moe_status_t st, const char *fmt, ...)
{
    va_list ap;
    va_start(ap, fmt);
    set_error(st, fmt, ap);
    va_end(ap);
    return st;
}

constexpr size_t kAlign = 256;
size_t align_up(size_t v) { return (v + kAlign - 1) / kAlign * kAlign; }
constexpr int kMinTileRows = 16;  // smallest M-tile any expert kernel uses: sizes the tile list

// Offsets of every intermediate inside the workspace.
struct Layout {
    size_t map, logits, ids, w, slot_rank, blk_hist, blk_cnt, counts, offs, perm, inv, tiles, n_tiles, units[2], unit_hdr, h, y, partials, total;
    size_t unit_cap, logit_tokens;
    bool has_partials;
};

size_t esize(int dtype) { return dtype == MOE_BF16 ? 2 : 4; }

moe_status_t check_config(const moe_config_t *c)
{
    if (!c) return fail(MOE_ERR_ARG, "config is NULL");
    if (c->hidden <= 0 || c->inter <= 0 || c->n_experts <= 0 || c->top_k <= 0 || c->n_slots <= 0 || c->max_tokens <= 0)
        return fail(MOE_ERR_SHAPE, "hidden, inter, n_experts, top_k, n_slots, max_tokens must all be positive");
    if (c->act_dtype != MOE_F32 && c->act_dtype != MOE_BF16) return fail(MOE_ERR_ARG, "act_dtype %d is not a moe_dtype_t", c->act_dtype);
    if (c->router_dtype != MOE_F32 && c->router_dtype != MOE_BF16) return fail(MOE_ERR_ARG, "router_dtype %d is not a moe_dtype_t", c->router_dtype);
    if (c->gate != MOE_GATE_SOFTMAX_TOPK && c->gate != MOE_GATE_SIGMOID_GROUP_TOPK) return fail(MOE_ERR_ARG, "gate %d is not a moe_gate_t", c->gate);
    if (c->n_shared < 0 || c->n_group <= 0 || c->topk_group <= 0) return fail(MOE_ERR_SHAPE, "n_shared >= 0, n_group >= 1, topk_group >= 1 required");
    if (c->top_k > c->n_experts) return fail(MOE_ERR_SHAPE, "top_k %d exceeds n_experts %d", c->top_k, c->n_experts);
    if (c->n_experts % c->n_group) return fail(MOE_ERR_SHAPE, "n_group %d does not divide n_experts %d", c->n_group, c->n_experts);
    if (c->topk_group > c->n_group) return fail(MOE_ERR_SHAPE, "topk_group %d exceeds n_group %d", c->topk_group, c->n_group);
    if (c->gate == MOE_GATE_SOFTMAX_TOPK && (c->n_group != 1 || c->topk_group != 1))
        return fail(MOE_ERR_SHAPE, "the softmax gate has no groups: n_group and topk_group must be 1");
    if ((long long)c->top_k > (long long)c->topk_group * (c->n_experts / c->n_group))
        return fail(MOE_ERR_SHAPE, "top_k %d exceeds the %d experts of %d kept groups", c->top_k, c->topk_group * (c->n_experts / c->n_group), c->topk_group);
    if (c->n_shared > c->n_slots) return fail(MOE_ERR_SHAPE, "n_shared %d exceeds n_slots %d", c->n_shared, c->n_slots);
    if (!(c->routed_scale == c->routed_scale)) return fail(MOE_ERR_ARG, "routed_scale is NaN");
    if (c->hidden % 8 || c->inter % 8) return fail(MOE_ERR_UNSUPPORTED, "hidden and inter must be multiples of 8 (16-byte rows)");
    if (c->n_experts > 1024) return fail(MOE_ERR_UNSUPPORTED, "n_experts > 1024");
    if (c->top_k > 32) return fail(MOE_ERR_UNSUPPORTED, "top_k > 32");
    if (c->n_group > 64) return fail(MOE_ERR_UNSUPPORTED, "n_group > 64");
    if (c->n_shared > 4) return fail(MOE_ERR_UNSUPPORTED, "n_shared > 4");
    if (c->n_slots > 2047) return fail(MOE_ERR_UNSUPPORTED, "n_slots > 2047");
    if ((long long)c->max_tokens * (c->top_k + c->n_shared) > (1ll << 26))
        return fail(MOE_ERR_UNSUPPORTED, "max_tokens * (top_k + n_shared) > 2^26");
    return MOE_OK;
}

// tight: where the size is fixed and the pass would not fit otherwise (moe_forward_static) -- the logits of an fp32
// layer share the memory of what is written after the selection has read them, as many tokens at a time as that
// holds, and the large-tile GEMMs serve small groups no more (no unit lists)
Layout make_layout(const moe_config_t &c, bool tight = false)
{
    Layout L;
    const size_t T = c.max_tokens, k = c.top_k, kk = c.top_k + c.n_shared, S = c.n_slots;
    const size_t A = T * kk;
    const size_t nb = (A + kAssignPerBlock - 1) / kAssignPerBlock;
    const size_t max_tiles = (A + kMinTileRows - 1) / kMinTileRows + S;
    size_t o = 0;
    auto take = [&](size_t bytes) { size_t at = o; o = align_up(o + bytes); return at; };
    // a table: E + n_shared entries, then the copy lists of replicated experts (count, slots...:
    // at most S slots in lists of at least two, so 3S/2 entries)
    L.map = take(4 * (c.n_experts + c.n_shared + 2 * S));
    // partial-sum planes of the K-split logits kernels (fp32 layers: only few tokens have several)
    size_t planes_of_tokens = T * kGatePlanes;
    if (c.act_dtype == MOE_F32) {
        const size_t few = T < (size_t)kGateFewTokens ? T : (size_t)kGateFewTokens;
        planes_of_tokens = few * gate_f32_planes((int)few, c.hidden) > T ? few * gate_f32_planes((int)few, c.hidden) : T;
    }
    const bool shared_logits = tight && c.act_dtype == MOE_F32;
    L.logits = take(shared_logits ? 0 : 4 * planes_of_tokens * c.n_experts);
    L.logit_tokens = planes_of_tokens;
    L.ids = take(4 * T * k);
    L.w = take(4 * T * k);
    L.slot_rank = take(4 * A);
    // block words of the bookkeeping: [blocks of 1024 assignments][S], or (fused with the selection) [S][blocks of 16 tokens]
    const size_t nbf = ((T < (size_t)kFusedMaxTokens ? T : (size_t)kFusedMaxTokens) + kFusedTokens - 1) / kFusedTokens;
    const size_t fused_words = (size_t)fused_row_stride((int)nbf) * S;
    L.blk_hist = take(4 * (nb * S > fused_words ? nb * S : fused_words));
    L.blk_cnt = take(fused_words);
    L.counts = take(4 * S);
    L.offs = take(4 * (S + 1));
    L.perm = take(4 * A);
    L.inv = take(4 * A);
    L.tiles = take(sizeof(MTile) * max_tiles);
    L.n_tiles = take(4);
    // unit lists of the large-tile GEMMs (layers they can serve): one entry per (tile, run of N-slices), in rows of 8
    L.unit_cap = 0;
    if (c.act_dtype == MOE_BF16 && c.hidden % 64 == 0 && c.inter % 64 == 0 && (!tight || A >= 48 * S)) {
        const size_t big_tiles = (A + mfma8_tile_rows() - 1) / mfma8_tile_rows() + S;
        const int ns0 = mfma8_n_slices(c.hidden, c.inter, 0), ns1 = mfma8_n_slices(c.hidden, c.inter, 1);
        L.unit_cap = 8 * (size_t)mfma8_grid_rows((int)big_tiles, ns0 > ns1 ? ns0 : ns1);
    }
    L.units[0] = take(sizeof(MUnit) * L.unit_cap);
    L.units[1] = take(sizeof(MUnit) * L.unit_cap);
    L.unit_hdr = take(L.unit_cap ? 2 * sizeof(UnitHdr) : 0);
    L.h = take(esize(c.act_dtype) * A * c.inter);
    L.y = take(esize(c.act_dtype) * A * c.hidden);
    // partial sums of split tiles: only layers whose large-tile GEMMs can have contractions long enough to split
    L.has_partials = c.act_dtype == MOE_BF16 && c.hidden % 64 == 0 && c.inter % 64 == 0 && (c.hidden >= 4096 || c.inter >= 4096) &&
                     A >= 48 * S;
    L.partials = take(L.has_partials ? mfma8_partial_bytes() : 0);
    if (shared_logits) {
        L.logits = L.perm;
        L.logit_tokens = (o - L.perm) / (4 * (size_t)c.n_experts);
    }
    L.total = o;
    return L;
}

bool aligned(const void *p, size_t a) { return ((uintptr_t)p % a) == 0; }

}  // namespace

constexpr int kProfRing = 64;  // forwards whose phase events are kept

struct moe_layer {
    bool prof_on = false;
    long long prof_count = 0;  // forwards recorded since profiling was enabled
    long long prof_seen = 0;   // forwards issued since then
    int prof_every = 1;        // every prof_every-th forward is recorded
    int prof_phase = -1;       // the one phase whose two events are recorded, or -1: all of them
    hipEvent_t ev[kProfRing][MOE_N_PHASES + 1] = {};
    moe_config_t cfg;
    moe_buffers_t buf;
    Layout lay;
    bool has_map;
    std::vector<int32_t> slot_owner;  // per slot: entry (expert, or E + shared expert) of the active table that uses it, or -1
    int slots_used = 0;               // of them, those that are used
    // slot fills that the next map switch has to wait for: one event per copy stream handle, recorded again by every
    // fill on that stream, the entries reused after the switch
    struct Fill { hipEvent_t ev; void *stream; };
    std::vector<Fill> load_ev;
    int n_pending = 0;
    const int32_t *table_arg = nullptr;   // host table of a moe_forward_static pass whose selecting kernel installs it
    hipEvent_t serve_ev = nullptr;  // "work enqueued on the serving stream so far", recorded by a fill that has to wait for it
    // whether a fill asks first if the serving stream has anything left (serve_pending below); a pass or a switch resets it
    std::atomic<bool> ask_serve{false};
    moe_vpool *vpool[2] = {nullptr, nullptr};  // the page pools under w13 and w2 when the layer was told (moe_layer_bind_vpools)
};

namespace emoe {
void layer_drop_vpool(moe_layer *l, const moe_vpool *p)
{
    for (int i = 0; i < 2; ++i)
        if (l->vpool[i] == p) l->vpool[i] = nullptr;
}
}  // namespace emoe

// With page pools bound: slot s must have a page under it in both.
static moe_status_t check_backed(const moe_layer *l, int32_t s, const char *what)
{
    static const char *const name[2] = {"w13", "w2"};
    for (int i = 0; i < 2; ++i)
        if (l->vpool[i] && !vpool_backed(l->vpool[i], s))
            return fail(MOE_ERR_MAP, "%s: slot %d has no page under it in the %s pool", what, s, name[i]);
    return MOE_OK;
}
static moe_status_t check_owned_backed(const moe_layer *l, const std::vector<int32_t> &owner, const char *what)
{
    if (!l->vpool[0] && !l->vpool[1]) return MOE_OK;
    for (int32_t s = 0; s < (int32_t)owner.size(); ++s)
        if (owner[s] >= 0) {
            const moe_status_t st = check_backed(l, s, what);
            if (st != MOE_OK) return st;
        }
    return MOE_OK;
}

extern "C" {

const char *moe_last_error(void) { return g_err; }

size_t moe_workspace_bytes(const moe_config_t *cfg)
{
    if (check_config(cfg) != MOE_OK) return 0;
    return make_layout(*cfg).total;
}

moe_status_t moe_layer_create(const moe_config_t *cfg, const moe_buffers_t *buf, moe_layer_t **out)
{
    if (!out) return fail(MOE_ERR_ARG, "out is NULL");
    *out = nullptr;
    moe_status_t st = check_config(cfg);
    if (st != MOE_OK) return st;
    if (!buf) return fail(MOE_ERR_ARG, "buffers is NULL");
    if (!buf->router_w || !buf->w13 || !buf->w2 || !buf->workspace)
        return fail(MOE_ERR_ARG, "router_w, w13, w2 and workspace must be non-NULL");
    if (!aligned(buf->router_w, 16) || !aligned(buf->w13, 16) || !aligned(buf->w2, 16))
        return fail(MOE_ERR_ARG, "router_w, w13 and w2 must be 16-byte aligned");
    if (!aligned(buf->workspace, kAlign)) return fail(MOE_ERR_ARG, "workspace must be 256-byte aligned");
    if ((buf->logit_bias && !aligned(buf->logit_bias, 4)) || (buf->select_bias && !aligned(buf->select_bias, 4)))
        return fail(MOE_ERR_ARG, "bias vectors must be 4-byte aligned");
    Layout L = make_layout(*cfg);
    if (buf->workspace_bytes < L.total)
        return fail(MOE_ERR_CAPACITY, "workspace has %zu bytes, layer needs %zu", buf->workspace_bytes, L.total);
    moe_layer *l = new (std::nothrow) moe_layer;
    if (!l) return fail(MOE_ERR_ARG, "out of host memory");
    l->cfg = *cfg;
    l->buf = *buf;
    l->lay = L;
    l->has_map = false;
    *out = l;
    return MOE_OK;
}

moe_status_t moe_ceiling_mfma(int32_t blocks, int32_t iters, int32_t random_operands, float *sink, void *hip_stream, double *flops)
{
    if (blocks <= 0 || iters <= 0 || !sink || !flops) return fail(MOE_ERR_ARG, "blocks and iters must be positive, sink and flops non-NULL");
    if (blocks > (1 << 20) || iters > (1 << 24)) return fail(MOE_ERR_ARG, "blocks <= 2^20 and iters <= 2^24");
    *flops = ceiling_mfma_flops(blocks, iters);
    const hipError_t e = launch_ceiling_mfma(blocks, iters, random_operands, sink, (hipStream_t)hip_stream);
    if (e != hipSuccess) return fail(MOE_ERR_HIP, "ceiling launch failed: %s", hipGetErrorString(e));
    return MOE_OK;
}

moe_status_t moe_ceiling_stream(const void *buf, size_t bytes, float *sink, void *hip_stream)
{
    if (!buf || !sink || bytes < 16) return fail(MOE_ERR_ARG, "buf and sink must be non-NULL and bytes >= 16");
    if (!aligned(buf, 16)) return fail(MOE_ERR_ARG, "buf must be 16-byte aligned");
    const hipError_t e = launch_ceiling_stream(buf, bytes, sink, (hipStream_t)hip_stream);
    if (e != hipSuccess) return fail(MOE_ERR_HIP, "ceiling launch failed: %s", hipGetErrorString(e));
    return MOE_OK;
}

moe_status_t moe_ceiling_tile_stream(const void *buf, int32_t n_tiles, size_t row_bytes, int32_t non_temporal, void *hip_stream)
{
    if (!buf || !aligned(buf, 16)) return fail(MOE_ERR_ARG, "buf must be non-NULL and 16-byte aligned");
    if (n_tiles <= 0) return fail(MOE_ERR_ARG, "n_tiles %d is not positive", n_tiles);
    if (row_bytes < 128 || row_bytes % 128 != 0 || row_bytes * 256 >= ((size_t)1 << 32))
        return fail(MOE_ERR_ARG, "row_bytes %zu must be a multiple of 128 below 2^24", row_bytes);
    const hipError_t e = launch_ceiling_tile_stream(buf, n_tiles, row_bytes, non_temporal, (hipStream_t)hip_stream);
    if (e != hipSuccess) return fail(MOE_ERR_HIP, "ceiling launch failed: %s", hipGetErrorString(e));
    return MOE_OK;
}

void moe_layer_destroy(moe_layer_t *layer)
{
    if (!layer) return;
    if (layer->prof_on) moe_profile_enable(layer, 0);
    for (const moe_layer::Fill &f : layer->load_ev) (void)hipEventDestroy(f.ev);
    if (layer->serve_ev) (void)hipEventDestroy(layer->serve_ev);
    for (int i = 0; i < 2; ++i)
        if (layer->vpool[i]) vpool_unbind(layer->vpool[i], layer);
    delete layer;
}

moe_status_t moe_profile_enable(moe_layer_t *l, int32_t enable)
{
    if (!l) return fail(MOE_ERR_ARG, "layer is NULL");
    if (enable < 0) return fail(MOE_ERR_ARG, "enable %d is negative", enable);
    if (enable && l->prof_on) {   // only the sampling changes
        l->prof_every = enable;
        l->prof_seen = 0;          // the next forward is recorded
        return MOE_OK;
    }
    if ((enable != 0) == l->prof_on) return MOE_OK;
    if (enable) {
        for (int i = 0; i < kProfRing; ++i)
            for (int j = 0; j <= MOE_N_PHASES; ++j) {
                hipError_t e = hipEventCreate(&l->ev[i][j]);
                if (e != hipSuccess) {
                    for (int a = 0; a <= i; ++a)
                        for (int b = 0; b <= MOE_N_PHASES; ++b)
                            if (l->ev[a][b]) { (void)hipEventDestroy(l->ev[a][b]); l->ev[a][b] = nullptr; }
                    return fail(MOE_ERR_HIP, "hipEventCreate: %s", hipGetErrorString(e));
                }
            }
        l->prof_count = 0;
        l->prof_seen = 0;
        l->prof_every = enable;
        l->prof_on = true;
    } else {
        for (int i = 0; i < kProfRing; ++i)
            for (int j = 0; j <= MOE_N_PHASES; ++j)
                if (l->ev[i][j]) { (void)hipEventDestroy(l->ev[i][j]); l->ev[i][j] = nullptr; }
        l->prof_on = false;
    }
    return MOE_OK;
}

moe_status_t moe_profile_select(moe_layer_t *l, int32_t phase)
{
    if (!l) return fail(MOE_ERR_ARG, "layer is NULL");
    if (phase < -1 || phase >= MOE_N_PHASES) return fail(MOE_ERR_ARG, "phase %d is outside [-1, %d)", phase, MOE_N_PHASES);
    l->prof_phase = phase;
    l->prof_count = 0;         // recordings made under another selection cannot be read as this one
    l->prof_seen = 0;
    return MOE_OK;
}

moe_status_t moe_profile_read(moe_layer_t *l, int32_t back, float *ms)
{
    if (!l || !ms) return fail(MOE_ERR_ARG, "layer or ms is NULL");
    if (!l->prof_on) return fail(MOE_ERR_ARG, "profiling is not enabled on this layer");
    if (back < 0 || back >= kProfRing || back >= l->prof_count)
        return fail(MOE_ERR_ARG, "no recorded forward %d steps back (recorded %lld, kept %d)", back, l->prof_count, kProfRing);
    hipEvent_t *ev = l->ev[(l->prof_count - 1 - back) % kProfRing];
    const int sel = l->prof_phase;
    hipError_t e = hipEventSynchronize(ev[sel < 0 ? MOE_N_PHASES : sel + 1]);
    if (e != hipSuccess) return fail(MOE_ERR_HIP, "hipEventSynchronize: %s", hipGetErrorString(e));
    for (int j = 0; j < MOE_N_PHASES; ++j) {
        ms[j] = 0.f;
        if (sel >= 0 && j != sel) continue;
        e = hipEventElapsedTime(&ms[j], ev[j], ev[j + 1]);
        if (e != hipSuccess) return fail(MOE_ERR_HIP, "hipEventElapsedTime: %s", hipGetErrorString(e));
    }
    return MOE_OK;
}

namespace {

int slots_in_use(const int32_t *owner, int n)
{
    int used = 0;
    for (int s = 0; s < n; ++s) used += owner[s] >= 0;
    return used;
}

// Validated placement -> the device table.  There is ONE table at a fixed address, rewritten in place by a
// kernel on hip_stream: passes enqueued on that stream before the switch have read it by then, passes after it
// (a replay of a captured graph included: the table's address is all a captured pass holds) read the new one.
moe_status_t install_table(moe_layer_t *l, std::vector<int32_t> &table, std::vector<int32_t> &owner, void *hip_stream)
{
    int32_t *dst = (int32_t *)((char *)l->buf.workspace + l->lay.map);
    const moe_status_t backed = check_owned_backed(l, owner, "the placement names a slot that cannot be read");
    if (backed != MOE_OK) return backed;
    hipError_t e = hipSuccess;
    // slot fills enqueued by moe_load_expert: everything after this switch on hip_stream sees them complete
    for (int i = 0; i < l->n_pending && e == hipSuccess; ++i) e = hipStreamWaitEvent((hipStream_t)hip_stream, l->load_ev[i].ev, 0);
    if (e != hipSuccess) return fail(MOE_ERR_HIP, "waiting for slot fills failed: %s", hipGetErrorString(e));
    l->n_pending = 0;
    e = launch_write_map(dst, table.data(), (int)table.size(), (hipStream_t)hip_stream);
    if (e != hipSuccess) return fail(MOE_ERR_HIP, "expert map upload failed: %s", hipGetErrorString(e));
    l->has_map = true;
    l->ask_serve.store(false, std::memory_order_relaxed);
    l->slot_owner.swap(owner);
    l->slots_used = slots_in_use(l->slot_owner.data(), l->cfg.n_slots);
    return MOE_OK;
}

// entry `who` (expert e, or E + shared expert) claims slot s
moe_status_t claim_slot(const moe_config_t &c, std::vector<int32_t> &owner, int32_t s, int who)
{
    const bool shared = who >= c.n_experts;
    if (s < 0 || s >= c.n_slots)
        return fail(MOE_ERR_MAP, "%s %d -> slot %d is outside [0, %d)", shared ? "shared expert" : "expert",
                    shared ? who - c.n_experts : who, s, c.n_slots);
    if (owner[s] >= 0) return fail(MOE_ERR_MAP, "slot %d is claimed twice (entries %d and %d)", s, owner[s], who);
    owner[s] = who;
    return MOE_OK;
}

}  // namespace

// Checks a plain placement (at most one slot per expert) and writes its device table (E + n_shared
// entries) and the slot -> entry index (S entries) into caller-provided arrays.
static moe_status_t validate_plain_map(const moe_config_t &c, const int32_t *host_map, int32_t n, const int32_t *host_shared_slots,
                                       int32_t *table, int32_t *owner)
{
    if (!host_map) return fail(MOE_ERR_ARG, "host_map is NULL");
    if (n != c.n_experts) return fail(MOE_ERR_MAP, "map has %d entries, layer has %d logical experts", n, c.n_experts);
    if ((c.n_shared > 0) != (host_shared_slots != nullptr))
        return fail(MOE_ERR_MAP, "host_shared_slots must be given exactly when n_shared > 0");
    for (int s = 0; s < c.n_slots; ++s) owner[s] = -1;
    for (int e = 0; e < c.n_experts + c.n_shared; ++e) {
        const bool shared = e >= c.n_experts;
        const int32_t s = shared ? host_shared_slots[e - c.n_experts] : host_map[e];
        if (s < -1 || (shared && s < 0))
            return fail(MOE_ERR_MAP, "%s %d -> slot %d is outside [%s, %d)", shared ? "shared expert" : "expert",
                        shared ? e - c.n_experts : e, s, shared ? "0" : "-1", c.n_slots);
        if (s >= 0) {
            if (s >= c.n_slots)
                return fail(MOE_ERR_MAP, "%s %d -> slot %d is outside [0, %d)", shared ? "shared expert" : "expert",
                            shared ? e - c.n_experts : e, s, c.n_slots);
            if (owner[s] >= 0) return fail(MOE_ERR_MAP, "slot %d is claimed twice (entries %d and %d)", s, owner[s], e);
            owner[s] = e;
        }
        table[e] = s;
    }
    return MOE_OK;
}

moe_status_t moe_set_expert_map(moe_layer_t *l, const int32_t *host_map, int32_t n,
                                const int32_t *host_shared_slots, void *hip_stream)
{
    if (!l) return fail(MOE_ERR_ARG, "layer is NULL");
    const moe_config_t &c = l->cfg;
    std::vector<int32_t> owner(c.n_slots, -1);  // slot -> entry index that claimed it
    std::vector<int32_t> table(c.n_experts + c.n_shared);
    const moe_status_t st = validate_plain_map(c, host_map, n, host_shared_slots, table.data(), owner.data());
    if (st != MOE_OK) return st;
    return install_table(l, table, owner, hip_stream);
}

moe_status_t moe_set_expert_replicas(moe_layer_t *l, const int32_t *host_rep_offsets, const int32_t *host_rep_slots,
                                     int32_t n, const int32_t *host_shared_slots, void *hip_stream)
{
    if (!l) return fail(MOE_ERR_ARG, "layer is NULL");
    if (!host_rep_offsets) return fail(MOE_ERR_ARG, "host_rep_offsets is NULL");
    const moe_config_t &c = l->cfg;
    if (n != c.n_experts) return fail(MOE_ERR_MAP, "placement has %d experts, layer has %d logical experts", n, c.n_experts);
    if ((c.n_shared > 0) != (host_shared_slots != nullptr))
        return fail(MOE_ERR_MAP, "host_shared_slots must be given exactly when n_shared > 0");
    if (host_rep_offsets[0] != 0) return fail(MOE_ERR_MAP, "host_rep_offsets[0] is %d, must be 0", host_rep_offsets[0]);
    for (int e = 0; e < n; ++e)
        if (host_rep_offsets[e + 1] < host_rep_offsets[e] || host_rep_offsets[e + 1] > c.n_slots)
            return fail(MOE_ERR_MAP, "host_rep_offsets must be non-decreasing and end at no more than n_slots = %d (entry %d is %d)",
                        c.n_slots, e + 1, host_rep_offsets[e + 1]);
    if (host_rep_offsets[n] > 0 && !host_rep_slots) return fail(MOE_ERR_ARG, "host_rep_slots is NULL");
    std::vector<int32_t> owner(c.n_slots, -1);
    std::vector<int32_t> table(c.n_experts + c.n_shared);
    for (int e = 0; e < n; ++e) {
        const int b = host_rep_offsets[e], R = host_rep_offsets[e + 1] - b;
        for (int r = 0; r < R; ++r) {
            const moe_status_t st = claim_slot(c, owner, host_rep_slots[b + r], e);
            if (st != MOE_OK) return st;
        }
        if (R == 0) {
            table[e] = -1;
        } else if (R == 1) {
            table[e] = host_rep_slots[b];
        } else {
            // the copy list (count, slots) goes behind the E + n_shared entries; the entry encodes where
            table[e] = -2 - (int32_t)(table.size() - (size_t)(c.n_experts + c.n_shared));
            table.push_back(R);
            for (int r = 0; r < R; ++r) table.push_back(host_rep_slots[b + r]);
        }
    }
    for (int i = 0; i < c.n_shared; ++i) {
        const moe_status_t st = claim_slot(c, owner, host_shared_slots[i], c.n_experts + i);
        if (st != MOE_OK) return st;
        table[c.n_experts + i] = host_shared_slots[i];
    }
    return install_table(l, table, owner, hip_stream);
}

moe_status_t moe_layer_bind_vpools(moe_layer_t *l, moe_vpool_t *w13_pool, moe_vpool_t *w2_pool)
{
    if (!l) return fail(MOE_ERR_ARG, "layer is NULL");
    const moe_config_t &c = l->cfg;
    const size_t es = esize(c.act_dtype);
    const size_t want[2] = {2 * (size_t)c.inter * c.hidden * es, (size_t)c.hidden * c.inter * es};
    moe_vpool_t *pool[2] = {w13_pool, w2_pool};
    const void *base[2] = {l->buf.w13, l->buf.w2};
    static const char *const name[2] = {"w13", "w2"};
    for (int i = 0; i < 2; ++i) {
        if (!pool[i]) continue;
        if (moe_vpool_base(pool[i]) != base[i]) return fail(MOE_ERR_ARG, "the %s pool does not start where the layer's %s does", name[i], name[i]);
        if (moe_vpool_slot_bytes(pool[i]) != want[i])
            return fail(MOE_ERR_ARG, "the %s pool has slots of %zu bytes, the layer's are %zu", name[i], moe_vpool_slot_bytes(pool[i]), want[i]);
        if (moe_vpool_slots(pool[i]) < c.n_slots)
            return fail(MOE_ERR_ARG, "the %s pool has %d slots, the layer has %d", name[i], moe_vpool_slots(pool[i]), c.n_slots);
    }
    moe_vpool *old[2] = {l->vpool[0], l->vpool[1]};
    l->vpool[0] = w13_pool;
    l->vpool[1] = w2_pool;
    if (l->has_map) {   // the placement in force must already be readable
        const moe_status_t st = check_owned_backed(l, l->slot_owner, "the active placement names a slot that cannot be read");
        if (st != MOE_OK) { l->vpool[0] = old[0]; l->vpool[1] = old[1]; return st; }
    }
    for (int i = 0; i < 2; ++i) {
        if (old[i] && old[i] != l->vpool[i]) vpool_unbind(old[i], l);
        if (l->vpool[i]) vpool_bind(l->vpool[i], l);
    }
    return MOE_OK;
}

// Whether a fill has to wait for work enqueued on the serving stream.  Making another stream wait for a pending event takes the
// host 12 us, asking the stream whether it is idle 0.2 (32 fills and two forwards of the Qwen3-shaped rank 950 -> 740 us, 64 tokens 900 -> 425), unless it has
// work that the runtime has not been asked about, which takes 17: so the first fill behind a pass or a switch of this layer
// does not ask, and neither does one after an answer that took long (somebody else's work between the fills).  The question is put in
// the relaxed capture mode: in the others it would end a graph capture under way on some other stream.  Capturing streams are
// not asked: their fill becomes part of the graph by the event, or is refused.
static bool serve_pending(moe_layer *l, hipStream_t serve, hipStream_t copy)
{
    if (!l->ask_serve.exchange(true, std::memory_order_relaxed)) return true;
    hipStreamCaptureStatus cs[2] = {hipStreamCaptureStatusActive, hipStreamCaptureStatusActive};
    if (hipStreamIsCapturing(serve, &cs[0]) != hipSuccess || hipStreamIsCapturing(copy, &cs[1]) != hipSuccess) return true;
    if (cs[0] != hipStreamCaptureStatusNone || cs[1] != hipStreamCaptureStatusNone) return true;
    hipStreamCaptureMode mode = hipStreamCaptureModeRelaxed;
    if (hipThreadExchangeStreamCaptureMode(&mode) != hipSuccess) return true;
    const auto start = std::chrono::steady_clock::now();
    const hipError_t q = hipStreamQuery(serve);
    if (std::chrono::steady_clock::now() - start > std::chrono::microseconds(5)) l->ask_serve.store(false, std::memory_order_relaxed);
    (void)hipThreadExchangeStreamCaptureMode(&mode);
    return q != hipSuccess;
}

moe_status_t moe_load_expert(moe_layer_t *l, int32_t slot, const void *src_w13, const void *src_w2,
                             void *copy_stream, void *serve_stream, int32_t copy_blocks)
{
    if (!l) return fail(MOE_ERR_ARG, "layer is NULL");
    const moe_config_t &c = l->cfg;
    if (slot < 0 || slot >= c.n_slots) return fail(MOE_ERR_ARG, "slot %d is outside [0, %d)", slot, c.n_slots);
    if (!src_w13 || !src_w2) return fail(MOE_ERR_ARG, "src_w13 and src_w2 must be non-NULL");
    if (!aligned(src_w13, 16) || !aligned(src_w2, 16)) return fail(MOE_ERR_ARG, "src_w13 and src_w2 must be 16-byte aligned");
    if (copy_blocks < 0 || copy_blocks > 65536) return fail(MOE_ERR_ARG, "copy_blocks %d is outside [0, 65536]", copy_blocks);
    if (copy_stream == serve_stream) return fail(MOE_ERR_ARG, "copy_stream and serve_stream must differ (the fill is meant to run beside the forwards)");
    if (l->has_map && l->slot_owner[slot] >= 0) {
        const int e = l->slot_owner[slot];
        return fail(MOE_ERR_MAP, "slot %d holds %s %d of the active map: it cannot be refilled while forwards may read it", slot,
                    e >= c.n_experts ? "shared expert" : "expert", e >= c.n_experts ? e - c.n_experts : e);
    }
    const moe_status_t backed = check_backed(l, slot, "the fill would write memory that is not there");
    if (backed != MOE_OK) return backed;
    hipError_t e = hipSuccess;
    if (!l->serve_ev) e = hipEventCreateWithFlags(&l->serve_ev, hipEventDisableTiming);
    int at = 0;
    while (at < l->n_pending && l->load_ev[at].stream != copy_stream) ++at;
    if (e == hipSuccess && at == (int)l->load_ev.size()) {
        moe_layer::Fill f = {nullptr, nullptr};
        e = hipEventCreateWithFlags(&f.ev, hipEventDisableTiming);
        if (e == hipSuccess) l->load_ev.push_back(f);
    }
    if (e != hipSuccess) return fail(MOE_ERR_HIP, "hipEventCreate: %s", hipGetErrorString(e));
    // a forward already enqueued on the serving stream may still read the slot under an older map
    if (serve_pending(l, (hipStream_t)serve_stream, (hipStream_t)copy_stream)) {
        e = hipEventRecord(l->serve_ev, (hipStream_t)serve_stream);
        if (e == hipSuccess) e = hipStreamWaitEvent((hipStream_t)copy_stream, l->serve_ev, 0);
    }
    const size_t es = esize(c.act_dtype);
    const size_t b13 = 2 * (size_t)c.inter * c.hidden * es, b2 = (size_t)c.hidden * c.inter * es;
    if (e == hipSuccess)
        e = launch_fill_slot((char *)const_cast<void *>(l->buf.w13) + (size_t)slot * b13, src_w13, b13,
                             (char *)const_cast<void *>(l->buf.w2) + (size_t)slot * b2, src_w2, b2, copy_blocks, (hipStream_t)copy_stream);
    // the event is about to stand for this fill alone: the one it stood for comes first.  (On one stream it does
    // anyway; a handle can also name another stream by now, a destroyed one's successor or another thread's own.)
    if (e == hipSuccess && at < l->n_pending) e = hipStreamWaitEvent((hipStream_t)copy_stream, l->load_ev[at].ev, 0);
    if (e == hipSuccess) e = hipEventRecord(l->load_ev[at].ev, (hipStream_t)copy_stream);
    if (e != hipSuccess) return fail(MOE_ERR_HIP, "slot fill failed: %s", hipGetErrorString(e));
    l->load_ev[at].stream = copy_stream;
    if (at == l->n_pending) l->n_pending++;
    return MOE_OK;
}

moe_status_t moe_workspace_view(const moe_layer_t *l, moe_workspace_view_t *v)
{
    if (!l || !v) return fail(MOE_ERR_ARG, "layer or view is NULL");
    char *ws = (char *)l->buf.workspace;
    v->topk_ids = (const int32_t *)(ws + l->lay.ids);
    v->topk_w = (const float *)(ws + l->lay.w);
    v->counts = (const int32_t *)(ws + l->lay.counts);
    v->offsets = (const int32_t *)(ws + l->lay.offs);
    v->perm = (const int32_t *)(ws + l->lay.perm);
    v->inv = (const int32_t *)(ws + l->lay.inv);
    v->h = ws + l->lay.h;
    v->y = ws + l->lay.y;
    v->active_map = (const int32_t *)(ws + l->lay.map);
    v->tiles = (const int32_t *)(ws + l->lay.tiles);
    v->n_tiles = (const int32_t *)(ws + l->lay.n_tiles);
    v->unit_hdr = l->lay.unit_cap ? (const int32_t *)(ws + l->lay.unit_hdr) : nullptr;
    v->units[0] = l->lay.unit_cap ? (const int32_t *)(ws + l->lay.units[0]) : nullptr;
    v->units[1] = l->lay.unit_cap ? (const int32_t *)(ws + l->lay.units[1]) : nullptr;
    return MOE_OK;
}

// One pass; routed_ids/routed_w non-NULL: the gate is skipped and the caller's routing is read in place.
static moe_status_t forward_pass(moe_layer_t *l, const void *x, int32_t T, const int32_t *routed_ids, const float *routed_w,
                                 int32_t shared_begin, int32_t shared_end, void *out, void *hip_stream, uint32_t flags)
{
    if (!l) return fail(MOE_ERR_ARG, "layer is NULL");
    const moe_config_t &c = l->cfg;
    if (T < 0) return fail(MOE_ERR_ARG, "T is negative");
    if (T > c.max_tokens) return fail(MOE_ERR_CAPACITY, "T %d exceeds max_tokens %d", T, c.max_tokens);
    if (shared_begin < 0 || shared_begin > shared_end || shared_end > T)
        return fail(MOE_ERR_ARG, "shared range [%d,%d) is not inside [0,%d]", shared_begin, shared_end, T);
    if (flags & ~(MOE_FLAG_IDENTITY_EXPERTS | MOE_FLAG_FORCE_GENERIC | MOE_FLAG_GATE_TILED | MOE_FLAG_PERMUTE_UNFUSED)) return fail(MOE_ERR_ARG, "unknown flag bits 0x%x", flags);
    if (!l->has_map) return fail(MOE_ERR_MAP, "no expert map installed: call moe_set_expert_map first");
    {   // page pools bound: a page taken from under a slot of the placement in force would fault the pass
        const moe_status_t backed = check_owned_backed(l, l->slot_owner, "the active placement names a slot whose page is gone");
        if (backed != MOE_OK) return backed;
    }
    if (T == 0) return MOE_OK;
    if (!x || !out) return fail(MOE_ERR_ARG, "x and out must be non-NULL");
    if (!aligned(x, 16) || !aligned(out, 16)) return fail(MOE_ERR_ARG, "x and out must be 16-byte aligned");

    hipStream_t st = (hipStream_t)hip_stream;
    l->ask_serve.store(false, std::memory_order_relaxed);
    char *ws = (char *)l->buf.workspace;
    Pass p;
    memset(&p, 0, sizeof p);
    p.T = T; p.H = c.hidden; p.I = c.inter; p.E = c.n_experts; p.k = c.top_k; p.S = c.n_slots;
    p.n_shared = c.n_shared; p.kk = c.top_k + c.n_shared;
    p.act_bf16 = c.act_dtype == MOE_BF16; p.router_bf16 = c.router_dtype == MOE_BF16;
    p.gate = c.gate; p.n_group = c.n_group; p.topk_group = c.topk_group; p.renormalize = c.renormalize;
    p.routed_scale = c.routed_scale;
    p.shared_begin = shared_begin; p.shared_end = shared_end;
    p.x = x; p.out = out;
    p.router_w = l->buf.router_w; p.logit_bias = l->buf.logit_bias; p.select_bias = l->buf.select_bias;
    p.w13 = l->buf.w13; p.w2 = l->buf.w2;
    p.map = (const int32_t *)(ws + l->lay.map);
    p.logits = (float *)(ws + l->lay.logits);
    p.logit_planes = 1;
    p.logit_tokens = (int32_t)l->lay.logit_tokens;
    p.host_table = l->table_arg;
    // the kernels after the gate only read ids and w
    p.ids = routed_ids ? const_cast<int32_t *>(routed_ids) : (int32_t *)(ws + l->lay.ids);
    p.w = routed_w ? const_cast<float *>(routed_w) : (float *)(ws + l->lay.w);
    p.slot_rank = (int32_t *)(ws + l->lay.slot_rank);
    p.blk_hist = (int32_t *)(ws + l->lay.blk_hist);
    p.blk_cnt = (uint8_t *)(ws + l->lay.blk_cnt);
    p.counts = (int32_t *)(ws + l->lay.counts);
    p.offs = (int32_t *)(ws + l->lay.offs);
    p.perm = (int32_t *)(ws + l->lay.perm);
    p.inv = (int32_t *)(ws + l->lay.inv);
    p.tiles = (MTile *)(ws + l->lay.tiles);
    p.n_tiles = (int32_t *)(ws + l->lay.n_tiles);
    p.units[0] = p.units[1] = nullptr;
    p.unit_hdr = nullptr;
    p.h = ws + l->lay.h;
    p.y = ws + l->lay.y;
    p.partials = l->lay.has_partials ? (float *)(ws + l->lay.partials) : nullptr;

    p.gate_tiled = (flags & MOE_FLAG_GATE_TILED) != 0;
    // gated passes up to kFusedMaxTokens tokens: the selection kernel ranks the assignments, one more kernel places them
    p.fused_hist = !routed_ids && T <= kFusedMaxTokens && T <= p.logit_tokens && !(flags & MOE_FLAG_PERMUTE_UNFUSED);
    const bool identity = flags & MOE_FLAG_IDENTITY_EXPERTS;
    const bool mfma = p.act_bf16 && !(flags & MOE_FLAG_FORCE_GENERIC);
    // bf16 passes: small weight-streaming tasks of one token tile when a slot expects only a handful of rows (tiny; routed: T*k/E on
    // average) and of up to 64 rows for a dozen or two (ring64), the large-tile kernels above that (wide, big), the 128 x 128 kernels for
    // small layers, whose time is the bookkeeping, and for contractions that are no whole K-steps.
    // Where ring64 ends (`few`).  Whole pass, us, large tiles or 128 x 128 -> ring64:
    //  * finer tasks and shorter bookkeeping win, the more so the fewer slots there are to fill the chip: Qwen3 shape with 2 local experts,
    //    50 tokens 55 -> 30; 8, 300 tokens 59 -> 46; 32, 140 tokens 96 -> 74; 64, 200 tokens 127 -> 120; 128, 100 tokens 219 -> 214;
    //    24 experts of 1024 x 768, 250 tokens 65 -> 52, of 128 x 128, 40 tokens 24 -> 24;
    //    (with the large tiles' last round in parts and the tiles derived in ring64's GEMM-1, large -> ring64: 8 experts, 310 tokens 42.9 -> 39.3; 16 50.9 -> 45.6; 24 65.4 -> 66.9; 32 73.2 -> 72.1; 64 123.3 ->
    //    119.0; 16 of DeepSeek-V2-Lite, 210 tokens 100.5 -> 90.2; past the line below 16 Qwen3 experts, 400 tokens 51.8 -> 48.4, 24 67.3 -> 68.5);
    //  * what it costs: an even load of 200 or 300 tokens on 32 Qwen3 experts 74.5 -> 75, 75.5 -> 77, of 160 on 24 of them 54 -> 58 (a
    //    Zipf(1.2) one, 310 tokens on 32, 98 -> 68);
    //  * rows of 2560, 3072 and 4096 gain as much: 768 wide, 80 to 300 tokens, 8 local experts -27 to -32 %, 16 -17 to -40 %, 32 0 to
    //    -28 %, 64 -6 to -11 %; 4096 x 1536 -2 to -30 %, an even load on 16 experts +0 to +6 % (Zipf -5 to -17 %).  Rows of 7168 lose at every size
    //    (DeepSeek-V3-shaped rank 140 tokens 489 -> 499, 512 tokens 512 -> 529).  Nothing was measured between, nor with more than 300 MB of
    //    rows shorter than 2048;
    //  * 20 rows a slot, 9 above 800 MB of slots in use: then a skewed load has slots with several chunks of 64 rows, which read their
    //    weights several times (Zipf(1.2): 128 Qwen3 experts, 140 tokens 122 -> 119, 165 tokens 122.5 -> 126, 333 tokens 138 -> 153; an even
    //    load gains 2 % up to 190; with 302 or 604 MB of slots 310 tokens 98 -> 68 and 109 -> 86, 500 tokens 84 -> 68 and 109 -> 110);
    //  * so does a shared expert with many rows: up to 320 of them, one tile of the large kernels (DeepSeek-V2-Lite shape, top-1 to top-6, 16
    //    local experts: 220 shared rows 100 -> 93, 320 of 1280 tokens 122 -> 103, 340 90 -> 98, 640 114.5 -> 117, 1280 125 -> 154; 64
    //    local experts: 150 199 -> 193, 220 209 -> 214, 340 222 -> 219, 640 234 -> 243, 1280 247 -> 293);
    //  * and so does a routed pass (at_once, below).
    // Elsewhere the large tiles serve what has 48 assignments of the whole batch per slot of the layer (a rank of many holds
    // a part of them), and less when there are weights to stream: 400 MB in the slots that the placement uses (32 Qwen3 experts in
    // 128 slots, 420 tokens, 128 x 128 -> large tiles: 94 -> 79, Zipf 83 -> 100).
    const bool can_big = mfma && mfma8_supports(p) && l->lay.unit_cap > 0;
    const long long used_bytes = 6ll * l->slots_used * p.H * p.I;
    const bool large = can_big && ((long long)T * p.kk >= 48ll * p.S || used_bytes >= 400000000ll);   // what the large tiles take unless `few` or `tiny` does
    // A gated pass has T k / E rows for a slot.  Tokens that arrive routed were sent because one of their experts is here: with few of the
    // experts that is many times as much, and several chunks read a slot's weights again.  us, the tokens' experts drawn from all of them, one
    // at least of the local ones:
    //  * ring64 against the large tiles (at_once): up to 24 rows a slot as in a gated pass (Qwen3 shape, 269 tokens on 12 of 64 experts, top-1
    //    53 -> 37; 48 of 256 3072 x 768 experts, top-8, 522 tokens 154 -> 136; 16 of 4096 x 1536 112 -> 112 at 16 rows, 113 -> 128 at 38); above, while
    //    all tasks of GEMM-1 have a place and few large tiles would (an N-slice of 128 columns per slot on less than a third of the chip:
    //    DeepSeek-V2-Lite shape, 1280 tokens on 2 and 4 of 64 experts, top-1, 99 -> 65 and 105 -> 77; 6 of 256 4096 x 1536 experts, top-6, 705
    //    tokens 118 -> 95.5; 4, top-1, 1024 tokens 150 -> 101; on 8 of them 512 tokens 100 -> 113, 1024 120 -> 128; 8 of DeepSeek-V2-Lite, 1280 tokens 76.5 ->
    //    95) or the tasks are fewer still (640 tokens on those 8: 67 -> 63; 372 tokens on 16 Qwen3 experts 52 -> 38).  What that leaves: rows of 1024
    //    would gain further up (24 experts of 1024 x 512, 2525 tokens, 384 tasks 49 -> 43);
    //  * where the large tiles do not take the pass ring64 has no such limit (DeepSeek-V2-Lite shape, 923 tokens on 20 experts, 128 x 128 -> ring64
    //    103 -> 85);
    //  * ring64 against the kernels of one token tile (several), whose register form has tiles of 16 rows: once more of those tasks
    //    are expected than run at a time (2 of 256 4096 x 1536 experts, top-1, 256 tokens 109 -> 58.5, 1024 tokens 404 -> 79, the large tiles 136; 512 tokens on
    //    8 of 128 Qwen3 experts 69 -> 39, on 2 69 -> 37.5; below, 128 tokens on 2 of them, 384 tasks, 30 -> 36).
    const int resident = l->slots_used - p.n_shared < p.E ? l->slots_used - p.n_shared : p.E;
    const double here = routed_ids ? 1.0 - std::pow(1.0 - (double)resident / p.E, p.k) : 1.0;   // share of all tokens that are sent here
    const double rows = resident > 0 ? (double)T * p.k / p.E / here : 0.0;
    const double tasks = std::ceil((rows + 2.0 * std::sqrt(rows)) / ring_tile_rows(true)) * resident * (p.I / 64);
    const bool at_once = rows <= 24.0 || tasks <= 360.0 || (tasks <= 560.0 && resident * (p.I / 128) <= 80);
    const bool few = (at_once || !large) && p.H <= 4096 && (p.H >= 2048 || used_bytes <= 300000000ll) &&
                     (long long)T * p.k <= (used_bytes <= 800000000ll ? 20ll : 9ll) * p.E && shared_end - shared_begin <= mfma8_tile_rows();
    const bool wide = can_big && !few && (long long)T * p.kk >= 48ll * p.S;
    const bool several = few && mfma8_supports(p) && rows > decode_tile_rows() && std::ceil(rows / decode_tile_rows()) * resident * (p.I / 16) > 576.0;
    const bool tiny = mfma && !wide && !several && (long long)T * p.k <= 4ll * p.E && shared_end - shared_begin <= 2 * decode_tile_rows();
    const bool ring64 = mfma && few && !tiny && mfma8_supports(p);
    const bool big = wide || (large && !few && !tiny);
    // Of the small-task kernels the LDS ring streams faster (whole pass, us, registers -> ring: Qwen3 shape 48 tokens 218 ->
    // 197, DeepSeek-V3-shaped rank 64 tokens 464 -> 416) once there are enough of its 128-row tasks for the chip's 256 compute
    // units, counted over the used slots that an even routing gives rows and for GEMM-1, which is two thirds of the bytes;
    // GEMM-2 follows (Qwen3 shape: 139 tasks, 27.7 -> 28.6; 175, 35.6 -> 32.5; 207, 35.1 -> 31.8).  A little more than one
    // task per compute unit is the other exception: a few units then stream two tasks while the rest stand idle (246 tasks,
    // 47.0 -> 51.5; 270, 49.5 -> 52.5; 318, 48.8 -> 52.2; 350, 59.8 -> 56.1).  Rows of 7168 hide that (262 tasks, 181.6 ->
    // 166.2); this exception was not measured between rows of 2048 and of 7168.  The register kernel with its 32-row tasks takes those
    // passes, as it takes contractions that are no whole K-steps.
    const double tiles_expected = resident * (1.0 - std::pow(1.0 - (double)p.k / p.E, T)) + (shared_end > shared_begin ? p.n_shared : 0);
    const double ring_tasks = tiles_expected * (p.I / 64);
    const bool second_round = p.H <= 4096 && ring_tasks >= 240. && ring_tasks < 330.;
    const bool ring = ring64 || (tiny && can_big && ring_tasks >= 160. && !second_round);
    const bool f32 = !p.act_bf16 && !(flags & MOE_FLAG_FORCE_GENERIC);
    enum class Kernels { big, ring, decode, mfma, f32, generic };
    const Kernels kernels = big ? Kernels::big : ring ? Kernels::ring : tiny ? Kernels::decode : mfma ? Kernels::mfma : f32 ? Kernels::f32 : Kernels::generic;
    int tile_rows = 0;
    switch (kernels) {
    case Kernels::big:     tile_rows = mfma8_tile_rows(); break;
    case Kernels::ring:    tile_rows = ring_tile_rows(ring64); break;
    case Kernels::decode:  tile_rows = decode_tile_rows(); break;
    case Kernels::mfma:    tile_rows = mfma_tile_rows(); break;
    case Kernels::f32:     tile_rows = f32_tile_rows(p); break;
    case Kernels::generic: tile_rows = kGenericTileRows; break;
    }
    auto launch_gemm = [&](int which) {
        switch (kernels) {
        case Kernels::big:    return launch_experts_mfma8(p, which, st);
        case Kernels::ring:   return launch_experts_ring(p, tile_rows, which, st);
        case Kernels::decode: return launch_experts_decode(p, which, st);
        case Kernels::mfma:   return launch_experts_mfma(p, which, st);
        case Kernels::f32:    return launch_experts_f32(p, tile_rows, which, st);
        default:              return launch_experts_generic(p, which, st);
        }
    };
    // Upper bound of the tile count, which sizes the grids: every slot with rows adds at most one partly filled
    // tile.  With a token or two most slots have none, and thousands of workgroups that only find out that their
    // tile does not exist take longer to dispatch than one token's experts take to stream.
    const long long assigned = (long long)T * p.k + (long long)(shared_end - shared_begin) * p.n_shared;
    const long long nonempty = assigned < p.S ? assigned : p.S;
    const long long tiles_most = (assigned + tile_rows - 1) / tile_rows + nonempty;
    p.max_tiles = (int)(tiles_most < assigned ? tiles_most : assigned);
    if (big) {   // the tile-list workgroup also deals the tiles' N-slices to the XCDs, per GEMM
        p.units[0] = (MUnit *)(ws + l->lay.units[0]);
        p.units[1] = (MUnit *)(ws + l->lay.units[1]);
        p.unit_hdr = (UnitHdr *)(ws + l->lay.unit_hdr);
        p.unit_cap = (int32_t)l->lay.unit_cap;
        p.n_slices[0] = mfma8_n_slices(p.H, p.I, 0);
        p.n_slices[1] = mfma8_n_slices(p.H, p.I, 1);
        const int most = mfma8_tile_rows();
        p.slot_tiles_expected = (int)std::ceil((rows + 2.0 * std::sqrt(rows)) / most);
        p.tile_rows_expected = p.slot_tiles_expected > 0 ? (int)(rows / p.slot_tiles_expected) : 0;
        p.tiles_expected = (int)(resident * (1.0 - std::exp(-rows)) + 0.5) * p.slot_tiles_expected + p.n_shared * ((shared_end - shared_begin + most - 1) / most);
    }

    // Where out lies on x: every pass writes out behind the last launch that reads x, except those that go token by token.  There a workgroup has read its own
    // row of x before it writes its row of out, but other workgroups may not have read theirs: out may be x itself, and nothing else that meets it.
    const size_t row_bytes = (size_t)T * p.H * esize(c.act_dtype);
    const bool apart = (uintptr_t)x + row_bytes <= (uintptr_t)out || (uintptr_t)out + row_bytes <= (uintptr_t)x;
    const bool whole = !identity && !(flags & MOE_FLAG_FORCE_GENERIC) && (apart || x == out) && token_experts_supports(p);   // GEMM-1, GEMM-2 and combine in one launch, recorded as GEMM-1
    // few tokens: the weight-streaming GEMM-1 (k_token_experts where that is the launch) derives its tiles itself and writes the tables beside its stream
    p.self_tiles = (tiny || f32 || (whole && !big)) && !identity && self_tiles_possible(p);
    // the ring's GEMM-1 for more tokens too (table_blocks workgroups write the tables then)
    if (kernels == Kernels::ring && !whole && !identity && !p.self_tiles) { p.table_blocks = self_table_blocks(p); p.self_tiles = p.table_blocks > 0; }
    // and the gate too, for which all of its workgroups read all token rows
    const bool one_launch = whole && !routed_ids && apart && token_pass_supports(p);
    // a token to four: it selects the experts too
    p.self_select = (kernels == Kernels::decode || (kernels == Kernels::ring && !ring64)) && !whole && !routed_ids &&
                    gemm1_selects(p, kernels == Kernels::decode ? decode_blocks(p) : ring_blocks(p)) && !one_gate_kernel(p);

    // optional phase events (benchmarks): event j is recorded before phase j, the last one after the pass
    hipEvent_t *ev = l->prof_on && l->prof_seen++ % l->prof_every == 0 ? l->ev[l->prof_count % kProfRing] : nullptr;
    hipError_t e = hipSuccess;
    const int sel = l->prof_phase;
    auto mark = [&](int j) { if (ev && e == hipSuccess && (sel < 0 || j == sel || j == sel + 1)) e = hipEventRecord(ev[j], st); };
    mark(MOE_PHASE_GATE);
    if (e == hipSuccess && !routed_ids && !one_launch) e = launch_gate(p, st);
    mark(MOE_PHASE_PERMUTE);
    if (e == hipSuccess && !p.self_tiles) e = launch_permute(p, tile_rows, big, st);   // the large-tile kernels deal a size-ordered list round-robin to the XCDs
    // GEMM-2 and combine in one launch (recorded as GEMM-2): one token, or two where rows are short (whole pass, us, two launches ->
    // one: Qwen3 shape 1 token 36.5 -> 33.9, 2 tokens 44.3 -> 40.9, 3 tokens 64.5 -> 62.5, 4 tokens 69.0 -> 68.8; DeepSeek-V2-Lite
    // shape 38.7 -> 33.3, 62.6 -> 57.2, 4 tokens 77.8 -> 80.5; DeepSeek-V3-shaped rank 41.7 -> 40.2, 78.9 -> 79.5, 4 tokens 89.0 -> 91.0)
    const bool fused2 = !whole && !identity && tiny && T <= (p.H <= 4096 ? 2 : 1);
    mark(MOE_PHASE_GEMM1);
    if (e == hipSuccess) e = one_launch ? launch_token_pass(p, tile_rows, st) : whole ? launch_token_experts(p, tile_rows, st) : identity ? launch_identity_experts(p, st) : launch_gemm(0);
    mark(MOE_PHASE_GEMM2);
    if (e == hipSuccess && !identity && !whole) e = fused2 ? launch_gemm2_combine(p, st) : launch_gemm(1);
    mark(MOE_PHASE_COMBINE);
    if (e == hipSuccess && !whole && !fused2) e = launch_combine(p, st);
    mark(MOE_N_PHASES);
    if (e != hipSuccess) return fail(MOE_ERR_HIP, "forward launch failed: %s", hipGetErrorString(e));
    if (ev) l->prof_count++;
    return MOE_OK;
}

moe_status_t moe_forward(moe_layer_t *layer, const void *x, int32_t T, int32_t shared_begin, int32_t shared_end,
                         void *out, void *hip_stream, uint32_t flags)
{
    return forward_pass(layer, x, T, nullptr, nullptr, shared_begin, shared_end, out, hip_stream, flags);
}

moe_status_t moe_forward_routed(moe_layer_t *layer, const void *x, int32_t T, const int32_t *topk_ids, const float *topk_w,
                                int32_t shared_begin, int32_t shared_end, void *out, void *hip_stream, uint32_t flags)
{
    if (T > 0 && (!topk_ids || !topk_w)) return fail(MOE_ERR_ARG, "topk_ids and topk_w must be non-NULL");
    if (!aligned(topk_ids, 4) || !aligned(topk_w, 4)) return fail(MOE_ERR_ARG, "topk_ids and topk_w must be 4-byte aligned");
    return forward_pass(layer, x, T, topk_ids, topk_w, shared_begin, shared_end, out, hip_stream, flags);
}

// ---- moe_forward_static: the pass with every intermediate in the library's own device array ----

namespace {
constexpr int kMaxDevices = 64;
std::mutex g_scratch_mu;
void *g_scratch_ptr[kMaxDevices] = {};   // device address of `scratch` on each GPU, looked up once per device

// Address of this GPU's copy of `scratch` (the current device's), found once per device.
moe_status_t scratch_of_current_device(void **ptr)
{
    int dev = -1;
    hipError_t e = hipGetDevice(&dev);
    if (e != hipSuccess) return fail(MOE_ERR_HIP, "hipGetDevice: %s", hipGetErrorString(e));
    if (dev < 0 || dev >= kMaxDevices) return fail(MOE_ERR_UNSUPPORTED, "device %d: moe_forward_static keeps scratch addresses for devices 0..%d", dev, kMaxDevices - 1);
    std::lock_guard<std::mutex> lock(g_scratch_mu);
    if (!g_scratch_ptr[dev]) {
        void *p = nullptr;
        e = hipGetSymbolAddress(&p, HIP_SYMBOL(scratch));
        if (e != hipSuccess || !p) return fail(MOE_ERR_HIP, "hipGetSymbolAddress(scratch) on device %d: %s", dev, hipGetErrorString(e));
        g_scratch_ptr[dev] = p;
    }
    *ptr = g_scratch_ptr[dev];
    return MOE_OK;
}
}  // namespace

moe_status_t moe_forward_static(const moe_config_t *cfg, const moe_buffers_t *buf,
                                const int32_t *host_map, int32_t n, const int32_t *host_shared_slots,
                                const void *x, int32_t T, int32_t shared_begin, int32_t shared_end,
                                void *out, void *hip_stream, uint32_t flags)
{
    moe_status_t st = check_config(cfg);
    if (st != MOE_OK) return st;
    if (T < 0) return fail(MOE_ERR_ARG, "T is negative");
    if (T > cfg->max_tokens) return fail(MOE_ERR_CAPACITY, "T %d exceeds max_tokens %d", T, cfg->max_tokens);
    // the workspace is laid out for THIS pass's T (max_tokens only bounds T): what must fit is the pass
    moe_config_t c = *cfg;
    c.max_tokens = T > 0 ? T : 1;
    Layout L = make_layout(c);
    if (L.total > (size_t)MOE_STATIC_SCRATCH_BYTES) L = make_layout(c, true);
    if (L.total > (size_t)MOE_STATIC_SCRATCH_BYTES || L.logit_tokens == 0)
        return fail(MOE_ERR_CAPACITY, "a pass of %d tokens of this layer needs %zu bytes of scratch, moe_forward_static has %zu: "
                    "use moe_forward with a workspace", T, L.total, (size_t)MOE_STATIC_SCRATCH_BYTES);
    if (!buf) return fail(MOE_ERR_ARG, "buffers is NULL");
    if (!buf->router_w || !buf->w13 || !buf->w2) return fail(MOE_ERR_ARG, "router_w, w13 and w2 must be non-NULL");
    if (!aligned(buf->router_w, 16) || !aligned(buf->w13, 16) || !aligned(buf->w2, 16))
        return fail(MOE_ERR_ARG, "router_w, w13 and w2 must be 16-byte aligned");
    if ((buf->logit_bias && !aligned(buf->logit_bias, 4)) || (buf->select_bias && !aligned(buf->select_bias, 4)))
        return fail(MOE_ERR_ARG, "bias vectors must be 4-byte aligned");
    // the placement, checked like moe_set_expert_map does; tables on the host stack (E <= 1024, S <= 2047)
    int32_t table[1024 + 4], owner[2048];
    st = validate_plain_map(c, host_map, n, host_shared_slots, table, owner);
    if (st != MOE_OK) return st;
    if (T == 0) return MOE_OK;

    void *ws = nullptr;
    st = scratch_of_current_device(&ws);
    if (st != MOE_OK) return st;
    moe_layer lay;                       // host object on the stack: no heap, no device memory
    lay.cfg = c;
    lay.buf = *buf;
    lay.buf.workspace = ws;              // kernels get the looked-up device address, never the symbol
    lay.buf.workspace_bytes = MOE_STATIC_SCRATCH_BYTES;
    lay.lay = L;
    lay.has_map = true;
    lay.slots_used = slots_in_use(owner, c.n_slots);
    // every pass writes what it reads (table, histograms, tile list, h, y): nothing has to start at zero
    // the table comes in with the kernel that selects when that kernel ranks the assignments too, or derives the tiles, and it fits an argument
    if (T <= kFusedMaxTokens && T <= (long long)L.logit_tokens && !(flags & MOE_FLAG_PERMUTE_UNFUSED) && c.n_experts + c.n_shared <= kTableArg) {
        lay.table_arg = table;
    } else {
        const hipError_t e = launch_write_map((int32_t *)((char *)ws + L.map), table, c.n_experts + c.n_shared, (hipStream_t)hip_stream);
        if (e != hipSuccess) return fail(MOE_ERR_HIP, "expert map upload failed: %s", hipGetErrorString(e));
    }
    return forward_pass(&lay, x, T, nullptr, nullptr, shared_begin, shared_end, out, hip_stream, flags);
}

}  // extern "C"
