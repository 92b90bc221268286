// Selection of a token's experts by one wavefront, and the look-up of their slots: shared by the selection kernels (k_gate.hip)
// and by the few-token GEMM-1 that selects itself (k_experts_decode.hip, k_experts_ring.hip).  Sec. 2.1 of the paper (gating) and 3.2 / 4.6 (placement is
// data); the rules are described in k_gate.hip.
#pragma once
#include "moe_internal.h"
#include "wave_ops.h"

namespace emoe {

// Monotone map float -> uint32 (larger float <-> larger integer).
__device__ __forceinline__ uint32_t orderable(float f)
{
    uint32_t b = __float_as_uint(f);
    return (b & 0x80000000u) ? ~b : (b | 0x80000000u);
}

// key: larger = better score, and among equal scores the LOWER index
__device__ __forceinline__ unsigned long long make_key(float score, int idx)
{
    return ((unsigned long long)orderable(score) << 32) | (unsigned long long)(0xffffffffu - (uint32_t)idx);
}
__device__ __forceinline__ int key_index(unsigned long long key) { return (int)(0xffffffffu - (uint32_t)(key & 0xffffffffull)); }

// Lane j < k holds the j-th selected expert and its score: ids and combine weights of the token (store: they go to the workspace;
// keep: where the weights go as well, or NULL).
__device__ __forceinline__ void finish_token(const Pass &p, int t, int lane, int my_id, float my_s, bool store, float *keep = nullptr)
{
    if (!store && !keep) return;   // uniform
    const float sum = wave_sum_f32(lane < p.k ? my_s : 0.f);
    if (lane < p.k) {
        const float wv = (p.renormalize ? my_s / sum : my_s) * p.routed_scale;
        if (store) {
            p.ids[(size_t)t * p.k + lane] = my_id;
            p.w[(size_t)t * p.k + lane] = wv;
        }
        if (keep) keep[lane] = wv;
    }
}

// Group scores and group limiting by way of LDS, any group size: cs [E] selection scores, those of dropped groups
// become -inf.
__device__ inline void limit_groups_lds(const Pass &p, float *cs, int lane)
{
    const int E = p.E;
    const float NEG = -__builtin_huge_valf();
    const int G = p.n_group, per = E / G;
    // L lanes share a group's experts (L a power of two, G * L <= 64): each finds the two largest
    // of its share, then the pairs are merged across the L lanes -- a group's score is the sum of
    // its two largest selection scores, which does not depend on the order they are found in
    int Lsh = 0;
    while ((2 * G) << Lsh <= 64) ++Lsh;
    const int L = 1 << Lsh;
    const int g = lane >> Lsh, sub = lane & (L - 1);
    float b1 = NEG, b2 = NEG;
    if (g < G) {
        for (int e = g * per + sub; e < (g + 1) * per; e += L) {
            const float v = cs[e];
            if (v > b1) { b2 = b1; b1 = v; } else if (v > b2) { b2 = v; }
        }
    }
    for (int d = 1; d < L; d <<= 1) {
        const float o1 = __shfl_xor(b1, d, 64), o2 = __shfl_xor(b2, d, 64);
        b2 = fmaxf(fminf(b1, o1), fmaxf(b2, o2));
        b1 = fmaxf(b1, o1);
    }
    // every lane of a group now holds the group's score.  The topk_group best groups are kept, the lower
    // index first among equal scores: a group's rank is the number of groups that come before it in that
    // order (the scores of all groups are read lane by lane), and it is kept when its rank is below topk_group
    const uint32_t mine = orderable((per > 1) ? b1 + b2 : b1);
    int rank = 0;
    for (int h = 0; h < G; ++h) {
        const uint32_t other = (uint32_t)__builtin_amdgcn_readlane((int)mine, h << Lsh);
        rank += (other > mine || (other == mine && h < g)) ? 1 : 0;
    }
    const unsigned long long keptmask = __ballot(g < G && rank < p.topk_group);   // bit g L: group g is kept
    const bool pow2 = (per & (per - 1)) == 0;
    const int psh = 31 - __clz(per);
    for (int e = lane; e < E; e += 64) {
        const int ge = pow2 ? e >> psh : e / per;
        if (!((keptmask >> (ge << Lsh)) & 1ull)) cs[e] = NEG;
    }
    wave_sync();
}

// Selection for one token, run by one wavefront, any number of experts.
//   lg   : LDS [E] logits in, scores out
//   cs   : LDS [E] selection scores (biased), destroyed (taken entries -> -inf)
// Returns the expert this lane holds (lane j < k: the j-th selected), which is also written to p.ids.
__device__ inline int select_token(const Pass &p, int t, float *lg, float *cs, int lane)
{
    const int E = p.E;
    const float NEG = -__builtin_huge_valf();
    // scores
    if (p.gate == MOE_GATE_SOFTMAX_TOPK) {
        float m = NEG;
        for (int e = lane; e < E; e += 64) m = fmaxf(m, lg[e]);
        m = wave_max_f32(m);
        float z = 0.f;
        for (int e = lane; e < E; e += 64) { float v = __expf(lg[e] - m); lg[e] = v; z += v; }   // hardware exp2: ~1e-7 relative, far inside the 1e-5 tie bar
        z = wave_sum_f32(z);
        for (int e = lane; e < E; e += 64) lg[e] = lg[e] / z;
    } else {
        for (int e = lane; e < E; e += 64) lg[e] = __builtin_amdgcn_rcpf(1.f + __expf(-lg[e]));   // hardware exp2 and reciprocal, ~1 ulp each
    }
    for (int e = lane; e < E; e += 64) cs[e] = lg[e] + (p.select_bias ? p.select_bias[e] : 0.f);
    wave_sync();
    // group limiting
    if (p.gate == MOE_GATE_SIGMOID_GROUP_TOPK && p.n_group > 1) {
        limit_groups_lds(p, cs, lane);
    }
    // top-k by repeated wavefront arg-max
    int my_id = 0;
    float my_s = 0.f;
    for (int j = 0; j < p.k; ++j) {
        unsigned long long key = 0ull;
        for (int e = lane; e < E; e += 64) {
            float v = cs[e];
            if (v != NEG) { unsigned long long kk = make_key(v, e); key = kk > key ? kk : key; }
        }
        key = wave_max_u64(key);
        if (key == 0ull) continue;                     // no candidate left: id 0, weight 0 (wave-uniform)
        int win = key_index(key);
        if (lane == j) { my_id = win; my_s = lg[win]; }
        if (lane == (win & 63)) cs[win] = NEG;
        wave_sync();
    }
    finish_token(p, t, lane, my_id, my_s, true);
    return my_id;
}

// largest and second largest of two pairs
__device__ __forceinline__ void merge_top2(float &b1, float &b2, float o1, float o2)
{
    b2 = fmaxf(fminf(b1, o1), fmaxf(b2, o2));
    b1 = fmaxf(b1, o1);
}
template <int CTRL>
__device__ __forceinline__ float dpp_f32(float v) { return __int_as_float(dpp_i32<CTRL, 0xf>(__float_as_int(v), __float_as_int(v))); }

// The same selection for up to 64 NR experts, NR <= 8, with the scores in registers: expert e is entry e / 64 of lane
// e % 64.  With few tokens a selection is one chain of dependent instructions (8 us of the LDS version on a grouped
// gate with 256 experts, 0.6 of it memory), with many it is bound by their number; both are why nothing here goes
// through LDS that a lane can keep, and why the candidates of a lane are sorted once, so that a round of the top-k
// is a wavefront maximum over the lanes' heads.
//   v    : logits of this lane's experts      lg : LDS [64 NR] scratch, scores out      cs : LDS [64 NR] scratch
template <int NR>
__device__ __forceinline__ int select_regs(const Pass &p, int t, float (&v)[NR], float *lg, float *cs, int lane, bool store = true, float *keep = nullptr)
{
    constexpr int kOrderBits = NR <= 4 ? 2 : 3;
    static_assert(NR <= 8, "a lane's order of experts is kept in fields of 2 or 3 bits");
    const int E = p.E;
    const float NEG = -__builtin_huge_valf();
    // scores
    if (p.gate == MOE_GATE_SOFTMAX_TOPK) {
        float m = NEG;
#pragma unroll
        for (int i = 0; i < NR; ++i) m = fmaxf(m, lane + 64 * i < E ? v[i] : NEG);
        m = wave_max_f32(m);
        float z = 0.f;
#pragma unroll
        for (int i = 0; i < NR; ++i) {
            v[i] = __expf(v[i] - m);   // hardware exp2: ~1e-7 relative, far inside the 1e-5 tie bar
            z += lane + 64 * i < E ? v[i] : 0.f;
        }
        z = wave_sum_f32(z);
#pragma unroll
        for (int i = 0; i < NR; ++i) v[i] = v[i] / z;
    } else {
#pragma unroll
        for (int i = 0; i < NR; ++i) v[i] = __builtin_amdgcn_rcpf(1.f + __expf(-v[i]));   // hardware exp2 and reciprocal, ~1 ulp each
    }
#pragma unroll
    for (int i = 0; i < NR; ++i) lg[64 * i + lane] = v[i];   // the winners' scores are fetched from here after the last round
#pragma unroll
    for (int i = 0; i < NR; ++i) v[i] = lane + 64 * i < E ? v[i] + (p.select_bias ? p.select_bias[lane + 64 * i] : 0.f) : NEG;
    // group limiting
    if (p.gate == MOE_GATE_SIGMOID_GROUP_TOPK && p.n_group > 1) {
        const int G = p.n_group, per = E / G;
        if ((per & (per - 1)) == 0 && per >= 16 && per <= 64) {
            // a group is one row of 16 lanes, two or four of one entry: the two largest of a row by rotations
            // (each doubles the set a lane has seen, all sets disjoint), of several rows by shuffles
            float b1[NR], b2[NR];
#pragma unroll
            for (int i = 0; i < NR; ++i) {
                b1[i] = v[i] == v[i] ? v[i] : NEG;   // a NaN does not count (merged, it would make its partner's score count twice)
                b2[i] = NEG;
                merge_top2(b1[i], b2[i], dpp_f32<0x128>(b1[i]), dpp_f32<0x128>(b2[i]));   // row_ror 8, 4, 2, 1
                merge_top2(b1[i], b2[i], dpp_f32<0x124>(b1[i]), dpp_f32<0x124>(b2[i]));
                merge_top2(b1[i], b2[i], dpp_f32<0x122>(b1[i]), dpp_f32<0x122>(b2[i]));
                merge_top2(b1[i], b2[i], dpp_f32<0x121>(b1[i]), dpp_f32<0x121>(b2[i]));
            }
            if (per >= 32) {
#pragma unroll
                for (int i = 0; i < NR; ++i) merge_top2(b1[i], b2[i], __shfl_xor(b1[i], 16, 64), __shfl_xor(b2[i], 16, 64));
            }
            if (per == 64) {
#pragma unroll
                for (int i = 0; i < NR; ++i) merge_top2(b1[i], b2[i], __shfl_xor(b1[i], 32, 64), __shfl_xor(b2[i], 32, 64));
            }
            // lane g < G takes group g's score; a group's rank is the number of groups before it in (score, lower
            // index first) order, and it is kept when its rank is below topk_group
            const int psh = 31 - __clz(per);
#pragma unroll
            for (int i = 0; i < NR; ++i)
                if ((lane & (per - 1)) == 0 && 64 * i + lane < E) cs[(64 * i + lane) >> psh] = b1[i] + b2[i];
            wave_sync();
            const uint32_t mine = lane < G ? orderable(cs[lane]) : 0u;
            int rank = 0;
            for (int h = 0; h < G; ++h) {
                const uint32_t other = (uint32_t)__builtin_amdgcn_readlane((int)mine, h);
                rank += (other > mine || (other == mine && h < lane)) ? 1 : 0;
            }
            const unsigned long long kept = __ballot(lane < G && rank < p.topk_group);
#pragma unroll
            for (int i = 0; i < NR; ++i)
                if (!((kept >> ((64 * i + lane) >> psh)) & 1ull)) v[i] = NEG;
        } else {
#pragma unroll
            for (int i = 0; i < NR; ++i) cs[64 * i + lane] = v[i];
            wave_sync();
            limit_groups_lds(p, cs, lane);
#pragma unroll
            for (int i = 0; i < NR; ++i) v[i] = cs[64 * i + lane];
        }
    }
    wave_sync();
    // Candidates as order-preserving integers (0 = absent), a lane's sorted once, largest first and among equal ones
    // the lower expert first; `order` has their entries in fields of kOrderBits.
    uint32_t c[NR];
    uint32_t at[NR];
#pragma unroll
    for (int i = 0; i < NR; ++i) { c[i] = v[i] != NEG ? orderable(v[i]) : 0u; at[i] = i; }
    auto put_first = [&](int i, int j) {                     // i < j: the larger one to i, equal ones stay (adjacent steps only: stable)
        const bool swap = c[j] > c[i];
        const uint32_t ci = c[i], ai = at[i];
        c[i] = swap ? c[j] : ci; at[i] = swap ? at[j] : ai;
        c[j] = swap ? ci : c[j]; at[j] = swap ? ai : at[j];
    };
#pragma unroll
    for (int r = 0; r < NR; ++r)                             // odd-even transposition: NR rounds of adjacent exchanges
#pragma unroll
        for (int i = r & 1; i + 1 < NR; i += 2) put_first(i, i + 1);
    uint32_t order = 0;
#pragma unroll
    for (int i = 0; i < NR; ++i) order |= at[i] << (kOrderBits * i);
    // top-k: a wavefront maximum over the lanes' heads; only when several lanes hold it (equal scores) a second
    // reduction for the lowest expert among them
    int my_id = 0;
    bool none = false;         // this lane's selection round found no candidate
    for (int j = 0; j < p.k; ++j) {
        const uint32_t m = wave_max_u32(c[0]);
        const int head = lane + 64 * (int)(order & ((1u << kOrderBits) - 1u));
        const unsigned long long holders = __ballot(c[0] == m && m != 0u);
        int win;
        if (__popcll(holders) == 1) {
            win = __builtin_amdgcn_readlane(head, __ffsll((long long)holders) - 1);
        } else {
            win = wave_min_i32(c[0] == m && m != 0u ? head : 0x7fffffff);
            if (win == 0x7fffffff) win = -1;             // no candidate left
        }
        // fewer than k candidates (non-finite biases or activations): the slot keeps id 0 with weight 0
        // (my_s is only fetched for a real winner), so that nothing is indexed by -1
        if (lane == j) { my_id = win < 0 ? 0 : win; none = win < 0; }
        const bool took = head == win;
#pragma unroll
        for (int i = 0; i < NR; ++i) c[i] = took ? (i + 1 < NR ? c[i + 1 < NR ? i + 1 : i] : 0u) : c[i];
        order = took ? order >> kOrderBits : order;
    }
    finish_token(p, t, lane, my_id, lane < p.k && !none ? lg[my_id] : 0.f, store, keep);
    return my_id;
}

// The same selection with a token on each group of L = 16 or 32 lanes (gates without groups, at most L experts, an expert per lane; L <= 32): v
// is the logit of expert `sub` of the lane's token t.  The sums run in select_regs's order, so ids and weights have the same bits; a wavefront selects 64 / L
// tokens with little more instructions than one.  active: the lane's token exists.
template <int L>
__device__ __forceinline__ int select_lanes(const Pass &p, int t, float v, int lane, bool active, bool store, float *keep)
{
    static_assert(L == 16 || L == 32, "groups of whole rows of 16 lanes");
    const int sub = lane & (L - 1);
    const float NEG = -__builtin_huge_valf();
    auto sum = [&](float s) {                 // in the group's last lane, from there to all of them
#define STEP(CTRL, MASK) s += __int_as_float(dpp_i32<CTRL, MASK>(0, __float_as_int(s)));
        STEP(0x111, 0xf) STEP(0x112, 0xf) STEP(0x114, 0xf) STEP(0x118, 0xf)
        if (L == 32) { STEP(0x142, 0xa) }
#undef STEP
        return __shfl(s, L - 1, L);
    };
    auto most = [&](uint32_t m) {             // row_ror 8, 4, 2, 1
        m = max(m, (uint32_t)dpp_i32<0x128, 0xf>(0, (int)m));
        m = max(m, (uint32_t)dpp_i32<0x124, 0xf>(0, (int)m));
        m = max(m, (uint32_t)dpp_i32<0x122, 0xf>(0, (int)m));
        m = max(m, (uint32_t)dpp_i32<0x121, 0xf>(0, (int)m));
        if (L == 32) m = max(m, (uint32_t)__shfl_xor((int)m, 16, 64));
        return m;
    };
    const bool is = sub < p.E;
    if (p.gate == MOE_GATE_SOFTMAX_TOPK) {
        float m = is ? v : NEG;
        m = fmaxf(m, dpp_f32<0x128>(m));
        m = fmaxf(m, dpp_f32<0x124>(m));
        m = fmaxf(m, dpp_f32<0x122>(m));
        m = fmaxf(m, dpp_f32<0x121>(m));
        if (L == 32) m = fmaxf(m, __shfl_xor(m, 16, 64));
        v = __expf(v - m);
        v = v / sum(is ? v : 0.f);
    } else {
        v = __builtin_amdgcn_rcpf(1.f + __expf(-v));
    }
    const float score = v;
    v = is ? v + (p.select_bias ? p.select_bias[sub] : 0.f) : NEG;
    uint32_t c = v != NEG ? orderable(v) : 0u;
    int my_id = 0;
    bool none = false;
    for (int j = 0; j < p.k; ++j) {
        const uint32_t m = most(c);
        const uint32_t holders = (uint32_t)(__ballot(c == m && m != 0u) >> (lane & (64 - L))) & (uint32_t)((1ull << L) - 1ull);
        const int win = __ffs((int)holders) - 1;   // equal scores: the lower expert; -1: no candidate left
        if (sub == j) { my_id = win < 0 ? 0 : win; none = win < 0; }
        c = sub == win ? 0u : c;
    }
    const float got = __shfl(score, my_id, L), my_s = sub < p.k && !none ? got : 0.f;
    const float total = sum(my_s);
    if (active && sub < p.k) {
        const float wv = (p.renormalize ? my_s / total : my_s) * p.routed_scale;
        if (store) {
            p.ids[(size_t)t * p.k + sub] = my_id;
            p.w[(size_t)t * p.k + sub] = wv;
        }
        if (keep) keep[sub] = wv;
    }
    return my_id;
}

// One token's selection from its logits: the planes (partial sums of the K ranges) are added in K order.  They come
// from other XCDs' L2s, so PZ planes of all of a lane's experts are requested before anything is added.  `beside` is called behind the
// first requests: what a workgroup stages for later goes there, in the shadow of that round trip.
template <int NR, int PZ, typename Beside>
__device__ __forceinline__ int select_from_planes(const Pass &p, int t, float *lg, float *cs, int lane, bool store, Beside beside)
{
    const float *src = p.logits + (size_t)t * p.E;
    const size_t plane = (size_t)p.T * p.E;
    float v[NR];
#pragma unroll
    for (int z0 = 0; z0 < kGatePlanes; z0 += PZ) {
        if (z0 >= p.logit_planes) break;
        float part[PZ][NR];
#pragma unroll
        for (int z = 0; z < PZ; ++z)
            if (z0 + z < p.logit_planes) {
#pragma unroll
                for (int i = 0; i < NR; ++i) part[z][i] = src[(z0 + z) * plane + min(64 * i + lane, p.E - 1)];
            }
        if (z0 == 0) beside();
#pragma unroll
        for (int z = 0; z < PZ; ++z)
            if (z0 + z < p.logit_planes) {
#pragma unroll
                for (int i = 0; i < NR; ++i) v[i] = z0 + z == 0 ? part[z][i] : v[i] + part[z][i];
            }
    }
    return select_regs<NR>(p, t, v, lg, cs, lane, store);
}
// Up to 512 experts in registers: above 256 the LDS form, which re-reads the scores in every round, costs more at every
// batch size (whole pass, us, LDS -> registers: 384 experts on rows of 7168, 64 tokens 119 -> 104 and 8192 tokens 239 -> 232;
// 512 experts on rows of 2048, 1 token 30 -> 20 and 30000 tokens 381 -> 339).
template <int PZ, typename Beside>
__device__ __forceinline__ int select_one(const Pass &p, int t, float *lg, float *cs, int lane, Beside beside)
{
    if (p.E <= 64)  return select_from_planes<1, PZ>(p, t, lg, cs, lane, true, beside);
    if (p.E <= 128) return select_from_planes<2, PZ>(p, t, lg, cs, lane, true, beside);
    if (p.E <= 256) return select_from_planes<4, PZ>(p, t, lg, cs, lane, true, beside);
    if (p.E <= 512) return select_from_planes<8, PZ>(p, t, lg, cs, lane, true, beside);
    beside();
    const float *src = p.logits + (size_t)t * p.E;
    const size_t plane = (size_t)p.T * p.E;
    for (int e = lane; e < p.E; e += 64) {
        float part[kGatePlanes];                         // all planes are requested at once, then added in K order
#pragma unroll
        for (int z = 0; z < kGatePlanes; ++z) part[z] = z < p.logit_planes ? src[z * plane + e] : 0.f;
        float v = part[0];
#pragma unroll
        for (int z = 1; z < kGatePlanes; ++z)
            if (z < p.logit_planes) v += part[z];
        lg[e] = v;
    }
    wave_sync();
    return select_token(p, t, lg, cs, lane);
}
// LDS floats per token: scores and selection scores (whole wavefronts of entries where they are kept in registers)
__host__ __device__ inline int select_stride(int E) { return E <= 64 ? 64 : E <= 128 ? 128 : E <= 256 ? 256 : E <= 512 ? 512 : E; }

// The expert table's entries [0, E + n_shared) -> LDS: from the workspace, or from the kernel's argument (a pass that
// brings its placement along: the first workgroup then leaves it in the workspace too).
struct NoTable {};
struct TableArg { int32_t v[kTableArg]; };
inline TableArg fill_table(const Pass &p)
{
    TableArg tab;
    for (int i = 0; i < kTableArg; ++i) tab.v[i] = i < p.E + p.n_shared ? p.host_table[i] : -1;
    return tab;
}
__device__ __forceinline__ void stage_table(const Pass &p, const NoTable &, int32_t *map, int threads)
{
    for (int e = threadIdx.x; e < p.E + p.n_shared; e += threads) map[e] = p.map[e];
}
__device__ __forceinline__ void stage_table(const Pass &p, const TableArg &tab, int32_t *map, int threads)
{
    for (int e = threadIdx.x; e < p.E + p.n_shared; e += threads) {
        const int32_t v = tab.v[e];
        map[e] = v;
        if (blockIdx.x == 0) const_cast<int32_t *>(p.map)[e] = v;
    }
}

// Slot of this lane's assignment of token t (lane j < k: the j-th selected expert `id`, then the shared experts), or -1.
__device__ __forceinline__ int slot_of_lane(const Pass &p, const int32_t *map, int t, int lane, int id)
{
    if (lane < p.k) {
        const int m = map[id];
        if (m >= -1) return m;
        // an expert with several copies: token t uses copy t mod R of the list behind the table's entries
        const int32_t *copies = p.map + p.E + p.n_shared + (-2 - m);
        return copies[1 + t % copies[0]];
    }
    if (lane < p.kk && t >= p.shared_begin && t < p.shared_end) return map[p.E + (lane - p.k)];
    return -1;
}

}  // namespace emoe
