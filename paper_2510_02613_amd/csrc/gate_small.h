// Products of a small router (up to 64 experts, 512 wide) with a workgroup's own tokens: shared by the kernel that gates such layers
// (k_gate.hip) and by the one that runs the whole pass of a small layer (k_token_experts.hip), which therefore give the same bits.
#pragma once
#include <type_traits>

#include "moe_internal.h"

namespace emoe {

typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef float f32x4 __attribute__((ext_vector_type(4)));

// 8 consecutive elements of a row (zeros past the end)
template <typename T> struct Run8 { uint4 v[sizeof(T) / 2]; };
template <typename T>
__device__ __forceinline__ void load_run8(Run8<T> &r, const T *row, int k, int H)
{
#pragma unroll
    for (int h = 0; h < (int)sizeof(T) / 2; ++h) r.v[h] = k < H ? *(const uint4 *)(row + k + h * (16 / sizeof(T))) : make_uint4(0, 0, 0, 0);
}
__device__ __forceinline__ void widen8(const Run8<uint16_t> &r, float (&f)[8])
{
    const uint32_t *u = (const uint32_t *)&r.v[0];
#pragma unroll
    for (int e = 0; e < 4; ++e) {
        f[2 * e] = __uint_as_float(u[e] << 16);
        f[2 * e + 1] = __uint_as_float(u[e] & 0xffff0000u);
    }
}
__device__ __forceinline__ void widen8(const Run8<float> &r, float (&f)[8])
{
#pragma unroll
    for (int e = 0; e < 8; ++e) f[e] = ((const float *)&r.v[0])[e];
}

constexpr int kSmallExperts = 64, kSmallHidden = 512;
constexpr int kSmallChunks = kSmallHidden / 32 / (kFusedTokens / (kSmallExperts / 16));   // most chunks of 32 k a wavefront has: 4

// Which part of a token tile's logits a wavefront of kFusedTokens computes: expert tile `et` over the chunks [c0, c1) of 32 k of the
// contraction, which is shared out over the wavefronts of an expert tile.
struct SmallShare {
    int n_et, parts, et, c0, c1;
    int added;                     // shares that are added up: all of them or, where LDS is short (exact), the first ones, up to the last chunk
    __device__ __forceinline__ int waves() const { return added * n_et; }
    __device__ __forceinline__ SmallShare(const Pass &p, int wave, bool exact)
    {
        n_et = (p.E + 15) >> 4;
        parts = kFusedTokens / n_et;
        et = wave % n_et;
        const int mine = wave / n_et, chunks = (p.H + 31) / 32, per = (chunks + parts - 1) / parts;
        c0 = min(mine * per, chunks);
        c1 = mine < parts ? min(c0 + per, chunks) : c0;
        added = exact ? (chunks + per - 1) / per : parts;
    }
};

// acc[i]: this wavefront's share of the logits of token tile t0 + 16 i (lane: token l % 16, experts 4 (l / 16) ..).  The products of a
// logit are added chunk by chunk whatever NTT is.
template <int NTT, typename XT, typename WT>
__device__ __forceinline__ void small_products(const Pass &p, int t0, const SmallShare &sh, int lane, f32x4 (&acc)[NTT])
{
    constexpr bool kBf16 = sizeof(XT) == 2 && sizeof(WT) == 2;
    constexpr int G = NTT == 1 ? kSmallChunks : 1;       // chunks requested together
    const int E = p.E, H = p.H, n = lane & 15, q = lane >> 4;
#pragma unroll
    for (int i = 0; i < NTT; ++i) acc[i] = (f32x4){0.f, 0.f, 0.f, 0.f};
    const XT *x[NTT];
#pragma unroll
    for (int i = 0; i < NTT; ++i) x[i] = (const XT *)p.x + (size_t)min(t0 + i * 16 + n, p.T - 1) * H;
    const WT *wr = (const WT *)p.router_w + (size_t)min(sh.et * 16 + n, E - 1) * H;
#pragma unroll
    for (int g = 0; g < kSmallChunks; g += G) {
        if (sh.c0 + g >= sh.c1) break;
        Run8<XT> xv[G][NTT];
        Run8<WT> wv[G];
#pragma unroll
        for (int j = 0; j < G; ++j) {                    // this lane's 8 k of every chunk (H % 8 == 0)
            const int c = sh.c0 + g + j, k = c * 32 + q * 8, end = c < sh.c1 ? H : 0;
#pragma unroll
            for (int i = 0; i < NTT; ++i) load_run8(xv[j][i], x[i], k, end);
            load_run8(wv[j], wr, k, end);
        }
#pragma unroll
        for (int j = 0; j < G; ++j) {
            if (sh.c0 + g + j >= sh.c1) break;
            float wf[8];
            if constexpr (!kBf16) widen8(wv[j], wf);
#pragma unroll
            for (int i = 0; i < NTT; ++i) {
                if constexpr (kBf16) {
                    acc[i] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(*(bf16x8 *)&wv[j].v[0], *(bf16x8 *)&xv[j][i].v[0], acc[i], 0, 0, 0);
                } else {
                    float xf[8];
                    widen8(xv[j][i], xf);
#pragma unroll
                    for (int e = 0; e < 8; ++e) acc[i] = __builtin_amdgcn_mfma_f32_16x16x4f32(wf[e], xf[e], acc[i], 0, 0, 0);
                }
            }
        }
    }
}

// The logit of expert e for token `token` of a tile: the wavefronts' shares (part: 256 floats each, row r of lane l at 64 r + l) in
// the order of the contraction; 0 past the last expert.
__device__ __forceinline__ float small_logit(const Pass &p, const SmallShare &sh, const float *part, int token, int e)
{
    float v = 0.f;
    if (e < p.E) {      // tile e / 16, row 4 q' + r of it
        const int at = (e & 3) * 64 + ((e & 15) >> 2) * 16 + token;
        for (int i = 0; i < sh.added; ++i) v += part[(i * sh.n_et + (e >> 4)) * 256 + at];
        if (p.logit_bias) v += p.logit_bias[e];
    }
    return v;
}

}  // namespace emoe
