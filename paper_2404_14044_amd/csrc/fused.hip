// Search, sampling and rendering in one kernel (Sec. 3.2-3.4): the samples of
// a ray never leave the workgroup.  Every wave searches and walks groups of
// rays of its own, as the forward search does, with the samples emitted into
// its LDS; the samples of the (up to four) rays of one walk are then packed
// into tiles of 16, aggregated, decoded and composited, as the render does.
// Every operation and its order are those of hp_search_sample followed by
// hp_render, so the outputs are identical; what is saved is the sample
// arrays' round trip through memory and a launch.
//
// Bound by the latency and the instructions of the search.  The decoder's
// operands are packed once per workgroup into the LDS and read by its waves
// when a tile needs them (as in the shared render): kept in a wave's registers
// beside the search's state, and loaded again for every ray, they held the
// kernel to two waves per SIMD, and a tile per ray was a fifth full.  One
// workgroup per CU, its waves dealing out its rays among themselves: a second
// workgroup to replace it, let alone four, leaves the CU idle while the first
// drains (425, 507, 540 us).  Frame of 640k rays of the object cloud, BF16: 1,511 us
// with one-wave workgroups, 428 here (the separate calls 283 + 179).
#include <type_traits>

#include "hp_kernels.hpp"
#include "hp_mlp.hpp"
#include "hp_search.hpp"

namespace hp {

constexpr int FUSED_S = 16;  // samples per ray the fused kernel holds

// The samples of RAYS rays: what the walk (or the uniform sampler) emits.
template <int RAYS, int KT>
struct FusedSamples {
    float t[RAYS][FUSED_S];
    int32_t idx[RAYS][FUSED_S][KT];
    float w[RAYS][FUSED_S][KT];  // inverse-distance weights, not normalised
    int32_t ray[RAYS], n[RAYS];
};

// A wave's LDS.  The walk's lists are dead when its samples are decoded, so
// the decoded samples take their place.
template <int KT>
struct FusedWalkLists : WalkLists {
    FusedSamples<GROUP, KT> smp;
};

template <int KT, bool MS>
struct FusedLds;

template <int KT>
struct FusedLds<KT, false> : WalkLdsOf<FusedWalkLists<KT>> {
    static constexpr int RAYS = GROUP;
    __device__ __forceinline__ FusedSamples<GROUP, KT> &samples() { return this->lists().smp; }
    __device__ __forceinline__ float4 *out() { return this->lists().p; }
    static_assert(sizeof(WalkLists) >= GROUP * FUSED_S * sizeof(float4), "decoded samples exceed the lists");
};

template <int KT>
struct FusedLds<KT, true> : SlabLds {
    static constexpr int RAYS = 1;
    FusedSamples<1, KT> smp;
    float4 dec[FUSED_S];
    __device__ __forceinline__ FusedSamples<1, KT> &samples() { return smp; }
    __device__ __forceinline__ float4 *out() { return dec; }
};

// Aggregate, decode and composite the samples of the first ns rays held.
template <int KT, int PREC, bool MS, typename Image>
__device__ __forceinline__ void fused_render(FusedLds<KT, MS> &sh, const Image &img, int ns)
{
    const SearchCtx c = phase_ctx();
    const FusedArgs a = phase_arg<FusedArgs>();
    constexpr int RAYS = FusedLds<KT, MS>::RAYS;
    const int l = phase_lane_id();
    const int r16 = l & 15, q = l >> 4;
    auto &smp = sh.samples();
    float4 *const out = sh.out();
    lds_sync();
    int pre[RAYS + 1];  // first sample of each ray
    pre[0] = 0;
#pragma unroll
    for (int k = 0; k < RAYS; ++k) pre[k + 1] = pre[k] + (k < ns ? uniform_i32(smp.n[k]) : 0);
    const int total = pre[RAYS];
    for (int s0 = 0; s0 < total; s0 += 16) {
        const int sidx = s0 + r16;
        const bool valid = sidx < total;
        // aggregation (lane: sample r16, features 8 q .. 8 q + 7): neighbours
        // four at a time, summed in order
        float f[8];
#pragma unroll
        for (int e = 0; e < 8; ++e) f[e] = 0.0f;
        if (valid) {
            int k = 0, s = sidx;
#pragma unroll
            for (int j = 1; j < RAYS; ++j) {
                k = sidx >= pre[j] ? j : k;
                s = sidx >= pre[j] ? sidx - pre[j] : s;
            }
            const int32_t *const ki = smp.idx[k][s];
            const float *const kw = smp.w[k][s];
            float wsum = 0.0f;
            for (int k0 = 0; k0 < c.K; k0 += 4) {
                const int4 iv = *reinterpret_cast<const int4 *>(ki + k0);
                const float4 wv = *reinterpret_cast<const float4 *>(kw + k0);
                const int idx[4] = {iv.x, iv.y, iv.z, iv.w};
                const float w[4] = {wv.x, wv.y, wv.z, wv.w};
                float4 x0[4], x1[4];
#pragma unroll
                for (int j = 0; j < 4; ++j) {
                    if (idx[j] >= 0) {
                        const float4 *src = reinterpret_cast<const float4 *>(
                            a.feat + (int64_t)idx[j] * HP_FEAT_DIM + 8 * q);
                        x0[j] = src[0];
                        x1[j] = src[1];
                    }
                }
#pragma unroll
                for (int j = 0; j < 4; ++j) {
                    if (idx[j] >= 0) {
                        f[0] = fma_rn(w[j], x0[j].x, f[0]);
                        f[1] = fma_rn(w[j], x0[j].y, f[1]);
                        f[2] = fma_rn(w[j], x0[j].z, f[2]);
                        f[3] = fma_rn(w[j], x0[j].w, f[3]);
                        f[4] = fma_rn(w[j], x1[j].x, f[4]);
                        f[5] = fma_rn(w[j], x1[j].y, f[5]);
                        f[6] = fma_rn(w[j], x1[j].z, f[6]);
                        f[7] = fma_rn(w[j], x1[j].w, f[7]);
                        wsum += w[j];
                    }
                }
                if (idx[3] < 0) break;
            }
            const float inv = wsum > 0.0f ? 1.0f / wsum : 0.0f;
#pragma unroll
            for (int e = 0; e < 8; ++e) f[e] *= inv;
        }
        f32x4 o;
        __asm__ volatile("" ::: "memory");
        if constexpr (PREC == HP_BF16) o = decode_bf16(img, f);
        else o = decode_f32(img, f);
        // the activations on all of the sample's lanes, one output each
        if (q == 0 && valid) out[sidx] = make_float4(o[0], o[1], o[2], o[3]);
        lds_sync();
        if (valid) {
            float *const v = reinterpret_cast<float *>(&out[sidx]) + q;
            const float x = *v;
            *v = q < 3 ? sigmoid_f(x) : softplus_f(x);
        }
    }
    lds_sync();
    if (l < ns) {
        // lane k composites ray k
        const int n = smp.n[l];
        const int64_t ray = smp.ray[l];
        int base = 0;
#pragma unroll
        for (int k = 1; k < RAYS; ++k) base = l >= k ? pre[k] : base;
        float T = 1.0f, cr = 0.0f, cg = 0.0f, cb = 0.0f, dep = 0.0f, ws = 0.0f;
        for (int s = 0; s < n; ++s) {
            const float4 v = out[base + s];
            const float t = smp.t[l][s];
            const float delta = (s + 1 < n) ? smp.t[l][s + 1] - t : a.delta_last;
            const float e = expf(-v.w * delta);
            const float w = T * (1.0f - e);
            cr = fma_rn(w, v.x, cr);
            cg = fma_rn(w, v.y, cg);
            cb = fma_rn(w, v.z, cb);
            dep = fma_rn(w, t, dep);
            ws += w;
            T *= e;
        }
        const float rest = 1.0f - ws;
        a.rgb[3 * ray + 0] = fma_rn(rest, a.bg[0], cr);
        a.rgb[3 * ray + 1] = fma_rn(rest, a.bg[1], cg);
        a.rgb[3 * ray + 2] = fma_rn(rest, a.bg[2], cb);
        if (a.depth) a.depth[ray] = dep;
        if (a.acc) a.acc[ray] = ws;
        if (a.n_sel) a.n_sel[ray] = n;
    }
    lds_sync();
}

// the composite of no sample, by one lane
__device__ __forceinline__ void fused_empty(int64_t ray)
{
    const FusedArgs a = phase_arg<FusedArgs>();
    a.rgb[3 * ray + 0] = fma_rn(1.0f, a.bg[0], 0.0f);
    a.rgb[3 * ray + 1] = fma_rn(1.0f, a.bg[1], 0.0f);
    a.rgb[3 * ray + 2] = fma_rn(1.0f, a.bg[2], 0.0f);
    if (a.depth) a.depth[ray] = 0.0f;
    if (a.acc) a.acc[ray] = 0.0f;
    if (a.n_sel) a.n_sel[ray] = 0;
}

template <int PREC>
using FusedImage = typename std::conditional<PREC == HP_BF16, MlpBf16Shared, MlpF32Shared>::type;

// Waves per workgroup, one of which fills a CU: as many as the LDS holds beside
// the decoder, up to 4 per SIMD (128 VGPRs; lists of 16 need more than that: 3).
template <int KT, int PREC, bool MS>
constexpr int fused_waves()
{
    const int fit = (int)((163840 - 16 - sizeof(FusedImage<PREC>)) / sizeof(FusedLds<KT, MS>));
    const int most = KT <= 8 ? 16 : 12;
    return fit < most ? fit : most;
}

template <int KT, int PREC, bool MS>
__global__ void __launch_bounds__((WAVE * fused_waves<KT, PREC, MS>())) k_fused(SearchCtx, FusedArgs)
{
    constexpr int NW = fused_waves<KT, PREC, MS>();
    __shared__ FusedImage<PREC> img;
    __shared__ FusedLds<KT, MS> waves[NW];
    __shared__ int take;
    if (threadIdx.x == 0) take = 0;
    {
        const FusedArgs a = phase_arg<FusedArgs>();
        const int w = threadIdx.x / WAVE;
        if constexpr (PREC == HP_BF16) store_mlp_bf16_shared(a.w, img, w, NW);
        else store_mlp_f32_shared(a.w, img, w, NW);
    }
    __syncthreads();
    FusedLds<KT, MS> &sh = waves[threadIdx.x / WAVE];
    auto &smp = sh.samples();
    auto empty = [&](int64_t ray) { fused_empty(ray); };
    auto weight = [](float d, float eps) { return 1.0f / (d > eps ? d : eps); };
    if constexpr (MS) {
        for_each_group_banded<1, NW>(sh.rs, &take, [&](int, int ray, int rec, bool) {
            SlabKeys slab;
            first_slab(sh, slab, rec);
            const RayGeom g = load_ray(sh.rs[rec]);
            const float eps = phase_arg<FusedArgs>().eps_idw;
            int prim;
            const int n = uniform_samples<KT>(g, sh, slab, prim,
                [&](int s, int q, float tj, const uint64_t(&kd)[KT], const float(&dq)[KT / 4], int kc) {
                    if (q == 0) smp.t[0][s] = tj;
#pragma unroll
                    for (int e = 0; e < KT / 4; ++e) {
                        const int k = 4 * e + q;
                        const bool v = k < kc;  // (kc <= K)
                        smp.idx[0][s][k] = v ? (int32_t)(uint32_t)quad_entry<KT>(kd, e) : -1;
                        smp.w[0][s][k] = weight(v ? dq[e] : 0.0f, eps);
                    }
                });
            if (lane_id() == 0) {
                smp.ray[0] = ray;
                smp.n[0] = n;
            }
            fused_render<KT, PREC, MS>(sh, img, 1);
        }, empty);
    } else {
        int ns = 0;  // slots filled
        for_each_group_banded<GROUP, NW>(sh.rs, &take, [&](int n, int ray, int rec, bool last) {
            while (n > 0) {
                const int m = min(n, GROUP - ns);
                lds_sync();
                if (lane_id() < m) {
                    sh.slot[ns + lane_id()].ray = ray + lane_id();
                    sh.slot[ns + lane_id()].rs = rec + lane_id();
                }
                lds_sync();
                search_group<GROUP, HELD_WALK>(sh.rs, sh.slot, sh.search(), ns, m, WAVE, HELD_WALK);
                ns += m;
                n -= m;
                ray += m;
                rec += m;
                if (!(ns == GROUP || (last && n == 0))) continue;
                // (a ray's slot is its lane's row of the walk)
                const int slot = lane_id() >> 4;
                const float eps = phase_arg<FusedArgs>().eps_idw;
                walk_batch<KT>(sh, ns, [](int, int, int, int, const uint64_t(&)[4]) {},
                    [&](int, int s, float tj, const uint64_t(&kd)[KT], const float(&dist)[KT], int kc) {
                        smp.t[slot][s] = tj;
#pragma unroll
                        for (int k = 0; k < KT; ++k) {
                            smp.idx[slot][s][k] = k < kc ? (int32_t)(uint32_t)kd[k] : -1;
                            smp.w[slot][s][k] = weight(dist[k], eps);
                        }
                    },
                    [](int, int) {},
                    [&](int rr, int nsel) {
                        smp.ray[slot] = rr;
                        smp.n[slot] = nsel;
                    });
                fused_render<KT, PREC, MS>(sh, img, ns);
                ns = 0;
            }
        }, empty);
    }
}

int fused_max_samples() { return FUSED_S; }

template <int KT, int PREC, bool MS>
static void launch_fused_kpm(const SearchCtx &c, const FusedArgs &a, hipStream_t s)
{
    constexpr int NW = fused_waves<KT, PREC, MS>();
    // (never more than one workgroup per CU, whatever grid the caller names: each
    // loads the decoder, and a second one waits for the first to drain; frames of
    // the object with 65,536 named, us, that many waves / one workgroup per CU:
    // 192x192 643 / 129, 400x400 809 / 206, 800x800 888 / 437)
    const int64_t blocks = banded_grid(c, c.blocks > 0 && c.blocks < CU_BLOCKS ? c.blocks : CU_BLOCKS);
    if (blocks == 0) return;
    k_fused<KT, PREC, MS><<<dim3((unsigned)blocks), dim3(WAVE * NW), 0, s>>>(c, a);
}

template <int KT>
static void launch_fused_k(const SearchCtx &c, const FusedArgs &a, int precision, hipStream_t s)
{
    const bool ms = c.sampler == HP_SAMPLER_MS;
    if (precision == HP_BF16) {
        if (ms) launch_fused_kpm<KT, HP_BF16, true>(c, a, s);
        else launch_fused_kpm<KT, HP_BF16, false>(c, a, s);
    } else {
        if (ms) launch_fused_kpm<KT, HP_FP32, true>(c, a, s);
        else launch_fused_kpm<KT, HP_FP32, false>(c, a, s);
    }
}

hipError_t launch_fused(const SearchCtx &ctx, const FusedArgs &a, int kt, int precision, hipStream_t s)
{
    SearchCtx c = ctx;
    c.chunk = launch_chunk(c, SEARCH_FUSED);
    if (kt == 4) launch_fused_k<4>(c, a, precision, s);
    else if (kt == 8) launch_fused_k<8>(c, a, precision, s);
    else launch_fused_k<16>(c, a, precision, s);
    return hipGetLastError();
}

}  // namespace hp
