// K-NP extraction and image-based blending (Sec. 3.1, Eq. 1): the K points
// nearest to each ray among its neighbours, found by the same hashed-point
// search with the kept list ordered by (squared distance to the ray, index),
// blended with geometric weights w_i = 1 / max(e_i, eps), normalised.
//
// One wave searches up to four neighbouring rays at a time, as the forward
// search does, and blends them one row of 16 lanes each: lane k of a row holds
// the points 4 k .. 4 k + 3 nearest to its ray and gathers their colours, and
// the row adds up the weighted sums pairwise in list order.
#include "hp_kernels.hpp"
#include "hp_search.hpp"

namespace hp {

constexpr int KNP_WAVES = 16;  // per workgroup that fills a CU

template <int NW>

__global__ void __launch_bounds__(WAVE *NW) __attribute__((amdgpu_waves_per_eu(4, 8))) k_knp(SearchCtx, KnpArgs)
{
    __shared__ KnpLds waves[NW];
    __shared__ int take;
    if (threadIdx.x == 0) take = 0;
    __syncthreads();
    KnpLds &sh = waves[threadIdx.x / WAVE];
    for_each_group_banded<GROUP, NW>(sh.rs, &take, [&](int n, int ray0, int rec, bool) {
        lds_sync();
        if (lane_id() < n) sh.slot[lane_id()].rs = rec + lane_id();
        lds_sync();
        search_group<GROUP, HELD_KNP, true>(sh.rs, sh.slot, sh.s, 0, n, phase_arg<KnpArgs>().K, WAVE);
        const KnpArgs a = phase_arg<KnpArgs>();
        const int l = phase_lane_id(), r = l >> 4, k16 = l & 15;
        const bool live = r < n;
        const RaySlot me = sh.slot[live ? r : 0];
        const int held = live ? me.n : 0, kk = live ? min(me.count, a.K) : 0;
        const int64_t ray = ray0 + r;
        uint64_t key[4];
        row_sorted_keys(sh.s.pend[r], held, WAVE, key);
        float d[4], w[4], c0[4], c1[4], c2[4];
#pragma unroll
        for (int e = 0; e < 4; ++e) {
            d[e] = w[e] = c0[e] = c1[e] = c2[e] = 0.0f;
            if (4 * k16 + e < kk) {
                d[e] = __builtin_sqrtf(__uint_as_float((uint32_t)(key[e] >> 32)));
                w[e] = 1.0f / (d[e] > a.eps_idw ? d[e] : a.eps_idw);
                const float *col = a.colors + 3 * (int64_t)(uint32_t)key[e];
                c0[e] = w[e] * col[0];
                c1[e] = w[e] * col[1];
                c2[e] = w[e] * col[2];
            }
        }
        auto row_sum = [](const float(&v)[4]) {
            float s = (v[0] + v[1]) + (v[2] + v[3]);
#pragma unroll
            for (int o = 1; o < 16; o <<= 1) s += __shfl_xor(s, o, WAVE);
            return s;
        };
        const float ws = row_sum(w), s0 = row_sum(c0), s1 = row_sum(c1), s2 = row_sum(c2);
        if (live && k16 == 0) {
            a.rgb[3 * ray + 0] = kk ? s0 / ws : a.bg[0];
            a.rgb[3 * ray + 1] = kk ? s1 / ws : a.bg[1];
            a.rgb[3 * ray + 2] = kk ? s2 / ws : a.bg[2];
            if (a.cnt) a.cnt[ray] = kk;
        }
        if (live && a.idx) {
#pragma unroll
            for (int e = 0; e < 4; ++e) {
                const int k = 4 * k16 + e;
                if (k < a.K) {
                    a.idx[ray * a.K + k] = k < kk ? (int32_t)(uint32_t)key[e] : -1;
                    a.dist[ray * a.K + k] = d[e];
                }
            }
        }
        lds_sync();
    }, [&](int64_t ray) {
        const KnpArgs a = phase_arg<KnpArgs>();
        // (one lane) a ray with no point near it: background, no point
        a.rgb[3 * ray + 0] = a.bg[0];
        a.rgb[3 * ray + 1] = a.bg[1];
        a.rgb[3 * ray + 2] = a.bg[2];
        if (a.cnt) a.cnt[ray] = 0;
        if (a.idx) {
            for (int i = 0; i < a.K; ++i) {
                a.idx[ray * a.K + i] = -1;
                a.dist[ray * a.K + i] = 0.0f;
            }
        }
    });
}

hipError_t launch_knp(const SearchCtx &ctx, const KnpArgs &a, hipStream_t s)
{
    SearchCtx c = ctx;
    c.chunk = launch_chunk(c, SEARCH_KNP);
    const int64_t blocks = dealt(c) ? banded_grid(c, CU_BLOCKS) : wave_grid(c);
    if (blocks == 0) return hipSuccess;
    if (dealt(c)) k_knp<KNP_WAVES><<<dim3((unsigned)blocks), dim3(WAVE * KNP_WAVES), 0, s>>>(c, a);
    else k_knp<1><<<dim3((unsigned)blocks), dim3(WAVE), 0, s>>>(c, a);
    return hipGetLastError();
}

}  // namespace hp
