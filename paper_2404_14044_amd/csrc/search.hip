// Forward search + sampling kernels: waves over XCD-banded chunks of rays.
#include "hp_kernels.hpp"
#include "hp_search.hpp"

namespace hp {

// (one lane) a ray with no point near it: no neighbour, no sample
__device__ __forceinline__ void put_empty(int64_t ray)
{
    const SearchCtx c = phase_ctx();
    const SampleOut o = phase_arg<SampleOut>();
    o.n_sel[ray] = 0;
    o.n_nbr[ray] = 0;
    o.flags[ray] = 0u;
    o.primary[ray] = -1;
    if (o.nbr_idx) {
        for (int i = 0; i < c.M; ++i) {
            o.nbr_idx[ray * c.M + i] = -1;
            o.nbr_t[ray * c.M + i] = 0.0f;
        }
    }
}

// Search neighbouring rays together, walk their candidates four rays at a time.
template <int KT, int NW>
__device__ __forceinline__ void search_sample_body()
{
    __shared__ WalkLds waves[NW];
    __shared__ int take;
    if (threadIdx.x == 0) take = 0;
    __syncthreads();
    WalkLds &sh = waves[threadIdx.x / WAVE];
    int ns = 0;  // slots filled
    for_each_group_banded<GROUP, NW>(sh.rs, &take, [&](int n, int ray, int rec, bool last) {
        // (as many of the group as there are slots left, the rest after the walk)
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
            const SearchCtx c = phase_ctx();
            const SampleOut o = phase_arg<SampleOut>();
            // rows of four values at a time where every row starts on 16 bytes
            const bool vec = nbr_vec_ok(o.knn_idx, o.knn_dist, c.K);
            walk_batch<KT>(sh, ns,
                [&](int rr, int i, int mm, int count, const uint64_t(&key)[4]) {
                    if (i == 0) {
                        o.n_nbr[rr] = mm;
                        o.flags[rr] = count > c.M ? 1u : 0u;
                    }
                    if (!o.nbr_idx) return;
#pragma unroll
                    for (int e = 0; e < 4; ++e) {
                        if (i + e >= c.M) break;
                        const int64_t at = (int64_t)rr * c.M + i + e;
                        o.nbr_idx[at] = i + e < mm ? (int32_t)(uint32_t)key[e] : -1;
                        o.nbr_t[at] = i + e < mm ? __uint_as_float((uint32_t)(key[e] >> 32)) : 0.0f;
                    }
                },
                [&](int rr, int s, float tj, const uint64_t(&kd)[KT], const float(&dist)[KT], int kc) {
                    const int64_t row = (int64_t)rr * c.S + s;
                    o.t[row] = tj;
                    int32_t *const pi = o.knn_idx + row * c.K;
                    float *const pd = o.knn_dist + row * c.K;
#pragma unroll
                    for (int k0 = 0; k0 < KT; k0 += 4) {
                        if (k0 >= c.K) break;
                        int32_t v[4];
#pragma unroll
                        for (int k = 0; k < 4; ++k) v[k] = k0 + k < kc ? (int32_t)(uint32_t)kd[k0 + k] : -1;
                        if (vec) {
                            *reinterpret_cast<int4 *>(pi + k0) = make_int4(v[0], v[1], v[2], v[3]);
                            *reinterpret_cast<float4 *>(pd + k0) =
                                make_float4(dist[k0], dist[k0 + 1], dist[k0 + 2], dist[k0 + 3]);
                        } else {
#pragma unroll
                            for (int k = 0; k < 4; ++k) {
                                if (k0 + k < c.K) {
                                    pi[k0 + k] = v[k];
                                    pd[k0 + k] = dist[k0 + k];
                                }
                            }
                        }
                    }
                },
                [&](int rr, int index) { o.primary[rr] = index; },
                [&](int rr, int nsel) {
                    o.n_sel[rr] = nsel;
                    if (nsel == 0) o.primary[rr] = -1;
                });
            ns = 0;
        }
    }, [&](int64_t ray) { put_empty(ray); });
}

// The same search with the uniform multi-surface sampler, one ray at a time.
template <int KT>
__device__ __forceinline__ void search_ms_body()
{
    __shared__ SlabLds sh;
    for_each_group_banded<1, 1>(sh.rs, nullptr, [&](int, int ray, int rec, bool) {
        SlabKeys slab;
        first_slab(sh, slab, rec);
        const int count = slab.rest;
        const RayGeom g = load_ray(sh.rs[rec]);
        const SearchCtx c = phase_ctx();
        const SampleOut o = phase_arg<SampleOut>();
        const int l = lane_id(), m = min(count, c.M);
        const int64_t rbase = (int64_t)ray * c.S;
        int prim;
        auto emit = [&](int s, int q, float tj, const uint64_t(&kd)[KT], const float(&dq)[KT / 4],
                        int kc) {
            // the position's four lanes share the row: lane q writes k = q, q + 4, ...
            const int64_t row = rbase + s;
            if (q == 0) o.t[row] = tj;
#pragma unroll
            for (int e = 0; e < KT / 4; ++e) {
                const int k = 4 * e + q;
                if (k < c.K) {
                    const bool v = k < kc;
                    o.knn_idx[row * c.K + k] = v ? (int32_t)(uint32_t)quad_entry<KT>(kd, e) : -1;
                    o.knn_dist[row * c.K + k] = v ? dq[e] : 0.0f;
                }
            }
        };
        if (o.nbr_idx && l < c.M) {
            o.nbr_idx[(int64_t)ray * c.M + l] = l < m ? (int)(uint32_t)slab.keys : -1;
            o.nbr_t[(int64_t)ray * c.M + l] = l < m ? __uint_as_float((uint32_t)(slab.keys >> 32)) : 0.0f;
        }
        const int nsel = uniform_samples<KT>(g, sh, slab, prim, emit);
        if (lane_id() == 0) {
            o.n_nbr[ray] = m;
            o.flags[ray] = (count > c.M) ? 1u : 0u;
            o.n_sel[ray] = nsel;
            o.primary[ray] = prim;
        }
        lds_sync();
    }, [&](int64_t ray) { put_empty(ray); });
}

// 4 waves per SIMD (128 VGPRs), 2 with lists of 32.  Lists of up to 8 do not spill
// at 4; those of 9 to 16 spill about ten registers, which costs less than a wave
// per SIMD does (4 waves / 3 without a spill, us: room of 5M points,
// lists of 16, 900x900 1310 / 1447, of 1M points, lists of 12, 400x400 357 / 421; 64x64
// equal).
constexpr int search_waves(int kt) { return kt <= 16 ? 16 : 8; }  // per workgroup that fills a CU

template <int KT, int NW>
__global__ void __launch_bounds__(WAVE *NW) __attribute__((amdgpu_waves_per_eu(KT <= 16 ? 4 : 2, 8)))
k_search_sample(SearchCtx, SampleOut)
{
    search_sample_body<KT, NW>();
}

// Bound by the latency of short chains (bisections in the LDS, gathers of a slab's
// points), so five waves per SIMD with lists of up to 8, though those of 5 to 8
// spill some 15 registers for it (200 positions, us, four / five waves: room of 500k points
// 900x900 6356 / 5973, plane of 5k 1371 / 1261, object cloud of 1M 1921 / 2028).
template <int KT>
__global__ void __launch_bounds__(WAVE) __attribute__((amdgpu_waves_per_eu(KT <= 8 ? 5 : KT <= 16 ? 4 : 2, 8)))
k_search_ms(SearchCtx, SampleOut)
{
    search_ms_body<KT>();
}

// The multi-surface sampler's single rays: few enough waves that one set-up pass
// of a wave serves about twelve rays, enough to fill the GPU (200 positions, us, by
// waves 65,536 / 24,576 / 16,384: object cloud of 1M points 300x300 443 / 431 / 459,
// 600x600 894 / 901 / 955, 900x900 1915 / 2212 / 2180; plane of 200k 300x300 174 /
// 141 / 135, 600x600 445 / 421 / 472, 900x900 897 / 935 / 955).
static int64_t ms_grid(const SearchCtx &c)
{
    if (c.blocks > 0 || c.chunk > 1) return wave_grid(c);
    const int64_t waves = c.n_rays / 12;
    return banded_grid(c, waves < 16384 ? 16384 : waves < WAVE_BLOCKS ? waves : WAVE_BLOCKS);
}

template <int KT>
static void launch_search_k(const SearchCtx &c, const SampleOut &o, hipStream_t s)
{
    constexpr int NW = search_waves(KT);
    if (dealt(c) && c.sampler != HP_SAMPLER_MS) {
        const int64_t blocks = banded_grid(c, CU_BLOCKS);
        k_search_sample<KT, NW><<<dim3((unsigned)blocks), dim3(WAVE * NW), 0, s>>>(c, o);
        return;
    }
    const int64_t blocks = c.sampler == HP_SAMPLER_MS ? ms_grid(c) : wave_grid(c);
    if (blocks == 0) return;
    const dim3 grid((unsigned)blocks), block(WAVE);
    if (c.sampler == HP_SAMPLER_MS) k_search_ms<KT><<<grid, block, 0, s>>>(c, o);
    else k_search_sample<KT, 1><<<grid, block, 0, s>>>(c, o);
}

hipError_t launch_search_sample(const SearchCtx &ctx, const SampleOut &o, int kt, hipStream_t s)
{
    SearchCtx c = ctx;
    c.chunk = launch_chunk(c, SEARCH_WALK);
    switch (kt) {
    case 4: launch_search_k<4>(c, o, s); break;
    case 8: launch_search_k<8>(c, o, s); break;
    case 16: launch_search_k<16>(c, o, s); break;
    default: launch_search_k<32>(c, o, s); break;
    }
    return hipGetLastError();
}

}  // namespace hp
