// Hashed-point search (Sec. 3.2) and adaptive primary-surface sampling
// (Sec. 3.3, Eq. 4, Eq. 5), one wave for up to four neighbouring rays.  Shared
// by the search + sampling kernels (also run by the backward pass to recompute
// its samples), the K-NP kernel and the fused search + render kernel.
//
// Search.  A neighbour of the ray is a point within rho(t) of it at its own
// parameter t in [t_near, t_far].  Such a point projects at most
//     delta(t) = f rho(t) L^2 / (t - rho(t) |w|)
// pixels from the ray's pixel centre (w: normalised image coordinate of the
// ray, L^2 = 1 + |w|^2, f = max(fx, fy)), and delta does not grow with t.
// Its depth z also bounds t from below, t >= (L z - |w| r) / (1 + |w| r
// inv_tref).  So
//   1. the minimum depth of the 8x8-bucket cells around the pixel is read; if
//      they are all empty the ray has no neighbour, else the smallest depth
//      bounds t and thus the window radius delta(t) (two rounds, each over the
//      cells of the previous radius; four lanes per ray do this for up to
//      sixteen rays at once, ray_setup);
//   2. inside a bucket at distance D from the pixel centre only points with
//      t <= f r L^2 / D + r |w|, i.e. z <= (f r L^2 / D + 2 r |w|) / L, can be
//      neighbours (fixed-radius branch of rho); buckets are ordered by z, so a
//      bucket whose first point is deeper is skipped.
// Every bound is widened by relative margins far above binary32 rounding; the
// exact predicate decides.
//
// Up to four rays of one image row are searched together (search_group): their
// windows overlap almost entirely, so the buckets' headers, the points' loads
// and the bookkeeping that deals points to lanes are paid once, and only the
// exact predicate is evaluated per ray.  Keys (t bits << 32 | point index) of
// passing points go to the ray's pending buffer, which is cut back to the
// smallest 64 to 128 when it fills (keep_smallest); it is never sorted there.
//
// Sampling (walk_batch).  Candidates are the neighbours in (t, index) order,
// sorted for four rays at once, one row of 16 lanes each; every lane serves
// one candidate.  The K nearest neighbours of candidate j within R_j =
// rho(t_j) lie in the window |t_i - t_j| <= R_j of the sorted list (distance
// >= |t_i - t_j| up to rounding).  The row then walks its candidates in order
// accumulating the transmittance of Eq. 5 and stops once no later candidate
// can pass eps_w (alpha <= gamma, so w_j <= gamma T), which usually happens
// within the first sixteen.
//
// The kernels are bound by instruction issue, vector and scalar, not by
// memory (object view, 640k rays, 1M points: 1.6 TB/s).  One ray at a time,
// with sorted lists kept by merging and four lanes to a candidate, took 309M
// vector and 123M scalar instructions and 0.509 ms there; this way it takes
// 157M, 63M and 0.346 ms (room view, 762k rays, 5M points: 2.82 and 1.32 ms).
#pragma once
#include "hp_device.hpp"

namespace hp {

struct SearchCtx {
    const int32_t *offsets;
    const float4 *pts;
    const float4 *pcam;    // camera-space points in point order, per view
    const float *bucket_z;
    const uint32_t *cell_zmin;
    const ViewK *views;
    int32_t n_views, layout;
    int64_t n_points;
    int64_t ray0, n_rays;   // rays ray0 .. ray0 + n_rays - 1 of the table's views
    float radius, inv_tref, t_near, t_far, gamma, inv_beta2, eps_w;
    int32_t K, S, M;
    int32_t chunk, blocks;  // rays per work chunk, persistent grid (0 = default)
    int32_t rmode;          // HP_RADIUS_*
    float rddot;            // Eq. 3 kernel disc radius (unit focal length)
    int32_t sampler;        // HP_SAMPLER_*
    int32_t ms_steps;       // uniform positions of the multi-surface sampler
    int32_t band;           // consecutive rays per XCD band (BAND_RAYS by default)
    int32_t window;         // HP_WINDOW_*: disc of buckets, or the square around it
};

// The kernel's argument number 0, which is the SearchCtx in every kernel that
// searches, and the argument after it, copied anew where a phase begins (a
// copy: read through the pointer, a field would be loaded again after every
// store).  Bound to the arguments themselves, the compiler loads all of them when the kernel
// starts; the search's own scalars then push them out to vector lanes, and
// every use costs a vector instruction per word to bring them back (a scalar
// load from the constant cache costs none).
template <typename T>
__device__ __forceinline__ T kernel_arg(size_t at)
{
    typedef const __attribute__((address_space(4))) char *ConstPtr;
    ConstPtr p = (ConstPtr)__builtin_amdgcn_kernarg_segment_ptr();
    asm volatile("" : "+s"(p));
    return *(const T *)(p + at);
}

__device__ __forceinline__ SearchCtx phase_ctx() { return kernel_arg<SearchCtx>(0); }

template <typename T>
__device__ __forceinline__ T phase_arg()
{
    return kernel_arg<T>((sizeof(SearchCtx) + alignof(T) - 1) / alignof(T) * alignof(T));
}

// One ray's geometry and search bounds, uniform across the wave that
// searches it (computed once per ray by one lane, see ray_setup).
struct RayGeom {
    int32_t vi, gx, gy;  // view, pixel position in the padded bucket grid
    int32_t h;           // window half-width in buckets; -1: nothing can be near
    float dx, dy, dz;    // unit direction (camera frame)
    float wn;            // |w|, the norm of the normalised image coordinate
    float kappa;         // Eq. 3 cone slope of this pixel (rho = kappa t), 0 in the linear mode
    float inv_L;         // 1 / L
    float z_lo, z_hi;    // depth range of possible neighbours
    float dinf;          // window radius once rho is on its linear branch
    float frL2, two_rw;  // f r L^2 and 2 r |w| of the per-bucket depth bound
    float Dmax;          // window radius in pixels
};

constexpr int RS_CAP = 16;              // rays whose set-up one pass computes
constexpr int RS_LANES = WAVE / RS_CAP;  // lanes per ray in that pass

// Neighbouring rays searched together, at most: rays of one image row whose
// windows overlap.  What a window costs (its buckets' headers, its points'
// loads, the bookkeeping that deals points to lanes) is then paid once for up
// to four rays, and only the exact predicate is evaluated for each.
constexpr int GROUP = 4;

// Keys a ray holds after a sweep step, at most (and 64 more during one).  Four
// rays share the LDS of a wave: 128 each are what the walk can sort without
// being told which 64 it needs, and 64 do for K-NP, which keeps few.  One ray
// alone, the multi-surface sampler's, has room for all its neighbours in most
// cases.
constexpr int HELD_WALK = 2 * WAVE;
constexpr int HELD_KNP = WAVE;
constexpr int HELD_SLAB = 7 * WAVE;
constexpr int BL_CAP = 3 * 64;  // listed buckets: a wave's worth, and two cells more

// A slab of the multi-surface sampler's neighbours with their points.
struct SlabList {
    float4 nb_p[WAVE];
    float nb_t[WAVE];
};

// One wave's LDS while it searches G rays, holding HELD keys of each.  A slab is
// read only between searches, in the place of what a search alone needs.
template <int G, int HELD>
struct SearchScratch {
    uint64_t pend[G][HELD + WAVE];  // keys of the neighbours found so far
    union {
        struct {
            int2 bl[BL_CAP];     // listed buckets: key, offset from the window's corner (16 bits each)
            int2 cl[WAVE];       // listed depth cells: first bucket in the window, width and prefix (16 bits each)
            int32_t head[WAVE];  // (indexed by flat point offset within a sweep step)
        };
        SlabList slab;
    };
};

// The rays a wave holds between search and walk.
struct RaySlot {
    int32_t ray;    // row of the outputs
    int32_t rs;     // set-up record
    int32_t n;      // keys held
    int32_t count;  // neighbours (any number above those asked for where there are more)
};

// The lists of the rays one walk serves (walk_batch): GROUP rows of 64
// points in (t, index) order, WALK_PAD empty entries before, between and
// after them, so that a batch of WALK_PAD entries that reaches past a list's
// ends needs no test.
constexpr int WALK_PAD = 8;
constexpr int WALK_STRIDE = WAVE + WALK_PAD;

struct WalkLists {
    float4 p[WALK_PAD + GROUP * WALK_STRIDE];
};

// Search, then walk: the two never hold data at the same time (the walk reads
// the keys into registers before it writes its lists).  LISTS begins with a
// WalkLists and may hold more that lives as long.
template <typename LISTS>
struct WalkLdsOf {
    RayGeom rs[RS_CAP];
    RaySlot slot[GROUP];
    alignas(16) unsigned char mem[sizeof(SearchScratch<GROUP, HELD_WALK>) > sizeof(LISTS)
                                      ? sizeof(SearchScratch<GROUP, HELD_WALK>)
                                      : sizeof(LISTS)];

    __device__ __forceinline__ SearchScratch<GROUP, HELD_WALK> &search()
    {
        return *reinterpret_cast<SearchScratch<GROUP, HELD_WALK> *>(mem);
    }
    __device__ __forceinline__ LISTS &lists() { return *reinterpret_cast<LISTS *>(mem); }
};
using WalkLds = WalkLdsOf<WalkLists>;
// (LDS is granted in pieces of 1,280 B: eight of them let 16 one-wave
// workgroups share a CU's 160 KB)
static_assert(sizeof(WalkLds) <= 10240, "walk LDS above 10240 B costs occupancy");

// K-NP: the search alone.
struct KnpLds {
    RayGeom rs[RS_CAP];
    RaySlot slot[GROUP];
    SearchScratch<GROUP, HELD_KNP> s;
};
static_assert(sizeof(KnpLds) <= 7680, "K-NP LDS above 7680 B costs occupancy");

// The multi-surface sampler: one ray's neighbours, a slab of 64 of them at a time
// with their points.
struct SlabLds {
    RayGeom rs[RS_CAP];
    RaySlot slot[1];
    SearchScratch<1, HELD_SLAB> s;
};
// (20 waves of a CU; see k_search_ms)
static_assert(sizeof(SlabLds) <= 7680, "slab LDS above 7680 B costs occupancy");

// Rays per XCD band: two image rows of an 800-pixel-wide view (object view
// 0.568 ms with bands of 12,800 rays, 0.545 with 3,200, 0.532 with 1,600,
// 0.534 with 800; room view 3.09, 2.83, 2.81, 2.81 ms).
constexpr int64_t BAND_RAYS = 1600;

// Two ways to share a launch's rays out, by their number.
// Up to DEALT_RAYS, and for the multi-surface sampler (whose rays are each
// long): one-wave workgroups, up to WAVE_BLOCKS of them, eight times what the
// GPU keeps resident, so that the hardware replaces those that drew little as
// they finish.
// Above: one workgroup per CU, as many waves as fit, which deal their share
// out among themselves as they go (for_each_group_banded): nothing is launched
// twice and a CU's waves end together.  The shares of the CUs are fixed, which
// costs more the fewer rays there are (us, one-wave workgroups / dealt: frame
// of 640k rays of the object 588 / 554, of 762k rays of the room 2508 / 2464,
// K-NP of 640k rays 246 / 234, search of 307k rays 389 / 386, of 160k 146 / 156,
// of 65k 99 / 126, of 16k 106 / 134).
constexpr int64_t WAVE_BLOCKS = 65536, CU_BLOCKS = 256, DEALT_RAYS = 262144;

inline bool dealt(const SearchCtx &c) { return c.blocks <= 0 && c.n_rays > DEALT_RAYS; }

// Rays per work chunk where the caller names none.  Neighbouring rays are
// searched together, so a chunk of four is the cheapest by ray; a launch of few
// rays leaves most of the GPU idle that way, or waiting for the few waves that
// drew four crowded rays, and is better split further.  The limits are those of
// the cloud whose rays differ most, an object's; a room or a plane, whose rays
// are alike, takes four earlier (us by rays per chunk 1 / 2 / 4.
// Object cloud of 1M points, squares of 64, 192, 256, 350 pixels: search 48 / 77 /
// 179, 102 / 75 / 116, 134 / 94 / 102, 199 / 129 / 94; K-NP 56 / 94 / 194, 76 / 71 /
// 139, 98 / 77 / 98, 136 / 90 / 80; search and render in one, whose CUs' shares are
// fixed, 64, 192, 400: 55 / 85 / 188, 106 / 103 / 129, 219 / 193 / 206.
// Room of 2M points, 64, 192, 256: search 107 / 140 / 340, 236 / 145 / 164, 366 / 214 /
// 150; K-NP 98 / 132 / 309, 193 / 122 / 145, 282 / 182 / 140; in one, 64, 192, 400:
// 130 / 151 / 355, 272 / 226 / 225, 878 / 667 / 568.
// Plane of 200k points, 64, 192: search 18 / 17 / 22, 93 / 54 / 34; K-NP 15 / 14 / 18,
// 73 / 42 / 27; in one, 64, 192, 400: 27 / 24 / 30, 71 / 62 / 50, 193 / 148 / 129).
// The multi-surface sampler takes its rays one at a time, each for long
// (640k rays, 400 positions 1970 / 2437 / 3290; 160k rays, 200 positions 587 / 761 / 1107).
enum SearchKind { SEARCH_WALK, SEARCH_KNP, SEARCH_FUSED };

inline int32_t default_chunk(const SearchCtx &c, SearchKind kind)
{
    if (c.sampler == HP_SAMPLER_MS && kind != SEARCH_KNP) return 1;
    const int64_t one = kind == SEARCH_FUSED ? 65536 : 6144;
    const int64_t two = kind == SEARCH_FUSED ? 196608 : kind == SEARCH_KNP ? 65536 : 49152;
    // (a cloud of few points per ray has no crowded rays to wait for: search / K-NP
    // of a plane of 200k points by rays per chunk 2 / 4, 200x200 65 / 39, 51 / 32,
    // 220x220 68 / 42, 55 / 35; object cloud of 100k 200x200 64 / 51, 44 / 37, but
    // 128x128 47 / 66, 57 / 72 and 150x150 48 / 56, 35 / 38)
    if (kind != SEARCH_FUSED && c.n_rays > 24576 && c.n_points * c.n_views < 8 * c.n_rays) return 4;
    return c.n_rays <= one ? 1 : c.n_rays <= two ? 2 : 4;
}

// Rays per work chunk of a launch.  A chunk named by the caller that is smaller
// than the default is raised to it in launches of many rays: it would leave
// neighbours to different waves, and a ray searched alone takes longer than
// its share of a group and than it took when there were none (search, us, by
// rays per chunk 1 / default, in brackets 1 before rays were searched together:
// plane of 200k points 256x256 137 / 49 [98], 500x500 261 / 148 [240]; object cloud of
// 1M points 350x350 199 / 99 [145], 500x500 294 / 175 [239]; K-NP of the plane
// 256x256 108 / 60 [86]).  Launches of up to 16,384 rays take what they are given,
// for which there are reasons either way (K-NP of the object cloud 100x100 44 / 65
// [49], search of the plane 100x100 35 / 24 [27]).
inline int32_t launch_chunk(const SearchCtx &c, SearchKind kind)
{
    const int32_t own = default_chunk(c, kind);
    if (c.chunk <= 0) return own;
    return kind != SEARCH_FUSED && c.n_rays > 16384 && c.chunk < own ? own : c.chunk;
}

// Grid of a search launch: at most `most` workgroups, a multiple of 8.
inline int64_t banded_grid(const SearchCtx &c, int64_t most)
{
    const int64_t chunks = (c.n_rays + c.chunk - 1) / c.chunk;
    const int64_t blocks = chunks < most ? chunks : most;
    if (blocks == 0) return 0;
    return blocks < 8 ? 8 : (blocks & ~(int64_t)7);
}
inline int64_t wave_grid(const SearchCtx &c) { return banded_grid(c, c.blocks > 0 ? c.blocks : WAVE_BLOCKS); }

// Search radius of a ray at parameter t.
__device__ __forceinline__ float rho_at(const SearchCtx &c, const RayGeom &g, float t)
{
    return c.rmode == HP_RADIUS_LINEAR ? search_radius(c.radius, c.inv_tref, t) : t * g.kappa;
}

__device__ __forceinline__ void lds_sync() { wave_lds_sync(); }

// ---------------------------------------------------------------------------
// cross-lane exchange: lane l receives lane l ^ j's value.  DPP for j < 16
// (row rotations act inside rows of 16 lanes), swizzle for 16, permute for 32.
// The last two run on the LDS crossbar, off the vector ALU, which bounds the
// search kernels (the gfx950 permlane swaps measured slower here for that).
// ---------------------------------------------------------------------------
template <int J>
__device__ __forceinline__ uint32_t xor_lane_u32(uint32_t v)
{
    // (mov_dpp with every row and bank enabled writes all lanes: no old value)
    const int x = (int)v;
    if constexpr (J == 1) return (uint32_t)__builtin_amdgcn_mov_dpp(x, 0xB1, 0xF, 0xF, false);
    if constexpr (J == 2) return (uint32_t)__builtin_amdgcn_mov_dpp(x, 0x4E, 0xF, 0xF, false);
    if constexpr (J == 4) {
        const int down = __builtin_amdgcn_mov_dpp(x, 0x124, 0xF, 0xF, false);  // from l - 4
        const int up = __builtin_amdgcn_mov_dpp(x, 0x12C, 0xF, 0xF, false);    // from l + 4
        return (uint32_t)((lane_id() & 4) ? down : up);
    }
    if constexpr (J == 8) return (uint32_t)__builtin_amdgcn_mov_dpp(x, 0x128, 0xF, 0xF, false);
    if constexpr (J == 16) return (uint32_t)__builtin_amdgcn_ds_swizzle(x, 0x401F);
    return (uint32_t)__shfl_xor(x, J, WAVE);
}

template <int J>
__device__ __forceinline__ uint64_t xor_lane_u64(uint64_t v)
{
    const uint32_t lo = xor_lane_u32<J>((uint32_t)v);
    const uint32_t hi = xor_lane_u32<J>((uint32_t)(v >> 32));
    return ((uint64_t)hi << 32) | lo;
}

// The lanes whose index has bit k set, as a 64-bit lane mask.
constexpr uint64_t lane_bit_mask(int k)
{
    return k == 0   ? 0xAAAAAAAAAAAAAAAAull
           : k == 1 ? 0xCCCCCCCCCCCCCCCCull
           : k == 2 ? 0xF0F0F0F0F0F0F0F0ull
           : k == 3 ? 0xFF00FF00FF00FF00ull
           : k == 4 ? 0xFFFF0000FFFF0000ull
                    : 0xFFFFFFFF00000000ull;
}

// Per-lane predicate "bit i of mask M" from a constant mask: the compiler
// builds the mask with two scalar moves where it is used, where a lane-index
// test was kept in a scalar register pair for the whole kernel (six of them
// for the sorts) and pushed other scalars out to vector lanes.
template <uint64_t M>
__device__ __forceinline__ bool lanes_in(void)
{
    return __builtin_amdgcn_inverse_ballot_w64(M);
}

constexpr int log2_lane(int j) { return j == 1 ? 0 : j == 2 ? 1 : j == 4 ? 2 : j == 8 ? 3 : j == 16 ? 4 : 5; }

// One compare-exchange stage in which every block ascends: lanes l and l ^ J
// keep the minimum in the lower lane (one 64-bit compare, two selects).
template <int J>
__device__ __forceinline__ uint64_t cx_stage(uint64_t x, int)
{
    const uint64_t y = xor_lane_u64<J>(x);
    const bool take = (y < x) != lanes_in<lane_bit_mask(log2_lane(J))>();
    return take ? y : x;
}

template <int J>
__device__ __forceinline__ uint64_t cx_merge(uint64_t x, int l)
{
    x = cx_stage<J>(x, l);
    if constexpr (J > 1) x = cx_merge<J / 2>(x, l);
    return x;
}

// Inverts the keys of the lanes whose lane-index bits A and B differ (B = -1:
// bit A alone): bitwise NOT reverses the order of keys.
template <int A, int B>
__device__ __forceinline__ uint64_t flip_keys(uint64_t x)
{
    constexpr uint64_t m = lane_bit_mask(A) ^ (B >= 0 ? lane_bit_mask(B) : 0ull);
    return lanes_in<m>() ? ~x : x;
}

// Bitonic sort of one key per lane across the wave.  In the merge of blocks
// of K lanes, the blocks that must descend hold inverted keys, so that every
// stage is the same ascending compare-exchange; the keys are re-inverted
// between block sizes as the block directions change.
__device__ __forceinline__ uint64_t wave_sort_fast(uint64_t x)
{
    const int l = lane_id();
    x = flip_keys<1, -1>(x);  // K = 2 blocks descend where lane bit 1 is set
    x = cx_merge<1>(x, l);
    x = flip_keys<1, 2>(x);
    x = cx_merge<2>(x, l);
    x = flip_keys<2, 3>(x);
    x = cx_merge<4>(x, l);
    x = flip_keys<3, 4>(x);
    x = cx_merge<8>(x, l);
    x = flip_keys<4, 5>(x);
    x = cx_merge<16>(x, l);
    x = flip_keys<5, -1>(x);  // one block of 64: ascends
    x = cx_merge<32>(x, l);
    return x;
}

// Lane p of each quad's value, on all four lanes (p a constant after unrolling).
__device__ __forceinline__ uint32_t quad_bcast_u32(uint32_t v, int p)
{
    const int x = (int)v;
    switch (p) {
    case 0: return (uint32_t)__builtin_amdgcn_mov_dpp(x, 0x00, 0xF, 0xF, false);
    case 1: return (uint32_t)__builtin_amdgcn_mov_dpp(x, 0x55, 0xF, 0xF, false);
    case 2: return (uint32_t)__builtin_amdgcn_mov_dpp(x, 0xAA, 0xF, 0xF, false);
    default: return (uint32_t)__builtin_amdgcn_mov_dpp(x, 0xFF, 0xF, 0xF, false);
    }
}

__device__ __forceinline__ uint64_t quad_bcast_u64(uint64_t v, int p)
{
    return ((uint64_t)quad_bcast_u32((uint32_t)(v >> 32), p) << 32) | quad_bcast_u32((uint32_t)v, p);
}

__device__ __forceinline__ uint64_t readlane_u64(uint64_t v, int l)
{
    const uint32_t lo = (uint32_t)__builtin_amdgcn_readlane((int)(uint32_t)v, l);
    const uint32_t hi = (uint32_t)__builtin_amdgcn_readlane((int)(uint32_t)(v >> 32), l);
    return ((uint64_t)hi << 32) | lo;
}

// Inclusive prefix maximum across the wave (row shifts, then row broadcasts).
// Lanes without a source read INT_MIN, the identity of max, which lets the
// compiler fold each shift into its max instruction.
__device__ __forceinline__ int wave_prefix_max_i32(int v)
{
    constexpr int I = (int)0x80000000;
    v = max(v, __builtin_amdgcn_update_dpp(I, v, 0x111, 0xF, 0xF, false));  // row_shr:1
    v = max(v, __builtin_amdgcn_update_dpp(I, v, 0x112, 0xF, 0xF, false));  // row_shr:2
    v = max(v, __builtin_amdgcn_update_dpp(I, v, 0x113, 0xF, 0xF, false));  // row_shr:3
    v = max(v, __builtin_amdgcn_update_dpp(I, v, 0x114, 0xF, 0xE, false));  // row_shr:4
    v = max(v, __builtin_amdgcn_update_dpp(I, v, 0x118, 0xF, 0xC, false));  // row_shr:8
    v = max(v, __builtin_amdgcn_update_dpp(I, v, 0x142, 0xA, 0xF, false));  // row_bcast:15
    v = max(v, __builtin_amdgcn_update_dpp(I, v, 0x143, 0xC, 0xF, false));  // row_bcast:31
    return v;
}

// Minimum depth over the depth cells holding the buckets within h of grid
// position (gx, gy) (+inf if they are all empty), by the RS_LANES lanes of a
// group (sub = lane within the group; every lane of the group returns it).
__device__ __forceinline__ float group_cells_zmin(const SearchCtx &c, const ViewK &V, int gx, int gy,
                                                  int h, int sub)
{
    const int cx0 = max(gx - h, 0) >> CELL_SHIFT, cx1 = min(gx + h, V.Wg - 1) >> CELL_SHIFT;
    const int cy0 = max(gy - h, 0) >> CELL_SHIFT, cy1 = min(gy + h, V.Hg - 1) >> CELL_SHIFT;
    float z = __builtin_inff();
    // cells in row-major order, cell sub, sub + RS_LANES, ... of the block to
    // this lane, four loads in flight at a time (a load per step of a nested
    // loop waited for each in turn); the minimum does not depend on the order
    const int nx = cx1 - cx0 + 1, ny = cy1 - cy0 + 1;
    const int ncell = (nx > 0 && ny > 0) ? nx * ny : 0;  // (nx >= 1 below)
    int cx = cx0 + sub, cy = cy0;
    if (ncell > 0)
        while (cx > cx1 && cy <= cy1) cx -= nx, ++cy;
    for (int ci = sub; ci < ncell; ci += 4 * RS_LANES) {
        float v[4];
#pragma unroll
        for (int j = 0; j < 4; ++j) {
            v[j] = ci + j * RS_LANES < ncell ? __uint_as_float(c.cell_zmin[V.cell_base + cy * V.ncx + cx])
                                             : __builtin_inff();
            cx += RS_LANES;
            while (cx > cx1 && cy <= cy1) cx -= nx, ++cy;
        }
#pragma unroll
        for (int j = 0; j < 4; ++j) z = __builtin_fminf(z, v[j]);
    }
    static_assert(RS_LANES == 4 || RS_LANES == 8, "groups of four or eight lanes");
    z = __builtin_fminf(z, __uint_as_float(xor_lane_u32<1>(__float_as_uint(z))));
    z = __builtin_fminf(z, __uint_as_float(xor_lane_u32<2>(__float_as_uint(z))));
    if constexpr (RS_LANES == 8)
        z = __builtin_fminf(z, __uint_as_float(xor_lane_u32<4>(__float_as_uint(z))));
    return z;
}

// Reciprocal for the search bounds only (within a few ulp: every bound
// carries a relative margin of at least 1e-4; the exact predicate decides).
__device__ __forceinline__ float bound_rcp(float x) { return __builtin_amdgcn_rcpf(x); }

// Window radius (pixels) for neighbours whose depth is at least zmin.
__device__ __forceinline__ float radius_for_depth(const SearchCtx &c, float kappa, float L, float wn,
                                                  float f, float L2, float zmin, float dcap,
                                                  float dinf)
{
    // a pure cone projects to a disc whose radius does not depend on depth
    if (c.rmode != HP_RADIUS_LINEAR) return dinf < dcap ? dinf : dcap;
    const float k = c.radius * c.inv_tref;
    float t = (L * zmin - wn * c.radius) * bound_rcp(1.0f + wn * k);
    t = t * 0.9999f - 1e-6f;
    if (!(t > c.t_near)) t = c.t_near;
    const float rho = search_radius(c.radius, c.inv_tref, t);
    const float den = t - rho * wn;
    if (!(den > 0.0f)) return dcap;
    const float d = (f * rho * L2 * bound_rcp(den)) * 1.0001f + 0.01f;
    return d < dcap ? d : dcap;
}

// Geometry and search bounds of one ray, computed by a group of RS_LANES
// lanes (sub = lane within the group), which share the depth-cell rounds.  The window:
// a neighbour projects at most delta(t) = f rho L^2 / (t - rho |w|) pixels
// from the pixel centre, and delta does not grow with t; the smallest depth
// of the depth cells around the pixel bounds t from below, so two rounds
// (each over the cells of the previous radius) shrink the window from the
// view-wide bound.  If every such cell is empty, no point is near the ray.
__device__ __forceinline__ int ray_view(const SearchCtx &c, int64_t ray)
{
    // bisection over the views' first rays (a walk along the list waits for
    // each load in turn): views[lo].ray_base <= ray < views[hi].ray_base
    int lo = 0, hi = c.n_views;
    while (hi - lo > 1) {
        const int mid = (lo + hi) >> 1;
        if (c.views[mid].ray_base <= ray) lo = mid;
        else hi = mid;
    }
    return lo;
}

// Window half-width of the first depth-cell round: the view-wide bound.
__device__ __forceinline__ int first_round_h(const ViewK &V)
{
    return min((int)__builtin_floorf(V.dmax + 0.5f), V.g);
}

// Minimum depth of the cells within the view-wide window of a ray (+inf:
// no point can be near it), by a group of RS_LANES lanes.
__device__ __forceinline__ float ray_first_zmin(const SearchCtx &c, int64_t ray, int sub)
{
    const int vi = ray_view(c, ray);
    const ViewK &V = c.views[vi];
    const int local = (int)(ray - V.ray_base);
    return group_cells_zmin(c, V, local % V.W + V.g, local / V.W + V.g, first_round_h(V), sub);
}

// (zmin1: the first round's minimum depth, ray_first_zmin, already taken; u: the ray's pixel column)
__device__ __forceinline__ RayGeom ray_setup(const SearchCtx &c, int64_t ray, int sub, float zmin1, int &u)
{
    RayGeom g;
    const int vi = ray_view(c, ray);
    const ViewK &V = c.views[vi];
    const int local = (int)(ray - V.ray_base);
    const int v = local / V.W;
    u = local % V.W;
    float a, b, L;
    ray_dir(V, u, v, g.dx, g.dy, g.dz, a, b, L);
    g.vi = vi;
    g.wn = __builtin_sqrtf(a * a + b * b);
    // Eq. 3 on the unit-focal image plane: BF = rddot / L over AB, AF or AE
    g.kappa = 0.0f;
    if (c.rmode != HP_RADIUS_LINEAR) {
        const float bf = c.rddot / L;
        if (c.rmode == HP_RADIUS_EQ3) {
            const float m = g.wn - c.rddot;
            g.kappa = bf / __builtin_sqrtf(fma_rn(m, m, 1.0f));
        } else if (c.rmode == HP_RADIUS_EQ3_AF) {
            g.kappa = bf / fma_rn(-bf, g.wn, L);
        } else {
            g.kappa = bf / L;
        }
    }
    const float L2 = fma_rn(g.wn, g.wn, 1.0f);
    const float f = V.fx > V.fy ? V.fx : V.fy;
    const float rho_n = rho_at(c, g, c.t_near);
    const float rho_f = rho_at(c, g, c.t_far);
    g.inv_L = bound_rcp(L);
    g.z_lo = ((c.t_near - g.wn * rho_n) * g.inv_L) * 0.999f - 1e-6f;
    g.z_hi = ((c.t_far + g.wn * rho_f) * g.inv_L) * 1.001f + 1e-6f;
    // pixel offset bound once rho has reached its linear branch
    g.dinf = 0.0f;
    const float klin = c.rmode == HP_RADIUS_LINEAR ? c.radius * c.inv_tref : g.kappa;
    if (klin > 0.0f) {
        const float den = 1.0f - klin * g.wn;
        g.dinf = den > 0.0f ? (f * klin * L2 * bound_rcp(den)) * 1.001f + 0.01f : __builtin_inff();
    }
    g.frL2 = f * c.radius * L2;
    g.two_rw = 2.0f * c.radius * g.wn;
    g.gx = u + V.g;
    g.gy = v + V.g;
    float Dmax = V.dmax;
    int h = first_round_h(V);
    for (int round = 0; round < 2; ++round) {
        const float zmin = round == 0 ? zmin1 : group_cells_zmin(c, V, g.gx, g.gy, h, sub);
        if (!(zmin < __builtin_inff())) {
            h = -1;  // no point anywhere near this ray
            break;
        }
        Dmax = radius_for_depth(c, g.kappa, L, g.wn, f, L2, zmin, Dmax, g.dinf);
        h = min((int)__builtin_floorf(Dmax + 0.5f), V.g);
    }
    g.h = h;
    g.Dmax = Dmax;
    return g;
}

__device__ __forceinline__ float uniform_f32(float v)
{
    return __int_as_float(__builtin_amdgcn_readfirstlane(__float_as_int(v)));
}

__device__ __forceinline__ int uniform_i32(int v) { return __builtin_amdgcn_readfirstlane(v); }

// A ray's set-up as the whole wave reads it back from the LDS.  A ray with
// nothing near it (h < 0) needs no more than h.
__device__ __forceinline__ RayGeom load_ray(const RayGeom &src)
{
    RayGeom g;
    g.h = uniform_i32(src.h);
    if (g.h < 0) {
        g.vi = g.gx = g.gy = 0;
        g.dx = g.dy = g.dz = g.wn = g.kappa = g.inv_L = 0.0f;
        g.z_lo = g.z_hi = g.dinf = g.frL2 = g.two_rw = g.Dmax = 0.0f;
        return g;
    }
    g.vi = uniform_i32(src.vi);
    g.gx = uniform_i32(src.gx);
    g.gy = uniform_i32(src.gy);
    g.dx = uniform_f32(src.dx);
    g.dy = uniform_f32(src.dy);
    g.dz = uniform_f32(src.dz);
    g.wn = uniform_f32(src.wn);
    g.kappa = uniform_f32(src.kappa);
    g.inv_L = uniform_f32(src.inv_L);
    g.z_lo = uniform_f32(src.z_lo);
    g.z_hi = uniform_f32(src.z_hi);
    g.dinf = uniform_f32(src.dinf);
    g.frL2 = uniform_f32(src.frL2);
    g.two_rw = uniform_f32(src.two_rw);
    g.Dmax = uniform_f32(src.Dmax);
    return g;
}

// Rays from ray i of a pass on that are searched together, at most `most`
// <= GROUP: bit RS_LANES k of `joined` is set where ray k follows ray k - 1.
__host__ __device__ constexpr int group_size(uint64_t joined, int i, int most)
{
    // (the bits from ray i on come down first, so that no shift below reaches
    // the width of the mask, whichever ray is the pass's last)
    const uint64_t run = joined >> (RS_LANES * i);
    int m = 1;
    while (m < most && ((run >> (RS_LANES * m)) & 1ull)) ++m;
    return m;
}
static_assert(RS_LANES * RS_CAP == WAVE && group_size(~0ull, RS_CAP - 1, GROUP) == 1 &&
                  group_size(~0ull, 0, GROUP) == GROUP,
              "groups end with the pass");

// Persistent iteration over the rays of a launch.  Workgroups take chunks of
// c.chunk consecutive rays (neighbouring pixels share table buckets).  They are
// dealt to the eight XCDs round-robin (workgroup b runs on XCD b % 8), each with
// its own L2, so the chunks are grouped into bands of BAND_RAYS consecutive rays
// and XCD x takes bands x, x + 8, ...: the rays one XCD's workgroups search at
// a time are then neighbours and share that L2's table lines.  Within its
// bands an XCD's workgroups stride by their number, so each still sees a mix
// of empty and busy regions.  The grid must be a multiple of 8.
// The per-ray set-up (divisions, square roots, the depth-cell rounds) is
// uniform work that a whole wave would repeat on every lane; groups of lanes
// instead compute it for up to RS_CAP rays of the chunk at once into the LDS.
// The first depth-cell round goes first: a ray whose view-wide window holds
// no point (most rays of a view that an object does not fill) is finished
// there by empty(ray), called on one lane per such ray, and neither gets the
// rest of the set-up nor a pass of the wave.  groups(n, ray, first, last) is then
// called for the others, up to MAXG rays of one image row with consecutive
// pixels at a time: their number, the first one's number (rays numbered from
// the launch's first one, which is their row in the outputs) and its record
// (the others' follow), and whether this pass ends with them.
// The NW waves of a workgroup take its chunks as they come, by the counter
// `take` in its LDS (zero at first): up to four at a time, fewer towards the
// end (measured on the frames above, search and render in one: 569 us with a
// fixed deal, 467 with passes taken as they come, 425 with the last ones short).
template <int MAXG, int NW, typename Groups, typename Empty>
__device__ __forceinline__ void for_each_group_banded(RayGeom *rs, int *take, Groups groups, Empty empty)
{
    const SearchCtx cl = phase_ctx();
    // (chunk, band and slot numbers in 32 bits: a launch has fewer than 2^31
    // rays, so every chunk number below fits an unsigned 32-bit integer, and
    // 64-bit ones held scalar registers that the body then spilled)
    const uint32_t n_chunks = (uint32_t)((cl.n_rays + cl.chunk - 1) / cl.chunk);
    const uint32_t chunk = (uint32_t)cl.chunk, n_rays = (uint32_t)cl.n_rays;
    // chunks per band (fewer when the launch has fewer than eight full bands,
    // so that every XCD gets a share)
    uint32_t band = (uint32_t)(((int64_t)cl.band + cl.chunk - 1) / cl.chunk);
    if ((uint64_t)band * 8 > n_chunks) band = (n_chunks + 7) / 8 > 0 ? (n_chunks + 7) / 8 : 1;
    const uint32_t xcd = blockIdx.x & 7;
    const uint32_t slot = blockIdx.x >> 3, n_slots = gridDim.x >> 3;
    const uint32_t n_bands = (n_chunks + band - 1) / band;
    const uint32_t my_chunks = (n_bands > xcd ? (n_bands - xcd + 7) / 8 : 0) * band;
    // first ray (relative to c.ray0) and ray count of this workgroup's li-th chunk
    auto chunk_rays = [&](uint32_t li, uint32_t &r0, int &n) {
        n = 0;
        r0 = 0;
        if (li >= my_chunks) return;
        const uint32_t ch = (xcd + 8 * (li / band)) * band + li % band;
        if (ch >= n_chunks) return;
        r0 = ch * chunk;
        n = (int)min(chunk, n_rays - r0);
    };
    // its share of them, up to four at a time (the chunks themselves stay
    // small, for balance), or RS_CAP rays' worth where none is searched with
    // its neighbours
    const uint32_t mine = slot < my_chunks ? (my_chunks - slot + n_slots - 1) / n_slots : 0;
    const uint32_t most = MAXG == 1 && NW == 1 && chunk < 4 ? RS_CAP / chunk : 4;
    for (uint32_t at = 0;;) {
        // (no chunk past the workgroup's last: sixteen of them ahead, in a grid as
        // large as a launch may have, would pass 2^32)
        uint32_t per = MAXG == 1 ? min(most, mine - at) : most;
        const int l = phase_lane_id();
        if constexpr (NW > 1) {
            per = min(max((mine - at) / (2 * NW), 1u), most);
            int j = 0;
            if (l == 0) j = atomicAdd(take, (int)per);
            at = (uint32_t)uniform_i32(j);
        }
        if (at >= mine) break;
        const uint32_t li = slot + at * n_slots;
        if constexpr (NW == 1) at += per;
        const SearchCtx c = phase_ctx();
        // n rays of a pass, lanes 4 k .. 4 k + 3 set up the k-th, ray rk (lanes
        // past the pass repeat its last ray)
        const int k = l / RS_LANES, sub = l % RS_LANES;
        auto pass = [&](uint32_t rk, int n) {
            const float z1 = ray_first_zmin(c, c.ray0 + rk, sub);
            const bool lead = sub == 0 && k < n;
            const uint64_t near = ballot(lead && z1 < __builtin_inff());  // bit RS_LANES k
            if (lead && !(z1 < __builtin_inff())) empty((int64_t)rk);
            if (near == 0) return;
            lds_sync();
            int u;
            const RayGeom gk = ray_setup(c, c.ray0 + rk, sub, z1, u);
            if (lead) rs[k] = gk;
            lds_sync();
            // rays whose left neighbour is the one before them in this pass
            const int prev = __shfl_up((int)rk, RS_LANES, WAVE);
            const uint64_t joined = near & (near << RS_LANES) & ballot((int)rk == prev + 1) &
                                    ballot(u > 0);
            for (uint64_t todo = near; todo != 0;) {
                const int i = __builtin_ctzll(todo) / RS_LANES;
                const int m = group_size(joined, i, MAXG);
                todo &= ~(((1ull << (RS_LANES * m)) - 1ull) << (RS_LANES * i));
                groups(m, readlane_i32((int)rk, RS_LANES * i), i, todo == 0);
            }
        };
        if constexpr (MAXG == 1) {
            for (uint32_t s0 = 0; s0 < per * chunk; s0 += RS_CAP) {
                // the k-th ray of these chunks (those past the last one follow all others)
                const uint32_t i = s0 + k;
                const uint32_t j = (uint32_t)(((float)i + 0.5f) * __builtin_amdgcn_rcpf((float)chunk));
                uint32_t r;
                int have;
                chunk_rays(j < per ? li + j * n_slots : ~0u, r, have);
                r += i - j * chunk;
                const bool in = (int)(i - j * chunk) < have;
                const int n = popc64(ballot(in)) / RS_LANES;
                if (n == 0) break;
                pass(in ? r : (uint32_t)readlane_i32((int)r, RS_LANES * (n - 1)), n);
            }
        } else {
            uint32_t ra, rb, rc, rd;
            int na, nb, nc, nd;
            chunk_rays(li, ra, na);
            chunk_rays(per > 1 ? li + n_slots : ~0u, rb, nb);
            chunk_rays(per > 2 ? li + 2 * n_slots : ~0u, rc, nc);
            chunk_rays(per > 3 ? li + 3 * n_slots : ~0u, rd, nd);
            const int nab = na + nb, nabc = nab + nc, ntot = nabc + nd;
            for (int s0 = 0; s0 < ntot; s0 += RS_CAP) {
                const int n = min(RS_CAP, ntot - s0), i = s0 + min(k, n - 1);
                pass(i < na ? ra + i : i < nab ? rb + (i - na) : i < nabc ? rc + (i - nab) : rd + (i - nabc), n);
            }
        }
    }
}

// Keep the `want` smallest of the n > want pending keys (n <= CAP) and at
// most `spare` others, in any order, at the front of `pend`; n becomes their
// number.  Returns an upper half that no dropped key's is below and no kept
// key's above.  The cut is found as quickselect finds it, on the keys' upper
// halves: one of the keys still in question is the next pivot, and a ballot
// and a population count per register of keys tell its rank (two or three
// steps where `spare` is 64; bisection of the range of values takes fifteen,
// and sorting every 64 keys that arrive and merging them into a sorted list
// took four times the vector instructions of that).  Equal upper halves at
// the cut are told apart by bisection on the lower halves.
template <int CAP>
__device__ __forceinline__ uint32_t keep_smallest(uint64_t *pend, int &n, int want, int spare)
{
    constexpr int NR = (CAP + WAVE - 1) / WAVE;
    const int l = phase_lane_id();
    lds_sync();
    // (upper halves are bits of non-negative binary32 values, infinity
    // included; the padding lies above all of them)
    int hi[NR];
    uint32_t lo[NR];
#pragma unroll
    for (int k = 0; k < NR; ++k) {
        const uint64_t key = WAVE * k + l < n ? pend[WAVE * k + l] : 0x7fffffffffffffffull;
        hi[k] = (int)(key >> 32);
        lo[k] = (uint32_t)key;
    }
    lds_sync();
    // fewer than `want` keys at or below a, s >= `want` at or below b
    int a = -1, b = 0x7ffffffe, s = n;
    while (s > want + spare) {
        int pivot = -1;
#pragma unroll
        for (int k = 0; k < NR; ++k) {
            const uint64_t in = ballot(hi[k] > a) & ballot(hi[k] < b);
            if (in) pivot = readlane_i32(hi[k], __builtin_ctzll(in));
        }
        if (pivot < 0) break;  // all that are left equal b
        int t = 0;
#pragma unroll
        for (int k = 0; k < NR; ++k) t += popc64(ballot(hi[k] <= pivot));
        if (t >= want) {
            b = pivot;
            s = t;
        } else {
            a = pivot;
        }
    }
    uint32_t cut = ~0u;  // lower halves kept at upper half b
    if (s > want + spare) {
        int need = want;  // of the keys at b
#pragma unroll
        for (int k = 0; k < NR; ++k) need -= popc64(ballot(hi[k] < b));
        auto tied = [&](uint32_t v) {
            int t = 0;
#pragma unroll
            for (int k = 0; k < NR; ++k) t += popc64(ballot(hi[k] == b) & ballot(lo[k] <= v));
            return t;
        };
        uint32_t c = 0u;
        if (tied(0u) >= need) {
            cut = 0u;
        } else {
            while (cut - c > 1u) {
                const uint32_t mid = c + ((cut - c) >> 1);
                if (tied(mid) >= need) cut = mid;
                else c = mid;
            }
        }
    }
    int at = 0;
#pragma unroll
    for (int k = 0; k < NR; ++k) {
        const uint64_t m = ballot(hi[k] < b) | (ballot(hi[k] == b) & ballot(lo[k] <= cut));
        if (in_mask(m)) pend[at + rank_below(m)] = ((uint64_t)(uint32_t)hi[k] << 32) | lo[k];
        at += popc64(m);
    }
    n = at;
    lds_sync();
    return (uint32_t)b;
}

// Windows of up to ROW_WIN rows that hold up to ROW_POINTS points are searched
// as runs of consecutive table slots, one lane per run.
// K-NP, which meets a ray's points in no order of depth and so must test nearly
// all of its window anyway, takes the runs of windows ten times as crowded
// (us, by limit 640 / 3,200 / 6,400: K-NP of the object cloud of 1M points at
// 350x350 92 / 93 / 81, 500x500 147 / 126 / 113, 800x800 236 / 211 / 210; a room of 5M,
// whose windows are deeper, gives some of it back, 350x350 155 / 169 / 215, 800x800
// 678 / 681 / 681; without a limit a room of 2M seen at 64x64 takes 586 instead of 98).
constexpr int ROW_WIN = 15;
constexpr int ROW_POINTS = 640;
constexpr int ROW_POINTS_KNP = 6400;

__device__ __forceinline__ float quad_max_f32(float v)
{
    v = __builtin_fmaxf(v, __uint_as_float(xor_lane_u32<1>(__float_as_uint(v))));
    return __builtin_fmaxf(v, __uint_as_float(xor_lane_u32<2>(__float_as_uint(v))));
}

__device__ __forceinline__ float quad_min_f32(float v) { return -quad_max_f32(-v); }

// Search the ng rays (ng <= G) of slots s0 .. s0 + ng - 1: neighbours in one
// image row, their records in the slots.  Leaves in each ray's row of
// sh.pend its `want` <= 64 smallest (t, index) keys (or all) and perhaps a few
// more, in no order, at most `most` <= HELD of them, and in its slot their
// number and the number of neighbours (any number above `want` where
// there are more); with `lo`, only the keys >= lo count (the
// multi-surface sampler walks a ray's neighbours 64 at a time this way).
// BY_E2 orders the kept neighbours by (squared distance to the ray, index)
// instead of (t, index): the K nearest points to the ray (K-NP, Eq. 1).
//
// The rays' windows are searched as one, under bounds that hold for each of
// them, and every point met is tested against each ray.  Three ways to the
// points, chosen by what the window holds; the kept keys are the same:
//  - runs: the buckets of a window row that are consecutive keys (the whole
//    row in a row-major table, its part in each tile of a tiled one) hold
//    consecutive slots, bounded by two offsets.  Small windows of few points
//    take the runs' points flattened across the lanes, with no look at the
//    buckets (no bucket is skipped for its depth: testing its points costs
//    less than looking at it);
//  - buckets: elsewhere the buckets of the 8x8-bucket cells that reach into
//    the window are probed and those that may hold a neighbour listed; they
//    are taken 64 at a time, one per lane (fewer: several lanes each), and the
//    lanes walk their bucket's points from the nearest on.  Buckets are ordered by depth, so the first
//    points of all of them are the front of what the rays meet: once more
//    than 64 neighbours of each ray are known, points too deep to be among
//    the 64 nearest are not visited any more, nor buckets behind them;
//  - what few lanes are left with, the tails of crowded buckets, is flattened
//    across the wave like the runs.
template <int G, int HELD, bool BY_E2 = false>
__device__ __forceinline__ void search_group(const RayGeom *rs, RaySlot *slot, SearchScratch<G, HELD> &sh, int s0,
                                             int ng, int want, int most, uint64_t lo = 0)
{
    const SearchCtx c = phase_ctx();
    const int l = phase_lane_id();
    // ray q of the group on lanes q, q + 4, ...
    const RayGeom R = rs[slot[s0 + min(l & 3, ng - 1)].rs];
    const int h = (int)uniform_f32(quad_max_f32((float)R.h));  // (half-widths are far below 2^24)
    float dx[G], dy[G], dz[G], kappa[G], zh[G];
    int count[G], np[G];
    uint32_t tau[G];  // no key with a larger upper half is among the `want` smallest
#pragma unroll
    for (int r = 0; r < G; ++r) {
        dx[r] = readlane_f32(R.dx, r);
        dy[r] = readlane_f32(R.dy, r);
        dz[r] = readlane_f32(R.dz, r);
        kappa[r] = readlane_f32(R.kappa, r);
        zh[r] = readlane_f32(R.z_hi, r);
        count[r] = np[r] = 0;
        tau[r] = ~0u;
    }
    const float wn_max = uniform_f32(quad_max_f32(R.wn));
    const float z_lo = uniform_f32(quad_min_f32(R.z_lo)), dinf = uniform_f32(quad_max_f32(R.dinf));
    float z_hi = uniform_f32(quad_max_f32(R.z_hi));
    const float frL2 = uniform_f32(quad_max_f32(R.frL2)), two_rw = uniform_f32(quad_max_f32(R.two_rw));
    const float inv_L = uniform_f32(quad_max_f32(R.inv_L)), Dmax = uniform_f32(quad_max_f32(R.Dmax));
    const int gy = uniform_i32(R.gy), gx0 = readlane_i32(R.gx, 0), gx1 = gx0 + ng - 1;
    const ViewK &V = c.views[uniform_i32(R.vi)];
    // (the square window also visits the corners beyond the proven radius)
    const bool square = c.window == HP_WINDOW_SQUARE;
    ViewK Vg;
    Vg.Wg = V.Wg;
    Vg.Hg = V.Hg;
    Vg.bucket_base = V.bucket_base;
    const int Wg = Vg.Wg, Hg = Vg.Hg, cell_base = V.cell_base, ncx = V.ncx;

    auto rho_of = [&](int r, float t) {
        return c.rmode == HP_RADIUS_LINEAR ? search_radius(c.radius, c.inv_tref, t) : t * kappa[r];
    };
    // keep the keys that fit: when more are held than a step's 64 would
    // leave room for
    auto cut_back = [&]() {
#pragma unroll
        for (int r = 0; r < G; ++r) {
            if (np[r] <= HELD) continue;
            // (a wide tolerance costs fewer steps, a narrow one lets fewer
            // later keys by; short lists gain more from the second)
            const int spare = BY_E2 ? min(HELD - want, 24) : min(HELD - want, WAVE);
            tau[r] = keep_smallest<HELD + WAVE>(sh.pend[s0 + r], np[r], want, spare);
            if constexpr (!BY_E2) {
                // (as z_hi at t_far: a neighbour at parameter t is at most this deep)
                const float tt = __uint_as_float(tau[r]);
                zh[r] = __builtin_fminf(zh[r], ((tt + wn_max * rho_of(r, tt)) * inv_L) * 1.001f + 1e-6f);
            }
        }
        if constexpr (!BY_E2) {
            z_hi = zh[0];
#pragma unroll
            for (int r = 1; r < G; ++r) z_hi = r < ng ? __builtin_fmaxf(z_hi, zh[r]) : z_hi;
            z_hi = uniform_f32(z_hi);
        }
    };
    // the exact predicate on one point per lane of mask `valid`; passing keys
    // are appended (lane masks of single comparisons, combined by the scalar
    // unit: a mask of a compound condition costs two vector instructions more)
    auto test_points = [&](uint64_t valid, const float4 &P) {
        bool full = false;
#pragma unroll
        for (int r = 0; r < G; ++r) {
            if (r >= ng) break;
            const float t = ray_param(P.x, P.y, P.z, dx[r], dy[r], dz[r]);
            const float e2 = dist2_at(P.x, P.y, P.z, dx[r], dy[r], dz[r], t);
            const float rho = rho_of(r, t);
            const uint32_t hi = __float_as_uint(BY_E2 ? e2 : t);
            const uint64_t key = ((uint64_t)hi << 32) | __float_as_uint(P.w);
            uint64_t live = valid & ballot(t >= c.t_near) & ballot(t <= c.t_far) & ballot(e2 <= rho * rho);
            if (lo != 0) live &= ballot(key >= lo);
            if (live == 0) continue;
            count[r] += popc64(live);
            const uint64_t km = live & ballot(hi <= tau[r]);
            if (in_mask(km)) sh.pend[s0 + r][np[r] + rank_below(km)] = key;
            np[r] += popc64(km);
            full |= np[r] > HELD;
        }
        if (full) cut_back();
    };
    auto load_point = [&](int slot_no) {
        float4 P = c.pts[slot_no];
        // one 16-byte load: otherwise the compiler loads the components in
        // two dependent pieces
        asm volatile("" : "+v"(P.x), "+v"(P.y), "+v"(P.z), "+v"(P.w));
        return P;
    };
    // the points of one run of slots per lane, at .. at + cnt - 1, flattened
    // across the wave; with `deep`, only up to the lane's depth bound zmax
    auto sweep_flat = [&](int at, int cnt, bool deep, float zmax) {
        const int inc = wave_incl_scan_i32(cnt);
        const int totp = readlane_i32(inc, WAVE - 1);
        const int pre = inc - cnt;
        const int shift = at - pre;  // slot of flat point p of this lane's run: p + shift
        int carry = 0;
        for (int p0 = 0; p0 < totp; p0 += WAVE) {
            // run of flat point p0 + l: the last run head at or before it
            lds_sync();
            sh.head[l] = -1;
            lds_sync();
            if (cnt > 0 && pre >= p0 && pre < p0 + WAVE) sh.head[pre - p0] = l;
            lds_sync();
            int own = sh.head[l];
            if (l == 0 && own < 0) own = carry;
            own = wave_prefix_max_i32(own);
            carry = readlane_i32(own, WAVE - 1);
            const int left = totp - p0;
            const int slot_no = p0 + l + __shfl(shift, own, WAVE);
            // (lanes past the end load the table's first point)
            const float4 P = load_point(l < left ? slot_no : 0);
            uint64_t in = left >= WAVE ? ~0ull : ~(~0ull << left);
            if (deep) {
                const float zm = __builtin_fminf(__shfl(zmax, own, WAVE), z_hi);
                in &= ballot(P.z <= zm) & ballot(P.z >= z_lo);
            }
            test_points(in, P);
        }
    };
    // the points of `share` neighbouring lanes' bucket, each lane every share-th
    // one from `at` on: slots up to end - 1 (none: end <= at), depth bound zmax;
    // `first` on the first of a bucket's lanes.  What is left to too few lanes is
    // flattened: below 12 where every lane has a bucket (visiting all buckets'
    // front points first is worth more than the idle lanes), below 24 where few
    // buckets are crowded (us, 12 / 24 / 32 / 44: K-NP of 1.5M points at 128x128
    // 192 / 102 / 115 / 147, 192x192 112 / 117 / 108 / 95, 257x257 163 / 154 / 153 /
    // 138; search at 128x128 111 / 107 / 111 / 140, 257x257 122 / 103 / 102 / 118).
    auto sweep_buckets = [&](int at, int end, float zmax, int share, bool first) {
        uint64_t go = ballot(at < end);
        const int few = share > 1 ? 24 : 12;
        while (popc64(go) >= few) {
            // (a lane without points left loads the table's first point)
            const float4 P = load_point(at < end ? at : 0);
            const uint64_t near = go & ballot(P.z <= __builtin_fminf(zmax, z_hi));
            test_points(near & ballot(P.z >= z_lo), P);
            // (points are ordered by depth: behind one too deep all are)
            at = in_mask(near) ? at + share : end;
            go = ballot(at < end);
        }
        // (a bucket's lanes step together, so what is left of it follows its
        // first lane's place)
        if (go) sweep_flat(at, first ? max(end - at, 0) : 0, true, zmax);
    };

    const int wx0 = max(gx0 - h, 0), wx1 = min(gx1 + h, Wg - 1);
    const int wy0 = max(gy - h, 0), wy1 = min(gy + h, Hg - 1);
    bool runs = false;
    if (h >= 0 && 2 * h + 1 <= ROW_WIN && c.layout != HP_LAYOUT_MORTON) {
        const bool tiled = c.layout != HP_LAYOUT_ROWMAJOR;
        const int ncol = tiled ? (wx1 >> 3) - (wx0 >> 3) + 1 : 1;  // at most 4
        const int row = ncol == 1 ? l : ncol == 2 ? l >> 1 : ncol == 3 ? (l * 171) >> 9 : l >> 2;
        const int col = l - row * ncol;
        const int dyi = row - h, by = gy + dyi;
        int st = 0, cnt = 0;
        if (row <= 2 * h && by >= 0 && by < Hg) {
            // half-width of the disc in this row (generous: bounds only)
            int hw = h;
            if (!square) {
                const float ey = __builtin_fmaxf(0.0f, (float)(dyi < 0 ? -dyi : dyi) - 0.5f);
                const float ex2 = Dmax * Dmax - ey * ey;
                hw = ex2 >= 0.0f ? min(h, (int)(__builtin_amdgcn_sqrtf(ex2) * 1.0001f + 0.501f)) : -1 - ng;
            }
            int x0 = max(gx0 - hw, 0), x1 = min(gx1 + hw, Wg - 1);
            if (tiled) {
                const int tx = ((wx0 >> 3) + col) << 3;
                x0 = max(x0, tx);
                x1 = min(x1, tx + 7);
            }
            if (x0 <= x1) {
                const int key = bucket_of(Vg, c.layout, x0, by);
                st = c.offsets[key];
                cnt = c.offsets[key + (x1 - x0) + 1] - st;
            }
        }
        const int totp = readlane_i32(wave_incl_scan_i32(cnt), WAVE - 1);
        runs = totp <= (BY_E2 ? ROW_POINTS_KNP : ROW_POINTS);
        if (runs) sweep_flat(st, cnt, false, 0.0f);
    }
    if (h >= 0 && !runs) {
        // depth bound of the window buckets at distance D from the rays' pixels
        auto zmax_at = [&](float D) -> float {
            // bounds only (margins of 1e-3 px and 0.1% dwarf 1-ulp approximations)
            const float Dp = D - 0.01f;
            const float zc = ((frL2 * __builtin_amdgcn_rcpf(Dp) + two_rw) * inv_L) * 1.001f + 1e-5f;
            return ((Dp > 0.0f) & (Dp > dinf) & (zc < z_hi)) ? zc : z_hi;
        };
        // distance of buckets x .. x + nx, y .. y + ny from the nearest of the rays' pixel centres
        auto distance = [&](int x, int y, int nx, int ny) -> float {
            const int ax = max(max(x - gx1, gx0 - (x + nx)), 0), ay = max(max(y - gy, gy - (y + ny)), 0);
            const float ex = __builtin_fmaxf(0.0f, (float)ax - 0.5f);
            const float ey = __builtin_fmaxf(0.0f, (float)ay - 0.5f);
            return __builtin_amdgcn_sqrtf(ex * ex + ey * ey);
        };
        // A cell whose nearest window bucket is at distance D is skipped when
        // its minimum depth exceeds the depth bound at D (the bound only
        // falls with D).  Surviving cells are listed (up to 64 at a time) with
        // the prefix of their window-bucket counts; each cell's buckets go to
        // one chunk of lanes, two cells per step so that their loads overlap.
        const int cx0 = wx0 >> CELL_SHIFT, cy0 = wy0 >> CELL_SHIFT;
        const int ncw = (wx1 >> CELL_SHIFT) - cx0 + 1;
        const int ncell = ncw * ((wy1 >> CELL_SHIFT) - cy0 + 1);
        int c0 = 0;                     // next cell to look at
        int k0 = 0, ncl = 0, total = 0;  // next listed cell, their number, their buckets
        int nbl = 0;                    // listed buckets
        for (;;) {
            while (nbl < WAVE) {
                if (k0 >= ncl) {
                    if (c0 >= ncell) break;
                    const int ci = min(c0 + l, ncell - 1);
                    const int cyy = cy0 + ci / ncw, cxx = cx0 + ci % ncw;
                    const int bx0 = max(cxx << CELL_SHIFT, wx0), by0 = max(cyy << CELL_SHIFT, wy0);
                    const int bx1 = min((cxx << CELL_SHIFT) + CELL - 1, wx1);
                    const int by1 = min((cyy << CELL_SHIFT) + CELL - 1, wy1);
                    const int bw = bx1 - bx0 + 1;
                    const float D = distance(bx0, by0, bx1 - bx0, by1 - by0);
                    const float cz = __uint_as_float(c.cell_zmin[cell_base + cyy * ncx + cxx]);
                    uint64_t km = ballot(c0 + l < ncell) & ballot(cz <= zmax_at(D));
                    if (!square) km &= ballot(D <= Dmax);
                    const int nk = in_mask(km) ? bw * (by1 - by0 + 1) : 0;
                    const int inc = wave_incl_scan_i32(nk);
                    total = readlane_i32(inc, WAVE - 1);
                    lds_sync();
                    if (in_mask(km))
                        sh.cl[rank_below(km)] = make_int2((bx0 - wx0) | ((by0 - wy0) << 16), bw | ((inc - nk) << 16));
                    lds_sync();
                    ncl = popc64(km);
                    k0 = 0;
                    c0 += WAVE;
                    continue;
                }
                // (every lane loads, those outside the window the view's first
                // bucket, so that the loads of both cells are in flight
                // together: behind a branch each waits for the one before)
                uint64_t in[2];
                int key[2], at[2], end[2], off[2];
                float zm[2], z0[2];
#pragma unroll
                for (int u = 0; u < 2; ++u) {
                    const int2 e = sh.cl[min(k0 + u, ncl - 1)];
                    const int next = sh.cl[min(k0 + u + 1, ncl - 1)].y >> 16;
                    const int nin = (k0 + u + 1 < ncl ? next : total) - (e.y >> 16);
                    const int bw = e.y & 0xffff;
                    const int ry = (int)(((float)l + 0.5f) * __builtin_amdgcn_rcpf((float)bw));
                    const int ox = (e.x & 0xffff) + (l - ry * bw), oy = (int)((uint32_t)e.x >> 16) + ry;
                    const float D = distance(wx0 + ox, wy0 + oy, 0, 0);
                    in[u] = k0 + u < ncl ? ballot(l < nin) : 0ull;
                    if (!square) in[u] &= ballot(D <= Dmax);
                    zm[u] = zmax_at(D);
                    off[u] = ox | (oy << 16);
                    key[u] = in_mask(in[u]) ? bucket_of(Vg, c.layout, wx0 + ox, wy0 + oy) : Vg.bucket_base;
                    at[u] = c.offsets[key[u]];
                    end[u] = c.offsets[key[u] + 1];
                    z0[u] = c.bucket_z[key[u]];
                }
                k0 += 2;
#pragma unroll
                for (int u = 0; u < 2; ++u) {
                    const uint64_t m = in[u] & ballot(end[u] > at[u]) & ballot(z0[u] <= zm[u]);
                    if (in_mask(m)) sh.bl[nbl + rank_below(m)] = make_int2(key[u], off[u]);
                    nbl += popc64(m);
                }
            }
            if (nbl == 0) break;
            // the last (up to) 64 of the list
            const int take = min(nbl, WAVE);
            nbl -= take;
            lds_sync();
            // each to as many lanes as there are for it (a bucket per lane at any
            // number of them left most lanes idle in the crowded windows of a
            // low resolution, 18 buckets of 70 to 400 points for four rays:
            // K-NP of 1.5M points at 257x257 336 us, 154 so, search 171 and 103)
            const int share = (int)(((float)WAVE + 0.5f) * __builtin_amdgcn_rcpf((float)take));
            const int own = (int)(((float)l + 0.5f) * __builtin_amdgcn_rcpf((float)share)), part = l - own * share;
            int at = 0, end = 0;
            float zmax = 0.0f;
            if (own < take) {
                const int2 e = sh.bl[nbl + own];
                at = c.offsets[e.x] + part;
                end = c.offsets[e.x + 1];
                zmax = zmax_at(distance(wx0 + (e.y & 0xffff), wy0 + (int)((uint32_t)e.y >> 16), 0, 0));
            }
            lds_sync();
            sweep_buckets(at, end, zmax, share, part == 0);
        }
    }
#pragma unroll
    for (int r = 0; r < G; ++r) {
        if (r >= ng) break;
        if (np[r] > most) (void)keep_smallest<HELD + WAVE>(sh.pend[s0 + r], np[r], want, most - want);
        if (l == 0) {
            slot[s0 + r].n = np[r];
            slot[s0 + r].count = count[r];
        }
    }
    lds_sync();
}

// Merge two ascending KT-lists and keep the KT smallest, ascending: the
// element-wise minimum of a and reversed b is a bitonic sequence holding the
// KT smallest, which half-cleaners then sort.
template <int KT>
__device__ __forceinline__ void merge_low(uint64_t (&a)[KT], const uint64_t (&b)[KT])
{
#pragma unroll
    for (int k = 0; k < KT; ++k) a[k] = kmin(a[k], b[KT - 1 - k]);
#pragma unroll
    for (int j = KT / 2; j > 0; j >>= 1) {
#pragma unroll
        for (int k = 0; k < KT; ++k) {
            if ((k & j) == 0) kswap(a[k], a[k + j]);
        }
    }
}

// Ascending sort of eight keys on the 19-comparator network for n = 8.
__device__ __forceinline__ void sort8(uint64_t (&x)[8])
{
    kswap(x[0], x[2]); kswap(x[1], x[3]); kswap(x[4], x[6]); kswap(x[5], x[7]);
    kswap(x[0], x[4]); kswap(x[1], x[5]); kswap(x[2], x[6]); kswap(x[3], x[7]);
    kswap(x[0], x[1]); kswap(x[2], x[3]); kswap(x[4], x[5]); kswap(x[6], x[7]);
    kswap(x[2], x[4]); kswap(x[3], x[5]);
    kswap(x[1], x[4]); kswap(x[3], x[6]);
    kswap(x[1], x[2]); kswap(x[3], x[4]); kswap(x[5], x[6]);
}

// Quad-split nearest neighbours of the ray point at tq among the sorted-list
// entries [lo, hi) within R2: lane q of each quad takes entries lo + q,
// lo + q + 4, ... into an ascending register list of (dist^2 bits << 32 |
// index); the quad then merges its four lists (DPP within the quad).
template <int KT>
__device__ __forceinline__ void knn_window(const RayGeom &g, const SlabList &sh, float tq, float R2,
                                           int lo, int hi, uint64_t (&kd)[KT])
{
    const int q = lane_id() & 3;
#pragma unroll
    for (int k = 0; k < KT; ++k) kd[k] = KEY_NONE;
    int n_it = (hi - lo - q + 3) >> 2;
    n_it = n_it > 0 ? n_it : 0;
    n_it = max(n_it, (int)xor_lane_u32<4>((uint32_t)n_it));
    n_it = max(n_it, (int)xor_lane_u32<8>((uint32_t)n_it));
    n_it = max(n_it, (int)xor_lane_u32<16>((uint32_t)n_it));
    n_it = max(n_it, (int)xor_lane_u32<32>((uint32_t)n_it));
    // (n_it is now the maximum over the lanes with this lane's q; the
    // quad-gather path below reads the other lanes of the quad, so all lanes
    // must take it together: its test uses the maximum over the whole wave)
    int n_all = max(n_it, (int)xor_lane_u32<1>((uint32_t)n_it));
    n_all = max(n_all, (int)xor_lane_u32<2>((uint32_t)n_all));
    if constexpr (KT >= 8) {
        if (n_all <= 2) {
            // at most two entries per lane: the quad's union fits eight; sort
            // each lane's pair, gather the quad's four pairs on every lane and
            // merge the sorted runs 2 -> 4 -> 8
            uint64_t x[2];
#pragma unroll
            for (int e = 0; e < 2; ++e) {
                const int i = lo + q + 4 * e;
                x[e] = KEY_NONE;
                if (e < n_it && i < hi) {
                    const float4 P = sh.nb_p[i];
                    const float d2 = dist2_at(P.x, P.y, P.z, g.dx, g.dy, g.dz, tq);
                    if (d2 <= R2) x[e] = ((uint64_t)__float_as_uint(d2) << 32) | __float_as_uint(P.w);
                }
            }
            kswap(x[0], x[1]);
            uint64_t v[8];
#pragma unroll
            for (int p = 0; p < 4; ++p) {
                v[2 * p] = quad_bcast_u64(x[0], p);
                v[2 * p + 1] = quad_bcast_u64(x[1], p);
            }
            // (each merge reverses its second run, making the pair of runs
            // bitonic, then half-cleaners sort it)
#pragma unroll
            for (int r0 = 0; r0 < 8; r0 += 4) {
                uint64_t *w = v + r0;
                const uint64_t t = w[2];
                w[2] = w[3];
                w[3] = t;
                kswap(w[0], w[2]);
                kswap(w[1], w[3]);
                kswap(w[0], w[1]);
                kswap(w[2], w[3]);
            }
#pragma unroll
            for (int k = 0; k < 2; ++k) {
                const uint64_t t = v[4 + k];
                v[4 + k] = v[7 - k];
                v[7 - k] = t;
            }
#pragma unroll
            for (int j = 4; j > 0; j >>= 1)
#pragma unroll
                for (int k = 0; k < 8; ++k)
                    if ((k & j) == 0) kswap(v[k], v[k + j]);
#pragma unroll
            for (int k = 0; k < KT; ++k) kd[k] = k < 8 ? v[k < 8 ? k : 0] : KEY_NONE;
            return;
        }
    }
    if constexpr (KT >= 16) {
        if (n_all <= 4) {
            // every lane holds at most four entries, so the quad's union fits
            // sixteen: sort each lane's four, gather the quad's sixteen keys
            // on every lane and merge the four sorted runs (no list merges)
            uint64_t x[4];
#pragma unroll
            for (int e = 0; e < 4; ++e) {
                const int i = lo + q + 4 * e;
                x[e] = KEY_NONE;
                if (e < n_it && i < hi) {
                    const float4 P = sh.nb_p[i];
                    const float d2 = dist2_at(P.x, P.y, P.z, g.dx, g.dy, g.dz, tq);
                    if (d2 <= R2) x[e] = ((uint64_t)__float_as_uint(d2) << 32) | __float_as_uint(P.w);
                }
            }
            kswap(x[0], x[1]);
            kswap(x[2], x[3]);
            kswap(x[0], x[2]);
            kswap(x[1], x[3]);
            kswap(x[1], x[2]);
            uint64_t v[16];
#pragma unroll
            for (int p = 0; p < 4; ++p)
#pragma unroll
                for (int e = 0; e < 4; ++e) v[4 * p + e] = quad_bcast_u64(x[e], p);
            // runs of 4 -> 8 -> 16: the second run reversed makes a bitonic
            // sequence, which half-cleaners sort
#pragma unroll
            for (int r0 = 0; r0 < 16; r0 += 8) {
                uint64_t *w = v + r0;
#pragma unroll
                for (int k = 0; k < 2; ++k) {
                    const uint64_t t = w[4 + k];
                    w[4 + k] = w[7 - k];
                    w[7 - k] = t;
                }
#pragma unroll
                for (int j = 4; j > 0; j >>= 1)
#pragma unroll
                    for (int k = 0; k < 8; ++k)
                        if ((k & j) == 0) kswap(w[k], w[k + j]);
            }
#pragma unroll
            for (int k = 0; k < 4; ++k) {
                const uint64_t t = v[8 + k];
                v[8 + k] = v[15 - k];
                v[15 - k] = t;
            }
#pragma unroll
            for (int j = 8; j > 0; j >>= 1)
#pragma unroll
                for (int k = 0; k < 16; ++k)
                    if ((k & j) == 0) kswap(v[k], v[k + j]);
#pragma unroll
            for (int k = 0; k < KT; ++k) kd[k] = k < 16 ? v[k < 16 ? k : 0] : KEY_NONE;
            return;
        }
    }
    // longer windows: the first eight entries are sorted outright (19
    // compare-exchanges) and their smallest KT are the list (the test is
    // wave-uniform: n_all is the maximum over the wave)
    int it0 = 0;
    if (n_all > 4) {
        it0 = 8;
        uint64_t x[8];
#pragma unroll
        for (int e = 0; e < 8; ++e) {
            const int i = lo + q + 4 * e;
            x[e] = KEY_NONE;
            if (e < n_it && i < hi) {
                const float4 P = sh.nb_p[i];
                const float d2 = dist2_at(P.x, P.y, P.z, g.dx, g.dy, g.dz, tq);
                if (d2 <= R2) x[e] = ((uint64_t)__float_as_uint(d2) << 32) | __float_as_uint(P.w);
            }
        }
        sort8(x);
#pragma unroll
        for (int k = 0; k < KT && k < 8; ++k) kd[k] = x[k];
    }
    // later entries four at a time: sort the four keys (five
    // compare-exchanges), then merge them into the list as the upper half of
    // a bitonic sequence
    for (int it = it0; it < n_it; it += 4) {
        uint64_t x[4];
#pragma unroll
        for (int e = 0; e < 4; ++e) {
            const int i = lo + q + 4 * (it + e);
            x[e] = KEY_NONE;
            if (i < hi) {
                const float4 P = sh.nb_p[i];
                const float d2 = dist2_at(P.x, P.y, P.z, g.dx, g.dy, g.dz, tq);
                if (d2 <= R2) x[e] = ((uint64_t)__float_as_uint(d2) << 32) | __float_as_uint(P.w);
            }
        }
        kswap(x[0], x[1]);
        kswap(x[2], x[3]);
        kswap(x[0], x[2]);
        kswap(x[1], x[3]);
        kswap(x[1], x[2]);
        static_assert(KT >= 4, "lists of at least four");
#pragma unroll
        for (int e = 0; e < 4; ++e) kd[KT - 4 + e] = kmin(kd[KT - 4 + e], x[3 - e]);
        // kd is now bitonic and holds the KT smallest: half-cleaners sort it
#pragma unroll
        for (int j = KT / 2; j > 0; j >>= 1) {
#pragma unroll
            for (int k = 0; k < KT; ++k)
                if ((k & j) == 0) kswap(kd[k], kd[k + j]);
        }
    }
    uint64_t other[KT];
#pragma unroll
    for (int k = 0; k < KT; ++k) other[k] = xor_lane_u64<1>(kd[k]);
    merge_low<KT>(kd, other);
#pragma unroll
    for (int k = 0; k < KT; ++k) other[k] = xor_lane_u64<2>(kd[k]);
    merge_low<KT>(kd, other);
}

// Distances of a quad's list entries split over its lanes: lane q takes the
// correctly rounded square roots of entries k = q, q + 4, ... (dq[e] for
// k = 4 e + q), so no lane computes more than KT / 4 of them.  Lane-local
// (every lane of a quad holds the same list).
template <int KT>
__device__ __forceinline__ uint64_t quad_entry(const uint64_t (&kd)[KT], int e)
{
    const int q = lane_id() & 3;
    uint64_t k0 = kd[4 * e], k1 = kd[4 * e + 1], k2 = kd[4 * e + 2], k3 = kd[4 * e + 3];
    // (an empty asm hides where the values came from: a select between
    // list elements would otherwise become a variable index into the list,
    // which then lives in scratch memory instead of registers)
    asm("" : "+v"(k0), "+v"(k1), "+v"(k2), "+v"(k3));
    return (q & 2) ? ((q & 1) ? k3 : k2) : ((q & 1) ? k1 : k0);
}

template <int KT>
__device__ __forceinline__ void quad_list_sqrt(const uint64_t (&kd)[KT], float (&dq)[KT / 4])
{
#pragma unroll
    for (int e = 0; e < KT / 4; ++e)
        dq[e] = __builtin_sqrtf(__uint_as_float((uint32_t)(quad_entry<KT>(kd, e) >> 32)));
}

// Sort of 16 R keys per row of 16 lanes, R per lane (key e of lane k is element
// R k + e when it returns): bitonic merges in the form that compares with the
// mirrored element first, so that every exchange leaves the smaller key at
// the lower element and no block descends.  Four rays' 64 keys each sort at
// once for little more than a wave takes to sort 64 keys one per lane.
template <int CTRL>
__device__ __forceinline__ uint64_t dpp_u64(uint64_t v)
{
    const uint32_t a = (uint32_t)__builtin_amdgcn_mov_dpp((int)(uint32_t)v, CTRL, 0xF, 0xF, false);
    const uint32_t b = (uint32_t)__builtin_amdgcn_mov_dpp((int)(uint32_t)(v >> 32), CTRL, 0xF, 0xF, false);
    return ((uint64_t)b << 32) | a;
}

// lane patterns of the exchanges: the lane's neighbour at distance 1, 2, and
// the mirror of its block of 4, 8 and 16 lanes, and the neighbour at distance 8
constexpr int DPP_XOR1 = 0xB1, DPP_XOR2 = 0x4E, DPP_REV4 = 0x1B, DPP_REV8 = 0x141, DPP_REV16 = 0x140, DPP_ROR8 = 0x128;

// One exchange between lanes: the smaller key of each pair on the lanes whose
// index bit BIT is clear, the larger on the others.  MIRROR pairs element e
// with the partner lane's element R - 1 - e.
template <int R, int BIT, int CTRL, bool MIRROR, int CTRL2 = 0>
__device__ __forceinline__ void row_exchange(uint64_t (&x)[R])
{
    uint64_t o[R];
#pragma unroll
    for (int e = 0; e < R; ++e) {
        o[e] = dpp_u64<CTRL>(x[MIRROR ? R - 1 - e : e]);
        if constexpr (CTRL2 != 0) o[e] = dpp_u64<CTRL2>(o[e]);
    }
#pragma unroll
    for (int e = 0; e < R; ++e) {
        const bool take = (key_f64(o[e]) < key_f64(x[e])) != lanes_in<lane_bit_mask(BIT)>();
        x[e] = take ? o[e] : x[e];
    }
}

// half-cleaners inside every lane
template <int R>
__device__ __forceinline__ void lane_merge(uint64_t (&x)[R])
{
#pragma unroll
    for (int h = R / 2; h > 0; h >>= 1)
#pragma unroll
        for (int e = 0; e < R; ++e)
            if ((e & h) == 0) kswap(x[e], x[e + h]);
}

template <int R>
__device__ __forceinline__ void row_sort(uint64_t (&x)[R])
{
    static_assert(R == 2 || R == 4 || R == 8, "two, four or eight keys per lane");
    if constexpr (R == 8) {
        sort8(x);
    } else if constexpr (R == 2) {
        kswap(x[0], x[1]);
    } else {
        kswap(x[0], x[1]);
        kswap(x[2], x[3]);
        kswap(x[0], x[2]);
        kswap(x[1], x[3]);
        kswap(x[1], x[2]);
    }
    // blocks of 2, 4, 8, 16 lanes
    row_exchange<R, 0, DPP_XOR1, true>(x);
    lane_merge(x);
    row_exchange<R, 1, DPP_REV4, true>(x);
    row_exchange<R, 0, DPP_XOR1, false>(x);
    lane_merge(x);
    row_exchange<R, 2, DPP_REV8, true>(x);
    row_exchange<R, 1, DPP_XOR2, false>(x);
    row_exchange<R, 0, DPP_XOR1, false>(x);
    lane_merge(x);
    row_exchange<R, 3, DPP_REV16, true>(x);
    // (lanes 4 apart: the mirror of 8 lanes, its halves mirrored back)
    row_exchange<R, 2, DPP_REV8, false, DPP_REV4>(x);
    row_exchange<R, 1, DPP_XOR2, false>(x);
    row_exchange<R, 0, DPP_XOR1, false>(x);
    lane_merge(x);
}

// Exchanges between lanes of different rows.
template <int R, int BIT, bool MIRROR>
__device__ __forceinline__ void wave_exchange(uint64_t (&x)[R], int xor_lane)
{
    uint64_t o[R];
#pragma unroll
    for (int e = 0; e < R; ++e) {
        const uint64_t v = x[MIRROR ? R - 1 - e : e];
        const uint32_t a = (uint32_t)__shfl_xor((int)(uint32_t)v, xor_lane, WAVE);
        const uint32_t b = (uint32_t)__shfl_xor((int)(uint32_t)(v >> 32), xor_lane, WAVE);
        o[e] = ((uint64_t)b << 32) | a;
    }
#pragma unroll
    for (int e = 0; e < R; ++e) {
        const bool take = (key_f64(o[e]) < key_f64(x[e])) != lanes_in<lane_bit_mask(BIT)>();
        x[e] = take ? o[e] : x[e];
    }
}

// Sort of 64 R keys across the wave (key e of lane l is element R l + e when
// it returns): the rows, then blocks of two and of four rows.
template <int R>
__device__ __forceinline__ void wave_sort_many(uint64_t (&x)[R])
{
    row_sort(x);
    wave_exchange<R, 4, true>(x, 31);
    row_exchange<R, 3, DPP_ROR8, false>(x);
    row_exchange<R, 2, DPP_REV8, false, DPP_REV4>(x);
    row_exchange<R, 1, DPP_XOR2, false>(x);
    row_exchange<R, 0, DPP_XOR1, false>(x);
    lane_merge(x);
    wave_exchange<R, 5, true>(x, 63);
    wave_exchange<R, 4, false>(x, 16);
    row_exchange<R, 3, DPP_ROR8, false>(x);
    row_exchange<R, 2, DPP_REV8, false, DPP_REV4>(x);
    row_exchange<R, 1, DPP_XOR2, false>(x);
    row_exchange<R, 0, DPP_XOR1, false>(x);
    lane_merge(x);
}

// Keys 4 k .. 4 k + 3 of the ascending list of the row's ray (KEY_NONE = none)
// on lane k of each row of 16 lanes, from the row of `pend` that holds `held`
// <= 128 keys in no order (which may be overwritten); `most`: the largest
// number held by a row.
__device__ __forceinline__ void row_sorted_keys(uint64_t *pend, int held, int most, uint64_t (&key)[4])
{
    const int k16 = phase_lane_id() & 15;
    if (most <= WAVE) {
#pragma unroll
        for (int e = 0; e < 4; ++e) key[e] = 16 * e + k16 < held ? pend[16 * e + k16] : KEY_NONE;
        row_sort(key);
        return;
    }
    uint64_t x[8];
#pragma unroll
    for (int e = 0; e < 8; ++e) x[e] = 16 * e + k16 < held ? pend[16 * e + k16] : KEY_NONE;
    row_sort(x);
    lds_sync();
    if (k16 < 8) {
#pragma unroll
        for (int e = 0; e < 8; ++e) pend[8 * k16 + e] = x[e];
    }
    lds_sync();
#pragma unroll
    for (int e = 0; e < 4; ++e) key[e] = pend[4 * k16 + e];
}

// Candidate walk of up to four rays at once, one row of 16 lanes each: lane
// 16 r + k serves candidate c0 + k of ray r (the neighbours in (t, index)
// order, 16 at a time).  One lane per candidate rather than four: the search
// kernels are bound by vector instructions, and the sorting networks, square
// roots and the transmittance products below cost a wave the same whether its
// lanes serve one ray or four.
//
// Nearest neighbours.  A lane takes the list in batches of eight consecutive
// entries, first those around its candidate, then on the side whose next
// entry is nearer in t, until both next entries lie further than R_j or than
// its KT-th distance so far (distance >= |t_i - t_j| up to rounding); each
// batch is sorted (19 compare-exchanges) and merged into the lane's ascending
// list of (dist^2 bits << 32 | index).
//
// Transmittance (Eq. 5).  The value in front of each candidate is the running
// product of (1 - alpha) in candidate order, one binary32 multiply after
// another as a sequential walk takes them: fifteen steps in which every lane
// takes its left neighbour's value times that neighbour's factor, the row's
// first lane keeping the value carried from the previous sixteen.  A lane's
// value is final once its left neighbour's is.
//
// The rays are those of the first ns slots, their keys in sh.pend; lists(ray,
// i, m, count, key) is called on every lane of theirs with entries i .. i + 3
// of the ray's list of m neighbours.
//
// emit(ray, s, tj, kd, dist, kc) is called on the lane of every candidate that
// became sample s, with its nearest neighbours kd (ascending, an empty slot's
// upper half is KEY_NONE's), their distances and their number kc among the
// first K; first(ray, index) on the lane of a ray's first sample, and
// ends(ray, n) on a ray's first lane with its sample count.
template <int KT, typename Lds, typename Lists, typename Emit, typename First, typename Ends>
__device__ __forceinline__ void walk_batch(Lds &sh, int ns, Lists lists, Emit emit, First first, Ends ends)
{
    const SearchCtx c = phase_ctx();
    const int l = phase_lane_id(), r = l >> 4, k16 = l & 15;
    const bool live = r < ns;
    const RaySlot me = sh.slot[live ? r : 0];
    const int held = live ? me.n : 0, m = min(held, c.M), ray = me.ray;
    RayGeom g;
    {
        const RayGeom &gr = sh.rs[me.rs];
        g.dx = gr.dx;
        g.dy = gr.dy;
        g.dz = gr.dz;
        g.kappa = gr.kappa;
        g.vi = gr.vi;
    }
    float4 *const nb = sh.lists().p;
    const float nan = __builtin_nanf("");
    {
        uint64_t key[4];
        int most = held;
        most = max(most, __shfl_xor(most, 16, WAVE));
        most = uniform_i32(max(most, __shfl_xor(most, 32, WAVE)));
        row_sorted_keys(sh.search().pend[r], held, most, key);
        if (live) lists(ray, 4 * k16, m, me.count, key);
        float4 P[4];
#pragma unroll
        for (int e = 0; e < 4; ++e) {
            P[e] = make_float4(nan, nan, nan, 0.0f);
            if (4 * k16 + e < m) P[e] = c.pcam[(int64_t)g.vi * c.n_points + (int)(uint32_t)key[e]];
        }
        lds_sync();
#pragma unroll
        for (int e = 0; e < 4; ++e) nb[WALK_PAD + WALK_STRIDE * r + 4 * k16 + e] = P[e];
        if (l < WALK_PAD * (GROUP + 1))
            nb[WALK_STRIDE * (l / WALK_PAD) + l % WALK_PAD] = make_float4(nan, nan, nan, 0.0f);
    }
    lds_sync();
    const float4 *const row = nb + WALK_PAD + WALK_STRIDE * r;
    auto t_at = [&](int i) {
        const float4 P = row[i];
        return ray_param(P.x, P.y, P.z, g.dx, g.dy, g.dz);
    };
    float T = 1.0f;
    int sel = 0;
    bool done = m == 0;
    for (int c0 = 0;; c0 += 16) {
        const int j = c0 + k16;
        const bool active = !done && j < m;
        if (!ballot(active)) break;
        uint64_t kd[KT];
#pragma unroll
        for (int k = 0; k < KT; ++k) kd[k] = KEY_NONE;
        float alpha = 0.0f, tj = 0.0f, dist[KT];
        int kc = 0;
        if (active) {
            tj = t_at(j);
            const float Rj = rho_at(c, g, tj);
            const float R2 = Rj * Rj;
            const float slack = (tj + Rj) * 4e-6f + 1e-7f;
            auto take8 = [&](int base, uint64_t(&x)[8]) {
#pragma unroll
                for (int e = 0; e < 8; ++e) {
                    if (e == 4) asm volatile("" ::: "memory");
                    const float4 P = row[base + e];
                    const float d2 = dist2_at(P.x, P.y, P.z, g.dx, g.dy, g.dz, tj);
                    const uint32_t hi = d2 <= R2 ? __float_as_uint(d2) : (uint32_t)(KEY_NONE >> 32);
                    x[e] = ((uint64_t)hi << 32) | __float_as_uint(P.w);
                }
                sort8(x);
            };
            int lo = max(j - 4, 0), hi = lo + 8;
            {
                uint64_t x[8];
                take8(lo, x);
#pragma unroll
                for (int k = 0; k < KT && k < 8; ++k) kd[k] = x[k];
            }
            for (;;) {
                // (a missing entry's t is NaN: neither comparison holds; an
                // unfilled list's last distance is NaN and the minimum R_j)
                const float dk = __uint_as_float((uint32_t)(kd[KT - 1] >> 32));
                const float reach = __builtin_fminf(Rj, __builtin_amdgcn_sqrtf(dk)) * 1.001f + slack;
                const float du = t_at(hi) - tj, dd = tj - t_at(lo - 1);
                const bool up = du <= reach, dn = dd <= reach;
                if (!(up | dn)) break;
                const bool go_up = up && (!dn || du <= dd);
                const int base = go_up ? hi : lo - 8;
                uint64_t x[8];
                take8(base, x);
                hi = go_up ? hi + 8 : hi;
                lo = go_up ? lo : lo - 8;
                if constexpr (KT <= 8) {
#pragma unroll
                    for (int k = 0; k < KT; ++k) kd[k] = kmin(kd[k], x[KT - 1 - k]);
                } else {
#pragma unroll
                    for (int e = 0; e < 8; ++e) kd[KT - 8 + e] = kmin(kd[KT - 8 + e], x[7 - e]);
                }
                // kd is bitonic and holds the KT smallest: half-cleaners sort it
#pragma unroll
                for (int h = KT / 2; h > 0; h >>= 1) {
#pragma unroll
                    for (int k = 0; k < KT; ++k)
                        if ((k & h) == 0) kswap(kd[k], kd[k + h]);
                }
            }
            // the list's valid entries form a prefix; the first K count
            float sum = 0.0f;  // (adding +0 past the prefix leaves it unchanged)
#pragma unroll
            for (int k = 0; k < KT; ++k) {
                const uint32_t hi32 = (uint32_t)(kd[k] >> 32);
                const bool v = hi32 != (uint32_t)(KEY_NONE >> 32) && k < c.K;
                dist[k] = v ? __builtin_sqrtf(__uint_as_float(hi32)) : 0.0f;
                kc += v ? 1 : 0;
                sum = sum + dist[k];
            }
            const float dj = (sum + (float)(c.K - kc) * Rj) / (float)c.K;
            const float uj = (dj * dj) * c.inv_beta2;
            alpha = c.gamma * exp_neg(-uj);
        }
        // (candidates past the list have alpha = 0, a factor of exactly 1)
        const float f = 1.0f - alpha;
        const float fs = __int_as_float(__builtin_amdgcn_update_dpp(
            0x3f800000, __float_as_int(f), 0x111, 0xF, 0xF, false));  // left neighbour's, 1 on first lanes
        float Tb = T;
#pragma unroll
        for (int k = 0; k < 15; ++k) {
            const int left = __builtin_amdgcn_update_dpp(__float_as_int(Tb), __float_as_int(Tb), 0x111, 0xF, 0xF, false);
            Tb = __int_as_float(left) * fs;
        }
        const float Ta = Tb * f;
        // the sequential walk's decisions: a candidate is visited if no
        // earlier one left gamma T <= eps_w behind it and fewer than S
        // samples were taken before it, and selected if its weight passes
        const uint64_t am = ballot(active);
        const uint64_t pm = am & ballot(alpha * Tb > c.eps_w);
        const uint64_t dm = am & ballot(c.gamma * Ta <= c.eps_w);
        const uint32_t prow = (uint32_t)(pm >> (16 * r)) & 0xffffu;
        const uint32_t drow = (uint32_t)(dm >> (16 * r)) & 0xffffu;
        const uint32_t below = (1u << k16) - 1u;
        const int rank = sel + __popc(prow & below);
        const bool mine = ((prow >> k16) & 1u) != 0 && (drow & below) == 0 && rank < c.S;
        if (mine) {
            if (rank == 0) first(ray, __float_as_int(row[j].w));
            emit(ray, rank, tj, kd, dist, kc);
        }
        // the row's totals on all of its lanes
        const uint64_t sm = ballot(mine);
        sel += __popc((uint32_t)(sm >> (16 * r)) & 0xffffu);
        done = done || drow != 0 || sel >= c.S || c0 + 16 >= m;
        // the last lane's value behind it is carried to the whole row
        T = __int_as_float(__shfl(__float_as_int(Ta), l | 15, WAVE));
    }
    if (live && k16 == 0) ends(ray, sel);
    lds_sync();
}

// A ray's neighbours in depth order, 64 at a time.  Where the search held all
// of them (up to HELD_SLAB), they are sorted once and a slab is a range of
// that list; else the ray is searched again for each slab, with the slab's
// bound as a filter.
struct SlabKeys {
    uint64_t keys;  // the current slab, one key per lane, ascending (n of them)
    int n;
    int rest;       // neighbours at or above the slab's first key (any number above n where there are more)
    int held;       // keys in the sorted list, -1: not all neighbours are held
};

__device__ __forceinline__ void slab_from(SlabLds &lds, SlabKeys &k, uint64_t from)
{
    const int l = phase_lane_id();
    lds_sync();
    if (k.held >= 0) {
        int at = 0;
#pragma unroll
        for (int e = 0; e < HELD_SLAB / WAVE; ++e)
            at += popc64(ballot(WAVE * e + l < k.held) & ballot(lds.s.pend[0][WAVE * e + l] < from));
        k.rest = k.held - at;
        k.n = min(k.rest, WAVE);
        k.keys = l < k.n ? lds.s.pend[0][at + l] : ~0ull;
        return;
    }
    search_group<1, HELD_SLAB>(lds.rs, lds.slot, lds.s, 0, 1, WAVE, WAVE, from);
    k.rest = uniform_i32(lds.slot[0].count);
    k.n = min(k.rest, WAVE);
    k.keys = wave_sort_fast(l < k.n ? lds.s.pend[0][l] : ~0ull);
}

// The first slab of the ray in slot 0 (its record: rec).
__device__ __forceinline__ void first_slab(SlabLds &lds, SlabKeys &k, int rec)
{
    const int l = phase_lane_id();
    lds_sync();
    if (l == 0) lds.slot[0].rs = rec;
    lds_sync();
    search_group<1, HELD_SLAB>(lds.rs, lds.slot, lds.s, 0, 1, WAVE, HELD_SLAB);
    k.rest = uniform_i32(lds.slot[0].count);
    const int held = uniform_i32(lds.slot[0].n);
    k.held = held == k.rest ? held : -1;
    k.n = min(k.rest, WAVE);
    if (held <= WAVE) {
        k.keys = wave_sort_fast(l < held ? lds.s.pend[0][l] : ~0ull);
        lds.s.pend[0][l] = k.keys;
        lds_sync();
        return;
    }
    constexpr int R = HELD_SLAB / WAVE + 1;
    static_assert(R == 8, "the keys held and their room for 64 more are sorted together");
    uint64_t x[R];
#pragma unroll
    for (int e = 0; e < R; ++e) x[e] = WAVE * e + l < held ? lds.s.pend[0][WAVE * e + l] : KEY_NONE;
    wave_sort_many(x);
    lds_sync();
#pragma unroll
    for (int e = 0; e < R; ++e) lds.s.pend[0][R * l + e] = x[e];
    lds_sync();
    k.keys = lds.s.pend[0][l];
}

// Uniform multi-surface sampling (the baseline of Sec. 3.5): positions
// t_k = t_near + (k + 1/2) step, k < ms_steps, each with a radius search: a
// position is a sample when some neighbour of the ray (any of them, not only
// the first m_cap) lies within R_k = rho(t_k) of it (the exact test), in
// depth order up to S, with its K nearest such neighbours.  The neighbours
// are walked in depth order 64 at a time (SlabKeys, the first slab as
// first_slab left it), their points in the LDS.
// Positions go 16 at a time, one per quad (lanes 4 g .. 4 g + 3), each
// keeping its K nearest over the slabs that reach its window |t - t_k| <= R_k
// (distance >= |t_i - t_k| up to rounding); a batch starts from the slab of
// keys at or above its first window and jumps over positions that no
// neighbour can reach.  emit(s, q, tj, kd, dq, kc) is called on the four lanes
// (q = 0..3) of every position that became sample s, with its nearest
// neighbours kd (ascending, KEY_NONE = none), the lane's share dq of their
// distances (quad_list_sqrt) and their number kc; first_idx is the nearest
// point of the first sample.
template <int KT, typename Emit>
__device__ __forceinline__ int uniform_samples(const RayGeom &g, SlabLds &lds, SlabKeys &slab, int &first_idx,
                                               Emit emit)
{
    const SearchCtx c = phase_ctx();
    const int l = lane_id();
    SlabList &sh = lds.s.slab;
    first_idx = -1;
    if (slab.rest == 0) return 0;
    const int nk = c.ms_steps;
    const float step = (c.t_far - c.t_near) / (float)nk;
    auto pos_t = [&](int k) { return fma_rn((float)k + 0.5f, step, c.t_near); };
    // |t_i - t_k| > span implies dist^2 > R_k^2 (margins above rounding)
    auto pos_span = [&](float tk) { return rho_at(c, g, tk) * 1.001f + tk * 4e-6f + 1e-7f; };
    // every window ends within smax of its position (rho grows with t)
    const float smax = pos_span(c.t_far);
    // a position before this one cannot reach a key at t (one spare)
    auto first_reaching = [&](float t) -> int {
        float f = (t - smax - c.t_near) / step - 0.5f;
        f = __builtin_fminf(__builtin_fmaxf(f, -2.0f), (float)nk + 2.0f);
        return max((int)__builtin_floorf(f) - 1, 0);
    };
    uint64_t &keys = slab.keys;
    int &n = slab.n, &rest = slab.rest;
    auto load_slab = [&]() {
        lds_sync();
        if (l < n) {
            const int idxj = (int)(uint32_t)keys;
            sh.nb_p[l] = c.pcam[(int64_t)g.vi * c.n_points + idxj];
            sh.nb_t[l] = __uint_as_float((uint32_t)(keys >> 32));
        }
        lds_sync();
    };
    // first slab entry with t >= tlo (n if none)
    auto slab_lower = [&](float tlo) {
        int a = 0, e = n;
        while (a < e) {
            const int mid = (a + e) >> 1;
            if (sh.nb_t[mid] < tlo) a = mid + 1;
            else e = mid;
        }
        return a;
    };
    load_slab();
    int sel = 0;
    const int gp = l >> 2;
    int b = first_reaching(sh.nb_t[0]);
    while (b < nk && sel < c.S) {
        const int k = b + gp;
        const bool active = k < nk;
        float tk = 0.0f, R2 = 0.0f, span = 0.0f;
        if (active) {
            tk = pos_t(k);
            const float Rk = rho_at(c, g, tk);
            R2 = Rk * Rk;
            span = pos_span(tk);
        }
        const float tl = pos_t(min(b + 15, nk - 1));
        const float t_end = tl + pos_span(tl);  // where the batch's last window ends
        uint64_t kd[KT];
#pragma unroll
        for (int q = 0; q < KT; ++q) kd[q] = KEY_NONE;
        for (;;) {
            int wlo = 0, whi = 0;
            if (active) {
                wlo = slab_lower(tk - span);
                whi = wlo;
                int e = n;  // first entry with t > tk + span
                while (whi < e) {
                    const int mid = (whi + e) >> 1;
                    if (sh.nb_t[mid] <= tk + span) whi = mid + 1;
                    else e = mid;
                }
            }
            uint64_t part[KT];
            knn_window<KT>(g, sh, tk, R2, wlo, whi, part);
            merge_low<KT>(kd, part);
            // the next slab, unless this one held every remaining key or
            // ends beyond the last window of the batch
            if (rest <= n || sh.nb_t[n - 1] > t_end) break;
            const uint64_t last = readlane_u64(keys, n - 1);
            slab_from(lds, slab, last + 1ull);
            load_slab();
        }
        const bool kept = active && kd[0] != KEY_NONE;
        const uint64_t km = ballot(kept && (l & 3) == 0);  // bit 4 p: position b + p kept
        const int room = c.S - sel;
        const int rank = popc64(km & ((1ull << (4 * gp)) - 1ull));
        if (km) {
            if (sel == 0) first_idx = readlane_i32((int)(uint32_t)kd[0], __builtin_ctzll(km));
            if (kept && rank < room) {
                int kc = 0;
#pragma unroll
                for (int q = 0; q < KT; ++q) kc += (q < c.K && kd[q] != KEY_NONE) ? 1 : 0;
                float dq[KT / 4];
                quad_list_sqrt<KT>(kd, dq);
                emit(sel + rank, l & 3, tk, kd, dq, kc);
            }
            const int nkept = popc64(km);
            sel += nkept < room ? nkept : room;
        }
        // the next batch starts from the keys at or above its first window
        b += 16;
        if (b >= nk || sel >= c.S) break;
        const float tb = pos_t(b);
        const float tlo = tb - pos_span(tb);
        if (!(sh.nb_t[0] <= tlo && rest <= n)) {
            // (the current slab does not hold every key from tlo on)
            const uint64_t lo_key = tlo > 0.0f ? ((uint64_t)__float_as_uint(tlo) << 32) : 0ull;
            slab_from(lds, slab, lo_key);
            if (rest == 0) break;
            load_slab();
        }
        const int j = slab_lower(tlo);
        if (j >= n) break;  // no key at or beyond the next window
        b = max(b, first_reaching(sh.nb_t[j]));
    }
    return sel;
}

}  // namespace hp
