// Gradient of the render (Sec. 3.4, Eq. 2) with respect to the point
// features and the decoder parameters, given the samples of every ray.
//
// The samples depend on geometry only, so the caller either keeps the
// forward pass's samples or recomputes them with the forward search kernel
// (hp_render_backward does the latter into its workspace).  This kernel then
// mirrors the render: a wave takes some consecutive rays at a time and packs
// their samples, up to 64 of them, densely into tiles of 16.
//   pass A   inverse-distance aggregation and decoder (BF16 or FP32 on MFMA)
//            -> raw decoder outputs of every sample, kept in LDS;
//   composite backward (Eq. 2), one lane per ray, FP32: the transmittance in
//            front of each sample forward, then the suffix sums of colour and
//            transmittance backward -> dL/d(decoder outputs), in place;
//   pass B   per tile: the decoder is replayed keeping its activations, the
//            gradient flows back through it on FP32 matrix cores to the
//            aggregated features, and through the aggregation to the point
//            features with atomics.
// With the BF16 decoder every rounding of a decoder operand (weights,
// aggregated feature, hidden activations) counts as adding a fixed offset:
// the backward products use the rounded operands (as FP32 values) and the
// ReLU masks use the unrounded pre-activations, so the result is the exact
// gradient of the BF16 forward with its rounding offsets held fixed.
//
// Decoder-parameter gradients stay in the waves' registers (96 accumulators)
// over all of their tiles and are added up once per workgroup; with one float
// atomic per parameter and tile instead, those atomics took a quarter of the
// kernel.  Room for them comes from reading the decoder's operands from the
// LDS where a product needs them.  Feature gradients are contracted on the
// matrix cores per distinct neighbour of a tile.  Eight waves of 256 registers
// fill a CU's registers and its LDS, so the kernel is bound by what two waves
// per SIMD cannot hide of each other: gathers, LDS round trips and the
// matrix-core chains (busy 18% of the time; vector issue 27%).
// Measured (start -> here): 262,144 rays of a 4 x 400 x 400 training step,
// K = 8, S = 16, BF16, 580k samples: 1.09 -> 0.53 ms; 160k rays, K = 12, S = 24,
// FP32 (whole call): 1.52 -> 0.66 ms.
#include <type_traits>

#include "hp_backward.hpp"
#include "hp_search.hpp"  // wave sorts

namespace hp {

constexpr int NPAR = HP_HIDDEN * HP_FEAT_DIM + HP_HIDDEN + HP_HIDDEN * HP_HIDDEN + HP_HIDDEN +
                     4 * HP_HIDDEN + 4;
constexpr int OFF_W1 = 0;
constexpr int OFF_B1 = OFF_W1 + HP_HIDDEN * HP_FEAT_DIM;
constexpr int OFF_W2 = OFF_B1 + HP_HIDDEN;
constexpr int OFF_B2 = OFF_W2 + HP_HIDDEN * HP_HIDDEN;
constexpr int OFF_W3 = OFF_B2 + HP_HIDDEN;
constexpr int OFF_B3 = OFF_W3 + 4 * HP_HIDDEN;
// Floats between workgroup gradient slices: whole 128-byte lines, so that a
// row's atomics never straddle a line (unaligned slices measured 1.3x slower).
constexpr int SSTRIDE = (NPAR + 31) / 32 * 32;

// Floats per row of the 16-sample images in LDS: a row's 16 values and four of
// padding, so that the four rows a store instruction writes (lanes 16 q .. of
// row 4 q + e) fall into different banks.
constexpr int TROW = 20;
constexpr int FROW = HP_FEAT_DIM + 4;  // the same for rows of 32 features

// One wave's LDS.
struct BwdWave {
    float4 o[BWD_CHUNK];            // raw decoder outputs, then their gradients
    float T[BWD_CHUNK];             // transmittance in front of each sample
    float t[BWD_CHUNK];             // ray parameter of each sample
    int32_t pre[WAVE];              // sample prefix over the rays taken
    float inv[16];                  // tile: 1 / sum of the inverse-distance weights
    float4 w[16][2];                // tile: eight inverse-distance weights per sample
    float F[HP_FEAT_DIM * TROW];    // tile: aggregated features [feature][sample], later their gradients [sample][feature]
    float H1T[HP_HIDDEN][TROW];     // tile: layer-1 activations, then their gradients
    float H2T[HP_HIDDEN][TROW];     // tile: layer-2 activations, then their gradients
};
static_assert(16 * FROW <= HP_FEAT_DIM * TROW, "feature gradients exceed the feature image");

// A tile's pairs of neighbour and sample in the area of the hidden activations
// once those are read: at most 16 KT of them.
template <int KT>
struct TilePairs {
    float m[16][TROW];         // weights of 16 distinct neighbours (rows) for the tile's samples
    float w[16][KT];           // normalised inverse-distance weights [sample][place in its list]
    int32_t index[16 * KT + 16];  // distinct neighbours
};
static_assert(sizeof(TilePairs<HP_MAX_K>) <= 2 * sizeof(float) * HP_HIDDEN * TROW && HP_MAX_K <= 32,
              "neighbour staging exceeds its LDS area");

// Aggregated feature slice (features 8 q .. 8 q + 7) of sample row `row`; the
// same arithmetic as the render (summed in neighbour order), NG neighbours at
// a time: their lists and then their rows in flight together, as there are
// only two waves per SIMD to hide each other's waits.  The sample's four lanes
// share the weights through `sw`.  Returns 1 / sum of the weights.
template <int NG>
__device__ __forceinline__ float idw_slice_bwd(const BwdArgs &A, int64_t row, int q, float4 (&sw)[2], float *f)
{
#pragma unroll
    for (int e = 0; e < 8; ++e) f[e] = 0.0f;
    float wsum = 0.0f;
    const int32_t *ki = A.knn_idx + row * A.K;
    const float *kd = A.knn_dist + row * A.K;
    const bool vec = nbr_vec_ok(A.knn_idx, A.knn_dist, A.K);
    for (int k0 = 0; k0 < A.K; k0 += NG) {
        int idx[NG];
        float d[NG], w[NG];
#pragma unroll
        for (int h = 0; h < NG; h += 4) {
            if (k0 + h < A.K) {
                load_nbr4(ki, kd, k0 + h, A.K, vec, idx + h, d + h);
            } else {
#pragma unroll
                for (int j = h; j < h + 4; ++j) idx[j] = -1, d[j] = 1.0f;
            }
        }
        // (a list ends with the group of four that its last neighbours do not fill)
        if constexpr (NG == 8)
            if (idx[3] < 0) idx[4] = idx[5] = idx[6] = idx[7] = -1;
        float4 x0[NG], x1[NG];
#pragma unroll
        for (int j = 0; j < NG; ++j) {
            const float4 *src =
                reinterpret_cast<const float4 *>(A.feat + (int64_t)(idx[j] >= 0 ? idx[j] : 0) * HP_FEAT_DIM + 8 * q);
            x0[j] = src[0];
            x1[j] = src[1];
        }
        // the sample's four lanes share the weights, one division per four each
        wave_lds_sync();  // the previous weights are read
#pragma unroll
        for (int h = 0; h < NG; h += 4) {
            const float dq = q == 0 ? d[h] : q == 1 ? d[h + 1] : q == 2 ? d[h + 2] : d[h + 3];
            reinterpret_cast<float *>(sw)[h + q] = 1.0f / (dq > A.eps_idw ? dq : A.eps_idw);
        }
        wave_lds_sync();
#pragma unroll
        for (int h = 0; h < NG; h += 4) {
            const float4 wv = sw[h / 4];
            w[h] = wv.x, w[h + 1] = wv.y, w[h + 2] = wv.z, w[h + 3] = wv.w;
        }
#pragma unroll
        for (int j = 0; j < NG; ++j) {
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
        if (idx[NG - 1] < 0) break;
    }
    const float inv = wsum > 0.0f ? 1.0f / wsum : 0.0f;
#pragma unroll
    for (int e = 0; e < 8; ++e) f[e] *= inv;
    return inv;
}

// Row of sample `sidx` of the rays a .. b - 1 taken (first: the first one's
// prefix): the last ray whose prefix is <= first + sidx.
__device__ __forceinline__ int64_t sample_row(const BwdWave &sh, const BwdArgs &A, int64_t ray0, int a, int b,
                                              int first, int sidx)
{
    int lo = a, hi = b;
    while (hi - lo > 1) {
        const int mid = (lo + hi) >> 1;
        if (sh.pre[mid] <= first + sidx) lo = mid;
        else hi = mid;
    }
    return (ray0 + lo) * A.S + (first + sidx - sh.pre[lo]);
}

// The decoder in the LDS, shared by the workgroup: the operands of the replay
// (as in the render), and of the backward products dZ2 W2 and dZ1 W1, whose A
// operands are the transposed weights in the C layout's unit order:
// w2t(o1, o2).e = W2[16 o2 + 4 q + e][16 o1 + r], w1t(cb, o1).e = W1[16 o1 +
// 4 q + e][16 cb + r].
template <int PREC>
struct BwdDecoder;

// BF16: the replay's fragments, and the rounded weights as FP32 images.
template <>
struct BwdDecoder<HP_BF16> {
    MlpBf16Shared m;
    float4 imgW2[16 * WAVE], imgW1[8 * WAVE];

    __device__ __forceinline__ void fill(const MlpWeights &a)
    {
        store_mlp_bf16_shared(a, m, threadIdx.x / WAVE, BWD_WAVES);
        for (int i = threadIdx.x; i < 16 * WAVE; i += blockDim.x) {
            const int ln = i % WAVE, blk = i / WAVE, o1 = blk >> 2, o2 = blk & 3;
            const float *w = a.W2 + (16 * o2 + 4 * (ln >> 4)) * HP_HIDDEN + 16 * o1 + (ln & 15);
            imgW2[i] = make_float4(bf16_round(w[0]), bf16_round(w[HP_HIDDEN]), bf16_round(w[2 * HP_HIDDEN]),
                                   bf16_round(w[3 * HP_HIDDEN]));
        }
        for (int i = threadIdx.x; i < 8 * WAVE; i += blockDim.x) {
            const int ln = i % WAVE, blk = i / WAVE, cb = blk >> 2, o1 = blk & 3;
            const float *w = a.W1 + (16 * o1 + 4 * (ln >> 4)) * HP_FEAT_DIM + 16 * cb + (ln & 15);
            imgW1[i] = make_float4(bf16_round(w[0]), bf16_round(w[HP_FEAT_DIM]), bf16_round(w[2 * HP_FEAT_DIM]),
                                   bf16_round(w[3 * HP_FEAT_DIM]));
        }
    }
    __device__ __forceinline__ const MlpBf16Shared &replay() const { return m; }
    __device__ __forceinline__ f32x4 w2t(int o1, int o2, int l) const
    {
        const float4 v = imgW2[(o1 * 4 + o2) * WAVE + l];
        return {v.x, v.y, v.z, v.w};
    }
    __device__ __forceinline__ f32x4 w1t(int cb, int o1, int l) const
    {
        const float4 v = imgW1[(cb * 4 + o1) * WAVE + l];
        return {v.x, v.y, v.z, v.w};
    }
};

// FP32: one copy serves both, as twice the size would not fit; the transposed
// operands are read from it a float at a time.  A quad of padding after every
// 16 lanes puts those reads into different banks.
template <>
struct BwdDecoder<HP_FP32> {
    static constexpr int ROW = WAVE + 4;
    float4 w1[4][2][ROW], w2[4][4][ROW], w3[4][WAVE], b1[16], b2[16], b3[4];

    static __device__ __forceinline__ int at(int l) { return l + (l >> 4); }
    static __device__ __forceinline__ f32x4 as_f32x4(const float4 &v) { return {v.x, v.y, v.z, v.w}; }
    __device__ __forceinline__ f32x4 W1q(int ob, int i) const { return as_f32x4(w1[ob][i][at(lane_id())]); }
    __device__ __forceinline__ f32x4 W2q(int ob, int i) const { return as_f32x4(w2[ob][i][at(lane_id())]); }
    __device__ __forceinline__ f32x4 W3q(int i) const { return as_f32x4(w3[i][lane_id()]); }
    __device__ __forceinline__ f32x4 B1(int ob) const { return as_f32x4(b1[4 * ob + (lane_id() >> 4)]); }
    __device__ __forceinline__ f32x4 B2(int ob) const { return as_f32x4(b2[4 * ob + (lane_id() >> 4)]); }
    __device__ __forceinline__ f32x4 B3() const { return as_f32x4(b3[lane_id() >> 4]); }

    __device__ __forceinline__ void fill(const MlpWeights &a)
    {
        const int l = lane_id();
        for (int p = threadIdx.x / WAVE; p < 28; p += BWD_WAVES) {
            if (p < 8) w1[p >> 1][p & 1][at(l)] = w1_quad_f32(a, p >> 1, p & 1, l);
            else if (p < 24) w2[(p - 8) >> 2][(p - 8) & 3][at(l)] = w2_quad_f32(a, (p - 8) >> 2, (p - 8) & 3, l);
            else w3[p - 24][l] = w3_quad_f32(a, p - 24, l);
        }
        if (threadIdx.x < WAVE) {
            reinterpret_cast<float *>(b1)[l] = a.b1[l];
            reinterpret_cast<float *>(b2)[l] = a.b2[l];
            if (l < 16) reinterpret_cast<float *>(b3)[l] = l < 4 ? a.b3[l] : 0.0f;
        }
    }
    __device__ __forceinline__ const BwdDecoder &replay() const { return *this; }
    // W2[16 ob + r'][16 i + 4 q' + c] is float c of lane 16 q' + r' of w2[ob][i]
    __device__ __forceinline__ f32x4 w2t(int o1, int o2, int l) const
    {
        const int r = l & 15, q = l >> 4;
        const float *p = reinterpret_cast<const float *>(&w2[o2][o1][at(16 * (r >> 2) + 4 * q)]) + (r & 3);
        return {p[0], p[4], p[8], p[12]};
    }
    // W1[16 ob + r'][8 q' + 4 i + c] is float c of lane 16 q' + r' of w1[ob][i]
    __device__ __forceinline__ f32x4 w1t(int cb, int o1, int l) const
    {
        const int r = l & 15, q = l >> 4;
        const float *p =
            reinterpret_cast<const float *>(&w1[o1][(r >> 2) & 1][at(16 * (2 * cb + (r >> 3)) + 4 * q)]) + (r & 3);
        return {p[0], p[4], p[8], p[12]};
    }
};

// KT: 8, 16 or 32, at least K (it bounds what a lane holds of a tile's neighbour lists)
template <int PREC, int KT>
__global__ void __launch_bounds__(WAVE *BWD_WAVES) k_render_backward(BwdArgs A)
{
    __shared__ BwdWave waves[BWD_WAVES];
    __shared__ BwdDecoder<PREC> dec;
    __shared__ float sW3[4 * HP_HIDDEN];
    // (the FP32 decoder's operands leave no registers for more than four rows)
    constexpr int NG = PREC == HP_BF16 ? 8 : 4;
    const int wave = threadIdx.x >> 6;
    BwdWave &sh = waves[wave];
    // decoder-parameter gradients: the workgroup's workspace slice, zeroed
    // before the first launch that adds to it
    float *const gpar = A.partial + (int64_t)blockIdx.x * SSTRIDE;
    const int l = lane_id();
    const int r16 = l & 15, q = l >> 4;

    // the decoder's operands are read where a product needs them (they hold no
    // registers otherwise)
    const auto &img = dec.replay();
    // a value as the decoder consumes it (bfloat16-rounded with the BF16 decoder)
    auto opnd = [](float w) { return PREC == HP_BF16 ? bf16_round(w) : w; };
    dec.fill(A.w);
    for (int i = threadIdx.x; i < 4 * HP_HIDDEN; i += blockDim.x) sW3[i] = opnd(A.w.W3[i]);
    __syncthreads();
    // lane l: column l of dW3, entry l of db1 and db2, a share of entry q of db3
    float gW3[4] = {0.0f, 0.0f, 0.0f, 0.0f};
    float gb1 = 0.0f, gb2 = 0.0f, gb3 = 0.0f;
    // blocks (o2, o1) of dW2 and (o1, cb) of dW1 over all of the wave's tiles:
    // lane holds dW2[16 o2 + 4 q + e][16 o1 + r16], dW1[16 o1 + 4 q + e][16 cb + r16]
    f32x4 aW2[16], aW1[8];
#pragma unroll
    for (int i = 0; i < 16; ++i) aW2[i] = f32x4{0.0f, 0.0f, 0.0f, 0.0f};
#pragma unroll
    for (int i = 0; i < 8; ++i) aW1[i] = f32x4{0.0f, 0.0f, 0.0f, 0.0f};

    // chunks of consecutive rays are taken from work counters, one per
    // wave at a time: a chunk's cost follows its sample count, which varies
    // from none (background) to rpw * S, so a fixed deal would leave the
    // launch waiting on the waves that drew the busiest chunks.  Counter c
    // deals chunks c, c + 8, ...; a wave starts with its workgroup's and goes
    // on to the next when that has none left (one counter for all took 4.7 ns
    // per chunk, a tenth of the launch).
    const int64_t n_chunks = (A.n_rays + A.rpw - 1) / A.rpw;
    for (int c = 0; c < BWD_QUEUES;) {
        const int own = (blockIdx.x + c) % BWD_QUEUES;
        int taken = 0;
        if (l == 0) taken = atomicAdd(A.queue + own * BWD_QUEUE_STRIDE, 1);
        const int64_t ch = (int64_t)__builtin_amdgcn_readfirstlane(taken) * BWD_QUEUES + own;
        if (ch >= n_chunks) {
            ++c;
            continue;
        }
        const int64_t ray0 = ch * A.rpw;
        const int nr = (A.n_rays - ray0) < A.rpw ? (int)(A.n_rays - ray0) : A.rpw;
        float g0 = 0.0f, g1 = 0.0f, g2 = 0.0f;
        int ns = 0;
        if (l < nr) {
            const int64_t ray = ray0 + l;
            g0 = A.grad_rgb[3 * ray];
            g1 = A.grad_rgb[3 * ray + 1];
            g2 = A.grad_rgb[3 * ray + 2];
            // a ray without incoming gradient contributes nothing
            // (a count beyond the sample cap would index past the ray's rows)
            if (g0 != 0.0f || g1 != 0.0f || g2 != 0.0f) ns = min(max(A.n_sel[ray], 0), A.S);
        }
        const int inc = wave_incl_scan_i32(ns);
        sh.pre[l] = inc - ns;
        const int taken_samples = readlane_i32(inc, WAVE - 1);
        wave_lds_sync();

        // as many consecutive rays at a time as BWD_CHUNK samples hold (a
        // ray's at least: S <= BWD_CHUNK), rays ra .. rb - 1
        for (int ra = 0, first = 0; first < taken_samples;) {
        const int rb = popc64(ballot(inc - first <= BWD_CHUNK) & ballot(l < nr));
        const int total = readlane_i32(inc, rb - 1) - first;

        // pass A: raw decoder outputs of every sample
        for (int s0 = 0; s0 < total; s0 += 16) {
            const int sidx = s0 + r16;
            float f[8];
            if (sidx < total) {
                const int64_t row = sample_row(sh, A, ray0, ra, rb, first, sidx);
                if (q == 0) sh.t[sidx] = A.t[row];
                idw_slice_bwd<NG>(A, row, q, sh.w[r16], f);
            } else {
#pragma unroll
                for (int e = 0; e < 8; ++e) f[e] = 0.0f;
            }
            f32x4 o;
            __asm__ volatile("" ::: "memory");
            if constexpr (PREC == HP_BF16) o = decode_bf16(img, f);
            else o = decode_f32(img, f);
            if (q == 0 && sidx < total) sh.o[sidx] = make_float4(o[0], o[1], o[2], o[3]);
        }
        wave_lds_sync();

        // compositing backward (Eq. 2): lane r walks ray r of the rays taken
        if (ns > 0 && l >= ra && l < rb) {
            const int base = sh.pre[l] - first;
            const float *const tr = sh.t + base;
            float T = 1.0f;
            for (int j = 0; j < ns; ++j) {
                sh.T[base + j] = T;
                const float sg = softplus_f(sh.o[base + j].w);
                const float dl = (j + 1 < ns) ? tr[j + 1] - tr[j] : A.delta_last;
                T *= expf(-sg * dl);
            }
            // U: colour composited behind sample j relative to T_{j+1};
            // P: transmittance through everything behind j (background weight)
            float U0 = 0.0f, U1 = 0.0f, U2 = 0.0f, P = 1.0f;
            for (int j = ns - 1; j >= 0; --j) {
                const float4 o = sh.o[base + j];
                const float c0 = sigmoid_f(o.x), c1 = sigmoid_f(o.y), c2 = sigmoid_f(o.z);
                const float sg = softplus_f(o.w);
                const float dl = (j + 1 < ns) ? tr[j + 1] - tr[j] : A.delta_last;
                const float e = expf(-sg * dl);
                const float a = 1.0f - e;
                const float Tj = sh.T[base + j];
                const float dLda = g0 * (Tj * (c0 - U0) - A.bg[0] * Tj * P) +
                                   g1 * (Tj * (c1 - U1) - A.bg[1] * Tj * P) +
                                   g2 * (Tj * (c2 - U2) - A.bg[2] * Tj * P);
                const float ws = Tj * a;
                sh.o[base + j] = make_float4(g0 * ws * c0 * (1.0f - c0), g1 * ws * c1 * (1.0f - c1),
                                             g2 * ws * c2 * (1.0f - c2), dLda * dl * e * sigmoid_f(o.w));
                U0 = a * c0 + e * U0;
                U1 = a * c1 + e * U1;
                U2 = a * c2 + e * U2;
                P = e * P;
            }
        }
        wave_lds_sync();

        // pass B: per tile, replay the decoder keeping its activations, then
        // run the decoder backward on FP32 MFMA (v_mfma_f32_16x16x4f32, lane
        // l = 16 q + r supplies A[r][q] and B[q][r] and holds D[4 q + e][r]).
        // Activation gradients chain through the C layout like the forward
        // (unit 16 b + 4 q + e of sample r), with the contraction index
        // permuted in the weight images.  The weight gradients contract over
        // the tile's samples, so their operands come from transposed LDS
        // images [unit][TP(s)], TP(s) = 4 (s mod 4) + s / 4, where a lane's
        // four samples q, q + 4, q + 8, q + 12 are one 16-byte read.
        const int ps = 4 * (r16 & 3) + (r16 >> 2);  // TP(r16)
        float *const FT = sh.F;  // [feature][TP(s)], later [s][feature]
        for (int s0 = 0; s0 < total; s0 += 16) {
            const int nt = (total - s0) < 16 ? total - s0 : 16;
            const int sidx = s0 + r16;
            const bool valid = sidx < total;
            f32x4 h1[4], h2[4];
            int64_t row = -1;
            {
                float f[8];
                float inv = 0.0f;
                if (valid) {
                    row = sample_row(sh, A, ray0, ra, rb, first, sidx);
                    inv = idw_slice_bwd<NG>(A, row, q, sh.w[r16], f);
                } else {
#pragma unroll
                    for (int e = 0; e < 8; ++e) f[e] = 0.0f;
                }
                __asm__ volatile("" ::: "memory");
                if constexpr (PREC == HP_BF16) decode_bf16(img, f, h1, h2);
                else decode_f32(img, f, h1, h2);
                if (q == 0) sh.inv[r16] = inv;
                // the weight gradients contract the activations as the next
                // layer consumed them (bfloat16-rounded with the BF16 decoder);
                // the registers keep the unrounded values for the ReLU masks
#pragma unroll
                for (int ob = 0; ob < 4; ++ob)
#pragma unroll
                    for (int e = 0; e < 4; ++e) {
                        if (!valid) {
                            h1[ob][e] = 0.0f;
                            h2[ob][e] = 0.0f;
                        }
                        sh.H1T[16 * ob + 4 * q + e][ps] = opnd(h1[ob][e]);
                        sh.H2T[16 * ob + 4 * q + e][ps] = opnd(h2[ob][e]);
                    }
#pragma unroll
                for (int e = 0; e < 8; ++e) FT[(8 * q + e) * TROW + ps] = opnd(f[e]);
            }
            // the tile's neighbour lists, fetched now (all loads independent,
            // in flight during the products) and staged in LDS after them
            // lane (r16, q): entries q, q + 4, ... of sample r16
            constexpr int PF = KT / 4;
            int32_t pf_i[PF];
            float pf_d[PF];
            {
                const int64_t prow = row;
#pragma unroll
                for (int m = 0; m < PF; ++m) {
                    const int k = q + 4 * m;
                    pf_i[m] = -1;
                    pf_d[m] = 0.0f;
                    if (prow >= 0 && k < A.K) {
                        pf_i[m] = A.knn_idx[prow * A.K + k];
                        pf_d[m] = A.knn_dist[prow * A.K + k];
                    }
                }
            }
            wave_lds_sync();
            // output layer: dW3 and db3 on the VALU, lane l = hidden unit l
            {
                float hrow[16];
#pragma unroll
                for (int k = 0; k < 4; ++k) {
                    const float4 v = *reinterpret_cast<const float4 *>(&sh.H2T[l][4 * k]);
                    hrow[4 * k] = v.x;
                    hrow[4 * k + 1] = v.y;
                    hrow[4 * k + 2] = v.z;
                    hrow[4 * k + 3] = v.w;
                }
#pragma unroll
                for (int s = 0; s < 16; ++s) {
                    if (s < nt) {
                        const float4 d = sh.o[s0 + s];
                        const float h = hrow[4 * (s & 3) + (s >> 2)];
                        gW3[0] = fma_rn(d.x, h, gW3[0]);
                        gW3[1] = fma_rn(d.y, h, gW3[1]);
                        gW3[2] = fma_rn(d.z, h, gW3[2]);
                        gW3[3] = fma_rn(d.w, h, gW3[3]);
                    }
                }
            }
            // dZ2 = (dO W3) masked by layer 2's ReLU: A = W3[q][unit], B = dO[s][q]
            f32x4 dz2[4];
            {
                float dOq = 0.0f;
                if (valid) {
                    const float4 d = sh.o[sidx];
                    dOq = q == 0 ? d.x : (q == 1 ? d.y : (q == 2 ? d.z : d.w));
                }
                gb3 += dOq;
#pragma unroll
                for (int ob = 0; ob < 4; ++ob) {
                    f32x4 acc = {0.0f, 0.0f, 0.0f, 0.0f};
                    acc = __builtin_amdgcn_mfma_f32_16x16x4f32(sW3[q * HP_HIDDEN + 16 * ob + r16], dOq, acc, 0, 0, 0);
#pragma unroll
                    for (int e = 0; e < 4; ++e) dz2[ob][e] = h2[ob][e] > 0.0f ? acc[e] : 0.0f;
                }
            }
            wave_lds_sync();  // H2T (activations) fully read
#pragma unroll
            for (int ob = 0; ob < 4; ++ob)
#pragma unroll
                for (int e = 0; e < 4; ++e) sh.H2T[16 * ob + 4 * q + e][ps] = dz2[ob][e];
            wave_lds_sync();
            // db2 (lane l = unit l) and dW2 += dZ2^T H1 over the tile's samples
            {
#pragma unroll
                for (int k = 0; k < 4; ++k) {
                    const float4 v = *reinterpret_cast<const float4 *>(&sh.H2T[l][4 * k]);
                    gb2 += v.x;
                    gb2 += v.y;
                    gb2 += v.z;
                    gb2 += v.w;
                }
                float4 b1[4];
#pragma unroll
                for (int ob = 0; ob < 4; ++ob)
                    b1[ob] = *reinterpret_cast<const float4 *>(&sh.H1T[16 * ob + r16][4 * q]);
#pragma unroll
                for (int o2 = 0; o2 < 4; ++o2) {
                    const float4 a2 = *reinterpret_cast<const float4 *>(&sh.H2T[16 * o2 + r16][4 * q]);
#pragma unroll
                    for (int o1 = 0; o1 < 4; ++o1) {
                        f32x4 &acc = aW2[4 * o2 + o1];
                        acc = __builtin_amdgcn_mfma_f32_16x16x4f32(a2.x, b1[o1].x, acc, 0, 0, 0);
                        acc = __builtin_amdgcn_mfma_f32_16x16x4f32(a2.y, b1[o1].y, acc, 0, 0, 0);
                        acc = __builtin_amdgcn_mfma_f32_16x16x4f32(a2.z, b1[o1].z, acc, 0, 0, 0);
                        acc = __builtin_amdgcn_mfma_f32_16x16x4f32(a2.w, b1[o1].w, acc, 0, 0, 0);
                    }
                }
            }
            // dZ1 = (dZ2 W2) masked by layer 1's ReLU; step (ob2, e) contracts
            // unit 16 ob2 + 4 q + e of layer 2
            f32x4 dz1[4];
#pragma unroll
            for (int o1 = 0; o1 < 4; ++o1) {
                f32x4 acc = {0.0f, 0.0f, 0.0f, 0.0f};
#pragma unroll
                for (int o2 = 0; o2 < 4; ++o2) {
                    const f32x4 w = dec.w2t(o1, o2, l);
#pragma unroll
                    for (int e = 0; e < 4; ++e)
                        acc = __builtin_amdgcn_mfma_f32_16x16x4f32(w[e], dz2[o2][e], acc, 0, 0, 0);
                }
#pragma unroll
                for (int e = 0; e < 4; ++e) dz1[o1][e] = h1[o1][e] > 0.0f ? acc[e] : 0.0f;
            }
            wave_lds_sync();  // H1T (activations) fully read
#pragma unroll
            for (int ob = 0; ob < 4; ++ob)
#pragma unroll
                for (int e = 0; e < 4; ++e) sh.H1T[16 * ob + 4 * q + e][ps] = dz1[ob][e];
            wave_lds_sync();
            // db1 (lane l = unit l) and dW1 += dZ1^T F over the tile's samples
            {
#pragma unroll
                for (int k = 0; k < 4; ++k) {
                    const float4 v = *reinterpret_cast<const float4 *>(&sh.H1T[l][4 * k]);
                    gb1 += v.x;
                    gb1 += v.y;
                    gb1 += v.z;
                    gb1 += v.w;
                }
                float4 bf[2];
#pragma unroll
                for (int cb = 0; cb < 2; ++cb)
                    bf[cb] = *reinterpret_cast<const float4 *>(&FT[(16 * cb + r16) * TROW + 4 * q]);
#pragma unroll
                for (int o1 = 0; o1 < 4; ++o1) {
                    const float4 a1 = *reinterpret_cast<const float4 *>(&sh.H1T[16 * o1 + r16][4 * q]);
#pragma unroll
                    for (int cb = 0; cb < 2; ++cb) {
                        f32x4 &acc = aW1[2 * o1 + cb];
                        acc = __builtin_amdgcn_mfma_f32_16x16x4f32(a1.x, bf[cb].x, acc, 0, 0, 0);
                        acc = __builtin_amdgcn_mfma_f32_16x16x4f32(a1.y, bf[cb].y, acc, 0, 0, 0);
                        acc = __builtin_amdgcn_mfma_f32_16x16x4f32(a1.z, bf[cb].z, acc, 0, 0, 0);
                        acc = __builtin_amdgcn_mfma_f32_16x16x4f32(a1.w, bf[cb].w, acc, 0, 0, 0);
                    }
                }
            }
            // dF = dZ1 W1 (gradient of the aggregated features), written as
            // [sample][feature] over the feature image once dW1 has read it
            f32x4 dF[2];
#pragma unroll
            for (int cb = 0; cb < 2; ++cb) {
                f32x4 acc = {0.0f, 0.0f, 0.0f, 0.0f};
#pragma unroll
                for (int o1 = 0; o1 < 4; ++o1) {
                    const f32x4 w = dec.w1t(cb, o1, l);
#pragma unroll
                    for (int e = 0; e < 4; ++e)
                        acc = __builtin_amdgcn_mfma_f32_16x16x4f32(w[e], dz1[o1][e], acc, 0, 0, 0);
                }
                dF[cb] = acc;
            }
            wave_lds_sync();  // the feature image fully read
#pragma unroll
            for (int cb = 0; cb < 2; ++cb)
                *reinterpret_cast<float4 *>(&FT[r16 * FROW + 16 * cb + 4 * q]) =
                    make_float4(dF[cb][0], dF[cb][1], dF[cb][2], dF[cb][3]);
            // aggregation backward: d feat[j] = sum over the tile's samples of
            // M[j][s] dF[s], M[j][s] = w_k / sum w where j is neighbour k of s.
            // Consecutive samples share most neighbours, so the tile's pairs
            // are sorted by neighbour and each distinct one becomes a row of
            // M; 16 rows at a time are contracted with dF on the matrix cores
            // and added with one atomic per (neighbour, channel).  (A loop
            // over each neighbour's pairs instead waited for two LDS reads
            // in turn per pair, 64 pairs per tile one after the other.)
            // Keys: neighbour index << 32 | sample << 5 | place in its list.
            TilePairs<KT> &tp = *reinterpret_cast<TilePairs<KT> *>(&sh.H1T[0][0]);
            {
                const float pinv = sh.inv[r16];
                uint64_t key[PF];
#pragma unroll
                for (int m = 0; m < PF; ++m) {
                    const int k = q + 4 * m;
                    const float d = pf_d[m];
                    tp.w[r16][k] = (1.0f / (d > A.eps_idw ? d : A.eps_idw)) * pinv;
                    key[m] = pf_i[m] >= 0 ? ((uint64_t)(uint32_t)pf_i[m] << 32) | (uint32_t)(r16 << 5 | k) : KEY_NONE;
                }
                wave_sort_many(key);
                // row of M of every pair: the heads (first pair of a distinct
                // neighbour) up to it
                int idx[PF], rank[PF], heads = 0;
#pragma unroll
                for (int m = 0; m < PF; ++m) idx[m] = key[m] != KEY_NONE ? (int)(key[m] >> 32) : -1;
                int prev = __shfl_up(idx[PF - 1], 1, WAVE);
                if (l == 0) prev = -1;
#pragma unroll
                for (int m = 0; m < PF; ++m) {
                    heads += (idx[m] >= 0 && prev != idx[m]) ? 1 : 0;
                    rank[m] = heads;
                    prev = idx[m];
                }
                const int inc = wave_incl_scan_i32(heads);
                const int nu = readlane_i32(inc, WAVE - 1);
                wave_lds_sync();
                float wp[PF];
#pragma unroll
                for (int m = 0; m < PF; ++m) {
                    rank[m] = idx[m] >= 0 ? rank[m] + inc - heads - 1 : -1;
                    // (every pair of a neighbour stores the same index)
                    if (idx[m] >= 0) tp.index[rank[m]] = idx[m];
                    wp[m] = tp.w[((uint32_t)key[m] >> 5) & 15u][(uint32_t)key[m] & (KT - 1u)];
                }
                float df[2][4];  // gradients of sample 4 q + e, channel 16 cb + r16
#pragma unroll
                for (int cb = 0; cb < 2; ++cb)
#pragma unroll
                    for (int e = 0; e < 4; ++e) df[cb][e] = FT[(4 * q + e) * FROW + 16 * cb + r16];
                // M holds zeros where a sample does not name a neighbour, and
                // zero times an infinity or a NaN is a NaN, which would reach
                // every point of the tile: a tile with a gradient that is not
                // finite adds its pairs one by one instead of contracting them.
                // (their sum is not finite then; a sum that overflows only
                // takes the slower way.  The test is not measurable: 160k
                // rays, K = 12, S = 24, FP32 660 us with and without it)
                float sum = 0.0f;
#pragma unroll
                for (int e = 0; e < 4; ++e) sum += df[0][e] + df[1][e];
                const bool pairs = ballot(!(__builtin_fabsf(sum) < __builtin_inff())) != 0;
                if (pairs) {
                    wave_lds_sync();
#pragma unroll
                    for (int m = 0; m < PF; ++m) {
                        if (rank[m] < 0) continue;
                        const float *const g = FT + (((uint32_t)key[m] >> 5) & 15u) * FROW;
                        float *const at = A.grad_feat + (int64_t)tp.index[rank[m]] * HP_FEAT_DIM;
#pragma unroll 1
                        for (int c = 0; c < HP_FEAT_DIM; ++c) atomicAdd(at + c, wp[m] * g[c]);
                    }
                }
                for (int j0 = 0; j0 < nu && !pairs; j0 += 16) {
                    *reinterpret_cast<float4 *>(&tp.m[r16][4 * q]) = make_float4(0.0f, 0.0f, 0.0f, 0.0f);
                    wave_lds_sync();
#pragma unroll
                    for (int m = 0; m < PF; ++m)
                        if (rank[m] >= j0 && rank[m] < j0 + 16)
                            // (added: a caller's list may name a point twice)
                            atomicAdd(&tp.m[rank[m] - j0][((uint32_t)key[m] >> 5) & 15u], wp[m]);
                    wave_lds_sync();
                    const float4 a = *reinterpret_cast<const float4 *>(&tp.m[r16][4 * q]);
                    const int4 at = *reinterpret_cast<const int4 *>(&tp.index[j0 + 4 * q]);
                    wave_lds_sync();
                    const int row4[4] = {at.x, at.y, at.z, at.w};
#pragma unroll
                    for (int cb = 0; cb < 2; ++cb) {
                        f32x4 acc = {0.0f, 0.0f, 0.0f, 0.0f};
                        acc = __builtin_amdgcn_mfma_f32_16x16x4f32(a.x, df[cb][0], acc, 0, 0, 0);
                        acc = __builtin_amdgcn_mfma_f32_16x16x4f32(a.y, df[cb][1], acc, 0, 0, 0);
                        acc = __builtin_amdgcn_mfma_f32_16x16x4f32(a.z, df[cb][2], acc, 0, 0, 0);
                        acc = __builtin_amdgcn_mfma_f32_16x16x4f32(a.w, df[cb][3], acc, 0, 0, 0);
#pragma unroll
                        for (int e = 0; e < 4; ++e)
                            if (j0 + 4 * q + e < nu)
                                atomicAdd(&A.grad_feat[(int64_t)row4[e] * HP_FEAT_DIM + 16 * cb + r16], acc[e]);
                    }
                }
            }
            wave_lds_sync();
        }
        first += total;
        ra = rb;
        }
    }

    // The waves' parameter gradients added up in the LDS, one wave after the
    // other (the tiles' area, dead now), and the sum to the workgroup's slice,
    // which no other workgroup touches.
    __syncthreads();
    float *const red = reinterpret_cast<float *>(waves);
    static_assert(NPAR * sizeof(float) <= sizeof(waves), "the parameter gradients exceed the tiles' area");
    for (int k = 1; k < 16; k <<= 1) gb3 += __shfl_xor(gb3, k, WAVE);
    for (int w = 0; w < BWD_WAVES; ++w) {
        if (w == wave) {
            auto put = [&](int at, float v) { red[at] = w ? red[at] + v : v; };
#pragma unroll
            for (int i = 0; i < 16; ++i)
#pragma unroll
                for (int e = 0; e < 4; ++e)
                    put(OFF_W2 + (16 * (i >> 2) + 4 * q + e) * HP_HIDDEN + 16 * (i & 3) + r16, aW2[i][e]);
#pragma unroll
            for (int i = 0; i < 8; ++i)
#pragma unroll
                for (int e = 0; e < 4; ++e)
                    put(OFF_W1 + (16 * (i >> 1) + 4 * q + e) * HP_FEAT_DIM + 16 * (i & 1) + r16, aW1[i][e]);
#pragma unroll
            for (int k = 0; k < 4; ++k) put(OFF_W3 + k * HP_HIDDEN + l, gW3[k]);
            put(OFF_B1 + l, gb1);
            put(OFF_B2 + l, gb2);
            if (r16 == 0) put(OFF_B3 + q, gb3);
        }
        __syncthreads();
    }
    for (int i = threadIdx.x; i < NPAR; i += blockDim.x) gpar[i] += red[i];
}

__global__ void __launch_bounds__(256) k_zero_f32(float *p, int64_t n)
{
    const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i < n) p[i] = 0.0f;
}

// Sum the per-workgroup slices and add to the gradients, in a fixed order: each of
// RED_G thread groups sums a contiguous range of slices in order, then the
// group sums are added in group order.  (One thread per parameter walking
// every slice would leave the chip idle: there are only 6,532 parameters.)
constexpr int RED_P = 64;  // parameters per workgroup
constexpr int RED_G = 16;  // slice ranges per parameter

__global__ void __launch_bounds__(RED_P * RED_G) k_reduce_partials(const float *__restrict__ partial,
                                                                  int nslice, float *gW1, float *gb1,
                                                                  float *gW2, float *gb2, float *gW3,
                                                                  float *gb3)
{
    __shared__ float sh[RED_G][RED_P];
    const int p = threadIdx.x % RED_P, grp = threadIdx.x / RED_P;
    const int i = blockIdx.x * RED_P + p;
    const int per = (nslice + RED_G - 1) / RED_G;
    const int b0 = grp * per, b1 = min(nslice, b0 + per);
    float s = 0.0f;
    if (i < NPAR) {
#pragma unroll 8
        for (int b = b0; b < b1; ++b) s += partial[(int64_t)b * SSTRIDE + i];
    }
    sh[grp][p] = s;
    __syncthreads();
    if (grp != 0 || i >= NPAR) return;
    float t = 0.0f;
#pragma unroll
    for (int k = 0; k < RED_G; ++k) t += sh[k][p];
    float *dst;
    int j;
    if (i < OFF_B1) { dst = gW1; j = i - OFF_W1; }
    else if (i < OFF_W2) { dst = gb1; j = i - OFF_B1; }
    else if (i < OFF_B2) { dst = gW2; j = i - OFF_W2; }
    else if (i < OFF_W3) { dst = gb2; j = i - OFF_B2; }
    else if (i < OFF_B3) { dst = gW3; j = i - OFF_W3; }
    else { dst = gb3; j = i - OFF_B3; }
    dst[j] += t;
}

// the slices, then the work counters
constexpr size_t QUEUE_BYTES = BWD_QUEUES * BWD_QUEUE_STRIDE * sizeof(int32_t);

size_t backward_partial_bytes()
{
    return (size_t)BWD_MAX_BLOCKS * SSTRIDE * sizeof(float) + QUEUE_BYTES;
}

static int32_t *queue_of(float *partial)
{
    return reinterpret_cast<int32_t *>(partial + (size_t)BWD_MAX_BLOCKS * SSTRIDE);
}

int backward_slices()
{
    int dev = 0, cus = 256;
    if (hipGetDevice(&dev) == hipSuccess)
        (void)hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, dev);
    // one workgroup fills a CU's LDS: a persistent grid of one per CU
    return cus < BWD_MAX_BLOCKS ? (cus > 0 ? cus : 1) : BWD_MAX_BLOCKS;
}

int backward_rays_per_wave(int S)
{
    const int r = BWD_TAKE / (S > 0 ? S : 1);
    return r > WAVE ? WAVE : r;
}

hipError_t backward_zero(float *partial, hipStream_t s)
{
    const int64_t nzero = (int64_t)backward_slices() * SSTRIDE;
    k_zero_f32<<<dim3((unsigned)((nzero + 255) / 256)), 256, 0, s>>>(partial, nzero);
    return hipGetLastError();
}

template <int KT>
static void launch_backward(const BwdArgs &A, int precision, dim3 grid, hipStream_t s)
{
    const dim3 block(WAVE * BWD_WAVES);
    if (precision == HP_BF16) k_render_backward<HP_BF16, KT><<<grid, block, 0, s>>>(A);
    else k_render_backward<HP_FP32, KT><<<grid, block, 0, s>>>(A);
}

hipError_t backward_accumulate(const BwdArgs &args, int precision, hipStream_t s)
{
    if (args.n_rays == 0) return hipSuccess;
    BwdArgs A = args;
    A.queue = queue_of(A.partial);
    // (a fill kernel, not a memset: callers may capture this in a graph)
    k_zero_f32<<<1, 256, 0, s>>>(reinterpret_cast<float *>(A.queue), BWD_QUEUES * BWD_QUEUE_STRIDE);
    const int64_t chunks = (A.n_rays + A.rpw - 1) / A.rpw;
    int64_t nblk = (chunks + BWD_WAVES - 1) / BWD_WAVES;
    const int64_t nslice = backward_slices();
    if (nblk > nslice) nblk = nslice;
    if (nblk < 1) nblk = 1;
    const dim3 grid((unsigned)nblk);
    if (A.K <= 8) launch_backward<8>(A, precision, grid, s);
    else if (A.K <= 16) launch_backward<16>(A, precision, grid, s);
    else launch_backward<32>(A, precision, grid, s);
    return hipGetLastError();
}

hipError_t backward_reduce(const float *partial, const MlpGrad &gm, hipStream_t s)
{
    k_reduce_partials<<<(NPAR + RED_P - 1) / RED_P, RED_P * RED_G, 0, s>>>(
        partial, backward_slices(), gm.W1, gm.b1, gm.W2, gm.b2, gm.W3, gm.b3);
    return hipGetLastError();
}

}  // namespace hp
