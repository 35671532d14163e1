// Launch interface of the render backward pass.
#pragma once

#include "hp_kernels.hpp"
#include "hp_mlp.hpp"

namespace hp {

constexpr int BWD_WAVES = 8;          // waves per workgroup (one workgroup per CU)
constexpr int BWD_CHUNK = 64;         // samples one wave holds at once (at least HP_MAX_SAMPLES)
constexpr int BWD_TAKE = 128;         // samples the rays that a wave takes at a time may have
constexpr int BWD_QUEUES = 8;         // work counters, a 128-byte line each
constexpr int BWD_QUEUE_STRIDE = 32;
constexpr int BWD_MAX_BLOCKS = 256;   // bound on the persistent grid (one gradient slice each)

static_assert(BWD_CHUNK >= HP_MAX_SAMPLES, "a ray's samples are held at once");

struct MlpGrad {
    float *W1, *b1, *W2, *b2, *W3, *b3;
};

struct BwdArgs {
    const int32_t *n_sel;
    const float *t;
    const int32_t *knn_idx;
    const float *knn_dist;
    int64_t n_rays;
    int32_t K, S, rpw;  // rpw: rays a wave takes at a time, rpw * S <= BWD_TAKE
    const float *feat;
    MlpWeights w;
    float eps_idw, delta_last;
    float bg[3];
    const float *grad_rgb;
    float *grad_feat;
    float *partial;  // per-workgroup decoder-gradient slices
    int32_t *queue;  // work counters of one accumulate launch (zeroed before it)
};

// Decoder-gradient slices: one per workgroup of the backward grid, which is
// at most backward_slices() workgroups for any number of rays, followed by
// the work counters of the accumulate launches.
size_t backward_partial_bytes();
int backward_slices();
int backward_rays_per_wave(int S);
// The three steps of a gradient: zero the slices, accumulate any number of
// ray chunks into them (and into the feature gradient), then add the slices
// in a fixed order to the caller's decoder gradients.
hipError_t backward_zero(float *partial, hipStream_t s);
hipError_t backward_accumulate(const BwdArgs &A, int precision, hipStream_t s);
hipError_t backward_reduce(const float *partial, const MlpGrad &gm, hipStream_t s);

}  // namespace hp
