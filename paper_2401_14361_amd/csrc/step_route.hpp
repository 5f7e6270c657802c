// The routing of an asynchronous layer step inside the launch that streams its experts.
//
// A launch of its own for the routing costs the step 5.5 us, and a fork to a side stream behind it 4.4 more, before the first
// weight is requested.  Here every streaming workgroup has one wavefront more than stream.  A wavefront forms a logit and stores
// it past the caches - those of the workgroups that match first, which are the first to run, so that the router's rows arrive before
// the weights' requests fill the queues - and one of every workgroup waits until the E logits are there, takes the top k (Sec. 2 of the
// paper) for itself and hands the picks to its workgroup through LDS.  Meanwhile the others stream the shared experts, which need no picks.
// (One wavefront that takes the picks and publishes them is three trips to memory more: 3 us beside the stream.)
//
// Every wait ends: a wavefront that has polled `spin` times (400: 0.2 - 1.2 ms) forms all the logits itself, a trip to memory or more a row, the same sums in the same
// order, so that workgroups which hold every compute unit (of two steps on two streams, say) never wait for one that has not
// been scheduled.
#pragma once

#include "common.hpp"
#include "topk.hpp"
#include "wtypes.hpp"

namespace moei {

constexpr int kStepPicks = 64;  // picks of a step at most
// The logits are stored this many times, and a workgroup reads one copy: 250 that poll the same lines wait for each other.
constexpr int kStepCopies = 8;
constexpr int kStepTailThreads = 256;
inline __host__ __device__ size_t step_copy_words(int E) { return (((size_t)E + 511) / 512) * 512 + 32; }  // whole pages, and a line

struct StepRouteArgs {
    const void* W;               // router matrix [E][H] in the weight dtype
    const float* bias;           // [E] or null
    const void* x;               // [H] in the weight dtype
    int H, vec_ok, E, k, renorm;
    // kStepCopies times [E] (step_copy_words apart): a logit in the lower half, 1 in the upper one: each word says by itself that it is
    // there.  Zero between steps.
    unsigned long long* words;
    const int32_t* slot_of_row;  // slot_of + layer*E
    int spin;
};

// What the reduction behind the experts does for the step besides: nobody waits for the words then.
struct StepTail {
    int E;
    unsigned long long* words;  // null: nothing
};

#if defined(__HIPCC__)

// <row, x> by one wavefront: a lane's products in ascending order of the chunks, then the lanes - in every form here and in
// route_fused_kernel the same bits.  NQ: chunk loads that go out together.
template <typename WT, int NQ>
__device__ __forceinline__ float wave_row_product(const WT* row, const WT* x, int H, bool vec_ok, int lane) {
    using V = WVec<WT>;
    constexpr int CW = kWave * V::N;
    float acc = 0.f;
    if (vec_ok) {
#pragma unroll 1
        for (int c0 = lane * V::N; c0 < H; c0 += NQ * CW) {
            typename V::raw wr[NQ], xv[NQ];
#pragma unroll
            for (int q = 0; q < NQ; ++q) {
                const int c = c0 + q * CW < H ? c0 + q * CW : c0;
                wr[q] = V::load(row + c);
                xv[q] = V::load(x + c);
            }
#pragma unroll
            for (int q = 0; q < NQ; ++q) {
                if (c0 + q * CW < H) {
                    float xf[V::N];
                    V::unpack(xv[q], xf);
                    acc = V::dot(wr[q], xf, acc);
                }
            }
        }
    } else {
        for (int c = lane; c < H; c += kWave) acc = __builtin_fmaf(V::one(row + c), V::one(x + c), acc);
    }
    return wave_sum_dpp(acc);
}

// LDS of the wavefront that takes the picks: E logits, kStepPicks indices and weights
__host__ __device__ constexpr size_t step_route_lds(int E) { return ((size_t)E + 2 * kStepPicks) * 4; }

// Rows first, first + n, ... of the router by one wavefront.
template <typename WT>
__device__ __forceinline__ void step_route_rows(const StepRouteArgs& a, int first, int n, int lane) {
    const WT* W = reinterpret_cast<const WT*>(a.W);
    const WT* x = reinterpret_cast<const WT*>(a.x);
#pragma unroll 1
    for (int e = first; e < a.E; e += n) {
        const WT* row = W + (size_t)e * a.H;
        const float bias = a.bias ? a.bias[e] : 0.f;
        const float z = (a.H <= 4 * kWave * WVec<WT>::N ? wave_row_product<WT, 4>(row, x, a.H, a.vec_ok, lane)
                                                        : wave_row_product<WT, 10>(row, x, a.H, a.vec_ok, lane)) + bias;
        if (lane < kStepCopies)
            __hip_atomic_store(&a.words[lane * step_copy_words(a.E) + e], (1ull << 32) | __float_as_uint(z), __ATOMIC_RELAXED,
                               __HIP_MEMORY_SCOPE_AGENT);
    }
}

struct StepPick {
    int e, slot;  // -1: none
    float w;
    bool bad;  // no softmax exists: no picks
};
constexpr int kRegsE = 256;  // logits that one wavefront holds in registers beside their slots

// Lane j < k of one wavefront: pick j.  z: step_route_lds.  SLOTS: the picks' slots too.
template <typename WT, bool SLOTS>
__device__ __forceinline__ StepPick step_picks(const StepRouteArgs& a, float* z, int lane) {
    constexpr int NR = kRegsE / kWave;
    const unsigned long long* words = a.words + (blockIdx.x % kStepCopies) * step_copy_words(a.E);
    int slot[NR] = {};
    if (SLOTS && a.E <= kRegsE) {
#pragma unroll
        for (int r = 0; r < NR; ++r) slot[r] = a.slot_of_row[min(lane + r * kWave, a.E - 1)];
    }
    bool there = false;
#pragma unroll 1
    for (int i = 0; i < a.spin && !there; ++i) {
        bool mine = true;
#pragma unroll 1
        for (int e0 = lane; e0 - lane < a.E; e0 += kRegsE) {
            unsigned long long v[NR];
#pragma unroll
            for (int r = 0; r < NR; ++r)
                v[r] = __hip_atomic_load(&words[min(e0 + r * kWave, a.E - 1)], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
#pragma unroll
            for (int r = 0; r < NR; ++r) {
                mine &= (uint32_t)(v[r] >> 32) != 0u;
                if (e0 + r * kWave < a.E) z[e0 + r * kWave] = __uint_as_float((uint32_t)v[r]);
            }
        }
        there = __ballot(!mine) == 0ull;
        if (!there) __builtin_amdgcn_s_sleep(1);
    }
    if (!there) {  // uniform
        const WT* W = reinterpret_cast<const WT*>(a.W);
        const WT* x = reinterpret_cast<const WT*>(a.x);
#pragma unroll 1
        for (int e = 0; e < a.E; ++e) {
            const float r = wave_row_product<WT, 1>(W + (size_t)e * a.H, x, a.H, a.vec_ok, lane) + (a.bias ? a.bias[e] : 0.f);
            if (lane == 0) z[e] = r;
        }
    }
    wave_lds_fence();
    StepPick p{-1, -1, 0.f, wave_logits_bad(z, a.E, lane)};
    if (p.bad) return p;  // uniform
    // Ranked are few experts for their picks: that takes 0.3 - 2 us for up to 64 experts, twice as long for up to 128, a round of the other 0.14.
    // us a layer, rounds / ranking, 9 experts, 8 picks 40.0 / 38.5; 64, 64 90 / 81; 64, 16 36.7 / 36.1; 64, 8 30.1 / 30.8; 32, 4 28.7 / 29.0; 16, 4 40.8 / 40.4.
    if (4 * a.k >= (a.E + kWave - 1) / kWave * a.E) {
        int* s_idx = reinterpret_cast<int*>(z + a.E);
        float* s_w = z + a.E + kStepPicks;
        const float sel = wave_topk_rank(z, a.E, a.k, a.renorm, lane, s_idx, s_w, false);
        wave_lds_fence();
        if (lane < a.k) {
            p.e = s_idx[lane];
            p.w = a.renorm ? s_w[lane] / sel : s_w[lane];
        }
    } else if (a.E <= kRegsE) {
        float zr[NR];
#pragma unroll
        for (int r = 0; r < NR; ++r) zr[r] = z[min(lane + r * kWave, a.E - 1)];
        const float sel = wave_topk_regs<NR>(zr, a.E, a.k, lane, p.e, p.w);
        if (a.renorm) p.w /= sel;
    } else if (a.E <= kRankMaxE) {
        constexpr int MR = kRankMaxE / kWave;
        float zr[MR];
#pragma unroll
        for (int r = 0; r < MR; ++r) zr[r] = z[min(lane + r * kWave, a.E - 1)];
        const float sel = wave_topk_regs<MR>(zr, a.E, a.k, lane, p.e, p.w);
        if (a.renorm) p.w /= sel;
    } else {
        wave_topk(z, a.E, a.k, a.renorm, lane, p.e, p.w);
    }
    if (SLOTS && a.E <= kRegsE) {
#pragma unroll
        for (int r = 0; r < NR; ++r) {
            const int held = __shfl(slot[r], p.e & (kWave - 1));
            if (p.e >= 0 && p.e / kWave == r) p.slot = held;
        }
    } else if (SLOTS && p.e >= 0) {
        p.slot = a.slot_of_row[p.e];
    }
    return p;
}

// By the first workgroups of the reduction, kStepTailThreads threads each: the words cleared for the next step.
__device__ __forceinline__ void step_tail(const StepTail& t) {
    for (unsigned c = blockIdx.x; c < kStepCopies; c += gridDim.x)
        for (int e = threadIdx.x; e < t.E; e += kStepTailThreads) t.words[c * step_copy_words(t.E) + e] = 0ull;
}

#endif  // __HIPCC__

}  // namespace moei
