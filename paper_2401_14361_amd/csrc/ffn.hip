// Step 5 of the layer step: the activated experts' FFN as ONE streaming pass over
// their cache slots.
//
// An expert is a feed-forward network (Sec. 2 of the paper); here in SwiGLU form,
//   o = W_down ( silu(W_gate x) * (W_up x) ),  y = sum_e w_e o_e.
// At batch 1 this is one flop per weight byte, so the only thing that matters is how
// the weight bytes stream out of HBM.  A slot stores an expert row-interleaved,
//   for i in 0..I-1:  W_gate[i][0..H) | W_up[i][0..H) | W_down[0..H)[i]
// (the down projection transposed), so that everything intermediate unit i needs is
// one contiguous run of 3*H values.  A wavefront takes such a run, forms the two dot
// products with x (held in LDS as fp32), reduces them over its 64 lanes, and adds
// a_i * W_down[:, i] into a running y kept in registers: no intermediate vector ever
// leaves the CU and each weight byte is read exactly once.  Work is dealt out
// statically (unit t goes to wavefront t mod W), one workgroup per compute unit, so
// the summation order - and with it every output bit - is the same on every run.
// Workgroup partial sums are added in index order by a small second kernel.
#include <stdlib.h>
#include <string.h>

#include <algorithm>
#include <type_traits>

#include "ffn_plan.hpp"
#include "kernels.hpp"
#include "lds_limit.hpp"
#include "step_match.hpp"
#include "wtypes.hpp"

namespace moei {

namespace {

struct FfnArgs {
    const void* pool;
    size_t slot_elems;
    int n_slots_total;
    const int32_t* slot_ids;
    const float* gate_w;
    const void* x;
    float* part;  // [n_wg][H] workgroup partial sums
    int n_wg;     // workgroups that stream; the launch's others, before them, match and score (StepMatchArgs)
    int H, I, n_act;
    int waves;    // wavefronts per workgroup that stream
    int ygroup;   // wavefronts whose y rows fit in LDS together
    int32_t* flags;
    // a layer step in one launch: slots and gate weights of the n_shared first experts are known, the picks' come from `route`
    int n_shared, shared_base;
    StepMatchArgs match;
    StepRouteArgs route;
};

__device__ __forceinline__ float silu(float g) { return g / (1.0f + expf(-g)); }

// Adds the wavefronts' y rows and writes the workgroup's partial row.  LDS holds `ygroup` of them (`row` floats apart; a multiple of four,
// as H): a wavefront beyond that many adds its row to one that is there, then the rows are added up in order, four columns a
// thread.  (With a round through global memory for every `ygroup` rows a launch of 9 wavefronts and H = 5,120 took 65.3 us, now 62.0;
// H = 4,096 its end 5.1, now 2.5; of 7 and H = 2,048 1.9, now 1.1.)  `put_my_row(dst, add)` stores or adds the calling wavefront's.
template <typename Put>
__device__ __forceinline__ void block_sum_rows(float* yp, int H, int row, int waves, int ygroup, int wv, float* out, Put put_my_row) {
    const int tid = threadIdx.x, nthr = blockDim.x;
    for (int g0 = 0; g0 < waves; g0 += ygroup) {
        if (wv >= g0 && wv < min(waves, g0 + ygroup)) put_my_row(yp + (size_t)(wv - g0) * row, g0 > 0);
        barrier_lds();
    }
    const int n = min(ygroup, waves);
    for (int c = 4 * tid; c < H; c += 4 * nthr) {
        float4 s = *reinterpret_cast<const float4*>(yp + c);
        for (int k = 1; k < n; ++k) {
            const float4 v = *reinterpret_cast<const float4*>(yp + (size_t)k * row + c);
            s.x += v.x; s.y += v.y; s.z += v.z; s.w += v.w;
        }
        *reinterpret_cast<float4*>(out + c) = s;
    }
}

// Fast path: H is NCH chunks of 64 lanes x 16 bytes, so unit i is a run of 3*NCH
// 16-byte loads per lane (gate and up chunks interleaved, then the down chunks).  The
// wavefront keeps a rolling window of PF loads in flight: each step consumes the oldest
// load and issues the one PF steps ahead, across unit boundaries, so its stream never
// drains.  grid = one workgroup per compute unit, block = waves * 64 threads,
// LDS = x (NCH chunks of floats) + ygroup y rows of that length.
// TAIL: H is any multiple of 16 bytes of up to NCH chunks.  The lanes past the end of the last chunk
// read its first piece (the same for all of them) and add nothing, so a row costs what its chunks cost.
// (The kernel for any H below reads two or four bytes a lane and keeps its sums in LDS: a call of four experts of
// 910 units, H = 1,792, takes 59.6 us with it and 17.4 with this one; eight of 301, H = 2,880, 90.7 and 16.4.)
constexpr int stream_max_waves(int nch) { return nch <= 4 ? 16 : (nch <= 10 ? 12 : 8); }
template <int NCH>
struct StreamShape {
    static constexpr int kSteps = 3 * NCH;
    // window depth: all steps of a unit if they are at most 16, else half of them if that is at most 12
    // (15 loads in flight for rows of 10 chunks left no registers: 3 spills), else a third
    static constexpr int kWindow = kSteps <= 16 ? kSteps : (kSteps / 2 <= 12 && kSteps % 2 == 0 ? kSteps / 2 : kSteps / 3);
    // register budget: window + y accumulators decide how many wavefronts fit a SIMD
    static constexpr int kMaxWaves = stream_max_waves(NCH);
};

// MATCH: the launch has workgroups that match and score beside the ones that stream.  An instance of its own: the code for those
// takes 126 registers (224 at most, for rows of sixteen chunks) and spills 90 - 105 scalar ones into lanes of vector registers; launches that
// only stream take 42 - 101 for up to four chunks and spill none, so that a scan on the side stream finds room beside them.
template <typename WT, int NCH, bool TAIL, bool MATCH>
__global__ void __launch_bounds__((StreamShape<NCH>::kMaxWaves * kWave)) ffn_fused_kernel(FfnArgs a) {
    using V = WVec<WT>;
    using Raw = typename V::raw;
    constexpr int N = V::N;
    constexpr int CW = kWave * N;  // columns per chunk
    constexpr int STEPS = StreamShape<NCH>::kSteps;
    constexpr int PF = StreamShape<NCH>::kWindow;
    static_assert(STEPS % PF == 0, "the window must divide the steps of a unit");
    extern __shared__ __align__(16) float smem[];
    if constexpr (MATCH) {
        if ((int)blockIdx.x < a.match.n_blocks) {
            step_match<WT>(a.match, a.route, blockIdx.x, a.n_wg, reinterpret_cast<unsigned char*>(smem));
            return;
        }
    }
    const int blk = MATCH ? (int)blockIdx.x - a.match.n_blocks : (int)blockIdx.x;
    float* xs = smem;
    float* yp = smem + NCH * CW;
    constexpr bool kPacked = std::is_same<WT, uint16_t>::value;  // bf16: x stays bf16 in LDS, products by v_dot2c_f32_bf16
    const int tid = threadIdx.x, lane = tid & (kWave - 1);
    // the wavefront index in a scalar register: unit ids, slot ids and base addresses are
    // then scalar too
    const int wv = __builtin_amdgcn_readfirstlane(tid / kWave);
    const int H = a.H, I = a.I;
    const int W = a.n_wg * a.waves;
    const int NT = a.n_act * I;
    const WT* pool = reinterpret_cast<const WT*>(a.pool);
    const unsigned lane_off = (unsigned)lane * N;  // this lane's elements inside a chunk
    int* s_slot = reinterpret_cast<int*>(yp);      // slot ids and gate weights of the call, staged
    float* s_gate = yp + 64;                       // in LDS (the y rows are not in use before the end)
    volatile int* s_known = reinterpret_cast<int*>(yp + 128);  // MATCH: 1 once the picks' are there
    const int nthr = a.waves * kWave;              // threads that stream
    float* out = a.part + (size_t)blk * H;
    if constexpr (MATCH) {
        if (wv == a.waves) {  // the wavefront that routes
            if (lane < a.n_shared) {
                s_slot[lane] = a.shared_base + lane;
                s_gate[lane] = 1.0f;
            }
            if (lane == 0) *s_known = 0;
            float* z = yp + 192;
            const int before = a.match.n_blocks * a.waves;  // wavefronts that have rows first
            step_route_rows<WT>(a.route, before + blk, before + a.n_wg, lane);
            barrier_lds();
            const StepPick p = step_picks<WT, true>(a.route, z, lane);
            if (lane < a.route.k) {
                s_slot[a.n_shared + lane] = p.slot;
                s_gate[a.n_shared + lane] = p.w;
            }
            wait_lds_fence();
            if (lane == 0) *s_known = 1;
            __syncthreads();
            block_sum_rows(yp, H, NCH * CW, a.waves, a.ygroup, wv, out, [](float*, bool) {});
            return;
        }
    }

    auto scalar = [](size_t v) -> size_t {
        uint32_t lo = __builtin_amdgcn_readfirstlane((uint32_t)v);
        uint32_t hi = __builtin_amdgcn_readfirstlane((uint32_t)((uint64_t)v >> 32));
        return (size_t)(((uint64_t)hi << 32) | lo);
    };
    // element offset of unit t in the pool; a bad slot id reads slot 0 and is weighted by zero
    auto unit_off = [&](int slot, int i, bool& ok) -> size_t {
        ok = slot >= 0 && slot < a.n_slots_total;
        if (!ok && lane == 0) atomicOr(a.flags, 1);
        return scalar((size_t)(ok ? slot : 0) * a.slot_elems + (size_t)i * 3 * H);
    };
    // element offset of load step s inside a unit: g0 u0 g1 u1 ... then d0 d1 ...
    auto step_off = [&](int s) -> int {
        return s < 2 * NCH ? ((s & 1) ? H : 0) + (s >> 1) * CW : 2 * H + (s - 2 * NCH) * CW;
    };
    // is load step s of the last chunk, which lanes from `lanes_in` on lie past the end of?
    auto last_chunk = [](int s) { return TAIL && (s < 2 * NCH ? s >> 1 : s - 2 * NCH) == NCH - 1; };
    const bool lane_in = !TAIL || (NCH - 1) * CW + lane * N < H;
    const unsigned tail_off = lane_in ? lane_off : 0u;
    auto ld = [&](size_t unit, int s) -> Raw { return V::load_once(pool + unit + step_off(s) + (last_chunk(s) ? tail_off : lane_off)); };

    float acc[NCH * N];
#pragma unroll
    for (int k = 0; k < NCH * N; ++k) acc[k] = 0.f;
    Raw win[PF];

    // unit t -> wavefront t mod W, numbered wavefront-major (w = wv * workgroups + workgroup): when
    // the units do not fill the last round, every compute unit keeps most of its wavefronts busy
    // instead of whole workgroups running out of work
    int t = wv * a.n_wg + blk;
    float gate = 0.f, gate_n = 0.f;
    bool ok = false, ok_n = false;
    size_t p = 0;
    // A wavefront's loads complete in issue order, so what is staged into LDS is requested BEFORE the
    // first window: its data is then there after one trip to the cache, the wavefront starts on the
    // window's first load as soon as that one arrives and refills from then on.  Requested behind the
    // window it would arrive after the window's last load, and until then no refill would be issued.
    constexpr int kXRounds = (NCH + 3) / 4;  // x is NCH x 64 pieces of 16 bytes, a workgroup has at least 256 threads
    static_assert(kXRounds <= 4, "four named registers sets hold the token");
    // (named variables, not an array: an array indexed in two loops is kept in scratch memory here)
    uint4 xv0 = make_uint4(0u, 0u, 0u, 0u), xv1 = xv0, xv2 = xv0, xv3 = xv0;
    if constexpr (kPacked) {
        // a piece past the row is read as the row's last one (and not stored)
        const int n_pieces = TAIL ? H / N : NCH * kWave;
        auto piece = [&](int u) { return reinterpret_cast<const uint4*>(a.x)[min(tid + u * nthr, n_pieces - 1)]; };
        xv0 = piece(0);
        if constexpr (kXRounds > 1) xv1 = piece(1);
        if constexpr (kXRounds > 2) xv2 = piece(2);
        if constexpr (kXRounds > 3) xv3 = piece(3);
    }
    const int NS = a.n_shared * I;  // MATCH: units whose slots are known from the start
    bool known = false;
    int my_slot = 0;
    float my_gate = 0.f;
    if constexpr (!MATCH) {
        const int act = min(tid, a.n_act - 1);
        my_slot = a.slot_ids[act];
        my_gate = a.gate_w[act];
    }
    {  // the first window is on its way while x is staged.  There is one path and the wait counts stay exact: a wavefront without units reads
       // the pool's first unit instead, and in a step in one launch one whose first unit is a pick's, whose slot is not known yet, goes
       // through the zeros behind the last slot first
        if constexpr (MATCH) {
            const int e = t / I;
            if (t < NS) {
                gate = 1.0f;
                p = unit_off(a.shared_base + e, t - e * I, ok);
            } else {
                p = (size_t)a.n_slots_total * a.slot_elems;
                t -= W;  // the unit itself comes next
            }
        } else {
            const bool any = t < NT;
            const int e = any ? t / I : 0;
            const int slot0 = a.slot_ids[e];
            gate = a.gate_w[e];
            if (any) p = unit_off(slot0, t - e * I, ok);
        }
#pragma unroll
        for (int s = 0; s < PF; ++s) win[s] = ld(p, s);
    }
    if constexpr (kPacked) {
        uint4* dst = reinterpret_cast<uint4*>(xs);
        auto put = [&](int u, uint4 v) {
            const int c = tid + u * nthr;
            if (c < NCH * kWave) dst[c] = !TAIL || c * N < H ? v : make_uint4(0u, 0u, 0u, 0u);
        };
        put(0, xv0);
        if constexpr (kXRounds > 1) put(1, xv1);
        if constexpr (kXRounds > 2) put(2, xv2);
        if constexpr (kXRounds > 3) put(3, xv3);
    } else {
        for (int c = tid; c < H; c += nthr) xs[c] = V::one(reinterpret_cast<const WT*>(a.x) + c);
        if constexpr (TAIL)
            for (int c = H + tid; c < NCH * CW; c += nthr) xs[c] = 0.f;
    }
    if constexpr (!MATCH) {
        if (tid < a.n_act) {
            s_slot[tid] = my_slot;
            s_gate[tid] = my_gate;
        }
        __syncthreads();
    } else {
        barrier_lds();
    }

    while (t < NT) {
        const int tn = t + W;
        const bool more = tn < NT;
        size_t pn = p;
        if (more) {
            if constexpr (MATCH) {
                if (!known && tn >= NS) {  // (uniform; what has been requested arrives meanwhile)
                    while (__builtin_amdgcn_readfirstlane(*s_known) == 0) __builtin_amdgcn_s_sleep(1);
                    wait_lds_fence();
                    known = true;
                }
            }
            const int e = tn / I;
            pn = unit_off(s_slot[e], tn - e * I, ok_n);
            gate_n = s_gate[e];
        }
        float g = 0.f, u = 0.f, ai = 0.f;
        float xf[N];
        uint4 xp = make_uint4(0u, 0u, 0u, 0u);
#pragma unroll
        for (int s = 0; s < STEPS; ++s) {
            const Raw cur = win[s % PF];
            if (s < 2 * NCH) {
                const float before = (s & 1) == 0 ? g : u;
                if constexpr (kPacked) {
                    if ((s & 1) == 0) xp = reinterpret_cast<const uint4*>(xs)[(s >> 1) * kWave + lane];
                    if ((s & 1) == 0)
                        g = V::dot_packed(cur, xp, g);
                    else
                        u = V::dot_packed(cur, xp, u);
                } else {
                    if ((s & 1) == 0) {
#pragma unroll
                        for (int k = 0; k < N; k += 4)
                            *reinterpret_cast<float4*>(xf + k) =
                                *reinterpret_cast<const float4*>(xs + (s >> 1) * CW + lane * N + k);
                        g = V::dot(cur, xf, g);
                    } else {
                        u = V::dot(cur, xf, u);
                    }
                }
                if (last_chunk(s)) {  // a lane past the row's end adds nothing (its columns of y are never stored)
                    if ((s & 1) == 0)
                        g = lane_in ? g : before;
                    else
                        u = lane_in ? u : before;
                }
            } else {
                if (s == 2 * NCH) {
                    g = wave_sum_dpp(g);
                    u = wave_sum_dpp(u);
                    ai = ok ? silu(g) * u * gate : 0.f;
                }
                float d[N];
                V::unpack(cur, d);
#pragma unroll
                for (int k = 0; k < N; ++k)
                    acc[(s - 2 * NCH) * N + k] = __builtin_fmaf(ai, d[k], acc[(s - 2 * NCH) * N + k]);
            }
            // The consumed slot is free again: refill it with the load PF steps ahead.  After
            // the last unit the refills read the pool's first chunk (the same kilobyte for every
            // wavefront, so it comes from the cache), so that every step issues exactly one load
            // and the loop body has no branch.  The scheduling barriers keep the compiler from
            // hoisting refills and growing the window.
            __builtin_amdgcn_sched_barrier(0);
            if (s + PF < STEPS)
                win[s % PF] = ld(p, s + PF);
            else
                win[s % PF] = V::load_once(pool + (more ? pn + step_off(s + PF - STEPS) : 0) +
                                           (last_chunk(s + PF - STEPS) ? tail_off : lane_off));
            __builtin_amdgcn_sched_barrier(0);
        }
        t = tn;
        p = pn;
        gate = gate_n;
        ok = ok_n;
    }
    __syncthreads();  // the LDS behind the y rows held the slot ids until here
    block_sum_rows(yp, H, NCH * CW, a.waves, a.ygroup, wv, out, [&](float* row, bool add) {
#pragma unroll
        for (int c = 0; c < NCH; ++c)
#pragma unroll
            for (int k = 0; k < N; k += 4) {
                float4* dst = reinterpret_cast<float4*>(row + c * CW + lane * N + k);
                float4 v = make_float4(acc[c * N + k], acc[c * N + k + 1], acc[c * N + k + 2], acc[c * N + k + 3]);
                if (add) {  // uniform
                    const float4 o = *dst;
                    v.x += o.x; v.y += o.y; v.z += o.z; v.w += o.w;
                }
                *dst = v;
            }
    });
}

// Any H: the same dealing of units to wavefronts, scalar loads, y rows accumulated in LDS.
template <typename WT>
__global__ void __launch_bounds__(1024) ffn_fused_generic_kernel(FfnArgs a) {
    using V = WVec<WT>;
    extern __shared__ __align__(16) float smem[];
    float* xs = smem;
    float* yp = smem + a.H;  // [waves][H]
    const int tid = threadIdx.x, lane = tid & (kWave - 1), wv = tid / kWave;
    const int H = a.H, I = a.I;
    const int W = gridDim.x * a.waves;
    const int NT = a.n_act * I;
    const WT* pool = reinterpret_cast<const WT*>(a.pool);
    float* my = yp + (size_t)wv * H;
    stage_as_f32(reinterpret_cast<const WT*>(a.x), xs, H);
    for (int c = lane; c < H; c += kWave) my[c] = 0.f;
    __syncthreads();
    for (int t = blockIdx.x * a.waves + wv; t < NT; t += W) {
        const int e = t / I, i = t - e * I;
        const int slot = a.slot_ids[e];
        if (slot < 0 || slot >= a.n_slots_total) {
            if (lane == 0) atomicOr(a.flags, 1);
            continue;
        }
        const WT* p = pool + (size_t)slot * a.slot_elems + (size_t)i * 3 * H;
        float g = 0.f, u = 0.f;
        for (int c = lane; c < H; c += kWave) {
            g = __builtin_fmaf(V::one(p + c), xs[c], g);
            u = __builtin_fmaf(V::one(p + H + c), xs[c], u);
        }
        g = wave_sum_dpp(g);
        u = wave_sum_dpp(u);
        const float ai = silu(g) * u * a.gate_w[e];
        for (int c = lane; c < H; c += kWave) my[c] = __builtin_fmaf(ai, V::one(p + 2 * H + c), my[c]);
    }
    __syncthreads();
    float* out = a.part + (size_t)blockIdx.x * H;
    for (int c = tid; c < H; c += blockDim.x) {
        float s = 0.f;
        for (int k = 0; k < a.waves; ++k) s += yp[(size_t)k * H + c];
        out[c] = s;
    }
}

// y[h] = sum of the n_part workgroup partials.  A workgroup owns 32 columns; its 256
// threads are 8 column quads x 32 slices of the partial list; every thread adds its
// slice in index order, then the 32 slice sums are added in slice order.
__global__ void __launch_bounds__(kStepTailThreads) ffn_reduce_kernel(const float* __restrict__ part, int n_part, int H,
                                                         float* __restrict__ y, StepTail tail) {
    __shared__ float s_sum[32][32];
    if (tail.words) step_tail(tail);
    const int cq = threadIdx.x & 7, sl = threadIdx.x >> 3;
    const int h = blockIdx.x * 32 + cq * 4;
    const int per = (n_part + 31) / 32;
    const int p0 = sl * per, p1 = min(n_part, p0 + per);
    float4 acc = make_float4(0.f, 0.f, 0.f, 0.f);
    if (h + 3 < H) {
#pragma unroll 8
        for (int p = p0; p < p1; ++p) {
            const float4 v = *reinterpret_cast<const float4*>(part + (size_t)p * H + h);
            acc.x += v.x; acc.y += v.y; acc.z += v.z; acc.w += v.w;
        }
    } else {
        for (int p = p0; p < p1; ++p) {
            const float* r = part + (size_t)p * H;
            if (h < H) acc.x += r[h];
            if (h + 1 < H) acc.y += r[h + 1];
            if (h + 2 < H) acc.z += r[h + 2];
        }
    }
    s_sum[sl][cq * 4 + 0] = acc.x;
    s_sum[sl][cq * 4 + 1] = acc.y;
    s_sum[sl][cq * 4 + 2] = acc.z;
    s_sum[sl][cq * 4 + 3] = acc.w;
    __syncthreads();
    if (threadIdx.x < 32) {
        const int hh = blockIdx.x * 32 + threadIdx.x;
        float t = 0.f;
#pragma unroll
        for (int k = 0; k < 32; ++k) t += s_sum[k][threadIdx.x];
        if (hh < H) y[hh] = t;
    }
}

}  // namespace

int compute_units() {
    static int g_cus = 0;
    if (g_cus == 0) {
        int dev = 0, n = 0;
        if (hipGetDevice(&dev) != hipSuccess ||
            hipDeviceGetAttribute(&n, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess || n <= 0)
            n = 256;
        g_cus = n;
    }
    return g_cus;
}

namespace {

int env_int(const char* name, int dflt) {
    const char* v = getenv(name);
    if (!v || !*v) return dflt;
    return atoi(v);
}


constexpr size_t kLdsBudget = 150 * 1024;  // of the 160 KiB per compute unit

int forced_waves() {
    static const int forced = env_int("MOEI_FFN_WAVES", 0);  // the environment is read once per process
    return forced;
}

// Wavefronts per workgroup that stream, and of those that match that scan, in a step in one launch with rows of `nch` chunks.
int step_waves(int n_units, int blocks, int nch) {
    const int most = stream_max_waves(nch) - 1;
    return plan_waves(n_units, blocks, most, kMatchWaves - 1, std::min(forced_waves(), most));
}

// Raises a kernel's dynamic-LDS limit above 64 KiB, once per kernel and size (the call
// is not a stream operation, so it stays out of the per-launch path and of captures).
template <typename K>
int allow_big_lds(K kernel, size_t bytes) {
    static LdsLimits<128> limits;  // kernels of one argument type: 104 streaming FFNs are the most
    if (bytes <= 64 * 1024) return MOEI_OK;
    const void* fn = reinterpret_cast<const void*>(kernel);
    return limits.at_least(fn, bytes, [&]() -> int {
        MOEI_HIP(hipFuncSetAttribute(fn, hipFuncAttributeMaxDynamicSharedMemorySize, (int)bytes));
        return MOEI_OK;
    });
}

template <typename WT>
int launch_ffn_typed(FfnArgs a, bool fast, int grid, size_t match_lds, const StepTail& tail, float* d_y, hipStream_t s) {
    using V = WVec<WT>;
    const int H = a.H;
    int rc = MOEI_OK;
    const int nch = (H + kWave * V::N - 1) / (kWave * V::N);
    const size_t row = (size_t)H * sizeof(float);
    if (fast) {
#define MOEI_FFN_CASE(N_, TAIL_)                                                                        \
    case N_: {                                                                                         \
        const bool step = a.match.n_blocks > 0; /* one wavefront more than stream */                   \
        a.waves = step ? step_waves(a.n_act * a.I, grid, N_)                                           \
                       : plan_waves(a.n_act * a.I, grid, StreamShape<N_>::kMaxWaves, 4, forced_waves()); \
        static_assert(StreamShape<N_>::kMaxWaves >= kMatchWaves, "the match finds its wavefronts");    \
        const size_t padded = (size_t)N_ * kWave * V::N * sizeof(float);                               \
        int yg = (int)((kLdsBudget - padded) / padded);                                                \
        a.ygroup = yg < 1 ? 1 : (yg > a.waves ? a.waves : yg);                                         \
        const size_t smem = std::max({padded * (1 + a.ygroup), match_lds, step ? padded + 192 * 4 + step_route_lds(a.route.E) : 0}); \
        if (step) step_scan_plan(&a.match, a.waves);                                                   \
        auto kernel = step ? ffn_fused_kernel<WT, N_, TAIL_, true> : ffn_fused_kernel<WT, N_, TAIL_, false>; \
        rc = allow_big_lds(kernel, smem);                                                              \
        if (rc) return rc;                                                                             \
        launch(K_FFN_FUSED, kernel, dim3(grid + a.match.n_blocks), dim3((a.waves + step) * kWave), smem, s, a); \
        break;                                                                                         \
    }
        // whole chunks, for the counts of chunks that configurations have; any other row through TAIL
        const int whole = H % (kWave * V::N) == 0 ? nch : 0;
        switch (whole) {
            MOEI_FFN_CASE(1, false)
            MOEI_FFN_CASE(2, false)
            MOEI_FFN_CASE(3, false)
            MOEI_FFN_CASE(4, false)
            MOEI_FFN_CASE(5, false)
            MOEI_FFN_CASE(6, false)
            MOEI_FFN_CASE(8, false)
            MOEI_FFN_CASE(10, false)
            MOEI_FFN_CASE(12, false)
            MOEI_FFN_CASE(16, false)
            default:
                switch ((uintptr_t)a.x % 16 == 0 ? nch : 0) {
                    MOEI_FFN_CASE(1, true)
                    MOEI_FFN_CASE(2, true)
                    MOEI_FFN_CASE(3, true)
                    MOEI_FFN_CASE(4, true)
                    MOEI_FFN_CASE(5, true)
                    MOEI_FFN_CASE(6, true)
                    MOEI_FFN_CASE(7, true)
                    MOEI_FFN_CASE(8, true)
                    MOEI_FFN_CASE(9, true)
                    MOEI_FFN_CASE(10, true)
                    MOEI_FFN_CASE(11, true)
                    MOEI_FFN_CASE(12, true)
                    MOEI_FFN_CASE(13, true)
                    MOEI_FFN_CASE(14, true)
                    MOEI_FFN_CASE(15, true)
                    MOEI_FFN_CASE(16, true)
                    default:
                        fast = false;
                }
        }
#undef MOEI_FFN_CASE
    }
    if (!fast) {
        if (a.match.n_blocks > 0) MOEI_FAIL(MOEI_EINVAL, "expert FFN: H = %d takes no match beside it", H);
        int m = (int)((kLdsBudget - row) / row);
        if (m > 8) m = 8;
        if (m < 1) MOEI_FAIL(MOEI_ECAPACITY, "expert_ffn_gemv: H = %d does not fit the LDS staging", H);
        a.waves = m;
        a.ygroup = m;
        const size_t smem = row * (1 + m);
        rc = allow_big_lds(ffn_fused_generic_kernel<WT>, smem);
        if (rc) return rc;
        launch(K_FFN_FUSED, ffn_fused_generic_kernel<WT>, dim3(grid), dim3(m * kWave), smem, s, a);
    }
    MOEI_LAUNCH_CHECK();
    launch(K_FFN_REDUCE, ffn_reduce_kernel, dim3((H + 31) / 32), dim3(256), 0, s, (const float*)a.part, grid, H, d_y, tail);
    MOEI_LAUNCH_CHECK();
    return MOEI_OK;
}


// ------------------------------------------------------------------ decode batch B > 1
// Tokens are grouped per activated expert; an "item" is one expert with up to kMaxGroup of its
// tokens, so the expert's weights are streamed once per item.  The items' intermediate units
// are split evenly over the workgroups as contiguous ranges.  A wavefront streams a unit once
// and uses it for every token of the item; y accumulators exist per token.
constexpr int kMaxGroup = 4;
constexpr int kGroupedWaves = 8;
constexpr int kMaxBatch = 16;

struct GroupItem {
    int32_t slot;
    int32_t ntok;
    int32_t tok[kMaxGroup];
    float w[kMaxGroup];
};

struct GroupArgs {
    const int32_t* idx;          // [B][k] picks
    const float* w;              // [B][k] gate weights
    const int32_t* slot_of_row;  // slot_of + layer*E
    int B, k, E, n_shared, shared_base, tb;
    void* items;  // GroupItem or GmItemOut
    int32_t* n_items;
    int32_t* flags;
};

// The item list of a call, built by every workgroup for itself (the picks of a batch are a few
// hundred bytes, the list a few kilobytes of LDS; a launch of its own would cost more than all
// workgroups repeating it).  The tokens routed to an expert, in token order, are cut into items of
// at most tb tokens; item positions follow expert order, the shared experts last.  The work is
// spread over the picks: the thread of pick p counts the earlier picks of the same expert (its
// rank there), LDS counters give every expert its number of tokens, a scan over the experts gives
// each its first item, and the thread then writes its token into place.  All threads of the
// workgroup call (at least 256 of them); with `publish` the list also goes to global memory for
// the reduction kernel and a pick that is not resident raises its flag.  Returns the item count
// (in every thread).  E <= 256 (checked by the host).
struct ItemScratch {
    int cnt[256];    // tokens routed to the expert
    int start[256];  // its first item
    int slot[256];   // its slot, -1: not resident
    int wsum[4];
};

__device__ __forceinline__ int build_items(const GroupArgs& a, GroupItem* s_items, int* s_pick, ItemScratch* sc,
                                           bool publish) {
    const int tid = threadIdx.x, lane = tid & (kWave - 1), wv = tid / kWave;
    const int n_pick = a.B * a.k;
    float* s_pickw = reinterpret_cast<float*>(s_pick + n_pick);
    const int row_slot = tid < a.E ? a.slot_of_row[tid] : -1;  // on its way with the picks
    for (int p = tid; p < n_pick; p += blockDim.x) {
        int e = a.idx[p];
        if (e < 0 || e >= a.E) e = -1;  // a token without picks (no softmax exists for its logits)
        s_pick[p] = e;
        s_pickw[p] = a.w[p];
    }
    if (tid < 256) sc->cnt[tid] = 0;
    __syncthreads();
    // rank of every pick among the picks of its expert; tokens per expert
    int my_rank[2] = {0, 0};  // a thread takes at most two picks (16 tokens x k picks over >= 256 threads)
    int my_n = 0;
    for (int p = tid; p < n_pick && my_n < 2; p += blockDim.x, ++my_n) {
        const int e = s_pick[p];
        int r = 0;  // four picks per LDS read (the weights behind the picks make the last read safe)
        for (int q = 0; q < p; q += 4) {
            const int4 v = *reinterpret_cast<const int4*>(s_pick + q);
            r += (v.x == e) + ((q + 1 < p) & (v.y == e)) + ((q + 2 < p) & (v.z == e)) + ((q + 3 < p) & (v.w == e));
        }
        my_rank[my_n] = r;
        if (e >= 0) atomicAdd(&sc->cnt[e], 1);
    }
    __syncthreads();
    // items per expert, scanned over the experts
    int mine = 0;
    if (tid < 256) {
        int slot = -1, ntok = tid < a.E ? sc->cnt[tid] : 0;
        if (ntok > 0) {
            slot = row_slot;
            if (slot < 0) {  // not resident: contributes nothing, flagged
                if (publish) atomicOr(a.flags, 2);
                ntok = 0;
            }
        }
        sc->slot[tid] = slot;
        mine = (ntok + a.tb - 1) / a.tb;
    }
    int incl = mine;
#pragma unroll
    for (int off = 1; off < kWave; off <<= 1) {
        const int up = __shfl_up(incl, off, kWave);
        if (lane >= off) incl += up;
    }
    if (lane == kWave - 1 && wv < 4) sc->wsum[wv] = incl;
    __syncthreads();
    if (tid < 256) {
        int before = 0;
        for (int w = 0; w < wv; ++w) before += sc->wsum[w];
        sc->start[tid] = before + incl - mine;
    }
    int n = sc->wsum[0] + sc->wsum[1] + sc->wsum[2] + sc->wsum[3];
    __syncthreads();
    // every pick writes its token into its item; the first of an item also writes the item's head
    my_n = 0;
    for (int p = tid; p < n_pick && my_n < 2; p += blockDim.x, ++my_n) {
        const int e = s_pick[p];
        if (e < 0 || sc->slot[e] < 0) continue;
        const int r = my_rank[my_n];
        GroupItem* it = s_items + sc->start[e] + r / a.tb;
        const int pos = r % a.tb;
        it->tok[pos] = p / a.k;
        it->w[pos] = s_pickw[p];
        if (pos == 0) {
            const int ntok = min(a.tb, sc->cnt[e] - r);
            it->slot = sc->slot[e];
            it->ntok = ntok;
            for (int j = ntok; j < kMaxGroup; ++j) {
                it->tok[j] = 0;
                it->w[j] = 0.f;
            }
        }
    }
    const int tiles = (a.B + a.tb - 1) / a.tb;
    for (int q = tid; q < a.n_shared * tiles; q += blockDim.x) {
        const int sh = q / tiles, t0 = (q - sh * tiles) * a.tb;
        GroupItem it;
        it.slot = a.shared_base + sh;
        it.ntok = min(a.tb, a.B - t0);
        for (int j = 0; j < kMaxGroup; ++j) {
            it.tok[j] = j < it.ntok ? t0 + j : 0;
            it.w[j] = j < it.ntok ? 1.0f : 0.f;
        }
        s_items[n + q] = it;
    }
    n += a.n_shared * tiles;
    __syncthreads();
    if (publish) {
        for (int q = tid; q < n; q += blockDim.x) reinterpret_cast<GroupItem*>(a.items)[q] = s_items[q];
        if (tid == 0) *a.n_items = n;
    }
    return n;
}

struct GroupedFfnArgs {
    const void* pool;
    size_t slot_elems;
    GroupArgs grp;   // picks, gate weights, slot row; the item list goes to grp.items / grp.n_items
    int max_items;   // room in the LDS item list
    const void* x;  // [B][H]
    float* part;    // [workgroups][seg_max][TB][H]
    int H, I;
    int cost;  // rows that an item's start counts for
    int seg_max;
};

template <int NCH>
struct GroupedShape {
    static constexpr int kTB = NCH <= 4 ? 4 : 1;  // y accumulators per token must fit the register file
};

// The activated items' intermediate units form one row space of n_items * (I + cost) rows, the first
// `cost` of an item standing for what its start costs a workgroup (the window drains, the partial rows of
// the item before are added up, the inputs are staged, the window fills: about as long as 180 KB of
// weights take); workgroup g takes the contiguous range [total*g/G, total*(g+1)/G).  A range crosses at
// most ceil(n_items / G) item boundaries, so it is cut into at most that many + 1 segments, each
// inside one item; a segment yields one partial y row per token of the item.
// (With even shares of the units alone the workgroups that change items ended last.  A call of 2 / 3 / 4 / 8 requests of
// the 64-expert shape (1,408 units, two shared experts) took 49.8 / 65.9 / 81.8 / 125.7 us, now 48.5 / 63.9 / 80.2 / 124.1; of
// sixteen, 54 items that leave few workgroups in one of them alone, 181.8 either way.  Shorter items gain more: 1 / 3 / 8 / 16
// requests of 32 experts of 700 units, H = 1,024, 17.3 / 23.1 / 35.6 / 42.7 and 14.9 / 21.0 / 32.0 / 40.0.)
// Where the items divide the workgroups nobody changes items and every share is the same as it is: there a
// start counts nothing (one request, 8 items: 34.4 us with it, 33.5 without).
// (32 bits hold it: a pool of 16 (k + n_shared) x I < 2^31 units of at least 3 KB is 400 GB.  A 64-bit division is some 150
// instructions, and a workgroup makes five before its first load.)
__device__ __forceinline__ int grouped_range_begin(int total, int g, int G) {  // total * g / G
    const int q = total / G, r = total - q * G;
    return q * g + r * g / G;
}
__host__ inline int grouped_cost(int H, int wb) { return (180 * 1024 + 3 * H * wb - 1) / (3 * H * wb); }
__device__ __forceinline__ int grouped_start(int n_items, int G, int cost) {
    return n_items > 0 && G % n_items == 0 ? 0 : cost;
}
// The next segment of a range: rows r0 .. r1 of `item` (none: r0 == r1); *row moves past it.
__device__ __forceinline__ void grouped_segment(int* row, int end, int I, int cost, int* item, int* r0, int* r1) {
    *item = *row / (I + cost);
    const int c0 = *row - *item * (I + cost);
    const int c1 = min(I + cost, c0 + (end - *row));
    *row += c1 - c0;
    *r0 = max(0, c0 - cost);
    *r1 = max(0, c1 - cost);
}

__host__ inline int grouped_seg_max(int max_items, int G) { return (max_items + G - 1) / G + 1; }

template <typename WT, int NCH>
__global__ void __launch_bounds__((kGroupedWaves * kWave)) ffn_grouped_kernel(GroupedFfnArgs a) {
    using V = WVec<WT>;
    using Raw = typename V::raw;
    constexpr int N = V::N;
    constexpr int CW = kWave * N;
    constexpr int TB = GroupedShape<NCH>::kTB;
    constexpr int STEPS = StreamShape<NCH>::kSteps;
    constexpr int PF = StreamShape<NCH>::kWindow;
    extern __shared__ __align__(16) float smem[];
    __shared__ ItemScratch s_is;
    // [TB][H] inputs of the item's tokens: fp32 for fp32 weights; for bf16 weights the stored bf16 values
    // themselves, in the first half of each row, for the two-element dot products
    constexpr bool kPacked = std::is_same<WT, uint16_t>::value;
    float* xs = smem;
    float* yp = smem + TB * a.H;   // [kGroupedWaves][H] y rows of one token, one per wavefront
    GroupItem* s_items = reinterpret_cast<GroupItem*>(yp + (size_t)kGroupedWaves * a.H);  // [max_items]
    const int tid = threadIdx.x, lane = tid & (kWave - 1);
    const int wv = __builtin_amdgcn_readfirstlane(tid / kWave);
    const int H = a.H, I = a.I;
    const WT* pool = reinterpret_cast<const WT*>(a.pool);
    const unsigned lane_off = (unsigned)lane * N;
    int* s_pick = reinterpret_cast<int*>(s_items + a.max_items);  // [2][B*k]
    const int n_items = build_items(a.grp, s_items, s_pick, &s_is, blockIdx.x == 0);
    const int cost = grouped_start(n_items, gridDim.x, a.cost);
    const int total = n_items * (I + cost);
    const int R0 = grouped_range_begin(total, blockIdx.x, gridDim.x);
    const int R1 = grouped_range_begin(total, blockIdx.x + 1, gridDim.x);
    auto scalar = [](size_t v) -> size_t {
        uint32_t lo = __builtin_amdgcn_readfirstlane((uint32_t)v);
        uint32_t hi = __builtin_amdgcn_readfirstlane((uint32_t)((uint64_t)v >> 32));
        return (size_t)(((uint64_t)hi << 32) | lo);
    };
    auto step_off = [&](int s) -> int {
        return s < 2 * NCH ? ((s & 1) ? H : 0) + (s >> 1) * CW : 2 * H + (s - 2 * NCH) * CW;
    };
    auto ld = [&](size_t unit, int off) -> Raw { return V::load_once(pool + unit + off + lane_off); };

    int seg = 0;
    for (int row = R0; row < R1 && seg < a.seg_max; ++seg) {  // uniform over the workgroup
        int item, r0, r1;
        grouped_segment(&row, R1, I, cost, &item, &r0, &r1);
        if (r0 == r1) continue;
        const GroupItem it = s_items[item];
        // this wavefront's rows of the segment: r0 + wv, r0 + wv + 8, ...
        const int nr = (r1 - r0 - wv + kGroupedWaves - 1) / kGroupedWaves;  // may be <= 0
        const size_t row_stride = (size_t)kGroupedWaves * 3 * H;
        size_t p = scalar((size_t)it.slot * a.slot_elems + (size_t)(r0 + wv) * 3 * H);
        Raw win[PF];
        if (nr > 0) {  // the first window is on its way while the inputs are staged
#pragma unroll
            for (int s = 0; s < PF; ++s) win[s] = ld(p, step_off(s));
        }
        __syncthreads();  // the previous segment is done with xs and yp
        for (int j = 0; j < TB; ++j)
            if (j < it.ntok) {
                const WT* xsrc = reinterpret_cast<const WT*>(a.x) + (size_t)it.tok[j] * H;
                if constexpr (kPacked) {
                    uint4* dst = reinterpret_cast<uint4*>(xs + (size_t)j * H);
                    for (int c = tid; c < H / 8; c += kGroupedWaves * kWave) dst[c] = *reinterpret_cast<const uint4*>(xsrc + c * 8);
                } else {
                    stage_as_f32(xsrc, xs + (size_t)j * H, H);
                }
            }
        __syncthreads();
        float acc[TB][NCH * N];
#pragma unroll
        for (int j = 0; j < TB; ++j)
#pragma unroll
            for (int q = 0; q < NCH * N; ++q) acc[j][q] = 0.f;
        for (int r = 0; r < nr; ++r) {
            const bool more = r + 1 < nr;
            const size_t pn = more ? p + row_stride : p;
            float gs[TB], us[TB], ai[TB];
#pragma unroll
            for (int j = 0; j < TB; ++j) gs[j] = us[j] = ai[j] = 0.f;
#pragma unroll
            for (int s = 0; s < STEPS; ++s) {
                const Raw cur = win[s % PF];
                if (s < 2 * NCH) {
#pragma unroll
                    for (int j = 0; j < TB; ++j) {
                        if (j < it.ntok) {  // uniform
                            if constexpr (kPacked) {
                                const uint4 xp = reinterpret_cast<const uint4*>(xs + (size_t)j * H)[(s >> 1) * kWave + lane];
                                if ((s & 1) == 0)
                                    gs[j] = V::dot_packed(cur, xp, gs[j]);
                                else
                                    us[j] = V::dot_packed(cur, xp, us[j]);
                            } else {
                                float xf[N];
#pragma unroll
                                for (int t = 0; t < N; t += 4)
                                    *reinterpret_cast<float4*>(xf + t) = *reinterpret_cast<const float4*>(
                                        xs + (size_t)j * H + (s >> 1) * CW + lane * N + t);
                                if ((s & 1) == 0)
                                    gs[j] = V::dot(cur, xf, gs[j]);
                                else
                                    us[j] = V::dot(cur, xf, us[j]);
                            }
                        }
                    }
                } else {
                    if (s == 2 * NCH) {
#pragma unroll
                        for (int j = 0; j < TB; ++j)
                            if (j < it.ntok) ai[j] = silu(wave_sum_dpp(gs[j])) * wave_sum_dpp(us[j]) * it.w[j];
                    }
                    float df[N];
                    V::unpack(cur, df);
#pragma unroll
                    for (int j = 0; j < TB; ++j)
#pragma unroll
                        for (int t = 0; t < N; ++t)
                            acc[j][(s - 2 * NCH) * N + t] = __builtin_fmaf(ai[j], df[t], acc[j][(s - 2 * NCH) * N + t]);
                }
                __builtin_amdgcn_sched_barrier(0);
                if (s + PF < STEPS)
                    win[s % PF] = ld(p, step_off(s + PF));
                else
                    win[s % PF] = ld(more ? pn : 0, more ? step_off(s + PF - STEPS) : 0);
                __builtin_amdgcn_sched_barrier(0);
            }
            p = pn;
        }
        // the segment's partial row of every token of the item: wavefront rows added in order
#pragma unroll
        for (int j = 0; j < TB; ++j) {
            if (j < it.ntok) {  // uniform
                __syncthreads();
                float* rowp = yp + (size_t)wv * H;
#pragma unroll
                for (int q = 0; q < NCH; ++q)
#pragma unroll
                    for (int t = 0; t < N; t += 4)
                        *reinterpret_cast<float4*>(rowp + q * CW + lane * N + t) =
                            make_float4(acc[j][q * N + t], acc[j][q * N + t + 1], acc[j][q * N + t + 2],
                                        acc[j][q * N + t + 3]);
                __syncthreads();
                float* out = a.part + (((size_t)blockIdx.x * a.seg_max + seg) * TB + j) * H;
                for (int h = tid; h < H; h += kGroupedWaves * kWave) {
                    float s = 0.f;
#pragma unroll
                    for (int k = 0; k < kGroupedWaves; ++k) s += yp[(size_t)k * H + h];
                    out[h] = s;
                }
            }
        }
    }
}

// ---- the same for bf16 weights on the matrix cores: an item is one expert with up to 16 of its picks, so a call streams every
// activated expert once (the shared ones too), whatever the batch.
//
// grid: a workgroup of eight wavefronts per compute unit.  Its range of the items' units is cut into blocks of 16 units, and
// wavefront w has columns w * HW .. + HW (HW = H / 8) of all three matrices: for gate and up its share of the sum over
// the columns (D = A B, A = 16 units x 32 columns, B = 32 columns x 16 tokens, bf16 products added in fp32), which eight
// partial tiles in LDS are added up in wavefront order; for down those columns of y, whose sums stay in its registers
// from an item's first block to its last.  The activations stay fp32: the down product runs on the fp32 matrix instruction (A =
// 16 tokens x 4 units, B = 4 units x 16 columns), which lets a lane use the eight columns of one 16-byte piece as the same column of
// eight tiles, so nothing is transposed; its rate is a quarter of what would hold the stream up.
// The weights go from global memory straight into a ring of two stages per wavefront (16 rows of the wavefront's columns; four of 128
// columns for rows of 4,096; no barrier, the waits are counted), the token rows of an item through the same ring before its first block.  The ring runs on across
// blocks and items: a block's down rows come behind the next block's gate and up rows, so that the exchange of the
// partial tiles (two barriers that wait for LDS only) does not hold it up, and what an item's end costs is the store of its rows.
// Bound by the stream: sixteen requests of the 64-expert shape 162 us a call, 865 MB at 5.7 TB/s between start and end; with
// items of four tokens in registers (the kernel above: the shared experts pass four times, and at a segment's end the window
// drains and eight rows a token are added through LDS) 190.  Nothing on the way waits for the whole ring: with sums in private memory
// and the exchange's lane address there too, 8 experts of 6,000 units, H = 4,096, 8 / 16 requests took 207 / 234 us, now 190 / 217.  Loads without the non-temporal hint took 12 % longer, stages of 128
// columns, four in the ring, 1 %.
// Rounding: sums run as several short chains (a chain per matrix instruction of a stage, two per block and down tile, a block's sum
// added to those before it), so that the error against 64 bits is that of the kernel above or less: relative 2-norm 1.6 - 2.0e-7, there
// 1.6 - 2.1e-7; with one chain for the columns of a wavefront and one for an item's units it was 3.3e-7.
constexpr int kGmTokens = 16;
constexpr int kGmUnits = 16;  // of a block
constexpr int kGmMaxSegs = 16;
typedef float gm_f32x4 __attribute__((ext_vector_type(4)));
typedef __bf16 gm_bf16x8 __attribute__((ext_vector_type(8)));

struct GmItem {   // in LDS
    int slot, first, ntok;  // its picks are entries first .. + ntok of the sorted list
};
struct GmItemOut {  // for the reduction: token j in bits 4 j .. + 4
    int32_t slot, ntok;
    unsigned long long toks;
};
struct GmSeg {
    int item, r0, r1;
};

struct GroupedMmArgs {
    const uint16_t* pool;
    size_t slot_elems;
    GroupArgs grp;  // items / n_items: GmItemOut
    int max_items, n_list;  // room in LDS: items, entries of the sorted list
    const uint16_t* x;      // [B][H]
    float* part;            // [workgroups][seg_max][kGmTokens][H]
    int H, I, cost, seg_max;
};

template <int HW>
struct GmShape {
    static constexpr int kCols = HW == 512 ? 128 : HW;  // of a stage (256 need registers that rows of 4,096 don't leave)
    static constexpr int kStages = HW / kCols;          // per matrix and block
    static constexpr bool kKeepX = HW != 512;           // the tokens of an item stay in registers, else they pass with every block
    static constexpr int kRing = HW == 512 ? 4 : 2;     // stages
    static constexpr int kStageBytes = kGmUnits * kCols * 2;
    static constexpr int kLoads = kStageBytes / 1024;
};
constexpr size_t kGmPartBytes = (size_t)kGroupedWaves * 2 * 256 * 4;
constexpr size_t kGmActBytes = (size_t)2 * 256 * 4;

template <int HW>
size_t gm_lds(int max_items, int n_list) {
    return (size_t)kGroupedWaves * GmShape<HW>::kRing * GmShape<HW>::kStageBytes + kGmPartBytes + kGmActBytes +
           (((size_t)n_list * 8 + (size_t)max_items * sizeof(GmItem) + 15) & ~(size_t)15);
}

// The item list of a call, as build_items forms it, with the picks sorted by expert (and by token within one) in a list of
// their own: s_tok / s_w, behind them the tokens 0 .. B - 1 with weight 1 for the shared experts.  `scratch` is free afterwards.
__device__ __forceinline__ int gm_build_items(const GroupArgs& a, GmItem* s_items, int* s_tok, float* s_w, unsigned char* scratch,
                                              bool publish) {
    ItemScratch* sc = reinterpret_cast<ItemScratch*>(scratch);
    int* s_pick = reinterpret_cast<int*>(scratch + ((sizeof(ItemScratch) + 15) & ~(size_t)15));
    int* s_first = s_pick + 512;  // [256] the expert's first entry of the list
    const int tid = threadIdx.x, lane = tid & (kWave - 1), wv = tid / kWave;
    const int n_pick = a.B * a.k;  // at most 512, one per thread
    const int row_slot = tid < a.E ? a.slot_of_row[tid] : -1;
    int my_e = -1;
    float my_w = 0.f;
    if (tid < n_pick) {
        my_e = a.idx[tid];
        my_w = a.w[tid];
        if (my_e < 0 || my_e >= a.E) my_e = -1;  // a token without picks (no softmax exists for its logits)
    }
    s_pick[tid] = my_e;
    if (tid < 256) sc->cnt[tid] = 0;
    __syncthreads();
    int rank = 0;
    if (tid < n_pick) {
        for (int q = 0; q < tid; q += 4) {
            const int4 v = *reinterpret_cast<const int4*>(s_pick + q);
            rank += (v.x == my_e) + ((q + 1 < tid) & (v.y == my_e)) + ((q + 2 < tid) & (v.z == my_e)) + ((q + 3 < tid) & (v.w == my_e));
        }
        if (my_e >= 0) atomicAdd(&sc->cnt[my_e], 1);
    }
    __syncthreads();
    // items and list entries per expert, both scanned over the experts (at most 512 each: one word)
    int ntok = tid < a.E ? sc->cnt[tid & 255] : 0;
    if (ntok > 0 && row_slot < 0) {  // not resident: contributes nothing, flagged
        if (publish) atomicOr(a.flags, 2);
        ntok = 0;
    }
    const int n_mine = (ntok + kGmTokens - 1) / kGmTokens;
    const int mine = n_mine << 16 | ntok;
    int incl = mine;
#pragma unroll
    for (int off = 1; off < kWave; off <<= 1) {
        const int up = __shfl_up(incl, off, kWave);
        if (lane >= off) incl += up;
    }
    if (lane == kWave - 1 && wv < 4) sc->wsum[wv] = incl;
    __syncthreads();
    const int total = sc->wsum[0] + sc->wsum[1] + sc->wsum[2] + sc->wsum[3];
    const int n_list = total & 0xffff;
    int n = total >> 16;
    if (tid < 256) {
        int before = incl - mine;
        for (int w = 0; w < wv; ++w) before += sc->wsum[w];
        s_first[tid] = before & 0xffff;
        sc->slot[tid] = ntok > 0 ? row_slot : -1;
        for (int i = 0; i < n_mine; ++i)
            s_items[(before >> 16) + i] = GmItem{row_slot, (before & 0xffff) + i * kGmTokens, min(kGmTokens, ntok - i * kGmTokens)};
    }
    __syncthreads();
    if (my_e >= 0 && sc->slot[my_e] >= 0) {
        const int at = s_first[my_e] + rank;
        s_tok[at] = tid / a.k;
        s_w[at] = my_w;
    }
    if (tid < a.B) {
        s_tok[n_list + tid] = tid;
        s_w[n_list + tid] = 1.0f;
    }
    for (int q = tid; q < a.n_shared; q += blockDim.x) s_items[n + q] = GmItem{a.shared_base + q, n_list, a.B};
    n += a.n_shared;
    __syncthreads();
    if (publish) {
        GmItemOut* out = reinterpret_cast<GmItemOut*>(a.items);
        for (int q = tid; q < n; q += blockDim.x) {
            const GmItem it = s_items[q];
            unsigned long long toks = 0;
            for (int j = 0; j < it.ntok; ++j) toks |= (unsigned long long)s_tok[it.first + j] << (4 * j);
            out[q] = GmItemOut{it.slot, it.ntok, toks};
        }
        if (tid == 0) *a.n_items = n;
    }
    return n;
}

template <int HW>
__global__ void __launch_bounds__((kGroupedWaves * kWave), 2) ffn_grouped_mm_kernel(GroupedMmArgs a) {
    using S = GmShape<HW>;
    constexpr int H = HW * kGroupedWaves;
    constexpr int RB = S::kCols * 2;       // bytes of a stage's row
    constexpr int CH = RB / 16;            // its 16-byte pieces: 8 to 32
    constexpr int KS = S::kCols / 32;      // matrix instructions per gate or up stage
    constexpr int CPL = S::kCols >= 128 ? 8 : 4;  // columns per lane of a group of 16 CPL columns
    constexpr int GR = S::kCols / (16 * CPL);     // such groups in a stage
    extern __shared__ __align__(16) float smem[];
    __shared__ GmSeg s_seg[kGmMaxSegs];
    unsigned char* ring0 = reinterpret_cast<unsigned char*>(smem);
    float* s_part = reinterpret_cast<float*>(ring0 + (size_t)kGroupedWaves * S::kRing * S::kStageBytes);  // [wavefront][gate, up][256]
    float* s_act = s_part + kGroupedWaves * 2 * 256;  // [2][unit][token]
    int* s_tok = reinterpret_cast<int*>(s_act + 2 * 256);
    float* s_w = reinterpret_cast<float*>(s_tok + a.n_list);
    GmItem* s_items = reinterpret_cast<GmItem*>(s_w + a.n_list);
    const int tid = threadIdx.x, lane = tid & (kWave - 1);
    const int wv = __builtin_amdgcn_readfirstlane(tid / kWave);
    const int I = a.I;
    const int n_items = gm_build_items(a.grp, s_items, s_tok, s_w, reinterpret_cast<unsigned char*>(s_part), blockIdx.x == 0);
    int n_seg = 0, n_blocks = 0;
    {  // the workgroup's segments (the empty ones keep their number: the reduction counts them too)
        const int cost = grouped_start(n_items, gridDim.x, a.cost);
        const int total = n_items * (I + cost);
        int row = grouped_range_begin(total, blockIdx.x, gridDim.x);
        const int R1 = grouped_range_begin(total, blockIdx.x + 1, gridDim.x);
        for (; row < R1 && n_seg < a.seg_max; ++n_seg) {
            GmSeg sg;
            grouped_segment(&row, R1, I, cost, &sg.item, &sg.r0, &sg.r1);
            if (tid == 0) s_seg[n_seg] = sg;
            n_blocks += (sg.r1 - sg.r0 + kGmUnits - 1) / kGmUnits;
        }
    }
    __syncthreads();
    if (n_blocks == 0) return;

    // One block of 16 units (the last of a segment may have fewer), as both the loads and the products walk through them.
    struct Block {
        const unsigned char* base;  // gate row of its first unit, this wavefront's first column
        int seg, row, valid, first_tok, ntok;
        bool first, last;  // of its segment
    };
    auto uniform = [](int v) { return __builtin_amdgcn_readfirstlane(v); };
    auto block_at = [&](Block& b, int seg, int row) {  // the block at `row` of segment `seg`, or of the next one that has rows
        int r0 = uniform(s_seg[seg].r0), r1 = uniform(s_seg[seg].r1);
        if (row < 0) row = r0;
        while (row >= r1) {  // (the caller knows that there is a block)
            ++seg;
            row = r0 = uniform(s_seg[seg].r0);
            r1 = uniform(s_seg[seg].r1);
        }
        const GmItem* it = s_items + uniform(s_seg[seg].item);
        b.seg = seg;
        b.row = row;
        b.first = row == r0;
        b.last = row + kGmUnits >= r1;
        b.valid = min(kGmUnits, r1 - row);
        b.first_tok = uniform(it->first);
        b.ntok = uniform(it->ntok);
        b.base = reinterpret_cast<const unsigned char*>(a.pool) + ((size_t)uniform(it->slot) * a.slot_elems + (size_t)row * 3 * H + wv * HW) * 2;
    };

    // ---- the ring's loads.  Piece p of row r of a stage lies at place p ^ r of the row (no bank conflicts in the reads below).
    const uint32_t my_ring = lds_address(ring0) + (uint32_t)wv * (S::kRing * S::kStageBytes);
    constexpr int RPL = 1024 / RB;  // rows per load
    // byte offset of this lane's piece in load i of a stage whose rows lie `stride` bytes apart, rows past `rows` repeating the last.
    // (Formed anew at each load: kept across the loop, these offsets push the sums of rows of 4,096 out of the registers.)
    auto opaque = [](int v) {
        asm volatile("" : "+v"(v));
        return v;
    };
    auto row_of = [&](int lv, int i, int rows) { return min(i * RPL + lv / CH, rows - 1); };
    auto piece_of = [&](int lv, int i) { return (uint32_t)(((lv % CH) ^ ((i * RPL + lv / CH) & (CH - 1))) * 16); };
    Block ib, ip;        // the block whose gate and up rows are loaded now, and the one before it (its down rows follow)
    bool have_b = true, have_p = false;
    int left = n_blocks, step = 0, slot_i = 0;
    block_at(ib, 0, -1);
    auto issue = [&]() {  // the next stage of the sequence; past its end one piece again and again, so that every stage has as many loads
        const uint32_t dst = my_ring + (uint32_t)slot_i * S::kStageBytes;
        slot_i = (slot_i + 1) % S::kRing;
        const int lv = opaque(lane);
        auto weights = [&](const unsigned char* base, int rows) {
#pragma unroll
            for (int i = 0; i < S::kLoads; ++i)
                load16_once_to_lds_at(base, (uint32_t)row_of(lv, i, rows) * (3 * H * 2) + piece_of(lv, i), dst + i * 1024);
        };
        const bool with_x = have_b && (ib.first || !S::kKeepX);
        const int per = with_x ? 3 : 2;
        const int n_gu = have_b ? per * S::kStages : 0;
        if (have_b && step < n_gu) {
            const int c = per == 3 ? step / 3 : step / 2;
            const int kind = step - c * per + (per == 2);  // 0: tokens, 1: gate, 2: up
            if (kind == 0) {
                const unsigned char* base = reinterpret_cast<const unsigned char*>(a.x) + (size_t)(wv * HW + c * S::kCols) * 2;
#pragma unroll
                for (int i = 0; i < S::kLoads; ++i)
                    load16_to_lds_at(base, (uint32_t)s_tok[ib.first_tok + row_of(lv, i, ib.ntok)] * (H * 2) + piece_of(lv, i), dst + i * 1024);
            } else {
                weights(ib.base + (size_t)((kind - 1) * H + c * S::kCols) * 2, ib.valid);
            }
        } else if (have_p) {
            weights(ip.base + (size_t)(2 * H + (step - n_gu) * S::kCols) * 2, ip.valid);
        } else {
#pragma unroll
            for (int i = 0; i < S::kLoads; ++i) load16_to_lds_at(a.x, 0u, dst + i * 1024);
        }
        ++step;
        if (step >= n_gu + (have_p ? S::kStages : 0) && (have_b || have_p)) {  // on to the next block
            step = 0;
            ip = ib;
            have_p = have_b;
            if (have_b && --left > 0)
                block_at(ib, ip.seg, ip.row + kGmUnits);
            else
                have_b = false;
        }
    };
#pragma unroll 1
    for (int i = 0; i < S::kRing; ++i) issue();

    // ---- the products
    int slot_c = 0;
    auto next_stage = [&]() {  // the oldest stage has landed; where it lies
        wait_vm_fence<(S::kRing - 1) * S::kLoads>();
        const unsigned char* st = ring0 + (size_t)wv * (S::kRing * S::kStageBytes) + (size_t)slot_c * S::kStageBytes;
        slot_c = (slot_c + 1) % S::kRing;
        return st;
    };
    auto read_rows = [&](const unsigned char* st, gm_bf16x8 (&v)[KS]) {  // lane: row lane % 16, columns 32 s + 8 grp .. + 8 of step s
        const int lv = opaque(lane), r = lv & 15;
#pragma unroll
        for (int s = 0; s < KS; ++s) v[s] = *reinterpret_cast<const gm_bf16x8*>(st + r * RB + (((4 * s + (lv >> 4)) ^ (r & (CH - 1))) * 16));
    };
    constexpr bool keep = S::kKeepX;
    gm_bf16x8 xr[keep ? S::kStages : 1][KS];  // the tokens of the item
    constexpr int NT = HW == 512 ? 2 : 4;  // down tiles at a time ...
    constexpr int NC = HW == 512 ? 1 : 2;  // ... and chains of products in each
    gm_f32x4 y[S::kStages * GR][CPL];
#pragma unroll
    for (int c = 0; c < S::kStages * GR; ++c)
#pragma unroll
        for (int j = 0; j < CPL; ++j) y[c][j] = gm_f32x4{0.f, 0.f, 0.f, 0.f};
    Block cb, cp;  // this block, the one before
    block_at(cb, 0, -1);
#pragma unroll 1
    for (int n = 0; n <= n_blocks; ++n) {
        if (n < n_blocks) {
            if (n > 0) block_at(cb, cp.seg, cp.row + kGmUnits);
            gm_f32x4 g[KS], u[KS];
#pragma unroll
            for (int q = 0; q < KS; ++q) g[q] = u[q] = gm_f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
            for (int c = 0; c < S::kStages; ++c) {
                if (!keep || cb.first) {
                    read_rows(next_stage(), xr[keep ? c : 0]);
                    wait_lds_fence();
                    issue();
                }
                gm_bf16x8 w[KS];
                __builtin_amdgcn_sched_barrier(0);  // (a stage's operands are read when they are due: rows of 4,096 have no registers to spare)
                read_rows(next_stage(), w);
                wait_lds_fence();
                issue();
                __builtin_amdgcn_sched_barrier(0);
#pragma unroll
                for (int s = 0; s < KS; ++s) g[s] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(w[s], xr[keep ? c : 0][s], g[s], 0, 0, 0);
                read_rows(next_stage(), w);
                wait_lds_fence();
                issue();
                __builtin_amdgcn_sched_barrier(0);
#pragma unroll
                for (int s = 0; s < KS; ++s) u[s] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(w[s], xr[keep ? c : 0][s], u[s], 0, 0, 0);
            }
#pragma unroll
            for (int d = KS / 2; d > 0; d /= 2)
#pragma unroll
                for (int q = 0; q < d; ++q) {
                    g[q] += g[q + d];
                    u[q] += u[q + d];
                }
            barrier_lds();  // the partial tiles of the block before have been added up
            float* part = s_part + wv * 512 + opaque(lane) * 4;  // units 4 (lane / 16) .. + 4 of token lane % 16
            *reinterpret_cast<gm_f32x4*>(part) = g[0];
            *reinterpret_cast<gm_f32x4*>(part + 256) = u[0];
        }
        barrier_lds();
        if (n < n_blocks) {  // a lane from 32 on adds a gate value up, one below the up value of the same unit and token
            const int lv = opaque(lane), e = wv * 32 + (lv & 31), unit = 4 * (e >> 6) + (e & 3), tok = (e >> 2) & 15;
            float p[kGroupedWaves];
#pragma unroll
            for (int w = 0; w < kGroupedWaves; ++w) p[w] = s_part[(w * 2 + (lv < 32)) * 256 + e];
            const float v = ((p[0] + p[1]) + (p[2] + p[3])) + ((p[4] + p[5]) + (p[6] + p[7]));
            const int b = __builtin_bit_cast(int, v);
            const float up = __builtin_bit_cast(float, __builtin_amdgcn_permlane32_swap(b, b, false, false)[0]);  // lanes 32..63 take lanes 0..31
            if (lv >= 32) {
                const float gate = tok < cb.ntok ? s_w[cb.first_tok + tok] : 0.f;
                s_act[(n & 1) * 256 + unit * 16 + tok] = unit < cb.valid && tok < cb.ntok ? silu(v) * up * gate : 0.f;
            }
        }
        if (n > 0) {  // the block before: its activations are complete since the barrier
            const float* act = s_act + ((n - 1) & 1) * 256;
            float av[4];
#pragma unroll
            for (int s = 0; s < 4; ++s) av[s] = act[s * 64 + opaque(lane)];  // token lane % 16, unit 4 s + grp
#pragma unroll
            for (int c = 0; c < S::kStages; ++c) {
                __builtin_amdgcn_sched_barrier(0);
                const unsigned char* st = next_stage();
#pragma unroll
                for (int h = 0; h < GR; ++h) {
                    const int lv = opaque(lane), l16 = lv & 15, grp = lv >> 4;
                    uint32_t w[4][CPL / 2];
#pragma unroll
                    for (int s = 0; s < 4; ++s) {  // unit 4 s + grp, columns CPL * (lane % 16) .. + CPL
                        const int r = 4 * s + grp;
                        if constexpr (CPL == 8) {
                            const uint4 v = *reinterpret_cast<const uint4*>(st + r * RB + (((h * 16 + l16) ^ (r & (CH - 1))) * 16));
                            w[s][0] = v.x; w[s][1] = v.y; w[s][2] = v.z; w[s][3] = v.w;
                        } else {
                            const uint2 v = *reinterpret_cast<const uint2*>(st + r * RB + (((l16 >> 1) ^ (r & (CH - 1))) * 16) + (l16 & 1) * 8);
                            w[s][0] = v.x; w[s][1] = v.y;
                        }
                    }
                    if (h == GR - 1) {
                        wait_lds_fence();
                        issue();
                    }
                    if (cp.valid < kGmUnits) {  // uniform: rows past the block repeat its last one, and zero times infinity is not zero
#pragma unroll
                        for (int s = 0; s < 4; ++s)
#pragma unroll
                            for (int j = 0; j < CPL / 2; ++j) w[s][j] = 4 * s + grp < cp.valid ? w[s][j] : 0u;
                    }
#pragma unroll
                    for (int j0 = 0; j0 < CPL; j0 += NT) {
                        __builtin_amdgcn_sched_barrier(0);
                        gm_f32x4 t[NC][NT];
#pragma unroll
                        for (int q = 0; q < NC; ++q)
#pragma unroll
                            for (int j = 0; j < NT; ++j) t[q][j] = gm_f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
                        for (int s = 0; s < 4; ++s)
#pragma unroll
                            for (int j = 0; j < NT; ++j) {
                                const uint32_t v = w[s][(j0 + j) / 2];
                                t[s % NC][j] = __builtin_amdgcn_mfma_f32_16x16x4f32(av[s], j & 1 ? bf16_hi(v) : bf16_lo(v), t[s % NC][j], 0, 0, 0);
                            }
#pragma unroll
                        for (int j = 0; j < NT; ++j)
#pragma unroll
                            for (int i = 0; i < 4; ++i) y[c * GR + h][j0 + j][i] = (cp.first ? 0.f : y[c * GR + h][j0 + j][i]) + (NC == 1 ? t[0][j][i] : t[0][j][i] + t[NC - 1][j][i]);
                        // added here and not where the sums are needed: the tiles would stay in registers until then, and those of
                        // rows of 4,096 were spilled (256 and scratch, now 205), each reload a wait for the whole ring
#pragma unroll
                        for (int j = 0; j < NT; ++j) asm volatile("" : "+v"(y[c * GR + h][j0 + j]));
                    }
                }
            }
            if (cp.last) {  // tokens 4 grp .. + 4, columns CPL * (lane % 16) .. + CPL of every stage
                const int lv = opaque(lane), l16 = lv & 15, grp = lv >> 4;
                float* out = a.part + ((size_t)blockIdx.x * a.seg_max + cp.seg) * kGmTokens * H + wv * HW + l16 * CPL;
#pragma unroll
                for (int i = 0; i < 4; ++i)
                    if (4 * grp + i < cp.ntok)
#pragma unroll
                        for (int c = 0; c < S::kStages * GR; ++c)
#pragma unroll
                            for (int j = 0; j < CPL; j += 4)
                                *reinterpret_cast<float4*>(out + (size_t)(4 * grp + i) * H + c * (16 * CPL) + j) =
                                    make_float4(y[c][j][i], y[c][j + 1][i], y[c][j + 2][i], y[c][j + 3][i]);
            }
        }
        cp = cb;
    }
    wait_vm_fence<0>();  // nothing is on its way into this LDS when it is given back
}

// y[b][h] = sum of the partial rows of the segments whose item holds token b.  The workgroup
// first lists those segments in order (workgroup-major) in LDS; 32 slices of the list are
// then added by a thread each, all of a slice's loads in flight together, and the slice sums are
// added in slice order.  grid (H / 32, B), 256 threads = 32 slices x 8 float4 columns;
// dynamic LDS: 2 * n_blocks * seg_max ints.
// The places of the item at which token b stands, a bit each (at most 16): more than one where the token lists the expert
// more than once.
__device__ __forceinline__ unsigned places_of(const GroupItem& it, int b) {
    unsigned m = 0;
    for (int q = 0; q < it.ntok; ++q)
        if (it.tok[q] == b) m |= 1u << q;
    return m;
}
__device__ __forceinline__ unsigned places_of(const GmItemOut& it, int b) {
    const unsigned long long t = it.toks;
    unsigned m = 0;
    for (int q = 0; q < it.ntok; ++q)
        if ((int)(t >> (4 * q) & 15) == b) m |= 1u << q;
    return m;
}
template <typename Item>
__global__ void __launch_bounds__(256) ffn_grouped_reduce_kernel(const float* __restrict__ part,
                                                                 const Item* __restrict__ items,
                                                                 const int32_t* __restrict__ n_items, int tb, int I,
                                                                 int cost, int H, int n_blocks, int seg_max,
                                                                 float* __restrict__ y) {
    extern __shared__ __align__(16) int32_t s_rows[];  // per segment: its number << 16 | the token's places in its item; -1: none
    __shared__ float s_sum[32][32];
    __shared__ int s_wbase[4];
    __shared__ int s_nv, s_more;  // s_more: the token has a second place somewhere
    const int n = n_blocks * seg_max;  // (below 2^15: a few segments for each compute unit)
    int32_t* s_list = s_rows + n;  // rows of the token: of its first place in every segment that holds it, in order
    const int b = blockIdx.y, tid = threadIdx.x, lane = tid & (kWave - 1), wv = tid / kWave;
    if (tid == 0) s_more = 0;
    cost = grouped_start(*n_items, n_blocks, cost);
    const int total = *n_items * (I + cost);
    for (int g = tid; g < n_blocks; g += 256) {
        int row = grouped_range_begin(total, g, n_blocks);
        const int R1 = grouped_range_begin(total, g + 1, n_blocks);
        for (int seg = 0; seg < seg_max; ++seg) {
            int entry = -1;
            if (row < R1) {
                int item, r0, r1;
                grouped_segment(&row, R1, I, cost, &item, &r0, &r1);
                const unsigned at = r0 < r1 ? places_of(items[item], b) : 0;
                if (at != 0) entry = (g * seg_max + seg) << 16 | (int)at;
            }
            s_rows[g * seg_max + seg] = entry;
        }
    }
    __syncthreads();
    // compaction in list order: ballots inside a wavefront, running offsets across wavefronts and rounds
    int base = 0;
    for (int e0 = 0; e0 < n; e0 += 256) {
        const int e = e0 + tid;
        const int r = e < n ? s_rows[e] : -1;
        const unsigned long long mask = __ballot(r >= 0);
        if (lane == 0) s_wbase[wv] = __popcll(mask);
        __syncthreads();
        int before = base;
        for (int w = 0; w < wv; ++w) before += s_wbase[w];
        if (r >= 0) {
            s_list[before + __popcll(mask & ((1ull << lane) - 1ull))] = (r >> 16) * tb + __ffs(r) - 1;
            if ((r & 0xffff & (r - 1)) != 0) s_more = 1;
        }
        base += s_wbase[0] + s_wbase[1] + s_wbase[2] + s_wbase[3];
        __syncthreads();
    }
    if (tid == 0) s_nv = base;
    __syncthreads();
    const int nv = s_nv;
    const int cq = tid & 7, sl = tid >> 3;
    const int h = blockIdx.x * 32 + cq * 4;
    const int per = (nv + 31) / 32;
    const int p0 = sl * per, p1 = min(nv, p0 + per);
    float4 acc = make_float4(0.f, 0.f, 0.f, 0.f);
    auto add = [&](const float4& v) {
        acc.x += v.x;
        acc.y += v.y;
        acc.z += v.z;
        acc.w += v.w;
    };
    auto row = [&](int at) { return *reinterpret_cast<const float4*>(part + (size_t)at * H + h); };
    for (int p = p0; p < p1; p += 8) {
        float4 v[8];
#pragma unroll
        for (int u = 0; u < 8; ++u) v[u] = p + u < p1 ? row(s_list[p + u]) : make_float4(0.f, 0.f, 0.f, 0.f);
#pragma unroll
        for (int u = 0; u < 8; ++u) add(v[u]);
    }
    if (s_more != 0)  // an expert that the token lists more than once
        for (int e = sl; e < n; e += 32)
            if (s_rows[e] >= 0)
                for (int places = s_rows[e] & 0xffff & (s_rows[e] - 1); places != 0; places &= places - 1)
                    add(row((s_rows[e] >> 16) * tb + __ffs(places) - 1));
    s_sum[sl][cq * 4 + 0] = acc.x;
    s_sum[sl][cq * 4 + 1] = acc.y;
    s_sum[sl][cq * 4 + 2] = acc.z;
    s_sum[sl][cq * 4 + 3] = acc.w;
    __syncthreads();
    if (tid < 32) {
        float t = 0.f;
#pragma unroll
        for (int k2 = 0; k2 < 32; ++k2) t += s_sum[k2][tid];
        y[(size_t)b * H + blockIdx.x * 32 + tid] = t;
    }
}

}  // namespace

int ffn_scratch_alloc(const moei_model_desc& d, int n_act_max, FfnScratch* out) {
    out->n_act_max = n_act_max;
    // the streaming kernels take one workgroup per compute unit; some units are left to the
    // side stream's match and priority kernels so that these never hold up a streaming workgroup
    // (the stream is bound by HBM, not by the number of units: measured per layer step on the
    // 64-expert shape, 42.9 us with 8 units left free, 41.1 us with 24, 43.4 us with 64)
    int reserve = env_int("MOEI_RESERVE_CUS", 24);
    if (reserve < 0 || reserve > compute_units() / 2) reserve = 0;
    out->n_part = compute_units() - reserve;
    out->n_free = reserve;
    float* unused = nullptr;  // the static scratch of expert_ffn_gemv_static: address looked up at set-up
    int rc = static_part_ptr(&unused);
    if (rc) return rc;
    hipError_t e = hipMalloc((void**)&out->d_part, (size_t)out->n_part * d.H * sizeof(float));
    if (e != hipSuccess) {
        out->d_part = nullptr;
        MOEI_FAIL(MOEI_ENOMEM, "FFN scratch allocation failed: %s", hipGetErrorString(e));
    }
    return MOEI_OK;
}

void ffn_scratch_free(FfnScratch* s) {
    (void)hipFree(s->d_part);
    s->d_part = nullptr;
}

// ------------------------------------------------------------------ scratch that is never allocated
// The workgroup partial rows of expert_ffn_gemv_static live in this array: one copy per GPU that
// the library runs on, held until the process ends.  Host code never uses the array's name as an
// address: its device address is looked up once per device and kept in g_static_part.
}  // namespace moei

static __device__ __align__(256) float scratch[moei::kStaticPartFloats];

namespace moei {

namespace {
constexpr int kMaxDevices = 64;
float* g_static_part[kMaxDevices] = {};
}  // namespace

// Device address of the static partial-row array on the current device (looked up at the
// first call on that device: cache creation, else the entry point itself).
int static_part_ptr(float** out) {
    int dev = -1;
    MOEI_HIP(hipGetDevice(&dev));
    if (dev < 0 || dev >= kMaxDevices) MOEI_FAIL(MOEI_EINVAL, "device ordinal %d outside [0, %d)", dev, kMaxDevices);
    if (!g_static_part[dev]) {
        float* ptr = nullptr;
        MOEI_HIP(hipGetSymbolAddress((void**)&ptr, HIP_SYMBOL(scratch)));
        if (!ptr) MOEI_FAIL(MOEI_EHIP, "the static scratch array has no device address");
        g_static_part[dev] = ptr;
    }
    *out = g_static_part[dev];
    return MOEI_OK;
}

int launch_expert_ffn_static(const moei_model_desc& d, const void* d_pool, size_t slot_elems, int n_slots_total,
                             int n_part, const int32_t* d_slot_ids, const float* d_gate_w, int n_act, const void* d_x,
                             float* d_y, int32_t* d_flags, hipStream_t s) {
    if ((size_t)n_part * (size_t)d.H > kStaticPartFloats)
        MOEI_FAIL(MOEI_ECAPACITY,
                  "expert_ffn_gemv_static: %d partial rows of H = %d floats exceed the static scratch of %zu floats "
                  "(H <= %zu on this device)",
                  n_part, d.H, kStaticPartFloats, kStaticPartFloats / (size_t)n_part);
    FfnScratch scr;
    int rc = static_part_ptr(&scr.d_part);
    if (rc) return rc;
    scr.n_part = n_part;
    return launch_expert_ffn(d, d_pool, slot_elems, n_slots_total, scr, d_slot_ids, d_gate_w, n_act, d_x, d_y, d_flags, nullptr, s);
}

namespace {
// The streaming kernel reads 16-byte pieces: rows and addresses have to allow it, and the registers hold up to 16 chunks
// of a row (other shapes take ffn_fused_generic_kernel).
bool ffn_streams(const moei_model_desc& d, const void* d_pool, size_t slot_elems) {
    const int wb = d.wdtype == MOEI_WDTYPE_BF16 ? 2 : 4;
    static const bool force_generic = env_int("MOEI_FFN_GENERIC", 0) != 0;
    return (d.H * wb) % 16 == 0 && (uintptr_t)d_pool % 16 == 0 && (slot_elems * wb) % 16 == 0 && !force_generic;
}
}  // namespace

int expert_ffn_scan_waves(const moei_model_desc& d, const void* d_pool, size_t slot_elems, const FfnScratch& scr, const void* d_x) {
    const int chunk = kWave * 16 / (d.wdtype == MOEI_WDTYPE_BF16 ? 2 : 4), nch = (d.H + chunk - 1) / chunk;
    const bool takes = ffn_streams(d, d_pool, slot_elems) && nch <= 16 && (uintptr_t)d_x % 16 == 0 && forced_takes_match(forced_waves());
    return takes ? step_waves((d.k + d.n_shared) * d.I, scr.n_part, nch) : 0;
}

int launch_expert_ffn(const moei_model_desc& d, const void* d_pool, size_t slot_elems, int n_slots_total,
                      const FfnScratch& scr, const int32_t* d_slot_ids, const float* d_gate_w, int n_act,
                      const void* d_x, float* d_y, int32_t* d_flags, const StepArgs* step, hipStream_t s) {
    if (n_act == 0) {  // an empty sum: the reduction over zero partial rows writes zeros
        launch(K_FFN_REDUCE, ffn_reduce_kernel, dim3((d.H + 31) / 32), dim3(256), 0, s, (const float*)scr.d_part, 0, d.H,
               d_y, StepTail{});
        MOEI_LAUNCH_CHECK();
        return MOEI_OK;
    }
    FfnArgs a{};
    a.pool = d_pool;
    a.slot_elems = slot_elems;
    a.n_slots_total = n_slots_total;
    a.slot_ids = d_slot_ids;
    a.gate_w = d_gate_w;
    a.x = d_x;
    a.part = scr.d_part;
    a.H = d.H;
    a.I = d.I;
    a.n_act = n_act;
    a.flags = d_flags;
    a.n_wg = scr.n_part;
    StepTail tail{};
    size_t match_lds = 0;
    if (step) {
        const bool bf16 = d.wdtype == MOEI_WDTYPE_BF16;
        a.match = step->match;
        a.route = step->route;
        a.route.vec_ok = ((uintptr_t)a.route.W | (uintptr_t)a.route.x) % 16 == 0 && d.H % (bf16 ? 8 : 4) == 0;
        a.n_shared = d.n_shared;
        a.shared_base = step->shared_base;
        match_lds = step->match_lds;
        tail = StepTail{a.route.E, a.route.words};
    }
    const bool fast = ffn_streams(d, d_pool, slot_elems);
    if (d.wdtype == MOEI_WDTYPE_BF16) return launch_ffn_typed<uint16_t>(a, fast, scr.n_part, match_lds, tail, d_y, s);
    return launch_ffn_typed<float>(a, fast, scr.n_part, match_lds, tail, d_y, s);
}


namespace {
// Which kernel a bf16 call takes.  Both stream an expert once for up to four requests (rows of 4,096: the vector kernel once per
// request), and the matrix kernel takes 1 - 7 us longer to start and to end, so it has to save something: it does from
// four requests on where an expert is expected to serve more than 1.25 of them, by as much as there is to stream.  us a call,
// vector / matrix kernel: 64 experts of 1,408 units + 2 shared, H = 2,048, top 6, 1 / 2 / 3 / 4 / 8 / 16 requests 30.8 / 35.7, 47.1 / 50.9, 65.5 /
// 66.1, 83.2 / 81.0, 129 / 119, 190 / 162; 8 of 6,000 units, H = 4,096, top 2, 3 / 8 / 16 requests 143 / 145, 269 / 190, 472 / 217.  Three
// requests of other models are slower too or the same (8 of 1,400 + 2, H = 2,048 33.9 / 37.5; 16 of 400, H = 512 13.0 / 15.2; 32 of 700 + 1, H = 1,024
// 19.9 / 19.3).
// 100 of 2,000, H = 1,024, top 8, 6 requests (1.2 of them an expert) 84.0 / 84.4; 20 of 300, H = 4,096, top 1, 8 requests (1.2) 20.9 /
// 26.7; 16 of 400, H = 512, top 4, 4 / 6 / 12 requests (1.5 / 1.8 / 3.1) 13.1 / 15.5, 15.3 / 15.9, 19.2 / 16.8.  Rows of 4,096, which start
// and end longest, have to save 100 MB (17 of 325 units, top 2, 13 requests, 71 MB: 44.9 / 47.5), and the partial rows - one per workgroup and
// token of its item - must not outweigh the weights (4 of 225 units, H = 1,024, 12 requests of all four: 12.6 MB of rows, 5.5 MB of
// weights, 18.7 / 22.8).  Over 606 calls of 4 - 16 requests that the rule gives to it (2 - 160 experts of 60 - 6,000 units) 0.78 of the vector
// kernel's time; 36 of them take 3 % longer or more (29 of 1,727, H = 512, top 2, 13 requests 27.8 / 34.6 is the worst), which neither the bytes it
// is expected to save nor the requests an expert set apart from those that gain.
bool grouped_mm(const moei_model_desc& d, int B) {
    if (d.wdtype != MOEI_WDTYPE_BF16 || B < 4) return false;
    double none = 1.0;  // share of the experts that nobody picks, picks being even
    for (int b = 0; b < B; ++b) none *= 1.0 - (double)d.k / d.E;
    const double streamed = d.E * (1.0 - none) + d.n_shared, expert = 6.0 * d.H * d.I;
    const double served = (double)B * (d.k + d.n_shared);
    if (compute_units() * (served / streamed) * 4.0 * d.H > 1.5 * streamed * expert) return false;
    return (served - 1.25 * streamed) * expert >= (d.H > 2048 ? 100e6 : 5e6);
}
// Whether any batch of the model takes it: its rows are up to four times those of the vector kernel (67 MB, 17 without, for the
// 64-expert shape).
bool grouped_mm_any(const moei_model_desc& d) {
    for (int B = 1; B <= kMaxBatch; ++B)
        if (grouped_mm(d, B)) return d.H == 512 || d.H == 1024 || d.H == 2048 || d.H == 4096;
    return false;
}
// items of 16 picks: the sum over the experts of ceil(picks / 16), and the shared experts
int gm_max_items(const moei_model_desc& d, int B) { return std::min(B * d.k, d.E + (B * d.k + kGmTokens - 1) / kGmTokens) + d.n_shared; }
int gm_segments(const moei_model_desc& d) { return grouped_seg_max(gm_max_items(d, kMaxBatch), compute_units()); }
size_t gm_rows(const moei_model_desc& d) { return (size_t)compute_units() * gm_segments(d) * kGmTokens; }
}  // namespace

int grouped_max_items(const moei_model_desc& d) { return kMaxBatch * d.k + d.n_shared * kMaxBatch; }
size_t grouped_item_bytes() { return std::max(sizeof(GroupItem), sizeof(GmItemOut)); }
size_t grouped_part_floats(const moei_model_desc& d) {
    const int G = compute_units();
    const size_t rows = (size_t)G * grouped_seg_max(grouped_max_items(d), G) * kMaxGroup;
    if (!grouped_mm_any(d)) return rows * d.H;
    return std::max(rows, gm_rows(d)) * d.H + (size_t)kMaxBatch * d.H / 2;  // behind the rows: an aligned copy of the tokens
}

namespace {
template <typename WT>
int launch_grouped_typed(const moei_model_desc& d, GroupedFfnArgs ga, int B, float* d_y, hipStream_t s) {
    using V = WVec<WT>;
    const int nch = d.H / (kWave * V::N);
    const int grid = compute_units();
    ga.seg_max = grouped_seg_max(grouped_max_items(d), grid);
    int rc;
#define MOEI_GROUPED_CASE(N_)                                                                           \
    case N_: {                                                                                          \
        ga.grp.tb = GroupedShape<N_>::kTB;                                                              \
        const size_t smem = (size_t)(GroupedShape<N_>::kTB + kGroupedWaves) * d.H * sizeof(float) +     \
                            (size_t)ga.max_items * sizeof(GroupItem) + (size_t)B * d.k * 8;             \
        if (smem > kLdsBudget) MOEI_FAIL(MOEI_ECAPACITY, "expert_ffn_grouped: H = %d does not fit the LDS staging", d.H); \
        rc = allow_big_lds(ffn_grouped_kernel<WT, N_>, smem);                                           \
        if (rc) return rc;                                                                              \
        launch(K_FFN_FUSED, ffn_grouped_kernel<WT, N_>, dim3(grid), dim3(kGroupedWaves * kWave), smem, s, ga); \
        MOEI_LAUNCH_CHECK();                                                                            \
        break;                                                                                          \
    }
    switch (nch) {
        MOEI_GROUPED_CASE(1)
        MOEI_GROUPED_CASE(2)
        MOEI_GROUPED_CASE(4)
        MOEI_GROUPED_CASE(8)
        MOEI_GROUPED_CASE(10)
        default:
            MOEI_FAIL(MOEI_EINVAL, "expert_ffn_grouped: H = %d is not supported (needs H / %d in {1,2,4,8,10})", d.H,
                      kWave * V::N);
    }
#undef MOEI_GROUPED_CASE
    launch(K_FFN_REDUCE, ffn_grouped_reduce_kernel<GroupItem>, dim3(d.H / 32, B), dim3(256),
           (size_t)2 * grid * ga.seg_max * sizeof(int32_t), s, (const float*)ga.part, (const GroupItem*)ga.grp.items,
           (const int32_t*)ga.grp.n_items, ga.grp.tb, d.I, ga.cost, d.H, grid, ga.seg_max, d_y);
    MOEI_LAUNCH_CHECK();
    return MOEI_OK;
}

int launch_grouped_mm(const moei_model_desc& d, GroupedMmArgs ga, int B, float* d_y, hipStream_t s) {
    const int grid = compute_units();
    int rc;
    if ((uintptr_t)ga.x % 16 != 0) {  // the ring's loads take 16-byte pieces
        uint16_t* copy = reinterpret_cast<uint16_t*>(ga.part + gm_rows(d) * d.H);
        MOEI_HIP(hipMemcpyAsync(copy, ga.x, (size_t)B * d.H * 2, hipMemcpyDeviceToDevice, s));
        ga.x = copy;
    }
    if (ga.seg_max > kGmMaxSegs) MOEI_FAIL(MOEI_ECAPACITY, "expert_ffn_grouped: %d segments a workgroup exceed %d", ga.seg_max, kGmMaxSegs);
#define MOEI_GM_CASE(HW_)                                                                              \
    case HW_ * kGroupedWaves: {                                                                        \
        const size_t smem = gm_lds<HW_>(ga.max_items, ga.n_list);                                      \
        rc = allow_big_lds(ffn_grouped_mm_kernel<HW_>, smem);                                          \
        if (rc) return rc;                                                                             \
        launch(K_FFN_GROUPED_MM, ffn_grouped_mm_kernel<HW_>, dim3(grid), dim3(kGroupedWaves * kWave), smem, s, ga); \
        MOEI_LAUNCH_CHECK();                                                                           \
        break;                                                                                         \
    }
    switch (d.H) {
        MOEI_GM_CASE(64)
        MOEI_GM_CASE(128)
        MOEI_GM_CASE(256)
        MOEI_GM_CASE(512)
        default:
            MOEI_FAIL(d.H == 5120 ? MOEI_ECAPACITY : MOEI_EINVAL, "expert_ffn_grouped: H = %d is not supported (needs H / 512 in {1,2,4,8})", d.H);
    }
#undef MOEI_GM_CASE
    launch(K_FFN_REDUCE, ffn_grouped_reduce_kernel<GmItemOut>, dim3(d.H / 32, B), dim3(256),
           (size_t)2 * grid * ga.seg_max * sizeof(int32_t), s, (const float*)ga.part, (const GmItemOut*)ga.grp.items,
           (const int32_t*)ga.grp.n_items, kGmTokens, d.I, ga.cost, d.H, grid, ga.seg_max, d_y);
    MOEI_LAUNCH_CHECK();
    return MOEI_OK;
}
}  // namespace

int launch_expert_ffn_grouped(const moei_model_desc& d, const void* d_pool, size_t slot_elems, void* d_items,
                              int32_t* d_n_items, float* d_part, const int32_t* d_slot_of_row, int shared_base,
                              const int32_t* d_idx, const float* d_w, int B, const void* d_x, float* d_y,
                              int32_t* d_flags, hipStream_t s) {
    if (B > kMaxBatch) MOEI_FAIL(MOEI_EINVAL, "expert_ffn_grouped: B = %d exceeds %d", B, kMaxBatch);
    // the item list is built by a thread per pick and per expert of a 256-thread group
    if (d.E > 256 || B * d.k > 512)
        MOEI_FAIL(MOEI_EINVAL, "expert_ffn_grouped: E = %d, B * k = %d exceed 256 experts or 512 picks", d.E, B * d.k);
    const int wb = d.wdtype == MOEI_WDTYPE_BF16 ? 2 : 4;
    const int n = 16 / wb;
    if (d.H % (kWave * n) != 0 || (uintptr_t)d_pool % 16 != 0 || (slot_elems * wb) % 16 != 0)
        MOEI_FAIL(MOEI_EINVAL, "expert_ffn_grouped: H = %d must be a multiple of %d", d.H, kWave * n);
    GroupArgs gr{d_idx, d_w, d_slot_of_row, B, d.k, d.E, d.n_shared, shared_base, 0, d_items, d_n_items, d_flags};
    if (grouped_mm(d, B)) {
        GroupedMmArgs ga{reinterpret_cast<const uint16_t*>(d_pool), slot_elems, gr, gm_max_items(d, B), B * (d.k + 1),
                         reinterpret_cast<const uint16_t*>(d_x), d_part, d.H, d.I, grouped_cost(d.H, 2), gm_segments(d)};
        return launch_grouped_mm(d, ga, B, d_y, s);
    }
    GroupedFfnArgs ga{d_pool, slot_elems, gr, grouped_max_items(d), d_x, d_part, d.H, d.I, grouped_cost(d.H, wb), 0};
    if (d.wdtype == MOEI_WDTYPE_BF16) return launch_grouped_typed<uint16_t>(d, ga, B, d_y, s);
    return launch_grouped_typed<float>(d, ga, B, d_y, s);
}

}  // namespace moei

using namespace moei;

// Slot layout from the three plain matrices (host memory, desc->wdtype elements).
extern "C" int moei_expert_pack(const moei_model_desc* desc, const void* h_gate, const void* h_up, const void* h_down,
                                void* h_slot) {
    MOEI_REQUIRE(desc && h_gate && h_up && h_down && h_slot, "moei_expert_pack: null pointer");
    int rc = check_desc(desc);
    if (rc) return rc;
    const size_t H = desc->H, I = desc->I;
    const size_t wb = desc->wdtype == MOEI_WDTYPE_BF16 ? 2 : 4;
    const unsigned char* g = static_cast<const unsigned char*>(h_gate);
    const unsigned char* u = static_cast<const unsigned char*>(h_up);
    const unsigned char* dn = static_cast<const unsigned char*>(h_down);
    unsigned char* out = static_cast<unsigned char*>(h_slot);
    for (size_t i = 0; i < I; ++i) {
        unsigned char* row = out + i * 3 * H * wb;
        memcpy(row, g + i * H * wb, H * wb);
        memcpy(row + H * wb, u + i * H * wb, H * wb);
        unsigned char* dcol = row + 2 * H * wb;
        if (wb == 2) {
            const uint16_t* src = reinterpret_cast<const uint16_t*>(dn) + i;
            uint16_t* dst = reinterpret_cast<uint16_t*>(dcol);
            for (size_t h = 0; h < H; ++h) dst[h] = src[h * I];
        } else {
            const uint32_t* src = reinterpret_cast<const uint32_t*>(dn) + i;
            uint32_t* dst = reinterpret_cast<uint32_t*>(dcol);
            for (size_t h = 0; h < H; ++h) dst[h] = src[h * I];
        }
    }
    return MOEI_OK;
}
