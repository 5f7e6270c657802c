// Step 4 of the layer step: PredictEAM aggregation + prefetch / eviction priorities.
//
// Prefetch score (Sec. 4.5 of the paper): the matched EAM's cell, normalised over
// its row, times the layer-proximity factor (1 - (i - l)/L) for future layers i > l.
// Eviction score (Alg. 1): (cell + eps)(1 - i/L) / row sum, lowest score evicted
// first.  Both are evaluated as one fp64 division of exact products so that equal
// rationals give equal keys; the orders are then produced by rank counting (a
// candidate's rank is the number of candidates that sort before it; ties go to the
// lower flat id, so ranks are unique) with wavefront ballots.
#include <atomic>

#include "kernels.hpp"
#include "score.hpp"

namespace moei {

namespace {

constexpr int kRankThreads = 256;

// Scores, keys and order of ONE list (0: prefetch, 1: eviction) in one launch; grid (workgroups, 2
// lists), dynamic LDS L*E keys.  What bounds it is latency: a few trips to the cache and a launch.
// Ranking needs every key, and forming them all is a gather of B*L*E cells that sit in L2 - less
// time than a second launch - so every workgroup forms the whole list's keys in LDS for itself,
// writes the scores of its own cells [f0, f1) only, and ranks those.  A wavefront scores one layer
// row at a time, all B traces' cells requested together, and then ranks one cell at a time: its 64
// lanes compare that key with 64 others per step and the ballots' population counts add up to the
// number of candidates that sort before it (smaller key; among the lower ids also an equal one).
// Measured (26 x 64 cells, beside the library's other kernels): one scoring workgroup and a ranking
// launch took 12.7 + 9.2 us for 3 or 8 traces and 22.8 + 9.3 us for 16 traces and 96 picks; this
// kernel takes 9.5 and 15.8 us.  More loads in flight do not help: flat over the cells, two
// cells of 16 traces of a thread at once, it took 11.2 and 16.5 us; of those 3.5 us are the launch, 2.6 us
// the ranking and, at 16 traces, 5.6 us the misses on 26 x 16 rows that lie all over the collection (every
// cell taken from one trace: 11.1 us).  Fewer workgroups rank longer (64 a list: 13.3 and 19.1 us).
constexpr int kOrderThreads = 1024;
constexpr int kOrderPerLane = 4;   // cells of a row held in registers (rows up to 256 wide)
constexpr int kOrderTraces = 8;    // traces whose cells are requested together

__global__ void __launch_bounds__(kOrderThreads)
    priority_order_kernel(ScoreArgs a, int32_t* __restrict__ pf_order, int32_t* __restrict__ ev_order) {
    extern __shared__ __align__(16) unsigned char smem_raw[];
    u64* keys = reinterpret_cast<u64*>(smem_raw);
    const int tid = threadIdx.x, lane = tid & (kWave - 1);
    const int wv = __builtin_amdgcn_readfirstlane(tid / kWave);
    constexpr int kWaves = kOrderThreads / kWave;
    const int L = a.L, E = a.E, l = a.cur_layer, LE = L * E;
    const bool evict = blockIdx.y == 1;
    const int per = (LE + gridDim.x - 1) / gridDim.x;
    const int f0 = blockIdx.x * per, f1 = min(LE, f0 + per);
    // the sum of the matched traces' cells (i, j); entries of `best` outside [0, N) are skipped
    auto cell_sum = [&](int i, int j) -> u64 {
        u64 t = 0;
        for (int b0 = 0; b0 < a.B; b0 += kOrderTraces) {
            uint32_t v[kOrderTraces];
            bool ok[kOrderTraces];
#pragma unroll
            for (int u = 0; u < kOrderTraces; ++u) {
                const int n = b0 + u < a.B ? a.best[b0 + u] : -1;
                ok[u] = n >= 0 && n < a.N;
                v[u] = ok[u] ? cell_at(a.traces, a.cell_bytes, ((size_t)i * a.n_cap + n) * E + j) : 0u;
            }
#pragma unroll
            for (int u = 0; u < kOrderTraces; ++u) t += v[u];
        }
        return t;
    };
    for (int i = wv; i < L; i += kWaves) {
        u64 tv[kOrderPerLane];
        int sv[kOrderPerLane];
        u64 rsum = 0;
#pragma unroll
        for (int r = 0; r < kOrderPerLane; ++r) {
            const int j = lane + r * kWave;
            tv[r] = 0;
            sv[r] = -1;
            if (j < E) {
                tv[r] = cell_sum(i, j);
                sv[r] = a.slot_of[(size_t)i * E + j];
            }
            rsum += tv[r];
        }
        for (int j = lane + kOrderPerLane * kWave; j < E; j += kWave) rsum += cell_sum(i, j);
        const u64 R = wave_sum_u64_dpp(rsum);
        const double den = (double)(R ? R : 1ull) * (double)L;
        auto put = [&](int j, u64 t, int slot) {
            const int f = i * E + j;
            const double td = (double)t;
            // positive doubles order like their bit patterns; ~bits turns descending into ascending
            u64 key;
            if (evict) {
                const double v = ((td + a.eps) * (double)(L - i)) / den;
                if (f >= f0 && f < f1) a.V[f] = (float)v;
                key = slot >= 0 ? (u64)__double_as_longlong(v) : kNone;
            } else {
                double p = 0.0;
                if (i > l && R > 0) p = (td * (double)(L - i + l)) / den;
                if (f >= f0 && f < f1) a.P[f] = (float)p;
                key = i > l && p > 0.0 && slot < 0 ? ~(u64)__double_as_longlong(p) : kNone;
            }
            keys[f] = key;
        };
#pragma unroll
        for (int r = 0; r < kOrderPerLane; ++r) {
            const int j = lane + r * kWave;
            if (j < E) put(j, tv[r], sv[r]);
        }
        for (int j = lane + kOrderPerLane * kWave; j < E; j += kWave) put(j, cell_sum(i, j), a.slot_of[(size_t)i * E + j]);
    }
    __syncthreads();
    if (evict && l >= 0 && a.n_cur > 0) {  // the experts about to run are no candidates
        for (int m = tid; m < a.n_cur; m += kOrderThreads) {
            const int j = a.cur_idx[m];
            if (j >= 0 && j < E) keys[(size_t)l * E + j] = kNone;
        }
        __syncthreads();
    }
    int32_t* order = evict ? ev_order : pf_order;
    for (int f = f0 + wv; f < f1; f += kWaves) {
        const u64 mine = keys[f];
        if (mine == kNone) continue;  // uniform over the wavefront
        int rank = 0;
        // cells of lower ids sort before this one also at an equal key, those of higher ids do not (a cell
        // that is no candidate has the largest key and never does)
        auto count = [&](int g0, int g1, auto before) {
            for (int g = g0; g < g1; g += 4 * kWave) {  // four LDS reads in flight, then four ballots
                u64 kg[4];
#pragma unroll
                for (int u = 0; u < 4; ++u) {
                    const int c = g + u * kWave + lane;
                    kg[u] = c < g1 ? keys[c] : kNone;
                }
#pragma unroll
                for (int u = 0; u < 4; ++u) rank += __popcll(__ballot(before(kg[u])));
            }
        };
        count(0, f, [&](u64 k) { return k <= mine; });
        count(f + 1, LE, [&](u64 k) { return k < mine; });
        if (lane == 0) order[rank] = f;
    }
    if (blockIdx.x == 0) {  // how many candidates the list has
        int mine = 0;
        for (int f = tid; f < LE; f += kOrderThreads) mine += keys[f] != kNone;
        mine = (int)wave_sum_u32_dpp((unsigned)mine);
        __syncthreads();  // the keys have been read: their LDS takes the wavefronts' counts
        int* cnt = reinterpret_cast<int*>(smem_raw);
        if (lane == 0) cnt[wv] = mine;
        __syncthreads();
        if (tid == 0) {
            int t = 0;
            for (int w = 0; w < kWaves; ++w) t += cnt[w];
            *(evict ? a.n_ev : a.n_pf) = t;
        }
    }
}

// grid (workgroups, 2 lists).  The workgroup stages the list's L*E keys in LDS; a wavefront
// then takes one candidate cell at a time, its 64 lanes compare that key with 64 keys per
// step, and the ballot population counts add up to the candidate's rank: the number of
// candidates that sort before it (smaller key, or equal key and lower flat id).
__global__ void __launch_bounds__(kRankThreads)
    priority_rank_kernel(const u64* __restrict__ keys_all, int LE, const int32_t* __restrict__ n_pf,
                         const int32_t* __restrict__ n_ev, int32_t* __restrict__ pf_order,
                         int32_t* __restrict__ ev_order) {
    extern __shared__ __align__(16) unsigned char smem_raw[];
    u64* keys = reinterpret_cast<u64*>(smem_raw);
    const int which = blockIdx.y;
    if ((which == 0 ? *n_pf : *n_ev) == 0) return;  // an empty list: nothing to order (uniform)
    const u64* src = keys_all + (size_t)which * LE;
    int32_t* order = which == 0 ? pf_order : ev_order;
    const int tid = threadIdx.x, lane = tid & (kWave - 1);
    const int wv = __builtin_amdgcn_readfirstlane(tid / kWave);
    // stage the keys: eight independent loads in flight per thread
    for (int i0 = 0; i0 < LE; i0 += 8 * kRankThreads) {
        u64 v[8];
#pragma unroll
        for (int r = 0; r < 8; ++r) {
            const int i = i0 + r * kRankThreads + tid;
            v[r] = i < LE ? src[i] : kNone;
        }
#pragma unroll
        for (int r = 0; r < 8; ++r) {
            const int i = i0 + r * kRankThreads + tid;
            if (i < LE) keys[i] = v[r];
        }
    }
    __syncthreads();
    const int W = gridDim.x * (kRankThreads / kWave);
    for (int f = blockIdx.x * (kRankThreads / kWave) + wv; f < LE; f += W) {
        const u64 mine = keys[f];
        if (mine == kNone) continue;  // uniform over the wavefront
        int rank = 0;
        for (int g0 = 0; g0 < LE; g0 += 4 * kWave) {  // four LDS reads in flight, then four ballots
            u64 kg[4];
#pragma unroll
            for (int u = 0; u < 4; ++u) {
                const int g = g0 + u * kWave + lane;
                kg[u] = g < LE ? keys[g] : kNone;
            }
#pragma unroll
            for (int u = 0; u < 4; ++u) {
                const int g = g0 + u * kWave + lane;
                const bool before = kg[u] < mine || (kg[u] == mine && g < f);  // a padding key is never before
                rank += __popcll(__ballot(before));
            }
        }
        if (lane == 0) order[rank] = f;
    }
}

// A list's keys may need more LDS than a kernel gets unasked: its limit is raised to all there is, once.
int allow_keys_lds(const void* kernel, size_t bytes, std::atomic<bool>& raised) {
    constexpr size_t kLds = 160 * 1024;
    if (bytes > kLds) MOEI_FAIL(MOEI_EHIP, "the sort keys of a list take %zu bytes of LDS, there are %zu", bytes, kLds);
    if (bytes <= 64 * 1024 || raised.load(std::memory_order_relaxed)) return MOEI_OK;
    MOEI_HIP(hipFuncSetAttribute(kernel, hipFuncAttributeMaxDynamicSharedMemorySize, (int)kLds));
    raised.store(true, std::memory_order_relaxed);
    return MOEI_OK;
}

}  // namespace

}  // namespace moei

namespace moei {

ScoreArgs make_score_args(const moei_eamc* c, const int32_t* d_best, int B, int cur_layer, const int32_t* d_slot_of,
                          float eps, const int32_t* d_cur_idx, int n_cur, float* d_prefetch, float* d_evict,
                          int32_t* d_n_pf, int32_t* d_n_ev) {
    return ScoreArgs{c->d_traces, c->cell_bytes, c->n_cap, c->N, c->d.L, c->d.E, d_best, B, cur_layer, d_slot_of,
                     (double)eps, d_cur_idx, d_cur_idx ? n_cur : 0, d_prefetch, d_evict, nullptr, d_n_pf, d_n_ev,
                     nullptr, nullptr, 0, 0, nullptr, nullptr, nullptr, nullptr, nullptr};
}

// The two orders from the keys that score_cells left in d_keys.
int launch_priority_rank(const moei_model_desc& d, const unsigned long long* d_keys, const int32_t* d_n_pf,
                         const int32_t* d_n_ev, int32_t* d_pf_order, int32_t* d_ev_order, hipStream_t s) {
    const size_t LE = (size_t)d.L * d.E;
    const size_t smem = LE * 8;
    static std::atomic<bool> raised{false};
    int rc = allow_keys_lds(reinterpret_cast<const void*>(priority_rank_kernel), smem, raised);
    if (rc) return rc;
    // enough wavefronts that each ranks only a few cells
    int blocks = (int)((LE + 4 * (kRankThreads / kWave) - 1) / (4 * (kRankThreads / kWave)));
    blocks = blocks < 1 ? 1 : (blocks > 256 ? 256 : blocks);
    launch(K_PRIO_RANK, priority_rank_kernel, dim3(blocks, 2), dim3(kRankThreads), smem, s, (const u64*)d_keys,
           (int)LE, d_n_pf, d_n_ev, d_pf_order, d_ev_order);
    MOEI_LAUNCH_CHECK();
    return MOEI_OK;
}

}  // namespace moei

using namespace moei;

extern "C" int expert_priority(const moei_eamc* c, const int32_t* d_best, int32_t B, int32_t cur_layer,
                               const int32_t* d_slot_of, float eps, const int32_t* d_cur_idx, int32_t n_cur,
                               float* d_prefetch, float* d_evict, int32_t* d_pf_order, int32_t* d_n_pf,
                               int32_t* d_ev_order, int32_t* d_n_ev, void* stream) {
    MOEI_REQUIRE(c && d_best && d_slot_of && d_prefetch && d_evict && d_pf_order && d_n_pf && d_ev_order && d_n_ev,
                 "expert_priority: null pointer");
    MOEI_REQUIRE(B >= 1 && B <= kMaxMatchBatch, "expert_priority: B = %d outside [1, %d]", B, kMaxMatchBatch);
    MOEI_REQUIRE(cur_layer >= -1 && cur_layer < c->d.L, "expert_priority: cur_layer = %d outside [-1, %d)", cur_layer,
                 c->d.L);
    MOEI_REQUIRE(eps >= 0.f, "expert_priority: eps must not be negative");
    MOEI_REQUIRE(!d_cur_idx || (n_cur >= 0 && n_cur <= kMaxMatchBatch * c->d.E),
                 "expert_priority: n_cur = %d outside [0, %d]", n_cur, kMaxMatchBatch * c->d.E);
    hipStream_t s = as_stream(stream);
    ScoreArgs a = make_score_args(c, d_best, B, cur_layer, d_slot_of, eps, d_cur_idx, n_cur, d_prefetch, d_evict, d_n_pf,
                                  d_n_ev);
    const size_t LE = (size_t)c->d.L * c->d.E;
    // the keys of a list, and at least the counts of the wavefronts, in LDS
    const size_t smem = LE * 8 < 64 ? 64 : LE * 8;
    static std::atomic<bool> raised{false};
    int rc = allow_keys_lds(reinterpret_cast<const void*>(priority_order_kernel), smem, raised);
    if (rc) return rc;
    // a cell per wavefront (each costs a pass over all keys) up to one workgroup per compute unit
    constexpr int kWaves = kOrderThreads / kWave;
    const int blocks = (int)((LE + kWaves - 1) / kWaves);
    launch(K_PRIO_SCORE, priority_order_kernel, dim3(blocks > 128 ? 128 : blocks, 2), dim3(kOrderThreads), smem, s, a,
           d_pf_order, d_ev_order);
    MOEI_LAUNCH_CHECK();
    return MOEI_OK;
}
