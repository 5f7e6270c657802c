// The match and the scoring of an asynchronous layer step inside the launch that routes it and streams its experts.
//
// That launch leaves some compute units free; a few more workgroups in it find the most similar trace of the EAM that holds the
// step's routing (Sec. 4.5 of the paper), score the matched trace and select the heads of both orders, while the
// others stream weights.  They do not wait for the picks to begin: the scan, the longest part, runs over the EAM as it
// was before the step, and the picks' k cells of every trace are added when they are known.  The workgroup that scores also stores
// what the routing has decided (picks, weights, the EAM's row, flags): calls that wait for the step wait for this workgroup.
// The step is then one chain of two launches on the caller's stream: no kernels of its own for the
// match, no event calls, no fork to the side stream.
#pragma once

#include "match.hpp"
#include "score.hpp"
#include "step_route.hpp"

namespace moei {

constexpr int kStepMatchMaxBlocks = 128;  // never more workgroups than that match
constexpr int kStepScanLayers = 16;        // loads of the scan that one thread has under way
constexpr int kStepMatchMaxTraces = 1024;  // traces of one of them (their dot products and norms are held in LDS)

// What such a step tells the host, in pinned memory
struct StepMatched {
    int32_t best;
    float best_sim;
    int32_t seq;  // number of the step, stored when all of its results are in place
};

struct StepMatchArgs {
    int n_blocks;            // workgroups that match, before the ones that stream (0: none)
    int per;                 // traces of each of them
    int vec;                 // cells of a load
    int span, groups;        // threads per pass over them, and how many such groups share the layers (step_scan_plan)
    const unsigned long long* norm2;  // [n_cap]
    int32_t* q;              // [L*E] the EAM; the workgroup that scores adds this step's picks
    unsigned long long* cand;  // [n_blocks][2] winners of the workgroups (dot, norm) ...
    int32_t* cand_idx;       // [n_blocks] ... and their trace indices
    unsigned* ticket;        // arrival counter, zero between launches
    int32_t* best;
    float* best_sim;
    StepMatched* host;       // null: a captured step
    int32_t seq;             // for host->seq
    int32_t* idx;            // [k] the picks
    float* w;                // [k] their weights
    int32_t* flags;          // error flags (bit 1: pick not resident, bit 2: no softmax)
    ScoreArgs sc;
};
// A layer step in one launch and the reduction behind it.
struct StepArgs {
    StepMatchArgs match;
    size_t match_lds;
    StepRouteArgs route;
    int shared_base;  // slots of the layer's shared experts: shared_base + s
};
// Fills in how a.n_blocks workgroups with `waves` wavefronts that scan go about it; returns the trips to memory this takes a thread.
int step_scan_plan(StepMatchArgs* a, int waves);
// 0: a step over this collection keeps the match on the side stream
int step_match_blocks(const moei_eamc* c, const moei_model_desc& d, int free_units, int waves, bool captured);
size_t step_match_lds(const moei_eamc* c, int n_blocks);

#if defined(__HIPCC__)

struct alignas(16) StepMatchLds {
    ScoreLds<false> score;
    u64 nq;
    Best win;
    int finish;
    int sn[2];
    int best[kMaxMatchBatch];
    int pick[kStepPicks];
    float pick_w[kStepPicks];
};
// behind it lie 16 bytes per trace, the query's cells, which are read as 16-byte vectors, and step_route_lds
static_assert(sizeof(StepMatchLds) % 16 == 0, "the query's cells in LDS begin at a 16-byte boundary");

// Dot products of the query (in LDS) with traces t0 .. t0 + nt, added into s_dot (zero before), by the first groups * span threads.  Per layer the tile is one run
// of cells; a thread owns a vector of it and, where the tile is small, every groups-th layer only, and sixteen of
// its layers are requested together: beside the streaming workgroups a trip to memory takes 2 - 3 us.
template <typename CT, int VEC>
__device__ __forceinline__ void step_scan(const ScoreArgs& a, int span, int groups, int t0, int nt, const int32_t* qs, u64* s_dot) {
    using CV = CellVec<CT, VEC>;
    constexpr int U = kStepScanLayers;
    const int tid = threadIdx.x, lane = tid & (kWave - 1), L = a.L, E = a.E;
    const int rowV = E / VEC, nvec = nt * rowV, g = tid / span;
    const bool lane_rows = rowV <= kWave && (rowV & (rowV - 1)) == 0;
    const size_t lstride = (size_t)a.n_cap * E;
    if (g >= groups) return;
    for (int p = tid - g * span; p - lane < nvec; p += span) {  // (uniform over a wavefront)
        const bool valid = p < nvec;
        const int pc = valid ? p : 0, row = pc / rowV, col = (pc - row * rowV) * VEC;
        const CT* src = reinterpret_cast<const CT*>(a.traces) + (size_t)t0 * E + (size_t)pc * VEC;
        u64 acc = 0;
        for (int l0 = g; l0 < L; l0 += U * groups) {
            typename CV::raw v[U];
#pragma unroll
            for (int u = 0; u < U; ++u) {
                const int l = l0 + u * groups;
                v[u] = CV::load(src + (size_t)(l < L ? l : l0) * lstride);
            }
#pragma unroll
            for (int u = 0; u < U; ++u) {
                const int l = l0 + u * groups;
                if (l < L) acc = CV::dot(v[u], qs + (size_t)l * E + col, acc);
            }
        }
        if (lane_rows) {
            const u64 t = group_sum_u64(valid ? acc : 0, rowV);  // rows are valid or not as a whole
            if (valid && (threadIdx.x & (rowV - 1)) == 0) atomicAdd(&s_dot[row], t);
        } else if (valid && acc != 0) {
            atomicAdd(&s_dot[row], acc);
        }
    }
}

// Workgroup `blk` of a.n_blocks; the last one to arrive picks among the winners and scores.  Eight to sixteen wavefronts, the last of
// which waits for the picks while the others scan (n_wg: workgroups that stream, each with a wavefront for routing too).  All of
// it is one chain, so what counts is its trips to memory and, since it runs once, the instructions to fetch: the
// arg-max over a workgroup's traces and the one over the winners are one loop of one wavefront.
template <typename WT>
__device__ __forceinline__ void step_match(const StepMatchArgs& a, const StepRouteArgs& ra, int blk, int n_wg, unsigned char* smem) {
    StepMatchLds& s = *reinterpret_cast<StepMatchLds*>(smem);
    ScoreArgs sc = a.sc;
    sc.cur_idx = s.pick;
    const int tid = threadIdx.x, T = blockDim.x, lane = tid & (kWave - 1), wv = tid / kWave;
    const int LE = sc.L * sc.E;
    const int per = a.per, t0 = min(sc.N, blk * per), nt = min(sc.N - t0, per);
    u64* s_dot = reinterpret_cast<u64*>(smem + sizeof(StepMatchLds));
    u64* s_norm = s_dot + per;
    int32_t* qs = reinterpret_cast<int32_t*>(smem + sizeof(StepMatchLds) + ((size_t)per * 16));
    for (int i = tid; i < nt; i += T) {
        s_dot[i] = 0;
        s_norm[i] = a.norm2[t0 + i];
    }
    for (int i = tid; i < LE; i += T) qs[i] = a.q[i];
    barrier_lds();
    const int Ts = T - kWave, scan_waves = Ts / kWave;
    if (tid < Ts) step_route_rows<WT>(ra, wv * a.n_blocks + blk, a.n_blocks * scan_waves + n_wg, lane);
    if (tid >= Ts) {
        const StepPick p = step_picks<WT, false>(ra, reinterpret_cast<float*>(qs + ((LE + 3) & ~3)), lane);
        if (lane < ra.k) {
            s.pick[lane] = p.e;
            s.pick_w[lane] = p.w;
        }
    } else if (sc.cell_bytes == 4) {
        if (a.vec > 1) step_scan<int32_t, 4>(sc, a.span, a.groups, t0, nt, qs, s_dot);
        else step_scan<int32_t, 1>(sc, a.span, a.groups, t0, nt, qs, s_dot);
    } else {
        if (a.vec > 1) step_scan<uint16_t, 8>(sc, a.span, a.groups, t0, nt, qs, s_dot);
        else step_scan<uint16_t, 1>(sc, a.span, a.groups, t0, nt, qs, s_dot);
    }
    barrier_lds();
    // each pick adds one to its cell of the query
    const size_t row = ((size_t)sc.cur_layer * sc.n_cap + t0) * sc.E;
    auto picked = [&](int i, int j0, int j1) {  // cells of trace i
        u64 sum = 0;
#pragma unroll 8
        for (int j = j0; j < j1; ++j) {
            const int e = s.pick[j];
            const uint32_t v = cell_at(sc.traces, sc.cell_bytes, row + (size_t)i * sc.E + max(e, 0));
            sum += e >= 0 ? v : 0u;
        }
        return sum;
    };
    if (ra.k <= 8) {
        for (int i = tid; i < nt; i += T) s_dot[i] += picked(i, 0, ra.k);
    } else {  // eight picks of a trace a thread (all k by one: 64 picks of 64 experts 90 us a layer with seven trips more, 81 like this)
        for (int p = tid; p < nt * ((ra.k + 7) / 8); p += T) {
            const int c = p / nt, i = p - c * nt;
            atomicAdd(&s_dot[i], picked(i, 8 * c, min(ra.k, 8 * c + 8)));
        }
    }
    if (tid < ra.k && s.pick[tid] >= 0) qs[sc.cur_layer * sc.E + s.pick[tid]] += 1;
    barrier_lds();
    int slot = 0;  // of the pick, in the last wavefront, which has least to do behind the match
    if (wv == 0) {
        Best me = make_best(0, 1, -1);
        bool finish = true;
#pragma unroll 1
        for (int stage = 0; stage < (a.n_blocks > 1 ? 2 : 1); ++stage) {
            if (stage == 1) {  // publish this workgroup's winner; the last one to arrive goes on
                unsigned arrived = 0;
                if (lane == 0) {
                    // (stored past the caches and acknowledged before the count: no write-back of the L2 by a fence)
                    __hip_atomic_store(&a.cand[2 * blk], me.dot, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
                    __hip_atomic_store(&a.cand[2 * blk + 1], me.nt, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
                    __hip_atomic_store(&a.cand_idx[blk], me.idx, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
                    wait_vm_fence<0>();
                    arrived = __hip_atomic_fetch_add(a.ticket, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
                    if (arrived == (unsigned)a.n_blocks - 1) *a.ticket = 0;  // ready for the next launch on this stream
                }
                finish = (int)__builtin_amdgcn_readfirstlane((int)arrived) == a.n_blocks - 1;
                if (!finish) break;
            }
            me = make_best(0, 1, -1);
            for (int i = lane; i < (stage == 0 ? nt : a.n_blocks); i += kWave) {
                u64 dot, norm;
                int idx;
                if (stage == 0) {
                    dot = s_dot[i];
                    norm = s_norm[i];
                    idx = t0 + i;
                } else {
                    dot = __hip_atomic_load(&a.cand[2 * i], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
                    norm = __hip_atomic_load(&a.cand[2 * i + 1], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
                    idx = __hip_atomic_load(&a.cand_idx[i], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
                }
                if (idx >= 0) me = pick(me, make_best(dot, norm, idx));
            }
            me = wave_pick(me);
        }
        if (lane == 0) {
            s.finish = finish;
            s.win = me;
            s.best[0] = me.idx;
        }
    } else if (wv == 1) {  // meanwhile: the query's norm, for the similarity
        u64 nq = 0;
        for (int i = lane; i < LE; i += kWave) nq += (u64)(uint32_t)qs[i] * (uint32_t)qs[i];
        nq = wave_sum_u64_dpp(nq);
        if (lane == 0) s.nq = nq;
    } else if (wv == scan_waves && lane < ra.k) {
        slot = ra.slot_of_row[max(s.pick[lane], 0)];
    }
    barrier_lds();
    if (!s.finish) return;  // uniform
    if (tid == kWave) {
        const float sim = s.win.idx >= 0 ? (float)cosine(s.win.dot, s.nq, s.win.nt) : 0.f;
        a.best[0] = s.win.idx;
        a.best_sim[0] = sim;
        if (a.host) {
            a.host->best = s.win.idx;
            a.host->best_sim = sim;
        }
    }
    // What the step leaves for later calls besides.  Here, and not in the workgroups that stream, since the number below says that
    // all of it is there; the EAM too: the other workgroups that match took their copies of it before they arrived.
    if (wv == scan_waves && lane < ra.k) {
        const int e = s.pick[lane];
        a.idx[lane] = e;
        a.w[lane] = s.pick_w[lane];
        if (e >= 0) a.q[sc.cur_layer * sc.E + e] = qs[sc.cur_layer * sc.E + e];  // one more (Sec. 4.3); a token's picks are distinct
        if (e < 0 && lane == 0) atomicOr(a.flags, 4);
        if (e >= 0 && slot < 0) atomicOr(a.flags, 2);
    }
    score_and_heads<false>(sc, s.score, s.sn, s.best);
    // The host waits for the step by this word, whatever has become of its stream.  Its way over the host link is hidden by the
    // experts (four steps of large ones 502 -> 503 us, of the tiny model 113 -> 113); stored by the reduction kernel it held every step
    // up by 5 us.
    if (a.host) {
        wait_vm_fence<0>();
        barrier_lds();
        if (tid == 0) {
            __threadfence_system();
            __hip_atomic_store(&a.host->seq, a.seq, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_SYSTEM);
        }
    }
}

#endif  // __HIPCC__

}  // namespace moei
