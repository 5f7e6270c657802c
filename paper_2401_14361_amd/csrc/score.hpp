// Scoring of every (layer, expert) cell from the matched traces by the workgroup that finishes the
// match (fused layer step).
#pragma once

#include <type_traits>

#include "kernels.hpp"

namespace moei {

#if defined(__HIPCC__)

typedef unsigned long long u64;
constexpr int kScoreThreads = 1024;
constexpr u64 kNone = ~0ull;

struct ScoreArgs {
    const void* traces;  // [L][n_cap][E]
    int cell_bytes, n_cap, N, L, E;
    const int32_t* best;  // [B]
    int B, cur_layer;
    const int32_t* slot_of;  // [L*E]
    double eps;
    const int32_t* cur_idx;  // [n_cur] experts of the current layer that are about to run, or null
    int n_cur;
    float* P;  // [L*E]
    float* V;  // [L*E]
    u64* keys;     // [2][L*E]: prefetch keys, eviction keys; kNone = not a candidate
    int32_t* n_pf;
    int32_t* n_ev;
    // h_pf / h_ev > 0: the scoring workgroup also writes that many leading entries of each order
    // (select_heads); the complete orders come from priority_rank_kernel over `keys`
    int32_t* pf_order;
    int32_t* ev_order;
    int h_pf, h_ev;
    // pinned host memory that receives what the synchronous layer step reads on the host (or null):
    // matched trace, list lengths, the heads, and - for the prefetch admission - the eviction scores
    int32_t* host_best;
    int32_t* host_n;        // [2]: n_pf, n_ev
    int32_t* host_pf_head;
    int32_t* host_ev_head;
    float* host_V;          // [L*E] or null
    // a host that polls instead of waiting for an event: after host_best has been written (and made
    // visible to the host) the step's number goes to *host_seq (pinned, or null)
    int32_t* host_seq;
    int32_t seq;
};

__device__ __forceinline__ uint32_t cell_at(const void* traces, int cell_bytes, size_t i) {
    return cell_bytes == 4 ? (uint32_t) reinterpret_cast<const int32_t*>(traces)[i]
                           : (uint32_t) reinterpret_cast<const uint16_t*>(traces)[i];
}

// What the workgroup that finishes a match does besides: nothing, or the scoring of a model of up to / of more than
// kKeyLdsCells cells.
enum class Scoring { none, small, large };
// Models of up to kKeyLdsCells cells (LARGE = false) keep a copy of the keys in LDS for the head selection, which
// then needs no second trip to memory.
constexpr int kKeyLdsCells = 2048;
struct KeyLds {
    u64 k[2][kKeyLdsCells];
};

// Adds the lanes' candidate counts.  (Every lane of the workgroup adding to the two words itself took 3.9 us.)
__device__ __forceinline__ void count_candidates(int my_pf, int my_ev, int* s_n) {
    const unsigned pf = wave_sum_u32_dpp((unsigned)my_pf), ev = wave_sum_u32_dpp((unsigned)my_ev);
    if ((threadIdx.x & (kWave - 1)) == 0) {
        atomicAdd(&s_n[0], (int)pf);
        atomicAdd(&s_n[1], (int)ev);
    }
}

// One thread: the candidate counts and what the host reads first.
__device__ __forceinline__ void publish_counts(const ScoreArgs& a, const int* s_n, const int* s_best) {
    *a.n_pf = s_n[0];
    *a.n_ev = s_n[1];
    if (a.host_n) {
        a.host_n[0] = s_n[0];
        a.host_n[1] = s_n[1];
    }
    if (a.host_best) *a.host_best = s_best[0];
    if (a.host_seq) {
        __threadfence_system();  // the matched trace is in host memory before the number that announces it
        __hip_atomic_store(a.host_seq, a.seq, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_SYSTEM);
    }
}

// Models of up to kKeyLdsCells cells: called by all threads (at least 512) of ONE workgroup: scores for every cell, a 64-bit sort
// key per cell and list (kNone where the cell is not a candidate) and the two candidate counts.  s_n[2] and
// s_best[kMaxMatchBatch] are LDS; the caller has put the matched trace indices (-1 = none) into s_best, before a barrier; s_cell holds
// kKeyLdsCells words.
// The workgroup is alone on its compute unit and goes through this code once, so what counts is the trips to memory and the
// instructions to fetch: all cells are requested together, whatever rows they belong to, then one short loop runs over the
// rows, 0.7 us each (26 x 64 cells by 16 wavefronts: 3.1 us, and 6.1 with a wavefront per row, its loads in the loop, and the
// counts added up by every lane).
__device__ __forceinline__ void score_cells_small(const ScoreArgs& a, int* s_n, const int* s_best, KeyLds& keys, uint32_t* s_cell) {
    const int tid = threadIdx.x, T = blockDim.x, lane = tid & (kWave - 1);
    const int L = a.L, E = a.E, l = a.cur_layer, LE = L * E;
    constexpr int kRounds = kKeyLdsCells / 512;
    constexpr uint32_t kResident = 0x80000000u;  // (an aggregate of 16 cells of 24 bits takes 28)
    uint32_t t[kRounds];
    size_t at[kRounds];
    const float inv = 1.0f / (float)E;
#pragma unroll
    for (int r = 0; r < kRounds; ++r) {
        const int f = min(tid + r * T, LE - 1);
        const int i = (int)(((float)f + 0.5f) * inv);  // f / E: (f + 0.5) / E is at least 0.5 / E away from an integer, the error of the product less than 2^-11 / E
        t[r] = a.slot_of[f] >= 0 ? kResident : 0u;
        at[r] = (size_t)i * (a.n_cap - 1) * E + f;  // the cell of trace 0
    }
    const int cur = lane < a.n_cur ? a.cur_idx[lane] : -1;  // lane m holds pick m of the current layer
#pragma unroll 1
    for (int b = 0; b < a.B; ++b) {
        const int n = s_best[b];
        if (n < 0) continue;  // uniform
#pragma unroll
        for (int r = 0; r < kRounds; ++r) t[r] += cell_at(a.traces, a.cell_bytes, at[r] + (size_t)n * E);
    }
    if (tid < 2) s_n[tid] = 0;
#pragma unroll
    for (int r = 0; r < kRounds; ++r)
        if (tid + r * T < LE) s_cell[tid + r * T] = t[r];
    barrier_lds();
    int my_ev = 0, my_pf = 0;
#pragma unroll 1
    for (int i = tid / kWave; i < L; i += T / kWave) {
        u64 R = 0;
#pragma unroll 1
        for (int j = lane; j - lane < E; j += kWave) {
            const uint32_t c = j < E ? s_cell[i * E + j] & ~kResident : 0u;
            R += wave_sum_u32_dpp(c & 0xffffu) + ((u64)wave_sum_u32_dpp(c >> 16) << 16);
        }
        const double den = (double)(R ? R : 1ull) * (double)L;
#pragma unroll 1
        for (int j = lane; j - lane < E; j += kWave) {
            bool excluded = false;  // is expert j one of the current picks?
            if (i == l)
                for (int m = 0; m < a.n_cur; ++m) excluded |= __builtin_amdgcn_readlane(cur, m) == j;
            if (j >= E) continue;
            const int f = i * E + j;
            const uint32_t c = s_cell[f];
            const double td = (double)(c & ~kResident);
            const double v = ((td + a.eps) * (double)(L - i)) / den;
            double p = 0.0;
            if (i > l && R > 0) p = (td * (double)(L - i + l)) / den;
            a.P[f] = (float)p;
            a.V[f] = (float)v;
            if (a.host_V) a.host_V[f] = (float)v;
            // positive doubles order like their bit patterns; ~bits turns descending into ascending
            const bool is_pf = i > l && p > 0.0 && !(c & kResident);
            const bool is_ev = (c & kResident) && !excluded;
            const u64 key_p = is_pf ? ~(u64)__double_as_longlong(p) : kNone;
            const u64 key_v = is_ev ? (u64)__double_as_longlong(v) : kNone;
            a.keys[f] = keys.k[0][f] = key_p;
            a.keys[LE + f] = keys.k[1][f] = key_v;
            my_pf += is_pf;
            my_ev += is_ev;
        }
    }
    count_candidates(my_pf, my_ev, s_n);
    barrier_lds();
    if (tid == 0) publish_counts(a, s_n, s_best);
}

// More cells than that: called by all kScoreThreads threads of ONE workgroup.  One wavefront per layer row, the next row's loads out before a row is scored (the trip to the
// matched cells is what a row costs, and beside the streaming FFN it is a long one).  s_n[2] and
// s_best[kMaxMatchBatch] are LDS; the caller has put the matched trace indices (-1 = none) into s_best.
__device__ __forceinline__ void score_cells_large(const ScoreArgs& a, int* s_n, const int* s_best) {
    u64 *kp = a.keys, *kv = a.keys + a.L * a.E;
    const int tid = threadIdx.x;
    const int lane = tid & (kWave - 1), wv = tid / kWave;
    const int L = a.L, E = a.E, l = a.cur_layer;
    if (tid < 2) s_n[tid] = 0;
    __syncthreads();
    constexpr int kPerLane = 4;  // cells of a row held in registers (rows up to 256 wide)
    struct Row {
        u64 tv[kPerLane];
        int sv[kPerLane];
        u64 rsum;
        int cur;  // lane m holds pick m of the current layer (used for row l only)
    };
    int my_ev = 0, my_pf = 0;
    auto cell_sum = [&](int i, int j) {
        u64 t = 0;
        for (int b = 0; b < a.B; ++b) {
            const int n = s_best[b];
            if (n >= 0) t += cell_at(a.traces, a.cell_bytes, ((size_t)i * a.n_cap + n) * E + j);
        }
        return t;
    };
    // all of a row's loads go out together: current picks, residency, matched cells (these last: their sum over
    // the traces is waited for)
    auto load_row = [&](int i, Row& w) {
        w.cur = -1;
        if (i == l && lane < a.n_cur) w.cur = a.cur_idx[lane];
#pragma unroll
        for (int r = 0; r < kPerLane; ++r) {
            const int j = lane + r * kWave;
            w.sv[r] = -1;
            if (r * kWave < E && j < E) w.sv[r] = a.slot_of[(size_t)i * E + j];
        }
        w.rsum = 0;
#pragma unroll
        for (int r = 0; r < kPerLane; ++r) {
            const int j = lane + r * kWave;
            w.tv[r] = 0;
            if (r * kWave < E) {  // uniform
                if (j < E) w.tv[r] = cell_sum(i, j);
                w.rsum += w.tv[r];
            }
        }
        for (int j = lane + kPerLane * kWave; j < E; j += kWave) w.rsum += cell_sum(i, j);
    };
    auto score_row = [&](int i, const Row& w) {
        const u64 R = wave_sum_u64_dpp(w.rsum);
        const double den = (double)(R ? R : 1ull) * (double)L;
        auto score = [&](int j, u64 t, int slot) {
            // is expert j one of the current picks?  (all 64 lanes take part in the shuffles)
            bool excluded = false;
            if (i == l) {
                for (int m0 = 0; m0 < a.n_cur; m0 += kWave) {
                    int c = w.cur;
                    if (m0 > 0) c = (m0 + lane < a.n_cur) ? a.cur_idx[m0 + lane] : -1;
                    const int lim = min(kWave, a.n_cur - m0);
                    for (int m = 0; m < lim; ++m) excluded |= (__shfl(c, m, kWave) == j);
                }
            }
            if (j >= E) return;
            const size_t f = (size_t)i * E + j;
            const double td = (double)t;
            const double v = ((td + a.eps) * (double)(L - i)) / den;
            double p = 0.0;
            if (i > l && R > 0) p = (td * (double)(L - i + l)) / den;
            a.P[f] = (float)p;
            a.V[f] = (float)v;
            if (a.host_V) a.host_V[f] = (float)v;
            // positive doubles order like their bit patterns; ~bits turns descending into ascending
            const bool is_pf = i > l && p > 0.0 && slot < 0;
            const bool is_ev = slot >= 0 && !excluded;
            kp[f] = is_pf ? ~(u64)__double_as_longlong(p) : kNone;
            kv[f] = is_ev ? (u64)__double_as_longlong(v) : kNone;
            my_pf += is_pf;
            my_ev += is_ev;
        };
#pragma unroll
        for (int r = 0; r < kPerLane; ++r)
            if (r * kWave < E) score(lane + r * kWave, w.tv[r], w.sv[r]);  // uniform
        for (int r = kPerLane; r * kWave < E; ++r) {
            const int j = lane + r * kWave;
            score(j, j < E ? cell_sum(i, j) : 0, j < E ? a.slot_of[(size_t)i * E + j] : -1);
        }
    };
    constexpr int kWaves = kScoreThreads / kWave;
    Row row;
    for (int i = wv - kWaves; i < L; i += kWaves) {  // (the code of a row stands here once)
        Row next;
        if (i + kWaves < L) load_row(i + kWaves, next);
        if (i >= 0) score_row(i, row);
        row = next;
    }
    count_candidates(my_pf, my_ev, s_n);
    __syncthreads();  // (the keys are read from memory next)
    if (tid == 0) publish_counts(a, s_n, s_best);
}

// ---- heads of the two orders
// Alg. 1 evicts the expert of lowest priority: serving one layer's k picks consumes at most k entries
// of the eviction order, and prefetching looks at `depth` entries of the prefetch order.  The layer
// step therefore selects only those heads (h rounds of a workgroup-wide arg-min over the keys that
// score_cells has left in global memory); the complete orders are ranked from the same keys by
// priority_rank_kernel when somebody asks for them.
struct KeyId {
    u64 k;
    int id;
};
__device__ __forceinline__ KeyId keyid_min(KeyId a, KeyId b) {
    const bool take_b = b.k < a.k || (b.k == a.k && b.id < a.id);
    KeyId r;
    r.k = take_b ? b.k : a.k;
    r.id = take_b ? b.id : a.id;
    return r;
}
// smallest (key, id) of the wavefront, in every lane (all 64 lanes active): three one-word minima -
// the key's high word, the low word among the lanes that hold that high word, the id among the
// lanes that hold that key
__device__ __forceinline__ KeyId wave_keyid_min(KeyId v) {
    const unsigned hi = (unsigned)(v.k >> 32), lo = (unsigned)v.k;
    const unsigned mh = wave_min_u32_dpp(hi);
    const unsigned ml = wave_min_u32_dpp(hi == mh ? lo : 0xffffffffu);
    const unsigned mi = wave_min_u32_dpp((hi == mh && lo == ml) ? (unsigned)v.id : 0x7fffffffu);
    return KeyId{((u64)mh << 32) | ml, (int)mi};
}

// Wavefronts that search one list, and keys a lane keeps in registers: up to kKeyLdsCells cells four (one per SIMD) and 8;
// up to 10,240 cells eight (half of the workgroup) and 20.  See select_heads.
template <bool LARGE>
struct Sel {
    static constexpr int kWaves = LARGE ? 8 : 4;
    static constexpr int kThreads = kWaves * kWave;
    static constexpr int kOwn = LARGE ? 20 : 8;
};
constexpr int kHeadMax = 96;                     // most entries of a head (picks + prefetch candidates)
static_assert(2 * Sel<true>::kThreads <= kScoreThreads, "both lists are searched at once");
static_assert(Sel<false>::kOwn * Sel<false>::kThreads >= kKeyLdsCells, "a small model's keys fit the registers");
template <bool LARGE>
struct ScoreLds {
    union {
        struct {
            u64 key[2][Sel<LARGE>::kWaves * kHeadMax];  // candidates of a list: wavefront w's at w * (entries asked for)
            int id[2][Sel<LARGE>::kWaves * kHeadMax];
        };
        uint32_t cell[LARGE ? 1 : kKeyLdsCells];  // before them
    };
    std::conditional_t<LARGE, char, KeyLds> keys;
};

// The h smallest (key, flat id) pairs of the calling wavefront's cells ltid, ltid + STRIDE, ... of one list,
// ascending, to okey / oid: h rounds of a DPP arg-min, no barrier - what remains after a round is what
// lies after its winner, and only the lane that held the winner looks through its cells again.  OWN:
// keys of a lane held in registers, all requested together (0: read again each time).
template <int STRIDE, int OWN>
__device__ __forceinline__ void wave_head(const u64* keys, int LE, int ltid, int lane, int want, u64* okey, int* oid) {
    u64 mine[OWN > 0 ? OWN : 1];
#pragma unroll
    for (int r = 0; r < OWN; ++r) {
        const int f = ltid + r * STRIDE;
        mine[r] = f < LE ? keys[f] : kNone;
    }
    // a lane keeps its two best remaining cells: it looks through its cells again only where it has lost both.  (Key and
    // id each by themselves: a choice between two structs is one between their addresses, and both lie in private memory then, a trip
    // there for every comparison.)
    bool have_last = false;
    KeyId last{0, -1};
    u64 cur_k = kNone, nxt_k = kNone;
    int cur_id = 0x7fffffff, nxt_id = 0x7fffffff;
    int known = 0;
    for (int round = 0; round < want; ++round) {
        if (known == 0) {
            cur_k = nxt_k = kNone;
            cur_id = nxt_id = 0x7fffffff;
            auto consider = [&](u64 k, int f) {
                if (k == kNone) return;
                if (have_last && (k < last.k || (k == last.k && f <= last.id))) return;
                const bool first = k < cur_k || (k == cur_k && f < cur_id);
                const bool second = k < nxt_k || (k == nxt_k && f < nxt_id);
                nxt_k = first ? cur_k : (second ? k : nxt_k);
                nxt_id = first ? cur_id : (second ? f : nxt_id);
                cur_k = first ? k : cur_k;
                cur_id = first ? f : cur_id;
            };
            if constexpr (OWN > 0) {
#pragma unroll
                for (int r = 0; r < OWN; ++r) consider(mine[r], ltid + r * STRIDE);
            } else {
                for (int f = ltid; f < LE; f += STRIDE) consider(keys[f], f);
            }
            known = 2;
        }
        const KeyId w = wave_keyid_min(KeyId{cur_k, cur_id});
        if (lane == 0) {
            okey[round] = w.k;
            oid[round] = w.id;
        }
        last = w;
        have_last = true;
        if (cur_id == w.id) {  // this lane's best has been taken: its next one
            cur_k = nxt_k;
            cur_id = nxt_id;
            --known;
        }
    }
}

// All threads of the scoring workgroup (at least 2 * Sel<LARGE>::kThreads) call, after score_cells (whose closing barrier
// has made the keys visible).  The first kWaves wavefronts search the prefetch list, the next as many the eviction
// list, others only meet the barrier.  First every wavefront extracts the h smallest pairs of its own cells, then the
// list's first wavefront the h smallest of those kWaves h candidates the same way.
// Writes pf_order[0 .. min(h_pf, n_pf)) and ev_order[0 .. min(h_ev, n_ev)).
// A chain of dependent steps, so what counts is their number: with four wavefronts a list and eight keys in
// registers, every round over 9,440 cells was one more trip to memory per 256 of them, and the finishing workgroup of the
// match took 60.8 us (59 x 160 cells, heads of 6 and 0 entries), 260 with a prefetch depth of 32; with eight and 20 keys 34.0
// and 90.1, and with a lane's two best cells kept as well 31.4 and 74.  Few cells are searched by four: with eight a list has
// twice the candidates to merge (26 x 64 cells, depth 32: 55.0
// us, with four 47.0, now 36.9), and both forms in one kernel are more than twice the instructions to fetch (4 x 8 cells 9.0 us, in a
// kernel of their own 8.4; 32 x 8 cells 16.0 and 15.2, now 13.9).
template <bool LARGE>
__device__ __forceinline__ void select_heads(const ScoreArgs& a, const u64* kp, const u64* kv, const int* s_n, ScoreLds<LARGE>& hl) {
    constexpr int kSelWaves = Sel<LARGE>::kWaves, kSelThreads = Sel<LARGE>::kThreads, kOwn = Sel<LARGE>::kOwn;
    const int tid = threadIdx.x;
    const int LE = a.L * a.E;
    const int list = tid / kSelThreads;
    const int ltid = tid % kSelThreads;
    const int lane = tid & (kWave - 1), lwave = ltid / kWave;
    const u64* keys = list == 0 ? kp : kv;
    int32_t* out = list == 0 ? a.pf_order : a.ev_order;
    int32_t* host_out = list == 0 ? a.host_pf_head : a.host_ev_head;
    const int want = list > 1 ? 0 : min(list == 0 ? min(a.h_pf, s_n[0]) : min(a.h_ev, s_n[1]), kHeadMax);
    if (want > 0) {  // uniform over the wavefront
        u64* okey = hl.key[list] + lwave * want;
        int* oid = hl.id[list] + lwave * want;
        if (!LARGE || LE <= kOwn * kSelThreads)
            wave_head<kSelThreads, kOwn>(keys, LE, ltid, lane, want, okey, oid);
        else
            wave_head<kSelThreads, 0>(keys, LE, ltid, lane, want, okey, oid);
    }
    barrier_lds();
    const int total = kSelWaves * want;
    if (want > 0 && lwave == 0 && total <= kWave) {
        // a candidate per lane: its place is the number of candidates before it (all pairs are different, and the rounds
        // below are a chain of want arg-mins)
        const u64* ck = hl.key[list];
        const int* ci = hl.id[list];
        const KeyId me = lane < total ? KeyId{ck[lane], ci[lane]} : KeyId{kNone, 0x7fffffff};
        int before = 0;
#pragma unroll 8
        for (int c = 0; c < total; ++c) before += (int)(ck[c] < me.k) | ((int)(ck[c] == me.k) & (int)(ci[c] < me.id));
        if (me.k != kNone && before < want) {
            out[before] = me.id;
            if (host_out) host_out[before] = me.id;
        }
    } else if (want > 0 && lwave == 0) {
        // kSelWaves * want candidates, lane-major: candidate c sits in lane c % 64
        constexpr int kPer = (kSelWaves * kHeadMax + kWave - 1) / kWave;
        KeyId cand[kPer];
#pragma unroll
        for (int r = 0; r < kPer; ++r) {
            const int c = lane + r * kWave;
            cand[r] = c < total ? KeyId{hl.key[list][c], hl.id[list][c]} : KeyId{kNone, 0x7fffffff};
        }
        bool have_last = false;
        KeyId last{0, -1};
        for (int round = 0; round < want; ++round) {
            KeyId cur{kNone, 0x7fffffff};
#pragma unroll
            for (int r = 0; r < kPer; ++r) {
                if (r * kWave < total) {  // uniform
                    const KeyId c = cand[r];
                    const bool taken = have_last && (c.k < last.k || (c.k == last.k && c.id <= last.id));
                    if (c.k != kNone && !taken) cur = keyid_min(cur, c);
                }
            }
            const KeyId w = wave_keyid_min(cur);
            if (lane == 0 && w.k != kNone) {
                out[round] = w.id;
                if (host_out) host_out[round] = w.id;
            }
            last = w;
            have_last = true;
        }
    }
}

// Scoring, then the heads of the orders when the caller has asked for them.  LARGE: more than kKeyLdsCells cells.
template <bool LARGE>
__device__ __forceinline__ void score_and_heads(const ScoreArgs& a, ScoreLds<LARGE>& sl, int* s_n, const int* s_best) {
    const u64 *kp = a.keys, *kv = a.keys + a.L * a.E;
    if constexpr (LARGE) {
        score_cells_large(a, s_n, s_best);
    } else {
        score_cells_small(a, s_n, s_best, sl.keys, sl.cell);
        kp = sl.keys.k[0];
        kv = sl.keys.k[1];
    }
    if (a.h_pf > 0 || a.h_ev > 0) select_heads<LARGE>(a, kp, kv, s_n, sl);
}

#endif

// priority.hip
ScoreArgs make_score_args(const moei_eamc* c, const int32_t* d_best, int B, int cur_layer, const int32_t* d_slot_of,
                          float eps, const int32_t* d_cur_idx, int n_cur, float* d_prefetch, float* d_evict,
                          int32_t* d_n_pf, int32_t* d_n_ev);
// the complete orders from the keys score_cells has left in d_keys[2][L*E]
int launch_priority_rank(const moei_model_desc& d, const unsigned long long* d_keys, const int32_t* d_n_pf,
                         const int32_t* d_n_ev, int32_t* d_pf_order, int32_t* d_ev_order, hipStream_t s);
// match.hip: the match, and - if `score` is given (B must be 1) - the scoring of the matched
// trace by the workgroup that finishes the match, in the same launch
int launch_match(const moei_eamc* c, const int32_t* d_eam, int B, int layer_hi, int32_t* d_best, float* d_best_sim,
                 float* d_sims, const ScoreArgs* score, hipStream_t s);
// the m most similar traces of one query; `score` (with B = m) scores their aggregate
int launch_match_topm(const moei_eamc* c, const int32_t* d_eam, int layer_hi, int m, int32_t* d_top, float* d_top_sim,
                      float* d_sims, const ScoreArgs* score, hipStream_t s);

}  // namespace moei
