// Pieces of the EAMC match (Sec. 4.5 of the paper) that more than one kernel is made of: 16-byte vectors of stored
// cells times a query's cells, sums of lane groups, and the exact comparison of two candidates.
#pragma once

#include "common.hpp"
#include "wtypes.hpp"

namespace moei {

#if defined(__HIPCC__)

typedef unsigned long long u64;
typedef unsigned __int128 u128;

template <typename CT, int VEC>
struct CellVec;

template <>
struct CellVec<int32_t, 4> {
    using raw = int4;
    static __device__ __forceinline__ raw load(const int32_t* p) { return *reinterpret_cast<const int4*>(p); }
    static __device__ __forceinline__ raw load_once(const int32_t* p) {
        const uint4 v = load_once_16(p);
        return make_int4((int)v.x, (int)v.y, (int)v.z, (int)v.w);
    }
    static __device__ __forceinline__ u64 dot(raw v, const int32_t* q, u64 acc) {
        int4 qq = *reinterpret_cast<const int4*>(q);
        acc += (u64)(uint32_t)v.x * (uint32_t)qq.x;
        acc += (u64)(uint32_t)v.y * (uint32_t)qq.y;
        acc += (u64)(uint32_t)v.z * (uint32_t)qq.z;
        acc += (u64)(uint32_t)v.w * (uint32_t)qq.w;
        return acc;
    }
};

template <>
struct CellVec<int32_t, 1> {
    using raw = int32_t;
    static __device__ __forceinline__ raw load(const int32_t* p) { return *p; }
    static __device__ __forceinline__ raw load_once(const int32_t* p) { return *p; }
    static __device__ __forceinline__ u64 dot(raw v, const int32_t* q, u64 acc) {
        return acc + (u64)(uint32_t)v * (uint32_t)q[0];
    }
};

template <>
struct CellVec<uint16_t, 8> {
    using raw = uint4;
    static __device__ __forceinline__ raw load(const uint16_t* p) { return *reinterpret_cast<const uint4*>(p); }
    static __device__ __forceinline__ raw load_once(const uint16_t* p) { return load_once_16(p); }
    static __device__ __forceinline__ u64 dot(raw v, const int32_t* q, u64 acc) {
        int4 q0 = *reinterpret_cast<const int4*>(q);
        int4 q1 = *reinterpret_cast<const int4*>(q + 4);
        acc += (u64)(v.x & 0xffffu) * (uint32_t)q0.x;
        acc += (u64)(v.x >> 16) * (uint32_t)q0.y;
        acc += (u64)(v.y & 0xffffu) * (uint32_t)q0.z;
        acc += (u64)(v.y >> 16) * (uint32_t)q0.w;
        acc += (u64)(v.z & 0xffffu) * (uint32_t)q1.x;
        acc += (u64)(v.z >> 16) * (uint32_t)q1.y;
        acc += (u64)(v.w & 0xffffu) * (uint32_t)q1.z;
        acc += (u64)(v.w >> 16) * (uint32_t)q1.w;
        return acc;
    }
};

template <>
struct CellVec<uint16_t, 1> {
    using raw = uint16_t;
    static __device__ __forceinline__ raw load(const uint16_t* p) { return *p; }
    static __device__ __forceinline__ raw load_once(const uint16_t* p) { return *p; }
    static __device__ __forceinline__ u64 dot(raw v, const int32_t* q, u64 acc) {
        return acc + (u64)v * (uint32_t)q[0];
    }
};

// Sum of a 64-bit value over each group of `group` consecutive lanes (a power of two up to 64; all 64
// lanes take part; every lane of a group ends with the group's sum): two-word adds with carry over
// DPP exchanges inside a row of 16 lanes, shuffles beyond.
__device__ __forceinline__ u64 add_step_dpp(u64 v, unsigned lo_o, unsigned hi_o) {
    const unsigned lo = (unsigned)v + lo_o;
    const unsigned hi = (unsigned)(v >> 32) + hi_o + (lo < lo_o ? 1u : 0u);
    return ((u64)hi << 32) | lo;
}
#define MOEI_GROUP_STEP(v, ctrl) (v) = add_step_dpp((v), MOEI_DPP_U32((unsigned)(v), ctrl), MOEI_DPP_U32((unsigned)((v) >> 32), ctrl))
__device__ __forceinline__ u64 group_sum_u64(u64 v, int group) {
    if (group >= 2) MOEI_GROUP_STEP(v, 0xB1);    // quad_perm [1,0,3,2]
    if (group >= 4) MOEI_GROUP_STEP(v, 0x4E);    // quad_perm [2,3,0,1]
    if (group >= 8) MOEI_GROUP_STEP(v, 0x141);   // row_half_mirror
    if (group >= 16) MOEI_GROUP_STEP(v, 0x140);  // row_mirror
    if (group >= 32) v += ((u64)__shfl_xor((unsigned)(v >> 32), 16, 64) << 32 | __shfl_xor((unsigned)v, 16, 64));
    if (group >= 64) v += ((u64)__shfl_xor((unsigned)(v >> 32), 32, 64) << 32 | __shfl_xor((unsigned)v, 32, 64));
    return v;
}

struct Best {
    u64 dot;     // <q, T>
    u64 nt;      // |T|^2, never 0 here (an all-zero trace enters as dot 0, nt 1)
    double key;  // dot^2 / nt in fp64: decides all but near ties
    int idx;     // -1: none
};

__device__ __forceinline__ Best make_best(u64 dot, u64 nt, int idx) {
    Best b;
    b.dot = nt ? dot : 0;
    b.nt = nt ? nt : 1;
    b.key = ((double)b.dot * (double)b.dot) / (double)b.nt;
    b.idx = idx;
    return b;
}

// a.dot^2 * b.nt  vs  b.dot^2 * a.nt, exactly, as 192-bit integers.
__device__ __noinline__ int cmp_sim_exact(u64 adot, u64 ant, u64 bdot, u64 bnt) {
    u128 a2 = (u128)adot * adot, b2 = (u128)bdot * bdot;
    u128 al = (u128)(u64)a2 * bnt, ah = (u128)(u64)(a2 >> 64) * bnt + (al >> 64);
    u128 bl = (u128)(u64)b2 * ant, bh = (u128)(u64)(b2 >> 64) * ant + (bl >> 64);
    if (ah != bh) return ah > bh ? 1 : -1;
    u64 all = (u64)al, bll = (u64)bl;
    if (all != bll) return all > bll ? 1 : -1;
    return 0;
}

// The fp64 keys carry a relative error below 2^-50; a gap wider than 2^-48 settles the
// order, anything closer is decided by the exact integer comparison.
__device__ __forceinline__ int cmp_sim(Best a, Best b) {
    const double d = a.key - b.key;
    const double tol = fmax(a.key, b.key) * 0x1p-48;
    if (d > tol) return 1;
    if (d < -tol) return -1;
    return cmp_sim_exact(a.dot, a.nt, b.dot, b.nt);
}

// The better of two candidates, field by field (the structs stay in registers).
__device__ __forceinline__ Best pick(Best a, Best b) {
    bool take_b;
    if (b.idx < 0) {
        take_b = false;
    } else if (a.idx < 0) {
        take_b = true;
    } else {
        const int c = cmp_sim(a, b);
        take_b = c < 0 || (c == 0 && b.idx < a.idx);  // equal similarity: lowest trace index
    }
    Best r;
    r.dot = take_b ? b.dot : a.dot;
    r.nt = take_b ? b.nt : a.nt;
    r.key = take_b ? b.key : a.key;
    r.idx = take_b ? b.idx : a.idx;
    return r;
}

// A candidate moved across lanes by a DPP pattern / read from one lane through scalar registers.
template <int CTRL>
__device__ __forceinline__ Best best_dpp(Best me) {
    auto mv = [](unsigned v) { return MOEI_DPP_U32(v, CTRL); };
    auto mv64 = [&](u64 v) { return ((u64)mv((unsigned)(v >> 32)) << 32) | mv((unsigned)v); };
    Best o;
    o.dot = mv64(me.dot);
    o.nt = mv64(me.nt);
    o.key = __longlong_as_double((long long)mv64((u64)__double_as_longlong(me.key)));
    o.idx = (int)mv((unsigned)me.idx);
    return o;
}
__device__ __forceinline__ Best best_lane(Best me, int lane) {
    auto rd = [&](unsigned v) { return (unsigned)__builtin_amdgcn_readlane((int)v, lane); };
    auto rd64 = [&](u64 v) { return ((u64)rd((unsigned)(v >> 32)) << 32) | rd((unsigned)v); };
    Best o;
    o.dot = rd64(me.dot);
    o.nt = rd64(me.nt);
    o.key = __longlong_as_double((long long)rd64((u64)__double_as_longlong(me.key)));
    o.idx = (int)rd((unsigned)me.idx);
    return o;
}

// The same search on (key, index) alone: three registers per exchange instead of seven.  It is
// final only if no comparison on the way was a near tie (keys within 2^-48 of each other and
// not both zero); `tie` reports that, and the caller then repeats the search with the exact
// comparison.  Two zero keys are two zero similarities: the lower index wins, exactly.
struct KeyIdx {
    double key;
    int idx;
};
__device__ __forceinline__ KeyIdx pick_key(KeyIdx a, KeyIdx b, bool& tie) {
    if (b.idx < 0) return a;
    if (a.idx < 0) return b;
    const double d = a.key - b.key;
    const double tol = fmax(a.key, b.key) * 0x1p-48;
    bool take_b;
    if (d > tol) {
        take_b = false;
    } else if (d < -tol) {
        take_b = true;
    } else if (a.key == 0.0 && b.key == 0.0) {
        take_b = b.idx < a.idx;
    } else {
        tie = true;
        take_b = false;
    }
    KeyIdx r;
    r.key = take_b ? b.key : a.key;
    r.idx = take_b ? b.idx : a.idx;
    return r;
}
template <int CTRL>
__device__ __forceinline__ KeyIdx keyidx_dpp(KeyIdx me) {
    const u64 k = (u64)__double_as_longlong(me.key);
    KeyIdx o;
    o.key = __longlong_as_double((long long)(((u64)MOEI_DPP_U32((unsigned)(k >> 32), CTRL) << 32) | MOEI_DPP_U32((unsigned)k, CTRL)));
    o.idx = (int)MOEI_DPP_U32((unsigned)me.idx, CTRL);
    return o;
}
__device__ __forceinline__ KeyIdx keyidx_lane(KeyIdx me, int lane) {
    const u64 k = (u64)__double_as_longlong(me.key);
    KeyIdx o;
    o.key = __longlong_as_double((long long)(((u64)(unsigned)__builtin_amdgcn_readlane((int)(k >> 32), lane) << 32) |
                                             (unsigned)__builtin_amdgcn_readlane((int)k, lane)));
    o.idx = __builtin_amdgcn_readlane(me.idx, lane);
    return o;
}

__device__ __forceinline__ Best wave_pick_exact(Best me) {
    me = pick(me, best_dpp<0xB1>(me));   // quad_perm [1,0,3,2]
    me = pick(me, best_dpp<0x4E>(me));   // quad_perm [2,3,0,1]
    me = pick(me, best_dpp<0x141>(me));  // row_half_mirror
    me = pick(me, best_dpp<0x140>(me));  // row_mirror
    const Best r0 = best_lane(me, 0), r1 = best_lane(me, 16), r2 = best_lane(me, 32), r3 = best_lane(me, 48);
    return pick(pick(r0, r1), pick(r2, r3));
}

// The wavefront's best candidate, in every lane: DPP inside each row of 16 lanes (the order is
// total, so both partners of an exchange keep the same winner), then the four row winners
// through scalar registers.  All 64 lanes must be active.
__device__ __forceinline__ Best wave_pick(Best me) {
    bool tie = false;
    KeyIdx k{me.key, me.idx};
    k = pick_key(k, keyidx_dpp<0xB1>(k), tie);
    k = pick_key(k, keyidx_dpp<0x4E>(k), tie);
    k = pick_key(k, keyidx_dpp<0x141>(k), tie);
    k = pick_key(k, keyidx_dpp<0x140>(k), tie);
    const KeyIdx r0 = keyidx_lane(k, 0), r1 = keyidx_lane(k, 16), r2 = keyidx_lane(k, 32), r3 = keyidx_lane(k, 48);
    const KeyIdx w = pick_key(pick_key(r0, r1, tie), pick_key(r2, r3, tie), tie);
    if (__ballot(tie) != 0ull) return wave_pick_exact(me);  // uniform
    if (w.idx < 0) return make_best(0, 1, -1);
    // the winner's dot product and norm come from the lane that holds it
    const int owner = __builtin_amdgcn_readfirstlane(__ffsll((long long)__ballot(me.idx == w.idx)) - 1);
    return best_lane(me, owner);
}

__device__ __forceinline__ double cosine(u64 dot, u64 nq, u64 nt) {
    if (nq == 0 || nt == 0) return 0.0;
    return (double)dot / (sqrt((double)nq) * sqrt((double)nt));
}

#endif  // __HIPCC__

}  // namespace moei
