// edge_flat.hpp -- edge-check building blocks shared by the collision
// translation unit and the extension pipeline: endpoint rows, the state count
// of a discretised edge, and the one-kernel edge check.
#pragma once

#include <algorithm>

#include "pipeline.hpp"
#include "st_internal.hpp"

namespace st {

// A space-time state in registers: the configuration in slots 0 .. d-1, zeros
// up to slot kMaxDof - 1, the time in slot kMaxDof whatever d is (a slot that
// depends on d would put the row into scratch memory).

// Both endpoint rows of edge e (rows of d + 1 floats: configuration, then
// time), earlier time first.  All the row loads are issued before the first
// use; a loop that consumed each element as it arrived would wait for every
// load in turn.
__device__ __forceinline__ void load_edge_rows(const float *xa, const float *xb, int64_t e, int d,
                                               float (&A)[kMaxDof + 1], float (&B)[kMaxDof + 1]) {
    const float *pa = xa + e * (d + 1), *pb = xb + e * (d + 1);
    A[kMaxDof] = pa[d];
    B[kMaxDof] = pb[d];
#pragma unroll
    for (int j = 0; j < kMaxDof; ++j) {
        A[j] = j < d ? pa[j] : 0.f;
        B[j] = j < d ? pb[j] : 0.f;
    }
    if (A[kMaxDof] > B[kMaxDof]) {
#pragma unroll
        for (int j = 0; j <= kMaxDof; ++j) {
            const float tmp = A[j];
            A[j] = B[j];
            B[j] = tmp;
        }
    }
}

// States of a discretised edge (Eq. 5 spacing): n = ceil(max(|dq|, v dt) / h),
// at least 1; the count is taken in double precision.
__device__ __forceinline__ int32_t edge_states(const float (&A)[kMaxDof + 1], const float (&B)[kMaxDof + 1], int d,
                                               double v, double h) {
    double D2 = 0.0;
#pragma unroll
    for (int j = 0; j < kMaxDof; ++j) {
        if (j < d) {
            const double dq = (double)B[j] - (double)A[j];
            D2 += dq * dq;
        }
    }
    const double span = fmax(sqrt(D2), v * ((double)B[kMaxDof] - (double)A[kMaxDof]));
    int64_t n = (int64_t)ceil(span / h);
    if (n < 1) n = 1;
    if (n > (1ll << 30)) n = 1ll << 30;
    return (int32_t)n;
}

// State j of an edge of n steps: the endpoint itself for j = n.
__device__ __forceinline__ void edge_state(const float (&A)[kMaxDof + 1], const float (&B)[kMaxDof + 1], int32_t j,
                                           int32_t n, float (&q)[kMaxDof], float &t) {
    const float s = (float)j * (1.0f / (float)n);
    const bool last = j == n;
#pragma unroll
    for (int k = 0; k < kMaxDof; ++k) q[k] = last ? B[k] : fmaf(s, B[k] - A[k], A[k]);
    t = last ? B[kMaxDof] : fmaf(s, B[kMaxDof] - A[kMaxDof], A[kMaxDof]);
}

// ---------------------------------------------------------------------------
// Edge check in one kernel.  A team of waves takes G consecutive edges (G <=
// 64) and decides them (state counts, checks, free / first hit, work counters)
// in phases.  A phase checks the states [lo, lo + width) of every edge of the
// team still without a hit, laid end to end and dealt to the team's waves in
// rounds; the next phase starts behind them, wider.  A team is the whole block,
// or, in launches with many edges for every wave of the device, one wave for
// the first phase (no barriers) and then, for what that leaves, the whole block:
// a wave by itself held up to eight times its share where the long free edges
// lie unevenly (3000 extension edges of the 7-DOF arm 59 us, 37 for the chunked
// kernels, 35 so; 65536 of them 270 and 192).
//
// Bound by VALU issue (a state check of the 6-DOF arm is about 3700
// instructions, 2700 of them sphere pairs) and, with a round or two per wave,
// by its dependent chain.  Most edges that collide do so within their first
// states (two on average for random extensions of the 6-DOF arm, one for the
// 7-DOF arm among 32 obstacles), and a lane that checks a state past its
// edge's first hit is wasted, so the first phase is narrow; what survives it
// is mostly free and needs all its states.  A round with fewer states than
// lanes gives each state 2, 4 or 8 adjacent lanes that share its spheres out
// (arms only), which shortens the chain of the narrow phases.
//
// A lane skips a state above a hit already found for its edge; within a round
// the lanes of one edge form a group of state_hits, and hits merge with an atomic
// minimum; phases run in state order, so the least colliding index
// is exact.
// ---------------------------------------------------------------------------

constexpr int kFlatMaxEdges = 64;  // edges per team at most (one per lane)
constexpr int kFlatMaxShift = 3;   // lanes per state at most (log2)
constexpr int kFlatMaxWidth = 4096;// states of one edge per phase at most
constexpr int kFlatWaves = 8;      // waves of a block with the planner's own edges at most
constexpr int kFlatApiWaves = 12;  // and of one of st_check_edges (three per SIMD, what 168 registers leave room for)

// Dynamic LDS behind the scene: of the block's edges both endpoint rows, state
// counts, least hits and, when the block pools its long edges, the first state
// left and the list of them; per wave the edges that start in its round.
inline __host__ __device__ int flat_words(int edges, int waves, bool pool) {
    return edges * (pool ? 20 : 18) + 64 * waves;
}
inline size_t flat_lds_bytes(int waves, int team, int G, bool pool = false) {
    return (size_t)flat_words(waves / team * G, waves, pool) * sizeof(int32_t);
}

// Inclusive scan over the wave's lanes in six cross-lane steps (row shifts,
// then the rows' last lanes broadcast).
template <class Op>
__device__ __forceinline__ int wave_scan(int x, int identity, Op op) {
    x = op(x, __builtin_amdgcn_update_dpp(identity, x, 0x111, 0xf, 0xf, false));  // row_shr:1
    x = op(x, __builtin_amdgcn_update_dpp(identity, x, 0x112, 0xf, 0xf, false));  // row_shr:2
    x = op(x, __builtin_amdgcn_update_dpp(identity, x, 0x114, 0xf, 0xf, false));  // row_shr:4
    x = op(x, __builtin_amdgcn_update_dpp(identity, x, 0x118, 0xf, 0xf, false));  // row_shr:8
    x = op(x, __builtin_amdgcn_update_dpp(identity, x, 0x142, 0xa, 0xf, false));  // row_bcast:15
    x = op(x, __builtin_amdgcn_update_dpp(identity, x, 0x143, 0xc, 0xf, false));  // row_bcast:31
    return x;
}

// Orders a wave's own LDS accesses across its lanes (they execute in order; this
// keeps the compiler from moving or forwarding them).
__device__ __forceinline__ void wave_lds_fence() {
    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
    __builtin_amdgcn_wave_barrier();
}

// A block's edges, G for every TW waves: the lane's edge e (lane < G; none from E
// on), at most w0 states of an edge in the first phase, no phase that starts at
// state `limit` or above.  POOL (teams of one wave): what the teams leave at the
// limit is checked by the whole block as one team, 64 edges at a time.
// rows(e, A, B) fills both endpoints, earlier time first, and returns false for
// an edge not to check; done(e, n, hit, lo) gets, on the lanes of a team's first
// wave that have an edge that was checked, its state count, its least hit and the
// first state that was left to the caller (above n without a limit or pooled).
template <int KIND, int OT, int OBS, bool POOL, class Rows, class Done>
__device__ __forceinline__ void edge_flat_team(const SceneDev &sc, float4 *lds, int64_t E, int64_t e, int G, int TW,
                                               int w0, int limit, Rows &&rows, Done &&done) {
    __shared__ int s_cnt;
    const int d = sc.d;
    const int wv = uniform(threadIdx.x >> 6), lane = threadIdx.x & 63, nwv = blockDim.x >> 6;
    const int team = wv / TW, NB = nwv / TW * G;
    float4 *s_row = lds + sc.lds_f4;  // edge i of the block: A at [4 i], B at [4 i + 2]
    int32_t *s_n = reinterpret_cast<int32_t *>(s_row + 4 * NB), *s_hit = s_n + NB;
    int32_t *s_lo = s_hit + NB, *s_list = s_lo + NB;  // (pooled blocks)
    int32_t *s_map = s_n + (POOL ? 4 : 2) * NB + 64 * wv;
    // waves of the lane's team, the wave's place in it, the lane's edge of the block
    int W = TW, tw = wv - team * TW, id = team * G + lane;
    bool has = lane < G;
    // the edges' rows first, so that the producer's loads are in flight while
    // other threads stage the scene; the staging's barrier also publishes the
    // rows
    if (tw == 0 && has) {
        int32_t n = -1;
        if (e < E) {
            float A[kMaxDof + 1], B[kMaxDof + 1];
            if (rows(e, A, B)) {
                n = edge_states(A, B, d, sc.v_d, sc.h_d);
                s_row[4 * id] = make_float4(A[0], A[1], A[2], A[3]);
                s_row[4 * id + 1] = make_float4(A[4], A[5], A[6], A[7]);
                s_row[4 * id + 2] = make_float4(B[0], B[1], B[2], B[3]);
                s_row[4 * id + 3] = make_float4(B[4], B[5], B[6], B[7]);
            }
        }
        s_n[id] = n;
        s_hit[id] = kNoHit;
    }
    if (POOL && threadIdx.x == 0) s_cnt = 0;
    stage_obstacles(sc, lds);
    int32_t n_own = has ? s_n[id] : -1, lo = 0;  // (an edge not to check has n = -1)
    int width = w0, pooled = 0;
    for (;;) {
        // the phase's states of the lane's edge and their place
        const int left = n_own - lo + 1;
        int c = 0;
        if (has && left > 0 && lo < limit && __atomic_load_n(&s_hit[id], __ATOMIC_RELAXED) == kNoHit) c = min(left, width);
        const int incl = wave_scan(c, 0, [](int x, int y) { return x + y; });
        const int off = incl - c, T = __builtin_amdgcn_readlane(incl, 63);
        const int m = __popcll(__ballot(c > 0));
        if (W > 1) __syncthreads();  // no wave merges a hit before all have read them
        if (T == 0) {
            if (!POOL) break;
            if (pooled == 0) {
                // the teams' long edges become the block's
                if (has && left > 0 && s_hit[id] == kNoHit) {
                    s_lo[id] = lo;
                    s_list[atomicAdd(&s_cnt, 1)] = id;
                }
                __syncthreads();
                W = nwv;
                tw = wv;
                limit = INT32_MAX;
            }
            const int R = uniform(s_cnt);
            if (pooled >= R) break;
            has = pooled + lane < R;
            id = has ? s_list[pooled + lane] : 0;
            n_own = has ? s_n[id] : -1;
            lo = has ? s_lo[id] : 0;
            width = max(64, 64 * W / min(64, R - pooled));
            pooled += 64;
            continue;
        }
        // lanes per state: what the phase's states leave free
        int shift = 0;
        if (KIND != kTranslate)
            while (shift < kFlatMaxShift && (T << (shift + 1)) <= 64 * W) ++shift;
        const int per = 64 >> shift, part = lane & ((1 << shift) - 1);
        for (int base = tw * per; base < T; base += per * W) {
            // the edge of each state of the round: edges mark the slot they
            // start in, a scan carries the mark on
            s_map[lane] = -1;
            wave_lds_fence();
            if (c > 0 && off < base + per && off + c > base) s_map[max(off - base, 0)] = lane;
            wave_lds_fence();
            const int mark = wave_scan(s_map[lane], -1, [](int x, int y) { return max(x, y); });
            const int k = __shfl(mark, lane >> shift, 64);
            const int o0 = __shfl(off, k, 64), i = __shfl(id, k, 64);
            const int32_t n = __shfl(n_own, k, 64);
            const int g = base + (lane >> shift), j = __shfl(lo, k, 64) + g - o0;
            // a state above a known hit of its edge is not needed
            const bool act = g < T && j <= __atomic_load_n(&s_hit[i], __ATOMIC_RELAXED);
            // the lanes of lower states of this edge in this round
            const uint64_t lower = ((1ull << (lane - part)) - 1ull) & ~((1ull << (max(o0 - base, 0) << shift)) - 1ull);
            const float4 a0 = s_row[4 * i], a1 = s_row[4 * i + 1], b0 = s_row[4 * i + 2], b1 = s_row[4 * i + 3];
            const float A[kMaxDof + 1] = {a0.x, a0.y, a0.z, a0.w, a1.x, a1.y, a1.z, a1.w};
            const float B[kMaxDof + 1] = {b0.x, b0.y, b0.z, b0.w, b1.x, b1.y, b1.z, b1.w};
            float q[kMaxDof];
            float t;
            edge_state(A, B, j, n, q, t);
            const bool hit =
                state_hits<KIND, OT, OBS, KIND == kTranslate ? 1 : kSplitAny>(sc, lds, q, t, act, lower, part, shift);
            if (hit && act && part == 0) atomicMin(&s_hit[i], j);
        }
        if (W > 1) __syncthreads();
        lo += width;
        // at least four times as wide, and half a state per lane
        width = min(kFlatMaxWidth, max(4 * width, 32 * W / m));
    }
    if (POOL) {
        __syncthreads();
        has = lane < G;
        id = team * G + lane;
        n_own = has ? s_n[id] : -1;
        lo = INT32_MAX;
    }
    if (wv == team * TW && has && n_own >= 0) done(e, n_own, s_hit[id], lo);
}

// A block's consecutive edges of an edge list: free / first hit, work counters.
// POOL: teams of one wave for the first phase only.
template <int KIND, int OT, int OBS, bool POOL, class Rows>
__device__ __forceinline__ void edge_flat_body(const EdgeArgs &a, float4 *lds, int bx, Rows &&rows) {
    const int G = a.flat, TW = a.flat_team;
    const int wv = uniform(threadIdx.x >> 6), lane = threadIdx.x & 63, nwv = blockDim.x >> 6;
    const int team = wv / TW, teams = nwv / TW;
    const int64_t e = ((int64_t)bx * teams + team) * G + lane;
    unsigned long long states = 0, edges = 0;
    edge_flat_team<KIND, OT, OBS, POOL>(a.sc, lds, a.E, e, G, TW, a.flat_w0, POOL ? 1 : INT32_MAX, rows,
                                        [&](int64_t, int32_t n, int32_t hit, int32_t) {
                                            const bool fr = hit == kNoHit;
                                            a.free_out[e] = fr ? 1 : 0;
                                            if (a.first_hit) a.first_hit[e] = fr ? -1 : hit;
                                            states = (unsigned long long)(fr ? n : hit) + 1ull;
                                            edges = 1;
                                        });
    if (a.work && wv == team * TW) {
        for (int o = 32; o > 0; o >>= 1) {
            states += __shfl_down(states, o, 64);
            edges += __shfl_down(edges, o, 64);
        }
        if (lane == 0 && edges) {
            atomicAdd(&a.work[0], edges);
            atomicAdd(&a.work[1], states);
        }
    }
}

// Launch shapes of the one-kernel check.  `w0` states per wave in the first
// phase, shared out among the team's edges.
inline void flat_set(EdgeArgs &a, int G, int team, int waves, int w0) {
    a.flat = G;
    a.flat_team = team;
    a.flat_waves = waves;
    a.flat_w0 = std::min(kFlatMaxWidth, std::max(1, w0 * team / G));
}

// st_check_edges.  Up to 8192 edges a block per CU with the whole block as the
// team, E / 256 edges each: of eight waves up to 512 edges, where more waves only
// add to the staging (512 extension edges of the 6-DOF arm 11.4 us, 12.8 with
// twelve), of twelve from there on, three per SIMD (8318 bridge-length edges of
// the 7-DOF arm 110 us, 135 with eight).  Above, a wave takes E / 3072 edges (up
// to 32) and the block pools what its first phase leaves; blocks of twelve
// waves, still one per CU, up to 49152 edges (20000 as above: 204 us, 235 with
// four), of four above, as more than one round of blocks balances better with
// small ones (2^18: 1650 us, 1850 with twelve).
// First phases of one state per lane, and of a state and a half where that takes
// long edges of a few per block (513 as above: 26 us, 37) or extension edges (up
// to 96 states: 3000 of the 7-DOF arm 35 us, 40) in one phase; elsewhere a wider
// one only adds states past a hit (2000 bridge-length edges 51 us, 58).
inline void flat_shape_api(EdgeArgs &a) {
    if (a.E <= 256) {
        flat_set(a, 1, 8, 8, 64);
    } else if (a.E <= 8192) {
        const int waves = a.E <= 512 ? 8 : kFlatApiWaves, G = (int)((a.E + 255) / 256);
        flat_set(a, G, waves, waves, 64);
        const int more = a.flat_w0 + a.flat_w0 / 2;
        if (G <= 3) a.flat_w0 = more;
        else if (more >= 72) a.flat_w0 = std::max(a.flat_w0, std::min(more, 96));
    } else {
        flat_set(a, (int)std::min<int64_t>(32, (a.E + 3071) / 3072), 1, a.E <= 49152 ? kFlatApiWaves : 4, 64);
    }
}

// Extension edges of one problem: 4 x `number` edges (16 by default) per block
// of eight waves, all their states in the first phase (at 4096 samples 98 us
// per iteration of the 6-DOF arm; 102 with a first phase of four states per
// edge, 126 with a wave per 4 edges, whose steering then has four lanes in use),
// fewer edges when the samples would not give every CU a block.
inline void flat_shape_extension(EdgeArgs &a, int number) {
    flat_set(a, (int)std::max<int64_t>(1, std::min<int64_t>(4 * number, (a.E + 255) / 256)), 8, 8, 128);
}

// Extension edges of a batch member: blocks of four waves, with as many edges as
// give the launch's `edges` (all members of the robot's kind) 768 blocks, three
// per CU, within 4 to 16.  A mixed batch of 128 (2 k arm edges per iteration): 204-243
// us per iteration; 203-243 with 4 throughout, 223-258 with 8, 234-264 with 16.  96 arms of 256 samples
// (24 k): 311 us; 398 with 4, 363 with 8.
inline void flat_shape_batch(EdgeArgs &a, int64_t edges) {
    flat_set(a, (int)std::max<int64_t>(4, std::min<int64_t>(16, (edges + 767) / 768)), 4, 4, 64);
}

// The bridge check.  One problem: its advanced workers over 256 blocks of eight
// waves (one block per CU: two do not fit the registers), first phases of 32
// states per wave (most bridges that collide do so within a few states, and a
// narrow phase gives each state several lanes); what is undecided when a phase
// would start at state 128 or above goes to the spread-out check, so that a
// few long bridges do not hold up one block.  6-DOF arm at 4096 samples, five
// problems: 88 to 136 us per iteration; 99 to 140 with one wave and 64 states per
// bridge and chunks of the rest, 86 to 133 (but 115 for 109) with 512 blocks and
// no limit; 7-DOF arm at 8192: 182 to 343; 186 to 354; 196 to 351.  A batch
// member: a block per four samples, at most 2048 in the launch within 16 to 64 per
// member (243 us for the mixed batch with 64, 248 without a bound, 268 with 16; 96
// arms of 256 samples 363 with 64, 333 with 16), no limit (its launch would be one more for
// every scene class): mixed batch of 128 341 us with eight waves per block, 358
// with four, 348 with a limit of 512, 390 with chunks (all with the scans of then).
constexpr int kBridgeBlocks = 256, kBridgeW0 = 32, kBridgeLimit = 128, kBridgeSamplesBatch = 4,
              kBridgeBlocksBatch = 2048;
inline void bridge_shape(BridgeArgs &a) {
    a.blocks = (int)std::max<int64_t>((a.B + kFlatMaxEdges - 1) / kFlatMaxEdges, std::min<int64_t>(kBridgeBlocks, a.B));
    a.w0 = kBridgeW0;
    a.limit = kBridgeLimit;
}
inline void bridge_shape_batch(BridgeArgs &a, int members) {
    const int64_t want = (a.B + kBridgeSamplesBatch - 1) / kBridgeSamplesBatch;
    const int64_t most = std::max(16, std::min(64, kBridgeBlocksBatch / members));
    a.blocks = (int)std::max<int64_t>((a.B + kFlatMaxEdges - 1) / kFlatMaxEdges,
                                      std::min<int64_t>(most, want));
    a.w0 = kBridgeW0;
    a.limit = INT32_MAX;
}
// Its dynamic LDS behind the scene: the team's and one word per edge.
inline size_t bridge_lds_bytes(const BridgeArgs &a) {
    const int G = (int)((a.B + a.blocks - 1) / a.blocks);
    return flat_lds_bytes(kFlatWaves, kFlatWaves, G) + (size_t)G * sizeof(uint32_t);
}

inline int64_t flat_blocks(const EdgeArgs &a) {
    const int64_t per = (int64_t)a.flat * (a.flat_waves / a.flat_team);
    return (a.E + per - 1) / per;
}
inline size_t flat_lds_bytes(const EdgeArgs &a) {
    return flat_lds_bytes(a.flat_waves, a.flat_team, a.flat, a.flat_team == 1);
}

}  // namespace st
