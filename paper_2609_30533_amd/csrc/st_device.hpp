// st_device.hpp -- device-side data layout and collision primitives (gfx950).
//
// Layout in HBM (all owned by the problem handle):
//   scene:  one image, staged into LDS as it is: the obstacle segment table
//           [O_pad][n_seg][2] float4 pre-scaled by -2: (-2 p_k, t_k) and
//           (-2 v_k, span_k); spheres sorted by link [S] float4 (x, y, z, r);
//           waypoint times ([n_seg+1], or [O_pad][n_seg+1] when obstacles
//           differ); the spheres' world centres at q_g [S]; fixed boxes [4 each];
//           the configuration box and one record per link.  Obstacle radii
//           [O_pad] (0 for padding obstacles) are read as scalars.
//   trees:  SoA x[d+1][total] (configuration rows, then time), parent[total],
//           cost[total], rootT[total]; pool p occupies [base(p), base(p)+cap(p)).
//
// The collision test keeps one space-time state per lane.  Forward kinematics
// runs in registers; the DH constants and the sphere offsets are staged in LDS
// and read as broadcasts; obstacle centres at the lane's own time come from the
// segment table, also staged in LDS.  A pair
// collides iff |c - o| < r_s + r_o + eps, evaluated in expanded form as a
// minimum over the obstacle tile (sphere_clear).
#pragma once

#include <hip/hip_runtime.h>
#include <type_traits>
#include <stdint.h>

namespace st {

constexpr int kMaxDof = 7;
constexpr int kWave = 64;

// Robot kinds as kernel template arguments: kDHStatic is an arm whose state
// test also covers its listed link pairs and the fixed boxes.
enum { kTranslate = 0, kDH = 1, kDHStatic = 2 };
enum { kObsShared = 0, kObsGeneric = 1 };

// Every robot/obstacle pair is tested against (r_s + r_o + kClearanceEps)^2:
// a state accepted in single precision then also clears the contact distance
// in double precision (the FP32 error of a sphere centre is ~1e-6 m).
constexpr double kClearanceEps = 2e-5;

struct SceneDev {
    int d, kind, S, O, O_pad, n_seg, obs_mode, lds_f4;  // lds_f4: float4 slots of the image
    // float4 offsets in the image: spheres, waypoint times, sphere centres at
    // q_g, boxes, constants (the segment table is at 0)
    int lds_sph, lds_t, lds_goal, lds_box, lds_const;
    int ot;                      // obstacles per register tile (4, 8 or 16; divides O_pad)
    float v, H, h;
    double v_d, h_d;
    float q_lo[8], q_hi[8], q_s[8], q_g[8];
    // static geometry (arms): boxes as 4 float4 rows: (axis_a, -axis_a . centre)
    // for a = 0..2, then (half extents, 0).  goal_blocked: q_g fails the static
    // terms.
    int stat, n_box, n_pair, goal_blocked;
    unsigned last_pair;         // 4 bits per link la: the last link lb of a listed pair (la, lb), or 0
    float r_uni;                // the common obstacle radius, or -1 when radii differ
    const float4 *image;        // [lds_f4]
    const float *ro;            // [O_pad] obstacle radii (0 for padding obstacles)
};

// Constants of the image (float4 slots from lds_const): the box's lower and
// upper corners (two slots each), then kLinkRec slots per link l = 0 .. d:
//   (a, cos alpha, sin alpha, d) of joint l (the one before link l; l > 0)
//   (theta0 of joint l, first sphere, one past the last sphere, self-pair mask),
//       the last three as integers; mask bit la = link pair (la, l) is tested
//   the link's bounding sphere (link frame centre, radius)
// They are read from LDS, the next link's while one is checked: as scalar
// loads from the kernel arguments each was waited for where it was used, and
// four fifths of the wave cycles of a launch with few states were such waits.
constexpr int kBoxRec = 4, kLinkRec = 3;
inline __host__ __device__ int const_f4(int d) { return kBoxRec + kLinkRec * (d + 1); }

struct LinkRec {
    float a, ca, sa, dd, t0;
    int s0, s1;
    unsigned mask;
    float4 bs;
};

__device__ __forceinline__ LinkRec link_rec(const SceneDev &sc, const float4 *lds, int l) {
    const float4 *r = lds + sc.lds_const + kBoxRec + kLinkRec * l;
    const float4 u = r[0], w = r[1];
    LinkRec k;
    k.a = u.x; k.ca = u.y; k.sa = u.z; k.dd = u.w;
    k.t0 = w.x;
    k.s0 = __float_as_int(w.y);
    k.s1 = __float_as_int(w.z);
    k.mask = (unsigned)__float_as_int(w.w);
    k.bs = r[2];
    return k;
}

// A value that is the same in every lane, as a scalar.
__device__ __forceinline__ int uniform(int v) { return __builtin_amdgcn_readfirstlane(v); }

// Stage the scene image into LDS, four loads of a thread in flight together
// (an index past the end repeats the last slot, so no load is guarded).
// Every thread of the block must call it.
__device__ __forceinline__ void stage_obstacles(const SceneDev &sc, float4 *lds) {
    const int bd = blockDim.x, last = sc.lds_f4 - 1;
    const float4 *src = sc.image;
    for (int i = threadIdx.x; i <= last; i += 4 * bd) {
        const int j = min(i + bd, last), k = min(i + 2 * bd, last), l = min(i + 3 * bd, last);
        const float4 v0 = src[i], v1 = src[j], v2 = src[k], v3 = src[l];
        lds[i] = v0;
        lds[j] = v1;
        lds[k] = v2;
        lds[l] = v3;
    }
    __syncthreads();
}

// World frame of a link of the chain: rotation (row-major) and origin.
struct Frame {
    float R00, R01, R02, R10, R11, R12, R20, R21, R22, p0, p1, p2;
};

__device__ __forceinline__ void frame_identity(Frame &f) {
    f.R00 = 1.f; f.R01 = 0.f; f.R02 = 0.f;
    f.R10 = 0.f; f.R11 = 1.f; f.R12 = 0.f;
    f.R20 = 0.f; f.R21 = 0.f; f.R22 = 1.f;
    f.p0 = 0.f; f.p1 = 0.f; f.p2 = 0.f;
}

// T <- T * Rz(theta_j + q_j) Tz(d_j) Tx(a_j) Rx(alpha_j) (standard DH, the joint
// before link record k).
__device__ __forceinline__ void dh_compose(const LinkRec &k, float qj, Frame &f) {
    float st_, ct;
    __sincosf(qj + k.t0, &st_, &ct);
    const float ca = k.ca, sa = k.sa;
    const float a = k.a, dd = k.dd;
    float u, w;
    u = fmaf(f.R00, ct, f.R01 * st_); w = fmaf(f.R01, ct, -f.R00 * st_);
    f.p0 = fmaf(a, u, fmaf(dd, f.R02, f.p0));
    f.R00 = u; f.R01 = fmaf(ca, w, sa * f.R02); f.R02 = fmaf(ca, f.R02, -sa * w);
    u = fmaf(f.R10, ct, f.R11 * st_); w = fmaf(f.R11, ct, -f.R10 * st_);
    f.p1 = fmaf(a, u, fmaf(dd, f.R12, f.p1));
    f.R10 = u; f.R11 = fmaf(ca, w, sa * f.R12); f.R12 = fmaf(ca, f.R12, -sa * w);
    u = fmaf(f.R20, ct, f.R21 * st_); w = fmaf(f.R21, ct, -f.R20 * st_);
    f.p2 = fmaf(a, u, fmaf(dd, f.R22, f.p2));
    f.R20 = u; f.R21 = fmaf(ca, w, sa * f.R22); f.R22 = fmaf(ca, f.R22, -sa * w);
}

// Frame of link b expressed in the frame of link a: R = Ra^T Rb,
// p = Ra^T (pb - pa).
__device__ __forceinline__ void frame_relative(const Frame &a, const Frame &b, Frame &m) {
    m.R00 = fmaf(a.R00, b.R00, fmaf(a.R10, b.R10, a.R20 * b.R20));
    m.R01 = fmaf(a.R00, b.R01, fmaf(a.R10, b.R11, a.R20 * b.R21));
    m.R02 = fmaf(a.R00, b.R02, fmaf(a.R10, b.R12, a.R20 * b.R22));
    m.R10 = fmaf(a.R01, b.R00, fmaf(a.R11, b.R10, a.R21 * b.R20));
    m.R11 = fmaf(a.R01, b.R01, fmaf(a.R11, b.R11, a.R21 * b.R21));
    m.R12 = fmaf(a.R01, b.R02, fmaf(a.R11, b.R12, a.R21 * b.R22));
    m.R20 = fmaf(a.R02, b.R00, fmaf(a.R12, b.R10, a.R22 * b.R20));
    m.R21 = fmaf(a.R02, b.R01, fmaf(a.R12, b.R11, a.R22 * b.R21));
    m.R22 = fmaf(a.R02, b.R02, fmaf(a.R12, b.R12, a.R22 * b.R22));
    const float dx = b.p0 - a.p0, dy = b.p1 - a.p1, dz = b.p2 - a.p2;
    m.p0 = fmaf(a.R00, dx, fmaf(a.R10, dy, a.R20 * dz));
    m.p1 = fmaf(a.R01, dx, fmaf(a.R11, dy, a.R21 * dz));
    m.p2 = fmaf(a.R02, dx, fmaf(a.R12, dy, a.R22 * dz));
}

// World centre of a sphere given in its link frame, and |c|^2.
__device__ __forceinline__ void sphere_world(const Frame &f, float4 sp, float &cx, float &cy, float &cz, float &as) {
    cx = fmaf(f.R00, sp.x, fmaf(f.R01, sp.y, fmaf(f.R02, sp.z, f.p0)));
    cy = fmaf(f.R10, sp.x, fmaf(f.R11, sp.y, fmaf(f.R12, sp.z, f.p1)));
    cz = fmaf(f.R20, sp.x, fmaf(f.R21, sp.y, fmaf(f.R22, sp.z, f.p2)));
    as = fmaf(cx, cx, fmaf(cy, cy, cz * cz));
}

// Translating robot: centre = (q0, q1, q2 or 0) + offset, and |c|^2.
__device__ __forceinline__ void sphere_translate(const SceneDev &sc, const float *q, float4 sp, float &cx, float &cy,
                                                 float &cz, float &as) {
    const float pz = sc.d >= 3 ? q[2] : 0.0f;
    cx = q[0] + sp.x;
    cy = q[1] + sp.y;
    cz = pz + sp.z;
    as = fmaf(cx, cx, fmaf(cy, cy, cz * cz));
}

// Segment index for time t with waypoint times shared by all obstacles:
// the number of interior waypoint times <= t.
__device__ __forceinline__ int shared_segment(const SceneDev &sc, const float4 *lds, float t) {
    const float *lt = reinterpret_cast<const float *>(lds + sc.lds_t);
    int k = 0;
#pragma unroll 4
    for (int j = 1; j < sc.n_seg; ++j) k += (t >= lt[j]) ? 1 : 0;
    return k;
}

// -2 * (obstacle centre at time t), from the pre-scaled segment table.
__device__ __forceinline__ void obstacle_n(const float4 *lds, int n_seg, int o, int k, float t, float &nx, float &ny,
                                           float &nz) {
    const float4 A = lds[(o * n_seg + k) * 2];
    const float4 B = lds[(o * n_seg + k) * 2 + 1];
    const float s = __builtin_amdgcn_fmed3f(t - A.w, 0.0f, B.w);
    nx = fmaf(s, B.x, A.x);
    ny = fmaf(s, B.y, A.y);
    nz = fmaf(s, B.z, A.z);
}

// The same with waypoint times of the obstacle's own.  Unrolled as above: the reads
// of a loop that is not were waited for one by one, 448 of them for 32 obstacles
// of 16 waypoints (1000 bridge-length edges of the 7-DOF arm 80 us, 66 so).
__device__ __forceinline__ int generic_segment(const SceneDev &sc, const float4 *lds, int o, float t) {
    const float *lt = reinterpret_cast<const float *>(lds + sc.lds_t) + o * (sc.n_seg + 1);
    int k = 0;
#pragma unroll 4
    for (int j = 1; j < sc.n_seg; ++j) k += (t >= lt[j]) ? 1 : 0;
    return k;
}

__device__ __forceinline__ int lane_id() { return __lane_id(); }

// The obstacles tile .. tile + OT - 1 at time t: n = -2 o and A = |o|^2 - r_o^2.
template <int OT, int OBS>
__device__ __forceinline__ void tile_obstacles(const SceneDev &sc, const float4 *lds, int tile, int kseg, float t,
                                               const float *ro, float *nx, float *ny, float *nz, float *A) {
    // four obstacles' rows in flight together
#pragma unroll
    for (int i0 = 0; i0 < OT; i0 += 4) {
        float4 P[4], V[4];
#pragma unroll
        for (int u = 0; u < 4; ++u) {
            const int o = tile + i0 + u;
            const int k = (OBS == kObsShared) ? kseg : generic_segment(sc, lds, o, t);
            P[u] = lds[(o * sc.n_seg + k) * 2];
            V[u] = lds[(o * sc.n_seg + k) * 2 + 1];
        }
#pragma unroll
        for (int u = 0; u < 4; ++u) {
            const int i = i0 + u;
            const float s = __builtin_amdgcn_fmed3f(t - P[u].w, 0.0f, V[u].w);
            nx[i] = fmaf(s, V[u].x, P[u].x);
            ny[i] = fmaf(s, V[u].y, P[u].y);
            nz[i] = fmaf(s, V[u].z, P[u].z);
            A[i] = fmaf(0.25f, fmaf(nx[i], nx[i], fmaf(ny[i], ny[i], nz[i] * nz[i])), -ro[i] * ro[i]);
        }
    }
}

// Sphere (centre c, a_s = |c|^2, radius r_s) against the OT obstacles of the
// tile.  With n = -2 o and A_o = |o|^2 - r_o^2 (per lane and obstacle, at the
// lane's time), a pair collides iff
//   A_o + c.n - 2 r r_o < r^2 - a_s,   r = r_s + eps,
// which is |c - o|^2 < (r + r_o)^2 expanded.  The loop keeps the minimum of
// the left side over the tile (three or four FMAs and half a min3 per pair,
// no scalar-unit work); the result is that minimum minus the right side,
// negative iff some pair collides.  With equal obstacle radii (UNI) the
// r_o term moves to the right side.
template <int OT, bool UNI>
__device__ __forceinline__ float sphere_clear(const SceneDev &sc, float cx, float cy, float cz, float as, float r_s,
                                              const float *nx, const float *ny, const float *nz, const float *A,
                                              const float *ro) {
    const float r = r_s + (float)kClearanceEps;
    const float k = -2.0f * r;
    float m = INFINITY;
#pragma unroll
    for (int i = 0; i < OT; ++i) {
        float v = fmaf(cx, nx[i], A[i]);
        v = fmaf(cy, ny[i], v);
        v = fmaf(cz, nz[i], v);
        if (!UNI) v = fmaf(k, ro[i], v);
        m = fminf(m, v);
    }
    float rhs = fmaf(r, r, -as);
    if (UNI) rhs = fmaf(-k, sc.r_uni, rhs);
    return m - rhs;
}

// Squared distance from point c to fixed box b: offsets along the box axes,
// their excess over the half extents (zero inside), and the squared norm.
__device__ __forceinline__ float box_dist2(const float4 *lds, const SceneDev &sc, int b, float cx, float cy,
                                           float cz) {
    const float4 *B = lds + sc.lds_box + 4 * b;
    const float4 a0 = B[0], a1 = B[1], a2 = B[2], hb = B[3];
    const float u0 = fmaf(a0.x, cx, fmaf(a0.y, cy, fmaf(a0.z, cz, a0.w)));
    const float u1 = fmaf(a1.x, cx, fmaf(a1.y, cy, fmaf(a1.z, cz, a1.w)));
    const float u2 = fmaf(a2.x, cx, fmaf(a2.y, cy, fmaf(a2.z, cz, a2.w)));
    const float e0 = fmaxf(fabsf(u0) - hb.x, 0.0f);
    const float e1 = fmaxf(fabsf(u1) - hb.y, 0.0f);
    const float e2 = fmaxf(fabsf(u2) - hb.z, 0.0f);
    return fmaf(e0, e0, fmaf(e1, e1, e2 * e2));
}

// Spheres [s0, s1) of link b, offsets p_b, against spheres [a0, a1) of link a,
// with m the frame of b in the frame of a: a pair collides iff
// |m p_b - p_a| < r_a + r_b + eps.  `first` is this lane's first sphere of b
// and `step` its stride (the lane split of a state).
__device__ __forceinline__ bool link_pair_hits(const float4 *lds, const SceneDev &sc, const Frame &m, int first,
                                               int s1, int step, int a0, int a1) {
    // (bitwise, not short-circuit, decisions: four reads in flight at a time
    // instead of a branch and a wait per sphere pair, which made a wave's static
    // terms take 50 us)
    bool h = false;
    for (int s = first; s < s1; s += step) {
        const float4 sp = lds[sc.lds_sph + s];
        const float cx = fmaf(m.R00, sp.x, fmaf(m.R01, sp.y, fmaf(m.R02, sp.z, m.p0)));
        const float cy = fmaf(m.R10, sp.x, fmaf(m.R11, sp.y, fmaf(m.R12, sp.z, m.p1)));
        const float cz = fmaf(m.R20, sp.x, fmaf(m.R21, sp.y, fmaf(m.R22, sp.z, m.p2)));
        const float rb = sp.w + (float)kClearanceEps;
#pragma unroll 4
        for (int a = a0; a < a1; ++a) {
            const float4 pa = lds[sc.lds_sph + a];
            const float dx = cx - pa.x, dy = cy - pa.y, dz = cz - pa.z;
            const float R = pa.w + rb;
            h = h | (fmaf(dx, dx, fmaf(dy, dy, dz * dz)) < R * R);
        }
    }
    return h;
}

// Broad phase of the static terms: a link's spheres lie inside its bounding
// sphere (centre and radius per link, in the link frame); when two bounding
// spheres, or a bounding sphere and a box, are more than kBroadMargin apart,
// every sphere pair between them clears contact by that much and the exact
// tests are skipped (they could only report free).
constexpr float kBroadMargin = 1e-3f;

// Lanes per state: the template argument, or (kSplitAny) 1 << shift at run time.
constexpr int kSplitAny = 0;
template <int SPLIT>
__device__ __forceinline__ int split_step(int shift) { return SPLIT == kSplitAny ? 1 << shift : SPLIT; }

template <int SPLIT>
__device__ __forceinline__ bool state_hit(uint64_t hm, int st_lane, int step);

// The next joint angle of a walk along the chain: q rotated by one.
__device__ __forceinline__ float next_angle(float (&q)[kMaxDof]) {
    const float v = q[0];
#pragma unroll
    for (int j = 0; j + 1 < kMaxDof; ++j) q[j] = q[j + 1];
    return v;
}

// Self-collision of the listed link pairs and the fixed boxes for the lane's
// configuration q (time-independent).  Outer turn la walks the chain to link
// la; its spheres near a box are tested against it in the world frame, and an
// inner walk on from link la meets every listed upper link lb, whose spheres
// are tested in la's frame when the links' bounds are near (one relative
// transform per link pair).  The walks repeat joint transforms (la to lb for
// every la with a listed pair) instead of keeping every link's frame in
// registers, which took a fully unrolled chain of 10000 instructions.
// Updates hit / hm / alive as the obstacle tiles do.  Every lane of the wave
// must call this.
template <int SPLIT>
__device__ __forceinline__ void static_pass(const SceneDev &sc, const float4 *lds, const float *q, bool &alive,
                                            bool &hit, uint64_t &hm, uint64_t lower_mask, int part, int st_lane,
                                            int step) {
    Frame Fa;
    frame_identity(Fa);
    float qa[kMaxDof];  // the joints above link la
#pragma unroll
    for (int j = 0; j < kMaxDof; ++j) qa[j] = q[j];
    auto decide = [&](bool h) {
        hm |= __ballot(h);
        hit = hit || state_hit<SPLIT>(hm, st_lane, step);
        const uint64_t mk = __ballot(hit);
        alive = alive && !hit && !(mk & lower_mask);
    };
    LinkRec ra = link_rec(sc, lds, 0);
#pragma nounroll
    for (int la = 0; la <= sc.d; ++la) {
        const LinkRec ka = ra;
        if (la < sc.d) ra = link_rec(sc, lds, la + 1);
        if (la > 0) {
            const float ang = next_angle(qa);
            if (alive) dh_compose(ka, ang, Fa);
        }
        if (__ballot(alive) == 0) break;
        const int a0 = uniform(ka.s0), a1 = uniform(ka.s1);
        if (a1 <= a0) continue;
        const float4 ba = ka.bs;
        if (sc.n_box > 0) {
            bool h = false;
            if (alive) {
                const int first = a0 + ((part - a0) & (step - 1));
                float bx, by, bz, bs;
                sphere_world(Fa, ba, bx, by, bz, bs);
                const float rb = ba.w + kBroadMargin;
                for (int b = 0; b < sc.n_box; ++b) {
                    if (box_dist2(lds, sc, b, bx, by, bz) < rb * rb) {
                        for (int s = first; s < a1; s += step) {
                            float cx, cy, cz, as;
                            const float4 sp = lds[sc.lds_sph + s];
                            sphere_world(Fa, sp, cx, cy, cz, as);
                            const float rr = sp.w + (float)kClearanceEps;
                            h = h | (box_dist2(lds, sc, b, cx, cy, cz) < rr * rr);
                        }
                    }
                }
            }
            decide(h);
        }
        if (!sc.n_pair) continue;
        Frame F = Fa;
        float qb[kMaxDof];
#pragma unroll
        for (int j = 0; j < kMaxDof; ++j) qb[j] = qa[j];
        LinkRec rb = ra;
        // up to the last listed upper link of la
        const int last = (int)((sc.last_pair >> (4 * la)) & 15u);
#pragma nounroll
        for (int lb = la + 1; lb <= last; ++lb) {
            const LinkRec kb = rb;
            if (lb < last) rb = link_rec(sc, lds, lb + 1);
            const float ang = next_angle(qb);
            if (alive) dh_compose(kb, ang, F);
            const int b0 = uniform(kb.s0), b1 = uniform(kb.s1);
            if (!(((unsigned)uniform((int)kb.mask) >> la) & 1u) || b1 <= b0) continue;
            bool h = false;
            if (alive) {
                Frame m;
                frame_relative(Fa, F, m);
                const float4 bl = kb.bs;
                const float dx = fmaf(m.R00, bl.x, fmaf(m.R01, bl.y, fmaf(m.R02, bl.z, m.p0))) - ba.x;
                const float dy = fmaf(m.R10, bl.x, fmaf(m.R11, bl.y, fmaf(m.R12, bl.z, m.p1))) - ba.y;
                const float dz = fmaf(m.R20, bl.x, fmaf(m.R21, bl.y, fmaf(m.R22, bl.z, m.p2))) - ba.z;
                const float R = ba.w + bl.w + kBroadMargin;
                if (fmaf(dx, dx, fmaf(dy, dy, dz * dz)) < R * R)
                    h = link_pair_hits(lds, sc, m, b0 + ((part - b0) & (step - 1)), b1, step, a0, a1);
            }
            decide(h);
        }
    }
}

// Hit of the lane's state from the lane's accumulated pair masks.  A lane
// knows its own bit exactly (its own ballots included it); with several lanes
// per state those ran different numbers of sphere iterations, so their
// own bits are exchanged by one more ballot of the whole wave.  Every lane of
// the wave must call this.
template <int SPLIT>
__device__ __forceinline__ bool state_hit(uint64_t hm, int st_lane, int step) {
    if (SPLIT == 1) return (hm >> lane_id()) & 1ull;
    const uint64_t own = __ballot(((hm >> lane_id()) & 1ull) != 0);
    return ((own >> st_lane) & ((1ull << step) - 1ull)) != 0;
}

// Does the lane's state (q, t) collide?  OT obstacles are held in registers
// per tile.  With SPLIT > 1 a state occupies SPLIT adjacent lanes (aligned;
// 1 << shift of them for SPLIT = kSplitAny, at most 16)
// and lane `part` of them tests the spheres s with s = part (mod SPLIT);
// every lane composes the kinematic chain itself, and a state's hit is the OR
// over its lanes, so all SPLIT lanes return the same answer.  This divides
// the dependent chain of one state check by about SPLIT for launches too
// small to fill the device.  `alive` enters true for lanes that must check;
// after every link the wave ballots the hits and a lane stops on a hit of its
// state, or when a lower state of its group has hit (so the least colliding
// index of a group is exact); lower_mask holds the lanes of the lower states.
// Every lane of the wave must call this (it contains ballots).
template <int KIND, int OT, int OBS, int SPLIT = 1>
__device__ __forceinline__ bool state_hits(const SceneDev &sc, const float4 *lds, const float *q, float t, bool alive,
                                           uint64_t lower_mask, int part = 0, int shift = 0) {
    static_assert(SPLIT == kSplitAny || SPLIT == 1 || SPLIT == 2 || SPLIT == 4, "state split");
    const int step = split_step<SPLIT>(shift);
    const int st_lane = lane_id() & ~(step - 1);  // first lane of this state
    bool hit = false;
    uint64_t hm = 0;  // wave mask of lanes with a colliding pair
    // configuration box and horizon
    {
        // (unused slots hold an infinite box; no short circuits, which would
        // wait for each bound in turn)
        const float4 *B = lds + sc.lds_const;
        const float4 l0 = B[0], l1 = B[1], u0 = B[2], u1 = B[3];
        const float lo[8] = {l0.x, l0.y, l0.z, l0.w, l1.x, l1.y, l1.z, l1.w};
        const float up[8] = {u0.x, u0.y, u0.z, u0.w, u1.x, u1.y, u1.z, u1.w};
        bool in = (t >= 0.0f) & (t <= sc.H);
#pragma unroll
        for (int j = 0; j < kMaxDof; ++j) in = in & (q[j] >= lo[j]) & (q[j] <= up[j]);
        hit = alive & !in;
    }
    {
        const uint64_t m = __ballot(hit);
        alive = alive && !hit && !(m & lower_mask);
    }
    int kseg = 0;
    if (OBS == kObsShared) kseg = shared_segment(sc, lds, t);
    for (int tile = 0; tile < sc.O_pad; tile += OT) {
        if (__ballot(alive) == 0) break;
        float nx[OT], ny[OT], nz[OT], A[OT], ro[OT];
#pragma unroll
        for (int i = 0; i < OT; ++i) ro[i] = sc.ro[tile + i];
        if (alive) tile_obstacles<OT, OBS>(sc, lds, tile, kseg, t, ro, nx, ny, nz, A);
        // one specialisation for equal obstacle radii, one for mixed radii
        auto run = [&](auto uni_c) {
            constexpr bool UNI = decltype(uni_c)::value;
            if (KIND == kTranslate) {
                float dmin = INFINITY;
                for (int s = part; s < sc.S; s += step) {
                    if (alive) {
                        float cx, cy, cz, as;
                        const float4 sp = lds[sc.lds_sph + s];
                        sphere_translate(sc, q, sp, cx, cy, cz, as);
                        dmin = fminf(dmin, sphere_clear<OT, UNI>(sc, cx, cy, cz, as, sp.w, nx, ny, nz, A, ro));
                    }
                }
                hm |= __ballot(alive && dmin < 0.0f);
                hit = hit || state_hit<SPLIT>(hm, st_lane, step);
                const uint64_t m = __ballot(hit);
                alive = alive && !hit && !(m & lower_mask);
            } else {
                // world <- link frame.  One link per turn of a loop that is not
                // unrolled: the unrolled chain was 5000 instructions (40 KB,
                // most of the instruction cache two CUs share), and the waves
                // of a launch with a round or two of states each waited for
                // its fetch, not for its arithmetic.
                Frame f;
                frame_identity(f);
                float qn[kMaxDof];  // the coming joints' angles, the next one first
#pragma unroll
                for (int j = 0; j < kMaxDof; ++j) qn[j] = q[j];
                LinkRec rec = link_rec(sc, lds, 0);
#pragma nounroll
                for (int l = 0; l <= sc.d; ++l) {
                    const LinkRec lk = rec;
                    if (l < sc.d) rec = link_rec(sc, lds, l + 1);  // in flight while this link is checked
                    if (l > 0) {
                        const float ang = next_angle(qn);
                        if (alive) dh_compose(lk, ang, f);
                    }
                    const int s0 = uniform(lk.s0), s1 = uniform(lk.s1);
                    if (s1 > s0 && __ballot(alive) != 0) {
                        // broad phase for links of three spheres or more: the
                        // link's bounding sphere (its spheres' radii included)
                        // clearing every obstacle of the tile by kBroadMargin
                        // clears each of its spheres (the margin is far above
                        // the FP32 error), so the pair tests decide the same;
                        // the wave skips the link when all its lanes clear it
                        bool need = alive;
                        if (alive && s1 - s0 >= 3) {
                            const float4 bl = lk.bs;
                            float bx, by, bz, bs;
                            sphere_world(f, make_float4(bl.x, bl.y, bl.z, 0.0f), bx, by, bz, bs);
                            need = sphere_clear<OT, UNI>(sc, bx, by, bz, bs, bl.w + kBroadMargin, nx, ny, nz, A, ro) <
                                   0.0f;
                        }
                        // this lane's spheres of the link: s = part (mod step)
                        float dmin = INFINITY;
                        if (__ballot(need) != 0 && need) {
                            // two spheres per step: both offset reads are in flight together
                            const int first = s0 + ((part - s0) & (step - 1));
                            int s = first;
#pragma nounroll
                            for (; s + step < s1; s += 2 * step) {
                                const float4 sp = lds[sc.lds_sph + s];
                                const float4 sq = lds[sc.lds_sph + s + step];
                                float cx, cy, cz, as, ex, ey, ez, bs;
                                sphere_world(f, sp, cx, cy, cz, as);
                                sphere_world(f, sq, ex, ey, ez, bs);
                                dmin = fminf(dmin, sphere_clear<OT, UNI>(sc, cx, cy, cz, as, sp.w, nx, ny, nz, A, ro));
                                dmin = fminf(dmin, sphere_clear<OT, UNI>(sc, ex, ey, ez, bs, sq.w, nx, ny, nz, A, ro));
                            }
                            if (s < s1) {
                                const float4 sp = lds[sc.lds_sph + s];
                                float cx, cy, cz, as;
                                sphere_world(f, sp, cx, cy, cz, as);
                                dmin = fminf(dmin, sphere_clear<OT, UNI>(sc, cx, cy, cz, as, sp.w, nx, ny, nz, A, ro));
                            }
                        }
                        hm |= __ballot(alive && dmin < 0.0f);
                        hit = hit || state_hit<SPLIT>(hm, st_lane, step);
                        const uint64_t m = __ballot(hit);
                        alive = alive && !hit && !(m & lower_mask);
                    }
                }
            }
        };
        if (sc.r_uni >= 0.0f) run(std::true_type{});
        else run(std::false_type{});
    }
    // time-independent terms for the lanes still undecided
    if (KIND == kDHStatic && __ballot(alive) != 0)
        static_pass<SPLIT>(sc, lds, q, alive, hit, hm, lower_mask, part, st_lane, step);
    return hit;
}

// Does (q_g, t) collide?  The same decision as state_hits at q = q_g, with
// the sphere centres at q_g read from LDS (they are computed once per
// problem by the same kinematics code), so only the obstacle positions at t
// and the pair tests remain; the static terms at q_g are decided once per
// problem by the state test itself (goal_blocked).  SPLIT lanes share a state as in state_hits;
// lanes are independent otherwise (`alive` false: nothing to check).
template <int OT, int OBS, int SPLIT>
__device__ __forceinline__ bool goal_hits(const SceneDev &sc, const float4 *lds, float t, bool alive, int part) {
    const int step = SPLIT, st_lane = lane_id() & ~(SPLIT - 1);
    bool hit = false;
    uint64_t hm = 0;
    if (alive) {
        bool out = !(t >= 0.0f) || !(t <= sc.H) || sc.goal_blocked;
#pragma unroll
        for (int j = 0; j < kMaxDof; ++j)
            if (j < sc.d) out = out || !(sc.q_g[j] >= sc.q_lo[j]) || !(sc.q_g[j] <= sc.q_hi[j]);
        hit = out;
    }
    alive = alive && !hit;
    int kseg = 0;
    if (OBS == kObsShared) kseg = shared_segment(sc, lds, t);
    for (int tile = 0; tile < sc.O_pad; tile += OT) {
        if (__ballot(alive) == 0) break;
        float nx[OT], ny[OT], nz[OT], A[OT], ro[OT];
#pragma unroll
        for (int i = 0; i < OT; ++i) ro[i] = sc.ro[tile + i];
        if (alive) tile_obstacles<OT, OBS>(sc, lds, tile, kseg, t, ro, nx, ny, nz, A);
        // (the lanes are independent: the wave stops only when all have hit)
        for (int c0 = 0; c0 < sc.S; c0 += 8 * SPLIT) {
            if (__ballot(alive) == 0) break;
            float dmin = INFINITY;
            if (alive) {
                const int c1 = min(c0 + 8 * SPLIT, sc.S);
                for (int s = c0 + part; s < c1; s += SPLIT) {
                    const float4 c = lds[sc.lds_goal + s];
                    const float r_s = lds[sc.lds_sph + s].w;
                    dmin = fminf(dmin, sphere_clear<OT, false>(sc, c.x, c.y, c.z, c.w, r_s, nx, ny, nz, A, ro));
                }
            }
            hm |= __ballot(alive && dmin < 0.0f);
            hit = hit || state_hit<SPLIT>(hm, st_lane, step);
            alive = alive && !hit;
        }
    }
    return hit;
}

}  // namespace st
