// rrtc.hip -- the RRT-Connect local planner LP(x, y; s, ell) of the
// generalized GTMP graph (Sec. III; construction in the proof of the
// local-planner reach proposition of the appendix), run on every edge whose
// straight line failed while both endpoints are collision-free.
//
// One wave per call, persistent over the candidate list.  A call is a chain
// of dependent wave steps (sample, nearest node, extension check): a wave alone
// on its SIMD issues a vector instruction in a quarter of its cycles, sixteen
// waves a CU in 0.86 of them, so what counts is how few instructions a step
// takes and how many waves a CU holds.
//   vectors  a configuration is spread over the lanes (lane holds component
//            lane mod 8), so steering and the ellipsoid's map cost one
//            instruction where a copy per lane costs eight;
//   trees    both trees share one pool of nodes in the wave's LDS
//            (coordinates as [coordinate][node], so that lanes reading
//            consecutive nodes touch consecutive banks), a node's tree in the
//            top bit of its parent word: the pool is sized for sixteen waves
//            per CU rather than for 2 tree_cap nodes, and a call that fills
//            it is given up and run again, from the start, by a second launch
//            whose pools hold 2 tree_cap nodes (calls are independent and
//            keyed, so the result is the same);
//   sample   64 ellipsoid attempts at a time; those inside the ball are
//            mapped one by one in attempt order, a row per lane;
//   nearest  lanes stride over the pool, wave minimum with the lowest index
//            on ties; while a tree connects to one target only the node just
//            added is compared with the nearest known;
//   check    (arms, up to 96 obstacles) eight states at a time: the sines and
//            cosines of (state, joint) pairs, the frame chains of (state,
//            axis) pairs and then (state, sphere) pairs over the lanes, each
//            sphere tested exactly against the obstacles its bins list;
//            otherwise the states share the lanes, which split the obstacles.
// Arm of 40 spheres, 30 obstacles, M 6, N 100, trees of 512: k_rrtc 1.81 ms at
// budget 100 where whole states per lane, every sphere against every obstacle
// and four waves per CU took 19.7 ms (scene seed 5); a plan with the repair 2.45
// against 25 ms at budget 100, 9.7 against 63 at 400, 38 against 120 at 1000,
// where most calls run again (scene seed 0).
// This file is compiled without floating-point contraction: sampling, nearest
// node and steering are FP32 computations with a fixed operation order (see
// include/gtmp.h), so the trees are reproducible bit for bit.
#define GTMP_FK_PLAIN 1
#include "edge_common.hpp"
#include "state_test.hpp"

namespace gtmp {

constexpr int kRrtcAttempts = 4096;
constexpr int kRrtcLdsObstacles = 2048;  // obstacle floats held in LDS (more: read from global memory)
enum { kTrapped = 0, kAdvanced = 1, kReached = 2 };

struct RrtcArgs {
    int d, M, N, G;
    const float *q0, *goals, *Q;
    float lo[GTMP_MAX_DOF], hi[GTMP_MAX_DOF];
    // candidates: cand[0 .. *n_cand) pulled through *cursor; cand == NULL runs
    // the single edge `single` on block 0
    const uint32_t *cand;
    const uint32_t *n_cand;
    uint32_t *cursor;
    uint32_t single;
    float *C_s, *C_h, *C_l;
    uint8_t *flags;
    int budget, cap;
    float eta, res, ell_factor;
    uint32_t k0, k1, stage;
    const uint32_t *stage_dev;  // when set, the stage is read here at kernel start (replayed graphs)
    unsigned long long *stats;  // calls, successes, iterations, nodes, states checked (whole rounds), distances
    // single-edge outputs (path mode)
    float *path;
    int32_t *path_count;
    float *path_cost;
};

__device__ __forceinline__ void edge_endpoints(const RrtcArgs &A, uint32_t e, const float *&u, const float *&v) {
    const uint32_t N = (uint32_t)A.N;
    const uint64_t inner = (uint64_t)(A.M - 1) * N * N;
    if (e < N) {
        u = A.q0;
        v = A.Q + (size_t)e * A.d;
    } else if ((uint64_t)e - N < inner) {
        const uint64_t r = (uint64_t)e - N;
        const uint64_t m = r / ((uint64_t)N * N), uv = r - m * N * N;
        u = A.Q + ((size_t)m * N + uv / N) * A.d;
        v = A.Q + ((size_t)(m + 1) * N + uv % N) * A.d;
    } else {
        const uint64_t r = (uint64_t)e - N - inner;
        const uint64_t n = r / (uint64_t)A.G, g = r - n * A.G;
        u = A.Q + ((size_t)(A.M - 1) * N + n) * A.d;
        v = A.goals + (size_t)g * A.d;
    }
}

__device__ __forceinline__ float *cost_slot_of(const RrtcArgs &A, uint32_t e) {
    const uint64_t N = (uint64_t)A.N, inner_end = N + (uint64_t)(A.M - 1) * N * N;
    if (e < N) return A.C_s + e;
    if (e < inner_end) return A.C_h + (e - N);
    return A.C_l + (e - inner_end);
}

// Vertex ids of flat edge e in the order [q0 | Q[0] | ... | Q[M-1] | goals].
__device__ __forceinline__ void edge_vertex_ids(const RrtcArgs &A, uint64_t e, uint32_t &u, uint32_t &v) {
    const uint64_t N = (uint64_t)A.N, inner = (uint64_t)(A.M - 1) * N * N;
    if (e < N) {
        u = 0;
        v = 1 + (uint32_t)e;
    } else if (e - N < inner) {
        const uint64_t r = e - N, m = r / (N * N), uv = r - m * N * N;
        u = 1 + (uint32_t)(m * N + uv / N);
        v = 1 + (uint32_t)((m + 1) * N + uv % N);
    } else {
        const uint64_t r = e - N - inner, n = r / (uint64_t)A.G, g = r - n * A.G;
        u = 1 + (uint32_t)((A.M - 1) * N + n);
        v = 1 + (uint32_t)(A.M * N + g);
    }
}

__device__ __forceinline__ const float *vertex_ptr(const RrtcArgs &A, uint32_t id) {
    const uint32_t MN = (uint32_t)A.M * (uint32_t)A.N;
    if (id == 0) return A.q0;
    if (id <= MN) return A.Q + (size_t)(id - 1) * A.d;
    return A.goals + (size_t)(id - 1 - MN) * A.d;
}

constexpr int kRrtcStates = 8;   // states per round of the bin-filtered check
constexpr uint32_t kTreeBit = 0x8000u, kNoParent = 0x7fffu;

// Where a block's LDS goes (bytes from its start; areas 16-byte aligned).
struct RrtcLayout {
    int pool;      // nodes a wave holds for both trees together
    int waves;     // waves (calls) per block
    uint32_t off_tab, off_wave, wave_bytes;  // sphere table (or obstacles); first wave's area, stride
    uint32_t off_par, off_chain, off_og, off_sc;  // inside a wave's area, after the coordinates
    uint32_t total;
};

__host__ __device__ inline uint32_t up16_r(uint32_t x) { return (x + 15u) & ~15u; }

// shared_bytes: the block's own area (bins and sphere table, or obstacles).
inline RrtcLayout rrtc_layout(int d, int pool, int waves, uint32_t bins, uint32_t tab, bool grid) {
    RrtcLayout L{};
    L.pool = pool;
    L.waves = waves;
    L.off_tab = up16_r(bins);
    L.off_wave = up16_r(L.off_tab + tab);
    uint32_t o = up16_r((uint32_t)sizeof(float) * d * pool);
    L.off_par = o; o = up16_r(o + 2u * pool);
    L.off_chain = o; o = up16_r(o + 2u * pool);
    L.off_og = o; o += grid ? (uint32_t)sizeof(float4) * kRrtcStates * (GTMP_MAX_JOINTS + 1) : 0u;
    L.off_sc = o; o += grid ? (uint32_t)sizeof(float2) * kRrtcStates * GTMP_MAX_JOINTS : 0u;
    L.wave_bytes = up16_r(o);
    L.total = L.off_wave + L.wave_bytes * waves;
    return L;
}

// Per robot sphere: fraction along its link, radius, link.
struct SphereTab {
    float t[GTMP_MAX_ROBOT_SPHERES], r[GTMP_MAX_ROBOT_SPHERES];
    int link[GTMP_MAX_ROBOT_SPHERES];
};

__device__ __forceinline__ float lane_f(float x, int lane) {
    return __int_as_float(__builtin_amdgcn_readlane(__float_as_int(x), lane));
}

// Sum over components 0..7 in that order, starting from 0 (components past d
// are zero and leave the sum as it is).
__device__ __forceinline__ float ordered_sum(float v) {
    float acc = 0.0f;
#pragma unroll
    for (int i = 0; i < GTMP_MAX_DOF; ++i) acc = acc + lane_f(v, i);
    return acc;
}

// Minimum over the wave of the bits of non-negative floats, by row shifts and
// row broadcasts (the last lane ends with all 64 lanes' minimum).
__device__ __forceinline__ uint32_t wave_min_u32(uint32_t x) {
#define GTMP_DPP_MIN(ctrl, rows)                                                                        \
    {                                                                                                   \
        const uint32_t y = (uint32_t)__builtin_amdgcn_update_dpp((int)x, (int)x, ctrl, rows, 0xf, false); \
        x = x < y ? x : y;                                                                              \
    }
    GTMP_DPP_MIN(0x111, 0xf)  // row_shr:1
    GTMP_DPP_MIN(0x112, 0xf)  // row_shr:2
    GTMP_DPP_MIN(0x114, 0xf)  // row_shr:4
    GTMP_DPP_MIN(0x118, 0xf)  // row_shr:8
    GTMP_DPP_MIN(0x142, 0xa)  // row_bcast:15 into rows 1 and 3
    GTMP_DPP_MIN(0x143, 0xc)  // row_bcast:31 into rows 2 and 3
#undef GTMP_DPP_MIN
    return (uint32_t)__builtin_amdgcn_readlane((int)x, kWave - 1);
}

// LDS written by some lanes of a wave, read by others: the LDS pipe serves a
// wave's instructions in order, so only the compiler has to keep them so.
__device__ __forceinline__ void wave_lds_fence() {
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

// Up to eight arm states at once, x being joint lane mod 8 of state lane / 8
// (states ns.. are not looked at): 1 bit per state in contact (ANY: some bit,
// found in the first pass that meets one).  og and sc are the wave's scratch.
// The kinematics are those of arm_fk_visit, one axis per lane: every axis of
// a frame's vectors goes through the same operations with the joint's sine
// and cosine.
template <int WORDS, bool ANY, class AP>
__device__ __forceinline__ uint32_t arm_hit8(const AP &R, const SphereTab &T, const ObsGrid &G, float x, int ns,
                                             float4 *og, float2 *sc) {
    const int lane = lane_id();
    {
        const int j = lane & 7;
        if (j < R.n_joints && (lane >> 3) < ns) {
            float st, ct;
            joint_sincos(x, st, ct);
            sc[lane] = make_float2(st, ct);
        }
    }
    wave_lds_fence();
    {
        const int sl = lane >> 2, c = lane & 3;  // lanes of c = 3 write the unused fourth entry
        if (sl < ns) {
            float *o = reinterpret_cast<float *>(og + sl * (GTMP_MAX_JOINTS + 1)) + c;
            o[0] = 0.f;
            float xa, ya, za, pa;
            {
                const float2 s0 = sc[sl * 8];
                const float st = s0.x, ct = s0.y, ca = R.ca[0], sa = R.sa[0];
                xa = c == 0 ? ct : c == 1 ? st : 0.f;
                pa = c == 0 ? R.a[0] * ct : c == 1 ? R.a[0] * st : R.dz[0];
                ya = c == 0 ? -(ca * st) : c == 1 ? ca * ct : sa;
                za = c == 0 ? sa * st : c == 1 ? -(sa * ct) : ca;
                o[4] = pa;
            }
#pragma unroll
            for (int j = 1; j < GTMP_MAX_JOINTS; ++j) {
                if (j >= R.n_joints) break;
                const float2 sj = sc[sl * 8 + j];
                const float st = sj.x, ct = sj.y;
                const float xn = ct * xa + st * ya;
                pa += R.a[j] * xn + R.dz[j] * za;
                const float yp = ct * ya - st * xa;
                const int tw = R.twist[j];
                if (tw == kTwistNone) {
                    ya = yp;
                } else if (tw == kTwistPlus) {
                    ya = za;
                    za = -yp;
                } else if (tw == kTwistMinus) {
                    ya = -za;
                    za = yp;
                } else {
                    const float ca = R.ca[j], sa = R.sa[j];
                    const float yn = ca * yp + sa * za, zn = ca * za - sa * yp;
                    ya = yn;
                    za = zn;
                }
                xa = xn;
                o[4 * (j + 1)] = pa;
            }
        }
    }
    wave_lds_fence();
    const int nsph = R.n_spheres, items = ns * nsph;
    // item / nsph for items below 8 * 64 + 64: exact, since item times the
    // excess of magic * nsph over 65536 (below nsph <= 64) stays below 65536
    const uint32_t magic = (65536u + (uint32_t)nsph - 1u) / (uint32_t)nsph;
    uint32_t found = 0;
    for (int base = 0; base < items; base += kWave) {
        const int it = base + lane;
        const bool live = it < items;
        const uint32_t st = live ? ((uint32_t)it * magic) >> 16 : 0u;
        const uint32_t k = live ? (uint32_t)it - st * (uint32_t)nsph : 0u;
        const int L = T.link[k];
        const float t = T.t[k];
        const float4 lo4 = og[st * (GTMP_MAX_JOINTS + 1) + L - 1], hi4 = og[st * (GTMP_MAX_JOINTS + 1) + L];
        const float lo[3] = {lo4.x, lo4.y, lo4.z}, hi[3] = {hi4.x, hi4.y, hi4.z};
        float c[3];
        uint32_t m[WORDS];
#pragma unroll
        for (int wd = 0; wd < WORDS; ++wd) m[wd] = live ? ~0u : 0u;
#pragma unroll
        for (int i = 0; i < 3; ++i) {
            c[i] = __builtin_fmaf(t, hi[i] - lo[i], lo[i]);
            const uint32_t bin = grid_bin(__builtin_fmaf(c[i], G.inv[i], G.off[i]));
#pragma unroll
            for (int wd = 0; wd < WORDS; ++wd) m[wd] &= G.mask[wd][i][bin];
        }
        bool hit = false;
#pragma unroll
        for (int wd = 0; wd < WORDS; ++wd) {
            uint32_t mm = m[wd];
            if (ballot(mm != 0) == 0) continue;
            const float pr = R.uniform_r ? R.r0 : T.r[k];
            while (mm != 0) {
                const int o = 32 * wd + __builtin_ctz(mm);
                mm &= mm - 1;
                const float4 a = G.rec[o][0], h = G.rec[o][1];
                const float Rk = a.w + pr;
                float g = -Rk * Rk;
                const float ol[3] = {a.x, a.y, a.z}, oh[3] = {h.x, h.y, h.z};
#pragma unroll
                for (int i = 0; i < 3; ++i) {
                    const float dlt = c[i] - __builtin_amdgcn_fmed3f(c[i], ol[i], oh[i]);
                    g = __builtin_fmaf(dlt, dlt, g);
                }
                if (g <= 0.f) {  // a gap that is not a number is no contact, as in the general test's minimum
                    hit = true;
                    mm = 0;
                }
            }
        }
        uint64_t hm = ballot(hit);
        if (hm != 0) {
            if constexpr (ANY) return 1u;
            while (hm != 0) {
                const int src = __builtin_ctzll(hm);
                hm &= hm - 1;
                found |= 1u << __builtin_amdgcn_readlane((int)st, src);
            }
        }
    }
    return found;
}

// One call.  WORDS > 0: an arm whose states go through the obstacle bins;
// 0: the lanes of a state split its obstacles.
template <bool ARM, int W, int KP, int WORDS>
struct RrtcCall {
    static constexpr int D = StateDim<ARM, W>::D;
    const RrtcArgs &A;
    const ArmParams &R;
    const ArmParams *Rg;  // WORDS > 0: the table in device memory
    const SceneParams &S;
    const SphereTab &T;
    const ObsGrid &G;
    float *pos;           // [d][pool]
    uint16_t *par;        // [pool] parent in the pool (kNoParent: root), kTreeBit: the y tree
    uint16_t *chain;      // [pool] path walk
    float4 *og;
    float2 *sc;
    int pool;
    int lane, comp;
    float off;            // WORDS > 0: joint comp's angle offset
    uint32_t stage;
    int n0, n1;           // node counts of the x and y trees
    unsigned long long it_count, states, dists;  // of the current call
    bool full;            // the pool ran out

    __device__ __forceinline__ int count(int t) const { return t ? n1 : n0; }
    __device__ __forceinline__ float &P(int i, int j) const { return pos[i * pool + j]; }

    // Nearest node of tree t to q: squared distance and index.
    __device__ __forceinline__ void nearest(int t, float vq, float &best, int &near) const {
        const int d = A.d, n = n0 + n1;
        float q[GTMP_MAX_DOF];
#pragma unroll
        for (int i = 0; i < GTMP_MAX_DOF; ++i) q[i] = lane_f(vq, i);
        float b = __builtin_inff();
        int bi = 0x7fffffff;
        for (int j = lane; j < n; j += kWave) {
            float acc = 0.0f;
#pragma unroll
            for (int i = 0; i < GTMP_MAX_DOF; ++i)
                if (i < d) {
                    const float tt = P(i, j) - q[i];
                    acc = acc + tt * tt;
                }
            const bool mine = (par[j] & kTreeBit) == (t ? kTreeBit : 0u);
            if (mine && acc < b) {  // j increases: the lowest index among equal values stays
                b = acc;
                bi = j;
            }
        }
        const uint32_t mn = wave_min_u32(__float_as_uint(b));
        uint64_t m = ballot(__float_as_uint(b) == mn);
        int w = 0x7fffffff;
        while (m != 0) {  // one lane, but for exact ties
            const int o = __builtin_amdgcn_readlane(bi, __builtin_ctzll(m));
            w = o < w ? o : w;
            m &= m - 1;
        }
        best = __uint_as_float(mn);
        near = w < n ? w : t;  // no finite distance: the root
    }

    // Whether the segment p -> qn (a tree node and the new one) is free at
    // its states 1 .. Hs - 1, counted in rounds of up to 64 (with the bins eight
    // states are evaluated at a time, fewer than are counted where one is in
    // contact).
    __device__ __forceinline__ bool segment_free(float vp, float vqn, int Hs) {
        const float den = (float)(Hs - 1);
        if constexpr (WORDS > 0) {
            // the robot table read through a pointer the compiler cannot see
            // through: short-lived scalar loads rather than registers held
            // (and spilled) across the call
            carm Rp = (carm)Rg;
            asm volatile("" : "+s"(Rp));
            for (int h0 = 1; h0 < Hs; h0 += kRrtcStates) {
                const int h = h0 + (lane >> 3);
                const float tt = (float)(h < Hs ? h : 1) / den;
                const float s = h == Hs - 1 ? vqn : __builtin_fmaf(tt, vqn - vp, vp);
                const int ns = Hs - h0 < kRrtcStates ? Hs - h0 : kRrtcStates;
                if (arm_hit8<WORDS, true>(*Rp, T, G, s + off, ns, og, sc) != 0) {
                    const int end = (((h0 - 1) >> 6) + 1) << 6;
                    states += (unsigned long long)(end < Hs - 1 ? end : Hs - 1);
                    return false;
                }
            }
            states += (unsigned long long)(Hs - 1);
            return true;
        } else {
            // spr states per round (a power of two), lps = 64 / spr lanes
            // sharing each state's obstacles
            float p[D], qn[D];
#pragma unroll
            for (int i = 0; i < D; ++i) {
                p[i] = lane_f(vp, i);
                qn[i] = lane_f(vqn, i);
            }
            int lg = 0;
            while ((1 << lg) < Hs - 1 && lg < 6) ++lg;
            const int spr = 1 << lg, lgl = 6 - lg, lps = 1 << lgl;
            const int sl = lane >> lgl, part = lane & (lps - 1);
            for (int h0 = 1; h0 < Hs; h0 += spr) {
                const int h = h0 + sl;
                const bool act = h < Hs;
                const float tt = (float)(act ? h : 1) / den;
                float s[D];
#pragma unroll
                for (int i = 0; i < D; ++i) s[i] = h == Hs - 1 ? qn[i] : __builtin_fmaf(tt, qn[i] - p[i], p[i]);
                float gap = state_gap_part<ARM, W, KP>(R, S, s, part, lps);
                for (int off = lps >> 1; off > 0; off >>= 1) gap = __builtin_fminf(gap, __shfl_xor(gap, off));
                states += (unsigned long long)(Hs - h0 < spr ? Hs - h0 : spr);
                if (ballot(act && !(gap > 0.f)) != 0) return false;
            }
            return true;
        }
    }

    // Extend tree t towards q from its nearest node (best, near); returns the
    // status, the new node in idx and its coordinates in vqn.
    __device__ __forceinline__ int extend(int t, float vq, float best, int near, int &idx, float &vqn) {
        const int nt = count(t);
        dists += (unsigned long long)nt;
        const bool in = comp < A.d;
        const float vp = in ? P(comp, near) : 0.f;
        const float dist = __builtin_sqrtf(best);
        const bool reached = dist <= A.eta;
        const float f = A.eta / dist;
        vqn = in ? (reached ? vq : vp + f * (vq - vp)) : 0.f;
        const float dl = vp - vqn;
        const float len = __builtin_sqrtf(ordered_sum(dl * dl));
        int Hs = (int)__builtin_ceilf(len / A.res) + 1;
        Hs = Hs < 2 ? 2 : Hs;
        Hs = (int)uniform((uint32_t)Hs);
        if (!segment_free(vp, vqn, Hs)) return kTrapped;
        const int k = n0 + n1;
        if (k >= pool) {
            full = true;
            return kTrapped;
        }
        if (lane < A.d) P(lane, k) = vqn;
        if (lane == 0) par[k] = (uint16_t)((uint32_t)near | (t ? kTreeBit : 0u));
        wave_lds_fence();
        if (t) ++n1; else ++n0;
        idx = k;
        return uniform(reached ? 1u : 0u) ? kReached : kAdvanced;
    }

    // The sample of iteration it: true and vq set when an attempt passes.
    // H: row comp of the ellipsoid's map.
    __device__ __forceinline__ bool sample(uint32_t e, uint32_t it, float centre, float r1, float r2,
                                           const float (&H)[GTMP_MAX_DOF], float lo, float hi, float &vq) const {
        const int d = A.d;
        for (int base = 0; base < kRrtcAttempts; base += kWave) {
            const uint32_t a = (uint32_t)(base + lane);
            const uint4 w0 = philox4x32_10(make_uint4(e, it, stage, (3u << 16) | (2u * a)), A.k0, A.k1);
            uint4 w1 = make_uint4(0u, 0u, 0u, 0u);
            if (d > 4) w1 = philox4x32_10(make_uint4(e, it, stage, (3u << 16) | (2u * a + 1u)), A.k0, A.k1);
            float y[GTMP_MAX_DOF];
            float s2 = 0.0f;
#pragma unroll
            for (int i = 0; i < GTMP_MAX_DOF; ++i) {
                const uint32_t wi = i == 0 ? w0.x : i == 1 ? w0.y : i == 2 ? w0.z : i == 3 ? w0.w
                                  : i == 4 ? w1.x : i == 5 ? w1.y : i == 6 ? w1.z : w1.w;
                y[i] = (float)(wi >> 8) * (1.0f / 8388608.0f) - 1.0f;
                if (i < d) s2 = s2 + y[i] * y[i];
            }
            uint64_t m = ballot(s2 < 1.0f);
            while (m != 0) {  // in attempt order
                const int src = __builtin_ctzll(m);
                m &= m - 1;
                float acc = 0.0f;
#pragma unroll
                for (int c = 0; c < GTMP_MAX_DOF; ++c)
                    if (c < d) acc = acc + H[c] * ((c == 0 ? r1 : r2) * lane_f(y[c], src));
                const float x = centre + acc;
                if (ballot(comp < d && !(x >= lo && x <= hi)) == 0) {
                    vq = comp < d ? x : 0.f;
                    return true;
                }
            }
        }
        return false;
    }

    // Run one call on edge e.  Returns success (not meaningful when `full`);
    // the path length in *cost.
    __device__ __forceinline__ bool run(uint32_t e, float *cost) {
        const int d = A.d;
        const float *pu, *pv;
        edge_endpoints(A, e, pu, pv);
        const bool in = comp < d;
        const float vx = in ? pu[comp] : 0.f, vy = in ? pv[comp] : 0.f;
        float lo = 0.f, hi = 0.f;
        if (in) {
            lo = A.lo[comp];
            hi = A.hi[comp];
        }
        // query ellipsoid: foci x, y, major axis ell (hyperspheroid map as in
        // the informed set of Sec. IV-E)
        const float dxy = vx - vy;
        const float cmin = __builtin_sqrtf(ordered_sum(dxy * dxy));
        const float ell = A.ell_factor * cmin;
        const float centre = (vx + vy) * 0.5f;
        const float r1 = ell * 0.5f;
        const float sq = ell * ell - cmin * cmin;
        const float r2 = __builtin_sqrtf(sq > 0.0f ? sq : 0.0f) * 0.5f;
        float H[GTMP_MAX_DOF];
        {
            const float a = (vy - vx) / cmin;
            const float w = in ? (comp == 0 ? 1.0f : 0.0f) - a : 0.f;
            const float ww = ordered_sum(w * w);
            const float s = 2.0f / ww;
#pragma unroll
            for (int c = 0; c < GTMP_MAX_DOF; ++c) {
                const float delta = comp == c ? 1.0f : 0.0f;
                H[c] = ww != 0.0f ? delta - (s * w) * lane_f(w, c) : delta;
            }
        }
        if (lane < d) {
            P(lane, 0) = vx;
            P(lane, 1) = vy;
        }
        if (lane == 0) {
            par[0] = (uint16_t)kNoParent;
            par[1] = (uint16_t)(kNoParent | kTreeBit);
        }
        wave_lds_fence();
        n0 = n1 = 1;
        full = false;
        it_count = states = dists = 0;
        int ta = 0;  // tree A: 0 = the x tree
        bool ok = false;
        int ax = -1, ay = -1;
        uint32_t it = 0;
        for (; it < (uint32_t)A.budget && !ok && !full; ++it) {
            float vq;
            if (count(ta) < A.cap && sample(e, it, centre, r1, r2, H, lo, hi, vq)) {
                int ia = -1, near;
                float best, vn;
                nearest(ta, vq, best, near);
                if (extend(ta, vq, best, near, ia, vn) != kTrapped) {
                    // tree B connects: the target stays, so after each new node
                    // the nearest is that node or the one known before it
                    const int tb = 1 - ta;
                    int ib = -1, st = kTrapped;
                    nearest(tb, vn, best, near);
                    while (count(tb) < A.cap) {
                        float vb;
                        st = extend(tb, vn, best, near, ib, vb);
                        if (st != kAdvanced) break;
                        st = kTrapped;
                        const float df = vb - vn;
                        const float d2 = ordered_sum(df * df);
                        if (d2 < best) {
                            best = d2;
                            near = ib;
                        }
                    }
                    if (st == kReached) {
                        ok = true;
                        ax = ta == 0 ? ia : ib;
                        ay = ta == 0 ? ib : ia;
                    }
                }
            }
            ta = 1 - ta;
        }
        it_count = it;
        *cost = __builtin_inff();
        if (!ok || full) return false;
        // path x -> ... -> junction -> ... -> y: the x tree's chain from the
        // junction to its root (stored junction first), then the y tree's
        // chain from the junction's parent to its root; the length is summed
        // along the path from x to y
        if (lane == 0) {
            auto up = [&](int j) { return (int)(par[j] & kNoParent); };
            int nc = 0;
            for (int j = ax; j != (int)kNoParent; j = up(j)) chain[nc++] = (uint16_t)j;  // x tree, junction first
            const int nx = nc;
            for (int j = up(ay); j != (int)kNoParent; j = up(j)) chain[nc++] = (uint16_t)j;  // y tree
            // k-th waypoint of the path: x chain reversed, then the y chain
            auto node = [&](int k) { return (int)(k < nx ? chain[nx - 1 - k] : chain[k]); };
            float Lsum = 0.0f;
            for (int k = 0; k + 1 < nc; ++k) {
                const int a = node(k), b = node(k + 1);
                float s2 = 0.0f;
                for (int i = 0; i < d; ++i) {
                    const float tt = P(i, b) - P(i, a);
                    s2 = s2 + tt * tt;
                }
                Lsum = Lsum + __builtin_sqrtf(s2);
            }
            *cost = Lsum;
            if (A.path) {
                for (int k = 0; k < nc; ++k)
                    for (int i = 0; i < d; ++i) A.path[(size_t)k * d + i] = P(i, node(k));
                *A.path_count = nc;
            }
        }
        *cost = __shfl(*cost, 0);
        return true;
    }
};

// flags[e] of a call whose pool ran out, until the second launch takes it.
constexpr uint8_t kRrtcAgain = 3;

// WPB waves per block, OCC: waves per SIMD the register allocation is made for.
template <bool ARM, int W, int KP, int WORDS, int WPB, int OCC>
__global__ void __launch_bounds__(WPB *kWave, OCC) k_rrtc(RrtcArgs A, ArmParams R, SceneParams Sg, RrtcLayout Y,
                                                          const ObsGrid *grid, const ArmParams *Rg) {
    extern __shared__ __align__(16) unsigned char rrtc_lds[];
    SceneParams S = Sg;
    SphereTab *T = reinterpret_cast<SphereTab *>(rrtc_lds + Y.off_tab);
    const ObsGrid *G = reinterpret_cast<const ObsGrid *>(rrtc_lds);
    if constexpr (WORDS > 0) {
        copy_to_lds<grid_lds_bytes<WORDS>(), WPB * kWave>(rrtc_lds, grid, threadIdx.x);
        for (int k = threadIdx.x; k < Rg->n_spheres; k += WPB * kWave) {
            T->t[k] = Rg->t[k];
            T->r[k] = Rg->r[k];
            T->link[k] = Rg->link[k];
        }
    } else {
        // obstacles copied into LDS when they fit (the extension checks read
        // them with per-lane indices)
        constexpr int PW = ARM ? 3 : W;
        const int ns = Sg.n_sph * (PW + 1), nb = Sg.n_box * 2 * PW;
        if (ns + nb <= kRrtcLdsObstacles) {
            float *obs = reinterpret_cast<float *>(T);
            for (int i = threadIdx.x; i < ns; i += WPB * kWave) obs[i] = Sg.sph[i];
            for (int i = threadIdx.x; i < nb; i += WPB * kWave) obs[ns + i] = Sg.box[i];
            S.sph = obs;
            S.box = obs + ns;
        }
    }
    __syncthreads();  // the block's last: every wave runs its own calls from here
    unsigned char *wl = rrtc_lds + Y.off_wave + wave_in_block() * Y.wave_bytes;
    const uint32_t stage = A.stage_dev ? *A.stage_dev : A.stage;
    const int lane = lane_id();
    RrtcCall<ARM, W, KP, WORDS> c{A, R, Rg, S, *T, *G, reinterpret_cast<float *>(wl),
                                  reinterpret_cast<uint16_t *>(wl + Y.off_par),
                                  reinterpret_cast<uint16_t *>(wl + Y.off_chain),
                                  reinterpret_cast<float4 *>(wl + Y.off_og),
                                  reinterpret_cast<float2 *>(wl + Y.off_sc), Y.pool, lane, lane & 7,
                                  WORDS > 0 ? Rg->off[lane & 7] : 0.f, stage,
                                  1, 1, 0ull, 0ull, 0ull, false};
    unsigned long long calls = 0, wins = 0, nodes = 0, its = 0, states = 0, dists = 0;
    if (A.cand == nullptr) {  // one edge, path mode (the pool holds both trees)
        if (blockIdx.x != 0 || threadIdx.x >= kWave) return;
        float cost;
        const bool ok = c.run(A.single, &cost);
        if (lane == 0) {
            *A.path_cost = cost;
            if (!ok) *A.path_count = 0;
        }
        return;
    }
    const uint32_t total = uniform(*A.n_cand);
    while (true) {
        uint32_t slot = 0;
        if (lane == 0) slot = atomicAdd(A.cursor, 1u);
        slot = uniform(slot);
        if (slot >= total) break;
        const uint32_t e = uniform(A.cand[slot]);
        float cost;
        const bool ok = c.run(e, &cost);
        if (c.full) {
            if (lane == 0) A.flags[e] = kRrtcAgain;
            continue;
        }
        ++calls;
        nodes += (unsigned long long)(c.n0 + c.n1);
        its += c.it_count;
        states += c.states;
        dists += c.dists;
        if (ok) {
            ++wins;
            if (lane == 0) {
                *cost_slot_of(A, e) = cost;
                A.flags[e] = 2;
            }
        }
    }
    if (A.stats && lane == 0) {
        atomicAdd(&A.stats[0], calls);
        atomicAdd(&A.stats[1], wins);
        atomicAdd(&A.stats[2], its);
        atomicAdd(&A.stats[3], nodes);
        atomicAdd(&A.stats[4], states);
        atomicAdd(&A.stats[5], dists);
    }
}

// ------------------------------------------------------------------ candidates
template <bool ARM, int W, int KP>
__global__ void __launch_bounds__(256) k_rrtc_vertices(RrtcArgs A, ArmParams R, SceneParams S, uint32_t nv,
                                                       uint8_t *vfree) {
    constexpr int D = StateDim<ARM, W>::D;
    const uint32_t i = blockIdx.x * blockDim.x + threadIdx.x;
    const uint32_t id = i < nv ? i : nv - 1;
    const float *p = vertex_ptr(A, id);
    float q[D];
#pragma unroll
    for (int k = 0; k < D; ++k) q[k] = k < A.d ? p[k] : 0.f;
    const float gap = state_gap<ARM, W, KP>(R, S, q);
    if (i < nv) vfree[i] = gap > 0.f ? 1 : 0;
}

// The same through the obstacle bins: eight vertices per wave.
template <int WORDS>
__global__ void __launch_bounds__(256) k_rrtc_vertices_bins(RrtcArgs A, const ArmParams *Rg, const ObsGrid *grid,
                                                            uint32_t nv, uint8_t *vfree) {
    __shared__ GridLds<WORDS> bins;
    __shared__ SphereTab T;
    __shared__ float4 og[256 / kWave][kRrtcStates * (GTMP_MAX_JOINTS + 1)];
    __shared__ float2 sc[256 / kWave][kRrtcStates * GTMP_MAX_JOINTS];
    copy_to_lds<grid_lds_bytes<WORDS>(), 256>(&bins, grid, threadIdx.x);
    const carm Rp = (carm)Rg;
    for (int k = threadIdx.x; k < Rg->n_spheres; k += 256) {
        T.t[k] = Rg->t[k];
        T.r[k] = Rg->r[k];
        T.link[k] = Rg->link[k];
    }
    __syncthreads();
    const uint32_t wv = wave_in_block();
    const int lane = lane_id(), j = lane & 7;
    const uint32_t id0 = (blockIdx.x * (256 / kWave) + wv) * kRrtcStates;
    if (id0 >= nv) return;
    const uint32_t left = nv - id0;
    const int ns = left < (uint32_t)kRrtcStates ? (int)left : kRrtcStates;
    float x = 0.f;
    if ((lane >> 3) < ns && j < A.d) x = vertex_ptr(A, id0 + (lane >> 3))[j] + Rg->off[j];
    const uint32_t hit = arm_hit8<WORDS, false>(*Rp, T, *reinterpret_cast<const ObsGrid *>(&bins), x, ns, og[wv], sc[wv]);
    if (lane < ns) vfree[id0 + lane] = (hit >> lane) & 1u ? 0 : 1;
}

// The obstacle bins (block 0) and the robot table (block 1) in device memory.
__global__ void __launch_bounds__(kGridBuildThreads) k_rrtc_bins(SceneParams S, GridBuild B, ObsGrid *G, ArmParams R,
                                                                 ArmParams *dst) {
    if (blockIdx.x == 0) {
        build_grid_block(S, 3, B, G);
        // a sphere whose centre is not a number touches nothing in the general
        // test; as a box of that centre it would span the axis
        const int o = threadIdx.x;  // the thread that wrote the record
        if (o < S.n_sph) {
            const float4 c = G->rec[o][0];
            if (__builtin_isnan(c.x) || __builtin_isnan(c.y) || __builtin_isnan(c.z)) G->rec[o][0].w = __builtin_nanf("");
        }
        return;
    }
    const uint32_t *src = reinterpret_cast<const uint32_t *>(&R);
    constexpr int n = sizeof(ArmParams) / 4;
    for (int i = threadIdx.x; i < n; i += kGridBuildThreads) reinterpret_cast<uint32_t *>(dst)[i] = src[i];
}

// counters: candidates, their cursor, calls to run again, their cursor
constexpr int kRrtcCounters = 4;
__global__ void k_rrtc_reset(uint32_t *counters) {
    if (threadIdx.x < kRrtcCounters) counters[threadIdx.x] = 0;
}

// Edges whose straight line failed with both endpoints free and within the
// length limit; appended in any order (each call is independent).
__global__ void __launch_bounds__(256) k_rrtc_collect(RrtcArgs A, const uint8_t *vfree, float max_len, uint64_t E,
                                                      uint32_t *cand, uint32_t *n_cand) {
    const uint64_t e = (uint64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (e >= E || A.flags[e] != 1) return;
    uint32_t u, v;
    edge_vertex_ids(A, e, u, v);
    if (!vfree[u] || !vfree[v]) return;
    const float *pu = vertex_ptr(A, u), *pv = vertex_ptr(A, v);
    float a[GTMP_MAX_DOF], b[GTMP_MAX_DOF];
    for (int i = 0; i < GTMP_MAX_DOF; ++i) {
        a[i] = i < A.d ? pu[i] : 0.f;
        b[i] = i < A.d ? pv[i] : 0.f;
    }
    if (edge_len<GTMP_MAX_DOF>(a, b, A.d) > max_len) return;  // as the edge check measures it
    cand[atomicAdd(n_cand, 1u)] = (uint32_t)e;
}

// The calls whose pool ran out, to run again.
__global__ void __launch_bounds__(256) k_rrtc_again(uint64_t E, uint8_t *flags, uint32_t *cand, uint32_t *n_cand) {
    const uint64_t e = (uint64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (e >= E || flags[e] != kRrtcAgain) return;
    flags[e] = 1;
    cand[atomicAdd(n_cand, 1u)] = (uint32_t)e;
}

// ------------------------------------------------------------------ host side
static size_t up256_r(size_t x) { return (x + 255) & ~size_t(255); }

RrtcPlan make_rrtc_plan(const gtmp_problem &p) {
    RrtcPlan r{};
    const uint64_t N = p.N, M = p.M, G = p.G;
    const uint64_t E = N + (M - 1) * N * N + N * G;
    const uint64_t nv = 1 + M * N + G;
    size_t off = 0;
    r.off_counters = off; off = up256_r(off + 64);
    r.off_grid = off; off = up256_r(off + sizeof(ObsGrid));
    r.off_params = off; off = up256_r(off + sizeof(ArmParams));
    r.off_vfree = off; off = up256_r(off + nv);
    r.off_cand = off; off = up256_r(off + sizeof(uint32_t) * E);
    r.total = off;
    return r;
}

// The bound on tree_cap that callers are held to: both trees of 2 d + 4 words
// a node (the pools take less).
size_t rrtc_lds_bytes(int d, int cap) {
    return sizeof(float) * ((size_t)2 * d * cap + (size_t)4 * cap + GTMP_MAX_DOF * GTMP_MAX_DOF);
}

static RrtcArgs rrtc_args(const gtmp_problem &p, const float *q0, const float *goals, const float *Q, float *C_s,
                          float *C_h, float *C_l, uint8_t *flags, uint64_t seed, uint64_t stage, const gtmp_rrtc_opts &o) {
    RrtcArgs A{};
    A.d = p.d; A.M = p.M; A.N = p.N; A.G = p.G;
    A.q0 = q0; A.goals = goals; A.Q = Q;
    for (int i = 0; i < GTMP_MAX_DOF; ++i) {
        A.lo[i] = i < p.d ? p.lo[i] : 0.f;
        A.hi[i] = i < p.d ? p.hi[i] : 0.f;
    }
    A.C_s = C_s; A.C_h = C_h; A.C_l = C_l; A.flags = flags;
    A.budget = o.budget; A.cap = o.tree_cap;
    A.eta = o.step; A.res = o.resolution; A.ell_factor = o.ell_factor;
    A.k0 = (uint32_t)(seed & 0xffffffffu);
    A.k1 = (uint32_t)(seed >> 32);
    A.stage = (uint32_t)(stage & 0xffffffffu);
    A.stats = o.stats;
    return A;
}

// Waves per block of the shared-LDS launches and the LDS of a block four of
// which fit in a CU's 160 KiB (four waves per SIMD, what the registers allow:
// a wave's steps are chains of LDS and scalar latencies).  213 nodes a wave
// for seven joints among 32 obstacles; the calls of the figures above hold 40
// nodes on average at budget 100, 77 at 400.
constexpr int kRrtcWaves = 4;
constexpr uint32_t kRrtcBlockLds = 40960;

struct RrtcLaunch {
    RrtcArgs A;
    ArmParams R;
    SceneParams S;
    uint64_t E;
    float max_len;
    uint8_t *vfree, *flags;
    uint32_t *cand, *counters;
    ObsGrid *grid;
    ArmParams *table;
    hipStream_t s;
};

// Calls of the list (counters[0], [1]: length and cursor) by kern: blocks of
// `waves` waves whose layout is Y.
template <class K>
static hipError_t launch_calls(const RrtcLaunch &L, K kern, const RrtcLayout &Y, uint32_t *counters) {
    RrtcArgs B = L.A;
    B.cand = L.cand;
    B.n_cand = counters;
    B.cursor = counters + 1;
    hipError_t e = hipFuncSetAttribute((const void *)kern, hipFuncAttributeMaxDynamicSharedMemorySize, (int)Y.total);
    if (e != hipSuccess) return e;
    int dev = 0, cus = 256, occ = 0;
    if (hipGetDevice(&dev) == hipSuccess) {
        int v = 0;
        if (hipDeviceGetAttribute(&v, hipDeviceAttributeMultiprocessorCount, dev) == hipSuccess && v > 0) cus = v;
    }
    if (hipOccupancyMaxActiveBlocksPerMultiprocessor(&occ, (const void *)kern, Y.waves * kWave, Y.total) != hipSuccess ||
        occ <= 0)
        occ = 1;
    occ = occ < 16 ? occ : 16;
    hipLaunchKernelGGL(kern, dim3(cus * occ), dim3(Y.waves * kWave), Y.total, L.s, B, L.R, L.S, Y, L.grid, L.table);
    return hipGetLastError();
}

// The list by `shared` (four calls per block, the pools sharing kRrtcBlockLds),
// then the calls whose pool ran out by `whole` (a call per block, its pool
// holding both trees).  Pools that hold both trees from the start need no
// second launch.
template <class KS, class KW>
static hipError_t launch_list(const RrtcLaunch &L, KS shared, KW whole, uint32_t bins, uint32_t tab, bool grid) {
    const int all = 2 * L.A.cap;
    int pool = all;
    RrtcLayout Y = rrtc_layout(L.A.d, pool, kRrtcWaves, bins, tab, grid);
    if (Y.total > kRrtcBlockLds) {
        const uint32_t fixed = rrtc_layout(L.A.d, 0, kRrtcWaves, bins, tab, grid).total + kRrtcWaves * 64u;
        pool = (int)((kRrtcBlockLds - fixed) / (kRrtcWaves * (4u * L.A.d + 4u)));
        Y = rrtc_layout(L.A.d, pool, kRrtcWaves, bins, tab, grid);
    }
    hipError_t e = launch_calls(L, shared, Y, L.counters);
    if (e != hipSuccess || pool >= all) return e;
    hipLaunchKernelGGL(k_rrtc_again, dim3((unsigned)((L.E + 255) / 256)), dim3(256), 0, L.s, L.E, L.flags, L.cand,
                       L.counters + 2);
    return launch_calls(L, whole, rrtc_layout(L.A.d, all, 1, bins, tab, grid), L.counters + 2);
}

static void launch_candidates(const RrtcLaunch &L) {
    hipLaunchKernelGGL(k_rrtc_reset, dim3(1), dim3(64), 0, L.s, L.counters);
    hipLaunchKernelGGL(k_rrtc_collect, dim3((unsigned)((L.E + 255) / 256)), dim3(256), 0, L.s, L.A, L.vfree, L.max_len,
                       L.E, L.cand, L.counters);
}

static uint32_t rrtc_vertex_count(const RrtcArgs &A) { return 1 + (uint32_t)A.M * A.N + A.G; }

// Arms behind the obstacle bins.
template <int WORDS>
static hipError_t launch_rrtc_bins(const RrtcLaunch &L) {
    const uint32_t nv = rrtc_vertex_count(L.A), per = kRrtcStates * (256 / kWave);
    float r_max = 0.f;
    for (int k = 0; k < L.R.n_spheres; ++k) r_max = r_max > L.R.r[k] ? r_max : L.R.r[k];
    hipLaunchKernelGGL(k_rrtc_bins, dim3(2), dim3(kGridBuildThreads), 0, L.s, L.S,
                       grid_build_arm(r_max, 0.f, 0.f, 1), L.grid, L.R, L.table);
    hipLaunchKernelGGL(k_rrtc_vertices_bins<WORDS>, dim3((nv + per - 1) / per), dim3(256), 0, L.s, L.A, L.table, L.grid, nv,
                       L.vfree);
    launch_candidates(L);
    return launch_list(L, k_rrtc<true, 3, 1, WORDS, kRrtcWaves, 4>, k_rrtc<true, 3, 1, WORDS, 1, 2>,
                       (uint32_t)grid_lds_bytes<WORDS>(), (uint32_t)sizeof(SphereTab), true);
}

// Point robots, arms among more obstacles than the bins hold, and the local
// path of one edge (no workspace to build bins in).
template <bool ARM, int W, int KP>
static hipError_t launch_rrtc_kernels(const RrtcLaunch &L, bool single) {
    constexpr int PW = ARM ? 3 : W;
    const int obs = L.S.n_sph * (PW + 1) + L.S.n_box * 2 * PW;
    const uint32_t tab = obs <= kRrtcLdsObstacles ? (uint32_t)sizeof(float) * obs : 0u;
    const RrtcLayout Y = rrtc_layout(L.A.d, 2 * L.A.cap, 1, 0u, tab, false);
    // registers for one wave a SIMD: an arm's spheres take all 256 (made for
    // two waves it spills 66 of them; 97 obstacles, M 3, N 48, trees of 256,
    // budget 60: 2.47 ms against 3.25 for 40 spheres, 4.38 against 5.67 for 64,
    // the same up to 24), a point's 96 leave room for five either way
    const auto kern = k_rrtc<ARM, W, KP, 0, 1, 1>;
    if (single) {
        hipError_t e = hipFuncSetAttribute((const void *)kern, hipFuncAttributeMaxDynamicSharedMemorySize, (int)Y.total);
        if (e != hipSuccess) return e;
        hipLaunchKernelGGL(kern, dim3(1), dim3(kWave), Y.total, L.s, L.A, L.R, L.S, Y, (const ObsGrid *)nullptr,
                           (const ArmParams *)nullptr);
        return hipGetLastError();
    }
    const uint32_t nv = rrtc_vertex_count(L.A);
    hipLaunchKernelGGL((k_rrtc_vertices<ARM, W, KP>), dim3((nv + 255) / 256), dim3(256), 0, L.s, L.A, L.R, L.S, nv,
                       L.vfree);
    launch_candidates(L);
    if constexpr (ARM) return launch_calls(L, kern, Y, L.counters);
    else return launch_list(L, k_rrtc<false, W, 1, 0, kRrtcWaves, 4>, kern, 0u, tab, false);
}

static hipError_t dispatch_rrtc(const ArmParams *arm, int wdim, RrtcLaunch &L, bool single) {
    if (arm) {
        L.R = *arm;
        const int n_obs = L.S.n_sph + L.S.n_box;
        if (!single) {
            switch (grid_words(n_obs)) {
                case 1: return launch_rrtc_bins<1>(L);
                case 2: return launch_rrtc_bins<2>(L);
                case 3: return launch_rrtc_bins<3>(L);
                default: break;
            }
        }
        switch (round8(L.R.n_spheres)) {
#define GTMP_RC(KP) case KP: return launch_rrtc_kernels<true, 3, KP>(L, single);
            GTMP_RC(8) GTMP_RC(16) GTMP_RC(24) GTMP_RC(32) GTMP_RC(40) GTMP_RC(48) GTMP_RC(56) GTMP_RC(64)
#undef GTMP_RC
            default: return hipErrorInvalidValue;
        }
    }
    if (wdim == 2) return launch_rrtc_kernels<false, 2, 1>(L, single);
    return launch_rrtc_kernels<false, 3, 1>(L, single);
}

hipError_t launch_rrtc_repair(const gtmp_problem &p, const ArmParams *arm, const SceneParams &S, int wdim,
                              const float *q0, const float *goals, const float *Q, float *C_s, float *C_h, float *C_l,
                              uint8_t *flags, uint64_t seed, uint64_t stage, const gtmp_rrtc_opts &o, void *workspace,
                              hipStream_t s, const uint32_t *stage_dev) {
    const RrtcPlan plan = make_rrtc_plan(p);
    char *ws = static_cast<char *>(workspace);
    const uint64_t N = p.N, M = p.M, G = p.G;
    const uint64_t E = N + (M - 1) * N * N + N * G;
    RrtcArgs A = rrtc_args(p, q0, goals, Q, C_s, C_h, C_l, flags, seed, stage, o);
    A.stage_dev = stage_dev;
    RrtcLaunch L{A, ArmParams{}, S, E, p.max_edge_len, reinterpret_cast<uint8_t *>(ws + plan.off_vfree), flags,
                 reinterpret_cast<uint32_t *>(ws + plan.off_cand), reinterpret_cast<uint32_t *>(ws + plan.off_counters),
                 reinterpret_cast<ObsGrid *>(ws + plan.off_grid),
                 reinterpret_cast<ArmParams *>(ws + plan.off_params), s};
    return dispatch_rrtc(arm, wdim, L, false);
}

hipError_t launch_rrtc_path(const gtmp_problem &p, const ArmParams *arm, const SceneParams &S, int wdim,
                            const float *q0, const float *goals, const float *Q, uint64_t edge, uint64_t seed,
                            uint64_t stage, const gtmp_rrtc_opts &o, float *path, int32_t *count, float *cost,
                            hipStream_t s) {
    RrtcArgs A = rrtc_args(p, q0, goals, Q, nullptr, nullptr, nullptr, nullptr, seed, stage, o);
    A.stats = nullptr;
    A.single = (uint32_t)edge;
    A.path = path;
    A.path_count = count;
    A.path_cost = cost;
    RrtcLaunch L{A, ArmParams{}, S, 1, p.max_edge_len, nullptr, nullptr, nullptr, nullptr, nullptr, nullptr, s};
    return dispatch_rrtc(arm, wdim, L, true);
}

}  // namespace gtmp
