// classes.hip -- class-augmented value iteration on the layered DAG (Sec. IV-B;
// Prop. 2) and the class-indexed archive of Anytime-GTMP (Sec. IV-D) for 2D
// point robots.
//
// Class label of an edge: its signed crossings with upward rays from up to 16
// representative obstacle points, one 8-bit field per point in a 128-bit
// label held as two 64-bit words (fields 0..7 in the first, 8..15 in the
// second).  A chain of at most 127 edges (M <= 126) crosses a ray at most 127
// times, so every count fits a field: chain labels are kept in offset binary
// (the empty label has every field at 128) and edge labels in two's
// complement, and a sum is a field-wise addition modulo 256 with no carries
// between fields (SWAR addition).  The crossing decision is taken in FP32
// with a fixed operation order; this file is compiled without contraction.
//
// Sweep: the list of a vertex u is what this sequential rule makes: for every
// successor v in index order the candidates kappa(u, v) + chi, C(u, v) +
// J(v, chi) are matched against u's entries, a lower cost replaces the entry's,
// a new label is appended in candidate order; when the list is full, a new
// label replaces the costliest entry if it is cheaper and the overflow counter
// counts every label dropped: results are exact whenever the counter stays
// zero.
// While a list is not full, the rule only keeps labels in order of first
// appearance with the first least cost, so runs of successors can be taken
// side by side and joined in order: a block of eight waves per vertex, a run
// of successors each, lane j of a wave holding entry j of its list, joined
// pairwise in three steps.  A list that would overflow anywhere is built again
// by one wave over all successors, by the rule itself.  A walk is a chain of
// memory round trips, so a wave loads the edges of up to 64 successors at once
// (their labels formed a successor per lane) and the next candidate list ahead.
// A layer of M 4, N 128 with 15 class points takes 21 us on average (one wave
// per vertex, one successor at a time: 130 us); what remains is the start
// vertex's list where it overflows (55-80 us).
#include "gtmp_launch.hpp"

namespace gtmp {

constexpr int kClassMaxReps = 16;
constexpr uint64_t kByteHigh = 0x8080808080808080ull;
constexpr uint64_t kEmptyWord = 0x8080808080808080ull;  // eight fields at zero, offset binary

struct Label {
    uint64_t w[2];
};

__device__ __forceinline__ uint64_t swar_add(uint64_t x, uint64_t y) {
    return ((x & ~kByteHigh) + (y & ~kByteHigh)) ^ ((x ^ y) & kByteHigh);
}

__device__ __forceinline__ Label label_add(const Label &a, const Label &b) {
    return Label{{swar_add(a.w[0], b.w[0]), swar_add(a.w[1], b.w[1])}};
}

__device__ __forceinline__ bool label_eq(const Label &a, const Label &b) {
    return a.w[0] == b.w[0] && a.w[1] == b.w[1];
}

// The class points in LDS (a read of memory per point inside the walk waited
// for memory k times); points past k are not looked at.
struct Reps {
    float x[kClassMaxReps], y[kClassMaxReps];
};

__device__ __forceinline__ uint32_t label_hash(const Label &a) {
    return (uint32_t)a.w[0] * 0x9E3779B1u ^ (uint32_t)(a.w[0] >> 32) * 0x85EBCA77u ^ (uint32_t)a.w[1] * 0xC2B2AE3Du ^
           (uint32_t)(a.w[1] >> 32) * 0x27D4EB2Fu;
}

// Signed crossings of u -> v with the upward rays of the k points, packed in
// two's complement.
__device__ __forceinline__ Label edge_label(float ux, float uy, float vx, float vy, const Reps &Z, int k) {
    Label lab{{0ull, 0ull}};
    const float dx = vx - ux, dy = vy - uy;
    const uint32_t field = dx > 0.f ? 1u : 255u;  // +1 or -1 mod 256
    uint32_t w[kClassMaxReps / 4] = {0u, 0u, 0u, 0u};
#pragma unroll
    for (int i = 0; i < kClassMaxReps; ++i) {
        const float ex = Z.x[i] - ux, ey = Z.y[i] - uy;
        const float cross = dx * ey - dy * ex;
        const bool above = dx > 0.f ? cross < 0.f : cross > 0.f;
        const bool on = i < k && (ux < Z.x[i]) != (vx < Z.x[i]) && above;
        w[i >> 2] |= on ? field << (8 * (i & 3)) : 0u;
    }
    lab.w[0] = (uint64_t)w[1] << 32 | w[0];
    lab.w[1] = (uint64_t)w[3] << 32 | w[2];
    return lab;
}

__device__ __forceinline__ uint64_t readlane64(uint64_t x, int l) {
    const uint32_t lo = __builtin_amdgcn_readlane((uint32_t)x, l);
    const uint32_t hi = __builtin_amdgcn_readlane((uint32_t)(x >> 32), l);
    return ((uint64_t)hi << 32) | lo;
}

__device__ __forceinline__ Label readlane_label(const Label &x, int l) {
    return Label{{readlane64(x.w[0], l), readlane64(x.w[1], l)}};
}

__device__ __forceinline__ uint64_t shfl64(uint64_t x, int l) {
    const uint32_t lo = (uint32_t)__shfl((int)(uint32_t)x, l);
    const uint32_t hi = (uint32_t)__shfl((int)(uint32_t)(x >> 32), l);
    return ((uint64_t)hi << 32) | lo;
}

__device__ __forceinline__ Label load_label(const uint64_t *p, size_t i) {
    const ulonglong2 v = reinterpret_cast<const ulonglong2 *>(p)[i];
    return Label{{v.x, v.y}};
}

__device__ __forceinline__ void store_label(uint64_t *p, size_t i, const Label &l) {
    reinterpret_cast<ulonglong2 *>(p)[i] = make_ulonglong2(l.w[0], l.w[1]);
}

struct ClassLists {
    uint64_t *lab;   // [M][N][L][2]
    float *cost;     // [M][N][L]
    uint32_t *nxt;   // [M][N][L]: successor << 8 | its entry
    int32_t *cnt;    // [M][N]
    uint64_t *s_lab; // start list [L][2]
    float *s_cost;
    uint32_t *s_nxt;
    int32_t *s_cnt;  // [1]
    uint32_t *overflow;  // [1] labels dropped by full lists
};

// A list: lane j holds entry j.
struct ClassList {
    Label lab;
    float cost;
    uint32_t nxt;
    int cnt;
    uint32_t dropped;
};

// The costliest of the list's entries (the highest lane among equals).
__device__ __forceinline__ int costliest(const ClassList &U, float &mx) {
    mx = lane_id() < U.cnt ? U.cost : -__builtin_inff();
#define GTMP_DPP_MAX(ctrl, rows)                                                                                  \
    mx = __builtin_fmaxf(mx, __int_as_float(__builtin_amdgcn_update_dpp(__float_as_int(mx), __float_as_int(mx), ctrl, \
                                                                        rows, 0xf, false)));
    GTMP_DPP_MAX(0x111, 0xf)  // row_shr:1
    GTMP_DPP_MAX(0x112, 0xf)  // row_shr:2
    GTMP_DPP_MAX(0x114, 0xf)  // row_shr:4
    GTMP_DPP_MAX(0x118, 0xf)  // row_shr:8
    GTMP_DPP_MAX(0x142, 0xa)  // row_bcast:15 into rows 1 and 3
    GTMP_DPP_MAX(0x143, 0xc)  // row_bcast:31 into rows 2 and 3
#undef GTMP_DPP_MAX
    mx = __int_as_float(__builtin_amdgcn_readlane(__float_as_int(mx), kWave - 1));
    return kWave - 1 - __builtin_clzll(ballot(lane_id() < U.cnt && U.cost == mx));
}

// The candidates of one successor (or list), one per lane, labels distinct,
// into U.  EXACT: a full list follows the replacement rule; otherwise false is
// returned and U is left as it was when the new labels do not fit.
template <bool EXACT>
__device__ __forceinline__ bool absorb(ClassList &U, int L, const Label &cl, float cc, uint32_t cn, int n_src) {
    const int lane = lane_id();
    // match: list lane j finds the candidate with its label (labels are
    // distinct within both), by broadcasting the fewer of candidates and
    // entries as 32-bit hashes; a pair that only the hash takes for equal shows
    // in the whole labels compared afterwards or in the number of pairs, and
    // the labels themselves are then broadcast
    uint64_t matched = 0;
    int src = -1;
    const uint32_t hu = label_hash(U.lab), hc = label_hash(cl);
    if (n_src <= U.cnt) {
        for (int e = 0; e < n_src; ++e) {
            const bool hit = lane < U.cnt && hu == (uint32_t)__builtin_amdgcn_readlane((int)hc, e);
            src = hit ? e : src;
            matched |= ballot(hit) != 0 ? 1ull << e : 0ull;
        }
    } else {
        for (int j = 0; j < U.cnt; ++j) {
            const uint64_t hit = ballot(lane < n_src && hc == (uint32_t)__builtin_amdgcn_readlane((int)hu, j));
            src = lane == j && hit != 0 ? __builtin_ctzll(hit) : src;
            matched |= hit;
        }
    }
    if (matched != 0) {
        const int from = src < 0 ? 0 : src;
        const Label l{{shfl64(cl.w[0], from), shfl64(cl.w[1], from)}};
        const bool wrong = src >= 0 && !label_eq(l, U.lab);
        if (ballot(wrong) != 0 || __popcll(matched) != __popcll(ballot(src >= 0))) {
            matched = 0;
            src = -1;
            for (int e = 0; e < n_src; ++e) {
                const bool hit = lane < U.cnt && label_eq(U.lab, readlane_label(cl, e));
                if (hit) src = e;
                if (ballot(hit) != 0) matched |= 1ull << e;
            }
        }
    }
    uint64_t pending = (n_src >= 64 ? ~0ull : ((1ull << n_src) - 1ull)) & ~matched;
    const int n_new = __popcll(pending), room = L - U.cnt;
    if (!EXACT && n_new > room) return false;
    if (matched != 0) {
        const float pc = __shfl(cc, src < 0 ? 0 : src);
        const uint32_t pn = (uint32_t)__shfl((int)cn, src < 0 ? 0 : src);
        if (src >= 0 && pc < U.cost) {
            U.cost = pc;
            U.nxt = pn;
        }
    }
    if (n_new == 0) return true;
    // new labels: appended in candidate order while there is room
    const int n_app = n_new < room ? n_new : room;
    if (n_app > 0) {
        int asrc = -1;
        for (int idx = 0; idx < n_app; ++idx) {
            const int e = __builtin_ctzll(pending);
            pending &= pending - 1;
            if (lane == U.cnt + idx) asrc = e;
        }
        const int from = asrc < 0 ? 0 : asrc;
        const Label pl{{shfl64(cl.w[0], from), shfl64(cl.w[1], from)}};
        const float pc = __shfl(cc, from);
        const uint32_t pn = (uint32_t)__shfl((int)cn, from);
        if (asrc >= 0) {
            U.lab = pl;
            U.cost = pc;
            U.nxt = pn;
        }
        U.cnt += n_app;
    }
    if constexpr (EXACT) {
        // full list: each remaining label replaces the costliest entry if
        // cheaper; that entry's cost never rises, so a candidate that is not
        // cheaper now is not later either
        U.dropped += (uint32_t)__popcll(pending);  // either the label or the one it replaces
        while (pending != 0) {
            float mx;
            const int arg = costliest(U, mx);
            pending &= ballot(cc < mx);
            if (pending == 0) break;
            const int e = __builtin_ctzll(pending);
            pending &= pending - 1;
            const Label el = readlane_label(cl, e);
            const float ec = __uint_as_float(__builtin_amdgcn_readlane(__float_as_uint(cc), e));
            const uint32_t en = __builtin_amdgcn_readlane(cn, e);
            if (lane == arg) {
                U.lab = el;
                U.cost = ec;
                U.nxt = en;
            }
        }
    }
    return true;
}

struct ClassArgs {
    int m, M, N, G, L, k;
    const float *Q, *q0, *goals, *C_s, *C_h, *C_l, *reps;
    float penalty;
};

// Successors [v0, v1) of vertex u into U in index order; false when a list
// that is not EXACT overflows.
template <bool EXACT>
__device__ __forceinline__ bool walk(const ClassArgs &A, const ClassLists &CL, int u, int v0, int v1,
                                     const Reps &Z, ClassList &U) {
    const int lane = lane_id(), m = A.m, N = A.N, L = A.L;
    const bool last = m == A.M - 1;
    const float *pu = m < 0 ? A.q0 : A.Q + ((size_t)m * N + u) * 2;
    const float *row = m < 0 ? A.C_s : last ? A.C_l + (size_t)u * A.G : A.C_h + ((size_t)m * N + u) * N;
    const float *succ = last ? A.goals : A.Q + (size_t)(m + 1) * N * 2;  // layer 0 for the start
    const size_t first = (size_t)(m + 1) * N;
    const float ux = pu[0], uy = pu[1];
    for (int base = v0; base < v1; base += kWave) {
        const int v = base + lane;
        float c = __builtin_inff();
        int ns = 0;
        Label kap{{0ull, 0ull}};
        if (v < v1) {
            c = row[v];
            ns = last ? 1 : CL.cnt[first + v];
            kap = edge_label(ux, uy, succ[2 * v], succ[2 * v + 1], Z, A.k);
        }
        uint64_t live = ballot(c < A.penalty && ns > 0);  // absent and failed edges are skipped
        // the next successor's candidates are requested before this one's are absorbed
        int b = 0, n = 0;
        Label cl{{kEmptyWord, kEmptyWord}};
        float cc = 0.f;
        auto next = [&]() {
            n = 0;
            if (live == 0) return;
            b = __builtin_ctzll(live);
            live &= live - 1;
            n = __builtin_amdgcn_readlane(ns, b);
            if (!last && lane < n) {
                const size_t at = (first + base + b) * L + lane;
                cl = load_label(CL.lab, at);
                cc = CL.cost[at];
            }
        };
        next();
        while (n != 0) {
            const float ce = __uint_as_float(__builtin_amdgcn_readlane(__float_as_uint(c), b));
            const Label l = label_add(readlane_label(kap, b), cl);
            const float cost = last ? ce : ce + cc;
            const uint32_t cn = ((uint32_t)(base + b) << 8) | (last ? 0u : (uint32_t)lane);
            const int ne = n;
            next();
            if (!absorb<EXACT>(U, L, l, cost, cn, ne)) return false;
        }
    }
    return true;
}

constexpr int kClassWaves = 8;  // waves (runs of successors) per vertex

// A block per vertex u of layer A.m (-1: the start vertex).
__global__ void __launch_bounds__(kClassWaves *kWave) k_class_layer(ClassArgs A, ClassLists CL) {
    __shared__ Label lab_s[kClassWaves][kWave];
    __shared__ float cost_s[kClassWaves][kWave];
    __shared__ uint32_t nxt_s[kClassWaves][kWave];
    __shared__ int cnt_s[kClassWaves], over_s;
    const int u = blockIdx.x, lane = lane_id(), w = (int)wave_in_block();
    const int nv = A.m == A.M - 1 ? A.G : A.N;
    const int per = (nv + kClassWaves - 1) / kClassWaves;
    ClassList U{Label{{0ull, 0ull}}, __builtin_inff(), 0u, 0, 0u};
    __shared__ Reps Z;
    if ((int)threadIdx.x < kClassMaxReps) {
        const int i = threadIdx.x;
        Z.x[i] = i < A.k ? A.reps[2 * i] : 0.f;
        Z.y[i] = i < A.k ? A.reps[2 * i + 1] : 0.f;
    }
    if (threadIdx.x == 0) over_s = 0;
    __syncthreads();
    {
        const int v0 = w * per < nv ? w * per : nv, v1 = v0 + per < nv ? v0 + per : nv;
        if (!walk<false>(A, CL, u, v0, v1, Z, U) && lane == 0) over_s = 1;
    }
    auto publish = [&]() {
        lab_s[w][lane] = U.lab;
        cost_s[w][lane] = U.cost;
        nxt_s[w][lane] = U.nxt;
        if (lane == 0) cnt_s[w] = U.cnt;
    };
#pragma unroll
    for (int step = 1; step < kClassWaves; step <<= 1) {  // list w takes list w + step
        if ((w & (2 * step - 1)) == step) publish();
        __syncthreads();
        if ((w & (2 * step - 1)) == 0) {
            const int o = w + step, n = cnt_s[o];
            if (n > 0 && over_s == 0 && !absorb<false>(U, A.L, lab_s[o][lane], cost_s[o][lane], nxt_s[o][lane], n) &&
                lane == 0)
                over_s = 1;
        }
        __syncthreads();
    }
    if (w != 0) return;
    if (over_s != 0) {
        U = ClassList{Label{{0ull, 0ull}}, __builtin_inff(), 0u, 0, 0u};
        walk<true>(A, CL, u, 0, nv, Z, U);
    }
    // store u's list
    if (A.m < 0) {
        if (lane < U.cnt) {
            store_label(CL.s_lab, lane, U.lab);
            CL.s_cost[lane] = U.cost;
            CL.s_nxt[lane] = U.nxt;
        }
        if (lane == 0) *CL.s_cnt = U.cnt;
    } else {
        const size_t base = ((size_t)A.m * A.N + u) * A.L;
        if (lane < U.cnt) {
            store_label(CL.lab, base + lane, U.lab);
            CL.cost[base + lane] = U.cost;
            CL.nxt[base + lane] = U.nxt;
        }
        if (lane == 0) CL.cnt[(size_t)A.m * A.N + u] = U.cnt;
    }
    if (lane == 0 && U.dropped) atomicAdd(CL.overflow, U.dropped);
}

// Chains of the start list: lane e follows entry e through the layers.
__global__ void __launch_bounds__(64) k_class_extract(int M, int N, int L, ClassLists CL, uint64_t *labels,
                                                      float *costs, int32_t *chains, int32_t *count) {
    const int e = threadIdx.x;
    const int n = *CL.s_cnt;
    if (e == 0) *count = n;
    if (e >= n) return;
    labels[2 * e] = CL.s_lab[2 * e];
    labels[2 * e + 1] = CL.s_lab[2 * e + 1];
    costs[e] = CL.s_cost[e];
    uint32_t nx = CL.s_nxt[e];
    for (int m = 0; m < M; ++m) {
        const int v = (int)(nx >> 8), ent = (int)(nx & 0xffu);
        chains[(size_t)e * (M + 1) + m] = v;
        nx = CL.nxt[((size_t)m * N + v) * L + ent];
    }
    chains[(size_t)e * (M + 1) + M] = (int)(nx >> 8);
}

__global__ void k_class_reset(uint32_t *overflow) {
    if (threadIdx.x == 0 && blockIdx.x == 0) *overflow = 0u;
}

// Class-indexed archive update (one block): per label the lowest cost, a later
// stage replacing an entry only with a strictly lower cost; waypoints copied
// from this stage's samples.  The labels of one stage are distinct, so only
// entries of earlier stages (the first na0) can match: the classes are looked
// up side by side, a wave each, the new ones then take slots in class order
// (one wave taking the classes in turn: 33 us a stage against 6.5).
constexpr int kArchiveThreads = 1024;

__global__ void __launch_bounds__(kArchiveThreads) k_class_archive(int M, int N, int stage, const float *__restrict__ Q,
                                                                   const float *__restrict__ q0,
                                                                   const float *__restrict__ goals,
                                                                   const uint64_t *labels, const float *costs,
                                                                   const int32_t *chains, const int32_t *count, int cap,
                                                                   uint64_t *a_lab, float *a_cost, int32_t *a_stage,
                                                                   float *a_wp, int32_t *a_count, uint32_t *overflow) {
    __shared__ int slot_s[kWave];  // per class: its archive slot, -1 new, -2 none
    const int lane = lane_id(), w = (int)wave_in_block();
    constexpr int kWaves = kArchiveThreads / kWave;
    const int n = *count;  // at most kWave
    const int na0 = *a_count;
    for (int e = w; e < n; e += kWaves) {
        const Label lab{{labels[2 * e], labels[2 * e + 1]}};
        int found = -1;
        for (int base = 0; base < na0 && found < 0; base += 4 * kWave) {
            bool hit[4];
#pragma unroll
            for (int q = 0; q < 4; ++q) {
                const int j = base + q * kWave + lane;
                hit[q] = j < na0 && a_lab[2 * j] == lab.w[0] && a_lab[2 * j + 1] == lab.w[1];
            }
#pragma unroll
            for (int q = 3; q >= 0; --q) {
                const uint64_t b = ballot(hit[q]);
                if (b != 0) found = base + q * kWave + __builtin_ctzll(b);
            }
        }
        if (lane == 0) slot_s[e] = found < 0 ? -1 : costs[e] < a_cost[found] ? found : -2;
    }
    __syncthreads();
    if (w == 0) {
        const bool fresh = lane < n && slot_s[lane] == -1;
        const uint64_t b = ballot(fresh);
        const int s = na0 + rank_in(b), total = __popcll(b);
        if (fresh) slot_s[lane] = s < cap ? s : -2;
        const int left = cap > na0 ? cap - na0 : 0, room = left < total ? left : total;
        if (lane == 0) {
            *a_count = na0 + room;
            if (total > room) atomicAdd(overflow, (uint32_t)(total - room));
        }
    }
    __syncthreads();
    for (int e = w; e < n; e += kWaves) {
        const int slot = slot_s[e];
        if (slot < 0) continue;
        if (lane == 0) {
            a_lab[2 * slot] = labels[2 * e];  // the caller's array: 8-byte words
            a_lab[2 * slot + 1] = labels[2 * e + 1];
            a_cost[slot] = costs[e];
            a_stage[slot] = stage;
        }
        // waypoints q0, Q[0][i0], ..., Q[M-1][i_{M-1}], goal
        const int32_t *ch = chains + (size_t)e * (M + 1);
        float *wp = a_wp + (size_t)slot * (M + 2) * 2;
        for (int p = lane; p < M + 2; p += kWave) {
            const float *src = p == 0 ? q0 : (p <= M ? Q + ((size_t)(p - 1) * N + ch[p - 1]) * 2 : goals + (size_t)ch[M] * 2);
            wp[2 * p] = src[0];
            wp[2 * p + 1] = src[1];
        }
    }
}

// ------------------------------------------------------------------ host side
static size_t up256c(size_t x) { return (x + 255) & ~size_t(255); }

ClassPlan make_class_plan(int M, int N, int L) {
    ClassPlan p{};
    size_t o = 0;
    const size_t e = (size_t)M * N * L;
    p.off_lab = o; o = up256c(o + 2 * sizeof(uint64_t) * e);
    p.off_cost = o; o = up256c(o + sizeof(float) * e);
    p.off_nxt = o; o = up256c(o + sizeof(uint32_t) * e);
    p.off_cnt = o; o = up256c(o + sizeof(int32_t) * (size_t)M * N);
    p.off_s = o; o = up256c(o + (2 * sizeof(uint64_t) + sizeof(float) + sizeof(uint32_t)) * (size_t)L + 64);
    p.total = o;
    return p;
}

static ClassLists carve_lists(const ClassPlan &p, int L, void *ws, uint32_t *overflow) {
    char *w = static_cast<char *>(ws);
    ClassLists CL{};
    CL.lab = reinterpret_cast<uint64_t *>(w + p.off_lab);
    CL.cost = reinterpret_cast<float *>(w + p.off_cost);
    CL.nxt = reinterpret_cast<uint32_t *>(w + p.off_nxt);
    CL.cnt = reinterpret_cast<int32_t *>(w + p.off_cnt);
    char *s = w + p.off_s;
    CL.s_lab = reinterpret_cast<uint64_t *>(s);
    CL.s_cost = reinterpret_cast<float *>(s + 2 * sizeof(uint64_t) * L);
    CL.s_nxt = reinterpret_cast<uint32_t *>(s + (2 * sizeof(uint64_t) + sizeof(float)) * L);
    CL.s_cnt = reinterpret_cast<int32_t *>(s + (2 * sizeof(uint64_t) + sizeof(float) + sizeof(uint32_t)) * L);
    CL.overflow = overflow;
    return CL;
}

hipError_t launch_class_sweep(int M, int N, int G, int L, const float *Q, const float *q0, const float *goals,
                              const float *C_s, const float *C_h, const float *C_l, float penalty, const float *reps,
                              int k, uint64_t *labels, float *costs, int32_t *chains, int32_t *count,
                              uint32_t *overflow, bool reset_overflow, void *ws, hipStream_t s) {
    const ClassPlan p = make_class_plan(M, N, L);
    const ClassLists CL = carve_lists(p, L, ws, overflow);
    if (reset_overflow) hipLaunchKernelGGL(k_class_reset, dim3(1), dim3(64), 0, s, overflow);
    ClassArgs A{0, M, N, G, L, k, Q, q0, goals, C_s, C_h, C_l, reps, penalty};
    for (A.m = M - 1; A.m >= -1; --A.m)
        hipLaunchKernelGGL(k_class_layer, dim3(A.m < 0 ? 1u : (unsigned)N), dim3(kClassWaves * kWave), 0, s, A, CL);
    hipLaunchKernelGGL(k_class_extract, dim3(1), dim3(64), 0, s, M, N, L, CL, labels, costs, chains, count);
    return hipGetLastError();
}

hipError_t launch_class_archive(int M, int N, int stage, const float *Q, const float *q0, const float *goals,
                                const uint64_t *labels, const float *costs, const int32_t *chains,
                                const int32_t *count, int cap, uint64_t *a_lab, float *a_cost, int32_t *a_stage,
                                float *a_wp, int32_t *a_count, uint32_t *overflow, hipStream_t s) {
    hipLaunchKernelGGL(k_class_archive, dim3(1), dim3(kArchiveThreads), 0, s, M, N, stage, Q, q0, goals, labels, costs,
                       chains, count, cap, a_lab, a_cost, a_stage, a_wp, a_count, overflow);
    return hipGetLastError();
}

ClassAnytimePlan make_class_anytime_plan(const gtmp_problem &p, int L) {
    ClassAnytimePlan a{};
    const uint64_t M = p.M, N = p.N, G = p.G;
    size_t o = 0;
    a.off_Q = o; o = up256c(o + sizeof(float) * M * N * 2);
    a.off_Cs = o; o = up256c(o + sizeof(float) * N);
    a.off_Ch = o; o = up256c(o + sizeof(float) * (M > 1 ? M - 1 : 1) * N * N);
    a.off_Cl = o; o = up256c(o + sizeof(float) * N * G);
    a.off_out = o; o = up256c(o + (2 * sizeof(uint64_t) + sizeof(float)) * (size_t)L + sizeof(int32_t) * (size_t)L * (M + 1) + 64);
    const EdgePlan ep = make_edge_plan(p);
    a.off_edge = o; o = up256c(o + ep.total);
    const ClassPlan cp = make_class_plan(p.M, p.N, L);
    a.off_class = o; o = up256c(o + cp.total);
    a.total = o;
    return a;
}

__global__ void k_class_archive_init(int32_t *a_count, uint32_t *overflow) {
    if (threadIdx.x == 0 && blockIdx.x == 0) {
        *a_count = 0;
        *overflow = 0u;
    }
}

hipError_t launch_plan_classes(const gtmp_problem &p, const SceneParams &scene, const float *q0, const float *goals,
                               uint64_t seed, int stages, const float *reps, int k, int L, int cap, uint64_t *a_lab,
                               float *a_cost, int32_t *a_stage, float *a_wp, int32_t *a_count, uint32_t *overflow,
                               const gtmp_edge_opts &eo, void *workspace, hipStream_t s) {
    const ClassAnytimePlan a = make_class_anytime_plan(p, L);
    char *ws = static_cast<char *>(workspace);
    float *Q = reinterpret_cast<float *>(ws + a.off_Q);
    float *Cs = reinterpret_cast<float *>(ws + a.off_Cs);
    float *Ch = reinterpret_cast<float *>(ws + a.off_Ch);
    float *Cl = reinterpret_cast<float *>(ws + a.off_Cl);
    char *out = ws + a.off_out;
    uint64_t *labels = reinterpret_cast<uint64_t *>(out);
    float *costs = reinterpret_cast<float *>(out + 2 * sizeof(uint64_t) * L);
    int32_t *chains = reinterpret_cast<int32_t *>(out + (2 * sizeof(uint64_t) + sizeof(float)) * L);
    int32_t *count = reinterpret_cast<int32_t *>(out + (2 * sizeof(uint64_t) + sizeof(float)) * L +
                                                 sizeof(int32_t) * (size_t)L * (p.M + 1));
    hipLaunchKernelGGL(k_class_archive_init, dim3(1), dim3(64), 0, s, a_count, overflow);
    const EdgePlan ep = make_edge_plan(p);
    gtmp_edge_opts e2 = eo;
    e2.ev_begin = nullptr;
    e2.ev_end = nullptr;
    for (int st = 0; st < stages; ++st) {
        hipError_t e = launch_sample_layers(p, seed, (uint64_t)st, Q, s);
        if (e != hipSuccess) return e;
        EdgeBuffers b{q0, goals, Q, Cs, Ch, Cl, nullptr, nullptr, nullptr, ws + a.off_edge};
        e = launch_edge_check(ep, nullptr, scene, 2, b, e2, s);
        if (e != hipSuccess) return e;
        e = launch_class_sweep(p.M, p.N, p.G, L, Q, q0, goals, Cs, Ch, Cl, p.penalty, reps, k, labels, costs, chains,
                               count, overflow, false, ws + a.off_class, s);
        if (e != hipSuccess) return e;
        e = launch_class_archive(p.M, p.N, st, Q, q0, goals, labels, costs, chains, count, cap, a_lab, a_cost, a_stage,
                                 a_wp, a_count, overflow, s);
        if (e != hipSuccess) return e;
    }
    return hipSuccess;
}

}  // namespace gtmp
