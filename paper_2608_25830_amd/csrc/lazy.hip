// lazy.hip -- lazy edge realisation on the layered graph (the lazy variant
// that realises only a subset of adjacent-layer pairs, named as future work
// in the paper's conclusion): every edge starts at its optimistic cost (its
// length; length + penalty when an endpoint collides or it is too long), and
// rounds of
//   backward sweep -> extraction -> stop if every edge of the path is known
//   -> forward sweep -> check the unknown edges whose best path through them
//      costs at most (1 + band) V_s, and those of the extracted path
// run until the extracted path holds only checked edges.  Checked costs are
// the true ones and unchecked costs are lower bounds, so the final path is
// optimal for the fully checked graph and its cost is the same FP32 number
// the full check gives (same edge costs, same summation order).
//
// Edge status (flags): 0 free, 1 failed, 0xFF not yet checked.
#include "edge_common.hpp"

namespace gtmp {

constexpr uint8_t kUnknown = 0xFF;

struct LazyArgs {
    int d, M, N, G;
    float penalty, max_len;
    const float *verts;    // packed vertices [1 + MN + G][vertex_stride]
    const uint8_t *vflag;  // vertex collision flags
    float *C_s, *C_h, *C_l;
    uint8_t *flags;
    const float *V, *F;  // cost-to-go [M][N], cost-from-start [M][N]
    const float *V_s;
    uint8_t *select;
    uint32_t *list;      // the round's selected edges (flat ids), counters[1] of them
    uint32_t *counters;  // [0] done, [1] edges selected this round, [2] unknown edges on the path
    unsigned long long *stats;  // optional: rounds, edges selected for checking
};

__device__ __forceinline__ void lazy_vertex_ids(const LazyArgs &A, uint64_t e, uint32_t &u, uint32_t &v, float *&c) {
    const uint64_t N = A.N, inner = (uint64_t)(A.M - 1) * N * N;
    if (e < N) {
        u = 0;
        v = 1 + (uint32_t)e;
        c = A.C_s + e;
    } else if (e - N < inner) {
        const uint64_t r = e - N, m = r / (N * N), uv = r - m * N * N;
        u = 1 + (uint32_t)(m * N + uv / N);
        v = 1 + (uint32_t)((m + 1) * N + uv % N);
        c = A.C_h + r;
    } else {
        const uint64_t r = e - N - inner, n = r / (uint64_t)A.G, g = r - n * A.G;
        u = 1 + (uint32_t)((A.M - 1) * N + n);
        v = 1 + (uint32_t)(A.M * N + g);
        c = A.C_l + r;
    }
}

// The passes over all edges (optimistic costs, selection) are bound by memory
// once nothing is decoded per edge: a block takes kLazyRows consecutive rows
// of C_h (a row: the edges of one source) by kLazyCols columns, four
// neighbouring columns a thread, so that costs move 16 bytes and statuses 4
// bytes at a time (VEC: rows and arrays aligned to that; otherwise the four
// columns lie 256 apart).  A block's rows may cross into the next layer; each
// row knows its own.  The last blocks take the edges of the start and the
// goals, one a thread.
constexpr int kLazyRows = 8, kLazyCols = 1024;

struct LazyGrid {
    uint32_t segs, inner, edge_blocks;  // column segments, blocks of inner rows, blocks of the other edges
};
static LazyGrid lazy_grid(const gtmp_problem &p) {
    LazyGrid g{};
    g.segs = (uint32_t)((p.N + kLazyCols - 1) / kLazyCols);
    const uint64_t rows = (uint64_t)(p.M - 1) * p.N;
    g.inner = (uint32_t)((rows + kLazyRows - 1) / kLazyRows) * g.segs;
    g.edge_blocks = (uint32_t)(((uint64_t)p.N * (1 + p.G) + 255) / 256);
    return g;
}

template <bool VEC>
__device__ __forceinline__ uint32_t lazy_col(uint32_t seg, int q) {
    return seg * kLazyCols + (VEC ? 4 * threadIdx.x + q : threadIdx.x + 256 * q);
}

// Flat id of edge i of the start's and the goals' edges.
__device__ __forceinline__ uint64_t lazy_outer_edge(const LazyArgs &A, uint64_t i) {
    return i < (uint64_t)A.N ? i : i + (uint64_t)(A.M - 1) * A.N * A.N;
}

// Optimistic costs: the length for edges with free endpoints (status
// unknown), the failed cost for the others.  D: coordinates taken (4 or 8;
// those past d are zero in both vertices and add nothing).  M 8, N 2048, d 7:
// 85 us an edge a thread, 33 like this.
template <int D, bool VEC>
__global__ void __launch_bounds__(256) k_lazy_init(LazyArgs A, LazyGrid B) {
    const uint32_t N = (uint32_t)A.N;
    if (blockIdx.x >= B.inner) {
        const uint64_t i = (uint64_t)(blockIdx.x - B.inner) * 256 + threadIdx.x;
        if (i >= (uint64_t)N * (1 + A.G)) return;
        const uint64_t e = lazy_outer_edge(A, i);
        uint32_t u, v;
        float *c;
        lazy_vertex_ids(A, e, u, v, c);
        float a[GTMP_MAX_DOF], b[GTMP_MAX_DOF];
        for (int k = 0; k < GTMP_MAX_DOF; ++k) {
            a[k] = A.verts[(size_t)u * GTMP_MAX_DOF + k];
            b[k] = A.verts[(size_t)v * GTMP_MAX_DOF + k];
        }
        const float len = edge_len<GTMP_MAX_DOF>(a, b, A.d);
        const bool failed = (A.vflag[u] | A.vflag[v]) != 0 || len > A.max_len;
        *c = failed ? failed_cost(len, A.penalty) : len;
        A.flags[e] = failed ? 1 : kUnknown;
        return;
    }
    __shared__ float src_x[kLazyRows][D];
    __shared__ uint32_t src_f[kLazyRows];
    const uint32_t seg = blockIdx.x % B.segs, row0 = blockIdx.x / B.segs * kLazyRows;
    const uint32_t rows = (uint32_t)(A.M - 1) * N;  // row r: source vertex 1 + r
    const int nr = (int)(rows - row0 < kLazyRows ? rows - row0 : kLazyRows);
    if ((int)threadIdx.x < nr * D) {
        const int r = threadIdx.x / D, k = threadIdx.x % D;
        src_x[r][k] = A.verts[(size_t)(1 + row0 + r) * GTMP_MAX_DOF + k];
        if (k == 0) src_f[r] = A.vflag[1 + row0 + r];
    }
    uint32_t m = row0 / N;
    float v[4][D];
    uint32_t vf[4];
    auto targets = [&]() {
#pragma unroll
        for (int q = 0; q < 4; ++q) {
            const uint32_t c = lazy_col<VEC>(seg, q);
            const uint32_t id = 1 + (m + 1) * N + (c < N ? c : N - 1);
            const float4 *p = reinterpret_cast<const float4 *>(A.verts + (size_t)id * GTMP_MAX_DOF);
#pragma unroll
            for (int h = 0; h < D / 4; ++h) {
                const float4 x = p[h];
                v[q][4 * h] = x.x; v[q][4 * h + 1] = x.y; v[q][4 * h + 2] = x.z; v[q][4 * h + 3] = x.w;
            }
            vf[q] = A.vflag[id];
        }
    };
    targets();
    __syncthreads();
    for (int r = 0; r < nr; ++r) {
        const uint32_t row = row0 + r;
        if (row >= (m + 1) * N) {
            ++m;
            targets();
        }
        float u[D], cost[4];
#pragma unroll
        for (int k = 0; k < D; ++k) u[k] = src_x[r][k];
        const uint32_t uf = src_f[r];
        uint32_t st[4];
#pragma unroll
        for (int q = 0; q < 4; ++q) {
            const float len = edge_len<D>(u, v[q], A.d);
            const bool failed = (uf | vf[q]) != 0 || len > A.max_len;
            cost[q] = failed ? failed_cost(len, A.penalty) : len;
            st[q] = failed ? 1u : (uint32_t)kUnknown;
        }
        const size_t base = (size_t)row * N;
        if constexpr (VEC) {
            const uint32_t c = lazy_col<true>(seg, 0);
            if (c < N) {
                *reinterpret_cast<float4 *>(A.C_h + base + c) = make_float4(cost[0], cost[1], cost[2], cost[3]);
                *reinterpret_cast<uint32_t *>(A.flags + N + base + c) = st[0] | st[1] << 8 | st[2] << 16 | st[3] << 24;
            }
        } else {
#pragma unroll
            for (int q = 0; q < 4; ++q) {
                const uint32_t c = lazy_col<false>(seg, q);
                if (c < N) {
                    A.C_h[base + c] = cost[q];
                    A.flags[N + base + c] = (uint8_t)st[q];
                }
            }
        }
    }
}

// Cost from the start: F[0][v] = C_s[v]; F[m+1][v] = min_u F[m][u] + C_h[m][u][v].
// A block takes kFwdCols columns by kFwdChunk sources, a wave a quarter of the
// sources and (VEC) four neighbouring columns a lane, sixteen 16-byte loads in
// flight; the waves' minima meet in LDS and one integer atomic minimum per
// column folds them into F: costs are non-negative, and the IEEE order of
// non-negative floats is the unsigned order of their bit patterns (the minimum
// is exact in any order).  One column a thread walking 64 sources took 27 us a
// layer of N 2048 (16.8 MB), this 5.1.
constexpr int kFwdChunk = 64, kFwdCols = 256;

template <bool VEC>
__global__ void __launch_bounds__(256) k_lazy_forward(LazyArgs A, int m, float *F) {
    __shared__ float part[256 / kWave][kFwdCols];
    const int lane = lane_id(), w = (int)wave_in_block(), N = A.N;
    constexpr int kPer = kFwdChunk / (256 / kWave);  // sources per wave
    const int c0 = blockIdx.x * kFwdCols, u0 = blockIdx.y * kFwdChunk + w * kPer;
    const float *Fp = F + (size_t)(m - 1) * N;
    const float *C = A.C_h + (size_t)(m - 1) * N * N;
    float best[4];
#pragma unroll
    for (int q = 0; q < 4; ++q) best[q] = __builtin_inff();
    if constexpr (VEC) {
        const int c = c0 + 4 * lane;
        const int cc = c < N ? c : N - 4;  // N is a multiple of four
        float4 x[kPer];
        float f[kPer];
#pragma unroll
        for (int k = 0; k < kPer; ++k) {
            const int u = u0 + k < N ? u0 + k : N - 1;  // past the end, the last source again
            x[k] = *reinterpret_cast<const float4 *>(C + (size_t)u * N + cc);
            f[k] = Fp[u];
        }
#pragma unroll
        for (int k = 0; k < kPer; ++k) {
            best[0] = __builtin_fminf(best[0], f[k] + x[k].x);
            best[1] = __builtin_fminf(best[1], f[k] + x[k].y);
            best[2] = __builtin_fminf(best[2], f[k] + x[k].z);
            best[3] = __builtin_fminf(best[3], f[k] + x[k].w);
        }
    } else {
        for (int k = 0; k < kPer && u0 + k < N; ++k) {
            const float f = Fp[u0 + k];
#pragma unroll
            for (int q = 0; q < 4; ++q) {
                const int c = c0 + lane + kWave * q;
                best[q] = __builtin_fminf(best[q], f + C[(size_t)(u0 + k) * N + (c < N ? c : N - 1)]);
            }
        }
    }
#pragma unroll
    for (int q = 0; q < 4; ++q) part[w][VEC ? 4 * lane + q : lane + kWave * q] = best[q];
    __syncthreads();
    const int c = c0 + (int)threadIdx.x;
    if (c < N) {
        float b = part[0][threadIdx.x];
#pragma unroll
        for (int k = 1; k < 256 / kWave; ++k) b = __builtin_fminf(b, part[k][threadIdx.x]);
        atomicMin(reinterpret_cast<unsigned int *>(F + (size_t)m * N + c), __float_as_uint(b));
    }
}

// Done test (block 0): the extracted path idx[0..M] (vertex per layer, then
// the goal) has no unknown edge.  With no path (idx[0] < 0) the loop is done
// as well.  The other blocks prepare the next round's forward sweep (F: the
// start's costs, +inf past the first layer), which is not enqueued if done.
__global__ void __launch_bounds__(256) k_lazy_done(LazyArgs A, const int32_t *idx, float *F) {
    if (blockIdx.x != 0) {
        const size_t i = (size_t)(blockIdx.x - 1) * 256 + threadIdx.x;
        if (i < (size_t)A.M * A.N) F[i] = i < (size_t)A.N ? A.C_s[i] : __builtin_inff();
        return;
    }
    if (threadIdx.x != 0) return;
    uint32_t unknown = 0;
    if (idx[0] >= 0) {
        const uint64_t N = A.N;
        unknown += A.flags[idx[0]] == kUnknown;
        for (int m = 0; m + 1 < A.M; ++m) {
            const uint64_t e = N + (uint64_t)m * N * N + (uint64_t)idx[m] * N + idx[m + 1];
            unknown += A.flags[e] == kUnknown;
        }
        const uint64_t e = N + (uint64_t)(A.M - 1) * N * N + (uint64_t)idx[A.M - 1] * A.G + idx[A.M];
        unknown += A.flags[e] == kUnknown;
    }
    A.counters[0] = unknown == 0 ? 1u : 0u;
    A.counters[1] = 0;
    A.counters[2] = unknown;
}

// Cost of the best path through edge e (F(u) + C(u, v) + V(v)), the sum in
// this order wherever it is formed.
__device__ __forceinline__ float lazy_through(const LazyArgs &A, uint64_t e) {
    const uint64_t N = A.N, inner = (uint64_t)(A.M - 1) * N * N;
    if (e < N) return A.C_s[e] + A.V[e];
    if (e - N < inner) {
        const uint64_t r = e - N, m = r / (N * N), uv = r - m * N * N;
        return (A.F[m * N + uv / N] + A.C_h[r]) + A.V[(m + 1) * N + uv % N];
    }
    const uint64_t r = e - N - inner, n = r / (uint64_t)A.G;
    return A.F[(uint64_t)(A.M - 1) * N + n] + A.C_l[r];
}

__device__ __forceinline__ float lazy_threshold(const LazyArgs &A, float band) { return (1.0f + band) * *A.V_s; }

// A block's `mine` (edges a thread appends), reserved with one atomic: where
// this thread's edges go.
__device__ __forceinline__ uint32_t lazy_reserve(const LazyArgs &A, uint32_t mine) {
    __shared__ uint32_t part[256 / kWave], base_s;
    const int lane = lane_id(), w = (int)wave_in_block();
    uint32_t incl = mine;
#pragma unroll
    for (int o = 1; o < kWave; o <<= 1) {
        const uint32_t y = lane_read(lane - o, incl);
        if (lane >= o) incl += y;
    }
    if (lane == kWave - 1) part[w] = incl;
    __syncthreads();
    uint32_t before = incl - mine, tot = 0;
#pragma unroll
    for (int k = 0; k < 256 / kWave; ++k) {
        if (k < w) before += part[k];
        tot += part[k];
    }
    if (threadIdx.x == 0) base_s = tot != 0 ? atomicAdd(&A.counters[1], tot) : 0u;
    __syncthreads();
    return base_s + before;
}

// Selection of the round: unknown edges whose best path through them is at
// most thr = (1 + band) V_s, appended to the round's list (its order is
// immaterial to the check) with select[e] = 1, which the check sets to 2 for
// those that collide; select is written and read for listed edges only.
// M 8, N 2048 (29.4 M edges, 25 k selected): 106 us an edge a thread with the
// selection written for every edge and read again, 43 like this.
template <bool VEC>
__global__ void __launch_bounds__(256) k_lazy_select(LazyArgs A, LazyGrid B, float band) {
    const uint32_t N = (uint32_t)A.N;
    const float thr = lazy_threshold(A, band);
    if (blockIdx.x >= B.inner) {
        const uint64_t i = (uint64_t)(blockIdx.x - B.inner) * 256 + threadIdx.x;
        bool sel = false;
        uint64_t e = 0;
        if (i < (uint64_t)N * (1 + A.G)) {
            e = lazy_outer_edge(A, i);
            sel = A.flags[e] == kUnknown && lazy_through(A, e) <= thr;
        }
        const uint32_t at = lazy_reserve(A, sel ? 1u : 0u);
        if (sel) {
            A.list[at] = (uint32_t)e;
            A.select[e] = 1;
        }
        return;
    }
    const uint32_t seg = blockIdx.x % B.segs, row0 = blockIdx.x / B.segs * kLazyRows;
    const uint32_t rows = (uint32_t)(A.M - 1) * N;
    const uint32_t nr = rows - row0 < kLazyRows ? rows - row0 : kLazyRows;
    const uint32_t m0 = row0 / N;
    const uint32_t c0 = lazy_col<VEC>(seg, 0);
    constexpr uint32_t kStep = VEC ? 1 : 256;  // columns c0 + q kStep
    uint32_t unknown = 0;                      // bit 4 r + q
    {
        uint32_t f[kLazyRows];
#pragma unroll
        for (int r = 0; r < kLazyRows; ++r) {
            const uint8_t *p = A.flags + N + (size_t)(row0 + r) * N + c0;
            f[r] = 0;
            if constexpr (VEC) {
                if ((uint32_t)r < nr && c0 < N) f[r] = *reinterpret_cast<const uint32_t *>(p);
            } else {
#pragma unroll
                for (int q = 0; q < 4; ++q)
                    if ((uint32_t)r < nr && c0 + q * kStep < N) f[r] |= (uint32_t)p[q * kStep] << (8 * q);
            }
        }
#pragma unroll
        for (int r = 0; r < kLazyRows; ++r)
#pragma unroll
            for (int q = 0; q < 4; ++q) unknown |= ((f[r] >> (8 * q)) & 0xffu) == kUnknown ? 1u << (4 * r + q) : 0u;
    }
    uint32_t sel = 0;
    if (unknown != 0) {
        float4 x[kLazyRows];
        float f[kLazyRows];
#pragma unroll
        for (int r = 0; r < kLazyRows; ++r) {
            const float *p = A.C_h + (size_t)(row0 + r) * N + c0;
            x[r] = make_float4(0.f, 0.f, 0.f, 0.f);
            f[r] = 0.f;
            const uint32_t u = unknown >> (4 * r) & 15u;
            if (u != 0) {
                f[r] = A.F[row0 + r];
                if constexpr (VEC) {
                    x[r] = *reinterpret_cast<const float4 *>(p);
                } else {
                    if (u & 1u) x[r].x = p[0];
                    if (u & 2u) x[r].y = p[kStep];
                    if (u & 4u) x[r].z = p[2 * kStep];
                    if (u & 8u) x[r].w = p[3 * kStep];
                }
            }
        }
        uint32_t m = m0;
        float4 v;
        auto targets = [&]() {  // V of the targets of layer m's rows
            const float *p = A.V + (size_t)(m + 1) * N;
            const uint32_t last = N - 1;
            v = make_float4(p[c0 < N ? c0 : last], p[c0 + kStep < N ? c0 + kStep : last],
                            p[c0 + 2 * kStep < N ? c0 + 2 * kStep : last], p[c0 + 3 * kStep < N ? c0 + 3 * kStep : last]);
        };
        targets();
#pragma unroll
        for (int r = 0; r < kLazyRows; ++r) {
            if ((uint32_t)r < nr && row0 + r >= (m + 1) * N) {
                ++m;
                targets();
            }
            uint32_t b = 0;
            b |= (f[r] + x[r].x) + v.x <= thr ? 1u : 0u;
            b |= (f[r] + x[r].y) + v.y <= thr ? 2u : 0u;
            b |= (f[r] + x[r].z) + v.z <= thr ? 4u : 0u;
            b |= (f[r] + x[r].w) + v.w <= thr ? 8u : 0u;
            sel |= b << (4 * r);
        }
        sel &= unknown;
    }
    uint32_t at = lazy_reserve(A, (uint32_t)__popc(sel));
    while (sel != 0) {
        const int b = __builtin_ctz(sel);
        sel &= sel - 1;
        const uint64_t e = (uint64_t)N + (uint64_t)(row0 + (b >> 2)) * N + c0 + kStep * (b & 3);
        A.list[at++] = (uint32_t)e;
        A.select[e] = 1;
    }
}

// The unchecked edges of the extracted path always join the round's
// selection (their through-cost equals V_s only up to the rounding of a
// different summation order), so every round checks at least one edge.
__global__ void k_lazy_mark_path(LazyArgs A, const int32_t *idx, float band) {
    if (idx[0] < 0) return;
    const uint64_t N = A.N;
    const float thr = lazy_threshold(A, band);
    for (int k = threadIdx.x; k <= A.M; k += blockDim.x) {  // edge k of the path
        const uint64_t e = k == 0     ? (uint64_t)idx[0]
                           : k < A.M ? N + (uint64_t)(k - 1) * N * N + (uint64_t)idx[k - 1] * N + idx[k]
                                     : N + (uint64_t)(A.M - 1) * N * N + (uint64_t)idx[A.M - 1] * A.G + idx[A.M];
        if (A.flags[e] == kUnknown && !(lazy_through(A, e) <= thr)) {  // not selected already
            A.select[e] = 1;
            A.list[atomicAdd(&A.counters[1], 1u)] = (uint32_t)e;
        }
    }
}

__global__ void k_lazy_count(LazyArgs A) {
    if (threadIdx.x != 0) return;
    A.stats[0] += 1;
    A.stats[1] += A.counters[1];
}

// ------------------------------------------------------------------ host side
static size_t up256_l(size_t x) { return (x + 255) & ~size_t(255); }

LazyPlan make_lazy_plan(const gtmp_problem &p) {
    LazyPlan L{};
    const uint64_t N = p.N, M = p.M, G = p.G;
    const uint64_t E = N + (M - 1) * N * N + N * G;
    const EdgePlan ep = make_edge_plan(p);
    size_t off = 0;
    L.off_edge = off; off = up256_l(off + ep.total);
    L.off_F = off; off = up256_l(off + sizeof(float) * M * N);
    L.off_select = off; off = up256_l(off + E);
    L.off_list = off; off = up256_l(off + sizeof(uint32_t) * E);
    L.off_counters = off; off = up256_l(off + 256);
    L.total = off;
    return L;
}

hipError_t launch_plan_lazy(const gtmp_problem &p, const ArmParams *arm, const SceneParams &S, int wdim,
                            const float *q0, const float *goals, const float *Q, float *C_s, float *C_h, float *C_l,
                            uint8_t *flags, float *V, int32_t *Am, float *V_s, int32_t *a_s, int32_t *idx, float *wp,
                            float *cost, float band, int max_rounds, unsigned long long *stats,
                            const gtmp_edge_opts &eo, void *workspace, int *rounds_host, bool *done_host,
                            hipStream_t s) {
    const LazyPlan plan = make_lazy_plan(p);
    const EdgePlan ep = make_edge_plan(p);
    char *ws = static_cast<char *>(workspace);
    EdgeBuffers b{q0, goals, Q, C_s, C_h, C_l, nullptr, flags, nullptr, ws + plan.off_edge};
    LazyArgs A{};
    A.d = p.d; A.M = p.M; A.N = p.N; A.G = p.G;
    A.penalty = p.penalty; A.max_len = p.max_edge_len;
    A.verts = reinterpret_cast<const float *>(ws + plan.off_edge + ep.off_verts);
    A.vflag = reinterpret_cast<const uint8_t *>(ws + plan.off_edge + ep.off_vflag);
    A.C_s = C_s; A.C_h = C_h; A.C_l = C_l; A.flags = flags;
    A.V = V;
    float *F = reinterpret_cast<float *>(ws + plan.off_F);
    A.F = F;
    A.V_s = V_s;
    A.select = reinterpret_cast<uint8_t *>(ws + plan.off_select);
    A.list = reinterpret_cast<uint32_t *>(ws + plan.off_list);
    A.counters = reinterpret_cast<uint32_t *>(ws + plan.off_counters);
    A.stats = stats;
    gtmp_edge_opts o = eo;
    o.mode = GTMP_CHECK_FAST;
    o.ev_begin = o.ev_end = nullptr;
    hipError_t e = launch_edge_phases(ep, arm, S, wdim, b, o, s, nullptr, nullptr, nullptr, kPhaseVertices);
    if (e != hipSuccess) return e;
    const LazyGrid B = lazy_grid(p);
    const dim3 blocks(B.inner + B.edge_blocks);
    const bool vec = p.N % 4 == 0 && ((uintptr_t)C_h & 15) == 0 && ((uintptr_t)flags & 3) == 0;
    const auto init = p.d <= 4 ? (vec ? k_lazy_init<4, true> : k_lazy_init<4, false>)
                               : (vec ? k_lazy_init<8, true> : k_lazy_init<8, false>);
    hipLaunchKernelGGL(init, blocks, dim3(256), 0, s, A, B);
    uint32_t done = 0;
    int r = 0;
    for (;;) {
        e = launch_minplus(p.M, p.N, p.G, C_s, C_h, C_l, nullptr, V, Am, V_s, a_s, s);
        if (e != hipSuccess) return e;
        e = launch_extract(p.M, p.N, p.G, p.d, a_s, Am, V_s, Q, q0, goals, idx, wp, cost, s);
        if (e != hipSuccess) return e;
        const size_t MN = (size_t)p.M * p.N;
        hipLaunchKernelGGL(k_lazy_done, dim3(1 + (unsigned)((MN + 255) / 256)), dim3(256), 0, s, A, idx, F);
        e = hipMemcpyAsync(&done, A.counters, sizeof(uint32_t), hipMemcpyDeviceToHost, s);
        if (e != hipSuccess) return e;
        e = hipStreamSynchronize(s);
        if (e != hipSuccess) return e;
        if (done || r >= max_rounds) break;
        const dim3 fb((unsigned)((p.N + kFwdCols - 1) / kFwdCols), (unsigned)((p.N + kFwdChunk - 1) / kFwdChunk));
        for (int m = 1; m < p.M; ++m)
            hipLaunchKernelGGL(vec ? k_lazy_forward<true> : k_lazy_forward<false>, fb, dim3(256), 0, s, A, m, F);
        hipLaunchKernelGGL(vec ? k_lazy_select<true> : k_lazy_select<false>, blocks, dim3(256), 0, s, A, B, band);
        hipLaunchKernelGGL(k_lazy_mark_path, dim3(1), dim3(64), 0, s, A, idx, band);
        e = launch_edge_phases(ep, arm, S, wdim, b, o, s, A.list, A.counters + 1, A.select, kPhaseEdges);
        if (e != hipSuccess) return e;
        if (stats) hipLaunchKernelGGL(k_lazy_count, dim3(1), dim3(64), 0, s, A);
        ++r;
    }
    *rounds_host = r;
    *done_host = done != 0;
    return hipGetLastError();
}

}  // namespace gtmp
