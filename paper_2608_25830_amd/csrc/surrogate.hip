// surrogate.hip -- the learned collision surrogate: a ReLU MLP on Fourier
// features of the configuration, with BF16 weights and activations and FP32
// accumulation on the matrix cores (v_mfma_f32_32x32x16_bf16), its BCE loss,
// backward pass and Adam update, and its two uses: edge pruning at the
// midpoint probe and scoring of heuristic sample candidates.
//
// Every reduction runs in a fixed order (split-K partials summed in split
// order, column sums over fixed row chunks, wave reductions by butterfly), so
// results are reproducible run to run.
#include <algorithm>

#include "surrogate.hpp"

namespace gtmp {

// ------------------------------------------------------------------ layout
SurLayout sur_layout() {
    SurLayout L{};
    int o = 0;
    const int W = GTMP_SUR_WIDTH, I = GTMP_SUR_IN;
    L.W[0] = o; o += W * I;
    L.b[0] = o; o += W;
    for (int l = 1; l < 4; ++l) {
        L.W[l] = o; o += W * W;
        L.b[l] = o; o += W;
    }
    L.w5 = o; o += W;
    L.b5 = o; o += 1;
    L.total = o;
    return L;
}

// ------------------------------------------------------------------ BF16
__device__ __forceinline__ uint16_t f2bf(float f) {
    // round to nearest, ties to even (finite inputs)
    uint32_t u = __float_as_uint(f);
    u += 0x7FFFu + ((u >> 16) & 1u);
    return (uint16_t)(u >> 16);
}
__device__ __forceinline__ float bf2f(uint16_t h) { return __uint_as_float((uint32_t)h << 16); }

typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef float f32x16 __attribute__((ext_vector_type(16)));

// ------------------------------------------------------------------ features
// Round a double to the nearest BF16 value, ties to even, in one step (no
// intermediate FP32 rounding): keep 7 of the 52 mantissa bits.  Finite
// inputs inside the FP32 normal range or zero.
__device__ __forceinline__ uint16_t d2bf(double x) {
    uint64_t u = (uint64_t)__double_as_longlong(x);
    const uint64_t drop = 45;  // 52 - 7 mantissa bits
    u += ((1ull << (drop - 1)) - 1) + ((u >> drop) & 1ull);
    u &= ~((1ull << drop) - 1);
    return (uint16_t)(__float_as_uint((float)__longlong_as_double((long long)u)) >> 16);
}

// ------------------------------------------------------------------ fused inference
// Whole network for 128 rows per block tile (inference only): features
// computed in FP64 straight into LDS, then four hidden layers whose BF16
// activations stay in LDS (one 128 x 256 tile, written back in place after a
// barrier), then the FP32 head.  Wave w owns output columns [64 w, 64 w + 64)
// of every layer: 4 x 2 tiles of 32 x 32 (v_mfma_f32_32x32x16_bf16, 128
// accumulators per lane); activation fragments come from LDS, weight
// fragments from a copy of the weights stored in fragment order (for every
// 32-column tile and 16-wide K slice, the 64 lanes' 16-byte operands side by
// side), so each weight load of a wave is one contiguous 1 KB read from L2.
// Two blocks share a CU (2 x 68 KB of LDS), so one block's feature or
// epilogue phase overlaps the other's MFMAs.  Sums run in K order.
constexpr int kFR = 128;                              // rows per block tile
constexpr int kFRow = GTMP_SUR_WIDTH + 8;             // LDS row stride (BF16), 528 bytes
constexpr int kColTiles = GTMP_SUR_WIDTH / 32;        // 32-column output tiles per layer

// Offsets (in 16-byte fragments) of the layers in the fragment-order copy.
__host__ __device__ constexpr int frag_offset(int l) {
    return l == 0 ? 0 : kColTiles * (GTMP_SUR_IN / 16) * 64 + (l - 1) * kColTiles * (GTMP_SUR_WIDTH / 16) * 64;
}
constexpr int kFragTotal = frag_offset(4);  // 16-byte fragments of the four hidden layers

// Feature order of the fused kernels' LDS rows: each of a row's two
// threads writes one half with four 16-byte stores, thread 0 [sin f0..7 |
// cos f0..7 | q/pi (8, zero past d) | 0 x 8], thread 1 [sin f8..15 |
// cos f8..15 | 0 x 16].  feature_at maps an LDS position to the input of the
// standard order [q/pi (d) | sin (16) | cos (16) | 0...], -1 for a zero; the
// first layer's weight fragments are stored in the LDS order, so the sums
// are over the same products.
__host__ __device__ inline int feature_at(int p, int d) {
    if (p < 8) return d + p;
    if (p < 16) return d + GTMP_SUR_FREQ + (p - 8);
    if (p < 24) return p - 16 < d ? p - 16 : -1;
    if (p < 32) return -1;
    if (p < 40) return d + 8 + (p - 32);
    if (p < 48) return d + GTMP_SUR_FREQ + 8 + (p - 40);
    return -1;
}

__device__ __forceinline__ uint32_t pack2(uint16_t lo, uint16_t hi) { return (uint32_t)lo | ((uint32_t)hi << 16); }

// Thread `half` of a row: sn, cs = its 8 frequencies' sines and cosines, qh
// (half 0) the d linear features; BF16-rounded and stored in the LDS order.
__device__ __forceinline__ void store_features(int d, int half, const double (&sn)[8], const double (&cs)[8],
                                               const double (&qh)[GTMP_MAX_DOF], uint16_t *row) {
    uint16_t v[32];
#pragma unroll
    for (int q = 0; q < 8; ++q) {
        v[q] = d2bf(sn[q]);
        v[8 + q] = d2bf(cs[q]);
        v[16 + q] = (half == 0 && q < d) ? d2bf(qh[q]) : (uint16_t)0;
        v[24 + q] = 0;
    }
    uint4 *dst = reinterpret_cast<uint4 *>(row + 32 * half);
#pragma unroll
    for (int c = 0; c < 4; ++c)
        dst[c] = make_uint4(pack2(v[8 * c], v[8 * c + 1]), pack2(v[8 * c + 2], v[8 * c + 3]),
                            pack2(v[8 * c + 4], v[8 * c + 5]), pack2(v[8 * c + 6], v[8 * c + 7]));
}

// Fragment f of layer l: lane = f % 64, K slice ks and column tile c from
// f / 64 = c * S + ks; it holds W_l[32 c + lane % 32][16 ks + 8 (lane / 32) ..+8].
// (Layer 1's columns in the LDS feature order of feature_at.)
__global__ void __launch_bounds__(256) k_weight_frag(int d, const uint16_t *__restrict__ P16, SurLayout L,
                                                     uint4 *__restrict__ Wf) {
    const int f = blockIdx.x * blockDim.x + threadIdx.x;
    if (f >= kFragTotal) return;
    const int l = f < frag_offset(1) ? 0 : 1 + (f - frag_offset(1)) / (frag_offset(2) - frag_offset(1));
    const int K = l == 0 ? GTMP_SUR_IN : GTMP_SUR_WIDTH;
    const int S = K / 16;
    const int r = f - frag_offset(l);
    const int lane = r & 63, ks = (r >> 6) % S, c = (r >> 6) / S;
    const int row = 32 * c + (lane & 31), col = 16 * ks + 8 * (lane >> 5);
    const uint16_t *src = P16 + L.W[l] + (size_t)row * K;
    if (l > 0) {
        Wf[f] = *reinterpret_cast<const uint4 *>(src + col);
        return;
    }
    uint16_t w[8];
#pragma unroll
    for (int k = 0; k < 8; ++k) {
        const int j = feature_at(col + k, d);
        w[k] = j < 0 ? (uint16_t)0 : src[j];
    }
    Wf[f] = make_uint4(pack2(w[0], w[1]), pack2(w[2], w[3]), pack2(w[4], w[5]), pack2(w[6], w[7]));
}

// One hidden layer on the block's LDS tile: K input columns -> 256 outputs,
// bias + ReLU, BF16, written back in place.  The MFMA computes the transposed
// product (weights as the A operand, activations as B), so each lane's
// accumulators hold four consecutive output columns of one row: they are
// converted with one packed instruction per pair and stored with one 8-byte
// LDS write.  Weight fragments are requested one K slice ahead.
typedef __bf16 bf16x4 __attribute__((ext_vector_type(4)));
typedef float f32x4v __attribute__((ext_vector_type(4)));

template <int K>
__device__ __forceinline__ void mlp_layer(const bf16x8 *__restrict__ Wf, const float *__restrict__ bias,
                                          uint16_t *act, int wave, int lane) {
    constexpr int S = K / 16;
    const int cl = lane & 31, kh = 8 * (lane >> 5);
    const int c0 = wave * 64;
    f32x16 acc[4][2];  // [row tile i][column tile j]
#pragma unroll
    for (int i = 0; i < 4; ++i)
#pragma unroll
        for (int j = 0; j < 2; ++j)
#pragma unroll
            for (int v = 0; v < 16; ++v) acc[i][j][v] = 0.f;
    const bf16x8 *wr0 = Wf + (size_t)(2 * wave) * S * 64 + lane;
    const bf16x8 *wr1 = Wf + (size_t)(2 * wave + 1) * S * 64 + lane;
    // weight fragments requested kWPre K slices ahead (an L2 round trip is
    // longer than one slice of MFMAs); the next slice's four activation
    // fragments are read from LDS while the current slice's MFMAs run
    constexpr int kWPre = 3;
    bf16x8 w0[S], w1[S];
#pragma unroll
    for (int k = 0; k < kWPre && k < S; ++k) {
        w0[k] = wr0[64 * k];
        w1[k] = wr1[64 * k];
    }
    auto act_frag = [&](int i, int ks) {
        return *reinterpret_cast<const bf16x8 *>(&act[(32 * i + cl) * kFRow + 16 * ks + kh]);
    };
    bf16x8 a_cur[4];
#pragma unroll
    for (int i = 0; i < 4; ++i) a_cur[i] = act_frag(i, 0);
#pragma unroll
    for (int ks = 0; ks < S; ++ks) {
        if (ks + kWPre < S) {
            w0[ks + kWPre] = wr0[64 * (ks + kWPre)];
            w1[ks + kWPre] = wr1[64 * (ks + kWPre)];
        }
        bf16x8 a_nxt[4];
        if (ks + 1 < S) {
#pragma unroll
            for (int i = 0; i < 4; ++i) a_nxt[i] = act_frag(i, ks + 1);
        }
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            acc[i][0] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(w0[ks], a_cur[i], acc[i][0], 0, 0, 0);
            acc[i][1] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(w1[ks], a_cur[i], acc[i][1], 0, 0, 0);
        }
        if (ks + 1 < S) {
#pragma unroll
            for (int i = 0; i < 4; ++i) a_cur[i] = a_nxt[i];
        }
    }
    // element v of tile (i, j): output column c0 + 32 j + 8 (v/4) + 4 (lane/32) + v%4, row 32 i + lane%32
    f32x4v bq[2][4];
#pragma unroll
    for (int j = 0; j < 2; ++j)
#pragma unroll
        for (int g = 0; g < 4; ++g)
            bq[j][g] = *reinterpret_cast<const f32x4v *>(bias + c0 + 32 * j + 8 * g + 4 * (lane >> 5));
    __syncthreads();  // every wave has read this layer's input
#pragma unroll
    for (int i = 0; i < 4; ++i)
#pragma unroll
        for (int j = 0; j < 2; ++j)
#pragma unroll
            for (int g = 0; g < 4; ++g) {
                f32x4v z;
#pragma unroll
                for (int r = 0; r < 4; ++r) {
                    const float t = acc[i][j][4 * g + r] + bq[j][g][r];
                    z[r] = t > 0.f ? t : 0.f;
                }
                const bf16x4 o = __builtin_convertvector(z, bf16x4);
                const int col = c0 + 32 * j + 8 * g + 4 * (lane >> 5);
                *reinterpret_cast<bf16x4 *>(&act[(32 * i + cl) * kFRow + col]) = o;
            }
    __syncthreads();
}

// Features of one row into its LDS slot; two threads per row (half 0 and 1),
// each taking half of the frequencies.  qh = q / pi in FP64.
__device__ __forceinline__ void row_features(int d, const double (&qh)[GTMP_MAX_DOF], int half,
                                             const float *__restrict__ Bf, uint16_t *dst) {
    constexpr double kPi = 3.14159265358979323846;
    double sn[8], cs[8];
#pragma unroll
    for (int q = 0; q < 8; ++q) {
        const int f = half * (GTMP_SUR_FREQ / 2) + q;
        double sarg = 0.0;
        for (int j = 0; j < d; ++j) sarg += (double)Bf[f * d + j] * qh[j];
        sarg *= 2.0 * kPi;
        sincos(sarg, &sn[q], &cs[q]);
    }
    store_features(d, half, sn, cs, qh, dst);
}

// The four hidden layers and the FP32 head of the block's tile; thread
// tid < kFR gets its row's logit.  Head: two threads per row, each summing
// one half of the 256 products in K order (8 activations per LDS read);
// z = first half + second half + b5.
__device__ __forceinline__ float mlp_tile(const bf16x8 *__restrict__ Wf, const float *__restrict__ P32,
                                          const SurLayout &L, uint16_t *act, const float *w5s, float *zpart,
                                          int tid) {
    const int lane = tid & 63, wave = tid >> 6;
    mlp_layer<GTMP_SUR_IN>(Wf + frag_offset(0), P32 + L.b[0], act, wave, lane);
    mlp_layer<GTMP_SUR_WIDTH>(Wf + frag_offset(1), P32 + L.b[1], act, wave, lane);
    mlp_layer<GTMP_SUR_WIDTH>(Wf + frag_offset(2), P32 + L.b[2], act, wave, lane);
    mlp_layer<GTMP_SUR_WIDTH>(Wf + frag_offset(3), P32 + L.b[3], act, wave, lane);
    const int r = tid & (kFR - 1), half = tid >> 7;
    constexpr int kHalf = GTMP_SUR_WIDTH / 2;
    const uint4 *a = reinterpret_cast<const uint4 *>(act + r * kFRow + half * kHalf);
    const float *w = w5s + half * kHalf;
    float z = 0.f;
#pragma unroll 4
    for (int q = 0; q < kHalf / 8; ++q) {
        const uint4 v = a[q];
        const uint32_t wd[4] = {v.x, v.y, v.z, v.w};
#pragma unroll
        for (int h = 0; h < 4; ++h) {
            z = __builtin_fmaf(w[8 * q + 2 * h], __uint_as_float(wd[h] << 16), z);
            z = __builtin_fmaf(w[8 * q + 2 * h + 1], __uint_as_float(wd[h] & 0xffff0000u), z);
        }
    }
    if (half == 1) zpart[r] = z;
    __syncthreads();
    return half == 0 ? z + zpart[r] + P32[L.b5] : 0.f;
}

__global__ void __launch_bounds__(256, 2) k_mlp_infer(int d, int64_t n, const float *__restrict__ X,
                                                     const float *__restrict__ Bf, const bf16x8 *__restrict__ Wf,
                                                     const uint16_t *__restrict__ P16,
                                                     const float *__restrict__ P32, SurLayout L,
                                                     float *__restrict__ logits) {
    __shared__ __attribute__((aligned(16))) uint16_t act[kFR * kFRow];
    __shared__ float w5s[GTMP_SUR_WIDTH];
    __shared__ float zpart[kFR];
    const int tid = threadIdx.x;
    const int64_t row0 = (int64_t)blockIdx.x * kFR;
    {
        const int r = tid & (kFR - 1), half = tid >> 7;
        const int64_t gr = row0 + r;
        constexpr double kPi = 3.14159265358979323846;
        double qh[GTMP_MAX_DOF];
        for (int j = 0; j < GTMP_MAX_DOF; ++j) qh[j] = (gr < n && j < d) ? (double)X[gr * d + j] / kPi : 0.0;
        row_features(d, qh, half, Bf, act + r * kFRow);
        if (tid < GTMP_SUR_WIDTH) w5s[tid] = bf2f(P16[L.w5 + tid]);
    }
    __syncthreads();
    const float z = mlp_tile(Wf, P32, L, act, w5s, zpart, tid);
    if (tid < kFR && row0 + tid < n) logits[row0 + tid] = z;
}

// ------------------------------------------------------------------ pruning
// Candidate edges: those whose two endpoints are free samples (an edge with
// a colliding endpoint fails the exact check at its vertex, so it is never
// inferred).  Per layer m the free samples in index order fl[m][0 .. nf[m]);
// candidate t lies in segment s with seg[s] <= t < seg[s + 1]: s = 0 start
// edges (q0 -> free layer-0 samples), s = 1 .. M-1 the free pairs of layers
// s-1 and s (row-major over the two free lists), s = M the edges from free
// layer M-1 samples to every goal.
__global__ void __launch_bounds__(256) k_free_lists(int N, const uint8_t *__restrict__ vcoll,
                                                    int32_t *__restrict__ fl, int32_t *__restrict__ nf) {
    __shared__ int wsum[256 / kWave];
    const int m = blockIdx.x, tid = threadIdx.x, lane = tid & 63, wv = tid >> 6;
    int count = 0;
    for (int base = 0; base < N; base += 256) {
        const int i = base + tid;
        const bool fr = i < N && (vcoll == nullptr || vcoll[(size_t)m * N + i] == 0);
        const uint64_t bal = __ballot(fr);
        if (lane == 0) wsum[wv] = __popcll(bal);
        __syncthreads();
        int before = count;
        for (int w = 0; w < wv; ++w) before += wsum[w];
        if (fr) fl[(size_t)m * N + before + __popcll(bal & ((1ull << lane) - 1ull))] = i;
        for (int w = 0; w < 256 / kWave; ++w) count += wsum[w];
        __syncthreads();
    }
    if (tid == 0) nf[m] = count;
}

// Phase table of the probe features.  The midpoint of u and v is
// (u + v) / 2 exactly (FP64), so its phases are 2 pi B (u + v) / (2 pi) =
// a(u) + a(v) with a(x) = pi sum_j B_fj (x_j / pi), and its sines and
// cosines follow from the endpoints' by angle addition.  Row of a sample
// (kPhaseRow doubles): sin a_f (16), cos a_f (16), x_j / pi (8, zero past d).
// Rows: the free samples in free-list order ([M][N] slots), then q0, then
// the goals.
constexpr int kPhaseRow = 2 * GTMP_SUR_FREQ + GTMP_MAX_DOF;

__global__ void __launch_bounds__(256) k_sample_phases(int d, int M, int N, int G, const float *__restrict__ Q,
                                                       const float *__restrict__ q0, const float *__restrict__ goals,
                                                       const int32_t *__restrict__ fl, const int32_t *__restrict__ nf,
                                                       const float *__restrict__ Bf, double *__restrict__ T) {
    const int64_t t = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    const int64_t MN = (int64_t)M * N;
    if (t >= MN + 1 + G) return;
    const float *x;
    if (t < MN) {
        const int m = (int)(t / N), i = (int)(t - (int64_t)m * N);
        if (i >= nf[m]) return;
        x = Q + ((size_t)m * N + fl[t]) * d;
    } else if (t == MN) {
        x = q0;
    } else {
        x = goals + (size_t)(t - MN - 1) * d;
    }
    constexpr double kPi = 3.14159265358979323846;
    double qh[GTMP_MAX_DOF];
    for (int j = 0; j < GTMP_MAX_DOF; ++j) qh[j] = j < d ? (double)x[j] / kPi : 0.0;
    double *row = T + (size_t)t * kPhaseRow;
    for (int f = 0; f < GTMP_SUR_FREQ; ++f) {
        double a = 0.0;
        for (int j = 0; j < d; ++j) a += (double)Bf[f * d + j] * qh[j];
        a *= kPi;
        double sn, cs;
        sincos(a, &sn, &cs);
        row[f] = sn;
        row[GTMP_SUR_FREQ + f] = cs;
    }
    for (int j = 0; j < GTMP_MAX_DOF; ++j) row[2 * GTMP_SUR_FREQ + j] = qh[j];
}

__global__ void k_cand_segments(int M, int G, const int32_t *__restrict__ nf, int64_t *__restrict__ seg) {
    if (threadIdx.x != 0 || blockIdx.x != 0) return;
    int64_t o = 0;
    seg[0] = 0;
    o += nf[0];
    seg[1] = o;
    for (int s = 1; s < M; ++s) {
        o += (int64_t)nf[s - 1] * nf[s];
        seg[s + 1] = o;
    }
    o += (int64_t)nf[M - 1] * G;
    seg[M + 1] = o;
}

__global__ void k_prune_fill(int64_t E, uint8_t *__restrict__ prune, float *__restrict__ logits) {
    const int64_t stride = (int64_t)gridDim.x * blockDim.x;
    for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < E; i += stride) {
        prune[i] = 0;
        if (logits) logits[i] = __builtin_nanf("");
    }
}

// Endpoints of candidate t (t < total): their rows in the phase table and
// the edge's flat id.  Segment bounds and list lengths come from LDS.
template <typename IDX>
__device__ __forceinline__ void cand_rows(int64_t t, int M, int N, int G, const int64_t *seg, const int32_t *nf,
                                          const int32_t *__restrict__ fl, int64_t &ru, int64_t &rv, int64_t &e) {
    int lo = 0, hi = M;  // largest s in [0, M] with seg[s] <= t
    while (lo < hi) {
        const int mid = (lo + hi + 1) >> 1;
        if (seg[mid] <= t) lo = mid;
        else hi = mid - 1;
    }
    const IDX loc = (IDX)(t - seg[lo]);
    const int64_t MN = (int64_t)M * N;
    if (lo == 0) {
        ru = MN;
        rv = (int64_t)loc;
        e = fl[loc];
    } else if (lo < M) {
        const int m = lo - 1;
        const IDX n1 = (IDX)nf[m + 1];
        const IDX i = loc / n1, j = loc - i * n1;
        ru = (int64_t)m * N + (int64_t)i;
        rv = (int64_t)(m + 1) * N + (int64_t)j;
        e = N + (int64_t)m * N * N + (int64_t)fl[ru] * N + fl[rv];
    } else {
        const IDX i = loc / (IDX)G, g = loc - i * (IDX)G;
        ru = (int64_t)(M - 1) * N + (int64_t)i;
        rv = MN + 1 + (int64_t)g;
        e = N + (int64_t)(M - 1) * N * N + (int64_t)fl[ru] * G + g;
    }
}

// Probe features of the midpoint of the samples with phase rows Tu and Tv:
// x_j / pi = (Tu_j + Tv_j) / 2, sin(a_u + a_v) = sin a_u cos a_v + cos a_u
// sin a_v, cos(a_u + a_v) = cos a_u cos a_v - sin a_u sin a_v (FP64), each
// rounded once to BF16; two threads per row as in row_features.
__device__ __forceinline__ void mid_features(int d, const double *__restrict__ Tu, const double *__restrict__ Tv,
                                             int half, uint16_t *dst) {
    double sn[8], cs[8], qh[GTMP_MAX_DOF];
#pragma unroll
    for (int j = 0; j < GTMP_MAX_DOF; ++j)
        qh[j] = half == 0 && j < d ? (Tu[2 * GTMP_SUR_FREQ + j] + Tv[2 * GTMP_SUR_FREQ + j]) * 0.5 : 0.0;
#pragma unroll
    for (int q = 0; q < 8; ++q) {
        const int f = half * (GTMP_SUR_FREQ / 2) + q;
        const double su = Tu[f], cu = Tu[GTMP_SUR_FREQ + f], sv = Tv[f], cv = Tv[GTMP_SUR_FREQ + f];
        sn[q] = __builtin_fma(su, cv, cu * sv);
        cs[q] = __builtin_fma(cu, cv, -(su * sv));
    }
    store_features(d, half, sn, cs, qh, dst);
}

constexpr int kSegLds = 130;  // segment bounds kept in LDS (M <= 128)

// One block per tile of 128 candidates, launched over the upper bound E / 128
// (the candidate count is known only on the device: blocks past it return
// at once).  Blocks of one CU start at different times, so one block's
// feature or head phase overlaps the other's MFMAs.  The candidate's
// endpoints give the features of the midpoint (u + v) / 2 (from their phase
// rows) and its logit z; prune[e] = z > tau and logits[e] = z at the edge's
// flat id e (C_s | C_h | C_l order).
template <typename IDX>
__global__ void __launch_bounds__(256, 2) k_mlp_prune(int d, int M, int N, int G, const double *__restrict__ T,
                                                     const int32_t *__restrict__ fl, const int32_t *__restrict__ nf,
                                                     const int64_t *__restrict__ seg, const bf16x8 *__restrict__ Wf,
                                                     const uint16_t *__restrict__ P16, const float *__restrict__ P32,
                                                     SurLayout L, float tau,
                                                     uint8_t *__restrict__ prune, float *__restrict__ logits) {
    __shared__ __attribute__((aligned(16))) uint16_t act[kFR * kFRow];
    __shared__ float w5s[GTMP_SUR_WIDTH];
    __shared__ float zpart[kFR];
    __shared__ int64_t eid[kFR];
    __shared__ int64_t seg_s[kSegLds];
    __shared__ int32_t nf_s[kSegLds];
    const int tid = threadIdx.x;
    const int64_t total = seg[M + 1];
    const int64_t tile = blockIdx.x;
    if (tile * kFR >= total) return;  // block-uniform
    const bool in_lds = M + 2 <= kSegLds;
    if (in_lds) {
        for (int i = tid; i < M + 2; i += blockDim.x) seg_s[i] = seg[i];
        for (int i = tid; i < M; i += blockDim.x) nf_s[i] = nf[i];
    }
    if (tid < GTMP_SUR_WIDTH) w5s[tid] = bf2f(P16[L.w5 + tid]);
    __syncthreads();
    const int64_t *sg = in_lds ? seg_s : seg;
    const int32_t *nl = in_lds ? nf_s : nf;
    {
        const int r = tid & (kFR - 1), half = tid >> 7;
        const int64_t t = tile * kFR + r;
        int64_t ru = 0, rv = 0, e = -1;
        if (t < total) cand_rows<IDX>(t, M, N, G, sg, nl, fl, ru, rv, e);
        if (half == 0) eid[r] = e;
        if (e >= 0) {
            mid_features(d, T + (size_t)ru * kPhaseRow, T + (size_t)rv * kPhaseRow, half, act + r * kFRow);
        } else {
            uint4 *z4 = reinterpret_cast<uint4 *>(act + r * kFRow + 32 * half);
            for (int c = 0; c < 4; ++c) z4[c] = make_uint4(0u, 0u, 0u, 0u);
        }
    }
    __syncthreads();
    const float z = mlp_tile(Wf, P32, L, act, w5s, zpart, tid);
    if (tid < kFR) {
        const int64_t e = eid[tid];
        if (e >= 0) {
            prune[e] = z > tau ? 1 : 0;
            if (logits) logits[e] = z;
        }
    }
}

// ------------------------------------------------------------------ training
// One step's loss and gradient in four launches (weight fragments, rows, weight
// gradients, sums).  A batch of 8192 rows is 10.5 GFLOP and a few megabytes,
// microseconds of either, so a step is bound by launches and by how often the
// activations cross memory: the layer-by-layer form (products, transposes,
// column sums and split sums one after another, 42 launches) took 596 us of
// kernel time for 8192 rows; these take 51 (rows 25, weight gradients 13, sums
// 5, Adam 4, fragments 3).
//
// k_train_rows takes kTR rows through the whole network and back in one block:
// the activations of every layer stay in LDS, each gradient dZ_l overwrites
// the activations it masks.  kTR = 32 puts 8192 rows on 256 CUs; eight waves
// share the 256 columns of a layer, a 32 x 32 tile each, the weights read from
// L2 in fragment order (forward and transposed copies).  What the weight
// gradients need, A_{l-1} and dZ_l, leaves the block once, as slabs in MFMA
// operand order of the product over the batch (per 32 columns and 16 rows the
// 64 lanes' 16-byte operands side by side: lane holds rows 8 (lane / 32) ..+8
// of column lane % 32), so k_train_weights reads its fragments with contiguous
// 1 KB loads, without LDS or transposes (with slabs [column][row], whose
// loads touch twice the lines, it took 18 us instead of 13).  Sums over rows (biases, output layer, loss) leave as one
// partial per half slab and are added in slab order.
// Every layer's sums run over K in the order of the inference kernels' MFMAs.
constexpr int kTR = 32;
constexpr int kTRow0 = GTMP_SUR_IN + 8;      // LDS row strides (BF16)
constexpr int kTRow = GTMP_SUR_WIDTH + 8;
constexpr int kTSplit = 8;                   // batch splits of the weight gradients
constexpr int kTVec = 5;                     // column sums per half slab: w5, b4, b3, b2, b1

// Backward fragments of layers 2..4 (l = 1..3): W_l transposed.
constexpr int kBackLayer = kColTiles * (GTMP_SUR_WIDTH / 16) * 64;

// Forward fragments as k_weight_frag lays them out but with layer 1's columns
// in the standard feature order, then the backward ones: lane's operand of
// (column tile c, K slice ks) is W_l[16 ks + 8 (lane / 32) ..+8][32 c + lane % 32].
__global__ void __launch_bounds__(256) k_train_frag(const uint16_t *__restrict__ P16, SurLayout L,
                                                    uint4 *__restrict__ Wf, uint4 *__restrict__ Wb) {
    const int f = blockIdx.x * blockDim.x + threadIdx.x;
    if (f < kFragTotal) {
        const int l = f < frag_offset(1) ? 0 : 1 + (f - frag_offset(1)) / (frag_offset(2) - frag_offset(1));
        const int K = l == 0 ? GTMP_SUR_IN : GTMP_SUR_WIDTH, S = K / 16;
        const int r = f - frag_offset(l);
        const int lane = r & 63, ks = (r >> 6) % S, c = (r >> 6) / S;
        Wf[f] = *reinterpret_cast<const uint4 *>(P16 + L.W[l] + (size_t)(32 * c + (lane & 31)) * K + 16 * ks +
                                                 8 * (lane >> 5));
        return;
    }
    const int b = f - kFragTotal;
    if (b >= 3 * kBackLayer) return;
    const int l = 1 + b / kBackLayer, r = b % kBackLayer;
    const int lane = r & 63, ks = (r >> 6) % (GTMP_SUR_WIDTH / 16), c = (r >> 6) / (GTMP_SUR_WIDTH / 16);
    const uint16_t *src = P16 + L.W[l] + (size_t)(16 * ks + 8 * (lane >> 5)) * GTMP_SUR_WIDTH + 32 * c + (lane & 31);
    uint16_t w[8];
#pragma unroll
    for (int i = 0; i < 8; ++i) w[i] = src[(size_t)i * GTMP_SUR_WIDTH];
    Wb[b] = make_uint4(pack2(w[0], w[1]), pack2(w[2], w[3]), pack2(w[4], w[5]), pack2(w[6], w[7]));
}

// A wave's weight fragments of one layer (its 32 columns), requested before
// the barrier that ends the layer before: a read of the weights goes past the
// XCD's L2 once per step, several layers' worth of MFMAs away.
template <int K>
struct TrainW {
    bf16x8 w[K / 16];
    __device__ __forceinline__ TrainW(const bf16x8 *__restrict__ W, int wave, int lane) {
#pragma unroll
        for (int k = 0; k < K / 16; ++k) w[k] = W[((size_t)wave * (K / 16) + k) * 64 + lane];
    }
};

// The wave's 32 output columns of in [kTR][K] (LDS, row stride RS): element v
// of the result is column 8 (v/4) + 4 (lane/32) + v%4 of the tile, row lane%32.
template <int K, int RS>
__device__ __forceinline__ f32x16 train_tile(const TrainW<K> &W, const uint16_t *in, int lane) {
    constexpr int S = K / 16;
    f32x16 acc;
#pragma unroll
    for (int v = 0; v < 16; ++v) acc[v] = 0.f;
    const uint16_t *a = in + (lane & 31) * RS + 8 * (lane >> 5);
#pragma unroll
    for (int k = 0; k < S; ++k)
        acc = __builtin_amdgcn_mfma_f32_32x32x16_bf16(W.w[k], *reinterpret_cast<const bf16x8 *>(a + 16 * k), acc, 0, 0, 0);
    return acc;
}

__device__ __forceinline__ uint2 pack4(const uint16_t (&h)[4]) { return make_uint2(pack2(h[0], h[1]), pack2(h[2], h[3])); }

// out = bf16(relu(in W^T + bias)), the wave's columns.
template <int K, int RS>
__device__ __forceinline__ void train_forward(const TrainW<K> &W, const float *__restrict__ bias, const uint16_t *in,
                                              uint16_t *out, int wave, int lane) {
    const f32x16 acc = train_tile<K, RS>(W, in, lane);
#pragma unroll
    for (int g = 0; g < 4; ++g) {
        const int col = 32 * wave + 8 * g + 4 * (lane >> 5);
        uint16_t h[4];
#pragma unroll
        for (int r = 0; r < 4; ++r) {
            const float z = acc[4 * g + r] + bias[col + r];
            h[r] = f2bf(z > 0.f ? z : 0.f);
        }
        *reinterpret_cast<uint2 *>(&out[(lane & 31) * kTRow + col]) = pack4(h);
    }
}

// act = bf16((dZ W) * [act > 0]), the wave's columns, in place.
__device__ __forceinline__ void train_backward(const TrainW<GTMP_SUR_WIDTH> &W, const uint16_t *dZ, uint16_t *act, int wave,
                                               int lane) {
    const f32x16 acc = train_tile<GTMP_SUR_WIDTH, kTRow>(W, dZ, lane);
#pragma unroll
    for (int g = 0; g < 4; ++g) {
        uint2 *p = reinterpret_cast<uint2 *>(&act[(lane & 31) * kTRow + 32 * wave + 8 * g + 4 * (lane >> 5)]);
        const uint2 m = *p;
        const uint32_t mw[2] = {m.x, m.y};
        uint16_t h[4];
#pragma unroll
        for (int r = 0; r < 4; ++r) {
            const bool on = bf2f((uint16_t)(mw[r >> 1] >> (16 * (r & 1)))) > 0.f;
            h[r] = f2bf(on ? acc[4 * g + r] : 0.f);
        }
        *p = pack4(h);
    }
}

// Half a column of t (16 rows from row 16 half) into its slab.
template <int RS>
__device__ __forceinline__ void read_half_column(const uint16_t *t, int c, int half, uint16_t (&h)[16]) {
#pragma unroll
    for (int r = 0; r < 16; ++r) h[r] = t[(16 * half + r) * RS + c];
}
__device__ __forceinline__ void store_half_column(uint16_t *slab, int c, int half, const uint16_t (&h)[16]) {
    uint4 *dst = reinterpret_cast<uint4 *>(slab) + ((c >> 5) * 2 + half) * 64 + (c & 31);
#pragma unroll
    for (int q = 0; q < 2; ++q)
        dst[32 * q] = make_uint4(pack2(h[8 * q], h[8 * q + 1]), pack2(h[8 * q + 2], h[8 * q + 3]),
                            pack2(h[8 * q + 4], h[8 * q + 5]), pack2(h[8 * q + 6], h[8 * q + 7]));
}

struct TrainBufs {
    uint4 *Wf, *Wb;
    uint16_t *X0, *A[3], *dZ[4];  // slabs: features, activations 1..3, gradients 1..4
    float *col;                   // [slab][half][kTVec][256]
    float *row;                   // [slab][2]: loss terms, dz
    float *part;                  // [kTSplit][weights]
    size_t total;
};

__global__ void __launch_bounds__(512, 2) k_train_rows(int d, const float *__restrict__ X, const uint8_t *__restrict__ y,
                                                       const float *__restrict__ Bf, const uint16_t *__restrict__ P16,
                                                       const float *__restrict__ P32, SurLayout L, float inv_n,
                                                       float *__restrict__ logits, TrainBufs T) {
    __shared__ __attribute__((aligned(16))) uint16_t x0[kTR * kTRow0];
    __shared__ __attribute__((aligned(16))) uint16_t act[4][kTR * kTRow];
    __shared__ float dz_s[kTR], loss_s[kTR];
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int c = tid & 255, half = tid >> 8;
    const size_t slab = blockIdx.x, row0 = slab * kTR;
    const bf16x8 *Wf = reinterpret_cast<const bf16x8 *>(T.Wf), *Wb = reinterpret_cast<const bf16x8 *>(T.Wb);
    const TrainW<GTMP_SUR_IN> w1(Wf + frag_offset(0), wave, lane);
    const TrainW<GTMP_SUR_WIDTH> w2(Wf + frag_offset(1), wave, lane);
    {  // features: a thread per (row, frequency), the first d also the linear ones
        constexpr double kPi = 3.14159265358979323846;
        const int r = tid >> 4, f = tid & 15;
        const float *x = X + (row0 + r) * d;
        double qh[GTMP_MAX_DOF];
        for (int j = 0; j < GTMP_MAX_DOF; ++j) qh[j] = j < d ? (double)x[j] / kPi : 0.0;
        double s = 0.0;
        for (int j = 0; j < d; ++j) s += (double)Bf[f * d + j] * qh[j];
        s *= 2.0 * kPi;
        double sn, cs;
        sincos(s, &sn, &cs);
        uint16_t *o = x0 + r * kTRow0;
        o[d + f] = d2bf(sn);
        o[d + GTMP_SUR_FREQ + f] = d2bf(cs);
        for (int j = 0; j < GTMP_MAX_DOF; ++j)
            if (j == f && j < d) o[j] = d2bf(qh[j]);
        for (int k = d + 2 * GTMP_SUR_FREQ + f; k < GTMP_SUR_IN; k += 16) o[k] = 0;
    }
    __syncthreads();
    if (tid < 2 * GTMP_SUR_IN) {
        uint16_t h[16];
        read_half_column<kTRow0>(x0, tid & (GTMP_SUR_IN - 1), tid / GTMP_SUR_IN, h);
        store_half_column(T.X0 + slab * kTR * GTMP_SUR_IN, tid & (GTMP_SUR_IN - 1), tid / GTMP_SUR_IN, h);
    }
    const size_t so = slab * kTR * GTMP_SUR_WIDTH;
    auto put = [&](const uint16_t *t, uint16_t *dst) {
        uint16_t h[16];
        read_half_column<kTRow>(t, c, half, h);
        store_half_column(dst + so, c, half, h);
    };
    train_forward<GTMP_SUR_IN, kTRow0>(w1, P32 + L.b[0], x0, act[0], wave, lane);
    const TrainW<GTMP_SUR_WIDTH> w3(Wf + frag_offset(2), wave, lane);
    __syncthreads();
    train_forward<GTMP_SUR_WIDTH, kTRow>(w2, P32 + L.b[1], act[0], act[1], wave, lane);
    const TrainW<GTMP_SUR_WIDTH> w4(Wf + frag_offset(3), wave, lane);
    put(act[0], T.A[0]);
    __syncthreads();
    train_forward<GTMP_SUR_WIDTH, kTRow>(w3, P32 + L.b[2], act[1], act[2], wave, lane);
    const TrainW<GTMP_SUR_WIDTH> v4(Wb + 2 * kBackLayer, wave, lane);
    put(act[1], T.A[1]);
    __syncthreads();
    train_forward<GTMP_SUR_WIDTH, kTRow>(w4, P32 + L.b[3], act[2], act[3], wave, lane);
    const TrainW<GTMP_SUR_WIDTH> v3(Wb + kBackLayer, wave, lane);
    put(act[2], T.A[2]);
    __syncthreads();
    // output layer, loss and its gradient: a wave per row, four products a lane
    //   z = sum_k bf16(w5)[k] a4[k] + b5;  loss_b = max(z,0) - y z + log1p(exp(-|z|));
    //   dz = (sigmoid(z) - y) / n
    for (int r = wave; r < kTR; r += 8) {
        const uint16_t *a = act[3] + r * kTRow;
        float s = 0.f;
#pragma unroll
        for (int q = 0; q < GTMP_SUR_WIDTH / kWave; ++q) {
            const int k = lane * (GTMP_SUR_WIDTH / kWave) + q;
            s = __builtin_fmaf(bf2f(P16[L.w5 + k]), bf2f(a[k]), s);
        }
#pragma unroll
        for (int off = kWave / 2; off > 0; off >>= 1) s += __shfl_xor(s, off);
        if (lane == 0) {
            const float z = s + P32[L.b5];
            if (logits) logits[row0 + r] = z;
            const float yy = y[row0 + r] ? 1.f : 0.f;
            const float az = __builtin_fabsf(z);
            const float e = __expf(-az);
            loss_s[r] = (z > 0.f ? z : 0.f) - yy * z + log1pf(e);
            const float sig = z >= 0.f ? 1.f / (1.f + e) : e / (1.f + e);
            dz_s[r] = (sig - yy) * inv_n;
        }
    }
    __syncthreads();
    float *col = T.col + ((2 * slab + half) * kTVec) * GTMP_SUR_WIDTH + c;
    {  // dw5's part, then dZ4 = bf16(dz[b] bf16(w5)[k] [a4 > 0]) over a4, its column sum and slab
        const float wk = bf2f(P16[L.w5 + c]);
        uint16_t h[16];
        float sw = 0.f, sb = 0.f;
#pragma unroll
        for (int r = 0; r < 16; ++r) {
            uint16_t *p = &act[3][(16 * half + r) * kTRow + c];
            const float a = bf2f(*p), g = dz_s[16 * half + r];
            sw = __builtin_fmaf(g, a, sw);
            h[r] = f2bf(a > 0.f ? g * wk : 0.f);
            *p = h[r];
            sb += bf2f(h[r]);
        }
        col[0] = sw;
        col[GTMP_SUR_WIDTH] = sb;
        store_half_column(T.dZ[3] + so, c, half, h);
        if (wave == 0) {
            float a = lane < kTR ? loss_s[lane] : 0.f, b = lane < kTR ? dz_s[lane] : 0.f;
#pragma unroll
            for (int off = kTR / 2; off > 0; off >>= 1) {
                a += __shfl_xor(a, off);
                b += __shfl_xor(b, off);
            }
            if (lane == 0) {
                T.row[2 * slab] = a;
                T.row[2 * slab + 1] = b;
            }
        }
    }
    __syncthreads();
    auto finish = [&](int l) {  // slab and column sum of dZ_{l+1}, in act[l]
        uint16_t h[16];
        read_half_column<kTRow>(act[l], c, half, h);
        store_half_column(T.dZ[l] + so, c, half, h);
        float sb = 0.f;
#pragma unroll
        for (int r = 0; r < 16; ++r) sb += bf2f(h[r]);
        col[(4 - l) * GTMP_SUR_WIDTH] = sb;
    };
    train_backward(v4, act[3], act[2], wave, lane);
    const TrainW<GTMP_SUR_WIDTH> v2(Wb, wave, lane);
    __syncthreads();
    train_backward(v3, act[2], act[1], wave, lane);
    finish(2);
    __syncthreads();
    train_backward(v2, act[1], act[0], wave, lane);
    finish(1);
    __syncthreads();
    finish(0);
}

// dW_l = dZ_l^T A_{l-1} over a split of the slabs, a 64 x 128 tile (layer 1:
// 64 x 64) per block of four waves, 32 x 64 (32 x 32) each; a slab's
// fragments are requested kTAhead slabs ahead.  Split k takes every kTSplit-th
// slab from k, and its blocks are the ones of index k modulo kTSplit: blocks
// are dealt to the eight XCDs in turn, so the XCD that wrote a slab reads it
// again, and each XCD reads an eighth of the slabs (splits of consecutive
// slabs over consecutive blocks, every XCD reading all of them, took 20 us).
// Tiles (64 x 128) rather
// than 128 x 128 so that eight splits, whose partials are 6.8 MB to write and
// add, already make 224 blocks.
constexpr int kTWeights = GTMP_SUR_WIDTH * GTMP_SUR_IN + 3 * GTMP_SUR_WIDTH * GTMP_SUR_WIDTH;
__host__ __device__ constexpr int train_part_offset(int l) {
    return l == 0 ? 0 : GTMP_SUR_WIDTH * GTMP_SUR_IN + (l - 1) * GTMP_SUR_WIDTH * GTMP_SUR_WIDTH;
}
constexpr int kTTiles = 4 + 3 * 8;  // blocks per split
constexpr int kTAhead = 4;          // slabs of fragments in flight per wave

template <int NJ>
__device__ __forceinline__ void train_weight_tile(const uint16_t *__restrict__ dZ, const uint16_t *__restrict__ Ap,
                                                  int K_in, int m0, int n0, size_t slab0, int slabs, float *out,
                                                  int lane) {
    const int cl = lane & 31;
    f32x16 acc[NJ];
#pragma unroll
    for (int j = 0; j < NJ; ++j)
#pragma unroll
        for (int v = 0; v < 16; ++v) acc[j][v] = 0.f;
    // in 16-byte fragments: a slab holds kTR / 8 of each column
    const bf16x8 *pa = reinterpret_cast<const bf16x8 *>(dZ) + (slab0 * GTMP_SUR_WIDTH + m0) * (kTR / 8) + lane;
    const bf16x8 *pb = reinterpret_cast<const bf16x8 *>(Ap) + (slab0 * K_in + n0) * (kTR / 8) + lane;
    const size_t sa = (size_t)kTSplit * (kTR / 8) * GTMP_SUR_WIDTH, sb = (size_t)kTSplit * (kTR / 8) * K_in;
    bf16x8 a[kTAhead][2], b[kTAhead][NJ][2];
    auto load = [&](int q, int s) {
#pragma unroll
        for (int k = 0; k < 2; ++k) {
            a[q][k] = pa[s * sa + 64 * k];
#pragma unroll
            for (int j = 0; j < NJ; ++j) b[q][j][k] = pb[s * sb + 128 * j + 64 * k];
        }
    };
#pragma unroll
    for (int q = 0; q < kTAhead; ++q) load(q, q < slabs ? q : 0);
    for (int s0 = 0; s0 < slabs; s0 += kTAhead) {
#pragma unroll
        for (int q = 0; q < kTAhead; ++q) {
            if (s0 + q < slabs) {
#pragma unroll
                for (int k = 0; k < 2; ++k)
#pragma unroll
                    for (int j = 0; j < NJ; ++j)
                        acc[j] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a[q][k], b[q][j][k], acc[j], 0, 0, 0);
            }
            const int nx = s0 + q + kTAhead;
            load(q, nx < slabs ? nx : 0);
        }
    }
#pragma unroll
    for (int j = 0; j < NJ; ++j)
#pragma unroll
        for (int v = 0; v < 16; ++v)
            out[(size_t)(m0 + 8 * (v >> 2) + 4 * (lane >> 5) + (v & 3)) * K_in + n0 + 32 * j + cl] = acc[j][v];
}

__global__ void __launch_bounds__(256) k_train_weights(int slabs_per_split, TrainBufs T) {
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const int split = blockIdx.x % kTSplit, t = blockIdx.x / kTSplit;
    const size_t slab0 = (size_t)split;
    float *part = T.part + (size_t)split * kTWeights;
    if (t < 4) {  // layer 1: 256 x 64
        train_weight_tile<1>(T.dZ[0], T.X0, GTMP_SUR_IN, 64 * t + 32 * (wave >> 1), 32 * (wave & 1), slab0,
                             slabs_per_split, part + train_part_offset(0), lane);
        return;
    }
    const int l = 1 + (t - 4) / 8, q = (t - 4) % 8;
    const uint16_t *dZ = l == 1 ? T.dZ[1] : l == 2 ? T.dZ[2] : T.dZ[3];
    const uint16_t *Ap = l == 1 ? T.A[0] : l == 2 ? T.A[1] : T.A[2];
    train_weight_tile<2>(dZ, Ap, GTMP_SUR_WIDTH, 64 * (q >> 1) + 32 * (wave >> 1), 128 * (q & 1) + 64 * (wave & 1),
                         slab0, slabs_per_split, part + train_part_offset(l), lane);
}

// The partials added in their order: weights (a thread per entry), then the
// column sums (16 columns per block, the half slabs in 16 runs), then the
// loss and db5.
constexpr int kTSumWeights = kTWeights / 256, kTSumCols = kTVec * GTMP_SUR_WIDTH / 16;
static_assert(kTWeights % 256 == 0, "whole blocks of weights");

__global__ void __launch_bounds__(256) k_train_sums(int slabs, SurLayout L, float inv_n, TrainBufs T,
                                                    float *__restrict__ grad, float *__restrict__ loss) {
    __shared__ float sh[2][256];
    const int tid = threadIdx.x, b = blockIdx.x;
    if (b < kTSumWeights) {
        const int i = b * 256 + tid;
        float p[kTSplit];
#pragma unroll
        for (int k = 0; k < kTSplit; ++k) p[k] = T.part[(size_t)k * kTWeights + i];
        float s = 0.f;
#pragma unroll
        for (int k = 0; k < kTSplit; ++k) s += p[k];
        const int l = i < train_part_offset(1) ? 0 : 1 + (i - train_part_offset(1)) / (GTMP_SUR_WIDTH * GTMP_SUR_WIDTH);
        grad[L.W[l] + i - train_part_offset(l)] = s;
        return;
    }
    if (b < kTSumWeights + kTSumCols) {
        const int c = (b - kTSumWeights) * 16 + (tid & 15), run = tid >> 4;  // c: vector * 256 + column
        const int per = slabs / 8;                                          // 2 slabs / 16 runs
        const float *p = T.col + (size_t)run * per * kTVec * GTMP_SUR_WIDTH + c;
        float s = 0.f;
#pragma unroll 8
        for (int k = 0; k < per; ++k) s += p[(size_t)k * kTVec * GTMP_SUR_WIDTH];
        sh[0][tid] = s;
        __syncthreads();
        if (run == 0) {
            for (int r = 1; r < 16; ++r) s += sh[0][16 * r + tid];
            const int v = c / GTMP_SUR_WIDTH, k = c % GTMP_SUR_WIDTH;
            grad[(v == 0 ? L.w5 : L.b[4 - v]) + k] = s;
        }
        return;
    }
    float a = 0.f, z = 0.f;
    for (int k = tid; k < slabs; k += 256) {
        a += T.row[2 * k];
        z += T.row[2 * k + 1];
    }
    sh[0][tid] = a;
    sh[1][tid] = z;
    for (int h = 128; h > 0; h >>= 1) {
        __syncthreads();
        if (tid < h) {
            sh[0][tid] += sh[0][tid + h];
            sh[1][tid] += sh[1][tid + h];
        }
    }
    if (tid == 0) {
        *loss = sh[0][0] * inv_n;
        grad[L.b5] = sh[1][0];
    }
}

// ------------------------------------------------------------------ small kernels
__global__ void __launch_bounds__(256) k_adam(int total, float *__restrict__ P, uint16_t *__restrict__ P16,
                                              const float *__restrict__ g, float *__restrict__ m,
                                              float *__restrict__ v, float lr, float b1, float b2, float eps,
                                              float c1, float c2) {
    const int i = blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= total) return;
    const float gi = g[i];
    const float mi = b1 * m[i] + (1.f - b1) * gi;
    const float vi = b2 * v[i] + (1.f - b2) * gi * gi;
    m[i] = mi;
    v[i] = vi;
    const float p = P[i] - lr * (mi * c1) / (__builtin_sqrtf(vi * c2) + eps);
    P[i] = p;
    P16[i] = f2bf(p);
}

__global__ void __launch_bounds__(256) k_to_bf16(int total, const float *__restrict__ P, uint16_t *__restrict__ P16) {
    const int i = blockIdx.x * blockDim.x + threadIdx.x;
    if (i < total) P16[i] = f2bf(P[i]);
}

// Training states: rows [0, n) uniform (layer 0), rows [n, 2n) interior
// lerp states of the edge (layer-1 sample j, layer-2 sample j).
__global__ void __launch_bounds__(256) k_label_states(int d, int64_t n, int H, uint32_t k0, uint32_t k1,
                                                      uint32_t stage, SurBox B, float *__restrict__ X) {
    const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= 2 * n) return;
    const int nblk = (d + 3) >> 2;
    auto sample = [&](uint32_t m, uint32_t s, float *x) {
        for (int blk = 0; blk < nblk; ++blk) {
            const uint4 w = philox4x32_10(make_uint4(s, m, stage, (uint32_t)blk), k0, k1);
            const uint32_t ws[4] = {w.x, w.y, w.z, w.w};
            for (int q = 0; q < 4; ++q) {
                const int j = blk * 4 + q;
                if (j < d) x[j] = __builtin_fmaf(unit_from_word(ws[q]), B.wd[j], B.lo[j]);
            }
        }
    };
    float x[GTMP_MAX_DOF];
    if (i < n) {
        sample(0u, (uint32_t)i, x);
    } else {
        const int64_t j = i - n;
        float u[GTMP_MAX_DOF], v[GTMP_MAX_DOF];
        sample(1u, (uint32_t)j, u);
        sample(2u, (uint32_t)j, v);
        const int h = 1 + (int)(j % (H - 2));
        const float t = (float)h / (float)(H - 1);
        for (int q = 0; q < d; ++q) x[q] = __builtin_fmaf(t, v[q] - u[q], u[q]);
    }
    for (int q = 0; q < d; ++q) X[i * d + q] = x[q];
}

// ------------------------------------------------------------------ host side
static unsigned blocks_for(int64_t n, int per = 256) { return (unsigned)((n + per - 1) / per); }

static size_t up256(size_t x) { return (x + 255) & ~size_t(255); }

// Workspace of a training step of n rows (a multiple of 256).
static TrainBufs carve_train(int64_t n, void *base) {
    TrainBufs w{};
    char *p = static_cast<char *>(base);
    size_t o = 0;
    auto take = [&](size_t bytes) { char *q = p ? p + o : nullptr; o = up256(o + bytes); return q; };
    const size_t act = sizeof(uint16_t) * n * GTMP_SUR_WIDTH, slabs = (size_t)n / kTR;
    w.Wf = reinterpret_cast<uint4 *>(take(sizeof(uint4) * kFragTotal));
    w.Wb = reinterpret_cast<uint4 *>(take(sizeof(uint4) * 3 * kBackLayer));
    w.X0 = reinterpret_cast<uint16_t *>(take(sizeof(uint16_t) * n * GTMP_SUR_IN));
    for (int l = 0; l < 3; ++l) w.A[l] = reinterpret_cast<uint16_t *>(take(act));
    for (int l = 0; l < 4; ++l) w.dZ[l] = reinterpret_cast<uint16_t *>(take(act));
    w.col = reinterpret_cast<float *>(take(sizeof(float) * 2 * slabs * kTVec * GTMP_SUR_WIDTH));
    w.row = reinterpret_cast<float *>(take(sizeof(float) * 2 * slabs));
    w.part = reinterpret_cast<float *>(take(sizeof(float) * kTSplit * kTWeights));
    w.total = o;
    return w;
}

size_t sur_workspace_bytes(int64_t n) { return carve_train(n, nullptr).total; }

// Inference keeps its activations in LDS: the weights in fragment order.
size_t sur_infer_bytes() { return up256(sizeof(uint4) * kFragTotal); }

static void weight_frag(const SurNet &net, uint4 *Wf, hipStream_t s) {
    hipLaunchKernelGGL(k_weight_frag, dim3((kFragTotal + 255) / 256), dim3(256), 0, s, net.d, net.p16, sur_layout(),
                       Wf);
}

hipError_t launch_sur_infer(const SurNet &net, int64_t n, const float *X, float *logits, void *ws, hipStream_t s) {
    if (n <= 0) return hipSuccess;
    uint4 *Wf = static_cast<uint4 *>(ws);
    weight_frag(net, Wf, s);
    // chunks bound the grid size
    constexpr int64_t kChunk = (int64_t)1 << 30;
    for (int64_t r = 0; r < n; r += kChunk) {
        const int64_t c = n - r < kChunk ? n - r : kChunk;
        hipLaunchKernelGGL(k_mlp_infer, dim3((unsigned)((c + kFR - 1) / kFR)), dim3(256), 0, s, net.d, c,
                           X + r * net.d, net.fourier, reinterpret_cast<const bf16x8 *>(Wf), net.p16, net.p32,
                           sur_layout(), logits + r);
    }
    return hipGetLastError();
}

hipError_t launch_sur_grad(const SurNet &net, int n, const float *X, const uint8_t *y, float *grad, float *loss,
                           float *logits, void *ws, hipStream_t s) {
    const SurLayout L = sur_layout();
    const TrainBufs w = carve_train(n, ws);
    const int slabs = n / kTR;  // a multiple of kTSplit
    static_assert(256 % (kTR * kTSplit) == 0, "every split takes whole slabs");
    const float inv_n = 1.f / (float)n;
    hipLaunchKernelGGL(k_train_frag, dim3(blocks_for(kFragTotal + 3 * kBackLayer)), dim3(256), 0, s, net.p16, L, w.Wf,
                       w.Wb);
    hipLaunchKernelGGL(k_train_rows, dim3((unsigned)slabs), dim3(512), 0, s, net.d, X, y, net.fourier, net.p16, net.p32,
                       L, inv_n, logits, w);
    hipLaunchKernelGGL(k_train_weights, dim3(kTSplit * kTTiles), dim3(256), 0, s, slabs / kTSplit, w);
    hipLaunchKernelGGL(k_train_sums, dim3(kTSumWeights + kTSumCols + 1), dim3(256), 0, s, slabs, L, inv_n, w, grad,
                       loss);
    return hipGetLastError();
}

hipError_t launch_sur_adam(const SurNet &net, const float *grad, float *m, float *v, int t, float lr, float b1,
                           float b2, float eps, hipStream_t s) {
    const int total = sur_layout().total;
    const double c1 = 1.0 / (1.0 - std::pow((double)b1, (double)t));
    const double c2 = 1.0 / (1.0 - std::pow((double)b2, (double)t));
    hipLaunchKernelGGL(k_adam, dim3(blocks_for(total)), dim3(256), 0, s, total, net.p32, net.p16, grad, m, v, lr, b1,
                       b2, eps, (float)c1, (float)c2);
    return hipGetLastError();
}

hipError_t launch_sur_refresh(const SurNet &net, hipStream_t s) {
    const int total = sur_layout().total;
    hipLaunchKernelGGL(k_to_bf16, dim3(blocks_for(total)), dim3(256), 0, s, total, net.p32, net.p16);
    return hipGetLastError();
}

hipError_t launch_sur_label_states(const gtmp_problem &p, uint64_t seed, uint64_t stage, int64_t n, float *X,
                                   hipStream_t s) {
    SurBox B{};
    for (int j = 0; j < p.d; ++j) {
        B.lo[j] = p.lo[j];
        B.wd[j] = p.hi[j] - p.lo[j];
    }
    if (n > 0)
        hipLaunchKernelGGL(k_label_states, dim3(blocks_for(2 * n)), dim3(256), 0, s, p.d, n, p.H,
                           (uint32_t)(seed & 0xffffffffu), (uint32_t)(seed >> 32), (uint32_t)stage, B, X);
    return hipGetLastError();
}

// Workspace of the pruning call: fragment-order weights, the free lists
// [M][N], their lengths [M] and the M + 2 segment bounds.
struct PruneWs {
    uint4 *Wf;
    int32_t *fl, *nf;
    double *T;
    int64_t *seg;
    size_t total;
};

static PruneWs carve_prune(const gtmp_problem &p, void *base) {
    PruneWs w{};
    char *q = static_cast<char *>(base);
    size_t o = 0;
    auto take = [&](size_t bytes) { char *r = q ? q + o : nullptr; o = up256(o + bytes); return r; };
    w.Wf = reinterpret_cast<uint4 *>(take(sizeof(uint4) * kFragTotal));
    w.fl = reinterpret_cast<int32_t *>(take(sizeof(int32_t) * (size_t)p.M * p.N));
    w.T = reinterpret_cast<double *>(take(sizeof(double) * kPhaseRow * ((size_t)p.M * p.N + 1 + p.G)));
    w.nf = reinterpret_cast<int32_t *>(take(sizeof(int32_t) * (size_t)p.M));
    w.seg = reinterpret_cast<int64_t *>(take(sizeof(int64_t) * ((size_t)p.M + 2)));
    w.total = o;
    return w;
}

size_t sur_prune_bytes(const gtmp_problem &p) { return carve_prune(p, nullptr).total; }

hipError_t launch_sur_prune(const gtmp_problem &p, const SurNet &net, const float *q0, const float *goals,
                            const float *Q, const uint8_t *vcoll, float tau, uint8_t *prune, float *logits, void *ws,
                            hipStream_t s) {
    const int64_t E = (int64_t)p.N + (int64_t)(p.M - 1) * p.N * p.N + (int64_t)p.N * p.G;
    const PruneWs w = carve_prune(p, ws);
    weight_frag(net, w.Wf, s);
    const int64_t fill_blocks = std::min<int64_t>((E + 255) / 256, 4096);
    hipLaunchKernelGGL(k_prune_fill, dim3((unsigned)fill_blocks), dim3(256), 0, s, E, prune, logits);
    hipLaunchKernelGGL(k_free_lists, dim3(p.M), dim3(256), 0, s, p.N, vcoll, w.fl, w.nf);
    const int64_t rows = (int64_t)p.M * p.N + 1 + p.G;
    hipLaunchKernelGGL(k_sample_phases, dim3((unsigned)((rows + 255) / 256)), dim3(256), 0, s, p.d, p.M, p.N, p.G, Q,
                       q0, goals, w.fl, w.nf, net.fourier, w.T);
    hipLaunchKernelGGL(k_cand_segments, dim3(1), dim3(64), 0, s, p.M, p.G, w.nf, w.seg);
    const int64_t grid = (E + kFR - 1) / kFR;  // candidates <= E
    if (grid > 0x7fffffff) return hipErrorInvalidValue;
    // 32-bit index arithmetic when every segment's local index fits
    const bool narrow = (uint64_t)p.N * p.N < (1ull << 32) && (uint64_t)p.N * p.G < (1ull << 32);
    const auto kern = narrow ? k_mlp_prune<uint32_t> : k_mlp_prune<uint64_t>;
    hipLaunchKernelGGL(kern, dim3((unsigned)grid), dim3(256), 0, s, net.d, p.M, p.N, p.G, w.T, w.fl, w.nf, w.seg,
                       reinterpret_cast<const bf16x8 *>(w.Wf), net.p16, net.p32, sur_layout(), tau, prune, logits);
    return hipGetLastError();
}

}  // namespace gtmp
