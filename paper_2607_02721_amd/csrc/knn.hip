// Per-Gaussian features of the learned proposal: 59 attributes plus five
// features of the k = 16 nearest neighbours of each mean (exact kNN;
// neighbours ordered by (squared distance, index), self excluded).
//
// Feature vector (64 float32 per Gaussian):
//   0-2 mean, 3-5 log-scale, 6-9 normalised quaternion with w >= 0,
//   10 logit(alpha), 11-58 SH coefficients (zero beyond the scene's degree),
//   59 log mean neighbour distance, 60 log distance to the 16th neighbour,
//   61 mean neighbour alpha, 62 max neighbour alpha,
//   63 log(sum of neighbour alphas / volume of the 16th-neighbour ball).
//
// Exact search: the points are sorted along a Hilbert curve, every 32 of them
// are a leaf with its bounding box, and every 64 nodes of a level are the
// children of one node of the next.  A wave answers the queries of 64
// consecutive points of the curve: it descends from the top level, takes the
// children nearest its queries' common box first and leaves out every subtree
// that is farther than the worst 16th distance of its queries.  The curve only
// decides what is visited when; which neighbours are found does not depend on
// it.
#include "gs_internal.hpp"

#include <hip/hip_fp16.h>

#include <algorithm>

namespace gs {

constexpr int kK = 16;

__device__ __forceinline__ float kload(const void *base, int64_t idx, int fmt, bool half_ieee) {
    if (fmt == 0) return static_cast<const float *>(base)[idx];
    const uint16_t b = static_cast<const uint16_t *>(base)[idx];
    if (half_ieee) return __half2float(__ushort_as_half(b));
    return __uint_as_float((uint32_t)b << 16);
}

__device__ __forceinline__ uint32_t ord_bits(float f) {
    const uint32_t u = __float_as_uint(f);
    return (u & 0x80000000u) ? ~u : (u | 0x80000000u);
}

// Bounding box of the means (order-preserving bits, so min / max are integer
// operations) and the sums of the coordinates and of their squares, over the
// points whose coordinates are all finite: a fixed grid strides over the
// points, each block folds its waves in LDS and adds one atomic per value
// (atomics on one address serialise, so one per wave would cost about a
// millisecond at 10^6 points).
struct CloudStats {
    uint32_t lo[3], hi[3];        // ordered bits
    unsigned long long finite;
    double sum[3], sq[3];
};
constexpr int kBoxBlocks = 256;

__global__ void k_cloud_init(CloudStats *cs) {
    for (int c = 0; c < 3; ++c) {
        cs->lo[c] = 0xFFFFFFFFu;
        cs->hi[c] = 0u;
        cs->sum[c] = cs->sq[c] = 0.0;
    }
    cs->finite = 0ull;
}

__global__ __launch_bounds__(256) void k_cloud_stats(SceneDev sc, CloudStats *cs) {
    __shared__ uint32_t red[4][6];
    __shared__ double sums[4][7];
    uint32_t lo[3] = {0xFFFFFFFFu, 0xFFFFFFFFu, 0xFFFFFFFFu}, hi[3] = {0u, 0u, 0u};
    double sum[3] = {0, 0, 0}, sq[3] = {0, 0, 0}, cnt = 0;
    for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < sc.n; i += (int64_t)gridDim.x * blockDim.x) {
        float x[3];
        for (int c = 0; c < 3; ++c) x[c] = kload(sc.mean, c * sc.n + i, sc.format, false);
        if (!(isfinite(x[0]) && isfinite(x[1]) && isfinite(x[2]))) continue;
        cnt += 1.0;
        for (int c = 0; c < 3; ++c) {
            const uint32_t b = ord_bits(x[c]);
            lo[c] = min(lo[c], b);
            hi[c] = max(hi[c], b);
            sum[c] += (double)x[c];
            sq[c] += (double)x[c] * (double)x[c];
        }
    }
    for (int off = 32; off > 0; off >>= 1) {
        for (int c = 0; c < 3; ++c) {
            lo[c] = min(lo[c], (uint32_t)__shfl_xor((int)lo[c], off));
            hi[c] = max(hi[c], (uint32_t)__shfl_xor((int)hi[c], off));
            sum[c] += __shfl_xor(sum[c], off);
            sq[c] += __shfl_xor(sq[c], off);
        }
        cnt += __shfl_xor(cnt, off);
    }
    const int w = threadIdx.x >> 6;
    if ((threadIdx.x & 63) == 0) {
        for (int c = 0; c < 3; ++c) {
            red[w][c] = lo[c];
            red[w][3 + c] = hi[c];
            sums[w][c] = sum[c];
            sums[w][3 + c] = sq[c];
        }
        sums[w][6] = cnt;
    }
    __syncthreads();
    const int t = threadIdx.x;
    if (t < 3) {
        atomicMin(&cs->lo[t], min(min(red[0][t], red[1][t]), min(red[2][t], red[3][t])));
        atomicMax(&cs->hi[t], max(max(red[0][3 + t], red[1][3 + t]), max(red[2][3 + t], red[3][3 + t])));
    }
    if (t < 7) {
        const double v = (sums[0][t] + sums[1][t]) + (sums[2][t] + sums[3][t]);
        if (t < 3)
            atomicAdd(&cs->sum[t], v);
        else if (t < 6)
            atomicAdd(&cs->sq[t - 3], v);
        else
            atomicAdd(&cs->finite, (unsigned long long)v);
    }
}

__device__ __forceinline__ float from_ord(uint32_t u) {
    return __uint_as_float((u & 0x80000000u) ? (u & 0x7FFFFFFFu) : ~u);
}

// Every third bit: 10 bits -> 30.
__device__ __forceinline__ uint32_t spread3(uint32_t x) {
    x = (x | (x << 16)) & 0x030000FFu;
    x = (x | (x << 8)) & 0x0300F00Fu;
    x = (x | (x << 4)) & 0x030C30C3u;
    return (x | (x << 2)) & 0x09249249u;
}

// Position of the cell (x[0], x[1], x[2]), 10 bits each, on a 3D Hilbert curve
// (Skilling, "Programming the Hilbert curve", 2004): consecutive positions are
// neighbouring cells, so 64 consecutive points of the curve stay together (on
// a Morton curve they may lie on both sides of a jump).
__device__ __forceinline__ uint32_t hilbert30(uint32_t (&x)[3]) {
#pragma unroll
    for (uint32_t q = 512u; q > 1u; q >>= 1) {
        const uint32_t low = q - 1u;
#pragma unroll
        for (int i = 0; i < 3; ++i) {
            const uint32_t t = (x[0] ^ x[i]) & low;
            if (x[i] & q) {
                x[0] ^= low;
            } else {
                x[0] ^= t;
                x[i] ^= t;
            }
        }
    }
    x[1] ^= x[0];
    x[2] ^= x[1];
    uint32_t t = 0u;
#pragma unroll
    for (uint32_t q = 512u; q > 1u; q >>= 1) t ^= (x[2] & q) ? q - 1u : 0u;
    return (spread3(x[0] ^ t) << 2) | (spread3(x[1] ^ t) << 1) | spread3(x[2] ^ t);
}

// 30-bit curve positions on a cubic grid of 1024 cells per side over the part of
// the bounding box within three standard deviations of the centroid (a few
// far points would otherwise leave most of the cloud in a handful of cells;
// points outside go to the border cells, non-finite ones to cell 0).
__global__ __launch_bounds__(256) void k_curve(SceneDev sc, const CloudStats *__restrict__ cs,
                                                uint32_t *__restrict__ code) {
    const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= sc.n) return;
    const double m = fmax((double)cs->finite, 1.0);
    float lo[3], ext = 1e-30f;
    for (int c = 0; c < 3; ++c) {
        const double mean = cs->sum[c] / m, sd = sqrt(fmax(cs->sq[c] / m - mean * mean, 0.0));
        lo[c] = fmaxf(from_ord(cs->lo[c]), (float)(mean - 3.0 * sd));
        ext = fmaxf(ext, fminf(from_ord(cs->hi[c]), (float)(mean + 3.0 * sd)) - lo[c]);
    }
    const float inv = 1024.0f / ext;
    uint32_t x[3];
    for (int c = 0; c < 3; ++c) {
        const float f = (kload(sc.mean, c * sc.n + i, sc.format, false) - lo[c]) * inv;
        x[c] = f > 0.0f ? (uint32_t)fminf(f, 1023.0f) : 0u;   // (a NaN goes to 0)
    }
    code[i] = hilbert30(x);
}

// A node's bounding box, 32 bytes, so that a lane reads its child's box as two
// 16-byte loads and a wave-uniform one is a single scalar load.
struct __align__(32) NodeBox {
    float lo[3], hi[3];
    uint32_t first;                     // leaves: the smallest index of their points
    float pad;
};

constexpr int kLeaf = 32, kFan = 64, kMaxLevels = 5;
struct Tree {
    const float4 *pts;                  // points along the curve: x, y, z, index (bits); NaN past n
    const NodeBox *box[kMaxLevels];     // level 0: leaves
    int count[kMaxLevels];
};

__device__ __forceinline__ float half_min(float v) {   // over each 32 lanes
    for (int off = 16; off > 0; off >>= 1) v = fminf(v, __shfl_xor(v, off));
    return v;
}
__device__ __forceinline__ float half_max(float v) {
    for (int off = 16; off > 0; off >>= 1) v = fmaxf(v, __shfl_xor(v, off));
    return v;
}

// Points in curve order and the boxes of the leaves (fminf / fmaxf leave NaN
// coordinates out; a point that holds one is nobody's neighbour).
__global__ __launch_bounds__(256) void k_leaves(SceneDev sc, const uint32_t *__restrict__ sorted, int64_t padded,
                                                float4 *__restrict__ pts, NodeBox *__restrict__ leaf) {
    const int64_t p = (int64_t)blockIdx.x * 256 + threadIdx.x;
    if (p >= padded) return;            // (padded: a multiple of 64, so whole waves stay)
    float x[3] = {NAN, NAN, NAN};
    uint32_t i = 0xFFFFFFFFu;
    if (p < sc.n) {
        i = sorted[p];
        for (int c = 0; c < 3; ++c) x[c] = kload(sc.mean, c * sc.n + i, sc.format, false);
    }
    pts[p] = make_float4(x[0], x[1], x[2], __uint_as_float(i));
    NodeBox b;
    for (int c = 0; c < 3; ++c) {
        b.lo[c] = half_min(fminf(x[c], INFINITY));
        b.hi[c] = half_max(fmaxf(x[c], -INFINITY));
    }
    b.first = i;
    for (int off = 16; off > 0; off >>= 1) b.first = min(b.first, (uint32_t)__shfl_xor((int)b.first, off));
    b.pad = 0.0f;
    if ((threadIdx.x & (kLeaf - 1)) == 0) leaf[p / kLeaf] = b;
}

// One wave per node: the box of its (up to) 64 children.
__global__ __launch_bounds__(64) void k_nodes(const NodeBox *__restrict__ child, int nchild,
                                              NodeBox *__restrict__ node) {
    const int c = blockIdx.x * kFan + (int)threadIdx.x;
    NodeBox b;
    for (int k = 0; k < 3; ++k) {
        b.lo[k] = c < nchild ? child[c].lo[k] : INFINITY;
        b.hi[k] = c < nchild ? child[c].hi[k] : -INFINITY;
        b.lo[k] = half_min(b.lo[k]);
        b.hi[k] = half_max(b.hi[k]);
        b.lo[k] = fminf(b.lo[k], __shfl_xor(b.lo[k], 32));
        b.hi[k] = fmaxf(b.hi[k], __shfl_xor(b.hi[k], 32));
    }
    b.first = 0u;
    b.pad = 0.0f;
    if (threadIdx.x == 0) node[blockIdx.x] = b;
}

// Wave-wide minimum: a DPP scan (shifts by 1, 2, 4, 8 inside rows of 16 lanes,
// then row_bcast:15 and row_bcast:31; lanes without a source keep their value)
// leaves it in lane 63.
template <int kCtrl, int kRowMask>
__device__ __forceinline__ uint32_t dpp_min_step(uint32_t v) {
    return min(v, (uint32_t)__builtin_amdgcn_update_dpp(-1, (int)v, kCtrl, kRowMask, 0xF, false));
}
__device__ __forceinline__ uint32_t wave_min_bits(uint32_t v) {
    v = dpp_min_step<0x111, 0xF>(v);
    v = dpp_min_step<0x112, 0xF>(v);
    v = dpp_min_step<0x114, 0xF>(v);
    v = dpp_min_step<0x118, 0xF>(v);
    v = dpp_min_step<0x142, 0xA>(v);
    v = dpp_min_step<0x143, 0xC>(v);
    return (uint32_t)__builtin_amdgcn_readlane((int)v, 63);
}

// A neighbour is one 64-bit word, the bits of its float32 squared distance
// above its index: words order as (distance, index).  Read as doubles they are
// non-negative and never NaN (a float's bits up to infinity's, 0x7F800000, are
// a finite double's upper half), so one v_min_f64 / v_max_f64 compares two of
// them (denormal doubles are kept: FP64 denormals are on).
// Inserting word w into the ascending list b: b[k] = min(b[k], max(b[k-1], w))
// from the last to the first, in place (31 instructions, two temporaries; as
// separate statements the compiler holds all sixteen maxima at once, and the
// kernel spills).  The list's registers are written before the last input is read,
// so none of them may be an input's, which the compiler would share where it knows
// the values to be equal, as at the start: hence the early clobbers.
__device__ __forceinline__ void insert_word(double (&b)[16], double w) {
    double t0, t1;
    asm("v_max_f64 %8, %6, %11\n v_max_f64 %9, %5, %11\n v_min_f64 %7, %7, %8\n v_min_f64 %6, %6, %9\n"
        "v_max_f64 %8, %4, %11\n v_max_f64 %9, %3, %11\n v_min_f64 %5, %5, %8\n v_min_f64 %4, %4, %9\n"
        "v_max_f64 %8, %2, %11\n v_max_f64 %9, %1, %11\n v_min_f64 %3, %3, %8\n v_min_f64 %2, %2, %9\n"
        "v_max_f64 %8, %0, %11\n v_max_f64 %9, %10, %11\n v_min_f64 %1, %1, %8\n v_min_f64 %0, %0, %9\n"
        : "+&v"(b[8]), "+&v"(b[9]), "+&v"(b[10]), "+&v"(b[11]), "+&v"(b[12]), "+&v"(b[13]), "+&v"(b[14]),
          "+&v"(b[15]), "=&v"(t0), "=&v"(t1)
        : "v"(b[7]), "v"(w));
    asm("v_max_f64 %8, %6, %10\n v_max_f64 %9, %5, %10\n v_min_f64 %7, %7, %8\n v_min_f64 %6, %6, %9\n"
        "v_max_f64 %8, %4, %10\n v_max_f64 %9, %3, %10\n v_min_f64 %5, %5, %8\n v_min_f64 %4, %4, %9\n"
        "v_max_f64 %8, %2, %10\n v_max_f64 %9, %1, %10\n v_min_f64 %3, %3, %8\n v_min_f64 %2, %2, %9\n"
        "v_max_f64 %8, %0, %10\n v_min_f64 %0, %0, %10\n v_min_f64 %1, %1, %8\n"
        : "+&v"(b[0]), "+&v"(b[1]), "+&v"(b[2]), "+&v"(b[3]), "+&v"(b[4]), "+&v"(b[5]), "+&v"(b[6]), "+&v"(b[7]),
          "=&v"(t0), "=&v"(t1)
        : "v"(w));
}
__device__ __forceinline__ double word_of(float d2, uint32_t i) {
    return __hiloint2double((int)__float_as_uint(d2), (int)i);
}

struct Query {
    float x, y, z;
    uint32_t self;
    float kth;                      // 16th distance so far (below 0: the lane asks for nothing)
    double best[kK];                // ascending
};

// The 32 points of a leaf against every lane's query.  The points are wave
// uniform (scalar loads); a lane takes a candidate when it is no farther than
// its 16th so far, and the wave then shifts it into the lists with 31 FP64
// minima and maxima and no branches.
__device__ __forceinline__ bool search_leaf(const float4 *__restrict__ pts, int leaf, Query &q) {
    const float4 *__restrict__ P = pts + (int64_t)leaf * kLeaf;
    bool changed = false;
    // (the next four points load while these are compared)
    float4 o[4], nx[4];
#pragma unroll
    for (int u = 0; u < 4; ++u) nx[u] = P[u];
#pragma unroll 1
    for (int u0 = 0; u0 < kLeaf; u0 += 4) {
        const int un = min(u0 + 4, kLeaf - 4);
#pragma unroll
        for (int u = 0; u < 4; ++u) o[u] = nx[u];
#pragma unroll
        for (int u = 0; u < 4; ++u) nx[u] = P[un + u];
#pragma unroll
        for (int u = 0; u < 4; ++u) {
            const float ex = o[u].x - q.x, ey = o[u].y - q.y, ez = o[u].z - q.z;
            const float d2 = ex * ex + ey * ey + ez * ez;
            const uint32_t i = __float_as_uint(o[u].w);
            const bool take = d2 <= q.kth && i != q.self;     // (false for a NaN)
            if (__ballot(take) == 0ull) continue;
            changed = true;
            insert_word(q.best, word_of(take ? d2 : INFINITY, take ? i : 0xFFFFFFFFu));
            q.kth = q.kth < 0.0f ? q.kth : __uint_as_float((uint32_t)__double2hiint(q.best[kK - 1]));
        }
    }
    return changed;
}

// Squared distance from a box to a box (or a point): every operation rounds
// monotonically, in the order the candidates' squared distances are formed in,
// so no point inside the first box is nearer in float32 than this.
__device__ __forceinline__ float box_dist(const float *blo, const float *bhi, const float *qlo, const float *qhi) {
    float g[3];
#pragma unroll
    for (int c = 0; c < 3; ++c) g[c] = fmaxf(0.0f, fmaxf(blo[c] - qhi[c], qlo[c] - bhi[c]));
    return g[0] * g[0] + g[1] * g[1] + g[2] * g[2];
}

struct Walk {
    float qlo[3], qhi[3];     // box of the wave's queries
    float R;                  // the worst 16th distance of its queries
    int own;                  // its first own leaf (own and own + 1 are searched first)
};

// The lane's word for child c0 + lane of a level: the distance of its box with
// the lane in the low 6 bits (which only lowers it), or all ones for a child
// that is not there, too far or, among leaves, searched already.  One wave
// minimum then picks the nearest child.
// The common box of queries that lie on both sides of a jump of the curve, or
// far out, may hold most of the cloud: when more than kWide children pass it,
// each is held against every query by itself.  (Without this one wave in 15 625
// opened 22 016 leaves at 10^6 points, of which 552 were near a query, and the
// launch waited 11 ms for it.)
constexpr int kWide = 16;
__device__ __forceinline__ float lane_value(float v, int j) {
    return __uint_as_float((uint32_t)__builtin_amdgcn_readlane((int)__float_as_uint(v), j));
}
__device__ __forceinline__ uint32_t child_words(const NodeBox *__restrict__ box, int c0, int cnt, const Walk &w,
                                                const Query &q, bool leaves) {
    const int lane = threadIdx.x;
    NodeBox b = {};
    float d = INFINITY;
    bool near = false;
    if (lane < cnt) {
        b = box[c0 + lane];
        d = box_dist(b.lo, b.hi, w.qlo, w.qhi);
        near = !(d > w.R) && !(leaves && (unsigned)(c0 + lane - w.own) < 2u);
    }
    if (__popcll(__ballot(near)) > kWide) {
        bool some = false;
        d = INFINITY;
#pragma unroll 4
        for (int j = 0; j < 64; ++j) {
            const float at[3] = {lane_value(q.x, j), lane_value(q.y, j), lane_value(q.z, j)};
            const float dj = box_dist(b.lo, b.hi, at, at);
            const bool hit = !(dj > lane_value(q.kth, j));
            some = some || hit;
            d = hit ? fminf(d, dj) : d;
        }
        near = near && some;
    }
    return near ? (__float_as_uint(d) & ~63u) | (uint32_t)lane : 0xFFFFFFFFu;
}

__device__ __forceinline__ float worst_kth(const Query &q) {
    return __uint_as_float(~wave_min_bits(~__float_as_uint(fmaxf(q.kth, 0.0f))));
}

// One wave per 64 points of the curve.  What bounds it: VALU issue, about 10
// instructions per (candidate, wave) and 40 per candidate that some lane takes;
// at 10^6 clustered points a wave compares some 2 300 candidates, takes 330 and
// opens 150 leaves.  1.05 ms there; on a Morton curve 2.0 ms.  (A uniform grid
// with one lane per query, its list in registers behind branches, scanned
// thousands of candidates per query where clusters are dense: 5 to 10 ms.)
// kNeighbours: write the neighbour lists (indices and float32 squared
// distances, ordered by (distance, index)); else the neighbourhood features
// 59 .. 63 of each point, by index, for k_feature_rows.
template <bool kNeighbours, int kTop>
__global__ __launch_bounds__(64, 4) void k_knn(SceneDev sc, Tree T, float *__restrict__ nf, uint32_t *__restrict__ nidx,
                                            float *__restrict__ nd2) {
    const int lane = threadIdx.x;
    // consecutive waves of the curve on one XCD: they visit the same leaves
    const int nw = (int)((sc.n + 63) / 64), per = (nw + 7) >> 3;
    const int wv = (int)(blockIdx.x & 7) * per + (int)(blockIdx.x >> 3);
    if (wv >= nw) return;
    const int64_t p = (int64_t)wv * 64 + lane;
    const float4 me = T.pts[p];
    Query q;
    q.x = me.x;
    q.y = me.y;
    q.z = me.z;
    q.self = __float_as_uint(me.w);
    const bool asks = p < sc.n && me.x == me.x && me.y == me.y && me.z == me.z;
    q.kth = asks ? INFINITY : -1.0f;
#pragma unroll
    for (int k = 0; k < kK; ++k) q.best[k] = word_of(INFINITY, 0xFFFFFFFFu);
    Walk w;
    const float x[3] = {me.x, me.y, me.z};
#pragma unroll
    for (int c = 0; c < 3; ++c) {
        float lo = half_min(asks ? x[c] : INFINITY), hi = half_max(asks ? x[c] : -INFINITY);
        lo = fminf(lo, __shfl_xor(lo, 32));
        hi = fmaxf(hi, __shfl_xor(hi, 32));
        w.qlo[c] = __uint_as_float((uint32_t)__builtin_amdgcn_readfirstlane((int)__float_as_uint(lo)));
        w.qhi[c] = __uint_as_float((uint32_t)__builtin_amdgcn_readfirstlane((int)__float_as_uint(hi)));
    }
    w.own = 2 * wv;
    w.R = INFINITY;
    if (__ballot(asks) != 0ull) {
        // depth first, nearest child first: key[l] holds what is left of the
        // open node of level l (its children), first[l] its first child
        uint32_t key[kTop + 1];
        int first[kTop + 1], l = kTop, own = 0;
#pragma unroll
        for (int k = 0; k <= kTop; ++k) {
            key[k] = 0xFFFFFFFFu;
            first[k] = 0;
        }
        for (;;) {
            int leaf;
            if (own < 2) {
                leaf = w.own + own++;
            } else {
                if (own == 2) {
                    key[kTop] = child_words(T.box[kTop], 0, T.count[kTop], w, q, kTop == 0);
                    ++own;
                }
                leaf = -1;
                while (leaf < 0 && l <= kTop) {
#pragma unroll
                    for (int k = 0; k <= kTop; ++k) {
                        if (k != l) continue;
                        const uint32_t m = wave_min_bits(key[k]);
                        if (m == 0xFFFFFFFFu || __uint_as_float(m & ~63u) > w.R) {
                            l = k + 1;                    // nothing near is left here
                            break;
                        }
                        if (lane == (int)(m & 63u)) key[k] = 0xFFFFFFFFu;
                        const int c = first[k] + (int)(m & 63u);
                        if (k == 0) {
                            leaf = c;
                        } else {
                            constexpr int kDown = 0;
                            first[k > 0 ? k - 1 : kDown] = c * kFan;
                            key[k > 0 ? k - 1 : kDown] =
                                child_words(T.box[k > 0 ? k - 1 : kDown], c * kFan,
                                            min(kFan, T.count[k > 0 ? k - 1 : kDown] - c * kFan), w, q, k == 1);
                            l = k - 1;
                        }
                        break;
                    }
                }
                if (leaf < 0) break;
                const NodeBox b = T.box[0][leaf];
                const float at[3] = {q.x, q.y, q.z};
                // (ties of a larger index than the list's last stay out: among
                // coincident points or on a lattice whole leaves hold nothing else,
                // and each tie searched costs an insertion.  100 000 coincident
                // points: 24.4 ms with ties searched, 2.2 so)
                const float d = box_dist(b.lo, b.hi, at, at);
                const uint32_t last = (uint32_t)__double2loint(q.best[kK - 1]);
                if (__ballot(!(d > q.kth) && !(d == q.kth && b.first > last)) == 0ull) continue;
            }
            if (search_leaf(T.pts, leaf, q)) w.R = worst_kth(q);
        }
    }
    if (p >= sc.n) return;
    if (kNeighbours) {
#pragma unroll
        for (int k = 0; k < kK; ++k) {
            nidx[(int64_t)q.self * kK + k] = (uint32_t)__double2loint(q.best[k]);
            nd2[(int64_t)q.self * kK + k] = __uint_as_float((uint32_t)__double2hiint(q.best[k]));
        }
        return;
    }
    int cnt = 0;
    float sd = 0.0f, sa = 0.0f, ma = 0.0f, last = 0.0f;
#pragma unroll
    for (int k = 0; k < kK; ++k) {
        const uint32_t i = (uint32_t)__double2loint(q.best[k]);
        if (i == 0xFFFFFFFFu) continue;
        const float d2 = __uint_as_float((uint32_t)__double2hiint(q.best[k]));
        const float al = kload(sc.opacity, i, sc.format, true);
        ++cnt;
        last = d2;
        sd += sqrtf(d2);
        sa += al;
        ma = fmaxf(ma, al);
    }
    const float d16 = cnt ? sqrtf(last) : 1.0f;
    const float tiny = 1e-12f;
    float4 f;
    f.x = logf(fmaxf(cnt ? sd / cnt : 1.0f, tiny));
    f.y = logf(fmaxf(d16, tiny));
    f.z = cnt ? sa / cnt : 0.0f;
    f.w = ma;
    float *row = nf + (int64_t)q.self * 8;
    *reinterpret_cast<float4 *>(row) = f;
    row[4] = logf(fmaxf(sa, tiny) / fmaxf(4.18879020f * d16 * d16 * d16, tiny));
}

// The feature rows, 64 points per block: the attribute planes are read in
// index order (a wave reads 64 consecutive values of a plane), transposed in
// LDS (65 floats per row: no bank conflicts) and stored as whole rows: 0.12 ms
// for 10^6 points, 4.3 TB/s.  (Assembled by the search itself, at scattered
// indices, a row takes a whole line of every plane for each 4 bytes.)
typedef float f32x4u __attribute__((ext_vector_type(4), aligned(4)));
__global__ __launch_bounds__(256) void k_feature_rows(SceneDev sc, const float *__restrict__ nf,
                                                      float *__restrict__ feat) {
    constexpr int kRows = 64, kPitch = kMlpIn + 1;
    __shared__ float sh[kRows * kPitch];
    const int64_t n = sc.n, r0 = (int64_t)blockIdx.x * kRows;
    const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
    const int64_t i = r0 + lane;
    const bool ok = i < n;
    float *row = sh + lane * kPitch;
    const int K = (sc.sh_degree + 1) * (sc.sh_degree + 1);
#pragma unroll 4
    for (int k = w; k < 48; k += 4)
        row[11 + k] = (ok && k < 3 * K) ? kload(sc.sh, (int64_t)k * n + i, sc.format, false) : 0.0f;
    if (ok) {
        if (w == 0) {
            for (int c = 0; c < 3; ++c) row[c] = kload(sc.mean, c * n + i, sc.format, false);
            for (int c = 0; c < 3; ++c) row[3 + c] = kload(sc.log_scale, c * n + i, sc.format, false);
        } else if (w == 1) {
            float qq[4], qn = 0.0f;
#pragma unroll
            for (int c = 0; c < 4; ++c) {
                qq[c] = kload(sc.quat, c * n + i, sc.format, true);
                qn += qq[c] * qq[c];
            }
            const float qs = (qq[0] < 0.0f ? -1.0f : 1.0f) * rsqrtf(fmaxf(qn, 1e-30f));
#pragma unroll
            for (int c = 0; c < 4; ++c) row[6 + c] = qq[c] * qs;
        } else if (w == 2) {
            const float al = fminf(fmaxf(kload(sc.opacity, i, sc.format, true), 1e-6f), 1.0f - 1e-6f);
            row[10] = logf(al / (1.0f - al));
        } else {
            const float4 f = *reinterpret_cast<const float4 *>(nf + i * 8);
            row[59] = f.x;
            row[60] = f.y;
            row[61] = f.z;
            row[62] = f.w;
            row[63] = nf[i * 8 + 4];
        }
    }
    __syncthreads();
    for (int t = threadIdx.x; t < kRows * (kMlpIn / 4); t += 256) {
        const int r = t >> 4, c = 4 * (t & 15);
        if (r0 + r < n) {
            const float *v = sh + r * kPitch + c;
            const f32x4u o = {v[0], v[1], v[2], v[3]};
            *reinterpret_cast<f32x4u *>(feat + (r0 + r) * kMlpIn + c) = o;
        }
    }
}

// Column means and 1/std (population) of an n x 64 float32 matrix, in FP64.
// Bound by reading the matrix once.  A block takes kStatRows consecutive rows:
// thread t reads the four columns 4 (t mod 16) .. + 3 of rows t / 16, t / 16 +
// 16, ... as one float4, so a wave reads 1 KiB of consecutive memory per load,
// and the block's sums go to its own slot; a second launch adds the slots in
// block order (fixed, so the result is deterministic).  With one block per
// column, every block read every 256-byte row for 4 bytes of it and only 64
// of the 256 CUs worked: 2.17 ms for 10^6 rows (features and their statistics
// together 7.58 -> 5.39 ms).
// (The rows are only known to be 4-byte aligned: f32x4u says so.)
constexpr int kStatRows = 1024;
static int64_t stat_blocks(int64_t n) { return (n + kStatRows - 1) / kStatRows; }
size_t feature_stats_scratch_bytes(int64_t n) { return sizeof(double) * 2 * kMlpIn * (size_t)stat_blocks(n) + 256; }

__global__ __launch_bounds__(256) void k_feature_sums(const float *__restrict__ feat, int64_t n,
                                                      double *__restrict__ part) {
    __shared__ double sh[16][2 * kMlpIn];
    const int cg = threadIdx.x & 15, rg = threadIdx.x >> 4;
    const int64_t lo = (int64_t)blockIdx.x * kStatRows, hi = min(lo + (int64_t)kStatRows, n);
    double a[4] = {0, 0, 0, 0}, b[4] = {0, 0, 0, 0};
#pragma unroll 4
    for (int64_t r = lo + rg; r < hi; r += 16) {
        const f32x4u v = *reinterpret_cast<const f32x4u *>(feat + r * kMlpIn + 4 * cg);
        const double x[4] = {v.x, v.y, v.z, v.w};
#pragma unroll
        for (int k = 0; k < 4; ++k) {
            a[k] += x[k];
            b[k] += x[k] * x[k];
        }
    }
#pragma unroll
    for (int k = 0; k < 4; ++k) {
        sh[rg][4 * cg + k] = a[k];
        sh[rg][kMlpIn + 4 * cg + k] = b[k];
    }
    __syncthreads();
    if (threadIdx.x < 2 * kMlpIn) {
        double s = 0.0;
        for (int k = 0; k < 16; ++k) s += sh[k][threadIdx.x];
        part[(int64_t)blockIdx.x * (2 * kMlpIn) + threadIdx.x] = s;
    }
}

// One block per column: thread t adds the slots t, t + 256, ... in order, then
// a fixed tree.
__global__ __launch_bounds__(256) void k_feature_norm(const double *__restrict__ part, int64_t nblk, int64_t n,
                                                      float *__restrict__ norm) {
    __shared__ double s1[256], s2[256];
    const int c = blockIdx.x;
    double a = 0.0, b = 0.0;
    for (int64_t r = threadIdx.x; r < nblk; r += 256) {
        a += part[r * (2 * kMlpIn) + c];
        b += part[r * (2 * kMlpIn) + kMlpIn + c];
    }
    s1[threadIdx.x] = a;
    s2[threadIdx.x] = b;
    __syncthreads();
    for (int o = 128; o > 0; o >>= 1) {
        if (threadIdx.x < o) {
            s1[threadIdx.x] += s1[threadIdx.x + o];
            s2[threadIdx.x] += s2[threadIdx.x + o];
        }
        __syncthreads();
    }
    if (threadIdx.x == 0) {
        const double mean = s1[0] / (double)n;
        const double var = fmax(s2[0] / (double)n - mean * mean, 0.0);
        norm[c] = (float)mean;
        norm[kMlpIn + c] = var > 1e-20 ? (float)(1.0 / sqrt(var)) : 1.0f;
    }
}

void feature_stats(const float *feat, int64_t n, float *norm, void *scratch, hipStream_t st) {
    double *part = (double *)scratch;
    const int64_t nblk = stat_blocks(n);
    hipLaunchKernelGGL(k_feature_sums, dim3((unsigned)nblk), dim3(256), 0, st, feat, n, part);
    hipLaunchKernelGGL(k_feature_norm, dim3(kMlpIn), dim3(256), 0, st, part, nblk, n, norm);
}

// Levels of the tree over n points: leaves, then 64 nodes per node until at
// most 64 are left.
static int tree_levels(int64_t n, int64_t (&count)[kMaxLevels]) {
    int top = 0;
    count[0] = (n + kLeaf - 1) / kLeaf;
    while (count[top] > kFan) {
        count[top + 1] = (count[top] + kFan - 1) / kFan;
        ++top;
    }
    return top;
}

size_t knn_scratch_bytes(int64_t n) {
    int64_t count[kMaxLevels];
    const int top = tree_levels(n, count);
    size_t b = (size_t)4 * 4 * n + sizeof(uint32_t) * (size_t)radix_sort_scratch_words(n, 1);   // codes and values, twice
    b += (size_t)(n + 64) * 16 + (size_t)n * 32;                                                 // points, features 59-63
    for (int l = 0; l <= top; ++l) b += sizeof(NodeBox) * (size_t)(count[l] + 2);
    return b + 64 * 256;
}

template <bool kNeighbours>
static void launch_knn(int top, const SceneDev &sc, const Tree &T, float *nf, uint32_t *nidx, float *nd2,
                       hipStream_t st) {
    const unsigned grid = (unsigned)(((sc.n + 63) / 64 + 7) / 8 * 8);
    auto go = [&](auto kernel) { hipLaunchKernelGGL(kernel, dim3(grid), dim3(64), 0, st, sc, T, nf, nidx, nd2); };
    switch (top) {
        case 0: go(k_knn<kNeighbours, 0>); break;
        case 1: go(k_knn<kNeighbours, 1>); break;
        case 2: go(k_knn<kNeighbours, 2>); break;
        default: go(k_knn<kNeighbours, 3>); break;      // n < 2^28: at most 2^23 leaves
    }
}

hipError_t knn_features(const SceneDev &sc, float *feat, void *scratch, hipStream_t st, uint32_t *nidx,
                        float *nd2) {
    const int64_t n = sc.n;
    char *p = (char *)scratch;
    size_t o = 0;
    auto take = [&](size_t bytes) {
        o = (o + 255) & ~(size_t)255;
        void *r = p + o;
        o += bytes;
        return r;
    };
    CloudStats *cs = (CloudStats *)take(sizeof(CloudStats));
    uint32_t *key0 = (uint32_t *)take((size_t)n * 4), *key1 = (uint32_t *)take((size_t)n * 4);
    uint32_t *val0 = (uint32_t *)take((size_t)n * 4), *val1 = (uint32_t *)take((size_t)n * 4);
    uint32_t *hist = (uint32_t *)take(sizeof(uint32_t) * (size_t)radix_sort_scratch_words(n, 1));
    const int64_t padded = (n + 63) / 64 * 64;
    float4 *pts = (float4 *)take((size_t)padded * 16);
    float *nf = (float *)take((size_t)n * 32);
    int64_t count[kMaxLevels];
    const int top = tree_levels(n, count);
    Tree T{};
    T.pts = pts;
    NodeBox *box[kMaxLevels] = {};
    for (int l = 0; l <= top; ++l) {
        T.box[l] = box[l] = (NodeBox *)take(sizeof(NodeBox) * (size_t)(count[l] + 2));
        T.count[l] = (int)count[l];
    }
    const unsigned per256 = (unsigned)((n + 255) / 256);
    hipLaunchKernelGGL(k_cloud_init, dim3(1), dim3(1), 0, st, cs);
    hipLaunchKernelGGL(k_cloud_stats, dim3(std::min(per256, (unsigned)kBoxBlocks)), dim3(256), 0, st, sc, cs);
    hipLaunchKernelGGL(k_curve, dim3(per256), dim3(256), 0, st, sc, (const CloudStats *)cs, key0);
    uint32_t *ko = nullptr, *sorted = nullptr;
    const hipError_t e =
        radix_sort_segments(key0, val0, key1, val1, hist, n, 1, true, 4, nullptr, nullptr, &ko, &sorted, st);
    if (e != hipSuccess) return e;
    hipLaunchKernelGGL(k_leaves, dim3((unsigned)((padded + 255) / 256)), dim3(256), 0, st, sc,
                       (const uint32_t *)sorted, padded, pts, box[0]);
    for (int l = 1; l <= top; ++l)
        hipLaunchKernelGGL(k_nodes, dim3((unsigned)count[l]), dim3(64), 0, st, (const NodeBox *)box[l - 1],
                           (int)count[l - 1], box[l]);
    if (nidx) {
        launch_knn<true>(top, sc, T, nullptr, nidx, nd2, st);
    } else {
        launch_knn<false>(top, sc, T, nf, nullptr, nullptr, st);
        hipLaunchKernelGGL(k_feature_rows, dim3((unsigned)((n + 63) / 64)), dim3(256), 0, st, sc, (const float *)nf,
                           feat);
    }
    return hipGetLastError();
}

}  // namespace gs
