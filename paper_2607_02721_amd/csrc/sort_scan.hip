// Segmented LSD radix sort of (u32 key, u32 value) pairs, exclusive prefix
// sums, fills and a fixed-order float sum.
//
// Radix sort: each of n_segs segments of n_per_seg items (one segment per
// view) is sorted independently and stably by key, 8 bits per pass, 3 or 4
// passes (3 when every segment's keys, minus the segment's smallest, fit in
// 24 bits).  Blocks never straddle segments.  Once, before the passes:
//   hist_all:   every pass's digit counts per segment (one read of the keys)
//   digit_base: per segment and pass, exclusive scan of the digit counts
// Per pass:
//   scatter: each wave ranks its 1024 keys in 16 rounds of 64 with ballot
//            matching (wave-private LDS digit counters, so no block barrier
//            inside the rounds); waves then add the counts of the waves
//            before them, which keeps the sort stable; the block's start in
//            each digit's run is the digit base plus the counts of the
//            segment's earlier blocks, found by decoupled look-back.
// Segments of one block (4096 items) or less: every pass in one launch.
#include "gs_internal.hpp"

namespace gs {

constexpr int kSortThreads = 256;
constexpr int kSortRounds = kSortTile / kSortThreads;  // 16

__device__ __forceinline__ uint64_t lanemask_lt() {
    const unsigned lane = threadIdx.x & 63;
    return lane == 0 ? 0ull : (~0ull >> (64 - lane));
}

// Lanes (among `active`) holding the same 8-bit digit as this lane.
__device__ __forceinline__ uint64_t match_digit(uint32_t d, uint64_t active) {
    uint64_t m = active;
#pragma unroll
    for (int b = 0; b < 8; ++b) {
        const uint64_t bal = __ballot((d >> b) & 1u);
        m &= ((d >> b) & 1u) ? bal : ~bal;
    }
    return m;
}

// Key as the pass sees it: with kbase, visible keys relative to their
// segment's smallest one (first pass only; later passes read rebased keys).
__device__ __forceinline__ uint32_t rebase(uint32_t k, const uint32_t *kbase, int seg) {
    return (kbase && k != kInvisibleKey) ? k - kbase[seg] : k;
}

// Inclusive DPP scan of a wave (lanes without a source add 0).
__device__ __forceinline__ uint32_t wave_incl_scan_u32(uint32_t v) {
    v += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0x111, 0xF, 0xF, false);
    v += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0x112, 0xF, 0xF, false);
    v += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0x114, 0xF, 0xF, false);
    v += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0x118, 0xF, 0xF, false);
    v += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0x142, 0xA, 0xF, false);
    v += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0x143, 0xC, 0xF, false);
    return v;
}

// Single-sweep form (look-back): one histogram kernel counts every pass's
// digits of the segment up front; each pass's scatter then takes its block
// number from a per-segment ticket, publishes its digit counts and sums
// those of the blocks before it (decoupled look-back), so no per-block
// histogram or offsets scan runs between the passes.
// Scratch after the status words, per segment: [4 passes][256] counts,
// [4][256] exclusive digit bases, [4] tickets (kSweepExtra words).
constexpr int kSweepExtra = 4 * 256 * 2 + 4;
// A status word is flag << 30 | pass << 28 | count (segments hold fewer than 2^28
// items): a word of an earlier pass counts as not yet written, so the words are
// cleared once for all passes.
constexpr uint32_t kFlagAgg = 1u << 30, kFlagPrefix = 2u << 30, kCountMask = (1u << 28) - 1u;
constexpr int kPassShift = 28;

// Sort tiles per histogram block: its counts go to the segment's by one atomic
// per digit and pass, so a large sort takes several tiles per block (100
// segments of 1M keys: 1 tile 180 us, 4 tiles 147, 8 tiles 157; keys loaded one at
// a time 217), a small one, which would leave CUs idle, one.
constexpr int kHistTiles = 4;
constexpr int64_t kHistManyTiles = 8192;
__global__ __launch_bounds__(kSortThreads) void k_radix_hist_all(const uint32_t *__restrict__ keys,
                                                                  int64_t n_per_seg, int passes,
                                                                  uint32_t *__restrict__ extra,
                                                                  const uint32_t *__restrict__ kbase,
                                                                  const uint32_t *__restrict__ seg_len, int tiles) {
    __shared__ uint32_t cnt[4][256];
    const int seg = blockIdx.y, b = blockIdx.x;
    for (int i = threadIdx.x; i < 4 * 256; i += kSortThreads) (&cnt[0][0])[i] = 0;
    __syncthreads();
    const int64_t base = (int64_t)seg * n_per_seg;
    const int64_t len = seg_len ? (int64_t)seg_len[seg] : n_per_seg;
    const int64_t lo = (int64_t)b * tiles * kSortTile;
    const int64_t hi = min(lo + (int64_t)tiles * kSortTile, len);
    for (int64_t i = lo + threadIdx.x; i < hi; i += 8 * kSortThreads) {
        uint32_t k[8];
#pragma unroll
        for (int u = 0; u < 8; ++u) k[u] = i + u * kSortThreads < hi ? keys[base + i + u * kSortThreads] : 0u;
#pragma unroll
        for (int u = 0; u < 8; ++u)
            if (i + u * kSortThreads < hi) {
                const uint32_t x = rebase(k[u], kbase, seg);
                for (int p = 0; p < passes; ++p) atomicAdd(&cnt[p][(x >> (8 * p)) & 255u], 1u);
            }
    }
    __syncthreads();
    uint32_t *gc = extra + (int64_t)seg * kSweepExtra;
    for (int p = 0; p < passes; ++p) {
        const uint32_t c = cnt[p][threadIdx.x];
        if (c) atomicAdd(&gc[p * 256 + threadIdx.x], c);
    }
}

// One block of 256 threads per segment: exclusive scan of each pass's digit
// counts into the digit bases; the tickets are cleared here too.
__global__ __launch_bounds__(256) void k_radix_digit_base(uint32_t *__restrict__ extra, int passes) {
    __shared__ uint32_t wsum[4];
    uint32_t *e = extra + (int64_t)blockIdx.x * kSweepExtra;
    const int d = threadIdx.x, w = d >> 6, lane = d & 63;
    for (int p = 0; p < passes; ++p) {
        const uint32_t c = e[p * 256 + d];
        const uint32_t incl = wave_incl_scan_u32(c);
        if (lane == 63) wsum[w] = incl;
        __syncthreads();
        uint32_t before = incl - c;
        for (int k = 0; k < 3; ++k) before += k < w ? wsum[k] : 0u;
        e[4 * 256 + p * 256 + d] = before;
        __syncthreads();
    }
    if (d < 4) e[8 * 256 + d] = 0u;
}

// What bounds it is latency (a tile's loads, 16 rounds of ranking, the look-back,
// then its stores), so it lives on the blocks a CU holds: the keys and then the
// values leave through one 16 KB buffer, which with 72 registers makes seven
// blocks (through a buffer each, four: 662 us per pass at 100 segments of 1M keys,
// 473 so; 20 segments of 248k 42 and 31).  Looking back at four blocks at a time
// brought nothing (731).
__global__ __launch_bounds__(kSortThreads, 7) void k_radix_scatter(const uint32_t *__restrict__ kin,
                                                                 const uint32_t *__restrict__ vin,
                                                                 uint32_t *__restrict__ kout,
                                                                 uint32_t *__restrict__ vout, int64_t n_per_seg,
                                                                 int nb, int shift, int vals_are_iota,
                                                                 const uint32_t *__restrict__ kbase,
                                                                 const uint32_t *__restrict__ seg_len,
                                                                 uint32_t *__restrict__ status,
                                                                 uint32_t *__restrict__ extra, int pass,
                                                                 int n_segs) {
    // per wave and digit: the wave's count while ranking, then (thread d
    // rewrites its own column once it has read it) the block-local start of
    // the wave's run of digit d
    __shared__ uint32_t wcnt[4][256];
    uint32_t (*wbase)[256] = wcnt;
    __shared__ uint32_t dstart[256];     // block-local start of each digit
    __shared__ uint32_t gdst[256];       // global start of the block's run of each digit
    __shared__ uint32_t wsum4[4];        // digit counts of each wave's 64 digits
    __shared__ uint32_t stage[kSortTile];   // the keys on their way out, then the values
    __shared__ int tick;
    // blocks go to the XCDs in turn (block i to XCD i mod 8): block i works
    // on segment 8 (i / 8 / nb) + i mod 8, so each segment's scattered lines
    // are written through one L2; its place in the segment is its ticket.
    // The last n_segs mod 8 segments are shared by every XCD instead (one XCD
    // each would leave the others idle at the end: a sort of one segment ran
    // on an eighth of the chip).
    const int64_t bi = blockIdx.x, whole = (int64_t)nb * (n_segs & ~7);
    const int seg = bi < whole ? (int)(((bi >> 3) / nb) * 8 + (bi & 7)) : (n_segs & ~7) + (int)((bi - whole) / nb);
    if (seg >= n_segs) return;
    int b;
    const int w = threadIdx.x >> 6, lane = threadIdx.x & 63;
    uint32_t *ex = extra + (int64_t)seg * kSweepExtra;
    // block number in the order the segment's blocks started: every block
    // this one waits for below has started and publishes its counts before
    // it waits for anything
    if (threadIdx.x == 0) tick = (int)atomicAdd(&ex[8 * 256 + pass], 1u);
    __syncthreads();
    b = tick;
    // items of the segment to sort (the whole block leaves if it holds none)
    const int64_t len = seg_len ? (int64_t)seg_len[seg] : n_per_seg;
    if ((int64_t)b * kSortTile >= len) return;
    const int64_t base = (int64_t)seg * n_per_seg;
    const int64_t wlo = (int64_t)b * kSortTile + (int64_t)w * (kSortRounds * 64);
    uint32_t key[kSortRounds], val[kSortRounds], rank[kSortRounds];
#pragma unroll
    for (int k = 0; k < kSortRounds; ++k) {
        const int64_t i = wlo + k * 64 + lane;
        key[k] = i < len ? kin[base + i] : 0u;
    }
#pragma unroll
    for (int k = 0; k < kSortRounds; ++k) {
        const int64_t i = wlo + k * 64 + lane;
        val[k] = i < len ? (vals_are_iota ? (uint32_t)i : vin[base + i]) : 0u;
    }
    for (int i = threadIdx.x; i < 4 * 256; i += kSortThreads) (&wcnt[0][0])[i] = 0;
    __syncthreads();
#pragma unroll
    for (int k = 0; k < kSortRounds; ++k) {
        const int64_t i = wlo + k * 64 + lane;
        const bool ok = i < len;
        if (ok) key[k] = rebase(key[k], kbase, seg);
        const uint32_t d = (key[k] >> shift) & 255u;
        const uint64_t active = __ballot(ok);
        const uint64_t peers = match_digit(d, active);
        const uint32_t before = (uint32_t)__popcll(peers & lanemask_lt());
        const uint32_t run = ok ? wcnt[w][d] : 0u;
        rank[k] = run + before;
        // the last peer advances the wave's counter for this digit
        if (ok && (peers >> lane) == 1ull) wcnt[w][d] = run + before + 1u;
        __builtin_amdgcn_wave_barrier();
    }
    __syncthreads();
    // digit counts of the block, their exclusive scan (block-local run
    // starts) and each wave's start inside its digit's run
    {
        const int d = threadIdx.x;
        const uint32_t c0 = wcnt[0][d], c1 = wcnt[1][d], c2 = wcnt[2][d], c3 = wcnt[3][d];
        const uint32_t tot = c0 + c1 + c2 + c3;
        {
            // publish this block's count of digit d, then add up the counts
            // of the blocks before it back to one that published its prefix
            uint32_t *st = status + (int64_t)seg * nb * 256;
            const uint32_t tag = (uint32_t)pass << kPassShift;
            uint32_t excl = 0;
            if (b == 0) {
                __hip_atomic_store(&st[d], kFlagPrefix | tag | tot, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            } else {
                __hip_atomic_store(&st[(int64_t)b * 256 + d], kFlagAgg | tag | tot, __ATOMIC_RELAXED,
                                   __HIP_MEMORY_SCOPE_AGENT);
                for (int j = b - 1;; --j) {
                    uint32_t v = 0;
                    // (bounded: the block waited for has started; the bound only
                    // keeps a broken invariant from hanging the device)
                    for (int spin = 0; spin < (1 << 24); ++spin) {
                        v = __hip_atomic_load(&st[(int64_t)j * 256 + d], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
                        if (v >= kFlagAgg && ((v >> kPassShift) & 3u) == (uint32_t)pass) break;
                        __builtin_amdgcn_s_sleep(1);
                    }
                    excl += v & kCountMask;
                    if ((v & kFlagPrefix) || j == 0) break;
                }
                __hip_atomic_store(&st[(int64_t)b * 256 + d], kFlagPrefix | tag | (excl + tot), __ATOMIC_RELAXED,
                                   __HIP_MEMORY_SCOPE_AGENT);
            }
            gdst[d] = ex[4 * 256 + pass * 256 + d] + excl;
        }
        // digits 64w .. 64w+63 are wave w's lanes: a DPP scan per wave, then
        // the sums of the waves before
        const uint32_t incl = wave_incl_scan_u32(tot);
        if (lane == 63) wsum4[w] = incl;
        __syncthreads();
        uint32_t start = incl - tot;
#pragma unroll
        for (int k = 0; k < 3; ++k) start += k < w ? wsum4[k] : 0u;
        dstart[d] = start;
        wbase[0][d] = start;
        wbase[1][d] = start + c0;
        wbase[2][d] = start + c0 + c1;
        wbase[3][d] = start + c0 + c1 + c2;
    }
    __syncthreads();
    // the block's keys, then its values, in LDS in stable digit order, written
    // out in that order: consecutive threads store consecutive positions of each
    // digit's run, so the stores of a wave cover a few runs instead of 64
    // scattered words
    const int nvalid = (int)min((int64_t)kSortTile, len - (int64_t)b * kSortTile);
#pragma unroll
    for (int k = 0; k < kSortRounds; ++k) {
        const int64_t i = wlo + k * 64 + lane;
        if (i < len) {
            rank[k] += wbase[w][(key[k] >> shift) & 255u];
            stage[rank[k]] = key[k];
        }
    }
    __syncthreads();
    uint32_t dst[kSortRounds];
#pragma unroll
    for (int k = 0; k < kSortRounds; ++k) {
        const int i = k * kSortThreads + threadIdx.x;
        if (i < nvalid) {
            const uint32_t kk = stage[i], d = (kk >> shift) & 255u;
            dst[k] = gdst[d] + ((uint32_t)i - dstart[d]);
            if (kout) kout[base + dst[k]] = kk;
        }
    }
    __syncthreads();
#pragma unroll
    for (int k = 0; k < kSortRounds; ++k)
        if (wlo + k * 64 + lane < len) stage[rank[k]] = val[k];
    __syncthreads();
#pragma unroll
    for (int k = 0; k < kSortRounds; ++k) {
        const int i = k * kSortThreads + threadIdx.x;
        if (i < nvalid) vout[base + dst[k]] = stage[i];
    }
}

// Segments of one tile or less: every pass in one block, keys and values in LDS
// between the passes.  (The general form is a chain of launches, each a chain of
// latencies: 4 segments of 2000 keys took 48 us in six launches, 10 so.)
// Wave w holds `rounds` runs of 64 neighbouring items, so that its ranks by
// ballots follow the order of the items, as in k_radix_scatter.
constexpr int kSmallThreads = 1024, kSmallWaves = kSmallThreads / 64, kSmallRounds = kSortTile / kSmallThreads;
__global__ __launch_bounds__(kSmallThreads) void k_sort_small(const uint32_t *__restrict__ kin,
                                                              const uint32_t *__restrict__ vin,
                                                              uint32_t *__restrict__ vout, int64_t n_per_seg,
                                                              int passes, const uint32_t *__restrict__ kbase,
                                                              const uint32_t *__restrict__ seg_len) {
    __shared__ uint32_t wcnt[kSmallWaves][256], dstart[256], wsum4[4];
    __shared__ uint32_t skey[kSortTile], sval[kSortTile];
    const int seg = blockIdx.x, w = threadIdx.x >> 6, lane = threadIdx.x & 63;
    const int len = (int)(seg_len ? (int64_t)seg_len[seg] : n_per_seg);
    const int64_t base = (int64_t)seg * n_per_seg;
    const int rounds = (len + kSmallThreads - 1) / kSmallThreads, wlo = w * rounds * 64;
    uint32_t key[kSmallRounds], val[kSmallRounds], rank[kSmallRounds];
#pragma unroll
    for (int k = 0; k < kSmallRounds; ++k) {
        const int i = wlo + k * 64 + lane;
        const bool ok = k < rounds && i < len;
        key[k] = ok ? rebase(kin[base + i], kbase, seg) : 0u;
        val[k] = ok ? (vin ? vin[base + i] : (uint32_t)i) : 0u;
    }
    for (int pass = 0; pass < passes; ++pass) {
        const int shift = 8 * pass;
        for (int i = threadIdx.x; i < kSmallWaves * 256; i += kSmallThreads) (&wcnt[0][0])[i] = 0u;
        __syncthreads();
#pragma unroll
        for (int k = 0; k < kSmallRounds; ++k) {
            if (k >= rounds) break;
            const bool ok = wlo + k * 64 + lane < len;
            const uint32_t d = (key[k] >> shift) & 255u;
            const uint64_t peers = match_digit(d, __ballot(ok));
            const uint32_t before = (uint32_t)__popcll(peers & lanemask_lt());
            const uint32_t run = ok ? wcnt[w][d] : 0u;
            rank[k] = run + before;
            if (ok && (peers >> lane) == 1ull) wcnt[w][d] = run + before + 1u;
            __builtin_amdgcn_wave_barrier();
        }
        __syncthreads();
        // digit starts: over the waves, then over the digits
        uint32_t tot = 0u, incl = 0u;
        if (threadIdx.x < 256) {
            for (int q = 0; q < kSmallWaves; ++q) {
                const uint32_t c = wcnt[q][threadIdx.x];
                wcnt[q][threadIdx.x] = tot;
                tot += c;
            }
            incl = wave_incl_scan_u32(tot);
            if (lane == 63) wsum4[w] = incl;
        }
        __syncthreads();
        if (threadIdx.x < 256) {
            uint32_t start = incl - tot;
            for (int q = 0; q < w; ++q) start += wsum4[q];
            dstart[threadIdx.x] = start;
        }
        __syncthreads();
#pragma unroll
        for (int k = 0; k < kSmallRounds; ++k)
            if (k < rounds && wlo + k * 64 + lane < len) {
                const uint32_t d = (key[k] >> shift) & 255u;
                const uint32_t pos = dstart[d] + wcnt[w][d] + rank[k];
                skey[pos] = key[k];
                sval[pos] = val[k];
            }
        __syncthreads();
#pragma unroll
        for (int k = 0; k < kSmallRounds; ++k) {
            const int i = wlo + k * 64 + lane;
            if (k < rounds && i < len) {
                key[k] = skey[i];
                val[k] = sval[i];
            }
        }
    }
#pragma unroll
    for (int k = 0; k < kSmallRounds; ++k) {
        const int i = wlo + k * 64 + lane;
        if (k < rounds && i < len) vout[base + i] = val[k];
    }
}

hipError_t radix_sort_segments(uint32_t *key0, uint32_t *val0, uint32_t *key1, uint32_t *val1, uint32_t *hist,
                               int64_t n_per_seg, int n_segs, bool vals_are_iota, int passes,
                               const uint32_t *kbase, const uint32_t *seg_len, uint32_t **key_out,
                               uint32_t **val_out, hipStream_t st) {
    if (n_per_seg <= kSortTile) {
        hipLaunchKernelGGL(k_sort_small, dim3((unsigned)n_segs), dim3(kSmallThreads), 0, st, key0,
                           vals_are_iota ? nullptr : val0, val1, n_per_seg, passes, kbase, seg_len);
        *key_out = nullptr;
        *val_out = val1;
        return hipGetLastError();
    }
    const int nb = (int)((n_per_seg + kSortTile - 1) / kSortTile);
    uint32_t *ki = key0, *vi = val0, *ko = key1, *vo = val1;
    // hist: [n_segs][256][nb] status words, then kSweepExtra words per segment
    const int64_t nstatus = (int64_t)n_segs * 256 * nb;
    uint32_t *extra = hist + nstatus;
    launch_fill_u32(hist, 0u, nstatus + (int64_t)n_segs * kSweepExtra, st);
    const int tiles = (int64_t)nb * n_segs >= kHistManyTiles ? kHistTiles : 1;
    hipLaunchKernelGGL(k_radix_hist_all, dim3((nb + tiles - 1) / tiles, n_segs), dim3(kSortThreads), 0, st, key0,
                       n_per_seg, passes, extra, kbase, seg_len, tiles);
    hipLaunchKernelGGL(k_radix_digit_base, dim3(n_segs), dim3(256), 0, st, extra, passes);
    for (int pass = 0; pass < passes; ++pass) {
        const int shift = 8 * pass;
        const uint32_t *kb = pass == 0 ? kbase : nullptr;
        // the last pass writes the values only (nothing reads the sorted keys)
        const int64_t blocks = (int64_t)nb * n_segs;
        hipLaunchKernelGGL(k_radix_scatter, dim3((unsigned)blocks), dim3(kSortThreads), 0, st, ki, vi,
                           pass + 1 < passes ? ko : nullptr, vo, n_per_seg, nb, shift,
                           (pass == 0 && vals_are_iota) ? 1 : 0, kb, seg_len, hist, extra, pass, n_segs);
        uint32_t *t = ki; ki = ko; ko = t;
        t = vi; vi = vo; vo = t;
    }
    *key_out = nullptr;
    *val_out = vi;
    return hipGetLastError();
}

int64_t radix_sort_scratch_words(int64_t n_per_seg, int n_segs) {
    const int64_t nb = (n_per_seg + kSortTile - 1) / kSortTile;
    return (int64_t)n_segs * (256 * nb + kSweepExtra);
}

// ---------------------------------------------------------------------------
// Exclusive prefix sums of u32 in u64, three phases with 2048-item blocks.
constexpr int kScanThreads = 256;
constexpr int kScanItems = 8;
constexpr int kScanBlock = kScanThreads * kScanItems;

int64_t scan_tmp_elems(int64_t n) { return (n + kScanBlock - 1) / kScanBlock + 1; }

__device__ __forceinline__ uint64_t block_exclusive_scan(uint64_t v, uint64_t *sh, uint64_t *total) {
    // sh: kScanThreads entries
    const int t = threadIdx.x;
    sh[t] = v;
    __syncthreads();
    for (int off = 1; off < kScanThreads; off <<= 1) {
        uint64_t x = t >= off ? sh[t - off] : 0ull;
        __syncthreads();
        sh[t] += x;
        __syncthreads();
    }
    const uint64_t incl = sh[t];
    *total = sh[kScanThreads - 1];
    __syncthreads();
    return incl - v;
}

__global__ __launch_bounds__(kScanThreads) void k_scan_reduce(const uint32_t *__restrict__ in, int64_t n,
                                                              uint64_t *__restrict__ partial) {
    __shared__ uint64_t sh[kScanThreads];
    const int64_t lo = (int64_t)blockIdx.x * kScanBlock;
    uint64_t s = 0;
    for (int k = 0; k < kScanItems; ++k) {
        const int64_t i = lo + (int64_t)k * kScanThreads + threadIdx.x;
        if (i < n) s += (uint64_t)in[i];
    }
    sh[threadIdx.x] = s;
    __syncthreads();
    for (int off = kScanThreads / 2; off > 0; off >>= 1) {
        if (threadIdx.x < off) sh[threadIdx.x] += sh[threadIdx.x + off];
        __syncthreads();
    }
    if (threadIdx.x == 0) partial[blockIdx.x] = sh[0];
}

// Exclusive scan of the block partials in place (single block); partial[nblk] = total.
__global__ __launch_bounds__(1024) void k_scan_partials(uint64_t *__restrict__ partial, int64_t nblk) {
    __shared__ uint64_t sh[1024];
    const int64_t per = (nblk + 1023) / 1024;
    const int64_t lo = threadIdx.x * per, hi = min(lo + per, nblk);
    uint64_t s = 0;
    for (int64_t i = lo; i < hi; ++i) s += partial[i];
    sh[threadIdx.x] = s;
    __syncthreads();
    for (int off = 1; off < 1024; off <<= 1) {
        uint64_t x = threadIdx.x >= off ? sh[threadIdx.x - off] : 0ull;
        __syncthreads();
        sh[threadIdx.x] += x;
        __syncthreads();
    }
    uint64_t run = threadIdx.x ? sh[threadIdx.x - 1] : 0ull;
    for (int64_t i = lo; i < hi; ++i) {
        const uint64_t c = partial[i];
        partial[i] = run;
        run += c;
    }
    if (threadIdx.x == 1023) partial[nblk] = sh[1023];
}

__global__ __launch_bounds__(kScanThreads) void k_scan_apply(const uint32_t *__restrict__ in, int64_t n,
                                                              const uint64_t *__restrict__ partial, int64_t nblk,
                                                              uint64_t *__restrict__ out) {
    __shared__ uint64_t sh[kScanThreads];
    const int64_t lo = (int64_t)blockIdx.x * kScanBlock + (int64_t)threadIdx.x * kScanItems;
    uint64_t v[kScanItems];
    uint64_t s = 0;
    for (int k = 0; k < kScanItems; ++k) {
        const int64_t i = lo + k;
        v[k] = i < n ? (uint64_t)in[i] : 0ull;
        s += v[k];
    }
    uint64_t total;
    uint64_t run = block_exclusive_scan(s, sh, &total) + partial[blockIdx.x];
    for (int k = 0; k < kScanItems; ++k) {
        const int64_t i = lo + k;
        if (i < n) out[i] = run;
        run += v[k];
    }
    if (blockIdx.x == 0 && threadIdx.x == 0) out[n] = partial[nblk];
}

// The whole scan in one block, for up to kScanSmall items: 16 per thread.  Three
// launches take about 15 us however few the items are; one about 5.
constexpr int kScanSmallItems = 16, kScanSmall = 1024 * kScanSmallItems;
__global__ __launch_bounds__(1024) void k_scan_small(const uint32_t *__restrict__ in, int n,
                                                     uint64_t *__restrict__ out) {
    __shared__ uint64_t wsum[16];
    const int lane = threadIdx.x & 63, w = threadIdx.x >> 6, lo = (int)threadIdx.x * kScanSmallItems;
    uint32_t v[kScanSmallItems];
    uint64_t s = 0;
#pragma unroll
    for (int k = 0; k < kScanSmallItems; ++k) v[k] = lo + k < n ? in[lo + k] : 0u;
#pragma unroll
    for (int k = 0; k < kScanSmallItems; ++k) s += v[k];
    uint64_t incl = s;
    for (int off = 1; off < 64; off <<= 1) {
        const uint64_t x = (uint64_t)__shfl_up((unsigned long long)incl, off);
        if (lane >= off) incl += x;
    }
    if (lane == 63) wsum[w] = incl;
    __syncthreads();
    uint64_t run = incl - s;
    for (int k = 0; k < w; ++k) run += wsum[k];
#pragma unroll
    for (int k = 0; k < kScanSmallItems; ++k) {
        if (lo + k < n) out[lo + k] = run;
        run += v[k];
    }
    if (threadIdx.x == 1023) out[n] = run;
}

// out[i] = sum_{j<i} in[j] for i in [0, n]; out has n+1 entries.  (Kernels only,
// so that the sequence can be captured into a graph.)
void scan_u32_to_u64_exclusive(const uint32_t *in, uint64_t *out, int64_t n, uint64_t *tmp, hipStream_t st) {
    if (n <= kScanSmall) {
        hipLaunchKernelGGL(k_scan_small, dim3(1), dim3(1024), 0, st, in, (int)n, out);
        return;
    }
    const int64_t nblk = (n + kScanBlock - 1) / kScanBlock;
    hipLaunchKernelGGL(k_scan_reduce, dim3((unsigned)nblk), dim3(kScanThreads), 0, st, in, n, tmp);
    hipLaunchKernelGGL(k_scan_partials, dim3(1), dim3(1024), 0, st, tmp, nblk);
    hipLaunchKernelGGL(k_scan_apply, dim3((unsigned)nblk), dim3(kScanThreads), 0, st, in, n, tmp, nblk, out);
}

// ---------------------------------------------------------------------------
__global__ void k_fill_u32(uint32_t *p, uint32_t v, int64_t n) {
    for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < n; i += (int64_t)gridDim.x * blockDim.x)
        p[i] = v;
}
__global__ void k_fill_u64(uint64_t *p, uint64_t v, int64_t n) {
    for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < n; i += (int64_t)gridDim.x * blockDim.x)
        p[i] = v;
}
// dst[k] = src[min(k stride, n)] for k = 0 .. ceil(n / stride).
__global__ void k_gather_u64(uint64_t *dst, const uint64_t *src, int64_t n, int64_t stride, int64_t count) {
    const int64_t k = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (k < count) dst[k] = src[min(k * stride, n)];
}
void launch_gather_u64(uint64_t *dst, const uint64_t *src, int64_t n, int64_t stride, hipStream_t st) {
    const int64_t count = (n + stride - 1) / stride + 1;
    hipLaunchKernelGGL(k_gather_u64, dim3((unsigned)((count + 255) / 256)), dim3(256), 0, st, dst, src, n, stride,
                       count);
}
void launch_fill_u32(uint32_t *p, uint32_t v, int64_t n, hipStream_t st) {
    if (n <= 0) return;
    const int64_t blocks = min((n + 255) / 256, (int64_t)65536);
    hipLaunchKernelGGL(k_fill_u32, dim3((unsigned)blocks), dim3(256), 0, st, p, v, n);
}
void launch_fill_u64(uint64_t *p, uint64_t v, int64_t n, hipStream_t st) {
    if (n <= 0) return;
    const int64_t blocks = min((n + 255) / 256, (int64_t)65536);
    hipLaunchKernelGGL(k_fill_u64, dim3((unsigned)blocks), dim3(256), 0, st, p, v, n);
}

// Fixed-order sum: per-block tree sums in double, then a sequential sum of
// the block results, so the total does not depend on scheduling.
__global__ __launch_bounds__(256) void k_sum_blocks(const float *__restrict__ x, int64_t n, double *partial) {
    __shared__ double sh[256];
    const int64_t lo = (int64_t)blockIdx.x * 4096;
    double s = 0.0;
    for (int k = 0; k < 16; ++k) {
        const int64_t i = lo + (int64_t)k * 256 + threadIdx.x;
        if (i < n) s += (double)x[i];
    }
    sh[threadIdx.x] = s;
    __syncthreads();
    for (int off = 128; off > 0; off >>= 1) {
        if (threadIdx.x < off) sh[threadIdx.x] += sh[threadIdx.x + off];
        __syncthreads();
    }
    if (threadIdx.x == 0) partial[blockIdx.x] = sh[0];
}
// (one thread adds in order, from LDS: straight from memory every 8 bytes waited
// for the addition before, 12 us for 245 blocks, 4 so)
__global__ __launch_bounds__(256) void k_sum_final(const double *__restrict__ partial, int64_t nblk,
                                                   double *__restrict__ out) {
    __shared__ double sh[1024];
    double s = 0.0;
    for (int64_t b0 = 0; b0 < nblk; b0 += 1024) {
        const int n = (int)min(nblk - b0, (int64_t)1024);
        for (int i = threadIdx.x; i < n; i += 256) sh[i] = partial[b0 + i];
        __syncthreads();
        if (threadIdx.x == 0)
            for (int i = 0; i < n; ++i) s += sh[i];
        __syncthreads();
    }
    if (threadIdx.x == 0) *out = s;
}
void launch_sum_f32_to_f64(const float *x, int64_t n, double *out, double *tmp, hipStream_t st) {
    const int64_t nblk = (n + 4095) / 4096;
    hipLaunchKernelGGL(k_sum_blocks, dim3((unsigned)nblk), dim3(256), 0, st, x, n, tmp);
    hipLaunchKernelGGL(k_sum_final, dim3(1), dim3(256), 0, st, tmp, nblk, out);
}

}  // namespace gs
