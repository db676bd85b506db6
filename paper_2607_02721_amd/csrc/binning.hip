// Tile binning: per-tile front-to-back lists of Gaussians.
//
// Input: per view, the visible Gaussians in depth order (position p of the
// radix-sorted (depth key, index) sequence; ties by index because the sort is
// stable and starts from index order).  A list entry is keyed by (tile, p)
// and the lists are built by a counting sort on that key:
//   1. count: one block per chunk of 2^8 to 2^14 consecutive positions counts its
//             entries per tile in LDS and stores them, one row per chunk;
//   2. scan:  per tile, the exclusive prefix over chunks (in place) and the
//             tile's total; a scan of the totals gives each tile's list start,
//             so a tile's list is its chunks' segments in order;
//   3. emit:  one wave per (chunk, group of tile rows) expands the chunk's
//             positions that meet its rows, in order and 2^10 (2^11 with a
//             ray mask) at a time, into
//             (position, tile) items packed 64 to a batch; every tile's next
//             slot comes from a wave-private LDS cursor, taken in the
//             positions' order, so each (tile, chunk) segment is written
//             already sorted by p, as g | sub-rectangle mask << 28.
// Chunks are long so that a tile's segment in a chunk spans whole cache
// lines: list entries are 4 bytes, and segments of a few entries each end in
// partial lines that cost a full write each.
// The mask's bits name the tile's sub-rectangles (halves in x and y, whatever the
// tile's size) that the Gaussian's pixel range meets; quad_subrect_bits says which
// 8x8 quadrants they hold.
#include "gs_internal.hpp"

#include <algorithm>

namespace gs {

constexpr int kBinThreads = 256;
constexpr int kCountGroup = 32;        // most chunks per XCD run (multiples of the 16 counts in a 64-byte line)
constexpr int kEmitGroupChunks = 4;    // chunks (times the row groups) per XCD run

static_assert(kChunkBitsMax <= 16, "queued positions are 16-bit chunk offsets");

// Workgroups are dealt to the 8 XCDs round-robin.  Renumbering hands out
// logical blocks in runs of `group` per XCD (run k to XCD k mod 8), so
// neighbouring chunks (which write neighbouring words of the same lines) and
// the row groups of one chunk (which read the same positions) share one L2,
// while all XCDs stay on nearby chunks of one view.  The grid size must be a
// multiple of 8 * group.
__device__ __forceinline__ int64_t xcd_block(int64_t b, int64_t group) {
    const int64_t xcd = b & 7, slot = b >> 3;
    return ((slot / group) * 8 + xcd) * group + slot % group;
}

// An entry's sub-rectangle bits (halves in x and y) of a tile that its range
// meets: bits 0 and 1 the left and right half, doubled by two bits for the lower
// half.  It meets the left (top) half iff it starts before the middle, and the
// right (bottom) half iff it ends after it; column_halves * row_halves is the
// mask.
__device__ __forceinline__ uint32_t column_halves(int xa, int xb, int tx) {
    return (xa <= 2 * tx ? 1u : 0u) | (xb > 2 * tx ? 2u : 0u);
}
__device__ __forceinline__ uint32_t row_halves(const HalfRange &h, int ty) {
    return (h.ya <= 2 * ty ? 1u : 0u) | (h.yb > 2 * ty ? 4u : 0u);
}

__global__ __launch_bounds__(kBinThreads) void k_bin_count(const ViewDev *__restrict__ views, int n_views,
                                                           int64_t N, int nchunks,
                                                           const uint32_t *__restrict__ nvis,
                                                           const uint32_t *__restrict__ xr_in,
                                                           const uint32_t *__restrict__ yr_in,
                                                           uint32_t *__restrict__ bin_count,
                                                           const uint16_t *__restrict__ active,
                                                           uint64_t *__restrict__ rowbits, int rows_stride,
                                                           int chunk_bits, int xcd_group, int half_ranges) {
    // A position adds 1 to every tile of its tile rectangle: +1 / -1 at the
    // rectangle's corners of a 2D difference array, whose prefix sums along
    // x and then y are the counts (four LDS atomics per position, whatever
    // its size).
    extern __shared__ int32_t dif[];                  // [tiles_y + 1][tiles_x + 1]
    __shared__ uint64_t rowword[kBinThreads / 64][128];   // per wave: row words on their way to the lanes
    const int64_t lb = xcd_block(blockIdx.x, xcd_group);   // logical block: chunk + nchunks * view
    const int v = (int)(lb / nchunks);
    if (v >= n_views) return;
    const ViewDev &V = views[v];
    const int64_t nv = nvis[v];
    const int chunk = (int)(lb - (int64_t)v * nchunks);
    const int64_t lo = (int64_t)chunk << chunk_bits;
    if (lo >= nv) return;
    const int64_t hi = min(lo + (1ll << chunk_bits), nv);
    const int tx_n = V.tiles_x, ty_n = V.tiles_y, ntiles = tx_n * ty_n;
    const int stride = tx_n + 1, cells = stride * (ty_n + 1);
    for (int i = threadIdx.x; i < cells; i += kBinThreads) dif[i] = 0;
    __syncthreads();
    // the view's row bitmaps for this chunk: word w of row r at
    // rb + r * row_pitch + w
    const int words = 1 << (chunk_bits - 6);
    const int64_t row_pitch = (int64_t)nchunks * words;
    uint64_t *rb = rowbits + (int64_t)v * rows_stride * row_pitch + (int64_t)chunk * words;
    // every lane of a wave runs each step (positions past the chunk's end
    // are invalid), so the row words gathered into the lanes can be stored
    // by the whole wave
    const int lane = threadIdx.x & 63;
    uint64_t *sw = rowword[threadIdx.x >> 6];
    for (int64_t p0 = lo + (threadIdx.x & ~63); p0 < hi; p0 += kBinThreads) {
        const int64_t p = p0 + lane;
        const bool valid = p < hi;
        // rows [ty0, ty0 + span]; invalid positions meet none (r - ty0 wraps
        // to a large unsigned value for every row r)
        int ty0 = 0x40000000;
        uint32_t span = 0u;
        if (valid) {
            const int64_t at = (int64_t)v * N + p;
            const HalfRange h = half_range(half_ranges, xr_in[at], half_ranges ? 0u : yr_in[at], V.tsx, V.tsy);
            const int x0 = h.xa >> 1, x1 = (h.xb >> 1) + 1;
            ty0 = h.ya >> 1;
            const int ty1 = h.yb >> 1;
            span = (uint32_t)(ty1 - ty0);
            const int y0 = ty0 * stride, y1 = (ty1 + 1) * stride;
            atomicAdd(&dif[y0 + x0], 1);
            atomicAdd(&dif[y0 + x1], -1);
            atomicAdd(&dif[y1 + x0], -1);
            atomicAdd(&dif[y1 + x1], 1);
        }
        // the wave's 64 positions form one bitmap word per tile row: one
        // ballot per row, written to LDS by lane 0 (128 rows at a time) and
        // read back by the lane that stores the row's word
        const int w = (int)((p0 - lo) >> 6);
        for (int rb0 = 0; rb0 < ty_n; rb0 += 128) {
            const int rn = __builtin_amdgcn_readfirstlane(min(128, ty_n - rb0));
            const uint32_t rel = (uint32_t)(rb0 - ty0);
#pragma unroll 8
            for (int k = 0; k < rn; ++k) {
                const uint64_t bits = __ballot(rel + (uint32_t)k <= span);
                if (lane == 0) sw[k] = bits;
            }
            wave_sync();
            if (lane < rn) rb[(int64_t)(rb0 + lane) * row_pitch + w] = sw[lane];
            if (lane + 64 < rn) rb[(int64_t)(rb0 + lane + 64) * row_pitch + w] = sw[lane + 64];
            wave_sync();   // the words are read before the next rows overwrite them
        }
    }
    __syncthreads();
    for (int ty = threadIdx.x; ty < ty_n; ty += kBinThreads) {       // along x, one row per thread
        int run = 0;
        for (int tx = 0; tx < tx_n; ++tx) {
            run += dif[ty * stride + tx];
            dif[ty * stride + tx] = run;
        }
    }
    __syncthreads();
    for (int tx = threadIdx.x; tx < tx_n; tx += kBinThreads) {       // along y, one column per thread
        int run = 0;
        for (int ty = 0; ty < ty_n; ++ty) {
            run += dif[ty * stride + tx];
            dif[ty * stride + tx] = run;
        }
    }
    __syncthreads();
    // this block is the only writer of (tile, chunk) for every tile of the
    // view; tiles without a selected ray get no entries
    uint32_t *row = bin_count + (int64_t)V.tile_base * nchunks + (int64_t)chunk * ntiles;
    for (int t = threadIdx.x; t < ntiles; t += kBinThreads) {
        const bool off = active && !active[V.tile_base + t];
        row[t] = off ? 0u : (uint32_t)dif[(t / tx_n) * stride + t % tx_n];
    }
}

// Column pass over one view's [chunk][tile] counts: each thread owns one tile
// and replaces its counts, chunk by chunk, with their exclusive prefix (the
// tile's segment offsets inside its list); the tile's total goes to tile_tot.
// (Chunks past the view's visible positions are neither written nor read.)
__global__ __launch_bounds__(kBinThreads) void k_chunk_prefix(const ViewDev *__restrict__ views, int nchunks,
                                                              const uint32_t *__restrict__ nvis, int chunk_bits,
                                                              uint32_t *__restrict__ bin_count,
                                                              uint32_t *__restrict__ tile_tot) {
    const ViewDev &V = views[blockIdx.y];
    const int ntiles = V.tiles_x * V.tiles_y;
    const int t = blockIdx.x * kBinThreads + threadIdx.x;
    if (t >= ntiles) return;
    uint32_t *col = bin_count + (int64_t)V.tile_base * nchunks + t;
    const int used = (int)(((int64_t)nvis[blockIdx.y] + (1ll << chunk_bits) - 1) >> chunk_bits);
    uint32_t run = 0;
    int c = 0;
    for (; c + 8 <= used; c += 8) {
        uint32_t x[8];
#pragma unroll
        for (int k = 0; k < 8; ++k) x[k] = col[(int64_t)(c + k) * ntiles];
#pragma unroll
        for (int k = 0; k < 8; ++k) {
            col[(int64_t)(c + k) * ntiles] = run;
            run += x[k];
        }
    }
    for (; c < used; ++c) {
        const uint32_t x = col[(int64_t)c * ntiles];
        col[(int64_t)c * ntiles] = run;
        run += x;
    }
    tile_tot[V.tile_base + t] = run;
}

// Ordered emission.  One wave per (group of kEmitRows tile rows and at most
// kEmitCols tile columns, chunk, view).  For each batch of kEmitBatch
// positions of its chunk, the wave first compacts, in order, the positions
// whose rectangle meets its rows (an LDS queue), then takes them 64 at a
// time and expands them into (position, tile) items in position order: a wave
// prefix sum of the per-position item counts numbers the items, and each 64-item
// batch finds every item's owner from the marks of the items that start a
// position (a ballot of the marks, counted up to the item's lane).  Items of
// one batch that hit the same tile must take their slots in position (= lane)
// order: a per-tile LDS lane mask gives each item the lanes that share its tile,
// its rank among them is its offset from the tile's cursor, which is read along
// with the mask, and the last of them moves the cursor.  A wave's LDS operations
// execute in issue order, so later positions always receive later slots and every
// (tile, chunk) segment is filled in increasing p.
//
// Positions left over from full rounds of 64 wait for the next batch.
//
// What bounds it is the chain of LDS accesses of an item batch, some eight, at the
// 20 or so waves per CU that the lines in LDS leave room for, and about 115 vector
// instructions per item batch (2 of 2.8 ms at 1M Gaussians x 100 views, 486
// million entries of 32-pixel tiles; writing them takes 0.5).  Scans for owners, an
// atomic add and a shuffle for each run's slots, three reads per owner and partly
// filled rounds at the end of every 2048 positions took 3.02 ms there and 545 us
// at 300k x 20 views of 1280x720 with 16-pixel tiles (461 so).
//
// Entries are not stored one by one: each tile keeps the block ("line") of
// its list that it is filling in LDS (slot = absolute entry index mod the
// line length), and a line goes out as one store of consecutive lanes once
// its last slot is filled.  Only the first and last line of a segment
// (shared with the neighbouring chunks' segments) are written partially.
// Scattered 4-byte stores leave the L2 as several partial-line writes per
// line (about 24 GB of writes for 4.3 GB of entries at 1M Gaussians x 100
// views with 16x16 tiles, against 6.6 GB with 32-byte lines).  Lines are 8
// entries (32 bytes) for tiles 8 or 16 pixels wide, which keeps the wave's
// LDS small, and 16 entries (64 bytes, streamed past the L2) for tiles 32
// pixels wide, whose segments per chunk are long enough to fill them.
constexpr int kEmitWave = 64;
constexpr int kEmitRows = 1;
constexpr int kEmitCols = 128;     // tile columns per wave (2048 pixels)
constexpr int kDirectTiles = 16;   // active tiles of a masked wave up to which it takes them one by one

__device__ __forceinline__ uint64_t lanemask_lt64_bin() {
    const unsigned lane = threadIdx.x & 63;
    return lane == 0 ? 0ull : (~0ull >> (64 - lane));
}

// Wave-wide inclusive scans over the 64 lanes with DPP: shifts by 1, 2, 4, 8
// inside each row of 16 lanes, then row_bcast:15 (row r-1's last lane into
// rows 1 and 3) and row_bcast:31 (lane 31 into rows 2 and 3).  Lanes without
// a source take the identity.
template <int kCtrl, int kRowMask>
__device__ __forceinline__ int dpp_src(int identity, int x) {
    return __builtin_amdgcn_update_dpp(identity, x, kCtrl, kRowMask, 0xF, false);
}

__device__ __forceinline__ int wave_scan_add(int v) {
    v += dpp_src<0x111, 0xF>(0, v);
    v += dpp_src<0x112, 0xF>(0, v);
    v += dpp_src<0x114, 0xF>(0, v);
    v += dpp_src<0x118, 0xF>(0, v);
    v += dpp_src<0x142, 0xA>(0, v);
    v += dpp_src<0x143, 0xC>(0, v);
    return v;
}

// Bits >= s of a 64-bit word (s may be negative or past 63).
__device__ __forceinline__ uint64_t bits_from(int s) {
    return s >= 64 ? 0ull : (s <= 0 ? ~0ull : (~0ull << s));
}

// The bits a..b (0 <= a <= b < 128) of the 128-bit set (lo, hi).
__device__ __forceinline__ void clip_range(uint64_t &lo, uint64_t &hi, int a, int b) {
    lo &= bits_from(a) & ~bits_from(b + 1);
    hi &= bits_from(a - 64) & ~bits_from(b + 1 - 64);
}

// Position of the j-th set bit (from 0) of a 128-bit set that has more than j.
__device__ __forceinline__ int nth_bit(uint64_t lo, uint64_t hi, int j) {
    const int c = __popcll(lo);
    const int base = j < c ? 0 : 64;
    uint64_t m = j < c ? lo : hi;
    for (int k = j < c ? j : j - c; k > 0; --k) m &= m - 1ull;
    return base + __ffsll((long long)m) - 1;
}

// A list entry's store: 64-byte lines bypass the L2 (they are whole write
// requests, and the lists are read only by a later launch); 32-byte lines
// go through it, where the halves of a request that two chunks' segments
// share are merged.
template <int kLine>
__device__ __forceinline__ void store_entry(uint32_t v, uint32_t *dst) {
    if (kLine >= 16)
        __builtin_nontemporal_store(v, dst);
    else
        *dst = v;
}

// A tile of an emission wave: the lanes of the current item batch on it (0
// between batches), its next entry and the first entry of its segment in this
// chunk, both relative to the view's first entry.
struct __align__(16) EmitTile {
    uint64_t lanes;
    uint32_t cur, seg0;
};

// A position expanded by the wave: its index; and in one word its range in half
// tiles from column c0 on, clipped to the wave's columns (first and last, a byte
// each), the halves of the tile row it meets (3 bits: 1 top, 4 bottom) and its
// first item of the round (13 bits: 64 positions of up to kEmitCols tiles).
struct __align__(8) EmitPos {
    uint32_t g, at;
};
static_assert(2 * 128 <= 256 && 64 * 128 <= 8192, "the fields of EmitPos::at");

// LDS layout of one emission wave.
struct EmitLds {
    EmitTile *tile;     // [tiles]
    EmitPos *pos;       // [64] the round's positions that have items
    uint2 *full;        // [64] lines to store: tile, and the entry in its last slot
    uint32_t *line;     // [tiles][2^kLineLog] the line each tile is filling
    uint32_t *mark;     // [64] the batch in which an item last started a position
    uint32_t *act;      // [tiles / 32] active tiles (masked form only)
    uint16_t *queue;    // [batch + 63] chunk-local positions meeting the rows
};

__host__ __device__ constexpr size_t emit_lds_bytes(int tiles, bool masked, int line_log, int batch) {
    return (size_t)tiles * (sizeof(EmitTile) + (sizeof(uint32_t) << line_log)) +
           (sizeof(EmitPos) + sizeof(uint2) + sizeof(uint32_t)) * kEmitWave +
           (masked ? sizeof(uint32_t) * (((size_t)tiles + 31) / 32) : 0) + sizeof(uint16_t) * ((size_t)batch + kEmitWave);
}

template <int kLine>
__device__ __forceinline__ EmitLds emit_lds(uint32_t *base, int tiles, int batch, bool masked) {
    EmitLds L;
    L.tile = (EmitTile *)base;
    L.pos = (EmitPos *)(L.tile + tiles);
    L.full = (uint2 *)(L.pos + kEmitWave);
    L.line = (uint32_t *)(L.full + kEmitWave);
    L.mark = L.line + (size_t)tiles * kLine;
    L.act = L.mark + kEmitWave;
    L.queue = (uint16_t *)(L.act + (masked ? (tiles + 31) / 32 : 0));
    return L;
}

// Stores the staged blocks ("lines") listed in L.full (n of them), 64 / kLine per step
// with kLine lanes each; entries before the tile's segment (another chunk's) and at or
// past `room` are left alone.  (A line that begins before the view's first entry
// has slots whose numbers wrap around: they lie past `last`.)
template <int kLine>
__device__ __forceinline__ void store_lines(const EmitLds &L, int n, uint32_t align, uint32_t *__restrict__ vl,
                                            uint32_t room) {
    const int lane = threadIdx.x;
    for (int f0 = 0; f0 < n; f0 += kEmitWave / kLine) {
        const int f = f0 + lane / kLine, k = lane % kLine;
        if (f < n) {
            const uint2 line = L.full[f];                            // tile, entry in the line's last slot
            const uint32_t e = line.y - ((align + line.y) & (kLine - 1u)) + (uint32_t)k;
            if (e >= L.tile[line.x].seg0 && e <= line.y && e < room)
                store_entry<kLine>(L.line[line.x * kLine + k], &vl[e]);
        }
    }
}

template <bool kMasked, int kLineLog>
__global__ __launch_bounds__(kEmitWave) void k_bin_emit(const ViewDev *__restrict__ views, int n_views, int64_t N,
                                                        int nchunks, int row_groups, int col_groups,
                                                        const uint32_t *__restrict__ nvis,
                                                        const uint32_t *__restrict__ xr_in,
                                                        const uint32_t *__restrict__ yr_in,
                                                        const uint32_t *__restrict__ sorted_g,
                                                        const uint32_t *__restrict__ bin_count,
                                                        const uint64_t *__restrict__ tile_off,
                                                        uint32_t *__restrict__ lists,
                                                        const uint16_t *__restrict__ active, uint64_t cap,
                                                        int group_tiles, const uint64_t *__restrict__ rowbits,
                                                        int rows_stride, int chunk_bits, int batch,
                                                        int half_ranges) {
    extern __shared__ uint32_t lds[];
    constexpr int kLine = 1 << kLineLog;
    const EmitLds L = emit_lds<kLine>(lds, group_tiles, batch, kMasked);
    // logical block: group + groups * (chunk + nchunks * view), with group =
    // row group + row_groups * column group
    const int groups = row_groups * col_groups;
    const int64_t lb = xcd_block(blockIdx.x, (int64_t)kEmitGroupChunks * groups);
    const int64_t per_view = (int64_t)groups * nchunks;
    const int v = (int)(lb / per_view);
    if (v >= n_views) return;
    const int grp = (int)(lb % groups);
    const int chunk = (int)((lb - (int64_t)v * per_view) / groups);
    const int lane = threadIdx.x;
    const ViewDev &V = views[v];
    const int sx = V.tsx, sy = V.tsy;
    const int64_t nv = nvis[v];
    const int64_t lo = (int64_t)chunk << chunk_bits;
    const int r0 = (grp % row_groups) * kEmitRows, c0 = (grp / row_groups) * kEmitCols;
    if (lo >= nv || r0 >= V.tiles_y || c0 >= V.tiles_x) return;
    const int r1 = min(r0 + kEmitRows, V.tiles_y);    // rows [r0, r1)
    const int c1 = min(c0 + kEmitCols, V.tiles_x);    // columns [c0, c1)
    const int hi = (int)(min(lo + (1ll << chunk_bits), nv) - lo);
    const int tiles_x = V.tiles_x, ncols = c1 - c0;
    const int ntiles = (r1 - r0) * ncols;             // local tile (ty - r0) * ncols + (tx - c0)
    const uint64_t vlist = tile_off[V.tile_base];
    const uint32_t align = (uint32_t)(vlist & (kLine - 1u));   // slot of the view's first entry in its line
    // segment start of each of the wave's tiles for this chunk, relative to
    // the view's first entry: the tile's list start plus the tile's prefix
    const uint32_t *pre = bin_count + (int64_t)V.tile_base * nchunks + (int64_t)chunk * (V.tiles_x * V.tiles_y);
    for (int t = lane; t < ntiles; t += kEmitWave) {
        const int vt = (r0 + t / ncols) * tiles_x + c0 + t % ncols;   // tile within the view
        const uint32_t s0 = (uint32_t)(tile_off[V.tile_base + vt] - vlist) + pre[vt];
        L.tile[t] = EmitTile{0ull, s0, s0};
    }
    L.mark[lane] = 0u;
    if (kMasked) {
        for (int w = lane; w < (ntiles + 31) / 32; w += kEmitWave) {
            uint32_t bits = 0;
            for (int b = 0; b < 32; ++b) {
                const int t = 32 * w + b;
                const int vt = (r0 + t / ncols) * tiles_x + c0 + t % ncols;
                bits |= (t < ntiles && active[V.tile_base + vt]) ? (1u << b) : 0u;
            }
            L.act[w] = bits;
        }
    }
    wave_sync();
    // masked form: the wave's active tiles as a 128-bit set (one tile row);
    // a wave with none has nothing to emit
    static_assert(!kMasked || (kEmitRows == 1 && kEmitCols <= 128), "one row of at most 128 tiles");
    uint64_t act_lo = 0ull, act_hi = 0ull;
    if (kMasked) {
        const int nw = (ntiles + 31) / 32;
        act_lo = (uint64_t)L.act[0] | (nw > 1 ? (uint64_t)L.act[1] << 32 : 0ull);
        act_hi = (nw > 2 ? (uint64_t)L.act[2] : 0ull) | (nw > 3 ? (uint64_t)L.act[3] << 32 : 0ull);
        if ((act_lo | act_hi) == 0ull) return;
    }
    // few active tiles (sparse masks): the queued positions are held against
    // each of them, 64 at a time, and the hits of a ballot go out in order at
    // the tile's cursor (lane a holds that of the a-th active tile).  The general
    // form's owner search, ranks and lines in LDS are a chain of some twenty LDS
    // accesses per round, which the 16 waves a CU has room for do not hide: 2.43
    // -> 1.16 ms at 1M Gaussians x 100 views, 1% of the 8x8 blocks (three active
    // tiles of 80 per row; bounds of 16 and of 64 tiles measured alike).
    const int n_act = kMasked ? __popcll(act_lo) + __popcll(act_hi) : 0;
    const bool direct = kMasked && n_act <= kDirectTiles;
    uint32_t cursor = 0u;
    if (direct && lane < n_act) cursor = L.tile[nth_bit(act_lo, act_hi, lane)].seg0;
    // entries at or past `room` would fall outside the list buffer
    // (entry numbers within a view have 32 bits)
    const uint32_t room = cap > vlist ? (uint32_t)min(cap - vlist, (uint64_t)0xFFFFFFFFull) : 0u;
    uint32_t *__restrict__ vl = lists + vlist;
    const int64_t o = (int64_t)v * N + lo;
    // this wave's row bitmap in the chunk (one word per 64 positions)
    static_assert(kEmitRows == 1, "the row bitmaps select one tile row");
    const int words = 1 << (chunk_bits - 6);
    const uint64_t *rbits =
        rowbits + ((int64_t)v * rows_stride + r0) * ((int64_t)nchunks * words) + (int64_t)chunk * words;
    static_assert(kEmitBatch % 64 == 0 && kEmitBatchMasked % 64 == 0 && kEmitBatch <= 64 * kEmitWave &&
                      kEmitBatchMasked <= 64 * kEmitWave, "one row-bitmap word per lane");
    uint32_t tick = 0u;
    auto bitmap_word = [&](int b0) {    // of positions b0 + 64 lane ... + 63 of a batch
        return lane < ((min(b0 + batch, hi) - b0 + 63) >> 6) ? __builtin_nontemporal_load(&rbits[(b0 >> 6) + lane]) : 0ull;
    };
    uint64_t ahead = bitmap_word(0);
    int left = 0;                       // queued positions of the batches before
    for (int b0 = 0; b0 < hi; b0 += batch) {
        // 1. positions of the batch that meet row r0, in order: lane l takes
        // the bitmap word of positions b0 + 64 l ... + 63 (bits past the chunk's
        // visible positions are clear), a wave prefix sum of the popcounts
        // places each lane's positions in the queue
        uint64_t word = ahead;
        if (b0 + batch < hi) ahead = bitmap_word(b0 + batch);
        const int cnt = __popcll(word);
        const int incl = wave_scan_add(cnt);
        const int nq = left + __builtin_amdgcn_readlane(incl, kEmitWave - 1);
        int slot = left + incl - cnt;
        while (word) {
            const int bit = __ffsll((long long)word) - 1;
            L.queue[slot++] = (uint16_t)(b0 + 64 * lane + bit);
            word &= word - 1ull;
        }
        wave_sync();
        // 2. expansion of the queued positions against this wave's tiles, 64 at
        // a time (what is left over waits for the next batch); the next round's
        // ranges and indices are loaded while this one expands
        const int rounds = b0 + batch < hi ? nq & ~(kEmitWave - 1) : nq;
        uint32_t nx_ = 0, ny_ = 0, ng_ = 0;
        if (lane < rounds) {
            const int p = L.queue[lane];
            nx_ = xr_in[o + p];
            if (!half_ranges) ny_ = yr_in[o + p];
            ng_ = sorted_g[o + p];
        }
        for (int base = 0; base < rounds; base += kEmitWave) {
            const int qi = base + lane;
            const uint32_t ux = nx_, uy = ny_, ug = ng_;
            if (qi + kEmitWave < rounds) {
                const int p = L.queue[qi + kEmitWave];
                nx_ = xr_in[o + p];
                if (!half_ranges) ny_ = yr_in[o + p];
                ng_ = sorted_g[o + p];
            }
            if (kMasked && direct) {
                // the positions against each active tile in turn
                const HalfRange h = half_range(half_ranges, ux, uy, sx, sy);
                const uint32_t rows = row_halves(h, r0);
                const int xa = qi < nq ? h.xa >> 1 : 0x7FFFFFFF, xb = h.xb >> 1;
                uint64_t lo64 = act_lo, hi64 = act_hi;
                for (int a = 0; a < n_act; ++a) {
                    const bool low = lo64 != 0ull;
                    const int tx = c0 + (low ? __ffsll((long long)lo64) - 1 : 63 + __ffsll((long long)hi64));
                    lo64 &= lo64 - (low ? 1ull : 0ull);
                    hi64 &= hi64 - (low ? 0ull : 1ull);
                    const bool hit = xa <= tx && tx <= xb;
                    const uint64_t bal = __ballot(hit);
                    if (bal == 0ull) continue;
                    const uint32_t at = (uint32_t)__builtin_amdgcn_readlane((int)cursor, a);
                    const uint32_t e = at + (uint32_t)__popcll(bal & lanemask_lt64_bin());
                    if (hit && e < room)
                        store_entry<kLine>(ug | (column_halves(h.xa, h.xb, tx) * rows) << 28, &vl[e]);
                    if (lane == a) cursor = at + (uint32_t)__popcll(bal);
                }
                continue;
            }
            // the tiles of its rectangle inside this wave's row and columns
            // (masked form: the active ones among them)
            int k = 0;
            EmitPos mine{ug, 0u};
            if (qi < nq) {
                const HalfRange h = half_range(half_ranges, ux, uy, sx, sy);
                const int xa = max(h.xa - 2 * c0, 0), xb = min(h.xb - 2 * c0, 2 * ncols - 1);
                mine.at = (uint32_t)(xa & 255) | (uint32_t)(xb & 255) << 8 | row_halves(h, r0) << 16;
                if (kMasked) {
                    if (xa <= xb) {
                        uint64_t lo64 = act_lo, hi64 = act_hi;
                        clip_range(lo64, hi64, xa >> 1, xb >> 1);
                        k = __popcll(lo64) + __popcll(hi64);
                    }
                } else {
                    k = max((xb >> 1) - (xa >> 1) + 1, 0);
                }
            }
            const int incl = wave_scan_add(k);
            const int K = __builtin_amdgcn_readlane(incl, kEmitWave - 1);
            const int excl = incl - k;   // first item of this lane's position
            mine.at |= (uint32_t)excl << 19;
            const uint64_t with = __ballot(k > 0);
            if (k > 0) L.pos[__popcll(with & lanemask_lt64_bin())] = mine;
            for (int i0 = 0; i0 < K; i0 += kEmitWave) {
                const int i = i0 + lane;
                const bool on = i < K;
                // owner of item i among the positions with items: those whose
                // first item is at or before i0, less one, and one more for every
                // position that starts between (each marks its first item with the
                // batch's number).
                ++tick;
                const int carry = __popcll(__ballot(k > 0 && excl <= i0)) - 1;
                if (k > 0 && excl > i0 && excl < i0 + kEmitWave) L.mark[excl - i0] = tick;
                wave_sync();
                const uint64_t starts = __ballot(L.mark[lane] == tick) >> 1;   // (item i0 marks nothing)
                const int own = (int)__builtin_amdgcn_mbcnt_hi(
                    (uint32_t)(starts >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)starts, (uint32_t)carry));
                const EmitPos P = L.pos[on ? own : 0];
                const int j = i - (int)(P.at >> 19), xa = (int)(P.at & 255u), xb = (int)((P.at >> 8) & 255u);
                int t = (xa >> 1) + j;                 // tile within the wave
                if (kMasked) {
                    uint64_t lo64 = act_lo, hi64 = act_hi;
                    clip_range(lo64, hi64, xa >> 1, xb >> 1);
                    if (on) t = nth_bit(lo64, hi64, j);
                }
                t = on ? t : 0;
                const uint32_t val = P.g | (column_halves(xa, xb, t) * ((P.at >> 16) & 7u)) << 28;
                // Lanes on the same tile: each lane ORs its bit into its tile's
                // 64-bit mask and reads the mask and the cursor back.  A lane's
                // rank among them (lanes are in position order) is its offset from
                // the cursor; the last of them moves the cursor and clears the mask.
                if (on) atomicOr((unsigned long long *)&L.tile[t].lanes, 1ull << lane);
                wave_sync();
                const EmitTile T = L.tile[t];
                wave_sync();
                const uint32_t rank = on ? (uint32_t)__popcll(T.lanes & lanemask_lt64_bin()) : 0u;
                const uint32_t c = T.cur + rank;
                if (on && (T.lanes & ~lanemask_lt64_bin()) == 1ull << lane) L.tile[t] = EmitTile{0ull, c + 1u, T.seg0};
                // The entries go into their tiles' lines one line at a time: in
                // step s every tile writes only within the s-th line its run
                // touches, and the lines whose last slot was filled are stored
                // before the next step reuses their slots.
                const uint32_t slot = (align + c) & (kLine - 1u);
                const int step = on ? (int)((((align + T.cur) & (kLine - 1u)) + rank) / kLine) : -1;
                for (int s = 0; __ballot(step >= s) != 0ull; ++s) {
                    const bool now = step == s;
                    if (now) L.line[t * kLine + slot] = val;
                    const bool full = now && slot == kLine - 1u;
                    const uint64_t need = __ballot(full);
                    if (need) {
                        if (full) {
                            const int r = __popcll(need & lanemask_lt64_bin());
                            L.full[r] = make_uint2((uint32_t)t, c);
                        }
                        wave_sync();
                        store_lines<kLine>(L, __popcll(need), align, vl, room);
                        wave_sync();
                    }
                }
                wave_sync();
            }
        }
        wave_sync();
        left = nq - rounds;
        if (left > 0) {
            const uint16_t p = lane < left ? L.queue[rounds + lane] : (uint16_t)0;
            wave_sync();
            if (lane < left) L.queue[lane] = p;
        }
    }
    if (direct) return;
    // 3. the last, partly filled line of every tile whose segment ends inside one
    for (int t4 = 0; t4 < ntiles; t4 += kEmitWave) {
        const int t = t4 + lane;
        bool part = false;
        uint32_t c = 0;
        if (t < ntiles) {
            c = L.tile[t].cur;
            part = c > L.tile[t].seg0 && ((align + c) & (kLine - 1u)) != 0u;
        }
        const uint64_t need = __ballot(part);
        // (the last entry: slots after it are not stored)
        if (part) L.full[__popcll(need & lanemask_lt64_bin())] = make_uint2((uint32_t)t, c - 1u);
        wave_sync();
        store_lines<kLine>(L, __popcll(need), align, vl, room);
        wave_sync();
    }
}

void launch_bin_count(const ViewDev *views_dev, int Vc, int64_t N, int nchunks, const ChunkBufs &b,
                      const uint32_t *xr, const uint32_t *yr, int max_cells, hipStream_t st) {
    // runs of neighbouring chunks per XCD, short enough that every XCD gets one
    // (runs of 32 left 96 blocks to three of the eight XCDs)
    const int64_t all = (int64_t)nchunks * Vc;
    const int group = (int)std::min<int64_t>(kCountGroup, std::max<int64_t>(1, all / 8));
    const int64_t run = 8 * (int64_t)group;
    const int64_t blocks = (all + run - 1) / run * run;
    static const bool lds_ok = [] {
        // views up to kMaxCellsPerView cells take more than 64 KiB of LDS
        const hipError_t e = hipFuncSetAttribute(reinterpret_cast<const void *>(k_bin_count),
                                                 hipFuncAttributeMaxDynamicSharedMemorySize,
                                                 kMaxCellsPerView * (int)sizeof(int32_t));
        if (e != hipSuccess) (void)hipGetLastError();
        return e == hipSuccess;
    }();
    (void)lds_ok;
    hipLaunchKernelGGL(k_bin_count, dim3((unsigned)blocks), dim3(kBinThreads), (size_t)max_cells * sizeof(int32_t),
                       st, views_dev, Vc, N, nchunks, b.nvis, xr, yr, b.bin_count, b.tile_active, b.rowbits,
                       b.rows_stride, b.chunk_bits, group, b.half_ranges);
}

void launch_chunk_prefix(const ViewDev *views_dev, int Vc, int nchunks, const ChunkBufs &b, int max_tiles,
                         hipStream_t st) {
    hipLaunchKernelGGL(k_chunk_prefix, dim3((unsigned)((max_tiles + kBinThreads - 1) / kBinThreads), (unsigned)Vc),
                       dim3(kBinThreads), 0, st, views_dev, nchunks, b.nvis, b.chunk_bits, b.bin_count, b.tile_tot);
}

void launch_bin_emit(const ViewDev *views_dev, int Vc, int64_t N, int nchunks, const ChunkBufs &b,
                     const uint32_t *xr, const uint32_t *yr, const uint32_t *sorted_g, int max_tiles_x,
                     int max_tiles_y, uint64_t cap, int tile_shift_x, hipStream_t st) {
    const int row_groups = (max_tiles_y + kEmitRows - 1) / kEmitRows;
    const int col_groups = (max_tiles_x + kEmitCols - 1) / kEmitCols;
    const int64_t run = 8 * (int64_t)kEmitGroupChunks * row_groups * col_groups;
    const int64_t blocks = ((int64_t)row_groups * col_groups * nchunks * Vc + run - 1) / run * run;
    const int group_tiles = kEmitRows * std::min(max_tiles_x, kEmitCols);
    const int line_log = tile_shift_x >= 5 ? 4 : 3;
    const int batch = std::min(b.tile_active ? kEmitBatchMasked : kEmitBatch, 1 << b.chunk_bits);
    const size_t lds = emit_lds_bytes(group_tiles, b.tile_active != nullptr, line_log, batch);
    const dim3 grid((unsigned)blocks);
    auto go = [&](auto kernel) {
        hipLaunchKernelGGL(kernel, grid, dim3(kEmitWave), lds, st, views_dev, Vc, N, nchunks, row_groups, col_groups,
                           b.nvis, xr, yr, sorted_g, b.bin_count, b.tile_off, b.lists, b.tile_active, cap,
                           group_tiles, b.rowbits, b.rows_stride, b.chunk_bits, batch, b.half_ranges);
    };
    if (b.tile_active)
        line_log == 4 ? go(k_bin_emit<true, 4>) : go(k_bin_emit<true, 3>);
    else
        line_log == 4 ? go(k_bin_emit<false, 4>) : go(k_bin_emit<false, 3>);
}

// Plan guards.  Lists sized in advance: if the counted entries exceed the
// capacity, every list of the scene is emptied, so that no later kernel reads
// past the buffer.  Three-pass depth sorts: a view's depth keys that span 2^24 - 1
// or more no longer sort before the invisible ones, which have no ranges, so the
// scene's views then hold no position at all; this runs before the sort, and
// nothing after it reads a position.  Either way the scene's output is zero this
// run and the sticky flag is raised.
__global__ void k_span_check(const uint32_t *__restrict__ kmin, int Vc, uint32_t *__restrict__ nvis,
                             uint32_t *__restrict__ over, uint32_t *__restrict__ flag) {
    bool bad = false;
    for (int v = threadIdx.x; v < Vc; v += blockDim.x)
        bad = bad || (kmin[Vc + v] >= kmin[v] && kmin[Vc + v] - kmin[v] >= 0xFFFFFFu);
    bad = __any(bad);
    if (bad)
        for (int v = threadIdx.x; v < Vc; v += blockDim.x) nvis[v] = 0u;
    if (threadIdx.x == 0) {
        *over = bad ? 1u : 0u;
        if (bad) atomicOr(flag, kGuardSpan);
    }
}
__global__ void k_guard_check(const uint64_t *__restrict__ tile_off, int64_t ntiles, uint64_t cap,
                              uint32_t *__restrict__ over, uint32_t *__restrict__ flag, int keep) {
    const bool o = tile_off[ntiles] > cap;
    *over = (o || (keep && *over)) ? 1u : 0u;
    if (o) atomicOr(flag, kGuardList);
}
__global__ void k_guard_apply(uint64_t *__restrict__ tile_off, int64_t ntiles, const uint32_t *__restrict__ over) {
    const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (*over && i <= ntiles) tile_off[i] = 0;
}
void launch_span_check(const ChunkBufs &b, int Vc, uint32_t *over, uint32_t *flag, hipStream_t st) {
    hipLaunchKernelGGL(k_span_check, dim3(1), dim3(64), 0, st, b.kmin, Vc, b.nvis, over, flag);
}
void launch_list_guard(uint64_t *tile_off, int64_t ntiles, uint64_t cap, uint32_t *over, uint32_t *flag, bool keep,
                       hipStream_t st) {
    hipLaunchKernelGGL(k_guard_check, dim3(1), dim3(1), 0, st, tile_off, ntiles, cap, over, flag, keep ? 1 : 0);
    hipLaunchKernelGGL(k_guard_apply, dim3((unsigned)((ntiles + 256) / 256)), dim3(256), 0, st, tile_off, ntiles,
                       over);
}

// A tile is active when at least one of its rays is selected by the ray mask;
// inactive tiles get empty lists.  active[t] holds one bit per 8x8 quadrant
// (bit q: quadrant q, row-major inside the tile, holds a selected ray).  One
// lane per pixel row of a tile: its up to 32 mask bits are consecutive, so one
// or two words give them; lanes of a tile then OR their quadrant bits.  (A wave
// per tile with a bit test per pixel took 146 us for 360 000 tiles of
// 16x16; this takes 35.)
__global__ __launch_bounds__(256) void k_tile_active(const ViewDev *__restrict__ views,
                                                     const int32_t *__restrict__ tile_view,
                                                     const uint32_t *__restrict__ mask, uint16_t *__restrict__ active,
                                                     int total_tiles, int tsy) {
    const int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x;
    const int gt = (int)(i >> tsy), row = (int)i & ((1 << tsy) - 1);
    uint32_t bits = 0u;
    if (gt < total_tiles) {
        const ViewDev &V = views[tile_view[gt]];
        const int tl = gt - V.tile_base;
        const int px = (tl % V.tiles_x) << V.tsx, py = ((tl / V.tiles_x) << V.tsy) + row;
        const int width = min(1 << V.tsx, V.W - px);
        if (py < V.H) {
            const int64_t ray = V.ray_base + (int64_t)py * V.W + px;
            const int sh = (int)(ray & 31);
            uint64_t w = mask[ray >> 5];
            if (sh + width > 32) w |= (uint64_t)mask[(ray >> 5) + 1] << 32;
            const uint32_t sel = (uint32_t)(w >> sh) & (width < 32 ? (1u << width) - 1u : ~0u);
            const int qlx = V.tsx - 3;
            uint32_t cols = 0u;
            for (int c = 0; c < (1 << qlx); ++c) cols |= ((sel >> (8 * c)) & 0xFFu) ? (1u << c) : 0u;
            bits = cols << ((row >> 3) << qlx);
        }
    }
    for (int off = 1; off < (1 << tsy); off <<= 1) bits |= (uint32_t)__shfl_xor((int)bits, off);
    if (gt < total_tiles && row == 0) active[gt] = (uint16_t)bits;
}

void launch_tile_active(const ViewDev *views_dev, const int32_t *tile_view, int total_tiles, int tile_shift_y,
                        const uint32_t *mask, uint16_t *active, hipStream_t st) {
    const int64_t lanes = (int64_t)total_tiles << tile_shift_y;
    hipLaunchKernelGGL(k_tile_active, dim3((unsigned)((lanes + 255) / 256)), dim3(256), 0, st, views_dev, tile_view,
                       mask, active, total_tiles, tile_shift_y);
}

// Row y + 1 of view v's table: running counts of active tiles along tile row
// y; row 0 is all zeros (written by the thread of row 0).
__global__ __launch_bounds__(64) void k_tile_sat_rows(const ViewDev *__restrict__ views,
                                                      const uint16_t *__restrict__ active, uint32_t *__restrict__ sat) {
    const ViewDev &V = views[blockIdx.y];
    const int ty = blockIdx.x * 64 + threadIdx.x;
    if (ty >= V.tiles_y) return;
    const int stride = V.tiles_x + 1;
    uint32_t *S = sat + V.sat_base;
    if (ty == 0)
        for (int x = 0; x < stride; ++x) S[x] = 0u;
    uint32_t *row = S + (int64_t)(ty + 1) * stride;
    const uint16_t *a = active + V.tile_base + (int64_t)ty * V.tiles_x;
    uint32_t run = 0;
    row[0] = 0u;
    for (int x = 0; x < V.tiles_x; ++x) {
        run += a[x] ? 1u : 0u;
        row[x + 1] = run;
    }
}

// Column x of view v's table: running sums down the rows.
__global__ __launch_bounds__(64) void k_tile_sat_cols(const ViewDev *__restrict__ views, uint32_t *__restrict__ sat) {
    const ViewDev &V = views[blockIdx.y];
    const int x = blockIdx.x * 64 + threadIdx.x;
    const int stride = V.tiles_x + 1;
    if (x >= stride) return;
    uint32_t *S = sat + V.sat_base;
    uint32_t run = 0;
    for (int y = 1; y <= V.tiles_y; ++y) {
        run += S[(int64_t)y * stride + x];
        S[(int64_t)y * stride + x] = run;
    }
}

__global__ __launch_bounds__(256) void k_quad_count(const uint16_t *__restrict__ active, int n,
                                                    uint32_t *__restrict__ qcnt) {
    const int t = blockIdx.x * 256 + threadIdx.x;
    if (t < n) qcnt[t] = (uint32_t)__popc((unsigned)active[t]);
}

__global__ __launch_bounds__(256) void k_quad_write(const uint16_t *__restrict__ active, int n, int quad_log,
                                                    const uint64_t *__restrict__ qoff, uint32_t *__restrict__ qlist) {
    const int t = blockIdx.x * 256 + threadIdx.x;
    if (t >= n) return;
    const unsigned bits = active[t];
    uint64_t o = qoff[t];
    for (int q = 0; q < (1 << quad_log); ++q)
        if ((bits >> q) & 1u) qlist[o++] = (uint32_t)(((uint32_t)t << quad_log) + q);
}

void launch_quad_list(const uint16_t *active, int total_tiles, int quad_log, uint32_t *qcnt, uint64_t *qoff,
                      uint64_t *scan_tmp, uint32_t *qlist, hipStream_t st) {
    const unsigned blocks = (unsigned)((total_tiles + 255) / 256);
    hipLaunchKernelGGL(k_quad_count, dim3(blocks), dim3(256), 0, st, active, total_tiles, qcnt);
    scan_u32_to_u64_exclusive(qcnt, qoff, total_tiles, scan_tmp, st);
    hipLaunchKernelGGL(k_quad_write, dim3(blocks), dim3(256), 0, st, active, total_tiles, quad_log, qoff, qlist);
}

void launch_tile_sat(const ViewDev *views_dev, int Vc, int max_tx, int max_ty, const uint16_t *active, uint32_t *sat,
                     hipStream_t st) {
    hipLaunchKernelGGL(k_tile_sat_rows, dim3((unsigned)((max_ty + 63) / 64), (unsigned)Vc), dim3(64), 0, st,
                       views_dev, active, sat);
    hipLaunchKernelGGL(k_tile_sat_cols, dim3((unsigned)((max_tx + 1 + 63) / 64), (unsigned)Vc), dim3(64), 0, st,
                       views_dev, sat);
}

}  // namespace gs
