// Stable radix partitioning (the radix-partition primitive of Section 2.3, used
// as the transformation of the partitioned hash join in Section 4.1.4 and of the
// partition-based group-by in Section 4.3).
//
// One pass reorders rows stably by a digit of at most 8 bits. A pass works on
// segments (pass 1: the whole input; pass 2: every partition of pass 1), which
// are cut into chunks of whole tiles:
//   k_chunk_table  chunks per segment and their exclusive prefix (several
//                  segments only)
//   k_hist         per chunk, rows per digit -> hist[seg][digit][chunk] (not for
//                  an input of one tile)
//   scan           flat exclusive scan of hist = absolute output offset of each
//                  (segment, digit, chunk) run, because that order is the
//                  output order (small passes: each scatter workgroup sums the
//                  counts before its own)
//   k_scatter      per chunk, tile by tile: wave-level ranking by ballot (no
//                  atomics, so equal digits keep input order), LDS staging in
//                  digit order, then runs written contiguously; the key and
//                  every payload column reuse the same positions. A segment's
//                  first chunk also writes its partition boundaries
// Two passes with the top bits first give rows sorted stably by the full digit,
// i.e. every partition contiguous and in input order.
#include <stdio.h>
#include <stdlib.h>

#include <vector>

#include "internal.hpp"

namespace gj {
namespace {

// Default scatter: the whole-line kernel for large passes (long_chunks), else the
// tiles of tile_shape. Group 0 names the wide kernel among the shapes (one column at
// a time with a rolling prefetch).
constexpr int kScatterBlock = 1024;
constexpr int kItems = 16;
constexpr int kGroup = -1;

// Where a chunk's output offsets come from: the scanned counts (hist), the raw
// counts of its segment, or the tile itself (the input is one tile).
enum OffsetMode : int { kOffScanned = 0, kOffDirect = 1, kOffSelf = 2 };

struct PassArgs {
    const void *key_in;
    void *key_out;
    int ncols;
    int n4;         // columns 0..n4-1 are 4 bytes wide, the rest 8 bytes
    int rowid_col;  // index of the generated row-id column, or -1
    const void *col_in[kMaxCols];
    void *col_out[kMaxCols];
    int col_w[kMaxCols];
    DigitFn dig;
    int bits;
    const uint32_t *seg_off;  // nseg + 1 row offsets (nullptr: one segment, the whole input)
    uint32_t nseg;
    const uint32_t *chunk_base;  // nseg + 1 chunk offsets (nullptr: one segment)
    uint32_t n_chunks;           // ceil(n_rows / chunk_rows): the chunks of a single segment
    uint32_t *poff;              // optional: receives the partition boundaries (segment, digit)
    int off_mode;                // OffsetMode
    uint32_t chunk_rows;
    bool cells;  // long chunks (below): cut at multiples of chunk_rows of the whole input
    uint32_t *hist;  // [chunks][2^bits], laid out as (segment, digit, chunk)
    uint32_t n_rows; // rows of the output columns; every store is checked against it
    const uint8_t *seg_bits;  // optional: digit bits per segment (<= bits; batches of instances)
    uint32_t row_bytes;       // k_scatter_lines: bytes of the key and every column
};

__device__ __forceinline__ uint32_t seg_begin(const PassArgs &a, uint32_t s) { return a.seg_off ? a.seg_off[s] : 0u; }
__device__ __forceinline__ uint32_t seg_end(const PassArgs &a, uint32_t s) {
    return a.seg_off ? a.seg_off[s + 1] : a.n_rows;
}

// The digit function of the segment a chunk belongs to.
__device__ __forceinline__ DigitFn seg_digit(const PassArgs &a, uint32_t seg) {
    DigitFn d = a.dig;
    if (a.seg_bits) d.mask = (1u << a.seg_bits[seg]) - 1u;
    return d;
}

// Chunks. Short ones: each segment is cut into pieces of chunk_rows rows, one
// workgroup each. Long ones (cells): the input is cut at multiples of chunk_rows
// into as many cells as there are workgroups and at the segments' ends; a
// workgroup takes the chunks of its cell one by one, so that every workgroup
// moves the same number of rows whatever the segments' sizes. (One workgroup per
// chunk of 2^20 rows: segments of 2^21 +- 2000 rows left a few chunks for a
// second round, 3.3 ms instead of 2.2 at 2^28 rows.)
struct ChunkLoc {
    uint32_t seg, j, m, row0, row1, hbase;
    int ok;
};

__device__ __forceinline__ uint32_t seg_chunks(uint32_t s0, uint32_t s1, uint32_t base, uint32_t chunk_rows, int cells) {
    if (s0 >= s1) return 0u;
    return cells ? (s1 - 1 - base) / chunk_rows - (s0 - base) / chunk_rows + 1 : ceil_div_u32(s1 - s0, chunk_rows);
}

// Uniform values in scalar registers (the loads they come from are vector ones).
__device__ __forceinline__ uint32_t uni(uint32_t x) { return __builtin_amdgcn_readfirstlane(x); }

// Segment `seg` of cell `cell`: its chunk there.
__device__ __forceinline__ ChunkLoc cell_chunk(const PassArgs &a, uint32_t cell, uint32_t seg) {
    ChunkLoc L{};
    const uint32_t base = uni(seg_begin(a, 0)), s0 = uni(seg_begin(a, seg)), s1 = uni(seg_end(a, seg));
    const uint32_t cb = a.chunk_base ? uni(a.chunk_base[seg]) : 0u, c0 = base + cell * a.chunk_rows;
    L.seg = seg;
    L.j = cell - (s0 - base) / a.chunk_rows;
    L.m = a.chunk_base ? uni(a.chunk_base[seg + 1]) - cb : a.n_chunks;
    L.row0 = max(s0, c0);
    L.row1 = min(s1, c0 + a.chunk_rows);
    L.hbase = cb << a.bits;
    L.ok = 1;
    return L;
}
// First segment with rows at or past the cell's first row.
__device__ uint32_t cell_first_seg(const PassArgs &a, uint32_t cell) {
    if (!a.seg_off) return 0u;
    const uint32_t row = a.seg_off[0] + cell * a.chunk_rows;
    uint32_t lo = 0, hi = a.nseg;  // seg_off[hi] > row
    while (hi - lo > 1) {
        const uint32_t mid = (lo + hi) >> 1;
        if (a.seg_off[mid] <= row) lo = mid;
        else hi = mid;
    }
    return uni(lo);
}

__device__ ChunkLoc locate_chunk(const PassArgs &a, uint32_t c) {
    ChunkLoc L{};
    if (!a.chunk_base) {  // one segment
        L.ok = c < a.n_chunks;
        L.j = c;
        L.m = a.n_chunks;
        L.row0 = c * a.chunk_rows;
        L.row1 = (uint32_t)min<uint64_t>((uint64_t)L.row0 + a.chunk_rows, a.n_rows);
        return L;
    }
    const uint32_t total = a.chunk_base[a.nseg];
    if (c >= total) {
        L.ok = 0;
        return L;
    }
    uint32_t lo = 0, hi = a.nseg;  // chunk_base[lo] <= c < chunk_base[hi]
    while (hi - lo > 1) {
        const uint32_t mid = (lo + hi) >> 1;
        if (a.chunk_base[mid] <= c) lo = mid;
        else hi = mid;
    }
    const uint32_t cb = a.chunk_base[lo];
    L.seg = lo;
    L.j = c - cb;
    L.m = a.chunk_base[lo + 1] - cb;
    const uint32_t s0 = a.seg_off[lo], s1 = a.seg_off[lo + 1];
    L.row0 = s0 + L.j * a.chunk_rows;
    L.row1 = min(L.row0 + a.chunk_rows, s1);
    L.hbase = cb << a.bits;
    L.ok = 1;
    return L;
}

// Also writes the partition boundaries of empty segments, which no chunk visits.
__global__ __launch_bounds__(1024) void k_chunk_table(const uint32_t *__restrict__ seg_off, uint32_t nseg,
                                                      uint32_t chunk_rows, int cells, int bits,
                                                      uint32_t *__restrict__ chunk_base, uint32_t *__restrict__ poff) {
    __shared__ uint32_t s_tmp[1024 / kWave];
    uint32_t carry = 0;
    for (uint32_t base = 0; base < nseg; base += 1024) {
        const uint32_t s = base + threadIdx.x;
        const uint32_t cnt = s < nseg ? seg_chunks(seg_off[s], seg_off[s + 1], seg_off[0], chunk_rows, cells) : 0u;
        uint32_t tot;
        const uint32_t ex = block_exclusive_sum<uint32_t, 1024 / kWave>(cnt, s_tmp, &tot);
        if (s < nseg) chunk_base[s] = carry + ex;
        if (s < nseg && cnt == 0 && poff)
            for (uint32_t d = 0; d < 1u << bits; ++d) poff[((uint64_t)s << bits) + d] = seg_off[s];
        carry += tot;
    }
    if (threadIdx.x == 0) {
        chunk_base[nseg] = carry;
        if (poff) poff[(uint64_t)nseg << bits] = seg_off[nseg];
    }
}

// Counts of one chunk's rows per digit.
template <typename K, int BLOCK>
__device__ __forceinline__ void hist_chunk(const PassArgs &a, const ChunkLoc &L, uint32_t (*s_cnt)[kRadix]) {
    constexpr int U = 16;  // loads in flight per thread
    constexpr int W = BLOCK / kWave;
    for (int i = threadIdx.x; i < W * kRadix; i += BLOCK) (&s_cnt[0][0])[i] = 0;
    __syncthreads();
    const K *__restrict__ keys = static_cast<const K *>(a.key_in);
    const int tid = threadIdx.x, w = tid / kWave;
    const DigitFn dig = seg_digit(a, L.seg);
    for (uint32_t base = L.row0; base < L.row1; base += BLOCK * U) {
        K k[U];
#pragma unroll
        for (int u = 0; u < U; ++u) {
            const uint32_t row = base + u * BLOCK + tid;
            k[u] = row < L.row1 ? keys[row] : K(0);
        }
        // counting needs no order, so plain LDS atomics into the wave's own histogram
#pragma unroll
        for (int u = 0; u < U; ++u) {
            if (base + u * BLOCK + tid < L.row1) atomicAdd(&s_cnt[w][digit_of<K>(k[u], dig)], 1u);
        }
    }
    __syncthreads();
    const uint32_t R = 1u << a.bits;
    for (uint32_t d = threadIdx.x; d < R; d += BLOCK) {
        uint32_t t = 0;
#pragma unroll
        for (int q = 0; q < W; ++q) t += s_cnt[q][d];
        a.hist[L.hbase + d * L.m + L.j] = t;
    }
}

template <typename K>
__global__ __launch_bounds__(kBlock) void k_hist(PassArgs a) {
    __shared__ uint32_t s_cnt[kWaves][kRadix];
    __shared__ ChunkLoc s_loc;
    if (threadIdx.x == 0) s_loc = locate_chunk(a, blockIdx.x);
    __syncthreads();
    if (s_loc.ok) hist_chunk<K, kBlock>(a, s_loc, s_cnt);
}

// Long chunks: a workgroup per cell; 1024 threads, since there are only about as
// many cells as compute units.
template <typename K>
__global__ __launch_bounds__(1024) void k_hist_cells(PassArgs a) {
    __shared__ uint32_t s_cnt[1024 / kWave][kRadix];
    const uint32_t end = uni(seg_begin(a, 0)) + min((blockIdx.x + 1) * a.chunk_rows, a.n_rows);
    for (uint32_t seg = cell_first_seg(a, blockIdx.x); seg < a.nseg && uni(seg_begin(a, seg)) < end; ++seg) {
        const ChunkLoc L = cell_chunk(a, blockIdx.x, seg);
        if (L.row0 >= L.row1) continue;
        hist_chunk<K, 1024>(a, L, s_cnt);
        __syncthreads();
    }
}

// Histogram of a single-segment pass from per-chunk counts of the low 8 bits
// of the digit source (made while the keys were read for another purpose):
// digit d of `bits` bits gathers the 8-bit values congruent to d.
__global__ void k_fold_hist(const uint32_t *__restrict__ hist8, uint32_t m, int bits, uint32_t *__restrict__ hist) {
    const uint32_t R = 1u << bits;
    const uint32_t per = 256u >> bits;  // 8-bit values per digit
    for (uint32_t idx = blockIdx.x * blockDim.x + threadIdx.x; idx < R * m; idx += gridDim.x * blockDim.x) {
        const uint32_t d = idx / m, j = idx % m;
        const uint32_t *h = hist8 + (size_t)j * 256u;
        uint32_t t = 0;
        for (uint32_t q = 0; q < per; ++q) t += h[d + (q << bits)];
        hist[idx] = t;  // (segment 0, digit d, chunk j)
    }
}

// Partition boundaries of a chunk that is its segment's first (cur: its offsets).
__device__ __forceinline__ void write_poff(const PassArgs &a, const ChunkLoc &L, const uint32_t *cur, int threads) {
    if (!a.poff || L.j != 0) return;
    const uint32_t R = 1u << a.bits;
    for (uint32_t d = threadIdx.x; d < R; d += threads) a.poff[(L.seg << a.bits) + d] = cur[d];
    if (!a.seg_off && threadIdx.x == 0) a.poff[R] = a.n_rows;  // several segments: k_chunk_table
}

// Offsets of a chunk from the raw counts of its segment: the rows of smaller
// digits, and of its digit in earlier chunks. 16 lanes sum a digit's chunks.
// s_tmp: 4 words.
template <int BLOCK>
__device__ __forceinline__ void direct_offsets(const PassArgs &a, const ChunkLoc &L, uint32_t *cur, uint32_t *s_tot,
                                               uint32_t *s_tmp) {
    const uint32_t R = 1u << a.bits;
    const uint32_t *__restrict__ h = a.hist + L.hbase;
    const uint32_t i = threadIdx.x % 16;
    for (uint32_t d = threadIdx.x / 16; d < R; d += BLOCK / 16) {
        uint32_t tot = 0, before = 0;
        for (uint32_t j = i; j < L.m; j += 64) {
            uint32_t c[4];
#pragma unroll
            for (int u = 0; u < 4; ++u) c[u] = j + u * 16 < L.m ? h[d * L.m + j + u * 16] : 0u;
#pragma unroll
            for (int u = 0; u < 4; ++u) {
                tot += c[u];
                if (j + u * 16 < L.j) before += c[u];
            }
        }
#pragma unroll
        for (int k = 8; k > 0; k >>= 1) {
            tot += __shfl_xor(tot, k, 16);
            before += __shfl_xor(before, k, 16);
        }
        if (i == 0) {
            s_tot[d] = tot;
            cur[d] = before;
        }
    }
    __syncthreads();
    const int t = threadIdx.x, w = t / kWave;
    uint32_t inc = 0, x = 0;
    if (t < kRadix) {
        x = (uint32_t)t < R ? s_tot[t] : 0u;
        inc = wave_inclusive_sum<uint32_t>(x);
        if (lane_id() == kWave - 1) s_tmp[w] = inc;
    }
    __syncthreads();
    if (t < kRadix && (uint32_t)t < R) {
        uint32_t pre = seg_begin(a, L.seg) + inc - x;
#pragma unroll
        for (int q = 0; q < kRadix / kWave; ++q) pre += q < w ? s_tmp[q] : 0u;
        cur[t] += pre;
    }
    __syncthreads();
}

// Loads of one tile: ITEMS keys per thread and the first group of up to G 4-byte
// columns (a generated row id is its row index). Rows past nt read as zero.
template <typename K, int BLOCK, int ITEMS, int G>
__device__ __forceinline__ void scatter_load_keys(const PassArgs &a, uint32_t tile0, uint32_t nt, K (&key)[ITEMS]) {
    const K *__restrict__ keys = static_cast<const K *>(a.key_in);
    const int w = threadIdx.x / kWave, lane = lane_id();
    const uint32_t lbase = (uint32_t)(w * kWave * ITEMS + lane);
#pragma unroll
    for (int r = 0; r < ITEMS; ++r) key[r] = lbase + r * kWave < nt ? keys[tile0 + lbase + r * kWave] : K(0);
}

template <int BLOCK, int ITEMS>
__device__ __forceinline__ void scatter_load_col(const PassArgs &a, int c, uint32_t tile0, uint32_t nt,
                                                 uint32_t (&v)[ITEMS]) {
    const int w = threadIdx.x / kWave, lane = lane_id();
    const uint32_t lbase = (uint32_t)(w * kWave * ITEMS + lane);
    const bool gen = (c == a.rowid_col);
    const uint32_t *__restrict__ in = static_cast<const uint32_t *>(a.col_in[c]);
#pragma unroll
    for (int r = 0; r < ITEMS; ++r) {
        const uint32_t row = tile0 + lbase + r * kWave;
        v[r] = gen ? row : (lbase + r * kWave < nt ? in[row] : 0u);
    }
}

// One tile of the stable scatter: nt rows from tile0, whose keys are already in
// `key`. Once the keys are in LDS, their registers receive the next tile's keys
// (next0, next_nt rows; next_nt = 0: none), so that those loads are in flight
// during this tile's column work and the next tile ranks without waiting.
// Columns 0..n4-1 are 4-byte (the generated row id among them), columns
// n4..ncols-1 are 8-byte.
template <int BLOCK>
struct ScatterShared {
    static constexpr int W = BLOCK / kWave;
    uint32_t wcnt[W][kRadix];
    uint32_t start[kRadix];
    uint32_t tot[kRadix];
    uint32_t cur[kRadix];
    uint32_t tmp[kWaves];
};

template <typename K, int BLOCK, int ITEMS, int G>
__device__ __forceinline__ void scatter_tile(const PassArgs &a, const ChunkLoc &L, const DigitFn &dig,
                                             ScatterShared<BLOCK> &S, uint32_t (*s_buf)[BLOCK * ITEMS], uint32_t tile0, uint32_t nt,
                                             K (&key)[ITEMS], uint32_t next0, uint32_t next_nt) {
    constexpr int W = BLOCK / kWave;
    const int tid = threadIdx.x, w = tid / kWave, lane = lane_id();
    K *__restrict__ kout = static_cast<K *>(a.key_out);
    K *sk = reinterpret_cast<K *>(&s_buf[0][0]);
    uint64_t *s8 = reinterpret_cast<uint64_t *>(&s_buf[0][0]);
    const int n4 = a.n4;
    const bool full = (nt == BLOCK * ITEMS);
    const uint32_t lbase = (uint32_t)(w * kWave * ITEMS + lane);
#define GJ_VALID(r) (full || lbase + (r) * kWave < nt)

    for (int i = tid; i < W * kRadix; i += BLOCK) (&S.wcnt[0][0])[i] = 0;
    // the first column group is loaded now and consumed after the ranking
    uint32_t v[G][ITEMS];
#pragma unroll
    for (int g = 0; g < G; ++g)
        if (g < n4) scatter_load_col<BLOCK, ITEMS>(a, g, tile0, nt, v[g]);
    __syncthreads();

    // stable rank within the wave: ballot peers, the leader bumps the wave counter
    uint32_t pos[ITEMS];
#pragma unroll
    for (int r = 0; r < ITEMS; ++r) {
        const bool valid = GJ_VALID(r);
        const uint32_t d = digit_of<K>(key[r], dig);
        const uint64_t peers = match_peers(d, a.bits, valid);
        uint32_t p = 0;
        if (valid) {
            const uint32_t rk = rank_below(peers);
            const uint32_t b = S.wcnt[w][d];
            if (rk == 0) S.wcnt[w][d] = b + (uint32_t)__popcll(peers);
            p = b + rk;
        }
        pos[r] = p;
    }
    __syncthreads();
    if (tid < kRadix) {
        // threads 0..255 (one per digit): tile totals and cross-wave exclusive prefix
        uint32_t t = 0;
#pragma unroll
        for (int q = 0; q < W; ++q) {
            const uint32_t c = S.wcnt[q][tid];
            S.wcnt[q][tid] = t;
            t += c;
        }
        S.tot[tid] = t;
        // exclusive scan over the 256 digits by the first four waves
        const uint32_t inc = wave_inclusive_sum<uint32_t>(t);
        if (lane == kWave - 1) S.tmp[w] = inc;
        S.start[tid] = inc - t;
    }
    __syncthreads();
    if (tid < kRadix) {
        uint32_t before = 0;
#pragma unroll
        for (int q = 0; q < kWaves; ++q) before += (q < w) ? S.tmp[q] : 0u;
        S.start[tid] += before;
        if (a.off_mode == kOffSelf) S.cur[tid] = S.start[tid];  // the only tile
    }
    __syncthreads();
    if (a.off_mode == kOffSelf) write_poff(a, L, S.cur, BLOCK);
#pragma unroll
    for (int r = 0; r < ITEMS; ++r) {
        if (GJ_VALID(r)) {
            const uint32_t d = digit_of<K>(key[r], dig);
            pos[r] += S.start[d] + S.wcnt[w][d];
            sk[pos[r]] = key[r];
        }
    }
    // the key registers are free: next tile's keys
    if (next_nt) scatter_load_keys<K, BLOCK, ITEMS, G>(a, next0, next_nt, key);
    __syncthreads();

    uint32_t dst[ITEMS];
#pragma unroll
    for (int k = 0; k < ITEMS; ++k) {
        const uint32_t i = (uint32_t)(k * BLOCK + tid);
        dst[k] = 0xFFFFFFFFu;
        if (full || i < nt) {
            const K kk = sk[i];
            const uint32_t d = digit_of<K>(kk, dig);
            const uint32_t t = S.cur[d] + i - S.start[d];
            if (t < a.n_rows) {  // always true when the offsets are right
                dst[k] = t;
                kout[t] = kk;
            }
        }
    }
    // 4-byte keys sit in buffer 0, so the first column goes to buffer 1; 8-byte
    // keys use both buffers and need a barrier before reuse.
    int par = 1;
    if constexpr (sizeof(K) == 8) {
        __syncthreads();
        par = 0;
    }
    for (int c0 = 0; c0 < n4; c0 += G) {
        if (c0 > 0) {
#pragma unroll
            for (int g = 0; g < G; ++g)
                if (c0 + g < n4) scatter_load_col<BLOCK, ITEMS>(a, c0 + g, tile0, nt, v[g]);
        }
#pragma unroll
        for (int g = 0; g < G; ++g) {
            if (c0 + g < n4) {
                uint32_t *sb = s_buf[par];
#pragma unroll
                for (int r = 0; r < ITEMS; ++r)
                    if (GJ_VALID(r)) sb[pos[r]] = v[g][r];
                __syncthreads();
                uint32_t *__restrict__ out = static_cast<uint32_t *>(a.col_out[c0 + g]);
#pragma unroll
                for (int k = 0; k < ITEMS; ++k)
                    if (dst[k] != 0xFFFFFFFFu) out[dst[k]] = sb[k * BLOCK + tid];
                par ^= 1;
            }
        }
    }
    for (int c = n4; c < a.ncols; ++c) {
        uint64_t x[ITEMS];
        const uint64_t *__restrict__ in = static_cast<const uint64_t *>(a.col_in[c]);
#pragma unroll
        for (int r = 0; r < ITEMS; ++r) x[r] = GJ_VALID(r) ? in[tile0 + lbase + r * kWave] : 0ull;
        __syncthreads();  // both buffers free
#pragma unroll
        for (int r = 0; r < ITEMS; ++r)
            if (GJ_VALID(r)) s8[pos[r]] = x[r];
        __syncthreads();
        uint64_t *__restrict__ out = static_cast<uint64_t *>(a.col_out[c]);
#pragma unroll
        for (int k = 0; k < ITEMS; ++k)
            if (dst[k] != 0xFFFFFFFFu) out[dst[k]] = s8[k * BLOCK + tid];
    }
#undef GJ_VALID
    __syncthreads();
    if (tid < kRadix) S.cur[tid] += S.tot[tid];
    __syncthreads();
}

// Loads of the wide kernel: one 64-bit base address per thread, every row at a
// constant offset from it (r * 64 rows), so that the 16 loads of a column need
// no per-row address registers. A full tile loads without row checks; in a
// partial one, rows past nt read as zero. A generated row id is its row index.
template <typename K, int ITEMS>
__device__ __forceinline__ void wide_load_keys(const PassArgs &a, uint32_t tile0, uint32_t nt, K (&key)[ITEMS]) {
    constexpr uint32_t TILE = 1024u * ITEMS;
    const uint32_t lbase = (uint32_t)((threadIdx.x / kWave) * kWave * ITEMS + lane_id());
    const K *__restrict__ p = static_cast<const K *>(a.key_in) + (tile0 + lbase);
    if (nt == TILE) {
#pragma unroll
        for (int r = 0; r < ITEMS; ++r) key[r] = p[r * kWave];
    } else {
        const uint32_t rem = nt > lbase ? nt - lbase : 0u;
#pragma unroll
        for (int r = 0; r < ITEMS; ++r) key[r] = (uint32_t)(r * kWave) < rem ? p[r * kWave] : K(0);
    }
}

template <int ITEMS>
__device__ __forceinline__ void wide_load_col(const PassArgs &a, int c, uint32_t tile0, uint32_t nt,
                                              uint32_t (&v)[ITEMS]) {
    constexpr uint32_t TILE = 1024u * ITEMS;
    const uint32_t lbase = (uint32_t)((threadIdx.x / kWave) * kWave * ITEMS + lane_id());
    if (c == a.rowid_col) {
#pragma unroll
        for (int r = 0; r < ITEMS; ++r) v[r] = tile0 + lbase + r * kWave;
        return;
    }
    const uint32_t *__restrict__ p = static_cast<const uint32_t *>(a.col_in[c]) + (tile0 + lbase);
    if (nt == TILE) {
#pragma unroll
        for (int r = 0; r < ITEMS; ++r) v[r] = p[r * kWave];
    } else {
        const uint32_t rem = nt > lbase ? nt - lbase : 0u;
#pragma unroll
        for (int r = 0; r < ITEMS; ++r) v[r] = (uint32_t)(r * kWave) < rem ? p[r * kWave] : 0u;
    }
}

// Wide tiles: 1024 threads x 16 rows = 16384-row tiles, twice the rows of the
// default shape, so that every digit's run per tile (the burst each column
// writes to HBM) is twice as long. The shorter the bursts, the slower the
// scatter: at equal work, 8-bit digits over 8192-row tiles write at about 55%
// of the rate of one-digit tiles. The larger tile fits the registers because
// columns move one at a time: while column c is staged and stored, column
// c + 1 (or the next tile's first column) is already loading into the one
// column register array, and 8-byte columns move in two halves of 8 rows.
// FULL tiles (all but a chunk's last) carry no per-row checks.
template <typename K, int BLOCK, int ITEMS, bool FULL>
__device__ __forceinline__ void scatter_tile_wide(const PassArgs &a, const DigitFn &dig, ScatterShared<BLOCK> &S,
                                                  uint32_t (*s_buf)[BLOCK * ITEMS], uint32_t tile0, uint32_t nt,
                                                  K (&key)[ITEMS], uint32_t (&v)[ITEMS], uint32_t next0,
                                                  uint32_t next_nt) {
    constexpr int W = BLOCK / kWave;
    // the thread index passes through an empty asm statement, so that nothing
    // derived from it is hoisted out of a caller's tile loop (it would hold
    // registers across the whole loop)
    int tid = threadIdx.x;
    asm volatile("" : "+v"(tid));
    const int w = tid / kWave, lane = tid % kWave;
    K *__restrict__ kout = static_cast<K *>(a.key_out);
    K *sk = reinterpret_cast<K *>(&s_buf[0][0]);
    uint64_t *s8 = reinterpret_cast<uint64_t *>(&s_buf[0][0]);
    const int n4 = a.n4;
    const uint32_t lbase = (uint32_t)(w * kWave * ITEMS + lane);
    // rows of this thread (r * 64 < lrem) and staged slots of this thread (k * BLOCK < srem)
    const uint32_t lrem = FULL ? 0xFFFFFFFFu : (nt > lbase ? nt - lbase : 0u);
    const uint32_t srem = FULL ? 0xFFFFFFFFu : (nt > (uint32_t)tid ? nt - (uint32_t)tid : 0u);
#define GJ_VALID(r) (FULL || (uint32_t)((r) * kWave) < lrem)

    for (int i = tid; i < W * kRadix; i += BLOCK) (&S.wcnt[0][0])[i] = 0;
    __syncthreads();

    // stable rank within the wave: ballot peers, the leader bumps the wave counter
    uint32_t pos[ITEMS];
#pragma unroll
    for (int r = 0; r < ITEMS; ++r) {
        const bool valid = GJ_VALID(r);
        const uint32_t d = digit_of<K>(key[r], dig);
        const uint64_t peers = match_peers(d, a.bits, valid);
        uint32_t p = 0;
        if (valid) {
            const uint32_t rk = rank_below(peers);
            const uint32_t b = S.wcnt[w][d];
            if (rk == 0) S.wcnt[w][d] = b + (uint32_t)__popcll(peers);
            p = b + rk;
        }
        pos[r] = p;
    }
    __syncthreads();
    if (tid < kRadix) {
        uint32_t t = 0;
#pragma unroll
        for (int q = 0; q < W; ++q) {
            const uint32_t c = S.wcnt[q][tid];
            S.wcnt[q][tid] = t;
            t += c;
        }
        S.tot[tid] = t;
        const uint32_t inc = wave_inclusive_sum<uint32_t>(t);
        if (lane == kWave - 1) S.tmp[w] = inc;
        S.start[tid] = inc - t;
    }
    __syncthreads();
    if (tid < kRadix) {
        uint32_t before = 0;
#pragma unroll
        for (int q = 0; q < kWaves; ++q) before += (q < w) ? S.tmp[q] : 0u;
        S.start[tid] += before;
    }
    __syncthreads();
#pragma unroll
    for (int r = 0; r < ITEMS; ++r) {
        if (GJ_VALID(r)) {
            const uint32_t d = digit_of<K>(key[r], dig);
            pos[r] += S.start[d] + S.wcnt[w][d];
            sk[pos[r]] = key[r];
        }
    }
    // the key registers are free: next tile's keys
    if (next_nt) wide_load_keys<K, ITEMS>(a, next0, next_nt, key);
    // LDS slots (< 16384) two to a register from here on
    uint32_t pp[ITEMS / 2];
#pragma unroll
    for (int r = 0; r < ITEMS / 2; ++r) pp[r] = (pos[2 * r] & 0xFFFFu) | (pos[2 * r + 1] << 16);
#define GJ_POS(r) ((pp[(r) >> 1] >> (16 * ((r) & 1))) & 0xFFFFu)
    __syncthreads();

    uint32_t dst[ITEMS];
#pragma unroll
    for (int k = 0; k < ITEMS; ++k) {
        const uint32_t i = (uint32_t)(k * BLOCK + tid);
        dst[k] = 0xFFFFFFFFu;
        if (FULL || (uint32_t)(k * BLOCK) < srem) {
            const K kk = sk[i];
            const uint32_t d = digit_of<K>(kk, dig);
            const uint32_t t = S.cur[d] + i - S.start[d];
            if (t < a.n_rows) {  // always true when the offsets are right
                dst[k] = t;
                kout[t] = kk;
            }
        }
    }

    // 4-byte keys sit in buffer 0, so the first column goes to buffer 1; 8-byte
    // keys use both buffers and need a barrier before reuse.
    int par = 1;
    if constexpr (sizeof(K) == 8) {
        __syncthreads();
        par = 0;
    }
#pragma unroll 1
    for (int c = 0; c < n4; ++c) {
        uint32_t *sb = s_buf[par];
#pragma unroll
        for (int r = 0; r < ITEMS; ++r)
            if (GJ_VALID(r)) sb[GJ_POS(r)] = v[r];
        // v is free: the next column of this tile, or the next tile's first one
        // (one load sequence for both cases keeps the register count down)
        const bool more = c + 1 < n4;
        if (more || next_nt)
            wide_load_col<ITEMS>(a, more ? c + 1 : 0, more ? tile0 : next0, more ? nt : next_nt, v);
        __syncthreads();
        uint32_t *__restrict__ out = static_cast<uint32_t *>(a.col_out[c]);
#pragma unroll
        for (int k = 0; k < ITEMS; ++k)
            if (dst[k] != 0xFFFFFFFFu) out[dst[k]] = sb[k * BLOCK + tid];
        par ^= 1;
    }
#pragma unroll 1
    for (int c = n4; c < a.ncols; ++c) {
        constexpr int HI = ITEMS / 2;
        const uint64_t *__restrict__ in = static_cast<const uint64_t *>(a.col_in[c]) + (tile0 + lbase);
        uint64_t x[HI];
#pragma unroll
        for (int r = 0; r < HI; ++r) x[r] = GJ_VALID(r) ? in[r * kWave] : 0ull;
        __syncthreads();  // both buffers free
#pragma unroll
        for (int r = 0; r < HI; ++r)
            if (GJ_VALID(r)) s8[GJ_POS(r)] = x[r];
#pragma unroll
        for (int r = 0; r < HI; ++r) x[r] = GJ_VALID(HI + r) ? in[(HI + r) * kWave] : 0ull;
#pragma unroll
        for (int r = 0; r < HI; ++r)
            if (GJ_VALID(HI + r)) s8[GJ_POS(HI + r)] = x[r];
        __syncthreads();
        uint64_t *__restrict__ out = static_cast<uint64_t *>(a.col_out[c]);
#pragma unroll
        for (int k = 0; k < ITEMS; ++k)
            if (dst[k] != 0xFFFFFFFFu) out[dst[k]] = s8[k * BLOCK + tid];
    }
#undef GJ_POS
#undef GJ_VALID
    __syncthreads();
    if (tid < kRadix) S.cur[tid] += S.tot[tid];
    __syncthreads();
}

template <typename K, int BLOCK, int ITEMS>
__global__ __launch_bounds__(BLOCK) void k_scatter_wide(PassArgs a) {
    constexpr uint32_t TILE = BLOCK * ITEMS;
    static_assert(BLOCK == 1024, "the wide loads assume 1024 threads");
    __shared__ ScatterShared<BLOCK> S;
    __shared__ uint32_t s_buf[2][TILE];  // double buffer for 4-byte columns; 8-byte data spans both
    __shared__ ChunkLoc s_loc;

    if (threadIdx.x == 0) s_loc = locate_chunk(a, blockIdx.x);
    __syncthreads();
    const ChunkLoc L = s_loc;
    if (!L.ok) return;

    const uint32_t R = 1u << a.bits;
    const uint32_t base_off = seg_begin(a, 0);
    for (uint32_t d = threadIdx.x; d < kRadix; d += BLOCK)
        S.cur[d] = d < R ? base_off + a.hist[L.hbase + d * L.m + L.j] : 0u;
    __syncthreads();
    write_poff(a, L, S.cur, BLOCK);

    const DigitFn dig = seg_digit(a, L.seg);
    K key[ITEMS];
    uint32_t v[ITEMS];
    uint32_t tile0 = L.row0;
    uint32_t nt = min(TILE, L.row1 - tile0);
    if (nt) {
        wide_load_keys<K, ITEMS>(a, tile0, nt, key);
        if (a.n4 > 0) wide_load_col<ITEMS>(a, 0, tile0, nt, v);
    }
    // full tiles, then at most one partial tile (a chunk's last)
    while (nt == TILE) {
        const uint32_t next0 = tile0 + nt;
        const uint32_t next_nt = next0 < L.row1 ? min(TILE, L.row1 - next0) : 0u;
        scatter_tile_wide<K, BLOCK, ITEMS, true>(a, dig, S, s_buf, tile0, nt, key, v, next0, next_nt);
        tile0 = next0;
        nt = next_nt;
    }
    if (nt) scatter_tile_wide<K, BLOCK, ITEMS, false>(a, dig, S, s_buf, tile0, nt, key, v, 0u, 0u);
}

// Whole-line scatter. What bounds the scatter is not how long a tile's run of a
// digit is but whether its two ends share 128-byte lines with other runs: with
// 512-byte runs a write probe moves 5.2 TB/s where they start on a line and 4.1
// where they start anywhere (128-byte runs: 5.1 against 2.8). So this kernel
// writes whole lines of A rows only: a digit's rows past its last full line stay
// in LDS (the carry, one line per digit and column) until a later tile of the
// chunk completes it. Only a chunk's first and last line of each digit are
// written in parts, so chunks are long (several tiles).
//
// Per tile: ranks as in the wide kernel; then, one column at a time, the carried
// rows of every digit with a full line move to the front of the digit's lines in
// the stage, the tile's rows go to their place behind them (or, past the last
// full line, into the carry), and the staged lines leave in 16-byte accesses.
struct LineLds {
    uint8_t *stage;   // the full lines of one column, then the carry of every column (key first)
    uint16_t *wcnt;   // [waves][D]: rows per wave and digit, then their exclusive prefix
    uint32_t *info;   // per digit: stage place of its next new row | end of its lines << 16
    uint4 *pos;       // per digit: output row before and after this tile, first row of the chunk, row of (line 0, value 0)
    uint16_t *lbase;  // first line per digit, D + 1
    uint8_t *tab;     // digit of every line
    uint32_t *tmp;
};
// The bytes that line_lds_bytes counts.
__device__ __forceinline__ LineLds line_lds(uint8_t *p, uint32_t D, uint32_t A, uint32_t row_bytes, uint32_t tile,
                                            uint32_t w) {
    LineLds S;
    S.stage = p;
    p += (size_t)line_max(D, A, tile) * A * w + (size_t)D * A * row_bytes;
    S.pos = reinterpret_cast<uint4 *>(p);
    p += (size_t)D * 16;
    S.wcnt = reinterpret_cast<uint16_t *>(p);
    p += align16((size_t)kLineWaves * D * 2);
    S.info = reinterpret_cast<uint32_t *>(p);
    p += align16((size_t)D * 4);
    S.lbase = reinterpret_cast<uint16_t *>(p);
    p += align16((size_t)(D + 1) * 2);
    S.tab = p;
    p += align16(line_max(D, A, tile));
    S.tmp = reinterpret_cast<uint32_t *>(p);
    return S;
}

// Lanes of the wave with this lane's digit of at most B bits (bits past the
// digit's are equal in all lanes). Four vector instructions a bit.
template <int B>
__device__ __forceinline__ uint64_t match_digit(uint32_t d) {
    uint32_t lo = 0, hi = 0;  // lanes that differ
#pragma unroll
    for (int k = 0; k < B; ++k) {
        uint32_t s = (uint32_t)__builtin_amdgcn_sbfe((int)d, k, 1);
        asm("" : "+v"(s));  // the ballot compares this value; no second shift
        const uint64_t bk = __ballot(s != 0);
        lo |= (uint32_t)bk ^ s;
        hi |= (uint32_t)(bk >> 32) ^ s;
    }
    return ~((uint64_t)hi << 32 | lo);
}

// Stable ranks of the wave's rows among its rows of the same digit, in input
// order: rank | digit << 16 per row; wc counts the wave's rows per digit. Rows
// from lrem on (r * 64 >= lrem) are not counted.
template <typename K, int ITEMS, int B>
__device__ __forceinline__ void line_rank(const DigitFn &dig, const K (&key)[ITEMS], uint32_t lrem, uint16_t *wc,
                                          uint32_t (&pos)[ITEMS]) {
    if (dig.mode == kDigitHash) {
#pragma unroll
        for (int r = 0; r < ITEMS; ++r) pos[r] = (uint32_t)(digit_source<K>(key[r], kDigitHash) >> dig.shift) & dig.mask;
    } else {
        using U = std::make_unsigned_t<K>;
        const U flip = dig.mode == kDigitOrdered ? U(1) << (8 * sizeof(K) - 1) : U(0);
#pragma unroll
        for (int r = 0; r < ITEMS; ++r) pos[r] = (uint32_t)(((U)key[r] ^ flip) >> dig.shift) & dig.mask;
    }
#pragma unroll
    for (int r = 0; r < ITEMS; ++r) {
        const uint32_t d = pos[r];
        const bool valid = (uint32_t)(r * kWave) < lrem;
        const uint64_t peers = match_digit<B>(d) & __ballot(valid);
        const uint32_t rk = rank_below(peers);
        const uint32_t b = wc[d];
        if (valid && rk == 0) wc[d] = (uint16_t)(b + (uint32_t)__popcll(peers));
        pos[r] = (b + rk) | d << 16;
        // rows one after another: their lane masks together would not fit the registers
        __builtin_amdgcn_sched_barrier(0);
    }
}

template <typename T, int ITEMS>
__device__ __forceinline__ void line_load(const T *__restrict__ in, uint32_t tile0, uint32_t nt, T (&v)[ITEMS]) {
    constexpr uint32_t TILE = 1024u * ITEMS;
    const uint32_t lbase = (uint32_t)((threadIdx.x / kWave) * kWave * ITEMS + lane_id());
    const T *__restrict__ p = in + (tile0 + lbase);
    if (nt == TILE) {
#pragma unroll
        for (int r = 0; r < ITEMS; ++r) v[r] = p[r * kWave];
    } else {
        const uint32_t rem = nt > lbase ? nt - lbase : 0u;
#pragma unroll
        for (int r = 0; r < ITEMS; ++r) v[r] = (uint32_t)(r * kWave) < rem ? p[r * kWave] : T(0);
    }
}

// A column's values of one tile, 4 or 8 bytes wide, in one raw register array.
template <int ITEMS, bool WIDE>
__device__ __forceinline__ void line_load_col(const PassArgs &a, int c, uint32_t tile0, uint32_t nt,
                                              uint32_t (&v)[WIDE ? 2 * ITEMS : ITEMS]) {
    if (c == a.rowid_col) {
        const uint32_t lbase = (uint32_t)((threadIdx.x / kWave) * kWave * ITEMS + lane_id());
#pragma unroll
        for (int r = 0; r < ITEMS; ++r) v[r] = tile0 + lbase + r * kWave;
        return;
    }
    if (!WIDE || c < a.n4) {
        uint32_t x[ITEMS];
        line_load<uint32_t, ITEMS>(static_cast<const uint32_t *>(a.col_in[c]), tile0, nt, x);
#pragma unroll
        for (int r = 0; r < ITEMS; ++r) v[r] = x[r];
    } else if constexpr (WIDE) {
        uint64_t x[ITEMS];
        line_load<uint64_t, ITEMS>(static_cast<const uint64_t *>(a.col_in[c]), tile0, nt, x);
#pragma unroll
        for (int r = 0; r < ITEMS; ++r) {
            v[r] = (uint32_t)x[r];
            v[ITEMS + r] = (uint32_t)(x[r] >> 32);
        }
    }
}

// What one tile's columns share: the stage or carry place of each row (two to a
// register), the output row of each of this thread's runs of four staged values,
// and where its carry slots move.
template <int ITEMS, int NS, int NV>
struct LineMap {
    uint32_t pp[ITEMS / 2];
    uint32_t dst[NV];   // 0xFFFFFFFF: past the tile's lines
    uint32_t part;      // bit k: run k starts before the chunk's first row of its digit
    uint16_t move[NS];  // stage place of carry slot k * 1024 + tid, or 0xFFFF
};

// One column's staged lines to global memory, four values a thread and step.
template <typename T, int ITEMS, int NS, int NV, int A>
__device__ __forceinline__ void line_flush(const LineLds &S, const LineMap<ITEMS, NS, NV> &m, T *__restrict__ out) {
    const T *stage = reinterpret_cast<const T *>(S.stage);
#pragma unroll
    for (int k = 0; k < NV; ++k) {
        const uint32_t row = m.dst[k];
        if (row == 0xFFFFFFFFu) continue;
        const uint32_t e = (uint32_t)(k * 1024 + threadIdx.x) * 4;
        T x[4];
        load_run16<T, 4>(stage + e, x);
        if ((m.part >> k) & 1u) {
            const uint32_t first = S.pos[S.tab[e / A]].z;
#pragma unroll
            for (int i = 0; i < 4; ++i)
                if (row + i >= first) out[row + i] = x[i];
        } else {
            store_run16<T, 4>(out + row, x);
        }
    }
}

// Stages one column: the carried values, then the tile's. Places from cbase on
// are the carry's, coff places further in this column.
template <typename T, int ITEMS, int NS, int NV, typename F>
__device__ __forceinline__ void line_stage(const LineLds &S, const LineMap<ITEMS, NS, NV> &m, uint32_t cbase,
                                           uint32_t coff, const T (&old)[NS], F value) {
    T *stage = reinterpret_cast<T *>(S.stage);
#pragma unroll
    for (int k = 0; k < NS; ++k)
        if (m.move[k] != 0xFFFFu) stage[m.move[k]] = old[k];
#pragma unroll
    for (int r = 0; r < ITEMS; ++r) {
        uint32_t p = (m.pp[r >> 1] >> (16 * (r & 1))) & 0xFFFFu;
        if (p >= cbase) p += coff;
        stage[p] = value(r);
    }
}

// The values in this thread's carry slots of a column.
template <typename T, int NS>
__device__ __forceinline__ void line_old(const T *carry, uint32_t slots, T (&old)[NS]) {
#pragma unroll
    for (int k = 0; k < NS; ++k) old[k] = carry[min((uint32_t)(k * 1024 + threadIdx.x), slots - 1)];
}

// ITEMS rows per thread and tile, lines of A rows; WIDE: the key or some column
// has 8 bytes; NS carry slots per thread (D * A <= 1024 * NS).
template <typename K, int ITEMS, int A, bool WIDE, int NS>
__device__ __forceinline__ void scatter_tile_lines(const PassArgs &a, const DigitFn &dig, const LineLds &S, uint32_t D,
                                                   uint32_t tile0, uint32_t nt, K (&key)[ITEMS],
                                                   uint32_t (&v)[WIDE ? 2 * ITEMS : ITEMS], uint32_t next0,
                                                   uint32_t next_nt) {
    constexpr uint32_t TILE = 1024u * ITEMS;
    constexpr int NV = (int)((TILE + 1024u * NS + 4095) / 4096);  // runs of four values per thread
    int tid = threadIdx.x;
    asm volatile("" : "+v"(tid));  // nothing derived from it is hoisted out of the tile loop
    const int w = tid / kWave, lane = tid % kWave;
    const uint32_t lbase = (uint32_t)(w * kWave * ITEMS + lane);
    const uint32_t lrem = nt > lbase ? nt - lbase : 0u;
    const uint32_t cbase = line_max(D, A, TILE) * A;  // places of the lines; the carry's follow
    constexpr uint32_t SW = WIDE ? 8 : 4;
    uint32_t *words = reinterpret_cast<uint32_t *>(S.wcnt);
    for (uint32_t i = tid; i < kLineWaves * D / 2; i += 1024) words[i] = 0;
    const uint8_t *carry = S.stage + (size_t)cbase * SW;
    __syncthreads();
    uint32_t pos[ITEMS];
    uint16_t *wc = S.wcnt + (uint32_t)w * D;
    line_rank<K, ITEMS, A == 32 && NS == 4 ? 7 : 8>(dig, key, lrem, wc, pos);
    __syncthreads();
    // per digit: rows and full lines of this tile, and the lines' exclusive prefix
    uint32_t lines = 0, pre = 0;
    uint4 q = make_uint4(0, 0, 0, 0);
    if ((uint32_t)tid < kRadix) {
        if ((uint32_t)tid < D) {
            uint32_t t = 0;
#pragma unroll
            for (int x = 0; x < kLineWaves; ++x) {
                const uint32_t c = S.wcnt[x * D + tid];
                S.wcnt[x * D + tid] = (uint16_t)t;
                t += c;
            }
            q = S.pos[tid];
            q.x = q.y;
            q.y += t;
            lines = q.y / A - q.x / A;
        }
        const uint32_t inc = wave_inclusive_sum<uint32_t>(lines);
        if (lane == kWave - 1) S.tmp[w] = inc;
        pre = inc - lines;
    }
    __syncthreads();
    if ((uint32_t)tid < D) {
#pragma unroll
        for (int x = 0; x < kRadix / kWave; ++x) pre += (x < w) ? S.tmp[x] : 0u;
        q.w = q.x / A * A - pre * A;
        S.pos[tid] = q;
        S.info[tid] = (pre * A + q.x % A) | (pre + lines) * A << 16;
        S.lbase[tid] = (uint16_t)pre;
        if ((uint32_t)tid == D - 1) S.lbase[D] = (uint16_t)(pre + lines);
    }
    K kold[NS];
    line_old<K, NS>(reinterpret_cast<const K *>(carry), D * A, kold);
    __syncthreads();
    LineMap<ITEMS, NS, NV> m;
#pragma unroll
    for (int r = 0; r < ITEMS; ++r) {
        const uint32_t d = pos[r] >> 16;
        const uint32_t f = S.info[d], end = f >> 16;
        uint32_t p = (f & 0xFFFFu) + wc[d] + (pos[r] & 0xFFFFu);
        if (p >= end) p = cbase + d * A + (p - end);
        if ((uint32_t)(r * kWave) >= lrem) p = cbase - 1;  // no row: a place past the lines
        if (r & 1) m.pp[r >> 1] |= p << 16;
        else m.pp[r >> 1] = p;
    }
#pragma unroll
    for (int k = 0; k < NS; ++k) {
        const uint32_t s = (uint32_t)(k * 1024 + tid), d = s / A;
        m.move[k] = 0xFFFFu;
        if (d < D) {
            const uint32_t l = S.lbase[d];
            if (s % A < S.pos[d].x % A && S.lbase[d + 1] > l) m.move[k] = (uint16_t)(l * A + s % A);
        }
    }
    // the places of this thread's runs: the line's digit by binary search, the run's output row from it
    const uint32_t nl = S.lbase[D];
    for (uint32_t l = tid; l < nl; l += 1024) {
        uint32_t lo = 0, hi = D;  // lbase[lo] <= l < lbase[hi]
        while (hi - lo > 1) {
            const uint32_t mid = (lo + hi) >> 1;
            if (S.lbase[mid] <= l) lo = mid;
            else hi = mid;
        }
        S.tab[l] = (uint8_t)lo;
    }
    // Place p of the carry of a T column lies at LDS byte cbase * SW + coff + (p - cbase) * sizeof(T).
    line_stage<K, ITEMS, NS, NV>(S, m, cbase, cbase * SW / (uint32_t)sizeof(K) - cbase, kold,
                                 [&](int r) { return key[r]; });
    if (next_nt) line_load<K, ITEMS>(static_cast<const K *>(a.key_in), next0, next_nt, key);
    __syncthreads();
    m.part = 0;
#pragma unroll
    for (int k = 0; k < NV; ++k) {
        const uint32_t e = (uint32_t)(k * 1024 + tid) * 4;
        m.dst[k] = 0xFFFFFFFFu;
        if (e < nl * A) {
            const uint4 f = S.pos[S.tab[e / A]];
            const uint32_t row = f.w + e;
            if (row < f.z) m.part |= 1u << k;
            if (row + 3 < a.n_rows) m.dst[k] = row;  // always true when the offsets are right
        }
    }
    line_flush<K, ITEMS, NS, NV, A>(S, m, static_cast<K *>(a.key_out));
    uint32_t coff = D * A * (uint32_t)sizeof(K);  // bytes of the carry before the column's
#pragma unroll 1
    for (int c = 0; c < a.ncols; ++c) {
        const bool more = c + 1 < a.ncols;
        // once v is staged: the next column of this tile, or the next tile's first one
        const auto load_next = [&]() {
            if (more || next_nt)
                line_load_col<ITEMS, WIDE>(a, more ? c + 1 : 0, more ? tile0 : next0, more ? nt : next_nt, v);
        };
        // the carried values leave the carry before this tile's replace them
        if (!WIDE || c < a.n4) {
            uint32_t old[NS];
            line_old<uint32_t, NS>(reinterpret_cast<const uint32_t *>(carry + coff), D * A, old);
            __syncthreads();
            line_stage<uint32_t, ITEMS, NS, NV>(S, m, cbase, (cbase * SW + coff) / 4 - cbase, old,
                                                [&](int r) { return v[r]; });
            load_next();
            __syncthreads();
            line_flush<uint32_t, ITEMS, NS, NV, A>(S, m, static_cast<uint32_t *>(a.col_out[c]));
            coff += D * A * 4;
        } else if constexpr (WIDE) {
            uint64_t old[NS];
            line_old<uint64_t, NS>(reinterpret_cast<const uint64_t *>(carry + coff), D * A, old);
            __syncthreads();
            line_stage<uint64_t, ITEMS, NS, NV>(S, m, cbase, (cbase * SW + coff) / 8 - cbase, old,
                                                [&](int r) { return (uint64_t)v[ITEMS + r] << 32 | v[r]; });
            load_next();
            __syncthreads();
            line_flush<uint64_t, ITEMS, NS, NV, A>(S, m, static_cast<uint64_t *>(a.col_out[c]));
            coff += D * A * 8;
        }
    }
    __syncthreads();  // the next tile stages its keys, and the ranks' counters restart
}

// The rows left in the carry at the end of a chunk.
template <typename T, int A>
__device__ __forceinline__ void line_rest(const LineLds &S, uint32_t D, const T *carry, T *__restrict__ out,
                                          uint32_t n_rows) {
    uint32_t s = threadIdx.x;
    asm volatile("" : "+v"(s));  // not hoisted out of the loop over chunks
    for (; s < D * A; s += 1024) {
        const uint4 q = S.pos[s / A];
        const uint32_t row = q.y / A * A + s % A;
        if (row < q.y && row >= q.z && row < n_rows) out[row] = carry[s];
    }
}

// One chunk: its tiles, then what is left in the carry.
template <typename K, int ITEMS, int A, bool WIDE, int NS>
__device__ __forceinline__ void scatter_chunk_lines(const PassArgs &a, const ChunkLoc &L, const LineLds &S, uint32_t D) {
    constexpr uint32_t TILE = 1024u * ITEMS;
    constexpr uint32_t SW = WIDE ? 8 : 4;
    const uint32_t base_off = uni(seg_begin(a, 0));
    for (uint32_t d = threadIdx.x; d < D; d += 1024) {
        const uint32_t first = base_off + a.hist[L.hbase + d * L.m + L.j];
        S.pos[d] = make_uint4(first, first, first, 0);
        if (a.poff && L.j == 0) a.poff[(L.seg << a.bits) + d] = first;
    }
    if (a.poff && L.j == 0 && !a.seg_off && threadIdx.x == 0) a.poff[D] = a.n_rows;
    const DigitFn dig = seg_digit(a, L.seg);
    K key[ITEMS];
    uint32_t v[WIDE ? 2 * ITEMS : ITEMS];
    uint32_t tile0 = L.row0;
    uint32_t nt = min(TILE, L.row1 - tile0);
    line_load<K, ITEMS>(static_cast<const K *>(a.key_in), tile0, nt, key);
    if (a.ncols > 0) line_load_col<ITEMS, WIDE>(a, 0, tile0, nt, v);
    while (nt) {
        const uint32_t next0 = tile0 + nt;
        const uint32_t next_nt = next0 < L.row1 ? min(TILE, L.row1 - next0) : 0u;
        scatter_tile_lines<K, ITEMS, A, WIDE, NS>(a, dig, S, D, tile0, nt, key, v, next0, next_nt);
        tile0 = next0;
        nt = next_nt;
    }
    const uint8_t *carry = S.stage + (size_t)line_max(D, A, TILE) * A * SW;
    line_rest<K, A>(S, D, reinterpret_cast<const K *>(carry), static_cast<K *>(a.key_out), a.n_rows);
    carry += (size_t)D * A * sizeof(K);
    for (int c = 0; c < a.ncols; ++c) {
        if (c < a.n4) {
            line_rest<uint32_t, A>(S, D, reinterpret_cast<const uint32_t *>(carry), static_cast<uint32_t *>(a.col_out[c]), a.n_rows);
            carry += (size_t)D * A * 4;
        } else {
            line_rest<uint64_t, A>(S, D, reinterpret_cast<const uint64_t *>(carry), static_cast<uint64_t *>(a.col_out[c]), a.n_rows);
            carry += (size_t)D * A * 8;
        }
    }
}

template <typename K, int ITEMS, int A, bool WIDE, int NS>
__global__ __launch_bounds__(1024) void k_scatter_lines(PassArgs a) {
    extern __shared__ uint4 s_dyn4[];
    const uint32_t D = 1u << a.bits;
    const LineLds S = line_lds(reinterpret_cast<uint8_t *>(s_dyn4), D, A, a.row_bytes, 1024u * ITEMS, WIDE ? 8 : 4);
    const uint32_t end = uni(seg_begin(a, 0)) + min((blockIdx.x + 1) * a.chunk_rows, a.n_rows);
    for (uint32_t seg = cell_first_seg(a, blockIdx.x); seg < a.nseg && uni(seg_begin(a, seg)) < end; ++seg) {
        const ChunkLoc L = cell_chunk(a, blockIdx.x, seg);
        if (L.row0 >= L.row1) continue;
        scatter_chunk_lines<K, ITEMS, A, WIDE, NS>(a, L, S, D);
        __syncthreads();
    }
}

// MINW: minimum waves per SIMD the register allocation must allow (4 lets two
// 512-thread workgroups share a compute unit).
template <typename K, int BLOCK, int ITEMS, int G, int MINW>
__global__ __launch_bounds__(BLOCK, MINW) void k_scatter(PassArgs a) {
    constexpr uint32_t TILE = BLOCK * ITEMS;
    __shared__ ScatterShared<BLOCK> S;
    __shared__ uint32_t s_buf[2][TILE];  // double buffer for 4-byte columns; 8-byte data spans both
    __shared__ ChunkLoc s_loc;

    if (threadIdx.x == 0) s_loc = locate_chunk(a, blockIdx.x);
    __syncthreads();
    const ChunkLoc L = s_loc;
    if (!L.ok) return;

    const uint32_t R = 1u << a.bits;
    if (a.off_mode == kOffDirect) {
        direct_offsets<BLOCK>(a, L, S.cur, S.tot, S.tmp);
    } else if (a.off_mode == kOffScanned) {
        const uint32_t base_off = seg_begin(a, 0);
        for (uint32_t d = threadIdx.x; d < kRadix; d += BLOCK)
            S.cur[d] = d < R ? base_off + a.hist[L.hbase + d * L.m + L.j] : 0u;
        __syncthreads();
    }
    if (a.off_mode != kOffSelf) write_poff(a, L, S.cur, BLOCK);

    const DigitFn dig = seg_digit(a, L.seg);
    K key[ITEMS];
    uint32_t tile0 = L.row0;
    uint32_t nt = min(TILE, L.row1 - tile0);
    if (nt) scatter_load_keys<K, BLOCK, ITEMS, G>(a, tile0, nt, key);
    while (nt) {
        const uint32_t next0 = tile0 + nt;
        const uint32_t next_nt = next0 < L.row1 ? min(TILE, L.row1 - next0) : 0u;
        scatter_tile<K, BLOCK, ITEMS, G>(a, L, dig, S, s_buf, tile0, nt, key, next0, next_nt);
        tile0 = next0;
        nt = next_nt;
    }
}

// Scatter tile shapes (rows per thread x 4-byte columns loaded together). The
// shape changes speed only; GJ_SCATTER_SHAPE=<items>x<group> picks one.
using Shape = TileShape;
// Group 0 is the wide-tile kernel (one column at a time, rolling prefetch).
constexpr Shape kVariants[kScatterVariants] = {{256, 8, 4},  {512, 8, 4},  {1024, 8, 4}, {512, 4, 4},
                                               {1024, 4, 4}, {256, 16, 2}, {512, 8, 2},  {512, 16, 2},
                                               {512, 16, 4}, {1024, 8, 2},  {1024, 16, 2}, {1024, 16, 1},
                                               {512, 16, 1}, {1024, 16, 0}};
thread_local int g_variant = 0;

Shape scatter_shape() {
    if (g_variant >= 1 && g_variant <= kScatterVariants) return kVariants[g_variant - 1];
    static Shape sh = [] {
        Shape x{kScatterBlock, kItems, kGroup};
        if (const char *e = getenv("GJ_SCATTER_SHAPE")) {
            int b = 0, i = 0, g = 0;
            if (sscanf(e, "%dx%dx%d", &b, &i, &g) == 3) x = Shape{b, i, g};
        }
        return x;
    }();
    return sh;
}

// The shape of a pass over n rows in nseg segments: the one asked for, else tile_shape's.
Shape pass_shape(uint32_t n, uint32_t nseg, int bits, int key_bytes, uint32_t row_bytes, bool narrow) {
    const Shape sh = scatter_shape();
    return sh.group >= 0 ? sh : tile_shape(n, nseg, bits, key_bytes, row_bytes, narrow);
}

// The whole-line kernel's launch for a pass of shape sh (line_shape).
template <typename K>
void launch_lines(const LineShape &sh, bool narrow, dim3 grid, hipStream_t s, const PassArgs &a, double bytes) {
    const uint32_t D = 1u << a.bits;
    const size_t lds = line_lds_bytes(D, (uint32_t)sh.rows, a.row_bytes, 1024u * (uint32_t)sh.items, narrow ? 4 : 8);
#define GJ_LN(I, A_, W)                                                                                              \
    if (narrow != W && sh.items == I && sh.rows == A_) {                                                             \
        GJ_LAUNCH("k_scatter", bytes, (k_scatter_lines<K, I, A_, W, kLineSlots>), grid, dim3(1024), lds, s, a);      \
        return;                                                                                                      \
    }
    if constexpr (sizeof(K) == 4) {
        GJ_LN(14, 32, false) GJ_LN(14, 16, false) GJ_LN(8, 16, false)
    }
    GJ_LN(8, 32, true) GJ_LN(8, 16, true)
#undef GJ_LN
    throw Error(GJ_EINVAL, "unknown line shape");
}

template <typename K>
void launch_scatter(const Shape &sh, dim3 grid, hipStream_t s, const PassArgs &a, double bytes) {
#define GJ_SC(B, I, G_)                                                                    \
    if (sh.block == B && sh.items == I && sh.group == G_) {                                \
        GJ_LAUNCH("k_scatter", bytes, (k_scatter<K, B, I, G_, (B == 512 && I == 16 && G_ == 1) ? 4 : 1>), grid, \
                  dim3(B), 0, s, a);                                                       \
        return;                                                                            \
    }
    GJ_SC(256, 8, 4) GJ_SC(512, 8, 4) GJ_SC(1024, 8, 4) GJ_SC(512, 4, 4) GJ_SC(1024, 4, 4)
    GJ_SC(256, 16, 2) GJ_SC(512, 8, 2) GJ_SC(512, 16, 2) GJ_SC(512, 16, 4) GJ_SC(1024, 8, 2)
    GJ_SC(1024, 16, 2) GJ_SC(1024, 16, 1) GJ_SC(512, 16, 1)
#undef GJ_SC
    if (sh.block == 1024 && sh.items == 16 && sh.group <= 0) {
        GJ_LAUNCH("k_scatter", bytes, (k_scatter_wide<K, 1024, 16>), grid, dim3(1024), 0, s, a);
        return;
    }
    throw Error(GJ_EINVAL, "unknown scatter shape");
}

// Fills the column part of PassArgs: 4-byte columns first (the scatter loads them in
// groups), then 8-byte ones. cin/cout are indexed by logical column (the row id, if
// generated, is column cols.n); map[c] receives the slot of logical column c.
void assign_cols(PassArgs &a, const PartCols &cols, const void *const *cin, void *const *cout, bool first_pass,
                 int *map) {
    const int ncols = cols.n + (cols.gen_rowid ? 1 : 0);
    a.ncols = ncols;
    a.rowid_col = -1;
    a.n4 = 0;
    int slot = 0;
    for (int pass4 = 1; pass4 >= 0; --pass4) {
        for (int c = 0; c < ncols; ++c) {
            const bool is_rowid = cols.gen_rowid && c == cols.n;
            const int w = is_rowid ? 4 : cols.width[c];
            if ((w == 4) != (pass4 == 1)) continue;
            a.col_w[slot] = w;
            a.col_in[slot] = cin[c];
            a.col_out[slot] = cout[c];
            // the row id is generated in the first pass and moved like a payload afterwards
            if (is_rowid && first_pass) a.rowid_col = slot;
            map[c] = slot;
            if (w == 4) a.n4++;
            ++slot;
        }
    }
}

template <typename K>
__global__ __launch_bounds__(256) void k_key_bits(const K *__restrict__ keys, uint32_t n, unsigned long long *__restrict__ acc) {
    // OR and AND of the order-preserving key bits over all keys, 16 loads in
    // flight per thread
    constexpr int U = 16;
    unsigned long long o = 0, x = ~0ull;
    const uint32_t step = gridDim.x * blockDim.x;
    for (uint32_t base = blockIdx.x * blockDim.x * U + threadIdx.x; base < n; base += step * U) {
        K k[U];
#pragma unroll
        for (int u = 0; u < U; ++u) {
            const uint32_t i = base + u * blockDim.x;
            k[u] = i < n ? keys[i] : keys[base];
        }
#pragma unroll
        for (int u = 0; u < U; ++u) {
            const unsigned long long v = digit_source<K>(k[u], kDigitOrdered);
            o |= v;
            x &= v;
        }
    }
    __shared__ unsigned long long s_bits[2 * (256 / kWave)];
    fold_key_bits<256 / kWave>(o, x, s_bits, acc);
}

// Rows per chunk: long ones, one for each of the 256 compute units (chunks share
// lines at their ends: 2^27 rows, 7 bits: 1.12 ms with 256 chunks, 1.20 with
// 1024); else one tile, at most ~4096 chunks.
uint32_t chunk_rows_for(uint32_t n, const Shape &sh, bool cells) {
    if (cells) return ceil_div_u32(ceil_div_u32(n, 256), 1024) * 1024;
    const uint32_t tile = (uint32_t)(sh.block * sh.items);
    const uint32_t tiles = ceil_div_u32(n, tile);
    const uint32_t per = tiles > 4096 ? ceil_div_u32(tiles, 4096) : 1;
    return per * tile;
}

// Counts a chunk's workgroup may sum itself instead of a scan (kOffDirect): 64 KB
// of them from L2 take about a microsecond, a scan's launch about five.
constexpr uint64_t kDirectCounts = 16384;

// Long chunks belong to the default shape.
bool long_chunks_for(uint32_t n, uint32_t nseg, int bits, uint32_t row_bytes, bool narrow, bool aligned) {
    return scatter_shape().group < 0 && long_chunks(n, nseg, bits, row_bytes, narrow, aligned);
}

// counts: what an earlier kernel counted per chunk; the pass then takes its chunks.
template <typename K>
void run_pass(Ctx &ctx, PassArgs &a, uint32_t n, const PassCounts *counts = nullptr) {
    hipStream_t s = ctx.stream;
    const uint32_t R = 1u << a.bits;
    a.row_bytes = (uint32_t)sizeof(K);
    for (int c = 0; c < a.ncols; ++c) a.row_bytes += (uint32_t)a.col_w[c];
    const bool narrow = sizeof(K) == 4 && a.n4 == a.ncols;
    uintptr_t at = (uintptr_t)a.key_out;
    for (int c = 0; c < a.ncols; ++c) at |= (uintptr_t)a.col_out[c];
    const bool aligned = (at & 15u) == 0;
    a.cells = counts ? counts->cells : long_chunks_for(n, a.nseg, a.bits, a.row_bytes, narrow, aligned);
    const Shape sh = counts ? counts->tile : pass_shape(n, a.nseg, a.bits, (int)sizeof(K), a.row_bytes, narrow);
    a.chunk_rows = counts ? counts->chunk_rows : chunk_rows_for(n, sh, a.cells);
    a.n_chunks = ceil_div_u32(n, a.chunk_rows);
    const uint64_t max_chunks = a.seg_off ? (uint64_t)a.n_chunks + a.nseg : a.n_chunks;
    // algorithmic bytes of one scatter: read and write the key and every column
    // once (a generated row id is only written)
    double row_bytes = 2.0 * sizeof(K);
    for (int c = 0; c < a.ncols; ++c) row_bytes += (c == a.rowid_col ? 0 : a.col_w[c]) + a.col_w[c];
    const bool tiled = !a.cells && sh.group > 0;  // k_scatter: it can find its offsets itself
    if (tiled && !a.seg_off && a.n_chunks == 1) {
        a.off_mode = kOffSelf;
        launch_scatter<K>(sh, dim3(1), s, a, (double)n * row_bytes);
        return;
    }
    if (a.seg_off) {
        uint32_t *chunk_base = ctx.scratch_n<uint32_t>(a.nseg + 1);
        a.chunk_base = chunk_base;
        GJ_LAUNCH("k_chunk_table", 8.0 * (a.nseg + 1), k_chunk_table, dim3(1), dim3(1024), 0, s, a.seg_off, a.nseg,
                  a.chunk_rows, a.cells, a.bits, chunk_base, a.poff);
    }
    // counts past the chunks in use stay unwritten: a scan carries them to no one
    const uint64_t hn = max_chunks * R;
    uint32_t *hist = ctx.scratch_n<uint32_t>(hn);
    a.hist = hist;
    if (counts) {
        // one segment: chunks 0..m-1, the digit the low bits of the same source
        const uint32_t m = a.n_chunks;
        GJ_LAUNCH("k_fold_hist", 4.0 * m * 256 + 4.0 * m * R, k_fold_hist,
                  dim3(std::min<uint32_t>(ceil_div_u32(R * m, kBlock), 4096)), dim3(kBlock), 0, s, counts->hist8, m, a.bits,
                  hist);
    } else {
        if (a.cells)
            GJ_LAUNCH("k_hist_cells", (double)n * sizeof(K), k_hist_cells<K>, dim3(a.n_chunks), dim3(1024), 0, s, a);
        else
            GJ_LAUNCH("k_hist", (double)n * sizeof(K), k_hist<K>, dim3((uint32_t)max_chunks), dim3(kBlock), 0, s, a);
    }
    if (tiled && hn <= kDirectCounts) a.off_mode = kOffDirect;
    else scan_exclusive_u32(ctx, hist, hist, hn, nullptr);
    const LineShape ls = line_shape(a.bits, a.row_bytes, narrow);
    if (a.cells && aligned && ls.items) launch_lines<K>(ls, narrow, dim3(a.n_chunks), s, a, (double)n * row_bytes);
    else launch_scatter<K>(sh, dim3((uint32_t)max_chunks), s, a, (double)n * row_bytes);
}

}  // namespace

void set_scatter_variant(int v) { g_variant = v; }

PassCounts pass_chunks(uint32_t n, int key_bytes, uint32_t row_bytes, bool narrow) {
    PassCounts c;
    c.tile = pass_shape(n, 1, 8, key_bytes, row_bytes, narrow);
    c.cells = long_chunks_for(n, 1, 8, row_bytes, narrow, true);
    c.chunk_rows = chunk_rows_for(n, c.tile, c.cells);
    // the counting workgroups, one a chunk, each fold a kilobyte of registers into the call's:
    // two small tiles a chunk from 2^20 rows (2^22 8-byte keys: 57 us with one, 30 with two)
    if (!c.cells && n > 1u << 20) c.chunk_rows = std::max<uint32_t>(c.chunk_rows, 4096);
    return c;
}

void partition_run(Ctx &ctx, int key_bytes, const void *key_in, void *key_out, const PartCols &cols,
                   uint32_t n, int bit_lo, int bits, int passes, int mode, uint32_t *poff, const PassCounts *counts) {
    require(!counts || (passes == 1 && bit_lo == 0), "a precomputed histogram serves one pass from bit 0");
    require(key_bytes == 4 || key_bytes == 8, "key width must be 4 or 8 bytes");
    require(bits >= 1 && bits <= 16, "partition bits must be 1..16");
    require(passes >= 1 && passes <= 2, "partition passes must be 1 or 2");
    require(bits <= 8 * passes, "at most 8 bits per pass");
    require(passes == 1 || bits >= 2, "two passes need at least 2 bits");
    const int ncols = cols.n + (cols.gen_rowid ? 1 : 0);
    require(ncols <= kMaxCols, "too many columns");
    hipStream_t s = ctx.stream;

    int b[2];
    b[0] = passes == 1 ? bits : (bits + 1) / 2;  // pass 1 takes the top bits
    b[1] = bits - b[0];

    // Per-pass output buffers: the last pass writes the caller's buffers.
    const void *kin = key_in;
    const void *cin[kMaxCols];
    for (int c = 0; c < cols.n; ++c) cin[c] = cols.in[c];
    if (cols.gen_rowid) cin[cols.n] = nullptr;

    if (n == 0) {
        fill_u32(s, poff, 0u, (1ull << bits) + 1);
        return;
    }
    int map[kMaxCols];
    const uint32_t *seg = nullptr;  // pass 1: the whole input
    uint32_t nseg = 1;

    for (int p = 0; p < passes; ++p) {
        const bool last = (p == passes - 1);
        PassArgs a{};
        a.key_in = kin;
        a.key_out = last ? key_out : ctx.scratch((size_t)n * key_bytes);
        void *cout[kMaxCols];
        for (int c = 0; c < ncols; ++c) {
            const bool is_rowid = cols.gen_rowid && c == cols.n;
            const int w = is_rowid ? 4 : cols.width[c];
            cout[c] = last ? (is_rowid ? cols.rowid_out : cols.out[c]) : ctx.scratch((size_t)n * w);
        }
        assign_cols(a, cols, cin, cout, p == 0, map);
        const int shift = bit_lo + (p == 0 ? b[1] : 0);
        a.bits = b[p];
        a.dig = DigitFn{mode, shift, (1u << b[p]) - 1u};
        a.seg_off = seg;
        a.nseg = nseg;
        a.n_rows = n;
        const uint64_t np = (uint64_t)nseg << b[p];
        uint32_t *next = last ? poff : ctx.scratch_n<uint32_t>(np + 1);
        a.poff = next;
        if (key_bytes == 4) run_pass<int32_t>(ctx, a, n, counts);
        else run_pass<int64_t>(ctx, a, n, counts);
        seg = next;
        nseg = (uint32_t)np;
        kin = a.key_out;
        for (int c = 0; c < ncols; ++c) cin[c] = a.col_out[map[c]];
    }
}


void sort_run(Ctx &ctx, int key_bytes, const void *key_in, void *key_out, const PartCols &cols, uint32_t n) {
    require(key_bytes == 4 || key_bytes == 8, "key width must be 4 or 8 bytes");
    hipStream_t s = ctx.stream;
    const int ncols = cols.n + (cols.gen_rowid ? 1 : 0);
    // bytes of the order-preserving key that differ between keys; equal bytes need no pass
    std::vector<int> passes;
    if (n > 0) {
        unsigned long long *acc = reinterpret_cast<unsigned long long *>(ctx.scratch_n<uint64_t>(2));
        fill_u64(s, reinterpret_cast<uint64_t *>(acc), 0ull, 1);
        fill_u64(s, reinterpret_cast<uint64_t *>(acc) + 1, ~0ull, 1);
        const uint32_t grid = std::min<uint32_t>(ceil_div_u32(n, 256 * 16), 2048);
        if (key_bytes == 4)
            GJ_LAUNCH("k_key_bits", 4.0 * n, k_key_bits<int32_t>, dim3(grid), dim3(256), 0, s,
                      static_cast<const int32_t *>(key_in), n, acc);
        else
            GJ_LAUNCH("k_key_bits", 8.0 * n, k_key_bits<int64_t>, dim3(grid), dim3(256), 0, s,
                      static_cast<const int64_t *>(key_in), n, acc);
        uint64_t h[2];
        read_back_parts(s, {{h, acc, 16}});
        const uint64_t diff = h[0] ^ h[1];
        for (int b = 0; b < key_bytes; ++b)
            if ((diff >> (8 * b)) & 0xFF) passes.push_back(b);
    }
    if (passes.empty()) passes.push_back(0);  // a pass on an equal digit is a stable copy
    const void *kin = key_in;
    const void *cin[kMaxCols];
    for (int c = 0; c < cols.n; ++c) cin[c] = cols.in[c];
    if (cols.gen_rowid) cin[cols.n] = nullptr;
    void *bufk[2] = {nullptr, nullptr};
    void *bufc[2][kMaxCols];
    const int P = (int)passes.size();
    for (int p = 0; p < P; ++p) {
        const bool last = (p == P - 1);
        PassArgs a{};
        void *cout[kMaxCols];
        void *kout;
        if (last) {
            kout = key_out;
            for (int c = 0; c < ncols; ++c) cout[c] = (cols.gen_rowid && c == cols.n) ? cols.rowid_out : cols.out[c];
        } else {
            const int b = p & 1;
            if (!bufk[b]) {
                bufk[b] = ctx.scratch((size_t)n * key_bytes);
                for (int c = 0; c < ncols; ++c)
                    bufc[b][c] = ctx.scratch((size_t)n * ((cols.gen_rowid && c == cols.n) ? 4 : cols.width[c]));
            }
            kout = bufk[b];
            for (int c = 0; c < ncols; ++c) cout[c] = bufc[b][c];
        }
        a.key_in = kin;
        a.key_out = kout;
        int map[kMaxCols];
        assign_cols(a, cols, cin, cout, p == 0, map);
        a.bits = 8;
        a.dig = DigitFn{kDigitOrdered, 8 * passes[p], 0xFFu};
        a.nseg = 1;
        a.n_rows = n;
        if (n > 0) {
            if (key_bytes == 4) run_pass<int32_t>(ctx, a, n);
            else run_pass<int64_t>(ctx, a, n);
        }
        kin = kout;
        for (int c = 0; c < ncols; ++c) cin[c] = cout[c];
    }
}


void partition_run_segments(Ctx &ctx, int key_bytes, const void *key_in, void *key_out, const PartCols &cols,
                            uint32_t n, const uint32_t *seg_off, uint32_t nseg, const uint8_t *seg_bits,
                            uint32_t *poff, int mode) {
    require(key_bytes == 4 || key_bytes == 8, "key width must be 4 or 8 bytes");
    hipStream_t s = ctx.stream;
    const int ncols = cols.n + (cols.gen_rowid ? 1 : 0);
    require(ncols <= kMaxCols, "too many columns");
    const void *cin[kMaxCols];
    void *cout[kMaxCols];
    for (int c = 0; c < ncols; ++c) {
        const bool is_rowid = cols.gen_rowid && c == cols.n;
        cin[c] = is_rowid ? nullptr : cols.in[c];
        cout[c] = is_rowid ? cols.rowid_out : cols.out[c];
    }
    PassArgs a{};
    a.key_in = key_in;
    a.key_out = key_out;
    int map[kMaxCols];
    assign_cols(a, cols, cin, cout, true, map);
    a.bits = 8;
    a.dig = DigitFn{mode, 0, 0xFFu};
    a.seg_off = seg_off;
    a.nseg = nseg;
    a.n_rows = n;
    a.seg_bits = seg_bits;
    a.poff = poff;
    if (n == 0) fill_u32(s, poff, 0u, ((uint64_t)nseg << 8) + 1);  // every segment is empty at row 0
    else if (key_bytes == 4) run_pass<int32_t>(ctx, a, n);
    else run_pass<int64_t>(ctx, a, n);
}

}  // namespace gj
