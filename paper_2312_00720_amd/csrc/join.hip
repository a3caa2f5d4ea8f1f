// Match finding and materialization of the partitioned hash join
// (Section 4.1.4, steps 2 and 3).
//
// After partitioning, partition p of R and of S are contiguous ranges. Work
// units cut a partition pair into (R block of at most r_block rows) x (S piece
// of at most 2 x table rows), so that an oversized or skewed partition is spread
// over many workgroups (the load balancing of Sections 3.1.2 and 4.1.4). Per
// unit, a workgroup builds a bucketed hash table on the R block in LDS and
// streams the S piece through it. The table has 4096, 8192 or 16384 rows (the
// smallest that holds r_block) and the workgroup 16 table rows per thread.
//
// The output size is unknown (Section 2.2), so a count pass runs first: every
// wave counts its matches and records each S row's match; an exclusive scan
// over (unit, wave) gives every wave its output range. The write pass then
// writes (key, R payloads, S payloads) contiguously. In the common case (one R
// block per partition, at most one match per S row) it streams S with the
// recorded matches and needs no table; otherwise it rebuilds the table and
// enumerates the matches again. GFTR reads payloads from the partitioned
// copies at partition-local positions (clustered), staged in LDS when they
// fit; GFUR reads the original columns through the partitioned row ids
// (unclustered).
//
// In the write pass, chains of the LDS table list R rows in input order, so an
// S row with several matches emits them in R's input order, and the output is
// the same on every run.
#include "internal.hpp"
#include "join_rule.hpp"

namespace gj {
namespace {

constexpr uint32_t kMaxChainSort = 32;
constexpr uint16_t kNoMatch = 0xFFFF;  // blocks hold at most 16384 rows
constexpr uint32_t kPersistentGrid = 4096;  // workgroups of a plan's count and write passes

// Shape of a work unit for a table of BUILD rows: threads, waves, S piece rows,
// bucket-count limit (as many buckets as keys in a table filled to half its
// rows: 2048 for 4096 rows, whose 32 KB of LDS then let four workgroups share a
// compute unit; 4096 for 8192 rows; 8192 for 16384) and probe rounds in flight
// per lane (the larger shapes have at most 128 registers per lane).
template <uint32_t BUILD, int NT>
struct Geo {
    static constexpr uint32_t kBuild = BUILD;
    static constexpr int kThreads = NT;
    static constexpr int kWv = kThreads / kWave;
    static constexpr uint32_t kSPiece = 2 * BUILD;
    static constexpr int kMaxLog2nb = BUILD >= 16384 ? 13 : (BUILD == 4096 ? 11 : 12);
    static constexpr uint32_t kMaxNb = 1u << kMaxLog2nb;
    static constexpr int kRows = (int)BUILD / NT;  // table rows per thread
    static constexpr int kPB = BUILD == 16384 || kRows < 16 ? 8 : 16;  // count pass
    static constexpr int kPBWrite = BUILD == 4096 && kRows == 16 ? 16 : 8;  // LDS write pass
    static constexpr int kPBStream = kRows < 16 ? 8 : 16;  // streaming write passes
    // waves per SIMD the register allocation must allow: the persistent
    // kernels and the one-unit-per-workgroup kernels (two 512-thread
    // workgroups per compute unit)
    static constexpr int kMinW = 4;
    static constexpr int kMinWWrite = BUILD == 4096 ? 3 : 4;
    static constexpr int kMinWEager = BUILD == 4096 ? 1 : 4;  // (1024 threads: at least 4 by themselves)
    // the eager count pass: two 1024-thread workgroups per compute unit when their
    // LDS (sized by the largest R block) fits twice
    static constexpr int kMinWCount = BUILD == 16384 ? 8 : kMinWEager;
    static constexpr int kMinWStaged = BUILD == 4096 ? 2 : 4;
};

struct JoinArgs {
    const void *rkey;
    const void *skey;
    const uint32_t *rpo;
    const uint32_t *spo;
    uint32_t np;
    const uint32_t *ubase;  // exclusive prefix of units per partition
    uint32_t rc;            // R rows per build block (at most the table rows)
    int skip_bits;          // partition bits, excluded from the bucket hash
    uint64_t *wcnt;         // count pass: matches per (unit, wave)
    const uint64_t *woff;   // write pass: output offset per (unit, wave)
    uint64_t t_rows;        // write pass: output rows; every store is checked against it
    void *tkey;
    int nr, ns;
    const void *rp[8];
    int rw[8];
    void *tr[8];
    const void *sp[8];
    int sw[8];
    void *ts[8];
    const int32_t *rrow;  // GFUR: partitioned row ids of R
    const int32_t *srow;  // GFUR: partitioned row ids of S
    const uint8_t *seg_bits;  // batches: partition bits of instance p >> 8 (skip_bits unused)
    const uint8_t *seg_bshift;  // batches: extra LDS bucket bits of instance p >> 8 (else bshift)
    int bshift;                 // LDS buckets = 2^(ceil(log2 rows) + bshift), within the table's limit
    const uint32_t *nunits;     // device: work units (the kernels loop over them)
    const uint32_t *umap;       // partition of every unit (written by k_unit_map)
    uint32_t lds_rows;          // count and LDS write passes: rows of the largest R block
    uint32_t cap_units;         // units beyond this are not processed (a plan's capacity)
    const uint64_t *out_base;   // device: first output row of this call (nullptr = 0)
    // Streaming write path: the count pass records each S row's match (its row
    // in the R block, or kNoMatch), used when every partition has one R block
    // and no S row matches twice; flags[0] / flags[1] mark the contrary.
    uint16_t *midx;
    uint32_t *flags;            // [2]: most R rows in one partition (for LDS staging)
    int lds_if_complex;         // LDS write pass: do nothing unless a flag is set (plans)
    uint32_t rlds_off[8];       // staged passes: byte offset of R column j in LDS
    int rstaged;                // LDS write pass: R columns 0..rstaged-1 have a place there
    uint8_t *wmulti;            // per (unit, wave): lanes with an S row of several matches (count pass)
    const uint64_t *total;      // output rows of all units
};

// Most work units one call may have: unit indices and their scanned offsets
// are 32-bit.
constexpr uint64_t kMaxUnits = 0x7FFFFFFFull;

// Units per partition pair. flags[0]: a partition spans several R blocks;
// flags[2]: most R rows in a partition that S rows probe; flags[3]: the units
// exceed kMaxUnits (their 64-bit total accumulates at flags + 4), and then no
// pass processes any unit, so a wrapped 32-bit scan is never read.
__global__ void k_unit_count(const uint32_t *__restrict__ rpo, const uint32_t *__restrict__ spo,
                             uint32_t np, uint32_t rc, uint32_t spiece, uint32_t *__restrict__ ucnt,
                             uint32_t *__restrict__ flags) {
    unsigned long long *total = reinterpret_cast<unsigned long long *>(flags + 4);
    unsigned long long sum = 0;
    uint32_t most = 0;
    for (uint32_t p = blockIdx.x * blockDim.x + threadIdx.x; p < np; p += gridDim.x * blockDim.x) {
        const uint32_t nr = rpo[p + 1] - rpo[p], ns = spo[p + 1] - spo[p];
        const uint64_t units = (nr && ns) ? (uint64_t)ceil_div_u32(nr, rc) * ceil_div_u32(ns, spiece) : 0ull;
        ucnt[p] = (uint32_t)min<uint64_t>(units, kMaxUnits);
        sum += units;
        if (ns) most = max(most, nr);
    }
    // one set of atomics per wave
#pragma unroll
    for (int d = kWave / 2; d > 0; d >>= 1) {
        sum += __shfl_xor(sum, d, kWave);
        most = max(most, (uint32_t)__shfl_xor(most, d, kWave));
    }
    if (lane_id() == 0 && sum) {
        const unsigned long long before = atomicAdd(total, sum);
        if (before + sum > kMaxUnits) atomicOr(&flags[3], 1u);
        if (most > rc) atomicOr(&flags[0], 1u);  // a partition spans several R blocks
        atomicMax(&flags[2], most);
    }
}

// Unit counts, their prefix, the flags and the unit map of a single join in one
// workgroup: up to kOneKernelUnits units this takes the time of two launches,
// where a fill, a count, a scan and a map are four. The map holds `cap` units.
constexpr uint64_t kOneKernelUnits = 65536;
__global__ __launch_bounds__(1024) void k_join_units(const uint32_t *__restrict__ rpo, const uint32_t *__restrict__ spo,
                                                     uint32_t np, uint32_t rc, uint32_t spiece,
                                                     uint32_t *__restrict__ ubase, uint32_t *__restrict__ flags,
                                                     uint32_t cap, uint32_t *__restrict__ umap) {
    constexpr int W = 1024 / kWave, PER = 4;  // consecutive partitions per thread and round
    __shared__ unsigned long long s_tmp[W];
    __shared__ uint32_t s_most[W];
    unsigned long long carry = 0;
    uint32_t most = 0;
    const int lane = lane_id();
    for (uint32_t base = 0; base < np; base += 1024 * PER) {
        const uint32_t p0 = base + threadIdx.x * PER;
        uint32_t ro[PER + 1], so[PER + 1];
#pragma unroll
        for (int k = 0; k <= PER; ++k) {
            ro[k] = rpo[min(p0 + k, np)];
            so[k] = spo[min(p0 + k, np)];
        }
        unsigned long long u[PER], sum = 0;
#pragma unroll
        for (int k = 0; k < PER; ++k) {
            const uint32_t nr = ro[k + 1] - ro[k], ns = so[k + 1] - so[k];  // 0 past the last partition
            u[k] = (nr && ns) ? (unsigned long long)ceil_div_u32(nr, rc) * ceil_div_u32(ns, spiece) : 0ull;
            sum += u[k];
            if (ns) most = max(most, nr);
        }
        unsigned long long all;
        unsigned long long at = carry + block_exclusive_sum<unsigned long long, W>(sum, s_tmp, &all);
        carry += all;
#pragma unroll
        for (int k = 0; k < PER; ++k) {
            const uint32_t first = (uint32_t)min(at, (unsigned long long)kMaxUnits);
            if (p0 + k < np) ubase[p0 + k] = first;
            const uint32_t cnt = at < cap ? (uint32_t)min(u[k], cap - at) : 0u;
            if (cnt <= 4) {
                for (uint32_t i = 0; i < cnt; ++i) umap[first + i] = p0 + k;
            }
            // a partition of many units (skew, few partitions): its wave writes them
            for (uint64_t many = __ballot(cnt > 4); many; many &= many - 1) {
                const int l = __ffsll((long long)many) - 1;
                const uint32_t f = __shfl(first, l, kWave), c = __shfl(cnt, l, kWave), p = __shfl(p0 + k, l, kWave);
                for (uint32_t i = lane; i < c; i += kWave) umap[f + i] = p;
            }
            at += u[k];
        }
    }
#pragma unroll
    for (int d = kWave / 2; d > 0; d >>= 1) most = max(most, (uint32_t)__shfl_xor(most, d, kWave));
    if (lane == 0) s_most[threadIdx.x / kWave] = most;
    __syncthreads();
    if (threadIdx.x == 0) {
        for (int w = 0; w < W; ++w) most = max(most, s_most[w]);
        ubase[np] = (uint32_t)min(carry, (unsigned long long)kMaxUnits);
        flags[0] = most > rc;  // a partition spans several R blocks
        flags[1] = 0;
        flags[2] = most;
        flags[3] = carry > kMaxUnits;
        flags[4] = (uint32_t)carry;
        flags[5] = (uint32_t)(carry >> 32);
    }
}

// Units the passes process: none once the count overflowed, else at most the
// launch's (or plan's) capacity.
__device__ __forceinline__ uint32_t units_to_run(const uint32_t *nunits, const uint32_t *flags, uint32_t cap) {
    return flags[3] ? 0u : min(*nunits, cap);
}

// The partition of every unit to run, found once for all passes: each pass then
// reads it with one load, where a binary search over the unit offsets made a
// workgroup wait on 14 dependent loads per unit at 2^14 partitions.
__global__ void k_unit_map(const uint32_t *__restrict__ ubase, uint32_t np, const uint32_t *__restrict__ nunits,
                           const uint32_t *__restrict__ flags, uint32_t cap, uint32_t *__restrict__ umap) {
    const uint32_t n = units_to_run(nunits, flags, cap);
    for (uint32_t u = blockIdx.x * blockDim.x + threadIdx.x; u < n; u += gridDim.x * blockDim.x) {
        uint32_t lo = 0, hi = np;  // ubase[lo] <= u < ubase[hi]
        while (hi - lo > 1) {
            const uint32_t mid = (lo + hi) >> 1;
            if (ubase[mid] <= u) lo = mid;
            else hi = mid;
        }
        umap[u] = lo;
    }
}

__device__ __forceinline__ void copy_val(void *dst, int dw, uint64_t di, const void *src, uint64_t si) {
    if (dw == 4) static_cast<uint32_t *>(dst)[di] = static_cast<const uint32_t *>(src)[si];
    else static_cast<uint64_t *>(dst)[di] = static_cast<const uint64_t *>(src)[si];
}

// Copies column values src[j][row[r]] to dst[j][pos[r]] for the PB rounds of a
// wave whose flag c[r] is set; all loads of one column are issued before its
// stores, so PB loads per lane are in flight.
template <int PB>
__device__ __forceinline__ void gather_cols(int ncols, const void *const *src, const int *width,
                                            void *const *dst, const uint32_t *row, const uint32_t *c,
                                            const uint64_t *pos, uint64_t t_rows) {
    for (int j = 0; j < ncols; ++j) {
        if (width[j] == 4) {
            const uint32_t *__restrict__ in = static_cast<const uint32_t *>(src[j]);
            uint32_t *__restrict__ out = static_cast<uint32_t *>(dst[j]);
            uint32_t v[PB];
#pragma unroll
            for (int r = 0; r < PB; ++r) v[r] = c[r] ? in[row[r]] : 0u;
#pragma unroll
            for (int r = 0; r < PB; ++r)
                if (c[r] && pos[r] < t_rows) out[pos[r]] = v[r];
        } else {
            const uint64_t *__restrict__ in = static_cast<const uint64_t *>(src[j]);
            uint64_t *__restrict__ out = static_cast<uint64_t *>(dst[j]);
            uint64_t v[PB];
#pragma unroll
            for (int r = 0; r < PB; ++r) v[r] = c[r] ? in[row[r]] : 0ull;
#pragma unroll
            for (int r = 0; r < PB; ++r)
                if (c[r] && pos[r] < t_rows) out[pos[r]] = v[r];
        }
    }
}

// Column moves of the streaming passes. Rows whose lrow[r] is ~0 have no match;
// output row = wbase + pos[r] (a 32-bit offset within the wave's range), dropped
// unless pos[r] < lim. gather_cols_wave reads src[j][rbase + row[r]];
// stream_cols_contig reads the contiguous rows row0 + r * 64 (one base address).
template <int PB>
__device__ __forceinline__ void gather_cols_wave(int ncols, const void *const *src, const int *width,
                                                 void *const *dst, uint32_t rbase,
                                                 const uint32_t *row, const uint32_t *lrow, const uint32_t *pos,
                                                 uint64_t wbase, uint32_t lim) {
    for (int j = 0; j < ncols; ++j) {
        if (width[j] == 4) {
            const uint32_t *__restrict__ in = static_cast<const uint32_t *>(src[j]) + rbase;
            uint32_t *__restrict__ out = static_cast<uint32_t *>(dst[j]) + wbase;
            uint32_t v[PB];
#pragma unroll
            for (int r = 0; r < PB; ++r) v[r] = lrow[r] != ~0u ? in[row[r]] : 0u;
#pragma unroll
            for (int r = 0; r < PB; ++r)
                if (lrow[r] != ~0u && pos[r] < lim) out[pos[r]] = v[r];
        } else {
            const uint64_t *__restrict__ in = static_cast<const uint64_t *>(src[j]) + rbase;
            uint64_t *__restrict__ out = static_cast<uint64_t *>(dst[j]) + wbase;
            uint64_t v[PB];
#pragma unroll
            for (int r = 0; r < PB; ++r) v[r] = lrow[r] != ~0u ? in[row[r]] : 0ull;
#pragma unroll
            for (int r = 0; r < PB; ++r)
                if (lrow[r] != ~0u && pos[r] < lim) out[pos[r]] = v[r];
        }
    }
}

template <int PB>
__device__ __forceinline__ void stream_cols_contig(int ncols, const void *const *src, const int *width,
                                                   void *const *dst, uint32_t row0, const uint32_t *lrow,
                                                   const uint32_t *pos, uint64_t wbase, uint32_t lim) {
    for (int j = 0; j < ncols; ++j) {
        if (width[j] == 4) {
            const uint32_t *__restrict__ in = static_cast<const uint32_t *>(src[j]) + row0;
            uint32_t *__restrict__ out = static_cast<uint32_t *>(dst[j]) + wbase;
            uint32_t v[PB];
#pragma unroll
            for (int r = 0; r < PB; ++r) v[r] = lrow[r] != ~0u ? in[r * kWave] : 0u;
#pragma unroll
            for (int r = 0; r < PB; ++r)
                if (lrow[r] != ~0u && pos[r] < lim) out[pos[r]] = v[r];
        } else {
            const uint64_t *__restrict__ in = static_cast<const uint64_t *>(src[j]) + row0;
            uint64_t *__restrict__ out = static_cast<uint64_t *>(dst[j]) + wbase;
            uint64_t v[PB];
#pragma unroll
            for (int r = 0; r < PB; ++r) v[r] = lrow[r] != ~0u ? in[r * kWave] : 0ull;
#pragma unroll
            for (int r = 0; r < PB; ++r)
                if (lrow[r] != ~0u && pos[r] < lim) out[pos[r]] = v[r];
        }
    }
}

// LDS of a count or LDS-write unit, carved from dynamic shared memory for R
// blocks of at most `rows` rows (the largest block the call has, known after the
// unit count): the block's keys and rows, the bucket bounds (16-bit: a block
// holds at most 16384 rows) and a few words of workgroup state. Blocks of about
// 8192 rows then take 64-68 KB, and two 1024-thread workgroups share a compute
// unit, one building or loading while the other probes.
template <typename K>
struct JoinLds {
    K *rkey;         // R block keys: input order while building, bucket order after
    uint16_t *entry; // R block rows, grouped by bucket
    uint16_t *b;     // bucket boundaries
    uint32_t *tmp;   // kWv words
    uint32_t *unit;  // 6 words
    int *is_long;    // a bucket is too long to sort; then: some wave writes in output order
};
constexpr size_t align8(size_t x) { return (x + 7) & ~(size_t)7; }
template <typename K, uint32_t BUILD, int NT>
constexpr size_t join_lds_bytes(uint32_t rows) {
    return align8((size_t)rows * sizeof(K)) + align8((size_t)rows * 2) + align8(((size_t)Geo<BUILD, NT>::kMaxNb + 1) * 2) +
           4 * ((size_t)Geo<BUILD, NT>::kWv + 8);
}
template <typename K, uint32_t BUILD, int NT>
__device__ __forceinline__ JoinLds<K> join_lds(uint8_t *p, uint32_t rows) {
    JoinLds<K> L;
    L.rkey = reinterpret_cast<K *>(p);
    p += align8((size_t)rows * sizeof(K));
    L.entry = reinterpret_cast<uint16_t *>(p);
    p += align8((size_t)rows * 2);
    L.b = reinterpret_cast<uint16_t *>(p);
    p += align8(((size_t)Geo<BUILD, NT>::kMaxNb + 1) * 2);
    L.tmp = reinterpret_cast<uint32_t *>(p);
    L.unit = L.tmp + Geo<BUILD, NT>::kWv;
    L.is_long = reinterpret_cast<int *>(L.unit + 6);
    return L;
}
// 16-bit bucket counters updated through their 32-bit word (no carry or borrow
// crosses the halves: counts stay below 2^16 and never drop below zero).
__device__ __forceinline__ void b16_add1(uint16_t *b, uint32_t i) {
    atomicAdd(reinterpret_cast<uint32_t *>(b) + (i >> 1), 1u << ((i & 1u) * 16u));
}
__device__ __forceinline__ uint32_t b16_dec(uint16_t *b, uint32_t i) {  // the value before
    const uint32_t sh = (i & 1u) * 16u;
    return (atomicSub(reinterpret_cast<uint32_t *>(b) + (i >> 1), 1u << sh) >> sh) & 0xFFFFu;
}

// Build on the R block of unit u and probe it with the unit's S piece: count
// (WRITE = false) or write (WRITE = true) the matches.
// Probes of PB keys against the LDS table, shaped so that the PB lookups are
// independent: bucket bounds, then the first entry of every chain, read for all
// rows at once (clamped indices, so every read is in range); chains longer than
// one entry, rare with at least as many buckets as rows, are walked afterwards.
// c[r] = matches of key r, e1[r] = its first match's entry (bucket order).
template <typename K, int PB>
__device__ __forceinline__ void probe_rows(const K *s_rkey, const uint16_t *s_b, const K (&key)[PB],
                                           const bool (&valid)[PB], int skip_bits, int log2nb, uint32_t rn,
                                           uint32_t (&c)[PB], uint32_t (&e1)[PB]) {
    uint32_t lo[PB], hi[PB];
#pragma unroll
    for (int r = 0; r < PB; ++r) {
        const uint32_t b = bucket_of<K>(key[r], skip_bits, log2nb);
        lo[r] = s_b[b];
        hi[r] = valid[r] ? s_b[b + 1] : lo[r];
    }
#pragma unroll
    for (int r = 0; r < PB; ++r) {
        const K k0 = s_rkey[min(lo[r], rn - 1)];
        c[r] = (lo[r] < hi[r] && k0 == key[r]) ? 1u : 0u;
        e1[r] = lo[r];
    }
#pragma unroll
    for (int r = 0; r < PB; ++r) {
        for (uint32_t e = lo[r] + 1; e < hi[r]; ++e) {
            if (s_rkey[e] == key[r]) {
                if (c[r] == 0) e1[r] = e;
                ++c[r];
            }
        }
    }
}

// Unit u of the (R block) x (S piece) decomposition: s_unit[0..5] = first R
// row, R rows, first S row, S rows, partition bits, extra bucket bits.
template <uint32_t kSPiece>
__device__ __forceinline__ void decode_unit(const JoinArgs &a, uint32_t u, uint32_t *s_unit) {
    const uint32_t p = a.umap[u];
    const uint32_t nr = a.rpo[p + 1] - a.rpo[p], ns = a.spo[p + 1] - a.spo[p];
    const uint32_t nsb = ceil_div_u32(ns, kSPiece);
    const uint32_t local = u - a.ubase[p];
    const uint32_t ra = local / nsb, sb = local % nsb;
    s_unit[0] = a.rpo[p] + ra * a.rc;
    s_unit[1] = min(a.rc, nr - ra * a.rc);
    s_unit[2] = a.spo[p] + sb * kSPiece;
    s_unit[3] = min(kSPiece, ns - sb * kSPiece);
    s_unit[4] = a.seg_bits ? a.seg_bits[p >> 8] : (uint32_t)a.skip_bits;
    s_unit[5] = a.seg_bshift ? a.seg_bshift[p >> 8] : (uint32_t)a.bshift;
}

// Inclusive scan of the nb bucket counts in s_b (s_b[b] = end of bucket b), and
// s_b[nb] = rn.
template <uint32_t BUILD, int NT>
__device__ __forceinline__ void scan_buckets(uint16_t *s_b, uint32_t *s_tmp, uint32_t nb, uint32_t rn) {
    using G = Geo<BUILD, NT>;
    constexpr int per = (int)((G::kMaxNb + G::kThreads - 1) / G::kThreads);
    const uint32_t first = threadIdx.x * per;
    uint32_t v[per];
    uint32_t sum = 0;
#pragma unroll
    for (int k = 0; k < per; ++k) {
        v[k] = (first + k < nb) ? s_b[first + k] : 0u;
        sum += v[k];
    }
    uint32_t run = block_exclusive_sum<uint32_t, G::kWv>(sum, s_tmp, (uint32_t *)nullptr);
#pragma unroll
    for (int k = 0; k < per; ++k) {
        run += v[k];
        if (first + k < nb) s_b[first + k] = (uint16_t)run;
    }
    if (threadIdx.x == 0) s_b[nb] = (uint16_t)rn;
}

// Count pass of unit u: matches per (unit, wave), each S row's match recorded
// for the streaming write pass, and the flag for S rows with several matches.
// The table is built straight into bucket order from registers (the R keys of
// this thread: counts, scan, placement), since counts need no ordered chains;
// the wave's first round of S keys loads during the build.
template <typename K, uint32_t BUILD, int NT>
__device__ __forceinline__ void count_unit(const JoinArgs &a, uint32_t u, const JoinLds<K> &sh) {
    using G = Geo<BUILD, NT>;
    constexpr int PB = G::kPB;
    constexpr int kT = G::kThreads;
    constexpr int kWv = G::kWv;
    constexpr int PER = (int)(BUILD / kT);
    K *s_rkey = sh.rkey;
    uint16_t *s_b = sh.b;
    uint16_t *s_entry = sh.entry;
    uint32_t *s_unit = sh.unit;
    const int tid = threadIdx.x, w = tid / kWave, lane = lane_id();
    if (tid == 0) decode_unit<G::kSPiece>(a, u, s_unit);
    __syncthreads();
    // the unit's shape is uniform: scalar registers (in vector ones they spilled)
    const uint32_t r0 = __builtin_amdgcn_readfirstlane(s_unit[0]), rn = __builtin_amdgcn_readfirstlane(s_unit[1]);
    const uint32_t s0 = __builtin_amdgcn_readfirstlane(s_unit[2]), sn = __builtin_amdgcn_readfirstlane(s_unit[3]);
    const int skip_bits = (int)__builtin_amdgcn_readfirstlane(s_unit[4]);
    int log2nb = 0;
    while ((1u << log2nb) < rn) ++log2nb;
    log2nb = min(log2nb + (int)__builtin_amdgcn_readfirstlane(s_unit[5]), G::kMaxLog2nb);
    const uint32_t nb = 1u << log2nb;

    // loads in flight during the build: this thread's R keys, its wave's first S keys
    const K *__restrict__ rk = static_cast<const K *>(a.rkey) + r0;
    K kr[PER];
#pragma unroll
    for (int k = 0; k < PER; ++k) kr[k] = (uint32_t)(tid + k * kT) < rn ? rk[tid + k * kT] : K(0);
    const uint32_t q = ceil_div_u32(sn, kWv);
    const uint32_t ws = __builtin_amdgcn_readfirstlane(min(sn, w * q)), we = __builtin_amdgcn_readfirstlane(min(sn, ws + q));
    const K *__restrict__ skey = static_cast<const K *>(a.skey) + s0;
    K key[PB];
#pragma unroll
    for (int r = 0; r < PB; ++r) key[r] = ws + r * kWave + lane < we ? skey[ws + r * kWave + lane] : K(0);

    for (uint32_t b = tid; b <= nb; b += kT) s_b[b] = 0;
    __syncthreads();
#pragma unroll
    for (int k = 0; k < PER; ++k)
        if ((uint32_t)(tid + k * kT) < rn) b16_add1(s_b, bucket_of<K>(kr[k], skip_bits, log2nb));
    __syncthreads();
    scan_buckets<BUILD, NT>(s_b, sh.tmp, nb, rn);
    __syncthreads();
    // placement from the end of each bucket; afterwards s_b[b] = start of bucket b
#pragma unroll
    for (int k = 0; k < PER; ++k) {
        if ((uint32_t)(tid + k * kT) < rn) {
            const uint32_t slot = b16_dec(s_b, bucket_of<K>(kr[k], skip_bits, log2nb)) - 1u;
            s_rkey[slot] = kr[k];
            s_entry[slot] = (uint16_t)(tid + k * kT);
        }
    }
    __syncthreads();

    uint32_t cnt = 0;
    bool multi = false;
    for (uint32_t base = ws; base < we; base += PB * kWave) {
        if (base != ws) {
#pragma unroll
            for (int r = 0; r < PB; ++r) key[r] = base + r * kWave + lane < we ? skey[base + r * kWave + lane] : K(0);
        }
        bool valid[PB];
#pragma unroll
        for (int r = 0; r < PB; ++r) valid[r] = base + r * kWave + lane < we;
        uint32_t c[PB], e1[PB];
        probe_rows<K, PB>(s_rkey, s_b, key, valid, skip_bits, log2nb, rn, c, e1);
#pragma unroll
        for (int r = 0; r < PB; ++r) {
            if (valid[r]) {
                cnt += c[r];
                multi |= c[r] > 1;
                if (a.midx) a.midx[s0 + base + r * kWave + lane] = c[r] ? s_entry[e1[r]] : kNoMatch;
            }
        }
    }
    const uint64_t tot = wave_sum<uint64_t>((uint64_t)cnt);
    const uint64_t many = __ballot(multi);
    if (lane == 0) {
        a.wcnt[(uint64_t)u * kWv + w] = tot;
        a.wmulti[(uint64_t)u * kWv + w] = (uint8_t)__popcll(many);
    }
    // one flag for every wave of the pass: an atomic only while it is not set yet
    // (2^24 x 2^24 rows with duplicate keys, 33 thousand waves: 396 -> 89 us)
    if (a.flags && many && lane == 0 &&
        !__hip_atomic_load(&a.flags[1], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT))
        atomicOr(&a.flags[1], 1u);
}

// Columns j0..ncols-1 of U output rows per lane: src[j][row[u]] to dst[j][p + u * 64],
// rows with u * 64 < n only. A column's loads are issued before its stores.
template <int U>
__device__ __forceinline__ void emit_cols(int j0, int ncols, const void *const *src, const int *width,
                                          void *const *dst, const uint32_t (&row)[U], uint64_t p, uint32_t n) {
    for (int j = j0; j < ncols; ++j) {
        if (width[j] == 4) {
            const uint32_t *__restrict__ in = static_cast<const uint32_t *>(src[j]);
            uint32_t *__restrict__ out = static_cast<uint32_t *>(dst[j]) + p;
            uint32_t v[U];
#pragma unroll
            for (int u = 0; u < U; ++u) v[u] = in[row[u]];
#pragma unroll
            for (int u = 0; u < U; ++u)
                if (u * kWave < n) out[u * kWave] = v[u];
        } else {
            const uint64_t *__restrict__ in = static_cast<const uint64_t *>(src[j]);
            uint64_t *__restrict__ out = static_cast<uint64_t *>(dst[j]) + p;
            uint64_t v[U];
#pragma unroll
            for (int u = 0; u < U; ++u) v[u] = in[row[u]];
#pragma unroll
            for (int u = 0; u < U; ++u)
                if (u * kWave < n) out[u * kWave] = v[u];
        }
    }
}

// Matches of S rows [ws, we) of a unit where S rows match several R rows and
// equal keys adjoin in the table's buckets. A wave takes 64 S rows at a time, and then
// its lanes take their output rows, 64 consecutive ones per access: lane o finds the S row
// that owns output o by a search over the rows' exclusive match counts, and its
// match at that distance from the row's first. (Each lane writing the matches of
// its own S row touched eight lines an access where this touches two: 2^24 x 2^24
// rows, four matches each, two payloads a side: 1.5-1.7 ms -> 0.95 ms, 0.80 ms with
// the R payloads in LDS. The waves wait for S payloads and for each other between
// build and probe; LDS and vector units are a quarter busy.)
template <typename K>
__device__ __forceinline__ void write_dups(const JoinArgs &a, const JoinLds<K> &sh, const uint8_t *s_pay, int staged,
                                           uint32_t r0, uint32_t s0, uint32_t ws, uint32_t we, int skip_bits, int log2nb,
                                           uint64_t outpos) {
    constexpr int U = 4;
    const int lane = lane_id();
    const K *__restrict__ skey = static_cast<const K *>(a.skey) + s0;
    K *__restrict__ tkey = static_cast<K *>(a.tkey);
    K next = ws + lane < we ? skey[ws + lane] : K(0);
    for (uint32_t base = ws; base < we; base += kWave) {
        const K key = next;
        const bool valid = base + lane < we;
        if (base + kWave < we) next = base + kWave + lane < we ? skey[base + kWave + lane] : K(0);
        uint32_t c = 0, e1 = 0;
        if (valid) {
            const uint32_t b = bucket_of<K>(key, skip_bits, log2nb);
            const uint32_t hi = sh.b[b + 1];
            e1 = sh.b[b];
            while (e1 < hi && sh.rkey[e1] != key) ++e1;
            uint32_t e2 = e1;
            while (e2 < hi && sh.rkey[e2] == key) ++e2;
            c = e2 - e1;
        }
        const uint32_t incl = wave_inclusive_sum<uint32_t>(c), ex = incl - c;
        const uint32_t t = __builtin_amdgcn_readlane(incl, kWave - 1);
        for (uint32_t o0 = 0; o0 < t; o0 += kWave * U) {
            uint32_t rrow[U], srow[U];
            K kv[U];
            const uint64_t p = outpos + o0 + lane;
            // rows of this lane: those with o0 + lane + u * 64 < t, within the output
            uint32_t n = o0 + lane < t ? t - o0 - lane : 0u;
            n = p < a.t_rows ? (uint32_t)min<uint64_t>(n, a.t_rows - p) : 0u;
#pragma unroll
            for (int u = 0; u < U; ++u) {
                const uint32_t o = min(o0 + lane + u * kWave, t - 1);
                int l = 0;  // the last lane with ex <= o: it has matches
#pragma unroll
                for (int d = kWave / 2; d > 0; d >>= 1) {
                    const uint32_t x = __shfl(ex, l + d, kWave);
                    if (x <= o) l += d;
                }
                const uint32_t e = __shfl(e1, l, kWave) + o - __shfl(ex, l, kWave);
                kv[u] = sh.rkey[e];
                rrow[u] = r0 + sh.entry[e];
                srow[u] = s0 + base + l;
            }
            if (a.srow) {
#pragma unroll
                for (int u = 0; u < U; ++u) {
                    srow[u] = (uint32_t)a.srow[srow[u]];
                    rrow[u] = (uint32_t)a.rrow[rrow[u]];
                }
            }
#pragma unroll
            for (int u = 0; u < U; ++u)
                if (u * kWave < n) tkey[p + u * kWave] = kv[u];
            emit_cols<U>(0, a.ns, a.sp, a.sw, a.ts, srow, p, n);
            for (int j = 0; j < staged; ++j) {
                uint32_t lrow[U];
#pragma unroll
                for (int u = 0; u < U; ++u) lrow[u] = rrow[u] - r0;
                if (a.rw[j] == 4) {
                    const uint32_t *col = reinterpret_cast<const uint32_t *>(s_pay + a.rlds_off[j]);
                    uint32_t *__restrict__ out = static_cast<uint32_t *>(a.tr[j]) + p;
#pragma unroll
                    for (int u = 0; u < U; ++u)
                        if (u * kWave < n) out[u * kWave] = col[lrow[u]];
                } else {
                    const uint64_t *col = reinterpret_cast<const uint64_t *>(s_pay + a.rlds_off[j]);
                    uint64_t *__restrict__ out = static_cast<uint64_t *>(a.tr[j]) + p;
#pragma unroll
                    for (int u = 0; u < U; ++u)
                        if (u * kWave < n) out[u * kWave] = col[lrow[u]];
                }
            }
            emit_cols<U>(staged, a.nr, a.rp, a.rw, a.tr, rrow, p, n);
        }
        outpos += t;
    }
}

// The same matches where some bucket is too long to sort: a bucket's rows are in input
// order, other keys between them. The wave writes the matches of an S row with
// kRowByWave or more by itself, 64 entries of the bucket at a time, consecutive output
// rows together; each lane writes those of its own row otherwise. (Every lane its own: each
// of the 16 waves of a unit wrote to 64 places at once. 2^16 x 2^20 rows, 64 matches each,
// one, two and eight payloads a side, write pass: 2777 -> 535, 4913 -> 828, 25029 -> 2742 us;
// units of four waves took 1936, 4217 and 19942.)
constexpr uint32_t kRowByWave = 8;
template <typename K>
__device__ __forceinline__ void write_long(const JoinArgs &a, const JoinLds<K> &sh, uint32_t r0, uint32_t s0, uint32_t ws,
                                           uint32_t we, int skip_bits, int log2nb, uint64_t outpos) {
    const int lane = lane_id();
    const K *__restrict__ skey = static_cast<const K *>(a.skey) + s0;
    K *__restrict__ tkey = static_cast<K *>(a.tkey);
    const auto write = [&](uint32_t e, K key, uint64_t p, uint64_t sr) {
        const uint32_t ri = r0 + sh.entry[e];
        const uint64_t rr = a.rrow ? (uint64_t)a.rrow[ri] : (uint64_t)ri;
        tkey[p] = key;
        for (int j = 0; j < a.nr; ++j) copy_val(a.tr[j], a.rw[j], p, a.rp[j], rr);
        for (int j = 0; j < a.ns; ++j) copy_val(a.ts[j], a.sw[j], p, a.sp[j], sr);
    };
    for (uint32_t base = ws; base < we; base += kWave) {
        const bool valid = base + lane < we;
        const K key = valid ? skey[base + lane] : K(0);
        const uint32_t b = bucket_of<K>(key, skip_bits, log2nb);
        const uint32_t lo = sh.b[b], hi = sh.b[b + 1];
        uint32_t c = 0;
        if (valid)
            for (uint32_t e = lo; e < hi; ++e) c += sh.rkey[e] == key ? 1u : 0u;
        const uint32_t incl = wave_inclusive_sum<uint32_t>(c), ex = incl - c;
        for (uint64_t rows = __ballot(c >= kRowByWave); rows; rows &= rows - 1) {
            const int l = __ffsll((long long)rows) - 1;
            const K k = __shfl(key, l, kWave);
            const uint32_t si = s0 + base + l, end = __shfl(hi, l, kWave);
            const uint64_t sr = a.srow ? (uint64_t)a.srow[si] : (uint64_t)si;
            uint64_t first = outpos + __shfl(ex, l, kWave);
            for (uint32_t e0 = __shfl(lo, l, kWave); e0 < end; e0 += kWave) {
                const uint32_t e = e0 + lane;
                const bool hit = e < end && sh.rkey[min(e, end - 1)] == k;
                const uint64_t hits = __ballot(hit);
                const uint64_t p = first + rank_below(hits);
                if (hit && p < a.t_rows) write(e, k, p, sr);
                first += (uint64_t)__popcll(hits);
            }
        }
        if (c && c < kRowByWave) {
            const uint32_t si = s0 + base + lane;
            const uint64_t sr = a.srow ? (uint64_t)a.srow[si] : (uint64_t)si;
            uint64_t p = outpos + ex;
            for (uint32_t e = lo; e < hi; ++e) {
                if (sh.rkey[e] != key || p >= a.t_rows) continue;
                write(e, key, p, sr);
                ++p;
            }
        }
        outpos += __builtin_amdgcn_readlane(incl, kWave - 1);
    }
}

// Write pass of unit u on the LDS table (the general case: partitions spanning
// several R blocks, or S rows with several matches): build with chains in row
// order, probe, and write every match at the positions the count pass sized.
template <typename K, uint32_t BUILD, int NT>
__device__ __forceinline__ void write_unit(const JoinArgs &a, uint32_t u, uint64_t out_base, const JoinLds<K> &sh) {
    using G = Geo<BUILD, NT>;
    constexpr int PB = G::kPBWrite;
    constexpr int kBlockT = G::kThreads;
    constexpr int kWv = G::kWv;
    constexpr uint32_t kSPiece = G::kSPiece;
    K *s_rkey = sh.rkey;
    uint16_t *s_b = sh.b;
    uint16_t *s_entry = sh.entry;
    uint32_t *s_unit = sh.unit;
    int &s_long = sh.is_long[0], &s_in_order = sh.is_long[1];
    const int tid = threadIdx.x, w = tid / kWave, lane = lane_id();
    if (tid == 0) {
        decode_unit<kSPiece>(a, u, s_unit);
        s_long = 0;
        s_in_order = 0;
    }
    __syncthreads();
    const uint32_t r0 = s_unit[0], rn = s_unit[1], s0 = s_unit[2], sn = s_unit[3];
    const int skip_bits = (int)s_unit[4];
    int log2nb = 0;
    while ((1u << log2nb) < rn) ++log2nb;
    log2nb = min(log2nb + (int)s_unit[5], G::kMaxLog2nb);
    const uint32_t nb = 1u << log2nb;
    // each wave's share of the S piece, and how it writes its matches
    const uint32_t q = ceil_div_u32(sn, kWv);
    const uint32_t ws = min(sn, w * q), we = min(sn, ws + q);
    const bool dups = a.flags[1] != 0;
    bool in_order = false;
    if (dups) {
        const uint64_t at = (uint64_t)u * kWv + w, slots = (uint64_t)units_to_run(a.nunits, a.flags, a.cap_units) * kWv;
        const uint64_t out = (at + 1 < slots ? a.woff[at + 1] : *a.total) - a.woff[at];
        in_order = __builtin_amdgcn_readfirstlane(write_in_order(a.nr + a.ns, a.wmulti[at], out, we - ws));
        if (in_order && lane == 0) s_in_order = 1;
    }

    // ---- build: bucket counts, scan, placement, per-bucket order by row ----
    const K *__restrict__ rkey = static_cast<const K *>(a.rkey);
    for (uint32_t i = tid; i < rn; i += kBlockT) s_rkey[i] = rkey[r0 + i];
    for (uint32_t b = tid; b <= nb; b += kBlockT) s_b[b] = 0;
    __syncthreads();
    for (uint32_t i = tid; i < rn; i += kBlockT) b16_add1(s_b, bucket_of<K>(s_rkey[i], skip_bits, log2nb));
    __syncthreads();
    scan_buckets<BUILD, NT>(s_b, sh.tmp, nb, rn);
    __syncthreads();
    // placement from the end of each bucket; afterwards s_b[b] = start of bucket b
    for (uint32_t i = tid; i < rn; i += kBlockT) {
        const uint32_t slot = b16_dec(s_b, bucket_of<K>(s_rkey[i], skip_bits, log2nb)) - 1u;
        s_entry[slot] = (uint16_t)i;
    }
    __syncthreads();
    // chains in row order, so that every S row emits its matches in R's input
    // order; where S rows match several R rows, in (key, row) order
    for (uint32_t b = tid; b < nb; b += kBlockT) {
        const uint32_t lo = s_b[b], hi = s_b[b + 1];
        if (hi - lo > kMaxChainSort) {
            s_long = 1;
        } else {
            for (uint32_t x = lo + 1; x < hi; ++x) {
                const uint16_t e = s_entry[x];
                const K ek = s_rkey[e];
                uint32_t y = x;
                while (y > lo && (dups && s_rkey[s_entry[y - 1]] != ek ? s_rkey[s_entry[y - 1]] > ek : s_entry[y - 1] > e)) {
                    s_entry[y] = s_entry[y - 1];
                    --y;
                }
                s_entry[y] = e;
            }
        }
    }
    __syncthreads();
    if (s_long) {
        // Rare (heavy duplicate keys): one wave places all rows again in row
        // order, ranking equal buckets within a round by ballot.
        if (w == 0) {
            for (uint32_t base = 0; base < rn; base += kWave) {
                const uint32_t i = base + lane;
                const bool valid = i < rn;
                const uint32_t b = valid ? bucket_of<K>(s_rkey[i], skip_bits, log2nb) : 0u;
                const uint64_t peers = match_peers(b, log2nb, valid);
                if (valid) {
                    const uint32_t rk = rank_below(peers);
                    const uint32_t st = s_b[b];
                    if (rk == 0) s_b[b] = (uint16_t)(st + (uint32_t)__popcll(peers));
                    s_entry[st + rk] = (uint16_t)i;
                }
            }
            // s_b[b] now holds the end of bucket b: shift right by one, top down
            for (int c = (int)((nb + kWave - 1) / kWave) - 1; c >= 0; --c) {
                const uint32_t b = (uint32_t)c * kWave + lane;
                const uint32_t v = b < nb ? s_b[b] : 0u;
                if (b < nb) s_b[b + 1] = (uint16_t)v;
            }
            if (lane == 0) s_b[0] = 0;
        }
        __syncthreads();
    }
    {
        // keys in bucket order (s_rkey[e] = key of entry e), so that a probe
        // compares keys without going through the row index
        constexpr int per = (int)(BUILD / kBlockT);
        K t[per];
#pragma unroll
        for (int k = 0; k < per; ++k) {
            const uint32_t e = tid + k * kBlockT;
            t[k] = e < rn ? s_rkey[s_entry[e]] : K(0);
        }
        __syncthreads();
#pragma unroll
        for (int k = 0; k < per; ++k) {
            const uint32_t e = tid + k * kBlockT;
            if (e < rn) s_rkey[e] = t[k];
        }
        __syncthreads();
    }

    // ---- probe: each wave streams a contiguous share of the S piece, PB
    // rounds of 64 rows at a time so that many loads are in flight ----
    const K *__restrict__ skey = static_cast<const K *>(a.skey);
    uint8_t *s_pay = reinterpret_cast<uint8_t *>(sh.is_long) + 8;
    int staged = 0;
    if (s_in_order && !s_long) {
        // R payloads that fit beside the table: read once, in order, into LDS (each
        // is used by several output rows, and their gathers were what the waves
        // waited for)
        staged = a.rstaged;
        for (int j = 0; j < staged; ++j) {
            if (a.rw[j] == 4) {
                const uint32_t *__restrict__ in = static_cast<const uint32_t *>(a.rp[j]) + r0;
                uint32_t *d = reinterpret_cast<uint32_t *>(s_pay + a.rlds_off[j]);
                for (uint32_t i = tid; i < rn; i += kBlockT) d[i] = in[i];
            } else {
                const uint64_t *__restrict__ in = static_cast<const uint64_t *>(a.rp[j]) + r0;
                uint64_t *d = reinterpret_cast<uint64_t *>(s_pay + a.rlds_off[j]);
                for (uint32_t i = tid; i < rn; i += kBlockT) d[i] = in[i];
            }
        }
        __syncthreads();
    }
    if (in_order && s_long) {
        write_long<K>(a, sh, r0, s0, ws, we, skip_bits, log2nb, out_base + a.woff[(uint64_t)u * kWv + w]);
    } else if (in_order) {
        write_dups<K>(a, sh, s_pay, staged, r0, s0, ws, we, skip_bits, log2nb, out_base + a.woff[(uint64_t)u * kWv + w]);
    } else {
        uint64_t outpos = out_base + a.woff[(uint64_t)u * kWv + w];
        K *__restrict__ tkey = static_cast<K *>(a.tkey);
        for (uint32_t base = ws; base < we; base += PB * kWave) {
            K key[PB];
            uint32_t c[PB], e1[PB];
#pragma unroll
            for (int r = 0; r < PB; ++r) {
                const uint32_t i = base + r * kWave + lane;
                key[r] = i < we ? skey[s0 + i] : K(0);
            }
            bool valid[PB];
#pragma unroll
            for (int r = 0; r < PB; ++r) valid[r] = base + r * kWave + lane < we;
            probe_rows<K, PB>(s_rkey, s_b, key, valid, skip_bits, log2nb, rn, c, e1);
#pragma unroll
            for (int r = 0; r < PB; ++r) e1[r] = c[r] ? (uint32_t)s_entry[e1[r]] : 0u;
            uint64_t pos[PB];
            bool multi = false;
#pragma unroll
            for (int r = 0; r < PB; ++r) {
                const uint32_t incl = wave_inclusive_sum<uint32_t>(c[r]);
                pos[r] = outpos + incl - c[r];
                outpos += __shfl(incl, kWave - 1, kWave);
                multi |= __ballot(c[r] > 1) != 0ull;
            }
            if (!multi) {
                // at most one match per S row: every output row is (S row, its R row)
#pragma unroll
                for (int r = 0; r < PB; ++r)
                    if (c[r] && pos[r] < a.t_rows) tkey[pos[r]] = key[r];
                uint32_t srow[PB], rrow[PB];
#pragma unroll
                for (int r = 0; r < PB; ++r) {
                    const uint32_t i = base + r * kWave + lane;
                    srow[r] = s0 + i;
                    rrow[r] = r0 + e1[r];
                    if (a.srow && c[r]) srow[r] = (uint32_t)a.srow[srow[r]];
                    if (a.rrow && c[r]) rrow[r] = (uint32_t)a.rrow[rrow[r]];
                }
                gather_cols<PB>(a.ns, a.sp, a.sw, a.ts, srow, c, pos, a.t_rows);
                gather_cols<PB>(a.nr, a.rp, a.rw, a.tr, rrow, c, pos, a.t_rows);
            } else {
                // several matches for some row: enumerate the chain per lane
#pragma unroll
                for (int r = 0; r < PB; ++r) {
                    if (!c[r]) continue;
                    const uint32_t i = base + r * kWave + lane;
                    uint64_t p = pos[r];
                    const uint64_t sr = a.srow ? (uint64_t)a.srow[s0 + i] : (uint64_t)(s0 + i);
                    const uint32_t b = bucket_of<K>(key[r], skip_bits, log2nb);
                    for (uint32_t e = s_b[b], end = s_b[b + 1]; e < end; ++e) {
                        if (s_rkey[e] != key[r] || p >= a.t_rows) continue;
                        const uint32_t ri = s_entry[e];
                        const uint64_t rr = a.rrow ? (uint64_t)a.rrow[r0 + ri] : (uint64_t)(r0 + ri);
                        tkey[p] = key[r];
                        for (int j = 0; j < a.nr; ++j) copy_val(a.tr[j], a.rw[j], p, a.rp[j], rr);
                        for (int j = 0; j < a.ns; ++j) copy_val(a.ts[j], a.sw[j], p, a.sp[j], sr);
                        ++p;
                    }
                }
            }
        }
    }
}

template <typename K, uint32_t BUILD, int NT, bool WRITE>
__device__ __forceinline__ void join_unit(const JoinArgs &a, uint32_t u, uint64_t out_base, const JoinLds<K> &sh) {
    if constexpr (WRITE) write_unit<K, BUILD, NT>(a, u, out_base, sh);
    else count_unit<K, BUILD, NT>(a, u, sh);
}

// One work unit per workgroup (eager calls: the grid is the unit count).
template <typename K, uint32_t BUILD, int NT, bool WRITE>
__global__ __launch_bounds__(NT, (WRITE ? Geo<BUILD, NT>::kMinWEager : Geo<BUILD, NT>::kMinWCount)) void k_join(JoinArgs a) {
    extern __shared__ uint4 s_dyn4[];
    const JoinLds<K> sh = join_lds<K, BUILD, NT>(reinterpret_cast<uint8_t *>(s_dyn4), a.lds_rows);
    // a block larger than the LDS was sized for (the host sees it and sizes again)
    if (min(a.flags[2], a.rc) > a.lds_rows) return;
    if (blockIdx.x < units_to_run(a.nunits, a.flags, a.cap_units)) join_unit<K, BUILD, NT, WRITE>(a, blockIdx.x, 0ull, sh);
}

// Write pass without a hash table, for the common case recorded by the count
// pass (one R block per partition, at most one match per S row): each wave
// streams its S rows with their recorded matches, takes output positions from
// the scanned counts plus a ballot prefix, and gathers the payloads (GFTR:
// partition-local R rows; GFUR: original rows through the row ids). It needs no
// LDS, so it always runs 256-thread workgroups whose waves take the count
// pass's (unit, wave) slots one by one, whatever the table shape.
template <typename K, uint32_t BUILD, int NT, bool GFUR>
__global__ __launch_bounds__(kBlock, GFUR ? 4 : 1) void k_join_stream(JoinArgs a) {
    using G = Geo<BUILD, NT>;
    constexpr int PB = G::kPBStream;
    constexpr int kWv = G::kWv;
    constexpr uint32_t kSPiece = G::kSPiece;
    if (a.flags[0] | a.flags[1]) return;  // the LDS write pass handles this input
    const int lane = lane_id();
    const uint32_t n_units = units_to_run(a.nunits, a.flags, a.cap_units);
    const uint64_t n_slots = (uint64_t)n_units * kWv;
    const uint64_t out_base = a.out_base ? *a.out_base : 0ull;
    const K *__restrict__ skey = static_cast<const K *>(a.skey);
    K *__restrict__ tkey = static_cast<K *>(a.tkey);
    for (uint64_t slot = (uint64_t)blockIdx.x * kWaves + threadIdx.x / kWave; slot < n_slots;
         slot += (uint64_t)gridDim.x * kWaves) {
        const uint32_t u = (uint32_t)(slot / kWv), w = (uint32_t)(slot % kWv);
        const uint32_t p = a.umap[u], sb = u - a.ubase[p];  // one R block: the unit is the S piece
        const uint32_t ns = a.spo[p + 1] - a.spo[p];
        const uint32_t s0 = a.spo[p] + sb * kSPiece, sn = min(kSPiece, ns - sb * kSPiece);
        const uint32_t r0 = a.rpo[p], rn = a.rpo[p + 1] - r0;
        const uint32_t q = ceil_div_u32(sn, kWv);
        const uint32_t ws = min(sn, w * q), we = min(sn, ws + q);
        // output rows of this wave: wbase + a 32-bit offset (a wave writes at most q rows)
        const uint64_t wbase = out_base + a.woff[slot];
        const uint32_t lim = a.t_rows > wbase ? (uint32_t)min<uint64_t>(a.t_rows - wbase, 0xFFFFFFFFull) : 0u;
        uint32_t off = 0;
        for (uint32_t base = ws; base < we; base += PB * kWave) {
            // lrow[r]: the match's row in the R block, or ~0 (none; a recorded row
            // past the block is impossible when the count pass ran on this input)
            uint32_t lrow[PB], pos[PB];
            {
                uint32_t m[PB];
                K key[PB];
                const uint16_t *__restrict__ mp = a.midx + (s0 + base + lane);
                const K *__restrict__ kp = skey + (s0 + base + lane);
#pragma unroll
                for (int r = 0; r < PB; ++r) {
                    const bool in = base + r * kWave + lane < we;
                    m[r] = in ? mp[r * kWave] : kNoMatch;
                    key[r] = in ? kp[r * kWave] : K(0);
                }
                K *__restrict__ tk = tkey + wbase;
#pragma unroll
                for (int r = 0; r < PB; ++r) {
                    lrow[r] = m[r] < rn ? m[r] : ~0u;
                    const uint64_t hit = __ballot(lrow[r] != ~0u);
                    pos[r] = off + rank_below(hit);
                    off += (uint32_t)__popcll(hit);
                    if (lrow[r] != ~0u && pos[r] < lim) tk[pos[r]] = key[r];
                }
            }
            if constexpr (!GFUR) {
                // GFTR: S rows are contiguous, R rows partition-local
                stream_cols_contig<PB>(a.ns, a.sp, a.sw, a.ts, s0 + base + lane, lrow, pos, wbase, lim);
                gather_cols_wave<PB>(a.nr, a.rp, a.rw, a.tr, r0, lrow, lrow, pos, wbase, lim);
            } else {
                // GFUR: original rows through the row ids
                uint32_t row[PB];
#pragma unroll
                for (int r = 0; r < PB; ++r) row[r] = lrow[r] != ~0u ? (uint32_t)a.srow[s0 + base + r * kWave + lane] : 0u;
                gather_cols_wave<PB>(a.ns, a.sp, a.sw, a.ts, 0u, row, lrow, pos, wbase, lim);
#pragma unroll
                for (int r = 0; r < PB; ++r) row[r] = lrow[r] != ~0u ? (uint32_t)a.rrow[r0 + lrow[r]] : 0u;
                gather_cols_wave<PB>(a.nr, a.rp, a.rw, a.tr, 0u, row, lrow, pos, wbase, lim);
            }
        }
    }
}

// Streaming write pass with the R side staged in LDS (GFTR, one R block per
// partition, at most one match per S row): a workgroup takes one unit (an S
// piece of one partition), copies the partition's R payload columns into LDS
// with coalesced reads, and streams the S piece as k_join_stream does, reading
// R values from LDS. Every R payload value then crosses HBM once per S piece,
// where the gathers of k_join_stream re-read lines that L2 has dropped when a
// compute unit's partitions outgrow its share of L2. A unit whose S piece has
// fewer rows than its R block (cold partitions under skew) gathers from HBM
// instead, since staging would move more bytes than it saves. Launched when
// the largest partition's R payload fits the dynamic LDS.
template <typename K, uint32_t BUILD, int NT>
__global__ __launch_bounds__(NT, (Geo<BUILD, NT>::kMinWStaged)) void k_join_stream_staged(JoinArgs a) {
    using G = Geo<BUILD, NT>;
    constexpr int PB = G::kPBStream;
    constexpr int kWv = G::kWv;
    constexpr int kT = G::kThreads;
    constexpr uint32_t kSPiece = G::kSPiece;
    extern __shared__ uint4 s_dyn4[];
    uint8_t *s_dyn = reinterpret_cast<uint8_t *>(s_dyn4);
    __shared__ uint32_t s_unit[4];
    if (a.flags[0] | a.flags[1]) return;
    const int tid = threadIdx.x, w = tid / kWave, lane = lane_id();
    const uint32_t n_units = units_to_run(a.nunits, a.flags, a.cap_units);
    const uint64_t out_base = a.out_base ? *a.out_base : 0ull;
    const K *__restrict__ skey = static_cast<const K *>(a.skey);
    K *__restrict__ tkey = static_cast<K *>(a.tkey);
    for (uint32_t u = blockIdx.x; u < n_units; u += gridDim.x) {
        if (tid == 0) {
            const uint32_t p = a.umap[u], sb = u - a.ubase[p];  // one R block: the unit is the S piece
            const uint32_t ns = a.spo[p + 1] - a.spo[p];
            s_unit[0] = a.rpo[p];
            s_unit[1] = min(a.rpo[p + 1] - a.rpo[p], a.flags[2]);  // never past the staged rows
            s_unit[2] = a.spo[p] + sb * kSPiece;
            s_unit[3] = min(kSPiece, ns - sb * kSPiece);
        }
        __syncthreads();
        const uint32_t r0 = s_unit[0], rn = s_unit[1], s0 = s_unit[2], sn = s_unit[3];
        const bool staged = sn >= rn;  // uniform over the workgroup
        for (int j = 0; j < a.nr && staged; ++j) {
            if (a.rw[j] == 4) {
                const uint32_t *__restrict__ in = static_cast<const uint32_t *>(a.rp[j]) + r0;
                uint32_t *d = reinterpret_cast<uint32_t *>(s_dyn + a.rlds_off[j]);
                for (uint32_t i = tid; i < rn; i += kT) d[i] = in[i];
            } else {
                const uint64_t *__restrict__ in = static_cast<const uint64_t *>(a.rp[j]) + r0;
                uint64_t *d = reinterpret_cast<uint64_t *>(s_dyn + a.rlds_off[j]);
                for (uint32_t i = tid; i < rn; i += kT) d[i] = in[i];
            }
        }
        __syncthreads();
        const uint32_t q = ceil_div_u32(sn, kWv);
        const uint32_t ws = min(sn, w * q), we = min(sn, ws + q);
        // output rows of this wave: wbase + a 32-bit offset (a wave writes at most q rows)
        const uint64_t wbase = out_base + a.woff[(uint64_t)u * kWv + w];
        const uint32_t lim = a.t_rows > wbase ? (uint32_t)min<uint64_t>(a.t_rows - wbase, 0xFFFFFFFFull) : 0u;
        uint32_t off = 0;
        for (uint32_t base = ws; base < we; base += PB * kWave) {
            // lrow[r]: LDS row of the match, or ~0 (no match, or a row past the
            // staged block, impossible when the count pass ran on the same input)
            uint32_t lrow[PB], pos[PB];
            {
                uint32_t m[PB];
                K key[PB];
                const uint16_t *__restrict__ mp = a.midx + (s0 + base + lane);
                const K *__restrict__ kp = skey + (s0 + base + lane);
#pragma unroll
                for (int r = 0; r < PB; ++r) {
                    const bool in = base + r * kWave + lane < we;
                    m[r] = in ? mp[r * kWave] : kNoMatch;
                    key[r] = in ? kp[r * kWave] : K(0);
                }
                K *__restrict__ tk = tkey + wbase;
#pragma unroll
                for (int r = 0; r < PB; ++r) {
                    lrow[r] = m[r] < rn ? m[r] : ~0u;
                    const uint64_t hit = __ballot(lrow[r] != ~0u);
                    pos[r] = off + rank_below(hit);
                    off += (uint32_t)__popcll(hit);
                    if (lrow[r] != ~0u && pos[r] < lim) tk[pos[r]] = key[r];
                }
            }
            // S payloads: contiguous partitioned rows, one base address per column
            for (int j = 0; j < a.ns; ++j) {
                if (a.sw[j] == 4) {
                    const uint32_t *__restrict__ in = static_cast<const uint32_t *>(a.sp[j]) + (s0 + base + lane);
                    uint32_t *__restrict__ out = static_cast<uint32_t *>(a.ts[j]) + wbase;
                    uint32_t v[PB];
#pragma unroll
                    for (int r = 0; r < PB; ++r) v[r] = lrow[r] != ~0u ? in[r * kWave] : 0u;
#pragma unroll
                    for (int r = 0; r < PB; ++r)
                        if (lrow[r] != ~0u && pos[r] < lim) out[pos[r]] = v[r];
                } else {
                    const uint64_t *__restrict__ in = static_cast<const uint64_t *>(a.sp[j]) + (s0 + base + lane);
                    uint64_t *__restrict__ out = static_cast<uint64_t *>(a.ts[j]) + wbase;
                    uint64_t v[PB];
#pragma unroll
                    for (int r = 0; r < PB; ++r) v[r] = lrow[r] != ~0u ? in[r * kWave] : 0ull;
#pragma unroll
                    for (int r = 0; r < PB; ++r)
                        if (lrow[r] != ~0u && pos[r] < lim) out[pos[r]] = v[r];
                }
            }
            // R payloads from LDS, or from the partitioned column in HBM
            for (int j = 0; j < a.nr; ++j) {
                if (!staged) {
                    if (a.rw[j] == 4) {
                        const uint32_t *__restrict__ col = static_cast<const uint32_t *>(a.rp[j]) + r0;
                        uint32_t *__restrict__ out = static_cast<uint32_t *>(a.tr[j]) + wbase;
                        uint32_t v[PB];
#pragma unroll
                        for (int r = 0; r < PB; ++r) v[r] = lrow[r] != ~0u ? col[lrow[r]] : 0u;
#pragma unroll
                        for (int r = 0; r < PB; ++r)
                            if (lrow[r] != ~0u && pos[r] < lim) out[pos[r]] = v[r];
                    } else {
                        const uint64_t *__restrict__ col = static_cast<const uint64_t *>(a.rp[j]) + r0;
                        uint64_t *__restrict__ out = static_cast<uint64_t *>(a.tr[j]) + wbase;
                        uint64_t v[PB];
#pragma unroll
                        for (int r = 0; r < PB; ++r) v[r] = lrow[r] != ~0u ? col[lrow[r]] : 0ull;
#pragma unroll
                        for (int r = 0; r < PB; ++r)
                            if (lrow[r] != ~0u && pos[r] < lim) out[pos[r]] = v[r];
                    }
                } else if (a.rw[j] == 4) {
                    const uint32_t *col = reinterpret_cast<const uint32_t *>(s_dyn + a.rlds_off[j]);
                    uint32_t *__restrict__ out = static_cast<uint32_t *>(a.tr[j]) + wbase;
#pragma unroll
                    for (int r = 0; r < PB; ++r)
                        if (lrow[r] != ~0u && pos[r] < lim) out[pos[r]] = col[lrow[r]];
                } else {
                    const uint64_t *col = reinterpret_cast<const uint64_t *>(s_dyn + a.rlds_off[j]);
                    uint64_t *__restrict__ out = static_cast<uint64_t *>(a.tr[j]) + wbase;
#pragma unroll
                    for (int r = 0; r < PB; ++r)
                        if (lrow[r] != ~0u && pos[r] < lim) out[pos[r]] = col[lrow[r]];
                }
            }
        }
        __syncthreads();  // the next unit restages the LDS
    }
}

// Persistent workgroups over the unit count held in device memory (plans).
template <typename K, uint32_t BUILD, int NT, bool WRITE>
__global__ __launch_bounds__(NT, (WRITE ? Geo<BUILD, NT>::kMinWWrite : Geo<BUILD, NT>::kMinW)) void k_join_persist(JoinArgs a) {
    extern __shared__ uint4 s_dyn4[];
    const JoinLds<K> sh = join_lds<K, BUILD, NT>(reinterpret_cast<uint8_t *>(s_dyn4), a.lds_rows);
    if (WRITE && a.lds_if_complex && !(a.flags[0] | a.flags[1])) return;  // the streaming pass writes
    const uint32_t n_units = units_to_run(a.nunits, a.flags, a.cap_units);
    const uint64_t out_base = a.out_base ? *a.out_base : 0ull;
    for (uint32_t u = blockIdx.x; u < n_units; u += gridDim.x) {
        join_unit<K, BUILD, NT, WRITE>(a, u, out_base, sh);
        __syncthreads();  // the unit's LDS state is rebuilt by the next one
    }
}

// Output offset of each instance of a batch: the write offset of its first unit.
// Units past the processed count (a plan's capacity) contribute nothing.
__global__ void k_instance_offsets(const uint32_t *__restrict__ ubase, const uint64_t *__restrict__ woff,
                                   uint32_t waves_per_unit, uint32_t n_inst, const uint32_t *__restrict__ nunits,
                                   const uint32_t *__restrict__ flags, uint32_t cap_units,
                                   const uint64_t *__restrict__ total, const uint64_t *__restrict__ base,
                                   uint64_t *__restrict__ out) {
    const uint32_t nu = units_to_run(nunits, flags, cap_units);
    const uint64_t b = base ? *base : 0ull;
    for (uint32_t i = blockIdx.x * blockDim.x + threadIdx.x; i <= n_inst; i += gridDim.x * blockDim.x) {
        const uint32_t u = (i == n_inst) ? nu : min(ubase[i << 8], nu);
        out[i] = b + (u == nu ? *total : woff[(uint64_t)u * waves_per_unit]);
    }
}

// next = base + total (the first output row of a plan's next group), and the
// group's unit count for the plan's capacity check.
// An overflowed unit count reports the largest count, so that the plan's result
// flags the group as beyond its capacity.
__global__ void k_advance_base(const uint64_t *__restrict__ base, const uint64_t *__restrict__ total,
                               uint64_t *__restrict__ next, const uint32_t *__restrict__ nunits,
                               const uint32_t *__restrict__ flags, uint32_t *__restrict__ units_out) {
    if (blockIdx.x == 0 && threadIdx.x == 0) {
        if (next) *next = (base ? *base : 0ull) + *total;
        if (units_out) *units_out = flags[3] ? 0xFFFFFFFFu : *nunits;
    }
}

// The count and write kernels of one table shape.
template <typename K, uint32_t BUILD, int NT>
struct JoinKernels {
    using G = Geo<BUILD, NT>;
    static void count(hipStream_t s, bool planned, uint32_t grid, const JoinArgs &a, double bytes) {
        const size_t shm = join_lds_bytes<K, BUILD, NT>(a.lds_rows);
        if constexpr (G::kRows == 16) {
            if (planned) {
                GJ_LAUNCH("k_join_count", bytes, (k_join_persist<K, BUILD, NT, false>), dim3(grid), dim3(G::kThreads), shm, s, a);
                return;
            }
        }
        GJ_LAUNCH("k_join_count", bytes, (k_join<K, BUILD, NT, false>), dim3(grid), dim3(G::kThreads), shm, s, a);
    }
    // grid: workgroups of the unit passes; the streaming pass has kWaves-wave workgroups
    static void stream(hipStream_t s, uint32_t grid, const JoinArgs &a, double bytes) {
        grid = (uint32_t)std::min<uint64_t>((uint64_t)grid * G::kWv / kWaves, 1u << 30);
        if (a.srow) GJ_LAUNCH("k_join_write", bytes, (k_join_stream<K, BUILD, NT, true>), dim3(grid), dim3(kBlock), 0, s, a);
        else GJ_LAUNCH("k_join_write", bytes, (k_join_stream<K, BUILD, NT, false>), dim3(grid), dim3(kBlock), 0, s, a);
    }
    static void staged(hipStream_t s, uint32_t grid, size_t shm, const JoinArgs &a, double bytes) {
        GJ_LAUNCH("k_join_write", bytes, (k_join_stream_staged<K, BUILD, NT>), dim3(grid), dim3(G::kThreads), shm, s, a);
    }
    // R payload columns beside the table, as many as leave waves enough (S rows with several matches)
    static size_t stage_r(JoinArgs &a) {
        size_t shm = join_lds_bytes<K, BUILD, NT>(a.lds_rows), used = 0;
        for (; a.rstaged < a.nr; ++a.rstaged) {
            const size_t b = ((size_t)a.lds_rows * a.rw[a.rstaged] + 15) & ~(size_t)15;
            if (!staging_fits(shm + used + b, G::kWv)) break;
            a.rlds_off[a.rstaged] = (uint32_t)used;
            used += b;
        }
        return shm + used;
    }
    static void write_lds(hipStream_t s, bool planned, uint32_t grid, JoinArgs a, double bytes, bool stage) {
        const size_t shm = stage ? stage_r(a) : join_lds_bytes<K, BUILD, NT>(a.lds_rows);
        if constexpr (G::kRows == 16) {
            if (planned) {
                GJ_LAUNCH("k_join_write_lds", bytes, (k_join_persist<K, BUILD, NT, true>), dim3(grid), dim3(G::kThreads), shm, s, a);
                return;
            }
        }
        GJ_LAUNCH("k_join_write_lds", bytes, (k_join<K, BUILD, NT, true>), dim3(grid), dim3(G::kThreads), shm, s, a);
    }
};

// Pass 0 = count, 1 = streaming write, 2 = LDS write, 3 = streaming write with
// the R side staged in shm bytes of LDS; the table shape holds r_block rows. Pass 2
// with shm != 0: R payloads may be staged.
// waves: of a unit (waves_per_unit).
void launch_join_pass(int pass, int key_bytes, uint32_t table_rows, uint32_t waves, hipStream_t s, bool planned,
                      uint32_t grid, const JoinArgs &a, double bytes, size_t shm = 0) {
#define GJ_JP(K, B, NT)                                             \
    do {                                                            \
        if (pass == 0) JoinKernels<K, B, NT>::count(s, planned, grid, a, bytes);     \
        else if (pass == 1) JoinKernels<K, B, NT>::stream(s, grid, a, bytes);        \
        else if (pass == 3) JoinKernels<K, B, NT>::staged(s, grid, shm, a, bytes);   \
        else JoinKernels<K, B, NT>::write_lds(s, planned, grid, a, bytes, shm != 0); \
    } while (0)
    if (key_bytes == 4) {
        if (table_rows == 4096 && waves == 16) GJ_JP(int32_t, 4096, 1024);
        else if (table_rows == 4096) GJ_JP(int32_t, 4096, 256);
        else if (table_rows == 8192) GJ_JP(int32_t, 8192, 512);
        else GJ_JP(int32_t, 16384, 1024);
    } else {
        if (table_rows == 4096 && waves == 16) GJ_JP(int64_t, 4096, 1024);
        else if (table_rows == 4096) GJ_JP(int64_t, 4096, 256);
        else GJ_JP(int64_t, 8192, 512);
    }
#undef GJ_JP
}

// Waves of a unit: one for 1024 table rows; 16 for 4096-row tables where an eager
// join has at most two units per compute unit, so that four waves each leave most
// of the chip idle, and on average four S rows for each of the 1024 threads.
// 2^16 x 2^20 rows: count 19 -> 12 us, write 28 -> 16 us, the call 149 -> 137; 322061
// x 1.4M rows: kernels 41 -> 27 us, the call the same. Past either bound the call
// does not gain: with fewer S rows per unit (322061 x 364065) 149 us against 152
// although the kernels take 32 -> 27; with more units the count pass loses (2^21
// x 2^24 rows: 50 against 60 us) what the write pass gains (156 against 145).
constexpr uint64_t kFewUnits = 512;
uint32_t waves_per_unit(uint32_t table_rows, uint64_t units, uint64_t s_rows) {
    return table_rows == 4096 && units <= kFewUnits && s_rows >= units * 4096 ? 16u : table_rows / 1024u;
}

// Largest LDS the staged streaming pass may take (GJ_JOIN_STAGED_LDS overrides;
// 0 turns the staged pass off).
size_t staged_lds_limit() {
    static const size_t lim = [] {
        if (const char *e = getenv("GJ_JOIN_STAGED_LDS")) return (size_t)strtoull(e, nullptr, 10);
        return kJoinStagedLds;
    }();
    return lim;
}

}  // namespace

int64_t join_partitioned(Ctx &ctx, int key_bytes, const JoinSide &R, const JoinSide &S, int bits,
                         int r_block, bool gfur, JoinOut *out, const uint8_t *seg_bits, uint32_t n_inst,
                         uint64_t *inst_off, const JoinPlanned *pl, JoinStats *stats) {
    hipStream_t s = ctx.stream;
    require(r_block >= 64 && r_block <= join_max_r_block(key_bytes),
            key_bytes == 4 ? "R build block must be 64..16384 rows" : "R build block must be 64..8192 rows for 8-byte keys");
    const uint32_t table_rows = join_table_rows(r_block);
    const uint32_t np = seg_bits ? (n_inst << 8) : (1u << bits);
    uint32_t *ucnt = ctx.scratch_n<uint32_t>(np + 1);
    uint32_t *flags = ctx.scratch_n<uint32_t>(6);  // [0..3] flags, [4..5] 64-bit unit total
    const uint32_t *nunits = ucnt + np;
    // Units of a single join whose partitions have one R block each.
    const uint64_t bound = (uint64_t)np + ceil_div_u32(S.rows, join_s_piece(r_block));
    const bool one_kernel = !pl && !seg_bits && bound <= kOneKernelUnits;
    const uint32_t wpu = one_kernel ? waves_per_unit(table_rows, bound, S.rows) : table_rows / 1024u;
    // Single joins with 4096-row tables do not wait for the unit count: the count
    // pass runs for the bound, with LDS for R blocks a quarter over the mean
    // partition, and the one read that sizes the output tells whether both held
    // (else the pass runs again, sized exactly). A join of 2^16 x 2^20 rows waits
    // once instead of twice: 142 -> 130 us (1000 x 4000 rows: 112 -> 90). Larger tables keep the first read: their
    // LDS decides how many workgroups share a compute unit, and it is under 1% of the join.
    // Nor is there a guess where it cannot hold: partitions near the build block's rows,
    // whose units the bound does not count (20000 x 2^22 rows, 2 partitions: the count pass ran
    // for the bound and again, 71 us instead of 35).
    const uint64_t guess_rows = (((uint64_t)R.rows >> bits) + 1) * 5 / 4;
    bool guess = one_kernel && table_rows == 4096 && guess_rows <= (uint64_t)r_block;
    bool units_known = false;
    uint32_t cap_units = (uint32_t)std::min<uint64_t>(bound, kMaxUnits), grid;
    uint32_t lds_rows = (uint32_t)r_block;  // rows of the largest R block a unit builds on
    uint32_t *umap = nullptr;
    if (one_kernel) {
        umap = ctx.scratch_n<uint32_t>(cap_units);
        GJ_LAUNCH("k_unit_count", 20.0 * np, k_join_units, dim3(1), dim3(1024), 0, s, R.poff, S.poff, np,
                  (uint32_t)r_block, join_s_piece(r_block), ucnt, flags, cap_units, umap);
    } else {
        fill_u32(s, flags, 0u, 6);
        GJ_LAUNCH("k_unit_count", 20.0 * np, k_unit_count, dim3(std::min<uint32_t>((np + 255) / 256, 1024)),
                  dim3(256), 0, s, R.poff, S.poff, np, (uint32_t)r_block, join_s_piece(r_block), ucnt, flags);
        scan_exclusive_u32(ctx, ucnt, ucnt, np, ucnt + np);
    }
    uint32_t units = 0, hf[6] = {0};
    // What the flags say before any pass: -1 where the caller may partition again.
    // hf[2]: most R rows in a partition that S probes (a block holds at most r_block)
    const auto check_units = [&]() -> bool {
        if (hf[3]) throw Error(GJ_EOVERFLOW, "more than 2^31-1 join work units (R partitions far larger than the "
                                             "build block)");
        if (!stats) return true;
        stats->max_r_rows = hf[2];
        stats->multi_block = hf[0] != 0;
        return !(stats->check_spread && hf[2] > stats->spread_limit);
    };
    const auto exact_rows = [&]() {
        return std::max<uint32_t>(64, (std::min<uint32_t>(hf[2], (uint32_t)r_block) + 63) & ~63u);
    };
    JoinArgs a{};
    a.rkey = R.key;
    a.skey = S.key;
    a.rpo = R.poff;
    a.spo = S.poff;
    a.np = np;
    a.ubase = ucnt;
    a.rc = (uint32_t)r_block;
    a.skip_bits = (stats && stats->hashed_digits) ? 0 : bits;
    a.seg_bits = seg_bits;
    a.seg_bshift = pl ? pl->seg_bshift : nullptr;
    a.bshift = 0;
    a.nunits = nunits;
    a.out_base = pl ? pl->out_base : nullptr;
    a.midx = ctx.scratch_n<uint16_t>(std::max<uint32_t>(S.rows, 1));
    a.flags = flags;
    a.lds_if_complex = pl ? 1 : 0;
    const double nrows_r = R.rows, nrows_s = S.rows;
    const double key_reads = (nrows_r + nrows_s) * key_bytes;
    uint64_t *wcnt = nullptr, *total = nullptr;
    uint64_t T = 0;
    bool complex = true;  // plans launch both write passes; each decides on the device
    bool dups = false;    // eager calls: some S row matches several R rows
    uint32_t max_r_rows = 0;
    for (;;) {
        if (pl) {
            cap_units = pl->cap_units;
            grid = std::max<uint32_t>(1, std::min<uint32_t>(cap_units, kPersistentGrid));
        } else if (guess) {
            grid = cap_units;
            lds_rows = std::min<uint32_t>((uint32_t)r_block, ((uint32_t)guess_rows + 255) & ~255u);
        } else {
            // eager calls read the unit count and size every launch exactly
            if (!units_known) {
                read_back_parts(s, {{&units, nunits, 4}, {hf, flags, sizeof(hf)}});
                if (!check_units()) return -1;
            }
            lds_rows = exact_rows();
            if (units == 0) {
                if (inst_off) fill_u64(s, inst_off, 0ull, (uint64_t)n_inst + 1);
                return 0;
            }
            if (units > cap_units) umap = nullptr;
            grid = cap_units = units;
        }
        a.lds_rows = lds_rows;
        a.cap_units = cap_units;
        if (!umap) {
            umap = ctx.scratch_n<uint32_t>(cap_units);
            GJ_LAUNCH("k_unit_map", 4.0 * cap_units, k_unit_map,
                      dim3(std::max<uint32_t>(1, std::min<uint32_t>(ceil_div_u32(cap_units, 256), 1024))),
                      dim3(256), 0, s, ucnt, np, nunits, (const uint32_t *)flags, cap_units, umap);
        }
        a.umap = umap;
        const uint64_t nw = (uint64_t)cap_units * wpu;
        wcnt = ctx.scratch_n<uint64_t>(nw + 1);
        total = pl ? pl->total : wcnt + nw;
        a.wcnt = wcnt;
        a.wmulti = ctx.scratch_n<uint8_t>(nw);
        a.total = total;
        launch_join_pass(0, key_bytes, table_rows, wpu, s, pl != nullptr, grid, a, key_reads);
        if (pl || guess) scan_exclusive_u64_dev(ctx, wcnt, wcnt, nw, nunits, wpu, total);
        else scan_exclusive_u64(ctx, wcnt, wcnt, nw, total);
        if (pl) {
            T = pl->out_cap;  // stores are checked against the capacity; the true count stays on the device
            *out = pl->out;
            break;
        }
        read_back_parts(s, {{&T, total, 8}, {&units, nunits, 4}, {hf, flags, sizeof(hf)}});
        if (guess) {
            if (!check_units()) return -1;
            if (units > cap_units || std::min<uint32_t>(hf[2], (uint32_t)r_block) > lds_rows) {
                guess = false;  // the bounds did not hold: nothing is known but the units
                units_known = true;
                continue;
            }
            if (units == 0) return 0;
            grid = units;
            a.lds_rows = exact_rows();
        }
        complex = (hf[0] | hf[1]) != 0;
        dups = hf[1] != 0;
        max_r_rows = hf[2];
        break;
    }
    if (inst_off)
        GJ_LAUNCH("k_instance_offsets", 16.0 * n_inst, k_instance_offsets,
                  dim3(std::min<uint32_t>(ceil_div_u32(n_inst + 1, 256), 1024)), dim3(256), 0, s, ucnt, wcnt, wpu,
                  n_inst, nunits, (const uint32_t *)flags, cap_units, total, a.out_base, inst_off);
    if (pl && (pl->next_base || pl->units_out))
        GJ_LAUNCH("k_advance_base", 16.0, k_advance_base, dim3(1), dim3(64), 0, s, a.out_base, total, pl->next_base,
                  (const uint32_t *)(ucnt + np), (const uint32_t *)flags, pl->units_out);
    if (T == 0) return 0;

    if (!pl) {
        out->key = ctx.output(T * (uint64_t)key_bytes);
        for (int j = 0; j < R.n_pay; ++j) out->r[j] = ctx.output(T * (uint64_t)R.width[j]);
        for (int j = 0; j < S.n_pay; ++j) out->s[j] = ctx.output(T * (uint64_t)S.width[j]);
    }
    a.woff = wcnt;
    a.t_rows = T;
    a.tkey = out->key;
    a.nr = R.n_pay;
    a.ns = S.n_pay;
    for (int j = 0; j < R.n_pay; ++j) {
        a.rp[j] = R.pay[j];
        a.rw[j] = R.width[j];
        a.tr[j] = out->r[j];
    }
    for (int j = 0; j < S.n_pay; ++j) {
        a.sp[j] = S.pay[j];
        a.sw[j] = S.width[j];
        a.ts[j] = out->s[j];
    }
    a.rrow = gfur ? R.rowid : nullptr;
    a.srow = gfur ? S.rowid : nullptr;
    // algorithmic bytes: keys of both sides, payload reads (GFTR: each partitioned
    // row once; GFUR: one gathered value per output row and column, plus row ids),
    // and the output rows (a plan counts its expected rows, given by the caller)
    double rw_sum = 0, sw_sum = 0;
    for (int j = 0; j < R.n_pay; ++j) rw_sum += R.width[j];
    for (int j = 0; j < S.n_pay; ++j) sw_sum += S.width[j];
    const double t_rows = pl ? (double)pl->expect_rows : (double)T;
    double wbytes = key_reads + t_rows * (key_bytes + rw_sum + sw_sum);
    if (gfur) wbytes += t_rows * (rw_sum + sw_sum) + 4.0 * (nrows_r + nrows_s);
    else wbytes += nrows_r * rw_sum + nrows_s * sw_sum;
    // the streaming pass reads no R keys
    const double sbytes = wbytes - nrows_r * key_bytes;
    // Eager GFTR calls stage the R side in LDS when the largest partition's R
    // payload fits (staged_lds_limit() bytes).
    size_t shm = 0;
    if (!pl && !complex && !gfur && R.n_pay > 0) {
        for (int j = 0; j < R.n_pay; ++j) {
            a.rlds_off[j] = (uint32_t)shm;
            shm += ((size_t)max_r_rows * R.width[j] + 15) & ~(size_t)15;
        }
        if (shm > staged_lds_limit()) shm = 0;
    }
    // Eager calls launch the one write pass the count pass chose; plans launch
    // both, and the one that does not apply returns at once.
    if (shm) launch_join_pass(3, key_bytes, table_rows, wpu, s, false, grid, a, sbytes, shm);
    else if (pl || !complex) launch_join_pass(1, key_bytes, table_rows, wpu, s, pl != nullptr, grid, a, sbytes);
    if (pl || complex) {
        const double lbytes = pl ? 0.0 : wbytes;  // a plan counts its bytes once, on the streaming pass
        launch_join_pass(2, key_bytes, table_rows, wpu, s, pl != nullptr, grid, a, lbytes,
                         dups && !gfur && stage_payloads(a.nr + a.ns, T, S.rows) ? 1 : 0);
    }
    return pl ? 0 : (int64_t)T;
}

}  // namespace gj
