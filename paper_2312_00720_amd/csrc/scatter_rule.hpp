// Which scatter and which tiles a partition pass takes: sizes and limits only, host code without
// HIP, so that the rule can be checked on its own.
#pragma once

#include <stddef.h>
#include <stdint.h>

namespace gj {

// LDS of the whole-line scatter (partition.hip: k_scatter_lines): D digits, lines of
// A rows, tiles of `tile` rows, row_bytes per row (key and columns), w bytes of the
// widest column.
constexpr int kLineWaves = 16;
constexpr size_t align16(size_t x) { return (x + 15) & ~(size_t)15; }
constexpr uint32_t line_max(uint32_t D, uint32_t A, uint32_t tile) { return (tile + D * (A - 1)) / A + 1; }  // full lines of a tile, and a spare one
constexpr size_t line_lds_bytes(uint32_t D, uint32_t A, uint32_t row_bytes, uint32_t tile, uint32_t w) {
    return (size_t)line_max(D, A, tile) * A * w + (size_t)D * A * row_bytes + align16((size_t)kLineWaves * D * 2) +
           align16((size_t)D * 4) + (size_t)D * 16 + align16((size_t)(D + 1) * 2) + align16(line_max(D, A, tile)) +
           4 * kLineWaves;
}

// Tiles of a pass in short chunks: threads, rows per thread, 4-byte columns loaded
// together (0: the wide kernel, one column at a time).
struct TileShape {
    int block, items, group;
};
constexpr TileShape kWideTile{1024, 16, 0}, kTile4096{512, 8, 4}, kTile2048{512, 4, 4};
// Tiles shrink with the input so that they still fill the chip. All kernels of a
// partition, 2048-row tiles : 4096-row tiles : wide, us.
//  - Up to 2^20 rows the small ones; 8 bytes a row, 5 bits, 2^20: 30 : 33 : 42.
//  - 8-byte keys: the 4096-row tiles lose to both others past 2^20 (12 bytes a row, 5 bits, 2^22: 56
//    : 70 : 54; 24 bytes, 8 + 5 bits, 6.2M: 237 : 299 : 260).
//  - 4-byte keys, to 2.6M rows the 4096-row tiles (20 bytes, 8 bits, 2^21: 72 : 62 : 67).
//  - Up to three bits: runs are long, and the wide kernel is ahead from there on, and
//    from 2^21 with 8-byte keys (20 bytes, 2 bits, 2^22: 100 : 76 : 62; 6.2M: 182 : 132 : 87; 24 bytes
//    with 8-byte keys 193 : 195 : 111).
//  - To 2^22 rows, whose wide tiles run in one round of the 256 compute units, the wide
//    kernel (20 bytes, 8 bits, 2^22: 102 : 90 : 81), but not over segments of narrow rows,
//    which end in part of a tile (8 + 5 bits, 2.9M: 4 bytes 95 : 96 : 100, 20 bytes with 8-byte
//    columns 123 : 124 : 136, 20 bytes of 4-byte columns 140 : 146 : 137).
//  - Past it the second round is nearly empty: the 4096-row tiles to 5.8M rows (5.0M, 8 bits: 8 bytes
//    73 : 70 : 77, 20 bytes with 8-byte columns 94 : 88 : 104) unless rows are wide (36 bytes 225 : 187 :
//    175; 68 bytes with 8-byte columns 355 : 304 : 273, but by 5 bits 226 : 206 : 228).
//  - Many segments (a batch): tiles end with its instances.
constexpr TileShape tile_shape(uint64_t n, uint32_t nseg, int bits, int key_bytes, uint32_t row_bytes, bool narrow) {
    if (nseg > 256) {
        if (n <= 1u << 20 || n / nseg <= 4096) return kTile2048;
        return n <= 3u << 21 || n / nseg <= 16384 ? kTile4096 : kWideTile;
    }
    if (n <= 1u << 20) return kTile2048;
    if (key_bytes == 8) return n <= (bits <= 3 ? 1u << 21 : 3u << 21) ? kTile2048 : kWideTile;
    if (n <= 5u << 19) return kTile4096;
    const bool second = n > 1u << 22 && n <= 11u << 19;  // wide tiles: a nearly empty round
    if (second && !narrow && row_bytes > 32 && bits <= 5) return kTile4096;
    if (bits <= 3) return kWideTile;
    if (n <= 1u << 22) return nseg > 1 && row_bytes < (narrow ? 12u : 32u) ? kTile4096 : kWideTile;
    return (second || (!narrow && n <= 3u << 21)) && row_bytes <= 32 ? kTile4096 : kWideTile;
}

// The whole-line kernel's shape for a pass of `bits` digit bits: lines of 32 rows
// (128 bytes of a 4-byte column) before lines of 16, long tiles before short ones;
// items 0: its LDS does not hold the carry of such rows.
// narrow: the key and every column are 4 bytes wide.
struct LineShape {
    int items, rows;  // rows per thread and tile, rows per line
};
constexpr size_t kLineLds = 160 * 1024 - 128;
constexpr uint32_t kLineSlots = 4;  // carry slots per thread
constexpr LineShape kLineShapes[2][3] = {{{8, 32}, {8, 16}, {0, 0}}, {{14, 32}, {14, 16}, {8, 16}}};  // [narrow]
constexpr LineShape line_shape(int bits, uint32_t row_bytes, bool narrow) {
    for (const LineShape &s : kLineShapes[narrow]) {
        const uint32_t D = 1u << bits, A = (uint32_t)s.rows;
        if (s.items && D * A <= 1024u * kLineSlots &&
            line_lds_bytes(D, A, row_bytes, 1024u * (uint32_t)s.items, narrow ? 4 : 8) <= kLineLds)
            return s;
    }
    return LineShape{0, 0};
}

// Whether a pass cuts its input into long chunks, which the whole-line kernel needs;
// else the wide kernel runs short ones. aligned: every output column starts at a
// multiple of 16 bytes. All kernels of a pass, whole lines against the wide kernel:
//  - From an output that outgrows the 256 MB memory-side cache, which until then puts
//    split lines together again: 2^29 bytes, with 8-byte data (half the rows in a
//    tile, whose fixed work weighs more) 2^31.
//  - From digits whose runs split many lines. 12 bytes a row, 2^31 bytes: 1 to 8 bits
//    1219 : 1220, 1104 : 1115, 1066 : 1103, 1054 : 1144, 1064 : 1203, 1081 : 1292, 1109 :
//    1429, 1332 : 1617 us; 20 bytes, 2^29: 303 : 285, 284 : 271, 278 : 280, 282 : 289,
//    281 : 306, ... With 8-byte data, 16 bytes, 2^31: 5 to 7 bits 1265 : 1217, 1275 :
//    1283, 1326 : 1383. One bit less where the output is larger still (12 bytes, 2^32,
//    3 bits: 2072 : 2152; 32 bytes with 8-byte data, 2^32, 5 bits: 2105 : 2166).
//  - Not with many segments (a batch's instances, mostly shorter than such a chunk).
// Where that kernel has no shape, the wide one runs long chunks only over one segment
// of an output as large (28 bytes, 8 bits: 2^30 790 : 769, 2^32 2989 : 3173); over several it would
// leave a few of them for a second round (16 bytes with 8-byte data, 2^31, 8 + 8 bits: 3388 : 3000).
constexpr bool long_chunks(uint64_t n, uint32_t nseg, int bits, uint32_t row_bytes, bool narrow, bool aligned) {
    const uint64_t bytes = n * row_bytes, least = narrow ? 1ull << 29 : 1ull << 31;
    if (nseg > 256 || !aligned || bytes < least) return false;
    const bool huge = bytes >= (narrow ? 4 : 2) * least;
    if (line_shape(bits, row_bytes, narrow).items == 0) return nseg == 1 && huge;
    return bits >= (narrow ? 4 : 6) - (huge ? 1 : 0);
}

}  // namespace gj
