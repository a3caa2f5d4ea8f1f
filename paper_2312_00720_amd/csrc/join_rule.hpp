// How a join's LDS write pass emits a wave's matches: sizes and limits only, host code
// without HIP, so that the rule can be checked on its own.
#pragma once

#include <stddef.h>
#include <stdint.h>

namespace gj {

// Whether a wave writes its output rows in order (join.hip: write_dups) or probes
// batches of S rows and lets every lane write its own matches. cols: payload columns of
// both sides; of the wave's `rows` S rows, those of `multi_lanes` lanes include one with
// several matches; out: the wave's output rows. 2^21 x 2^24 rows, write pass, each lane
// its own matches : in order, with a share of 0.0001, 0.0005, 0.001, 0.01, 0.1 R rows
// whose key occurs twice, and 2 and 4 rows per key:
//   two payloads a side   435 : 558, 484 : 556, 500 : 483, 650 : 567, 746 : 588, 777 : 639, 1428 : 940 us
//   four payloads a side  776 : 860, 879 : 857, 945 : 748, 1263 : 882, 1502 : 918, 1535 : 1030, 3269 : 1615
// A batch without such a row keeps 8 or 16 probe rounds in flight; from about one such
// row in a thousand most batches have one. One payload a side has little to write in
// order: 283 : 422, 282 : 422, 295 : 370, 362 : 432, 424 : 457, 425 : 470, 702 : 622.
constexpr bool write_in_order(int cols, uint32_t multi_lanes, uint64_t out, uint32_t rows) {
    return multi_lanes != 0 && (cols <= 2 ? out >= 3ull * rows : multi_lanes * 1024ull >= rows);
}

// R payloads in LDS beside the table: whether it is worth room (waves that write in
// order read them often; the room costs the others workgroups), by the call's payload
// columns, output and S rows; and whether a compute unit keeps 12 waves with workgroups
// of `waves` waves and `lds` bytes. 12 are three workgroups of the 4096-row tables, as
// many as their registers allow, two of the 8192-row ones, and one of the largest. 2^21 x
// 2^24 rows, four rows per key, write pass with 4, 8, 12 and 16 waves: two payloads a
// side 937, 942, 942, 939 us, four 1613, 1616, 1628, 1779, eight 4578, 3366, 3325, 3450; 2^24
// x 2^24 rows, 8-byte keys, 8 and 16 waves: 2034, 1461. No room at all: 1068, 1853, 3495; 1487.
constexpr size_t kCuLds = 160 * 1024, kJoinWriteLds = 156 * 1024;
constexpr bool stage_payloads(int cols, uint64_t out, uint64_t s_rows) {
    return cols <= 2 ? out >= 3 * s_rows : out > s_rows + s_rows / 1024;
}
constexpr bool staging_fits(size_t lds, int waves) { return lds <= kJoinWriteLds && kCuLds / lds * (size_t)waves >= 12; }

}  // namespace gj
