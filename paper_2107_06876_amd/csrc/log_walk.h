// Which kernel a sweep or a query of a sparse kernel, whose values are held as logs, takes, in
// plain C++ so that it can be checked on a host.
#pragma once

namespace lcn {

// Lanes of a row x entries of a lane at a time; the record walked flat, or round by round (logpass_kernel).
enum LogWalk { FLAT_16x2, FLAT_32x4, FLAT_64x4, ROUNDS_16x2, ROUNDS_16x4, ROUNDS_32x2, ROUNDS_32x4 };

// R rounds, `rows` rows with `nnz` stored values together; L: of a row, p: of a row's piece of a round.  us per half-iteration:
//
// A whole wavefront where looking up an entry's round weighs more than lanes without an entry at the record's end: 5000 rows
// of 420 values in five rounds 5.9 against 7.5, of 670 in eight 7.3 / 10.3, 20 000 of 250 in five 13.6 / 17.0, of 1600 in eight 37 / 57, but
// 5000 of 65 in eight 5.4 / 5.1; in four rounds 60 000 of 1390 102 / 114.
//
// More than four rounds otherwise, flat, sixteen lanes / 32: 20 000 rows of 33 in five 7.7 / 11.0, but 5000 of 40 in five 5.2 / 4.6.
//
// One round: nothing is looked up either way, and round by round the loads' distances are fixed (flat / so: 40 000 rows of
// 418 19.8 / 19.0, 8500 of 390 7.1 / 6.3, 6000 of 385 5.3 / 5.1).  Sixteen lanes x 2 up to 28 values, x 4 up to 140, longer ones 32 x 4; with
// fewer than 12 000 rows, too few for the chip with sixteen lanes, 32 x 2 (8500 of 390 x 4 6.8), but x 4 where they are few and long (6000
// of 385 x 2 5.8).
//
// Two to four rounds, flat: a round that is walked by itself costs a trip of its own, however short (flat / round by round, either
// at its best: 20 000 rows of 3 x 5 5.0 / 5.6, of 3 x 179 14.4 / 15.2, 40 000 of 4 x 10 8.8 / 9.7, of 4 x 178 30.0 / 32.9).
//  * Sixteen lanes x 2 for short records, longer ones the more rows there are to fill the chip (sixteen lanes / 32 x 4): 3000 rows
//    of 2 x 21 3.6 / 3.8, of 3 x 27 4.2 / 3.8; 8500 of 3 x 21 4.5 / 4.7, 5500 of 3 x 25 4.3 / 4.2; 12 500 of 3 x 52 6.1 / 6.5, of 3 x 73 7.4 / 7.1; 30 000
//    of 3 x 53 10.6 / 11.4, of 3 x 74 12.9 / 12.4.
//  * Round by round 32 x 4 (x 2 with 8000 to 12 000 rows) only where rows are few and their pieces long (flat / so): 6000 rows of
//    3 x 307 8.8 / 7.7, 3000 of 4 x 173 6.5 / 6.1, 8500 of 2 x 485 11.8 / 10.9, 12 500 of 2 x 499 15.3 / 14.7; but 7500 of 3 x 140 6.7 / 7.2, 20 000 of
//    2 x 520 22.1 / 22.5.
//
// A query of both sides goes on from row to row.  Sixteen lanes x 4 round by round for pieces of middling length from
// 12 000 rows on (flat / so: 20 000 of 2 x 105 60 / 52, 16 000 of 3 x 135 64 / 57, but 40 000 of 4 x 10 51 / 57), and 32 x 4 for longer ones of
// fewer rows (9000 of 3 x 106 45, x 2 51).
inline LogWalk log_walk(int R, long long rows, long long nnz, bool query)
{
    const long long pieces = R * rows;
    if (R > 4) return nnz > 80 * rows ? FLAT_64x4 : nnz <= 48 * rows ? FLAT_16x2 : FLAT_32x4;
    if (R == 4 && nnz > 1000 * rows) return FLAT_64x4;
    if (R == 1) {
        if (nnz <= 28 * rows) return ROUNDS_16x2;
        if (rows < 12000) return nnz >= 90 * rows && (rows < 8000 || query) ? ROUNDS_32x4 : ROUNDS_32x2;
        return nnz < 140 * rows ? ROUNDS_16x4 : ROUNDS_32x4;
    }
    if (query) {
        if (rows < 12000 && nnz >= 90 * pieces) return ROUNDS_32x4;
        if (rows >= 12000 && nnz > 28 * pieces && nnz < 300 * pieces) return ROUNDS_16x4;
    }
    if (nnz <= (rows >= 10000 ? 180 : rows >= 5000 ? 64 : 40) * rows) return FLAT_16x2;
    if (!query && rows < 18000 && nnz >= (rows < 8000 ? 160 : 200) * pieces)
        return rows >= 8000 && rows < 12000 ? ROUNDS_32x2 : ROUNDS_32x4;
    return FLAT_32x4;
}

}  // namespace lcn
