// Where the weight requests of the small-batch kernel (fq_batch.hip) go and how it divides a launch: plain integer
// code, so that a host program can check every request against the array it reads, and every division.
//
// A run of `rows` weight rows is read through a buffer descriptor of rows * row_bytes bytes.  Whether a request is
// in range must not depend on the scalar offset of the instruction (compilers are free to leave it out of the
// check, and a scalar offset beyond the descriptor's size has no defined meaning), so tile, line and half
// line are all in the lane's offset and the scalar offset is zero.  Requests that leave the run -- rows past the
// last one of a partial tile, the second half line of an odd last group at 2, 3 and 4 bits, requests ahead past the
// last tile -- are then beyond the descriptor's end: no access, zeros.
#ifndef FQ_BATCH_AT_H
#define FQ_BATCH_AT_H

#include <stdint.h>

#ifdef __HIPCC__
#define FQ_BATCH_FN __host__ __device__ inline __attribute__((always_inline))
#else
#define FQ_BATCH_FN inline
#endif

// Descriptor size of a run of `tiles` tiles of 16 rows that starts `rows_left` rows ahead of the weight's end.
FQ_BATCH_FN uint32_t batch_run_bytes(uint32_t row_bytes, int tiles, int rows_left)
{
    return (uint32_t)(tiles * 16 < rows_left ? tiles * 16 : rows_left) * row_bytes;
}

// A line is what a request reads of a row: 128 bytes, at 2 and 3 bits the 64 or 96 of two quantization groups (256
// inputs as at 4 bits, so that eight wavefronts share a panel's lines evenly), in two halves of four pieces.
FQ_BATCH_FN constexpr int batch_line_bytes(int bits) { return bits < 4 ? 32 * bits : 128; }
FQ_BATCH_FN constexpr int batch_line_inputs(int bits) { return bits < 4 ? 256 : 1024 / bits; }

// A lane's part of the offset: row `n` of 16, piece `c` of four in a half line.
FQ_BATCH_FN uint32_t batch_lane_offset(uint32_t row_bytes, int n, int c, int line_bytes = 128)
{
    return (uint32_t)n * row_bytes + (uint32_t)(c * (line_bytes / 8));
}

// Lane offset of a request's first half line; the second is half a line on.  `line0`: the panel's first byte in a row.
FQ_BATCH_FN uint32_t batch_request(uint32_t row_bytes, uint32_t lane_offset, int tile, uint32_t line0, int line,
                                   int line_bytes = 128)
{
    return lane_offset + ((uint32_t)tile * 16 * row_bytes + line0 + (uint32_t)(line * line_bytes));
}

// x sits in LDS, so many bytes of it at a time: a panel.  `blocks`: blocks of 16 batch rows a launch takes, 1 or 2.
constexpr int BATCH_X_BYTES = 128 * 1024;
FQ_BATCH_FN constexpr int batch_panel(int blocks) { return BATCH_X_BYTES / (32 * blocks); } // inputs: 4096 or 2048

// What a tile of 16 rows costs, in units of 10 ns, fitted to single calls of 128 to 11008 inputs and 1024 to 98304
// rows: a part that does not depend on K (sums, stores, its share of a run's start), its bytes, its lines in turns of
// the eight wavefronts -- a panel that does not fill its last turn pays for all of
// it -- and, for each panel after the first, its share of the wait for x and scales.  Without the first part
// short rows look free beside long ones, and one workgroup gets hundreds of their tiles: rows 14848 x 5120, 12741 x
// 512, 1408 x 5120, 21248 x 5120 at 16, 4, 8 and 4 bits, 4 batch rows, took 205 us against 71 on the register-fed kernel; now
// 60.  An entry's first tile also pays for the start on it (100 to 200 units do the same; 50 are 1 % slower over 1200 plans).
// The panel follows from `blocks` here and nowhere else, so that nobody costs a launch by a panel that it does not have.
constexpr uint32_t BATCH_START_COST = 160;
FQ_BATCH_FN int batch_tile_cost(int blocks, int K, int bits)
{
    const int panel = batch_panel(blocks);
    const int line_bits = bits < 4 ? 4 : bits; // (their lines hold as many inputs as those of 4 bits)
    const int turns = K / panel * (panel / 1024 * line_bits / 8) + (((K % panel * line_bits + 1023) >> 10) + 7) / 8;
    const int per_group = bits == 2 ? 46 : bits == 3 ? 54 : bits == 4 ? 54 : bits == 8 ? 75 : 142;
    return (bits == 16 ? 40 : 66) + (K >> 7) * per_group / 10 + turns * (blocks == 1 ? 11 : 25) +
           ((K + panel - 1) / panel - 1) * (blocks == 1 ? 55 : 30);
}

// Share i of n of a launch's cost begins here; `step`: batch_step(n).  (A share is a few instructions, worked out by every
// wavefront ahead of its first request: integer divisions here and below were half of the 0.9 us between
// the table's arrival and that request.)
FQ_BATCH_FN uint32_t batch_step(uint32_t n) { return 0xffffffffu / n; }
FQ_BATCH_FN uint32_t batch_share_at(uint32_t all, uint32_t i, uint32_t n, uint32_t step)
{
    return i >= n ? all : (uint32_t)(((uint64_t)all * (i * step)) >> 32);
}
FQ_BATCH_FN uint32_t batch_share(uint32_t all, uint32_t i, uint32_t n) { return batch_share_at(all, i, n, batch_step(n)); }

// The first tile of an entry that does not begin ahead of `at`; the entry begins at `begin`.  The quotient may be
// one off: what counts is that it grows with `at`, and that the share before and the share after an `at` find
// the same one.
FQ_BATCH_FN int batch_first_tile(uint32_t at, uint32_t begin, int cost, int tiles)
{
    const uint32_t first = begin + BATCH_START_COST;
    if (at <= first)
        return 0;
    if (at - first >= (uint32_t)cost * (uint32_t)tiles)
        return tiles;
#ifdef __HIP_DEVICE_COMPILE__
    const float inverse = __builtin_amdgcn_rcpf((float)cost);
#else
    const float inverse = 1.0f / (float)cost;
#endif
    const int t = (int)((float)(at - first + (uint32_t)cost - 1) * inverse);
    return t < tiles ? t : tiles;
}

#endif
