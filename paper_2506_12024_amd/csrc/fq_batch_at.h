// Where the weight requests of the small-batch kernel (fq_batch.hip) go: plain integer code, so that a host
// program can check every request of a launch against the array it reads.
//
// A run of `rows` weight rows is read through a buffer descriptor of rows * row_bytes bytes.  Whether a request is
// in range must not depend on the scalar offset of the instruction (compilers are free to leave it out of the
// check, and a scalar offset beyond the descriptor's size has no defined meaning), so tile, line and half
// line are all in the lane's offset and the scalar offset is zero.  Requests that leave the run -- rows past the
// last one of a partial tile, the second half line of an odd last group at 4 bits, requests ahead past the
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

// A lane's part of the offset: row `n` of 16, piece `c` of four in a half line.
FQ_BATCH_FN uint32_t batch_lane_offset(uint32_t row_bytes, int n, int c) { return (uint32_t)n * row_bytes + (uint32_t)c * 16; }

// Lane offset of a request's first half line; the second is 64 bytes on.  `line0`: the panel's first byte in a row.
FQ_BATCH_FN uint32_t batch_request(uint32_t row_bytes, uint32_t lane_offset, int tile, uint32_t line0, int line)
{
    return lane_offset + ((uint32_t)tile * 16 * row_bytes + line0 + (uint32_t)line * 128);
}

#endif
