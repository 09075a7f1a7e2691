// Shared between the translation units of libsdnn only.
#pragma once
#include <cstddef>
#include <cstdint>

#include "../../include/sdnn.h"

#include <hip/hip_vector_types.h> // int4, int2

void sdnn_set_global_error(const char *fmt, ...);
const char *sdnn_global_error();

// Per-layer descriptor, readable by the kernels (a copy lives in the workspace).
struct LayerDev {
    int32_t n_out, n_in, nnz, pad_;
    const int32_t *row_ptr;   // [n_out+1]
    const int32_t *col_idx;   // [nnz]
    float *vals;              // [nnz]
    float *bias;              // [n_out]
    const int32_t *t_row_ptr; // [n_in+1]   transposed index (rows of W^T = columns of W)
    const int32_t *t_row_idx; // [nnz]
    const int32_t *t_perm;    // [nnz]      position of the entry in vals
    const int4 *sched;        // [n_out]    {row, first entry, end, 0}, rows of W by decreasing length
    const int4 *t_sched;      // [n_in]     the same for the rows of W^T
    float *X_prev;            // X_{l-1}  [n_in][B]   (training mode)
    float *X;                 // X_l      [n_out][B]  (training mode)
    float *D;                 // Delta_l  [n_out][B]  (training mode)
    float *G[2];              // [nnz] each: gradient of the stored entries over one half of the batch, in the order of
                              // the transposed index (fused backward sweep; training mode)
    float *vals_t;            // [nnz]: the values in the order of the transposed index (vals_t[q] == vals[t_perm[q]]),
                              // read by the fused backward sweep; NULL where that sweep is not set up
    // The way back from the transposed order to the CSR order, in two passes that both move whole runs (NULL with
    // vals_t).  `mid` holds the values grouped by the TR_CHUNK-entry chunk of the CSR array they belong to, inside
    // a chunk in the order of the transposed index, so that chunk c of the CSR array is filled from entries
    // [c TR_CHUNK, (c+1) TR_CHUNK) of mid.  A span of TR_SPAN consecutive entries of the transposed index lands
    // in mid as one run per chunk; the span's workgroup first puts its values into that order in LDS.
    const uint16_t *mid_slot; // [nnz]: rank of entry q among the entries of its span, by place in mid
    const int32_t *mid_dst;   // [nnz]: mid_dst[span start + k] = the place in mid of the span's entry of rank k
    const uint16_t *mid_loc;  // [nnz]: t_perm of the entry at that place of mid, minus its chunk's start
    float *mid;               // [nnz]
    // Nets made for one sample per step: lane-major copies of W (0) and W^T (1), the only values such a net steps.  The
    // rows, longest first, in blocks of 64; a block's entries come in chunks of eight per lane (B1_CHUNK_BYTES: the
    // lanes' eight columns, 2 or 4 bytes each, then twice four weights), zero weights past the end of a row.
    int32_t b1_blocks[2];
    const int32_t *b1_cs[2];  // [b1_blocks + 1]: first chunk of a block
    const int2 *b1_row[2];    // [64 b1_blocks]: {row, entries} of a lane, row -1 past the last row
    int4 *b1_lm[2];
};
