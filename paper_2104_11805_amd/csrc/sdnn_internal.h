// Shared between the translation units of libsdnn only.
#pragma once
#include <cstddef>
#include <cstdint>
#include <vector>

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
                              // the transposed index (fused backward sweep; training mode).  Where G[0] holds all of it,
                              // G[1] is scratch of sdnn_weight_grad
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
    // Nets for k_fwd_long: one of W, of 2-byte columns, beside the values (two chunks more at its end; nothing at (1)).
    int32_t b1_blocks[2];
    const int32_t *b1_cs[2];  // [b1_blocks + 1]: first chunk of a block
    const int2 *b1_row[2];    // [64 b1_blocks]: {row, entries} of a lane, row -1 past the last row
    int4 *b1_lm[2];
};

// One layer as k_fwd_pan walks it: its operand in panels, its rows in ranges.
struct PanLayer {
    int32_t panel_cols, panel, n_panels, in_pos;      // neurons and positions per panel; positions of the operand
    int32_t range_rows, range, n_ranges, nb, out_pos; // rows and positions per range; blocks of 64 rows per wavefront
    size_t halves;                                    // room for the stream, in halves of eight slots
};
#define PAN_WAVES 16
#define PAN_POS 16384  // positions of a panel (two samples: 128 KiB of LDS) and of a range (64 registers per lane)
#define PAN_MAX 16     // panels at most
#define PAN_SLOTS 1.75 // room for so many slots per entry; a layout that needs more is not used
// below: the layer before this one, NULL for the first (its operand is stored in the order of its neurons)
void sdnn_pan_geometry(const sdnn_layer &y, const PanLayer *below, PanLayer &g);
// Which row sits where in that layer's stream, see k_fwd_pan.  rows [out_pos]: row or -1; pos [n_out]; seg [ranges][wavefronts]
// [panels + 1] and slot [ranges][wavefronts][panels][nb + 1]: where panels (in halves) and blocks (in slots) start; ends: a byte
// per half.  fullest: entries in the fullest panel; depth: slots of the deepest wavefront, panel by panel.
struct PanLayout {
    std::vector<int32_t> rows, pos, seg, slot;
    std::vector<uint8_t> ends;
    int64_t fullest = 0;
    double depth = 0;
};
void sdnn_pan_layout(const sdnn_layer &y, const PanLayer &g, PanLayout &out);
