// libsdnn: HIP kernels (gfx950) and the C-ABI entry points that launch them.
//
// Mapping to the hardware (64-wide wavefronts; none of the three passes is a
// dense contraction: matrix cores only add up lanes, in k_bwd_long):
//   * forward / backward product: one wavefront per matrix row, the 64 lanes
//     walk the row together and each lane owns V consecutive samples, so the
//     row's column indices and weights are wave-uniform (scalar loads) and each
//     gathered activation row is one contiguous 256*V-byte read.  Each lane adds
//     its terms in storage order in fp64: the sum is the same as a sequential
//     CPU loop's, whatever the batch size.
//   * pattern-confined gradient: one wavefront per row, lanes split as
//     4 edge groups x 16 sample lanes, so that only a 16-lane butterfly is
//     needed per 8 edges before the weight is rewritten in place.
//   * W^T: the transposed index lists, per column, the source rows and the
//     positions of the values in the CSR array.
//   * short rows: several rows per wavefront, four samples per lane (k_rows).
//   * nets with enough entries per layer: the backward sweep also forms the
//     gradient of the stored entries (k_bwd_rows; long rows and many samples:
//     k_bwd_long; few short rows: k_bwd_grad, gathered rows parked in LDS) and reads the values from a copy in the order
//     of the transposed index; the descent step is then a streaming pass over
//     that copy (k_apply) and a second one that rebuilds the CSR copy
//     (k_spread_vals).
//   * inference on layers of up to 32768 neurons: one launch, activations in LDS
//     (k_fwd_lds).
//   * training on narrow layers: one launch per pass, activations in LDS
//     (k_train_lds).
//   * training on layers of long rows: the forward pass with four samples of a
//     layer's whole operand in LDS (k_fwd_long).
//   * inference on wider layers: a launch per layer, a panel of the activations in LDS
//     at a time (k_fwd_pan).
//   * inference on large activation blocks goes through all layers in
//     sub-blocks of samples, so that a layer's output is still in the
//     memory-side cache when the next layer gathers it.
//   * one sample per step (B = 1): a lane per row over lane-major copies of W and
//     W^T (k_spmv_lm, k_update_lm), or lanes over entries / rows (k_spmv_stage,
//     k_spmv_wave, k_spmv, k_update_b1).
//   * inference that drops dead samples: stretches of layers in LDS with the live
//     samples listed between them (k_fwd_lds_part, k_live_columns), or flags set by
//     the forward epilogue and in-place packing (k_pack); no host synchronisation.
#include <hip/hip_runtime.h>

#include <cmath>
#include <cstdarg>
#include <cstdio>
#include <cstdlib>
#include <cstring>
#include <algorithm>
#include <atomic>
#include <functional>
#include <mutex>
#include <new>
#include <thread>
#include <type_traits>
#include <vector>

#include "sdnn_internal.h"

// ---------------------------------------------------------------------------
// device helpers
// ---------------------------------------------------------------------------

#define WAVES_PER_BLOCK 4 // product kernels: 4 rows per workgroup (measured best of 1, 2, 4, 8)
#define UPD_WAVES 1       // update kernel: one wavefront per workgroup (measured best of 1, 2, 4, 8)
#define BLOCK_THREADS (64 * WAVES_PER_BLOCK)

template <int V> __device__ __forceinline__ void ldv(const float *p, float (&x)[V]);
template <> __device__ __forceinline__ void ldv<1>(const float *p, float (&x)[1]) { x[0] = *p; }
template <> __device__ __forceinline__ void ldv<2>(const float *p, float (&x)[2])
{
    const float2 t = *reinterpret_cast<const float2 *>(p);
    x[0] = t.x; x[1] = t.y;
}
template <> __device__ __forceinline__ void ldv<4>(const float *p, float (&x)[4])
{
    const float4 t = *reinterpret_cast<const float4 *>(p);
    x[0] = t.x; x[1] = t.y; x[2] = t.z; x[3] = t.w;
}
template <int V> __device__ __forceinline__ void stv(float *p, const float (&x)[V]);
template <> __device__ __forceinline__ void stv<1>(float *p, const float (&x)[1]) { *p = x[0]; }
template <> __device__ __forceinline__ void stv<2>(float *p, const float (&x)[2])
{
    *reinterpret_cast<float2 *>(p) = make_float2(x[0], x[1]);
}
template <> __device__ __forceinline__ void stv<4>(float *p, const float (&x)[4])
{
    *reinterpret_cast<float4 *>(p) = make_float4(x[0], x[1], x[2], x[3]);
}

// Gather of V consecutive floats of an activation row through a buffer
// descriptor: the address is (uniform base) + (scalar row offset) + (lane
// offset), so a load costs one SGPR and no per-load address VGPRs.  Offsets are
// 32-bit byte offsets: an activation block must stay below 4 GiB (checked by the
// host).  Reads past num_records return 0 instead of faulting.
typedef unsigned int u32x2 __attribute__((ext_vector_type(2)));
typedef unsigned int u32x4 __attribute__((ext_vector_type(4)));
__device__ __forceinline__ __amdgpu_buffer_rsrc_t make_rsrc(const float *base, size_t bytes)
{
    return __builtin_amdgcn_make_buffer_rsrc((void *)base, 0, (int)(unsigned)bytes, 0x00020000);
}
template <int V>
__device__ __forceinline__ void gatherv(__amdgpu_buffer_rsrc_t r, unsigned lane_off, unsigned row_off,
                                        float (&x)[V])
{
    if constexpr (V == 1) {
        x[0] = __uint_as_float(__builtin_amdgcn_raw_buffer_load_b32(r, (int)lane_off, (int)row_off, 0));
    } else if constexpr (V == 2) {
        const u32x2 t = __builtin_amdgcn_raw_buffer_load_b64(r, (int)lane_off, (int)row_off, 0);
        x[0] = __uint_as_float(t.x); x[1] = __uint_as_float(t.y);
    } else {
        const u32x4 t = __builtin_amdgcn_raw_buffer_load_b128(r, (int)lane_off, (int)row_off, 0);
        x[0] = __uint_as_float(t.x); x[1] = __uint_as_float(t.y);
        x[2] = __uint_as_float(t.z); x[3] = __uint_as_float(t.w);
    }
}

// Activations (the paper's Eq. 3 leaves f open; Section 6.1 trains with the sigmoid).
//   ACT_RELU_CAP: f(z) = min(max(z, 0), cap), f' = [0 < x < cap] from the stored output x
//   ACT_SIGMOID:  f(z) = 1 / (1 + exp(-z)),   f' = x (1 - x)     from the stored output x
#define ACT_RELU_CAP 0
#define ACT_SIGMOID 1
__device__ __forceinline__ float act_apply(int act, double z, float capf)
{
    if (act == ACT_SIGMOID) return (float)(1.0 / (1.0 + exp(-z)));
    const double cap = (double)capf;
    z = z < 0.0 ? 0.0 : z;
    z = z > cap ? cap : z;
    return (float)z;
}
// value * f'(z) with f' taken from the stored output x
__device__ __forceinline__ float act_backprop(int act, double value, float x, float capf)
{
    if (act == ACT_SIGMOID) {
        const double xd = (double)x;
        return (float)(value * (xd * (1.0 - xd)));
    }
    return (x > 0.0f && x < capf) ? (float)value : 0.0f;
}

// Orders the LDS (or in-place global) accesses of the lanes of one wavefront: what the lanes wrote before
// is visible to the other lanes after, and nothing is moved across.  Costs no instruction beyond the wait
// for the outstanding accesses.
__device__ __forceinline__ void wave_lds_sync()
{
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

// Workgroup ids are handed to the 8 XCDs round-robin and each XCD has its own
// L2.  Give every XCD whole batch tiles (all row groups of tile x, x+8, ...)
// so that the activation slab of a tile is gathered through one L2 only.  The
// tiles left over when the tile count is not a multiple of 8 are shared.
__device__ __forceinline__ void map_block(unsigned bid, unsigned n_tiles, unsigned n_rg,
                                          unsigned &tile, unsigned &rg)
{
    const unsigned t8 = n_tiles & ~7u;
    const unsigned n8 = t8 * n_rg;
    if (bid < n8) {
        const unsigned xcd = bid & 7u, k = bid >> 3;
        tile = xcd + 8u * (k / n_rg);
        rg = k % n_rg;
    } else {
        const unsigned k = bid - n8;
        tile = t8 + k / n_rg;
        rg = k % n_rg;
    }
}

// ---------------------------------------------------------------------------
// K1 / K2: row-per-wavefront sparse product with fused epilogue
//   MODE 0 (forward, Eq. 3):   out = min(max(sum + bias[row], 0), cap)
//   MODE 1 (backward, Eq. 7):  out = sum * [0 < Xprev[row] < cap]; the values
//                              are read through the transposed index (perm)
// ---------------------------------------------------------------------------
// 128 bytes: two cache lines of kernel arguments, which every wavefront of a launch waits for (with what only the gradient
// sweeps need in it, and 64-bit sizes, a launch of 256 workgroups takes 0.04 us longer).
struct SpmmArgs {
    const int32_t *idx;
    const float *vals;
    const int32_t *perm;  // MODE 1 only
    const int4 *sched;    // per task: {row, first entry, end of entries, 0}, rows by decreasing length
    const float *in;      // [n_cols][ld_in]
    uint32_t in_bytes;
    int32_t n_cols;
    float *out;           // [n_rows][ld_out]
    const float *aux;     // MODE 0: bias [n_rows] (may be NULL); MODE 1: Xprev [n_rows][ld_out]
    int32_t n_rows, B;    // B: samples (columns that matter); fills_up(B, ld_out): zeros are stored up to a group of four
    int32_t ld_in, ld_out; // floats per activation row
    uint32_t n_tiles, n_rg, n_vblocks, tile_base;
    float cap;
    int32_t act;
    const int32_t *n_live; // NULL, or the number of leading columns of the block that still matter (device)
    int32_t *flags;        // NULL, or MODE 0: flags[s] is set to 1 for every sample s with a non-zero output
    const int32_t *row_ptr;
};
// Whether the rows of an output have room for whole groups of four samples (the library's own arrays) and B leaves the last one
// part-filled: its other columns are stored as zeros, which the kernels with four samples per lane rely on.  (Uniform, from
// what a kernel has loaded anyway: as an argument of its own, masked value by value, it took 0.7 % of the products.)
__device__ __forceinline__ bool fills_up(int B, int ld_out) { return (B & 3) != 0 && ld_out > B; }
__device__ __forceinline__ bool is_fill(int s, int B) { return s >= B && s < ((B + 3) & ~3); }
// The lane's number, made where it is used: as a value that the compiler may keep or move ahead of the loops, the rare store
// of zeros costs k_spmm 2 to 8 registers throughout, and some of its variants a wavefront per SIMD.  (Not in the panel sweep:
// there it took the forward of 65536 neurons from 20.4 to 27.3 ms.)
__device__ __forceinline__ int lane_number()
{
    int n;
    asm volatile("v_mbcnt_lo_u32_b32 %0, -1, 0\n\tv_mbcnt_hi_u32_b32 %0, -1, %0" : "=v"(n));
    return n;
}

struct GradArgs : SpmmArgs {
    float *g_part[2];  // gradient of the stored entries over the samples of the first / second tile, in the order of the
                       // transposed index [nnz]
    int32_t store_out; // 0 = only the gradient is wanted (first layer: there is no Delta_0)
};
static_assert(sizeof(SpmmArgs) == 128, "see above");

// The part of a row task that does not depend on the previous layer's output:
// which row, where its entries are, and its first (up to) 64 entries, entry k
// held by lane k.
struct RowMeta {
    int row, beg, end;
    int c_l;
    float w_l;
    int p_l; // MODE 1: position of the entry in the CSR arrays
};

template <int MODE>
__device__ __forceinline__ void load_chunk(const int32_t *idx, const float *vals, const int32_t *perm,
                                           int base, int end, int lane, int &c_l, float &w_l, int &p_l)
{
    c_l = 0;
    w_l = 0.0f;
    p_l = 0;
    if (base + lane < end) {
        c_l = idx[base + lane];
        if (MODE == 1) {
            p_l = perm[base + lane];
            w_l = vals[p_l];
        } else {
            w_l = vals[base + lane];
        }
    }
}

template <int MODE>
__device__ __forceinline__ RowMeta load_meta(const int4 *sched, const int32_t *idx, const float *vals,
                                             const int32_t *perm, int r, int lane)
{
    RowMeta m;
    const int4 t = sched[r]; // one (scalar) load instead of the chain order -> row_ptr
    m.row = t.x;
    m.beg = t.y;
    m.end = t.z;
    load_chunk<MODE>(idx, vals, perm, m.beg, m.end, lane, m.c_l, m.w_l, m.p_l);
    return m;
}

// One row of the product for the 64*V samples of one batch tile.  All 64 lanes
// must be active (lane k's registers are read by readlane); lanes past the end
// of the batch redo sample 0 and do not store.
template <int V, int MODE, int U, int ACT>
__device__ __forceinline__ void spmm_row(RowMeta m, const int32_t *idx, const float *vals,
                                         const int32_t *perm, const float *in, size_t in_bytes,
                                         float *out, const float *aux, int B, int ld_in, int ld_out, float capf,
                                         int act, unsigned tile, int lane, int32_t *flags)
{
    const int s_own = (int)tile * (64 * V) + lane * V;
    const bool live = s_own < B;
    const int s = live ? s_own : 0;
    const size_t ld = (size_t)ld_out;
    const unsigned so = 4u * (unsigned)s;      // byte offset of the lane inside an activation row
    const unsigned ldb = 4u * (unsigned)ld_in; // bytes per activation row
    const __amdgpu_buffer_rsrc_t rin = make_rsrc(in, in_bytes);

    // operands of the epilogue, requested early so that they arrive with the gathers
    float xp[V];
    double b = 0.0;
    if (MODE == 0) {
        if (aux) b = (double)aux[m.row];
    } else {
        ldv<V>(aux + (size_t)m.row * ld + s, xp);
    }

    double acc[V];
#pragma unroll
    for (int v = 0; v < V; ++v) acc[v] = 0.0;

    // Long rows (U == 16), forward: a row's entries are the same for all lanes and never change inside a kernel, so they
    // are read through the scalar cache, 16 columns and 16 weights at a time and a group ahead, straight into scalar
    // registers: no lane broadcasts (2 of 11 vector instructions per entry at four samples per lane).
    if constexpr (MODE == 0 && U == 16) {
        typedef int i32x16 __attribute__((ext_vector_type(16)));
        typedef float f32x16 __attribute__((ext_vector_type(16)));
        const int __attribute__((address_space(4))) *sidx = (const int __attribute__((address_space(4))) *)idx;
        const float __attribute__((address_space(4))) *svals = (const float __attribute__((address_space(4))) *)vals;
        int g = m.beg;
        i32x16 c, cn;
        f32x16 w, wn;
        if (g + 16 <= m.end) {
#pragma unroll
            for (int k = 0; k < 16; ++k) { c[k] = sidx[g + k]; w[k] = svals[g + k]; }
        }
        for (; g + 16 <= m.end; g += 16) {
            if (g + 32 <= m.end) {
#pragma unroll
                for (int k = 0; k < 16; ++k) { cn[k] = sidx[g + 16 + k]; wn[k] = svals[g + 16 + k]; }
            }
            float x[16][V];
#pragma unroll
            for (int k = 0; k < 16; ++k) gatherv<V>(rin, so, (unsigned)c[k] * ldb, x[k]);
#pragma unroll
            for (int k = 0; k < 16; ++k) {
                const double wk = (double)w[k];
#pragma unroll
                for (int v = 0; v < V; ++v) acc[v] = fma(wk, (double)x[k][v], acc[v]);
            }
            c = cn;
            w = wn;
        }
        if (g < m.end) { // the row's last entries, fewer than 16: same order, every entry guarded (wave-uniform)
            const int n = m.end - g;
            float x[16][V];
#pragma unroll
            for (int k = 0; k < 16; ++k)
                if (k < n) gatherv<V>(rin, so, (unsigned)sidx[g + k] * ldb, x[k]);
#pragma unroll
            for (int k = 0; k < 16; ++k)
                if (k < n) {
                    const double wk = (double)svals[g + k];
#pragma unroll
                    for (int v = 0; v < V; ++v) acc[v] = fma(wk, (double)x[k][v], acc[v]);
                }
        }
    } else {
    // U gathers are in flight per lane before the first of them is consumed
    int c_l = m.c_l, p_l = m.p_l;
    float w_l = m.w_l;
    for (int base = m.beg; base < m.end; base += 64) {
        const int n = min(64, m.end - base);
        // the entries of the next 64 are requested before this chunk's gathers, not after them
        int c_n = 0, p_n = 0;
        float w_n = 0.0f;
        if (base + 64 < m.end) load_chunk<MODE>(idx, vals, perm, base + 64, m.end, lane, c_n, w_n, p_n);
        for (int g = 0; g < n; g += U) {
            float x[U][V];
            if (g + U <= n) {
#pragma unroll
                for (int k = 0; k < U; ++k) {
                    const int c = __builtin_amdgcn_readlane(c_l, g + k);
                    gatherv<V>(rin, so, (unsigned)c * ldb, x[k]);
                }
#pragma unroll
                for (int k = 0; k < U; ++k) {
                    const double wk = (double)__int_as_float(__builtin_amdgcn_readlane(__float_as_int(w_l), g + k));
#pragma unroll
                    for (int v = 0; v < V; ++v) acc[v] = fma(wk, (double)x[k][v], acc[v]);
                }
            } else {
                // ragged end of the row: same order, every entry guarded (wave-uniform branches)
#pragma unroll
                for (int k = 0; k < U; ++k)
                    if (g + k < n) {
                        const int c = __builtin_amdgcn_readlane(c_l, g + k);
                        gatherv<V>(rin, so, (unsigned)c * ldb, x[k]);
                    }
#pragma unroll
                for (int k = 0; k < U; ++k)
                    if (g + k < n) {
                        const double wk = (double)__int_as_float(__builtin_amdgcn_readlane(__float_as_int(w_l), g + k));
#pragma unroll
                        for (int v = 0; v < V; ++v) acc[v] = fma(wk, (double)x[k][v], acc[v]);
                    }
            }
        }
        c_l = c_n;
        w_l = w_n;
        p_l = p_n;
    }
    }

    float o[V];
    if (MODE == 0) {
#pragma unroll
        for (int v = 0; v < V; ++v) o[v] = act_apply(ACT, acc[v] + b, capf); // compile-time: exp() costs registers
    } else {
#pragma unroll
        for (int v = 0; v < V; ++v) o[v] = act_backprop(act, acc[v], xp[v], capf);
    }
    if (V > 1 && s + V > B) { // the batch's last piece
#pragma unroll
        for (int v = 0; v < V; ++v)
            if (s + v >= B) o[v] = 0.0f;
    }
    if (live) stv<V>(out + (size_t)m.row * ld + s, o);
    if (MODE == 0 && flags != nullptr && live) { // other rows store the same 1: no ordering needed
#pragma unroll
        for (int v = 0; v < V; ++v)
            if (o[v] != 0.0f) flags[s + v] = 1;
    }
}

// Zeros after a row's last sample, by the wavefront of its last tile.  (In spmm_row itself they take 2 to 6 more registers
// where a wavefront walks the tiles, and a wavefront per SIMD with them.)
template <int V> __device__ __forceinline__ void fill_row(const SpmmArgs &a, int row, unsigned tile)
{
    if (V < 4 && fills_up(a.B, a.ld_out) && (tile + 1) * (64 * V) >= (unsigned)a.B) {
        const int s = a.B + lane_number();
        if (is_fill(s, a.B)) a.out[(size_t)row * a.ld_out + s] = 0.0f;
    }
}

// The grid is sized to what the chip holds at once and every workgroup walks
// "virtual blocks" blockIdx.x, blockIdx.x + gridDim.x, ...: a wavefront that
// handles one short row and exits costs more to dispatch than to run.
// gridDim.x is a multiple of 8, so a workgroup keeps its XCD's tiles.
// ACT: the activation of the forward epilogue, fixed at compile time (the sigmoid's exp() would
// otherwise set the register count, and with it the occupancy, of the ReLU kernels too); the
// backward epilogue reads a.act.
template <int V, int MODE, int U, bool TILES_INNER, int ACT>
__global__ void __launch_bounds__(BLOCK_THREADS) k_spmm(const SpmmArgs a)
{
    const int lane = threadIdx.x & 63;
    const unsigned wave = threadIdx.x >> 6;
    unsigned n_tiles = a.n_tiles, n_vblocks = a.n_vblocks;
    if (a.n_live) { // only the batch tiles that hold live columns
        n_tiles = min(n_tiles, ((unsigned)*a.n_live + 64u * V - 1u) / (64u * V));
        n_vblocks = n_tiles * a.n_rg;
    }
    if constexpr (TILES_INNER) {
        // a few batch tiles shared by all XCDs: a wavefront keeps its row and walks the tiles, so the row's
        // task record and entries are fetched once, and the whole chip gathers from one tile's slab at a time
        for (unsigned rg = blockIdx.x; rg < a.n_rg; rg += gridDim.x) {
            const int r = __builtin_amdgcn_readfirstlane((int)(rg * WAVES_PER_BLOCK + wave));
            if (r >= a.n_rows) continue;
            const RowMeta m = load_meta<MODE>(a.sched, a.idx, a.vals, a.perm, r, lane);
            // (one sample per lane comes here only where an operand's rows are not filled up: nobody reads the zeros)
            if constexpr (V > 1) fill_row<V>(a, m.row, n_tiles - 1 + a.tile_base);
            for (unsigned tile = 0; tile < n_tiles; ++tile)
                spmm_row<V, MODE, U, ACT>(m, a.idx, a.vals, a.perm, a.in, a.in_bytes, a.out, a.aux, a.B, a.ld_in, a.ld_out, a.cap, a.act,
                                          tile + a.tile_base, lane, a.flags);
        }
        return;
    }
    for (unsigned vb = blockIdx.x; vb < n_vblocks; vb += gridDim.x) {
        unsigned tile, rg;
        map_block(vb, n_tiles, a.n_rg, tile, rg);
        const int r = __builtin_amdgcn_readfirstlane((int)(rg * WAVES_PER_BLOCK + wave));
        if (r >= a.n_rows) continue;
        const RowMeta m = load_meta<MODE>(a.sched, a.idx, a.vals, a.perm, r, lane);
        spmm_row<V, MODE, U, ACT>(m, a.idx, a.vals, a.perm, a.in, a.in_bytes, a.out, a.aux, a.B, a.ld_in, a.ld_out, a.cap, a.act, tile + a.tile_base, lane, a.flags);
        fill_row<V>(a, m.row, tile + a.tile_base);
    }
}

// ---------------------------------------------------------------------------
// K1r / K2r: the product with several rows per wavefront, for batches that do not fill it with one.
// A row takes G lanes, four consecutive samples per lane (so G = 16 for 64 samples, 32 for 128), and a
// wavefront 64 / G rows: one gather instruction fetches 16 bytes a lane for 64 / G entries.  Every quad of
// lanes holds 16 entries of its row, four per lane, and hands them round with quad_perm; slots past the end of
// a row carry weight 0 and a column outside the operand, which reads as 0 (a neuron's activation might be infinite or NaN):
// they add an exact zero.  Same order of the sums as in k_spmm.
//
// A wavefront per row (k_spmm with one sample per lane) is bound by the rate of gather instructions (10 clocks each,
// whatever the number of samples) up to 64 samples, and by the L2 misses of a 256-sample tile beyond.  Here
// one instruction serves 2 to 16 entries.  Forward, us per layer, before and after: 65536 neurons, 16 samples 49.8 ->
// 17.8; 16384 neurons 12.7 -> 6.8 (16), 13.4 -> 10.2 (64), 23.1 -> 17.4 (100), 53 -> 31 (256); no gain at 4096 neurons and 128
// samples (6.7 in two half batches on two streams, 6.8 in this one launch).
// A last tile that the batch fills only in part must not touch lines of its own for the idle lanes (when they read the
// batch's first samples: 32000 neurons, 33 samples 31.2 us per layer, with the tile's first 19.6; 100 samples 50 and 38.4).
// ---------------------------------------------------------------------------
template <int LANE> __device__ __forceinline__ int quad_bcast(int v)
{
    return __builtin_amdgcn_mov_dpp(v, LANE * 0x55, 0xf, 0xf, true);
}
__device__ __forceinline__ float4 as_f4(u32x4 t)
{
    return make_float4(__uint_as_float(t.x), __uint_as_float(t.y), __uint_as_float(t.z), __uint_as_float(t.w));
}
struct __attribute__((packed, aligned(4))) I4 { int v[4]; };
struct __attribute__((packed, aligned(4))) F4 { float v[4]; };
// The entries of a quad's row in groups of sixteen, four per lane: entries past the end of the row (what follows it in
// the arrays is read) count as zeros, at column n_cols: past the end of the operand.
struct QuadEntries {
    I4 c;
    F4 w;
    __device__ __forceinline__ void fetch(const int32_t *idx, const float *vals, int p, int end, int n_cols)
    {
        if (p < end) {
            c = *(const I4 *)(idx + p);
            w = *(const F4 *)(vals + p);
        }
#pragma unroll
        for (int i = 0; i < 4; ++i)
            if (p + i >= end) { c.v[i] = n_cols; w.v[i] = 0.0f; }
    }
};
// The operand rows of the four entries that quad lane H holds, and their weights.
template <int H>
__device__ __forceinline__ void quad_gather(const QuadEntries &q, __amdgpu_buffer_rsrc_t rin, unsigned ldb, unsigned so,
                                            float4 (&x)[4], int (&wv)[4])
{
#pragma unroll
    for (int u = 0; u < 4; ++u) {
        const unsigned c = (unsigned)quad_bcast<H>(q.c.v[u]);
        wv[u] = quad_bcast<H>(__float_as_int(q.w.v[u]));
        x[u] = as_f4(__builtin_amdgcn_raw_buffer_load_b128(rin, (int)(__umul24(c, ldb) + so), 0, 0));
    }
}
template <int G, int ACT>
__global__ void __launch_bounds__(BLOCK_THREADS) k_rows(const SpmmArgs a)
{
    constexpr int R = 64 / G;
    const int lane = threadIdx.x & 63;
    // all row groups of the first tile of samples, then those of the second, ...
    const unsigned tile = blockIdx.x / a.n_rg, rg = blockIdx.x - tile * a.n_rg;
    const int r = (int)((rg * WAVES_PER_BLOCK + (threadIdx.x >> 6)) * R) + lane / G;
    const unsigned ldb = 4u * (unsigned)a.ld_in;
    // lanes past the end of the batch redo the tile's first samples: the lines that the other lanes fetch anyway
    const int s_tile = (int)(tile + a.tile_base) * (4 * G), s_own = s_tile + 4 * (lane & (G - 1));
    const bool live = s_own < a.B;
    const int s = live ? s_own : s_tile;
    const unsigned so = 4u * (unsigned)s;
    const __amdgpu_buffer_rsrc_t rin = make_rsrc(a.in, a.in_bytes);
    int4 t = make_int4(0, 0, 0, 0);
    if (r < a.n_rows) t = a.sched[r];
    const int row = t.x, end = t.z;
    int p = t.y + 4 * (lane & 3), left = end - t.y; // left: entries of this lane's row still to do
    QuadEntries q;
    q.fetch(a.idx, a.vals, p, end, a.n_cols);
    const double b = a.aux ? (double)a.aux[row] : 0.0;
    double acc[4] = {0.0, 0.0, 0.0, 0.0};
    for (bool more = __ballot(left > 0) != 0; more;) {
        more = __ballot(left > 16) != 0;
        float4 x[4][4];
        int wv[4][4];
        quad_gather<0>(q, rin, ldb, so, x[0], wv[0]);
        quad_gather<1>(q, rin, ldb, so, x[1], wv[1]);
        quad_gather<2>(q, rin, ldb, so, x[2], wv[2]);
        quad_gather<3>(q, rin, ldb, so, x[3], wv[3]);
        p += 16;
        left -= 16;
        if (more) q.fetch(a.idx, a.vals, p, end, a.n_cols);
#pragma unroll
        for (int h = 0; h < 4; ++h)
#pragma unroll
            for (int u = 0; u < 4; ++u) {
                const double wk = (double)__int_as_float(wv[h][u]);
                acc[0] = fma(wk, (double)x[h][u].x, acc[0]);
                acc[1] = fma(wk, (double)x[h][u].y, acc[1]);
                acc[2] = fma(wk, (double)x[h][u].z, acc[2]);
                acc[3] = fma(wk, (double)x[h][u].w, acc[3]);
            }
    }
    if (r >= a.n_rows || !live) return;
    float o[4];
#pragma unroll
    for (int v = 0; v < 4; ++v) o[v] = act_apply(ACT, acc[v] + b, a.cap);
    if (s + 4 > a.B) { // the batch's last group
#pragma unroll
        for (int v = 1; v < 4; ++v)
            if (s + v >= a.B) o[v] = 0.0f;
    }
    float *dst = a.out + (size_t)row * a.ld_out + s;
    if ((a.ld_out & 3) == 0 && ((size_t)a.out & 15) == 0) {
        stv<4>(dst, o);
    } else { // the caller's rows of B floats
#pragma unroll
        for (int v = 0; v < 4; ++v)
            if (s + v < a.B) dst[v] = o[v];
    }
}

// Exchange with the lane that differs in one bit of its number (bits 1 and 0: exactly that lane; bit 3: lane ^ 8; bit 2:
// lane ^ 7, which is as good where all lanes that agree in the higher bits hold the same set of values).
template <int BIT> __device__ __forceinline__ double lane_exchange(double v)
{
    constexpr int CTRL = BIT == 3 ? 0x128 : BIT == 2 ? 0x141 : BIT == 1 ? 0x4e : 0xb1; // row_ror:8, row_half_mirror, quad_perm
    const int lo = __builtin_amdgcn_mov_dpp(__double2loint(v), CTRL, 0xf, 0xf, true);
    const int hi = __builtin_amdgcn_mov_dpp(__double2hiint(v), CTRL, 0xf, 0xf, true);
    return __hiloint2double(hi, lo);
}
// The value of the lane whose number differs in exactly that bit (bits 0 to 3), and the sum with it (bits 4 and 5).
template <int BIT> __device__ __forceinline__ double lane_xor(double v)
{
    if constexpr (BIT != 2) {
        return lane_exchange<BIT>(v);
    } else { // lane ^ 7, then ^ 3
        const int lo = __builtin_amdgcn_mov_dpp(__builtin_amdgcn_mov_dpp(__double2loint(v), 0x141, 0xf, 0xf, true), 0x1b, 0xf, 0xf, true);
        const int hi = __builtin_amdgcn_mov_dpp(__builtin_amdgcn_mov_dpp(__double2hiint(v), 0x141, 0xf, 0xf, true), 0x1b, 0xf, 0xf, true);
        return __hiloint2double(hi, lo);
    }
}
template <int BIT> __device__ __forceinline__ double add_lane_xor(double v)
{
    const unsigned l = (unsigned)__double2loint(v), h = (unsigned)__double2hiint(v);
    const auto lo = BIT == 5 ? __builtin_amdgcn_permlane32_swap(l, l, false, false) : __builtin_amdgcn_permlane16_swap(l, l, false, false);
    const auto hi = BIT == 5 ? __builtin_amdgcn_permlane32_swap(h, h, false, false) : __builtin_amdgcn_permlane16_swap(h, h, false, false);
    return __hiloint2double((int)hi[0], (int)lo[0]) + __hiloint2double((int)hi[1], (int)lo[1]);
}
// The value of the lane N places on in its group of sixteen.
template <int N> __device__ __forceinline__ double row_rotate(double v)
{
    const int lo = __builtin_amdgcn_mov_dpp(__double2loint(v), 0x120 + N, 0xf, 0xf, true);
    const int hi = __builtin_amdgcn_mov_dpp(__double2hiint(v), 0x120 + N, 0xf, 0xf, true);
    return __hiloint2double(hi, lo);
}
// One halving step of a sum over lanes of N values: the lane keeps the half of the values whose number has the bit that
// its own number has in place BIT, and adds its partner's share of them.
template <int N, int BIT> __device__ __forceinline__ void halve(double (&p)[4], int lane)
{
#pragma unroll
    for (int j = 0; j < N / 2; ++j) {
        if constexpr (BIT >= 4) {
            const unsigned al = (unsigned)__double2loint(p[j]), ah = (unsigned)__double2hiint(p[j]);
            const unsigned bl = (unsigned)__double2loint(p[j + N / 2]), bh = (unsigned)__double2hiint(p[j + N / 2]);
            const auto lo = BIT == 5 ? __builtin_amdgcn_permlane32_swap(al, bl, false, false) : __builtin_amdgcn_permlane16_swap(al, bl, false, false);
            const auto hi = BIT == 5 ? __builtin_amdgcn_permlane32_swap(ah, bh, false, false) : __builtin_amdgcn_permlane16_swap(ah, bh, false, false);
            p[j] = __hiloint2double((int)hi[0], (int)lo[0]) + __hiloint2double((int)hi[1], (int)lo[1]);
        } else {
            const bool up = (lane >> BIT) & 1;
            const double keep = up ? p[j + N / 2] : p[j], send = up ? p[j] : p[j + N / 2];
            p[j] = keep + lane_exchange<BIT>(send);
        }
    }
}
// Sums of four values over the G lanes of a row: afterwards p[0] holds the sum of value reduced_index<G>(lane).
template <int G> __device__ __forceinline__ void reduce4(double (&p)[4], int lane)
{
    if constexpr (G == 64) { halve<4, 5>(p, lane); halve<2, 4>(p, lane); }
    if constexpr (G == 32) { halve<4, 4>(p, lane); halve<2, 3>(p, lane); }
    if constexpr (G == 16) { halve<4, 3>(p, lane); halve<2, 2>(p, lane); }
    if constexpr (G == 8) { halve<4, 2>(p, lane); halve<2, 1>(p, lane); }
    if constexpr (G == 4) { halve<4, 1>(p, lane); halve<2, 0>(p, lane); }
    if constexpr (G >= 64) p[0] += lane_exchange<3>(p[0]);
    if constexpr (G >= 32) p[0] += lane_exchange<2>(p[0]);
    if constexpr (G >= 16) p[0] += lane_exchange<1>(p[0]);
    if constexpr (G >= 8) p[0] += lane_exchange<0>(p[0]);
}
template <int G> __device__ __forceinline__ int reduced_index(int lane) { return (lane / (G / 4)) & 3; }
// The sum of a float over two neighbouring groups of 16 lanes, in all of them.
__device__ __forceinline__ float add_neighbour16(float g)
{
    const auto t = __builtin_amdgcn_permlane16_swap(__float_as_uint(g), __float_as_uint(g), false, false);
    return (float)((double)__uint_as_float(t[0]) + (double)__uint_as_float(t[1]));
}

// The backward sweep that also forms the gradient of the stored entries, in the manner of k_rows.  The lanes of row i of
// W_l^T hold X_{l-1}(i, :), four samples each, gather Delta_l(j, :) for every entry (j, i) and sum its products with
// X_{l-1}(i, :) over the samples: four in the lane, the rest over the row's lanes, four entries at a time while the
// operand rows of the next four are on their way.
// Against the sweep that parks the gathered rows in LDS (k_bwd_grad; four samples per lane for long rows): one instead of
// twelve vector instructions per entry and 64 samples for the parking and its re-reading, and a gather instruction per 1024
// bytes.  Backward and gradient, us per layer: 65536 neurons 80 -> 69.7 (64 samples), 70.6 -> 29.1 (16); 16384 neurons 21.1 ->
// 14.4 (64), 31.8 -> 25.3 (128; two launches on two streams before); 10007 neurons, 99 samples 32.5 (two
// separate kernels) -> 17.6 + 3; 8192 neurons of 820 entries 420 -> 331 (256 samples), 410 -> 127 (64).
// TWO (G = 32, 128 samples): the gradient is the sum of two windows of 64 samples, each rounded to fp32 (two_windows).
template <int G, bool TWO>
__global__ void __launch_bounds__(BLOCK_THREADS) k_bwd_rows(const GradArgs a)
{
    static_assert(!TWO || G == 32, "two windows of 16 lanes");
    constexpr int R = 64 / G;
    const int lane = threadIdx.x & 63;
    const unsigned tile = blockIdx.x / a.n_rg, rg = blockIdx.x - tile * a.n_rg;
    const int r = (int)((rg * WAVES_PER_BLOCK + (threadIdx.x >> 6)) * R) + lane / G;
    const unsigned ldb = 4u * (unsigned)a.ld_in;
    const int s_own = (int)tile * (4 * G) + 4 * (lane & (G - 1));
    const bool live = s_own < a.B && r < a.n_rows;
    const int s = s_own < a.B ? s_own : 0;
    const unsigned so = 4u * (unsigned)s;
    const __amdgpu_buffer_rsrc_t rin = make_rsrc(a.in, a.in_bytes);
    float *__restrict__ g_part = tile == 0 ? a.g_part[0] : a.g_part[1];
    int4 t = make_int4(0, 0, 0, 0);
    if (r < a.n_rows) t = a.sched[r];
    const int row = t.x, end = t.z;
    int p = t.y + 4 * (lane & 3), left = end - t.y; // left: entries of this lane's row still to do
    QuadEntries q, qn;
    q.fetch(a.idx, a.vals, p, end, a.n_cols);
    float xp[4] = {0.0f, 0.0f, 0.0f, 0.0f}; // lanes outside the batch add nothing to the gradient
    if (live) ldv<4>(a.aux + (size_t)row * a.ld_out + s, xp);
    double xd[4], acc[4] = {0.0, 0.0, 0.0, 0.0};
#pragma unroll
    for (int v = 0; v < 4; ++v) xd[v] = (double)xp[v];
    constexpr int SUM = TWO ? 16 : G; // lanes of a window
    int e0 = t.y + reduced_index<SUM>(lane); // the entry whose gradient this lane stores
    float4 x0[4], x1[4];
    int w0[4], w1[4];
    auto consume = [&](const float4 (&x)[4], const int (&wv)[4]) {
        double pr[4];
#pragma unroll
        for (int u = 0; u < 4; ++u) {
            const double wk = (double)__int_as_float(wv[u]);
            const double d0 = (double)x[u].x, d1 = (double)x[u].y, d2 = (double)x[u].z, d3 = (double)x[u].w;
            acc[0] = fma(wk, d0, acc[0]);
            acc[1] = fma(wk, d1, acc[1]);
            acc[2] = fma(wk, d2, acc[2]);
            acc[3] = fma(wk, d3, acc[3]);
            pr[u] = fma(d3, xd[3], fma(d2, xd[2], fma(d1, xd[1], d0 * xd[0])));
        }
        // added here: the compiler would move these sums past the branches below and keep every converted operand until
        // then (214 registers instead of 120)
        asm volatile("" : "+v"(acc[0]), "+v"(acc[1]), "+v"(acc[2]), "+v"(acc[3]));
        reduce4<SUM>(pr, lane);
        float g = (float)pr[0];
        if (TWO) g = add_neighbour16(g);
        if ((lane & (SUM / 4 - 1)) == 0 && !(TWO && (lane & 16)) && e0 < end) g_part[e0] = g;
        e0 += 4;
    };
    quad_gather<0>(q, rin, ldb, so, x0, w0);
    for (bool more = __ballot(left > 0) != 0; more;) {
        more = __ballot(left > 16) != 0;
        p += 16;
        left -= 16;
        if (more) qn.fetch(a.idx, a.vals, p, end, a.n_cols);
        quad_gather<1>(q, rin, ldb, so, x1, w1);
        consume(x0, w0);
        quad_gather<2>(q, rin, ldb, so, x0, w0);
        consume(x1, w1);
        quad_gather<3>(q, rin, ldb, so, x1, w1);
        consume(x0, w0);
        if (more) {
            q = qn;
            quad_gather<0>(q, rin, ldb, so, x0, w0);
        }
        consume(x1, w1);
    }
    if (!a.store_out || !live) return;
    float o[4];
#pragma unroll
    for (int v = 0; v < 4; ++v) o[v] = act_backprop(a.act, acc[v], xp[v], a.cap);
    if (s + 4 > a.B) { // the batch's last group
#pragma unroll
        for (int v = 1; v < 4; ++v)
            if (s + v >= a.B) o[v] = 0.0f;
    }
    stv<4>(a.out + (size_t)row * a.ld_out + s, o);
}

// The same sweep for long rows and more than 128 samples: a wavefront per row.  k_bwd_rows<64> keeps the vector units issuing in
// 91 % of its clocks there (23 instructions per entry, 6.5 of them the sum over the lanes, 3 to hand the entries round).  Here a
// row's entries come through the scalar cache, a group of sixteen ahead, and the sums over the lanes are products with ones on the
// matrix cores (4x4x4, fp64), which run beside the vector units: 15 vector and 1.25 matrix instructions per entry.
//   The product of lanes (16 k + 4 b + i) with B[k][j] = [j == u] leaves the sums over k of entry u in the lanes (16 i + 4 b + u) and
//   adds nothing to the others; the sums of four entries, as the right operand of A[i][k] = [i == q], go to the lanes (16 q + 4 b + u).
//   Sixteen entries end up in sixteen lanes, and two rotations add the four b.
// 0 times infinity is NaN, so where one of the sixteen sums is not finite they are formed one by one instead.
// Per layer of 8192 neurons of 820 entries, 256 samples, between other kernels 344 -> 291 us: 6.9 GB of gathered rows at 24 TB/s, where
// a stream of such gathers alone reaches 26 to 31.  (Eight to sixteen gathers in flight, four or five wavefronts per SIMD: the same.)
typedef int i32x16 __attribute__((ext_vector_type(16)));
typedef float f32x16 __attribute__((ext_vector_type(16)));
__global__ void __launch_bounds__(BLOCK_THREADS) k_bwd_long(const GradArgs a)
{
    typedef const int __attribute__((address_space(4))) *int_ptr;
    typedef const float __attribute__((address_space(4))) *float_ptr;
    const int lane = threadIdx.x & 63;
    const int r = __builtin_amdgcn_readfirstlane((int)(blockIdx.x * WAVES_PER_BLOCK + (threadIdx.x >> 6)));
    if (r >= a.n_rows) return;
    const int_ptr task = (int_ptr)(const int *)(a.sched + r);
    const int row = task[0], beg = task[1], end = task[2];
    const int_ptr idx = (int_ptr)a.idx;
    const float_ptr vals = (float_ptr)a.vals;
    const unsigned ldb = 4u * (unsigned)a.ld_in;
    const int s_own = 4 * lane;
    const bool live = s_own < a.B;
    const int s = live ? s_own : 0;
    const unsigned so = 4u * (unsigned)s;
    const __amdgpu_buffer_rsrc_t rin = make_rsrc(a.in, a.in_bytes);
    float *__restrict__ g_part = a.g_part[0];
    float xp[4] = {0.0f, 0.0f, 0.0f, 0.0f}; // lanes outside the batch add nothing to the gradient
    if (live) ldv<4>(a.aux + (size_t)row * a.ld_out + s, xp);
    double xd[4], acc[4] = {0.0, 0.0, 0.0, 0.0}, one_at[4];
#pragma unroll
    for (int v = 0; v < 4; ++v) {
        xd[v] = (double)xp[v];
        one_at[v] = (lane & 3) == v ? 1.0 : 0.0;
    }
    // sixteen entries: past the end of the row, zero weights at a column outside the operand
    auto fetch = [&](int g, i32x16 &c, f32x16 &w) {
        if (g + 16 <= end) {
#pragma unroll
            for (int k = 0; k < 16; ++k) { c[k] = idx[g + k]; w[k] = vals[g + k]; }
        } else {
#pragma unroll
            for (int k = 0; k < 16; ++k) {
                const int e = min(g + k, end - 1);
                const int ck = idx[e];
                const float wk = vals[e];
                c[k] = g + k < end ? ck : a.n_cols;
                w[k] = g + k < end ? wk : 0.0f;
            }
        }
    };
    float4 x0[4], x1[4];
    auto gather = [&](const i32x16 &c, int k, float4 (&x)[4]) {
#pragma unroll
        for (int u = 0; u < 4; ++u) x[u] = as_f4(__builtin_amdgcn_raw_buffer_load_b128(rin, (int)so, (int)((unsigned)c[k + u] * ldb), 0));
    };
    auto consume = [&](const float4 (&x)[4], const f32x16 &w, int k, double &sums) {
        double pr[4];
#pragma unroll
        for (int u = 0; u < 4; ++u) {
            const double wk = (double)w[k + u];
            const double d0 = (double)x[u].x, d1 = (double)x[u].y, d2 = (double)x[u].z, d3 = (double)x[u].w;
            acc[0] = fma(wk, d0, acc[0]);
            acc[1] = fma(wk, d1, acc[1]);
            acc[2] = fma(wk, d2, acc[2]);
            acc[3] = fma(wk, d3, acc[3]);
            pr[u] = fma(d3, xd[3], fma(d2, xd[2], fma(d1, xd[1], d0 * xd[0])));
        }
        asm volatile("" : "+v"(acc[0]), "+v"(acc[1]), "+v"(acc[2]), "+v"(acc[3])); // see k_bwd_rows
        sums = 0.0;
#pragma unroll
        for (int u = 0; u < 4; ++u) sums = __builtin_amdgcn_mfma_f64_4x4x4f64(pr[u], one_at[u], sums, 0, 0, 0);
    };
    i32x16 c, cn;
    f32x16 w, wn;
    if (beg < end) {
        fetch(beg, c, w);
        gather(c, 0, x0);
    }
    for (int g = beg; g < end; g += 16) {
        const bool more = g + 16 < end;
        if (more) fetch(g + 16, cn, wn);
        double part[4];
        gather(c, 4, x1);
        consume(x0, w, 0, part[0]);
        gather(c, 8, x0);
        consume(x1, w, 4, part[1]);
        gather(c, 12, x1);
        consume(x0, w, 8, part[2]);
        if (more) gather(cn, 0, x0);
        consume(x1, w, 12, part[3]);
        double sum = 0.0;
#pragma unroll
        for (int q = 0; q < 4; ++q) sum = __builtin_amdgcn_mfma_f64_4x4x4f64(one_at[q], part[q], sum, 0, 0, 0);
        sum += row_rotate<8>(sum);
        sum += row_rotate<4>(sum);
        const int e = g + 4 * (lane >> 4) + (lane & 3);
        if (__ballot(!(fabs(sum) < HUGE_VAL)) == 0) {
            if ((lane & 12) == 0 && e < end) g_part[e] = (float)sum;
        } else { // an infinity or NaN is in all the sums: one by one
            for (int k = g; k < min(g + 16, end); ++k) {
                const float4 x = as_f4(__builtin_amdgcn_raw_buffer_load_b128(rin, (int)so, (int)((unsigned)idx[k] * ldb), 0));
                double pr[4] = {fma((double)x.w, xd[3], fma((double)x.z, xd[2], fma((double)x.y, xd[1], (double)x.x * xd[0]))), 0.0, 0.0, 0.0};
                reduce4<64>(pr, lane);
                if (lane == 0) g_part[k] = (float)pr[0];
            }
        }
        c = cn;
        w = wn;
    }
    if (!a.store_out || !live) return;
    float o[4];
#pragma unroll
    for (int v = 0; v < 4; ++v) o[v] = act_backprop(a.act, acc[v], xp[v], a.cap);
    if (s + 4 > a.B) { // the batch's last group
#pragma unroll
        for (int v = 1; v < 4; ++v)
            if (s + v >= a.B) o[v] = 0.0f;
    }
    stv<4>(a.out + (size_t)row * a.ld_out + s, o);
}

// ---------------------------------------------------------------------------
// K1p / K2p: the same product for wide layers with short rows, swept in column panels.
//
// A 64-sample tile of a wide layer's operand (n_cols x 256 B) is several times the 4 MiB L2 of an
// XCD, and a row's 32 or so gathers land all over it, so without further care most gathers miss
// L2.  Here a wavefront owns R rows and keeps their entries (entry k of a row in lane k) and their
// R accumulators in registers; it walks the operand in panels of panel_cols rows, and in each
// panel every one of its rows consumes the entries whose column falls into the panel.  Column
// indices ascend inside a row, so each row still adds its terms in storage order: the sums are the
// same as in k_spmm.  The wavefronts resident on an XCD advance through the panels at about the
// same pace (nothing enforces it: a wavefront that runs ahead or behind only loses L2 hits), so
// an XCD's L2 holds one panel at a time and pulls each operand row in once per launch.
// Rows must have at most 64 entries (checked by the host); one sample per lane.
// ---------------------------------------------------------------------------
#define PANEL_MIN_SAMPLES 40 // AUTO: narrower batches gather with several rows per wavefront (k_rows)
#define PANEL_SLOTS 8 // gathers of one row segment that are in flight together; longer segments go round again

// Requests the operand rows of entries k .. min(k + PANEL_SLOTS, ke) - 1 of a row (wave-uniform branches).
__device__ __forceinline__ void panel_issue(__amdgpu_buffer_rsrc_t rin, unsigned so, unsigned ldb, int c_l, int k, int ke,
                                            float (&x)[PANEL_SLOTS])
{
#define PANEL_G(j) x[j] = __uint_as_float(__builtin_amdgcn_raw_buffer_load_b32(rin, (int)so, (int)((unsigned)__builtin_amdgcn_readlane(c_l, k + j) * ldb), 0))
    const int n = ke - k;
    if (n > 0) { PANEL_G(0);
    if (n > 1) { PANEL_G(1);
    if (n > 2) { PANEL_G(2);
    if (n > 3) { PANEL_G(3);
    if (n > 4) { PANEL_G(4);
    if (n > 5) { PANEL_G(5);
    if (n > 6) { PANEL_G(6);
    if (n > 7) { PANEL_G(7); } } } } } } } }
#undef PANEL_G
}

// Adds the terms of the same entries, in storage order.
__device__ __forceinline__ void panel_consume(float w_l, int k, int ke, const float (&x)[PANEL_SLOTS], double &acc)
{
#define PANEL_F(j) acc = fma((double)__int_as_float(__builtin_amdgcn_readlane(__float_as_int(w_l), k + j)), (double)x[j], acc)
    const int n = ke - k;
    if (n > 0) { PANEL_F(0);
    if (n > 1) { PANEL_F(1);
    if (n > 2) { PANEL_F(2);
    if (n > 3) { PANEL_F(3);
    if (n > 4) { PANEL_F(4);
    if (n > 5) { PANEL_F(5);
    if (n > 6) { PANEL_F(6);
    if (n > 7) { PANEL_F(7); } } } } } } } }
#undef PANEL_F
}

template <int R, int MODE, int ACT>
__global__ void __launch_bounds__(BLOCK_THREADS) k_spmm_panel(const SpmmArgs a, int n_cols, int panel_cols)
{
    const int lane = threadIdx.x & 63;
    const unsigned wave = threadIdx.x >> 6;
    const int B = a.B;
    const size_t ld = (size_t)a.ld_out;
    const unsigned ldb = 4u * (unsigned)a.ld_in;
    const __amdgpu_buffer_rsrc_t rin = make_rsrc(a.in, a.in_bytes);
    for (unsigned vb = blockIdx.x; vb < a.n_vblocks; vb += gridDim.x) {
        unsigned tile, rg;
        map_block(vb, a.n_tiles, a.n_rg, tile, rg); // n_rg counts groups of WAVES_PER_BLOCK * R rows here
        const int r0 = __builtin_amdgcn_readfirstlane((int)((rg * WAVES_PER_BLOCK + wave) * R));
        if (r0 >= a.n_rows) continue;
        const int s_own = (int)(tile + a.tile_base) * 64 + lane;
        const bool live = s_own < B;
        const int s = live ? s_own : 0;
        const unsigned so = 4u * (unsigned)s;

        int row[R], c_l[R], kcur[R];
        float w_l[R], xp[R];
        double acc[R];
#pragma unroll
        for (int r = 0; r < R; ++r) {
            row[r] = -1;
            c_l[r] = 0x7fffffff; // past every panel: lanes beyond the end of a row, and rows beyond the last
            w_l[r] = 0.0f;
            xp[r] = 0.0f;
            acc[r] = 0.0;
            kcur[r] = 0;
            if (r0 + r < a.n_rows) {
                const int4 t = a.sched[r0 + r];
                row[r] = t.x;
                if (t.y + lane < t.z) {
                    c_l[r] = a.idx[t.y + lane];
                    w_l[r] = MODE == 1 ? a.vals[a.perm[t.y + lane]] : a.vals[t.y + lane];
                }
                if (MODE == 1) xp[r] = a.aux[(size_t)t.x * ld + s];
            }
        }
        for (int pe = panel_cols;; pe += panel_cols) {
            const bool last = pe >= n_cols;
            const int bound = last ? 0x7fffffff : pe;
#pragma unroll
            for (int r = 0; r < R; r += 2) {
                // columns ascend inside a row: the entries below the bound are a prefix of the lanes
                const int ke0 = (int)__popcll(__ballot(c_l[r] < bound));
                int k0 = kcur[r];
                kcur[r] = ke0;
                float x0[PANEL_SLOTS];
                panel_issue(rin, so, ldb, c_l[r], k0, ke0, x0);
                if constexpr (R > 1) {
                    const int ke1 = (int)__popcll(__ballot(c_l[r + 1] < bound));
                    int k1 = kcur[r + 1];
                    kcur[r + 1] = ke1;
                    float x1[PANEL_SLOTS];
                    panel_issue(rin, so, ldb, c_l[r + 1], k1, ke1, x1);
                    panel_consume(w_l[r], k0, ke0, x0, acc[r]);
                    panel_consume(w_l[r + 1], k1, ke1, x1, acc[r + 1]);
                    for (k1 += PANEL_SLOTS; k1 < ke1; k1 += PANEL_SLOTS) {
                        panel_issue(rin, so, ldb, c_l[r + 1], k1, ke1, x1);
                        panel_consume(w_l[r + 1], k1, ke1, x1, acc[r + 1]);
                    }
                } else {
                    panel_consume(w_l[r], k0, ke0, x0, acc[r]);
                }
                for (k0 += PANEL_SLOTS; k0 < ke0; k0 += PANEL_SLOTS) {
                    panel_issue(rin, so, ldb, c_l[r], k0, ke0, x0);
                    panel_consume(w_l[r], k0, ke0, x0, acc[r]);
                }
            }
            if (last) break;
        }
#pragma unroll
        for (int r = 0; r < R; ++r) {
            if (row[r] < 0) continue;
            float o;
            if (MODE == 0) o = act_apply(ACT, acc[r] + (a.aux ? (double)a.aux[row[r]] : 0.0), a.cap);
            else o = act_backprop(a.act, acc[r], xp[r], a.cap);
            if (live) a.out[(size_t)row[r] * ld + s] = o;
        }
        if (fills_up(B, a.ld_out) && is_fill(s_own, B)) {
#pragma unroll
            for (int r = 0; r < R; ++r)
                if (row[r] >= 0) a.out[(size_t)row[r] * ld + s_own] = 0.0f;
        }
    }
}

// ---------------------------------------------------------------------------
// K1f: the whole feed-forward sweep (Eq. 3 for l = 1..L) in one launch, for nets whose widest layer
// fits in LDS.  The batch vectors are independent (they are the columns of X, Section 5.1), so a
// workgroup of 16 wavefronts takes T of them (1, 2 or 4) through all layers by itself, their
// activations in one LDS buffer of [position][T] floats, and only W is streamed, from a lane-major copy.
//
// Copy of W: the rows of a layer, longest first, in blocks of 64 that are dealt to the wavefronts; lane r of
// a wavefront walks row r of the block.  A block's entries come in chunks of sixteen per lane (past the end of a row:
// zero weights at a position of their own that always holds zeros), each as two halves of 3 KiB: the 64 lanes' eight 16-bit positions
// (16 bytes a lane), then two times four weights (16 bytes a lane): 6 bytes per entry in coalesced 16-byte
// loads.  The chunks of one wavefront follow each other through all its blocks and all layers; the half after
// next, of whatever block or layer, is requested as soon as the registers of the current one are free, so nothing
// waits at the head of a row or of a layer.
// Activations: row (block j of wavefront w, lane r) of a layer sits at position 64 (16 j + w) + r; the columns of
// the next layer are stored as those positions.  Every lane adds its row's terms in storage order in fp64 (the
// same sums as k_spmm).  A layer's results wait in registers until every wavefront has read its operands, and
// then replace them: one buffer instead of two, i.e. twice the samples or twice the width per CU.  Where four samples fit twice (up to
// 4096 positions) every other layer has its operand max_pos positions higher (the copy's positions say so): results are stored as they
// come, and one barrier ends a layer (us per pass of 120 layers, one buffer / two: 1024 neurons, 64 samples 306 / 295; 2001, 100 samples
// 493 / 480; 4096, 200 samples 880 / 866, 1024 samples 1633 / 1600; 3001 with 777 samples of which some die 799 / 781).
//
// What bounds it, in clocks of a CU per wavefront-wide entry (T = 1 / 2 / 4): vector instructions 4 / 6.5 / 10.5 (one
// address, one weight conversion, T conversions and T multiply-adds), LDS reads at random positions 7 / 7 / 13 (measured
// with reads alone; conflict-free 2.5 / 3 / 4.6, but making them so gained only 2 to 5 %), the stream of W 6 at the L1's
// 64 bytes per clock.  Measured 8.1 / 9 / 14.  Against the earlier version (two LDS buffers, four samples, 8-byte entries
// requested block by block, up to 4096 neurons): 4096 neurons, 1024 samples, 120 layers 2.28 -> 1.69 ms; and against a
// launch per layer: 16384 neurons, 4096 samples, 48 layers 40.6 -> 14.0 ms; 1024 neurons, 64 samples, 120 layers 561 ->
// 305 us; 8192 neurons with 820 entries per row, 2048 samples, 6 layers 11.6 -> 7.7 ms.
// ---------------------------------------------------------------------------
#define LDS_WAVES 16            // wavefronts per workgroup: one workgroup per CU
#define LDS_CHUNK 16            // entries per lane and chunk, in two halves of eight
#define LDS_HALF_BYTES 3072     // a half: 64 lanes x (eight positions, weights 0..3, weights 4..7), 16 bytes each
#define LDS_CHUNK_BYTES (2 * LDS_HALF_BYTES)
#define LDS_MAX_FLOATS 32768    // positions x samples a workgroup holds: 128 KiB, and 32 result registers per lane
struct LmLayer {                // one layer as k_fwd_lds walks it
    int32_t nb;                 // blocks per wavefront
    int32_t cs;                 // its chunk table: wavefront w's blocks start at lm_cs[cs + w (nb + 1) + j]
    int32_t pos;                // its first position in the row and bias tables
    int32_t n_pos;              // positions: 1024 nb
};
typedef float f32x32 __attribute__((ext_vector_type(32)));

// Ends a phase in which the wavefronts of the workgroup exchange data through LDS only: waits for the LDS accesses, not
// for the requested chunks of W.
__device__ __forceinline__ void lds_barrier()
{
    asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory");
}

// The hardware serves the oldest wavefront of a SIMD first, so that of four with equal work the youngest is done a third later,
// and everyone waits for it at the next barrier.  With a priority that goes round, block by block, they end closer together
// (16384 neurons, 256 samples 35.4 -> 33.6 us per layer; 4096 neurons, 1024 samples 14.6 -> 14.1; 8192 neurons with 820 entries
// per row, 1024 samples 640 -> 617).  In which layers: lm_turns.  A launch through the whole net: up to two rounds of workgroups only.
// In later ones the workgroups of an XCD are further apart in the stream of W that they share, and the turns made that worse (16384
// neurons, 4096 samples, eight rounds, 48 layers 13.8 -> 14.4 ms; four rounds 6.85 -> 6.97; two rounds 605 -> 587 us per 8 layers).
// The stretches of a pass that drops dead samples are launches of their own, at whose starts the workgroups are together again: turns
// in any number of rounds (us per pass of 48 layers without turns / in up to two rounds / in all: 16384 neurons, 4096 samples, eight
// rounds at first 6873 / 6750 / 6600; 2048 samples, four rounds 3364 / 3335 / 3321; 9973 neurons, 3000 samples 3245 / 3151 / 3125).
__device__ __forceinline__ void take_turns(int turn)
{
    switch (turn & 3) {
    case 0: __builtin_amdgcn_s_setprio(0); break;
    case 1: __builtin_amdgcn_s_setprio(1); break;
    case 2: __builtin_amdgcn_s_setprio(2); break;
    default: __builtin_amdgcn_s_setprio(3);
    }
}

// Byte address of a position in the activation buffer: (low or high half of `pair`) << shift, in one instruction.
template <int HI> __device__ __forceinline__ unsigned lds_address(unsigned pair, unsigned shift)
{
    unsigned a;
    if constexpr (HI)
        asm("v_lshlrev_b32_sdwa %0, %1, %2 dst_sel:DWORD dst_unused:UNUSED_PAD src0_sel:DWORD src1_sel:WORD_1" : "=v"(a) : "v"(shift), "v"(pair));
    else
        asm("v_lshlrev_b32_sdwa %0, %1, %2 dst_sel:DWORD dst_unused:UNUSED_PAD src0_sel:DWORD src1_sel:WORD_0" : "=v"(a) : "v"(shift), "v"(pair));
    return a;
}

template <int T> struct LdsPiece;
template <> struct LdsPiece<1> { typedef float type; };
template <> struct LdsPiece<2> { typedef float type __attribute__((ext_vector_type(2))); };
template <> struct LdsPiece<4> { typedef float type __attribute__((ext_vector_type(4))); };

#define LM_IN_ORDER 8          // a bit of sdnn_net::turns beside those of 1, 2 and 4 samples, see lm_turns

// What a launch takes through which layers.
struct LdsForward {
    const LmLayer *tab;
    const int32_t *lm_cs;
    const uint4 *lm;
    const float *lm_bias;
    const int32_t *lm_row;
    unsigned lm_bytes;
    int32_t l0, l1;        // layers l0 .. l1 - 1 (0-based)
    int32_t n_in;          // neurons of the input (l0 == 0: at positions of their own number)
    const float *in;       // [n_in][ld_in]
    float *out;            // [n_out(l1 - 1)][ld_out]
    int32_t ld_in, ld_out;
    int32_t B;             // samples
    int32_t vec_io;        // rows of in and out are whole T-float pieces
    int32_t turns;         // whether the wavefronts take turns, see take_turns (k_fwd_lds_part: with how many samples, lm_turns)
    float cap;
    // parts of a pass that drops dead samples (k_fwd_lds_part)
    const int32_t *n_live; // samples that are left; workgroups past them end at once
    const int32_t *src_col; // the column of `in` that holds sample k of them
    const int32_t *dst_col; // the column of `out` that sample k goes to (NULL: k)
    int32_t *alive;        // alive[k] = whether sample k has a non-zero activation at the end (NULL: not wanted)
    int32_t max_pos;       // positions of the LDS buffer
    int32_t two;           // max_pos, where odd layers (l0 and so on: 0-based) have their operand in a second buffer behind the first, else 0
};                         // one more position follows, which holds zeros

// PART: a stretch of layers for the samples that are still alive.  ORDER: a wavefront requests its halves of W strictly one after the
// other (see take, below).
// TWO (!PART): a.two != 0; looked at in every block it costs the nets that have one buffer up to 1 %.
template <int T, int ACT, bool PART, bool ORDER, bool TWO>
__device__ __forceinline__ void lds_forward(const LdsForward &a, int grp, int n_samples)
{
    const int second = PART || TWO ? a.two : 0; // where the second buffer starts
    extern __shared__ __attribute__((aligned(16))) float lds_act[];
    typedef typename LdsPiece<T>::type piece; // the T samples of one position: one LDS access
    typedef __attribute__((address_space(3))) piece *lds_ptr;
    typedef __attribute__((address_space(3))) char *lds_bytes;
    const lds_ptr act = (lds_ptr)(__attribute__((address_space(3))) float *)lds_act; // the kernel's only LDS: at address 0
    unsigned shift = T == 1 ? 2 : T == 2 ? 3 : 4;
    asm("" : "+v"(shift)); // kept in a register for lds_address
    typedef const LmLayer __attribute__((address_space(4))) *tab_ptr;
    typedef const int32_t __attribute__((address_space(4))) *cs_ptr;
    const tab_ptr stab = (tab_ptr)a.tab;
    const cs_ptr scs = (cs_ptr)a.lm_cs;
    const float *__restrict__ lm_bias = a.lm_bias;
    const int32_t *__restrict__ lm_row = a.lm_row;

    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int s0 = grp * T;
    const bool full = s0 + T <= n_samples && a.vec_io; // all T samples exist and T-float pieces of a row of X are aligned
    int src[T]; // PART: the samples' columns
    if constexpr (PART) {
#pragma unroll
        for (int t = 0; t < T; ++t) src[t] = a.src_col[min(s0 + t, n_samples - 1)];
    }

    // the input at its positions (l0 == 0: a neuron's own number; else where the layer below would have put it), zeros
    // past the end of the batch
    const int n_fill = PART && a.l0 > 0 ? stab[a.l0 - 1].n_pos : a.n_in;
    for (int i = tid; i < n_fill; i += 64 * LDS_WAVES) {
        const int row = PART && a.l0 > 0 ? lm_row[stab[a.l0 - 1].pos + i] : i;
        const float *p = a.in + (size_t)max(row, 0) * a.ld_in;
        piece v;
        if constexpr (PART) {
            if constexpr (T == 1) v = p[src[0]];
            else {
#pragma unroll
                for (int t = 0; t < T; ++t) v[t] = p[src[t]];
            }
        } else if (full) {
            v = *reinterpret_cast<const piece *>(p + s0);
        } else if constexpr (T == 1) {
            v = s0 < n_samples ? p[s0] : 0.0f;
        } else {
#pragma unroll
            for (int t = 0; t < T; ++t) v[t] = s0 + t < n_samples ? p[s0 + t] : 0.0f;
        }
        act[(PART && (a.l0 & 1) ? second : 0) + i] = v;
    }
    if (tid < T) lds_act[T * (a.max_pos + second) + tid] = 0.0f; // where the slots past the end of a row point

    // the wavefront's place in the copy of W, in bytes (the copy is smaller than 4 GiB), goes into the loads as a scalar
    const __amdgpu_buffer_rsrc_t rlm = make_rsrc((const float *)a.lm, a.lm_bytes);
    unsigned at = (unsigned)scs[stab[a.l0].cs + wave * (stab[a.l0].nb + 1)] * LDS_CHUNK_BYTES;
    const int lane16 = 16 * lane;
    struct Half { u32x4 c, wa, wb; } ha, hb;
    auto request = [&](Half &h) {
        h.c = __builtin_amdgcn_raw_buffer_load_b128(rlm, lane16, (int)at, 0);
        h.wa = __builtin_amdgcn_raw_buffer_load_b128(rlm, lane16 + 1024, (int)at, 0);
        h.wb = __builtin_amdgcn_raw_buffer_load_b128(rlm, lane16 + 2048, (int)at, 0);
        at += LDS_HALF_BYTES;
    };
    request(ha);
    request(hb);
    // All the workgroups of an XCD stream through the same copy of W at about the same time, and whoever comes first to a
    // line waits for memory.  So they share that out: before a layer's last block each wavefront touches one line in so many
    // of the next layer's stream (3001 neurons, 120 layers, copies of W that come from HBM: 1.08 -> 0.92 ms).
    const bool turns = PART ? (a.turns & T) != 0 : a.turns != 0;
    const unsigned xcd_wg = (blockIdx.x >> 3) % max(1u, min(32u, gridDim.x >> 3));
    unsigned touched = 0;
    lds_barrier();

    for (int l = a.l0; l < a.l1; ++l) {
        const int nb = stab[l].nb, cs0 = stab[l].cs + wave * (nb + 1), pos0 = stab[l].pos + 64 * wave + lane;
        f32x32 res;
        auto result = [&](int j) {
            piece v;
            if constexpr (T == 1) v = res[j];
            else {
#pragma unroll
                for (int t = 0; t < T; ++t) v[t] = res[j * T + t];
            }
            return v;
        };
        for (int j = 0; j < nb; ++j) {
            if (j > 0 && j == nb - 1 && l + 1 < a.l1) { // see above (one block per layer: it would only hold the wavefront up)
                asm volatile("" ::"v"(touched));
                const int c0 = scs[stab[l + 1].cs + wave * (stab[l + 1].nb + 1)], c1 = scs[stab[l + 1].cs + wave * (stab[l + 1].nb + 1) + stab[l + 1].nb];
                const unsigned line = (unsigned)c0 * LDS_CHUNK_BYTES + 128u * (64u * xcd_wg + (unsigned)lane);
                if (line < (unsigned)c1 * LDS_CHUNK_BYTES) touched = __builtin_amdgcn_raw_buffer_load_b32(rlm, (int)line, 0, 0);
            }
            const int n = scs[cs0 + j + 1] - scs[cs0 + j];
            const float bias = lm_bias[pos0 + 1024 * j];
            double acc[T];
#pragma unroll
            for (int t = 0; t < T; ++t) acc[t] = 0.0;
            auto take = [&](Half &h) { // eight entries; then their registers are free for the half after next
                unsigned ad[8];
                double w[8];
                piece x[8];
#pragma unroll
                for (int u = 0; u < 4; ++u) {
                    ad[2 * u] = lds_address<0>(h.c[u], shift);
                    ad[2 * u + 1] = lds_address<1>(h.c[u], shift);
                }
#pragma unroll
                for (int u = 0; u < 8; ++u) x[u] = *(lds_ptr)((lds_bytes)0 + ad[u]);
#pragma unroll
                for (int u = 0; u < 4; ++u) {
                    w[u] = (double)__uint_as_float(h.wa[u]);
                    w[u + 4] = (double)__uint_as_float(h.wb[u]);
                }
                request(h);
#pragma unroll
                for (int u = 0; u < 8; ++u)
#pragma unroll
                    for (int t = 0; t < T; ++t) {
                        float xv;
                        if constexpr (T == 1) xv = x[u];
                        else xv = x[u][t];
                        acc[t] = fma(w[u], (double)xv, acc[t]);
                    }
            };
            if (turns) take_turns(wave / 4 + j);
            for (int i = 0; i < n; ++i) { // (ORDER: nothing moves across; else the loads are requested with those of the other half)
                take(ha);
                if constexpr (ORDER) __builtin_amdgcn_sched_barrier(0);
                take(hb);
                if constexpr (ORDER) __builtin_amdgcn_sched_barrier(0);
            }
            const double bd = (double)bias;
#pragma unroll
            for (int t = 0; t < T; ++t) res[j * T + t] = act_apply(ACT, acc[t] + bd, a.cap);
            if (second && l < a.l1 - 1) act[(l & 1 ? 0 : second) + 64 * (LDS_WAVES * j + wave) + lane] = result(j);
        }
        if (l == a.l1 - 1) {
            unsigned nz = 0; // bit t: this lane has a non-zero result for sample t
            for (int j = 0; j < nb; ++j) {
                const int row = lm_row[pos0 + 1024 * j];
                if (row < 0) continue;
                float *dst = a.out + (size_t)row * a.ld_out;
                const piece v = result(j);
                if constexpr (PART) {
#pragma unroll
                    for (int t = 0; t < T; ++t) {
                        float x;
                        if constexpr (T == 1) x = v;
                        else x = v[t];
                        if (s0 + t < n_samples) dst[a.dst_col ? a.dst_col[s0 + t] : s0 + t] = x;
                        nz |= x != 0.0f ? 1u << t : 0u;
                    }
                } else if (full) {
                    *reinterpret_cast<piece *>(dst + s0) = v;
                } else if constexpr (T == 1) {
                    if (s0 < n_samples) dst[s0] = v;
                } else {
#pragma unroll
                    for (int t = 0; t < T; ++t)
                        if (s0 + t < n_samples) dst[s0 + t] = v[t];
                }
            }
            if constexpr (PART) {
                if (a.alive) { // the buffer is free: every wavefront leaves a word in it
                    lds_barrier();
                    __attribute__((address_space(3))) unsigned *word = (__attribute__((address_space(3))) unsigned *)(__attribute__((address_space(3))) float *)lds_act;
#pragma unroll
                    for (int t = 0; t < T; ++t) {
                        const bool any = __ballot((nz >> t) & 1u) != 0;
                        if (lane == 0) word[wave * T + t] = any ? 1u : 0u;
                    }
                    lds_barrier();
                    if (tid < T && s0 + tid < n_samples) {
                        unsigned any = 0;
                        for (int w = 0; w < LDS_WAVES; ++w) any |= word[w * T + tid];
                        a.alive[s0 + tid] = (int)any;
                    }
                }
            }
            return;
        }
        if (!second) {
            lds_barrier(); // every wavefront has read its operands
            for (int j = 0; j < nb; ++j) act[64 * (LDS_WAVES * j + wave) + lane] = result(j);
        }
        lds_barrier(); // the layer is complete before anyone reads it
    }
}

template <int T, int ACT, bool ORDER, bool TWO>
__global__ void __launch_bounds__(64 * LDS_WAVES) k_fwd_lds(const LdsForward a)
{
    // neighbouring samples share cache lines of X: an XCD takes a contiguous stretch of them
    const int nwg = (int)gridDim.x, per = nwg >> 3, wg = (int)blockIdx.x;
    lds_forward<T, ACT, false, ORDER, TWO>(a, wg < 8 * per ? (wg & 7) * per + (wg >> 3) : wg, a.B);
}

// A stretch of layers for the samples that are still alive, as many per workgroup as it takes to give every CU one (the
// fewer, the sooner a layer is done).
__global__ void __launch_bounds__(64 * LDS_WAVES) k_fwd_lds_part(const LdsForward a, int n_cu)
{
    const int n = *a.n_live, wg = (int)blockIdx.x;
    if (4 * a.max_pos <= LDS_MAX_FLOATS && n > 2 * n_cu) {
        if (4 * wg < n) lds_forward<4, ACT_RELU_CAP, true, true, true>(a, wg, n);
    } else if (2 * a.max_pos <= LDS_MAX_FLOATS && n > n_cu) {
        if (2 * wg < n) lds_forward<2, ACT_RELU_CAP, true, true, true>(a, wg, n);
    } else {
        if (wg >= n) return;
        if (a.turns & LM_IN_ORDER) lds_forward<1, ACT_RELU_CAP, true, true, true>(a, wg, n);
        else lds_forward<1, ACT_RELU_CAP, true, false, true>(a, wg, n);
    }
}

// After a stretch: the samples that are left, in order (src_col: their columns in the stretch's output, sample: their numbers
// in the caller's block).  One workgroup; alive == NULL: all of the B samples, the start of a pass.
__global__ void __launch_bounds__(1024) k_live_columns(const int32_t *__restrict__ alive, const int32_t *__restrict__ n_in,
                                                       const int32_t *__restrict__ sample_in, int B, int32_t *__restrict__ n_out,
                                                       int32_t *__restrict__ src_col, int32_t *__restrict__ sample)
{
    __shared__ int wave_sum[16];
    const int t = threadIdx.x, lane = t & 63, wave = t >> 6;
    const int n = alive ? *n_in : B;
    int base = 0;
    for (int c0 = 0; c0 < n; c0 += 1024) {
        const int c = c0 + t;
        const bool on = c < n && (!alive || alive[c] != 0);
        const unsigned long long m = __ballot(on);
        if (lane == 0) wave_sum[wave] = (int)__popcll(m);
        __syncthreads();
        int before = base, all = 0;
        for (int w = 0; w < 16; ++w) {
            if (w < wave) before += wave_sum[w];
            all += wave_sum[w];
        }
        if (on) {
            const int k = before + (int)__popcll(m & ((1ull << lane) - 1ull));
            src_col[k] = c;
            sample[k] = alive ? sample_in[c] : c;
        }
        base += all;
        __syncthreads();
    }
    if (t == 0) *n_out = base;
}

// Writes a layer's part of the lane-major copy from its CSR arrays: biases and weights, and with prev_pos (the position of
// every neuron of the layer below, NULL for the first layer: its own index) also the positions (prev_pos is looked at only
// if with_cols).  grid = (blocks per wavefront, 16 wavefronts, parts): a workgroup of one wavefront takes every parts-th half
// chunk of a block of 64 rows (all of them one after the other: sdnn_set_weights on 8192 rows of up to 2048 entries 199 us, in
// parts 57).
__global__ void __launch_bounds__(64) k_lm_fill(const LayerDev *__restrict__ layer, const LmLayer *__restrict__ tab,
                                                const int32_t *__restrict__ lm_cs, uint4 *__restrict__ lm,
                                                float *__restrict__ lm_bias, const int32_t *__restrict__ lm_row,
                                                const int32_t *__restrict__ prev_pos, int with_cols, int pad_pos, int first_pos)
{
    const LayerDev &L = *layer;
    const int j = blockIdx.x, w = blockIdx.y, lane = threadIdx.x, nb = tab->nb;
    const int at = tab->pos + 64 * (LDS_WAVES * j + w) + lane;
    const int row = lm_row[at];
    const int c0 = lm_cs[tab->cs + w * (nb + 1) + j], c1 = lm_cs[tab->cs + w * (nb + 1) + j + 1];
    int beg = 0, end = 0;
    float bias = 0.0f;
    if (row >= 0) {
        beg = L.row_ptr[row];
        end = L.row_ptr[row + 1];
        bias = L.bias[row];
    }
    if (blockIdx.z == 0) lm_bias[at] = bias;
    for (int hf = blockIdx.z; hf < 2 * (c1 - c0); hf += gridDim.z) {
        uint4 *o = lm + ((size_t)c0 * LDS_CHUNK_BYTES + (size_t)hf * LDS_HALF_BYTES) / 16 + lane;
        unsigned pk[4], wt[8];
#pragma unroll
        for (int k = 0; k < 8; ++k) {
            const int e = beg + hf * 8 + k;
            unsigned pos = (unsigned)pad_pos; // zeros in k_fwd_lds, past the end of the operand in k_spmv_lm
            wt[k] = 0;
            if (e < end) {
                wt[k] = __float_as_uint(L.vals[e]);
                if (with_cols) pos = (unsigned)(first_pos + (prev_pos ? prev_pos[L.col_idx[e]] : L.col_idx[e]));
            }
            if (k & 1) pk[k >> 1] |= pos << 16;
            else pk[k >> 1] = pos;
        }
        if (with_cols) o[0] = make_uint4(pk[0], pk[1], pk[2], pk[3]);
        o[64] = make_uint4(wt[0], wt[1], wt[2], wt[3]);
        o[128] = make_uint4(wt[4], wt[5], wt[6], wt[7]);
    }
}

// ---------------------------------------------------------------------------
// K1t / K2t: training on nets so narrow that a launch per layer is bound by its chain of dependent loads: the whole forward pass
// (MODE 0, Eq. 3 for l = 1..L) or the whole back-propagation (MODE 1, Eq. 7 for l = L..2) in one launch.  A workgroup of
// 16 wavefronts takes one sample through all layers as k_fwd_lds<1> does, over lane-major copies of W and of W^T that follow the
// stepped values (k_train_fill); the gradient is formed by k_update as before.  The activations of up to 2048 neurons lie in LDS
// twice, so a layer's results replace nothing that is still read and one barrier ends a layer (the positions of every other step
// are stored 2048 higher).  Both passes keep a layer's neurons in the same order, that of the rows of W_{l+1}^T by length, so that
// a sample's X_l and Delta_l are stored and read back in whole lines [step][sample][position]; k_train_turn then brings them to where
// the other kernels expect them.  (Stored there at once, four bytes a line, the passes took 3.5 and 4.6 us per layer.)  Every
// lane adds its row's terms in storage order: same bits as k_spmm.
//
// What bounds it: per layer of 1024 neurons of 32 entries 1.6 us of LDS reads (back 1.8), 1.35 us of the stream of W (1.75), 1.0 us of
// vector instructions (1.2) by their counters, and the chain between two barriers; 2.4 us forward, 3.0 back (columns of 16 to 50
// entries in chunks of sixteen), where a launch per layer takes 4.5 and 5.8.  The copies come
// from HBM, and a workgroup that waits for a line holds up everyone on its XCD: workgroups on the compute units that the samples
// leave idle read the copy through once as fast as they can, so that it comes from the memory-side cache (a step of 120 layers whose
// arrays are not on chip, 64 samples: 910 us, 300 more without them; 1406 with a launch per layer).
// ---------------------------------------------------------------------------
#define TRAIN_LDS_POS 2048 // neurons at most: two blocks per wavefront
struct TrainLds {
    const LayerDev *layers;
    const LmLayer *tab, *tab_x; // per step: layer 1.. (MODE 0), layer L.. down to 2 (MODE 1); and those of MODE 0
    const int32_t *cs;
    const uint4 *lm;
    const float *bias;          // MODE 0: by position
    float *out;                 // [step][max_batch][position]
    const float *x;             // MODE 1: what MODE 0 has stored there
    unsigned lm_bytes;
    int32_t n_steps, n_layers, max_batch, ld, B;
    float cap;
};
template <int MODE, int ACT>
__global__ void __launch_bounds__(64 * LDS_WAVES) k_train_lds(const TrainLds a)
{
    __shared__ float act[2 * TRAIN_LDS_POS + 1];
    typedef __attribute__((address_space(3))) float *lds_ptr;
    typedef __attribute__((address_space(3))) char *lds_bytes;
    const lds_bytes base = (lds_bytes)(lds_ptr)act;
    typedef const LmLayer __attribute__((address_space(4))) *tab_ptr;
    typedef const int32_t __attribute__((address_space(4))) *cs_ptr;
    const tab_ptr tab = (tab_ptr)a.tab, tab_x = (tab_ptr)a.tab_x;
    const cs_ptr cs = (cs_ptr)a.cs;
    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    if ((int)blockIdx.x >= a.B) { // on compute units that the samples leave idle: the copy of W into the memory-side cache at once
        const uint4 *p = a.lm;
        const size_t n = a.lm_bytes / 16, stride = (size_t)(gridDim.x - a.B) * blockDim.x;
        for (size_t i = (size_t)(blockIdx.x - a.B) * blockDim.x + tid; i < n; i += 8 * stride) {
            unsigned t[8];
#pragma unroll
            for (int u = 0; u < 8; ++u) t[u] = i + u * stride < n ? p[i + u * stride].x : 0u;
#pragma unroll
            for (int u = 0; u < 8; ++u) asm volatile("" ::"v"(t[u]));
        }
        return;
    }
    // neighbouring samples share cache lines of the input: an XCD takes a contiguous stretch of them
    const int nwg = a.B, per = nwg >> 3, wg = (int)blockIdx.x;
    const int s = wg < 8 * per ? (wg & 7) * per + (wg >> 3) : wg;
    unsigned shift = 2;
    asm("" : "+v"(shift)); // kept in a register for lds_address
    const __amdgpu_buffer_rsrc_t rlm = make_rsrc((const float *)a.lm, a.lm_bytes);
    unsigned at = (unsigned)cs[tab[0].cs + wave * (tab[0].nb + 1)] * LDS_CHUNK_BYTES;
    const int lane16 = 16 * lane;
    struct Half { u32x4 c, wa, wb; } ha, hb;
    auto request = [&](Half &h) {
        h.c = __builtin_amdgcn_raw_buffer_load_b128(rlm, lane16, (int)at, 0);
        h.wa = __builtin_amdgcn_raw_buffer_load_b128(rlm, lane16 + 1024, (int)at, 0);
        h.wb = __builtin_amdgcn_raw_buffer_load_b128(rlm, lane16 + 2048, (int)at, 0);
        at += LDS_HALF_BYTES;
    };
    request(ha);
    request(hb);
    {
        const LayerDev &L = a.layers[MODE == 0 ? 0 : a.n_layers - 1];
        const int n = MODE == 0 ? L.n_in : L.n_out;
        const float *in = MODE == 0 ? L.X_prev : L.D;
        for (int i = tid; i < n; i += 64 * LDS_WAVES) act[i] = in[(size_t)i * a.ld + s];
    }
    if (tid == 0) act[2 * TRAIN_LDS_POS] = 0.0f; // where the slots past the end of a row point
    __syncthreads();
    for (int k = 0; k < a.n_steps; ++k) {
        const int nb = tab[k].nb, cs0 = tab[k].cs + wave * (nb + 1), pos0 = 64 * wave + lane;
        // what this lane's results wait for: biases, or the X_l that the derivative is taken from (step a.n_layers - 2 - k of MODE 0)
        const float *aux = MODE == 0 ? a.bias + tab[k].pos : a.x + (size_t)tab_x[a.n_layers - 2 - k].pos * a.max_batch + (size_t)s * tab[k].n_pos;
        float *out = a.out + (size_t)tab[k].pos * a.max_batch + (size_t)s * tab[k].n_pos;
        float *next = act + ((k + 1) & 1) * TRAIN_LDS_POS;
        for (int j = 0; j < nb; ++j) {
            const float e = aux[pos0 + 1024 * j];
            double acc = 0.0;
            auto take = [&](Half &h) { // eight entries; then their registers are free for the half after next
                unsigned ad[8];
                double w[8];
                float x[8];
#pragma unroll
                for (int u = 0; u < 4; ++u) {
                    ad[2 * u] = lds_address<0>(h.c[u], shift);
                    ad[2 * u + 1] = lds_address<1>(h.c[u], shift);
                }
#pragma unroll
                for (int u = 0; u < 8; ++u) x[u] = *(lds_ptr)(base + ad[u]);
#pragma unroll
                for (int u = 0; u < 4; ++u) {
                    w[u] = (double)__uint_as_float(h.wa[u]);
                    w[u + 4] = (double)__uint_as_float(h.wb[u]);
                }
                request(h);
#pragma unroll
                for (int u = 0; u < 8; ++u) acc = fma(w[u], (double)x[u], acc);
            };
            for (int i = cs[cs0 + j + 1] - cs[cs0 + j]; i > 0; --i) {
                take(ha);
                __builtin_amdgcn_sched_barrier(0);
                take(hb);
                __builtin_amdgcn_sched_barrier(0);
            }
            const float r = MODE == 0 ? act_apply(ACT, acc + (double)e, a.cap) : act_backprop(ACT, acc, e, a.cap);
            next[pos0 + 1024 * j] = r;
            out[pos0 + 1024 * j] = r;
        }
        lds_barrier(); // the layer is complete before anyone reads it
    }
}

// From [step][max_batch][position] to X_l (MODE 0) or Delta_{l-1} (MODE 1), [neuron][ld]: tiles of 64 positions and 64 samples
// through LDS, zeros for the samples that fill up the batch.  grid = (tiles of positions, tiles of samples, steps).
template <int MODE>
__global__ void __launch_bounds__(256) k_train_turn(const LayerDev *__restrict__ layers, int n_layers, int step0, const LmLayer *__restrict__ tab,
                                                    const int32_t *__restrict__ rows, const float *__restrict__ from, int max_batch, int ld, int B, int Bp)
{
    __shared__ float tile[64][65];
    const int k = step0 + (int)blockIdx.z, tid = threadIdx.x, p0 = 64 * blockIdx.x, s0 = 64 * blockIdx.y;
    const LmLayer t = tab[k];
    if (p0 >= t.n_pos) return;
    float *out = MODE == 0 ? layers[k].X : layers[n_layers - 2 - k].D;
    const float *in = from + (size_t)t.pos * max_batch;
    for (int i = tid; i < 4096; i += 256) {
        const int p = i & 63, s = i >> 6;
        tile[s][p] = s0 + s < B ? in[(size_t)(s0 + s) * t.n_pos + p0 + p] : 0.0f;
    }
    __syncthreads();
    for (int i = tid; i < 4096; i += 256) {
        const int s = i & 63, p = i >> 6, row = rows[t.pos + p0 + p];
        if (row >= 0 && s0 + s < Bp) out[(size_t)row * ld + s0 + s] = tile[s][p];
    }
}

// Writes the weights of the steps' copies from the CSR values (COLS: and the positions of the operand), and the biases by position:
// steps step0 .. step0 + n_steps - 1, eight steps to a row of the grid, each on an XCD of its own (MODE 1 reads a layer's values in
// any order: by all XCDs 77 us for 120 layers of 1024 neurons).  grid = (8 max_nb wavefronts, eights of steps).  pos: the positions of every step's rows, step after step; first[k]: where
// step k's start.
template <int MODE, bool COLS>
__global__ void __launch_bounds__(256) k_train_fill(const LayerDev *__restrict__ layers, int n_layers, int step0, int n_steps, const LmLayer *__restrict__ tab,
                                                    const int32_t *__restrict__ cs, uint4 *__restrict__ lm, const int32_t *__restrict__ rows,
                                                    const int32_t *__restrict__ pos, const int32_t *__restrict__ first, float *__restrict__ bias)
{
    const int step = 8 * (int)blockIdx.y + (int)(blockIdx.x & 7u), k = step0 + step, w = (int)(blockIdx.x >> 3) & (LDS_WAVES - 1);
    const int j = (int)(blockIdx.x >> 3) / LDS_WAVES, lane = threadIdx.x & 63;
    if (step >= n_steps) return;
    const int nb = tab[k].nb;
    if (j >= nb) return;
    const LayerDev &L = layers[MODE == 0 ? k : n_layers - 1 - k];
    const int at = tab[k].pos + 64 * (LDS_WAVES * j + w) + lane, row = rows[at];
    const int c0 = cs[tab[k].cs + w * (nb + 1) + j], c1 = cs[tab[k].cs + w * (nb + 1) + j + 1];
    const int32_t *ptr = MODE == 0 ? L.row_ptr : L.t_row_ptr, *idx = MODE == 0 ? L.col_idx : L.t_row_idx;
    int beg = 0, end = 0;
    if (row >= 0) {
        beg = ptr[row];
        end = ptr[row + 1];
    }
    if (MODE == 0 && threadIdx.x < 64) bias[at] = row >= 0 ? L.bias[row] : 0.0f;
    for (int hf = threadIdx.x >> 6; hf < 2 * (c1 - c0); hf += 4) {
        uint4 *o = lm + ((size_t)c0 * LDS_CHUNK_BYTES + (size_t)hf * LDS_HALF_BYTES) / 16 + lane;
        unsigned pk[4], wt[8];
        int from[8]; // where the values are
        const int e0 = beg + hf * 8;
        if (MODE == 1 && e0 + 8 <= end) {
            const I4 a = *(const I4 *)(L.t_perm + e0), b = *(const I4 *)(L.t_perm + e0 + 4);
#pragma unroll
            for (int u = 0; u < 4; ++u) { from[u] = a.v[u]; from[u + 4] = b.v[u]; }
        } else {
#pragma unroll
            for (int u = 0; u < 8; ++u) from[u] = e0 + u >= end ? 0 : MODE == 0 ? e0 + u : L.t_perm[e0 + u];
        }
#pragma unroll
        for (int u = 0; u < 8; ++u) {
            const int e = e0 + u;
            unsigned p = 2 * TRAIN_LDS_POS;
            wt[u] = 0;
            if (e < end) {
                wt[u] = __float_as_uint(L.vals[from[u]]);
                if (COLS) p = (unsigned)((k & 1) * TRAIN_LDS_POS + (k > 0 ? pos[first[k - 1] + idx[e]] : idx[e]));
            }
            if (u & 1) pk[u >> 1] |= p << 16;
            else pk[u >> 1] = p;
        }
        if (COLS) o[0] = make_uint4(pk[0], pk[1], pk[2], pk[3]);
        o[64] = make_uint4(wt[0], wt[1], wt[2], wt[3]);
        o[128] = make_uint4(wt[4], wt[5], wt[6], wt[7]);
    }
}

// ---------------------------------------------------------------------------
// K1l: Eq. 3 for one layer of long rows in training: a workgroup of 16 wavefronts holds four samples of the whole operand in LDS and
// takes every n_ranges-th block of 64 rows, a lane per row, over a lane-major copy of W that follows the stepped values
// (k_long_fill).  The blocks, longest first, are handed to whichever wavefront is free.  Every lane adds its row's terms in storage
// order: same bits as k_spmm.
//
// What bounds it: per wavefront-wide entry LDS returns 1024 bytes at 128 a clock and the L1 384 bytes of W at 64 a clock, by the same way
// into the registers: 14 clocks of a CU, of which vector instructions take 10.  A gather through the L1 returns the same 1024 bytes in
// 16 clocks, and 24 where half of them miss L2 (an operand of 8 MB).  8192 neurons of 820 entries, 256 samples, us per layer: k_spmm
// 280, this 182, and k_long_fill 18.
// ---------------------------------------------------------------------------
#define LONG_MIN_BATCH 65 // see long_forward
#define LONG_POS 8192 // neurons of the operand at most: four samples in 128 KiB
struct FwdLong {
    const int32_t *cs;  // [blocks + 1]: first half of a block
    const int2 *row;    // [64 blocks]: {row, entries}, row -1 past the last
    const uint4 *lm;    // halves of LDS_HALF_BYTES, and two more: a wavefront requests two past its last
    const float *bias;
    const float *in;    // [n_in][ld]
    float *out;         // [n_out][ld]
    uint32_t lm_bytes;
    int32_t blocks, n_in, ld, B;
    int32_t groups, n_ranges; // groups of four samples
    float cap;
};
template <int ACT>
__global__ void __launch_bounds__(64 * LDS_WAVES) k_fwd_long(const FwdLong a)
{
    extern __shared__ __attribute__((aligned(16))) float lds_act[];
    typedef float piece __attribute__((ext_vector_type(4)));
    typedef __attribute__((address_space(3))) piece *lds_ptr;
    typedef __attribute__((address_space(3))) char *lds_bytes;
    const lds_ptr act = (lds_ptr)(__attribute__((address_space(3))) float *)lds_act; // the kernel's only LDS: at address 0
    int *next = (int *)(lds_act + 4 * (a.n_in + 1)); // the next block of this workgroup's that nobody has taken
    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    // An XCD takes a stretch of the samples, whose rows of X share cache lines, and all ranges of W side by side.
    const int per = (a.groups + 7) >> 3, k = (int)(blockIdx.x >> 3), q = k / per, g = (int)(blockIdx.x & 7u) * per + k % per;
    if (g >= a.groups) return;
    for (int i = tid; i < a.n_in; i += 64 * LDS_WAVES) act[i] = *(const piece *)(a.in + (size_t)i * a.ld + 4 * g);
    if (tid == 0) {
        act[a.n_in] = piece{0.0f, 0.0f, 0.0f, 0.0f}; // where the slots past the end of a row point
        *next = LDS_WAVES;
    }
    unsigned shift = 4;
    asm("" : "+v"(shift)); // kept in a register for lds_address
    const __amdgpu_buffer_rsrc_t rlm = make_rsrc((const float *)a.lm, a.lm_bytes);
    const int lane16 = 16 * lane;
    unsigned at = 0;
    struct Half { u32x4 c, wa, wb; } ha, hb;
    auto request = [&](Half &h) {
        h.c = __builtin_amdgcn_raw_buffer_load_b128(rlm, lane16, (int)at, 0);
        h.wa = __builtin_amdgcn_raw_buffer_load_b128(rlm, lane16 + 1024, (int)at, 0);
        h.wb = __builtin_amdgcn_raw_buffer_load_b128(rlm, lane16 + 2048, (int)at, 0);
        at += LDS_HALF_BYTES;
    };
    __syncthreads();
    for (int b = q + a.n_ranges * wave; b < a.blocks;) {
        const int c0 = a.cs[b];
        int n = a.cs[b + 1] - c0;
        const int row = a.row[64 * b + lane].x;
        at = (unsigned)c0 * LDS_HALF_BYTES;
        request(ha);
        request(hb);
        const double bias = a.bias && row >= 0 ? (double)a.bias[row] : 0.0;
        double acc[4] = {0.0, 0.0, 0.0, 0.0};
        auto take = [&](Half &h) { // eight entries; then their registers are free for the half after next
            unsigned ad[8];
            double w[8];
            piece x[8];
#pragma unroll
            for (int u = 0; u < 4; ++u) {
                ad[2 * u] = lds_address<0>(h.c[u], shift);
                ad[2 * u + 1] = lds_address<1>(h.c[u], shift);
            }
#pragma unroll
            for (int u = 0; u < 8; ++u) x[u] = *(lds_ptr)((lds_bytes)0 + ad[u]);
#pragma unroll
            for (int u = 0; u < 4; ++u) {
                w[u] = (double)__uint_as_float(h.wa[u]);
                w[u + 4] = (double)__uint_as_float(h.wb[u]);
            }
            request(h);
#pragma unroll
            for (int u = 0; u < 8; ++u)
#pragma unroll
                for (int t = 0; t < 4; ++t) acc[t] = fma(w[u], (double)x[u][t], acc[t]);
        };
        while (n > 0) {
            take(ha);
            __builtin_amdgcn_sched_barrier(0);
            if (--n == 0) break;
            take(hb);
            __builtin_amdgcn_sched_barrier(0);
            --n;
        }
        piece o;
#pragma unroll
        for (int t = 0; t < 4; ++t) o[t] = 4 * g + t < a.B ? act_apply(ACT, acc[t] + bias, a.cap) : 0.0f;
        if (row >= 0) *(piece *)(a.out + (size_t)row * a.ld + 4 * g) = o;
        int take_next = 0;
        if (lane == 0) take_next = __hip_atomic_fetch_add(next, 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
        b = q + a.n_ranges * __builtin_amdgcn_readfirstlane(take_next);
    }
}

// Writes the weights of those copies from the CSR values (COLS: and the columns).  grid = (blocks, parts, layers): a workgroup's
// wavefronts take neighbouring halves, so that a line of the values is read once.
template <bool COLS>
__global__ void __launch_bounds__(256) k_long_fill(const LayerDev *__restrict__ layers)
{
    const LayerDev &L = layers[blockIdx.z];
    const int b = blockIdx.x, lane = threadIdx.x & 63;
    if (b >= L.b1_blocks[0]) return;
    const int c0 = L.b1_cs[0][b], n = L.b1_cs[0][b + 1] - c0, parts = gridDim.y;
    const int from = (int)((int64_t)n * blockIdx.y / parts), to = (int)((int64_t)n * (blockIdx.y + 1) / parts);
    const int2 r = L.b1_row[0][64 * b + lane];
    const int beg = r.x >= 0 ? L.row_ptr[r.x] : 0;
    for (int i = from + (int)(threadIdx.x >> 6); i < to; i += 4) {
        const int e = beg + 8 * i, left = r.y - 8 * i;
        uint4 *dst = (uint4 *)L.b1_lm[0] + (size_t)(c0 + i) * (LDS_HALF_BYTES / 16) + lane;
        float w[8];
        if (left >= 8) {
            const F4 u = *(const F4 *)(L.vals + e), v = *(const F4 *)(L.vals + e + 4);
#pragma unroll
            for (int k = 0; k < 4; ++k) { w[k] = u.v[k]; w[k + 4] = v.v[k]; }
        } else {
#pragma unroll
            for (int k = 0; k < 8; ++k) w[k] = k < left ? L.vals[e + k] : 0.0f;
        }
        if constexpr (COLS) {
            unsigned c[8];
#pragma unroll
            for (int k = 0; k < 8; ++k) c[k] = k < left ? (unsigned)L.col_idx[e + k] : (unsigned)L.n_in;
            dst[0] = make_uint4(c[0] | c[1] << 16, c[2] | c[3] << 16, c[4] | c[5] << 16, c[6] | c[7] << 16);
        }
        dst[64] = make_uint4(__float_as_uint(w[0]), __float_as_uint(w[1]), __float_as_uint(w[2]), __float_as_uint(w[3]));
        dst[128] = make_uint4(__float_as_uint(w[4]), __float_as_uint(w[5]), __float_as_uint(w[6]), __float_as_uint(w[7]));
    }
}

// ---------------------------------------------------------------------------
// K1p: Eq. 3 for one layer whose operand does not fit LDS: a workgroup of 16 wavefronts takes two samples and one range of up
// to 16384 of the layer's rows, and walks the operand in panels of up to 16384 neurons that it holds in LDS one after the other.
// A lane owns a row per block of 64 (up to 16 blocks per wavefront) and keeps their fp64 sums in registers across the
// panels.  Column indices ascend inside a row and panels are column ranges, so every sum keeps its storage order.
//
// Copy of W: for every range and wavefront one stream of slots (a slot: 64 lanes, a 16-bit position in the panel and a weight
// each; halves of eight slots as in k_fwd_lds), panel by panel, in a panel block by block.  A block is as deep in a panel as its
// fullest row there; the rows of a block are chosen with about equal numbers of entries in every panel (sdnn_pan_layout).
// `ends` has a bit for every slot after which the next block's turn follows.  A panel's slots are filled up to a whole half.
// Activations between the layers: [pair of samples][position][2], a panel is one contiguous piece, brought into LDS
// without passing through registers.
//
// What bounds it: the stream of W from L2 (384 bytes a slot), with two samples to share it; a slot takes 10.7 clocks of a CU
// (counted: 6.95 vector instructions, that is 7 clocks of the four SIMDs; LDS reads at random positions 7.8, 4.8 of them conflicts; W 6
// at the L1's 64 bytes per clock, 9 at what an L2 delivers to 32 CUs at once; over the whole launch, panels included, none of them is
// busy for more than 58 % of the time).  Per panel 1.6 us to load it and 1.4 us until the last wavefront is done with the one before:
// 65536 neurons, 55 us per workgroup.  Four samples and panels of 8192 neurons share W better, but 32 entries are then too few for eight panels
// (1.64 slots per entry instead of 1.10; 65536 neurons, 1024 samples 583 against 476 us per layer; 20001 neurons 110 against 121).
// Against k_spmm_panel and k_fwd_lds<1> (24 layers of 32 entries per row, us per layer, before / with it): 65536 neurons, 1024
// samples 849 / 476; 40000 neurons, 1024 samples 618 / 270; 32768 neurons, 512 samples 123 / 96; 65536 neurons, 64 samples
// 53 / 65 (half of the CUs: not taken).
// ---------------------------------------------------------------------------
static_assert(PAN_WAVES == LDS_WAVES, "the same halves, the same workgroups");
struct PanForward {
    const uint4 *stream;   // halves of LDS_HALF_BYTES, and two more
    const int32_t *seg;    // [range][wavefront][panels + 1]: where the panels' slots start, in halves
    const uint32_t *ends;  // a byte per half
    const float *bias;     // by position
    const float2 *in;      // [pairs][in_pos]
    float2 *out;           // [pairs][out_pos]
    uint32_t stream_bytes;
    int32_t in_pos, out_pos; // positions of a sample's activations
    int32_t panel, n_panels; // positions per panel
    int32_t range, n_ranges, nb; // positions per range, and blocks per wavefront
    int32_t n_pairs;
    float cap;
};
// Registers v64 .. v127 of k_fwd_pan are an array of two doubles per block, reached by index: the multiply-adds name the first
// block's registers and `at` (four words per block) is added to them.  The compiler has the 64 below (amdgpu_num_vgpr counts half
// of them) and knows nothing of these: as a variable that is indexed by the block they would be copied, or go through memory, at
// every block.
// Four slots: w[u] x[u][t] is added to the current block's sums; where bit u of `ends` is set, the next block's turn follows.
__device__ __forceinline__ void add_four(int &at, unsigned ends, const double (&w)[4], const double (&x)[4][2])
{
    unsigned s;
#define PAN_ADD(w, x0, x1, bit)                                                                              \
    "v_fma_f64 v[64:65], " w ", " x0 ", v[64:65]\n\tv_fma_f64 v[66:67], " w ", " x1 ", v[66:67]\n\t"           \
    "s_bfe_u32 %1, %2, " bit "\n\ts_lshl2_add_u32 %0, %1, %0\n\t"
    asm volatile("s_set_gpr_idx_on %0, gpr_idx(SRC2,DST)\n\t"
                 PAN_ADD("%3", "%4", "%5", "0x10000") "s_set_gpr_idx_idx %0\n\t"
                 PAN_ADD("%6", "%7", "%8", "0x10001") "s_set_gpr_idx_idx %0\n\t"
                 PAN_ADD("%9", "%10", "%11", "0x10002") "s_set_gpr_idx_idx %0\n\t"
                 PAN_ADD("%12", "%13", "%14", "0x10003")
                 "s_set_gpr_idx_off"
                 : "+s"(at), "=&s"(s)
                 : "s"(ends), "v"(w[0]), "v"(x[0][0]), "v"(x[0][1]), "v"(w[1]), "v"(x[1][0]), "v"(x[1][1]), "v"(w[2]), "v"(x[2][0]), "v"(x[2][1]),
                   "v"(w[3]), "v"(x[3][0]), "v"(x[3][1])
                 : "m0", "scc");
#undef PAN_ADD
}
// All of them to zero; naming the last one as written makes the kernel have them.
__device__ __forceinline__ void clear_sums()
{
    asm volatile("v_mov_b32 v127, 0" ::: "v127");
#pragma unroll
    for (int at = 0; at < 64; at += 4)
        asm volatile("s_set_gpr_idx_on %0, gpr_idx(DST)\n\tv_mov_b32 v64, 0\n\tv_mov_b32 v65, 0\n\tv_mov_b32 v66, 0\n\tv_mov_b32 v67, 0\n\ts_set_gpr_idx_off" ::"s"(at) : "m0");
}
__device__ __forceinline__ void get_sums(int at, double &v0, double &v1)
{
    int w[4];
    asm volatile("s_set_gpr_idx_on %4, gpr_idx(SRC0)\n\t"
                 "v_mov_b32 %0, v64\n\tv_mov_b32 %1, v65\n\tv_mov_b32 %2, v66\n\tv_mov_b32 %3, v67\n\t"
                 "s_set_gpr_idx_off"
                 : "=&v"(w[0]), "=&v"(w[1]), "=&v"(w[2]), "=&v"(w[3])
                 : "s"(at)
                 : "m0");
    v0 = __hiloint2double(w[1], w[0]);
    v1 = __hiloint2double(w[3], w[2]);
}

// STAY: a workgroup takes one piece (a range of a pair) after the other; see forward_pan.
template <int ACT, bool STAY>
__global__ void __launch_bounds__(64 * LDS_WAVES) __attribute__((amdgpu_num_vgpr(32))) k_fwd_pan(const PanForward a)
{
    extern __shared__ __attribute__((aligned(16))) float lds_act[];
    typedef float pair __attribute__((ext_vector_type(2)));
    typedef __attribute__((address_space(3))) pair *lds_ptr;
    typedef __attribute__((address_space(3))) char *lds_bytes;
    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    // The ranges of a pair run side by side on one XCD: they read the same panels (one range of all pairs after the other, so
    // that all the workgroups of an XCD share one stream of W: 602 against 511 us at 65536 neurons, 1024 samples)
    const int xcd = (int)(blockIdx.x & 7u), stride = (int)(gridDim.x >> 3);
    int k = (int)(blockIdx.x >> 3), q = k % a.n_ranges, g = k / a.n_ranges * 8 + xcd; // range and pair of samples
    if (g >= a.n_pairs) return;
    unsigned shift = 3;
    asm("" : "+v"(shift)); // kept in a register for lds_address
    if (tid < 2) lds_act[2 * a.panel + tid] = 0.0f; // where the slots past a row's entries point

    typedef const int32_t __attribute__((address_space(4))) *seg_ptr;
    auto seg_of = [&](int range) { return (seg_ptr)a.seg + (range * LDS_WAVES + wave) * (a.n_panels + 1); };
    seg_ptr seg = seg_of(q);
    const __amdgpu_buffer_rsrc_t rst = make_rsrc((const float *)a.stream, a.stream_bytes);
    const __amdgpu_buffer_rsrc_t ren = make_rsrc((const float *)a.ends, (size_t)a.stream_bytes / LDS_HALF_BYTES);
    int first = seg[0], n = seg[a.n_panels] - first; // this wavefront's halves
    unsigned at = (unsigned)first * LDS_HALF_BYTES, at_end = 0xffffffffu, at_next = 0; // STAY: at the stream's end the next one's halves follow
    const int lane16 = 16 * lane;
    struct Half { u32x4 c, wa, wb; } ha, hb;
    auto request = [&](Half &h) {
        h.c = __builtin_amdgcn_raw_buffer_load_b128(rst, lane16, (int)at, 0);
        h.wa = __builtin_amdgcn_raw_buffer_load_b128(rst, lane16 + 1024, (int)at, 0);
        h.wb = __builtin_amdgcn_raw_buffer_load_b128(rst, lane16 + 2048, (int)at, 0);
        at += LDS_HALF_BYTES;
        if constexpr (STAY) at = at == at_end ? at_next : at;
    };
    clear_sums();
    int block = 0, p = 0, left = 0, half = 0; // block: the current one's words
    unsigned four_ends = 0, word = 0;         // the ends of four halves per lane, of the current four
    auto request_panel = [&](int pair) {
        const __amdgpu_buffer_rsrc_t rin = make_rsrc((const float *)(a.in + (size_t)pair * a.in_pos), (size_t)a.in_pos * 8);
        const int bytes = min(a.panel, a.in_pos - p * a.panel) * 8;
        for (int i = 1024 * wave; i < bytes; i += 1024 * LDS_WAVES)
            if (i + lane16 < bytes)
                __builtin_amdgcn_raw_ptr_buffer_load_lds(rin, (__attribute__((address_space(3))) void *)((lds_bytes)0 + i), 16, lane16, p * a.panel * 8 + i, 0, 0);
    };
    auto panel_there = [&]() {
        __builtin_amdgcn_s_waitcnt(0xf70); // vmcnt(0)
        lds_barrier();
    };
    // The next panel into LDS, once every wavefront is done with the one before.
    auto advance = [&]() {
        if (++p >= a.n_panels) return;
        left = seg[p + 1] - seg[p];
        block = 0;
        lds_barrier();
        request_panel(g);
        panel_there();
    };
    auto take = [&](Half &h) { // eight slots; then their registers are free for the half after next
        unsigned ad[8];
        pair x[8];
#pragma unroll
        for (int u = 0; u < 4; ++u) {
            ad[2 * u] = lds_address<0>(h.c[u], shift);
            ad[2 * u + 1] = lds_address<1>(h.c[u], shift);
        }
#pragma unroll
        for (int u = 0; u < 8; ++u) x[u] = *(lds_ptr)((lds_bytes)0 + ad[u]);
#pragma unroll
        for (int v = 0; v < 8; v += 4) {
            double w[4], xd[4][2];
#pragma unroll
            for (int u = 0; u < 4; ++u) w[u] = (double)__uint_as_float(v ? h.wb[u] : h.wa[u]);
            if (v) request(h);
#pragma unroll
            for (int u = 0; u < 4; ++u) {
                xd[u][0] = (double)x[v + u][0];
                xd[u][1] = (double)x[v + u][1];
            }
            add_four(block, word >> v, w, xd);
        }
        if (--left == 0) advance();
    };
    request_panel(g);
    request(ha);
    request(hb);
    for (;;) {
        const int k_next = k + stride, q_next = k_next % a.n_ranges, g_next = k_next / a.n_ranges * 8 + xcd;
        const bool more = STAY && g_next < a.n_pairs;
        left = seg[1] - first;
        if constexpr (STAY) {
            at_end = (unsigned)(first + n) * LDS_HALF_BYTES;
            at_next = (unsigned)seg_of(q_next)[0] * LDS_HALF_BYTES;
            if (at == at_end) at = at_next; // a stream of two halves
            four_ends = __builtin_amdgcn_raw_buffer_load_b32(ren, 4 * lane, first, 0);
        }
        panel_there();
        for (half = 0; half < n; half += 2) { // a stream starts on a multiple of four halves and has an even number of them
            if ((!STAY || half > 0) && (half & 255) == 0) {
                four_ends = __builtin_amdgcn_raw_buffer_load_b32(ren, 4 * lane, first + half, 0);
                __builtin_amdgcn_s_waitcnt(0xf70);
            }
            if ((half & 3) == 0) word = (unsigned)__builtin_amdgcn_readlane((int)four_ends, (half >> 2) & 63);
            if ((half & 6) == 0) take_turns(wave / 4 + (half >> 3));
            take(ha);
            word >>= 8;
            take(hb);
            word >>= 8;
        }
        // the next piece's first panel comes while this one's results are stored
        if (more) {
            lds_barrier();
            p = 0;
            request_panel(g_next);
        }
        const int at0 = q * a.range + 64 * wave + lane;
        pair *out = (pair *)(a.out + (size_t)g * a.out_pos + (size_t)at0);
        constexpr int K = ACT == ACT_SIGMOID ? 4 : 16; // biases at once (exp() takes their registers)
        for (int b0 = 0; b0 < a.nb; b0 += K) {
            float bias[K];
#pragma unroll
            for (int b = 0; b < K; ++b) bias[b] = a.bias[at0 + 1024 * min(b0 + b, a.nb - 1)];
#pragma unroll
            for (int b = 0; b < K; ++b) {
                if (b0 + b >= a.nb) break;
                double s0, s1;
                get_sums(4 * (b0 + b), s0, s1);
                pair v;
                v[0] = act_apply(ACT, s0 + (double)bias[b], a.cap);
                v[1] = act_apply(ACT, s1 + (double)bias[b], a.cap);
                out[1024 * (b0 + b)] = v;
            }
        }
        if constexpr (!STAY) return;
        if (!more) return;
        clear_sums();
        k = k_next; q = q_next; g = g_next;
        seg = seg_of(q);
        first = seg[0];
        n = seg[a.n_panels] - first;
        block = 0;
    }
}

// Writes the slots of one block in one panel (grid: blocks per wavefront x ranges, wavefronts, panels), and in panel 0 its biases.
__global__ void __launch_bounds__(64) k_pan_fill(const LayerDev *__restrict__ layer, uint4 *__restrict__ stream,
                                                 const int32_t *__restrict__ slot, const int32_t *__restrict__ rows,
                                                 float *__restrict__ bias, int nb, int panel_cols, int panel_pos,
                                                 const int32_t *__restrict__ prev_pos)
{
    const LayerDev &L = *layer;
    const int j = blockIdx.x % nb, q = blockIdx.x / nb, w = blockIdx.y, p = blockIdx.z, lane = threadIdx.x, np = gridDim.z;
    const int at = 1024 * nb * q + 64 * (LDS_WAVES * j + w) + lane;
    const int row = rows[at];
    const int32_t *sl = slot + (size_t)((q * LDS_WAVES + w) * np + p) * (nb + 1) + j;
    const int s0 = sl[0], s1 = sl[1];
    int beg = 0, end = 0;
    if (row >= 0) {
        beg = L.row_ptr[row];
        end = L.row_ptr[row + 1];
    }
    if (p == 0) bias[at] = row >= 0 ? L.bias[row] : 0.0f;
    // the row's entries in this panel: its columns ascend
    auto below = [&](int64_t col) {
        int lo = beg, hi = end;
        while (lo < hi) {
            const int mid = (lo + hi) >> 1;
            if (L.col_idx[mid] < col) lo = mid + 1;
            else hi = mid;
        }
        return lo;
    };
    const int e0 = below((int64_t)p * panel_cols), n = below((int64_t)(p + 1) * panel_cols) - e0;
    for (int s = s0; s < s1; ++s) {
        char *half = (char *)stream + (size_t)(s >> 3) * LDS_HALF_BYTES;
        unsigned pos = (unsigned)panel_pos;
        float wt = 0.0f;
        if (s - s0 < n) {
            const int e = e0 + s - s0, c = L.col_idx[e];
            wt = L.vals[e];
            pos = (unsigned)((prev_pos ? prev_pos[c] : c) - p * panel_pos);
        }
        *(uint16_t *)(half + 16 * lane + 2 * (s & 7)) = (uint16_t)pos;
        *(float *)(half + 1024 + ((s & 4) << 8) + 16 * lane + 4 * (s & 3)) = wt;
    }
}

// Between [neuron][sample] and [pair of samples][position][2]: tiles of 64 neurons and 64 samples through LDS.
// IN: rows of X (row r at position r) to pairs, a zero past the last sample; else pairs to the rows that `rows` names.
template <bool IN>
__global__ void __launch_bounds__(256) k_pan_turn(float *__restrict__ x, int ld, int n, int B, float2 *__restrict__ pairs, int n_pos,
                                                  const int32_t *__restrict__ rows)
{
    __shared__ float tile[64][65];
    const int tid = threadIdx.x, p0 = 64 * blockIdx.x, s0 = 64 * blockIdx.y;
    const int n_pairs = (B + 1) / 2;
    if constexpr (IN) {
        for (int i = tid; i < 4096; i += 256) {
            const int r = i >> 6, s = i & 63;
            tile[r][s] = p0 + r < n && s0 + s < B ? x[(size_t)(p0 + r) * ld + s0 + s] : 0.0f;
        }
        __syncthreads();
        for (int i = tid; i < 2048; i += 256) {
            const int r = i & 63, g = i >> 6;
            if (s0 / 2 + g < n_pairs && p0 + r < n_pos) pairs[(size_t)(s0 / 2 + g) * n_pos + p0 + r] = make_float2(tile[r][2 * g], tile[r][2 * g + 1]);
        }
    } else {
        for (int i = tid; i < 2048; i += 256) {
            const int r = i & 63, g = i >> 6;
            if (s0 / 2 + g < n_pairs && p0 + r < n_pos) {
                const float2 v = pairs[(size_t)(s0 / 2 + g) * n_pos + p0 + r];
                tile[r][2 * g] = v.x;
                tile[r][2 * g + 1] = v.y;
            }
        }
        __syncthreads();
        for (int i = tid; i < 4096; i += 256) {
            const int r = i >> 6, s = i & 63;
            const int row = p0 + r < n_pos ? rows[p0 + r] : -1;
            if (row >= 0 && s0 + s < B) x[(size_t)row * ld + s0 + s] = tile[r][s];
        }
    }
}

// ---------------------------------------------------------------------------
// K2 + K4a: back-propagation through W_l fused with the gradient of W_l's stored entries, for
// launches of at most 64 samples (one sample per lane).  The wavefront of row i of W_l^T gathers
// Delta_l(j, :) for every stored entry (j, i) anyway and holds X_{l-1}(i, :), the two operands of
// Eq. 4 for exactly that entry.  The gathered rows are parked in LDS, 16 entries at a time
// ([entry][sample], padded), and then lane (e, q) sums entry e over quarter q of the samples in fp64;
// the four quarters are added and lane e stores g(j, i) = sum_s Delta_l(j, s) X_{l-1}(i, s) at the
// entry's place in the transposed index.  Every stored entry lies in exactly one row of W_l^T, so the
// launch writes the whole gradient array; nothing is accumulated in memory.  The values are read from
// their copy in the same order (vals_t): the sweep streams through index, values and gradient, and
// only the rows of Delta_l are gathered.  This removes the update's own gather pass over X_{l-1}.
// ---------------------------------------------------------------------------
#define TR_CHUNK 16384 // entries of the CSR array that one workgroup of k_spread_vals fills from LDS (64 KiB)
#define TR_THREADS 512
#define TR_SPAN 8192   // consecutive entries of the transposed index that one workgroup of k_apply takes (32 KiB of LDS)
#define GRAD_LD 68 // floats per parked entry: 64 samples + pad (rows stay 16-byte aligned, banks spread)
#define GRAD_GE 16 // entries parked at a time: 4.6 KB of LDS per wavefront, which keeps 8 wavefronts per SIMD
template <int U>
__device__ __forceinline__ void spmm_row_grad(RowMeta m, const GradArgs &a, int lane,
                                              float *__restrict__ dt, float *__restrict__ xt)
{
    const int B = a.B;
    const bool live = lane < B;
    const int s = live ? lane : 0;
    const size_t ld = (size_t)a.ld_out;
    const unsigned so = 4u * (unsigned)s;
    const unsigned ldb = 4u * (unsigned)a.ld_in;
    const __amdgpu_buffer_rsrc_t rin = make_rsrc(a.in, a.in_bytes);

    const float xp = a.aux[(size_t)m.row * ld + s]; // X_{l-1}(i, s): mask operand and gradient operand
    xt[lane] = live ? xp : 0.0f;                    // samples outside the launch add nothing to the gradient

    double acc = 0.0;
    int c_l = m.c_l, p_l;
    float w_l = m.w_l;
    const int e = lane & (GRAD_GE - 1), q = lane / GRAD_GE; // reducer of entry e over quarter q of the samples
    for (int base = m.beg; base < m.end; base += 64) {
        const int n = min(64, m.end - base);
        // a.vals is the copy of the values in the order of the transposed index: read like a forward row
        if (base != m.beg) load_chunk<0>(a.idx, a.vals, nullptr, base, m.end, lane, c_l, w_l, p_l);
        for (int g0 = 0; g0 < n; g0 += GRAD_GE) { // GRAD_GE entries are parked at a time
            const int ng = min(GRAD_GE, n - g0);
            for (int g = 0; g < ng; g += U) {
                float x[U];
                if (g + U <= ng) {
#pragma unroll
                    for (int k = 0; k < U; ++k) {
                        const int c = __builtin_amdgcn_readlane(c_l, g0 + g + k);
                        x[k] = __uint_as_float(__builtin_amdgcn_raw_buffer_load_b32(rin, (int)so, (int)((unsigned)c * ldb), 0));
                    }
#pragma unroll
                    for (int k = 0; k < U; ++k) {
                        const double wk = (double)__int_as_float(__builtin_amdgcn_readlane(__float_as_int(w_l), g0 + g + k));
                        acc = fma(wk, (double)x[k], acc);
                        dt[(g + k) * GRAD_LD + lane] = x[k];
                    }
                } else { // ragged end of the row: same order, every entry guarded (wave-uniform branches)
#pragma unroll
                    for (int k = 0; k < U; ++k)
                        if (g + k < ng) {
                            const int c = __builtin_amdgcn_readlane(c_l, g0 + g + k);
                            x[k] = __uint_as_float(__builtin_amdgcn_raw_buffer_load_b32(rin, (int)so, (int)((unsigned)c * ldb), 0));
                        }
#pragma unroll
                    for (int k = 0; k < U; ++k)
                        if (g + k < ng) {
                            const double wk = (double)__int_as_float(__builtin_amdgcn_readlane(__float_as_int(w_l), g0 + g + k));
                            acc = fma(wk, (double)x[k], acc);
                            dt[(g + k) * GRAD_LD + lane] = x[k];
                        }
                }
            }
            // entry e of this group, samples 16q .. 16q+15: the lanes now read what other lanes of the
            // wavefront have parked
            wave_lds_sync();
            double sum = 0.0;
            if (e < ng) {
                const float4 *dp = reinterpret_cast<const float4 *>(dt + e * GRAD_LD + 16 * q);
                const float4 *xq = reinterpret_cast<const float4 *>(xt + 16 * q);
#pragma unroll
                for (int t = 0; t < 4; ++t) {
                    const float4 d4 = dp[t], x4 = xq[t];
                    sum = fma((double)d4.x, (double)x4.x, sum);
                    sum = fma((double)d4.y, (double)x4.y, sum);
                    sum = fma((double)d4.z, (double)x4.z, sum);
                    sum = fma((double)d4.w, (double)x4.w, sum);
                }
            }
            sum += __shfl_xor(sum, 16);
            sum += __shfl_xor(sum, 32);
            if (q == 0 && e < ng) a.g_part[0][base + g0 + e] = (float)sum; // the entry's place in the transposed index
            wave_lds_sync(); // the next group's rows are parked over the ones just read
        }
    }
    if (a.store_out && lane < (fills_up(B, a.ld_out) ? (B + 3) & ~3 : B))
        a.out[(size_t)m.row * ld + lane] = live ? act_backprop(a.act, acc, xp, a.cap) : 0.0f;
}
template <int U>
__global__ void __launch_bounds__(BLOCK_THREADS) k_bwd_grad(const GradArgs a)
{
    __shared__ __attribute__((aligned(16))) float dt[WAVES_PER_BLOCK][GRAD_GE * GRAD_LD];
    __shared__ __attribute__((aligned(16))) float xt[WAVES_PER_BLOCK][64];
    const int lane = threadIdx.x & 63;
    const unsigned wave = threadIdx.x >> 6;
    for (unsigned vb = blockIdx.x; vb < a.n_vblocks; vb += gridDim.x) {
        const int r = __builtin_amdgcn_readfirstlane((int)(vb * WAVES_PER_BLOCK + wave));
        if (r >= a.n_rows) continue;
        const RowMeta m = load_meta<0>(a.sched, a.idx, a.vals, nullptr, r, lane);
        spmm_row_grad<U>(m, a, lane, dt[wave], xt[wave]);
    }
}

// ---------------------------------------------------------------------------
// K3: output delta (Eq. 6):  D = dLoss * [0 < X_L < cap]
// ---------------------------------------------------------------------------
// Elementwise passes between the caller's rows of B floats and the library's rows of ld: a row takes 1 << w_log2 threads
// of a workgroup (Bp, or all 256), columns B .. Bp - 1 of the destination are zeroed.
#define FOR_ROW_ELEMENTS(n_rows, Bp, w_log2)                                                                  \
    for (int row = (int)(blockIdx.x * (256u >> (w_log2)) + (threadIdx.x >> (w_log2))); row < (n_rows);          \
         row += (int)(gridDim.x * (256u >> (w_log2))))                                                          \
        for (int s = (int)(threadIdx.x & ((1u << (w_log2)) - 1u)); s < (Bp); s += 1 << (w_log2))
__global__ void __launch_bounds__(256) k_output_delta(const float *__restrict__ dloss, const float *__restrict__ xl,
                                                      float *__restrict__ d, int n_rows, int B, int ld, int Bp, int w_log2,
                                                      float cap, int act)
{
    FOR_ROW_ELEMENTS(n_rows, Bp, w_log2)
    {
        const size_t at = (size_t)row * ld + s;
        d[at] = s < B ? act_backprop(act, (double)dloss[(size_t)row * B + s], xl[at], cap) : 0.0f;
    }
}
__global__ void __launch_bounds__(256) k_copy_rows(const float *__restrict__ src, int ld_src, float *__restrict__ dst, int ld_dst,
                                                   int n_rows, int B, int Bp, int w_log2)
{
    FOR_ROW_ELEMENTS(n_rows, Bp, w_log2)
        dst[(size_t)row * ld_dst + s] = s < B ? src[(size_t)row * ld_src + s] : 0.0f;
}

// ---------------------------------------------------------------------------
// One sample per step (B = 1, the paper's own training experiments: one input
// vector per SGD step, Section 6.1).  Lanes over samples would idle 63 of 64
// lanes, so there are three products of their own, all taking each row's sum in
// storage order (same result as everywhere else):
//   k_spmv_stage  wide layers with short rows: lanes over a contiguous stretch of entries,
//                 products parked in LDS, then a lane per row adds them up;
//   k_spmv_wave   narrow layers, or long rows up to 16384 rows: a wavefront per row;
//   k_spmv        the rest (wide layers with long rows): a lane per row.
// ---------------------------------------------------------------------------
template <int MODE>
__global__ void __launch_bounds__(256) k_spmv(const SpmmArgs a)
{
    const int row = blockIdx.x * blockDim.x + threadIdx.x;
    if (row >= a.n_rows) return;
    const int beg = a.row_ptr[row], end = a.row_ptr[row + 1];
    double acc = 0.0;
    constexpr int U = 16; // entries requested together; the additions stay in storage order
    for (int p0 = beg; p0 < end; p0 += U) {
        int c[U];
        float w[U], x[U];
#pragma unroll
        for (int k = 0; k < U; ++k) {
            const int p = min(p0 + k, end - 1);
            c[k] = a.idx[p];
            w[k] = MODE == 1 ? a.vals[a.perm[p]] : a.vals[p];
        }
#pragma unroll
        for (int k = 0; k < U; ++k) x[k] = a.in[c[k]];
#pragma unroll
        for (int k = 0; k < U; ++k)
            if (p0 + k < end) acc = fma((double)w[k], (double)x[k], acc);
    }
    if (MODE == 0) a.out[row] = act_apply(a.act, acc + (a.aux ? (double)a.aux[row] : 0.0), a.cap);
    else a.out[row] = act_backprop(a.act, acc, a.aux[row], a.cap);
}

// Same product for narrow layers, where a lane per row leaves most of the chip idle: a wavefront
// per row.  The row's entries and the activations they point at are fetched by two wave-wide loads
// (entry k in lane k); the sum itself is still taken in storage order, every lane redoing it from
// the broadcast operands.
template <int MODE>
__global__ void __launch_bounds__(BLOCK_THREADS) k_spmv_wave(const SpmmArgs a)
{
    const int lane = threadIdx.x & 63;
    const int row = __builtin_amdgcn_readfirstlane((int)(blockIdx.x * WAVES_PER_BLOCK + (threadIdx.x >> 6)));
    if (row >= a.n_rows) return;
    const int beg = a.row_ptr[row], end = a.row_ptr[row + 1];
    double acc = 0.0;
    for (int base = beg; base < end; base += 64) {
        const int n = min(64, end - base);
        float w_l = 0.0f, x_l = 0.0f;
        if (lane < n) {
            const int p = base + lane;
            w_l = MODE == 1 ? a.vals[a.perm[p]] : a.vals[p];
            x_l = a.in[a.idx[p]];
        }
        for (int k = 0; k < n; ++k) {
            const double wk = (double)__int_as_float(__builtin_amdgcn_readlane(__float_as_int(w_l), k));
            const double xk = (double)__int_as_float(__builtin_amdgcn_readlane(__float_as_int(x_l), k));
            acc = fma(wk, xk, acc);
        }
    }
    if (lane == 0) {
        if (MODE == 0) a.out[row] = act_apply(a.act, acc + (a.aux ? (double)a.aux[row] : 0.0), a.cap);
        else a.out[row] = act_backprop(a.act, acc, a.aux[row], a.cap);
    }
}

// Wide layers at B = 1: a 64-lane workgroup owns R consecutive rows, whose entries are one contiguous
// stretch of the index arrays.  All lanes walk that stretch together (coalesced index and value
// loads, one gathered activation per entry) and park the products w*x, which are exact in fp64, in
// LDS; then lane r adds the products of row r in storage order, the same sum as everywhere else.
// The stretch is taken in segments of SPMV_STAGE entries, so rows of any length work.
#define SPMV_STAGE 1024
#define SPMV_STAGE_MIN_ROWS 2048 // below this a wavefront per row is as fast (measured)
template <int MODE, int J>
__global__ void __launch_bounds__(64) k_spmv_stage(const SpmmArgs a, int R)
{
    __shared__ double prod[SPMV_STAGE + SPMV_STAGE / 32]; // one pad per 32 entries: lanes that start 32 apart hit different banks
    const int lane = threadIdx.x;
    const int r0 = blockIdx.x * R;
    const int nr = min(R, a.n_rows - r0); // >= 1 by the grid size
    const int row = r0 + lane;
    int p = 0, end = 0;
    if (lane < nr) { p = a.row_ptr[row]; end = a.row_ptr[row + 1]; }
    const int e0 = a.row_ptr[r0], e1 = a.row_ptr[r0 + nr];
    double acc = 0.0;
    for (int sb = e0; sb < e1; sb += SPMV_STAGE) {
        const int se = min(sb + SPMV_STAGE, e1);
        for (int j0 = 0; j0 * 64 < se - sb; j0 += J) {
            int c[J];
            float w[J], x[J];
#pragma unroll
            for (int j = 0; j < J; ++j) {
                const int e = sb + (j0 + j) * 64 + lane;
                c[j] = -1;
                if (e < se) {
                    c[j] = a.idx[e];
                    w[j] = MODE == 1 ? a.vals[a.perm[e]] : a.vals[e];
                }
            }
#pragma unroll
            for (int j = 0; j < J; ++j)
                if (c[j] >= 0) x[j] = a.in[c[j]];
#pragma unroll
            for (int j = 0; j < J; ++j)
                if (c[j] >= 0) {
                    const int q = (j0 + j) * 64 + lane;
                    prod[q + (q >> 5)] = (double)w[j] * (double)x[j];
                }
        }
        __syncthreads();
        const int pe = min(end, se); // my row's entries inside this segment are [p, pe)
        if (p < pe) {
            for (; p < pe; p += 4) { // four parked products requested together, added one after the other
                double v[4];
#pragma unroll
                for (int k = 0; k < 4; ++k) {
                    const int q = min(p + k, pe - 1) - sb;
                    v[k] = prod[q + (q >> 5)];
                }
#pragma unroll
                for (int k = 0; k < 4; ++k)
                    if (p + k < pe) acc += v[k];
            }
            p = pe;
        }
        __syncthreads();
    }
    if (lane < nr) {
        if (MODE == 0) a.out[row] = act_apply(a.act, acc + (a.aux ? (double)a.aux[row] : 0.0), a.cap);
        else a.out[row] = act_backprop(a.act, acc, a.aux[row], a.cap);
    }
}

// ---------------------------------------------------------------------------
// Nets made for one sample per step (max_batch == 1, rows of moderate length), and inference calls with one sample on
// nets that hold the lane-major copy of k_fwd_lds: a lane per row over a lane-major copy, so that columns and weights come
// in coalesced 16-byte loads and nothing is parked or exchanged; up to 32 gathers of single activations (back: 64) are in flight per
// lane.  Training nets keep one copy of W and one of W^T and step both (no gradient of the entries is stored and no value
// moves from one order to the other); the CSR values are written out when they are asked for.
// What bounds them: a launch and its chain of dependent loads (3.3 us at 1024 neurons) plus, on wide layers, a 128-byte line from L2
// for every gathered activation (with it 4.3 and 4.5 us at 16384).  Forward / backward / step, us per layer, before (products staged in
// LDS, a gradient array, the values moved from the transposed to the CSR order; arrays partly on chip) and now (three nets in turn, their
// arrays from HBM): 1024 neurons 4.6 / 4.8 / 0.2, 3.3 / 3.4 / 0.1; 16384 neurons 6.1 / 8.7 / 3.9, 4.3 / 4.5 / 2.4; 65536 neurons 14.9 /
// 22.3 / 15.7, 11.0 / 11.1 / 20.8.
// ---------------------------------------------------------------------------
#define B1_MAX_LDS (160 * 1024) // bytes of the step's LDS copy of a vector
template <bool WIDE> struct B1 { // columns of 2 bytes, or (more than 65536 of them) 4
    static constexpr unsigned CHUNK_BYTES = WIDE ? 4096 : 3072, WEIGHTS = WIDE ? 2048 : 1024;
};
struct SpmvLmArgs {
    const int32_t *cs;   // training: chunk table of the layer; inference: lm_cs
    const int2 *row;     // training: {row, entries} per lane; inference: NULL
    const int32_t *lm_row; // inference, last layer: the row of a position (NULL on the layers before: results stay at their positions)
    const uint4 *lm;
    unsigned lm_bytes;
    const float *in;
    unsigned in_bytes;
    const float *aux;    // MODE 0: biases, MODE 1 and 2: X_{l-1}; in the order of the results' places
    float *out;
    float cap;
    int32_t act;
    int32_t nb, tab_cs, tab_pos; // inference: the layer's LmLayer
};
template <int MODE, bool WIDE, bool TRAIN>
__global__ void __launch_bounds__(64) k_spmv_lm(const SpmvLmArgs a)
{
    const int lane = threadIdx.x, b = blockIdx.x;
    typedef const int32_t __attribute__((address_space(4))) *cs_ptr;
    const cs_ptr scs = (cs_ptr)a.cs;
    // Chunks requested together.  Back-propagation (MODE 1): the longest of a few thousand random columns with 32 entries in the mean
    // have about sixty, and a second round of loads and gathers for them is what the whole layer would wait for.  Not in layers of more
    // than three wavefronts per CU, which the L2 is busy with (MODE 2).  Step, us per layer, four chunks / eight: 1024 neurons 6.92 /
    // 6.70, 4096 7.53 / 7.25, 8192 9.51 / 9.12, 16384 11.66 / 11.22, 32768 17.33 / 17.08; forward and back-propagation 40001 neurons
    // 14.81 / 14.69, 49000 16.87 / 16.82, 49200 17.10 / 17.17, 60000 19.95 / 20.05, 65504 21.31 / 21.51, 65536 22.45 / 22.75.
    constexpr int LOAD = TRAIN && MODE == 1 && !WIDE ? 8 : 4;
    int c0, n, place; // first chunk, chunks, where the result goes
    [[maybe_unused]] int len = 0; // TRAIN: entries of the lane's row
    if constexpr (TRAIN) {
        c0 = scs[b];
        n = scs[b + 1] - c0;
        const int2 r = a.row[64 * b + lane];
        place = r.x;
        len = r.y;
    } else { // position 64 (16 j + w) + lane: block j of wavefront w, two chunks of eight for each of its sixteen entries
        const int j = b / LDS_WAVES, w = b - j * LDS_WAVES, at = a.tab_cs + w * (a.nb + 1) + j;
        c0 = 2 * scs[at];
        n = 2 * scs[at + 1] - c0;
        place = 64 * b + lane;
    }
    const __amdgpu_buffer_rsrc_t rlm = make_rsrc((const float *)a.lm, a.lm_bytes), rin = make_rsrc(a.in, a.in_bytes);
    float aux = 0.0f;
    int dst = place;
    if constexpr (TRAIN) {
        if (a.aux) aux = a.aux[max(place, 0)];
    } else {
        aux = a.aux[a.tab_pos + place];
        if (a.lm_row) dst = a.lm_row[a.tab_pos + place];
    }
    double acc = 0.0;
    unsigned at = (unsigned)c0 * B1<WIDE>::CHUNK_BYTES;
    for (int i = 0; i < n; i += LOAD, at += LOAD * B1<WIDE>::CHUNK_BYTES) {
        u32x4 c[LOAD], ch[LOAD], wa[LOAD], wb[LOAD];
        float x[LOAD][8];
#pragma unroll
        for (int u = 0; u < LOAD; ++u)
            if (i + u < n) {
                const int o = (int)(at + u * B1<WIDE>::CHUNK_BYTES);
                c[u] = __builtin_amdgcn_raw_buffer_load_b128(rlm, 16 * lane, o, 0);
                if (WIDE) ch[u] = __builtin_amdgcn_raw_buffer_load_b128(rlm, 16 * lane + 1024, o, 0);
                wa[u] = __builtin_amdgcn_raw_buffer_load_b128(rlm, 16 * lane + B1<WIDE>::WEIGHTS, o, 0);
                wb[u] = __builtin_amdgcn_raw_buffer_load_b128(rlm, 16 * lane + B1<WIDE>::WEIGHTS + 1024, o, 0);
            }
#pragma unroll
        for (int u = 0; u < LOAD; ++u)
            if (i + u < n) {
#pragma unroll
                for (int k = 0; k < 8; ++k) {
                    const unsigned col = WIDE ? (k < 4 ? c[u][k & 3] : ch[u][k & 3]) : (k & 1) ? c[u][k >> 1] >> 16 : c[u][k >> 1] & 0xffffu;
                    x[u][k] = __uint_as_float(__builtin_amdgcn_raw_buffer_load_b32(rin, (int)(4u * col), 0, 0));
                }
            }
        if (TRAIN && !WIDE && a.in_bytes > 4u * 0xffffu) { // 65536 columns: no 2-byte column is outside the operand
#pragma unroll
            for (int u = 0; u < LOAD; ++u)
                if (i + u < n) {
#pragma unroll
                    for (int k = 0; k < 8; ++k)
                        if (8 * (i + u) + k >= len) x[u][k] = 0.0f;
                }
        }
#pragma unroll
        for (int u = 0; u < LOAD; ++u)
            if (i + u < n) {
#pragma unroll
                for (int k = 0; k < 8; ++k)
                    acc = fma((double)__uint_as_float(k < 4 ? wa[u][k & 3] : wb[u][k & 3]), (double)x[u][k], acc);
            }
    }
    if (dst < 0) return;
    if (MODE == 0) a.out[dst] = act_apply(a.act, acc + (double)aux, a.cap);
    else a.out[dst] = act_backprop(a.act, acc, aux, a.cap);
}

// The step of such a net: w -= lr (delta_j x_i) on both copies, in a stream over each; the lane's own row gives one of the
// two factors, the other is gathered: from the vector's copy in LDS where it fits, since from L2 every 4-byte gather pulls in
// a 128-byte line (16384 neurons: 3.6 -> 1.9 us per layer).  grid = (parts, 2, layers): a workgroup takes every parts-th group
// of 16 blocks of W (blockIdx.y = 0) or of W^T.
template <bool WIDE, bool IN_LDS> // not both: more than 65536 neurons do not fit LDS
__global__ void __launch_bounds__(64 * LDS_WAVES) k_update_lm(const LayerDev *__restrict__ layers, float lr, int update_bias)
{
    extern __shared__ __attribute__((aligned(16))) float lds_vec[];
    typedef __attribute__((address_space(1))) float *gf;
    typedef const __attribute__((address_space(1))) float *gcf;
    typedef float f32x4 __attribute__((ext_vector_type(4)));
    typedef const __attribute__((address_space(1))) f32x4 *gcf4;
    const LayerDev &L = layers[blockIdx.z];
    const int lane = threadIdx.x & 63, o = blockIdx.y, nb = L.b1_blocks[o];
    int b = __builtin_amdgcn_readfirstlane((int)(blockIdx.x * LDS_WAVES + (threadIdx.x >> 6)));
    const gcf mine = (gcf)(o ? L.X_prev : L.D), other = (gcf)(o ? L.D : L.X_prev);
    const int n_other = o ? L.n_out : L.n_in;
    if constexpr (IN_LDS) {
        for (int i = threadIdx.x; i < n_other / 4; i += 64 * LDS_WAVES) reinterpret_cast<f32x4 *>(lds_vec)[i] = ((gcf4)other)[i];
        if ((int)threadIdx.x < (n_other & 3)) lds_vec[(n_other & ~3) + threadIdx.x] = other[(n_other & ~3) + threadIdx.x];
        __syncthreads();
    }
    const __amdgpu_buffer_rsrc_t rv = make_rsrc(o ? L.D : L.X_prev, 4 * (size_t)n_other);
    const __amdgpu_buffer_rsrc_t rlm = make_rsrc((const float *)L.b1_lm[o], (size_t)L.b1_cs[o][nb] * B1<WIDE>::CHUNK_BYTES);
    const double dlr = (double)lr;
    for (; b < nb; b += gridDim.x * LDS_WAVES) {
        const int c0 = L.b1_cs[o][b], n = L.b1_cs[o][b + 1] - c0;
        const int2 r = L.b1_row[o][64 * b + lane];
        const double d = r.x >= 0 ? (double)mine[r.x] : 0.0;
        unsigned at = (unsigned)c0 * B1<WIDE>::CHUNK_BYTES;
        for (int i = 0; i < n; i += 2, at += 2 * B1<WIDE>::CHUNK_BYTES) {
            u32x4 c[2], ch[2], w[2][2];
            float v[2][8];
#pragma unroll
            for (int u = 0; u < 2; ++u)
                if (i + u < n) {
                    const int q = (int)(at + u * B1<WIDE>::CHUNK_BYTES);
                    c[u] = __builtin_amdgcn_raw_buffer_load_b128(rlm, 16 * lane, q, 0);
                    if (WIDE) ch[u] = __builtin_amdgcn_raw_buffer_load_b128(rlm, 16 * lane + 1024, q, 0);
                    w[u][0] = __builtin_amdgcn_raw_buffer_load_b128(rlm, 16 * lane + B1<WIDE>::WEIGHTS, q, 0);
                    w[u][1] = __builtin_amdgcn_raw_buffer_load_b128(rlm, 16 * lane + B1<WIDE>::WEIGHTS + 1024, q, 0);
                }
#pragma unroll
            for (int u = 0; u < 2; ++u)
                if (i + u < n) {
#pragma unroll
                    for (int k = 0; k < 8; ++k) {
                        const unsigned col = WIDE ? (k < 4 ? c[u][k & 3] : ch[u][k & 3]) : (k & 1) ? c[u][k >> 1] >> 16 : c[u][k >> 1] & 0xffffu;
                        if (IN_LDS) v[u][k] = lds_vec[col];
                        else v[u][k] = __uint_as_float(__builtin_amdgcn_raw_buffer_load_b32(rv, (int)(4u * col), 0, 0));
                    }
                }
#pragma unroll
            for (int u = 0; u < 2; ++u)
                if (i + u < n) {
#pragma unroll
                    for (int k = 0; k < 8; ++k) {
                        const float g = (float)(d * (double)v[u][k]);
                        const float old = __uint_as_float(w[u][k >> 2][k & 3]);
                        if (8 * (i + u) + k < r.y) w[u][k >> 2][k & 3] = __float_as_uint((float)((double)old - dlr * (double)g)); // padding stays zero
                    }
                    const int q = (int)(at + u * B1<WIDE>::CHUNK_BYTES);
                    __builtin_amdgcn_raw_buffer_store_b128(w[u][0], rlm, 16 * lane + B1<WIDE>::WEIGHTS, q, 0);
                    __builtin_amdgcn_raw_buffer_store_b128(w[u][1], rlm, 16 * lane + B1<WIDE>::WEIGHTS + 1024, q, 0);
                }
        }
        if (o == 0 && update_bias && r.x >= 0) {
            const gf bias = (gf)L.bias;
            bias[r.x] = (float)((double)bias[r.x] - dlr * d);
        }
    }
}

// Writes one of the two copies of a layer from its CSR arrays (o = 0: W, 1: W^T through the transposed index).  grid = (blocks,
// parts): a workgroup takes every parts-th chunk of a block.
template <bool WIDE>
__global__ void __launch_bounds__(64) k_b1_fill(const LayerDev *__restrict__ layer, int o, int with_cols)
{
    const LayerDev &L = *layer;
    const int lane = threadIdx.x, b = blockIdx.x;
    const int c0 = L.b1_cs[o][b], n = L.b1_cs[o][b + 1] - c0;
    const int2 r = L.b1_row[o][64 * b + lane];
    const int beg = r.x >= 0 ? (o ? L.t_row_ptr[r.x] : L.row_ptr[r.x]) : 0;
    // slots past the end of a row: weight 0, and a column past the end of the operand, which k_spmv_lm reads as 0 (a masked one
    // where 2 bytes hold none)
    const unsigned n_cols = (unsigned)(o ? L.n_out : L.n_in), pad = WIDE ? n_cols : min(n_cols, 0xffffu);
    for (int i = blockIdx.y; i < n; i += gridDim.y) {
        unsigned col[8], w[8];
#pragma unroll
        for (int k = 0; k < 8; ++k) {
            col[k] = pad;
            w[k] = 0;
            if (8 * i + k < r.y) {
                const int e = beg + 8 * i + k;
                w[k] = __float_as_uint(L.vals[o ? L.t_perm[e] : e]);
                if (with_cols) col[k] = (unsigned)(o ? L.t_row_idx[e] : L.col_idx[e]);
            }
        }
        uint4 *dst = (uint4 *)L.b1_lm[o] + (size_t)(c0 + i) * (B1<WIDE>::CHUNK_BYTES / 16) + lane;
        if (with_cols) {
            if (WIDE) {
                dst[0] = make_uint4(col[0], col[1], col[2], col[3]);
                dst[64] = make_uint4(col[4], col[5], col[6], col[7]);
            } else {
                dst[0] = make_uint4(col[0] | col[1] << 16, col[2] | col[3] << 16, col[4] | col[5] << 16, col[6] | col[7] << 16);
            }
        }
        dst[B1<WIDE>::WEIGHTS / 16] = make_uint4(w[0], w[1], w[2], w[3]);
        dst[B1<WIDE>::WEIGHTS / 16 + 64] = make_uint4(w[4], w[5], w[6], w[7]);
    }
}

// The values of a layer in CSR order, from the copy of W.  grid = (blocks, parts), as above (1024 rows of up to 256 entries:
// 47 us with a block's chunks one after the other, 15 in parts).
template <bool WIDE>
__global__ void __launch_bounds__(64) k_b1_values(const LayerDev *__restrict__ layer, float *__restrict__ values)
{
    const LayerDev &L = *layer;
    const int lane = threadIdx.x, b = blockIdx.x;
    const int c0 = L.b1_cs[0][b], n = L.b1_cs[0][b + 1] - c0;
    const int2 r = L.b1_row[0][64 * b + lane];
    if (r.x < 0) return;
    float *dst = values + L.row_ptr[r.x];
    for (int i = blockIdx.y; i < n; i += gridDim.y) {
        const uint4 *src = (const uint4 *)L.b1_lm[0] + (size_t)(c0 + i) * (B1<WIDE>::CHUNK_BYTES / 16) + B1<WIDE>::WEIGHTS / 16 + lane;
        const uint4 a = src[0], c = src[64];
        const unsigned w[8] = {a.x, a.y, a.z, a.w, c.x, c.y, c.z, c.w};
#pragma unroll
        for (int k = 0; k < 8; ++k)
            if (8 * i + k < r.y) dst[8 * i + k] = __uint_as_float(w[k]);
    }
}

// Update for B = 1: no sum over samples, so the lanes take the entries of the rows:
// vals[p] -= lr * delta(row) * x(col[p]).  A wavefront holds 64 >> lpr_log2 rows of 1 << lpr_log2
// lanes each (chosen from the mean row length, so that short rows do not idle half the lanes);
// the first lane of a row does its bias.
__global__ void __launch_bounds__(BLOCK_THREADS)
k_update_b1(const LayerDev *__restrict__ layers, int layer0, int lpr_log2, float lr, int update_bias, int emit,
            float *__restrict__ g_out, float *__restrict__ gb_out)
{
    const LayerDev &L = layers[layer0 + blockIdx.y];
    const int lane = threadIdx.x & 63;
    const int lpr = 1 << lpr_log2;
    const int l = lane & (lpr - 1);
    const int row = ((blockIdx.x * WAVES_PER_BLOCK + (threadIdx.x >> 6)) << (6 - lpr_log2)) + (lane >> lpr_log2);
    if (row >= L.n_out) return;
    const int beg = L.row_ptr[row], end = L.row_ptr[row + 1];
    const float d = L.D[row];
    const double dlr = (double)lr;
    for (int p = beg + l; p < end; p += lpr) {
        const float g = (float)((double)d * (double)L.X_prev[L.col_idx[p]]);
        if (emit) { if (g_out) g_out[p] = g; }
        else L.vals[p] = (float)((double)L.vals[p] - dlr * (double)g);
    }
    if (l == 0) {
        if (emit) { if (gb_out) gb_out[row] = d; }
        else if (update_bias) L.bias[row] = (float)((double)L.bias[row] - dlr * (double)d);
    }
}

// ---------------------------------------------------------------------------
// K4: gradient on the stored pattern (Eq. 4) fused with the update (Eq. 5)
//   blockIdx.y = layer; a wavefront takes rows_per_wave rows one after the other (several when rows
//   are short: fewer, longer-lived wavefronts).  Lane = 16*eg + sg: edge group
//   eg handles 8 consecutive entries of a 32-entry chunk of the row, sample
//   lane sg handles samples sg*V + 16*V*t.  A 16-lane butterfly then leaves
//   the 8 sums of an edge group in 8 different lanes, which write them back.
//   emit == 0: vals -= lr*g, bias -= lr*gb (if update_bias)
//   emit == 1: g_out / gb_out receive the gradient of the single layer
// ---------------------------------------------------------------------------
// HOLD > 0: the batch has at most 16 * V * HOLD samples and the lane keeps its share of the row of Delta in
// registers for the whole row (long rows: otherwise it is read again for every 32-entry chunk).
template <int V, int HOLD>
__global__ void __launch_bounds__(64 * UPD_WAVES)
k_update(const LayerDev *__restrict__ layers, int layer0, int n_layers, int interleave, int rows_per_wave, int B, int ld_,
         float lr, int update_bias, int emit, float *__restrict__ g_out, float *__restrict__ gb_out)
{
    // interleaved: grid = (8 * row groups, groups of 8 layers), blockIdx.x % 8 is both the XCD and the
    // layer inside the group, so all gathers of one layer go through one L2, which then fetches that
    // layer's activations once instead of once per XCD.  Plain (few layers: the XCDs would not all
    // have one): grid = (row groups, layers).
    const int layer_rel = interleave ? (int)(8u * blockIdx.y + (blockIdx.x & 7u)) : (int)blockIdx.y;
    if (layer_rel >= n_layers) return;
    const LayerDev &L = layers[layer0 + layer_rel];
    const int lane = threadIdx.x & 63;
    const unsigned rgi = interleave ? (blockIdx.x >> 3) : blockIdx.x;
    const int r0 = __builtin_amdgcn_readfirstlane((int)((rgi * UPD_WAVES + (threadIdx.x >> 6)) * rows_per_wave));
  for (int r = r0; r < min(r0 + rows_per_wave, L.n_out); ++r) {
    const int4 task = L.sched[r];
    const int row = task.x, beg = task.y, end = task.z;
    const size_t ld = (size_t)ld_;
    const float *drow = L.D + (size_t)row * ld;
    const float *xp = L.X_prev;
    const double dlr = (double)lr;

    // bias gradient: sum of the row of Delta over the samples
    if (emit ? gb_out != nullptr : update_bias != 0) {
        double sum = 0.0;
        for (int s = lane * V; s < B; s += 64 * V) {
            float d[V];
            ldv<V>(drow + s, d);
#pragma unroll
            for (int v = 0; v < V; ++v) sum += (double)d[v];
        }
        sum = add_lane_xor<4>(add_lane_xor<5>(sum));
        sum += lane_xor<3>(sum);
        sum += lane_xor<2>(sum);
        sum += lane_xor<1>(sum);
        sum += lane_xor<0>(sum);
        if (lane == 0) {
            const float gb = (float)sum;
            if (emit) gb_out[row] = gb;
            else L.bias[row] = (float)((double)L.bias[row] - dlr * (double)gb);
        }
    }
    if (emit && g_out == nullptr) continue;

    const int sg = lane & 15, eg = lane >> 4;
    float dh[HOLD > 0 ? HOLD : 1][V];
    if constexpr (HOLD > 0) {
#pragma unroll
        for (int t = 0; t < HOLD; ++t) {
            const int s = sg * V + 16 * V * t;
#pragma unroll
            for (int v = 0; v < V; ++v) dh[t][v] = 0.0f;
            if (s < B) ldv<V>(drow + s, dh[t]);
        }
    }
    for (int base = beg; base < end; base += 32) {
        const int p0 = base + eg * 8;
        size_t coff[8];
#pragma unroll
        for (int k = 0; k < 8; ++k) {
            const int p = p0 + k;
            coff[k] = (size_t)(p < end ? L.col_idx[p] : L.col_idx[beg]) * ld;
        }
        // the weight this lane will rewrite at the end of the chunk, requested now
        const int kw = ((lane >> 3) & 1) * 4 + ((lane >> 2) & 1) * 2 + ((lane >> 1) & 1);
        const bool writer = (lane & 1) == 0 && p0 + kw < end;
        float w_old = 0.0f;
        if (writer && !emit) w_old = L.vals[p0 + kw];
        double a[8];
#pragma unroll
        for (int k = 0; k < 8; ++k) a[k] = 0.0;
        auto pass = [&](int s, const float (&df)[V]) { // the chunk's 8 entries against V samples of this lane
            float x[8][V];
#pragma unroll
            for (int k = 0; k < 8; ++k) ldv<V>(xp + coff[k] + s, x[k]);
            double d[V];
#pragma unroll
            for (int v = 0; v < V; ++v) d[v] = (double)df[v];
#pragma unroll
            for (int k = 0; k < 8; ++k)
#pragma unroll
                for (int v = 0; v < V; ++v) a[k] = fma(d[v], (double)x[k][v], a[k]);
        };
        if constexpr (HOLD > 0) {
#pragma unroll
            for (int t = 0; t < HOLD; ++t) {
                const int s = sg * V + 16 * V * t;
                if (s < B) pass(s, dh[t]);
            }
        } else {
            for (int s = sg * V; s < B; s += 16 * V) {
                float df[V];
                ldv<V>(drow + s, df);
                pass(s, df);
            }
        }
        // 16-lane transpose-reduce: 8 values/lane -> 1 value/lane (register indices are compile-time)
        {
            const bool up8 = (lane & 8) != 0, up4 = (lane & 4) != 0, up2 = (lane & 2) != 0;
#pragma unroll
            for (int j = 0; j < 4; ++j) {
                const double send = up8 ? a[j] : a[j + 4];
                const double keep = up8 ? a[j + 4] : a[j];
                a[j] = keep + lane_xor<3>(send);
            }
#pragma unroll
            for (int j = 0; j < 2; ++j) {
                const double send = up4 ? a[j] : a[j + 2];
                const double keep = up4 ? a[j + 2] : a[j];
                a[j] = keep + lane_xor<2>(send);
            }
            {
                const double send = up2 ? a[0] : a[1];
                const double keep = up2 ? a[1] : a[0];
                a[0] = keep + lane_xor<1>(send);
            }
        }
        a[0] += lane_xor<0>(a[0]);
        if (writer) {
            const float g = (float)a[0];
            if (emit) g_out[p0 + kw] = g;
            else L.vals[p0 + kw] = (float)((double)w_old - dlr * (double)g);
        }
    }
  }
}

// ---------------------------------------------------------------------------
// K4b: the descent step when the fused backward kernels have left the gradient of the stored
// entries in G[0] (and G[1], the other half of the batch): vals -= lr * g, a flat streaming pass
// over the entries of every layer (grid = (chunks of entries, layers)); k_apply_bias forms the bias
// gradient sum_s Delta(row, s).
// ---------------------------------------------------------------------------
// GRAD: no step, the gradient itself goes that way, through G[1] instead of mid (n_parts == 1: nothing else uses it).
template <bool GRAD>
__global__ void __launch_bounds__(TR_THREADS) k_apply(const LayerDev *__restrict__ layers, int n_parts, float lr)
{
    // The gradient and one copy of the values are in the order of the transposed index: this pass is a stream over
    // both.  The new values also go to `mid`, grouped by the chunk of the CSR array they belong to: a workgroup
    // takes a span of TR_SPAN consecutive entries, puts the new values into the order they have in mid in LDS
    // (mid_slot) and stores them from there, neighbouring threads into neighbouring places of a run (mid_dst).
    // k_spread_vals then fills the CSR copy, which the forward pass reads, chunk by chunk.  The workgroups of
    // one XCD take neighbouring spans, so that the pieces of a cache line of mid meet in one L2.
    __shared__ __attribute__((aligned(16))) float stage[TR_SPAN];
    const LayerDev &L = layers[blockIdx.y];
    const int nb = (int)gridDim.x; // a multiple of 8
    const int vb = ((int)blockIdx.x & 7) * (nb >> 3) + ((int)blockIdx.x >> 3);
    const int64_t q0 = (int64_t)vb * TR_SPAN;
    if (q0 >= L.nnz) return;
    const int cnt = (int)min((int64_t)TR_SPAN, (int64_t)L.nnz - q0), cnt4 = cnt >> 2;
    const double dlr = (double)lr;
    const float *__restrict__ g0 = L.G[0] + q0;
    const float *__restrict__ g1 = L.G[1] + q0;
    const uint16_t *__restrict__ slot = L.mid_slot + q0;
    const int32_t *__restrict__ dst = L.mid_dst + q0;
    float *__restrict__ vals_t = L.vals_t + q0;
    float *__restrict__ mid = GRAD ? L.G[1] : L.mid;
    const int tid = (int)threadIdx.x;
#define APPLY_ONE(G0, G1, W) (float)((double)(W) - dlr * (double)(float)(n_parts == 2 ? (double)(G0) + (double)(G1) : (double)(G0)))
    for (int k = tid; k < cnt4; k += TR_THREADS) { // q0 is a multiple of 4 and the arrays are 16-byte aligned
        const float4 a = reinterpret_cast<const float4 *>(g0)[k];
        const ushort4 o = reinterpret_cast<const ushort4 *>(slot)[k];
        float4 w = a;
        if constexpr (!GRAD) {
            float4 b = make_float4(0.0f, 0.0f, 0.0f, 0.0f);
            if (n_parts == 2) b = reinterpret_cast<const float4 *>(g1)[k];
            w = reinterpret_cast<const float4 *>(vals_t)[k];
            w.x = APPLY_ONE(a.x, b.x, w.x); w.y = APPLY_ONE(a.y, b.y, w.y);
            w.z = APPLY_ONE(a.z, b.z, w.z); w.w = APPLY_ONE(a.w, b.w, w.w);
            reinterpret_cast<float4 *>(vals_t)[k] = w;
        }
        stage[o.x] = w.x; stage[o.y] = w.y; stage[o.z] = w.z; stage[o.w] = w.w;
    }
    if (tid < (cnt & 3)) {
        const int k = 4 * cnt4 + tid;
        float w = g0[k];
        if constexpr (!GRAD) {
            w = APPLY_ONE(w, n_parts == 2 ? g1[k] : 0.0f, vals_t[k]);
            vals_t[k] = w;
        }
        stage[slot[k]] = w;
    }
#undef APPLY_ONE
    __syncthreads();
    for (int k = tid; k < cnt; k += TR_THREADS) mid[dst[k]] = stage[k];
}

// Chunk c of the CSR values from entries [c TR_CHUNK, (c+1) TR_CHUNK) of mid: placed in LDS by mid_loc, then
// written out in order.  grid = (chunks, layers).  GRAD: chunk c of the gradient `g` of one layer, from G[1].
template <bool GRAD>
__global__ void __launch_bounds__(TR_THREADS) k_spread_vals(const LayerDev *__restrict__ layers, float *__restrict__ g)
{
    __shared__ __attribute__((aligned(16))) float chunk[TR_CHUNK];
    const LayerDev &L = layers[blockIdx.y];
    const int64_t c0 = (int64_t)blockIdx.x * TR_CHUNK;
    if (c0 >= L.nnz) return;
    const int cnt = (int)min((int64_t)TR_CHUNK, (int64_t)L.nnz - c0), cnt4 = cnt >> 2;
    const float *__restrict__ mid = (GRAD ? L.G[1] : L.mid) + c0;
    const uint16_t *__restrict__ loc = L.mid_loc + c0;
    float *__restrict__ vals = (GRAD ? g : L.vals) + c0;
    for (int k = (int)threadIdx.x; k < cnt4; k += TR_THREADS) { // c0 is a multiple of 4 and the arrays are 16-byte aligned
        const float4 v = reinterpret_cast<const float4 *>(mid)[k];
        const ushort4 o = reinterpret_cast<const ushort4 *>(loc)[k];
        chunk[o.x] = v.x; chunk[o.y] = v.y; chunk[o.z] = v.z; chunk[o.w] = v.w;
    }
    if ((int)threadIdx.x < (cnt & 3)) chunk[loc[4 * cnt4 + (int)threadIdx.x]] = mid[4 * cnt4 + (int)threadIdx.x];
    __syncthreads();
    if (GRAD && ((size_t)g & 15) != 0) { // the caller's array
        for (int k = (int)threadIdx.x; k < cnt; k += TR_THREADS) vals[k] = chunk[k];
        return;
    }
    for (int k = (int)threadIdx.x; k < cnt4; k += TR_THREADS)
        reinterpret_cast<float4 *>(vals)[k] = reinterpret_cast<const float4 *>(chunk)[k];
    if ((int)threadIdx.x < (cnt & 3)) vals[4 * cnt4 + (int)threadIdx.x] = chunk[4 * cnt4 + (int)threadIdx.x];
}

// The gradient that k_apply applies, for inspection, in CSR order: out[t_perm[q]] = g0[q] (+ g1[q]), the same
// rounding as in k_apply.
__global__ void __launch_bounds__(256) k_sum_parts(const float *__restrict__ g0, const float *__restrict__ g1,
                                                   const int32_t *__restrict__ perm, float *__restrict__ out, int n)
{
    for (int q = blockIdx.x * 256 + threadIdx.x; q < n; q += gridDim.x * 256) {
        double g = (double)g0[q];
        if (g1) g += (double)g1[q];
        out[perm[q]] = (float)g;
    }
}

// vals_t[q] = vals[t_perm[q]]: brings the transposed-order copy of the values up to date after the CSR copy
// was changed by something other than k_apply (sdnn_set_weights, the separate update kernel).
__global__ void __launch_bounds__(256) k_refresh_vals_t(const LayerDev *__restrict__ layers)
{
    const LayerDev &L = layers[blockIdx.y];
    if (!L.vals_t) return;
    for (int q = blockIdx.x * 256 + threadIdx.x; q < L.nnz; q += gridDim.x * 256) L.vals_t[q] = L.vals[L.t_perm[q]];
}

// 16 lanes per row, four rows per wavefront at a time, 16 consecutive rows per wavefront.
// gb_out == NULL: bias -= lr * gb; otherwise the bias gradient of the one layer is stored there instead.
__global__ void __launch_bounds__(BLOCK_THREADS) k_apply_bias(const LayerDev *__restrict__ layers, int B, int ld, float lr,
                                                              float *__restrict__ gb_out)
{
    const LayerDev &L = layers[blockIdx.y];
    const int lane = threadIdx.x & 63, l = lane & 15;
    const int row0 = (blockIdx.x * WAVES_PER_BLOCK + (threadIdx.x >> 6)) * 16 + (lane >> 4);
    const bool vec = (ld & 3) == 0; // rows of Delta are 16-byte aligned; columns past B are zero
    for (int k = 0; k < 4; ++k) {
        const int row = row0 + 4 * k;
        double sum = 0.0;
        if (row < L.n_out) {
            const float *drow = L.D + (size_t)row * ld;
            if (vec) {
                for (int s = 4 * l; s < B; s += 64) {
                    const float4 d = *reinterpret_cast<const float4 *>(drow + s);
                    sum += (double)d.x; sum += (double)d.y; sum += (double)d.z; sum += (double)d.w;
                }
            } else {
                for (int s = l; s < B; s += 16) sum += (double)drow[s];
            }
        }
#pragma unroll
        for (int off = 8; off >= 1; off >>= 1) sum += __shfl_xor(sum, off);
        if (l == 0 && row < L.n_out) {
            if (gb_out) gb_out[row] = (float)sum;
            else L.bias[row] = (float)((double)L.bias[row] - (double)lr * (double)(float)sum);
        }
    }
}

// ---------------------------------------------------------------------------
// Inference that drops dead samples.  With ReLU and biases <= 0 a sample whose activations are all
// zero after some layer stays all zero in every later layer, so its column need not be computed any
// more.  Every few layers the live columns of the activation block are moved to the front (in
// order) and the product kernels are told how many columns still matter; the count lives in device
// memory, so nothing waits for the host.  map[c] remembers which sample sits in column c.
// ---------------------------------------------------------------------------
#define LIVE_ROWS 64  // rows per workgroup of the final scatter
#define PACK_ROWS 16  // rows per workgroup of k_pack
#define PACK_MAX_B 8192

// map = identity, both flag arrays cleared, n_live = B
__global__ void __launch_bounds__(256) k_skip_init(int32_t *__restrict__ map, int32_t *__restrict__ flags0,
                                                   int32_t *__restrict__ flags1, int32_t *__restrict__ n_live, int B)
{
    for (int s = blockIdx.x * 256 + threadIdx.x; s < B; s += gridDim.x * 256) { map[s] = s; flags0[s] = 0; flags1[s] = 0; }
    if (blockIdx.x == 0 && threadIdx.x == 0) *n_live = B;
}

// Packs the flagged columns of X [n_rows][ld] to the front, in order and in place.  Every workgroup
// derives the new position of each column from the flags by itself (a prefix sum over at most
// PACK_MAX_B flags) and then moves its own rows: a wavefront walks a row in chunks of 64 columns,
// front to back; a chunk is read completely before any of it is written and lands at or before its
// own place, so nothing unread is overwritten.  Workgroup 0 also writes the state of the next
// round, which nobody reads during this launch: the sample ids of the packed columns, the new
// count, and a cleared flag array.  If no column died nothing moves.
__global__ void __launch_bounds__(256) k_pack(float *X, int n_rows, int ld, const int32_t *__restrict__ flags,
                                              const int32_t *__restrict__ n_live_in, const int32_t *__restrict__ map_in,
                                              int32_t *__restrict__ n_live_out, int32_t *__restrict__ map_out,
                                              int32_t *__restrict__ flags_next)
{
    __shared__ int32_t newpos[PACK_MAX_B];
    __shared__ int wave_sum[4];
    const int t = threadIdx.x, lane = t & 63, wave = t >> 6;
    const int nl = *n_live_in;
    const int per = (nl + 255) / 256;
    const int c0 = min(t * per, nl), c1 = min(c0 + per, nl);
    int cnt = 0;
    for (int c = c0; c < c1; ++c) cnt += flags[c] != 0;
    int x = cnt; // inclusive prefix sum over the 256 threads
    for (int off = 1; off < 64; off <<= 1) {
        const int y = __shfl_up(x, off);
        if (lane >= off) x += y;
    }
    if (lane == 63) wave_sum[wave] = x;
    __syncthreads();
    int before = 0, nl_new = 0;
    for (int w = 0; w < 4; ++w) {
        const int v = wave_sum[w];
        if (w < wave) before += v;
        nl_new += v;
    }
    int pos = before + x - cnt;
    for (int c = c0; c < c1; ++c) newpos[c] = flags[c] != 0 ? pos++ : -1;
    __syncthreads();
    if (blockIdx.x == 0) {
        for (int c = c0; c < c1; ++c)
            if (newpos[c] >= 0) map_out[newpos[c]] = map_in[c];
        for (int c = t; c < ld; c += 256) flags_next[c] = 0;
        if (t == 0) *n_live_out = nl_new;
    }
    if (nl_new == nl) return;
    const int r_end = min(n_rows, ((int)blockIdx.x + 1) * PACK_ROWS);
    for (int r = (int)blockIdx.x * PACK_ROWS + wave; r < r_end; r += 4) {
        float *row = X + (size_t)r * ld;
        for (int cb = 0; cb < nl; cb += 64) {
            const int c = cb + lane;
            int np = -1;
            float v = 0.0f;
            if (c < nl) { np = newpos[c]; v = row[c]; }
            wave_lds_sync(); // every lane has read its column before any lane overwrites one
            if (np >= 0) row[np] = v;
        }
    }
}

// XL[r][map[c]] = X[r][c] for c < n_live (the other columns of XL were zeroed before)
__global__ void __launch_bounds__(256) k_scatter_cols(const float *__restrict__ X, float *__restrict__ XL, int n,
                                                      int ld, const int32_t *__restrict__ map,
                                                      const int32_t *__restrict__ n_live)
{
    const int c = blockIdx.x * 256 + threadIdx.x;
    if (c >= *n_live) return;
    const int dc = map[c];
    const int r0 = blockIdx.y * LIVE_ROWS, r1 = min(n, r0 + LIVE_ROWS);
    for (int r = r0; r < r1; ++r) XL[(size_t)r * ld + dc] = X[(size_t)r * ld + c];
}

__global__ void __launch_bounds__(256) k_fill_f32(float *__restrict__ p, size_t n, float v)
{
    for (size_t e = (size_t)blockIdx.x * blockDim.x + threadIdx.x; e < n; e += (size_t)gridDim.x * blockDim.x) p[e] = v;
}

// ---------------------------------------------------------------------------
// Measurement aid: the ceiling of the gather path.  Every wavefront streams per_wave gathers of
// random rows (64 * V floats, one V-float piece per lane, through the same buffer loads as the
// product kernels) from a table, 8 in flight, and does nothing else with them.  What this reaches for
// a table of a given size is what the product kernels can reach at best for an operand of that size.
// ---------------------------------------------------------------------------
template <int V>
__global__ void __launch_bounds__(BLOCK_THREADS) k_gather_probe(const int32_t *__restrict__ idx, const float *__restrict__ table,
                                                                size_t table_bytes, int per_wave, float *__restrict__ out)
{
    const int lane = threadIdx.x & 63;
    const size_t wave = (size_t)blockIdx.x * WAVES_PER_BLOCK + (threadIdx.x >> 6);
    const int32_t *my = idx + wave * (size_t)per_wave;
    const __amdgpu_buffer_rsrc_t r = make_rsrc(table, table_bytes);
    const unsigned so = 4u * (unsigned)(lane * V), ldb = 4u * 64u * V;
    float sum = 0.0f;
    for (int base = 0; base < per_wave; base += 64) {
        const int c_l = base + lane < per_wave ? my[base + lane] : 0;
        const int n = min(64, per_wave - base);
        for (int g = 0; g + 8 <= n; g += 8) {
            float x[8][V];
#pragma unroll
            for (int k = 0; k < 8; ++k) gatherv<V>(r, so, (unsigned)__builtin_amdgcn_readlane(c_l, g + k) * ldb, x[k]);
#pragma unroll
            for (int k = 0; k < 8; ++k)
#pragma unroll
                for (int v = 0; v < V; ++v) sum += x[k][v];
        }
    }
    out[wave * 64 + lane] = sum;
}

// ---------------------------------------------------------------------------
// loss-gradient helpers
// ---------------------------------------------------------------------------
__global__ void __launch_bounds__(256) k_mse_dloss(const float *__restrict__ x,
                                                   const float *__restrict__ y,
                                                   float *__restrict__ out, size_t n, double B)
{
    for (size_t e = (size_t)blockIdx.x * blockDim.x + threadIdx.x; e < n;
         e += (size_t)gridDim.x * blockDim.x)
        out[e] = (float)(((double)x[e] - (double)y[e]) / B);
}

__global__ void __launch_bounds__(256) k_softmax_ce_dloss(const float *__restrict__ x,
                                                          const int32_t *__restrict__ labels,
                                                          float *__restrict__ out, int n, int B,
                                                          int n_classes)
{
    const int first = n - n_classes;
    // zero the rows that carry no logit
    for (size_t e = (size_t)blockIdx.x * blockDim.x + threadIdx.x; e < (size_t)first * B;
         e += (size_t)gridDim.x * blockDim.x)
        out[e] = 0.0f;
    for (int s = blockIdx.x * blockDim.x + threadIdx.x; s < B; s += gridDim.x * blockDim.x) {
        double m = -INFINITY;
        for (int c = 0; c < n_classes; ++c) m = fmax(m, (double)x[(size_t)(first + c) * B + s]);
        double z = 0.0;
        for (int c = 0; c < n_classes; ++c) z += exp((double)x[(size_t)(first + c) * B + s] - m);
        const int lab = labels[s];
        for (int c = 0; c < n_classes; ++c) {
            double pr = exp((double)x[(size_t)(first + c) * B + s] - m) / z;
            if (c == lab) pr -= 1.0;
            out[(size_t)(first + c) * B + s] = (float)(pr / (double)B);
        }
    }
}

// ---------------------------------------------------------------------------
// host side
// ---------------------------------------------------------------------------
enum { ST_IDLE = 0, ST_FORWARD = 1, ST_BACKWARD = 2 };

struct sdnn_net {
    int32_t n_layers = 0;
    sdnn_config cfg{};
    std::vector<LayerDev> layers; // host copy of the descriptors (device pointers inside)
    LayerDev *d_layers = nullptr; // device copy
    float *d_x0 = nullptr;        // training: X_0 [n_in(1)][max_batch]
    float *d_ping = nullptr, *d_pong = nullptr; // inference: two activation buffers
    int n_cu = 0;                 // compute units of the device
    int occ_spmm[2][3][2][2] = {}; // resident workgroups per CU of k_spmm<V,MODE,U,tiles inner>, U = 8, 16
    int occ_grad = 0;             // the same for k_bwd_grad
    bool b1_attr_set = false;
    bool b1 = false, b1_wide = false; // made for one sample per step: lane-major copies of W and W^T; with 4-byte columns
    int occ_panel[2][4] = {};     // the same for k_spmm_panel<R,MODE>, R = 1, 2, 4, 8
    std::vector<int32_t> max_len[2]; // per layer: longest row of W (0) and of W^T (1)
    std::vector<char> grad_spread;   // per layer: sdnn_weight_grad in two passes, where one partial gradient holds it
    std::vector<char> clustered[2];  // per layer: reorder_rows found clusters in W (0), in W^T (1)
    uint4 *lm = nullptr;             // lane-major copy of W for k_fwd_lds, NULL: there is none
    int32_t *lm_cs = nullptr, *lm_row = nullptr;
    float *lm_bias = nullptr;
    LmLayer *lm_layers = nullptr;
    std::vector<LmLayer> lm_tab;     // host copy of lm_layers
    size_t lm_chunks = 0;
    int32_t lm_max_pos = 0, lm_two = 0; // see LdsForward
    int32_t turns = 0;               // lm_turns of three quarters of its chunks and more
    bool lds_part_attr_set = false;
    struct Train {                   // a copy of W (0) or W^T (1) for k_train_lds
        std::vector<LmLayer> tab;    // empty: there is none
        LmLayer *d_tab = nullptr;
        int32_t *cs = nullptr, *row = nullptr, *pos = nullptr, *first = nullptr;
        uint4 *lm = nullptr;
        float *bias = nullptr, *out = nullptr;
        size_t chunks = 0;
        int32_t max_nb = 0;
    } train[2];
    // seconds that both passes take with a launch per layer, their gathers of one sample, those with a single launch, and what is
    // added where the samples leave no compute unit idle (train_lds_pays)
    double train_per_layer = 0, train_gathers = 0, train_single = 0, train_cold = 0;
    bool train_stale = false;     // the values were stepped or replaced and the copies did not follow
    bool train_replaced = false;  // a layer's values were replaced since the last pass that reads the copies
    bool train_kept = false;      // a captured graph reads the copies: they always follow
    bool long_lm = false, long_attr_set = false; // copies of W for k_fwd_long
    std::vector<uint32_t> long_bytes;            // their sizes
    bool long_even = true;                       // every layer has a block for each wavefront, none with more than an eighth of its halves
    std::vector<char> long_stale;                // per layer: as train_stale
    bool long_kept = false;                      // as train_kept
    bool pan_attr_set = false;
    struct Pan {                     // a layer's copy of W for k_fwd_pan
        PanLayer g{};
        uint4 *stream = nullptr;
        int32_t *seg = nullptr, *slot = nullptr, *rows = nullptr, *pos = nullptr;
        uint32_t *ends = nullptr;
        float *bias = nullptr;
        double depth = 0;
    };
    std::vector<Pan> pan;            // empty: the net has no such copy
    bool lds_attr_set[3] = {};       // the dynamic LDS limit of k_fwd_lds<1 << k> has been raised
    int grad_parts = 0;           // > 0: the last backward pass left the entries' gradient in G[0..grad_parts)
    bool two_windows = false;     // that gradient is the sum of two rounded windows of samples
    bool vals_t_stale = false;    // the CSR values were changed by something that does not maintain vals_t
    int32_t *d_alive = nullptr;
    int32_t *d_flags[2] = {nullptr, nullptr}, *d_map[2] = {nullptr, nullptr}, *d_n_live[2] = {nullptr, nullptr}; // inference: dead-sample skipping, two rounds' state
    bool bias_nonpos = false;     // every bias of layers 2..L is <= 0 (as uploaded; cleared when a bias is replaced)
    int state = ST_IDLE;
    int32_t B = 0;                // samples of the last forward pass
    int32_t Bp = 0, ld = 0;       // training: samples the kernels work on (padded_batch) and floats per row of X_l, Delta_l
    int32_t max_n = 0;
    char err[512] = "";
};

static int fail(sdnn_net *net, int code, const char *fmt, ...)
{
    char buf[512];
    va_list ap;
    va_start(ap, fmt);
    vsnprintf(buf, sizeof buf, fmt, ap);
    va_end(ap);
    if (net) snprintf(net->err, sizeof net->err, "%s", buf);
    sdnn_set_global_error("%s", buf);
    return code;
}

#define HIP_TRY(net, expr)                                                                   \
    do {                                                                                     \
        hipError_t e_ = (expr);                                                              \
        if (e_ != hipSuccess)                                                                \
            return fail(net, SDNN_EHIP, "%s: %s", #expr, hipGetErrorString(e_));              \
    } while (0)

extern "C" const char *sdnn_last_error(const sdnn_net *net)
{
    return net ? net->err : sdnn_global_error();
}

// Fixed staging array of sdnn_forward_noalloc (the variant of sdnn_forward for callers that cannot
// allocate): it lives in the library's device image, one copy per GPU, until the process ends.
static __device__ __align__(256) unsigned char scratch[SDNN_NOALLOC_SCRATCH_BYTES];
#define MAX_DEVICES 64
static void *g_scratch_ptr[MAX_DEVICES]; // device address of `scratch` on each GPU, looked up once per GPU
static std::mutex g_scratch_mutex;

// Address of this GPU's copy of the array (the array's name is only a host-side handle of the
// symbol: kernels and copies must be given the address that the runtime reports).
static int scratch_address(sdnn_net *net, void **ptr)
{
    int devid = -1;
    HIP_TRY(net, hipGetDevice(&devid));
    if (devid < 0 || devid >= MAX_DEVICES) return fail(net, SDNN_EINVAL, "device %d: more GPUs than supported", devid);
    std::lock_guard<std::mutex> lock(g_scratch_mutex);
    if (!g_scratch_ptr[devid]) {
        void *p = nullptr;
        HIP_TRY(net, hipGetSymbolAddress(&p, HIP_SYMBOL(scratch)));
        if (!p) return fail(net, SDNN_EHIP, "hipGetSymbolAddress returned NULL");
        g_scratch_ptr[devid] = p;
    }
    *ptr = g_scratch_ptr[devid];
    return SDNN_OK;
}

static inline size_t align_up(size_t x) { return (x + 255) & ~(size_t)255; }

// Workspace plan: offsets of every array, in one pass (also used to size it).
struct Plan {
    struct PerLayer {
        size_t row_ptr, col_idx, vals, bias, t_row_ptr, t_row_idx, t_perm, sched, t_sched, X, D, G[2], vals_t, mid_slot, mid_dst, mid_loc, mid, b1_cs[2], b1_row[2], b1_lm[2];
        int32_t b1_blocks[2];
        size_t b1_chunks[2];
        PanLayer pan;
        size_t pan_stream, pan_seg, pan_slot, pan_rows, pan_pos, pan_ends, pan_bias;
    };
    bool pan = false;            // a copy of W for k_fwd_pan
    struct Train {               // the copies of W and W^T for k_train_lds
        std::vector<LmLayer> tab;
        size_t n_cs = 0, n_pos = 0, n_rows = 0, n_chunks = 0, d_tab = 0, cs = 0, row = 0, pos = 0, first = 0, lm = 0, bias = 0, out = 0;
    } train[2];
    bool train_lds = false;
    bool long_lm = false;        // copies of W for k_fwd_long (in the places of b1_*[0])
    std::vector<PerLayer> pl;
    size_t b1_chunk_bytes = 0;   // 0: no lane-major copies for one sample per step
    std::vector<LmLayer> lm_tab; // empty: no lane-major copy
    size_t lm_n_chunks = 0, lm_n_cs = 0, lm_n_pos = 0, lm_n_rows = 0; // sizes of its arrays, all layers together
    size_t lm = 0, lm_cs = 0, lm_layers = 0, lm_row = 0, lm_bias = 0, lm_pos = 0;
    size_t table = 0, x0 = 0, ping = 0, pong = 0, alive = 0, flags[2] = {0, 0}, map[2] = {0, 0}, n_live[2] = {0, 0}, total = 0;
};

// Samples that the kernels of a training net work on for a batch of B: whole groups of four.  The samples past B are zero
// in every X_l and Delta_l (the kernels store zeros for them: what a zero input turns into on its way may be infinite), so
// that they add exact zeros to every gradient.
static int padded_batch(int B) { return B == 1 ? 1 : (B + 3) & ~3; }
// Floats per row of the library's own activation and delta arrays: 16-byte pieces stay aligned, a row touches as few
// 128-byte lines as it can.
static int row_stride(int B)
{
    if (B == 1) return 1;
    for (int w = 4; w <= 32; w *= 2)
        if (B <= w) return w;
    return (B + 31) & ~31;
}
// The same on a net whose widest layer has max_n neurons: where the filled-up rows would make a block of 4 GiB or more, which
// the products refuse, rows of whole groups of four samples, or else of B floats (kernels without wide loads).
static int row_pitch(int64_t max_n, int B)
{
    for (const int w : {row_stride(B), padded_batch(B)})
        if (4 * max_n * w < ((int64_t)1 << 32)) return w;
    return B;
}

static int check_config(const sdnn_layer *layers, int32_t n_layers, const sdnn_config *cfg)
{
    if (!layers || !cfg) return fail(nullptr, SDNN_EINVAL, "layers or cfg is NULL");
    if (n_layers < 1) return fail(nullptr, SDNN_EINVAL, "n_layers must be >= 1");
    if (cfg->max_batch < 1) return fail(nullptr, SDNN_EINVAL, "max_batch must be >= 1");
    if (cfg->activation != SDNN_ACT_RELU_CAP && cfg->activation != SDNN_ACT_SIGMOID)
        return fail(nullptr, SDNN_EINVAL, "unknown activation %d", cfg->activation);
    if (cfg->activation == SDNN_ACT_RELU_CAP && !(cfg->act_cap > 0.0f))
        return fail(nullptr, SDNN_EINVAL, "act_cap must be > 0 (or +inf)");
    if (cfg->fuse_gradient < SDNN_FUSE_OFF || cfg->fuse_gradient > SDNN_FUSE_ON)
        return fail(nullptr, SDNN_EINVAL, "unknown fuse_gradient %d", cfg->fuse_gradient);
    if (cfg->panel_cols < SDNN_PANEL_OFF) return fail(nullptr, SDNN_EINVAL, "panel_cols must be >= -1");
    if (cfg->reorder_rows != 0 && cfg->reorder_rows != 1) return fail(nullptr, SDNN_EINVAL, "reorder_rows must be 0 or 1");
    if (cfg->lds_forward < SDNN_LDS_OFF || cfg->lds_forward > SDNN_LDS_ON)
        return fail(nullptr, SDNN_EINVAL, "unknown lds_forward %d", cfg->lds_forward);
    for (int32_t l = 0; l < n_layers; ++l) {
        const sdnn_layer &y = layers[l];
        if (y.n_out < 0 || y.n_in < 0 || !y.row_ptr)
            return fail(nullptr, SDNN_EINVAL, "layer %d: bad size or NULL row_ptr", l + 1);
        if (l > 0 && y.n_in != layers[l - 1].n_out)
            return fail(nullptr, SDNN_EINVAL, "layer %d: n_in %d != n_out %d of layer %d", l + 1,
                        y.n_in, layers[l - 1].n_out, l);
        if ((int64_t)y.n_out * cfg->max_batch >= ((int64_t)1 << 40))
            return fail(nullptr, SDNN_EINVAL, "layer %d: activation block too large", l + 1);
    }
    return SDNN_OK;
}

// The fused backward + gradient kernels pay where launches are bound by gather throughput; where their latency binds,
// the separate update is faster (measured, backward + update per layer, separate / fused: 2048 neurons of 32 entries,
// 64 samples 7.3 / 7.7 us, 99 samples 9.7 / 8.8; 1024 neurons, 99 samples 7.6 / 8.6, 200 samples 10.3 / 8.5; 4096 neurons, 64
// samples 9.9 / 8.4; 2048 neurons of 205 entries, 64 samples 24 / 28 us, 256 samples 43 / 33).  AUTO decides by the entries per layer and by whether the net is made for more than 64 samples.
static bool grad_buffers_wanted(const sdnn_layer *layers, int32_t n_layers, const sdnn_config *cfg)
{
    if (!cfg->training || cfg->fuse_gradient == SDNN_FUSE_OFF || cfg->max_batch == 1) return false;
    if (cfg->fuse_gradient == SDNN_FUSE_ON) return true;
    int64_t nnz = 0, rows = 0;
    for (int32_t l = 0; l < n_layers; ++l) {
        rows += layers[l].n_out;
        nnz += layers[l].row_ptr ? layers[l].row_ptr[layers[l].n_out] : 0;
    }
    if (cfg->max_batch > 256 && nnz >= 128 * rows) return false; // batches that wide take the separate kernels
    if (cfg->max_batch > 64) return nnz >= (int64_t)48000 * n_layers;
    return nnz >= (int64_t)85000 * n_layers && (nnz < 128 * rows || rows >= (int64_t)4096 * n_layers); // few long rows: too few wavefronts
}

// Chunks of a layer's lane-major copy: its rows, longest first, in blocks of 64, each as deep as its first row.
static size_t lm_chunks(const sdnn_layer &y, size_t per = LDS_CHUNK)
{
    std::vector<int32_t> rows_of_len; // a histogram is enough: the first rows of the blocks are rows 0, 64, 128, ... by length
    for (int32_t r = 0; r < y.n_out; ++r) {
        const size_t len = (size_t)(y.row_ptr[r + 1] - y.row_ptr[r]);
        if (len >= rows_of_len.size()) rows_of_len.resize(len + 1, 0);
        rows_of_len[len]++;
    }
    size_t total = 0;
    int64_t before = 0; // rows longer than len
    for (size_t len = rows_of_len.size(); len-- > 0;) {
        const int64_t after = before + rows_of_len[len];
        const int64_t firsts = (after + 63) / 64 - (before + 63) / 64; // multiples of 64 in [before, after)
        total += (size_t)firsts * ((len + per - 1) / per);
        before = after;
    }
    return total;
}

// The LDS-resident forward (k_fwd_lds) carries samples through all layers with their activations in LDS; it is set up
// for inference nets whose widest layer fits with at least one sample.
static bool lds_forward_wanted(const sdnn_layer *layers, int32_t n_layers, const sdnn_config *cfg)
{
    if (cfg->training || cfg->lds_forward == SDNN_LDS_OFF) return false;
    size_t chunks = 1;
    for (int32_t l = 0; l < n_layers; ++l) {
        if (layers[l].n_out > LDS_MAX_FLOATS || layers[l].n_in > LDS_MAX_FLOATS) return false;
        chunks += lm_chunks(layers[l]);
    }
    return chunks * LDS_CHUNK_BYTES < ((size_t)1 << 32); // the kernel addresses the copy with 32-bit offsets
}

// One layer's blocks dealt to the wavefronts: the deepest first, each to the wavefront with the fewest chunks so far that
// has room (at most tab.nb blocks each).  Fills the layer's part of the row table (row[position], -1 where there is none),
// of the position table (pos[row]) and of the chunk table, the latter with the blocks' depths for now.
static void lm_deal_blocks(const sdnn_layer &y, const LmLayer &tab, int32_t *row, int32_t *pos, int32_t *cs)
{
    std::vector<int32_t> order((size_t)y.n_out);
    sdnn_row_schedule(y.n_out, y.row_ptr, order.data());
    std::fill(row, row + tab.n_pos, -1);
    std::fill(cs, cs + LDS_WAVES * (tab.nb + 1), 0);
    int32_t load[LDS_WAVES] = {}, used[LDS_WAVES] = {};
    for (int32_t r0 = 0; r0 < y.n_out; r0 += 64) {
        const int32_t depth = (y.row_ptr[order[r0] + 1] - y.row_ptr[order[r0]] + LDS_CHUNK - 1) / LDS_CHUNK;
        int w = -1;
        for (int k = 0; k < LDS_WAVES; ++k)
            if (used[k] < tab.nb && (w < 0 || load[k] < load[w])) w = k;
        const int32_t j = used[w]++;
        load[w] += depth;
        cs[w * (tab.nb + 1) + j] = depth;
        for (int32_t k = 0; k < 64 && r0 + k < y.n_out; ++k) {
            const int32_t at = 64 * (LDS_WAVES * j + w) + k;
            row[at] = order[(size_t)(r0 + k)];
            pos[order[(size_t)(r0 + k)]] = at;
        }
    }
}

// With how many samples per workgroup (bits 1, 2 and 4) the wavefronts take turns at priority in a layer whose blocks have the
// depths that lm_deal_blocks left in cs: where their shares of the layer, in chunks, are about equal.  The first wavefronts have the
// deepest blocks and those left over; by age they are served first, and turns hold them up.  Later rounds of blocks make up for a
// share that is a little longer, with four samples sooner.  us per layer, 32 entries per row, by age / in turns, with 1, 2 and 4
// samples: 300 neurons (a round: nobody is later than the others) 1.55 / 1.66, 1.76 / 1.87, 2.38 / 2.55; 1089 (two rounds, the longest
// share 1.78 of the mean one) 2.88 / 3.28, 3.15 / 3.56, 4.82 / 5.08; 1792 (1.14) 3.74 / 3.80, 4.04 / 4.19, 6.07 / 6.23; 1856 (1.10)
// 4.01 / 3.89, 4.38 / 4.26, 6.65 / 6.31; 2112 (three rounds, 1.45) 4.66 / 4.91, 5.14 / 5.34, 7.87 / 7.58; 2432 (1.26) 5.02 / 5.06,
// 5.61 / 5.55, 8.60 / 8.26; 3136 (four, 1.31) 6.46 / 6.31, 7.27 / 6.99, 11.00 / 10.88.
// Not on rows of 28 chunks and more in the mean with one sample, nor, where all blocks are about as deep, with two: the workgroups of
// an XCD come apart in the stream of W by deep blocks, which its L2 then fetches again and again (820 entries per row, 8192 neurons,
// 220 and 500 samples 390 / 473, 477 / 570; a tenth of the columns with a heavy tail, 220 samples, 4097 neurons 92.3 / 87.5, 5000
// neurons 132 / 142, 6000 neurons 187 / 232, 8192 neurons 397 / 567; 500 samples, 8192 neurons 465 / 446).
// Nor with one sample on half of that in a layer of more than 12 MB (8192 neurons of 256 entries, 16 / 64 / 200 samples 125 / 116 / 110 by age,
// 127 / 117 / 113 in turns).
// LM_IN_ORDER: whether with one sample the loads of W are requested strictly in their order, as with more samples they always are.
// Without turns: with one round of blocks, and with short rows or fewer second blocks than SIMDs in two.  With turns: in up to three
// rounds, and where the layer is larger than an L2, whose misses hold up loads that are requested late (6 MB; it is 4 MB, shared).
// us per layer, 32 entries per row and 200 samples (else: entries x samples), in order / in the compiler's: by age 300 neurons 1.51 / 1.53 (64), 1300
// 3.08 / 3.13, 2112 4.89 / 4.81 (64); a tenth of the columns with a heavy tail, 64 samples 1024 neurons 7.85 / 8.24, 1180 9.51 / 9.65 (100),
// 1249 10.6 / 10.5, 2000 24.6 / 23.8, 6000 244 / 254; in turns 2048 neurons 5.10 / 5.13, x 64 8.16 / 8.18 (64), 3001 6.91 / 6.90, 4096 9.15 /
// 8.98, x 64 15.9 / 15.2 (64), x 128 28.3 / 27.1, 8192 16.4 / 16.2, x 64 29.0 / 28.6, x 128 55.0 / 57.1, 16384 31.7 / 31.3, x 128 117 / 138.
static int lm_turns(int32_t nb, const int32_t *cs)
{
    int64_t longest = 0, all = 0, blocks = 0, deepest = 0;
    for (int w = 0; w < LDS_WAVES; ++w) {
        int64_t share = 0;
        for (int32_t j = 0; j < nb; ++j) {
            const int64_t depth = cs[w * (nb + 1) + j];
            share += depth;
            blocks += depth > 0;
            deepest = std::max(deepest, depth);
        }
        longest = std::max(longest, share);
        all += share;
    }
    const bool equal = (double)longest * LDS_WAVES <= (1.0 + 0.13 * (nb - 1)) * (double)all, deep = all >= 28 * blocks;
    const bool deep_1 = deep || (all >= 14 * blocks && all * LDS_CHUNK_BYTES > 12000000), beyond_l2 = all * LDS_CHUNK_BYTES > 6000000;
    const bool in_turns = nb > 1 && equal && !deep_1;
    const bool in_order = in_turns ? nb <= 3 || beyond_l2 : nb == 1 || deep_1 || (nb == 2 && (all < 3 * blocks || blocks < LDS_WAVES + 4));
    const int order = in_order ? LM_IN_ORDER : 0;
    if (nb < 2) return order;
    return order | (in_turns ? 1 : 0) | (equal && !(deep && 2 * all > deepest * blocks) ? 2 : 0) | (equal || nb > 2 ? 4 : 0);
}

// Runs fn(0 .. n - 1) on up to 16 host threads (here if there are no more threads); fn must not throw.
template <class F> static void for_each_layer(int32_t n, F fn)
{
    const int32_t hw = (int32_t)std::max(1u, std::min(std::thread::hardware_concurrency(), 16u)), nt = std::min(n, hw);
    std::vector<std::thread> workers;
    auto work = [&](int32_t first) {
        for (int32_t l = first; l < n; l += nt) fn(l);
    };
    int32_t started = 1;
    for (; started < nt; ++started) {
        try {
            workers.emplace_back(work, started);
        } catch (...) {
            break;
        }
    }
    work(0);
    for (int32_t k = started; k < nt; ++k) work(k);
    for (std::thread &w : workers) w.join();
}

// Nets made for one sample per step take a lane per row over lane-major copies of W and W^T where no row is so long that its
// lane would run on by itself.  Chunks of eight entries of the rows, longest first, in blocks of 64; false: too long a row.
#define B1_MAX_ROW 512
static bool b1_chunks(const int32_t *len, int32_t n, size_t *chunks)
{
    int64_t rows_of_len[B1_MAX_ROW + 1] = {}, before = 0;
    for (int32_t r = 0; r < n; ++r) {
        if (len[r] > B1_MAX_ROW) return false;
        rows_of_len[len[r]]++;
    }
    *chunks = 0;
    for (int k = B1_MAX_ROW; k >= 0; --k) { // a block is as deep as its first row
        const int64_t after = before + rows_of_len[k];
        *chunks += (size_t)((after + 63) / 64 - (before + 63) / 64) * (size_t)((k + 7) / 8);
        before = after;
    }
    return true;
}
// At most as many chunks as b1_chunks counts for n rows of nnz entries together (none longer than B1_MAX_ROW, or it counts
// none): the first block is no deeper than the longest row that there can be, and every later one no deeper than the mean
// of the 64 rows before it.
static size_t b1_chunks_bound(int32_t n, int64_t nnz, int32_t longest)
{
    const int64_t nb = ((int64_t)n + 63) / 64;
    return (size_t)((std::min(longest, B1_MAX_ROW) + 7) / 8 + (nnz / 64 + 7 * nb) / 8 + 1);
}
// Fills the plan's chunk counts; leaves b1_chunk_bytes 0 where the net does not take that layout.  Without col_idx (only the
// sizes are asked for): a bound.
static void plan_b1(const sdnn_layer *layers, int32_t n_layers, const sdnn_config *cfg, Plan &pl)
{
    pl.b1_chunk_bytes = 0;
    if (!cfg->training || cfg->max_batch != 1) return;
    bool wide = false;
    for (int32_t l = 0; l < n_layers; ++l) {
        const sdnn_layer &y = layers[l];
        const int64_t nnz = y.row_ptr[y.n_out];
        if (nnz > ((int64_t)1 << 28) || y.n_out > (1 << 24) || y.n_in > (1 << 24)) return; // a copy stays below 4 GiB
        if (nnz >= 128 * (int64_t)std::max(y.n_out, 1) || nnz >= 128 * (int64_t)std::max(y.n_in, 1)) return;
        wide |= y.n_out > 65536 || y.n_in > 65536;
    }
    std::atomic<bool> fits(true);
    for_each_layer(n_layers, [&](int32_t l) {
        const sdnn_layer &y = layers[l];
        Plan::PerLayer &q = pl.pl[l];
        if (!fits) return;
        try {
            std::vector<int32_t> len((size_t)std::max(y.n_out, y.n_in));
            for (int32_t r = 0; r < y.n_out; ++r) len[(size_t)r] = y.row_ptr[r + 1] - y.row_ptr[r];
            if (!b1_chunks(len.data(), y.n_out, &q.b1_chunks[0])) { fits = false; return; }
            std::fill(len.begin(), len.end(), 0);
            const int32_t nnz = y.row_ptr[y.n_out];
            if (nnz > 0 && !y.col_idx) {
                q.b1_chunks[1] = b1_chunks_bound(y.n_in, nnz, y.n_out);
            } else {
                for (int32_t p = 0; p < nnz; ++p)
                    if ((uint32_t)y.col_idx[p] < (uint32_t)y.n_in) len[(size_t)y.col_idx[p]]++;
                if (!b1_chunks(len.data(), y.n_in, &q.b1_chunks[1])) { fits = false; return; }
            }
        } catch (...) {
            fits = false;
            return;
        }
        q.b1_blocks[0] = (y.n_out + 63) / 64;
        q.b1_blocks[1] = (y.n_in + 63) / 64;
    });
    if (fits) pl.b1_chunk_bytes = wide ? 4096 : 3072;
}

// Training with a launch per pass (k_train_lds): narrow nets of short rows, whose gradient is not formed in the backward sweep; four
// layers and more (a step launches two kernels more, to bring the copies up to date).
// Fills in the tables' sizes; the chunks are a bound, from the lengths of the rows of W alone (the columns may not be known here).
// W_L, by the length of its rows: as many as there are.  The other W follow the rows of the W^T above, in any order for all that
// is known here: no more than if every block had one of their longest rows.  W^T: its first block is no deeper than the most entries
// a column can have, every later one no deeper than the mean of the 64 rows before it.
#define TRAIN_LDS_MAX_ROW 512
static void plan_train(const sdnn_layer *layers, int32_t n_layers, const sdnn_config *cfg, Plan &pl)
{
    pl.train_lds = false;
    if (!cfg->training || cfg->max_batch < 2 || cfg->max_batch > 256 || n_layers < 4 || cfg->lds_forward == SDNN_LDS_OFF || cfg->panel_cols > 0 ||
        cfg->reorder_rows || grad_buffers_wanted(layers, n_layers, cfg))
        return;
    for (int32_t l = 0; l < n_layers; ++l) {
        const sdnn_layer &y = layers[l];
        if (y.n_out < 1 || y.n_in < 1 || y.n_out > TRAIN_LDS_POS || y.n_in > TRAIN_LDS_POS) return;
        for (int32_t r = 0; r < y.n_out; ++r)
            if (y.row_ptr[r + 1] - y.row_ptr[r] > TRAIN_LDS_MAX_ROW) return;
    }
    for (int o = 0; o < 2; ++o) {
        Plan::Train &t = pl.train[o];
        for (int32_t k = 0; k < n_layers - o; ++k) {
            const sdnn_layer &y = layers[o ? n_layers - 1 - k : k];
            const int32_t n = o ? y.n_in : y.n_out;
            LmLayer e;
            e.nb = (n + 64 * LDS_WAVES - 1) / (64 * LDS_WAVES);
            e.n_pos = 64 * LDS_WAVES * e.nb;
            e.cs = (int32_t)t.n_cs;
            e.pos = (int32_t)t.n_pos;
            t.tab.push_back(e);
            t.n_cs += (size_t)LDS_WAVES * (size_t)(e.nb + 1);
            t.n_pos += (size_t)e.n_pos;
            t.n_rows += (size_t)n;
            const size_t nnz = (size_t)y.row_ptr[y.n_out], blocks = ((size_t)n + 63) / 64;
            if (o) {
                t.n_chunks += (size_t)(std::min(y.n_out, TRAIN_LDS_MAX_ROW) + LDS_CHUNK - 1) / LDS_CHUNK + (nnz / 64 + (LDS_CHUNK - 1) * blocks) / LDS_CHUNK;
            } else if (k == n_layers - 1) {
                t.n_chunks += lm_chunks(y);
            } else {
                std::vector<int32_t> chunks((size_t)n);
                for (int32_t r = 0; r < n; ++r) chunks[(size_t)r] = (y.row_ptr[r + 1] - y.row_ptr[r] + LDS_CHUNK - 1) / LDS_CHUNK;
                std::partial_sort(chunks.begin(), chunks.begin() + (ptrdiff_t)blocks, chunks.end(), std::greater<int32_t>());
                for (size_t b = 0; b < blocks; ++b) t.n_chunks += (size_t)chunks[b];
            }
        }
        if (t.n_chunks * LDS_CHUNK_BYTES >= ((size_t)1 << 32)) return; // the kernel addresses a copy with 32-bit offsets
    }
    pl.train_lds = true;
}

// The copies for k_fwd_long: training nets of long rows whose operands fit its LDS, made for batches that take it (long_forward), with
// enough entries per layer to pay for bringing the copies up to date after a step (a step of two layers of 1000 neurons of 130 entries
// takes 77 us without them and 82 with).
static void plan_long(const sdnn_layer *layers, int32_t n_layers, const sdnn_config *cfg, Plan &pl)
{
    pl.long_lm = false;
    if (!cfg->training || cfg->max_batch < LONG_MIN_BATCH || cfg->lds_forward == SDNN_LDS_OFF || cfg->panel_cols > 0 || cfg->reorder_rows ||
        pl.train_lds)
        return;
    int64_t nnz = 0;
    for (int32_t l = 0; l < n_layers; ++l) {
        const sdnn_layer &y = layers[l];
        if (y.n_out < 1 || y.n_in < 1 || y.n_in > LONG_POS || (int64_t)y.row_ptr[y.n_out] < 128 * (int64_t)y.n_out) return;
        nnz += y.row_ptr[y.n_out];
    }
    if (nnz < (int64_t)150000 * n_layers) return;
    for (int32_t l = 0; l < n_layers; ++l) {
        Plan::PerLayer &q = pl.pl[l];
        q.b1_blocks[0] = (layers[l].n_out + 63) / 64;
        q.b1_chunks[0] = lm_chunks(layers[l], LDS_CHUNK / 2);
        if ((q.b1_chunks[0] + 2) * LDS_HALF_BYTES >= ((size_t)1 << 32) - 65536) { // the kernel addresses a copy with 32-bit offsets
            for (int32_t k = 0; k <= l; ++k) pl.pl[k].b1_blocks[0] = 0;
            return;
        }
    }
    pl.long_lm = true;
}

// The forward in panels (k_fwd_pan) is set up for inference nets wider than a panel, of at least three layers (the two passes that
// turn the samples around take about as long as a layer), with at least four entries per row and panel in the mean, made for
// batches that can fill the chip (pan_forward_pays); not where lds_forward = ON takes k_fwd_lds with every batch (`lm`: the net has its copy).
// Fills in the layers' geometry.
static bool pan_wanted(const sdnn_layer *layers, int32_t n_layers, const sdnn_config *cfg, bool lm, std::vector<Plan::PerLayer> &pl)
{
    if (lm && cfg->lds_forward == SDNN_LDS_ON) return false;
    if (cfg->training || cfg->lds_forward == SDNN_LDS_OFF || cfg->panel_cols > 0 || cfg->reorder_rows || n_layers < 3 || cfg->max_batch <= 64) return false;
    int64_t nnz = 0, rows = 0, widest = 0;
    for (int32_t l = 0; l < n_layers; ++l) {
        if (layers[l].n_out == 0 || layers[l].n_in == 0) return false;
        nnz += layers[l].row_ptr[layers[l].n_out];
        rows += layers[l].n_out;
        widest = std::max<int64_t>(widest, std::max(layers[l].n_out, layers[l].n_in));
    }
    const int64_t n_panels = (widest + PAN_POS - 1) / PAN_POS;
    if (n_panels < 2 || n_panels > PAN_MAX || nnz < 4 * rows * n_panels || cfg->max_batch * widest < 3200000) return false;
    for (int32_t l = 0; l < n_layers; ++l) {
        PanLayer &g = pl[l].pan;
        sdnn_pan_geometry(layers[l], l > 0 ? &pl[l - 1].pan : nullptr, g);
        if ((g.halves + 2) * LDS_HALF_BYTES >= ((size_t)1 << 32)) return false; // the kernel addresses a layer's copy with 32-bit offsets
    }
    return true;
}

static void make_plan(const sdnn_layer *layers, int32_t n_layers, const sdnn_config *cfg, Plan &pl)
{
    // Arrays of 1 MiB and more start on a multiple of their size rounded down to a power of two, at most
    // 2 MiB: where the gathered activation blocks lie relative to the 2 MiB granules of the address
    // translation is worth 9 % of the inference time on 16384-neuron layers (measured: 452 vs 414 ms).
    // The arrays are laid out kind by kind, all layers of a kind in a row, so that arrays of equal
    // size follow each other without padding.
    size_t off = 0;
    auto take = [&](size_t bytes) {
        size_t align = 256;
        if (bytes >= ((size_t)1 << 20)) {
            align = (size_t)1 << 20;
            while (align < ((size_t)2 << 20) && 2 * align <= bytes) align *= 2;
        }
        off = (off + align - 1) & ~(align - 1);
        const size_t o = off;
        off += align_up(bytes);
        return o;
    };
    pl.pl.resize(n_layers);
    pl.table = take(sizeof(LayerDev) * (size_t)n_layers);
    const bool gw = grad_buffers_wanted(layers, n_layers, cfg);
    const bool lm = lds_forward_wanted(layers, n_layers, cfg);
    size_t max_n = 0, max_pos = 0;
    std::vector<size_t> nnz((size_t)n_layers);
    for (int32_t l = 0; l < n_layers; ++l) {
        const sdnn_layer &y = layers[l];
        nnz[l] = (size_t)y.row_ptr[y.n_out];
        Plan::PerLayer &q = pl.pl[l];
        q.t_row_ptr = q.t_row_idx = q.t_perm = q.t_sched = 0;
        q.X = q.D = q.G[0] = q.G[1] = q.vals_t = q.mid_slot = q.mid_dst = q.mid_loc = q.mid = 0;
        q.b1_cs[0] = q.b1_cs[1] = q.b1_row[0] = q.b1_row[1] = q.b1_lm[0] = q.b1_lm[1] = 0;
        q.b1_blocks[0] = q.b1_blocks[1] = 0;
        q.b1_chunks[0] = q.b1_chunks[1] = 0;
        if (lm) {
            LmLayer t;
            t.nb = ((y.n_out + 63) / 64 + LDS_WAVES - 1) / LDS_WAVES;
            t.n_pos = 64 * LDS_WAVES * t.nb;
            max_pos = std::max(max_pos, (size_t)t.n_pos);
            t.cs = (int32_t)pl.lm_n_cs;
            t.pos = (int32_t)pl.lm_n_pos;
            pl.lm_tab.push_back(t);
            pl.lm_n_cs += (size_t)LDS_WAVES * (size_t)(t.nb + 1);
            pl.lm_n_pos += (size_t)t.n_pos;
            pl.lm_n_rows += (size_t)y.n_out;
            pl.lm_n_chunks += lm_chunks(y);
        }
        max_n = std::max(max_n, (size_t)std::max(y.n_out, y.n_in));
    }
    const size_t mb = (size_t)cfg->max_batch, mld = (size_t)row_pitch((int64_t)max_n, cfg->max_batch);
    plan_b1(layers, n_layers, cfg, pl);
    const bool b1 = pl.b1_chunk_bytes != 0;
    pl.pan = pan_wanted(layers, n_layers, cfg, lm, pl.pl);
    plan_train(layers, n_layers, cfg, pl);
    plan_long(layers, n_layers, cfg, pl);
    size_t paired = 0; // floats of the largest block of activations between its layers
    if (pl.pan) {
        for (int32_t l = 0; l < n_layers; ++l) paired = std::max(paired, (size_t)std::max(pl.pl[l].pan.in_pos, pl.pl[l].pan.out_pos));
        paired *= (mb + 1) / 2 * 2;
    }
#define PLAN_KIND(field, bytes_expr)                                   \
    for (int32_t l = 0; l < n_layers; ++l) {                           \
        const sdnn_layer &y = layers[l];                               \
        Plan::PerLayer &q = pl.pl[l];                                  \
        (void)y;                                                       \
        q.field = take(bytes_expr);                                    \
    }
    PLAN_KIND(row_ptr, 4 * ((size_t)y.n_out + 1))
    PLAN_KIND(col_idx, 4 * nnz[l])
    PLAN_KIND(vals, 4 * nnz[l])
    PLAN_KIND(bias, 4 * (size_t)y.n_out)
    PLAN_KIND(sched, 16 * (size_t)y.n_out)
    if (lm) {
        pl.lm = take(LDS_CHUNK_BYTES * (pl.lm_n_chunks + 1)); // a wavefront requests one chunk past its last
        pl.lm_cs = take(4 * pl.lm_n_cs);
        pl.lm_layers = take(sizeof(LmLayer) * (size_t)n_layers);
        pl.lm_row = take(4 * pl.lm_n_pos);
        pl.lm_bias = take(4 * pl.lm_n_pos);
        pl.lm_pos = take(4 * pl.lm_n_rows);
    }
    if (pl.pan) {
        PLAN_KIND(pan_stream, LDS_HALF_BYTES * (q.pan.halves + 2)) // a wavefront requests two halves past its last
        PLAN_KIND(pan_ends, q.pan.halves + 2)
        PLAN_KIND(pan_seg, 4 * (size_t)q.pan.n_ranges * LDS_WAVES * (size_t)(q.pan.n_panels + 1))
        PLAN_KIND(pan_slot, 4 * (size_t)q.pan.n_ranges * LDS_WAVES * (size_t)q.pan.n_panels * (size_t)(q.pan.nb + 1))
        PLAN_KIND(pan_rows, 4 * (size_t)q.pan.out_pos)
        PLAN_KIND(pan_bias, 4 * (size_t)q.pan.out_pos)
        PLAN_KIND(pan_pos, 4 * (size_t)y.n_out)
    }
    if (cfg->training) {
        PLAN_KIND(t_row_ptr, 4 * ((size_t)y.n_in + 1))
        PLAN_KIND(t_row_idx, 4 * nnz[l])
        PLAN_KIND(t_perm, 4 * nnz[l])
        PLAN_KIND(t_sched, 16 * (size_t)y.n_in)
        pl.x0 = take(4 * (size_t)layers[0].n_in * mld);
        PLAN_KIND(X, 4 * (size_t)y.n_out * mld)
        PLAN_KIND(D, 4 * (size_t)y.n_out * mld)
        if (gw) {
            PLAN_KIND(G[0], 4 * nnz[l])
            PLAN_KIND(G[1], 4 * nnz[l])
            PLAN_KIND(vals_t, 4 * nnz[l])
            PLAN_KIND(mid_slot, 2 * nnz[l])
            PLAN_KIND(mid_dst, 4 * nnz[l])
            PLAN_KIND(mid_loc, 2 * nnz[l])
            PLAN_KIND(mid, 4 * nnz[l])
        }
        for (Plan::Train &t : pl.train) {
            if (!pl.train_lds) break;
            t.lm = take(LDS_CHUNK_BYTES * (t.n_chunks + 1)); // a wavefront requests one chunk past its last
            t.cs = take(4 * t.n_cs);
            t.d_tab = take(sizeof(LmLayer) * t.tab.size());
            t.row = take(4 * t.n_pos);
            t.pos = take(4 * t.n_rows);
            t.first = take(4 * t.tab.size());
            t.bias = take(4 * t.n_pos);
            t.out = take(4 * t.n_pos * mb);
        }
        if (pl.long_lm) {
            PLAN_KIND(b1_cs[0], 4 * ((size_t)q.b1_blocks[0] + 1))
            PLAN_KIND(b1_row[0], 8 * 64 * (size_t)q.b1_blocks[0])
            PLAN_KIND(b1_lm[0], LDS_HALF_BYTES * (q.b1_chunks[0] + 2)) // a wavefront requests two halves past its last
        }
        if (b1) {
            PLAN_KIND(b1_cs[0], 4 * ((size_t)q.b1_blocks[0] + 1))
            PLAN_KIND(b1_cs[1], 4 * ((size_t)q.b1_blocks[1] + 1))
            PLAN_KIND(b1_row[0], 8 * 64 * (size_t)q.b1_blocks[0])
            PLAN_KIND(b1_row[1], 8 * 64 * (size_t)q.b1_blocks[1])
            PLAN_KIND(b1_lm[0], pl.b1_chunk_bytes * q.b1_chunks[0])
            PLAN_KIND(b1_lm[1], pl.b1_chunk_bytes * q.b1_chunks[1])
        }
    } else {
        const size_t buffer = 4 * std::max({max_n * mld, max_pos, paired}); // one sample on the lane-major copy: a float per position
        pl.ping = take(buffer);
        pl.pong = take(buffer);
        pl.alive = take(4 * mb);
        for (int k = 0; k < 2; ++k) {
            pl.flags[k] = take(4 * mb);
            pl.map[k] = take(4 * mb);
            pl.n_live[k] = take(4);
        }
    }
#undef PLAN_KIND
    pl.total = off;
}

extern "C" int sdnn_workspace_bytes(const sdnn_layer *layers, int32_t n_layers,
                                    const sdnn_config *cfg, size_t *bytes)
{
    if (!bytes) return fail(nullptr, SDNN_EINVAL, "bytes is NULL");
    int rc = check_config(layers, n_layers, cfg);
    if (rc) return rc;
    for (int32_t l = 0; l < n_layers; ++l) { // the plan counts rows by their length
        const sdnn_layer &y = layers[l];
        bool ok = y.row_ptr[0] == 0;
        for (int32_t r = 0; ok && r < y.n_out; ++r)
            ok = y.row_ptr[r + 1] >= y.row_ptr[r] && y.row_ptr[r + 1] - y.row_ptr[r] <= y.n_in;
        if (!ok) return fail(nullptr, SDNN_EINVAL, "layer %d: malformed row_ptr", l + 1);
    }
    Plan pl;
    try {
        make_plan(layers, n_layers, cfg, pl);
    } catch (...) {
        return fail(nullptr, SDNN_ENOMEM, "host allocation failed");
    }
    *bytes = pl.total;
    return SDNN_OK;
}

// Parts that the passes over a lane-major copy cut its blocks into: at most four chunks of eight entries one after the other
// in the longest row, at most 64 parts.
static unsigned fill_parts(int32_t longest) { return (unsigned)std::min(std::max((longest + 31) / 32, 1), 64); }

// (Re)writes layer l's part of the lane-major copy from its CSR arrays.
static int launch_lm_fill(sdnn_net *net, int l, const int32_t *prev_pos, int with_cols, hipStream_t stream)
{
    if (net->lm_tab[l].nb == 0) return SDNN_OK;
    hipLaunchKernelGGL(k_lm_fill, dim3((unsigned)net->lm_tab[l].nb, LDS_WAVES, fill_parts(net->max_len[0][l])), dim3(64), 0, stream, net->d_layers + l, net->lm_layers + l,
                       net->lm_cs, net->lm, net->lm_bias, net->lm_row, prev_pos, with_cols, net->lm_max_pos + net->lm_two, l & 1 ? net->lm_two : 0);
    HIP_TRY(net, hipGetLastError());
    return SDNN_OK;
}

// (Re)writes the copies for k_train_lds from the CSR arrays: those of layer l, or of all (l < 0).
static int launch_train_fill(sdnn_net *net, int l, bool cols, hipStream_t stream)
{
    for (int o = 0; o < 2; ++o) {
        const sdnn_net::Train &t = net->train[o];
        const int n = (int)t.tab.size(), from = l < 0 ? 0 : o ? net->n_layers - 1 - l : l, to = l < 0 ? n : std::min(n, from + 1);
        const void *fn = o ? cols ? (const void *)k_train_fill<1, true> : (const void *)k_train_fill<1, false>
                           : cols ? (const void *)k_train_fill<0, true> : (const void *)k_train_fill<0, false>;
        for (int k0 = from; k0 < to; k0 += 65536) {
            const int n_steps = std::min(65536, to - k0);
            void *args[] = {(void *)&net->d_layers, (void *)&net->n_layers, (void *)&k0, (void *)&n_steps, (void *)&t.d_tab, (void *)&t.cs, (void *)&t.lm, (void *)&t.row,
                            (void *)&t.pos, (void *)&t.first, (void *)&t.bias};
            HIP_TRY(net, hipLaunchKernel(fn, dim3((unsigned)(8 * LDS_WAVES * t.max_nb), (unsigned)((n_steps + 7) / 8)), dim3(256), args, 0, stream));
        }
    }
    return SDNN_OK;
}

// Whether the passes over B samples go through k_train_lds: where both together are done sooner than with a launch per layer.
// A launch per layer takes 3.2 us forward and 4.0 us back, 28 ns per entry of its longest row and its gathers, at 20 TB/s; 0.2 us more
// where the entries of W no longer stay in the L2s (4 MB each) from one pass to the next, since nothing reads ahead.  A step of a
// single launch takes 1.9 us (barrier, turning the samples around, bringing the copies up to date) and 56 ns per chunk of a wavefront;
// with a sample on every compute unit nobody reads ahead, and the copies take 39 ns per chunk more to come from HBM.  us per layer of a
// training step, 48 layers of 32 entries per row, a launch per layer / single: 300 neurons 8.9 / 4.2 (2 samples), 12.8 / 7.2 (256); 1024
// neurons 9.6 / 7.6 (2), 10.6 / 7.6 (64), 16.6 / 10.4 (200), 16.9 / 11.0 (248), 16.5 / 13.3 (256); 1450 neurons 10.6 / 10.6 (2), 11.4 /
// 10.6 (64), 19.6 / 14.6 (200), 19.7 / 19.2 (256); 1800 neurons 10.9 / 12.4 (2), 11.1 / 12.4 (16), 12.4 / 12.3 (64); 2048 neurons 11.0 /
// 13.5 (2), 12.5 / 13.2 (64), 14.4 / 14.3 (96), 15.4 / 14.8 (127); of 8 entries 8.6 / 8.0 (2), 14.6 / 14.4 (256); 1024 neurons of 64
// entries 13.0 / 12.2 (2); 512 neurons of 160 entries 20.9 / 14.6 (2).  120 layers, one net over and over and (three in turn): 1536 neurons
// 10.81 / 10.77 (11.50 / 11.34) with 2 samples, 1600 10.83 / 11.19 (11.63 / 11.78) with 2 and 11.08 / 11.02 (11.86 / 11.49) with 16, 1850 11.95 /
// 12.05 (12.88 / 12.23) with 64, 2048 12.11 / 13.01 (12.93 / 13.14) with 64.
static bool train_lds_pays(const sdnn_net *net, int B)
{
    const int width = B <= 64 ? B : (B + 63) & ~63;
    return net->train_single + (B >= net->n_cu ? net->train_cold : 0.0) < net->train_per_layer + net->train_gathers * width;
}
static bool train_lds(const sdnn_net *net, int B) { return B > 1 && B <= net->n_cu && !net->train[0].tab.empty() && train_lds_pays(net, B); }

// A graph's replays are not seen here: what is captured leaves the copies current by itself.
static bool capturing(hipStream_t stream)
{
    hipStreamCaptureStatus status = hipStreamCaptureStatusNone;
    if (hipStreamIsCapturing(stream, &status) == hipSuccess) return status != hipStreamCaptureStatusNone;
    (void)hipGetLastError(); // another stream's capture is in the way
    return true;
}

static int launch_train_lds(sdnn_net *net, int o, int B, int Bp, int ld, hipStream_t stream)
{
    const bool captured = capturing(stream);
    net->train_kept |= captured;
    if (net->train_stale) {
        const int rc = launch_train_fill(net, -1, false, stream);
        if (rc) return rc;
        net->train_stale = captured;
    }
    net->train_replaced &= captured;
    const sdnn_net::Train &t = net->train[o];
    TrainLds a;
    a.layers = net->d_layers; a.tab = t.d_tab; a.tab_x = net->train[0].d_tab; a.cs = t.cs; a.lm = t.lm; a.bias = t.bias; a.out = t.out;
    a.x = net->train[0].out; a.lm_bytes = (unsigned)(LDS_CHUNK_BYTES * (t.chunks + 1));
    a.n_steps = (int)t.tab.size(); a.n_layers = net->n_layers; a.max_batch = net->cfg.max_batch; a.ld = ld; a.B = B; a.cap = net->cfg.act_cap;
    const bool sig = net->cfg.activation == ACT_SIGMOID;
    const void *fn = o ? sig ? (const void *)k_train_lds<1, ACT_SIGMOID> : (const void *)k_train_lds<1, ACT_RELU_CAP>
                       : sig ? (const void *)k_train_lds<0, ACT_SIGMOID> : (const void *)k_train_lds<0, ACT_RELU_CAP>;
    void *args[] = {(void *)&a};
    HIP_TRY(net, hipLaunchKernel(fn, dim3((unsigned)(B + std::min(128, std::max(0, net->n_cu - B)))), dim3(64 * LDS_WAVES), args, 0, stream));
    fn = o ? (const void *)k_train_turn<1> : (const void *)k_train_turn<0>;
    for (int k0 = 0; k0 < a.n_steps; k0 += 65535) {
        void *targs[] = {(void *)&net->d_layers, (void *)&net->n_layers, (void *)&k0, (void *)&t.d_tab, (void *)&t.row, (void *)&t.out,
                         (void *)&net->cfg.max_batch, (void *)&ld, (void *)&B, (void *)&Bp};
        HIP_TRY(net, hipLaunchKernel(fn, dim3((unsigned)(LDS_WAVES * t.max_nb), (unsigned)((Bp + 63) / 64), (unsigned)std::min(65535, a.n_steps - k0)),
                                     dim3(256), targs, 0, stream));
    }
    return SDNN_OK;
}

// (Re)writes layer l's copy for k_fwd_pan from its CSR arrays.
static int launch_pan_fill(sdnn_net *net, int l, hipStream_t stream)
{
    const sdnn_net::Pan &f = net->pan[l];
    hipLaunchKernelGGL(k_pan_fill, dim3((unsigned)(f.g.nb * f.g.n_ranges), LDS_WAVES, (unsigned)f.g.n_panels), dim3(64), 0, stream,
                       net->d_layers + l, f.stream, f.slot, f.rows, f.bias, f.g.nb, f.g.panel_cols, f.g.panel,
                       l > 0 ? (const int32_t *)net->pan[l - 1].pos : nullptr);
    HIP_TRY(net, hipGetLastError());
    return SDNN_OK;
}

// (Re)writes both copies of layer l from its CSR arrays.
static int launch_b1_fill(sdnn_net *net, int l, int with_cols, hipStream_t stream)
{
    const LayerDev &d = net->layers[l];
    for (int o = 0; o < 2; ++o) {
        if (d.b1_blocks[o] == 0) continue;
        const dim3 grid((unsigned)d.b1_blocks[o], fill_parts(net->max_len[o][l]));
        if (net->b1_wide) hipLaunchKernelGGL(k_b1_fill<true>, grid, dim3(64), 0, stream, net->d_layers + l, o, with_cols);
        else hipLaunchKernelGGL(k_b1_fill<false>, grid, dim3(64), 0, stream, net->d_layers + l, o, with_cols);
        HIP_TRY(net, hipGetLastError());
    }
    return SDNN_OK;
}

// sdnn_weight_grad brings the gradient into CSR order in the two passes that the stepped values go through, or by a scatter of single values,
// which is the faster way where its lines stay on chip: in small layers, and in layers of short rows whose columns lie close together (few
// runs per span).  With the bias, us, scatter / two passes: random columns, 32 entries per row, 1.05e6 entries 20 / 23, 1.44e6 23.2 / 24.4, 1.60e6
// 26.5 / 24.9, 2.10e6 31.9 / 26.4; 64 per row 1.54e6 22.2 / 24.4, 1.79e6 27.0 / 24.6; 820 per row, 6.72e6 77 / 34; columns on a diagonal, 32 per row
// (2 runs), 2.10e6 16 / 22, 8.39e6 44.5 / 46.3; 64 per row, 4.19e6 32 / 26; in a window of 4096 columns, 32 per row (9 runs), 2.10e6 25.7 / 24.9, 4.19e6
// 50 / 31; of 512 columns (2 runs), 2.10e6 22.6 / 24.4.
#define GRAD_SPREAD_MIN (7 << 18)
static bool grad_spread_pays(const sdnn_layer &y, size_t runs)
{
    const int64_t nnz = y.row_ptr[y.n_out];
    return nnz >= GRAD_SPREAD_MIN && (runs >= 6 * (size_t)((nnz + TR_SPAN - 1) / TR_SPAN) || nnz >= 64 * (int64_t)y.n_out);
}

// Brings the copies for k_fwd_long of layers l0 .. l0 + n - 1 up to date with the CSR values (cols: and writes their columns).
static int launch_long_fill(sdnn_net *net, int l0, int n, bool cols, hipStream_t stream)
{
    int blocks = 1;
    for (int l = l0; l < l0 + n; ++l) blocks = std::max(blocks, net->layers[l].b1_blocks[0]);
    for (int k = 0; k < n; k += 65535) {
        const dim3 grid((unsigned)blocks, 16, (unsigned)std::min(65535, n - k)); // (8 parts: 105 us for six layers of 8192 neurons of 820 entries, 16: 97)
        if (cols) hipLaunchKernelGGL(k_long_fill<true>, grid, dim3(256), 0, stream, net->d_layers + l0 + k);
        else hipLaunchKernelGGL(k_long_fill<false>, grid, dim3(256), 0, stream, net->d_layers + l0 + k);
        HIP_TRY(net, hipGetLastError());
    }
    return SDNN_OK;
}
// From 65 samples on: narrower batches are gathered in rows of 256 bytes by k_spmm<1>, where a step is 4 to 12 % slower with the copies
// (step of 6 layers, a tenth of the columns with a heavy tail, us without / with, 64, 66, 128 and 256 samples: 1301 neurons 218 / 227, 268 /
// 255, 268 / 255, 279 / 262; 3001 neurons 487 / 534, 600 / 569, 588 / 562, 667 / 611; 8192 neurons 1803 / 1948, 2639 / 2236, 2644 / 2299,
// 3602 / 3090).
// More groups of four samples than compute units take a second round and more: not where the last one leaves more than a quarter of
// all places empty, nor where a workgroup waits for the deepest block of a layer, which k_spmm's wavefronts of all samples do at the
// same time (forward pass, us, k_spmm / this; 6 layers of 1024 neurons of 256 entries, 1024 samples 295 / 189, 1028 276 / 296, 1536 342 /
// 304, 2048 427 / 327; 3 of 8192 neurons of 820, 1536 samples 3613 / 2518, 2048 4253 / 2820; 64 rows of 2400 entries, 1028 samples 156 / 194,
// 2052 152 / 295; 2 layers of 8192 neurons, 64 rows of all of them, 130 entries else, 2048 samples 1444 / 1505; 6 of 513 neurons of 300, 2304
// samples 305 / 335).
static bool long_forward(const sdnn_net *net, int B)
{
    if (!net->long_lm || B < LONG_MIN_BATCH) return false;
    const int groups = padded_batch(B) / 4, n_cu = std::max(net->n_cu, 1), rounds = ((groups + 7) / 8 * 8 + n_cu - 1) / n_cu;
    return rounds == 1 || (net->long_even && 4 * (int64_t)groups >= 3 * (int64_t)rounds * n_cu);
}

extern "C" int sdnn_create(const sdnn_layer *layers, int32_t n_layers, const sdnn_config *cfg,
                           void *d_workspace, size_t workspace_bytes, void *stream_,
                           sdnn_net **out)
{
    if (!out) return fail(nullptr, SDNN_EINVAL, "out is NULL");
    *out = nullptr;
    int rc = check_config(layers, n_layers, cfg);
    if (rc) return rc;
    for (int32_t l = 0; l < n_layers; ++l) {
        rc = sdnn_check_csr(layers[l].n_out, layers[l].n_in, layers[l].row_ptr, layers[l].col_idx);
        if (rc) return fail(nullptr, rc, "layer %d: %s", l + 1, sdnn_global_error());
        if (layers[l].row_ptr[layers[l].n_out] > 0 && !layers[l].values)
            return fail(nullptr, SDNN_EINVAL, "layer %d: values is NULL", l + 1);
    }
    if (!d_workspace) return fail(nullptr, SDNN_EINVAL, "d_workspace is NULL");
    if (((uintptr_t)d_workspace & 255) != 0)
        return fail(nullptr, SDNN_EINVAL, "d_workspace must be 256-byte aligned");
    Plan pl;
    try {
        make_plan(layers, n_layers, cfg, pl);
    } catch (...) {
        return fail(nullptr, SDNN_ENOMEM, "host allocation failed");
    }
    if (workspace_bytes < pl.total)
        return fail(nullptr, SDNN_ENOMEM, "workspace too small: %zu < %zu", workspace_bytes, pl.total);

    hipStream_t stream = (hipStream_t)stream_;
    sdnn_net *net = new (std::nothrow) sdnn_net;
    if (!net) return fail(nullptr, SDNN_ENOMEM, "host allocation failed");
    net->n_layers = n_layers;
    net->cfg = *cfg;
    try {
        net->layers.resize(n_layers);
        net->pan.resize(pl.pan ? n_layers : 0);
        net->max_len[0].resize(n_layers);
        net->max_len[1].resize(n_layers);
        net->grad_spread.resize(n_layers);
        net->clustered[0].resize(n_layers);
        net->clustered[1].resize(n_layers);
    } catch (...) {
        delete net;
        return fail(nullptr, SDNN_ENOMEM, "host allocation failed");
    }
    char *base = (char *)d_workspace;
    auto fail_free = [&](int code) { sdnn_destroy(net); return code; };
    {
        int devid = 0;
        hipDeviceProp_t prop;
        if (hipGetDevice(&devid) != hipSuccess || hipGetDeviceProperties(&prop, devid) != hipSuccess)
            return fail_free(fail(nullptr, SDNN_EHIP, "cannot query the device"));
        net->n_cu = prop.multiProcessorCount;
    }

    // Host part of the setup (transposed index, row schedules): independent per layer, so a group of layers is
    // prepared by one host thread each, then uploaded with one synchronisation for the whole group.
    struct HostIdx {
        std::vector<int32_t> t_row_ptr, t_row_idx, t_perm, order, t_order;
        std::vector<int4> sched, t_sched;
        std::vector<float> vals_t;
        std::vector<int32_t> mid_dst;
        std::vector<uint16_t> mid_slot, mid_loc;
        std::vector<int32_t> b1_cs[2];
        std::vector<int2> b1_row[2];
        PanLayout pan;
        int32_t max_len = 0, t_max_len = 0;
        size_t runs = 0; // of entries that k_apply writes one after the other
        bool clustered = false, t_clustered = false; // reorder_rows found rows that share columns
        int rc = SDNN_OK;
    };
    const bool want_lm = !pl.lm_tab.empty();
    struct { std::vector<int32_t> cs, row, pos, first; } tl[2];
    std::vector<int32_t> lm_cs, lm_row, lm_pos;
    std::vector<size_t> lm_first_row((size_t)n_layers, 0); // where a layer's part of lm_pos starts
    try {
        lm_cs.resize(pl.lm_n_cs);
        lm_row.resize(pl.lm_n_pos);
        lm_pos.resize(pl.lm_n_rows);
        for (int o = 0; o < (pl.train_lds ? 2 : 0); ++o) {
            const Plan::Train &t = pl.train[o];
            tl[o].cs.resize(t.n_cs);
            tl[o].row.resize(t.n_pos);
            tl[o].pos.resize(t.n_rows);
            tl[o].first.resize(t.tab.size(), 0);
            for (size_t k = 1; k < t.tab.size(); ++k) {
                const sdnn_layer &y = layers[o ? n_layers - (int32_t)k : (int32_t)k - 1];
                tl[o].first[k] = tl[o].first[k - 1] + (o ? y.n_in : y.n_out);
            }
        }
    } catch (...) {
        return fail_free(fail(nullptr, SDNN_ENOMEM, "host allocation failed"));
    }
    for (int32_t l = 1; l < n_layers; ++l) lm_first_row[l] = lm_first_row[l - 1] + (size_t)layers[l - 1].n_out;
    const bool training = cfg->training != 0; // the transposed index serves the backward pass only
    const bool gw_ = grad_buffers_wanted(layers, n_layers, cfg);
    const bool b1 = pl.b1_chunk_bytes != 0;
    net->b1_wide = pl.b1_chunk_bytes == 4096;
    net->long_lm = pl.long_lm;
    net->b1 = b1;
    auto prepare = [&](int32_t l, HostIdx &h) {
        try {
            const sdnn_layer &y = layers[l];
            const size_t nnz = (size_t)y.row_ptr[y.n_out];
            h.order.resize(y.n_out);
            h.sched.resize(y.n_out);
            if (training) {
                h.t_row_ptr.resize((size_t)y.n_in + 1);
                h.t_row_idx.resize(nnz);
                h.t_perm.resize(nnz);
                h.t_order.resize(y.n_in);
                h.t_sched.resize(y.n_in);
                h.rc = sdnn_transpose_pattern(y.n_out, y.n_in, y.row_ptr, y.col_idx, h.t_row_ptr.data(),
                                              h.t_row_idx.data(), h.t_perm.data());
                if (h.rc) return;
            }
            if (cfg->reorder_rows) {
                // rows that share columns become neighbours and are dealt to one XCD
                const size_t n_max = (size_t)std::max(y.n_out, y.n_in);
                std::vector<int32_t> clustered(n_max), cluster_of(n_max);
                // "found something": on average at least two rows per cluster
                auto found = [&](int32_t n) {
                    int32_t n_clusters = 0;
                    for (int32_t r = 0; r < n; ++r) n_clusters = std::max(n_clusters, cluster_of[r] + 1);
                    return 2 * (int64_t)n_clusters <= n;
                };
                h.rc = sdnn_cluster_rows(y.n_out, y.n_in, y.row_ptr, y.col_idx, SDNN_CLUSTER_ROWS, clustered.data(),
                                         cluster_of.data());
                if (!h.rc) h.clustered = found(y.n_out);
                if (!h.rc) h.rc = sdnn_deal_rows_to_xcds(y.n_out, y.row_ptr, clustered.data(), h.order.data());
                if (training) {
                    if (!h.rc) h.rc = sdnn_cluster_rows(y.n_in, y.n_out, h.t_row_ptr.data(), h.t_row_idx.data(), SDNN_CLUSTER_ROWS,
                                                        clustered.data(), cluster_of.data());
                    if (!h.rc) h.t_clustered = found(y.n_in);
                    if (!h.rc) h.rc = sdnn_deal_rows_to_xcds(y.n_in, h.t_row_ptr.data(), clustered.data(), h.t_order.data());
                }
                if (h.rc) return;
            } else {
                sdnn_row_schedule(y.n_out, y.row_ptr, h.order.data());
                if (training) sdnn_row_schedule(y.n_in, h.t_row_ptr.data(), h.t_order.data());
            }
            for (int32_t r = 0; r < y.n_out; ++r)
                h.sched[r] = make_int4(h.order[r], y.row_ptr[h.order[r]], y.row_ptr[h.order[r] + 1], 0);
            for (size_t r = 0; r < h.t_sched.size(); ++r)
                h.t_sched[r] = make_int4(h.t_order[r], h.t_row_ptr[h.t_order[r]], h.t_row_ptr[h.t_order[r] + 1], 0);
            for (int o = 0; o < (b1 ? 2 : pl.long_lm ? 1 : 0); ++o) { // blocks of 64 rows, longest first, whatever the row schedule is
                const int32_t n = o ? y.n_in : y.n_out, *ptr = o ? h.t_row_ptr.data() : y.row_ptr;
                std::vector<int32_t> by_len((size_t)n);
                sdnn_row_schedule(n, ptr, by_len.data());
                const int32_t nb = pl.pl[l].b1_blocks[o];
                h.b1_cs[o].assign((size_t)nb + 1, 0);
                h.b1_row[o].assign((size_t)nb * 64, make_int2(-1, 0));
                for (int32_t b = 0; b < nb; ++b) {
                    const int32_t first = by_len[(size_t)b * 64];
                    h.b1_cs[o][(size_t)b + 1] = h.b1_cs[o][(size_t)b] + (ptr[first + 1] - ptr[first] + 7) / 8;
                    for (int32_t k = 0; k < 64 && 64 * b + k < n; ++k) {
                        const int32_t row = by_len[(size_t)b * 64 + k];
                        h.b1_row[o][(size_t)b * 64 + k] = make_int2(row, ptr[row + 1] - ptr[row]);
                    }
                }
            }
            if (gw_) { // the values in the order of the transposed index, for the fused backward sweep
                h.vals_t.resize(nnz);
                h.mid_slot.resize(nnz);
                h.mid_dst.resize(nnz);
                h.mid_loc.resize(nnz);
                // every chunk of the CSR array but the last holds TR_CHUNK entries, so chunk c's group starts at c TR_CHUNK
                const size_t n_chunks = (nnz + TR_CHUNK - 1) / TR_CHUNK;
                std::vector<int32_t> filled(n_chunks, 0), in_span(n_chunks, 0), touched;
                for (size_t s0 = 0; s0 < nnz; s0 += TR_SPAN) {
                    const size_t s1 = std::min(nnz, s0 + (size_t)TR_SPAN);
                    touched.clear();
                    for (size_t q = s0; q < s1; ++q) {
                        const size_t c = (size_t)h.t_perm[q] / TR_CHUNK;
                        if (in_span[c]++ == 0) touched.push_back((int32_t)c);
                    }
                    std::sort(touched.begin(), touched.end());
                    h.runs += touched.size();
                    int32_t run = 0; // in_span[c]: from the span's count for chunk c to the rank of its next entry
                    for (int32_t c : touched) { const int32_t n = in_span[c]; in_span[c] = run; run += n; }
                    for (size_t q = s0; q < s1; ++q) {
                        const size_t p = (size_t)h.t_perm[q], c = p / TR_CHUNK;
                        const size_t m = c * TR_CHUNK + (size_t)filled[c]++;
                        const int32_t k = in_span[c]++;
                        h.vals_t[q] = y.values[p];
                        h.mid_slot[q] = (uint16_t)k;
                        h.mid_dst[s0 + (size_t)k] = (int32_t)m;
                        h.mid_loc[m] = (uint16_t)(p - c * TR_CHUNK);
                    }
                    for (int32_t c : touched) in_span[c] = 0;
                }
            }
            if (want_lm) {
                const LmLayer &t = pl.lm_tab[l];
                lm_deal_blocks(y, t, lm_row.data() + t.pos, lm_pos.data() + lm_first_row[l], lm_cs.data() + t.cs);
            }
            if (pl.train_lds) { // the rows of W_l^T by length (l > 1), and those of the last W; the others follow them (below)
                const int32_t o = l > 0, k = o ? n_layers - 1 - l : n_layers - 1;
                const LmLayer &t = pl.train[o].tab[(size_t)k];
                sdnn_layer v = o ? y : layers[n_layers - 1];
                if (o) {
                    v.n_out = y.n_in;
                    v.row_ptr = h.t_row_ptr.data();
                }
                lm_deal_blocks(v, t, tl[o].row.data() + t.pos, tl[o].pos.data() + tl[o].first[(size_t)k], tl[o].cs.data() + t.cs);
            }
            if (pl.pan) sdnn_pan_layout(y, pl.pl[l].pan, h.pan);
            h.max_len = h.t_max_len = 0;
            for (int32_t r = 0; r < y.n_out; ++r) h.max_len = std::max(h.max_len, y.row_ptr[r + 1] - y.row_ptr[r]);
            if (training)
                for (int32_t r = 0; r < y.n_in; ++r) h.t_max_len = std::max(h.t_max_len, h.t_row_ptr[r + 1] - h.t_row_ptr[r]);
        } catch (...) {
            h.rc = SDNN_ENOMEM;
        }
    };
#define UP(dst, src, bytes)                                                                   \
    do {                                                                                      \
        if ((bytes) > 0) {                                                                    \
            hipError_t e_ = hipMemcpyAsync((void *)(dst), (src), (bytes), hipMemcpyHostToDevice, stream); \
            if (e_ != hipSuccess)                                                             \
                return fail_free(fail(nullptr, SDNN_EHIP, "upload: %s", hipGetErrorString(e_))); \
        }                                                                                     \
    } while (0)
#define SYNC()                                                                                \
    do {                                                                                      \
        hipError_t e_ = hipStreamSynchronize(stream);                                         \
        if (e_ != hipSuccess)                                                                 \
            return fail_free(fail(nullptr, SDNN_EHIP, "upload: %s", hipGetErrorString(e_)));  \
    } while (0)
    try {
        const bool gw = grad_buffers_wanted(layers, n_layers, cfg);
        int32_t max_out = 0;
        for (int32_t l = 0; l < n_layers; ++l) max_out = std::max(max_out, layers[l].n_out);
        const std::vector<float> zeros((size_t)max_out, 0.0f); // stands in for a NULL bias
        bool pan_fits = pl.pan;
        double pan_fullest = 0.0, pan_mean = 0.0;
        unsigned hw = std::thread::hardware_concurrency();
        const int32_t group = (int32_t)std::max(1u, std::min({hw ? hw : 1u, 16u, (unsigned)n_layers}));
        std::vector<HostIdx> idx((size_t)group);
        for (int32_t l0 = 0; l0 < n_layers; l0 += group) {
            const int32_t ng = std::min(group, n_layers - l0);
            {
                std::vector<std::thread> workers;
                for (int32_t k = 1; k < ng; ++k) {
                    try {
                        workers.emplace_back(prepare, l0 + k, std::ref(idx[k]));
                    } catch (...) { // no more threads: do it here
                        prepare(l0 + k, idx[k]);
                    }
                }
                prepare(l0, idx[0]);
                for (std::thread &w : workers) w.join();
            }
            for (int32_t k = 0; k < ng; ++k) {
                const int32_t l = l0 + k;
                const HostIdx &h = idx[k];
                if (h.rc) return fail_free(fail(nullptr, h.rc, "layer %d: host setup failed (out of memory?)", l + 1));
                const sdnn_layer &y = layers[l];
                const Plan::PerLayer &q = pl.pl[l];
                const size_t nnz = (size_t)y.row_ptr[y.n_out];
                LayerDev &d = net->layers[l];
                d.n_out = y.n_out; d.n_in = y.n_in; d.nnz = (int32_t)nnz; d.pad_ = 0;
                d.row_ptr = (const int32_t *)(base + q.row_ptr);
                d.col_idx = (const int32_t *)(base + q.col_idx);
                d.vals = (float *)(base + q.vals);
                d.bias = (float *)(base + q.bias);
                d.t_row_ptr = training ? (const int32_t *)(base + q.t_row_ptr) : nullptr;
                d.t_row_idx = training ? (const int32_t *)(base + q.t_row_idx) : nullptr;
                d.t_perm = training ? (const int32_t *)(base + q.t_perm) : nullptr;
                d.sched = (const int4 *)(base + q.sched);
                d.t_sched = training ? (const int4 *)(base + q.t_sched) : nullptr;
                d.X = cfg->training ? (float *)(base + q.X) : nullptr;
                d.D = cfg->training ? (float *)(base + q.D) : nullptr;
                d.G[0] = gw ? (float *)(base + q.G[0]) : nullptr;
                d.G[1] = gw ? (float *)(base + q.G[1]) : nullptr;
                d.vals_t = gw ? (float *)(base + q.vals_t) : nullptr;
                d.mid_slot = gw ? (const uint16_t *)(base + q.mid_slot) : nullptr;
                d.mid_dst = gw ? (const int32_t *)(base + q.mid_dst) : nullptr;
                d.mid_loc = gw ? (const uint16_t *)(base + q.mid_loc) : nullptr;
                d.mid = gw ? (float *)(base + q.mid) : nullptr;
                for (int o = 0; o < 2; ++o) {
                    d.b1_blocks[o] = q.b1_blocks[o];
                    const bool copied = b1 || (pl.long_lm && o == 0);
                    d.b1_cs[o] = copied ? (const int32_t *)(base + q.b1_cs[o]) : nullptr;
                    d.b1_row[o] = copied ? (const int2 *)(base + q.b1_row[o]) : nullptr;
                    d.b1_lm[o] = copied ? (int4 *)(base + q.b1_lm[o]) : nullptr;
                    if (copied) {
                        UP(d.b1_cs[o], h.b1_cs[o].data(), 4 * h.b1_cs[o].size());
                        UP(d.b1_row[o], h.b1_row[o].data(), 8 * h.b1_row[o].size());
                    }
                }
                d.X_prev = !cfg->training ? nullptr
                           : l == 0       ? (float *)(base + pl.x0)
                                          : net->layers[l - 1].X;
                net->max_n = std::max(net->max_n, std::max(y.n_out, y.n_in));
                net->grad_spread[l] = gw && grad_spread_pays(y, h.runs);
                net->max_len[0][l] = h.max_len;
                net->max_len[1][l] = h.t_max_len;
                net->clustered[0][l] = h.clustered;
                net->clustered[1][l] = h.t_clustered;
                UP(d.row_ptr, y.row_ptr, 4 * ((size_t)y.n_out + 1));
                UP(d.col_idx, y.col_idx, 4 * nnz);
                UP(d.vals, y.values, 4 * nnz);
                UP(d.bias, y.bias ? y.bias : zeros.data(), 4 * (size_t)y.n_out);
                UP(d.sched, h.sched.data(), 16 * (size_t)y.n_out);
                if (training) {
                    UP(d.t_row_ptr, h.t_row_ptr.data(), 4 * ((size_t)y.n_in + 1));
                    UP(d.t_row_idx, h.t_row_idx.data(), 4 * nnz);
                    UP(d.t_perm, h.t_perm.data(), 4 * nnz);
                    UP(d.t_sched, h.t_sched.data(), 16 * (size_t)y.n_in);
                }
                if (pl.pan) {
                    sdnn_net::Pan &f = net->pan[l];
                    f.g = q.pan;
                    f.depth = h.pan.depth;
                    f.stream = (uint4 *)(base + q.pan_stream); f.ends = (uint32_t *)(base + q.pan_ends);
                    f.seg = (int32_t *)(base + q.pan_seg); f.slot = (int32_t *)(base + q.pan_slot);
                    f.rows = (int32_t *)(base + q.pan_rows); f.pos = (int32_t *)(base + q.pan_pos); f.bias = (float *)(base + q.pan_bias);
                    pan_fits &= h.pan.ends.size() <= q.pan.halves;
                    pan_fullest += (double)h.pan.fullest;
                    pan_mean += (double)nnz / q.pan.n_panels;
                    if (pan_fits) {
                        UP(f.ends, h.pan.ends.data(), h.pan.ends.size());
                        UP(f.seg, h.pan.seg.data(), 4 * h.pan.seg.size());
                        UP(f.slot, h.pan.slot.data(), 4 * h.pan.slot.size());
                        UP(f.rows, h.pan.rows.data(), 4 * h.pan.rows.size());
                        UP(f.pos, h.pan.pos.data(), 4 * h.pan.pos.size());
                    }
                }
                if (gw) UP(d.vals_t, h.vals_t.data(), 4 * nnz);
                if (gw) UP(d.mid_slot, h.mid_slot.data(), 2 * nnz);
                if (gw) UP(d.mid_dst, h.mid_dst.data(), 4 * nnz);
                if (gw) UP(d.mid_loc, h.mid_loc.data(), 2 * nnz);
            }
            SYNC(); // the group's host arrays are reused by the next group
        }
        net->d_layers = (LayerDev *)(base + pl.table);
        UP(net->d_layers, net->layers.data(), sizeof(LayerDev) * (size_t)n_layers);
        if (b1)
            for (int32_t l = 0; l < n_layers; ++l) {
                const int rc_fill = launch_b1_fill(net, l, 1, stream);
                if (rc_fill) return fail_free(rc_fill);
            }
        if (net->long_lm) {
            net->long_stale.assign((size_t)n_layers, 0);
            for (const Plan::PerLayer &q : pl.pl) {
                net->long_bytes.push_back((uint32_t)(LDS_HALF_BYTES * (q.b1_chunks[0] + 2)));
                net->long_even &= q.b1_blocks[0] >= LDS_WAVES && 8 * (size_t)((net->max_len[0][&q - pl.pl.data()] + 7) / 8) <= q.b1_chunks[0];
            }
            const int rc_fill = launch_long_fill(net, 0, n_layers, true, stream);
            if (rc_fill) return fail_free(rc_fill);
        }
        if (pl.train_lds) {
            // layer l's neurons in the order of the rows of W_{l+1}^T in both passes
            for (int32_t k = 0; k + 1 < n_layers; ++k) {
                const LmLayer &t = pl.train[0].tab[(size_t)k], &u = pl.train[1].tab[(size_t)(n_layers - 2 - k)];
                std::copy_n(tl[1].row.data() + u.pos, t.n_pos, tl[0].row.data() + t.pos);
                std::copy_n(tl[1].pos.data() + tl[1].first[(size_t)(n_layers - 2 - k)], layers[k].n_out, tl[0].pos.data() + tl[0].first[(size_t)k]);
                for (int32_t w = 0; w < LDS_WAVES; ++w)
                    for (int32_t j = 0; j < t.nb; ++j) {
                        int32_t len = 0;
                        for (int32_t i = 0; i < 64; ++i) {
                            const int32_t r = tl[0].row[(size_t)(t.pos + 64 * (LDS_WAVES * j + w) + i)];
                            if (r >= 0) len = std::max(len, layers[k].row_ptr[r + 1] - layers[k].row_ptr[r]);
                        }
                        tl[0].cs[(size_t)(t.cs + w * (t.nb + 1) + j)] = (len + LDS_CHUNK - 1) / LDS_CHUNK;
                    }
            }
            bool fits = true, pays = false;
            for (int o = 0; o < 2; ++o) {
                int64_t chunks = 0;
                for (const int32_t depth : tl[o].cs) chunks += depth;
                fits &= (size_t)chunks <= pl.train[o].n_chunks;
                net->train_single += 1.9e-6 * (double)pl.train[o].tab.size() + 56e-9 * (double)chunks;
                net->train_cold += 39e-9 * (double)chunks;
                size_t entries = 0;
                for (int32_t l = 0; l < n_layers; ++l) entries += (size_t)net->layers[l].nnz;
                for (int32_t l = o; l < n_layers; ++l) {
                    net->train_per_layer += (o ? 4.0e-6 : 3.2e-6) + (8 * entries > ((size_t)32 << 20) ? 0.2e-6 : 0.0) + 28e-9 * net->max_len[o][l];
                    net->train_gathers += 4.0 * net->layers[l].nnz / 20e12;
                    fits &= net->max_len[o][l] <= TRAIN_LDS_MAX_ROW;
                }
            }
            for (int32_t B = 2; B <= std::min(cfg->max_batch, net->n_cu); ++B) pays |= train_lds_pays(net, B);
            for (int o = 0; o < (fits && pays ? 2 : 0); ++o) {
                const Plan::Train &t = pl.train[o];
                sdnn_net::Train &n = net->train[o];
                int64_t at = 0; // as for the LDS-resident forward below
                for (int w = 0; w < LDS_WAVES; ++w)
                    for (const LmLayer &e : t.tab) {
                        int32_t *c = tl[o].cs.data() + e.cs + w * (e.nb + 1);
                        for (int32_t j = 0; j <= e.nb; ++j) {
                            const int32_t depth = c[j];
                            c[j] = (int32_t)at;
                            if (j < e.nb) at += depth;
                        }
                    }
                for (const LmLayer &e : t.tab) n.max_nb = std::max(n.max_nb, e.nb);
                n.d_tab = (LmLayer *)(base + t.d_tab);
                n.cs = (int32_t *)(base + t.cs);
                n.row = (int32_t *)(base + t.row);
                n.pos = (int32_t *)(base + t.pos);
                n.first = (int32_t *)(base + t.first);
                n.lm = (uint4 *)(base + t.lm);
                n.bias = (float *)(base + t.bias);
                n.out = (float *)(base + t.out);
                n.chunks = (size_t)at;
                n.tab = t.tab;
                UP(n.cs, tl[o].cs.data(), 4 * tl[o].cs.size());
                UP(n.d_tab, t.tab.data(), sizeof(LmLayer) * t.tab.size());
                UP(n.row, tl[o].row.data(), 4 * tl[o].row.size());
                UP(n.pos, tl[o].pos.data(), 4 * tl[o].pos.size());
                UP(n.first, tl[o].first.data(), 4 * tl[o].first.size());
            }
            const int rc_fill = launch_train_fill(net, -1, true, stream);
            if (rc_fill) return fail_free(rc_fill);
        }
        // not where a layout took too many slots, or where the links stay within few panels: the operand of the other kernels is
        // on chip then
        if (!pan_fits || pan_fullest > 1.5 * pan_mean) net->pan.clear();
        for (int32_t l = 0; l < (int32_t)net->pan.size(); ++l) {
            const int rc_fill = launch_pan_fill(net, l, stream);
            if (rc_fill) return fail_free(rc_fill);
        }
        if (want_lm) {
            int64_t of_bit[LM_IN_ORDER + 1] = {};
            for (const LmLayer &t : pl.lm_tab) {
                const int32_t *c = lm_cs.data() + t.cs, mask = lm_turns(t.nb, c);
                int64_t chunks = 0;
                for (int32_t k = 0; k < LDS_WAVES * (t.nb + 1); ++k) chunks += c[k];
                for (int bit = 1; bit <= LM_IN_ORDER; bit *= 2) of_bit[bit] += mask & bit ? chunks : 0;
            }
            for (int bit = 1; bit <= LM_IN_ORDER; bit *= 2)
                if (4 * of_bit[bit] >= 3 * (int64_t)pl.lm_n_chunks) net->turns |= bit;
            // from the blocks' depths to where their chunks lie: one wavefront's chunks follow each other through all layers
            int64_t at = 0;
            for (int w = 0; w < LDS_WAVES; ++w)
                for (int32_t l = 0; l < n_layers; ++l) {
                    const LmLayer &t = pl.lm_tab[l];
                    int32_t *c = lm_cs.data() + t.cs + w * (t.nb + 1);
                    for (int32_t j = 0; j <= t.nb; ++j) {
                        const int32_t depth = c[j];
                        c[j] = (int32_t)at;
                        if (j < t.nb) at += depth;
                    }
                }
            if ((size_t)at != pl.lm_n_chunks)
                return fail_free(fail(nullptr, SDNN_EINVAL, "lane-major copy does not match its plan"));
            net->lm = (uint4 *)(base + pl.lm);
            net->lm_cs = (int32_t *)(base + pl.lm_cs);
            net->lm_layers = (LmLayer *)(base + pl.lm_layers);
            net->lm_row = (int32_t *)(base + pl.lm_row);
            net->lm_bias = (float *)(base + pl.lm_bias);
            net->lm_chunks = pl.lm_n_chunks;
            net->lm_tab = pl.lm_tab;
            net->lm_max_pos = layers[0].n_in;
            for (const LmLayer &t : pl.lm_tab) net->lm_max_pos = std::max(net->lm_max_pos, t.n_pos);
            net->lm_two = 2 * 4 * net->lm_max_pos <= LDS_MAX_FLOATS ? net->lm_max_pos : 0;
            int32_t *d_pos = (int32_t *)(base + pl.lm_pos);
            UP(net->lm_cs, lm_cs.data(), 4 * lm_cs.size());
            UP(net->lm_layers, pl.lm_tab.data(), sizeof(LmLayer) * (size_t)n_layers);
            UP(net->lm_row, lm_row.data(), 4 * lm_row.size());
            UP(d_pos, lm_pos.data(), 4 * lm_pos.size());
            for (int32_t l = 0; l < n_layers; ++l) {
                const int rc_fill = launch_lm_fill(net, l, l > 0 ? d_pos + lm_first_row[l - 1] : nullptr, 1, stream);
                if (rc_fill) return fail_free(rc_fill);
            }
        }
        SYNC();
    } catch (...) {
        return fail_free(fail(nullptr, SDNN_ENOMEM, "host allocation failed during setup"));
    }
#undef UP
#undef SYNC
    {
        void *scratch_dev = nullptr; // this GPU's copy of the fixed staging array of sdnn_forward_noalloc
        if (scratch_address(nullptr, &scratch_dev) != SDNN_OK) return fail_free(SDNN_EHIP);
    }
    if (cfg->training) {
        net->d_x0 = (float *)(base + pl.x0);
    } else {
        net->d_ping = (float *)(base + pl.ping);
        net->d_pong = (float *)(base + pl.pong);
        net->d_alive = (int32_t *)(base + pl.alive);
        for (int k = 0; k < 2; ++k) {
            net->d_flags[k] = (int32_t *)(base + pl.flags[k]);
            net->d_map[k] = (int32_t *)(base + pl.map[k]);
            net->d_n_live[k] = (int32_t *)(base + pl.n_live[k]);
        }
    }
    net->bias_nonpos = true;
    for (int32_t l = 1; l < n_layers; ++l)
        if (layers[l].bias)
            for (int32_t r = 0; r < layers[l].n_out; ++r)
                if (!(layers[l].bias[r] <= 0.0f)) net->bias_nonpos = false;
    *out = net;
    return SDNN_OK;
}

extern "C" void sdnn_destroy(sdnn_net *net)
{
    if (!net) return;
    delete net;
}

static unsigned ew_blocks(size_t n) // workgroups of 256 threads for an elementwise pass
{
    size_t b = (n + 255) / 256;
    return (unsigned)std::min<size_t>(std::max<size_t>(b, 1), 8192);
}

// The same for FOR_ROW_ELEMENTS: threads per row, and workgroups for n rows.
static int row_threads_log2(int Bp)
{
    int w = 0;
    while (w < 8 && (1 << w) < Bp) ++w;
    return w;
}
static unsigned row_blocks(int n, int w_log2) { return ew_blocks((size_t)n << w_log2); }

static inline bool aligned(const void *p, size_t a) { return ((uintptr_t)p & (a - 1)) == 0; }

// Samples per lane for the row-per-wavefront product: as wide as the batch and the alignment of the operands' rows
// allow without idling most of the wave.
static int pick_v_spmm(int B, int ld_in, int ld_out, const void *in, const void *out)
{
    if (ld_in % 4 == 0 && ld_out % 4 == 0 && B > 128 && aligned(in, 16) && aligned(out, 16)) return 4;
    if (ld_in % 2 == 0 && ld_out % 2 == 0 && B > 64 && aligned(in, 8) && aligned(out, 8)) return 2;
    return 1;
}

// Kernel tables.  The forward kernels are compiled per activation, the backward ones once (ACT = 0).
template <int MODE, int V, int U, bool TI>
static const void *spmm_fn_act(int act)
{
    if (MODE == 0 && act == ACT_SIGMOID) return (const void *)k_spmm<V, MODE, U, TI, (MODE == 0 ? ACT_SIGMOID : 0)>;
    return (const void *)k_spmm<V, MODE, U, TI, 0>;
}
template <int MODE, int V>
static const void *spmm_fn_v(int U, bool ti, int act)
{
    if (ti) return spmm_fn_act<MODE, V, 8, true>(act);
    if (U == 16) return spmm_fn_act<MODE, V, 16, false>(act);
    return spmm_fn_act<MODE, V, 8, false>(act);
}
template <int MODE>
static const void *spmm_fn(int V, int U, bool ti, int act)
{
    return V == 4 ? spmm_fn_v<MODE, 4>(U, ti, act) : V == 2 ? spmm_fn_v<MODE, 2>(U, ti, act) : spmm_fn_v<MODE, 1>(U, ti, act);
}
template <int MODE, int R>
static const void *panel_fn_act(int act)
{
    if (MODE == 0 && act == ACT_SIGMOID) return (const void *)k_spmm_panel<R, MODE, (MODE == 0 ? ACT_SIGMOID : 0)>;
    return (const void *)k_spmm_panel<R, MODE, 0>;
}
template <int MODE>
static const void *panel_fn(int ri, int act)
{
    return ri == 0 ? panel_fn_act<MODE, 1>(act) : ri == 1 ? panel_fn_act<MODE, 2>(act)
           : ri == 2 ? panel_fn_act<MODE, 4>(act) : panel_fn_act<MODE, 8>(act);
}

// The panel sweep (k_spmm_panel) over all 64-sample tiles of the batch; a's operand fields are filled in.
template <int MODE>
static int launch_spmm_panel(sdnn_net *net, const LayerDev &d, SpmmArgs a, int B, int panel, hipStream_t stream,
                             int sub_begin, int sub_end)
{
    a.tile_base = (uint32_t)(sub_begin / 64);
    a.n_tiles = (uint32_t)((sub_end - sub_begin + 63) / 64);
    const int n_cols = MODE == 0 ? d.n_in : d.n_out;
    // rows per wavefront: enough for the wavefronts resident on an XCD to hold all the rows that the XCD
    // has of one tile, so that the whole tile is swept panel by panel in one go (at most 8)
    const int xcds = 8;
    const int64_t rows_per_xcd = a.n_tiles >= 8 ? a.n_rows : (a.n_rows + xcds - 1) / xcds;
    int ri = 0;
    for (;; ++ri) {
        const void *fn_r = panel_fn<MODE>(ri, net->cfg.activation);
        int &occ = net->occ_panel[MODE][ri];
        if (occ == 0) {
            HIP_TRY(net, hipOccupancyMaxActiveBlocksPerMultiprocessor(&occ, fn_r, BLOCK_THREADS, 0));
            if (occ < 1) occ = 1;
        }
        const int64_t resident = (int64_t)occ * WAVES_PER_BLOCK * (net->n_cu / xcds);
        if ((resident << ri) >= rows_per_xcd) break;
        if (ri == 3) break;
    }
    const int R = 1 << ri;
    const void *fn = panel_fn<MODE>(ri, net->cfg.activation);
    a.n_rg = (uint32_t)((a.n_rows + WAVES_PER_BLOCK * R - 1) / (WAVES_PER_BLOCK * R));
    const uint64_t blocks = (uint64_t)a.n_tiles * a.n_rg;
    if (blocks > 0x7fffffffull) return fail(net, SDNN_EINVAL, "grid too large");
    a.n_vblocks = (uint32_t)blocks;
    uint64_t g = std::min<uint64_t>(blocks, (uint64_t)net->occ_panel[MODE][ri] * (uint64_t)net->n_cu);
    if (g >= 8 && g < blocks) g &= ~(uint64_t)7;
    int n_cols_arg = n_cols;
    void *args[] = {(void *)&a, (void *)&n_cols_arg, (void *)&panel};
    HIP_TRY(net, hipLaunchKernel(fn, dim3((unsigned)g), dim3(BLOCK_THREADS), args, 0, stream));
    HIP_TRY(net, hipGetLastError());
    return SDNN_OK;
}

// The several-rows-per-wavefront kernels form byte offsets as (24-bit column) x (24-bit row pitch) in 32 bits, up to and
// including those of the row past the end.
static bool rows_addressable(int n_cols, int ld)
{
    return n_cols < (1 << 24) && ld < (1 << 22) && 4 * ((int64_t)n_cols + 2) * ld < ((int64_t)1 << 32);
}
// Lanes per row of the several-rows-per-wavefront kernels that a tile of `width` samples needs.
static int lanes_per_row(int width) { return width <= 16 ? 4 : width <= 32 ? 8 : width <= 64 ? 16 : width <= 128 ? 32 : 64; }
// The same, doubled while the wavefronts are fewer than the chip's SIMDs (idle lanes cost nothing there: 4096 neurons,
// 16 samples 5.4 -> 4.6 us).
static int spread_lanes(const sdnn_net *net, int G, int n_rows)
{
    while (G < 32 && (int64_t)n_rows * (2 * G) <= (int64_t)64 * 4 * net->n_cu) G *= 2;
    return G;
}
// Samples per tile of the forward product: as many as let a tile's operand stay in an XCD's L2 (launch_spmm has the figures).
static int forward_tile(int n_cols)
{
    int tile = 128;
    while (tile > 32 && 4 * (int64_t)n_cols * tile > 4000000) tile /= 2;
    return tile;
}
template <int G>
static const void *rows_fn_act(int act)
{
    return act == ACT_SIGMOID ? (const void *)k_rows<G, ACT_SIGMOID> : (const void *)k_rows<G, ACT_RELU_CAP>;
}
static const void *rows_fn(int G, int act)
{
    return G == 4 ? rows_fn_act<4>(act) : G == 8 ? rows_fn_act<8>(act) : G == 16 ? rows_fn_act<16>(act) : rows_fn_act<32>(act);
}

// in / out: rows of ld_in / ld_out floats.  sub_begin .. sub_end: the launch covers these samples only (sub_begin a
// multiple of SUB_ALIGN, or of 64 where every layer takes the panel sweep for all but the narrowest blocks; sub_end == 0: all
// of them).
template <int MODE>
static int launch_spmm(sdnn_net *net, const LayerDev &d, const float *in, int ld_in, float *out, int ld_out,
                       const float *aux, int B, hipStream_t stream, const int32_t *n_live = nullptr, int32_t *flags = nullptr,
                       int sub_begin = 0, int sub_end = 0)
{
    if (sub_end == 0) sub_end = B;
    SpmmArgs a;
    a.n_live = n_live;
    a.flags = flags;
    if (MODE == 0) {
        a.row_ptr = d.row_ptr; a.idx = d.col_idx; a.perm = nullptr; a.sched = d.sched;
        a.n_rows = d.n_out;
    } else {
        a.row_ptr = d.t_row_ptr; a.idx = d.t_row_idx; a.perm = d.t_perm; a.sched = d.t_sched;
        a.n_rows = d.n_in;
    }
    a.vals = d.vals; a.in = in; a.out = out; a.aux = aux; a.B = B; a.ld_in = ld_in; a.ld_out = ld_out;
    a.cap = net->cfg.act_cap; a.act = net->cfg.activation;
    if (a.n_rows == 0) return SDNN_OK;
    const int n_cols = MODE == 0 ? d.n_in : d.n_out;
    a.n_cols = n_cols;
    const size_t in_bytes = 4 * (size_t)n_cols * (size_t)ld_in;
    if (in_bytes >= ((size_t)1 << 32))
        return fail(net, SDNN_EINVAL, "activation block of %zu bytes exceeds 4 GiB: use a smaller B", in_bytes);
    a.in_bytes = (uint32_t)in_bytes;
    if (B == 1 && net->b1) {
        const int o = MODE;
        SpmvLmArgs b;
        memset(&b, 0, sizeof b);
        b.cs = d.b1_cs[o]; b.row = d.b1_row[o]; b.lm = (const uint4 *)d.b1_lm[o]; b.in = in; b.in_bytes = a.in_bytes; b.aux = aux; b.out = out;
        b.lm_bytes = 0xffffffffu; // every chunk that the table names is there
        b.cap = a.cap; b.act = a.act;
        if (net->b1_wide) hipLaunchKernelGGL((k_spmv_lm<MODE, true, true>), dim3((unsigned)d.b1_blocks[o]), dim3(64), 0, stream, b);
        else if (MODE == 1 && d.b1_blocks[o] > 3 * net->n_cu)
            hipLaunchKernelGGL((k_spmv_lm<2 * MODE, false, true>), dim3((unsigned)d.b1_blocks[o]), dim3(64), 0, stream, b);
        else hipLaunchKernelGGL((k_spmv_lm<MODE, false, true>), dim3((unsigned)d.b1_blocks[o]), dim3(64), 0, stream, b);
        HIP_TRY(net, hipGetLastError());
        return SDNN_OK;
    }
    if (B == 1) {
        const int64_t nnz = d.nnz;
        if (a.n_rows >= SPMV_STAGE_MIN_ROWS && nnz < 128 * (int64_t)a.n_rows) {
            // short rows, wide layer: R consecutive rows per 64-lane workgroup (measured: 8, and 16 from 32768 rows)
            const int R = a.n_rows >= 32768 ? 16 : 8;
            hipLaunchKernelGGL((k_spmv_stage<MODE, 8>), dim3((unsigned)((a.n_rows + R - 1) / R)), dim3(64), 0, stream, a, R);
        } else if (a.n_rows <= 16384) // a wavefront per row while that still fits the chip a few times over
            hipLaunchKernelGGL(k_spmv_wave<MODE>, dim3((unsigned)((a.n_rows + WAVES_PER_BLOCK - 1) / WAVES_PER_BLOCK)),
                               dim3(BLOCK_THREADS), 0, stream, a);
        else
            hipLaunchKernelGGL(k_spmv<MODE>, dim3((unsigned)((a.n_rows + 255) / 256)), dim3(256), 0, stream, a);
        HIP_TRY(net, hipGetLastError());
        return SDNN_OK;
    }
    const int l = (int)(&d - net->layers.data());
    const int width = sub_end - sub_begin;
    // Wide layers with short rows: when a 64-sample tile of the operand (n_cols x 256 B) is at least twice
    // the chip's eight L2s, the panel sweep is faster (measured, 65536 columns: forward of a 64-sample
    // minibatch 64.8 -> 53.6 us per layer, inference in blocks of 1024 samples 217 -> 179 ms per 24 layers;
    // 16384 columns and fewer: slower than the kernels below).  sdnn_config.panel_cols overrides.
    if (!n_live && !flags && net->cfg.panel_cols >= 0) {
        int panel = net->cfg.panel_cols;
        // (not where reorder_rows has found clusters: their locality comes from the row order, which the
        // panel kernel's larger workgroups would deal to the XCDs differently: 9.8 vs 6.8 ms on a structured net)
        if (panel == 0 && width > PANEL_MIN_SAMPLES && (int64_t)n_cols * 256 >= ((int64_t)8 << 20) && d.nnz > 0 && !net->clustered[MODE][l])
            panel = width > 448 ? 6144 : 8192; // eight or more tiles: every XCD sweeps tiles of its own
        if (panel > 0 && net->max_len[MODE][l] <= 64)
            return launch_spmm_panel<MODE>(net, d, a, B, panel, stream, sub_begin, sub_end);
    }
    const bool long_rows = (int64_t)d.nnz >= 128 * (int64_t)a.n_rows;
    // Forward over short rows: several rows per wavefront, in tiles of 128 samples, or of 64 or 32 where the operand of a
    // wider tile would not fit an XCD's L2 (forward of 128 / 256 samples, us per layer, tiles of 32 / 64 / 128: 10007
    // neurons 13.0 / 12.7 / 13.0 and 22.2 / 21.6 / 23.8; 16384: 17.7 / 19.1 / 25.7 and 31.8 / 35.3 / 48.3; 30000: 35.6 / 44.7 / 55.4
    // and 67.8 / 85.9 / 108).  Few rows and few samples: a wavefront per row keeps more of the chip busy (1024
    // neurons, 64 samples: 4.6 vs 4.7).  Long rows are too uneven to share a wavefront.
    // (A launch holds less than 2^32 threads, 2^24 of these workgroups of 1024 results each: k_spmm walks its blocks.)
    if (MODE == 0 && !n_live && !flags && !long_rows && (width > 64 || a.n_rows >= 2048) && !net->clustered[MODE][l] &&
        rows_addressable(n_cols, ld_in) && ((int64_t)a.n_rows + 64) * (width + 128) < ((int64_t)1 << 34)) {
        const int tile = forward_tile(n_cols);
        const int G = sub_begin == 0 && width <= tile ? spread_lanes(net, lanes_per_row(width), a.n_rows) : lanes_per_row(std::min(tile, width));
        const int rows_per_block = 64 / G * WAVES_PER_BLOCK;
        a.tile_base = (uint32_t)(sub_begin / (4 * G));
        a.n_tiles = (uint32_t)((width + 4 * G - 1) / (4 * G));
        a.n_rg = (uint32_t)((a.n_rows + rows_per_block - 1) / rows_per_block);
        const uint64_t grid = (uint64_t)a.n_tiles * a.n_rg;
        void *args[] = {(void *)&a};
        HIP_TRY(net, hipLaunchKernel(rows_fn(G, net->cfg.activation), dim3((unsigned)grid), dim3(BLOCK_THREADS), args, 0, stream));
        HIP_TRY(net, hipGetLastError());
        return SDNN_OK;
    }
    int V = pick_v_spmm(B, ld_in, ld_out, in, out);
    // a sub-block starts at a multiple of 64 samples: in a pass cut for the panel sweep the last one comes here if it is narrow
    while (sub_begin % (64 * V) != 0) V /= 2;
    a.tile_base = (uint32_t)(sub_begin / (64 * V));
    a.n_tiles = (uint32_t)((width + 64 * V - 1) / (64 * V));
    if (a.n_tiles == 0) return SDNN_OK;
    a.n_rg = (uint32_t)((a.n_rows + WAVES_PER_BLOCK - 1) / WAVES_PER_BLOCK);
    const uint64_t blocks = (uint64_t)a.n_tiles * a.n_rg;
    if (blocks > 0x7fffffffull) return fail(net, SDNN_EINVAL, "grid too large");
    a.n_vblocks = (uint32_t)blocks;
    // Measured policy.  Short rows (a few tens of entries): 8 gathers in flight per lane (16 costs a
    // third of the occupancy) and a grid of what the chip holds at once, whose workgroups walk the
    // virtual blocks.  Long, uneven rows (hundreds of entries): 16 in flight and one workgroup per
    // virtual block, so that the hardware hands out the rows, longest first, as wavefronts retire.
    uint64_t g = blocks;
    // short rows and a few batch tiles (shared by all XCDs): workgroups are dealt row groups and walk the tiles
    const bool tiles_inner = !long_rows && a.n_tiles >= 2 && a.n_tiles < 8;
    if (tiles_inner) g = a.n_rg;
    const int U = long_rows ? 16 : 8;
    const void *fn = spmm_fn<MODE>(V, U, tiles_inner, net->cfg.activation);
    if (!long_rows) {
        int &per_cu = net->occ_spmm[MODE][V == 4 ? 2 : V == 2 ? 1 : 0][tiles_inner ? 1 : 0][U == 16 ? 1 : 0];
        if (per_cu == 0) {
            HIP_TRY(net, hipOccupancyMaxActiveBlocksPerMultiprocessor(&per_cu, fn, BLOCK_THREADS, 0));
            if (per_cu < 1) per_cu = 1;
        }
        g = std::min(g, (uint64_t)per_cu * (uint64_t)net->n_cu);
    }
    // a walking grid keeps virtual block id % 8 == workgroup id % 8 (XCD-wise tiles); one that covers every block at once
    // is not cut (the few blocks left over would run by themselves: 1500 rows 5.7 instead of 4.3 us)
    if (g >= 8 && g < (tiles_inner ? (uint64_t)a.n_rg : blocks)) g &= ~(uint64_t)7;
    void *args[] = {(void *)&a};
    HIP_TRY(net, hipLaunchKernel(fn, dim3((unsigned)g), dim3(BLOCK_THREADS), args, 0, stream));
    HIP_TRY(net, hipGetLastError());
    return SDNN_OK;
}

// A block of n rows of B floats copied between arrays of different row strides; columns B .. Bp - 1 of dst are zeroed.
static int launch_copy_rows(sdnn_net *net, const float *src, int ld_src, float *dst, int ld_dst, int n, int B, int Bp, hipStream_t stream)
{
    if (n == 0) return SDNN_OK;
    if (ld_src == B && ld_dst == B && Bp == B) {
        HIP_TRY(net, hipMemcpyAsync(dst, src, 4 * (size_t)n * B, hipMemcpyDeviceToDevice, stream));
        return SDNN_OK;
    }
    const int w = row_threads_log2(Bp);
    hipLaunchKernelGGL(k_copy_rows, dim3(row_blocks(n, w)), dim3(256), 0, stream, src, ld_src, dst, ld_dst, n, B, Bp, w);
    HIP_TRY(net, hipGetLastError());
    return SDNN_OK;
}

// What a forward pass over B samples takes with a launch per layer, in seconds: 4.4 us per layer to launch, fetch the
// entries and store, plus the longer of two things: the gathered rows, in whole tiles of samples, at the rate that the
// memory they come from delivers, and the chain of gathers of the longest row.
static double per_layer_forward_seconds(const sdnn_net *net, int B)
{
    double t = 0.0;
    for (int l = 0; l < net->n_layers; ++l) {
        const LayerDev &d = net->layers[l];
        const double nnz = (double)d.nnz, longest = net->max_len[0][l];
        if (B == 1) { // a lane per row
            t += 3.7e-6 + 5.1e-12 * nnz + 28e-9 * std::max(0.0, longest - 32.0);
            continue;
        }
        double rate, chain;
        int width;
        if (net->cfg.panel_cols >= 0 && B > PANEL_MIN_SAMPLES && (int64_t)d.n_in * 256 >= ((int64_t)8 << 20) && longest <= 64 && !net->clustered[0][l]) {
            width = (B + 63) & ~63; // k_spmm_panel (40000, 50000, 65536 neurons: 9.6, 9.6, 11.3e12)
            rate = 10e12;
            chain = 28e-9;
        } else if ((int64_t)d.nnz >= 128 * (int64_t)d.n_out) { // a wavefront per row
            width = B > 128 ? (B + 255) & ~255 : B > 64 ? 128 : 64;
            rate = B > 128 ? 22e12 : B > 64 ? 17e12 : 14e12;
            chain = B > 64 ? 50e-9 : 28e-9;
        } else if (B <= 64 && d.n_out < 2048) {
            width = 64;
            rate = 20e12;
            chain = 28e-9;
        } else { // several rows per wavefront
            const int tile = std::min(forward_tile(d.n_in), 4 * lanes_per_row(B));
            width = (B + tile - 1) / tile * tile;
            rate = (B > 256 ? 0.9 : 1.0) * (23e12 - 9e12 * std::min(std::max((d.n_in - 5000) / 27768.0, 0.0), 1.0));
            chain = 54e-9;
        }
        t += 4.4e-6 + std::max(4.0 * nnz * width / rate, chain * longest);
    }
    return t;
}

// Samples per workgroup with which the single-launch LDS-resident forward is the faster way to run this block of B
// samples, 0: a launch per layer is.  A workgroup takes 0.8 us per layer plus 3.5 / 3.9 / 6.2 ns per wavefront-wide entry with
// 1 / 2 / 4 samples; a CU runs one workgroup at a time, and where few of them share the stream of W (a round of fewer than 96),
// they wait for it: up to 1 us per layer and 0.35 ns per entry more.
// Against both paths measured at 1500 to 32000 neurons of 32 entries and 16 to 1100 samples (24 layers), and at 1024 to 8192 neurons
// of uneven rows (a tenth of the columns in the mean), the choice costs at most 2 %.  us per pass, per layer / single launch:
// 3001 neurons 141 / 153 (64 samples), 169 / 150 (100); 8000 neurons 311 / 358 (150), 388 / 359 (200); 16384 neurons 668 / 717
// (200), 948 / 793 (300); 32000 neurons 1197 / 1382 (150), 1604 / 1385 (200), 2374 / 2987 (300: a second round), 3526 / 2907 (450);
// uneven rows, 1024 neurons 107 / 49 (100), 2000 neurons 129 / 143 (64), 172 / 140 (100).
// shifted: the single launch cannot run, d_XL lies across d_X0.  *seconds (not NULL): what the faster one of those that can run takes.
static int lds_forward_samples(const sdnn_net *net, int B, bool shifted = false, double *seconds = nullptr)
{
    const double per_layer = seconds || net->cfg.lds_forward == SDNN_LDS_AUTO ? per_layer_forward_seconds(net, B) : 0.0;
    if (seconds) *seconds = per_layer;
    if (shifted || !net->lm || net->cfg.lds_forward == SDNN_LDS_OFF) return 0;
    for (const LayerDev &d : net->layers)
        if (d.n_out == 0) return 0; // an empty layer: leave it to the general path
    static const double entry[3] = {3.5e-9, 3.9e-9, 6.2e-9};
    const double L = net->n_layers, entries = LDS_CHUNK * (double)net->lm_chunks;
    int best = 0;
    double t_best = 0.0;
    for (int k = 0; k < 3; ++k) {
        const int T = 1 << k, n_cu = std::max(net->n_cu, 1);
        if (T * net->lm_max_pos > LDS_MAX_FLOATS) break;
        const int wgs = (B + T - 1) / T, rounds = (wgs + n_cu - 1) / n_cu, last = wgs - (rounds - 1) * n_cu;
        const double t = rounds * (L * 0.8e-6 + entries * entry[k]) + std::max(0.0, 1.0 - last / 96.0) * (L * 1e-6 + entries * 0.35e-9);
        if (!best || t < t_best) { best = T; t_best = t; }
    }
    if (!best) return 0;
    if (seconds) *seconds = std::min(t_best, per_layer);
    if (net->cfg.lds_forward == SDNN_LDS_ON) return best;
    return t_best < per_layer ? best : 0;
}

// Whether the pass in panels (k_fwd_pan) is the faster way to run B samples than one that takes `other` seconds.  Per layer 3.5 us
// to launch and, for every round of workgroups, 6 us plus 1.1 us per panel and range (they share an XCD's L2) plus 4.2 ns
// per wavefront-wide slot; and the two passes that turn the samples around.  Measured, us per layer without / in panels (24 layers of 32 entries):
// 20001 neurons 23.3 / 28.3 (100 samples), 37.1 / 30.4 (200), 52.9 / 53.8 (300: a second round), 110 / 90 (700); 32768 neurons
// 27.9 / 45.8 (64), 62.8 / 46.8 (100), 123 / 96 (512); 40000 neurons 38.7 / 42.5 (64), 73.1 / 45.7 (100), 309 / 131 (512);
// 65536 neurons 53.0 / 64.5 (64), 136 / 66.4 (100), 137 / 114 (150), 849 / 476 (1024).
static bool pan_forward_pays(const sdnn_net *net, int B, double other)
{
    if (net->pan.empty() || B < 2) return false;
    const int n_cu = std::max(net->n_cu, 1);
    double t = 10e-6 + 8.0 * (net->pan.front().g.in_pos + (double)net->pan.back().g.out_pos) * B / 4e12;
    for (const sdnn_net::Pan &f : net->pan) {
        const int64_t wgs = (int64_t)((B + 15) / 16 * 8) * f.g.n_ranges, rounds = (wgs + n_cu - 1) / n_cu;
        t += 3.5e-6 + (double)rounds * (6e-6 + 1.1e-6 * f.g.n_panels * f.g.n_ranges + 4.2e-9 * LDS_WAVES * f.depth);
    }
    return t < other;
}

static LdsForward lds_args(const sdnn_net *net, int l0, int l1, const float *in, int ld_in, float *out, int ld_out, int B)
{
    LdsForward a;
    memset(&a, 0, sizeof a);
    a.tab = net->lm_layers; a.lm_cs = net->lm_cs; a.lm = net->lm; a.lm_bias = net->lm_bias; a.lm_row = net->lm_row;
    a.lm_bytes = (unsigned)(LDS_CHUNK_BYTES * (net->lm_chunks + 1));
    a.l0 = l0; a.l1 = l1; a.n_in = net->layers[l0].n_in;
    a.in = in; a.out = out; a.ld_in = ld_in; a.ld_out = ld_out; a.B = B;
    a.cap = net->cfg.act_cap; a.max_pos = net->lm_max_pos; a.two = net->lm_two;
    return a;
}

// Whether a block of n_a rows of B floats at a and one of n_b rows at b share memory.
static bool overlap(const float *a, int n_a, const float *b, int n_b, int B)
{
    const uintptr_t pa = (uintptr_t)a, pb = (uintptr_t)b;
    return pa < pb + 4 * (size_t)n_b * B && pb < pa + 4 * (size_t)n_a * B;
}

// Eq. 3 for l = 1..L.  Inference nets stage the activations between the layers in ping / pong
// (each at least 4 * max_n * B bytes); training nets keep every X_l in the workspace and ignore them.
// Width in samples of the sub-blocks that an inference pass is cut into, 0 = one piece.  A sub-block's share of an
// activation buffer is held to SUB_BYTES; the width is a multiple of SUB_ALIGN (the widest tile of the product
// kernels), or of 64 where every layer takes the panel sweep (64-sample tiles; a last block of at most PANEL_MIN_SAMPLES goes to
// other kernels, whose tiles then have to start at its first sample).
#define SUB_BYTES ((int64_t)16 << 20)
#define SUB_ALIGN 256
static int sub_block_width(const sdnn_net *net, int B)
{
    if ((int64_t)net->max_n * B * 4 <= 2 * SUB_BYTES || B == 1) return 0;
    int64_t nnz = 0, rows = 0; // long rows: bound by the L1 and the VALU, not by where the operand comes from (slower: 61 -> 67 ms)
    for (const LayerDev &d : net->layers) { nnz += d.nnz; rows += d.n_out; }
    if (nnz >= 128 * rows) return 0;
    bool all_panel = net->cfg.panel_cols >= 0;
    for (int l = 0; l < net->n_layers && all_panel; ++l) {
        const LayerDev &d = net->layers[l];
        const bool wide = net->cfg.panel_cols > 0 || ((int64_t)d.n_in * 256 >= ((int64_t)8 << 20) && d.nnz > 0 && !net->clustered[0][l]);
        all_panel = wide && net->max_len[0][l] <= 64;
    }
    const int align = all_panel ? 64 : SUB_ALIGN;
    int64_t w = SUB_BYTES / (4 * (int64_t)net->max_n) / align * align;
    if (w < align) w = align;
    return w >= B ? 0 : (int)w;
}

// The pass in panels: samples turned to pairs, a launch per layer, and back.
static int forward_pan(sdnn_net *net, const float *d_X0, int B, float *d_XL, hipStream_t stream, float *ping, float *pong)
{
    const bool sig = net->cfg.activation == ACT_SIGMOID;
    const void *const one = sig ? (const void *)k_fwd_pan<ACT_SIGMOID, false> : (const void *)k_fwd_pan<ACT_RELU_CAP, false>;
    const void *const stay = (const void *)k_fwd_pan<ACT_RELU_CAP, true>;
    if (!net->pan_attr_set) { // more than the default 64 KiB of dynamic LDS per workgroup
        HIP_TRY(net, hipFuncSetAttribute(one, hipFuncAttributeMaxDynamicSharedMemorySize, 8 * (PAN_POS + 1)));
        HIP_TRY(net, hipFuncSetAttribute(stay, hipFuncAttributeMaxDynamicSharedMemorySize, 8 * (PAN_POS + 1)));
        net->pan_attr_set = true;
    }
    const int n_pairs = (B + 1) / 2, tiles = (B + 63) / 64;
    const PanLayer &g0 = net->pan.front().g, &gl = net->pan.back().g;
    hipLaunchKernelGGL(k_pan_turn<true>, dim3((unsigned)((g0.in_pos + 63) / 64), (unsigned)tiles), dim3(256), 0, stream,
                       (float *)d_X0, B, net->layers[0].n_in, B, (float2 *)ping, g0.in_pos, (const int32_t *)nullptr);
    HIP_TRY(net, hipGetLastError());
    for (const sdnn_net::Pan &f : net->pan) {
        PanForward a;
        a.stream = f.stream; a.seg = f.seg; a.ends = f.ends; a.bias = f.bias; a.in = (const float2 *)ping; a.out = (float2 *)pong;
        a.stream_bytes = (uint32_t)((f.g.halves + 2) * LDS_HALF_BYTES);
        a.in_pos = f.g.in_pos; a.out_pos = f.g.out_pos; a.panel = f.g.panel; a.n_panels = f.g.n_panels;
        a.range = f.g.range; a.n_ranges = f.g.n_ranges; a.nb = f.g.nb; a.n_pairs = n_pairs; a.cap = net->cfg.act_cap;
        void *args[] = {(void *)&a};
        // From eight pieces (a range of a pair) for five places on, a workgroup takes one after the other: the first panel of the next one comes
        // while the results of this one are stored, and its first halves of W before that.  With fewer, one look more at every half costs
        // what that gives, and with the sigmoid, whose exp() needs the registers (us per pass, a workgroup per piece / staying: 65536
        // neurons, 200 samples (13 pieces for 8 places), 8 layers 884 / 860; 40001, 1024 samples 2287 / 2215; 80001, 300 samples 1368 / 1332; 45000,
        // 257 samples (3 for 2), 6 layers 530 / 557; 32768, 200 samples (a piece each) 350 / 357, 300 (19 for 16) 669 / 677, 1024 1570 / 1584).
        const int pieces = (n_pairs + 7) / 8 * f.g.n_ranges, places = std::max(net->n_cu / 8, 1); // of an XCD
        const bool stays = !sig && 5 * (int64_t)pieces >= 8 * (int64_t)places;
        HIP_TRY(net, hipLaunchKernel(stays ? stay : one, dim3(8u * (unsigned)(stays ? places : pieces)), dim3(64 * LDS_WAVES), args, 8 * ((size_t)f.g.panel + 1),
                                     stream));
        std::swap(ping, pong);
    }
    hipLaunchKernelGGL(k_pan_turn<false>, dim3((unsigned)((gl.out_pos + 63) / 64), (unsigned)tiles), dim3(256), 0, stream,
                       d_XL, B, net->layers.back().n_out, B, (float2 *)ping, gl.out_pos, (const int32_t *)net->pan.back().rows);
    HIP_TRY(net, hipGetLastError());
    net->B = B;
    net->state = ST_FORWARD;
    return SDNN_OK;
}

// The forward pass of a training net through k_fwd_long, from d_x0.
static int forward_long(sdnn_net *net, int B, int Bp, int ld, hipStream_t stream)
{
    const void *fn = net->cfg.activation == ACT_SIGMOID ? (const void *)k_fwd_long<ACT_SIGMOID> : (const void *)k_fwd_long<ACT_RELU_CAP>;
    if (!net->long_attr_set) { // more than the default 64 KiB of dynamic LDS per workgroup
        HIP_TRY(net, hipFuncSetAttribute(fn, hipFuncAttributeMaxDynamicSharedMemorySize, 16 * (LONG_POS + 2)));
        net->long_attr_set = true;
    }
    const bool captured = capturing(stream);
    net->long_kept |= captured;
    for (int l = 0, n; l < net->n_layers; l += n) { // runs of layers whose copies are behind
        n = 1;
        if (!net->long_stale[l]) continue;
        while (l + n < net->n_layers && net->long_stale[l + n]) ++n;
        const int rc = launch_long_fill(net, l, n, false, stream);
        if (rc) return rc;
        if (!captured) std::fill_n(net->long_stale.begin() + l, n, 0);
    }
    for (int l = 0; l < net->n_layers; ++l) {
        const LayerDev &d = net->layers[l];
        FwdLong a;
        a.cs = d.b1_cs[0]; a.row = d.b1_row[0]; a.lm = (const uint4 *)d.b1_lm[0]; a.bias = d.bias; a.in = d.X_prev; a.out = d.X;
        a.lm_bytes = net->long_bytes[(size_t)l];
        a.blocks = d.b1_blocks[0]; a.n_in = d.n_in; a.ld = ld; a.B = B; a.cap = net->cfg.act_cap;
        a.groups = Bp / 4;
        const int per = (a.groups + 7) / 8;
        a.n_ranges = std::max(1, std::min(net->n_cu / 8 / per, a.blocks));
        void *args[] = {(void *)&a};
        HIP_TRY(net, hipLaunchKernel(fn, dim3((unsigned)(8 * per * a.n_ranges)), dim3(64 * LDS_WAVES), args, 16 * ((size_t)d.n_in + 2), stream));
    }
    return SDNN_OK;
}

template <int ACT, bool TWO> static const void *lds_fn(int T, int turns)
{
    return T == 4 ? (const void *)k_fwd_lds<4, ACT, true, TWO> : T == 2 ? (const void *)k_fwd_lds<2, ACT, true, TWO>
           : turns & LM_IN_ORDER ? (const void *)k_fwd_lds<1, ACT, true, TWO> : (const void *)k_fwd_lds<1, ACT, false, TWO>;
}

// `ld`: floats per row of the activations between the layers.
static int forward_impl(sdnn_net *net, const float *d_X0, int32_t B, float *d_XL, void *stream_, float *ping,
                        float *pong, int ld)
{
    const bool training = net->cfg.training != 0;
    hipStream_t stream = (hipStream_t)stream_;
    net->state = ST_IDLE;
    const int L = net->n_layers;
    // a workgroup reads and writes columns of its own: d_XL may be d_X0 itself, but not lie across it
    const bool shifted = d_XL && d_XL != d_X0 && overlap(d_X0, net->layers[0].n_in, d_XL, net->layers[L - 1].n_out, B);
    double other = 0.0;
    const int T = lds_forward_samples(net, B, shifted, net->pan.empty() ? nullptr : &other);
    if (ping == net->d_ping && pan_forward_pays(net, B, other)) // (in the workspace's buffers: what it keeps there is larger than X)
        return forward_pan(net, d_X0, B, d_XL, stream, ping, pong);
    if (T) {
        const bool sig = net->cfg.activation == ACT_SIGMOID;
        const int ti = T == 1 ? 0 : T == 2 ? 1 : 2;
        const void *const fns[2][2] = {{lds_fn<ACT_RELU_CAP, false>(T, net->turns), lds_fn<ACT_RELU_CAP, true>(T, net->turns)},
                                       {lds_fn<ACT_SIGMOID, false>(T, net->turns), lds_fn<ACT_SIGMOID, true>(T, net->turns)}};
        const void *fn = fns[sig ? 1 : 0][net->lm_two ? 1 : 0]; // (a net has one of those for T)
        const size_t lds_bytes = sizeof(float) * (size_t)T * ((size_t)net->lm_max_pos + net->lm_two + 1);
        if (!net->lds_attr_set[ti]) { // more than the default 64 KiB of dynamic LDS per workgroup
            HIP_TRY(net, hipFuncSetAttribute(fn, hipFuncAttributeMaxDynamicSharedMemorySize, 4 * (LDS_MAX_FLOATS + 4)));
            net->lds_attr_set[ti] = true;
        }
        LdsForward a = lds_args(net, 0, L, d_X0, B, d_XL, B, B);
        a.vec_io = (B % T == 0 && aligned(d_X0, 4 * T) && aligned(d_XL, 4 * T)) ? 1 : 0;
        a.turns = (net->turns & T) && (B + T - 1) / T <= 2 * net->n_cu;
        void *args[] = {(void *)&a};
        HIP_TRY(net, hipLaunchKernel(fn, dim3((unsigned)((B + T - 1) / T)), dim3(64 * LDS_WAVES), args, lds_bytes, stream));
        HIP_TRY(net, hipGetLastError());
        net->B = B;
        net->state = ST_FORWARD;
        return SDNN_OK;
    }
    if (B == 1 && !training && net->lm && net->cfg.panel_cols <= 0) { // a lane per row over the same copy of W
        const float *in = d_X0;
        size_t n_in = (size_t)net->layers[0].n_in;
        for (int l = 0; l < L; ++l) {
            const bool last = l == L - 1;
            SpmvLmArgs b;
            memset(&b, 0, sizeof b);
            b.cs = net->lm_cs; b.lm = net->lm; b.lm_bytes = (unsigned)(LDS_CHUNK_BYTES * (net->lm_chunks + 1));
            b.lm_row = last ? net->lm_row : nullptr; b.aux = net->lm_bias;
            const int first = l & 1 ? net->lm_two : 0; // the position that the copy has for the operand's first
            b.in = in - first; b.in_bytes = (unsigned)(4 * (n_in + first)); b.out = last ? d_XL : ((l & 1) ? pong : ping);
            b.cap = net->cfg.act_cap; b.act = net->cfg.activation;
            b.nb = net->lm_tab[l].nb; b.tab_cs = net->lm_tab[l].cs; b.tab_pos = net->lm_tab[l].pos;
            n_in = (size_t)net->lm_tab[l].n_pos;
            in = b.out;
            if (b.nb > 0) hipLaunchKernelGGL((k_spmv_lm<0, false, false>), dim3((unsigned)(LDS_WAVES * b.nb)), dim3(64), 0, stream, b);
            HIP_TRY(net, hipGetLastError());
        }
        net->B = B;
        net->state = ST_FORWARD;
        return SDNN_OK;
    }
    const float *in = d_X0;
    int ld_in = B;
    const int Bp = ld < padded_batch(B) ? B : padded_batch(B);
    if (training) {
        const int rc = launch_copy_rows(net, d_X0, B, net->d_x0, ld, net->layers[0].n_in, B, Bp, stream);
        if (rc) return rc;
        in = net->d_x0;
        ld_in = ld;
    }
    // Inference on large activation blocks: the samples are independent (the columns of X, Section 5.1), so the
    // block is taken through all layers in sub-blocks whose two activation buffers stay in the memory-side
    // cache (what a layer wrote is what the next one gathers): measured on 65536-neuron layers, blocks of 1024
    // samples: 179 ms per 24 layers in one piece, 161 ms in sub-blocks of 64; 16384 neurons, 4096 samples: 41.5 ms
    // per 48 layers in one piece, 39.1 in sub-blocks of 256.
    // (Not where d_XL lies across d_X0: a sub-block's results would replace inputs of the later ones.)
    const int sub_w = training || shifted ? 0 : sub_block_width(net, B);
    if (sub_w > 0) {
        for (int s0 = 0; s0 < B; s0 += sub_w) {
            const int s1 = std::min(B, s0 + sub_w);
            const float *sin = d_X0;
            for (int l = 0; l < L; ++l) {
                const LayerDev &d = net->layers[l];
                float *out = l == L - 1 ? d_XL : ((l & 1) ? pong : ping);
                const int rc = launch_spmm<0>(net, d, sin, l == 0 ? B : ld, out, l == L - 1 ? B : ld, d.bias, B, stream, nullptr, nullptr, s0, s1);
                if (rc) return rc;
                sin = out;
            }
        }
        net->B = B;
        net->state = ST_FORWARD;
        return SDNN_OK;
    }
    const bool single = training && train_lds(net, B);
    if (single) {
        const int rc = launch_train_lds(net, 0, B, Bp, ld, stream);
        if (rc) return rc;
    }
    // (operands of 4 GiB, of LONG_POS neurons at most here, are launch_spmm's to refuse)
    const bool by_four = training && !single && (ld & 3) == 0 && 4 * (int64_t)LONG_POS * ld < ((int64_t)1 << 32) && long_forward(net, B);
    if (by_four) {
        const int rc = forward_long(net, B, Bp, ld, stream);
        if (rc) return rc;
    }
    for (int l = 0; l < (single || by_four ? 0 : L); ++l) {
        const LayerDev &d = net->layers[l];
        float *out = training ? d.X : (l == L - 1 ? d_XL : ((l & 1) ? pong : ping));
        const int ld_out = !training && l == L - 1 ? B : ld;
        const int rc = launch_spmm<0>(net, d, in, ld_in, out, ld_out, d.bias, B, stream);
        if (rc) return rc;
        in = out;
        ld_in = ld_out;
    }
    if (training && d_XL) {
        const int rc = launch_copy_rows(net, net->layers[L - 1].X, ld, d_XL, B, net->layers[L - 1].n_out, B, B, stream);
        if (rc) return rc;
    }
    net->B = B;
    net->Bp = Bp;
    net->ld = ld;
    net->state = ST_FORWARD;
    return SDNN_OK;
}

static int check_forward_args(sdnn_net *net, const float *d_X0, int32_t B, const float *d_XL)
{
    if (!net) return fail(nullptr, SDNN_EINVAL, "net is NULL");
    if (!d_X0) return fail(net, SDNN_EINVAL, "d_X0 is NULL");
    if (B < 1 || B > net->cfg.max_batch)
        return fail(net, SDNN_EINVAL, "B = %d outside 1..max_batch = %d", B, net->cfg.max_batch);
    if (!net->cfg.training && !d_XL) return fail(net, SDNN_EINVAL, "d_XL is NULL");
    return SDNN_OK;
}

extern "C" int sdnn_forward(sdnn_net *net, const float *d_X0, int32_t B, float *d_XL, void *stream_)
{
    const int rc = check_forward_args(net, d_X0, B, d_XL);
    if (rc) return rc;
    return forward_impl(net, d_X0, B, d_XL, stream_, net->d_ping, net->d_pong, row_pitch(net->max_n, B));
}

// ---------------------------------------------------------------------------
// sdnn_forward for callers that cannot allocate: the activations between the layers are staged in
// a fixed array that lives in the library's device image, one copy per GPU, instead of in two
// buffers of a caller-allocated workspace.
// ---------------------------------------------------------------------------
extern "C" int sdnn_forward_noalloc(sdnn_net *net, const float *d_X0, int32_t B, float *d_XL, void *stream_)
{
    int rc = check_forward_args(net, d_X0, B, d_XL);
    if (rc) return rc;
    if (net->cfg.training)
        return fail(net, SDNN_ESTATE, "sdnn_forward_noalloc is for inference nets (training = 0): a training net "
                                      "keeps every X_l in its workspace");
    const size_t half = (size_t)SDNN_NOALLOC_SCRATCH_BYTES / 2;
    const size_t need = 4 * (size_t)net->max_n * (size_t)B; // one activation buffer, 256-byte aligned by `half`
    if (need > half)
        return fail(net, SDNN_EINVAL, "sdnn_forward_noalloc: an activation block of %d neurons x %d samples needs "
                                      "%zu bytes, the fixed staging array holds %zu per buffer: use a smaller B",
                    net->max_n, B, need, half);
    void *base = nullptr;
    rc = scratch_address(net, &base);
    if (rc) return rc;
    const int ld = 4 * (size_t)net->max_n * (size_t)row_stride(B) <= half ? row_stride(B) : B;
    return forward_impl(net, d_X0, B, d_XL, stream_, (float *)base, (float *)((char *)base + half), ld);
}


// The pass in stretches of layers with the activations in LDS: after 1, 3, 7, 15, ... times check_every layers and at the last
// check the samples that are left are counted and their columns listed; the next stretch reads those columns and gives each
// workgroup as few of them as fill the chip.  Nothing waits for the host: workgroups past the live samples end at once.
static int skip_dead_lds(sdnn_net *net, const float *d_X0, int B, float *d_XL, int check_every, int32_t *d_n_live, hipStream_t stream)
{
    const int L = net->n_layers, n_last = net->layers[L - 1].n_out, ld = row_pitch(net->max_n, B);
    const int last_check = (L - 1) / check_every * check_every;
    int t_max = 4;
    while (t_max > 1 && t_max * net->lm_max_pos > LDS_MAX_FLOATS) t_max /= 2;
    const size_t lds_bytes = sizeof(float) * (size_t)t_max * ((size_t)net->lm_max_pos + net->lm_two + 1);
    if (!net->lds_part_attr_set) {
        HIP_TRY(net, hipFuncSetAttribute((const void *)k_fwd_lds_part, hipFuncAttributeMaxDynamicSharedMemorySize, 4 * (LDS_MAX_FLOATS + 4)));
        net->lds_part_attr_set = true;
    }
    const unsigned grid = (unsigned)std::max(std::min(B, net->n_cu), (B + t_max - 1) / t_max);
    // slot k & 1 holds the state of stretch k: d_n_live how many samples it takes, d_flags their columns in its input,
    // d_map their numbers in the caller's block
    int32_t *alive = net->d_alive;
    hipLaunchKernelGGL(k_live_columns, dim3(1), dim3(1024), 0, stream, (const int32_t *)nullptr, (const int32_t *)nullptr,
                       (const int32_t *)nullptr, B, net->d_n_live[0], net->d_flags[0], net->d_map[0]);
    HIP_TRY(net, hipGetLastError());
    // d_XL may share memory with d_X0: it is written once d_X0 has been read, by a pass of one stretch through a buffer
    const bool staged = last_check == 0 && overlap(d_X0, net->layers[0].n_in, d_XL, n_last, B);
    const float *in = d_X0;
    int ld_in = B, k = 0, step = check_every;
    for (int l0 = 0; l0 < L; ++k) {
        const bool last = l0 >= last_check;
        int l1 = L;
        if (!last) {
            l1 = std::min(last_check, l0 + step);
            step = (int)std::min<int64_t>(2 * (int64_t)step, 1 << 30) / check_every * check_every;
        }
        float *out = last && !staged ? d_XL : (k & 1) ? net->d_pong : net->d_ping;
        if (last && k > 0) // the samples that have died (a pass of one stretch stores every column)
            hipLaunchKernelGGL(k_fill_f32, dim3(ew_blocks((size_t)n_last * B)), dim3(256), 0, stream, d_XL, (size_t)n_last * B, 0.0f);
        LdsForward a = lds_args(net, l0, l1, in, ld_in, out, last ? B : ld, B);
        a.turns = net->turns;
        a.n_live = net->d_n_live[k & 1];
        a.src_col = net->d_flags[k & 1];
        a.dst_col = last ? net->d_map[k & 1] : nullptr;
        a.alive = last ? nullptr : alive;
        hipLaunchKernelGGL(k_fwd_lds_part, dim3(grid), dim3(64 * LDS_WAVES), lds_bytes, stream, a, net->n_cu);
        if (!last)
            hipLaunchKernelGGL(k_live_columns, dim3(1), dim3(1024), 0, stream, (const int32_t *)alive, net->d_n_live[k & 1], net->d_map[k & 1],
                               B, net->d_n_live[(k + 1) & 1], net->d_flags[(k + 1) & 1], net->d_map[(k + 1) & 1]);
        HIP_TRY(net, hipGetLastError());
        if (staged) HIP_TRY(net, hipMemcpyAsync(d_XL, out, 4 * (size_t)n_last * B, hipMemcpyDeviceToDevice, stream));
        if (last && d_n_live) HIP_TRY(net, hipMemcpyAsync(d_n_live, net->d_n_live[k & 1], 4, hipMemcpyDeviceToDevice, stream));
        in = out;
        ld_in = ld;
        l0 = l1;
    }
    return SDNN_OK;
}

extern "C" int sdnn_forward_skip_dead(sdnn_net *net, const float *d_X0, int32_t B, float *d_XL,
                                      int32_t check_every, int32_t *d_n_live, void *stream_)
{
    if (!net) return fail(nullptr, SDNN_EINVAL, "net is NULL");
    if (!d_X0 || !d_XL) return fail(net, SDNN_EINVAL, "d_X0 or d_XL is NULL");
    if (B < 1 || B > net->cfg.max_batch)
        return fail(net, SDNN_EINVAL, "B = %d outside 1..max_batch = %d", B, net->cfg.max_batch);
    if (check_every < 1) return fail(net, SDNN_EINVAL, "check_every must be >= 1");
    if (net->cfg.training) return fail(net, SDNN_ESTATE, "dead-sample skipping is for inference nets (training = 0)");
    if (net->cfg.activation != SDNN_ACT_RELU_CAP)
        return fail(net, SDNN_ESTATE, "dead-sample skipping needs the ReLU activation (f(0) = 0)");
    if (!net->bias_nonpos)
        return fail(net, SDNN_ESTATE, "dead-sample skipping needs every bias of layers 2..L to be <= 0 "
                                      "(a positive bias revives a dead sample; replaced biases are not inspected)");
    if (B > PACK_MAX_B) return fail(net, SDNN_EINVAL, "B = %d: dead-sample skipping packs blocks of at most %d samples", B, PACK_MAX_B);
    hipStream_t stream = (hipStream_t)stream_;
    net->state = ST_IDLE;
    const int L = net->n_layers;
    if (B > 1 && lds_forward_samples(net, B)) {
        const int rc = skip_dead_lds(net, d_X0, B, d_XL, check_every, d_n_live, stream);
        if (rc) return rc;
        net->B = B;
        return SDNN_OK;
    }
    hipLaunchKernelGGL(k_skip_init, dim3(ew_blocks((size_t)B)), dim3(256), 0, stream, net->d_map[0], net->d_flags[0],
                       net->d_flags[1], net->d_n_live[0], B);
    HIP_TRY(net, hipGetLastError());
    const float *in = d_X0;
    int k = 0; // packing round: its state is in slot k & 1, the next round's in the other slot
    for (int l = 0; l < L; ++l) {
        const LayerDev &d = net->layers[l];
        float *out = (l & 1) ? net->d_pong : net->d_ping;
        // one sample: nothing to pack, this is the plain pass
        const bool check = (l + 1) % check_every == 0 && l + 1 < L && B > 1 && d.n_out > 0;
        const int rc = launch_spmm<0>(net, d, in, B, out, B, d.bias, B, stream, net->d_n_live[k & 1],
                                      check ? net->d_flags[k & 1] : nullptr);
        if (rc) return rc;
        if (check) {
            hipLaunchKernelGGL(k_pack, dim3((unsigned)((d.n_out + PACK_ROWS - 1) / PACK_ROWS)), dim3(256), 0, stream, out,
                               d.n_out, B, net->d_flags[k & 1], net->d_n_live[k & 1], net->d_map[k & 1],
                               net->d_n_live[(k + 1) & 1], net->d_map[(k + 1) & 1], net->d_flags[(k + 1) & 1]);
            HIP_TRY(net, hipGetLastError());
            ++k;
        }
        in = out;
    }
    const int n_last = net->layers[L - 1].n_out;
    if (n_last > 0) {
        hipLaunchKernelGGL(k_fill_f32, dim3(ew_blocks((size_t)n_last * B)), dim3(256), 0, stream, d_XL,
                           (size_t)n_last * B, 0.0f);
        hipLaunchKernelGGL(k_scatter_cols, dim3((unsigned)((B + 255) / 256), (unsigned)((n_last + LIVE_ROWS - 1) / LIVE_ROWS)),
                           dim3(256), 0, stream, in, d_XL, n_last, B, net->d_map[k & 1], net->d_n_live[k & 1]);
        HIP_TRY(net, hipGetLastError());
    }
    if (d_n_live) HIP_TRY(net, hipMemcpyAsync(d_n_live, net->d_n_live[k & 1], 4, hipMemcpyDeviceToDevice, stream));
    net->B = B;
    return SDNN_OK;
}

// Batches of 128 samples on nets of short rows and up to 16384 neurons: the gradient is the sum of two windows of 64, each
// rounded to fp32, as it has been since these batches ran as two halves.  Where the operand is larger than L2 that is a gain
// (two tiles, each with a partial gradient of its own: 16384 neurons 27.5 -> 25.3 us per layer); below, one sum over the whole
// tile would be about as fast (4096 neurons, a step of 120 layers: 2.17 to 2.20 ms), but its other rounding moved the outputs of
// that case's steps by 7e-5 of their norm.  This is the caller's batch: one that is filled up to 128 has one sum over all its
// samples in fp64, rounded once, like every other.
static bool two_windows(const sdnn_net *net)
{
    if (net->B != 128 || (int64_t)net->max_n * 128 > ((int64_t)1 << 21)) return false;
    int64_t nnz = 0, rows = 0;
    for (const LayerDev &d : net->layers) { nnz += d.nnz; rows += d.n_out; }
    return nnz < 128 * rows;
}

// Whether k_bwd_rows can take this layer's Delta: rows of whole 16-byte pieces, within its offsets.
static bool wide_rows(const sdnn_net *net, const LayerDev &d) { return (net->ld & 3) == 0 && rows_addressable(d.n_out, net->ld); }

// Whether a sweep of more than 128 samples, with a wavefront per row either way, goes by scalar loads and matrix products (k_bwd_long).  Its
// start takes a row longer, and it has fewer gathers in flight, which tells where the operand is larger than the L2s: not below 64 entries
// per row, of operands over 10.7 MB only where the rows are the longer the larger it is, and not over 26 MB (with rows of 1024 bytes 16 MB).
// Sweep of all layers, us, k_bwd_rows / k_bwd_long, layers of n neurons of k entries, s samples: n = 1024, k = 64, s = 256 132 / 115; 8192, 64, 256
// 130 / 126; 16000 x 12000, 90, 256 (12.3 MB) 99 / 101; 14000, 64, 224 (12.5 MB) 225 / 231; 14000, 100, 256 (14.3 MB) 267 / 285; 16384, 64, 200 (14.7
// MB) 291 / 298; 16384, 160, 224 458 / 429; 20000, 200, 224 (17.9 MB) 721 / 691; 20000, 1200, 256 (20.5 MB) 2453 / 3057; 25000, 820, 224 (22.4 MB)
// 2156 / 1772; 32768, 200, 224 (29.4 MB) 1037 / 1051; 8192, 820, 256 1014 / 818.  (Steps with 32 entries, 4096 neurons 2954 / 2983, 8001 neurons
// 2255 / 2239.)
static bool bwd_long(const LayerDev &d, uint32_t in_bytes, int B)
{
    const double mb = 1e-6 * in_bytes;
    return mb <= (B > 224 ? 16.0 : 26.0) && (double)d.nnz >= std::max(64.0, 20.0 * mb - 150.0) * d.n_in;
}

// Fused back-propagation + entry gradient of one layer.  store_out = 0 for the first layer (gradient only: there is no
// Delta_0, out may be NULL).
static int launch_bwd_grad(sdnn_net *net, const LayerDev &d, float *out, hipStream_t stream, int store_out)
{
    const int B = net->Bp;
    GradArgs a;
    a.row_ptr = d.t_row_ptr; a.idx = d.t_row_idx; a.perm = nullptr; a.sched = d.t_sched; a.n_rows = d.n_in;
    a.vals = d.vals_t; a.in = d.D; a.out = out; a.aux = d.X_prev; a.B = net->B; a.ld_in = a.ld_out = net->ld; a.cap = net->cfg.act_cap;
    a.act = net->cfg.activation; a.n_live = nullptr; a.flags = nullptr;
    a.g_part[0] = d.G[0]; a.g_part[1] = d.G[1]; a.store_out = store_out;
    if (a.n_rows == 0 || d.nnz == 0) {
        if (d.nnz == 0 && store_out && a.n_rows > 0) // no entries: Delta_{l-1} = 0, nothing to differentiate
            return launch_spmm<1>(net, d, d.D, net->ld, out, net->ld, d.X_prev, net->B, stream);
        return SDNN_OK;
    }
    a.n_cols = d.n_out;
    a.in_bytes = (uint32_t)(4 * (size_t)d.n_out * (size_t)net->ld);
    a.tile_base = 0;
    a.n_tiles = 1;
    a.n_rg = (uint32_t)((a.n_rows + WAVES_PER_BLOCK - 1) / WAVES_PER_BLOCK);
    a.n_vblocks = a.n_rg;
    void *args[] = {(void *)&a};
    if (B <= 64 && ((a.n_rows <= 6144 && (int64_t)d.nnz < 128 * (int64_t)a.n_rows) || !wide_rows(net, d))) {
        // few short rows: a wavefront for each keeps more of the chip busy than several rows per wavefront (4096 rows, 64
        // samples: 7.3 vs 8.2 us; 6500 rows: 9.9 vs 9.0)
        const void *fn = (const void *)k_bwd_grad<8>;
        if (net->occ_grad == 0) {
            HIP_TRY(net, hipOccupancyMaxActiveBlocksPerMultiprocessor(&net->occ_grad, fn, BLOCK_THREADS, 0));
            if (net->occ_grad < 1) net->occ_grad = 1;
        }
        uint64_t g = std::min<uint64_t>(a.n_vblocks, (uint64_t)net->occ_grad * (uint64_t)net->n_cu);
        if (g >= 8 && g < a.n_vblocks) g &= ~(uint64_t)7;
        HIP_TRY(net, hipLaunchKernel(fn, dim3((unsigned)g), dim3(BLOCK_THREADS), args, 0, stream));
        HIP_TRY(net, hipGetLastError());
        return SDNN_OK;
    }
    // two windows: as two tiles (and two partial gradients) where the operand is larger than L2, else in one
    const bool two = net->two_windows;
    int G = lanes_per_row(net->grad_parts == 2 ? 64 : B);
    if (!two) G = spread_lanes(net, G, a.n_rows);
    const int rows_per_block = 64 / G * WAVES_PER_BLOCK;
    a.n_tiles = (uint32_t)net->grad_parts;
    a.n_rg = (uint32_t)((a.n_rows + rows_per_block - 1) / rows_per_block);
    const void *fn = G == 4 ? (const void *)k_bwd_rows<4, false> : G == 8 ? (const void *)k_bwd_rows<8, false>
                     : G == 16 ? (const void *)k_bwd_rows<16, false>
                     : G == 64 ? (bwd_long(d, a.in_bytes, B) ? (const void *)k_bwd_long : (const void *)k_bwd_rows<64, false>)
                     : two ? (const void *)k_bwd_rows<32, true> : (const void *)k_bwd_rows<32, false>;
    HIP_TRY(net, hipLaunchKernel(fn, dim3(a.n_tiles * a.n_rg), dim3(BLOCK_THREADS), args, 0, stream));
    HIP_TRY(net, hipGetLastError());
    return SDNN_OK;
}

// Whether the backward pass over this batch also forms the gradient: the number of partial gradients, 0 = it does not.
static int grad_fusable(const sdnn_net *net, int B)
{
    if (net->layers[0].G[0] == nullptr || B == 1) return 0;
    if (B > 256) return 0;
    for (const LayerDev &d : net->layers)
        if (B > 64 && !wide_rows(net, d)) return 0;
    return net->two_windows && 4 * (int64_t)net->max_n * B > 6500000 ? 2 : 1;
}

extern "C" int sdnn_backward(sdnn_net *net, const float *d_dLoss, void *stream_)
{
    if (!net) return fail(nullptr, SDNN_EINVAL, "net is NULL");
    if (!net->cfg.training) return fail(net, SDNN_ESTATE, "net was not created for training");
    if (net->state != ST_FORWARD)
        return fail(net, SDNN_ESTATE, "sdnn_backward needs a directly preceding sdnn_forward");
    if (!d_dLoss) return fail(net, SDNN_EINVAL, "d_dLoss is NULL");
    hipStream_t stream = (hipStream_t)stream_;
    const int L = net->n_layers, B = net->Bp;
    const LayerDev &last = net->layers[L - 1];
    net->two_windows = two_windows(net);
    const int gp = grad_fusable(net, B);
    for (int l = gp ? 0 : 1; l < L; ++l) { // the operands of the products below: refused before anything is launched
        const LayerDev &d = net->layers[l];
        const size_t bytes = 4 * (size_t)d.n_out * (size_t)net->ld;
        if (d.n_in > 0 && (l > 0 || d.nnz > 0) && bytes >= ((size_t)1 << 32))
            return fail(net, SDNN_EINVAL, "activation block of %zu bytes exceeds 4 GiB: use a smaller B", bytes);
    }
    if (last.n_out > 0) {
        const int w = row_threads_log2(B);
        hipLaunchKernelGGL(k_output_delta, dim3(row_blocks(last.n_out, w)), dim3(256), 0, stream, d_dLoss, last.X, last.D, last.n_out,
                           net->B, net->ld, B, w, net->cfg.act_cap, net->cfg.activation);
        HIP_TRY(net, hipGetLastError());
    }
    net->grad_parts = gp;
    if (gp && net->vals_t_stale) { // the CSR values were replaced or stepped by the separate update since the last sweep
        int max_nnz = 0;
        for (const LayerDev &d : net->layers) max_nnz = std::max(max_nnz, d.nnz);
        for (int l0 = 0; l0 < L && max_nnz > 0; l0 += 65535) {
            const int nl = std::min(65535, L - l0);
            hipLaunchKernelGGL(k_refresh_vals_t, dim3((unsigned)std::min(4096, (max_nnz + 2047) / 2048), (unsigned)nl), dim3(256), 0,
                               stream, net->d_layers + l0);
            HIP_TRY(net, hipGetLastError());
        }
        net->vals_t_stale = false;
    }
    const bool single = !gp && train_lds(net, net->B);
    if (single) {
        const int rc = launch_train_lds(net, 1, net->B, net->Bp, net->ld, stream);
        if (rc) return rc;
    }
    for (int l = L - 1; l >= (gp ? 0 : 1) && !single; --l) {
        const LayerDev &d = net->layers[l];
        // Delta_{l} (0-based l-1) = (W^T Delta_{l+1}) masked by X_{l}
        float *dprev = l >= 1 ? net->layers[l - 1].D : nullptr;
        const int rc = gp ? launch_bwd_grad(net, d, dprev, stream, l >= 1)
                          : launch_spmm<1>(net, d, d.D, net->ld, dprev, net->ld, d.X_prev, net->B, stream);
        if (rc) return rc;
    }
    net->state = ST_BACKWARD;
    return SDNN_OK;
}

static int launch_update(sdnn_net *net, int layer0, int n_layers, float lr, int emit, float *g,
                         float *gb, hipStream_t stream)
{
    int max_rows = 0;
    for (int l = layer0; l < layer0 + n_layers; ++l) max_rows = std::max(max_rows, net->layers[l].n_out);
    if (max_rows == 0) return SDNN_OK;
    const int B = net->Bp;
    if (B == 1) {
        // lanes per row: the power of two that covers the mean row length, 8..64
        int64_t nnz = 0, rows = 0;
        for (int l = layer0; l < layer0 + n_layers; ++l) { nnz += net->layers[l].nnz; rows += net->layers[l].n_out; }
        int lpr_log2 = 3;
        while (lpr_log2 < 6 && ((int64_t)rows << lpr_log2) < nnz) ++lpr_log2;
        const int rows_per_block = WAVES_PER_BLOCK << (6 - lpr_log2);
        for (int l0 = 0; l0 < n_layers; l0 += 65535) {
            const int nl = std::min(65535, n_layers - l0);
            dim3 grid((unsigned)((max_rows + rows_per_block - 1) / rows_per_block), (unsigned)nl);
            hipLaunchKernelGGL(k_update_b1, grid, dim3(BLOCK_THREADS), 0, stream, net->d_layers, layer0 + l0, lpr_log2,
                               lr, net->cfg.update_bias, emit, g, gb);
            HIP_TRY(net, hipGetLastError());
        }
        return SDNN_OK;
    }
    // short rows: a wavefront takes several rows one after the other (fewer, longer-lived wavefronts); long rows: one
    int64_t nnz = 0, rows = 0;
    for (int l = layer0; l < layer0 + n_layers; ++l) { nnz += net->layers[l].nnz; rows += net->layers[l].n_out; }
    const int rpw = nnz < 128 * rows ? 4 : 1; // measured on config 2: 2.49 / 2.37 / 2.32 / 2.33 ms for 1 / 2 / 4 / 8
    const unsigned n_rg = (unsigned)((max_rows + UPD_WAVES * rpw - 1) / (UPD_WAVES * rpw));
    // with many layers, interleave them over the XCDs (one L2 per layer); with few, keep all XCDs on each layer
    const int interleave = n_layers >= 64;
    for (int l0 = 0; l0 < n_layers; l0 += 65535) {
        const int nl = std::min(65535, n_layers - l0);
        dim3 grid(interleave ? 8u * n_rg : n_rg, (unsigned)(interleave ? (nl + 7) / 8 : nl));
        // rows of Delta and X are whole 16-byte pieces, but for the blocks that row_pitch says; long rows: the row of Delta stays
        // in registers
        if (net->ld & 3)
            hipLaunchKernelGGL((k_update<1, 0>), grid, dim3(64 * UPD_WAVES), 0, stream, net->d_layers,
                               layer0 + l0, nl, interleave, rpw, B, net->ld, lr, net->cfg.update_bias, emit, g, gb);
        else if (rpw == 1 && B <= 256)
            hipLaunchKernelGGL((k_update<4, 4>), grid, dim3(64 * UPD_WAVES), 0, stream, net->d_layers,
                               layer0 + l0, nl, interleave, rpw, B, net->ld, lr, net->cfg.update_bias, emit, g, gb);
        else
            hipLaunchKernelGGL((k_update<4, 0>), grid, dim3(64 * UPD_WAVES), 0, stream, net->d_layers,
                               layer0 + l0, nl, interleave, rpw, B, net->ld, lr, net->cfg.update_bias, emit, g, gb);
        HIP_TRY(net, hipGetLastError());
    }
    return SDNN_OK;
}

extern "C" int sdnn_sgd_step(sdnn_net *net, float lr, void *stream_)
{
    if (!net) return fail(nullptr, SDNN_EINVAL, "net is NULL");
    if (!net->cfg.training) return fail(net, SDNN_ESTATE, "net was not created for training");
    if (net->state != ST_BACKWARD)
        return fail(net, SDNN_ESTATE, "sdnn_sgd_step needs a preceding sdnn_backward");
    int rc = SDNN_OK;
    if (net->grad_parts > 0) { // the gradient of the entries is already there
        int max_rows = 0, max_nnz = 0;
        for (const LayerDev &d : net->layers) { max_rows = std::max(max_rows, d.n_out); max_nnz = std::max(max_nnz, d.nnz); }
        for (int l0 = 0; l0 < net->n_layers; l0 += 65535) {
            const int nl = std::min(65535, net->n_layers - l0);
            if (max_nnz > 0) { // a span per workgroup, a multiple of 8 workgroups per layer
                const unsigned gx = (unsigned)((((int64_t)max_nnz + TR_SPAN - 1) / TR_SPAN + 7) & ~(int64_t)7);
                hipLaunchKernelGGL(k_apply<false>, dim3(gx, (unsigned)nl), dim3(TR_THREADS), 0, (hipStream_t)stream_,
                                   net->d_layers + l0, net->grad_parts, lr);
                hipLaunchKernelGGL(k_spread_vals<false>, dim3((unsigned)((max_nnz + TR_CHUNK - 1) / TR_CHUNK), (unsigned)nl),
                                   dim3(TR_THREADS), 0, (hipStream_t)stream_, net->d_layers + l0, (float *)nullptr);
            }
            if (max_rows > 0 && net->cfg.update_bias)
                hipLaunchKernelGGL(k_apply_bias, dim3((unsigned)((max_rows + 16 * WAVES_PER_BLOCK - 1) / (16 * WAVES_PER_BLOCK)), (unsigned)nl),
                                   dim3(BLOCK_THREADS), 0, (hipStream_t)stream_, net->d_layers + l0, net->Bp, net->ld, lr, (float *)nullptr);
            HIP_TRY(net, hipGetLastError());
        }
    } else if (net->b1) {
        int max_blocks = 1;
        for (const LayerDev &d : net->layers) max_blocks = std::max({max_blocks, d.b1_blocks[0], d.b1_blocks[1]});
        const bool in_lds = 4 * ((int64_t)net->max_n + 4) <= B1_MAX_LDS; // the slots past the end of a row read one place more
        const int groups = (max_blocks + LDS_WAVES - 1) / LDS_WAVES;
        // In LDS: enough workgroups to fill the chip twice, and no more of them than pay for filling their LDS.  Else as many as
        // there are groups of blocks, so that the chip works on few layers at a time and their vectors stay in L2.
        const int parts = in_lds ? std::min(groups, std::max(8, 2 * net->n_cu / net->n_layers)) : groups;
        const void *fn = in_lds ? (const void *)k_update_lm<false, true>
                         : net->b1_wide ? (const void *)k_update_lm<true, false> : (const void *)k_update_lm<false, false>;
        const size_t lds = in_lds ? (4 * ((size_t)net->max_n + 1) + 15) & ~(size_t)15 : 0;
        if (in_lds && !net->b1_attr_set) {
            HIP_TRY(net, hipFuncSetAttribute(fn, hipFuncAttributeMaxDynamicSharedMemorySize, B1_MAX_LDS));
            net->b1_attr_set = true;
        }
        for (int l0 = 0; l0 < net->n_layers; l0 += 65535) {
            const LayerDev *first = net->d_layers + l0;
            void *args[] = {(void *)&first, (void *)&lr, (void *)&net->cfg.update_bias};
            HIP_TRY(net, hipLaunchKernel(fn, dim3((unsigned)parts, 2, (unsigned)std::min(65535, net->n_layers - l0)), dim3(64 * LDS_WAVES), args, lds,
                                         (hipStream_t)stream_));
        }
    } else {
        rc = launch_update(net, 0, net->n_layers, lr, 0, nullptr, nullptr, (hipStream_t)stream_);
        if (net->layers[0].vals_t) net->vals_t_stale = true; // this kernel steps the CSR copy only
        // the copies of narrow nets follow, or (120 layers of 1024 neurons: 39 us) do so when a pass needs them
        if (!rc && !net->train[0].tab.empty()) {
            if (train_lds(net, net->B) || net->train_kept || capturing((hipStream_t)stream_)) rc = launch_train_fill(net, -1, false, (hipStream_t)stream_);
            else net->train_stale = true;
        }
    }
    if (!rc && net->long_lm) { // the copies for k_fwd_long follow, or do so when a pass needs them
        if (long_forward(net, net->B) || net->long_kept || capturing((hipStream_t)stream_)) rc = launch_long_fill(net, 0, net->n_layers, false, (hipStream_t)stream_);
        else std::fill(net->long_stale.begin(), net->long_stale.end(), 1);
    }
    if (rc) return rc;
    net->state = ST_IDLE;
    return SDNN_OK;
}

extern "C" int sdnn_weight_grad(sdnn_net *net, int32_t layer, float *d_g, float *d_gb, void *stream_)
{
    if (!net) return fail(nullptr, SDNN_EINVAL, "net is NULL");
    if (!net->cfg.training) return fail(net, SDNN_ESTATE, "net was not created for training");
    if (net->state != ST_BACKWARD)
        return fail(net, SDNN_ESTATE, "sdnn_weight_grad needs a preceding sdnn_backward");
    if (layer < 1 || layer > net->n_layers) return fail(net, SDNN_EINVAL, "layer out of range");
    if (!d_g && !d_gb) return SDNN_OK;
    if (net->grad_parts > 0) {
        // the backward sweep has already formed the gradient that sdnn_sgd_step will apply: hand out that one
        const LayerDev &d = net->layers[layer - 1];
        hipStream_t stream = (hipStream_t)stream_;
        if (d_g && net->grad_spread[layer - 1] && net->grad_parts == 1) {
            const unsigned gx = (unsigned)((((int64_t)d.nnz + TR_SPAN - 1) / TR_SPAN + 7) & ~(int64_t)7);
            hipLaunchKernelGGL(k_apply<true>, dim3(gx), dim3(TR_THREADS), 0, stream, net->d_layers + (layer - 1), 1, 0.0f);
            hipLaunchKernelGGL(k_spread_vals<true>, dim3((unsigned)(((int64_t)d.nnz + TR_CHUNK - 1) / TR_CHUNK)), dim3(TR_THREADS), 0, stream,
                               net->d_layers + (layer - 1), d_g);
        } else if (d_g && d.nnz > 0)
            hipLaunchKernelGGL(k_sum_parts, dim3((unsigned)std::min(4096, (d.nnz + 2047) / 2048)), dim3(256), 0, stream,
                               (const float *)d.G[0], net->grad_parts == 2 ? (const float *)d.G[1] : (const float *)nullptr,
                               d.t_perm, d_g, d.nnz);
        if (d_gb && d.n_out > 0)
            hipLaunchKernelGGL(k_apply_bias, dim3((unsigned)((d.n_out + 16 * WAVES_PER_BLOCK - 1) / (16 * WAVES_PER_BLOCK)), 1u),
                               dim3(BLOCK_THREADS), 0, stream, net->d_layers + (layer - 1), net->Bp, net->ld, 0.0f, d_gb);
        HIP_TRY(net, hipGetLastError());
        return SDNN_OK;
    }
    return launch_update(net, layer - 1, 1, 0.0f, 1, d_g, d_gb, (hipStream_t)stream_);
}

static int copy_dd(sdnn_net *net, void *dst, const void *src, size_t bytes, void *stream_)
{
    if (bytes) HIP_TRY(net, hipMemcpyAsync(dst, src, bytes, hipMemcpyDeviceToDevice, (hipStream_t)stream_));
    return SDNN_OK;
}

extern "C" int sdnn_get_activation(sdnn_net *net, int32_t layer, float *d_dst, void *stream_)
{
    if (!net) return fail(nullptr, SDNN_EINVAL, "net is NULL");
    if (!net->cfg.training) return fail(net, SDNN_ESTATE, "activations are kept in training mode only");
    if (net->state == ST_IDLE && net->B == 0) return fail(net, SDNN_ESTATE, "no forward pass yet");
    if (layer < 0 || layer > net->n_layers) return fail(net, SDNN_EINVAL, "layer out of range");
    if (!d_dst) return fail(net, SDNN_EINVAL, "d_dst is NULL");
    const float *src = layer == 0 ? net->d_x0 : net->layers[layer - 1].X;
    const size_t n = layer == 0 ? net->layers[0].n_in : net->layers[layer - 1].n_out;
    return launch_copy_rows(net, src, net->ld, d_dst, net->B, (int)n, net->B, net->B, (hipStream_t)stream_);
}

extern "C" int sdnn_get_delta(sdnn_net *net, int32_t layer, float *d_dst, void *stream_)
{
    if (!net) return fail(nullptr, SDNN_EINVAL, "net is NULL");
    if (!net->cfg.training) return fail(net, SDNN_ESTATE, "deltas are kept in training mode only");
    if (net->state != ST_BACKWARD) return fail(net, SDNN_ESTATE, "no backward pass to read");
    if (layer < 1 || layer > net->n_layers) return fail(net, SDNN_EINVAL, "layer out of range");
    if (!d_dst) return fail(net, SDNN_EINVAL, "d_dst is NULL");
    return launch_copy_rows(net, net->layers[layer - 1].D, net->ld, d_dst, net->B, net->layers[layer - 1].n_out, net->B, net->B,
                            (hipStream_t)stream_);
}

extern "C" int sdnn_get_weights(sdnn_net *net, int32_t layer, float *d_values, float *d_bias, void *stream_)
{
    if (!net) return fail(nullptr, SDNN_EINVAL, "net is NULL");
    if (layer < 1 || layer > net->n_layers) return fail(net, SDNN_EINVAL, "layer out of range");
    const LayerDev &d = net->layers[layer - 1];
    int rc = SDNN_OK;
    if (d_values && net->b1) { // the values that are stepped are those of the lane-major copy
        if (d.nnz > 0) {
            const dim3 grid((unsigned)d.b1_blocks[0], fill_parts(net->max_len[0][layer - 1]));
            if (net->b1_wide) hipLaunchKernelGGL(k_b1_values<true>, grid, dim3(64), 0, (hipStream_t)stream_, net->d_layers + (layer - 1), d_values);
            else hipLaunchKernelGGL(k_b1_values<false>, grid, dim3(64), 0, (hipStream_t)stream_, net->d_layers + (layer - 1), d_values);
            HIP_TRY(net, hipGetLastError());
        }
    } else if (d_values) {
        rc = copy_dd(net, d_values, d.vals, 4 * (size_t)d.nnz, stream_);
    }
    if (!rc && d_bias) rc = copy_dd(net, d_bias, d.bias, 4 * (size_t)d.n_out, stream_);
    return rc;
}

extern "C" int sdnn_set_weights(sdnn_net *net, int32_t layer, const float *d_values,
                                const float *d_bias, void *stream_)
{
    if (!net) return fail(nullptr, SDNN_EINVAL, "net is NULL");
    if (layer < 1 || layer > net->n_layers) return fail(net, SDNN_EINVAL, "layer out of range");
    const LayerDev &d = net->layers[layer - 1];
    int rc = SDNN_OK;
    if (d_values) {
        rc = copy_dd(net, d.vals, d_values, 4 * (size_t)d.nnz, stream_);
        if (!rc && d.vals_t && d.nnz > 0) { // the transposed-order copy follows at once
            hipLaunchKernelGGL(k_refresh_vals_t, dim3((unsigned)std::min(4096, (d.nnz + 2047) / 2048), 1u), dim3(256), 0,
                               (hipStream_t)stream_, net->d_layers + (layer - 1));
            HIP_TRY(net, hipGetLastError());
        }
    }
    if (!rc && d_bias) {
        rc = copy_dd(net, d.bias, d_bias, 4 * (size_t)d.n_out, stream_);
        if (layer > 1) net->bias_nonpos = false; // device data: its signs are not inspected
    }
    if (!rc && d_values && net->b1) rc = launch_b1_fill(net, layer - 1, 0, (hipStream_t)stream_);
    if (!rc && d_values && net->long_lm) { // its copy follows, or does so when a pass needs it (8192 rows of 820 entries: 74 us without, 94 with it)
        if (net->long_kept || capturing((hipStream_t)stream_)) rc = launch_long_fill(net, layer - 1, 1, false, (hipStream_t)stream_);
        else net->long_stale[layer - 1] = 1;
    }
    if (!rc && (d_values || d_bias) && net->lm) // keep the lane-major copy current
        rc = launch_lm_fill(net, layer - 1, nullptr, 0, (hipStream_t)stream_);
    if (!rc && (d_values || d_bias) && !net->train[0].tab.empty()) { // the first layer's copies follow at once, all others' in one go with the next pass
        if (!net->train_replaced || net->train_kept || capturing((hipStream_t)stream_)) rc = launch_train_fill(net, layer - 1, false, (hipStream_t)stream_);
        else net->train_stale = true;
        net->train_replaced = true;
    }
    if (!rc && (d_values || d_bias) && !net->pan.empty()) rc = launch_pan_fill(net, layer - 1, (hipStream_t)stream_);
    return rc;
}

extern "C" int sdnn_layer_shape(const sdnn_net *net, int32_t layer, int32_t *n_out, int32_t *n_in,
                                int64_t *nnz)
{
    if (!net) return fail(nullptr, SDNN_EINVAL, "net is NULL");
    if (layer < 1 || layer > net->n_layers) return fail(nullptr, SDNN_EINVAL, "layer out of range");
    const LayerDev &d = net->layers[layer - 1];
    if (n_out) *n_out = d.n_out;
    if (n_in) *n_in = d.n_in;
    if (nnz) *nnz = d.nnz;
    return SDNN_OK;
}

extern "C" int sdnn_mse_dloss(const float *d_XL, const float *d_Y, int32_t n, int32_t B,
                              float *d_out, void *stream_)
{
    if (!d_XL || !d_Y || !d_out) return fail(nullptr, SDNN_EINVAL, "NULL pointer");
    if (n < 0 || B < 1) return fail(nullptr, SDNN_EINVAL, "bad size");
    const size_t cnt = (size_t)n * B;
    if (!cnt) return SDNN_OK;
    hipLaunchKernelGGL(k_mse_dloss, dim3(ew_blocks(cnt)), dim3(256), 0, (hipStream_t)stream_, d_XL,
                       d_Y, d_out, cnt, (double)B);
    HIP_TRY(nullptr, hipGetLastError());
    return SDNN_OK;
}

extern "C" int sdnn_softmax_ce_dloss(const float *d_XL, const int32_t *d_labels, int32_t n,
                                     int32_t B, int32_t n_classes, float *d_out, void *stream_)
{
    if (!d_XL || !d_labels || !d_out) return fail(nullptr, SDNN_EINVAL, "NULL pointer");
    if (n < 1 || B < 1 || n_classes < 1 || n_classes > n) return fail(nullptr, SDNN_EINVAL, "bad size");
    const size_t cnt = std::max((size_t)(n - n_classes) * B, (size_t)B);
    hipLaunchKernelGGL(k_softmax_ce_dloss, dim3(ew_blocks(cnt)), dim3(256), 0, (hipStream_t)stream_,
                       d_XL, d_labels, d_out, n, B, n_classes);
    HIP_TRY(nullptr, hipGetLastError());
    return SDNN_OK;
}

extern "C" int sdnn_gather_probe(const float *d_table, int32_t table_rows, int32_t v, const int32_t *d_idx,
                                 int32_t n_waves, int32_t per_wave, float *d_out, void *stream_)
{
    if (!d_table || !d_idx || !d_out) return fail(nullptr, SDNN_EINVAL, "NULL pointer");
    if (v != 1 && v != 2 && v != 4) return fail(nullptr, SDNN_EINVAL, "v must be 1, 2 or 4");
    if (table_rows < 1 || n_waves < WAVES_PER_BLOCK || n_waves % WAVES_PER_BLOCK || per_wave < 8 || per_wave % 8)
        return fail(nullptr, SDNN_EINVAL, "table_rows >= 1, n_waves a positive multiple of %d, per_wave a positive multiple of 8",
                    WAVES_PER_BLOCK);
    const size_t bytes = (size_t)table_rows * 256 * (size_t)v;
    if (bytes >= ((size_t)1 << 32)) return fail(nullptr, SDNN_EINVAL, "table of %zu bytes exceeds 4 GiB", bytes);
    const dim3 grid((unsigned)(n_waves / WAVES_PER_BLOCK)), block(BLOCK_THREADS);
    hipStream_t stream = (hipStream_t)stream_;
    if (v == 4) hipLaunchKernelGGL(k_gather_probe<4>, grid, block, 0, stream, d_idx, d_table, bytes, per_wave, d_out);
    else if (v == 2) hipLaunchKernelGGL(k_gather_probe<2>, grid, block, 0, stream, d_idx, d_table, bytes, per_wave, d_out);
    else hipLaunchKernelGGL(k_gather_probe<1>, grid, block, 0, stream, d_idx, d_table, bytes, per_wave, d_out);
    HIP_TRY(nullptr, hipGetLastError());
    return SDNN_OK;
}
